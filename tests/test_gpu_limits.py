"""GPU parity at the edges of the supported range: the longest sequence,
the widest model, many heads, ragged group and tile sizes, k = T, fp32
beyond one tile, local heads over many tiles.  Same bars as the other
parity tests (indices bit-exact, relative errors per tensor)."""
import pytest
import torch

import workloads as wl
from paper_2505_00315_amd import mosa
from test_gpu_variants import check_backward, check_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(batch=1, seq_len=16384, d_model=64, heads=2, d_head=32, k=64),       # longest T
    dict(batch=1, seq_len=16384, d_model=64, heads=1, d_head=64, k=2048),     # longest T, k > 128
    dict(batch=1, seq_len=64, d_model=2048, heads=2, d_head=64, k=16),        # widest d
    dict(batch=2, seq_len=128, d_model=64, heads=300, d_head=32, k=8),        # heads past 4 x 64
    dict(batch=2, seq_len=77, d_model=64, heads=2, d_head=32, k=77),          # k = T, ragged T
    dict(batch=5, seq_len=100, d_model=128, heads=3, d_head=64, k=48),        # group not dividing 128
    dict(batch=1, seq_len=300, d_model=64, heads=2, d_head=32, k=200, dtype="f32"),
    dict(batch=1, seq_len=400, d_model=64, heads=2, d_head=64, k=300, causal=False),
    dict(batch=1, seq_len=2048, d_model=64, heads=1, d_head=32, k=32, dense_heads=1, window=200),
])
def test_limits(orc, kw):
    w = wl.small(**kw)
    check_forward(orc, w)
    check_backward(orc, w)


def test_f32_attention_past_one_launch():
    """fp32 dense heads of 8193 x 64 (b, h) pairs of 113 rows: the attention
    backward needs just over 2^32 threads, so two launches.  Y and dX of a batch
    element do not depend on the others, so its first and last elements equal
    those of calls on a quarter of the batch bit for bit (the same kernels, one
    launch)."""
    B, T, d, dh, Hd = 8193, 113, 64, 32, 64
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of free GPU memory")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def rand(*size, std=1.0):
        return torch.randn(size, generator=gen, device="cuda") * std

    X, dY = rand(B, T, d), rand(B, T, d)
    w = {n: rand(Hd, d, dh, std=d ** -0.5) for n in ("Wq_d", "Wk_d", "Wv_d")}
    w["Wo_d"] = rand(Hd, dh, d, std=d ** -0.5)

    def step(X, dY):
        print(f"[case] batch {X.shape[0]}", flush=True)
        shape = mosa.make_shape(X.shape[0], T, d, 0, dh, 0, True, Hd, "f32")
        Y, saved, scratch = mosa.forward(shape, X, w)
        grads = {"d" + n: torch.empty_like(t) for n, t in w.items()}
        dX = mosa.backward(shape, X, w, dY, saved, grads, scratch=scratch)
        torch.cuda.synchronize()
        return Y, dX

    Y, dX = step(X, dY)
    for part in (slice(0, 2048), slice(B - 2048, B)):
        y, dx = step(X[part].contiguous(), dY[part].contiguous())
        assert torch.equal(Y[part], y) and torch.equal(dX[part], dx)
    del Y, dX
    torch.cuda.empty_cache()
