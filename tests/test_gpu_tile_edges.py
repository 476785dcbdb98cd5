"""GPU parity at the edges of the tiled kernels: contraction lengths around the
pipelines' stage and unroll counts, and row counts around their tiles, forward
and backward against the oracle (the bars of test_gpu_forward.py)."""
import pytest

import workloads as wl
from test_gpu_backward import check_backward
from test_gpu_forward import check_forward

pytestmark = pytest.mark.gpu


def _check(orc, w):
    inp = wl.make_inputs(w, with_grad=True)
    check_forward(orc, w, inp)
    if w.batch * w.k == 1:
        return  # one row attends to itself: dS = 0 exactly, and dW^Q, dW^K are bf16 rounding residue alone
    check_backward(orc, w, inp, row_bar_mosa_weights=w.batch * w.k >= 8)


# d / 32 or d / 64 chunks: fewer than the stages, one more, and every remainder
# of the unrolled loop
@pytest.mark.parametrize("d", [64, 128, 192, 256, 320, 384, 448])
@pytest.mark.parametrize("dh", [32, 64])
def test_contraction_lengths(orc, d, dh):
    _check(orc, wl.small(seq_len=72, d_model=d, d_head=dh, heads=2, dense_heads=1, k=32, seed=d))


# rows per head (batch * k): 1, one short of and one past a 64- and a 128-row
# tile; k: the fused attention's group sizes and others
@pytest.mark.parametrize("batch,k", [(1, 1), (3, 16), (5, 16), (9, 16), (1, 32), (5, 32), (1, 64), (3, 64), (1, 128),
                                     (2, 128), (1, 63), (1, 127), (1, 129), (3, 43)])
@pytest.mark.parametrize("rope,causal", [(True, True), (False, False)])
def test_row_tiles(orc, batch, k, rope, causal):
    _check(orc, wl.small(batch=batch, seq_len=131, d_model=128, d_head=64 if k % 2 else 32, heads=3, k=k, rope=rope,
                         causal=causal, seed=100 * batch + k))
    if k % 16 == 0:
        _check(orc, wl.small(batch=batch, seq_len=131, d_model=64, d_head=64, heads=2, k=k, rope=rope, causal=causal,
                             seed=100 * batch + k + 1))
