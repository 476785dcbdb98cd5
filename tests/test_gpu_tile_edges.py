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


# fp32: the small tiles (few workgroups) and the large ones (64 heads of 260
# rows for the forward and the rows' products, the last two cases for the
# others), rows and blocks of 16 short of, at and past their edges, 1 to 8 waves
# sharing a block's loop, dense heads with and without a window
@pytest.mark.parametrize("kw", [
    dict(seq_len=15, k=7, heads=1, dense_heads=1, d_head=64),
    dict(seq_len=33, k=17, heads=2, dense_heads=1, d_model=128, d_head=32, rope=True),
    dict(seq_len=65, k=33, heads=2, dense_heads=2, d_model=192, d_head=64, window=16),
    dict(seq_len=129, k=65, heads=3, dense_heads=1, d_head=64, causal=False),
    dict(seq_len=150, k=130, heads=64, dense_heads=0, d_head=32, batch=2),
    dict(seq_len=150, k=130, heads=64, dense_heads=0, d_head=64, batch=2, rope=True),
    dict(seq_len=300, k=3, heads=1, dense_heads=9, d_model=256, d_head=64, window=100),
    # the large tiles of the weight gradients with the router column (256 heads of one tile) and of the dense heads
    dict(seq_len=45, k=20, heads=256, dense_heads=0, d_model=64, d_head=64, batch=2),
    dict(seq_len=1030, k=3, heads=1, dense_heads=4, d_model=512, d_head=64, batch=4),
])
def test_f32_tiles(orc, kw):
    _check(orc, wl.small(dtype="f32", seed=77, **kw))


# the weight gradients' row tables and tiles: rows per head short of, at and
# past a chunk of 32 or 64, one to many chunks, the 64- and the 128-column tiles
# (128 heads of d 256; with 1250 rows, 64 columns again, with 2100, 128), two and
# three tiles per workgroup of 1, 2, 3 or 5 chunks with a shorter last
# workgroup (from 208 heads on), dense row ranges
@pytest.mark.parametrize("kw", [
    dict(batch=1, seq_len=150, k=133, heads=2, d_model=192, d_head=64),
    dict(batch=3, seq_len=90, k=64, heads=3, d_model=320, d_head=64),
    dict(batch=2, seq_len=150, k=65, heads=5, d_model=128, d_head=32),
    dict(batch=1, seq_len=160, k=160, heads=128, d_model=256, d_head=64),
    dict(batch=2, seq_len=100, k=67, heads=130, d_model=256, d_head=64),
    dict(batch=5, seq_len=260, k=250, heads=128, d_model=256, d_head=64),
    dict(batch=7, seq_len=310, k=300, heads=128, d_model=256, d_head=64),
    dict(batch=1, seq_len=50, k=20, heads=208, d_model=320, d_head=32),
    dict(batch=1, seq_len=120, k=97, heads=208, d_model=320, d_head=32),
    dict(batch=1, seq_len=170, k=161, heads=208, d_model=320, d_head=32),
    dict(batch=1, seq_len=60, k=33, heads=256, d_model=448, d_head=32),
    dict(batch=1, seq_len=140, k=133, heads=256, d_model=640, d_head=64),
    dict(batch=1, seq_len=33, k=5, heads=1, dense_heads=3, d_model=128, d_head=64),
    dict(batch=3, seq_len=171, k=5, heads=1, dense_heads=2, d_model=64, d_head=32),
])
def test_weight_gradient_tiles(orc, kw):
    _check(orc, wl.small(seed=31, **kw))


# the flash kernel's blocks of 64 and of 128 queries: short of, at and past a
# block and a key tile, 256 blocks and more (whole heads per XCD, full and
# partial rounds of its CUs), more than 512 blocks of 128, a head too short for
# a second block, MoSA heads
@pytest.mark.parametrize("kw", [
    dict(batch=1, seq_len=129, dense_heads=3),
    dict(batch=1, seq_len=512, dense_heads=1, causal=False),
    dict(batch=1, seq_len=513, dense_heads=3),
    dict(batch=8, seq_len=449, dense_heads=8),
    dict(batch=4, seq_len=520, dense_heads=8),
    dict(batch=4, seq_len=520, dense_heads=8, causal=False),
    dict(batch=5, seq_len=1000, dense_heads=8),
    dict(batch=9, seq_len=1024, dense_heads=8),
    dict(batch=2, seq_len=400, dense_heads=0, heads=16, k=193),
])
def test_flash_blocks(orc, kw):
    w = wl.small(**{**dict(d_model=64, d_head=64, heads=1, k=4, backward=False, seed=63), **kw})
    check_forward(orc, w, wl.make_inputs(w))
