"""GEMM tiles of more than 128 tokens at the edges of their row tiles, column
tiles and k-loops, against float64: the MFMA-bound 256-row tiles (test_*_ring*;
the host test of the plans pins that these calls take them) and the smaller
ones that small matrices take."""
import pytest
import torch

import oracle
from paper_2608_01891_amd import aflex, synth
from tests.parity import check_rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# 256-row tiles with one K split (bf16 output). Rows: one short of and one past a
# 32-row block (instances of 5 to 8 blocks in one tile), two tiles of 5 and 4 blocks,
# nine and ten tiles whose last holds 72 rows and one (3 and 2 blocks). k: one, two
# and three k-steps, one turn of the ring and past it. Columns: a quarter, a half, three
# quarters and whole tiles at the end.
RING_LINEAR = [(129, 64, 41024), (160, 128, 41088), (161, 192, 41152), (193, 64, 41216), (256, 192, 41024),
               (257, 320, 23040), (300, 64, 25600), (2120, 128, 4672), (2305, 64, 4160), (2305, 192, 4352),
               (2305, 320, 5120), (513, 448, 13888), (385, 960, 20544)]
# ... and with several (fp32 partials)
RING_LINEAR_SPLIT = [(2305, 4096, 2560), (1400, 6144, 3072), (300, 8192, 5376), (256, 7168, 9216), (257, 8192, 5120)]


def _linear(T, K, N):
    x = synth.normal_tensor(31, 1, (T, K))
    w = synth.normal_tensor(31, 2, (N, K), synth.WEIGHT_SIGMA)
    y = torch.full((T + 1, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    aflex.linear(x.to(DEV), w.to(DEV), y=y[:T])
    check_rows(y[:T].cpu(), x.double() @ w.double().t(), what=f"linear {T}x{K}x{N}")
    assert torch.isnan(y[T]).all()  # nothing past the last row


@pytest.mark.parametrize("T,K,N", RING_LINEAR + RING_LINEAR_SPLIT)
def test_linear_ring(gpu_lib, T, K, N):
    _linear(T, K, N)


# 64- and 128-row tiles: rows one short of and one past a 16-row block and a 128- and
# 256-row tile; k: one, two and three k-steps and more; columns: a quarter, three
# quarters and one and a quarter tiles of 256
@pytest.mark.parametrize("T,K,N", [(129, 64, 64), (143, 128, 192), (145, 192, 320), (255, 256, 256), (256, 320, 448),
                                   (257, 384, 64), (300, 640, 256), (513, 704, 320), (2305, 192, 512),
                                   (2305, 2048, 320)])
def test_linear_tile_edges(gpu_lib, T, K, N):
    _linear(T, K, N)


def _swiglu(T, H, I):
    x, w, _ = synth.custom_ffn(32, T, H, I)
    y = aflex.ffn_swiglu(x.to(DEV), w.to(DEV)).cpu()
    check_rows(y, oracle.swiglu_ffn(x, w.w_gate, w.w_up, w.w_down), what=f"swiglu {T}x{H}x{I}")


RING_SWIGLU = [(129, 64, 20544), (300, 64, 20544), (257, 448, 10304), (700, 128, 10304), (192, 192, 20608)]


@pytest.mark.parametrize("T,H,I", RING_SWIGLU)
def test_swiglu_ring(gpu_lib, T, H, I):
    _swiglu(T, H, I)


@pytest.mark.parametrize("T,H,I", [(129, 64, 64), (257, 192, 320), (300, 448, 128), (769, 128, 1088)])
def test_swiglu_tile_edges(gpu_lib, T, H, I):
    _swiglu(T, H, I)


def _moe(T, H, I, E, k):
    x, w, logits = synth.custom_ffn(33, T, H, I, E=E)
    logits[:, 0] += 0.7  # an uneven load
    y = aflex.moe_ffn(x.to(DEV), w.to(DEV), logits.to(DEV), k).cpu()
    ref, _, _ = oracle.moe_ffn(x, logits, w.w_gate, w.w_up, w.w_down, k)
    check_rows(y, ref, what=f"moe {T} E={E} k={k}")


# experts of one, two, two to four and four to eight row tiles, whose rows are split evenly
RING_MOE = [(290, 64, 7232, 2, 1), (400, 64, 14400, 2, 2), (650, 128, 3712, 4, 2), (2700, 64, 1216, 2, 1)]


@pytest.mark.parametrize("T,H,I,E,k", RING_MOE)
def test_moe_ring(gpu_lib, T, H, I, E, k):
    _moe(T, H, I, E, k)


@pytest.mark.parametrize("T,H,I,E,k", [(290, 64, 64, 2, 1), (400, 192, 128, 2, 2), (650, 128, 192, 4, 2),
                                         (2700, 64, 1088, 2, 1)])
def test_moe_even_row_tiles(gpu_lib, T, H, I, E, k):
    """Experts of one to more than eight 64- and 128-row tiles."""
    _moe(T, H, I, E, k)


# (tokens, attention columns, H): the projection of a microbatch in 256-row tiles and one
# K split, which adds the residual in the GEMM's own epilogue
RING_RESIDUAL = [(700, 64, 13888), (513, 128, 14016)]


@pytest.mark.parametrize("T,K,H", RING_RESIDUAL)
def test_residual_ring(gpu_lib, T, K, H):
    """A decode layer step whose FFN adds nothing (zero down weights), so that y is
    the projection plus the layer input."""
    a = synth.custom_attention(34, T, K // 64, 1, 64, [1] * T, ctx_hi=16)  # one token each: attention returns its V row
    _, w, _ = synth.custom_ffn(34, 1, H, 64, E=2)
    w.w_down = torch.zeros_like(w.w_down)
    layer = synth.make_layer(34, T, K // 64, 1, 64, H, 2)
    y = aflex.af_layer_step(a.to(DEV), w.to(DEV), layer.to(DEV), 1, [T]).cpu()
    o = layer.v_new.double().view(T, 1, 64).expand(T, K // 64, 64).reshape(T, K)
    check_rows(y, layer.x_in.double() + o @ layer.w_o.double().t(), what=f"residual {T}x{K}x{H}")
