"""The MFMA-bound GEMM tiles (more than 128 rows) at the edges of their row
tiles, column tiles and k-loops, against float64."""
import pytest
import torch

import oracle
from paper_2608_01891_amd import aflex, synth
from tests.parity import check_rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# rows: one short of and one past a 16-row block and a 128- and 256-row tile, an
# even split over three tiles; k: one, two and three k-steps and past one turn
# of the ring; columns: a quarter, three quarters and one and a quarter tiles
LINEAR = [(129, 64, 64), (143, 128, 192), (145, 192, 320), (255, 256, 256), (256, 320, 448), (257, 384, 64),
          (300, 640, 256), (513, 704, 320), (2305, 192, 512),
          (2305, 2048, 320)]  # ten row tiles (a group of 8 and one of 2) in several k-splits


@pytest.mark.parametrize("T,K,N", LINEAR)
def test_linear_tile_edges(gpu_lib, T, K, N):
    x = synth.normal_tensor(31, 1, (T, K))
    w = synth.normal_tensor(31, 2, (N, K), synth.WEIGHT_SIGMA)
    y = torch.full((T + 1, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    aflex.linear(x.to(DEV), w.to(DEV), y=y[:T])
    check_rows(y[:T].cpu(), x.double() @ w.double().t(), what=f"linear {T}x{K}x{N}")
    assert torch.isnan(y[T]).all()  # nothing past the last row


@pytest.mark.parametrize("T,H,I", [(129, 64, 64), (257, 192, 320), (300, 448, 128), (769, 128, 1088)])
def test_swiglu_tile_edges(gpu_lib, T, H, I):
    x, w, _ = synth.custom_ffn(32, T, H, I)
    y = aflex.ffn_swiglu(x.to(DEV), w.to(DEV)).cpu()
    check_rows(y, oracle.swiglu_ffn(x, w.w_gate, w.w_up, w.w_down), what=f"swiglu {T}x{H}x{I}")


@pytest.mark.parametrize("T,H,I,E,k", [(290, 64, 64, 2, 1), (400, 192, 128, 2, 2), (650, 128, 192, 4, 2),
                                         (2700, 64, 1088, 2, 1)])
def test_moe_even_row_tiles(gpu_lib, T, H, I, E, k):
    """Experts of one, two, three and more than eight row tiles, whose rows are split evenly."""
    x, w, logits = synth.custom_ffn(33, T, H, I, E=E)
    logits[:, 0] += 0.7  # an uneven load
    y = aflex.moe_ffn(x.to(DEV), w.to(DEV), logits.to(DEV), k).cpu()
    ref, _, _ = oracle.moe_ffn(x, logits, w.w_gate, w.w_up, w.w_down, k)
    check_rows(y, ref, what=f"moe {T} E={E} k={k}")
