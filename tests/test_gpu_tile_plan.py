"""GEMM tile plans: each tile height at its edges, with weights small enough to
stay cached (ordinary loads) and larger ones (non-temporal loads), against
float64."""
import functools

import pytest
import torch

import oracle
from paper_2608_01891_amd import aflex, synth
from tests.parity import check_rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@functools.lru_cache(maxsize=1)
def _linear(K, N):
    return (synth.normal_tensor(51, 1, (300, K)).to(DEV),
            synth.normal_tensor(51, 2, (N, K), synth.WEIGHT_SIGMA).to(DEV))


@functools.lru_cache(maxsize=1)
def _ffn(H, I, E):
    x, w, logits = synth.custom_ffn(52, 512, H, I, E=E)
    return x.to(DEV), w.to(DEV), None if logits is None else logits.to(DEV)


def _swiglu64(x, w):
    g, u = x @ w.w_gate.double().t(), x @ w.w_up.double().t()
    return (g / (1.0 + torch.exp(-g)) * u) @ w.w_down.double().t()


# Rows per tile of each call (the host test of the plans pins them): 168 MB of
# weights, past what is kept, and 4 MB, few work-groups
LINEAR_T = [1, 32, 33, 64, 65, 128, 129, 256, 257]
LINEAR_ROWS = {(8192, 10304): [32, 32, 128, 128, 128, 128, 256, 256, 256],
               (1024, 1984): [32, 32, 64, 64, 64, 64, 64, 64, 64]}


@pytest.mark.parametrize("T", LINEAR_T)
@pytest.mark.parametrize("K,N", LINEAR_ROWS)
def test_linear(gpu_lib, T, K, N):
    x, w = _linear(K, N)
    x = x[:T]
    y = torch.full((T + 1, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    aflex.linear(x, w, y=y[:T])
    check_rows(y[:T].cpu(), (x.double() @ w.double().t()).cpu(), what=f"linear {T}x{K}x{N}")
    assert torch.isnan(y[T]).all()


# first GEMMs of few (112, at 256 rows) and of enough work-groups; 176, 352 and 2 MB
SWIGLU_T = [31, 33, 64, 100, 129, 256, 290]
SWIGLU_ROWS = {(2048, 14336): [32, 64, 64, 128, 128, 128, 256], (2752, 21376): [32, 128, 128, 128, 256, 256, 256],
               (576, 640): [32, 64, 64, 64, 64, 64, 64]}


@pytest.mark.parametrize("T", SWIGLU_T)
@pytest.mark.parametrize("H,I", SWIGLU_ROWS)
def test_swiglu(gpu_lib, T, H, I):
    x, w, _ = _ffn(H, I, 0)
    x = x[:T]
    check_rows(aflex.ffn_swiglu(x, w).cpu(), _swiglu64(x.double(), w).cpu(), what=f"swiglu {T}x{H}x{I}")


# experts over and under one tile; 264 and 2 MB
MOE_T = [30, 80, 190, 200, 380, 500]
MOE_ROWS = {(2048, 5376): [32, 64, 128, 256, 256, 256], (256, 320): [32, 64, 64, 64, 64, 64]}


@pytest.mark.parametrize("T", MOE_T)
@pytest.mark.parametrize("H,I", MOE_ROWS)
def test_moe(gpu_lib, T, H, I):
    E, k = 4, 2
    x, w, logits = _ffn(H, I, E)
    x, logits = x[:T], logits[:T].contiguous()
    y = aflex.moe_ffn(x, w, logits, k)
    top, ids = torch.sort(logits.double(), dim=-1, descending=True, stable=True)
    ids, p = ids[:, :k], torch.softmax(top[:, :k], -1)
    ref = torch.zeros(T, H, dtype=torch.float64, device=DEV)
    for e in range(E):
        t, j = torch.nonzero(ids == e, as_tuple=True)
        one = type("W", (), {"w_gate": w.w_gate[e], "w_up": w.w_up[e], "w_down": w.w_down[e]})
        ref[t] += p[t, j, None] * _swiglu64(x[t].double(), one)
    check_rows(y.cpu(), ref.cpu(), what=f"moe {T}x{H}x{I}")


# 320-row tiles: experts of one tile and a few rows more, and of two tiles
MOE_ONE_ROUND = [(1000, 128, 3584, 8, 2), (1100, 64, 3520, 8, 2), (1120, 128, 4096, 4, 2), (300, 64, 16384, 2, 2)]


@pytest.mark.parametrize("T,H,I,E,k", MOE_ONE_ROUND)
@pytest.mark.parametrize("skew", [0.0, 0.5])
def test_moe_320_row_tiles(gpu_lib, T, H, I, E, k, skew):
    x, w, logits = synth.custom_ffn(54, T, H, I, E=E)
    logits[:, E - 1] += skew  # a crowded last expert: past its tile, or into a third one
    y = aflex.moe_ffn(x.to(DEV), w.to(DEV), logits.to(DEV), k).cpu()
    ref, _, _ = oracle.moe_ffn(x, logits, w.w_gate, w.w_up, w.w_down, k)
    check_rows(y, ref, what=f"moe {T}x{H}x{I} E={E} k={k}")
