"""Packed KV-cache write: the exchange of V rows between threads (up to 256
threads per work-group, whole groups of 16) and the direct stores beside it, at
partial first and last blocks, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_01891_amd import aflex, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (Hkv, D): a lone half group, whole groups, a trailing half group, the most
# threads of the exchange, and more (direct stores)
@pytest.mark.parametrize("Hkv,D", [(1, 64), (2, 64), (5, 64), (1, 128), (3, 128), (16, 128), (17, 128), (33, 64)])
def test_kv_write_bitwise(gpu_lib, Hkv, D):
    new, ctx = [16, 1, 40, 0, 31, 17], [16, 1, 53, 20, 64, 49]  # whole, partial first, last and both
    a = synth.custom_attention(7, len(ctx), Hkv, Hkv, D, ctx, ctx_hi=80)
    T = sum(new)
    k, v = synth.normal_tensor(7, 21, (T, Hkv, D)), synth.normal_tensor(7, 22, (T, Hkv, D))
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(new)]).astype(np.int32))
    rk, rv = oracle.kv_write(a.k_cache, a.v_cache, a.block_table, a.context_lens, cu, k, v)
    ad = a.to(DEV)
    aflex.kv_write(ad, k.to(DEV), v.to(DEV), cu.to(DEV), max_seqlen=max(new))
    assert torch.equal(ad.k_cache.cpu(), rk) and torch.equal(ad.v_cache.cpu(), rv)


# fewer than 16 new tokens per sequence and more than 256 threads: only a block's own rows are loaded
@pytest.mark.parametrize("Hkv,D", [(17, 128), (33, 64), (64, 128)])
@pytest.mark.parametrize("max_seqlen", [15, 16])  # (16: the general form on the same tokens)
def test_kv_write_few_tokens_bitwise(gpu_lib, Hkv, D, max_seqlen):
    new, ctx = [1, 1, 15, 0, 15, 7, 1], [1, 16, 15, 20, 33, 23, 17]  # first, last and both sides of a block's edge
    a = synth.custom_attention(8, len(ctx), Hkv, Hkv, D, ctx, ctx_hi=48)
    T = sum(new)
    k, v = synth.normal_tensor(8, 21, (T, Hkv, D)), synth.normal_tensor(8, 22, (T, Hkv, D))
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(new)]).astype(np.int32))
    rk, rv = oracle.kv_write(a.k_cache, a.v_cache, a.block_table, a.context_lens, cu, k, v)
    ad = a.to(DEV)
    aflex.kv_write(ad, k.to(DEV), v.to(DEV), cu.to(DEV), max_seqlen=max_seqlen)
    assert torch.equal(ad.k_cache.cpu(), rk) and torch.equal(ad.v_cache.cpu(), rv)
