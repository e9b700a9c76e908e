"""The append of 32 or more new tokens, whose workgroups take whole cache
blocks: bit for bit the oracle's caches at starts and ends inside blocks,
contexts shorter than the new tokens, and a block id outside the pool."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from paper_2405_11143_amd import pda_append_kv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,D", [(32, 8, 128), (8, 2, 64), (16, 1, 128)], ids=str)
@pytest.mark.parametrize("n", [31, 32, 33, 47, 48, 100])
def test_append_bit_exact(Hq, Hkv, D, n):
    dev = torch.device("cuda:0")
    lens = [0, 1, 15, 16, 17, n - 1, n, n + 1, n + 15, n + 16, n + 17, 333, -3, 1000]
    st = W.custom_structure(len(lens), Hq, Hkv, D, lens, seed=40 + n)
    _, k, v = W.fill_values(st, dev, fill="nan")
    kn, vn = W.fill_new_kv(st, n, dev)
    table = st.block_table.copy()
    table[11, (333 - 1) // 16] = st.num_blocks + 5  # its tokens are skipped
    k_ref, v_ref = oracle.append(W.bf16_bits(kn), W.bf16_bits(vn), st.block_table, st.context_lens, W.bf16_bits(k),
                                 W.bf16_bits(v))
    skipped = int(st.block_table[11, (333 - 1) // 16])
    k_ref[skipped], v_ref[skipped] = W.bf16_bits(k)[skipped], W.bf16_bits(v)[skipped]
    pda_append_kv(kn, vn, torch.from_numpy(table).to(dev), torch.from_numpy(st.context_lens).to(dev), k, v,
                  max_context_len=st.max_context_len, num_q_heads=Hq)
    torch.cuda.synchronize()
    assert np.array_equal(W.bf16_bits(k), k_ref), "K cache"
    assert np.array_equal(W.bf16_bits(v), v_ref), "V cache"
