"""GPU parity of the merge pass at the edges of its slot handling: slots
per row around 4 and the 8 loaded ahead, the 64 states of a wavefront and the load
rounds in between, at both head dims, without and with a shared prefix (whose
slots come first and are followed by unused ones)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from parity_common import THREADS, check
from paper_2405_11143_amd import pda_decode, pda_decode_shared_prefix

pytestmark = pytest.mark.gpu

TP = 16  # one partition per block


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("parts", [2, 4, 5, 8, 9, 16, 17, 63, 64, 65, 72, 73, 129])
@pytest.mark.parametrize("prefix", [0, 1, 9, 70])
def test_slot_edges(dev, D, parts, prefix):
    own = sorted({1, 2, parts // 2 + 1, parts - 1, parts})
    lens = [TP * (prefix + k) - (7 if k % 2 else 0) for k in own]
    if prefix:
        st = W.custom_shared_structure(8, 2, D, [(TP * prefix, lens)], [TP * k for k in own], seed=800 + parts)
    else:
        st = W.custom_structure(len(lens), 8, 2, D, lens, seed=800 + parts)
    q, k, v = W.fill_values(st, dev, fill="nan")
    bt, ln = torch.from_numpy(st.block_table).to(dev), torch.from_numpy(st.context_lens).to(dev)
    if prefix:
        got = pda_decode_shared_prefix(q, k, v, bt, ln, st.scale, torch.from_numpy(st.group_start).to(dev),
                                       torch.from_numpy(st.group_prefix_len).to(dev), max_context_len=st.max_context_len,
                                       max_group_size=len(lens), max_prefix_len=TP * prefix, partition_tokens=TP)
    else:
        ws = torch.full((1 << 24,), 0xFF, dtype=torch.uint8, device=dev)  # unused slots hold NaN
        got = pda_decode(q, k, v, bt, ln, st.scale, max_context_len=st.max_context_len, partition_tokens=TP, workspace=ws)
    ref = oracle.decode(W.bf16_bits(q), W.bf16_bits(k), W.bf16_bits(v), st.block_table, st.context_lens, st.scale,
                        threads=THREADS)
    check(got.cpu().numpy(), ref, f"merge of up to {prefix} + {parts} partitions, D={D}")
