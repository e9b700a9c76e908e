"""GPU parity of the wide steps (more than 4 query chunks per sequence) at the
edges of their kernel: chunk counts around 8 and 16 (one and two workgroups
per item, tiles with one chunk, wavefronts without any), group sizes whose
chunks do not fill 16 rows, partitions that are no multiple of the 32-token
step, and contexts past the 1024 block ids that are held at a time.  Bar as
for the other steps; non-finite values stay with the chunks that see them."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from parity_common import THREADS, check
from paper_2405_11143_amd import pda_decode

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


def run(st, q, k, v, dev, partition_tokens=0):
    bt = torch.from_numpy(st.block_table).to(dev)
    lens = torch.from_numpy(st.context_lens).to(dev)
    return pda_decode(q, k, v, bt, lens, st.scale, max_context_len=st.max_context_len,
                      partition_tokens=partition_tokens).cpu().numpy()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,n", [(8, 2, 17), (8, 2, 33), (4, 1, 61), (8, 1, 35), (7, 1, 19), (10, 2, 26),
                                      (16, 1, 9), (16, 1, 17), (3, 3, 81), (3, 3, 257)], ids=str)
@pytest.mark.parametrize("partition_tokens", [0, 16, 80])
def test_chunk_and_partition_edges(dev, D, Hq, Hkv, n, partition_tokens):
    lens = [1, n - 1, n, n + 1, n + 15, n + 16, 2 * n + 31, 700]
    st = W.custom_structure(len(lens), Hq, Hkv, D, lens, seed=500 + n + D)
    _, k, v = W.fill_values(st, dev, fill="nan")
    q = W.fill_multi_q(st, n, dev)
    ref = oracle.decode_multi(W.bf16_bits(q), W.bf16_bits(k), W.bf16_bits(v), st.block_table, st.context_lens,
                              st.scale, threads=THREADS)
    check(run(st, q, k, v, dev, partition_tokens), ref, f"wide Hq={Hq} Hkv={Hkv} D={D} n={n} Tp={partition_tokens}")


@pytest.mark.parametrize("n,partition_tokens", [(20, 0), (40, 0), (40, 33 * 1024)], ids=str)
def test_long_contexts(dev, n, partition_tokens):
    lens = [16 * 1024, 16 * 1024 + 1, 33000, 16 * 1024 + 47]
    st = W.custom_structure(len(lens), 8, 2, 128, lens, seed=600 + n)
    _, k, v = W.fill_values(st, dev, fill="nan")
    q = W.fill_multi_q(st, n, dev)
    got = run(st, q, k, v, dev, partition_tokens)
    assert np.isfinite(got).all()
    rows = np.asarray([(b, i, h) for b in range(len(lens)) for i in (0, n // 2, n - 1) for h in (0, 3, 5)], np.int32)
    ref = oracle.decode_multi_rows(W.bf16_bits(q), W.bf16_bits(k), W.bf16_bits(v), st.block_table, st.context_lens,
                                   st.scale, rows, threads=THREADS)
    check(got[rows[:, 0], rows[:, 1], rows[:, 2]], ref, f"long contexts n={n} Tp={partition_tokens}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=str)
@pytest.mark.parametrize("partition_tokens", [0, 48])
def test_non_finite_new_rows_stay_with_their_chunk(dev, D, value, partition_tokens):
    """A non-finite V element of a new token reaches the rows that see it and
    at most those of their chunk of 16 / G = 4 tokens; the chunk before it,
    which shares a wavefront's tile, keeps finite rows that meet the bar."""
    n, lens = 64, [64, 100, 333]
    st = W.custom_structure(len(lens), 8, 2, D, lens, seed=700)
    _, k, v = W.fill_values(st, dev, fill="nan")
    q = W.fill_multi_q(st, n, dev)
    ref = oracle.decode_multi(W.bf16_bits(q), W.bf16_bits(k), W.bf16_bits(v), st.block_table, st.context_lens,
                              st.scale, threads=THREADS)
    tokens = (5, 14, 47)  # new tokens of the second, fourth and twelfth chunk, one for each sequence
    for b, x in enumerate(tokens):
        t = lens[b] - n + x
        v[int(st.block_table[b, t // 16]), 1, t % 16, 37] = value
    got = run(st, q, k, v, dev, partition_tokens)
    for b, x in enumerate(tokens):
        first = x // 4 * 4  # the chunk's first token
        assert not np.isfinite(got[b, x:, 4:, 37]).any(), (b, x)
        got[b, first:, 4:, 37] = ref[b, first:, 4:, 37]
    check(got, ref, f"non-finite new rows D={D} Tp={partition_tokens}")
