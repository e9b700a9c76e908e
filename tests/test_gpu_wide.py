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
from paper_2405_11143_amd import make_problem, pda_decode, pda_plan

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


def rows_of(st, cache_rows, b, g, n):
    """The first n K or V rows of (sequence, KV head) as float64."""
    t = np.arange(n)
    return cache_rows[st.block_table[b, t // 16], g, t % 16].astype(np.float64)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("factor", [1.0, 25.0, -3.0])
@pytest.mark.parametrize("n,partition_tokens", [(17, 0), (40, 0), (40, 16), (100, 0)])
def test_one_token_rows_return_v(dev, D, factor, n, partition_tokens):
    """The row that sees one token gives it probability exactly 1 and returns
    its V row bit for bit, as the first row of every fresh prompt does."""
    Hq, Hkv, lens = 8, 2, [n, n - 3, 1, n - 1]
    st = W.custom_structure(len(lens), Hq, Hkv, D, lens, seed=900 + n)
    _, k, v = W.fill_values(st, dev, fill="nan")
    q = W.fill_multi_q(st, n, dev)
    bt, ln = torch.from_numpy(st.block_table).to(dev), torch.from_numpy(st.context_lens).to(dev)
    got = pda_decode(q, k, v, bt, ln, st.scale * factor, max_context_len=st.max_context_len,
                     partition_tokens=partition_tokens).cpu().numpy()
    vh = v.float().cpu().numpy()
    for b, L in enumerate(lens):
        for h in range(Hq):
            assert np.array_equal(got[b, n - L, h], vh[st.block_table[b, 0], h * Hkv // Hq, 0]), (b, h)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("exponent", [5, 17], ids=["2^10", "2^34"])
@pytest.mark.parametrize("partition_tokens", [0, 48])
def test_large_scores(dev, D, exponent, partition_tokens):
    """Finite q and K of a size whose scaled scores reach 2^14 and 2^34: the
    softmax is all on one token, and the rows are that token's V row within
    2^-15 of it (a running maximum may stay up to 2^8 below, and then the
    token's probability is kept in two bf16 halves, to 2^-16).  Rows whose two largest scores differ by less than the rounding of two
    fp32 dot products (D terms, each within 2^-24 of the sum of magnitudes) and
    of two running maxima, plus 64 powers of two, are left out."""
    n, Hq, Hkv = 40, 8, 2
    lens = [n, n + 41, 300, 17]
    st = W.custom_structure(len(lens), Hq, Hkv, D, lens, seed=950)
    _, k, v = W.fill_values(st, dev, fill="zero")
    q = W.fill_multi_q(st, n, dev) * 2.0 ** exponent
    k = k * 2.0 ** exponent
    got = run(st, q, k, v, dev, partition_tokens)
    assert np.isfinite(got).all()
    kr = W.k_cache_to_rows(k).float().cpu().numpy()
    vh, qh = v.float().cpu().numpy(), q.float().cpu().numpy().astype(np.float64)
    scale_log2 = st.scale * np.log2(np.e)
    checked = total = 0
    for b, L in enumerate(lens):
        for h in range(Hq):
            K, V = rows_of(st, kr, b, h * Hkv // Hq, L), rows_of(st, vh, b, h * Hkv // Hq, L)
            s = qh[b, :, h] @ K.T * scale_log2
            size = np.abs(qh[b, :, h]) @ np.abs(K.T) * scale_log2
            for i in range(max(0, n - L), n):
                vis = L - n + 1 + i
                best, second = np.argsort(-s[i, :vis])[[0, min(1, vis - 1)]]
                bound = 2 * D * 2.0 ** -24 * size[i, :vis].max() + 2 * 2.0 ** -24 * np.abs(s[i, :vis]).max() + 64
                total += 1
                if vis > 1 and s[i, best] - s[i, second] < bound:
                    continue
                checked += 1
                assert (np.abs(got[b, i, h] - V[best]) <= 2.0 ** -15 * np.abs(V[best])).all(), (b, i, h)
    print(f"large scores 2^{exponent}: {checked} of {total} rows", flush=True)
    assert checked > total // 2


WIDE_SHAPES = [(8, 2, 24), (8, 2, 64), (8, 2, 100), (16, 1, 9)]  # 6, 16, 25 and 9 chunks per sequence


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,n", WIDE_SHAPES, ids=str)
@pytest.mark.parametrize("partition_tokens", [0, 64])
def test_out_of_range_block_ids_give_nan_rows(dev, D, Hq, Hkv, n, partition_tokens):
    """A block id outside the pool is never dereferenced, and every row of an
    item (up to 16 chunks of a sequence in one partition) that looks at it is
    NaN, whichever workgroup of the item holds the row: ids that all chunks
    see, that only the last chunk sees, and that only the second eight chunks
    reach.  Rows of other items and sequences meet the bar."""
    lens = [n + 200, 333, n + 37, 700, 150]
    st = W.custom_structure(len(lens), Hq, Hkv, D, lens, seed=960 + n)
    _, k, v = W.fill_values(st, dev, fill="nan")
    q = W.fill_multi_q(st, n, dev)
    qc = min(n, 16 // (Hq // Hkv))
    nqc = -(-n // qc)
    per_item = 16 if nqc > 8 else 8
    tp = pda_plan(make_problem(st.B, Hq, Hkv, D, st.num_blocks, st.max_blocks_per_seq, st.max_context_len,
                               partition_tokens, num_query_tokens=n))["partition_tokens"]
    table = st.block_table.copy()
    visible = lambda L, c: L - n + min(n, (c + 1) * qc)  # tokens the chunk's last row sees
    bad = {0: [3], 1: [(333 - 1) // 16], 2: [(visible(n + 37, min(8, nqc - 1)) - 1) // 16, 1]}
    bad[1].append((visible(333, min(per_item, nqc) - 1) - 1) // 16)  # the last block the first item looks at
    for b, js in bad.items():
        for i, j in enumerate(js):
            table[b, j] = (st.num_blocks + 7, -1, 2 ** 31 - 1, -2 ** 31)[(b + i) % 4]
    bt, ln = torch.from_numpy(table).to(dev), torch.from_numpy(st.context_lens).to(dev)
    got = pda_decode(q, k, v, bt, ln, st.scale, max_context_len=st.max_context_len,
                     partition_tokens=partition_tokens).cpu().numpy()
    ref = oracle.decode_multi(W.bf16_bits(q), W.bf16_bits(k), W.bf16_bits(v), st.block_table, st.context_lens,
                              st.scale, threads=THREADS)
    for b, js in bad.items():
        L = lens[b]
        for c in range(nqc):
            last = min(nqc, (c // per_item + 1) * per_item) - 1
            blocks = -(-visible(L, last) // 16)  # the item's chunks look at blocks below it
            nan = any(j < blocks and j * 16 // tp < -(-visible(L, c) // tp) for j in js)
            rows = slice(c * qc, (c + 1) * qc)
            assert np.isnan(got[b, rows]).all() == nan and np.isnan(got[b, rows]).any() == nan, (b, c)
            if nan:
                got[b, rows] = ref[b, rows]
    check(got, ref, f"wide, bad ids n={n} D={D} Tp={partition_tokens}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,n", WIDE_SHAPES, ids=str)
@pytest.mark.parametrize("factor", [-1.0, 0.0, 3.0, 25.0, 1e-39])
@pytest.mark.parametrize("partition_tokens", [0, 48])
def test_scale_sign_zero_and_peaked(dev, D, Hq, Hkv, n, factor, partition_tokens):
    """Negative, zero, large and subnormal scales: the kernel folds the sign
    into q and takes a zero scale's scores from a zeroed q."""
    lens = [1, n - 1, n + 5, 300, 1040]
    st = W.custom_structure(len(lens), Hq, Hkv, D, lens, seed=970 + n)
    _, k, v = W.fill_values(st, dev, fill="nan")
    q = W.fill_multi_q(st, n, dev)
    scale = float(np.float32(st.scale * factor))
    bt, ln = torch.from_numpy(st.block_table).to(dev), torch.from_numpy(st.context_lens).to(dev)
    got = pda_decode(q, k, v, bt, ln, scale, max_context_len=st.max_context_len,
                     partition_tokens=partition_tokens).cpu().numpy()
    ref = oracle.decode_multi(W.bf16_bits(q), W.bf16_bits(k), W.bf16_bits(v), st.block_table, st.context_lens, scale,
                              threads=THREADS)
    check(got, ref, f"wide, scale x{factor} n={n} D={D} Tp={partition_tokens}")
