"""The partition sizes of steps with few (sequence, KV head) pairs, and that
the rule for them stops where the general one takes over (no GPU)."""
import pytest

import paper_2405_11143_amd as pda


def plan(B, Hq, Hkv, max_len, n=1, D=128):
    info = pda.pda_plan(pda.make_problem(B, Hq, Hkv, D, 1 << 20, -(-max_len // 16), max_len, num_query_tokens=n))
    return info["partition_tokens"], info["num_partitions"]


@pytest.mark.parametrize("args,want", [
    ((4, 32, 8, 512), (512, 1)),         # short contexts stay whole
    ((4, 32, 8, 513), (256, 3)),         # 256 slots / 32 pairs = 8 pieces, at least 256 tokens
    ((12, 32, 8, 768), (768, 1)),        # 96 pairs in 256s would be more items than slots
    ((12, 32, 8, 769), (256, 4)),        # (192 of 256 slots: the share)
    ((4, 32, 8, 4096), (512, 8)),
    ((4, 32, 8, 8192), (1024, 8)),
    ((4, 32, 8, 8400), (1024, 9)),       # to the nearest 256
    ((4, 32, 8, 16384), (512, 32)),      # 2048 would be too long: the share
    ((8, 32, 8, 4096), (1024, 4)),
    ((12, 32, 8, 4096), (256, 16)),      # 96 pairs x 2 leave a quarter of the slots empty: the share
    ((17, 32, 8, 1024), (1024, 1)),      # no second item per slot
    ((17, 32, 8, 1025), (256, 5)),
    ((96, 32, 8, 1024), (1024, 1)),
    ((97, 32, 8, 1024), (768, 2)),       # more pairs than items run at once: the share
    ((4, 32, 8, 4096, 64), (512, 8)),    # items of two workgroups, one per compute unit
    ((4, 32, 8, 4096, 32), (256, 16)),   # of one: 512 slots
    ((16, 32, 8, 1024, 64), (1024, 1)),  # many wide rows are not split further
    ((32, 32, 8, 1025, 64), (1040, 1)),  # one piece is one partition
    ((32, 32, 8, 1151, 64), (1152, 1)),
    ((28, 32, 8, 2048, 64), (2048, 1)),
    ((28, 32, 8, 2049, 64), (768, 3)),   # (the share)
    ((16, 32, 8, 1536, 64), (1536, 1)),  # 2 pieces
    ((16, 32, 8, 1537, 64), (1024, 2)),
    ((10, 32, 8, 1152, 64), (1152, 1)),  # 3
    ((10, 32, 8, 1153, 64), (512, 3)),
    ((8, 32, 8, 768, 64), (768, 1)),     # 4
    ((8, 32, 8, 1024, 64), (512, 2)),
    ((8, 32, 8, 1024, 32), (256, 4)),    # 8
    ((8, 32, 8, 384, 32), (384, 1)),
    ((8, 32, 8, 385, 32), (256, 2)),
    ((4, 32, 8, 1024, 5), (256, 4)),     # staged items of 2-4 chunks: the share
])
def test_partition_choice(args, want):
    assert plan(*args) == want
