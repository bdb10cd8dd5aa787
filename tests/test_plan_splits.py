"""Plans of small launches, whose key ranges are split finer than a batch's:
every row produced exactly once, within the workspace bound, the decode
array of the call without a workspace and the staging buffers' plan size."""
import numpy as np
import pytest

from paper_2605_11232_amd import binding as B
from paper_2605_11232_amd import synth
from paper_2605_11232_amd.runtime import plan_words_bound
from tests.test_capi_host import H_N_GROUP_TMPL, H_N_GROUPS, check_plan, parse_plan

H_N_GROUP_NARROW = 28  # header word: merge groups of at most four rows


def _tables(r, L, prefix):
    """Block tables of sequences that share their first prefix // 16 blocks."""
    mb = int((L.max() + 15) // 16)
    bt = np.full((len(L), mb), -1, np.int32)
    nxt = 10 ** 6
    for i, x in enumerate(L):
        nb, p = int((x + 15) // 16), prefix // 16
        bt[i, :p] = np.arange(p)
        bt[i, p:nb] = np.arange(nxt, nxt + nb - p)
        nxt += nb
    return bt


@pytest.mark.parametrize("kind", ["decode", "verify", "prefill", "mixed"])
def test_small_launch_plans(kind):
    r = np.random.default_rng(31)
    code = {"decode": B.KIND_DECODE, "verify": B.KIND_VERIFY}.get(kind, B.KIND_PREFILL)
    split = 0
    for trial in range(16):
        n = int(r.integers(1, 6 if trial % 4 else 60))
        hkv, G = int(r.choice([1, 2, 3, 4, 8])), int(r.choice([1, 4, 7, 8, 16]))
        D = int(r.choice([64, 128]))
        n_q = int(r.integers(2, 9))
        prefix = int(r.choice([0, 256, 1000, 4096, 9000])) // 16 * 16
        q = {"decode": np.ones(n), "verify": np.full(n, n_q),
             "prefill": r.integers(1, 500, size=n),
             "mixed": np.where(r.random(n) < 0.2, r.integers(1, 600, size=n), 1)}[kind].astype(int)
        L = prefix + q + r.integers(0, int(r.choice([2, 700, 6000])), size=n)
        cu = np.concatenate([[0], np.cumsum(q)])
        bt = _tables(r, L, prefix)
        for table in (bt, None):
            plan, info = B.plan(code, n_q, L, cu, hkv * G, hkv, D, 16, B.PA_BF16, 256,
                                block_table=table)
            check_plan(plan, info, L, cu, G, hkv, D)
            cfg = synth.AttnConfig("", "bf16", hkv * G, hkv, D, 16, 0)
            assert info.plan_words <= plan_words_bound(cfg, n, int(cu[-1]), bt.shape[1])
            split += plan[H_N_GROUP_NARROW] < plan[H_N_GROUP_TMPL]
    # some launches' tiles have split keys (merge groups of a tile's rows)
    assert split > 0 or kind in ("decode", "verify")


def test_decode_plans_keep_fitting_the_array_without_workspace():
    """The finer splits never take a decode plan past the array that decode
    without a workspace holds: 16 heads per kv-head, where the rows of one
    part are the most, around the limit."""
    fits = 0
    for n in (8, 40, 60, 70, 100, 128):
        for own in (40, 500, 1500, 5000):
            L = np.full(n, 2048 + own + 1)
            bt = _tables(None, L, 2048)
            _, info = B.plan(B.KIND_DECODE, 1, L, np.arange(n + 1), 64, 4, 128, 16, B.PA_BF16,
                             256, block_table=bt)
            # a part per 256 private keys (at least one wavefront's share) and one shared
            parts = 1 + -(-(own + 1) // 256)
            if n * 64 * parts * 129 * 4 <= B.NOALLOC_WORKSPACE_BYTES:
                assert info.workspace_bytes <= B.NOALLOC_WORKSPACE_BYTES
                fits += 1
    assert fits > 5
    # few-row tiles for a caller that names more compute units than there are
    _, info = B.plan(B.KIND_DECODE, 1, [1 << 20], [0, 1], 64, 1, 128, 16, B.PA_BF16, 4096)
    assert 0 < info.workspace_bytes <= B.NOALLOC_WORKSPACE_BYTES


def test_plan_info_counts_merge_groups():
    """n_groups is the number of groups the merge combines, whatever the number of
    rows of a group, and the header's."""
    wide = 0
    for q, L in [([389], [2437]), ([100, 1], [4196, 900]), ([1, 1], [1000, 257]), ([40], [60])]:
        plan, info = B.plan(B.KIND_PREFILL, 0, np.array(L), np.concatenate([[0], np.cumsum(q)]), 32, 8, 128, 16,
                            B.PA_BF16, 256)
        groups = plan[H_N_GROUP_TMPL] * 8
        assert info.n_groups == plan[H_N_GROUPS] == groups
        is_wide = plan[H_N_GROUP_NARROW] < plan[H_N_GROUP_TMPL]
        assert (info.n_merge_items > groups) == is_wide
        wide += is_wide
    assert wide == 2


@pytest.mark.parametrize("D", [64, 128])
def test_decode_plans_of_many_heads_fit_the_array_without_workspace(D):
    """More than 64 heads per kv-head: such decode runs on tile items, which need no
    workspace whole, so their key splits never take a plan past the array."""
    split = 0
    for hkv, G in [(1, 96), (1, 128), (2, 128), (1, 256), (2, 256)]:
        for n in (1, 4, 8, 16, 64):
            for own in (700, 8192, 65536, 131072):
                L = np.full(n, own)
                L[1:] -= 3
                plan, info = B.plan(B.KIND_DECODE, 1, L, np.arange(n + 1), hkv * G, hkv, D, 16, B.PA_BF16, 256)
                assert info.workspace_bytes <= B.NOALLOC_WORKSPACE_BYTES
                split += info.workspace_bytes > 0
                if own < 10000:
                    check_plan(plan, info, L, np.arange(n + 1), G, hkv, D)
    assert split > 20


def test_row_items_are_split_finer_only_where_they_leave_the_chip_room():
    """Row items of 192 keys up to 3 of them per compute unit (6 at head_dim 64), beyond
    that of 256 (769 private keys: five parts of 160, or four of 224)."""
    for n, hkv, D, most in [(4, 8, 128, 160), (23, 8, 128, 160), (25, 8, 128, 224), (46, 4, 128, 160),
                            (50, 4, 128, 224), (46, 8, 64, 160), (50, 8, 64, 224)]:
        L = np.full(n, 960 + 769)
        bt = _tables(None, L, 960)
        plan, info = B.plan(B.KIND_DECODE, 1, L, np.arange(n + 1), 4 * hkv, hkv, D, 16, B.PA_BF16, 256, block_table=bt)
        assert max(t[5] - t[4] for t in parse_plan(plan)[3] if t[0] >= 0) == most


def test_prefix_chunks_beside_enough_other_work_stay_whole():
    """1024 shared keys of 48 decode requests: two chunks in a launch of their own, one
    beside a 512-token prefill chunk, whose steps they run beside."""
    for chunk, chunks in [(0, 2), (512, 1)]:
        q = np.array([chunk] * (chunk > 0) + [1] * 48)
        L = np.array([chunk] * (chunk > 0) + [1024 + 704] * 48)
        cu = np.concatenate([[0], np.cumsum(q)])
        bt = _tables(None, L, 1024)
        if chunk:
            bt[0] = -1
            bt[0, :32] = np.arange(32) + 5 * 10 ** 7
        plan, info = B.plan(B.KIND_PREFILL, 0, L, cu, 64, 8, 128, 16, B.PA_BF16, 256, block_table=bt)
        check_plan(plan, info, L, cu, 8, 8, 128)
        assert info.n_shared_items == chunks * 3 * 8


def test_few_row_tiles_fill_idle_compute_units():
    """33 to 64 rows per sequence: a launch that leaves compute units idle gets more
    items, one per compute unit at most; one key range of up to 512 keys that needs
    no merge stays whole, and so does everything once the sequences fill the chip or
    too few of them could be split to pay for the merge."""
    for n, own, hkv, prefix, more in [(1, 512, 8, 0, False), (1, 513, 8, 0, True), (1, 9000, 8, 0, True),
                                      (5, 3000, 4, 768, True), (16, 700, 8, 0, True), (31, 700, 8, 0, False),
                                      (32, 4100, 8, 4096, False), (33, 4100, 8, 0, False)]:
        L = np.full(n, prefix + own)
        L[1:] -= own // 3
        cu = np.arange(n + 1) * 5
        plan, info = B.plan(B.KIND_VERIFY, 5, L, cu, 8 * hkv, hkv, 128, 16, B.PA_BF16, 256,
                            block_table=_tables(None, L, prefix))
        check_plan(plan, info, L, cu, 8, hkv, 128)
        whole = n * hkv
        assert whole <= info.n_tile_items <= max(whole, 256)
        assert (info.n_tile_items > whole) == more


def test_launches_of_few_workgroups_have_no_tail_lists():
    for n, tail in [(1, False), (4, False), (5, True)]:  # 32 full tiles each
        L = np.full(n, 256)
        plan, info = B.plan(B.KIND_PREFILL, 0, L, np.arange(n + 1) * 128, 32, 8, 128, 16, B.PA_BF16, 256)
        check_plan(plan, info, L, np.arange(n + 1) * 128, 4, 8, 128)
        assert bool(info.variant & 4) == tail


def test_key_split_tiles_hold_plain_ranges():
    """A key-split tile's item is what its words say: no flag but the streaming
    one, the parts of a tile one after another from key 0 to the sequence's end."""
    plan, info = B.plan(B.KIND_PREFILL, 0, np.array([4196, 3000]), np.array([0, 100, 165]), 28, 4, 128, 16,
                        B.PA_BF16, 256)
    tiles = parse_plan(plan)[2]
    assert plan[H_N_GROUP_NARROW] == 0 and len(tiles) > 4 * plan[H_N_GROUP_TMPL]
    assert {t[7] for t in tiles} == {0}
    check_plan(plan, info, np.array([4196, 3000]), np.array([0, 100, 165]), 7, 4, 128)


def _f32(hq, hkv, d, q, L):
    _, info = B.plan(B.KIND_PREFILL, 0, np.array(L), np.concatenate([[0], np.cumsum(q)]), hq, hkv, d, 16, B.PA_F32, 256)
    assert info.workspace_bytes == 0 and info.n_groups == 0
    return info


def test_float32_plans_count_their_workgroups():
    """Row tiles: 16 or 32 rows of a sequence and kv-head to a workgroup, at most one
    workgroup more per sequence than its rows fill."""
    for hq, hkv, q, tile in [(8, 2, [40, 3, 0], 16), (32, 8, [64] * 16, 32), (32, 8, [500, 530], 32), (28, 4, [1] * 9, 16)]:
        info = _f32(hq, hkv, 128, q, [x + 100 for x in q])
        rows = np.array(q) * (hq // hkv)
        assert info.variant == 0
        assert sum(-(-rows // tile)) * hkv <= info.grid <= (sum(rows) // tile + len(q)) * hkv


def test_float32_short_sequences_of_one_row_run_by_row():
    """One wavefront per (token, head) where every sequence has one row per kv-head (or
    two), few keys, and the chip is full; a single longer or taller one: tiles."""
    for hq, hkv, d, q, L, by_row in [
            (32, 32, 64, [1] * 64, [144] * 64, True), (32, 32, 64, [1] * 64, [144] * 63 + [145], False),
            (32, 32, 128, [1] * 64, [64] * 64, True), (32, 32, 128, [1] * 64, [65] * 64, False),
            (32, 32, 64, [1] * 63, [20] * 63, False), (32, 32, 64, [1] * 64 + [0], [20] * 64 + [500], True),
            (32, 16, 64, [1] * 128, [32] * 128, True), (32, 16, 64, [1] * 128, [33] * 128, False),
            (32, 32, 64, [2] * 64, [48] * 64, True), (32, 32, 64, [2] * 64, [49] * 64, False),
            (32, 32, 128, [2] * 64, [33] * 64, False), (32, 32, 64, [3] + [1] * 70, [20] * 71, False),
            (32, 8, 64, [1] * 400, [4] * 400, False)]:
        info = _f32(hq, hkv, d, q, L)
        assert (info.variant == 16) == by_row
        if by_row:
            assert info.grid == sum(q) * hq


def test_few_row_tiles_beside_longer_work_stay_whole():
    """Items whose keys take less than half of what the row items take are not split;
    longer ones are."""
    for own, decodes, more in [(1300, 8, True), (1300, 256, False), (7000, 256, True)]:
        q = np.array([12] + [1] * decodes)
        L = np.array([own] + [1024 + 704] * decodes)
        cu = np.concatenate([[0], np.cumsum(q)])
        bt = _tables(None, np.concatenate([L[1:], L[:1]]), 1024)
        bt = np.concatenate([bt[-1:], bt[:-1]])
        bt[0, :64] += 5 * 10 ** 7
        plan, info = B.plan(B.KIND_PREFILL, 0, L, cu, 32, 8, 128, 16, B.PA_BF16, 256, block_table=bt)
        check_plan(plan, info, L, cu, 4, 8, 128)
        assert (info.n_tile_items > 8 * -(-own // 4160)) == more


def test_few_row_tiles_are_split_together():
    """Where the longest sequences are split, so are the others that hold two parts: an
    item left whole would be what the launch waits for."""
    L = np.array([700] + [467] * 3)
    plan, info = B.plan(B.KIND_VERIFY, 5, L, np.arange(5) * 5, 64, 8, 128, 16, B.PA_BF16, 256)
    check_plan(plan, info, L, np.arange(5) * 5, 8, 8, 128)
    assert max(t[5] - t[4] for t in parse_plan(plan)[2]) <= 256


def test_tiles_beside_longer_row_work_stay_whole():
    """One prefill chunk's tiles are split beside few decode requests, and whole beside
    so many that their row items take twice as long."""
    for hq, hkv, decodes, more in [(32, 8, 8, True), (32, 8, 64, True), (28, 4, 256, True), (32, 8, 256, False),
                                   (32, 8, 512, False)]:
        q = np.array([512] + [1] * decodes)
        L = np.array([2560] + [2048 + 704] * decodes)
        cu = np.concatenate([[0], np.cumsum(q)])
        plan, info = B.plan(B.KIND_PREFILL, 0, L, cu, hq, hkv, 128, 16, B.PA_BF16, 256, block_table=_tables(None, L, 2048))
        check_plan(plan, info, L, cu, hq // hkv, hkv, 128)
        assert (info.n_tile_items > 512 * hq // 128) == more


def test_tiles_beside_other_long_items_stay_whole():
    """Splitting a long sequence's tiles gains nothing while few-row items walk as many
    keys in series."""
    q = np.array([1] * 85 + [30] * 11)
    L = np.linspace(1056, 3235, 96).astype(int)
    cu = np.concatenate([[0], np.cumsum(q)])
    plan, info = B.plan(B.KIND_PREFILL, 0, L, cu, 96, 2, 64, 16, B.PA_BF16, 256)
    check_plan(plan, info, L, cu, 48, 2, 64)
    assert info.workspace_bytes == 0


def test_short_few_row_sequences_stay_whole_beside_merged_ones():
    """A sequence of up to 512 keys that needs no merge is not split because others of the
    launch, members of a shared prefix with few keys of their own, have one."""
    q = np.array([10] * 6 + [12])
    L = np.array([266] * 6 + [300])
    cu = np.concatenate([[0], np.cumsum(q)])
    plan, info = B.plan(B.KIND_PREFILL, 0, L, cu, 32, 8, 128, 16, B.PA_BF16, 256, block_table=_tables(None, L, 256))
    check_plan(plan, info, L, cu, 4, 8, 128)
    assert info.n_shared_items > 0 and info.n_tile_items == 7 * 8
