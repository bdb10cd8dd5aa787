"""GPU parity of single kernel paths at the sizes where they can go wrong
(tile edges, remainders, the smallest and largest of a path's range), against
the float64 oracle at the tolerances of tests/parity.py."""
import numpy as np
import pytest
import torch

from paper_2605_11232_amd import binding as B, synth
from tests.parity import LSE_TOL, TOL, close, run_parity, say

pytestmark = pytest.mark.gpu


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def launch_workload(cfg, q_lens, lens, seed, prefix=0):
    """One launch of sequences of lens[i] tokens whose last q_lens[i] are
    queried; the first ``prefix`` (whole blocks) are one cached prefix."""
    r = np.random.default_rng(seed)
    Val, bs = synth.Values, cfg.block_size
    kv = (cfg.num_kv_heads, cfg.head_dim)

    def values(tag, *shape):
        return Val((cfg.seed, seed) + tag, shape, cfg.dtype)

    pt = r.integers(0, 1 << 17, size=prefix).astype(np.int32)
    setup, pre = [], []
    if prefix:
        sid = synth.PREFIX_SEQ_BASE
        setup += [synth.Op("add", sid, pt),
                  synth.Op("write_kv", sid, k=values((1,), prefix, *kv),
                           v=values((2,), prefix, *kv)), synth.Op("free", sid)]
    for i, (q, L) in enumerate(zip(q_lens, lens)):
        toks = np.concatenate([pt, r.integers(0, 1 << 17, size=L - prefix).astype(np.int32)])
        own = L - q - prefix  # cached tokens of the sequence's own
        if own > 0:
            setup += [synth.Op("add", i, toks[:L - q]),
                      synth.Op("write_kv", i, k=values((3, i), own, *kv),
                               v=values((4, i), own, *kv))]
            pre.append(synth.Op("extend", i, toks[L - q:]))
        else:
            pre.append(synth.Op("add", i, toks))
    T = sum(q_lens)
    launch = synth.Launch(pre, list(range(len(lens))), list(q_lens),
                          values((5,), T, cfg.num_q_heads, cfg.head_dim),
                          values((6,), T, *kv), values((7,), T, *kv))
    nb = sum(-(-x // bs) for x in lens) + prefix // bs + 8
    return synth.Workload(cfg, nb, np.random.default_rng(seed).permutation(nb).astype(np.int32),
                          setup, [launch], None, -(-max(lens) // bs))


# (q heads, kv heads, head_dim, query tokens, lengths): 16- and 32-row
# workgroups (the latter from 512 of them), partial last tiles, group sizes
# that do not divide a tile and ones above it, sequences of one token and of
# none, more wavefronts than blocks, more sequences than one round of the
# sequence search probes, a table of more than 64 blocks per wavefront
F32 = [
    (4, 4, 64, [1], [1]),
    (8, 2, 64, [0, 7, 0, 5, 1], [4, 7, 33, 16, 300]),
    (6, 2, 128, [17, 33], [40, 33]),
    (40, 1, 64, [3, 1], [20, 129]),
    (16, 2, 128, [1] * 70, [3 + 2 * i for i in range(70)]),
    (8, 2, 128, [2, 1], [4200, 4097]),
    (32, 32, 64, [520, 9], [600, 31]),
    (32, 8, 128, [300, 230, 0], [317, 530, 64]),
    # one wavefront per (token, head): one row per kv-head, two by tokens and by heads
    (32, 32, 64, [1] * 70 + [0], [1 + 2 * i for i in range(70)] + [40]),
    (32, 32, 128, [1] * 70, [64 - i % 17 for i in range(70)]),
    (32, 32, 64, [2, 1] * 35, [48 - i % 46 for i in range(70)]),
    (32, 16, 128, [1] * 130, [1 + i % 32 for i in range(130)]),
]
F32_BY_ROW = 4  # of them, the last


@pytest.mark.parametrize("case", range(len(F32)))
def test_f32_tiles(case):
    _gpu()
    hq, hkv, d, q_lens, lens = F32[case]
    cfg = synth.AttnConfig(f"f32-{case}", "f32", hq, hkv, d, 16, 6100 + case)
    errs, dev, _ = run_parity(launch_workload(cfg, q_lens, lens, 40 + case), label=cfg.name)
    say(f"{cfg.name} normalized errors", errs)
    assert (dev.infos[0].variant == 16) == (case >= len(F32) - F32_BY_ROW)


def test_f32_values_that_are_not_finite_stay_with_their_rows():
    """A new token's infinite or NaN values reach that token's row and later
    ones, in those dimensions, and no earlier row of the same tile."""
    _gpu()
    from paper_2605_11232_amd.runtime import DeviceReplay
    cfg = synth.AttnConfig("f32-inf", "f32", 4, 2, 64, 16, 6190)
    wl = launch_workload(cfg, [20], [52], 77)
    dev = DeviceReplay(wl).setup()
    p = dev.prepare(wl.launches[0])
    dev.append(p)
    dev.attend(p)
    plain = p.out.clone()
    bad = 13
    p.v_new[bad, :, 5], p.v_new[bad, :, 9] = float("inf"), float("nan")
    dev.append(p)
    dev.attend(p)
    torch.cuda.synchronize()
    assert torch.equal(p.out[:bad], plain[:bad])
    dims = [i for i in range(cfg.head_dim) if i not in (5, 9)]
    # same products in the same order
    assert torch.equal(p.out[:, :, dims], plain[:, :, dims])
    assert torch.isposinf(p.out[bad:, :, 5]).all() and torch.isnan(p.out[bad:, :, 9]).all()


# (kind, q heads, kv heads, head_dim, query tokens, lengths, prefix): launches
# small enough that their splits are finer than a batch's
SMALL = {
    # a shared prefix in chunks of 256 keys, a partial block past it
    "decode-chunks": ("decode", 8, 2, 128, [1] * 3, [2100, 2049, 2563], 2048),
    # one kv-head, 40 members: chunks limited by their workgroups
    "decode-one-head": ("decode", 7, 1, 64, [1] * 40, [1600 + 9 * i for i in range(40)], 1584),
    # no prefix: private ranges at the workspace bound's part count
    "decode-private": ("decode", 32, 8, 128, [1, 1], [1000, 257], 0),
    # 24-row row items beside the chunks
    "verify-wide-rows": ("verify", 6, 2, 64, [8] * 3, [1040, 1999, 1033], 1024),
    # 40 rows: private tile items split to a few steps each, alone and past a prefix
    "verify-tiles": ("verify", 16, 2, 128, [5] * 3, [1000, 515, 2053], 0),
    "verify-tiles-prefix": ("verify", 16, 2, 64, [5] * 3, [2000, 1030, 1800], 1024),
}


@pytest.mark.parametrize("name", list(SMALL))
def test_small_launch_splits(name):
    _gpu()
    kind, hq, hkv, d, q_lens, lens, prefix = SMALL[name]
    cfg = synth.AttnConfig(name, "bf16", hq, hkv, d, 16, 6200 + len(name))
    errs, dev, _ = run_parity(launch_workload(cfg, q_lens, lens, 60, prefix), label=name)
    say(name, "normalized errors", errs)
    info = dev.infos[0]
    assert info.n_groups > 0
    if prefix:  # more than one chunk
        row_tiles = -(-sum(q_lens) * (hq // hkv) // 128)
        assert info.n_shared_items >= 2 * row_tiles * hkv


# (q heads, kv heads, head_dim, query tokens, lengths): tiles whose keys are
# split: rows that a part's keys are all hidden from, a part of one step, a partial
# last tile, a cached context that ends inside a step, head_dim 64
TILE_SPLIT = [
    (8, 2, 128, [100], [2100]),
    (4, 4, 64, [129, 3], [1300, 700]),
    (28, 4, 128, [65, 40], [577 + 64, 4000]),
    (16, 1, 128, [600, 1], [1111, 900]),
]


@pytest.mark.parametrize("case", range(len(TILE_SPLIT)))
def test_key_split_tiles(case):
    _gpu()
    hq, hkv, d, q_lens, lens = TILE_SPLIT[case]
    cfg = synth.AttnConfig(f"split-{case}", "bf16", hq, hkv, d, 16, 6300 + case)
    errs, dev, _ = run_parity(launch_workload(cfg, q_lens, lens, 80 + case), label=cfg.name)
    say(f"{cfg.name} normalized errors", errs)
    info = dev.infos[0]
    tiles = sum(-(-q * (hq // hkv) // 128) for q in q_lens if q * (hq // hkv) > 64) * hkv
    assert info.n_tile_items > tiles and info.n_merge_rows >= 128


@pytest.mark.parametrize("d", [64, 128])
def test_tile_rows_without_a_finite_first_score(d):
    """The scores of a row's first keys (more than one 64-key step) are minus
    infinity: the result is the softmax over the others, whose scores lie far
    below zero; later keys raise the maximum by more than the tile path's
    sums allow without moving its reference."""
    _gpu()
    from paper_2605_11232_amd.runtime import DeviceReplay
    cfg = synth.AttnConfig(f"late-{d}", "bf16", 4, 2, d, 16, 6400 + d)
    n, L, first = 130, 500, 100
    wl = launch_workload(cfg, [n], [L], 91)
    dev = DeviceReplay(wl).setup()
    p = dev.prepare(wl.launches[0])
    dev.append(p)
    bt = p.block_table[0].long()
    t = torch.arange(L, device="cuda")
    off = t % 16
    pos = (off & ~12) | ((off & 4) << 1) | ((off & 8) >> 1)
    # dim 0 of the queries is 8 and that of a key sets its score
    p.q[:, :, 0] = 8.0
    k0 = torch.full((L,), -512.0, device="cuda")
    k0[:first] = -float("inf")
    k0[300:] = torch.linspace(-512.0, 64.0, L - 300, device="cuda")
    dev.k_cache[bt[t // 16], :, 0, pos, 0] = k0.to(torch.bfloat16)[:, None]
    dev.attend(p)
    torch.cuda.synchronize()
    k = dev.k_cache[bt[t // 16], :, :, pos].double().reshape(L, 2, d).permute(1, 2, 0).contiguous()
    v = dev.v_cache[bt[t // 16], :, :, off].double().permute(1, 0, 2).contiguous()
    q = p.q.double().view(n, 2, 2, d).permute(1, 0, 2, 3).reshape(2, 2 * n, d).contiguous()
    s = torch.bmm(q, k).view(2, n, 2, L) * d ** -0.5
    s.masked_fill_(t > (L - n + torch.arange(n, device="cuda"))[:, None, None], -float("inf"))
    ref = torch.bmm(torch.softmax(s, 3).view(2, 2 * n, L), v).view(2, n, 2, d).permute(1, 0, 2, 3)
    lse = torch.logsumexp(s, 3).permute(1, 0, 2).reshape(n, 4)
    close(p.out.float().cpu().numpy(), ref.reshape(n, 4, d).cpu().numpy(), *TOL["bf16"], cfg.name)
    close(p.lse.cpu().numpy(), lse.cpu().numpy(), *LSE_TOL["bf16"], cfg.name + " lse")


@pytest.mark.parametrize("d", [64, 128])
def test_tile_values_near_the_largest_stay_finite(d):
    """A key whose probability lies 2^11 above the first step's, with values of 3e35: the row's
    output is finite, as the reference moves before the product leaves float32."""
    _gpu()
    from paper_2605_11232_amd.runtime import DeviceReplay
    cfg = synth.AttnConfig(f"large-{d}", "bf16", 4, 2, d, 16, 6700 + d)
    n, L, at = 130, 500, 300
    dev = DeviceReplay(launch_workload(cfg, [n], [L], 92)).setup()
    p = dev.prepare(dev.wl.launches[0])
    dev.append(p)
    bt = p.block_table[0].long()
    t = torch.arange(L, device="cuda")
    off = t % 16
    pos = (off & ~12) | ((off & 4) << 1) | ((off & 8) >> 1)
    # every score 0 (dim 0 of the queries is 8, the other dims of the keys 0) but one
    p.q[:, :, 0] = 8.0
    dev.k_cache[bt[t // 16], :, :, pos] = 0
    score = 11 * 0.6931
    dev.k_cache[bt[at // 16], :, 0, pos[at], 0] = score * d ** 0.5 / 8
    dev.v_cache[bt[t // 16], :, :, off] = 0
    dev.v_cache[bt[at // 16], :, :, off[at]] = 3e35
    dev.attend(p)
    torch.cuda.synchronize()
    w = float(dev.k_cache[bt[at // 16], 0, 0, pos[at], 0].double()) * 8 * d ** -0.5
    seen = (L - n + torch.arange(n, device="cuda") + 1).double()
    v = float(dev.v_cache[bt[at // 16], 0, 0, off[at]].double())
    ref = np.exp(w) * v / (np.exp(w) + seen - 1).cpu().numpy()
    ref = np.where((seen > at).cpu().numpy(), ref, 0.0)[:, None, None] * np.ones((1, 4, d))
    close(p.out.float().cpu().numpy() / v, ref / v, *TOL["bf16"], cfg.name)


def test_calls_use_the_current_stream():
    """A call without a stream argument goes to the stream torch has as current on the
    current device, whichever it is, and an explicit one to itself."""
    _gpu()
    assert B._stream(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert B._stream(None) == side.cuda_stream
    assert B._stream(side) == B._stream(side.cuda_stream) == side.cuda_stream
    assert B._stream(None) == torch.cuda.current_stream().cuda_stream


# (kind, q heads, kv heads, head_dim, query tokens, lengths, prefix): rows merged
# from key-split tiles, few-row tiles, row items, a shared prefix's chunks, and
# whole tiles beside them
NAN = {
    "tiles": ("prefill", 8, 2, 128, [100], [2100], 0),
    "tiles-whole": ("prefill", 8, 2, 128, [100], [120], 0),
    "verify-tiles": ("verify", 16, 2, 64, [5] * 2, [1000, 2053], 0),
    "decode": ("decode", 32, 8, 128, [1, 1], [1000, 257], 0),
    "decode-shared": ("decode", 8, 2, 128, [1] * 3, [2100, 2049, 2563], 2048),
}


@pytest.mark.parametrize("where", ["query", "key"])
@pytest.mark.parametrize("name", list(NAN))
def test_rows_without_a_number_stay_visible(name, where):
    """A row whose query, or a key it sees, is NaN comes out NaN (its log-sum-exp
    minus infinity) however its keys are split; no other row is touched."""
    _gpu()
    from paper_2605_11232_amd.runtime import DeviceReplay
    kind, hq, hkv, d, q_lens, lens, prefix = NAN[name]
    cfg = synth.AttnConfig(f"nan-{name}", "bf16", hq, hkv, d, 16, 6500 + len(name))
    dev = DeviceReplay(launch_workload(cfg, q_lens, lens, 61, prefix)).setup()
    p = dev.prepare(dev.wl.launches[0])
    dev.append(p)
    dev.attend(p)
    plain = p.out.float().cpu().numpy()
    bad = torch.zeros(plain.shape[:2], dtype=torch.bool)
    if where == "query":
        p.q[q_lens[0] - 1, 1, 3] = float("nan")
        bad[q_lens[0] - 1, 1] = True
    else:
        # the last token's key, of the first kv-head, in the first sequence: its last query
        slot = int(p.slots[q_lens[0] - 1])
        off = slot % 16
        pos = (off & ~12) | ((off & 4) << 1) | ((off & 8) >> 1)
        dev.k_cache[slot // 16, 0, 0, pos, 3] = float("nan")
        bad[q_lens[0] - 1, :hq // hkv] = True
    dev.attend(p)
    torch.cuda.synchronize()
    out, lse = p.out.float().cpu(), p.lse.cpu()
    assert torch.equal(torch.isnan(out).all(2), bad) and torch.equal(torch.isnan(out).any(2), bad)
    assert torch.equal(lse == -float("inf"), bad)
    close(out[~bad].numpy(), plain[~bad.numpy()], *TOL["bf16"], cfg.name)


def test_plans_of_earlier_libraries_keep_merging():
    """A plan whose header does not count its narrow merge groups, and whose info
    does not count merge workgroups, as libraries without wide groups wrote them,
    gives the same result."""
    _gpu()
    from paper_2605_11232_amd.runtime import DeviceReplay
    cfg = synth.AttnConfig("old-plan", "bf16", 32, 8, 128, 16, 6600)
    dev = DeviceReplay(launch_workload(cfg, [1] * 3, [1000, 257, 2300], 62)).setup()
    p = dev.prepare(dev.wl.launches[0])
    dev.append(p)
    dev.attend(p)
    plain, plain_lse = p.out.clone(), p.lse.clone()
    assert p.info.n_groups > 8
    p.plan[28] = 0  # groups of at most four rows
    p.info.n_merge_items = 0
    p.info.variant &= ~8
    p.out.zero_()
    p.lse.zero_()
    dev.attend(p)
    torch.cuda.synchronize()
    assert torch.equal(p.out, plain) and torch.equal(p.lse, plain_lse)
