"""The holder index's build (netkv_cache_load): membership of every decode
against numpy, over the forms the resident sets take.  Needs an MI355X and
the built library."""
import numpy as np
import pytest

from paper_2606_03910_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

D = 48   # decodes of the 64-GPU cluster


@pytest.fixture(scope="module")
def nk():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_03910_amd import netkv
    netkv.load_library()
    return netkv


def _u64(rng, n):
    return rng.integers(1, 1 << 63, n, dtype=np.uint64) * np.uint64(2) + rng.integers(0, 2, n, dtype=np.uint64)


def _sets(form, rng):
    """Per decode the resident hashes, and the load factor."""
    if form == "empty":
        return [np.zeros(0, np.uint64)] * D, 0.5
    if form == "one":
        return [np.array([7], np.uint64)] + [np.zeros(0, np.uint64)] * (D - 1), 0.5
    if form == "part":        # all in one part, with repeats in a set
        x = _u64(rng, 300)
        return [np.concatenate([x[d:d + 40], x[d:d + 7]]) for d in range(D)], 0.5
    if form == "same":        # every decode holds the same set: many parts per block
        x = _u64(rng, 5000)
        return [rng.permutation(x) for _ in range(D)], 0.5
    if form == "sequential":  # hashes that differ in their low bits only
        return [np.arange(1 + 3000 * d, 1 + 3000 * d + 4000, dtype=np.uint64) for d in range(D)], 0.5
    if form == "sparse":      # several blocks per part
        return [_u64(rng, 700) for _ in range(D)], 0.02
    if form == "dense":
        return [_u64(rng, 9100) for _ in range(D)], 0.85
    if form == "large":       # parts told apart by two sort digits
        x = _u64(rng, 200000)
        return [np.concatenate([_u64(rng, 1600000), rng.choice(x, 50000)]) for _ in range(D)], 0.5
    raise AssertionError(form)


FORMS = ["empty", "one", "part", "same", "sequential", "sparse", "dense", "large"]


def _check(nk, sel, snap, sets, lf, rng, host, also=()):
    off = np.zeros(D + 1, np.uint64)
    off[1:] = np.cumsum([len(x) for x in sets])
    lead = 3   # the first set need not start at 0
    hs = np.concatenate([np.full(lead, 5, np.uint64)] + list(sets))
    off += np.uint64(lead)
    if host:   # (the C call takes host arrays too)
        assert nk.load_library().netkv_cache_load(sel.h, D, off.ctypes.data, hs.ctypes.data, len(hs), lf, None) == 0
    else:
        nk.netkv_cache_load(sel.h, D, nk.to_device(off, sel.device), nk.to_device(hs, sel.device), lf, sel.device)
    allh = hs[lead:]
    owner = np.repeat(np.arange(D), [len(x) for x in sets])
    uniq, inv = np.unique(allh, return_inverse=True)
    holds = np.zeros((len(uniq) + 1, D), bool)
    holds[inv, owner] = True
    ci = nk.netkv_cache_info(sel.h)
    assert ci["distinct_hashes"] == len(uniq)
    assert ci["shared_hashes"] == int((holds.sum(1) >= 2).sum())
    buckets = 8
    while 2 * buckets * lf < len(uniq):
        buckets *= 2
    assert ci["index_slots"] in (2 * buckets, 4 * buckets, 8 * buckets)
    # one-block requests: resident hashes of every kind, and others
    q = np.concatenate([rng.choice(uniq, 1200) if len(uniq) else uniq, _u64(rng, 300), np.zeros(1, np.uint64),
                        np.asarray(also, np.uint64)])
    bt = int(snap["block_tokens"])
    req = dict(prefill=np.zeros(len(q), np.uint32), len_tokens=np.full(len(q), bt, np.uint32),
               hash_off=np.arange(len(q) + 1, dtype=np.uint64), hashes=q)
    out = sel.select(nk.requests_to_device(req, sel.device), k=1, pairs=True)
    sel.sync_errors()
    got = nk.to_numpy(out["pairs"]["prefix_blocks"]).reshape(len(q), D)
    pos = np.minimum(np.searchsorted(uniq, q), max(0, len(uniq) - 1))
    hit = uniq[pos] == q if len(uniq) else np.zeros(len(q), bool)
    want = holds[np.where(hit, pos, len(uniq))]
    assert np.array_equal(got, want.astype(got.dtype))


@pytest.mark.parametrize("form", FORMS)
def test_membership(nk, form):
    """Resident hashes are found on exactly their decodes and nothing else
    is found, from host and from device arrays, on a handle of their own;
    then again on a handle whose buffers an index of another size, and one of
    the same size, left behind."""
    print("[gpu-case] index", form, flush=True)
    rng = np.random.default_rng(91)
    cfg = W.scaled(W.CONFIGS["c0"], n_requests=8, cache_per_decode=64)
    snap = W.make_snapshot(cfg, 3)
    sets, lf = _sets(form, rng)
    sel = nk.Selector(0)
    sel.load_snapshot(snap)
    _check(nk, sel, snap, sets, lf, rng, host=True)
    _check(nk, sel, snap, sets, lf, rng, host=False)
    other, lf2 = _sets("same" if form != "same" else "part", rng)
    _check(nk, sel, snap, other, lf2, rng, host=False)
    _check(nk, sel, snap, sets, lf, rng, host=False)
    # the reserved value is refused and the index stays
    bad = [x.copy() for x in sets]
    bad[-1] = np.concatenate([bad[-1], np.zeros(1, np.uint64)])
    before = nk.netkv_cache_info(sel.h)
    off = np.zeros(D + 1, np.uint64)
    off[1:] = np.cumsum([len(x) for x in bad])
    with pytest.raises(nk.NetKVError):
        nk.netkv_cache_load(sel.h, D, nk.to_device(off, sel.device), nk.to_device(np.concatenate(bad), sel.device), lf,
                            sel.device)
    assert nk.netkv_cache_info(sel.h) == before
    sel.close()


def test_load_waits_for_selections_on_other_streams(nk):
    """A selection in flight on one stream keeps the index it was called
    with while another stream loads one of the same size (whose buffers it
    takes over)."""
    print("[gpu-case] index load beside a selection", flush=True)
    rng = np.random.default_rng(5)
    cfg = W.scaled(W.CONFIGS["c0"], n_requests=200000, cache_per_decode=4096)
    snap = W.make_snapshot(cfg, 3)
    ch = W.prefix_chains(cfg, 3)
    req, cache = W.make_requests(cfg, 3, chains=ch), W.make_caches(cfg, 3, chains=ch)
    sel = nk.Selector(0)
    sel.load_snapshot(snap)
    sel.load_cache(cache, 0.5)
    rd = nk.requests_to_device(req, sel.device)
    want = sel.select(rd, k=1)
    want = [nk.to_numpy(want["idx"]), nk.to_numpy(want["score"])]
    off = nk.to_device(cache["hash_off"].astype(np.uint64), sel.device)
    other = nk.to_device(_u64(rng, len(cache["hashes"])), sel.device)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        outs = [sel.select(rd, k=1) for _ in range(20)]
    with torch.cuda.stream(b):
        nk.netkv_cache_load(sel.h, D, off, other, 0.5, sel.device)
    torch.cuda.synchronize()
    for o in outs:
        assert np.array_equal(nk.to_numpy(o["idx"]), want[0])
        assert np.array_equal(nk.to_numpy(o["score"]).view(np.uint32), want[1].view(np.uint32))
    sel.close()


def _crowd(n, first=0):
    """Hashes whose mixed values (the hash times the odd multiplier 0x9E37...15)
    are neighbours: all of them fall in one part and one block of the set."""
    inv = np.uint64(pow(0x9E3779B97F4A7C15, -1, 1 << 64))
    with np.errstate(over="ignore"):
        return (np.arange(1, n + 1, dtype=np.uint64) + (np.uint64(first) << np.uint64(40))) * inv


@pytest.mark.parametrize("crowd", [3000, 5000, 20000])
def test_crowded_sets(nk, crowd):
    """Hashes that crowd in one block among ordinary ones: more of them than the
    block's second buckets can take (3,000) and than the part has slots (5,000
    and 20,000).  Such a set is built whole: membership, and the selections
    that look hashes up in their own ways (direct, bounded, sequential) against
    the ordering pipeline; then an ordinary set on the same handle."""
    print("[gpu-case] crowded set", crowd, flush=True)
    rng = np.random.default_rng(17)
    cfg = W.scaled(W.CONFIGS["c0"], n_requests=8, cache_per_decode=64)
    snap = W.make_snapshot(cfg, 3)
    x = _crowd(crowd)
    sets = [np.concatenate([_u64(rng, 22000), x[d * crowd // 64:d * crowd // 64 + crowd // 4]]) for d in range(D)]
    sel = nk.Selector(0)
    sel.load_snapshot(snap)
    also = np.concatenate([rng.choice(x, 800), _crowd(300, 1)])
    _check(nk, sel, snap, sets, 0.5, rng, True, also)
    _check(nk, sel, snap, sets, 0.5, rng, False, also)
    bt, n = int(snap["block_tokens"]), 20000
    runs = [sets[rng.integers(D)][a:a + int(rng.integers(1, 40))] for a in rng.integers(21900, 22000 + crowd // 4 - 40, n)]
    ln = np.array([len(r) for r in runs])
    req = dict(prefill=rng.integers(0, cfg.n_prefill, n).astype(np.uint32), len_tokens=(ln * bt).astype(np.uint32),
               hash_off=np.concatenate([[0], np.cumsum(ln)]).astype(np.uint64), hashes=np.concatenate(runs))
    for m in (2000, n):
        part = dict(req, prefill=req["prefill"][:m], len_tokens=req["len_tokens"][:m], hash_off=req["hash_off"][:m + 1],
                    hashes=req["hashes"][:int(req["hash_off"][m])])
        rd = nk.requests_to_device(part, sel.device)
        got = []
        for run_len in (0, 8):   # an explicit run length asks for the ordering pipeline
            nk.netkv_set_option(sel.h, nk.NETKV_OPT_RUN_LEN, run_len)
            o, q = sel.select(rd, k=3), sel.select_sequential(rd, 16)
            got.append([nk.to_numpy(v[key]).view(np.uint32).copy() for v in (o, q) for key in ("idx", "score")])
        nk.netkv_set_option(sel.h, nk.NETKV_OPT_RUN_LEN, 0)
        sel.sync_errors()
        assert all(np.array_equal(a, b) for a, b in zip(*got))
    _check(nk, sel, snap, [rng.permutation(s[:9000]) for s in sets], 0.5, rng, False)
    sel.close()


def _windows(dev, width, stride):
    """Per decode a window of `width` of a sequence of distinct hashes (the
    finaliser of splitmix64 of the position, a bijection), `stride` apart."""
    x = torch.arange(1, (D - 1) * stride + width + 1, device=dev)
    for s, m in ((30, 0xBF58476D1CE4E5B9), (27, 0x94D049BB133111EB)):
        x = (x ^ ((x >> s) & ((1 << (64 - s)) - 1))) * (m - (1 << 64))
    x = x ^ ((x >> 31) & ((1 << 33) - 1))
    return x, x.unfold(0, width, stride).reshape(-1)


@pytest.mark.parametrize("form", ["0.79", "0.82", "0.849", "parts of 2^12 buckets"])
def test_large_sets(nk, form):
    """Sets of thousands of blocks near the largest occupancy: as planned up to
    0.80, twice the buckets beyond; and one of more than 2^27 hashes, whose
    parts and blocks are of 2^12 buckets."""
    print("[gpu-case] large set", form, flush=True)
    dev = torch.device("cuda", 0)
    cfg = W.scaled(W.CONFIGS["c0"], n_requests=8, cache_per_decode=64)
    snap = W.make_snapshot(cfg, 3)
    if form.startswith("0."):
        lf, occ = 0.85, float(form)
        stride = int(occ * (1 << 23)) // D
        width, slots = stride, (1 << 23) * (2 if occ > 0.8 else 1)
    else:
        lf, stride, width, slots = 0.5, 2850000, 2950000, 1 << 29
    seq, hashes = _windows(dev, width, stride)
    off = torch.arange(D + 1, device=dev) * width
    sel = nk.Selector(0)
    sel.load_snapshot(snap)
    nk.netkv_cache_load(sel.h, D, off.view(torch.uint64), hashes.view(torch.uint64), lf, dev)
    n = len(seq)
    ci = nk.netkv_cache_info(sel.h)
    assert ci["distinct_hashes"] == n and ci["index_slots"] == slots
    assert ci["shared_hashes"] == (D - 1) * (width - stride)
    g = torch.Generator(device=dev)
    g.manual_seed(4)
    at = torch.randint(0, n, (40000,), generator=g, device=dev)
    q = torch.cat([seq[at], torch.randint(1, 1 << 62, (2000,), generator=g, device=dev)])
    m = len(q)
    req = dict(prefill=torch.zeros(m, dtype=torch.int32, device=dev).view(torch.uint32),
               len_tokens=torch.full((m,), int(snap["block_tokens"]), dtype=torch.int32, device=dev).view(torch.uint32),
               hash_off=torch.arange(m + 1, device=dev).view(torch.uint64), hashes=q.view(torch.uint64))
    out = sel.select(req, k=1, pairs=True)
    sel.sync_errors()
    got = nk.to_numpy(out["pairs"]["prefix_blocks"]).reshape(m, D)
    pos, d = at.cpu().numpy()[:, None], np.arange(D)[None, :]
    want = np.zeros((m, D), got.dtype)
    want[:len(pos)] = (pos >= d * stride) & (pos < d * stride + width)
    assert np.array_equal(got, want)
    sel.close()
