"""The selections without ordering -- direct (small batches, one launch) and
bounded (the others) -- against the ordering pipeline on the same handle:
every output bit for bit, over pool sizes around the 64-decode groups and the
column chunks, one and four wavefronts per request, factors computed in place
and read from the derived rows.  An explicit run length asks for the
pipeline."""
import numpy as np
import pytest

from paper_2606_03910_amd import workload as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _shape(D, P=3):
    """A snapshot and caches over P prefills and D decodes cut from a larger cluster."""
    nodes = -(-max(D, 3 * P) // 6)
    cl = W.Cluster(8, 4, 4, -(-nodes // 16))
    return W.scaled(W.CONFIGS["c0"], cluster=cl)


def _inputs(D, R, seed, law="lognormal", mem=(20, 200), inflight="random", per=600, bt=512):
    cfg = W.scaled(_shape(D), n_requests=R, length_law=law, free_mem_gb=mem, block_tokens=bt, n_prefixes=40)
    P0, D0 = cfg.n_prefill, cfg.n_decode
    P = min(P0, 5)
    snap = W.make_snapshot(cfg, seed, inflight=inflight)
    cut = lambda a: np.ascontiguousarray(a.reshape(P0, D0)[:P, :D]).reshape(-1)
    snap.update(n_prefill=P, n_decode=D, tier_map=cut(snap["tier_map"]), util=cut(snap["util"]),
                n_inflight=np.ascontiguousarray(snap["n_inflight"].reshape(4, P0)[:, :P]).reshape(-1))
    for key in ("free_mem", "queue_depth", "batch_size"):
        snap[key] = snap[key][:D]
    ch = W.prefix_chains(cfg, seed)
    cache = W.make_caches(cfg, seed, chains=ch, n_decode=D, per_decode=per)
    req = W.make_requests(cfg, seed, chains=ch)
    req["prefill"] = (req["prefill"] % P).astype(np.uint32)
    return snap, cache, req


def _handle(netkv, snap, cache):
    sel = netkv.Selector(0)
    sel.load_snapshot(snap)
    sel.load_cache(cache, 0.5)
    return sel


def _bits(netkv, out):
    return netkv.to_numpy(out["idx"]).copy(), netkv.to_numpy(out["score"]).view(np.uint32).copy()


@pytest.mark.parametrize("D", [1, 2, 63, 64, 65, 256, 257, 768, 769, 1030, 3072])
@pytest.mark.parametrize("R", [1, 3, 70, 2049])
def test_direct_equals_pipeline(D, R):
    from paper_2606_03910_amd import netkv
    # runs of up to 63 blocks at 512 tokens, and of many 64-block steps at 16
    for bt, law in ((512, "lognormal"), (64, "lognormal")):
        snap, cache, req = _inputs(D, R, D + R, law=law, bt=bt)
        sel = _handle(netkv, snap, cache)
        if R > 1:
            req["prefill"][R // 2] = 1 << 20   # an invalid request
        rd = netkv.requests_to_device(req, sel.device)
        for k in (1, 2, 3, 8):
            got = _bits(netkv, sel.select(rd, k=k))
            netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_RUN_LEN, 8)
            want = _bits(netkv, sel.select(rd, k=k))
            netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_RUN_LEN, 0)
            print("[direct] D", D, "R", R, "bt", bt, "k", k, flush=True)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        sel.close()


def _grown(rng, req, cache, P, bt):
    """The batch with an invalid request, requests of 2^24 tokens and more, runs
    that one decode alone holds (and a hash 0 in one), and a run longer than 64
    blocks of a decode's private ones."""
    runs = [req["hashes"][int(req["hash_off"][r]):int(req["hash_off"][r + 1])] for r in range(len(req["prefill"]))]
    length, pre = list(req["len_tokens"]), list(req["prefill"])
    off = cache["hash_off"].astype(np.int64)
    for _ in range(24):
        d = int(rng.integers(len(off) - 1))
        own = cache["hashes"][off[d]:off[d + 1]]
        a = int(rng.integers(max(1, len(own) - 200)))
        run = own[a:a + int(rng.integers(1, 200))].copy()
        if rng.random() < 0.3:
            run[len(run) // 2] = 0
        runs.append(run)
        length.append(len(run) * bt + int(rng.integers(bt)))
        pre.append(int(rng.integers(P)))
    for x in (1 << 24, (1 << 24) - 1, (1 << 24) + 77):
        n = x // bt
        run = rng.integers(1, 1 << 63, n, dtype=np.uint64)
        run[:7] = runs[0][:7] if len(runs[0]) >= 7 else run[:7]
        runs.append(run)
        length.append(x)
        pre.append(int(rng.integers(P)))
    pre[len(pre) // 2] = 1 << 20
    n = np.array([len(r) for r in runs])
    return dict(prefill=np.array(pre, np.uint32), len_tokens=np.array(length, np.uint32),
                hash_off=np.concatenate([[0], np.cumsum(n)]).astype(np.uint64), hashes=np.concatenate(runs))


@pytest.mark.parametrize("D", [1, 48, 64, 65, 130, 768, 1602, 3072, 4096])
@pytest.mark.parametrize("mem,bt,routes", [((20, 200), 512, False), ((1, 30), 64, False), ((2, 200), 512, True)])
def test_bounded_equals_pipeline(D, mem, bt, routes):
    from paper_2606_03910_amd import netkv
    R = (1 << 14) // (-(-D // 64)) + 41
    snap, cache, req = _inputs(D, R, D, mem=mem, bt=bt)
    P = snap["n_prefill"]
    rng = np.random.default_rng(D)
    req = _grown(rng, req, cache, P, bt)
    sel = _handle(netkv, snap, cache)
    if routes:
        n = P * D
        sel.load_routes(rng.integers(1, 4, n), rng.uniform(0, 0.9, n), rng.integers(0, 2, n), rng.uniform(0, 0.9, n))
    rd = netkv.requests_to_device(req, sel.device)
    for k, policy in ((1, 0), (1, 2), (2, 0), (3, 1), (8, 0)):
        sel.set_policy(policy)
        auto = _bits(netkv, sel.select(rd, k=k))
        netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_FORM, 2)
        got = _bits(netkv, sel.select(rd, k=k))
        assert netkv.netkv_last_form(sel.h) == 2
        netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_FORM, 0)
        assert np.array_equal(got[0], auto[0]) and np.array_equal(got[1], auto[1])
        netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_RUN_LEN, 64)
        want = _bits(netkv, sel.select(rd, k=k))
        netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_RUN_LEN, 0)
        print("[bounded] D", D, "R", R, "mem", mem, "bt", bt, "routes", routes, "k", k, flush=True)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    sel.close()


def test_bounded_ties_and_rejects():
    """Identical decodes (every group survives the bound, ties go to the lowest
    index) and pools where nothing is feasible."""
    from paper_2606_03910_amd import netkv
    D, R = 1602, 700
    snap, cache, req = _inputs(D, R, 11)
    P = snap["n_prefill"]
    snap.update(tier_map=np.full(P * D, 2, np.uint8), util=np.zeros(P * D, np.float32),
                queue_depth=np.zeros(D, np.uint32), free_mem=np.full(D, 10 ** 12, np.uint64))
    for m_min in (0, 1 << 62):
        snap["m_min"] = m_min
        sel = _handle(netkv, snap, dict(hash_off=np.zeros(D + 1, np.uint64), hashes=np.ones(1, np.uint64)))
        netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_FORM, 2)
        rd = netkv.requests_to_device(req, sel.device)
        for k in (1, 3, 8):
            i, s = _bits(netkv, sel.select(rd, k=k))
            if m_min:
                assert np.all(i == -1) and np.all(s == np.float32(np.inf).view(np.uint32))
            else:
                assert np.array_equal(i.reshape(R, k), np.tile(np.arange(k), (R, 1)))
        sel.close()


@pytest.mark.parametrize("D", [48, 90, 800])
def test_direct_forms(D):
    """Staged routes, policies, memory pressure, records for the sweep and the
    sequential form."""
    from paper_2606_03910_amd import netkv
    R = 300
    snap, cache, req = _inputs(D, R, 7, mem=(1, 4))
    P = snap["n_prefill"]
    sel = _handle(netkv, snap, cache)
    rd = netkv.requests_to_device(req, sel.device)
    util = torch.from_numpy(np.random.default_rng(3).uniform(0, 0.9, (9, P * D)).astype(np.float32)).to(sel.device).reshape(-1)

    def calls():
        o = [*_bits(netkv, sel.select(rd, k=2))]
        sw = sel.rank_sweep(rd, util, 3)
        o += [*_bits(netkv, sw), netkv.to_numpy(sw["flips"]).copy(), netkv.to_numpy(sw["inversions"]).copy()]
        o += [*_bits(netkv, sel.select_sequential(rd, 16))]
        return o
    for policy in (0, 1, 2):
        sel.set_policy(policy)
        for routes in (False, True):
            if routes:
                rng = np.random.default_rng(5)
                n = P * D
                sel.load_routes(rng.integers(1, 4, n), rng.uniform(0, 0.9, n), rng.integers(0, 2, n), rng.uniform(0, 0.9, n))
            else:
                sel.clear_routes()
            got = calls()
            netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_RUN_LEN, 8)
            want = calls()
            netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_RUN_LEN, 0)
            print("[direct] forms D", D, "policy", policy, "routes", routes, flush=True)
            assert all(np.array_equal(a, b) for a, b in zip(got, want))
    sel.close()


@pytest.mark.parametrize("D", [48, 5440, 5600])
@pytest.mark.parametrize("R", [1, 64, 5000])
def test_commit_forms(D, R):
    """The between-batch update against the oracle on pools whose sums fit a
    workgroup's LDS (12 D + 16 P bytes of 64 KiB: 5,440 decodes and 5 prefills
    take 65,360) and on one beyond, with rejected requests; twice, so that the
    admitted bytes come back; then an invalid request and an index past the
    pool."""
    import oracle
    from paper_2606_03910_amd import netkv
    snap, cache, req = _inputs(D, R, D + R, bt=64)
    P = snap["n_prefill"]
    assert P == 5
    rng = np.random.default_rng(R)
    sel = _handle(netkv, snap, cache)
    oc = oracle.Cache(cache, n_threads=8)
    state = dict(n_inflight=snap["n_inflight"].copy(), queue_depth=snap["queue_depth"].copy(),
                 free_mem=snap["free_mem"].copy(), admitted_prev=np.zeros(D, np.uint64))
    rd = netkv.requests_to_device(req, sel.device)
    for step in range(2):
        idx = rng.integers(-1, D, R).astype(np.int32)
        idx[:R // 2] = rng.integers(0, 3, R // 2)   # many on few counters
        print("[gpu-case] commit D", D, "R", R, "step", step, flush=True)
        sel.commit(rd, netkv.to_device(idx, sel.device), 16, 7)
        sel.sync_errors()
        state = oracle.commit(dict(snap, **{k: state[k] for k in ("n_inflight", "queue_depth", "free_mem")}), oc, req, idx,
                              16, 7, state)
        got = sel.state()
        for key in ("n_inflight", "queue_depth", "free_mem", "admitted_prev"):
            np.testing.assert_array_equal(got[key], state[key], err_msg=key)
    # what the update refuses changes nothing else
    before = sel.state()
    bad = dict(req, prefill=req["prefill"].copy())
    bad["prefill"][0] = 1 << 20
    idx = np.full(R, -1, np.int32)
    idx[0], idx[-1] = 0, D if R > 1 else 0
    sel.commit(netkv.requests_to_device(bad, sel.device), netkv.to_device(idx, sel.device), 16, 0)
    with pytest.raises(netkv.NetKVError):
        sel.sync_errors()
    got = sel.state()
    assert np.all(got["n_inflight"] == 0) and np.array_equal(got["queue_depth"], before["queue_depth"])
    assert np.all(got["admitted_prev"] == 0)
    sel.close()


@pytest.mark.parametrize("D", [1, 48, 65, 768, 1602, 3072])
def test_long_runs(D):
    """Runs of up to 5,000 held blocks, cut at different blocks on different
    decodes (about every multiple of 64 and 128), some with a tail that one
    decode alone holds, in the middle or at the end of the batch: the direct
    and the bounded selection, the records of the sequential form and the
    ranking sweep against the ordering pipeline."""
    from paper_2606_03910_amd import netkv
    rng = np.random.default_rng(D)
    bt = 64
    snap, _, _ = _inputs(D, 4, D, bt=bt, mem=(20, 200))
    P = snap["n_prefill"]
    cuts = np.array([1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 319, 320, 321, 511, 512, 513, 1000, 4999, 5000])
    chains = [rng.integers(1, 1 << 63, 5000, dtype=np.uint64) for _ in range(3)]
    sets = []
    for d in range(D):
        own = [c[:rng.choice(cuts)] for c in chains if rng.random() < 0.5]
        if d == D // 2:
            own.append(chains[0])
        sets.append(np.concatenate(own + [rng.integers(1, 1 << 63, 5, dtype=np.uint64)]))
    off = np.zeros(D + 1, np.uint64)
    off[1:] = np.cumsum([len(x) for x in sets])
    sel = _handle(netkv, snap, dict(hash_off=off, hashes=np.concatenate(sets)))

    def batch(n):
        runs = []
        for _ in range(n):
            c = chains[rng.integers(3)][:rng.choice(cuts)] if rng.random() < min(1.0, 300 / n) else chains[0][:rng.integers(1, 30)]
            runs.append(np.concatenate([c, rng.integers(1, 1 << 63, int(rng.integers(0, 200)) if len(c) > 60 else 0, dtype=np.uint64)]))
        ln = np.array([len(r) for r in runs])
        return dict(prefill=rng.integers(0, P, n).astype(np.uint32), len_tokens=(ln * bt + rng.integers(0, bt, n)).astype(np.uint32),
                    hash_off=np.concatenate([[0], np.cumsum(ln)]).astype(np.uint64), hashes=np.concatenate(runs))
    util = torch.from_numpy(rng.uniform(0, 0.9, (3, P * D)).astype(np.float32)).to(sel.device).reshape(-1)
    for n in (1, 7, 150, 20000 // (-(-D // 64)) + 50):
        rd = netkv.requests_to_device(batch(n), sel.device)
        for k in (1, 3, 8):
            both = []
            for run_len in (0, 0, 8):
                netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_RUN_LEN, run_len)
                netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_FORM, 2 if len(both) == 1 else 0)
                out = sel.select(rd, k=k)
                both.append([*_bits(netkv, out)])
                if k == 1:
                    both[-1] += [*_bits(netkv, sel.select_sequential(rd, 16)), *_bits(netkv, sel.rank_sweep(rd, util, 2))]
            netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_RUN_LEN, 0)
            print("[direct] long runs D", D, "R", n, "k", k, flush=True)
            assert all(np.array_equal(a, b) and np.array_equal(a, c) for a, b, c in zip(*both))
    sel.sync_errors()
    sel.close()


@pytest.mark.parametrize("form", ["identical", "one tier", "tiers"])
def test_form_follows_the_snapshot(form):
    """A snapshot whose groups of 64 decodes the bounds cannot tell apart is
    selected along the batch order, which bounds would take several times as
    long for (150,001 requests on 3,072 identical decodes: 1,378 us against 285);
    one of distinct tiers by bounds.  The selections agree in every form."""
    from paper_2606_03910_amd import netkv
    D, R = 3072, 60000
    snap, cache, req = _inputs(D, R, 3)
    P = snap["n_prefill"]
    rng = np.random.default_rng(8)
    if form == "identical":
        snap.update(tier_map=np.full(P * D, 2, np.uint8), util=np.zeros(P * D, np.float32),
                    queue_depth=np.zeros(D, np.uint32), batch_size=np.zeros(D, np.uint32))
    elif form == "one tier":
        snap.update(tier_map=np.full(P * D, 3, np.uint8), util=rng.uniform(0, 0.9, P * D).astype(np.float32))
    sel = _handle(netkv, snap, cache)
    rd = netkv.requests_to_device(req, sel.device)
    out = {}
    for how in (0, 1, 2):
        netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_FORM, how)
        out[how] = _bits(netkv, sel.select(rd, k=1))
        took = netkv.netkv_last_form(sel.h)
        assert took == (how or (2 if form == "tiers" else 1)), (form, how, took)
    print("[gpu-case] form", form, flush=True)
    assert all(np.array_equal(out[0][i], out[h][i]) for h in (1, 2) for i in (0, 1))
    # a congestion map alone does not tell one tier's groups apart either
    if form == "one tier":
        sel.set_util(np.zeros(P * D, np.float32))
        netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_FORM, 0)
        sel.select(rd, k=1)
        assert netkv.netkv_last_form(sel.h) == 1
    netkv.netkv_set_option(sel.h, netkv.NETKV_OPT_FORM, 0)
    sel.select(netkv.requests_to_device(_inputs(D, 100, 3)[2], sel.device), k=1)
    assert netkv.netkv_last_form(sel.h) == 3
    sel.close()
