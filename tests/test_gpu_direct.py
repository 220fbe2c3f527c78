"""The direct selection (small batches, one launch) against the ordering
pipeline on the same handle: every output bit for bit, over pool sizes around
the 64-decode groups and the column chunks, one and four wavefronts per
request, factors computed in place and read from the derived rows.  An
explicit run length asks for the pipeline."""
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
