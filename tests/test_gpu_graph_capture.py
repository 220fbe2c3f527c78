"""The allocation-free selection captured into a HIP graph and replayed:
every replay bit-identical to the allocating call.  A batch of 100,000
requests: a first sub-batch of 65,536 (which forks the handle's second
stream; the capture takes both branches) and a second of 34,464."""
import numpy as np
import pytest

from paper_2606_03910_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def nk():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_03910_amd import netkv
    netkv.load_library()
    return netkv


def test_noalloc_selection_replays_from_a_graph(nk):
    print("[gpu-case] graph capture of the allocation-free selection", flush=True)
    cfg = W.scaled(W.CONFIGS["c0"], n_requests=100000)
    snap = W.make_snapshot(cfg, 17, inflight="random")
    ch = W.prefix_chains(cfg, 17)
    req = W.make_requests(cfg, 17, chains=ch)
    cache = W.make_caches(cfg, 17, chains=ch)
    sel = nk.Selector(0)
    sel.load_snapshot(snap)
    sel.load_cache(cache, 0.5)
    rd = nk.requests_to_device(req, sel.device)
    k = 2
    n = cfg.n_requests
    ref = sel.select(rd, k=k)
    sel.sync_errors()
    ri, rs = nk.to_numpy(ref["idx"]), nk.to_numpy(ref["score"])
    bi = torch.empty(n * k, dtype=torch.int32, device=sel.device)
    bs = torch.empty(n * k, dtype=torch.float32, device=sel.device)
    nk.netkv_select_batch_noalloc(sel.h, rd, k, bi, bs, sel.device)   # eager once
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        nk.netkv_select_batch_noalloc(sel.h, rd, k, bi, bs, sel.device)
    torch.cuda.synchronize()
    for rep in range(3):
        bi.fill_(-7)
        bs.fill_(-7.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        gi, gs = nk.to_numpy(bi), nk.to_numpy(bs)
        assert np.array_equal(gi, ri), f"replay {rep}: {int((gi != ri).sum())} selections differ"
        assert np.array_equal(gs.view(np.uint32), rs.view(np.uint32)), f"replay {rep}: scores differ"
        # eager work between replays
        sel.select(rd, k=1)
        torch.cuda.synchronize()
    sel.sync_errors()
    del g
    sel.close()


@pytest.mark.parametrize("how", ["select", "reserve"])
@pytest.mark.parametrize("n", [300, 100000])
def test_forms_share_their_buffers(nk, n, how):
    """One plain selection, or a reservation (whatever options are set then),
    sizes the work buffers for every form of a batch of its size: per-pair
    outputs, staged routes, the ordering pipeline and the bounds of another
    snapshot of the same decodes (with more prefills) are captured afterwards,
    where nothing can be allocated, and their replays equal another handle's
    eager results.  300 requests are selected directly, 100,000 by bounds."""
    print("[gpu-case] forms after one", how, n, flush=True)
    cfg = W.scaled(W.CONFIGS["c0"], n_requests=n, cluster=W.Cluster(8, 4, 4, 2))
    D = cfg.n_decode
    snap = W.make_snapshot(cfg, 17, inflight="random")
    ch = W.prefix_chains(cfg, 17)
    req = W.make_requests(cfg, 17, chains=ch)
    cache = W.make_caches(cfg, 17, chains=ch)
    P = cfg.n_prefill
    rng = np.random.default_rng(5)
    more = dict(snap, n_prefill=P + 3, n_inflight=rng.integers(0, 9, 4 * (P + 3)).astype(np.uint16))
    for key in ("tier_map", "util"):
        more[key] = np.concatenate([snap[key].reshape(P, D), snap[key].reshape(P, D)[:3]]).reshape(-1)

    def routes(sel, p):
        r = np.random.default_rng(6)
        sel.load_routes(r.integers(1, 4, p * D), r.uniform(0, 0.9, p * D), r.integers(0, 2, p * D), r.uniform(0, 0.9, p * D))
    ref, sel = nk.Selector(0), nk.Selector(0)
    for h in (ref, sel):
        h.load_snapshot(snap)
        h.load_cache(cache, 0.5)
    rd = nk.requests_to_device(req, sel.device)
    if how == "select":
        sel.select(rd, k=2)   # the only eager selection of this size
    else:
        nk.netkv_set_option(sel.h, nk.NETKV_OPT_RUN_LEN, 64)
        nk.netkv_reserve(sel.h, n, len(req["hashes"]), 2, sel.device)
    torch.cuda.synchronize()
    bi = torch.empty(n * 2, dtype=torch.int32, device=sel.device)
    bs = torch.empty(n * 2, dtype=torch.float32, device=sel.device)
    pp = dict(n_decode=D, prefix_blocks=torch.empty(n * D, dtype=torch.uint16, device=sel.device),
              feasible=torch.empty(n * D, dtype=torch.uint8, device=sel.device),
              score=torch.empty(n * D, dtype=torch.float32, device=sel.device))
    small = nk.requests_to_device(W.make_requests(W.scaled(cfg, n_requests=50), 18, chains=ch), sel.device)
    for step in ("plain", "pairs", "pipeline", "prefills", "routes"):
        for h in (ref, sel):
            nk.netkv_set_option(h.h, nk.NETKV_OPT_RUN_LEN, 64 if step == "pipeline" else 0)
            if step == "prefills":
                h.load_snapshot(more)
            if step == "routes":
                routes(h, P + 3)
        pairs = pp if step == "pairs" else None
        want = ref.select(rd, k=2, pairs=step == "pairs")
        ref.sync_errors()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            nk.netkv_select_batch(sel.h, rd, 2, bi, bs, pairs, sel.device)
        torch.cuda.synchronize()
        for rep in range(3):
            bi.fill_(-7)
            bs.fill_(-7.0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(bi, want["idx"]), (step, rep)
            assert torch.equal(bs.view(torch.int32), want["score"].view(torch.int32)), (step, rep)
            if pairs:
                for key in ("prefix_blocks", "feasible", "score"):
                    assert np.array_equal(nk.to_numpy(pp[key]).view(np.uint8), nk.to_numpy(want["pairs"][key]).view(np.uint8)), key
            sel.select(small, k=1)   # eager work between replays
            torch.cuda.synchronize()
        sel.sync_errors()
        del g
    ref.close()
    sel.close()
