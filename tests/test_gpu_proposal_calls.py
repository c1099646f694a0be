"""Proposal calls as programs overlap them on streams and capture them into graphs."""
import numpy as np
import pytest
import torch

from paper_2606_15846_amd.navsim import NavSim
from paper_2606_15846_amd.reset_proposal import ResetProposer
from workloads import configs

pytestmark = pytest.mark.gpu

KEYS = ("pose", "hops", "source", "checks")


def say(*a):
    print(*a, flush=True)


def make_sim(num_maps=4):
    w = configs.build_workload("c5", num_envs=64)
    return NavSim(w["cfg"], w["maps"][:num_maps], w["res"][:num_maps],
                  (np.arange(64) % num_maps).astype(np.int32), device=0), w["proposer"]


def requests(n, seed, num_maps=4):
    r = np.random.default_rng(seed)
    q = [r.integers(0, num_maps, n), r.integers(0, 8, n), r.integers(0, 1 << 20, n),
         r.integers(0, 50, n)]
    return [torch.from_numpy(v.astype(np.int32)).cuda() for v in q]


def outputs(n):
    z = dict(device="cuda", dtype=torch.int32)
    return dict(pose=torch.zeros(n, 5, device="cuda"), hops=torch.zeros(n, **z),
                source=torch.zeros(n, **z), checks=torch.zeros(n, **z))


def same(a, b):
    return all(torch.equal(a[k], b[k]) for k in KEYS)


def test_overlapping_rejection_only_noalloc_calls():
    """Two proposers' rejection-only noalloc calls of different sizes, in flight on
    two streams at once, give what each gives alone."""
    sim, cfg = make_sim()
    rps = [ResetProposer(sim, **dict(cfg, seed=s)) for s in (5, 6)]
    reqs = [requests(2000, 1), requests(150, 2)]
    say("rejection-only noalloc proposals: 2,000 and 150 requests on two streams")
    alone = [rp.propose_into(*q, 0, 64, outputs(q[0].numel())) for rp, q in zip(rps, reqs)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in rps]
    got = [[outputs(q[0].numel()) for _ in range(4)] for q in reqs]
    torch.cuda.synchronize()
    for t in range(4):
        for s, rp, q, o in zip(streams, rps, reqs, got):
            with torch.cuda.stream(s):
                rp.propose_into(*q, 0, 64, o[t], noalloc=True)
    torch.cuda.synchronize()
    for a, o in zip(alone, got):
        assert all(same(a, x) for x in o)
    for rp in rps:
        rp.close()
    sim.close()


def test_rejection_only_proposals_captured_first():
    """A proposer's first rejection-only call can be captured into a graph; every
    replay gives the eager call's pairs, eager calls in between."""
    sim, cfg = make_sim()
    rp = ResetProposer(sim, **cfg)
    q = requests(300, 3)
    got = outputs(300)
    torch.cuda.synchronize()
    say("rejection-only proposal captured: 300 requests")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rp.propose_into(*q, 0, 64, got)
    want = rp.propose_into(*q, 0, 64, outputs(300))
    for t in range(3):
        for v in got.values():
            v.zero_()
        graph.replay()
        rp.propose_into(*requests(500, t), 0, 16, outputs(500))
        torch.cuda.synchronize()
        assert same(got, want), t
    rp.close()
    sim.close()


@pytest.mark.parametrize("hidden", [64, 256])
def test_proposals_captured_with_more_attempts(hidden):
    """A call with network draws is captured after one with as many draws and no
    attempts has run; replays agree with the eager call, other calls in between."""
    sim, cfg = make_sim()
    rp = ResetProposer(sim, **dict(cfg, hidden=hidden))
    q = requests(260, 4)
    rp.propose_into(*q, 4, 0, outputs(260))
    got = outputs(260)
    torch.cuda.synchronize()
    say(f"proposal captured: 260 requests of 4 draws and 64 attempts, hidden width {hidden}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rp.propose_into(*q, 4, 64, got)
    want = rp.propose_into(*q, 4, 64, outputs(260))
    for t in range(3):
        for v in got.values():
            v.zero_()
        graph.replay()
        rp.propose_into(*requests(200, t), 5, 300, outputs(200))
        torch.cuda.synchronize()
        assert same(got, want), t
    rp.close()
    sim.close()


def test_labels_of_wide_maps_alone_and_beside_others():
    """Labels on maps that no register search holds, from a proposer of such maps
    alone and from one that has others too; unknown maps get none from either."""
    rng = np.random.default_rng(8)
    occ = [(rng.random(s) < 0.02).astype(np.uint8) for s in ((40, 1040), (36, 1100), (60, 200))]
    cfg = dict(configs.build_workload("c5", num_envs=6)["cfg"], radius_m=0.02)
    ids = np.array([0, 1, -1, 1, 0, 7, 1])
    got = []
    for maps in (occ[:2], occ):
        sim = NavSim(cfg, maps, [0.05] * len(maps), np.arange(6) % len(maps), device=0)
        rp = ResetProposer(sim, d_lo_m=0.5, d_hi_m=6.0)
        got.append({k: v.cpu().numpy() for k, v in rp.label(ids, first_sid=30).items()})
        rp.close()
        sim.close()
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
        assert (got[0][k][[2, 5]] == -1).all(), k
    assert (got[0]["goal"][[0, 1, 3, 4, 6]] >= 0).mean() > 0.5


def test_rejection_only_tail_agrees_with_one_launch():
    """Rejection-only calls on both sides of the tail's limits (one workgroup's
    pass, the widths of a round, the most requests it takes): a request's result
    does not depend on the call it is in.  8,193 requests are checked by one launch."""
    sim, cfg = make_sim()
    rp = ResetProposer(sim, **dict(cfg, d_hi_m=20.0))
    q = requests(8193, 9)
    q[0][::50] = 9  # unknown maps
    q[1][7::90] = -1  # no bin
    say("rejection-only proposals of 1 to 8,193 requests, 75 attempts")
    want = rp.propose_into(*q, 0, 75, outputs(8193))
    for n in (1, 63, 64, 65, 511, 2047, 2048, 2049, 4097, 8192):
        for noalloc in (False, True):
            got = rp.propose_into(*[v[:n].clone() for v in q], 0, 75, outputs(n), noalloc=noalloc)
            torch.cuda.synchronize()
            assert same(got, {k: want[k][:n] for k in KEYS}), (n, noalloc)
    src = want["source"].cpu().numpy()
    assert (src > 24).any() and (src == -1).any() and (want["checks"].cpu().numpy() == 75).any()
    rp.close()
    sim.close()
