"""Steps captured into a program's own graphs, and scans selected around them."""
import math

import numpy as np
import pytest
import torch

from paper_2606_15846_amd import navsim
from paper_2606_15846_amd.navsim import NavSim
from workloads import configs
from workloads import maps as gm

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


# the second shape's 360 sectors leave 32-env tiles of 512 threads room for the
# traversal but not for the march
@pytest.mark.parametrize("n,side,beams,sectors", [(200, 128, 90, 30), (5000, 64, 360, 360)])
@pytest.mark.parametrize("inside", [False, True])
def test_captured_step_and_scan_selection(n, side, beams, sectors, inside):
    """A captured step keeps its scan and its tiles while others are selected; a
    scan can be selected during the capture.  Replays agree with eager steps of
    another handle."""
    say(f"captured steps: {n} envs, {beams} beams, {sectors} sectors, "
        f"scan selected {'inside' if inside else 'after'} the capture")
    cfg = configs.make_config(num_envs=n, num_beams=beams, num_sectors=sectors,
                              fov_rad=2 * math.pi, max_range_m=3.0, dt_s=0.1, footprint=0,
                              radius_m=0.15, v_min=0.0, v_max=0.5, w_min=-1.0, w_max=1.0)
    occ = [gm.gen_rect_disc_map(50 + k, w=side + k, h=side) for k in range(2)]
    sims = [NavSim(cfg, occ, [0.05] * 2, configs.contiguous_env_map(n, 2), device=0) for _ in "ab"]
    for s in sims:
        s.reset()
    acts = torch.from_numpy(configs.uniform_actions(1, n, seed=3)[0]).cuda()
    sims[1].set_scan(int(inside), 0.03)
    state = sims[0].get_state()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        if inside:
            sims[0].set_scan(navsim.NAVSIM_SCAN_MARCH, 0.03)
        sims[0].step(acts)
    for t in range(3):
        sims[0].set_scan(1 - t % 2, 0.03)
        for s in sims:
            s.set_state(state)
            s.obs.zero_()
            s.final_obs.zero_()
        graph.replay()
        sims[1].step(acts)
        torch.cuda.synchronize()
        for k in ("obs", "reward", "terminated", "truncated", "final_obs"):
            assert torch.equal(getattr(sims[0], k), getattr(sims[1], k)), (t, k)
        a, b = (s.get_state() for s in sims)
        for k in a:
            assert np.array_equal(a[k], b[k]), (t, k)
    for s in sims:
        s.close()
