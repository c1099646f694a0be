"""What the library's host code asks of the HIP runtime, on the CPU (see
stand_in.py): which kernels a call launches, what it allocates, frees and waits
for, and what is left when an allocation fails."""
import pytest

from tests import stand_in


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("stand_in")
    return lambda body: stand_in.run(tmp, body)


def test_rejection_only_noalloc_calls_keep_off_the_shared_array(run):
    """The rejection sampler alone takes nothing from the array that all proposers
    of a device share, whatever it launches (calls with network draws do)."""
    run("""
    r = proposer(handle(8, [(256, 256)] * 3))
    for n in (1, 31, 200, 3000, 8192):
        for tries in (0, 1, 16, 64, 5000):
            clear()
            assert propose(r, n, 0, tries, noalloc=True) == 0
            assert launches()[0] == "propose_kernel<%d>" % (8 if n <= 2048 else 4), (n, tries)
            assert counts()[1:4] == (0, 0, 0)
            assert R.stand_in_scratch_pointers() == 0, (n, tries)
    clear()
    assert propose(r, 200, 8, 64, noalloc=True) == 0
    assert R.stand_in_scratch_pointers() > 0
    """)


def test_rejection_only_proposals_need_no_workspace(run):
    """Rejection-only calls allocate nothing and work during a stream capture and
    with no device memory left, whatever their size."""
    run("""
    r = proposer(handle(8, [(256, 256)] * 3))
    R.stand_in_capturing(1)
    R.stand_in_fail_malloc(0)
    for n in (1, 31, 200, 3000, 8192):
        for tries in (0, 16, 64, 5000):
            clear()
            assert propose(r, n, 0, tries) == 0, lib.navsim_last_error()
            assert counts()[1:4] == (0, 0, 0)
    """)


def test_rejection_only_tail_where_its_state_fits(run):
    """The tail launches run where the requests' state fits their output rows: at
    least two rounds left, attempt numbers below 2^16, and arrays that share no
    memory; elsewhere one launch checks every round."""
    run("""
    def kernels_of(n, tries, alias=None):
        v = [np.zeros(n, np.int32) for _ in range(7)]
        if alias:
            v[alias[0]] = v[alias[1]]
        pose = np.zeros((n, 5), np.float32)
        clear()
        assert lib.navsim_rp_propose(r, n, *[a.ctypes.data for a in v[:4]], 0, tries, pose.ctypes.data,
                                     *[a.ctypes.data for a in v[4:]], None, None) == 0
        return launches()
    r = proposer(handle(8, [(256, 256)] * 3))
    for n, W, head in ((64, 8, 1), (2048, 8, 1), (2049, 4, 3)):
        one = ["propose_kernel<%d>" % W]
        three = one + ["propose_tail_own_kernel<%d>" % W, "propose_final_own_kernel"]
        assert kernels_of(n, W * (head + 1)) == one
        assert kernels_of(n, W * (head + 1) + 1) == three
        assert kernels_of(n, 400) == three
        for alias in ((4, 5), (4, 6), (5, 6)):
            assert kernels_of(n, 400, alias) == one
    assert kernels_of(64, 65535) == ["propose_kernel<8>", "propose_tail_own_kernel<8>",
                                     "propose_final_own_kernel"]
    assert kernels_of(64, 65536) == ["propose_kernel<8>"]
    assert kernels_of(4096, 65535) == ["propose_kernel<4>"]  # more than 2^22 rounds
    assert kernels_of(8192, 400) == three and kernels_of(8193, 400) == one
    """)


def test_more_attempts_need_no_more_workspace(run):
    """The workspace of a call with network draws depends on requests times draws
    alone, as its activations' does: once a call has run, one with the same draws
    and any number of attempts can be captured, and a captured call's workspace
    stays where it is."""
    run("""
    for hidden in (64, 256):
        h = handle(8, [(256, 256)] * 3)
        for n, proposals in ((1, 1), (100, 8), (128, 1), (256, 8), (2000, 32), (4096, 2), (70000, 1)):
            r = proposer(h, hidden=hidden)
            assert propose(r, n, proposals, 0) == 0
            R.stand_in_capturing(1)
            for tries in (16, 64, 100, 512, 5000, 100000):
                clear()
                assert propose(r, n, proposals, tries) == 0, (n, proposals, tries)
                assert counts()[1:4] == (0, 0, 0), (n, proposals, tries)
            # the usual calls are still split into head and tail launches
            clear()
            assert propose(r, n, proposals, 64) == 0
            assert ("propose_final_kernel" in launches()) == (n >= 128), launches()
            # fewer requests of as many draws in all
            clear()
            assert propose(r, max(1, n // 2), proposals, 64) == 0
            assert counts()[1:4] == (0, 0, 0)
            R.stand_in_capturing(0)
            assert lib.navsim_rp_destroy(r) == 0
    """)


def test_attach_limit_counts_every_round_after_the_first(run):
    """navsim_rp_attach refuses more than 2^24 rounds of candidates after each
    request's first, whatever the width of a round."""
    run("""
    h = handle(4096, [(256, 256)])
    r = proposer(h)
    bins = np.zeros(4096, np.int32)
    attach = lambda proposals, tries, cap: lib.navsim_rp_attach(r, bins.ctypes.data, proposals, tries, cap)
    # 4 candidates a round past 2,048 requests a step, 8 up to there
    for cap, width in ((4096, 4), (2048, 8)):
        most = width * ((1 << 24) // cap + 1)
        assert attach(8, most - 8, cap) == 0
        clear()
        assert attach(8, most - 7, cap) == -1
        assert counts().malloc == 0
        assert lib.navsim_rp_detach(r) == 0
    """)


def test_labels_of_wide_maps_take_one_launch(run):
    """Maps that no register search holds are labelled by one launch, mixed sets by
    two, the others by one."""
    run("""
    def label(sides):
        r = proposer(handle(8, sides))
        m = np.arange(40, dtype=np.int32) % len(sides)
        o = np.zeros((3, 40, 8), np.int32)
        clear()
        assert lib.navsim_rp_label(r, 40, m.ctypes.data, 0, *[o[i].ctypes.data for i in range(3)], None) == 0
        assert counts()[1:4] == (0, 0, 0)
        return launches()
    assert label([(256, 256)] * 2) == ["label_wave_kernel"]
    assert label([(1040, 40)] * 2) == ["label_kernel"]
    assert label([(256, 256), (1040, 40)]) == ["label_wave_kernel", "label_kernel"]
    """)


# shapes on both sides of what a launch shape's LDS holds, of either scan
SCAN_SHAPES = """
    shapes = [(n, side, s, per * s) for n in (1, 64, 5000) for side in (64, 128, 256, 384, 512, 600)
              for s in (1, 36, 180, 360, 720) for per in (1, 4)]
"""


def test_set_scan_leaves_the_envs_and_the_device_alone(run):
    """Selecting a scan regroups no envs, frees nothing and waits for nothing, so
    launches in flight or captured stay valid; it works during a stream capture,
    and the launch shape stays as loaded."""
    run(SCAN_SHAPES + """
    seen = set()
    for n, side, sectors, beams in shapes:
        for first in (0, 1):
            h = ns.navsim_create(configs.make_config(
                num_envs=n, num_beams=beams, num_sectors=sectors, fov_rad=6.28, max_range_m=4.0,
                dt_s=0.1, footprint=0, radius_m=0.18, v_min=0.0, v_max=0.5, w_min=-1.0, w_max=1.0))
            assert lib.navsim_set_scan(h, first, 0.03) == 0
            try:
                load(h, n, [(side, side)])
            except ns.NavsimError as e:
                assert e.status == -7
                lib.navsim_destroy(h)
                continue
            obs = np.zeros((n, sectors + 4), np.float32)
            assert lib.navsim_reset(h, None, obs.ctypes.data, None) == 0
            shape = ns.navsim_get_tuning(h)
            for scan in (1 - first, first, 1 - first):
                clear()
                R.stand_in_capturing(1)
                rc = lib.navsim_set_scan(h, scan, 0.03)
                assert rc in (0, -7), lib.navsim_last_error()
                c = counts()
                assert (c.launches, c.free, c.sync) == (0, 0, 0), (n, side, sectors, c)
                seen.add((scan, rc, c.malloc))
                assert step(h, n, sectors) == 0
                R.stand_in_capturing(0)
                assert ns.navsim_get_tuning(h) == shape
            assert lib.navsim_destroy(h) == 0
    # refused, with clearances to build, built already or without, both scans
    assert {(1, 0, 0), (1, 0, 1), (1, -7, 0), (0, 0, 0)} <= seen, seen
    """)


def test_march_without_memory_for_clearances(run):
    """The march needs no device memory: without the clearances every sample is
    evaluated (and they are built once a later selection finds the memory)."""
    run("""
    march = lambda: (clear(), step(h, 64), launches())[2][0]
    h = handle(64, [(128, 128)] * 2, beams=360)
    R.stand_in_fail_malloc(0)
    assert lib.navsim_set_scan(h, 1, 0.03) == 0
    assert march() == "fused_step_kernel<32, 1024, false, false>"
    t = ns.NavsimTuning(8, 40, 8, 0, 3, 0, 256, 0)
    R.stand_in_fail_malloc(-1)
    R.stand_in_fail_one_malloc(0)
    assert lib.navsim_set_tuning(h, C.byref(t)) == 0
    assert march() == "fused_step_kernel<8, 256, false, false>"
    assert lib.navsim_set_scan(h, 1, 0.03) == 0
    assert march() == "fused_step_kernel<8, 256, false, true>"
    R.stand_in_fail_one_malloc(7)  # after what a load of maps takes otherwise
    load(h, 64, [(100, 100)] * 2)
    assert lib.navsim_reset(h, None, np.zeros((64, 40), np.float32).ctypes.data, None) == 0
    assert march() == "fused_step_kernel<8, 256, false, false>"
    """)


def test_launch_shape_without_memory_leaves_the_handle_as_it_was(run):
    """A launch shape whose tiles cannot be put on the device is refused: the old
    tiles are neither freed nor replaced, and the next one starts from them."""
    run("""
    h = handle(300, [(64, 64)] * 3)
    t = ns.NavsimTuning(4, 40, 8, 0, 3, 0, 256, 0)
    before = ns.navsim_get_tuning(h)
    for nth in (0, 1):  # the order of the envs, the tiles
        clear()
        R.stand_in_fail_one_malloc(nth)
        assert lib.navsim_set_tuning(h, C.byref(t)) == -5
        c = counts()
        assert c.free == c.malloc - 1 and c.free == nth, c  # what this call allocated
        assert ns.navsim_get_tuning(h) == before
        clear()
        assert step(h, 300) == 0 and launches() == ["fused_early_kernel<4>"]
    assert lib.navsim_set_tuning(h, C.byref(t)) == 0
    clear()
    assert step(h, 300) == 0 and launches() == ["fused_step_kernel<4, 256, false, false>"]
    """)


def test_every_product_kernel_is_launched(run):
    """Small and large products of both layouts, and the gradients' own: no compiled
    product variant is out of reach."""
    run("""
    seen = set()
    for hidden in (64, 512):
        r = proposer(handle(8, [(64, 64)]), hidden=hidden)
        cnt = C.c_int64()
        assert lib.navsim_rp_layout(r, None, None, None, C.byref(cnt)) == 0
        g = np.zeros(cnt.value, np.float32)
        for n in (40, 9000):
            x, t = np.zeros((n, 1048), np.uint16), np.zeros((n, 5), np.float32)
            clear()
            assert lib.navsim_rp_loss_grad(r, n, x.ctypes.data, t.ctypes.data, None, g.ctypes.data, None) == 0
            seen |= set(launches())
    made = {n for n in kernels() if "gemm" in n or "gradient" in n}
    assert made and made <= seen, (made, seen)
    """)


# 256 CUs: 1,024 threads up to 128 tiles of 32 envs; byte copies up to 24 KiB
@pytest.mark.parametrize("n,sides,beams,sectors,shape,kernel", [
    (1, [(64, 64)], 36, 36, (32, 4, 1024), "fused_early_kernel<4>"),
    (4096, [(128, 128)] * 5, 20, 10, (32, 4, 1024), "fused_step_kernel<32, 1024, false, false>"),
    (4097, [(128, 128)] * 5, 20, 10, (32, 5, 512), "fused_step_kernel<32, 512, false, false>"),
    (300, [(136, 128)] * 2, 90, 30, (32, 4, 1024), None),
    (300, [(160, 160)] * 7, 90, 30, (32, 5, 1024), None),
    (5000, [(64, 64)], 360, 360, (32, 5, 1024), "fused_step_kernel<32, 1024, false, false>"),
    (64, [(512, 512)], 360, 360, (32, 3, 1024), None),
    (40, [(96, 96)] * 2, 1080, 1080, (16, 4, 1024), None),
    (24, [(600, 600)], 720, 720, (16, 3, 1024), None),
])
def test_automatic_launch_shape(run, n, sides, beams, sectors, shape, kernel):
    """The shape picked at load on both sides of its rules, the kernel it leads to,
    and no message of a shape that did not fit."""
    run(f"""
    h = handle({n}, {sides}, {beams}, {sectors})
    t = ns.navsim_get_tuning(h)
    assert (t["tile_envs"], t["walk"], t["threads"]) == {shape}, t
    assert lib.navsim_last_error() == b""
    clear()
    assert step(h, {n}, {sectors}) == 0
    assert {kernel!r} in (None, *launches()), launches()
    """)


def test_bench_names_the_step_kernel_that_runs(run):
    run("""
    import bench
    for tile, walk, persist, threads in ((16, 4, 0, 1024), (8, 5, 0, 1024), (16, 3, 2, 1024),
                                         (16, 2, 0, 1024), (32, 5, 0, 512), (8, 3, 0, 256)):
        h = handle(64, [(64, 64)] * 2)
        ns.navsim_set_tuning(h, tile, 32, 16, 0, walk, persist, threads, 1)
        clear()
        assert step(h, 64) == 0
        assert launches()[0].split("<")[0] == bench.step_kernel(ns.navsim_get_tuning(h))
    """)
