"""The library's dispatch on the host: which kernels a call launches, and how
many workgroups (no GPU; see launches.py)."""
import re

import pytest

from launches import build_recorder, launches, spilled_vgprs
from test_gpu_parity import LAG_HAND_OVER

CUS = 256


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return build_recorder(tmp_path_factory.mktemp("recorder"))


def template_args(name):
    return [a.strip() for a in re.search(r"<(.*)>", name).group(1).split(",")]


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    return spilled_vgprs(tmp_path_factory.mktemp("objects"))


def kernels(recorder, call, R, S, T, window=1):
    return [ls.name for ls in launches(recorder, [(call, R, S, T, window)])[0]]


def is_narrow(name):
    return name.startswith("k_median_spread") and template_args(name)[7] == "true"


def test_lag_hand_over_shapes_take_the_narrow_pass(recorder):
    """The shapes of the GPU test of the lag's hand-over are handed over: the
    32-bit pass first, then the 64-bit kernel."""
    cases = [("sf_frontier_lag", R, S, T, 1) for R, S, T in LAG_HAND_OVER]
    for c, ls in zip(cases, launches(recorder, cases)):
        assert len(ls) == 2 and is_narrow(ls[0].name), (c, ls)


@pytest.mark.parametrize("call", ["sf_frontier_lag", "sf_rank_spread"])
def test_hand_over_is_as_wide_as_the_chip(recorder, call):
    """With every step handed over, its workgroups are through in little more
    than the rounds that a workgroup per step would take, and there are few
    enough of them where nothing is handed over."""
    cases = [(call, R, S, T, 100) for R in (513, 1023, 1024, 3000, 4097, 8192, 12289, 16384, 24576, 32767)
             for S in (1, 6, 8, 12) for T in (1, 64, 256, 300, 500, 512, 1000, 2000, 4000, 10000, 50000)]
    seen = 0
    for c, ls in zip(cases, launches(recorder, cases)):
        if not is_narrow(ls[0].name):
            continue
        seen += 1
        steps, redo = ls[0].grid, ls[1]
        waves = 32 if redo.name.startswith("k_median_stream") else 16  # resident per CU
        at_once = CUS * waves * 64 // redo.block
        rows = -(-steps // redo.grid)
        assert rows <= 8
        depth = rows if redo.grid <= at_once else steps / at_once + rows - 1
        assert depth <= 1.25 * -(-steps // at_once) + 2, (c, ls)
        assert redo.grid <= max(4096, steps // 4), (c, ls)
    assert seen > 50


def test_hand_over_kernels_spill_nothing(spills):
    redo = {k: n for k, n in spills.items() if k.startswith("k_median_spread") and template_args(k)[8] == "true"}
    assert len(redo) >= 14 and not any(redo.values()), redo

def test_twelve_wave_lag_keeps_its_registers(spills):
    """More than 16384 ranks, 80 VGPRs: two loads of a stage at once (four
    spilled 20 to 24)."""
    twelve = {k: n for k, n in spills.items() if k.startswith("k_median_spread") and template_args(k)[3] == "768"}
    assert len(twelve) == 4 and max(twelve.values()) <= 10, twelve

def test_checked_frontier_spills_nothing(spills):
    checked = {k: n for k, n in spills.items() if k.startswith("k_frontier<") and template_args(k)[4] == "true"}
    assert len(checked) >= 20 and not any(checked.values()), checked

@pytest.mark.parametrize("R,S,T,rows", [
    (2, 9, 100000, 1), (2, 48, 100000, 8), (8, 16, 8192, 1), (8, 25, 8192, 8), (16, 12, 2048, 1), (16, 17, 2048, 8),
    (32, 9, 2048, 8), (33, 9, 8192, 1), (64, 13, 2048, 8), (100, 9, 2048, 1), (128, 12, 2048, 8), (200, 9, 2000, 8),
    (512, 12, 64, 1), (512, 13, 64, 8), (1500, 4, 3000, 1), (1500, 8, 3000, 4), (5120, 2, 3000, 1), (5120, 4, 3000, 2)])
def test_frontier_rows_in_flight(recorder, R, S, T, rows):
    """Rows kept in flight take as many stages as pay for them."""
    (name,) = kernels(recorder, "sf_frontier", R, S, T)
    assert template_args(name)[6] == str(rows), name

@pytest.mark.parametrize("R,S,T,shape", [
    (4, 5, 100000, "2, 4, 64, false, 1"), (4, 8, 100000, "2, 4, 64, false, 4"), (16, 7, 100000, "2, 8, 64, false, 1"),
    (100, 12, 1024, "2, 64, 64, false, 4"), (100, 12, 1200, "8, 16, 256, false, 1"), (200, 6, 1536, "2, 128, 128, false, 4"),
    (129, 6, 2000, "8, 32, 64, false, 1"), (240, 12, 16000, "8, 16, 256, false, 1"), (16384, 8, 256, "16, 1024, 1024, false, 1"),
    (16384, 8, 300, "32, 256, 256, false, 1"), (24576, 8, 50, "32, 256, 256, false, 1"), (32768, 8, 50, "16, 1024, 1024, false, 1"),
    (8192, 204, 1, "16, 512, 512, false, 1"), (8192, 205, 1, "32, 256, 256, false, 1"), (5001, 260, 20, "32, 256, 256, false, 1"),
    (12000, 260, 500, "32, 256, 256, false, 1"), (8192, 410, 1, "16, 128, 128, false, 1")])
def test_evidence_shapes(recorder, R, S, T, shape):
    """The shapes for few steps and few ranks end where they were measured to
    be the faster ones."""
    (name,) = kernels(recorder, "sf_frontier_evidence", R, S, T)
    assert ", ".join(template_args(name)[1:]) == shape, name

def test_window_sum_of_short_windows_is_not_unrolled(recorder):
    assert kernels(recorder, "sf_rank_spread", 16, 6, 100000, 1)[-1] == "k_window_sum<1>"
    assert kernels(recorder, "sf_rank_spread", 16, 2, 200000, 20000)[-1] == "k_window_sum<4>"

@pytest.mark.parametrize("call,R,S,T,window,whole", [
    ("sf_window_summary", 4096, 1, 100, 50, True), ("sf_window_summary", 8192, 1, 100, 50, False),
    ("sf_window_summary", 16384, 1, 55, 55, False), ("sf_window_summary", 6000, 6, 50, 50, False),
    ("sf_window_summary", 6144, 2, 500, 250, True), ("sf_window_summary", 15, 260, 1000, 250, False),
    ("sf_window_summary", 15, 260, 4000, 250, True), ("sf_window_summary", 361, 68, 250, 250, False),
    ("sf_window_summary", 60, 68, 1000, 250, True), ("sf_window_summary", 128, 6, 100000, 1000, True),
    ("sf_window_lead_exposed", 16384, 1, 100, 50, False), ("sf_window_lead_exposed", 15, 260, 1000, 250, True)])
def test_whole_windows(recorder, call, R, S, T, window, whole):
    """One workgroup per window where that is the faster way."""
    assert kernels(recorder, call, R, S, T, window)[0].startswith("k_window_whole") == whole

@pytest.mark.parametrize("R,S,window,fused", [
    (8, 6, 100, True), (8, 12, 100, True), (8, 12, 200, False), (16, 6, 100, True), (16, 6, 200, False), (32, 6, 50, True),
    (8, 6, 256, True), (8, 1, 1024, True), (8, 1, 1025, False), (4, 2, 640, True), (2, 3, 427, False), (16, 1, 400, True),
    (16, 1, 401, False), (16, 2, 321, False), (17, 1, 257, False),
    (32, 6, 100, False), (64, 4, 20, True), (64, 8, 1, True), (64, 6, 50, False), (256, 4, 20, True), (256, 6, 50, False),
    (200, 8, 1, True), (257, 1, 1, False), (8, 13, 10, False)])
def test_fused_summary(recorder, R, S, window, fused):
    """The one-launch summary takes windows of about one round of steps, at up
    to 256 ranks."""
    assert kernels(recorder, "sf_frontier_summary", R, S, 10 * window, window)[0].startswith("k_frontier_summary") == fused


@pytest.mark.parametrize("R,S,kernel", [
    (32769, 25, "k_exposure_gain<2, 256, 256, 32"), (65536, 32, "k_exposure_gain<2, 256, 256, 32"),
    (45000, 33, "k_exposure_gain<1, 256, 256, 64"), (32769, 64, "k_exposure_gain<1, 256, 256, 64"),
    (32769, 65, "k_exposure_gain_wide"), (32768, 25, "k_exposure_gain_near"), (20, 25, "k_exposure_gain_wide")])
def test_gain_of_many_stages(recorder, R, S, kernel):
    """Up to 64 stages in registers past the ranks of the near-frontier pass."""
    assert kernels(recorder, "sf_exposure_gain", R, S, 20, 10)[0].startswith(kernel)


@pytest.mark.parametrize("R,S,T,near", [
    (16384, 5, 1, True), (16384, 5, 256, True), (16384, 5, 257, False), (8192, 4, 8, True), (8192, 4, 9, False),
    (8194, 4, 64, True), (32768, 5, 8, True), (32768, 5, 9, False), (32768, 8, 64, True), (32768, 8, 65, False),
    (24576, 12, 256, True), (24576, 12, 257, False), (24576, 13, 1000, True), (4096, 8, 512, True), (4096, 8, 513, False),
    (2048, 8, 4000, True), (4096, 9, 4000, True)])
def test_gain_of_few_steps(recorder, R, S, T, near):
    """The near-frontier pass, a whole workgroup per step, where few steps leave
    the other kernels' chip idle, and not where it lost to them."""
    assert kernels(recorder, "sf_exposure_gain", R, S, T, 50)[0].startswith("k_exposure_gain_near") == near


@pytest.mark.parametrize("R,T,shape", [(200, 256, "1024, 1, 8"), (200, 257, "256, 1, 2"), (512, 257, "256, 1, 1"),
                                       (1024, 256, "1024, 1, 2"), (1024, 257, "256, 2, 1"), (2048, 512, "1024, 1, 1"),
                                       (2048, 513, "256, 4, 1")])
def test_gain_wide_workgroups_for_few_steps(recorder, R, T, shape):
    assert ", ".join(template_args(kernels(recorder, "sf_exposure_gain", R, 12, T, 50)[0])) == shape


@pytest.mark.parametrize("R,S,T,window,tiled", [
    (65536, 512, 3, 2, True), (65536, 520, 3, 2, True), (65536, 9000, 2, 2, True), (65536, 520, 300, 300, True),
    (4096, 12, 4096, 4096, True), (4096, 12, 4097, 4097, False), (1, 1, 50, 10, False)])
def test_median_tiles(recorder, R, S, T, window, tiled):
    """Windows of up to 4096 steps are held in tiles, at any stage and rank
    count."""
    name = kernels(recorder, "sf_window_median", R, S, T, window)[0]
    assert name.startswith("k_window_median<") == tiled, name


def test_bench_names_the_gain_kernel_that_runs(recorder):
    import bench
    import synth
    for wl in synth.WORKLOADS.values():
        name = kernels(recorder, "sf_exposure_gain", wl.R, wl.S, wl.T, wl.window)[0]
        assert name.startswith(bench.gain_kernel(wl.R, wl.S) + "<"), (wl.name, name)


def test_hand_over_grid_meets_no_short_period(recorder):
    """Every second to tenth step marked is not one workgroup's every time."""
    import math
    cases = [("sf_frontier_lag", R, S, T, 1) for R, S, T in ((16384, 12, 2000), (8192, 3, 5000), (5001, 8, 10000), (20000, 8, 6000))]
    cases.append(("sf_rank_spread", 1024, 9, 20000, 100))
    for c, ls in zip(cases, launches(recorder, cases)):
        steps, redo = ls[0].grid, ls[1]
        assert redo.grid < steps and math.gcd(redo.grid, 210) == 1, (c, ls)


@pytest.mark.parametrize("R,S,T,groups,size", [
    (4098, 1, 500, 1, 512), (4099, 2, 512, 1, 512), (4140, 8, 48, 4, 512), (4140, 8, 160, 3, 512), (4140, 8, 256, 2, 512),
    (4140, 4, 160, 1, 512), (6001, 8, 160, 3, 512), (6001, 8, 200, 1, 512), (8190, 8, 256, 1, 512), (8192, 12, 1, 12, 512),
    (8193, 7, 220, 1, 1024), (10000, 8, 160, 1, 1024), (10000, 12, 48, 4, 1024), (16384, 12, 128, 2, 1024), (16384, 2, 1, 1, 1024),
    (16384, 12, 256, 1, 1024)])
def test_lag_of_few_steps(recorder, R, S, T, groups, size):
    """Past 4096 ranks a few steps are one launch of one round: the stages
    shared where two workgroups or more have a CU, else 64 bits and no
    hand-over."""
    (ls,) = launches(recorder, [("sf_frontier_lag", R, S, T, 1)])[0]
    assert (ls.grid, ls.block) == (T * groups, size) and not is_narrow(ls.name), ls


@pytest.mark.parametrize("R,T", [(8192, 513), (5001, 513), (8193, 257), (16384, 257)])
def test_lag_of_more_steps_than_a_round(recorder, R, T):
    ls = launches(recorder, [("sf_frontier_lag", R, 4, T, 1)])[0]
    assert len(ls) == 2 and is_narrow(ls[0].name), ls


@pytest.mark.parametrize("R,rows", [(513, 4096), (1024, 4096), (1025, 2048), (2048, 2048), (2049, 1024), (4096, 1024), (4097, 512),
                                    (8192, 512), (8193, 256), (16383, 256), (16384, 256)])
def test_spread_of_few_rows(recorder, R, rows):
    """Rows that all run at once take the 64-bit shapes and hand nothing over."""
    cases = [("sf_rank_spread", R, S, T, 100) for S, T in ((1, rows), (4, rows // 4), (1, rows + 1), (4, rows // 4 + 1))]
    names = [[k.name for k in ls] for ls in launches(recorder, cases)]
    assert [is_narrow(n[0]) for n in names] == [False, False, True, True], names
    assert [len(n) for n in names] == [2, 2, 3, 3], names
