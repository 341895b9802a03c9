"""GPU parity where a call's route changes with its size, alignment or data:
the one-launch discretisation (up to 32,768 voxels) and the three kernels
beyond, whole and partial groups of four voxels, pointers off the vector
alignment; maps written directly (up to 4,096 voxels) and through staging
rows; the allocation-free entry point with and without room for the MCC
stash; and the order statistics over every size of the sorted subset.
"""
import numpy as np
import pytest

from helpers import format_report, parity_report, to_dev
from oracle import oracle as O
from paper_2609_19190_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_19190_amd import binding
    binding.lib()
    return binding


def shifted(x, by):
    """x on the device, `by` elements past an aligned address."""
    import torch
    buf = torch.empty(x.size + by, dtype=torch.from_numpy(x).dtype, device="cuda:0")
    buf[by:] = torch.from_numpy(x.reshape(-1)).to("cuda:0")
    return buf[by:].reshape(x.shape)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 3), (3, 5, 7), (16, 64, 64), (16, 64, 65), (17, 61, 63),
                                   (33, 45, 47), (64, 64, 16)])
@pytest.mark.parametrize("dt,mode,value,lower", [(np.float32, O.FBN, 32, float("nan")),
                                                 (np.int16, O.FBW, 25.0, -200.0)])
@pytest.mark.parametrize("off", [0, 1])
def test_discretise_sizes_and_alignment(B, shape, dt, mode, value, lower, off):
    import torch
    rng = np.random.default_rng(shape[2] + off)
    vol = synth.ct_mixture(rng, shape) if dt == np.int16 else rng.gamma(2.0, 1.5, size=shape).astype(np.float32)
    mask = (rng.random(shape) < 0.6).astype(np.uint8) * 3
    mask.reshape(-1)[-1] = 1  # at least one, the last
    levels = shifted(np.full(shape, 77, np.uint8), off)
    lev, ng, xmin, xmax, n = B.fr_discretise(shifted(vol, off), shifted(mask, off), mode, value, lower,
                                             levels=levels)
    olev, ong, oxmin, oxmax = O.discretise(vol, mask, mode, value, lower)
    torch.cuda.synchronize()
    assert (ng, xmin, xmax, n) == (ong, oxmin, oxmax, int(np.count_nonzero(mask)))
    assert np.array_equal(lev.cpu().numpy(), olev)


@pytest.mark.parametrize("n_mask", [1, 4095, 4096, 4097, 20000])
def test_direct_and_staged_output(B, n_mask):
    import torch
    rng = np.random.default_rng(n_mask)
    shape = (26, 30, 34)
    vol = rng.gamma(2.0, 1.5, size=shape).astype(np.float32)
    mask = np.zeros(shape, np.uint8)
    mask.reshape(-1)[rng.choice(mask.size, n_mask, replace=False)] = 1
    case = synth.Case("route", vol, mask, (1.0, 1.0, 1.0), O.FBN, 12.0, float("nan"), 1, 63)
    v, m = to_dev(case)
    args = (v, m, case.spacing, case.mode, case.value, case.lower, 1, 63, n_mask)
    out = B.fr_map(*args)
    B.fr_map_check()
    gpu = out.cpu().numpy()
    ok, rows = parity_report(gpu, O.spatial_map(case), O.map_names(63))
    assert ok, format_report(rows, only_bad=True)
    na = torch.empty_like(out)
    B.fr_map_noalloc(*args, na)
    B.fr_map_check()
    assert np.array_equal(na.cpu().numpy().view(np.uint32), gpu.view(np.uint32))


def test_noalloc_with_and_without_room_for_the_stash(B):
    import torch
    # about 1,500 bytes a voxel with the stash: the second does not fit 64 MiB with it
    for n in (40000, 60000):
        shape = (40, 45, 50)
        rng = np.random.default_rng(n)
        vol = rng.gamma(2.0, 1.5, size=shape).astype(np.float32)
        mask = np.zeros(shape, np.uint8)
        mask.reshape(-1)[:n] = 1
        v, m = to_dev(synth.Case("stash", vol, mask, (1.0, 1.0, 1.0), O.FBN, 24.0, float("nan"), 1, 2))
        args = (v, m, (1.0, 1.0, 1.0), O.FBN, 24.0, float("nan"), 1, 2, n)
        ref = B.fr_map(*args)
        out = torch.empty_like(ref)
        B.fr_map_noalloc(*args, out)
        B.fr_map_check()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.cpu().numpy().view(np.uint32))


def test_count_mismatch_is_reported_on_both_discretisations(B):
    import torch
    for shape in ((16, 32, 32), (32, 64, 64)):
        vol = torch.rand(shape, device="cuda:0")
        mask = torch.ones(shape, dtype=torch.uint8, device="cuda:0")
        out = torch.full((18, 10), 5.0, device="cuda:0")
        for f in (B.fr_map, B.fr_map_noalloc):
            f(vol, mask, (1, 1, 1), O.FBN, 8, float("nan"), 1, 1, 10, out)
            rc, _ = B.fr_map_status()
            assert rc == B.FR_E_ARG
            assert bool((out == 5.0).all())


@pytest.mark.parametrize("radius", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("bins", [1, 2, 4, 9, 40])
def test_order_statistics_by_level_subset(B, radius, bins):
    """Continuous values, so that ranks inside a level matter; a heavy tail
    puts most of V into a few levels."""
    case = synth.random_case(900 + 7 * bins + radius, shape=(11, 12, 13), dtype=np.float32, radius=radius,
                             mode=O.FBN, value=bins, families=1, mask_fill=0.9)
    case.volume = (case.volume ** 2).astype(np.float32)
    v, m = to_dev(case)
    gpu = B.fr_map(v, m, case.spacing, case.mode, case.value, case.lower, radius, 1, case.n_mask)
    B.fr_map_check()
    ok, rows = parity_report(gpu.cpu().numpy(), O.spatial_map(case), O.map_names(1))
    assert ok, format_report(rows, only_bad=True)


@pytest.mark.parametrize("shape", [(2, 512, 1024), (2, 512, 1028), (3, 512, 1024)])  # 256, 257, 384 segments
def test_list_order_over_the_segment_scan(B, shape):
    """One segment a thread of the scan, and a second or half a one: every
    mask voxel at its place of the list, isolated voxels among them."""
    rng = np.random.default_rng(shape[2] + shape[0])
    vol = rng.gamma(2.0, 1.5, size=shape).astype(np.float32)
    mask = np.zeros(shape, np.uint8)
    flat = mask.reshape(-1)
    flat[rng.choice(flat.size, 300, replace=False)] = 1
    flat[[0, -1]] = 1
    mask[1, 100:104, 200:206] = 1
    case = synth.Case("segments", vol, mask, (1.0, 1.0, 1.0), O.FBN, 20.0, float("nan"), 1, 63)
    v, m = to_dev(case)
    out = B.fr_map(v, m, case.spacing, case.mode, case.value, case.lower, 1, 63, case.n_mask)
    B.fr_map_check()
    ok, rows = parity_report(out.cpu().numpy(), O.spatial_map(case), O.map_names(63))
    assert ok, format_report(rows, only_bad=True)


@pytest.mark.parametrize("shape", [(16, 32, 32), (24, 48, 64)])  # one launch, three kernels
def test_range_error_with_a_small_n_mask_leaves_other_jobs_alone(B, shape):
    """More than 255 levels and an n_mask below the mask's count: only the
    first error is reported, and nothing past the n_mask entries of the job's
    own list is written (a neighbour's list in a batch, a block in a server,
    the buffers after it in the allocation-free entry point)."""
    import torch
    rng = np.random.default_rng(shape[1])
    vol = rng.integers(0, 3000, size=shape).astype(np.int16)
    bad = (torch.from_numpy(vol).to("cuda:0"), torch.ones(shape, dtype=torch.uint8, device="cuda:0"), (1.0, 1.0, 1.0),
           O.FBW, 5.0, float("nan"), 1, 1, 10)
    case = synth.random_case(41, shape=(12, 13, 14), dtype=np.int16, radius=1, mode=O.FBN, value=12, families=63)
    v, m = to_dev(case)
    good = (v, m, case.spacing, case.mode, case.value, case.lower, 1, 63, case.n_mask)
    ref = B.fr_map(*good)
    B.fr_map_check()
    ref = ref.cpu().numpy().view(np.uint32)
    for f in (B.fr_map, B.fr_map_noalloc):
        out = torch.full((18, 10), 5.0, device="cuda:0")
        f(*bad, out)
        rc, _ = B.fr_map_status()
        assert rc == B.FR_E_RANGE
        assert bool((out == 5.0).all())
        nxt = torch.empty(ref.shape, device="cuda:0")
        f(*good, nxt)
        B.fr_map_check()
        assert np.array_equal(nxt.cpu().numpy().view(np.uint32), ref)
    keys = ("volume", "mask", "spacing", "mode", "value", "lower", "radius", "families", "n_mask")
    bt = B.Batch([dict(zip(keys, a)) for a in (good, bad, good, bad, good)])
    try:
        bt.launch()
        rc, st, _ = bt.status()
        assert rc != B.FR_OK and st == [0, B.FR_E_RANGE, 0, B.FR_E_RANGE, 0]
        for k in (0, 2, 4):
            assert np.array_equal(bt.outs[k].cpu().numpy().view(np.uint32), ref)
    finally:
        bt.close()
    srv = B.Server(1 << 28, slots=2)
    try:
        tickets = [srv.submit(*a) for a in (good, bad, good, bad, good)]
        for k, t in enumerate(tickets):
            if k % 2:
                srv.wait(t)
                assert srv.result(t).status == B.FR_E_RANGE
            else:
                srv.wait(t)
                got = srv.maps(t)
                torch.cuda.synchronize()
                assert np.array_equal(got.cpu().numpy().view(np.uint32), ref)
            srv.release(t)
    finally:
        srv.close()


@pytest.mark.parametrize("shape", [(16, 32, 32), (31, 33, 32), (32, 32, 32), (32, 32, 33), (29, 31, 37)])  # 16,384 .. 33,792
@pytest.mark.parametrize("dt", [np.float32, np.int16])
def test_edge_of_the_one_launch_discretisation(B, shape, dt):
    import torch
    rng = np.random.default_rng(shape[2])
    vol = synth.ct_mixture(rng, shape) if dt == np.int16 else rng.gamma(2.0, 1.5, size=shape).astype(np.float32)
    mask = (rng.random(shape) < 0.4).astype(np.uint8)
    mask.reshape(-1)[[0, -1]] = 1
    case = synth.Case("edge", vol, mask, (1.0, 1.0, 1.0), O.FBN, 14.0, float("nan"), 1, 1)
    v, m = to_dev(case)
    lev, ng, xmin, xmax, n = B.fr_discretise(v, m, case.mode, case.value, case.lower)
    olev, ong, oxmin, oxmax = O.discretise(vol, mask, case.mode, case.value, case.lower)
    torch.cuda.synchronize()
    assert (ng, xmin, xmax, n) == (ong, oxmin, oxmax, case.n_mask)
    assert np.array_equal(lev.cpu().numpy(), olev)
    out = B.fr_map(v, m, case.spacing, case.mode, case.value, case.lower, 1, 1, case.n_mask)
    B.fr_map_check()
    ok, rows = parity_report(out.cpu().numpy(), O.spatial_map(case), O.map_names(1))
    assert ok, format_report(rows, only_bad=True)


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("dt", [np.float32, np.int16])
def test_segments_without_a_mask_voxel(B, dt, off):
    """Empty segments before, between and after those with one mask voxel or
    more, a partial last one among them: their levels are 0, whatever was in
    the buffer; the same maps from a batch of such volumes."""
    import torch
    shape = (11, 64, 65)  # 12 segments of 4,096, the last of 704
    rng = np.random.default_rng(off)
    vol = synth.ct_mixture(rng, shape) if dt == np.int16 else rng.gamma(2.0, 1.5, size=shape).astype(np.float32)
    for at in ([4096 * 3, 4096 * 3 + 70, 4096 * 7 - 1], [0, 1, 45759], list(range(20000, 20600))):
        mask = np.zeros(shape, np.uint8)
        mask.reshape(-1)[at] = 1
        v, m = shifted(vol, off), shifted(mask, off)
        levels = shifted(np.full(shape, 77, np.uint8), off)
        B.fr_discretise(v, m, O.FBN, 9, float("nan"), levels=levels)
        olev, _, _, _ = O.discretise(vol, mask, O.FBN, 9, float("nan"))
        torch.cuda.synchronize()
        assert np.array_equal(levels.cpu().numpy(), olev)
        case = synth.Case("sparse", vol, mask, (1.0, 1.0, 1.0), O.FBN, 9.0, float("nan"), 1, 63)
        job = dict(volume=v, mask=m, spacing=case.spacing, mode=case.mode, value=case.value, lower=case.lower, radius=1,
                   families=63, n_mask=case.n_mask)
        out = B.fr_map(*job.values())
        B.fr_map_check()
        ok, rows = parity_report(out.cpu().numpy(), O.spatial_map(case), O.map_names(63))
        assert ok, format_report(rows, only_bad=True)
        bt = B.Batch([job, job])
        try:
            bt.launch()
            assert bt.status()[0] == B.FR_OK
            for o in bt.outs:
                assert np.array_equal(o.cpu().numpy().view(np.uint32), out.cpu().numpy().view(np.uint32))
        finally:
            bt.close()


@pytest.mark.parametrize("radius", [1, 2, 3])
def test_neighbourhoods_without_a_value(B, radius):
    """Fixed bin width gives a NaN no level: where a whole neighbourhood is
    NaN, the sums are empty and the means undefined."""
    rng = np.random.default_rng(radius)
    vol = rng.gamma(2.0, 1.5, size=(16, 17, 18)).astype(np.float32)
    vol[4:13, 4:13, 4:13] = np.nan
    mask = np.ones(vol.shape, np.uint8)
    v, m = to_dev(synth.Case("nan", vol, mask, (1.0, 1.0, 1.0), O.FBW, 1.0, 0.0, radius, 1))
    out = B.fr_map(v, m, (1.0, 1.0, 1.0), O.FBW, 1.0, 0.0, radius, 1, mask.size)
    B.fr_map_check()
    names = O.map_names(1)
    f = dict(zip(names, out.cpu().numpy().reshape(len(names), *vol.shape)[:, 8, 8, 8]))
    for k in ("Energy", "TotalEnergy", "Entropy", "Uniformity"):
        assert f["firstorder_" + k] == 0.0, k
    for k in ("Mean", "Variance", "MeanAbsoluteDeviation", "RobustMeanAbsoluteDeviation", "RootMeanSquared"):
        assert np.isnan(f["firstorder_" + k]), k
    assert f["firstorder_Minimum"] == np.inf
