"""The LDS-resident triangular and chain / cubic kernel at the edges of its
forms, bit for bit against the oracle: one or two Philox blocks per item
(plane rows of an odd or even number of blocks), one item or several per lane
(up to the 64 KiB limit), a ragged last workgroup wave, absent and two-site
dimensions, thresholds that underflow to 0, and recorded sweeps that do not
start or end with the call."""
import numpy as np
import pytest

from oracle import chain as orc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _check(reps, run, seed=0x77_0000_0031, n=7, every=3):
    from paper_2304_01772_amd.sampler import Sampler
    smp = Sampler(reps, seed, init=True)
    init = [smp.get_state(r) for r in range(len(reps))]
    smp.sweep(2)
    st = smp.sweep(n, every).cpu().numpy()
    for r, d in enumerate(reps):
        s1, _ = run(init[r], d, seed, 0, 2, 0)
        s2, ost = run(s1, d, seed, 2, n, every)
        assert np.array_equal(smp.get_state(r), s2), r
        assert np.array_equal(st[:, r], ost), r
    smp.close()


@pytest.mark.parametrize("Ly,Lx,n_rep,beta", [
    (3, 12, 1, 0.27),      # one block a row
    (9, 36, 3, 0.27),      # three blocks a row (one per item)
    (6, 24, 2, 0.27),      # two blocks a row (two per item)
    (102, 120, 2, 0.27),   # two per item, 510 items: a ragged wave
    (180, 192, 2, 0.27),   # two per item, several items a lane
    (243, 252, 2, 0.27),   # one per item, several items a lane
    (27, 2424, 1, 0.27),   # near the 64 KiB limit, long rows
    (12, 24, 2, 90.0),     # T = 0 for the largest energy changes
])
def test_triangular(Ly, Lx, n_rep, beta):
    reps = [dict(model=3, Lx=Lx, Ly=Ly, Jx=1.0 - 0.5 * r, Jy=1.0 - 0.5 * r, h=0.05, beta=beta,
                 rid=40 + r) for r in range(n_rep)]
    _check(reps, lambda s, d, seed, t, n, e: orc.tri_run(s, d["Jx"], d["h"], beta, seed, d["rid"],
                                                         t, n, e))


@pytest.mark.parametrize("Lz,Ly,Lx,beta", [
    (1, 1, 8, 0.4), (1, 1, 48, 0.4), (1, 1, 4104, 0.4),
    (1, 2, 16, 0.4), (2, 2, 8, 0.3), (1, 66, 72, 0.4), (4, 1, 16, 0.3),
    (34, 30, 32, 0.22),    # two blocks per item, several items a lane
    (34, 38, 40, 0.22),    # one per item, several items a lane
    (2, 4, 16, 130.0),     # T = 0 for the largest energy changes
])
def test_chain_square_cubic(Lz, Ly, Lx, beta):
    reps = [dict(model=4, Lx=Lx, Ly=Ly, Lz=Lz, Jx=1.0 - 0.7 * r, Jy=1.0 - 0.7 * r, h=-0.03,
                 beta=beta, rid=50 + r) for r in range(2)]
    _check(reps, lambda s, d, seed, t, n, e: orc.hc_run(s, d["Jx"], d["h"], beta, seed, d["rid"],
                                                        t, n, e))


def test_two_blocks_an_item_in_a_ragged_wave():
    """612 and 594 items of two blocks, one a lane."""
    reps = [dict(model=3, Lx=144, Ly=102, Jx=1.0, Jy=1.0, h=0.05, beta=0.27, rid=60)]
    _check(reps, lambda s, d, seed, t, n, e: orc.tri_run(s, 1.0, 0.05, 0.27, seed, 60, t, n, e))
    reps = [dict(model=4, Lx=144, Ly=66, Lz=1, Jx=1.0, Jy=1.0, h=0.05, beta=0.4, rid=61)]
    _check(reps, lambda s, d, seed, t, n, e: orc.hc_run(s, 1.0, 0.05, 0.4, seed, 61, t, n, e))


@pytest.mark.parametrize("dims", [
    dict(model=3, Lx=12, Ly=3), dict(model=3, Lx=36, Ly=9), dict(model=3, Lx=120, Ly=102),
    dict(model=4, Lx=8, Ly=1, Lz=1), dict(model=4, Lx=48, Ly=1, Lz=1),
    dict(model=4, Lx=16, Ly=2, Lz=1), dict(model=4, Lx=24, Ly=2, Lz=2),
    dict(model=4, Lx=32, Ly=34, Lz=6), dict(model=4, Lx=4, Ly=6, Lz=4),
])
def test_measured_statistics_equal_recorded_ones(dims):
    """measure() after a recorded sweep: one and two blocks an item, absent
    dimensions, a lattice whose rows are no whole blocks."""
    from paper_2304_01772_amd.sampler import Sampler
    reps = [dict(dims, Jx=1.0, Jy=1.0, h=0.0, beta=0.3, rid=r) for r in range(3)]
    smp = Sampler(reps, 62, init=True)
    st = smp.sweep(2, 1)[-1]
    got, _ = smp.measure()
    assert torch.equal(got, st)
    smp.set_schedule(mode="stream")
    st = smp.sweep(2, 2)[-1]
    smp.set_schedule(mode="auto")
    got, _ = smp.measure()
    assert torch.equal(got, st)
    smp.close()


def _check_both(reps, run):
    """Resident whatever the size, then streamed passes, of one chain."""
    from paper_2304_01772_amd.sampler import Sampler
    smp = Sampler(reps, 64, init=True)
    cur = [smp.get_state(r) for r in range(len(reps))]
    t = 0
    for mode, n, every in (("hybrid", 2, 0), ("hybrid", 7, 3), ("stream", 3, 2)):
        smp.set_schedule(mode=mode)
        st = smp.sweep(n, every)
        for r, d in enumerate(reps):
            cur[r], ost = run(cur[r], d, t, n, every)
            assert np.array_equal(smp.get_state(r), cur[r]), (r, mode)
            if every:
                assert np.array_equal(st[:, r].cpu().numpy(), ost), (r, mode)
        t += n
    smp.set_schedule(mode="hybrid")
    st = smp.sweep(1, 1)[-1]
    assert torch.equal(smp.measure()[0], st)
    smp.close()


@pytest.mark.parametrize("Ly,Lx,n_rep,beta", [
    (3, 15, 1, 0.27), (6, 21, 2, 0.27), (27, 33, 3, 0.27),  # blocks across rows
    (102, 123, 2, 0.27), (243, 267, 1, 0.27), (3, 21843, 1, 0.27),  # rounds of blocks; the limit
    (12, 27, 2, 90.0),  # T = 0 for the largest energy changes
])
def test_triangular_blocks_across_rows(Ly, Lx, n_rep, beta):
    reps = [dict(model=3, Lx=Lx, Ly=Ly, Jx=1.0 - 0.5 * r, Jy=1.0 - 0.5 * r, h=0.05, beta=beta,
                 rid=70 + r) for r in range(n_rep)]
    reps.append(dict(reps[0], Lx=12, Ly=3, rid=79))  # whole blocks beside the others
    _check_both(reps, lambda s, d, t, n, e: orc.tri_run(s, d["Jx"], d["h"], beta, 64, d["rid"], t, n, e))


@pytest.mark.parametrize("Lz,Ly,Lx,beta", [
    (1, 1, 10, 0.4), (1, 1, 4098, 0.4), (1, 1, 65534, 0.4), (1, 2, 14, 0.4), (2, 2, 10, 0.3),
    (1, 66, 70, 0.4), (4, 1, 18, 0.3), (34, 30, 34, 0.22), (40, 38, 42, 0.22),
    (2, 4, 10, 130.0),  # T = 0 for the largest energy changes
])
def test_chain_square_cubic_blocks_across_rows(Lz, Ly, Lx, beta):
    reps = [dict(model=4, Lx=Lx, Ly=Ly, Lz=Lz, Jx=1.0 - 0.7 * r, Jy=1.0 - 0.7 * r, h=-0.03,
                 beta=beta, rid=80 + r) for r in range(2)]
    _check_both(reps, lambda s, d, t, n, e: orc.hc_run(s, d["Jx"], d["h"], beta, 64, d["rid"], t, n, e))


def test_large_lattices_in_numbers_across_rows():
    """Lattices above 64 KiB of which every compute unit has one."""
    from paper_2304_01772_amd.sampler import Sampler
    reps = [dict(model=3, Lx=375, Ly=375, Jx=1.0, Jy=1.0, h=0.02, beta=0.27, rid=r)
            for r in range(128)]
    smp = Sampler(reps, 63, init=True)
    init = smp.get_state(127)
    st = smp.sweep(3, 1).cpu().numpy()
    want, ost = orc.tri_run(init, 1.0, 0.02, 0.27, 63, 127, 0, 3, 1)
    assert np.array_equal(smp.get_state(127), want)
    assert np.array_equal(st[:, 127], ost)
    smp.close()
