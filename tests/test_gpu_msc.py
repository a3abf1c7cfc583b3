"""GPU parity of the multispin-coded Ising chain (32 replicas per uint32,
shared random words) against the oracle: initial words, whole runs and the
per-replica statistics bit-exact, resumed counters, observables."""
import numpy as np
import pytest

from oracle import chain as orc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _grp(Ly, Lx, Jx, Jy, h, beta, rid):
    return dict(model=5, Lx=Lx, Ly=Ly, Jx=Jx, Jy=Jy, h=h, beta=beta, rid=rid)


@pytest.mark.parametrize("shapes", [
    [(2, 8), (6, 16), (8, 8)],
    [(64, 40), (130, 128)],  # several workgroups per group, ragged tails
])
def test_msc_runs_match_oracle(shapes):
    from paper_2304_01772_amd.sampler import Sampler
    params = [(1.0, 1.0, 0.0, 0.4407), (0.7, -0.3, 0.05, 0.9), (1.2, 0.4, -0.1, 0.3)]
    groups = [_grp(Ly, Lx, *params[i % 3], 40 + i) for i, (Ly, Lx) in enumerate(shapes)]
    seed = 0xBEEF_0042
    smp = Sampler(groups, seed, init=True)
    assert smp.R == 32 * len(groups)
    init = [smp.get_state(g) for g in range(len(groups))]
    for g, (Ly, Lx) in enumerate(shapes):
        assert np.array_equal(init[g], orc.msc_init(Lx, Ly, seed, 40 + g)), g
    n = 5
    st = smp.sweep(n, 1).cpu().numpy()
    st2 = smp.sweep(4, 4).cpu().numpy()
    stats, obs = smp.measure()
    stats, obs = stats.cpu().numpy(), obs.cpu().numpy()
    for g, (Ly, Lx) in enumerate(shapes):
        Jx, Jy, h, beta = params[g % 3]
        w1, ost = orc.msc_run(init[g], Jx, Jy, h, beta, seed, 40 + g, 0, n, 1)
        assert np.array_equal(st[:, 32 * g:32 * g + 32], ost), g
        w2, ost2 = orc.msc_run(w1, Jx, Jy, h, beta, seed, 40 + g, n, 4, 4)
        assert np.array_equal(smp.get_state(g), w2), g
        assert np.array_equal(st2[:, 32 * g:32 * g + 32], ost2), g
        want = orc.msc_stats(w2)
        assert np.array_equal(stats[32 * g:32 * g + 32], want)
        N = Ly * Lx
        for b in (0, 17, 31):
            M, Bx, By = want[b, :3]
            e = -(float(np.float32(Jx)) * Bx + float(np.float32(Jy)) * By
                  + float(np.float32(h)) * M) / N
            assert abs(obs[32 * g + b, 0] - e) < 1e-12
    smp.close()


def test_msc_set_state_and_thresholds():
    from paper_2304_01772_amd.sampler import Sampler
    smp = Sampler([_grp(4, 16, 0.9, 0.6, 0.0, 0.5, 3)], 7, init=False)
    assert np.all(smp.get_state(0) == 0)
    T, _ = smp.thresholds(0)
    assert np.array_equal(T, orc.ising_table(np.float32(0.9), np.float32(0.6), 0.0, 0.5))
    rng = np.random.default_rng(0)
    w = rng.integers(0, 2 ** 32, size=(4, 16), dtype=np.uint64).astype(np.uint32)
    smp.set_state(0, w)
    smp.sweep(3)
    want, _ = orc.msc_run(w, 0.9, 0.6, 0.0, 0.5, 7, 3, 0, 3)
    assert np.array_equal(smp.get_state(0), want)
    smp.close()
    with pytest.raises(Exception):
        Sampler([_grp(4, 12, 1.0, 1.0, 0.0, 0.5, 0)], 1)  # Lx not a multiple of 8


# (Jx, Jy, h, beta): the rules of two, nine and eighteen compares, each with
# classes that always flip on either side, and thresholds of 0 and 2^32
_RULES = [(1.0, 1.0, 0.0, 0.44), (-0.8, -0.8, 0.0, 0.6), (0.9, -0.4, 0.0, 0.7),
          (0.8, 0.8, 0.1, 0.5), (1.0, 1.0, 0.0, 40.0), (1.0, 1.0, 0.0, 0.0)]


@pytest.mark.parametrize("schedule", ["auto", "stream"])
@pytest.mark.parametrize("rules", [[0, 1, 4], [2, 1, 0], [3, 0, 5], [5, 0, 0]])
def test_msc_rules_match_oracle(rules, schedule):
    from paper_2304_01772_amd.sampler import Sampler
    shapes = [(10, 16), (4, 8), (34, 72)]
    groups = [_grp(Ly, Lx, *_RULES[k], 70 + k) for k, (Ly, Lx) in zip(rules, shapes)]
    smp = Sampler(groups, 99, init=True)
    smp.set_schedule(mode=schedule)
    init = [smp.get_state(g) for g in range(3)]
    st = smp.sweep(7, 2).cpu().numpy()
    for g, k in enumerate(rules):
        w, want = orc.msc_run(init[g], *_RULES[k], 99, 70 + k, 0, 7, 2)
        assert np.array_equal(smp.get_state(g), w), g
        assert np.array_equal(st[:, 32 * g:32 * g + 32], want), g
    smp.close()


# rows a lane 2, 4 and 8 with whole and ragged last chunks, the most lanes of a
# workgroup, one lane, and one quad a row next to a larger lattice
@pytest.mark.parametrize("shapes", [
    [(2, 8)], [(128, 128)], [(6, 8), (126, 256)], [(128, 256)], [(250, 256), (250, 256)],
    [(256, 256)], [(8, 8192)],
])
def test_msc_resident_at_its_limits(shapes):
    from paper_2304_01772_amd.sampler import Sampler
    par = (1.0, 1.0, 0.0, 0.44)
    # (enough groups that large lattices are resident; the later ones repeat the last)
    shapes = shapes + shapes[-1:] * (64 if np.prod(shapes[0]) > 32768 else 0)
    smp = Sampler([_grp(Ly, Lx, *par, 9 + g) for g, (Ly, Lx) in enumerate(shapes)], 5, init=True)
    init = [smp.get_state(g) for g in range(len(shapes))]
    smp.sweep(1)
    st = smp.sweep(2, 1).cpu().numpy()
    obs = smp.measure()[0].cpu().numpy()
    for g in [*range(min(2, len(shapes))), len(shapes) - 1]:
        w, _ = orc.msc_run(init[g], *par, 5, 9 + g, 0, 1)
        w, want = orc.msc_run(w, *par, 5, 9 + g, 1, 2, 1)
        assert np.array_equal(smp.get_state(g), w), g
        assert np.array_equal(st[:, 32 * g:32 * g + 32], want), g
        assert np.array_equal(obs[32 * g:32 * g + 32], want[-1]), g
    smp.close()
