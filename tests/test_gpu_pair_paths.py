"""The paths of two-step launches that small mixes do not reach, against single
steps (the same bits) and the oracle: marching under graph replay from both
buffer phases, forms that march and forms in tiles in one batch, single steps in
every launch configuration, a work list with no room for pairs, the largest grid."""
import numpy as np
import pytest

from paper_1810_09299_amd import inputs

pytestmark = pytest.mark.gpu


def _spec(nr, nz, collision="mrt", zper=True, seed=None):
    if seed is None:
        s = inputs.static_droplet(nr=nr, nz=nz, R=max(2.0, 0.3 * min(nr, nz)), W=4.0, ratio=10.0, sigma=1e-3,
                                  z_periodic=zper)
    else:
        s = inputs.oscillating_droplet(nr=nr, nz=nz, R0=0.25 * min(nr, nz), seed=seed, W=4.0, ratio=10.0, sigma=1e-3,
                                       z_periodic=zper)
    s.collision = "mrt" if collision == "general" else collision
    if collision in ("general", "nmrt"):
        s.s_g = (1.0, 1.1, 1.2, 1.1, 1.1, 0.9, 0.9, 1.0, 1.0)
        s.free_s1 = True
    return s


def _batch(specs, precision, steps):
    from paper_1810_09299_amd.batch import Batch
    b = Batch(pool_bytes=Batch.pool_for(specs, precision), max_cases=len(specs), precision=precision)
    return b, [b.admit(s, steps) for s in specs]


def _single_steps(spec, precision, n):
    from paper_1810_09299_amd.case import AxiCase
    c = AxiCase(spec, precision=precision)
    for _ in range(n):
        c.step(1)
    st = c.get_state()
    c.close()
    return st


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a[:3], b[:3])) and a[3] == b[3]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_marching_and_tiled_forms_replayed_in_odd_and_even_chunks(precision):
    """Ten cases of 256 x 512 (unit-rate MRT) and three of 512 x 900 (non-orthogonal)
    march, SRT and general MRT go in tiles; no gravity ramp, so that full chunks
    replay graphs, from either phase after an odd one."""
    specs = [_spec(256, 512, seed=q + 1) for q in range(10)]
    specs += [_spec(512, 900, "nmrt", zper=q == 0) for q in range(3)]
    specs += [_spec(60, 286, "srt"), _spec(33, 130, "srt", zper=False), _spec(70, 201, "general")]
    b, slots = _batch(specs, precision, 10 ** 6)
    done = 0
    for chunk in (7, 7, 10, 10, 6, 6, 5, 5, 4):
        b.run(chunk)
        done += chunk
    checked = (0, 9, 10, 12, 13, 14, 15)
    got = [b.get_state(slots[q]) for q in checked]
    b.close()
    for q, st in zip(checked, got):
        assert np.isfinite(st[0]).all() and np.isfinite(st[1]).all()
        assert _same(st, _single_steps(specs[q], precision, done)), (q, specs[q].nr, specs[q].nz, specs[q].collision)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("tile,persistent,schedule,bands", [(2, 0, 0, 8), (4, 1, 1, 32), (16, 1, 0, 16), (16, 0, 2, 32),
                                                            (8, 1, 3, 8), (4, 0, 3, 32), (8, 0, 2, 16)])
def test_single_steps_in_every_launch_configuration(precision, tile, persistent, schedule, bands):
    """Runs of one step, which the configuration governs, against pairs."""
    specs = [_spec(40, 96, zper=False), _spec(33, 200), _spec(36, 80, "srt"), _spec(40, 90, "general"),
             _spec(20, 130, "nmrt")]
    states = []
    for chunk, n in ((8, 2), (1, 16)):
        b, slots = _batch(specs, precision, 16)
        b.set_config(tile, persistent, schedule, bands)
        for _ in range(n):
            b.run(chunk)
        states.append([b.get_state(s) for s in slots])
        b.close()
    for x, y in zip(*states):
        assert x[3] == 16 and _same(x, y)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("tile", [2, 4, 16])
def test_case_tile_is_bitwise_invariant_in_single_steps(precision, tile):
    from paper_1810_09299_amd.case import AxiCase
    spec = _spec(37, 150)
    c = AxiCase(spec, precision=precision)
    c.set_tile(tile)
    for _ in range(6):
        c.step(1)
    got = c.get_state()
    c.close()
    ref = AxiCase(spec, precision=precision)
    ref.step(6)
    assert _same(got, ref.get_state())
    ref.close()


def test_full_work_list_leaves_no_room_for_pairs():
    """Four tall narrow cases whose 64 x 2 tiles fill the work list to its 2^20
    items: steps go singly, with the results of pairs."""
    spec = _spec(524280, 4)
    b, slots = _batch([spec] * 4, "fp32", 100)
    b.set_config(2, 0, 1, 8)
    b.run(3)
    b.run(4)
    got = b.get_state(slots[3])
    assert b.info()["launches"] == 7
    b.set_config(8, 0, 1, 16)                        # room for both lists again
    b.run(5)
    more = b.get_state(slots[0])
    b.close()
    assert _same(got, _single_steps(spec, "fp32", 7))
    assert _same(more, _single_steps(spec, "fp32", 12))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_largest_grid_marches_as_it_steps(precision):
    """nr * nz = 2^25 (the nine FP64 planes of a buffer span 2.25 GiB): one
    marching launch against two single steps, at every node."""
    from paper_1810_09299_amd.case import AxiCase
    spec = _spec(4096, 8192, zper=False)
    states = []
    for runs in ((2,), (1, 1)):
        c = AxiCase(spec, precision=precision)
        for n in runs:
            c.step(n)
        states.append(c.get_state())
        c.close()
    assert np.isfinite(states[0][0]).all() and np.isfinite(states[0][1]).all()
    assert _same(*states)


# two steps from the exported state: each within the one-step bound of
# test_gpu_batch, the second also carrying the first's rounding, hence twice
@pytest.mark.parametrize("precision,rel", [("fp64", 2e-12), ("fp32", 2e-5)])
@pytest.mark.parametrize("cases", [1, 10])
def test_two_steps_of_the_benchmark_match_the_oracle(precision, rel, cases):
    """256 x 512 oscillating droplets in one batch, in tiles (one case) and
    marching (ten): a launch of two steps against two oracle steps."""
    import bench
    import oracle
    specs = bench.batch_specs(cases)
    b, slots = _batch(specs, precision, 10 ** 6)
    b.run(100)
    f, g, aux, t = b.get_state(slots[-1])
    assert t == 100
    b.run(2)
    got = b.get_state(slots[-1])
    b.close()
    ora = oracle.OracleCase(specs[-1])
    ora.set_state(f, g, aux, t)
    ora.step(2)
    assert got[3] == 102
    for x, y, name in zip(got, ora.get_state(), "fga"):
        err = np.abs(x - y).max()
        assert err <= rel * np.abs(y).max(), (name, err)
