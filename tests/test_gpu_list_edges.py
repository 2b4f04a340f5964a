"""The list rebuild where its fixed widths end: cells of more members than a group's 8 or 16 lanes,
rows of more candidates than one (20) or two (32) tests at once take, lists longer than a thread's run
in LDS (32), frames that wrap onto themselves, a tile remainder of one cell.  FP64 steps against the
oracle, and the mixed path's staged build against its build from global memory."""
import time

import numpy as np
import pytest

from oracle import oracle as o
from tests import inputs

pytestmark = pytest.mark.gpu

kg = pytest.importorskip("paper_2109_11001_amd")
torch = pytest.importorskip("torch")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

CASES = [
    dict(M=20, N=50, rho=0.85),   # 5 cells a side, 8 members a cell (groups of 16), rows of 24
    dict(M=20, N=50, rho=1.8),    # 4 cells a side, 16 a cell, rows of 47, lists of 40
    dict(M=40, N=100, rho=1.3),   # rows of 24, lists of 29: some past 32
    dict(M=100, N=100, rho=0.85),  # five a cell (groups of 8, some cells past it)
    dict(M=37, N=61, rho=0.6),
]


@pytest.mark.parametrize("kw", CASES)
def test_lists_at_the_edges(kw):
    kw = dict(kw, kappa=1.0, seed=13)
    om = o.Melt(warmup_steps=300, **kw)
    st = om.get_state()
    st["v"] = np.clip(inputs.random_velocities(kw["M"] * kw["N"], 5), -3.0, 3.0)
    om.set_state(x=st["x"], v=st["v"], fl=st["fl"], chains=st["chains"], counters=st["counters"])
    melts = {}
    for name, more in (("fp64", dict(precision=0)), ("mixed", dict(precision=1)),
                       ("global", dict(precision=1, test_flags=kg.TF_NL_GLOBAL))):
        g = kg.Melt(warmup_steps=0, nl_every=5, **more, **kw)
        g.set_state(0, x=st["x"], v=st["v"], fl=st["fl"], chains=st["chains"], counters=st["counters"])
        g.md_steps(12)
        melts[name] = g
    om.md_steps(12)
    d = melts["fp64"].get_state()["x"] - om.get_state()["x"]
    d -= om.L * np.rint(d / om.L)
    assert np.max(np.abs(d)) < 1e-11  # a short window of FP64 steps
    a, b = melts["mixed"].get_state(), melts["global"].get_state()
    assert np.array_equal(a["x"], b["x"]) and np.array_equal(a["v"], b["v"])
    assert melts["mixed"].nl_info()["K"] == 5
    assert melts["mixed"].nl_info()["mean_list"] == melts["global"].nl_info()["mean_list"]


def test_lists_on_both_sides_of_the_run():
    # rows and lists on both sides of 32, in the same wavefronts
    test_lists_at_the_edges(dict(M=64, N=100, rho=1.5))


@pytest.mark.parametrize("shape", [(5, 5), (5, 3), (3, 5)])
def test_frames_that_wrap_keep_their_stage(shape):
    # 5 cells a side: frames of 7 cells hold some cells twice, in x, in y or in both; the record of
    # their stage keeps which one a member is.  The mixed path equals the one that reads global memory
    # at every step, bit for bit.
    kw = dict(M=20, N=50, seed=3, kappa=1.0, warmup_steps=200, nl_every=5, precision=1)
    flat, wrapped = kg.Melt(test_flags=kg.TF_NL_GLOBAL, **kw), kg.Melt(**kw)
    wrapped.set_tiles(*shape)
    for m in (flat, wrapped):
        m.md_steps(60)
        m.db_sweep(40)
        m.md_steps(35)
    assert wrapped.nl_stats()["stage_overflows"] == 0
    s0, s1 = flat.get_state(), wrapped.get_state()
    for f in ("x", "v", "fl", "fc", "chains"):
        assert np.array_equal(s0[f], s1[f]), f


def test_small_melts_take_other_tiles_in_a_large_batch():
    # a mixed batch that leaves CUs idle takes tiles of one wavefront, a larger one full tiles; the
    # trajectory is the same, bit for bit
    small = dict(M=40, N=100, kappa=1.0, warmup_steps=100, nl_every=5, precision=1)
    alone = kg.Melt(seed=1, melt_id=0, **small)
    batch = kg.Batch([dict(small, seed=1, melt_id=0),
                      dict(M=300, N=200, kappa=1.0, seed=1, melt_id=1, warmup_steps=100, nl_every=5, precision=1)])
    assert alone.nl_stats()["tile_shape"] != batch.nl_stats()["tile_shape"]
    for m in (alone, batch):
        m.md_steps(60)
        m.db_sweep(40)
        m.md_steps(35)
    s0, s1 = alone.get_state(), batch.get_state(0)
    for f in ("x", "v", "fl", "fc", "chains"):
        assert np.array_equal(s0[f], s1[f]), f


@pytest.mark.parametrize("melts,kw,shapes", [
    (1, dict(M=500, N=100, rho=0.1, nl_every=2), [(15, 9), (9, 15)]),
    (3, dict(M=80, N=100, rho=0.85, dt=0.02, nl_every=5), [(3, 3)]),
    (3, dict(M=100, N=100, rho=0.85, dt=0.02, nl_every=5), [(2, 5), (5, 2)]),
])
def test_shapes_of_the_home_cost_fit_the_tile_map(melts, kw, shapes):
    # shapes among the three cheapest by the cost of a home monomer, whatever the batch's own candidates are
    b = kg.Batch([dict(kw, seed=2, melt_id=i, warmup_steps=0, precision=1) for i in range(melts)])
    for s in shapes:
        b.set_tiles(*s)
        assert b.nl_stats()["tile_shape"] == s


@pytest.mark.parametrize("kw,tiles", [
    (dict(nl_every=2), 880),           # 11 x 9 cells of 232 homes; three deviations in hand: 1,056, 24% slower
    (dict(nl_every=5, T=2.0), 900),    # 6 x 5 of 222; two deviations in hand: 960, 11% slower
    (dict(nl_every=5), 952),
])
def test_tiles_of_a_full_chip_run_at_once(kw, tiles):
    m = kg.Melt(M=200, N=1000, kappa=2.0, warmup_steps=0, precision=1, **kw)
    assert m.nl_stats()["tiles"] == tiles and tiles <= 4 * 256


def test_stage_capacity_follows_the_exponent():
    # FP64: the smaller stage that makes room for a fourth workgroup a CU is for the steps of n = 2 and 12; the
    # step of a general exponent runs two and keeps the stage's full room
    m = kg.Melt(M=200, N=1000, kappa=2.0, warmup_steps=0, precision=0, nl_every=5, n_exp=3.0)
    wide = m.nl_stats()["stage_cap"]
    seen = [wide]
    for n in (2.0, 12.0, 5.75):
        m.set_potential(n)
        seen.append(m.nl_stats()["stage_cap"])
    assert wide > 1472 and seen == [wide, 1472, 1472, wide]


def test_step_time_of_long_lists():
    # 50,000 monomers at T = 2, whose lists hold 30 entries (a wider skin) instead of 19: 1.24 times the step
    # time of T = 1 (1.57 times when lists past the run were built a second time)
    t = []
    for T in (1.0, 2.0):
        m = kg.Melt(M=250, N=200, kappa=1.0, T=T, seed=3, warmup_steps=500, precision=1, nl_every=5)
        m.md_steps(400)
        t.append(1e9)
        for _ in range(12):
            t0 = time.perf_counter()
            m.md_steps(200)
            t[-1] = min(t[-1], time.perf_counter() - t0)
        assert m.nl_info()["K"] == 5
    assert t[1] < 1.5 * t[0]
