"""Reading a melt's state where its read-out ends: an odd number of monomers, arrays and the chain table
cut by the 2 MB chunks, a melt that starts at an odd slot of its batch."""
import numpy as np
import pytest

from oracle import oracle as o
from tests import inputs

pytestmark = pytest.mark.gpu

kg = pytest.importorskip("paper_2109_11001_amd")
torch = pytest.importorskip("torch")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("M,N", [(7, 31), (21, 1041), (131, 211), (400, 111)])
def test_state_in_id_order(M, N):
    # a chunk holds 262,144 words: 217 monomers take one, 21,861 end inside the chain table, 27,641 inside
    # the last force array, 44,400 take three chunks
    kw = dict(kappa=1.0, nl_every=5, warmup_steps=120, precision=0)
    om = o.Melt(M=M, N=N, seed=4, warmup_steps=120, kappa=1.0)
    b = kg.Batch([dict(M=7, N=31, seed=9, **kw), dict(M=M, N=N, seed=4, **kw)])
    st = om.get_state()
    st["v"] = np.clip(inputs.random_velocities(M * N, 5), -3.0, 3.0)
    full = dict(x=st["x"], v=st["v"], fl=st["fl"], chains=st["chains"], counters=st["counters"])
    om.set_state(**full)
    b.set_state(1, **full)
    s = b.get_state(1)
    for f in ("x", "v", "fl", "chains"):
        assert np.array_equal(s[f], om.get_state()[f]), f
    # now out of id order in the storage: a few steps (the lists sort it), a sweep, a few steps more
    for m in (om, b):
        m.md_steps(6)
        m.db_sweep(M)
        m.md_steps(3)
    s, t = b.get_state(1), om.get_state()
    d = s["x"] - t["x"]
    d -= om.L * np.rint(d / om.L)
    assert np.max(np.abs(d)) < 1e-11 and np.max(np.abs(s["v"] - t["v"])) < 1e-9  # as short FP64 windows elsewhere
    assert np.array_equal(s["chains"], t["chains"])
    # an array asked for alone is the one of the whole state
    F, S, _ = b.forces(1)
    Ft, St, _ = om.forces()
    assert np.all(np.abs(F - Ft) <= 1e-9 * np.maximum(St, 1.0)) and np.all(np.abs(S - St) <= 1e-9 * np.maximum(St, 1.0))


@pytest.mark.parametrize("M,N", [(7, 31), (400, 111)])
def test_some_arrays_of_a_state(M, N):
    # any of a state's arrays may be left out: the others are those of the whole state, and nothing else of the
    # caller's memory is written (44,400 monomers: chunks end inside arrays)
    b = kg.Batch([dict(M=5, N=33, seed=9, warmup_steps=50), dict(M=M, N=N, seed=4, kappa=1.0, warmup_steps=50)])
    b.md_steps(4)
    full = b.get_state(1)
    names = ("x", "v", "fc", "fl", "chains")
    L = kg.load()
    for take in (("x",), ("v", "chains"), ("fc",), ("fl", "x"), ("chains",), ("v", "fc", "fl"), ()):
        guard = 64
        bufs = {f: np.full(full[f].size + 2 * guard, -77, full[f].dtype) for f in take}
        args = [kg.ptr(bufs[f][guard:]) if f in take else None for f in names]
        kg.check(L.kgdb_get_state(b._h, 1, *args, None))
        for f in take:
            assert np.array_equal(bufs[f][guard:-guard], full[f].ravel()), (take, f)
            assert np.all(bufs[f][:guard] == -77) and np.all(bufs[f][-guard:] == -77), (take, f)
