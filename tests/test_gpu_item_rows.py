"""The automatic item height and kernel choice depend on what a call asks for (energies, traces,
storage type): calls of different kinds follow one another on one context, and the states, energies
and traces are those of one fixed configuration (states and traces bit for bit; energies within the
oracle bar's 1e-12 in FP64 and 1e-6 of FP32 sums)."""
import numpy as np
import pytest

from paper_2005_11931_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("dtype_name,sizes", [("f64", [1100]), ("f32", [1250]), ("f64", [90, 700, 1300]),
                                              ("f32", [64, 1100])])
def test_mixed_calls_equal_one_configuration(dtype_name, sizes, graph):
    import torch

    from paper_2005_11931_amd import fdw

    dt = fdw.FDW_F64 if dtype_name == "f64" else fdw.FDW_F32
    cases = [I.line_case(n=n, nsteps=60, width2=0.05) for n in sizes]
    rec = torch.as_tensor(np.array([[5, 7], [30, 7], [sizes[0] // 2, sizes[0] // 2]], dtype=np.int32))
    print("mixed calls", dtype_name, sizes, graph, flush=True)
    out = []
    for fixed in (True, False):
        s = fdw.family_solver(cases, dtype=dt)
        s.configure(fdw.FDW_CFG_USE_GRAPH, graph)
        if fixed:
            s.configure(fdw.FDW_CFG_SMALL_TILES, 1)
            s.configure(fdw.FDW_CFG_SEGMENT_ROWS, 16)
        e = [s.step(9, energy=True)]
        s.step(10)
        tr = s.record_traces(rec)
        s.step(7)
        e.append(s.step(9, energy=True))
        s.record_traces(None)
        s.step(12)
        e.append(s.step(13, energy=True))
        st = [[t.cpu().numpy() for t in s.get_state(m)[:2]] for m in range(len(sizes))]
        out.append((st, torch.cat(e, dim=1).cpu().numpy(), tr.cpu().numpy()))
        s.close()
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert np.array_equal(out[0][2], out[1][2])
    assert np.allclose(out[0][1], out[1][1], rtol=1e-12 if dt == fdw.FDW_F64 else 1e-6, atol=0)
