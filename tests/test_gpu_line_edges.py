"""Line solver of the implicit scheme at the edges of its decomposition, against the oracle's Thomas
algorithm: x lines around the changes of chunk length and around lines that fill their threads
exactly; y lines around the change from column strips to blocks of 64 rows, with full and partial
last chunks, blocks and strips.  Bars as for the other parity tests of the scheme: FP64 within 1e-12
of the amplitude, FP32 within 1e-5 of the largest value."""
import math
import sys

import numpy as np
import pytest

import oracle
from paper_2005_11931_amd import inputs as I

pytestmark = pytest.mark.gpu


def _case(nx, ny, N):
    x, y, X, Y = I.mesh(nx, ny)
    h1 = 1.0 + 0.5 * np.exp(-((X + 0.2) ** 2) / 0.02) + 0.2 * Y
    h2 = 0.9 + 0.3 * np.cos(3 * X) * np.sin(2 * Y)
    u0 = I.zero_ring(np.exp(-((X - 0.1) ** 2 + (Y + 0.2) ** 2) / 0.05))
    u1 = I.zero_ring(0.2 * np.exp(-((X + 0.4) ** 2 + (Y - 0.3) ** 2) / 0.05))
    dx, dy = 2.0 / (nx - 1), 2.0 / (ny - 1)
    tau = 3.0 * 2.0 / math.sqrt(4 * h1.max() / dx**2 + 4 * h2.max() / dy**2)
    return I.Case("edges", nx, ny, -1, 1, -1, 1, tau, N, h1, h2, u0, u1)


@pytest.mark.parametrize("dtype_name,nx,ny", [
    (d, nx, ny) for d in ("f64", "f32")
    for nx, ny in [(257, 34), (258, 35), (513, 12), (514, 13), (515, 14), (1026, 9), (4354, 5),  # x chunks
                   (35, 514), (36, 515), (65, 1026), (66, 1027), (64, 1090), (130, 1091), (67, 2200),  # y lines
                   (1700, 40), (1537, 600)]  # strips of several columns
] + [("f32", 4609, 6), ("f32", 4610, 6), ("f32", 5, 8450)])
def test_line_solver_edges(dtype_name, nx, ny):
    from paper_2005_11931_amd import fdw

    dt = fdw.FDW_F64 if dtype_name == "f64" else fdw.FDW_F32
    case = _case(nx, ny, 12)
    print("line edges", dtype_name, nx, ny, flush=True)
    sys.stdout.flush()
    s = fdw.implicit_solver_for_case(case, sigma=0.25, dtype=dt)
    s.step(12)
    u, du, _ = (t.cpu().numpy().astype(np.float64) if hasattr(t, "cpu") else t for t in s.get_state())
    s.close()
    ref = oracle.adi_forward_case(case, sigma=0.25)
    if dt == fdw.FDW_F64:
        assert np.abs(u - ref["u_cur"]).max() <= 1e-12
        assert np.abs(du - (ref["u_cur"] - ref["u_prev"])).max() <= 1e-12
    else:
        assert np.abs(u - ref["u_cur"]).max() <= 1e-5 * np.abs(ref["u_cur"]).max()
    # boundary ring untouched
    for a in (u, du):
        assert not a[0].any() and not a[-1].any() and not a[:, 0].any() and not a[:, -1].any()
