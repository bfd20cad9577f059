"""The automatic choices (small-grid tiles, their rows, rows per streaming item) go by what one launch
holds.  Members that differ in coefficient layout are launched one by one: such a family takes the
choices of its members alone, not those of all their nodes together; members of one layout share
their launches, and the choices with them."""
import numpy as np
import pytest

from paper_2005_11931_amd import inputs as I

pytestmark = pytest.mark.gpu


def _cases(n, members, mixed):
    out = []
    for m in range(members):
        x, y, X, Y = I.mesh(n, n)
        h = 1.0 + 0.3 * np.cos(3 * X + Y + m) + I.gaussian_1d(X, 0.1)
        h2 = 1.0 + 0.2 * np.sin(2 * Y - m) * np.ones_like(h)
        u0 = I.zero_ring(np.exp(-((X - 0.1 * m) ** 2 + Y**2) / 0.02))
        out.append(I.Case(f"rule{m}", n, n, -1, 1, -1, 1, 0.2 * 2.0 / (n - 1), 24, h, h2 if mixed and m % 2 else None, u0,
                          np.zeros_like(u0)))
    return out


# 1024^2 FP32 and 1000^2 FP64: streamed where three of them share a launch, tiles alone; 400^2: tiles of
# 32 rows alone and of 48 for a dozen; 1300^2: streamed either way, in items of other heights
@pytest.mark.parametrize("dtype_name,n,members", [("f64", 1000, 3), ("f32", 1024, 3), ("f64", 400, 12), ("f64", 1300, 4),
                                                  ("f32", 1300, 4)])
def test_mixed_layouts_choose_per_launch(dtype_name, n, members):
    from paper_2005_11931_amd import fdw

    dt = fdw.FDW_F64 if dtype_name == "f64" else fdw.FDW_F32
    cases = _cases(n, members, True)
    keys = (fdw.FDW_CFG_TILE_ROWS, fdw.FDW_CFG_SEGMENT_ROWS)
    print("launch rules", dtype_name, n, members, flush=True)
    alone, states = [], []
    for c in cases[:2]:
        s = fdw.solver_for_case(c, dtype=dt)
        s.step(24)
        alone.append([s.config(k) for k in keys])
        states.append([t.cpu().numpy() for t in s.get_state()[:2]])
        s.close()
    assert alone[0] == alone[1]
    s = fdw.family_solver(cases, dtype=dt)
    s.step(24)
    assert [s.config(k) for k in keys] == alone[0]
    for m in range(2):
        for a, b in zip(states[m], s.get_state(m)[:2]):
            assert np.array_equal(a, b.cpu().numpy()), m
    s.close()


@pytest.mark.parametrize("mixed", [False, True])
def test_family_takes_tiles_by_the_launch(mixed):
    """FP64 energies name the kernel: tiles and streaming items sum them in another order.  Three members
    of 700^2 nodes are beyond the tiles' range in one launch, and within it one by one."""
    from paper_2005_11931_amd import fdw

    cases = _cases(700, 3, mixed)
    print("tiles by the launch", mixed, flush=True)
    got = {}
    for mode in (0, 1, 2):
        s = fdw.family_solver(cases, dtype=fdw.FDW_F64)
        s.configure(fdw.FDW_CFG_SMALL_TILES, mode)
        got[mode] = s.step(24, energy=True).cpu().numpy()
        s.close()
    assert not np.array_equal(got[1], got[2])
    assert np.array_equal(got[0], got[2 if mixed else 1])


def test_gradient_of_a_family_member_equals_its_own():
    """The replay of a member's gradient is launched for that member alone, whatever the family holds."""
    import torch

    from paper_2005_11931_amd import fdw

    cases = _cases(400, 12, False)
    rec = torch.as_tensor(np.array([[50, 60], [200, 200], [333, 60]], dtype=np.int32))
    tg = torch.as_tensor(np.random.default_rng(4).normal(size=(25, 3)))
    print("family gradient", flush=True)
    a = fdw.solver_for_case(cases[5], dtype=fdw.FDW_F64)
    b = fdw.family_solver(cases, dtype=fdw.FDW_F64)
    ga = a.adjoint(rec, tg, ckpt_every=10).cpu().numpy()
    gb = b.adjoint(rec, tg, ckpt_every=10, member=5).cpu().numpy()
    a.close(), b.close()
    assert np.abs(ga).max() > 0 and np.array_equal(ga, gb)
