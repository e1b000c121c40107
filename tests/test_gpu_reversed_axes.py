"""Boxes along the axes whose elements are numbered with two reference axes
reversed (turned by 180 degrees about the third): Ja is diagonal with negative
entries and the outward normal of face 2d+1 is -e_d.  U_t and RK steps against
the oracle on the structured box, node for node through the relabelling, at the
bar of the other oriented meshes; and in a batch, whose launch also holds boxes
numbered along the axes, or full-metric elements, bit for bit as alone."""
import numpy as np
import pytest

import helpers
from helpers import oracle_for, oracle_init
from paper_2208_05310_amd import workloads as wl
from test_gpu_curved import (TOL, gpu_solver, perturbed_state, rotated_solver, state_err, term_scale, to_gpu,  # noqa: F401
                             torch_cuda)
from test_gpu_stage_variants import alone_and_batched

pytestmark = pytest.mark.gpu

TURN = {a: np.diag([1 if d == k else -1 for d in range(3)]) for k, a in enumerate("xyz")}
PERIODIC, WALL, MOVING = wl.c1().with_(n=(3, 3, 3)), wl.c4(scale=12), wl.c5(scale=10)
# every element turned about one axis, or a part of them about any
CASES = [("periodic_N3_x", PERIODIC, "x"), ("periodic_N3_y", PERIODIC, "y"), ("periodic_N3_z", PERIODIC, "z"),
         ("wall_N2_y", WALL.with_(N=2), "y"), ("wall_N4_z", WALL.with_(N=4, n=(3, 3, 2)), "z"),
         ("moving_N3_x", MOVING, "x"), ("periodic_N5_mixed", PERIODIC.with_(N=5, n=(2, 3, 2)), "1xyz"),
         ("wall_N3_mixed", WALL, "1xyz"),
         ("model2_N4_mixed", PERIODIC.with_(N=4, params=dict(wl.TABLE1, model=2)), "1x")]
IDS = [c[0] for c in CASES]


def turned_solver(monkeypatch, w, turns, precision="fp64"):
    """Each element of w's box turned by one of `turns` (1: as it is)."""
    monkeypatch.setattr(helpers, "cube_rotations",
                        lambda: [np.eye(3, dtype=int) if a == "1" else TURN[a] for a in turns])
    out = rotated_solver(w, precision)
    monkeypatch.undo()
    return out


@pytest.mark.parametrize("name,w,turns", CASES, ids=IDS)
def test_rhs_and_steps_match_the_oracle(torch_cuda, monkeypatch, name, w, turns):  # noqa: F811
    torch = torch_cuda
    print(f"[case] reversed axes {name}", flush=True)
    o = oracle_for(w)
    s, perm = turned_solver(monkeypatch, w, turns)
    V = perturbed_state(o, w)
    Ut = s.rhs(to_gpu(torch, V[:, perm]), s.new_state())
    torch.cuda.synchronize()
    scale, _, ref = term_scale(o, V, w.params)
    err = np.max(np.abs(Ut.cpu().numpy() - ref[:, perm]), axis=1) / scale
    print("rhs", err, flush=True)
    U = oracle_init(o, w)
    dt = o.dt(U)
    Ug = to_gpu(torch, U[:, perm])
    s.rk_steps(Ug, s.new_state(), dt, 5)
    torch.cuda.synchronize()
    o.run(U, np.zeros_like(U), 0.0, dt, 5)
    err_s = state_err(Ug.cpu().numpy(), U[:, perm], w.params)
    print("steps", err_s, flush=True)
    assert np.all(err <= TOL), err
    assert np.all(err_s <= TOL), err_s


@pytest.mark.parametrize("prec", ("fp64", "fp32_mixed"))
@pytest.mark.parametrize("other", ("1", "xyz1", "full"))
def test_batched_equals_alone_bitwise(torch_cuda, monkeypatch, prec, other):  # noqa: F811
    torch = torch_cuda
    from paper_2208_05310_amd.nskr import init_workload
    print(f"[case] reversed axes batched {other} {prec}", flush=True)
    held = []
    for w, turns in ((PERIODIC, "y"), (WALL, "1xyz")):
        s, perm = turned_solver(monkeypatch, w, turns, prec)
        held.append((s, to_gpu(torch, oracle_init(oracle_for(w), w)[:, perm], s.dtype)))
    if other == "full":
        s, perm = rotated_solver(PERIODIC, prec)
        held.append((s, to_gpu(torch, oracle_init(oracle_for(PERIODIC), PERIODIC)[:, perm], s.dtype)))
    elif other == "1":
        s = gpu_solver(PERIODIC, prec)
        held.append((s, init_workload(s, PERIODIC)))
    alone, batched = alone_and_batched(torch, held, 3)
    for a, b in zip(alone, batched):
        assert torch.equal(a, b)
