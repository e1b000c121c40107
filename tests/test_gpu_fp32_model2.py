"""U_t in FP32-mixed for relaxation model 2 on ragged meshes, where the
divergence of p_alpha and the source all but cancel and each rounding of a value
of the size of p_alpha shows: against stored values of an evaluation that sums
volume and surface terms in one accumulator and rounds every flux once
(golden/ut_fp32_model2.json: every `stride`-th node of the droplet's interface;
the library of commit da4c5de).

The bars are those of an FP32 result against another evaluation of it: 2e-5 in
the 2-norm, and 40 times that for one value against the larger of itself and the
root mean square.  (Volume parts and fluxes rounded once more on their way
through memory: 2.2e-5 to 8.3e-5; kept apart: 2e-7 to 7e-7.)

The state is made of sums, products and quotients of doubles alone, so that the
inputs are the same on every machine."""
import json
import os

import numpy as np
import pytest

from paper_2208_05310_amd import workloads as wl

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "ut_fp32_model2.json")
# name: degree, elements, extents, floor and lid (None: periodic), curvature
MESHES = {
    "N2_38x35x34": (2, (38, 35, 34), (1.0, 1.0, 1.0), False, 0.0),
    "N3_27x25x23": (3, (27, 25, 23), (1.0, 1.0, 1.0), False, 0.0),
    "N4_19x18x17": (4, (19, 18, 17), (1.0, 1.0, 1.0), False, 0.0),
    "N5_17x15x14": (5, (17, 15, 14), (1.0, 1.0, 1.0), False, 0.0),
    "N4_wall_23x22x11": (4, (23, 22, 11), (1.0, 1.0, 0.5), True, 0.0),
    "N4_curved_19x18x17": (4, (19, 18, 17), (1.0, 1.0, 1.0), False, 0.02),
}


def state(N, n, length):
    """A droplet of smooth rational profile moving through a swirl."""
    x1 = np.round(np.polynomial.legendre.leggauss(N + 1)[0], 9)
    h = [length[d] / n[d] for d in range(3)]
    axis = [((np.arange(n[d])[:, None] + 0.5 * (x1[None] + 1.0)) * h[d]) for d in range(3)]
    # nodes as [ez, ey, ex, k, j, i]
    X = [axis[d].reshape([n[d] if q == 2 - d else (N + 1 if q == 5 - d else 1) for q in range(6)]) for d in range(3)]
    r2 = sum((X[d] - 0.5 * length[d]) * (X[d] - 0.5 * length[d]) for d in range(3)) / 0.04
    r4 = r2 * r2
    s = 1.0 / (1.0 + r4 * r4)
    bump = [16.0 * (X[d] / length[d]) * (X[d] / length[d]) * (1.0 - X[d] / length[d]) * (1.0 - X[d] / length[d])
            for d in range(3)]
    rho = 0.32 + 1.45 * s
    u = [0.05 * s + 0.02 * bump[1], 0.03 * bump[0] - 0.04 * s, 0.02 * bump[0] * bump[1] * bump[2]]
    c = rho + 0.0001 * bump[0] * bump[2]
    p = wl.TABLE1
    g = 1.45 * 4.0 * r4 * r2 * s * s * 2.0 / 0.04  # |grad c| is g times the distance from the centre, up to the bumps
    E = (rho * (p["R"] * p["cv"] * 0.85 - p["a"] * rho) + 0.5 * p["alpha"] * (rho - c) * (rho - c) +
         0.5 * p["gam"] * g * g * r2 * 0.04 +
         0.5 * rho * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]))
    U = np.stack(np.broadcast_arrays(rho, rho * u[0], rho * u[1], rho * u[2], E, c))
    return np.ascontiguousarray(U.reshape(6, -1)).astype(np.float32)


def evaluate(name):
    """U_t at the interface's nodes of a mesh, [6, nodes]."""
    import torch
    from paper_2208_05310_amd.nskr import Solver
    N, n, length, wall, curve = MESHES[name]
    s = Solver(dict(wl.TABLE1, model=2), N, "fp32_mixed")
    if wall:
        s.upload_box(n, length, (1, 1, 0), (0, 0, 0, 0, wl.NOSLIP_CA, wl.SLIP), (0.0,) * 4 + (0.9, 0.0),
                     (90.0,) * 4 + (60.0, 90.0))
    else:
        s.upload_box(n, length, curve_amp=curve, ngeo=N if curve else 1)
    U = state(N, n, length)
    Ut = s.rhs(torch.tensor(U, device="cuda:0"), s.new_state())
    return Ut.cpu().numpy()[:, (U[0] > 0.4) & (U[0] < 1.7)]


@pytest.mark.parametrize("name", list(MESHES))
def test_rounds_like_one_accumulator(name):
    print(f"[case] {name}", flush=True)
    with open(GOLDEN, encoding="utf-8") as f:
        g = json.load(f)[name]
    got = evaluate(name)[:, ::g["stride"]].astype(np.float64)
    ref = np.array(g["ut"], dtype=np.float64).reshape(6, -1)
    d, rms = got - ref, np.linalg.norm(ref) / np.sqrt(ref.size)
    rel, most = np.linalg.norm(d) / np.linalg.norm(ref), np.max(np.abs(d) / np.maximum(np.abs(ref), rms))
    print("2-norm", rel, "max", most, flush=True)
    assert rel <= 2e-5 and most <= 8e-4, (rel, most)
