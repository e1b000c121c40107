"""The instances that the launches choose between, against the oracle or each
other: parallelepipeds whose metric is full against boxes along the axes, walls
or none, long meshes (each workgroup of the first lifting handles several
groups of elements) against the plain kernel that a batch runs, and the nodal
reductions where a workgroup handles several tiles."""
import numpy as np
import pytest

from helpers import oracle_for, oracle_init, rotated_box_mesh
from paper_2208_05310_amd import workloads as wl
from test_gpu_parity import TOL, gpu_solver, perturbed_state, rhs_term_scale, to_gpu, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def turned(w):
    """The box of w turned rigidly out of the axes, and the rotation."""
    from paper_2208_05310_amd.nskr import Solver, box_mesh
    Q, _ = np.linalg.qr(np.random.default_rng(5).standard_normal((3, 3)))
    if np.linalg.det(Q) < 0:
        Q[:, 0] = -Q[:, 0]
    corners, nbr, nbf, bc, bcs = box_mesh(w.n, w.length, w.periodic, w.side_kind, w.side_twall, w.side_theta)
    s = Solver(w.params, w.N, "fp64")
    s.upload_mesh(corners @ Q.T, nbr, nbf, bc, bcs)
    return s, Q


# tiles with a remainder at every degree
TURNED = [wl.c4(scale=12).with_(name="turned_wall_5x3x3_N2", N=2, n=(5, 3, 3), length=(1.0, 0.6, 0.6)),
          wl.c1().with_(name="turned_3x3x5_N3", N=3, n=(3, 3, 5), length=(1.0, 1.0, 1.7)),
          wl.c4(scale=12).with_(name="turned_wall_3x3x3_N4", N=4, n=(3, 3, 3), length=(1.0, 1.0, 1.0)),
          wl.c1().with_(name="turned_3x2x1_N5", N=5, n=(3, 2, 1), length=(1.5, 1.0, 0.5))]


@pytest.mark.parametrize("w", TURNED, ids=[w.name for w in TURNED])
def test_turned_boxes_match_the_oracle(torch_cuda, w):  # noqa: F811
    """U_t of the turned box is the turned U_t of the box.  The turned metric
    and momenta carry three more roundings each than those of the box, on top
    of what the parity bar holds some tens of times over."""
    torch = torch_cuda
    print(f"[case] {w.name}", flush=True)
    o = oracle_for(w)
    U = perturbed_state(o, w)
    s, Q = turned(w)
    V = U.copy()
    V[1:4] = Q @ U[1:4]
    Ut = s.new_state()
    s.rhs(to_gpu(torch, V), Ut)
    got = Ut.cpu().numpy()
    got[1:4] = Q.T @ got[1:4]
    scale, ref = rhs_term_scale(o, U, w.params)
    err = np.max(np.abs(got - ref), axis=1) / scale
    print("errors", err, flush=True)
    assert np.all(err <= TOL), err


def alone_and_batched(torch, solvers, nsteps):
    """Each solver's state after nsteps on its own, and in one batch."""
    from paper_2208_05310_amd.nskr import Batch
    b = Batch(64 << 30)
    alone, held = [], []
    for s, U in solvers:
        dt = 0.5 * s.dt(U)
        A, B = U.clone(), U.clone()
        s.rk_steps(A, s.new_state(), dt, nsteps)
        torch.cuda.synchronize()
        assert torch.isfinite(A).all()
        R = s.new_state()
        assert b.admit(s, B, R, dt, nsteps) is not None
        alone.append(A)
        held.append((B, R))
    stream = torch.cuda.Stream()
    for _ in range(nsteps):
        b.step(stream)
    stream.synchronize()
    return alone, [h[0] for h in held]


@pytest.mark.parametrize("N", (2, 3, 4, 5))
@pytest.mark.parametrize("prec", ("fp64", "fp32_mixed"))
def test_mixed_group_equals_single_bitwise(torch_cuda, N, prec):  # noqa: F811
    """Boxes, boxes with walls and relabelled elements (whose Ja is not
    diagonal) of one degree share a batch's launch, and with it the instance
    with walls and the full metric; alone each has its own instance."""
    torch = torch_cuda
    from paper_2208_05310_amd.nskr import Solver, init_workload
    box = wl.c1().with_(N=N, n=(3, 3, 3))
    wall = wl.c4(scale=12).with_(N=N)
    turn = wl.c1().with_(N=N, n=(2, 3, 3))
    solvers = []
    for w in (box, wall):
        s = gpu_solver(w, prec)
        solvers.append((s, init_workload(s, w)))
    m = rotated_box_mesh(turn)
    s = Solver(turn.params, N, prec)
    s.upload_mesh(m["xgeo"], m["nbr"], m["nbf"], m["bc"], m["bcs"], ngeo=m["ngeo"], nbo=m["nbo"])
    solvers.append((s, to_gpu(torch, oracle_init(oracle_for(turn), turn)[:, m["perm"]], s.dtype)))
    alone, held = alone_and_batched(torch, solvers, 3)
    for a, h in zip(alone, held):
        assert torch.equal(a, h)


# from four groups of elements for each workgroup that the card holds on
LONG = [(2, (42, 42, 42), "fp32_mixed"), (3, (33, 32, 32), "fp64"), (4, (26, 26, 25), "fp32_mixed"),
        (5, (19, 18, 19), "fp64"), (5, (19, 18, 21), "fp32_mixed")]


@pytest.mark.parametrize("N,n,prec", LONG, ids=[f"N{N}_{p}" for N, _, p in LONG])
def test_long_mesh_equals_plain_kernel_bitwise(torch_cuda, N, n, prec):  # noqa: F811
    torch = torch_cuda
    from paper_2208_05310_amd.nskr import init_workload
    w = wl.c1().with_(N=N, n=n)
    s = gpu_solver(w, prec)
    alone, held = alone_and_batched(torch, [(s, init_workload(s, w))], 2)
    assert torch.equal(alone[0], held[0])


# one tile more than 1024 or a few, the last one ragged; and a single element
TILES = [(2, (22, 21, 20)), (3, (17, 16, 16)), (4, (13, 13, 13)), (5, (11, 11, 9)), (5, (1, 1, 1))]


@pytest.mark.parametrize("N,n", TILES, ids=[f"N{N}_{n[0]}x{n[1]}x{n[2]}" for N, n in TILES])
@pytest.mark.parametrize("wall", (False, True))
def test_reductions_over_many_tiles(torch_cuda, N, n, wall):  # noqa: F811
    """Time step and integrals where a workgroup handles more than one tile.
    Extrema differ by the last roundings of their arguments; sums over up to
    2.5e5 nodes by the order of summation, sqrt(n) eps = 5e-14 each way."""
    torch = torch_cuda
    w = (wl.c4(scale=12) if wall else wl.c1()).with_(N=N, n=n, length=(1.0, 1.0, 1.0))
    print(f"[case] {w.name} N={N} {n}", flush=True)
    o = oracle_for(w)
    U = perturbed_state(o, w)
    s = gpu_solver(w)
    Ug = to_gpu(torch, U)
    do = o.dt(U)
    assert abs(s.dt(Ug) - do) <= 1e-13 * do
    assert s.dt_noalloc(Ug) == s.dt(Ug)
    rg, ro = s.reduce(Ug), o.reduce(U)
    assert ro[19] == pytest.approx(1.0, rel=1e-11)
    ro[19] = 1.0  # the volume: the oracle's serial sum of equal terms drifts from it by up to 4e-12
    for k in range(20):
        scale = max(abs(ro[0]), 1.0) if k in (1, 2, 3) else abs(ro[k])
        assert abs(rg[k] - ro[k]) <= 1e-12 * scale + 1e-300, (k, rg[k], ro[k])


@pytest.mark.parametrize("N", (4, 5))
@pytest.mark.parametrize("prec", ("fp64", "fp32_mixed"))
@pytest.mark.parametrize("curve", (0.0, 0.02))
def test_few_tiles_equal_many_bitwise(torch_cuda, N, prec, curve):  # noqa: F811
    """A small mesh updates one element per workgroup alone, and a tile of four
    in a batch whose group has more than 768 tiles (1024 + 7 + 16)."""
    torch = torch_cuda
    from paper_2208_05310_amd.nskr import init_workload
    solvers = []
    for n in ((3, 3, 3), (16, 16, 16), (8, 8, 1)):
        w = wl.c1().with_(N=N, n=n, curve_amp=curve)
        s = gpu_solver(w, prec)
        solvers.append((s, init_workload(s, w)))
    alone, held = alone_and_batched(torch, solvers, 2)
    for a, h in zip(alone, held):
        assert torch.equal(a, h)
