"""The pipelined first lifting (meshes of at least four groups of elements for
each workgroup that the card holds) against the plain kernel that a batch runs,
bit for bit, at every degree and precision.  A CU holds at most 8 waves per SIMD,
so 4 * 256 * 4 * 8 waves' worth of groups reach that rule whatever occupancy an
instance is built for; one row of elements more leaves a ragged last group."""
import pytest

from paper_2208_05310_amd import workloads as wl
from test_gpu_parity import gpu_solver, torch_cuda  # noqa: F401
from test_gpu_stage_variants import alone_and_batched

pytestmark = pytest.mark.gpu

# degree: elements of a group, waves of its workgroup, mesh
GROUPS = {2: (9, 4, (43, 42, 41)), 3: (2, 2, (33, 32, 33)), 4: (2, 4, (27, 25, 25)), 5: (1, 4, (21, 20, 20))}


@pytest.mark.parametrize("prec", ("fp64", "fp32_mixed"))
@pytest.mark.parametrize("N", list(GROUPS))
def test_pipelined_equals_plain_bitwise(torch_cuda, N, prec):  # noqa: F811
    torch = torch_cuda
    from paper_2208_05310_amd.nskr import init_workload
    elements, waves, n = GROUPS[N]
    assert n[0] * n[1] * n[2] >= 4 * (256 * 4 * 8 // waves) * elements
    print(f"[case] long N={N} {n} {prec}", flush=True)
    w = wl.c1().with_(N=N, n=n)
    s = gpu_solver(w, prec)
    alone, held = alone_and_batched(torch, [(s, init_workload(s, w))], 2)
    assert torch.equal(alone[0], held[0])
