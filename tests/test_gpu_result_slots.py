"""More contexts than the block of reduction results has slots (256): each
context's time step and integrals are its own, in any order, from several host
threads with a stream each, and after some contexts have given their slots back."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from paper_2208_05310_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_results_of_many_contexts():
    import torch
    from paper_2208_05310_amd.nskr import init_workload, solver_for
    w = wl.c1().with_(N=2, n=(2, 2, 2))

    def make(k):
        s = solver_for(w.with_(length=(1.0 + 0.01 * k, 1.0, 1.0)))
        return s, init_workload(s, w)

    def results(c):
        return np.concatenate([[c[0].dt(c[1])], c[0].reduce(c[1])])

    held = [make(k) for k in range(264)]
    first = [results(c) for c in held]
    assert len({r[0] for r in first}) == len(held)  # every context has its own time step

    def worker(j):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            return [(k, results(held[k])) for _ in range(3) for k in range(len(held) - 1 - j, -1, -4)]

    def agree():
        torch.cuda.synchronize()
        with ThreadPoolExecutor(4) as pool:
            for part in pool.map(worker, range(4)):
                for k, r in part:
                    assert np.array_equal(r, first[k]), k

    print("[case] 264 contexts, 4 threads", flush=True)
    agree()
    for k in range(3, len(held), 5):
        held[k] = None  # gives its slot back
    for k in range(3, len(held), 5):
        held[k] = make(k)
    print("[case] a fifth of them made again", flush=True)
    agree()
