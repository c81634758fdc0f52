"""The one-workgroup PCG of small systems: its iterates against a CG on the
host, its forms, threads and launches."""
import threading

import numpy as np
import pytest
import torch

from paper_1708_01773_amd import fe as F
from tests.gpu_util import Pair, rel, say

pytestmark = pytest.mark.gpu


def test_threads_solve_small_systems_of_different_lds_sizes():
    """Systems that need 70 to 150 KB of LDS, each thread its own, at the same
    time: every solve launches with what its system needs and gives the bits
    of the solve alone."""
    pairs = [Pair(3, [8, 8, 8], 1, seed=101), Pair(2, [33, 33], 1, seed=102), Pair(2, [38, 38], 1, seed=103),
             Pair(3, [8, 9, 9], 1, seed=104)]
    systems = []
    for p in pairs:
        A = p.gpu_assembly()
        ws = torch.empty(F.pcg_query(A.n_rows), dtype=torch.uint8, device="cuda")
        x = torch.zeros(A.n_rows, dtype=torch.float64, device="cuda")
        info = F.pcg_solve(A.csr, A.rhs, x, 1e-10, 2000, ws)
        lds = 16 * A.n_rows + 4 * A.n_rows + 10 * A.nnz
        say(f"[threads] rows {A.n_rows} nnz {A.nnz} lds about {lds}")
        assert info["status"] == F.FE_OK and 64 * 1024 < lds < 156 * 1024
        systems.append((A, ws, x, info))
    torch.cuda.synchronize()
    bad = []

    def work(A, ws, ref, info):
        try:
            s = torch.cuda.Stream()
            x = torch.empty_like(ref)
            with torch.cuda.stream(s):
                for _ in range(40):
                    x.zero_()
                    i = F.pcg_solve(A.csr, A.rhs, x, 1e-10, 2000, ws, s)
                    if i != info or not torch.equal(x, ref):
                        bad.append((A.n_rows, i))
                        return
        except Exception as e:  # reported by the main thread
            bad.append((A.n_rows, repr(e)))

    ts = [threading.Thread(target=work, args=s) for s in systems]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
