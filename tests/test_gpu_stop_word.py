"""The layer loop follows the launches' progress in a pinned word, one launch
queued behind the one that runs: solves end where they should whatever ends them,
and none is misled by the word of the one before."""

import numpy as np
import pytest

from gpu_util import banner, to_dev
from workloads import random_orthogonal_hamiltonian

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import paper_2107_02737_amd as pk
    pk.load_library()
    return pk


@pytest.mark.parametrize("max_iter", [1, 2, 3, 4, 9, 100])
def test_layer_cap_and_stop(pk, max_iter):
    """A capped solve applies exactly max_iter layers, those of the full one."""
    H = to_dev(random_orthogonal_hamiltonian(130, 65, seed=3).astype(np.float32))
    banner(f"stop word max_iter={max_iter}")
    opts = dict(precision="fp16x3", refine="none", return_info=True)
    _, full = pk.density(H, 65, **opts)
    ref = pk.sp2_history(full["workspace"])
    _, info = pk.density(H, 65, max_iter=max_iter, allow_unconverged=True, **opts)
    hist = pk.sp2_history(info["workspace"])
    k = min(max_iter, full["n_iter"])
    assert 9 < full["n_iter"] < 100 and full["converged"]
    assert info["n_iter"] == k and info["converged"] == (max_iter == 100)
    assert list(info["branches"]) == list(full["branches"][:k])
    # the traces that the layers recorded (at the cap another kernel sums the last)
    assert np.array_equal(hist["t1"][:k], ref["t1"][:k])
    assert np.array_equal(hist["t2"][:k], ref["t2"][:k])


def test_after_failed_solves_on_other_streams(pk):
    import torch
    H = to_dev(random_orthogonal_hamiltonian(130, 65, seed=3).astype(np.float32))
    ref = pk.density(H, 65)
    bad = H.clone()
    bad[5, 7] = float("nan")
    for k in range(4):
        banner(f"stop word after failures {k}")
        with torch.cuda.stream(torch.cuda.Stream()):
            with pytest.raises(pk.SP2Error):
                pk.density(bad if k % 2 else torch.eye(130, device="cuda"), 65)
        with torch.cuda.stream(torch.cuda.Stream()):
            P = pk.density(H, 65)
            torch.cuda.current_stream().synchronize()
        assert torch.equal(P, ref)


def test_wait_leaves_the_other_threads_alone(pk):
    """While the calling thread waits for the layers of a large solve, the process's
    other threads idle: 2% of a core behind the runtime's event waits, 17% with a
    stream query every 0.15 ms; a tenth separates them.  Other load only adds, so
    the least of three counts."""
    import time

    import torch
    n = 6144
    banner(f"stop word host threads N={n}")
    g = torch.Generator(device="cuda").manual_seed(1)
    a = torch.randn(n, n, generator=g, device="cuda") / n ** 0.5
    H = a + a.T
    ws = pk.allocate_workspace(n)

    def solve():
        pk.density(H, n // 2, workspace=ws, precision="fp16x3", refine="split", max_iter=30,
                   allow_unconverged=True)

    solve()   # what the first call of a process sets up is not counted
    share = []
    for _ in range(3):
        wall, own, all_ = time.perf_counter(), time.thread_time(), time.process_time()
        for _ in range(4):
            solve()
        wall = time.perf_counter() - wall
        share.append((time.process_time() - all_ - (time.thread_time() - own)) / wall)
    print(f"  other threads: {share}", flush=True)
    assert min(share) < 0.1
