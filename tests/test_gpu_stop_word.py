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
