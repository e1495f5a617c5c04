"""One workspace for calls of different batch sizes: of the size queried for the largest, it serves every smaller one; one of
the size that a kernel without digit or activation images needs still serves calls that would prefer such a kernel."""
import numpy as np
import pytest

import oracle
from synth import LayerSpec, make_activations, make_layer, paper_config

from conftest import gpu_available
from gpu_util import log, pack_layer, run_gemm, sample_rows

pytestmark = pytest.mark.gpu

LAYERS = [LayerSpec("ws_coarse", M=5001, N=14001, Kb=2, Ks=1, mu=8, S=301, g_r=256, g_s=301, outlier_frac=0.001, seed=111),
          LayerSpec("ws_mu4", M=4177, N=17000, Kb=2, Ks=1, mu=4, S=700, g_r=128, g_s=700, outlier_frac=0.001, seed=112),
          paper_config("ws_s16", 2050, 4224, 2, 16, 128, seed=113)]
BATCHES = list(range(1, 34)) + [48, 100]


@pytest.mark.parametrize("spec", LAYERS, ids=[s.name for s in LAYERS])
def test_shared_workspace(spec):
    """Query sizes do not fall as B grows to one launch's 16 rows; calls on the workspace of 16 and of 32 rows, at every
    kernel's batch sizes, against the oracle (2e-6: the random-walk bound of a few hundred fp32 roundings); a workspace
    smaller than a batch-1 call's is refused."""
    import torch
    from paper_2608_15602_amd import fluxbin as fb
    if not gpu_available():
        pytest.skip("no GPU")
    L = make_layer(spec)
    packed = pack_layer(L)
    need = {B: fb.fluxbin_workspace_query(packed, B) for B in BATCHES}
    assert all(need[a] <= need[b] for a, b in zip(range(1, 16), range(2, 17))), need
    rows = sample_rows(spec.M, 64, seed=1)
    for owner, batches in ((16, (1, 2, 3, 5, 8, 9, 16)), (32, (1, 4, 17, 32, 48, 100))):
        ws = fb.make_workspace(packed, owner)
        for B in batches:
            log(f"case workspace {spec.name} of B={owner} at B={B}: needs {need.get(B)}")
            x = make_activations(L, B)
            assert B > owner or ws.numel() * ws.element_size() >= need[B]
            y = run_gemm(packed, x, out_fp32=True, ws=ws)
            y_ref = oracle.gemv_dense(L, x, rows=rows)
            y = np.atleast_2d(y)[:, rows]
            assert np.linalg.norm(y - np.atleast_2d(y_ref)) / np.linalg.norm(y_ref) < 2e-6
    small = torch.zeros(need[1] - 256 if need[1] > 256 else 0, dtype=torch.uint8, device="cuda")
    with pytest.raises(fb.FluxbinError):
        run_gemm(packed, make_activations(L, 16), out_fp32=True, ws=small)
