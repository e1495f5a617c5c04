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


# layers whose many-row and block-scaled plans want more for some batches than for larger ones
GROWING = [LayerSpec("ws_tall", M=28672, N=2048, Kb=2, Ks=1, mu=8, S=60, g_r=128, g_s=60, seed=114),
           LayerSpec("ws_wide", M=1024, N=8192, Kb=2, Ks=0, mu=8, S=0, g_r=128, g_s=1, seed=115),
           LayerSpec("ws_square", M=4096, N=4096, Kb=1, Ks=0, mu=4, S=0, g_r=128, g_s=1, seed=116), LAYERS[2]]


@pytest.mark.parametrize("spec", GROWING, ids=[s.name for s in GROWING])
def test_largest_batch_serves_the_smaller_ones(spec):
    """The queried size does not fall as B grows, and on the workspace of a large batch every smaller one gets the launches
    of its own workspace: the same y bit for bit."""
    from paper_2608_15602_amd import fluxbin as fb
    if not gpu_available():
        pytest.skip("no GPU")
    log(f"case workspace sizes {spec.name}")
    L = make_layer(spec)
    packed = pack_layer(L)
    need = [fb.fluxbin_workspace_query(packed, B) for B in range(1, 1100)]
    assert all(a <= b for a, b in zip(need, need[1:])), [(B + 1, need[B:B + 2]) for B in range(1098) if need[B] > need[B + 1]]
    ws = fb.make_workspace(packed, 600)
    x = make_activations(L, 600)
    for B in (2, 5, 16, 40, 64, 100, 130, 200, 257, 320, 448, 552):
        log(f"  B={B}")
        assert np.array_equal(run_gemm(packed, x[:B], out_fp32=True, ws=ws), run_gemm(packed, x[:B], out_fp32=True)), B


def test_smaller_workspace_takes_the_other_launches():
    """A call of 192 rows whose many-row launch wants more than the workspace of 32 rows holds runs as 32-row launches on
    that one: the rows of each as a call of their own gives them."""
    from paper_2608_15602_amd import fluxbin as fb
    if not gpu_available():
        pytest.skip("no GPU")
    log("case workspace too small for the preferred launch")
    spec, B = LayerSpec("ws_sums", M=28672, N=8192, Kb=1, Ks=0, mu=8, S=0, g_r=128, g_s=1, seed=117), 192
    L = make_layer(spec)
    packed = pack_layer(L)
    info = fb.fluxbin_plan_query(packed, B)
    assert info["batch_tile_rows"] == 512 and info["workspace_bytes"] > fb.fluxbin_workspace_query(packed, 32), info
    ws = fb.make_workspace(packed, 32)
    x = make_activations(L, B)
    y = run_gemm(packed, x, out_fp32=True, ws=ws)
    for b in range(0, B, 32):
        assert np.array_equal(y[b:b + 32], run_gemm(packed, x[b:b + 32], out_fp32=True, ws=ws)), b
    own = run_gemm(packed, x, out_fp32=True)
    assert not np.array_equal(y, own) and np.linalg.norm(y - own) < 2e-6 * np.linalg.norm(own)
