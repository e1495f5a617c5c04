"""The many-row matrix-core kernel (calls of 48 or 80 rows and more) against the fp64 oracle.

Tolerance (fp32 output): products are exact, and a chunk's sum, its product with the row scale and the sum over chunks
round in fp32 n times one after another (n at most a few hundred): for random signs about sqrt(n) * 2^-24 of the result's
norm, 1e-6; the tests allow 2e-6."""
import numpy as np
import pytest

import oracle
from synth import LayerSpec, make_activations, make_layer

from conftest import gpu_available
from gpu_util import log, pack_layer, run_gemm, sample_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not gpu_available():
        pytest.skip("no GPU")
    from paper_2608_15602_amd import fluxbin as fb
    fb.lib()


SMALL = [LayerSpec("pf_mu8", M=333, N=300, Kb=3, Ks=2, mu=8, S=177, g_r=128, g_s=177, seed=111),
         LayerSpec("pf_mu4", M=257, N=1000, Kb=4, Ks=1, mu=4, S=40, g_r=256, g_s=40, seed=112),
         LayerSpec("pf_one", M=1, N=1, Kb=1, Ks=0, mu=8, S=0, g_r=1, g_s=1, seed=113),
         LayerSpec("pf_all_salient", M=130, N=129, Kb=1, Ks=3, mu=8, S=129, g_r=129, g_s=128, seed=114)]
LARGE = LayerSpec("pf_8M", M=4099, N=2050, Kb=2, Ks=1, mu=8, S=90, g_r=128, g_s=90, outlier_frac=0.001, seed=115)
# one row tile, just below and above a workgroup's 64 batch rows, one launch's 512 rows and a few and many more
CASES = [(s, B) for s in SMALL for B in (80, 129)] + [(SMALL[0], B) for B in (512, 513, 600)] + \
        [(LARGE, B) for B in (48, 64, 65, 200)]


@pytest.mark.parametrize("spec,B", CASES, ids=[f"{s.name}-{B}" for s, B in CASES])
def test_many_rows(spec, B):
    """Rows against the oracle (sampled on the large layer), fp16 output with row strides past the row lengths, and
    bitwise repeatable on one workspace."""
    import torch
    from paper_2608_15602_amd import fluxbin as fb
    log(f"case many rows {spec.name} B={B}")
    L = make_layer(spec)
    packed = pack_layer(L)
    info = fb.fluxbin_plan_query(packed, B)
    assert (info["kernel_name"], info["batch_tile_rows"], info["batch_tiles"]) == ("mfma", 512, -(-B // 512)), info
    x = make_activations(L, B)
    rows = np.arange(spec.M) if spec.M < 1000 else sample_rows(spec.M, 64, seed=B)
    y_ref = oracle.gemv_dense(L, x, rows=rows)
    ws = fb.make_workspace(packed, B)
    y = run_gemm(packed, x, out_fp32=True, ws=ws)
    err = np.linalg.norm(y[:, rows] - y_ref) / np.linalg.norm(y_ref)
    worst = (np.linalg.norm(y[:, rows] - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)).max()
    log(f"  rel={err:.2e}, worst batch row {worst:.2e}")
    assert err < 2e-6 and worst < 4e-6
    assert np.array_equal(run_gemm(packed, x, out_fp32=True, ws=ws), y), "repeat differs"
    xs = torch.zeros((B, spec.N + 3), dtype=torch.float16, device="cuda")
    xs[:, :spec.N] = torch.from_numpy(x.view(np.float16)).cuda()
    ys = torch.zeros((B, spec.M + 5), dtype=torch.float16, device="cuda")
    fb.fluxbin_lut_gemm_smallbatch(packed, xs[:, :spec.N], y=ys[:, :spec.M], workspace=ws)
    torch.cuda.synchronize()
    got = ys.cpu().numpy()
    assert np.array_equal(got[:, :spec.M], y.astype(np.float32).astype(np.float16))
    assert not got[:, spec.M:].any()


def test_many_rows_infinities_and_subnormals():
    """A batch row with an infinity or NaN leaves the others as they are; subnormal activations and column scales are
    honoured."""
    spec, B = SMALL[0], 80
    log("case many rows, special values")
    L = make_layer(spec)
    x = make_activations(L, B)
    packed = pack_layer(L)
    clean = run_gemm(packed, x, out_fp32=True)
    xb = x.copy().view(np.float16)
    xb[3, 17], xb[70, 255] = np.inf, np.nan
    y = run_gemm(packed, xb.view(np.uint16), out_fp32=True)
    assert not np.isfinite(y[3]).any() and np.isnan(y[70]).all()
    keep = [b for b in range(B) if b not in (3, 70)]
    assert np.array_equal(y[keep], clean[keep])
    rng = np.random.default_rng(116)
    sub = lambda shape: rng.integers(1, 1024, size=shape).astype(np.uint16)
    xs = sub(x.shape)
    y, y_ref = run_gemm(packed, xs, out_fp32=True), oracle.gemv_dense(L, xs)
    assert np.linalg.norm(y - y_ref) < 2e-6 * np.linalg.norm(y_ref) and np.abs(y_ref).max() > 0
    L.alpha_c[:] = sub(L.alpha_c.shape)
    L.alpha_sc[:] = sub(L.alpha_sc.shape)
    y, y_ref = run_gemm(pack_layer(L), x, out_fp32=True), oracle.gemv_dense(L, x)
    assert np.linalg.norm(y - y_ref) < 2e-6 * np.linalg.norm(y_ref) and np.abs(y_ref).max() > 0


# the last rows of a call: fewer than a many-row call of their own has on the small layer (40, 79) and on the large one
# (47), enough for one (88), and both below and above one small launch's rows (1, 31)
@pytest.mark.parametrize("spec,B", [(SMALL[0], 513), (SMALL[0], 543), (SMALL[0], 552), (SMALL[0], 591), (SMALL[0], 600),
                                    (LARGE, 559)], ids=lambda v: getattr(v, "name", str(v)))
def test_tiles_equal_calls_of_their_rows(spec, B):
    """Every batch tile's rows, the last ones included, are bit for bit those of a call on these rows alone."""
    import torch
    log(f"case tiles {spec.name} B={B}")
    L = make_layer(spec)
    packed = pack_layer(L)
    x = make_activations(L, B)
    y = run_gemm(packed, x, out_fp32=True)
    for b0 in range(0, B, 512):
        assert np.array_equal(y[b0:b0 + 512], run_gemm(packed, x[b0:b0 + 512], out_fp32=True)), b0
    torch.cuda.synchronize()


def test_parts_are_worth_their_sums():
    """A layer of many rows and few columns at 512 batch rows: one workgroup per tile, because the sums of several (117 MB
    each) would take longer to write and add than the product. Sampled rows against the oracle."""
    from paper_2608_15602_amd import fluxbin as fb
    spec, B = LayerSpec("pf_tall", M=57344, N=512, Kb=2, Ks=0, mu=4, S=0, g_r=128, g_s=1, seed=117), 512
    log("case many rows, tall layer")
    L = make_layer(spec)
    packed = pack_layer(L)
    info = fb.fluxbin_plan_query(packed, B)
    assert info["workgroups"] == 224 * 8 and info["workspace_bytes"] < 4 * spec.M * B, info
    x = make_activations(L, B)
    rows = sample_rows(spec.M, 32, seed=B)
    y_ref = oracle.gemv_dense(L, x, rows=rows)
    assert np.linalg.norm(run_gemm(packed, x, out_fp32=True)[:, rows] - y_ref) < 2e-6 * np.linalg.norm(y_ref)


@pytest.mark.parametrize("spec", [LayerSpec("pf_long", M=16640, N=8192, Kb=2, Ks=1, mu=8, S=200, g_r=128, g_s=200,
                                            outlier_frac=0.001, seed=118),
                                  LayerSpec("pf_odd_run", M=20001, N=3000, Kb=3, Ks=2, mu=4, S=140, g_r=128, g_s=140,
                                            outlier_frac=0.001, seed=119)], ids=lambda s: s.name)
def test_no_further_off_than_32_row_launches(spec):
    """Sums of a hundred chunks and more per part: over sampled rows no further from the oracle than the 32-row launches of
    the small-batch kernel on the same rows (3% for the spread of the two errors over the sample)."""
    from paper_2608_15602_amd import fluxbin as fb
    log(f"case error {spec.name}")
    L, B = make_layer(spec), 256
    packed = pack_layer(L)
    x = make_activations(L, B)
    rows = sample_rows(spec.M, 400, seed=3)
    y_ref = oracle.gemv_dense(L, x, rows=rows)
    y = run_gemm(packed, x, out_fp32=True)[:, rows]
    with fb.tuning(mfma=1):
        assert fb.fluxbin_plan_query(packed, B)["batch_tile_rows"] == 32
        y32 = run_gemm(packed, x, out_fp32=True)[:, rows]
    err, err32 = np.linalg.norm(y - y_ref), np.linalg.norm(y32 - y_ref)
    log(f"  {err / np.linalg.norm(y_ref):.2e}, 32-row launches {err32 / np.linalg.norm(y_ref):.2e}")
    assert err < 1.03 * err32
