"""The block-scaled matrix-core kernel (B = 2..16) against the fp64 oracle.

Tolerance (fp32 output). Each activation product is off by up to 2^-29 of its 32-column block's largest with six digits, by
up to 2^-24 with the five of 9 to 16 rows on layers with one row scale per chunk: for random signs, if one column of every
block held all of its norm, sqrt(31) * 2^-24 = 3.3e-7 of the result's norm at most. Everything else is fp32: a chunk's sum,
its product with the row scale and the sum over chunks, n roundings of 2^-24 of the running value one after another, for
random signs about sqrt(n) * 2^-24 of the result's norm with n the chunks (at most a few hundred here), 1e-6. The tests
allow 2e-6."""
import numpy as np
import pytest

import oracle
from synth import LayerSpec, make_activations, make_layer, paper_config

from conftest import gpu_available
from gpu_util import log, pack_layer, run_gemm, sample_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not gpu_available():
        pytest.skip("no GPU")
    from paper_2608_15602_amd import fluxbin as fb
    fb.lib()


# coarse layers just past the size from which the plan takes the kernel: ragged rows and columns, several workgroups per
# row tile; one base and more row tiles than CUs (up to 4 rows); every salient chunk partly filled
COARSE = [LayerSpec("mx_mu4", M=4177, N=17000, Kb=2, Ks=1, mu=4, S=700, g_r=128, g_s=700, outlier_frac=0.001, seed=91),
          LayerSpec("mx_tall_mu4", M=32801, N=4400, Kb=1, Ks=0, mu=4, S=0, g_r=4400, g_s=1, seed=92)]
COARSE8 = LayerSpec("mx_mu8", M=5001, N=14001, Kb=2, Ks=1, mu=8, S=301, g_r=256, g_s=301, outlier_frac=0.001, seed=93)
FINE = [paper_config("mx_s8", 333, 1152, 3, 8, 128, seed=94), paper_config("mx_s16", 65, 640, 1, 16, 128, seed=95),
        paper_config("mx_s16_wide", 1000, 4096, 2, 16, 128, seed=96)]
FINE_SMALL_BATCH = [paper_config("mx_s8_8M", 2050, 4224, 2, 8, 128, seed=97),
                    paper_config("mx_s16_8M", 4100, 2176, 1, 16, 128, seed=98)]
CASES = ([(COARSE[0], B) for B in (2, 3, 8, 9, 16)] + [(COARSE[1], B) for B in (2, 3, 4)] +
         [(COARSE8, B) for B in (5, 8, 9, 16)] +
         [(s, B) for s in FINE for B in (9, 16)] + [(s, B) for s in FINE_SMALL_BATCH for B in (3, 4, 7)])


@pytest.mark.parametrize("spec,B", CASES, ids=[f"{s.name}-{B}" for s, B in CASES])
def test_block_scaled_kernel(spec, B):
    """Rows against the oracle (sampled on the large layers, the last ones included), fp16 output and strides past the
    row lengths, bitwise repeatable on one workspace, and y(2x) == 2 y(x) bit for bit (block scales move with x)."""
    import torch
    from paper_2608_15602_amd import fluxbin as fb
    log(f"case block-scaled {spec.name} M={spec.M} N={spec.N} mu={spec.mu} B={B}")
    L = make_layer(spec)
    packed = pack_layer(L)
    info = fb.fluxbin_plan_query(packed, B)
    assert info["kernel_name"] == "mfma" and info["rows_per_tile"] in (64, 128), info
    assert (info["batch_tile_rows"] >= B, info["batch_tiles"]) == (True, 1), info
    x = make_activations(L, B)
    rows = np.arange(spec.M) if spec.M * spec.N < 5e6 else sample_rows(spec.M, 128, seed=B)
    y_ref = oracle.gemv_dense(L, x, rows=rows)
    ws = fb.make_workspace(packed, B)
    y = run_gemm(packed, x, out_fp32=True, ws=ws)
    err = np.linalg.norm(y[:, rows] - y_ref) / np.linalg.norm(y_ref)
    log(f"  rel={err:.2e}")
    assert err < 2e-6
    assert np.array_equal(run_gemm(packed, x, out_fp32=True, ws=ws), y), "repeat differs"
    x2 = (oracle.f16_to_f64(x) * 2).astype(np.float16).view(np.uint16)
    assert np.array_equal(run_gemm(packed, x2, out_fp32=True, ws=ws), 2 * y)
    xs = torch.zeros((B, spec.N + 5), dtype=torch.float16, device="cuda")
    xs[:, :spec.N] = torch.from_numpy(x.view(np.float16)).cuda()
    ys = torch.zeros((B, spec.M + 3), dtype=torch.float16, device="cuda")
    fb.fluxbin_lut_gemm_smallbatch(packed, xs[:, :spec.N], y=ys[:, :spec.M], workspace=ws)
    torch.cuda.synchronize()
    got = ys.cpu().numpy()
    assert np.array_equal(got[:, :spec.M], y.astype(np.float32).astype(np.float16))
    assert not got[:, spec.M:].any()


# tall layers with few columns: a workgroup's eight wavefronts share fewer than two chunks each
FEW_COARSE = [LayerSpec("mx_few_4", M=205001, N=250, Kb=2, Ks=0, mu=8, S=0, g_r=128, g_s=1, seed=120),
              LayerSpec("mx_few_12", M=76001, N=700, Kb=2, Ks=0, mu=4, S=0, g_r=128, g_s=1, seed=121)]
FEW_FINE = [paper_config("mx_few_s8", 66000, 512, 2, 8, 128, seed=122),
            paper_config("mx_few_s16", 132000, 256, 1, 16, 128, seed=123),
            paper_config("mx_few_s8_small", 2000, 256, 1, 8, 128, seed=124)]
# layers of enough chunks, where it is 1.3 to 1.4 times as fast as batch-1 launches at two rows
MANY_FINE = [paper_config("mx_many_s8", 14770, 1792, 4, 8, 128, seed=125),
             paper_config("mx_many_s8_wide", 2208, 12160, 4, 8, 128, seed=126)]


@pytest.mark.parametrize("spec,B,rows", [(FEW_COARSE[0], 3, 256), (FEW_COARSE[0], 8, 256), (FEW_COARSE[1], 5, 256),
                                         (FEW_COARSE[1], 2, 128), (FEW_FINE[0], 2, 1), (FEW_FINE[0], 3, 1),
                                         (FEW_FINE[1], 3, 1), (FEW_FINE[0], 8, 64), (FEW_FINE[1], 9, 64),
                                         (FEW_FINE[2], 9, 0), (FEW_FINE[2], 21, 0), (MANY_FINE[0], 2, 64),
                                         (MANY_FINE[1], 2, 64), (MANY_FINE[1], 3, 64)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_tall_layers_with_few_chunks(spec, B, rows):
    """Where most of a workgroup's wavefronts would have no chunk, the kernel is slower than those it takes over from: the
    fp16 form (256-row tiles), or on layers with fine salient groups one batch-1 launch per row (rows = 1) or the generic
    kernel (rows = 0); where they have enough, it is chosen. Sampled rows against the oracle."""
    from paper_2608_15602_amd import fluxbin as fb
    log(f"case few chunks {spec.name} B={B}")
    L = make_layer(spec)
    packed = pack_layer(L)
    info = fb.fluxbin_plan_query(packed, B)
    if rows == 0:
        assert info["kernel_name"] == "generic", info
    else:
        assert (info["batch_tile_rows"] if rows == 1 else info["rows_per_tile"]) == rows, info
    x = make_activations(L, B)
    keep = sample_rows(spec.M, 64, seed=B)
    y_ref = oracle.gemv_dense(L, x, rows=keep)
    y = run_gemm(packed, x, out_fp32=True)[:, keep]
    assert np.linalg.norm(y - y_ref) < 2e-6 * np.linalg.norm(y_ref)


def _nonfinite_reference(L, x):
    """The non-finite outputs of activations x [N] (fp16): every base adds r * (+-c * x_j) of each infinite x_j, so a row is
    +-inf where all of them agree, else NaN; NaN activations and zero row scales give NaN. 0 where y is finite."""
    s = L.spec
    M = s.M
    pos, neg, nan = np.zeros(M, bool), np.zeros(M, bool), np.zeros(M, bool)
    bad = np.flatnonzero(~np.isfinite(x))
    bases = [(L.signs, L.alpha_r, k, s.g_r, {int(j): int(j) for j in bad}) for k in range(s.Kb)]
    where = {int(j): t for t, j in enumerate(L.sal_idx)}
    bases += [(L.sal_signs, L.alpha_sr, k, s.g_s, {int(j): where[int(j)] for j in bad if int(j) in where})
              for k in range(s.Ks)]
    for signs, scale, k, g, cols in bases:
        for j, place in cols.items():
            r = oracle.f16_to_f64(scale[k][:, place // g])
            plus = ((signs[k][:, j // 32] >> (j % 32)) & 1).astype(bool)
            with np.errstate(invalid="ignore"):
                v = r * np.where(plus, 1.0, -1.0) * float(x[j])
            pos |= v == np.inf
            neg |= v == -np.inf
            nan |= np.isnan(v)
    out = np.zeros(M)
    out[pos] = np.inf
    out[neg] = -np.inf
    out[(pos & neg) | nan] = np.nan
    return out


@pytest.mark.parametrize("spec,B", [(COARSE8, 6), (FINE[0], 9), (FINE[2], 16)], ids=lambda v: getattr(v, "name", str(v)))
def test_infinities_and_nan(spec, B):
    """Infinities and NaN among the activations (global and salient columns; alone, and with opposite signs in one row)
    give the infinities and NaN of the sum; the batch rows without them keep their values."""
    log(f"case non-finite {spec.name} B={B}")
    L = make_layer(spec)
    packed = pack_layer(L)
    x = make_activations(L, B)
    clean = run_gemm(packed, x, out_fp32=True)
    xb = x.copy().view(np.float16)
    xb[1, int(L.sal_idx[3])] = np.inf
    xb[2, [5, spec.N - 1]] = [np.inf, -np.inf]
    xb[B - 1, 130] = np.nan
    y = run_gemm(packed, xb.view(np.uint16), out_fp32=True)
    for b in (1, 2, B - 1):
        assert np.array_equal(np.where(np.isfinite(y[b]), 0, y[b]), _nonfinite_reference(L, xb[b]), equal_nan=True), b
    assert np.isinf(y[1]).any() and np.isnan(y[B - 1]).all()
    for b in set(range(B)) - {1, 2, B - 1}:
        assert np.array_equal(y[b], clean[b]), b


@pytest.mark.parametrize("which", ["colscale", "x", "spread"])
def test_block_scaled_subnormals_and_range(which):
    """Subnormal column scales or activations, and activations spread over the whole fp16 range (each 32-column block
    has its own scale), against the oracle: within 2e-6 of each row's norm of |scale| |product| sums."""
    spec = FINE[2]
    B = 11
    log(f"case block-scaled {which}")
    L = make_layer(spec)
    rng = np.random.default_rng(5)
    x = make_activations(L, B)
    sub = lambda shape: rng.integers(1, 1024, size=shape).astype(np.uint16)
    if which == "colscale":
        L.alpha_c[:] = sub(L.alpha_c.shape)
        L.alpha_sc[:] = sub(L.alpha_sc.shape)
    elif which == "x":
        x = sub(x.shape) | (rng.integers(0, 2, size=x.shape).astype(np.uint16) << 15)
    else:
        x = (rng.normal(size=x.shape) * 2.0 ** rng.uniform(-20, 14, size=x.shape)).astype(np.float16).view(np.uint16)
    y = run_gemm(pack_layer(L), x, out_fp32=True)
    y_ref = oracle.gemv_dense(L, x)
    assert np.abs(y_ref).max() > 0
    for b in range(B):
        assert np.linalg.norm(y[b] - y_ref[b]) < 2e-6 * np.linalg.norm(y_ref[b]), b


@pytest.mark.parametrize("which", ["colscale", "x", "spread", "spike", "few"])
def test_five_digit_range(which):
    """Five digits (9 to 16 rows, one row scale per chunk) on subnormal scales and activations, activations over the whole
    fp16 range, one column in 32 or a few columns thousands of times larger than the others: every batch row within 2e-6 of
    the oracle, and no further off than the fp16 form, whose products are exact (1.05: the two forms' fp32 sums differ)."""
    from paper_2608_15602_amd import fluxbin as fb
    spec, B = COARSE8, 11
    log(f"case five digits {which}")
    L = make_layer(spec)
    rng = np.random.default_rng(6)
    x = make_activations(L, B)
    sub = lambda shape: rng.integers(1, 1024, size=shape).astype(np.uint16)
    half = lambda v: v.astype(np.float16).view(np.uint16)
    if which == "colscale":
        L.alpha_c[:] = sub(L.alpha_c.shape)
        L.alpha_sc[:] = sub(L.alpha_sc.shape)
    elif which == "x":
        x = sub(x.shape) | (rng.integers(0, 2, size=x.shape).astype(np.uint16) << 15)
    elif which == "spread":
        x = half(rng.normal(size=x.shape) * 2.0 ** rng.uniform(-20, 14, size=x.shape))
    else:
        large = np.arange(spec.N) % 32 == 5 if which == "spike" else rng.random(spec.N) < 0.002
        x = half(rng.normal(size=x.shape) * np.where(large, 4096.0, 1.0))
    packed = pack_layer(L)
    assert fb.fluxbin_plan_query(packed, B)["rows_per_tile"] == 128
    rows = sample_rows(spec.M, 512, seed=7)
    y_ref = oracle.gemv_dense(L, x, rows=rows)
    y = run_gemm(packed, x, out_fp32=True)[:, rows]
    with fb.tuning(mfma=1):
        assert fb.fluxbin_plan_query(packed, B)["rows_per_tile"] == 256
        y16 = run_gemm(packed, x, out_fp32=True)[:, rows]
    norm = np.linalg.norm(y_ref, axis=1)
    err, err16 = np.linalg.norm(y - y_ref, axis=1) / norm, np.linalg.norm(y16 - y_ref, axis=1) / norm
    log(f"  five digits {err.mean():.2e} (worst row {err.max():.2e}), fp16 form {err16.mean():.2e}")
    assert err.max() < 2e-6 and err.mean() < 1.05 * err16.mean()


@pytest.mark.parametrize("spec,B", [(FINE_SMALL_BATCH[0], 3), (FINE_SMALL_BATCH[0], 4), (FINE_SMALL_BATCH[1], 4),
                                    (FINE_SMALL_BATCH[0], 8)], ids=lambda v: getattr(v, "name", str(v)))
def test_no_further_off_than_batch_1(spec, B):
    """On layers with fine salient groups the kernel stands in for batch-1 launches: over rows and batch rows it is no
    further from the oracle than they are."""
    from paper_2608_15602_amd import fluxbin as fb
    log(f"case error {spec.name} B={B}")
    L = make_layer(spec)
    packed = pack_layer(L)
    assert fb.fluxbin_plan_query(packed, B)["rows_per_tile"] == 64
    x = make_activations(L, B)
    y_ref = oracle.gemv_dense(L, x)
    y = run_gemm(packed, x, out_fp32=True)
    y1 = np.concatenate([run_gemm(packed, x[b:b + 1], out_fp32=True) for b in range(B)])
    err, err1 = np.linalg.norm(y - y_ref), np.linalg.norm(y1 - y_ref)
    log(f"  {err / np.linalg.norm(y_ref):.2e}, batch-1 launches {err1 / np.linalg.norm(y_ref):.2e}")
    assert err < err1
