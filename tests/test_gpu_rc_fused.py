"""The decomposition's fused passes (blocks of at most 128 columns) at the edges of their shapes against the fp64 oracle:
signs and masks bit-exact, scales within 1e-9 relative or 1e-10 of the largest scale (fp64 sums in another order, magnified
where a later base's quotient divides a residual that cancels), as in the other decomposition tests."""
import numpy as np
import pytest

from oracle import rc_oracle as rc
from synth import make_weight_matrix

from conftest import gpu_available
from gpu_util import log
from test_gpu_rc import _bits, _close, _gpu_rc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not gpu_available():
        pytest.skip("no GPU")
    from paper_2608_15602_amd import fluxbin as fb
    fb.lib()


def _compare(out, ref, what):
    signs, ar, ac = out
    assert np.array_equal(signs.cpu().numpy().view(np.uint32), _bits(ref["B"])), what
    _close(ar.cpu().numpy(), ref["alpha_r"], f"{what} alpha_r")
    _close(ac.cpu().numpy(), ref["alpha_c"], f"{what} alpha_c")


@pytest.mark.parametrize("M,N,K,g,T", [(257, 300, 2, 128, 3), (600, 129, 4, 128, 2), (301, 520, 1, 96, 3),
                                       (97, 77, 3, 40, 0), (2100, 128, 2, 128, 1), (260, 640, 2, 65, 2)])
def test_all_columns(M, N, K, g, T):
    """Ragged last blocks and rows, row slices of one and several workgroups, blocks of up to 64 and up to 128 columns
    whose boundaries fall inside sign words, one to four bases, no rounds."""
    log(f"case fused rc M={M} N={N} K={K} g={g} T={T}")
    W, _ = make_weight_matrix(M, N, seed=70 + M)
    ref = rc.rc_decomp(W.astype(np.float64), np.ones(N, bool), K=K, T=T, g=g)
    _compare(_gpu_rc(W, K, T, g), ref, "global")


@pytest.mark.parametrize("counts", [(8, 3, 0), (16, 9, 1), (30, 17, 32), (64, 33, 5), (100, 128, 65)])
def test_masked_columns(counts):
    """Masks that list few, many, all or no columns of a block (8 to 64 lanes per row, two columns per lane; copied and
    recomputed x), on the residual of an earlier decomposition and on the matrix itself."""
    import torch
    M, g, K = 261, 128, 2
    N = g * len(counts)
    log(f"case fused rc mask {counts}")
    W, _ = make_weight_matrix(M, N, seed=80 + counts[0])
    rng = np.random.default_rng(81)
    mask = np.zeros(N, bool)
    for b, n in enumerate(counts):
        mask[b * g + rng.choice(g, size=n, replace=False)] = True
    Wd = W.astype(np.float64)
    _compare(_gpu_rc(W, K, 2, g, mask=mask), rc.rc_decomp(Wd, mask, K=K, T=2, g=g), "masked")
    glob = _gpu_rc(W, 2, 2, g)
    ref = rc.rc_decomp(Wd, np.ones(N, bool), K=2, T=2, g=g)
    R = Wd - rc.reconstruct(ref["B"], ref["alpha_r"], ref["alpha_c"], g)
    _compare(_gpu_rc(W, 1, 2, g, mask=mask, prior=glob + (g,)), rc.rc_decomp(R, mask, K=1, T=2, g=g), "masked residual")
    torch.cuda.synchronize()


def test_residual_of_all_columns():
    """Prior bases without a mask, their row-scale groups other than this decomposition's blocks."""
    M, N = 270, 200
    log("case fused rc residual, no mask")
    W, _ = make_weight_matrix(M, N, seed=90)
    prior = _gpu_rc(W, 2, 2, 50)
    ref0 = rc.rc_decomp(W.astype(np.float64), np.ones(N, bool), K=2, T=2, g=50)
    R = W.astype(np.float64) - rc.reconstruct(ref0["B"], ref0["alpha_r"], ref0["alpha_c"], 50)
    _compare(_gpu_rc(W, 2, 2, 128, prior=prior + (50,)), rc.rc_decomp(R, np.ones(N, bool), K=2, T=2, g=128), "residual")


@pytest.mark.parametrize("M", [1, 70, 257, 700])
def test_structural_search_wide(M):
    """As many columns as fill the CUs with 64-column workgroups (few and many rows), and a column fewer than that."""
    import torch
    from paper_2608_15602_amd import fluxbin as fb
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for N in (64 * cus - 1, 64 * cus, 64 * cus + 70):
        log(f"case saliency {M}x{N}")
        rng = np.random.default_rng(91)
        W, hinv = rng.normal(size=(M, N)).astype(np.float32), rng.uniform(0.5, 2.0, size=N)
        scores, idx, mask = fb.fluxbin_structural_search(torch.from_numpy(W).cuda(), torch.from_numpy(hinv).cuda(), 128, 8)
        torch.cuda.synchronize()
        want = rc.structural_search(W.astype(np.float64), hinv, 128, 8)
        assert np.array_equal(idx.cpu().numpy().astype(np.int64), want)
        assert np.array_equal(np.flatnonzero(mask.cpu().numpy()), want)
        _close(scores.cpu().numpy(), rc.saliency(W.astype(np.float64), hinv), "saliency", rtol=1e-12)


@pytest.mark.parametrize("M,N,K,g,T,masked", [(700, 500, 3, 192, 2, False), (620, 520, 4, 256, 1, True),
                                              (1300, 300, 2, 300, 2, True), (600, 260, 2, 129, 2, False),
                                              (600, 260, 2, 128, 2, False), (530, 390, 4, 130, 0, True)])
def test_general_kernels(M, N, K, g, T, masked):
    """Blocks of more than 128 columns (and, beside them, of 128): several row slices, three and four bases, masks."""
    log(f"case general rc M={M} N={N} K={K} g={g} T={T} mask={masked}")
    W, _ = make_weight_matrix(M, N, seed=100 + g)
    mask = np.ones(N, bool)
    if masked:
        mask[:] = np.random.default_rng(101).random(N) < 0.3
    ref = rc.rc_decomp(W.astype(np.float64), mask, K=K, T=T, g=g)
    _compare(_gpu_rc(W, K, T, g, mask=mask if masked else None), ref, "general")


def test_general_kernels_residual_and_zero_eps():
    """Prior bases (with and without a mask) in blocks of more than 128 columns, and eps = 0."""
    import torch
    from paper_2608_15602_amd import fluxbin as fb
    M, N, g = 600, 500, 250
    log("case general rc residual")
    W, _ = make_weight_matrix(M, N, seed=102)
    Wd, every = W.astype(np.float64), np.ones(N, bool)
    prior = _gpu_rc(W, 2, 2, 100)
    ref0 = rc.rc_decomp(Wd, every, K=2, T=2, g=100)
    R = Wd - rc.reconstruct(ref0["B"], ref0["alpha_r"], ref0["alpha_c"], 100)
    mask = np.random.default_rng(103).random(N) < 0.2
    _compare(_gpu_rc(W, 2, 2, g, prior=prior + (100,)), rc.rc_decomp(R, every, K=2, T=2, g=g), "residual")
    _compare(_gpu_rc(W, 3, 1, g, mask=mask, prior=prior + (100,)), rc.rc_decomp(R, mask, K=3, T=1, g=g), "masked residual")
    for block in (128, g):
        out = fb.fluxbin_rc_decompose(torch.from_numpy(W).cuda(), 2, 2, block, eps=0.0)
        torch.cuda.synchronize()
        _compare(out, rc.rc_decomp(Wd, every, K=2, T=2, g=block, eps=0.0), f"eps 0, g {block}")
