"""Solves whose H fits one workgroup (d <= 256): whole blocks of iterations run
in one launch, against the oracle at the edges of the 16-column groups, of the
padded widths, of the 64-iteration coefficient tables and of the blocks."""
import numpy as np
import pytest

import oracle
from gpu_util import gpu_solve, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2512_13886_amd as lib
    return lib


def _problem(d, n, seed):
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((2 * d + 16, d)) * np.exp(rng.normal(0.0, 0.5, d))
    H = A.T @ A
    H = (H + 0.01 * np.trace(H) / d * np.eye(d)).astype(np.float32)
    W0 = (0.02 * rng.standard_normal((n, d))).astype(np.float32)
    M = (rng.random((n, d)) < 0.5).astype(np.uint8)
    M[0] = 1   # no compressed form, whatever the other rows keep
    M[-1] = 0 if n > 1 else M[-1]
    lam = np.float32(np.linalg.eigvalsh(H.astype(np.float64))[-1])
    return H, W0, M, lam


# Before the first check both sides follow the same continuous map: rounding
# separates them by 2^-24 (fp32) or up to 3 * 2^-16 (bf16x3) per product.
@pytest.mark.parametrize("prec, bound", [(0, 1e-5), (1, 1e-4)])
@pytest.mark.parametrize("d, n", [(4, 1), (100, 15), (128, 16), (129, 17), (255, 40), (256, 9)])
@pytest.mark.parametrize("iters", [1, 64, 150])
def test_one_block_matches_the_oracle(L, prec, bound, d, n, iters):
    H, W0, M, lam = _problem(d, n, d + n)
    ref = oracle.rapdhg(H.astype(np.float64), W0, M, float(lam),
                        oracle.SolverOptions(max_iters=iters, fixed_iters=True, check_every=iters))
    W, st, info = gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0, M,
                            L.SolverOpts.default(max_iters=iters, fixed_iters=1,
                                                 check_every=iters, precision=prec))
    W = W.cpu().numpy()
    assert info["sparse_products"] == 0 and info["iterations"] == iters
    assert np.all(W[M == 0].view(np.uint32) == 0)
    norm = np.maximum(np.linalg.norm(ref.W, axis=1), 1e-30)
    assert np.max(np.linalg.norm(W - ref.W, axis=1) / norm) <= bound
    np.testing.assert_array_equal(st["iters"], iters)


# Batches whose sums have fewer ranges than 32-wide steps of the contraction (3 of
# 4, 5 of 8 and 2 of 8); columns are independent, so the oracle runs on a sample.
@pytest.mark.parametrize("prec, bound", [(0, 1e-5), (1, 1e-4)])
@pytest.mark.parametrize("d, n", [(128, 16500), (200, 9000), (256, 40000)])
def test_large_batches_match_the_oracle(L, prec, bound, d, n):
    H, W0, M, lam = _problem(d, n, d + n)
    W, _, _ = gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0, M,
                        L.SolverOpts.default(max_iters=40, fixed_iters=1, precision=prec))
    W = W.cpu().numpy()
    assert np.all(W[M == 0].view(np.uint32) == 0)
    cols = np.concatenate([np.arange(1, 20), np.arange(n - 20, n - 1)])
    ref = oracle.rapdhg(H.astype(np.float64), W0[cols], M[cols], float(lam),
                        oracle.SolverOptions(max_iters=40, fixed_iters=True))
    err = np.linalg.norm(W[cols] - ref.W, axis=1) / np.linalg.norm(ref.W, axis=1)
    assert err.max() <= bound


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("d, n", [(128, 33), (250, 33)])
def test_restarted_blocks_reach_the_optimum(L, prec, d, n):
    H, W0, M, lam = _problem(d, n, 7 * d)
    ref = oracle.closed_form(H.astype(np.float64), W0, M)
    W, st, _ = gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0, M,
                         L.SolverOpts.default(max_iters=1000, fixed_iters=1, check_every=48,
                                              precision=prec))
    W = W.cpu().numpy()
    assert np.all(W[M == 0].view(np.uint32) == 0)
    assert np.linalg.norm(W - ref) <= 1e-4 * np.linalg.norm(ref)
    assert np.all(st["restarts"][1:-1] > 0)


# The same columns as part of a 384-wide layer, whose other entries are zero, take a
# launch per iteration on the tiles: the same sums (a range a 32-wide step, and zeros)
# and the same update, rounding for rounding.
@pytest.mark.parametrize("d, n", [(128, 40), (256, 3), (256, 40)])
def test_blocks_round_as_the_tiles_do(L, d, n):
    H, W0, M, lam = _problem(d, n, d + n)
    H2 = np.eye(384, dtype=np.float32)
    W2, M2 = np.zeros((n, 384), np.float32), np.zeros((n, 384), np.uint8)
    H2[:d, :d], W2[:, :d], M2[:, :d] = H, W0, M
    o = L.SolverOpts.default(max_iters=40, fixed_iters=1, precision=L.PREC_FP32)
    W, _, _ = gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0, M, o)
    ref, _, _ = gpu_solve(L, to_dev(H2), to_dev(np.array([lam])), W2, M2, o)
    np.testing.assert_array_equal(W.cpu().numpy(), ref[:, :d].cpu().numpy())


def test_columns_do_not_depend_on_the_batch(L):
    H, W0, M, lam = _problem(192, 50, 3)
    o = L.SolverOpts.default(eps_rel=1e-4, eps_abs=0.0)
    W, st, _ = gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0, M, o)
    sub, st2, _ = gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0[20:31], M[20:31], o)
    np.testing.assert_array_equal(W[20:31].cpu().numpy(), sub.cpu().numpy())
    np.testing.assert_array_equal(st["iters"][20:31], st2["iters"])


@pytest.mark.parametrize("d, n", [(128, 3), (256, 3), (256, 40)])
def test_counters_do_not_depend_on_the_cooperative_option(L, d, n):
    # No cooperative launch and no few-column kernel runs here.
    H, W0, M, lam = _problem(d, n, d + n)
    out = [gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0, M,
                     L.SolverOpts.default(max_iters=130, fixed_iters=1, cooperative=c))
           for c in (0, 1)]
    np.testing.assert_array_equal(out[0][0].cpu().numpy(), out[1][0].cpu().numpy())
    for _, _, info in out:
        assert info["persistent_launches"] == info["few_launches"] == 0
        assert info["timed_launches"] == 130 and info["checks"] == 4
