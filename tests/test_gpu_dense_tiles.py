"""The iteration products on every tile that their plans take, at the tiles'
and loops' remainders: ragged batches, half a 256-wide tile at the end of H,
split contractions down to one stage a range. Columns are independent, so the
oracle runs on a sample of them, the batch's last rows among it."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, gpu_solve, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2512_13886_amd as lib
    return lib


# (d, columns): the 256 x 256 tile with a half tile of H and a ragged last row
# tile; the same split in three; the 128 x 128 ring with one, two and three
# stages left over and split into 5 and 16 ranges; the 4-wave 128 x 128 tile.
@pytest.mark.parametrize("d, n", [(1100, 9000), (2944, 1500), (2176, 1030), (1152, 2000),
                                  (300, 300), (640, 700), (512, 33), (1100, 6000)])
def test_products_match_the_oracle(L, d, n):
    rng = np.random.default_rng(d + n)
    A = rng.standard_normal((d + 64, d)) * np.exp(rng.normal(0.0, 0.5, d))
    H = A.T @ A
    H = ((H + H.T) / 2 + 0.01 * np.trace(H) / d * np.eye(d)).astype(np.float32)
    W0 = (0.02 * rng.standard_normal((n, d))).astype(np.float32)
    M = (rng.random((n, d)) < 0.5).astype(np.uint8)
    M[0] = 1  # dense products
    lam = np.float32(1.05 * np.linalg.norm(H.astype(np.float64) @ rng.standard_normal(d)))
    W, st, info = gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0, M,
                            L.SolverOpts.default(max_iters=6, fixed_iters=1))
    assert info["sparse_products"] == 0
    W = W.cpu().numpy()
    assert np.all(W[M == 0].view(np.uint32) == 0)
    cols = np.unique(np.concatenate([rng.choice(n, min(n, 24), replace=False),
                                     np.arange(max(0, n - 8), n)]))
    ref = oracle.rapdhg(H.astype(np.float64), W0[cols], M[cols], float(lam),
                        oracle.SolverOptions(max_iters=6, fixed_iters=True))
    # Before the first check both follow the same continuous map; bf16x3 products
    # are off by up to 3 * 2^-16 each.
    err = np.linalg.norm(W[cols] - ref.W, axis=1) / np.linalg.norm(ref.W, axis=1)
    assert err.max() <= 1e-4
    np.testing.assert_allclose(st["f_initial"][cols], ref.f_initial, rtol=1e-5, atol=1e-12)


# The sums keep to short chains of MFMA additions, at most `stages` of 32 products,
# whatever the tile: the ring with ranges that end in registers, the 256 x 256 tile
# with a workgroup for each of three, the split plan of few columns. The inputs are
# bf16 values, so that W after one iteration is off by the rounding of two sums and
# of what follows them alone. A stage rounds the running sum a few times by up to
# 2^-25 of it each, and partial sums and roundings both grow as the root of their
# number: sqrt(stages) 2^-24 of the result, and a few roundings outside the chains.
# (Chains of a whole contraction have 1.4 to 2.2 times these errors, beyond the bound
# in every case.)
@pytest.mark.parametrize("d, n, stages", [(512, 606, 1), (640, 4000, 4), (768, 3072, 5),
                                          (1792, 55, 4), (1792, 6144, 19), (2944, 893, 31),
                                          (2048, 2048, 22), (2048, 3072, 32)])
def test_chains_of_sums_stay_short(L, d, n, stages):
    g = torch.Generator(device=dev()).manual_seed(d)

    def values(*shape):
        return torch.randn(*shape, generator=g, device=dev()).bfloat16().float()

    H = torch.tril(values(d, d))
    H = H + torch.tril(H, -1).t()
    W0 = values(n, d)
    M = (torch.rand(n, d, generator=g, device=dev()) < 0.5).to(torch.uint8)
    M[0] = 1  # dense products
    opts = L.SolverOpts.default(max_iters=1, fixed_iters=1)
    # A step of 1 / 2: W = sel(M, x0 - (H x0 - H w0), 0).
    lam = torch.full((1,), 0.5 / (1 + opts.step_safety), device=dev())
    W, _, _ = gpu_solve(L, H, lam, W0, M, opts)
    X = (W0 * M).double()
    ref = torch.where(M != 0, X - (X - W0.double()) @ H.double(), 0.0)
    rel = float((W.double() - ref).norm() / ref.norm())
    print(f"d={d} n={n}: {rel * 2 ** 24:.2f} x 2^-24")
    assert rel <= (stages + 3) ** 0.5 * 2.0 ** -24


# (d, columns): the 256 x 128 tile of the 2:4 products in one range of 24 stages
# and in 2 to 11 ranges of 1 to 8 stages, odd counts among them, with one row and
# one full tile in the last row tile, and a padded d.
@pytest.mark.parametrize("d, n", [(640, 2100), (1536, 4096), (768, 3073), (512, 257), (768, 300),
                                  (2048, 130), (1100, 512), (4096, 9)])
def test_sparse_products_match_the_oracle(L, d, n):
    rng = np.random.default_rng(d + n)
    A = rng.standard_normal((d + 64, d)) * np.exp(rng.normal(0.0, 0.5, d))
    H = A.T @ A
    H = ((H + H.T) / 2 + 0.01 * np.trace(H) / d * np.eye(d)).astype(np.float32)
    W0 = (0.02 * rng.standard_normal((n, d))).astype(np.float32)
    order = rng.random((n, d // 4, 4)).argsort(axis=2)
    M = (order < rng.integers(0, 3, (n, d // 4, 1))).astype(np.uint8).reshape(n, d)
    lam = np.float32(1.05 * np.linalg.norm(H.astype(np.float64) @ rng.standard_normal(d)))
    W, st, info = gpu_solve(L, to_dev(H), to_dev(np.array([lam])), W0, M,
                            L.SolverOpts.default(max_iters=6, fixed_iters=1))
    assert info["sparse_products"] == 1
    W = W.cpu().numpy()
    assert np.all(W[M == 0].view(np.uint32) == 0)
    cols = np.unique(np.concatenate([rng.choice(n, min(n, 24), replace=False),
                                     np.arange(max(0, n - 8), n)]))
    ref = oracle.rapdhg(H.astype(np.float64), W0[cols], M[cols], float(lam),
                        oracle.SolverOptions(max_iters=6, fixed_iters=True))
    # The bound of the dense products.
    norm = np.linalg.norm(ref.W, axis=1)
    err = np.linalg.norm(W[cols] - ref.W, axis=1) / np.maximum(norm, 1e-30)
    assert err.max() <= 1e-4
    np.testing.assert_allclose(st["f_initial"][cols], ref.f_initial, rtol=1e-5, atol=1e-12)


def test_conjugate_gradients_on_the_large_tile(L):
    # kPlain products: 4096 columns of 1024, one range, 256 x 256 tiles.
    d, n = 1024, 9000
    g = torch.Generator(device=dev()).manual_seed(5)
    A = torch.randn(2 * d, d, generator=g, device=dev(), dtype=torch.float64)
    H = (A.t() @ A + d * torch.eye(d, device=dev(), dtype=torch.float64)).float()
    H = torch.tril(H) + torch.tril(H, -1).t()
    W0 = 0.02 * torch.randn(n, d, generator=g, device=dev())
    M = (torch.rand(n, d, generator=g, device=dev()) < 0.5).to(torch.uint8)
    W, _, _ = gpu_solve(L, H, None, W0, M,
                        L.SolverOpts.default(method=L.METHOD_CG, max_iters=40, fixed_iters=1))
    x = W.double()
    r = torch.where(M != 0, (W0.double() - x) @ H.double(), 0.0)
    b = torch.where(M != 0, W0.double() @ H.double(), 0.0)
    assert bool((W[M == 0] == 0).all())
    assert float((r.norm(dim=1) / b.norm(dim=1)).max()) <= 1e-4
