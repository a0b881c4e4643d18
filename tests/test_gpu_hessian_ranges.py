"""Short bf16 token ranges: one workgroup runs all ranges of a 256 x 256 tile.

Each range (a few 64-token stages) is one chain of fp32 sums and the ranges are
added in order, so the error stays that of chains of a few stages however they
are spread over workgroups.
"""
import numpy as np
import pytest
import torch

import paper_2512_13886_amd as L

pytestmark = pytest.mark.gpu


def _x(n_tok, d, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n_tok, d, device="cuda", generator=g).to(torch.bfloat16)


# One stage (whole and with a remainder); several ranges of unequal numbers of
# stages, ending in the rows of a partial stage or without them; widths whose
# last XCD share is short; d = 2048 keeps the split plan.
@pytest.mark.parametrize("d", [2048, 4096, 5120])
@pytest.mark.parametrize("n_tok", [40, 64, 100, 700, 2048, 2111])
def test_sum_and_accumulation(n_tok, d):
    X, Y = _x(n_tok, d, n_tok + d), _x(n_tok, d, n_tok + d + 1)
    H = torch.full((d, d), float("nan"), device="cuda")
    L.optima_hessian_accumulate(X, H)
    again = torch.full((d, d), float("nan"), device="cuda")
    L.optima_hessian_accumulate(X, again)
    assert torch.equal(H, again) and torch.equal(H, H.T)
    X64 = X.double()
    ref = X64.T @ X64
    # The bf16 products are exact in fp32. A range of these sizes is at most 6
    # stages of two MFMA steps, and at most 11 ranges are added: no entry passes
    # through more than 12 + 10 roundings, and one with the incoming sum, each off
    # by at most 2^-23 of the magnitudes' sum.
    bound = 24 * 2.0 ** -23 * (X64.abs().T @ X64.abs())
    assert bool(((H.double() - ref).abs() <= bound).all())
    # Typical rounding adds in the root of the number of terms: the error over
    # the whole matrix is within a small multiple of one rounding, where a single
    # chain of 64 steps has three times as much.
    rel = float((H.double() - ref).norm() / ref.norm())
    print(f"d={d} n_tok={n_tok}: {rel:.2e}")
    assert rel <= 2.0 ** -23
    before = H.clone()
    L.optima_hessian_accumulate(Y, H, accumulate=True)
    Z = torch.empty_like(H)
    L.optima_hessian_accumulate(Y, Z)
    assert torch.equal(H, before + Z)


# Widths whose tiles fill the chip once take whole stages in one chain of sums, and
# token counts with last rows in two at least. The error of a chain grows as the root
# of its length or faster: at 2000 tokens it is at most 1 / sqrt(2) of that of one
# chain, and one part in eight more for the scatter of the two.
@pytest.mark.parametrize("d", [5632, 7936])
def test_last_rows_come_with_two_chains(d):
    X = _x(2000, d, d)

    def error(n_tok):
        H = torch.empty((d, d), device="cuda")
        L.optima_hessian_accumulate(X[:n_tok], H)
        X64 = X[:n_tok].double()
        ref = X64.T @ X64
        return float((H.double() - ref).norm() / ref.norm())

    assert error(2000) <= 2 ** -0.5 * 1.125 * error(1984)


@pytest.mark.parametrize("d", [256, 1024, 2048, 4096, 6144, 14336])
def test_workspace_never_shrinks_with_more_tokens(d):
    need = [L.optima_hessian_workspace_bytes(n, d, L.DTYPE_BF16)
            for n in np.unique(np.geomspace(1, 262144, 60).astype(int)).tolist()]
    assert all(a <= b for a, b in zip(need, need[1:]))
