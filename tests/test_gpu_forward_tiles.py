"""The forward pass on 256 x 256 tiles, at the edges of the tiles and of the
two-stage loop (one, two and three stages of 64 inputs), against fp64."""
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import paper_2512_13886_amd as lib
    return lib


# All of these take the large tile: two rounds of it against three or more of
# two 128 x 128 tiles a CU. The last has a misaligned W.
@pytest.mark.parametrize("n_tok, d_in, d_out, off", [(4097, 64, 4100, 0), (4096, 128, 4096, 0),
                                                     (4200, 192, 3972, 0), (20001, 320, 1284, 1)])
def test_wide_tile_matches_fp64(L, n_tok, d_in, d_out, off):
    g = torch.Generator(device=dev()).manual_seed(n_tok)
    X = torch.randn(n_tok, d_in, generator=g, device=dev()).bfloat16()
    W = torch.randn(d_out * d_in + off, generator=g, device=dev())[off:].view(d_out, d_in)
    W2 = W * 1.25
    Z = X.double() @ W.bfloat16().double().t()
    Z2 = X.double() @ W2.bfloat16().double().t()
    # fp32 sums of d_in exact products in any order.
    bound = d_in * 2.0 ** -24 * (X.double().abs() @ W.bfloat16().double().abs().t())
    Y = torch.full((n_tok, d_out), float("nan"), device=dev())
    L.optima_linear_forward(X, W, Y=Y)
    assert bool(((Y.double() - Z).abs() <= bound).all())
    out = torch.full((n_tok, d_out), float("nan"), dtype=torch.bfloat16, device=dev())
    err = torch.zeros(1, dtype=torch.float64, device=dev())
    L.optima_linear_forward(X, W2, Y=out, act=L.ACT_SILU, Y_ref=Y, err_out=err)
    ref = torch.nn.functional.silu(Z2)
    # half a bf16 step, and what the sum and expf can move it by
    assert bool(((out.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 3 * bound + 1e-30).all())
    want = (Z2 - Z).square().sum().item()
    assert abs(err.item() - want) <= 1e-5 * want


def test_wide_tile_leaves_outputs_alone_on_nonfinite_weights(L):
    X = torch.ones(4096, 64, device=dev()).bfloat16()
    W = torch.ones(4096, 64, device=dev())
    W[17, 3] = float("inf")
    Y = torch.full((4096, 4096), 7.0, device=dev())
    with pytest.raises(L.OptimaError) as e:
        L.optima_linear_forward(X, W, Y=Y)
    assert e.value.status == -3
    assert bool((Y == 7.0).all())
