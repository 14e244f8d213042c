"""The prior's forward pass and gradient at the edges of their tiles and
blocks: waves without rows, a last tile of one row, a second pass of the first
block's waves; the gradient is added to what the caller's buffers hold."""
import numpy as np
import pytest

from oracle import prior as oprior

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def acs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1605_02669_amd import acs as mod
    mod.load()
    return mod


# tiles of 32 rows, 8 waves a block, 256 blocks: 65536 rows are one pass
@pytest.mark.parametrize("rows", [1, 32, 33, 256, 257, 65536 + 33])
def test_gradient_at_tile_edges(acs, rows):
    import torch
    from paper_1605_02669_amd import prior
    g = np.random.default_rng(rows)
    X = g.uniform(-1, 1, size=(rows, 4)).astype(np.float32)
    Y = g.uniform(0, 1, size=rows).astype(np.float32)
    flat = prior.init_params(rows)
    P = torch.tensor(flat, device="cuda")
    G = torch.full((acs.PRIOR_PARAMS,), 0.25, dtype=torch.float32, device="cuda")
    L = torch.full((1,), 8.0, dtype=torch.float32, device="cuda")
    print("rows", rows, flush=True)
    acs.prior_grad(P, torch.tensor(X, device="cuda"), torch.tensor(Y, device="cuda"), G, L)
    torch.cuda.synchronize()
    p = acs.unpack_prior(flat)
    got = acs.unpack_prior(G.cpu().numpy().astype(np.float64) - 0.25)
    ref = oprior.grads(p, X, Y.astype(np.float64), bf16_ops=True)
    # bf16 operands: 2^-8 relative per rounded activation, some of which round
    # the other way after fp32 sums; adding to 0.25 rounds to 2^-25 absolute
    for k in ("W1", "b1", "W2", "b2", "W3", "b3"):
        a, b = got[k].reshape(-1).astype(np.float64), ref[k].reshape(-1)
        assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b) + 2.0**-24 * np.sqrt(b.size), k
    lo = oprior.loss(p, X, Y.astype(np.float64), bf16_ops=True)
    assert abs((L.item() - 8.0) / rows - lo) <= 1e-3 * (1 + abs(lo)) + 8.0 * 2.0**-23 / rows


# tiles of 32 rows, 4 waves a block, 768 blocks: 98304 rows are one pass
@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 98304 + 17])
def test_forward_at_tile_edges(acs, rows):
    import torch
    from paper_1605_02669_amd import prior
    g = np.random.default_rng(rows)
    X = g.uniform(-1, 1, size=(rows, 4)).astype(np.float32)
    flat = prior.init_params(rows)
    print("rows", rows, flush=True)
    P, Xd = torch.tensor(flat, device="cuda"), torch.tensor(X, device="cuda")
    z = torch.full((rows + 64,), 7.0, dtype=torch.float32, device="cuda")
    acs._check(acs.load().acs_prior_forward(acs.C.c_void_p(P.data_ptr()),
                                            acs.C.c_void_p(Xd.data_ptr()), rows,
                                            acs.C.c_void_p(z.data_ptr()), None))
    torch.cuda.synchronize()
    z = z.cpu().numpy()
    assert np.all(z[rows:] == 7.0)
    zo, _ = oprior.forward(acs.unpack_prior(flat), X, bf16_ops=True)
    # as for the random sizes: fp32 sums, bf16 activations that round the other way
    assert np.all(np.abs(z[:rows] - zo) <= 1e-2 * (1 + np.abs(zo)))
