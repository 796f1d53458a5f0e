"""The backward pass's grouped launches against the oracle: the 128 x 128 tiles
of the weight gradients (mini-batches with enough of them for the chip), the
64 x 64 ones, more layers than one group holds (8), one hidden layer (whose dZ
has no pre-activation above it to take the place of), and numbers of K slices
that are no multiple of the four staged together.

Gradients per layer in relative Frobenius norm: a rounding that lands on the
other side of a BF16 tie moves a value by 2^-8; with at most 1% of a layer's
values moved, 4e-4 per rounding, growing with the root of their number (two a
layer): 2e-3 for up to eleven layers."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import mlp as M
from paper_2404_07780_amd import gmfit as G


@pytest.mark.parametrize("dims,n", [((1056, 512, 3, 16), 4096), ((1056, 512, 3, 16), 2050), ((64, 64, 10, 16), 300),
                                    ((40, 72, 8, 8), 97), ((168, 136, 1, 24), 600), ((8, 8, 2, 8), 5)])
def test_gradients_match_oracle(dims, n):
    print(f"backward dims {dims} n {n}", flush=True)
    n_out = 7
    flat = M.init_params(21, *dims, n_out=n_out)
    rng = np.random.default_rng(22)
    x = M.bf16(rng.normal(size=(n, dims[0])))
    t = np.zeros((n, dims[3]), np.float32)
    t[:, :n_out] = rng.normal(size=(n, n_out))
    mlp = G.MLP(flat, *dims, n_out=n_out)
    xd = torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda().to(torch.bfloat16)
    td = torch.from_numpy(t).cuda()
    loss = G.gm_mlp_backward(mlp, xd, td).item()
    grad = mlp.grad.cpu().numpy().astype(np.float64)
    rl, rg, _ = M.loss_and_grad(flat.astype(np.float64), x, t.astype(np.float64), n_out=n_out, dims=dims)
    assert abs(loss - rl) <= 1e-5 * rl, (loss, rl)
    for l, ((gW, gb), (rW, rb)) in enumerate(zip(M.unpack(grad, *dims), M.unpack(rg, *dims))):
        for name, a, b in (("W", gW, rW), ("b", gb, rb)):
            rel = np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)
            print(f"layer {l} {name}: rel err {rel:.2e}", flush=True)
            assert rel <= 2e-3, (l, name, rel)
    first = mlp.grad.clone()
    G.gm_mlp_backward(mlp, xd, td)
    assert torch.equal(first, mlp.grad)
