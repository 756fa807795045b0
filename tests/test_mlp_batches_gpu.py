"""The ladder network's kernels at the edges of their splits: batches around the 16 rows of a
workgroup, the 64 rows of a wave of the weight gradients, and its 16 waves; and parameters
and inputs at addresses of any float.

Tolerance: a value is a chain of at most three sums of 128 products and, for gradients, one
over the batch, each rounded to 2^-24 relative per term: a root-mean-square error of about
sqrt(3 * 128 + B) 2^-24, and four times that (and of the approximate exponentials, a few 2^-23)
for the 2-norm of the whole output."""
import numpy as np
import pytest

from oracle import mlp
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu


def problem(B):
    rng = np.random.default_rng([7, B])
    p = ptqmc.init_ladder_params(B)
    p[-64 * 128 - 64:] = rng.normal(0, 0.1, 64 * 128 + 64).astype(np.float32)
    x = rng.normal(size=(B, 32)).astype(np.float32)
    q = rng.random((B, 64)).astype(np.float32)
    return p, x, q


def close(got, want, B):
    tol = 4 * (np.sqrt(3 * 128 + B) * 2.0 ** -24 + 4 * 2.0 ** -23)
    got = np.asarray(got, np.float64)
    assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("kind", ["softmax", "sigmoid"])
@pytest.mark.parametrize("B", [1, 3, 15, 16, 17, 63, 64, 65, 129, 1023, 1024, 1025, 2049])
def test_batches(B, kind):
    print(f"case: ladder network, batch {B}, {kind}", flush=True)
    p, x, q = problem(B)
    if kind == "softmax":
        q = q / q.sum(1, keepdims=True)
    net = ptqmc.LadderNet(p)
    p64, x64, q64 = (a.astype(np.float64) for a in (p, x, q))
    close(net.forward(x).cpu().numpy(), mlp.forward(p64, x64)[0], B)
    loss = net.loss_grad(x, q, ptqmc.MLP_LOSS_SOFTMAX if kind == "softmax" else ptqmc.MLP_LOSS_SIGMOID)
    want, grads = mlp.loss_grad(p64, x64, q64, kind)
    close([loss], np.array([want]), B)
    close(net.grads.cpu().numpy(), grads, B)


def test_unaligned_addresses():
    import torch
    print("case: ladder network at odd float addresses", flush=True)
    p, x, q = problem(20)
    shifted = lambda a: torch.cat([torch.zeros(1), torch.from_numpy(a).flatten()]).cuda()[1:]
    L, B = ptqmc.lib(), 20
    dp, dx, dq = shifted(p), shifted(x), shifted(q)
    ws = torch.empty(L.pt_mlp_workspace_bytes(B) + 4, dtype=torch.uint8, device="cuda")[4:]
    out, g, loss = (torch.empty(n + 1, device="cuda")[1:] for n in (B * 64, p.size, 1))
    s = torch.cuda.current_stream().cuda_stream
    assert L.pt_mlp_forward_static(dp.data_ptr(), dx.data_ptr(), out.data_ptr(), B, s) == 0
    assert L.pt_mlp_loss_grad(dp.data_ptr(), dx.data_ptr(), dq.data_ptr(), B, ptqmc.MLP_LOSS_SIGMOID,
                              g.data_ptr(), loss.data_ptr(), ws.data_ptr(), s) == 0
    p64, x64, q64 = (a.astype(np.float64) for a in (p, x, q))
    close(out.cpu().numpy().reshape(B, 64), mlp.forward(p64, x64)[0], B)
    close(g.cpu().numpy(), mlp.loss_grad(p64, x64, q64, "sigmoid")[1], B)
