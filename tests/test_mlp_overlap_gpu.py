"""Forward passes whose logits overlap their inputs: the logits of a call that keeps them apart."""
import ctypes as C

import numpy as np
import pytest

from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu

# one tile of rows, a ragged last one, and (with a workspace) more workgroups than run at once
CASES = [(16, True), (16, False), (1000, True), (1000, False), (4096, False), (65541, True)]


@pytest.mark.parametrize("over", ["x", "params"])
@pytest.mark.parametrize("batch,workspace", CASES)
def test_logits_over_inputs(batch, workspace, over):
    import torch
    print(f"case: logits over {over}, batch {batch}, workspace {workspace}", flush=True)
    L = ptqmc.lib()
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    rng = np.random.default_rng(batch)
    n = int(L.pt_mlp_param_count())
    params = torch.from_numpy(rng.normal(0, 0.1, n).astype(np.float32)).cuda()
    x = torch.from_numpy(rng.normal(size=(batch, 32)).astype(np.float32)).cuda()
    ws = torch.empty(int(L.pt_mlp_workspace_bytes(batch)), dtype=torch.uint8, device="cuda")

    def forward(p, features, logits):
        if workspace:
            rc = L.pt_mlp_forward(p.data_ptr(), features.data_ptr(), logits.data_ptr(), batch, ws.data_ptr(), stream)
        else:
            rc = L.pt_mlp_forward_static(p.data_ptr(), features.data_ptr(), logits.data_ptr(), batch, stream)
        assert rc == 0, L.pt_last_error()
        torch.cuda.synchronize()

    want = torch.empty((batch, 64), dtype=torch.float32, device="cuda")
    forward(params, x, want)
    if over == "x":
        both = torch.empty(batch * 64, dtype=torch.float32, device="cuda")
        both[:batch * 32] = x.reshape(-1)
        forward(params, both[:batch * 32], both)
        got = both
    else:
        both = torch.empty(n + batch * 64, dtype=torch.float32, device="cuda")
        both[:n] = params
        got = both[n - 1:n - 1 + batch * 64]  # starts at the last bias
        forward(both[:n], x, got)
    assert torch.equal(got.reshape(batch, 64), want)
