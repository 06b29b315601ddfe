"""The least-squares fit at the edges of its token steps (128 bf16 or 64 fp32 tokens, 16 or 8 per wave), with fewer output tiles than
CUs, with tiles that two workgroups share, and with one or two block columns."""
import numpy as np
import pytest
import torch

from oracle import calibration_oracle as C
from paper_2501_19392_amd import synth
from tests import parity_utils as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,T,d0,d1,d_out", [
    ("bf16", 1, 64, 0, 64), ("fp32", 7, 64, 0, 128), ("bf16", 17, 64, 64, 64), ("bf16", 127, 128, 0, 64), ("bf16", 128, 64, 0, 64),
    ("bf16", 129, 192, 64, 128), ("fp32", 63, 128, 0, 64), ("fp32", 65, 64, 128, 192), ("bf16", 1025, 1024, 0, 1024),
    ("fp32", 300, 1024, 0, 1024), ("bf16", 2111, 1024, 576, 640)])
def test_fit_at_step_and_tile_edges(dtype, T, d0, d1, d_out):
    from paper_2501_19392_amd import binding as B
    print(f"case fit edges dtype={dtype} T={T} d0={d0} d1={d1} d_out={d_out}", flush=True)
    sd = synth.torch_dtype(dtype)
    g = torch.Generator().manual_seed(T)
    X = torch.randn(T, d0 + d1, generator=g).to(sd)
    Y = torch.randn(T, d_out, generator=g).to(sd)
    d = d0 + d1
    x1 = X[:, d0:].contiguous().cuda() if d1 else None
    W = torch.empty(d_out, d, dtype=sd, device="cuda")
    W64 = torch.empty(d_out, d, dtype=torch.float64, device="cuda")
    ws = torch.empty(B.aquakv_fit_workspace_bytes(d, d_out), dtype=torch.uint8, device="cuda")
    first = None
    for _ in range(2):
        ws.fill_(0xff)                                         # NaNs: nothing may be read before it is written
        B.aquakv_fit_predictor(sd, T, X[:, :d0].contiguous().cuda(), d0, x1, d1, Y.cuda(), d_out, 1e-2, W, W64, ws)
        torch.cuda.synchronize()
        got = W64.cpu().numpy()
        assert first is None or np.array_equal(first, got)     # the order of every sum is fixed
        first = got
    want = C.fit_predictor(U.np64(X), U.np64(Y), 1e-2)
    rel = np.linalg.norm(got - want) / np.linalg.norm(want)
    assert rel < 1e-9, rel
