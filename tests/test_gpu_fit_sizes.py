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


def _columns(kind, T, d, g):
    """bf16 data of kinds that the integer form of the Gram products treats differently."""
    x = torch.randn(T, d, generator=g)
    if kind == "spread":                                       # every column has values 13 and more binades below its largest
        n = min(T, 40)
        rows = torch.randperm(T, generator=g)[:n]
        x[rows] *= torch.exp2(torch.randint(-30, -8, (n, d), generator=g).float())
        x[:, 5] = 0.0
    elif kind == "many small":                                 # more such values than the lists hold: the fp64 form
        x[1:, : d // 2] *= 2.0 ** -20
    elif kind.endswith("small"):                               # about so many of them in every column
        small = torch.rand(T, d, generator=g) < int(kind.split()[0]) / T
        x = torch.where(small, x * 2.0 ** -20, x)
    elif kind == "one column":
        x[1:901, 7] *= 2.0 ** -20
    elif kind == "tiny column":                                # no fp32 scale takes its values to integers: the fp64 form
        x[:, 3] *= 2.0 ** -118
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("kind", ["gauss", "spread", "many small", "tiny column", "3 small", "one column"])
@pytest.mark.parametrize("T,d0,d1,d_out", [
    (2559, 256, 0, 128), (2560, 256, 0, 128), (2561, 128, 128, 128), (2623, 256, 128, 128), (4097, 128, 384, 384), (847, 1024, 1024, 1024),
    (2048, 1024, 1024, 1024), (32769, 256, 0, 128)])
def test_fit_from_integer_products(T, d0, d1, d_out, kind):
    """Edges of the sizes that are formed in integers, of the steps of 64 tokens, of the 512 steps that int32 sums hold and of the 32 workgroups of an XCD.  The Gram products are
    exact but for one rounding each (their fp64 form: T), so the solution is off by the condition number, below 1e5 for these data, times 2^-53
    times the order of the matrix, 2e-8 at worst; 1e-9 is asked, as of the fp64 form above."""
    from paper_2501_19392_amd import binding as B
    print(f"case fit integer T={T} d0={d0} d1={d1} d_out={d_out} {kind}", flush=True)
    d = d0 + d1
    g = torch.Generator().manual_seed(T + d)
    X, Y = _columns(kind, T, d, g), _columns("spread" if kind == "spread" else "gauss", T, d_out, g)
    x1 = X[:, d0:].contiguous().cuda() if d1 else None
    W = torch.empty(d_out, d, dtype=torch.bfloat16, device="cuda")
    W64 = torch.empty(d_out, d, dtype=torch.float64, device="cuda")
    ws = torch.empty(B.aquakv_fit_workspace_bytes(d, d_out), dtype=torch.uint8, device="cuda")
    bias = torch.empty(d_out, dtype=torch.float32, device="cuda") if d1 else None
    first = None
    for _ in range(2):
        ws.fill_(0xff)
        B.aquakv_fit_predictor(torch.bfloat16, T, X[:, :d0].contiguous().cuda(), d0, x1, d1, Y.cuda(), d_out, 1e-2, W, W64, ws, bias=bias)
        torch.cuda.synchronize()
        got = W64.cpu().numpy()
        assert first is None or np.array_equal(first, got)
        first = got
    want = C.fit_predictor(U.np64(X), U.np64(Y), 1e-2, bias=bias is not None)
    if bias is not None:
        want, want_b = want
        assert np.allclose(bias.cpu().numpy(), want_b, rtol=1e-5, atol=1e-6 * np.abs(want_b).max() + 1e-7)
    rel = np.linalg.norm(got - want) / np.linalg.norm(want)
    print("rel", rel, flush=True)
    assert rel < 1e-9, rel


@pytest.mark.parametrize("kind,T,d,most", [("many small", 16384, 1024, 1.5), ("800 small", 16384, 2048, 1.25),
                                                 ("100 small", 16384, 2048, 0.85), ("one column", 16384, 2048, 0.85)])
def test_lists_cost_no_more_than_the_fp64_form(kind, T, d, most):
    """Time of a fit over that of one whose data is known not to fit before anything is listed, which is that of the fp64 form plus two
    passes over the data.  Half of the columns with nothing but small values: the lists overflow, and counting them takes a workgroup an
    atomic per column (1.0 of the time; 3.1 with an atomic per value).  Lists that would cost more than the integers gain: the fp64
    form (1.0; 1.6 if they are gone through all the same).  Shorter ones, or a long one alone: integers (0.63 and 0.55)."""
    from paper_2501_19392_amd import binding as B
    d_out = 1024
    print(f"case fit lists {kind} T={T} d={d} d_out={d_out}", flush=True)
    W = torch.empty(d_out, d, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(B.aquakv_fit_workspace_bytes(d, d_out), dtype=torch.uint8, device="cuda")
    times = {}
    for which in ("tiny column", kind):
        X, Y = (_columns(which, T, n, torch.Generator().manual_seed(n)).cuda() for n in (d, d_out))
        best = []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            B.aquakv_fit_predictor(torch.bfloat16, T, X, d, None, 0, Y, d_out, 1e-2, W, None, ws)
            end.record()
            torch.cuda.synchronize()
            best.append(start.elapsed_time(end))
        times[which] = min(best)
    print(times, flush=True)
    assert times[kind] / times["tiny column"] < most, times


@pytest.mark.parametrize("T", [2559, 2560])                    # the fp64 form, and integers, which leave the data to it
def test_fit_of_infinities_is_nan_in_both_forms(T):
    from paper_2501_19392_amd import binding as B
    print(f"case fit infinity T={T}", flush=True)
    d, d_out = 256, 128
    g = torch.Generator().manual_seed(3)
    X, Y = torch.randn(T, d, generator=g).bfloat16().cuda(), torch.randn(T, d_out, generator=g).bfloat16().cuda()
    W = torch.zeros(d_out, d, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(B.aquakv_fit_workspace_bytes(d, d_out), dtype=torch.uint8, device="cuda")
    X[7, 9] = float("inf")
    B.aquakv_fit_predictor(torch.bfloat16, T, X, d, None, 0, Y, d_out, 1e-2, W, None, ws)
    assert W.isnan().all()
