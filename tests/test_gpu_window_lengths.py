"""Window lengths 9 to 15, which take the streaming schedule in every form of
a call: against the fp64 oracle with the tolerances of the entry points' own
parity tests (EAL gradients: widened by a bound on K rounded acceptances);
and the properties that callers get from one schedule for all forms: the same
bits whichever flag is set and whether or not a gradient is asked for, and no
waits between workgroups, so that calls on several streams hold nothing from
each other."""
import math

import pytest
import torch

import oracle as O
import test_gpu_general as general
import test_gpu_parity as parity_cases
from parity import check_grad, eal_coef, host64, loss_tol, rel_err

pytestmark = pytest.mark.gpu

BF16, F32 = torch.bfloat16, torch.float32


@pytest.fixture(scope="module")
def A():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_24150_amd as lib
    return lib


@pytest.mark.parametrize("dtype,gdtype", [(BF16, BF16), (BF16, F32), (F32, F32), (F32, BF16)])
@pytest.mark.parametrize("K", range(9, 16))
def test_losses(A, K, dtype, gdtype):
    dev = torch.device("cuda:0")
    zd, zt = parity_cases._inputs("c1" if dtype == F32 else "c2", (100, K, 8808), dtype, seed=K, dev=dev)
    parity_cases._check_wtv(A, zd, zt, 0.9, 1.1, gdtype, 0)
    # A row's coefficient multiplies up to K acceptances q(x*) = 2^(z sc - msc - l2s); the
    # exponent's two roundings (|msc|, |l2s| < 32: half a unit is 2^-20 each, times ln 2) put up to
    # 1.4 * 2^-20 of relative error on each, so K of them exceed the 2^-18 of check_grad from K = 3 on.
    zd, zt = parity_cases._inputs("c1" if dtype == F32 else "c2", (60, K, 24584), dtype, seed=K, dev=dev)
    r = A.aal_eal_fwd_bwd(zd, zt, 0.9, grad_dtype=gdtype)
    torch.cuda.synchronize()
    o = O.eal_loss(host64(zd), host64(zt), 0.9)
    tol = loss_tol(dtype)
    assert rel_err(r["loss"].item(), o["loss"]) <= tol
    assert rel_err(host64(r["E"]), o["E"]) <= tol
    assert rel_err(host64(r["accept"]), o["a"]) <= tol
    assert (r["xstar"].cpu().numpy() == o["xstar"]).all()
    coef = eal_coef(o, 60, 0.9)
    extra = (K * 1.4 * 2.0 ** -20 * abs(coef))[..., None] * torch.ones(24584, dtype=torch.float64).numpy()
    check_grad(host64(r["grad"]), o["grad"], coef, dtype, gdtype, extra_tol=extra)


@pytest.mark.parametrize("dtype,gdtype", [(BF16, BF16), (BF16, F32), (F32, F32)])
@pytest.mark.parametrize("weights", general.WEIGHTS)
@pytest.mark.parametrize("K", range(9, 16))
def test_combined(A, K, weights, dtype, gdtype):
    zd, zt = general._inputs(2, 3 * K + 4, 8808, dtype, seed=K)
    general._check(A, zd, zt, K, weights, general.SEQ, Td=0.8, Tt=1.2, gdt=gdtype)
    general._check(A, zd[:, :K].contiguous(), zt[:, :K].contiguous(), K, weights, general.WIN, gdt=gdtype)


def _calls(A, K, dev):
    """The loss calls at window length K, over shapes whose rows span several workgroups' worth of
    vectors; each takes grad and flags."""
    zd, zt = parity_cases._inputs("c2", (60, K, 24584), BF16, seed=K, dev=dev)
    fd, ft = parity_cases._inputs("c1", (30, K, 8808), F32, seed=K, dev=dev)
    sd, st = parity_cases._inputs("c2", (2, 3 * K + 4, 8808), BF16, seed=K, dev=dev)
    calls = {
        "eal": lambda **kw: A.aal_eal_fwd_bwd(zd, zt, 0.9, **kw),
        "wtv": lambda **kw: A.aal_wtv_fwd_bwd(zd, zt, 0.9, 1.1, **kw),
        "wtv fp32": lambda **kw: A.aal_wtv_fwd_bwd(fd, ft, 0.9, 1.1, **kw),
        "wtv, fp32 gradient": lambda **kw: A.aal_wtv_fwd_bwd(zd, zt, 0.9, 1.1, grad_dtype=F32, **kw),
    }
    for weights in general.WEIGHTS:
        calls[f"windows {weights}"] = lambda w=weights, **kw: A.aal_loss_fwd_bwd(zd, zt, K, weights=w, **kw)
        calls[f"sequences {weights}"] = lambda w=weights, **kw: A.aal_loss_fwd_bwd(
            sd, st, K, weights=w, layout=A.AAL_LAYOUT_SEQUENCES, **kw)
    return calls


@pytest.mark.parametrize("K", range(9, 16))
def test_same_bits_in_every_form(A, K):
    dev = torch.device("cuda:0")
    for name, call in _calls(A, K, dev).items():
        ref = call(grad=True, flags=0)
        forms = {"cooperative": call(grad=True, flags=A.AAL_FLAG_COOPERATIVE),
                 "streaming": call(grad=True, flags=A.AAL_FLAG_STREAMING),
                 "forward only": call(grad=False, flags=0)}
        torch.cuda.synchronize()
        for form, r in forms.items():
            for k, v in ref.items():
                if v is not None and not (k == "grad" and form == "forward only"):
                    assert torch.equal(r[k].view(torch.uint8), v.view(torch.uint8)), (name, form, k)


@pytest.mark.parametrize("K", range(9, 16))
def test_no_waits_between_workgroups(A, K, monkeypatch):
    """A schedule whose workgroups wait for each other reads NaN when it is started in its timed-out
    state (see test_gpu_timeout); these calls have no such state."""
    calls = _calls(A, K, torch.device("cuda:0"))
    monkeypatch.setenv("AAL_TEST_PRESET_TIMEOUT", "1")
    for name, call in calls.items():
        r = call(grad=True, flags=0)
        torch.cuda.synchronize()
        assert math.isfinite(r["loss"].item()), name


@pytest.mark.parametrize("K", [9, 12, 15])
def test_unflagged_calls_on_two_streams(A, K):
    """Two device-filling calls at once, without AAL_FLAG_COOPERATIVE: each gives a lone call's bits."""
    dev = torch.device("cuda:0")
    calls = [c for name, c in _calls(A, K, dev).items() if name in ("wtv", "eal", "wtv fp32")]
    refs = [c() for c in calls]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(dev), torch.cuda.Stream(dev)]
    outs = []
    for _ in range(3):
        for call, ref in zip(calls, refs):
            for s in streams:
                with torch.cuda.stream(s):
                    outs.append((call(stream=s), ref))
    torch.cuda.synchronize()
    for r, ref in outs:
        for k, v in ref.items():
            if v is not None:
                assert torch.equal(r[k].view(torch.uint8), v.view(torch.uint8)), k


@pytest.mark.parametrize("K", [9, 12, 15])
def test_flagged_calls_can_be_captured(A, K):
    """AAL_FLAG_COOPERATIVE needs no cooperative launch at these lengths, so the call goes into a graph;
    three replays with eager work between them."""
    calls = _calls(A, K, torch.device("cuda:0"))
    for name in ("wtv", "eal"):
        ref = calls[name](flags=A.AAL_FLAG_COOPERATIVE)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            r = calls[name](flags=A.AAL_FLAG_COOPERATIVE)
        for _ in range(3):
            for v in r.values():
                if v is not None:
                    v.zero_()
            calls[name]()
            graph.replay()
            torch.cuda.synchronize()
            for k, v in ref.items():
                if v is not None:
                    assert torch.equal(r[k].view(torch.uint8), v.view(torch.uint8)), (name, k)
