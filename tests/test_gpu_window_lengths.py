"""The register-resident schedules at window lengths 9 to 15 (one vector per
row and thread; at 10 and above part of a window is not staged in LDS),
against the fp64 oracle with the tolerances of the entry points' own parity
tests: several windows per team, teams of several members with a ragged last
one, sequences whose last chunk is short."""
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
    # WTV: 3 (bf16) or 5 (fp32) members per team, the last one ragged; 85 or 51 teams
    zd, zt = parity_cases._inputs("c1" if dtype == F32 else "c2", (100, K, 8808), dtype, seed=K, dev=dev)
    parity_cases._check_wtv(A, zd, zt, 0.9, 1.1, gdtype, 0)
    # EAL: 6 or 12 members (shorter rows take the streaming schedule); 42 or 21 teams.
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
