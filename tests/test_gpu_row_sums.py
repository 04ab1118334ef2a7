"""Rounding of the row sums, seen where they leave the library undisturbed: the
sum-exp of a slice's row records.  Each row has one dominant entry, the first,
whose term is 1, and terms that add up to 0.1: every addition on the dominant
entry's way to the row's sum rounds at the size of the sum, half a unit of
2^-23 at most and uniformly, so n of them leave a root mean square error of
2^-24 sqrt(n / 3).  In pairs n is log2 of the values of a chunk (32 bf16, 16
fp32 per thread), one more per chunk of the row, six across a wave and at most
four across the waves; one after the other it was 31 in the first chunk alone."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

BF16, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("dtype,V,rows,n", [
    (BF16, 16385, 600, 5 + 3 + 6 + 4), (BF16, 16384, 600, 5 + 2 + 6 + 4),  # 256 threads
    (BF16, 40001, 250, 5 + 5 + 6 + 4), (BF16, 40000, 250, 5 + 5 + 6 + 4),  # few long rows
    (F32, 40001, 250, 4 + 10 + 6 + 4)])
def test_sum_exp_rounds_in_pairs(dtype, V, rows, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_24150_amd as A
    g = torch.Generator(device="cuda:0").manual_seed(V + rows)
    sums = []
    for _ in range(2):
        z = (math.log(0.1 / V) + 0.5 * torch.randn(rows, V, generator=g, device="cuda:0")).to(dtype)
        z[:, 0] = 0.0
        parts = A.aal_vp_row_partials(z, z, 0, A.AAL_VP_WTV, 1.0, 1.0, V_total=V)
        torch.cuda.synchronize()
        s = parts.view(torch.float32)[:, 1].double()
        sums.append(s / z.double().exp().sum(-1) - 1)
    rms = torch.cat(sums).square().mean().sqrt().item()
    assert rms <= 2.0 ** -24 * math.sqrt(n / 3), rms * 2.0 ** 24
