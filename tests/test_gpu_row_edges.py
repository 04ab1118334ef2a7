"""Rows that start and end inside 16-byte vectors, and every shape that the
workgroup-per-row kernels are launched in, against the fp64 oracle with the
tolerances of the entry points' own parity tests.

The sizes put a row's edges everywhere they can fall: rows shorter than a
vector, rows whose first and last vectors are the same, a last row that ends
the allocation inside a vector; and rows and lengths on both sides of each
limit at which a pass takes other workgroups."""
import pytest
import torch

import test_gpu_general as general
import test_gpu_grpo as grpo
import test_gpu_parity as parity_cases
import test_gpu_vp as vp

pytestmark = pytest.mark.gpu

BF16, F32 = torch.bfloat16, torch.float32
SHAPES = [(3, 3, 5), (9, 2, 3), (17, 1, 2), (8193, 3, 2), (8200, 2, 2), (20003, 5, 1), (8197, 1, 513),
          (1023, 2, 3), (1024, 2, 3), (2047, 2, 3), (2048, 2, 3), (4095, 2, 3), (4096, 2, 3),
          # arrays that end 1, 3 and 4 elements into a vector (and 2, 5, 6, 7 above), arrays shorter than one
          (5, 1, 5), (11, 3, 3), (3, 1, 4), (3, 1, 2), (1, 1, 3),
          # either side of the row shapes' limits in vectors (64, 128, 256, 512, 1024, 2048, 4096) and rows
          (511, 3, 3), (513, 2, 3), (2049, 5, 210), (4095, 5, 210), (8201, 1, 257), (16400, 1, 257),
          (32777, 1, 4)]  # V, K, N


@pytest.fixture(scope="module")
def A():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_24150_amd as lib
    return lib


@pytest.mark.parametrize("dtype,gdtype", [(BF16, BF16), (BF16, F32), (F32, F32)])
@pytest.mark.parametrize("V,K,N", SHAPES)
def test_losses(A, V, K, N, dtype, gdtype):
    dev = torch.device("cuda:0")
    zd, zt = parity_cases._inputs("c2", (N, K, V), dtype, seed=V + K, dev=dev)
    parity_cases._check_eal(A, zd, zt, 0.9, gdtype, A.AAL_FLAG_STREAMING)
    parity_cases._check_wtv(A, zd, zt, 0.9, 1.1, gdtype, A.AAL_FLAG_STREAMING)
    general._check(A, zd, zt, K, (0.7, 0.4, 1.3, 0.9), general.WIN, gdt=gdtype, flags=A.AAL_FLAG_STREAMING)
    first = 2 * (V // 5)
    vp.check_eal(A, zd, zt, [first, V - first] if first else [V], 0.9, gdtype)
    vp.check_wtv(A, zd, zt, [first, V - first] if first else [V], 0.9, 1.1, gdtype)


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("V,K,N", SHAPES)
def test_simulation_and_grpo(A, V, K, N, dtype):
    from paper_2609_24150_amd.inputs import make_uniforms
    dev = torch.device("cuda:0")
    zd, zt = parity_cases._inputs("c5", (N, 2, K, V), dtype, seed=V + K, dev=dev)
    u1, u2 = make_uniforms((N, 2, K), seed=V, device="cpu")
    parity_cases._check_sim(A, zd, zt, u1.to(dev), u2.to(dev), 1.0)
    zth, zrf, zt = grpo._inputs((N, 2 * K, V), dtype, seed=V + K)
    grpo._check(A, zth, zrf, zt, 2, K, grpo.WIN, T=0.9)
