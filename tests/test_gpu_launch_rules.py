"""The rules by which the library picks a launch shape or a kernel from sizes, types and alignment, at the sizes where each
rule turns, against the CPU oracle.  Tolerances are parity_util's."""
import pytest
import torch

from paper_2511_02017_amd import binding
from tests import parity_util as pu
from tests.test_gpu_parity import random_arms, random_round

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def mixed_round(B, K, V, dt, tt, seed, **kw):
    rnd = random_round(B, K, V, torch.float32 if dt == tt == torch.float32 else torch.bfloat16, seed=seed, **kw)
    rnd["draft"], rnd["target"] = rnd["draft"].to(dt), rnd["target"].to(tt)
    return rnd


f32, bf16 = torch.float32, torch.bfloat16


@pytest.mark.parametrize("B,K,V,dt,tt", [
    (3, 2, 8192, bf16, bf16),        # one batch of 16 KB exactly: one slice
    (3, 2, 8193, bf16, bf16),        # one element more: two slices, rows at every alignment
    (2, 3, 8199, bf16, f32),         # three and a bit batches of binary32 rows beside one and a bit of bfloat16 rows
    (2, 3, 4096, f32, f32),
    (2, 3, 4101, f32, bf16),
    (1, 8, 131072, bf16, bf16),      # sixteen batches: as many slices as are merged across lanes
    (1, 8, 131080, bf16, bf16),      # one vector more: two batches per slice
    (1, 31, 70001, bf16, bf16),      # 32 target rows of nine slices in groups of sixteen lanes: the largest such shape
    (1, 32, 70001, bf16, bf16),      # 33 target rows: groups of eight lanes
    (1, 64, 40003, f32, f32),        # 65 target rows: the staged merge, as many slices as there are batches
    (300, 2, 12289, bf16, bf16),     # 1500 rows of both tensors together: a batch and a half
])
def test_slices_of_whole_batches(B, K, V, dt, tt):
    rnd = mixed_round(B, K, V, dt, tt, seed=V + K)
    tp = binding.Tapout(B, K, V)
    arm = random_arms(B, seed=K)
    c = [pu.check_round(tp, rnd), pu.check_round(tp, rnd, arm=arm),
         pu.check_round_call(tp, rnd, arm.clone(), truncate=False), pu.check_round_call(tp, rnd, arm.clone(), truncate=True)]
    # near ties: a few per thousand decisions at the tolerance of 1e-5
    assert sum(x["accept_flagged"] + x["icdf_flagged"] + x["stop_flagged"] for x in c) <= 2 + 4 * B * K // 500
