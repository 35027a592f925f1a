"""GPU parity of the k-means steps at the sizes where their launch shapes and tiles change."""
import numpy as np
import pytest
import torch

from oracle import wave_oracle as wo
from paper_2505_02922_amd import binding as wb
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def _unit_rows(g, n, d, dtype):
    x = g.standard_normal((n, d))
    return wo.quant(x / np.linalg.norm(x, axis=1, keepdims=True), dtype)


# (256 f32 rows of 128 channels are the most that stay resident in LDS, 512 bf16 rows likewise;
# one more centroid than a multiple of 32 leaves a tile with one row; 33 points leave a fragment
# with one point; 40000 points take more than one fragment per wave)
@pytest.mark.parametrize("dtype,d,L,k", [
    ("f32", 128, 1000, 256), ("f32", 128, 1000, 289), ("f32", 128, 33, 33), ("f32", 64, 4097, 129),
    ("f32", 64, 1, 1), ("f32", 64, 700, 600), ("bf16", 128, 2049, 512), ("bf16", 128, 1100, 545),
    ("bf16", 64, 65, 31), ("bf16", 64, 40000, 97)])
def test_assign_step_tile_edges(dtype, d, L, k):
    g = np.random.default_rng(L * 1000 + k)
    xhat, chat = _unit_rows(g, L, d, dtype), _unit_rows(g, k, d, dtype)
    chat[k // 2:k // 2 + 2] = chat[0]          # exact ties: the lowest id wins
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    a = wb.wave_kmeans_assign_step(torch.from_numpy(xhat).to(tdt).cuda(), torch.from_numpy(chat).to(tdt).cuda())
    torch.cuda.synchronize()
    pu.check_assign(a.cpu().numpy(), xhat, chat, f"{dtype} d={d} L={L} k={k}")
