"""Rank check at the edges of its pieces (8192 fp32 / 16384 bf16 scores; per workgroup size 4096 to 32768), of the workgroup
sizes (512, 1024 drafts), of the rule that cuts rows into pieces (256 to 512 drafts, 96 MiB) and of the wave's search for a draft's request
(64 requests, 64 x 64 requests, runs of requests without drafts), bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import announce, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,V", [(1, 8192), (64, 8199), (65, 16384), (300, 16391), (4097, 33), (512, 4096), (700, 2051), (1024, 2047),
                                 (330, 100003)])
def test_pieces_and_search(oracle, B, V, dtype):
    import paper_2604_20503_amd as fsr
    announce(f"rank pieces B={B} V={V} {dtype}")
    rng = np.random.default_rng(B + V)
    spec = rng.integers(0, 3, size=B).astype(np.int32)
    spec[B // 3:B // 2] = 0
    spec[-1] = 2
    cu_q, cu_d = workloads.exclusive_offsets(spec + 1), workloads.exclusive_offsets(spec)
    z = (rng.integers(-40, 41, size=(int(cu_q[-1]), V)) * 0.125).astype(np.float32)
    toks = rng.integers(0, V, size=int(cu_d[-1])).astype(np.int32)
    zh = z if dtype == "f32" else workloads.f32_to_bf16_bits(z)
    rank, keep = fsr.topk_rank_check(dev(zh, dtype == "bf16"), dev(toks), dev(cu_q), dev(cu_d), K=100)
    torch.cuda.synchronize()
    ref = oracle.topk_rank_check(zh, toks, cu_q, cu_d, K=100, dtype=dtype)
    assert np.array_equal(rank.cpu().numpy(), ref["rank"]) and np.array_equal(keep.cpu().numpy(), ref["keep"])
