"""Rank check at the edges of its pieces (8192 fp32 / 16384 bf16 scores; of a workgroup that takes a row 8192 to 32768), of the
rules that choose between three launches and one (rows of 384 KB and 512 rows, of 320 KB and 48, of 288 KB and 12; 1536 drafts) and between its workgroup sizes (rows of
192 KB), and of the wave's search for a draft's request (64 requests, 64 x 64 requests, runs of requests without drafts),
bit-exact against the oracle."""
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


def check(oracle, spec, q_len, V, dtype, seed):
    """Every draft's and row's outcome; some ids outside the vocabulary, q_len rows of a request (fewer than drafts + 1, none)."""
    import paper_2604_20503_amd as fsr
    rng = np.random.default_rng(seed)
    cu_q, cu_d = workloads.exclusive_offsets(q_len), workloads.exclusive_offsets(spec)
    N, D = int(cu_q[-1]), int(cu_d[-1])
    rows = (rng.integers(-40, 41, size=(8, V)) * 0.125).astype(np.float32)  # (a row may be any of eight: the draft's own score differs)
    z = rows[rng.integers(0, 8, size=N)]
    toks = rng.integers(0, V, size=D).astype(np.int32)
    toks[::37] = V
    toks[5::41] = -1
    zh = z if dtype == "f32" else workloads.f32_to_bf16_bits(z)
    rank, keep = fsr.topk_rank_check(dev(zh, dtype == "bf16"), dev(toks), dev(cu_q), dev(cu_d), K=V // 2)
    torch.cuda.synchronize()
    ref = oracle.topk_rank_check(zh, toks, cu_q, cu_d, K=V // 2, dtype=dtype)
    assert np.array_equal(rank.cpu().numpy(), ref["rank"]) and np.array_equal(keep.cpu().numpy(), ref["keep"])
    return N, D


@pytest.mark.parametrize("dtype,V,n,drafts", [
    ("f32", 98304, 128, 511), ("f32", 98303, 128, 511), ("f32", 98304, 128, 512), ("f32", 98305, 75, 300), ("f32", 100003, 16, 1),
    ("bf16", 196608, 100, 400), ("bf16", 196607, 100, 400), ("bf16", 196615, 128, 511), ("bf16", 196608, 128, 512),
    ("f32", 81920, 12, 47), ("f32", 81919, 12, 47), ("bf16", 163840, 12, 48), ("bf16", 147456, 3, 11), ("bf16", 147457, 3, 12), ("f32", 73727, 3, 11),
    ("f32", 49151, 64, 257), ("f32", 49152, 64, 257), ("bf16", 98304, 64, 256), ("bf16", 98303, 64, 255)])
def test_both_sides_of_the_launch_rules(oracle, dtype, V, n, drafts):
    announce(f"rank rules {dtype} V={V} drafts={drafts}")
    spec = np.full(n, drafts // n, np.int32)
    spec[:drafts - spec.sum()] += 1
    N, D = check(oracle, spec, spec + 1, V, dtype, V + drafts)
    assert D == drafts and N == drafts + n
    row = V * (4 if dtype == "f32" else 2) >> 10
    three = min(N, D) < (512 if row >= 384 else 48 if row >= 320 else 12 if row >= 288 else 0)
    print("three launches" if three else "one launch")


@pytest.mark.parametrize("dtype,V", [("f32", 98309), ("bf16", 98311), ("bf16", 4099)])
@pytest.mark.parametrize("n,live", [(90, 9), (190, 40), (200, 3)])
def test_drafts_far_beyond_the_live_rows(oracle, dtype, V, n, live):
    """Most requests have lost their rows to an earlier check, some keep fewer rows than drafts; 720 to 1600 drafts."""
    announce(f"rank live rows {dtype} V={V} requests={n} live={live}")
    rng = np.random.default_rng(n)
    spec = np.full(n, 8, np.int32)
    q_len = np.zeros(n, np.int32)
    q_len[rng.permutation(n)[:live]] = rng.integers(1, 10, size=live)
    assert check(oracle, spec, q_len, V, dtype, V + n)[1] == 8 * n
