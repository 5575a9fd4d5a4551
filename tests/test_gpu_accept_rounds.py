"""LOGITS-mode acceptance of few requests with many drafts, against the oracle: drafts tested in rounds of twelve waves or by a
lane each, rejections at the edges of the rounds, with and without a bonus row, rows of more than 64 chunks."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import announce, check_accept, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V,S,rejections", [
    (131072, 11, [0, 11, 5]), (131072, 12, [11, 0, 12]), (131072, 13, [12, 11, 13]),  # one and two rounds of rows of 32 pairs
    (131072, 24, [12, 23, 24]), (131072, 25, [24, 0, 25]), (131072, 40, [35, 36, 39]),
    (20001, 11, [11, 3, 0]), (20001, 12, [11, 12, 0]), (20001, 25, [12, 24, 25]), (20001, 70, [63, 64, 69]),  # 5 pairs
    (4096, 11, [0, 10, 11]), (4096, 13, [0, 12, 13]), (270001, 3, [0, 2, 1])])
def test_rounds_of_drafts(oracle, V, S, rejections, dtype):
    """Every draft's rows are equal, so that it is accepted, but for the request's rejected one, whose token is e^-6 as likely to
    the target; a rejection at S is none.  Odd requests have no bonus row."""
    import paper_2604_20503_amd as fsr
    announce(f"accept rounds V={V} S={S} {dtype}")
    rng = np.random.default_rng(V + S)
    B = len(rejections) + 1
    d_len = np.full(B, S)
    d_len[-1] = max(0, S - 2)
    t_len = d_len + 1 - np.arange(B) % 2
    cu_t, cu_d = workloads.exclusive_offsets(t_len), workloads.exclusive_offsets(d_len)
    z_t = rng.standard_normal((int(cu_t[-1]), V), dtype=np.float32) * 2
    z_d = np.empty((int(cu_d[-1]), V), np.float32)
    toks = rng.integers(0, V, size=len(z_d)).astype(np.int32)
    u_a, u_s = rng.uniform(0.05, 0.95, len(z_d)).astype(np.float32), rng.random(B, dtype=np.float32)
    for i in range(B):
        z_d[cu_d[i]:cu_d[i + 1]] = z_t[cu_t[i]:cu_t[i] + d_len[i]]
        if i < len(rejections) and rejections[i] < S:
            z_t[cu_t[i] + rejections[i], toks[cu_d[i] + rejections[i]]] -= 6.0
    if dtype == "bf16":
        z_t, z_d = workloads.f32_to_bf16_bits(z_t), workloads.f32_to_bf16_bits(z_d)
    t, d = dev(z_t, dtype == "bf16"), dev(z_d, dtype == "bf16")
    if dtype == "bf16":
        z_t, z_d = t.float().cpu().numpy(), d.float().cpu().numpy()
    ref = oracle.spec_accept(z_t, z_d, toks, u_a, u_s, cu_t, cu_d, S_max=S, mode=1, temperature=0.9)
    assert ref["accepted_len"].tolist() == rejections + [int(d_len[-1])]
    got = fsr.spec_accept(t, d, dev(toks), dev(u_a), dev(u_s), dev(cu_t), dev(cu_d), S_max=S, mode=1, temperature=0.9)
    torch.cuda.synchronize()
    assert check_accept(got, ref, u_s)[1] == 0
