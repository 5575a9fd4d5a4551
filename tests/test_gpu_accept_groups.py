"""PROBS-mode sampling at the numbers of chunks that a workgroup takes (1 to 8, by requests and vocabulary), against the oracle."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import DeviceBatch, announce, check_accept

pytestmark = pytest.mark.gpu


# chunks (whole ones and the ragged end), requests: workgroups that take one chunk, several and all of a row, and a last one with fewer
@pytest.mark.parametrize("V,B", [(3 * 4096, 300), (4 * 4096 + 1, 400), (9 * 4096 - 3, 320), (10 * 4096, 500), (38 * 4096 - 5, 250),
                                 (26 * 4096 + 7, 480), (47 * 4096, 340), (4097, 2000)])
def test_chunks_of_a_workgroup(oracle, V, B):
    import paper_2604_20503_amd as fsr
    announce(f"accept sampling groups V={V} B={B}")
    rng = np.random.default_rng(V)
    distinct = 4  # rows that differ; requests share them
    b = workloads.make_batch(2, rep=5, with_kv=False, V=V, spec_lens=[1] * distinct, ctx_lens=[8] * distinct, keep_logits=False,
                             draft_mode="noise")
    x = DeviceBatch(b, kv=False)
    pick = rng.integers(0, distinct, B)
    spec = rng.integers(0, 2, B)
    cu_t, cu_d = (workloads.exclusive_offsets(n).astype(np.int32) for n in (spec + 1, spec))
    t_rows = np.concatenate([b.cu_q[p] + np.arange(s + 1) + (1 - s) for p, s in zip(pick, spec)]).astype(np.int32)
    d_rows = np.concatenate([b.cu_d[p] + np.arange(s) for p, s in zip(pick, spec)]).astype(np.int32)
    u = rng.random(B).astype(np.float32)
    u[0], u[-1] = 0.0, np.nextafter(np.float32(1), np.float32(0))
    kw = dict(S_max=1, mode=0)
    ref = oracle.spec_accept(b.p_target, b.p_draft, b.draft_tokens, b.u_accept, u, cu_t, cu_d, t_rows=t_rows, d_rows=d_rows, **kw)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    got = fsr.spec_accept(x.p_target, x.p_draft, x.draft_tokens, x.u_accept, dev(u), dev(cu_t), dev(cu_d), t_rows=dev(t_rows),
                          d_rows=dev(d_rows), **kw)
    torch.cuda.synchronize()
    check_accept(got, ref, u)
