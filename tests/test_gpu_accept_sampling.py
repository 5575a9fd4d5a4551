"""The rare ways through the sampling kernel, against the oracle: a residual that is zero everywhere (the token comes from
the target row), whole chunks of masked or NaN logits, a uniform of exactly zero."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import DeviceBatch, announce, check_accept, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsr():
    import paper_2604_20503_amd as f
    f.load_library()
    return f


@pytest.mark.parametrize("V", [4096, 9001, 300000])  # one chunk; unaligned rows; more chunks (74) than a wave has lanes
@pytest.mark.parametrize("mode", ["probs", "logits"])
def test_residual_that_is_zero_everywhere(fsr, oracle, V, mode):
    """Draft and target rows are equal and the drafted token has no probability: it is rejected, p - q is zero for every
    token, and the recovery token is drawn from the target row."""
    announce(f"accept zero residual {mode} V={V}")
    b = workloads.make_batch(2, rep=3, with_kv=False, V=V, spec_lens=[3, 1, 2, 4], ctx_lens=[8] * 4, keep_logits=True,
                             draft_mode="noise")
    for i in range(b.B):
        for n in range(int(b.spec_lens[i])):
            t, d = int(b.cu_q[i]) + n, int(b.cu_d[i]) + n
            x = int(b.draft_tokens[d])
            b.p_target[t, x], b.z_target[t, x] = 0.0, -np.inf
            b.p_draft[d], b.z_draft[d] = b.p_target[t], b.z_target[t]
    b.u_sample[0] = 0.0
    x = DeviceBatch(b, kv=False, logits=True)
    if mode == "probs":
        args_o, args_g, m = (b.p_target, b.p_draft), (x.p_target, x.p_draft), 0
    else:
        args_o, args_g, m = (b.z_target, b.z_draft), (x.z_target, x.z_draft), 1
    ref = oracle.spec_accept(*args_o, b.draft_tokens, b.u_accept, b.u_sample, b.cu_q, b.cu_d, S_max=b.S_max, mode=m)
    gpu = fsr.spec_accept(*args_g, x.draft_tokens, x.u_accept, x.u_sample, x.cu_q, x.cu_d, S_max=b.S_max, mode=m)
    torch.cuda.synchronize()
    assert np.array_equal(ref["accepted_len"], np.zeros(b.B, np.int32))
    check_accept(gpu, ref, b.u_sample)


@pytest.mark.parametrize("spec", [[2, 0, 3, 1], [0, 0, 0, 0]])
def test_masked_chunks_and_zero_uniforms(fsr, oracle, spec):
    """Vocabulary of three chunks: the first and half of the second are masked in every row (some by NaN), all uniforms
    are zero, so that the first token with any mass must be drawn."""
    announce(f"accept masked chunks spec={spec}")
    V = 3 * 4096
    b = workloads.make_batch(2, rep=7, with_kv=False, V=V, spec_lens=spec, ctx_lens=[8] * 4, keep_logits=True,
                             draft_mode="independent")
    for z in (b.z_target, b.z_draft):
        z[:, :4096 + 2048] = -np.inf
    b.draft_tokens[:] = 4096 + 2048 + b.draft_tokens % 2048
    b.u_sample[:] = 0.0
    ref = oracle.spec_accept(b.z_target, b.z_draft, b.draft_tokens, b.u_accept, b.u_sample, b.cu_q, b.cu_d, S_max=b.S_max, mode=1)
    for z in (b.z_target, b.z_draft):  # (the oracle would carry a NaN; a NaN logit counts as masked)
        z[:, 100:4096 + 2048:97] = np.nan
    x = DeviceBatch(b, kv=False, logits=True)
    gpu = fsr.spec_accept(x.z_target, x.z_draft, x.draft_tokens, x.u_accept, dev(b.u_sample), x.cu_q, x.cu_d, S_max=b.S_max, mode=1)
    torch.cuda.synchronize()
    check_accept(gpu, ref, b.u_sample)
