"""LOGITS-mode acceptance where exp(z / T) is formed from the logits themselves, up to |z / T| = 600 and for rows whose reference
is within 580, and on both sides of those lines: against the oracle."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import announce, check_accept, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsr():
    import paper_2604_20503_amd as f
    f.load_library()
    return f


# shift of every z / T; what happens to a third of the tokens: nothing, masked, NaN, z / T moved down by so much (values around
# the table's range of 700 and the end of fp64's at 745 below the row's reference; masks of finite, far lower values)
@pytest.mark.parametrize("T", [1.0, 0.05])
@pytest.mark.parametrize("shift", [0.0, 300.0, -300.0, 565.0, 575.0, 597.0, -575.0, -597.0, 640.0, 3000.0, -3000.0])
@pytest.mark.parametrize("third", [None, -np.inf, np.nan, -500.0, -690.0, -705.0, -742.0, -1e4])
def test_logits_within_reach_and_beyond(fsr, oracle, T, shift, third):
    announce(f"accept reach T={T} shift={shift} third={third}")
    spec, V = [3, 0, 2, 5], 8193 if shift < 0 else 4099  # whole chunks and the vocabulary's ragged end
    b = workloads.make_batch(2, rep=11, with_kv=False, V=V, spec_lens=spec, ctx_lens=[8] * 4, keep_logits=True, draft_mode="noise")
    rng = np.random.default_rng(5)
    rows = []
    for z in (b.z_target, b.z_draft):
        z = ((z.astype(np.float64) + shift) * T).astype(np.float32)
        if third is not None:
            low = rng.random(z.shape[1]) < 1 / 3
            low[b.draft_tokens] = False
            z[:, low] = z[:, low] + third * T if np.isfinite(third) else third
        rows.append(z)
    z_t, z_d = rows
    if shift == 565.0:
        b.u_sample[:] = 0.0  # the first token that has any mass
    masked = [np.where(np.isnan(z), -np.inf, z).astype(np.float32) for z in rows]  # what a NaN logit counts as
    ref = oracle.spec_accept(*masked, b.draft_tokens, b.u_accept, b.u_sample, b.cu_q, b.cu_d, S_max=b.S_max, mode=1, temperature=T)
    gpu = fsr.spec_accept(dev(z_t), dev(z_d), dev(b.draft_tokens), dev(b.u_accept), dev(b.u_sample), dev(b.cu_q), dev(b.cu_d),
                          S_max=b.S_max, mode=1, temperature=T)
    torch.cuda.synchronize()
    check_accept(gpu, ref, b.u_sample)
