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


# one chunk; unaligned rows; more chunks (74) than a wave has lanes; several chunks a workgroup
@pytest.mark.parametrize("V,B", [(4096, 4), (9001, 4), (300000, 4), (8196, 1024)])
@pytest.mark.parametrize("mode", ["probs", "logits"])
def test_residual_that_is_zero_everywhere(fsr, oracle, V, B, mode):
    """Draft and target rows are equal and the drafted token has no probability: it is rejected, p - q is zero for every
    token, and the recovery token is drawn from the target row (whose masses every workgroup leaves for this)."""
    announce(f"accept zero residual {mode} V={V} B={B}")
    b = workloads.make_batch(2, rep=3, with_kv=False, V=V, spec_lens=[3, 1, 2, 4] if B == 4 else [1] * B, ctx_lens=[8] * B,
                             keep_logits=True, draft_mode="noise")
    for i in range(b.B):
        for n in range(int(b.spec_lens[i])):
            t, d = int(b.cu_q[i]) + n, int(b.cu_d[i]) + n
            x = int(b.draft_tokens[d])
            b.p_target[t, x], b.z_target[t, x] = 0.0, -np.inf
            if B > 4:  # masked tokens in some of the rows, whole chunks of them in a few
                lo, step = (0, 1) if d % 8 == 0 else (d % 4096, 3)
                b.p_target[t, lo:5000:step], b.z_target[t, lo:5000:step] = 0.0, -np.inf
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


def test_a_chunk_with_mass_holds_a_token_with_mass(fsr):
    """Draft logits = target logits + a constant: the distributions are equal, and what p - q leaves is rounding.  Rejected
    (the drafted token is masked), such a request must still draw a token that has a probability.  All of them are in the
    second chunk, which holds two values of logits only, so that its rounding errors are few and may all be negative."""
    announce("accept residual of rounding errors")
    B, V = 512, 8192
    rng = np.random.default_rng(17)
    z = np.full((2 * B, V), -np.inf, np.float32)  # rows 2 i: verifies the draft, 2 i + 1: bonus
    grid = lambda lo, hi, n: rng.integers(int(lo * 1024), int(hi * 1024), n) / 1024.0  # noqa: E731  (sums are exact in fp32)
    top, gap, shift = grid(-4, 4, B), grid(1, 30, B), grid(-3, 3, B)
    z[0::2, 4096:] = (top - gap)[:, None]
    z[np.arange(0, 2 * B, 2), 4096 + rng.integers(0, 4096, B)] = top
    z[1::2, 4096:] = 0.0
    q = z[0::2] + shift[:, None].astype(np.float32)
    tok = rng.integers(0, 4096, B).astype(np.int32)
    u = rng.random(B).astype(np.float32)
    acc, n, em = fsr.spec_accept(dev(z), dev(q), dev(tok), dev(u), dev(u), dev(np.arange(0, 2 * B + 1, 2, dtype=np.int32)),
                                 dev(np.arange(B + 1, dtype=np.int32)), S_max=1, mode=1, temperature=0.7)
    torch.cuda.synchronize()
    assert not acc.any() and (n == 1).all()
    bad = (em[:, 0] < 4096).nonzero()[:, 0].tolist()
    assert not bad, f"{len(bad)} requests drew a masked token, e.g. {bad[:5]}"


@pytest.mark.parametrize("kind", ["top-50", "lowest", "far", "one"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_masked_and_far_spread_rows(fsr, oracle, kind, dtype):
    """The ways through a whole chunk: most logits masked with -inf or with the type's lowest value, exponents from 0 to -900
    (some in fp64's last range, where the table ends), a single masked token."""
    announce(f"accept masked {kind} {dtype}")
    V = 4 * 4096 + 100
    b = workloads.make_batch(2, rep=9, with_kv=False, V=V, spec_lens=[3, 1, 0, 4, 2, 5], ctx_lens=[8] * 6, keep_logits=True,
                             draft_mode="independent")
    T = 0.01 if kind == "far" else 0.9
    for z in (b.z_target, b.z_draft):
        if kind in ("top-50", "lowest"):
            z[z < np.sort(z, axis=1)[:, -50][:, None]] = -np.inf if kind == "top-50" else np.finfo(np.float32).min
        if kind == "one":
            z[:, 5000] = -np.inf
    up = lambda a: torch.from_numpy(a).to(dtype)  # noqa: E731
    zt, zd = up(b.z_target), up(b.z_draft)
    b.u_sample[::2] = 0.0
    ref = oracle.spec_accept(zt.float().numpy(), zd.float().numpy(), b.draft_tokens, b.u_accept, b.u_sample, b.cu_q, b.cu_d,
                             S_max=b.S_max, mode=1, temperature=T)
    gpu = fsr.spec_accept(zt.cuda(), zd.cuda(), dev(b.draft_tokens), dev(b.u_accept), dev(b.u_sample), dev(b.cu_q), dev(b.cu_d),
                          S_max=b.S_max, mode=1, temperature=T)
    torch.cuda.synchronize()
    check_accept(gpu, ref, b.u_sample)
