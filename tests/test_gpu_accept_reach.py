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


# Temperatures at which 600 of them are no normal float.  Small ones: a certain token (log-probabilities, the largest logit is
# 0) drafted by a row whose largest logit is 1; large ones: every token alike, half of them masked in the draft's row, and a
# uniform that is decided by how many.  Powers of two, whose products with 1 / T are exact, or whole numbers: of 1e17 and more a
# quotient's rounding is whole units of the exponent.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("powers", [True, False])
@pytest.mark.parametrize("T", [1e-300, 1e-60, 1e-50, 1e-44, 1.9e-41, 2.1e-41, 1e-30, 1e30, 5e35, 6e35, 1e38, 3e38, 1e45, 1e300])
def test_extreme_temperatures(fsr, oracle, T, powers, dtype):
    announce(f"accept extreme temperature T={T} powers={powers} {dtype}")
    rng = np.random.default_rng(3)
    spec, V = np.array([1, 2, 0, 3]), 8197
    cu_t, cu_d = (np.concatenate([[0], np.cumsum(n)]).astype(np.int32) for n in (spec + 1, spec))
    x = rng.integers(0, V, cu_d[-1]).astype(np.int32)
    low = (lambda n: -(2.0 ** rng.integers(0, 5, (n, V)))) if powers else (lambda n: -rng.integers(1, 10, (n, V)))
    z_t, z_d = low(cu_t[-1]).astype(np.float32), low(cu_d[-1]).astype(np.float32)
    if T < 1:
        z_t[np.arange(len(z_t)), rng.integers(0, V, len(z_t))] = 0.0 if powers else -0.75
        for i in range(len(spec)):
            for j in range(spec[i]):
                z_t[cu_t[i] + j] = np.minimum(z_t[cu_t[i] + j], -1.0)
                z_t[cu_t[i] + j, x[cu_d[i] + j]] = 0.0 if powers else -0.75  # (three quarters: its quotient is rounded too)
                z_d[cu_d[i] + j, x[cu_d[i] + j]] = 1.0 if powers else 3.0
        u_a = np.full(cu_d[-1], 0.5, np.float32)
    else:
        drop = rng.random(z_d.shape) < 0.5
        drop[np.arange(len(x)), x] = False
        z_d[drop] = -np.inf
        # p = 1 / V against q = 1 / (tokens left): the quotient, less and more 0.5 %
        u_a = ((~drop).sum(axis=1) / V * np.where(np.arange(len(x)) % 3 == 2, 1.005, 0.995)).astype(np.float32)
    u_s = rng.random(len(spec)).astype(np.float32)
    ref = oracle.spec_accept(z_t, z_d, x, u_a, u_s, cu_t, cu_d, S_max=3, mode=1, temperature=T)
    as_dtype = (lambda z: dev(z).bfloat16()) if dtype == "bf16" else dev  # exact
    gpu = fsr.spec_accept(as_dtype(z_t), as_dtype(z_d), dev(x), dev(u_a), dev(u_s), dev(cu_t), dev(cu_d), S_max=3, mode=1, temperature=T)
    torch.cuda.synchronize()
    check_accept(gpu, ref, u_s)


# Requests and drafts that give a workgroup several chunks: of the statistics 8, 4 and 2 (the first and last leave rows behind a
# rejection out), of the draw 8, 8 and 2.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,S,nc", [(520, 3, 9), (512, 1, 10), (256, 4, 5)])
@pytest.mark.parametrize("T", [1.0, 0.004])
@pytest.mark.parametrize("level", [0.0, -590.0, 900.0, 2e6])
def test_chunks_at_different_levels(fsr, oracle, T, level, B, S, nc, dtype):
    """Rows whose chunks lie apart: beside each other some whose logits are taken as they are, some that are masked (-inf, NaN, a finite
    number), some that are far above, far below or between, and a ragged last one."""
    announce(f"accept levels T={T} level={level} B={B} S={S} nc={nc} {dtype}")
    rng = np.random.default_rng(nc + B)
    V, D = nc * 4096 - 1003, 12  # distinct pairs of rows; requests share them
    # of a chunk, below the row's level, in z / T.  (bf16 has 8 bits, a level of 2e6 in fp32 a grid of 1/8)
    steps = [0.0, -3.0, -30.0, -480.0, -560.0, -640.0, -693.0, -703.0, -712.0, -2e4, -1e30, -np.inf, np.nan]
    z_t, z_d = np.empty((D, V), np.float32), np.empty((D, V), np.float32)
    x = np.empty(D, np.int32)
    for j in range(D):
        at = rng.choice(len(steps), nc)
        at[rng.integers(nc)] = 0
        if j % 3 == 2:
            at[:] = np.where(at > 1, len(steps) - 2, at)  # all others masked
        base = level + np.array(steps)[at] if j % 2 == 0 else np.array(steps)[at]
        for c in range(nc):
            e = slice(c * 4096, min(V, (c + 1) * 4096))
            n = e.stop - e.start
            z = base[c] + rng.normal(0, 2.0, n)
            with np.errstate(invalid="ignore"):
                z_t[j, e] = z * T
                z_d[j, e] = (z + rng.normal(0, 0.5, n)) * T
                if j % 4 == 3:
                    z_d[j, e] += np.float32(300 * T)  # another reference for the draft's row
        finite = np.where(np.isfinite(z_t[j]), z_t[j], -np.inf)
        x[j] = rng.choice(np.argsort(finite)[-6:])
    if dtype == "bf16":
        z_t, z_d = (torch.from_numpy(z).bfloat16().float().numpy() for z in (z_t, z_d))
    spec = rng.integers(0, S + 1, B)
    cu_t, cu_d = (np.concatenate([[0], np.cumsum(n)]).astype(np.int32) for n in (spec + 1, spec))
    t_rows, d_rows = rng.integers(0, D, cu_t[-1]).astype(np.int32), np.empty(cu_d[-1], np.int32)
    for i in range(B):
        d_rows[cu_d[i]:cu_d[i + 1]] = t_rows[cu_t[i]:cu_t[i + 1] - 1]
    u_a, u_s = (rng.random(n).astype(np.float32) for n in (D, B))
    u_s[::7] = 0.0
    masked = [np.where(np.isnan(z), -np.inf, z).astype(np.float32) for z in (z_t, z_d)]
    ref = oracle.spec_accept(*masked, x, u_a, u_s, cu_t, cu_d, S_max=S, t_rows=t_rows, d_rows=d_rows, mode=1, temperature=T)
    as_dtype = (lambda z: dev(z).bfloat16()) if dtype == "bf16" else dev  # exact
    gpu = fsr.spec_accept(as_dtype(z_t), as_dtype(z_d), dev(x), dev(u_a), dev(u_s), dev(cu_t), dev(cu_d), S_max=S,
                          t_rows=dev(t_rows), d_rows=dev(d_rows), mode=1, temperature=T)
    torch.cuda.synchronize()
    check_accept(gpu, ref, u_s)


# A NaN that is quiet, or signalling as bits read from anywhere can be, in front of and behind the row's largest logit.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bits", [0x7FC0, 0x7F81, 0xFFA0])
@pytest.mark.parametrize("level", [0.0, 900.0, -900.0])
@pytest.mark.parametrize("at", [2 * 256 * 4 + 2, 8192 + 507])  # of a whole chunk, of the ragged one
def test_a_nan_beside_the_largest_logit(fsr, oracle, at, level, bits, dtype):
    announce(f"accept nan {bits:x} beside {at} level={level} {dtype}")
    rng = np.random.default_rng(at)
    spec, V = np.array([1, 3, 0, 2]), 9001
    cu_t, cu_d = (np.concatenate([[0], np.cumsum(n)]).astype(np.int32) for n in (spec + 1, spec))
    z_t, z_d = (np.round(level + rng.normal(0, 2, (n, V)) * 4).astype(np.float32) / 4 for n in (cu_t[-1], cu_d[-1]))
    x = rng.integers(0, V, cu_d[-1]).astype(np.int32)
    x[::2] = at
    for z in (z_t, z_d):
        z[:] = torch.from_numpy(z).bfloat16().float().numpy()
        z[:, at] = level + 650.0 if level == 0.0 else level + 40.0
        z[:, at] = torch.from_numpy(z[:, at]).bfloat16().float().numpy()
        z[:, at ^ 1] = -np.inf  # what a NaN logit counts as
    x[x == at ^ 1] = at
    u_a, u_s = (rng.random(n).astype(np.float32) for n in (cu_d[-1], len(spec)))
    ref = oracle.spec_accept(z_t, z_d, x, u_a, u_s, cu_t, cu_d, S_max=3, mode=1)
    tensors = []
    for z in (z_t, z_d):
        b = z.view(np.uint32).copy()
        b[:, at ^ 1] = np.uint32(bits << 16)
        tensors.append(dev((b >> 16).astype(np.uint16), True) if dtype == "bf16" else dev(b.view(np.int32)).view(torch.float32))
    gpu = fsr.spec_accept(*tensors, dev(x), dev(u_a), dev(u_s), dev(cu_t), dev(cu_d), S_max=3, mode=1)
    torch.cuda.synchronize()
    check_accept(gpu, ref, u_s)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [1.0, 1e-30, 1e-300])
@pytest.mark.parametrize("nothing", [-np.inf, np.nan, np.inf])
def test_rows_without_any_mass(fsr, oracle, nothing, T, dtype):
    """Target and draft rows that are masked throughout: they accept nothing, and a draw from one has no token to give but the first."""
    announce(f"accept rows of {nothing} T={T} {dtype}")
    rng = np.random.default_rng(1)
    spec, V = np.array([2, 2, 1, 2, 1, 0]), 9001
    cu_t, cu_d = (np.concatenate([[0], np.cumsum(n)]).astype(np.int32) for n in (spec + 1, spec))
    z_t, z_d = (rng.integers(-8, 8, (n, V)).astype(np.float32) * np.float32(2.0 ** round(np.log2(max(T, 1e-30)))) for n in (cu_t[-1], cu_d[-1]))
    x = rng.integers(0, V, cu_d[-1]).astype(np.int32)
    for i in range(len(spec)):
        for j in range(spec[i]):
            z_t[cu_t[i] + j, x[cu_d[i] + j]] = 16 * np.abs(z_t).max()
    for row in (cu_t[0], cu_t[2] + 1, cu_t[3] + 1, cu_t[5]):
        z_t[row] = nothing
    z_d[cu_d[3] + 1] = nothing
    u_a, u_s = np.full(cu_d[-1], 0.01, np.float32), np.linspace(0, 0.99, len(spec)).astype(np.float32)
    masked = [np.where(np.isnan(z), -np.inf, z).astype(np.float32) for z in (z_t, z_d)]
    with np.errstate(all="ignore"):
        ref = oracle.spec_accept(*masked, x, u_a, u_s, cu_t, cu_d, S_max=2, mode=1, temperature=T)
    as_dtype = (lambda z: dev(z).bfloat16()) if dtype == "bf16" else dev  # exact
    acc, nem, em = (t.cpu().numpy() for t in fsr.spec_accept(as_dtype(z_t), as_dtype(z_d), dev(x), dev(u_a), dev(u_s), dev(cu_t), dev(cu_d),
                                                             S_max=2, mode=1, temperature=T))
    assert np.array_equal(acc, ref["accepted_len"]) and np.array_equal(acc, [0, 2, 1, 1, 1, 0])
    assert np.array_equal(nem, acc + 1)
    for i in range(len(spec)):
        want = list(ref["emitted"][i][:acc[i] + (i in (1, 4))]) + ([0] if i not in (1, 4) else [])  # (the oracle gives no token at all)
        assert list(em[i]) == want + [-1] * (3 - len(want)), i
