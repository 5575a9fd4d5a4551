"""GPU parity of bf16 attention over heads of 64 whose items are cut by their lengths (more items than half the compute units, at
most one and a half times as many): against the oracle, with and without scratch memory, and in graph replays over other lengths."""
import numpy as np
import pytest
import torch

from gpu_utils import announce, check_attention, dev
from test_gpu_attention_items import make

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsr():
    import paper_2604_20503_amd as f
    f.load_library()
    return f


def lengths(kind, B, rng):
    if kind == "equal":
        return np.full(B, 1600), np.full(B, 2)
    if kind == "one long":
        ctx = rng.integers(0, 70, B)
        ctx[B // 2] = 3000
        return ctx, rng.integers(0, 4, B)
    return rng.integers(0, 1700, B), rng.integers(0, 4, B)


# items per call; one, two and three query tiles; in two of the ragged calls a request has rows beyond the bound that is given
@pytest.mark.parametrize("H_q,H_kv,B,hint,token_major,P", [(16, 16, 9, 4, False, 16), (8, 4, 64, 4, True, 16), (64, 8, 17, 4, False, 24),
                                                           (48, 4, 40, 4, False, 16), (32, 8, 48, 2, True, 16), (24, 6, 30, 1, False, 16)])
@pytest.mark.parametrize("kind", ["ragged", "one long", "equal"])
def test_items_balanced_by_length(fsr, oracle, H_q, H_kv, B, hint, token_major, P, kind):
    announce(f"balanced items {H_q}/{H_kv} B={B} hint={hint} token_major={token_major} P={P} {kind}")
    rng = np.random.Generator(np.random.PCG64(B + H_q))
    ctx, spec = lengths(kind, B, rng)
    if kind != "equal":
        ctx[0] = 1690  # the block tables are wide enough for pieces
        ctx[B // 3 + 1] = 100
    x = make(rng, "bf16", H_q, H_kv, 64, P, ctx, spec)
    if kind == "ragged":
        x["cu"][B // 3 + 1] = x["cu"][B // 3]  # a request without rows; the one behind it has its rows as well,
        x["ctx"][B // 3 + 1] = 90              # on the pages it has
    scale = 1.0 / 8.0
    swap = (lambda t: np.ascontiguousarray(np.swapaxes(t, 1, 2))) if token_major else (lambda t: t)
    q, k, v = dev(x["q"], True), dev(swap(x["k"]), True), dev(swap(x["v"]), True)
    ref, lse_ref = oracle.verify_attention(x["q"], x["k"], x["v"], x["bt"], x["ctx"], x["cu"], H_q=H_q, H_kv=H_kv, D=64, P=P,
                                           dtype="bf16", scale=float(np.float32(scale)))
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
    for ws in (None, None, torch.empty(256, dtype=torch.uint8, device="cuda")):  # the second call finds the first one's counts
        out.fill_(float("nan"))
        fsr.verify_attention(q, k, v, dev(x["bt"]), dev(x["ctx"]), None, dev(x["cu"]), scale=scale, out=out, lse=lse,
                             max_q_len=hint, workspace=ws, kv_layout=1 if token_major else 0)
        torch.cuda.synchronize()
        check_attention(out, ref, "f32", len(ref))
        np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)


def test_balanced_items_in_a_graph(fsr):
    """Replays over contexts that change, with eager calls on the same workspace between them: the bits of an eager call on a
    workspace of its own."""
    announce("balanced items in a graph")
    rng = np.random.Generator(np.random.PCG64(2))
    B = 20
    x = make(rng, "bf16", 32, 8, 64, 16, rng.integers(1000, 1700, B), rng.integers(0, 4, B))
    q, k, v, bt, cu = dev(x["q"], True), dev(x["k"], True), dev(x["v"], True), dev(x["bt"]), dev(x["cu"])
    need = fsr.attn_workspace_bytes(B=B, N_cap=q.shape[0], H_q=32, H_kv=8, D=64, P=16, max_pages=bt.shape[1], n_pages=k.shape[0],
                                    dtype=torch.bfloat16, out_dtype=torch.bfloat16, max_q_len=4)
    ws, own = (torch.full((need,), 0x55, dtype=torch.uint8, device="cuda") for _ in range(2))
    c, out, want = dev(x["ctx"]), torch.empty_like(q), torch.empty_like(q)

    def call(ctx, into, workspace):
        fsr.verify_attention(q, k, v, bt, ctx, None, cu, scale=0.125, out=into, max_q_len=4, workspace=workspace)

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call(c, out, ws)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            call(c, out, ws)
        for rep in range(4):
            c.copy_(dev(np.minimum(x["ctx"], rng.integers(0, 1700, B)).astype(np.int32)))
            out.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            call(c, want, own)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), want.view(torch.int16))
            call(c, out, ws)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("H_q,H_kv,B,hint", [(12, 3, 60, 2), (20, 5, 41, 4), (28, 7, 37, 3), (35, 7, 25, 9), (32, 8, 32, 2)])
def test_rows_beyond_the_bound_beside_others(fsr, oracle, H_q, H_kv, B, hint):
    """Requests, short and long, with more rows than the bound allows (up to five rounds of 16 to 48 query rows), in workgroups that
    they share with requests of one round (where the KV heads are an odd number) and with other heads of their own."""
    announce(f"balanced items, rows beyond the bound {H_q}/{H_kv} B={B} hint={hint}")
    rng = np.random.Generator(np.random.PCG64(7 * B + hint))
    ctx, spec = rng.integers(0, 1700, B), rng.integers(0, hint, B)
    ctx[0] = 1690
    over = rng.permutation(B)[:B // 3]
    spec[over] = rng.integers(hint + 2, 5 * hint + 4, len(over))
    ctx[over[::2]] = rng.integers(0, 100, len(over[::2]))
    x = make(rng, "bf16", H_q, H_kv, 64, 16, ctx, spec)
    scale = 1.0 / 8.0
    ref, lse_ref = oracle.verify_attention(x["q"], x["k"], x["v"], x["bt"], x["ctx"], x["cu"], H_q=H_q, H_kv=H_kv, D=64, P=16,
                                           dtype="bf16", scale=float(np.float32(scale)))
    q = dev(x["q"], True)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
    fsr.verify_attention(q, dev(x["k"], True), dev(x["v"], True), dev(x["bt"]), dev(x["ctx"]), None, dev(x["cu"]), scale=scale, out=out,
                         lse=lse, max_q_len=hint)
    torch.cuda.synchronize()
    check_attention(out, ref, "f32", len(ref))
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("H_q,H_kv,B,hint,ctx_hi", [(32, 8, 32, 4, 300), (28, 7, 36, 4, 90), (12, 3, 61, 3, 700), (64, 8, 17, 4, 1), (32, 8, 32, 2, 256)])
def test_short_contexts_in_wide_tables(fsr, oracle, H_q, H_kv, B, hint, ctx_hi):
    """Little to gain by cutting: an item to a workgroup, requests without rows and (the last call) rows beyond the bound among them."""
    announce(f"short contexts in wide tables {H_q}/{H_kv} B={B} hint={hint} ctx_hi={ctx_hi}")
    rng = np.random.Generator(np.random.PCG64(B + ctx_hi))
    spec = rng.integers(0, hint, B)
    if hint == 2:
        spec[rng.permutation(B)[:9]] = rng.integers(3, 12, 9)
    x = make(rng, "bf16", H_q, H_kv, 64, 16, rng.integers(0, ctx_hi + 1, B), spec)
    x["bt"] = np.ascontiguousarray(np.pad(x["bt"], ((0, 0), (0, 200 - x["bt"].shape[1])), constant_values=-1))
    x["cu"][5] = x["cu"][4]  # no rows; the request behind it has them as well, on the pages it has
    x["ctx"][5] = 0
    scale = 1.0 / 8.0
    x["bt"][5, :3] = x["bt"][5, 0]
    ref, lse_ref = oracle.verify_attention(x["q"], x["k"], x["v"], x["bt"], x["ctx"], x["cu"], H_q=H_q, H_kv=H_kv, D=64, P=16,
                                           dtype="bf16", scale=float(np.float32(scale)))
    q = dev(x["q"], True)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
    fsr.verify_attention(q, dev(x["k"], True), dev(x["v"], True), dev(x["bt"]), dev(x["ctx"]), None, dev(x["cu"]), scale=scale, out=out,
                         lse=lse, max_q_len=hint)
    torch.cuda.synchronize()
    check_attention(out, ref, "f32", len(ref))
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("longest", [1690, 4100])  # cut only where the items do not fit otherwise, cut
@pytest.mark.parametrize("units,B", [(33, 5), (64, 9), (65, 5), (128, 15)])
def test_balanced_within_the_callers_workgroups(fsr, oracle, units, B, longest):
    """Items between half the units that the caller owns, odd numbers of them too, and one and a half times as many."""
    announce(f"balanced items max_workgroups={units} longest={longest}")
    rng = np.random.Generator(np.random.PCG64(units))
    ctx, spec = rng.integers(0, 1700, B), rng.integers(0, 4, B)
    ctx[0], ctx[1:3] = longest, 60
    x = make(rng, "bf16", 32, 8, 64, 16, ctx, spec)
    ref, lse_ref = oracle.verify_attention(x["q"], x["k"], x["v"], x["bt"], x["ctx"], x["cu"], H_q=32, H_kv=8, D=64, P=16, dtype="bf16", scale=0.125)
    q = dev(x["q"], True)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
    fsr.verify_attention(q, dev(x["k"], True), dev(x["v"], True), dev(x["bt"]), dev(x["ctx"]), None, dev(x["cu"]), scale=0.125, out=out,
                         lse=lse, max_q_len=4, max_workgroups=units)
    torch.cuda.synchronize()
    check_attention(out, ref, "f32", len(ref))
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("longest", [1690, 4100])  # whole items, cut ones
def test_balanced_through_the_built_in_scratch(fsr, longest):
    """fsr_verify_attention_static against fsr_verify_attention, bit for bit."""
    announce(f"balanced items static longest={longest}")
    rng = np.random.Generator(np.random.PCG64(4))
    ctx, spec = rng.integers(0, 1700, 20), rng.integers(0, 4, 20)
    ctx[0] = longest
    x = make(rng, "bf16", 32, 8, 64, 16, ctx, spec)
    q, k, v, bt, c, cu = dev(x["q"], True), dev(x["k"], True), dev(x["v"], True), dev(x["bt"]), dev(x["ctx"]), dev(x["cu"])
    outs = [torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    lses = [torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda") for _ in range(2)]
    fsr.verify_attention(q, k, v, bt, c, None, cu, scale=0.125, out=outs[0], lse=lses[0], max_q_len=4)
    fsr.verify_attention_static(q, k, v, bt, c, cu, scale=0.125, out=outs[1], lse=lses[1], max_q_len=4)
    torch.cuda.synchronize()
    assert not torch.isnan(outs[0].float()).any()
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16)) and torch.equal(lses[0], lses[1])


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_values_that_are_not_finite_in_balanced_pieces(fsr, oracle, bad):
    """Such values of V reach exactly the rows that see their key: across the cuts of an item, and beside another item of the workgroup."""
    announce(f"balanced items bad={bad}")
    rng = np.random.Generator(np.random.PCG64(12))
    H_kv, B = 7, 29  # an odd number of pieces side by side
    ctx, spec = rng.integers(100, 1700, B), rng.integers(0, 4, B)
    ctx[:6:2] = 4100, 3300, 2900  # long enough to be cut
    x = make(rng, "bf16", 14, H_kv, 64, 16, ctx, spec)
    store = np.uint16(0x7FC0 if np.isnan(bad) else 0x7F80 if bad > 0 else 0xFF80)
    hit = {}
    for i in range(0, B, 3):  # a key of one KV head; some only the later rows see
        key = int(ctx[i]) + int(spec[i]) if i % 2 else int(rng.integers(0, ctx[i]))
        g, d = int(rng.integers(H_kv)), int(rng.integers(64))
        x["v"].view(np.uint16)[x["bt"][i, key // 16], g, key % 16, d] = store
        hit[i] = (g, key, d)
    q = dev(x["q"], True)
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    fsr.verify_attention(q, dev(x["k"], True), dev(x["v"], True), dev(x["bt"]), dev(x["ctx"]), None, dev(x["cu"]), scale=0.125, out=out, max_q_len=4)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    want_bad = np.zeros(got.shape, bool)
    for i, (g, key, d) in hit.items():
        for j in range(spec[i] + 1):
            if key <= ctx[i] + j:
                want_bad[x["cu"][i] + j, 2 * g:2 * g + 2, d] = True
    assert np.array_equal(~np.isfinite(got), want_bad)
    assert np.array_equal(np.isnan(got[want_bad]), np.full(want_bad.sum(), np.isnan(bad)))
    clean = x["v"].copy()
    for i, (g, key, d) in hit.items():
        clean.view(np.uint16)[x["bt"][i, key // 16], g, key % 16, d] = 0
    ref, _ = oracle.verify_attention(x["q"], x["k"], clean, x["bt"], x["ctx"], x["cu"], H_q=14, H_kv=H_kv, D=64, P=16, dtype="bf16", scale=0.125)
    got[want_bad] = ref[want_bad]
    check_attention(torch.from_numpy(got), ref, "f32", len(ref))


def test_cut_and_whole_items_in_a_graph(fsr):
    """Replays over contexts that are worth cutting and others that are not, with eager calls on the same workspace between them: the
    bits of an eager call on a workspace of its own."""
    announce("cut and whole items in a graph")
    rng = np.random.Generator(np.random.PCG64(3))
    B = 20
    x = make(rng, "bf16", 32, 8, 64, 16, np.full(B, 4100), rng.integers(0, 4, B))
    q, k, v, bt, cu = dev(x["q"], True), dev(x["k"], True), dev(x["v"], True), dev(x["bt"]), dev(x["cu"])
    need = fsr.attn_workspace_bytes(B=B, N_cap=q.shape[0], H_q=32, H_kv=8, D=64, P=16, max_pages=bt.shape[1], n_pages=k.shape[0],
                                    dtype=torch.bfloat16, out_dtype=torch.bfloat16, max_q_len=4)
    ws, own = (torch.full((need,), 0x55, dtype=torch.uint8, device="cuda") for _ in range(2))
    c, out, want = dev(x["ctx"]), torch.empty_like(q), torch.empty_like(q)

    def call(into, workspace):
        fsr.verify_attention(q, k, v, bt, c, None, cu, scale=0.125, out=into, max_q_len=4, workspace=workspace)

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call(out, ws)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            call(out, ws)
        for rep in range(6):
            ctx = rng.integers(0, 200 if rep == 2 else 1700, B)
            if rep in (0, 1, 4):
                ctx[rng.permutation(B)[:3]] = 3900, 4100, 2500
            c.copy_(dev(ctx.astype(np.int32)))
            out.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            before = own.clone()
            call(want, own)
            torch.cuda.synchronize()
            assert (not torch.equal(before, own)) == (rep in (0, 1, 4))  # whole items leave no pieces
            assert torch.equal(out.view(torch.int16), want.view(torch.int16))
            call(out, ws)
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), want.view(torch.int16))
