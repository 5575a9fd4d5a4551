"""GPU parity of the attention shapes outside the stream kernel (fp32, heads of 64, other page sizes, wide query groups)
against the oracle: edges of key tiles and of query-row groups, both layouts, any alignment, Inf and NaN values."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import announce, check_attention, dev

pytestmark = pytest.mark.gpu

# contexts around the 16- and 32-key tiles, their stride over four and eight waves, and page ends
CTX = [0, 1, 14, 15, 16, 31, 32, 63, 64, 127, 128, 240, 255, 256, 257, 300, 511, 513, 700]
SPEC = [2, 0, 1, 0, 3, 7, 1, 4, 0, 8, 2, 15, 0, 5, 1, 9, 0, 3, 6]


@pytest.fixture(scope="module")
def fsr():
    import paper_2604_20503_amd as f
    f.load_library()
    return f


def make(rng, dtype, H_q, H_kv, D, P, ctx, spec):
    ctx, spec = np.asarray(ctx, np.int32), np.asarray(spec, np.int32)
    tok = ctx + spec + 1
    npg = (tok + P - 1) // P
    n_pages = int(npg.sum()) + 2
    perm = rng.permutation(n_pages).astype(np.int32)
    bt = np.full((len(ctx), int(npg.max()) + 1), -1, np.int32)
    at = 0
    for i, n in enumerate(npg):
        bt[i, :n] = perm[at:at + n]
        at += n
    cu = workloads.exclusive_offsets(spec + 1)
    st = lambda s: workloads._normal_store(rng, s, dtype)  # noqa: E731
    return dict(ctx=ctx, cu=cu, bt=bt, q=st((int(cu[-1]), H_q, D)), k=st((n_pages, H_kv, P, D)), v=st((n_pages, H_kv, P, D)))


def run(fsr, oracle, x, dtype, H_q, H_kv, D, P, *, token_major=False, out_dtype=torch.float32, hint=0, shift=0):
    bf = dtype == "bf16"
    swap = (lambda t: np.ascontiguousarray(np.swapaxes(t, 1, 2))) if token_major else (lambda t: t)

    def place(t):  # the tensor at an address `shift` elements past an aligned one
        flat = dev(t, bf).reshape(-1)
        room = torch.empty(flat.numel() + shift, dtype=flat.dtype, device="cuda")
        room[shift:] = flat
        return room[shift:].view(t.shape)

    q, k, v = place(x["q"]), place(swap(x["k"])), place(swap(x["v"]))
    out = torch.empty(q.numel() + shift, dtype=out_dtype, device="cuda")[shift:].view(q.shape)
    lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
    scale = 1.0 / np.sqrt(D)
    fsr.verify_attention(q, k, v, dev(x["bt"]), dev(x["ctx"]), None, dev(x["cu"]), scale=scale, out=out, lse=lse,
                         max_q_len=hint, kv_layout=1 if token_major else 0)
    torch.cuda.synchronize()
    ref, lse_ref = oracle.verify_attention(x["q"], x["k"], x["v"], x["bt"], x["ctx"], x["cu"], H_q=H_q, H_kv=H_kv, D=D, P=P,
                                           dtype=dtype, scale=float(np.float32(scale)))
    return out, lse, ref, lse_ref


@pytest.mark.parametrize("dtype,H_q,H_kv,D,P,token_major", [
    ("f32", 8, 2, 64, 16, False), ("f32", 6, 6, 128, 16, True), ("f32", 14, 2, 64, 24, False), ("f32", 40, 2, 128, 8, False),
    ("bf16", 8, 2, 64, 16, False), ("bf16", 6, 6, 64, 16, True), ("bf16", 14, 2, 64, 24, True), ("bf16", 20, 1, 64, 1, False),
    ("bf16", 8, 2, 128, 32, False), ("bf16", 34, 2, 128, 16, True), ("bf16", 80, 1, 128, 16, False)])
def test_shapes_outside_the_stream_kernel(fsr, oracle, dtype, H_q, H_kv, D, P, token_major):
    rng = np.random.Generator(np.random.PCG64(31 * H_q + D + P))
    x = make(rng, dtype, H_q, H_kv, D, P, CTX, SPEC)
    # the bound on a request's rows given, given too small, not given (different query tiles and groups)
    for hint in (max(SPEC) + 1, 2, 0):
        announce(f"items {dtype} heads={H_q}/{H_kv} D={D} P={P} token_major={token_major} hint={hint}")
        out, lse, ref, lse_ref = run(fsr, oracle, x, dtype, H_q, H_kv, D, P, token_major=token_major, hint=hint)
        err = check_attention(out, ref, "f32", len(ref))  # fp32 accuracy for bf16 inputs too: nothing is rounded to 16 bits
        np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)
        print(f"max rel err {err:.2e}")


@pytest.mark.parametrize("H_q,H_kv,D,P,hint", [(8, 2, 64, 16, 16), (40, 4, 64, 8, 4), (6, 6, 128, 32, 16), (17, 1, 128, 16, 2), (32, 2, 128, 24, 3)])
@pytest.mark.parametrize("scratch", ["own", "none", "short", "misaligned"])
def test_items_in_pieces(fsr, oracle, H_q, H_kv, D, P, hint, scratch):
    """Contexts around the multiples of the least piece (512 keys), more rows than the bound says, one to four query tiles; the
    same without scratch memory that holds the pieces."""
    announce(f"items in pieces heads={H_q}/{H_kv} D={D} P={P} hint={hint} scratch={scratch}")
    rng = np.random.Generator(np.random.PCG64(H_q + D))
    ctx, spec = [1022, 510, 1023, 1024, 4100, 0, 2600, 1535], [0, 1, 2, 0, 1, 1, 0, 3]
    x = make(rng, "bf16", H_q, H_kv, D, P, ctx, spec)
    q, k, v = (dev(x[n], True) for n in "qkv")
    need = fsr.attn_workspace_bytes(B=len(ctx), N_cap=q.shape[0], H_q=H_q, H_kv=H_kv, D=D, P=P, max_pages=x["bt"].shape[1],
                                    n_pages=k.shape[0], dtype=torch.bfloat16, out_dtype=torch.float32, max_q_len=hint)
    assert need > 0
    room = torch.full((need + 256,), 0x55, dtype=torch.uint8, device="cuda")
    ws = {"own": None, "none": room[:0], "short": room[:256], "misaligned": room[16:16 + need]}[scratch]
    scale = 1.0 / np.sqrt(D)
    ref, lse_ref = oracle.verify_attention(x["q"], x["k"], x["v"], x["bt"], x["ctx"], x["cu"], H_q=H_q, H_kv=H_kv, D=D, P=P,
                                           dtype="bf16", scale=float(np.float32(scale)))
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
    for _ in range(2):  # the second call finds the first one's counts
        out.fill_(float("nan"))
        fsr.verify_attention(q, k, v, dev(x["bt"]), dev(x["ctx"]), None, dev(x["cu"]), scale=scale, out=out, lse=lse,
                             max_q_len=hint, workspace=ws)
        torch.cuda.synchronize()
        check_attention(out, ref, "f32", len(ref))
        np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)
    if scratch != "own":
        assert (room == 0x55).all()


@pytest.mark.parametrize("D,P", [(64, 16), (128, 32)])
def test_items_in_pieces_in_a_graph(fsr, D, P):
    """A captured call whose items are cut, replayed over caches that change, with eager calls of another batch on the same
    workspace between the replays: every replay gives the bits of an eager call on a workspace of its own."""
    announce(f"items in pieces, graph D={D}")
    rng = np.random.Generator(np.random.PCG64(D))
    x = make(rng, "bf16", 8, 2, D, P, [4100, 30, 1500, 2600], [2, 0, 1, 3])
    q, k, v = (dev(x[n], True) for n in "qkv")
    bt, c, cu = dev(x["bt"]), dev(x["ctx"]), dev(x["cu"])
    need = fsr.attn_workspace_bytes(B=4, N_cap=q.shape[0], H_q=8, H_kv=2, D=D, P=P, max_pages=bt.shape[1], n_pages=k.shape[0],
                                    dtype=torch.bfloat16, out_dtype=torch.float32, max_q_len=4)
    assert need > 0
    room = [torch.full((need,), 0x55, dtype=torch.uint8, device="cuda") for _ in range(2)]
    out, other, want = (torch.zeros(q.shape, dtype=torch.float32, device="cuda") for _ in range(3))
    c2 = dev(np.array([2000, 4000, 0, 700], np.int32))

    def call(ctx, into, workspace):
        fsr.verify_attention(q, k, v, bt, ctx, None, cu, scale=0.1, out=into, max_q_len=4, workspace=workspace)

    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        call(c, out, room[0])
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            call(c, out, room[0])
        for turn in range(4):
            v.copy_(torch.randn(v.shape, device="cuda"))
            out.fill_(float("nan"))
            g.replay()
            call(c2, other, room[0])
            call(c, want, room[1])
            torch.cuda.synchronize()
            assert torch.isfinite(want).all() and torch.equal(out.view(torch.int32), want.view(torch.int32)), turn
    torch.cuda.synchronize()
    call(c, want, room[0])  # the calls of the other stream are done: its workspace may be used here
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("D,P", [(64, 16), (128, 32)])
@pytest.mark.parametrize("bad", [(np.inf,), (-np.inf,), (np.nan,), (np.inf, -np.inf)])
def test_values_that_are_not_finite_in_pieces(fsr, oracle, D, P, bad):
    """V that is not finite on both sides of where an item of 4104 keys is cut into eight, and at a drafted token in the last piece:
    the rows that see the key carry the value in that element, all else is untouched; +Inf and -Inf from two pieces make NaN."""
    announce(f"items in pieces D={D} V={bad}")
    rng = np.random.Generator(np.random.PCG64(12))
    ctx, spec = [4100, 900], [3, 2]
    x = make(rng, "bf16", 4, 1, D, P, ctx, spec)
    ref, _ = oracle.verify_attention(x["q"], x["k"], x["v"], x["bt"], x["ctx"], x["cu"], H_q=4, H_kv=1, D=D, P=P, dtype="bf16",
                                     scale=float(np.float32(1.0 / np.sqrt(D))))
    tiles = (4104 + 31) // 32
    code = lambda b: np.uint16(np.float32(b).view(np.uint32) >> 16)  # noqa: E731
    want = ref.copy()
    for d, at in ((3, 32 * (tiles // 8) - 1), (9, 32 * (tiles // 8)), (20, 32 * (tiles * 5 // 8)), (41, ctx[0] + 2)):
        x["v"][x["bt"][0, at // P], 0, at % P, d] = code(bad[0])
        first = max(0, at - ctx[0])
        if len(bad) > 1:  # the other value in the first tile, i.e. in another piece
            x["v"][x["bt"][0, 7 // P], 0, 7 % P, d] = code(bad[1])
            want[0:first, :, d] = bad[1]
        want[first:4, :, d] = bad[0] if len(bad) == 1 else np.nan
    out, _, _, _ = run(fsr, oracle, x, "bf16", 4, 1, D, P, hint=4)
    o = out.cpu().numpy()
    odd = ~np.isfinite(want)
    assert np.array_equal(o[odd], want[odd].astype(np.float32), equal_nan=True)
    np.testing.assert_allclose(o[~odd], want[~odd], rtol=0, atol=1e-5 * np.abs(ref).max())


@pytest.mark.parametrize("units,cut", [(0, True), (4, True), (3, False), (2, False)])
def test_pieces_stay_within_the_callers_workgroups(fsr, units, cut):
    """Two items on a stream that owns `units` compute units (0: the device): with fewer than four they are not cut, i.e. give the
    bits of a call whose workspace is too small for pieces."""
    announce(f"items max_workgroups={units}")
    x = make(np.random.Generator(np.random.PCG64(17)), "bf16", 8, 2, 64, 16, [4000], [2])
    q, k, v = (dev(x[n], True) for n in "qkv")
    bt, c, cu, outs = dev(x["bt"]), dev(x["ctx"]), dev(x["cu"]), []
    for ws in (None, torch.empty(256, dtype=torch.uint8, device="cuda")):
        outs.append(torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda"))
        fsr.verify_attention(q, k, v, bt, c, None, cu, scale=0.1, out=outs[-1], max_q_len=3, max_workgroups=units, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32)) != cut


@pytest.mark.parametrize("dtype,H_q,H_kv,D,P,ctx", [
    ("bf16", 8, 2, 64, 16, [4100, 510, 1024, 2600]), ("bf16", 40, 4, 64, 8, [1023, 3000]), ("bf16", 17, 1, 128, 16, [8000]),
    ("bf16", 32, 2, 128, 24, [2000] * 70), ("f32", 8, 2, 64, 16, [2000, 30])])
def test_built_in_scratch_gives_the_same_bits(fsr, dtype, H_q, H_kv, D, P, ctx):
    """fsr_verify_attention_static against fsr_verify_attention: items in pieces, too many of them for that, fp32."""
    announce(f"items static {dtype} heads={H_q}/{H_kv} D={D} P={P} B={len(ctx)}")
    rng = np.random.Generator(np.random.PCG64(H_q + D + len(ctx)))
    x = make(rng, dtype, H_q, H_kv, D, P, ctx, [i % 3 for i in range(len(ctx))])
    q, k, v = (dev(x[n], dtype == "bf16") for n in "qkv")
    bt, c, cu = dev(x["bt"]), dev(x["ctx"]), dev(x["cu"])
    outs, lses = ([torch.full(shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)] for shape in (q.shape, q.shape[:2]))
    fsr.verify_attention(q, k, v, bt, c, None, cu, scale=0.1, out=outs[0], lse=lses[0], max_q_len=3)
    fsr.verify_attention_static(q, k, v, bt, c, cu, scale=0.1, out=outs[1], lse=lses[1], max_q_len=3)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32)) and torch.equal(lses[0].view(torch.int32), lses[1].view(torch.int32))


@pytest.mark.parametrize("H_q,H_kv,D,P,token_major", [(8, 2, 64, 16, False), (14, 2, 64, 24, True), (20, 1, 64, 1, False),
                                                      (6, 6, 128, 32, False), (34, 2, 128, 16, True), (80, 1, 128, 16, False)])
def test_bf16_output(fsr, oracle, H_q, H_kv, D, P, token_major):
    """One to four query tiles, one and several row groups, page sizes and wide query groups, with the result in bf16."""
    rng = np.random.Generator(np.random.PCG64(13 * H_q + D + P))
    x = make(rng, "bf16", H_q, H_kv, D, P, CTX, SPEC)
    for hint in (max(SPEC) + 1, 2, 0):
        announce(f"items bf16 output heads={H_q}/{H_kv} D={D} P={P} token_major={token_major} hint={hint}")
        out, lse, ref, lse_ref = run(fsr, oracle, x, "bf16", H_q, H_kv, D, P, token_major=token_major, out_dtype=torch.bfloat16, hint=hint)
        check_attention(out, ref, "f32", len(ref))
        np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("dtype,D,P,out_dtype", [("bf16", 64, 16, torch.bfloat16), ("bf16", 128, 8, torch.float32),
                                                 ("f32", 64, 16, torch.float32)])
def test_more_row_groups_than_workgroups(fsr, oracle, dtype, D, P, out_dtype):
    """One request of 241 rows with 20 query heads: 4820 rows of a KV head, in groups of 64 (D = 64) or 48, of which an item
    has at most 64 in flight; beside it requests of few rows and of none at all."""
    rng = np.random.Generator(np.random.PCG64(77))
    x = make(rng, dtype, 20, 1, D, P, [70, 0, 33, 5], [240, 0, 2, 3])
    x["cu"] = np.concatenate([x["cu"][:2], x["cu"][1:2], x["cu"][2:-1]]).astype(np.int32)  # request 1 has no rows, 2 one
    for hint in (0, 241, 3):
        announce(f"items many groups {dtype} D={D} hint={hint}")
        out, lse, ref, lse_ref = run(fsr, oracle, x, dtype, 20, 1, D, P, out_dtype=out_dtype, hint=hint)
        n = int(x["cu"][-1])
        check_attention(out[:n], ref[:n], "f32", n)
        np.testing.assert_allclose(lse[:n].cpu().numpy(), lse_ref[:n], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("dtype,D,P", [("f32", 64, 16), ("bf16", 64, 16), ("bf16", 128, 32)])
@pytest.mark.parametrize("size", [1e37, 4e35])
def test_values_near_the_end_of_the_range(fsr, oracle, dtype, D, P, size):
    """Two keys of score 0 and 5 with large values among others of score -20 and ordinary values: an exponent's reference may
    lag behind by 5.5, but a probability of e^5 must not meet such values (the result, about the value itself, is finite)."""
    announce(f"items large values {dtype} D={D} {size}")
    rng = np.random.Generator(np.random.PCG64(3))
    ctx = [1000, 700]
    x = make(rng, dtype, 4, 1, D, P, ctx, [0, 2])
    code = (lambda a: np.asarray(a, np.float32)) if dtype == "f32" else (lambda a: (np.asarray(a, np.float32).view(np.uint32) >> 16).astype(np.uint16))
    unit = np.zeros(D, np.float32)
    unit[3] = np.sqrt(D)
    x["q"][:] = code(unit / np.sqrt(D))
    x["k"][:] = code(-20.0 * unit)
    for i, c in enumerate(ctx):
        for t, score in ((1, 0.0), (1 + 512 + i * 128, 5.0)):
            x["k"][x["bt"][i, t // P], 0, t % P] = code(score * unit)
            x["v"][x["bt"][i, t // P], 0, t % P] = code(rng.uniform(0.5, 1.0, D).astype(np.float32) * size)
    out, _, ref, _ = run(fsr, oracle, x, dtype, 4, 1, D, P, hint=3)
    check_attention(out, ref, "f32", len(ref))


@pytest.mark.parametrize("dtype,D,shift,out_dtype", [("f32", 64, 1, torch.float32), ("bf16", 64, 1, torch.bfloat16),
                                                     ("bf16", 64, 3, torch.float32)])
def test_inputs_aligned_to_their_elements_only(fsr, oracle, dtype, D, shift, out_dtype):
    announce(f"items {dtype} shift={shift} out={out_dtype}")
    rng = np.random.Generator(np.random.PCG64(5))
    x = make(rng, dtype, 8, 2, D, 16, CTX[:8], SPEC[:8])
    out, _, ref, _ = run(fsr, oracle, x, dtype, 8, 2, D, 16, out_dtype=out_dtype, hint=9, shift=shift)
    check_attention(out, ref, "f32" if out_dtype == torch.float32 else "bf16", len(ref))


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_values_that_are_not_finite_reach_their_rows_only(fsr, oracle, dtype, D, bad):
    """One element of V at the second drafted token's position: rows before it are untouched, rows from it on carry the
    value in that element (and only there); keys of another request never matter."""
    announce(f"items {dtype} D={D} V={bad}")
    rng = np.random.Generator(np.random.PCG64(9))
    P = 16 if D == 64 else 32
    ctx, spec = [40, 33], [4, 3]
    x = make(rng, dtype, 4, 1, D, P, ctx, spec)
    ref, _ = oracle.verify_attention(x["q"], x["k"], x["v"], x["bt"], x["ctx"], x["cu"], H_q=4, H_kv=1, D=D, P=P, dtype=dtype,
                                     scale=float(np.float32(1.0 / np.sqrt(D))))
    t, d = ctx[0] + 2, 5
    code = np.float32(bad) if dtype == "f32" else np.uint16(np.float32(bad).view(np.uint32) >> 16)
    x["v"][x["bt"][0, t // P], 0, t % P, d] = code
    out, _, _, _ = run(fsr, oracle, x, dtype, 4, 1, D, P, hint=5)
    o = out.cpu().numpy()
    hit = np.zeros(ref.shape, bool)
    hit[2:5, :, d] = True
    assert np.array_equal(o[hit], np.full(hit.sum(), bad, np.float32), equal_nan=True)
    np.testing.assert_allclose(o[~hit], ref[~hit], rtol=0, atol=1e-5 * np.abs(ref).max())


@pytest.mark.parametrize("D,P", [(64, 16), (128, 32)])
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_probabilities_keep_32_bits(fsr, oracle, D, P, out_dtype):
    """Outputs that are differences of nearly equal probabilities: two keys that differ by one unit in the last place of one
    component, with values A and -A among zeros, so that an output is A (p1 - p2).  Error bound relative to A, besides the
    output's own rounding: 2^-20.  It holds for 32-bit arithmetic (scores around 6 enter the exponential's argument with half
    a unit of 2^-20, the rest are a few 2^-24 of p <= 1/2), and not for probabilities cut to 17 bits, off by up to 2^-18."""
    announce(f"items probabilities D={D} out={out_dtype}")
    rng = np.random.Generator(np.random.PCG64(21))
    H_q, H_kv, B = 8, 2, 64
    widen = lambda a: (a.astype(np.uint32) << 16).view(np.float32)  # noqa: E731
    narrow = lambda a: (np.asarray(a, np.float32).view(np.uint32) >> 16).astype(np.uint16)  # noqa: E731
    x = make(rng, "bf16", H_q, H_kv, D, P, np.full(B, 33), np.zeros(B))
    x["k"][:] = 0
    x["v"][:] = 0
    size = np.empty((B, H_q, D))
    for i in range(B):
        mean = widen(x["q"][i]).reshape(H_kv, H_q // H_kv, D).mean(1)
        key = narrow(mean * 6.0 * np.sqrt(D) / (mean ** 2).sum(-1, keepdims=True))  # score 6 at the group's mean query
        val = narrow(rng.uniform(1.0, 2.0, (H_kv, D)))
        for t, k, v in ((7, key, val), (20, key.copy(), val ^ np.uint16(0x8000))):
            if t == 20:
                k[:, i % D] ^= 1
            page = x["bt"][i, t // P]
            x["k"][page, :, t % P], x["v"][page, :, t % P] = k, v
        size[i] = np.repeat(widen(val), H_q // H_kv, 0)
    out, _, ref, _ = run(fsr, oracle, x, "bf16", H_q, H_kv, D, P, out_dtype=out_dtype, hint=1)
    err = np.abs(out.float().cpu().numpy().astype(np.float64) - ref)
    err -= (2.0 ** -8 if out_dtype == torch.bfloat16 else 2.0 ** -23) * np.abs(ref)  # the output's rounding
    small = np.abs(ref) < 2.0 ** -10 * size  # where that does not hide the probabilities
    print(f"{small.sum()} of {small.size} elements, worst {(err / size)[small].max():.2e}")
    assert small.sum() > small.size // 4
    assert (err[small] <= 2.0 ** -20 * size[small]).all()
