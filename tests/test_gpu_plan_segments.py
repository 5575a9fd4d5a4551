"""Plans whose shares hold many segments: the planned call is bit-identical to the one that schedules itself (the oracle
covers the latter)."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import announce, check_attention, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsr():
    import paper_2604_20503_amd as f
    f.load_library()
    return f


@pytest.mark.parametrize("B,H_q,H_kv,spec_hi,max_workgroups,hint", [
    (300, 8, 8, 3, 3, 4),      # 2400 items on three shares: a wave takes more than 64 segments; two rounds of the prefix
    (65, 32, 8, 20, 7, 0),     # no bound on the rows: several row groups per request (two-team kernel)
    (65, 32, 8, 20, 0, 2),     # a bound that is too small: several one-tile groups per request
    (1, 16, 1, 0, 0, 1),       # one item, cut into as many pieces as it has tiles or workgroups
])
def test_many_segments_per_share(fsr, B, H_q, H_kv, spec_hi, max_workgroups, hint):
    announce(f"plan segments B={B} heads={H_q}/{H_kv} workgroups={max_workgroups} hint={hint}")
    rng = np.random.Generator(np.random.PCG64(B + H_q))
    ctx = rng.integers(0, 200, size=B) if B > 1 else np.array([3000])
    spec = rng.integers(0, spec_hi + 1, size=B)
    b = workloads.make_batch(2, with_probs=False, H_q=H_q, H_kv=H_kv, ctx_lens=ctx, spec_lens=spec)
    cu = b.cu_q.copy()
    if B > 1:  # every fifth request has no rows: its rows go to the next one's neighbour
        lens = np.diff(cu)
        lens[::5] = 0
        cu = workloads.exclusive_offsets(lens)
    q, k, v = dev(b.q, True), dev(b.k_cache, True), dev(b.v_cache, True)
    bt, ctx_d, cu_d = dev(b.block_tables), dev(b.ctx_lens), dev(cu)
    kw = dict(scale=b.scale, max_q_len=hint, max_workgroups=max_workgroups)
    outs = []
    for plan in (None, fsr.attn_plan(q, k, bt, ctx_d, cu_d, **kw)):
        out = torch.zeros(q.shape, dtype=torch.float32, device="cuda")
        lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
        fsr.verify_attention(q, k, v, bt, ctx_d, None, cu_d, out=out, lse=lse, plan=plan, **kw)
        torch.cuda.synchronize()
        assert torch.isfinite(out).all()
        outs.append((out, lse))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("H_q,H_kv,ctx,spec,max_workgroups,hint", [
    (32, 8, [765, 766, 767, 768, 1535], [0, 1, 2, 3, 8], 0, 9),      # around the least piece of 24 tiles; 1 to 3 query tiles
    (32, 8, [5000], [3], 0, 4), (8, 1, [9000, 1], [0, 1], 9, 2),     # few workgroups: 9 for two items
    (4, 4, list(range(1, 1280, 20)), [1] * 64, 0, 2),                # 64 requests x 4 heads: as many items as workgroups
    (4, 4, [40] * 60 + [4000] * 4, [1] * 64, 0, 2),                  # ... too uneven: the cost line
    (4, 4, [300] * 65, [1] * 65, 0, 2),                              # a request more than a wave has lanes: the cost line
    (64, 8, [900, 2000, 33], [10, 1, 5], 0, 11),                     # two-team groups beside ordinary ones
    (32, 8, [100, 700, 900], [2, 8, 0], 0, 0),                       # no bound on the rows
    (32, 8, [100, 900], [8, 8], 0, 2)])                              # a bound that is too small: the cost line
def test_a_piece_of_an_item_per_share(fsr, oracle, H_q, H_kv, ctx, spec, max_workgroups, hint):
    announce(f"plan pieces heads={H_q}/{H_kv} B={len(ctx)} workgroups={max_workgroups} hint={hint}")
    b = workloads.make_batch(2, with_probs=False, H_q=H_q, H_kv=H_kv, ctx_lens=np.array(ctx), spec_lens=np.array(spec))
    q, k, v = dev(b.q, True), dev(b.k_cache, True), dev(b.v_cache, True)
    bt, ctx_d, cu = dev(b.block_tables), dev(b.ctx_lens), dev(b.cu_q)
    kw = dict(scale=b.scale, max_q_len=hint, max_workgroups=max_workgroups)
    ref, lse_ref = oracle.verify_attention(b.q, b.k_cache, b.v_cache, b.block_tables, b.ctx_lens, b.cu_q, H_q=H_q, H_kv=H_kv, D=b.D,
                                           P=b.P, dtype=b.dtype, scale=b.scale)
    outs = []
    for plan in (None, fsr.attn_plan(q, k, bt, ctx_d, cu, **kw)):
        out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
        lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
        fsr.verify_attention(q, k, v, bt, ctx_d, None, cu, out=out, lse=lse, plan=plan, **kw)
        torch.cuda.synchronize()
        check_attention(out, ref, "bf16", b.N)
        np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=1e-4, atol=1e-4)
        outs.append((out, lse))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("B", [1, 2, 7, 12, 13, 16, 25, 40, 64])
def test_plan_and_call_cut_items_alike(fsr, B):
    """Where items are cut follows from quotients rounded at many places, by the plan kernel and by each stream kernel for itself:
    40 batches of random lengths, on all and on some workgroups, give the same bits with a plan and without."""
    announce(f"plan and call cut alike B={B}")
    rng = np.random.Generator(np.random.PCG64(B))
    H_q, H_kv, pages = 16, 4, 1200
    gen = torch.Generator(device="cuda").manual_seed(B)
    k, v = (torch.randn((pages, H_kv, 16, 128), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    for case in range(40):
        hi = int(np.exp(rng.uniform(np.log(600), np.log(6000))))
        ctx = np.minimum(rng.integers(0, hi, size=B) if case % 2 else np.exp(rng.normal(6.5, 1.2, size=B)), 10000).astype(np.int32)
        spec = rng.integers(0, 10, size=B).astype(np.int32)
        q = torch.randn((int((spec + 1).sum()), H_q, 128), generator=gen, device="cuda").to(torch.bfloat16)
        bt = dev(rng.integers(0, pages, size=(B, int((ctx + spec).max()) // 16 + 1)).astype(np.int32))
        c, cu = dev(ctx), dev(workloads.exclusive_offsets(spec + 1))
        kw = dict(scale=0.09, max_q_len=10, max_workgroups=int(rng.choice([0, 0, 4 * B + 3])))
        outs = []
        for plan in (None, fsr.attn_plan(q, k, bt, c, cu, **kw)):
            outs.append(torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda"))
            fsr.verify_attention(q, k, v, bt, c, None, cu, out=outs[-1], plan=plan, **kw)
        assert torch.isfinite(outs[0]).all() and torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32)), (case, ctx, spec)


@pytest.mark.parametrize("max_workgroups", [20, 32, 0])
def test_neighbouring_shares_of_the_cost_line_stay_on_one_die(fsr, max_workgroups):
    """A batch of few items for which the cost line is cut all the same (more rows than the bound says): workgroup w takes the share
    that it takes without a plan, i.e. the workgroups w, w + 8, w + 16, ... of one die take consecutive shares."""
    announce(f"plan places workgroups={max_workgroups}")
    b = workloads.make_batch(2, with_probs=False, H_q=32, H_kv=8, ctx_lens=np.array([3000, 2900]), spec_lens=np.array([8, 8]))
    q, k = dev(b.q, True), dev(b.k_cache, True)
    plan = fsr.attn_plan(q, k, dev(b.block_tables), dev(b.ctx_lens), dev(b.cu_q), scale=b.scale, max_q_len=2, max_workgroups=max_workgroups)
    torch.cuda.synchronize()
    rec = plan.view(torch.int32).view(-1, 32).cpu().numpy()
    nb, used = max_workgroups or 256, rec[0, 2]
    assert rec[1:1 + nb, 13].max() > 1  # the cost line: shares of several segments
    cuts = 0
    places = [w for die in range(8) for w in range(die, nb, 8)]  # workgroups in the order of their shares
    for share, w in enumerate(places):
        r = rec[1 + w]
        assert r[13] == 0 or share < used
        if r[13] > 0 and r[9] & 2:
            assert r[12] // 2 == share and r[10] <= share <= r[11]
            cuts += 1
    assert cuts > nb // 4


def test_segment_count_stays_within_the_plan(fsr):
    """Offsets past N_cap, one share: more segments than the buffer has records.  The share's count is the number of records
    written, and nothing is written behind the buffer.  (Only the plan is built here: no attention call reads it.)"""
    announce("plan segments beyond the buffer")
    H_q, H_kv, N_cap = 32, 8, 16
    i32 = dict(dtype=torch.int32, device="cuda")
    q = torch.zeros((N_cap, H_q, 128), dtype=torch.bfloat16, device="cuda")
    cache = torch.zeros((64, H_kv, 16, 128), dtype=torch.bfloat16, device="cuda")
    bt = torch.arange(2 * 64, **i32).view(2, 64) % 64
    ctx, cu = torch.tensor([5, 7], **i32), torch.tensor([0, 4, 4 + 600], **i32)  # 1 + 150 groups of four rows, 8 heads
    kw = dict(scale=1.0, max_q_len=1, max_workgroups=1)
    need = fsr.attn_plan(q, cache, bt, ctx, torch.tensor([0, 4, 8], **i32), **kw).numel()
    room = torch.full((need + 65536,), 0x77, dtype=torch.uint8, device="cuda")
    fsr.attn_plan(q, cache, bt, ctx, cu, plan=room[:need], **kw)
    torch.cuda.synchronize()
    rec = room[:need].view(torch.int32).view(-1, 32).cpu().numpy()
    further = len(rec) - 1 - 1024  # records behind the header and the shares' first ones
    assert further < 8 * 151 - 1
    assert rec[1, 13] == 1 + further
    assert (room[need:] == 0x77).all()
    assert (rec[1 + 1024:, 0] < 2).all() and (rec[1 + 1024:, 1] < H_kv).all()
