"""LOGITS-mode acceptance that leaves out rows behind a rejected draft: against the oracle, eagerly and in replays of one
captured call over inputs whose rejections change, on one workspace."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import DeviceBatch, announce, check_accept

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsr():
    import paper_2604_20503_amd as f
    f.load_library()
    return f


def batches(B, V, spec, reps):
    return [workloads.make_batch(2, rep=40 + r, with_kv=False, V=V, spec_lens=spec, ctx_lens=[8] * B, keep_logits=True,
                                 draft_mode=("noise", "independent")[r % 2]) for r in range(reps)]


@pytest.mark.parametrize("B,V,spec_hi", [   # rows are left out from 2048 rows, B * (2 * drafts + 1), on
    (190, 9000, 5),    # the longest drafts whose workgroups can be counted in the chunk masses' place (3 chunks: 5)
    (190, 9000, 6),    # one more: nothing is left out, the drafts are tested at the end
    (683, 4096, 1),    # a single chunk, one draft: 2049 rows
    (682, 4096, 1),    # 2046 rows: nothing is left out
    (300, 20001, 8),   # rows that are not aligned
    (2048, 4097, 0),   # bonus rows only
])
def test_rows_behind_a_rejection(fsr, oracle, B, V, spec_hi):
    announce(f"accept skipping B={B} V={V} drafts<={spec_hi}")
    spec = np.random.default_rng(V + B).integers(0, spec_hi + 1, size=B).astype(np.int32)
    spec[0] = spec_hi
    bs = batches(B, V, spec, 3)
    S = bs[0].S_max
    ws = torch.full((fsr.accept_workspace_bytes(B=B, V=V, S_max=S, mode=1),), 0xFF, dtype=torch.uint8, device="cuda")
    d = DeviceBatch(bs[0], kv=False, logits=True)
    outs = [torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda"),
            torch.empty((B, S + 1), dtype=torch.int32, device="cuda")]

    def call():
        fsr.spec_accept(d.z_target, d.z_draft, d.draft_tokens, d.u_accept, d.u_sample, d.cu_q, d.cu_d, S_max=S, mode=1,
                        temperature=0.8, accepted_len=outs[0], n_emitted=outs[1], emitted=outs[2], workspace=ws)

    def load(b):
        x = DeviceBatch(b, kv=False, logits=True)
        for name in ("z_target", "z_draft", "draft_tokens", "u_accept", "u_sample"):
            getattr(d, name).copy_(getattr(x, name))

    refs = [oracle.spec_accept(b.z_target, b.z_draft, b.draft_tokens, b.u_accept, b.u_sample, b.cu_q, b.cu_d, S_max=S, mode=1,
                               temperature=0.8) for b in bs]
    for b, ref in zip(bs, refs):
        load(b)
        call()
        torch.cuda.synchronize()
        check_accept(outs, ref, b.u_sample)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            call()
        for k in (0, 1, 1, 2, 0):  # replays, with an eager call on the same workspace in between
            load(bs[k])
            g.replay()
            torch.cuda.synchronize()
            check_accept(outs, refs[k], bs[k].u_sample)
            load(bs[(k + 1) % 3])
            call()
            torch.cuda.synchronize()
            check_accept(outs, refs[(k + 1) % 3], bs[(k + 1) % 3].u_sample)


def test_statistics_are_whole_or_left_out(fsr):
    """A row behind a rejection is left out by its whole workgroup or by none of it: whatever pair (reference, sum) a call
    leaves in its workspace is that row's own, and the others keep their bytes."""
    announce("accept statistics whole or left out")
    B, V = 400, 9000  # 4400 rows: one pair a row
    spec = np.random.default_rng(3).integers(4, 6, size=B).astype(np.int32)
    b = batches(B, V, spec, 2)[1]  # (drafts of a distribution of their own: most first drafts are rejected)
    S = b.S_max
    d = DeviceBatch(b, kv=False, logits=True)
    ws = torch.full((fsr.accept_workspace_bytes(B=B, V=V, S_max=S, mode=1),), 0xFF, dtype=torch.uint8, device="cuda")
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    at_t = up(B * 56) + 2 * up(B * 3 * 8) + up(B * 4)  # decisions, two arrays of chunk masses, arrivals
    at_d = at_t + up(B * (S + 1) * 3 * 16)
    lse_t, lse_d = (torch.logsumexp(z.double() / 0.8, dim=1) for z in (d.z_target, d.z_draft))
    left_out = 0
    for _ in range(20):
        ws.fill_(0xFF)
        fsr.spec_accept(d.z_target, d.z_draft, d.draft_tokens, d.u_accept, d.u_sample, d.cu_q, d.cu_d, S_max=S, mode=1,
                        temperature=0.8, workspace=ws)
        for at, lse in ((at_t, lse_t), (at_d, lse_d)):
            raw = ws[at:at + len(lse) * 16].view(torch.float64).view(-1, 2)
            untouched = (raw.view(torch.int64) == -1).all(1)
            left_out += int(untouched.sum())
            err = (raw[:, 0] + torch.log(raw[:, 1]) - lse)[~untouched].abs()
            assert bool((err < 1e-12 * lse.abs().max()).all()), float(err.max())
    assert left_out > 0


@pytest.mark.parametrize("steps", [(0, 130, 260, 390), (390, 260, 130, 0), (0, 95, 190, 90)])
def test_logits_that_climb_far_above_a_reference(fsr, oracle, steps):
    """Eight chunks a workgroup at most (4200 rows): from chunk to chunk a row's logits climb by more than the statistics let
    an exponent grow (100), by less, or fall."""
    announce(f"accept statistics steps={steps}")
    B, V, T = 600, 4 * 4096, 0.7
    spec = np.random.default_rng(5).integers(0, 4, size=B).astype(np.int32)
    spec[0] = 3
    b = batches(B, V, spec, 1)[0]
    lift = (np.repeat(np.array(steps, np.float32), 4096) * T).astype(np.float32)
    for z in (b.z_target, b.z_draft):
        z += lift
    best = int(np.argmax(steps)) * 4096
    b.draft_tokens[::2] = best + b.draft_tokens[::2] % 4096  # drafts among the likely tokens and elsewhere
    d = DeviceBatch(b, kv=False, logits=True)
    ref = oracle.spec_accept(b.z_target, b.z_draft, b.draft_tokens, b.u_accept, b.u_sample, b.cu_q, b.cu_d, S_max=b.S_max, mode=1,
                             temperature=T)
    gpu = fsr.spec_accept(d.z_target, d.z_draft, d.draft_tokens, d.u_accept, d.u_sample, d.cu_q, d.cu_d, S_max=b.S_max, mode=1,
                          temperature=T)
    torch.cuda.synchronize()
    check_accept(gpu, ref, b.u_sample)
    assert 0 < ref["accepted_len"].sum() < spec.sum()
