"""Greedy acceptance where most rows lie behind a mismatch and are left out: against the oracle, with row maps, ragged
vocabularies, draft ids outside the vocabulary and a call repeated on one workspace and one set of outputs."""
import numpy as np
import pytest
import torch

import workloads
from gpu_utils import announce, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsr():
    import paper_2604_20503_amd as f
    f.load_library()
    return f


# rows are left out from 3072 pieces on: B * (S + 1) rows of ceil(V / 16384) pieces; below 12288 the pieces are of 8192 scores.  Where
# none is, pieces are of 8192 scores for rows of up to 98304 and for calls of up to 128 pieces
@pytest.mark.parametrize("B,V,S", [(384, 8193, 7), (1536, 8192, 7), (1535, 8191, 7), (768, 16385, 7),(384, 16384, 7), (192, 16385, 7), (171, 32767, 8), (511, 501, 5), (512, 2048, 5),(1, 4095, 70), (200, 4097, 8), (64, 30003, 6), (700, 100, 3),
                                   (2500, 100, 7), (1100, 4097, 7), (64, 150001, 6), (2048, 20, 7), (2047, 20, 7),
                                   (383, 16384, 7), (64, 98309, 6), (3, 98304, 8), (3, 98305, 8), (2, 98305, 8), (1, 8191, 3), (1, 24577, 3)])
def test_rows_behind_a_mismatch(fsr, oracle, B, V, S):
    announce(f"greedy skipping B={B} V={V} S={S}")
    rng = np.random.default_rng(V)
    spec = rng.integers(0, S + 1, size=B).astype(np.int32)
    spec[0] = S
    cu_t, cu_d = workloads.exclusive_offsets(spec + 1), workloads.exclusive_offsets(spec)
    outs = [torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda"),
            torch.empty((B, S + 1), dtype=torch.int32, device="cuda")]
    ws = torch.empty(max(256, fsr.accept_workspace_bytes(B=B, V=V, S_max=S, mode=2)), dtype=torch.uint8, device="cuda")
    for match in (0.0, 0.5, 1.0):  # share of drafts that are their row's arg-max
        z = rng.standard_normal((int(cu_t[-1]), V)).astype(np.float32)
        best = z.argmax(1)
        owner = np.repeat(np.arange(B), spec)
        rows = cu_t[owner] + np.arange(int(cu_d[-1])) - cu_d[owner]
        toks = np.where(rng.random(len(rows)) < match, best[rows], rng.integers(0, V, len(rows))).astype(np.int32)
        if match == 0.5:
            toks[rng.random(len(toks)) < 0.1] = V + 3
            toks[rng.random(len(toks)) < 0.1] = -1
        ref = oracle.greedy_accept(z, toks, cu_t, cu_d, S_max=S)
        fsr.spec_accept(dev(z), None, dev(toks), None, None, dev(cu_t), dev(cu_d), S_max=S, mode=2, accepted_len=outs[0],
                        n_emitted=outs[1], emitted=outs[2], workspace=ws)
        torch.cuda.synchronize()
        for name, t in zip(("accepted_len", "n_emitted", "emitted"), outs):
            assert np.array_equal(t.cpu().numpy(), ref[name]), (name, match)


@pytest.mark.parametrize("B", [3, 16400])  # without and with rows left out
def test_drafts_of_a_flagged_request_are_not_read(fsr, B):
    """S_max = 0 and no draft array: a request whose offsets claim a draft is flagged, the others get their arg-max."""
    announce(f"greedy S_max=0 with a draft claimed B={B}")
    V = 501
    z = np.random.default_rng(1).standard_normal((B, V)).astype(np.float32)
    cu_d = np.zeros(B + 1, np.int32)
    cu_d[2:] = 1
    acc, n, em = fsr.spec_accept(dev(z), None, None, None, None, dev(np.arange(B + 1, dtype=np.int32)), dev(cu_d), S_max=0, mode=2)
    torch.cuda.synchronize()
    want = z.argmax(1)
    want[1] = -1
    assert acc.tolist() == [0, -1] + [0] * (B - 2) and n.tolist() == [1, -1] + [1] * (B - 2)
    assert np.array_equal(em[:, 0].cpu().numpy(), want)
