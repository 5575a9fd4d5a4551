"""GPU parity: prune_compact / prune_restore / prune_scatter vs the oracle, bit-exact."""
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


def _compare(fsr, oracle, keep, cu, suffix_close, pay, N_cap):
    ref = oracle.prune_compact(keep[: int(cu[-1])], cu, suffix_close=suffix_close, payload=pay[: int(cu[-1])])
    keep_d = dev(keep)
    r = fsr.prune_compact(keep_d, dev(cu), suffix_close=suffix_close, payload=dev(pay))
    torch.cuda.synchronize()
    N = int(cu[-1])
    n_new = int(ref["new_cu_q"][-1])
    assert np.array_equal(r["new_cu_q"].cpu().numpy(), ref["new_cu_q"])
    assert np.array_equal(r["new_q_lens"].cpu().numpy(), ref["new_q_lens"])
    src = r["src_row"].cpu().numpy()
    dst = r["dst_row"].cpu().numpy()
    assert np.array_equal(src[:N], ref["src_row"]) and (src[N:] == -1).all()
    assert np.array_equal(dst[:N], ref["dst_row"]) and (dst[N:] == -1).all()
    assert int(r["n_active"].item()) == ref["n_active"]
    assert np.array_equal(r["active_ids"].cpu().numpy(), ref["active_ids"])
    assert np.array_equal(r["payload"].cpu().numpy()[:n_new], ref["payload"])
    # restore and scatter
    back_ref, has_ref = oracle.prune_restore(ref["payload"], ref["dst_row"], pad_byte=0xAB)
    back, has = fsr.prune_restore(r["payload"], r["dst_row"], pad_word=0xABABABAB)
    torch.cuda.synchronize()
    assert np.array_equal(has.cpu().numpy()[:N], has_ref)
    assert np.array_equal(back.cpu().numpy()[:N], back_ref)
    base = torch.full_like(r["payload"], -7)
    fsr.prune_scatter(r["payload"], r["src_row"], r["new_cu_q"][len(cu) - 1:], base)
    torch.cuda.synchronize()
    exp = np.full_like(pay, -7)
    exp[ref["src_row"][:n_new]] = ref["payload"]
    assert np.array_equal(base.cpu().numpy(), exp)


@pytest.mark.parametrize("width", [4, 1023, 1024, 1028, 1025])  # words: 16-byte rows, one vector short of, exactly and past a lane's four
@pytest.mark.parametrize("B,maxlen", [(1, 8), (1025, 5), (1500, 9)])  # one window; a second tile of requests; windows of more than 8 rows
def test_survivor_windows(fsr, oracle, B, maxlen, width):
    announce(f"survivor_windows B={B} width={width}")
    rng = np.random.default_rng(B + width)
    lens = rng.integers(1, maxlen + 1, size=B)
    acc = np.minimum(rng.integers(-1, maxlen, size=B), lens - 1).astype(np.int32)
    cu = workloads.exclusive_offsets(lens)
    N = int(cu[-1])
    keep = np.concatenate([np.arange(n) <= a for n, a in zip(lens, acc)]).astype(np.uint8)
    pay = rng.integers(-1000, 1000, size=(N, width)).astype(np.int32)
    ref = oracle.prune_compact(keep, cu, suffix_close=True, payload=pay)
    mask = dev(np.full(N, 7, np.uint8))
    r = fsr.survivor_compact(dev(acc), dev(cu), N, keep_mask=mask, payload=dev(pay), payload_out=torch.full((N, width), -7, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    n_new = int(ref["new_cu_q"][-1])
    for name in ("new_cu_q", "new_q_lens", "src_row", "dst_row", "active_ids"):
        assert np.array_equal(r[name].cpu().numpy(), ref[name]), name
    assert np.array_equal(mask.cpu().numpy(), keep)
    got = r["payload"].cpu().numpy()
    assert np.array_equal(got[:n_new], ref["payload"]) and (got[n_new:] == -7).all()


@pytest.mark.parametrize("N,width", [(255, 3), (256, 3), (4096, 8), (4097, 8), (512, 8192), (513, 8192), (5, 8193), (6144, 769), (6145, 769), (6145, 3073)])
def test_copy_forms(fsr, oracle, N, width):
    """Edges of the rules that deal the payload's rows out: windows of one row and of more, 4096 and 6144 rows, rows of 12 and 32 KB, 16 MB."""
    announce(f"copy forms N={N} width={width}")
    rng = np.random.default_rng(N + width)
    cu = np.arange(0, N + 7, 7).clip(max=N).astype(np.int32)
    pay = rng.integers(-2**31, 2**31 - 1, size=(N, width), dtype=np.int64).astype(np.int32)
    for suffix_close in (True, False):
        _compare(fsr, oracle, (rng.random(N) < 0.8).astype(np.uint8), cu, suffix_close, pay, N)


@pytest.mark.parametrize("suffix_close", [True, False])
@pytest.mark.parametrize("drop", [0.0, 0.02, 0.3])
@pytest.mark.parametrize("copies,width", [(1, 4), (1, 1025), (17, 3), (17, 1024)])
def test_requests_of_many_rows(fsr, oracle, copies, width, drop, suffix_close):
    """Requests around the multiples of 8 rows, which are read together, up to 49; 374 rows, and 6358, which take one launch or two by the size of a row."""
    announce(f"many rows copies={copies} width={width} drop={drop} suffix_close={suffix_close}")
    lens = np.tile([0, 1, 7, 8, 9, 15, 16, 17, 24, 31, 32, 33, 47, 48, 49, 2, 3, 0, 20, 2, 10], copies)
    cu = workloads.exclusive_offsets(lens)
    N = int(cu[-1])
    assert N == 374 * copies
    rng = np.random.default_rng(width + copies)
    pay = rng.integers(-1000, 1000, size=(N, width)).astype(np.int32)
    _compare(fsr, oracle, (rng.random(N) >= drop).astype(np.uint8), cu, suffix_close, pay, N)


@pytest.mark.parametrize("suffix_close", [True, False])
@pytest.mark.parametrize("seed,B,maxlen,width", [(0, 1, 5, 4), (1, 37, 9, 6), (2, 512, 11, 64), (3, 2500, 4, 3), (4, 300, 0, 4)])
def test_prune_random(fsr, oracle, suffix_close, seed, B, maxlen, width):
    announce(f"prune_random seed={seed} B={B} suffix_close={suffix_close}")
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, maxlen + 1, size=B)
    cu = workloads.exclusive_offsets(lens)
    N = int(cu[-1])
    N_cap = N + 5
    keep = ((rng.random(N_cap) < 0.75) * rng.integers(1, 255, size=N_cap)).astype(np.uint8)
    pay = rng.integers(-1000, 1000, size=(N_cap, width)).astype(np.int32)
    _compare(fsr, oracle, keep, cu, suffix_close, pay, N_cap)


def test_prune_all_keep_all_drop_and_figure_shape(fsr, oracle):
    announce("prune identities")
    cu = workloads.exclusive_offsets(np.array([4, 4, 4]))
    pay = np.arange(12 * 8, dtype=np.int32).reshape(12, 8)
    for keep in (np.ones(12, np.uint8), np.zeros(12, np.uint8),
                 np.array([1, 1, 0, 0, 1, 1, 1, 1, 1, 0, 0, 0], np.uint8)):
        _compare(fsr, oracle, keep, cu, True, pay, 12)


def test_prune_wide_rows_16B_path(fsr, oracle):
    announce("prune wide bf16-like rows")
    rng = np.random.default_rng(9)
    lens = rng.integers(1, 10, size=64)
    cu = workloads.exclusive_offsets(lens)
    N = int(cu[-1])
    keep = (rng.random(N) < 0.6).astype(np.uint8)
    pay = rng.integers(-2**31, 2**31 - 1, size=(N, 2048), dtype=np.int64).astype(np.int32)  # 8 KB rows
    _compare(fsr, oracle, keep, cu, True, pay, N)


@pytest.mark.parametrize("seed,B,maxlen", [(0, 1, 5), (1, 37, 9), (2, 700, 11), (3, 2500, 4)])
def test_survivor_compact_equals_mask_then_compact(fsr, oracle, seed, B, maxlen):
    """The one-call form (accepted lengths in, re-packed batch out) against the oracle's mask + compaction and
    against the two separate calls, bit for bit; invalid requests (accepted_len = -1) keep nothing."""
    announce(f"survivor_compact seed={seed} B={B}")
    rng = np.random.default_rng(100 + seed)
    lens = rng.integers(0, maxlen + 1, size=B)
    cu = workloads.exclusive_offsets(lens)
    N = int(cu[-1])
    N_cap = N + 3
    acc = rng.integers(-1, maxlen + 2, size=B).astype(np.int32)      # some beyond the request's rows, some -1
    pay = rng.integers(-1000, 1000, size=(N_cap, 8)).astype(np.int32)
    keep_ref = np.concatenate([np.arange(l) <= a for l, a in zip(lens, acc)] + [np.zeros(0, bool)]).astype(np.uint8)
    ref = oracle.prune_compact(keep_ref, cu, suffix_close=True, payload=pay[:N])
    keep_d = torch.full((N_cap,), 9, dtype=torch.uint8, device="cuda")
    r = fsr.survivor_compact(dev(acc), dev(cu), N_cap, keep_mask=keep_d, payload=dev(pay))
    keep2 = torch.full((N_cap,), 9, dtype=torch.uint8, device="cuda")
    fsr.survivor_mask(dev(acc), dev(cu), keep2)
    r2 = fsr.prune_compact(keep2, dev(cu), suffix_close=True, payload=dev(pay))
    torch.cuda.synchronize()
    n_new = int(ref["new_cu_q"][-1])
    assert np.array_equal(keep_d.cpu().numpy()[:N], keep_ref) and (keep_d.cpu().numpy()[N:] == 9).all()
    assert torch.equal(keep_d, keep2)
    for name in ("new_cu_q", "new_q_lens", "src_row", "dst_row", "n_active", "active_ids"):
        assert torch.equal(r[name], r2[name]), name
    assert np.array_equal(r["new_cu_q"].cpu().numpy(), ref["new_cu_q"])
    assert np.array_equal(r["src_row"].cpu().numpy()[:N], ref["src_row"])
    assert np.array_equal(r["dst_row"].cpu().numpy()[:N], ref["dst_row"])
    assert np.array_equal(r["payload"].cpu().numpy()[:n_new], ref["payload"])
    # without the optional mask output
    r3 = fsr.survivor_compact(dev(acc), dev(cu), N_cap)
    torch.cuda.synchronize()
    assert torch.equal(r3["src_row"], r["src_row"])


@pytest.mark.parametrize("width", [4, 1025, 5000])  # words of a payload row; 0 bytes of it would not need the offsets
@pytest.mark.parametrize("B,maxlen", [(1, 8), (37, 9), (1500, 9)])
def test_offsets_replaced_in_place(fsr, oracle, B, maxlen, width):
    """new_cu_q is cu_q itself, new_q_lens accepted_len itself: the payload rows must come from the offsets as they were."""
    announce(f"prune in place B={B} width={width}")
    rng = np.random.default_rng(B + width)
    lens = rng.integers(1, maxlen + 1, size=B)
    acc = np.minimum(rng.integers(-1, maxlen, size=B), lens - 1).astype(np.int32)
    cu = workloads.exclusive_offsets(lens)
    N = int(cu[-1])
    keep = np.concatenate([np.arange(n) <= a for n, a in zip(lens, acc)]).astype(np.uint8)
    pay = rng.integers(-1000, 1000, size=(N, width)).astype(np.int32)
    ref = oracle.prune_compact(keep, cu, suffix_close=True, payload=pay)
    n_new = int(ref["new_cu_q"][-1])
    for survivors in (True, False):
        cu_d, acc_d = dev(cu), dev(acc)
        if survivors:
            r = fsr.survivor_compact(acc_d, cu_d, N, payload=dev(pay), out=dict(new_cu_q=cu_d, new_q_lens=acc_d))
        else:
            r = fsr.prune_compact(dev(keep), cu_d, payload=dev(pay), out=dict(new_cu_q=cu_d))
        torch.cuda.synchronize()
        assert r["new_cu_q"] is cu_d
        for name in ("new_cu_q", "new_q_lens", "src_row", "dst_row", "active_ids"):
            assert np.array_equal(r[name].cpu().numpy(), ref[name]), name
        assert np.array_equal(r["payload"].cpu().numpy()[:n_new], ref["payload"])
