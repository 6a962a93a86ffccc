"""Recall of few rows per key (Q < 16, or batches split over the keys; fewer keys
or more rows take the other paths): gates
from the candidate lists, one scan of the keys for a KV group's rows, float64
decisions.  Exact sets and hits against float64 numpy."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
S = pytest.importorskip("paper_2608_03228_amd.saki")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 128


def _inputs(seed, B, H_q, H_kv, N, Q, bf16, mean=0.0):
    rng = np.random.default_rng(seed)
    scale = np.arange(1, D + 1) ** -0.5
    keys = torch.from_numpy(((rng.standard_normal((B, H_kv, N + 5, D)) + mean) * scale).astype(np.float32))
    q = torch.from_numpy((rng.standard_normal((B, H_q, Q, D)) * scale).astype(np.float32))
    return keys.to(torch.bfloat16) if bf16 else keys, q


def _exact(keys, q, N, k, pos):
    """Exact lists [B, H_q, Q, k] (score descending, index ascending, -1 past a
    row's keys) from float64 scores."""
    B, H_q, Q, _ = q.shape
    G = H_q // keys.shape[1]
    lim = O.candidate_limits(Q, N, pos)
    out = np.full((B, H_q, Q, k), -1, np.int32)
    for b in range(B):
        for h in range(H_q):
            s = q[b, h].double().numpy() @ keys[b, h // G, :N].double().numpy().T
            for i in range(Q):
                best = np.lexsort((np.arange(lim[i]), -s[i, :lim[i]]))[:k]
                out[b, h, i, :len(best)] = best
    return out


def _check(keys, q, N, k, approx, pos=None, ws=None):
    want = _exact(keys, q, N, k, pos)
    p = None if pos is None else torch.from_numpy(np.asarray(pos, np.int32)).to(DEV)
    args = (keys.to(DEV), q.to(DEV), torch.from_numpy(approx).to(DEV), N)
    for full in (True, False):
        hits, ex = S.saki_recall(*args, q_pos=p, k=k, want_exact=full, ws=ws)
        if full:
            np.testing.assert_array_equal(ex.cpu().numpy(), want)
        np.testing.assert_array_equal(hits.cpu().numpy(), O.recall_hits(approx, want))


def _near(want, N, seed):
    """Lists like an index's: the exact ones with a few entries replaced."""
    rng = np.random.default_rng(seed)
    out = want.copy()
    for row in out.reshape(-1, out.shape[-1]):
        free = np.setdiff1d(np.arange(N), row)
        n = min(len(row) // 10, len(free))
        row[len(row) - n:] = rng.permutation(free)[:n]
    return out


# one key block, its edges, several chunks; 1, 2 and more column blocks; both
# key types; lists shorter than a wave
@pytest.mark.parametrize("B,H_q,H_kv,N,Q,k,bf16", [
    (1, 4, 1, 65, 1, 64, False), (2, 2, 2, 255, 3, 64, True), (1, 8, 1, 257, 2, 10, False),
    (1, 8, 2, 1001, 5, 64, False), (2, 7, 1, 3000, 15, 32, True), (1, 4, 2, 20011, 1, 64, False),
    (1, 2, 1, 9000, 17, 64, False), (1, 4, 1, 70001, 16, 64, True)])
def test_recall_once_matches_float64(B, H_q, H_kv, N, Q, k, bf16):
    keys, q = _inputs(N + Q, B, H_q, H_kv, N, Q, bf16)
    _check(keys, q, N, k, _near(_exact(keys, q, N, k, None), N, N))


@pytest.mark.parametrize("bf16", [False, True])
def test_recall_once_causal(bf16):
    """Limits inside, at and past the keys, rows with fewer keys than k and none."""
    N, pos = 1500, [-1, 0, 62, 63, 64, 700, 1023, 1024, 1499, 4000]
    keys, q = _inputs(5, 1, 4, 2, N, len(pos), bf16)
    approx = _exact(keys, q, N, 64, pos)
    _check(keys, q, N, 64, approx, pos)


@pytest.mark.parametrize("lists", ["far", "pads", "duplicates"])
def test_recall_once_poor_lists(lists):
    """Lists that give no useful gate: every chunk's list fills and raises its own."""
    N, Q = 30_000, 3
    keys, q = _inputs(9, 1, 4, 1, N, Q, False, mean=0.5)
    want = _exact(keys, q, N, 64, None)
    rng = np.random.default_rng(3)
    approx = np.stack([rng.permutation(N)[:64] for _ in range(4 * Q)]).reshape(1, 4, Q, 64).astype(np.int32)
    if lists == "pads":
        approx = want.copy()
        approx[..., 60:] = -1
    elif lists == "duplicates":
        approx = want.copy()
        approx[..., 63] = approx[..., 0]
    _check(keys, q, N, 64, approx)


def test_recall_once_ties_and_non_finite():
    """Equal keys (a list that cannot shrink: the row is redone) and keys with
    infinite and NaN entries."""
    N = 4000
    keys, q = _inputs(11, 1, 2, 1, N, 2, False)
    keys[0, 0, 100:3000] = keys[0, 0, 50]
    _check(keys, q, N, 64, _exact(keys, q, N, 64, None))
    keys, q = _inputs(12, 1, 2, 1, N, 2, False)
    keys[0, 0, 777, 3] = float("inf")
    keys[0, 0, 778, 3] = float("nan")
    q[:, 0] = q[:, 0].abs()  # +inf for head 0; whatever sign head 1 gives
    kk, B = keys[0, 0, :N].double().numpy(), 64
    want = np.full((1, 2, 2, B), -1, np.int32)
    with np.errstate(invalid="ignore"):
        for h in range(2):
            for i in range(2):
                s = (kk * q[0, h, i].double().numpy()).sum(1)
                s = np.where(np.isnan(s), -np.inf, s)  # never listed
                o = np.lexsort((np.arange(N), -s))[:B]
                want[0, h, i] = o
    hits, ex = S.saki_recall(keys.to(DEV), q.to(DEV), torch.from_numpy(want).to(DEV), N)
    np.testing.assert_array_equal(ex.cpu().numpy(), want)
    assert (hits.cpu().numpy() == B).all()


def test_recall_once_small_workspace():
    """A workspace of the partial lists alone (none for one chunk) is still taken."""
    keys, q = _inputs(13, 1, 2, 1, 1500, 2, False)
    want = _exact(keys, q, 1500, 64, None)
    _check(keys, q, 1500, 64, want, ws=torch.empty(1, dtype=torch.uint8, device=DEV))


# both sides of the rule that chooses the path: keys for a few rows of a head,
# for many rows, and rows of a KV group
@pytest.mark.parametrize("B,H_q,H_kv,N,Q,k", [
    (1, 4, 1, 128, 1, 64), (1, 4, 2, 129, 3, 64), (1, 4, 1, 20, 4, 64), (52, 30, 2, 32, 1, 64),
    (52, 30, 2, 33, 1, 64), (26, 30, 6, 65, 2, 20), (8, 33, 3, 128, 4, 64), (8, 33, 3, 129, 4, 64),
    (8, 28, 4, 256, 11, 64), (8, 28, 4, 257, 11, 64), (8, 28, 4, 352, 15, 64), (8, 28, 4, 353, 15, 64), (1, 16, 1, 4100, 40, 64), (1, 8, 1, 4100, 64, 64),
    (1, 17, 1, 8192, 31, 64)])
def test_recall_path_rule(B, H_q, H_kv, N, Q, k):
    keys, q = _inputs(N + Q, B, H_q, H_kv, N, Q, False)
    _check(keys, q, N, k, _near(_exact(keys, q, N, k, None), N, N))


def test_recall_of_many_rows_over_few_keys():
    """30,720 rows over 64 keys: decided row by row from scanned lists 760 us, one
    wave per four rows 204."""
    B, H, Q, N = 64, 32, 15, 64
    g = torch.Generator(device=DEV).manual_seed(0)
    keys, q = (torch.randn((B, h, n, D), generator=g, device=DEV) for h, n in ((8, N), (H, Q)))
    lists = torch.argsort(torch.rand((B, H, Q, N), generator=g, device=DEV), dim=-1).int().contiguous()
    ws = torch.empty(max(1, S.saki_recall_workspace_bytes(B, H, 8, Q, N, D, 64)), dtype=torch.uint8, device=DEV)
    best = float("inf")
    for _ in range(6):
        t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        t0.record()
        hits, _ = S.saki_recall(keys, q, lists, N, ws=ws)
        t1.record()
        t1.synchronize()
        best = min(best, t0.elapsed_time(t1) * 1e3)
    assert (hits == 64).all() and best <= 400


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("which", ["keys", "q"])
def test_recall_of_unaligned_tensors(which, bf16):
    """Keys and queries that begin one element past a 16-byte boundary."""
    N, Q = 1300, 3
    keys, q = _inputs(15, 1, 4, 2, N, Q, bf16)
    want = _exact(keys, q, N, 64, None)

    def odd(t):
        flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)[1:]
        flat.copy_(t.to(DEV).view(-1))
        return flat.view(t.shape)

    args = (odd(keys), q.to(DEV)) if which == "keys" else (keys.to(DEV), odd(q))
    hits, ex = S.saki_recall(*args, torch.from_numpy(want).to(DEV), N)
    assert args[which == "q"].data_ptr() % 16 != 0 and (hits == 64).all()
    np.testing.assert_array_equal(ex.cpu().numpy(), want)
