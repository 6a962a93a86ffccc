"""Recall hits alone of many rows (rows of at most k keys counted from their
lists) against the call that also wants the exact lists, which
test_gpu_parity.py and test_gpu_recall_once.py pin to float64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
S = pytest.importorskip("paper_2608_03228_amd.saki")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 128


def _case(B, H_q, H_kv, N, Q, start, bf16, seed, mean=0.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    scale = torch.arange(1, D + 1, device=DEV) ** -0.5
    keys = (torch.randn((B, H_kv, N + 3, D), generator=g, device=DEV) + mean) * scale
    q = torch.randn((B, H_q, Q, D), generator=g, device=DEV) * scale
    pos = torch.arange(start, start + Q, dtype=torch.int32, device=DEV) if start is not None else None
    return keys.to(torch.bfloat16).contiguous() if bf16 else keys.contiguous(), q.contiguous(), pos


def _lists(keys, q, pos, N, k, noise, seed):
    """The top k of scores with noise (of their spread) added: an index's lists."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    B, H_q, Q, _ = q.shape
    G = H_q // keys.shape[1]
    out = torch.full((B, H_q, Q, k), -1, dtype=torch.int32, device=DEV)
    for b in range(B):
        for h in range(H_q):
            s = q[b, h] @ keys[b, h // G, :N].float().T
            s = s + noise * s.std() * torch.randn(s.shape, generator=g, device=DEV)
            if pos is not None:
                s.masked_fill_(torch.arange(N, device=DEV)[None] > pos[:, None], -float("inf"))
            v, x = s.topk(min(k, N), dim=1)
            out[b, h, :, :v.shape[1]] = torch.where(v == -float("inf"), -1, x).int()
    return out


def _check(keys, q, pos, N, k, lists):
    want, _ = S.saki_recall(keys, q, lists, N, q_pos=pos, k=k, want_exact=True)
    got, none = S.saki_recall(keys, q, lists, N, q_pos=pos, k=k, want_exact=False)
    assert none is None
    assert torch.equal(got, want), (got != want).nonzero()[:5].tolist()
    return want


# rows that do not fill their last block, causal rows of few keys at the start of
# a block, inside one and alone, list lengths, both key types
@pytest.mark.parametrize("B,H_q,H_kv,N,Q,start,k,bf16", [
    (1, 32, 8, 700, 1030, 0, 64, False), (2, 16, 16, 515, 1030, 10, 10, False), (1, 8, 2, 65, 4099, 0, 64, True),
    (1, 32, 8, 200, 1024, 50, 64, False), (1, 28, 4, 40, 1201, None, 64, False)])
def test_rows_hits(B, H_q, H_kv, N, Q, start, k, bf16):
    keys, q, pos = _case(B, H_q, H_kv, N, Q, start, bf16, N)
    hits = _check(keys, q, pos, N, k, _lists(keys, q, pos, N, k, 0.02, 1))
    assert N <= k or 0.5 * k < hits[..., -1].float().mean().item() <= k


def test_rows_hits_bad_lists():
    """Pads, duplicates and keys past a row's limit, in rows of few keys too."""
    keys, q, pos = _case(1, 32, 8, 900, 1040, 0, False, 5)
    bad = _lists(keys, q, pos, 900, 64, 0.02, 3)
    bad[0, 0, 10:14, 5] = -1
    bad[0, 0, 30:70, 1] = bad[0, 0, 30:70, 0]
    bad[0, 1, 40, 63] = bad[0, 1, 40, 0]
    bad[0, 1, 20:80, 2] = 899
    bad[0, 3, 0] = 10 ** 6
    bad[0, 4, :64] = -7
    _check(keys, q, pos, 900, 64, bad)


def test_rows_hits_non_finite():
    """Keys with infinite and NaN entries and queries of both kinds: scores that
    are no numbers, or -inf, are not counted where the exact set leaves them out,
    also of rows of at most k keys whose list names them."""
    g = torch.Generator(device=DEV).manual_seed(8)
    N, Q = 700, 1040
    keys, q, pos = _case(1, 32, 8, N, Q, 0, False, 6)
    keys[0, 0, 3, 5] = float("nan")
    keys[0, 0, 7] = float("inf")
    keys[0, 1, 9, 2] = -float("inf")
    q[0, 9, 30, 1] = float("nan")
    q[0, 10, 31, 2] = float("inf")
    rank = torch.rand((1, 32, Q, N), generator=g, device=DEV)
    rank.masked_fill_(torch.arange(N, device=DEV) > pos[:, None], 2.0)
    v, lists = rank.sort(dim=-1)
    lists = torch.where(v[..., :64] < 2.0, lists[..., :64], -1).int().contiguous()
    hits = _check(keys, q, pos, N, 64, lists)
    assert hits[0, 0, 20] == 19 and hits[0, 9, 30] == 0  # 21 keys, two without a score; a NaN query
    assert torch.equal(hits[0, 31, :64], torch.arange(1, 65, device=DEV).int())
