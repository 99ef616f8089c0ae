"""How a call's work is cut over the chip: every rule that picks a split by
size (blocks per pooling workgroup, keys per saliency workgroup, parts of the
block ranking, launch schedule of the sparse attention) at sizes on each side
of its lines and at ragged remainders, against plain fp64 torch."""
import numpy as np
import pytest
import torch

import paper_2608_15522_amd as sa
from sa_parity import SAL_ABS, SAL_REL, TOL_LSE, TOL_O

pytestmark = pytest.mark.gpu


def _randn(*shape, seed, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(*shape, generator=g, device="cuda").to(dtype)


@pytest.mark.parametrize("n_b", [1, 31, 32, 33, 257, 2047, 2048])
def test_block_ranking(n_b):
    rng = np.random.default_rng(n_b)
    s = rng.integers(0, max(2, n_b // 3), (2, n_b)).astype(np.float32)  # many ties
    for k in sorted({0, 1, n_b // 3, n_b}):
        idx, flag = sa.sa_select_protected(torch.from_numpy(s).cuda(), k)
        for b in range(2):
            want = np.argsort(-s[b], kind="stable")[:k]
            assert np.array_equal(idx[b].cpu().numpy(), want), (n_b, k)
            ref = np.zeros(n_b, np.uint8)
            ref[want] = 1
            assert np.array_equal(flag[b].cpu().numpy(), ref)


# more batch items than the second and third grid dimensions hold; ranks by sorting
# (many long items), and by counting just below that line
@pytest.mark.parametrize("B,n_b", [(65536 + 7, 1), (65536 + 7, 40), (1217, 257), (1210, 257),
                                   (20, 2048), (19, 2047), (600, 401)])
def test_block_ranking_of_many_items(B, n_b):
    print(f"case ranking B={B} n_b={n_b}", flush=True)
    s = _randn(B, n_b, seed=n_b, dtype=torch.float32).round_(decimals=1)  # ties
    k = (n_b + 2) // 3
    idx, flag = sa.sa_select_protected(s, k)
    want = torch.sort(s, dim=1, descending=True, stable=True)[1][:, :k]
    assert torch.equal(idx.long(), want)
    ref = torch.zeros_like(flag).scatter_(1, want, 1)
    assert torch.equal(flag, ref)


# 1, 2, 4 and 8 blocks per pooling workgroup (384 workgroups are wanted)
@pytest.mark.parametrize("H,n_b,tail,dtype", [(24, 7, 5, torch.bfloat16), (64, 12, 9, torch.bfloat16),
                                              (64, 24, 64, torch.bfloat16),
                                              (64, 47, 1, torch.float32), (64, 97, 33, torch.bfloat16)])
def test_pooled_scores(H, n_b, tail, dtype):
    d, block = 64, 64
    L = (n_b - 1) * block + tail
    print(f"case pooling H={H} n_b={n_b} tail={tail} {dtype}", flush=True)
    q, k = (_randn(1, H, L, d, seed=i, dtype=dtype) for i in (1, 2))
    G = sa.sa_build_block_mask(q, k, 0.125, block, 1, want_scores=True)[3]

    def mean(x):
        x = torch.nn.functional.pad(x.double(), (0, 0, 0, n_b * block - L))
        n = torch.full((n_b, 1), float(block), dtype=torch.float64, device="cuda")
        n[-1] = tail
        return x.view(H, n_b, block, d).sum(2) / n

    ref = 0.125 * torch.stack([a @ b.T.contiguous() for a, b in zip(mean(q[0]), mean(k[0]))])
    assert ((G[0].double() - ref).abs() <= 2.0**-24 * ref.abs() + 1e-12).all()


# audio slabs 1 and 2; chunks of 128 to 1024 video keys, more than 16 of them
@pytest.mark.parametrize("H,L_v,L_a,d", [(1, 2100, 40, 64), (3, 32760, 512, 128), (7, 9001, 513, 64),
                                         (24, 16000, 70, 128)])
def test_saliency_chunks(H, L_v, L_a, d):
    print(f"case saliency H={H} L_v={L_v} L_a={L_a} d={d}", flush=True)
    scale = d**-0.5
    q_a, k_a = (_randn(1, H, L_a, d, seed=i) for i in (1, 2))
    q_v, k_v = (_randn(1, H, L_v, d, seed=i) for i in (3, 4))
    ref_v = torch.zeros(L_v, dtype=torch.float64, device="cuda")
    ref_a = torch.zeros(L_a, dtype=torch.float64, device="cuda")
    lse_a = torch.empty(1, H, L_a, device="cuda")
    lse_v = torch.empty(1, H, L_v, device="cuda")
    for h in range(H):
        s = scale * (q_a[0, h].double() @ k_v[0, h].double().T.contiguous())
        lse_a[0, h] = torch.logsumexp(s, 1)
        ref_v += torch.softmax(s, 1).sum(0) / (H * L_a)
        s = scale * (q_v[0, h].double() @ k_a[0, h].double().T.contiguous())
        lse_v[0, h] = torch.logsumexp(s, 1)
        ref_a += torch.softmax(s, 1).sum(0) / (H * L_v)
    n_b = -(-L_v // 128)
    ref_b = torch.nn.functional.pad(ref_v, (0, n_b * 128 - L_v)).view(n_b, 128).sum(1)
    for got in (sa.sa_cross_scores(q_a, k_v, q_v, k_a, scale, 128),
                sa.sa_cross_scores_from_lse(q_a, k_v, q_v, k_a, lse_a, lse_v, scale, 128),
                sa.sa_cross_scores_pooled(q_a, k_v, q_v, k_a, scale, 128)[:3]):
        for x, ref in zip(got, (ref_v, ref_b, ref_a)):
            assert ((x[0].double() - ref).abs() <= SAL_REL * ref + SAL_ABS).all()


# pair counts that are no multiple of 8, fewer than 8, and a multiple; lists of
# every length; rows that go out directly (at most one a CU, at most what the chip
# holds at once, short pairs, a small call) and by the schedule
@pytest.mark.parametrize("H,n_b,tail,d,block", [
    (3, 20, 7, 128, 128), (5, 110, 128, 128, 128), (12, 87, 50, 64, 64), (8, 65, 1, 64, 128),
    (1, 600, 64, 128, 64), (17, 31, 64, 128, 64), (20, 25, 7, 128, 64), (16, 63, 1, 64, 64),
    (700, 4, 30, 64, 64), (40, 33, 9, 128, 128), (71, 61, 5, 64, 64)])
def test_sparse_attention_schedule(H, n_b, tail, d, block):
    L = (n_b - 1) * block + tail
    print(f"case schedule H={H} n_b={n_b} tail={tail} d={d} block={block}", flush=True)
    rng = np.random.default_rng(n_b)
    idx = np.full((1, H, n_b, n_b), -1, np.int32)
    cnt = rng.integers(0, min(n_b, 24) + 1, (1, H, n_b)).astype(np.int32)
    cnt[0, rng.integers(0, H, 4), rng.integers(0, n_b, 4)] = n_b  # full rows
    cnt[0, H - 1, n_b - 1] = n_b
    for h in range(H):
        for r in range(n_b):
            idx[0, h, r, :cnt[0, h, r]] = np.sort(rng.permutation(n_b)[:cnt[0, h, r]])
    q, k, v = (_randn(1, H, L, d, seed=i) for i in (1, 2, 3))
    scale = d**-0.5
    o, lse = sa.sa_sparse_attention(q, k, v, scale, block, torch.from_numpy(idx).cuda(),
                                    torch.from_numpy(cnt).cuda(), want_lse=True)
    members = torch.arange(L, device="cuda") // block
    for h in range(H):
        qd, kd, vd = (x[0, h].double() for x in (q, k, v))
        for r in range(n_b):
            rows = slice(r * block, min(L, (r + 1) * block))
            if cnt[0, h, r] == 0:
                assert (o[0, h, rows] == 0).all() and torch.isneginf(lse[0, h, rows]).all()
                continue
            keep = torch.zeros(n_b, dtype=torch.bool, device="cuda")
            keep[torch.from_numpy(idx[0, h, r, :cnt[0, h, r]]).long().cuda()] = True
            at = keep[members].nonzero()[:, 0]
            p = torch.softmax(scale * (qd[rows] @ kd[at].T.contiguous()), 1)
            assert (o[0, h, rows].double() - p @ vd[at]).abs().max() <= TOL_O["bf16"], (h, r)


def _uses_runs(ws, H, n_b, d, block):
    """What the schedule wrote behind the least workspace: (row, entry) of every
    run's first entry, one more, and whether the runs are used."""
    least = 2 * -(-4 * H * n_b // 256) * 256 + 2048
    slots = 1024 if d == 64 and block == 64 else 512
    return bool(ws[least:least + 8 * (slots + 2)].view(torch.int32)[2 * (slots + 1)].item())


# Lists cut into equal runs: the shortest lists that are cut and the most rows,
# rows held by many runs, runs of several rows, empty and full rows, entries
# outside the range, a tail block; and calls on the other side of the decision.
# Against the same lists in one piece (a workspace without room for the partial
# rows): P is rounded against another running maximum, so that a row's channels
# differ by independent roundings of 2^-9 a term (2.3e-3 of the row's norm at each
# side, 1e-2 taken; without one of n parts about n^-1/2), and the lse by that of its
# bf16 row sum.  Full rows and some others against fp64; the entry point without a
# workspace gives the same bits.
@pytest.mark.parametrize("H,n_b,tail,d,block,kind,cut", [
    (1, 64, 64, 128, 64, "full", True), (32, 64, 3, 128, 128, "mixed", False),
    (32, 64, 3, 128, 128, "thin", True), (1, 65, 1, 64, 128, "one", True),
    (9, 70, 33, 64, 64, "one", True), (3, 256, 120, 128, 128, "mixed", True),
    (5, 200, 64, 64, 64, "mixed", True), (4, 128, 17, 64, 128, "mixed", True),
    (2, 70, 9, 64, 64, "empty", False)])
def test_sparse_attention_runs(H, n_b, tail, d, block, kind, cut):
    L = (n_b - 1) * block + tail
    print(f"case runs H={H} n_b={n_b} tail={tail} d={d} block={block} {kind}", flush=True)
    rng = np.random.default_rng(n_b + H)
    cnt = {"full": np.full((1, H, n_b), n_b), "empty": np.zeros((1, H, n_b)),
           "one": np.zeros((1, H, n_b)), "thin": rng.integers(0, 3, (1, H, n_b)),
           "mixed": rng.integers(0, n_b // 4 + 1, (1, H, n_b))}[kind].astype(np.int32)
    if kind in ("one", "thin"):
        cnt[0, :, n_b - 1] = n_b
    if kind == "mixed":
        cnt[0, :, rng.integers(0, n_b, n_b // 16)] = n_b
    idx = np.full((1, H, n_b, n_b), -1, np.int32)
    for h in range(H):
        for r in range(n_b):
            idx[0, h, r, :cnt[0, h, r]] = np.sort(rng.permutation(n_b)[:cnt[0, h, r]])
    idx[0, 0, n_b // 2, :2] = (-3, n_b)  # ignored
    lists = idx, cnt
    idx, cnt = torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda()
    q, k, v = (_randn(1, H, L, d, seed=i) for i in (1, 2, 3))
    need = sa.sa_workspace_size(sa.SA_CALL_SPARSE_ATTENTION, 1, H, L, 1, d, block)
    least = 2 * -(-4 * H * n_b // 256) * 256 + 2048
    assert need > least
    out = []
    for n in (need, least):
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
        out.append(sa.sa_sparse_attention(q, k, v, d**-0.5, block, idx, cnt, want_lse=True, ws=ws))
        if n == need:
            assert _uses_runs(ws, H, n_b, d, block) == cut
    with pytest.raises(sa.binding.SaError):
        sa.sa_sparse_attention(q, k, v, d**-0.5, block, idx, cnt, ws=ws[:least - 1])
    (o, lse), (o1, lse1) = out

    def close(got, ref):
        assert ((got.double() - ref).norm(dim=-1) <= 1e-2 * ref.norm(dim=-1)).all()

    close(o, o1.double())
    assert cut or torch.equal(o, o1)
    assert torch.equal(torch.isneginf(lse), torch.isneginf(lse1))
    some = ~torch.isneginf(lse1)
    assert (o[~some] == 0).all()
    if some.any():
        assert (lse - lse1)[some].abs().max() <= 2 * TOL_LSE["bf16"]
    members = torch.arange(L, device="cuda") // block
    full = np.argwhere(lists[1][0] == n_b)
    other = np.argwhere(lists[1][0] < n_b)
    for h, r in [*rng.permutation(full)[:8], *rng.permutation(other)[:4]]:
        rows = slice(r * block, min(L, (r + 1) * block))
        lst = lists[0][0, h, r, :lists[1][0, h, r]]
        keep = torch.zeros(n_b, dtype=torch.bool, device="cuda")
        keep[torch.from_numpy(lst[(lst >= 0) & (lst < n_b)]).long().cuda()] = True
        at = keep[members].nonzero()[:, 0]
        if len(at) == 0:
            assert (o[0, h, rows] == 0).all()
            continue
        s = d**-0.5 * (q[0, h, rows].double() @ k[0, h, at].double().T.contiguous())
        close(o[0, h, rows], torch.softmax(s, 1) @ v[0, h, at].double())
        assert (lse[0, h, rows].double() - torch.logsumexp(s, 1)).abs().max() <= TOL_LSE["bf16"]
    o2, lse2 = torch.full_like(o, float("nan")), torch.full_like(lse, float("nan"))
    sa.sa_sparse_attention_noalloc(q, k, v, d**-0.5, block, idx, cnt, o2, lse2)
    assert torch.equal(o.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, lse2)


# fp32 saliency: 16-wave and 4-wave column masses, key chunks of 256 to 1024
# keys and of a sixteenth of the clip, two windows of audio queries, tails of
# one row.  A term's error is that of its logit (2^-24 of |s| <= 8 or so, twice)
# and of the sums' few roundings, relative to a positive sum: 1e-5 covers it.
@pytest.mark.parametrize("H,L_v,L_a,d", [(2, 1024, 128, 64), (1, 300, 5, 128), (4, 4680, 513, 128),
                                         (8, 2100, 40, 64), (1, 16500, 33, 64)])
def test_saliency_f32_chunks(H, L_v, L_a, d):
    print(f"case saliency f32 H={H} L_v={L_v} L_a={L_a} d={d}", flush=True)
    scale = float(np.float32(d**-0.5))
    q_a, k_a = (_randn(1, H, L_a, d, seed=i, dtype=torch.float32) for i in (1, 2))
    q_v, k_v = (_randn(1, H, L_v, d, seed=i, dtype=torch.float32) for i in (3, 4))
    ref_v = torch.zeros(L_v, dtype=torch.float64, device="cuda")
    ref_a = torch.zeros(L_a, dtype=torch.float64, device="cuda")
    for h in range(H):
        ref_v += torch.softmax(scale * (q_a[0, h].double() @ k_v[0, h].double().T.contiguous()), 1).sum(0)
        ref_a += torch.softmax(scale * (q_v[0, h].double() @ k_a[0, h].double().T.contiguous()), 1).sum(0)
    v_tok, _, a_tok = sa.sa_cross_scores(q_a, k_v, q_v, k_a, scale, 64)
    for x, ref in ((v_tok, ref_v / (H * L_a)), (a_tok, ref_a / (H * L_v))):
        assert ((x[0].double() - ref).abs() <= 1e-5 * ref).all()
    only_v = sa.sa_cross_scores(q_a, k_v, None, None, scale, 64)[0]  # one direction
    assert ((only_v[0].double() - ref_v / (H * L_a)).abs() <= 1e-5 * ref_v / (H * L_a)).all()


# token selection by digits of eight bits: both sides of every register form,
# keys that differ in the last bits only, in the sign, in few values, in none, in
# few tokens (a wave's keys that share their digits are added together)
@pytest.mark.parametrize("L", [1, 65, 512, 513, 4096, 4097, 16385, 32768, 32769, 70001])
@pytest.mark.parametrize("kind", ["map", "adjacent", "signs", "few", "equal", "floor", "one"])
def test_token_selection_digits(L, kind):
    rng = np.random.default_rng(L)
    s = {"map": np.exp(rng.standard_normal((2, L))),
         "adjacent": (np.float32(1.0).view(np.int32) + rng.integers(0, 300, (2, L))).astype(np.int32)
         .view(np.float32),
         "signs": rng.standard_normal((2, L)) * 10.0 ** rng.integers(-30, 30, (2, L)),
         "few": rng.integers(-2, 3, (2, L)) * 0.25, "equal": np.full((2, L), 0.5),
         "floor": np.where(np.arange(L) % 97 < L % 97, rng.random((2, L)), 1e-3),
         "one": np.where(np.arange(L) == L // 2, 2.0, np.full((2, L), 0.5))}[kind]
    s = s.astype(np.float32)
    for k in sorted({1, max(1, L // 20), max(1, L - 1)}):
        idx, flag = sa.sa_select_protected_tokens(torch.from_numpy(s).cuda(), k)
        for b in range(2):
            want = np.sort(np.argsort(-s[b], kind="stable")[:k])
            assert np.array_equal(idx[b].cpu().numpy(), want), (L, kind, k)
            ref = np.zeros(L, np.uint8)
            ref[want] = 1
            assert np.array_equal(flag[b].cpu().numpy(), ref)
