"""Keys whose logits are -inf (a bias channel of -inf, as padding masks make
them) weigh 0 wherever they lie: at the start of a list, over whole key blocks,
at the start of a run, key split or chunk.  Against fp64 torch.  And a logit that is a
NaN leaves no finite saliency."""
import math

import pytest
import torch

import paper_2608_15522_amd as sa

pytestmark = pytest.mark.gpu

# key ranges of -inf logits, of L = 8200 keys: one key first, several tiles
# first, across and inside the blocks that runs, splits and chunks begin at
L = 8200
SEGMENTS = {"first1": (0, 1), "first200": (0, 200), "mid": (512, 600), "blocks": (1024, 1664),
            "half": (4100, 8200), "single": (2733, 2734)}


def _randn(*shape, seed, dtype):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(*shape, generator=g, device="cuda").to(dtype)


def _masked_inputs(H, Lq, d, seg, dtype):
    """q [1,H,Lq,d] with a bias channel of ones, k, v [1,H,L,d] with -inf there
    on the keys of `seg`, and the fp64 probabilities and row LSEs."""
    q = _randn(1, H, Lq, d, seed=1, dtype=dtype)
    k, v = (_randn(1, H, L, d, seed=i, dtype=dtype) for i in (2, 3))
    q[..., 0] = 1
    k[:, :, slice(*SEGMENTS[seg]), 0] = -math.inf
    s = d**-0.5 * (q[0].double() @ k[0].double().transpose(1, 2).contiguous())
    return q, k, v, torch.softmax(s, 2), torch.logsumexp(s, 2)


def _rows_close(o, ref, rel):
    """2-norm over a row's channels, relative to the row."""
    assert torch.isfinite(o).all()
    assert ((o.double() - ref).norm(dim=-1) <= rel * ref.norm(dim=-1)).all()


# bf16: P and O are rounded to 2^-9 each, independently from key to key: 2.3e-3
# of a row's norm, taken four times; fp32: the bound of the other parity tests
# (1e-5 on values near 1) on rows of norm sqrt(d / keys) or so
REL_O = {torch.bfloat16: 1e-2, torch.float32: 1e-5}
TOL_LSE = {torch.bfloat16: 2.5e-3, torch.float32: 1e-5}


@pytest.mark.parametrize("seg", SEGMENTS)
@pytest.mark.parametrize("d,block,dtype", [(128, 128, torch.bfloat16), (64, 64, torch.bfloat16),
                                           (128, 64, torch.bfloat16), (64, 128, torch.bfloat16),
                                           (64, 64, torch.float32), (128, 128, torch.float32)])
def test_attention(seg, d, block, dtype):
    H = 2
    print(f"case -inf attention {seg} d={d} block={block} {dtype}", flush=True)
    q, k, v, p, lse_ref = _masked_inputs(H, L, d, seg, dtype)
    ref = p @ v[0].double()
    del p
    n_b = -(-L // block)
    idx = torch.arange(n_b, dtype=torch.int32, device="cuda").expand(1, H, n_b, n_b).contiguous()
    cnt = torch.full((1, H, n_b), n_b, dtype=torch.int32, device="cuda")
    # lists in one piece, and with room to cut them into runs
    least = 2 * -(-4 * H * n_b // 256) * 256 + 2048
    full = sa.sa_workspace_size(sa.SA_CALL_SPARSE_ATTENTION, 1, H, L, 1, d, block)
    for n in (least, full):
        ws = torch.zeros(n, dtype=torch.uint8, device="cuda")
        o, lse = sa.sa_sparse_attention(q, k, v, d**-0.5, block, idx, cnt, want_lse=True, ws=ws)
        _rows_close(o[0], ref, REL_O[dtype])
        assert (lse[0].double() - lse_ref).abs().max() <= TOL_LSE[dtype]
    # dense rows of chosen tokens (key splits)
    tok = torch.arange(0, L, 7, dtype=torch.int32, device="cuda")[None].contiguous()
    o, lse = torch.zeros_like(q), torch.zeros(1, H, L, device="cuda")
    sa.sa_protected_token_attention(q, k, v, d**-0.5, tok, o, lse)
    at = tok[0].long()
    _rows_close(o[0][:, at], ref[:, at], REL_O[dtype])
    assert (lse[0][:, at].double() - lse_ref[:, at]).abs().max() <= TOL_LSE[dtype]


@pytest.mark.parametrize("seg", SEGMENTS)
@pytest.mark.parametrize("d", [64, 128])
def test_cross_attention(seg, d):
    print(f"case -inf cross attention {seg} d={d}", flush=True)
    q, k, v, p, lse_ref = _masked_inputs(2, 300, d, seg, torch.bfloat16)
    o, lse = sa.sa_cross_attention(q, k, v, d**-0.5, want_lse=True)
    _rows_close(o[0], p @ v[0].double(), REL_O[torch.bfloat16])
    assert (lse[0].double() - lse_ref).abs().max() <= TOL_LSE[torch.bfloat16]


def _check_saliency(L_a, d, seg, dtype, rel):
    H = 2
    q, k, _, p, _ = _masked_inputs(H, L_a, d, seg, dtype)
    ref = p.sum((0, 1)) / (H * L_a)
    got = sa.sa_cross_scores(q, k, None, None, d**-0.5, 64)[0][0].double()
    assert torch.isfinite(got).all()
    assert ((got - ref).abs() <= rel * ref).all()  # masked keys: exactly 0


# whole and ragged 16-query tiles; the bound of the other fp32 saliency tests
@pytest.mark.parametrize("seg", SEGMENTS)
@pytest.mark.parametrize("L_a,d", [(512, 128), (37, 128), (512, 64), (37, 64)])
def test_saliency_f32(seg, L_a, d):
    print(f"case -inf saliency f32 {seg} L_a={L_a} d={d}", flush=True)
    _check_saliency(L_a, d, seg, torch.float32, 1e-5)


# scales whose fp32 product with log2(e) is above and below the exact one
@pytest.mark.parametrize("scale", [1.0, 0.5, 0.3, 0.1, 0.07, 0.044194174, 0.01, 1e-6])
def test_saliency_f32_of_any_scale(scale):
    print(f"case -inf saliency f32 scale={scale}", flush=True)
    q, k, _, _, _ = _masked_inputs(1, 40, 64, "mid", torch.float32)
    ref = torch.softmax(torch.tensor(scale).double() * (q[0, 0].double() @ k[0, 0].double().T.contiguous()), 1)
    got = sa.sa_cross_scores(q, k, None, None, scale, 64)[0][0].double()
    # logits of up to 40: 2^-24 * 40 of a weight, thrice
    assert ((got - ref.sum(0) / 40).abs() <= 1e-5 * ref.sum(0) / 40).all()


# L_a = 512: whole query slabs, as rows past L_a hold zeros (0 * -inf); chunks of
# 128 to 1024 video keys by the number of heads.  The bound of the other bf16
# saliency tests.
@pytest.mark.parametrize("seg", SEGMENTS)
@pytest.mark.parametrize("d", [64, 128])
def test_saliency_bf16(seg, d):
    print(f"case -inf saliency bf16 {seg} d={d}", flush=True)
    _check_saliency(512, d, seg, torch.bfloat16, 1e-4)


def test_rows_of_infinite_logits_only():
    """A list whose keys all carry -inf logits has no key that weighs: zeros
    and lse = -inf, as for a list without a valid entry."""
    H, n_b, d, block = 1, 70, 64, 64
    n = n_b * block
    q, k, v = (_randn(1, H, n, d, seed=i, dtype=torch.bfloat16) for i in (1, 2, 3))
    q[..., 0] = 1
    k[:, :, :2 * block, 0] = -math.inf
    idx = torch.arange(n_b, dtype=torch.int32, device="cuda").expand(1, H, n_b, n_b).contiguous()
    cnt = torch.full((1, H, n_b), 2, dtype=torch.int32, device="cuda")
    o, lse = sa.sa_sparse_attention(q, k, v, d**-0.5, block, idx, cnt, want_lse=True)
    assert (o == 0).all() and torch.isneginf(lse).all()


@pytest.mark.parametrize("L_v", [700, 8200])  # chunks of 128 and more keys
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_saliency_with_a_nan_key(L_v, dtype):
    """The normaliser of every query is a NaN, and so is all it divides."""
    print(f"case NaN saliency L_v={L_v} {dtype}", flush=True)
    q, k = (_randn(1, 2, n, 64, seed=i, dtype=dtype) for i, n in ((1, 512), (2, L_v)))
    k[0, 0, L_v // 2, 5] = math.nan
    v_tok, v_blk, _ = sa.sa_cross_scores(q, k, None, None, 0.125, 64)
    assert torch.isnan(v_tok).all() and torch.isnan(v_blk).all()
