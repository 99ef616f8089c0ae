"""Host side of the C ABI, on the CPU: the library loads, exports every symbol
the header declares, sizes workspaces, and rejects bad arguments before any
launch.  No call here reaches a kernel (every call is invalid)."""
import ctypes
import os
import re

import pytest

import paper_2608_15522_amd as sa
from paper_2608_15522_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "sa.h")
BENCH_HEADER = os.path.join(ROOT, "include", "sa_bench.h")

FAKE = 0x10000          # aligned stand-in pointer, never dereferenced
MISALIGNED = 0x10001

pytestmark = pytest.mark.skipif(not os.path.exists(binding.LIB_PATH),
                                reason="libsa.so not built")


def declared_symbols(header=HEADER):
    text = open(header).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sa_[a-z_]+)\s*\(", text)))


def test_exports_every_declared_symbol():
    names = declared_symbols()
    assert set(names) == set(binding.SIGNATURES), names
    lib = sa.lib()
    for n in names:
        assert hasattr(lib, n), n
    assert sa.sa_version() == 100


def test_library_matches_the_sources():
    """The binding refuses a library built from other sources; the one that
    loaded reports the id of the sources in the tree."""
    from paper_2608_15522_amd.srcid import source_id
    assert sa.sa_build_id() == source_id()


@pytest.mark.skipif(not os.path.exists(binding.BENCH_LIB_PATH),
                    reason="libsa_bench.so not built")
def test_bench_library_exports_and_rejects_bad_arguments():
    names = declared_symbols(BENCH_HEADER)
    assert set(names) == set(binding.BENCH_SIGNATURES), names
    lib = binding.bench_lib()
    tf, ghz = ctypes.c_float(), ctypes.c_float()
    # rejected before any device call
    assert lib.sa_bench_mfma_peak(1, 0, 1, ctypes.byref(tf), ctypes.byref(ghz)) == -1
    assert lib.sa_bench_mfma_peak(1, 8, 0, ctypes.byref(tf), ctypes.byref(ghz)) == -1
    assert lib.sa_bench_mfma_peak(1, 8, 1, None, ctypes.byref(ghz)) == -1


def test_workspace_sizes():
    for call in (sa.SA_CALL_CROSS_SCORES, sa.SA_CALL_BUILD_BLOCK_MASK,
                 sa.SA_CALL_SPARSE_ATTENTION):
        a = sa.sa_workspace_size(call, 1, 24, 32760, 512, 128, 128)
        b = sa.sa_workspace_size(call, 2, 24, 75600, 1024, 128, 128)
        assert 0 < a < b
    # attention: the per-head launch order of the query blocks (int32)
    assert sa.sa_workspace_size(sa.SA_CALL_SPARSE_ATTENTION, 1, 24, 32760, 512,
                                128, 128) == 2 * 24 * 256 * 4 + 8 * 64 * 4
    assert sa.sa_workspace_size(sa.SA_CALL_SELECT_PROTECTED, 1, 1, 10, 1, 64, 64) == 0
    for bad in [(0, 1, 10, 1, 64, 64), (1, 1, 10, 1, 96, 64),
                (1, 1, 10, 1, 64, 32), (1, 1, 2049 * 128, 1, 64, 128)]:
        assert sa.sa_workspace_size(sa.SA_CALL_SPARSE_ATTENTION, *bad) == 0
    assert sa.sa_workspace_size(sa.SA_CALL_CROSS_SCORES, 1, 1, 10, 0, 64, 64) == 0
    assert sa.sa_workspace_size(9, 1, 1, 10, 1, 64, 64) == 0
    assert sa.sa_workspace_size(sa.SA_CALL_SPARSE_ATTENTION, 256, 256, 10, 1, 64, 64) == 0
    # cache indicator: 9 fp32 partials per workgroup (1024 video, 64 audio)
    assert sa.sa_workspace_size(sa.SA_CALL_CACHE_INDICATOR, 1, 0, 32760, 512, 0, 0) == \
        ((1024 + 64) * 36 + 255) // 256 * 256
    assert sa.sa_workspace_size(sa.SA_CALL_CACHE_INDICATOR, 1, 0, 10, 0, 0, 0) == 512
    assert sa.sa_workspace_size(sa.SA_CALL_CACHE_INDICATOR, 0, 0, 10, 0, 0, 0) == 0


class _Call:
    """One C entry point with default arguments (keyword order = C order);
    calling it with overrides passes them positionally through ctypes."""

    def __init__(self, name, **defaults):
        self.name, self.defaults = name, defaults

    def args(self, **kw):
        a = dict(self.defaults)
        a.update(kw)
        return list(a.values())

    def __call__(self, **kw):
        return getattr(sa.lib(), self.name)(*self.args(**kw))


def _splits(P, k_tok, n_b):
    """The key-split rule of the protected-token rows, restated."""
    units = P * -(-k_tok // 128)
    smax = min(8, max(1, n_b // 4))
    costs = [(-(-units * s // 512)) / s * (1 + 0.02 * s) for s in range(1, smax + 1)]
    return 1 + min(range(len(costs)), key=lambda i: (costs[i] - 1e-9 * (i == 0), i))


@pytest.mark.parametrize("B,H,L,k_tok,d,splits", [
    (1, 24, 32760, 1638, 128, 3),   # Ovi-like, 5 % of the tokens: 312 row blocks
    (1, 1, 1000, 10, 128, 2),       # one row block, 8 key blocks
    (1, 24, 32760, 100, 64, 8),     # 24 row blocks
    (2, 24, 75600, 3780, 128, 1),   # 1440 row blocks fill the chip
    (1, 1, 300, 5, 64, 1),          # 3 key blocks: no split
])
def test_token_attention_workspace(B, H, L, k_tok, d, splits):
    """Partial rows (d f32 + m, l) per split, none without a split."""
    assert _splits(B * H, k_tok, -(-L // 128)) == splits
    need = sa.sa_workspace_size(sa.SA_CALL_TOKEN_ATTENTION, B, H, L, k_tok, d, 0)
    want = 0 if splits == 1 else (splits * B * H * k_tok * (4 * d + 8) + 255) // 256 * 256
    assert need == want


def test_cross_attention_workspace():
    """The split rule of the gathered rows with Lq rows over Lk keys."""
    # a->v at the Ovi-like shape: 24 x 4 row blocks, 256 key blocks -> 5 runs
    assert _splits(24, 512, 256) == 5
    assert sa.sa_workspace_size(sa.SA_CALL_CROSS_ATTENTION, 1, 24, 512, 32760, 128, 0) == \
        (5 * 24 * 512 * (4 * 128 + 8) + 255) // 256 * 256
    # v->a: 6144 row blocks of 4 key blocks -> no split
    assert sa.sa_workspace_size(sa.SA_CALL_CROSS_ATTENTION, 1, 24, 32760, 512, 128, 0) == 0
    for bad in [(0, 1, 10, 10, 64, 0), (1, 1, 0, 10, 64, 0), (1, 1, 10, 0, 64, 0),
                (1, 1, 10, 10, 96, 0), (1, 1, 10, 262145, 64, 0)]:
        assert sa.sa_workspace_size(sa.SA_CALL_CROSS_ATTENTION, *bad) == 0


def test_fp32_attention_workspace():
    """Partial rows are bf16 calls' only: an fp32 layer of few rows holds no room
    for them (68 MB at d = 128), a bf16 one does."""
    import torch
    from paper_2608_15522_amd.binding import sparse_attention_workspace
    from paper_2608_15522_amd.layer import LayerPlan
    for B, H, L, d, block in [(1, 4, 4680, 128, 64), (1, 2, 9000, 64, 128), (2, 24, 75600, 128, 128)]:
        n_b = -(-L // block)
        least = 2 * -(-4 * B * H * n_b // 256) * 256 + 2048
        full = sa.sa_workspace_size(sa.SA_CALL_SPARSE_ATTENTION, B, H, L, 1, d, block)
        assert sparse_attention_workspace(B, H, L, d, block, torch.float32) == least
        assert sparse_attention_workspace(B, H, L, d, block, torch.bfloat16) == full >= least
    sizes = {}
    for dtype in (torch.float32, torch.bfloat16):
        plan = LayerPlan(1, 4, 4680, 128, 128, 64, 18, 3, 0.088, dtype=dtype, device="cpu")
        sizes[dtype] = plan.ws.numel()
    cross = sa.sa_workspace_size(sa.SA_CALL_CROSS_SCORES, 1, 4, 4680, 128, 128, 64)
    mask = sa.sa_workspace_size(sa.SA_CALL_BUILD_BLOCK_MASK, 1, 4, 4680, 128, 128, 64)
    assert sizes[torch.float32] == max(cross, mask) < 2**23 < sizes[torch.bfloat16]


def test_token_attention_workspace_rejects():
    for bad in [(0, 1, 10, 1, 64, 0), (1, 1, 10, 11, 64, 0), (1, 1, 10, -1, 64, 0),
                (1, 1, 10, 1, 96, 0)]:
        assert sa.sa_workspace_size(sa.SA_CALL_TOKEN_ATTENTION, *bad) == 0
    assert sa.sa_workspace_size(sa.SA_CALL_TOKEN_ATTENTION, 1, 24, 32760, 0, 128, 0) == 0


_attn = _Call("sa_sparse_attention", q=FAKE, k=FAKE, v=FAKE, o=FAKE, lse=None, B=1, H=1, L=1000, d=128,
             dtype=0, scale=0.088, block=128, kv_idx=FAKE, kv_cnt=FAKE, ws=FAKE,
             ws_bytes=1 << 40, stream=None)


_attn_na = _Call("sa_sparse_attention_noalloc", q=FAKE, k=FAKE, v=FAKE, o=FAKE, lse=None, B=1, H=1, L=1000, d=128,
             dtype=0, scale=0.088, block=128, kv_idx=FAKE, kv_cnt=FAKE, stream=None)


_mask = _Call("sa_build_block_mask", q_v=FAKE, k_v=FAKE, B=1, H=1, L_v=1000, d=128, dtype=0, scale=0.088,
             block=128, k_keep=2, prot_flag=None, kv_idx=FAKE, kv_cnt=FAKE,
             mask=None, scores=None, ws=FAKE, ws_bytes=1 << 40, stream=None)


_cross = _Call("sa_cross_scores", q_a=FAKE, k_v=FAKE, q_v=FAKE, k_a=FAKE, B=1, H=1, L_v=1000, L_a=64,
             d=128, dtype=0, scale=0.088, block=128, sal_v_tok=None,
             sal_v_blk=FAKE, sal_a_tok=FAKE, accumulate=0, ws=FAKE,
             ws_bytes=1 << 40, stream=None)


_xfwd = _Call("sa_cross_attention", q=FAKE, k=FAKE, v=FAKE, o=FAKE, lse=None, B=1, H=1, Lq=512, Lk=4000, d=128,
             dtype=0, scale=0.088, ws=FAKE, ws_bytes=1 << 40, stream=None)


_xlse = _Call("sa_cross_scores_from_lse", q_a=FAKE, k_v=FAKE, q_v=FAKE, k_a=FAKE, lse_a=FAKE, lse_v=FAKE, B=1, H=1,
             L_v=1000, L_a=64, d=128, dtype=0, scale=0.088, block=128, sal_v_tok=None,
             sal_v_blk=FAKE, sal_a_tok=FAKE, accumulate=0, ws=FAKE, ws_bytes=1 << 40,
             stream=None)


_xpool = _Call("sa_cross_scores_pooled", q_a=FAKE, k_v=FAKE, q_v=FAKE, k_a=FAKE, lse_a=None, lse_v=None,
               B=1, H=1, L_v=1000, L_a=64, d=128, dtype=0, scale=0.088, block=128,
               sal_v_tok=None, sal_v_blk=FAKE, sal_a_tok=FAKE, accumulate=0, qbar=FAKE,
               kbar=FAKE + (1 << 20), ws=FAKE, ws_bytes=1 << 40, stream=None)


_mpool = _Call("sa_build_block_mask_pooled", qbar=FAKE, kbar=FAKE + (1 << 20), B=1, H=1, L_v=1000, d=128,
               scale=0.088, block=128, k_keep=2, prot_flag=None, kv_idx=FAKE, kv_cnt=FAKE,
               mask=None, scores=None, stream=None)


_select = _Call("sa_select_protected", sal_blk=FAKE, B=1, n_b=8, k_prot=2, prot_idx=None, prot_flag=FAKE,
             stream=None)


_ema = _Call("sa_saliency_ema", sal_bar=FAKE, sal=FAKE, n=1000, alpha=0.5, stream=None)


_tokens = _Call("sa_select_protected_tokens", sal_tok=FAKE, B=1, L=1000, k_tok=50, tok_idx=FAKE, tok_flag=None,
             stream=None)


_ptok = _Call("sa_protected_token_attention", q=FAKE, k=FAKE, v=FAKE, o=FAKE, lse=None, B=1, H=1, L=1000, d=128,
             dtype=0, scale=0.088, tok_idx=FAKE, k_tok=10, ws=FAKE, ws_bytes=1 << 40,
             stream=None)


_cache = _Call("sa_cache_indicator", y_v=FAKE, y_v_hat=FAKE, prot_flag=None, y_a=None, y_a_hat=None,
             s_bar=None, s_hat=None, B=1, L_v=1000, L_a=0, C=64, dtype=0,
             lambda_p=0.5, lambda_s=0.1, tau=0.2, eps=1e-6, out=FAKE, ws=FAKE,
             ws_bytes=1 << 40, stream=None)


INVALID = [
    (_cache, dict(C=12), sa.SA_ERR_INVALID_ARG, "multiple of 8"),
    (_cache, dict(C=0), sa.SA_ERR_INVALID_ARG, "multiple of 8"),
    (_cache, dict(B=1 << 20, L_v=1 << 10, C=1 << 16), sa.SA_ERR_INVALID_ARG, "too large"),
    (_cache, dict(L_v=0), sa.SA_ERR_INVALID_ARG, "L_v=0"),
    (_cache, dict(dtype=3), sa.SA_ERR_UNSUPPORTED, "dtype"),
    (_cache, dict(y_a=FAKE), sa.SA_ERR_INVALID_ARG, "y_a and y_a_hat"),
    (_cache, dict(y_a=FAKE, y_a_hat=FAKE, L_a=0), sa.SA_ERR_INVALID_ARG, "L_a=0"),
    (_cache, dict(s_hat=FAKE), sa.SA_ERR_INVALID_ARG, "s_bar and s_hat"),
    (_cache, dict(eps=-1.0), sa.SA_ERR_INVALID_ARG, "eps"),
    (_cache, dict(tau=float("nan")), sa.SA_ERR_INVALID_ARG, "tau"),
    (_cache, dict(lambda_p=float("inf")), sa.SA_ERR_INVALID_ARG, "lambda_p"),
    (_cache, dict(out=None), sa.SA_ERR_INVALID_ARG, "out is NULL"),
    (_cache, dict(y_v_hat=MISALIGNED), sa.SA_ERR_INVALID_ARG, "aligned"),
    (_cache, dict(ws_bytes=4), sa.SA_ERR_WORKSPACE, "workspace"),
    (_ema, dict(alpha=1.5), sa.SA_ERR_INVALID_ARG, "alpha"),
    (_ema, dict(alpha=float("nan")), sa.SA_ERR_INVALID_ARG, "alpha"),
    (_ema, dict(sal_bar=None), sa.SA_ERR_INVALID_ARG, "sal_bar is NULL"),
    (_ema, dict(sal=FAKE + 64), sa.SA_ERR_INVALID_ARG, "overlap"),
    (_ema, dict(sal=MISALIGNED + 1), sa.SA_ERR_INVALID_ARG, "aligned"),
    (_tokens, dict(k_tok=-1), sa.SA_ERR_INVALID_ARG, "k_tok"),
    (_tokens, dict(k_tok=1001), sa.SA_ERR_INVALID_ARG, "k_tok"),
    (_tokens, dict(L=0), sa.SA_ERR_INVALID_ARG, "L=0"),
    (_tokens, dict(L=2048 * 128 + 1, k_tok=1), sa.SA_ERR_UNSUPPORTED, "exceeds"),
    (_tokens, dict(tok_idx=None), sa.SA_ERR_INVALID_ARG, "both NULL"),
    (_tokens, dict(sal_tok=None), sa.SA_ERR_INVALID_ARG, "sal_tok is NULL"),
    (_tokens, dict(tok_flag=FAKE, tok_idx=MISALIGNED + 1), sa.SA_ERR_INVALID_ARG, "aligned"),
    (_xfwd, dict(dtype=1), sa.SA_ERR_UNSUPPORTED, "SA_BF16"),
    (_xfwd, dict(Lq=0), sa.SA_ERR_INVALID_ARG, "Lq=0"),
    (_xfwd, dict(Lq=262145), sa.SA_ERR_INVALID_ARG, "Lq=262145"),
    (_xfwd, dict(Lk=2049 * 128), sa.SA_ERR_UNSUPPORTED, "n_b"),
    (_xfwd, dict(d=96), sa.SA_ERR_UNSUPPORTED, "head dim"),
    (_xfwd, dict(o=None), sa.SA_ERR_INVALID_ARG, "o is NULL"),
    (_xfwd, dict(ws_bytes=4), sa.SA_ERR_WORKSPACE, "workspace"),
    (_xfwd, dict(scale=0.0), sa.SA_ERR_INVALID_ARG, "scale"),
    (_xlse, dict(dtype=1), sa.SA_ERR_UNSUPPORTED, "SA_BF16"),
    (_xlse, dict(lse_v=None), sa.SA_ERR_INVALID_ARG, "lse_v"),
    (_xlse, dict(lse_a=None), sa.SA_ERR_INVALID_ARG, "lse_a is NULL"),
    (_xlse, dict(q_v=None, k_a=None, sal_a_tok=None), sa.SA_ERR_INVALID_ARG, "lse_v"),
    (_xlse, dict(L_a=0), sa.SA_ERR_INVALID_ARG, "L_a=0"),
    (_xlse, dict(ws_bytes=4), sa.SA_ERR_WORKSPACE, "workspace"),
    (_ptok, dict(k_tok=1001), sa.SA_ERR_INVALID_ARG, "k_tok"),
    (_ptok, dict(k_tok=-1), sa.SA_ERR_INVALID_ARG, "k_tok"),
    (_ptok, dict(d=96), sa.SA_ERR_UNSUPPORTED, "head dim"),
    (_ptok, dict(L=2049 * 128), sa.SA_ERR_UNSUPPORTED, "n_b"),
    (_ptok, dict(tok_idx=None), sa.SA_ERR_INVALID_ARG, "tok_idx is NULL"),
    (_ptok, dict(o=None), sa.SA_ERR_INVALID_ARG, "o is NULL"),
    (_ptok, dict(scale=-1.0), sa.SA_ERR_INVALID_ARG, "scale"),
    (_ptok, dict(ws_bytes=4), sa.SA_ERR_WORKSPACE, "workspace"),
    (_ptok, dict(ws=None), sa.SA_ERR_INVALID_ARG, "ws is NULL"),
    (_attn, dict(d=96), sa.SA_ERR_UNSUPPORTED, "head dim"),
    (_attn, dict(block=32), sa.SA_ERR_UNSUPPORTED, "block"),
    (_attn, dict(dtype=7), sa.SA_ERR_UNSUPPORTED, "dtype"),
    (_attn, dict(L=2049 * 128), sa.SA_ERR_UNSUPPORTED, "n_b"),
    (_attn, dict(B=0), sa.SA_ERR_INVALID_ARG, ">= 1"),
    (_attn, dict(B=256, H=256), sa.SA_ERR_UNSUPPORTED, "B*H=65536"),
    (_cross, dict(B=65536), sa.SA_ERR_UNSUPPORTED, "B*H=65536"),
    (_xfwd, dict(H=70000), sa.SA_ERR_UNSUPPORTED, "B*H=70000"),
    (_attn, dict(L=0), sa.SA_ERR_INVALID_ARG, ">= 1"),
    (_attn, dict(scale=0.0), sa.SA_ERR_INVALID_ARG, "scale"),
    (_attn, dict(scale=float("nan")), sa.SA_ERR_INVALID_ARG, "scale"),
    (_attn, dict(scale=float("inf")), sa.SA_ERR_INVALID_ARG, "scale"),
    (_attn, dict(q=None), sa.SA_ERR_INVALID_ARG, "q is NULL"),
    (_attn, dict(o=None), sa.SA_ERR_INVALID_ARG, "o is NULL"),
    (_attn, dict(kv_cnt=None), sa.SA_ERR_INVALID_ARG, "kv_cnt is NULL"),
    (_attn, dict(v=MISALIGNED), sa.SA_ERR_INVALID_ARG, "aligned"),
    (_attn, dict(lse=MISALIGNED), sa.SA_ERR_INVALID_ARG, "aligned"),
    (_attn, dict(ws_bytes=16), sa.SA_ERR_WORKSPACE, "workspace"),
    (_attn, dict(ws=None), sa.SA_ERR_INVALID_ARG, "ws is NULL"),
    (_attn_na, dict(q=None), sa.SA_ERR_INVALID_ARG, "q is NULL"),
    (_attn_na, dict(kv_cnt=MISALIGNED), sa.SA_ERR_INVALID_ARG, "aligned"),
    (_attn_na, dict(d=96), sa.SA_ERR_UNSUPPORTED, "head dim"),
    # B*H*n_b = 600 * 2048 entries of launch order and schedule exceed the 4 MiB scratch
    (_attn_na, dict(H=600, L=262144), sa.SA_ERR_UNSUPPORTED, "scratch"),
    (_mask, dict(k_keep=0), sa.SA_ERR_INVALID_ARG, "k_keep"),
    (_mask, dict(k_keep=9), sa.SA_ERR_INVALID_ARG, "k_keep"),
    (_mask, dict(kv_idx=None), sa.SA_ERR_INVALID_ARG, "kv_idx is NULL"),
    (_mask, dict(scores=MISALIGNED), sa.SA_ERR_INVALID_ARG, "aligned"),
    (_mask, dict(ws_bytes=0), sa.SA_ERR_WORKSPACE, "workspace"),
    (_mask, dict(d=32), sa.SA_ERR_UNSUPPORTED, "head dim"),
    (_cross, dict(L_a=0), sa.SA_ERR_INVALID_ARG, "L_a"),
    (_cross, dict(accumulate=2), sa.SA_ERR_INVALID_ARG, "accumulate"),
    (_cross, dict(k_a=None), sa.SA_ERR_INVALID_ARG, "all NULL"),
    (_cross, dict(sal_a_tok=None), sa.SA_ERR_INVALID_ARG, "all NULL"),
    (_cross, dict(q_v=None, k_a=None), sa.SA_ERR_INVALID_ARG, "all NULL"),
    (_cross, dict(sal_v_blk=None), sa.SA_ERR_INVALID_ARG, "sal_v_blk is NULL"),
    (_cross, dict(q_a=None), sa.SA_ERR_INVALID_ARG, "q_a is NULL"),
    (_cross, dict(ws_bytes=1), sa.SA_ERR_WORKSPACE, "workspace"),
    (_xpool, dict(lse_a=FAKE), sa.SA_ERR_INVALID_ARG, "lse_a and lse_v"),
    (_xpool, dict(lse_a=FAKE, lse_v=FAKE, dtype=1), sa.SA_ERR_UNSUPPORTED, "SA_BF16"),
    (_xpool, dict(q_v=None), sa.SA_ERR_INVALID_ARG, "q_v is NULL"),
    (_xpool, dict(sal_a_tok=None), sa.SA_ERR_INVALID_ARG, "sal_a_tok is NULL"),
    (_xpool, dict(qbar=None), sa.SA_ERR_INVALID_ARG, "qbar is NULL"),
    (_xpool, dict(kbar=FAKE + 4), sa.SA_ERR_INVALID_ARG, "aligned"),
    # 1 x 1 x 128 x 64 doubles (64 KB) each: kbar 32 KB after qbar overlaps it
    (_xpool, dict(kbar=FAKE + 32 * 1024), sa.SA_ERR_INVALID_ARG, "overlap"),
    (_xpool, dict(L_a=0), sa.SA_ERR_INVALID_ARG, "L_a=0"),
    (_xpool, dict(accumulate=3), sa.SA_ERR_INVALID_ARG, "accumulate"),
    (_xpool, dict(block=32), sa.SA_ERR_UNSUPPORTED, "block"),
    (_xpool, dict(ws_bytes=4), sa.SA_ERR_WORKSPACE, "workspace"),
    (_mpool, dict(k_keep=0), sa.SA_ERR_INVALID_ARG, "k_keep"),
    (_mpool, dict(k_keep=9), sa.SA_ERR_INVALID_ARG, "k_keep"),
    (_mpool, dict(qbar=None), sa.SA_ERR_INVALID_ARG, "qbar is NULL"),
    (_mpool, dict(kbar=MISALIGNED), sa.SA_ERR_INVALID_ARG, "aligned"),
    (_mpool, dict(kv_cnt=None), sa.SA_ERR_INVALID_ARG, "kv_cnt is NULL"),
    (_mpool, dict(d=96), sa.SA_ERR_UNSUPPORTED, "head dim"),
    (_mpool, dict(L_v=2049 * 128), sa.SA_ERR_UNSUPPORTED, "n_b"),
    (_select, dict(k_prot=-1), sa.SA_ERR_INVALID_ARG, "k_prot"),
    (_select, dict(k_prot=9), sa.SA_ERR_INVALID_ARG, "k_prot"),
    (_select, dict(n_b=0), sa.SA_ERR_INVALID_ARG, "n_b"),
    (_select, dict(n_b=4096, k_prot=1), sa.SA_ERR_UNSUPPORTED, "n_b"),
    (_select, dict(prot_flag=None), sa.SA_ERR_INVALID_ARG, "prot_flag is NULL"),
    (_select, dict(sal_blk=MISALIGNED + 1), sa.SA_ERR_INVALID_ARG, "aligned"),
]


@pytest.mark.parametrize("call,kw,code,needle", INVALID)
def test_invalid_arguments_are_rejected(call, kw, code, needle):
    rc = call(**kw)
    assert rc == code
    msg = sa.sa_last_error()
    assert needle in msg, msg


def test_pool_columns():
    """The pooled means are padded to the mask's row width: 64 * E with E the
    smallest of 1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32 covering n_b."""
    widths = [1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32]
    for n_b in (1, 16, 64, 65, 256, 257, 384, 591, 640, 641, 1024, 1537, 2048):
        assert sa.sa_pool_columns(n_b) == 64 * min(e for e in widths if 64 * e >= n_b)
    assert sa.sa_pool_columns(0) == 0 and sa.sa_pool_columns(2049) == 0


def test_empty_token_calls_launch_nothing():
    """k_tok = 0 and n = 0 are valid and return before any launch."""
    assert _ptok(k_tok=0, tok_idx=None) == sa.SA_OK
    assert _ema(n=0) == sa.SA_OK


def test_binding_raises_without_gpu_tensors():
    import torch
    x = torch.zeros(1, 1, 128, 64)
    with pytest.raises(ValueError):
        sa.sa_sparse_attention(x, x, x, 0.125, 64,
                               torch.zeros(1, 1, 2, 2, dtype=torch.int32),
                               torch.zeros(1, 1, 2, dtype=torch.int32), ws=x)


def test_binding_refuses_mismatched_tensors():
    """The C ABI sees pointers only; the binding refuses tensors whose shape
    or dtype disagrees with the call before anything reaches the library."""
    import torch
    bf, f32 = torch.bfloat16, torch.float32
    q = torch.zeros(1, 2, 256, 64, dtype=bf)
    with pytest.raises(ValueError, match="k: shape"):
        sa.sa_sparse_attention(q, torch.zeros(1, 2, 128, 64, dtype=bf), q, 0.1, 64,
                               torch.zeros(1, 2, 4, 4, dtype=torch.int32),
                               torch.zeros(1, 2, 4, dtype=torch.int32))
    with pytest.raises(TypeError, match="v: dtype"):
        sa.sa_sparse_attention(q, q, q.float(), 0.1, 64,
                               torch.zeros(1, 2, 4, 4, dtype=torch.int32),
                               torch.zeros(1, 2, 4, dtype=torch.int32))
    with pytest.raises(ValueError, match="kv_cnt: shape"):
        sa.sa_sparse_attention(q, q, q, 0.1, 64, torch.zeros(1, 2, 4, 4, dtype=torch.int32),
                               torch.zeros(1, 2, 3, dtype=torch.int32))
    with pytest.raises(ValueError, match="k_v: shape"):
        sa.sa_cross_scores(torch.zeros(1, 2, 16, 64, dtype=bf),
                           torch.zeros(1, 3, 256, 64, dtype=bf), None, None, 0.1, 64)
    with pytest.raises(ValueError, match="v: shape"):
        sa.sa_cross_attention(torch.zeros(1, 2, 16, 64, dtype=bf),
                              torch.zeros(1, 2, 100, 64, dtype=bf),
                              torch.zeros(1, 2, 99, 64, dtype=bf), 0.1)
    with pytest.raises(ValueError, match="tok_idx: shape"):
        sa.sa_select_protected_tokens(torch.zeros(2, 50, dtype=f32), 5,
                                      tok_idx=torch.zeros(2, 4, dtype=torch.int32))
    with pytest.raises(ValueError, match="y_v_hat: shape"):
        sa.sa_cache_indicator(torch.zeros(1, 10, 8, dtype=bf), torch.zeros(1, 9, 8, dtype=bf))
    with pytest.raises(ValueError, match="prot_flag: shape"):
        sa.sa_build_block_mask(q, q, 0.1, 64, 2, torch.zeros(1, 5, dtype=torch.uint8))
