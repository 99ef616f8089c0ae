"""The fp32 kernels (16-row matrix tiles, keys split over the waves of a
workgroup) at the sizes where a tile, a wave's share or a chunk ends: one
token, one below and above a 16-row tile and a 64-key workgroup, around the
1024-key chunk of the a->v log-sum-exp and the 512-query chunk of the v->a
column mass, fewer key tiles than waves.  Against the oracle with the fp32
bounds of the other parity tests."""
import numpy as np
import pytest
import torch

import synth
import paper_2608_15522_amd as sa
from sa_parity import TOL_LSE, TOL_O, compare_layer, gpu_layer, to_dev

pytestmark = pytest.mark.gpu

BASE = synth.WORKLOADS["tiny_f32"]


@pytest.mark.parametrize("L_v,L_a,d,block,k_keep,k_prot", [
    (1, 1, 64, 64, 1, 0), (15, 17, 128, 128, 1, 1), (17, 16, 64, 64, 1, 0),
    (63, 65, 128, 64, 1, 0), (65, 63, 64, 64, 1, 1), (129, 15, 128, 128, 1, 0),
    (511, 33, 64, 128, 2, 1), (513, 130, 128, 64, 3, 2), (1024, 512, 64, 64, 4, 0),
    (1025, 513, 128, 128, 9, 0), (2049, 1, 64, 64, 5, 3),
])
def test_f32_layer_at_tile_edges(L_v, L_a, d, block, k_keep, k_prot):
    w = BASE.with_(name="edge", B=1, H=2, d=d, block=block, frames=1, rows=1, cols=L_v, L_a=L_a,
                   n_plant=0)
    print(f"case f32 layer L_v={L_v} L_a={L_a} d={d} block={block}", flush=True)
    x = synth.make_inputs(w)
    g = gpu_layer(x, w, k_keep, k_prot)
    print(compare_layer(x, w, g, k_keep, k_prot), flush=True)


@pytest.mark.parametrize("L,k_tok,d", [(1, 1, 64), (17, 16, 128), (50, 17, 64), (333, 1, 128)])
def test_f32_token_rows_at_tile_edges(L, k_tok, d):
    w = BASE.with_(name="tok", B=2, H=2, d=d, frames=1, rows=1, cols=L, L_a=3, n_plant=0)
    print(f"case f32 tokens L={L} k_tok={k_tok} d={d}", flush=True)
    x = synth.make_inputs(w)
    t = {n: to_dev(x[n], "f32") for n in ("q_v", "k_v", "v_v")}
    rng = np.random.default_rng(L)
    idx = np.sort(np.stack([rng.permutation(L)[:k_tok] for _ in range(w.B)]), axis=1)
    o = torch.full((w.B, w.H, L, d), 7.0, device="cuda")
    lse = torch.full((w.B, w.H, L), 7.0, device="cuda")
    sa.sa_protected_token_attention(t["q_v"], t["k_v"], t["v_v"], w.scale,
                                    torch.from_numpy(idx.astype(np.int32)).cuda(), o, lse)
    o, lse = o.cpu().numpy(), lse.cpu().numpy()
    for b in range(w.B):
        rest = np.setdiff1d(np.arange(L), idx[b])
        assert np.all(o[b][:, rest] == 7.0) and np.all(lse[b][:, rest] == 7.0)
        for h in range(w.H):
            s = w.scale * (x["q_v"][b, h, idx[b]].astype(np.float64) @
                           x["k_v"][b, h].astype(np.float64).T)
            ref_lse = np.log(np.exp(s - s.max(1, keepdims=True)).sum(1)) + s.max(1)
            ref = np.exp(s - ref_lse[:, None]) @ x["v_v"][b, h].astype(np.float64)
            assert np.abs(o[b, h, idx[b]] - ref).max() <= TOL_O["f32"]
            assert np.abs(lse[b, h, idx[b]] - ref_lse).max() <= TOL_LSE["f32"]


@pytest.mark.parametrize("d", [64, 128])
def test_f32_attention_of_values_near_the_top_of_the_range(d):
    """Weights are at most 1 before they are normalised too: one value of 2^125
    among zeros gives its weight times itself.  Scores rise along the keys, by
    less than the slack between two rescales."""
    L, block = 700, 64
    g = torch.Generator(device="cuda").manual_seed(d)
    q, k = (torch.randn(1, 1, L, d, generator=g, device="cuda") for _ in range(2))
    q[..., 0] = d**0.5
    k[..., 0] = torch.arange(L, device="cuda") * (5.0 / L)  # 5 nats: 7.2 log2 units
    v = torch.zeros(1, 1, L, d, device="cuda")
    v[0, 0, L - 1] = 2.0**125
    n_b = -(-L // block)
    idx = torch.arange(n_b, dtype=torch.int32, device="cuda").expand(1, 1, n_b, n_b).contiguous()
    cnt = torch.full((1, 1, n_b), n_b, dtype=torch.int32, device="cuda")
    scale = float(np.float32(d**-0.5))
    o, lse = sa.sa_sparse_attention(q, k, v, scale, block, idx, cnt, want_lse=True)
    s = scale * (q[0, 0].double() @ k[0, 0].double().T.contiguous())
    ref = torch.softmax(s, 1) @ v[0, 0].double()
    assert ((o[0, 0].double() - ref).abs() <= 1e-5 * ref).all()
    assert (lse[0, 0].double() - torch.logsumexp(s, 1)).abs().max() <= TOL_LSE["f32"]
