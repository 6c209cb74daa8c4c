"""Products at the edges of their kernels' tiles, through the entry points
that run them, against float64 references.

Tolerances: cosines of exact bf16 inputs carry only the float32 accumulation
over D terms (far below 1e-5 for D <= 4096); p_hat and the selection's gains
meet the bars of the fused-prune tests (2e-2 for bf16 scores; 1e-3 for gains
against the replayed selection, whose norms and cosines are the oracle's)."""
import numpy as np
import pytest
import torch

import oracle
from workloads import PredictorShape, get_config, make_inputs

from gpu_util import announce, dev_inputs, device, oracle_weights

pytestmark = pytest.mark.gpu


# 256 x 256 tiles: the shortest K loop (four slices) and one of eight, a last
# tile that reaches into both of its halves or into one only
@pytest.mark.parametrize("B,N,D", [(16, 1000, 256), (20, 769, 512)])
def test_big_tiles_cosine(B, N, D):
    from paper_2608_06411_amd import map_similarity
    dev = device()
    announce(f"big tiles, cosine B={B} N={N} D={D}")
    g = torch.Generator(device=dev)
    g.manual_seed(N)
    V = torch.randn(B, N, D, generator=g, device=dev).to(torch.bfloat16)
    S, norms = map_similarity(V)
    v = V.double()
    want_n = v.norm(dim=2)
    v = v / want_n[:, :, None]
    for b in range(B):
        assert float((S[b].double() - v[b] @ v[b].t()).abs().max()) < 1e-5
        assert torch.equal(S[b], S[b].t())
    assert float((norms.double() / want_n - 1).abs().max()) < 2e-6


# The row norms formed by the 256 x 256 tiles: two and four tile columns, a
# last tile row that is nearly empty
@pytest.mark.parametrize("B,N,Dh", [(18, 1000, 512), (16, 1001, 1024)])
def test_big_tiles_row_norms(B, N, Dh):
    from paper_2608_06411_amd import map_prune
    dev = device()
    announce(f"big tiles, row norms B={B} N={N} D_h={Dh}")
    cfg = get_config("sweep", B=B, N=N, M=(5, 20), K=32, K0=16, clusters=90, pred=PredictorShape(D=256, D_h=Dh, d_p=64))
    x = make_inputs(cfg)
    d = dev_inputs(x, dev)
    o = map_prune(d["w"], d["V"], d["pos_v"], d["T"], d["pos_t"], x["t_off"], cfg.K, cfg.K0, cfg.tau)
    p = o["p"].cpu().numpy().astype(np.float64)
    p_ref = oracle.predicted_attention_batch(x["V_f32"], x["T_f32"], x["t_off"], x["pos_v"], x["pos_t"], oracle_weights(x),
                                             cfg.pred.rope_theta)
    np.testing.assert_allclose(p, p_ref, rtol=2e-2, atol=0)
    order, gain = o["order"].cpu().numpy(), o["gain"].cpu().numpy()
    for b in range(B):
        rep = oracle.replay_check(p[b], x["V_f32"][b], cfg.K, cfg.K0, cfg.tau, order[b], gain[b])
        assert rep.ok, f"image {b}: {rep.failure}"
        assert rep.max_gain_rel_err < 1e-5


# float32 tiles (64 x 64, K in slices of 32 that two groups of waves take in
# turn): one slice only, an odd count, more than the ring holds, one row past a
# tile, and K that is no multiple of 32 (the register-staged kernel)
@pytest.mark.parametrize("B,N,D", [(1, 65, 32), (2, 64, 96), (1, 129, 544), (3, 33, 4128), (1, 70, 40)])
def test_f32_tiles_cosine(B, N, D):
    from paper_2608_06411_amd import map_similarity
    dev = device()
    announce(f"float32 tiles, cosine B={B} N={N} D={D}")
    g = torch.Generator(device=dev)
    g.manual_seed(D)
    V = torch.randn(B, N, D, generator=g, device=dev)
    S, norms = map_similarity(V)
    v = V.double() / V.double().norm(dim=2, keepdim=True)
    for b in range(B):
        assert float((S[b].double() - v[b] @ v[b].t()).abs().max()) < 1e-5
        assert torch.equal(S[b], S[b].t())


# bf16 launches on 64 x 64 tiles: four slices only (fewer than the ring
# holds), one row past a tile, several images, and one tile too many for one
# round of workgroups (128 x 128 tiles)
@pytest.mark.parametrize("B,N,D", [(1, 65, 256), (3, 33, 512), (2, 128, 768), (1, 1408, 256), (1, 1409, 256)])
def test_small_bf16_tiles_cosine(B, N, D):
    from paper_2608_06411_amd import map_similarity
    dev = device()
    announce(f"64 x 64 bf16 tiles, cosine B={B} N={N} D={D}")
    g = torch.Generator(device=dev)
    g.manual_seed(N + D)
    V = torch.randn(B, N, D, generator=g, device=dev).to(torch.bfloat16)
    S, norms = map_similarity(V)
    v = V.double() / V.double().norm(dim=2, keepdim=True)
    for b in range(B):
        assert float((S[b].double() - v[b] @ v[b].t()).abs().max()) < 1e-5
        assert torch.equal(S[b], S[b].t())


# Layer-1 launches around the sizes where 192-row tiles, which cannot form
# the row norms, would be the shortest, and small ones whose norms come from
# the preparation: the call runs and its norms (through the gains) are right
@pytest.mark.parametrize("B,N,M", [(8, 1000, (30, 45)), (9, 900, (60, 70)), (10, 1050, (20, 30)), (2, 500, (9, 20)), (1, 600, (40, 40))])
def test_layer1_norms_across_tile_choices(B, N, M):
    from paper_2608_06411_amd import map_prune
    dev = device()
    announce(f"layer-1 tile choices B={B} N={N} M={M}")
    cfg = get_config("sweep", B=B, N=N, M=M, K=40, K0=20, clusters=90, pred=PredictorShape(D=256, D_h=1024, d_p=64))
    x = make_inputs(cfg)
    d = dev_inputs(x, dev)
    o = map_prune(d["w"], d["V"], d["pos_v"], d["T"], d["pos_t"], x["t_off"], cfg.K, cfg.K0, cfg.tau)
    p = o["p"].cpu().numpy().astype(np.float64)
    p_ref = oracle.predicted_attention_batch(x["V_f32"], x["T_f32"], x["t_off"], x["pos_v"], x["pos_t"], oracle_weights(x),
                                             cfg.pred.rope_theta)
    np.testing.assert_allclose(p, p_ref, rtol=2e-2, atol=0)
    order, gain = o["order"].cpu().numpy(), o["gain"].cpu().numpy()
    for b in range(B):
        rep = oracle.replay_check(p[b], x["V_f32"][b], cfg.K, cfg.K0, cfg.tau, order[b], gain[b])
        assert rep.ok, f"image {b}: {rep.failure}"
        assert rep.max_gain_rel_err < 1e-5


# K in whole slices of 64 but no multiple of 256: an odd count of slices, and
# even ones on 128 x 128 and 256 x 256 tiles; five slices on 64 x 64 tiles;
# K below four slices (the register-staged kernel); five and ten slices on 128 x
# 128 tiles, whose loop then ends with the last of its five stages
@pytest.mark.parametrize("B,N,D", [(1, 1500, 1088), (2, 1500, 1152), (16, 1000, 1152), (3, 700, 320), (2, 1500, 192),
                                   (1, 1500, 320), (1, 1500, 640)])
def test_cosine_slice_counts(B, N, D):
    from paper_2608_06411_amd import map_similarity
    dev = device()
    announce(f"slice counts, cosine B={B} N={N} D={D}")
    g = torch.Generator(device=dev)
    g.manual_seed(N + D)
    V = torch.randn(B, N, D, generator=g, device=dev).to(torch.bfloat16)
    S, norms = map_similarity(V)
    for b in range(B):
        v = V[b].double()
        v = v / v.norm(dim=1, keepdim=True)
        assert float((S[b].double() - v @ v.t()).abs().max()) < 1e-5
        assert torch.equal(S[b], S[b].t())
