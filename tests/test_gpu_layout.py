"""GPU parity of the conv-layout front end: X[B, C, H, W] -> tokens X'[B, HW, C]
(Supp. implementation details, the 4-D branch) against the oracle's re-layout, and the
token paths run on the tokenized map."""
import numpy as np
import pytest
import torch

from oracle import tdq_oracle as O
from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)


def _feature_map(B, C, H, W, dtype, seed):
    rng = np.random.Generator(np.random.PCG64([seed, B, C, H, W]))
    X = rng.standard_normal((B, C, H, W)) * np.exp(rng.normal(0, 1.0, (B, 1, H, W)))
    X[rng.random((B, C, H, W)) < 0.01] *= 25.0
    return X.astype(dtype)


@pytest.mark.parametrize("B,C,H,W,dtype", [
    (2, 64, 16, 8, np.float16),       # exactly one tile per image
    (1, 320, 22, 22, np.float16),     # 484 tokens: ragged token tiles
    (3, 100, 7, 9, np.float16),       # nothing aligned: scalar loads and stores
    (1, 1, 1, 1, np.float16),
    (2, 72, 12, 16, np.float16),      # ragged channel tile, aligned rows
    (2, 64, 8, 8, np.float32),
    (1, 130, 11, 13, np.float32),
    (1, 1024, 64, 64, np.float16),    # a 4096-token, 1024-channel map
])
def test_tokenize_chw_is_an_exact_relayout(B, C, H, W, dtype):
    _say(f"[tokenize] B={B} C={C} H={H} W={W} dtype={dtype.__name__}")
    X = _feature_map(B, C, H, W, dtype, 3)
    Xt = tdq.tdq_tokenize_chw(torch.from_numpy(X).to(U.dev()))
    torch.cuda.synchronize()
    assert np.array_equal(Xt.cpu().numpy().view(np.uint8), O.tokenize_chw(X).view(np.uint8))


def test_tokenize_chw_strided_views():
    """Channel and image strides larger than the data (a crop of a wider buffer), and an
    output with a padded row stride: junk around the data is neither read into the result
    nor overwritten."""
    B, C, H, W = 2, 48, 6, 10
    X = _feature_map(B, C + 5, H + 2, W, np.float16, 4)
    Xd = torch.from_numpy(X).to(U.dev())[:, 2:2 + C, 1:1 + H, :]      # spatial axes stay contiguous
    out = torch.full((B, H * W, C + 8), 9.0, dtype=torch.float16, device=U.dev())
    tdq.tdq_tokenize_chw(Xd, out=out[:, :, :C])
    torch.cuda.synchronize()
    ref = O.tokenize_chw(X[:, 2:2 + C, 1:1 + H, :])
    got = out.cpu().numpy()
    assert np.array_equal(got[:, :, :C], ref)
    assert (got[:, :, C:] == 9.0).all()


def test_conv_layout_through_both_token_paths():
    """A feature map through tokenize -> token-set path and -> per-block path gives what
    the oracle gives on the oracle's tokens."""
    B, C, H, W = 2, 96, 12, 12
    X = _feature_map(B, C, H, W, np.float16, 5)
    Xt_ref = O.tokenize_chw(X)
    Xt = tdq.tdq_tokenize_chw(torch.from_numpy(X).to(U.dev()))
    # token sets
    p = tdq.default_params(4)
    gid, clip, scale, _, ws = tdq.tdq_calibrate_groups(Xt, p)
    Q = tdq.tdq_quantize_act(Xt, p, gid, clip, scale)
    torch.cuda.synchronize()
    og, oc, osc, _ = O.calibrate_groups(Xt_ref, U.oracle_params(p))
    assert np.array_equal(gid.cpu().numpy(), og)
    assert np.allclose(scale.cpu().numpy(), osc, rtol=U.SCALE_RTOL, atol=0)
    q_ref = O.quantize_act(Xt_ref, og, oc, osc, U.oracle_params(p)).reshape(B * H * W, C)
    rows = np.arange(B)[:, None]
    U.assert_codes_match(U.unpack_device_codes(Q, C), q_ref, Xt_ref,
                         oc[rows, og].reshape(-1), osc[rows, og].reshape(-1),
                         np.array_equal(scale.cpu().numpy(), osc))
    # blocks of 32 channels per pixel (the paper's 4-D branch)
    pb = tdq.block_params(flags=2)
    Qb, bs, bc = tdq.tdq_quantize_act_blocks(Xt, pb, want_clip=True)
    torch.cuda.synchronize()
    _, qb_ref, cb, sb = O.dstg_dcrp_blocks(Xt_ref.reshape(B * H * W, C), 32,
                                           O.Params(n_groups=1, flags=2))
    assert np.array_equal(bc.cpu().numpy(), cb) and np.array_equal(bs.cpu().numpy(), sb)
    assert np.array_equal(U.unpack_device_codes(Qb, C), qb_ref)


def _blocks_view(a, C):
    M = a.shape[0]
    KB = -(-C // 32)
    out = np.zeros((M, KB * 32), dtype=a.dtype)
    out[:, :C] = a
    return out.reshape(M * KB, 32)


@pytest.mark.parametrize("B,C,H,W,dtype,kw", [
    (2, 128, 16, 8, np.float16, {}),                 # one channel tile, one token tile
    (1, 320, 22, 22, np.float16, {}),                # ragged in both axes
    (3, 100, 7, 9, np.float16, {}),                  # last block partly padding, unaligned rows
    (1, 40, 5, 5, np.float16, dict(flags=2)),
    (1, 7, 3, 3, np.float16, dict(flags=0)),
    (2, 256, 16, 16, np.float16, dict(flags=2, zr=0.3)),        # bisection route (rank 10)
    (1, 192, 12, 12, np.float16, dict(flags=3, base_pct=0.9)),
    (2, 64, 8, 8, np.float32, {}),
    (1, 130, 11, 13, np.float32, dict(flags=2)),
    (1, 1024, 32, 32, np.float16, {}),               # eight channel tiles
])
def test_blocks_quantizer_reads_conv_layout_directly(B, C, H, W, dtype, kw):
    """The fused 4-D branch: same bits as the token-major sweep on the tokenized map, and
    the oracle's Algorithm 1 on the oracle's tokens."""
    _say(f"[blocks-chw] B={B} C={C} H={H} W={W} dtype={dtype.__name__} {kw}")
    X = _feature_map(B, C, H, W, dtype, 6)
    p = tdq.block_params(**kw)
    Xd = torch.from_numpy(X).to(U.dev())
    Q, bs, bc = tdq.tdq_quantize_act_blocks_chw(Xd, p, want_clip=True)
    Q2, bs2, bc2 = tdq.tdq_quantize_act_blocks(tdq.tdq_tokenize_chw(Xd), p, want_clip=True)
    torch.cuda.synchronize()
    assert torch.equal(Q, Q2) and torch.equal(bs, bs2) and torch.equal(bc, bc2)
    Xt = O.tokenize_chw(X).reshape(B * H * W, C)
    op = O.Params(n_groups=1, flags=p.flags & 3, tau=p.tau, zr=p.zr, base_pct=p.base_pct)
    _, q_ref, clip, scale = O.dstg_dcrp_blocks(Xt, 32, op)
    cg, sg = bc.cpu().numpy(), bs.cpu().numpy()
    if not (p.flags & tdq.FLAG_C1):
        assert np.array_equal(cg, clip) and np.array_equal(sg, scale)
    assert np.allclose(cg, clip, rtol=U.SCALE_RTOL, atol=0)
    assert np.allclose(sg, scale, rtol=U.SCALE_RTOL, atol=0)
    exact = np.array_equal(cg, clip) and np.array_equal(sg, scale)
    U.assert_codes_match(_blocks_view(U.unpack_device_codes(Q, C), C), _blocks_view(q_ref, C),
                         _blocks_view(Xt.astype(np.float32), C), clip.reshape(-1),
                         scale.reshape(-1), exact)


def test_blocks_quantizer_conv_layout_strided_view():
    B, C, H, W = 2, 72, 6, 12
    X = _feature_map(B, C + 3, H + 1, W, np.float16, 7)
    Xd = torch.from_numpy(X).to(U.dev())[:, 1:1 + C, :H, :]
    p = tdq.block_params(flags=2)
    Q, bs, bc = tdq.tdq_quantize_act_blocks_chw(Xd, p, want_clip=True)
    torch.cuda.synchronize()
    Xt = O.tokenize_chw(X[:, 1:1 + C, :H, :]).reshape(B * H * W, C)
    _, q_ref, clip, scale = O.dstg_dcrp_blocks(Xt, 32, O.Params(n_groups=1, flags=2))
    assert np.array_equal(bc.cpu().numpy(), clip) and np.array_equal(bs.cpu().numpy(), scale)
    assert np.array_equal(U.unpack_device_codes(Q, C), q_ref)


@pytest.mark.parametrize("B,C,H,W,dtype,G", [
    (2, 64, 16, 8, np.float16, 4), (1, 320, 22, 22, np.float16, 16), (3, 100, 7, 9, np.float16, 5),
    (2, 72, 12, 16, np.float16, 8), (2, 64, 8, 8, np.float32, 4), (1, 130, 11, 13, np.float32, 3),
    (1, 1024, 32, 32, np.float16, 32), (1, 1, 1, 1, np.float16, 2)])
def test_token_set_calibration_reads_conv_layout(B, C, H, W, dtype, G):
    """tdq_calibrate_groups_chw: the token-major copy is exact, and ids, thresholds and
    steps are the oracle's on the oracle's tokens."""
    _say(f"[calibrate-chw] B={B} C={C} H={H} W={W} dtype={dtype.__name__} G={G}")
    X = _feature_map(B, C, H, W, dtype, 8)
    p = tdq.default_params(G)
    Xt, gid, clip, scale, stats, ws = tdq.tdq_calibrate_groups_chw(torch.from_numpy(X).to(U.dev()), p,
                                                                  want_stats=True)
    Q = tdq.tdq_quantize_act(Xt, p, gid, clip, scale)
    torch.cuda.synchronize()
    Xt_ref = O.tokenize_chw(X)
    assert np.array_equal(Xt.cpu().numpy().view(np.uint8), Xt_ref.view(np.uint8))
    assert tdq.device_status(ws) == 0
    g = dict(gid=gid.cpu().numpy(), clip=clip.cpu().numpy(), scale=scale.cpu().numpy(),
             stats=tdq.stats_to_numpy(stats))
    og, oc, osc, _ = U.assert_calibration_matches(g, Xt_ref, p)
    q_ref = O.quantize_act(Xt_ref, og, oc, osc, U.oracle_params(p)).reshape(B * H * W, C)
    rows = np.arange(B)[:, None]
    exact = np.array_equal(g["scale"], osc) and np.array_equal(g["clip"], oc)
    U.assert_codes_match(U.unpack_device_codes(Q, C), q_ref, Xt_ref, oc[rows, og].reshape(-1),
                         osc[rows, og].reshape(-1), exact)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("B,C,H,W", [(2, 1, 1, 1), (1, 63, 3, 21), (2, 64, 8, 8), (1, 65, 5, 13), (3, 130, 1, 129),
                                     (2, 40, 9, 7), (1, 200, 16, 40)])
def test_fused_statistics_tile_edges(B, C, H, W, dtype):
    """One tile, one channel or token past a tile, odd token counts (a thread takes two tokens
    at a time), maps that allow 16-byte loads and maps that do not."""
    rng = np.random.Generator(np.random.PCG64(B + 3 * C + H * W))
    X = (rng.laplace(0, 1, (B, C, H, W)) * rng.lognormal(0, 1, (B, 1, H, W)) + 2.0)
    X = X.astype(np.float16 if dtype == "f16" else np.float32)
    p = tdq.default_params(5)
    Xt, gid, clip, scale, stats, ws = tdq.tdq_calibrate_groups_chw(torch.from_numpy(X).to(U.dev()), p, want_stats=True)
    torch.cuda.synchronize()
    ref = O.tokenize_chw(X)
    assert np.array_equal(Xt.cpu().numpy(), ref)
    g = dict(gid=gid.cpu().numpy(), clip=clip.cpu().numpy(), scale=scale.cpu().numpy(),
             stats=tdq.stats_to_numpy(stats))
    U.assert_calibration_matches(g, ref, p)


def test_calibrate_chw_of_many_tokens():
    """More tiles of tokens in one image than an axis of a grid takes (2^29 tokens are 2^24 tiles)."""
    T = (1 << 29) + 70
    X = torch.randn((1, 1, T), device=U.dev())
    p = tdq.default_params(1)
    p.flags = 0                                   # the radius is the largest magnitude
    Xt, gid, clip, scale, _, ws = tdq.tdq_calibrate_groups_chw(X, p)
    assert torch.equal(Xt.view(-1), X.view(-1))
    assert clip.item() == X.abs().max().item() and int(gid.max()) == 0
    assert tdq.device_status(ws) == 0


@pytest.mark.parametrize("B,C,H,W,dtype", [(8, 65, 32, 64, np.float16), (9, 65, 32, 64, np.float16),
                                           (9, 129, 31, 65, np.float16), (8, 129, 31, 33, np.float32),
                                           (9, 129, 31, 33, np.float32), (2, 257, 3, 11, np.float16),
                                           (1, 128, 4, 4, np.float32)])
def test_feature_map_tiles(B, C, H, W, dtype):
    """256 workgroups of 64 x 8 tiles and more, where the tile changes; one and several tiles of channels,
    tokens that end inside a tile."""
    X = _feature_map(B, C, H, W, dtype, 3)
    p = tdq.default_params(5)
    Xt, gid, clip, scale, stats, ws = tdq.tdq_calibrate_groups_chw(torch.from_numpy(X).to(U.dev()), p, want_stats=True)
    torch.cuda.synchronize()
    ref = O.tokenize_chw(X)
    assert np.array_equal(Xt.cpu().numpy().view(np.uint8), ref.view(np.uint8)) and tdq.device_status(ws) == 0
    g = dict(gid=gid.cpu().numpy(), clip=clip.cpu().numpy(), scale=scale.cpu().numpy(),
             stats=tdq.stats_to_numpy(stats))
    U.assert_calibration_matches(g, ref, p)
