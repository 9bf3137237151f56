"""GPU parity of the single-launch activation path (tdq_calibrate_quantize_fused) against
the CPU oracle, with the bars of the multi-kernel path: group ids, thresholds and codes
(given the steps) bit-exact, sigma and steps to 1e-6."""
import numpy as np
import pytest
import torch

from oracle import tdq_oracle as O
from paper_2604_16855_amd import inputs as I
from paper_2604_16855_amd import tdq

import parity_util as U

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)


def _fused(X, p, ld_pad=0):
    Xd = U.to_device(X, ld_pad)
    gid, clip, scale, stats, flags, Q, ws = tdq.tdq_calibrate_quantize_fused(Xd, p, want_stats=True)
    torch.cuda.synchronize()
    return dict(Xd=Xd, gid=gid.cpu().numpy(), clip=clip.cpu().numpy(), scale=scale.cpu().numpy(),
                stats=tdq.stats_to_numpy(stats), flags=flags.cpu().numpy(), Q=Q, gid_d=gid,
                clip_d=clip, scale_d=scale)


def _check(X, p, ld_pad=0):
    B, T, C = X.shape
    _say(f"[fused] B={B} T={T} C={C} G={p.n_groups} dtype={X.dtype} flags={p.flags} "
         f"base_pct={p.base_pct} ld_pad={ld_pad}")
    g = _fused(X, p, ld_pad)
    assert not g["flags"].any()
    gid, clip, scale, _ = U.assert_calibration_matches(g, X, p)
    q_ref = O.quantize_act(X, gid, clip, scale, U.oracle_params(p)).reshape(B * T, C)
    rows = np.arange(B)[:, None]
    exact = np.array_equal(g["scale"], scale) and np.array_equal(g["clip"], clip)
    flips = U.assert_codes_match(U.unpack_device_codes(g["Q"], C), q_ref, X,
                                 clip[rows, gid].reshape(-1), scale[rows, gid].reshape(-1), exact)
    # the codes are those of tdq_quantize_act for the radii this call produced
    Q2 = tdq.tdq_quantize_act(g["Xd"], p, g["gid_d"], g["clip_d"], g["scale_d"])
    torch.cuda.synchronize()
    assert torch.equal(Q2[:, :(C + 1) // 2], g["Q"][:, :(C + 1) // 2])
    _say(f"  scales bit-identical: {exact}; code flips: {flips}")
    return g


@pytest.mark.parametrize("name,over", [("cfg0", {}), ("cfg1", {}), ("cfg2_qkv", {}),
                                       ("cfg2_fc2", dict(B=4)), ("cfg3_s4_fc1", dict(B=3))])
def test_fused_on_small_configs(name, over):
    lc = I.case(name, **over)
    X, _ = I.make_activations(lc)
    _check(X, tdq.default_params(lc.G))


@pytest.mark.parametrize("B,T,C,G,dtype,ld_pad", [
    (3, 37, 70, 5, "f16", 0), (2, 50, 33, 4, "f16", 0), (2, 41, 64, 8, "f16", 3),
    (1, 1, 8, 4, "f32", 0), (2, 3, 24, 16, "f16", 0), (2, 129, 100, 32, "f32", 1),
    (1, 300, 520, 1, "f16", 0), (1, 64, 2050, 8, "f16", 0), (2, 1500, 48, 64, "f16", 0),
    (1, 2000, 7, 3, "f32", 0)])
def test_fused_ragged_shapes(B, T, C, G, dtype, ld_pad):
    lc = I.LinearCase("ragged", B, T, C, 8, G, dtype, 0.1, 0.1, False, (T, 1), 700 + C)
    X, _ = I.make_activations(lc)
    _check(X, tdq.default_params(G), ld_pad)


@pytest.mark.parametrize("flags,tau,zr,base_pct", [(0, 1.0, 0.2, 0.0), (1, 0.3, 0.2, 0.0),
                                                   (2, 1.0, 0.05, 0.0), (3, 2.0, 0.9, 0.0),
                                                   (3, 1.0, 0.2, 0.99), (0, 1.0, 0.2, 0.5)])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_fused_variants(flags, tau, zr, base_pct, dtype):
    lc = I.case("cfg2_proj", B=2, dtype=dtype)
    X, _ = I.make_activations(lc)
    p = tdq.default_params(lc.G, tau=tau, zr=zr, flags=flags)
    p.base_pct = base_pct
    _check(X, p)


def test_fused_degenerate_and_nonfinite():
    rng = np.random.Generator(np.random.PCG64(9))
    X = rng.laplace(0, 1, (4, 40, 32)).astype(np.float16)
    X[0] = 0
    X[1] = np.float16(2.5)
    X[2, :20] = 0
    X[3, :, ::2] = 0
    g = _check(X, tdq.default_params(4))
    assert (g["clip"][0] == np.float32(1e-8)).all() and (g["clip"][1] == np.float32(1e-8)).all()
    Xn = np.ones((3, 16, 16), dtype=np.float16)
    Xn[1, 3, 5] = np.inf
    assert list(_fused(Xn, tdq.default_params(2))["flags"]) == [0, tdq.DEV_NONFINITE, 0]


def test_fused_agrees_with_the_multi_kernel_path():
    lc = I.case("cfg2_fc1", B=3)
    X, _ = I.make_activations(lc)
    p = tdq.default_params(lc.G)
    g = _fused(X, p)
    h = U.gpu_calibrate(X, p)
    assert np.array_equal(g["gid"], h["gid"])
    assert np.array_equal(g["stats"]["thr"], h["stats"]["thr"])
    assert np.array_equal(g["stats"]["c_base"], h["stats"]["c_base"])
    assert np.allclose(g["scale"], h["scale"], rtol=U.SCALE_RTOL, atol=0)


def test_fused_refuses_too_many_sets():
    X = torch.zeros((1, 16, 8), dtype=torch.float16, device=U.dev())
    with pytest.raises(tdq.TdqError) as e:
        tdq.tdq_calibrate_quantize_fused(X, tdq.default_params(65))
    assert e.value.status == tdq.ERR_UNSUPPORTED


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("B,T,C,G", [(2, 1, 8, 3), (1, 64, 64, 32), (3, 65, 32, 33), (2, 256, 64, 8), (2, 257, 64, 64),
                                     (1, 1024, 16, 17), (1, 1025, 16, 5), (2, 32, 512, 4), (2, 33, 520, 9)])
def test_register_resident_edges(B, T, C, G, dtype):
    """Images at and past the edge of what the single launch keeps in registers (tokens, row
    length, pieces), one and two LDS histograms, both passes of the rank select."""
    rng = np.random.Generator(np.random.PCG64(T + C))
    X = (rng.laplace(0, 1, (B, T, C)) * rng.lognormal(0, 1.2, (B, T, 1)) + 0.5)
    X = X.astype(np.float16 if dtype == "f16" else np.float32)
    for pct in (0.0, 0.9):
        p = tdq.default_params(G)
        p.base_pct = pct
        gid, clip, scale, stats, flags, Q, _ = tdq.tdq_calibrate_quantize_fused(
            torch.from_numpy(X).to(U.dev()), p, want_stats=True)
        torch.cuda.synchronize()
        assert int(flags.abs().sum()) == 0
        g = dict(gid=gid.cpu().numpy(), clip=clip.cpu().numpy(), scale=scale.cpu().numpy(),
                 stats=tdq.stats_to_numpy(stats))
        U.assert_calibration_matches(g, X, p)
        want = O.quantize_act(X, g["gid"], g["clip"], g["scale"], U.oracle_params(p)).reshape(B * T, C)
        assert np.array_equal(U.unpack_device_codes(Q, C), want)


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("B,T,C,G", [(128, 20, 64, 4), (171, 20, 64, 3), (8, 40, 32, 64), (9, 40, 32, 64), (1, 1024, 8, 2)])
def test_workgroup_per_set_and_per_image(B, T, C, G, dtype):
    """512 sets in all take a workgroup each, more of them one per image; with zeros, empty sets and a
    percentile, against the oracle."""
    rng = np.random.default_rng(B + G)
    X = np.maximum(rng.laplace(0, 1, (B, T, C)) * np.exp(rng.normal(0, 1.5, (B, T, 1))), -0.1).astype(dtype)
    X[0, : T // 2] = 0
    for pct in (0.0, 0.95):
        p = tdq.default_params(G)
        p.base_pct = pct
        _check(X, p)
