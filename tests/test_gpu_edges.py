"""GPU parity at the sizes where a kernel's tiling or a dispatch rule has its edges: tiles plus or minus one,
remainders, the smallest layers, both sides of a line between two variants."""
import numpy as np
import pytest

import workloads
from test_gpu_parity import both_configs, dev, gpu_bwd, gpu_fwd, rel_l2, xb  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def close_codes(got, want):
    """The code bar (one LSB on at most 1e-4 of the conversions) for few conversions: two may differ."""
    diff = np.abs(got.astype(np.int64) - want.astype(np.int64))
    return diff.max() <= 1 and (diff > 0).sum() <= max(2, 1e-4 * diff.size)


# M, K, N: odd weight counts (no 16-byte rows), one batch partial, the 8- and 32-group reductions, many weights; one kernel for
# gradient and write: one row, tiles of 32 plus and minus one, one and several rounds of partials, the largest batch and both
# sides of it, rows in fours or not, one or four weights per thread, many blocks
@pytest.mark.parametrize("M,K,N", [(5, 3, 7), (9000, 9, 5), (40000, 16, 12), (3000, 33, 65), (33, 1023, 513), (1025, 40, 16), (1, 1, 1),
                                   (31, 16, 17), (128, 15, 33), (129, 48, 16), (1024, 31, 20), (127, 65537, 5),
                                   (768, 33, 64), (769, 64, 33), (1024, 65, 516), (100, 500, 321), (17, 1000, 2044)])
@pytest.mark.parametrize("pair", [False, True])
def test_update_write(xo, xb, M, K, N, pair):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, False, 1), seed=M + K)
    co, cg = both_configs(xo, xb, flags=xo.UPD_NL | xo.UPD_NOISE, upd_nl_v=0.3, upd_noise_gamma=2.0, seed=5)
    w_max = 2.0 * float(np.abs(W).max())
    Wg = dev(W.copy())
    if pair:
        Gp, Gn = xo.pair_init(W, w_max)
        Gpg, Gng = dev(Gp.copy()), dev(Gn.copy())
        want = xo.update_pair(co, Gp, Gn, X, dY, w_max, 1.0 / w_max, 0.01, step=4)[2]
        xb.update_pair(cg, Gpg, Gng, Wg, dev(X), dev(dY), w_max, 1.0 / w_max, 0.01, step=4)
    else:
        want = xo.update(co, W, X, dY, w_max, 1.0 / w_max, 0.01, step=4)
        xb.update(cg, Wg, dev(X), dev(dY), w_max, 1.0 / w_max, 0.01, step=4)
    torch.cuda.synchronize()
    assert rel_l2(Wg.cpu().numpy() - W, want - W) <= 1e-3


# patches of 64 x 64 (32 x 32 with 4-bit cycles) weights, slices in pairs: one less, exact, one more; odd slice counts;
# arrays of whole 64-row steps and others (48: each copy on its own)
@pytest.mark.parametrize("R,sb,wb,slb", [(64, 1, 8, 2), (128, 1, 6, 2), (64, 4, 6, 2), (48, 1, 4, 2), (48, 4, 3, 1), (192, 2, 4, 4)])
@pytest.mark.parametrize("ni", ["aam", "var", "var+pa", "ideal"])
@pytest.mark.parametrize("K,N", [(1, 1), (63, 33), (64, 64), (65, 31), (193, 129)])
def test_generator(xo, xb, R, sb, wb, slb, ni, K, N):
    M = 4
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=K + 3 * N)
    flags = {"aam": xo.WIRE_AAM, "var": xo.VARIATION | xo.WIRE_AAM, "var+pa": xo.VARIATION | xo.ADC_PER_ARRAY, "ideal": 0}[ni]
    fs = 1.037 * workloads.adc_full_scale(R, sb, slb)             # off the binary grid: no ties
    co, cg = both_configs(xo, xb, xbar_rows=R, xbar_cols=R, weight_bits=wb, slice_bits=slb, stream_bits=sb,
                          flags=flags | xo.INPUT_SIGNED, var_sigma=0.1, seed=9, adc_fs_fwd=fs, adc_fs_bwd=fs)
    w_max, xs, gs = float(np.abs(W).max()), float(np.abs(X).max()), float(np.abs(dY).max())
    assert close_codes(gpu_fwd(xb, cg, W, X, w_max, xs, step=2)[1], xo.fwd(co, W, X, w_max, xs, step=2, want_codes=True)[1])
    assert close_codes(gpu_bwd(xb, cg, W, dY, w_max, gs, step=2)[1], xo.bwd(co, W, dY, w_max, gs, step=2, want_codes=True)[1])


E2M3 = np.array([m / 8 if e == 0 else (8 + m) / 8 * 2 ** (e - 1) for e in range(4) for m in range(8)])


def plane_terms(planes, R, K, N, S_w, arrays, exps, backward):
    """The terms of every plane value of one copy of a 6-bit plane buffer: [array][term][slice][K][N]."""
    Lc, Lo = (N, K) if backward else (K, N)
    T, OP, ks, terms = -(-Lc // R), -(-Lo // 32), -(-R // 64), len(exps)
    pol_bytes = T * OP * S_w * terms * ks * 1536
    start = 0
    if backward:
        start = (-(-K // R) * -(-N // 32) * S_w * terms * ks * 1536 * arrays + 1024 + 255) // 256 * 256
    raw = planes[start:start + pol_bytes * arrays].reshape(arrays, T, OP, S_w, terms, ks, 1536)
    records = np.concatenate([raw[..., :1024].reshape(raw.shape[:-1] + (64, 16)), raw[..., 1024:].reshape(raw.shape[:-1] + (64, 8))], axis=-1)
    bits = np.unpackbits(records, axis=-1, bitorder="little").reshape(raw.shape[:-1] + (64, 32, 6))
    codes = bits @ (1 << np.arange(6))
    values = E2M3[codes & 31] * np.where(codes & 32, -1.0, 1.0) * (2.0 ** np.array(exps))[None, None, None, None, :, None, None, None]
    lane, e = np.meshgrid(np.arange(64), np.arange(32), indexing="ij")
    row = 16 * (e // 8) + 8 * (lane // 32) + (e % 8) // 2 + 4 * (e % 2)
    out = np.zeros((arrays, terms, S_w, T, ks, 64, OP, 32))
    out[:, :, :, :, :, row, :, lane % 32] = values.transpose(6, 7, 0, 4, 3, 1, 5, 2)
    out = out.reshape(arrays, terms, S_w, T, ks * 64, OP * 32)[:, :, :, :, :R].reshape(arrays, terms, S_w, T * R, OP * 32)[..., :Lc, :Lo]
    return out.swapaxes(-1, -2) if backward else out


def nearest_terms(u, exps):
    """The E2M3 number nearest to what the terms before it left, times its power of two, term after term, in double precision
    (where that is exact the terms are); what cannot be held saturates."""
    terms = []
    for x in exps:
        a = np.fmin(np.abs(u), 7.5 * 2.0 ** x) / 2.0 ** x
        step = np.where(a < 2, 0.125, np.where(a < 4, 0.25, 0.5))
        terms.append(np.copysign(np.rint(a / step) * step * 2.0 ** x, u))
        u = u - terms[-1]
    return np.stack(terms, axis=1)


def profile_planes(xb, R, arrays, adc, distortion, seed):
    """Planes of 100 x 70 weights of two 2-bit slices with that stored distortion [slice][array][K][N], and what their terms have to be:
    conductances of whole quarters, so that every plane value of a distortion of 40 bits is exact in double precision."""
    K, N = 100, 70
    exps = [0, -4, -9, -14, -19]
    rng = np.random.default_rng(seed)
    q = rng.integers(-15, 16, size=(K, N))
    q[0, 0] = 15
    cfg = xb.make_config(xbar_rows=R, xbar_cols=R, weight_bits=4, slice_bits=2, stream_bits=1, adc_bits=adc, r_min=1.0, r_max=4.0,
                         flags=xb.NI_WIRE_PROFILE | (xb.ADC_PER_ARRAY if arrays == 2 else 0))
    planes = xb.tile(cfg, dev((q / 15.0).astype(np.float32)), 1.0, 0, dev(distortion.astype(np.float32))).cpu().numpy()
    digit = np.stack([(np.abs(q) >> (2 * s)) & 3 for s in range(2)])
    g = np.stack([np.where(q > 0, digit, 0), np.where(q < 0, digit, 0)]) * 0.25 + 0.25     # [array][slice][K][N]
    with np.errstate(invalid="ignore"):
        g = g * (1.0 - distortion.astype(np.float32).astype(np.float64).swapaxes(0, 1))
        u = g * 4.0 if arrays == 2 else (g[0] - g[1])[None] * 4.0
        want = nearest_terms(u, exps)
    return [plane_terms(planes, R, K, N, 2, arrays, exps, backward) for backward in (False, True)], want, u


# Arrays of whole 64-row steps and others write their planes through different kernels
@pytest.mark.parametrize("R", [64, 128, 48])
@pytest.mark.parametrize("arrays", [1, 2])
def test_plane_values_beyond_the_format(xb, R, arrays):
    rng = np.random.default_rng(7)
    distortion = rng.choice([np.inf, -np.inf, -1e30, -3.0, -6.25, -20.0, 0.5, 1.0, 0.0, np.nan], size=(2, 2, 100, 70))
    copies, want, u = profile_planes(xb, R, arrays, 13, distortion, seed=5)
    for got in copies:
        number = np.broadcast_to(~np.isnan(u)[:, None], want.shape)
        assert np.array_equal(got[number], want[number])
        assert np.array_equal(np.abs(got), np.abs(want))       # what is no number: the largest of either sign


# Values of some 40 bits, and values on the midpoints between two codes of a term or one bit of 2^-40 beside them: the terms are
# those that double precision gives, to the bit
@pytest.mark.parametrize("R", [64, 128, 48])
@pytest.mark.parametrize("arrays", [1, 2])
@pytest.mark.parametrize("kind", ["any", "midpoints", "beside"])
def test_terms_of_plane_values(xb, R, arrays, kind):
    rng = np.random.default_rng(R + arrays)
    shape = (2, 2, 100, 70)
    distortion = rng.uniform(2.0 ** -16, 0.3, size=shape).astype(np.float32)     # multiples of 2^-41
    if kind != "any":
        depth = rng.integers(4, 23, size=shape)                                  # odd multiples of 2^-depth, below 0.5
        distortion = (2 * rng.integers(0, 2 ** (depth - 2)) + 1) / 2.0 ** depth
        if kind == "beside":
            # ... and one single-precision step of that beside it: far below the last term's codes where it is small
            distortion = distortion.astype(np.float32) + np.ldexp(distortion, -23) * rng.choice([-1, 1], size=shape)
    copies, want, _ = profile_planes(xb, R, arrays, 13, distortion, seed=3)
    for got in copies:
        assert np.array_equal(got, want)


# Streamed walk: blocks of one device to fifteen, one device, queues that never fill and ones that always do,
# the power series of the non-linearity (v up to 1 / 32) and exp(), states that start beyond the range
@pytest.mark.parametrize("M,K,N,density,v,ni", [
    (2048, 1, 1, 4.0, 0.01, "nl+noise"), (2100, 31, 33, 4.0, 1.0 / 32, "nl"), (4200, 31, 33, 0.02, 0.01, "nl+noise"),
    (2049, 23, 45, 0.3, 0.0, ""), (4200, 96, 37, 0.5, 0.04, "nl+noise"), (2100, 96, 37, 0.05, 0.0, ""),
    (2049, 160, 80, 0.05, 0.01, "nl+noise"), (2048, 160, 80, 0.05, 0.04, "nl"), (2048, 300, 170, 0.02, 0.01, "nl+noise"),
    (2048, 51, 50, 0.3, 1.0 / 32, "nl+noise"), (2048, 51, 51, 0.3, 1.0 / 32, "nl"), (2048, 96, 63, 0.1, 0.01, "nl"), (2048, 96, 64, 0.1, 0.01, "nl")])
def test_pulsed_walk(xo, xb, M, K, N, density, v, ni):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=M + K + N)
    w_max = 0.5 * float(np.abs(W).max())
    flags = (xo.UPD_NL if "nl" in ni else 0) | (xo.UPD_NOISE if "noise" in ni else 0)
    co, cg = both_configs(xo, xb, flags=flags, upd_nl_v=v, upd_noise_gamma=0.4, seed=3)
    xr, dr, dw = 1.0 / density ** 0.5, 0.01 / density ** 0.5, 2.0 ** -10
    Wo, pulses_o = xo.update_pulsed(co, W, X, dY, w_max, xr, dr, 31, dw, step=6, want_pulses=True)
    Wg, pulses_g = xb.update_pulsed(cg, dev(W.copy()), dev(X), dev(dY), w_max, xr, dr, 31, dw, step=6, want_pulses=True)
    torch.cuda.synchronize()
    assert np.array_equal(pulses_g.cpu().numpy(), pulses_o)
    if ni:
        assert np.abs(Wg.cpu().numpy() - Wo).max() <= 2e-7 * np.abs(W).max()
    else:
        assert np.array_equal(Wg.cpu().numpy(), Wo)


# Moves far below the range, from weights of zero: the state is as exact about zero as a double is (moves of 2^-40 on a grid of
# 2^-53 would be off by 1e-4 of themselves); each pulse adds a few units in the last place of a move
@pytest.mark.parametrize("K,N", [(31, 33), (60, 60), (96, 70)])     # 4, 15 and 14 devices per block
@pytest.mark.parametrize("ni", ["nl", "nl+noise"])
def test_pulsed_walk_of_short_moves(xo, xb, K, N, ni):
    M = 2100
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=K + N)
    W[:] = 0.0
    flags = xo.UPD_NL | (xo.UPD_NOISE if "noise" in ni else 0)
    co, cg = both_configs(xo, xb, flags=flags, upd_nl_v=1.0 / 32, upd_noise_gamma=0.4, seed=3)
    Wo = xo.update_pulsed(co, W, X, dY, 0.7, 1.0, 0.01, 31, 2.0 ** -40, step=6)
    Wg = xb.update_pulsed(cg, dev(W.copy()), dev(X), dev(dY), 0.7, 1.0, 0.01, 31, 2.0 ** -40, step=6).cpu().numpy()
    assert np.abs(Wo).max() > 2.0 ** -39
    assert np.abs(Wg - Wo).max() <= 2.0 ** -23 * np.abs(Wo).max()


# ... layers of a wide range of device counts, for each cost of a move
@pytest.mark.parametrize("K,N,v,ni", [(128, 255, 0.0, ""), (128, 257, 0.0, ""), (128, 159, 0.01, "nl"), (128, 161, 0.01, "nl"), (64, 127, 0.04, "nl"),
                                      (64, 129, 0.04, "nl"), (128, 383, 0.0, "noise"), (128, 385, 0.0, "noise"), (128, 319, 0.01, "nl+noise"),
                                      (128, 321, 0.01, "nl+noise"), (128, 223, 0.04, "nl+noise"), (128, 225, 0.04, "nl+noise")])
def test_lines_of_the_pulsed_walk(xo, xb, K, N, v, ni):
    test_pulsed_walk(xo, xb, 2048, K, N, 0.02, v, ni)


# ... on both sides of the lines between the streamed walk and a lane per device
@pytest.mark.parametrize("K,N,v,ni", [(128, 431, 0.0, ""), (128, 433, 0.0, ""), (128, 367, 0.01, "nl"), (128, 369, 0.01, "nl"), (128, 207, 0.04, "nl"),
                                      (128, 209, 0.04, "nl"), (128, 575, 0.0, "noise"), (128, 577, 0.0, "noise"), (128, 239, 0.04, "nl+noise"),
                                      (128, 241, 0.04, "nl+noise"),
                                      (128, 511, 0.0, ""), (128, 513, 0.0, ""), (128, 607, 0.01, "nl"), (128, 609, 0.01, "nl"), (128, 703, 0.0, "noise"),
                                      (128, 705, 0.0, "noise"), (128, 543, 0.01, "nl+noise"), (128, 545, 0.01, "nl+noise"),
                                      (128, 415, 0.04, "nl+noise"), (128, 417, 0.04, "nl+noise")])
def test_lines_of_the_streamed_walk(xo, xb, K, N, v, ni):
    test_pulsed_walk(xo, xb, 2048, K, N, 0.02, v, ni)


# ... without marks: up to 8192 devices and fewer than 2048 samples; samples that fill no group of 64 or 256, rings that run full in the
# middle of a group, a last block of fewer devices, one block per compute unit and one device more
@pytest.mark.parametrize("M,K,N,density,v,ni", [
    (64, 1, 1, 4.0, 0.01, "nl+noise"), (63, 31, 33, 4.0, 0.01, "nl+noise"), (65, 31, 33, 4.0, 0.0, ""), (255, 31, 33, 4.0, 0.04, "nl+noise"),
    (257, 15, 17, 0.05, 0.01, "nl"), (320, 60, 64, 0.5, 0.01, "nl+noise"), (513, 60, 65, 0.02, 0.0, "noise"), (2047, 3, 7, 4.0, 0.01, "nl+noise"),
    (2047, 128, 64, 0.05, 0.04, "nl"), (300, 128, 65, 0.3, 0.01, "nl+noise")])
def test_streamed_walk_without_marks(xo, xb, M, K, N, density, v, ni):
    test_pulsed_walk(xo, xb, M, K, N, density, v, ni)


# ... and trains so dense that the rings run full in the middle of 64 samples: pulses in every slot, in most, and devices that run out
# of pulses at different times
@pytest.mark.parametrize("M,K,N", [(2048, 20, 40), (2100, 90, 64), (2048, 3, 5), (300, 20, 40)])
@pytest.mark.parametrize("v,ni", [(0.01, "nl"), (0.0, ""), (0.04, "nl"), (0.01, "nl+noise"), (0.0, "noise"), (0.04, "nl+noise")])
def test_streamed_walk_of_dense_trains(xo, xb, M, K, N, v, ni):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=M + K + N)
    X, dY = X / np.abs(X).max(), dY / np.abs(dY).max()
    X[:, ::2] = np.sign(X[:, ::2])
    dY[:, ::3] = np.sign(dY[:, ::3])
    X[: M // 2, 1::4] = 0.0
    w_max = float(np.abs(W).max())
    flags = (xo.UPD_NL if "nl" in ni else 0) | (xo.UPD_NOISE if "noise" in ni else 0)
    co, cg = both_configs(xo, xb, flags=flags, upd_nl_v=v, upd_noise_gamma=0.4, seed=3)
    Wo, pulses_o = xo.update_pulsed(co, W, X, dY, w_max, 1.0, 1.0, 31, 2.0 ** -10, step=6, want_pulses=True)
    Wg, pulses_g = xb.update_pulsed(cg, dev(W.copy()), dev(X), dev(dY), w_max, 1.0, 1.0, 31, 2.0 ** -10, step=6, want_pulses=True)
    assert np.array_equal(pulses_g.cpu().numpy(), pulses_o)
    assert np.abs(Wg.cpu().numpy() - Wo).max() <= 2e-7 * w_max     # one rounding to single precision


# Weights that are no numbers or lie at or beyond the range, in devices with pulses in every batch, in some and in none (rows
# that are driven often, rarely and never): every walk leaves what the pulse-by-pulse clamp leaves, to the bit of a zero
@pytest.mark.parametrize("M,K,N", [(2100, 20, 40), (2100, 64, 40), (2048, 300, 170), (300, 20, 40)])
@pytest.mark.parametrize("v,ni", [(0.01, "nl+noise"), (0.04, "nl"), (0.0, "")])
def test_pulsed_walk_of_special_weights(xo, xb, M, K, N, v, ni):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=M + K + N)
    w_max = 0.5 * float(np.abs(W).max())
    special = np.array([np.nan, -0.0, np.inf, -np.inf, 3e38, -w_max, w_max, 0.0], np.float32)
    rng = np.random.default_rng(K)
    at = rng.integers(0, K * N, K * N // 4)
    W.reshape(-1)[at] = special[rng.integers(0, special.size, at.size)]
    X[:, ::3] *= 0.02
    X[:, 1::3] = 0.0
    flags = (xo.UPD_NL if "nl" in ni else 0) | (xo.UPD_NOISE if "noise" in ni else 0)
    co, cg = both_configs(xo, xb, flags=flags, upd_nl_v=v, upd_noise_gamma=0.4, seed=3)
    Wo, pulses_o = xo.update_pulsed(co, W, X, dY, w_max, 1.0, 0.01, 31, 2.0 ** -10, step=6, want_pulses=True)
    Wg, pulses_g = xb.update_pulsed(cg, dev(W.copy()), dev(X), dev(dY), w_max, 1.0, 0.01, 31, 2.0 ** -10, step=6, want_pulses=True)
    Wg = Wg.cpu().numpy()
    assert np.array_equal(pulses_g.cpu().numpy(), pulses_o)
    assert np.array_equal(np.isnan(Wg), np.isnan(Wo)) and np.isnan(Wo).any()
    rest = np.isfinite(Wo)
    assert np.array_equal(Wg[~rest], Wo[~rest], equal_nan=True)
    assert np.abs(Wg[rest] - Wo[rest]).max() <= 2e-7 * w_max       # one rounding to single precision
    zero = Wo == 0
    assert np.array_equal(np.signbit(Wg[zero]), np.signbit(Wo[zero]))


# Gradient of layers whose rows are whole quads: one quad, tiles plus one, both stage lengths, batch rows that fill no stage or chunk,
# patches that lie outside the image, every width of tile; and layers beside them, whose rows are no quads.  A weight moves by the
# learning rate times its gradient, whose products are good to 2^-15 of themselves and whose sums are in single precision
@pytest.mark.parametrize("B,image,cin,cout,k,stride", [(5, 15, 4, 4, 1, 1), (9, 11, 4, 32, 3, 1), (42, 9, 20, 36, 3, 2), (21, 7, 64, 64, 3, 1), (27, 13, 8, 68, 5, 2),
                                                       (65, 8, 192, 128, 1, 2), (13, 9, 196, 132, 1, 1), (5, 16, 24, 12, 3, 1), (13, 9, 12, 200, 3, 1),
                                                       (1, 5, 24, 12, 3, 1), (13, 9, 6, 36, 3, 1), (13, 9, 8, 37, 3, 1), (40, 30, 16, 16, 3, 1)])
def test_gradient_of_whole_quads(xb, B, image, cin, cout, k, stride):
    from oracle import conv
    rng = np.random.default_rng(cin + cout)
    geom = xb.conv_geom(B, image, image, cin, k, k, stride, k // 2)
    X = rng.standard_normal((B, image, image, cin)).astype(np.float32)
    dY = rng.standard_normal((B, geom.out_h, geom.out_w, cout)).astype(np.float32)
    W = (rng.standard_normal((k * k * cin, cout)) * 0.1).astype(np.float32)
    cfg = xb.make_config(**dict(workloads.config_kwargs("resnet20"), flags=0))
    Wg = dev(W.copy())
    lr = np.float64(np.float32(1e-3))
    xb.conv_update(cfg, Wg, dev(X), dev(dY), geom, 64.0, 1.0 / 64.0, 1e-3, 0)
    P = conv.im2col(X, k, k, stride, k // 2).reshape(-1, k * k * cin).astype(np.float64)
    D = dY.reshape(-1, cout).astype(np.float64)
    bound = lr * 2.0 ** -15 * (np.abs(P).T @ np.abs(D)) + 2.0 ** -23 * 64.0
    assert (np.abs(Wg.cpu().numpy() - (W - lr * (P.T @ D))) <= bound).all()


# Circuit-level model, state on chip: one device, one row, one column, tiles plus one; wires that matter (many iterations)
@pytest.mark.parametrize("R,K,N,r_min", [(64, 1, 1, 1e5), (64, 65, 3, 1e3), (128, 1, 129, 1e5), (128, 130, 1, 1e4), (128, 40, 20, 1e3)])
def test_circuit_model_on_chip(xo, xb, R, K, N, r_min):
    from oracle import fcm
    W, _, _ = workloads.layer_tensors_np(workloads.Gemm("t", K, N, 1, True, 1), seed=K + 5 * N)
    co, cg = both_configs(xo, xb, xbar_rows=R, xbar_cols=R, weight_bits=2, slice_bits=2, flags=xo.VARIATION, var_sigma=0.05, seed=2,
                          r_min=r_min, r_max=10 * r_min, r_source=2.0, r_sense=3.0)
    w_max = float(np.abs(W).max())
    Dg = xb.fcm_profile(cg, dev(W), w_max, step=1)
    torch.cuda.synchronize()
    assert np.abs(Dg.cpu().numpy() - fcm.fcm_profile(co, W, w_max, step=1)).max() <= 2e-7


# ... solves that take over the coefficients of a block's first one: the first row of every block, or all but one device of it, off, so
# that the first solve hardly sees what the others do; two and many rows to a block; at 100 Ohm more iterations than coefficients are
# of, at 1 kOhm just about as many
@pytest.mark.parametrize("R,K,N,wb,r_min,off", [(64, 64, 40, 16, 1e2, "rows"), (64, 64, 64, 16, 1e3, "device"), (64, 300, 200, 2, 1e4, "rows"),
                                                (64, 128, 128, 16, 1e3, "rows"), (128, 150, 128, 2, 1e3, "device"), (128, 140, 30, 2, 1e5, "rows"),
                                                (128, 128, 20, 8, 1e2, "rows"), (128, 128, 20, 16, 1e4, "device")])
def test_circuit_model_with_shared_coefficients(xo, xb, R, K, N, wb, r_min, off):
    from oracle import fcm
    W, _, _ = workloads.layer_tensors_np(workloads.Gemm("t", K, N, 1, True, 1), seed=K + N)
    w_max = float(np.abs(W).max())
    co, cg = both_configs(xo, xb, xbar_rows=R, xbar_cols=R, weight_bits=wb, slice_bits=2, flags=0, r_min=r_min, r_max=10 * r_min,
                          r_source=2.0, r_sense=3.0)
    rows = xb.lib().xbar_fcm_rows_per_block(cg, K, N)
    assert rows >= 2
    W[::rows, (0 if off == "rows" else 1):] = 0.0
    Dg = xb.fcm_profile(cg, dev(W), w_max, step=1).cpu().numpy()
    assert np.abs(Dg - fcm.fcm_profile(co, W, w_max, step=1)).max() <= 2e-7


# ... and rows that see nothing of each other (no column wires), the first one of every block all off: its coefficients multiply the
# others' residuals by up to 1e20.  Each row is a system of its own.  (A profile of 64-bit sums, stored in single precision)
@pytest.mark.parametrize("R,r_min,r_row,r_source", [(128, 1e3, 4.6, 0.0), (128, 1e2, 1.0, 0.0), (64, 1e2, 4.6, 2.0), (64, 1e2, 10.0, 2.0),
                                                    (64, 1e4, 4.6, 2.0)])
def test_circuit_model_of_rows_apart(xo, xb, R, r_min, r_row, r_source):
    co, cg = both_configs(xo, xb, xbar_rows=R, xbar_cols=R, weight_bits=16, slice_bits=2, flags=0, r_min=r_min, r_max=10 * r_min,
                          r_row=r_row, r_col=0.0, r_source=r_source, r_sense=0.0)
    K, N = R, 2 * R
    W, _, _ = workloads.layer_tensors_np(workloads.Gemm("t", K, N, 1, True, 1), seed=R)
    w_max = float(np.abs(W).max())
    rows = xb.lib().xbar_fcm_rows_per_block(cg, K, N)
    assert rows >= 2
    W[::rows] = 0.0
    Dg = xb.fcm_profile(cg, dev(W), w_max, step=1).cpu().numpy()
    G = xo.device_conductances(co, W, w_max, 1)
    wires = r_source + r_row * (np.minimum.outer(np.arange(R), np.arange(R)) + 1.0)
    want = np.empty_like(G)
    for n0 in (0, R):
        g = G[..., n0:n0 + R]
        x = np.linalg.solve(np.eye(R) / g[..., None] + wires, np.ones(g.shape + (1,)))[..., 0]
        want[..., n0:n0 + R] = (g - x) / g
    assert np.abs(Dg - want).max() <= 2e-7


# One kernel for a whole pass (layers of few patches): its outputs are those of the chunked kernels, which the code tap
# runs, bit for bit -- one row, patches plus and minus one, slices that do not fill a block's waves, arrays of 16 .. 256
# rows, one and several blocks per patch, sums within and beyond 32 bits, every way of coding inputs and reading arrays
@pytest.mark.parametrize("R,sb,wb,slb,adc", [(64, 4, 8, 2, 8), (128, 1, 16, 2, 8), (48, 1, 5, 1, 12), (256, 2, 16, 4, 16),
                                             (192, 1, 6, 2, 8), (16, 8, 4, 4, 9), (256, 4, 10, 2, 15)])
@pytest.mark.parametrize("flags", ["", "aam", "aam+signed", "var+offset+signed", "pa+signed"])
@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (33, 300, 31), (32, 65, 130)])
def test_pass_of_a_small_layer(xb, R, sb, wb, slb, adc, flags, M, K, N):
    f = {"": 0, "aam": xb.NI_WIRE_AAM, "var": xb.NI_VARIATION, "signed": xb.INPUT_SIGNED, "offset": xb.INPUT_OFFSET,
         "pa": xb.ADC_PER_ARRAY}
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, "signed" in flags, 1), seed=M + K)
    fs = 1.037 * workloads.adc_full_scale(R, sb, slb)
    cfg = xb.make_config(xbar_rows=R, xbar_cols=R, weight_bits=wb, slice_bits=slb, stream_bits=sb, adc_bits=min(adc, 15), var_sigma=0.1,
                         flags=sum(f[x] for x in flags.split("+")), adc_fs_fwd=fs, adc_fs_bwd=fs, seed=4)
    w_max, xs, gs = float(np.abs(W).max()), float(np.abs(X).max()), float(np.abs(dY).max())
    assert np.array_equal(gpu_fwd(xb, cfg, W, X, w_max, xs, codes=False), gpu_fwd(xb, cfg, W, X, w_max, xs)[0])
    assert np.array_equal(gpu_bwd(xb, cfg, W, dY, w_max, gs, codes=False), gpu_bwd(xb, cfg, W, dY, w_max, gs)[0])


# Both sides of the lines beyond which several kernels take a pass again: blocks that fill the chip once (192 rows, fp16 planes),
# blocks whose time meets the chunked kernel's (6-bit planes), and a convolution that only its gathered inputs take beyond
@pytest.mark.parametrize("R,sb,wb,flags,M,K,N", [(192, 4, 8, 0, 512, 192, 512), (192, 4, 8, 0, 513, 192, 512),
                                                 (128, 1, 16, 1, 992, 64, 992), (128, 1, 16, 1, 993, 64, 992)])
def test_lines_of_the_small_pass(xb, R, sb, wb, flags, M, K, N):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, False, 1), seed=M + K)
    fs = 1.037 * workloads.adc_full_scale(R, sb, 2)
    cfg = xb.make_config(xbar_rows=R, xbar_cols=R, weight_bits=wb, slice_bits=2, stream_bits=sb, var_sigma=0.1,
                         flags=xb.NI_VARIATION if flags else xb.NI_WIRE_AAM, adc_fs_fwd=fs, adc_fs_bwd=fs, seed=4)
    w_max, xs, gs = float(np.abs(W).max()), float(np.abs(X).max()), float(np.abs(dY).max())
    assert np.array_equal(gpu_fwd(xb, cfg, W, X, w_max, xs, codes=False), gpu_fwd(xb, cfg, W, X, w_max, xs)[0])
    assert np.array_equal(gpu_bwd(xb, cfg, W, dY, w_max, gs, codes=False), gpu_bwd(xb, cfg, W, dY, w_max, gs)[0])


# Blocks of eight waves: weights of more than four slices whose patches take one block, or more blocks of four than there are
# compute units (240, 264); five, eight and sixteen slices, an odd number of cycles, one to four k-steps, one term, fp16 planes
@pytest.mark.parametrize("R,ib,sb,wb,slb,M,K,N", [(128, 8, 1, 16, 2, 320, 200, 180), (128, 8, 1, 16, 2, 350, 200, 180), (64, 8, 1, 10, 2, 350, 100, 180),
                                                  (192, 8, 1, 16, 1, 96, 300, 130), (128, 6, 2, 16, 2, 350, 200, 180), (128, 8, 4, 16, 2, 350, 200, 180),
                                                  (256, 8, 4, 16, 2, 97, 300, 180), (48, 8, 1, 14, 2, 350, 90, 180)])
@pytest.mark.parametrize("flags", ["", "aam", "aam+signed", "pa+signed"])
def test_eight_waves_of_the_small_pass(xb, R, ib, sb, wb, slb, M, K, N, flags):
    f = {"": 0, "aam": xb.NI_WIRE_AAM, "signed": xb.INPUT_SIGNED, "pa": xb.ADC_PER_ARRAY}
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, "signed" in flags, 1), seed=M + K)
    fs = 1.037 * workloads.adc_full_scale(R, sb, slb)
    cfg = xb.make_config(xbar_rows=R, xbar_cols=R, weight_bits=wb, slice_bits=slb, input_bits=ib, stream_bits=sb, adc_fs_fwd=fs, adc_fs_bwd=fs,
                         flags=sum(f[x] for x in flags.split("+")), seed=4)
    w_max, xs, gs = float(np.abs(W).max()), float(np.abs(X).max()), float(np.abs(dY).max())
    assert np.array_equal(gpu_fwd(xb, cfg, W, X, w_max, xs, codes=False), gpu_fwd(xb, cfg, W, X, w_max, xs)[0])
    assert np.array_equal(gpu_bwd(xb, cfg, W, dY, w_max, gs, codes=False), gpu_bwd(xb, cfg, W, dY, w_max, gs)[0])


# ... and both sides of the lines between which few inputs and up to four terms take blocks of four again (256, 272, 384, 400 blocks of eight)
@pytest.mark.parametrize("M", [512, 513, 768, 769])
@pytest.mark.parametrize("flags", ["aam+signed", "var+signed"])
def test_four_waves_of_few_inputs(xb, M, flags):
    K, N = 40, 256
    W, X, _ = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=M)
    fs = 1.037 * workloads.adc_full_scale(128, 1, 2)
    cfg = xb.make_config(xbar_rows=128, xbar_cols=128, weight_bits=16, slice_bits=2, stream_bits=1, var_sigma=0.1, adc_fs_fwd=fs, adc_fs_bwd=fs, seed=4,
                         flags=xb.INPUT_SIGNED | (xb.NI_VARIATION if "var" in flags else xb.NI_WIRE_AAM))
    assert xb.plane_format(cfg) == (1, 5 if "var" in flags else 4)
    w_max, xs = float(np.abs(W).max()), float(np.abs(X).max())
    assert np.array_equal(gpu_fwd(xb, cfg, W, X, w_max, xs, codes=False), gpu_fwd(xb, cfg, W, X, w_max, xs)[0])


# fp16 planes whose staged slices would be an odd number: six k-steps (64 KiB hold five slices of them), the same on 256-row arrays
# (eleven: two), slices that are an odd number themselves, one slice that no group of two holds
@pytest.mark.parametrize("R,wb,slb,M,K,N", [(128, 16, 2, 3000, 90, 200), (128, 14, 2, 3000, 90, 200), (256, 16, 2, 3000, 170, 100),
                                            (256, 16, 2, 3000, 250, 100), (256, 12, 1, 2500, 81, 100), (96, 10, 2, 2500, 250, 90)])
def test_staged_slices_come_in_pairs(xb, R, wb, slb, M, K, N):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=M + K)
    fs = 1.037 * workloads.adc_full_scale(R, 4, slb)
    cfg = xb.make_config(xbar_rows=R, xbar_cols=R, weight_bits=wb, slice_bits=slb, input_bits=8, stream_bits=4, adc_fs_fwd=fs, adc_fs_bwd=fs,
                         flags=xb.NI_WIRE_AAM | xb.INPUT_SIGNED, seed=4)
    w_max, xs, gs = float(np.abs(W).max()), float(np.abs(X).max()), float(np.abs(dY).max())
    assert np.array_equal(gpu_fwd(xb, cfg, W, X, w_max, xs, codes=False), gpu_fwd(xb, cfg, W, X, w_max, xs)[0])
    assert np.array_equal(gpu_bwd(xb, cfg, W, dY, w_max, gs, codes=False), gpu_bwd(xb, cfg, W, dY, w_max, gs)[0])


@pytest.mark.parametrize("cin,image", [(7, 31), (7, 25), (8, 31)])
def test_gathered_inputs_of_the_small_pass(xb, cin, image):
    from oracle import conv
    cout, K, M = 928, 9 * cin, image * image
    kw = dict(workloads.config_kwargs("resnet50"), var_sigma=0.1, seed=4)
    kw["flags"] |= xb.NI_VARIATION
    cfg = xb.make_config(**kw)
    W, X, _ = workloads.layer_tensors_np(workloads.Gemm("t", K, cout, M, False, 1), seed=image)
    X = np.abs(np.random.default_rng(image).standard_normal((1, image, image, cin))).astype(np.float32)
    w_max = float(np.abs(W).max())
    planes = xb.tile(cfg, dev(W), w_max, 0)
    Y = xb.conv_fwd(cfg, planes, dev(X), xb.conv_geom(1, image, image, cin, 3, 3, 1, 1), cout, w_max, 3.0)
    patches = np.ascontiguousarray(conv.im2col(X, 3, 3, 1, 1).reshape(M, K))
    assert torch.equal(Y.reshape(M, cout), xb.fwd(cfg, planes, dev(patches), cout, w_max, 3.0))


# Blocks that share a patch and find it never opened end by themselves after a bounded number of looks and say so with NaN
# (or, behind the sums that a gather reads, with what no sum is); the next pass on the same workspace is right, and so is
# every replay of a graph that holds one
@pytest.mark.parametrize("sb,flags", [(1, 0), (4, 0), (1, 512)])
def test_wait_for_a_patch_has_an_end(xb, sb, flags, M=40, K=300, N=70, wb=8):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=6)
    fs = 1.037 * workloads.adc_full_scale(64, sb, 2)
    cfg = xb.make_config(xbar_rows=64, xbar_cols=64, weight_bits=wb, slice_bits=2, stream_bits=sb, flags=flags | xb.INPUT_SIGNED,
                         adc_fs_fwd=fs, adc_fs_bwd=fs, seed=4)
    w_max = float(np.abs(W).max())
    planes, Xd = xb.tile(cfg, dev(W), w_max, 0), dev(X)
    ws = torch.empty(xb.workspace_bytes(cfg, xb.OP_FWD, M, K, N), dtype=torch.uint8, device="cuda").random_(0, 256)
    want = xb.fwd(cfg, planes, Xd, N, w_max, 3.0, ws=ws).clone()
    out = torch.empty_like(want)
    for turns in (0, 50):
        xb.lib().xbar_withhold_next_small_vmm(turns)
        xb.fwd(cfg, planes, Xd, N, w_max, 3.0, ws=ws, out=out)
        assert bool(torch.isnan(out).all())
        xb.fwd(cfg, planes, Xd, N, w_max, 3.0, ws=ws, out=out)
        assert torch.equal(out, want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        xb.fwd(cfg, planes, Xd, N, w_max, 3.0, ws=ws, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        xb.lib().xbar_withhold_next_small_vmm(3)
        xb.fwd(cfg, planes, Xd, N, w_max, 3.0, ws=ws, out=torch.empty_like(out))


@pytest.mark.parametrize("sb,flags", [(1, 0), (4, 0), (1, 512)])
def test_wait_for_a_patch_of_eight_waves_has_an_end(xb, sb, flags):
    test_wait_for_a_patch_has_an_end(xb, sb, flags, 200, 300, 130, 16)


# All-paths wire model: fewer rows than row segments, both strip widths (up to 128 rows and beyond), one to four columns
# per lane of the row scan, partial tiles down to one row or column
@pytest.mark.parametrize("R,C,slb", [(16, 16, 2), (48, 64, 4), (128, 128, 2), (144, 80, 1), (256, 256, 2)])
@pytest.mark.parametrize("ni", ["", "var", "var+pa"])
@pytest.mark.parametrize("K,N", [(1, 1), (129, 17), (65, 257), (300, 91)])
def test_all_paths_wire_model(xo, xb, R, C, slb, ni, K, N):
    M = 4
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=K + 7 * N)
    flags = xo.WIRE_AAM2 | xo.INPUT_SIGNED | (xo.VARIATION if "var" in ni else 0) | (xo.ADC_PER_ARRAY if "pa" in ni else 0)
    fs = 1.037 * workloads.adc_full_scale(max(R, C), 1, slb)
    co, cg = both_configs(xo, xb, xbar_rows=R, xbar_cols=C, weight_bits=4, slice_bits=slb, stream_bits=1, flags=flags,
                          var_sigma=0.1, seed=8, adc_fs_fwd=fs, adc_fs_bwd=fs, r_source=20.0, r_sense=30.0)
    w_max, xs, gs = float(np.abs(W).max()), float(np.abs(X).max()), float(np.abs(dY).max())
    assert close_codes(gpu_fwd(xb, cg, W, X, w_max, xs, step=2)[1], xo.fwd(co, W, X, w_max, xs, step=2, want_codes=True)[1])
    assert close_codes(gpu_bwd(xb, cg, W, dY, w_max, gs, step=2)[1], xo.bwd(co, W, dY, w_max, gs, step=2, want_codes=True)[1])


# One kernel for gradient and write: the partial sums of the two kernels, added up alike -- a convolution with a stride,
# which always takes those, writes the same weights bit for bit
@pytest.mark.parametrize("M,K,N", [(1, 5, 4), (33, 40, 16), (64, 256, 256), (700, 64, 30), (128, 784, 500), (1024, 300, 100)])
def test_update_of_few_rows_is_that_of_many(xb, M, K, N):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, False, 1), seed=M + N)
    cfg = xb.make_config(flags=xb.NI_UPD_NL | xb.NI_UPD_NOISE, upd_nl_v=0.3, upd_noise_gamma=2.0, seed=5)
    w_max = 2.0 * float(np.abs(W).max())
    one, two = dev(W.copy()), dev(W.copy())
    xb.update(cfg, one, dev(X), dev(dY), w_max, 1.0 / w_max, 0.01, step=4)
    geom = xb.conv_geom(M, 1, 1, K, 1, 1, 2, 0)
    xb.conv_update(cfg, two, dev(X).reshape(M, 1, 1, K), dev(dY).reshape(M, 1, 1, N), geom, w_max, 1.0 / w_max, 0.01, step=4)
    torch.cuda.synchronize()
    assert torch.equal(one, two)


# ... and on both sides of the lines: rows times blocks, blocks of rows in quads and of others with few rows, one and four
# weights per thread
@pytest.mark.parametrize("M,K,N", [(1024, 512, 1024), (1024, 544, 1024), (513, 1024, 1024), (40, 768, 767), (40, 800, 767), (96, 800, 767),
                                   (64, 512, 512), (64, 512, 516), (64, 2048, 1024), (64, 2080, 1024)])
def test_lines_of_the_update_in_one_kernel(xb, M, K, N):
    test_update_of_few_rows_is_that_of_many(xb, M, K, N)


# Batch rows many orders of magnitude apart: the partial sums are no longer added exactly, and the two ways of adding them may
# round differently, by the last bit of a weight.  Against the oracle: operands of two bfloat16 halves and products without
# the two low ones, 2^-15 of the sum of magnitudes, and the rounding of a weight.
@pytest.mark.parametrize("M,K,N", [(64, 256, 256), (700, 64, 30), (1024, 300, 100)])
def test_update_of_rows_of_all_magnitudes(xo, xb, M, K, N):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, True, 1), seed=M + N)
    rng = np.random.default_rng(M)
    X *= (2.0 ** rng.integers(-40, 1, (M, 1))).astype(np.float32)
    dY *= (2.0 ** rng.integers(-40, 1, (M, 1))).astype(np.float32)
    co, cg = both_configs(xo, xb, seed=5)
    w_max = 2.0 * float(np.abs(W).max())
    magnitude = np.abs(X).T.astype(np.float64) @ np.abs(dY).astype(np.float64)
    lr = 0.4 / float(magnitude.max())
    want = xo.update(co, W, X, dY, w_max, 1.0, lr, step=4)
    one, two = dev(W.copy()), dev(W.copy())
    xb.update(cg, one, dev(X), dev(dY), w_max, 1.0, lr, step=4)
    geom = xb.conv_geom(M, 1, 1, K, 1, 1, 2, 0)
    xb.conv_update(cg, two, dev(X).reshape(M, 1, 1, K), dev(dY).reshape(M, 1, 1, N), geom, w_max, 1.0, lr, step=4)
    one, two = one.cpu().numpy(), two.cpu().numpy()
    assert np.all(np.abs(one - two) <= np.spacing(np.abs(one)))
    assert np.all(np.abs(one.astype(np.float64) - want) <= 2.0 ** -15 * w_max * lr * magnitude + np.spacing(np.abs(want)))


# Convolution passes from NHWC images against the matrix passes on the patches: the same codes, and a pixel's errors added in
# single precision by kernel row and column -- equal bit for bit.  Kernels of no whole rounds of three positions, strides that
# leave pixels without a position, channels in fours or not, several partial sums, 64-bit sums, offset-coded inputs.
@pytest.mark.parametrize("batch,image,cin,cout,kernel,stride,pad,more", [
    (2, 7, 4, 33, 5, 3, 2, {}), (1, 9, 3, 16, 3, 2, 0, {}), (3, 6, 8, 40, 1, 2, 0, {}), (2, 5, 4, 17, 7, 1, 3, {}),
    (2, 8, 5, 64, 4, 1, 1, {}), (1, 1, 4, 5, 1, 3, 1, {}), (8, 28, 64, 600, 3, 1, 1, {}), (8, 28, 12, 300, 3, 2, 1, dict(adc_bits=12)),
    (2, 11, 6, 20, 3, 1, 1, dict(offset=True)), (2, 11, 8, 20, 4, 3, 1, dict(offset=True))])
def test_conv_is_its_patches(xb, batch, image, cin, cout, kernel, stride, pad, more):
    from oracle import conv
    kw = workloads.config_kwargs("resnet50")
    kw["flags"] |= xb.INPUT_OFFSET if more.get("offset") else xb.INPUT_SIGNED
    kw["adc_bits"] = more.get("adc_bits", kw["adc_bits"])
    cfg = xb.make_config(**kw)
    geom = xb.conv_geom(batch, image, image, cin, kernel, kernel, stride, pad)
    M, K = batch * geom.out_h * geom.out_w, kernel * kernel * cin
    rng = np.random.default_rng(M + K)
    W = rng.standard_normal((K, cout)).astype(np.float32) * 0.05
    X = rng.standard_normal((batch, image, image, cin)).astype(np.float32)
    dY = rng.standard_normal((M, cout)).astype(np.float32)
    w_max = float(np.abs(W).max())
    planes = xb.tile(cfg, dev(W), w_max, 0)
    Y = xb.conv_fwd(cfg, planes, dev(X), geom, cout, w_max, 3.0)
    patches = np.ascontiguousarray(conv.im2col(X, kernel, kernel, stride, pad).reshape(M, K))
    assert torch.equal(Y.reshape(M, cout), xb.fwd(cfg, planes, dev(patches), cout, w_max, 3.0))
    dX = xb.conv_bwd(cfg, planes, dev(dY).reshape(batch, geom.out_h, geom.out_w, cout), geom, cout, w_max, 3.0).cpu().numpy()
    cols = xb.bwd(cfg, planes, dev(dY), K, w_max, 3.0).cpu().numpy().reshape(batch, geom.out_h, geom.out_w, kernel, kernel, cin)
    side = (max(geom.out_h, geom.out_w) - 1) * stride + kernel + image + pad
    want = np.zeros((batch, side, side, cin), np.float32)
    for kh in range(kernel):
        for kw_ in range(kernel):
            want[:, kh:kh + geom.out_h * stride:stride, kw_:kw_ + geom.out_w * stride:stride] += cols[:, :, :, kh, kw_]
    assert np.array_equal(dX, want[:, pad:pad + image, pad:pad + image])


# How a block leaves its sums: scaled outputs, 32- and 64-bit partial sums, sums widened on the way, rows that are whole quads
# and others, the last patch of rows and outputs.  A row's outputs do not depend on the rows beside it, and few rows are cut
# into more chunks of the contraction, or taken by one kernel.
@pytest.mark.parametrize("R,sb,wb,adc,M,K,signed", [(128, 1, 16, 8, 40000, 64, False), (128, 1, 16, 8, 3000, 300, True), (16, 1, 16, 8, 52500, 128, True),
                                                    (128, 4, 16, 8, 30000, 144, True), (64, 4, 16, 12, 3000, 300, True),
                                                    (128, 1, 16, 10, 40000, 64, False), (128, 1, 12, 13, 3000, 300, True), (256, 1, 16, 10, 9000, 300, True),
                                                    (128, 1, 16, 15, 20000, 2000, True)])
@pytest.mark.parametrize("N", [97, 98, 99, 100])
def test_rows_do_not_depend_on_the_batch(xb, R, sb, wb, adc, M, K, signed, N):
    fs = 1.037 * workloads.adc_full_scale(R, sb, 2)
    cfg = xb.make_config(xbar_rows=R, xbar_cols=R, weight_bits=wb, slice_bits=2, stream_bits=sb, adc_bits=adc,
                         flags=xb.NI_WIRE_AAM | (xb.INPUT_SIGNED if signed else 0), adc_fs_fwd=fs, adc_fs_bwd=fs, seed=4)
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    W = torch.randn((K, N), generator=gen, device="cuda")
    X = torch.randn((M, K), generator=gen, device="cuda")
    dY = torch.randn((M, N), generator=gen, device="cuda")
    planes = xb.tile(cfg, W, 5.0, 0)
    Y, dX = xb.fwd(cfg, planes, X, N, 5.0, 3.0), xb.bwd(cfg, planes, dY, K, 5.0, 3.0)
    for rows in (slice(0, 70), slice(M - 1000, M)):
        assert torch.equal(Y[rows], xb.fwd(cfg, planes, X[rows].clone(), N, 5.0, 3.0))
        assert torch.equal(dX[rows], xb.bwd(cfg, planes, dY[rows].clone(), K, 5.0, 3.0))


# Two 32-bit sums per output, widened on the way because a chunk has more virtual tiles than they hold: five, seven and six of three,
# 46 of 45 (fp16 planes), five of three with one converter per array.  Ideal arrays: the oracle's bits, of the first and the last rows
@pytest.mark.parametrize("R,sb,adc,M,K,N,backward,per_array", [
    (64, 1, 16, 20000, 2000, 97, False, False), (64, 1, 16, 20000, 100, 2000, True, False), (16, 1, 16, 20000, 700, 99, False, False),
    (16, 4, 16, 40000, 2576, 100, False, False), (128, 1, 15, 20000, 2000, 98, False, True)])
def test_two_sums_widened_on_the_way(xo, xb, R, sb, adc, M, K, N, backward, per_array):
    fs = workloads.adc_full_scale(R, sb, 2)
    co, cg = both_configs(xo, xb, xbar_rows=R, xbar_cols=R, weight_bits=16, slice_bits=2, input_bits=8, stream_bits=sb, adc_bits=adc,
                          flags=xo.INPUT_SIGNED | (xo.ADC_PER_ARRAY if per_array else 0), adc_fs_fwd=fs, adc_fs_bwd=fs)
    # what the plan has to be for the case to be one, read off the workspace
    Lin, Lout = (N, K) if backward else (K, N)
    q_adc = 2 ** adc - 1 if per_array else 2 ** (adc - 1) - 1
    weights = [sum(1 << (2 * s + sb * b) for s in range(n) for b in range(8 // sb)) for n in (4, 8)]
    held = (2 ** 31 - 1) // (weights[0] * q_adc)
    tiles = -(-Lin // R)
    digits = -(-(2 * -(-M // 32) * tiles * (R // 16) * 512) // 256) * 256
    chunks = (xb.workspace_bytes(cg, xb.OP_BWD if backward else xb.OP_FWD, M, K, N) - digits) // (8 * M * Lout)
    longest = -(-2 * tiles * (2 if per_array else 1) // chunks)
    assert weights[1] * q_adc >= 2 ** 31 and 1 <= held < longest and longest % held

    rng = np.random.default_rng(M + N)
    W = rng.standard_normal((K, N), dtype=np.float32)
    rows = np.r_[0:40, M - 40:M]
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    A = torch.randn((M, Lin), generator=gen, device="cuda")
    planes = xb.tile(cg, dev(W), 5.0, 0)
    got = (xb.bwd(cg, planes, A, K, 5.0, 4.0) if backward else xb.fwd(cg, planes, A, N, 5.0, 4.0))[rows].cpu().numpy()
    want = (xo.bwd if backward else xo.fwd)(co, W, A[rows].cpu().numpy(), 5.0, 4.0)
    if per_array:
        # planes that are no whole device levels: the bits of the launch that reports codes and adds them up in 64 bits, and the output bar
        assert np.array_equal(got, xb.fwd(cg, planes, A[rows].clone(), N, 5.0, 4.0, want_codes=True)[0].cpu().numpy())
        assert rel_l2(got, want) <= 1e-3
    else:
        assert np.array_equal(got, want)


# Few rows: waves without rows of their own share the streaming cycles (eight, two, one; sums in 32 bits, two of them, 64-bit
# ones of odd slice counts), also in shorter chunks where sums hold fewer tiles than a batch that fills the waves has in one
# (32-row arrays): the outputs are those of the same rows in such a batch
@pytest.mark.parametrize("R,sb,wb,adc,signed", [(128, 1, 16, 8, True), (256, 2, 16, 10, False), (128, 4, 16, 8, True), (64, 8, 8, 8, False),
                                                (128, 1, 16, 12, True), (128, 1, 14, 14, False), (32, 1, 16, 8, True)])
@pytest.mark.parametrize("M", [1, 33, 64, 65, 128, 129])
def test_few_rows_share_the_cycles(xb, R, sb, wb, adc, signed, M):
    K, N = 2500, 4100
    fs = 1.037 * workloads.adc_full_scale(R, sb, 2)
    cfg = xb.make_config(xbar_rows=R, xbar_cols=R, weight_bits=wb, slice_bits=2, stream_bits=sb, adc_bits=adc,
                         flags=xb.NI_WIRE_AAM | (xb.INPUT_SIGNED if signed else 0), adc_fs_fwd=fs, adc_fs_bwd=fs, seed=4)
    gen = torch.Generator(device="cuda").manual_seed(M)
    W = torch.randn((K, N), generator=gen, device="cuda")
    X = torch.randn((300, K), generator=gen, device="cuda")
    dY = torch.randn((300, N), generator=gen, device="cuda")
    planes = xb.tile(cfg, W, 5.0, 0)
    assert torch.equal(xb.fwd(cfg, planes, X[:M].clone(), N, 5.0, 3.0), xb.fwd(cfg, planes, X, N, 5.0, 3.0)[:M])
    assert torch.equal(xb.bwd(cfg, planes, dY[:M].clone(), K, 5.0, 3.0), xb.bwd(cfg, planes, dY, K, 5.0, 3.0)[:M])
