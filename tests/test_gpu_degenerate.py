"""GPU parity on the degenerate inputs the quantizers special-case, for every
family: all-zero tokens and groups (scale or norm 0), constant rows (KIVI's
min-max range 0), single-channel spikes, and bf16 values beyond the fp16
range (the fp16 metadata saturates at 65504), and queries far above and
below unit scale.  Codes, metadata and the window must match the oracle
(TurboQuant codes by its near-threshold rule); attention must match it
everywhere, to 1e-2 at unit scale and in proportion beyond."""
import numpy as np
import pytest

import paper_2605_06675_amd as rq
import workloads
from oracle import cache as ocache
from tests import gpu_helpers as gh
from tests import test_gpu_parity as gp
from tests import test_gpu_turbo as gt

pytestmark = pytest.mark.gpu

H, G, T, R, BATCH = 4, 4, 224, 32, 2


def _data(seed, scale=1.0):
    """[B][H][T][128] float32: every 7th token zero, then constant rows,
    single spikes, whole-zero 32-token blocks for one head, Gaussian rest."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((BATCH, H, T, 128))
    t = np.arange(T)
    x[:, :, t % 7 == 0] = 0.0
    x[:, :, t % 7 == 1] = 0.5
    spike = t % 7 == 2
    x[:, :, spike] = 0.0
    x[:, :, spike, 17] = 12.0
    x[:, 1, 32:64] = 0.0                      # one block all zero (keys: s = 0)
    x[:, 2, 64:96, :40] = -3.0                # constant channels over a block
    return x * scale


def _fill(family, dtype, bits, kf, vf, rotation=None):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    ks = [workloads.bits16_from_f32(kf[b], dtype) for b in range(BATCH)]
    vs = [workloads.bits16_from_f32(vf[b], dtype) for b in range(BATCH)]
    kvc = rq.KVCache(family, dtype, 1, BATCH, H, H * G, T, R, bits,
                     rotation=rotation)
    K, V = gh.dev(np.stack(ks), dtype), gh.dev(np.stack(vs), dtype)
    kvc.append(0, K[:, :, :150].contiguous(), V[:, :, :150].contiguous())
    kvc.append(0, K[:, :, 150:].contiguous(), V[:, :, 150:].contiguous())
    torch.cuda.synchronize()
    return kvc, ks, vs


@pytest.mark.parametrize("family,bits", [
    (workloads.KIVI, [[1, 4], [2, 3], [3, 2], [8, 1]]),
    (workloads.QUAROT, [[2, 4], [3, 3], [4, 2], [8, 5]]),
    (workloads.RTN, [[2, 4], [3, 3], [4, 2], [8, 5]]),
    (workloads.KIVI_RTN, [[1, 4], [2, 3], [3, 2], [8, 2]])],
    ids=["kivi", "quarot", "rtn", "kivi_rtn"])
@pytest.mark.parametrize("dtype", [workloads.F16, workloads.BF16])
def test_degenerate_affine_families(family, bits, dtype):
    print(f"degenerate family {family} dtype {dtype}", flush=True)
    bits = np.array([bits])
    kvc, ks, vs = _fill(family, dtype, bits, _data(1), _data(2))
    units = gp._check_cache(family, dtype, kvc, ks, vs, bits, R, BATCH, H, T)
    gp._check_attention(kvc, units, dtype, BATCH, H, G)


@pytest.mark.parametrize("family", [workloads.KIVI, workloads.QUAROT,
                                    workloads.RTN, workloads.KIVI_RTN],
                         ids=["kivi", "quarot", "rtn", "kivi_rtn"])
def test_saturated_metadata_bf16(family):
    # |x| up to ~1e7: scales and zero points saturate at the fp16 maximum
    print(f"saturated metadata family {family}", flush=True)
    bits = np.array([[[2, 3], [3, 2], [4, 4], [5, 6]]])
    kvc, ks, vs = _fill(family, workloads.BF16, bits, _data(3, 2.0e5), _data(4, 2.0e5))
    units = gp._check_cache(family, workloads.BF16, kvc, ks, vs, bits, R, BATCH, H, T)
    gp._check_attention(kvc, units, workloads.BF16, BATCH, H, G)


@pytest.mark.parametrize("q_mult", [1.0e6, 1.0e-6], ids=["q1e6", "q1e-6"])
@pytest.mark.parametrize("family", [workloads.KIVI, workloads.QUAROT,
                                    workloads.RTN, workloads.KIVI_RTN],
                         ids=["kivi", "quarot", "rtn", "kivi_rtn"])
def test_large_values_and_queries(family, q_mult):
    # value scales near the fp16 maximum (probability x scale beyond the
    # fp16 range) and queries whose scaled elements leave it (q1e6) or
    # underflow it (q1e-6)
    print(f"large values family {family} q x {q_mult:g}", flush=True)
    bits = np.array([[[2, 2], [3, 2], [4, 3], [8, 5]]])
    rng = np.random.default_rng(11)
    kf = rng.standard_normal((BATCH, H, T, 128))
    vf = rng.standard_normal((BATCH, H, T, 128)) * 3.0e4
    kvc, ks, vs = _fill(family, workloads.BF16, bits, kf, vf)
    units = gp._check_cache(family, workloads.BF16, kvc, ks, vs, bits, R, BATCH, H, T)
    gp._check_attention(kvc, units, workloads.BF16, BATCH, H, G, q_mult=q_mult)


def test_degenerate_turbo():
    print("degenerate turbo", flush=True)
    dtype = workloads.BF16
    bits = np.array([[[1, 4], [2, 3], [3, 2], [4, 4]]])
    r16, rf = gt._rotations(1, H)
    kvc, ks, vs = _fill(workloads.TURBO, dtype, bits, _data(5), _data(6),
                        rotation=gh.dev(r16, workloads.BF16))
    units = gt._check(dtype, kvc, ks, vs, rf[0], bits, R, BATCH, H)
    gt._attention(kvc, units, dtype, BATCH, H, G)


@pytest.mark.parametrize("q_mult", [1.0e6, 1.0e-6], ids=["q1e6", "q1e-6"])
def test_large_values_and_queries_turbo(q_mult):
    # norms near the fp16 maximum (probability x norm / sqrt(128) beyond
    # the fp16 range) and queries far from unit scale; widths 1..8
    print(f"large values turbo q x {q_mult:g}", flush=True)
    dtype = workloads.BF16
    bits = np.array([[[1, 6], [3, 8], [5, 2], [7, 4]]])
    rng = np.random.default_rng(12)
    kf = rng.standard_normal((BATCH, H, T, 128))
    vf = rng.standard_normal((BATCH, H, T, 128)) * 5.0e3
    r16, rf = gt._rotations(1, H)
    kvc, ks, vs = _fill(workloads.TURBO, dtype, bits, kf, vf,
                        rotation=gh.dev(r16, workloads.BF16))
    units = gt._check(dtype, kvc, ks, vs, rf[0], bits, R, BATCH, H)
    gt._attention(kvc, units, dtype, BATCH, H, G, q_mult=q_mult)


@pytest.mark.parametrize("family,bits", [(workloads.KIVI, [2, 4]), (workloads.RTN, [2, 3]),
                                         (workloads.KIVI_RTN, [2, 2])],
                         ids=["kivi", "rtn", "kivi_rtn"])
@pytest.mark.parametrize("phase", range(4))
def test_large_value_scales_at_some_tokens(family, bits, phase):
    # value scales beyond 4094 at every fourth token only: a lane of the
    # attention kernel holds four token pairs, and whichever of them carries
    # the large scale, the value exponent has to follow (probabilities above
    # 1 against a lagging maximum times such a scale leave fp16's range)
    import torch
    B, Hk, Tl = 8, 8, 4096
    rng = np.random.default_rng(31 + phase)
    base = rng.standard_normal((Tl, 128))
    base[np.arange(Tl) % 4 == phase] *= 12000.0
    v16 = workloads.bits16_from_f32(np.clip(base, -60000, 60000), workloads.F16)
    k16 = workloads.bits16_from_f32(rng.standard_normal((Hk, Tl, 128)), workloads.F16)
    K = gh.dev(k16, workloads.F16)[None].expand(B, Hk, Tl, 128).contiguous()
    V = gh.dev(v16, workloads.F16)[None, None].expand(B, Hk, Tl, 128).contiguous()
    table = np.array([[bits] * Hk])
    kvc = rq.KVCache(family, workloads.F16, 1, B, Hk, Hk * G, Tl, 0, table)
    kvc.append(0, K, V)
    q16 = workloads.bits16_from_f32(2.0 * rng.standard_normal((B, Hk * G, 128)), workloads.F16)
    out = kvc.attention(0, gh.dev(q16, workloads.F16))
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert np.all(np.isfinite(out))
    from oracle import attention as oatt
    for b, h in ((0, 0), (B - 1, Hk - 1)):
        u = ocache.Unit(family, workloads.u16_to_f32(k16[h], workloads.F16),
                        workloads.u16_to_f32(v16, workloads.F16), *bits, 0)
        q = workloads.u16_to_f32(q16[b, h * G:(h + 1) * G], workloads.F16)
        v_hat = u.values()
        want = oatt.decode_attention(q, u.keys(), v_hat)
        err = np.max(np.abs(out[b, h * G:(h + 1) * G] - want))
        assert err < gp.attention_tol(v_hat), (b, h, err)


@pytest.mark.parametrize("q_exp", [122, 44, -121])
def test_scales_far_from_one(q_exp):
    # queries around 2^q_exp and a scale that brings them back to 2^-3: the
    # raw products of the 16-bit window's rows leave fp32's range (q_exp 122;
    # 44 is inside it on both sides) or fall among its least normal numbers
    # (-121), while scale * q is ordinary, for the window and for the blocks
    import torch
    from oracle import attention as oatt
    scale = 2.0 ** (-3 - q_exp)
    bits = np.array([[[2, 2], [3, 2], [4, 3], [8, 5]]])
    rng = np.random.default_rng(13)
    kf = 8.0 * rng.standard_normal((BATCH, H, T, 128))
    kvc, ks, vs = _fill(workloads.KIVI, workloads.BF16, bits, kf, rng.standard_normal(kf.shape))
    units = gp._check_cache(workloads.KIVI, workloads.BF16, kvc, ks, vs, bits, R, BATCH, H, T)
    q16 = workloads.bits16_from_f32(
        (rng.standard_normal((BATCH, H * G, 128)) * 2.0 ** q_exp).astype(np.float32),
        workloads.BF16)
    out = kvc.attention(0, gh.dev(q16, workloads.BF16), scale=scale)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert np.all(np.isfinite(out))
    for (b, h), u in units.items():
        q = workloads.u16_to_f32(q16[b, h * G:(h + 1) * G], workloads.BF16).astype(np.float64)
        v_hat = u.values()
        want = oatt.decode_attention(q, u.keys(), v_hat, scale)
        err = np.max(np.abs(out[b, h * G:(h + 1) * G] - want))
        assert err < gp.attention_tol(v_hat), (b, h, err)


@pytest.mark.parametrize("T_win", [1, 21, 32, 45])
def test_infinite_value_of_the_last_window_token(T_win):
    # an infinity in the newest token's values shows in its own channel only:
    # the places behind it, up to a whole chunk of 32, have no part in it
    import torch
    dtype = workloads.F16
    rng = np.random.default_rng(14)
    kf, vf = rng.standard_normal((2, 1, 2, T_win, 128))
    vf[:, :, -1, 5] = np.inf
    k16, v16 = (workloads.bits16_from_f32(x, dtype) for x in (kf, vf))
    kvc = rq.KVCache(workloads.KIVI, dtype, 1, 1, 2, 2 * G, 64, 64, np.array([[[2, 2], [3, 3]]]))
    kvc.append(0, gh.dev(k16, dtype), gh.dev(v16, dtype))
    q16 = workloads.bits16_from_f32(rng.standard_normal((1, 2 * G, 128)), dtype)
    out = kvc.attention(0, gh.dev(q16, dtype))
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert np.all(out[:, :, 5] == np.inf)
    assert np.all(np.isfinite(np.delete(out, 5, axis=2)))


@pytest.mark.parametrize("group", [1, 4, 6, 16])
def test_equal_values_give_equal_channels(group):
    # the query replicas behind the four 32-channel groups of KIVI's values
    # hold the same probabilities to the bit, so values that are equal over
    # the channels give outputs that are; keys with outlier channels make the
    # zero-point sums large, whose order would otherwise show (many units, so
    # that a wave has several blocks under one running maximum)
    import torch
    dtype, batch, heads, tokens = workloads.F16, 128, 4, 1024
    rng = np.random.default_rng(15)
    kf = rng.standard_normal((heads, tokens, 128))
    kf[..., 7::16] += 3000.0 * np.abs(rng.standard_normal((heads, 1, 8)))
    vf = np.broadcast_to(rng.choice([-2.0, -1.0, 0.5, 3.0], (heads, tokens, 1)), kf.shape)
    K, V = (gh.dev(workloads.bits16_from_f32(np.ascontiguousarray(x), dtype), dtype)[None]
            .expand(batch, heads, tokens, 128).contiguous() for x in (kf, vf))
    kvc = rq.KVCache(workloads.KIVI, dtype, 1, batch, heads, heads * group, tokens, 0,
                     np.array([[[2, 2], [4, 3], [3, 1], [6, 5]]]))
    kvc.append(0, K, V)
    q16 = workloads.bits16_from_f32(
        np.abs(rng.standard_normal((batch, heads * group, 128))), dtype)
    out = kvc.attention(0, gh.dev(q16, dtype))
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert np.all(np.isfinite(out))
    np.testing.assert_array_equal(out, np.broadcast_to(out[..., :1], out.shape))
