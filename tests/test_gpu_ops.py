"""Kernel-level parity on the GPU: each kernel of the step against the
oracle's layer function on the same (bf16-representable) inputs."""
import math

import numpy as np
import pytest

from fixtures import bf16_round
from oracle import ops as O
from tests.gpu_util import log, rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = {"f32": 2e-6, "bf16": 1.2e-2}


def _tdt(dt):
    return torch.bfloat16 if dt == "bf16" else torch.float32


def _vals(rng, shape, dt, scale=1.0):
    x = (rng.standard_normal(shape) * scale).astype(np.float32)
    return bf16_round(x) if dt == "bf16" else x


def _dev(x, dt=None):
    t = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return t.to(_tdt(dt)) if dt else t


@pytest.fixture(scope="module")
def ops():
    from paper_2605_08835_amd import ops as P
    return P


def _pack(w):
    cout, cin, k, _ = w.shape
    return np.ascontiguousarray(w.transpose(0, 2, 3, 1).reshape(cout, k * k * cin))


CONV_CASES = [
    # n, H, W, c0, c1, cout, ks, stride, up, affine
    (2, 12, 10, 64, 0, 96, 3, 1, 0, False),
    (3, 8, 8, 32, 48, 64, 3, 1, 0, True),
    (2, 16, 16, 64, 0, 64, 3, 2, 0, False),
    (2, 6, 5, 64, 0, 128, 3, 1, 1, False),
    (2, 9, 7, 40, 24, 136, 1, 1, 0, False),
    (1, 20, 20, 8, 0, 320, 3, 1, 0, False),
    (3, 8, 8, 320, 0, 4, 3, 1, 0, True),
    # widths that take the direct-to-LDS pipeline (N % 160, cin % 32), ragged M
    (3, 10, 9, 64, 0, 160, 3, 1, 0, False),
    (2, 8, 8, 64, 96, 320, 3, 1, 0, False),
    (2, 12, 12, 160, 0, 160, 3, 2, 0, False),
    (2, 5, 7, 160, 0, 320, 3, 1, 1, False),
    (2, 9, 7, 64, 32, 160, 1, 1, 0, False),
    (64, 16, 16, 64, 0, 160, 3, 1, 0, False),
    # long-K layers on small images: split K (ragged row counts)
    (3, 4, 4, 640, 0, 320, 3, 1, 0, False),
    (5, 2, 2, 1280, 0, 160, 3, 1, 0, False),
    (2, 4, 4, 640, 640, 320, 3, 1, 0, False),
    (3, 4, 4, 1280, 0, 160, 3, 2, 0, False),
    (2, 2, 2, 640, 0, 320, 3, 1, 1, False),
    # many rows (ragged, concat, stride 2, upsampling)
    (65, 32, 32, 64, 0, 320, 3, 1, 0, False),
    (32, 32, 32, 64, 64, 640, 3, 1, 0, False),
    (64, 64, 64, 32, 0, 320, 3, 2, 0, False),
    (64, 16, 16, 64, 0, 320, 3, 1, 1, False),
    (67, 32, 32, 320, 0, 320, 1, 1, 0, False),
    # more blocks than fit on the chip at once (ragged, split K)
    (130, 32, 32, 64, 0, 160, 3, 1, 0, False),
    (150, 8, 8, 640, 0, 320, 3, 1, 0, False),
    # stride-1 3x3 beyond 8x8: split K whose second half starts inside a
    # channel block's kernel row (19 blocks, 171 K tiles), concat sources
    (2, 16, 16, 608, 0, 160, 3, 1, 0, False),
    (3, 16, 16, 320, 320, 320, 3, 1, 0, False),
    (2, 24, 40, 96, 64, 160, 3, 1, 0, False),
    (1, 17, 9, 32, 0, 160, 3, 1, 0, False),
    # widths that are multiples of 128 but not of 160 (the VAE decoder's): 64x64
    # and, for the last, 128x128 direct-to-LDS tiles (ragged, concat, upsampling, 1x1)
    (2, 12, 12, 128, 0, 128, 3, 1, 0, False),
    (3, 9, 10, 256, 0, 256, 3, 1, 0, False),
    (2, 6, 6, 512, 0, 256, 3, 1, 1, False),
    (2, 16, 16, 128, 128, 256, 1, 1, 0, False),
    (40, 16, 16, 128, 0, 512, 3, 1, 0, False),
]


@pytest.mark.parametrize("with_resid", [True, False])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", CONV_CASES)
def test_conv(ops, dt, case, with_resid):
    n, H, W, c0, c1, cout, ks, stride, up, aff = case
    log(f"conv {dt} {case} resid={with_resid}")
    rng = np.random.default_rng(hash(case) % 2**32)
    x0 = _vals(rng, (n, H, W, c0), dt)
    x1 = _vals(rng, (n, H, W, c1), dt) if c1 else None
    w = _vals(rng, (cout, c0 + c1, ks, ks), dt, 1.0 / math.sqrt(ks * ks * (c0 + c1)))
    b = rng.standard_normal(cout).astype(np.float32)
    Ho, Wo = (2 * H, 2 * W) if up else (H // stride, W // stride)
    res = _vals(rng, (n, Ho, Wo, cout), dt)
    scale = shift = None
    if aff:
        scale = (1 + 0.3 * rng.standard_normal((n, c0 + c1))).astype(np.float32)
        shift = (0.3 * rng.standard_normal((n, c0 + c1))).astype(np.float32)
    out_f32 = cout == 4
    got = ops.conv(_dev(x0, dt), _dev(_pack(w), dt), cout, ks, stride, up,
                   x1=_dev(x1, dt) if c1 else None,
                   scale=_dev(scale) if aff else None, shift=_dev(shift) if aff else None, silu=int(aff),
                   bias=_dev(b), resid=_dev(res, dt) if with_resid and not out_f32 else None, out_f32=out_f32)
    torch.cuda.synchronize()
    got = got.float().cpu().numpy()
    for i in range(n):
        a = x0[i].astype(np.float64) if not c1 else np.concatenate([x0[i], x1[i]], axis=2).astype(np.float64)
        if aff:
            a = O.silu(a * scale[i] + shift[i])
        if up:
            a = O.upsample_nearest2x(a)
        ref = O.conv2d(a, w, b, stride) + (res[i] if with_resid and not out_f32 else 0)
        err = rel_l2(got[i], ref)
        assert err <= TOL[dt], (i, err)


def _phase_weights(w):
    """[cout, cin, 3, 3] -> [4, cout, 4 cin]: the 2x2 kernel of each output
    phase (py, px) of a nearest-2x upsample followed by the 3x3 conv (the
    taps that land on the same input pixel, summed)."""
    cout, cin = w.shape[:2]
    out = np.zeros((4, cout, 4, cin), np.float64)
    for py in range(2):
        for px in range(2):
            for ky in range(3):
                for kx in range(3):
                    # upsampled row 2y + py + ky - 1 is input row y + (py + ky - 1) // 2
                    ty, tx = (py + ky - 1) // 2 - (py - 1), (px + kx - 1) // 2 - (px - 1)
                    out[2 * py + px, :, 2 * ty + tx, :] += w[:, :, ky, kx]
    return out.reshape(4, cout, 4 * cin)


# n, H, W, cin, cout: ragged grids and the SD-1.5 / SDXL upsampling widths
UPCONV_CASES = [(2, 5, 7, 64, 160), (3, 8, 9, 32, 320), (2, 16, 16, 160, 320), (1, 4, 4, 640, 640),
                (4, 8, 8, 1280, 1280), (1, 1, 3, 32, 160), (70, 4, 4, 64, 160)]


@pytest.mark.parametrize("case", UPCONV_CASES)
def test_upconv_phases(ops, case):
    """The four-phase form of upsample + 3x3 conv against the oracle's
    nearest upsampling and direct convolution (fp64)."""
    n, H, W, cin, cout = case
    log(f"upconv {case}")
    rng = np.random.default_rng(n * 1000 + H * 10 + cin + cout)
    x = _vals(rng, (n, H, W, cin), "bf16")
    w = _vals(rng, (cout, cin, 3, 3), "bf16", 1.0 / math.sqrt(9 * cin))
    b = rng.standard_normal(cout).astype(np.float32)
    wp = bf16_round(_phase_weights(w.astype(np.float64)).astype(np.float32))
    got = ops.upconv(_dev(x, "bf16"), _dev(wp, "bf16"), cout, bias=_dev(b))
    torch.cuda.synchronize()
    got = got.float().cpu().numpy()
    for i in range(n):
        ref = O.conv2d(O.upsample_nearest2x(x[i].astype(np.float64)), w, b, 1)
        err = rel_l2(got[i], ref)
        assert err <= TOL["bf16"], (i, err)


def test_upconv_rejects_unsupported_widths(ops):
    x = torch.zeros(1, 4, 4, 32, device="cuda", dtype=torch.bfloat16)
    w = torch.zeros(4, 36, 4 * 32, device="cuda", dtype=torch.bfloat16)
    with pytest.raises(RuntimeError):
        ops.upconv(x, w, 36)


@pytest.mark.parametrize("qmode", ["plain", "log2"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("heads,d,nq,nk,scale,cross", [
    (2, 8, 70, 70, 1.0, False), (2, 16, 33, 8, 1.0, True), (4, 32, 200, 200, 1.0, False),
    (8, 40, 300, 300, 1.0, False), (8, 40, 129, 77, 1.0, True), (2, 64, 256, 256, 30.0, False),
    (8, 80, 160, 160, 1.0, False), (8, 160, 64, 64, 1.0, False), (8, 160, 90, 77, 1.0, True),
    (2, 40, 36, 36, 1.0, False), (2, 24, 130, 130, 1.0, False), (1, 48, 64, 200, 30.0, True),
    (4, 56, 65, 129, 1.0, False), (2, 72, 100, 100, 1.0, False), (2, 128, 70, 70, 1.0, False),
    # key counts in whole 8-key chunks take the direct-to-LDS tiles (partial last tile, folded max)
    (8, 40, 130, 256, 1.0, False), (2, 24, 100, 64, 30.0, True), (8, 40, 64, 200, 1.0, True),
    (4, 56, 96, 136, 1.0, False), (8, 40, 32, 8, 1.0, True), (2, 64, 70, 520, 30.0, False),
    # last tiles of at most 32 keys (the half tail at d = 40, 72, 80, 160)
    (2, 72, 50, 90, 1.0, True), (4, 80, 40, 96, 1.0, True),
])
def test_attention(ops, dt, qmode, heads, d, nq, nk, scale, cross):
    """bf16 takes V transposed (channel-major, padded token stride, as the
    step stores it), fp32 row-major V; "log2" passes Q pre-multiplied by
    scale * log2(e) and rounded once, as the projection epilogue writes it,
    and the reference uses exactly that Q (divided back in float64)."""
    log(f"attention {dt} {qmode} heads={heads} d={d} nq={nq} nk={nk} x{scale} cross={cross}")
    rng = np.random.default_rng(d * 1000 + nq)
    C = heads * d
    n = 3
    nkv = 2 if cross else n
    q = _vals(rng, (n, nq, C), dt, scale)
    k = _vals(rng, (nkv, nk, C), dt, scale)
    v = _vals(rng, (nkv, nk, C), dt)
    idx = np.array([1, 0, 1], np.int32) if cross else None
    o = torch.empty(n, nq, C, device="cuda", dtype=_tdt(dt))
    sm = 1.0 / math.sqrt(d)
    qref = q.astype(np.float64)
    if qmode == "log2":
        sl2 = sm * math.log2(math.e)
        q = bf16_round((q.astype(np.float64) * sl2).astype(np.float32))
        qref = q.astype(np.float64) / sl2
    if dt == "bf16":  # channel-major V with a padded token stride
        ld = (nk + 7) // 8 * 8
        vdev = torch.zeros(nkv, C, ld, device="cuda", dtype=_tdt(dt))
        vdev[:, :, :nk] = _dev(v, dt).transpose(1, 2)
        v_ld, v_img = ld, C * ld
    else:
        vdev, v_ld, v_img = _dev(v, dt), C, nk * C
    ops.attention(_dev(q, dt), _dev(k, dt), vdev, o, n, heads, d, nq, nk, C, nq * C, C, nk * C, v_ld, v_img,
                  C, nq * C, sm, kv_index=_dev(idx) if cross else None, v_transposed=dt == "bf16",
                  q_log2=qmode == "log2")
    torch.cuda.synchronize()
    got = o.float().cpu().numpy()
    for i in range(n):
        j = idx[i] if cross else i
        ref = O.attention(qref[i], k[j].astype(np.float64), v[j].astype(np.float64), heads)
        err = rel_l2(got[i], ref)
        # fp32 scores carry a relative rounding error ~2^-24 |s|; with logits
        # scaled x30 (|s| ~ 1e3) that reaches the output as ~1e-4.
        tol = TOL[dt] if (dt == "bf16" or scale == 1.0) else 2e-4
        assert err <= tol, (i, err)


@pytest.mark.parametrize("log2", [False, True])
@pytest.mark.parametrize("d,nk,dead", [(8, 8, (3,)), (8, 8, (0,)), (16, 77, tuple(range(10, 77))), (40, 130, (0, 16, 32, 48, 64)),
                                       (64, 65, tuple(range(64))), (128, 40, (0, 1, 33)), (32, 6, tuple(range(6)))])
def test_attention_f32_minus_inf_scores(ops, d, nk, dead, log2):
    """Keys that score -inf have no weight, whichever lane or tile they fall
    to and also as the first ones; with no other key the result is NaN."""
    heads, n, nq = 2, 1, 21
    log(f"attention f32 -inf d={d} nk={nk} dead={len(dead)}")
    rng = np.random.default_rng(d + nk)
    C = heads * d
    q, k, v = (rng.standard_normal((n, t, C)).astype(np.float32) for t in (nq, nk, nk))
    q[:, :, ::d] = np.abs(q[:, :, ::d]) + 0.1  # channel 0 of each head: positive, so -inf there scores -inf
    kd = k.copy()
    kd[:, dead, ::d] = -np.inf
    o = torch.empty(n, nq, C, device="cuda")
    ops.attention(_dev(q), _dev(kd), _dev(v), o, n, heads, d, nq, nk, C, nq * C, C, nk * C, C, nk * C, C, nq * C,
                  1.0 / math.sqrt(d), q_log2=log2)
    got = o.cpu().numpy()[0].astype(np.float64)
    if len(dead) == nk:
        assert np.isnan(got).all()
        return
    live = [i for i in range(nk) if i not in dead]
    qs = q[0].astype(np.float64) * (math.sqrt(d) * math.log(2) if log2 else 1.0)  # base-2 scores, no scale
    ref = O.attention(qs, k[0][live].astype(np.float64), v[0][live].astype(np.float64), heads)
    # base-2 scores reach some 20: a relative rounding of 2^-24 each is 1e-6 in the probabilities
    assert rel_l2(got, ref) <= (1e-5 if log2 else TOL["f32"])


@pytest.mark.parametrize("d", [8, 16, 40, 64])
@pytest.mark.parametrize("nk", [1, 2, 16, 17, 32, 33, 65])
def test_attention_f32_key_counts(ops, d, nk):
    """fp32 attention at the edges of its forms (1, up to 32 and more keys),
    ragged query blocks; the first image alone gives the same bits."""
    heads, n, nq = 3, 2, 70
    log(f"attention f32 keys d={d} nk={nk}")
    rng = np.random.default_rng(100 * d + nk)
    C = heads * d
    q, k, v = (rng.standard_normal((n, t, C)).astype(np.float32) for t in (nq, nk, nk))

    def run(m):
        o = torch.empty(m, nq, C, device="cuda")
        ops.attention(_dev(q), _dev(k), _dev(v), o, m, heads, d, nq, nk, C, nq * C, C, nk * C, C, nk * C, C, nq * C,
                      1.0 / math.sqrt(d))
        return o.cpu().numpy()

    got = run(n)
    assert np.array_equal(run(1), got[:1])
    for i in range(n):
        ref = O.attention(*(t[i].astype(np.float64) for t in (q, k, v)), heads)
        assert rel_l2(got[i], ref) <= TOL["f32"]


@pytest.mark.parametrize("pad,off", [(16, 0), (4, 0), (16, 4)])
@pytest.mark.parametrize("d,nq,nk", [(40, 129, 77), (40, 128, 77), (64, 300, 64), (80, 33, 130), (160, 70, 90),
                                     (160, 193, 90), (24, 5, 8)])
def test_attention_strided_output(ops, d, nq, nk, pad, off):
    """Output rows wider than the heads (ragged last query block): the columns
    and rows outside the result keep their values.  Rows may start at multiples
    of 8 bytes only (pad 4: every other one; off 4: all of them)."""
    heads, n = 2, 2
    log(f"attention strided output d={d} nq={nq} nk={nk} pad={pad} off={off}")
    rng = np.random.default_rng(d + nq)
    C = heads * d
    q, k, v = (_vals(rng, (n, t, C), "bf16") for t in (nq, nk, nk))
    ld = (nk + 7) // 8 * 8
    vdev = torch.zeros(n, C, ld, device="cuda", dtype=torch.bfloat16)
    vdev[:, :, :nk] = _dev(v, "bf16").transpose(1, 2)
    flat = torch.full((off + n * (nq + 3) * (C + pad),), 7.0, device="cuda", dtype=torch.bfloat16)
    o = flat[off:]
    ops.attention(_dev(q, "bf16"), _dev(k, "bf16"), vdev, o, n, heads, d, nq, nk, C, nq * C, C, nk * C, ld, C * ld,
                  C + pad, (nq + 3) * (C + pad), 1.0 / math.sqrt(d), v_transposed=True)
    torch.cuda.synchronize()
    assert (flat[:off] == 7.0).all()
    got = o.float().cpu().numpy().reshape(n, nq + 3, C + pad)
    assert (got[:, nq:] == 7.0).all() and (got[:, :, C:] == 7.0).all()
    for i in range(n):
        ref = O.attention(q[i].astype(np.float64), k[i].astype(np.float64), v[i].astype(np.float64), heads)
        assert rel_l2(got[i, :nq, :C], ref) <= TOL["bf16"]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("n,H,W,c0,c1,G,eps", [(2, 8, 8, 64, 0, 32, 1e-5), (2, 16, 12, 320, 0, 32, 1e-6),
                                               (3, 8, 8, 64, 32, 32, 1e-5), (2, 4, 4, 1280, 640, 32, 1e-5),
                                               (2, 64, 64, 320, 0, 32, 1e-5), (1, 16, 16, 32, 32, 8, 1e-5),
                                               # many pixel ranges (four-wave finalize; 256 at most, ragged)
                                               (1, 301, 277, 128, 0, 32, 1e-6), (2, 130, 131, 256, 64, 32, 1e-6)])
def test_groupnorm(ops, dt, n, H, W, c0, c1, G, eps):
    log(f"groupnorm {dt} {(n, H, W, c0, c1, G)}")
    rng = np.random.default_rng(c0 + c1 + H)
    x0 = _vals(rng, (n, H, W, c0), dt, 2.0) + np.float32(0.5)
    x0 = bf16_round(x0) if dt == "bf16" else x0
    x1 = _vals(rng, (n, H, W, c1), dt) if c1 else None
    g = (1 + 0.1 * rng.standard_normal(c0 + c1)).astype(np.float32)
    b = (0.1 * rng.standard_normal(c0 + c1)).astype(np.float32)
    sc, sh = ops.groupnorm_stats(_dev(x0, dt), G, eps, _dev(g), _dev(b), x1=_dev(x1, dt) if c1 else None)
    torch.cuda.synchronize()
    sc, sh = sc.cpu().numpy().astype(np.float64), sh.cpu().numpy().astype(np.float64)
    for i in range(n):
        a = x0[i].astype(np.float64) if not c1 else np.concatenate([x0[i], x1[i]], axis=2).astype(np.float64)
        ref = O.group_norm(a, G, g, b, eps)
        err = rel_l2(a * sc[i] + sh[i], ref)
        assert err <= 1e-5, (i, err)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("T,C", [(37, 64), (300, 320), (64, 1280), (5, 2048)])
def test_layernorm(ops, dt, T, C):
    log(f"layernorm {dt} {(T, C)}")
    rng = np.random.default_rng(T + C)
    x = _vals(rng, (T, C), dt, 3.0)
    g = (1 + 0.1 * rng.standard_normal(C)).astype(np.float32)
    b = (0.1 * rng.standard_normal(C)).astype(np.float32)
    y = ops.layernorm(_dev(x, dt), _dev(g), _dev(b))
    torch.cuda.synchronize()
    err = rel_l2(y.float().cpu().numpy(), O.layer_norm(x.astype(np.float64), g, b))
    assert err <= (2e-6 if dt == "f32" else 6e-3), err


# every tokens-per-wave variant (C <= 512: 4 tokens per wave; wider: 2, with
# 2-4 vectors per lane) and token counts that end inside a wave's group
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("T,C", [(1, 8), (19, 40), (1003, 320), (6, 512), (9, 640), (131, 1280), (7, 2048),
                                 (0, 320)])
def test_layernorm_rstd(ops, dt, T, C):
    log(f"layernorm_rstd {dt} {(T, C)}")
    rng = np.random.default_rng(7 * T + C)
    x = _vals(rng, (T, C), dt, 3.0) + _vals(rng, (T, 1), dt, 2.0)
    x = bf16_round(x) if dt == "bf16" else x
    r = ops.layernorm_rstd(_dev(x, dt))
    torch.cuda.synchronize()
    r = r.cpu().numpy().astype(np.float64)
    assert r.shape == (T,)
    if T == 0:
        return
    # (x - mean) * rstd is the oracle's LayerNorm with unit gain and no shift
    xd = x.astype(np.float64)
    got = (xd - xd.mean(axis=1, keepdims=True)) * r[:, None]
    err = rel_l2(got, O.layer_norm(xd, np.ones(C), np.zeros(C)))
    assert err <= 2e-6, err


def _silu(x):
    return x / (1.0 + np.exp(-x))


# M, K, N, weight dtype, silu_in, silu_out, bias, add: the time-embedding
# shapes (320 -> 1280 -> 1280, SDXL's 2816 -> 1280, the stacked time
# projections 1280 -> 20160) and ragged ones (K not a multiple of the
# 256-wide chunk, N not a multiple of a block's 16 columns, M over 32).
LINEAR_ROWS_CASES = [
    (2, 32, 128, "f32", 0, 1, True, False),
    (3, 36, 5, "f32", 1, 0, False, True),
    (32, 320, 1280, "bf16", 0, 1, True, False),
    (32, 1280, 1280, "bf16", 1, 0, True, True),
    (33, 1280, 20160, "bf16", 1, 0, True, False),
    (70, 2816, 1280, "bf16", 0, 1, True, False),
    (1, 1000, 37, "bf16", 1, 1, False, False),
    (0, 64, 16, "bf16", 0, 0, True, False),
]


@pytest.mark.parametrize("case", LINEAR_ROWS_CASES)
def test_linear_rows(ops, case):
    M, K, N, dt, si, so, with_bias, with_add = case
    log(f"linear_rows {case}")
    rng = np.random.default_rng(M * 7 + K + N)
    x = rng.standard_normal((M, K)).astype(np.float32)
    w = _vals(rng, (N, K), dt, 0.05)
    b = (0.1 * rng.standard_normal(N)).astype(np.float32) if with_bias else None
    add = rng.standard_normal((M, N)).astype(np.float32) if with_add else None
    y = ops.linear_rows(_dev(x), _dev(w, dt), None if b is None else _dev(b), None if add is None else _dev(add),
                        si, so)
    torch.cuda.synchronize()
    xd = x.astype(np.float64)
    ref = (_silu(xd) if si else xd) @ w.astype(np.float64).T
    if b is not None:
        ref = ref + b
    if add is not None:
        ref = ref + add
    if so:
        ref = _silu(ref)
    if M == 0:
        assert y.shape == (0, N)
        return
    assert rel_l2(y.cpu().numpy(), ref) <= 2e-6


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_geglu(ops, dt):
    log(f"geglu {dt}")
    rng = np.random.default_rng(5)
    x = _vals(rng, (77, 2 * 320), dt, 2.0)
    y = ops.geglu(_dev(x, dt))
    torch.cuda.synchronize()
    xd = x.astype(np.float64)
    ref = xd[:, :320] * O.gelu(xd[:, 320:])
    err = rel_l2(y.float().cpu().numpy(), ref)
    assert err <= (2e-6 if dt == "f32" else 6e-3), err


@pytest.mark.parametrize("n", [1, 3, 6])
def test_conv_split_k_rows_independent(ops, n):
    """The split-K path gives each image the same bits whatever the batch."""
    rng = np.random.default_rng(21)
    x = _vals(rng, (6, 4, 4, 640), "bf16")
    w = _vals(rng, (320, 640, 3, 3), "bf16", 0.01)
    wp = _dev(_pack(w), "bf16")
    full = ops.conv(_dev(x, "bf16"), wp, 320).float().cpu().numpy()
    part = ops.conv(_dev(x[:n], "bf16"), wp, 320).float().cpu().numpy()
    nosplit = ops.conv(_dev(x[:n], "bf16"), wp, 320, split=False).float().cpu().numpy()
    assert np.array_equal(full[:n], part)
    err = rel_l2(part, nosplit)
    log(f"split-K n={n}: rel L2 vs one pass {err:.2e}")
    assert err < 1e-2


def test_conv_large_grid_rows_independent(ops):
    """An image gets the same bits in a grid of 560 tiles as alone."""
    rng = np.random.default_rng(22)
    x = _vals(rng, (140, 32, 32, 64), "bf16")
    w = _vals(rng, (160, 64, 3, 3), "bf16", 0.05)
    wp = _dev(_pack(w), "bf16")
    full = ops.conv(_dev(x, "bf16"), wp, 160)[:3].float().cpu().numpy()
    part = ops.conv(_dev(x[:3], "bf16"), wp, 160).float().cpu().numpy()
    assert np.array_equal(full, part)


WIDE_CASES = [
    # n, H, W, c0, c1, cout, resid, split.  The whole batch takes the wide tile
    # named, its first three images alone the 64x64 or 128x64 one.
    (40, 16, 16, 1280, 0, 1280, True, True),    # 256x256, split in 2 (16x16 images), 400 blocks
    (40, 16, 16, 1280, 0, 1280, True, False),   # 256x256, one pass, 200 blocks
    (130, 8, 8, 640, 0, 1280, True, True),      # 256x256, 8x8 images: tap-outer K order, split in 4
    (113, 12, 12, 1280, 0, 512, False, True),   # 128x128, ragged last row tile (16272 rows), no split
    (35, 31, 31, 128, 192, 256, True, True),    # 256x256, concat sources, K = 2880, ragged (33635 rows)
    (90, 12, 12, 1280, 0, 1280, True, True),    # 256x256, split in 2 with a ragged last row tile (12960 rows)
    # source widths that are no multiples of 64: the 32-deep 256x128 tile for the
    # batch and the three images alike (here only the oracle checks it)
    (35, 31, 31, 160, 160, 256, True, True),
]


@pytest.mark.parametrize("case", WIDE_CASES)
def test_conv_wide_tiles(ops, case):
    """The wide tiles on long K give every image the same bits as the narrow
    ones (its first images run alone on those) and match the oracle on the first
    and last image."""
    n, H, W, c0, c1, cout, with_resid, split = case
    log(f"wide tiles {case}")
    rng = np.random.default_rng(hash(case) % 2**32)
    x0 = _vals(rng, (n, H, W, c0), "bf16")
    x1 = _vals(rng, (n, H, W, c1), "bf16") if c1 else None
    w = _vals(rng, (cout, c0 + c1, 3, 3), "bf16", 1.0 / math.sqrt(9 * (c0 + c1)))
    b = rng.standard_normal(cout).astype(np.float32)
    res = _vals(rng, (n, H, W, cout), "bf16") if with_resid else None
    wp, bd = _dev(_pack(w), "bf16"), _dev(b)

    def run(k):
        return ops.conv(_dev(x0[:k], "bf16"), wp, cout, x1=_dev(x1[:k], "bf16") if c1 else None, bias=bd,
                        resid=_dev(res[:k], "bf16") if with_resid else None, split=split).float().cpu().numpy()

    full, part = run(n), run(3)
    torch.cuda.synchronize()
    assert np.array_equal(full[:3], part)
    for i in (0, n - 1):
        a = x0[i].astype(np.float64) if not c1 else np.concatenate([x0[i], x1[i]], axis=2).astype(np.float64)
        ref = O.conv2d(a, w, b, 1) + (res[i] if with_resid else 0)
        err = rel_l2(full[i], ref)
        assert err <= TOL["bf16"], (i, err)


TILE64_CASES = [
    # n, H, W, c0, c1, cout, ks, stride, up: 64-deep K stages.  The whole batch
    # takes one tile, its first image alone the 64x64 (width 160: 128x160) one;
    # ragged row counts, so that the last row tile is partly empty.
    (11, 53, 57, 64, 0, 64, 3, 1, 0),     # 128x64 (33231 rows)
    (7, 71, 67, 64, 0, 128, 3, 1, 0),     # 128x128 (33299 rows), one channel block
    (5, 61, 67, 64, 64, 160, 3, 1, 0),    # 128x160 only, concat sources
    (33, 33, 31, 128, 64, 256, 3, 1, 0),  # 256x256 (33759 rows), concat sources
    (9, 61, 61, 64, 0, 320, 3, 1, 0),     # 256x320 (33489 rows)
    (130, 8, 8, 64, 128, 1280, 3, 1, 0),  # 256x256 on 8x8 images (taps outer), concat sources
    (33, 32, 32, 64, 0, 256, 3, 2, 0),    # 128x64, stride 2
    (33, 66, 62, 64, 0, 256, 3, 2, 0),    # 256x256, stride 2 (33759 rows)
    (33, 66, 62, 64, 0, 320, 3, 2, 0),    # 256x320, stride 2 (33759 rows)
    (9, 30, 31, 64, 0, 320, 3, 1, 1),     # 256x320, upsampling
    (1, 1, 33003, 192, 64, 320, 1, 1, 0),  # linear, concat sources
    (2, 3, 1, 64, 0, 64, 3, 1, 0),        # six rows
    (1, 1, 1, 64, 0, 64, 1, 1, 0),        # one row, one K stage
    (1, 1, 49100, 128, 128, 256, 1, 1, 0),  # few channels, 384 blocks: 32-deep 256x128, concat sources
    # linear layers of one source, which have a setup of their own, on every tile
    (1, 1, 49100, 192, 0, 256, 1, 1, 0),   # 32-deep 256x128, two per CU
    (1, 1, 33231, 128, 0, 64, 1, 1, 0),    # 128x64
    (1, 1, 33299, 128, 0, 128, 1, 1, 0),   # 128x128
    (1, 1, 20435, 64, 0, 160, 1, 1, 0),    # 128x160
    (1, 1, 33759, 320, 0, 256, 1, 1, 0),   # 256x256
    (1, 1, 65300, 64, 0, 320, 1, 1, 0),    # 256x320
    (1, 1, 301, 96, 0, 160, 1, 1, 0),      # 32-deep 64x160
    (1, 1, 65600, 32, 0, 160, 1, 1, 0),    # 32-deep 256x160, one K tile
    (1, 1, 7001, 1056, 0, 256, 1, 1, 0),   # 32-deep 256x128
]


@pytest.mark.parametrize("case", TILE64_CASES)
def test_conv_tiles64(ops, case):
    """Every tile of the 64-deep direct-to-LDS kernel: the first image gets the
    same bits in the whole batch as alone, and the last one (ragged rows)
    matches the oracle."""
    n, H, W, c0, c1, cout, ks, stride, up = case
    log(f"tiles64 {case}")
    rng = np.random.default_rng(hash(case) % 2**32)
    x0 = _vals(rng, (n, H, W, c0), "bf16")
    x1 = _vals(rng, (n, H, W, c1), "bf16") if c1 else None
    w = _vals(rng, (cout, c0 + c1, ks, ks), "bf16", 1.0 / math.sqrt(ks * ks * (c0 + c1)))
    b = rng.standard_normal(cout).astype(np.float32)
    wp, bd = _dev(_pack(w), "bf16"), _dev(b)

    def run(k, wd=W):
        return ops.conv(_dev(x0[:k, :, :wd], "bf16"), wp, cout, ks, stride, up,
                        x1=_dev(x1[:k, :, :wd], "bf16") if c1 else None, bias=bd).float().cpu().numpy()

    full = run(n)
    if n > 1:
        assert np.array_equal(full[:1], run(1))
    elif ks == 1:
        assert np.array_equal(full[:, :, :min(W, 100)], run(1, min(W, 100)))
    i = n - 1
    wd = W if ks == 3 else min(W, 500)  # (the last columns of a linear's row)
    a = x0[i].astype(np.float64) if not c1 else np.concatenate([x0[i], x1[i]], axis=2).astype(np.float64)
    a = a[:, W - wd:]
    ref = O.conv2d(O.upsample_nearest2x(a) if up else a, w, b, stride)
    err = rel_l2(full[i][:, full.shape[2] - ref.shape[1]:], ref)
    assert err <= TOL["bf16"], err


# rows, K, N: one partial K chunk, the edges of the 2 / 4 / 8-wave splits (K 64,
# 72, 248, 256), a chunk count that is no multiple of the waves, ragged 16x16
# tiles; two cases take 32x32 tiles (over 1024 tiles of 16x16); the rest 64x64 ones
# through LDS (256 of them and more) at the same edges of K, one with an odd
# width; at 16 columns the small tiles again.
F32_LINEAR_CASES = [(1, 8, 4), (17, 64, 16), (33, 72, 20), (40, 248, 36), (16, 256, 64), (5, 1032, 12),
                    (4113, 40, 68), (8200, 264, 40),
                    (16321, 8, 20), (16390, 64, 33), (16385, 72, 36), (8200, 248, 100), (4100, 256, 196),
                    (5470, 1032, 132), (16385, 264, 16)]


@pytest.mark.parametrize("case", F32_LINEAR_CASES)
def test_linear_f32(ops, case):
    """The fp32 GEMM against float64, and a row's bits whatever the row count."""
    M, K, N = case
    log(f"linear f32 {case}")
    rng = np.random.default_rng(M + K + N)
    x, w = _vals(rng, (1, 1, M, K), "f32"), _vals(rng, (N, K), "f32", 1.0 / math.sqrt(K))
    b, r = rng.standard_normal(N).astype(np.float32), _vals(rng, (1, 1, M, N), "f32")
    k = min(M, 19)

    def run(m):
        return ops.conv(_dev(x[:, :, :m]), _dev(w), N, ks=1, bias=_dev(b), resid=_dev(r[:, :, :m])).cpu().numpy()[0, 0]

    full = run(M)
    assert np.array_equal(full[:k], run(k))
    ref = x[0, 0].astype(np.float64) @ w.astype(np.float64).T + b + r[0, 0]
    assert rel_l2(full, ref) <= TOL["f32"]


# n, H, W, c0, c1, cout, stride, up, affine: 256 tiles of 64x64 and more for the
# batch, fewer for its first image (the small tiles).
F32_TILED_CASES = [(17, 31, 33, 16, 8, 40, 1, 0, False), (17, 31, 33, 24, 0, 40, 1, 0, True),
                   (18, 64, 60, 8, 0, 36, 2, 0, False), (9, 20, 24, 24, 0, 70, 1, 1, True)]


@pytest.mark.parametrize("case", F32_TILED_CASES)
def test_conv_f32_tiled(ops, case):
    """The fp32 GEMM's 64x64 tiles: every loader option gives the first image
    the bits it has alone and the last one the oracle's values."""
    n, H, W, c0, c1, cout, stride, up, aff = case
    rng = np.random.default_rng(hash(case) % 2**32)
    x0 = _vals(rng, (n, H, W, c0), "f32")
    x1 = _vals(rng, (n, H, W, c1), "f32") if c1 else None
    w = _vals(rng, (cout, c0 + c1, 3, 3), "f32", 1.0 / math.sqrt(9 * (c0 + c1)))
    b = rng.standard_normal(cout).astype(np.float32)
    sc, sh = (1 + 0.3 * rng.standard_normal((n, c0 + c1))).astype(np.float32), _vals(rng, (n, c0 + c1), "f32")
    wp, bd = _dev(_pack(w)), _dev(b)

    def run(k):
        return ops.conv(_dev(x0[:k]), wp, cout, 3, stride, up, x1=_dev(x1[:k]) if c1 else None,
                        scale=_dev(sc[:k]) if aff else None, shift=_dev(sh[:k]) if aff else None, silu=int(aff),
                        bias=bd).cpu().numpy()

    full = run(n)
    assert np.array_equal(full[:1], run(1))
    a = (x0[-1] if not c1 else np.concatenate([x0[-1], x1[-1]], axis=2)).astype(np.float64)
    if aff:
        a = O.silu(a * sc[-1] + sh[-1])
    ref = O.conv2d(O.upsample_nearest2x(a) if up else a, w, b, stride)
    assert rel_l2(full[-1], ref) <= TOL["f32"]


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("K", [8, 1020, 1024, 1284, 2816])
def test_linear_rows_few(ops, K, dt):
    """Up to 8 rows (staged whole, 2 / 4 / 8 at a time; 2816 columns of 8 rows
    exceed the stage) give the bits that the same rows have among 40."""
    rng = np.random.default_rng(K)
    N = 50
    x, w = rng.standard_normal((40, K)).astype(np.float32), _vals(rng, (N, K), dt, 1.0 / math.sqrt(K))
    b, add = rng.standard_normal(N).astype(np.float32), rng.standard_normal((40, N)).astype(np.float32)

    def run(m):
        return ops.linear_rows(_dev(x[:m]), _dev(w, dt), _dev(b), _dev(add[:m]), 1, 1).cpu().numpy()

    full = run(40)
    for m in (1, 2, 3, 4, 5, 8):
        assert np.array_equal(run(m), full[:m]), m


@pytest.mark.parametrize("P", [64, 128, 256])
def test_conv_out_cfg_ddim_splits(ops, P):
    """The 8-wave form at 64, 128 and 256 pixels a block gives the bits of the
    4-wave form (over 256 blocks of 256 pixels)."""
    H, W, C, n = 18, 32, 64, 128  # 576 pixels: 9, 5 and 3 blocks a request, the last ones ragged
    rng = np.random.default_rng(7)
    few = {64: 28, 128: 50, 256: 85}[P]
    x = _dev(_vals(rng, (2 * n, H, W, C), "bf16"), "bf16")
    w, b = _dev(_vals(rng, (4, 36 * C // 4), "bf16", 0.05), "bf16"), _dev(rng.standard_normal(4).astype(np.float32))
    ru = np.where(np.arange(n) % 3 == 1, -1, n + np.arange(n)).astype(np.int32)
    coef = _dev(rng.uniform(0.5, 2.0, (n, 3)).astype(np.float32))
    lat = _dev(rng.standard_normal((n, 4, H, W)).astype(np.float32))

    def run(k):
        out, eps = torch.empty_like(lat[:k]), torch.empty_like(lat[:k])
        ops.conv_out_cfg_ddim(x, w, b, _dev(ru[:k]), coef[:k], lat[:k], out, eps)
        return torch.stack((out, eps)).cpu()

    assert torch.equal(run(few), run(n)[:, :few])


OUT_CASES = [
    # n_req, cfg flags, H, W, C, in place, eps_out
    (3, (1, 0, 1), 12, 10, 64, False, True),     # one ragged tile (120 pixels)
    (5, (0, 1, 1, 0, 1), 16, 16, 320, False, True),
    (2, (1, 1), 64, 64, 320, True, True),       # 16 tiles, halo rows across tiles
    (2, (1, 0), 20, 20, 96, False, False),      # 3 MFMA steps, ragged last tile
    (1, (1,), 8, 128, 32, False, True),         # widest rows (LDS above 64 KB)
    (2, (0, 0), 1, 5, 32, False, True),         # one image row
    (4, (1, 0, 0, 1), 33, 7, 160, True, False),
]


@pytest.mark.parametrize("case", OUT_CASES)
def test_conv_out_cfg_ddim(ops, case):
    """The fused output kernel against the oracle's conv2d, CFG combine and
    DDIM update (x' = A x + B eps with the same A, B) per request."""
    from oracle.sampler import cfg_combine
    n_req, cfg, H, W, C, inplace, want_eps = case
    rng = np.random.default_rng(1000 + H * W + C)
    cfg = np.array(cfg, np.int32)
    n_rows = n_req + int(cfg.sum())
    ru = np.full(n_req, -1, np.int32)
    ru[cfg == 1] = n_req + np.arange(int(cfg.sum()))
    x = _vals(rng, (n_rows, H, W, C), "bf16")
    w = _vals(rng, (4, C, 3, 3), "bf16", 0.05)
    b = (rng.standard_normal(4) * 0.1).astype(np.float32)
    coef = np.stack([rng.uniform(0.9, 1.3, n_req), rng.uniform(-0.3, 0.0, n_req),
                     rng.uniform(5.0, 9.0, n_req)], 1).astype(np.float32)
    lat = rng.standard_normal((n_req, 4, H, W)).astype(np.float32)
    lat_in = _dev(lat)
    lat_out = lat_in if inplace else torch.empty_like(lat_in)
    eps_out = torch.empty_like(lat_in) if want_eps else None
    ops.conv_out_cfg_ddim(_dev(x, "bf16"), _dev(_pack(w), "bf16"), _dev(b), _dev(ru), _dev(coef), lat_in,
                          lat_out, eps_out)
    torch.cuda.synchronize()
    got = lat_out.cpu().double().numpy()
    got_e = eps_out.cpu().double().numpy() if want_eps else None
    for r in range(n_req):
        ec = O.conv2d(x[r].astype(np.float64), w, b)
        e = cfg_combine(ec, O.conv2d(x[ru[r]].astype(np.float64), w, b), float(coef[r, 2])) if ru[r] >= 0 else ec
        e = e.transpose(2, 0, 1)  # (4, H, W)
        ref = float(coef[r, 0]) * lat[r].astype(np.float64) + float(coef[r, 1]) * e
        err = rel_l2(got[r], ref)
        log(f"  out+cfg+ddim {case} request {r}: rel L2 latents {err:.2e}")
        assert err <= 1e-5, (r, err)
        if want_eps:
            assert rel_l2(got_e[r], e) <= 1e-5, r


def test_conv_out_cfg_ddim_rejects_unsupported(ops):
    from paper_2605_08835_amd.binding import SynerDiffError
    x = torch.zeros(2, 4, 4, 48, device="cuda", dtype=torch.bfloat16)   # C % 32 != 0
    w = torch.zeros(4, 9 * 48, device="cuda", dtype=torch.bfloat16)
    ru = torch.tensor([-1, -1], device="cuda", dtype=torch.int32)
    coef = torch.ones(2, 3, device="cuda")
    lat = torch.zeros(2, 4, 4, 4, device="cuda")
    with pytest.raises(SynerDiffError):
        ops.conv_out_cfg_ddim(x, w, torch.zeros(4, device="cuda"), ru, coef, lat)


GN_FUSED_CASES = [
    # n, H, W, c0, c1, groups, silu  (variant: vectors per thread x channels per load)
    (3, 8, 8, 1280, 0, 32, 1),      # 4 x 8
    (2, 16, 16, 1280, 0, 32, 1),    # 8 x 8
    (2, 16, 16, 2560, 0, 32, 1),    # 10 x 8
    (2, 16, 16, 1280, 640, 32, 1),  # 20 x 4 (a group straddles the two sources)
    (2, 16, 16, 64, 32, 8, 0),      # 4 x 4, 12 channels per group, no SiLU
    (3, 16, 16, 640, 0, 32, 1),     # 8 x 4
    (2, 8, 8, 2560, 0, 32, 0),      # 4 x 8
    (1, 3, 5, 320, 320, 32, 1),     # ragged image
]


@pytest.mark.parametrize("case", GN_FUSED_CASES)
def test_groupnorm_fused(ops, case):
    """The one-kernel GroupNorm + SiLU of the small levels against the
    oracle's group_norm (and silu), per image."""
    n, H, W, c0, c1, G, silu = case
    rng = np.random.default_rng(7 * c0 + c1 + H)
    x0 = bf16_round(_vals(rng, (n, H, W, c0), "bf16", 2.0) + np.float32(0.5))
    x1 = _vals(rng, (n, H, W, c1), "bf16") if c1 else None
    g = (1 + 0.1 * rng.standard_normal(c0 + c1)).astype(np.float32)
    b = (0.1 * rng.standard_normal(c0 + c1)).astype(np.float32)
    y = ops.groupnorm_fused(_dev(x0, "bf16"), G, 1e-5, _dev(g), _dev(b), x1=_dev(x1, "bf16") if c1 else None,
                            silu=bool(silu))
    torch.cuda.synchronize()
    y = y.float().cpu().numpy().astype(np.float64)
    for i in range(n):
        a = x0[i].astype(np.float64) if not c1 else np.concatenate([x0[i], x1[i]], axis=2).astype(np.float64)
        ref = O.group_norm(a, G, g, b, 1e-5)
        if silu:
            ref = O.silu(ref)
        err = rel_l2(y[i], ref)
        log(f"  groupnorm fused {case} image {i}: rel L2 {err:.2e}")
        assert err <= 6e-3, (i, err)  # one bf16 rounding of the output


def test_groupnorm_fused_rejects_large_images(ops):
    from paper_2605_08835_amd.binding import SynerDiffError
    x = torch.zeros(1, 64, 64, 320, device="cuda", dtype=torch.bfloat16)
    g = torch.ones(320, device="cuda")
    with pytest.raises(SynerDiffError):
        ops.groupnorm_fused(x, 32, 1e-5, g, g)
