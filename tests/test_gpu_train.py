"""Training-side gradients on the GPU against the oracle, through the C ABI:
the backward of the sequential and channel-split FInC units (chain rule over
their blocks), actnorm's backward, and the per-image negative log-likelihood
and bits per dimension (Sec. 3 NLL equation, Sec. 5 BPD equation).

Bar: 1e-4 * max(1, |oracle|) elementwise (gpu_util.assert_close); a weight
gradient that sums many pixels is held to the root sum of squares of its
terms where that is larger (fp32 rounding scales with the terms, not with a
sum that cancels).  Every result is also bitwise the same on a second run.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2301_09266_amd import finc, synth

pytestmark = pytest.mark.gpu

from gpu_util import assert_close, dev, f64, host, poisoned  # noqa: E402


@pytest.fixture(scope="module")
def orc():
    return oracle.default()


def unit_kernels(C, k, seed):
    """Four blocks TL, TR, BL, BR with junk in their masked slots."""
    return np.stack([synth.garbage_in_mask(synth.masked_kernel(C, k, q, seed + q), q,
                                           seed=seed + 10 + q) for q in range(4)])


def term_scale_unit(orc, x, dy, K4):
    """Per weight-gradient entry of each block, the root sum of squares of
    the products it adds: the oracle's dK of the squared block input and
    squared incoming gradient (the block inputs and gradients themselves from
    the oracle's forward and per-block backward)."""
    hs = [x]
    for q in range(3):
        hs.append(orc.forward(hs[-1], K4[q], q))
    g, out = dy, [None] * 4
    for q in range(3, -1, -1):
        _, sq = orc.backward(hs[q] ** 2, g ** 2, K4[q], q, 0.0)
        out[q] = np.sqrt(sq)
        g, _ = orc.backward(hs[q], g, K4[q], q, 0.0)
    return np.stack(out)


UNIT_SHAPES = [(2, 3, 5, 7, 3), (3, 12, 16, 16, 3), (1, 5, 9, 6, 2), (2, 4, 6, 6, 1),
               (1, 7, 6, 5, 5), (2, 20, 8, 9, 3)]


@pytest.mark.parametrize("shape", UNIT_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_unit_backward(orc, shape):
    B, C, H, W, k = shape
    rng = np.random.default_rng(B * 1000 + C)
    x, dy = rng.normal(size=(B, C, H, W)), rng.normal(size=(B, C, H, W))
    K4 = unit_kernels(C, k, 300 + C)
    gld = -0.5
    dx, dK4 = finc.unit_backward(dev(x), dev(dy), dev(K4), gld, dx=poisoned(x.shape),
                                 dK4=poisoned(K4.shape))
    want_dx, want_dK4 = orc.unit_backward(f64(x), f64(dy), f64(K4), gld)
    assert_close(host(dx), want_dx, f"unit backward dx {shape}")
    assert_close(host(dK4), want_dK4, f"unit backward dK {shape}",
                 scale=term_scale_unit(orc, f64(x), f64(dy), f64(K4)))
    dx2, dK42 = finc.unit_backward(dev(x), dev(dy), dev(K4), gld)
    assert torch.equal(dx, dx2) and torch.equal(dK4, dK42)


# The tiles of dK and of the launch that holds both gradients: one part (written
# in place) and several, channel tiles of 1 / 15 / 16 / 17 / 33, every k (taps in
# groups of nine from k = 3), rows wider than a band with a remainder of one
# column, rows of one pixel, bands shorter than the image, and the input
# gradient's other kernel (48 channels at k = 5: its weights outgrow LDS).
GRAD_SHAPES = [(1, 1, 1, 1, 1), (1, 15, 3, 33, 3), (2, 16, 5, 65, 2), (3, 17, 33, 7, 4),
               (2, 33, 9, 8, 3), (5, 3, 40, 1, 5), (1, 4, 11, 31, 6), (2, 5, 7, 64, 7),
               (70, 2, 8, 8, 3), (2, 48, 6, 9, 5)]


@pytest.mark.parametrize("corner", [0, 2, 3])
@pytest.mark.parametrize("shape", GRAD_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_layer_gradient_tiles(orc, shape, corner):
    B, C, H, W, k = shape
    rng = np.random.default_rng(C * 10 + corner)
    x, dy = rng.normal(size=(B, C, H, W)), rng.normal(size=(B, C, H, W))
    K = synth.garbage_in_mask(synth.masked_kernel(C, k, corner, 40 + C), corner, seed=k)
    print("layer backward", shape, corner, flush=True)
    dx, dK = finc.backward(dev(x), dev(dy), dev(K), corner, -1.0, dx=poisoned(x.shape),
                           dK=poisoned(K.shape))
    want_dx, want_dK = orc.backward(f64(x), f64(dy), f64(K), corner, -1.0)
    assert_close(host(dx), want_dx, f"dx {shape}")
    _, sq = orc.backward(f64(x) ** 2, f64(dy) ** 2, f64(K), corner, 0.0)
    assert_close(host(dK), want_dK, f"dK {shape}", scale=np.sqrt(sq))
    assert torch.equal(finc.backward(dev(x), dev(dy), dev(K), corner, -1.0, want_dK=False)[0], dx)
    assert torch.equal(finc.backward(dev(x), dev(dy), dev(K), corner, -1.0, want_dx=False)[1], dK)


# Small images (several a band of dK; fewer rows or columns than the kernel; of
# a pixel), with a band that holds fewer than the others; blocks of the input
# gradient that take several images, of one (64 channels) and more a compute
# unit; rows cut into segments of columns, the last one narrower.
SMALL_SHAPES = [(1, 2, 2, 2, 3), (300, 3, 1, 1, 3), (70, 17, 2, 2, 3), (33, 5, 4, 4, 7),
                (23, 16, 8, 8, 2), (45, 2, 3, 7, 4), (100, 4, 1, 5, 5), (50, 3, 7, 1, 6),
                (1100, 3, 3, 3, 3), (300, 64, 3, 3, 3), (29, 33, 4, 3, 1), (2, 12, 3, 300, 3),
                (1, 20, 2, 133, 2), (3, 1, 1, 515, 5)]


@pytest.mark.parametrize("corner", [0, 1, 3])
@pytest.mark.parametrize("shape", SMALL_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_layer_gradient_small_images(orc, shape, corner):
    B, C, H, W, k = shape
    rng = np.random.default_rng(C * 10 + corner)
    x, dy = rng.normal(size=(B, C, H, W)), rng.normal(size=(B, C, H, W))
    K = synth.garbage_in_mask(synth.masked_kernel(C, k, corner, 40 + C), corner, seed=k)
    print("layer backward", shape, corner, flush=True)
    dx, dK = finc.backward(dev(x), dev(dy), dev(K), corner, -1.0, dx=poisoned(x.shape),
                           dK=poisoned(K.shape))
    want_dx, want_dK = orc.backward(f64(x), f64(dy), f64(K), corner, -1.0)
    assert_close(host(dx), want_dx, f"dx {shape}")
    _, sq = orc.backward(f64(x) ** 2, f64(dy) ** 2, f64(K), corner, 0.0)
    assert_close(host(dK), want_dK, f"dK {shape}", scale=np.sqrt(sq))
    assert torch.equal(finc.backward(dev(x), dev(dy), dev(K), corner, want_dK=False)[0], dx)
    assert torch.equal(finc.backward(dev(x), dev(dy), dev(K), corner, -1.0, want_dx=False)[1], dK)
    # an image's dx does not depend on the batch
    one = finc.backward(dev(x[-1:]), dev(dy[-1:]), dev(K), corner, want_dK=False)[0]
    assert torch.equal(one[0], dx[-1])


@pytest.mark.parametrize("corner", [0, 3])
@pytest.mark.parametrize("shape", [(2, 4, 5, 5, 3), (1, 4, 13, 17, 3), (3, 4, 1, 3, 3), (2, 4, 6, 7, 5)],
                         ids=lambda s: "x".join(map(str, s)))
def test_layer_gradient_infinities(orc, shape, corner):
    """One infinite input value, at the last position of a band whose positions
    are not a multiple of four: dK is infinite where a tap reads it and finite
    elsewhere.  One infinite value of dy, in a channel that no masked weight
    multiplies: the same for dx.  (Padding takes part in neither.)"""
    B, C, H, W, k = shape
    rng = np.random.default_rng(7)
    x, dy = rng.normal(size=(B, C, H, W)), rng.normal(size=(B, C, H, W))
    K = synth.masked_kernel(C, k, corner, 3)
    xi, dyi = x.copy(), dy.copy()
    xi[-1, 1, -1, -1], dyi[0, C - 1, H // 2, W // 2] = np.inf, -np.inf
    print("infinities", shape, corner, flush=True)
    dK = finc.backward(dev(xi), dev(dy), dev(K), corner, want_dx=False)[1]
    dx = finc.backward(dev(x), dev(dyi), dev(K), corner, want_dK=False)[0]
    for got, want, what in ((dK, orc.backward(f64(xi), f64(dy), f64(K), corner, 0.0)[1], "dK"),
                            (dx, orc.backward(f64(x), f64(dyi), f64(K), corner, 0.0)[0], "dx")):
        assert not np.isnan(want).any() and np.isinf(want).any()
        inf = np.isinf(want)
        assert np.array_equal(host(got)[inf], want[inf]), what
        assert_close(np.where(inf, 0.0, host(got)), np.where(inf, 0.0, want), f"{what} {shape}")


def test_unit_backward_workload(orc):
    """The unit workload's shape (256 images of 12 x 16 x 16, k = 3): dK4
    sums 65,536 pixels per tap; dx on three sampled images; dx alone and dK
    alone give the same bits."""
    c = synth.unit_case(256, 12, 16, 16, 3)
    x, K4 = c["x"], c["K4"]
    dy = np.random.default_rng(8).normal(size=x.shape)
    print("unit backward 256 x 12 x 16 x 16", flush=True)
    dx, dK4 = finc.unit_backward(dev(x), dev(dy), dev(K4), -1.0)
    want_dx, want_dK4 = orc.unit_backward(f64(x), f64(dy), f64(K4), -1.0)
    assert_close(host(dK4), want_dK4, "unit backward dK, 256 images",
                 scale=term_scale_unit(orc, f64(x), f64(dy), f64(K4)))
    pick = [0, 100, 255]
    assert_close(host(dx)[pick], want_dx[pick], "unit backward dx, 256 images")
    only_dk = finc.unit_backward(dev(x), dev(dy), dev(K4), -1.0, want_dx=False)
    assert only_dk[0] is None and torch.equal(only_dk[1], dK4)
    only_dx = finc.unit_backward(dev(x), dev(dy), dev(K4), -1.0, want_dK=False)
    assert only_dx[1] is None and torch.equal(only_dx[0], dx)


SPLIT_SHAPES = [(2, 8, 5, 7, 3), (3, 48, 8, 8, 3), (1, 4, 9, 6, 5), (2, 16, 16, 16, 2),
                (2, 12, 7, 4, 7), (1, 64, 6, 6, 3)]


@pytest.mark.parametrize("shape", SPLIT_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_split_backward(orc, shape):
    B, C, H, W, k = shape
    q = C // 4
    rng = np.random.default_rng(B * 100 + C + k)
    x, dy = rng.normal(size=(B, C, H, W)), rng.normal(size=(B, C, H, W))
    Kq4 = np.stack([synth.garbage_in_mask(synth.masked_kernel(q, k, g, 500 + g), g, seed=g + 3)
                    for g in range(4)])
    gld = 0.8
    dx, dKq4 = finc.split_backward(dev(x), dev(dy), dev(Kq4), gld, dx=poisoned(x.shape),
                                   dKq4=poisoned(Kq4.shape))
    want_dx, want_dKq4 = orc.split_backward(f64(x), f64(dy), f64(Kq4), gld)
    assert_close(host(dx), want_dx, f"split backward dx {shape}")
    _, sq = orc.split_backward(f64(x) ** 2, f64(dy) ** 2, f64(Kq4), 0.0)
    assert_close(host(dKq4), want_dKq4, f"split backward dK {shape}", scale=np.sqrt(sq))
    dx2, dKq42 = finc.split_backward(dev(x), dev(dy), dev(Kq4), gld)
    assert torch.equal(dx, dx2) and torch.equal(dKq4, dKq42)


def test_unit_backward_empty_batch(orc):
    """No images: dx empty, each block's dK only its log|det| term."""
    C, H, W, k = 5, 6, 7, 3
    K4 = unit_kernels(C, k, 90)
    x = np.zeros((0, C, H, W))
    _, dK4 = finc.unit_backward(dev(x), dev(x), dev(K4), -1.0, dK4=poisoned(K4.shape))
    assert_close(host(dK4), orc.unit_backward(f64(x), f64(x), f64(K4), -1.0)[1],
                 "unit backward dK, no images")
    Kq4 = np.stack([synth.masked_kernel(2, k, g, 60 + g) for g in range(4)])
    x8 = np.zeros((0, 8, H, W))
    _, dKq4 = finc.split_backward(dev(x8), dev(x8), dev(Kq4), -1.0, dKq4=poisoned(Kq4.shape))
    assert_close(host(dKq4), orc.split_backward(f64(x8), f64(x8), f64(Kq4), -1.0)[1],
                 "split backward dK, no images")


@pytest.mark.parametrize("shape", [(3, 5, 4, 6), (64, 12, 16, 16), (1, 96, 3, 5), (0, 4, 4, 4),
                                   (300, 3, 8, 8)],
                         ids=lambda s: "x".join(map(str, s)))
def test_actnorm_backward(orc, shape):
    B, C, H, W = shape
    rng = np.random.default_rng(C + H)
    x, dy = rng.normal(size=shape), rng.normal(size=shape)
    s = rng.uniform(0.5, 1.5, size=C) * rng.choice([-1.0, 1.0], size=C)
    gld = -0.25
    dx, ds, db = finc.actnorm_backward(dev(x), dev(dy), dev(s), gld)
    want = orc.actnorm_backward(f64(x), f64(dy), f64(s), gld)
    assert_close(host(dx), want[0], f"actnorm dx {shape}")
    assert_close(host(ds), want[1], f"actnorm ds {shape}")
    assert_close(host(db), want[2], f"actnorm db {shape}")
    again = finc.actnorm_backward(dev(x), dev(dy), dev(s), gld)
    assert all(torch.equal(a, b) for a, b in zip((dx, ds, db), again))


@pytest.mark.parametrize("shape", [(1, 2, 1, 4), (5, 3, 3, 5), (3, 7, 9, 12), (9, 2, 64, 68),
                                   (2, 1, 33, 131)], ids=lambda s: "x".join(map(str, s)))
def test_actnorm_backward_wide_loads(orc, shape):
    """Planes of a multiple of four values (16-byte loads) and others, fewer
    values than threads, a remainder of the loads in flight; and the same from
    buffers that are not 16-byte aligned."""
    B, C, H, W = shape
    rng = np.random.default_rng(H)
    x, dy = rng.normal(size=shape), rng.normal(size=shape)
    s = rng.uniform(0.5, 1.5, size=C)
    got = finc.actnorm_backward(dev(x), dev(dy), dev(s), -0.25)
    want = orc.actnorm_backward(f64(x), f64(dy), f64(s), -0.25)
    for g, w, what in zip(got, want, ("dx", "ds", "db")):
        assert_close(host(g), w, f"actnorm {what} {shape}")

    def shifted(t):
        return torch.cat([t.new_zeros(1), t.reshape(-1)])[1:].view(t.shape)
    off = finc.actnorm_backward(shifted(dev(x)), shifted(dev(dy)), dev(s), -0.25)
    for g, w, what in zip(off, want, ("dx", "ds", "db")):
        assert_close(host(g), w, f"actnorm {what} {shape}, unaligned")


@pytest.mark.parametrize("B", [1, 3, 100])
def test_gauss_nll(orc, B):
    """Three latents of the CIFAR-10 flow's shapes ([28, 28, 28] with L = 3
    on 3 x 32 x 32 images: 6 x 16 x 16, 12 x 8 x 8, 48 x 4 x 4); fp64 sums
    of the fp32 latents on both sides, so the bar is 1e-12 relative."""
    rng = np.random.default_rng(B)
    zs = [rng.normal(size=(B, 6, 16, 16)), rng.normal(size=(B, 12, 8, 8)),
          rng.normal(size=(B, 48, 4, 4)) * 1.5]
    logdet = rng.normal(size=B) * 100.0
    nll, bpd = finc.gauss_nll([dev(z) for z in zs],
                              torch.tensor(logdet, dtype=torch.float64, device="cuda:0"))
    want_nll, want_bpd = orc.gauss_nll([f64(z) for z in zs], logdet)
    g_nll, g_bpd = nll.cpu().numpy(), bpd.cpu().numpy()
    assert np.max(np.abs(g_nll - want_nll) / np.abs(want_nll)) < 1e-12
    assert np.max(np.abs(g_bpd - want_bpd) / np.abs(want_bpd)) < 1e-12


def _stack_flat(c):
    return (np.concatenate([np.ravel(a) for a in c["K"]]),
            np.concatenate([np.ravel(a) for a in c["scale"]]),
            np.concatenate([np.ravel(a) for a in c["bias"]]))


STACK_CASES = [
    # (B, C1, H1, W1, levels, units, k)
    (2, 4, 16, 16, 2, 2, 3), (3, 2, 8, 12, 3, 1, 2), (1, 6, 8, 8, 1, 3, 3),
    (4, 12, 32, 32, 3, 8, 3),   # the sampling stack's shape (4 images)
]


@pytest.mark.parametrize("case", STACK_CASES, ids=lambda c: "x".join(map(str, c)))
def test_stack_training_step(orc, case):
    """One training step of the multi-scale stack: the forward's latents and
    log|det| against the oracle; the batch's NLL; and the gradients of the
    summed NLL (latent gradients z, gld = -B) of the input, the blocks'
    weights, the actnorms' scales and biases against the oracle's backward of
    the same latents.  Weight, scale and bias gradients sum over the batch
    and, through the chain, over many paths: each is held to 1e-4 of
    max(1, |oracle|, the largest |oracle| of its parameter block), the scale
    of the rounding of sums that cancel (the terms' own sizes are not
    available through the chain).  The 24-unit stack with random weights
    grows its latents to |z| ~ 1e5 (level 1) and 1e9 (level 2), and fp32
    rounding there is set by those magnitudes: as for its inverse, every
    tensor is held to max |gpu - oracle| <= 1e-4 max(1, max |oracle|)."""
    B, C1, H1, W1, L, U, k = case
    print(f"stack training step {case}", flush=True)
    c = synth.stack_case(B=B, C1=C1, H1=H1, W1=W1, levels=L, units=U, k=k)
    x = c["x"][:, :C1, :H1, :W1]
    # the parameters as the GPU sees them (fp32), for both sides
    c = dict(c, K=[f64(a) for a in c["K"]], scale=[f64(a) for a in c["scale"]],
             bias=[f64(a) for a in c["bias"]])
    Kf, sf, bf = _stack_flat(c)
    deep = L * U >= 8

    def check(g, r, what, scale=None):
        if deep:
            err = float(np.max(np.abs(g - r)))
            assert err <= 1e-4 * max(1.0, float(np.max(np.abs(r)))), (what, err)
        else:
            assert_close(g, r, what, scale=scale)

    z, ld = finc.stack_forward(dev(x), dev(Kf), dev(sf), dev(bf), L, U, k)
    want_z = orc.stack_forward(f64(x), c["K"], c["scale"], c["bias"], levels=L, units=U, k=k)
    for l in range(L):
        check(host(z[l]), want_z[l], f"stack forward latent {l} {case}")
    want_ld = orc.stack_logdet(c["K"], c["scale"], levels=L, units=U, C1=C1, H1=H1, W1=W1, k=k)
    assert np.allclose(ld.cpu().numpy(), want_ld, rtol=1e-9, atol=1e-9), (ld, want_ld)
    nll, bpd = finc.gauss_nll(z, ld)
    want_nll, _ = orc.gauss_nll([host(t) for t in z], np.full(B, want_ld))
    assert np.max(np.abs(nll.cpu().numpy() - want_nll) / np.abs(want_nll)) < 1e-9
    dx, dK, ds, db = finc.stack_backward(dev(x), z, dev(Kf), dev(sf), dev(bf), L, U, k,
                                         gld=-float(B))
    wx, wK, ws_, wb = orc.stack_backward(f64(x), [host(t) for t in z], c["K"], c["scale"],
                                         c["bias"], levels=L, units=U, k=k, gld=-float(B))
    check(host(dx), wx, f"stack backward dx {case}")
    # per parameter block (a unit's weights, an actnorm's scale or bias): the
    # block's largest magnitude sets the scale of its sums' rounding
    blocks = []
    o = 0
    for l in range(L):
        n = 4 * (C1 << l) ** 2 * k * k
        for u in range(U):
            blocks.append((o, o + n))
            o += n
    scale_K = np.concatenate([np.full(e - b0, np.abs(wK[b0:e]).max()) for b0, e in blocks])
    check(host(dK), wK, f"stack backward dK {case}", scale=scale_K)
    check(host(ds), ws_, f"stack backward dscale {case}", scale=np.abs(ws_).max())
    check(host(db), wb, f"stack backward dbias {case}", scale=np.abs(wb).max())
    again = finc.stack_backward(dev(x), z, dev(Kf), dev(sf), dev(bf), L, U, k, gld=-float(B))
    assert all(torch.equal(a, b) for a, b in zip((dx, dK, ds, db), again))
