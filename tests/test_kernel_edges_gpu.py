"""Kernels at the edges of their tiles and dispatch ranges, against the FP64 reference of each."""
import numpy as np
import pytest

from oracle import as_tax as O
from oracle import fd_tea as T
from paper_2412_02413_amd import synth


pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2412_02413_amd import nn, pam
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pam._lib()
    return torch, nn


def bf16(torch, a):
    """The array rounded to BF16, as FP64 and as a device tensor."""
    t = torch.tensor(a, dtype=torch.float32).to(torch.bfloat16)
    return t.double().numpy(), t.cuda()


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# The products of BF16 values are exact in FP32 and n of them are summed in FP32 in some order: each
# addition rounds by at most 2^-24 of the partial sum, so by about 2^-24 sqrt(n) of the result's own
# size in a random walk; 1e-6 holds up to n = 250 times over that.
@pytest.mark.parametrize("B,h,w,c_in,c_out,bias", [
    (1, 1, 1, 32, 32, True),         # one pixel: every other pixel of the tile is outside
    (2, 8, 32, 32, 32, True),        # exactly one tile per image
    (1, 9, 33, 64, 32, False),       # a remainder of one row and one column, no bias gradient
    (3, 7, 31, 32, 64, True),        # one short of a tile in both directions
    (8, 64, 32, 256, 256, True),     # the deepest layer: 64 channel pairs, four runs of tiles
])
def test_conv3x3_wgrad_tile_edges(env, B, h, w, c_in, c_out, bias):
    torch, nn = env
    rng = np.random.default_rng(h * w + c_in)
    x, xd = bf16(torch, rng.standard_normal((B, h, w, c_in)))
    dy, dyd = bf16(torch, rng.standard_normal((B, h, w, c_out)))
    dw0 = rng.standard_normal((9, c_in, c_out)).astype(np.float32)
    dw = torch.tensor(dw0, device="cuda")                 # the gradients add to what is there
    db = torch.zeros(c_out, device="cuda") if bias else None
    nn.conv3x3_wgrad(xd, c_in, dyd, c_out, B, h, w, c_in, c_out, dw, db)
    torch.cuda.synchronize()
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    want = np.stack([xp[:, t // 3: t // 3 + h, t % 3: t % 3 + w].reshape(-1, c_in).T @ dy.reshape(-1, c_out)
                     for t in range(9)]) + dw0
    e = rel(dw.cpu().numpy().astype(np.float64), want)
    print(f"dW rel L2 {e:.2e}", flush=True)
    assert e < 1e-6
    if bias:
        assert rel(db.cpu().numpy().astype(np.float64), dy.sum((0, 1, 2))) < 1e-6


@pytest.mark.parametrize("pixels,c,pad", [(1, 8, 0), (257, 32, 64), (33, 24, 8), (100, 12, 4), (64, 8, 4)])
def test_relu_backward_forms(env, pixels, c, pad):
    """Eight channels per thread where c and both strides are multiples of 8, else one: the values
    kept and those cleared are exact, and nothing outside the c channels changes."""
    torch, nn = env
    rng = np.random.default_rng(pixels + c)
    y, yd = bf16(torch, rng.standard_normal((pixels, c + pad)))
    y[0, 0], yd[0, 0] = 0.0, 0.0
    dy, dyd = bf16(torch, rng.standard_normal((pixels, c + pad)))
    nn.relu_backward(yd, c + pad, dyd, c + pad, pixels, c)
    want = dy.copy()
    want[:, :c] *= y[:, :c] > 0
    np.testing.assert_array_equal(dyd.double().cpu().numpy(), want)


@pytest.mark.parametrize("pixels,c", [(1, 8), (1000, 24), (262145, 32), (70, 120), (300, 12)])
def test_head_forms(env, pixels, c):
    """The head's loss and gradients at the edges of its pixel loops (one pixel; one past 256
    workgroups of 1024) and of its channel groups (1, 3, 4, 15 of 8; 12 channels take the other
    form).  Sums of n terms in FP32 in some order: 2^-24 sqrt(n) of the largest partial sum, so 1e-4
    of the loss and of a gradient's norm covers cancellation; the BF16 output rounds by 2^-9."""
    torch, nn = env
    rng = np.random.default_rng(c + pixels)
    f, fd = bf16(torch, rng.standard_normal((pixels, c)))
    w = (rng.standard_normal((c, 2)) / np.sqrt(c)).astype(np.float32)
    b = np.float32([0.1, -0.2])
    t = rng.uniform(0, 1, pixels).astype(np.float32)
    wt = (rng.uniform(0.5, 1.5, pixels) / pixels).astype(np.float32)
    dev = [torch.tensor(a, device="cuda") for a in (w, b, t, wt)]
    mask, err = torch.empty(pixels, device="cuda"), torch.empty(pixels, device="cuda")
    dz, loss = torch.empty((pixels, 2), device="cuda"), torch.zeros(3, device="cuda")
    nn.head(fd, c, pixels, dev[0], dev[1], dev[2], dev[3], mask, err, dz, loss, pixels)
    df = torch.empty((pixels, c), dtype=torch.bfloat16, device="cuda")
    dw, db = torch.zeros((c, 2), device="cuda"), torch.zeros(2, device="cuda")
    nn.head_backward(fd, c, pixels, dev[0], dz, df, dw, db)
    plain = torch.empty(pixels, device="cuda")
    nn.head(fd, c, pixels, dev[0], dev[1], None, None, plain, err, None, None, pixels)
    assert torch.equal(plain, mask)
    z = f @ w.astype(np.float64) + b
    m, e = 1 / (1 + np.exp(-z.T))
    ae = np.abs(m - t)
    lz = np.logaddexp(0, z)
    want = [np.sum(wt * (t * (lz[:, 0] - z[:, 0]) + (1 - t) * lz[:, 0])),
            np.sum(wt * (ae * (lz[:, 1] - z[:, 1]) + (1 - ae) * lz[:, 1])), np.sum(wt * ae)]
    np.testing.assert_allclose(loss.cpu().numpy(), want, rtol=1e-4)
    g = np.stack([(m - t) * wt, (e - ae) * wt], 1)
    assert rel(dz.double().cpu().numpy(), g) < 1e-5
    assert rel(dw.double().cpu().numpy(), f.T @ g) < 1e-4
    assert rel(db.double().cpu().numpy(), g.sum(0)) < 1e-4
    assert rel(df.double().cpu().numpy(), g @ w.astype(np.float64).T) < 2 ** -8


# FP32 outputs of FP64 arithmetic on the same FP32 partial sums: one rounding (2^-24) besides the
# 1e-12 of the Newton forms.
@pytest.mark.parametrize("n_sub,eps,frames", [(3, 1e-3, 1), (3, 1e-20, 1), (3, 1e-3, 24), (2, 1e-3, 1), (1, 1e-3, 2)])
def test_weight_and_energy_from_partial_sums(env, n_sub, eps, frames):
    """NCC, weight and energy against their definition on the call's own partial sums: one frame
    (many bin splits) and 24 (few), a clamp so low that the cube root leaves the FP32 range."""
    torch, _ = env
    from paper_2412_02413_amd import pam
    g = synth.cfg1_geometry().replace(n_sub=n_sub, eps=eps)
    rf = synth.batch(synth.cfg1_frame, list(range(40, 40 + frames)))
    plan = pam.pam_plan(g, 0, "fp32")
    try:
        out = pam.reconstruct(plan, torch.from_numpy(rf).cuda())
        torch.cuda.synchronize()
        lay = pam.pam_workspace_layout(plan, frames, g.n_samples)
    finally:
        pam.pam_destroy(plan)
    pix = g.n_z * g.n_x

    def view(offset, n):
        return out["workspace"][offset: offset + 4 * n].cpu().numpy().view(np.float32).astype(np.float64)

    acc = view(lay.accum, lay.n_split * frames * lay.n_acc * pix).reshape(lay.n_split, frames, lay.n_acc, pix).sum(0)
    S, C = acc[:, :n_sub], acc[:, n_sub:]
    E, w = S.sum(1) + 2 * C.sum(1), np.ones((frames, pix))
    for q, (i, j) in enumerate({1: [], 2: [(0, 1)], 3: [(0, 1), (1, 2), (2, 0)]}[n_sub]):
        den = np.sqrt(S[:, i]) * np.sqrt(S[:, j])
        w *= np.clip(np.where(den > 0, C[:, q] / np.where(den > 0, den, 1), 0), eps, 1)
    w = np.cbrt(w) if n_sub == 3 else w
    print(f"{lay.n_split} splits, smallest weight {w.min():.1e}", flush=True)
    np.testing.assert_allclose(view(lay.weight, frames * pix).reshape(frames, pix), w, rtol=2.0 ** -23)
    np.testing.assert_allclose(view(lay.energy, frames * pix).reshape(frames, pix), E, rtol=2.0 ** -23)


MM = 1e-3


def lateral_case(n_x, n_sub, n_depths, **kw):
    """A small array on n_x columns: 52 bins, 5 of them with evanescent wavenumbers in range."""
    L = min(32, n_x)
    g = synth.Geometry(n_elements=L, pitch_m=0.3 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=256,
                       bands_hz=[(2e6, 6e6)], depths_m=(15 + 0.4 * np.arange(n_depths)) * MM, n_x=n_x, n_sub=n_sub,
                       pattern_m=4).replace(**kw)
    rng = np.random.default_rng(n_x + n_sub)
    em = [synth.Emitter(-1.0 * MM, 19 * MM, "broadband"), synth.Emitter(2.0 * MM, 24 * MM, "broadband")]
    return g, synth.render(g, em, rng, snr_db=20.0)


# The tolerances of the FP32 path everywhere: image 1e-5 relative, NNCC 1e-4 absolute.
@pytest.mark.parametrize("n_x", list(range(32, 513, 32)))
@pytest.mark.parametrize("n_sub", [1, 2, 3])
def test_every_lateral_size(env, n_x, n_sub):
    """The vector FFT kernels (lateral and fields) at every size, against the oracle: a depth count
    that leaves a ragged last tile, padded columns; zero-stuffed ones where 32 divides n_x."""
    torch, _ = env
    from paper_2412_02413_amd import pam
    for kw in ({}, {"lateral": "stuff", "evanescent": "zero"}):
        g, rf = lateral_case(n_x, n_sub, 19, **kw)
        plan = pam.pam_plan(g, 0, "fp32")
        try:
            out = pam.reconstruct(plan, torch.from_numpy(rf[None]).cuda())
            torch.cuda.synchronize()
        finally:
            pam.pam_destroy(plan)
        ref = O.as_tax(rf, g)
        e_i = rel(out["image"][0].double().cpu().numpy(), ref["I"])
        e_r = float(np.abs(out["nncc"][0].double().cpu().numpy() - ref["rho_n"]).max())
        print(f"{n_x} {n_sub} {kw}: image {e_i:.1e} nncc {e_r:.1e}", flush=True)
        assert e_i <= 1e-5 and e_r <= 1e-4


@pytest.mark.parametrize("n_x", [96, 192, 384])
def test_smaller_reservation_of_partial_sums(env, n_x):
    """A call whose workspace lacks the full reservation of partial-sum planes splits its bins fewer
    ways: the same results up to the order of FP32 sums; one byte less than that still fails."""
    torch, _ = env
    from paper_2412_02413_amd import pam
    g, rf = lateral_case(n_x, 3, 64)
    plan = pam.pam_plan(g, 0, "fp32")
    try:
        x = torch.from_numpy(rf[None]).cuda()
        want = pam.reconstruct(plan, x)["image"].clone()
        img = torch.empty_like(want)
        lay = pam.pam_workspace_layout(plan, 1, g.n_samples)
        plane = 4 * 6 * g.n_z * g.n_x
        fits, lo, hi = lay.total, lay.total - (lay.energy - lay.accum) + plane, lay.total
        while hi - lo > 256:                                  # smallest accepted size, to 256 bytes
            mid = (lo + hi) // 512 * 256
            ws = torch.empty(mid, dtype=torch.uint8, device="cuda")
            try:
                pam.pam_as_tax(plan, x, img, None, None, ws)
                assert rel(img.double().cpu().numpy(), want.double().cpu().numpy()) < 1e-6, mid
                fits = hi = mid
            except pam.PamError as e:
                assert e.status == pam.PAM_ERR_WORKSPACE
                lo = mid
        print(f"{n_x}: {lay.total} bytes reserved, {fits} accepted", flush=True)
        assert fits < lay.total
    finally:
        pam.pam_destroy(plan)


@pytest.mark.parametrize("L,n_x,n_sub,kw", [
    (1, 32, 1, {}),                                        # one element, eight rows of pixels per wave
    (13, 32, 3, {"pattern_m": 3}),                         # units of eight that mix sub-apertures, a ragged last one
    (48, 96, 3, {"lateral": "stuff"}),                     # rows of 48 pixels, 12 lanes each
    (32, 128, 2, {"lateral": "stuff", "pattern_m": 8}),    # four residues a column step
    (9, 288, 3, {"lateral": "stuff", "pattern_m": 1}),     # 32 residues of nine pixels: ragged lanes
    (160, 480, 3, {"pattern_m": 8}),                       # more than 64 lanes a row: two waves per depth
    (512, 512, 3, {"pattern_m": 16}),                      # the largest phasor table
    (40, 64, 3, {"overlap": True}),                        # elements in several sub-apertures and in none
])
def test_fd_tea_shapes(env, L, n_x, n_sub, kw):
    """FD-TEA-TAX at the edges of its split of pixels into lanes and of elements into units of eight."""
    torch, _ = env
    from paper_2412_02413_amd import pam
    overlap = "overlap" in kw
    apod = None
    if overlap:
        l = np.arange(L)
        apod = np.stack([l % 3 != 0, l < 24, (l >= 8) & (l < 16)]).astype(np.uint8)
    g = synth.Geometry(n_elements=L, pitch_m=0.1 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=64, bands_hz=[(2e6, 6e6)],
                       depths_m=(12 + 0.7 * np.arange(11)) * MM, n_x=n_x, n_sub=n_sub, apod=apod)
    g = g.replace(**{k: v for k, v in kw.items() if k != "overlap"})
    rng = np.random.default_rng(L + n_x)
    rf = synth.render(g, [synth.Emitter(0.5 * MM, 15 * MM, "broadband")], rng, snr_db=20.0)
    plan = pam.pam_plan(g, 0, "fp32")
    try:
        x = torch.from_numpy(np.stack([rf, rf])).cuda()
        img = torch.full((2, plan.n_z, plan.n_x), -1.0, device="cuda")
        nncc = torch.full_like(img, -1.0)
        pam.pam_fd_tea_tax(plan, x, img, nncc, None, pam.alloc_workspace(plan, 2, g.n_samples))
        torch.cuda.synchronize()
    finally:
        pam.pam_destroy(plan)
    ref = T.fd_tea_tax(rf, g)
    for f in range(2):
        assert rel(img[f].double().cpu().numpy(), ref["I"]) <= 1e-5
        assert np.abs(nncc[f].double().cpu().numpy() - ref["rho_n"]).max() <= 1e-4


# Operands in {-1, 0, 1}: every partial sum is a small integer, exact in FP32 in any order, so the result is the
# exact sum rounded once to BF16 and has to match bit for bit.
@pytest.mark.parametrize("B,h,w,k_in,n_out,acc", [
    (2, 131, 512, 32, 64, False),    # 544 workgroups of 8 rows x 64 channels: full tiles, several per workgroup
    (2, 245, 512, 32, 32, True),     # 512 of 16 rows x 32 channels, ragged rows
    (2, 37, 256, 64, 128, False),    # 160: tiles of 4 rows x 64 channels
    (1, 253, 128, 32, 64, True),     # 128, the first of that form, one row short of a tile
    (2, 53, 128, 64, 160, False),    # 160: tiles of 8 rows x 32 channels
    (1, 248, 128, 32, 64, False),    # 124, the last of the smallest form
    (1, 124, 256, 64, 32, True),     # 64: tiles of 4 rows x 32 channels
    (1, 3, 32, 64, 64, False),       # one tile, fewer rows than it has
])
def test_conv3x3_tile_forms(env, B, h, w, k_in, n_out, acc):
    """The 3x3 convolution at each tile form its dispatch chooses by the number of tiles."""
    torch, nn = env
    rng = np.random.default_rng(h * w + n_out)
    x, xd = bf16(torch, rng.integers(-1, 2, (B, h, w, k_in)))
    wt, wd = bf16(torch, rng.integers(-1, 2, (n_out, 9, k_in)))
    y0, y = bf16(torch, rng.integers(-8, 9, (B, h, w, n_out)))
    b = rng.integers(-8, 9, n_out).astype(np.float32)
    bd = None if acc else torch.from_numpy(b).cuda()
    nn.conv3x3(xd, k_in, B, h, w, k_in, wd, bd, y, n_out, n_out, relu=not acc, accumulate=acc)
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    want = np.zeros((B, h, w, n_out))
    for t in range(9):
        want += xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w] @ wt[:, t].T
    want = want + y0 if acc else np.maximum(want + b, 0.0)
    assert np.array_equal(y.double().cpu().numpy(), bf16(torch, want)[0])


# The kernel sums FP64 products of the FP32 inputs, so what is left is the one rounding of the result to FP32
# (2^-24) and the FP64 sums' own rounding.
@pytest.mark.parametrize("pixels", [1, 1025, 7 * 1024 + 1, 8 * 1024 - 1, 8 * 1024, 8 * 1024 + 3, 17 * 1024 + 5])
def test_error_estimate_lengths(env, pixels):
    """The predicted image error around the lengths where its batched loads begin and end."""
    torch, nn = env
    rng = np.random.default_rng(pixels)
    m, r, e = (rng.random((2, pixels)).astype(np.float32) for _ in range(3))
    est = torch.empty(2, device="cuda")
    nn.error_estimate(*(torch.from_numpy(v).cuda() for v in (m, r, e)), 2, pixels, est)
    m, r, e = (v.astype(np.float64) for v in (m, r, e))
    want = np.linalg.norm(2 * m * r * e, axis=1) / np.linalg.norm(m * m * e, axis=1)
    np.testing.assert_allclose(est.double().cpu().numpy(), want, rtol=2.0 ** -23)
