"""Weight gradient of the 3x3 convolution where a tile reaches past the image: pixels that do not
exist contribute nothing, whatever the activations beside them hold."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2412_02413_amd import nn, pam
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pam._lib()
    return torch, nn


# x in {-1, 0, 1} and dy in {-1, 1}: every partial sum is an integer far below 2^24, exact in FP32 in any
# order, so finite gradients have to match exactly.
@pytest.mark.parametrize("B,h,w,c_in,c_out,bias", [
    (1, 1, 1, 32, 32, True),          # one pixel
    (2, 8, 32, 32, 32, True),         # exactly one tile an image: nothing outside
    (1, 9, 33, 64, 32, False),        # one row and one column over
    (3, 7, 31, 32, 64, True),         # one short both ways
    (2, 13, 48, 32, 32, True),        # half a tile of columns over
    (1, 16, 40, 32, 32, False),       # eight columns over: one operand fragment
    (2, 3, 64, 32, 32, True),         # rows missing only
    (8, 64, 32, 256, 256, True),      # the deepest layer
])
def test_non_finite_activations_stay_in_their_taps(env, B, h, w, c_in, c_out, bias):
    torch, nn = env
    rng = np.random.default_rng(h * w + c_in)
    x = rng.integers(-1, 2, (B, h, w, c_in)).astype(np.float32)
    dy = (2 * rng.integers(0, 2, (B, h, w, c_out)) - 1).astype(np.float32)
    x[0, h - 1, rng.integers(w), 0] = np.inf            # last row, channel 0
    x[B - 1, rng.integers(h), w - 1, 1] = np.nan        # last column, channel 1
    x[B - 1, h - 1, w - 1, 2] = -np.inf                 # the corner, channel 2
    xd, dyd = (torch.from_numpy(v).to(torch.bfloat16).cuda() for v in (x, dy))
    dw = torch.zeros((9, c_in, c_out), device="cuda")
    db = torch.zeros(c_out, device="cuda") if bias else None
    nn.conv3x3_wgrad(xd, c_in, dyd, c_out, B, h, w, c_in, c_out, dw, db)
    torch.cuda.synchronize()
    xp = np.pad(x.astype(np.float64), ((0, 0), (1, 1), (1, 1), (0, 0)))
    with np.errstate(invalid="ignore"):
        want = np.stack([xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(-1, c_in).T
                         @ dy.astype(np.float64).reshape(-1, c_out) for t in range(9)])
    # channels 0, 1 and 2 tap by tap from the definition (a matrix product may spread a NaN over its block)
    for c in range(3):
        for t in range(9):
            v = xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w, c].reshape(-1)
            if np.isfinite(v).all():
                want[t, c] = v @ dy.astype(np.float64).reshape(-1, c_out)
            else:
                want[t, c] = np.nan
    for c in range(3, c_in):
        assert np.isfinite(want[:, c]).all()
    got = dw.double().cpu().numpy()
    finite = np.isfinite(want)
    print(f"{finite[:, :3, 0].sum()} of 27 taps finite in the three channels, got "
          f"{np.isfinite(got[:, :3, 0]).sum()}", flush=True)
    assert np.array_equal(np.isfinite(got), finite)
    assert np.array_equal(got[finite], want[finite])
    if bias:
        assert np.array_equal(db.double().cpu().numpy(), dy.astype(np.float64).sum((0, 1, 2)))
