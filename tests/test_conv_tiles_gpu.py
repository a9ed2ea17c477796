"""The 3x3 convolution on either side of the line between whole and half tiles (512 half tiles)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# Operands in {-1, 0, 1}: partial sums are small integers, exact in FP32 in any order, so the result is the exact sum
# rounded once to BF16 (sums beyond 256 lose their last bits there) and has to match bit for bit.
@pytest.mark.parametrize("B,h,w,k_in,n_out", [
    (8, 64, 32, 96, 256),      # 512 half tiles of 4 rows x 64 channels, 256 whole
    (8, 65, 32, 96, 256),      # 544 half tiles: whole ones, a remainder of one row
    (2, 128, 512, 32, 32),     # 512 half tiles of 8 rows x 32 channels
    (2, 129, 512, 32, 32),     # 544
    (64, 4, 128, 32, 128),     # no more half tiles (512) than whole ones
    (4, 59, 224, 64, 128),     # 840 half tiles
])
def test_half_tiles_line(B, h, w, k_in, n_out):
    import torch
    from paper_2412_02413_amd import nn
    rng = np.random.default_rng(h * w + n_out)
    x = rng.integers(-1, 2, (B, h, w, k_in)).astype(np.float32)
    wt = rng.integers(-1, 2, (n_out, 9, k_in)).astype(np.float32)
    xd, wd = (torch.from_numpy(v).to(torch.bfloat16).cuda() for v in (x, wt))
    y = torch.full((B, h, w, n_out), -7.0, dtype=torch.bfloat16, device="cuda")
    nn.conv3x3(xd, k_in, B, h, w, k_in, wd, None, y, n_out, n_out, relu=False)
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    want = np.zeros((B, h, w, n_out), np.float32)
    for t in range(9):
        want += xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w] @ wt[:, t].T
    assert np.array_equal(y.float().cpu().numpy(), torch.from_numpy(want).to(torch.bfloat16).float().numpy())
