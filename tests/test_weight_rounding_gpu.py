"""The weight step's FP64 arithmetic, seen through its FP32 outputs."""
import numpy as np
import pytest

from paper_2412_02413_amd import synth

pytestmark = pytest.mark.gpu
MM = 1e-3


# The partial sums are FP32 values of one bin split, so they enter FP64 exactly.  In FP64 with every operation
# rounded correctly an NCC carries at most 4 roundings (two roots or one product, a division), the product of three
# NCCs 2 more and the cube root divides these 14 by 3 and adds one: below 6 x 2^-53.  The FP32 weight therefore is
# the rounding of some value within 2^-50 of the true one.
@pytest.mark.parametrize("eps", [1e-3, 1e-12])
def test_weight_is_the_rounded_value(eps):
    """Every weight equals the FP32 rounding of its 80-bit value, but for those that lie within 2^-50 of a
    rounding boundary."""
    import torch
    from paper_2412_02413_amd import pam
    F = 6
    g = synth.Geometry(n_elements=48, pitch_m=0.3 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=64, bands_hz=[(2e6, 3e6)],
                       depths_m=(12 + 0.1 * np.arange(512)) * MM, n_x=256, n_sub=3, pattern_m=4, eps=eps)
    rng = np.random.default_rng(11)
    rf = torch.from_numpy(rng.standard_normal((F, 48, 64)).astype(np.float32)).cuda()
    plan = pam.pam_plan(g, 0, "fp32")
    try:
        out = pam.reconstruct(plan, rf, want_pairs=True)
        torch.cuda.synchronize()
        lay = pam.pam_workspace_layout(plan, F, g.n_samples)
    finally:
        pam.pam_destroy(plan)
    assert lay.n_split == 1
    pix = g.n_z * g.n_x

    def view(offset, n):
        return out["workspace"][offset: offset + 4 * n].cpu().numpy().view(np.float32)

    acc = view(lay.accum, F * 6 * pix).reshape(F, 6, pix).astype(np.longdouble)
    S, C = acc[:, :3], acc[:, 3:]
    r = [C[:, q] / np.sqrt(S[:, i] * S[:, j]) for q, (i, j) in enumerate([(0, 1), (1, 2), (2, 0)])]
    w = np.ones((F, pix), np.longdouble)
    for v in r:
        w *= np.clip(v, np.longdouble(eps), 1)
    w = np.cbrt(w)
    got = view(lay.weight, F * pix).reshape(F, pix)
    d = np.longdouble(2.0) ** -50
    off = (got < (w * (1 - d)).astype(np.float32)) | (got > (w * (1 + d)).astype(np.float32))
    pairs = out["rho_pairs"].cpu().numpy().reshape(F, 3, pix)
    off_r = 0
    for q in range(3):
        lo, hi = (r[q] * (1 - d)).astype(np.float32), (r[q] * (1 + d)).astype(np.float32)
        off_r += int(((pairs[:, q] < np.minimum(lo, hi)) | (pairs[:, q] > np.maximum(lo, hi))).sum())
    print(f"eps {eps}: smallest weight {float(w.min()):.1e}; {int(off.sum())} weights and {off_r} NCCs of {F * pix} "
          "off their rounding", flush=True)
    assert not off.any() and off_r == 0
