"""The weight step's two forms (one and four threads a pixel) on either side of their line."""
import numpy as np
import pytest

from paper_2412_02413_amd import synth

pytestmark = pytest.mark.gpu
MM = 1e-3


# FP64 sums of the same FP32 partial sums, rounded once to FP32 (2^-24), whatever the order of the FP64 additions.
@pytest.mark.parametrize("n_x,n_z,n_sub,frames", [
    (128, 16, 3, 1),      # 8 workgroups of 256 pixels: four threads
    (256, 256, 3, 1),     # 256, the last of that form with three sub-apertures
    (256, 260, 3, 1),     # 260: one thread
    (256, 260, 1, 1),     # with one sub-aperture four threads up to 512
    (256, 520, 1, 1),     # 520: one thread
    (128, 151, 2, 6),     # 456 with few splits
])
def test_weight_forms(n_x, n_z, n_sub, frames):
    import torch
    from paper_2412_02413_amd import pam
    g = synth.Geometry(n_elements=64, pitch_m=0.3 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=1024, bands_hz=[(1e6, 5e6)],
                       depths_m=(15 + 0.1 * np.arange(n_z)) * MM, n_x=n_x, n_sub=n_sub)
    gen = torch.Generator(device="cuda").manual_seed(n_z)
    rf = torch.randn((frames, 64, 1024), generator=gen, device="cuda")
    plan = pam.pam_plan(g, 0, "fp32")
    try:
        out = pam.reconstruct(plan, rf)
        torch.cuda.synchronize()
        lay = pam.pam_workspace_layout(plan, frames)
    finally:
        pam.pam_destroy(plan)
    pix = n_z * n_x

    def view(offset, n):
        return out["workspace"][offset: offset + 4 * n].cpu().numpy().view(np.float32).astype(np.float64)

    acc = view(lay.accum, lay.n_split * frames * lay.n_acc * pix).reshape(lay.n_split, frames, lay.n_acc, pix).sum(0)
    S, C = acc[:, :n_sub], acc[:, n_sub:]
    w = np.ones((frames, pix))
    for q, (i, j) in enumerate({1: [], 2: [(0, 1)], 3: [(0, 1), (1, 2), (2, 0)]}[n_sub]):
        w *= np.clip(C[:, q] / np.sqrt(S[:, i] * S[:, j]), 1e-3, 1)
    w = np.cbrt(w) if n_sub == 3 else w
    print(f"{lay.n_split} splits, {-(-pix // 256) * frames} workgroups", flush=True)
    np.testing.assert_allclose(view(lay.weight, frames * pix).reshape(frames, pix), w, rtol=2.0 ** -23)
    np.testing.assert_allclose(view(lay.energy, frames * pix).reshape(frames, pix), S.sum(1) + 2 * C.sum(1), rtol=2.0 ** -23,
                               atol=2.0 ** -48 * np.abs(acc).sum(1).max())
    rho = out["nncc"].double().cpu().numpy().reshape(frames, pix)
    np.testing.assert_allclose(rho, w / w.max(axis=1, keepdims=True), rtol=2.0 ** -22)
