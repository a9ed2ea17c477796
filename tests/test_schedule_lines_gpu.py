"""Which side of their lines the bin split and the grouped launch take, at calls measured on both sides."""
import numpy as np
import pytest

from paper_2412_02413_amd import synth

pytestmark = pytest.mark.gpu
MM = 1e-3


def geometry(n_x, n_z, n_sub, n_samples, hi, precision="fp32"):
    return synth.Geometry(n_elements=64, pitch_m=0.3 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=n_samples,
                          bands_hz=[(1e6, hi)], depths_m=(15 + 0.2 * np.arange(n_z)) * MM, n_x=n_x, n_sub=n_sub)


@pytest.mark.parametrize("n_x,n_z,n_sub,n_samples,hi,frames,splits,precision", [
    (128, 151, 3, 1024, 5e6, 1, 52, "fp32"),         # empty CUs: 4 bins a workgroup (53.1 us with 8, 45.7)
    (384, 93, 3, 1024, 5e6, 1, 41, "fp32"),          # the same with wider workgroups (82.1 us with 8, 65.9)
    (128, 166, 2, 256, 2e6, 19, 2, "fp32"),          # a workgroup on each CU already (44.7 us with 4 bins, 39.0)
    (256, 9, 1, 256, 3e6, 62, 4, "split_bf16"),      # 16-bit workgroups gain nothing from sharing a CU (35.2 us, 33.6)
])
def test_bin_split(n_x, n_z, n_sub, n_samples, hi, frames, splits, precision):
    from paper_2412_02413_amd import pam
    plan = pam.pam_plan(geometry(n_x, n_z, n_sub, n_samples, hi), 0, precision)
    try:
        n = pam.pam_workspace_layout(plan, frames).n_split
        print(f"{plan.info.n_bins} bins in {n} splits", flush=True)
        assert n == splits
    finally:
        pam.pam_destroy(plan)


@pytest.mark.parametrize("n_x,n_z,n_sub,n_samples,hi,groups,one", [
    (256, 219, 3, 256, 9e6, [(64, 1), (32, 13)], True),              # 92 us in one launch, 105 apart
    (96, 502, 2, 256, 9e6, [(32, 10), (128, 6), (32, 3)], True),     # 117, 130
    (384, 17, 2, 8192, 5e6, [(8192, 23), (1024, 1)], False),         # 1,446, 1,257
])
def test_grouped_launch(n_x, n_z, n_sub, n_samples, hi, groups, one):
    """The schedule taken, and every frame equal to the per-length call up to the order of FP32 sums (1e-5 of the
    image, as for the grouped call everywhere)."""
    import torch
    from paper_2412_02413_amd import pam
    g = geometry(n_x, n_z, n_sub, n_samples, hi)
    plan = pam.pam_plan(g, 0, "fp32")
    try:
        assert pam.debug_grouped_one_launch(plan, groups) == one
        F = sum(f for _, f in groups)
        gen = torch.Generator(device="cuda").manual_seed(5)
        parts = [torch.randn((f, 64, n), generator=gen, device="cuda") for n, f in groups]
        img = torch.empty((F, n_z, n_x), device="cuda")
        pam.pam_as_tax_grouped(plan, torch.cat([p.view(-1) for p in parts]), groups, img, None, None,
                               pam.alloc_workspace_grouped(plan, groups))
        at = 0
        for p in parts:
            alone = pam.reconstruct(plan, p)["image"]
            got = img[at: at + len(p)]
            e = ((got - alone).double().norm(dim=(1, 2)) / alone.double().norm(dim=(1, 2))).max().item()
            assert e <= 1e-5, e
            at += len(p)
    finally:
        pam.pam_destroy(plan)
