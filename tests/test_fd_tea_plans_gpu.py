"""FD-TEA-TAX on every kind of plan that accepts it, against the FP64 oracle (relative L2 of the
image <= 1e-5, absolute NNCC error <= 1e-4, as for the FP32 path everywhere)."""
import numpy as np
import pytest

from oracle import fd_tea as T
from paper_2412_02413_amd import synth

pytestmark = pytest.mark.gpu
MM = 1e-3


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2412_02413_amd import pam
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pam._lib()
    return torch, pam


def check_fd_tea(env, g, frames, seed):
    """Frames of different content through a workspace that holds NaN wherever the call does not
    write: a partial sum read from a place that was not written shows in the image."""
    torch, pam = env
    rng = np.random.default_rng(seed)
    rf = np.stack([synth.render(g, [synth.Emitter((0.4 * f - 0.5) * MM, (14 + f) * MM, "broadband")], rng, snr_db=20.0)
                   for f in range(frames)])
    plan = pam.pam_plan(g, 0, "fp32")
    try:
        img = torch.full((frames, plan.n_z, plan.n_x), -1.0, device="cuda")
        nncc = torch.full_like(img, -1.0)
        ws = pam.alloc_workspace(plan, frames, g.n_samples).fill_(255)
        pam.pam_fd_tea_tax(plan, torch.from_numpy(rf).cuda(), img, nncc, None, ws)
        torch.cuda.synchronize()
        n_split = pam.pam_workspace_layout(plan, frames, g.n_samples).n_split
    finally:
        pam.pam_destroy(plan)
    for f in range(frames):
        ref = T.fd_tea_tax(rf[f], g)
        I, rho = img[f].double().cpu().numpy(), nncc[f].double().cpu().numpy()
        e_i = float(np.linalg.norm(I - ref["I"]) / np.linalg.norm(ref["I"]))
        e_r = float(np.abs(rho - ref["rho_n"]).max())
        print(f"frame {f}: relL2(I)={e_i:.2e} max|d rho_n|={e_r:.2e}", flush=True)
        assert e_i <= 1e-5 and e_r <= 1e-4
    return n_split


@pytest.mark.parametrize("frames,bins_hi", [(1, 9e6), (2, 9e6), (2, 2.5e6)])
def test_plan_with_pair_sums(env, frames, bins_hi):
    """A coherence plan keeps five accumulator planes a frame, of which delay-and-sum writes the
    first: several frames and several bin splits have to land where the weight step reads them."""
    g = synth.Geometry(n_elements=32, pitch_m=0.3 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=512,
                       bands_hz=[(2e6, bins_hi)], depths_m=(12 + 0.5 * np.arange(14)) * MM, n_x=256, n_sub=1,
                       apod=np.ones((1, 32), np.uint8), coherence=1)
    n_split = check_fd_tea(env, g, frames, 5)
    assert n_split > 1


@pytest.mark.parametrize("L,n_x,lateral,n_sub,kw", [
    (1, 32, "pad", 1, {}),                                    # one thread a pixel from here ...
    (1, 512, "stuff", 2, {}),
    (2, 96, "stuff", 3, {"pattern_m": 1}),
    (2, 512, "pad", 3, {"pattern_m": 1}),
    (4, 64, "stuff", 3, {"apod": np.uint8([[1, 1, 0, 0], [0, 1, 1, 0], [0, 1, 0, 1]])}),   # in several and in none
    (5, 288, "pad", 3, {"pattern_m": 2}),
    (3, 512, "pad", 3, {"pattern_m": 1}),
    (7, 224, "stuff", 3, {"pattern_m": 2}),                   # ... to the most it takes
    (4, 448, "pad", 3, {"pattern_m": 1}),                     # the table's first
    (8, 32, "stuff", 3, {"pattern_m": 2}),
])
def test_few_elements(env, L, n_x, lateral, n_sub, kw):
    """Both sides of the line between one thread a pixel and the phasor table; 11 depths leave a ragged last tile."""
    g = synth.Geometry(n_elements=L, pitch_m=0.3 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=128, bands_hz=[(2e6, 6e6)],
                       depths_m=(12 + 0.7 * np.arange(11)) * MM, n_x=n_x, n_sub=n_sub, lateral=lateral).replace(**kw)
    check_fd_tea(env, g, 2, L + n_x)


@pytest.mark.parametrize("L,n_x,lateral,n_z,kw", [
    (13, 32, "pad", 2101, {"pattern_m": 3}),       # several rows a wave, a ragged last wave; mixed units
    (9, 288, "stuff", 130, {"pattern_m": 1}),      # 32 residues a depth
    (48, 96, "stuff", 601, {}),                    # rows of 12 lanes
    (190, 288, "pad", 34, {"pattern_m": 3}),       # one row a wave, two waves a row, 24 units
])
def test_rows_per_wave(env, L, n_x, lateral, n_z, kw):
    """Launches of more and of less than a wave per SIMD, which pack several rows or one into a wave."""
    g = synth.Geometry(n_elements=L, pitch_m=0.1 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=64, bands_hz=[(2e6, 5e6)],
                       depths_m=(12 + 8.0 / n_z * np.arange(n_z)) * MM, n_x=n_x, n_sub=3, lateral=lateral).replace(**kw)
    check_fd_tea(env, g, 2, L)
