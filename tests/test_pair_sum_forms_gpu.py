"""The two forms of the FP32 pair-sum fields kernel: launches of up to two (or four) workgroups per CU, and others."""
import numpy as np
import pytest

from oracle import as_tax as O
from paper_2412_02413_amd import synth

pytestmark = pytest.mark.gpu
MM = 1e-3


def test_both_forms_give_the_same_bits():
    """The pair sums become BF16 features, so which form a call takes must not show: 16 frames of 512 x 256
    pixels (512 workgroups, two per CU) and the same 16 inside 48 frames (six per CU) have equal sums, bit for bit;
    one frame of the 16 and one of the others agrees with the oracle's pair sums (2e-5 of the largest, the FP32 path's bound)."""
    import torch
    from paper_2412_02413_amd import pam
    g = synth.cfg2_geometry()
    g = g.replace(n_samples=256, n_sub=1, apod=np.ones((1, g.n_elements), np.uint8), coherence=1)
    rng = np.random.default_rng(17)
    em = [synth.Emitter(-2 * MM, 30 * MM, "broadband"), synth.Emitter(3 * MM, 22 * MM, "broadband")]
    rf = np.stack([synth.render(g, em, rng, snr_db=10.0) for _ in range(48)])
    x = torch.from_numpy(rf).cuda()
    plan = pam.pam_plan(g, 0, "fp32")
    sums = {}
    try:
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        for F in (16, 48):
            lay = pam.pam_workspace_layout(plan, F, g.n_samples)
            assert lay.n_split == 1 and lay.n_acc == 5
            per_cu = -(-F * (g.n_z // 16) // cus)
            assert per_cu == (2 if F == 16 else 6), "the two launches must take the two forms"
            out = pam.reconstruct(plan, x[:F].contiguous())
            torch.cuda.synchronize()
            n = F * 5 * g.n_z * g.n_x
            acc = out["workspace"][lay.accum: lay.accum + 4 * n].view(torch.float32)
            sums[F] = acc.view(F, 5, g.n_z, g.n_x).cpu().numpy()
            assert np.isfinite(sums[F]).all() and (sums[F][:, 0] > 0).any()
    finally:
        pam.pam_destroy(plan)
    assert np.array_equal(sums[16].view(np.uint32), sums[48][:16].view(np.uint32))
    for f in (3, 29):
        ref = O.pair_cross_spectra(rf[f], g)
        a, smax = sums[48][f].astype(np.float64), ref["S"].max()
        e = [np.abs(a[0] - ref["S"]).max() / smax, np.abs(a[1] + 1j * a[2] - ref["Gx"]).max() / smax,
             np.abs(a[3] + 1j * a[4] - ref["Gz"]).max() / smax]
        print(f"frame {f}: S {e[0]:.1e} Gx {e[1]:.1e} Gz {e[2]:.1e}", flush=True)
        assert max(e) <= 2e-5
