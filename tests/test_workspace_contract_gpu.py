"""What a caller may rely on about workspaces: the layout that a call uses in a workspace of a given
size, the least size accepted, and the allocation-free call at its scratch limit."""
import numpy as np
import pytest

from paper_2412_02413_amd import synth

pytestmark = pytest.mark.gpu
MM = 1e-3
FIELDS = ("spectra", "coeffs", "scales", "accum", "energy", "weight", "blockmax", "total", "n_sel", "n_split", "n_acc")


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2412_02413_amd import pam
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pam._lib()
    return torch, pam


def case(n_x, n_sub, n_z=64, n_samples=1024):
    """A small array: 205 bins at 1,024 samples."""
    g = synth.Geometry(n_elements=32, pitch_m=0.3 * MM, fs_hz=20e6, c_mps=1540.0, n_samples=n_samples, bands_hz=[(2e6, 6e6)],
                       depths_m=(15 + 0.1 * np.arange(n_z)) * MM, n_x=n_x, n_sub=n_sub, pattern_m=4)
    rng = np.random.default_rng(n_x + n_sub)
    em = [synth.Emitter(-1.0 * MM, 17 * MM, "broadband"), synth.Emitter(2.0 * MM, 20 * MM, "broadband")]
    return g, np.stack([synth.render(g, em, rng, snr_db=20.0) for _ in range(2)])


@pytest.mark.parametrize("n_x,n_sub,precision", [(96, 3, "fp32"), (192, 2, "fp32"), (384, 3, "fp32"), (480, 1, "fp32"),
                                                 (128, 3, "fp32"), (256, 2, "fp32"), (512, 3, "fp32"),
                                                 (96, 3, "split_bf16"), (256, 3, "bf16")])
def test_layout_in_is_the_one_used(env, n_x, n_sub, precision):
    torch, pam = env
    g, rf = case(n_x, n_sub)
    F, pix = 2, g.n_z * n_x
    plan = pam.pam_plan(g, 0, precision)
    try:
        x = torch.from_numpy(rf).cuda()
        img, nncc = (torch.empty((F, g.n_z, n_x), device="cuda") for _ in range(2))
        full = pam.pam_workspace_layout(plan, F)
        least = pam.pam_workspace_layout_in(plan, F, 0)
        same = [getattr(pam.pam_workspace_layout_in(plan, F, full.total), k) for k in FIELDS]
        assert same == [getattr(full, k) for k in FIELDS]
        if precision == "fp32" and n_x not in (128, 256, 512):
            assert least.total < full.total and least.accum == full.accum
            # at 384 columns the smaller reservation's 43 spare planes allow 2 frames 22 splits, the call would take more
            assert least.n_split <= full.n_split and (n_x != 384 or least.n_split <= 22 < full.n_split)
        else:
            assert [getattr(least, k) for k in FIELDS] == same

        def call(nbytes):
            """Outputs and the workspace's bytes; the bytes after the workspace have to stay."""
            buf = torch.full((nbytes + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
            img.fill_(-7.0)
            nncc.fill_(-7.0)
            pam.pam_as_tax(plan, x, img, nncc, None, buf[:nbytes])
            torch.cuda.synchronize()
            assert bool((buf[nbytes:] == 0xA5).all())
            return img.cpu().numpy(), nncc.cpu().numpy(), buf.cpu().numpy()

        # one byte less than the least: refused, nothing written
        img.fill_(-7.0)
        short = torch.full((least.total,), 0xA5, dtype=torch.uint8, device="cuda")
        with pytest.raises(pam.PamError) as e:
            pam.pam_as_tax(plan, x, img, None, None, short[:least.total - 1])
        assert e.value.status == pam.PAM_ERR_WORKSPACE
        torch.cuda.synchronize()
        assert bool((img == -7.0).all()) and bool((short == 0xA5).all())

        ref, _, _ = call(full.total)
        for nbytes in sorted({least.total, (least.total + full.total) // 2, full.total}):
            lay = pam.pam_workspace_layout_in(plan, F, nbytes)
            assert lay.total <= nbytes
            I, rho, ws = call(nbytes)

            def view(offset, n):
                return ws[offset: offset + 4 * n].view(np.float32).astype(np.float64)

            acc = view(lay.accum, lay.n_split * F * lay.n_acc * pix).reshape(lay.n_split, F, lay.n_acc, pix).sum(0)
            E = acc[:, :n_sub].sum(1) + 2 * acc[:, n_sub:].sum(1)
            energy, weight = view(lay.energy, F * pix).reshape(F, pix), view(lay.weight, F * pix).reshape(F, pix)
            # FP32 outputs of FP64 sums of the same partial sums
            np.testing.assert_allclose(energy, E, rtol=2.0 ** -23)
            r = weight / weight.max(axis=1, keepdims=True)
            np.testing.assert_allclose(rho.reshape(F, pix), r, rtol=2.0 ** -23)
            np.testing.assert_allclose(I.reshape(F, pix), r * r * energy, rtol=2.0 ** -21)
            assert np.linalg.norm(I - ref) <= 1e-6 * np.linalg.norm(ref)
            if nbytes < full.total:
                least_bits = I if nbytes == least.total else least_bits
                assert np.array_equal(I, least_bits)
            print(f"{n_x}/{n_sub} {precision}: {nbytes} bytes, {lay.n_split} splits", flush=True)
    finally:
        pam.pam_destroy(plan)


@pytest.mark.parametrize("n_x,n_z", [(96, 64), (224, 151)])
def test_noalloc_at_its_limit(env, n_x, n_z):
    """The allocation-free call takes as many frames as fit its scratch with the smaller reservation,
    beyond what pam_workspace_size asks for, and not one more; results as with a workspace of its size."""
    torch, pam = env
    g, rf = case(n_x, 3, n_z, 256)
    limit = pam.NOALLOC_SCRATCH_BYTES
    plan = pam.pam_plan(g, 0, "fp32")
    try:
        F = 1
        while pam.pam_workspace_layout_in(plan, F + 1, limit).total <= limit:
            F += 1
        assert pam.pam_workspace_size(plan, F) > limit
        print(f"{n_x}: {F} frames", flush=True)
        x = torch.from_numpy(rf[np.arange(F + 1) % 2]).cuda()
        a, b = (torch.full((F + 1, g.n_z, n_x), -7.0, device="cuda") for _ in range(2))
        pam.pam_as_tax_noalloc(plan, x[:F], a[:F])
        pam.pam_as_tax(plan, x[:F], b[:F], None, None, torch.empty(limit, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        assert torch.equal(a, b) and bool((a[:F] >= 0).all())
        with pytest.raises(pam.PamError) as e:
            pam.pam_as_tax_noalloc(plan, x, b)
        assert e.value.status == pam.PAM_ERR_WORKSPACE
        torch.cuda.synchronize()
        assert torch.equal(a, b)
    finally:
        pam.pam_destroy(plan)
