"""The impulse response at the edges of its kernel: fewer and more elements than
a wave, bins narrower and wider than the surface (one bin a slot, or one an
element), the number of bins around one pass of the counters, bin widths whose
reciprocal does not divide exactly."""
import numpy as np
import pytest

from paper_2402_13034_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


@pytest.mark.parametrize("n_elem", [1, 63, 64, 65, 127, 400])
def test_bins_against_the_kept_paths(ctx, n_elem):
    """Every bin against the sum of the paths that the channel keeps, with the
    bins of NumPy's division: the FP32 result's rounding is all they differ by
    (2^-24 of it; the sums of at most 10^5 terms in 64 bits are closer)."""
    import torch
    from paper_2402_13034_amd import risrt
    p = synth.lab_room(nx=5, ny=3, n_rays=20_000, order=2)
    lam = p.wavelength
    side = int(np.ceil(np.sqrt(n_elem)))
    k = np.arange(n_elem)
    p.ris.elems = p.ris.centre + lam / 2 * np.stack([0.0 * k, k % side - side / 2, k // side - side / 2], 1)
    rng = np.random.default_rng(n_elem)
    g = np.exp(2j * np.pi * rng.random(n_elem)).astype(np.complex64)
    scene, ris = risrt.upload_problem(ctx, p)
    ch, _ = risrt.trace_problem(ctx, p, scene, ris, flags=risrt.FLAG_KEEP_CIR | risrt.FLAG_KEEP_PATHS)
    kept = ctx.paths_read(ch)
    amp, length = ctx.ris_paths_read(ch)
    R = p.rx_pos.shape[0]
    # a receiver's slots: the direct one, then its sequences'
    slot_rx = np.repeat(np.arange(R), 1 + np.bincount(kept["useq"][:, 0], minlength=R))
    amp = amp.reshape(len(slot_rx), n_elem).astype(np.complex128)
    env = kept["env"]
    rx = np.r_[env["rx"], np.repeat(slot_rx, n_elem)]
    a = np.r_[env["amp"][:, 0] + 1j * env["amp"][:, 1].astype(np.float64), (amp * g.astype(np.complex128)).ravel()]
    length = np.r_[env["length"], length.ravel()]
    on = a != 0
    rx, a, length = rx[on], a[on], length[on]
    gd = torch.from_numpy(g).cuda()
    # 3 ps: a millimetre a bin; 100 ns: all in one; powers of two and not; one bin, a pass and its neighbours, two
    for bin_s, n_bins in ((3e-12, 3072), (3e-12, 3073), (2.5e-10, 400), (1e-10, 1), (1.0 / 299792458.0 / 8, 3071),
                          (1e-7, 6144), (7.3e-12, 6145)):
        print("case cir", n_elem, bin_s, n_bins, flush=True)
        h = ctx.cir(ch, gd, bin_s, n_bins)
        torch.cuda.synchronize()
        h = h.cpu().numpy().astype(np.complex128)
        b = np.floor(length / (299792458.0 * bin_s))
        keep = b < n_bins
        want, inc = np.zeros((R, n_bins), np.complex128), np.zeros((R, n_bins))
        np.add.at(want, (rx[keep], b[keep].astype(np.int64)), a[keep])
        np.add.at(inc, (rx[keep], b[keep].astype(np.int64)), np.abs(a[keep]))
        for x, y in ((h.real, want.real), (h.imag, want.imag)):
            assert np.all(np.abs(x - y) <= 2.0 ** -24 * np.abs(y) + 2.0 ** -35 * inc), (bin_s, n_bins)
    for o in (ch, scene, ris):
        ctx.destroy(o)
