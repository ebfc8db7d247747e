"""S(q, t) from the bins at the edges of its lag blocks (8 lags share a bin's
phase), for negative and large wave-vector indices, sc, bcc and flat boxes:
against the same sum over the raw bins in numpy.  Both sides sum n_bins
terms in FP64; the phases agree to a few 2^-53, so 1e-13 of the absolute sum
holds with a wide margin over the rounding of up to 2000 terms."""
import numpy as np
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_L", [1, 7, 8, 9, 65])
@pytest.mark.parametrize("kind,L", [("sc", (3, 5, 7)), ("bcc", (4, 3, 2)), ("sc", (30, 33, 1)), ("sc", (1, 1, 2))])
def test_structure_factor_from_bins(kind, L, n_L):
    import torch
    from paper_2308_07487_amd import sdc as S
    print(f"[case] sqt {kind} {L} n_L={n_L}", flush=True)
    bcc = kind == "bcc"
    pos = inputs.bcc_positions(L) if bcc else inputs.sc_positions(L)
    n, n_o = pos.shape[0], 6
    fr = torch.from_numpy(inputs.random_unit_frames(n_o + n_L - 1, n, 4)).cuda()
    m = np.array([[0, 0, 0], [1, -2, 3], [-(1 << 20), 1 << 20, 7], [L[0], -L[1], 2 * L[2] + 1]], dtype=np.int32)
    with S.Plan(pos, S.BINS_BCC if bcc else S.BINS_SC, n_o, n_L, "fp32", cells=L) as p:
        p.accumulate(fr)
        H = p.raw()[0]
        for _ in range(2):  # the second call reuses the first one's scratch
            sqt, sqw = p.structure_factor(m)
        st, sw = p.structure_factor_static(m)
        few = p.structure_factor(m[:1])
    np.testing.assert_array_equal(few[0], sqt[:1])
    np.testing.assert_array_equal(st, sqt)
    np.testing.assert_array_equal(sw, sqw)
    cell = inputs.sc_positions(L).astype(np.float64)
    d = np.stack([cell, cell + 0.5], 1).reshape(-1, 3) if bcc else cell
    # phases reduced in integers first: 2 m_a d_a mod 2 L_a
    k = (2 * m[:, None, :].astype(np.int64) * (2 * d[None]).astype(np.int64)) // 2 % (2 * np.array(L))
    ph = np.exp(-1j * np.pi * (k / np.array(L, dtype=np.float64)).sum(-1))
    ref = ph @ H.T / (n * n_o)
    scale = np.abs(H).sum(1) / (n * n_o)
    assert np.all(np.abs(sqt - ref) <= 1e-13 * scale[None, :])
    w = 0.5 * (1.0 + np.cos(np.pi * np.arange(n_L) / n_L))
    assert np.all(np.abs(sqw - np.fft.fft(w * ref, axis=1)) <= 1e-13 * n_L * scale.max())
