"""The self sums and what is formed beside them (site sums, spectra, the i = j
part of the dropped products) where their work split changes: fewer sites
than a workgroup takes, ragged last groups, lag counts around the thread
counts, long series that leave the LDS budget of the pieces and of the plain
series, the connected form, and every precision.

Self and site sums are FP64 sums of at most n n_o products of fp32 values:
each is held to 1e-12 of the sum of the absolute products (4e5 terms at
2^-53 each, worst case 5e-11, random 3e-13)."""
import numpy as np
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu

# (n sites in a ball, n_o, n_L, stride)
SHAPES = [(1, 1, 1, 1), (3, 2, 5, 1), (67, 8, 63, 2), (130, 9, 65, 1), (1025, 5, 257, 1), (40, 16, 300, 3),
          (5, 900, 1024, 1), (2, 1024, 40, 8), (20, 4, 130, 64)]


@pytest.mark.parametrize("prec", ["fp32", "split_bf16", "split_fp16", "bf16x3"])
@pytest.mark.parametrize("n,n_o,n_L,stride", SHAPES)
def test_self_and_site_sums(n, n_o, n_L, stride, prec):
    import torch
    from paper_2308_07487_amd import sdc as S
    print(f"[case] self sums n={n} n_o={n_o} n_L={n_L} stride={stride} {prec}", flush=True)
    pos = inputs.ball_positions(n, 2.0, 3)
    T = (n_o - 1) * stride + n_L
    fr = inputs.random_unit_frames(T, n, seed=5)
    for connected in (False, True):
        with S.Plan(pos, S.BINS_RADIAL, n_o, n_L, prec, n_shells=4, r_max=4.0, origin_stride=stride,
                    connected=connected) as p:
            p.accumulate(torch.from_numpy(fr).cuda())
            out = p.finalize()
            _, no, sf, ms = p.raw()
        x = fr.astype(np.float64)
        e = x[0:(n_o - 1) * stride + 1:stride]
        if connected:  # the mean the device subtracts is rounded to fp32
            m = e.mean(0).astype(np.float32)
            e_site = (fr[0:(n_o - 1) * stride + 1:stride] - m).astype(np.float64)
            e_sum = e.sum(1) - e.sum(1).mean(0)
        else:
            e_site, e_sum = e, e.sum(1)
        tot = x.sum(1)
        for t in range(n_L):
            k = slice(t, t + (n_o - 1) * stride + 1, stride)
            prod = e_site * x[k]
            assert abs(sf[t] - prod.sum()) <= 1e-12 * max(np.abs(prod).sum(), 1.0)
            prod = e_sum * tot[k]
            assert abs(ms[t] - prod.sum()) <= 1e-12 * max(np.abs(prod).sum(), n * n_o)
        np.testing.assert_array_equal(no, n_o)
        w = 0.5 * (1.0 + np.cos(np.pi * np.arange(n_L) / n_L))
        for c, s in ((out["Csum"], out["Ssum"]), (out["Cself"], out["Sself"])):
            # n_L terms, each phase and weight within a few 2^-53
            np.testing.assert_allclose(s, np.fft.fft(w * c), rtol=0, atol=1e-14 * n_L * max(np.abs(c).max(), 1.0))
