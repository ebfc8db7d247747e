"""FP32 one-pass leaves out the zero samples of an odd block count's last K-step:
the same element sums as the lag-split schedule, which multiplies all of them.
The two differ by the order of the FP64 histogram adds alone, so a bin of
n <= N terms |x| <= n_o agrees to n 2^-53 sum|x| <= N^2 n_o 2^-53."""
import numpy as np
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_o", [1, 7, 8, 9, 17, 18, 23, 24, 33, 41, 50, 64])
@pytest.mark.parametrize("kind,L,n_L,stride", [("sc", (7, 5, 4), 21, 1), ("radial", (150, 40), 37, 2)])
def test_last_step_without_its_zeros(kind, L, n_L, stride, n_o):
    import torch
    from paper_2308_07487_amd import sdc as S
    print(f"[case] fp32 tail {kind} {L} n_o {n_o}", flush=True)
    if kind == "radial":
        pos, k, kw = inputs.ball_positions(L[0], 4.0, 3), S.BINS_RADIAL, dict(n_shells=L[1], r_max=8.0)
    else:
        pos, k, kw = inputs.sc_positions(L), S.BINS_SC, dict(cells=L)
    n, T = pos.shape[0], (n_o - 1) * stride + n_L
    rng = np.random.default_rng(n_o)
    x = rng.standard_normal((T, n, 3)).astype(np.float32)
    x /= np.linalg.norm(x, axis=2, keepdims=True)
    H = []
    for sched in ("one_pass", "lag_split"):
        with S.Plan(pos, k, n_o, n_L, "fp32", schedule=sched, origin_stride=stride, **kw) as p:
            p.accumulate(torch.from_numpy(x).cuda())
            H.append(p.raw()[0])
    assert np.abs(H[1]).max() > 0
    np.testing.assert_allclose(H[0], H[1], rtol=0, atol=n * n * n_o * 2.0 ** -53)
