"""Default stream segments, which are fitted to the sample: the same bins as
segments of one tile pair and as whole streams, bit for bit on dyadic spins
(every product and sum is exact, so any split of the work must agree)."""
import numpy as np
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [("sc", (2, 2, 2), 5, 3), ("sc", (12, 12, 8), 16, 40), ("sc", (23, 24, 1), 9, 17), ("bcc", (5, 6, 4), 20, 33),
         ("radial", (130, 33), 8, 12), ("radial", (1500, 1024), 24, 70)]


@pytest.mark.parametrize("prec", ["split_bf16", "fp32"])
@pytest.mark.parametrize("kind,L,n_o,n_L", CASES, ids=[f"{c[0]}{c[1]}" for c in CASES])
def test_default_segments_equal_any_other(kind, L, n_o, n_L, prec):
    import torch
    from paper_2308_07487_amd import sdc as S
    print(f"[case] segments {kind} {L} {prec}", flush=True)
    if kind == "radial":
        pos, k, kw = inputs.ball_positions(L[0], 4.0, 3), S.BINS_RADIAL, dict(n_shells=L[1], r_max=8.0)
    else:
        pos = inputs.sc_positions(L) if kind == "sc" else inputs.bcc_positions(L)
        k, kw = (S.BINS_SC if kind == "sc" else S.BINS_BCC), dict(cells=L)
    fr = torch.from_numpy(inputs.dyadic_frames(n_o + n_L - 1, pos.shape[0], 7)).cuda()
    H = []
    for seg in (None, 1, 1 << 20):
        with S.Plan(pos, k, n_o, n_L, prec, segment_pairs=seg, **kw) as p:
            p.accumulate(fr)
            H.append(p.raw()[0])
    np.testing.assert_array_equal(H[0], H[1])
    np.testing.assert_array_equal(H[0], H[2])
