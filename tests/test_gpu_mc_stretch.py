"""Small Metropolis samples of many classes: a launch runs as many sweeps as
come to 2048 class updates, so their schedules cross launches after 256 sweeps
(eight classes), 136 (15) and 70 (29), inside and at the end
of a temperature.  Against the oracle: accepted moves per sweep equal, states to
the fp32 output (2^-24 of a unit component, doubled)."""
import numpy as np
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,r_cut,per_T,final,classes", [((7, 7, 7), 1.8, 128, 150, 8), ((6, 6, 6), 2.1, 50, 64, (13, 16)),
                                                         ((6, 6, 6), 2.5, 33, 20, (25, 32)), ((40, 30, 1), 1.0, 1024, 1030, 2)])
def test_many_classes_cross_launches(orc, L, r_cut, per_T, final, classes):
    import torch
    from paper_2308_07487_amd import sdc as S
    print(f"[case] mc stretch {L} r_cut={r_cut}", flush=True)
    pos = inputs.sc_positions(L)
    n = pos.shape[0]
    spec = S.mc_spec(S.BINS_RADIAL, coupling=S.COUPLING_EXP_CUTOFF, r_cut=r_cut, J=-1.0, Hz=0.2, seed=5, T_start=2.0,
                     T_end=1.1, cool=0.7, sweeps_per_T=per_T, sweeps_final=final)
    init = inputs.random_unit_frames(1, n, seed=35)[0]
    d = (pos[None] - pos[:, None]).astype(np.float32)
    d2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
    hit = (d2 <= np.float32(r_cut) * np.float32(r_cut)) & ~np.eye(n, dtype=bool)
    row = np.concatenate([[0], np.cumsum(hit.sum(1))]).astype(np.int64)
    col = np.nonzero(hit)[1].astype(np.int32)
    J = (-np.exp(-np.sqrt(d2[hit].astype(np.float64)))).astype(np.float32).astype(np.float64)
    ref = orc.mc_anneal(row, col, J, init, 5, 2.0, 1.1, 0.7, per_T, final, Hz=0.2)
    lo, hi = classes if isinstance(classes, tuple) else (classes, classes)
    assert lo <= ref[5] <= hi
    st = torch.from_numpy(init).cuda()
    acc, E, cone, T, ncol = S.mc_anneal(pos, spec, st, st)
    assert ncol == ref[5] and T == ref[4]
    np.testing.assert_array_equal(acc, ref[1])
    assert np.abs(st.cpu().numpy() - ref[0]).max() < 2 ** -23
    assert abs(cone - ref[3]) < 1e-12
