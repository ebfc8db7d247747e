"""Metropolis sweeps at the edges of their two forms (one workgroup with the
state in LDS up to 768 sites per class and 32 classes, a launch per class above):
class sizes around the workgroup's 512 threads and the limit, stretches of 1024
sweeps that end inside and at the end of a temperature, single sites, flat
boxes, many classes.  Against the oracle: accepted moves per sweep equal,
states to the fp32 output (2^-24 of a unit component, doubled)."""
import numpy as np
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu


def _bonds(L, J, D):
    n = L[0] * L[1] * L[2]
    i = np.arange(n).reshape(L)
    row, col, dv = [0], [], []
    nb = [np.roll(i, -s, a).reshape(-1) for a in range(3) for s in (1, -1)]
    for k in range(n):
        for e in range(6):
            if nb[e][k] != k:
                d = np.zeros(3)
                d[e // 2] = D * (1 if e % 2 == 0 else -1)
                col.append(nb[e][k])
                dv.append(d)
        row.append(len(col))
    f = lambda x: np.asarray(x, np.float32).astype(np.float64)
    return np.array(row, np.int64), np.array(col, np.int32), f(np.full(len(col), J)), f(np.array(dv).reshape(-1, 3))


# (cells, sweeps per temperature, sweeps at the end)
CASES = [((1, 1, 1), 2, 3), ((32, 32, 1), 3, 5), ((32, 32, 2), 3, 5), ((38, 40, 1), 2, 4), ((48, 32, 1), 2, 4), ((50, 31, 1), 2, 4),
         ((6, 6, 6), 100, 330), ((6, 6, 6), 512, 1), ((5, 4, 3), 341, 2048), ((2, 4, 2), 1, 1)]


@pytest.mark.parametrize("D", [0.0, 0.3])
@pytest.mark.parametrize("L,per_T,final", CASES)
def test_lattice_sweeps_match_oracle(orc, L, per_T, final, D):
    import torch
    from paper_2308_07487_amd import sdc as S
    print(f"[case] mc small {L} {per_T} {final} D={D}", flush=True)
    pos = inputs.sc_positions(L)
    n = pos.shape[0]
    spec = S.mc_spec(S.BINS_SC, cells=L, J=-1.0, D=D, A=0.1, Hz=0.4, seed=0x5DC0A301, T_start=2.0, T_end=0.4,
                     cool=0.6, sweeps_per_T=per_T, sweeps_final=final)
    init = inputs.random_unit_frames(1, n, seed=31)[0]
    st = torch.from_numpy(init).cuda()
    acc, E, cone, T, ncol = S.mc_anneal(pos, spec, st, st)
    row, col, J, Dv = _bonds(L, -1.0, D)
    ref = orc.mc_anneal(row, col, J, init, spec.seed, 2.0, 0.4, 0.6, per_T, final, D=Dv, A=0.1, Hz=0.4)
    assert ncol == ref[5] and T == ref[4]
    np.testing.assert_array_equal(acc, ref[1])
    assert np.abs(st.cpu().numpy() - ref[0]).max() < 2 ** -23
    assert abs(E - ref[2]) < 1e-10 * max(1.0, abs(ref[2])) and abs(cone - ref[3]) < 1e-12


@pytest.mark.parametrize("n,r_cut", [(200, 0.8), (200, 2.5), (300, 4.0)])
def test_open_samples_continue(orc, n, r_cut):
    """Few and many colour classes; a second run continues the first."""
    import torch
    from paper_2308_07487_amd import sdc as S
    print(f"[case] mc open n={n} r_cut={r_cut}", flush=True)
    pos = inputs.ball_positions(n, 3.0, seed=9)
    spec = S.mc_spec(S.BINS_RADIAL, coupling=S.COUPLING_EXP_CUTOFF, r_cut=r_cut, J=1.0, Hz=0.2, seed=3, T_start=1.0,
                     T_end=0.5, cool=0.8, sweeps_per_T=2, sweeps_final=3)
    init = inputs.random_unit_frames(1, n, seed=33)[0]
    d = (pos[None] - pos[:, None]).astype(np.float32)
    d2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
    hit = (d2 <= np.float32(r_cut) * np.float32(r_cut)) & ~np.eye(n, dtype=bool)
    row = np.concatenate([[0], np.cumsum(hit.sum(1))]).astype(np.int64)
    col = np.nonzero(hit)[1].astype(np.int32)
    J = np.exp(-np.sqrt(d2[hit].astype(np.float64))).astype(np.float32).astype(np.float64)
    ref = orc.mc_anneal(row, col, J, init, 3, 1.0, 0.5, 0.8, 2, 3, Hz=0.2)
    st = torch.from_numpy(init).cuda()
    with S.MonteCarlo(pos, spec) as mc:
        acc, info = mc.run(spec, st, init_state=st, history=True, info=True)
        np.testing.assert_array_equal(acc, ref[1])
        assert int(info[3]) == ref[5]
        assert np.abs(st.cpu().numpy() - ref[0]).max() < 2 ** -23
        # a run from the kept FP64 state starts at the first run's end
        again = torch.zeros_like(st)
        one = S.mc_spec(S.BINS_RADIAL, coupling=S.COUPLING_EXP_CUTOFF, r_cut=r_cut, J=1.0, Hz=0.2, seed=3,
                        T_start=0.5, T_end=0.5, sweeps_final=0)
        mc.run(one, again)
        np.testing.assert_array_equal(again.cpu().numpy(), st.cpu().numpy())
