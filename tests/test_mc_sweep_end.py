"""The end of a sweep that runs a launch per colour class: the last workgroup
of the last class sums the accepted moves and adapts the cone.

On the CPU, from the device code's intermediate form: the counts reach that
workgroup in the values of read-modify-write atomics, never by reading a
counter that other workgroups of the launch add to (nothing orders such a read
after their adds).  On the GPU, against the oracle: fewer, as many and more
workgroups in the last class than there are counters, and last classes much
smaller than the others, whose counters then hold moves of earlier launches."""
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2308_07487_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_counts_travel_in_read_modify_writes(tmp_path):
    ll = tmp_path / "mc.ll"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-S", "-emit-llvm",
                           "--cuda-device-only", "-I", os.path.join(ROOT, "include"),
                           os.path.join(ROOT, "paper_2308_07487_amd", "csrc", "sdc_mc.hip"), "-o", str(ll)],
                          stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^define [^\n]*amdgpu_kernel void @\S*mc_colour_kernel.*?^}", ll.read_text(), re.M | re.S)
    assert len(kernels) == 4
    for k in kernels:
        assert len(re.findall(r"= atomicrmw add .*agent", k)) == 3  # inner classes, counter, ticket
        assert "load atomic" not in k


def _bonds(L, J, D):
    n = L[0] * L[1] * L[2]
    i = np.arange(n).reshape(L)
    nb = np.stack([np.roll(i, -s, a).reshape(-1) for a in range(3) for s in (1, -1)], 1)
    dv = np.zeros((n, 6, 3))
    for e in range(6):
        dv[:, e, e // 2] = D * (1 if e % 2 == 0 else -1)
    f = lambda x: np.ascontiguousarray(np.asarray(x, np.float32).astype(np.float64))
    return (np.arange(n + 1, dtype=np.int64) * 6, nb.reshape(-1).astype(np.int32), f(np.full(6 * n, J)),
            f(dv.reshape(-1, 3)))


# workgroups of the last class: 4, 63, 64, 65, one of a few sites after larger classes (odd edges)
@pytest.mark.gpu
@pytest.mark.parametrize("L", [(16, 16, 8), (36, 28, 32), (32, 32, 32), (40, 26, 32), (33, 32, 32), (31, 33, 35)])
def test_sweeps_match_oracle(orc, L):
    import torch
    from paper_2308_07487_amd import sdc as S
    print(f"[case] mc sweep end {L}", flush=True)
    pos = inputs.sc_positions(L)
    n = pos.shape[0]
    spec = S.mc_spec(S.BINS_SC, cells=L, J=-1.0, D=0.2, A=0.1, Hz=0.4, seed=0x5DC0A302, T_start=2.0, T_end=0.9,
                     cool=0.7, sweeps_per_T=2, sweeps_final=3)
    init = inputs.random_unit_frames(1, n, seed=31)[0]
    st = torch.from_numpy(init).cuda()
    acc, E, cone, T, ncol = S.mc_anneal(pos, spec, st, st)
    ref = orc.mc_anneal(*_bonds(L, -1.0, 0.2)[:3], init, spec.seed, 2.0, 0.9, 0.7, 2, 3, D=_bonds(L, -1.0, 0.2)[3],
                        A=0.1, Hz=0.4)
    assert ncol == ref[5] and T == ref[4]
    np.testing.assert_array_equal(acc, ref[1])
    assert np.abs(st.cpu().numpy() - ref[0]).max() < 2 ** -23
    assert abs(E - ref[2]) < 1e-10 * max(1.0, abs(ref[2])) and abs(cone - ref[3]) < 1e-12
