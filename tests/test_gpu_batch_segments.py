"""Default segments in a batch: cut for each plan's share of the device, so a
batch of many small samples has fewer tasks than its plans alone; a batch of one
plan, and plans of a given length, keep the plan's own; the bins are those of
the plans alone, bit for bit on dyadic spins."""
import numpy as np
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [("sc", (8, 8, 8), 16, 40), ("sc", (7, 7, 7), 9, 24), ("bcc", (6, 6, 6), 20, 33), ("sc", (12, 12, 12), 16, 20),
          ("sc", (3, 2, 1), 4, 5)]


def _plan(S, kind, L, n_o, n_L, prec, **kw):
    pos = inputs.sc_positions(L) if kind == "sc" else inputs.bcc_positions(L)
    return S.Plan(pos, S.BINS_SC if kind == "sc" else S.BINS_BCC, n_o, n_L, prec, cells=L, **kw)


@pytest.mark.parametrize("prec", ["split_bf16", "fp32"])
def test_batch_cuts_for_its_share(prec):
    import torch
    from paper_2308_07487_amd import sdc as S
    assert torch.cuda.is_available()
    print(f"[case] batch segments {prec}", flush=True)
    plans = [_plan(S, *s, prec) for s in SHAPES * 6]
    alone = []
    for p in plans[:len(SHAPES)]:
        with S.Batch([p]) as b:
            alone.append(b.info()[0])
    fixed = _plan(S, *SHAPES[0], prec, segment_pairs=1)
    with S.Batch([fixed]) as b:
        fixed_tasks = b.info()[0]
    frames = [torch.from_numpy(inputs.dyadic_frames(s[2] + s[3] - 1, p.n_sites, 7 + k)).cuda()
              for k, (s, p) in enumerate(zip(SHAPES * 6, plans))]
    with S.Batch(plans + [fixed]) as b:
        assert b.info()[0] - fixed_tasks < 6 * sum(alone)
        b.accumulate(frames + [frames[0]])
        H = [p.raw()[0] for p in plans + [fixed]]
    for p, f, h in zip(plans, frames, H):
        p.reset()
        p.accumulate(f)
        np.testing.assert_array_equal(p.raw()[0], h)
    np.testing.assert_array_equal(H[0], H[-1])


def test_radial_batch():
    import torch
    from paper_2308_07487_amd import sdc as S
    print("[case] batch segments radial", flush=True)
    plans = [S.Plan(inputs.ball_positions(n, 4.0, n), S.BINS_RADIAL, 8, 20, n_shells=100, r_max=8.0)
             for n in (1000, 300, 700, 64, 1500, 1000, 900, 800)]
    frames = [torch.from_numpy(inputs.dyadic_frames(27, p.n_sites, 3)).cuda() for p in plans]
    with S.Batch(plans) as b:
        b.accumulate(frames)
        H = [p.raw()[0] for p in plans]
    for p, f, h in zip(plans, frames, H):
        p.reset()
        p.accumulate(f)
        np.testing.assert_array_equal(p.raw()[0], h)
