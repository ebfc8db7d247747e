"""A batch of more fused tasks than 32-bit indices of half the range hold: the
default segments give plans up to three times the tasks of 96-pair ones, and
batches near 2^30 of those are accepted as before.  Created, not run."""
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu


def test_batch_of_1_2e9_tasks_is_accepted():
    import torch
    assert torch.cuda.is_available()
    from paper_2308_07487_amd import sdc as S
    print("[case] batch of 3 x sc 64x64x28, 1024 lags, one pair per task", flush=True)
    L = (64, 64, 28)
    pos = inputs.sc_positions(L)
    plans = [S.Plan(pos, S.BINS_SC, 1, 1024, "split_bf16", cells=L, segment_pairs=1) for _ in range(3)]
    with S.Batch(plans) as b:
        n_tasks, grid = b.info()
        assert n_tasks == 3 * (1792 * 1792) * 128 > 2 ** 30
        assert 8 <= grid <= 4096
    for p in plans:
        p.close()
