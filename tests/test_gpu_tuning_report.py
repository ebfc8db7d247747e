"""What a plan reports as its tuning makes the same work list again, the tuner
times the default length under that name, and a tuning file that holds it gives
the default: the tasks of a batch of one plan are those of its streams."""
import pytest

from paper_2308_07487_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [("sc", (8, 8, 8), 32, 64), ("sc", (20, 20, 20), 16, 40), ("bcc", (7, 5, 3), 9, 18), ("radial", (1500, 100), 8, 12)]


def _make(S, kind, L, n_o, n_L, **tu):
    if kind == "radial":
        return S.Plan(inputs.ball_positions(L[0], 4.0, 3), S.BINS_RADIAL, n_o, n_L, n_shells=L[1], r_max=8.0, **tu)
    pos = inputs.sc_positions(L) if kind == "sc" else inputs.bcc_positions(L)
    return S.Plan(pos, S.BINS_SC if kind == "sc" else S.BINS_BCC, n_o, n_L, cells=L, **tu)


def _tasks(S, p):
    with S.Batch([p]) as b:
        return b.info()[0]


@pytest.mark.parametrize("kind,L,n_o,n_L", CASES, ids=[f"{c[0]}{c[1]}" for c in CASES])
def test_reported_tuning_makes_the_same_plan(kind, L, n_o, n_L):
    import torch
    from paper_2308_07487_amd import sdc as S
    assert torch.cuda.is_available()
    print(f"[case] tuning report {kind} {L}", flush=True)
    default = 1 << 20 if kind == "radial" else 96
    with _make(S, kind, L, n_o, n_L) as p:
        tu, seg, tasks = p.tuning, p.segment_pairs, _tasks(S, p)
    assert tu == {"schedule": "two_pass", "segment_pairs": default}
    assert 1 <= seg <= (64 if kind == "radial" else 32)
    with _make(S, kind, L, n_o, n_L, **tu) as p:
        assert (p.tuning, p.segment_pairs, _tasks(S, p)) == (tu, seg, tasks)
    # any other length is taken as it is
    for other in (1, 5, default - 1):
        with _make(S, kind, L, n_o, n_L, segment_pairs=other) as p:
            assert p.tuning["segment_pairs"] == other and p.segment_pairs <= other
            if other > seg:
                assert _tasks(S, p) <= tasks


def test_tuner_times_the_default_and_its_file_gives_it(tmp_path, monkeypatch):
    import torch
    from paper_2308_07487_amd import sdc as S
    assert torch.cuda.is_available()
    print("[case] tuner default sc 8^3", flush=True)
    L = (8, 8, 8)
    cache = tmp_path / "tuning.json"
    with _make(S, "sc", L, 32, 64) as p:
        seg, tasks = p.segment_pairs, _tasks(S, p)
    _, _, times = S.autotune(inputs.sc_positions(L), S.BINS_SC, 32, 64, cells=L)  # the built-in list
    assert ("two_pass", 96) in [(c["schedule"], c["segment_pairs"]) for c, _ in times]
    S.autotune(inputs.sc_positions(L), S.BINS_SC, 32, 64, cells=L, candidates=[("two_pass", 96)], cache_path=str(cache))
    monkeypatch.setenv("SDC_TUNING_FILE", str(cache))
    with _make(S, "sc", L, 32, 64) as p:
        assert p.tuning == {"schedule": "two_pass", "segment_pairs": 96}
        assert (p.segment_pairs, _tasks(S, p)) == (seg, tasks)
