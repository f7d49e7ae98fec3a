"""GPU tests of the autotuner and cost-model boundary: the exhaustive choice
follows the selection rule on measured medians, the timing database is
reused, tuning never writes the caller's arrays, a cost model trained on
the GPU from the database is written, loaded and picks the argmin of its
predictions, a loop without a configuration runs the model's pick with
unchanged results, and a corrupt model file falls back to the tuner."""
import json

import numpy as np
import pytest

import oracle
from oracle import tuner as OT
from paper_2110_14340_amd import inputs, jacc, tuner
from gpu_util import context, say

pytestmark = pytest.mark.gpu


def test_tune_selection_rule_database_reuse_and_scratch_replicas(tmp_path):
    say("jacc_tune 130x258, K in {1,2,4}")
    shape = (130, 258)
    u0 = inputs.jacobi_grid(*shape, seed=31)
    db = str(tmp_path / "timings.db")
    u, v = u0.copy(), u0.copy()
    v[1:-1, 1:-1] = -1.0
    before = v.copy()
    with context(4) as c:
        c.enter(u, halo=(1, 1), K=2)
        c.enter(v, halo=(1, 1), K=2)
        best, cands, med = c.tune(u, v, ks=[1, 2, 4], db_path=db, reps=5)
        assert len(cands) == 3 * 70 and med.shape == (len(cands),) and np.all(med > 0)
        assert cands.index(best) == OT.select([[m] for m in med])
        lines = [ln for ln in open(db) if ln[0] not in "#@"]
        assert len(lines) == len(cands)
        best2, _, med2 = c.tune(u, v, ks=[1, 2, 4], db_path=db)  # served from the database
        assert best2 == best and np.array_equal(med2, med)
        c.exit(v)
        c.exit(u)
    assert np.array_equal(v, before)  # candidates ran on scratch replicas


def test_model_trained_from_database_file_pick_and_unconfigured_loop(tmp_path):
    say("cost model: tune 8 shapes, train, load, pick")
    db = str(tmp_path / "train.db")
    path = str(tmp_path / "model.bin")
    shapes = inputs.batch_shapes(40, 5, 3, side2d=(64, 600), side3d=(32, 64))
    with context(8) as c:
        for i, sh in enumerate(shapes):
            data = inputs.jacobi_grid(*sh, seed=i) if len(sh) == 2 else inputs.heat_field(*sh, seed=i)
            tuner.tune(c, sh, data, db_path=db, ks=[1, 2], reps=3)
        rep = c.model_train(db, path, members=2, epochs=60, seed=3, holdout=4)
        say(f"  {rep}")
        assert rep["signatures"] == len(shapes) and rep["loss_last"] < rep["loss_first"]
        assert rep["heldout_mse"] > 0
        c.model_load(path)
        for sh in ((300, 514), (40, 36, 66)):
            best, cands, pred = c.model_pick(sh, [1, 2])
            assert pred.shape == (len(cands),) and np.all(np.isfinite(pred))
            assert cands.index(best) == OT.argmin_predicted(pred)
        # a Jacobi loop with no configuration runs the model's eager pick
        u0 = inputs.jacobi_grid(300, 514, seed=5)
        a, b = u0.copy(), u0.copy()
        c.enter(a, halo=(1, 1), K=2)
        c.enter(b, halo=(1, 1), K=2)
        for t in range(4):
            (c.jacobi2d(a, b) if t % 2 == 0 else c.jacobi2d(b, a))
        c.exit(b)
        c.exit(a)
        assert np.array_equal(a, oracle.jacobi2d(u0, 4))
        # the file loads again in a fresh context and gives the same picks
        with context(2) as c2:
            c2.model_load(path)
            assert c2.model_pick((300, 514), [1, 2])[0] == c.model_pick((300, 514), [1, 2])[0]


def test_corrupt_model_falls_back_to_the_tuner(tmp_path):
    say("jacc_choose with a corrupt model file")
    bad = tmp_path / "bad.bin"
    bad.write_bytes(b"JACCCM01" + b"\0" * 64)
    u0 = inputs.jacobi_grid(66, 130, seed=32)
    u, v = u0.copy(), u0.copy()
    with context(2) as c:
        c.enter(u, halo=(1, 1))
        c.enter(v, halo=(1, 1))
        cand, src = c.choose(u, v, model_path=str(bad), ks=[1, 2], db_path=str(tmp_path / "t.db"), reps=3)
        assert src == jacc.CHOICE_TUNER and "model:" in c.last_error()
        assert cand in jacc.candidates((66, 130), [1, 2])
        cand, src = c.choose(u, v, model_path=str(bad), tune=False)
        assert src == jacc.CHOICE_DEFAULT and cand["K"] == 2


def _database(path, key, shape, K, ms, default_ms):
    """A timing database in which every candidate of the shape takes `ms`(index)
    and the library's defaults (the row with bx = 0) `default_ms`."""
    kind = jacc.stencil_kind(shape)
    e = list(shape) + [0] * (3 - len(shape))
    lines = [f"@ {key}"]
    for i, c in enumerate(jacc.candidates(shape, [K])):
        lines.append(" ".join(map(str, [kind, *e, K, c["bx"], c["by"], c["tile"], c["vec"], c["persistent"], c["rows"], 1,
                                        ms(i)])))
    if default_ms:
        lines.append(" ".join(map(str, [kind, *e, K, 0, 0, 0, 0, 0, 0, 1, default_ms])))
    path.write_text("\n".join(lines) + "\n")


def _record_of_one_sweep(shape, K, monkeypatch, tmp_path, model=None):
    log = tmp_path / "loops.jsonl"
    monkeypatch.setenv("JACC_LOG", str(log))
    u0 = inputs.jacobi_grid(*shape, seed=1)
    a, b = u0.copy(), u0.copy()
    with context(K) as c:
        if model:
            c.model_load(model)
        c.enter(a, halo=(1, 1))
        c.enter(b, halo=(1, 1))
        c.jacobi2d(a, b)
        c.exit(b)
    assert np.array_equal(b, oracle.jacobi2d(u0, 1))
    return json.loads(log.read_text().splitlines()[-1])["cfg"]


@pytest.mark.parametrize("shape", [(66, 131), (66, 130)])
@pytest.mark.parametrize("faster", ["defaults", "candidate"])
def test_exhaustive_tuning_runs_the_defaults_unless_a_candidate_is_faster(shape, faster, monkeypatch, tmp_path):
    """By recorded times: the defaults (two doubles a lane in rows of odd length
    too) where they are as fast as every candidate, else the fastest one."""
    say(f"tuned or default {shape} {faster}")
    db = tmp_path / "t.db"
    with context(1) as c:
        key = c.build_key()
    best = 17
    _database(db, key, shape, 1, lambda i: 1.0 if i == best else 2.0, 1.0 if faster == "defaults" else 1.5)
    monkeypatch.setenv("JACC_TUNE", "exhaustive")
    monkeypatch.setenv("JACC_TUNE_DB", str(db))
    cfg = _record_of_one_sweep(shape, 1, monkeypatch, tmp_path)
    want = jacc.candidates(shape, [1])[best]
    picked = all(cfg[k] == want[k] for k in ("bx", "by", "tile", "vec"))
    assert picked == (faster == "candidate")
    if faster == "defaults":
        assert cfg["vec"] == 2


def test_defaults_are_timed_and_recorded_once_and_no_training_row(monkeypatch, tmp_path):
    say("defaults in the timing database")
    db, shape = tmp_path / "t.db", (66, 131)
    with context(1) as c:
        key = c.build_key()
    _database(db, key, shape, 1, lambda i: 1.0, 0)
    n = len(jacc.candidates(shape, [1]))
    monkeypatch.setenv("JACC_TUNE", "exhaustive")
    monkeypatch.setenv("JACC_TUNE_DB", str(db))
    for _ in range(2):
        _record_of_one_sweep(shape, 1, monkeypatch, tmp_path)
        rows = [ln for ln in db.read_text().splitlines() if ln[0] not in "#@"]
        assert len(rows) == n + 1 and sum(ln.split()[5] == "0" for ln in rows) == 1
    monkeypatch.setenv("JACC_TUNE", "model")
    path = str(tmp_path / "model.bin")
    with context(1) as c:
        assert c.model_train(str(db), path, members=1, epochs=2)["rows"] == n
    # with the model attached, rows of odd length keep the defaults
    assert _record_of_one_sweep(shape, 1, monkeypatch, tmp_path, model=path)["vec"] == 2
