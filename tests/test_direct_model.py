"""The model that decides between copying operands off the 16-byte grid and reading them where they lie (no GPU): the C++ formula equals
the Python one, the committed constants are what the fit gives on the committed timings, and the built library's choices on those
timings are not slower than the copies."""
import numpy as np
import pytest

import paper_2512_02551_amd as hg
from paper_2512_02551_amd import direct_model as dm


@pytest.fixture(scope="module")
def timings():
    return dm.load([dm.DATA])


def test_cpp_prediction_equals_python_prediction(timings):
    tiles, _ = dm.read_inc()
    for r in timings[0][::7]:
        for bm, bn, sk, fr, _ in r["direct"][::3]:
            x, per, eff, mib = dm.features(r["shape"], bm, bn, sk)
            spec = f"mfma,{dm.TILES[bm, bn]},sk={sk},gm=8{',fr=1' if fr else ''},di=1"
            assert hg.predict_us(*r["shape"], spec) == pytest.approx(float(dm.predict_us(tiles[bm, bn], x, per, eff, mib, fr)), rel=1e-9), (r["shape"], spec)


def test_committed_constants_are_the_fit(timings):
    tiles, copies, late, errors = dm.fit(*timings)
    committed, committed_copies = dm.read_inc()
    assert max(e for _, e in errors.values()) < 0.12
    for t in dm.TILES:
        assert np.allclose(committed[t], [*tiles[t], late[t]], atol=2e-3), t
    assert np.allclose(committed_copies, copies, atol=2e-3)


def test_reading_in_place_is_chosen_where_it_is_not_slower(timings):
    """Every problem of the committed timings that the library reads in place (a third random, the others where it was in doubt): one in
    a hundred slower than the copies from HBM by more than 3 %, fewer from the cache, next to none by both."""
    chosen = np.array([[r["copies"][1] / r["direct"][1], r["copies"][2] / r["direct"][2]] for r in timings[1]
                       if ",di=1" in hg.plan_choice(*r["shape"], hg.Layouts.make(r["tn"], *r["ld"]))])
    assert len(chosen) > 5500
    assert (chosen[:, 0] < 0.97).mean() < 0.011 and (chosen[:, 1] < 0.97).mean() < 0.002
    assert (np.sqrt(chosen[:, 0] * chosen[:, 1]) < 0.97).mean() < 0.003
    assert np.exp(np.log(chosen).mean(axis=0)).min() > 1.35
