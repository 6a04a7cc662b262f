"""The tuner's score: candidates whose damage rounds are the same launches (128 nodes and up) count
them with one time, so the fastest explicit step wins among them; a smaller candidate's rounds,
shorter but of a lower degree, count by the work of a default round."""
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_tuner_counts_equal_rounds_equally(dtype):
    from paper_2606_23458_amd import tune_tiles
    p = w.small_plate(256, 128)
    rep = tune_tiles([p], dtype, candidates=[64, 128, 192, 256, 384, 512], reps=10)
    small, rows = rep["candidates"][0], rep["candidates"][1:]
    assert all(r["status"] == "PF_OK" for r in rep["candidates"])
    assert len({r["cg_round_us"] for r in rows}) == 1, rows
    assert rep["best"] == min(rows, key=lambda r: r["explicit_us"])["tile_nodes"], rep
    # a solve on 64-node tiles takes about twice as long on this plate (FP64: 407 us a step against 212)
    assert small["cg_round_us"] > rows[0]["cg_round_us"], rep
