"""The profile summary attributes counters to the kernel instance they were
taken on: another tile shape of the same pass is another kernel."""
import sqlite3

import pytest

from paper_2003_07504_amd import rocprof_summary as R

K13 = "void ilsk::k_row<30, 32, 13, {}, 0>(ilsk::WorkList)"
K17 = "void ilsk::k_row<30, 32, 17, {}, 0>(ilsk::WorkList)"
COL = "void ilsk::k_col<30, 36, 16>(ilsk::WorkList)"


def test_counters_of_another_shape_are_not_taken():
    kt = {"row_mid": (K13.format(1), 30, 24.0, 23.0, 25.0)}
    assert R.by_kind({K17.format(1): {"SQ_WAVES": 2550.0}}, kt, "row_mid") == {}
    assert R.by_kind({K13.format(1): {"SQ_WAVES": 2040.0}, K17.format(1): {"SQ_WAVES": 2550.0}}, kt,
                     "row_mid") == {"SQ_WAVES": 2040.0}
    assert R.by_kind({K13.format(1): {"SQ_WAVES": 2040.0}}, kt, "column") == {}


def _db(path, kernels, counter, row_shape):
    con = sqlite3.connect(path)
    con.execute("create table kernels (name, start, end, duration)")
    con.execute("create table counters_collection (kernel_name, counter_name, value)")
    for i, (name, us) in enumerate(kernels):
        con.execute("insert into kernels values (?, ?, ?, ?)", (name, 100000 * i, 100000 * i + us * 1000, us * 1000))
    for m in range(3):
        con.execute("insert into counters_collection values (?, ?, 1000.0)", (row_shape.format(m), counter))
    con.execute("insert into counters_collection values (?, ?, 2000.0)", (COL, counter))
    con.execute("insert into counters_collection values (?, ?, 524288.0)", ("__amd_rocclr_copyBuffer", counter))
    con.commit()
    con.close()


@pytest.mark.parametrize("same", [True, False])
def test_summary_refuses_runs_of_different_shapes(tmp_path, monkeypatch, same):
    seq = [(K13.format(0), 20), (COL, 16), (K13.format(1), 24), (COL, 16), (K13.format(2), 11)]
    _db(tmp_path / "kt.db", seq, "none", K13)
    _db(tmp_path / "fe.db", [], "FETCH_SIZE", K13 if same else K17)
    _db(tmp_path / "wr.db", [], "WRITE_SIZE", K13)
    out = tmp_path / "o.txt"
    monkeypatch.setattr("sys.argv", ["x", "--trace", str(tmp_path / "kt.db"), "--fetch", str(tmp_path / "fe.db"),
                                     "--write", str(tmp_path / "wr.db"), "--size", "1080x1920x3", "--iters", "2",
                                     "--shapes", "2,0", "--command", "c", "--out", str(out),
                                     "--traffic", str(tmp_path / "t.json")])
    if same:
        R.main()
        assert "row, column shape 2,0" in out.read_text()
        assert '"shapes": [\n   2,\n   0\n  ]' in (tmp_path / "t.json").read_text()
    else:
        with pytest.raises(SystemExit):
            R.main()
        assert not out.exists()
