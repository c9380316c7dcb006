"""Profiler summaries keep a kernel's template arguments apart (the modes, and the single- and
several-view builds, are different kernels), on a database of counters made here."""
import sqlite3

import pytest

from paper_2605_31419_amd import profsum

ONE = "void tsr::k_train_fused<1, true>(tsr::ViewTable, float const*) [clone .kd]"
MANY = "void tsr::k_train_fused<1, false>(tsr::ViewTable, float const*) [clone .kd]"


@pytest.mark.parametrize("name,short", [(ONE, "k_train_fused<1,true>"), (MANY, "k_train_fused<1,false>"),
                                        ("void tsr::k_face_stats<4>(tsr::ViewTable)", "k_face_stats<4>"),
                                        ("tsr::k_scan_tiles(unsigned int*)", "k_scan_tiles"),
                                        ("__amd_rocclr_copyBuffer", "__amd_rocclr_copyBuffer")])
def test_short_names(name, short):
    assert profsum._short(name) == short


def _db(path, counter, rows):
    con = sqlite3.connect(path)
    con.execute("create table counters_collection (kernel_name text, counter_name text, value real)")
    copy = profsum.COPY_BYTES / 1024.0
    for name, value in [("__amd_rocclr_copyBuffer", copy)] + rows:
        con.execute("insert into counters_collection values (?, ?, ?)", (name, counter, value))
    con.commit()
    con.close()
    return str(path)


def test_traffic_of_one_instantiation(tmp_path):
    f = _db(tmp_path / "f.db", "FETCH_SIZE", [(ONE, 10.0), (ONE, 20.0), (MANY, 100.0)])
    w = _db(tmp_path / "w.db", "WRITE_SIZE", [(ONE, 1.0), (MANY, 7.0)])
    t = profsum.traffic(f, w, "k_train_fused<1,true>")
    assert t["kernel"] == "k_train_fused<1,true>" and (t["fetch_bytes"], t["write_bytes"]) == (15 * 1024, 1024)
    with pytest.raises(SystemExit, match="several kernels"):
        profsum.traffic(f, w, "k_train_fused")
    f = _db(tmp_path / "f1.db", "FETCH_SIZE", [(ONE, 10.0)])
    w = _db(tmp_path / "w1.db", "WRITE_SIZE", [(ONE, 1.0)])
    assert profsum.traffic(f, w, "k_train_fused")["kernel"] == "k_train_fused<1,true>"
