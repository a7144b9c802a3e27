"""The tuning table that a batch takes is the one in its file now (CPU only)."""
import json
import os

from paper_2607_05302_amd import tune


def write(path, classes):
    with open(path, "w") as f:
        json.dump({"classes": classes}, f)


def test_a_changed_table_is_read_whatever_its_time_and_size(tmp_path, monkeypatch):
    monkeypatch.setattr(tune, "HERE", str(tmp_path))
    os.makedirs(tmp_path / "tuning")
    path = tune.table_path(4, 4)
    assert tune.load_table(4, 4) is None
    write(path, [[14, 512, 8]])
    assert tune.load_table(4, 4) == [(14, 512, 8)]
    st = os.stat(path)
    write(path, [[15, 256, 4]])  # the same file and size, within the clock's tick
    os.utime(path, ns=(st.st_atime_ns, st.st_mtime_ns))
    assert tune.load_table(4, 4) == [(15, 256, 4)]
    got = tune.load_table(4, 4)
    got.append("the caller's own")
    assert tune.load_table(4, 4) == [(15, 256, 4)]
    write(path, [])
    assert tune.load_table(4, 4) == []
    open(path, "w").write("no table")
    assert tune.load_table(4, 4) is None
    os.remove(path)
    assert tune.load_table(4, 4) is None
