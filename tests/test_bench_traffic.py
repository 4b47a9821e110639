"""Which build a summary of byte counters belongs to (bench.py --summarise-pmc, traffic_stale): one written for the present kernel sources is
taken, one of other sources or with a field changed afterwards is not."""
import glob
import json
import os

import pytest

import bench


@pytest.fixture
def summary(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_2006_11735_amd" / "csrc"
    csrc.mkdir(parents=True)
    (tmp_path / "profiles").mkdir()
    (csrc / "a.hip").write_text("one")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    files = []
    for name, copied, conv in (("fetch", 131072, 500), ("write", 262144, 300)):
        files.append(str(tmp_path / (name + ".csv")))
        rows = [("icnn::stream_copy_kernel(int)", copied)] * 3 + [("icnn::avgpool_kernel(int)", 1)] * 2 + [("icnn::conv_x_kernel(int)", conv)] * 4
        with open(files[-1], "w") as f:
            f.write("Kernel_Name,Counter_Value\n" + "".join("%s,%d\n" % r for r in rows))
    bench.summarise_pmc("cfgx", *files)
    return csrc, tmp_path / "profiles" / "traffic_cfgx.json"


def test_a_summary_of_the_present_sources(summary):
    _csrc, path = summary
    assert bench.byte_counters(str(path)) == ((2 * 500 + 300) * 1024, False)      # the copies say that reads count half
    assert bench.byte_counters(str(path) + "x") == (None, None)


def test_a_summary_of_other_sources_whatever_its_digest_says(summary):
    csrc, path = summary
    (csrc / "a.hip").write_text("two")
    assert bench.byte_counters(str(path))[1] is True
    fields = json.loads(path.read_text())
    fields["csrc_digest"] = bench.csrc_digest()                                   # put right by hand: no counter was taken
    path.write_text(json.dumps(fields))
    assert bench.byte_counters(str(path))[1] is True


def test_the_stored_summaries_are_as_they_were_written():
    stored = glob.glob(os.path.join(bench.ROOT, "profiles", "traffic_*.json"))
    assert stored
    for path in stored:
        with open(path) as f:
            fields = json.load(f)
        assert fields["stamp"] == bench.summary_stamp(fields), path
