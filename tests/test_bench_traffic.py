"""bench.py reports recorded memory traffic only for the kernel sources it was taken on."""
import shutil

import pytest

import bench


@pytest.mark.parametrize("rec,name,old,new", [
    ("PULL_TRAFFIC", "pull_common.h", "__builtin_nontemporal_load(reinterpret_cast<const typename Vec<VEC>::type*>(p))",
     "*reinterpret_cast<const typename Vec<VEC>::type*>(p)"),          # another cache policy of the streams
    ("PULL_TRAFFIC", "pull_update.hip", "4 << 20", "8 << 20"),
    ("MC_TRAFFIC", "mc_grad.hip", "kBinRows = 128", "kBinRows = 64"),
])
def test_changed_kernel_code_retires_the_record(tmp_path, monkeypatch, rec, name, old, new):
    rec = getattr(bench, rec)
    csrc = tmp_path / "csrc"
    shutil.copytree(bench.CSRC, csrc)
    monkeypatch.setattr(bench, "CSRC", str(csrc))
    assert bench._traffic(rec, rec["key"]) == rec["bytes_per_launch"]
    text = (csrc / name).read_text()
    (csrc / name).write_text("// a comment\n" + text)
    assert bench._traffic(rec, rec["key"]) == rec["bytes_per_launch"]
    assert text.count(old) == 1
    (csrc / name).write_text(text.replace(old, new))
    assert bench._traffic(rec, rec["key"]) is None
