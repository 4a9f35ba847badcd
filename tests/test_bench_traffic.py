"""bench.py divides counted traffic by a kernel's time only while the counters are of the kernel's present source."""
import shutil

import bench


def test_traffic_belongs_to_the_present_source(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_1909_04823_amd" / "csrc"
    shutil.copytree(bench.ROOT + "/paper_1909_04823_amd/csrc", csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    (tmp_path / "profiles").mkdir()
    profile = tmp_path / "profiles" / "deepfm_hbm_traffic.md"
    table = "| `k_a` | sort_scatter | 2.0 | 1.5 | 9 |\n| `k_b` | sort_scatter | 0.5 | 0.0 | 9 |\n| `k_c` | forward_gather_pool | 7 | 1 | 9 |\n"
    profile.write_text("Measured at commit: `abc`\n\n" + table)
    assert bench.measured_traffic(2, "sort_scatter") == (None, "abc")          # nothing says which source was counted
    profile.write_text(f"Measured at commit: `abc`\n\nSource `des_sort.hip`: `{bench.source_digest('des_sort.hip')}`\n" + table)
    assert bench.measured_traffic(2, "sort_scatter") == (4000000, "abc")
    assert bench.measured_traffic(2, "forward_gather_pool") == (None, "abc")
    assert bench.measured_traffic(3, "sort_scatter") == (None, None)
    source = csrc / "des_sort.hip"
    source.write_text("// a remark /* of no consequence\n" + source.read_text().replace("namespace des {", "namespace des   {  // more", 1))
    assert bench.measured_traffic(2, "sort_scatter") == (4000000, "abc")
    source.write_text(source.read_text().replace("kCopies = 4", "kCopies = 8", 1))
    assert bench.measured_traffic(2, "sort_scatter") == (None, "abc")
