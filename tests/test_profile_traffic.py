"""The traffic summary names every kernel once."""
import re

from paper_1603_06188_amd import profile_traffic


def _csv(path, counter, rows):
    path.write_text("Kernel_Name,Grid_Size,Counter_Name,Counter_Value\n" +
                    "".join(f'"{name}",{grid},{counter},{value}\n' for name, grid, value in rows))


def test_instantiations_of_one_kernel(tmp_path):
    rows = [("__amd_rocclr_copyBuffer", 4096, 131072.0)]
    rows += [("void apic::k_bin_records<3, true>(apic::BinLists)", 64, 300.0)] * 2
    rows += [("void apic::k_bin_records<3, false>(apic::BinLists)", 64, 100.0)] * 5
    rows += [("void apic::k_p2g<float, 3, 2, false, false>(apic::Parts<float>)", 64, 50.0)] * 5
    _csv(tmp_path / "f.csv", "FETCH_SIZE", rows)
    _csv(tmp_path / "w.csv", "WRITE_SIZE", rows)
    out = tmp_path / "out.txt"
    profile_traffic.main(["x", str(tmp_path / "f.csv"), str(tmp_path / "w.csv"), str(out), "command"])
    keys = re.findall(r"^(k_\w+)_fetch_bytes:", out.read_text(), re.M)
    assert sorted(keys) == ["k_bin_records", "k_bin_records_3_true", "k_p2g"]
    values = profile_traffic.read_summary(str(out))
    assert values["k_bin_records_fetch_bytes"] == str(100 * 1024 * 2)
    assert values["k_bin_records_3_true_fetch_bytes"] == str(300 * 1024 * 2)
