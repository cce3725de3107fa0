"""Host-side checks of bench.py: figures that it reads from committed profiles are those of the kernels
that the library launches now."""
import re

import pytest

import bench
from paper_2509_01085_amd import binding as B


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_keep", [16, 32, 64])
@pytest.mark.parametrize("walk", [True, False])
def test_named_kernels_are_in_the_library(d, n_keep, walk):
    code = open(B._LIB_PATH, "rb").read()
    for name, args in bench.kernel_instances(d, n_keep, walk).items():
        vals = [{"true": "Lb1E", "false": "Lb0E"}.get(a, f"Li{a}E") for a in args.strip("<>").split(", ")]
        assert f"{len(name)}{name}I{''.join(vals)}E".encode() in code, name + args


def test_traffic_of_another_instance_is_not_reported(tmp_path):
    (tmp_path / "profiles").mkdir()
    row = "| `bsa::{}` | 10.0 | 2.5 |\n"
    (tmp_path / "profiles" / "bench_x.md").write_text(
        row.format("k<9>") + "## Traffic\n\n" + row.format("k<128, 1, false>") + row.format("other<1>"))
    assert bench.measured_traffic_bytes("x", "k<128, 1, false>", str(tmp_path)) == 12.5e6
    assert bench.measured_traffic_bytes("x", "k<128, false>", str(tmp_path)) is None
    assert bench.measured_traffic_bytes("x", "k<9>", str(tmp_path)) is None  # listed, but not under Traffic
    assert bench.measured_traffic_bytes("absent", "k<9>", str(tmp_path)) is None


@pytest.mark.parametrize("workload", ["wan1p3b", "hd720p"])
def test_committed_traffic_tables_hold_no_removed_attention_kernel(workload):
    text = open(f"{bench.ROOT}/profiles/bench_{workload}.md").read().split("## Traffic", 1)[1]
    code = open(B._LIB_PATH, "rb").read()
    for name, args in re.findall(r"^\| `bsa::(\w+)<([^`]*)>`", text, re.M):
        vals = [{"true": "Lb1E", "false": "Lb0E"}.get(a, f"Li{a}E") for a in args.split(", ")]
        assert f"{len(name)}{name}I{''.join(vals)}E".encode() in code, f"{name}<{args}>"
