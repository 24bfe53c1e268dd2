"""HBM bytes per launch that bench.py reports from the committed counter summaries."""
import hashlib

import pytest

import bench

TABLE = """# HBM traffic

| kernel | dispatches | fetch MiB | write MiB | source | sha256[:16] |
|---|---|---|---|---|---|
| `k_two<3, 3>` | 5 | 9.000 | 1.000 | a.hip | {a} |
| `k_two<3, 0>` | 5 | 4.000 | 1.000 | a.hip | {a} |
| `k_rows<2>` [layer 2] | 25 | 3.000 | 314.000 | a.hip | {a} |
| `k_rows<2>` [layer 1] | 25 | 2.000 | 39.000 | a.hip | {a} |
| `k_old<3>` | 25 | 2.000 | 39.000 | a.hip | 0123456789abcdef |
"""


@pytest.fixture
def summary(tmp_path, monkeypatch):
    src = tmp_path / "paper_2605_22698_amd" / "csrc"
    src.mkdir(parents=True)
    (src / "a.hip").write_text("kernels")
    (tmp_path / "profiles").mkdir()
    sha = hashlib.sha256(b"kernels").hexdigest()[:16]
    (tmp_path / "profiles" / "s.md").write_text(TABLE.format(a=sha))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    return "s.md"


@pytest.mark.parametrize("kernel,layer,mib", [
    ("k_rows", 2, 317), ("k_rows<2>", 1, 41),      # the layer's own row
    ("k_rows", 3, None), ("k_rows", None, None),   # a kernel of several layers without a row for this one
    ("k_two<3, 3>", 1, 10), ("k_two<3, 0>", 2, 5), ("k_two", 2, None),  # which of the two is not said
    ("k_old", 1, None), ("k_none", 1, None)])      # source changed; not listed
def test_the_row_of_the_kernel_and_layer(summary, kernel, layer, mib):
    got = bench.measured_traffic(kernel, summary, layer)
    assert got == (None if mib is None else mib * 2 ** 20)


@pytest.mark.parametrize("summary", ["md_step_3000_hbm_traffic.md", "product_hbm_traffic.md", "coulomb_hbm_traffic.md",
                                     "scale_100k_hbm_traffic.md"])
def test_rows_of_several_layers_are_listed_by_layer(summary):
    # k_radial_rows runs the first layer's hidden rows and R, R' of every later layer
    for line in open(f"{bench.ROOT}/profiles/{summary}"):
        if "`k_radial_rows" in line:
            assert "] |" in line, line
