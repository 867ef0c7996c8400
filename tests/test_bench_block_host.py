"""Counter summaries of the block kernel are keyed by the sources it is built
from: its own header besides the marching kernels', whose summaries an edit of
that header leaves valid."""
import os
import shutil
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

BLOCK = {"kernel": 3, "tile_x": 32, "tile_y": 8, "tile_z": 4, "graph_steps": 0}
ROWS = {"kernel": 3, "tile_x": 64, "tile_y": 8, "tile_z": 64, "graph_steps": 0}


@pytest.fixture()
def tree(tmp_path, monkeypatch):
    """A copy of the kernel sources, with summaries of this code for a block
    and a marching plan of the force model and a block plan of the other."""
    csrc = tmp_path / "paper_1202_4748_amd" / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_1202_4748_amd", "csrc"), csrc)
    prof = tmp_path / "profiles"
    prof.mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    eq = bench.sources_of("k_block", bench.PAPER_MODEL_SOURCES["eq"])
    for kernel, workload, plan, names, unit in (
            ("k_block", "w_fp32", "rows:32:8:4:0", bench.sources_of("k_block"), "launch"),
            ("k_fused_staged", "w_fp32", "rows:64:8:64:0", bench.sources_of("k_fused_staged"), "launch"),
            ("k_block", "w_eq", "rows:32:8:2:0", eq, "step")):
        key = bench.kernel_source_hash(names=names)
        (prof / f"traffic_{kernel}_{workload}.md").write_text(
            f"plan {plan}\ntraffic_bytes_per_{unit}: 2.5e+07\nsource_hash: {key}\n")
        (prof / f"valu_{kernel}_{workload}.md").write_text(f"plan {plan}\nvalu_busy: 0.5\nsource_hash: {key}\n")
    return csrc


def _read():
    eq_plan = dict(BLOCK, tile_z=2)
    eq = bench.sources_of("k_block", bench.PAPER_MODEL_SOURCES["eq"])
    return [bench.read_traffic("k_block", "w", "fp32", BLOCK), bench.read_step_traffic("eq", "w_eq", ("k_block",), eq_plan),
            bench.read_valu_busy("k_block", "w_fp32", bench.sources_of("k_block"), BLOCK),
            bench.read_valu_busy("k_block", "w_eq", eq, eq_plan),
            bench.read_traffic("k_fused_staged", "w", "fp32", ROWS),
            bench.read_valu_busy("k_fused_staged", "w_fp32", bench.sources_of("k_fused_staged"), ROWS)]


def test_an_edit_of_the_block_kernel_voids_its_summaries_alone(tree):
    assert _read() == [2.5e7, 2.5e7, 0.5, 0.5, 2.5e7, 0.5]
    p = tree / "lbfss_block.hpp"
    p.write_text(p.read_text() + "\n// a remark\n")
    assert _read() == [2.5e7, 2.5e7, 0.5, 0.5, 2.5e7, 0.5]
    p.write_text(p.read_text() + "\ninline int lbfss_edit() { return 1; }\n")
    assert _read() == [None, None, None, None, 2.5e7, 0.5]
