"""Recorded traffic counts only while every file that decides it is the one it
was taken on."""
import shutil
from pathlib import Path

import pytest

from paper_2411_06405_amd import profsum

CSRC = Path(profsum.__file__).resolve().parent / "csrc"


@pytest.mark.parametrize("kernel,file", [
    ("k_level", "hotruss_kernels.hip"), ("k_level", "hotruss_team.hip"), ("k_support", "hotruss_team.hip"),
    ("k_support", "hotruss_dev.h"), ("k_hx_edges", "hotruss_hindex.hip"), ("k_hx_paths", "hotruss_dev.h"),
])
def test_a_changed_source_makes_a_record_stale(tmp_path, kernel, file):
    for f in (*CSRC.glob("*.hip"), *CSRC.glob("*.h")):
        shutil.copy(f, tmp_path)
    sources = profsum.KERNEL_SOURCES[kernel]
    assert profsum.source_sha(sources, tmp_path) == profsum.source_sha(sources)
    with open(tmp_path / file, "a") as f:
        f.write("\n")
    assert profsum.source_sha(sources, tmp_path) != profsum.source_sha(sources)
