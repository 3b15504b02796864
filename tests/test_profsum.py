"""The staleness guard of the recorded HBM traffic: a record is valid only
while every source of the projection kernels is the one it was taken on."""
import os
import shutil

import pytest

from paper_2609_12075_amd import build, profsum


def test_every_projection_source_is_hashed():
    files = profsum.projection_sources()
    gemms = [f for f in build.SOURCES if f.startswith("k_gemm")]
    assert gemms and set(gemms) <= set(files)
    for header in ("common.h", "gemm_epi.h", "gemm_kernels.h", "rownorm.h"):
        assert header in files
    assert not {"k_attn.hip", "k_elem.hip", "model.hip"} & set(files)


@pytest.mark.parametrize("name", profsum.projection_sources())
def test_an_edit_of_any_of_them_drops_the_record(name, tmp_path):
    csrc = tmp_path / "csrc"
    shutil.copytree(profsum.CSRC, csrc)
    before = profsum.source_hash(str(csrc))
    assert before == profsum.source_hash()
    with open(os.path.join(csrc, name), "a") as f:
        f.write("\n// edited\n")
    assert profsum.source_hash(str(csrc)) != before


def test_other_sources_leave_it(tmp_path):
    csrc = tmp_path / "csrc"
    shutil.copytree(profsum.CSRC, csrc)
    with open(os.path.join(csrc, "k_attn.hip"), "a") as f:
        f.write("\n// edited\n")
    assert profsum.source_hash(str(csrc)) == profsum.source_hash()
