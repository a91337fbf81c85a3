"""bench.py reports a measured HBM traffic figure only for the code it was measured on: a change of
anything that decides what a history-sum launch reads and writes must void the record, a change of a
comment or of another kernel must not."""
import os
import re
import shutil

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2505_19467_amd", "csrc")


@pytest.mark.parametrize("name,function,line,voids", [
    ("kbe_kernels.hip", "k_hist_pair", "m += 0;", True),
    ("kbe_kernels.hip", "hist_lgseg", "m += 0;", True),        # rows per block
    ("kbe_kernels.hip", "hist_waves", "m += 0;", True),        # wavefronts per block
    ("kbe_kernels.hip", "hist_tasks", "m += 0;", True),
    ("kbe_kernels.hip", "extras_block", "blk += 0;", True),    # the blocks that ride in the launch
    ("kbe_kernels.hip", "diag_block", "m += 0;", True),
    ("kbe_kernels.hip", "props_block", "blk += 0;", True),
    ("kbe_kernels.hip", "obs_block", "lds += 0;", True),
    ("kbe_kernels.hip", "collide", "m += 0;", True),           # the launch
    ("kbe_api.hip", "make_layout", "c += 0;", True),           # its column-sum slots
    ("kbe_api.hip", "collision_parts", "m += 0;", True),       # what rides in which pass
    ("kbe_api.hip", "one_step", "more |= false;", True),
    ("kbe_device.hpp", "hist_task", "m += 0;", True),
    ("kbe_kernels.hpp", "obs_in_pass", "int unused;", True),
    ("kbe_kernels.hip", "k_hist_pair", "// a comment", False),
    ("kbe_kernels.hip", "k_row", "m += 0;", False),            # another kernel
    ("kbe_api.hip", "kbe_timing", "enable += 0;", False),
])
def test_record_is_void_when_the_measured_code_changes(tmp_path, name, function, line, voids):
    for f in os.listdir(CSRC):
        shutil.copy(os.path.join(CSRC, f), tmp_path)
    before = bench._kernel_source_sha1(str(tmp_path))
    assert before == bench._kernel_source_sha1()
    text = (tmp_path / name).read_text()
    body = re.search(r"\b" + function + r"\((?:[^()]|\([^()]*\))*\)\s*(?:const\s*)?\{", text)
    assert body, f"{name} defines no {function}"
    (tmp_path / name).write_text(text[:body.end()] + "\n  " + line + "\n" + text[body.end():])
    assert (bench._kernel_source_sha1(str(tmp_path)) != before) == voids
