"""What the compiler made of the kernels, read from the metadata of the library that was built."""

import os
import subprocess

import pytest
import yaml

import paper_2602_16994_amd as mpv

LLVM = "/opt/rocm/llvm/bin"


def kernels_of(library, tmp_path):
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={bundle}", library, str(tmp_path / "copy.so")], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle", f"--input={bundle}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--output={code}"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    text = notes[notes.index("---"):notes.index("\n...")]
    return {k[".name"]: k for k in yaml.safe_load(text)["amdhsa.kernels"]}


@pytest.mark.skipif(not os.path.exists(f"{LLVM}/clang-offload-bundler"), reason="no LLVM tools of ROCm")
def test_the_task_kernels_keep_their_registers(tmp_path):
    """Three workgroups per compute unit (168 registers a lane), and next to nothing in private memory: what the functions that
    are not inlined save when they are entered, and a handful of numbers that a task loop keeps outside its sweeps."""
    task_kernels = {n: k for n, k in kernels_of(mpv.lib_path(), tmp_path).items() if "node_task_kernel" in n}
    assert len(task_kernels) == 6
    for name, k in task_kernels.items():
        assert k[".vgpr_count"] <= 168, name
        assert k[".vgpr_spill_count"] <= 5 and k[".private_segment_fixed_size"] <= 48, name


@pytest.mark.skipif(not os.path.exists(f"{LLVM}/clang-offload-bundler"), reason="no LLVM tools of ROCm")
def test_so_do_the_kernels_for_short_parts(tmp_path):
    short = {n: k for n, k in kernels_of(mpv.lib_path(), tmp_path).items() if "short_part_kernel" in n}
    assert len(short) == 2
    for name, k in short.items():
        assert k[".vgpr_count"] <= 168, name
        assert k[".vgpr_spill_count"] <= 5 and k[".private_segment_fixed_size"] <= 48, name


@pytest.mark.skipif(not os.path.exists(f"{LLVM}/clang-offload-bundler"), reason="no LLVM tools of ROCm")
@pytest.mark.parametrize("kernel", ["walk_kernel", "staged_part_kernel"])
def test_so_do_the_kernels_of_walks_and_of_short_parts_without_draws(tmp_path, kernel):
    """(Estimates and debug outputs run without the code of the draws, walks without that of the estimates.)"""
    found = {n: k for n, k in kernels_of(mpv.lib_path(), tmp_path).items() if kernel in n}
    assert len(found) == 2
    for name, k in found.items():
        assert k[".vgpr_count"] <= 168, name
        assert k[".vgpr_spill_count"] <= 5 and k[".private_segment_fixed_size"] <= 48, name


def test_rows_that_go_straight_to_lds_are_waited_for_before_they_are_read():
    """The compiler does not tie a read of LDS to the load that brings the row there: the source waits in between, and not only
    by what other loads there happen to need."""
    with open(os.path.join(os.path.dirname(mpv.lib_path()), "csrc", "mpv_device.h")) as f:
        text = f.read()
    for function, ask, read in (("void weigh_row(", "ask_row(", "row_vector("), ("void first_pass(", "first_pass(", "lt[")):
        body = text[text.index(function):]
        body = body[:body.index("\n    }\n")]
        before = body[body.index(ask):body.index(read)]
        assert "!there) asm volatile(\"s_waitcnt vmcnt(0)\"" in before, function
