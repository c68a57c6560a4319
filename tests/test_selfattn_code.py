"""What the self-attention's kernel relies on in its compiled code (on the CPU: the library's own gfx950 code objects).

The ring's stages are written by copies that the wait counts of LDS reads do not see: a wave may pass the barrier in
front of such a copy only with all its reads back, by a wait that stands with the barrier and not by the chance that
something in front of it needed the data.

And up to 64 dims two workgroups of eight wavefronts are to share a CU, for which nothing in the source asks."""
import glob
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    """The code object that holds k_selfattn."""
    import paper_2501_04304_amd as dgq
    if not os.path.exists(dgq.LIB_PATH):
        from paper_2501_04304_amd import build
        build.build()
    tmp = str(tmp_path_factory.mktemp("code"))
    shutil.copy(dgq.LIB_PATH, tmp)
    subprocess.check_call([LLVM + "llvm-objdump", "--offloading", "libdgq.so"], cwd=tmp, stdout=subprocess.DEVNULL)
    for f in glob.glob(tmp + "/*gfx950"):
        if "k_selfattn" in subprocess.check_output([LLVM + "llvm-readelf", "-s", "-W", f], text=True):
            return f
    raise AssertionError("no code object holds k_selfattn")


def _kernels(code_object):
    """name -> its instructions, in the order of the listing"""
    text = subprocess.check_output([LLVM + "llvm-objdump", "-d", code_object], text=True)
    found, name = {}, None
    for line in text.splitlines():
        head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if head:
            name = head[1]
            if "k_selfattnI" in name:
                found[name] = []
        elif name in found and line.strip():
            found[name].append(line.split("//")[0].strip())
    assert len(found) == 22  # eleven widths, with and without the code dump
    return found


def test_barriers_wait_for_the_lds_reads(code_object):
    for name, code in _kernels(code_object).items():
        barriers = [i for i, text in enumerate(code) if text.startswith("s_barrier")]
        assert len(barriers) >= 3, name
        for i in barriers:
            # going up: a wait for every LDS operation before anything that goes to LDS or memory
            while not code[i - 1].startswith("s_waitcnt"):
                i -= 1
                assert not code[i].startswith(("ds_", "global_")), (name, code[i])
            assert "lgkmcnt(0)" in code[i - 1], (name, code[i - 1])


def test_registers_leave_room_for_two_workgroups(code_object):
    """512 registers to a SIMD, four wavefronts: at most 128 each, and nothing spilled."""
    notes = subprocess.check_output([LLVM + "llvm-readelf", "--notes", code_object], text=True)
    counts = {}
    for kernel in notes.split("- .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S*)", kernel)[1]
        width = re.search(r"k_selfattnINS0_4SCfgILi(\d+)ELb[01]EEELb0", name)
        assert "k_selfattnI" not in name or re.search(r"\.private_segment_fixed_size:\s+0\b", kernel), name
        if width and int(width[1]) <= 4:
            counts[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", kernel)[1]) + int(kernel.split()[0])
    assert len(counts) == 8 and max(counts.values()) <= 128, counts
