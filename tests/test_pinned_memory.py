"""Pinned memory that the library keeps (mmee_decode's short lists, the fronts' records) is remembered only
when both of its addresses were obtained: after a failed first use the next one starts over.  The helper is
compiled for the host with calls that fail on demand."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_failed_first_use_leaves_nothing_behind(tmp_path):
    exe = str(tmp_path / "pinned_memory")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", os.path.join(ROOT, "tests", "c_client", "pinned_memory.cpp"), "-o", exe], check=True)
    assert subprocess.run([exe], capture_output=True, text=True, check=True).stdout == "ok\n"


def test_kept_pinned_memory_goes_through_the_helper():
    """Of the addresses that hipHostGetDevicePointer gives, only the result records are handled elsewhere
    (ensure_slots: remembered by the number of slots, which is set last)."""
    text = open(os.path.join(ROOT, "paper_2604_03446_amd", "csrc", "mmee.hip")).read()
    callers = re.findall(r"hipHostGetDevicePointer\(([^;]*);", text)
    assert len(callers) == 2 and sum("final_map" in c for c in callers) == 1
