"""CPU-only check of where several workgroups share a factor's lambda_max estimate: they wait for each other, so all of them have to
find room at once.  The rule of the kernel's own header, compiled for the host."""
import ctypes
import subprocess

import paper_2605_16184_amd.build as build

SOURCE = r"""
#include "root_factor.h"
extern "C" int members(int n) { return asteria::lanczos_members(n); }
extern "C" int room(int n, int cus) { return asteria::lanczos_cluster_room(n, cus) ? 1 : 0; }
"""


def test_workgroups_that_wait_for_each_other_find_room(tmp_path):
    src, lib = str(tmp_path / "room.hip"), str(tmp_path / "room.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-host-only", "-shared", "-I", build.CSRC, src, "-o", lib], check=True,
                   capture_output=True)
    rule = ctypes.CDLL(lib)
    most = 0
    for n in range(1, 2049):
        assert rule.members(n) >= most                          # so the largest factor of a batch decides
        most = rule.members(n)
        assert rule.room(n, 256)
        for cus in (0, 1, 8, 32, 64, 128):
            # the frontier of four calls and one workgroup that gets on
            assert not rule.room(n, cus) or 4 * (most - 1) + 1 <= cus
    assert most == 43
    assert not rule.room(2049, 256)
    assert [rule.room(n, 32) for n in (257, 768, 769, 2048)] == [1, 1, 0, 0]
