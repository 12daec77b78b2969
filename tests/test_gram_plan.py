"""The bitmap route's cut (plan_gram), checked on the CPU: every (tile, stage) is counted once, fp32
parts stay within 2^24 transactions, and the reduction finds every part."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("gram") / "libgramcheck.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC",
                    os.path.join(ROOT, "paper_1102_1003_amd", "csrc", "plan.cpp"),
                    os.path.join(ROOT, "tests", "gram_check.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)

    def run(na, nb, tri, m, n_cu=256, pinned=0, max_ws=2**64 - 1):
        msg = ctypes.create_string_buffer(256)
        assert lib.gram_check(na, nb, int(tri), ctypes.c_uint32(m), n_cu, pinned, ctypes.c_uint64(max_ws), msg,
                              256) == 0, msg.value.decode()
    run.lib = lib
    return run


@pytest.mark.parametrize("pinned", [0, 64, 128, 256])
@pytest.mark.parametrize("m", [1, 511, 512, 513, 10_000, 1_000_003, 2**24 + 1, 2**32 - 1])
def test_cut(check, m, pinned):
    for n in (2, 63, 64, 65, 129, 257, 2000):
        if n < 300 or m < 2**24:
            check(n, n, True, m, pinned=pinned)
            check(n, 31, False, m, pinned=pinned)
    check(300, 1, False, m, n_cu=8, pinned=pinned)
    for max_ws in (0, 10_000, 200_000, 9_000_000):          # less scratch than the full cut takes
        check(200, 200, True, m, pinned=pinned, max_ws=max_ws)


@pytest.mark.parametrize("pinned", [0, 64, 128, 256])
def test_set(check, pinned):
    """Families of a joint launch: one, many small, small beside large, more than workgroups."""
    for fam in ([(2, 1)], [(64, 1000), (65, 513), (700, 100_000)], [(3000, 400_000), (16, 16)],
                [(4096, 2**20), (100, 100_000), (2, 2**32 - 1)], [(20, 5000)] * 1000):
        n = (ctypes.c_uint32 * len(fam))(*[f[0] for f in fam])
        m = (ctypes.c_uint32 * len(fam))(*[f[1] for f in fam])
        joint, groups, msg = ctypes.c_uint32(), ctypes.c_uint32(), ctypes.create_string_buffer(256)
        assert check.lib.gram_set_check(n, m, len(fam), 256, pinned, ctypes.byref(joint), ctypes.byref(groups), msg,
                                        256) == 0, (fam[:4], msg.value.decode())
        # a family that fills the chip for over 200 us goes alone
        alone = sum(f in fam for f in [(3000, 400_000), (4096, 2**20), (2, 2**32 - 1)])
        assert joint.value == (0 if pinned == 256 else len(fam) - alone)
