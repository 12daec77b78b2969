"""What the host computes before a launch, checked on the CPU.  Launch sizes at the far end of what the
calls take: a launch of 2^32 work-items or more is refused by the runtime, so every grid has to stay below
that, whatever the sizes.  And the expected times that choose how pairs are counted."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIMIT = 2**32


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("launch") / "liblaunchcheck.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC",
                    os.path.join(ROOT, "paper_1102_1003_amd", "csrc", "plan.cpp"),
                    os.path.join(ROOT, "tests", "launch_check.cpp"), "-o", out], check=True)
    L = ctypes.CDLL(out)
    for f in ("triple_bits_items", "gram_reduce_items", "bit_rows_items", "bit_ingest_items"):
        getattr(L, f).restype = ctypes.c_uint64
    L.txn_price.restype = ctypes.c_double
    return L


@pytest.mark.parametrize("m,count", [
    (1, 1), (512, 7), (10**6, 41_664), (10**6, 134_300_000), (10**7, 436 * 435 * 434 // 6),
    (10**7, 437 * 436 * 435 // 6), (2**32 - 1, 2**31), (1, 2**40),
])
def test_triples_from_bits(lib, m, count):
    covered = ctypes.c_int()
    items = lib.triple_bits_items(ctypes.c_uint64(count), ctypes.c_uint32(m), 256, ctypes.byref(covered))
    assert covered.value and 0 < items < LIMIT


@pytest.mark.parametrize("pinned", [0, 64, 128, 256])
@pytest.mark.parametrize("na,nb,m", [
    (2, 2, 1), (4096, 4096, 2**20), (185_088, 185_088, 100_000), (185_089, 185_089, 100_000),
    (370_000, 370_000, 300_000),                             # 2.7 * 10^11 bytes of counts
    (185_000, 360_000, 50_000), (16, 16_000_000, 512),       # rectangles
])
def test_parts_of_the_product(lib, na, nb, m, pinned):
    covered = ctypes.c_int()
    items = lib.gram_reduce_items(na, nb, int(na == nb), ctypes.c_uint32(m), 256, pinned, ctypes.byref(covered))
    assert covered.value and items < LIMIT


@pytest.mark.parametrize("rows,m", [(1, 1), (2**24 - 2, 512), (2**24 - 1, 512), (2**24, 512), (511, 2**32 - 1),
                                    (512, 2**32 - 1), (280_000_000, 512)])
def test_bit_rows(lib, rows, m):
    fits = ctypes.c_int()
    items = lib.bit_rows_items(ctypes.c_uint64(rows), ctypes.c_uint32(m), ctypes.byref(fits))
    assert bool(fits.value) == (items < LIMIT)


@pytest.mark.parametrize("m", [1, 10**6, 2**31, 2**32 - 8193, 2**32 - 8192, 2**32 - 512, 2**32 - 1])
@pytest.mark.parametrize("n", [1, 34, 1200, 2400, 4500, 10**6])
def test_transactions_through_bit_rows(lib, m, n):
    whole = ctypes.c_int()
    items = lib.bit_ingest_items(ctypes.c_uint32(m), n, 163_840, 256, ctypes.byref(whole))
    assert whole.value and items < LIMIT
    if m <= 10**6 and n <= 4500:
        assert items


# (n, m, density, long transactions, their items): measured by transactions and by slots (MI355X, us)
TXN_MEASURED = [
    ((8192, 2**20, 0.0005, 0, 0), 186, 4742), ((8192, 2**20, 0.0005, 1, 256), 214, 4700),
    ((8192, 2**20, 0.0005, 1, 1024), 382, 4722), ((8192, 2**20, 0.0005, 1, 4096), 2299, 4811),
    ((8192, 2**20, 0.0005, 1, 8192), 7198, 4924), ((8192, 2**20, 0.0005, 16, 1024), 1495, 4774),
    ((8192, 2**20, 0.0005, 16, 8192), 22_073, 5429), ((8192, 2**20, 0.0005, 200, 1024), 3525, 5863),
    ((4000, 2**20, 0.0005, 0, 0), 63, 1277), ((4000, 2**20, 0.0005, 1, 500), 116, 1317),
    ((4000, 2**20, 0.0005, 1, 4000), 949, 1378), ((16_000, 2**20, 0.0002, 0, 0), 245, 5976),
    ((16_000, 2**20, 0.0002, 1, 2000), 1469, 6012), ((16_000, 2**20, 0.0002, 1, 16_000), 53_718, 8045),
]


@pytest.mark.parametrize("shape,txn,slots", TXN_MEASURED)
def test_long_transactions_are_priced(lib, shape, txn, slots):
    """The faster of the two ways is the one that the expected time names, and it is within a factor of two."""
    n, m, p, longs, d = shape
    us = lib.txn_price(n, m, ctypes.c_double(p), longs, d)
    assert txn / 2 < us < txn * 2
    assert (us < slots) == (txn < slots)


@pytest.mark.parametrize("pinned", [0, 64, 128, 256])
@pytest.mark.parametrize("m", [1, 512, 513, 10_000, 1_000_003, 2**24 + 1, 2**32 - 1])
def test_product_without_scratch(lib, m, pinned):
    """Parts within fp32's whole numbers, and added wherever a tile is shared."""
    for n in (2, 64, 65, 257, 3000):
        if n < 300 or m < 2**24:
            assert lib.gram_add_check(n, n, 1, ctypes.c_uint32(m), 256, pinned) == 0
    assert lib.gram_add_check(300, 1, 0, ctypes.c_uint32(m), 8, pinned) == 0


# (slot bits, m, corrections, width classes, measured by slots, from bit rows): MI355X, us, a call and a wait
ROUTES_MEASURED = [
    (8, 10**7, 0, [(131072, 3)], 23, 42), (8, 10**7, 0, [(131072, 12)], 22, 42), (8, 10**7, 0, [(1048576, 3)], 21, 41),
    (8, 5 * 10**6, 0, [(65536, 32)], 25, 35), (8, 5 * 10**6, 0, [(65536, 64)], 188, 33),
    (8, 10**6, 0, [(8192, 10), (16384, 8), (32768, 18), (65536, 4)], 61, 25),
    (8, 10**4, 2, [(128, 38), (256, 9), (512, 5), (1024, 2), (2048, 1), (4096, 1)], 76, 19),
    (8, 10**5, 1, [(1024, 1), (2048, 2), (4096, 3), (8192, 8), (16384, 22), (32768, 4)], 69, 20),
    (8, 10**4, 0, [(128, 1600)], 28, 37), (8, 10**4, 0, [(128, 3000)], 39, 58), (8, 10**6, 0, [(8192, 3000)], 1010, 1359),
    (8, 10**6, 0, [(32768, 1600)], 1223, 461), (8, 10**5, 0, [(1024, 200)], 78, 24), (8, 10**6, 0, [(8192, 400)], 331, 76),
    (8, 10**5, 31640, [(2048, 3000)], 329, 183), (16, 10**7, 8, [(2048, 800)], 356, 1515),
    (16, 10**7, 0, [(512, 17), (1024, 9), (2048, 27), (4096, 47)], 34, 79),
    (16, 10**6, 1, [(128, 255), (256, 275), (512, 270)], 74, 172), (16, 10**5, 85, [(256, 1600)], 59, 84),
    (16, 10**6, 0, [(1024, 1), (16384, 2), (32768, 6), (65536, 3)], 216, 24),
    (16, 10**6, 0, [(1024, 5), (2048, 4), (4096, 2), (8192, 1)], 41, 23), (32, 10**7, 0, [(2048, 12)], 31, 42),
    (16, 10**6, 0, [(32768, 20), (65536, 36)], 1060, 24), (32, 10**5, 63, [(2048, 104), (4096, 148), (8192, 131)], 1260, 28),
]


@pytest.mark.parametrize("planes,m,corr,classes,slots,bits", ROUTES_MEASURED)
def test_slots_or_bits(lib, planes, m, corr, classes, slots, bits):
    """The way that the expected times name is the faster one, where the two are a fifth apart."""
    r = (ctypes.c_uint32 * len(classes))(*[c[0] for c in classes])
    n = (ctypes.c_uint32 * len(classes))(*[c[1] for c in classes])
    by_slots, by_bits = ctypes.c_double(), ctypes.c_double()
    lib.route_prices(r, n, len(classes), planes, ctypes.c_uint32(m), corr, ctypes.byref(by_slots), ctypes.byref(by_bits))
    assert (by_slots.value <= by_bits.value) == (slots < bits), (by_slots.value, by_bits.value)
