"""How stage 3 hands out its rows, on the host: which calls claim their last ones, against a count of the blocks one by
one; every row of the call in one XCD's share, enough workgroups for the claimed ones, and no call refused because it claims."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

from paper_2603_06274_amd import binding as sb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_06274_amd", "csrc")
NO_CLAIM = 0x7fffffff


@pytest.fixture(scope="module")
def grid_of(tmp_path_factory):
    """The host code with stand-ins for the launches: the library under test if it is such a build, else built here."""
    path = sb.library_path()
    if not hasattr(ctypes.CDLL(path), "stem_test_attention_grid"):
        if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
            pytest.skip("needs g++ and the HIP headers")
        path = str(tmp_path_factory.mktemp("grid") / "libstem_host.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(CSRC, "stem_api.cpp"),
                        os.path.join(ROOT, "tests", "host_launch_stubs.cpp"), "-o", path], check=True)
    fn = ctypes.CDLL(path).stem_test_attention_grid
    fn.argtypes = [ctypes.POINTER(sb.stem_shape)] + [ctypes.c_int32] * 3 + [ctypes.POINTER(ctypes.c_int64),
                                                                          ctypes.POINTER(ctypes.c_int32)]

    def call(hq, hkv, d, B, lens, kmax, chunk=None, units=256, queue=True):
        cu = [0]
        for n in lens:
            cu.append(cu[-1] + n)
        shape = sb.Shape(hq, hkv, d, B, cu, (d * hq, d), (d * hkv, d), chunk)
        out, asked = (ctypes.c_int64 * 13)(), ctypes.c_int32()
        assert fn(shape.ref(), kmax, units, int(queue), out, ctypes.byref(asked)) == sb.STEM_OK
        claims, m, items, claim_from, slots = out[:5]
        return dict(claims=bool(claims), m=m, items=items, claim_from=claim_from, slots=slots, rows=list(out[5:]),
                    asked=asked.value)
    return call


def block_rows(lens, B, chunk):
    """(rows, block index of each) of the call, one by one"""
    index = []
    for s, n in enumerate(lens):
        lo, hi = (chunk[0][s], chunk[1][s]) if chunk else (0, n)
        if hi > lo:
            index += range(lo // B, -(-hi // B))
    return index


def check(g, hq, hkv, d, B, lens, kmax, chunk, units, queue):
    index = block_rows(lens, B, chunk)
    ops = sum(min(kmax, i + 1) for i in index) * hq * 4.0 * d * B * B
    at_a_time = units * (128 // B if d == 256 else 256 // B)
    assert g["claims"] == (ops >= 1e12 and units > 0 and hq * len(index) >= 8 * at_a_time)
    assert (g["asked"] > 0) == (ops >= 1e12)           # a short call does not ask the device
    rows = [max(0, r) for r in g["rows"]]
    assert sum(rows) == hq * len(index) and max(rows) <= g["items"]
    if not (g["claims"] and queue):
        assert g["claim_from"] == NO_CLAIM and g["slots"] == g["items"]
        return
    assert 0 < g["claim_from"] <= g["items"]
    claimable = sum(max(0, r - g["claim_from"]) for r in rows)
    claimers = 8 * (g["slots"] - g["claim_from"])
    assert claimable <= claimers                       # who claims finds every row
    share = 4 if kmax > max(i + 1 for i in index) // 2 else 8
    assert g["items"] - g["claim_from"] == g["items"] // share


def test_grid_of_random_calls(grid_of):
    r = random.Random(5)
    claimed = 0
    for turn in range(1500):
        hkv = r.choice([1, 2, 3, 4, 5, 8, 16])
        hq = hkv * r.choice([1, 2, 4, 7])
        d, B, units = r.choice([64, 128, 256]), r.choice([64, 128]), r.choice([256, 256, 128, 0])
        lens = [r.choice([0, 1, B - 1, B, r.randint(1, 200 * B)]) for _ in range(r.choice([1, 1, 2, 5, 17]))]
        if r.random() < 0.5:
            lens[0] = r.randint(100, 1000) * B - r.randint(0, 5)
        chunk = None
        if r.random() < 0.4:
            starts = [B * r.randint(0, n // B) for n in lens]
            chunk = (starts, [n if r.random() < 0.7 else r.randint(a // B, n // B) * B for a, n in zip(starts, lens)])
        kmax = max(1, int(-(-max(lens) // B) * r.choice([0.05, 0.3, 0.5, 0.6, 1.0])))
        queue = r.random() < 0.8
        if not block_rows(lens, B, chunk):
            continue
        g = grid_of(hq, hkv, d, B, lens, kmax, chunk, units, queue)
        check(g, hq, hkv, d, B, lens, kmax, chunk, units, queue)
        claimed += g["claims"]
    assert claimed > 100


@pytest.mark.parametrize("B", [64, 128])
def test_calls_at_the_line(grid_of, B):
    """The lengths around which a dense call's operations reach the line: by one block of rows more or less."""
    d, hq, hkv = 128, 32, 8
    seen = []
    for nb in range(8 * 4, 400):
        g = grid_of(hq, hkv, d, B, [nb * B - 1], nb)
        check(g, hq, hkv, d, B, [nb * B - 1], nb, None, 256, True)
        seen.append(g["claims"])
    assert not seen[0] and seen[-1] and sorted(seen) == seen


def test_claiming_refuses_no_call(grid_of):
    """Rows that just fit one launch leave no room for workgroups beyond them: then none is claimed."""
    g = grid_of(2 ** 15 - 8, 8, 64, 64, [64 * 4096] * 16, 1)
    assert g["claims"] and g["slots"] * 8 <= 0x7fffffff and g["claim_from"] == NO_CLAIM
    assert sum(g["rows"]) == (2 ** 15 - 8) * 2 ** 16
    g = grid_of(2 ** 14, 8, 64, 64, [64 * 4096] * 16, 1)
    assert g["claims"] and g["slots"] * 8 <= 0x7fffffff and g["claim_from"] < NO_CLAIM
