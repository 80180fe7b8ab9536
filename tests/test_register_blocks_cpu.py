"""The register-block kernels (ka_square.hip, ka_cube.hip) compiled for the CPU against the oracle,
with the threads of a workgroup run one after another from barrier to barrier: once in ascending
and once in descending order, so that of any two threads each runs first once in every
stretch between barriers.  A read that no barrier orders against another thread's write of the same
word, before or after it, then sees the wrong side in one of the two."""
import ctypes
import functools
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1710_05155_amd", "csrc")
HERE = os.path.join(ROOT, "tests", "cpu_workgroup")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)
    if cxx is None:
        pytest.skip("clang++ not found")   # the sources use its vector types
    out = tmp_path_factory.mktemp("blocks")
    sources = [os.path.join(HERE, "run.cpp")]
    for name in ("ka_square", "ka_cube"):
        with open(os.path.join(CSRC, name + ".hip")) as fh:
            text = fh.read()
        text = text.replace("extern __shared__ u64 sq_lds[];", "u64 *sq_lds = reinterpret_cast<u64 *>(cpu::dynamic_lds);")
        text = re.sub(r'asm volatile\("" : "\+[sv]"\(\S+\)\);', ";", text)   # names register files that are not here
        sources.append(str(out / (name + ".cpp")))
        with open(sources[-1], "w") as fh:
            fh.write(text)
    path = str(out / "libblocks.so")
    subprocess.run([cxx, "-x", "c++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wno-everything", "-I", HERE, "-I", CSRC,
                    *sources, "-o", path], check=True)
    return ctypes.CDLL(path)


@functools.lru_cache(maxsize=None)
def expected(oracle, d, L, W, m, noise, sweeps):
    """Packed occupations at the start, then occupations and moved-ever bits after the sweeps."""
    og = oracle.lattice(d, L)
    orc = oracle.Sim(og, m, og.N // 2, 11 + L, range(64 * W), shared=bool(noise))
    first = oracle.pack(orc.occ)
    orc.sweep(sweeps)
    return first, oracle.pack(orc.occ), oracle.pack(orc.moved)


def check(lib, oracle, d, L, W, m, noise, sweeps, given, tile_sweeps, order):
    first, occ, moved = expected(oracle, d, L, W, m, noise, sweeps)
    n, f = first.copy(), np.zeros_like(first)
    rc = lib.run_blocks(d, L, W, m, noise, ctypes.c_uint64(11 + L), 0, sweeps, given, tile_sweeps, order,
                        n.ctypes.data_as(ctypes.c_void_p), f.ctypes.data_as(ctypes.c_void_p))
    assert rc == 0
    assert np.array_equal(n, occ)
    assert np.array_equal(f, moved)


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("given", [0, 1])
@pytest.mark.parametrize("L,W,m,noise", [(16, 1, 5, 0), (16, 2, 3, 1), (20, 1, 5, 0)])
def test_cube(lib, oracle, L, W, m, noise, given, order):
    check(lib, oracle, 3, L, W, m, noise, 3, given, 0, order)


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("given", [0, 1])
@pytest.mark.parametrize("L,W,m,noise", [(4, 1, 3, 0), (12, 3, 2, 0), (32, 2, 3, 0), (36, 1, 3, 1), (68, 1, 3, 0)])
def test_square(lib, oracle, L, W, m, noise, given, order):
    check(lib, oracle, 2, L, W, m, noise, 5, given, 0, order)


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("given,tile_sweeps", [(0, 1), (1, 1), (1, 2), (1, 3)])
@pytest.mark.parametrize("L,W", [(92, 2), (100, 1)])
def test_tiles(lib, oracle, L, W, given, tile_sweeps, order):
    check(lib, oracle, 2, L, W, 3, 0, 7, given, tile_sweeps, order)
