"""Chunk indices of pair offsets up to the largest that the binning admits (2^32 - 256
pairs), on the host: the same function the kernels use, compiled by g++."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def first_chunk(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("chunks")
    src = d / "c.cpp"
    src.write_text('#include "chunks.h"\n'
                   'extern "C" uint32_t first(uint32_t i, uint32_t chunk) { return gs::first_chunk(i, chunk); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2507_23006_amd", "csrc"), str(src), "-o", str(d / "c.so")], check=True)
    fn = ctypes.CDLL(str(d / "c.so")).first
    fn.restype, fn.argtypes = ctypes.c_uint32, [ctypes.c_uint32, ctypes.c_uint32]
    return fn


@pytest.mark.parametrize("chunk", [1, 256, 1000, 1024, 2048])
def test_first_chunk(first_chunk, chunk):
    last = 0xFFFFFF00
    for i in [0, 1, chunk - 1, chunk, chunk + 1, 2 ** 31, last - 2 * chunk, last - chunk, last - 1025, last - 1024,
              last - 1023, last - 769, last - 768, last - 767, last - 1]:
        assert first_chunk(i, chunk) == -(-i // chunk), i
