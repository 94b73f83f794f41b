"""Loop bounds the device code shares with the host (csrc/zf_device.hpp),
stepped on the CPU at chunk sizes up to the format's 2^32 - 1 bytes: every
loop ends, and a lane takes its share of the bytes once."""
import os
import struct
import subprocess

import numpy as np
import pytest

import oracle.zfo as zo
from paper_2602_08190_amd import zf

import helpers as H
from conftest import gpu_available

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_08190_amd", "csrc")
TOP = 2**32
SIZES = [1, 15, 16, 17, 63, 64, 1023, 1024, 1025, 65536, 100_003, TOP - 1040, TOP - 1025, TOP - 1024, TOP - 1008,
         TOP - 64, TOP - 63, TOP - 17, TOP - 16, TOP - 1]

# Arguments: first byte, end, lane: prints the lane's bytes and whether each was
# its own; or n, aligned, lane, "fill": prints the rounds of 64, the lane's 16-byte pieces
# and single bytes, and whether each index was its own and above the one before;
# a loop that goes back or past n ends with "again".
SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "zf_device.hpp"
int main(int argc, char **argv) {
    if (argc == 4) {
        const uint32_t a = uint32_t(std::strtoull(argv[1], nullptr, 10)), lane = uint32_t(std::atoi(argv[3]));
        const uint32_t b = uint32_t(std::strtoull(argv[2], nullptr, 10));
        unsigned long long next = a, bytes = 0;
        bool own = true;
        zf::lane_bytes(a, b, lane, [&](uint32_t i) {
            if (i < next || i >= b) {
                std::printf("again\n");
                std::exit(0);
            }
            own = own && (i - a) % 64 == lane;
            next = i + 1ull;
            bytes++;
        });
        std::printf("%llu %d\n", bytes, int(own));
        return 0;
    }
    const uint32_t n = uint32_t(std::strtoull(argv[1], nullptr, 10)), lane = uint32_t(std::atoi(argv[3]));
    const bool aligned = argv[2][0] == '1';
    const uint32_t m = aligned ? n & ~15u : 0u;
    unsigned long long next = 0, pieces = 0, bytes = 0;
    bool own = true;
    auto put = [&](uint32_t i, uint32_t len) {
        if (i < next || (unsigned long long)i + len > n) {
            std::printf("again\n");
            std::exit(0);
        }
        own = own && (len == 16 ? i % 1024 == 16 * lane : (i - m) % 64 == lane);
        next = (unsigned long long)i + len;
        (len == 16 ? pieces : bytes)++;
    };
    zf::fill_lane(n, aligned, lane, [&](uint32_t i) { put(i, 16); }, [&](uint32_t i) { put(i, 1); });
    std::printf("%u %llu %llu %d\n", zf::rounds_of(n, 64), pieces, bytes, int(own));
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("loops")
    src, exe = d / "loops.cpp", d / "loops"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                    "-o", str(exe), str(src)], check=True)
    return str(exe)


@pytest.mark.parametrize("n", SIZES)
def test_one_byte_fill_and_step_count(program, n):
    for aligned in (1, 0):
        m = n & ~15 if aligned else 0
        for lane in (0, 1, 14, 31, 63):
            got = subprocess.run([program, str(n), str(aligned), str(lane), "fill"], check=True, capture_output=True,
                                 text=True, timeout=60).stdout.split()
            want = [-(-n // 64), len(range(16 * lane, m, 1024)), len(range(m + lane, n, 64)), 1]
            assert got == [str(x) for x in want], (n, aligned, lane)


@pytest.mark.parametrize("a,b", [(0, 1), (0, 65), (8192, 16384), (TOP - 65536, TOP - 1), (TOP - 65536, TOP - 64),
                                 (TOP - 17, TOP - 1), (TOP - 1, TOP - 1), (1, TOP - 1)])
def test_bytes_of_a_plain_unit(program, a, b):
    for lane in (0, 1, 16, 62, 63):
        got = subprocess.run([program, str(a), str(b), str(lane)], check=True, capture_output=True, text=True,
                             timeout=60).stdout.split()
        assert got == [str(len(range(a + lane, b, 64))), "1"], lane


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("before", [0, 1])
def test_chunk_of_one_byte_of_4_gib(before):
    # the format's largest chunk, on and off the output's 16-byte grid
    import torch
    b = zo.encode(np.full(1000, 77, np.uint8), zo.ANS)
    c = zo.chunks(b)[0]
    s = bytes(b[c["comp_off"]:c["comp_off"] + c["comp_len"]])
    assert s[:8] == struct.pack("<II", 1000, 0)     # the size, no words
    sizes = [1] * before + [TOP - 1]
    print("one-byte chunks of", sizes, flush=True)
    col = zf.Column.from_bytes(H.container(zf.BYTES, [(struct.pack("<I", n) + s[4:], n, zf.ANS) for n in sizes]))
    plan = zf.Plan([col], device=0)
    img = zf.upload_image(plan, [col])
    out = torch.zeros(sum(sizes) + 16, dtype=torch.uint8, device="cuda")
    plan.decompress_async(img, img.numel(), [out])
    plan.sync()
    assert bool((out[:-16] == 77).all()) and not bool(out[-16:].any())
