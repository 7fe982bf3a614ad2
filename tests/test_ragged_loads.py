"""The loads of lines that start on any byte stay inside their operand, and what they fetch is the line: every
phase modulo four bytes and every remainder behind the whole units, on the host, in an operand of exactly its size."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_03675_amd", "csrc")

PROGRAM = r"""
#include "ragged.hpp"
#include <stdio.h>
#include <string.h>
#include <vector>
using namespace hdqt;
int main()
{
    for (uint32_t units = 1; units <= 2; ++units)
        for (uint32_t pitch = 32 * units; pitch <= 32 * units + 33; ++pitch)
            for (uint32_t rows = 1; rows <= 9; ++rows) {
                const uint32_t bytes = 32 * units, size = rows * pitch;
                std::vector<uint8_t> q(size);
                for (uint32_t i = 0; i < size; ++i) q[i] = (uint8_t)(37 * i + 11 * (i >> 8));
                auto word = [&](uint32_t at) {
                    if (at + 4 > size || at + 4 < 4) { printf("%u rows of %u: bytes %u to %u\n", rows, pitch, at, at + 4); return false; }
                    return true;
                };
                for (uint32_t line = 0; line < size; line += pitch) {
                    std::vector<uint32_t> w;      // the line's aligned dwords
                    for (uint32_t u = 0; u < units; ++u)
                        for (int half = 0; half < 2; ++half)
                            for (uint32_t i = 0; i < 4; ++i) {
                                const uint32_t at = ragged_at(line, half) + 32 * u + 4 * i;
                                if (!word(at)) return 1;
                                w.push_back(0);
                                memcpy(&w.back(), &q[at], 4);
                            }
                    if (!word(ragged_last_at(line, bytes))) return 1;
                    uint32_t last;
                    memcpy(&last, &q[ragged_last_at(line, bytes)], 4);
                    for (uint32_t i = 0; 4 * i < bytes; ++i) {
                        const bool end = 4 * i + 4 == bytes;
                        const uint32_t got = end ? last : (uint32_t)(((uint64_t)w[i + 1] << 32 | w[i]) >> 8 * (line & 3));
                        if (memcmp(&got, &q[line + 4 * i], 4)) { printf("%u rows of %u: dword %u\n", rows, pitch, i); return 1; }
                    }
                }
            }
    return 0;
}
"""


def test_ragged_loads_stay_in_their_operand(tmp_path):
    src, exe = tmp_path / "ragged.cpp", tmp_path / "ragged"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
