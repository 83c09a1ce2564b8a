"""The queue of weights that launches read ahead (csrc/read_queue.hpp), on the CPU: whatever the budgets and the room, the parts follow
each other in order of use, skip what has been launched, stay within the lead, and cover each byte at most once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "read_queue.hpp"
using namespace sd;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)
int main() {
    ReadAhead none;
    CHECK(none.take(1 << 20, 512, 8).wgs == 0);
    none.launched();
    CHECK(none.take(1 << 20, 512, 8).n == 0);
    unsigned s = 1;
    auto rnd = [&](unsigned n) { s = s * 1664525u + 1013904223u; return (s >> 8) % n; };
    for (int round = 0; round < 300; ++round) {
        ReadAhead q;
        // ranges laid out behind each other, so that a byte's address says where in the string it is
        const char* const base = reinterpret_cast<const char*>(1 << 20);
        uint64_t at = 0;
        std::vector<uint64_t> ends;
        const int launches = 1 + rnd(12);
        for (int l = 0; l < launches; ++l) {
            for (int i = rnd(7); i > 0; --i) {
                const uint64_t n = 16ull * rnd(round % 3 == 0 ? 64 : 2000000);
                q.add(base + at, n + rnd(16));       // a remainder below 16 bytes is left out
                at += n;
            }
            q.add(nullptr, 64);
            q.mark();
            ends.push_back(at);
        }
        CHECK(q.total == at);
        uint64_t read = 0, launched = 0;
        int calls = 0;
        for (int l = 0; l <= launches; ++l) {
            for (int k = rnd(4); k > 0; --k, ++calls) {
                const uint64_t budget = rnd(2) ? rnd(40) << 20 : rnd(100000);
                const long room = (long)rnd(700) - 50;
                const int loads = rnd(2) ? 8 : 16;
                const ReadRanges r = q.take(budget, room, loads);
                CHECK(r.n >= 0 && r.n <= ReadRanges::MAX);
                uint64_t got = 0;
                for (int i = 0; i < r.n; ++i) {
                    const uint64_t from = (uint64_t)((const char*)r.p[i] - base);
                    CHECK(r.bytes[i] > 0 && r.bytes[i] % 16 == 0 && r.start[i] == got);
                    CHECK(from == (read > launched ? read : launched));      // next in order, nothing twice, nothing that has run
                    read = from + r.bytes[i];
                    got += r.bytes[i];
                }
                CHECK(got == 0 || (got <= budget && room >= 16 && r.wgs <= room && read <= launched + ReadAhead::LEAD && read <= at));
                CHECK((uint64_t)r.wgs * loads * READ_AHEAD_STEP >= got && (r.wgs == 0) == (got == 0));
                CHECK(got == 0 || (uint64_t)(r.wgs - 1) * loads * READ_AHEAD_STEP < got);
            }
            q.launched();
            if (l < launches) launched = ends[l];
        }
    }
    std::printf("ok\n");
}
"""


def test_parts_follow_each_other_and_the_launches(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "queue.cpp", tmp_path / "queue"
    src.write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2407_02031_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, timeout=60).stdout.strip() == "ok"
