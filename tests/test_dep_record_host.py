"""Dependency records (csrc/dep_record.hpp) on the CPU: the functions that the kernels call, over plain memory, in every
order that a launch, a reader that gives up and the replays after it can take."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <vector>
#include "dep_record.hpp"
using namespace sd;
struct HostMem {
    static uint64_t load64(const uint64_t* p) { return *p; }
    static void store64(uint64_t* p, uint64_t v) { *p = v; }
    static void store32(int32_t* p, int32_t v) { *p = v; }
    static int32_t add32(int32_t* p, int32_t v) { int32_t o = *p; *p = o + v; return o; }
};
typedef DepRecord<HostMem> D;
enum Look { WAIT, READY, GIVEN_UP };
static Look look(const uint64_t* rec, int need, uint64_t nonce) {
    bool all = true, any = false;
    for (int lane = 0; lane < 64; ++lane) {
        const uint64_t v = HostMem::load64(rec + dep_record_word(lane, need));
        all = all && dep_record_ready(lane, need, v, nonce);
        any = any || dep_record_given_up(lane, need, v, nonce);
    }
    return all ? READY : any ? GIVEN_UP : WAIT;
}
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)

// One launch.  Steps 0 .. need-1 are the producers, need .. need+readers-1 the readers, in the given order; a reader whose
// turn comes before the record is ready gives up if `impatient`, else it is taken again at the end.  Returns how many readers
// believed the record; *stale: one of them did so before every producer of this launch had published.
static int launch(uint64_t* rec, uint64_t nonce, int need, int readers, std::vector<int> order, bool impatient, bool* stale) {
    int published = 0, believed = 0;
    std::vector<int> later;
    auto reader = [&](bool last) {
        const Look l = look(rec, need, nonce);
        if (l == WAIT && !impatient && !last) return false;
        CHECK(l != WAIT || impatient);
        if (l == READY) {
            ++believed;
            if (published < need) *stale = true;
        } else {
            D::give_up(rec, nonce);
        }
        if (D::leave(rec) == readers - 1) D::clear(rec);
        return true;
    };
    for (int s : order) {
        if (s < need) {
            D::open(rec, s);
            D::publish(rec, s, nonce);
            ++published;
        } else if (!reader(false)) {
            later.push_back(s);
        }
    }
    for (size_t i = 0; i < later.size(); ++i) reader(true);
    return believed;
}

int main() {
    const uint64_t a = 0x123456789abcdef1ull, b = 0x9e3779b97f4a7c15ull;
    const uint64_t contents[3] = {0, ~0ull, 0x0000000500000003ull};
    long launches = 0;
    for (int need = 1; need <= DEP_PRODUCERS; ++need)
        for (int readers = 1; readers <= 3; ++readers) {
            std::vector<int> order(need + readers);
            for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
            const std::vector<int> usual = order;
            do {
                for (uint64_t was : contents) {
                    uint64_t rec[DEP_RECORD / 8];
                    // patient readers: everybody believes, nobody early, and replays the same
                    std::fill(rec, rec + 4, was);
                    bool stale = false;
                    for (int replay = 0; replay < 3; ++replay, ++launches) CHECK(launch(rec, a, need, readers, order, false, &stale) == readers && !stale);
                    CHECK(rec[0] != a && rec[1] != a);
                    // impatient ones: whatever this launch leaves behind, no reader of a replay believes it too early
                    for (bool again : {true, false}) {
                        std::fill(rec, rec + 4, was);
                        stale = false;
                        const int first = launch(rec, a, need, readers, order, true, &stale);
                        CHECK(!stale);
                        std::vector<int> early(usual);               // readers ahead of their producers
                        std::reverse(early.begin(), early.end());
                        for (int replay = 0; replay < 3; ++replay, ++launches) launch(rec, a, need, readers, again ? order : early, true, &stale);
                        CHECK(!stale);
                        // a replay with patient readers ends: ready, or given up at once
                        if (first < readers) CHECK(launch(rec, a, need, readers, usual, false, &stale) < readers && !stale);
                        // another launch, and the same one on cleared memory, are not held up
                        CHECK(launch(rec, b, need, readers, usual, false, &stale) == readers && !stale);
                        std::fill(rec, rec + 4, 0);
                        CHECK(launch(rec, a, need, readers, order, false, &stale) == readers && !stale);
                    }
                }
            } while (std::next_permutation(order.begin(), order.end()));
        }
    std::printf("%ld launches\n", launches);
    return 0;
}
"""


def test_no_order_of_a_launch_leaves_a_record_that_a_replay_believes(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    src, exe = tmp_path / "dep.cpp", tmp_path / "dep"
    src.write_text(MAIN)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2407_02031_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0]) > 1000
