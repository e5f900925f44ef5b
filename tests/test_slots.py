"""Walking the last slots of an adjacency of 2^31 - 1 edges, the most a graph may
have, with a look ahead (csrc/slots.h, which every sweep's loops use): compiled
for the CPU and compared with 64-bit arithmetic."""
import os
import subprocess

import pytest

from tests.conftest import ROOT

PROGRAM = r"""
#include <cstdio>
#include <cstdint>
#include <initializer_list>
#include "slots.h"
using namespace pp;
// one lane's walk over [b, e): lookahead U, stride S; counts the slots taken and
// checks every position that would be loaded
static long long walk(int64_t b, int64_t e, int64_t lane, int U, int64_t S) {
    long long n = 0;
    int64_t want = b + lane;
    for (slot_t j0 = (slot_t)b + (slot_t)lane; j0 < (slot_t)e; j0 += (slot_t)(U * S)) {
        for (int k = 0; k < U; ++k) {
            const int64_t at = slot_at(j0, (slot_t)(k * S), (slot_t)e);
            if (at < b || at >= e) return -1;               // a load outside the row
            if (slot_in(j0, (slot_t)(k * S), (slot_t)e)) {
                if (at != want) return -2;                  // not the next slot of the lane
                want += S;
                ++n;
            } else if (at != e - 1) return -3;
        }
    }
    return want >= e ? n : -4;
}
int main() {
    const int64_t M = INT32_MAX;
    const int64_t ends[] = {M, M - 1, M - 255, M - 4096, 1000, 1};
    const int64_t lens[] = {1, 2, 63, 64, 65, 511, 512, 513, 1000, 5000};
    const int64_t lanes[] = {0, 1, 31, 63, 255, 1023};
    const int shapes[][2] = {{1, 1}, {4, 1}, {8, 1}, {4, 16}, {8, 32}, {8, 64}, {16, 64}, {8, 128}, {1, 1024}, {8, 1024}};
    for (int64_t e : ends) for (int64_t len : lens) if (len <= e) for (int64_t lane : lanes) for (auto& s : shapes) {
        const int64_t b = e - len;
        if (lane >= s[1]) continue;  // lanes of a group lie a slot apart
        const long long got = walk(b, e, lane, s[0], s[1]);
        const long long want = lane < len ? (len - lane + s[1] - 1) / s[1] : 0;
        if (got != want) { std::printf("b=%lld e=%lld lane=%lld U=%d S=%d: %lld, not %lld\n", (long long)b, (long long)e, (long long)lane, s[0], s[1], got, want); return 1; }
    }
    for (int64_t len : lens) for (int64_t piece : {32, 64, 128, 256}) {
        const int64_t b = M - len;
        for (int64_t k = 0; k * piece < len; ++k) {
            const int64_t want = b + (k + 1) * piece < M ? b + (k + 1) * piece : M;
            if (slot_piece_end((slot_t)b, (slot_t)k, (slot_t)piece, (slot_t)M) != want) { std::printf("piece\n"); return 2; }
        }
    }
    return 0;
}
"""


def test_last_slots_of_the_largest_graph(tmp_path):
    src = tmp_path / "slots.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "slots"
    csrc = os.path.join(ROOT, "paper_2010_16012_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{csrc}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("name", ["bc", "bfs", "graph", "multi", "ppr", "pr", "push", "tc"])
def test_no_signed_look_ahead_in_the_sweeps(name):
    # a position ahead is never formed as a signed sum and clamped afterwards
    import re
    with open(os.path.join(ROOT, "paper_2010_16012_amd", "csrc", name + ".hip")) as fh:
        text = fh.read()
    bad = re.findall(r"\[(?:\(uint32_t\))?min\((?:j0|jb|at)\b(?![^\]]*int64_t)[^\]]*\]|for \(int32_t j[0b]? = \w+ \+ \w+; j", text)
    assert bad == []
