"""The FP32 walk's ring counters (host build of the same code): the fill level, the slots and the
neighbour count stay exact however many entries pass through a ring."""
import os
import subprocess

import pytest

import paper_1805_05128_amd as P

CSRC = os.path.join(os.path.dirname(os.path.abspath(P.__file__)), "csrc")
# One lane as the walk drives it: up to three candidates a look, drains of two while the ring is
# nearly full, every fifth entry turned down at its pop, every seventh a mirror entry.
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "ring.h"
constexpr unsigned kSlot = 1024, kQ = 8, kRing = kQ * kSlot;
int main(int, char **argv) {
    const long long total = atoll(argv[1]);
    csph::RingCount<kSlot, kRing> c;
    long long in = 0, out = 0, members = 0;
    static long long ring[kQ];
    auto drain = [&]() {
        if (c.qr == c.qw) return;
        if (ring[(c.qr & (kRing - 1)) / kSlot] != out) { puts("slot"); exit(1); }
        c.qr += kSlot;
        const bool ghost = out % 7 == 0, in64 = out % 5 != 0;
        c.drop += in64 || ghost ? 0 : 1;
        c.ghosts += ghost ? 1 : 0;
        members += in64 && !ghost;
        ++out;
    };
    while (in < total) {
        for (int u = 0; u < 3 && in < total; ++u) {
            ring[(c.qw & (kRing - 1)) / kSlot] = in++;
            c.qw += kSlot;
        }
        if (c.qw - c.qr > (kQ - 3) * kSlot) {
            do {
                drain();
                drain();
                c.popped(2);
            } while (c.qw - c.qr > (kQ - 3) * kSlot);
            c.settle_counters();
        }
        if ((long long)((c.qw - c.qr) / kSlot) != in - out) { puts("fill"); return 1; }
    }
    while (c.qr != c.qw) drain();
    printf("%lld %lld\n", members, (long long)c.count());
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("ring")
    (d / "ring.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(d / "ring.cpp"), "-o",
                    str(d / "ring")], check=True)
    return str(d / "ring")


# around 2^22 entries, where 32 bits of bytes run out, and the largest particle set
@pytest.mark.parametrize("total", [0, 1, 100, (1 << 20) + 3, (1 << 22) - 1, (1 << 22) + 1,
                                   10000019, (1 << 27) - 1])
def test_count(program, total):
    r = subprocess.run([program, str(total)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    members, count = map(int, r.stdout.split())
    assert count == members
