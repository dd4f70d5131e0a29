"""Which side streams the batch groups of a forward take, and the fork to them and back (csrc/side_streams.h), compiled for the host on counters
in place of streams."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2209_09130_amd", "csrc")
SOURCE = r"""
#include "side_streams.h"
#include <cstring>
#include <set>
#include <string>
static long created, destroyed;
static std::set<long> captured;
static std::string trace;
static const char *failing = "";
struct Fake {
    typedef long Stream;
    typedef long Event;
    typedef int Error;
    static int create(long *s) { *s = ++created; return 0; }
    static void destroy(long) { destroyed++; }
    static bool capturing(long s) { return captured.count(s) != 0; }
    static int step(std::string what)
    {
        const bool bad = what == failing;
        trace += what + (bad ? "! " : " ");
        return bad ? 7 : 0;
    }
    static int record(long e, long s) { return step("r" + std::to_string(e) + "@" + std::to_string(s)); }
    static int wait(long s, long e) { return step("w" + std::to_string(e) + "@" + std::to_string(s)); }
    static int rc(int e) { return e ? -e : 0; }
};
typedef samp::HeldSides<Fake> Held;
static samp::SidePool<Fake> pool;
extern "C" {
Held *encoder() { return new Held; }
void close_encoder(Held *h) { delete h; }
long take(Held *h, int device, long caller, int shareable, int count)       // its first side stream, or -1 if the set is not the caller's
{
    std::shared_ptr<samp::SideStreams<Fake>> s;
    if (pool.take(*h, device, caller, shareable, count, &s)) return -2;
    for (int i = 0; i < samp::MAX_GROUPS - 1; i++)
        if (i < count && !s->side[i]) return -3;
    return s->caller == caller && s->device == device ? s->side[0] : -1;
}
long held(Held *h) { return (long)h->size(); }
long made() { return created; }
long gone() { return destroyed; }
void capture(long s, int on) { if (on) captured.insert(s); else captured.erase(s); }
const char *fork(int groups, const char *fails, int bad_group, int *rc)
{
    const long side[3] = {101, 102, 103}, join[3] = {11, 12, 13};
    trace.clear();
    failing = fails;
    *rc = samp::fork_join<Fake>(groups, 100L, side, 10L, join, [&](int g, long s) { trace += "g" + std::to_string(g) + "@" + std::to_string(s) + " "; return g == bad_group ? -5 : 0; });
    return trace.c_str();
}
}
"""


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    d = tmp_path_factory.mktemp("sides")
    (d / "s.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-pthread", "-I", CSRC, "-o", str(d / "s.so"), str(d / "s.cpp")],
                   check=True)
    return d / "s.so"


@pytest.fixture
def lib(built, tmp_path):
    lib = C.CDLL(str(shutil.copy(built, tmp_path / "s.so")))      # a copy, and with it counters and a pool, of this test's own
    lib.encoder.restype = C.c_void_p
    lib.close_encoder.argtypes = lib.held.argtypes = [C.c_void_p]
    lib.take.argtypes, lib.take.restype = [C.c_void_p, C.c_int, C.c_long, C.c_int, C.c_int], C.c_long
    lib.held.restype = lib.made.restype = lib.gone.restype = C.c_long
    lib.capture.argtypes = [C.c_long, C.c_int]
    lib.fork.argtypes, lib.fork.restype = [C.c_int, C.c_char_p, C.c_int, C.POINTER(C.c_int)], C.c_char_p
    return lib


@pytest.mark.parametrize("encoders", [1, 2, 3, 7])
@pytest.mark.parametrize("streams", [4, 5, 6, 8, 32])
@pytest.mark.parametrize("fresh", [False, True])
def test_many_callers_in_turn_create_and_destroy_nothing(lib, encoders, streams, fresh):
    """Callers in turn, each with every encoder; then encoders that start at different callers; `fresh`: a stream that nobody has seen before
    instead of the first one, each time."""
    encs = [lib.encoder() for _ in range(encoders)]
    new = [1000]

    def turn(offset):
        for k in range(streams):
            for i, e in enumerate(encs):
                caller = 1 + (k + offset * i) % streams
                if fresh and caller == 1:
                    new[0] += 1
                    caller = new[0]
                assert lib.take(e, 0, caller, 1, 1) > 0
                assert lib.held(e) <= 4

    for offset in (0, 1, 2, 3):
        for _ in range(4 * encoders):                             # each encoder may still have to get sets of its own
            turn(offset)
        made = lib.made()
        for _ in range(5):
            turn(offset)
        assert lib.made() == made and lib.gone() == 0
    assert lib.made() <= 4 * encoders
    for e in encs:
        lib.close_encoder(e)
    assert lib.gone() == lib.made()


def test_encoders_on_one_stream_share_and_on_different_streams_do_not(lib):
    a, b = lib.encoder(), lib.encoder()
    one = lib.take(a, 0, 1, 1, 1)
    assert lib.take(b, 0, 1, 1, 3) == one and lib.made() == 3     # the streams that b needs more join the shared set
    assert lib.take(b, 1, 1, 1, 1) != one and lib.take(b, 0, 2, 1, 1) != one
    own = lib.take(a, 0, 9, 0, 1)                                 # a handle that is another stream in every thread
    assert lib.take(b, 0, 9, 0, 1) != own and lib.take(a, 0, 9, 0, 1) == own
    lib.close_encoder(a)
    assert lib.gone() == 1                                        # its own one; the shared set is b's now
    assert lib.take(b, 0, 1, 1, 1) == one
    lib.close_encoder(b)
    assert lib.gone() == lib.made()


def test_the_set_unused_for_longest_goes_over_and_none_that_is_captured(lib):
    a, b = lib.encoder(), lib.encoder()
    sets = {c: lib.take(a, 0, c, 1, 1) for c in (1, 2, 3, 4)}
    lib.take(a, 0, 1, 1, 1)
    lib.capture(sets[2], 1)
    assert lib.take(a, 0, 5, 1, 1) == sets[3]                     # 2 is captured, 1 was used after 3
    assert lib.take(a, 0, 2, 1, 1) == sets[2]
    for s in sets.values():
        lib.capture(s, 1)
    extra = lib.take(a, 0, 6, 1, 1)                               # all of them captured: one more
    assert extra not in sets.values() and lib.held(a) == 5
    for s in sets.values():
        lib.capture(s, 0)
    assert lib.take(b, 0, 4, 1, 1) == sets[4]                     # shared now, the one that a has not used for longest
    assert lib.take(a, 0, 7, 1, 1) != sets[4] and lib.take(b, 0, 4, 1, 1) == sets[4]
    assert lib.made() == 5 and lib.gone() == 0
    lib.close_encoder(a)
    lib.close_encoder(b)


def test_every_forked_stream_is_joined_whatever_fails(lib):
    rc = C.c_int()

    def run(groups, fails="", bad=-1):
        steps = lib.fork(groups, fails.encode(), bad, C.byref(rc)).decode().split()
        return steps, rc.value

    steps, code = run(4)
    assert code == 0
    assert steps == ("r10@100 g0@100 w10@101 g1@101 w10@102 g2@102 w10@103 g3@103 r11@101 w11@100 r12@102 w12@100 r13@103 w13@100").split()
    assert run(1) == (["r10@100", "g0@100"], 0)
    assert run(4, bad=0) == (["r10@100", "g0@100"], -5)
    # a group fails: no further one is started, and those before it and its own stream are joined
    assert run(4, bad=2) == ("r10@100 g0@100 w10@101 g1@101 w10@102 g2@102 r11@101 w11@100 r12@102 w12@100".split(), -5)
    # so with a stream that cannot be forked, and with one that cannot be joined; the first error is the one returned
    assert run(3, "w10@102") == ("r10@100 g0@100 w10@101 g1@101 w10@102! r11@101 w11@100".split(), -7)
    assert run(3, "r11@101") == ("r10@100 g0@100 w10@101 g1@101 w10@102 g2@102 r11@101! r12@102 w12@100".split(), -7)
    assert run(3, "w11@100", bad=2)[1] == -5
    assert run(2, "r10@100") == (["r10@100!"], -7)
