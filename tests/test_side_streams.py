"""Which side streams the batch groups of a forward take, and the fork to them and back (csrc/side_streams.h), compiled for the host on counters
in place of streams.  Streams lie on hardware queues, a new one on a queue that has the fewest."""
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
#include <map>
static long created, destroyed, questions;
static int queues = 4, later;                          // later: questions are answered by answer() only
static std::map<long, int> queue_of;                   // of every stream there is, the callers' too
struct Question { uint64_t *at, what; };
static std::vector<Question> open_questions;
static int lie_down(long s)
{
    std::vector<int> load(queues);
    for (auto &q : queue_of) load[q.second]++;
    int best = 0;
    for (int q = 1; q < queues; q++) if (load[q] < load[best]) best = q;
    return queue_of[s] = best;
}
static std::set<long> captured;
static std::string trace;
static const char *failing = "";
struct Fake {
    typedef long Stream;
    typedef long Event;
    typedef int Error;
    static int create(long *s) { *s = 1000000 + ++created; lie_down(*s); return 0; }
    static void destroy(long s) { destroyed++; queue_of.erase(s); }
    static void ask(long s, uint64_t *answer, unsigned tag)
    {
        questions++;
        const Question q{answer, (uint64_t)tag << 48 | 64u * (queue_of.count(s) ? queue_of[s] + 1 : 9)};
        if (later) open_questions.push_back(q); else *q.at = q.what;
    }
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
static samp::AnswerPage page;
static samp::SidePool<Fake> pool(page);
extern "C" {
Held *encoder() { return new Held; }
void close_encoder(Held *h) { delete h; }
void provide_page() { page.at = new uint64_t[samp::AnswerPage::BLOCKS * samp::AnswerPage::ANSWERS](); }
void queue_count(int n, int answered_later) { queues = n; later = answered_later; }
int caller(long s) { return lie_down(s); }
void caller_on(long s, int queue) { queue_of[s] = queue; }
int queue(long s) { return queue_of[s]; }
long asked() { return questions; }
void answer() { for (auto &q : open_questions) *q.at = q.what; open_questions.clear(); }
long take(Held *h, int device, long caller, int shareable, int count, long *out)      // the first side stream
{
    long s[samp::MAX_GROUPS - 1] = {};
    if (pool.take(*h, device, caller, shareable, count, s)) return -2;
    for (int i = 0; i < count; i++) if (!s[i]) return -3;
    if (h->front()->caller.stream != caller || h->front()->device != device) return -1;
    for (int i = 0; i < count && out; i++) out[i] = s[i];
    return s[0];
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
    take = lib.take
    take.argtypes, take.restype = [C.c_void_p, C.c_int, C.c_long, C.c_int, C.c_int, C.c_void_p], C.c_long
    lib.take = lambda *a: take(*a, *[None] * (6 - len(a)))
    lib.caller.argtypes = lib.queue.argtypes = [C.c_long]
    lib.caller_on.argtypes, lib.asked.restype = [C.c_long, C.c_int], C.c_long
    lib.held.restype = lib.made.restype = lib.gone.restype = C.c_long
    lib.capture.argtypes = [C.c_long, C.c_int]
    lib.fork.argtypes, lib.fork.restype = [C.c_int, C.c_char_p, C.c_int, C.POINTER(C.c_int)], C.c_char_p
    return lib


@pytest.mark.parametrize("encoders", [1, 2, 3, 7])
@pytest.mark.parametrize("streams", [4, 5, 6, 8, 32])
@pytest.mark.parametrize("fresh", [False, True])
@pytest.mark.parametrize("page", [False, True])
def test_many_callers_in_turn_create_and_destroy_nothing(lib, encoders, streams, fresh, page):
    """Callers in turn, each with every encoder; then encoders that start at different callers; `fresh`: a stream that nobody has seen before
    instead of the first one, each time.  With the page, streams that lie on one queue may have to be parted: a few more are created."""
    if page:
        lib.provide_page()
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
        for _ in range(4 * encoders + 8 * page):                  # each encoder may still have to get sets of its own, and these their spares
            turn(offset)
        made = lib.made()
        for _ in range(5):
            turn(offset)
        assert lib.made() == made and lib.gone() == 0
    assert lib.made() <= (4 + 5 * page) * encoders
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


@pytest.mark.parametrize("queues", [4, 5, 8])
@pytest.mark.parametrize("groups", [2, 3, 4])
@pytest.mark.parametrize("later", [False, True])
def test_groups_lie_on_queues_apart_as_soon_as_the_answers_are_there(lib, queues, groups, later):
    """Callers on every queue (for two groups, which a forward chooses by itself, unevenly); nothing is asked or created any more once the streams
    lie apart."""
    lib.provide_page()
    lib.queue_count(queues, int(later))
    out = (C.c_long * 3)()
    encs = [lib.encoder() for _ in range(5)]
    for n in range(40):
        lib.caller_on(n, n * 7 % 5 % queues if groups == 2 else n * 7 % 40 % queues)
    for n in range(20):
        e = encs[n % 5]
        for _ in range(8):
            assert lib.take(e, 0, n, 1, groups - 1, out) > 0
            lib.answer()
        on = [lib.queue(n)] + [lib.queue(s) for s in out[:groups - 1]]
        assert len(set(on)) == groups, on
        asked, made, before = lib.asked(), lib.made(), out[:]
        for _ in range(40):
            lib.take(e, 0, n, 1, groups - 1, out)
        assert (lib.asked(), lib.made(), out[:]) == (asked, made, before)
    assert lib.made() <= 6 * 20


def test_fewer_queues_than_groups_settle_too(lib):
    """One queue for everything, or two for three groups: no more than the spares are created."""
    lib.provide_page()
    e = lib.encoder()
    for queues in (1, 2):
        lib.queue_count(queues, 0)
        for n in (10 * queues, 10 * queues + 1):
            lib.caller(n)
            for _ in range(20):
                lib.take(e, 0, n, 1, 2)
            asked, made = lib.asked(), lib.made()
            for _ in range(30):
                lib.take(e, 0, n, 1, 2)
            assert (lib.asked(), lib.made()) == (asked, made)
    assert lib.made() <= 4 * 6


def test_a_handle_that_comes_to_be_another_stream_is_noticed(lib):
    lib.provide_page()
    e = lib.encoder()
    for q in (0, 1, 2, 3, 0):
        lib.caller_on(5, q)
        for _ in range(64 + 5):
            side = lib.take(e, 0, 5, 1, 1)
        assert lib.queue(side) != q
    assert lib.made() <= 2


def test_answers_that_take_their_time(lib):
    """A program that enqueues hundreds of forwards ahead: the questions wait behind them, are not asked again, and count when they are answered;
    one that is never answered is asked again after a thousand forwards."""
    lib.provide_page()
    lib.queue_count(1, 1)
    e = lib.encoder()
    lib.caller(5)
    lib.take(e, 0, 5, 1, 1)
    lib.queue_count(4, 1)
    for _ in range(500):
        lib.take(e, 0, 5, 1, 1)
    assert (lib.asked(), lib.made()) == (2, 1)
    lib.answer()
    for _ in range(3):
        side = lib.take(e, 0, 5, 1, 1)
        lib.answer()
    assert lib.queue(side) != lib.queue(5) and lib.made() == 2
    other = lib.encoder()
    lib.caller(6)
    asked = lib.asked()
    for _ in range(1030):
        lib.take(other, 0, 6, 1, 1)
    assert lib.asked() == asked + 4


def test_nothing_is_asked_in_a_capture_and_without_a_page(lib):
    e = lib.encoder()
    lib.caller(5)
    for _ in range(70):
        lib.take(e, 0, 5, 1, 1)
    assert lib.asked() == 0 and lib.made() == 1
    lib.provide_page()
    other = lib.encoder()
    lib.caller(6)
    lib.capture(6, 1)
    lib.take(other, 0, 6, 1, 1)
    assert lib.asked() == 0
    lib.capture(6, 0)
    lib.take(other, 0, 6, 1, 1)
    assert lib.asked() == 2


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
