// The streams on which batch groups run beside a caller's stream: which ones a forward takes, and the fork to them and back.  Written against a
// small set of operations (Hip), so that the host can test the rules on their own.
#pragma once

#include <atomic>
#include <cstddef>
#include <cstdint>
#include <memory>
#include <mutex>
#include <utility>
#include <vector>

namespace samp {

constexpr int MAX_GROUPS = 4;

// A page of host memory that the device can write, in blocks of one cache line: blocks are handed out and taken back.
struct AnswerPage {
    static constexpr int BLOCKS = 64, ANSWERS = 8;
    std::atomic<uint64_t *> at{nullptr};            // BLOCKS * ANSWERS zeros; null: there is none
    std::atomic<uint64_t> taken{0};
    uint64_t *take()
    {
        uint64_t *const page = at.load(std::memory_order_acquire);
        for (uint64_t t = taken.load(); page && ~t;) {
            const int i = __builtin_ctzll(~t);
            if (taken.compare_exchange_weak(t, t | 1ull << i)) return page + i * ANSWERS;
        }
        return nullptr;
    }
    void give_back(uint64_t *block)
    {
        if (block) taken.fetch_and(~(1ull << (block - at.load()) / ANSWERS));
    }
};

// A caller's stream and the ones beside it.  Streams lie on a few hardware queues (four), each on one for as long as it exists, and what lies on one queue
// runs one after the other: with its side stream on the caller's queue, a forward of two groups takes longer than one group (BERT-base 32 x 128
// Fully-Quant on ten streams, each on its own: two of them 1100 us, the others 690; one group 765).  Only a kernel can see its queue.  So each stream is
// asked once, by a kernel that nobody waits for, and a later forward that finds the answers takes streams that lie apart.
template <class Hip> struct SideStreams {
    typedef typename Hip::Stream Stream;
    static constexpr int CANDIDATES = 6;            // side streams beyond those in use are spares
    struct Asked { Stream stream{}; int slot = 0; unsigned tag = 0; };      // tag 0: not asked
    int device;
    AnswerPage *page;
    uint64_t *answers;
    Asked caller, side[CANDIDATES];
    int settled = 0;                                // so many in front lie apart, or cannot
    unsigned uses = 0;

    SideStreams(int d, Stream c, AnswerPage *p) : device(d), page(p), answers(p->take())
    {
        caller.stream = c;
        for (int i = 0; i < CANDIDATES; i++) side[i].slot = i + 1;
    }
    SideStreams(const SideStreams &) = delete;
    ~SideStreams()
    {
        for (Asked &s : side)
            if (s.stream) Hip::destroy(s.stream);
        page->give_back(answers);
    }
    bool in_capture() const { return side[0].stream && Hip::capturing(side[0].stream); }      // (groups take side[0] first)
    void serve(Stream c)
    {
        caller.stream = c;
        caller.tag = 0;
        settled = 0;
    }

    // 0: not known yet.  An answer carries the tag of its question in the 16 bits that an address leaves.
    uint64_t queue(const Asked &s) const
    {
        const uint64_t answer = *static_cast<volatile const uint64_t *>(answers + s.slot);
        return s.tag && answer >> 48 == s.tag ? answer & ~(~0ull << 48) : 0;
    }
    bool meets(const Asked &s, int before) const
    {
        const uint64_t q = queue(s);
        bool met = q && q == queue(caller);
        for (int j = 0; j < before; j++) met = met || (q && q == queue(side[j]));
        return met;
    }
    // Puts `count` streams in front that lie apart from each other and from the caller's, as far as is known.
    void part(int count, unsigned *last_tag)
    {
        const bool again = ++uses % 64 == 0, lost = uses % 1024 == 0;      // (a handle may be another stream's by now; an answer may not have come)
        if (settled >= count && !again) return;
        if (!answers || in_capture() || Hip::capturing(caller.stream)) return;
        bool known = true;
        auto ask = [&](Asked &s) {
            if (!s.tag || (lost && !queue(s))) {
                s.tag = *last_tag = *last_tag % 0xffff + 1;
                Hip::ask(s.stream, answers + s.slot, s.tag);
            }
            known = known && queue(s);
        };
        if (again && queue(caller)) caller.tag = 0;
        ask(caller);
        for (Asked &s : side)
            if (s.stream) ask(s);
        bool apart = true, room = true;
        for (int i = 0; i < count; i++) {
            if (!meets(side[i], i)) continue;
            int k = count;
            while (k < CANDIDATES && side[k].stream && (!queue(side[k]) || meets(side[k], i))) k++;
            if (k < CANDIDATES && side[k].stream) {
                std::swap(side[i], side[k]);
                continue;
            }
            apart = false;
            room = k < CANDIDATES;
            if (known && room && !Hip::create(&side[k].stream)) known = false;      // one more, asked by the next forward
        }
        settled = known && (apart || !room) ? count : 0;
    }
};

// The sets that an encoder holds, the one used last in front.
template <class Hip> using HeldSides = std::vector<std::shared_ptr<SideStreams<Hip>>>;

// Encoders that are used on the same stream share a set: a forward that takes up a stream which has been idle starts some 60 us late (three BERT-base
// encoders in turn, 32 x 128 Fully-Quant, streams of their own / shared: 740 / 700 us), and the forwards of one caller's stream have one order anyway.
// An encoder holds up to MAX_SIDES sets, so that callers that take turns do not wait for each other.  Beyond, nothing is created or destroyed in a
// forward: the set that this encoder alone holds and has not used for longest goes over to the new caller (events order what is still queued on it),
// one that others hold too is left to them.  A set that is part of a capture still open stays with its caller.  So n encoders never have more than
// MAX_SIDES n sets (one more per capture open), and a set ends with the last encoder that holds it.
template <class Hip> class SidePool {
    typedef SideStreams<Hip> Set;
    typedef typename Hip::Stream Stream;
    std::mutex mutex_;
    std::vector<std::weak_ptr<Set>> all_;
    unsigned last_tag_ = 0;
    AnswerPage &page_;

public:
    static constexpr size_t MAX_SIDES = 4;
    explicit SidePool(AnswerPage &page) : page_(page) {}

    // `count` streams for the groups beside the caller's, good as long as `held` is.  shareable: the same handle always is the same stream.  May
    // throw std::bad_alloc.
    typename Hip::Error take(HeldSides<Hip> &held, int device, Stream caller, bool shareable, int count, Stream *out)
    {
        std::shared_ptr<Set> left, found;           // (left: destroyed, should it be the last reference after all, when the lock is gone)
        const std::lock_guard<std::mutex> lock(mutex_);
        held.reserve(held.size() + 1);
        auto serves = [&](const Set &s) { return s.caller.stream == caller && s.device == device; };
        auto move_out = [&](size_t i) {
            std::shared_ptr<Set> s = std::move(held[i]);
            held.erase(held.begin() + (std::ptrdiff_t)i);
            return s;
        };
        for (size_t i = 0; i < held.size() && !found; i++)
            if (serves(*held[i])) found = move_out(i);
        if (!found && held.size() >= MAX_SIDES) {
            for (size_t i = held.size(); i-- > 0 && !found;)
                if (held[i].use_count() == 1 && held[i]->device == device && !held[i]->in_capture()) {
                    found = move_out(i);
                    found->serve(caller);
                }
            for (size_t i = held.size(); i-- > 0 && !found && !left;)
                if (held[i].use_count() > 1) left = move_out(i);
        }
        if (!found) {
            for (size_t i = 0; i < all_.size();) {
                const std::shared_ptr<Set> s = all_[i].lock();
                if (s && shareable && serves(*s)) found = s;
                if (s) i++;
                else all_.erase(all_.begin() + (std::ptrdiff_t)i);
            }
        }
        if (!found) {
            all_.reserve(all_.size() + 1);
            found = std::make_shared<Set>(device, caller, &page_);
            all_.push_back(found);
        }
        held.insert(held.begin(), found);
        for (int i = 0; i < count; i++)
            if (!found->side[i].stream)
                if (const typename Hip::Error e = Hip::create(&found->side[i].stream)) return e;
        found->part(count, &last_tag_);
        for (int i = 0; i < count; i++) out[i] = found->side[i].stream;
        return {};
    }
};

// Runs each(g, stream) for every group, group 0 on the caller's stream and the others beside it.  Whatever fails, every side stream that was forked is
// joined again: the caller's stream then stands for all work that was started (and a caller's capture has no loose ends).  Returns the first error.
template <class Hip, class Each>
int fork_join(int groups, typename Hip::Stream st, const typename Hip::Stream *side, typename Hip::Event fork, const typename Hip::Event *join, Each each)
{
    int rc = Hip::rc(Hip::record(fork, st)), forked = 0;
    for (int g = 0; g < groups && !rc; g++) {
        if (g) {
            rc = Hip::rc(Hip::wait(side[g - 1], fork));
            if (rc) break;
            forked = g;
        }
        rc = each(g, g ? side[g - 1] : st);
    }
    for (int g = 0; g < forked; g++) {
        typename Hip::Error e = Hip::record(join[g], side[g]);
        if (!e) e = Hip::wait(st, join[g]);
        if (!rc) rc = Hip::rc(e);
    }
    return rc;
}

}  // namespace samp
