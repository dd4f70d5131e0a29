// The streams on which batch groups run beside a caller's stream: which ones a forward takes, and the fork to them and back.  Written against a
// small set of operations (Hip), so that the host can test the rules on their own.
#pragma once

#include <cstddef>
#include <memory>
#include <mutex>
#include <vector>

namespace samp {

constexpr int MAX_GROUPS = 4;

template <class Hip> struct SideStreams {
    typedef typename Hip::Stream Stream;
    int device;
    Stream caller, side[MAX_GROUPS - 1] = {};
    SideStreams(int d, Stream c) : device(d), caller(c) {}
    SideStreams(const SideStreams &) = delete;
    ~SideStreams()
    {
        for (Stream s : side)
            if (s) Hip::destroy(s);
    }
    bool in_capture() const { return side[0] && Hip::capturing(side[0]); }      // (groups take side[0] first)
};

// The sets that an encoder holds, the one used last in front.
template <class Hip> using HeldSides = std::vector<std::shared_ptr<SideStreams<Hip>>>;

// Encoders that are used on the same stream share a set: a forward that takes up a stream which has been idle starts some 60 us late (three BERT-base
// encoders in turn, 32 x 128 Fully-Quant, streams of their own / shared: 740 / 680 us), and the forwards of one caller's stream have one order anyway.
// An encoder holds up to MAX_SIDES sets, so that callers that take turns do not wait for each other.  Beyond, nothing is created or destroyed in a
// forward: the set that this encoder alone holds and has not used for longest goes over to the new caller (events order what is still queued on it),
// one that others hold too is left to them.  A set that is part of a capture still open stays with its caller.  So n encoders never have more than
// MAX_SIDES n sets (one more per capture open), and a set ends with the last encoder that holds it.
template <class Hip> class SidePool {
    typedef SideStreams<Hip> Set;
    typedef typename Hip::Stream Stream;
    std::mutex mutex_;
    std::vector<std::weak_ptr<Set>> all_;

public:
    static constexpr size_t MAX_SIDES = 4;

    // A set with `count` streams for the caller.  shareable: the same handle always is the same stream.  May throw std::bad_alloc.
    typename Hip::Error take(HeldSides<Hip> &held, int device, Stream caller, bool shareable, int count, std::shared_ptr<Set> *out)
    {
        std::shared_ptr<Set> left, found;           // (left: destroyed, should it be the last reference after all, when the lock is gone)
        const std::lock_guard<std::mutex> lock(mutex_);
        held.reserve(held.size() + 1);
        auto serves = [&](const Set &s) { return s.caller == caller && s.device == device; };
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
                    found->caller = caller;
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
            found = std::make_shared<Set>(device, caller);
            all_.push_back(found);
        }
        held.insert(held.begin(), found);
        *out = found;
        for (int i = 0; i < count; i++)
            if (!found->side[i])
                if (const typename Hip::Error e = Hip::create(&found->side[i])) return e;
        return {};
    }

    size_t sets() const { return all_.size(); }
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
