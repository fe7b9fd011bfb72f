// Turns of the launches whose blocks wait for each other: the host side's
// books, without a call into the device's runtime.
//
// Such a launch may take the whole device, so on each device one is under way
// at a time.  Launches are numbered; the last block of a launch writes its
// number to a word of host memory, and that word says whether another owner
// may launch.  The stream of the last launch is not asked: it may have been
// destroyed meanwhile, or be under capture by the caller that owns it.
#pragma once

#include <cstdint>
#include <map>
#include <new>

namespace rdos {

// One device's turn.
class LaunchTurn {
public:
    // The number of a launch of so many periods by `owner`, or 0 while another
    // owner's launches are not known to have ended (`ended`: the number in the
    // device's word).  An owner's launches follow one another on its stream.
    uint64_t take(uint64_t owner, uint64_t ended, uint64_t periods)
    {
        if (owner != owner_ && ended < last_) return 0;
        return take_behind(owner, periods);
    }
    // The same for a launch that waits for the last one on the device.
    uint64_t take_behind(uint64_t owner, uint64_t periods)
    {
        owner_ = owner;
        const uint64_t before = sum_[last_ % kKept];
        sum_[++last_ % kKept] = before + periods;
        return last_;
    }
    // The launch that took the last number was refused by the runtime.
    void give_back() { --last_; }
    // Whether a launch of so many periods should wait for those that have not
    // ended, rather than leave its periods to the queue: for up to twice as
    // many periods as its own, which is what the queue costs it.  Its owner's
    // own last launch (`mine`) it waits for in any case.
    bool worth_waiting(uint64_t ended, uint64_t mine, uint64_t periods) const
    {
        const uint64_t from = ended > mine ? ended : mine;
        return last_ - from < kKept && sum_[last_ % kKept] - sum_[from % kKept] <= 2 * periods;
    }

private:
    static constexpr uint64_t kKept = 256;
    uint64_t owner_ = 0;
    uint64_t last_ = 0;
    uint64_t sum_[kKept] = {};  // periods of launches 1 .. n, by n
};

// Owners, by stream: simulations on one stream are one owner, since their
// launches follow one another.  The library's own streams get a number each;
// a caller's stream keeps its number while some simulation is on it (which
// leaves it drained), so that a stream that is made later at the same address
// is another owner.
class StreamOwners {
public:
    uint64_t own_stream() { return ++next_; }
    uint64_t join(const void *stream)
    {
        try {
            Use &u = streams_[stream];
            if (u.users++ == 0) u.number = ++next_;
            return u.number;
        } catch (const std::bad_alloc &) {  // not in the books: an owner to itself
            return ++next_;
        }
    }
    void leave(const void *stream)
    {
        const auto it = streams_.find(stream);
        if (it != streams_.end() && --it->second.users == 0) streams_.erase(it);
    }

private:
    struct Use {
        uint64_t number = 0;
        int64_t users = 0;
    };
    std::map<const void *, Use> streams_;
    uint64_t next_ = 0;
};

}  // namespace rdos
