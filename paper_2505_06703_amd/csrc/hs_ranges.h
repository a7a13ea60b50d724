// The memory that a call reads and writes, for the check that its outputs are
// disjoint from its inputs and from each other.  Host code.
#pragma once

#include <cstddef>
#include <cstdint>
#include <initializer_list>
#include <vector>

namespace hs {

struct Range {
    const void *p;
    size_t bytes;
    const char *name;
};

// A call's arrays.  The first 16 need no allocation (no call has more than a
// dozen).
class Ranges {
public:
    Ranges() = default;
    Ranges(std::initializer_list<Range> list)
    {
        for (const Range &x : list) push_back(x);
    }
    void push_back(const Range &x)
    {
        if (n_ < kFirst) first_[n_] = x;
        else more_.push_back(x);
        ++n_;
    }
    size_t size() const { return n_; }
    const Range &operator[](size_t i) const { return i < kFirst ? first_[i] : more_[i - kFirst]; }

private:
    static constexpr size_t kFirst = 16;
    Range first_[kFirst];
    std::vector<Range> more_;
    size_t n_ = 0;
};

inline bool overlap(const Range &a, const Range &b)
{
    if (!a.p || !b.p || a.bytes == 0 || b.bytes == 0) return false;
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a.p), b0 = reinterpret_cast<uintptr_t>(b.p);
    return a0 < b0 + b.bytes && b0 < a0 + a.bytes;
}

// The first output that overlaps an input or another output, with what it
// overlaps; false if there is none.
struct Clash {
    const char *out, *other;
    bool input;  // other is an input
};
inline bool find_clash(const Ranges &outs, const Ranges &ins, Clash &clash)
{
    for (size_t i = 0; i < outs.size(); ++i) {
        for (size_t k = 0; k < ins.size(); ++k)
            if (overlap(outs[i], ins[k])) {
                clash = {outs[i].name, ins[k].name, true};
                return true;
            }
        for (size_t k = i + 1; k < outs.size(); ++k)
            if (overlap(outs[i], outs[k])) {
                clash = {outs[i].name, outs[k].name, false};
                return true;
            }
    }
    return false;
}

}  // namespace hs
