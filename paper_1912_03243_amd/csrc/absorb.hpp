// Greedy choice of the bits of a tile or of a stage's registers: which gates
// of a list, in order, a set of bits lets through.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace juqcs {

// Bits of a gate (fewer than 64): those it is diagonal on, and the others.
struct AbsorbMask {
  uint64_t full = 0, diag = 0;
  uint64_t weight = 1;
};

// A set of bits takes a gate if it holds all of the bits that the gate is not
// diagonal on and at least one of any, and no earlier gate is left behind that
// the gate does not commute with (gates that are diagonal on a bit commute
// there).
struct Absorb {
  uint64_t set, full = 0, diag = 0;  // bits of gates left behind
  explicit Absorb(uint64_t s) : set(s) {}
  bool take(const AbsorbMask& m) {
    if (!(m.full & (~set | full | diag)) && !(m.diag & full) && ((m.full | m.diag) & set)) return true;
    full |= m.full;
    diag |= m.diag;
    return false;
  }
  bool done() const { return !(set & ~full); }
};

// Weights that a growing set of bits takes.  What a set takes, a larger one
// takes too (it leaves fewer gates behind), so a candidate is tried on the gates
// that the set so far leaves behind only; eight candidates run side by side.
// Gates after the point where a set is wholly blocked are not looked at, nor
// those that come after window gates in a row of which no set takes any.
class AbsorbSearch {
 public:
  // Gates head, then count more (which outlive the search).
  AbsorbSearch(std::vector<AbsorbMask> head, const AbsorbMask* gates, size_t count, uint64_t set, size_t window)
      : gates_(gates), count_(count), window_(window), left_(std::move(head)) {
    left_.reserve(std::min<size_t>(left_.size() + count_, 256));
    grow(set);
  }
  AbsorbSearch(const std::vector<AbsorbMask>& gates, uint64_t set)
      : AbsorbSearch({}, gates.data(), gates.size(), set, gates.size()) {}
  // The set takes on bits.
  void grow(uint64_t set) {
    Absorb ab(set);
    size_t k = 0;
    for (size_t i = 0; i < left_.size(); ++i) {
      if (ab.take(left_[i])) taken_ += left_[i].weight;
      else left_[k++] = left_[i];
    }
    left_.resize(k);
    for (size_t i = next_; i < count_ && i - next_ <= window_ && !ab.done(); ++i) {
      if (!ab.take(gates_[i])) continue;
      taken_ += gates_[i].weight;
      left_.insert(left_.end(), gates_ + next_, gates_ + i);
      next_ = i + 1;
    }
  }
  uint64_t taken() const { return taken_; }
  // out[i]: what set[i], a superset of the set so far, takes.
  void weights(const uint64_t* set, int count, uint64_t* out) const;

 private:
  const AbsorbMask* gates_;  // from next_ on: not looked at yet, all left behind
  size_t count_, window_;
  std::vector<AbsorbMask> left_;  // left behind before that
  size_t next_ = 0;
  uint64_t taken_ = 0;
};

}  // namespace juqcs
