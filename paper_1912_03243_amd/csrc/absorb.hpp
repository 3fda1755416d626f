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
// Gates after the point where a set is wholly blocked are not looked at.
class AbsorbSearch {
 public:
  AbsorbSearch(std::vector<AbsorbMask> gates, uint64_t set) : gates_(std::move(gates)) {
    left_.reserve(std::min<size_t>(gates_.size(), 256));
    grow(set);
  }
  // The set takes on bits.
  void grow(uint64_t set) {
    Absorb ab(set);
    size_t k = 0;
    for (size_t i = 0; i < left_.size(); ++i) {
      if (ab.take(left_[i])) taken_ += left_[i].weight;
      else left_[k++] = left_[i];
    }
    left_.resize(k);
    for (; next_ < gates_.size() && !ab.done(); ++next_) {
      if (ab.take(gates_[next_])) taken_ += gates_[next_].weight;
      else left_.push_back(gates_[next_]);
    }
  }
  uint64_t taken() const { return taken_; }
  // out[i]: what set[i], a superset of the set so far, takes.
  void weights(const uint64_t* set, int count, uint64_t* out) const;

 private:
  std::vector<AbsorbMask> gates_;  // from next_ on: not looked at yet, all left behind
  std::vector<AbsorbMask> left_;   // left behind before that
  size_t next_ = 0;
  uint64_t taken_ = 0;
};

}  // namespace juqcs
