// The mailbox words by which the workgroups of a batch of SOR iterations hand
// their boundary values to each other (kernels_sor.hip).
//
// A value travels as one 64-bit word into a slot of its receiver, which polls
// the slot until its word has changed.  A sender therefore never stores a word
// twice in a row: a value whose word the slot already holds goes as AGAIN, the
// next one as itself again.  No flag follows the data and no fence is needed,
// since nothing else is read because of a word, and a slot has one writer.
// (Emptied by its reader instead, a slot had two, and only the time between
// their stores put them in order: an emptying store that landed after the next
// value lost it, and the reader waited for it until it gave up.  Two words a
// value, each with 32 bits of it and the iteration's number, have one writer too
// but twice the traffic: a solve of 64x64x128 took 2.08 ms, so 1.42.)
//
// Iteration g uses slot set g & 1.  A sender stores iteration g + 2 into the set
// of g once it holds the reader's values of g + 1, and the reader sent those
// after it had loaded all of g.  A launch begins with UNSENT in every slot:
// launches use two banks of slots in turn, and each fills the next one's bank
// (which nothing else touches meanwhile) before it does anything else.
#pragma once

#include <cstdint>

namespace ek {

constexpr int SOR_BANKS = 2, SOR_SETS = 2;

// NaNs that no arithmetic produces.
constexpr uint64_t SOR_UNSENT = 0xFFF7A5C35A3C7F11ull;
constexpr uint64_t SOR_AGAIN = 0xFFF7A5C35A3C7F22ull;

// The word of a value for a slot that holds `before`, and the way back.
constexpr uint64_t sor_word(uint64_t value, uint64_t before) {
  if (value == SOR_UNSENT || value == SOR_AGAIN) value ^= 4;
  return value == before ? SOR_AGAIN : value;
}
constexpr uint64_t sor_value(uint64_t word, uint64_t before) {
  return word == SOR_AGAIN ? before : word;
}

}  // namespace ek
