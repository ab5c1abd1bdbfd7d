// The words by which the workgroups of a resident solve (resident.hip) meet: per barrier parity a
// slot for each workgroup with its minD and its threshold, then a slot for each with its count of
// shared records. A word says itself which barrier it is for, so none is cleared between phases, or
// between the queries that a team of a batch solves one after the other: what an earlier barrier
// left must never read as the one that is awaited. Plain constant expressions, so that a host
// program can enumerate them.
#pragma once
#include <stdint.h>

constexpr uint32_t kResMaxW = 256;
constexpr uint32_t kSlotStride = 8;    // u64 between two workgroups' words (64 bytes)

// minD and threshold: tag (4 bits) and value (all ones: infinity; distances and thresholds stay below
// 2^58 + 2^32). Every workgroup writes them at every barrier, so a word holds the awaited barrier's
// value or that of the last one of the same parity.
constexpr unsigned long long kVal = (1ull << 60) - 1, kTag = ~kVal;
constexpr unsigned long long bar_tag(uint32_t b) { return (unsigned long long)((b >> 1) % 15u + 1u) << 60; }
constexpr uint32_t bar_words(uint32_t b, uint32_t W) { return (b & 1u) * W * kSlotStride; }
// Workgroup wg's words at a barrier without values (a team's set-up): both, since after a run of
// queries of one phase each, whose set-ups are the only barriers of their parity, a word left out
// would carry the tag of a later phase.
template <class Put>
constexpr void bar_put_empty(uint32_t b, uint32_t W, uint32_t wg, Put put) {
    for (uint32_t i = 0; i < 2; ++i) put(bar_words(b, W) + wg * kSlotStride + i, bar_tag(b) | kVal);
}

// Counts of shared records are written by solves that share only, so that a word may be older than
// any number of barriers: it holds the whole number of the barrier that follows it (never 0, which is
// what the words start with). One region: a count is read before the barrier it precedes, and the
// next one published after that.
constexpr unsigned long long count_word(uint32_t next, uint32_t count) { return (unsigned long long)next << 32 | count; }
constexpr bool count_is_for(unsigned long long word, uint32_t next) { return (uint32_t)(word >> 32) == next; }
constexpr uint32_t count_words(uint32_t W) { return 2u * W * kSlotStride; }

constexpr uint32_t team_words(uint32_t W) { return 3u * W * kSlotStride; }
