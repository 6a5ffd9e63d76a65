// The words by which the parts of a small block in one launch (block_once_kernel) tell that they have delivered: plain C++, the same on the
// GPU and the host, so that what passes for a delivered word can be checked without a GPU.
//
// A word carries bits of the call's tag beside what is handed over.  The space holds anything before a call, and nobody clears
// it first: a word is there when its tag bits match, and whoever goes on clears all of them, so that a graph that is replayed, whose
// calls carry the same tag each time, meets none of the last replay.  A leftover passes for a part that is still on its way
// if all words of that part match by accident: 120 bits of tag in the four words of a draft's position, 62 in the one of the bonus position,
// which hands nothing over and is compared whole.
#pragma once

#include <atomic>
#include <chrono>
#include <cstdint>

namespace {

struct CallTag {
    uint32_t a, b;
};

// Another tag for each of 2^64 - 1 calls, begun anywhere, never 0; mixed (the finalizer of SplitMix64, which maps no two to one, and 0 to
// 0), so that calls that follow one another differ in both halves.
inline CallTag next_call_tag() {
    static std::atomic<uint64_t> calls{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count()};
    const auto next = [] { return calls.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed); };
    uint64_t x = next();
    if (x == 0) x = next();
    x = (x ^ x >> 30) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ x >> 27) * 0x94D049BB133111EBull;
    x ^= x >> 31;
    return CallTag{(uint32_t)(x >> 32), (uint32_t)x};
}

// The upper half of word i: 30 bits of the tag, another value for every word, so that a space filled with one pattern matches one
// of them at most, and none that a cleared word has, whole or cut to its upper bits.  Neighbouring words take different halves of the tag.
constexpr uint32_t word_tag(CallTag t, int i) { return ((i & 1 ? t.b : t.a) + (uint32_t)i * 0x9E3779B1u) | 0x80000001u; }
// The lower half of a word that hands nothing over: the tag's other half, 32 bits.
constexpr uint32_t rest_tag(CallTag t, int i) { return (i & 1 ? t.a : t.b) + (uint32_t)i * 0x9E3779B1u; }

constexpr uint64_t value_word(CallTag t, int i, uint32_t v) { return (uint64_t)word_tag(t, i) << 32 | v; }
constexpr uint64_t arrival_word(CallTag t, int i) { return (uint64_t)word_tag(t, i) << 32 | rest_tag(t, i); }
// Whether x is word i, with a value or without.
constexpr bool is_word(CallTag t, int i, bool value, uint64_t x) {
    return ((uint32_t)(x >> 32) == word_tag(t, i)) & (value | ((uint32_t)x == rest_tag(t, i)));
}

// What the part that goes on leaves in word 0, which nobody else writes.
constexpr uint64_t claim_word(CallTag t) { return (uint64_t)t.a << 32 | t.b; }

// A greedy candidate in words i and i + 1: 64 bits of the value (`v`), 21 of the token (up to SS_MAX_VOCAB, for none), and the
// upper 21 and 22 bits of the words' tags, of which 20 and 21 are free.
constexpr uint64_t best_word(CallTag t, int i, uint64_t v) { return (uint64_t)(word_tag(t, i) >> 11) << 43 | v >> 21; }
constexpr uint64_t best_word2(CallTag t, int i, uint64_t v, uint32_t token) {
    return (uint64_t)(word_tag(t, i + 1) >> 10) << 42 | (v & 0x1FFFFFu) << 21 | token;
}
constexpr bool are_best_words(CallTag t, int i, uint64_t x, uint64_t y) {
    return (uint32_t)(x >> 43) == word_tag(t, i) >> 11 && (uint32_t)(y >> 42) == word_tag(t, i + 1) >> 10;
}
constexpr uint64_t best_value(uint64_t x, uint64_t y) { return x << 21 | (y >> 21 & 0x1FFFFFu); }
constexpr uint32_t best_token(uint64_t y) { return (uint32_t)(y & 0x1FFFFFu); }

}  // namespace
