"""The words by which the parts of a small block in one launch tell that they have delivered (csrc/words.h, plain C++), compiled on their
own: a space that holds anything must not pass for what a part has delivered (CPU)."""
import os
import random
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cinttypes>
#include <cstdio>
#include <cstring>
#include "words.h"
int main() {
    char what[16];
    unsigned a, b, token;
    int i;
    uint64_t x, y;
    while (std::scanf("%15s", what) == 1) {
        if (!std::strcmp(what, "calls")) {  // how many tags
            if (std::scanf("%d", &i) != 1) return 1;
            for (; i > 0; --i) {
                const CallTag t = next_call_tag();
                std::printf("%u %u\n", t.a, t.b);
            }
            continue;
        }
        if (std::scanf("%u %u %d %" SCNu64, &a, &b, &i, &x) != 4) return 1;  // tag, word, a value or what lies there
        const CallTag t{a, b};
        if (!std::strcmp(what, "value")) std::printf("%" PRIu64 "\n", value_word(t, i, (uint32_t)x));
        else if (!std::strcmp(what, "isvalue")) std::printf("%d\n", is_word(t, i, true, x) ? 1 : 0);
        else if (!std::strcmp(what, "arrival")) std::printf("%" PRIu64 "\n", arrival_word(t, i));
        else if (!std::strcmp(what, "isarrival")) std::printf("%d\n", is_word(t, i, false, x) ? 1 : 0);
        else if (!std::strcmp(what, "best")) {
            if (std::scanf("%u", &token) != 1) return 1;
            std::printf("%" PRIu64 " %" PRIu64 "\n", best_word(t, i, x), best_word2(t, i, x, token));
        } else {  // "isbest", with the second word
            if (std::scanf("%" SCNu64, &y) != 1) return 1;
            std::printf("%d %" PRIu64 " %u\n", are_best_words(t, i, x, y) ? 1 : 0, best_value(x, y), best_token(y));
        }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def words(tmp_path_factory):
    d = tmp_path_factory.mktemp("words")
    src, exe = d / "words.cpp", d / "words"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "paper_2603_16219_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)

    def ask(lines):
        out = subprocess.run([str(exe)], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]

    return ask


def tags(n, seed):
    rng = random.Random(seed)
    return [(0, 0), (1, 1 << 31), (1 << 31, 1), ((1 << 32) - 1,) * 2] + [(rng.getrandbits(32), rng.getrandbits(32)) for _ in range(n)]


def test_an_arrival_that_differs_in_any_bit_is_none(words):
    """What the bonus position's parts leave is one word each, which hands nothing over: all of its bits have to be there."""
    for a, b in tags(40, 1):
        for i in (0, 2, 3, 130, 4097):
            w, = words([f"arrival {a} {b} {i} 0"])[0]
            left = [w ^ 1 << k for k in range(64)] + [x for x in (0, (1 << 64) - 1, w >> 32 << 32, w & 0xFFFFFFFF) if x != w]
            assert w != 0 and words([f"isarrival {a} {b} {i} {x}" for x in [w] + left]) == [(1,)] + [(0,)] * len(left)


def test_sixty_two_bits_of_an_arrival_come_from_the_tag(words):
    """Flipping a bit of the tag changes the word, but for the two that keep cleared words out."""
    a, b, i = 0x12345678, 0x9ABCDEF0, 6
    same = [words([f"arrival {a ^ (1 << k if k < 32 else 0)} {b ^ (1 << k - 32 if k >= 32 else 0)} {i} 0"]) == words([f"arrival {a} {b} {i} 0"])
            for k in range(64)]
    assert sum(same) <= 2 and not any(same[k] for k in range(64) if k % 32 not in (0, 31))


def test_value_words_carry_their_value_and_no_cleared_or_other_word_passes(words):
    rng = random.Random(2)
    for a, b in tags(40, 3):
        for i in (2, 3, 77):
            v = rng.choice([0, 1, (1 << 32) - 1, rng.getrandbits(32)])
            w, = words([f"value {a} {b} {i} {v}"])[0]
            assert w & 0xFFFFFFFF == v
            got = words([f"isvalue {a} {b} {i} {x}" for x in (w, w ^ 1, 0, 0xFFFFFFFF, w ^ 1 << 40)] + [f"isvalue {a} {b} {i + 1} {w}", f"isvalue {a} {b} {i + 2} {w}"])
            assert got == [(1,), (1,), (0,), (0,), (0,), (0,), (0,)]


def test_greedy_candidates_come_back_whole(words):
    rng = random.Random(4)
    values = [0.0, -0.0, 1.5, -3.25e300, 5e-324, float("inf"), float("-inf")] + [rng.uniform(-50, 50) for _ in range(20)]
    for (a, b), v in zip(tags(len(values), 5), values):
        bits = struct.unpack("<Q", struct.pack("<d", v))[0]
        for token in (0, 12345, (1 << 20) - 1, 1 << 20):
            i = rng.randrange(2, 500)
            x, y = words([f"best {a} {b} {i} {bits} {token}"])[0]
            assert words([f"isbest {a} {b} {i} {x} {y}"]) == [(1, bits, token)]
            spoiled = [(0, y), (x, 0), (0, 0), (x ^ 1 << 50, y), (x, y ^ 1 << 50), (y, x)]
            assert all(got[0] == 0 for got in words([f"isbest {a} {b} {i} {p} {q}" for p, q in spoiled]))


def test_calls_that_follow_one_another_differ_in_both_halves(words):
    got = words(["calls 50000"])
    assert len(set(got)) == 50000
    for half in (0, 1):  # as random 30-bit numbers: some one pair of 50000 is alike, not more
        assert len({t[half] & 0x7FFFFFFE for t in got}) > 50000 - 20
