"""CPU-only test of the table that keeps a thread's answers by value (csrc/kept.h)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "kept.h"
#include <cstdio>
#include <random>
struct Key { int64_t w[10]; };
struct Value { int64_t of[10]; };
static bool asked(nt::Kept<Key, Value> &t, const Key &k)          // whether it was known; a known answer must be the question's own
{
    if (const Value *v = t.find(k)) { if (memcmp(v, &k, sizeof k)) { puts("another question's answer"); exit(1); } return true; }
    Value v;
    memcpy(&v, &k, sizeof k);
    t.put(k, v);
    return false;
}
int main()
{
    std::mt19937_64 r(5);
    int lost = 0, wrong = 0;
    for (int round = 0; round < 200; ++round) {
        // two questions that differ in one word, in turn: both stay
        nt::Kept<Key, Value> &t = *new nt::Kept<Key, Value>;
        Key a, b;
        for (int64_t &w : a.w) w = (int64_t)(r() % 300);
        b = a;
        b.w[round % 10] ^= 1;
        asked(t, a); asked(t, b);
        for (int i = 0; i < 3; ++i) wrong += !asked(t, a) + !asked(t, b);
        // the layers of a network, pass after pass: none is lost
        Key layer[62];
        for (Key &k : layer)
            for (int64_t &w : k.w) w = (int64_t)(r() % 40);
        for (const Key &k : layer) asked(t, k);
        for (const Key &k : layer) lost += !asked(t, k);
        // many more than there is room for: never a wrong answer
        for (int i = 0; i < 2000; ++i) { Key k = a; k.w[i % 10] = (int64_t)(r() % 40); asked(t, k); }
        delete &t;
    }
    printf("%d %d\n", wrong, lost);
}
"""


def test_answers_are_kept_by_all_words_of_the_question(tmp_path):
    (tmp_path / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2507_11978_amd", "csrc"), "t.cpp", "-o", "t"], cwd=tmp_path, check=True)
    out = subprocess.run([str(tmp_path / "t")], check=True, capture_output=True, text=True).stdout.split()
    assert out == ["0", "0"]
