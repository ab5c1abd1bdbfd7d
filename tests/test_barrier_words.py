"""The words by which a resident team meets (csrc/words.h), enumerated on the host over the queries
that one team of a batch solves one after the other: at no barrier may a word that an earlier one left
read as the awaited one."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
U64, U32 = ctypes.c_ulonglong, ctypes.c_uint32


@pytest.fixture(scope="module")
def words(tmp_path_factory):
    d = tmp_path_factory.mktemp("words")
    src = d / "words.cpp"
    src.write_text('#include "words.h"\nextern "C" {\n'
                   "unsigned long long t_tag(uint32_t b) { return bar_tag(b); }\n"
                   "unsigned long long t_tag_mask() { return kTag; }\n"
                   "uint32_t t_words(uint32_t b, uint32_t W) { return bar_words(b, W); }\n"
                   "unsigned long long t_count(uint32_t next, uint32_t c) { return count_word(next, c); }\n"
                   "int t_is_for(unsigned long long w, uint32_t next) { return count_is_for(w, next); }\n"
                   "uint32_t t_count_words(uint32_t W) { return count_words(W); }\n"
                   "void t_empty(unsigned long long *bar, uint32_t b, uint32_t W, uint32_t wg) {\n"
                   "    bar_put_empty(b, W, wg, [&](uint32_t i, unsigned long long x) { bar[i] = x; }); }\n"
                   "uint32_t t_team(uint32_t W) { return team_words(W); }\n}\n")
    lib = str(d / "libwords.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1903_12085_amd", "csrc"), str(src), "-o", lib], check=True)
    w = ctypes.CDLL(lib)
    for f in (w.t_tag, w.t_tag_mask, w.t_count):
        f.restype = U64
    w.t_tag.argtypes, w.t_words.argtypes = [U32], [U32, U32]
    w.t_count.argtypes, w.t_is_for.argtypes = [U32, U32], [U64, U32]
    return w


def stale_counts(w, queries, nb=0):
    """(query, phase) pairs in which a count word of an earlier phase would be taken for the awaited one.
    queries: (shares, phases). One barrier sets a query up, one ends each phase; a sharing phase awaits
    the count that carries the number of the barrier after it, and then holds it."""
    held, bad = 0, []
    for q, (shares, phases) in enumerate(queries):
        nb += 1
        for k in range(phases):
            nb = (nb + 1) & 0xFFFFFFFF
            if not shares:
                continue
            if w.t_is_for(held, nb):
                bad.append((q, k))
            held = w.t_count(nb, 1024)
            assert w.t_is_for(held, nb) and held & 0xFFFFFFFF == 1024
    return bad


@pytest.mark.parametrize("first", [1, 2, 9, 30])
def test_counts_of_an_earlier_query_are_never_current(words, first):
    for middle in range(0, 200):
        assert not stale_counts(words, [(1, first), (0, middle), (1, 40)]), middle
    for a in range(0, 62):  # two queries without shared records in between, and none
        assert not stale_counts(words, [(1, first), (0, a), (0, 27 - a % 27), (1, 3), (1, 3)]), a


def test_counts_of_a_long_batch_are_never_current(words):
    assert not stale_counts(words, [(1, 5), (0, 60000), (1, 70000)])
    assert not stale_counts(words, [(q % 3 != 1, 1 + q * 7 % 61) for q in range(2000)])


def test_words_of_a_team_do_not_overlap(words):
    for W in (1, 2, 32, 256):
        starts = {words.t_words(b, W) for b in range(8)} | {words.t_count_words(W)}
        assert sorted(starts) == [0, 8 * W, 16 * W] and words.t_team(W) == 24 * W


def stale_values(w, phases, W=2):
    """(query, phase, workgroup, word) where the minD (0) or threshold (1) word of a barrier carries its
    tag before it is written, over the queries of one team. A phase writes a workgroup's two words; what a
    set-up writes is bar_put_empty's."""
    bar, nb, bad = (U64 * w.t_team(W))(), 0, []
    for q, count in enumerate(phases):
        for wg in range(W):
            w.t_empty(bar, nb, W, wg)
        nb += 1
        for k in range(count):
            for wg in range(W):
                for i in (0, 1):
                    at = w.t_words(nb, W) + 8 * wg + i
                    if bar[at] & w.t_tag_mask() == w.t_tag(nb):
                        bad.append((q, k, wg, i))
                    bar[at] = w.t_tag(nb) | 77
            nb += 1
    return bad


def test_values_of_an_earlier_query_are_never_current(words):
    for ones in range(70):  # sources without out-edges: one phase each
        assert not stale_values(words, [4] + [1] * ones + [4, 2, 9]), ones
    assert not stale_values(words, [1 + q * 5 % 17 for q in range(400)] + [1] * 100 + [3] * 50)
