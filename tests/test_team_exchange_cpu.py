"""The exchange between the members of a team (csrc/mpv_exchange.h), modelled on the host: every order in which the
members of a small team can take their steps, with the kernels' own rules of who waits for whom and which area is written."""

import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "mpv_exchange.h"
extern "C" int area_of(unsigned seq) { return static_cast<int>(mpv::exchange_area(seq)); }
extern "C" unsigned long long arrival(int chiplet) { return mpv::arrival_of(chiplet); }
extern "C" int count(unsigned long long word) { return mpv::arrived(word); }
extern "C" int count_on(unsigned long long word, int chiplet) { return mpv::arrived_on(word, chiplet); }
extern "C" unsigned before_first(int one_chiplet) { return mpv::before_first_exchange(one_chiplet != 0); }
extern "C" int on_one(unsigned seq) { return mpv::on_one_chiplet(seq) ? 1 : 0; }
// the largest upper half of the arrival word, over every placement of up to `most` members from chiplet `from` on (16: of any other)
static unsigned highest(unsigned long long word, int from, int most) {
    unsigned top = static_cast<unsigned>(word >> 32);
    for (int c = from; c <= mpv::kChiplets && most > 0; ++c) {
        const unsigned t = highest(word + mpv::arrival_of(c), c, most - 1);
        top = t > top ? t : top;
    }
    return top;
}
extern "C" unsigned highest_arrival(int most) { return highest(0, 0, most); }
extern "C" int lane_waits(int rows, int lane, int size, int also) {
    return rows == 1 ? mpv::exchange_waits<1>(lane, size, also != 0) : mpv::exchange_waits<2>(lane, size, also != 0);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("exchange")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2602_16994_amd", "csrc"),
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    return ctypes.CDLL(str(d / "shim.so"))


def a_member_can_miss_a_word(size, exchanges, area_of, waits_for):
    """Token-following walks, one draw after the other: odd exchanges carry the masses, even ones the drawn token, and a
    member other than the leader goes on after a token only when the leader has.  True if in some order of the steps a
    member waits for a word that has been overwritten."""
    start = (tuple((1, False, 0) for _ in range(size)), tuple((0,) * size for _ in range(2)))
    seen, todo = {start}, [start]                     # a member: (exchange, word written, partners whose word it has)
    while todo:
        members, areas = todo.pop()
        for m, (seq, written, have) in enumerate(members):
            if seq > exchanges:
                continue
            new_areas, step = areas, None
            if not written:
                if m != 0 and seq > 1 and seq % 2 == 1 and members[0][0] < seq:
                    continue                          # the next draw has not been announced
                a = area_of(seq)
                new_areas = tuple(tuple(seq if (i, w) == (a, m) else v for w, v in enumerate(line)) for i, line in enumerate(areas))
                step = [(seq, True, 1 << m)]
            else:
                step, due = [], [p for p in range(size) if waits_for(seq, m, p) and not have >> p & 1]
                for p in due:
                    word = areas[area_of(seq)][p]
                    if word > seq:
                        return True
                    if word == seq:
                        step.append((seq, True, have | 1 << p))
                if not due:
                    step = [(seq + 1, False, 0)]
            for s in step:
                state = (members[:m] + (s,) + members[m + 1:], new_areas)
                if state not in seen:
                    seen.add(state)
                    todo.append(state)
    return False


@pytest.mark.parametrize("size", [2, 3])
def test_no_member_misses_a_word(rules, size):
    assert not a_member_can_miss_a_word(size, 5, rules.area_of, lambda seq, m, p: rules.lane_waits(1, p, size, 0))


@pytest.mark.parametrize("size,owner", [(3, 0), (3, 1), (2, 0)])
def test_the_model_finds_a_token_exchange_that_waits_for_its_owner_alone(rules, size, owner):
    """(the mistake is in the model's rule: the drawn token comes from one member, and only that one's word is waited for)"""
    assert a_member_can_miss_a_word(size, 5, rules.area_of, lambda seq, m, p: seq % 2 == 1 or p == owner)


@pytest.mark.parametrize("rows", [1, 2])
def test_every_exchange_waits_for_every_member(rules, rows):
    for size in range(1, 17):
        for lane in range(64):
            expect = lane % 16 < size and lane // 16 < rows
            assert rules.lane_waits(rows, lane, size, 0) == expect
            assert rules.lane_waits(rows, lane, size, 1) == (lane % 16 < size)


@pytest.mark.parametrize("size", [2, 15, 16])
def test_a_team_on_one_chiplet_is_told_from_one_that_is_not(rules, size):
    """The last to arrive sees every member on its own chiplet, or not: also with one member elsewhere, or on a chiplet that
    the word has no field for (16 is the largest team, 0..15 what the hardware's number can be)."""
    rules.arrival.restype = ctypes.c_ulonglong
    rules.count.argtypes = [ctypes.c_ulonglong]
    rules.count_on.argtypes = [ctypes.c_ulonglong, ctypes.c_int]
    for on in range(16):
        for other in range(16):
            word = (size - 1) * rules.arrival(on) + rules.arrival(other)
            assert rules.count(word) == size
            assert (rules.count_on(word, other) == size) == (on == other and on < 8)


def test_no_arrival_word_passes_for_an_exchange(rules):
    """The members' count lies where exchange words are written later: whatever chiplets up to 16 members run on, its upper half
    is not the number of any exchange (one on chiplet 5 and one on 4 made it 2, the number of the first exchange there)."""
    for f in (rules.before_first, rules.highest_arrival):
        f.restype = ctypes.c_uint32
    rules.on_one.argtypes = [ctypes.c_uint32]
    top = rules.highest_arrival(16)
    assert top >= 2                                   # (numbers that begin at 1 would be among them)
    for one in (0, 1):
        first, last = rules.before_first(one), rules.before_first(one) + 10 ** 9      # (more exchanges than two seconds hold)
        assert top < first and last < 2 ** 32 and rules.area_of(ctypes.c_uint32(first + 1)) == 1
        assert rules.on_one(first) == rules.on_one(last) == one


def test_the_kernels_number_exchanges_by_these_rules():
    with open(os.path.join(ROOT, "paper_2602_16994_amd", "csrc", "mpv.hip")) as f:
        text = f.read()
    starts = [line.strip() for line in text.split("\n") if ".seq = " in line]
    assert len(starts) == 2 and all(".seq = before_first_exchange(" in line for line in starts), starts


def test_the_kernels_exchange_by_these_rules():
    with open(os.path.join(ROOT, "paper_2602_16994_amd", "csrc", "mpv.hip")) as f:
        text = f.read()
    body = text[text.index("int swap_words("):]
    body = body[:body.index("\n}\n")]
    assert "exchange_area(t.seq)" in body and "exchange_waits<ROWS>(lane, t.size, also)" in body
    assert text.count("swap_words<") == text.count("swap_words") - 1       # no other way to exchange


def test_a_walk_s_position_is_performed_before_the_next_draw_is_announced():
    """The members read the position from memory when they hear of the task, so the leader waits for its store in between
    (in the source, not by what a call happens to wait for)."""
    with open(os.path.join(ROOT, "paper_2602_16994_amd", "csrc", "mpv.hip")) as f:
        text = f.read()
    handed_on = text[text.index("const int next = sample_task<E, METHOD>("):]
    handed_on = handed_on[:handed_on.index("run_node_task<E, KIND>(task, flags);")]
    assert handed_on.count("team_announce(") == 1
    before = handed_on[:handed_on.index("team_announce(")]
    assert "wait_memory();" in before[before.index("next >= 0"):]
