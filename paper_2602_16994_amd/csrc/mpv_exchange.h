// mpv_exchange.h -- the rules that keep a team's exchanges apart (see "teams" in mpv.hip).
//
// Plain constant functions without a header of the GPU's: the kernels use them, and a model of the exchange on the host
// can be run with the same ones.
#pragma once

namespace mpv {

// A wave's lanes in rows of 16: lane 16 r + m looks after member m.
constexpr int kTeamRow = 16;

// The area that holds the words of exchange number seq: two areas take turns, so exchange s + 2 overwrites exchange s.
constexpr unsigned exchange_area(unsigned seq) { return seq & 1u; }

// Whether a lane waits for the words of member lane % 16: in `rows` rows of lanes (one at least), and in others where the
// caller says so (also).  Every exchange waits for every member, also where the words of one are enough: a member that
// waited for less could write exchange s + 1 over its words of exchange s - 1 before a slow one has read those, and the
// slow one would wait for a number that is gone.
template <int ROWS>
constexpr bool exchange_waits(int lane, int size, bool also) {
    static_assert(ROWS >= 1 && ROWS <= 4, "every exchange waits for every member");
    return (lane & (kTeamRow - 1)) < size && (lane < ROWS * kTeamRow || also);
}

// The word in which a team's members count themselves as they start: how many there are, and how many on each chiplet.
// Members on chiplets that it has no field for are nobody's neighbours.  It is word 0 of the first member's line in area 0
// and stays there until exchange words overwrite it; so the numbers of exchanges, which tell a word that has been written from
// one that has not (an exchange's number is the upper half of its words), begin above everything its upper half can hold.
constexpr int kArrivedOn = 8, kArrivedBits = 5, kChiplets = 8;
static_assert(kArrivedOn + kChiplets * kArrivedBits <= 64, "the counts of a team's arrivals fit a word");
constexpr unsigned long long arrival_of(int chiplet) {
    return 1ull + (chiplet < kChiplets ? 1ull << (kArrivedOn + kArrivedBits * chiplet) : 0ull);
}
constexpr int arrived(unsigned long long word) { return static_cast<int>(word & ((1ull << kArrivedOn) - 1ull)); }
constexpr int arrived_on(unsigned long long word, int chiplet) {
    return chiplet < kChiplets ? static_cast<int>((word >> (kArrivedOn + kArrivedBits * chiplet)) & ((1ull << kArrivedBits) - 1ull)) : 0;
}

// The number before a team's first exchange.  The top bit says for the whole launch that the team runs on one chiplet (a
// word of its own for that is one more scalar register through the task loops).  Even: the first exchange uses area 1, as the
// team's first task is announced in area 0, which the next one overwrites only when everybody has read it.
constexpr unsigned before_first_exchange(bool one_chiplet) { return one_chiplet ? 1u << 31 : 1u << 16; }
constexpr bool on_one_chiplet(unsigned seq) { return (seq >> 31) != 0u; }
static_assert(kArrivedOn + kChiplets * kArrivedBits - 32 <= 16, "an exchange's number is above the upper half of the arrival word");

}  // namespace mpv
