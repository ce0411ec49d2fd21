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

}  // namespace mpv
