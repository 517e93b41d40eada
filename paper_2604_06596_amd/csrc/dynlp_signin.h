// Which workgroups of a launch of k_xcd_rounds share its rounds.
//
// The first workgroup that writes the launch's number into the word `turn` has its XCD chosen; workgroups of other XCDs leave.
// Those of the chosen one take a place by adding to the list; the one that chose closes the list once as many as wanted are
// there, or after `looks` looks.  How many there are is what its closing operation returned, and nothing else: it publishes that
// number under the launch's number, and all others take it from there.  (An addition that comes after the close stays in the
// list: read from there, the number depends on when it is read, and workgroups that disagree on it wait for words that nobody
// will write.)  So whoever takes part is running when the list is closed, all of them know of exactly the same ones, and every
// wait between them ends.
//
// Lists are used by turns, by parity of the launch's number: a launch clears the next one's.  The numbers of a context's launches
// must therefore follow each other.
//
// Mem carries the accesses (each of them one atomic access to a word), so that a model on the host can run them in any order:
//   unsigned read_turn();  bool set_turn(unsigned* seen, unsigned value)  compare and swap, *seen as found
//   unsigned add(parity);  unsigned look(parity);  unsigned close(parity)  what the list held before; close sets kListClosed
//   void clear(parity);  void publish(unsigned);  unsigned published()     waited on until it carries the launch's number
#pragma once

namespace dynlp {

constexpr unsigned int kListClosed = 0x80000000u;

struct SignedIn {
    int place;            // among those that share the launch's rounds, or -1: the workgroup leaves
    unsigned int groups;  // how many they are, at most `want` (place >= 0)
};

// launch: 1 .. 2^24 - 1; xcd, want: below 256.
template <class Mem>
__host__ __device__ inline SignedIn sign_in(Mem& mem, unsigned int launch, unsigned int xcd, unsigned int want, int looks) {
    const unsigned int mine = launch << 8 | xcd;
    const int parity = (int)(launch & 1u);
    unsigned int seen = mem.read_turn();
    bool chose = false;
    if (seen >> 8 != launch) {
        chose = mem.set_turn(&seen, mine);
        if (chose) seen = mine;
    }
    if (seen != mine) return SignedIn{-1, 0u};
    const unsigned int at = mem.add(parity);
    unsigned int groups;
    if (chose) {
        mem.clear(parity ^ 1);
        for (int i = 0; i < looks; ++i)
            if (mem.look(parity) >= want) break;
        const unsigned int there = mem.close(parity);
        groups = there < want ? there : want;
        mem.publish(launch << 8 | groups);
    } else {
        if (at & kListClosed) return SignedIn{-1, 0u};
        unsigned int word;
        do word = mem.published();
        while (word >> 8 != launch);  // (the workgroup that chose is running and waits for nothing)
        groups = word & 255u;
    }
    return SignedIn{at < groups ? (int)at : -1, groups};
}

}  // namespace dynlp
