// Every interleaving of the workgroups of a launch that sign in (csrc/dynlp_signin.h, the code the GPU runs), on the host.
//
//   sign_in_model WANT OWN OTHERS SLOTS LOOKS LAUNCHES PLANT
//
// OWN workgroups start on XCD 0 and OTHERS on XCD 1, in any order, at most SLOTS of an XCD at a time (a workgroup that takes part
// holds its slot until all that it knows of have met).  A launch begins with any memory that one before it can leave.  PLANT: a
// mistake put into the model: 1 = the number of workgroups is read from the list after the close, 2 = a launch's number is left out.
// Prints "ok STATES" or what went wrong.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <string>
#include <vector>

#include "dynlp_signin.h"

using namespace dynlp;

namespace {

int g_want, g_slots, g_looks, g_plant;

struct Memory {
    unsigned turn = 0, list[2] = {0, 0}, groups = 0;
};

// What a workgroup has got from its accesses so far.  Its code is run from the start on these, up to the access after them.
using History = std::vector<unsigned>;

struct Stop {};  // at the access that has not been made yet

struct Replay {
    const History* past;
    size_t at = 0;
    Memory* memory = nullptr;  // the access is made on it
    bool spins = false;
    unsigned got = 0;

    // A word that is polled without a bound: the same answer again changes nothing, so only another one is a step.
    template <class F>
    unsigned access(F f, bool polled = false) {
        if (at < past->size()) {
            was_poll = polled;
            return (*past)[at++];
        }
        got = f(*memory);
        spins = polled && was_poll && past->back() == got;
        throw Stop{};
    }
    bool was_poll = false;

    unsigned read_turn() { return access([](Memory& m) { return m.turn; }); }
    bool set_turn(unsigned* seen, unsigned value) {
        // (found word; set where it is what was seen)
        const unsigned expected = *seen;
        *seen = access([=](Memory& m) {
            const unsigned found = m.turn;
            if (found == expected) m.turn = value;
            return found;
        });
        return *seen == expected;
    }
    unsigned add(int p) {
        return access([=](Memory& m) { return m.list[p]++; });
    }
    unsigned look(int p) {
        return access([=](Memory& m) { return m.list[p]; });
    }
    unsigned close(int p) {
        return access([=](Memory& m) {
            const unsigned was = m.list[p];
            m.list[p] |= kListClosed;
            return was;
        });
    }
    void clear(int p) {
        access([=](Memory& m) { return m.list[p] = 0u; });
    }
    void publish(unsigned word) {
        access([=](Memory& m) { return m.groups = word; });
    }
    unsigned published() {
        // planted: the list itself, as the one that chose read it before it closed it
        if (g_plant == 1)
            return access([=](Memory& m) {
                const unsigned t = m.list[launch & 1];
                const unsigned n = t & ~kListClosed;
                return t & kListClosed ? launch << 8 | (n < (unsigned)g_want ? n : (unsigned)g_want) : 0u;
            }, true);
        return access([](Memory& m) { return m.groups; }, true);
    }
    unsigned launch = 0;
};

enum Phase : unsigned char { kNotStarted, kSigning, kMeeting, kGone };

struct State {
    Memory memory;
    std::vector<Phase> phase;
    std::vector<History> past;
    std::vector<SignedIn> in;
    // (workgroups of one XCD are alike: which of them has come how far makes no difference)
    std::string key(size_t own) const {
        std::vector<std::string> each(phase.size());
        for (size_t i = 0; i < phase.size(); ++i) {
            each[i] += (char)phase[i];
            if (phase[i] == kSigning) each[i].append(reinterpret_cast<const char*>(past[i].data()), past[i].size() * sizeof(unsigned));
            each[i].append(reinterpret_cast<const char*>(&in[i]), sizeof in[i]);
            each[i] += '|';
        }
        std::sort(each.begin(), each.begin() + (long)own);
        std::sort(each.begin() + (long)own, each.end());
        std::string k(reinterpret_cast<const char*>(&memory), sizeof memory);
        for (const std::string& e : each) k += e;
        return k;
    }
};

std::string g_wrong;
size_t g_states = 0;

// One step of workgroup i; false: none is possible, or it would change nothing.
bool step(State& s, size_t i, size_t own, unsigned launch) {
    const unsigned xcd = i < own ? 0u : 1u;
    if (s.phase[i] == kGone) return false;
    if (s.phase[i] == kNotStarted) {
        int held = 0;
        for (size_t j = 0; j < s.phase.size(); ++j)
            if ((j < own) == (i < own) && (s.phase[j] == kSigning || s.phase[j] == kMeeting)) ++held;
        if (held >= g_slots) return false;
        s.phase[i] = kSigning;
        return true;
    }
    if (s.phase[i] == kMeeting) {  // leaves when everybody it knows of is there or has been there
        unsigned there = 0;
        for (const SignedIn& x : s.in) there += x.place >= 0 && (unsigned)x.place < s.in[i].groups ? 1u : 0u;
        if (there < s.in[i].groups) return false;
        s.phase[i] = kGone;
        return true;
    }
    Replay r;
    r.past = &s.past[i];
    r.memory = &s.memory;
    r.launch = launch;
    try {
        const SignedIn in = sign_in(r, launch, xcd, (unsigned)g_want, g_looks);
        s.in[i] = in;
        s.phase[i] = in.place < 0 ? kGone : kMeeting;
        return true;
    } catch (const Stop&) {
        if (r.spins) return false;
        s.past[i].push_back(r.got);
        return true;
    }
}

// What a launch has to come to: at least one workgroup, places 0 .. groups - 1, and all know the same number.
std::string check(const State& s) {
    unsigned groups = 0, part = 0;
    for (const SignedIn& x : s.in)
        if (x.place >= 0) {
            if (groups && x.groups != groups) return "workgroups disagree on how many they are";
            groups = x.groups;
            ++part;
        }
    if (!part) return "no workgroup takes part";
    if (part != groups || groups > (unsigned)g_want) return "as many places as workgroups";
    for (unsigned p = 0; p < groups; ++p) {
        unsigned n = 0;
        for (const SignedIn& x : s.in) n += x.place == (int)p ? 1u : 0u;
        if (n != 1) return "a place is taken by one workgroup";
    }
    return "";
}

void explore(const State& first, size_t own, unsigned launch, std::set<std::string>& ends, std::vector<Memory>& left) {
    std::set<std::string> seen;
    std::vector<State> todo{first};
    seen.insert(first.key(own));
    while (!todo.empty() && g_wrong.empty()) {
        const State s = todo.back();
        todo.pop_back();
        ++g_states;
        bool moved = false, all_gone = true;
        for (size_t i = 0; i < s.phase.size(); ++i) {
            all_gone = all_gone && s.phase[i] == kGone;
            State t = s;
            if (!step(t, i, own, launch)) continue;
            moved = true;
            if (seen.insert(t.key(own)).second) todo.push_back(t);
        }
        if (all_gone) {
            const std::string wrong = check(s);
            if (!wrong.empty()) g_wrong = wrong;
            if (ends.insert(std::string(reinterpret_cast<const char*>(&s.memory), sizeof s.memory)).second) left.push_back(s.memory);
        } else if (!moved) {
            const std::string wrong = check(s);
            g_wrong = "a wait that does not end" + (wrong.empty() ? "" : ": " + wrong);
        }
    }
}

}  // namespace

int main(int argc, char** argv) {
    if (argc != 8) return 2;
    g_want = std::atoi(argv[1]);
    const size_t own = (size_t)std::atoi(argv[2]), others = (size_t)std::atoi(argv[3]);
    g_slots = std::atoi(argv[4]);
    g_looks = std::atoi(argv[5]);
    const int launches = std::atoi(argv[6]);
    g_plant = std::atoi(argv[7]);
    std::vector<Memory> begin{Memory{}};
    unsigned number = 0;
    for (int l = 0; l < launches && g_wrong.empty(); ++l) {
        ++number;
        if (g_plant == 2 && l == 1) ++number;
        std::set<std::string> ends;
        std::vector<Memory> left;
        for (const Memory& m : begin) {
            State s;
            s.memory = m;
            s.phase.assign(own + others, kNotStarted);
            s.past.resize(own + others);
            s.in.assign(own + others, SignedIn{-1, 0u});
            explore(s, own, number, ends, left);
            if (!g_wrong.empty()) break;
        }
        begin = left;
    }
    if (!g_wrong.empty()) {
        std::printf("wrong: %s\n", g_wrong.c_str());
        return 1;
    }
    std::printf("ok %zu\n", g_states);
    return 0;
}
