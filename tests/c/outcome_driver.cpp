// The rule by which workgroups that wait for each other keep or give up their
// launch (outcome.hpp), over every order of events: each workgroup stores its
// word of the last meeting, reads the words until all are there or it stops
// waiting, and stores its results if it may.  In every end of every order all
// workgroups store or none does, and every wait ends.  Prints "outcome driver
// ok" and exits 0 when that holds.
#include <cstdint>
#include <cstdio>
#include <set>
#include <vector>

#include "../../paper_2209_06478_amd/csrc/outcome.hpp"

enum Pc : int { START, WAITING, PASSED, LEFT, STORED };
struct State {
    std::vector<int> pc;
    uint32_t word = 0;
    bool operator<(const State &o) const { return pc != o.pc ? pc < o.pc : word < o.word; }
};

// a load returns the word, or what it was before (`stale`)
struct Word {
    uint32_t *w;
    bool stale;
    uint32_t load() const { return stale ? (uint32_t)dsm::OUTCOME_OPEN : *w; }
    uint32_t swap(uint32_t from, uint32_t to) const {
        const uint32_t was = *w;
        if (was == from) *w = to;
        return was;
    }
};

static std::set<State> seen;
static long ends = 0, kept = 0, split = 0, stuck = 0;

static void explore(const State &s) {
    if (!seen.insert(s).second) return;
    bool moved = false;
    bool all = true;
    for (int p : s.pc) all = all && p != START;
    auto go = [&](size_t g, int pc, uint32_t word) {
        State t = s;
        t.pc[g] = pc;
        t.word = word;
        moved = true;
        explore(t);
    };
    for (size_t g = 0; g < s.pc.size(); g++) {
        if (s.pc[g] == START) go(g, WAITING, s.word);  // (or it comes much later: every other order)
        if (s.pc[g] == WAITING) {
            if (all) go(g, PASSED, s.word);
            for (int late = 0; late < 2; late++)
                for (int stale = 0; stale < 2; stale++) {
                    uint32_t w = s.word;
                    if (dsm::outcome_gives_up(Word{&w, stale != 0}, late != 0)) go(g, LEFT, w);
                }
        }
        if (s.pc[g] == PASSED) {
            uint32_t w = s.word;
            const bool ok = dsm::outcome_keeps(Word{&w, false});
            go(g, ok ? STORED : LEFT, w);
        }
    }
    if (moved) return;
    ends++;
    size_t st = 0, fin = 0;
    for (int p : s.pc) {
        st += p == STORED;
        fin += p == STORED || p == LEFT;
    }
    kept += st == s.pc.size();
    split += st != 0 && st != s.pc.size();
    stuck += fin != s.pc.size();
}

int main() {
    for (size_t n = 1; n <= 4; n++)
        for (uint32_t first : {(uint32_t)dsm::OUTCOME_OPEN, (uint32_t)dsm::OUTCOME_GIVEN_UP}) {
            seen.clear();
            ends = kept = split = stuck = 0;
            State s;
            s.pc.assign(n, START);
            s.word = first;
            explore(s);
            std::printf("%zu workgroups, word %u at the start: %zu states, %ld ends, %ld kept, %ld split, %ld stuck\n", n,
                        first, seen.size(), ends, kept, split, stuck);
            if (split || stuck || ends == 0 || (kept > 0) != (first == dsm::OUTCOME_OPEN)) return 1;
        }
    std::printf("outcome driver ok\n");
    return 0;
}
