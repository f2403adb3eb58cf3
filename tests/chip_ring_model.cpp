// The exchange of words between the workgroups of a factor (csrc/eig_chip_ring.h), run one memory access at a time in any order: every
// workgroup's stores, looks and emptyings are single steps, a workgroup can be stopped before each of them for as long as the others
// can go on, and what it has emptied becomes visible at any time up to its next publication.  Prints "ok", or what went wrong.
//   chip_ring_model RULE ORDERS      RULE: ring, or unacknowledged (a workgroup leaves without a receipt; the model must see that fail)
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <string>
#include <vector>
#include "eig_chip_ring.h"

struct Unacknowledged {
    static int slot(int t) { return t & (CHIP_RING - 1); }
    static bool leaves(int r0, int nr, int t) { return r0 + nr <= t; }
    static int receipt(int, int, int) { return -1; }
    static int first(int t) { return t; }
    static int emptied(int t) { return t - 1; }
};

constexpr int EMPTY = -1;
typedef std::mt19937 Rng;

struct Memory {
    std::vector<int> word[2][CHIP_RING];      // [half][slot][row]: the column that the word was published for
    explicit Memory(int rows) { for (auto &h : word) for (auto &s : h) s.assign(rows, EMPTY); }
};

template <class Rule> struct Launch {
    struct Store { int half, slot, row; };
    struct Workgroup {
        int r0, nr, t = 0, at = 0;
        enum { BEGIN, PUBLISH, GATHER, GONE } phase = BEGIN;
        std::vector<int> unread;
        std::vector<Store> emptying;          // stores on their way
    };
    Memory &mem;
    const int half, m, steps;
    std::vector<Workgroup> wgs;
    std::string fault;
    Rng &rng;

    Launch(Memory &mem_, int half_, int m_, int rows, int steps_, Rng &rng_) : mem(mem_), half(half_), m(m_), steps(steps_), rng(rng_) {
        for (int r0 = 0; r0 < m; r0 += rows) {
            Workgroup w;
            w.r0 = r0;
            w.nr = std::min(rows, m - r0);
            for (int r = r0; r < r0 + w.nr; ++r)
                for (int s = 0; s < CHIP_RING; ++s) w.emptying.push_back({half ^ 1, s, r});      // the next launch's half
            wgs.push_back(w);
        }
        for (int s = 0; s < CHIP_RING; ++s)
            for (int r = 0; r < m; ++r)
                if (mem.word[half][s][r] != EMPTY) fault = "a launch began with a word of an earlier one";
    }
    int pick(int n) { return (int)(rng() % (unsigned)n); }
    void empty_one(Workgroup &w) {
        const int k = pick((int)w.emptying.size());
        const Store s = w.emptying[k];
        mem.word[s.half][s.slot][s.row] = EMPTY;
        w.emptying.erase(w.emptying.begin() + k);
    }
    // one memory access; false: nothing that it can do now
    bool step(Workgroup &w) {
        if (!w.emptying.empty() && (w.phase == Workgroup::GONE || w.phase == Workgroup::PUBLISH || pick(3) == 0)) {   // (all of it before a publication)
            empty_one(w);
            return true;
        }
        auto &slot = mem.word[half][Rule::slot(w.t)];
        switch (w.phase) {
            case Workgroup::BEGIN:
                if (w.t == steps) {
                    w.phase = Workgroup::GONE;
                } else if (Rule::leaves(w.r0, w.nr, w.t)) {
                    const int row = Rule::receipt(w.r0, w.nr, w.t);
                    if (row >= 0) slot[row] = w.t;
                    w.phase = Workgroup::GONE;
                } else {
                    w.phase = Workgroup::PUBLISH;
                    w.at = 0;
                }
                return true;
            case Workgroup::PUBLISH:
                slot[w.r0 + w.at] = w.t;
                if (++w.at == w.nr) {
                    w.phase = Workgroup::GATHER;
                    for (int r = Rule::first(w.t); r < m; ++r) w.unread.push_back(r);
                }
                return true;
            case Workgroup::GATHER: {
                std::vector<int> there;
                for (int k = 0; k < (int)w.unread.size(); ++k)
                    if (slot[w.unread[k]] != EMPTY) there.push_back(k);
                if (there.empty()) {
                    if (w.emptying.empty()) return false;
                    empty_one(w);
                    return true;
                }
                const int k = there[pick((int)there.size())];
                if (slot[w.unread[k]] != w.t) fault = "column " + std::to_string(w.t) + " took a word of column " + std::to_string(slot[w.unread[k]]);
                w.unread.erase(w.unread.begin() + k);
                if (w.unread.empty()) {
                    const int done = Rule::emptied(w.t);
                    if (done >= 0)
                        for (int r = w.r0; r < w.r0 + w.nr; ++r) w.emptying.push_back({half, Rule::slot(done), r});
                    ++w.t;
                    w.phase = Workgroup::BEGIN;
                }
                return true;
            }
            default: return false;
        }
    }
    // `late` moves only when nobody else can (-1: nobody is late), up to `burst` accesses at a time
    void run(int late, int burst) {
        const int n = (int)wgs.size();
        while (fault.empty()) {
            bool moved = false;
            if (late < 0) {
                const int first = pick(n);
                for (int k = 0; k < n && !moved; ++k) moved = step(wgs[(first + k) % n]);
            } else {
                for (bool on = true; on && fault.empty();) {
                    on = false;
                    const int first = pick(n);
                    for (int k = 0; k < n; ++k)
                        if ((first + k) % n != late) on |= step(wgs[(first + k) % n]);
                }
                for (int k = 1 + pick(burst); k > 0 && fault.empty(); --k) moved |= step(wgs[late]);
            }
            if (!moved) break;
        }
        for (auto &w : wgs)
            if (fault.empty() && (w.phase != Workgroup::GONE || !w.emptying.empty()))
                fault = "workgroup of rows " + std::to_string(w.r0) + ".. waits for ever in column " + std::to_string(w.t);
    }
};

template <class Rule> std::string model(int orders) {
    struct Shape { int m, rows; };
    const Shape shapes[] = {{1, 4}, {2, 1}, {3, 2}, {5, 1}, {9, 4}, {12, 4}, {13, 3}, {20, 8}, {24, 5}};
    Rng rng(7);
    for (int o = 0; o < orders; ++o)
        for (const Shape &s : shapes) {
            const int n = (s.m + s.rows - 1) / s.rows;
            for (int late = -1; late < n; ++late)
                for (int burst : {1, 4}) {
                    Memory mem(s.m);
                    int m = s.m, turn = 0;
                    while (m > 0) {      // some columns a launch; the last one takes what is left
                        const int steps = m > 4 && turn < 3 ? 1 + (int)(rng() % (unsigned)(m - 1)) : m, rows = std::max(1, s.rows - turn);
                        Launch<Rule> L(mem, turn & 1, m, rows, steps, rng);
                        L.run(late < (int)L.wgs.size() ? late : -1, burst);
                        if (!L.fault.empty())
                            return std::to_string(m) + " rows, " + std::to_string(rows) + " per workgroup, late " + std::to_string(late) + ": " + L.fault;
                        m -= steps;
                        ++turn;
                    }
                }
        }
    return "ok";
}

int main(int argc, char **argv) {
    const int orders = argc > 2 ? atoi(argv[2]) : 20;
    printf("%s\n", (argc > 1 && !strcmp(argv[1], "unacknowledged") ? model<Unacknowledged>(orders) : model<ChipRing>(orders)).c_str());
    return 0;
}
