// Runs the marks' protocol (csrc/handshake.h, the very code the kernels run) through every order in which stores and loads of
// its workgroups may take effect, and checks that no work is lost, done too soon or done twice.  Built with g++ by
// tests/test_handshake.py, no GPU involved.
//
// A workgroup is a fiber that stops before every access.  A store first goes into its own buffer, from which it reaches the
// memory at any later time, stores of different marks in any order; a load takes what is in the memory (or its own last store of
// that mark); settle() waits until the own buffer is empty.  A look at several marks takes them one by one, upwards or
// downwards, a wait may run out after any look.  Steps that nobody else can notice are taken at once, and of two runs that have seen the same
// and left the same memory behind, which go on alike, the second is cut short.
//   interleavings meet|keep <workgroups> <keepers> <looks until a wait runs out> <settle works: 0|1>  ->  "<runs> <violations>"
//   interleavings ticks <asked>  ->  how long a share and a keeper wait at most
#include <ucontext.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <memory>
#include <string>
#include <unordered_set>
#include <vector>

#include "handshake.h"

using namespace reader;

constexpr mark_t kToken = 64 * 1234567ull, kStale = 64 * 1234566ull | kLeft;
enum Op { kStart, kStore, kLoad, kSettle, kSwap, kOver, kOrder, kDone };

struct Sim;
struct Group {
    ucontext_t ctx;
    std::unique_ptr<char[]> stack;
    std::function<void()> body;
    Op next = kStart;
    int options = 1, picked = 0;                // of its next step
    std::vector<std::pair<int, mark_t>> buffer;
    std::string history;
};
struct Sim {
    std::vector<mark_t> mem;
    std::vector<Group> groups;
    ucontext_t main;
    int now = -1;
    bool settle_works;

    void stop(Op op, int options = 1) {         // called by the running group: its next step is `op`
        Group &g = groups[now];
        g.next = op;
        g.options = options;
        swapcontext(&g.ctx, &main);
    }
    void note(mark_t v) { groups[now].history.append(reinterpret_cast<char *>(&v), sizeof v); }
};
static Sim *sim;

static void run_group() {
    sim->groups[sim->now].body();
    sim->groups[sim->now].next = kDone;
}

struct Wave {
    int at(const mark_t *m) const { return (int)(m - sim->mem.data()); }
    void set(mark_t *m, mark_t v) const {
        sim->stop(kStore);
        sim->groups[sim->now].buffer.push_back({at(m), v});
        sim->note(1);
    }
    mark_t get(const mark_t *m) const {
        sim->stop(kLoad);
        mark_t v = *m;
        for (auto &e : sim->groups[sim->now].buffer)
            if (e.first == at(m)) v = e.second;
        sim->note(v);
        return v;
    }
    void settle() const {
        sim->stop(kSettle);
        sim->note(2);
    }
    bool swap(mark_t *m, mark_t from, mark_t to) const {
        sim->stop(kSwap);
        const bool done = *m == from;
        if (done) *m = to;
        sim->note(done);
        return done;
    }
    template <class F>
    bool wait_until(F &&f, unsigned long long looks) const {
        for (unsigned long long look = 1;; ++look) {
            if (f()) return true;
            if (look == looks) return false;
            sim->stop(kOver, 2);
            const int over = sim->groups[sim->now].picked;
            sim->note(over);
            if (over) return false;
        }
    }
    // all n marks from `m` on, upwards or downwards
    void look(const mark_t *m, int n, mark_t *v) const {
        sim->stop(kOrder, n > 1 ? 2 : 1);
        const int down = sim->groups[sim->now].picked;
        sim->note(down);
        for (int i = 0; i < n; ++i) {
            const int k = down ? n - 1 - i : i;
            v[k] = get(m + k);
        }
    }
};

struct Check {
    int n, keepers, looks;
    std::vector<int> merged, acted;
    bool too_soon;
};

static void set_up(Check &c, bool meeting) {
    c.merged.assign(c.n, 0);
    c.acted.assign(c.keepers, 0);
    c.too_soon = false;
    const int n = c.n, keepers = c.keepers, looks = c.looks;
    sim->mem.assign(n + keepers + 1, kStale);                 // arrivals, keepers, whether any keeper has left
    mark_t *marks = sim->mem.data(), *kept = marks + n, *any_left = kept + keepers;
    auto everybody = [marks, n](Wave w, mark_t *seen) {
        w.look(marks, n, seen);
        return std::all_of(seen, seen + n, [](mark_t v) { return (v & ~kMarkBits) == kToken; });
    };
    auto all_arrived = [marks, n] { return std::all_of(marks, marks + n, [](mark_t v) { return (v & ~kMarkBits) == kToken; }); };
    auto act = [&c, all_arrived](int k) {
        if (!all_arrived()) c.too_soon = true;
        ++c.acted[k];
    };
    sim->groups.clear();
    sim->groups.resize(meeting ? n : n + keepers);
    for (int i = 0; i < (int)sim->groups.size(); ++i) {
        Group &g = sim->groups[i];
        if (meeting)
            g.body = [=, &c] {
                std::vector<mark_t> seen(n);
                if (!meet(Wave(), marks + i, kToken | (mark_t)1 << kXccShift, [&] { return everybody(Wave(), seen.data()); }, looks)) return;
                if (!all_arrived()) c.too_soon = true;
                for (int s = 0; s < n; ++s)
                    if (s == i || (seen[s] & kStateBits) == kLeft) ++c.merged[s];
            };
        else if (i < n)
            g.body = [=, &c] {
                std::vector<mark_t> seen(n);
                if (arrive(Wave(), marks + i, any_left, kToken))
                    act_for_those_who_left(Wave(), kept, keepers, kToken, [&] { return everybody(Wave(), seen.data()); }, act);
            };
        else
            g.body = [=] {
                std::vector<mark_t> seen(n);
                if (keep(Wave(), kept + (i - n), any_left, kToken, [&] { return everybody(Wave(), seen.data()); }, looks)) act(i - n);
            };
        g.stack.reset(new char[32768]);
        getcontext(&g.ctx);
        g.ctx.uc_stack.ss_sp = g.stack.get();
        g.ctx.uc_stack.ss_size = 32768;
        g.ctx.uc_link = &sim->main;
        makecontext(&g.ctx, run_group, 0);
    }
}

struct Step {
    int group, pick, flush;                     // flush >= 0: that entry of the group's buffer reaches the memory
};

static std::vector<Step> steps() {
    std::vector<Step> out;
    for (int i = 0; i < (int)sim->groups.size(); ++i) {
        const Group &g = sim->groups[i];
        if (g.next == kStart || g.next == kStore || g.next == kOver || g.next == kOrder ||
            (g.next == kSettle && (g.buffer.empty() || !sim->settle_works))) {     // (its own affair)
            out.clear();
            for (int o = 0; o < g.options; ++o) out.push_back({i, o, -1});
            return out;
        }
        for (int e = 0; e < (int)g.buffer.size(); ++e) {
            bool first = true;                  // (stores of one mark stay in order)
            for (int d = 0; d < e; ++d) first &= g.buffer[d].first != g.buffer[e].first;
            if (first) out.push_back({i, 0, e});
        }
        if (g.next == kLoad || (g.next == kSwap && g.buffer.empty())) out.push_back({i, 0, -1});
    }
    return out;
}

static void take(const Step &s) {
    Group &g = sim->groups[s.group];
    if (s.flush >= 0) {
        sim->mem[g.buffer[s.flush].first] = g.buffer[s.flush].second;
        g.buffer.erase(g.buffer.begin() + s.flush);
        return;
    }
    sim->now = s.group;
    g.picked = s.pick;
    swapcontext(&sim->main, &g.ctx);
}

static std::string state(const Check &c) {
    std::string k(reinterpret_cast<char *>(sim->mem.data()), sim->mem.size() * sizeof(mark_t));
    k += c.too_soon ? '!' : '.';
    for (auto &g : sim->groups) {
        k += '|';
        k += g.history;
        k += (char)('a' + g.next);
        for (auto &e : g.buffer) {
            k += (char)e.first;
            k.append(reinterpret_cast<const char *>(&e.second), sizeof e.second);
        }
    }
    return k;
}

int main(int argc, char **argv) {
    if (argc == 3 && std::string(argv[1]) == "ticks") {
        const int ticks = wait_ticks(atoll(argv[2]));
        std::printf("%d %lld\n", ticks, (unsigned)ticks * kKeeperPatience);
        return 0;
    }
    if (argc != 6) return 2;
    const bool meeting = std::string(argv[1]) == "meet";
    Check c;
    c.n = atoi(argv[2]);
    c.keepers = atoi(argv[3]);
    c.looks = atoi(argv[4]);
    Sim s;
    sim = &s;
    s.settle_works = atoi(argv[5]) != 0;
    std::unordered_set<std::string> known;
    std::vector<std::vector<int>> open{{}};
    long runs = 0, violations = 0;
    while (!open.empty()) {
        std::vector<int> path = open.back();
        open.pop_back();
        set_up(c, meeting);
        for (int choice : path) take(steps()[choice]);
        ++runs;
        for (;;) {
            const std::vector<Step> next = steps();
            if (next.empty()) {
                bool ok = !c.too_soon;
                if (meeting) ok &= std::all_of(c.merged.begin(), c.merged.end(), [](int m) { return m >= 1; });   // (twice is the same bytes)
                else ok &= std::all_of(c.acted.begin(), c.acted.end(), [](int m) { return m == 1; });
                if (!ok) ++violations;
                break;
            }
            if (!known.insert(state(c)).second) break;
            for (int o = 1; o < (int)next.size(); ++o) {
                open.push_back(path);
                open.back().push_back(o);
            }
            path.push_back(0);
            take(next[0]);
        }
    }
    std::printf("%ld %ld\n", runs, violations);
    return 0;
}
