// Random schedules through plan_rounds and build_strips, executed entry by entry against the serial semantics.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <algorithm>
#include "strips.hpp"
using namespace adpsgd_impl;
int main() {
    std::mt19937 rng(1);
    long its = 0, rounds = 0;
    for (int trial = 0; trial < 4000; ++trial) {
        int n = 2 + rng() % 20, K = 1 + rng() % 150, T = rng() % 12, look = rng() % 2 ? std::min<int>(K, rng() % (T + 3)) : 0;
        int A = K - look; bool comp = rng() % 3 == 0, extra = rng() % 3 == 0, renum = rng() % 2;
        int n_slots = T + 1 + rng() % 20, window = T + 1 + rng() % 10; if (window > n_slots) window = n_slots;
        // a handle whose T_max is beyond the slots of its workspace (4096 at most) and the taus of its calls
        const bool far = rng() % 4 == 0;
        if (far) window = strip_window(100 + rng() % 50, false, 0, n_slots);
        std::vector<int> w(K), nb(K), tau(K), carried(K, -1);
        int npend = rng() % 2 ? rng() % (std::min(K, T) + 1) : 0;   // leading events that may be carried
        std::vector<int> sl(n_slots); for (int i = 0; i < n_slots; ++i) sl[i] = i; std::shuffle(sl.begin(), sl.end(), rng);
        int used = 0; bool anyc = false;
        std::vector<int64_t> ep(K + 1, 0); std::vector<int32_t> ea, eb;
        for (int k = 0; k < K; ++k) {
            w[k] = rng() % n; do nb[k] = rng() % n; while (nb[k] == w[k] && rng() % 8);
            tau[k] = rng() % (std::min(k, T) + 1);
            if (k < npend && k < T && rng() % 2) { tau[k] = k + 1 + rng() % (T - k); carried[k] = sl[used++]; anyc = true; }
            if (extra && n >= 6 && rng() % 3 == 0) { int a, b; do { a = rng() % n; b = rng() % n; } while (a == b || a == w[k] || b == w[k] || a == nb[k] || b == nb[k]); ea.push_back(a); eb.push_back(b); }
            ep[k + 1] = ea.size();
        }
        if (far) renum = false;
        Plan plan; std::string err;
        int rc = plan_rounds(n, K, w.data(), nb.data(), tau.data(), n_slots, true, plan, err, extra ? ep.data() : nullptr, ea.data(), eb.data(), comp, A, anyc ? carried.data() : nullptr);
        if (rc) { continue; }
        std::vector<WorkerData> data(n); for (int i = 0; i < n; ++i) { data[i].features = (void*)(uintptr_t)(0x1000 + i); data[i].targets = (void*)(uintptr_t)(0x2000 + i); data[i].ld = 5; data[i].rows = 3; }
        int teamsv[4] = {12, 6, 4, 2}; int teams = teamsv[rng() % 4], P = teams / 2;
        StripCall c{n, n_slots, window, K, A, w.data(), nb.data(), tau.data(), nullptr, 0.5f, extra ? ep.data() : nullptr, ea.data(), eb.data(), &plan, anyc ? carried.data() : nullptr, data.data(), renum, 7u, 3};
        StripProgram pr;
        auto die = [&](const char* m) { printf("trial %d: %s\n", trial, m); exit(1); };
        if (!build_strips(c, teams, pr)) die("no order");
        if ((int64_t)pr.recs.size() != (pr.iterations + 3) * pr.rec_len || pr.rec_len > kStripMaxRec || pr.rec_len < 2 + 4 * P) die("size");
        its += pr.iterations; rounds += plan.n_rounds;
        // simulate
        std::vector<std::vector<int>> ver(n);            // events applied per row
        std::vector<int> team_load(teams, -1), team_when(teams, -1), gdone(K, -1), appl(K, 0);
        int cap = renum ? pr.n_slots : n_slots; if (renum && pr.n_slots > std::max(window, 1)) die("slots exceed window");
        std::vector<int> slot_has(cap, -1);
        for (int k = 0; k < K; ++k) if (anyc && carried[k] >= 0) { slot_has[pr.slot[k]] = k; gdone[k] = -2; if (!renum && pr.slot[k] != carried[k]) die("carried slot"); }
        std::vector<std::pair<int,int>> finish;   // (event, slot) of the previous record, written at its end
        int evc = 0;
        for (int64_t it = 0; it < pr.iterations; ++it) {
            const StripEntry* r = &pr.recs[it * pr.rec_len];
            for (auto& f : finish) slot_has[f.second] = f.first, gdone[f.first] = it - 1;
            finish.clear();
            std::vector<int> uprow;
            int nu = r[0].x; if (1 + 4 * P + nu > pr.rec_len) die("updates overflow");
            for (int u = 0; u < nu; ++u) {
                if (u % 4 == 0) uprow.clear();
                const StripEntry& e = r[1 + 4 * P + u];
                if (e.w & kStripEmpty) continue;
                int i = e.x & 0xFFFF, j = e.x >> 16;
                for (int x : uprow) if (x == i || x == j) die("batch rows clash");
                uprow.push_back(i); uprow.push_back(j);
                if (e.w & kStripAverage) { ver[i].push_back(-1); ver[j].push_back(-1); continue; }
                int k = slot_has[e.y]; if (k < 0) die("empty slot");
                if (w[k] != i || nb[k] != j) die("wrong gradient in slot");
                if (gdone[k] == -1) die("not done");
                ver[i].push_back(k); if (j != i) ver[j].push_back(k); appl[k] = 1; slot_has[e.y] = -1;
            }
            // evaluations
            int ne = __builtin_popcount(r[0].z), last = -1; if (ne > P) die("evals");
            for (int q = 0; q < ne; ++q) {
                const StripEntry &a = r[1 + 2 * q], &b = r[2 + 2 * q];
                int team = a.x, k = b.z; if (team <= last || !(r[0].z >> team & 1)) die("team order"); last = team;
                if (team_load[team] != k || team_when[team] >= it) die("not loaded"); team_load[team] = -1;
                if ((int)a.z != w[k]) die("worker");
                int s = k - tau[k]; 
                // row version: own updates with event < s exactly
                std::vector<int> want; for (int m = 0; m < std::min(s, A); ++m) { if (w[m] == w[k] || nb[m] == w[k]) want.push_back(m); else if (extra) for (int64_t x = ep[m]; x < ep[m + 1]; ++x) if (ea[x] == w[k] || eb[x] == w[k]) want.push_back(-1); }
                if (want != ver[w[k]]) die("row version");
                if (plan.prev[k] >= 0) { if (b.x >= (unsigned)cap || slot_has[b.x] != plan.prev[k]) die("comp"); } else if (b.x != 0xFFFFFFFFu) die("comp none");
                if (a.y != 7u + (unsigned)(std::find(pr.order.begin(), pr.order.end(), k) - pr.order.begin())) die("seq");
                if (slot_has[a.w] != -1) die("slot in use");
                for (auto& f : finish) if (f.second == (int)a.w) die("slot twice");
                finish.push_back({k, (int)a.w}); ++evc;
            }
            int nl = __builtin_popcount(r[0].y); if (nl > P) die("loads"); int q = 0;
            for (int t = 0; t < teams; ++t) if (r[0].y >> t & 1) {
                const StripEntry& e = r[1 + 2 * P + 2 * q++];
                if (team_load[t] != -1) die("team busy"); if (r[0].z >> t & 1) die("load and eval");
                team_load[t] = pr.order[e.x]; team_when[t] = it; if (e.z != 0x1000u + w[team_load[t]] || e.y != 5) die("load worker");
            }
        }
        if (!finish.empty()) die("unfinished");
        for (int k = 0; k < A; ++k) if (!appl[k]) die("not applied");
        int need = 0; for (int k = 0; k < K; ++k) need += plan.r_round[k] >= 0; if (need != evc) die("evaluations missing");
        for (int k = A; k < K; ++k) if (plan.r_round[k] >= 0 || (anyc && carried[k] >= 0)) if (slot_has[pr.slot[k]] != k) die("pending slot");
        for (int r = 0; r < n; ++r) { std::vector<int> want; for (int m = 0; m < A; ++m) { if (w[m] == r || nb[m] == r) want.push_back(m); else if (extra) for (int64_t x = ep[m]; x < ep[m + 1]; ++x) if (ea[x] == r || eb[x] == r) want.push_back(-1); } if (want != ver[r]) die("final versions"); }
    }
    printf("ok, iterations %ld rounds %ld\n", its, rounds);
}
