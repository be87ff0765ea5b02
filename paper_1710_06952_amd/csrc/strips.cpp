// Layout of a call of a linear model as one persistent launch: the rounds of the plan, cut into iterations of the
// kernel (kernels_strips.hip).
#include <algorithm>
#include <cstring>
#include <utility>

#include "strips.hpp"

namespace adpsgd_impl {

namespace {

uint32_t bits(float f) {
    uint32_t u;
    std::memcpy(&u, &f, 4);
    return u;
}

struct Builder {
    const StripCall& c;
    StripProgram& out;
    const int32_t T;
    int32_t max_updates = 0;
    std::vector<int32_t> free_slots;

    Builder(const StripCall& call, int32_t teams, StripProgram& program) : c(call), out(program), T(teams), P(teams / 2) {}

    const int32_t P;              // evaluations and loads of a record, at most
    std::vector<int32_t> free_teams;
    int64_t loaded = 0;           // gradients whose rows have been requested, in the order of evaluation
    std::vector<int32_t> team_of;

    // a new record; the teams that the previous one has left idle request the rows of the next gradients
    StripEntry* open() {
        out.recs.resize(out.recs.size() + out.rec_len, StripEntry{0, 0, 0, 0});
        ++out.iterations;
        StripEntry* rec = out.recs.data() + out.recs.size() - out.rec_len;
        const size_t n = std::min<size_t>(free_teams.size(), P);
        std::sort(free_teams.begin(), free_teams.begin() + n);
        // the order of the gradients is that of the loads; a record evaluates and loads in the order of the teams
        StripEntry* e = rec + 1 + 2 * P;
        for (size_t i = 0; i < n && loaded < static_cast<int64_t>(out.order.size()); ++i, e += 2) {
            const WorkerData& w = c.data[c.worker[out.order[loaded]]];
            const uint64_t f = reinterpret_cast<uint64_t>(w.features), t = reinterpret_cast<uint64_t>(w.targets);
            e[0] = StripEntry{static_cast<uint32_t>(loaded), static_cast<uint32_t>(w.ld), static_cast<uint32_t>(f), static_cast<uint32_t>(f >> 32)};
            e[1] = StripEntry{static_cast<uint32_t>(t), static_cast<uint32_t>(t >> 32), 0, 0};
            rec[0].y |= 1u << free_teams[i];
            team_of[loaded++] = free_teams[i];
        }
        free_teams.erase(free_teams.begin(), free_teams.begin() + n);
        return rec;
    }
    int32_t take_slot() {
        if (free_slots.empty()) return out.n_slots++;
        const int32_t s = free_slots.back();
        free_slots.pop_back();
        return s;
    }
    void update(StripEntry* rec, int32_t i, int32_t j, int32_t slot, float gamma, bool average_only) {
        rec[1 + 4 * P + rec[0].x++] = StripEntry{static_cast<uint32_t>(i) | static_cast<uint32_t>(j) << 16,
                                                 static_cast<uint32_t>(slot), bits(gamma), average_only ? 1u : 0u};
    }
};

}  // namespace

// Iteration order.  The gradients of a round come first, one for half of the teams at a time; the updates of the
// round open the next iteration.  Minibatch rows are requested in the order of evaluation, each set by a team whose
// last gradient was finished in the iteration before, so a team's next rows are in flight while the others work.
void build_strips(const StripCall& c, int32_t teams, StripProgram& out) {
    const Plan& plan = *c.plan;
    const int32_t R = plan.n_rounds;
    out = StripProgram{};
    out.teams = teams;
    out.slot.assign(static_cast<size_t>(c.K), -1);

    // events by round (counting sort): evaluations and updates
    std::vector<int64_t> r_off(static_cast<size_t>(R) + 1, 0), u_off(static_cast<size_t>(R) + 1, 0);
    std::vector<int64_t> u_ops(static_cast<size_t>(R), 0);
    for (int64_t k = 0; k < c.K; ++k) {
        if (plan.r_round[k] >= 0) ++r_off[plan.r_round[k] + 1];
        if (k < c.A) {
            ++u_off[plan.u_round[k] + 1];
            u_ops[plan.u_round[k]] += 1 + (c.extra_ptr ? c.extra_ptr[k + 1] - c.extra_ptr[k] : 0);
        }
    }
    int64_t widest = 1;
    for (int32_t r = 0; r < R; ++r) {
        widest = std::max(widest, u_ops[r]);
        r_off[r + 1] += r_off[r];
        u_off[r + 1] += u_off[r];
    }
    out.order.resize(static_cast<size_t>(r_off[R]));
    std::vector<int64_t> updates(static_cast<size_t>(u_off[R]));
    {
        std::vector<int64_t> ra(r_off.begin(), r_off.end() - 1), ua(u_off.begin(), u_off.end() - 1);
        for (int64_t k = 0; k < c.K; ++k) {
            if (plan.r_round[k] >= 0) out.order[ra[plan.r_round[k]]++] = k;
            if (k < c.A) updates[ua[plan.u_round[k]]++] = k;
        }
    }

    Builder b(c, teams, out);
    const int64_t room = kStripMaxRec - 1 - 4 * (teams / 2);
    b.max_updates = static_cast<int32_t>(std::min(widest, room));
    out.rec_len = 1 + 4 * (teams / 2) + b.max_updates;
    out.recs.reserve(static_cast<size_t>(2 * out.order.size() / teams + 2 * R + 8) * out.rec_len);

    if (c.renumber) {
        if (c.carried_slot)
            for (int64_t k = 0; k < c.K; ++k)
                if (c.carried_slot[k] >= 0) out.slot[k] = b.take_slot();
    } else {
        for (int64_t k = 0; k < c.K; ++k) out.slot[k] = plan.slot[k];
    }

    b.team_of.assign(out.order.size(), -1);
    for (int32_t t = 0; t < teams; ++t) b.free_teams.push_back(t);
    b.open();
    std::vector<std::pair<int32_t, int64_t>> evals;      // (team, position) of a record

    int64_t pending = 0, pending_end = 0;       // range of `updates` not laid out yet, of one round
    int64_t extra_at = 0;                       // next extra pair of updates[pending], 0: its own pair
    // as many of the pending updates as the record holds; they touch pairwise different rows
    auto put_updates = [&](StripEntry* rec) {
        while (pending < pending_end) {
            const int64_t k = updates[pending];
            const int64_t n_extra = c.extra_ptr ? c.extra_ptr[k + 1] - c.extra_ptr[k] : 0;
            for (; extra_at <= n_extra; ++extra_at) {
                if (static_cast<int32_t>(rec[0].x) >= b.max_updates) return;
                if (extra_at == 0) {
                    b.update(rec, c.worker[k], c.neighbour[k], out.slot[k], c.gamma ? c.gamma[k] : c.gamma_default, false);
                    if (c.renumber) b.free_slots.push_back(out.slot[k]);
                } else {
                    const int64_t q = c.extra_ptr[k] + extra_at - 1;
                    b.update(rec, c.extra_a[q], c.extra_b[q], 0, 0.0f, true);
                }
            }
            extra_at = 0;
            ++pending;
        }
    };
    auto flush_updates = [&] {
        while (pending < pending_end) put_updates(b.open());
    };
    for (int32_t r = 0; r < R; ++r) {
        for (int64_t q = r_off[r]; q < r_off[r + 1];) {
            const int64_t room_left = b.max_updates;
            // the last record of the pending updates also carries gradients
            while (pending < pending_end) {
                int64_t ops = 0;
                for (int64_t u = pending; u < pending_end && ops <= room_left; ++u)
                    ops += 1 + (c.extra_ptr ? c.extra_ptr[updates[u] + 1] - c.extra_ptr[updates[u]] : 0);
                ops -= extra_at;
                if (ops <= room_left) break;
                put_updates(b.open());
            }
            const int64_t ready = b.loaded;        // requested by an earlier record
            StripEntry* rec = b.open();
            put_updates(rec);
            const int64_t end = std::min(std::min(q + b.P, r_off[r + 1]), ready);
            evals.clear();
            for (; q < end; ++q) evals.push_back({b.team_of[q], q});
            std::sort(evals.begin(), evals.end());
            StripEntry* e = rec + 1;
            for (const auto& [team, at] : evals) {
                const int64_t k = out.order[at], kp = plan.prev[k];
                if (c.renumber) out.slot[k] = b.take_slot();
                e[0] = StripEntry{static_cast<uint32_t>(team), c.seq0 + static_cast<uint32_t>(at), static_cast<uint32_t>(c.worker[k]),
                                  static_cast<uint32_t>(out.slot[k])};
                e[1] = StripEntry{0xFFFFFFFFu, 0, static_cast<uint32_t>(k), static_cast<uint32_t>(at % c.strips)};
                if (kp >= 0) {
                    e[1].x = static_cast<uint32_t>(out.slot[kp]);
                    e[1].y = bits(c.gamma ? c.gamma[kp] : c.gamma_default);
                }
                rec[0].z |= 1u << team;
                b.free_teams.push_back(team);
                e += 2;
            }
        }
        flush_updates();       // left over where the round evaluates no gradient
        pending = u_off[r];
        pending_end = u_off[r + 1];
        extra_at = 0;
    }
    flush_updates();
    b.open();                  // finishes the gradients of the last record
    out.recs.resize(out.recs.size() + 3 * static_cast<size_t>(out.rec_len), StripEntry{0, 0, 0, 0});
}

}  // namespace adpsgd_impl
