// Layout of a call of a linear model as one persistent launch: its events in the order of their dependences, cut into
// iterations of the kernel (kernels_strips.hip).
#include <algorithm>
#include <cstring>
#include <functional>
#include <queue>
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
    std::vector<int32_t> free_slots;
    const int32_t P;              // evaluations and loads of a record, at most
    std::vector<int32_t> free_holders;
    int64_t loaded = 0;           // gradients whose rows have been requested, in the order of evaluation
    std::vector<int32_t> holder_of;

    Builder(const StripCall& call, int32_t teams, StripProgram& program) : c(call), out(program), P(teams / 2) {}

    // a new record; the holders that the previous one has left idle request the rows of the next gradients
    StripEntry* open() {
        out.recs.resize(out.recs.size() + out.rec_len, StripEntry{0, 0, 0, 0});
        ++out.iterations;
        StripEntry* rec = out.recs.data() + out.recs.size() - out.rec_len;
        const size_t n = std::min<size_t>(free_holders.size(), P);
        std::sort(free_holders.begin(), free_holders.begin() + n);
        // the order of the gradients is that of the loads; a record evaluates and loads in the order of the holders
        StripEntry* e = rec + 1 + 2 * P;
        for (size_t i = 0; i < n && loaded < static_cast<int64_t>(out.order.size()); ++i, e += 2) {
            const WorkerData& w = c.data[c.worker[out.order[loaded]]];
            const uint64_t f = reinterpret_cast<uint64_t>(w.features), t = reinterpret_cast<uint64_t>(w.targets);
            e[0] = StripEntry{static_cast<uint32_t>(loaded), static_cast<uint32_t>(w.ld), static_cast<uint32_t>(f), static_cast<uint32_t>(f >> 32)};
            e[1] = StripEntry{static_cast<uint32_t>(t), static_cast<uint32_t>(t >> 32), 0, 0};
            rec[0].y |= 1u << free_holders[i];
            holder_of[loaded++] = free_holders[i];
        }
        free_holders.erase(free_holders.begin(), free_holders.begin() + n);
        return rec;
    }
    int32_t take_slot() {         // -1: none left
        if (free_slots.empty()) return c.renumber ? out.n_slots++ : -1;
        const int32_t s = free_slots.back();
        free_slots.pop_back();
        return s;
    }
};

}  // namespace

namespace {

// What the schedule of a call depends on, per event and per row.
struct Order {
    std::vector<std::vector<int32_t>> updates;     // per row: the events that update it, in order ...
    std::vector<int32_t> next;                     // ... and the first one not applied yet
    std::vector<std::vector<std::pair<int32_t, int32_t>>> reads;    // per row: (updates before the read, event), sorted ...
    std::vector<int32_t> ready;                    // ... reads whose row has reached their version
    std::vector<int32_t> done;                     // ... reads evaluated
};

}  // namespace

// Iteration order.  An update is applied when its gradient is there, the earlier updates of its rows are applied and
// the reads that precede it are evaluated; an iteration applies all that can be (in waves of pairwise different rows,
// each filled up to whole batches of the kernel) and then evaluates the gradients that are ready, the oldest events
// first, teams / 2 at most.  So an iteration is spent per link of a chain of gradients, not per round.
// Gradients run at most `window` events ahead of the first event not applied: that bounds the slots, and as no read is
// further than the largest tau ahead of an update that waits for it, a window beyond that cannot block.
// Minibatch rows are requested in the order of evaluation, each set for a holder whose last gradient was finished in the
// iteration before, so the next rows are in flight while others are worked on.  All gradients before an iteration's own are
// evaluated by then, so with teams / 2 holders or more its rows are there or go out at its start.
bool build_strips(const StripCall& c, int32_t teams, StripProgram& out, int32_t holders) {
    const Plan& plan = *c.plan;
    out = StripProgram{};
    out.teams = teams;
    out.holders = holders > 0 ? holders : teams;
    out.slot.assign(static_cast<size_t>(c.K), -1);
    auto carried = [&](int64_t k) { return c.carried_slot && c.carried_slot[k] >= 0; };
    auto rows_of = [&](int64_t k, auto&& f) {
        f(c.worker[k]);
        if (c.neighbour[k] != c.worker[k]) f(c.neighbour[k]);
        if (c.extra_ptr)
            for (int64_t q = c.extra_ptr[k]; q < c.extra_ptr[k + 1]; ++q) {
                f(c.extra_a[q]);
                f(c.extra_b[q]);
            }
    };

    Order o;
    o.updates.resize(c.n);
    o.reads.resize(c.n);
    o.next.assign(c.n, 0);
    o.ready.assign(c.n, 0);
    o.done.assign(c.n, 0);
    for (int64_t k = 0; k < c.A; ++k) rows_of(k, [&](int32_t r) { o.updates[r].push_back(static_cast<int32_t>(k)); });
    int64_t reads_left = 0;
    for (int64_t k = 0; k < c.K; ++k) {
        if (plan.r_round[k] < 0) continue;                     // carried, or left to the next call
        const auto& u = o.updates[c.worker[k]];
        const int64_t before = k - c.tau[k];
        o.reads[c.worker[k]].push_back({static_cast<int32_t>(std::lower_bound(u.begin(), u.end(), before) - u.begin()), static_cast<int32_t>(k)});
        ++reads_left;
    }
    for (auto& r : o.reads) std::sort(r.begin(), r.end());

    Builder b(c, teams, out);
    const int32_t room = (kStripMaxRec - 1 - 4 * b.P) / kStripBatch * kStripBatch;
    if (c.renumber) {
        for (int64_t k = 0; k < c.K; ++k)
            if (carried(k)) out.slot[k] = b.take_slot();
    } else {
        std::vector<char> taken(static_cast<size_t>(c.n_slots), 0);
        for (int64_t k = 0; k < c.K; ++k)
            if (carried(k)) {
                out.slot[k] = c.carried_slot[k];
                taken[c.carried_slot[k]] = 1;
            }
        for (int32_t s = c.n_slots - 1; s >= 0; --s)
            if (!taken[s]) b.free_slots.push_back(s);
    }

    // first pass: what every iteration applies and evaluates
    struct Step {
        size_t updates, order;        // where its updates and its evaluations begin
    };
    std::vector<Step> steps;
    std::vector<StripEntry> ops;
    steps.reserve(static_cast<size_t>(c.K) + 2);
    ops.reserve(static_cast<size_t>(2 * c.K) + 64);
    out.order.reserve(static_cast<size_t>(c.K));
    std::vector<int32_t> evaluated(static_cast<size_t>(c.K), -1);      // step of the evaluation
    std::vector<char> applied(static_cast<size_t>(c.A), 0);
    std::priority_queue<int32_t, std::vector<int32_t>, std::greater<int32_t>> ready;
    std::vector<int32_t> candidates, again, wave, deferred;
    int64_t first = 0;
    auto open_reads = [&](int32_t r) {
        for (auto& at = o.ready[r]; at < static_cast<int32_t>(o.reads[r].size()) && o.reads[r][at].first <= o.next[r]; ++at)
            ready.push(o.reads[r][at].second);
    };
    // the first event of a row that is not applied yet, if its gradient is there (otherwise its evaluation brings it up)
    auto consider = [&](int32_t r) {
        if (o.next[r] >= static_cast<int32_t>(o.updates[r].size())) return;
        const int32_t k = o.updates[r][o.next[r]];
        if (evaluated[k] >= 0 || plan.r_round[k] < 0) candidates.push_back(k);
    };
    for (int32_t r = 0; r < c.n; ++r) {
        open_reads(r);
        consider(r);
    }
    while (first < c.A || reads_left > 0) {
        const int32_t now = static_cast<int32_t>(steps.size());
        const size_t ops0 = ops.size(), order0 = out.order.size();
        steps.push_back(Step{ops0, order0});
        auto applicable = [&](int32_t k) {
            if (applied[k] || (plan.r_round[k] >= 0 ? evaluated[k] < 0 || evaluated[k] >= now : !carried(k))) return false;
            bool ok = true;
            rows_of(k, [&](int32_t r) {
                const int32_t at = o.next[r];
                ok = ok && at < static_cast<int32_t>(o.updates[r].size()) && o.updates[r][at] == k &&
                     (o.done[r] == static_cast<int32_t>(o.reads[r].size()) || o.reads[r][o.done[r]].first > at);
            });
            return ok;
        };
        again.clear();
        while (!candidates.empty()) {
            if (candidates.size() > 1) {
                std::sort(candidates.begin(), candidates.end());
                candidates.erase(std::unique(candidates.begin(), candidates.end()), candidates.end());
            }
            wave.clear();
            for (const int32_t k : candidates)
                if (applicable(k)) wave.push_back(k);
            candidates.clear();
            if (wave.empty()) break;
            while ((ops.size() - ops0) % kStripBatch != 0) ops.push_back(StripEntry{0, 0, 0, kStripEmpty});
            for (const int32_t k : wave) {
                const int32_t pairs = 1 + static_cast<int32_t>(c.extra_ptr ? c.extra_ptr[k + 1] - c.extra_ptr[k] : 0);
                if (static_cast<int32_t>(ops.size() - ops0) + pairs > room && ops.size() > ops0) {
                    again.push_back(k);          // the record is full
                    continue;
                }
                auto put = [&](int32_t i, int32_t j, int32_t slot, float gamma, uint32_t flags) {
                    ops.push_back(StripEntry{static_cast<uint32_t>(i) | static_cast<uint32_t>(j) << 16, static_cast<uint32_t>(slot), bits(gamma), flags});
                };
                put(c.worker[k], c.neighbour[k], out.slot[k], c.gamma ? c.gamma[k] : c.gamma_default, 0);
                if (c.extra_ptr)
                    for (int64_t q = c.extra_ptr[k]; q < c.extra_ptr[k + 1]; ++q) put(c.extra_a[q], c.extra_b[q], 0, 0.0f, kStripAverage);
                b.free_slots.push_back(out.slot[k]);
                applied[k] = 1;
                rows_of(k, [&](int32_t r) {
                    ++o.next[r];
                    consider(r);
                    open_reads(r);
                });
            }
        }
        while (first < c.A && applied[first]) ++first;
        candidates = again;
        deferred.clear();
        while (!ready.empty() && out.order.size() < order0 + b.P) {
            const int32_t k = ready.top();
            ready.pop();
            const int64_t kp = plan.prev[k];
            if (k >= first + c.window || (kp >= 0 && !carried(kp) && (evaluated[kp] < 0 || evaluated[kp] >= now))) {
                deferred.push_back(k);
                continue;
            }
            evaluated[k] = now;
            out.slot[k] = b.take_slot();
            if (out.slot[k] < 0) return false;
            out.order.push_back(k);
            const int32_t r = c.worker[k];
            ++o.done[r];
            --reads_left;
            consider(r);                  // the read was what its next update waited for, or that update is event k
        }
        for (const int32_t k : deferred) ready.push(k);
        if (ops.size() == ops0 && out.order.size() == order0) return false;      // cannot happen with a valid plan
    }

    // second pass: the records, with the loads
    size_t widest = 1;
    steps.push_back(Step{ops.size(), out.order.size()});
    for (size_t i = 0; i + 1 < steps.size(); ++i) widest = std::max(widest, steps[i + 1].updates - steps[i].updates);
    const int32_t width = std::min<int32_t>(room, static_cast<int32_t>((widest + kStripBatch - 1) / kStripBatch) * kStripBatch);
    out.rec_len = 1 + 4 * b.P + width;
    out.n_slots = std::max(out.n_slots, 1);
    out.recs.reserve((steps.size() + ops.size() / width + 6) * out.rec_len);
    b.holder_of.assign(out.order.size(), -1);
    for (int32_t t = 0; t < out.holders; ++t) b.free_holders.push_back(t);
    b.open();
    std::vector<std::pair<int32_t, int64_t>> evals;      // (holder, position) of a record
    for (size_t i = 0; i + 1 < steps.size(); ++i) {
        StripEntry* rec = b.open();
        const size_t count = steps[i + 1].updates - steps[i].updates;
        for (size_t from = 0; from < count; from += width) {
            if (from > 0) rec = b.open();                // an event with more pairs than a record holds
            const size_t n = std::min<size_t>(width, count - from);
            std::copy_n(ops.begin() + steps[i].updates + from, n, rec + 1 + 4 * b.P);
            rec[0].x = static_cast<uint32_t>(n);
        }
        evals.clear();
        for (size_t q = steps[i].order; q < steps[i + 1].order; ++q) evals.push_back({b.holder_of[q], static_cast<int64_t>(q)});
        std::sort(evals.begin(), evals.end());
        StripEntry* e = rec + 1;
        for (const auto& [holder, at] : evals) {
            const int64_t k = out.order[at], kp = plan.prev[k];
            e[0] = StripEntry{static_cast<uint32_t>(holder), c.seq0 + static_cast<uint32_t>(at), static_cast<uint32_t>(c.worker[k]),
                              static_cast<uint32_t>(out.slot[k])};
            e[1] = StripEntry{0xFFFFFFFFu, 0, static_cast<uint32_t>(k), static_cast<uint32_t>(at % c.strips)};
            if (kp >= 0) {
                e[1].x = static_cast<uint32_t>(out.slot[kp]);
                e[1].y = bits(c.gamma ? c.gamma[kp] : c.gamma_default);
            }
            rec[0].z |= 1u << holder;
            b.free_holders.push_back(holder);
            e += 2;
        }
    }
    b.open();                  // finishes the gradients of the last record
    out.recs.resize(out.recs.size() + 3 * static_cast<size_t>(out.rec_len), StripEntry{0, 0, 0, 0});
    return true;
}

namespace {

// One averaging that a row takes part in: the event, and the other row.
struct RowUpdate {
    int64_t event;
    int32_t partner;
    bool extra;
};

struct Checker {
    const StripCall& c;
    const StripProgram& p;
    std::string& err;
    std::vector<std::vector<RowUpdate>> due;       // per row: its updates in the order of the events ...
    std::vector<size_t> done;                      // ... and how many are applied
    std::vector<int64_t> slot_event;               // gradient held by a slot, or -1
    std::vector<int64_t> loaded;                   // per holder: position whose minibatch rows it holds or has requested, or -1
    std::vector<int64_t> loaded_in;                // ... and the record that requested them
    std::vector<char> evaluated, applied;

    bool fail(const char* what, int64_t record) {
        err = "strip layout: " + std::string(what) + " in record " + std::to_string(record);
        return false;
    }
    bool slot_ok(uint32_t s) const { return s < slot_event.size(); }

    bool update(const StripEntry& e, int64_t record, std::vector<int32_t>& batch) {
        const int32_t i = static_cast<int32_t>(e.x & 0xFFFFu), j = static_cast<int32_t>(e.x >> 16);
        if (i >= c.n || j >= c.n) return fail("row out of range", record);
        for (const int32_t r : batch)
            if (r == i || r == j) return fail("a batch names a row twice", record);
        batch.push_back(i);
        batch.push_back(j);
        const bool extra = (e.w & kStripAverage) != 0;
        if (done[i] >= due[i].size() || done[j] >= due[j].size()) return fail("an update that no event makes", record);
        const RowUpdate &a = due[i][done[i]], &b = due[j][done[j]];
        if (a.event != b.event || a.partner != j || b.partner != i || a.extra != extra || b.extra != extra)
            return fail("an update out of the order of its rows", record);
        ++done[i];
        if (j != i) ++done[j];
        if (extra) return true;
        if (!slot_ok(e.y) || slot_event[e.y] != a.event || c.worker[a.event] != i) return fail("an update without its gradient", record);
        if (e.z != bits(c.gamma ? c.gamma[a.event] : c.gamma_default)) return fail("a wrong step size", record);
        slot_event[e.y] = -1;
        applied[a.event] = 1;
        return true;
    }

    bool evaluation(const StripEntry& a, const StripEntry& b, int64_t record, std::vector<std::pair<uint32_t, int64_t>>& finished) {
        const int64_t k = b.z;
        if (k >= c.K || a.x >= loaded.size()) return fail("an evaluation of no event", record);
        const int64_t at = static_cast<int64_t>(a.y - c.seq0);
        if (at < 0 || at >= static_cast<int64_t>(p.order.size()) || p.order[at] != k) return fail("a wrong sequence number", record);
        if (loaded[a.x] != at || loaded_in[a.x] > record) return fail("a holder without the rows of its gradient", record);
        loaded[a.x] = -1;
        if (evaluated[k] || static_cast<int32_t>(a.z) != c.worker[k]) return fail("a gradient of the wrong worker", record);
        evaluated[k] = 1;
        const auto& u = due[c.worker[k]];
        const int64_t before = k - c.tau[k];
        const size_t seen = std::lower_bound(u.begin(), u.end(), before, [](const RowUpdate& r, int64_t e) { return r.event < e; }) - u.begin();
        if (done[c.worker[k]] != seen) return fail("a read of the wrong version", record);
        const int64_t kp = c.plan->prev[k];
        if (kp < 0 ? b.x != 0xFFFFFFFFu : !slot_ok(b.x) || slot_event[b.x] != kp || b.y != bits(c.gamma ? c.gamma[kp] : c.gamma_default))
            return fail("a read compensated with the wrong gradient", record);
        if (!slot_ok(a.w) || slot_event[a.w] != -1) return fail("a gradient into a slot that is in use", record);
        for (const auto& f : finished)
            if (f.first == a.w) return fail("two gradients into one slot", record);
        if (b.w >= static_cast<uint32_t>(c.strips)) return fail("a loss that no block writes", record);
        finished.push_back({a.w, k});
        return true;
    }

    bool load(const StripEntry& a, const StripEntry& b, int32_t holder, int64_t record) {
        if (a.x >= p.order.size()) return fail("rows of no gradient requested", record);
        const WorkerData& w = c.data[c.worker[p.order[a.x]]];
        const uint64_t f = reinterpret_cast<uint64_t>(w.features), t = reinterpret_cast<uint64_t>(w.targets);
        if (loaded[holder] != -1) return fail("rows requested for a holder that is not idle", record);
        if (a.y != w.ld || (static_cast<uint64_t>(a.w) << 32 | a.z) != f || (static_cast<uint64_t>(b.y) << 32 | b.x) != t)
            return fail("rows of the wrong worker requested", record);
        loaded[holder] = a.x;
        loaded_in[holder] = record;
        return true;
    }

    bool run() {
        const int32_t holders = p.holders, half = p.teams / 2;
        if (static_cast<int64_t>(p.recs.size()) != (p.iterations + 3) * p.rec_len || p.rec_len > kStripMaxRec || p.rec_len < 2 + 4 * half)
            return fail("a table of the wrong size", 0);
        const int64_t slots = c.renumber ? p.n_slots : c.n_slots;
        if (c.renumber && p.n_slots > std::max(c.window, 1)) return fail("more slots than the window", 0);
        due.resize(c.n);
        done.assign(c.n, 0);
        slot_event.assign(slots, -1);
        loaded.assign(holders, -1);
        loaded_in.assign(holders, -1);
        evaluated.assign(c.K, 0);
        applied.assign(c.K, 0);
        for (int64_t k = 0; k < c.A; ++k) {
            const int32_t i = c.worker[k], j = c.neighbour[k];
            due[i].push_back({k, j, false});
            if (j != i) due[j].push_back({k, i, false});
            if (c.extra_ptr)
                for (int64_t q = c.extra_ptr[k]; q < c.extra_ptr[k + 1]; ++q) {
                    due[c.extra_a[q]].push_back({k, c.extra_b[q], true});
                    due[c.extra_b[q]].push_back({k, c.extra_a[q], true});
                }
        }
        for (int64_t k = 0; k < c.K; ++k)
            if (c.carried_slot && c.carried_slot[k] >= 0) {
                if (!slot_ok(p.slot[k]) || slot_event[p.slot[k]] != -1 || (!c.renumber && p.slot[k] != c.carried_slot[k])) return fail("a pending gradient in the wrong slot", 0);
                slot_event[p.slot[k]] = k;
            }
        std::vector<std::pair<uint32_t, int64_t>> finished;
        std::vector<int32_t> batch;
        for (int64_t it = 0; it < p.iterations; ++it) {
            const StripEntry* rec = &p.recs[it * p.rec_len];
            for (const auto& f : finished) slot_event[f.first] = f.second;      // the gradients of the record before
            finished.clear();
            if (1 + 4 * half + static_cast<int64_t>(rec[0].x) > p.rec_len) return fail("more updates than a record holds", it);
            for (uint32_t u = 0; u < rec[0].x; ++u) {
                if (u % kStripBatch == 0) batch.clear();
                const StripEntry& e = rec[1 + 4 * half + u];
                if ((e.w & kStripEmpty) == 0 && !update(e, it, batch)) return false;
            }
            if (holders < 32 && (rec[0].y >> holders != 0 || rec[0].z >> holders != 0)) return fail("a holder that does not exist", it);
            int32_t evals = 0, loads = 0;
            for (int32_t t = 0; t < holders; ++t)
                if (rec[0].y >> t & 1) {
                    const StripEntry* e = rec + 1 + 2 * half + 2 * loads;
                    if (++loads > half) return fail("more loads than a record holds", it);
                    if (!load(e[0], e[1], t, it)) return false;
                }
            for (int32_t t = 0; t < holders; ++t)
                if (rec[0].z >> t & 1) {
                    const StripEntry* e = rec + 1 + 2 * evals;
                    if (++evals > half || static_cast<int32_t>(e[0].x) != t) return fail("evaluations out of the order of their holders", it);
                    if (!evaluation(e[0], e[1], it, finished)) return false;
                }
        }
        if (!finished.empty()) return fail("gradients left unfinished", p.iterations);
        for (int64_t k = 0; k < c.K; ++k) {
            const bool carried = c.carried_slot && c.carried_slot[k] >= 0;
            if (k < c.A ? !applied[k] : (c.plan->r_round[k] >= 0 || carried) && slot_event[p.slot[k]] != k) return fail("an event left out", p.iterations);
            if (evaluated[k] != (c.plan->r_round[k] >= 0)) return fail("a gradient left out", p.iterations);
        }
        for (int32_t r = 0; r < c.n; ++r)
            if (done[r] != due[r].size()) return fail("an averaging left out", p.iterations);
        return true;
    }
};

}  // namespace

bool verify_strips(const StripCall& c, const StripProgram& p, std::string& err) { return Checker{c, p, err, {}, {}, {}, {}, {}, {}, {}}.run(); }

}  // namespace adpsgd_impl
