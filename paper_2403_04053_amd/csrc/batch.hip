// Batched solves: many independent scattering problems (incident directions,
// energies, potentials, uneven grids) advanced together.  The instances are
// dealt to sets that share the Infinity Cache; a set takes all the steps of a
// launch group before the next one starts, so its fields stay in the cache
// from pass to pass and step to step, and the sets run on a few branches side
// by side, so that one's launch gaps and last workgroups overlap with
// another's work.  Within a set, per axis, the instances are grouped by
// compiled tile shape; one launch covers every instance of a group (the
// workgroups look up their instance from a prefix table of tiles), and each
// instance's step counter lives in device memory, so whole groups of steps are
// captured once in a HIP graph and replayed.  An instance whose own step count
// is reached does no further work.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>
#include <string>
#include <vector>

#include "solver.hpp"

namespace {

constexpr int kBatchGraphSteps = 8;
// Branches that run side by side, and the bytes of fields (psi pair and L, 24 B
// per cell) of the sets on them at a time: under the 256 MB Infinity Cache.
// Twelve instances of 96-192 points per axis (775 MB), 16 steps: all instances
// pass by pass 11.55 ms; sets of 64 or 128 MB one after another 8.70; two
// branches 6.94 (128 MB) to 7.04 (200 MB), three 6.68 (200 MB), 6.70 (128), 6.84
// (300), four 6.95.  64 instances: 63.4 -> 78.9 Gcell/s.
constexpr int kBranches = 3;
constexpr double kBatchBytes = 200e6;
constexpr double kSetBytes = kBatchBytes / kBranches;
// Launches (of all instances together, pass by pass) from which steps fork onto the
// branches, which takes about 40 us: 12, or 48 where the cache holds the whole batch
// and only tails and gaps are to be gained.  Forked and pass by pass, us: four of
// 160^3, 1, 4, 7 steps 294 and 252, 950 and 927, 1586 and 1602; twelve of 96-192, one
// step (24 launches) 606 and 719; 32 of 24 to 64 points (87 MB), 2 and 4 steps (24, 48)
// 230 and 215, 406 and 394; six of 96^3, 8 and 16 steps 602 and 590, 1104 and 1157.
constexpr int64_t kForkLaunches = 12, kForkLaunchesCached = 48;

thread_local std::string g_batch_error;

struct Group {
    int variant = 0;
    bool seg = false;
    int potx = 0;       // x and z passes: where the members take the potential term
    std::vector<int> members;
    pstd::PassArgs* d_desc = nullptr;
    int* d_off = nullptr;
    int tiles = 0;
};

// instances that take a launch group's steps together
struct Set {
    std::vector<int> members;
    std::vector<Group> groups[3];
    int branch = 0;
};

}  // namespace

struct pstd_batch {
    std::vector<pstd_solver*> inst;
    hipStream_t stream = nullptr;
    int64_t* ctr = nullptr;  // [count][2]: step, end
    std::vector<Set> sets;
    Set all;                 // every instance in one set, where there is more than one
    hipStream_t cap_stream = nullptr;
    hipStream_t branch[kBranches] = {};      // streams of the other branches ([0] unused)
    hipEvent_t fork = nullptr, join[kBranches] = {};
    hipGraphExec_t graph = nullptr;
    std::vector<int> gen;  // table generation of each instance when the groups were built
    int64_t fork_from = 0; // launches from which steps fork
    int nt = 0;            // an instance's fields outgrow the Infinity Cache
    std::string err;
};

namespace {

pstd_status bfail(pstd_batch* b, pstd_status st, const std::string& m) {
    if (b) b->err = m;
    else g_batch_error = m;
    return st;
}

pstd_status bhip(pstd_batch* b, hipError_t e, const char* what) {
    return bfail(b, e == hipErrorOutOfMemory ? PSTD_ENOMEM : PSTD_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define BHIP_TRY(b, call)                                    \
    do {                                                     \
        hipError_t _e = (call);                              \
        if (_e != hipSuccess) return bhip((b), _e, #call);   \
    } while (0)

void free_set(Set& set) {
    for (auto& gs : set.groups)
        for (auto& g : gs) {
            (void)hipFree(g.d_desc);
            (void)hipFree(g.d_off);
        }
    set = Set{};
}

void free_sets(std::vector<Set>& sets) {
    for (Set& set : sets) free_set(set);
    sets.clear();
}

void drop_graph(pstd_batch* b) {
    if (b->graph) (void)hipGraphExecDestroy(b->graph);
    b->graph = nullptr;
}

// the per-axis launch groups of a set
pstd_status build_set(pstd_batch* b, Set& set) {
    for (int axis = 0; axis < 3; ++axis) {
        std::vector<Group>& gs = set.groups[axis];
        for (int i : set.members) {
            const pstd_solver* s = b->inst[i];
            const bool seg = s->prob.sub_core[axis] > 0;
            const int potx = axis == 1 ? 0 : s->potx;
            auto it = std::find_if(gs.begin(), gs.end(), [&](const Group& g) {
                return g.variant == s->variant[axis] && g.seg == seg && g.potx == potx;
            });
            if (it == gs.end()) {
                gs.push_back(Group{});
                it = gs.end() - 1;
                it->variant = s->variant[axis];
                it->seg = seg;
                it->potx = potx;
            }
            it->members.push_back(i);
        }
        for (Group& g : gs) {
            std::vector<pstd::PassArgs> desc(g.members.size());
            std::vector<int> off(g.members.size() + 1, 0);
            for (size_t k = 0; k < g.members.size(); ++k) {
                pstd::solver_args(b->inst[g.members[k]], axis, desc[k]);
                off[k + 1] = off[k] + desc[k].tiles;
            }
            g.tiles = off.back();
            BHIP_TRY(b, hipMalloc(&g.d_desc, desc.size() * sizeof(pstd::PassArgs)));
            BHIP_TRY(b, hipMalloc(&g.d_off, off.size() * sizeof(int)));
            BHIP_TRY(b, hipMemcpy(g.d_desc, desc.data(), desc.size() * sizeof(pstd::PassArgs), hipMemcpyHostToDevice));
            BHIP_TRY(b, hipMemcpy(g.d_off, off.data(), off.size() * sizeof(int), hipMemcpyHostToDevice));
        }
    }
    return PSTD_OK;
}

// first indexes of runs of consecutive sizes of at most `limit` each (an item
// beyond it is a run by itself)
std::vector<int> set_starts(const std::vector<double>& size, double limit) {
    std::vector<int> starts;
    double sum = 0;
    for (size_t i = 0; i < size.size(); ++i) {
        if (starts.empty() || sum + size[i] > limit) {
            starts.push_back((int)i);
            sum = 0;
        }
        sum += size[i];
    }
    return starts;
}

// the least limit that gives at most k runs
double even_limit(const std::vector<double>& size, int k) {
    double lo = *std::max_element(size.begin(), size.end()), hi = 0;
    for (double x : size) hi += x;
    if ((int)set_starts(size, lo).size() <= k) return lo;
    for (int i = 0; i < 50; ++i) {
        const double mid = 0.5 * (lo + hi);
        ((int)set_starts(size, mid).size() <= k ? hi : lo) = mid;
    }
    return hi;
}

// (re)build the sets and their per-axis launch groups from the instances'
// current tile shapes and tables.  The old ones go when the new ones are whole: a
// failure leaves them and their table generations, so that a run that needs new
// ones builds them again.
pstd_status build_groups(pstd_batch* b) {
    BHIP_TRY(b, hipStreamSynchronize(b->stream));
    std::vector<int> gen(b->inst.size());
    // non-temporal z-pass loads when an instance alone outgrows the Infinity
    // Cache (as for a single solve); for many instances that each fit, the
    // hint measured slower (64 instances of 96-192 per axis: 59.0 -> 57.6
    // Gcell/s)
    double largest = 0;
    for (size_t i = 0; i < b->inst.size(); ++i) {
        gen[i] = b->inst[i]->tab_gen;
        const pstd_problem& p = b->inst[i]->prob;
        largest = std::max(largest, 24.0 * p.n[0] * p.n[1] * p.n[2]);
    }
    // instances of like shape next to each other, so that a set's launches are few
    std::vector<int> order(b->inst.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
        const int32_t *nx = b->inst[x]->prob.n, *ny = b->inst[y]->prob.n;
        return std::lexicographical_compare(nx, nx + 3, ny, ny + 3);
    });
    std::vector<double> size;
    double total = 0;
    for (int i : order) {
        size.push_back(24.0 * (double)b->inst[i]->cells);
        total += size.back();
    }
    const bool cached = total <= 1.02 * kBatchBytes;
    Set all;
    all.members = order;
    if (pstd_status st = build_set(b, all)) {
        free_set(all);
        return st;
    }
    int64_t launches = 0;
    for (const auto& gs : all.groups) launches += (int64_t)gs.size();
    // Sets: each filled to its share of the cache; where the cache holds the whole
    // batch, even ones, as many as the branches, or, for instances of one shape, as
    // many as such shares, whichever fewer are as even.  16 steps, filled and even:
    // four of 128^3 (sets of one and of two) 1830 and 1613 us, four of 48 to 160 points
    // 1209 and 909, 32 of 24 to 64 points 1576 and 1420.  One set up to a share.
    double limit = kSetBytes;
    if (cached) {
        const int most = launches == 3 ? std::min(kBranches, (int)std::ceil(total / kSetBytes)) : kBranches;
        const double best = even_limit(size, most);
        for (int k = most; k >= 1; --k)
            if (const double l = even_limit(size, k); l <= 1.1 * best) limit = l;
        if (total <= kSetBytes) limit = total;
    }
    const std::vector<int> starts = set_starts(size, limit);
    std::vector<Set> sets(starts.size());
    std::vector<double> bytes(starts.size(), 0);
    for (size_t i = 0, k = 0; i < order.size(); ++i) {
        if (k + 1 < starts.size() && (int)i == starts[k + 1]) ++k;
        sets[k].members.push_back(order[i]);
        bytes[k] += size[i];
    }
    // largest sets first onto the branch with the least work
    double load[kBranches] = {};
    std::vector<int> by(sets.size());
    for (size_t i = 0; i < by.size(); ++i) by[i] = (int)i;
    std::stable_sort(by.begin(), by.end(), [&](int x, int y) { return bytes[x] > bytes[y]; });
    for (int i : by) {
        const int k = (int)(std::min_element(load, load + kBranches) - load);
        sets[i].branch = k;
        load[k] += bytes[i];
    }
    pstd_status st = PSTD_OK;
    if (sets.size() == 1) std::swap(sets[0], all);
    else
        for (Set& set : sets)
            if (!st) st = build_set(b, set);
    if (st) {
        free_sets(sets);
        free_set(all);
        return st;
    }
    drop_graph(b);  // it holds the old descriptor buffers
    free_sets(b->sets);
    free_set(b->all);
    b->sets.swap(sets);
    std::swap(b->all, all);
    b->gen.swap(gen);
    b->fork_from = cached ? kForkLaunchesCached : kForkLaunches;
    b->nt = largest > pstd::kInfinityCacheBytes ? 1 : 0;
    return PSTD_OK;
}

// step k of a launch group, of a set
pstd_status launch_step(pstd_batch* b, const Set& set, hipStream_t stream, int k) {
    for (int axis = 0; axis < 3; ++axis)
        for (const Group& g : set.groups[axis]) {
            hipError_t e = pstd::launch_variant(g.variant, g.seg, axis, g.d_desc, g.d_off, (int)g.members.size(),
                                                g.tiles, k, g.potx, b->nt, stream);
            if (e != hipSuccess) return bhip(b, e, "batch pass launch");
        }
    return PSTD_OK;
}

// the streams and events of the branches
pstd_status ensure_branches(pstd_batch* b) {
    if (!b->fork) BHIP_TRY(b, hipEventCreateWithFlags(&b->fork, hipEventDisableTiming));
    for (int k = 1; k < kBranches; ++k) {
        if (!b->branch[k]) BHIP_TRY(b, hipStreamCreateWithFlags(&b->branch[k], hipStreamNonBlocking));
        if (!b->join[k]) BHIP_TRY(b, hipEventCreateWithFlags(&b->join[k], hipEventDisableTiming));
    }
    return PSTD_OK;
}

// whether `steps` steps are worth a fork
bool forks(const pstd_batch* b, int64_t steps) {
    int64_t launches = 0;
    for (const auto& gs : b->all.groups) launches += (int64_t)gs.size();
    return b->sets.size() > 1 && steps * launches >= b->fork_from;
}

// `count` consecutive steps of every instance, then one counter advance: the
// branches side by side, or all instances pass by pass
pstd_status launch_batch_steps(pstd_batch* b, hipStream_t stream, int count, bool fork, bool capturing = false) {
    pstd_status st = PSTD_OK;
    if (!fork) {
        const Set& set = b->sets.size() > 1 ? b->all : b->sets[0];
        for (int k = 0; k < count && !st; ++k) st = launch_step(b, set, stream, k);
    } else {
        if ((st = ensure_branches(b))) return st;
        hipStream_t on[kBranches] = {stream};
        std::vector<const Set*> of[kBranches];
        for (const Set& set : b->sets) of[set.branch].push_back(&set);
        BHIP_TRY(b, hipEventRecord(b->fork, stream));
        for (int i = 1; i < kBranches; ++i) {
            on[i] = b->branch[i];
            BHIP_TRY(b, hipStreamWaitEvent(on[i], b->fork, 0));
        }
        // A step of each branch's current set by turns, so that they start together:
        // 32 of 24 to 64 points, 4 steps 362 us (branch by branch 433), 16 as graphs 1261
        // (1425).  Graphs of batches beyond the cache branch by branch, the one with the
        // largest set last: twelve of 96-192, 16 steps 7306 us (by turns 7460).
        const bool turns = !capturing || b->fork_from == kForkLaunchesCached;
        const size_t run = turns ? 1 : SIZE_MAX;
        size_t at[kBranches] = {};
        for (bool more = true; more && !st;) {
            more = false;
            for (int n = 0; n < kBranches; ++n) {
                const int i = turns ? n : (n + 1) % kBranches;
                for (size_t r = 0; r < run && at[i] < of[i].size() * count && !st; ++r, ++at[i])
                    st = launch_step(b, *of[i][at[i] / count], on[i], (int)(at[i] % count));
                more |= at[i] < of[i].size() * count;
            }
        }
        // joined also after a failure: what has been queued is waited for
        for (int i = 1; i < kBranches; ++i) {
            BHIP_TRY(b, hipEventRecord(b->join[i], on[i]));
            BHIP_TRY(b, hipStreamWaitEvent(stream, b->join[i], 0));
        }
    }
    if (st) return st;
    hipError_t e = pstd::launch_advance(b->ctr, (int)b->inst.size(), count, stream);
    if (e != hipSuccess) return bhip(b, e, "batch advance");
    return PSTD_OK;
}

pstd_status build_batch_graph(pstd_batch* b) {
    if (b->graph) return PSTD_OK;
    if (!b->cap_stream) BHIP_TRY(b, hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking));
    if (pstd_status st = ensure_branches(b)) return st;  // nothing is created in a capture
    BHIP_TRY(b, hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal));
    pstd_status st = launch_batch_steps(b, b->cap_stream, kBatchGraphSteps, b->sets.size() > 1, true);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(b->cap_stream, &g);
    if (st) {
        if (g) (void)hipGraphDestroy(g);
        return st;
    }
    if (e != hipSuccess) return bhip(b, e, "batch graph capture");
    e = hipGraphInstantiate(&b->graph, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
        b->graph = nullptr;
        return bhip(b, e, "batch graph instantiate");
    }
    return PSTD_OK;
}

}  // namespace

extern "C" {

pstd_status pstd_batch_create(const pstd_problem* problems, int32_t count, void* hip_stream, pstd_batch** out) {
    if (!problems || !out || count < 1) return PSTD_EINVAL;
    *out = nullptr;
    pstd_batch* b = new pstd_batch();
    b->stream = (hipStream_t)hip_stream;
    hipError_t e = hipMalloc(&b->ctr, 2 * sizeof(int64_t) * count);
    if (e) {
        delete b;
        return bhip(nullptr, e, "hipMalloc counters");
    }
    for (int i = 0; i < count; ++i) {
        pstd_solver* s = nullptr;
        pstd_status st = pstd::solver_create(&problems[i], b->stream, b->ctr + 2 * i, &s);
        if (st) {
            std::string m = "instance " + std::to_string(i) + ": " + pstd_last_error(nullptr);
            pstd_batch_destroy(b);
            return bfail(nullptr, st, m);
        }
        b->inst.push_back(s);
    }
    pstd_status st = build_groups(b);
    if (st) {
        std::string m = b->err;
        pstd_batch_destroy(b);
        return bfail(nullptr, st, m);
    }
    *out = b;
    return PSTD_OK;
}

pstd_status pstd_batch_size(const pstd_batch* b, int32_t* count_out) {
    if (!b || !count_out) return PSTD_EINVAL;
    *count_out = (int32_t)b->inst.size();
    return PSTD_OK;
}

pstd_status pstd_batch_solver(pstd_batch* b, int32_t idx, pstd_solver** out) {
    if (!b || !out || idx < 0 || idx >= (int32_t)b->inst.size()) return PSTD_EINVAL;
    *out = b->inst[idx];
    return PSTD_OK;
}

pstd_status pstd_batch_set_potential(pstd_batch* b, int32_t idx, const float* V_dev, int64_t n_cells) {
    if (!b || idx < 0 || idx >= (int32_t)b->inst.size()) return PSTD_EINVAL;
    pstd_status st = pstd_set_potential(b->inst[idx], V_dev, n_cells);
    if (st) return bfail(b, st, "instance " + std::to_string(idx) + ": " + b->inst[idx]->err);
    return PSTD_OK;
}

pstd_status pstd_batch_autotune(pstd_batch* b, int32_t reps) {
    if (!b || reps < 1) return PSTD_EINVAL;
    // tune the largest instance of every distinct (axis pass) length and share
    // its choice with the instances of that length
    for (int axis = 0; axis < 3; ++axis) {
        std::vector<std::pair<int, int>> done;  // (local length, variant)
        std::vector<int> order(b->inst.size());
        for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
        std::sort(order.begin(), order.end(), [&](int x, int y) { return b->inst[x]->cells > b->inst[y]->cells; });
        for (int i : order) {
            pstd_solver* s = b->inst[i];
            const int len = s->prob.sub_core[axis] > 0 ? s->prob.sub_core[axis] + 2 * s->prob.sub_halo : s->prob.n[axis];
            auto it = std::find_if(done.begin(), done.end(), [&](const std::pair<int, int>& d) { return d.first == len; });
            if (it != done.end()) {
                s->variant[axis] = it->second;
                continue;
            }
            pstd_status st = pstd::solver_autotune(s, reps);
            if (st) return bfail(b, st, s->err);
            done.push_back({len, s->variant[axis]});
        }
    }
    drop_graph(b);
    return build_groups(b);
}

pstd_status pstd_batch_run(pstd_batch* b, const int64_t* n_steps_host) {
    if (!b || !n_steps_host) return PSTD_EINVAL;
    const int count = (int)b->inst.size();
    std::vector<int64_t> c(2 * count);
    int64_t most = 0;
    bool grew = false;
    for (int i = 0; i < count; ++i) {
        if (n_steps_host[i] < 0) return bfail(b, PSTD_EINVAL, "negative step count");
        pstd_solver* s = b->inst[i];
        pstd_status st = pstd::solver_ensure_tables(s, s->step + n_steps_host[i]);
        if (st) return bfail(b, st, s->err);
        grew |= s->tab_gen != b->gen[i];
        c[2 * i] = s->step;
        c[2 * i + 1] = s->step + n_steps_host[i];
        most = std::max(most, n_steps_host[i]);
    }
    if (grew) {
        pstd_status st = build_groups(b);
        if (st) return st;
    }
    BHIP_TRY(b, hipStreamSynchronize(b->stream));
    BHIP_TRY(b, hipMemcpy(b->ctr, c.data(), c.size() * sizeof(int64_t), hipMemcpyHostToDevice));
    int64_t left = most;
    // (the graph forks where there are branches; a run too short for that is at most
    // 15 steps)
    if (left >= kBatchGraphSteps && (b->sets.size() == 1 || forks(b, left))) {
        pstd_status st = build_batch_graph(b);
        if (st) return st;
        for (; left >= kBatchGraphSteps; left -= kBatchGraphSteps) BHIP_TRY(b, hipGraphLaunch(b->graph, b->stream));
    }
    if (left > 0) {
        pstd_status st = launch_batch_steps(b, b->stream, (int)left, forks(b, left));
        if (st) return st;
    }
    for (int i = 0; i < count; ++i) {
        pstd_solver* s = b->inst[i];
        pstd::solver_account_steps(s, s->step, s->step + n_steps_host[i]);
        s->step += n_steps_host[i];
    }
    return PSTD_OK;
}

pstd_status pstd_batch_destroy(pstd_batch* b) {
    if (!b) return PSTD_OK;
    if (b->stream) (void)hipStreamSynchronize(b->stream);
    else (void)hipDeviceSynchronize();
    drop_graph(b);
    if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
    for (int k = 1; k < kBranches; ++k) {
        if (b->branch[k]) (void)hipStreamDestroy(b->branch[k]);
        if (b->join[k]) (void)hipEventDestroy(b->join[k]);
    }
    if (b->fork) (void)hipEventDestroy(b->fork);
    free_sets(b->sets);
    free_set(b->all);
    for (pstd_solver* s : b->inst) pstd_destroy(s);
    (void)hipFree(b->ctr);
    delete b;
    return PSTD_OK;
}

const char* pstd_batch_last_error(const pstd_batch* b) { return b ? b->err.c_str() : g_batch_error.c_str(); }

}  // extern "C"
