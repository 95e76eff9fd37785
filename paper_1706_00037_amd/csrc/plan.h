// Generation launch tables shared by the multi-start run/batch (plan.hip) and
// the request server (serve.hip).
//
// One generation of the multi-start loop of Fig. 2 is a fixed sequence of
// launches, each covering every instance of a set:
//   diversify (one plane: clears f) -> [two planes: eval_init] -> eval (row dot, one
//   launch for each tiling variant) -> [f dump] -> screen and ascent order (one launch up
//   to 16384 candidates, four beyond) -> Delta init of the first passer chunk (one launch
//   for each coefficient width; a server: one for each group) -> for each (planes, 16-column
//   blocks) group, on its stream: team and one-wave ascent, later chunks behind it ->
//   incumbent, statistics, generation counter and ranking -> placement and seed fill.
// A launch table holds, for one step, each instance's kernel arguments and the
// prefix of the blocks (or waves) each instance needs.  Instances are independent:
// each one's results depend only on its own problem, parameters and state.
#pragma once

#include <string.h>

#include <vector>

#include "ubqp_internal.h"

inline size_t ubqp_align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Offsets of one instance's device state inside its allocation.
struct InstLayout {
    size_t seeds, X, f, flips, idx, oidx, rank, scal, bestx, stats, part, err, Y, total;
    int64_t S, cap;
};
InstLayout ubqp_inst_layout(const ubqp_problem *p, const ubqp_params *pr);

// One instance as the launch tables see it.
struct InstRef {
    const ubqp_problem *p;
    ubqp_params pr;
    InstLayout L;
    char *base;      // device state, L.total bytes
    int64_t *dump;   // optional G x M objective dump (device)
    int32_t *err;    // device error flag the instance's ascent reports to
    template <typename T> T *at(size_t off) const { return (T *)(base + off); }
};

template <typename A> struct Table {
    std::vector<A> args;
    std::vector<int64_t> prefix{0};
    size_t args_off = 0, pre_off = 0;
    const A *d_args = nullptr;
    const int64_t *d_pre = nullptr;
    void add(const A &a, int64_t blocks)
    {
        args.push_back(a);
        prefix.push_back(prefix.back() + blocks);
    }
    int count() const { return (int)args.size(); }
    int64_t total() const { return prefix.back(); }
    void stage(std::vector<char> &host)
    {
        args_off = ubqp_align256(host.size());
        host.resize(args_off + args.size() * sizeof(A));
        if (!args.empty()) memcpy(host.data() + args_off, args.data(), args.size() * sizeof(A));
        pre_off = ubqp_align256(host.size());
        host.resize(pre_off + prefix.size() * sizeof(int64_t));
        memcpy(host.data() + pre_off, prefix.data(), prefix.size() * sizeof(int64_t));
    }
    void bind(char *dev)
    {
        d_args = (const A *)(dev + args_off);
        d_pre = (const int64_t *)(dev + pre_off);
    }
};

// Ascents of one passer chunk (entries [j cap, (j + 1) cap) of every instance's list)
// of the instances of one coefficient width and lane range.
struct Chunk {
    int planes, nb;
    int lane;  // 0: the generation's stream, k: side stream k - 1; the same for every chunk of a group
    bool split = false;  // split rows for the one-wave ascent (AscArgs::split_one) among them
    Table<EvalArgs> yr;   // its Delta initialisation, where that runs beside other groups' ascents
    Table<AscArgs> asc;
    Table<AscArgs> team;  // the same ascents' team launch (few passers), empty when the group never uses teams
    int n_pad_max = 0;
};

// The (planes, NB) groups of the ascent run concurrently (they touch different
// instances): a run's on the generation's own stream and three side streams, the largest
// group on the generation's (six int16 instances 15.9 ms, 17.0 with two side streams; a
// process has four hardware queues, and streams that share one run in turn), a server's
// on the three side streams, the smallest first.  One launch for neighbouring lane
// ranges was measured 2 to 4% faster on the largest batches and a third slower where
// one instance's team ascent then held up the other's one-wave ascent (five int16
// instances of 1206 to 3534 variables, 1465 candidates: 5.7 against 3.7 ms, 4.2 with
// the initialisations on the side streams).  The Delta initialisation of all groups of a
// run goes first, on the generation's stream: its workgroups fill the chip, and started
// beside another group's ascent they wait for its waves to leave.  That holds for the
// first passer chunk; a later one (its list is longer than the Delta workspace)
// follows its group's previous chunk on the group's stream, so that a group with many
// passers does not hold up the others (three int16 instances of 3000 to 7000 variables,
// 25000 to 30000 passers in two chunks, at most 64 flips each: 36.6 ms, 37.8 with all
// groups joined after each chunk, 36.1 with every initialisation on its group's stream;
// with the second chunks empty 33.3, 33.4 and 36.6).  A server's many
// groups fill the chip between them, and there each group's initialisation goes before
// its ascent in the group's own stream, so that no ascent waits for all of them: ms,
// this way / with the initialisations first, medians of 4 to 8 processes within 1%:
// eleven requests of 716 to 3261 variables 6.70 / 7.06, ten int16 of 600 to 5000 variables
// 23.6 / 24.8, sixteen of 500 to 7000 variables 57.5 / 60.3 where the process had run other
// plans, but 66.7 / 61.2 where the server's were its first streams: two of the three side
// streams then share a hardware queue (a kernel trace shows the queue of each).
#define UBQP_ASCENT_LANES 4
struct SideStreams {
    hipStream_t s[UBQP_ASCENT_LANES - 1] = {};
    hipEvent_t fork = nullptr, join[UBQP_ASCENT_LANES - 1] = {};
    hipError_t create();
    void destroy();
};

struct EvalGroup {         // instances whose row-dot contraction uses one variant
    int variant;
    std::vector<EvalArgs> args;  // before their K ranges are shared
    Table<EvalArgs> t;
};

struct GenTables {
    int count = 0;
    Table<DivArgs> div;
    Table<EvalArgs> einit;              // two planes only (one plane: the diversification clears f)
    std::vector<EvalGroup> ev;
    Table<ScrOrdArgs> scr_ord;          // screening and ascent order by one block per instance
    Table<ScreenArgs> scr;              // instances of more candidates than one block takes
    Table<OrdArgs> ord;                 // ... one block per instance
    Table<SelArgs> sel_rank, sel_fill;  // same arguments, two prefixes
    Table<SelArgs> dump;                // instances with a dump of their objectives
    Table<SelArgs> init;                // generation-0 seeds of the joining instances
    // Delta initialisation of every instance's first chunk, by coefficient width (one
    // plane: ascent keys, two: Y rows); a server's is with its chunks
    Table<EvalArgs> dinit[2];
    std::vector<Chunk> chunks;          // in order of chunk number, the largest lane ranges first
    std::vector<char> host;             // staged image of every table

    // Builds every table for the instances and stages them into `host`; the
    // init table covers the instances with join[i] != 0 (all when join is null).
    // server: the Delta initialisations and lanes of a server's groups (above).
    void build(const std::vector<InstRef> &inst, const std::vector<char> *join = nullptr,
               bool server = false);
    // Points the tables at the device copy of `host`.
    void bind(char *dev);
    // Streams that a generation's ascents run on (one (planes, NB) group: 1, no fork).
    int lanes() const;
};

// Generation-0 seeds and scalars of the instances in the init table.
hipError_t ubqp_queue_seed_init(const GenTables &t, hipStream_t st);
// All launches of one generation.  When pe != null, events pe[0..5] bound the five
// sequential phases and ae[2c], ae[2c + 1] the ascent launch of chunk group c; the
// groups then run in order on st.  Otherwise, with side != null and more than one
// group, the groups run concurrently on the side streams.
hipError_t ubqp_queue_generation(const GenTables &t, hipStream_t st, hipEvent_t *pe, hipEvent_t *ae = nullptr,
                                 const SideStreams *side = nullptr);
