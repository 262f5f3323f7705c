// How a batched attention launch is cut: host code without HIP, so that it can be built and tested on its own.
//
// A workgroup has a compute unit to itself and owns (KV head, block of query rows - 64 or 128 in the staged
// kernel, up to 256 in the pipelined one - and one of `cuts` ranges of a step's 64-key chunks).  The steps of
// a launch share the kernel and the height of the row block.  plan_batch plans the staged kernel, plan_launch
// (which the launcher calls) chooses between that and the pipelined one.
#pragma once

namespace la {

constexpr int kMaxBatch = 16;    // steps of a launch
constexpr int kXcds = 8, kXcdUnits = 32;  // XCDs, and compute units of one

// What the steps of a launch that are cut amount to at most: ranges of at least a 384th of the
// launch's chunks make twice as many workgroups at most when they are rounded up.
constexpr int kMaxCutWorkgroups = 768, kMaxCutGroups = 384;

struct BatchPlan {
    bool rows128;            // 128-row workgroups (head_dim 128 only), else 64
    int cuts[kMaxBatch];     // ranges of step i
    int place[kMaxBatch];    // the steps in slot order
};

// Workgroups of a step on every XCD (they are numbered XCD by XCD).
inline int batch_wgs_per_xcd(int units, int cuts) { return (int)(((long long)units * cuts + kXcds - 1) / kXcds); }

// The workgroups that share a row block's keys exchange partial results through the L2 of their XCD;
// the last one of a group that lies on two XCDs computes the rows again over all keys instead.
inline bool batch_groups_whole(int units, int cuts) { return batch_wgs_per_xcd(units, cuts) % cuts == 0; }

namespace batch_plan {

// Chunk and fixed times: a workgroup costs its chunks plus a part that does not depend on them
// (start, merge, writing the rows): 6 chunks' time of 1.22 us in the 128-row form, 5 of 0.76 us in the
// 64-row one, and 1 or 2 more with partial results to exchange; from steps of 4 to 66 chunks, one and
// two rounds, cut and uncut.  The two forms are compared with a chunk of the 128-row form counting 16
// and one of the 64-row form 11: it takes 0.76 us in one round but 0.84 in several, which pull twice
// the traffic of the 128-row form through the L2s.  (10 for a single round changes none of 120 plans.)
// Over those 120 batches the launches take between 0.60 and 1.02 of the time under the bounding rule below
// alone, 0.92 in the geometric mean.
struct Form {
    int units;      // (KV head, row block) pairs of a step
    int fixed, exchange, chunk;
};
inline Form form_of(bool rows128, int kv_heads, int tiles)
{
    return rows128 ? Form{kv_heads * ((tiles + 3) / 4), 6, 1, 16} : Form{kv_heads * ((tiles + 1) / 2), 5, 2, 11};
}

// Time, in chunks, at which the compute units of an XCD are done when they take the workgroups in
// slot order as they become free: m equal workgroups at a time go to the emptiest units, which are
// kept as runs of equal load.
inline long long launch_end(const int* order, int n, const int* wgs, const long long* cost)
{
    long long load[kXcdUnits], end = 0;
    int count[kXcdUnits], runs = 1;
    load[0] = 0;
    count[0] = kXcdUnits;
    for (int k = 0; k < n; ++k) {
        const long long c = cost[order[k]];
        for (int m = wgs[order[k]]; m > 0;) {
            const int take = m < count[0] ? m : count[0];
            const long long v = load[0] + c;
            m -= take;
            if (v > end) end = v;
            int first = 0;                     // the emptiest run, or what is left of it, goes on at 0
            if (take == count[0]) first = 1;
            else count[0] -= take;
            int at = first;                    // where the filled units belong among the rest
            while (at < runs && load[at] < v) ++at;
            if (at < runs && load[at] == v) {
                count[at] += take;
                if (first) {
                    for (int j = 1; j < runs; ++j) { load[j - 1] = load[j]; count[j - 1] = count[j]; }
                    --runs;
                }
            } else if (first) {
                for (int j = 1; j < at; ++j) { load[j - 1] = load[j]; count[j - 1] = count[j]; }
                load[at - 1] = v;
                count[at - 1] = take;
            } else {
                for (int j = runs; j > at; --j) { load[j] = load[j - 1]; count[j] = count[j - 1]; }
                load[at] = v;
                count[at] = take;
                ++runs;
            }
        }
    }
    return end;
}

// A set of cuts as workgroups: keys of each (in chunks), how many on every XCD, what each costs, longest first.
struct Layout {
    int cuts[kMaxBatch], range[kMaxBatch], wgs[kMaxBatch], order[kMaxBatch];
    long long cost[kMaxBatch], sum;  // sum: of all workgroups of an XCD

    void cut(int i, int x, int chunks, const Form& f)
    {
        cuts[i] = x;
        wgs[i] = batch_wgs_per_xcd(f.units, x);
        range[i] = (chunks + x - 1) / x;
        cost[i] = range[i] + f.fixed + (x > 1 ? f.exchange : 0);
    }
    void arrange(int n, bool longest_first)
    {
        sum = 0;
        for (int i = 0; i < n; ++i) {
            int j = i;
            for (; longest_first && j > 0 && cost[order[j - 1]] < cost[i]; --j) order[j] = order[j - 1];
            order[j] = i;
            sum += wgs[i] * cost[i];
        }
    }
};

// Cuts and order for one form: all cuts allowed (limit[i]), the steps as they come, or what ends earlier:
// longest ranges first, and fewer cuts.  (Longest first alone is no rule: 8 steps of 1253 to 14559 keys, 161
// rows, 32/8 heads take 219 us as they come and 224 longest first, 81 rows 122.9 and 122.3.)  From uncut
// steps on, the step with the longest ranges is cut once more as long as the sum of all
// workgroups leaves room for a better end than the best one seen; cuts whose longest workgroup alone
// takes that long are passed over unplaced.  Returns the launch's end.
// (Host time, which every call and so every layer pays for: of this plan, over 3000 batches of 2 to 16 steps
// of all sizes in use, median 0.4 us, one in ten above 2.0, at most 11; with the pipelined kernel's, `search_wide`,
// 0.7, 2.8 and 16.  Placing every set of cuts, one workgroup at a time, with no bound on the cuts: 5.3, 25.5
// and 68 for this one.)
inline long long search(const int* chunks, const int* limit, int n, const Form& f, int* cuts, int* place)
{
    Layout l;
    long long best = -1;
    auto consider = [&] {
        if (best >= 0 && l.cost[l.order[0]] >= best) return;
        const long long end = launch_end(l.order, n, l.wgs, l.cost);
        if (best >= 0 && end >= best) return;
        best = end;
        for (int i = 0; i < n; ++i) { cuts[i] = l.cuts[i]; place[i] = l.order[i]; }
    };
    for (int i = 0; i < n; ++i) {
        int x = limit[i];
        while (!batch_groups_whole(f.units, x)) --x;
        l.cut(i, x, chunks[i], f);
    }
    l.arrange(n, false);
    consider();
    l.arrange(n, true);
    consider();
    for (int i = 0; i < n; ++i) l.cut(i, 1, chunks[i], f);
    for (;;) {
        l.arrange(n, true);
        consider();
        if (l.sum >= best * kXcdUnits) break;
        int longest = -1, more = 0;
        for (int i = 0; i < n; ++i) {
            int x = l.cuts[i] + 1;
            while (x <= limit[i] && !batch_groups_whole(f.units, x)) ++x;
            if (x > limit[i] || (longest >= 0 && l.range[i] <= l.range[longest])) continue;
            longest = i;
            more = x;
        }
        if (longest < 0) break;
        l.cut(longest, more, chunks[longest], f);
    }
    return best * f.chunk;
}

}  // namespace batch_plan

// chunks[i]: 64-key chunks of step i (longest steps first); tiles: 32-row tiles of a KV head's query rows;
// rows: 128 or 64 to force the form (a testing hook), 0 to choose it.
inline BatchPlan plan_batch(const int* chunks, int n, int tiles, int kv_heads, int head_dim, int rows = 0)
{
    using namespace batch_plan;
    BatchPlan p;
    // The plan that bounds the others.  128-row workgroups (a chunk of K/V staged once for four row
    // tiles: half the traffic into LDS per flop) as soon as the batch fills three quarters of the GPU
    // with them, otherwise 64-row workgroups; ranges of at least four chunks, one round of workgroups
    // when the steps are alike, half a round more when their lengths differ; no cuts that leave a group
    // on two XCDs (3 steps of 4096 keys, 4/1 heads, 81 rows: 6 units cut into 14 ranges 57.6 us, uncut 45.1;
    // 12 of 350 to 900 keys, 16/4 heads of 64, 43 rows: 22.4 and 17.1).
    // Nothing below takes a step to a plan of less accuracy.  A cut step's partial results are rounded to
    // bf16 (against 64 bits, 12 steps of 4096 keys, 32/8 heads, 81 rows: 2.6e-3 uncut, 3.1e-3 cut), and so
    // are the sums of three of a 64-row workgroup's four key-split waves, but of one in two of a 128-row
    // one (10 steps of 14 to 184 keys, 32/8 heads, 121 rows: 2.44e-3 and 2.36e-3).  So only a step that is
    // cut here may be cut, and the form may only change from 64 to 128 rows.  (What the number of cuts
    // changes beyond that is the last 2 %: 4 steps of 512 keys, 41 rows, 3.04e-3 in three ranges, 3.09e-3 in two.
    // Of 100 batches that one alone has a larger error than under this rule alone; others up to 15 % less.)
    // (Cutting those 12 steps, too, would take 126 us instead of 158; partial results in fp32 cost every
    // cut launch 1 to 4 us.)
    p.rows128 = head_dim == 128 && (rows ? rows == 128 : tiles >= 3 && (long long)n * kv_heads * ((tiles + 3) / 4) >= 192);
    const Form f = form_of(p.rows128, kv_heads, tiles);
    long long work = 0;
    bool alike = true, may_cut = false;
    for (int i = 0; i < n; ++i) {
        work += (long long)f.units * chunks[i];
        alike = alike && chunks[i] == chunks[0];
    }
    const long long wgs = alike ? 256 : 384;
    long long target = (work + wgs - 1) / wgs;   // chunks per workgroup
    if (target < 4) target = 4;
    int limit[kMaxBatch];
    for (int i = 0; i < n; ++i) {
        long long x = (chunks[i] + target - 1) / target;
        if (x > chunks[i] / 2) x = chunks[i] / 2;
        if (x > 64) x = 64;
        if (x < 1 || !batch_groups_whole(f.units, (int)x)) x = 1;
        limit[i] = p.cuts[i] = (int)x;
        p.place[i] = i;
        may_cut = may_cut || x > 1;
    }
    // Fewer cuts, or 128 rows, where the launch ends earlier by the times above.  Measured at 32/8 heads, this rule alone
    // and with what follows: 8 steps of 512 keys, 81 rows 29.9 and 19.4 us (uncut); 16 of 466 to 1021
    // keys, 81 rows 52.3 and 48.1 (504 workgroups of 128 rows instead of 528); 8 of 1253 to 14559 keys, 121 rows
    // 175 and 170; 6 of 1024 keys, 81 rows 33.9 and 28.0 (128 rows).  Where the ends are equal all cuts
    // stay: 12 of 148 to 1278 keys, 32/32 heads, 25 rows 27.9 us, uncut 28.9.
    const bool may_grow = !p.rows128 && !rows && head_dim == 128 && tiles >= 3;
    // The times hold for the two forms of head_dim 128.  The four-wave workgroups of head_dim 64 gain from
    // every cut the rule allows (3 steps of 509 to 3864 keys, 32/8 heads, 121 rows: 19.5 us, with the times
    // above 30.1; 9 of 688 to 7706 keys, 81 rows: 54.9 and 61.4): they stay with it.
    if (head_dim != 128 || (!may_cut && !may_grow)) return p;
    const long long end = search(chunks, limit, n, f, p.cuts, p.place);
    if (may_grow) {
        BatchPlan g;
        g.rows128 = true;
        if (search(chunks, limit, n, form_of(true, kv_heads, tiles), g.cuts, g.place) < end) p = g;
    }
    return p;
}

// ---- staged or pipelined kernel (la_attention_wide.h: workgroups of up to 256 rows, head_dim 128)

// What the cut steps of a pipelined launch amount to at most.  Their partial results are in fp32 and a
// second kernel adds them up, so a step may be cut whatever the rule above says, and its ranges may lie
// on any XCD.
constexpr int kMaxWideCutWorkgroups = 448;
constexpr int kPipelinedRows = 256;
inline bool pipelined_applies(int tiles, int head_dim) { return head_dim == 128 && tiles >= 4; }  // (fewer tiles fit one staged workgroup)

struct LaunchPlan {
    int rows;                // rows of a workgroup: 64 or 128 (staged kernel), or kPipelinedRows
    int cuts[kMaxBatch], place[kMaxBatch];  // as in BatchPlan
};

namespace batch_plan {

struct WideForm {
    int units, chunk, fixed;   // times in 10 ns
};

// A set of cuts of a pipelined launch as workgroups, longest first (equal ones in the steps' order).
struct WideLayout {
    const int* chunks;
    WideForm f;
    int n, cuts[kMaxBatch], range[kMaxBatch], wgs[kMaxBatch], order[kMaxBatch];
    long long cost[kMaxBatch];
    long long sum = 0;                        // of all workgroups of an XCD
    long long workgroups = 0, cut_workgroups = 0, work = 0;   // of the launch; work: its chunks' time

    WideLayout(const int* chunks_, int n_, const WideForm& f_) : chunks(chunks_), f(f_), n(n_)
    {
        for (int i = 0; i < n; ++i) {
            work += (long long)f.units * chunks[i] * f.chunk;
            set(i, 1);
            order[i] = i;
            settle(i);
        }
    }
    void set(int i, int x)
    {
        cuts[i] = x;
        range[i] = (chunks[i] + x - 1) / x;
        wgs[i] = batch_wgs_per_xcd(f.units, x);
        cost[i] = (long long)range[i] * f.chunk + f.fixed;
        sum += wgs[i] * cost[i];
        workgroups += (long long)f.units * x;
        if (x > 1) cut_workgroups += (long long)f.units * x;
    }
    void cut(int i, int x)
    {
        sum -= wgs[i] * cost[i];
        workgroups -= (long long)f.units * cuts[i];
        if (cuts[i] > 1) cut_workgroups -= (long long)f.units * cuts[i];
        set(i, x);
    }
    void settle(int at)  // order[at] among the steps before it
    {
        const int i = order[at];
        for (; at > 0 && (cost[order[at - 1]] < cost[i] || (cost[order[at - 1]] == cost[i] && order[at - 1] > i)); --at) order[at] = order[at - 1];
        order[at] = i;
    }
    int longest() const { return range[order[0]]; }
    // No range of more than `most` chunks; false: that takes more workgroups than a launch may have.
    bool cut_to(int most)
    {
        for (int i = 0; i < n; ++i)
            if (range[i] > most) {
                cut(i, (int)(((long long)chunks[i] + most - 1) / most));
                if (!allowed()) return false;
            }
        for (int i = 1; i < n; ++i) settle(i);
        return true;
    }
    void cut_longest()
    {
        const int i = order[0];
        cut(i, cuts[i] + 1);
        int at = 0;
        for (; at + 1 < n && (cost[order[at + 1]] > cost[i] || (cost[order[at + 1]] == cost[i] && order[at + 1] < i)); ++at) order[at] = order[at + 1];
        order[at] = i;
    }
    bool allowed() const { return cut_workgroups <= kMaxWideCutWorkgroups; }
    // the second kernel, and what storing and reading fp32 partial results takes
    long long extra() const { return cut_workgroups ? 350 + cut_workgroups : 0; }
    // what no launch of these cuts or of more ends before
    long long floor() const { return (work + workgroups * f.fixed) / (kXcds * kXcdUnits) + extra(); }
    // when the launch ends, or `late` if that is no earlier
    long long end(long long late) const
    {
        const long long before = late - extra();
        if (cost[order[0]] >= before || sum / kXcdUnits >= before) return late;
        for (int k = 0, rounds = 1, at = 0; k < n; ++k)   // of 32 * r + 1 workgroups r + 1 share a unit
            for (at += wgs[order[k]]; at > rounds * kXcdUnits;)
                if (++rounds * cost[order[k]] >= before) return late;
        const long long e = launch_end(order, n, wgs, cost);
        return e < before ? e + extra() : late;
    }
};

// As `search`, for the pipelined kernel, whose steps may all be cut: from uncut steps on, the step with the
// longest ranges is cut once more, down to ranges of four to seven chunks, and the plan is that of the
// earliest end, if one ends before `late`.  This runs in every call, so only what can still win is placed:
// the cuts at which a workgroup's own time meets the average unit's are placed first, which bounds the
// longest range of a better plan from above (the walk starts there) and the number of its workgroups (it
// ends there).  (Of 20000 drawn batches nine have another plan than if every set of cuts is placed until the
// sum of its workgroups exceeds the best end, all of an earlier end.  Host time of a launch's plan, placed and as
// here: 16 steps of 16k keys, 8 tiles, one KV head 23 and 2.6 us; 16 of 4096 keys, 41 rows, 8/2 heads 12.6
// and 3.3; eight of 1253 to 14559 keys, 121 rows, 32/8 heads 3.9 and 1.7; one in a hundred of 3000 above 14 and 6.5.)
inline bool search_wide(const int* chunks, int n, const WideForm& f, long long late, LaunchPlan& p)
{
    constexpr int kShort = 7;    // no longer ranges are cut
    const WideLayout uncut(chunks, n, f);
    if (uncut.floor() >= late) return false;
    long long even = uncut.longest();
    for (int k = 0; k < 4; ++k) {
        const long long workgroups = uncut.work / (even * f.chunk) + (long long)f.units * n / 2;
        const long long r = ((uncut.work + workgroups * f.fixed) / (kXcds * kXcdUnits) - f.fixed) / f.chunk + 1;
        even = r < kShort ? kShort : r < uncut.longest() ? r : uncut.longest();
    }
    WideLayout l = uncut;
    if (l.cut_to((int)even)) {
        const long long e = l.end(late);
        if (e < late) late = e + 1;    // (found again below, if nothing is better)
    }
    l = uncut;
    const long long fits = (late - 1 - f.fixed) / f.chunk;
    if (fits < l.longest() && !l.cut_to(fits > kShort ? (int)fits : kShort)) return false;
    for (bool found = false;; l.cut_longest()) {
        if (!l.allowed() || l.floor() >= late) return found;
        const long long e = l.end(late);
        if (e < late) {
            late = e;
            found = true;
            p.rows = kPipelinedRows;
            for (int i = 0; i < n; ++i) { p.cuts[i] = l.cuts[i]; p.place[i] = l.order[i]; }
        }
        if (l.longest() <= kShort) return found;
    }
}

}  // namespace batch_plan

// As plan_batch; rows: kPipelinedRows to force that form, too; pipelined: false to leave that form out.
inline LaunchPlan plan_launch(const int* chunks, int n, int tiles, int kv_heads, int head_dim, int rows = 0, bool pipelined = true)
{
    using namespace batch_plan;
    LaunchPlan p;
    long long end = -1;
    const bool can = pipelined && pipelined_applies(tiles, head_dim);
    if (rows != kPipelinedRows || !can) {
        const BatchPlan b = plan_batch(chunks, n, tiles, kv_heads, head_dim, rows == kPipelinedRows ? 0 : rows);
        p.rows = b.rows128 ? 128 : 64;
        for (int i = 0; i < n; ++i) { p.cuts[i] = b.cuts[i]; p.place[i] = b.place[i]; }
        if (rows || !can) return p;
        const Form f = form_of(b.rows128, kv_heads, tiles);
        int wgs[kMaxBatch];
        long long cost[kMaxBatch];
        for (int i = 0; i < n; ++i) {
            const int range = (chunks[i] + b.cuts[i] - 1) / b.cuts[i];
            wgs[i] = batch_wgs_per_xcd(f.units, b.cuts[i]);
            cost[i] = (long long)(range + f.fixed + (b.cuts[i] > 1 ? f.exchange : 0)) * (b.rows128 ? 122 : 80);
        }
        end = launch_end(b.place, n, wgs, cost);
    }
    // Times of the pipelined form, us: a chunk 1.81 with eight tiles (8 prefixes of 1024 and 3072 keys, 64/8 heads, 121
    // rows: 50.2 and 108.0 a launch) and 0.4 of that however few, start and end 7 and 0.65 a tile.  Taken
    // where the launch then ends 7 % sooner: of 240 drawn batches (2 to 16 steps of 1 to 8000 keys, 25 to 361 rows)
    // measured in every form it is taken for 61, at 0.56 to 1.03 of the staged form's time, 0.81 in the geometric
    // mean; two are slower, by 2 and 3 % (of 70 others one, by 5 %: five steps of 30 to 341 keys, 201 rows, 32/8
    // heads).  At 14 % none would be, for an eighth of the gain; where the times say 0.93 to 1.0 it measures 0.78
    // to 1.05, where they say 1.0 to 1.1 0.86 to 1.16.
    const int blocks = (tiles + 7) / 8, per_block = (tiles + blocks - 1) / blocks;
    const WideForm f = {kv_heads * blocks, 72 + 109 * per_block / 8, 700 + 65 * per_block};
    LaunchPlan q;
    return search_wide(chunks, n, f, end < 0 ? 1ll << 60 : (end * 93 + 99) / 100, q) ? q : p;
}

// ---- one step alone

// Ranges of its keys: one round of workgroups, two chunks each at least, and the ranges of a row block on one XCD, whose L2
// they exchange their results in; it has `step_units_per_xcd` row blocks at most.  Workgroups handed out without regard to
// that put the ranges of a row block on two XCDs where the number of row blocks is no multiple of eight, and such a group is
// computed again over all keys: 20/20 heads, 57 rows on 4096 keys 52.5 -> 21.2 us, 42/42 on 1000 21.7 -> 13.7 (8-bit cache
// 20.8 -> 10.7, pages 24.1 -> 14.2), 4/4, head_dim 64, 31 rows on 4096 keys 53.6 -> 11.3, on 512 13.2 -> 6.3.  (Compute units
// that this leaves idle do not matter: spreading the row blocks evenly over the XCDs measured the same.)
constexpr int kMaxStepWorkgroups = kXcds * kXcdUnits, kMaxStepGroups = kMaxStepWorkgroups / 2;   // of a step that is cut
inline int step_units_per_xcd(int units) { return (units + kXcds - 1) / kXcds; }
inline int step_cuts_clipped(int x, int chunks)
{
    if (x > chunks / 2) x = chunks / 2;
    if (x > 64) x = 64;
    return x < 1 ? 1 : x;
}
inline int step_cuts(int units, int chunks) { return step_cuts_clipped(kXcdUnits / step_units_per_xcd(units), chunks); }
// Whether there are several ranges and every row block's are on one XCD without that rule too, dealt out evenly.
inline bool step_cuts_even(int units, int chunks)
{
    const int x = step_cuts_clipped(kXcdUnits * kXcds / units, chunks);
    return x > 1 && (units * x + kXcds - 1) / kXcds % x == 0;
}

// In how many ranges, and whether they exchange fp32.  One workgroup per compute unit is not always best: a range to add up
// costs 0.16 to 0.20 us in bf16 and 0.18 to 0.31 in fp32 where the last workgroup of a group reads all of them, and a chunk of a range
// takes 0.55 to 0.80 (64 rows of 128 dimensions in pairs of chunks, one tile, 64 dimensions; 13 to 361 rows on 1024 to
// 16384 keys).  Since waves of all workgroups read them the choice is within 1 to 2 % of the best one (72 steps measured with every
// number of ranges; the best weights for these are within 0.8 to 1.3 %), so the line stays.  Fewer ranges in bf16 would be further from 64 bits (4/4 heads, 121 rows on 4096 keys: 2.98e-3 with 32 ranges,
// 3.11e-3 with 12), in fp32 they are nearer (2.64e-3): so fewer are taken where the results are fp32 anyway or that is half a
// microsecond ahead in fp32 too.  Where 32 ranges fit (8 row blocks at most) that is at 65 to 72 chunks and at 53, 57, 59, 61 and 63
// (an odd number leaves the most ranges three chunks, walked as four) with 64 rows of 128 dimensions, at 65 to 70, 59 and 63 with one
// tile, and with 64 dimensions at 51 to 90, 97 to 110, 129 to 132 and odd numbers from 33 to 49; where 16 fit, at 33 with 64
// dimensions alone.  4/4 heads 14.8 -> 13.6 us, 8/1, 57 rows 15.3 -> 12.0, 32/8, 13 rows 15.1 -> 13.8 (all on 4096 keys), 4/4
// with 64 dimensions 11.0 -> 10.1, 4/4, 31 rows (fp32 before) 16.7 -> 13.2.
struct StepRanges {
    int x;
    bool fp32;
};
inline StepRanges step_ranges(int units, int chunks, int rows, int head_dim, bool fp32)
{
    const int most = step_cuts(units, chunks);
    if (most == 1 || rows > 64) return StepRanges{most, fp32 && most > 1};
    const bool pairs = head_dim == 128 && rows == 64;
    const int chunk = head_dim == 64 ? 64 : pairs ? 55 : 80, r32 = head_dim == 64 ? 18 : 30, r16 = head_dim == 64 ? 16 : pairs ? 17 : 20;
    auto walk = [&](int x) {
        const int n = (chunks + x - 1) / x;
        return (pairs ? (n + 1) / 2 * 2 : n) * chunk;
    };
    int best = 2;
    for (int x = 3; x <= most; ++x)
        if (walk(x) + x * r32 < walk(best) + best * r32) best = x;
    return fp32 || walk(best) + best * r32 + 50 < walk(most) + most * r16 ? StepRanges{best, true} : StepRanges{most, false};
}

namespace batch_plan {

// When the staged kernel ends a step, in 10 ns, from 200 drawn steps of 300 to 16384 keys, 9 to 361 rows, 4 to 64 heads in groups
// of 1 to 8, measured in both forms: a round of workgroups takes 3.9 us and 0.78 a chunk with 64 rows, 4.9 and 1.13 with 128
// (8-bit cache: 0.66 and 1.20), or what the chunks that its workgroups do not share take from HBM if that is more (7.2 and 5.6
// ns a chunk and workgroup; 8-bit cache half), and a range to exchange 0.13 and 0.24.
inline long long staged_step_end(bool rows128, int chunks, int tiles, int kv_heads, bool codes)
{
    const int blocks = rows128 ? (tiles + 3) / 4 : (tiles + 1) / 2, units = kv_heads * blocks, x = step_cuts(units, chunks);
    const long long wgs = (long long)units * x, rounds = (wgs + 255) / 256, range = (chunks + x - 1) / x;
    const long long apart = (wgs < 256 ? wgs : 256) / blocks, stream = range * apart * (rows128 ? 56 : 72) / (codes ? 200 : 100);
    const long long walk = range * (rows128 ? (codes ? 120 : 113) : codes ? 66 : 78);
    return 150 + rounds * ((rows128 ? 490 : 390) + (walk > stream ? walk : stream)) + (rows128 ? 24 : 13) * x;
}

}  // namespace batch_plan

// Whether a step alone takes 128-row workgroups of the staged kernel (head_dim 128) instead of 64-row ones, which pull twice the
// chunks into LDS: where its times end it 0.75 us sooner.  Of 200 drawn steps (bf16 packed and paged, 8-bit) 40 are on that side of
// the line and take 0.88 of the time they take with 64 rows in the geometric mean, 1.01 at worst; the better form for each would
// be 0.1 % ahead of the rule over all 200.  32/32 heads, 105 rows on 4829 keys 26.8 -> 24.2 us, 161 rows on 1687 19.1 -> 17.0, 64/8,
// 101 rows on 2535 21.3 -> 19.0, 40/40, 241 rows on 2845 43.2 -> 28.5.  (Near the line, left with 64 rows: 64/8, 57 rows on 4096
// keys 18.2 and 17.7, 40/40, 81 rows on 2048 17.1 and 16.9.)
// Errors against 64 bits are 3 to 10 % smaller.
// A step with one range has no partial results: 128 rows then have to be 4.4 us ahead: fp32
// partial results take 1 to 4, and the noalloc entry point 2 to clear its tickets.  many_rows: a step that has always had 128 rows, which round fewer
// sums between key-split waves, goes back to 64 only with fp32 results and where 128 rows would be cut 16 times or more, to 20
// chunks at most (8/1 heads, 121 rows on 4096 keys 15.6 -> 11.7 us, on 16384 24.9 -> 21.5; 3.05e-3 -> 2.70e-3).  codes: the 8-bit cache.
inline bool step_rows128(int chunks, int tiles, int kv_heads, bool many_rows, bool codes)
{
    using namespace batch_plan;
    if (many_rows) {
        const int x = step_cuts(kv_heads * ((tiles + 3) / 4), chunks);
        return x < 16 || chunks > 20 * x;
    }
    const bool cut64 = step_cuts(kv_heads * ((tiles + 1) / 2), chunks) > 1, cut128 = step_cuts(kv_heads * ((tiles + 3) / 4), chunks) > 1;
    return staged_step_end(true, chunks, tiles, kv_heads, codes) + (cut128 && !cut64 ? 440 : 75) <
           staged_step_end(false, chunks, tiles, kv_heads, codes);
}

// Chunks that a step alone requests before its loop, where an iteration takes one (rows: of a workgroup; blocks: row blocks
// of a KV head; range: chunks of the longest range).  Each request up front holds the first chunk back: 32/32 heads, 121 rows on
// 1024, 3 chunks 12.4 us with one, 12.7 with two.  From four chunks on two are ahead: 40/40, 81 rows on 2048, 6 chunks 17.7 and
// 16.9, 32/4, 151 rows on 3917, 11 chunks 22.7 and 21.6, 40/40, 241 rows on 2845, 17 chunks 32.5 and 28.3.  A full ring (four)
// is behind (29.8 for the last; 32/32, 121 rows on 16000, 32 chunks 55.5 and 57.4) until row blocks share 32 chunks or more
// (64/64, 181 rows on 6064, 49 chunks 69.8 and 68.2; 64/8, 121 on 16384, 65 chunks 82.9 and 81.9).  One tile: two (32/32, 25
// rows on 3000: 18.4, 15.9, 16.4, 17.1 with one to four).  64 dimensions, whose chunks are half as large, gain from a third
// from 16 on (32/8, 121 rows on 8000: 28.7 and 28.0).
inline int step_chunks_ahead(int rows, int head_dim, int blocks, int range)
{
    if (head_dim == 64) return range > 16 ? 3 : 2;
    if (rows != 128) return 2;
    if (blocks > 1 && range >= 32) return 4;
    return range < 4 ? 1 : 2;
}

}  // namespace la
