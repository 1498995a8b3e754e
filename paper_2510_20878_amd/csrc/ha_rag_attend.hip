// Host side of attention over packed chunks: argument checks, the workspace layout, and the
// launches (attention launches of up to 512 runs, as many as their descriptors fit, one merge launch per 64
// requests).
#include "ha_rag_internal.h"

#include <algorithm>
#include <cstdio>
#include <memory>
#include <type_traits>

using namespace ha_rag_host;

namespace {

// A list in storage its owner provides: the planning below fills such lists, so that one of
// its callers can keep them on the stack and allocate nothing.
template <class T>
struct Fixed {
    T *data = nullptr;
    uint32_t cap = 0, n = 0;
    Fixed() = default;
    Fixed(T *d, uint32_t c) : data(d), cap(c) {}
    bool push_back(const T &v)
    {
        if (n == cap) return false;
        data[n++] = v;
        return true;
    }
    T &operator[](size_t i) const { return data[i]; }
    uint32_t size() const { return n; }
    void clear() { n = 0; }
};

// One document of a request: keys and values, from one whole chunk or from a keys-only and a
// values-only chunk (paired in list order).
struct Doc {
    const uint8_t *k = nullptr, *v = nullptr;  // packed bytes holding the keys / the values
    uint64_t k_tile = 0, v_tile = 0;           // bytes of one tile record
    uint32_t k_first = 0, v_first = 0;         // tile record of (layer 0, head 0): 0, or H for the
                                               // values of a whole chunk; a layer is k_step records on
    uint32_t k_step = 0, v_step = 0;
    uint32_t n_tokens = 0, info = 0;
    uint32_t n_blocks = 0;                     // layout blocks (16 tokens each)
};

struct Plan {               // one request
    uint32_t first_doc = 0, n_docs = 0;  // its documents that hold tokens
    uint32_t n_mt = 1;
    uint32_t shared = 0;       // goes to the kernel whose waves share each decoded block: more than two query
                               // tiles, or two in some calls whose largest request has three to eight
    uint32_t run_blocks = 0;   // layout blocks per run (what one workgroup takes)
    uint64_t all_blocks = 0;   // layout blocks of all its documents
    uint64_t wide_blocks = 0;  // those of documents with a 16-bit side
    uint32_t least_blocks = 0; // of its shortest document
    uint32_t n_runs = 0;       // records per (KV head, tile)
    uint32_t final = 0;        // one run of the shared kernel is all there is: it writes the output itself
    uint64_t part_floats = 0;  // offset of its records in the workspace
};

// A run of the shared kernel: the blocks one workgroup takes, a range of the request's blocks in list order.  It may
// start and end inside a document and span several.
struct Run {
    uint32_t doc, first_block;  // first document (index into the request's documents) and block in it
    uint32_t n_docs, end_block; // documents touched; end of the range in the last of them
};
constexpr uint32_t kMaxRunDocs = 128;  // a run's documents are descriptors of one launch

// How a document of a request that is not the shared kernel's is cut: equal pieces, none longer than
// run_blocks.  Their length; *n = how many.
uint32_t piece_blocks(const Plan &pl, const Doc &doc, uint32_t *n)
{
    const uint32_t nb = doc.n_blocks, parts = (nb + pl.run_blocks - 1u) / pl.run_blocks;
    const uint32_t len = parts == 1u ? nb : (nb + parts - 1u) / parts;
    *n = parts == 1u ? 1u : (nb + len - 1u) / len;
    return len;
}

// The run that starts at block `blk` of document `doc` of the request (both moved to the next
// run's start); false when the request has no block left.
bool next_run(const Plan &pl, const Doc *docs, uint32_t &doc, uint32_t &blk, Run *out)
{
    if (doc >= pl.n_docs) return false;
    out->doc = doc;
    out->first_block = blk;
    out->n_docs = 0;
    uint32_t left = pl.run_blocks;
    for (;;) {
        const uint32_t nb = docs[doc].n_blocks;
        ++out->n_docs;
        if (nb - blk > left) {  // the run ends inside this document
            blk += left;
            out->end_block = blk;
            return true;
        }
        left -= nb - blk;
        out->end_block = nb;
        ++doc;
        blk = 0;
        if (left == 0 || doc >= pl.n_docs || out->n_docs == kMaxRunDocs) return true;
    }
}

uint32_t count_runs(const Plan &pl, const Doc *docs)
{
    uint32_t doc = 0, blk = 0, n = 0;
    if (!pl.shared) {
        for (uint32_t i = 0; i < pl.n_docs; ++i) {
            piece_blocks(pl, docs[i], &blk);
            n += blk;
        }
        return n;
    }
    // No run ends for its documents: 127 whole ones and a block of another are as long as a run.
    if (pl.n_docs <= kMaxRunDocs || (uint64_t)(kMaxRunDocs - 1u) * pl.least_blocks + 1u >= pl.run_blocks)
        return (uint32_t)((pl.all_blocks + pl.run_blocks - 1u) / pl.run_blocks);
    Run r;
    while (next_run(pl, docs, doc, blk, &r)) ++n;
    return n;
}

// Steps of the longest of a request's runs of `len` blocks: a workgroup of the shared kernel takes
// up to 1 << shift blocks at a time, all of one document.
uint32_t longest_run_steps(const Plan &pl, const Doc *docs, uint32_t len, uint32_t shift)
{
    const uint32_t up = (1u << shift) - 1u;
    uint32_t most = 0, steps = 0, left = len;
    for (uint32_t i = 0; i < pl.n_docs; ++i) {
        uint32_t nb = docs[i].n_blocks;
        if (nb >= left) {  // a run ends in this document, the next ones lie inside it
            steps += (left + up) >> shift;
            if (steps > most) most = steps;
            nb -= left;
            if (nb >= len) {
                nb %= len;
                if ((len + up) >> shift > most) most = (len + up) >> shift;
            }
            steps = 0;
            left = len;
        }
        steps += (nb + up) >> shift;
        left -= nb;
    }
    return steps > most ? steps : most;
}

// The requests of a call that go to the shared kernel, those of one size together.
struct SharedCall {
    struct Size {
        uint64_t blocks;
        uint32_t n_mt, count;
    };
    static constexpr uint32_t kSizes = 32;
    const Plan *plans = nullptr;
    const Doc *docs = nullptr;
    uint32_t n_reqs = 0, H = 0;
    Size sizes[kSizes];             // in the order they come up first
    uint32_t n_sizes = 0, rest = 0; // requests from `rest` on are looked at one by one
    const Plan *largest = nullptr;
    uint32_t least_mt = ~0u, most_mt = 0;  // query tiles
    uint64_t all = 0, wide = 0;     // blocks; those of documents with a 16-bit side
    uint64_t fewest = ~0ull;        // blocks of the shortest request that has any

    SharedCall() = default;
    SharedCall(const Plan *plans_, uint32_t n_reqs_, const Doc *docs_, uint32_t H_) : plans(plans_), docs(docs_), n_reqs(n_reqs_), H(H_)
    {
        for (; rest < n_reqs; ++rest) {
            const Plan &pl = plans[rest];
            if (!pl.shared) continue;
            uint32_t i = 0;
            while (i < n_sizes && (sizes[i].blocks != pl.all_blocks || sizes[i].n_mt != pl.n_mt)) ++i;
            if (i == kSizes) break;
            if (i == n_sizes) sizes[n_sizes++] = Size{pl.all_blocks, pl.n_mt, 0u};
            ++sizes[i].count;
        }
        for (uint32_t r = 0; r < n_reqs; ++r) {
            if (!plans[r].shared) continue;
            if (!largest || plans[r].all_blocks > largest->all_blocks) largest = &plans[r];
            if (plans[r].all_blocks && plans[r].all_blocks < fewest) fewest = plans[r].all_blocks;
            if (plans[r].n_mt > most_mt) most_mt = plans[r].n_mt;
            if (plans[r].n_mt < least_mt) least_mt = plans[r].n_mt;
            all += plans[r].all_blocks;
            wide += plans[r].wide_blocks;
        }
    }
    template <class F>
    void each(F f) const
    {
        for (uint32_t i = 0; i < n_sizes; ++i) f(sizes[i].blocks, sizes[i].n_mt, sizes[i].count);
        for (uint32_t r = rest; r < n_reqs; ++r)
            if (plans[r].shared) f(plans[r].all_blocks, plans[r].n_mt, 1u);
    }
    // Workgroups of a run when 1 << wshift waves take two tiles each.
    uint32_t groups(uint32_t n_mt, uint32_t wshift) const { return H * ((n_mt + (2u << wshift) - 1u) >> (wshift + 1u)); }
    static uint64_t runs_of(uint64_t blocks, uint64_t len)
    {
        const uint64_t up = blocks + len - 1u;
        return up >> 32 ? up / len : (uint32_t)up / (uint32_t)len;
    }
    // Workgroups and records with runs of len blocks.
    uint64_t wgs = 0, recs = 0;
    void count(uint64_t len, uint32_t wshift)
    {
        if (len == counted_len && wshift == counted_wshift) return;
        counted_len = len;
        counted_wshift = wshift;
        wgs = recs = 0;
        each([&](uint64_t blocks, uint32_t n_mt, uint32_t times) {
            const uint64_t runs = runs_of(blocks, len) * times;
            wgs += runs * groups(n_mt, wshift);
            if (blocks > len) recs += runs * H * n_mt;
        });
    }
    uint64_t counted_len = 0;
    uint32_t counted_wshift = 0;
    // Blocks that all workgroups take together: their number times their length is no less.
    uint64_t work(uint32_t wshift) const
    {
        uint64_t w = 0;
        each([&](uint64_t blocks, uint32_t n_mt, uint32_t times) { w += blocks * times * groups(n_mt, wshift); });
        return w;
    }
    // Rounds that wgs workgroups (those counted last) take, `side` of them at a time.  A launch is as wide as its widest run and
    // workgroups beyond a narrower one's exit at once.  The hardware deals the launch's workgroups, those too, to the
    // chip's 32 shader engines in turn, so that an engine may get one more than it has places for while others have
    // none: 6 requests of 4, 4 and 2 groups in 9 runs, 240 workgroups of one head's width 4, took 32.6 us where one round
    // takes 17; 5 requests of 5 to 7 groups 146.9 instead of 86.6.
    uint64_t rounds(uint64_t side) const
    {
        const uint64_t even = (wgs + side - 1u) / side;
        const uint32_t width = groups(most_mt, counted_wshift);
        if (groups(least_mt, counted_wshift) == width || even > 4u) return even;  // (then they even out)
        constexpr uint32_t kEngines = 32;
        uint32_t got[kEngines] = {};
        uint32_t most = 0, whole = 0, at = 0;
        for (uint32_t r = 0; r < n_reqs; ++r) {
            if (!plans[r].shared) continue;
            const uint32_t mine = groups(plans[r].n_mt, counted_wshift);
            for (uint64_t k = runs_of(plans[r].all_blocks, counted_len); k; --k, at += width) {
                whole += mine / kEngines;
                for (uint32_t i = 0; i < mine % kEngines; ++i) ++got[(at + i) % kEngines];
            }
        }
        for (uint32_t n : got)
            if (n > most) most = n;
        const uint64_t places = side / kEngines;
        return (whole + most + places - 1u) / places;
    }
};

// The run lengths there are, by how many runs n the largest request gets: n = 1 .. last(), of ceil(blocks / n) blocks
// each, at least kAttendMinRunBlocks unless there is one.
struct RunLengths {
    uint64_t blocks;  // of the largest request, not 0
    uint64_t last() const { return blocks > kAttendMinRunBlocks ? (blocks - 1u) / (kAttendMinRunBlocks - 1u) : 1u; }
    uint64_t of(uint64_t n) const { return (blocks + n - 1u) / n; }
    uint64_t first_n(uint64_t len) const { return of(len); }                                          // the fewest runs of this length
    uint64_t last_n(uint64_t len) const { return len > 1u ? (blocks - 1u) / (len - 1u) : blocks; }  // the most
    // the largest n up to last() for whose length ok() holds, if it holds for 1 and ends to hold once; else 1
    template <class F>
    uint64_t last_where(F ok) const
    {
        uint64_t lo = 1, hi = last();
        if (hi == 1u || ok(of(hi))) return hi;
        --hi;
        while (2u * lo <= hi && ok(of(2u * lo))) lo *= 2u;  // often few: many requests fill the chip
        if (2u * lo <= hi) hi = 2u * lo - 1u;
        while (lo < hi) {
            const uint64_t mid = hi - (hi - lo) / 2u;
            if (ok(of(mid))) lo = mid;
            else hi = mid - 1u;
        }
        return lo;
    }
};

// What the cost of a run length counts as a workgroup's steps: those of the average run of the largest request (no run
// length's longest has fewer), and of a request of few documents those of its longest run too.
struct Steps {
    const SharedCall &call;
    uint32_t shift;    // a step takes up to 1 << shift blocks of one document
    uint64_t of_all;   // steps of all blocks in one run
    Steps(const SharedCall &c, uint32_t shift_)
        : call(c), shift(shift_), of_all(longest_run_steps(*c.largest, c.docs + c.largest->first_doc, ~0u, shift_)) {}
    uint64_t average(uint64_t n, uint64_t len) const
    {
        const uint64_t steps = (len + (1u << shift) - 1u) >> shift, mean = (of_all + n - 1u) / n;
        return steps > mean ? steps : mean;
    }
    bool few_docs() const { return call.largest->n_docs <= kAttendFewDocs; }
    uint64_t longest(uint64_t len) const { return longest_run_steps(*call.largest, call.docs + call.largest->first_doc, (uint32_t)len, shift); }
};

// The rule that a call's workspace is sized by.  It is older than the kernels' forms and stays what it was, since callers
// keep workspaces: for requests of up to 4, up to 8 and more tiles as if 2, 4 and 8 waves took as many blocks a
// step (in turn), which costs rounds x (blocks + 8) and a block's time for every so many records.  Of the lengths up to the
// one that takes the fewest rounds x blocks, that bounds the records.
struct Limit {
    uint32_t wshift;         // 1 << wshift waves
    uint32_t side_by_side;   // workgroups on the chip
    uint32_t recs_per_block;
};
constexpr Limit kLimits[3] = {{1u, 4u * kChipCUs, 600u}, {2u, 2u * kChipCUs, 450u}, {3u, kChipCUs, 280u}};

// in_steps: blocks count by step, not one by one (which is for a call that otherwise does not fit the array of the
// entry point without a workspace).
uint64_t limit_run(const Limit &f, SharedCall &call, bool in_steps)
{
    if (!call.largest || !call.largest->all_blocks) return 1;
    const RunLengths lengths = {call.largest->all_blocks};
    const uint64_t last = lengths.last(), side = f.side_by_side;
    auto rounds = [&](uint64_t len) {
        call.count(len, f.wshift);
        return (call.wgs + side - 1u) / side;
    };
    // The fewest rounds x blocks.  Up to the last length of one round that is the shortest; from there on until no
    // later one can take fewer (more rounds of at least 8 blocks, or all workgroups' blocks in full rounds).
    const uint64_t full = (call.work(f.wshift) + side - 1u) / side;
    uint64_t n = lengths.last_where([&](uint64_t len) { return rounds(len) <= 1u; });
    uint64_t bound = n, fewest = ~0ull;
    while (n <= last) {
        const uint64_t len = lengths.of(n), k = rounds(len);
        if (k * len < fewest) {
            fewest = k * len;
            bound = n;
        }
        if (fewest <= full || k * kAttendMinRunBlocks >= fewest || call.wgs >= 64u * side) break;
        n = lengths.last_n(len) + 1u;
    }
    // The least cost of n = 1 .. bound, the smaller n of equals.  Of the n of one length the largest costs least.
    const Steps steps(call, in_steps ? f.wshift : 0u);
    constexpr uint64_t kStart = 8;
    uint64_t best = lengths.of(bound), least = ~0ull;
    for (n = lengths.first_n(best); n; n = lengths.first_n(lengths.of(n)) - 1u) {
        const uint64_t len = lengths.of(n);
        if (len + kStart > least) break;  // and so for all longer ones
        const uint64_t k = rounds(len), mean = steps.average(n, len);
        auto cost = [&](uint64_t s) { return k * ((s << steps.shift) + kStart) + call.recs / f.recs_per_block; };
        uint64_t c = cost(mean);
        if (c <= least && steps.few_docs()) {
            const uint64_t longest = steps.longest(len);
            if (longest > mean) c = cost(longest);
        }
        if (c <= least) {
            least = c;
            best = len;
        }
    }
    return best;
}

// What a call costs the shared kernel in each of its forms, in ns.  Workgroups of one size finish in rounds of as many as
// the chip holds side by side; a round costs what starting and ending a workgroup does, its steps (a workgroup takes a few
// blocks at a time, all of one document), and for k6_attend_roles<4>, alone on its compute unit, a trip to memory at the start
// of every document; steps get slower the more workgroups share a compute unit, or the memory and the power there is, and
// for k6_attend_roles they are quicker with few blocks in them (documents of 60 tokens: half).  A run that is longer
// than the average one costs a third of the difference: its neighbours are done by then.  Every record is 8 KiB that is
// written, flushed at the kernel's end and read by another launch.  k6_attend_shared<2> and k6_attend_roles<8> were fitted to
// timings of 142 calls whose runs and forms were set by hand, <4> of both to 79 and 492 timings of random calls, of which they
// are off by 8 and 6 %.  180 random calls that were no part of it, of 1 to 32 requests, 1 to 16 documents and 3 and more
// tiles, take 0.92 of the time on average that they took when forms went by tiles alone, 1.11 at worst, 0.69 at best.  The
// time to choose is not part of it: 1 to 5 us of host time a call.
struct Form {
    uint32_t wshift, shift, side_by_side;  // 1 << wshift waves; 1 << shift blocks a step
    uint32_t call, round, doc;             // ns: once; a round; a document
    uint32_t step[4];                      // ns: a step with up to a quarter, a half, three quarters and all places taken
    uint32_t wide;                         // added to a step times the share of blocks with a 16-bit side
    uint32_t idle;                         // percent: what a step without any block would take less than a full one
};
constexpr Form kForms[4] = {  // by SharedForm
    {1u, 1u, 4u * kChipCUs, 2000u, 5600u, 0u, {1330u, 2115u, 2120u, 2300u}, 460u, 0u},
    {2u, 2u, 2u * kChipCUs, 7800u, 0u, 0u, {1220u, 2530u, 2710u, 2710u}, 0u, 0u},
    {2u, 3u, kChipCUs, 4700u, 2500u, 300u, {1700u, 2780u, 2780u, 2940u}, 180u, 50u},
    {3u, 3u, kChipCUs, 2500u, 6100u, 0u, {3050u, 3230u, 3540u, 3960u}, 210u, 50u},
};
constexpr uint64_t kMergeNs = 3740, kRecNsNum = 19, kRecNsDen = 10;  // a merge at all; a record
// Without a merge: the runs' own end, which divides the rows and finds their place in the output.  1.6 to 3.5 us were missing
// from such calls; left out, 9 requests of 2 x 256 tokens at 3 tiles went to four scorers for 20.0 us instead of 17.7, 10 of
// 4 x 256 at 16 tiles for 35.6 instead of 32.8.
constexpr uint64_t kFinalNs = 2500;

struct FormCost {
    const Form &f;
    SharedCall &call;
    const RunLengths lengths;
    const Steps steps;
    const uint64_t wide_ns, fill;  // fill: of 1024, blocks in the steps of the largest request


    FormCost(const Form &f_, SharedCall &c)
        : f(f_), call(c), lengths{c.largest->all_blocks}, steps(c, f_.shift), wide_ns(f_.wide * c.wide / c.all),
          fill(1024u * lengths.blocks / (steps.of_all << f_.shift)) {}
    uint64_t filled(uint64_t ns) const { return ns + wide_ns - (ns + wide_ns) * (1024u - fill) * f.idle / (1024u * 100u); }
    uint64_t full_rounds(uint64_t len)  // no more than it takes
    {
        call.count(len, f.wshift);
        return (call.wgs + f.side_by_side - 1u) / f.side_by_side;
    }
    uint64_t step_ns() const  // with as many workgroups as counted last, between two of the four
    {
        const uint64_t taken = call.wgs < f.side_by_side ? call.wgs : f.side_by_side;  // places
        const uint64_t quarter = f.side_by_side / 4u, q = taken <= quarter ? 0u : (taken - 1u) / quarter - 1u;
        uint64_t step = f.step[q];
        if (taken > quarter) step += (f.step[q + 1u] - f.step[q]) * (taken - (q + 1u) * quarter) / quarter;
        return filled(step);
    }
    uint64_t end_ns() const { return call.recs ? kMergeNs + call.recs * kRecNsNum / kRecNsDen : kFinalNs; }
    // of n runs, len = lengths.of(n), if that is no more than `most`; else at least not less than it costs on average
    uint64_t of(uint64_t n, uint64_t len, uint64_t most)
    {
        const uint64_t full = full_rounds(len), more = call.rounds(f.side_by_side) - full, step = step_ns(), mean = steps.average(n, len);
        const uint64_t in_docs = (call.largest->n_docs * len + lengths.blocks - 1u) / lengths.blocks * f.doc;
        // Of eight scorers a later round counts three quarters: 8 such calls of 14 to 29 requests took 0.76 to 0.85 of what
        // whole rounds come to (115 us of 136), four scorers 0.78 to 1.16 (141 of 131).
        const uint64_t quarters = f.wshift == 3u ? 1u + 3u * full : 4u * full;
        uint64_t c = f.call + quarters * (f.round + mean * step + in_docs) / 4u + end_ns();
        if (more) {  // what an engine has no place for starts when its first workgroups end
            const uint64_t blocks = call.fewest < len ? call.fewest : len;
            c += more * (f.round + ((blocks + (1u << f.shift) - 1u) >> f.shift) * step);
        }
        if (c <= most && steps.few_docs()) {
            const uint64_t longest = steps.longest(len);
            if (longest > mean) c += quarters * ((longest - mean) * step / 3u) / 4u;
        }
        return c;
    }
    // The length that costs least of those whose records take no more than most_floats words (one run a request takes
    // none), the smaller n of equals; of the n of one length the largest costs least.  *ns: what it costs, or as it was if
    // that is no more.
    uint64_t best(uint64_t most_floats, uint64_t *ns)
    {
        const uint64_t last = lengths.last(), side = f.side_by_side;
        auto fits = [&]() { return call.recs * kAttendRecFloats <= most_floats; };
        const uint64_t start = lengths.last_where([&](uint64_t len) { return full_rounds(len) <= 1u && fits(); });
        uint64_t least = *ns, best_len = lengths.of(start);
        auto most_n = [&](uint64_t len) {
            const uint64_t n = lengths.last_n(len);
            return n < last ? n : last;
        };
        for (uint64_t n = most_n(best_len); n; n = lengths.first_n(lengths.of(n)) - 1u) {  // longer and longer ones
            const uint64_t len = lengths.of(n);
            if (f.call + f.round + ((len + (1u << f.shift) - 1u) >> f.shift) * filled(f.step[0]) > least) break;
            const uint64_t c = of(n, len, least);
            if (c <= least) {
                least = c;
                best_len = len;
            }
        }
        // shorter and shorter ones, until rounds, records and all workgroups' blocks in full rounds cost as much
        const uint64_t full = call.work(f.wshift), full_steps = (full + (side << f.shift) - 1u) / (side << f.shift);
        uint64_t len = lengths.of(start);
        full_rounds(len);
        while (call.wgs < 64u * side && lengths.last_n(len) < last) {  // finer than this gains nothing
            uint64_t n = lengths.last_n(len) + 1u;
            len = lengths.of(n);
            const uint64_t k = full_rounds(len);
            if (!fits() || f.call + k * f.round + full_steps * step_ns() + end_ns() >= least) break;
            if (call.wgs < 64u * side) n = most_n(len);
            const uint64_t c = of(n, len, least);
            if (c < least) {
                least = c;
                best_len = len;
            }
        }
        *ns = least;
        return best_len;
    }
};

// Cuts the requests of one kernel (the shared one or the other) into runs and lays their part of the workspace out,
// from word `total` on.  Returns where it ends.
uint64_t cut(Plan *plans, uint32_t n_reqs, const Doc *docs, uint32_t H, bool shared, uint64_t run_blocks, uint64_t total)
{
    for (uint32_t r = 0; r < n_reqs; ++r) {
        Plan &pl = plans[r];
        if ((pl.shared != 0u) != shared) continue;
        pl.run_blocks = run_blocks > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)(run_blocks ? run_blocks : 1u);
        pl.n_runs = count_runs(pl, docs + pl.first_doc);
        pl.final = shared && pl.n_runs == 1u;  // no record, no merge
        pl.part_floats = total;
        if (!pl.final) total += (uint64_t)pl.n_runs * H * pl.n_mt * kAttendRecFloats;
    }
    return total;
}

// Requests of at most two query tiles: a run is a piece of one document, as long as
// possible (every workgroup pays for fetching the queries and for writing a record), but
// short enough that the launch fills the chip a few times over, since the hardware then
// evens out what documents of different formats and lengths take.
uint32_t piece_length(const Plan *plans, uint32_t n_reqs, const Doc *docs, uint32_t H)
{
    auto groups_at = [&](uint32_t shift) {  // workgroups with pieces of 1 << shift blocks
        uint64_t groups = 0;
        for (uint32_t r = 0; r < n_reqs; ++r) {
            const Plan &pl = plans[r];
            if (pl.shared) continue;
            uint64_t runs = 0;
            for (uint32_t i = 0; i < pl.n_docs; ++i) runs += (docs[pl.first_doc + i].n_blocks + (1u << shift) - 1u) >> shift;
            groups += runs * H * ((pl.n_mt + 1u) / 2u);
        }
        return groups;
    };
    static_assert(kAttendMaxRunBlocks == 128u, "a power of two");
    uint32_t shift = 7;
    while ((1u << shift) > kAttendMinRunBlocks && groups_at(shift) < kAttendTargetGroups) --shift;
    // A call of so few workgroups that even twice as many run side by side (four per CU) is
    // bound by how long one of them takes: halve once more (one request of 10 x 512 tokens:
    // 13.7 against 14.7 us; with two requests, 1,280 workgroups, it would cost 1.5 us).
    if ((1u << shift) == kAttendMinRunBlocks && groups_at(shift - 1u) <= 4ull * kChipCUs) --shift;
    return 1u << shift;
}

void set_shared(Plan *plans, uint32_t n_reqs, bool two_tiles)  // two_tiles: requests of two tiles as well
{
    for (uint32_t r = 0; r < n_reqs; ++r) plans[r].shared = plans[r].n_mt > 2u || (two_tiles && plans[r].n_mt == 2u);
}

// Lays out the requests that are not the shared kernel's; words.
uint64_t lay_out_pieces(Plan *plans, uint32_t n_reqs, const Doc *docs, uint32_t H)
{
    for (uint32_t r = 0; r < n_reqs; ++r)
        if (!plans[r].shared) return cut(plans, n_reqs, docs, H, false, piece_length(plans, n_reqs, docs, H), 0);
    return 0;
}

// What k6_attend_partial costs a call whose largest request has five to eight tiles, in ns: a launch, and per block and KV
// head 1.25 ns up to 28,000 of them, 0.82 from there on, when pieces are long and all places taken.  Two-tile requests in a
// launch of their own or with the others in k6_attend_roles<4>, where each keeps one of four scorers busy; us a layer, 10 x
// 512 tokens: one request of 32 query tokens and 31 of 8: 110.6 / 127.0 (paper's formats 117.4 / 124.2), 8 of 20 and 24 of 5:
// 117.5 / 126.1 (123.5 / 123.9), 16 of 32 and 16 of 8: 140.2 / 130.1 (145.6 / 127.3), one of 32 and 15 of 8: 76.5 / 70.6, one
// and seven: 59.3 / 41.0, one and one: 38.7 / 23.9; 16 of 700 and 333 tokens at 20, 6, 1 and 8, where there is a launch for the
// one-tile requests anyway: 42.0 / 44.4.  Fitted to these and 35 calls like them, where it chooses the faster way each time; of 34 others drawn
// at random it was off the faster one by 5 to 6 % in three, by up to 2 % in two, and the other way would have cost up to 71 %.
uint64_t pieces_ns(const Plan *plans, uint32_t n_reqs, uint32_t H)
{
    uint64_t blocks = 0;
    for (uint32_t r = 0; r < n_reqs; ++r)
        if (!plans[r].shared) blocks += plans[r].all_blocks * H;
    if (!blocks) return 0;
    constexpr uint64_t kFew = 28000;
    return 14000u + (blocks < kFew ? blocks * 5u / 4u : kFew * 5u / 4u + (blocks - kFew) * 41u / 50u);
}

// Lays out a call whose largest request has most_mt > 2 tiles.  Returns the words of the workspace it asks for (see
// Limit), which the layout stays within; *form: the shared kernel's.
uint64_t lay_out_shared(Plan *plans, uint32_t n_reqs, const Doc *docs, uint32_t H, uint32_t most_mt, uint64_t most_floats, SharedForm *form)
{
    SharedCall call;
    uint64_t pieces = 0;
    auto set = [&](bool two_tiles) {  // the shared kernel's requests, those of two tiles among them or not; lays out the others
        for (uint32_t r = 0; r < n_reqs; ++r) plans[r].shared = plans[r].n_mt > 2u || (two_tiles && plans[r].n_mt == 2u);
        call = SharedCall(plans, n_reqs, docs, H);
        pieces = lay_out_pieces(plans, n_reqs, docs, H);
    };
    auto lay_out = [&](uint64_t run_blocks) { return cut(plans, n_reqs, docs, H, true, run_blocks, pieces); };
    bool twos = false;
    for (uint32_t r = 0; r < n_reqs; ++r) twos |= plans[r].n_mt == 2u;

    // The layout that the workspace is sized by.  A call whose largest request has three or four tiles takes its requests of
    // two to the shared kernel as well, unless that needs more workspace: a block costs that kernel what it costs the
    // other one (103 against 100 us per call of 32 requests), and one launch fills the chip where two in a row
    // do not (12 requests of 6 to 16 query tokens: 46 against 63 us per layer).
    const Limit &limit = kLimits[most_mt > 8u ? 2 : most_mt > 4u ? 1 : 0];
    const SharedForm limit_form = most_mt > 8u ? SharedForm::kRoles8 : most_mt > 4u ? SharedForm::kShared4 : SharedForm::kShared2;
    bool limit_twos = false;
    uint64_t limit_len = 1, total = 0;
    for (bool in_steps : {true, false}) {
        set(limit_twos = false);
        limit_len = limit_run(limit, call, in_steps);
        total = lay_out(limit_len);
        if (twos && most_mt <= 4u) {
            set(limit_twos = true);
            const uint64_t len = limit_run(limit, call, in_steps), together = lay_out(len);
            if (together <= total) {
                total = together;
                limit_len = len;
            } else {
                set(limit_twos = false);
                lay_out(limit_len);
            }
        }
        if (total <= most_floats) break;
    }
    *form = limit_form;
    if (!call.all) return total;

    // The forms: four scorers (up to 8 tiles a workgroup) for every call; eight where a request has more
    // tiles, which then decodes every block once less; and k6_attend_shared, whose workgroups on a compute unit (four of two
    // waves, two of four) all decode and score in turn, for requests of up to four tiles, where half of four scorers would have
    // none, and of five to eight (see there).  Measured, us
    // a layer, k6_attend_shared / four scorers / eight: 12 query tokens, 8 requests x 4 x 512 tokens 23.9 / 23.0, 32 x 10 x
    // 512 109 / 136, 12 ragged requests in the paper's formats 42 / 53; 64 query tokens, 2 x 4 x 512 - / 23.1 / 26.5, 16 x
    // 4 x 512 - / 72.9 / 60.7, 32 x 10 x 512 - / 288 / 205.
    // Four scorers are as exact in long runs as in short ones (role_add_round) and take the length that costs least; the
    // others keep the runs that the workspace is sized for: longer ones cost them up to 1.8 times the error.
    const bool middle = limit_form == SharedForm::kShared4;
    const Form &four = kForms[(uint32_t)SharedForm::kRoles4];
    uint64_t used = ~0ull;
    if (twos && middle) {  // those of two tiles go there too if that costs less and the workspace holds it
        uint64_t apart_ns = ~0ull, ns = ~0ull;
        FormCost(four, call).best(total > pieces ? total - pieces : 0u, &apart_ns);
        apart_ns += pieces_ns(plans, n_reqs, H);
        set(true);
        const uint64_t len = FormCost(four, call).best(total > pieces ? total - pieces : 0u, &ns);
        if (ns + pieces_ns(plans, n_reqs, H) <= apart_ns) used = lay_out(len);
        *form = SharedForm::kRoles4;
        if (used > total) {
            set(false);
            lay_out(limit_len);
        }
    }
    if (used > total) {
        FormCost other(kForms[(uint32_t)limit_form], call);
        const uint64_t other_ns = other.of(other.lengths.first_n(limit_len), limit_len, ~0ull);
        uint64_t ns = middle ? ~0ull : other_ns;
        const uint64_t len = FormCost(four, call).best(total > pieces ? total - pieces : 0u, &ns);
        // The form that the workspace is sized by also on an even estimate; k6_attend_shared<4>, whose costs are the least
        // certain, where it is expected to take a sixteenth less: 43 of 213 calls, 0.73 to 1.08 times what four scorers take.
        *form = limit_form;
        if (other_ns <= (middle ? ns - ns / 16u : ns + ns / 32u)) return total;  // laid out already
        *form = SharedForm::kRoles4;
        used = lay_out(len);
    }
    // The run length was chosen by the quotient of blocks and length, but a run also ends after kMaxRunDocs
    // documents, so that a request of more than that may have more runs.  Any form takes runs of any length:
    // where they do not fit, those that the workspace is sized by.
    if (used > total) {
        lay_out(limit_len);
        *form = limit_form;
    }
    return total;
}

// Checks everything and lays the workspace out.  *floats = workspace size in binary32 words.
// plans: n_reqs entries; docs, open_k, open_v: filled here, ENOSPC if one of them is too small
// (never with lists as long as the call's chunk list).  most_floats: what a workspace of fixed size holds.
int plan_attend(ha_rag_ctx *c, const ha_rag_packed_chunk *chunks, const ha_rag_attend_request *reqs,
                uint32_t n_reqs, uint32_t n_q_heads, Plan *plans, Fixed<Doc> *docs,
                Fixed<uint32_t> open_k, Fixed<uint32_t> open_v, uint64_t *floats,
                SharedForm *form, bool need_buffers, uint64_t most_floats = ~0ull)
{
    if (!c || !reqs || n_reqs == 0 || n_reqs > HA_RAG_MAX_ATTEND_REQUESTS) return HA_RAG_EINVAL;
    if (c->cfg.head_dim != kAttendHeadDim) return HA_RAG_EFORMAT;
    const uint32_t H = c->cfg.n_kv_heads;
    if (n_q_heads == 0 || n_q_heads % H || n_q_heads / H > 64) return HA_RAG_EINVAL;
    const uint32_t G = n_q_heads / H;
    uint64_t n_chunks = 0;
    docs->clear();
    // open_k / open_v: documents still waiting for their values / keys
    for (uint32_t r = 0; r < n_reqs; ++r) {
        const ha_rag_attend_request &rq = reqs[r];
        Plan &pl = plans[r];
        pl = Plan();
        if (rq.n_q == 0 || rq.n_q > HA_RAG_MAX_ATTEND_Q) return HA_RAG_EINVAL;
        if (need_buffers && (!rq.q || !rq.out || ((uintptr_t)rq.q & 15u) || ((uintptr_t)rq.out & 15u)))
            return HA_RAG_EINVAL;
        if (n_chunks + rq.n_chunks > HA_RAG_MAX_REQUEST_CHUNKS || (rq.n_chunks && !chunks))
            return HA_RAG_EINVAL;
        pl.first_doc = (uint32_t)docs->size();
        pl.n_mt = (rq.n_q * G + 15u) / 16u;
        pl.shared = pl.n_mt > 2u;
        open_k.clear();
        open_v.clear();
        size_t next_k = 0, next_v = 0;  // first entries of open_k / open_v not yet matched
        for (uint32_t i = 0; i < rq.n_chunks; ++i) {
            const ha_rag_packed_chunk &pc = chunks[n_chunks + i];
            size_t tile = 0;  // bytes of one tile record: what a keys-only chunk of one layer and head takes
            int rc = chunk_bytes_impl(1, 1, c->cfg.head_dim, pc.prec, pc.group, pc.n_tokens, nullptr,
                                      nullptr, &tile, pc.part == HA_RAG_PART_KV ? (uint32_t)HA_RAG_PART_K : pc.part);
            if (rc) return rc;
            if (pc.n_tokens == 0) continue;  // holds nothing, pairs with nothing
            if (need_buffers && (!pc.packed || ((uintptr_t)pc.packed & 15u))) return HA_RAG_EINVAL;
            const uint8_t *ptr = static_cast<const uint8_t *>(pc.packed);
            const uint32_t fmt = pc.prec | ((has_meta(pc.prec) ? log2u(pc.group) : 0u) << 4);
            if (pc.part == HA_RAG_PART_KV) {
                Doc d;
                d.k = d.v = ptr;
                d.k_tile = d.v_tile = tile;
                d.k_first = 0;
                d.v_first = H;
                d.k_step = d.v_step = 2u * H;
                d.n_tokens = pc.n_tokens;
                d.n_blocks = (pc.n_tokens + 15u) / 16u;
                d.info = fmt | (fmt << 8);
                if (!docs->push_back(d)) return HA_RAG_ENOSPC;
            } else {
                // the i-th keys-only chunk of the request and its i-th values-only chunk are one
                // document: they must hold the same tokens
                const bool is_k = pc.part == HA_RAG_PART_K;
                Fixed<uint32_t> &mine = is_k ? open_k : open_v, &other = is_k ? open_v : open_k;
                size_t &other_next = is_k ? next_v : next_k;
                uint32_t di;
                if (other_next < other.size()) {
                    di = other[other_next++];
                    if ((*docs)[di].n_tokens != pc.n_tokens) return HA_RAG_EINVAL;
                } else {
                    di = (uint32_t)docs->size();
                    if (!docs->push_back(Doc()) || !mine.push_back(di)) return HA_RAG_ENOSPC;
                    (*docs)[di].n_tokens = pc.n_tokens;
                    (*docs)[di].n_blocks = (pc.n_tokens + 15u) / 16u;
                }
                Doc &d = (*docs)[di];
                (is_k ? d.k : d.v) = ptr;
                (is_k ? d.k_tile : d.v_tile) = tile;
                (is_k ? d.k_step : d.v_step) = H;
                d.info |= is_k ? fmt : fmt << 8;
            }
        }
        if (next_k != open_k.size() || next_v != open_v.size()) return HA_RAG_EINVAL;  // keys without values or the reverse
        pl.n_docs = (uint32_t)docs->size() - pl.first_doc;
        n_chunks += rq.n_chunks;
    }
    uint32_t most_mt = 0;  // of the requests with more than two tiles
    for (uint32_t r = 0; r < n_reqs; ++r) {
        Plan &pl = plans[r];
        if (pl.shared && pl.n_mt > most_mt) most_mt = pl.n_mt;
        pl.all_blocks = pl.wide_blocks = 0;
        for (uint32_t i = 0; i < pl.n_docs; ++i) {
            const Doc &doc = (*docs)[pl.first_doc + i];
            pl.all_blocks += doc.n_blocks;
            if ((doc.info & 0xFu) == HA_RAG_PREC_16 || ((doc.info >> 8) & 0xFu) == HA_RAG_PREC_16) pl.wide_blocks += doc.n_blocks;
            if (i == 0 || doc.n_blocks < pl.least_blocks) pl.least_blocks = doc.n_blocks;
        }
    }
    *form = SharedForm::kShared2;
    const uint64_t total = most_mt ? lay_out_shared(plans, n_reqs, docs->data, H, most_mt, most_floats, form)
                                   : lay_out_pieces(plans, n_reqs, docs->data, H);
    if (total * 4ull > (1ull << 40)) return HA_RAG_EINVAL;
    *floats = total;
    return HA_RAG_OK;
}


// How many of a call's documents were listed before, of those looked at: all, or if they are more than kMost a part
// that is chosen by where their keys lie, so that a document is looked at each time that it is listed or never.
struct RepeatedDocs {
    uint32_t looked = 0, repeated = 0;
};
RepeatedDocs repeated_docs(const Plan *plans, uint32_t n_reqs, const Doc *docs)
{
    constexpr uint32_t kMost = 1024;
    const uint8_t *place[2 * kMost];  // a call of few documents clears and uses few
    auto mixed = [](const uint8_t *at) {  // the finaliser of splitmix64: addresses come evenly spaced
        uint64_t x = (uint64_t)(uintptr_t)at;
        x = (x ^ x >> 30) * 0xBF58476D1CE4E5B9ull;
        x = (x ^ x >> 27) * 0x94D049BB133111EBull;
        return x ^ x >> 31;
    };
    uint32_t all = 0, shift = 0;
    for (uint32_t r = 0; r < n_reqs; ++r)
        if (!plans[r].shared) all += plans[r].n_docs;
    while (all >> shift > kMost) ++shift;
    uint32_t places = 16;
    while (places < 2u * (all >> shift)) places *= 2u;
    std::fill_n(place, places, nullptr);
    RepeatedDocs n;
    for (uint32_t r = 0; r < n_reqs; ++r) {
        if (plans[r].shared) continue;
        const Doc *d = docs + plans[r].first_doc;
        for (uint32_t i = 0; i < plans[r].n_docs; ++i) {
            const uint64_t x = mixed(d[i].k);
            if (x & ((1u << shift) - 1u)) continue;
            uint32_t at = (uint32_t)(x >> 32) & (places - 1u);
            while (place[at] && place[at] != d[i].k) at = (at + 1u) & (places - 1u);
            if (place[at]) ++n.repeated;
            else if (n.looked - n.repeated == places / 4u * 3u) return n;  // more than expected; places stay empty
            else place[at] = d[i].k;
            ++n.looked;
        }
    }
    if (!n.looked) n.looked = 1;
    return n;
}

// Whether k6_attend_partial reads its documents past the last-level cache, with nontemporal loads.  A layer's bytes are asked
// for again by the next query token, after those of all other layers, so what counts is their sum over the layers: up to the
// cache's size they come out of it, from a fifth more on they do not.  Beyond that it is the work that decides: short
// runs wait for their first loads, which take longer this way, and 16-bit blocks, four times the bytes of 4-bit ones, still find
// some of them in the cache.  Nontemporal loads / ordinary ones, means of the ratio of a pass at one query token, 4,400 random
// calls of 1 to 32 layers (up to 1,000 MB, 2 to 16 KV heads, 128 to 2,000 tokens a document), by the MB of all layers:
//                                            200-256  256-290  290-320  320-360  360-420  420-537  537-700  from 700
//   no 16-bit side, runs of 4 to 8 blocks       1.05     1.02     0.99     0.98     0.98     0.98     0.97     0.97
//   no 16-bit side, 13 blocks and more          1.08     1.05     1.00     0.95     0.94     0.95     0.94     0.94
//   a fifth to a half in 16 bits, 7 to 9        1.14     1.09     1.04     1.04     1.02     1.03     1.02     1.02
//   a fifth to a half in 16 bits, 18 to 125     1.07     1.07     1.06     0.97     0.95     0.95     0.94     0.95
//   all in 16 bits, 7 to 9                      1.28     1.24     1.18     1.17     1.15     1.12     1.07     1.10
//   all in 16 bits, 18 to 40                       -        -        -        -     0.97        -     0.97     0.98
// (13 to 18 blocks, partly or all in 16 bits: 0.98 to 1.05.)  With the cache full of other data, as behind the
// weights of a layer, the same: 0.99, 0.95, 1.03, 0.96, 1.11 and 0.98.  Calls with a fifth to a half in 16 bits whose workgroups are
// all on the chip at once (four a compute unit) are faster this way with short runs too: 0.96 to 0.99, with the cache full of
// other data 0.97 to 1.03; all in 16 bits 1.00 to 1.06.  us a pass, ordinary / nontemporal, 10 x 512 tokens
// a request: 32 requests in 20 / 30 / 50 % of 16, 8 and 4 bits, two layers (655 MB) 151 / 141; 12, four layers (467 MB) 142 /
// 154; two, 32 layers (655 MB) 439 / 421, six 763 / 768; FP8, 20 requests, two layers (419 MB) 98 / 93; 16 bits, 10 requests, two
// layers (419 MB) 101 / 118.  By this rule 1.4 % of the calls take more than 2 % longer than with ordinary loads: 4-bit ones of
// eight layers, up to 7 %.
// Documents that several requests of the call list come out of the cache for the second of them.  They count once, and where
// they are many ordinary loads are faster: 32 or 48 requests of 10 x 512 tokens, 503 to 1,342 MB, of which this share was listed
// before (nearby, or after all others), ratio as above: FP8 and GSE-8, a tenth 0.90 to 0.95, a quarter 0.94 to 0.99, a
// third 0.96 to 1.02, half 1.00 to 1.07; with a fifth of the documents in 16 bits, a twentieth 0.95 to 0.98, a tenth 0.96 to 0.99, a
// fifth 0.96 to 1.02, a quarter 0.96 to 1.04.
// Documents in pinned host memory come over the link and slow a call that has any of them down to its pace; nontemporal
// loads fetch them in smaller pieces: ten requests of 10 x 512 tokens, two layers, 16 bits 6,274 / 8,729 us, five of eight
// layers, FP8, 6,347 / 6,753.  Hence ordinary loads for such calls.  in_host: the caller knows of one; those listed by address are
// looked up in the slabs of that tier.
bool read_past_cache(const ha_rag_ctx *c, const Plan *plans, uint32_t n_reqs, const Doc *docs, bool in_host)
{
    if (in_host) return false;
    uint64_t bytes = 0, blocks = 0, wide = 0, n_runs = 0;  // bytes: of one layer and head
    for (uint32_t r = 0; r < n_reqs; ++r) {
        const Plan &pl = plans[r];
        if (pl.shared) continue;
        const Doc *d = docs + pl.first_doc;
        for (uint32_t i = 0; i < pl.n_docs; ++i) bytes += d[i].k_tile + d[i].v_tile;
        blocks += pl.all_blocks;
        wide += pl.wide_blocks;
        n_runs += pl.n_runs;
    }
    const uint64_t H = c->cfg.n_kv_heads, most = (wide ? kLastLevelBytes / 4u * 5u : kLastLevelBytes / 5u * 6u) / c->cfg.n_layers;
    if (bytes * H <= most) return false;
    const bool few = n_runs * H <= 4u * kChipCUs && wide * 3u <= blocks;
    if (wide && blocks < n_runs * kPastWideRunBlocks && !few) return false;
    for (const Slab &sl : c->slab[HA_RAG_TIER_PINNED]) {
        if (!sl.holds_copies()) continue;
        const uintptr_t base = (uintptr_t)sl.base, size = (uintptr_t)sl.n_slots * sl.slot_bytes;
        for (uint32_t r = 0; r < n_reqs; ++r) {
            if (plans[r].shared) continue;
            const Doc *d = docs + plans[r].first_doc;
            for (uint32_t i = 0; i < plans[r].n_docs; ++i)
                if ((uintptr_t)d[i].k - base < size || (uintptr_t)d[i].v - base < size) return false;
        }
    }
    const RepeatedDocs again = repeated_docs(plans, n_reqs, docs);
    if (again.repeated * (wide ? 8u : 4u) > again.looked) return false;
    return (bytes - bytes / again.looked * again.repeated) * H > most;
}

// Storage of one call's plan.  The ordinary entry points size it for the call on the heap; the
// entry point that allocates nothing keeps a small one on the stack.
struct PlanStore {
    Plan *plans;
    Fixed<Doc> docs;
    Fixed<uint32_t> open_k, open_v;
};

struct HeapPlanStore {  // one allocation, not cleared: the lists' entries are written when they are added
    std::unique_ptr<char[]> mem;
    PlanStore ps{};
    HeapPlanStore(const ha_rag_attend_request *reqs, uint32_t n_reqs)
    {
        uint64_t n = 0;
        if (reqs && n_reqs <= HA_RAG_MAX_ATTEND_REQUESTS)
            for (uint32_t r = 0; r < n_reqs; ++r) n += reqs[r].n_chunks;
        if (n > HA_RAG_MAX_REQUEST_CHUNKS) n = 0;  // the planning refuses the call anyway
        const size_t np = n_reqs <= HA_RAG_MAX_ATTEND_REQUESTS ? n_reqs : 0;
        static_assert(std::is_trivially_copyable<Plan>::value && std::is_trivially_copyable<Doc>::value && alignof(Plan) == 8 && alignof(Doc) == 8, "");
        mem.reset(new char[np * sizeof(Plan) + (size_t)n * (sizeof(Doc) + 2u * sizeof(uint32_t))]);
        ps.plans = reinterpret_cast<Plan *>(mem.get());
        Doc *docs = reinterpret_cast<Doc *>(ps.plans + np);
        uint32_t *open = reinterpret_cast<uint32_t *>(docs + n);
        ps.docs = Fixed<Doc>(docs, (uint32_t)n);
        ps.open_k = Fixed<uint32_t>(open, (uint32_t)n);
        ps.open_v = Fixed<uint32_t>(open + n, (uint32_t)n);
    }
    PlanStore store() { return ps; }
};

// checks, workspace layout and launches; the caller holds the context's lock.  in_host: some chunk is known to lie in
// pinned host memory.  *need (nullable)
// receives the workspace bytes the lists ask for, also when the call then fails with ENOSPC; it is given
// where the workspace's size is fixed and not the one asked for.
int attend_locked(ha_rag_ctx *c, PlanStore ps, const ha_rag_packed_chunk *chunks,
                  const ha_rag_attend_request *reqs, uint32_t n_reqs, uint32_t layer,
                  uint32_t n_q_heads, float sm_scale, void *workspace, size_t workspace_bytes,
                  void *stream, bool in_host = false, uint64_t *need = nullptr)
{
    uint64_t floats = 0;
    SharedForm form = SharedForm::kShared2;
    int rc = plan_attend(c, chunks, reqs, n_reqs, n_q_heads, ps.plans, &ps.docs, ps.open_k, ps.open_v,
                         &floats, &form, true, need ? workspace_bytes / 4u : ~0ull);
    if (rc) return rc;
    const Plan *plans = ps.plans;
    const Fixed<Doc> &docs = ps.docs;
    if (need) *need = floats * 4ull;
    if (layer >= c->cfg.n_layers || !(sm_scale > 0.0f) || !(sm_scale < 1e30f)) return HA_RAG_EINVAL;
    if (floats && (!workspace || ((uintptr_t)workspace & 15u))) return HA_RAG_EINVAL;
    if (floats * 4ull > workspace_bytes) return HA_RAG_ENOSPC;
    // a context without a device fills and checks the launches' descriptors all the same
    const bool dry = c->dry();
    hipStream_t st = (hipStream_t)stream;
    const uint32_t H = c->cfg.n_kv_heads;
    float *ws = static_cast<float *>(workspace);

    // The launch in the making (36 KiB, of which only what it uses is written): first the requests for
    // k6_attend_partial, then those for the shared kernel.
    K6Params kq;
    kq.n_kv_heads = H;
    kq.n_q_heads = n_q_heads;
    kq.layer = layer;
    kq.scale_log2 = sm_scale * 1.44269504088896341f;
    auto doc_k = [&](const Doc &doc) { return doc.k + (uint64_t)(doc.k_first + layer * doc.k_step) * doc.k_tile; };
    auto doc_v = [&](const Doc &doc) { return doc.v + (uint64_t)(doc.v_first + layer * doc.v_step) * doc.v_tile; };
    // Every run's records lie in the workspace (the planning sees to it; nothing is launched that would not).
    auto record_fits = [&](const float *part, const Plan &pl) {
        const uint64_t at = (uint64_t)((uintptr_t)part - (uintptr_t)ws) / 4u;
        return at + (uint64_t)H * pl.n_mt * kAttendRecFloats <= floats;
    };
    // ---- requests of at most two tiles: every run is a piece of one document
    kq.n_runs = 0;
    kq.past = read_past_cache(c, plans, n_reqs, docs.data, in_host);
    kq.heads_first = 0;
    for (uint32_t r = 0; r < n_reqs; ++r)  // the call's longest run
        kq.heads_first |= plans[r].shared && std::min<uint64_t>(plans[r].run_blocks, plans[r].all_blocks) >= kHeadsFirstBlocks;
    auto launch_pieces = [&]() {
        kq.doc_first = kq.doc_end = K6Params::docs_behind(kq.n_runs);
        const hipError_t e = launch_k6(kq, st, dry);
        kq.n_runs = 0;
        return e;
    };
    for (uint32_t r = 0; r < n_reqs; ++r) {
        const Plan &pl = plans[r];
        if (pl.shared) continue;
        const ha_rag_attend_request &rq = reqs[r];
        float *part = ws + pl.part_floats;
        for (uint32_t i = 0; i < pl.n_docs; ++i) {
            const Doc &doc = docs[pl.first_doc + i];
            uint32_t n_pieces = 0;
            const uint32_t len = piece_blocks(pl, doc, &n_pieces);
            K6Run d;
            d.k = doc_k(doc);
            d.v = doc_v(doc);
            d.q = static_cast<const uint16_t *>(rq.q);
            d.n_tokens = doc.n_tokens;
            d.info = doc.info;
            d.n_q = rq.n_q;
            d.final = 0;
            d.n_docs = 1;
            d.more = 0;
            d.lse = nullptr;
            for (uint32_t at = 0; at < doc.n_blocks; at += len) {
                if (kq.n_runs == kAttendMaxRuns) HIPCHK(c, launch_pieces());
                if (!record_fits(part, pl)) return HA_RAG_EINVAL;
                d.part = part;
                d.first_block = at;
                d.end_block = doc.n_blocks - at > len ? at + len : doc.n_blocks;
                kq.run[kq.n_runs++] = d;
                part += (uint64_t)H * pl.n_mt * kAttendRecFloats;
            }
        }
    }
    if (kq.n_runs) HIPCHK(c, launch_pieces());

    // ---- the others: a launch lists its runs (one grid row each), then the runs' further documents run by run.
    // A run never straddles two launches: first count the runs that fit, then fill.
    struct RunPos {
        uint32_t r, doc, blk, run_no;  // request, start of the next run in it, number of that run
    };
    auto settle = [&](RunPos &p) {  // moves p to the next run there is; false at the end
        while (p.r < n_reqs && (!plans[p.r].shared || p.doc >= plans[p.r].n_docs)) {
            ++p.r;
            p.doc = p.blk = p.run_no = 0;
        }
        return p.r < n_reqs;
    };
    auto take = [&](RunPos &p, Run *run) {  // the run at p; p moves behind it
        const Plan &pl = plans[p.r];
        next_run(pl, docs.data + pl.first_doc, p.doc, p.blk, run);
        ++p.run_no;
    };
    RunPos at = {0, 0, 0, 0};
    while (settle(at)) {
        uint32_t n_runs = 0, n_more = 0;
        for (RunPos p = at; settle(p);) {
            Run run;
            take(p, &run);
            if ((uint64_t)(K6Params::docs_behind(n_runs + 1u) + n_more + run.n_docs - 1u) > kAttendMaxDocs) break;
            ++n_runs;
            n_more += run.n_docs - 1u;
        }
        kq.n_runs = n_runs;
        kq.doc_first = K6Params::docs_behind(n_runs);
        uint32_t later = kq.doc_first;  // where the next run's further documents go
        for (uint32_t k = 0; k < n_runs; ++k) {
            settle(at);
            const Plan &pl = plans[at.r];
            const ha_rag_attend_request &rq = reqs[at.r];
            const uint32_t run_no = at.run_no;
            Run run;
            take(at, &run);
            const Doc &first = docs[pl.first_doc + run.doc];
            K6Run &d = kq.run[k];
            d.k = doc_k(first);
            d.v = doc_v(first);
            d.q = static_cast<const uint16_t *>(rq.q);
            d.part = pl.final ? rq.out : ws + pl.part_floats + (uint64_t)run_no * H * pl.n_mt * kAttendRecFloats;
            if (!pl.final && !record_fits(d.part, pl)) return HA_RAG_EINVAL;
            d.final = pl.final;
            d.lse = pl.final ? rq.lse : nullptr;
            d.n_tokens = first.n_tokens;
            d.info = first.info;
            d.n_q = rq.n_q;
            d.n_docs = run.n_docs;
            d.more = later;
            d.first_block = run.first_block;
            d.end_block = run.end_block;
            for (uint32_t i = 1; i < run.n_docs; ++i) {
                const Doc &doc = docs[pl.first_doc + run.doc + i];
                kq.doc[later++] = K6Doc{doc_k(doc), doc_v(doc), doc.n_tokens, doc.info};
            }
        }
        kq.doc_end = later;
        HIPCHK(c, launch_k6_shared(kq, form, st, dry));
    }

    K7Params mp;
    mp.n_kv_heads = H;
    mp.n_q_heads = n_q_heads;
    mp.n_reqs = mp.pad = 0;
    for (uint32_t r = 0; r < n_reqs; ++r) {
        if (plans[r].final) continue;  // written by the run's own workgroups
        K7Req &d = mp.r[mp.n_reqs++];
        d.part = ws + plans[r].part_floats;
        d.out = reqs[r].out;
        d.lse = reqs[r].lse;
        d.n_q = reqs[r].n_q;
        d.n_runs = plans[r].n_runs;
        d.pad[0] = d.pad[1] = 0;
        if (mp.n_reqs == kMaxMergeReqs) {
            HIPCHK(c, launch_k7(mp, st, dry));
            mp.n_reqs = 0;
        }
    }
    if (mp.n_reqs) HIPCHK(c, launch_k7(mp, st, dry));
    return HA_RAG_OK;
}

// ids -> descriptors of the copies the kernel can read in place (HBM, else pinned memory)
int resolve_ids(ha_rag_ctx *c, const uint64_t *ids, const ha_rag_attend_request *reqs,
                       uint32_t n_reqs, std::vector<ha_rag_packed_chunk> *out,
                       std::vector<uint32_t> *cis)
{
    if (!c || !reqs || n_reqs == 0 || n_reqs > HA_RAG_MAX_ATTEND_REQUESTS) return HA_RAG_EINVAL;
    uint64_t n = 0;
    for (uint32_t r = 0; r < n_reqs; ++r) n += reqs[r].n_chunks;
    if (n > HA_RAG_MAX_REQUEST_CHUNKS || (n && !ids)) return HA_RAG_EINVAL;
    out->resize((size_t)n);
    cis->resize((size_t)n);
    for (uint64_t i = 0; i < n; ++i) {
        uint32_t ci = 0;
        const Chunk *ch = find_chunk(c, ids[i], &ci);
        if (!ch) return HA_RAG_ENOENT;
        const int t = ch->fastest();
        if (t != (int)HA_RAG_TIER_HBM && t != (int)HA_RAG_TIER_PINNED) return HA_RAG_ENOENT;
        ha_rag_packed_chunk &pc = (*out)[(size_t)i];
        pc.packed = c->slab[t][ch->prec].ptr(ch->slot[t]);
        pc.n_tokens = ch->n_tokens;
        pc.prec = ch->prec;
        pc.group = c->group_of(ch->prec);
        pc.part = ch->part;
        (*cis)[(size_t)i] = ci;
    }
    return HA_RAG_OK;
}

// ---- scratch of ha_rag_attend_packed_static ------------------------------------------------
// The partial results of that entry point live in this array instead of a caller's workspace.
// Every GPU holds its own copy at its own address, from the moment the code object is loaded
// there until the process ends.  In host code the name is only a handle for
// hipGetSymbolAddress: what kernels and copies get is the address that call returned for the
// current device, kept in g_scratch_ptr.
constexpr size_t kStaticScratchBytes = (size_t)HA_RAG_ATTEND_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

}  // namespace

namespace ha_rag_host {

// Address of the scratch array on the current device; looked up once per device.
int attend_static_scratch(void **ptr, std::string *err)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        if (err) *err = std::string("hipGetDevice: ") + (e != hipSuccess ? hipGetErrorString(e) : "device index out of range");
        return HA_RAG_EHIP;
    }
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            if (err) *err = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
            return HA_RAG_EHIP;
        }
        g_scratch_ptr[dev] = p;
    }
    if (ptr) *ptr = g_scratch_ptr[dev];
    return HA_RAG_OK;
}

}  // namespace ha_rag_host

extern "C" {

int ha_rag_attend_workspace_bytes(ha_rag_ctx *c, const ha_rag_packed_chunk *chunks,
                                  const ha_rag_attend_request *reqs, uint32_t n_reqs,
                                  uint32_t n_q_heads, size_t *bytes)
{
    if (!bytes) return HA_RAG_EINVAL;
    HeapPlanStore hs(reqs, n_reqs);
    PlanStore ps = hs.store();
    uint64_t floats = 0;
    SharedForm form;
    int rc = plan_attend(c, chunks, reqs, n_reqs, n_q_heads, ps.plans, &ps.docs, ps.open_k, ps.open_v,
                         &floats, &form, false);
    if (rc) return rc;
    *bytes = (size_t)(floats * 4ull);
    return HA_RAG_OK;
}

int ha_rag_attend_packed(ha_rag_ctx *c, const ha_rag_packed_chunk *chunks,
                         const ha_rag_attend_request *reqs, uint32_t n_reqs, uint32_t layer,
                         uint32_t n_q_heads, float sm_scale, void *workspace, size_t workspace_bytes,
                         void *stream)
{
    if (!c) return HA_RAG_EINVAL;
    HeapPlanStore hs(reqs, n_reqs);
    std::lock_guard<std::mutex> g(c->mu);
    return attend_locked(c, hs.store(), chunks, reqs, n_reqs, layer, n_q_heads, sm_scale, workspace,
                         workspace_bytes, stream);
}

int ha_rag_attend_packed_static(ha_rag_ctx *c, const ha_rag_packed_chunk *chunks,
                                const ha_rag_attend_request *reqs, uint32_t n_reqs, uint32_t layer,
                                uint32_t n_q_heads, float sm_scale, void *stream)
{
    if (!c || !reqs || n_reqs == 0) return HA_RAG_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    if (n_reqs > HA_RAG_ATTEND_STATIC_MAX_REQUESTS) {
        c->err = "ha_rag_attend_packed_static: more than " +
                 std::to_string(HA_RAG_ATTEND_STATIC_MAX_REQUESTS) + " requests in one call";
        return HA_RAG_ENOSPC;
    }
    // the plan of the call on the stack: no list here grows
    Plan plans[HA_RAG_ATTEND_STATIC_MAX_REQUESTS];
    Doc docs[HA_RAG_ATTEND_STATIC_MAX_DOCS];
    uint32_t open_k[HA_RAG_ATTEND_STATIC_MAX_DOCS], open_v[HA_RAG_ATTEND_STATIC_MAX_DOCS];
    PlanStore ps{plans, Fixed<Doc>(docs, HA_RAG_ATTEND_STATIC_MAX_DOCS),
                 Fixed<uint32_t>(open_k, HA_RAG_ATTEND_STATIC_MAX_DOCS),
                 Fixed<uint32_t>(open_v, HA_RAG_ATTEND_STATIC_MAX_DOCS)};
    void *ws = nullptr;
    if (!c->dry()) {
        int rc = attend_static_scratch(&ws, &c->err);
        if (rc) return rc;
    } else {
        ws = reinterpret_cast<void *>((uintptr_t)256);  // never dereferenced
    }
    uint64_t need = 0;
    int rc = attend_locked(c, ps, chunks, reqs, n_reqs, layer, n_q_heads, sm_scale, ws,
                           kStaticScratchBytes, stream, false, &need);
    if (rc == HA_RAG_ENOSPC) {
        char msg[192];
        if (need > kStaticScratchBytes)
            std::snprintf(msg, sizeof msg,
                          "ha_rag_attend_packed_static: the call needs %llu bytes of partial results, the scratch array holds %llu",
                          (unsigned long long)need, (unsigned long long)kStaticScratchBytes);
        else
            std::snprintf(msg, sizeof msg,
                          "ha_rag_attend_packed_static: more than %u documents in one call",
                          (unsigned)HA_RAG_ATTEND_STATIC_MAX_DOCS);
        c->err = msg;
    }
    return rc;
}

int ha_rag_attend_chunks_workspace_bytes(ha_rag_ctx *c, const uint64_t *ids,
                                         const ha_rag_attend_request *reqs, uint32_t n_reqs,
                                         uint32_t n_q_heads, size_t *bytes)
{
    if (!c || !bytes) return HA_RAG_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    std::vector<ha_rag_packed_chunk> chunks;
    std::vector<uint32_t> cis;
    int rc = resolve_ids(c, ids, reqs, n_reqs, &chunks, &cis);
    if (rc) return rc;
    HeapPlanStore hs(reqs, n_reqs);
    PlanStore ps = hs.store();
    uint64_t floats = 0;
    SharedForm form;
    rc = plan_attend(c, chunks.data(), reqs, n_reqs, n_q_heads, ps.plans, &ps.docs, ps.open_k, ps.open_v,
                     &floats, &form, false);
    if (rc) return rc;
    *bytes = (size_t)(floats * 4ull);
    return HA_RAG_OK;
}

int ha_rag_attend_chunks(ha_rag_ctx *c, const uint64_t *ids, const ha_rag_attend_request *reqs,
                         uint32_t n_reqs, uint32_t layer, uint32_t n_q_heads, float sm_scale,
                         uint32_t flags, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!c || (flags & ~(uint32_t)HA_RAG_ATTEND_COUNT)) return HA_RAG_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    std::vector<ha_rag_packed_chunk> chunks;
    std::vector<uint32_t> cis;
    int rc = resolve_ids(c, ids, reqs, n_reqs, &chunks, &cis);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    // the kernels read the slots where they lie: wait for whoever wrote them on another stream
    bool in_host = false;
    for (size_t i = 0; i < cis.size(); ++i) {
        const Chunk &ch = c->chunks[cis[i]];
        const int t = ch.fastest();
        in_host |= t == (int)HA_RAG_TIER_PINNED;
        rc = before_read(c, c->slab[t][ch.prec].use[ch.slot[t]], s);
        if (rc) return rc;
    }
    HeapPlanStore hs(reqs, n_reqs);
    rc = attend_locked(c, hs.store(), chunks.data(), reqs, n_reqs, layer, n_q_heads, sm_scale, workspace,
                       workspace_bytes, stream, in_host);
    if (rc) return rc;
    if (flags & HA_RAG_ATTEND_COUNT) {  // Algorithm 1's access counts and the LRU order of Algorithm 2
        if (c->cfg.rerank_interval && c->n_loads && (c->n_loads % c->cfg.rerank_interval) == 0)
            rerank_locked(c);
        ++c->n_loads;
        for (uint32_t ci : cis) {
            Chunk &ch = c->chunks[ci];
            ch.count += 1;
            tier_touch(c, (uint32_t)ch.fastest(), ci);
        }
    }
    return mark_stream(c, s);  // a later writer of one of these slots waits for this point
}

}  // extern "C"
