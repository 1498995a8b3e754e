// What an attention call lays out in its workspace and launches, seen from the launches: this program takes the
// place of the kernels' launchers, so every descriptor the planning fills arrives here (dry_run contexts, no HIP call).
// For every call it checks that each record lies inside the workspace that was asked for (or the fixed array of the entry
// point without one), that no two records overlap, that the merge reads exactly what the runs write, and that the
// runs take every block of every document once.
//
//   plans_host random SEED CALLS   calls of any shape, many of more documents than one run may hold
//   plans_host calls               one call a line on stdin; prints a line each (see run_line)
//   plans_host share TILES TOKENS ..  tiles to a workgroup of every chunk of a GSE-8 class
//   plans_host pinned N            the same call of documents in HBM, and of which N lie in pinned memory, through each way to
//                                  list them; prints for each whether it reads past the last-level cache
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/ha_rag.h"
#include "../../paper_2510_20878_amd/csrc/ha_rag_kernels.h"

using namespace ha_rag;

namespace {

[[noreturn]] void fail(const char *what)
{
    std::fprintf(stderr, "plans_host: %s\n", what);
    std::exit(1);
}

// What the launches of the call in the making came to.  Requests are told apart by their output's address.
constexpr uintptr_t kWorkspace = 0x760000000000ull, kStaticWorkspace = 256, kOut = 0x10000000000ull, kOutStep = 0x1000000000ull;
struct Range {
    uint64_t at, end;  // bytes from the workspace's start
};
struct Seen {
    uintptr_t ws = 0;
    std::vector<Range> records;
    std::vector<Range> merged;
    std::vector<uint64_t> blocks;        // by request, told from the queries' address
    uint32_t form = 0, pieces = 0, runs = 0, longest = 0;
    uint64_t end = 0;                    // of the last record
    bool quiet = false;                  // only timed
    uint32_t doc_end = 0;                // of the launch with the most descriptors
    bool past = false;                   // k6_attend_partial reads past the last-level cache
} seen;

uint32_t request_of(const void *p) { return (uint32_t)(((uintptr_t)p - kOut) / kOutStep); }

void take_run(const K6Params &p, uint32_t i, bool shared)
{
    const K6Run &d = p.run[i];
    const uint32_t H = p.n_kv_heads, n_mt = (d.n_q * (p.n_q_heads / H) + 15u) / 16u;
    if (!shared && n_mt > 2u) fail("a request of more than two tiles in the kernel of two");
    uint64_t blocks = 0;
    for (uint32_t k = 0; k < d.n_docs; ++k) {
        const uint32_t T = k ? p.doc[d.more + k - 1u].n_tokens : d.n_tokens, nb = (T + 15u) / 16u;
        const uint32_t b0 = k ? 0u : d.first_block, b1 = k + 1u < d.n_docs ? nb : d.end_block;
        if (b0 >= b1 || b1 > nb) fail("a run's blocks do not lie in its documents");
        blocks += b1 - b0;
    }
    const uint32_t r = request_of(d.q);
    if (r >= seen.blocks.size()) fail("a run of no request");
    seen.blocks[r] += blocks;
    if (blocks > seen.longest) seen.longest = (uint32_t)blocks;
    if (d.final) {
        if (request_of(d.part) != r) fail("a final run does not write its request's output");
        return;
    }
    const uint64_t at = (uint64_t)((uintptr_t)d.part - seen.ws);
    seen.records.push_back(Range{at, at + (uint64_t)H * n_mt * kAttendRecFloats * 4u});
}

}  // namespace

namespace ha_rag {

hipError_t launch_k6(K6Params &p, hipStream_t, bool)
{
    if (seen.quiet) return hipSuccess;
    seen.pieces += p.n_runs;
    seen.past = p.past;
    seen.doc_end = std::max(seen.doc_end, p.doc_end);
    for (uint32_t i = 0; i < p.n_runs; ++i) take_run(p, i, false);
    return hipSuccess;
}

hipError_t launch_k6_shared(K6Params &p, SharedForm form, hipStream_t, bool)
{
    if (seen.quiet) return hipSuccess;
    const uint32_t id = 10u * scoring_waves(form) + (form >= SharedForm::kRoles4);  // 20, 40: k6_attend_shared; 41, 81: k6_attend_roles
    if (seen.form && seen.form != id) fail("two forms of the shared kernel in one call");
    seen.form = id;
    seen.runs += p.n_runs;
    seen.doc_end = std::max(seen.doc_end, p.doc_end);
    for (uint32_t i = 0; i < p.n_runs; ++i) take_run(p, i, true);
    return hipSuccess;
}

hipError_t launch_k7(K7Params &p, hipStream_t, bool)
{
    if (seen.quiet) return hipSuccess;
    for (uint32_t i = 0; i < p.n_reqs; ++i) {
        const K7Req &d = p.r[i];
        const uint64_t n_mt = (d.n_q * (p.n_q_heads / p.n_kv_heads) + 15u) / 16u, at = (uint64_t)((uintptr_t)d.part - seen.ws);
        seen.merged.push_back(Range{at, at + (uint64_t)d.n_runs * p.n_kv_heads * n_mt * kAttendRecFloats * 4u});
    }
    return hipSuccess;
}

// the other launchers that the host runtime refers to
hipError_t launch_k1(K1Params &, const K1Launch &, hipStream_t) { fail("a load"); }
hipError_t launch_k2(const K2Params &, uint32_t, uint32_t, hipStream_t) { fail("a pack"); }
hipError_t launch_k8(const void *, const void *, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, double *, hipStream_t) { fail("an error sum"); }
hipError_t check_k6_args(const K6Params &, uint32_t *, bool *) { return hipSuccess; }
hipError_t prepare_k6_shared() { return hipSuccess; }

}  // namespace ha_rag

namespace {

struct Call {
    uint32_t H, n_q_heads, layers = 2;
    uint64_t apart = 0;  // bytes between chunks
    std::vector<ha_rag_attend_request> reqs;
    std::vector<ha_rag_packed_chunk> chunks;
    void request(uint32_t n_q)
    {
        ha_rag_attend_request rq;
        std::memset(&rq, 0, sizeof rq);
        const uintptr_t base = kOut + reqs.size() * kOutStep;
        rq.q = (const void *)base;
        rq.out = (float *)base;
        rq.n_q = n_q;
        reqs.push_back(rq);
    }
    // back: each is the chunk listed so many before it
    void documents(uint32_t n_tokens, uint32_t count, uint32_t prec = HA_RAG_PREC_INT4, uint32_t back = 0, uint32_t part = HA_RAG_PART_KV)
    {
        ha_rag_packed_chunk pc;
        std::memset(&pc, 0, sizeof pc);
        pc.n_tokens = n_tokens;
        pc.prec = prec;
        pc.group = prec == HA_RAG_PREC_INT8 || prec == HA_RAG_PREC_INT4 ? 128 : 0;
        pc.part = part;
        for (uint32_t i = 0; i < count; ++i) {
            const size_t n = chunks.size();
            if (back > n) fail("a document listed before the first");
            pc.packed = back ? chunks[n - back].packed : (const void *)(0x750000000000ull + apart * n);
            chunks.push_back(pc);
        }
        reqs.back().n_chunks += count;
    }
};

ha_rag_ctx *context(uint32_t H, uint32_t layers = 2)
{
    static ha_rag_ctx *all[65][257] = {};
    if (H == 0 || H > 256 || layers > 64) fail("heads or layers");
    ha_rag_ctx **ctx = all[layers];
    if (!ctx[H]) {
        ha_rag_config cfg;
        std::memset(&cfg, 0, sizeof cfg);
        cfg.n_layers = layers;
        cfg.n_kv_heads = H;
        cfg.head_dim = 128;
        cfg.max_chunk_tokens = 4096;
        cfg.group_int8 = cfg.group_int4 = 128;
        cfg.dry_run = 1;
        if (ha_rag_create(&cfg, &ctx[H]) != HA_RAG_OK) fail("ha_rag_create");
    }
    return ctx[H];
}

// One call through an entry point; everything it launched is checked against `bytes` of workspace.
int attend(Call &c, bool fixed, size_t bytes)
{
    seen = Seen();
    seen.ws = fixed ? kStaticWorkspace : kWorkspace;
    seen.blocks.assign(c.reqs.size(), 0);
    ha_rag_ctx *ctx = context(c.H, c.layers);
    const uint32_t n = (uint32_t)c.reqs.size();
    const int rc = fixed ? ha_rag_attend_packed_static(ctx, c.chunks.data(), c.reqs.data(), n, 0, c.n_q_heads, 0.1f, nullptr)
                         : ha_rag_attend_packed(ctx, c.chunks.data(), c.reqs.data(), n, 0, c.n_q_heads, 0.1f, (void *)kWorkspace, bytes, nullptr);
    if (rc != HA_RAG_OK) {
        if (!seen.records.empty() || !seen.merged.empty()) fail("a refused call launched something");
        return rc;
    }
    size_t at = 0;
    for (uint32_t r = 0; r < n; ++r) {
        uint64_t blocks = 0;
        for (uint32_t i = 0; i < c.reqs[r].n_chunks; ++i, ++at)
            if (c.chunks[at].part != HA_RAG_PART_V) blocks += (c.chunks[at].n_tokens + 15u) / 16u;
        if (blocks != seen.blocks[r]) fail("a request's runs do not take its blocks once");
    }
    auto by_start = [](const Range &a, const Range &b) { return a.at < b.at || (a.at == b.at && a.end < b.end); };
    std::sort(seen.records.begin(), seen.records.end(), by_start);
    std::sort(seen.merged.begin(), seen.merged.end(), by_start);
    std::vector<Range> join;  // the records, with those that touch put together per merged range
    for (const Range &r : seen.records) {
        if (r.end > seen.end) seen.end = r.end;
        if (r.end > bytes) {
            std::fprintf(stderr, "record ends at byte %llu of %llu\n", (unsigned long long)r.end, (unsigned long long)bytes);
            fail("a record lies outside the workspace");
        }
    }
    size_t next = 0;
    for (const Range &m : seen.merged) {
        uint64_t to = m.at;
        while (to < m.end) {
            if (next == seen.records.size() || seen.records[next].at != to) fail("the merge reads what no run writes, or records overlap");
            to = seen.records[next++].end;
        }
        if (to != m.end) fail("a record beyond what the merge reads");
    }
    if (next != seen.records.size()) fail("a record that no merge reads");
    return rc;
}

uint64_t rng_state;
uint64_t rnd(uint64_t n)
{
    rng_state ^= rng_state << 13;
    rng_state ^= rng_state >> 7;
    rng_state ^= rng_state << 17;
    return rng_state % n;
}
uint32_t any_size(uint32_t most)  // spread over its logarithm
{
    uint32_t bits = 0;
    while ((2u << bits) <= most) ++bits;
    const uint32_t b = (uint32_t)rnd(bits + 1u);
    return std::min(most, (1u << b) + (uint32_t)rnd(1u << b));
}

void random_call(Call &c)
{
    const uint32_t heads[] = {1, 2, 8, 8, 16, 150}, per[] = {1, 4, 4, 8}, queries[] = {9, 20, 64, 300};
    c = Call();
    c.H = heads[rnd(6)];
    c.n_q_heads = c.H * per[rnd(4)];
    const uint32_t n_reqs = any_size(24), most_q = queries[rnd(4)], long_lists = (uint32_t)rnd(3);
    for (uint32_t r = 0; r < n_reqs; ++r) {
        c.request(rnd(3) ? any_size(most_q) : most_q);
        const uint32_t groups = 1 + (uint32_t)rnd(3);  // documents of one length in a row
        for (uint32_t g = 0; g < groups; ++g) {
            uint32_t count = long_lists ? any_size(400) : any_size(12);
            const uint32_t room = HA_RAG_MAX_REQUEST_CHUNKS - (uint32_t)c.chunks.size();
            c.documents(any_size(rnd(2) ? 64 : 4000), std::min(count, room), (uint32_t)rnd(HA_RAG_N_PREC));
        }
    }
}

// One call: "static|workspace|ends|time N|past LAYERS APART HEADS QUERY_HEADS" then per request "/ n_q tokens*count*format*back*part ..."
// (APART: bytes between chunks; back: see documents()).  Prints the return
// code, the workspace asked for, the end of the last record, the shared kernel's form (0: not
// launched), pieces and runs launched and the blocks of the longest; or the us of a call; or whether it reads past the cache, and the pieces
// launched; or the end of the descriptors of the launch that has the most.
void run_line(char *line)
{
    Call c = Call();
    char *save = nullptr;
    char *w = strtok_r(line, " \n", &save);
    if (!w) return;
    const std::string how = w;
    const int times = how == "time" ? std::atoi(strtok_r(nullptr, " \n", &save)) : 0;
    if (how == "past") {
        c.layers = (uint32_t)std::atoi(strtok_r(nullptr, " \n", &save));
        c.apart = std::strtoull(strtok_r(nullptr, " \n", &save), nullptr, 10);
    }
    c.H = (uint32_t)std::atoi(strtok_r(nullptr, " \n", &save));
    c.n_q_heads = (uint32_t)std::atoi(strtok_r(nullptr, " \n", &save));
    bool first = false;
    while ((w = strtok_r(nullptr, " \n", &save))) {
        if (!std::strcmp(w, "/")) {
            first = true;
            continue;
        }
        if (first) c.request((uint32_t)std::atoi(w));
        else {
            unsigned tokens = 0, count = 1, prec = HA_RAG_PREC_INT4, back = 0, part = HA_RAG_PART_KV;
            if (std::sscanf(w, "%u*%u*%u*%u*%u", &tokens, &count, &prec, &back, &part) < 1) fail("a call's line");
            c.documents(tokens, count, prec, back, part);
        }
        first = false;
    }
    ha_rag_ctx *ctx = context(c.H, c.layers);
    size_t need = 0;
    const uint32_t n = (uint32_t)c.reqs.size();
    int rc = ha_rag_attend_workspace_bytes(ctx, c.chunks.data(), c.reqs.data(), n, c.n_q_heads, &need);
    if (times) {
        double best = 1e30;
        for (int k = 0; k < 7; ++k) {
            seen.quiet = true;
            const auto a = std::chrono::steady_clock::now();
            for (int i = 0; i < times; ++i)
                rc |= ha_rag_attend_packed(ctx, c.chunks.data(), c.reqs.data(), n, 0, c.n_q_heads, 0.1f, (void *)kWorkspace, need, nullptr);
            const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - a).count() / times;
            if (us < best) best = us;
        }
        seen.quiet = false;
        std::printf("%d %.2f\n", rc, best);
        return;
    }
    if (rc == HA_RAG_OK) rc = attend(c, how == "static", how == "static" ? HA_RAG_ATTEND_STATIC_SCRATCH_BYTES : need);
    if (how == "ends") {
        std::printf("%d %u\n", rc, seen.doc_end);
        return;
    }
    if (how == "past") {
        std::printf("%d %d %u\n", rc, (int)seen.past, seen.pieces);
        return;
    }
    std::printf("%d %zu %llu %u %u %u %u\n", rc, need, (unsigned long long)(rc ? 0 : seen.end), rc ? 0 : seen.form, rc ? 0 : seen.pieces, rc ? 0 : seen.runs, rc ? 0 : seen.longest);
}

// 32 requests of ten documents of 512 tokens, two layers, n_pinned of the documents in pinned memory: in the pool's slab there,
// by id and by address, and at addresses of the caller's, by id.
void pinned_calls(uint32_t n_pinned)
{
    constexpr uint32_t kDocs = 320, kTokens = 512, kPrec = HA_RAG_PREC_FP8_E4M3;
    for (const bool external : {false, true}) {
        ha_rag_config cfg;
        std::memset(&cfg, 0, sizeof cfg);
        cfg.n_layers = 2;
        cfg.n_kv_heads = 8;
        cfg.head_dim = 128;
        cfg.max_chunk_tokens = kTokens;
        cfg.group_int8 = cfg.group_int4 = 128;
        cfg.dry_run = 1;
        ha_rag_ctx *ctx = nullptr;
        if (ha_rag_create(&cfg, &ctx) != HA_RAG_OK) fail("ha_rag_create");
        const size_t slot = 2ull * 2 * 8 * kTokens * 128;
        const uintptr_t hbm = 0x750000000000ull, pinned = 0x740000000000ull;
        if (ha_rag_register_slab(ctx, HA_RAG_TIER_HBM, kPrec, (void *)hbm, slot * kDocs) != HA_RAG_OK) fail("the HBM slab");
        if (external ? ha_rag_register_external(ctx, kPrec) : ha_rag_register_slab(ctx, HA_RAG_TIER_PINNED, kPrec, (void *)pinned, slot * kDocs))
            fail("the pinned slab");
        Call c;
        c.H = 8;
        c.n_q_heads = 32;
        std::vector<uint64_t> ids;
        for (uint32_t i = 0; i < kDocs; ++i) {
            const bool there = i >= kDocs - n_pinned;
            if (there && external ? ha_rag_pool_insert_external(ctx, i, HA_RAG_PART_KV, kPrec, kTokens, (const void *)(pinned + slot * i))
                                  : ha_rag_pool_insert(ctx, i, kPrec, kTokens, nullptr, 0, there ? HA_RAG_TIER_PINNED : HA_RAG_TIER_HBM, nullptr))
                fail("a chunk of the pool");
            void *at = nullptr;
            size_t bytes = 0;
            if (ha_rag_pool_slot(ctx, i, there ? HA_RAG_TIER_PINNED : HA_RAG_TIER_HBM, &at, &bytes) != HA_RAG_OK) fail("a chunk's place");
            if (i % 10u == 0) c.request(1);
            c.documents(kTokens, 1, kPrec);
            c.chunks.back().packed = at;
            ids.push_back(i);
        }
        const uint32_t n = (uint32_t)c.reqs.size();
        size_t need = 0;
        if (ha_rag_attend_workspace_bytes(ctx, c.chunks.data(), c.reqs.data(), n, c.n_q_heads, &need) != HA_RAG_OK) fail("the size of a well-formed call");
        for (const bool by_id : {true, false}) {
            seen = Seen();
            seen.ws = kWorkspace;
            seen.blocks.assign(n, 0);
            if (by_id ? ha_rag_attend_chunks(ctx, ids.data(), c.reqs.data(), n, 0, c.n_q_heads, 0.1f, 0, (void *)kWorkspace, need, nullptr)
                      : ha_rag_attend_packed(ctx, c.chunks.data(), c.reqs.data(), n, 0, c.n_q_heads, 0.1f, (void *)kWorkspace, need, nullptr))
                fail("a well-formed call");
            if (by_id || !external) std::printf("%d ", (int)seen.past);
        }
        ha_rag_destroy(ctx);
    }
    std::printf("\n");
}

void share(uint32_t n_tiles, char **tokens, uint32_t n)
{
    K2Params p{};
    p.n_tiles = n_tiles;
    p.head_dim = 128;
    if (n > kMaxK2Chunks) fail("chunks");
    uint32_t max_blk = 1;
    for (uint32_t i = 0; i < n; ++i) {
        p.c[p.n_chunks++].n_tokens = (uint32_t)std::atoi(tokens[i]);
        max_blk = std::max(max_blk, (p.c[i].n_tokens + 15u) / 16u);
    }
    share_gse8_tiles(p);
    const uint32_t wg = gse8_wg_waves(max_blk), held = gse8_held(max_blk);
    for (uint32_t i = 0; i < n; ++i) {
        const uint32_t per_wg = p.c[i].share & 0xFFu, waves = (p.c[i].share >> 8) & 0xFFu, mul = p.c[i].share >> 16;
        if (!per_wg || !waves || per_wg * waves > wg) fail("waves that a workgroup does not have");
        if (held && held * waves < (p.c[i].n_tokens + 15u) / 16u) fail("a tile's waves do not hold its blocks");
        for (uint32_t w = 0; w < wg; ++w)
            if ((w * mul) >> 8 != w / waves) fail("a wave's tile");
        std::printf("%u ", per_wg);
    }
    std::printf("\n");
}

}  // namespace

int main(int argc, char **argv)
{
    if (argc == 4 && !std::strcmp(argv[1], "random")) {
        rng_state = 0x9E3779B97F4A7C15ull ^ (std::strtoull(argv[2], nullptr, 10) * 0x100000001B3ull);
        const int calls = std::atoi(argv[3]);
        Call c;
        int fit = 0, many = 0;
        for (int i = 0; i < calls; ++i) {
            random_call(c);
            size_t need = 0;
            const uint32_t n = (uint32_t)c.reqs.size();
            if (ha_rag_attend_workspace_bytes(context(c.H), c.chunks.data(), c.reqs.data(), n, c.n_q_heads, &need) != HA_RAG_OK) fail("the size of a well-formed call");
            if (attend(c, false, need) != HA_RAG_OK) fail("a well-formed call");
            const int rc = attend(c, true, HA_RAG_ATTEND_STATIC_SCRATCH_BYTES);
            if (rc != HA_RAG_OK && rc != HA_RAG_ENOSPC) fail("a well-formed call without a workspace");
            fit += rc == HA_RAG_OK;
            for (const ha_rag_attend_request &rq : c.reqs) many += rq.n_chunks > 128;
        }
        std::printf("plans_host ok: %d calls, %d fit the fixed array, %d requests of more than 128 documents\n", calls, fit, many);
        return 0;
    }
    if (argc == 2 && !std::strcmp(argv[1], "calls")) {
        std::vector<char> line(1 << 20);
        while (std::fgets(line.data(), (int)line.size(), stdin)) run_line(line.data());
        return 0;
    }
    if (argc > 3 && !std::strcmp(argv[1], "share")) {
        share((uint32_t)std::atoi(argv[2]), argv + 3, (uint32_t)argc - 3u);
        return 0;
    }
    if (argc == 3 && !std::strcmp(argv[1], "pinned")) {
        for (const int n : {0, std::atoi(argv[2])}) pinned_calls((uint32_t)n);
        return 0;
    }
    fail("usage: plans_host random SEED CALLS | plans_host calls | plans_host pinned N | plans_host share TILES TOKENS ..");
}
