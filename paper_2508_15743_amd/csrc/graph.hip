// Offline stage (paper Sec. III.D.1): validate the detector error model, derive
// the channel LLRs, build the member schedules and upload everything once.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <queue>
#include <thread>

#include "internal.h"

namespace vibe {

static thread_local std::string g_last_error;

void set_error(const std::string& msg) { g_last_error = msg; }

int fail(int code, const std::string& msg) {
    set_error(msg);
    return code;
}

int hip_fail(hipError_t e, const char* what) {
    return fail(VIBE_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

namespace {

template <class T>
int upload(GraphHost& h, const T* src, size_t count, const T** dst) {
    if (count == 0) count = 1;  // keep every pointer valid
    void* p = nullptr;
    hipError_t e = hipMalloc(&p, sizeof(T) * count);
    if (e != hipSuccess) return fail(VIBE_ENOMEM, "hipMalloc of graph data failed");
    h.allocations.push_back(p);
    h.device_bytes += sizeof(T) * count;
    if (src) {
        e = hipMemcpy(p, src, sizeof(T) * count, hipMemcpyHostToDevice);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpy of graph data");
    }
    *dst = static_cast<const T*>(p);
    return VIBE_OK;
}

// One member's schedule: its chunk records, and its part of the compact item
// body's data.
struct MemberSched {
    std::vector<unsigned char> recs;
    std::vector<uint32_t> csched, crec0, row0, row2;
    uint32_t levels = 0, chunks = 0, groups = 0, dense0 = 0;
    uint64_t kept = 0;  // chunks whose records are expected to fit
    bool whole = true;  // every column is placed
};

// What building one needs besides, reused from member to member.  Per chunk
// slot (64 a chunk): the meta word, the column, its channel LLR and the
// initial suffix state.
struct SchedScratch {
    std::vector<uint32_t> meta, v, init32;
    std::vector<float> lam32;
    std::vector<double> lam64;
    std::vector<uint64_t> init64;
    std::vector<uint32_t> last, level, height, npred, pos, succ, taken, running32, later;
    std::vector<uint64_t> skipped, running64;
    std::vector<float> expected;
};

// fn(i, scratch) for i < count, in any order, on up to eight threads where
// `work` (edges x members) is worth starting them, which takes 0.15 ms: 2^13
// take 1 to 4 ms on one.
// Returns false if memory ran out.
template <class Scratch, class F>
bool for_members(uint32_t count, uint64_t work, F&& fn) {
    std::atomic<uint32_t> next{0};
    std::atomic<bool> ok{true};
    auto run = [&]() {
        try {
            Scratch scratch;
            for (uint32_t i; ok && (i = next.fetch_add(1)) < count;) fn(i, scratch);
        } catch (...) {
            ok = false;
        }
    };
    std::vector<std::thread> helpers;
    uint32_t n = work < (1u << 13) ? 1u : std::min(8u, std::max(1u, std::thread::hardware_concurrency()));
    n = std::min(n, count);
    try {
        while (helpers.size() + 1 < n) helpers.emplace_back(run);
    } catch (...) {  // as many as could be started
    }
    run();
    for (std::thread& t : helpers) t.join();
    return ok;
}

void free_all(GraphHost& h) {
    for (void* p : h.allocations) (void)hipFree(p);
    h.allocations.clear();
}

}  // namespace

// Decode schedules for P = 2 or 4 shots per wavefront.  The 64-edge chunks
// are recut into chunks of at most W = 64 / P edges, columns kept whole and
// in slot order; a subset of an independent set of columns is independent,
// so the sweep computes the same messages.  Two edges of one row lie in
// different 64-edge chunks, whose order the recut keeps, so the suffix
// state of every slot for the initial messages (the row's later edges) is
// the one of the 64-edge schedule and is copied over.  Each recut chunk
// carries its own largest column degree.
int build_multi_schedule(vibe_graph* G, uint32_t P) {
    if (P != 2 && P != 4) return fail(VIBE_EINVAL, "shots per wavefront must be 1, 2 or 4");
    const uint32_t idx = P / 4;
    if (G->multi_recs[idx]) return VIBE_OK;
    const DevGraph& d = G->h.dg;
    if (d.layered) return fail(VIBE_EUNSUPPORTED, "the layered schedule runs one shot per wavefront");
    const bool f64 = d.fp64 != 0;
    const uint32_t W = kWave / P, L = d.L, mb = f64 ? 8u : 4u;
    std::vector<uint32_t> mc(L + 1);
    hipError_t e = hipMemcpy(mc.data(), d.member_chunk, 4ull * (L + 1), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpy(member_chunk)");
    const size_t nrec = mc[L];
    const uint32_t rb = rec_bytes(f64), ri0 = rec_init(f64), wrb = rec_bytes_w(f64, W);
    std::vector<unsigned char> recs(std::max<size_t>(nrec, 1) * rb);
    if (nrec && (e = hipMemcpy(recs.data(), d.sched, nrec * rb, hipMemcpyDeviceToHost)) != hipSuccess)
        return hip_fail(e, "hipMemcpy(schedule)");
    std::vector<unsigned char> out;
    std::vector<uint32_t> gmc(L + 1, 0);
    std::vector<std::pair<uint32_t, uint32_t>> cols;  // (first slot, degree)
    uint32_t maxc = 0;
    for (uint32_t i = 0; i < L; i++) {
        gmc[i] = (uint32_t)(out.size() / wrb);
        for (size_t k = mc[i]; k < mc[i + 1]; k++) {
            const unsigned char* r = recs.data() + k * rb;
            uint32_t meta[kWave], vv[kWave];
            std::memcpy(meta, r, sizeof(meta));
            std::memcpy(vv, r + kRecV, sizeof(vv));
            cols.clear();
            for (uint32_t q = 0; q < (uint32_t)kWave;) {
                const uint32_t deg = (meta[q] >> kMetaDegShift) & 15u;
                if (!deg) break;
                cols.push_back({q, deg});
                q += deg;
            }
            size_t a = 0;
            while (a < cols.size()) {
                size_t b = a;
                uint32_t fill = 0, dmax = 0;
                while (b < cols.size() && fill + cols[b].second <= W) {
                    fill += cols[b].second;
                    dmax = std::max(dmax, cols[b].second);
                    b++;
                }
                const size_t at = out.size();
                out.resize(at + wrb, 0);
                unsigned char* o = out.data() + at;
                uint32_t slot = 0;
                auto put = [&](uint32_t mw, uint32_t v, const unsigned char* lam, const void* init) {
                    std::memcpy(o + 4 * slot, &mw, 4);
                    std::memcpy(o + 4 * W + 4 * slot, &v, 4);
                    if (lam) std::memcpy(o + 8 * W + mb * slot, lam, mb);
                    std::memcpy(o + 8 * W + mb * W + mb * slot, init, mb);
                    slot++;
                };
                for (size_t cc = a; cc < b; cc++)
                    for (uint32_t j = 0; j < cols[cc].second; j++) {
                        const uint32_t q = cols[cc].first + j;
                        put((meta[q] & ~(15u << kMetaDmaxShift)) | (dmax << kMetaDmaxShift), vv[q],
                            r + kRecLam + mb * q, r + ri0 + mb * q);
                    }
                while (slot < W)  // unused slots: c = v = 0, lambda 0, no message
                    put(dmax << kMetaDmaxShift, 0u, nullptr, f64 ? (const void*)&d.ident64 : (const void*)&d.ident32);
                a = b;
            }
        }
        maxc = std::max(maxc, (uint32_t)(out.size() / wrb) - gmc[i]);
    }
    gmc[L] = (uint32_t)(out.size() / wrb);
    if (out.empty()) {  // no edges: one unused record
        out.assign(wrb, 0);
        for (uint32_t q = 0; q < W; q++)
            std::memcpy(out.data() + 8 * W + mb * W + mb * q, f64 ? (const void*)&d.ident64 : (const void*)&d.ident32, mb);
    }
    const unsigned char* dr = nullptr;
    const uint32_t* dm = nullptr;
    int rc;
    if ((rc = upload(G->h, out.data(), out.size(), &dr)) || (rc = upload(G->h, gmc.data(), gmc.size(), &dm)))
        return rc;
    G->multi_recs[idx] = dr;
    G->multi_member_chunk[idx] = dm;
    G->multi_max_chunks[idx] = maxc;
    return VIBE_OK;
}

DevGraph compact_view(DevGraph d) {
    d.compact = 0;
    if (d.layered) {
        if (d.lcols) d.compact = d.ccols;
    } else if (d.csched && d.P == 1) {
        d.compact = d.ccols;
        d.dec_global = 0;  // its decisions are masks in global memory in any case
    }
    return d;
}

// The compact bodies keep two or four words per check in LDS, the general one
// one, so on graphs of thousands of checks fewer of them reside.  One runs an
// item in about 0.62 of the other's time where few reside, and neither gains
// from more than 16 wavefronts per CU.  Rows of 2.5 edges, m = n = 3000, 8
// members (general: 13 wavefronts per CU), parallel schedule (3): 40 shots
// 0.11 ms against 0.19, 600 0.48 against 0.42, 3000 1.96 against 1.19; one
// member, 3000 shots (four times what resides) 0.36 against 0.41; serial (6):
// 40 shots 0.12 against 0.18, 600 0.34 against 0.34, 3000 1.15 against 1.01.
DevGraph compact_choice(const DevGraph& d, uint64_t items) {
    const DevGraph c = compact_view(d);
    if (!c.compact || c.layered) return c;
    const int resident = bp_grid(c, false);
    if (items <= 4ull * resident) return c;
    DevGraph a = d;
    a.dec_global = dec_global_pays(d) ? 1 : 0;
    const int enough = bp_grid_for(false, c.flood != 0, false, 0, false, false, 1, false, false, c.compact);
    return resident >= 0.6 * std::min(bp_grid(a, false), enough) ? c : d;
}

DevGraph decode_view(const vibe_graph* G, bool allow_multi, uint64_t shots, bool allow_compact) {
    DevGraph d = G->h.dg;
    const uint32_t P = G->tune_P;
    if (allow_multi && (P == 2 || P == 4) && G->multi_recs[P / 4]) {
        d.sched = G->multi_recs[P / 4];
        d.member_chunk = G->multi_member_chunk[P / 4];
        d.max_chunks = G->multi_max_chunks[P / 4];
        d.P = P;
    }
    if (allow_compact) d = compact_choice(d, shots == UINT64_MAX ? shots : bp_items(d, shots));
    if (!d.layered && !d.compact) {
        if (G->tune_dec >= 0) {
            d.dec_global = G->tune_dec;
        } else {
            // automatic: only a launch with more items than fit at once with
            // the decisions in LDS gains from more residency (a small batch
            // is bound by its chains, which the global masks lengthen)
            d.dec_global = 0;
            const uint64_t items = shots == UINT64_MAX ? UINT64_MAX : bp_items(d, shots);
            if (items > (uint64_t)bp_grid(d, false) && dec_global_pays(d)) d.dec_global = 1;
        }
    }
    return d;
}

}  // namespace vibe

using namespace vibe;

extern "C" const char* vibe_last_error(void) { return g_last_error.c_str(); }

extern "C" const char* vibe_version(void) { return "vibelsd-gfx950 0.1.0"; }

extern "C" int vibe_graph_create(uint32_t m, uint32_t n, const uint32_t* h_indptr,
                                 const uint32_t* h_indices, const double* priors, uint32_t k,
                                 const uint32_t* l_indptr, const uint32_t* l_indices,
                                 const uint32_t* perms, const vibe_config* cfg, vibe_graph** out) {
    set_error("");
    if (!out) return fail(VIBE_EINVAL, "out is NULL");
    *out = nullptr;
    if (!h_indptr || !priors || !perms || !cfg || (k && !l_indptr))
        return fail(VIBE_EINVAL, "a required pointer is NULL");
    if (n == 0) return fail(VIBE_EINVAL, "n must be >= 1");
    if (m >= 65536u) return fail(VIBE_EUNSUPPORTED, "m must be < 65536");
    if (n >= (1u << 24)) return fail(VIBE_EUNSUPPORTED, "n must be < 2^24");
    const vibe_config c = *cfg;
    if (c.L < 1 || c.L > (uint32_t)kMaxL) return fail(VIBE_EINVAL, "L must be in 1..64");
    if (c.M < 1 || c.M > c.L) return fail(VIBE_EINVAL, "M must be in 1..L");
    if (c.T_max < 1 || c.T_max > (uint32_t)kMaxT) return fail(VIBE_EINVAL, "T_max must be in 1..64");
    if (c.lsd_order > kMaxLsdOrder) return fail(VIBE_EINVAL, "lsd_order must be in 0..64");
    if (!(c.alpha > 0.0) || !(c.alpha <= 1e6)) return fail(VIBE_EINVAL, "alpha must be in (0, 1e6]");
    if (!(c.clamp >= 1.0) || !(c.clamp <= 1e30)) return fail(VIBE_EINVAL, "clamp must be in [1, 1e30]");
    if (c.message_bits != 0 && c.message_bits != 32 && c.message_bits != 64)
        return fail(VIBE_EINVAL, "message_bits must be 0, 32 or 64");
    if (c.schedule > 2) return fail(VIBE_EINVAL, "schedule must be 0 (serial), 1 (parallel) or 2 (layered)");
    const bool layered = c.schedule == 2;
    if (m && (size_t)m * (c.message_bits == 64 ? 8 : 4) + 8 * (2 * (size_t)((m + 63) / 64) + (n + 63) / 64) >
                 150 * 1024)
        return fail(VIBE_EUNSUPPORTED, "per-decoder LDS state exceeds 150 KB");

    // ---- H in CSR: validate
    if (h_indptr[0] != 0) return fail(VIBE_EINVAL, "h_indptr[0] must be 0");
    for (uint32_t r = 0; r < m; r++)
        if (h_indptr[r + 1] < h_indptr[r]) return fail(VIBE_EINVAL, "h_indptr must be non-decreasing");
    const uint64_t E = h_indptr[m];
    if (E >= (1ull << 31)) return fail(VIBE_EUNSUPPORTED, "nnz must be < 2^31");
    if (E && !h_indices) return fail(VIBE_EINVAL, "h_indices is NULL");
    uint32_t max_row = 0;
    for (uint32_t r = 0; r < m; r++) {
        uint32_t lo = h_indptr[r], hi = h_indptr[r + 1];
        if (hi - lo >= 65536u) return fail(VIBE_EUNSUPPORTED, "a row has >= 65536 entries");
        max_row = std::max(max_row, hi - lo);
        for (uint32_t a = lo; a < hi; a++) {
            if (h_indices[a] >= n) return fail(VIBE_EINVAL, "a column index is >= n");
            if (a > lo && h_indices[a] <= h_indices[a - 1])
                return fail(VIBE_EINVAL, "column indices must be strictly ascending in each row");
        }
    }
    for (uint32_t v = 0; v < n; v++)
        if (!(priors[v] > 0.0 && priors[v] < 1.0))
            return fail(VIBE_EINVAL, "every prior must lie strictly between 0 and 1");
    if (k) {
        if (l_indptr[0] != 0) return fail(VIBE_EINVAL, "l_indptr[0] must be 0");
        for (uint32_t r = 0; r < k; r++) {
            if (l_indptr[r + 1] < l_indptr[r]) return fail(VIBE_EINVAL, "l_indptr must be non-decreasing");
            for (uint32_t a = l_indptr[r]; a < l_indptr[r + 1]; a++)
                if (!l_indices || l_indices[a] >= n) return fail(VIBE_EINVAL, "bad observable column");
        }
    }
    // ---- permutations: of the n columns, or of the m checks (layered)
    {
        const uint32_t len = layered ? m : n;
        std::vector<uint8_t> seen(len);
        for (uint32_t i = 0; i < c.L; i++) {
            std::fill(seen.begin(), seen.end(), 0);
            for (uint32_t a = 0; a < len; a++) {
                uint32_t v = perms[(size_t)i * len + a];
                if (v >= len || seen[v])
                    return fail(VIBE_EINVAL, layered ? "perms rows must be permutations of 0..m-1 (layered)"
                                                     : "perms rows must be permutations of 0..n-1");
                seen[v] = 1;
            }
        }
    }

    // ---- CSC with the CSR position of every edge
    std::vector<uint32_t> cp(n + 1, 0), ci(E), ce(E);
    for (uint64_t a = 0; a < E; a++) cp[h_indices[a] + 1]++;
    for (uint32_t v = 0; v < n; v++) cp[v + 1] += cp[v];
    {
        std::vector<uint32_t> fill(cp.begin(), cp.end() - 1);
        for (uint32_t r = 0; r < m; r++)
            for (uint32_t a = h_indptr[r]; a < h_indptr[r + 1]; a++) {
                uint32_t v = h_indices[a];
                ci[fill[v]] = r;  // rows visited ascending -> checks ascending per column
                ce[fill[v]] = a;
                fill[v]++;
            }
    }
    uint32_t max_col = 0;
    for (uint32_t v = 0; v < n; v++) max_col = std::max(max_col, cp[v + 1] - cp[v]);
    if (max_col > (uint32_t)kMaxColDeg) return fail(VIBE_EUNSUPPORTED, "a column is in more than 15 checks");

    // ---- channel LLRs, in FP64 with the C library's log
    const double lim = c.clamp;
    const bool fp64 = c.message_bits == 64;
    std::vector<double> lam64(n);
    std::vector<float> lam32(n);
    int all_pos = 1;
    for (uint32_t v = 0; v < n; v++) {
        double l = std::log((1.0 - priors[v]) / priors[v]);
        l = std::min(std::max(l, -lim), lim);
        lam64[v] = l;
        lam32[v] = (float)l;
        if (!(fp64 ? l > 0.0 : lam32[v] > 0.0f)) all_pos = 0;
    }
    const uint32_t words_n = (n + 63) / 64, words_m = (m + 63) / 64;
    std::vector<uint64_t> e0(words_n, 0);
    for (uint32_t v = 0; v < n; v++)
        if (cp[v + 1] == cp[v] && !(fp64 ? lam64[v] > 0.0 : lam32[v] > 0.0f)) e0[v / 64] |= 1ull << (v % 64);
    std::vector<uint64_t> lobs((size_t)std::max<uint32_t>(k, 1) * words_n, 0);
    for (uint32_t r = 0; r < k; r++)
        for (uint32_t a = l_indptr[r]; a < l_indptr[r + 1]; a++) {
            uint32_t v = l_indices[a];
            lobs[(size_t)r * words_n + v / 64] ^= 1ull << (v % 64);
        }
    // row states (magnitude bits with the sign of the message as parity)
    auto enc32 = [](float x) -> uint32_t {
        float a = std::fabs(x);
        uint32_t bits;
        std::memcpy(&bits, &a, 4);
        return bits | (x < 0.0f ? 0x80000000u : 0u);
    };
    auto enc64 = [](double x) -> uint64_t {
        double a = std::fabs(x);
        uint64_t bits;
        std::memcpy(&bits, &a, 8);
        return bits | (x < 0.0 ? 1ull << 63 : 0ull);
    };
    const float limf = (float)lim;
    uint32_t ident32;
    uint64_t ident64;
    std::memcpy(&ident32, &limf, 4);
    std::memcpy(&ident64, &lim, 8);

    // ---- member schedules (Sec. III.D.1: one fixed serial order per member).
    //      Two columns that share a check must keep their permutation order:
    //      the later one reads the earlier one's new message, and the earlier
    //      one reads the later one's previous message.  Columns that share no
    //      check commute.  So the sweep is any topological order of the DAG
    //      whose arcs join consecutive columns of each row, cut into chunks
    //      of columns that are mutually independent.  Chunks are packed by
    //      list scheduling (ready columns by decreasing height, the longest
    //      chain of successors below them, then by permutation position) into
    //      at most 64 edges each, which reaches max(#levels, ceil(E / 64))
    //      chunks on the workloads here.
    // compact item bodies (bp_compact.h): FP32, serial or parallel schedule,
    // columns of at most 8 checks, row states within 64 KB of LDS
    DevGraph dc{};
    dc.m = m;
    dc.words_m = words_m;
    dc.words_n = words_n;
    dc.flood = c.schedule == 1 ? 1 : 0;
    dc.compact = 1;
    const bool want_compact =
        !fp64 && !layered && max_col <= 8 && E && m < 8192 && bp_lds_bytes(dc, false) <= 64 * 1024;
    const uint32_t kNone = UINT32_MAX;
    const uint32_t rb = rec_bytes(fp64), ri0 = rec_init(fp64), fb = fp64 ? 8u : 4u;
    auto member = [&](uint32_t i, SchedScratch& w, MemberSched& o) {
        std::vector<uint32_t>&s_meta = w.meta, &s_v = w.v, &init32 = w.init32, &c_sched = o.csched, &c_rec0 = o.crec0;
        std::vector<float>& s_lam32 = w.lam32;
        std::vector<double>& s_lam64 = w.lam64;
        std::vector<uint64_t>& init64 = w.init64;
        std::vector<uint32_t>&last = w.last, &level = w.level, &height = w.height, &npred = w.npred, &pos = w.pos;
        std::vector<uint32_t>&succ = w.succ, &taken = w.taken, &running32 = w.running32, &c_later = w.later;
        std::vector<uint64_t>&skipped = w.skipped, &running64 = w.running64;
        std::vector<float>& c_exp = w.expected;
        last.resize(m), running32.resize(m), running64.resize(m), c_later.resize(m);
        level.resize(n), height.resize(n), npred.resize(n), pos.resize(n), succ.resize(E);
        s_meta.clear(), s_v.clear(), s_lam32.clear(), s_lam64.clear();
        size_t nchunks = 0;
        const uint32_t* pi = perms + (size_t)i * n;
        std::fill(last.begin(), last.end(), kNone);
        std::fill(succ.begin(), succ.end(), kNone);
        uint32_t nlev = 0, ncols = 0;
        for (uint32_t a = 0; a < n; a++) {
            const uint32_t v = pi[a];
            pos[v] = a;
            npred[v] = 0;
            uint32_t lv = 0;
            for (uint32_t j = cp[v]; j < cp[v + 1]; j++) {
                const uint32_t r = ci[j], u = last[r];
                if (u != kNone) {
                    // arc u -> v through row r; u's edge on r is the one
                    // whose check is r
                    uint32_t ju = cp[u];
                    while (ci[ju] != r) ju++;
                    succ[ju] = v;
                    bool dup = false;
                    for (uint32_t j2 = cp[v]; j2 < j; j2++) dup |= last[ci[j2]] == u;
                    if (!dup) npred[v]++;
                    lv = std::max(lv, level[u]);
                }
            }
            for (uint32_t j = cp[v]; j < cp[v + 1]; j++) last[ci[j]] = v;
            level[v] = lv + 1;
            if (cp[v + 1] > cp[v]) {
                nlev = std::max(nlev, level[v]);
                ncols++;
            }
        }
        for (uint32_t a = n; a-- > 0;) {
            const uint32_t u = pi[a];
            uint32_t h = 0;
            for (uint32_t j = cp[u]; j < cp[u + 1]; j++)
                if (succ[j] != kNone) h = std::max(h, height[succ[j]]);
            height[u] = h + 1;
        }
        o.levels = nlev;
        // ready queue keyed by (larger height, earlier position)
        auto key = [&](uint32_t v) { return ((uint64_t)(~height[v]) << 32) | pos[v]; };
        std::priority_queue<uint64_t, std::vector<uint64_t>, std::greater<uint64_t>> ready;
        for (uint32_t a = 0; a < n; a++) {
            const uint32_t v = pi[a];
            if (cp[v + 1] > cp[v] && npred[v] == 0) ready.push(key(v));
        }
        uint32_t placed = 0;
        while (!ready.empty()) {
            uint32_t cap = kWave, dmax = 0;
            taken.clear();
            skipped.clear();
            while (!ready.empty() && cap > 0 && skipped.size() < (size_t)kWave) {
                const uint64_t kv = ready.top();
                ready.pop();
                const uint32_t v = pi[(uint32_t)kv];
                const uint32_t d = cp[v + 1] - cp[v];
                if (d <= cap) {
                    taken.push_back(v);
                    cap -= d;
                    dmax = std::max(dmax, d);
                } else {
                    skipped.push_back(kv);
                }
            }
            for (uint64_t kv : skipped) ready.push(kv);
            for (uint32_t v : taken) {
                const uint32_t d = cp[v + 1] - cp[v];
                for (uint32_t j = 0; j < d; j++) {
                    s_meta.push_back(ci[cp[v] + j] | (j << 16) | (d << kMetaDegShift) | (dmax << kMetaDmaxShift));
                    s_v.push_back(v);
                    if (fp64) s_lam64.push_back(lam64[v]);
                    else s_lam32.push_back(lam32[v]);
                }
            }
            for (uint32_t q = kWave - cap; q < (uint32_t)kWave; q++) {  // unused slots
                s_meta.push_back(dmax << kMetaDmaxShift);
                s_v.push_back(0);
                if (fp64) s_lam64.push_back(0.0);
                else s_lam32.push_back(0.0f);
            }
            nchunks++;
            placed += (uint32_t)taken.size();
            // successors become ready once this chunk is complete
            for (uint32_t u : taken)
                for (uint32_t j = cp[u]; j < cp[u + 1]; j++) {
                    const uint32_t v = succ[j];
                    if (v == kNone) continue;
                    bool dup = false;
                    for (uint32_t j2 = cp[u]; j2 < j; j2++) dup |= succ[j2] == v;
                    if (!dup && --npred[v] == 0) ready.push(key(v));
                }
        }
        o.whole = placed == ncols;
        const uint32_t nch = (uint32_t)nchunks;
        o.chunks = nch;
        // suffix states of the initial messages mu = lambda, from the end
        // of the sweep backwards
        const size_t end_slot = nchunks * kWave;
        if (fp64) {
            init64.resize(end_slot);
            std::fill(running64.begin(), running64.end(), ident64);
            for (size_t q = end_slot; q-- > 0;) {
                if (!((s_meta[q] >> kMetaDegShift) & 15u)) {
                    init64[q] = ident64;
                    continue;
                }
                const uint32_t r = s_meta[q] & 0xffffu;
                init64[q] = running64[r];
                running64[r] = rs_combine<uint64_t>(enc64(lam64[s_v[q]]), running64[r]);
            }
        } else {
            init32.resize(end_slot);
            std::fill(running32.begin(), running32.end(), ident32);
            for (size_t q = end_slot; q-- > 0;) {
                if (!((s_meta[q] >> kMetaDegShift) & 15u)) {
                    init32[q] = ident32;
                    continue;
                }
                const uint32_t r = s_meta[q] & 0xffffu;
                init32[q] = running32[r];
                running32[r] = rs_combine<uint32_t>(enc32(lam32[s_v[q]]), running32[r]);
            }
            if (want_compact) {
                // the compact schedule; the record of the initial
                // messages of every chunk; and how many records a chunk
                // is expected to hold: an edge with r later ones in its
                // row is the least of them with probability 1 / (r + 1)
                // (groups of four chunks, an even number of them)
                const uint32_t ng = (nch + 7) / 8 * 2;
                o.groups = ng;
                c_sched.assign((size_t)ng * 512, 0u);
                c_rec0.assign((size_t)ng * 64, 0u);
                c_exp.assign(nch, 0.0f);
                std::fill(c_later.begin(), c_later.end(), 0u);
                for (uint32_t k = ng * 4; k-- > 0;) {
                    const size_t at = (size_t)k * kWave;
                    uint32_t* sc = &c_sched[(size_t)(k / 4) * 512];
                    uint32_t* rc = &c_rec0[(size_t)k * 16];
                    uint32_t vals = 0;
                    for (uint32_t q = 0; q < (uint32_t)kWave; q++) {
                        const uint32_t mw = k < nch ? s_meta[at + q] : 0u, deg = (mw >> kMetaDegShift) & 15u;
                        const uint32_t seg = (mw >> 16) & 15u, r = mw & 0xffffu;
                        uint32_t& meta = sc[q * 4 + k % 4];
                        if (!deg) {
                            meta = m << 18 | q << 2;
                            continue;
                        }
                        std::memcpy(&sc[256 + q * 4 + k % 4], &s_lam32[at + q], 4);
                        meta = (seg + 1 == deg ? 1u << 31 : 0u) | r << 18 |
                               (((1u << deg) - 1u) & ~(1u << seg)) << 8 | (q - seg) << 2;
                        const uint32_t bits = enc32(s_lam32[at + q]), mag = init32[at + q] & 0x7fffffffu;
                        if (bits >> 31) rc[q / 32] |= 1u << (q % 32);
                        if ((bits & 0x7fffffffu) < mag) {
                            if (vals < 12) rc[4 + vals] = mag;
                            vals++;
                            rc[2 + q / 32] |= 1u << (q % 32);
                        }
                        c_exp[k] += 1.0f / (float)(++c_later[r]);
                    }
                    if (vals > 12) rc[2] = rc[3] = 0xffffffffu;
                }
                if (i == 0) {
                    o.row0 = running32;
                    if (c.schedule == 1) {  // the rows' next least magnitudes
                        o.row2.assign(m, ident32);
                        std::vector<uint32_t> least(m, ident32);
                        for (size_t q = 0; q < end_slot; q++) {
                            if (!((s_meta[q] >> kMetaDegShift) & 15u)) continue;
                            const uint32_t r = s_meta[q] & 0xffffu, mag = enc32(s_lam32[q]) & 0x7fffffffu;
                            o.row2[r] = std::min(o.row2[r], std::max(least[r], mag));
                            least[r] = std::min(least[r], mag);
                        }
                    }
                }
                // the first group that keeps its states in the slab
                // slots: least bytes over the sweep, 64 for a record that
                // fits, 256 for states in the slots, and for a record
                // that may not fit (expected count plus 2.5 standard
                // deviations above 12) what the late load costs
                uint32_t kd = nch;
                double cost = 0.0, best = 0.0;
                for (uint32_t k = nch; k-- > 0;) {
                    const double ex = c_exp[k];
                    cost += 256.0 - (ex + 2.5 * std::sqrt(ex) <= 12.0 ? 64.0 : 1024.0);
                    if (k % 8 == 0 && cost < best) {
                        best = cost;
                        kd = k;
                    }
                }
                o.dense0 = kd == nch ? ng : kd / 4;
                o.kept = kd;
            }
        }
        // interleave the schedule fields into chunk records
        o.recs.resize(nchunks * rb);
        for (size_t k = 0; k < nchunks; k++) {
            unsigned char* r = o.recs.data() + k * rb;
            std::memcpy(r, &s_meta[k * kWave], 4 * kWave);
            std::memcpy(r + kRecV, &s_v[k * kWave], 4 * kWave);
            std::memcpy(r + kRecLam, fp64 ? (const void*)&s_lam64[k * kWave] : (const void*)&s_lam32[k * kWave], fb * kWave);
            std::memcpy(r + ri0, fp64 ? (const void*)&init64[k * kWave] : (const void*)&init32[k * kWave], fb * kWave);
        }
    };
    std::vector<MemberSched> ms(layered ? 0u : c.L);  // the layered schedule has no chunks
    if (!for_members<SchedScratch>((uint32_t)ms.size(), E * c.L,
                                   [&](uint32_t i, SchedScratch& w) { member(i, w, ms[i]); }))
        return fail(VIBE_ENOMEM, "host allocation failed");
    std::vector<uint32_t> member_chunk(c.L + 1, 0), c_group(c.L + 1, 0), c_dense0(c.L, 0);
    uint32_t lev_min = UINT32_MAX, lev_max = 0, ch_min = UINT32_MAX, ch_max = 0;
    uint64_t nchunks = 0, c_chunks = 0;
    for (uint32_t i = 0; i < ms.size(); i++) {
        const MemberSched& o = ms[i];
        if (!o.whole) return fail(VIBE_EINVAL, "internal: schedule does not cover every column");
        lev_min = std::min(lev_min, o.levels);
        lev_max = std::max(lev_max, o.levels);
        ch_min = std::min(ch_min, o.chunks);
        ch_max = std::max(ch_max, o.chunks);
        nchunks += o.chunks;
        if (nchunks * kWave >= (1ull << 32)) return fail(VIBE_EUNSUPPORTED, "schedules exceed 2^32 slots");
        member_chunk[i + 1] = (uint32_t)nchunks;
        c_group[i + 1] = c_group[i] + o.groups;
        c_dense0[i] = o.dense0;
        c_chunks += o.kept;
    }
    if (ch_min == UINT32_MAX) ch_min = 0;
    vibe_graph* g = new (std::nothrow) vibe_graph();
    if (!g) return fail(VIBE_ENOMEM, "host allocation failed");
    GraphHost& h = g->h;
    (void)hipGetDevice(&g->device);
    h.cfg = c;
    h.m = m;
    h.n = n;
    h.k = k;
    h.E = E;
    h.max_row = max_row;
    h.max_col = max_col;
    h.levels_min = lev_min == UINT32_MAX ? 0 : lev_min;
    h.levels_max = lev_max;
    h.chunks_min = ch_min;
    h.chunks_max = ch_max;
    h.device_bytes = 0;
    h.perms.assign(perms, perms + (size_t)c.L * (layered ? m : n));
    DevGraph& d = h.dg;
    d.m = m;
    d.n = n;
    d.k = k;
    d.L = c.L;
    d.M = c.M;
    d.T = c.T_max;
    d.E = (uint32_t)E;
    d.words_n = words_n;
    d.words_m = words_m;
    // the layered schedule keeps its check messages (E) and running
    // posteriors (n) in the slab
    d.max_chunks = layered ? (uint32_t)((E + n + kWave - 1) / kWave) : ch_max;
    d.P = 1;
    d.dec_global = 0;
    d.compact = 0;
    d.ccols = max_col <= 6 ? 6 : 8;
    d.csched = d.crec0 = nullptr;
    d.crow0 = d.crow2 = d.cgroup = d.dense0 = nullptr;
    d.ssched = nullptr;
    d.lcols = d.lorder = nullptr;
    d.lgroups = 0;
    d.scols = d.sshape = 0;
    d.sfree = d.sitems = 0;
    d.cgroups = 0;
    d.fp64 = fp64 ? 1 : 0;
    d.flood = c.schedule == 1 ? 1 : 0;
    d.layered = layered ? 1 : 0;
    d.lsd_order = c.lsd_order;
    d.alpha = c.alpha;
    d.alpha_t = nullptr;
    d.clamp = lim;
    d.ident32 = ident32;
    d.ident64 = ident64;
    d.all_lam_positive = all_pos;
    std::vector<uint32_t> rp(h_indptr, h_indptr + m + 1);
    std::vector<uint32_t> ri(h_indices, h_indices + E);
    if (lsd_lds_bytes(d) > 150 * 1024) {
        delete g;
        return fail(VIBE_EUNSUPPORTED, "the per-shot LSD state exceeds 150 KB of LDS");
    }
    // layered sweep with the posteriors in LDS (bp_layered.h): FP32, rows of
    // at most 256 edges, posteriors within a workgroup's 160 KB
    std::vector<uint32_t> l_cols, l_order;
    if (layered && !fp64 && m && max_row <= 256 && bp_layered_lds(d) <= 160 * 1024) {
        const uint32_t NR = max_row <= 64 ? 1 : max_row <= 128 ? 2 : 4;
        const uint32_t W = 16 * bp_layered_lds(d) > 160 * 1024 ? kLayeredWaves : 1;
        d.ccols = (int)(NR | W << 3);
        l_cols.assign((size_t)(m + 1) * 64 * NR, 4u * n);
        for (uint32_t r = 0; r < m; r++)
            for (uint32_t a = h_indptr[r]; a < h_indptr[r + 1]; a++) {
                const uint32_t q = a - h_indptr[r];
                l_cols[((size_t)r * 64 + q % 64) * NR + q / 64] = 4u * h_indices[a];
            }
        // One wavefront takes the checks in the member's order.  For more, a
        // check's level: one more than that of the checks before it in the
        // member's order that share a column, which is the highest so far on
        // its columns; two of a level share none.  Levels count from 1.
        struct Columns {
            std::vector<uint32_t> level;
        };
        std::vector<uint32_t> lev((size_t)c.L * m, 0);
        std::vector<std::vector<uint32_t>> first(c.L);  // first group of each level, then the end
        // (some 3 to 8 ns an edge; building a chunked schedule takes 50 times that)
        const bool ok = W == 1 || for_members<Columns>(c.L, E * c.L / 16, [&](uint32_t i, Columns& w) {
            w.level.assign(n, 0);
            uint32_t* l = lev.data() + (size_t)i * m;
            std::vector<uint32_t> size(1, 0);
            for (uint32_t a = 0; a < m; a++) {
                const uint32_t r = perms[(size_t)i * m + a];
                uint32_t x = 0;
                for (uint32_t b = h_indptr[r]; b < h_indptr[r + 1]; b++) x = std::max(x, w.level[h_indices[b]]);
                for (uint32_t b = h_indptr[r]; b < h_indptr[r + 1]; b++) w.level[h_indices[b]] = x + 1;
                l[r] = x + 1;
                if (size.size() <= x) size.resize(x + 1, 0);
                size[x]++;
            }
            first[i].assign(1, 0);
            for (uint32_t q : size) first[i].push_back(first[i].back() + (q + W - 1) / W);
        });
        if (!ok) {
            delete g;
            return fail(VIBE_ENOMEM, "host allocation failed");
        }
        for (uint32_t i = 0; i < c.L; i++) d.lgroups = std::max(d.lgroups, W == 1 ? m : first[i].back());
        l_order.assign((size_t)c.L * d.lgroups * W, m);
        if (W == 1) l_order.assign(perms, perms + (size_t)c.L * m);
        for (uint32_t i = 0; W > 1 && i < c.L; i++) {
            for (uint32_t& f : first[i]) f *= W;
            for (uint32_t a = 0; a < m; a++) {
                const uint32_t r = perms[(size_t)i * m + a];
                l_order[(size_t)i * d.lgroups * W + first[i][lev[(size_t)i * m + r] - 1]++] = r;
            }
        }
    }
    // one lane per shot (bp_small.h): the members' columns in their order
    std::vector<uint32_t> s_sched;
    if (!fp64 && c.schedule == 0 && m && m <= 64 && n <= 64 && E && E <= kSmallMaxE && max_row <= kSmallMaxRow &&
        max_col <= kSmallMaxCol) {
        const int RO = max_row <= 6 && max_col <= 3 ? 5 : 7, DM = RO == 5 ? 3 : 4;
        const uint32_t EW = small_edge_words(RO), CWD = small_col_words(RO, DM);
        for (uint32_t v = 0; v < n; v++)
            if (cp[v + 1] == cp[v])
                d.sfree |= 1ull << v;
            else
                d.scols++;
        d.sshape = (uint32_t)RO << 4 | (uint32_t)DM;
        // One lane per shot takes up to T x columns steps however few shots
        // there are; one wavefront per item takes the items in turn, each for
        // as long as it runs, which grows with the faults a shot has.  With
        // x = shots x members / (T x columns^2) they meet at about x = 0.35 for
        // 61 columns and 0.6 faults a shot (B = 20000, L = 4, T = 64: 2.27 ms
        // and 2.21), 0.4 for 37 and 0.4 (1.28, 1.24), 0.14 for 19 and 1
        // (0.70, 0.69), below 0.1 for 7, and at 7 faults below 0.1 for 61.
        double faults = 0.0;
        for (uint32_t v = 0; v < n; v++) faults += std::min(priors[v], 1.0 - priors[v]);
        const double sq = std::max((double)d.scols * d.scols - 40.0, 0.0);
        d.sitems = std::max<uint64_t>(72, (uint64_t)(0.8 * c.T_max * sq / (1.0 + 2.0 * faults)));
        s_sched.assign((size_t)c.L * d.scols * CWD, 0);
        uint32_t* w = s_sched.data();
        for (uint32_t i = 0; i < c.L; i++)
            for (uint32_t a = 0; a < n; a++) {
                const uint32_t v = perms[(size_t)i * n + a], deg = cp[v + 1] - cp[v];
                if (!deg) continue;
                w[0] = v | deg << 8;
                std::memcpy(&w[1], &lam32[v], 4);
                for (uint32_t j = 0; j < (uint32_t)DM; j++) {
                    uint32_t* ew = w + 2 + j * EW;
                    uint32_t oth[8];
                    uint32_t no = 0, slot = (uint32_t)E, r = 0;
                    if (j < deg) {
                        r = ci[cp[v] + j];
                        slot = ce[cp[v] + j];
                        for (uint32_t b = h_indptr[r]; b < h_indptr[r + 1]; b++)
                            if (b != slot) oth[no++] = b;
                    }
                    while (no < 8) oth[no++] = (uint32_t)E;
                    ew[0] = slot * 256u | r << 16;
                    for (uint32_t q = 0; q < EW - 1; q++) ew[1 + q] = oth[2 * q] * 256u | oth[2 * q + 1] * 256u << 16;
                }
                w += CWD;
            }
        for (uint32_t a = 0; a < E; a++) {  // lambda of each message slot's column
            uint32_t bits;
            std::memcpy(&bits, &lam32[h_indices[a]], 4);
            s_sched.push_back(bits);
        }
    }
    std::vector<unsigned char> sched(std::max<size_t>(nchunks, 1) * rb);
    if (nchunks == 0)  // no edges at all: one (unused) record
        for (uint32_t q = 0; q < (uint32_t)kWave; q++)
            std::memcpy(&sched[ri0 + fb * q], fp64 ? (const void*)&ident64 : (const void*)&ident32, fb);
    for (size_t i = 0; i < ms.size(); i++)
        std::copy(ms[i].recs.begin(), ms[i].recs.end(), sched.begin() + (size_t)member_chunk[i] * rb);
    int rc = VIBE_OK;
    const float* lam32_d = nullptr;
    // Graphs of at least 16 chunks, where the padding to whole groups is
    // small: 17 chunks of rows of 5 gain 15% (8192 shots: 2.36 ms against
    // 2.79), 20 chunks of rows of 6 10%, 57 chunks of rows of 7 14% (15.4 /
    // 17.8), 118 chunks of rows of 16 9%, 464 chunks of rows of 64 29%; 12
    // chunks of 9 rows of 5 lose 3%.  Rows of a few edges have a record at
    // every second or third edge: where most chunks would not fit theirs,
    // all keep their states in the slab.
    //
    // The slabs are streamed where the messages alone, 1 KB a group, of 4096
    // wavefronts (16 on each of 256 CUs) exceed the 256 MB of the last-level
    // cache: 60 KB each take 4.87 ms, streamed 5.72; 79 KB 29.5 and 26.1.
    // That is decided here, for the graph, and so also for a launch whose few
    // slabs would stay in the caches.
    auto compact_upload = [&]() -> int {
        if (!want_compact || ch_min < 16) return VIBE_OK;
        if (2 * c_chunks < member_chunk[c.L]) std::fill(c_dense0.begin(), c_dense0.end(), 0u);
        // one allocation: the schedule, the records, then the small arrays
        const size_t groups = c_group[c.L];
        std::vector<uint32_t> all;
        all.reserve(groups * (512 + 64) + 2 * (size_t)m + 2 * c.L + 4 * 64 + 1);
        for (MemberSched& o : ms) all.insert(all.end(), o.csched.begin(), o.csched.end());
        for (MemberSched& o : ms) all.insert(all.end(), o.crec0.begin(), o.crec0.end());
        size_t at[4], i4 = 0;
        for (const std::vector<uint32_t>* v : {&ms[0].row0, &ms[0].row2, &c_group, &c_dense0}) {
            all.resize((all.size() + 63) / 64 * 64);
            at[i4++] = all.size();
            all.insert(all.end(), v->begin(), v->end());
        }
        const uint32_t* p = nullptr;
        if (int r = upload(h, all.data(), all.size(), &p)) return r;
        d.csched = reinterpret_cast<const unsigned char*>(p);
        d.crec0 = reinterpret_cast<const unsigned char*>(p + groups * 512);
        d.crow0 = p + at[0];
        d.crow2 = p + at[1];
        d.cgroup = p + at[2];
        d.dense0 = p + at[3];
        for (uint32_t i = 0; i < c.L; i++) d.cgroups = std::max(d.cgroups, c_group[i + 1] - c_group[i]);
        if (d.cgroups > 64) d.ccols |= kCompactStream;
        return VIBE_OK;
    };
    if ((rc = upload(h, rp.data(), rp.size(), &d.rp)) ||
        (rc = upload(h, ri.data(), ri.size(), &d.ri)) ||
        (rc = upload(h, cp.data(), cp.size(), &d.cp)) ||
        (rc = upload(h, ci.data(), ci.size(), &d.ci)) ||
        (rc = upload(h, lam64.data(), lam64.size(), &d.lam64)) ||
        (!fp64 && (rc = upload(h, lam32.data(), lam32.size(), &lam32_d))) ||
        (rc = upload(h, e0.data(), e0.size(), &d.e0)) ||
        (rc = upload(h, sched.data(), sched.size(), &d.sched)) ||
        (rc = upload(h, member_chunk.data(), member_chunk.size(), &d.member_chunk)) ||
        (rc = upload(h, layered ? perms : (const uint32_t*)nullptr, layered ? (size_t)c.L * m : 1, &d.cperm)) ||
        (rc = upload(h, lobs.data(), lobs.size(), &d.lobs)) || (rc = compact_upload()) ||
        (!l_cols.empty() && ((rc = upload(h, l_cols.data(), l_cols.size(), &d.lcols)) ||
                             (rc = upload(h, l_order.data(), l_order.size(), &d.lorder)))) ||
        (!s_sched.empty() && (rc = upload(h, s_sched.data(), s_sched.size(), &d.ssched)))) {
        free_all(h);
        delete g;
        return rc;
    }
    d.lam = fp64 ? (const void*)d.lam64 : (const void*)lam32_d;
    *out = g;
    return VIBE_OK;
}

extern "C" void vibe_graph_destroy(vibe_graph* g) {
    if (!g) return;
    (void)hipDeviceSynchronize();
    for (auto& v : g->ev)
        for (auto& pr : v) {
            (void)hipEventDestroy(pr.first);
            (void)hipEventDestroy(pr.second);
        }
    free_all(g->h);
    if (g->ws.base) (void)hipFree(g->ws.base);
    if (g->ws_in.base) (void)hipFree(g->ws_in.base);
    delete g;
}

extern "C" int vibe_graph_set_alpha(vibe_graph* g, const double* alpha, uint32_t count) {
    set_error("");
    if (!g) return fail(VIBE_EINVAL, "graph handle is NULL");
    if (count > (uint32_t)kMaxT) return fail(VIBE_EINVAL, "count must be in 0..64");
    if (count == 0) {
        g->h.dg.alpha_t = nullptr;
        return VIBE_OK;
    }
    if (!alpha) return fail(VIBE_EINVAL, "alpha is NULL");
    double table[kMaxT];
    for (uint32_t t = 0; t < (uint32_t)kMaxT; t++) {
        const double a = alpha[t < count ? t : count - 1];
        if (!(a > 0.0) || !(a <= 1e6)) return fail(VIBE_EINVAL, "every alpha must be in (0, 1e6]");
        table[t] = a;
    }
    // a new table every call: launches already queued and captured
    // sequences keep reading the table they were given (512 bytes each,
    // freed with the graph)
    const double* dev = nullptr;
    int rc = upload(g->h, table, kMaxT, &dev);
    if (rc) return rc;
    g->h.dg.alpha_t = dev;
    return VIBE_OK;
}

extern "C" int vibe_graph_get_schedules(const vibe_graph* g, uint32_t* perms) {
    if (!g || !perms) return fail(VIBE_EINVAL, "NULL argument");
    std::memcpy(perms, g->h.perms.data(), 4 * g->h.perms.size());
    return VIBE_OK;
}

extern "C" int vibe_graph_info(const vibe_graph* g, vibe_graph_info_t* info) {
    if (!g || !info) return fail(VIBE_EINVAL, "NULL argument");
    const GraphHost& h = g->h;
    info->m = h.m;
    info->n = h.n;
    info->k = h.k;
    info->L = h.cfg.L;
    info->M = h.cfg.M;
    info->T_max = h.cfg.T_max;
    info->nnz = h.E;
    info->max_row_degree = h.max_row;
    info->max_col_degree = h.max_col;
    info->levels_min = h.levels_min;
    info->levels_max = h.levels_max;
    info->chunks_min = h.chunks_min;
    info->chunks_max = h.chunks_max;
    info->message_bits = h.dg.fp64 ? 64 : 32;
    info->grad_width = g->grad_width;
    info->device_bytes = h.device_bytes;
    return VIBE_OK;
}
