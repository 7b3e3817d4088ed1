// The layered (check-serial) sweep with the posteriors in LDS (FP32, rows of
// at most 256 edges).  Included by bp.hip; the operations of layered_sweep on
// every message, in an order that gives the same values.
//
// With the posteriors in global memory every edge of a check reads and
// writes a 64-byte sector of its own, and each check waits for what the one
// before it stored.  Here a check's gather, its row reductions (DPP, no LDS)
// and its scatter are the chain.  Rows are padded to NR edges per lane, so a
// check's columns and its messages are one load each, issued four steps
// ahead (no other check touches them); an edge that pads a row works on a
// dummy posterior of +inf, which clamps to the limit, joins no minimum and
// stays what it is whatever message its slot holds.
//
// Checks that share no column commute, so the host groups W such checks
// (level by level of the member's order) and each of W wavefronts takes one
// of a group, with a barrier between groups: the posteriors in LDS leave room
// for few items per CU (two of the d = 9 circuit graph), and a wavefront
// alone issues an instruction every four or five cycles at best.
//
// A row's least magnitude m1 is the wave's minimum; the next least, m2, is
// m1 itself if it occurs twice, else the minimum of the rest; every edge at
// m1 takes m2, the others m1.
//
// Bound by each check's chain (0.4 us a group) and by instruction issue.  With
// 32 members: d = 9 circuit graph, 1 shot 21.2 -> 1.9 ms, a decode of 200
// shots 86.7 -> 25.9 ms (this kernel 81.8 -> 22.4); d = 5, 2000 shots 24.6 ->
// 15.3 ms; d = 11, 200 shots 216 -> 70 ms; one wavefront per item 49 ms on the
// 200 shots of d = 9, two checks interleaved in it 45.6.

constexpr uint32_t kLAhead = 4;

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_min(uint32_t x) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, CTRL, ROWS, 0xf, false);
    return o < x ? o : x;
}
// the minimum over the wavefront's 64 lanes (all active), wave-uniform
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
    x = dpp_min<0x111, 0xf>(x);  // row_shr 1, 2, 4, 8: lane 15 of each row
    x = dpp_min<0x112, 0xf>(x);
    x = dpp_min<0x114, 0xf>(x);
    x = dpp_min<0x118, 0xf>(x);
    x = dpp_min<0x142, 0xa>(x);  // row_bcast 15 into rows 1 and 3
    x = dpp_min<0x143, 0xc>(x);  // row_bcast 31 into rows 2 and 3: lane 63
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// NR 32-bit words of a lane, as one load or store
template <int NR>
struct LWords {
    uint32_t w[NR];
};
template <int NR>
__device__ __forceinline__ void lload(LWords<NR>& d, Rsrc r, uint32_t voff, uint32_t soff) {
    if constexpr (NR == 1) {
        d.w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0);
    } else if constexpr (NR == 2) {
        const auto u = __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0);
        d.w[0] = u[0], d.w[1] = u[1];
    } else {
        const auto u = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0);
        d.w[0] = u[0], d.w[1] = u[1], d.w[2] = u[2], d.w[3] = u[3];
    }
}
template <int NR>
__device__ __forceinline__ void lstore(const LWords<NR>& d, Rsrc r, uint32_t voff, uint32_t soff) {
    if constexpr (NR == 1) {
        __builtin_amdgcn_raw_buffer_store_b32(d.w[0], r, (int)voff, (int)soff, 0);
    } else if constexpr (NR == 2) {
        using V2 = __attribute__((ext_vector_type(2))) unsigned int;
        __builtin_amdgcn_raw_buffer_store_b64(V2{d.w[0], d.w[1]}, r, (int)voff, (int)soff, 0);
    } else {
        bstore4<0>(u32x4{d.w[0], d.w[1], d.w[2], d.w[3]}, r, voff, soff);
    }
}

struct LCtx {
    Rsrc cols, msg;  // per check [64][NR]: 4 * column (padding: 4 n), the check messages
    unsigned char* L;  // posteriors (LDS), then +inf
    const uint64_t* sb;
    float al, lim;
    uint32_t lane;
    bool first;      // the first sweep: every check message is 0 and none is stored yet
};

template <int NR>
struct LEdges {
    LWords<NR> v, r;
};

template <int NR>
__device__ __forceinline__ void lfetch(const LCtx& x, LEdges<NR>& e, uint32_t c) {
    lload<NR>(e.v, x.cols, x.lane * 4u * NR, c * 256u * NR);
    lload<NR>(e.r, x.msg, x.lane * 4u * NR, c * 256u * NR);
}

// Check c, loaded in e; pads: how many of its 64 NR edges are padding.
template <int NR>
__device__ __forceinline__ void lcheck(const LCtx& x, const LEdges<NR>& e, uint32_t c, uint32_t pads, uint32_t& sat) {
    constexpr uint32_t kS = 0x80000000u;
    const uint64_t sw = x.sb[c >> 6];
    float mraw[NR], mu[NR], m1 = x.lim, m2 = x.lim;
#pragma unroll
    for (int q = 0; q < NR; q++) mraw[q] = *reinterpret_cast<float*>(x.L + e.v.w[q]);
    uint32_t sg = 0, hit = 0;
#pragma unroll
    for (int q = 0; q < NR; q++) {
        mraw[q] -= x.first ? 0.0f : __uint_as_float(e.r.w[q]);
        mu[q] = Prec<float>::clamp(mraw[q], x.lim);
        const float mag = fabsf(mu[q]);
        hit += (uint32_t)__popcll(__ballot(mag >= x.lim));
        m2 = __builtin_amdgcn_fmed3f(m1, m2, mag);
        m1 = __builtin_amdgcn_fmed3f(0.0f, m1, mag);  // the lesser of two that are not negative
        sg ^= __float_as_uint(mu[q]);
    }
    sat |= hit != pads ? 1u : 0u;
    const uint32_t g1 = wave_min(__float_as_uint(m1));
    const bool mine = __float_as_uint(m1) == g1;
    const uint32_t rest = wave_min(__float_as_uint(mine ? m2 : m1));
    const uint32_t g2 = __popcll(__ballot(mine)) > 1 ? g1 : rest;
    const uint32_t odd = (uint32_t)__popcll(__ballot((int32_t)sg < 0)) ^ (uint32_t)(sw >> (c & 63u));
    const uint32_t flip = uni(odd << 31);
    const uint32_t r1 = __float_as_uint(x.al * __uint_as_float(g1)), r2 = __float_as_uint(x.al * __uint_as_float(g2));
    LWords<NR> rn;
#pragma unroll
    for (int q = 0; q < NR; q++) {
        const uint32_t u = __float_as_uint(mu[q]);
        rn.w[q] = ((u & ~kS) == g1 ? r2 : r1) | ((u ^ flip) & kS);
        *reinterpret_cast<float*>(x.L + e.v.w[q]) = mraw[q] + __uint_as_float(rn.w[q]);
    }
    lstore<NR>(rn, x.msg, x.lane * 4u * NR, c * 256u * NR);
}

// The sweep over the groups of order (W entries each; m: no check) by the W
// wavefronts of the block, then the decisions: eb and the residual follow the
// clamped posteriors (a column without checks keeps lambda_v and its
// decision).
template <int NR, int W>
__device__ __forceinline__ void lsweep(const DevGraph& g, const LCtx& x, uint32_t wv, const uint32_t* order,
                                       uint64_t* eb, uint64_t* res, float* post, bool want_post, uint32_t& sat) {
    const uint32_t lane = x.lane;
    // the wavefront's checks of 64 groups at a time, described by its lanes:
    // this block's and the next one's (past the last: the empty check m)
    uint32_t bc, bp, nc, np;
    auto block = [&](uint32_t base, uint32_t& c, uint32_t& pads) {
        c = base + lane < g.lgroups ? order[(base + lane) * W + wv] : g.m;
        pads = 64u * NR - (c < g.m ? g.rp[c + 1] - g.rp[c] : 0u);
    };
    auto pick = [](uint32_t v, uint32_t i) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)i); };
    block(0, bc, bp);
    LEdges<NR> ring[kLAhead];
#pragma unroll
    for (uint32_t d = 0; d < kLAhead; d++) {
        lfetch<NR>(x, ring[d], pick(bc, d));
        __builtin_amdgcn_sched_barrier(0);
    }
    for (uint32_t base = 0; base < g.lgroups; base += kWave) {
        block(base + kWave, nc, np);
        const uint32_t cnt = min((uint32_t)kWave, (g.lgroups - base + kLAhead - 1) / kLAhead * kLAhead);
        for (uint32_t i = 0; i < cnt; i += kLAhead) {
            const bool over = i + kLAhead >= kWave;  // the next steps are the next block's first
#pragma unroll
            for (uint32_t d = 0; d < kLAhead; d++) {
                lcheck<NR>(x, ring[d], pick(bc, i + d), pick(bp, i + d), sat);
                lfetch<NR>(x, ring[d], over ? pick(nc, d) : pick(bc, (i + d + kLAhead) & 63u));
                if constexpr (W > 1) {
                    // posteriors written before the next group reads them
                    // (loads in flight are not waited for)
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                } else {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        bc = nc;
        bp = np;
    }
    const float* L = reinterpret_cast<const float*>(x.L);
    for (uint32_t w = wv; w < g.words_n; w += W) {
        const uint32_t v = w * 64u + lane;
        const float Lv = v < g.n ? Prec<float>::clamp(L[v], x.lim) : 1.0f;
        const bool lim_hit = v < g.n && fabsf(Lv) >= x.lim;
        if (__ballot(lim_hit)) sat |= __ballot(lim_hit && g.cp[v + 1] != g.cp[v]) ? 1u : 0u;
        if (want_post && v < g.n) post[v] = g.cp[v + 1] != g.cp[v] ? Lv : reinterpret_cast<const float*>(g.lam)[v];
        const uint64_t now = __ballot(Lv <= 0.0f), was = eb[w];
        if (now != was) {
            if (lane == 0) eb[w] = now;
            if (((now ^ was) >> lane) & 1ull)
                for (uint32_t j = g.cp[v]; j < g.cp[v + 1]; j++) {
                    const uint32_t c = g.ci[j];
                    atomicXor(reinterpret_cast<unsigned long long*>(&res[c >> 6]), 1ull << (c & 63));
                }
        }
    }
}

// One work item by a block of W wavefronts, as run_item.  What depends on
// other items' progress is decided by the first wavefront and passed through
// LDS, so that all take the same path.
template <int NR, int W>
__device__ __forceinline__ void run_item_l(const DevGraph& g, const BpLaunch& a, uint32_t item, unsigned char* lds,
                                           Rsrc slb, float* post) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = uni(tid >> 6);
    uint64_t* sb = reinterpret_cast<uint64_t*>(lds);
    uint64_t* res = sb + g.words_m;
    uint64_t* eb = res + g.words_m;
    float* L = reinterpret_cast<float*>(eb + g.words_n);
    uint32_t* ctl = reinterpret_cast<uint32_t*>(L + g.n + 1);  // [0] stop, [1] saturation
    const float* lamv = reinterpret_cast<const float*>(g.lam);
    const float lim = (float)g.clamp;
    uint32_t shot, mem;
    if (a.member_major) {
        mem = item / a.n_shots;
        shot = item % a.n_shots;
    } else {
        shot = item / g.L;
        mem = item % g.L;
    }
    const uint32_t rec = shot * g.L + mem;
    const uint8_t* s = a.syndromes + (size_t)(a.shot0 + shot) * g.m;
    uint64_t* cmask = a.conv_mask + (size_t)shot * (kMaxT + 1);
    for (uint32_t w = wv; w < g.words_m; w += W) {
        const uint32_t c = w * 64u + lane;
        const uint64_t mask = __ballot(c < g.m && s[c] != 0);
        if (lane == 0) sb[w] = res[w] = mask;
    }
    for (uint32_t w = tid; w < g.words_n; w += 64u * W) eb[w] = g.e0[w];
    for (uint32_t v = tid; v < g.n; v += 64u * W) L[v] = Prec<float>::clamp(lamv[v], lim);
    if (tid == 0) {
        L[g.n] = INFINITY;
        ctl[1] = 0u;
    }
    // stop: M members of lower index converged at the first iteration
    auto stop_before = [&](uint32_t t) {
        if (wv == 0) {
            const uint32_t stop = a.use_M && preceding_converged(cmask, t, mem, (int)lane) >= g.M ? 1u : 0u;
            if (lane == 0) ctl[0] = stop;
        }
        __syncthreads();
        const uint32_t stop = uni(ctl[0]);
        __syncthreads();
        return stop != 0;
    };
    if (stop_before(1)) {
        if (tid == 0) a.t_conv[rec] = 0;
        return;
    }
    bool any = false;
    for (uint32_t w = lane; w < g.words_m; w += kWave) any |= sb[w] != 0;
    if (__ballot(any) == 0 && a.fast_zero && g.all_lam_positive) {
        if (wv == 0) zero_item(g, a, shot, mem, (int)lane);
        return;
    }
    float* post_out = a.post_out ? reinterpret_cast<float*>(a.post_out) + (size_t)rec * g.n : nullptr;
    LCtx x{make_rsrc(g.lcols, (g.m + 1u) * 256u * NR), slb, reinterpret_cast<unsigned char*>(L), sb, (float)g.alpha, lim,
           lane, true};
    const uint32_t* order = g.lorder + (size_t)mem * g.lgroups * W;
    uint32_t conv_t = 0, ran = 0, sat = 0;
    bool stopped = false;
    for (uint32_t t = 1; t <= a.T_run; t++) {
        if (t >= 2 && a.use_M && stop_before(t)) {
            stopped = true;
            break;
        }
        if (g.alpha_t) x.al = (float)g.alpha_t[t - 1];
        const bool want_post = post_out != nullptr || (a.accumulate_q && t == a.T_run);
        x.first = t == 1;
        lsweep<NR, W>(g, x, wv, order, eb, res, post, want_post, sat);
        if (post_out)  // each lane copies what it wrote
            for (uint32_t w = wv; w < g.words_n; w += W)
                if (w * 64u + lane < g.n) post_out[w * 64u + lane] = post[w * 64u + lane];
        __syncthreads();
        ran = t;
        bool nz = false;
        for (uint32_t w = lane; w < g.words_m; w += kWave) nz |= res[w] != 0;
        const bool met = __ballot(nz) == 0;
        __syncthreads();  // the residual is read before the next sweep changes it
        if (met) {
            if (!conv_t) conv_t = t;
            if (a.stop_on_converge) break;
        }
    }
    if (sat && lane == 0) atomicOr(&ctl[1], 1u);
    __threadfence();  // posteriors, read by the first wavefront
    __syncthreads();
    if (wv == 0) finish_item<float>(g, a, shot, mem, conv_t, ran, stopped, uni(ctl[1]) != 0, eb, post, (int)lane);
}
