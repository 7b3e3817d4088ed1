// K1 for graphs of a few columns (code capacity): one lane per shot.
// Included by bp.hip.
//
// With one wavefront per (shot, member), a graph of some ten chunks with a
// few edges each spends its time on half-empty steps, barriers and the loads
// of the correction limit.  Here one wavefront runs a member on 64 shots,
// one per lane, column by column in the member's order: every lane does the
// same column at the same time, so the column's description (its checks, the
// message slots of each check's other edges) is scalar, the messages lie in
// LDS at [slot][lane] without bank conflicts, sums over a column need no
// shuffles, and a shot's syndrome, residual and decisions are one 64-bit
// word each in its lane's registers.  A check message is formed from the
// row's other messages as they stand, which is the serial schedule itself.
//
// A wavefront has an even share of the member's shots.  A lane whose shot is
// decided (converged, out of the first M, or at the iteration limit) waits
// until there are kSmallRefill of them; then their outputs are written and
// they take the next shots of the share.  So the work is that of the shots,
// and only the last ones leave lanes idle.  Where 64 shots were taken and run
// until the last was decided, one that ran to the limit held all lanes: d = 9
// (61 columns), p = 0.01, T = 64, 20000 shots of 16 members took 16.0 ms, one
// wavefront per item 4.4, this form 2.3; at p = 0.12, where many reach the
// limit, 17.3, 38.7 and 19.3 ms.
//
// The correction limit: when it takes shots and on every eighth iteration, a
// wavefront counts the members that precede its own from each shot's
// convergence masks.  Looking on every iteration cost 0.25 us of 3 (7 columns).
//
// Bound by instruction issue, about 200 per column and 64 shots, scalar ones
// among them (0.45 us a column): d = 5 code capacity, 16 members, p = 0.05,
// T = 32, 10000 shots 374 us against 2.29 ms with one wavefront per shot and
// member.  Loading the next column's description during the current one's work
// gained nothing.

// idle lanes at which a wavefront writes the outputs of decided shots and
// starts new ones, which costs the same however many there are
constexpr int kSmallRefill = 16;

// bit b of the result: byte b of w is not 0
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t w) {
    const uint32_t x = ((((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u) >> 7;
    return (x * 0x10204080u) >> 28;
}

// Members converged by iteration t (0: none are looked at).
__device__ __forceinline__ uint32_t converged_upto(const uint64_t* cmask, uint32_t t) {
    uint32_t cnt = 0;
    for (uint32_t i = 1; __ballot(i <= t); i += 16) {
        uint64_t m[16];
#pragma unroll
        for (uint32_t j = 0; j < 16; j++) m[j] = load_mask(&cmask[min(i + j, (uint32_t)kMaxT)]);
#pragma unroll
        for (uint32_t j = 0; j < 16; j++) cnt += i + j <= t ? (uint32_t)__popcll(m[j]) : 0u;
    }
    return cnt;
}

// The m <= 64 syndrome bytes of a shot as bits.
__device__ __forceinline__ uint64_t syndrome_bits(const uint8_t* s, uint32_t m) {
    uint64_t b = 0;
    if (m < 4) {
        for (uint32_t c = 0; c < m; c++) b |= (uint64_t)(s[c] != 0 ? 1u : 0u) << c;
        return b;
    }
#pragma unroll 4
    for (uint32_t c = 0; c < m; c += 4) {
        const uint32_t at = min(c, m - 4);  // the last four may overlap
        uint32_t w;
        __builtin_memcpy(&w, s + at, 4);
        b |= (uint64_t)nonzero_bytes(w) << at;
    }
    return b;
}

template <int RO, int DM>
__global__ __launch_bounds__(kWave) void bp_small_kernel(DevGraph g, BpLaunch a) {
    constexpr uint32_t EW = small_edge_words(RO), CWD = small_col_words(RO, DM);
    using CWord = const __attribute__((address_space(4))) uint32_t;
    const uint32_t lane = threadIdx.x, lane4 = lane * 4u;
    const uint32_t post0 = (g.E + 1u) * 256u;  // posteriors [v][lane] after the messages
    const float lim = (float)g.clamp;
    const float* lamv = reinterpret_cast<const float*>(g.lam);
    CWord* lam_e = (CWord*)(g.ssched + (size_t)g.L * g.scols * CWD);
    // fewer than M other members never stop one
    const bool limited = a.use_M && g.M < g.L;
    const uint64_t e0 = g.e0[0];
    const float alpha = (float)g.alpha;
    *lds_at(g.E * 256u + lane4) = g.ident32;
    // The wavefront's member, or members where there are fewer wavefronts, and
    // its share of the shots: those of a member are split evenly over the
    // member's wavefronts.  (Shots taken from a counter as lanes fall idle left
    // some wavefronts with none and others with a second run to the limit.)
    const uint32_t G = gridDim.x, b = blockIdx.x;
    uint32_t mem = uni((uint32_t)((uint64_t)b * g.L / G));
    const uint32_t end = max(mem + 1, uni((uint32_t)(((uint64_t)b + 1) * g.L / G)));
    for (; mem < end; mem++) {
        uint32_t next = 0, last = a.n_shots;
        if (G > g.L) {
            const uint32_t b0 = uni((uint32_t)(((uint64_t)mem * G + g.L - 1) / g.L));
            const uint32_t b1 = uni((uint32_t)((((uint64_t)mem + 1) * G + g.L - 1) / g.L));
            next = uni((uint32_t)((uint64_t)a.n_shots * (b - b0) / (b1 - b0)));
            last = uni((uint32_t)((uint64_t)a.n_shots * (b - b0 + 1) / (b1 - b0)));
        }
        CWord* cols = (CWord*)(g.ssched + (size_t)mem * g.scols * CWD);
        const uint64_t lower = (1ull << mem) - 1ull, own = 1ull << mem;
        // the 64 shots taken last, one a lane: their syndromes, and those not
        // yet started
        uint32_t block = 0;
        uint64_t bsynd = 0, avail = 0;
        uint64_t busy = 0;  // lanes with a shot in work
        uint64_t fin = 0;   // lanes whose shot is decided, its outputs to be written
        // of the lane's shot: its index, syndrome, iteration and saturation
        // witness; when decided: whether it converged, its decisions, and
        // whether it ran to the limit
        uint32_t shot = 0, t = 1;
        uint64_t s = 0, e_conv = 0;
        float satm = 0.0f, satf = 0.0f;
        bool conv = false, ran_out = false;
        for (uint32_t step = 0;; step++) {
            while (__popcll(~busy) >= kSmallRefill) {
                if (!avail && next < last) {
                    block = next;
                    next = min(next + (uint32_t)kWave, last);
                    bool start = lane < next - block;
                    if (start) {
                        const uint32_t sh = block + lane, rec = sh * g.L + mem;
                        uint64_t* cmask = a.conv_mask + (size_t)sh * (kMaxT + 1);
                        const uint64_t at_1 = limited ? load_mask(&cmask[1]) : 0ull;
                        bsynd = syndrome_bits(a.syndromes + (size_t)(a.shot0 + sh) * g.m, g.m);
                        if (limited && (uint32_t)__popcll(at_1 & lower) >= g.M) {
                            a.t_conv[rec] = 0;
                            start = false;
                        } else if (bsynd == 0 && a.fast_zero && g.all_lam_positive) {
                            // converges at once to e = 0
                            a.t_conv[rec] = 1;
                            a.cand[rec] = 0;
                            a.weight[rec] = 0.0;
                            atomicAdd(&a.iters[sh], 1u);
                            atomicOr(reinterpret_cast<unsigned long long*>(&cmask[1]), own);
                            start = false;
                        }
                    }
                    avail = __ballot(start);
                    if (!avail) continue;
                }
                // (with no more shots to come, once for all lanes)
                if (fin && (avail || !busy)) {
                    if ((fin >> lane) & 1ull) {
                        const uint32_t rec = shot * g.L + mem;
                        a.t_conv[rec] = conv ? (int32_t)t : 0;
                        atomicAdd(&a.iters[shot], t);
                        if (conv) {
                            a.cand[rec] = e_conv;
                            // W(e) = sum_v e_v lambda_v in FP64, ascending v (a
                            // column that is 0 adds an exact zero)
                            double W = 0.0;
#pragma unroll 4
                            for (uint32_t v = 0; v < g.n; v++) W += (e_conv >> v) & 1ull ? g.lam64[v] : 0.0;
                            a.weight[rec] = W;
                        }
                        if (satf >= lim)
                            atomicOr(reinterpret_cast<unsigned long long*>(a.conv_mask + (size_t)shot * (kMaxT + 1)), own);
                        if (ran_out) {
                            // the normalised posterior, as in finish_item;
                            // columns without checks keep lambda.  The sum
                            // is read only where no member has converged:
                            // finding that out costs more than adding.
                            auto post = [&](uint32_t v) {
                                return (double)((g.sfree >> v) & 1ull ? lamv[v] : __uint_as_float(*lds_at(post0 + v * 256u + lane4)));
                            };
                            double ss = 0.0;
                            for (uint32_t v = 0; v < g.n; v++) {
                                const double xv = post(v), sq = xv * xv;
                                ss += sq;
                            }
                            if (ss > 0.0) {
                                const double scale = kQScale / sqrt(ss);
                                int64_t* q = a.qfix + (size_t)shot * g.n;
                                for (uint32_t v = 0; v < g.n; v++)
                                    atomicAdd(reinterpret_cast<unsigned long long*>(&q[v]),
                                              (unsigned long long)llrint(post(v) * scale));
                            }
                        }
                    }
                    fin = 0;
                }
                if (!avail) break;
                // the k-th idle lane takes the k-th available shot: lane k
                // receives that shot's place in the block, then passes it on
                const uint32_t give = (uint32_t)__popcll(avail), rank = lane_rank(~busy);
                const uint32_t to = (avail >> lane) & 1ull ? lane_rank(avail) : give + lane - lane_rank(avail);
                const uint32_t kth = (uint32_t)__builtin_amdgcn_ds_permute((int)(to * 4u), (int)lane);
                const uint32_t from = 4u * (uint32_t)__builtin_amdgcn_ds_bpermute((int)(rank * 4u), (int)kth);
                const uint32_t s_lo = (uint32_t)__builtin_amdgcn_ds_bpermute((int)from, (int)(uint32_t)bsynd);
                const uint32_t s_hi = (uint32_t)__builtin_amdgcn_ds_bpermute((int)from, (int)(uint32_t)(bsynd >> 32));
                const bool start = !((busy >> lane) & 1ull) && rank < give;
                if (start) {
                    shot = block + from / 4u;
                    s = (uint64_t)s_hi << 32 | s_lo;
                    t = 1;
                    satm = 0.0f;
                    // the initial messages: lambda of each slot's column
#pragma unroll 8
                    for (uint32_t q = 0; q < g.E; q++) *lds_at(q * 256u + lane4) = lam_e[q];
                }
                // the first `rank` available ones are taken: those whose
                // place among them is below the number of idle lanes
                const uint32_t idle = (uint32_t)__popcll(~busy);
                busy |= __ballot(start);
                avail &= ~__ballot(((avail >> lane) & 1ull) && lane_rank(avail) < idle);
            }
            if (!busy) break;
            const bool act = (busy >> lane) & 1ull, ends = act && t == a.T_run;
            uint64_t* cmask = a.conv_mask + (size_t)shot * (kMaxT + 1);
            const float al = g.alpha_t ? (float)g.alpha_t[t - 1] : alpha;
            const bool want_post = __ballot(ends) != 0;
            uint64_t e = e0, res = s;
            for (uint32_t q = 0; q < g.scols; q++) {
                CWord* w = cols + (size_t)q * CWD;
                uint32_t wd[CWD];
#pragma unroll
                for (uint32_t i = 0; i < CWD; i++) wd[i] = w[i];
                const uint32_t v = wd[0] & 0xffu, deg = wd[0] >> 8;
                uint32_t x[DM][RO];
#pragma unroll
                for (int j = 0; j < DM; j++)
#pragma unroll
                    for (int i = 0; i < RO; i++) {
                        const uint32_t o = wd[2 + j * EW + 1 + i / 2];
                        x[j][i] = *lds_at((i & 1 ? o >> 16 : o & 0xffffu) + lane4);
                    }
                float r[DM];
                uint64_t flip = 0;
#pragma unroll
                for (int j = 0; j < DM; j++) {
                    const uint32_t c = wd[2 + j * EW] >> 16;
                    uint32_t mag = x[j][0], sg = x[j][0] ^ ((c < 32 ? (uint32_t)s : (uint32_t)(s >> 32)) << (31u - (c & 31u)));
#pragma unroll
                    for (int i = 1; i < RO; i++) {
                        mag = min_abs(mag, x[j][i]);
                        sg ^= x[j][i];
                    }
                    const float rr = al * __uint_as_float(mag & kMag);
                    r[j] = (uint32_t)j < deg ? __uint_as_float(mag_sign(__float_as_uint(rr), sg)) : 0.0f;
                    flip |= (uint32_t)j < deg ? 1ull << c : 0ull;
                }
                const float lam = __uint_as_float(wd[1]);
                float L = lam;
#pragma unroll
                for (int j = 0; j < DM; j++) {
                    float mu = lam;
#pragma unroll
                    for (int i = 0; i < DM; i++)
                        if (i != j) mu += r[i];
                    L += r[j];
                    if ((uint32_t)j < deg) {
                        satm = fmaxf(satm, fabsf(mu));
                        *lds_at((wd[2 + j * EW] & 0xffffu) + lane4) = __float_as_uint(Prec<float>::clamp(mu, lim));
                    }
                }
                satm = fmaxf(satm, fabsf(L));
                const bool one = L <= 0.0f;
                e |= one ? 1ull << v : 0ull;
                res ^= one ? flip : 0ull;
                if (want_post && ends) *lds_at(post0 + v * 256u + lane4) = __float_as_uint(Prec<float>::clamp(L, lim));
            }
            const bool met = act && res == 0, out = ends && !met;
            bool stop = false;
            if (limited && step % 8 == 7) {
                // M members precede this one at its next iteration
                const bool go_on = act && !met && !ends;
                const uint32_t at = go_on ? t : 0u;
                stop = converged_upto(cmask, at) + (uint32_t)__popcll(load_mask(&cmask[at + 1]) & lower) >= g.M && go_on;
            }
            const uint64_t done = __ballot(met || out || stop);
            if (done) {
                if (met) atomicOr(reinterpret_cast<unsigned long long*>(&cmask[t]), own);
                if ((done >> lane) & 1ull) {
                    conv = met;
                    e_conv = e;
                    satf = satm;
                    ran_out = out;
                }
                busy &= ~done;
                fin |= done;
            }
            t += (busy >> lane) & 1ull ? 1u : 0u;
        }
    }
}
