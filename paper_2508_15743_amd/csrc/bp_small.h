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
// The wavefront runs until each of its shots has converged or reached the
// iteration limit.  The correction limit is not looked at: among 64 shots
// some run to the limit in any case, and stopping a member that cannot be
// among the first M changes no result.  For the same reason every member
// without convergence adds its normalised posterior: the sum is only read
// for shots in which none converged.
//
// Bound by instruction issue, about 200 per column and 64 shots, scalar ones
// among them (0.45 us a column): d = 5 code capacity, 16 members, 20000 shots
// 832 us against 4.27 ms with one wavefront per shot and member.  Loading the
// next column's description during the current one's work gained nothing.

template <int RO, int DM>
__global__ __launch_bounds__(kWave) void bp_small_kernel(DevGraph g, BpLaunch a) {
    constexpr uint32_t EW = small_edge_words(RO), CWD = small_col_words(RO, DM);
    using CWord = const __attribute__((address_space(4))) uint32_t;
    const uint32_t lane = threadIdx.x, lane4 = lane * 4u;
    const uint32_t post0 = (g.E + 1u) * 256u;  // posteriors [v][lane] after the messages
    const uint32_t groups = (a.n_shots + kWave - 1) / kWave, n_items = groups * g.L;
    const float lim = (float)g.clamp;
    const float* lamv = reinterpret_cast<const float*>(g.lam);
    for (;;) {
        const uint32_t item = wave_ticket(a.counter, 1u);
        if (item >= n_items) break;
        const uint32_t mem = item / groups, shot = (item % groups) * kWave + lane;
        const bool act = shot < a.n_shots;
        uint64_t s = 0;
        if (act) {
            const uint8_t* sp = a.syndromes + (size_t)(a.shot0 + shot) * g.m;
            for (uint32_t c = 0; c < g.m; c++) s |= (uint64_t)(sp[c] != 0 ? 1u : 0u) << c;
        }
        CWord* cols = (CWord*)(g.ssched + (size_t)mem * g.scols * CWD);
        for (uint32_t q = 0; q < g.scols; q++) {
            CWord* w = cols + (size_t)q * CWD;
            const uint32_t deg = w[0] >> 8, lam = w[1];
#pragma unroll
            for (int j = 0; j < DM; j++)
                if ((uint32_t)j < deg) *lds_at((w[2 + j * EW] & 0xffffu) + lane4) = lam;
        }
        *lds_at(g.E * 256u + lane4) = g.ident32;
        // a zero syndrome with every lambda > 0 converges at once to e = 0
        const bool quick = s == 0 && a.fast_zero && g.all_lam_positive;
        uint32_t conv_t = quick ? 1u : 0u;
        uint64_t e_conv = 0;
        bool sat = false;
        float satm = 0.0f;
        uint64_t alive = __ballot(act && !quick);
        for (uint32_t t = 1; t <= a.T_run && alive; t++) {
            const float al = g.alpha_t ? (float)g.alpha_t[t - 1] : (float)g.alpha;
            const bool want_post = t == a.T_run;
            uint64_t e = g.e0[0], res = s;
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
                if (want_post) *lds_at(post0 + v * 256u + lane4) = __float_as_uint(Prec<float>::clamp(L, lim));
            }
            const bool met = ((alive >> lane) & 1ull) && res == 0;
            if (met) {
                conv_t = t;
                e_conv = e;
                sat = satm >= lim;
            }
            alive &= ~__ballot(met);
        }
        if (act) {
            if (!conv_t) sat = satm >= lim;
            const uint32_t rec = shot * g.L + mem;
            uint64_t* cmask = a.conv_mask + (size_t)shot * (kMaxT + 1);
            a.t_conv[rec] = (int32_t)conv_t;
            atomicAdd(&a.iters[shot], conv_t ? conv_t : a.T_run);
            if (sat) atomicOr(reinterpret_cast<unsigned long long*>(&cmask[0]), 1ull << mem);
            if (conv_t) {
                a.cand[rec] = e_conv;
                // W(e) = sum_v e_v lambda_v in FP64, ascending v (a column that
                // is 0 adds an exact zero)
                double W = 0.0;
                for (uint32_t v = 0; v < g.n; v++) W += (e_conv >> v) & 1ull ? g.lam64[v] : 0.0;
                a.weight[rec] = W;
                atomicOr(reinterpret_cast<unsigned long long*>(&cmask[conv_t]), 1ull << mem);
            } else {
                // the normalised posterior, as in finish_item; columns without
                // checks keep lambda
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
                        atomicAdd(reinterpret_cast<unsigned long long*>(&q[v]), (unsigned long long)llrint(post(v) * scale));
                }
            }
        }
        __syncthreads();
    }
}
