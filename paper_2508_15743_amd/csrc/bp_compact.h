// The item bodies of K1 with compact row states (FP32, serial or parallel
// schedule, slab in global memory, one shot per wavefront).  Included by
// bp.hip.  The serial one first; for the parallel one see FRow.
//
// The general body keeps every edge's suffix state (least magnitude and
// sign parity of the previous sweep's messages on the row's later edges) in
// the edge's own slab slot: the backward pass reads a message and writes a
// state, the sweep reads the state and writes a message, 16 bytes per edge
// and iteration.  But a row's suffix minimum only changes at a record, an
// edge whose message is smaller than all later ones of its row: about
// ln(d) + 0.6 edges of a row of degree d (5.5 of 131 on the d = 9 circuit
// graph).  So the state lives per check, in LDS beside the prefix state, and
// the backward pass stores per chunk a record of 16 words:
//   words 0-1   the signs of the chunk's 64 messages
//   words 2-3   which of them are records
//   words 4-15  for each record, in lane order, the row's least magnitude
//               over the later edges (what the state becomes once the sweep
//               has passed the edge)
// The sweep steps the check's state over each edge: the sign leaves the
// parity, and at a record the magnitude becomes the stored one.  8 bytes of
// messages and 2 of records per edge remain.
//
// A chunk with more than 12 records keeps the states in its slab slots, as
// in the general body, and says so by words 2-3 all ones.  Near the end of a
// sweep most edges are records, so from the member's group `dense0` on, all
// chunks keep them there and are loaded ahead like that.
//
// Chunks are handled in groups of four: a lane's four messages (and schedule
// words) lie together, so that every access of the slab, the records and the
// schedule moves 1 KB or 256 bytes at once.  Where the slabs of all resident
// wavefronts exceed the last-level cache, they are streamed past the caches
// that hold the schedule (DevGraph.cstream).
//
// Decisions: a column's decision is 0 almost always, so nothing is kept
// from sweep to sweep.  Each sweep starts its residual at the syndrome, and
// a chunk with a decision of 1 (one ballot) flips its columns' checks and
// stores the chunk's mask, from which the bitmap is formed when the run
// ends.  The syndrome enters as the initial parity of the prefix states.
// Unused slots work on a dummy check m, whose states stay 0.
//
// What bounds it, and what it measured, is stated at bp_compact_kernel.

constexpr uint32_t kMag = 0x7fffffffu;
constexpr uint32_t kCVals = 12;    // values of a chunk's record
constexpr uint32_t kCSch = 2048;   // bytes of a group in the compact schedule: meta[64][4], lambda[64][4]
constexpr uint32_t kCSlab = 1024;  // bytes of a group in the slab: [64][4]
constexpr uint32_t kCRec = 256;    // bytes of a group's records
constexpr int kStream = 2;         // cache policy of a streamed slab
constexpr int kCAhead = 4;         // groups loaded ahead

using u32x4 = __attribute__((ext_vector_type(4))) unsigned int;
using LdsWord = __attribute__((address_space(3))) uint32_t;

// The row states start at LDS address 0: these kernels have no static LDS.
__device__ __forceinline__ LdsWord* lds_at(uint32_t byte) { return (LdsWord*)(uintptr_t)byte; }

template <int AUX>
__device__ __forceinline__ u32x4 bload4(Rsrc r, uint32_t voff, uint32_t soff) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, AUX);
}
// A 16-byte store reads its data registers for some cycles after it issues:
// an instruction right behind it that writes them changed what was stored
// (seen: four lanes of each row of 16, where two wavefronts contend).  The
// compiler leaves the two wait states out where soffset is a register, so
// they are placed here, with the data kept until after them.
template <int AUX>
__device__ __forceinline__ void bstore4(u32x4 v, Rsrc r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)voff, (int)soff, AUX);
    asm volatile("s_nop 1" ::"v"(v));
}

// min(|a|, |b|) of two finite floats, as bits
__device__ __forceinline__ uint32_t min_abs(uint32_t a, uint32_t b) {
    uint32_t d;
    asm("v_min_f32 %0, |%1|, |%2|" : "=v"(d) : "v"(a), "v"(b));
    return d;
}

// magnitude of a, sign of b
__device__ __forceinline__ uint32_t mag_sign(uint32_t a, uint32_t b) {
    uint32_t d;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(d) : "v"(kMag), "v"(a), "v"(b));
    return d;
}

// a where bit BIT of mask is set, else 0
template <int BIT>
__device__ __forceinline__ float keep_if(uint32_t a, uint32_t mask) {
    uint32_t d;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(d) : "v"(mask), "n"(BIT));
    return __uint_as_float(a & d);
}

__device__ __forceinline__ uint32_t lane_rank(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint64_t lane_pair(uint32_t x, int lo) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)x, lo) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)x, lo + 1) << 32;
}

// Fields of the compact schedule's meta word
__device__ __forceinline__ uint32_t cm_row4(uint32_t meta) { return __builtin_amdgcn_ubfe(meta, 16u, 15u); }  // 4 c
__device__ __forceinline__ uint32_t cm_first4(uint32_t meta) { return meta & 0xfcu; }  // 4 * the column's first lane

struct CCtx {
    Rsrc sch;    // the member's compact schedule
    Rsrc osch;   // the member's chunk records (columns, initial states), addressed by
                 // lane offsets only: padding chunks lie past its end
    Rsrc slb;    // the block's slab: messages (states in dense chunks), then the records and
                 // the decision mask of each chunk
    Rsrc recs;   // where the sweep reads its records: the slab, or those of the initial messages
    uint32_t rec_at;              // offset of the records in recs
    uint32_t rec_slab, msk_slab;  // offsets of records and masks in the slab
    uint32_t pre;                 // LDS address of the prefix states (suffix states: 0)
    uint32_t f_old, f_new;        // flooding: LDS addresses of the rows' values
    uint32_t* res;                // residual s + H e, 32 checks a word
    float* post;
    float* trash;
    float al, lim;
    uint32_t lane, lane4, lane16;
};

// What a group needs of its four chunks, loaded ahead.
struct CStage {
    u32x4 meta, lam;
    uint32_t rec;  // word `lane` of the group's records
    u32x4 st;      // dense: the slots' states
    uint32_t v[4]; // only with posteriors
};

template <bool DENSE, bool POST, int NT>
__device__ __forceinline__ void cfetch(const CCtx& x, CStage& s, uint32_t g) {
    s.meta = bload4<0>(x.sch, x.lane16, g * kCSch);
    s.lam = bload4<0>(x.sch, x.lane16 + 1024u, g * kCSch);
    if constexpr (DENSE)
        s.st = bload4<NT>(x.slb, x.lane16, g * kCSlab);
    else
        s.rec = __builtin_amdgcn_raw_buffer_load_b32(x.recs, (int)x.lane4, (int)(x.rec_at + g * kCRec), NT);
    if constexpr (POST) {
#pragma unroll
        for (int j = 0; j < 4; j++) s.v[j] = bload<uint32_t>(x.osch, x.lane4 + kRecV + (g * 4 + j) * rec_bytes(false), 0);
    }
}

// A chunk's row states, as read from LDS, and its record's part.
struct CRow {
    uint32_t pre, suf, val;
    uint64_t sg, rc;
};

template <int J>
__device__ __forceinline__ void crecord(const CStage& s, CRow& w) {
    w.sg = lane_pair(s.rec, 16 * J);
    w.rc = lane_pair(s.rec, 16 * J + 2);
    w.val = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane_rank(w.rc) << 2) + 64u * J + 16u), (int)s.rec);
}

template <bool DENSE, int J>
__device__ __forceinline__ void crows(const CCtx& x, const CStage& s, CRow& w) {
    const uint32_t a = cm_row4(s.meta[J]);
    w.pre = *lds_at(a + x.pre);
    if constexpr (!DENSE) w.suf = *lds_at(a);
}

// The check messages of the lane's column: position q of the column is lane
// b0 + q.
template <int DC>
__device__ __forceinline__ void cgather(uint32_t meta, uint32_t r, uint32_t* rj) {
#pragma unroll
    for (int q = 0; q < DC; q++)
        rj[q] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(cm_first4(meta) + 4u * (uint32_t)q), (int)r);
}

// lambda_v + the column's other messages in ascending check order: bit 8 + q
// of meta says whether position q exists and is another lane (others add an
// exact zero)
template <int DC>
__device__ __forceinline__ float csum(uint32_t meta, uint32_t lam, const uint32_t* rj) {
    float mu = __uint_as_float(lam);
    mu += keep_if<8>(rj[0], meta);
    mu += keep_if<9>(rj[1], meta);
    mu += keep_if<10>(rj[2], meta);
    mu += keep_if<11>(rj[3], meta);
    mu += keep_if<12>(rj[4], meta);
    mu += keep_if<13>(rj[5], meta);
    if constexpr (DC > 6) {
        mu += keep_if<14>(rj[6], meta);
        mu += keep_if<15>(rj[7], meta);
    }
    return mu;
}

// What follows from a chunk's messages mu (not clamped) and r: posteriors,
// decisions, the residual and the saturation witness.
template <bool POST>
__device__ __forceinline__ void cdecide(const CCtx& x, uint32_t meta, uint32_t k, float mu, uint32_t r, uint32_t v,
                                        float& satm) {
    const bool last = (int32_t)meta < 0;      // the column's last lane
    const float L = mu + __uint_as_float(r);  // L_v there
    const float both = last ? L : mu;
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(satm) : "v"(mu), "v"(both));
    const uint64_t dec = __ballot(L <= 0.0f) & __ballot(last);
    if (dec) {
        // columns decided 1: flip their checks, keep the mask (a column's
        // bit is its last lane's)
        const uint32_t b0 = cm_first4(meta) >> 2, inc = (meta >> 8) & 0xffu;
        const uint32_t ll = b0 + 31u - (uint32_t)__clz((int)(inc | 1u << (x.lane - b0)));
        if ((inc || last) && ((dec >> ll) & 1ull)) {
            const uint32_t c = cm_row4(meta) >> 2;
            atomicXor(&x.res[c >> 5], 1u << (c & 31u));
        }
        if (x.lane == (k & 63u)) bstore<uint64_t>(dec, x.slb, 0u, x.msk_slab + k * 8u);
    }
    if constexpr (POST) {
        float* dst = last ? x.post + v : x.trash + x.lane;
        *dst = Prec<float>::clamp(L, x.lim);
    }
}

// Chunk J of group g (Algorithm 1, serial branch): the operations of
// sweep_chunk on every message, in the same order.  Its row states are in w
// and are replaced by those of the group's next chunk, which are read as
// soon as this chunk's are written; what does not feed the next chunk
// (decisions, saturation, posteriors) follows in that read's shadow.
template <int DC, bool DENSE, bool POST, int J>
__device__ __forceinline__ void csweep_chunk(const CCtx& x, const CStage& s, CRow& w, uint32_t g, bool first,
                                             u32x4& out, float& satm) {
    const uint32_t meta = s.meta[J], k = g * 4 + J;
    const uint32_t a = cm_row4(meta);
    uint32_t X;  // state of the row's later edges
    if constexpr (DENSE) {
        X = s.st[J];
    } else {
        const uint32_t mag = __builtin_amdgcn_inverse_ballot_w64(w.rc) ? w.val : w.suf;
        const uint32_t sgn = __builtin_amdgcn_inverse_ballot_w64(w.sg) ? ~kMag : 0u;
        X = mag_sign(mag, w.suf ^ sgn);
        asm("" : "+v"(X));
        if (w.rc == ~0ull) {  // more records than fit: the states are in the slots
            X = first ? bload<uint32_t>(x.osch, x.lane4 + rec_init(false) + k * rec_bytes(false), 0)
                      : bload<uint32_t>(x.slb, x.lane16 + 4u * J, g * kCSlab);
            // waited for here, so that the next groups' loads in flight are
            // not waited for where the paths join
            asm volatile("" : "+v"(X));
        }
        *lds_at(a) = X;
    }
    const uint32_t pre = w.pre;
    const float rr = x.al * __uint_as_float(min_abs(pre, X));
    const uint32_t r = mag_sign(__float_as_uint(rr), pre ^ X);
    uint32_t rj[8];
    cgather<DC>(meta, r, rj);
    if constexpr (!DENSE && J < 3) crecord<J + 1>(s, w);
    const float mu = csum<DC>(meta, s.lam[J], rj);
    const uint32_t mb = __float_as_uint(Prec<float>::clamp(mu, x.lim));
    *lds_at(a + x.pre) = mag_sign(min_abs(pre, mb), pre ^ mb);
    out[J] = mb;
    // the next chunk's reads follow this chunk's writes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (J < 3) crows<DENSE, J + 1>(x, s, w);
    __builtin_amdgcn_sched_barrier(0);
    cdecide<POST>(x, meta, k, mu, r, POST ? s.v[J] : 0u, satm);
    __builtin_amdgcn_sched_barrier(0);
}

template <int DC, bool DENSE, bool POST, int NT>
__device__ __forceinline__ void csweep_group(const CCtx& x, const CStage& s, uint32_t g, bool first, float& satm) {
    CRow w;
    u32x4 out;
    crows<DENSE, 0>(x, s, w);
    if constexpr (!DENSE) crecord<0>(s, w);
    csweep_chunk<DC, DENSE, POST, 0>(x, s, w, g, first, out, satm);
    csweep_chunk<DC, DENSE, POST, 1>(x, s, w, g, first, out, satm);
    csweep_chunk<DC, DENSE, POST, 2>(x, s, w, g, first, out, satm);
    csweep_chunk<DC, DENSE, POST, 3>(x, s, w, g, first, out, satm);
    bstore4<NT>(out, x.slb, x.lane16, g * kCSlab);
}

// Groups g0 .. g1-1 of the sweep (an even number), loaded A ahead.  The loop
// runs A groups without an exit between them: one would join paths in which
// different stages are the last loaded, and the compiler would wait for all
// of them at the loop's head.
template <int DC, bool DENSE, bool POST, int A, int NT>
__device__ __forceinline__ void csweep(const CCtx& x, uint32_t g0, uint32_t g1, bool first, float& satm) {
    if (g0 >= g1) return;
    CStage ring[A];
#pragma unroll
    for (int d = 0; d < A; d++) {
        cfetch<DENSE, POST, NT>(x, ring[d], min(g0 + d, g1 - 1));
        __builtin_amdgcn_sched_barrier(0);
    }
    uint32_t g = g0;
    for (; g + A <= g1; g += A) {
#pragma unroll
        for (int d = 0; d < A; d++) {
            csweep_group<DC, DENSE, POST, NT>(x, ring[d], g + d, first, satm);
            cfetch<DENSE, POST, NT>(x, ring[d], min(g + d + A, g1 - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (A > 2) {
#pragma unroll
        for (int d = 0; d < A - 2; d += 2) {
            if (g + d >= g1) break;
            csweep_group<DC, DENSE, POST, NT>(x, ring[d], g + d, first, satm);
            csweep_group<DC, DENSE, POST, NT>(x, ring[d + 1], g + d + 1, first, satm);
        }
    }
}

struct CBStage {
    u32x4 meta, msg;
};

template <int NT>
__device__ __forceinline__ void cbfetch(const CCtx& x, CBStage& s, uint32_t g) {
    s.meta = bload4<0>(x.sch, x.lane16, g * kCSch);
    s.msg = bload4<NT>(x.slb, x.lane16, g * kCSlab);
}

// Chunk J of group g in the backward pass: its messages join the states of
// their checks (run: those states; replaced by those of chunk J - 1), then
// its record goes to lanes 16 J .. 16 J + 15 of rec.
template <bool DENSE, int J>
__device__ __forceinline__ void cback_chunk(const CCtx& x, const CBStage& s, uint32_t& run, uint32_t g, u32x4& out,
                                            uint32_t& rec) {
    const uint32_t msg = s.msg[J], st = run;
    *lds_at(cm_row4(s.meta[J])) = mag_sign(min_abs(st, msg), st ^ msg);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (J > 0) run = *lds_at(cm_row4(s.meta[J > 0 ? J - 1 : 0]));
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (DENSE) {
        out[J] = st;
    } else {
        const uint64_t sg = __ballot((int32_t)msg < 0);
        uint64_t rc = __ballot(fabsf(__uint_as_float(msg)) < fabsf(__uint_as_float(st)));
        if (__popcll(rc) > (int)kCVals) {
            bstore<uint32_t>(st, x.slb, x.lane16 + 4u * J, g * kCSlab);
            rc = ~0ull;
        }
        // values to lanes 16 J + 4 and up in lane order, the others' to a
        // lane outside
        const uint32_t slot = (lane_rank(rc) << 2) + 64u * J + 16u;
        const uint32_t to = __builtin_amdgcn_inverse_ballot_w64(rc) ? slot : 64u * ((J + 2) % 4);
        uint32_t w = (uint32_t)__builtin_amdgcn_ds_permute((int)to, (int)(st & kMag));
        // (two wait states between the compares' scalar results and their use)
        asm("s_nop 1\n\t"
            "v_writelane_b32 %0, %1, %5\n\t"
            "v_writelane_b32 %0, %2, %6\n\t"
            "v_writelane_b32 %0, %3, %7\n\t"
            "v_writelane_b32 %0, %4, %8"
            : "+v"(w)
            : "s"((uint32_t)sg), "s"((uint32_t)(sg >> 32)), "s"((uint32_t)rc), "s"((uint32_t)(rc >> 32)), "n"(16 * J),
              "n"(16 * J + 1), "n"(16 * J + 2), "n"(16 * J + 3));
        rec = (x.lane >> 4) == J ? w : rec;
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <bool DENSE, int NT>
__device__ __forceinline__ void cback_group(const CCtx& x, const CBStage& s, uint32_t g) {
    u32x4 out;
    uint32_t rec = 0, run = *lds_at(cm_row4(s.meta[3]));
    cback_chunk<DENSE, 3>(x, s, run, g, out, rec);
    cback_chunk<DENSE, 2>(x, s, run, g, out, rec);
    cback_chunk<DENSE, 1>(x, s, run, g, out, rec);
    cback_chunk<DENSE, 0>(x, s, run, g, out, rec);
    if constexpr (DENSE)
        bstore4<NT>(out, x.slb, x.lane16, g * kCSlab);
    else
        __builtin_amdgcn_raw_buffer_store_b32(rec, x.slb, (int)x.lane4, (int)(x.rec_slab + g * kCRec), NT);
}

// Groups g1-1 .. g0 of the backward pass (an even number), loaded A ahead.
template <bool DENSE, int A, int NT>
__device__ __forceinline__ void cbackward(const CCtx& x, uint32_t g0, uint32_t g1) {
    if (g0 >= g1) return;
    const uint32_t cnt = g1 - g0;
    CBStage ring[A];
    auto at = [=](uint32_t e) { return e < cnt ? g1 - 1 - e : g0; };  // e groups from the end
#pragma unroll
    for (int d = 0; d < A; d++) {
        cbfetch<NT>(x, ring[d], uni(at(d)));
        __builtin_amdgcn_sched_barrier(0);
    }
    uint32_t e = 0;
    for (; e + A <= cnt; e += A) {
#pragma unroll
        for (int d = 0; d < A; d++) {
            cback_group<DENSE, NT>(x, ring[d], g1 - 1 - e - d);
            cbfetch<NT>(x, ring[d], at(e + d + A));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (A > 2) {
#pragma unroll
        for (int d = 0; d < A - 2; d += 2) {
            if (e + d >= cnt) break;
            cback_group<DENSE, NT>(x, ring[d], g1 - 1 - e - d);
            cback_group<DENSE, NT>(x, ring[d + 1], g1 - 2 - e - d);
        }
    }
}

// The parallel (flooding) schedule: every message of an iteration comes from
// the previous iteration's, so a check message needs its row's least and
// next least magnitude and the parity of all signs (Algorithm 1, parallel
// branch): the least magnitude of the others is the next least for the edge
// that has the least, and the least for all others.  The rows' values are
// two words of LDS per check, read for the previous iteration and formed
// for the next in the same pass; an edge's message stays in its slab slot.
// Row values: x.f_old, and x.f_old + x.pre; the next: x.f_new, likewise.
struct FRow {
    uint32_t o1, o2, n1, n2;
};

template <int J>
__device__ __forceinline__ void fold(const CCtx& x, const CStage& s, FRow& w) {
    const uint32_t a = cm_row4(s.meta[J]);
    w.o1 = *lds_at(a + x.f_old);
    w.o2 = *lds_at(a + x.f_old + x.pre);
}

template <int J>
__device__ __forceinline__ void fnew(const CCtx& x, const CStage& s, FRow& w) {
    const uint32_t a = cm_row4(s.meta[J]);
    w.n1 = *lds_at(a + x.f_new);
    w.n2 = *lds_at(a + x.f_new + x.pre);
}

template <int DC, bool POST, int J>
__device__ __forceinline__ void fsweep_chunk(const CCtx& x, const CStage& s, FRow& w, uint32_t g, bool first,
                                             u32x4& out, float& satm) {
    const uint32_t meta = s.meta[J], old = first ? s.lam[J] : s.st[J];
    const uint32_t mag = fabsf(__uint_as_float(old)) == fabsf(__uint_as_float(w.o1)) ? w.o2 : w.o1;
    const float rr = x.al * fabsf(__uint_as_float(mag));
    const uint32_t r = mag_sign(__float_as_uint(rr), w.o1 ^ old);
    uint32_t rj[8];
    cgather<DC>(meta, r, rj);
    if constexpr (J < 3) fold<J + 1>(x, s, w);
    const float mu = csum<DC>(meta, s.lam[J], rj);
    const uint32_t mb = __float_as_uint(Prec<float>::clamp(mu, x.lim)), a = cm_row4(meta);
    *lds_at(a + x.f_new) = mag_sign(min_abs(w.n1, mb), w.n1 ^ mb);
    *lds_at(a + x.f_new + x.pre) = __float_as_uint(
        __builtin_amdgcn_fmed3f(fabsf(__uint_as_float(w.n1)), __uint_as_float(w.n2), fabsf(__uint_as_float(mb))));
    out[J] = mb;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (J < 3) fnew<J + 1>(x, s, w);
    __builtin_amdgcn_sched_barrier(0);
    cdecide<POST>(x, meta, g * 4 + J, mu, r, POST ? s.v[J] : 0u, satm);
    __builtin_amdgcn_sched_barrier(0);
}

template <int DC, bool POST, int NT>
__device__ __forceinline__ void fsweep_group(const CCtx& x, const CStage& s, uint32_t g, bool first, float& satm) {
    FRow w;
    u32x4 out;
    fold<0>(x, s, w);
    fnew<0>(x, s, w);
    fsweep_chunk<DC, POST, 0>(x, s, w, g, first, out, satm);
    fsweep_chunk<DC, POST, 1>(x, s, w, g, first, out, satm);
    fsweep_chunk<DC, POST, 2>(x, s, w, g, first, out, satm);
    fsweep_chunk<DC, POST, 3>(x, s, w, g, first, out, satm);
    bstore4<NT>(out, x.slb, x.lane16, g * kCSlab);
}

// One iteration over ng groups (an even number), loaded A ahead as csweep
// (before the first one the slab's words are loaded but not used).
template <int DC, bool POST, int A, int NT>
__device__ __forceinline__ void fsweep(const CCtx& x, uint32_t ng, bool first, float& satm) {
    if (!ng) return;
    CStage ring[A];
#pragma unroll
    for (int d = 0; d < A; d++) {
        cfetch<true, POST, NT>(x, ring[d], min((uint32_t)d, ng - 1));
        __builtin_amdgcn_sched_barrier(0);
    }
    uint32_t g = 0;
    for (; g + A <= ng; g += A) {
#pragma unroll
        for (int d = 0; d < A; d++) {
            fsweep_group<DC, POST, NT>(x, ring[d], g + d, first, satm);
            cfetch<true, POST, NT>(x, ring[d], min(g + d + A, ng - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (A > 2) {
#pragma unroll
        for (int d = 0; d < A - 2; d += 2) {
            if (g + d >= ng) break;
            fsweep_group<DC, POST, NT>(x, ring[d], g + d, first, satm);
            fsweep_group<DC, POST, NT>(x, ring[d + 1], g + d + 1, first, satm);
        }
    }
}

// One work item, as run_item.  slb: the block's slab (bp_slab_elems words);
// post: its posteriors.
template <int DC, int NT, bool FLOOD = false>
__device__ __forceinline__ void run_item_c(const DevGraph& g, const BpLaunch& a, uint32_t item, unsigned char* lds,
                                           Rsrc slb, float* post) {
    CCtx x;
    const uint32_t lane = threadIdx.x;
    uint32_t* suf = reinterpret_cast<uint32_t*>(lds);
    uint32_t* pre = suf + g.m + 1;
    uint64_t* sb = reinterpret_cast<uint64_t*>(lds) + bp_compact_rows(g);
    uint64_t* res = sb + g.words_m;
    x.pre = 4u * (g.m + 1u);
    x.res = reinterpret_cast<uint32_t*>(res);
    x.slb = slb;
    x.rec_slab = g.cgroups * kCSlab;
    x.msk_slab = g.cgroups * (kCSlab + kCRec);
    x.post = post;
    x.trash = post + g.n;
    x.al = (float)g.alpha;
    x.lim = (float)g.clamp;
    x.lane = lane;
    x.lane4 = lane * 4u;
    x.lane16 = lane * 16u;
    const float* lamv = reinterpret_cast<const float*>(g.lam);

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

    uint64_t any = 0;
    for (uint32_t base = 0; base < g.m; base += kWave) {
        const uint32_t c = base + lane;
        const uint64_t mask = __ballot(c < g.m && s[c] != 0);
        if (lane == 0) sb[base / kWave] = mask;
        any |= mask;
    }
    if (a.use_M && preceding_converged(cmask, 1, mem, (int)lane) >= g.M) {
        if (lane == 0) a.t_conv[rec] = 0;
        return;
    }
    if (!any && a.fast_zero && g.all_lam_positive) {
        zero_item(g, a, shot, mem, (int)lane);
        return;
    }
    const uint32_t c0 = uni(g.member_chunk[mem]), nch = uni(g.member_chunk[mem + 1]) - c0;
    // groups of the member, of which gd .. ng-1 keep their states in the slab
    const uint32_t cg0 = uni(g.cgroup[mem]), ng = uni(g.cgroup[mem + 1]) - cg0, gd = FLOOD ? 0u : uni(g.dense0[mem]);
    x.sch = make_rsrc(g.csched + (size_t)cg0 * kCSch, ng * kCSch);
    x.osch = make_rsrc(g.sched + (size_t)c0 * rec_bytes(false), nch * rec_bytes(false));
    if constexpr (!FLOOD) {
        x.recs = make_rsrc(g.crec0 + (size_t)cg0 * kCRec, ng * kCRec);
        x.rec_at = 0;
        // the initial states of the dense groups.  Chunks past the member's
        // last read 0: the chunk is part of the lane's offset, which the
        // resource's size bounds; a scalar offset is outside that check
        for (uint32_t q = gd; q < ng; q++) {
            u32x4 st;
#pragma unroll
            for (int j = 0; j < 4; j++)
                st[j] = bload<uint32_t>(x.osch, x.lane4 + rec_init(false) + (q * 4 + j) * rec_bytes(false), 0);
            bstore4<0>(st, slb, x.lane16, q * kCSlab);
        }
    }
    float* post_out = a.post_out ? reinterpret_cast<float*>(a.post_out) + (size_t)rec * g.n : nullptr;
    // before the first sweep: all of the row's initial messages
    for (uint32_t c = lane; c <= g.m; c += kWave) {
        suf[c] = c < g.m ? g.crow0[c] : 0u;
        if constexpr (FLOOD) {
            const uint64_t w = c < g.m ? sb[c >> 6] : 0ull;
            suf[c] ^= ((uint32_t)(w >> (c & 63u)) & 1u) << 31;
            pre[c] = c < g.m ? g.crow2[c] : 0u;
        }
    }
    x.f_old = 0u;
    x.f_new = 2u * x.pre;

    uint32_t conv_t = 0, ran = 0;
    bool stopped = false;
    float satm = 0.0f;
    for (uint32_t t = 1; t <= a.T_run; t++) {
        if (a.use_M && t >= 2 && preceding_converged(cmask, t, mem, (int)lane) >= g.M) {
            stopped = true;
            break;
        }
        if (g.alpha_t) x.al = (float)g.alpha_t[t - 1];
        const bool want_post = post_out != nullptr || (a.accumulate_q && t == a.T_run);
        if (want_post)
            for (uint32_t v = lane; v < g.n; v += kWave) post[v] = lamv[v];
        // prefix states (flooding: the row values of the messages to come)
        for (uint32_t c = lane; c <= g.m; c += kWave) {
            const uint64_t w = c < g.m ? sb[c >> 6] : 0ull;
            const uint32_t none = c < g.m ? g.ident32 | ((uint32_t)(w >> (c & 63u)) & 1u) << 31 : 0u;
            if constexpr (FLOOD) {
                *lds_at(x.f_new + 4u * c) = none;
                *lds_at(x.f_new + x.pre + 4u * c) = none & kMag;
            } else {
                pre[c] = none;
            }
        }
        for (uint32_t w = lane; w < g.words_m; w += kWave) res[w] = sb[w];
        for (uint32_t k = lane; k < nch; k += kWave) bstore<uint64_t>(0ull, slb, k * 8u, x.msk_slab);
        __syncthreads();
        if constexpr (FLOOD) {
            if (want_post)
                fsweep<DC, true, kCAhead, NT>(x, ng, t == 1, satm);
            else
                fsweep<DC, false, kCAhead, NT>(x, ng, t == 1, satm);
            x.f_old = x.f_new;
            x.f_new = 2u * x.pre - x.f_old;
        } else if (want_post) {
            csweep<DC, false, true, kCAhead, NT>(x, 0, gd, t == 1, satm);
            csweep<DC, true, true, kCAhead, NT>(x, gd, ng, t == 1, satm);
        } else {
            csweep<DC, false, false, kCAhead, NT>(x, 0, gd, t == 1, satm);
            csweep<DC, true, false, kCAhead, NT>(x, gd, ng, t == 1, satm);
        }
        __syncthreads();
        if (post_out) {
            // post[v] was written by the lane that swept v: read it past the L1
            for (uint32_t v = lane; v < g.n; v += kWave)
                post_out[v] = __hip_atomic_load(&post[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        ran = t;
        bool nz = false;
        for (uint32_t w = lane; w < g.words_m; w += kWave) nz |= res[w] != 0;
        if (__ballot(nz) == 0) {
            if (!conv_t) conv_t = t;
            if (a.stop_on_converge) break;
        }
        if (!FLOOD && t < a.T_run) {
            for (uint32_t c = lane; c <= g.m; c += kWave) suf[c] = c < g.m ? g.ident32 : 0u;
            __syncthreads();
            cbackward<true, kCAhead, NT>(x, gd, ng);
            cbackward<false, kCAhead, NT>(x, 0, gd);
            x.recs = slb;
            x.rec_at = x.rec_slab;
            __syncthreads();
        }
    }
    // the decision bitmap of the last sweep, over the row states
    uint64_t* eb = reinterpret_cast<uint64_t*>(lds);
    if ((a.cand && (conv_t || !a.use_M)) || (a.weight && conv_t)) {
        __syncthreads();
        for (uint32_t w = lane; w < g.words_n; w += kWave) eb[w] = g.e0[w];
        __syncthreads();
        for (uint32_t k = lane; k < nch; k += kWave) {
            uint64_t mk = bload<uint64_t>(x.slb, k * 8u, x.msk_slab);  // stored by this lane
            while (mk) {
                const uint32_t q = (uint32_t)__ffsll((long long)mk) - 1u;
                mk &= mk - 1;
                const uint32_t v = bload<uint32_t>(x.osch, k * rec_bytes(false) + kRecV + 4u * q, 0);
                atomicOr(reinterpret_cast<unsigned long long*>(&eb[v >> 6]), 1ull << (v & 63u));
            }
        }
        __syncthreads();
    }
    finish_item<float>(g, a, shot, mem, conv_t, ran, stopped, __ballot(satm >= x.lim) != 0, eb, post, (int)lane);
}
