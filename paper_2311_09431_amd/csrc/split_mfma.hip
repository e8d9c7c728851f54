// Ring step for launches that leave most of the chip idle with 128-row workgroups (bf16 matrix cores,
// head dimension up to 128): same operands and products as fwd_mfma.hip and bwd_mfma.hip, other split
// of the work.
//
// What bounds such a launch is the walk of one workgroup.  Here a workgroup owns 32 rows and its
// wavefronts (8 forward, 4 backward) take every eighth (fourth) 32-row sub-tile of the streamed side; the
// partial results meet in LDS at the end.  That is four times the workgroups, and a fraction of the walk.
//
// A wavefront streams its sub-tiles by itself: stages of LDS that nobody else touches, filled by
// direct global -> LDS loads and ordered by its own vmcnt, no barrier before the end.  A sub-tile is read
// into registers as soon as it has landed and its stage requested anew, so that about 100 KiB are in
// flight on a compute unit all the time (64 KiB per 0.43 us with nothing but the loads, what its path to
// the L2 carries).  What is left is the number of instructions: with one wavefront per SIMD each takes
// its four cycles.
//
// Blocks shorter than one tile keep the precision of the fp32 kernels, which take them otherwise:
// EXACT.  Products of bf16 operands are exact in fp32 anyway; probabilities and dS go into theirs as
// three bf16 terms, and the exponents are formed with fp32's own rounding.
//
// The wavefront that takes a sub-tile is given by the sub-tile's place in the walk without emulated
// coarse skipping, so summation orders are fixed and the same under it.

#include "split_parts.h"

namespace sa {

namespace {

constexpr int FWD_WAVES = 8, BWD_WAVES = 4;
template <int DP> constexpr int SUB_BYTES = tile_bytes(DP) / 2;              // 32 rows
template <int DP> constexpr int PIECES = SUB_BYTES<DP> / 1024;               // loads of 1 KiB they take
template <int DP> constexpr int STAGE_BYTES = 2 * SUB_BYTES<DP>;             // of both streamed operands

// byte offset (global side) that this lane fetches of piece j of 32 rows
template <int DP>
__device__ inline uint32_t piece_offset(int j, int lane, int pitch, int d) {
    const int lr = lane >> 4, pc = lane & 15;
    int r = 4 * j + lr, chunk = pc ^ dt_swz(r);
    if (DP <= 64) {
        const int s = 4 * j + lr, x = pc ^ (((s & 1) << 2) | ((s >> 1) & 3));
        r = 2 * s + (x >> 3);
        chunk = x & 7;
    }
    return 8 * chunk < d ? r * pitch + (chunk << 4) : DT_OUT_OF_RANGE;
}

// what every kernel of this file keeps per lane
template <int DP>
struct Lane {
    int lane, n, h, wave;
    uint32_t arow[8], tr0[4], tr1[4];
    __device__ Lane() {
        lane = threadIdx.x & 63;
        n = lane & 31;
        h = lane >> 5;
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        dt_row_addrs<DP>(arow, n, h);
        dt_tr_addrs<DP>(tr0, tr1, lane);
    }
};

// 32 rows of a matrix from row `first` on, this wavefront's share of the pieces (rows beyond the
// matrix arrive as zeros)
template <int DP, int WAVES>
__device__ inline void load_own(dt_rsrc m, int first, int pitch, int d, char* lds, const Lane<DP>& ln) {
#pragma unroll
    for (int j = 0; j < PIECES<DP>; j += WAVES)
        if (PIECES<DP> % WAVES == 0 || j + ln.wave < PIECES<DP>)
            dt_load_piece(m, first * pitch, piece_offset<DP>(j + ln.wave, ln.lane, pitch, d), lds + (j + ln.wave) * 1024);
}
// their B operands
template <int DP, bool PART>
__device__ inline void read_own(bf16x8 (&f)[8], const char* rows, const Lane<DP>& ln, int part_ks) {
#pragma unroll
    for (int ks = 0; ks < ksteps_of(DP); ++ks) {
        const bf16x8 x = dt_read_row(rows, ln.arow[ks]);
        f[ks] = PART ? zero_beyond_d(x, ks == part_ks) : x;
    }
}

// The loads of a streamed sub-tile.  An instruction's immediate offset counts on both sides, so that the pieces
// of 16 rows share one setting of m0: the lane's offset of piece j is 1024 j less, and to keep it from
// getting negative the descriptor starts 4096 bytes ahead of the matrix.  (Each with an m0 of its own,
// the 16 loads of a sub-tile were 64 instructions.)
constexpr int AHEAD_BYTES = 4096;
__device__ inline dt_rsrc stream_rsrc(const void* matrix, int rows, int pitch, int d) {
    dt_rsrc r = dt_make_rsrc((const char*)matrix - AHEAD_BYTES, rows, pitch, d);
    r[2] += AHEAD_BYTES;
    return r;
}
template <int DP>
struct Loader {
    static constexpr int HALF = PIECES<DP> / 2;         // pieces of 16 rows
    uint32_t at[HALF];
    int pitch;
    __device__ Loader(int pitch_, int d, int lane) : pitch(pitch_) {
#pragma unroll
        for (int j = 0; j < HALF; ++j) {
            const uint32_t x = piece_offset<DP>(j, lane, pitch, d);
            at[j] = x == DT_OUT_OF_RANGE ? x : x + AHEAD_BYTES - 1024 * j;
        }
    }
    // 16 rows from row `row` on (the swizzle is the same for all such groups)
    __device__ inline void rows16(dt_rsrc m, int row, const char* to) const {
        const uint32_t dst = (uint32_t)reinterpret_cast<uintptr_t>((const lds_char_t*)to);
        const int byte = row * pitch;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
        if constexpr (HALF == 4)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                         "buffer_load_dwordx4 %1, %5, %6 offen lds\n\t"
                         "buffer_load_dwordx4 %2, %5, %6 offen offset:1024 lds\n\t"
                         "buffer_load_dwordx4 %3, %5, %6 offen offset:2048 lds\n\t"
                         "buffer_load_dwordx4 %4, %5, %6 offen offset:3072 lds"
                         :
                         : "s"(dst), "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "s"(m), "s"(byte)
                         : "memory", "m0");
        else
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                         "buffer_load_dwordx4 %1, %3, %4 offen lds\n\t"
                         "buffer_load_dwordx4 %2, %3, %4 offen offset:1024 lds"
                         :
                         : "s"(dst), "v"(at[0]), "v"(at[1]), "s"(m), "s"(byte)
                         : "memory", "m0");
#pragma clang diagnostic pop
    }
    // both operands' 32 rows, in four parts
    __device__ inline void part(int i, dt_rsrc a, dt_rsrc b, int row, const char* stage) const {
        rows16(i / 2 ? b : a, row + 16 * (i % 2), stage + i * (SUB_BYTES<DP> / 2));
    }
    __device__ inline void all(dt_rsrc a, dt_rsrc b, int row, const char* stage) const {
#pragma unroll
        for (int i = 0; i < 4; ++i) part(i, a, b, row, stage);
    }
};
template <int DP>
__device__ inline void read_rows(bf16x8 (&x)[8], const char* rows, const Lane<DP>& ln) {
#pragma unroll
    for (int ks = 0; ks < ksteps_of(DP); ++ks) x[ks] = dt_read_row(rows, ln.arow[ks]);
}
// operand i of 2 blocks_of(DP): 32-column block i % blocks_of(DP) of 16 of the rows
template <int DP>
__device__ inline void read_transposed(bf16x8 (&x)[8], int i, const char* rows, const Lane<DP>& ln) {
    const int g = i / blocks_of(DP), mb = i % blocks_of(DP);
    x[4 * g + mb] = dt_read_tr(rows + g * 16 * row_bytes(DP), ln.tr0[mb], ln.tr1[mb]);
}
// One step of a score product whose result vector instructions read.  Its operands may have been fetched
// from accumulation registers, which counts as a vector instruction; the wait states for that are
// always there (the product before takes longer).
template <bool PART, int DP>
__device__ __forceinline__ bf16x8 row_operand(bf16x8 a, int ks, int part_ks) {
    return PART && ks >= part_from(DP) ? zero_beyond_d(a, ks == part_ks) : a;
}
template <bool PART, int DP>
__device__ __forceinline__ void score_product(f32x16& acc, bf16x8 a, bf16x8 b, int ks, int part_ks) {
    const bf16x8 x = row_operand<PART, DP>(a, ks, part_ks);
    if (ks == 0) mfma_vgpr_first(acc, x, b, true);
    else mfma_vgpr_acc(acc, x, b, true);
}
// a weight tile as B operands, rounded to bf16 or (EXACT) as three terms
template <bool EXACT>
__device__ inline void as_operand(const f32x16& w, int g, bf16x8 (&b)[3]) {
    if (EXACT) {
        split_regs(w, 8 * g, b);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) b[0][e] = (__bf16)w[8 * g + e];
    }
}

// Backward, what makes a row odd: a score that is not finite (z: NaN then), or a dS that is not, which
// leaves no column of its sum finite.  (Elements of the operands reach one of the two; masked pairs
// have a dS of 0 * (dP - delta).)
__device__ inline void look_at(float (&z)[2], const f32x16& s) {
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r % 2] = fmaf(s[r], 0.f, z[r % 2]);
}
__device__ inline bool odd_sum(const float (&z)[2], const f32x16 (&ds_sum)[4]) {
    return z[0] + z[1] != 0.f || not_finite<1>(ds_sum);
}
// ------------------------------------------------------------------ forward
// Eight wavefronts, two to a SIMD: one's products run beside the other's vector instructions.  One stage each,
// which is requested anew when the sub-tile has been read into registers.
constexpr float RESCALE_SUM = 16777216.f;       // 2^24, see fwd_mfma.hip
// ROPE: the query rows are rotated by their position ids (d == DP).
template <int DP, bool PART, bool EXACT, bool ROPE = false>
__global__ void __launch_bounds__(64 * FWD_WAVES, 2)
fwd_split_kernel(StepArgs p, int n_tiles) {
    constexpr int MB = blocks_of(DP), KS = ksteps_of(DP), WAVES = FWD_WAVES;
    // the wavefronts' stages and the owned rows; at the end the statistics and partial results
    constexpr int TILES = WAVES * STAGE_BYTES<DP> > PARTIAL_BYTES<DP, WAVES> ? WAVES * STAGE_BYTES<DP> : PARTIAL_BYTES<DP, WAVES>;
    __shared__ __attribute__((aligned(1024))) char lds[TILES + SUB_BYTES<DP>];
    __shared__ float stats[WAVES * 64];                // [wave][m | l][32]
    __shared__ uint32_t masks[WAVES];
    __shared__ double rope_turns[ROPE ? DP / 2 : 1];

    const Lane<DP> ln;
    const int n = ln.n, h = ln.h;
    int rank, bh, dev_rank;
    decode((int)blockIdx.x, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * OWN, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int pitch = 2 * (int)p.kv_stride_s, own_pitch = 2 * (int)p.stride_s;

    const int a_own = q0 + n, a = min(a_own, p.c - 1);
    char* const own_rows = lds + TILES;
    char* const k = lds + ln.wave * STAGE_BYTES<DP>;
    char* const v = k + SUB_BYTES<DP>;
    load_own<DP, WAVES>(dt_make_rsrc((const __bf16*)p.q + base, p.c, own_pitch, d), q0, own_pitch, d, own_rows, ln);

    KeyCursor at(p, dev, q0, ln.wave);
    const Loader<DP> loader(pitch, d, ln.lane);
    dt_rsrc K = stream_rsrc((const __bf16*)p.k + kv_base, p.c, pitch, d);
    dt_rsrc V = stream_rsrc((const __bf16*)p.v + kv_base, p.c, pitch, d);
    int kv_loaded = at.kv, kv = 0, key0 = 0, shift = 0;
    // requests the next sub-tile
    auto request = [&]() {
        at.settle<WAVES>();
        kv = at.kv;
        key0 = 32 * at.v;
        shift = at.shift;
        if (kv == at.kv_end) return;
        if (kv != kv_loaded) {
            K = dt_advance(K, (kv - kv_loaded) * 2 * p.kv_shard);
            V = dt_advance(V, (kv - kv_loaded) * 2 * p.kv_shard);
            kv_loaded = kv;
        }
        loader.all(K, V, key0, k);
        at.v += WAVES;
    };
    at.enter<WAVES>();
    request();

    float* L = p.lse + b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c + a;
    const Scale2 kappa(p.scale);
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    float m = -INFINITY, l = 0.f;           // m in base-2 units; l: this half-wave's share of the row sum
    f32x16 acc[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acc[mb] = zero16();
    // as in fwd_mfma.hip: a walk over striped shards sets its references anew at each
    const bool rebase_shards = !EXACT && p.n_kv > 1 && p.layout == SA_STRIPED;
    int kv_before = -1;

    int position = 0;
    if (ROPE) {
        position = p.q_pos[b * p.pos_stride_b + a];
        fill_rope_turns<DP>(rope_turns, threadIdx.x, p.rope_log2_base);
        wait_lds();
    }
    wait_all_but<0>();
    __builtin_amdgcn_s_barrier();
    bf16x8 qf[8];
    read_own<DP, PART>(qf, own_rows, ln, part_ks);
    if (ROPE) rope_rotate<DP>(qf, rope_turns, position, h);
    while (kv < at.kv_end) {
        wait_all_but<0>();
        bf16x8 kr[8], vt[8];
        read_rows<DP>(kr, k, ln);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * MB; ++i) read_transposed<DP>(vt, i, v, ln);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 x;
        // the first two products only need half of the rows: the other reads meanwhile
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) score_product<PART, DP>(x, kr[ks], qf[ks], ks, part_ks);
        __builtin_amdgcn_sched_barrier(0);
        wait_lds();
        const bool masked = key0 + 31 > min(p.c - 1, q0 + shift);          // some pair of the sub-tile is
        const int lane_last = min(p.c - 1, a_own + shift) - key0;
        const bool rebase = rebase_shards && kv != kv_before;
        kv_before = kv;
        request();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 2; ks < KS; ++ks) score_product<PART, DP>(x, kr[ks], qf[ks], ks, part_ks);
        mfma_results_to_valu(x);
        if (masked) {
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = reg_row(r, h) <= lane_last ? x[r] : -INFINITY;
        }
        auto highest = [&]() {
            float mx[2] = {x[0], x[1]};
#pragma unroll
            for (int r = 2; r < 16; ++r) mx[r % 2] = fmaxf(mx[r % 2], x[r]);
            return half_wave_max(fmaxf(mx[0], mx[1])) * kappa.hi;
        };
        auto rescale = [&](float alpha) {
            l *= alpha;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mb][r] *= alpha;
        };
        float sum[2] = {0.f, 0.f};
        if (EXACT) {
            const float m_new = fmaxf(m, highest());
            const float ref = m_new == -INFINITY ? 0.f : m_new;                 // a row without a key so far
            if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) rescale(__builtin_amdgcn_exp2f(m - ref));
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                x[r] = kappa.exp2(x[r], ref, 0.f);
                sum[r % 2] += x[r];
            }
            m = m_new;
        } else {
            // the reference moves when it has to, as in fwd_mfma.hip
            f32x16 pr;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                pr[r] = __builtin_amdgcn_exp2f(fmaf(x[r], kappa.hi, -m));
                sum[r % 2] += pr[r];
            }
            if (rebase || __builtin_amdgcn_ballot_w64(!(sum[0] + sum[1] < RESCALE_SUM)) != 0) {
                const float mx = highest();
                float m_new = fmaxf(m, mx);
                if (rebase && mx != -INFINITY)
                    m_new = fmaxf(mx, m + __builtin_amdgcn_logf(half_wave_sum(l) * (1.f / RESCALE_SUM)));
                const float ref = m_new == -INFINITY ? 0.f : m_new;
                rescale(__builtin_amdgcn_exp2f(m - ref));
                m = m_new;
                sum[0] = sum[1] = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    pr[r] = __builtin_amdgcn_exp2f(fmaf(x[r], kappa.hi, -ref));
                    sum[r % 2] += pr[r];
                }
            }
            x = pr;
        }
        l += sum[0] + sum[1];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            bf16x8 w[3];
            as_operand<EXACT>(x, g, w);
#pragma unroll
            for (int t = EXACT ? 2 : 0; t >= 0; --t)          // smallest terms first
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb] = mfma(vt[4 * g + mb], w[t], acc[mb]);
        }
    }

    const uint32_t odd_rows = fold_forward<DP, WAVES, EXACT, false>(p, acc, m, l, lds, stats, masks, ln, dev, a_own, a, L,
                                                             p.o + base + (int64_t)a * p.stride_s);
    if (EXACT) each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { fwd_row<__hip_bfloat16>(again, b, hd, dev_i, q0 + i, ln.lane); });
}

// ----------------------------------------------------------------- backward
// One wavefront per SIMD (the key-owning side's registers), so what overlaps is arranged by hand: a
// product leaves room for five or six other instructions.  In sub-tile u:
//     S(u)      beside the transposing reads of u
//     dP(u)     beside the exponentials of S(u), and the first requests of u + 2
//     dQ (or dV and dK) += ...(u)   beside dS(u), the other requests and the row reads of u + 1
// Products whose result vector instructions read go through asm forms, which keep it out of the
// accumulation registers (the owned operands are pinned to those, which the streamed ones leave
// free).  What the compiler's hazard recogniser cannot see (mfma_tiles.h) is kept by the order: vector
// instructions on S start behind the second product of dP, those on dP behind the second product
// that follows its last.
template <bool PART, int DP>
__device__ __forceinline__ void score_product_own(f32x16& acc, bf16x8 a, bf16x8 own, int ks, int part_ks) {
    const bf16x8 x = row_operand<PART, DP>(a, ks, part_ks);
    if (PART && ks >= part_from(DP)) {          // a vector select before it
        if (ks == 0) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(x), "a"(own));
        else asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(x), "a"(own));
        return;
    }
    if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(x), "a"(own));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(x), "a"(own));
}
// the same with other start values than zero
template <bool PART, int DP>
__device__ __forceinline__ void score_product_from(f32x16& acc, const f32x16& start, bf16x8 a, bf16x8 own, int part_ks) {
    const bf16x8 x = row_operand<PART, DP>(a, 0, part_ks);
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(acc) : "v"(x), "a"(own), "v"(start));
}
__device__ inline bf16x8 negated(bf16x8 x) {
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(bf16x8, __builtin_bit_cast(i32x4, x) ^ (int)0x80008000);
}

// dQ: a workgroup owns queries
template <int DP, bool PART, bool EXACT>
__device__ inline void bwd_dq(const StepArgs& p, int n_tiles, int linear, char* lds, char* stats, uint32_t* masks) {
    constexpr int KS = ksteps_of(DP), MB = blocks_of(DP), WAVES = BWD_WAVES, LOADS = 2 * PIECES<DP>, TERMS = EXACT ? 3 : 1;
    constexpr int LATE = KS > 2 ? KS - 2 : KS / 2, NEXT = MB > 1 ? 1 : 0;          // (32 columns: two k-steps, one block)
    const Lane<DP> ln;
    const int n = ln.n, h = ln.h;
    int rank, bh, dev_rank;
    decode_near(linear, n_tiles * p.n_q, p.B * p.H, uneven(p), rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * OWN, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c;
    const int pitch = 2 * (int)p.kv_stride_s, own_pitch = 2 * (int)p.stride_s;

    const int a_own = q0 + n, a = min(a_own, p.c - 1);
    char* const own_rows = lds + WAVES * 2 * STAGE_BYTES<DP>;
    load_own<DP, WAVES>(dt_make_rsrc((const __bf16*)p.q + base, p.c, own_pitch, d), q0, own_pitch, d, own_rows, ln);
    load_own<DP, WAVES>(dt_make_rsrc((const __bf16*)p.dout + base, p.c, own_pitch, d), q0, own_pitch, d, own_rows + SUB_BYTES<DP>, ln);
    char* const own_stats = stats + ln.wave * 2 * STAT_BYTES;       // every wavefront has its own
    load_stat(dt_make_rsrc(p.lse + sbase, p.c, 4, 2), q0, own_stats, ln.lane);
    load_stat(dt_make_rsrc(p.delta + sbase, p.c, 4, 2), q0, own_stats + 256, ln.lane);

    KeyCursor at(p, dev, q0, ln.wave);
    const Loader<DP> loader(pitch, d, ln.lane);
    char* const tiles = lds + ln.wave * 2 * STAGE_BYTES<DP>;
    dt_rsrc K = stream_rsrc((const __bf16*)p.k + kv_base, p.c, pitch, d);
    dt_rsrc V = stream_rsrc((const __bf16*)p.v + kv_base, p.c, pitch, d);
    int kv_at = at.kv;
    // (behind the walk's end: rows beyond the matrix, whose loads deliver zeros without a look at memory)
    const int beyond = 32 * at.n_full;
    struct Tile { int key0, shift; };               // key0 == beyond: none
    // the walk's next sub-tile; K, V: of its block
    auto take = [&](Tile& t) {
        at.settle<WAVES>();
        t.key0 = at.kv < at.kv_end ? 32 * at.v : beyond;
        t.shift = at.shift;
        at.v += WAVES;
        if (at.kv != kv_at) {
            K = dt_advance(K, (at.kv - kv_at) * 2 * p.kv_shard);
            V = dt_advance(V, (at.kv - kv_at) * 2 * p.kv_shard);
            kv_at = at.kv;
        }
    };
    Tile t0, t1 = {beyond, 0}, t2;
    at.enter<WAVES>();
#pragma unroll 1
    for (int i = 0; i < 2; ++i) {
        t0 = t1;
        take(t1);
        loader.all(K, V, t1.key0, tiles + i * STAGE_BYTES<DP>);
    }
    const Scale2 kappa(p.scale);
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    f32x16 acc[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acc[mb] = zero16();
    wait_all_but<2 * LOADS>();
    __builtin_amdgcn_s_barrier();
    bf16x8 qf[8], gf[8], kr[8], vr[8];
    read_own<DP, PART>(qf, own_rows, ln, part_ks);
    read_own<DP, PART>(gf, own_rows + SUB_BYTES<DP>, ln, part_ks);
    float lse2, lse2_lo;
    to_base2(reinterpret_cast<const float*>(own_stats)[n], lse2, lse2_lo);
    f32x16 neg_delta;           // dP starts from it
#pragma unroll
    for (int r = 0; r < 16; ++r) neg_delta[r] = -reinterpret_cast<const float*>(own_stats)[64 + n];
    float z[2] = {0.f, 0.f};
    wait_all_but<LOADS>();
    read_rows<DP>(kr, tiles, ln);
    read_rows<DP>(vr, tiles + SUB_BYTES<DP>, ln);
    for (int stage = 0; t0.key0 != beyond; stage ^= 1) {
        char* const k = tiles + stage * STAGE_BYTES<DP>;
        const char* const k_next = tiles + (stage ^ 1) * STAGE_BYTES<DP>;
        bf16x8 kt[8];
        f32x16 s, dp, pr;
        take(t2);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            __builtin_amdgcn_sched_barrier(0);
            score_product_own<PART, DP>(s, kr[ks], qf[ks], ks, part_ks);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 2 * MB * ks / KS; i < 2 * MB * (ks + 1) / KS; ++i) read_transposed<DP>(kt, i, k, ln);
        }
        constexpr int EACH = (16 + KS - 2) / (KS - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 0) score_product_from<PART, DP>(dp, neg_delta, vr[0], gf[0], part_ks);
            else score_product_own<PART, DP>(dp, vr[ks], gf[ks], ks, part_ks);
            __builtin_amdgcn_sched_barrier(0);
            if (ks >= 1) {
#pragma unroll
                for (int r = (ks - 1) * EACH; r < min(16, ks * EACH); ++r)
                    pr[r] = EXACT ? kappa.exp2(s[r], lse2, lse2_lo) : __builtin_amdgcn_exp2f(fmaf(s[r], kappa.hi, -lse2));
            }
            if (ks == KS / 2) wait_lds();           // the stage's last reads
            if (ks == KS / 2) loader.part(0, K, V, t2.key0, k);
            if (ks == LATE) loader.part(1, K, V, t2.key0, k);
        }
        asm volatile("" : "+v"(pr));            // there, beside the products
        __builtin_amdgcn_sched_barrier(0);
        if (t0.key0 + 31 > min(p.c - 1, q0 + t0.shift)) {          // some pair of the sub-tile is masked
            const int lane_last = min(p.c - 1, a_own + t0.shift) - t0.key0;
#pragma unroll
            for (int r = 0; r < 16; ++r) pr[r] = reg_row(r, h) <= lane_last ? pr[r] : 0.f;
        }
        if (EXACT) look_at(z, s);
        mfma_results_to_valu(dp);
        bf16x8 w[2][3];
#pragma unroll
        for (int r = 0; r < 8; ++r) pr[r] *= dp[r];
        as_operand<EXACT>(pr, 0, w[0]);
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int t = TERMS - 1; t >= 0; --t)          // smallest terms first
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    __builtin_amdgcn_sched_barrier(0);
                    acc[mb] = mfma(kt[4 * g + mb], w[g][t], acc[mb]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (t != TERMS - 1) continue;
                    if (g == 0 && mb == 0) {
#pragma unroll
                        for (int r = 8; r < 16; ++r) pr[r] *= dp[r];
                        as_operand<EXACT>(pr, 1, w[1]);
                    }
                    if (g == 0 && mb == MB - 1) loader.part(2, K, V, t2.key0, k);
                    if (g == 1 && mb == 0) {
                        loader.part(3, K, V, t2.key0, k);
                        wait_all_but<LOADS>();
                        read_rows<DP>(kr, k_next, ln);
                    }
                    if (g == 1 && mb == NEXT) read_rows<DP>(vr, k_next + SUB_BYTES<DP>, ln);
                }
        __builtin_amdgcn_sched_barrier(0);
        t0 = t1;
        t1 = t2;
    }
    wait_all_but<0>();

    float* const DQ = p.dq + base + (int64_t)a * p.stride_s;
    float4 old[MB];
    load_old<DP, WAVES>(old, DQ, d, !p.fresh && a_own < p.c, ln);
    __syncthreads();
    put_partial<DP>(lds, acc, ln);
    if (EXACT) put_odd(masks, a_own < p.c && odd_sum(z, acc), ln.wave, ln.lane);
    __syncthreads();
    const uint32_t odd_rows = EXACT ? take_odd<WAVES>(masks) : 0;
    if (a_own < p.c && !((odd_rows >> n) & 1))
        add_rows<DP, WAVES>(DQ, old, lds, p.scale, d, ln);
    if (EXACT) each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { dq_row<__hip_bfloat16>(again, b, hd, dev_i, q0 + i, ln.lane); });
}

// dK, dV: owned rows are keys, the streamed ones queries with their LSE and delta beside them; the query heads
// that share the key/value head and the query shards that see it come one after the other.  The owned V is
// negated, so that delta - dP comes out of the product that starts from delta; dK changes its sign
// at the end.
template <int DP, bool PART, bool EXACT>
__device__ inline void bwd_dkdv(const StepArgs& p, int n_tiles, int linear, char* lds, char* stats, uint32_t* masks) {
    constexpr int KS = ksteps_of(DP), MB = blocks_of(DP), WAVES = BWD_WAVES, LOADS = 2 * PIECES<DP> + 2, TERMS = EXACT ? 3 : 1;
    constexpr int LATE = KS > 2 ? KS - 2 : KS / 2, NEXT = MB > 1 ? 1 : 0;          // as in bwd_dq
    const Lane<DP> ln;
    const int n = ln.n, h = ln.h, wave = ln.wave;
    int tile, bh, dev_i;                                // low key tiles see most queries: first
    decode_near(linear, n_tiles * p.n_kv, p.B * p.H_kv, uneven(p), tile, bh);
    decode_rank(tile, n_tiles, p.n_kv, p.layout, tile, dev_i);
    const int k0 = tile * OWN, dev = p.kv_dev + dev_i;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv, group = p.H / p.H_kv, d = p.d;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + dev_i * p.kv_shard;
    const int pitch = 2 * (int)p.stride_s, own_pitch = 2 * (int)p.kv_stride_s;

    const int key_own = k0 + n, key = min(key_own, p.c - 1);
    const int64_t row = kv_base + (int64_t)key * p.kv_stride_s;
    char* const own_rows = lds + WAVES * 2 * STAGE_BYTES<DP>;
    load_own<DP, WAVES>(dt_make_rsrc((const __bf16*)p.k + kv_base, p.c, own_pitch, d), k0, own_pitch, d, own_rows, ln);
    load_own<DP, WAVES>(dt_make_rsrc((const __bf16*)p.v + kv_base, p.c, own_pitch, d), k0, own_pitch, d, own_rows + SUB_BYTES<DP>, ln);

    // Blocks: the members of the group, each with the query shards that see the keys.  Of a block this
    // wavefront takes the sub-tiles of 32 queries whose number less k0 / 32 (full blocks: whose number) is
    // wave - turn modulo 4, turn counting the sub-tiles of the blocks before.
    const Loader<DP> loader(pitch, d, ln.lane);
    char* const tiles = lds + wave * 2 * STAGE_BYTES<DP>;
    char* const tile_stats = stats + wave * 2 * STAT_BYTES;
    const int q_dev0 = p.layout == SA_STRIPED ? p.q_dev : max(p.q_dev, dev), q_end = p.q_dev + p.n_q;
    const int n_sub = (p.c + 31) / 32;
    int member = q_dev0 < q_end ? 0 : group, q_dev = q_dev0, v = 0, turn = 0;
    int shift = 0;              // key b is seen by the block's queries from b + shift on
    dt_rsrc Q, G, S, E;
    auto enter = [&]() {
        const bool full = block_kind(q_dev, dev, p.layout) == MASK_FULL;
        const int off = block_off(q_dev, dev, p.layout), fine = full ? 0 : k0 / 32;
        // first query a workgroup of these keys looks at (emulated coarse skipping: from the first
        // skip_bq-tall tile that shares an allowed pair with the keys' skip_bk-wide one)
        int first = fine;
        if (!full && p.skip_bq > 0) first = (k0 / p.skip_bk * p.skip_bk + off) / p.skip_bq * p.skip_bq / 32;
        v = first + ((fine + wave - turn - first) & (WAVES - 1));
        turn += n_sub - fine;
        shift = full ? -(p.c + OWN) : off;
        const int hd = kvh * group + member;
        const int64_t base = b * p.stride_b + hd * p.stride_h + (q_dev - p.q_dev) * p.q_shard;
        const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(q_dev - p.q_dev) * p.c;
        Q = stream_rsrc((const __bf16*)p.q + base, p.c, pitch, d);
        G = stream_rsrc((const __bf16*)p.dout + base, p.c, pitch, d);
        S = dt_make_rsrc(p.lse + sbase, p.c, 4, 2);
        E = dt_make_rsrc(p.delta + sbase, p.c, 4, 2);
    };
    const int beyond = 32 * n_sub;             // behind the walk's end, as above
    struct Tile { int a0, shift; };            // a0 == beyond: none
    // the walk's next sub-tile; Q, G, S, E: of its block
    auto take = [&](Tile& t) {
        while (v >= n_sub && member < group) {
            if (++q_dev >= q_end) {
                q_dev = q_dev0;
                ++member;
            }
            if (member < group) enter();
        }
        t.a0 = member < group ? 32 * v : beyond;
        t.shift = shift;
        v += WAVES;
    };
    auto load_stats = [&](const Tile& t, int stage) {
        load_stat(S, t.a0, tile_stats + stage * STAT_BYTES, ln.lane);
        load_stat(E, t.a0, tile_stats + stage * STAT_BYTES + 256, ln.lane);
    };
    enter();
    Tile t0, t1 = {beyond, 0}, t2;
#pragma unroll 1
    for (int i = 0; i < 2; ++i) {
        t0 = t1;
        take(t1);
        loader.all(Q, G, t1.a0, tiles + i * STAGE_BYTES<DP>);
        load_stats(t1, i);
    }
    const Scale2 kappa(p.scale);
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    f32x16 acck[4], accv[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acck[mb] = accv[mb] = zero16();
    wait_all_but<2 * LOADS>();
    __builtin_amdgcn_s_barrier();
    bf16x8 kf[8], vf[8], qr[8], gr[8];
    read_own<DP, PART>(kf, own_rows, ln, part_ks);
    read_own<DP, PART>(vf, own_rows + SUB_BYTES<DP>, ln, part_ks);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) vf[ks] = negated(vf[ks]);
    // LSE (in base-2 units unless EXACT) and delta of this lane's registers' rows.  The 32 LSE of a sub-tile are
    // scaled where they lie, by one instruction on one of each lane instead of one on each of 16.
    f32x16 lse, delta;
    float raw;
    auto read_next = [&](int stage) {
        if (!EXACT) raw = reinterpret_cast<const float*>(tile_stats + stage * STAT_BYTES)[ln.lane];
        read_rows<DP>(qr, tiles + stage * STAGE_BYTES<DP>, ln);
        read_rows<DP>(gr, tiles + stage * STAGE_BYTES<DP> + SUB_BYTES<DP>, ln);
    };
    float z[2] = {0.f, 0.f};
    wait_all_but<LOADS>();
    read_next(0);
    for (int stage = 0; t0.a0 != beyond; stage ^= 1) {
        char* const q = tiles + stage * STAGE_BYTES<DP>;
        char* const g = q + SUB_BYTES<DP>;
        char* const stat = tile_stats + stage * STAT_BYTES;
        bf16x8 gt[8], qt[8];
        f32x16 s, dp, pr, ds;
        if (!EXACT) reinterpret_cast<float*>(stat)[ln.lane] = raw * LOG2E;         // (lanes 32 .. 63: nobody's)
        take(t2);
        // LDS reads: delta, LSE, transposed operands of dO and of Q
        constexpr int READS = 8 + 4 * MB;
        auto read = [&](int i) {
            if (i < 8) {
                const float4 y = *reinterpret_cast<const float4*>(stat + (i < 4 ? 256 : 0) + 4 * (8 * (i % 4) + 4 * h));
                f32x16& x = i < 4 ? delta : lse;
                const int r = 4 * (i % 4);
                x[r] = y.x; x[r + 1] = y.y; x[r + 2] = y.z; x[r + 3] = y.w;
            } else if (i < 8 + 2 * MB) {
                read_transposed<DP>(gt, i - 8, g, ln);
            } else {
                read_transposed<DP>(qt, i - 8 - 2 * MB, q, ln);
            }
        };
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            __builtin_amdgcn_sched_barrier(0);
            score_product_own<PART, DP>(s, qr[ks], kf[ks], ks, part_ks);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = READS * ks / KS; i < READS * (ks + 1) / KS; ++i) read(i);
        }
        constexpr int EACH = (16 + KS - 2) / (KS - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 0) score_product_from<PART, DP>(dp, delta, gr[0], vf[0], part_ks);
            else score_product_own<PART, DP>(dp, gr[ks], vf[ks], ks, part_ks);
            __builtin_amdgcn_sched_barrier(0);
            if (ks >= 1) {
#pragma unroll
                for (int r = (ks - 1) * EACH; r < min(16, ks * EACH); ++r) {
                    if (EXACT) {
                        float hi, lo;
                        to_base2(lse[r], hi, lo);
                        pr[r] = kappa.exp2(s[r], hi, lo);
                    } else {
                        pr[r] = __builtin_amdgcn_exp2f(fmaf(s[r], kappa.hi, -lse[r]));
                    }
                }
            }
            if (ks == KS / 2) wait_lds();           // the stage's last reads
            if (ks == KS / 2) loader.part(0, Q, G, t2.a0, q);
            if (ks == LATE) loader.part(1, Q, G, t2.a0, q);
        }
        asm volatile("" : "+v"(pr));            // there, beside the products
        __builtin_amdgcn_sched_barrier(0);
        if (t0.a0 < k0 + OWN - 1 + t0.shift || t0.a0 + 32 > p.c) {       // some pair of the sub-tile is masked
            const int lane_first = key_own + t0.shift - t0.a0, rows = p.c - t0.a0;
#pragma unroll
            for (int r = 0; r < 16; ++r) pr[r] = reg_row(r, h) >= lane_first && reg_row(r, h) < rows ? pr[r] : 0.f;
        }
        if (EXACT) look_at(z, s);
        bf16x8 wp[2][3], wd[2][3];
        as_operand<EXACT>(pr, 0, wp[0]);
        // dV over the first 16 rows, dK over them, dV and dK over the other 16
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = TERMS - 1; t >= 0; --t)          // smallest terms first
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (i % 2 == 0) accv[mb] = mfma(gt[4 * (i / 2) + mb], wp[i / 2][t], accv[mb]);
                    else acck[mb] = mfma(qt[4 * (i / 2) + mb], wd[i / 2][t], acck[mb]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (t != TERMS - 1) continue;
                    // beside each of the first rounds something else
                    if (i == 0 && mb == NEXT) {
                        if (MB > 1) asm volatile("" : "+v"(dp));
                        else mfma_results_to_valu(dp);          // (one product behind its last)
#pragma unroll
                        for (int r = 0; r < 8; ++r) ds[r] = pr[r] * dp[r];
                        as_operand<EXACT>(ds, 0, wd[0]);
                    }
                    if (i == 0 && mb == MB - 1) as_operand<EXACT>(pr, 1, wp[1]);
                    if (i == 1 && mb == 0) loader.part(2, Q, G, t2.a0, q);
                    if (i == 1 && mb == NEXT) loader.part(3, Q, G, t2.a0, q);
                    if (i == 1 && mb == MB - 1) {
#pragma unroll
                        for (int r = 8; r < 16; ++r) ds[r] = pr[r] * dp[r];
                        as_operand<EXACT>(ds, 1, wd[1]);
                    }
                    if (i == 2 && mb == 0) load_stats(t2, stage);
                    if (i == 3 && mb == 0) {
                        wait_all_but<LOADS>();
                        read_next(stage ^ 1);
                    }
                }
        __builtin_amdgcn_sched_barrier(0);
        t0 = t1;
        t1 = t2;
    }
    wait_all_but<0>();

    constexpr int HALF = PARTIAL_BYTES<DP, WAVES>;
    static_assert(2 * HALF <= WAVES * 2 * STAGE_BYTES<DP>, "partial results");
    float4 old_v[MB], old_k[MB];
    load_old<DP, WAVES>(old_v, p.dv + row, d, !p.fresh && key_own < p.c, ln);
    load_old<DP, WAVES>(old_k, p.dk + row, d, !p.fresh && key_own < p.c, ln);
    __syncthreads();
    put_partial<DP>(lds, accv, ln);
    put_partial<DP>(lds + HALF, acck, ln);
    if (EXACT) put_odd(masks, key_own < p.c && odd_sum(z, acck), ln.wave, ln.lane);
    __syncthreads();
    const uint32_t odd_rows = EXACT ? take_odd<WAVES>(masks) : 0;
    if (key_own < p.c && !((odd_rows >> n) & 1)) {
        add_rows<DP, WAVES>(p.dv + row, old_v, lds, 1.f, d, ln);
        add_rows<DP, WAVES>(p.dk + row, old_k, lds + HALF, -p.scale, d, ln);
    }
    if (EXACT)
        each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { dkdv_row<__hip_bfloat16>(again, b, kvh, dev_i, k0 + i, 0, d, ln.lane); });
}

// Both in one launch (they share nothing but the inputs).
template <int DP, bool PART, bool EXACT>
__global__ void __launch_bounds__(64 * BWD_WAVES, DP <= 64 ? 2 : 1)
bwd_split_kernel(StepArgs p, int n_tiles, BothKinds kinds) {
    __shared__ __attribute__((aligned(1024))) char lds[BWD_WAVES * 2 * STAGE_BYTES<DP> + 2 * SUB_BYTES<DP>];
    __shared__ __attribute__((aligned(1024))) char stats[BWD_WAVES * 2 * STAT_BYTES];
    __shared__ uint32_t masks[BWD_WAVES];
    int linear = (int)blockIdx.x;
    if (owns_keys(kinds, linear)) bwd_dkdv<DP, PART, EXACT>(p, n_tiles, linear, lds, stats, masks);
    else bwd_dq<DP, PART, EXACT>(p, n_tiles, linear, lds, stats, masks);
}

enum Pass { FWD, FWD_EXACT, BWD_EXACT, BWD };
template <int DP, bool PART>
hipError_t run(const StepArgs& a, Pass pass, hipStream_t st) {
    const int n_tiles = (a.c + OWN - 1) / OWN;
    const int n_dkdv = n_tiles * a.n_kv * a.B * a.H_kv, n_dq = n_tiles * a.n_q * a.B * a.H;
    const bool forward = pass == FWD || pass == FWD_EXACT;
    // (short blocks, all key-owning ones first: 2048 heads of 16 rows, d 128, 124 -> 116 us, 512 of 96 98 -> 94, ring of 8 x
    // 96, 32 heads, 97 -> 92)
    const BothKinds kinds = both_kinds(a, n_dkdv, n_dq, pass == BWD_EXACT ? INFINITY : 1.25);
    const dim3 grid((unsigned)(forward ? n_dq : n_dkdv + n_dq)), block(64 * (forward ? FWD_WAVES : BWD_WAVES));
    if (pass == FWD && a.q_pos) {           // (d is 64 or 128: the other forms only exist for these)
        if constexpr ((DP == 64 || DP == 128) && !PART)
            hipLaunchKernelGGL((fwd_split_kernel<DP, PART, false, true>), grid, block, 0, st, a, n_tiles);
    } else if (pass == FWD) hipLaunchKernelGGL((fwd_split_kernel<DP, PART, false>), grid, block, 0, st, a, n_tiles);
    else if (pass == FWD_EXACT) hipLaunchKernelGGL((fwd_split_kernel<DP, PART, true>), grid, block, 0, st, a, n_tiles);
    else if (pass == BWD_EXACT) hipLaunchKernelGGL((bwd_split_kernel<DP, PART, true>), grid, block, 0, st, a, n_tiles, kinds);
    else hipLaunchKernelGGL((bwd_split_kernel<DP, PART, false>), grid, block, 0, st, a, n_tiles, kinds);
    return hipGetLastError();
}
template <int DP>
hipError_t run(const StepArgs& a, Pass pass, hipStream_t st) {
    return a.d % 8 ? run<DP, true>(a, pass, st) : run<DP, false>(a, pass, st);
}
hipError_t run(const StepArgs& a, Pass pass, hipStream_t st) {
    if (a.d <= 32 && a.d % 8 == 0) return run<32, false>(a, pass, st);
    if (a.d <= 64) return run<64>(a, pass, st);
    if (a.d <= 112) return run<112>(a, pass, st);
    return run<128>(a, pass, st);
}

// Both sides' rows come through descriptors with 32-bit byte offsets (fwd_mfma.hip reads Q by 64-bit pointers, and
// fwd_mfma_supported looks at the rows of K and V only).  Requests behind a walk's end name up to 32 rows behind the
// block's last sub-tile: their offsets must not wrap into the matrix.
bool rows_in_reach(const StepArgs& a) {
    const int64_t widest = a.stride_s > a.kv_stride_s ? a.stride_s : a.kv_stride_s;
    return ((int64_t)(a.c + 127) / 128 * 128 + OWN) * 2 * widest + 2 * a.d < (int64_t(1) << 31);
}

}  // namespace

// (of shapes that the 128-row matrix-core kernels take.)  128-row kernels / these, us, d 128.
// Forward, by 128-row tiles of all queries: up to 64 always: 2 heads of 256 rows 11 / 8.4, one of 4096 61 / 22
// (full 61 / 24), ring of 4 x 1024, 2 heads 65 / 26.  128: triangular 64 heads of 200 12.1 / 13.0, 32 of 512 16 / 15, 8 of 2048 36 / 23;
// full 32 of 512 15.5 / 17.2, 8 of 2048 35.1 / 32.5, ring of 4 x 128, 32 heads, contiguous 15.1 / 15.4.  256:
// triangular 16 heads of 2048 39 / 42, 4 of 8192 122 / 108, ring of 4 x 1024, 8 heads 66.7 / 68.3, of
// 4 x 2048, 4 heads 121 / 112, full 8 of 4096 78 / 107; d 64: ring of 4 x 1024, 8 heads 49.7 / 45.9.  A single
// block of 128 rows is as well off in one 128-row tile up to 112 columns (d 64 7.9 / 8.3, d 128 10 / 8.5).  An odd number
// of heads has every XCD stream all of them, full blocks of 65 to 128 tiles above 64 columns: d 128, 11 heads of
// 1024 23.0 / 24.3, 13 of 1100 26.0 / 27.4, 15 of 1024 24.2 / 28.0, 9 of 1700 34.3 / 32.0, but 14 of 1152 25.2 / 23.6,
// 15 on 3 of 1024 22.5 / 21.0.  32 columns: 12 heads of 1000 rows, full, 13.8 / 9.8, 32 of 512 8.6 / 8.0; triangular 16
// of 2048 23.7 / 17.5, 32 of 1024 14.4 / 14.3.
bool narrow(const StepArgs& a) { return a.d <= 32 && a.d % 8 == 0; }          // 32 columns computed
bool fwd_split_wanted(const StepArgs& a) {
    const int64_t tiles = (int64_t)((a.c + 127) / 128) * a.B * a.n_q * a.H, walk = (int64_t)a.c * a.n_kv;
    if (a.d > TD || (walk <= 128 && a.d <= 112)) return false;
    if (!rows_in_reach(a)) return false;
    if (tiles <= 64) return true;
    if (tiles <= 128) return walk >= (a.layout == SA_STRIPED || narrow(a) ? 512 : a.d > 64 && a.H == a.H_kv && a.B * a.H % 2 ? 1536 : 1024);
    return tiles <= 256 && uneven(a) && walk >= (narrow(a) ? 2048 : a.d <= 112 ? 4096 : 8192);
}
hipError_t launch_fwd_split(const StepArgs& a, hipStream_t st) { return run(a, FWD, st); }
// Backward step, by 128-row tiles of all keys ("tiles") and key/value heads: four times the workgroups walk a quarter
// of the rows each, which pays while a head has many of them; a last 128-row tile that is nearly empty counts for it,
// so the heads are weighed by the square of what 32-row tiles save there.  Several hundred drawn shapes a line, geometric mean
// (worst) of 128-row time / this one:
//  * up to 64 tiles 1.2 to 2.3; full blocks above 64 columns 1.2 to 1.4 (1.0) up to 40 heads, beyond 1.0 (0.8)
//  * 65 to 128 tiles above 64 columns: triangular, walks of 2048 rows of the group and more, up to 8 heads 1.4 to 2.1
//    (1.2), 16 1.2 (1.05), 20 1.1 (0.9), 30 0.9 (0.8); full with groups of four and more, up to 16 heads 1.5 (1.0), 24 1.3
//    (1.0), 40 1.15 (0.9), beyond 0.9 (0.7); without groups 2 heads of 8192 rows 233 / 257 us
//  * 65 to 128 tiles up to 64 columns, where two workgroups fit a compute unit: 1.2 to 2.5 (1.0), full blocks of short
//    walks excepted (32 heads of 512 rows 19.6 / 18.3 us, but at d 32 16.1 / 17.0, 20 of 512 15.2 / 13.4)
//  * 129 to 512 tiles up to 64 columns, triangular: up to 24 heads 1.15 to 1.5 (1.05), 56 1.1 (0.94), 100 1.0 (0.85),
//    beyond 0.9 (0.7); 32 heads of 2048 rows (512 tiles) 99 / 99, d 32 80 / 82; full, 256: 46.4 / 45.8, 254 / 263
//  * 256 tiles above 64 columns: 8 heads of 4096 137 / 160, 32 on 8 of 4096 500 / 574
//  * 129 to 512 tiles, 32 columns computed, triangular: 32 heads of 1024 28.1 / 21.4 us in 128-row tiles, 16 of 2048 36.8 /
//    34.6, 8 of 4096 57 / 62, 8 of 8192 192 / 205; where the last round of 256 is not three quarters full, 8 of 3000 37 / 50,
//    16 of 3000 69 / 86; one device's queries against all shards' keys leave the 128-row kernel's queries' side short: 8
//    heads 4 x 1024 34 / 55, 4 heads 4 x 4096 136 / 218, 32 on 8 of 8 x 1024 124 / 158; 32 heads 2 x 512 25 / 22.  The rule
//    is 0.3 % (worst 1.2) behind the better kernel of each of 312 shapes
bool bwd_split_wanted(const StepArgs& a) {
    const int64_t t128 = (a.c + 127) / 128, t32 = (a.c + 31) / 32, heads = (int64_t)a.B * a.H_kv, group = a.H / a.H_kv;
    const int64_t keys = t128 * a.n_kv * heads, walk = (int64_t)a.c * a.n_q * group;
    auto up_to = [&](int64_t most) { return heads * t32 * t32 <= most * 16 * t128 * t128; };
    if (a.d > TD || !rows_in_reach(a)) return false;
    if (keys <= 64) return a.d <= 64 || uneven(a) || up_to(40);
    if (a.d > 64) return keys <= 128 && (uneven(a) ? walk >= 2048 && up_to(16) : group >= 4 && up_to(24));
    if (!uneven(a)) return keys <= 128 && walk >= (a.d <= 32 ? 6 : 4) * keys;
    if (keys > 128 && narrow(a)) {
        const int64_t queries = t128 * a.n_q * heads * group;
        if (keys > 512) return false;
        return 2 * queries <= keys ? walk >= 5 * queries : walk >= 12 * keys || (keys <= (keys <= 256 ? 192 : 384) && walk >= 6 * keys);
    }
    return up_to(56) && (keys <= 256 ? walk >= 4 * keys : keys <= 512 && walk > 4 * keys);
}
hipError_t launch_bwd_split(const StepArgs& a, hipStream_t st) { return run(a, BWD, st); }

// bf16 blocks shorter than a 128-row tile, probabilities and dS in fp32 precision.  Against the fp32 instruction on widened
// operands (f32_step.hip), us: forward step, d 128, 4 heads of 64 tokens 15.7 / 7.7, 64 of 96 17.1 / 8.3, 256 of
// 120 38.9 / 25.5, d 64 10.3 / 7.8, 11.1 / 8.0, 20.7 / 14.0, d 32 7.9 / 7.8, 8.0 / 7.8, 13.0 / 13.2 (7.7 is
// what a launch takes).  Error against 64 bits (2-norm, 16 x 127 tokens, d 128): O 2.2e-7 -> 1.6e-7, dQ
// 3.7e-7 -> 3.2e-7, dK 6.1e-7 -> 4.3e-7, dV 6.0e-7 -> 4.1e-7.  A single forward block of many heads stays with the fp32
// instruction up to 32 columns (half of the columns computed here are padding): d 16, 600 heads of 30 rows 10.0 / 11.0,
// 512 8.7 / 8.4, 400 heads of 60 11.4 / 13.1, of 96 15.1 / 16.1, of 127 18.5 / 21.2, 360 11.4 / 11.1, 15.1 / 16.1, 18.6 /
// 18.5; 1024 of 96 23.9 / 33.8, d 32 26.2 / 34.1, d 36 54 / 41.
bool short_exact_wanted(const StepArgs& a, int dtype, bool backward) {
    if (dtype != SA_BF16 || a.d % 4 || a.d > TD || a.c >= 128 || !rows_in_reach(a)) return false;
    return backward || a.n_kv > 1 || a.d > 32 || (int64_t)a.B * a.n_q * a.H <= (a.c <= 32 ? 512 : 384);
}
hipError_t launch_short_exact(const StepArgs& a, bool backward, hipStream_t st) {
    return run(a, backward ? BWD_EXACT : FWD_EXACT, st);
}

}  // namespace sa
