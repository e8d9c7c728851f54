// Ring step for fp32 launches that leave much of the chip idle with 128-row workgroups, head dimension up to 128:
// products of three bf16 terms a number, as in f32x3_step.hip, in the work split of split_mfma.hip.
//
// What bounds such a launch is the walk of one workgroup, and in it the matrix cores and the vector instructions
// that make terms of the streamed rows (5.5 an element, once for the products over the head dimension and once for
// those over the rows) about alike: a 32 x 32 sub-tile at 128 columns is 48 products and 352 such instructions a
// contraction.  So a workgroup owns 32 rows, its wavefronts take every fourth (up to 64 columns, where two of
// them fit a SIMD, every eighth) sub-tile of 32 streamed rows, each through a stage of LDS of its own that
// direct loads fill with the fp32 rows as they are, and the terms of one k-step are made beside the products of
// the one before.  A stage is requested anew as soon as its last read is in registers, and the order of the
// contractions is such that another one lies between that and the next use.
#include "f32x3_parts.h"
#include "split_parts.h"

namespace sa {

namespace {

template <int DP> constexpr int WAVES_OF = DP <= 64 ? 8 : 4;
template <int DP> constexpr int ROW_BYTES = 4 * DP;
template <int DP> constexpr int RAW_BYTES = 32 * ROW_BYTES<DP>;          // 32 rows of one streamed operand
template <int DP> constexpr int LOADS = RAW_BYTES<DP> / 1024;            // direct loads they take
template <int DP> constexpr int STAGES_BYTES = WAVES_OF<DP> * 2 * RAW_BYTES<DP>;

// Rows of 16-byte chunks; chunk c of row r lies at chunk position c ^ swizzle(r), so that the row reads of 16
// consecutive rows (one logical chunk) hit different positions of a 256-byte line: at 32 columns, two rows to
// a line, rows of equal parity have to differ.
template <int DP>
constexpr int swizzle(int r) { return DP <= 32 ? (r >> 1) & 7 : r & 15; }

template <int DP>
struct RawLane {
    int lane, n, h, wave;
    uint32_t row[8];            // row n, chunk 4 ks + 2 h + j at [2 (ks % 4) + j]
    uint32_t tr[8];             // column n of row 4 h + e % 4 + 8 (e / 4)
    __device__ RawLane() {
        lane = threadIdx.x & 63;
        n = lane & 31;
        h = lane >> 5;
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            row[i] = n * ROW_BYTES<DP> + ((((4 * (i / 2) + 2 * h + i % 2) & (DP / 4 - 1)) ^ swizzle<DP>(n)) << 4);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int r = 4 * h + e % 4 + 8 * (e / 4);
            tr[e] = r * ROW_BYTES<DP> + (((n >> 2) ^ swizzle<DP>(r)) << 4) + (n & 3) * 4;
        }
    }
};

// The loads of a streamed sub-tile, as split_mfma.hip's Loader: four pieces share one setting of m0.
constexpr int AHEAD_BYTES = 4096;
__device__ inline dt_rsrc stream_rsrc(const void* matrix, int rows, int pitch, int d) {
    dt_rsrc r = dt_make_rsrc((const char*)matrix - AHEAD_BYTES, rows, pitch, 2 * d);        // (2 d bf16 columns)
    r[2] += AHEAD_BYTES;
    return r;
}
template <int DP>
struct RawLoader {
    static constexpr int HALF = LOADS<DP> / 2, GROUP = HALF < 4 ? HALF : 4;      // pieces of 16 rows, of one m0
    uint32_t at[HALF];
    int pitch;
    __device__ RawLoader(int pitch_, int d, int lane) : pitch(pitch_) {
        constexpr int CHUNKS = DP / 4;
#pragma unroll
        for (int j = 0; j < HALF; ++j) {
            const int r = 64 / CHUNKS * j + lane / CHUNKS, chunk = lane % CHUNKS ^ swizzle<DP>(r);
            at[j] = 4 * chunk < d ? r * pitch + 16 * chunk + AHEAD_BYTES - 1024 * (j % GROUP) : DT_OUT_OF_RANGE;
        }
    }
    // 32 rows from row `row` on (the swizzle is the same for both halves)
    __device__ inline void load(dt_rsrc m, int row, const char* to) const {
#pragma unroll
        for (int i = 0; i < LOADS<DP>; i += GROUP) {
            const uint32_t dst = (uint32_t)reinterpret_cast<uintptr_t>((const lds_char_t*)to) + 1024 * i;
            const int byte = (row + (i >= HALF ? 16 : 0)) * pitch, j = i % HALF;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
            if constexpr (GROUP == 4)
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                             "buffer_load_dwordx4 %1, %5, %6 offen lds\n\t"
                             "buffer_load_dwordx4 %2, %5, %6 offen offset:1024 lds\n\t"
                             "buffer_load_dwordx4 %3, %5, %6 offen offset:2048 lds\n\t"
                             "buffer_load_dwordx4 %4, %5, %6 offen offset:3072 lds"
                             :
                             : "s"(dst), "v"(at[j]), "v"(at[j + 1]), "v"(at[j + 2]), "v"(at[j + 3]), "s"(m), "s"(byte)
                             : "memory", "m0");
            else
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                             "buffer_load_dwordx4 %1, %3, %4 offen lds\n\t"
                             "buffer_load_dwordx4 %2, %3, %4 offen offset:1024 lds"
                             :
                             : "s"(dst), "v"(at[j]), "v"(at[j + 1]), "s"(m), "s"(byte)
                             : "memory", "m0");
#pragma clang diagnostic pop
        }
    }
};

// ---------------------------------------------------------------- operands
// k-step ks of a row: 8 consecutive columns
template <int DP>
__device__ inline void read_row(float (&x)[8], const char* raw, int ks, const RawLane<DP>& ln) {
    const char* at = raw + (DP > 64 ? 256 * (ks / 4) : 0);
    const float4 a = *reinterpret_cast<const float4*>(at + ln.row[2 * (ks % 4)]);
    const float4 b = *reinterpret_cast<const float4*>(at + ln.row[2 * (ks % 4) + 1]);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}
// 32-column block mb of 16 rows: 8 of them, one column (an odd block's chunks differ in bit 3, which the swizzle
// sets for the rows from 8 on)
template <int DP>
__device__ inline void read_column(float (&x)[8], const char* raw, int mb, int g, const RawLane<DP>& ln) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int at = 16 * g * ROW_BYTES<DP> + 256 * (mb / 2) + (mb % 2 ? (e < 4 ? 128 : -128) : 0);
        x[e] = *reinterpret_cast<const float*>(raw + at + ln.tr[e]);
    }
}
// k-step ks of an owned row (its d columns, zeros beyond)
__device__ __forceinline__ void load_own(bf16x8 (&o)[3], const float* row, int ks, int h, int d) {
    const int col = 16 * ks + 8 * h;
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 a = col < d ? *reinterpret_cast<const float4*>(row + col) : z;
    const float4 b = col + 4 < d ? *reinterpret_cast<const float4*>(row + col + 4) : z;
    const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    split8(x, o);
}
// The owned rows' B operands.  Up to 64 columns, two wavefronts to a SIMD, in LDS ([k-step][term][lane], 16 bytes
// each), where the wavefronts make them once for all: in registers they sent 49 others to scratch memory, and the
// reloads of those wait for the streamed rows (backward step of 4 heads of 256 rows, d 64, 18.5 -> 14.7 us).
// Above, one wavefront to a SIMD and LDS full of the streamed rows, in the wavefront's own registers.
template <int DP> constexpr bool OWN_IN_LDS = DP <= 64;
template <int DP> constexpr int OWN_BYTES = OWN_IN_LDS<DP> ? DP / 16 * 3 * 1024 : 0;
template <int DP, bool IN_LDS = OWN_IN_LDS<DP>>
struct Own {
    const char* at;
    // operand `which` of the N whose rows are at hand: everybody makes its share of all of them
    template <int N>
    static __device__ __forceinline__ void make(char* to, Own (&own)[N], const float* const (&row)[N], const RawLane<DP>& ln, int d) {
        constexpr int KS = DP / 16, WAVES = WAVES_OF<DP>;
#pragma unroll
        for (int i = 0; i < N * KS; i += WAVES) {
            const int at = i + ln.wave;
            if (N * KS % WAVES != 0 && at >= N * KS) break;
            bf16x8 o[3];
            load_own(o, N == 1 || at < KS ? row[0] : row[N - 1], at % KS, ln.h, d);
#pragma unroll
            for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x8*>(to + (3 * at + t) * 1024 + ln.lane * 16) = o[t];
        }
#pragma unroll
        for (int i = 0; i < N; ++i) own[i].at = to + i * OWN_BYTES<DP>;
        meet();
    }
    __device__ __forceinline__ void get(bf16x8 (&o)[3], int ks, int lane) const {
#pragma unroll
        for (int t = 0; t < 3; ++t) o[t] = *reinterpret_cast<const bf16x8*>(at + (3 * ks + t) * 1024 + lane * 16);
    }
};
template <int DP>
struct Own<DP, false> {
    bf16x8x3 f[DP / 16];
    template <int N>
    static __device__ __forceinline__ void make(char*, Own (&own)[N], const float* const (&row)[N], const RawLane<DP>& ln, int d) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int ks = 0; ks < DP / 16; ++ks) load_own(own[i].f[ks], row[i], ks, ln.h, d);
    }
    __device__ __forceinline__ void get(bf16x8 (&o)[3], int ks, int) const {
#pragma unroll
        for (int t = 0; t < 3; ++t) o[t] = f[ks][t];
    }
};
// 32 x 32 scores: rows = the 32 streamed rows, columns = the owned ones.  NaN where an operand is infinite or
// rounds to an infinite hi.  beside(i), i = 0 .. KS - 1: vector work to go with the products.
template <int DP, typename Beside>
__device__ __forceinline__ f32x16 scores(const char* raw, const Own<DP>& own, const RawLane<DP>& ln, Beside beside) {
    constexpr int KS = DP / 16;
    f32x16 hi = zero16(), lo = zero16();
    Split8 x[KS];
    bf16x8x3 a[KS], f[KS];
    read_row<DP>(x[0].x, raw, 0, ln);
    own.get(f[0], 0, ln.lane);
    read_row<DP>(x[1].x, raw, 1, ln);
#pragma unroll
    for (int i = 0; i < 6; ++i) x[0].step(i);
    x[0].operands(a[0]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        products(a[ks], f[ks], hi, lo, [&](int i) {
            if (i == 0 && ks + 1 < KS) own.get(f[ks + 1], ks + 1, ln.lane);
            if (i == 0 && ks + 2 < KS) read_row<DP>(x[ks + 2].x, raw, ks + 2, ln);
            if (ks + 1 < KS) x[ks + 1].step(i);
            if (i == 5) beside(ks);
        });
        if (ks + 1 < KS) x[ks + 1].operands(a[ks + 1]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 16; ++r) hi[r] += lo[r];
    return hi;
}
// acc (32-column blocks x owned rows) += streamed^T w, the sub-tile's sum formed by itself (f32x3_step.hip)
template <int DP>
__device__ __forceinline__ void accumulate(f32x16 (&acc)[4], const char* raw, const f32x16& w, const RawLane<DP>& ln) {
    constexpr int N = 2 * blocks_of(DP);
    Split8 x[N], y;
    bf16x8x3 a[N], b[2];
    f32x16 t[2];
    read_column<DP>(x[0].x, raw, 0, 0, ln);
    read_column<DP>(x[1].x, raw, 0, 1, ln);
    split_tile(w, 0, b[0]);
#pragma unroll
    for (int i = 0; i < 6; ++i) x[0].step(i);
    x[0].operands(a[0]);
#pragma unroll
    for (int e = 0; e < 8; ++e) y.x[e] = w[8 + e];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        f32x16& s = t[n / 2 % 2];
        if (n % 2 == 0) s = zero16();
        products(a[n], b[n % 2], s, s, [&](int i) {
            if (i == 0 && n + 2 < N) read_column<DP>(x[n + 2].x, raw, (n + 2) / 2, n % 2, ln);
            if (n + 1 < N) x[n + 1].step(i);
            if (n == 0) y.step(i);
            // the block before, four rows a product
            if (n % 2 == 1 && n > 1 && i >= 2) {
#pragma unroll
                for (int r = 4 * (i - 2); r < 4 * (i - 1); ++r) acc[n / 2 - 1][r] += t[(n / 2 - 1) % 2][r];
            }
        });
        if (n == 0) y.operands(b[1]);
        if (n + 1 < N) x[n + 1].operands(a[n + 1]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[N / 2 - 1][r] += t[(N / 2 - 1) % 2][r];
}

// ------------------------------------------------------------------ forward
template <int DP>
__global__ void __launch_bounds__(64 * WAVES_OF<DP>, WAVES_OF<DP> / 4)
fwd_f32x3_split_kernel(StepArgs p, int n_tiles) {
    constexpr int WAVES = WAVES_OF<DP>, MB = blocks_of(DP);
    static_assert(PARTIAL_BYTES<DP, WAVES> <= STAGES_BYTES<DP>, "partial results");
    __shared__ __attribute__((aligned(1024))) char lds[STAGES_BYTES<DP> + OWN_BYTES<DP>];
    __shared__ float stats[WAVES * 64];                // [wave][m | l][32]
    __shared__ __attribute__((aligned(16))) uint32_t masks[4 * WAVES];          // (RowsToRedo)

    const RawLane<DP> ln;
    const int n = ln.n, h = ln.h;
    int rank, bh, dev_rank;
    decode((int)blockIdx.x, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * OWN, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int pitch = 4 * (int)p.kv_stride_s;
    const int a_own = q0 + n, a = min(a_own, p.c - 1);

    KeyCursor at(p, dev, q0, ln.wave);
    const RawLoader<DP> loader(pitch, d, ln.lane);
    char* const k = lds + ln.wave * 2 * RAW_BYTES<DP>;
    char* const v = k + RAW_BYTES<DP>;
    dt_rsrc K = stream_rsrc((const float*)p.k + kv_base, p.c, pitch, d);
    dt_rsrc V = stream_rsrc((const float*)p.v + kv_base, p.c, pitch, d);
    int kv_at = at.kv;
    // (behind the walk's end: rows beyond the matrix, whose loads deliver zeros without a look at memory)
    const int beyond = 32 * at.n_full;
    int key0, shift;                    // the sub-tile; key0 == beyond: none
    auto take = [&]() {
        at.settle<WAVES>();
        key0 = at.kv < at.kv_end ? 32 * at.v : beyond;
        shift = at.shift;
        at.v += WAVES;
        if (at.kv != kv_at) {
            K = dt_advance(K, (at.kv - kv_at) * 4 * p.kv_shard);
            V = dt_advance(V, (at.kv - kv_at) * 4 * p.kv_shard);
            kv_at = at.kv;
        }
    };
    at.enter<WAVES>();
    take();
    loader.load(K, key0, k);
    loader.load(V, key0, v);

    Own<DP> own[1];
    Own<DP>::make(lds + STAGES_BYTES<DP>, own, {(const float*)p.q + base + (int64_t)a * p.stride_s}, ln, d);
    const Scale2 kappa(p.scale);
    float m = -INFINITY, l = 0.f;           // m in base-2 units; l: this half-wave's share of the row sum
    f32x16 acc[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acc[mb] = zero16();
    while (key0 != beyond) {
        wait_all_but<LOADS<DP>>();
        f32x16 x = scores<DP>(k, own[0], ln, [](int) {});
        const bool masked = key0 + 31 > min(p.c - 1, q0 + shift);          // some pair of the sub-tile is
        const int lane_last = min(p.c - 1, a_own + shift) - key0;
        take();
        wait_lds();
        loader.load(K, key0, k);
        if (masked) {
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = reg_row(r, h) <= lane_last ? x[r] : -INFINITY;
        }
        float mx[2] = {x[0], x[1]};
#pragma unroll
        for (int r = 2; r < 16; ++r) mx[r % 2] = fmaxf(mx[r % 2], x[r]);
        const float m_new = fmaxf(m, half_wave_max(fmaxf(mx[0], mx[1])) * kappa.hi);
        const float ref = m_new == -INFINITY ? 0.f : m_new;                 // a row without a key so far
        if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {
            const float alpha = __builtin_amdgcn_exp2f(m - ref);
            l *= alpha;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mb][r] *= alpha;
        }
        m = m_new;
        float sum[2] = {0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            x[r] = kappa.exp2(x[r], ref, 0.f);
            sum[r % 2] += x[r];
        }
        l += sum[0] + sum[1];
        wait_all_but<LOADS<DP>>();
        accumulate<DP>(acc, v, x, ln);
        wait_lds();
        loader.load(V, key0, v);
    }
    wait_all_but<0>();
    float* L = p.lse + b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c + a;
    const uint32_t odd_rows = fold_forward<DP, WAVES, true, true>(p, acc, m, l, lds, stats, masks, ln, dev, a_own, a, L,
                                                            p.o + base + (int64_t)a * p.stride_s);
    each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { fwd_row<float>(again, b, hd, dev_i, q0 + i, ln.lane); });
}

// ----------------------------------------------------------------------- dQ
template <int DP>
__device__ inline void bwd_dq(const StepArgs& p, int n_tiles, int linear, char* lds, uint32_t* masks) {
    constexpr int WAVES = WAVES_OF<DP>, N = share_of(DP, WAVES);
    const RawLane<DP> ln;
    const int n = ln.n, h = ln.h;
    int rank, bh, dev_rank;
    decode_near(linear, n_tiles * p.n_q, p.B * p.H, uneven(p), rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * OWN, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c;
    const int pitch = 4 * (int)p.kv_stride_s;
    const int a_own = q0 + n, a = min(a_own, p.c - 1);

    KeyCursor at(p, dev, q0, ln.wave);
    const RawLoader<DP> loader(pitch, d, ln.lane);
    char* const k = lds + ln.wave * 2 * RAW_BYTES<DP>;
    char* const v = k + RAW_BYTES<DP>;
    dt_rsrc K = stream_rsrc((const float*)p.k + kv_base, p.c, pitch, d);
    dt_rsrc V = stream_rsrc((const float*)p.v + kv_base, p.c, pitch, d);
    int kv_at = at.kv;
    const int beyond = 32 * at.n_full;          // as in the forward kernel
    int key0, shift;
    auto take = [&]() {
        at.settle<WAVES>();
        key0 = at.kv < at.kv_end ? 32 * at.v : beyond;
        shift = at.shift;
        at.v += WAVES;
        if (at.kv != kv_at) {
            K = dt_advance(K, (at.kv - kv_at) * 4 * p.kv_shard);
            V = dt_advance(V, (at.kv - kv_at) * 4 * p.kv_shard);
            kv_at = at.kv;
        }
    };
    at.enter<WAVES>();
    take();
    loader.load(V, key0, v);
    loader.load(K, key0, k);

    Own<DP> own[2];
    Own<DP>::make(lds + STAGES_BYTES<DP>, own, {(const float*)p.q + base + (int64_t)a * p.stride_s,
                                                (const float*)p.dout + base + (int64_t)a * p.stride_s}, ln, d);
    const float delta = p.delta[sbase + a];
    const Scale2 kappa(p.scale);
    float lse, lse_lo;
    to_base2(p.lse[sbase + a], lse, lse_lo);
    f32x16 acc[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acc[mb] = zero16();
    // dP first: K, which the walk's step before has read last, is on its way meanwhile
    while (key0 != beyond) {
        wait_all_but<LOADS<DP>>();
        const f32x16 dp = scores<DP>(v, own[1], ln, [](int) {});
        const bool masked = key0 + 31 > min(p.c - 1, q0 + shift);
        const int lane_last = min(p.c - 1, a_own + shift) - key0;
        take();
        wait_lds();
        loader.load(V, key0, v);
        wait_all_but<LOADS<DP>>();
        f32x16 x = scores<DP>(k, own[0], ln, [](int) {});
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = kappa.exp2(x[r], lse, lse_lo);
        if (masked) {
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = reg_row(r, h) <= lane_last ? x[r] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] *= dp[r] - delta;
        accumulate<DP>(acc, k, x, ln);
        wait_lds();
        loader.load(K, key0, k);
    }
    wait_all_but<0>();

    float* const DQ = p.dq + base + (int64_t)a * p.stride_s;
    float4 old[N];
    load_old<DP, WAVES>(old, DQ, d, !p.fresh && a_own < p.c, ln);
    const RowsToRedo<WAVES> redo = {reinterpret_cast<uint4*>(masks), ln.lane, ln.wave, row_mask(a_own < p.c)};
    const float top = loudest<blocks_of(DP)>(acc);          // (beside the loads)
    const bool odd = a_own < p.c && not_finite<blocks_of(DP)>(acc);
    __syncthreads();
    put_partial<DP>(lds, acc, ln);
    redo.put(odd, top, top);
    __syncthreads();
    const uint32_t odd_rows = redo.take(top, top);
    if (a_own < p.c && !((odd_rows >> n) & 1)) add_rows<DP, WAVES>(DQ, old, lds, p.scale, d, ln);
    each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { dq_row<float>(again, b, hd, dev_i, q0 + i, ln.lane); });
}

// -------------------------------------------------------------------- dK/dV
// Owned rows are keys, the streamed ones queries with their LSE and delta beside them; the query heads that share
// the key/value head and the query shards that see it come one after the other.
template <int DP>
__device__ inline void bwd_dkdv(const StepArgs& p, int n_tiles, int linear, char* lds, char* stats, uint32_t* masks) {
    constexpr int WAVES = WAVES_OF<DP>, KS = DP / 16, N = share_of(DP, WAVES);
    const RawLane<DP> ln;
    const int n = ln.n, h = ln.h;
    int tile, bh, dev_i;                                // low key tiles see most queries: first
    decode_near(linear, n_tiles * p.n_kv, p.B * p.H_kv, uneven(p), tile, bh);
    decode_rank(tile, n_tiles, p.n_kv, p.layout, tile, dev_i);
    const int k0 = tile * OWN, dev = p.kv_dev + dev_i;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv, group = p.H / p.H_kv, d = p.d;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + dev_i * p.kv_shard;
    const int pitch = 4 * (int)p.stride_s;
    const int key_own = k0 + n, key = min(key_own, p.c - 1);
    const int64_t row = kv_base + (int64_t)key * p.kv_stride_s;

    // Blocks: the members of the group, each with the query shards that see the keys.  Of a block this
    // wavefront takes the sub-tiles of 32 queries whose number less k0 / 32 (full blocks: whose number) is
    // wave - turn modulo the wavefronts, turn counting the sub-tiles of the blocks before.
    const RawLoader<DP> loader(pitch, d, ln.lane);
    char* const q = lds + ln.wave * 2 * RAW_BYTES<DP>;
    char* const g = q + RAW_BYTES<DP>;
    char* const stat = stats + ln.wave * STAT_BYTES;
    const int q_dev0 = p.layout == SA_STRIPED ? p.q_dev : max(p.q_dev, dev), q_end = p.q_dev + p.n_q;
    const int n_sub = (p.c + 31) / 32;
    int member = q_dev0 < q_end ? 0 : group, q_dev = q_dev0, v = 0, turn = 0;
    int block_shift = 0;              // key b is seen by the block's queries from b + block_shift on
    dt_rsrc Q, G, S, E;
    auto enter = [&]() {
        const bool full = block_kind(q_dev, dev, p.layout) == MASK_FULL;
        const int off = block_off(q_dev, dev, p.layout), first = full ? 0 : k0 / 32;
        v = first + ((ln.wave - turn) & (WAVES - 1));
        turn += n_sub - first;
        block_shift = full ? -(p.c + OWN) : off;
        const int hd = kvh * group + member;
        const int64_t base = b * p.stride_b + hd * p.stride_h + (q_dev - p.q_dev) * p.q_shard;
        const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(q_dev - p.q_dev) * p.c;
        Q = stream_rsrc((const float*)p.q + base, p.c, pitch, d);
        G = stream_rsrc((const float*)p.dout + base, p.c, pitch, d);
        S = dt_make_rsrc(p.lse + sbase, p.c, 4, 2);
        E = dt_make_rsrc(p.delta + sbase, p.c, 4, 2);
    };
    const int beyond = 32 * n_sub;
    int a0, shift;                      // the sub-tile; a0 == beyond: none
    auto take = [&]() {
        while (v >= n_sub && member < group) {
            if (++q_dev >= q_end) {
                q_dev = q_dev0;
                ++member;
            }
            if (member < group) enter();
        }
        a0 = member < group ? 32 * v : beyond;
        shift = block_shift;
        v += WAVES;
    };
    auto load_q = [&]() {
        loader.load(Q, a0, q);
        load_stat(S, a0, stat, ln.lane);
        load_stat(E, a0, stat + 256, ln.lane);
    };
    enter();
    take();
    load_q();
    loader.load(G, a0, g);

    Own<DP> own[2];
    Own<DP>::make(lds + STAGES_BYTES<DP>, own, {(const float*)p.k + row, (const float*)p.v + row}, ln, d);
    const Scale2 kappa(p.scale);
    f32x16 acck[4], accv[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acck[mb] = accv[mb] = zero16();
    while (a0 != beyond) {
        wait_all_but<LOADS<DP>>();
        f32x16 pr = scores<DP>(q, own[0], ln, [](int) {});
        wait_all_but<0>();
        // beside dP: the probabilities
        f32x16 ds = scores<DP>(g, own[1], ln, [&](int ks) {
#pragma unroll
            for (int r = 16 / KS * ks; r < 16 / KS * (ks + 1); r += 2) {
                const float2 y = *reinterpret_cast<const float2*>(stat + 4 * reg_row(r, h));
                float hi, lo;
                to_base2(y.x, hi, lo);
                pr[r] = kappa.exp2(pr[r], hi, lo);
                to_base2(y.y, hi, lo);
                pr[r + 1] = kappa.exp2(pr[r + 1], hi, lo);
            }
        });
        if (a0 < k0 + OWN - 1 + shift || a0 + 32 > p.c) {       // some pair of the sub-tile is masked
            const int lane_first = key_own + shift - a0, rows = p.c - a0;
#pragma unroll
            for (int r = 0; r < 16; ++r) pr[r] = reg_row(r, h) >= lane_first && reg_row(r, h) < rows ? pr[r] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            const float4 e = *reinterpret_cast<const float4*>(stat + 256 + 4 * reg_row(r, h));
            ds[r] = pr[r] * (ds[r] - e.x); ds[r + 1] = pr[r + 1] * (ds[r + 1] - e.y);
            ds[r + 2] = pr[r + 2] * (ds[r + 2] - e.z); ds[r + 3] = pr[r + 3] * (ds[r + 3] - e.w);
        }
        take();
        accumulate<DP>(acck, q, ds, ln);
        wait_lds();
        load_q();
        accumulate<DP>(accv, g, pr, ln);
        wait_lds();
        loader.load(G, a0, g);
    }
    wait_all_but<0>();

    constexpr int HALF = PARTIAL_BYTES<DP, WAVES>;
    static_assert(2 * HALF <= STAGES_BYTES<DP>, "partial results");
    float4 old_v[N], old_k[N];
    load_old<DP, WAVES>(old_v, p.dv + row, d, !p.fresh && key_own < p.c, ln);
    load_old<DP, WAVES>(old_k, p.dk + row, d, !p.fresh && key_own < p.c, ln);
    const RowsToRedo<WAVES> redo = {reinterpret_cast<uint4*>(masks), ln.lane, ln.wave, row_mask(key_own < p.c)};
    const float top_v = loudest<blocks_of(DP)>(accv), top_k = loudest<blocks_of(DP)>(acck);
    const bool odd = key_own < p.c && (not_finite<blocks_of(DP)>(accv) || not_finite<blocks_of(DP)>(acck));
    __syncthreads();
    put_partial<DP>(lds, accv, ln);
    put_partial<DP>(lds + HALF, acck, ln);
    redo.put(odd, top_v, top_k);
    __syncthreads();
    const uint32_t odd_rows = redo.take(top_v, top_k);
    if (key_own < p.c && !((odd_rows >> n) & 1)) {
        add_rows<DP, WAVES>(p.dv + row, old_v, lds, 1.f, d, ln);
        add_rows<DP, WAVES>(p.dk + row, old_k, lds + HALF, p.scale, d, ln);
    }
    each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { dkdv_row<float>(again, b, kvh, dev_i, k0 + i, 0, d, ln.lane); });
}

// Both in one launch (they share nothing but the inputs).
template <int DP>
__global__ void __launch_bounds__(64 * WAVES_OF<DP>, WAVES_OF<DP> / 4)
bwd_f32x3_split_kernel(StepArgs p, int n_tiles, BothKinds kinds) {
    __shared__ __attribute__((aligned(1024))) char lds[STAGES_BYTES<DP> + 2 * OWN_BYTES<DP>];
    __shared__ __attribute__((aligned(1024))) char stats[WAVES_OF<DP> * STAT_BYTES];
    __shared__ __attribute__((aligned(16))) uint32_t masks[4 * WAVES_OF<DP>];          // (RowsToRedo)
    int linear = (int)blockIdx.x;
    if (owns_keys(kinds, linear)) bwd_dkdv<DP>(p, n_tiles, linear, lds, stats, masks);
    else bwd_dq<DP>(p, n_tiles, linear, lds, masks);
}

template <int DP>
hipError_t run(const StepArgs& a, bool backward, hipStream_t st) {
    const int n_tiles = (a.c + OWN - 1) / OWN;
    const int n_dkdv = n_tiles * a.n_kv * a.B * a.H_kv, n_dq = n_tiles * a.n_q * a.B * a.H;
    const dim3 block(64 * WAVES_OF<DP>);
    if (backward)
        hipLaunchKernelGGL((bwd_f32x3_split_kernel<DP>), dim3((unsigned)(n_dkdv + n_dq)), block, 0, st, a, n_tiles,
                           both_kinds(a, n_dkdv, n_dq, 1.25));
    else hipLaunchKernelGGL((fwd_f32x3_split_kernel<DP>), dim3((unsigned)n_dq), block, 0, st, a, n_tiles);
    return hipGetLastError();
}

}  // namespace

bool f32x3_split_supported(const StepArgs& a, bool backward) {
    // both sides' rows come through descriptors with 32-bit byte offsets, up to 32 rows behind the block's last sub-tile
    const int64_t widest = a.stride_s > a.kv_stride_s ? a.stride_s : a.kv_stride_s;
    if (((int64_t)(a.c + 31) / 32 * 32 + OWN) * 4 * widest + 4 * a.d + 4096 >= (int64_t(1) << 31)) return false;
    // HIP takes fewer than 2^32 threads a launch.  (One beyond it, in parts, would be faster here than in 128-row
    // workgroups; nothing near such sizes has been measured.)
    const int64_t tiles = (a.c + OWN - 1) / OWN, owners = (int64_t)a.n_q * a.B * a.H + (backward ? (int64_t)a.n_kv * a.B * a.H_kv : 0);
    return a.d <= TD && tiles * owners * 64 * (a.d <= 64 ? WAVES_OF<64> : WAVES_OF<128>) < (int64_t(1) << 32);
}

hipError_t launch_f32x3_split(const StepArgs& a, bool backward, hipStream_t st) {
    if (a.d <= 32) return run<32>(a, backward, st);
    return a.d <= 64 ? run<64>(a, backward, st) : run<128>(a, backward, st);
}

}  // namespace sa
