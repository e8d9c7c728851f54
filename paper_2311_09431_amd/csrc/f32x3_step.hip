// Ring-step kernels for fp32 operands on the bf16 matrix cores, head dimension up to 128, launches
// with enough 128-row workgroups to fill the chip (fewer: f32x3_split.hip; the rule: f32_route.hip).
//
// The fp32 matrix cores run at a sixteenth of the bf16 rate.  A fp32 number is the sum of three
// bf16 ones (each the rounding of what the ones before leave: 3 x 8 bits and two signs cover its 24
// bits), and a product of two such sums needs six of the nine bf16 products: the three dropped
// ones, mid x lo twice and lo x lo, are below 2^-26 of the whole, a quarter of fp32's own rounding.  So
// every product of the step is six v_mfma_f32_32x32x16_bf16 with fp32 accumulation, six
// sixteenths of the time of the fp32 instruction.  Error against 64 bits (2-norm of the error over
// that of the result; one head, 2048 tokens, d 128), fp32 instruction -> here: O 3.7e-7 -> 1.8e-7,
// dQ 5.4e-7 -> 3.3e-7, dK 7.1e-7 -> 3.7e-7, dV 6.4e-7 -> 3.4e-7.  Whole ring, 16 heads, d 128,
// 4 x 2048 tokens, forward + backward: 12.1 -> 6.5 ms.
//
// Everything else is as in f32_step.hip: transposed scores, a score register is the B operand of
// the product over the streamed rows, one wavefront owns 32 rows (backward: two share 32), four (eight)
// make a workgroup.  The owned rows sit in registers as three bf16 operands; the streamed ones go global -> registers
// (a tile ahead) -> split -> three swizzled bf16 planes in LDS, two buffers, one barrier per 32-row
// tile (backward: two).
#include "f32_rows.h"
#include "f32_terms.h"
#include "f32x3_parts.h"
#include "sa_internal.h"

namespace sa {

namespace {

constexpr int TILE = 32;
constexpr int PLANE = TILE * 256, OPERAND = 3 * PLANE, BUFFER = 2 * OPERAND;

// Wavefronts of a workgroup.  Eight share the splitting of a tile and hide each other's latency,
// which the forward kernel's registers allow (256 a wavefront): whole ring above, forward, 2.09 ms
// with four, 1.57 with eight; but 0.23 against 0.29 where eight leave half of the chip idle
// (256 row tiles of 128).

__device__ inline f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

// 8 consecutive floats of a row from column col on, zeros from column d on (d a multiple of 4)
struct Chunk { float4 a, b; };
__device__ inline Chunk load_chunk(const float* row, int col, int d, bool ok) {
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    Chunk x = {z, z};
    if (ok && col < d) x.a = *reinterpret_cast<const float4*>(row + col);
    if (ok && col + 4 < d) x.b = *reinterpret_cast<const float4*>(row + col + 4);
    return x;
}
__device__ inline void split_chunk(const Chunk& x, bf16x8 (&o)[3]) {
    const float v[8] = {x.a.x, x.a.y, x.a.z, x.a.w, x.b.x, x.b.y, x.b.z, x.b.w};
    split8(v, o);
}
// a b = hi + lo: the leading product, and the five others smallest first
__device__ inline void mfma6(const bf16x8 (&a)[3], const bf16x8 (&b)[3], f32x16& hi, f32x16& lo) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        f32x16& c = i == LEADING ? hi : lo;
        c = mfma(a[TERM_A[i]], b[TERM_B[i]], c);
    }
}

// an owned row as B operands
template <int KS>
__device__ inline void load_row(bf16x8x3 (&f)[KS], const float* row, int h, int d) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) split_chunk(load_chunk(row, 16 * ks + 8 * h, d, true), f[ks]);
}

// What a thread stages of a tile: chunks tid, tid + THREADS, ... of 8 columns, row-major
template <int DP, int WAVES>
struct Staged {
    static constexpr int PER_ROW = DP / 8, CHUNKS = TILE * PER_ROW, THREADS = 64 * WAVES;
    static constexpr int N = (CHUNKS + THREADS - 1) / THREADS;
    static constexpr bool SOME_IDLE = CHUNKS % THREADS != 0;
    Chunk x[N];
    __device__ inline void fetch(const float* m, int64_t ss, int first, int c, int d) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int at = (int)threadIdx.x + i * THREADS, row = first + at / PER_ROW;
            if (SOME_IDLE && at >= CHUNKS) continue;
            x[i] = load_chunk(m + (int64_t)min(row, c - 1) * ss, 8 * (at % PER_ROW), d, row < c);
        }
    }
    __device__ inline void put(char* lds) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int at = (int)threadIdx.x + i * THREADS, row = at / PER_ROW, chunk = at % PER_ROW;
            if (SOME_IDLE && at >= CHUNKS) continue;
            bf16x8 o[3];
            split_chunk(x[i], o);
            char* to = lds + row * 256 + ((chunk ^ dt_swz(row)) << 4);
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<bf16x8*>(to + p * PLANE) = o[p];
        }
    }
};

struct Lane {
    int lane, n, h, wave;
    uint32_t arow[8], tr0[4], tr1[4];
    __device__ Lane() {
        lane = threadIdx.x & 63;
        n = lane & 31;
        h = lane >> 5;
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        dt_row_addrs<TD>(arow, n, h);
        dt_tr_addrs<TD>(tr0, tr1, lane);
    }
};

// 32 x 32 scores: rows = the tile at `planes`, columns = the wavefront's owned rows.  NaN where an
// operand is infinite or rounds to an infinite hi (its other terms are NaN).
template <int KS>
__device__ inline f32x16 scores(const char* planes, const bf16x8x3 (&f)[KS], const Lane& ln) {
    f32x16 hi = zero16(), lo = zero16();
    bf16x8x3 a[KS];
    auto read = [&](int ks) {
#pragma unroll
        for (int p = 0; p < 3; ++p) a[ks][p] = dt_read_row(planes + p * PLANE, ln.arow[ks]);
    };
    read(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        __builtin_amdgcn_sched_barrier(0);          // (all reads at once: registers)
        if (ks + 1 < KS) read(ks + 1);
        mfma6(a[ks], f[ks], hi, lo);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) hi[r] += lo[r];
    return hi;
}
// the terms of a weight tile, as B operands of a product over its rows
__device__ __forceinline__ void terms_of(bf16x8x3 (&b)[2], const f32x16& w) {
#pragma unroll
    for (int g = 0; g < 2; ++g) split_tile(w, 8 * g, b[g]);
}
// acc (NB 32-column blocks x owned rows) += tile^T w; tr0, tr1: the lane's transposing reads of these blocks.  The
// tile's sum is formed by itself and added once: the instruction does not round its sums to nearest, and against the
// accumulator's magnitude that error is larger than the fp32 instruction's (dV of 2048 rows: 8.5e-7 against
// 6.4e-7; this way 3.4e-7).
template <int NB>
__device__ inline void accumulate(f32x16 (&acc)[NB], const char* planes, const bf16x8x3 (&b)[2], const uint32_t* tr0, const uint32_t* tr1) {
    bf16x8x3 a[2 * NB];
    auto read = [&](int i, int p) {
        a[i][p] = dt_read_tr(planes + p * PLANE + i % 2 * 16 * 256, tr0[i / 2], tr1[i / 2]);
    };
    read(0, 1);
    read(0, 2);
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) {
        f32x16 t = zero16();
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int i = 2 * mb + g;
            __builtin_amdgcn_sched_barrier(0);          // (all reads at once: registers)
            read(i, 0);
            t = mfma(a[i][TERM_A[0]], b[g][TERM_B[0]], t);
            t = mfma(a[i][TERM_A[1]], b[g][TERM_B[1]], t);
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < 2 * NB) read(i + 1, 2);
#pragma unroll
            for (int j = 2; j < 5; ++j) t = mfma(a[i][TERM_A[j]], b[g][TERM_B[j]], t);
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < 2 * NB) read(i + 1, 1);
            t = mfma(a[i][TERM_A[5]], b[g][TERM_B[5]], t);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mb][r] += t[r];
    }
}

// The walk of a query-owning workgroup over the 32-key tiles of its shards, q0 its first query:
// body(k, v, key0, full, off) on one tile.
template <int DP, int WAVES, typename Body>
__device__ inline void walk_keys(const StepArgs& p, int dev, int q0, int64_t kv_base, char* lds, Body body) {
    const int kv_end = last_shard(p, dev), q_last = min(q0 + 32 * WAVES, p.c) - 1;
    const float* K = (const float*)p.k + kv_base;
    const float* V = (const float*)p.v + kv_base;
    Staged<DP, WAVES> sk, sv;
    // tile after tile of the walk: `ahead` is the next one to fetch
    int kv_a = p.kv_dev, t_a = 0;
    auto last_key = [&](int kv) {
        return block_kind(dev, kv, p.layout) == MASK_FULL ? p.c - 1 : q_last - block_off(dev, kv, p.layout);
    };
    auto fetch = [&]() {
        sk.fetch(K + (kv_a - p.kv_dev) * p.kv_shard, p.kv_stride_s, t_a, p.c, p.d);
        sv.fetch(V + (kv_a - p.kv_dev) * p.kv_shard, p.kv_stride_s, t_a, p.c, p.d);
        t_a += TILE;
        if (t_a > last_key(kv_a)) {
            t_a = 0;
            ++kv_a;
        }
    };
    int kv = kv_a, t0 = t_a, parity = 0;
    fetch();
    sk.put(lds);
    sv.put(lds + OPERAND);
    for (;;) {
        const int kv_n = kv_a, t_n = t_a;
        const bool more = kv_n < kv_end;
        if (more) fetch();
        __syncthreads();                // this tile is written, the other buffer read
        const char* k = lds + parity * BUFFER;
        body(k, k + OPERAND, t0, block_kind(dev, kv, p.layout) == MASK_FULL, block_off(dev, kv, p.layout));
        if (!more) break;
        char* to = lds + (1 - parity) * BUFFER;
        sk.put(to);
        sv.put(to + OPERAND);
        kv = kv_n;
        t0 = t_n;
        parity ^= 1;
    }
}

// ------------------------------------------------------------------ forward
template <int DP, int WAVES>
__global__ void __launch_bounds__(64 * WAVES, WAVES / 4)
fwd_f32x3_kernel(StepArgs p, int n_tiles) {
    constexpr int KS = ksteps_of(DP), NB = blocks_of(DP);
    __shared__ __attribute__((aligned(1024))) char lds[2 * BUFFER];

    const Lane ln;
    const int n = ln.n, h = ln.h;
    int rank, bh, dev_rank;
    decode((int)blockIdx.x, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * 32 * WAVES, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;

    const int a_own = q0 + 32 * ln.wave + n, a = min(a_own, p.c - 1);
    bf16x8x3 qf[KS];
    load_row<KS>(qf, (const float*)p.q + base + (int64_t)a * p.stride_s, h, d);
    float* L = p.lse + b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c + a;
    const float old = p.fresh ? -INFINITY : *L;
    f32x16 acc[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) acc[mb] = zero16();
    const Scale2 kappa(p.scale);
    float m = -INFINITY, l = 0.f;           // m in base-2 units; l: this half-wave's share of the row sum

    walk_keys<DP, WAVES>(p, dev, q0, kv_base, lds, [&](const char* k, const char* v, int key0, bool full, int off) {
        const int wave_last = full ? p.c - 1 : min(q0 + 32 * ln.wave + 31, p.c - 1) - off;
        if (key0 > wave_last) return;
        const int lane_last = (full ? p.c - 1 : a - off) - key0;
        f32x16 x = scores<KS>(k, qf, ln);
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            x[r] = reg_row(r, h) <= lane_last ? x[r] : -INFINITY;
            mx = fmaxf(mx, x[r]);
        }
        const float m_new = fmaxf(m, half_wave_max(mx) * kappa.hi);         // base 2
        const float ref = m_new == -INFINITY ? 0.f : m_new;                 // a row without a key so far
        const float alpha = __builtin_amdgcn_exp2f(m - ref);
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            x[r] = kappa.exp2(x[r], ref, 0.f);
            sum += x[r];
        }
        l = l * alpha + sum;
        if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {
#pragma unroll
            for (int mb = 0; mb < NB; ++mb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mb][r] *= alpha;
        }
        m = m_new;
        bf16x8x3 w[2];
        terms_of(w, x);
        accumulate<NB>(acc, v, w, ln.tr0, ln.tr1);
    });

    // fold the partial result into the running (O, LSE)
    const float l_tot = half_wave_sum(l);
    const float part = l_tot > 0.f ? fmaf(m, LN2_HI, fmaf(m, LN2_LO, logf(l_tot))) : -INFINITY;
    const float top = fmaxf(old, part);
    // a row sum that is no positive number although the row sees a key: see f32_rows.h
    const uint32_t odd_rows =
        row_mask(a_own < p.c && (not_finite<NB>(acc) || (!(l_tot > 0.f && l_tot < INFINITY) && sees_a_key(p, dev, a)))) |
        faint_rows(loudest<NB>(acc), a_own < p.c);
    // no row here, or no key seen: state unchanged
    if (a_own < p.c && !((odd_rows >> n) & 1) && (part != -INFINITY || p.fresh)) {
        const float ref = top == -INFINITY ? 0.f : top;
        const float w_old = expf(old - ref), w_part = expf(part - ref), w_sum = w_old + w_part;
        const float inv = w_sum > 0.f ? 1.f / w_sum : 0.f;
        const float f_old = w_old * inv, f_part = l_tot > 0.f ? w_part * inv / l_tot : 0.f;
        float* O = p.o + base + (int64_t)a * p.stride_s;
#pragma unroll
        for (int mb = 0; mb < NB; ++mb)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = 32 * mb + 8 * g + 4 * h;
                if (col >= d) continue;
                float4* dst = reinterpret_cast<float4*>(O + col);
                float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
                if (f_old != 0.f) {
                    x = *dst;
                    x.x *= f_old; x.y *= f_old; x.z *= f_old; x.w *= f_old;
                }
                x.x = fmaf(acc[mb][4 * g + 0], f_part, x.x); x.y = fmaf(acc[mb][4 * g + 1], f_part, x.y);
                x.z = fmaf(acc[mb][4 * g + 2], f_part, x.z); x.w = fmaf(acc[mb][4 * g + 3], f_part, x.w);
                *dst = x;
            }
        if (h == 0) *L = top + logf(w_sum);
    }
    each_row<1>(odd_rows, 0, [&](const StepArgs& again, int i) { fwd_row<float>(again, b, hd, dev_i, q0 + 32 * ln.wave + i, ln.lane); });
}

// scale * acc to this lane's row, added to what is there unless fresh
template <int NB>
__device__ inline void add_rows(float* row, const f32x16 (&acc)[NB], float scale, int col0, int d, int h, bool fresh) {
#pragma unroll
    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = col0 + 32 * mb + 8 * g + 4 * h;
            if (col >= d) continue;
            float4* dst = reinterpret_cast<float4*>(row + col);
            float4 x = fresh ? make_float4(0.f, 0.f, 0.f, 0.f) : *dst;
            x.x = fmaf(scale, acc[mb][4 * g + 0], x.x); x.y = fmaf(scale, acc[mb][4 * g + 1], x.y);
            x.z = fmaf(scale, acc[mb][4 * g + 2], x.z); x.w = fmaf(scale, acc[mb][4 * g + 3], x.w);
            *dst = x;
        }
}

// ----------------------------------------------------------------- backward
// Two wavefronts share 32 owned rows (w and w + 4, of one SIMD): one forms the scores and the probabilities, the other
// dP, each with the owned operand for that in its registers; they exchange tiles through LDS.  By itself a wavefront
// takes the terms of two owned operands and, key-owning, two accumulators, 320 registers beside all others: one to a
// SIMD, nothing beside its products but what is in its own stream, and 200 to 330 registers copied a tile.
// Whole ring of 4 x 2048 tokens, 16 heads, d 128, backward (time of the kernel): 6.65 -> 5.81 ms.
constexpr int GROUPS = 4;
struct Exchange {
    char* at;                   // a 32 x 32 tile of this pair's [4 registers][lane]
    __device__ Exchange(char* tiles, int group, int lane) : at(tiles + group * 4096 + lane * 16) {}
    __device__ __forceinline__ void put(const f32x16& x) const {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<float4*>(at + i * 1024) = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
    }
    __device__ __forceinline__ f32x16 get() const {
        f32x16 x;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 y = *reinterpret_cast<const float4*>(at + i * 1024);
            x[4 * i] = y.x; x[4 * i + 1] = y.y; x[4 * i + 2] = y.z; x[4 * i + 3] = y.w;
        }
        return x;
    }
};
constexpr int EXCHANGED = 2 * GROUPS * 4096;
// rows that either wavefront of a pair names, and, if all are faint in what both hold of them, those with something
__device__ inline uint32_t odd_of_pair(uint32_t* masks, uint32_t odd, uint32_t some, uint32_t loud, int wave, int lane) {
    if (lane == 0) {
        masks[wave] = odd;
        masks[2 * GROUPS + wave] = some;
        masks[4 * GROUPS + wave] = loud;
    }
    __syncthreads();
    const uint32_t* const own = masks + wave % GROUPS;
    auto either = [&](int i) { return own[2 * GROUPS * i] | own[2 * GROUPS * i + GROUPS]; };
    return __builtin_amdgcn_readfirstlane(either(0) | (either(2) ? 0 : either(1)));
}

// dQ.  The pair's wavefronts take half of its columns each.
template <int DP>
__device__ inline void bwd_dq(const StepArgs& p, int n_tiles, int linear, char* lds, char* tiles, uint32_t* masks) {
    constexpr int KS = ksteps_of(DP), NB = blocks_of(DP) / 2;
    const Lane ln;
    const int n = ln.n, h = ln.h, group = ln.wave % GROUPS, role = ln.wave / GROUPS;
    int rank, bh, dev_rank;
    decode(linear, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * 32 * GROUPS, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c;

    const int a_own = q0 + 32 * group + n, a = min(a_own, p.c - 1);
    bf16x8x3 own[KS];
    load_row<KS>(own, (const float*)(role ? p.dout : p.q) + base + (int64_t)a * p.stride_s, h, d);
    const float delta = p.delta[sbase + a];
    const Scale2 kappa(p.scale);
    float lse, lse_lo;
    to_base2(p.lse[sbase + a], lse, lse_lo);
    uint32_t tr0[NB], tr1[NB];
    f32x16 acc[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) {
        acc[mb] = zero16();
        tr0[mb] = role ? ln.tr0[NB + mb] : ln.tr0[mb];
        tr1[mb] = role ? ln.tr1[NB + mb] : ln.tr1[mb];
    }
    const Exchange own_tile(tiles + role * GROUPS * 4096, group, ln.lane), others_tile(tiles + (1 - role) * GROUPS * 4096, group, ln.lane);

    const int kv_end = last_shard(p, dev), q_last = min(q0 + 32 * GROUPS, p.c) - 1;
    Staged<DP, 2 * GROUPS> sk, sv;
    int kv_a = p.kv_dev, t_a = 0;               // the next tile to fetch
    auto fetch = [&]() {
        sk.fetch((const float*)p.k + kv_base + (kv_a - p.kv_dev) * p.kv_shard, p.kv_stride_s, t_a, p.c, d);
        sv.fetch((const float*)p.v + kv_base + (kv_a - p.kv_dev) * p.kv_shard, p.kv_stride_s, t_a, p.c, d);
        t_a += TILE;
        if (t_a > (block_kind(dev, kv_a, p.layout) == MASK_FULL ? p.c - 1 : q_last - block_off(dev, kv_a, p.layout))) {
            t_a = 0;
            ++kv_a;
        }
    };
    int kv = kv_a, t0 = t_a, parity = 0;
    fetch();
    sk.put(lds);
    sv.put(lds + OPERAND);
    int kv_n = kv_a, t_n = t_a;                 // the tile behind the present one, on its way
    if (kv_n < kv_end) fetch();
    for (;;) {
        __syncthreads();                // this tile is written, the other buffer and the exchanged tiles read
        const char* k = lds + parity * BUFFER;
        const bool full = block_kind(dev, kv, p.layout) == MASK_FULL;
        const int off = block_off(dev, kv, p.layout);
        const bool active = t0 <= (full ? p.c - 1 : min(q0 + 32 * group + 31, p.c - 1) - off);
        const int kv_nn = kv_a, t_nn = t_a;
        auto stage = [&]() {
            sk.put(lds + (1 - parity) * BUFFER);
            sv.put(lds + (1 - parity) * BUFFER + OPERAND);
            if (kv_nn < kv_end) fetch();
        };
        if (role != 0) stage();
        f32x16 x;
        if (active) {
            x = scores<KS>(k + role * OPERAND, own, ln);
            if (role == 0) {
                const int lane_last = (full ? p.c - 1 : a - off) - t0;
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = kappa.exp2(x[r], lse, lse_lo);
                if (t0 + 31 > (full ? p.c - 1 : min(q0 + 32 * group, p.c) - 1 - off)) {        // some pair is masked
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[r] = reg_row(r, h) <= lane_last ? x[r] : 0.f;
                }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] -= delta;
            }
            own_tile.put(x);
        }
        meet();
        if (active) {
            const f32x16 y = others_tile.get();
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] *= y[r];
            bf16x8x3 w[2];
            terms_of(w, x);
            accumulate<NB>(acc, k, w, tr0, tr1);
        }
        if (kv_n >= kv_end) break;
        if (role == 0) stage();
        kv = kv_n;
        t0 = t_n;
        kv_n = kv_nn;
        t_n = t_nn;
        parity ^= 1;
    }
    const float top = loudest<NB>(acc);
    const uint32_t odd_rows = odd_of_pair(masks, row_mask(a_own < p.c && not_finite<NB>(acc)), row_mask(a_own < p.c && top > 0.f),
                                          row_mask(top >= FAINT), ln.wave, ln.lane);
    if (a_own < p.c && !((odd_rows >> n) & 1))
        add_rows<NB>(p.dq + base + (int64_t)a * p.stride_s, acc, p.scale, 32 * NB * role, d, h, p.fresh);
    each_row<2>(odd_rows, role, [&](const StepArgs& again, int i) { dq_row<float>(again, b, hd, dev_i, q0 + 32 * group + i, ln.lane); });
}

// dK (by the wavefront that forms dP) and dV (by the one that forms the probabilities).  Owned rows are keys, streamed
// rows queries; the query heads of the group that shares the key/value head and the query shards that see it come one
// after the other.
template <int DP>
__device__ inline void bwd_dkdv(const StepArgs& p, int n_tiles, int linear, char* lds, char* tiles, float* stats, uint32_t* masks) {
    constexpr int KS = ksteps_of(DP), NB = blocks_of(DP);
    const Lane ln;
    const int n = ln.n, h = ln.h, tid = threadIdx.x, group = ln.wave % GROUPS, role = ln.wave / GROUPS;
    int tile, bh, dev_i;                                // low key tiles see most queries: first
    decode(linear, p.B * p.H_kv, tile, bh);
    decode_rank(tile, n_tiles, p.n_kv, p.layout, tile, dev_i);
    const int k0 = tile * 32 * GROUPS, dev = p.kv_dev + dev_i;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv, members = p.H / p.H_kv, d = p.d;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + dev_i * p.kv_shard;

    const int key_own = k0 + 32 * group + n, key = min(key_own, p.c - 1);
    const int64_t row = kv_base + (int64_t)key * p.kv_stride_s;
    const Scale2 kappa(p.scale);
    bf16x8x3 own[KS];
    load_row<KS>(own, (const float*)(role ? p.v : p.k) + row, h, d);
    f32x16 acc[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) acc[mb] = zero16();
    const Exchange probabilities(tiles, group, ln.lane);

    // contiguous layout: earlier devices' queries see nothing of these keys
    const int q_dev0 = p.layout == SA_STRIPED ? p.q_dev : max(p.q_dev, dev);
    auto first_tile = [&](int q_dev) {
        return block_kind(q_dev, dev, p.layout) == MASK_FULL ? 0 : (k0 + block_off(q_dev, dev, p.layout)) / TILE * TILE;
    };
    Staged<DP, 2 * GROUPS> sq, sg;
    float stat = 0.f;           // LSE (threads 0 .. 31) or delta (32 .. 63) of a row of the tile
    int member_a = 0, dev_a = q_dev0, t_a = first_tile(q_dev0);
    auto fetch = [&]() {
        const int hd = kvh * members + member_a;
        const int64_t base = b * p.stride_b + hd * p.stride_h + (dev_a - p.q_dev) * p.q_shard;
        sq.fetch((const float*)p.q + base, p.stride_s, t_a, p.c, d);
        sg.fetch((const float*)p.dout + base, p.stride_s, t_a, p.c, d);
        if (tid < 2 * TILE) {
            const int64_t at = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(dev_a - p.q_dev) * p.c +
                               min(t_a + tid % TILE, p.c - 1);
            stat = tid < TILE ? p.lse[at] : p.delta[at];
        }
        t_a += TILE;
        // a tile row may lie beyond the shard (last tile of a block) but a tile may not
        if (t_a >= p.c) {
            if (++dev_a == p.q_dev + p.n_q) {
                dev_a = q_dev0;
                ++member_a;
            }
            t_a = first_tile(dev_a);
        }
    };
    auto put = [&](int parity) {
        sq.put(lds + parity * BUFFER);
        sg.put(lds + parity * BUFFER + OPERAND);
        float* st = stats + parity * 3 * TILE;
        if (tid < TILE) to_base2(stat, st[tid], st[TILE + tid]);
        else if (tid < 2 * TILE) st[TILE + tid] = stat;
    };
    // keys whose first query lies beyond the shard (last key, off = 1) start at row c: nothing there
    // is in the mask, and rows beyond the shard read as zeros
    int q_dev = dev_a, t0 = t_a, parity = 0;
    fetch();
    put(0);
    int dev_n = dev_a, t_n = t_a;               // the tile behind the present one, on its way if there is one
    bool more = member_a < members;
    if (more) fetch();
    for (;;) {
        __syncthreads();                // this tile is written, the other buffer and the exchanged tiles read
        const int dev_nn = dev_a, t_nn = t_a;
        const bool more_n = member_a < members;
        auto stage = [&]() {
            put(1 - parity);
            if (more_n) fetch();
        };
        // one splits the next tile ahead of its products, the other behind them, so that the matrix core has work
        if (role != 0) stage();
        const bool full = block_kind(q_dev, dev, p.layout) == MASK_FULL;
        const int off = block_off(q_dev, dev, p.layout);
        const char* q = lds + parity * BUFFER;
        const float* st = stats + parity * 3 * TILE;
        const bool active = full || t0 + 31 >= k0 + 32 * group + off;
        f32x16 x;
        bf16x8x3 w[2];
        if (active) {
            x = scores<KS>(q + role * OPERAND, own, ln);
            if (role == 0) {
                const int lane_first = (full ? 0 : key_own + off) - t0, rows = p.c - t0;
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = kappa.exp2(x[r], st[reg_row(r, h)], st[TILE + reg_row(r, h)]);
                if (t0 < (full ? 0 : k0 + 32 * group + 31 + off) || rows < TILE) {        // some pair is masked
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[r] = reg_row(r, h) >= lane_first && reg_row(r, h) < rows ? x[r] : 0.f;
                }
                probabilities.put(x);
                terms_of(w, x);
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] -= st[2 * TILE + reg_row(r, h)];
            }
        }
        meet();
        if (active) {
            if (role != 0) {
                const f32x16 pr = probabilities.get();
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] *= pr[r];
                terms_of(w, x);
            }
            accumulate<NB>(acc, q + (1 - role) * OPERAND, w, ln.tr0, ln.tr1);
        }
        if (!more) break;
        if (role == 0) stage();
        parity ^= 1;
        q_dev = dev_n;
        t0 = t_n;
        dev_n = dev_nn;
        t_n = t_nn;
        more = more_n;
    }
    // (each has all columns of its result)
    const uint32_t odd_rows = odd_of_pair(masks, row_mask(key_own < p.c && not_finite<NB>(acc)) |
                                                     faint_rows(loudest<NB>(acc), key_own < p.c), 0, 0, ln.wave, ln.lane);
    if (key_own < p.c && !((odd_rows >> n) & 1))
        add_rows<NB>((role ? p.dk : p.dv) + row, acc, role ? p.scale : 1.f, 0, d, h, p.fresh);
    each_row<2>(odd_rows, role, [&](const StepArgs& again, int i) { dkdv_row<float>(again, b, kvh, dev_i, k0 + 32 * group + i, 0, d, ln.lane); });
}

// Both in one launch, the kind with the longer walks first (they share nothing but the inputs; one compute unit each, so
// the second kind fills the tail of the first).
template <int DP>
__global__ void __launch_bounds__(64 * 2 * GROUPS, 2)
bwd_f32x3_kernel(StepArgs p, int n_tiles, int n_first, bool keys_first) {
    __shared__ __attribute__((aligned(1024))) char lds[2 * BUFFER];
    __shared__ __attribute__((aligned(1024))) char tiles[EXCHANGED];
    __shared__ float stats[2 * 3 * TILE];          // [buffer][LSE hi | LSE lo | delta][row]
    __shared__ uint32_t masks[6 * GROUPS];
    const bool first = (int)blockIdx.x < n_first;
    const int linear = first ? (int)blockIdx.x : (int)blockIdx.x - n_first;
    if (first == keys_first) bwd_dkdv<DP>(p, n_tiles, linear, lds, tiles, stats, masks);
    else bwd_dq<DP>(p, n_tiles, linear, lds, tiles, masks);
}

// The same with both operands and accumulators in one wavefront, above 64 columns: no exchange, and triangular blocks,
// where a wavefront has work in some of the tiles only, cost less.  Faster for many heads of one or two tiles
// (f32_route.hip: 128 heads of 128 rows, d 128, 58 : 46 us; 32 of 700 143 : 161).
constexpr int ALONE = 4;
template <int DP>
__device__ inline void bwd_dq_alone(const StepArgs& p, int n_tiles, int linear, char* lds) {
    constexpr int KS = ksteps_of(DP), NB = blocks_of(DP);
    const Lane ln;
    const int n = ln.n, h = ln.h;
    int rank, bh, dev_rank;
    decode(linear, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * 32 * ALONE, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c;

    const int a_own = q0 + 32 * ln.wave + n, a = min(a_own, p.c - 1);
    bf16x8x3 qf[KS], gf[KS];
    load_row<KS>(qf, (const float*)p.q + base + (int64_t)a * p.stride_s, h, d);
    load_row<KS>(gf, (const float*)p.dout + base + (int64_t)a * p.stride_s, h, d);
    const float delta = p.delta[sbase + a];
    const Scale2 kappa(p.scale);
    float lse, lse_lo;
    to_base2(p.lse[sbase + a], lse, lse_lo);
    f32x16 acc[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) acc[mb] = zero16();

    walk_keys<DP, ALONE>(p, dev, q0, kv_base, lds, [&](const char* k, const char* v, int key0, bool full, int off) {
        const int wave_last = full ? p.c - 1 : min(q0 + 32 * ln.wave + 31, p.c - 1) - off;
        if (key0 > wave_last) return;
        const int lane_last = (full ? p.c - 1 : a - off) - key0;
        f32x16 x = scores<KS>(k, qf, ln);
        const f32x16 dp = scores<KS>(v, gf, ln);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float pr = reg_row(r, h) <= lane_last ? kappa.exp2(x[r], lse, lse_lo) : 0.f;
            x[r] = pr * (dp[r] - delta);
        }
        bf16x8x3 w[2];
        terms_of(w, x);
        accumulate<NB>(acc, k, w, ln.tr0, ln.tr1);
    });
    const uint32_t odd_rows = row_mask(a_own < p.c && not_finite<NB>(acc)) | faint_rows(loudest<NB>(acc), a_own < p.c);
    if (a_own < p.c && !((odd_rows >> n) & 1))
        add_rows<NB>(p.dq + base + (int64_t)a * p.stride_s, acc, p.scale, 0, d, h, p.fresh);
    each_row<1>(odd_rows, 0, [&](const StepArgs& again, int i) { dq_row<float>(again, b, hd, dev_i, q0 + 32 * ln.wave + i, ln.lane); });
}
template <int DP>
__device__ inline void bwd_dkdv_alone(const StepArgs& p, int n_tiles, int linear, char* lds, float* stats) {
    constexpr int KS = ksteps_of(DP), NB = blocks_of(DP);
    const Lane ln;
    const int n = ln.n, h = ln.h, tid = threadIdx.x;
    int tile, bh, dev_i;                                // low key tiles see most queries: first
    decode(linear, p.B * p.H_kv, tile, bh);
    decode_rank(tile, n_tiles, p.n_kv, p.layout, tile, dev_i);
    const int k0 = tile * 32 * ALONE, dev = p.kv_dev + dev_i;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv, members = p.H / p.H_kv, d = p.d;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + dev_i * p.kv_shard;

    const int key_own = k0 + 32 * ln.wave + n, key = min(key_own, p.c - 1);
    const int64_t row = kv_base + (int64_t)key * p.kv_stride_s;
    const Scale2 kappa(p.scale);
    bf16x8x3 kf[KS], vf[KS];
    load_row<KS>(kf, (const float*)p.k + row, h, d);
    load_row<KS>(vf, (const float*)p.v + row, h, d);
    f32x16 acck[NB], accv[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) acck[mb] = accv[mb] = zero16();

    // (tiles and their statistics as in bwd_dkdv)
    const int q_dev0 = p.layout == SA_STRIPED ? p.q_dev : max(p.q_dev, dev);
    auto first_tile = [&](int q_dev) {
        return block_kind(q_dev, dev, p.layout) == MASK_FULL ? 0 : (k0 + block_off(q_dev, dev, p.layout)) / TILE * TILE;
    };
    Staged<DP, ALONE> sq, sg;
    float stat = 0.f;
    int member_a = 0, dev_a = q_dev0, t_a = first_tile(q_dev0);
    auto fetch = [&]() {
        const int hd = kvh * members + member_a;
        const int64_t base = b * p.stride_b + hd * p.stride_h + (dev_a - p.q_dev) * p.q_shard;
        sq.fetch((const float*)p.q + base, p.stride_s, t_a, p.c, d);
        sg.fetch((const float*)p.dout + base, p.stride_s, t_a, p.c, d);
        if (tid < 2 * TILE) {
            const int64_t at = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(dev_a - p.q_dev) * p.c +
                               min(t_a + tid % TILE, p.c - 1);
            stat = tid < TILE ? p.lse[at] : p.delta[at];
        }
        t_a += TILE;
        if (t_a >= p.c) {
            if (++dev_a == p.q_dev + p.n_q) {
                dev_a = q_dev0;
                ++member_a;
            }
            t_a = first_tile(dev_a);
        }
    };
    auto put = [&](int parity) {
        sq.put(lds + parity * BUFFER);
        sg.put(lds + parity * BUFFER + OPERAND);
        float* st = stats + parity * 3 * TILE;
        if (tid < TILE) to_base2(stat, st[tid], st[TILE + tid]);
        else if (tid < 2 * TILE) st[TILE + tid] = stat;
    };
    int q_dev = dev_a, t0 = t_a, parity = 0;
    fetch();
    put(0);
    for (;;) {
        const int dev_n = dev_a, t_n = t_a;
        const bool more = member_a < members;
        if (more) fetch();
        __syncthreads();                // this tile is written, the other buffer read
        const bool full = block_kind(q_dev, dev, p.layout) == MASK_FULL;
        const int off = block_off(q_dev, dev, p.layout);
        if (full || t0 + 31 >= k0 + 32 * ln.wave + off) {
            const char* q = lds + parity * BUFFER;
            const float* st = stats + parity * 3 * TILE;
            const int lane_first = (full ? 0 : key_own + off) - t0, rows = p.c - t0;
            const f32x16 x = scores<KS>(q, kf, ln);
            f32x16 dp = scores<KS>(q + OPERAND, vf, ln), pr;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = reg_row(r, h);
                pr[r] = i >= lane_first && i < rows ? kappa.exp2(x[r], st[i], st[TILE + i]) : 0.f;
                dp[r] = pr[r] * (dp[r] - st[2 * TILE + i]);
            }
            bf16x8x3 w[2];
            terms_of(w, pr);
            accumulate<NB>(accv, q + OPERAND, w, ln.tr0, ln.tr1);
            terms_of(w, dp);
            accumulate<NB>(acck, q, w, ln.tr0, ln.tr1);
        }
        if (!more) break;
        parity ^= 1;
        put(parity);
        q_dev = dev_n;
        t0 = t_n;
    }
    const bool in_shard = key_own < p.c;
    const uint32_t odd_rows = row_mask(in_shard && (not_finite<NB>(accv) || not_finite<NB>(acck))) |
                              faint_rows(loudest<NB>(accv), in_shard) | faint_rows(loudest<NB>(acck), in_shard);
    if (in_shard && !((odd_rows >> n) & 1)) {
        add_rows<NB>(p.dv + row, accv, 1.f, 0, d, h, p.fresh);
        add_rows<NB>(p.dk + row, acck, p.scale, 0, d, h, p.fresh);
    }
    each_row<1>(odd_rows, 0, [&](const StepArgs& again, int i) { dkdv_row<float>(again, b, kvh, dev_i, k0 + 32 * ln.wave + i, 0, d, ln.lane); });
}
template <int DP>
__global__ void __launch_bounds__(64 * ALONE, 1)
bwd_f32x3_alone_kernel(StepArgs p, int n_tiles, int n_dkdv) {
    __shared__ __attribute__((aligned(1024))) char lds[2 * BUFFER];
    __shared__ float stats[2 * 3 * TILE];          // [buffer][LSE hi | LSE lo | delta][row]
    if ((int)blockIdx.x < n_dkdv) bwd_dkdv_alone<DP>(p, n_tiles, (int)blockIdx.x, lds, stats);
    else bwd_dq_alone<DP>(p, n_tiles, (int)blockIdx.x - n_dkdv, lds);
}

template <int DP, int WAVES>
hipError_t run_fwd(const StepArgs& a, hipStream_t st) {
    const int rows = 32 * WAVES, n_tiles = (a.c + rows - 1) / rows;
    hipLaunchKernelGGL((fwd_f32x3_kernel<DP, WAVES>), dim3((unsigned)n_tiles * a.n_q * a.B * a.H), dim3(64 * WAVES), 0, st,
                       a, n_tiles);
    return hipGetLastError();
}
template <int DP>
hipError_t run_alone(const StepArgs& a, hipStream_t st) {
    const int rows = 32 * ALONE, n_tiles = (a.c + rows - 1) / rows;
    const int n_dkdv = n_tiles * a.n_kv * a.B * a.H_kv, n_dq = n_tiles * a.n_q * a.B * a.H;
    hipLaunchKernelGGL((bwd_f32x3_alone_kernel<DP>), dim3((unsigned)(n_dkdv + n_dq)), dim3(64 * ALONE), 0, st, a, n_tiles,
                       n_dkdv);
    return hipGetLastError();
}
template <int DP>
hipError_t run(const StepArgs& a, bool backward, hipStream_t st) {
    const int rows = 32 * GROUPS, n_tiles = (a.c + rows - 1) / rows;
    if (!backward) return (int64_t)n_tiles * a.n_q * a.B * a.H >= 512 ? run_fwd<DP, 8>(a, st) : run_fwd<DP, 4>(a, st);
    const int n_dkdv = n_tiles * a.n_kv * a.B * a.H_kv, n_dq = n_tiles * a.n_q * a.B * a.H;
    // one device's queries against more than two shards (d 64: 3 of 2048 tokens, 8 heads, 617 -> 501 us, 4 of 512, 32
    // heads, 215 -> 156; two of 512, 32 heads, d 128, 176 -> 201)
    const bool keys_first = 2 * (int64_t)a.n_q * (a.H / a.H_kv) >= a.n_kv;
    hipLaunchKernelGGL((bwd_f32x3_kernel<DP>), dim3((unsigned)(n_dkdv + n_dq)), dim3(64 * 2 * GROUPS), 0, st, a, n_tiles,
                       keys_first ? n_dkdv : n_dq, keys_first);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_f32x3(const StepArgs& a, bool backward, bool alone, hipStream_t st) {
    if (alone) return run_alone<128>(a, st);
    return a.d <= 64 ? run<64>(a, backward, st) : run<128>(a, backward, st);
}

}  // namespace sa
