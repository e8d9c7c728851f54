// Backward ring step for launches that leave most of the chip idle with 128-row workgroups (bf16
// matrix cores, head dimension up to 128, blocks of at least 128 rows): same operands, same
// products and same precision as bwd_mfma.hip, other split of the work.
//
// What bounds such a launch is the walk of one workgroup: about 1.4 us (dQ) or 1.7 us (dK/dV) per
// 64 streamed rows, however few workgroups there are.  Here a workgroup owns 32 rows and its four
// wavefronts take the 32-row sub-tiles of each 128-row group of the streamed side, one each; the
// partial results meet in LDS at the end.  Four times the workgroups and a walk of about 2 us per
// 128 rows; groups are double buffered, one barrier per group.  Nothing is interleaved by hand and
// a tile load feeds a quarter of the products, so a fuller chip is better served by the other
// kernels (figures at bwd_split_wanted).  Whole ring, 4 x 1024 tokens, 2 heads, forward +
// backward: 272 -> 162 us.  A forward kernel of this form was no faster than the 128-row one
// (37 us both for 2048 x 2048, 2 heads).
//
// Blocks shorter than one tile keep the precision of the fp32 kernels, which take them otherwise:
// EXACT.  Products of bf16 operands are exact in fp32 anyway; probabilities and dS go into theirs as
// three bf16 terms, and the exponents are formed with fp32's own rounding.
//
// The wavefront that takes a sub-tile is given by the sub-tile's place in its shard, so summation
// orders are fixed and the same under emulated coarse skipping.
#include "f32_rows.h"
#include "f32_terms.h"
#include "mfma_tiles.h"
#include "sa_internal.h"

namespace sa {

namespace {

constexpr int WAVES = 4, OWN = 32, GROUP = 32 * WAVES;
template <int DP> constexpr int SUB_BYTES = tile_bytes(DP) / 2;              // 32 rows
template <int DP> constexpr int GROUP_BYTES = 2 * tile_bytes(DP);            // one operand's 128 rows

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

// 128 rows starting at row first of c, as two 64-row tiles (rows beyond the matrix arrive as zeros; a
// second tile beyond it is not read by anyone)
template <int DP>
__device__ inline void load_group(dt_rsrc m, int first, int c, int pitch, char* lds, const uint32_t (&gl)[4], int wave) {
    dt_load<DP>(m, first * pitch, lds, gl, wave);
    if (first + DT_ROWS < c) dt_load<DP>(m, (first + DT_ROWS) * pitch, lds + tile_bytes(DP), gl, wave);
}

__device__ inline f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

// 32 x 32 scores: rows = the sub-tile at `rows`, columns = the owned rows
template <int DP, bool PART>
__device__ inline f32x16 scores(const char* rows, const bf16x8 (&f)[8], const Lane<DP>& ln, int part_ks) {
    f32x16 s = zero16();
#pragma unroll
    for (int ks = 0; ks < ksteps_of(DP); ++ks) {
        const bf16x8 x = dt_read_row(rows, ln.arow[ks]);
        s = mfma(PART ? zero_beyond_d(x, ks == part_ks) : x, f[ks], s);
    }
    return s;
}
// acc (32-column blocks x owned rows) += streamed^T w, w rounded to bf16 or (EXACT) as three terms,
// smallest first
template <int DP, bool EXACT>
__device__ inline void accumulate(f32x16 (&acc)[4], const char* rows, const f32x16& w, const Lane<DP>& ln) {
    constexpr int TERMS = EXACT ? 3 : 1;
    bf16x8 b[2][3];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        if (EXACT) {
            split_regs(w, 8 * g, b[g]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) b[g][0][e] = (__bf16)w[8 * g + e];
        }
    }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int mb = 0; mb < blocks_of(DP); ++mb) {
            const bf16x8 a = dt_read_tr(rows + g * 16 * row_bytes(DP), ln.tr0[mb], ln.tr1[mb]);
#pragma unroll
            for (int t = TERMS - 1; t >= 0; --t) acc[mb] = mfma(a, b[g][t], acc[mb]);
        }
}

// bytes of the four wavefronts' accumulators
template <int DP> constexpr int PARTIAL_BYTES = WAVES * blocks_of(DP) * 16 * 64 * 4;

// Sum of the four wavefronts' accumulators through LDS: each writes its own and takes a share of the
// sum, pieces blocks wave .. of 8 columns (4 a lane), so that a row's columns stay together.
template <int DP>
__device__ inline void put_partial(char* buf, const f32x16 (&acc)[4], const Lane<DP>& ln) {
    float4* mine = reinterpret_cast<float4*>(buf) + ln.wave * blocks_of(DP) * 4 * 64;
#pragma unroll
    for (int mb = 0; mb < blocks_of(DP); ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            mine[(mb * 4 + g) * 64 + ln.lane] =
                make_float4(acc[mb][4 * g], acc[mb][4 * g + 1], acc[mb][4 * g + 2], acc[mb][4 * g + 3]);
}
template <int DP>
__device__ inline float4 take_sum(const char* buf, int piece, const Lane<DP>& ln) {
    const float4* at = reinterpret_cast<const float4*>(buf) + piece * 64 + ln.lane;
    float4 x = at[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
        const float4 y = at[w * blocks_of(DP) * 4 * 64];
        x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
    }
    return x;
}
// EXACT: rows that are done over one by one (f32_rows.h): each wavefront puts its mask beside its
// partial accumulators, and after the barrier takes every fourth of the rows that one of them names
__device__ inline void put_odd(uint32_t* masks, bool odd, int wave, int lane) {
    const uint32_t rows = row_mask(odd);
    if (lane == 0) masks[wave] = rows;
}
__device__ inline uint32_t take_odd(const uint32_t* masks) {
    uint32_t rows = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) rows |= masks[w];
    return __builtin_amdgcn_readfirstlane(rows);
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
// piece i of this wavefront's share and its first column
template <int DP>
__device__ inline int piece_of(int i, const Lane<DP>& ln) { return ln.wave * blocks_of(DP) + i; }
template <int DP>
__device__ inline int column_of(int i, const Lane<DP>& ln) { return 8 * piece_of<DP>(i, ln) + 4 * ln.h; }

// last key of a block that the workgroup of queries q0 .. q0 + 31 looks at: the last allowed one,
// or under emulated coarse skipping the last one of the skip_bk-wide tile that shares an allowed
// pair with its skip_bq-tall tile
__device__ inline int last_key_of(const StepArgs& p, int q0, bool full, int off) {
    if (full) return p.c - 1;
    if (p.skip_bq > 0) {
        const int q_hi = (q0 / p.skip_bq + 1) * p.skip_bq - 1;
        return min(p.c, ((q_hi - off) / p.skip_bk + 1) * p.skip_bk) - 1;
    }
    return min(q0 + OWN, p.c) - 1 - off;
}

// The walk of a query-owning workgroup over the 128-key groups of its shards.  body(k, v, g0):
// one group, its keys at LDS addresses k, v, the first one key g0 of the present block.
struct Block { int kv; bool full; int off, last_key; };
template <int DP, typename Body>
__device__ inline void walk_keys(const StepArgs& p, int dev, int q0, dt_rsrc K, dt_rsrc V, char* lds, const Lane<DP>& ln,
                                 Body body) {
    const int pitch = 2 * (int)p.kv_stride_s, kv_end = last_shard(p, dev);
    uint32_t gl[4];
    dt_load_offsets<DP>(gl, ln.lane, ln.wave, pitch, p.d);
    auto block = [&](int kv) {
        Block b;
        b.kv = kv;
        b.full = block_kind(dev, kv, p.layout) == MASK_FULL;
        b.off = block_off(dev, kv, p.layout);
        b.last_key = last_key_of(p, q0, b.full, b.off);
        return b;
    };
    Block now = block(p.kv_dev);
    int g0 = 0, parity = 0;
    load_group<DP>(K, 0, p.c, pitch, lds, gl, ln.wave);
    load_group<DP>(V, 0, p.c, pitch, lds + GROUP_BYTES<DP>, gl, ln.wave);
    for (;;) {
        Block next = now;
        int next_g0 = g0 + GROUP;
        if (next_g0 > now.last_key) {
            next_g0 = 0;
            next.kv = now.kv + 1;
        }
        const bool more = next.kv < kv_end;
        __builtin_amdgcn_s_waitcnt(0);         // this group has landed (vmcnt) ...
        __syncthreads();                       // ... for every wavefront, and all are done with the last one
        if (more) {
            if (next.kv != now.kv) {
                next = block(next.kv);
                K = dt_advance(K, 2 * p.kv_shard);
                V = dt_advance(V, 2 * p.kv_shard);
            }
            char* to = lds + (1 - parity) * 2 * GROUP_BYTES<DP>;
            load_group<DP>(K, next_g0, p.c, pitch, to, gl, ln.wave);
            load_group<DP>(V, next_g0, p.c, pitch, to + GROUP_BYTES<DP>, gl, ln.wave);
        }
        const char* k = lds + parity * 2 * GROUP_BYTES<DP> + ln.wave * SUB_BYTES<DP>;
        if (g0 + OWN * ln.wave <= now.last_key) body(k, k + GROUP_BYTES<DP>, g0 + OWN * ln.wave, now);
        if (!more) break;
        now = next;
        g0 = next_g0;
        parity ^= 1;
    }
}


// ------------------------------------------------------------------ forward
template <int DP, bool PART>
__global__ void __launch_bounds__(64 * WAVES, DP <= 64 ? 2 : 1)
fwd_split_kernel(StepArgs p, int n_tiles) {
    constexpr int MB = blocks_of(DP);
    // two buffers of K and V; at the end the statistics and four wavefronts' partial results
    __shared__ __attribute__((aligned(1024))) char lds[4 * GROUP_BYTES<DP>];
    static_assert(1024 + PARTIAL_BYTES<DP> <= 4 * GROUP_BYTES<DP>, "partial results");
    __shared__ uint32_t masks[WAVES];

    const Lane<DP> ln;
    const int n = ln.n, h = ln.h;
    int rank, bh, dev_rank;
    decode((int)blockIdx.x, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * OWN, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int pitch = 2 * (int)p.kv_stride_s;

    const int a_own = q0 + n, a = min(a_own, p.c - 1);
    bf16x8 qf[8];
    load_b_frags<8>(qf, (const __bf16*)p.q + base + (int64_t)a * p.stride_s, h, d);
    float* L = p.lse + b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c + a;
    const float old = p.fresh ? -INFINITY : *L;
    const Scale2 kappa(p.scale);
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    float m = -INFINITY, l = 0.f;           // m in base-2 units; l: this half-wave's share of the row sum
    f32x16 acc[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acc[mb] = zero16();

    walk_keys<DP>(p, dev, q0, dt_make_rsrc((const __bf16*)p.k + kv_base, p.c, pitch, d),
              dt_make_rsrc((const __bf16*)p.v + kv_base, p.c, pitch, d), lds, ln,
              [&](const char* k, const char* v, int key0, const Block& blk) {
        f32x16 x = scores<DP, PART>(k, qf, ln, part_ks);
        const int lane_last = (blk.full ? p.c - 1 : a_own - blk.off) - key0;
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            x[r] = reg_row(r, h) <= lane_last ? x[r] : -INFINITY;
            mx = fmaxf(mx, x[r]);
        }
        const float m_new = fmaxf(m, half_wave_max(mx) * kappa.hi);
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
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mb][r] *= alpha;
        }
        m = m_new;
        accumulate<DP, true>(acc, v, x, ln);
    });

    // the four wavefronts' partial results against a common reference
    float* const stats = reinterpret_cast<float*>(lds);                // [wave][m | l][32]
    char* const buf = lds + 1024;
    const float l_own = half_wave_sum(l);
    __syncthreads();
    if (h == 0) {
        stats[ln.wave * 64 + n] = m;
        stats[ln.wave * 64 + 32 + n] = l_own;
    }
    __syncthreads();
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) m_all = fmaxf(m_all, stats[w * 64 + n]);
    const float m_ref = m_all == -INFINITY ? 0.f : m_all;
    float l_tot = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w)
        l_tot += stats[w * 64 + 32 + n] * __builtin_amdgcn_exp2f(stats[w * 64 + n] - m_ref);
    const float f = __builtin_amdgcn_exp2f(m - m_ref);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mb][r] *= f;
    put_partial<DP>(buf, acc, ln);
    // a row sum that is no positive number although the row sees a key: see f32_rows.h
    put_odd(masks, a_own < p.c && (not_finite<MB>(acc) ||
                                   (!(l_tot > 0.f && l_tot < INFINITY) && sees_a_key(p, dev, a))), ln.wave, ln.lane);

    const float part = l_tot > 0.f ? fmaf(m_all, LN2_HI, fmaf(m_all, LN2_LO, logf(l_tot))) : -INFINITY;
    const float top = fmaxf(old, part);
    const float ref = top == -INFINITY ? 0.f : top;
    const float w_old = expf(old - ref), w_part = expf(part - ref), w_sum = w_old + w_part;
    const float inv = w_sum > 0.f ? 1.f / w_sum : 0.f;
    const float f_old = w_old * inv, f_part = l_tot > 0.f ? w_part * inv / l_tot : 0.f;
    float* O = p.o + base + (int64_t)a * p.stride_s;
    float4 o_old[MB];           // on its way while the partial results meet
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        o_old[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (f_old != 0.f && column_of<DP>(i, ln) < d) o_old[i] = *reinterpret_cast<const float4*>(O + column_of<DP>(i, ln));
    }
    __syncthreads();
    const uint32_t odd_rows = take_odd(masks);
    // no row here, or no key seen: state unchanged
    if (a_own < p.c && !((odd_rows >> n) & 1) && (part != -INFINITY || p.fresh)) {
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int col = column_of<DP>(i, ln);
            if (col >= d) continue;
            float4* dst = reinterpret_cast<float4*>(O + col);
            const float4 s = take_sum<DP>(buf, piece_of<DP>(i, ln), ln);
            float4 x = o_old[i];
            x.x *= f_old; x.y *= f_old; x.z *= f_old; x.w *= f_old;
            x.x = fmaf(s.x, f_part, x.x); x.y = fmaf(s.y, f_part, x.y);
            x.z = fmaf(s.z, f_part, x.z); x.w = fmaf(s.w, f_part, x.w);
            *dst = x;
        }
        if (ln.wave == 0 && h == 0) *L = top + logf(w_sum);
    }
    each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { fwd_row<__hip_bfloat16>(again, b, hd, dev_i, q0 + i, ln.lane); });
}

// this wavefront's share of the lane's row as it stands (zeros if not wanted): on its way while the
// partial results meet
template <int DP>
__device__ inline void load_old(float4 (&x)[blocks_of(DP)], const float* row, int d, bool wanted, const Lane<DP>& ln) {
#pragma unroll
    for (int i = 0; i < blocks_of(DP); ++i) {
        x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (wanted && column_of<DP>(i, ln) < d) x[i] = *reinterpret_cast<const float4*>(row + column_of<DP>(i, ln));
    }
}
// x + scale * (sum of the partial results at buf) to the lane's row
template <int DP>
__device__ inline void add_rows(float* row, float4 (&x)[blocks_of(DP)], const char* buf, float scale, int d,
                                const Lane<DP>& ln) {
#pragma unroll
    for (int i = 0; i < blocks_of(DP); ++i) {
        const int col = column_of<DP>(i, ln);
        if (col >= d) continue;
        const float4 s = take_sum<DP>(buf, piece_of<DP>(i, ln), ln);
        x[i].x = fmaf(scale, s.x, x[i].x); x[i].y = fmaf(scale, s.y, x[i].y);
        x[i].z = fmaf(scale, s.z, x[i].z); x[i].w = fmaf(scale, s.w, x[i].w);
        *reinterpret_cast<float4*>(row + col) = x[i];
    }
}

// ----------------------------------------------------------------------- dQ
template <int DP, bool PART, bool EXACT>
__device__ inline void bwd_dq(const StepArgs& p, int n_tiles, int linear, char* lds, uint32_t* masks) {
    const Lane<DP> ln;
    const int n = ln.n, h = ln.h;
    int rank, bh, dev_rank;
    decode(linear, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int q0 = (n_tiles - 1 - rank) * OWN, dev_i = p.n_q - 1 - dev_rank, dev = p.q_dev + dev_i;
    const int b = bh / p.H, hd = bh - b * p.H, d = p.d;
    const int64_t base = b * p.stride_b + hd * p.stride_h + dev_i * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)dev_i * p.c;
    const int pitch = 2 * (int)p.kv_stride_s;

    const int a_own = q0 + n, a = min(a_own, p.c - 1);
    bf16x8 qf[8], gf[8];
    load_b_frags<8>(qf, (const __bf16*)p.q + base + (int64_t)a * p.stride_s, h, d);
    load_b_frags<8>(gf, (const __bf16*)p.dout + base + (int64_t)a * p.stride_s, h, d);
    const float delta = p.delta[sbase + a];
    const Scale2 kappa(p.scale);
    float lse2, lse2_lo;
    to_base2(p.lse[sbase + a], lse2, lse2_lo);
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    f32x16 acc[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acc[mb] = zero16();

    float z[2] = {0.f, 0.f};
    walk_keys<DP>(p, dev, q0, dt_make_rsrc((const __bf16*)p.k + kv_base, p.c, pitch, d),
              dt_make_rsrc((const __bf16*)p.v + kv_base, p.c, pitch, d), lds, ln,
              [&](const char* k, const char* v, int key0, const Block& blk) {
        const f32x16 s = scores<DP, PART>(k, qf, ln, part_ks), dp = scores<DP, PART>(v, gf, ln, part_ks);
        const int lane_last = (blk.full ? p.c - 1 : a_own - blk.off) - key0;
        f32x16 ds;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float pr = EXACT ? kappa.exp2(s[r], lse2, lse2_lo) : __builtin_amdgcn_exp2f(fmaf(s[r], kappa.hi, -lse2));
            if (reg_row(r, h) > lane_last) pr = 0.f;
            ds[r] = pr * (dp[r] - delta);
        }
        if (EXACT) look_at(z, s);
        accumulate<DP, EXACT>(acc, k, ds, ln);
    });

    float* const DQ = p.dq + base + (int64_t)a * p.stride_s;
    float4 old[blocks_of(DP)];
    load_old<DP>(old, DQ, d, !p.fresh && a_own < p.c, ln);
    __syncthreads();
    put_partial<DP>(lds, acc, ln);
    if (EXACT) put_odd(masks, a_own < p.c && odd_sum(z, acc), ln.wave, ln.lane);
    __syncthreads();
    const uint32_t odd_rows = EXACT ? take_odd(masks) : 0;
    if (a_own < p.c && !((odd_rows >> n) & 1))
        add_rows<DP>(DQ, old, lds, p.scale, d, ln);
    if (EXACT) each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { dq_row<__hip_bfloat16>(again, b, hd, dev_i, q0 + i, ln.lane); });
}

// -------------------------------------------------------------------- dK/dV
// Owned rows are keys, the streamed groups 128 queries with their LSE and delta beside them; the
// query heads that share the key/value head and the query shards that see it come one after the
// other.
template <int DP, bool PART, bool EXACT>
__device__ inline void bwd_dkdv(const StepArgs& p, int n_tiles, int linear, char* lds, float* stats, uint32_t* masks) {
    const Lane<DP> ln;
    const int n = ln.n, h = ln.h, tid = threadIdx.x;
    int tile, bh, dev_i;                                // low key tiles see most queries: first
    decode(linear, p.B * p.H_kv, tile, bh);
    decode_rank(tile, n_tiles, p.n_kv, p.layout, tile, dev_i);
    const int k0 = tile * OWN, dev = p.kv_dev + dev_i;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv, group = p.H / p.H_kv, d = p.d;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + dev_i * p.kv_shard;
    const int pitch = 2 * (int)p.stride_s;

    const int key_own = k0 + n, key = min(key_own, p.c - 1);
    const int64_t row = kv_base + (int64_t)key * p.kv_stride_s;
    bf16x8 kf[8], vf[8];
    load_b_frags<8>(kf, (const __bf16*)p.k + row, h, d);
    load_b_frags<8>(vf, (const __bf16*)p.v + row, h, d);
    const Scale2 kappa(p.scale);
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    f32x16 acck[4], accv[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) acck[mb] = accv[mb] = zero16();
    uint32_t gl[4];
    dt_load_offsets<DP>(gl, ln.lane, ln.wave, pitch, d);

    // the block being walked: query head and shard, its queries' first group, sub-tile and mask
    const int q_dev0 = p.layout == SA_STRIPED ? p.q_dev : max(p.q_dev, dev);
    int member = 0, q_dev = q_dev0, first, off;
    bool full;
    dt_rsrc Q, G;
    const float* stat_src;          // this thread's statistic: LSE (threads 0..127) or delta of a group's row
    auto enter_block = [&]() {
        const int hd = kvh * group + member;
        full = block_kind(q_dev, dev, p.layout) == MASK_FULL;
        off = block_off(q_dev, dev, p.layout);
        // first query a workgroup of these keys looks at (emulated coarse skipping: from the first
        // skip_bq-tall tile that shares an allowed pair with the keys' skip_bk-wide one)
        first = full ? 0 : k0;
        if (!full && p.skip_bq > 0) first = (k0 / p.skip_bk * p.skip_bk + off) / p.skip_bq * p.skip_bq;
        const int64_t base = b * p.stride_b + hd * p.stride_h + (q_dev - p.q_dev) * p.q_shard;
        Q = dt_make_rsrc((const __bf16*)p.q + base, p.c, pitch, d);
        G = dt_make_rsrc((const __bf16*)p.dout + base, p.c, pitch, d);
        stat_src = (tid < GROUP ? p.lse : p.delta) + b * p.stat_stride_b + hd * p.stat_stride_h +
                   (int64_t)(q_dev - p.q_dev) * p.c;
    };
    float stat;
    auto request = [&](int g0, char* to) {
        load_group<DP>(Q, g0, p.c, pitch, to, gl, ln.wave);
        load_group<DP>(G, g0, p.c, pitch, to + GROUP_BYTES<DP>, gl, ln.wave);
        // rows beyond the shard arrive as zeros; LSE = +inf makes their P and dS zero
        const int r = g0 + (tid & (GROUP - 1));
        stat = stat_src[min(r, p.c - 1)];
        if (tid < GROUP && r >= p.c) stat = INFINITY;
    };
    enter_block();
    float z[2] = {0.f, 0.f};
    int g0 = first / GROUP * GROUP, parity = 0;
    request(g0, lds);
    for (;;) {
        const int now_first = first, lane_first = full ? 0 : key_own + off;
        int next_g0 = g0 + GROUP;
        bool more = next_g0 < p.c;
        __builtin_amdgcn_s_waitcnt(0);
        float* const st_now = stats + parity * 3 * GROUP;       // LSE in base-2 units, its rest, delta
        if (tid < GROUP) to_base2(stat, st_now[tid], st_now[GROUP + tid]);
        else st_now[GROUP + tid] = stat;
        __syncthreads();
        if (!more) {
            if (++q_dev == p.q_dev + p.n_q) {
                q_dev = q_dev0;
                ++member;
            }
            more = member < group;
            if (more) {
                enter_block();
                next_g0 = first / GROUP * GROUP;
            }
        }
        if (more) request(next_g0, lds + (1 - parity) * 2 * GROUP_BYTES<DP>);
        const int a0 = g0 + OWN * ln.wave;
        if (a0 + 31 >= now_first && a0 < p.c) {
            const char* q = lds + parity * 2 * GROUP_BYTES<DP> + ln.wave * SUB_BYTES<DP>;
            const char* g = q + GROUP_BYTES<DP>;
            const float* st = st_now + OWN * ln.wave;
            const f32x16 s = scores<DP, PART>(q, kf, ln, part_ks), dp = scores<DP, PART>(g, vf, ln, part_ks);
            f32x16 pr, ds;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = reg_row(r, h);
                pr[r] = EXACT ? kappa.exp2(s[r], st[i], st[GROUP + i])
                              : __builtin_amdgcn_exp2f(fmaf(s[r], kappa.hi, -st[i]));
                if (a0 + i < lane_first) pr[r] = 0.f;
                ds[r] = pr[r] * (dp[r] - st[2 * GROUP + i]);
            }
            if (EXACT) look_at(z, s);
            accumulate<DP, EXACT>(accv, g, pr, ln);
            accumulate<DP, EXACT>(acck, q, ds, ln);
        }
        if (!more) break;
        g0 = next_g0;
        parity ^= 1;
    }

    constexpr int HALF = PARTIAL_BYTES<DP>;
    static_assert(2 * HALF <= 4 * GROUP_BYTES<DP>, "partial results");
    float4 old_v[blocks_of(DP)], old_k[blocks_of(DP)];
    load_old<DP>(old_v, p.dv + row, d, !p.fresh && key_own < p.c, ln);
    load_old<DP>(old_k, p.dk + row, d, !p.fresh && key_own < p.c, ln);
    __syncthreads();
    put_partial<DP>(lds, accv, ln);
    put_partial<DP>(lds + HALF, acck, ln);
    if (EXACT) put_odd(masks, key_own < p.c && odd_sum(z, acck), ln.wave, ln.lane);
    __syncthreads();
    const uint32_t odd_rows = EXACT ? take_odd(masks) : 0;
    if (key_own < p.c && !((odd_rows >> n) & 1)) {
        add_rows<DP>(p.dv + row, old_v, lds, 1.f, d, ln);
        add_rows<DP>(p.dk + row, old_k, lds + HALF, p.scale, d, ln);
    }
    if (EXACT)
        each_row<WAVES>(odd_rows, ln.wave, [&](const StepArgs& again, int i) { dkdv_row<__hip_bfloat16>(again, b, kvh, dev_i, k0 + i, 0, d, ln.lane); });
}

// Both in one launch, the two sequences of n_dkdv key-owning and n_dq query-owning workgroups
// evenly interleaved (each heaviest first): they share nothing but the inputs.
template <int DP, bool PART, bool EXACT>
__global__ void __launch_bounds__(64 * WAVES, DP <= 64 ? 2 : 1)
bwd_split_kernel(StepArgs p, int n_tiles, int n_dkdv, int n_dq) {
    __shared__ __attribute__((aligned(1024))) char lds[4 * GROUP_BYTES<DP>];
    __shared__ float stats[2 * 3 * GROUP];
    __shared__ uint32_t masks[WAVES];
    const int total = n_dkdv + n_dq, before = (int)((int64_t)blockIdx.x * n_dkdv / total);
    const bool keys = (int)(((int64_t)blockIdx.x + 1) * n_dkdv / total) > before;
    if (keys) bwd_dkdv<DP, PART, EXACT>(p, n_tiles, before, lds, stats, masks);
    else bwd_dq<DP, PART, EXACT>(p, n_tiles, (int)blockIdx.x - before, lds, masks);
}

enum Pass { FWD_EXACT, BWD_EXACT, BWD };
template <int DP, bool PART>
hipError_t run(const StepArgs& a, Pass pass, hipStream_t st) {
    const int n_tiles = (a.c + OWN - 1) / OWN;
    const int n_dkdv = n_tiles * a.n_kv * a.B * a.H_kv, n_dq = n_tiles * a.n_q * a.B * a.H;
    const dim3 grid((unsigned)(pass == FWD_EXACT ? n_dq : n_dkdv + n_dq)), block(64 * WAVES);
    if (pass == FWD_EXACT) hipLaunchKernelGGL((fwd_split_kernel<DP, PART>), grid, block, 0, st, a, n_tiles);
    else if (pass == BWD_EXACT) hipLaunchKernelGGL((bwd_split_kernel<DP, PART, true>), grid, block, 0, st, a, n_tiles, n_dkdv, n_dq);
    else hipLaunchKernelGGL((bwd_split_kernel<DP, PART, false>), grid, block, 0, st, a, n_tiles, n_dkdv, n_dq);
    return hipGetLastError();
}
template <int DP>
hipError_t run(const StepArgs& a, Pass pass, hipStream_t st) {
    return a.d % 8 ? run<DP, true>(a, pass, st) : run<DP, false>(a, pass, st);
}
hipError_t run(const StepArgs& a, Pass pass, hipStream_t st) {
    if (a.d <= 64) return run<64>(a, pass, st);
    if (a.d <= 112) return run<112>(a, pass, st);
    return run<128>(a, pass, st);
}

}  // namespace

// (of shapes that the 128-row matrix-core kernels take.)  Measured against those, us per backward step,
// here / there.  Triangular, d 128, 64 key tiles: 16 heads of 512 rows 25.5 / 27.7, 64 heads on 8 of 1024
// 188 / 212, 32 on 4 of 2048 308 / 396, on 2 of 4096 1138 / 1514, on one of 8192 4555 / 6093; 128 key tiles:
// 54.3 / 41.6, 32 on 8 of 2048 293 / 214, on 4 of 4096 1048 / 796, on 2 of 8192 4065 / 3174.  Full blocks have
// twice the work, 32 key tiles: 2 heads of 2048 rows 40 / 61, 32 on 8 of 512 66.0 / 64.7, on 4 of 1024 210 /
// 238, on 2 of 2048 823 / 865, on one of 4096 3292 / 3376; 64: 16 heads of 512 30.3 / 27.5, 32 on 8 of 1024
// 178 / 142, on one of 8192 10543 / 7427.  d 64 alike (32 on 4, full, 32 key tiles 129 / 216, 64 335 / 378).
bool bwd_split_wanted(const StepArgs& a) {
    return a.d <= TD && (int64_t)((a.c + 127) / 128) * a.B * a.n_kv * a.H_kv <= (uneven(a) ? 64 : 32);
}
hipError_t launch_bwd_split(const StepArgs& a, hipStream_t st) { return run(a, BWD, st); }

// bf16 blocks shorter than a 128-row tile, probabilities and dS in fp32 precision.  (Tile loads
// address a group of 128 rows with 32-bit byte offsets.)  Against the fp32 instruction on widened
// operands (f32_step.hip), us: whole ring, 8 x 96 tokens, 32 heads, d 64, forward 51 / 99, backward
// 78 / 215; 4 x 120 tokens, 64 heads, d 128: 69 / 112 and 141 / 342; one backward step 12 / 15 and
// 22 / 46.  A single forward block gains while few workgroups share the memory system: 2 heads of
// 64 tokens, d 128, 8.4 / 15.4, 16 heads of 120 tokens (64 workgroups) 12.6 / 17.3, but 96
// workgroups at d 64 12.6 / 10.9, 256 at d 128 21 / 18.  Error against 64 bits (2-norm, 16 x 127
// tokens, d 128): O 2.2e-7 -> 1.6e-7, dQ 3.7e-7 -> 3.2e-7, dK 6.1e-7 -> 4.3e-7, dV 6.0e-7 -> 4.1e-7.
bool short_exact_wanted(const StepArgs& a, int dtype, bool backward) {
    const int64_t widest = a.stride_s > a.kv_stride_s ? a.stride_s : a.kv_stride_s;
    if (dtype != SA_BF16 || a.d % 4 || a.d > TD || a.c >= GROUP || GROUP * 2 * widest + 2 * a.d >= (int64_t(1) << 31)) return false;
    return backward || a.n_kv > 1 || (int64_t)((a.c + OWN - 1) / OWN) * a.n_q * a.B * a.H <= 64;
}
hipError_t launch_short_exact(const StepArgs& a, bool backward, hipStream_t st) {
    return run(a, backward ? BWD_EXACT : FWD_EXACT, st);
}

}  // namespace sa
