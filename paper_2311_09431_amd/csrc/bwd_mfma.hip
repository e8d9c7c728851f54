// Backward ring step on the CDNA4 matrix cores (bf16 operands, fp32 accumulate),
// head dimension up to 256 (32, 64, 112, 128 or 256 columns computed).  The paper describes no
// backward pass; this is the analytic gradient of causal attention (Sec. 2.1) restricted to the pairs that
// GetMask(j, k) allows, with P recomputed from the saved log-sum-exp:
//   P = exp(scale q.k - LSE),  dV += P^T dO,  dP = dO V^T,
//   dS = P * (dP - delta),     dQ += scale dS K,  dK += scale dS^T Q.
// Two deterministic kernels, no atomics: every output row is read-modify-written
// by exactly one wavefront.  (dK and dV at 65 to 128 columns, and dQ there where it shares their launch: bwd_ring.hip.)
//
//  * dq kernel: a workgroup owns 128 query rows (Q and dO stay in registers as
//    B operands), key tiles stream through LDS.  S^T = K Q^T and dP^T = V dO^T
//    put 16 + 16 keys of ONE query in a lane, so LSE and delta are per-lane
//    scalars and dS^T is already the B operand of dQ^T += K^T dS^T.
//  * dkdv kernel: a workgroup owns 128 key rows (K and V in registers), query
//    tiles stream through LDS.  S = Q K^T and dP = dO V^T put 16 + 16 queries of
//    ONE key in a lane; P and dS are the B operands of dV^T += dO^T P and
//    dK^T += Q^T dS.
// Both skip every tile the mask empties (Sec. 2.2.1) per 32-row wavefront and
// apply the element mask only on the tiles that can cross the diagonal (the dq
// kernel also on the last tile pair of a full block, where it removes nothing
// unless the block size is not a multiple of 128).
#include <hip/hip_bf16.h>

#include <type_traits>

#include "acc_file.h"
#include "mfma_tiles.h"
#include "sa_internal.h"

namespace sa {

namespace {

constexpr int BM = 128;   // rows owned by a workgroup (queries in dq, keys in dkdv)
constexpr int BN = TR;    // rows streamed per tile
constexpr int D = TD;

__device__ inline bf16x8 pack8(const f32x16& x, int first) {
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (__bf16)x[first + e];
    return r;
}

// ---------------------------------------------------------------- dQ kernel
// K and V tiles (64 key rows) stream global -> LDS directly into swizzled tiles, two
// buffers each.  The loop runs over 32-key sub-tiles u; iteration u issues, interleaved
// slice by slice,
//     S^T(u+1) = K(u+1) Q^T, dP^T(u+1) = V(u+1) dO^T   (16 MFMA)
//     P(u) = exp2(S(u) kappa - LSE), dS(u) = P (dP(u) - delta)   (VALU)
// and then dQ^T += K(u)^T dS(u)^T (8 MFMA, K^T through the transposing LDS read).
// Two barriers per 64-key tile: one makes the tile requested one iteration earlier
// visible, one releases the tile just finished for the next request.

// DP: columns computed.  64 for head dimensions up to 64 (k-steps 4..7 of the S and dP
// products and column blocks 2, 3 of the dQ product do not exist then), half of that up to 32 that are a multiple of 8, 112 for those up to 112
// (no k-step 7), 128, or 256 for head dimensions above 128: the K and V tiles then come as two 128-column halves, tile_bytes(DP) apart in
// LDS, and every slice holds one MFMA of each product per half.  PART: d % 8 == 4, the K and V
// fragments that hold column d are cleared beyond it (part_ks = the k-step, or -1 for the lanes
// of the other half-wave).
template <bool NEXT, bool MASK, int DP, bool PART>
__device__ __forceinline__ void dq_step(f32x16& s_cur, f32x16& dp_cur, f32x16& s_next, f32x16& dp_next,
                               f32x16 (&acc)[4 * halves_of(DP)], const bf16x8 (&qf)[8 * halves_of(DP)],
                               const bf16x8 (&gf)[8 * halves_of(DP)], float kappa, float lse2, float delta,
                               const uint32_t (&arow)[8], const uint32_t (&tr0)[4], const uint32_t (&tr1)[4],
                               const char* k_next, const char* v_next, const char* k_cur, int mask_lim,
                               int part_ks) {
    constexpr int NH = halves_of(DP), KS = ksteps_of(DP), MB = blocks_of(DP);      // per half
    bf16x8 ka[NH][8], va[NH][8], kt[NH][8], dsb[2];
    auto fetch = [&](int i) {
        if (NEXT && i < KS) {
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) {
                ka[hh][i] = dt_read_row(k_next + hh * tile_bytes(DP), arow[i]);
                va[hh][i] = dt_read_row(v_next + hh * tile_bytes(DP), arow[i]);
            }
        }
    };
    auto fetch_t = [&](int i) {
        if (i % 4 < MB) {
#pragma unroll
            for (int hh = 0; hh < NH; ++hh)
                kt[hh][i] = dt_read_tr(k_cur + hh * tile_bytes(DP) + (i / 4) * 16 * row_bytes(DP), tr0[i % 4], tr1[i % 4]);
        }
    };
    fetch(0);
    fetch(1);
    if (NEXT) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s_next[r] = dp_next[r] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        __builtin_amdgcn_sched_barrier(0);          // slices stay in program order
        if (i + 2 < 8) fetch(i + 2);
        if (i >= 4) fetch_t(i - 4);                 // first half of the K^T operands
        if (NEXT && i < KS) {
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) {
                const bool last_chunk = 8 * hh + i == part_ks;
                const bool select = PART && i >= part_from(DP);
                s_next = mfma(select ? zero_beyond_d(ka[hh][i], last_chunk) : ka[hh][i], qf[8 * hh + i], s_next);
                dp_next = mfma(select ? zero_beyond_d(va[hh][i], last_chunk) : va[hh][i], gf[8 * hh + i], dp_next);
            }
        }
#pragma unroll
        for (int r = 2 * i; r < 2 * i + 2; ++r) {
            float pr = __builtin_amdgcn_exp2f(fmaf(s_cur[r], kappa, -lse2));
            if (MASK && 8 * (r / 4) + (r % 4) > mask_lim) pr = 0.f;
            dsb[r / 8][r % 8] = (__bf16)(pr * (dp_cur[r] - delta));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i + 4 < 8) fetch_t(i + 4);
        if (i % 4 < MB) {
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) acc[4 * hh + i % 4] = mfma(kt[hh][i], dsb[i / 4], acc[4 * hh + i % 4]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// One code path serves triangular and full blocks, as in the forward kernel: the last two
// tiles of the walk carry the element mask, whose limit is the query's own position, or the
// last key (c - 1) for a full block.  RAGGED (c not a multiple of 128): loads of rows beyond
// the shard are clamped, their results are not stored, keys beyond it come in as zero rows
// and are removed by the mask.
// WALK: one block, or (WALK_RING) the blocks of several key shards one after the other, as in
// the forward kernel: dQ stays in registers over all of them.
// k_lds0 .. v_lds1: the tile buffers (two 128-column halves each when DP = 256), LDS objects of their
// own: as parts of one array the compiler arranges the d = 256 kernels otherwise and a full step of
// 8 heads, 8192 rows, takes 2.197 instead of 2.177 ms
template <bool RAGGED, int WALK, int DP, bool PART, bool BY_RANK>
__device__ __forceinline__ void bwd_dq(const StepArgs& p, int n_tiles, int linear, char* k_lds0, char* k_lds1,
                                       char* v_lds0, char* v_lds1) {
    constexpr int NH = halves_of(DP), KS = ksteps_of(DP), MB = halves_of(DP) * blocks_of(DP);      // k-steps per half, column blocks

    const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform, kept scalar
    constexpr bool RING = WALK == WALK_RING;
    int rank, bh, dev = p.q_dev;
    decode_block<true, BY_RANK>(linear, RING ? n_tiles * p.n_q : n_tiles, p.B * p.H, rank, bh);
    if (RING) {
        int dev_rank;
        decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
        dev += p.n_q - 1 - dev_rank;
    }
    const int qt = n_tiles - 1 - rank;      // heaviest query tiles first
    const int b = bh / p.H, hd = bh - b * p.H;
    const int64_t base = b * p.stride_b + hd * p.stride_h + (RING ? (dev - p.q_dev) * p.q_shard : 0);
    // key/value head of this query head's group (the same head when H_kv == H)
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (RING ? (int64_t)(dev - p.q_dev) * p.c : 0);
    const __bf16* Q = (const __bf16*)p.q + base;
    const int d = p.d;                                 // d <= DP, zero-padded to DP columns
    const int64_t ss = p.stride_s;                     // elements between consecutive rows of Q, dO, dQ
    const int pitch = 2 * (int)p.kv_stride_s;          // bytes between consecutive rows of K and V
    const int tile_pitch = DT_ROWS * pitch;            // bytes between 64-row tiles in global memory
    dt_rsrc Kr = dt_make_rsrc((const __bf16*)p.k + kv_base, p.c, pitch, d);
    dt_rsrc Vr = dt_make_rsrc((const __bf16*)p.v + kv_base, p.c, pitch, d);
    const __bf16* G = (const __bf16*)p.dout + base;
    float* DQ = p.dq + base;

    const int q0 = qt * BM, a_own = q0 + 32 * wave + n;
    const bool row_ok = !RAGGED || a_own < p.c;
    const int a = RAGGED ? min(a_own, p.c - 1) : a_own;      // the row this lane loads
    // The block being walked, as in the forward kernel: key shard kv, its 64-key tiles, those of
    // the walk without emulated coarse skipping (the last two carry the element mask) and the
    // mask: sub-tile v is allowed iff 8 (r/4) + r%4 <= mask_base - 32 v.  All four wavefronts
    // walk the 2 n_kt sub-tiles (at most three are entirely masked for a wavefront).
    int kv = p.kv_dev, n_kt, n_kt_fine, mask_base;
    auto enter_block = [&]() {
        const bool full = RING ? block_kind(dev, kv, p.layout) == MASK_FULL : WALK == WALK_FULL;
        const int off = block_off(dev, kv, p.layout);
        n_kt = n_kt_fine = full ? 2 * n_tiles : (q0 + BM) / DT_ROWS;
        if (!full && p.skip_bq > 0) {       // emulated coarse skipping, as in the forward kernel
            const int q_hi = (q0 / p.skip_bq + 1) * p.skip_bq - 1;
            n_kt = min(p.c, ((q_hi - off) / p.skip_bk + 1) * p.skip_bk) / DT_ROWS;
        }
        mask_base = (full ? p.c - 1 : a_own - off) - 4 * h;
    };
    enter_block();
    // contiguous layout: the blocks of devices further on are entirely masked
    const int kv_end = !RING ? kv + 1
                             : (p.layout == SA_STRIPED ? p.kv_dev + p.n_kv : min(p.kv_dev + p.n_kv, dev + 1));

    uint32_t arow[8], tr0[4], tr1[4], gl[NH][4];
    dt_row_addrs<DP>(arow, n, h);
    dt_tr_addrs<DP>(tr0, tr1, lane);
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) dt_load_offsets<DP>(gl[hh], lane, wave, pitch, d, hh);
    auto load_tile = [&](dt_rsrc m, int tile_byte_offset, char* buf) {
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) dt_load<DP>(m, tile_byte_offset, buf + hh * tile_bytes(DP), gl[hh], wave);
    };
    load_tile(Kr, 0, k_lds0);
    load_tile(Vr, 0, v_lds0);
    load_tile(Kr, tile_pitch, k_lds1);       // n_kt >= 2 always
    load_tile(Vr, tile_pitch, v_lds1);

    bf16x8 qf[8 * NH], gf[8 * NH];
    load_b_frags<8 * NH>(qf, Q + (int64_t)a * ss, h, d);
    load_b_frags<8 * NH>(gf, G + (int64_t)a * ss, h, d);
    const float kappa = p.scale * LOG2E;
    float lse2 = p.lse[sbase + a] * LOG2E;
    float delta = p.delta[sbase + a];
    f32x16 acc[4 * NH];
#pragma unroll
    for (int mb = 0; mb < 4 * NH; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mb][r] = 0.f;

    // the statistics are complete here: a load left pending into the loop would be waited
    // for there, together with the tile loads just issued
    asm volatile("" : "+v"(lse2), "+v"(delta));
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // PART: k-step whose fragment, in this half-wave, is the chunk holding column d
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    f32x16 s_a, s_b, dp_a, dp_b;
    {   // prologue: S(0), dP(0)
#pragma unroll
        for (int r = 0; r < 16; ++r) s_a[r] = dp_a[r] = 0.f;
#pragma unroll
        for (int hh = 0; hh < NH; ++hh)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 ka = dt_read_row(k_lds0 + hh * tile_bytes(DP), arow[ks]);
                const bf16x8 va = dt_read_row(v_lds0 + hh * tile_bytes(DP), arow[ks]);
                s_a = mfma(PART ? zero_beyond_d(ka, 8 * hh + ks == part_ks) : ka, qf[8 * hh + ks], s_a);
                dp_a = mfma(PART ? zero_beyond_d(va, 8 * hh + ks == part_ks) : va, gf[8 * hh + ks], dp_a);
            }
    }

    // Trip t = iterations 2t (scores in *_a) and 2t+1 (scores in *_b); PAR = t & 1 selects
    // the buffers of tile t at compile time.  REQ: the tiles of kr, vr at `at` are requested into
    // the buffers this trip frees.
    auto trip = [&](auto last_c, auto mask_c, auto par_c, auto req_c, int t, dt_rsrc kr, dt_rsrc vr, int at) {
        constexpr bool LAST = decltype(last_c)::value, MASK = decltype(mask_c)::value;
        constexpr bool REQ = decltype(req_c)::value;
        constexpr int PAR = decltype(par_c)::value;
        char* const k_cur = PAR ? k_lds1 : k_lds0;
        char* const v_cur = PAR ? v_lds1 : v_lds0;
        char* const k_nxt = PAR ? k_lds0 : k_lds1;
        char* const v_nxt = PAR ? v_lds0 : v_lds1;
        dq_step<true, MASK, DP, PART>(s_a, dp_a, s_b, dp_b, acc, qf, gf, kappa, lse2, delta, arow, tr0, tr1,
                                      k_cur + tile_bytes(DP) / 2, v_cur + tile_bytes(DP) / 2, k_cur, mask_base - 64 * t,
                                      part_ks);
        if (!LAST) {
            __builtin_amdgcn_s_waitcnt(0);      // tile t+1, requested one iteration ago, has landed
            __syncthreads();
        }
        dq_step<!LAST, MASK, DP, PART>(s_b, dp_b, s_a, dp_a, acc, qf, gf, kappa, lse2, delta, arow, tr0, tr1,
                                       k_nxt, v_nxt, k_cur + tile_bytes(DP) / 2, mask_base - 64 * t - 32, part_ks);
        if (REQ) {
            __syncthreads();                    // every wavefront is done with tile t
            load_tile(kr, at, k_cur);
            load_tile(vr, at, v_cur);
        }
    };
    using T = std::true_type;
    using F = std::false_type;
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    // per block: trips before the last tile pair of the fine walk without the element mask, then
    // masked trips: two, more under emulated coarse skipping (n_kt_fine and n_kt are even)
    int t = 0;
    for (;;) {
        for (; t + 2 < n_kt_fine; t += 2) {
            trip(F{}, F{}, P0{}, T{}, t, Kr, Vr, (t + 2) * tile_pitch);
            trip(F{}, F{}, P1{}, T{}, t + 1, Kr, Vr, (t + 3) * tile_pitch);
        }
        if (!RING) {
            for (; t + 2 < n_kt; t += 2) {
                trip(F{}, T{}, P0{}, T{}, t, Kr, Vr, (t + 2) * tile_pitch);
                trip(F{}, T{}, P1{}, T{}, t + 1, Kr, Vr, (t + 3) * tile_pitch);
            }
            break;
        }
        // a masked pair and what follows it: the next pair of the block, the next block, or the
        // last pair of the walk
        const bool leave = t + 2 >= n_kt;
        if (leave && kv + 1 == kv_end) break;
        const int64_t move = leave ? 2 * p.kv_shard : 0;
        const dt_rsrc kr = dt_advance(Kr, move), vr = dt_advance(Vr, move);
        const int at = leave ? 0 : (t + 2) * tile_pitch;
        trip(F{}, T{}, P0{}, T{}, t, kr, vr, at);
        trip(F{}, T{}, P1{}, T{}, t + 1, kr, vr, at + tile_pitch);
        t += 2;
        if (leave) {
            Kr = kr;
            Vr = vr;
            t = 0;
            ++kv;
            enter_block();
        }
    }
    trip(F{}, T{}, P0{}, F{}, t, Kr, Vr, 0);
    trip(T{}, T{}, P1{}, F{}, t + 1, Kr, Vr, 0);

#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = 32 * mb + 8 * g + 4 * h;
            if (col >= d || !row_ok) continue;            // padding columns, rows beyond the shard
            float4* dst = reinterpret_cast<float4*>(DQ + (int64_t)a * ss + col);
            float4 x = RING && p.fresh ? make_float4(0.f, 0.f, 0.f, 0.f) : *dst;
            x.x = fmaf(p.scale, acc[mb][4 * g + 0], x.x); x.y = fmaf(p.scale, acc[mb][4 * g + 1], x.y);
            x.z = fmaf(p.scale, acc[mb][4 * g + 2], x.z); x.w = fmaf(p.scale, acc[mb][4 * g + 3], x.w);
            *dst = x;
        }
}

// ------------------------------------------------------------- dK/dV kernel
// S / dP product of the dK/dV kernel.  DP <= 128: the asm forms above (results stay in VGPRs).
// DP = 256: the compiler's own MFMA; K and V alone are 128 registers there, the asm forms would
// pin them and the score tiles to VGPRs and spill a hundred registers, while the compiler keeps
// part of them in AGPRs and copies a score tile back when the VALU code wants it (32 copies
// against 48 MFMAs per step, affordable at this head dimension).
template <int DP>
__device__ __forceinline__ void score_mfma(f32x16& acc, bf16x8 a, bf16x8 b, bool first, bool after_valu) {
    if (DP > 128) {
        if (first) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        }
        acc = mfma(a, b, acc);
    } else if (first) {
        mfma_vgpr_first(acc, a, b, after_valu);
    } else {
        mfma_vgpr_acc(acc, a, b, after_valu);
    }
}

// A workgroup owns 128 key rows (K and V rows in registers as B operands, dK^T and
// dV^T accumulators in registers: one wavefront per SIMD with the large register
// budget).  Q and dO tiles (64 query rows) stream global -> LDS directly into swizzled
// tiles, two buffers each; LSE * log2(e) and delta of the tile's rows are staged
// beside them.  Iteration u over 32-query sub-tiles issues, interleaved slice by slice,
//     S(u+1) = Q(u+1) K^T, dP(u+1) = dO(u+1) V^T - delta   (16 MFMA; the dP accumulators
//                              start from -delta, read from LDS, instead of from zero)
//     P(u) = exp2(S(u) kappa - LSE), dS(u) = P dP(u)   (VALU)
// and then dV^T += dO(u)^T P(u), dK^T += Q(u)^T dS(u) (16 MFMA, the transposed
// operands through the transposing LDS read).
constexpr int KV_STAT_FLOATS = 2 * 2 * DT_ROWS;              // [buffer][lse2 | -delta][64]

// -delta of the 32 query rows of a sub-tile as the initial dP^T accumulator: register r holds
// query row 8 (r/4) + 4h + r%4
__device__ inline void load_neg_delta(f32x16& dp, const float* neg_delta, int h) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 x = *reinterpret_cast<const float4*>(neg_delta + 8 * g + 4 * h);
        dp[4 * g + 0] = x.x; dp[4 * g + 1] = x.y; dp[4 * g + 2] = x.z; dp[4 * g + 3] = x.w;
    }
}

// DP = 256 (head dimensions above 128): the Q and dO tiles come as two 128-column halves,
// tile_bytes(DP) apart in LDS.  S and dP contract over both; a workgroup accumulates only ONE half of
// the columns of dK^T and dV^T (256 columns of both do not fit the register file beside K, V and
// the score tiles), so tr0 / tr1 arrive with that half's LDS offset added and the other half is
// another workgroup's, which computes S and dP again.
template <bool NEXT, bool MASK, int DP, bool PART>
__device__ __forceinline__ void dkdv_step(f32x16& s_cur, f32x16& dp_cur, f32x16& s_next, f32x16& dp_next,
                                 f32x16 (&acck)[4], f32x16 (&accv)[4], const bf16x8 (&kf)[8 * halves_of(DP)],
                                 const bf16x8 (&vf)[8 * halves_of(DP)], float kappa, const uint32_t (&arow)[8],
                                 const uint32_t (&tr0)[4], const uint32_t (&tr1)[4], const char* q_next,
                                 const char* g_next, const char* q_cur, const char* g_cur,
                                 const float* stat_cur, const float* stat_next, int h, int mask_lim,
                                 int part_ks) {
    constexpr int NH = halves_of(DP), KS = ksteps_of(DP), MB = blocks_of(DP);      // per half
    bf16x8 qa[NH][8], ga[NH][8], qt[8], gt[8], pb[2], dsb[2];
    if (NEXT) load_neg_delta(dp_next, stat_next + DT_ROWS, h);
    auto fetch = [&](int i) {
        if (NEXT && i < KS) {
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) {
                qa[hh][i] = dt_read_row(q_next + hh * tile_bytes(DP), arow[i]);
                ga[hh][i] = dt_read_row(g_next + hh * tile_bytes(DP), arow[i]);
            }
        }
    };
    auto fetch_t = [&](int i) {
        if (i % 4 < MB) {
            gt[i] = dt_read_tr(g_cur + (i / 4) * 16 * row_bytes(DP), tr0[i % 4], tr1[i % 4]);
            qt[i] = dt_read_tr(q_cur + (i / 4) * 16 * row_bytes(DP), tr0[i % 4], tr1[i % 4]);
        }
    };
    // LSE * log2(e) of this lane's query rows 8 (r/4) + 4h + r%4, two per slice
    float2 lv[8];
    auto fetch_stat = [&](int i) {
        lv[i] = *reinterpret_cast<const float2*>(stat_cur + 8 * (i / 2) + 4 * h + 2 * (i % 2));
    };
    // operands requested this many slices ahead of their use: row reads 2, transposed reads 3
    // (3 / 4 and 4 / 5 measured the same to 1 % at d 128, when that ran here: LDS latency is covered)
    constexpr int AHEAD = 2, TAHEAD = 3;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
        fetch(i);
        fetch_stat(i);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        __builtin_amdgcn_sched_barrier(0);          // slices stay in program order
        if (i + AHEAD < 8) {
            fetch(i + AHEAD);
            fetch_stat(i + AHEAD);
        }
        if (i >= 8 - TAHEAD) fetch_t(i - (8 - TAHEAD));     // the first transposed operands ahead of their use
        // One wavefront per SIMD: a second MFMA issued right behind the first stalls the
        // wavefront until the matrix pipeline is free again, and nothing else is issued
        // meanwhile.  So each MFMA is followed by one score's worth of VALU work, which runs
        // while it executes.
        auto score = [&](int r) {
            const float lr = (r & 1) ? lv[i].y : lv[i].x;
            float pr = __builtin_amdgcn_exp2f(fmaf(s_cur[r], kappa, -lr));
            if (MASK && 8 * (r / 4) + (r % 4) < mask_lim) pr = 0.f;
            pb[r / 8][r % 8] = (__bf16)pr;
            dsb[r / 8][r % 8] = (__bf16)(pr * dp_cur[r]);
        };
        if (NEXT && i < KS) {
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) {
                const bool select = PART && i >= part_from(DP);
                const bf16x8 qx = select ? zero_beyond_d(qa[hh][i], 8 * hh + i == part_ks) : qa[hh][i];
                const bf16x8 gx = select ? zero_beyond_d(ga[hh][i], 8 * hh + i == part_ks) : ga[hh][i];
                score_mfma<DP>(s_next, qx, kf[8 * hh + i], i == 0 && hh == 0, select);
                if (hh == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    score(2 * i);
                    __builtin_amdgcn_sched_barrier(0);
                }
                score_mfma<DP>(dp_next, gx, vf[8 * hh + i], false, select);
            }
            score(2 * i + 1);
        } else {
            score(2 * i);
            score(2 * i + 1);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i + TAHEAD < 8) fetch_t(i + TAHEAD);
        if (i % 4 < MB) {
            accv[i % 4] = mfma(gt[i], pb[i / 4], accv[i % 4]);
            acck[i % 4] = mfma(qt[i], dsb[i / 4], acck[i % 4]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// RAGGED (c not a multiple of 128): key rows beyond the shard are loaded from its last row and
// not stored; query rows beyond it come in as zero rows of Q and dO with LSE = +inf, so their
// P and dS are exactly zero.
// WALK: one block, or (WALK_RING) several one after the other with dK and dV in registers from the
// first to the last: the query heads that share this key/value head, each with the query shards of
// the devices that see these keys.
// q_lds0 .. g_lds1: the tile buffers, as in the dQ kernel; stat: KV_STAT_FLOATS floats
template <int WALK, bool RAGGED, int DP, bool PART, bool BY_RANK>
__device__ __forceinline__ void bwd_dkdv(const StepArgs& p, int n_tiles, int linear, char* q_lds0, char* q_lds1,
                                         char* g_lds0, char* g_lds1, float* stat) {
    constexpr int NH = halves_of(DP), KS = ksteps_of(DP), MB = blocks_of(DP);      // per half

    const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform, kept scalar
    constexpr bool RING = WALK == WALK_RING;
    int ktile, bhh, dev = p.kv_dev;               // triangular blocks: low key tiles see most queries: first
    // one workgroup per (key tile, device, batch, key/value head, 128-column half of dK / dV)
    decode_block<false, BY_RANK>(linear, RING ? n_tiles * p.n_kv : n_tiles, p.B * p.H_kv * NH, ktile, bhh);
    if (RING) {
        int dev_rank;
        decode_rank(ktile, n_tiles, p.n_kv, p.layout, ktile, dev_rank);
        dev += dev_rank;
    }
    const int bh = bhh / NH, ohalf = bhh - bh * NH;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + (RING ? (dev - p.kv_dev) * p.kv_shard : 0);
    const int d = p.d;                                 // d <= DP, zero-padded to DP columns
    const int64_t ss = p.kv_stride_s;                  // elements between consecutive rows of K, V, dK, dV
    const int pitch = 2 * (int)p.stride_s;             // bytes between consecutive rows of Q and dO
    const int tile_pitch = DT_ROWS * pitch;            // bytes between 64-row tiles in global memory
    const __bf16* K = (const __bf16*)p.k + kv_base;
    const __bf16* V = (const __bf16*)p.v + kv_base;
    float* DK = p.dk + kv_base;
    float* DV = p.dv + kv_base;

    const int k0 = ktile * BM, key_own = k0 + 32 * wave + n;
    const bool key_ok = !RAGGED || key_own < p.c;
    const int key = RAGGED ? min(key_own, p.c - 1) : key_own;     // the row this lane loads
    const int n_qt = RAGGED ? 2 * n_tiles : p.c / DT_ROWS;
    // The block being walked: query head q_head of the group and query shard q_dev.  Query tiles
    // holding at least one allowed pair (query a >= key + off) are those from k0 / 64 on; only the
    // first four 32-query sub-tiles of these can cross the diagonal for some wavefront, the trips
    // before t_plain carry the mask.  Sub-tile u: register r (query 32 u + 8 (r/4) + 4h + r%4) is
    // allowed iff 8 (r/4) + r%4 >= mask_base - 32 u.
    const int group = RING ? p.H / p.H_kv : 1;
    // contiguous layout: earlier devices' queries see nothing of these keys
    const int dev0 = RING && p.layout != SA_STRIPED ? max(p.q_dev, dev) : p.q_dev;
    int q_head = 0, q_dev = dev0, t_first, t_plain, mask_base;
    dt_rsrc Qr, Gr;
    const float* stat_src;      // this thread's next statistics row
    int stat_row;               // its number (RAGGED only)
    auto enter_block = [&]() {
        const int hd = kvh * group + q_head;
        const bool tri = RING ? block_kind(q_dev, dev, p.layout) == MASK_TRI : WALK == WALK_TRI;
        const int off = block_off(q_dev, dev, p.layout);
        t_first = tri ? k0 / DT_ROWS : 0;
        t_plain = tri ? t_first + 2 : 0;
        if (tri && p.skip_bq > 0)   // emulated coarse skipping: from the first skip_bq-tall query tile
                                    // that shares an allowed pair with these keys' skip_bk-wide tile
            t_first = ((k0 / p.skip_bk * p.skip_bk + off) / p.skip_bq) * p.skip_bq / DT_ROWS;
        mask_base = tri ? key_own + off - 4 * h : 0;
        const int64_t base = b * p.stride_b + hd * p.stride_h + (RING ? (q_dev - p.q_dev) * p.q_shard : 0);
        const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h +
                              (RING ? (int64_t)(q_dev - p.q_dev) * p.c : 0);
        Qr = dt_make_rsrc((const __bf16*)p.q + base, p.c, pitch, d);
        Gr = dt_make_rsrc((const __bf16*)p.dout + base, p.c, pitch, d);
        stat_row = (tid & (DT_ROWS - 1)) + t_first * DT_ROWS;
        stat_src = ((tid & DT_ROWS) ? p.delta : p.lse) + sbase + stat_row;
    };
    enter_block();

    uint32_t arow[8], tr0[4], tr1[4], gl[NH][4];
    dt_row_addrs<DP>(arow, n, h);
    dt_tr_addrs<DP>(tr0, tr1, lane);
    if (NH > 1) {       // the transposed operands come from this workgroup's half of the columns
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
            tr0[mb] += ohalf * tile_bytes(DP);
            tr1[mb] += ohalf * tile_bytes(DP);
        }
    }
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) dt_load_offsets<DP>(gl[hh], lane, wave, pitch, d, hh);
    auto load_tile = [&](dt_rsrc m, int tile_byte_offset, char* buf) {
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) dt_load<DP>(m, tile_byte_offset, buf + hh * tile_bytes(DP), gl[hh], wave);
    };
    // t_first and n_qt are even (k0 and c are multiples of 128): tile t_first goes to buffer 0
    // and there are always at least two tiles
    load_tile(Qr, t_first * tile_pitch, q_lds0);
    load_tile(Gr, t_first * tile_pitch, g_lds0);
    load_tile(Qr, (t_first + 1) * tile_pitch, q_lds1);
    load_tile(Gr, (t_first + 1) * tile_pitch, g_lds1);
    // statistics of query tile t -> stat[(t & 1)][0 | 1][64]: threads 0..63 LSE * log2(e), 64..127
    // -delta.  The fetch is branch-free (wavefronts 2 and 3 re-read what 0 and 1 read and drop
    // it), so nothing waits for it before the store one trip later.
    const float stat_mul = (tid & DT_ROWS) ? -1.f : LOG2E;
    auto stat_fetch = [&]() -> float {          // tiles in order: the pointer walks with them
        float x;
        if (RAGGED) {       // rows beyond the shard: LSE = +inf, delta = 0 (still branch-free)
            x = stat_src[min(stat_row, p.c - 1) - stat_row];
            if (stat_row >= p.c) x = (tid & DT_ROWS) ? 0.f : INFINITY;
            stat_row += DT_ROWS;
        } else {
            x = *stat_src;
        }
        stat_src += DT_ROWS;
        return x;
    };
    auto stat_store = [&](int t, float x) {
        if (tid < 2 * DT_ROWS) stat[(t & 1) * 2 * DT_ROWS + tid] = x * stat_mul;
    };
    stat_store(t_first, stat_fetch());
    float rstat = stat_fetch();         // statistics of the tile after the present one

    bf16x8 kf[8 * NH], vf[8 * NH];
    load_b_frags<8 * NH>(kf, K + (int64_t)key * ss, h, d);
    load_b_frags<8 * NH>(vf, V + (int64_t)key * ss, h, d);
    const float kappa = p.scale * LOG2E;
    f32x16 acck[4], accv[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acck[mb][r] = accv[mb][r] = 0.f;

    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // PART: k-step whose fragment, in this half-wave, is the chunk holding column d
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    f32x16 s_a, s_b, dp_a, dp_b;
    {   // prologue: S, dP of the first sub-tile
        const char* q0p = q_lds0;
        const char* g0p = g_lds0;
        load_neg_delta(dp_a, stat + DT_ROWS, h);          // tile t_first is in buffer 0
        // same order of the partial products as in dkdv_step (k-step outside, half inside): a
        // sub-tile's scores have the same bits whether this prologue or a step computes them
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) {
                bf16x8 qx = dt_read_row(q0p + hh * tile_bytes(DP), arow[ks]), gx = dt_read_row(g0p + hh * tile_bytes(DP), arow[ks]);
                if (PART) {
                    qx = zero_beyond_d(qx, 8 * hh + ks == part_ks);
                    gx = zero_beyond_d(gx, 8 * hh + ks == part_ks);
                }
                score_mfma<DP>(s_a, qx, kf[8 * hh + ks], ks == 0 && hh == 0, PART);
                score_mfma<DP>(dp_a, gx, vf[8 * hh + ks], false, PART);
            }
        if (DP <= 128) mfma_results_to_valu(s_a, dp_a);
    }

    // Trip t = iterations 2t (scores in *_a) and 2t+1 (scores in *_b) on query tile t.  REQ: the
    // tile at `at` of the present Qr, Gr (which the caller may have moved on to the next block's)
    // is requested into the buffers this trip frees.  mask_at = mask_base - 64 t.
    auto trip = [&](auto mask_c, auto par_c, auto last_c, auto req_c, int mask_at, int at) {
        constexpr bool MASK = decltype(mask_c)::value, last = decltype(last_c)::value;
        constexpr bool REQ = decltype(req_c)::value;
        constexpr int PAR = decltype(par_c)::value;
        char* const q_cur = PAR ? q_lds1 : q_lds0;
        char* const g_cur = PAR ? g_lds1 : g_lds0;
        char* const q_nxt = PAR ? q_lds0 : q_lds1;
        char* const g_nxt = PAR ? g_lds0 : g_lds1;
        const float* st = stat + PAR * 2 * DT_ROWS;
        const float* st_nxt = stat + (1 - PAR) * 2 * DT_ROWS;       // statistics of tile t + 1
        dkdv_step<true, MASK, DP, PART>(s_a, dp_a, s_b, dp_b, acck, accv, kf, vf, kappa, arow, tr0, tr1,
                              q_cur + tile_bytes(DP) / 2, g_cur + tile_bytes(DP) / 2, q_cur, g_cur, st, st + 32, h,
                              mask_at, part_ks);
        if (!last) {
            stat_store(1 - PAR, rstat);          // fetched at the end of the previous trip
            __builtin_amdgcn_s_waitcnt(0);       // tile t+1, requested one iteration ago, has landed
            __syncthreads();
        }
        dkdv_step<!last, MASK, DP, PART>(s_b, dp_b, s_a, dp_a, acck, accv, kf, vf, kappa, arow, tr0, tr1, q_nxt,
                              g_nxt, q_cur + tile_bytes(DP) / 2, g_cur + tile_bytes(DP) / 2, st + 32, st_nxt, h,
                              mask_at - 32, part_ks);
        if (REQ) {
            __syncthreads();                     // every wavefront is done with tile t
            load_tile(Qr, at, q_cur);
            load_tile(Gr, at, g_cur);
            rstat = stat_fetch();
        }
    };
    using T = std::true_type;
    using F = std::false_type;
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using M = std::integral_constant<bool, WALK != WALK_FULL>;
    // t_first and n_qt are even (c and k0 are multiples of 128, or tiles are counted in pairs): trips
    // come in pairs.  Masked pairs up to the diagonal (one, more under emulated coarse skipping),
    // plain pairs, and the last pair of the block, in masked form (beyond the diagonal the limit is
    // negative and removes nothing).
    // DP = 256: one form (masked unless the block is full) for every pair but the last.  With a second, unmasked copy of the
    // loop this instantiation, which is over the register budget, kept spilled registers live
    // across its hot loop, and every reload there waits for the tile loads in flight as well.
    constexpr bool ONE_FORM = DP > 128;
    int t = t_first;
    for (;;) {
        int mask_at = mask_base - 64 * t, at = (t + 2) * tile_pitch;
        if (t + 2 < n_qt && !ONE_FORM && t >= t_plain) {
            for (; t + 2 < n_qt; t += 2) {              // the hot loop
                trip(F{}, P0{}, F{}, T{}, 0, (t + 2) * tile_pitch);
                trip(F{}, P1{}, F{}, T{}, 0, (t + 3) * tile_pitch);
            }
            if (WALK == WALK_FULL) break;               // nothing else comes before the last pair
            continue;
        }
        if (WALK == WALK_FULL && !ONE_FORM) break;
        if (t + 2 >= n_qt) {                            // last pair of the block
            if (!RING) break;
            if (++q_dev == p.q_dev + p.n_q) {
                q_dev = dev0;
                if (++q_head == group) break;
            }
            enter_block();
            t = t_first - 2;
            at = t_first * tile_pitch;
        }
        trip(M{}, P0{}, F{}, T{}, mask_at, at);
        trip(M{}, P1{}, F{}, T{}, mask_at - 64, at + tile_pitch);
        t += 2;
    }
    trip(M{}, P0{}, F{}, F{}, mask_base - 64 * t, 0);
    trip(M{}, P1{}, T{}, F{}, mask_base - 64 * t - 64, 0);

#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = 128 * ohalf + 32 * mb + 8 * g + 4 * h;
            if (col >= d || !key_ok) continue;            // padding columns, keys beyond the shard
            const int64_t o = (int64_t)key * ss + col;
            float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
            if (!RING || !p.fresh) {
                x = *reinterpret_cast<float4*>(DV + o);
                y = *reinterpret_cast<float4*>(DK + o);
            }
            x.x += accv[mb][4 * g + 0]; x.y += accv[mb][4 * g + 1];
            x.z += accv[mb][4 * g + 2]; x.w += accv[mb][4 * g + 3];
            *reinterpret_cast<float4*>(DV + o) = x;
            y.x = fmaf(p.scale, acck[mb][4 * g + 0], y.x); y.y = fmaf(p.scale, acck[mb][4 * g + 1], y.y);
            y.z = fmaf(p.scale, acck[mb][4 * g + 2], y.z); y.w = fmaf(p.scale, acck[mb][4 * g + 3], y.w);
            *reinterpret_cast<float4*>(DK + o) = y;
        }
}

// Head dimensions above 128, both column halves of dK and dV in one workgroup.  The kernel above forms
// S and dP once per half: 12 products of d columns a pair where 8 do.  Here dK^T and dV^T of 32
// keys and 256 columns are the 256 accumulation registers of a wavefront (one per SIMD), the K rows
// 64 of its vector registers and the V rows WIDE_V_REGS k-steps there, the others in LDS, written and
// read by their own wavefront alone.  Q and dO come in stages of 32 rows, three in LDS: stage u + 2 is
// requested when everyone is done with u - 1 and has the whole step u to land, one barrier a step.
// The walk over blocks is the requests' own, two stages ahead; a step knows only its stage's limit
// of the element mask, which is far below zero where nothing is masked (64 matrix products a step
// hide the 16 selects).
// Bound by the matrix cores at the clock the power limit leaves: 8 instead of 12 products of d a pair,
// one wavefront per SIMD.  Backward step (with its dQ kernel), 8 heads of 8192 rows, d 256, full block
// 2210 -> 1761 us, triangular 1282 -> 1014; 12500 rows 6276 -> 5363, 2905 -> 2212; 16 heads of 4096 1166 ->
// 944, 708 -> 562.  One or two k-steps of V in registers measured the same.
constexpr int WIDE_ROWS = 32, WIDE_PART = WIDE_ROWS * 256;         // one 128-column half of a stage's Q or dO
constexpr int WIDE_STAGE = 4 * WIDE_PART;                          // Q, Q, dO, dO
constexpr int WIDE_V_REGS = 1;                                     // of 16 k-steps: what LDS has no room for
constexpr int WIDE_V_LDS = (16 - WIDE_V_REGS) * 1024;              // per wavefront
constexpr int WIDE_NO_MASK = -(1 << 20);

// products of one step, as dkdv_step.  arow: row reads in the next stage, tr0 / tr1: transposing reads
// in the present one.
template <bool NEXT>
__device__ __forceinline__ void wide_step(f32x16& s_cur, f32x16& dp_cur, f32x16& s_next, f32x16& dp_next,
                                 const bf16x8 (&kf)[16],
                                 const bf16x8 (&vf)[WIDE_V_REGS], const char* v_own, float kappa, const char* lds,
                                 const uint32_t (&arow)[8], const uint32_t (&tr0)[4], const uint32_t (&tr1)[4],
                                 const float* stat_cur, const float* stat_next, int h, int mask_lim) {
    bf16x8 qa[16], ga[16], va[16], qt[16], gt[16], pb[2], dsb[2];
    if (NEXT) load_neg_delta(dp_next, stat_next + WIDE_ROWS, h);
    auto fetch = [&](int ks) {
        if (!NEXT) return;
        const char* rows = lds + (ks / 8) * WIDE_PART;
        qa[ks] = dt_read_row(rows, arow[ks % 8]);
        ga[ks] = dt_read_row(rows + 2 * WIDE_PART, arow[ks % 8]);
        va[ks] = ks < WIDE_V_REGS ? vf[ks % WIDE_V_REGS] : dt_read_row(v_own, (ks - WIDE_V_REGS) * 1024);
    };
    // i = 8 (group of 16 rows) + column block
    auto fetch_t = [&](int i) {
        const char* rows = lds + (i % 8 / 4) * WIDE_PART + (i / 8) * 16 * 256;
        gt[i] = dt_read_tr(rows + 2 * WIDE_PART, tr0[i % 4], tr1[i % 4]);
        qt[i] = dt_read_tr(rows, tr0[i % 4], tr1[i % 4]);
    };
    float2 lv[8];
    auto fetch_stat = [&](int i) {
        lv[i] = *reinterpret_cast<const float2*>(stat_cur + 8 * (i / 2) + 4 * h + 2 * (i % 2));
    };
    constexpr int AHEAD = 2, TAHEAD = 3;
    fetch_stat(0);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fetch(i);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        __builtin_amdgcn_sched_barrier(0);          // slices stay in program order
        if (i + AHEAD < 16) fetch(i + AHEAD);
        if (i % 2 == 0 && i < 14) fetch_stat(i / 2 + 1);
        if (i >= 16 - TAHEAD) fetch_t(i - (16 - TAHEAD));
        if (NEXT) {
            if (i == 0) mfma_vgpr_first(s_next, qa[i], kf[i], false);
            else mfma_vgpr_acc(s_next, qa[i], kf[i], false);
            __builtin_amdgcn_sched_barrier(0);
        }
        const float lr = i % 2 ? lv[i / 2].y : lv[i / 2].x;
        float pr = __builtin_amdgcn_exp2f(fmaf(s_cur[i], kappa, -lr));
        if (8 * (i / 4) + (i % 4) < mask_lim) pr = 0.f;
        pb[i / 8][i % 8] = (__bf16)pr;
        dsb[i / 8][i % 8] = (__bf16)(pr * dp_cur[i]);
        if (NEXT) {
            __builtin_amdgcn_sched_barrier(0);
            mfma_vgpr_acc(dp_next, ga[i], va[i], false);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        if (i + TAHEAD < 16) fetch_t(i + TAHEAD);
        acc_mfma(i % 8, gt[i], pb[i / 8]);
        acc_mfma(8 + i % 8, qt[i], dsb[i / 8]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <bool BY_RANK>
__global__ void __launch_bounds__(256, 1)
bwd_dkdv_wide_kernel(StepArgs p, int n_tiles) {
    __shared__ __attribute__((aligned(1024))) char lds[3 * WIDE_STAGE];
    __shared__ __attribute__((aligned(1024))) char v_lds[4 * WIDE_V_LDS];
    __shared__ __attribute__((aligned(16))) float stat[3 * 2 * WIDE_ROWS];         // [stage][lse2 | -delta][32]
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int ktile, bh, dev_rank;
    decode_block<false, BY_RANK>((int)blockIdx.x, n_tiles * p.n_kv, p.B * p.H_kv, ktile, bh);
    decode_rank(ktile, n_tiles, p.n_kv, p.layout, ktile, dev_rank);
    const int dev = p.kv_dev + dev_rank;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + (dev - p.kv_dev) * p.kv_shard;
    const int d = p.d;
    const int64_t ss = p.kv_stride_s;
    const int pitch = 2 * (int)p.stride_s, stage_pitch = WIDE_ROWS * pitch;
    const int k0 = ktile * BM, key_own = k0 + 32 * wave + n, key = min(key_own, p.c - 1);

    // The requests: query head, query shard and 32-row stage of the next one, as in the kernel above.
    const int group = p.H / p.H_kv;
    const int dev0 = p.layout != SA_STRIPED ? max(p.q_dev, dev) : p.q_dev, n_st = (p.c + DT_ROWS - 1) / DT_ROWS * 2;
    int q_head = 0, q_dev = dev0, t, lim;           // lim: mask limit of stage 0 but for the lane's part
    dt_rsrc Qr, Gr;
    const float* stat_src;
    auto enter_block = [&]() {
        const int hd = kvh * group + q_head;
        const bool tri = block_kind(q_dev, dev, p.layout) == MASK_TRI;
        const int off = block_off(q_dev, dev, p.layout);
        t = tri ? k0 / WIDE_ROWS : 0;
        if (tri && p.skip_bq > 0)
            t = ((k0 / p.skip_bk * p.skip_bk + off) / p.skip_bq) * p.skip_bq / WIDE_ROWS;
        lim = tri ? k0 + 32 * wave + off : WIDE_NO_MASK;
        const int64_t base = b * p.stride_b + hd * p.stride_h + (q_dev - p.q_dev) * p.q_shard;
        const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(q_dev - p.q_dev) * p.c;
        Qr = dt_make_rsrc((const __bf16*)p.q + base, p.c, pitch, d);
        Gr = dt_make_rsrc((const __bf16*)p.dout + base, p.c, pitch, d);
        stat_src = ((tid & WIDE_ROWS) ? p.delta : p.lse) + sbase;
    };
    enter_block();
    uint32_t gl[2][2];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int r = 8 * wave + 4 * j + (lane >> 4), chunk = (lane & 15) ^ dt_swz(r);
            gl[hh][j] = 128 * hh + 8 * chunk < d ? r * pitch + 256 * hh + (chunk << 4) : DT_OUT_OF_RANGE;
        }
    float rstat;                                    // statistics of the stage requested last
    int lim_req;                                    // and its limit
    bool more = true;                               // stages are left to request
    auto request = [&](int stage) {
        const int at = t * stage_pitch;
        char* dst = lds + stage * WIDE_STAGE + 2 * wave * 1024;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                dt_load_piece(Qr, at, gl[hh][j], dst + hh * WIDE_PART + j * 1024);
                dt_load_piece(Gr, at, gl[hh][j], dst + (2 + hh) * WIDE_PART + j * 1024);
            }
        const int row = t * WIDE_ROWS + (tid & (WIDE_ROWS - 1));
        rstat = stat_src[min(row, p.c - 1)];
        if (row >= p.c) rstat = (tid & WIDE_ROWS) ? 0.f : INFINITY;       // no query: P and dS are exact zeros
        lim_req = lim == WIDE_NO_MASK ? lim : lim - t * WIDE_ROWS;
        if (++t == n_st) {
            if (++q_dev == p.q_dev + p.n_q) {
                q_dev = dev0;
                more = ++q_head < group;
            }
            if (more) enter_block();
        }
    };
    auto stat_store = [&](int stage) {
        if (tid < 2 * WIDE_ROWS) stat[stage * 2 * WIDE_ROWS + tid] = rstat * ((tid & WIDE_ROWS) ? -1.f : LOG2E);
    };

    bf16x8 kf[16], vf[WIDE_V_REGS];
    char* const v_own = v_lds + wave * WIDE_V_LDS + lane * 16;
    {
        bf16x8 v_all[16];
        load_b_frags<16>(v_all, (const __bf16*)p.v + kv_base + (int64_t)key * ss, h, d);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) {
            if (ks < WIDE_V_REGS) vf[ks % WIDE_V_REGS] = v_all[ks];
            else *reinterpret_cast<bf16x8*>(v_own + (ks - WIDE_V_REGS) * 1024) = v_all[ks];
        }
    }
    load_b_frags<16>(kf, (const __bf16*)p.k + kv_base + (int64_t)key * ss, h, d);
    request(0);
    const int lim_first = lim_req;
    stat_store(0);
    request(1);
    uint32_t arow[8], tr0[4], tr1[4];
    dt_row_addrs<256>(arow, n, h);
    dt_tr_addrs<256>(tr0, tr1, lane);
    const float kappa = p.scale * LOG2E;
#pragma unroll
    for (int r = 0; r < 256; ++r) acc_zero(r);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    f32x16 s_a, s_b, dp_a, dp_b;
    load_neg_delta(dp_a, stat + WIDE_ROWS, h);
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const char* rows = lds + (ks / 8) * WIDE_PART;
        const bf16x8 qx = dt_read_row(rows, arow[ks % 8]), gx = dt_read_row(rows + 2 * WIDE_PART, arow[ks % 8]);
        const bf16x8 vx = ks < WIDE_V_REGS ? vf[ks % WIDE_V_REGS] : dt_read_row(v_own, (ks - WIDE_V_REGS) * 1024);
        if (ks == 0) mfma_vgpr_first(s_a, qx, kf[ks], false);
        else mfma_vgpr_acc(s_a, qx, kf[ks], false);
        mfma_vgpr_acc(dp_a, gx, vx, false);
    }
    mfma_results_to_valu(s_a, dp_a);

    // stage: of the present step.  The row reads are one stage further on.
    int stage = 0, ahead = 2, lim_cur = lim_first, lim_next = lim_req;         // ahead: stages requested and not done
    auto after = [](int x) { return x == 2 ? 0 : x + 1; };
    auto move = [&](uint32_t (&a)[8], int from) {
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] += from == 2 ? -2 * WIDE_STAGE : WIDE_STAGE;
    };
    move(arow, 0);
    auto step = [&](f32x16& s_cur, f32x16& dp_cur, f32x16& s_next, f32x16& dp_next) {
        const int next = after(stage), free = after(next);
        stat_store(next);
        __builtin_amdgcn_s_waitcnt(0);              // the next stage has landed
        __syncthreads();                            // for everyone; everyone is done with the one before this
        if (more) {
            request(free);
            ++ahead;
        }
        wide_step<true>(s_cur, dp_cur, s_next, dp_next, kf, vf, v_own, kappa, lds, arow, tr0, tr1,
                        stat + stage * 2 * WIDE_ROWS, stat + next * 2 * WIDE_ROWS, h, lim_cur + n - 4 * h);
        lim_cur = lim_next;
        lim_next = lim_req;
        move(arow, next);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            tr0[i] += stage == 2 ? -2 * WIDE_STAGE : WIDE_STAGE;
            tr1[i] += stage == 2 ? -2 * WIDE_STAGE : WIDE_STAGE;
        }
        stage = next;
        --ahead;
    };
    for (;;) {          // every block has an even number of stages
        step(s_a, dp_a, s_b, dp_b);
        if (ahead == 1) break;
        step(s_b, dp_b, s_a, dp_a);
    }
    wide_step<false>(s_b, dp_b, s_a, dp_a, kf, vf, v_own, kappa, lds, arow, tr0, tr1,
                     stat + stage * 2 * WIDE_ROWS, stat, h, lim_cur + n - 4 * h);

    acc_settle();
    if (key_own >= p.c) return;
    float* DK = p.dk + kv_base + (int64_t)key * ss;
    float* DV = p.dv + kv_base + (int64_t)key * ss;
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int col = 32 * mb + 8 * g + 4 * h;
            if (col >= d) continue;
            float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
            if (!p.fresh) {
                x = *reinterpret_cast<float4*>(DV + col);
                y = *reinterpret_cast<float4*>(DK + col);
            }
            x.x += acc_read(16 * mb + 4 * g + 0); x.y += acc_read(16 * mb + 4 * g + 1);
            x.z += acc_read(16 * mb + 4 * g + 2); x.w += acc_read(16 * mb + 4 * g + 3);
            *reinterpret_cast<float4*>(DV + col) = x;
            y.x = fmaf(p.scale, acc_read(128 + 16 * mb + 4 * g + 0), y.x); y.y = fmaf(p.scale, acc_read(128 + 16 * mb + 4 * g + 1), y.y);
            y.z = fmaf(p.scale, acc_read(128 + 16 * mb + 4 * g + 2), y.z); y.w = fmaf(p.scale, acc_read(128 + 16 * mb + 4 * g + 3), y.w);
            *reinterpret_cast<float4*>(DK + col) = y;
        }
}

template <bool RAGGED, int WALK, int DP, bool PART, bool BY_RANK>
__global__ void __launch_bounds__(256, DP > 128 ? 1 : 2)
bwd_dq_mfma_kernel(StepArgs p, int n_tiles) {
    __shared__ __attribute__((aligned(1024))) char lds0[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds1[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds2[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds3[tile_bytes(DP) * halves_of(DP)];
    bwd_dq<RAGGED, WALK, DP, PART, BY_RANK>(p, n_tiles, (int)blockIdx.x, lds0, lds1, lds2, lds3);
}
// WAVES: wavefronts per SIMD the register budget is cut for.  Up to 64 columns two fit (half the
// operands and accumulators; the loops do not spill), and with half of the products per score it is
// the vector work that needs hiding: 16 heads, d 64, backward step, 12500 tokens triangular
// 1.46 -> 1.37 ms, full 2.87 -> 2.46; 32 heads of 32768, triangular, 17.3 -> 14.7 ms.
template <int WALK, bool RAGGED, int DP, bool PART, int WAVES, bool BY_RANK>
__global__ void __launch_bounds__(256, WAVES)
bwd_dkdv_mfma_kernel(StepArgs p, int n_tiles) {
    __shared__ __attribute__((aligned(1024))) char lds0[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds1[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds2[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds3[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(16))) float stat[KV_STAT_FLOATS];
    bwd_dkdv<WALK, RAGGED, DP, PART, BY_RANK>(p, n_tiles, (int)blockIdx.x, lds0, lds1, lds2, lds3, stat);
}
// Both kinds of workgroups in one launch (each sequence heaviest first; above 512 of a kind by groups of
// heads, see decode_block): where the key-owning ones do not fill the chip, or fill it once and last
// as long as the heaviest, the query-owning ones run beside and behind them instead of after.
// One workgroup per compute unit (the key-owning side's registers).  Up to 64 columns and above 128.
template <bool RAGGED, int DP, bool PART>
__global__ void __launch_bounds__(256, 1)
bwd_both_mfma_kernel(StepArgs p, int n_tiles, PlacedKinds kinds) {
    __shared__ __attribute__((aligned(1024))) char lds0[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds1[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds2[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(1024))) char lds3[tile_bytes(DP) * halves_of(DP)];
    __shared__ __attribute__((aligned(16))) float stat[KV_STAT_FLOATS];
    int linear = (int)blockIdx.x;
    const int keys = __builtin_amdgcn_readfirstlane(owns_keys(kinds, linear));
    linear = __builtin_amdgcn_readfirstlane(linear);        // (both kept scalar)
    if (keys) bwd_dkdv<WALK_RING, RAGGED, DP, PART, false>(p, n_tiles, linear, lds0, lds1, lds2, lds3, stat);
    // (by heads or groups of them, both)
    else bwd_dq<RAGGED, WALK_RING, DP, PART, false>(p, n_tiles, linear, lds0, lds1, lds2, lds3);
}

}  // namespace

bool bwd_mfma_supported(const StepArgs& a, int dtype) {
    // the tile loads address a shard through a buffer descriptor with 32-bit byte offsets:
    // the last row of its last (possibly partial) tile pair must end below 2^31 bytes from
    // its first
    const int64_t widest = a.stride_s > a.kv_stride_s ? a.stride_s : a.kv_stride_s;
    const int64_t rows = (int64_t)(a.c + BM - 1) / BM * BM;
    // one workgroup per (128-row tile, device, batch, head) in a 1-D grid
    if (rows / BM * a.B * a.H * (a.n_q > a.n_kv ? a.n_q : a.n_kv) >= (int64_t(1) << 31)) return false;
    // head dimensions above 128 (two 128-column halves) in whole 16-byte chunks only
    if (a.d > 2 * D || (a.d > D && a.d % 8)) return false;
    return dtype == SA_BF16 && a.d % 4 == 0 && a.c >= BM &&
           rows * 2 * widest + 2 * a.d < (int64_t(1) << 31);
}

// Key-owning workgroups by ranks (decode_block).  Above 128 columns up to 1408 tiles; d 192 and 256, triangular step, us,
// groups : ranks: 24 heads of 4096 529 : 465, 540 : 472, 44 of 4096 856 : 815, 897 : 878, 48 of 4096 849 : 891, 1030 : 1073,
// 64 of 4096 1134 : 1217, 1186 : 1357; heads of few tiles a round or two more, whole backward, 384 of 512 624 : 592, 512 of 512
// 872 : 851, 192 of 1024 .98.
// A device's own queries against more shards of keys: every walk is that device's rows, and short ones leave little to
// balance while an XCD's heads, all at a time, fall out of its L2.  Striped shares, whole backward, groups : ranks: d 128,
// 32 heads 4 x 1024 195 : 211, 64 of 4 x 1024 346 : 390, d 100, 64 of 4 x 1000 319 : 342, d 256, 32 of 8 x 512 340 : 434, of
// 2 x 2048 1 : 1.05; but 64 columns, 32 of 2 x 4096 1 : .94, 64 of 2 x 1024 124 : 118, up to three rounds 24 of 4 x 1000 1 :
// .96, 24 of 2 x 2048 1 : .94, and with 32 columns computed, whose rows are few bytes, all: 64 of 2 x 1024 78 : 70, 32 of 8 x
// 1024 155 : 150.
bool dkdv_by_rank(const StepArgs& a) {
    const int64_t ranks = (int64_t)((a.c + BM - 1) / BM) * a.n_kv, tiles = ranks * a.B * a.H_kv, walk = (int64_t)a.c * a.n_q * (a.H / a.H_kv);
    if (!by_rank(uneven(a), tiles, a.d > 128 ? (ranks <= 4 ? 8 * N_CU : ranks <= 8 ? 6 * N_CU : 6 * N_CU - 1) : a.d > 112 ? MOST_BY_RANK<128, false> : MOST_BY_RANK<64, false>)) return false;
    if (a.n_kv <= a.n_q || a.d <= 32) return true;
    return walk > (a.d > 128 ? 2048 : 2047) || (walk > 512 && tiles <= (a.d <= 112 && a.n_kv <= 2 * a.n_q ? 4 : 3) * N_CU);
}

// Both kinds of workgroups in one launch.  Measured per backward step, one launch / two, us.  Up to 64 columns and above 128 (this
// file's kernels; measured at d 128, when they ran there too): uneven work up to one key-owning workgroup per compute unit: 2048 x
// 2048 triangular, 2 heads 60 / 102, 8 heads 66 / 106, 16 heads (256 workgroups) 92 / 115, 24 heads 137 / 131.  Even work (a full
// block) has no tail to fill, only idle compute units: 128 + 128 workgroups 75 / 108, 256 + 256 144 / 133.  d 256 (two
// key-owning workgroups per tile): 256 of them 109 / 189, 512 207 / 225.
// 65 to 128 columns (bwd_ring.hip, whose query-owning workgroups lose less where one is alone on its compute unit), d 128 and d 100:
//  * uneven work, key tiles: 192 (16 heads of 1536) 51 / 83, 44 / 78, 256 (16 of 2048) 75 / 104, 67 / 98, (32 on 8 of 4096) 452 / 546,
//    419 / 525, 294 (3 of 12500) 392 / 525, 364 / 510, 320 (10 of 4096) 170 / 199, 147 / 186, (20 of 2048) 101 / 111, 88 / 104, (5 of 8192) 292 /
//    361, 270 / 348, 384 (12 of 4096) 191 / 203, 174 / 193, (24 of 2048) 113 / 119, 101 / 109; behind the line 512 (16 of 4096) 263 / 248;
//    four query heads to a key/value head 320 (10 of 4096) 582 / 622, 539 / 591, behind the line 384 699 / 692;
//  * of these, walks of many blocks of two or three tiles: two launches again from 257 key tiles on.  The kinds go out evenly (see
//    launch_both) and the last key walks start late: 987 heads on 141 of 256 rows, d 96, 164 / 144, 1540 on 140 of 235, d 80, 224 /
//    190, 240 on 80, 2 x 253 rows, d 128, 139 / 123; but one tile, 2264 on 283 of 128 rows, d 100, 167 / 196, four, 455 on 65 of 512 205 /
//    210, twelve, 152 on 19 of 1445 351 / 410;
//  * a full block, workgroups of both kinds: 256 (8 heads of 2048) 65 / 99, 59 / 96, 320 (10 of 2048) 93 / 102, 87 / 99, (40 of 512) 38 / 45, 34 / 41,
//    352 (44 of 512) 43 / 45, 38 / 43; behind the line 384 (12 of 2048) 110 / 107;
//  * one device's queries against more shards of keys: its query-owning workgroups, one round at most, walk all of them, and the
//    others fill the chip meanwhile.  Striped, device 7 of 8: 4 heads of 2048 295 / 367, 293 / 361, 16 of 1024 173 / 258, 166 / 248, 32 of
//    1024 (256 and 2048 tiles) 332 / 393, 297 / 353, 32 on 8 of 1024 285 / 323, 263 / 305; 2 of 8192, N 4, 609 / 805, 592 / 789;
//    contiguous 8 of 2048, N 4, 208 / 276, 196 / 266, 4 of 4096, N 8, 797 / 1027, 743 / 991; behind the line, with the key walks in front,
//    64 of 1024, N 4 (512 query tiles) 393 / 342, 32 of 896, N 16 (3584 key tiles) 860 / 658.
bool bwd_one_launch(const StepArgs& a) {
    const int n_tiles = (a.c + BM - 1) / BM, halves = a.d > D ? 2 : 1, group = a.H / a.H_kv;
    const int64_t keys = (int64_t)n_tiles * a.n_kv * a.B * a.H_kv * halves, queries = (int64_t)n_tiles * a.n_q * a.B * a.H;
    if (a.d <= 64 || a.d > D) return uneven(a) ? keys <= N_CU * halves : keys + queries <= N_CU;
    if (a.n_kv > a.n_q && queries <= N_CU && keys <= 8 * N_CU) return true;
    if (!uneven(a)) return keys + queries <= 11 * N_CU / 8;
    if (keys > N_CU && (n_tiles == 2 || n_tiles == 3) && (int64_t)group * a.n_q > 5) return false;
    return keys <= (group < 4 ? 6 : 5) * N_CU / 4;
}

namespace {
template <int WALK, int DP, bool PART, bool BY_RANK = false>
void launch_dq(const StepArgs& a, hipStream_t st, int n_tiles) {
    const dim3 grid((unsigned)n_tiles * a.n_q * a.B * a.H), block(256);
    if constexpr (WALK != WALK_FULL && !BY_RANK)
        // (between 64 and 128 columns computed many heads or few tiles lose, us, groups : ranks: d 100, whole backward, 336 heads of
        // 384 153 : 162, 256 of 2 x 512 409 : 422, 512 of 768 627 : 648)
        if (by_rank(uneven(a), grid.x, MOST_BY_RANK<DP, false>) && (DP != 112 || (a.B * a.H <= 192 && n_tiles * a.n_q >= 4))) return launch_dq<WALK, DP, PART, true>(a, st, n_tiles);
    if (a.c % BM) hipLaunchKernelGGL((bwd_dq_mfma_kernel<true, WALK, DP, PART, BY_RANK>), grid, block, 0, st, a, n_tiles);
    else hipLaunchKernelGGL((bwd_dq_mfma_kernel<false, WALK, DP, PART, BY_RANK>), grid, block, 0, st, a, n_tiles);
}
template <int WALK, int DP, bool PART, int WAVES, bool BY_RANK = false>
void launch_dkdv_waves(const StepArgs& a, hipStream_t st, int n_tiles) {
    const dim3 grid((unsigned)n_tiles * a.n_kv * a.B * a.H_kv * halves_of(DP)), block(256);
    if constexpr (WALK != WALK_FULL && DP <= 128 && !BY_RANK)          // (above: bwd_dkdv_wide_kernel)
        if (dkdv_by_rank(a)) return launch_dkdv_waves<WALK, DP, PART, WAVES, true>(a, st, n_tiles);
    if (a.c % BM) hipLaunchKernelGGL((bwd_dkdv_mfma_kernel<WALK, true, DP, PART, WAVES, BY_RANK>), grid, block, 0, st, a, n_tiles);
    else hipLaunchKernelGGL((bwd_dkdv_mfma_kernel<WALK, false, DP, PART, WAVES, BY_RANK>), grid, block, 0, st, a, n_tiles);
}
template <int WALK, int DP, bool PART>
void launch_dkdv(const StepArgs& a, hipStream_t st, int n_tiles) {
    if constexpr (DP <= 64) {
        // Uneven work that two workgroups per compute unit would hold all at once, or whose longest walk is
        // short, is better taken up one after the other, heaviest first (triangular, whole step: 512
        // workgroups of 4096 rows 0.168 against 0.177 ms; 768 of 1024, 2048 and 4096 rows 116 / 124, 157 /
        // 173, 266 / 257 us; 1536 of 2048 and 4096 291 / 304, 460 / 458).
        const int64_t wgs = (int64_t)n_tiles * a.n_kv * a.B * a.H_kv;
        if (!uneven(a) || (wgs > 2 * N_CU && n_tiles >= 32))
            return launch_dkdv_waves<WALK, DP, PART, 2>(a, st, n_tiles);
    }
    launch_dkdv_waves<WALK, DP, PART, 1>(a, st, n_tiles);
}
template <int DP, bool PART>
hipError_t launch_both(const StepArgs& a, hipStream_t st, int n_tiles) {
    const int n_dkdv = n_tiles * a.n_kv * a.B * a.H_kv * halves_of(DP), n_dq = n_tiles * a.n_q * a.B * a.H;
    // (The ratio, and none for groups: a group's long key walks in front are no gain.  25 calls of 65 to 384 key tiles with
    // bwd_ring.hip's kernels, at d 128 and d 100, time against these: ratio 1.25 0.98 to 1.02, 1.7 0.97 to 1.03; for groups 0.35
    // 0.99 to 1.05, 0.5 0.98 to 1.04: 455 heads on 65 of 512 rows 205 / 211 and 214 us, 32 on 8 of 4096 463 / 461 and 456.)
    // (numbers that are no multiple of 8 one by one: 11 heads of 1600 rows, d 136, 92 us, in units of 8 97; those that are:
    // see both_kinds)
    const double ratio = a.H == a.H_kv ? 1.45 : 0.;
    const PlacedKinds kinds = placed_kinds(a, n_dkdv, n_dq, ratio);
    if constexpr (DP == 112 || DP == 128) {
        return launch_bwd_ring(a, &kinds, n_dkdv + n_dq, st);
    } else {
        const dim3 grid((unsigned)(n_dkdv + n_dq)), block(256);
        if (a.c % BM) hipLaunchKernelGGL((bwd_both_mfma_kernel<true, DP, PART>), grid, block, 0, st, a, n_tiles, kinds);
        else hipLaunchKernelGGL((bwd_both_mfma_kernel<false, DP, PART>), grid, block, 0, st, a, n_tiles, kinds);
        return hipGetLastError();
    }
}
template <int DP, bool PART>
hipError_t launch_bwd_variant(const StepArgs& a, hipStream_t st) {
    const int n_tiles = (a.c + BM - 1) / BM;
    if (bwd_one_launch(a)) return launch_both<DP, PART>(a, st, n_tiles);
    const bool one_block = a.n_q == 1 && a.n_kv == 1 && !a.fresh;
    const bool full = block_kind(a.q_dev, a.kv_dev, a.layout) == MASK_FULL;
    if (!one_block) launch_dq<WALK_RING, DP, PART>(a, st, n_tiles);
    else if (full) launch_dq<WALK_FULL, DP, PART>(a, st, n_tiles);
    else launch_dq<WALK_TRI, DP, PART>(a, st, n_tiles);
    if (hipError_t e = hipGetLastError()) return e;
    if constexpr (DP > 128) {
        // Up to half a key tile per compute unit the two column halves side by side are faster: a wide workgroup
        // lasts 4 / 3 as long.  Full block, d 256, us, halves : wide: 128 tiles (8 heads of 2048) 197 : 224, (32
        // heads on 4 of 4096) 2251 : 2718, 144 278 : 228, 192 280 : 227, 256 315 : 256, 320 475 : 463.  Triangular
        // blocks of up to 256 tiles went to launch_both (16 heads of 2048 204 : 218, 8 of 4096 342 : 385; above it
        // 320 tiles 285 : 239).
        const int64_t tiles = (int64_t)n_tiles * a.n_kv * a.B * a.H_kv;
        if (tiles > N_CU / 2) {
            if (dkdv_by_rank(a)) hipLaunchKernelGGL(bwd_dkdv_wide_kernel<true>, dim3((unsigned)tiles), dim3(256), 0, st, a, n_tiles);
            else hipLaunchKernelGGL(bwd_dkdv_wide_kernel<false>, dim3((unsigned)tiles), dim3(256), 0, st, a, n_tiles);
            return hipGetLastError();
        }
    }
    if constexpr (DP == 112 || DP == 128) return launch_bwd_ring(a, nullptr, n_tiles * a.n_kv * a.B * a.H_kv, st);
    // query heads that share a key/value head are blocks of one walk
    else if (!one_block || a.H != a.H_kv) launch_dkdv<WALK_RING, DP, PART>(a, st, n_tiles);
    else if (full) launch_dkdv<WALK_FULL, DP, PART>(a, st, n_tiles);
    else if constexpr (DP <= 128) launch_dkdv<WALK_TRI, DP, PART>(a, st, n_tiles);      // above: launch_both or wide
    return hipGetLastError();
}
}  // namespace

hipError_t launch_bwd_mfma(const StepArgs& a, hipStream_t st) {
    const bool part = a.d % 8 != 0;
    if (a.d > 128) return launch_bwd_variant<256, false>(a, st);
    if (a.d <= 32 && !part) return launch_bwd_variant<32, false>(a, st);
    if (a.d <= 64) return part ? launch_bwd_variant<64, true>(a, st) : launch_bwd_variant<64, false>(a, st);
    if (a.d <= 112) return part ? launch_bwd_variant<112, true>(a, st) : launch_bwd_variant<112, false>(a, st);
    return part ? launch_bwd_variant<128, true>(a, st) : launch_bwd_variant<128, false>(a, st);
}

}  // namespace sa
