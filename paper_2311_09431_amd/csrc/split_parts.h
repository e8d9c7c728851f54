// What the kernels share that give a workgroup 32 rows and split the streamed side over its wavefronts, each of
// which streams by itself (split_mfma.hip: bf16, f32x3_split.hip: fp32): waits, the walks' order, and the meeting of
// the partial results.
#pragma once
#include "f32_rows.h"
#include "f32_terms.h"
#include "mfma_tiles.h"
#include "sa_internal.h"

namespace sa {

constexpr int OWN = 32;
constexpr int STAT_BYTES = 512;         // 32 LSE, 32 delta, a load of 256 bytes each

__device__ inline f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

// 32 statistics from row `first` on
__device__ inline void load_stat(dt_rsrc m, int first, char* lds, int lane) {
    dt_load_dword(m, 4 * first, lane < 32 ? 4 * lane : DT_OUT_OF_RANGE, lds);
}

// bytes of the wavefronts' accumulators
template <int DP, int WAVES> constexpr int PARTIAL_BYTES = WAVES * blocks_of(DP) * 16 * 64 * 4;

// Sum of the wavefronts' accumulators through LDS: each writes its own and takes a share of the
// sum, pieces of 8 columns (4 a lane), so that a row's columns stay together.
template <int DP, typename Lane>
__device__ inline void put_partial(char* buf, const f32x16 (&acc)[4], const Lane& ln) {
    float4* mine = reinterpret_cast<float4*>(buf) + ln.wave * blocks_of(DP) * 4 * 64;
#pragma unroll
    for (int mb = 0; mb < blocks_of(DP); ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            mine[(mb * 4 + g) * 64 + ln.lane] =
                make_float4(acc[mb][4 * g], acc[mb][4 * g + 1], acc[mb][4 * g + 2], acc[mb][4 * g + 3]);
}
constexpr int share_of(int DP, int waves) { return (blocks_of(DP) * 4 + waves - 1) / waves; }   // pieces a wavefront takes
// (columns beyond the row's: no piece)
template <int DP, int WAVES, typename Lane>
__device__ inline int piece_of(int i, const Lane& ln) { return ln.wave * share_of(DP, WAVES) + i; }
template <int DP, int WAVES, typename Lane>
__device__ inline int column_of(int i, const Lane& ln) { return 8 * piece_of<DP, WAVES>(i, ln) + 4 * ln.h; }
template <int DP, int WAVES, typename Lane>
__device__ inline float4 take_sum(const char* buf, int i, const Lane& ln) {
    const float4* at = reinterpret_cast<const float4*>(buf) + piece_of<DP, WAVES>(i, ln) * 64 + ln.lane;
    float4 x = at[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
        const float4 y = at[w * blocks_of(DP) * 4 * 64];
        x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
    }
    return x;
}
// this wavefront's share of the lane's row as it stands (zeros if not wanted): on its way while the
// partial results meet
template <int DP, int WAVES, typename Lane>
__device__ inline void load_old(float4 (&x)[share_of(DP, WAVES)], const float* row, int d, bool wanted, const Lane& ln) {
#pragma unroll
    for (int i = 0; i < share_of(DP, WAVES); ++i) {
        const int col = column_of<DP, WAVES>(i, ln);
        x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (wanted && col < d) x[i] = *reinterpret_cast<const float4*>(row + col);
    }
}
// EXACT: rows that are done over one by one (f32_rows.h): each wavefront puts its mask beside its
// partial accumulators, and after the barrier takes every WAVES-th of the rows that one of them names
__device__ inline void put_odd(uint32_t* masks, bool odd, int wave, int lane) {
    const uint32_t rows = row_mask(odd);
    if (lane == 0) masks[wave] = rows;
}
template <int WAVES>
__device__ inline uint32_t take_odd(const uint32_t* masks) {
    uint32_t rows = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) rows |= masks[w];
    return __builtin_amdgcn_readfirstlane(rows);
}
// Rows to do over where operands are three bf16 terms: those that some wavefront names, and all with something in them if
// all are faint (f32_rows.h) in all wavefronts' partial results of one sum or of the other.  Each wavefront puts what it says
// of its 32 rows beside its partial results; behind the barrier a lane takes one wavefront's word and the lanes put them
// together.  Whether rows are all zero is asked only where no wavefront finds one loud.  (Words that the wavefronts add
// their bits to: 0.1 us of a small forward launch's 6, 0.3 of a backward one's 7.)
template <int WAVES>
struct RowsToRedo {
    uint4* words;               // one for each wavefront
    int lane, wave;
    uint32_t in_shard;
    __device__ inline void put(uint32_t x, uint32_t y, uint32_t z) const {
        if (lane == 0) words[wave] = make_uint4(x, y, z, 0);
    }
    template <int TURN>
    static __device__ inline uint32_t with_turned(uint32_t x) {         // of 16 lanes, TURN further on
        return x | (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x120 + TURN, 0xf, 0xf, true);
    }
    static __device__ inline uint32_t over_wavefronts(uint32_t x) {
        static_assert(WAVES == 4 || WAVES == 8, "");
        x = with_turned<2>(with_turned<1>(x));
        if (WAVES == 8) x = with_turned<4>(x);
        return __builtin_amdgcn_readfirstlane(x);
    }
    // top0, top1: the largest magnitudes of this wavefront's partial sums
    __device__ inline void put(bool odd, float top0, float top1) const {
        put(row_mask(odd), row_mask(top0 >= FAINT), row_mask(top1 >= FAINT));
    }
    __device__ inline uint32_t take(float top0, float top1) const {
        uint4 w = words[lane % WAVES];
        const uint32_t named = over_wavefronts(w.x), loud0 = over_wavefronts(w.y), loud1 = over_wavefronts(w.z);
        if (loud0 && loud1) return named;            // (as all wavefronts find)
        __syncthreads();
        put(0, row_mask(top0 > 0.f), row_mask(top1 > 0.f));
        __syncthreads();
        w = words[lane % WAVES];
        return named | (in_shard & ((loud0 ? 0 : over_wavefronts(w.y)) | (loud1 ? 0 : over_wavefronts(w.z))));
    }
};
// The sub-tiles of 32 keys that one wavefront of a query-owning workgroup takes: those of block kv whose
// number v is `turn` modulo the number of wavefronts, turn being the wavefront's number less the sub-tiles of
// the blocks before.
// Sub-tiles of a block that hold work for queries q0 .. q0 + 31: all of a full block; of a triangular
// one those up to the last allowed key, or under emulated coarse skipping up to the end of the
// skip_bk-wide tile that shares an allowed pair with the queries' skip_bq-tall tile.
struct KeyCursor {
    int kv, kv_end;             // present block; at kv_end the walk is over
    int v, n;                   // sub-tile, how many the block has
    int shift;                  // query a sees the block's keys up to min(a + shift, c - 1)
    int dev, layout, c, turn, n_full, n_off0, n_off1, n_fine;
    __device__ KeyCursor(const StepArgs& p, int dev_, int q0, int wave)
        : kv(p.kv_dev), kv_end(last_shard(p, dev_)), dev(dev_), layout(p.layout), c(p.c), turn(wave) {
        n_full = (p.c + 31) / 32;
        int end0 = min(q0 + OWN, p.c), end1 = end0 - 1;
        if (p.skip_bq > 0) {
            const int q_hi = (q0 / p.skip_bq + 1) * p.skip_bq - 1;
            end0 = min(p.c, (q_hi / p.skip_bk + 1) * p.skip_bk);
            end1 = min(p.c, ((q_hi - 1) / p.skip_bk + 1) * p.skip_bk);
        }
        n_off0 = (end0 + 31) / 32;
        n_off1 = (end1 + 31) / 32;
        n_fine = q0 / 32 + 1;
    }
    // to the wavefront's first sub-tile of block kv
    template <int WAVES>
    __device__ void enter() {
        const bool full = block_kind(dev, kv, layout) == MASK_FULL;
        const int off = block_off(dev, kv, layout);
        // (values, not members, to choose from: a choice between addresses keeps the object in memory)
        const int all = n_full, tri0 = n_off0, tri1 = n_off1, tri = n_fine;
        n = full ? all : off ? tri1 : tri0;
        shift = full ? c : -off;
        v = turn & (WAVES - 1);
        turn -= full ? all : tri;
    }
    template <int WAVES>
    __device__ void settle() {
        while (v >= n && kv < kv_end) {
            ++kv;
            enter<WAVES>();
        }
    }
};

// Forward, the end: the wavefronts' partial results (accumulators, base-2 reference m, half-wave row sum l) folded
// into the running state of the lane's row (base: of the workgroup's rows' matrix, a: the row, clamped to the shard).
// Returns the rows to do over (EXACT only; TERMS: V was three bf16 terms, masks are the words of RowsToRedo).
template <int DP, int WAVES, bool EXACT, bool TERMS, typename Lane>
__device__ __forceinline__ uint32_t fold_forward(const StepArgs& p, f32x16 (&acc)[4], float m, float l, char* lds, float* stats,
                                                 uint32_t* masks, const Lane& ln, int dev, int a_own, int a, float* L, float* O) {
    constexpr int MB = blocks_of(DP), N = share_of(DP, WAVES);
    const int n = ln.n, h = ln.h, d = p.d;
    const float old = p.fresh ? -INFINITY : *L;
    float4 o_old[N];
    load_old<DP, WAVES>(o_old, O, d, !p.fresh && a_own < p.c, ln);
    const float top_acc = TERMS ? loudest<MB>(acc) : 0.f;           // (beside the loads)
    // the wavefronts' partial results against a common reference
    const float l_own = half_wave_sum(l);
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
    put_partial<DP>(lds, acc, ln);
    // a row sum that is no positive number although the row sees a key: see f32_rows.h
    const RowsToRedo<WAVES> redo = {reinterpret_cast<uint4*>(masks), ln.lane, ln.wave, row_mask(a_own < p.c)};
    if (EXACT) {
        const bool odd = a_own < p.c && (not_finite<MB>(acc) || (!(l_tot > 0.f && l_tot < INFINITY) && sees_a_key(p, dev, a)));
        if (TERMS) redo.put(odd, top_acc * f, top_acc * f);
        else put_odd(masks, odd, ln.wave, ln.lane);
    }

    const float part = l_tot == 0.f ? -INFINITY : fmaf(m_all, LN2_HI, fmaf(m_all, LN2_LO, logf(l_tot)));
    const float top = fmaxf(old, part);
    const float ref = top == -INFINITY ? 0.f : top;
    const float w_old = expf(old - ref), w_part = expf(part - ref), w_sum = w_old + w_part;
    const float inv = w_sum > 0.f ? 1.f / w_sum : 0.f;
    const float f_old = w_old * inv, f_part = l_tot > 0.f ? w_part * inv / l_tot : 0.f;
    __syncthreads();
    const uint32_t odd_rows = TERMS ? redo.take(top_acc * f, top_acc * f) : EXACT ? take_odd<WAVES>(masks) : 0;
    // no row here, or no key seen: state unchanged
    if (a_own < p.c && !((odd_rows >> n) & 1) && (part != -INFINITY || p.fresh)) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int col = column_of<DP, WAVES>(i, ln);
            if (col >= d) continue;
            float4* dst = reinterpret_cast<float4*>(O + col);
            const float4 s = take_sum<DP, WAVES>(lds, i, ln);
            float4 x = o_old[i];
            if (f_old != 0.f) {
                x.x *= f_old; x.y *= f_old; x.z *= f_old; x.w *= f_old;
            } else {                    // an empty state: nothing of O is looked at
                x = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            x.x = fmaf(s.x, f_part, x.x); x.y = fmaf(s.y, f_part, x.y);
            x.z = fmaf(s.z, f_part, x.z); x.w = fmaf(s.w, f_part, x.w);
            *dst = x;
        }
        if (ln.wave == 0 && h == 0) *L = top + logf(w_sum);
    }
    return odd_rows;
}

// x + scale * (sum of the partial results at buf) to the lane's row
template <int DP, int WAVES, typename Lane>
__device__ inline void add_rows(float* row, float4 (&x)[share_of(DP, WAVES)], const char* buf, float scale, int d,
                                const Lane& ln) {
#pragma unroll
    for (int i = 0; i < share_of(DP, WAVES); ++i) {
        const int col = column_of<DP, WAVES>(i, ln);
        if (col >= d) continue;
        const float4 s = take_sum<DP, WAVES>(buf, i, ln);
        x[i].x = fmaf(scale, s.x, x[i].x); x[i].y = fmaf(scale, s.y, x[i].y);
        x[i].z = fmaf(scale, s.z, x[i].z); x[i].w = fmaf(scale, s.w, x[i].w);
        *reinterpret_cast<float4*>(row + col) = x[i];
    }
}

}  // namespace sa
