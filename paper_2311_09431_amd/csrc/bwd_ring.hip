// Backward ring step, 65 to 128 columns: kernels whose wavefronts are alone on their SIMD (dK and dV always, dQ where both kinds
// of workgroups share a launch).
//
// A wavefront issues an instruction of any kind every four to five clocks (vector 5, exponential 9, wait and s_nop 4, dependent
// scalar 8; LDS reads share the compute unit: a row read 4, a transposing one 2), a product of 32 x 32 x 16 takes the matrix core
// 33, and behind a product there is room for about six others.  With all vector work beside the products of the scores and none
// beside the others, as in bwd_mfma.hip, the first half of a sub-tile takes 760 clocks for 16 products and requests and walk 450
// a tile on top.  So here:
//  * behind every product an even share of everything else; half of a sub-tile's exponentials run beside the last products of the
//    one before it, where its scores are complete;
//  * Q and dO (K and V) tiles in a ring of four in LDS, one barrier a tile, in the middle of it: a tile is requested two
//    tiles ahead, piece by piece in gaps of the products, and the first operands behind the barrier are read before it;
//  * accumulators and the rows that stay (K and V, Q and dO) in accumulation registers by number, so that the vector ones hold
//    everything else without spills.
//
// What bounds them: issue and the matrix cores (16 or 8 + 16 products a sub-tile and its vector work beside them), at long blocks the
// clock that their power leaves.  Long dK/dV walks at d 128: 57 clocks a product, matrix cores 56 % busy at 1.9 GHz; of a wavefront's
// cycles 15 % in waits and 30 % waiting to issue; LDS busy 36 %.  Backward step, d 128, triangular unless said, with bwd_mfma.hip's
// kernels (keys up to 256 tiles in one launch) and with these and their launches, us, on one box.  One launch: 9 heads of 1100 44.6 /
// 38.4, 6 of 3000 92.9 / 78.8, 16 of 1536 54.6 / 51.2, 32 heads on 8 of 4096 489 / 458, 10 of 4096 202 / 161, 3 of 12500 573 / 388; two: 32 of
// 640 36.7 / 33.7, 32 of 4096 492 / 490, (full) 844 / 827, 128 of 1024 (full) 282 / 275, 32 of 32768 25720 / 24730.  Slower: a device's share
// of a ring of 128-row shards with few heads, all of whose tiles are masked: 31 heads, 7 shards, d 120, 35.2 / 38.0, 32 on 16, 14, d 96,
// 53.1 / 56.9.
//
// bwd_mfma.hip says what the products are; every sum has the order it has there, so the results have the same bits.
#include <hip/hip_bf16.h>

#include <type_traits>

#include "acc_file.h"
#include "mfma_tiles.h"
#include "sa_internal.h"

namespace sa {

namespace {

constexpr int BM = 128, SLOTS = 4, PRE = 2;
constexpr int ACC_DV = 0, ACC_DK = 64, ACC_DQ = 0, ACC_A = 128, ACC_B = 160;      // ACC_A: K rows or Q rows, ACC_B: V or dO
template <int DP> constexpr int SLOT = 2 * tile_bytes(DP);
constexpr int STAT_FLOATS = SLOTS * 2 * DT_ROWS + 4 * 2 * 2 * DT_ROWS;            // as loaded, per slot; as used, per wavefront and tile's parity

// score product: acc (+)= a x rows[16 columns]
__device__ __forceinline__ void score(f32x16& acc, bf16x8 a, int reg, bool first, bool after_valu) {
    if (first) {
        if (after_valu) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0" : "=&v"(acc) : "v"(a), "n"(reg), "n"(reg + 3) : ACC_FILE);
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0" : "=&v"(acc) : "v"(a), "n"(reg), "n"(reg + 3) : ACC_FILE);
    } else {
        if (after_valu) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0" : "+v"(acc) : "v"(a), "n"(reg), "n"(reg + 3) : ACC_FILE);
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0" : "+v"(acc) : "v"(a), "n"(reg), "n"(reg + 3) : ACC_FILE);
    }
}
// The rows that stay, as score operands: requested, and put into accumulation registers with the accumulators cleared meanwhile
struct Rows {
    bf16x8 a[8], b[8];
    __device__ __forceinline__ Rows(const __bf16* row_a, const __bf16* row_b, int h, int d) {
        load_b_frags<8>(a, row_a, h, d);
        load_b_frags<8>(b, row_b, h, d);
        asm volatile("" : : : "memory");
    }
    template <int N_ACC>
    __device__ __forceinline__ void keep() const {
        typedef int i32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int i = 0; i < N_ACC; ++i) acc_zero(i);
#pragma unroll
        for (int i = 0; i < 32; ++i) acc_write(ACC_A + i, __int_as_float(__builtin_bit_cast(i32x4, a[i / 4])[i % 4]));
#pragma unroll
        for (int i = 0; i < 32; ++i) acc_write(ACC_B + i, __int_as_float(__builtin_bit_cast(i32x4, b[i / 4])[i % 4]));
    }
};
// Blocks of accumulators into a row of dK, dV or dQ.  What is there is requested all at once, all workgroups of a launch are here
// at about the same time: two rows at a time by turns took 2 us more than that.  Where nothing is there (fresh) neither
// requests nor zeros stand in the way: with them launches of short walks lost 1.1 us (ring of one shard, 70 heads of 128 rows, d 128, 14.3 : 13.2, d 100 12.1 : 11.4).
template <int DP>
struct OutRow {
    float* row;
    float4 old[4 * blocks_of(DP)];
    // columns 8 i + 4 h .. + 3 lie in the row (more than 64 columns at DP = 112, more than 112 at 128)
    __device__ __forceinline__ static bool inside(int i, int h, int d) { return 8 * i + 8 <= (DP == 112 ? 64 : 112) || 8 * i + 4 * h < d; }
    __device__ __forceinline__ OutRow(float* r, int h, int d) : row(r + 4 * h) {
#pragma unroll
        for (int i = 0; i < 4 * blocks_of(DP); ++i)
            if (inside(i, h, d)) old[i] = *reinterpret_cast<const float4*>(row + 8 * i);
    }
    __device__ __forceinline__ static void put(float* row, int i, float4 x, float mul, int first, int h, int d) {
        x.x = fmaf(mul, acc_read(first + 4 * i), x.x); x.y = fmaf(mul, acc_read(first + 4 * i + 1), x.y);
        x.z = fmaf(mul, acc_read(first + 4 * i + 2), x.z); x.w = fmaf(mul, acc_read(first + 4 * i + 3), x.w);
        if (inside(i, h, d)) *reinterpret_cast<float4*>(row + 8 * i) = x;       // no padding columns
    }
    __device__ __forceinline__ void add(float mul, int first, int h, int d) const {
#pragma unroll
        for (int i = 0; i < 4 * blocks_of(DP); ++i) put(row, i, old[i], mul, first, h, d);
    }
    __device__ __forceinline__ static void set(float* r, float mul, int first, int h, int d) {
#pragma unroll
        for (int i = 0; i < 4 * blocks_of(DP); ++i) put(r + 4 * h, i, make_float4(0.f, 0.f, 0.f, 0.f), mul, first, h, d);
    }
};
// 16 values of an LDS array as a sub-tile's accumulator: register r holds row 8 (r/4) + r%4 (+ 4h: in the pointer)
__device__ inline void load_rows(f32x16& x, const float* rows) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 v = *reinterpret_cast<const float4*>(rows + 8 * g);
        x[4 * g + 0] = v.x; x[4 * g + 1] = v.y; x[4 * g + 2] = v.z; x[4 * g + 3] = v.w;
    }
}

// what a step has done for the one after it: first row fragments, half of the exponentials
struct Ahead {
    bf16x8 a[PRE], b[PRE];
    float e[8];
};

// The vector work of a step, on scores 2 j and 2 j + 1 at a time.
struct Scores {
    float e[16], ds[16];
    __device__ __forceinline__ static void arg(float* to, const f32x16& s, float kappa, float l0, float l1, int j) {
        to[0] = fmaf(s[2 * j], kappa, -l0);
        to[1] = fmaf(s[2 * j + 1], kappa, -l1);
    }
    __device__ __forceinline__ static void exps(float* x) {
        x[0] = __builtin_amdgcn_exp2f(x[0]);
        x[1] = __builtin_amdgcn_exp2f(x[1]);
    }
    __device__ __forceinline__ void pack(bf16x8 (&to)[2], const float (&x)[16], int j) const {
        to[j / 4][2 * j % 8] = (__bf16)x[2 * j];
        to[j / 4][2 * j % 8 + 1] = (__bf16)x[2 * j + 1];
    }
};
__device__ __forceinline__ float of4(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// ---------------------------------------------------------------- dK, dV
// One 32-query sub-tile: S and dP of the next one, P, dS, dV^T += dO^T P, dK^T += Q^T dS of this one.  lse_*: LSE log2(e) of the
// lane's rows; dp_next comes in as -delta.
template <bool NEXT, bool MASK, int DP, bool PART, typename Hook>
__device__ __forceinline__ void keys_step(const f32x16& s_cur, const f32x16& dp_cur, f32x16& s_next, f32x16& dp_next, float kappa,
                                 const uint32_t (&arow)[8], const uint32_t (&tr0)[4], const uint32_t (&tr1)[4], Ahead& pre, const char* next,
                                 const char* cur, const float* lse_cur, const float* lse_next, int mask_lim, int part_ks, Hook hook) {
    constexpr int KS = ksteps_of(DP), MB = blocks_of(DP), TAHEAD = 3;
    bf16x8 qa[8], ga[8], qt[8], gt[8], pb[2], dsb[2];
    float4 lv[2], ln[2];
    Scores w;
#pragma unroll
    for (int i = 0; i < PRE; ++i) {
        qa[i] = pre.a[i];
        ga[i] = pre.b[i];
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) w.e[r] = pre.e[r];
    // (what a product reads first is requested last: LDS answers in order, and one wait does for both)
    auto fetch = [&](int i) {
        if (NEXT && i < KS) {
            ga[i] = dt_read_row(next + tile_bytes(DP), arow[i]);
            qa[i] = dt_read_row(next, arow[i]);
        }
    };
    auto fetch_t = [&](int i) {
        if (i < 8 && i % 4 < MB) {
            const char* rows = cur + (i / 4) * 16 * row_bytes(DP);
            qt[i] = dt_read_tr(rows, tr0[i % 4], tr1[i % 4]);
            gt[i] = dt_read_tr(rows + tile_bytes(DP), tr0[i % 4], tr1[i % 4]);
        }
    };
    auto arg = [&](int j) { w.arg(w.e + 2 * j, s_cur, kappa, of4(lv[j / 2 - 2], 2 * j % 4), of4(lv[j / 2 - 2], 2 * j % 4 + 1), j); };
    auto times = [&](int j) {
#pragma unroll
        for (int r = 2 * j; r < 2 * j + 2; ++r) {
            if (MASK && 8 * (r / 4) + (r % 4) < mask_lim) w.e[r] = 0.f;
            w.ds[r] = w.e[r] * dp_cur[r];
        }
    };
    auto pack = [&](int j) {
        w.pack(pb, w.e, j);
        w.pack(dsb, w.ds, j);
    };
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        const int i = k / 2, j = k / 4;
        const bool select = PART && i >= part_from(DP);
        if (NEXT && i < KS) {
            if (k % 2 == 0) score(s_next, select ? zero_beyond_d(qa[i], i == part_ks) : qa[i], ACC_A + 4 * i, i == 0, select);
            else score(dp_next, select ? zero_beyond_d(ga[i], i == part_ks) : ga[i], ACC_B + 4 * i, false, select || i == 0);     // (-delta may have been moved here)
        }
        __builtin_amdgcn_sched_barrier(0);
        if (k % 2 == 0) {
            if (i + PRE < 8) fetch(i + PRE);
        } else {
            if (k == 1) {
                lv[0] = *reinterpret_cast<const float4*>(lse_cur + 16);
                lv[1] = *reinterpret_cast<const float4*>(lse_cur + 24);
            }
            if (i >= 8 - TAHEAD) fetch_t(i - (8 - TAHEAD));
        }
        if (k % 4 == 0) times(j);
        if (k % 4 == 1 && j > 0) arg(j + 3);
        if (k % 4 == 2) pack(j);
        if (k % 4 == 3 && j > 0) w.exps(w.e + 2 * (j + 3));
        hook(k);
    }
#pragma unroll
    for (int k = 16; k < 32; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        const int i = (k - 16) / 2;
        if (i % 4 < MB) {
            if (k % 2 == 0) acc_mfma_far(ACC_DV / 16 + i % 4, gt[i], pb[i / 4]);
            else acc_mfma_far(ACC_DK / 16 + i % 4, qt[i], dsb[i / 4]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (k % 2 == 0) fetch_t(i + TAHEAD);
        if (k == 16) arg(7);
        if (k == 17) w.exps(w.e + 14);
        if (k < 23 && k % 2 == 0) times(4 + i);
        if (k < 22 ? k % 2 == 1 : k == 22) pack(4 + i);
        hook(k);
        if (NEXT && k == 22) {
            ln[0] = *reinterpret_cast<const float4*>(lse_next);
            ln[1] = *reinterpret_cast<const float4*>(lse_next + 8);
        }
        if (NEXT && k >= 24) {
            const int j = i - 4;
            if (k % 2 == 0) w.arg(pre.e + 2 * j, s_next, kappa, of4(ln[j / 2], 2 * j % 4), of4(ln[j / 2], 2 * j % 4 + 1), j);
            else w.exps(pre.e + 2 * j);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

// RAGGED without instantiations of its own: rows beyond the shard come in as zeros (clamped for the rows that stay), their LSE as
// +inf, and they are not stored.  Pairs of (query head of the group, query shard) are blocks of one walk, as in bwd_mfma.hip.
template <int DP, bool PART, bool BY_RANK>
__device__ __forceinline__ void dkdv_ring(const StepArgs& p, int n_tiles, int linear, char* lds, float* stat) {
    constexpr int KS = ksteps_of(DP), MB = blocks_of(DP), PIECES = load_pieces(DP), HALF = tile_bytes(DP) / 2;
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int ktile, bh, dev_rank;
    decode_block<false, BY_RANK>(linear, n_tiles * p.n_kv, p.B * p.H_kv, ktile, bh);
    decode_rank(ktile, n_tiles, p.n_kv, p.layout, ktile, dev_rank);
    const int dev = p.kv_dev + dev_rank;
    const int b = bh / p.H_kv, kvh = bh - b * p.H_kv;
    const int64_t kv_base = b * p.kv_stride_b + kvh * p.kv_stride_h + (dev - p.kv_dev) * p.kv_shard;
    const int d = p.d;
    const int64_t ss = p.kv_stride_s;
    const int pitch = 2 * (int)p.stride_s;
    const int k0 = ktile * BM, key_own = k0 + 32 * wave + n, key = min(key_own, p.c - 1);

    const Rows rows_kv((const __bf16*)p.k + kv_base + (int64_t)key * ss, (const __bf16*)p.v + kv_base + (int64_t)key * ss, h, d);
    const int group = p.H / p.H_kv, dev_end = p.q_dev + p.n_q, n_qt = (p.c + DT_ROWS - 1) / DT_ROWS;
    // contiguous layout: earlier devices' queries see nothing of these keys
    const int dev0 = p.layout != SA_STRIPED ? max(p.q_dev, dev) : p.q_dev;
    auto first_tile = [&](int q_dev) {
        if (block_kind(q_dev, dev, p.layout) != MASK_TRI) return 0;
        if (p.skip_bq > 0)      // emulated coarse skipping, as in bwd_mfma.hip
            return ((k0 / p.skip_bk * p.skip_bk + block_off(q_dev, dev, p.layout)) / p.skip_bq) * p.skip_bq / DT_ROWS;
        return k0 / DT_ROWS;
    };
    struct { int q_head, q_dev, t; } at{0, dev0, 0}, req{0, dev0, 0};       // of the products, of the requests
    int plain, lim;     // first tile of the block without a masked pair; the lane's mask limit for query row 0
    auto enter_at = [&]() {
        const bool tri = block_kind(at.q_dev, dev, p.layout) == MASK_TRI;
        const int off = block_off(at.q_dev, dev, p.layout);
        at.t = first_tile(at.q_dev);
        plain = tri ? (k0 + BM + off + DT_ROWS - 2) / DT_ROWS : 0;
        lim = tri ? key_own + off - 4 * h : -(1 << 30);
    };
    enter_at();
    dt_rsrc Qr, Gr, Sr;
    TileByte byte{0, DT_ROWS * pitch};      // of the tile to request, in Q and dO
    auto enter_req = [&]() {
        const int hd = kvh * group + req.q_head;
        req.t = first_tile(req.q_dev);
        byte.block(req.t);
        const int64_t base = b * p.stride_b + hd * p.stride_h + (req.q_dev - p.q_dev) * p.q_shard;
        const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(req.q_dev - p.q_dev) * p.c;
        Qr = dt_make_rsrc((const __bf16*)p.q + base, p.c, pitch, d);
        Gr = dt_make_rsrc((const __bf16*)p.dout + base, p.c, pitch, d);
        Sr = dt_make_rsrc((wave & 1 ? p.delta : p.lse) + sbase, p.c, 4, 2);
    };
    enter_req();
    int left = 0;                           // tiles of the walk that are not done
    for (int q = dev0; q < dev_end; ++q) left += n_qt - first_tile(q);
    left *= group;
    // the next tile; false: the first of another block
    auto next_of = [&](auto& w) -> bool {
        if (++w.t < n_qt) return true;
        if (++w.q_dev == dev_end) {
            w.q_dev = dev0;
            ++w.q_head;
        }
        return false;
    };
    uint32_t gl[4];
    dt_load_offsets<DP>(gl, lane, wave, pitch, d);
    // A wavefront's share of a tile: 32 of its 128 statistics, eight pieces of 1 KiB.
    int slot_byte = 0;                      // where the tile to request goes
    char* const stat_own = reinterpret_cast<char*>(stat) + (wave & 1) * 256 + (wave >> 1) * 128;
    auto request_stat = [&]() {
        if (lane < 32) dt_load_dword(Sr, 4 * DT_ROWS * req.t + 128 * (wave >> 1), 4 * lane, stat_own + slot_byte / (SLOT<DP> / 512));
    };
    auto request_piece = [&](int j) {
        char* const dst = lds + slot_byte + PIECES * wave * 1024;
        if (j < PIECES) dt_load_piece(Qr, byte.at, gl[j], dst + j * 1024);
        else dt_load_piece(Gr, byte.at, gl[j - PIECES], dst + tile_bytes(DP) + (j - PIECES) * 1024);
    };
    auto requested = [&]() {
        slot_byte = (slot_byte + SLOT<DP>) & (SLOTS * SLOT<DP> - 1);
        byte.next();
        if (!next_of(req)) {
            if (req.q_head < group) {
                enter_req();
            } else {            // behind the walk's end: nothing is fetched, zeros go where nobody reads
                Qr[2] = Gr[2] = Sr[2] = 0;
                byte.stop();
            }
        }
    };
    auto request = [&]() {
#pragma unroll
        for (int j = 0; j < 2 * PIECES; ++j) request_piece(j);
        request_stat();
        requested();
    };
    request();
    request();
    rows_kv.keep<128>();
    const float kappa = p.scale * LOG2E;
    uint32_t arow[8], tr0[4], tr1[4];
    dt_row_addrs<DP>(arow, n, h);
    dt_tr_addrs<DP>(tr0, tr1, lane);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // LSE log2(e) and -delta of a tile, each wavefront for itself; queries beyond the shard: +inf
    float* const own = stat + SLOTS * 2 * DT_ROWS + wave * 4 * DT_ROWS;
    auto put_stat = [&](float* to, float lse, float delta, int rows) {
        to[lane] = lane < rows ? lse * LOG2E : INFINITY;
        to[DT_ROWS + lane] = -delta;
    };

    // PART: k-step whose fragment, in this half-wave, is the chunk holding column d
    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    f32x16 s_a, s_b, dp_a, dp_b;
    Ahead pre;
    load_rows(dp_a, stat + DT_ROWS + 4 * h);
#pragma unroll
    for (int r = 0; r < 16; ++r) dp_a[r] = -dp_a[r];
    put_stat(own, stat[lane], stat[DT_ROWS + lane], p.c - DT_ROWS * at.t);
    // (the third tile only now: one less that all workgroups of a launch wait for at the same time)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        if (ks < 2 * PIECES) request_piece(ks);
        bf16x8 qx = dt_read_row(lds, arow[ks]), gx = dt_read_row(lds + tile_bytes(DP), arow[ks]);
        if (PART) {
            qx = zero_beyond_d(qx, ks == part_ks);
            gx = zero_beyond_d(gx, ks == part_ks);
        }
        score(s_a, qx, ACC_A + 4 * ks, ks == 0, PART);
        score(dp_a, gx, ACC_B + 4 * ks, false, PART || ks == 0);
    }
#pragma unroll
    for (int j = KS; j < 2 * PIECES; ++j) request_piece(j);
    request_stat();
    requested();
    mfma_results_to_valu(s_a, dp_a);
    auto ahead_rows = [&](int i, const char* rows) {
        pre.b[i] = dt_read_row(rows + tile_bytes(DP), arow[i]);
        pre.a[i] = dt_read_row(rows, arow[i]);
    };
#pragma unroll
    for (int i = 0; i < PRE; ++i) ahead_rows(i, lds + HALF);
    load_rows(dp_b, own + DT_ROWS + 32 + 4 * h);
#pragma unroll
    for (int r = 0; r < 8; ++r) pre.e[r] = __builtin_amdgcn_exp2f(fmaf(s_a[r], kappa, -own[8 * (r / 4) + 4 * h + r % 4]));

    int slot = 0;                           // of the present tile, in bytes
    float* cur = own;                       // its statistics
    // Tile t: sub-tile 0 with the scores of sub-tile 1 beside it, then sub-tile 1 with those of the next tile's first.  In the
    // middle of the former, tile t + 1, requested two tiles ago, has landed for everyone, and everyone is done with t - 1, into whose
    // slot t + 3 is requested from then on.
    auto tile = [&](auto mask_c) {
        constexpr bool MASK = decltype(mask_c)::value;
        const int next = (slot + SLOT<DP>) & (SLOTS * SLOT<DP> - 1), by = next - slot;
        float* const after = own + 2 * DT_ROWS - (cur - own);
        const float* const lse = cur + 4 * h;
        const int lim_at = lim - DT_ROWS * at.t;
        if (!next_of(at)) enter_at();       // (there is one: this is not the last tile)
        const int rows = p.c - DT_ROWS * at.t;
        const float* const landed = stat + next / (SLOT<DP> / (2 * DT_ROWS));
        float raw_lse, raw_delta;
        keys_step<true, MASK, DP, PART>(s_a, dp_a, s_b, dp_b, kappa, arow, tr0, tr1, pre, lds + HALF, lds, lse, lse + 32, lim_at, part_ks, [&](int k) {
            if (k == 16) {
                wait_all_but<2 * PIECES + 1>();
                meet();
            }
            if (k == 17) {
                raw_lse = landed[lane];
                raw_delta = landed[DT_ROWS + lane];
            }
            if (k == 24) put_stat(after, raw_lse, raw_delta, rows);
            if (k >= 18 && k % 2 == 0 && k < 18 + 2 * PIECES) request_piece((k - 18) / 2);
            if (k >= 24 && k < 28) {
                arow[2 * (k - 24)] += by;
                arow[2 * (k - 24) + 1] += by;
            }
            if (k >= 28 && k < 28 + PRE) ahead_rows(k - 28, lds);
            if (k == 30) load_rows(dp_a, after + DT_ROWS + 4 * h);
        });
        keys_step<true, MASK, DP, PART>(s_b, dp_b, s_a, dp_a, kappa, arow, tr0, tr1, pre, lds, lds + HALF, lse + 32, after + 4 * h, lim_at - 32, part_ks, [&](int k) {
            if (k >= 17 && k % 2 == 1 && k < 17 + 2 * PIECES) request_piece(PIECES + (k - 17) / 2);
            if (k == 25) request_stat();
            if (k >= 26 && k < 28) {
#pragma unroll
                for (int i = 2 * (k - 26); i < 2 * (k - 25); ++i) {
                    tr0[i] += by;
                    tr1[i] += by;
                }
            }
            if (k >= 28 && k < 28 + PRE) ahead_rows(k - 28, lds + HALF);
            if (k == 30) load_rows(dp_b, after + DT_ROWS + 32 + 4 * h);
            if (k == 31) requested();
        });
        slot = next;
        cur = after;
        --left;
    };
    for (;;) {          // all but the last tile, whose second sub-tile has no scores beside it
        while (at.t >= plain && left > 1) tile(std::false_type{});
        if (left == 1) break;
        tile(std::true_type{});
    }
    {
        const float* const lse = cur + 4 * h;
        const int lim_at = lim - DT_ROWS * at.t;
        const auto none = [](int) {};
        keys_step<true, true, DP, PART>(s_a, dp_a, s_b, dp_b, kappa, arow, tr0, tr1, pre, lds + HALF, lds, lse, lse + 32, lim_at, part_ks, none);
        keys_step<false, true, DP, PART>(s_b, dp_b, s_a, dp_a, kappa, arow, tr0, tr1, pre, lds, lds + HALF, lse + 32, lse, lim_at - 32, part_ks, none);
    }
    wait_all_but<0>();  // (the last requests are on their way into this workgroup's slots)
    acc_settle();
    if (key_own >= p.c) return;
    float* const v_at = p.dv + kv_base + (int64_t)key * ss;
    float* const k_at = p.dk + kv_base + (int64_t)key * ss;
    if (p.fresh) {
        OutRow<DP>::set(v_at, 1.f, ACC_DV, h, d);
        OutRow<DP>::set(k_at, p.scale, ACC_DK, h, d);
    } else {
        const OutRow<DP> v_row(v_at, h, d), k_row(k_at, h, d);
        v_row.add(1.f, ACC_DV, h, d);
        k_row.add(p.scale, ACC_DK, h, d);
    }
}

// -------------------------------------------------------------------- dQ
// One 32-key sub-tile: S^T and dP^T of the next one, P, dS, dQ^T += K^T dS^T of this one.
template <bool NEXT, bool MASK, int DP, bool PART, typename Hook>
__device__ __forceinline__ void queries_step(const f32x16& s_cur, const f32x16& dp_cur, f32x16& s_next, f32x16& dp_next, float kappa, float lse2,
                                    float delta, const uint32_t (&arow)[8], const uint32_t (&tr0)[4], const uint32_t (&tr1)[4], Ahead& pre,
                                    const char* next, const char* cur, int mask_lim, int part_ks, Hook hook) {
    constexpr int KS = ksteps_of(DP), MB = blocks_of(DP), TAHEAD = 3;
    bf16x8 ka[8], va[8], kt[8], dsb[2];
    Scores w;
#pragma unroll
    for (int i = 0; i < PRE; ++i) {
        ka[i] = pre.a[i];
        va[i] = pre.b[i];
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) w.e[r] = pre.e[r];
    auto fetch = [&](int i) {
        if (NEXT && i < KS) {
            va[i] = dt_read_row(next + tile_bytes(DP), arow[i]);
            ka[i] = dt_read_row(next, arow[i]);
        }
    };
    auto fetch_t = [&](int i) {
        if (i < 8 && i % 4 < MB) kt[i] = dt_read_tr(cur + (i / 4) * 16 * row_bytes(DP), tr0[i % 4], tr1[i % 4]);
    };
    auto times = [&](int j) {
#pragma unroll
        for (int r = 2 * j; r < 2 * j + 2; ++r) {
            if (MASK && 8 * (r / 4) + (r % 4) > mask_lim) w.e[r] = 0.f;
            w.ds[r] = w.e[r] * (dp_cur[r] - delta);
        }
    };
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        const int i = k / 2, j = k / 4;
        const bool select = PART && i >= part_from(DP);
        if (NEXT && i < KS) {
            if (k % 2 == 0) score(s_next, select ? zero_beyond_d(ka[i], i == part_ks) : ka[i], ACC_A + 4 * i, i == 0, select);
            else score(dp_next, select ? zero_beyond_d(va[i], i == part_ks) : va[i], ACC_B + 4 * i, i == 0, select);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (k % 2 == 0) {
            if (i + PRE < 8) fetch(i + PRE);
        } else if (i >= 8 - TAHEAD) {
            fetch_t(i - (8 - TAHEAD));
        }
        if (k % 4 == 0) times(j);
        if (k % 4 == 1) w.arg(w.e + 2 * (j + 4), s_cur, kappa, lse2, lse2, j + 4);
        if (k % 4 == 2) w.pack(dsb, w.ds, j);
        if (k % 4 == 3) w.exps(w.e + 2 * (j + 4));
        hook(k);
    }
#pragma unroll
    for (int k = 16; k < 24; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        const int i = k - 16;
        if (i % 4 == 0) acc_mfma(ACC_DQ / 16, kt[i], dsb[i / 4]);       // (packed just before)
        else if (i % 4 < MB) acc_mfma_far(ACC_DQ / 16 + i % 4, kt[i], dsb[i / 4]);
        __builtin_amdgcn_sched_barrier(0);
        if (k < 20) {
            times(k - 12);
            w.pack(dsb, w.ds, k - 12);
        }
        fetch_t(i + TAHEAD);
        hook(k);
        if (NEXT && k >= 20) {
            const int j = (k - 20) / 2 * 2;
#pragma unroll
            for (int x = j; x < j + 2; ++x) {
                if (k % 2 == 0) w.arg(pre.e + 2 * x, s_next, kappa, lse2, lse2, x);
                else w.exps(pre.e + 2 * x);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <int DP, bool PART>
__device__ __forceinline__ void dq_ring(const StepArgs& p, int n_tiles, int linear, char* lds) {
    constexpr int KS = ksteps_of(DP), MB = blocks_of(DP), PIECES = load_pieces(DP), HALF = tile_bytes(DP) / 2;
    const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int rank, bh, dev_rank;
    decode_block<true, false>(linear, n_tiles * p.n_q, p.B * p.H, rank, bh);
    decode_rank(rank, n_tiles, p.n_q, p.layout, rank, dev_rank);
    const int dev = p.q_dev + p.n_q - 1 - dev_rank, qt = n_tiles - 1 - rank;      // heaviest first
    const int b = bh / p.H, hd = bh - b * p.H;
    const int64_t base = b * p.stride_b + hd * p.stride_h + (dev - p.q_dev) * p.q_shard;
    const int64_t kv_base = b * p.kv_stride_b + (hd / (p.H / p.H_kv)) * p.kv_stride_h;
    const int64_t sbase = b * p.stat_stride_b + hd * p.stat_stride_h + (int64_t)(dev - p.q_dev) * p.c;
    const int d = p.d;
    const int64_t ss = p.stride_s;
    const int pitch = 2 * (int)p.kv_stride_s;
    const int q0 = qt * BM, a_own = q0 + 32 * wave + n, a = min(a_own, p.c - 1);

    const Rows rows_qg((const __bf16*)p.q + base + (int64_t)a * ss, (const __bf16*)p.dout + base + (int64_t)a * ss, h, d);
    float lse2 = p.lse[sbase + a] * LOG2E, delta = p.delta[sbase + a];
    // contiguous layout: the blocks of devices further on are entirely masked
    const int kv_end = p.layout == SA_STRIPED ? p.kv_dev + p.n_kv : min(p.kv_dev + p.n_kv, dev + 1);
    auto tiles_of = [&](int kv) {
        if (block_kind(dev, kv, p.layout) == MASK_FULL) return (p.c + DT_ROWS - 1) / DT_ROWS;
        if (p.skip_bq > 0) {
            const int q_hi = (q0 / p.skip_bq + 1) * p.skip_bq - 1;
            return min(p.c, ((q_hi - block_off(dev, kv, p.layout)) / p.skip_bk + 1) * p.skip_bk) / DT_ROWS;
        }
        return (q0 + BM) / DT_ROWS;
    };
    struct { int kv, t, n; } at{p.kv_dev, 0, 0}, req{p.kv_dev, 0, 0};
    int plain, lim;     // tiles of the block before the first with a masked pair; the lane's mask limit for key row 0
    auto enter_at = [&]() {
        const bool full = block_kind(dev, at.kv, p.layout) == MASK_FULL;
        const int off = block_off(dev, at.kv, p.layout);
        at.t = 0;
        at.n = tiles_of(at.kv);
        plain = (full ? p.c : max(0, q0 - off + 1)) / DT_ROWS;
        lim = (full ? p.c - 1 : a_own - off) - 4 * h;
    };
    enter_at();
    dt_rsrc Kr, Vr;
    TileByte byte{0, DT_ROWS * pitch};
    auto enter_req = [&]() {
        req.t = 0;
        req.n = tiles_of(req.kv);
        byte.block(0);
        const int64_t from = kv_base + (req.kv - p.kv_dev) * p.kv_shard;
        Kr = dt_make_rsrc((const __bf16*)p.k + from, p.c, pitch, d);
        Vr = dt_make_rsrc((const __bf16*)p.v + from, p.c, pitch, d);
    };
    enter_req();
    int left = 0;
    for (int kv = p.kv_dev; kv < kv_end; ++kv) left += tiles_of(kv);
    auto next_of = [&](auto& w) -> bool {
        if (++w.t < w.n) return true;
        ++w.kv;
        return false;
    };
    uint32_t gl[4];
    dt_load_offsets<DP>(gl, lane, wave, pitch, d);
    int slot_byte = 0;
    auto request_piece = [&](int j) {
        char* const dst = lds + slot_byte + PIECES * wave * 1024;
        if (j < PIECES) dt_load_piece(Kr, byte.at, gl[j], dst + j * 1024);
        else dt_load_piece(Vr, byte.at, gl[j - PIECES], dst + tile_bytes(DP) + (j - PIECES) * 1024);
    };
    auto requested = [&]() {
        slot_byte = (slot_byte + SLOT<DP>) & (SLOTS * SLOT<DP> - 1);
        byte.next();
        if (!next_of(req)) {
            if (req.kv < kv_end) {
                enter_req();
            } else {
                Kr[2] = Vr[2] = 0;
                byte.stop();
            }
        }
    };
    auto request = [&]() {
#pragma unroll
        for (int j = 0; j < 2 * PIECES; ++j) request_piece(j);
        requested();
    };
    request();
    request();
    rows_qg.keep<64>();
    const float kappa = p.scale * LOG2E;
    // (complete here: a load left pending would be waited for with the tile requested next)
    asm volatile("" : "+v"(lse2), "+v"(delta));
    uint32_t arow[8], tr0[4], tr1[4];
    dt_row_addrs<DP>(arow, n, h);
    dt_tr_addrs<DP>(tr0, tr1, lane);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    const int part_ks = (PART && ((d >> 3) & 1) == h) ? (d >> 4) : -1;
    f32x16 s_a, s_b, dp_a, dp_b;
    Ahead pre;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        if (ks < 2 * PIECES) request_piece(ks);
        bf16x8 kx = dt_read_row(lds, arow[ks]), vx = dt_read_row(lds + tile_bytes(DP), arow[ks]);
        if (PART) {
            kx = zero_beyond_d(kx, ks == part_ks);
            vx = zero_beyond_d(vx, ks == part_ks);
        }
        score(s_a, kx, ACC_A + 4 * ks, ks == 0, PART);
        score(dp_a, vx, ACC_B + 4 * ks, ks == 0, PART);
    }
#pragma unroll
    for (int j = KS; j < 2 * PIECES; ++j) request_piece(j);
    requested();
    mfma_results_to_valu(s_a, dp_a);
    auto ahead_rows = [&](int i, const char* rows) {
        pre.b[i] = dt_read_row(rows + tile_bytes(DP), arow[i]);
        pre.a[i] = dt_read_row(rows, arow[i]);
    };
#pragma unroll
    for (int i = 0; i < PRE; ++i) ahead_rows(i, lds + HALF);
#pragma unroll
    for (int r = 0; r < 8; ++r) pre.e[r] = __builtin_amdgcn_exp2f(fmaf(s_a[r], kappa, -lse2));

    int slot = 0;
    auto tile = [&](auto mask_c) {          // as in dkdv_ring
        constexpr bool MASK = decltype(mask_c)::value;
        const int next = (slot + SLOT<DP>) & (SLOTS * SLOT<DP> - 1), by = next - slot, lim_at = lim - DT_ROWS * at.t;
        if (!next_of(at)) enter_at();
        queries_step<true, MASK, DP, PART>(s_a, dp_a, s_b, dp_b, kappa, lse2, delta, arow, tr0, tr1, pre, lds + HALF, lds, lim_at, part_ks, [&](int k) {
            if (k == 16) {
                wait_all_but<2 * PIECES>();
                meet();
            }
            if (k >= 17 && k < 21) {
                arow[2 * (k - 17)] += by;
                arow[2 * (k - 17) + 1] += by;
            }
            if (k >= 17 && k % 2 == 1 && k < 17 + 2 * PIECES) request_piece((k - 17) / 2);
            if (k >= 22 && k < 22 + PRE) ahead_rows(k - 22, lds);
        });
        queries_step<true, MASK, DP, PART>(s_b, dp_b, s_a, dp_a, kappa, lse2, delta, arow, tr0, tr1, pre, lds, lds + HALF, lim_at - 32, part_ks, [&](int k) {
            if (k >= 9 && k % 2 == 1 && k < 9 + 2 * PIECES) request_piece(PIECES + (k - 9) / 2);
            if (k >= 21 && k < 23) {
#pragma unroll
                for (int i = 2 * (k - 21); i < 2 * (k - 20); ++i) {
                    tr0[i] += by;
                    tr1[i] += by;
                }
            }
            if (k >= 22 && k < 22 + PRE) ahead_rows(k - 22, lds + HALF);
            if (k == 18) requested();
        });
        slot = next;
        --left;
    };
    for (;;) {
        while (at.t < plain && left > 1) tile(std::false_type{});
        if (left == 1) break;
        tile(std::true_type{});
    }
    const int lim_at = lim - DT_ROWS * at.t;
    const auto none = [](int) {};
    queries_step<true, true, DP, PART>(s_a, dp_a, s_b, dp_b, kappa, lse2, delta, arow, tr0, tr1, pre, lds + HALF, lds, lim_at, part_ks, none);
    queries_step<false, true, DP, PART>(s_b, dp_b, s_a, dp_a, kappa, lse2, delta, arow, tr0, tr1, pre, lds, lds + HALF, lim_at - 32, part_ks, none);
    wait_all_but<0>();
    acc_settle();
    if (a_own >= p.c) return;
    float* const q_at = p.dq + base + (int64_t)a * ss;
    if (p.fresh) OutRow<DP>::set(q_at, p.scale, ACC_DQ, h, d);
    else OutRow<DP>(q_at, h, d).add(p.scale, ACC_DQ, h, d);
}

template <int DP, bool PART, bool BY_RANK>
__global__ void __launch_bounds__(256, 1)
bwd_dkdv_ring_kernel(StepArgs p, int n_tiles) {
    __shared__ __attribute__((aligned(1024))) char lds[SLOTS * SLOT<DP>];
    __shared__ __attribute__((aligned(16))) float stat[STAT_FLOATS];
    dkdv_ring<DP, PART, BY_RANK>(p, n_tiles, (int)blockIdx.x, lds, stat);
}
template <int DP, bool PART>
__global__ void __launch_bounds__(256, 1)
bwd_both_ring_kernel(StepArgs p, int n_tiles, PlacedKinds kinds) {
    __shared__ __attribute__((aligned(1024))) char lds[SLOTS * SLOT<DP>];
    __shared__ __attribute__((aligned(16))) float stat[STAT_FLOATS];
    int linear = (int)blockIdx.x;
    const int keys = __builtin_amdgcn_readfirstlane(owns_keys(kinds, linear));
    linear = __builtin_amdgcn_readfirstlane(linear);        // (both kept scalar)
    if (keys) dkdv_ring<DP, PART, false>(p, n_tiles, linear, lds, stat);
    else dq_ring<DP, PART>(p, n_tiles, linear, lds);
}

template <int DP, bool PART>
hipError_t launch(const StepArgs& a, const PlacedKinds* kinds, int workgroups, hipStream_t st) {
    const dim3 grid((unsigned)workgroups), block(256);
    const int n_tiles = (a.c + BM - 1) / BM;
    if (kinds) hipLaunchKernelGGL((bwd_both_ring_kernel<DP, PART>), grid, block, 0, st, a, n_tiles, *kinds);
    else if (dkdv_by_rank(a)) hipLaunchKernelGGL((bwd_dkdv_ring_kernel<DP, PART, true>), grid, block, 0, st, a, n_tiles);
    else hipLaunchKernelGGL((bwd_dkdv_ring_kernel<DP, PART, false>), grid, block, 0, st, a, n_tiles);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_bwd_ring(const StepArgs& a, const PlacedKinds* kinds, int workgroups, hipStream_t st) {
    const bool part = a.d % 8 != 0;
    if (a.d <= 112) return part ? launch<112, true>(a, kinds, workgroups, st) : launch<112, false>(a, kinds, workgroups, st);
    return part ? launch<128, true>(a, kinds, workgroups, st) : launch<128, false>(a, kinds, workgroups, st);
}

}  // namespace sa
