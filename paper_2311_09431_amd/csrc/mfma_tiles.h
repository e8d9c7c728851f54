// Tile staging shared by the matrix-core kernels: 64-row x 128-column bf16 tiles
// go from global memory straight into swizzled LDS tiles and are read from there
// in the layouts the v_mfma_f32_32x32x16_bf16 operands want.
//
// Register layouts of that instruction (lane = 32*h + n):
//   A operand: row n of the 32 x 16 left matrix, 8 consecutive k starting at 8h
//   B operand: column n of the 16 x 32 right matrix, the same 8 k
//   C/D:       column n, rows 8*(r/4) + 4h + r%4 for register r = 0..15
// A C/D tile whose rows are the contraction index of the next product can be
// fed to it as a B operand straight from registers: registers 8g'..8g'+7 of a
// 32-row block are rows {0..3, 8..11} + 4h of a group of 16; the transposing LDS
// reads below deliver the other operand in the same order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int TD = 128;          // tile columns: head dimensions up to 128 are zero-padded to it;
                                 // larger ones (up to 256) are held as two such tiles, columns
                                 // 0..127 and 128..255 of the same rows ("halves")
constexpr int TR = 64;           // tile rows streamed per iteration

// DP, the number of columns a kernel instantiation computes: 32 (whole 16-byte chunks only), 64, 112, 128 or 256.  Tiles
// are 128 columns wide (two of them, "halves", for 256), 64 for DP = 32 and 64; otherwise a smaller DP only leaves
// out work: a contraction over the head dimension takes ksteps_of(DP) steps of 16 columns per half, a
// product whose output has head-dimension columns blocks_of(DP) blocks of 32 per half.
// 112 (head dimensions 65..112, e.g. the 100 of the paper's 3B model, Table 1) drops the last
// k-step and keeps all four output blocks.
constexpr int halves_of(int DP) { return DP > 128 ? 2 : 1; }
constexpr int ksteps_of(int DP) { return (DP / halves_of(DP) + 15) / 16; }
constexpr int blocks_of(int DP) { return (DP / halves_of(DP) + 31) / 32; }
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// ---------------------------------------------------------------------------
// Swizzled tiles filled by direct global -> LDS loads.
//
// A tile is 64 rows x 256 bytes (128 bf16; up to 64 columns see below) with NO padding: a direct load
// writes the 64 lanes' 16-byte pieces contiguously (1 KiB per wavefront
// instruction, 4 rows), so a 16 KiB tile takes 16 instructions, 4 per
// wavefront.  Bank conflicts are avoided by storing the 16-byte chunk c of row
// r at chunk position c ^ f(r), f(r) = ((r & 3) << 2) | ((r >> 2) & 3):
//  * 16-byte A-operand row reads (16 consecutive rows, same logical chunk) hit
//    16 different chunks, because f is a bijection of r & 15;
//  * the transposing 8-byte reads (ds_read_b64_tr_b16: 4 consecutive rows x two
//    neighbouring 32-byte chunk pairs per half-wave) hit 8 different pairs.
// The swizzle is applied on the global side: the lane that fills chunk position
// pc of row r fetches logical chunk pc ^ f(r).
//
// Transposing read.  Within each block of 16 lanes the instruction hands lane i
// the i-th 16-bit element of what lanes 4e + i/4 (e = 0..3) point at, so lane j
// of a block points at row j/4, columns 4 (j%4) .. +3 of a 4 x 16 patch and every
// lane receives 4 consecutive rows of one column.  Two reads (rows +0 and +8)
// give the 8 contraction values {0..3, 8..11} + 4h of a group of 16 rows that
// match a C/D tile used as B operand.
constexpr int DT_ROWS = 64;
constexpr int DT_BYTES = DT_ROWS * 256;          // 16 KiB
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char_t;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4_t;

__device__ inline int dt_swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// Up to 64 columns two rows share a 256-byte line (8 KiB a tile, half the loads): row r, chunk c at
// line r / 2, chunk position (c + 8 (r & 1)) ^ g(r / 2), g(s) = ((s & 1) << 2) | ((s >> 1) & 3).
//  * row reads: 16 consecutive rows, one logical chunk: lines 0..7 with both parities; g is a
//    bijection of s & 7 and leaves bit 3 alone, so 16 different positions;
//  * transposing reads: 4 consecutive rows = 2 neighbouring lines with both parities, whose g differ
//    in bit 2: 8 different 32-byte pairs.
// Offsets of 16 rows leave g alone, as they leave f.  Against 64-column rows in 256-byte lines whose
// other half was written as zeros (16 heads, d 64, 12500 tokens, triangular): forward step
// 0.463 -> 0.423 ms, backward 1.37 -> 1.26; full blocks 0.83 -> 0.74 and 2.46 -> 2.34.
constexpr int row_bytes(int DP) { return DP <= 64 ? 128 : 256; }
constexpr int tile_bytes(int DP) { return DT_ROWS * row_bytes(DP); }          // per 128-column half
constexpr int load_pieces(int DP) { return DP <= 64 ? 2 : 4; }                // 1 KiB loads per wavefront
// where chunk c of row r lies in a tile
template <int DP>
__device__ inline uint32_t dt_chunk_at(int r, int c) {
    if (DP > 64) return r * 256 + ((c ^ dt_swz(r)) << 4);
    const int s = r >> 1;
    return s * 256 + (((c + 8 * (r & 1)) ^ (((s & 1) << 2) | ((s >> 1) & 3))) << 4);
}

// Head dimensions below 128.  A lane fetches the 16-byte chunk at logical position
// pc ^ f(r) of its row.  A chunk that starts at or beyond column d is not fetched at all:
// the lane's offset is set beyond the descriptor's range, for which the load is defined to
// deliver zeros, so those LDS columns hold zeros whatever follows the row in memory.  When d
// is not a multiple of 8 the last chunk of a row holds 4 valid columns and 4 columns of
// whatever follows the row (the next row, a gap of the caller's layout); the kernels'
// PART instantiations clear those four after reading the chunk from LDS (zero_beyond_d).
constexpr uint32_t DT_OUT_OF_RANGE = 0x80000000u;     // >= any descriptor range (all are < 2^31)

// byte offsets (within a tile, global side) of the 4 pieces this lane fetches
// (pitch = bytes between rows in global memory, >= 2 d)
// (half: which 128-column half of the rows this tile holds, 0 unless d > 128)
template <int DP>
__device__ inline void dt_load_offsets(uint32_t (&g)[4], int lane, int wave, int pitch, int d, int half = 0) {
    const int lr = lane >> 4, pc = lane & 15;
#pragma unroll
    for (int j = 0; j < load_pieces(DP); ++j) {
        int r = 16 * wave + 4 * j + lr, chunk = pc ^ dt_swz(r);
        if (DP <= 64) {
            const int s = 8 * wave + 4 * j + lr, x = pc ^ (((s & 1) << 2) | ((s >> 1) & 3));
            r = 2 * s + (x >> 3);
            chunk = x & 7;
        }
        g[j] = 128 * half + 8 * chunk < d ? r * pitch + 256 * half + (chunk << 4) : DT_OUT_OF_RANGE;
    }
}
// PART (d % 8 == 4): fragment of k-step ks read by half h is the chunk 2 ks + h; in the chunk
// that holds column d the elements 4..7 are beyond the row
__device__ inline bf16x8 zero_beyond_d(bf16x8 x, bool is_last_chunk) {
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    i32x4 v = __builtin_bit_cast(i32x4, x);
    v[2] = is_last_chunk ? 0 : v[2];
    v[3] = is_last_chunk ? 0 : v[3];
    return __builtin_bit_cast(bf16x8, v);
}
// Only the k-steps that can hold column d need that: d > 64 for DP = 112 (k-steps 4..6), > 112 for
// 128 (the last one).  32 heads, d 100, 8192 tokens, triangular step, selects on every k-step against
// these: forward 0.604 / 0.585 ms, backward 1.91 / 1.84.
constexpr int part_from(int DP) { return DP <= 64 ? 0 : DP <= 112 ? 4 : 7; }
// The loads go through a buffer descriptor held in scalar registers: the tile's byte
// offset within the (batch, head) matrix is a scalar operand and the lane offset a 32-bit
// vector operand, so a load costs no address arithmetic at all.  The descriptor's range is
// the c rows of the matrix (stride 0, raw 32-bit data format).
//
// The instruction is issued from inline assembly on purpose.  The compiler orders LDS reads
// after a direct load it knows about with a conservative model of what the load writes, and
// puts a wait for ALL loads in flight in front of reads of a different buffer, i.e. right
// after the loads were issued.  Issued this way the loads are invisible to that model; the
// kernels order them by hand: s_waitcnt vmcnt(0) followed by a workgroup barrier before a
// buffer is read, a barrier after its last read before it is requested again.  The
// "memory" clobber keeps the compiler from moving LDS accesses across the request.
typedef int dt_rsrc __attribute__((ext_vector_type(4)));
__device__ inline dt_rsrc dt_make_rsrc(const void* matrix, int rows, int pitch, int d) {
    const uint64_t a = reinterpret_cast<uint64_t>(matrix);
    dt_rsrc r;
    r[0] = (int)(uint32_t)a;
    r[1] = (int)((uint32_t)(a >> 32) & 0xffffu);
    r[2] = (rows - 1) * pitch + 2 * d;     // ends with the last row; the range check is per dword
                                           // and reads past the end return 0
    r[3] = 0x00020000;
    return r;
}
// the same rows `bytes` further on (another device's shard)
__device__ inline dt_rsrc dt_advance(dt_rsrc r, int64_t bytes) {
    const uint64_t a = (((uint64_t)(uint32_t)r[1] << 32) | (uint32_t)r[0]) + (uint64_t)bytes;
    r[0] = (int)(uint32_t)a;
    r[1] = (int)((uint32_t)(a >> 32) & 0xffffu);
    return r;
}
// one 1 KiB piece: 64 lanes x 16 bytes from matrix + tile_byte_offset + lane_offset to
// lds_dst + 16 * lane (lds_dst wave-uniform)
// (m0 is named as clobbered although the compiler calls it reserved: nothing else in these
// kernels uses it, and the note it prints about that is switched off for this function)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void dt_load_piece(dt_rsrc matrix, int tile_byte_offset, uint32_t lane_offset, const char* lds_dst) {
    const uint32_t dst = (uint32_t)reinterpret_cast<uintptr_t>((const lds_char_t*)lds_dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(dst), "v"(lane_offset), "s"(matrix), "s"(tile_byte_offset)
                 : "memory", "m0");
}
// 64 lanes x 4 bytes, to lds_dst + 4 * lane
__device__ inline void dt_load_dword(dt_rsrc matrix, int byte_offset, uint32_t lane_offset, const char* lds_dst) {
    const uint32_t dst = (uint32_t)reinterpret_cast<uintptr_t>((const lds_char_t*)lds_dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 :
                 : "s"(dst), "v"(lane_offset), "s"(matrix), "s"(byte_offset)
                 : "memory", "m0");
}
#pragma clang diagnostic pop
// at most the last n vector memory operations of this wavefront are still on their way
template <int N>
__device__ inline void wait_all_but() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
// all LDS reads so far are in registers: what they read may be overwritten
__device__ inline void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

// what the wavefronts have written to LDS is there for all (direct loads on their way stay so)
__device__ inline void meet() {
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
}

// wave must be wave-uniform (scalar): it selects the LDS destination of each load
template <int DP>
__device__ inline void dt_load(dt_rsrc matrix, int tile_byte_offset, char* lds_tile, const uint32_t (&g)[4], int wave) {
    constexpr int N = load_pieces(DP);
#pragma unroll
    for (int j = 0; j < N; ++j) dt_load_piece(matrix, tile_byte_offset, g[j], lds_tile + (N * wave + j) * 1024);
}
// A-operand row reads: address of row n (within a 32-row half tile), k-step ks, half h
template <int DP>
__device__ inline void dt_row_addrs(uint32_t (&a)[8], int n, int h) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) a[ks] = dt_chunk_at<DP>(n, DP <= 64 ? (2 * ks + h) & 7 : 2 * ks + h);
}
__device__ inline bf16x8 dt_read_row(const char* lds_half, uint32_t addr) {
    return *reinterpret_cast<const bf16x8*>(lds_half + addr);
}
// Transposing reads: addresses (within a group of 16 rows) for 32-column block mb,
// first read (rows +0) and second read (rows +8)
template <int DP>
__device__ inline void dt_tr_addrs(uint32_t (&t0)[4], uint32_t (&t1)[4], int lane) {
    const int i = lane & 15, h = lane >> 5, nh = (lane >> 4) & 1, j4 = i >> 2;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
        const int c = 4 * mb + 2 * nh + ((i & 3) >> 1);      // logical 16-byte chunk
        const int r0 = 4 * h + j4, r1 = r0 + 8;
        t0[mb] = dt_chunk_at<DP>(r0, DP <= 64 ? c & 7 : c) + (i & 1) * 8;
        t1[mb] = dt_chunk_at<DP>(r1, DP <= 64 ? c & 7 : c) + (i & 1) * 8;
    }
}
__device__ inline bf16x8 dt_read_tr(const char* lds_group, uint32_t a0, uint32_t a1) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(lds_group + a0));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(lds_group + a1));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// max / sum over the two half-waves (lanes n and n + 32)
__device__ inline float half_wave_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float half_wave_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ inline f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// MFMA whose accumulator is pinned to ordinary VGPRs.  The dK/dV kernel needs more than 256
// registers, and once a kernel uses AGPRs the compiler places EVERY MFMA result there; the
// S / dP tiles are consumed by VALU instructions, so they would be copied back register by
// register.
//
// Issued from inline assembly, these MFMAs are invisible to the compiler's hazard recogniser,
// so the one software-managed hazard they have is kept by hand.  ISA guide, "Manually inserted
// wait states (NOPs)": XDL (matrix core) write of a VGPR followed by a VALU read or write of
// it needs passes + 3 wait states: 11 for this 8-pass instruction (19 for a 16-pass one).
//  * In the loops the distance is structural: the last S / dP MFMA of a pipeline step is
//    followed by that step's dV / dK products, 4 * MB >= 4 further MFMAs of 8 passes each
//    (>= 128 cycles of the same in-order pipeline), before the next step's first VALU read.
//  * In the prologue nothing lies between: mfma_results_to_valu() inserts 32 wait states and
//    ties the two tiles to the asm statement, so no read of them can be scheduled before it.
__device__ inline void mfma_results_to_valu(f32x16& a) { asm volatile("s_nop 15" : "+v"(a)); }
__device__ inline void mfma_results_to_valu(f32x16& a, f32x16& b) {
    asm volatile("s_nop 15\n\ts_nop 15" : "+v"(a), "+v"(b));
}
// The other software-managed hazard is on the input side: a VALU write of a VGPR followed by
// an MFMA read of it needs 2 wait states (same table).  The operands normally come straight
// from LDS reads (ordered by s_waitcnt, no hazard); only the PART instantiations pass some of them
// through VALU selects first (zero_beyond_d), and then after_valu (known when compiled) puts the
// wait in front of the instruction.
__device__ __forceinline__ void mfma_vgpr_first(f32x16& acc, bf16x8 a, bf16x8 b, bool after_valu) {
    if (after_valu) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_vgpr_acc(f32x16& acc, bf16x8 a, bf16x8 b, bool after_valu) {
    if (after_valu) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}

// Workgroup -> (tile rank, head), ranks heaviest first.  Consecutive workgroups go round-robin to the 8 XCDs; taken
// in chunks of as many ranks as make a multiple of 8 workgroups, an XCD gets the same heads (and at most two others'
// shares) of every chunk, and its L2 holds what they stream.  Head by head, an odd number of heads has every XCD
// stream all of them: d 64, triangular, 25 heads of 2048 rows 125 -> 75 us, 15 of 4096 260 -> 145, 7 of 8192 360 ->
// 242, 128 on 32 of 2048 343 -> 315.  Small launches of uneven work with few ranks, where a chunk is a large part of
// the order, and ranks behind the last whole chunk stay head by head (9 heads of 500 rows, d 100, in chunks 15.3 ->
// 16.1).  (Of the 32-row workgroups the backward's only: the forward gained as often as it lost, full blocks, d 128, 15 heads of 1024 28.0 -> 21.7, 3
// of 5000 60.8 -> 63.7.)
__device__ inline void decode_near(int linear, int n_ranks, int n_heads, bool uneven, int& rank, int& head) {
    const int chunk = n_heads % 8 == 0 ? 1 : n_heads % 4 == 0 ? 2 : n_heads % 2 == 0 ? 4 : 8, size = chunk * n_heads;
    const bool by_head = uneven && n_ranks < 4 * chunk && n_ranks * n_heads < 1024;
    const int i = by_head ? n_ranks : linear / size;
    if ((i + 1) * chunk > n_ranks) {
        rank = linear / n_heads;
        head = linear - rank * n_heads;
        return;
    }
    const int j = linear - i * size, at = j % 8 * (size / 8) + j / 8;
    head = at / chunk;
    rank = i * chunk + at - head * chunk;
}

// Workgroup order of a 1-D grid over (tile rank, batch*head), rank 0 = heaviest tile.
// Large grids: heads are taken in groups of 8; inside a group the index runs over
// heads fastest and tile ranks slowest, so (i) every group runs heaviest-first and
// the last workgroups to start are the lightest, and (ii) as consecutive workgroups
// go round-robin to the 8 XCDs, all tiles of one head land on one XCD and share its
// L2 while they stream the same K/V (or Q/dO) rows.
// Small grids (every workgroup resident at once, at most 2 per CU): plain
// heaviest-first over all heads; with SNAKE the second 256 workgroups run
// lightest-first, so that the two workgroups sharing a CU (indices L and L + 256)
// carry about the same total work.
// Uneven launches in between: by ranks over all heads.  With groups the last heaviest workgroups start when half of
// the launch is over, and it ends with them: 32 tiles of 32 heads, two workgroups to a compute unit, 1.46 times the
// mean load, by ranks 1.0.  An XCD keeps its heads (decode_near), but all at a time.  Triangular step, us, forward /
// backward, groups : ranks: d 128, 24 heads of 4096 122 / 426 : 109 / 381, 64 of 2048 97 / 342 : 86 / 306, 32 of 8192 (2048
// workgroups) 515 / 1791 : 499 / 1740, but 32 of 16384 (4096) 1868 / 6724 : 1895 / 6838 and a ring of 8 x 4096, 16 heads
// (4096), backward 12.97 : 13.43 ms; d 64, 40 of 2560 61 / 198 : 50 / 164, 16 of 12500 354 / 1136 : 320 / 1106.  The line
// is where the gain ends, in workgroups: 3072 below 128 columns (48 heads of 8192, d 64, forward 452 : 419, d 100 740 : 723),
// 2560 at 128 (40 of 8192 663 / 2280 : 641 / 2236, but 192 of 2048 forward 289 : 296, 24 of 16384 backward 5070 : 5153),
// 2048 forward above (64 of 4096, d 256, 710 : 706, 40 of 8192 1498 : 1543, 96 of 4096 1054 : 1102).
// A kernel has one of the two (BY_RANK): with both in its prologue small launches lost, us, one : both, 130 heads of 129
// rows, d 128, forward 13.1 : 13.4, full block 15.5 : 15.9, 32 of 1024, d 256, full, 47.9 : 48.7, one of 512 25.4 : 25.9.
constexpr int HEAD_GROUP = 8;
constexpr int N_CU = 256;
template <int DP, bool FORWARD> constexpr int MOST_BY_RANK = (DP < 128 ? 12 : DP > 128 && FORWARD ? 8 : 10) * N_CU;
inline bool by_rank(bool uneven, int64_t workgroups, int most) { return uneven && workgroups > 2 * N_CU && workgroups <= most; }
template <bool SNAKE, bool BY_RANK>
__device__ inline void decode_block(int linear, int n_tiles, int n_bh, int& rank, int& bh) {
    if constexpr (BY_RANK) return decode_near(linear, n_tiles, n_bh, true, rank, bh);
    const int total = n_tiles * n_bh;
    if (total <= 2 * N_CU) {
        int s = linear;
        if (SNAKE && linear >= N_CU) s = total - 1 - (linear - N_CU);
        rank = s / n_bh;
        bh = s - rank * n_bh;
        return;
    }
    const int per_group = HEAD_GROUP * n_tiles;
    const int grp = linear / per_group;
    const int within = linear - grp * per_group;
    const int heads = min(HEAD_GROUP, n_bh - grp * HEAD_GROUP);
    rank = within / heads;
    bh = grp * HEAD_GROUP + (within - rank * heads);
}

// Row of d <= 16 NF elements (d a multiple of 4) as B-operand fragments, NF k-steps of 16,
// zero-padded to 16 NF columns.  Nothing beyond the row is read.
template <int NF>
__device__ inline void load_b_frags(bf16x8 (&f)[NF], const __bf16* __restrict__ row, int h, int d) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) {
        const int col = 16 * ks + 8 * h;
        if (col + 8 <= d) {
            f[ks] = *reinterpret_cast<const bf16x8*>(row + col);
        } else {
            bf16x4 lo = {0, 0, 0, 0};
            if (col + 4 <= d) lo = *reinterpret_cast<const bf16x4*>(row + col);
            const bf16x4 z = {0, 0, 0, 0};
            f[ks] = __builtin_shufflevector(lo, z, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    }
}

// Rotary embedding of a query row held as B-operand fragments (Sec. 2.3: a token keeps the
// position id of its original place, whatever device it sits on).  Rotate-half pairing: column
// i < d/2 with column i + d/2; with d == DP both sit in the same lane, KS/2 fragments apart.
// turns[i] = base^(-2i/d) / (2 pi) in double precision (LDS, filled once per workgroup); the
// angle in revolutions is reduced to [-1/2, 1/2] in double (position ids reach 10^6, where an
// fp32 angle is off by 0.05 rad) and only then handed to the fp32 sine / cosine instructions,
// which take revolutions.
template <int DP>
__device__ inline void rope_rotate(bf16x8 (&f)[8 * halves_of(DP)], const double* turns, int pos, int h) {
    constexpr int KS = DP / 16;
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double t = (double)pos * turns[16 * ks + 8 * h + e];
            const float r = (float)(t - rint(t));
            const float sn = __builtin_amdgcn_sinf(r), cs = __builtin_amdgcn_cosf(r);
            const float lo = (float)f[ks][e], hi = (float)f[ks + KS / 2][e];
            f[ks][e] = (__bf16)fmaf(lo, cs, -hi * sn);
            f[ks + KS / 2][e] = (__bf16)fmaf(hi, cs, lo * sn);
        }
}
template <int DP>
__device__ inline void fill_rope_turns(double* turns, int tid, double log2_base) {
    if (tid < DP / 2) turns[tid] = exp2(-2.0 * tid / DP * log2_base) * 0.15915494309189535;
}

}  // namespace sa
