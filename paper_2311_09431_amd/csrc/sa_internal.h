// Internal declarations shared by the HIP translation units of libstriped_attn.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "striped_attn.h"

namespace sa {

// Mask of one ring step in local indices: key b is allowed for query a iff
// b <= a - off (kind == TRI) or always (kind == FULL).  Derived from the
// original token positions: striped a*N + dev, contiguous dev*c + a.
enum MaskKind : int { MASK_EMPTY = 0, MASK_TRI = 1, MASK_FULL = 2 };

// GetMask(j, k) in local indices (Sec. 2.2, 2.3): query a = original position j*c + a
// (contiguous) or a*N + j (striped); key b likewise with k.  Allowed iff key position <= query
// position, which reduces to b <= a - off.
__host__ __device__ inline int block_kind(int q_dev, int kv_dev, int layout) {
    if (layout == SA_STRIPED || q_dev == kv_dev) return MASK_TRI;
    return q_dev < kv_dev ? MASK_EMPTY : MASK_FULL;
}
__host__ __device__ inline int block_off(int q_dev, int kv_dev, int layout) {
    return layout == SA_STRIPED && kv_dev > q_dev ? 1 : 0;
}

// What a workgroup of the matrix-core kernels walks: one triangular or one full block (a ring
// step; the mask form is then known when the kernel is compiled), or the blocks of several shards
// one after the other without draining the pipeline between them.
enum Walk : int { WALK_TRI = 0, WALK_FULL = 1, WALK_RING = 2 };

// Rank of a (tile, device) pair -> both, heaviest first.  Striped blocks all have the same
// shape, so the tile decides; contiguous ones are walked whole for every device further on, so
// the device does.  tile_rank: 0 = the heaviest tile of a triangular block, dev_rank: 0 = the
// device with the most blocks.
__device__ inline void decode_rank(int rank, int n_tiles, int n_dev, int layout, int& tile_rank, int& dev_rank) {
    if (layout == SA_STRIPED) {
        tile_rank = rank / n_dev;
        dev_rank = rank - tile_rank * n_dev;
    } else {
        dev_rank = rank / n_tiles;
        tile_rank = rank - dev_rank * n_tiles;
    }
}

struct StepArgs {
    const void* q;
    const void* k;
    const void* v;
    const void* dout;     // backward only
    float* o;             // forward: running output
    float* lse;           // forward: running log-sum-exp; backward: final (read-only)
    const float* delta;   // backward only
    float* dq;
    float* dk;
    float* dv;
    int B, H, c, d;
    int64_t stride_b, stride_h, stat_stride_b, stat_stride_h;
    int64_t stride_s;     // elements between consecutive rows (>= d)
    // K, V, dK, dV: H_kv heads (H_kv divides H; query head h reads head h / (H / H_kv)) with
    // strides of their own; equal to H and the strides above for plain multi-head attention
    int H_kv;
    int64_t kv_stride_b, kv_stride_h, kv_stride_s;
    float scale;
    // Blocks of this launch: query shards of devices q_dev .. q_dev + n_q - 1 against key shards
    // of devices kv_dev .. kv_dev + n_kv - 1 (the pointers are those of the first of each; further
    // ones follow q_shard / kv_shard elements on, statistics c rows on).  One ring step is 1 x 1
    // (never an empty block); the ring drivers hand over all blocks of a device or of the ring at
    // once, and each workgroup walks the other side's shards in the order of their device index.
    int layout, q_dev, n_q, kv_dev, n_kv;
    int64_t q_shard, kv_shard;
    // results start from an empty state (forward) or zero accumulators (backward): nothing of
    // o, lse, dq, dk, dv is read.  Otherwise they are folded into what is there.
    bool fresh;
    // Emulated tile-skipping granularity (Sec. 3.1), MFMA kernels only: 0 = the kernel's own
    // (32 x 32); otherwise every sub-tile of a skip_bq x skip_bk tile of the block that holds
    // at least one allowed pair is computed (masked elements contribute exact zeros).
    // Both are multiples of 128 that divide c.
    int skip_bq, skip_bk;
    // Forward only, MFMA kernels only: rotary embedding of the QUERY rows applied while they
    // are loaded (q holds unrotated rows; k is expected rotated already).  q_pos: position ids
    // of the c query rows per batch (int32, pos_stride_b elements between batches, 0 = shared),
    // NULL = no rotation.  rope_log2_base = log2 of the frequency base.
    const int32_t* q_pos;
    int64_t pos_stride_b;
    double rope_log2_base;
};

// The workgroups of a launch carry uneven work: triangular blocks, or contiguous blocks of
// several query devices (a key shard is seen by the devices from its own on).
__host__ __device__ inline bool uneven(const StepArgs& a) { return a.layout == SA_STRIPED || a.n_q > 1 || a.q_dev == a.kv_dev; }

// Order of a backward launch of n_keys key-owning and n_queries query-owning workgroups, each sequence
// heaviest first: `first` key-owning ones, whose walks are longer than the longest query-owning one, then the
// rest of both evenly interleaved, in units of 8 workgroups: consecutive workgroups go round-robin to the 8 XCDs,
// and one by one equal numbers of both kinds left each kind four of them (2 heads of 4096 rows, full block,
// split kernels 81 -> 66 us; 16 of 2048, triangular, 128-row kernels 87 -> 81).  What fills no unit, less than 8
// of each kind, the lightest, comes last.  All of an even launch's key-owning walks are longer (`ratio` times,
// times the group); of an uneven one, whose walks shrink evenly to almost nothing, those before that point
// are.  ratio 0: both kinds from the start.
struct BothKinds { int first, unit, keys, total, last; };      // keys, total: units; last: key-owning ones of the end
inline BothKinds both_kinds(const StepArgs& a, int64_t n_keys, int64_t n_queries, double ratio, int unit = 8) {
    BothKinds b;
    const double longer = ratio * (a.H / a.H_kv);
    b.first = !uneven(a) ? (int)n_keys : longer > 1. ? (int)(n_keys * (1. - 1. / longer)) / 8 * 8 : 0;
    b.unit = unit;
    b.keys = (int)(n_keys - b.first) / unit;
    b.total = b.keys + (int)n_queries / unit;
    b.last = (int)(n_keys - b.first) % unit;
    return b;
}
// the kind of workgroup `linear` and its place among those of its kind
__device__ inline bool owns_keys(const BothKinds& b, int& linear) {
    if (linear < b.first) return true;
    const int u = (linear - b.first) / b.unit, at = linear - b.first - u * b.unit;
    if (u >= b.total) {
        const int end = linear - b.first - b.total * b.unit;
        const bool keys = end < b.last;
        linear = keys ? b.first + b.keys * b.unit + end : (b.total - b.keys) * b.unit + end - b.last;
        return keys;
    }
    const int before = (int)((int64_t)u * b.keys / b.total);
    const bool keys = (int)(((int64_t)u + 1) * b.keys / b.total) > before;
    linear = keys ? b.first + before * b.unit + at : (u - before) * b.unit + at;
    return keys;
}

// The same for workgroups that have a compute unit to themselves (bwd_both_ring_kernel, bwd_both_mfma_kernel).  Consecutive ones go to the 8 XCDs
// in turn and, within one, to its 4 shader engines in turn, whether there is room or not: 32 places.  One of a kind evenly
// among the others comes back to the same places wherever their numbers are near a simple ratio (every fourth, with three
// query heads to a key/value head: two XCDs, or in units of 8 one shader engine of each), and the launch waits for
// those.  So the rarer kind's units go through the columns of rows of 32 places one after the other, as many in each row as
// its share is.  Backward step, d 128 unless said, us, evenly : so: 72 heads on 24 of 1664 rows (312 key tiles) 350 : 228, 455 on
// 65 of 512 569 : 212, 4050 on 270 of 128 1143 : 350, 160 on 32 of 1024 252 : 204; numbers that were no such ratio as before (32 on 8
// of 4096 472 : 467, 16 of 2048 78.4 : 77.0, 10 of 4096 167 : 164).
// One device's queries against more shards of keys: where their walks (of products, 3 a pair, each shard) outlast the keys' (4 a
// pair, each head of the group), all of them go first and the short walks behind them fill up.  Last device, its share of a
// ring, evenly and behind the first third or (contiguous) all of the keys : so: 16 heads of 8 x 1024 201 : 176, 25 of 14 x 505 434 :
// 176, 8 on 2 of 12 x 3968, d 96, 1660 : 1156, 4 of 8 x 2048 303 : 297, contiguous 8 of 4 x 2048 253 : 215, 4 of 8 x 4096 979 : 826; but 2 of 4 x
// 8192 607 : 616.
// Units: 8 where both numbers are multiples (48 heads of 871 rows, d 116, 61.7, one by one 65.9, 16 of 2048 the same), else one by one.
struct PlacedKinds {
    int queries_first, keys_first, shift;       // workgroups; log2 of a unit of the rest
    int keys, total, to_row, rows, last;        // of the rest, units; log2 of a row's, rows; key-owning workgroups of the end
    uint32_t per_row, rarer;                    // units of the rarer kind: in 2^-24 a row, all
};
// Up to 64 columns and above 128 (bwd_both_mfma_kernel) only where the rarer kind would be exactly in step, every second, fourth ...
// workgroup or unit: 855 heads on 57 of 512 rows, d 48, 1406 : 256, 539 on 77 of 350, d 64, 338 : 119, 204 on 68 of 384 84 : 53, 30 on 15 of
// 1280, d 136, 182 : 141.  Launches whose numbers are no such ratio, and shares, keep to the even order (rows of one place): some
// gained and some lost by the other (378 heads on 126 of 128 rows, d 136, 72.5 : 78.7, 18 of 219 23.7 : 25.8).
inline PlacedKinds placed_kinds(const StepArgs& a, int64_t n_keys, int64_t n_queries, double ratio) {
    const bool ring = a.d > 64 && a.d <= 128, ahead = ring && a.n_kv > a.n_q && 3 * a.n_kv >= 4 * a.n_q * (a.H / a.H_kv);
    PlacedKinds k;
    k.queries_first = ahead ? (int)n_queries : 0;
    if (ahead) n_queries = 0;
    const BothKinds b = both_kinds(a, n_keys, n_queries, ratio, n_keys % 8 || n_queries % 8 ? 1 : 8);
    k.keys_first = ahead ? (int)n_keys : b.first;
    k.shift = b.unit == 8 ? 3 : 0;
    k.keys = b.keys; k.total = b.total; k.last = b.last;
    k.rarer = (uint32_t)(b.keys < b.total - b.keys ? b.keys : b.total - b.keys);
    const bool in_step = k.rarer && b.total % (int)k.rarer == 0 && b.total / (int)k.rarer % 2 == 0;
    k.to_row = ring || in_step ? 5 - k.shift : 0;           // 32 places
    k.rows = b.total >> k.to_row ? b.total >> k.to_row : 1;
    k.per_row = (uint32_t)(((uint64_t)k.rarer << 24) / k.rows);
    return k;
}
__host__ __device__ inline bool owns_keys(const PlacedKinds& k, int& linear) {
    if (linear < k.queries_first) return false;
    linear -= k.queries_first;
    if (linear < k.keys_first) return true;
    const int in_rest = linear - k.keys_first, u = in_rest >> k.shift, at = in_rest - (u << k.shift);
    if (u >= k.total) {
        const int end = in_rest - (k.total << k.shift);
        const bool keys = end < k.last;
        linear = keys ? k.keys_first + (k.keys << k.shift) + end : ((k.total - k.keys) << k.shift) + end - k.last;
        return keys;
    }
    const int cols = 1 << k.to_row, row = u >> k.to_row, col = u & (cols - 1);
    auto before = [&](int r) -> int { return r >= k.rows ? (int)k.rarer : (int)(((uint64_t)r * k.per_row + (1u << 24) - 1) >> 24); };
    // the rarer kind's units follow one another through the columns: those of this row are n from column `from` on, around the end
    const int before_row = before(row), n = before(row + 1) - before_row, from = before_row & (cols - 1);
    const bool is_rarer = ((col - from) & (cols - 1)) < n, keys = is_rarer == (2 * k.keys <= k.total);
    const int behind = col - from < 0 ? 0 : col - from < n ? col - from : n, around = from + n - cols;
    const int rarer = before_row + behind + (around < 0 ? 0 : around < col ? around : col);
    linear = (keys ? k.keys_first : 0) + ((is_rarer ? rarer : u - rarer) << k.shift) + at;
    return keys;
}

// Where the tile to request begins, in bytes.  Behind a walk's end, where requests fetch nothing, it stays: counted on it would
// pass 2^31 at the widest row strides, a negative scalar offset, which the range check of a descriptor is not known to stop
// (offsets from 0 to 2^31 behind the range, which may be empty, read as zeros: measured, 4 and 16 bytes a lane).
// (Set to 0 there instead, the compiler gives every tile a jump or scalar registers it lacks: 32 heads of 32768 rows, d 128, 24460
// -> 24640 us, 26 of d 100, 8 x 8192 rows, 18570 -> 18965.)
struct TileByte {
    int at, pitch;
    __host__ __device__ void block(int first_tile) { at = first_tile * pitch; }
    __host__ __device__ void next() { at += pitch; }
    __host__ __device__ void stop() { pitch = 0; }
};

// The fp32 instruction's kernels: 128-row workgroups would leave compute units idle, and the streamed rows are split
// over the wavefronts instead.  In the backward a key-owning workgroup walks the queries of its whole
// group of heads, so with few key/value heads it is their number that counts.  One step, 32 query
// heads, d 256, 128-row kernel against the split one, ms, triangular and full block: 64 key tiles (8 key/value heads
// of 1024 tokens) 2.37 : 1.42, 2.38 : 1.64; 128 (8 of 2048) 4.90 : 3.66, 5.58 : 6.46; 256 (16 of 2048) 3.12 : 3.58,
// 5.62 : 6.38; one head of 4096 (32 tiles) 64 : 38, 70 : 43.
inline bool few_row_tiles(const StepArgs& a, bool backward) {
    const int64_t tiles = (int64_t)((a.c + 127) / 128) * a.B, keys = tiles * a.n_kv * a.H_kv;
    return tiles * a.n_q * a.H < 256 || (backward && keys <= (uneven(a) ? 128 : 64));
}

// launchers: return hipSuccess or the launch error
hipError_t launch_permute(const void* src, void* dst, int64_t outer, int64_t n_seq,
                          int64_t inner_bytes, int N, bool inverse, hipStream_t st);
hipError_t launch_state_init(float* o, float* lse, const sa_shape& s, hipStream_t st);
hipError_t launch_finalize(const float* o, void* out, const sa_shape& s, hipStream_t st);
// rows: of each (batch, head), with the shape's strides; its c is not used
hipError_t launch_bwd_preprocess(const float* o, const void* dout, float* delta,
                                 const sa_shape& s, int64_t rows, hipStream_t st);
hipError_t launch_zero_f32(float* p, const sa_shape& s, int64_t rows, hipStream_t st);
hipError_t launch_rope(const void* x, void* y, const int32_t* pos, int64_t pos_stride_b, const sa_shape& s,
                       float base, bool inverse, hipStream_t st);

hipError_t launch_fwd_f32(const StepArgs& a, int dtype, hipStream_t st);
hipError_t launch_bwd_f32(const StepArgs& a, int dtype, hipStream_t st);
// fp32 storage of up to 128 columns: the fp32 instruction, or three-term products in workgroups of 32 or of 128 rows (ALONE:
// the backward's with one wavefront to 32 rows)
enum F32Route : int { F32_INSTRUCTION = 0, F32_SPLIT = 1, F32_TERMS = 2, F32_TERMS_ALONE = 3 };
F32Route f32_route(const StepArgs& a, bool backward);
hipError_t launch_f32x3(const StepArgs& a, bool backward, bool alone, hipStream_t st);
bool f32x3_split_supported(const StepArgs& a, bool backward);
hipError_t launch_f32x3_split(const StepArgs& a, bool backward, hipStream_t st);
bool fwd_mfma_supported(const StepArgs& a, int dtype);
bool fwd_mfma_rope_supported(const StepArgs& a, int dtype);
hipError_t launch_fwd_mfma(const StepArgs& a, hipStream_t st);
bool bwd_mfma_supported(const StepArgs& a, int dtype);
hipError_t launch_bwd_mfma(const StepArgs& a, hipStream_t st);
// whether the 128-row kernels' two kinds of workgroups share a launch
bool bwd_one_launch(const StepArgs& a);
// 65 to 128 columns: dK and dV, or (kinds) both kinds of workgroups in one launch
hipError_t launch_bwd_ring(const StepArgs& a, const PlacedKinds* kinds, int workgroups, hipStream_t st);
bool bwd_split_wanted(const StepArgs& a);
bool dkdv_by_rank(const StepArgs& a);
hipError_t launch_bwd_split(const StepArgs& a, hipStream_t st);
bool fwd_split_wanted(const StepArgs& a);
bool fwd_by_rank(const StepArgs& a);
hipError_t launch_fwd_split(const StepArgs& a, hipStream_t st);
bool few_rows_wanted(const StepArgs& a, int dtype, bool backward);
hipError_t launch_few_rows(const StepArgs& a, int dtype, bool backward, hipStream_t st);
bool short_exact_wanted(const StepArgs& a, int dtype, bool backward);
hipError_t launch_short_exact(const StepArgs& a, bool backward, hipStream_t st);

}  // namespace sa
