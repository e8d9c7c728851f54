// Which kernels play an fp32 launch of up to 128 columns (host code).
//
// Three kinds compete: 32-row workgroups on the fp32 instruction (f32_step.hip, the cheapest start, the dearest tile), 32-row
// workgroups of three-term products (f32x3_split.hip), and 128-row (forward launches of 512 such tiles and more: 256-row)
// workgroups of them that share the splitting of the streamed rows (f32x3_step.hip), in the backward with two wavefronts to
// 32 rows or, where alone_wanted says so, one.  Neither the number of tiles nor the walk decides alone, so each kind's time is put together from what a
// workgroup takes, and the least wins.
//
// The figures are fitted to 3374 launches (d 32, 64, 100, 128; 1 to 1024 heads, groups of 4, of 17 to 4096 rows, steps and rings
// of 2 to 16, both layouts), each measured with every kind, to 5 to 10 %.  What the rule picks takes, forward / backward, 0.3 /
// 0.6 % more than the best kind (geometric mean).  Without the first kind and the one wavefront: 64 heads of 128 rows, d 128, forward 13.7 ->
// 17.3 us, backward 37.9 -> 52.7; one of 128 12.9 -> 16.4, 21.9 -> 29.0; ring of 8 x 256, 32 heads, 263 -> 345.
#include <math.h>

#include "mfma_tiles.h"
#include "sa_internal.h"

namespace sa {

namespace {

// us: until the first product and behind the last, per round of a walk, and as a share of that what a workgroup takes of
// its compute unit beside others (less than 1 where several fit)
struct Takes { double start, tile, share; };
struct Kind {
    int rows, round;            // rows a workgroup owns, streamed rows a round
    Takes by[4];                // up to 32, 64, 112 and 128 columns
    double queries;             // a query-owning workgroup's time as a share of a key-owning one's
    double tail;                // of the longest walk, added to the mean load
    double whole;               // 1: workgroups take their compute units in whole rounds
    double staged;              // what a round costs a workgroup whose wavefronts see nothing in it
    double crowd;               // the longest walk is longer by this where the chip is full
};
constexpr Kind FWD_INSTRUCTION = {32, 128, {{4.4, 3.1, .522}, {4.7, 4.14, .79}, {5.19, 7.8, 1.02}, {5.85, 7.49, .956}}, 1, .0481, .434, 1, 0};
constexpr Kind FWD_SPLIT = {32, 32, {{4.95, .274, .944}, {5.61, .383, 1.12}, {8.43, .789, 1.05}, {13.2, .774, 1.09}}, 1, .0683, .612, 1, 0};
constexpr Kind FWD_TERMS = {128, 32, {{3.89, 2.08, .862}, {4.96, 1.84, .965}, {7.75, 3.08, .658}, {7.39, 3.02, .937}}, 1, .148, .898, 1, 0};
constexpr Kind FWD_TERMS_WIDE = {256, 32, {{5.5, 2.55, 1.03}, {6.29, 2.55, 1.02}, {9, 4.35, 1.06}, {11.8, 4.21, 1.26}}, 1, 0, .635, .5, 0};
constexpr Kind BWD_INSTRUCTION = {32, 128, {{4.38, 4.37, .547}, {5.36, 8.85, .669}, {7.35, 10.7, .989}, {7.59, 12.8, .75}}, .758, .175, 1, 1, .0802};
constexpr Kind BWD_SPLIT = {32, 32, {{5.18, .314, 1.19}, {6.33, .584, 1.35}, {17.1, 1.3, 1.15}, {22.8, 1.39, 1.03}}, .79, .0916, .801, 1, .101};
constexpr Kind BWD_TERMS = {128, 32, {{5.12, 2.46, 1.23}, {4.98, 2.45, 1.09}, {10.3, 4.28, 1.18}, {13.2, 4.38, 1.09}}, .812, 0, .513, 1, .0576};

int up(int x, int by) { return (x - 1) / by + 1; }

// waves: how many wavefronts share a walk by taking whole rounds in turn (1: all take part in each)
double time_of(const Kind& k, const StepArgs& a, bool backward, int waves) {
    const Takes& t = k.by[a.d <= 32 ? 0 : a.d <= 64 ? 1 : a.d <= 112 ? 2 : 3];
    // contiguous layout: key shards behind the last played device are seen by nobody
    const int n_kv = a.layout == SA_STRIPED ? a.n_kv : a.q_dev + a.n_q - a.kv_dev < a.n_kv ? a.q_dev + a.n_q - a.kv_dev : a.n_kv;
    const int tiles = up(a.c, k.rows), m = up(a.c, k.round), m32 = up(a.c, 32);
    // the mean walk as a share of the longest, given a triangular block's
    auto mean = [&](double tri) {
        if (a.layout == SA_STRIPED) return tri;
        if (a.n_q > 1) return ((n_kv - 1) / 2. + tri) / n_kv;
        return a.kv_dev + n_kv > a.q_dev ? (n_kv - 1 + tri) / n_kv : 1.;
    };
    const int steps = up(a.c, k.rows > k.round ? k.rows : k.round);
    const double share = k.staged * mean((steps + 1) / (2. * steps)) + (1 - k.staged) * mean((m32 + 1) / (2. * m32));
    // the longest: of a triangular block the heaviest tile, whose wavefronts see nothing of the last rounds
    const int own = k.rows / 32 < m32 ? k.rows / 32 : m32;
    const double last = (m32 - (own - 1) / 2.) / m32;
    const double seen = a.layout == SA_STRIPED ? last : a.n_q == 1 && a.kv_dev + n_kv <= a.q_dev ? 1. : (n_kv - 1 + last) / n_kv;
    const double longest_share = k.staged + (1 - k.staged) * seen;
    const double queries = (double)a.B * a.H * a.n_q * tiles, keys = backward ? (double)a.B * a.H_kv * n_kv * tiles : 0.;
    const double query_walk = (double)m * n_kv, key_walk = (double)m * a.n_q * (a.H / a.H_kv);
    auto whole_rounds = [&](double walk) { return ceil(walk / waves) * waves; };
    const double q = backward ? k.queries : 1.;
    double longest = q * (t.start + t.tile * longest_share * whole_rounds(query_walk));
    if (backward) longest = fmax(longest, t.start + t.tile * longest_share * whole_rounds(key_walk));
    const double n = queries + keys;
    longest *= 1 + k.crowd * fmin(1., n / 192);
    const double load = keys * (t.start + t.tile * share * key_walk) + queries * q * (t.start + t.tile * share * query_walk);
    const double filled = 1 - k.whole + k.whole * N_CU * ceil(n / N_CU) / n;
    return fmax(longest, load * filled * t.share / N_CU + k.tail * longest);
}

}  // namespace

// One wavefront to 32 rows in the 128-row backward: a triangular block of one or two tiles, of more heads than half fill the
// chip.  Two : one, us: 100 heads of 40 rows, d 128, 29.9 : 27.7, 128 of 96 46.0 : 37.8, 128 of 128 57.8 : 46.5, d 100 55.8 : 44.5,
// 256 of 200 179 : 172, 512 of 256, d 100, 445 : 416, 1024 of 128 388 : 339; but 64 of 96, d 100, 30.9 : 31.4, 128 of 300 as long,
// 64 of 512 142 : 149, 32 of 1024 224 : 235, full block, 1024 of 64, d 100, 164 : 185, ring of 2 x 384, 32 heads, 162 : 175.
static bool alone_wanted(const StepArgs& a) {
    return a.d > 64 && uneven(a) && a.n_q == 1 && a.n_kv == 1 && a.c <= 256 && (int64_t)up(a.c, 128) * a.B * (a.H + a.H_kv) > 128;
}

F32Route f32_route(const StepArgs& a, bool backward) {
    F32Route route = F32_TERMS;
    const bool wide = !backward && (int64_t)a.B * a.H * a.n_q * up(a.c, 128) >= 512;        // (as f32x3_step.hip decides)
    double least = time_of(backward ? BWD_TERMS : wide ? FWD_TERMS_WIDE : FWD_TERMS, a, backward, 1);
    auto compete = [&](F32Route with, const Kind& k, int waves) {
        const double t = time_of(k, a, backward, waves);
        if (t < least) {
            least = t;
            route = with;
        }
    };
    if (f32x3_split_supported(a, backward)) compete(F32_SPLIT, backward ? BWD_SPLIT : FWD_SPLIT, a.d <= 64 ? 8 : 4);
    if (few_row_tiles(a, backward)) compete(F32_INSTRUCTION, backward ? BWD_INSTRUCTION : FWD_INSTRUCTION, 1);
    if (route == F32_TERMS && backward && alone_wanted(a)) route = F32_TERMS_ALONE;
    return route;
}

}  // namespace sa
