// Device code of libfastgrid: pyramid, FAST score, 3x3 NMS and per-cell
// arg-max over all pyramid levels ("Faster than FAST", Sections II-B to II-D).
//
// Work decomposition
// ------------------
// A workgroup owns a region of whole grid cells (a multiple of 16 level-0
// pixels wide and tall) and walks it in 64x64 level-0 sub-tiles.  A sub-tile is
// loaded once with a 4*2^(L-1)-pixel halo for its first L <= 3 levels, and levels
// 1 and 2 are built from it in LDS (one pass over HBM: level 0 read once, levels
// 1.. written once).  Levels 3.. follow in one more pass per three levels, by
// regions of 128 level-0 pixels (16 of level 3), which build and detect theirs
// alike.
//
// Detection of a sub-tile scores every pixel of its area plus a 1-pixel ring
// at every level:
//
//   P1 compass test, 8 pixels per lane, four to a register.  An arc of N
//      circle pixels contains floor(N/4) consecutive compass points (circle
//      indices 0, 4, 8, 12) of its label.  The 8-pixel groups of all levels
//      are dealt to the waves round-robin in rounds of 64.
//   P2 compaction of the survivors into a wave-private LDS list (ballot +
//      mbcnt over groups, then a DPP prefix scan over pixels).
//   P3 8-point test, one survivor per lane: the arc also contains floor(N/2)
//      consecutive even circle points of its label.  In-place compaction.
//   P4 full segment test and score (Section II-D, Eq. (1)) into the level's
//      score map (the sub-tile area plus its ring).
//   P5 after one workgroup barrier, 3x3 NMS (Section I-B, n=1) of the
//      sub-tile's own pixels and an LDS atomicMax of a 32-bit key per cell:
//      (score << 19) | ((7-level) << 16) | (0xFFFF - row-major index inside
//      the cell), which orders candidates by (score desc, level asc, index
//      asc), so the cell's answer does not depend on thread order.
//
// P1-P4 need no workgroup barrier.  Both filters are necessary conditions of
// the segment test, so a pixel they reject has score 0; the cascade never
// changes a result.
#include <type_traits>

#include "fg_internal.h"

namespace {

constexpr int SUB = FG_SUB;             // sub-tile side at level 0
constexpr int MAX_FUSED = FG_MAX_FUSED;   // levels built in LDS from one load

// All level tiles share one LDS row pitch, so circle offsets are constants.
// Band A (rows 0..95): level 0 of a fused sub-tile, or the first level of an upper
// region.  Band B (rows 96..143): the next level at byte 8, the one after at byte 68.
// For a sub-tile whose origin is a multiple of 16 pixels, the compass groups
// of every level then start 4 bytes past a multiple of 8, so the row words
// around a group are two aligned 8-byte reads (load8<true>).
constexpr int LP = 112;
constexpr int T0 = 16;
constexpr int T1 = 96 * LP + 8;
constexpr int T2 = 96 * LP + 68;
constexpr int TILE_BYTES = 144 * LP;
static_assert(T0 % 16 == 0 && LP % 16 == 0, "16-byte tile stores in band A");
static_assert(T1 % 8 == 0 && T2 % 4 == 0, "8-byte reads when halving level 1");
static_assert(LP % 8 == 0 && T0 % 8 == 0 && T1 % 8 == 0 && T2 % 8 == 4, "aligned compass row reads");
static_assert(TILE_BYTES <= 16384, "entries hold 14-bit LDS offsets");
// Score maps: a level's sub-tile area plus a 1-pixel ring.
constexpr int M0_ROWS = SUB + 2, M1_ROWS = SUB / 2 + 2, M2_ROWS = SUB / 4 + 2;
constexpr int MP = SUB + 4;   // one pitch for every level's score map
constexpr int MAX_RCELLS = 16;
constexpr int MAX_KEYS = MAX_RCELLS * MAX_RCELLS;
// Groups of 8 pixels scored per sub-tile, at most: every level's area plus a
// 1-pixel ring, in whole groups (66 x 9 + 34 x 5 + 18 x 3 for three levels).
constexpr int MAX_GROUPS = 66 * 9 + 34 * 5 + 18 * 3;
constexpr uint16_t NO_ENTRY = 0xFFFF;

constexpr int OFF_M0 = TILE_BYTES;
// levels 1 and 2 share a band of M1_ROWS rows: level 1 in columns 0..35,
// level 2 in columns 40..59
constexpr int OFF_M1 = OFF_M0 + M0_ROWS * MP * 2;
constexpr int OFF_M2 = OFF_M1 + 40 * 2;
constexpr int OFF_KEYS = (OFF_M1 + M1_ROWS * MP * 2 + 15) & ~15;
static_assert(SUB / 2 + 4 <= 40 && 40 + SUB / 4 + 4 <= MP && M2_ROWS <= M1_ROWS, "level 1 and 2 maps share a band");
constexpr int OFF_KEYS2 = OFF_KEYS + MAX_KEYS * 4;   // second buffer for the pipelined kernel
constexpr int OFF_WAVES = OFF_KEYS2 + MAX_KEYS * 4;
static_assert(OFF_WAVES % 16 == 0, "aligned scratch");

// Per-wave scratch for V waves.  Compass rounds are dealt to the waves in
// turn, so a wave sees at most ceil(MAX_GROUPS / 64V) rounds of 64 groups:
// its group list holds that many words (64 per round) and its pixel list
// eight pixels per group plus one spare slot per lane.
__host__ __device__ constexpr int blist_cap(int waves) {
    return (MAX_GROUPS + 64 * waves - 1) / (64 * waves) * 64;
}
__host__ __device__ constexpr int list_cap(int waves) { return 8 * blist_cap(waves); }
__host__ __device__ constexpr int wave_bytes(int waves) {
    return (blist_cap(waves) * 4 + (list_cap(waves) + 64) * 2 + 15) & ~15;
}

}  // namespace

size_t fg_smem_bytes(int block) { return (size_t)OFF_WAVES + (size_t)(block / 64) * wave_bytes(block / 64); }

namespace {

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Image planes and outputs reach the kernels as generic pointers inside job
// structs.  Accessing them through global-address-space pointers makes the
// compiler emit global (not flat) loads and stores, which are counted by
// vmcnt only: outstanding HBM traffic then never holds up an LDS wait.
#define GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ T gload(const void *p) {
    return *(const GLOBAL T *)p;
}
template <class T>
__device__ __forceinline__ void gstore(void *p, T v) {
    *(GLOBAL T *)p = v;
}

__device__ __forceinline__ s16x2 vmax(s16x2 a, s16x2 b) { return __builtin_elementwise_max(a, b); }
__device__ __forceinline__ s16x2 vmin(s16x2 a, s16x2 b) { return __builtin_elementwise_min(a, b); }

// floor(a / b) for 0 <= a < 2^21 and b >= 1 with the approximate reciprocal:
// (a + 0.5) / b lies at least 0.5 / b from an integer, and the relative error
// of rcp and of the product (< 2^-22) keeps the estimate closer than that.
__device__ __forceinline__ int div_small(int a, int b) {
    return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b));
}

// An LDS pointer the compiler cannot see through.  Reads at constant
// non-negative offsets from it then share one address register and carry the
// offsets in the instructions' (unsigned) immediate fields, instead of the
// compiler folding the base into each address and adding negative offsets
// with separate instructions.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(3))) T *lds_base(const T *p) {
    const __attribute__((address_space(3))) T *q = (const __attribute__((address_space(3))) T *)p;
    asm("" : "+v"(q));
    return q;
}

__device__ __forceinline__ int lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Orders this wave's LDS accesses across its lanes (LDS executes one wave's
// operations in order; this keeps the compiler from reordering them).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Inclusive prefix sum over the 64 lanes: shifts within rows of 16 lanes,
// then the row totals are broadcast into the following rows.
__device__ __forceinline__ int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return x;
}

// Bit i of the result is set iff bits i..i+n-1 of m are all set (1 <= n <=
// 16): runs of 2, 4, 8, 16 by doubling while they fit in n, then the
// remainder.  The shift amounts depend on n only (uniform, so they are scalar
// and hoisted out of the callers' loops); a step that does not apply shifts by
// 0, so the code has no branches.
__device__ __forceinline__ uint32_t runs(uint32_t m, int n) {
    const int s1 = n >= 2 ? 1 : 0, s2 = n >= 4 ? 2 : 0, s4 = n >= 8 ? 4 : 0, s8 = n >= 16 ? 8 : 0;
    m &= m >> s1;
    m &= m >> s2;
    m &= m >> s4;
    m &= m >> s8;
    return m & (m >> (n - 1 - s1 - s2 - s4 - s8));
}

// The same for n <= 8.
__device__ __forceinline__ uint32_t runs8(uint32_t m, int n) {
    const int s1 = n >= 2 ? 1 : 0, s2 = n >= 4 ? 2 : 0, s4 = n >= 8 ? 4 : 0;
    m &= m >> s1;
    m &= m >> s2;
    m &= m >> s4;
    return m & (m >> (n - 1 - s1 - s2 - s4));
}

// Threshold constants of the compass test, one byte per pixel (uniform).
//
// v_lerp_u8 halves the sum of two bytes, for four pixels at once, rounding down
// or (third operand 1) up.  Of a circle point X and the centre C,
// q = (X + (255 - C)) / 2 is 127.5 + (X - C) / 2 rounded, so X > C + t and
// X < C - t are thresholds on q, and bit 7 of lerp(q, 256 - b) says q >= b:
//   brighter       q >= 128 + ceil(t/2), exact when q is rounded up for odd t;
//   not darker     q >= 128 - floor(t/2), which takes a point exactly t darker
//                  for darker too (the filter only has to keep every corner).
struct CompassT {
    uint32_t round, bright, dark;
};

__device__ __forceinline__ CompassT compass_t(int t) {
    return CompassT{(uint32_t)(t & 1) * 0x01010101u, (uint32_t)(128 - ((t + 1) >> 1)) * 0x01010101u,
                    (uint32_t)(128 + (t >> 1)) * 0x01010101u};
}

// Compass test of the four pixels of C: bit 7 of a byte is set where the pixel
// may be a corner (the other bits are not cleared).  K = floor(N/4) consecutive
// points of (N, E, S, W) must all be brighter, or all darker.
template <int K>
__device__ __forceinline__ uint32_t compass4(uint32_t C, uint32_t N, uint32_t E, uint32_t S, uint32_t W,
                                             const CompassT &T) {
    auto q = [&](uint32_t x) { return __builtin_amdgcn_lerp(x, ~C, T.round); };
    const uint32_t qn = q(N), qe = q(E), qs = q(S), qw = q(W);
    auto bright = [&](uint32_t x) { return __builtin_amdgcn_lerp(x, T.bright, 0u); };
    auto keep = [&](uint32_t x) { return __builtin_amdgcn_lerp(x, T.dark, 0u); };   // not darker
    const uint32_t bn = bright(qn), be = bright(qe), bs = bright(qs), bw = bright(qw);
    const uint32_t kn = keep(qn), ke = keep(qe), ks = keep(qs), kw = keep(qw);
    if constexpr (K == 1) return bn | be | bs | bw | ~(kn & ke & ks & kw);
    // adjacent pairs (N,E) (E,S) (S,W) (W,N): (N or S) and (E or W)
    if constexpr (K == 2) return ((bn | bs) & (be | bw)) | ~((kn & ks) | (ke & kw));
    // any 3 of the 4 are consecutive
    if constexpr (K == 3)
        return (bn & bs & (be | bw)) | (be & bw & (bn | bs)) | ~((kn | ks | (ke & kw)) & (ke | kw | (kn & ks)));
    return (bn & be & bs & bw) | ~(kn | ke | ks | kw);
}

// Circle of radius 3 (Section II-D) in cyclic order, as LDS byte offsets.
#define CIRC(j) (CDY[j] * LP + CDX[j])
// Offset of a pixel from the top-left corner of its circle's bounding box.
constexpr int CORNER = 3 * LP + 3;
constexpr int CDX[16] = {0, 1, 2, 3, 3, 3, 2, 1, 0, -1, -2, -3, -3, -3, -2, -1};
constexpr int CDY[16] = {-3, -3, -2, -1, 0, 1, 2, 3, 3, 3, 2, 1, 0, -1, -2, -3};

// Bits i .. i+n-1 (circularly, 0 <= i < 16) set for every bit i of `starts`
// (a 16-bit mask): the circle points covered by the arcs starting there.
__device__ __forceinline__ uint32_t arc_cover(uint32_t starts, int n) {
    uint32_t c = starts;
    int have = 1;
    while (have * 2 <= n) {
        c |= c << have;
        have *= 2;
    }
    if (have < n) c |= c << (n - have);
    return (c | (c >> 16)) & 0xFFFFu;
}

// w[i] <- min(w[i], w[(i + k) & 15]) for both 16-bit halves.
template <int K>
__device__ __forceinline__ void window_step(s16x2 (&w)[16]) {
    s16x2 u[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) u[i] = vmin(w[i], w[(i + K) & 15]);
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = u[i];
}

template <int K>
__device__ __forceinline__ void rotate(s16x2 (&w)[16]) {
    s16x2 u[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) u[i] = w[(i + K) & 15];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = u[i];
}

// Maximum-threshold score from the 16 circle values: the largest d such that
// n consecutive points all exceed the centre by at least d (low half: v - c)
// or fall below it by at least d (high half: c - v).  Window minima by
// doubling (uniform steps), the remainder by a barrel rotation, so every
// register index is static.
__device__ __forceinline__ int max_threshold(const uint32_t (&v)[16], uint32_t cv, int n) {
    s16x2 w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = s16x2{(short)((int)v[i] - (int)cv), (short)((int)cv - (int)v[i])};
    int have = 1;
    if (n >= 2) { window_step<1>(w); have = 2; }
    if (n >= 4) { window_step<2>(w); have = 4; }
    if (n >= 8) { window_step<4>(w); have = 8; }
    if (n >= 16) { window_step<8>(w); have = 16; }
    const int r = n - have;   // 0 <= r < have
    if (r) {
        s16x2 u[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) u[i] = w[i];
        if (r & 1) rotate<1>(u);
        if (r & 2) rotate<2>(u);
        if (r & 4) rotate<4>(u);
#pragma unroll
        for (int i = 0; i < 16; ++i) w[i] = vmin(w[i], u[i]);
    }
    s16x2 m = w[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) m = vmax(m, w[i]);
    return m.x > m.y ? m.x : m.y;
}

// Corner score kinds (Section II-D): FAST_SCORE_SADB sums over the whole
// circle, FAST_SCORE_SADA over the points on a qualifying arc, FAST_SCORE_MT
// is the maximum threshold at which the test still passes (plus one).
// Segment test and score of the pixel at p; 0 if the test fails.  The sums
// accumulate max(v - (c+t), 0) and max((c-t) - v, 0), each one saturating
// unsigned subtraction.
template <int KIND>
__device__ __forceinline__ uint32_t full_score(const uint8_t *p, int t, int n) {
    // every read is at a non-negative constant offset from the circle's
    // top-left corner, so all 17 share one address register
    const auto q = lds_base(p - CORNER);
    const uint32_t cv = q[CORNER];
    const uint32_t hi = cv + (uint32_t)t;
    const uint32_t lo = (int)cv - t > 0 ? cv - (uint32_t)t : 0u;   // darker needs v < c-t; none if c-t <= 0
    uint32_t v[16];
    uint32_t bm = 0, dm = 0, sb = 0, sd = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        v[j] = q[CORNER + CIRC(j)];
        bm = __builtin_amdgcn_alignbit(bm, hi - v[j], 31);   // sign: v > c+t; point j at bit 15-j
        dm = __builtin_amdgcn_alignbit(dm, v[j] - lo, 31);   // sign: v < c-t
    }
    if constexpr (KIND == FAST_SCORE_SADB) {
        // the sums in 16-bit lanes, points j and j+8 side by side: each lane
        // sums 8 terms of at most 255, so nothing saturates but the terms
        const u16x2 hi2 = {(unsigned short)hi, (unsigned short)hi}, lo2 = {(unsigned short)lo, (unsigned short)lo};
        u16x2 b2 = {0, 0}, d2 = {0, 0};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const u16x2 p = __builtin_bit_cast(u16x2, v[j] | (v[j + 8] << 16));
            b2 += __builtin_elementwise_sub_sat(p, hi2);
            d2 += __builtin_elementwise_sub_sat(lo2, p);
        }
        sb = (uint32_t)b2.x + b2.y;
        sd = (uint32_t)d2.x + d2.y;
    }
    const uint32_t b2 = bm | (bm << 16), d2 = dm | (dm << 16);
    const uint32_t rb = runs(b2, n) & 0xFFFFu, rd = runs(d2, n) & 0xFFFFu;
    if ((rb | rd) == 0) return 0;
    if constexpr (KIND == FAST_SCORE_MT) return (uint32_t)max_threshold(v, cv, n);
    if constexpr (KIND == FAST_SCORE_SADA) {
        if (n >= 9) {
            // only one side can have an arc: its circle is flipped where it is
            // the darker one (255 - v above 255 - lo instead of v below lo),
            // and the points on the arc are summed in 16-bit lanes, j and j+8
            // side by side, each term times its bit of the arc
            const uint32_t flip = rb ? 0u : 0x00FF00FFu;
            const uint32_t th = rb ? hi : 255u - lo;
            const u16x2 th2 = {(unsigned short)th, (unsigned short)th};
            const uint32_t arc = arc_cover(rb | rd, n);   // point j at bit 15-j
            const uint32_t on = (arc >> 8) | (arc & 0xFFu) << 16;   // j at bit 7-j, j+8 at bit 23-j
            u16x2 sum = {0, 0};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const u16x2 p = __builtin_bit_cast(u16x2, (v[j] | (v[j + 8] << 16)) ^ flip);
                const u16x2 bit = __builtin_bit_cast(u16x2, (on >> (7 - j)) & 0x00010001u);
                sum += __builtin_elementwise_sub_sat(p, th2) * bit;
            }
            return (uint32_t)sum.x + sum.y;
        }
        const uint32_t cb = arc_cover(rb, n), cd = arc_cover(rd, n);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            sb += __builtin_elementwise_sub_sat(v[j], hi) & (0u - ((cb >> (15 - j)) & 1u));
            sd += __builtin_elementwise_sub_sat(lo, v[j]) & (0u - ((cd >> (15 - j)) & 1u));
        }
    }
    return sb > sd ? sb : sd;
}

// One pyramid level of the current sub-tile as staged in LDS (uniform).
struct Geo {
    int tbase;           // LDS offset of tile (0,0)
    int tx, ty;          // level coordinates of tile (0,0)
    int W, H;            // level size
    int sx, sy, ex, ey;  // sub-tile area at this level (NMS targets), clipped
    int moff, mp;        // score map: LDS offset and pitch (u16) of [sx-1, ex+1) x [sy-1, ey+1)
    int gc0, ncolg;      // first group column (tile coords) and groups per row (even)
    int k;               // level index
};

struct Params {
    int t, n, kc, k8;    // threshold, arc length, floor(N/4), floor(N/2)
    int kind;            // corner score kind (FAST_SCORE_*)
    // score-map mode (smap[0] != null): the passes write each level's area
    // scores to smap[l] (pitch spitch[l] elements) instead of running NMS;
    // index l follows the levels handed to run_passes
    uint16_t *smap[3];
    int spitch[3];
    int cell;            // level-0 cell side
    int rx0, ry0;        // region origin in level-0 pixels
    int ncx;             // cells across the region
};

__device__ __forceinline__ void set_groups(Geo &g) {
    const int c_first = g.sx - 1 - g.tx;
    g.gc0 = c_first & ~3;
    g.ncolg = (g.ex + 1 - g.tx - g.gc0 + 3) >> 2;
    g.ncolg += g.ncolg & 1;   // whole pairs of groups
}

__device__ __forceinline__ bool has_area(const Geo &g) { return g.ex > g.sx && g.ey > g.sy; }

template <class T>
__device__ __forceinline__ T sel3(int l, T a, T b, T c) {
    return l == 0 ? a : (l == 1 ? b : c);
}

// Scored area of one level in a sub-tile: rows [r0, r0 + nrows) of the tile
// band, groups of 8 pixels from column gc0, ppr groups per row; pixels
// outside [c_lo, c_hi] x [r_lo, r_hi] (tile coordinates) are not testable.
struct Seg {
    int tbase, r0, nrows, gc0, ppr, n;   // n = nrows * ppr groups
    int c_lo, c_hi, r_lo, r_hi;
};

__device__ __forceinline__ Seg make_seg(const Geo &g, bool on) {
    Seg q;
    q.tbase = g.tbase;
    q.r0 = g.sy - 1 - g.ty;
    q.nrows = on ? g.ey - g.sy + 2 : 0;
    q.gc0 = g.gc0;
    q.ppr = g.ncolg >> 1;
    q.n = q.nrows * q.ppr;
    q.c_lo = max(g.sx - 1, 3) - g.tx;
    q.c_hi = min(g.ex, g.W - 4) - g.tx;
    q.r_lo = max(q.r0, 3 - g.ty);
    q.r_hi = min(q.r0 + q.nrows - 1, g.H - 4 - g.ty);
    return q;
}

// The groups of all levels of a sub-tile form one sequence: level 0's rows
// first, then level 1's, then level 2's.  A group's entry is the LDS offset of
// its first pixel | level << 14, or NO_GROUP past the end.
constexpr uint32_t NO_GROUP = 0xFFFFu;
// Any offset whose 8 pixels and compass points lie inside the tile; a lane
// with no group reads there and discards the result.
constexpr uint32_t SAFE_OFF = T0 + 3 * LP + 4;
static_assert(SAFE_OFF % 8 == 4, "aligned compass row reads at SAFE_OFF");

struct GroupSeq {
    int b1, b2, total;   // first group of level 1, of level 2; group count
};

__device__ __forceinline__ GroupSeq group_seq(const Seg &s0, const Seg &s1, const Seg &s2) {
    GroupSeq q;
    q.b1 = s0.n;
    q.b2 = s0.n + s1.n;
    q.total = s0.n + s1.n + s2.n;
    return q;
}

__device__ __forceinline__ uint32_t group_entry(const Seg &s0, const Seg &s1, const Seg &s2,
                                                const GroupSeq &q, int i) {
    const uint32_t lvl = i < q.b1 ? 0u : (i < q.b2 ? 1u : 2u);
    const int local = i - (lvl == 0 ? 0 : (lvl == 1 ? q.b1 : q.b2));
    const int ppr = max(sel3(lvl, s0.ppr, s1.ppr, s2.ppr), 1);
    // row = floor((local + 0.5) / ppr), exact with the approximate reciprocal
    // since local < 1024 and ppr <= 9
    const int row = (int)(((float)local + 0.5f) * __builtin_amdgcn_rcpf((float)ppr)), pp = local - row * ppr;
    const uint32_t off = (uint32_t)(sel3(lvl, s0.tbase, s1.tbase, s2.tbase) +
                                    (sel3(lvl, s0.r0, s1.r0, s2.r0) + row) * LP +
                                    sel3(lvl, s0.gc0, s1.gc0, s2.gc0) + 8 * pp);
    return i < q.total ? off | (lvl << 14) : NO_GROUP;
}

// Group entries of one lane for the (at most four) compass rounds it takes
// when four or more waves share a sub-tile, two 16-bit entries per word.
// Regions of the same staged geometry have the same entries (all whole ones
// do), so the pipelined kernels keep them.
struct GroupCache {
    uint32_t e01, e23;
};

// The words a compass test of 8 pixels reads: the 16 bytes around the group
// on its own row (4 before, 4 after) and 8 bytes three rows above and below.
// With A8 every group starts 4 bytes past a multiple of 8 (see the tile
// layout), and the row is read as two aligned 8-byte words.
struct Px8 {
    uint32_t D0, D1, D2, D3, N0, N1, S0, S1;
};

template <bool A8>
__device__ __forceinline__ Px8 load8(const uint8_t *smem, uint32_t off) {
    // every read at a non-negative offset from the word 4 bytes before the
    // group's pixel three rows up
    const auto b = lds_base((const uint32_t *)(smem + off - 3 * LP - 4));
    constexpr int R3 = 3 * LP / 4;   // three rows, in words
    Px8 x;
    if constexpr (A8) {
        // b is 8-aligned here (LP and the group's offset - 4 are)
        const auto b2 = (const __attribute__((address_space(3))) u32x2 *)b;
        const u32x2 lo = b2[R3 / 2], hi = b2[R3 / 2 + 1];
        x.D0 = lo.x;
        x.D1 = lo.y;
        x.D2 = hi.x;
        x.D3 = hi.y;
    } else {
        x.D0 = b[R3];
        x.D1 = b[R3 + 1];
        x.D2 = b[R3 + 2];
        x.D3 = b[R3 + 3];
    }
    x.N0 = b[1];
    x.N1 = b[2];
    x.S0 = b[2 * R3 + 1];
    x.S1 = b[2 * R3 + 2];
    return x;
}

// Compass test of the 8 pixels of x: bit j <- pixel j (set = may be a corner).
// 45 instructions; unpacked to 16-bit lanes, two pixels each, it took 71.
template <int K>
__device__ __forceinline__ uint32_t compass8(const Px8 &x, const CompassT &T) {
    if constexpr (K > 0) {
        auto east = [](uint32_t hi, uint32_t lo) { return __builtin_amdgcn_alignbyte(hi, lo, 3); };
        auto west = [](uint32_t hi, uint32_t lo) { return __builtin_amdgcn_alignbyte(hi, lo, 1); };
        const uint32_t a = compass4<K>(x.D1, x.N0, east(x.D2, x.D1), x.S0, west(x.D1, x.D0), T);
        const uint32_t b = compass4<K>(x.D2, x.N1, east(x.D3, x.D2), x.S1, west(x.D2, x.D1), T);
        // bits 0 and 4 of byte j: pixels j and 4 + j; the dot product adds
        // byte j shifted by j
        const uint32_t m = ((a >> 7) & 0x01010101u) | ((b >> 3) & 0x10101010u);
        return __builtin_amdgcn_udot4(m, 0x08040201u, 0u, false);
    } else {
        return 0xFFu;
    }
}

// LDS offset a lane with entry e reads (a safe one for NO_GROUP).
__device__ __forceinline__ uint32_t entry_off(uint32_t e) { return e != NO_GROUP ? (e & 0x3FFFu) : SAFE_OFF; }

// Bits b with lo <= b < hi (0 <= lo <= hi < 32).
__device__ __forceinline__ uint32_t bit_range(int lo, int hi) { return (1u << hi) - (1u << lo); }

// P1+P2: compass test of every scored pixel of every level, 8 pixels per
// lane.  The groups of all levels form one sequence
// dealt to the waves round-robin in rounds of 64, so every wave does the
// same share whatever the level sizes; a wave tests two rounds at a time so
// that the LDS reads of one overlap the arithmetic of the other.  Groups with
// a survivor are compacted into the wave's group list (ballot + mbcnt; word =
// level << 22 | LDS offset of the group << 8 | survivor mask), which is then
// expanded into the wave's pixel list, keeping testable pixels only; an entry
// is (level << 14) | LDS offset of the pixel.  Returns the wave's pixel count.
// With `cached` (four or more waves), the group entries are e01 and e23
// (GroupCache).
template <int K, bool A8>
__device__ int collect(const uint8_t *smem, const Seg &s0, const Seg &s1, const Seg &s2, int t,
                       bool cached, uint32_t e01, uint32_t e23, uint32_t *blist, uint16_t *list) {
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const GroupSeq q = group_seq(s0, s1, s2);
    const CompassT T1 = compass_t(t);
    const int stride = nwaves * 64;
    int nb = 0;
    // survivors go to nb + (survivors below the lane); the other lanes write
    // past them, inside the round's own 64 words, where a later round
    // overwrites them, so the stores need no branch
    auto push = [&](uint32_t e, uint32_t sv) {
        const uint64_t bal = __ballot(sv != 0);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        const int cnt = __popcll(bal);
        blist[sv ? nb + rank : nb + cnt + lane - rank] = (e << 8) | sv;
        nb += cnt;
    };
    for (int r = 0;; r += 2) {
        const int i0 = wave * 64 + r * stride;
        if (i0 >= q.total) break;
        uint32_t ea, eb;
        if (cached) {
            const uint32_t w = r == 0 ? e01 : e23;
            ea = w & 0xFFFFu;
            eb = w >> 16;
        } else {
            ea = group_entry(s0, s1, s2, q, i0 + lane);
            eb = group_entry(s0, s1, s2, q, i0 + stride + lane);
        }
        const Px8 xa = load8<A8>(smem, entry_off(ea));
        if (i0 + stride < q.total) {
            // two rounds: both rounds' LDS reads are issued before either is
            // evaluated
            const Px8 xb = load8<A8>(smem, entry_off(eb));
            const uint32_t sva = compass8<K>(xa, T1) & (0u - (uint32_t)(ea != NO_GROUP));
            const uint32_t svb = compass8<K>(xb, T1) & (0u - (uint32_t)(eb != NO_GROUP));
            push(ea, sva);
            push(eb, svb);
        } else {
            push(ea, compass8<K>(xa, T1) & (0u - (uint32_t)(ea != NO_GROUP)));
        }
    }
    wave_sync();
    int count = 0;
    const int spare = list_cap(nwaves) + lane;
    for (int j0 = 0; j0 < nb; j0 += 64) {
        const int j = j0 + lane;
        const uint32_t w = j < nb ? blist[j] : 0u;
        const uint32_t l = w >> 22;
        const int off0 = (int)((w >> 8) & 0x3FFFu);
        const int rel = off0 - sel3(l, s0.tbase, s1.tbase, s2.tbase);
        const int r = (int)(((uint32_t)rel * 18725u) >> 21);   // rel / LP
        const int c0 = rel - r * LP;
        const bool row_ok = r >= sel3(l, s0.r_lo, s1.r_lo, s2.r_lo) && r <= sel3(l, s0.r_hi, s1.r_hi, s2.r_hi);
        // pixel p of the group (column c0 + p) is testable iff lo <= p < hi
        const int lo = min(max(sel3(l, s0.c_lo, s1.c_lo, s2.c_lo) - c0, 0), 8);
        const int hi = max(min(max(sel3(l, s0.c_hi, s1.c_hi, s2.c_hi) - c0 + 1, 0), 8), lo);
        const uint32_t valid = bit_range(lo, hi);
        const uint32_t m = row_ok ? (w & valid) : 0u;
        const int cnt = __builtin_popcount(m);
        const int incl = wave_scan(cnt);
        const int pos = count + incl - cnt;
        count += __builtin_amdgcn_readlane(incl, 63);
        const uint32_t base = (l << 14) | (uint32_t)off0;
        // a kept pixel goes to pos + (kept pixels before it); the others write
        // to the lane's spare slot, so the loop has no branches
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const int at = (m >> b) & 1u ? pos + __builtin_popcount(m & ((1u << b) - 1u)) : spare;
            list[at] = (uint16_t)(base + (uint32_t)b);
        }
    }
    return count;
}

// Entries of this lane's compass rounds when at least four waves share the
// sub-tile (at most four rounds: MAX_GROUPS <= 4 * 256); rounds past the last
// group are left out (uniform).
__device__ __forceinline__ void group_cache_fill(GroupCache &c, const Seg &s0, const Seg &s1, const Seg &s2) {
    const int lane = lane_id(), wave = threadIdx.x >> 6, stride = (blockDim.x >> 6) * 64;
    const GroupSeq q = group_seq(s0, s1, s2);
    const int i = wave * 64 + lane;
    c.e23 = NO_GROUP | (NO_GROUP << 16);
    c.e01 = group_entry(s0, s1, s2, q, i) | (NO_GROUP << 16);
    if (q.total > stride) c.e01 = (c.e01 & 0xFFFFu) | (group_entry(s0, s1, s2, q, i + stride) << 16);
    if (q.total > 2 * stride)
        c.e23 = group_entry(s0, s1, s2, q, i + 2 * stride) | (group_entry(s0, s1, s2, q, i + 3 * stride) << 16);
}
static_assert(MAX_GROUPS <= 4 * 256, "four compass rounds per wave with four or more waves");

__device__ __forceinline__ void group_cache_fill(GroupCache &c, const Geo &g0, const Geo &g1, const Geo &g2,
                                                 int nl) {
    group_cache_fill(c, make_seg(g0, has_area(g0)), make_seg(g1, nl > 1 && has_area(g1)),
                     make_seg(g2, nl > 2 && has_area(g2)));
}

// P3: keep entries that pass the 8-point test, compacted in place.  A lane
// past the end reads a stale slot (the list has a spare slot per lane beyond
// its capacity, and n1 <= capacity), tests the pixel at SAFE_OFF instead and
// is masked off; entries that fail go to the lane's spare slot.  The pass
// therefore has no branches.
__device__ int pass_even8(const uint8_t *smem, int t, int k8, uint16_t *list, int n1) {
    const int lane = lane_id();
    const int spare = list_cap(blockDim.x >> 6) + lane;
    int n2 = 0;
    for (int i0 = 0; i0 < n1; i0 += 64) {
        const int i = i0 + lane;
        const uint16_t e = list[i];
        const bool valid = i < n1 && e != NO_ENTRY;
        const auto q = lds_base(smem + (valid ? (e & 0x3FFFu) : SAFE_OFF) - CORNER);
        const int cv = q[CORNER];
        const int hi = cv + t, lo = cv - t;
        uint32_t bm = 0, dm = 0;
#pragma unroll
        for (int j = 0; j < 16; j += 2) {
            const int v = q[CORNER + CIRC(j)];
            bm = __builtin_amdgcn_alignbit(bm, (uint32_t)(hi - v), 31);
            dm = __builtin_amdgcn_alignbit(dm, (uint32_t)(v - lo), 31);
        }
        // bright arcs in bits 0-15, dark arcs in bits 16-31, each 8-point
        // mask doubled for the circular wrap: a run of k8 <= 8 starting at
        // bit 0-7 (16-23) stays below bit 15 (31)
        const uint32_t w = (bm | (dm << 16)) * 0x101u;
        const bool pass = valid && (k8 == 0 || (runs8(w, k8) & 0x00FF00FFu) != 0);
        const uint64_t bal = __ballot(pass);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        list[pass ? n2 + rank : spare] = e;
        n2 += __popcll(bal);
        wave_sync();
    }
    return n2;
}


// Row and column inside the LDS tile band of an entry's offset.
__device__ __forceinline__ void tile_rc(uint32_t off, int &row, int &col) {
    row = (int)((off * 18725u) >> 21);   // off / LP, exact for off < 16384
    col = (int)off - row * LP;
}

// Per-level constants for mapping an entry to its score map and cell.
struct LevelMap {
    int mbias;           // map index = row * MP + col + mbias (row, col in the tile band)
    int rlo, rhi;        // band rows of the sub-tile area: [rlo, rhi)
    int clo, chi;        // band columns of the sub-tile area: [clo, chi)
    int xo, yo;          // cell-relative position = (col + xo, row + yo)
    int cw;              // cell side at this level
    float inv_cw;        // ~1/cw: floor((v + 0.5) * inv_cw) = v / cw for 0 <= v < 2^12
};

__device__ __forceinline__ LevelMap level_map(const Geo &g, int band_row, int band_col, int ra,
                                             int rb, const Params &P) {
    LevelMap m;
    const int ybias = g.ty - band_row, xbias = g.tx - band_col;   // level y = row + ybias
    m.mbias = (g.moff >> 1) + (ybias - (g.sy - 1)) * g.mp + (xbias - (g.sx - 1));
    m.rlo = ra - ybias;
    m.rhi = rb - ybias;
    m.clo = g.sx - xbias;
    m.chi = g.ex - xbias;
    m.xo = xbias - (P.rx0 >> g.k);
    m.yo = ybias - (P.ry0 >> g.k);
    m.cw = P.cell >> g.k;
    m.inv_cw = __builtin_amdgcn_rcpf((float)max(m.cw, 1));
    return m;
}

// Write the scores of level g's sub-tile area from its LDS score map to a
// global map (row y at dst + y * pitch elements, rows at any even address),
// eight to a thread: one 16-byte store in place of eight of two bytes with an
// address each (score maps of a 1920x1080 frame, level-0 pass: 14.6 us before,
// 13.2 now).
typedef u32x4 __attribute__((aligned(2))) u32x4_at2;

__device__ void store_scores(const uint8_t *smem, const Geo &g, uint16_t *dst, int pitch) {
    const int w = g.ex - g.sx, h = g.ey - g.sy, nch = (w + 7) >> 3;
    if (w <= 0 || h <= 0) return;
    for (int i = threadIdx.x; i < nch * h; i += blockDim.x) {
        const int yy = div_small(i, nch), xx = 8 * (i - yy * nch);
        // map columns xx .. xx+9, of which xx+1 .. xx+8 are wanted
        const uint8_t *m = smem + g.moff + ((yy + 1) * MP + xx) * 2;
        const u32x2 a = *(const u32x2 *)m, b = *(const u32x2 *)(m + 8);
        const uint32_t c = *(const uint32_t *)(m + 16);
        const u32x4 v = {__builtin_amdgcn_alignbit(a.y, a.x, 16), __builtin_amdgcn_alignbit(b.x, a.y, 16),
                         __builtin_amdgcn_alignbit(b.y, b.x, 16), __builtin_amdgcn_alignbit(c, b.y, 16)};
        uint16_t *d = dst + (ptrdiff_t)(g.sy + yy) * pitch + (g.sx + xx);
        if (xx + 8 <= w) {
            *(GLOBAL u32x4_at2 *)d = v;
        } else {
            const uint16_t *s = (const uint16_t *)m + 1;
            for (int e = 0; e < w - xx; ++e) gstore<uint16_t>(d + e, s[e]);
        }
    }
}
static_assert(OFF_M0 % 8 == 0 && OFF_M1 % 8 == 0 && OFF_M2 % 8 == 0 && MP * 2 % 8 == 0, "8-byte map reads");

// A staged sub-tile for the passes: its levels' scored areas, and whether every
// level's groups start 4 bytes past a multiple of 8 (uniform): true for fused
// sub-tiles, whose origins are on the 16-pixel grid; the levels of an upper
// region may start elsewhere.
struct Segs {
    Seg s0, s1, s2;
    bool a8;
};

// The levels' score maps and cells.
struct Maps {
    LevelMap m0, m1, m2;
};

__device__ __forceinline__ Segs segs_of(const Geo &g0, const Geo &g1, const Geo &g2, int nl) {
    Segs s;
    s.s0 = make_seg(g0, has_area(g0));
    s.s1 = make_seg(g1, nl > 1 && has_area(g1));
    s.s2 = make_seg(g2, nl > 2 && has_area(g2));
    s.a8 = ((s.s0.tbase + s.s0.gc0) & 7) == 4 && (!s.s1.n || ((s.s1.tbase + s.s1.gc0) & 7) == 4) &&
           (!s.s2.n || ((s.s2.tbase + s.s2.gc0) & 7) == 4);
    return s;
}

__device__ __forceinline__ Maps maps_of(const Geo &g0, const Geo &g1, const Geo &g2, const Params &P) {
    Maps m;
    m.m0 = level_map(g0, 0, T0, g0.sy, g0.ey, P);
    m.m1 = level_map(g1, 96, T1 - 96 * LP, g1.sy, g1.ey, P);
    m.m2 = level_map(g2, 96, T2 - 96 * LP, g2.sy, g2.ey, P);
    return m;
}

// The wave's lists.
__device__ __forceinline__ uint32_t *group_list(uint8_t *smem) {
    return (uint32_t *)(smem + OFF_WAVES + (threadIdx.x >> 6) * wave_bytes(blockDim.x >> 6));
}
__device__ __forceinline__ uint16_t *pixel_list(uint8_t *smem) {
    return (uint16_t *)((uint8_t *)group_list(smem) + blist_cap(blockDim.x >> 6) * 4);
}

// P1-P4 of a staged sub-tile whose score maps are zero, on every wave without
// workgroup barriers: scores into the maps; the wave's scored pixels stay in
// its list.  Returns their count.  With `cached` (workgroups of four or more
// waves) the wave's group entries are e01 and e23 (GroupCache).
__device__ __forceinline__ int score_phase(uint8_t *smem, const Segs &S, const Maps &M, const Params &P, bool cached,
                                           uint32_t e01, uint32_t e23) {
    uint32_t *blist = group_list(smem);
    uint16_t *list = pixel_list(smem);
    int n1 = 0;
    auto run_collect = [&](auto aligned) {
        constexpr bool A = decltype(aligned)::value;
        switch (P.kc) {
            case 0: n1 = collect<0, A>(smem, S.s0, S.s1, S.s2, P.t, cached, e01, e23, blist, list); break;
            case 1: n1 = collect<1, A>(smem, S.s0, S.s1, S.s2, P.t, cached, e01, e23, blist, list); break;
            case 2: n1 = collect<2, A>(smem, S.s0, S.s1, S.s2, P.t, cached, e01, e23, blist, list); break;
            case 3: n1 = collect<3, A>(smem, S.s0, S.s1, S.s2, P.t, cached, e01, e23, blist, list); break;
            default: n1 = collect<4, A>(smem, S.s0, S.s1, S.s2, P.t, cached, e01, e23, blist, list); break;
        }
    };
    if (S.a8)
        run_collect(std::true_type());
    else
        run_collect(std::false_type());
    wave_sync();
    // the later passes run at a raised wave priority: a wave that is further
    // through its sub-tile issues first, so workgroups reach their barriers
    // sooner (the waves sharing a SIMD belong to different workgroups)
    __builtin_amdgcn_s_setprio(1);
    // a wave with one round of survivors scores them at once: the 8-point test
    // would take a round of its own and save none (1920x1080 20.15 -> 19.97 us,
    // 4096x2160 39.4 -> 39.0, the 64-frame batch 102.7 -> 101.6; with two rounds
    // it saves more than it takes: 39.6 and 102.6 us)
    const int n2 = n1 <= 64 ? n1 : pass_even8(smem, P.t, P.k8, list, n1);
    uint16_t *maps = (uint16_t *)smem;
    const int lane = lane_id();
    // P4: full segment test and score into the level's score map (one loop
    // per score kind, so each compiles to straight-line code)
    auto score_pass = [&](auto kind) {
        for (int i = lane; i < n2; i += 64) {
            const uint16_t e = list[i];
            const uint32_t s = full_score<decltype(kind)::value>(smem + (e & 0x3FFF), P.t, P.n);
            if (s) {
                const int l = e >> 14;
                int row, col;
                tile_rc(e & 0x3FFF, row, col);
                maps[row * MP + col + sel3(l, M.m0.mbias, M.m1.mbias, M.m2.mbias)] = (uint16_t)s;
            }
        }
    };
    switch (P.kind) {
        case FAST_SCORE_SADA: score_pass(std::integral_constant<int, FAST_SCORE_SADA>()); break;
        case FAST_SCORE_MT: score_pass(std::integral_constant<int, FAST_SCORE_MT>()); break;
        default: score_pass(std::integral_constant<int, FAST_SCORE_SADB>()); break;
    }
    return n2;
}

// P5 after the workgroup's scores are complete: 3x3 NMS of the sub-tile's own
// pixels among the wave's n2 listed ones, then the cell keys.  A lane issues
// its nine score reads together, so the test costs one LDS round trip; a ring
// pixel (its own sub-tile suppresses it) reads around a fixed entry of the
// level-0 map instead and is masked off.  k0: the first level.
__device__ __forceinline__ void nms_phase(uint8_t *smem, const Maps &M, int k0, int ncx, uint32_t *keys, int n2) {
    const uint16_t *list = pixel_list(smem);
    const uint16_t *maps = (const uint16_t *)smem;
    const LevelMap &m0 = M.m0, &m1 = M.m1, &m2 = M.m2;
    for (int i = lane_id(); i < n2; i += 64) {
        const uint16_t e = list[i];
        const int l = e >> 14;
        int row, col;
        tile_rc(e & 0x3FFF, row, col);
        const bool own = (row >= sel3(l, m0.rlo, m1.rlo, m2.rlo)) & (row < sel3(l, m0.rhi, m1.rhi, m2.rhi)) &
                         (col >= sel3(l, m0.clo, m1.clo, m2.clo)) & (col < sel3(l, m0.chi, m1.chi, m2.chi));
        constexpr int mp = MP;
        // q: the upper-left neighbour
        const auto q = lds_base(maps + (own ? row * mp + col + sel3(l, m0.mbias, m1.mbias, m2.mbias) : OFF_M0 / 2 + mp + 1) -
                                mp - 1);
        const uint32_t s = q[mp + 1];
        // earlier neighbours in row-major order must be strictly lower,
        // later ones lower or equal
        const uint32_t earlier = max(max((uint32_t)q[0], (uint32_t)q[1]), max((uint32_t)q[2], (uint32_t)q[mp]));
        const uint32_t later =
            max(max((uint32_t)q[mp + 2], (uint32_t)q[2 * mp]), max((uint32_t)q[2 * mp + 1], (uint32_t)q[2 * mp + 2]));
        if (!(own & (s != 0) & (s > earlier) & (s >= later))) continue;
        const int cw = sel3(l, m0.cw, m1.cw, m2.cw);
        const int ox = col + sel3(l, m0.xo, m1.xo, m2.xo);
        const int oy = row + sel3(l, m0.yo, m1.yo, m2.yo);
        // exact: v + 0.5 is at least 0.5 / cw from a multiple of cw, far above
        // the error of the approximate reciprocal for v < 2^12
        const float inv = sel3(l, m0.inv_cw, m1.inv_cw, m2.inv_cw);
        const int cy = (int)(((float)oy + 0.5f) * inv), cx = (int)(((float)ox + 0.5f) * inv);
        const uint32_t local = (uint32_t)((oy - cy * cw) * cw + (ox - cx * cw));
        const uint32_t key = (s << 19) | ((uint32_t)(7 - (k0 + l)) << 16) | (0xFFFFu - local);
        atomicMax(&keys[cy * ncx + cx], key);
    }
    __builtin_amdgcn_s_setprio(0);
}

// The sub-tile's own scores to the global maps (P.smap).
__device__ __forceinline__ void store_maps(const uint8_t *smem, const Geo &g0, const Geo &g1, const Geo &g2, int nl,
                                           const Params &P) {
    store_scores(smem, g0, P.smap[0], P.spitch[0]);
    if (nl > 1) store_scores(smem, g1, P.smap[1], P.spitch[1]);
    if (nl > 2) store_scores(smem, g2, P.smap[2], P.spitch[2]);
    __builtin_amdgcn_s_setprio(0);
}

// Detect levels g0..g(nl-1) of the staged sub-tile (score maps zeroed) and fold
// the survivors into the region's cell keys, or write its scores to the global
// maps (P.smap).  One barrier makes all scores visible before NMS.  With `cached`
// (workgroups of four or more waves only) `cache` holds the group entries, filled
// by the caller; a value, since a pointer that may be null keeps it in memory.
__device__ void run_passes(uint8_t *smem, const Geo &g0, const Geo &g1, const Geo &g2, int nl, const Params &P,
                           uint32_t *keys, bool cached = false, GroupCache cache = GroupCache{0u, 0u}) {
    const Segs S = segs_of(g0, g1, g2, nl);
    const Maps M = maps_of(g0, g1, g2, P);
    const int n2 = score_phase(smem, S, M, P, cached, cache.e01, cache.e23);
    __syncthreads();   // every level's scores, ring included, are in the maps
    if (P.smap[0]) {   // score-map mode
        store_maps(smem, g0, g1, g2, nl, P);
        return;
    }
    nms_phase(smem, M, g0.k, P.ncx, keys, n2);
}

// The passes of a whole region of SIDE x SIDE pixels with NL levels, which most
// regions of a frame are: everything but the testable columns and rows (the
// region may lie at the frame's edge) and the cell side is a constant, which
// takes the set-up of the general case, and the scalar registers that hold it,
// off every region's path.  With it, and with items that name a region by its
// place, a region of the 64-frame batch takes 456 scalar instructions a wave where
// it took about 930 (98.6 -> 86.6 us when both came).
// (rx0, ry0): the region's origin; W, H: level 0.
template <int SIDE, int NL>
struct Whole {
    static constexpr int HALO = 4 << (NL - 1);   // the tile starts at the origin less (HALO + 15) & ~15 across
    static constexpr int LEFT = (HALO + 15) & ~15;

    // Level l < NL, in tile coordinates.
    static constexpr Geo geo(int l) {
        Geo g{};
        g.tbase = l == 0 ? T0 : (l == 1 ? T1 : T2);
        g.sx = LEFT >> l;
        g.sy = HALO >> l;
        g.ex = g.sx + (SIDE >> l);
        g.ey = g.sy + (SIDE >> l);
        g.moff = l == 0 ? OFF_M0 : (l == 1 ? OFF_M1 : OFF_M2);
        g.mp = MP;
        g.k = l;
        g.gc0 = (g.sx - 1) & ~3;
        g.ncolg = (g.ex + 1 - g.gc0 + 3) >> 2;
        g.ncolg += g.ncolg & 1;
        return g;
    }
    static_assert(((T0 + geo(0).gc0) & 7) == 4 && ((T1 + geo(1).gc0) & 7) == 4 && ((T2 + geo(2).gc0) & 7) == 4,
                  "aligned compass row reads");

    static __device__ __forceinline__ Seg seg(int l, int rx0, int ry0, int W, int H) {
        const Geo g = geo(l);
        Seg q;
        q.tbase = g.tbase;
        q.r0 = g.sy - 1;
        q.nrows = l < NL ? g.ey - g.sy + 2 : 0;
        q.gc0 = g.gc0;
        q.ppr = g.ncolg >> 1;
        q.n = q.nrows * q.ppr;
        const int tx = (rx0 - LEFT) >> l, ty = (ry0 - HALO) >> l;
        q.c_lo = max(g.sx - 1, 3 - tx);
        q.c_hi = min(g.ex, (W >> l) - 4 - tx);
        q.r_lo = max(q.r0, 3 - ty);
        q.r_hi = min(q.r0 + q.nrows - 1, (H >> l) - 4 - ty);
        return q;
    }
    static __device__ __forceinline__ Segs segs(int rx0, int ry0, int W, int H) {
        return Segs{seg(0, rx0, ry0, W, H), seg(1, rx0, ry0, W, H), seg(2, rx0, ry0, W, H), true};
    }
    static __device__ __forceinline__ void fill(GroupCache &c) {
        group_cache_fill(c, seg(0, 0, 0, 0, 0), seg(1, 0, 0, 0, 0), seg(2, 0, 0, 0, 0));
    }

    static __device__ __forceinline__ LevelMap map(int l, int cell) {
        const Geo g = geo(l);
        const int row0 = l == 0 ? 0 : 96, col0 = g.tbase - row0 * LP;   // the tile's corner in its band
        LevelMap m;
        m.mbias = (g.moff >> 1) + (1 - g.sy - row0) * MP + 1 - g.sx - col0;
        m.rlo = g.sy + row0;
        m.rhi = g.ey + row0;
        m.clo = g.sx + col0;
        m.chi = g.ex + col0;
        m.xo = -g.sx - col0;
        m.yo = -g.sy - row0;
        m.cw = cell >> l;
        m.inv_cw = __builtin_amdgcn_rcpf((float)max(m.cw, 1));
        return m;
    }
    static __device__ __forceinline__ Maps maps(int cell) { return Maps{map(0, cell), map(1, cell), map(2, cell)}; }

    // Whether region R of J is one (R's origin is a multiple of 16).
    template <class Region>
    static __device__ __forceinline__ bool is(const fg_job &J, const Region &R) {
        return R.xr1 - R.P.rx0 == SIDE && R.yr1 - R.P.ry0 == SIDE && min(J.levels, MAX_FUSED) == NL;
    }
};

// Stage level pixels [tx, tx+tw) x [ty, ty+th) into an LDS tile with 16-byte
// loads (tx % 16 == 0, so no chunk straddles the pitch; tw <= 128).  Chunks
// outside the plane are zero and never used as pixel values.  Thread i owns
// chunk column i % 8 of rows i/8 + j * (block/8); the first four of its rows
// are loaded into registers (TileRegs) before any store.
struct TileRegs {
    u32x4 v[4];
};

__device__ __forceinline__ void tile_issue(TileRegs &R, const uint8_t *img, int H, int P, int tx, int ty,
                                           int tw, int th) {
    const int ch = threadIdx.x & 7;
    const int gx = tx + 16 * ch;
    const bool col_ok = ch < (tw >> 4) && gx >= 0 && gx < P;
    const int r0 = threadIdx.x >> 3, dr = blockDim.x >> 3;
    // row pointers advance by a uniform stride: one 64-bit multiply per thread
    const uint8_t *row = img + (ptrdiff_t)(ty + r0) * P + gx;
    const ptrdiff_t step = (ptrdiff_t)dr * P;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = r0 + j * dr, gy = ty + r;
        R.v[j] = u32x4{0u, 0u, 0u, 0u};
        if (r < th && col_ok && gy >= 0 && gy < H) R.v[j] = gload<u32x4>(row);
        row += step;
    }
}

__device__ __forceinline__ void tile_commit(uint8_t *tile, const TileRegs &R, int tw, int th) {
    const int ch = threadIdx.x & 7;
    if (ch >= (tw >> 4)) return;
    const int r0 = threadIdx.x >> 3, dr = blockDim.x >> 3;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = r0 + j * dr;
        if (r < th) *(u32x4 *)(tile + r * LP + 16 * ch) = R.v[j];
    }
}

__device__ void load_tile(uint8_t *tile, const uint8_t *img, int H, int P, int tx, int ty, int tw,
                          int th) {
    TileRegs R;
    tile_issue(R, img, H, P, tx, ty, tw, th);
    tile_commit(tile, R, tw, th);
    const int ch = threadIdx.x & 7;
    if (ch >= (tw >> 4)) return;
    const int gx = tx + 16 * ch;
    const bool col_ok = gx >= 0 && gx < P;
    const int dr = blockDim.x >> 3;
    for (int r = (threadIdx.x >> 3) + 4 * dr; r < th; r += dr) {   // small workgroups only
        const int gy = ty + r;
        u32x4 w = u32x4{0u, 0u, 0u, 0u};
        if (col_ok && gy >= 0 && gy < H) w = gload<u32x4>(img + (size_t)gy * P + gx);
        *(u32x4 *)(tile + r * LP + 16 * ch) = w;
    }
}

// Four pyramid pixels from two rows of eight: (a+b+c+d+2)>>2 per 2x2 block.
// Bytes 0, 2 and bytes 1, 3 of each word go to 16-bit lanes with one v_perm
// each; a block's sum is at most 4 * 255 + 2, so no lane carries into the
// next.  After the shift by 2 each lane's result is its low byte (the bits
// shifted in from the lane above land in the byte the final v_perm skips).
__device__ __forceinline__ uint32_t halve4(uint2 a, uint2 b) {
    auto even = [](uint32_t x) { return __builtin_amdgcn_perm(0u, x, 0x0c020c00u); };
    auto odd = [](uint32_t x) { return __builtin_amdgcn_perm(0u, x, 0x0c030c01u); };
    const uint32_t s0 = even(a.x) + odd(a.x) + even(b.x) + odd(b.x) + 0x00020002u;
    const uint32_t s1 = even(a.y) + odd(a.y) + even(b.y) + odd(b.y) + 0x00020002u;
    return __builtin_amdgcn_perm(s1 >> 2, s0 >> 2, 0x06040200u);
}

// Levels 1 and 2 of a fused tile in one pass (tw a multiple of 16): a task
// reads a 16 x 4 block of level 0 and writes the 8 x 2 level-1 block and the
// 4 x 1 level-2 block it covers, each by successive (a+b+c+d+2)>>2 rounding.
// With an odd number of level-1 rows the last one has tasks of its own.
__device__ void halve_two(const uint8_t *l0, uint8_t *l1, uint8_t *l2, int tw, int th, bool need_l2) {
    const int wpr = tw >> 4, rows2 = th >> 2;
    const int tasks = wpr * rows2 + (((th >> 1) & 1) ? wpr : 0);
    for (int i = threadIdx.x; i < tasks; i += blockDim.x) {
        const int y2 = div_small(i, wpr), x4 = i - y2 * wpr;
        const uint8_t *s = l0 + (4 * y2) * LP + 16 * x4;
        if (y2 < rows2) {
            const u32x4 a = *(const u32x4 *)s, b = *(const u32x4 *)(s + LP);
            const u32x4 c = *(const u32x4 *)(s + 2 * LP), d = *(const u32x4 *)(s + 3 * LP);
            const uint32_t r0a = halve4(make_uint2(a.x, a.y), make_uint2(b.x, b.y));
            const uint32_t r0b = halve4(make_uint2(a.z, a.w), make_uint2(b.z, b.w));
            const uint32_t r1a = halve4(make_uint2(c.x, c.y), make_uint2(d.x, d.y));
            const uint32_t r1b = halve4(make_uint2(c.z, c.w), make_uint2(d.z, d.w));
            *(uint2 *)(l1 + (2 * y2) * LP + 8 * x4) = make_uint2(r0a, r0b);
            *(uint2 *)(l1 + (2 * y2 + 1) * LP + 8 * x4) = make_uint2(r1a, r1b);
            if (need_l2) *(uint32_t *)(l2 + y2 * LP + 4 * x4) = halve4(make_uint2(r0a, r0b), make_uint2(r1a, r1b));
        } else {
            // last level-1 row, 2 * rows2, from level-0 rows 4 * rows2 and 4 * rows2 + 1
            const u32x4 a = *(const u32x4 *)s, b = *(const u32x4 *)(s + LP);
            *(uint2 *)(l1 + (2 * y2) * LP + 8 * x4) =
                make_uint2(halve4(make_uint2(a.x, a.y), make_uint2(b.x, b.y)),
                           halve4(make_uint2(a.z, a.w), make_uint2(b.z, b.w)));
        }
    }
}

// Copy the sub-tile's own pixels of an LDS level to the pyramid plane
// (sx % 4 == 0, ex - sx <= 32).  The last word of a row is written byte by
// byte when it would cross the level width.
__device__ void store_level(const uint8_t *tile, int tx, int ty, uint8_t *img, int P, int sx, int sy,
                            int ex, int ey) {
    const int w = threadIdx.x & 7;               // 8 word slots per row
    const int x = sx + 4 * w;
    if (x >= ex) return;
    for (int y = sy + (threadIdx.x >> 3); y < ey; y += blockDim.x >> 3) {
        const uint8_t *s = tile + (y - ty) * LP + (x - tx);
        uint8_t *d = img + (size_t)y * P + x;
        if (x + 4 <= ex) {
            gstore<uint32_t>(d, *(const uint32_t *)s);
        } else {
            for (int q = 0; q < ex - x; ++q) gstore<uint8_t>(d + q, s[q]);
        }
    }
}

// Zero [p, p+bytes) with 16-byte stores (p and bytes multiples of 16).
__device__ void zero_lds(uint8_t *p, int bytes) {
    for (int i = threadIdx.x; i < (bytes >> 4); i += blockDim.x) ((uint4 *)p)[i] = make_uint4(0, 0, 0, 0);
}

// Level-k area of the level-0 sub-tile at (sx0, sy0), clipped to the region
// end (xr1, yr1 at level 0) and the level size.
__device__ __forceinline__ void level_area(const fg_job &J, int k, int sx0, int sy0, int xr1,
                                           int yr1, Geo &g) {
    g.k = k;
    g.W = J.w[k];
    g.H = J.h[k];
    g.sx = sx0 >> k;
    g.sy = sy0 >> k;
    g.ex = min(min((sx0 + SUB) >> k, xr1 >> k), g.W);
    g.ey = min(min((sy0 + SUB) >> k, yr1 >> k), g.H);
}

// Levels 0 .. fused_levels(J)-1 are detected from one level-0 load; levels
// beyond (jobs with more than MAX_FUSED levels) are detected afterwards by
// the upper-level pass.
__device__ __forceinline__ int fused_levels(const fg_job &J) { return min(J.levels, MAX_FUSED); }

// Level-0 tile of a fused sub-tile: the sub-tile plus a 4*2^(F-1) halo (F
// fused levels), with the left edge rounded down to 16 pixels.
struct Stage {
    int tx, ty, tw, th;
};

__device__ __forceinline__ Stage fused_stage(const fg_job &J, int sx0, int sy0, int xr1, int yr1) {
    const int H0 = 4 << (fused_levels(J) - 1);
    Stage st;
    st.tx = (sx0 - H0) & ~15;
    st.ty = sy0 - H0;
    st.tw = ((min(sx0 + SUB, xr1) + H0 + 15) & ~15) - st.tx;
    st.th = min(sy0 + SUB, yr1) + H0 - st.ty;
    return st;
}

// Describe levels 0 .. F-1 of a fused sub-tile staged as `st`.
__device__ void describe_fused(const fg_job &J, int sx0, int sy0, int xr1, int yr1, const Stage &st, Geo &g0,
                               Geo &g1, Geo &g2) {
    level_area(J, 0, sx0, sy0, xr1, yr1, g0);
    g0.tbase = T0;
    g0.tx = st.tx;
    g0.ty = st.ty;
    g0.moff = OFF_M0;
    g0.mp = MP;
    set_groups(g0);
    g1 = g0;
    g2 = g0;
    const int nl = fused_levels(J);
    if (nl > 1) {
        level_area(J, 1, sx0, sy0, xr1, yr1, g1);
        g1.tbase = T1;
        g1.tx = st.tx >> 1;
        g1.ty = st.ty >> 1;
        g1.moff = OFF_M1;
        g1.mp = MP;
        set_groups(g1);
    }
    if (nl > 2) {
        level_area(J, 2, sx0, sy0, xr1, yr1, g2);
        g2.tbase = T2;
        g2.tx = st.tx >> 2;
        g2.ty = st.ty >> 2;
        g2.moff = OFF_M2;
        g2.mp = MP;
        set_groups(g2);
    }
}

// With level 0 of a fused sub-tile in LDS: build levels 1.. in LDS, describe
// every level, and write levels 1.. of the sub-tile to their planes.
__device__ void build_fused(const fg_job &J, int sx0, int sy0, int xr1, int yr1, const Stage &st,
                            uint8_t *smem, Geo &g0, Geo &g1, Geo &g2) {
    describe_fused(J, sx0, sy0, xr1, yr1, st, g0, g1, g2);
    const int nl = fused_levels(J);
    if (nl > 1) {
        __syncthreads();
        halve_two(smem + T0, smem + T1, smem + T2, st.tw, st.th, nl > 2);
    }
    __syncthreads();
    if (nl > 1 && has_area(g1))
        store_level(smem + T1, g1.tx, g1.ty, J.lvl[1], J.pitch[1], g1.sx, g1.sy, g1.ex, g1.ey);
    if (nl > 2 && has_area(g2))
        store_level(smem + T2, g2.tx, g2.ty, J.lvl[2], J.pitch[2], g2.sx, g2.sy, g2.ex, g2.ey);
}

// One level-0 sub-tile of a region: stage levels 0 .. F-1, detect, fold into
// keys.
__device__ void process_subtile(const fg_job &J, int sx0, int sy0, int xr1, int yr1,
                                const Params &P, uint8_t *smem) {
    // one load with a 4*2^(F-1) halo; levels 1 .. F-1 built in LDS
    const Stage st = fused_stage(J, sx0, sy0, xr1, yr1);
    __syncthreads();
    load_tile(smem + T0, J.lvl[0], J.h[0], J.pitch[0], st.tx, st.ty, st.tw, st.th);
    zero_lds(smem + OFF_M0, OFF_KEYS - OFF_M0);
    Geo g0, g1, g2;
    build_fused(J, sx0, sy0, xr1, yr1, st, smem, g0, g1, g2);
    run_passes(smem, g0, g1, g2, fused_levels(J), P, (uint32_t *)(smem + OFF_KEYS));
}

// A region of a job: its cells and its level-0 extent.
struct Region {
    int rxi, ryi;        // region column and row
    int rcells;          // cells per region side
    int ncx, ncy;        // cells across and down (clipped at the grid edge)
    int xr1, yr1;        // level-0 end of the region (clipped at the image)
    Params P;
};

// The region in column rxi and row ryi of a job's regions; `whole`: it is known
// not to be clipped.
__device__ __forceinline__ Region region_at(const fg_job &J, int rxi, int ryi, bool whole = false) {
    Region R;
    R.rxi = rxi;
    R.ryi = ryi;
    R.rcells = J.rcells;
    R.P.t = J.t;
    R.P.n = J.n;
    R.P.kind = J.score;
    R.P.smap[0] = R.P.smap[1] = R.P.smap[2] = nullptr;
    R.P.spitch[0] = R.P.spitch[1] = R.P.spitch[2] = 0;
    R.P.kc = J.n >> 2;
    R.P.k8 = J.n >> 1;
    R.P.cell = J.cell;
    if (whole) {   // FG_WHOLE
        R.ncx = R.ncy = J.rcells;
        R.P.rx0 = rxi * SUB;
        R.P.ry0 = ryi * SUB;
        R.xr1 = R.P.rx0 + SUB;
        R.yr1 = R.P.ry0 + SUB;
    } else {
        R.ncx = min(J.rcells, J.gw - rxi * J.rcells);
        R.ncy = min(J.rcells, J.gh - ryi * J.rcells);
        R.P.rx0 = rxi * J.rcells * J.cell;
        R.P.ry0 = ryi * J.rcells * J.cell;
        R.xr1 = min(R.P.rx0 + R.ncx * J.cell, J.w[0]);
        R.yr1 = min(R.P.ry0 + R.ncy * J.cell, J.h[0]);
    }
    R.P.ncx = R.ncx;
    return R;
}

__device__ __forceinline__ Region item_region(const fg_job &J, uint32_t code) {
    return region_at(J, (int)(code & (FG_WHOLE - 1)), (int)(code >> 16));
}
// The region of an item for the general passes, its column (and with VROW its row)
// in a vector register, and with it what follows from it: of the general set-up's
// hundred words that are the same in every lane, more are spilled and reloaded lane
// by lane in the passes when all compete for the scalar registers.  Tile loads and
// commits take item_region: vector coordinates lengthen their chains (16 frames of
// 752x480, SAD-A, N = 12: 26.2 us, 27.0 with them there too).
template <bool VROW>
__device__ __forceinline__ Region general_region(const fg_job &J, uint32_t code) {
    int column = (int)(code & (FG_WHOLE - 1)), row = (int)(code >> 16);
    asm("" : "+v"(column));
    if (VROW) asm("" : "+v"(row));
    return region_at(J, column, row);
}
__device__ __forceinline__ Region whole_region(const fg_job &J, uint32_t code) {
    return region_at(J, (int)(code & (FG_WHOLE - 1)), (int)(code >> 16), true);
}

// A job's regions in row-major order.
__device__ __forceinline__ Region region_of(const fg_job &J, int region) {
    const int ryi = region < (1 << 21) ? div_small(region, J.rx) : region / J.rx;
    return region_at(J, region - ryi * J.rx, ryi);
}

__device__ __forceinline__ void keys_clear(uint32_t *keys, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) keys[i] = 0;
}

// Decode the region's cell keys into output slots.
__device__ void keys_write(const fg_job &J, const Region &R, const uint32_t *keys, int tid = threadIdx.x,
                           int nthreads = blockDim.x) {
    for (int i = tid; i < R.ncx * R.ncy; i += nthreads) {
        const int qy = div_small(i, R.ncx);   // i < MAX_KEYS
        const int cx = R.rxi * R.rcells + i - qy * R.ncx, cy = R.ryi * R.rcells + qy;
        const uint32_t key = keys[i];
        // fast_feature {x, y, score, level, reserved} as one little-endian word
        uint64_t f;
        if (key == 0) {
            f = 0x00FF0000FFFFFFFFull;
        } else {
            const int level = 7 - (int)((key >> 16) & 7u);
            const uint32_t local = 0xFFFFu - (key & 0xFFFFu);
            const int cw = J.cell >> level;
            const int ly = div_small((int)local, cw);   // local < cw * cw <= 2^16
            const uint32_t x = (uint32_t)(((cx * J.cell) >> level) + (int)local - ly * cw);
            const uint32_t y = (uint32_t)(((cy * J.cell) >> level) + ly);
            f = (uint64_t)(x | (y << 16)) | ((uint64_t)(key >> 19) << 32) | ((uint64_t)level << 48);
        }
        gstore<uint64_t>(J.out + (size_t)cy * J.gw + cx, f);
    }
}

__device__ void detect_region(const fg_job &J, const Region &R, uint8_t *smem) {
    uint32_t *keys = (uint32_t *)(smem + OFF_KEYS);
    __syncthreads();   // previous region's slot writes have read the keys
    keys_clear(keys, R.ncx * R.ncy);
    for (int sy0 = R.P.ry0; sy0 < R.yr1; sy0 += SUB)
        for (int sx0 = R.P.rx0; sx0 < R.xr1; sx0 += SUB)
            process_subtile(J, sx0, sy0, R.xr1, R.yr1, R.P, smem);
    __syncthreads();
    keys_write(J, R, keys);
}

// Cell keys of a region from the slots an earlier pass wrote (the inverse
// of keys_write).
__device__ void keys_from_slots(const fg_job &J, const Region &R, uint32_t *keys) {
    for (int i = threadIdx.x; i < R.ncx * R.ncy; i += blockDim.x) {
        const int qy = div_small(i, R.ncx);
        const int cx = R.rxi * R.rcells + i - qy * R.ncx, cy = R.ryi * R.rcells + qy;
        const uint64_t f = gload<uint64_t>(J.out + (size_t)cy * J.gw + cx);
        const uint32_t score = (uint32_t)(f >> 32) & 0xFFFFu;
        uint32_t key = 0;
        if (score) {
            const int level = (int)((f >> 48) & 0xFFu);
            const int cw = J.cell >> level;
            const int lx = (int)(f & 0xFFFFu) - ((cx * J.cell) >> level);
            const int ly = (int)((f >> 16) & 0xFFFFu) - ((cy * J.cell) >> level);
            key = (score << 19) | ((uint32_t)(7 - level) << 16) | (0xFFFFu - (uint32_t)(ly * cw + lx));
        }
        keys[i] = key;
    }
}

// Threads that own a quad of a fused level-0 tile (at most 96 rows of 4).
constexpr int QUAD_THREADS = 8 * (96 / 4);
static_assert(SUB + 2 * (4 << (MAX_FUSED - 1)) <= 96, "fused tiles have at most 96 level-0 rows");

// Tile staging of the pipelined kernel: thread i owns the 16-byte chunk
// column i % 8 of level-0 tile rows 4(i/8) .. 4(i/8)+3 (workgroups of at
// least 256 threads cover a fused tile), so it holds whole 16 x 4 blocks and
// builds the 8 x 2 level-1 and 4 x 1 level-2 pixels they cover in registers.
//
// The loads go through a buffer resource over the plane rows the tile covers
// (H * P bytes of a plane are addressable): a row above or below the plane
// reads zero through the buffer's range check.  A chunk left or right of the
// plane is not loaded and keeps stale register values.  No pixel outside the
// plane is ever used as a pixel value (it is never testable, never inside a
// testable pixel's circle, and never written to a level plane), so the tile
// needs no zeros there.  Chunks a thread does not own keep stale values too,
// which quad_commit never reads.
__device__ __forceinline__ void quad_issue(TileRegs &R, const uint8_t *img, int H, int P, const Stage &st) {
    const int ch = threadIdx.x & 7, q = threadIdx.x >> 3;
    const int gx = st.tx + 16 * ch;
    if (ch >= (st.tw >> 4) || 4 * q >= st.th || gx < 0 || gx >= P) return;
    const int y0 = max(st.ty, 0), y1 = min(st.ty + st.th, H);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(img + (ptrdiff_t)y0 * P), (short)0, max(y1 - y0, 0) * P, 0x00020000);
    int off = (st.ty + 4 * q - y0) * P + gx;   // negative: out of range, reads zero
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        R.v[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
        off += P;
    }
}

// Write the n-pixel piece w (n = 4 or 8, little-endian) of row y of a plane,
// starting at column x (a multiple of n), clipped to [sx, ex) x [sy, ey).
__device__ __forceinline__ void store_piece(uint8_t *plane, int P, int y, int x, uint64_t w, int n,
                                            const Geo &g) {
    if (y < g.sy || y >= g.ey || x + n <= g.sx || x >= g.ex) return;
    uint8_t *d = plane + (ptrdiff_t)y * P + x;
    if (x >= g.sx && x + n <= g.ex) {
        if (n == 8)
            gstore<uint64_t>(d, w);
        else
            gstore<uint32_t>(d, (uint32_t)w);
    } else {
        for (int i = 0; i < n; ++i)
            if (x + i >= g.sx && x + i < g.ex) gstore<uint8_t>(d + i, (uint8_t)(w >> (8 * i)));
    }
}

// Commit the quad R (rows 4q .. 4q+3 of chunk column ch) of a level-B tile of
// F levels to LDS, build levels B+1 and B+2 of it into LDS from registers, and
// write the area's own pixels of those levels to their planes.  A quad's rows
// past the tile (at most three, still inside the 96 rows of the LDS tile) are
// committed too: nothing reads them, and the level rows they feed lie past the
// level tiles.
__device__ __forceinline__ void quad_commit(uint8_t *smem, const TileRegs &R, int q, int ch, const Stage &st,
                                            const fg_job &J, int B, int F, const Geo &g1, const Geo &g2) {
    uint8_t *t0 = smem + T0 + 4 * q * LP + 16 * ch;
#pragma unroll
    for (int j = 0; j < 4; ++j) *(u32x4 *)(t0 + j * LP) = R.v[j];
    if (F < 2) return;
    const u32x4 a = R.v[0], b = R.v[1], c = R.v[2], d = R.v[3];
    const uint32_t r0a = halve4(make_uint2(a.x, a.y), make_uint2(b.x, b.y));
    const uint32_t r0b = halve4(make_uint2(a.z, a.w), make_uint2(b.z, b.w));
    const uint32_t r1a = halve4(make_uint2(c.x, c.y), make_uint2(d.x, d.y));
    const uint32_t r1b = halve4(make_uint2(c.z, c.w), make_uint2(d.z, d.w));
    *(uint2 *)(smem + T1 + (2 * q) * LP + 8 * ch) = make_uint2(r0a, r0b);
    *(uint2 *)(smem + T1 + (2 * q + 1) * LP + 8 * ch) = make_uint2(r1a, r1b);
    const int x1 = (st.tx >> 1) + 8 * ch, y1 = (st.ty >> 1) + 2 * q;
    store_piece(J.lvl[B + 1], J.pitch[B + 1], y1, x1, (uint64_t)r0b << 32 | r0a, 8, g1);
    store_piece(J.lvl[B + 1], J.pitch[B + 1], y1 + 1, x1, (uint64_t)r1b << 32 | r1a, 8, g1);
    if (F < 3) return;
    const uint32_t l2 = halve4(make_uint2(r0a, r0b), make_uint2(r1a, r1b));
    *(uint32_t *)(smem + T2 + q * LP + 4 * ch) = l2;
    store_piece(J.lvl[B + 2], J.pitch[B + 2], (st.ty >> 2) + q, (st.tx >> 2) + 4 * ch, l2, 4, g2);
}

// ---------------------------------------------------------------------------
// Levels past the fused ones, three at a time: levels B .. B+F-1 (B a multiple
// of MAX_FUSED, F <= MAX_FUSED) of an upper region, built from level B-1 and
// detected by one workgroup, folded into the slots of the levels below.
//
// The levels are small (level 3 holds 1/64 of the pixels), so what bounds the
// pass is one workgroup's chain of loads, halvings and passes, and the launch.
// One launch in place of one per level and a detection by level-0 regions (8
// pixels of level 3 a workgroup): 4096x2160, 5 levels, 10.3 us instead of 33;
// 1920x1080, 4 levels, 7.9 instead of 8 to 10.

// Copy a level's area from its LDS tile to the plane, in pieces of 4 pixels
// from columns that are multiples of 4.
__device__ void store_area(const uint8_t *tile, const Geo &g, uint8_t *img, int P) {
    const int x0 = g.sx & ~3, wpr = (g.ex - x0 + 3) >> 2, h = g.ey - g.sy;
    if (wpr <= 0 || h <= 0) return;
    for (int i = threadIdx.x; i < wpr * h; i += blockDim.x) {
        const int yy = div_small(i, wpr), y = g.sy + yy, x = x0 + 4 * (i - yy * wpr);
        store_piece(img, P, y, x, *(const uint32_t *)(tile + (y - g.ty) * LP + (x - g.tx)), 4, g);
    }
}

// Level-B tile of an upper region: task i halves two rows of 32 bytes of level
// B-1 into the 16 pixels of chunk column i % nch of tile row i / nch, and
// writes those of the area to the level-B plane.  One row a task: a wave
// issues an instruction every four cycles here, with one wave per SIMD, so the
// work is spread over every lane (four rows a thread took 10.5 us where one
// took 8.8).  Rows outside the plane read zero
// through the buffer's range check; like the columns past it (row padding or
// the next row), they feed no pixel that is used.
struct UpperRows {
    u32x4 a0, a1, b0, b1;
};

__device__ __forceinline__ void upper_issue(UpperRows &u, const __amdgpu_buffer_rsrc_t &rs, int i, int tasks,
                                            int nch, int sp, int y0, const Stage &st, const Geo &g) {
    const int r = div_small(i, nch), gx = st.tx + 16 * (i - r * nch);
    u.a0 = u.a1 = u.b0 = u.b1 = u32x4{0u, 0u, 0u, 0u};
    if (i >= tasks || gx < 0 || gx >= g.W) return;
    const int off = (st.ty + r - y0) * 2 * sp + 2 * gx;   // negative: out of range, reads zero
    u.a0 = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    u.a1 = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16, 0, 0);
    u.b0 = __builtin_amdgcn_raw_buffer_load_b128(rs, off + sp, 0, 0);
    u.b1 = __builtin_amdgcn_raw_buffer_load_b128(rs, off + sp + 16, 0, 0);
}

__device__ __forceinline__ void upper_commit(const UpperRows &u, uint8_t *tile, const fg_job &J, int B, int i,
                                             int tasks, int nch, const Stage &st, const Geo &g) {
    if (i >= tasks) return;
    const int r = div_small(i, nch), ch = i - r * nch;
    u32x4 o;
    o.x = halve4(make_uint2(u.a0.x, u.a0.y), make_uint2(u.b0.x, u.b0.y));
    o.y = halve4(make_uint2(u.a0.z, u.a0.w), make_uint2(u.b0.z, u.b0.w));
    o.z = halve4(make_uint2(u.a1.x, u.a1.y), make_uint2(u.b1.x, u.b1.y));
    o.w = halve4(make_uint2(u.a1.z, u.a1.w), make_uint2(u.b1.z, u.b1.w));
    *(u32x4 *)(tile + r * LP + 16 * ch) = o;
    const int gx = st.tx + 16 * ch, gy = st.ty + r;
    store_piece(J.lvl[B], J.pitch[B], gy, gx, (uint64_t)o.y << 32 | o.x, 8, g);
    store_piece(J.lvl[B], J.pitch[B], gy, gx + 8, (uint64_t)o.w << 32 | o.z, 8, g);
}

// The upper region in column rxi and row ryi of the grid of fg_upper_cells
// cells.
__device__ Region upper_region_at(const fg_job &J, int rxi, int ryi) {
    Region R = region_at(J, 0, 0);   // the parameters every region shares
    const int rc = fg_upper_cells(J.cell, J.rcells);
    R.ryi = ryi;
    R.rxi = rxi;
    R.rcells = rc;
    R.ncx = min(rc, J.gw - R.rxi * rc);
    R.ncy = min(rc, J.gh - R.ryi * rc);
    R.P.rx0 = R.rxi * rc * J.cell;
    R.P.ry0 = R.ryi * rc * J.cell;
    R.P.ncx = R.ncx;
    R.xr1 = min(R.P.rx0 + R.ncx * J.cell, J.w[0]);
    R.yr1 = min(R.P.ry0 + R.ncy * J.cell, J.h[0]);
    return R;
}

// Area of level k of an upper region staged at `st` on level B.
__device__ __forceinline__ void upper_geo(const fg_job &J, const Region &R, int k, int B, const Stage &st, Geo &g) {
    g.k = k;
    g.W = J.w[k];
    g.H = J.h[k];
    g.sx = R.P.rx0 >> k;
    g.sy = R.P.ry0 >> k;
    g.ex = min(R.xr1 >> k, g.W);
    g.ey = min(R.yr1 >> k, g.H);
    const int d = k - B;
    g.tbase = sel3(d, T0, T1, T2);
    g.tx = st.tx >> d;
    g.ty = st.ty >> d;
    g.moff = sel3(d, OFF_M0, OFF_M1, OFF_M2);
    g.mp = MP;
    set_groups(g);
}

// SCORES: write the score maps of the levels instead of selecting features.  B
// is a template argument because a by-value job indexed by a variable is copied
// to scratch memory (13 us instead of 7.9 for a 1920x1080 frame).
template <int B, bool SCORES>
__device__ __forceinline__ void upper_region(const fg_job &J, int rxi, int ryi, uint8_t *smem) {
    Region R = upper_region_at(J, rxi, ryi);
    constexpr int TOP = B + MAX_FUSED <= FAST_MAX_LEVELS ? MAX_FUSED : FAST_MAX_LEVELS - B;   // levels there can be
    const int F = min(J.levels - B, TOP);
    const int sx = R.P.rx0 >> B, sy = R.P.ry0 >> B;
    const int ex = min(R.xr1 >> B, J.w[B]), ey = min(R.yr1 >> B, J.h[B]);
    if (ex <= sx || ey <= sy) return;   // no pixel of level B, so none above
    const int H0 = 4 << (F - 1);
    Stage st;
    st.tx = (sx - H0) & ~15;
    st.ty = (sy - H0) & ~3;   // the two levels above start on whole rows
    st.tw = ((ex + H0 + 15) & ~15) - st.tx;
    st.th = ey + H0 - st.ty;
    Geo g0, g1, g2;
    upper_geo(J, R, B, B, st, g0);
    g1 = g0;
    g2 = g0;
    if (F > 1) upper_geo(J, R, B + 1, B, st, g1);
    if constexpr (TOP > 2)
        if (F > 2) upper_geo(J, R, B + 2, B, st, g2);
    uint32_t *keys = (uint32_t *)(smem + OFF_KEYS);
    const int nch = st.tw >> 4, tasks = nch * st.th, sp = J.pitch[B - 1];
    const int y0 = max(st.ty, 0), y1 = min(st.ty + st.th, g0.H);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(J.lvl[B - 1] + (ptrdiff_t)(2 * y0) * sp), (short)0, max(y1 - y0, 0) * 2 * sp, 0x00020000);
    UpperRows u;
    upper_issue(u, rs, threadIdx.x, tasks, nch, sp, y0, st, g0);
    // while the first rows load: the maps, the slots so far, the compass groups
    zero_lds(smem + OFF_M0, OFF_KEYS - OFF_M0);
    if (!SCORES) keys_from_slots(J, R, keys);
    GroupCache cache{0u, 0u};
    const bool cached = blockDim.x >= 256;
    if (cached) group_cache_fill(cache, g0, g1, g2, F);
    for (int i = threadIdx.x;;) {
        upper_commit(u, smem + T0, J, B, i, tasks, nch, st, g0);
        i += blockDim.x;
        if (i - (int)threadIdx.x >= tasks) break;   // uniform
        upper_issue(u, rs, i, tasks, nch, sp, y0, st, g0);
    }
    __syncthreads();
    if (F > 1) {
        halve_two(smem + T0, smem + T1, smem + T2, st.tw, st.th, F > 2);
        __syncthreads();
        if (has_area(g1)) store_area(smem + T1, g1, J.lvl[B + 1], J.pitch[B + 1]);
        if constexpr (TOP > 2)
            if (F > 2 && has_area(g2)) store_area(smem + T2, g2, J.lvl[B + 2], J.pitch[B + 2]);
    }
    if (SCORES)
        for (int l = 0; l < TOP; ++l) {   // entries past F are not used
            R.P.smap[l] = J.smap[B + l];
            R.P.spitch[l] = J.smap_pitch[B + l];
        }
    run_passes(smem, g0, g1, g2, F, R.P, keys, cached, cache);
    if (SCORES) return;
    __syncthreads();
    keys_write(J, R, keys);
}

// Stage of a whole region (FG_WHOLE).
__device__ __forceinline__ Stage whole_stage(const Region &R) {
    constexpr int HALO = 4 << (MAX_FUSED - 1);
    return Stage{R.P.rx0 - HALO, R.P.ry0 - HALO, SUB + 2 * HALO, SUB + 2 * HALO};
}

// Commit a whole region's quad (quad_commit).  Its level pieces lie whole
// inside or outside the region, those of one quad together, so one test takes
// the place of their clipping, and the planes are addressed from scalar bases.
__device__ __forceinline__ void whole_commit(uint8_t *smem, const TileRegs &R, const fg_job &J, const Region &rg) {
    const int ch = threadIdx.x & 7, q = threadIdx.x >> 3;
    if (ch >= 6 || q >= 24) return;
    uint8_t *t0 = smem + T0 + 4 * q * LP + 16 * ch;
#pragma unroll
    for (int j = 0; j < 4; ++j) *(u32x4 *)(t0 + j * LP) = R.v[j];
    const u32x4 a = R.v[0], b = R.v[1], c = R.v[2], d = R.v[3];
    const uint2 r0 = make_uint2(halve4(make_uint2(a.x, a.y), make_uint2(b.x, b.y)),
                                halve4(make_uint2(a.z, a.w), make_uint2(b.z, b.w)));
    const uint2 r1 = make_uint2(halve4(make_uint2(c.x, c.y), make_uint2(d.x, d.y)),
                                halve4(make_uint2(c.z, c.w), make_uint2(d.z, d.w)));
    const uint32_t l2 = halve4(r0, r1);
    *(uint2 *)(smem + T1 + (2 * q) * LP + 8 * ch) = r0;
    *(uint2 *)(smem + T1 + (2 * q + 1) * LP + 8 * ch) = r1;
    *(uint32_t *)(smem + T2 + q * LP + 4 * ch) = l2;
    // quads 4 .. 19 of chunk columns 1 .. 4 are the region's own
    const uint32_t oy = (uint32_t)q - 4, ox = (uint32_t)ch - 1;
    if (oy >= 16 || ox >= 4) return;
    uint8_t *p1 = J.lvl[1] + (ptrdiff_t)(rg.P.ry0 >> 1) * J.pitch[1] + (rg.P.rx0 >> 1);
    uint8_t *p2 = J.lvl[2] + (ptrdiff_t)(rg.P.ry0 >> 2) * J.pitch[2] + (rg.P.rx0 >> 2);
    const uint32_t o1 = 2 * oy * (uint32_t)J.pitch[1] + 8 * ox;
    gstore<uint64_t>(p1 + o1, (uint64_t)r0.y << 32 | r0.x);
    gstore<uint64_t>(p1 + o1 + (uint32_t)J.pitch[1], (uint64_t)r1.y << 32 | r1.x);
    gstore<uint32_t>(p2 + (oy * (uint32_t)J.pitch[2] + 4 * ox), l2);
}

// Issue the level-0 tile loads of an item's region (a single fused sub-tile).
template <bool WHOLE>
__device__ __forceinline__ void region_prefetch(const fg_job &J, uint32_t code, TileRegs &T) {
    if (WHOLE && (code & FG_WHOLE)) {
        quad_issue(T, J.lvl[0], J.h[0], J.pitch[0], whole_stage(whole_region(J, code)));
    } else {
        const Region R = item_region(J, code);
        quad_issue(T, J.lvl[0], J.h[0], J.pitch[0], fused_stage(J, R.P.rx0, R.P.ry0, R.xr1, R.yr1));
    }
}

// Commit a prefetched region's tile and build its levels 1-2.
template <bool WHOLE>
__device__ __forceinline__ void region_commit(uint8_t *smem, const fg_job &J, uint32_t code, const TileRegs &T) {
    if (WHOLE && (code & FG_WHOLE)) {
        whole_commit(smem, T, J, whole_region(J, code));
        return;
    }
    const Region R = item_region(J, code);
    const Stage st = fused_stage(J, R.P.rx0, R.P.ry0, R.xr1, R.yr1);
    Geo g0, g1, g2;
    describe_fused(J, R.P.rx0, R.P.ry0, R.xr1, R.yr1, st, g0, g1, g2);
    const int ch = threadIdx.x & 7, q = threadIdx.x >> 3;
    if (ch < (st.tw >> 4) && 4 * q < st.th) quad_commit(smem, T, q, ch, st, J, 0, fused_levels(J), g1, g2);
}

// Bijective block -> item map that gives each XCD (blocks are dealt to the 8
// XCDs round-robin) a contiguous run of items, so neighbouring regions share
// halo lines in the same L2.
__device__ __forceinline__ int xcd_item(int b, int n) {
    const int q = n >> 3, r = n & 7;
    const int xcd = b & 7, local = b >> 3;
    return xcd < r ? xcd * (q + 1) + local : r * (q + 1) + (xcd - r) * q + local;
}

// Score-map mode of a region: levels 0 .. F-1 from one load, no cell keys.
__device__ void scores_region(const fg_job &J, int region, uint8_t *smem) {
    const Region R = region_of(J, region);
    Params P = R.P;
    for (int l = 0; l < MAX_FUSED; ++l) {
        P.smap[l] = J.smap[l < J.levels ? l : 0];
        P.spitch[l] = J.smap_pitch[l < J.levels ? l : 0];
    }
    for (int sy0 = P.ry0; sy0 < R.yr1; sy0 += SUB)
        for (int sx0 = P.rx0; sx0 < R.xr1; sx0 += SUB) process_subtile(J, sx0, sy0, R.xr1, R.yr1, P, smem);
}

// The kernel arguments' cache lines, fetched together at a kernel's start.
// They lie in host-visible memory and each costs a first access about 700
// cycles; read where they are first used, they queue one behind the other
// (3000 of the 12300 cycles of a 320x240 frame's workgroup, 1700 this way).
__device__ __forceinline__ void touch_arguments() {
    const auto p = (const __attribute__((address_space(4))) uint32_t *)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert(sizeof(fg_job) + 16 <= 384, "the argument and the block size lie in six lines");
    const uint32_t a = p[0], b = p[16], c = p[32], d = p[48], e = p[64], f = p[80];
    asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d), "s"(e), "s"(f));
}

// Standalone NMS over (2R+1) x (2R+1) neighbourhoods and the cell arg-max
// across levels, from global score maps (J.smap).  One workgroup per region;
// the region is walked in 64 x 64 sub-tiles, every level's part of a sub-tile
// (64 >> k pixels a side) staged in LDS at once with an R-pixel halo (zero
// outside the map).
//
// Few pixels score (about 2%), so the pixels that do are gathered into a list
// as they are staged, and only they are compared with their windows: a pixel
// survives when its score is above every earlier one of its window in
// row-major order and not below any later one.  What bounds it is the chain
// of one workgroup (load, gather, compare) and the maps' bytes.  Comparing
// every pixel by separable window maxima, level after level, took 9.7 us for
// 641x479 with 3 levels and R = 1, and 30.4 for 1920x1080 with 4 levels and
// R = 4; this takes 6.7 and 10.2.  With every pixel of the second frame scoring
// it takes 18.2 us at R = 1 and 23.6 at R = 4 (20.6 and 31.6 before).
//
// A map's rows start at any even address, so a row's 8-pixel chunks are loaded
// from where they lie (16-byte loads at 2-byte alignment); a chunk across the
// row's end is loaded from inside the row and shifted.
constexpr int NMS_THREADS = 256;

// Elements gx .. gx+7 of a map row of W elements (zero outside it).
__device__ __forceinline__ u32x4 map_chunk(const uint16_t *row, int W, int gx) {
    if (gx >= W || gx + 8 <= 0) return u32x4{0u, 0u, 0u, 0u};
    if (W < 8) {   // the row is shorter than a chunk
        u32x4 v = {0u, 0u, 0u, 0u};
        for (int x = max(gx, 0); x < W; ++x) {
            const int e = x - gx;
            if (e < 8) v[e >> 1] |= (uint32_t)gload<uint16_t>(row + x) << (16 * (e & 1));
        }
        return v;
    }
    const int at = min(max(gx, 0), W - 8), d = gx - at;
    const u32x4 v = *(const GLOBAL u32x4_at2 *)(row + at);
    if (d == 0) return v;
    uint64_t lo = (uint64_t)v.y << 32 | v.x, hi = (uint64_t)v.w << 32 | v.z;
    if (d < 0) {   // the first -d elements lie before the row
        const int sh = 16 * -d;
        hi = sh >= 64 ? lo << (sh - 64) : hi << sh | lo >> (64 - sh);
        lo = sh >= 64 ? 0 : lo << sh;
    } else {       // the last d lie past it
        const int sh = 16 * d;
        lo = sh >= 64 ? hi >> (sh - 64) : lo >> sh | hi << (64 - sh);
        hi = sh >= 64 ? 0 : hi >> sh;
    }
    return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// Level k's tile in LDS, at its largest: rows, row pitch and first element.
template <int R>
struct NmsTiles {
    static constexpr int side(int k) { return (SUB >> k) > 0 ? SUB >> k : 1; }
    static constexpr int rows(int k) { return side(k) + 2 * R; }
    static constexpr int pitch(int k) { return (side(k) + 2 * R + 7) & ~7; }
    static constexpr int first(int k) { return k == 0 ? 0 : first(k - 1) + rows(k - 1) * pitch(k - 1); }
    // staging steps: threads take one chunk each
    static constexpr int steps(int k) { return (rows(k) * (pitch(k) / 8) + NMS_THREADS - 1) / NMS_THREADS; }
    static constexpr int pixels() {
        int n = 0;
        for (int k = 0; k < FAST_MAX_LEVELS; ++k) n += side(k) * side(k);
        return n;
    }
    static constexpr int LIST = first(FAST_MAX_LEVELS) * 2;     // byte offset of the pixel list
    static constexpr int KEYS = LIST + pixels() * 4;
    static constexpr int BYTES = KEYS + MAX_KEYS * 4;
    static_assert(LIST % 16 == 0, "16-byte tile stores");
    static_assert(steps(0) == 3 && steps(1) == 1, "chunks a thread holds");
};

// A level's part of the sub-tile at (sx0, sy0), from (x0, y0) to (x1, y1).
struct NmsPart {
    int x0, y0, x1, y1;
    __device__ NmsPart(const fg_job &J, const Region &R, int sx0, int sy0, int k) {
        x0 = sx0 >> k;
        y0 = sy0 >> k;
        x1 = min(min((sx0 + SUB) >> k, R.xr1 >> k), J.w[k]);
        y1 = min(min((sy0 + SUB) >> k, R.yr1 >> k), J.h[k]);
    }
    __device__ bool empty() const { return x1 <= x0 || y1 <= y0; }
};

// The score of a listed pixel if it wins its (2W+1) x (2W+1) window (W <= R),
// else 0: it is above every earlier pixel in row-major order and not below any
// later one.
template <int R, int W>
__device__ __forceinline__ uint32_t nms_peak(const uint16_t *tile, uint32_t entry) {
    using L = NmsTiles<R>;
    const int k = entry >> 16, yy = (entry >> 8) & 0xFF, xx = entry & 0xFF;
    int first = 0, pitch = L::pitch(0);
#pragma unroll
    for (int l = 1; l < FAST_MAX_LEVELS; ++l) {
        first = k == l ? L::first(l) : first;
        pitch = k == l ? L::pitch(l) : pitch;
    }
    const uint16_t *q = tile + first + (yy - W) * pitch + xx - W;   // the window's corner
    uint32_t s = 0, earlier = 0, later = 0;
#pragma unroll
    for (int dy = 0; dy <= 2 * W; ++dy) {
        const auto row = lds_base(q + dy * pitch);
#pragma unroll
        for (int dx = 0; dx <= 2 * W; ++dx) {
            const uint32_t x = row[dx];
            if (dy == W && dx == W)
                s = x;
            else if (dy < W || (dy == W && dx < W))
                earlier = max(earlier, x);
            else
                later = max(later, x);
        }
    }
    return s > earlier && s >= later ? s : 0u;
}

template <int R>
__global__ void __launch_bounds__(NMS_THREADS) nms_grid_kernel(fg_job J) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    __shared__ int s_count;
    using L = NmsTiles<R>;
    touch_arguments();
    const Region rg = region_of(J, xcd_item(blockIdx.x, gridDim.x));
    uint16_t *tile = (uint16_t *)smem;
    uint32_t *list = (uint32_t *)(smem + L::LIST), *keys = (uint32_t *)(smem + L::KEYS);
    keys_clear(keys, rg.ncx * rg.ncy);
    const int lane = lane_id();
    for (int sy0 = rg.P.ry0; sy0 < rg.yr1; sy0 += SUB) {
        for (int sx0 = rg.P.rx0; sx0 < rg.xr1; sx0 += SUB) {
            // this thread's chunks of every level: level 0 three, the others one
            constexpr int N = FAST_MAX_LEVELS + 2;
            u32x4 v[N];
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int k = n < 3 ? 0 : n - 2;
                v[n] = u32x4{0u, 0u, 0u, 0u};
                if (k >= J.levels) continue;
                const NmsPart p(J, rg, sx0, sy0, k);
                const int nch = (p.x1 - p.x0 + 2 * R + 7) >> 3;
                const int i = (int)threadIdx.x + (n < 3 ? n * NMS_THREADS : 0);
                const int yy = div_small(i, max(nch, 1)), gy = p.y0 - R + yy;
                if (p.empty() || gy >= p.y1 + R || gy < 0 || gy >= J.h[k]) continue;
                v[n] = map_chunk(J.smap[k] + (ptrdiff_t)gy * J.smap_pitch[k], J.w[k],
                                 p.x0 - R + 8 * (i - yy * nch));
            }
            __syncthreads();   // the previous sub-tile's tiles and list have been read
            if (threadIdx.x == 0) s_count = 0;
            // to LDS; bit j of a chunk's mask: its element 2j scores and is the
            // part's own, bit 16 + j: element 2j + 1
            uint32_t own[N];
            int mine = 0;
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int k = n < 3 ? 0 : n - 2;
                own[n] = 0;
                if (k >= J.levels) continue;
                const NmsPart p(J, rg, sx0, sy0, k);
                const int nch = (p.x1 - p.x0 + 2 * R + 7) >> 3;
                const int i = (int)threadIdx.x + (n < 3 ? n * NMS_THREADS : 0);
                const int yy = div_small(i, max(nch, 1)), xx = 8 * (i - yy * nch), gy = p.y0 - R + yy;
                if (p.empty() || gy >= p.y1 + R) continue;
                *(u32x4 *)(tile + L::first(k) + yy * L::pitch(k) + xx) = v[n];
                if (gy < p.y0 || gy >= p.y1) continue;
                auto ones = [](uint32_t x) {
                    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, x),
                                                                                  u16x2{1, 1}));
                };
                const uint32_t m = ones(v[n].x) | ones(v[n].y) << 1 | ones(v[n].z) << 2 | ones(v[n].w) << 3;
                // own elements: lo <= e < hi
                const int lo = min(max(R - xx, 0), 8), hi = max(min(p.x1 - p.x0 + R - xx, 8), lo);
                own[n] = m & (bit_range((lo + 1) >> 1, (hi + 1) >> 1) | bit_range(lo >> 1, hi >> 1) << 16);
                mine += __builtin_popcount(own[n]);
            }
            __syncthreads();   // the count is zero
            const int incl = wave_scan(mine);
            int at = 0;
            if (lane == 63) at = incl ? atomicAdd(&s_count, incl) : 0;
            at = __builtin_amdgcn_readlane(at, 63) + incl - mine;
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int k = n < 3 ? 0 : n - 2;
                if (k >= J.levels) continue;
                const NmsPart p(J, rg, sx0, sy0, k);
                const int nch = (p.x1 - p.x0 + 2 * R + 7) >> 3;
                const int i = (int)threadIdx.x + (n < 3 ? n * NMS_THREADS : 0);
                uint32_t m = own[n];
                if (!__any(m != 0)) continue;
                const int yy = div_small(i, max(nch, 1)), xx = 8 * (i - yy * nch);
                while (m) {   // entry: level, tile row, tile column
                    const int j = __builtin_ctz(m);
                    m &= m - 1;
                    list[at++] = (uint32_t)(k << 16 | yy << 8 | (xx + (j < 16 ? 2 * j : 2 * (j - 16) + 1)));
                }
            }
            __syncthreads();   // tiles and list are complete
            // each wave takes a part of the list; with more than two rounds
            // a thread (maps scored far denser than corners are), what
            // loses inside its 3 x 3 neighbourhood leaves the list first
            const int count = s_count, part = (count + NMS_THREADS / 64 - 1) / (NMS_THREADS / 64);
            uint32_t *mylist = list + (threadIdx.x >> 6) * part;
            int n = min(part, max(count - (int)(threadIdx.x >> 6) * part, 0));
            if (R > 1 && count > 2 * NMS_THREADS) {
                int kept = 0;
                for (int i0 = 0; i0 < n; i0 += 64) {
                    const uint32_t e = mylist[min(i0 + lane, n - 1)];
                    const bool keep = i0 + lane < n && nms_peak<R, 1>(tile, e) != 0;
                    const uint64_t bal = __ballot(keep);
                    const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                    wave_sync();
                    if (keep) mylist[kept + rank] = e;
                    wave_sync();
                    kept += __popcll(bal);
                }
                n = kept;
            }
            for (int i = lane; i < n; i += 64) {
                const uint32_t e = mylist[i];
                const int k = e >> 16, yy = (e >> 8) & 0xFF, xx = e & 0xFF;
                const uint32_t s = nms_peak<R, R>(tile, e);
                if (s == 0) continue;
                // position in the region at level k, then in its cell
                const int ox = (sx0 >> k) + xx - R - (rg.P.rx0 >> k), oy = (sy0 >> k) + yy - R - (rg.P.ry0 >> k);
                const int cw = J.cell >> k;
                const int cx = div_small(ox, cw), cy = div_small(oy, cw);
                const uint32_t local = (uint32_t)((oy - cy * cw) * cw + (ox - cx * cw));
                atomicMax(&keys[cy * rg.ncx + cx], (s << 19) | ((uint32_t)(7 - k) << 16) | (0xFFFFu - local));
            }
        }
    }
    __syncthreads();
    keys_write(J, rg, keys);
}

// One frame whose regions are single fused sub-tiles, workgroups of at least
// 256 threads: one region per block, staged as the pipelined kernel stages
// (quad_issue, quad_commit), with everything that does not need the pixels
// done while they load.  One wave per SIMD runs on a small frame, so the time
// is the chain of one workgroup, not the throughput: barriers and LDS round
// trips count, and a wave's instructions one by one (four cycles each).
// `scores`: write score maps instead of selecting features.
template <bool SCORES, int SIDE, int NL>
__device__ __forceinline__ void single_region(const fg_job &J, uint8_t *smem) {
    using WR = Whole<SIDE, NL>;
    touch_arguments();
    Region R = region_of(J, xcd_item(blockIdx.x, gridDim.x));
    const Stage st = fused_stage(J, R.P.rx0, R.P.ry0, R.xr1, R.yr1);
    TileRegs T;
    quad_issue(T, J.lvl[0], J.h[0], J.pitch[0], st);
    uint32_t *keys = (uint32_t *)(smem + OFF_KEYS);
    zero_lds(smem + OFF_M0, OFF_KEYS - OFF_M0);
    if (!SCORES) keys_clear(keys, R.ncx * R.ncy);
    const int nl = fused_levels(J);
    const bool full = WR::is(J, R);
    Geo g0, g1, g2;
    describe_fused(J, R.P.rx0, R.P.ry0, R.xr1, R.yr1, st, g0, g1, g2);
    GroupCache cache;
    if (full)
        WR::fill(cache);
    else
        group_cache_fill(cache, g0, g1, g2, nl);
    if (SCORES) {
        for (int l = 0; l < MAX_FUSED; ++l) {
            R.P.smap[l] = J.smap[l < J.levels ? l : 0];
            R.P.spitch[l] = J.smap_pitch[l < J.levels ? l : 0];
        }
    }
    const int ch = threadIdx.x & 7, q = threadIdx.x >> 3;
    if (ch < (st.tw >> 4) && 4 * q < st.th) quad_commit(smem, T, q, ch, st, J, 0, nl, g1, g2);
    __syncthreads();
    if (!full) {
        run_passes(smem, g0, g1, g2, nl, R.P, keys, true, cache);
    } else {
        const int n2 = score_phase(smem, WR::segs(R.P.rx0, R.P.ry0, J.w[0], J.h[0]), WR::maps(J.cell), R.P, true,
                                   cache.e01, cache.e23);
        __syncthreads();
        if (SCORES)
            store_maps(smem, g0, g1, g2, nl, R.P);
        else
            nms_phase(smem, WR::maps(J.cell), 0, R.ncx, keys, n2);
    }
    if (SCORES) return;
    __syncthreads();
    keys_write(J, R, keys);
}

template <int SIDE, int NL>
__global__ void __launch_bounds__(512) detect_single_kernel(fg_job J) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    single_region<false, SIDE, NL>(J, smem);
}

template <int SIDE, int NL>
__global__ void __launch_bounds__(512) score_single_kernel(fg_job J) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    single_region<true, SIDE, NL>(J, smem);
}

__global__ void __launch_bounds__(512) score_plain_kernel(fg_job J) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    scores_region(J, xcd_item(blockIdx.x, gridDim.x), smem);
}

__global__ void __launch_bounds__(512) detect_plain_kernel(fg_job J) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    detect_region(J, region_of(J, xcd_item(blockIdx.x, gridDim.x)), smem);
}

// Levels B .. B+2 of one frame, one upper region per block.
template <int B, bool SCORES>
__global__ void __launch_bounds__(512) upper_plain_kernel(fg_job J) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    touch_arguments();
    upper_region<B, SCORES>(J, blockIdx.x, blockIdx.y, smem);
}

// Levels B .. B+2 of the batch's jobs that have them, one listed upper region
// per block.
template <int B>
__global__ void __launch_bounds__(512) upper_batch_kernel(const fg_job *__restrict__ jobs,
                                                          const fg_item *__restrict__ items) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const fg_item it = items[blockIdx.x];
    const fg_job &J = jobs[it.job];
    if (J.levels > B) upper_region<B, false>(J, (int)(it.region & 0xFFFFu), (int)(it.region >> 16), smem);
}

// Persistent batched detectors.  Work items are regions of all jobs (items[]
// gives each one's job and region, row by row within a job, whole regions
// first and clipped ones last), split over FG_QUEUES queues.  The list is
// cut into runs of FG_QUEUE_RUN consecutive items dealt round-robin: queue c
// holds runs c, c + 8, c + 16, ... and then, past the last full round of
// runs, items c, c + 8, ... of the remainder, so the queues stay within one
// run of each other.  Workgroup g uses queue g % 8; it starts with that
// queue's positions g / 8 and g / 8 + n (n workgroups on the queue) and then
// takes position 2n + k for its k-th ticket of the queue's counter.  Eight
// heads on separate cache lines keep the tickets from queueing behind each
// other.  Workgroups are placed on the XCDs round-robin, so one queue's
// workgroups share one XCD and its L2: a run's regions lie side by side in
// their frame and share the cache lines of their tiles, which a run of one
// region (neighbours on eight different L2s) fetches again from memory.
struct Queue {
    unsigned *head;
    int c, n, first;    // queue index, its workgroups, this workgroup's first position
};

__device__ __forceinline__ Queue queue_of(unsigned *counter) {
    Queue q;
    const int G = (int)gridDim.x;
    q.c = (int)(blockIdx.x % FG_QUEUES);
    q.first = (int)(blockIdx.x / FG_QUEUES);
    q.n = (G - q.c + FG_QUEUES - 1) / FG_QUEUES;
    q.head = counter + q.c * FG_QUEUE_STRIDE;
    return q;
}

// Item at queue position pos, or total past the end.
__device__ __forceinline__ int queue_item(const Queue &q, long long pos, int total) {
    const long long runs = total / (FG_QUEUES * FG_QUEUE_RUN);   // full rounds of runs
    const long long in_runs = runs * FG_QUEUE_RUN;               // positions per queue inside them
    const long long it = pos < in_runs
                             ? ((pos / FG_QUEUE_RUN) * FG_QUEUES + q.c) * FG_QUEUE_RUN + pos % FG_QUEUE_RUN
                             : in_runs * FG_QUEUES + q.c + (long long)FG_QUEUES * (pos - in_runs);
    return it < total ? (int)it : total;
}

// A ticket of the queue.  The ticket's value is first needed after the
// passes of a whole region, so no wait may follow the atomic at once (the
// library is built without the atomic optimiser, whose wave-level rewrite
// reads the result right after the atomic).
__device__ __forceinline__ unsigned queue_ticket(const Queue &q) {
    return __hip_atomic_fetch_add(q.head, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The last workgroup out re-arms the queues for the next launch (every ticket
// a workgroup drew has been resolved by then).
__device__ __forceinline__ void queue_exit(unsigned *counter) {
    if (threadIdx.x == 0) {
        __threadfence();
        const unsigned done = atomicAdd(&counter[FG_EXIT_WORD], 1u);
        if (done == gridDim.x - 1) {
            for (int c = 0; c < FG_QUEUES; ++c) atomicExch(&counter[c * FG_QUEUE_STRIDE], 0u);
            atomicExch(&counter[FG_EXIT_WORD], 0u);
        }
    }
}

// Pipelined kernels, for batches whose regions are all single fused sub-tiles
// and workgroups of at least 256 threads (32 quads of tile rows cover a
// fused tile).  Per region there are three workgroup barriers:
//   [A] the previous region's NMS is done; this region's levels 0-2 are in
//       LDS: clear the score maps and this region's cell keys (two key buffers
//       alternate);
//   [B] draw the ticket of the region after next, run the compass, 8-point
//       and scoring passes; the last wave's first lane resolves the ticket;
//   [C] the scores are complete and the tiles are no longer read: commit
//       the next region's level-0 tile (loaded into registers one region
//       earlier) to LDS, build its levels 1-2 from the registers into LDS
//       and their planes, start loading the tile after it, write the previous
//       region's slots by the threads the commit leaves idle, then run NMS into
//       the keys.
// With WHOLE, whole regions have a path on constant geometry; the others' general
// one then sets up past [B] and keeps no group entries, which would take the
// registers that the whole ones' constants live in (64 frames of three levels 93.8 us,
// 96.1 with them).  Without it, group entries are kept while the staged geometry stays,
// and the set-up hides under the clearing.
template <bool WHOLE>
__device__ __forceinline__ void batch_regions(const fg_job *__restrict__ jobs, const fg_item *__restrict__ items,
                                              int total, unsigned *counter, uint8_t *smem) {
    // s_next[b] carries the item after next from its ticket's lane to the workgroup;
    // the two buffers alternate, so a value is never overwritten before every
    // wave has read it.
    __shared__ int s_next[2];
    const Queue q = queue_of(counter);
    int item = queue_item(q, q.first, total);
    if (item >= total) {   // a queue with fewer items than workgroups
        queue_exit(counter);
        return;
    }
    int next = queue_item(q, q.first + (long long)q.n, total);
    fg_item il = items[item];
    fg_item in = next < total ? items[next] : fg_item{0u, 0u};
    TileRegs T;
    region_prefetch<WHOLE>(jobs[il.job], il.region, T);
    region_commit<WHOLE>(smem, jobs[il.job], il.region, T);
    if (next < total) region_prefetch<WHOLE>(jobs[in.job], in.region, T);
    fg_item prev{0u, 0u};
    bool have_prev = false;
    int b = 0;
    using W3 = Whole<SUB, MAX_FUSED>;
    GroupCache cache{0u, 0u};   // with WHOLE, the whole regions' entries; without, those of geometry cache_key
    if (WHOLE) W3::fill(cache);
    int cache_key = -1;
    auto slots_region = [](const fg_job &J, uint32_t code) {
        return WHOLE && (code & FG_WHOLE) ? whole_region(J, code) : general_region<WHOLE>(J, code);
    };
    while (item < total) {
        const fg_job &J = jobs[il.job];   // uniform: read through the scalar cache
        const bool full = WHOLE && (il.region & FG_WHOLE);
        const Region R = full ? whole_region(J, il.region) : general_region<WHOLE>(J, il.region);
        uint32_t *keys = (uint32_t *)(smem + (b ? OFF_KEYS2 : OFF_KEYS));
        __syncthreads();   // [A]
        zero_lds(smem + OFF_M0, OFF_KEYS - OFF_M0);
        keys_clear(keys, R.ncx * R.ncy);
        Geo g0, g1, g2;
        auto set_up = [&]() {
            const Stage st = fused_stage(J, R.P.rx0, R.P.ry0, R.xr1, R.yr1);
            describe_fused(J, R.P.rx0, R.P.ry0, R.xr1, R.yr1, st, g0, g1, g2);
        };
        if (!WHOLE) set_up();
        __syncthreads();   // [B]
        // one lane only, read only where it was set; left without a value
        // elsewhere so that no copy of the atomic's result (which would wait
        // for it at once) is needed where the branch rejoins
        unsigned ticket;
        // (the first lane of the last wave: wave 0 already carries the extra
        // compass round of a full region, so it sets the region's pace)
        if (threadIdx.x == blockDim.x - 64 && next < total) ticket = queue_ticket(q);
        int n2;
        if (full) {
            n2 = score_phase(smem, W3::segs(R.P.rx0, R.P.ry0, J.w[0], J.h[0]), W3::maps(J.cell), R.P, true, cache.e01,
                             cache.e23);
        } else {
            if (WHOLE) set_up();
            const Segs S = segs_of(g0, g1, g2, fused_levels(J));
            if (!WHOLE) {
                // the staged geometry depends only on the fused level count and the
                // region's size: its origin is 16-aligned
                const int key = fused_levels(J) | (R.xr1 - R.P.rx0) << 2 | (R.yr1 - R.P.ry0) << 9;
                if (__builtin_amdgcn_readfirstlane(cache_key ^ key)) {
                    group_cache_fill(cache, S.s0, S.s1, S.s2);
                    cache_key = key;
                }
            }
            n2 = score_phase(smem, S, maps_of(g0, g1, g2, R.P), R.P, !WHOLE, cache.e01, cache.e23);
        }
        if (threadIdx.x == blockDim.x - 64)
            s_next[b] = next < total ? queue_item(q, 2LL * q.n + ticket, total) : total;
        __syncthreads();   // [C]
        const int after = __builtin_amdgcn_readfirstlane(s_next[b]);
        if (next < total) {
            region_commit<WHOLE>(smem, jobs[in.job], in.region, T);
            if (after < total) {
                const fg_item ia = items[after];
                region_prefetch<WHOLE>(jobs[ia.job], ia.region, T);
            }
        }
        // the previous region's slots, written by the threads the tile commit
        // leaves idle (quads past level-0 row 96); its keys buffer is next
        // cleared after the next [A]
        if (have_prev && threadIdx.x >= QUAD_THREADS) {
            const fg_job &Jp = jobs[prev.job];
            keys_write(Jp, slots_region(Jp, prev.region), (const uint32_t *)(smem + (b ? OFF_KEYS : OFF_KEYS2)),
                       threadIdx.x - QUAD_THREADS, blockDim.x - QUAD_THREADS);
        }
        if (full)
            nms_phase(smem, W3::maps(J.cell), 0, R.ncx, keys, n2);
        else
            nms_phase(smem, maps_of(g0, g1, g2, R.P), 0, R.ncx, keys, n2);
        prev = il;
        have_prev = true;
        item = next;
        il = in;
        next = after;
        in = after < total ? items[after] : fg_item{0u, 0u};
        b ^= 1;
    }
    __syncthreads();
    if (have_prev) {   // the last region used the buffer before the final flip of b
        const fg_job &Jp = jobs[prev.job];
        keys_write(Jp, slots_region(Jp, prev.region), (const uint32_t *)(smem + (b ? OFF_KEYS : OFF_KEYS2)));
    }
    queue_exit(counter);
}

// For batches with whole regions, but not for several workgroups past 256 threads
// a CU (fg_choose_batch).  What bounds it: vector issue 60% of the time (1324
// vector instructions a wave and region) and, between the three barriers, the
// latency of LDS and of the chains.  With whole regions' geometry constant, the
// compass by byte averages and the sums in 16-bit lanes the 64-frame batch went
// from 103 to 89.7 us, with clipped regions' coordinates in vector registers (54
// scalar registers spilled instead of 94) to 87.7.
// Three waves a SIMD, which the LDS of three workgroups of 256 threads a CU allows
// anyway: the constants of a whole region then stay in registers (at four waves,
// 128 registers, 72 of them are spilled and the kernel takes 214 us instead of 90).
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(3, 3)))
detect_batch_kernel(const fg_job *__restrict__ jobs, const fg_item *__restrict__ items, int total,
                    unsigned *counter) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    batch_regions<true>(jobs, items, total, counter, smem);
}

// For batches with few whole regions or none, and for several workgroups past 256
// threads a CU.  Four waves a SIMD, 128 registers.
// A region's columns in vector registers and its rows in scalar ones: 15 scalar
// registers are spilled and no vector one; with both in vector ones 9 and 3.
// 64 frames of one level and 32-pixel cells 85.7 us (95.3 while such regions shared
// a kernel with whole ones, both coordinates in scalar registers), of two levels
// 97.9 (107.6), of three levels and 48-pixel cells 137.1 (155.4).
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
detect_batch_any_kernel(const fg_job *__restrict__ jobs, const fg_item *__restrict__ items, int total,
                        unsigned *counter) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    batch_regions<false>(jobs, items, total, counter, smem);
}

// Generic persistent kernel: any region size and workgroup size, one region
// at a time.  Its general geometry, a hundred words the same in every lane, takes
// the scalar registers or the vector ones:
//   from the region's index by div_small, whose value lies in a vector register,
//   157 registers and 60 scalar ones spilled;
//   from the item's row and column, 112 registers, which let two workgroups past
//   256 threads share a CU (WIDE), and 116 spilled.
// 64 frames of three levels, 40-pixel cells, 256 threads 192.5 us by the index and
// 209.2 by row and column; regions of 128 pixels, 512 threads and 2 a CU, 235 and 159.
template <bool WIDE>
__global__ void __launch_bounds__(512) detect_batch_generic_kernel(const fg_job *__restrict__ jobs,
                                                                   const fg_item *__restrict__ items,
                                                                   int total, unsigned *counter) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    __shared__ int s_item;
    const Queue q = queue_of(counter);
    for (int k = 0;; ++k) {
        __syncthreads();   // every wave has read the previous s_item
        if (threadIdx.x == 0) {
            long long pos = q.first + (long long)k * q.n;
            if (k >= 2) pos = 2LL * q.n + queue_ticket(q);
            s_item = queue_item(q, pos, total);
        }
        __syncthreads();
        const int item = s_item;
        if (item >= total) break;
        const fg_item it = items[item];
        const fg_job &J = jobs[it.job];
        const int column = (int)(it.region & (FG_WHOLE - 1)), row = (int)(it.region >> 16);
        detect_region(J, WIDE ? region_at(J, column, row) : region_of(J, row * J.rx + column), smem);
    }
    queue_exit(counter);
}

// The pyramid alone: up to PYR_STEP levels above `src` in one launch.  A wave
// takes 256 x 32 pixels of src, a lane a 16 x 8 block of them: eight 16-byte
// loads in flight, from which it holds 8 x 4 pixels of the next level, 4 x 2 of
// the second and 2 x 1 of the third in registers.  The fourth and fifth come
// from the wave's third through 128 bytes of LDS, so no level is read back and
// no workgroup barrier is needed.  What bounds it is the launch and one round
// of loads: 1920x1080 with 4 levels, read once and written once, takes 3.0 us
// (4.0 a call), where a launch per level took 9 to 14 us a call.
constexpr int PYR_STEP = 5;
struct PyrArgs {
    const uint8_t *src;
    int32_t w, h, pitch;    // of src
    int32_t n;              // levels to build, 1 .. PYR_STEP
    uint8_t *lvl[PYR_STEP];
    int32_t lw[PYR_STEP], lh[PYR_STEP], lpitch[PYR_STEP];
};

// Pixels x .. x+N-1 of row y of built level i (N = 1, 2, 4, 8; x a multiple of
// N), clipped to the level.
template <int N>
__device__ __forceinline__ void pyr_store(const PyrArgs &A, int i, int x, int y, uint64_t v) {
    if (y >= A.lh[i] || x >= A.lw[i]) return;
    uint8_t *d = A.lvl[i] + (ptrdiff_t)y * A.lpitch[i] + x;
    if (x + N <= A.lw[i]) {
        if constexpr (N == 8) gstore<uint64_t>(d, v);
        else if constexpr (N == 4) gstore<uint32_t>(d, (uint32_t)v);
        else if constexpr (N == 2) gstore<uint16_t>(d, (uint16_t)v);
        else gstore<uint8_t>(d, (uint8_t)v);
    } else {
        for (int q = 0; q < A.lw[i] - x; ++q) gstore<uint8_t>(d + q, (uint8_t)(v >> (8 * q)));
    }
}

__global__ void __launch_bounds__(64) pyr_kernel(PyrArgs A) {
    __shared__ uint8_t third[4][32], fourth[2][16];
    const int lane = threadIdx.x, tx = lane & 15, ty = lane >> 4;
    const int x0 = 256 * blockIdx.x + 16 * tx, y0 = 32 * blockIdx.y + 8 * ty;
    u32x4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = u32x4{0u, 0u, 0u, 0u};   // rows and columns past the plane feed no pixel of a level
        if (y0 + j < A.h && x0 < A.w) v[j] = gload<u32x4>(A.src + (ptrdiff_t)(y0 + j) * A.pitch + x0);
    }
    uint2 a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const u32x4 t = v[2 * j], b = v[2 * j + 1];
        a[j] = make_uint2(halve4(make_uint2(t.x, t.y), make_uint2(b.x, b.y)),
                          halve4(make_uint2(t.z, t.w), make_uint2(b.z, b.w)));
        pyr_store<8>(A, 0, x0 >> 1, (y0 >> 1) + j, (uint64_t)a[j].y << 32 | a[j].x);
    }
    if (A.n < 2) return;
    uint32_t b[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        b[j] = halve4(a[2 * j], a[2 * j + 1]);
        pyr_store<4>(A, 1, x0 >> 2, (y0 >> 2) + j, b[j]);
    }
    if (A.n < 3) return;
    const uint32_t c = halve4(make_uint2(b[0], 0u), make_uint2(b[1], 0u)) & 0xFFFFu;
    pyr_store<2>(A, 2, x0 >> 3, y0 >> 3, c);
    if (A.n < 4) return;
    *(uint16_t *)&third[ty][2 * tx] = (uint16_t)c;
    wave_sync();
    if (lane < 32) {   // 16 x 2 pixels
        const int x = lane & 15, y = lane >> 4;
        const uint32_t d = (third[2 * y][2 * x] + third[2 * y][2 * x + 1] + third[2 * y + 1][2 * x] +
                            third[2 * y + 1][2 * x + 1] + 2u) >> 2;
        fourth[y][x] = (uint8_t)d;
        pyr_store<1>(A, 3, 16 * blockIdx.x + x, 2 * blockIdx.y + y, d);
    }
    wave_sync();
    if (A.n < 5 || lane >= 8) return;   // 8 x 1 pixels
    const uint32_t e = (fourth[0][2 * lane] + fourth[0][2 * lane + 1] + fourth[1][2 * lane] +
                        fourth[1][2 * lane + 1] + 2u) >> 2;
    pyr_store<1>(A, 4, 8 * blockIdx.x + lane, blockIdx.y, e);
}

// A submission's tables, from pinned host memory to their device copy, one
// 8-byte word a thread.  Bound by one trip over the host link.  The copy engine
// takes the stream from the kernels and back: a submission's upload cost 17 us
// of the 85 of 8 mixed frames that way, 7 of 74 this way.  The loads are of system
// scope, so they never see what an earlier submission left in a cache.
__global__ void __launch_bounds__(256) upload_kernel(uint64_t *__restrict__ dst, const uint64_t *src, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n)
        gstore<uint64_t>(dst + i, __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM));
}

}  // namespace

hipError_t fg_launch_upload(void *dev, const void *host, size_t bytes, hipStream_t s) {
    const int n = (int)(bytes / 8);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(upload_kernel, dim3((n + 255) / 256), dim3(256), 0, s, (uint64_t *)dev,
                       (const uint64_t *)host, n);
    return hipGetLastError();
}

void fg_job_layout(fg_job &j, const fg_launch &L) {
    j.gw = (j.w[0] + j.cell - 1) / j.cell;
    j.gh = (j.h[0] + j.cell - 1) / j.cell;
    // cells per region side: a multiple of 16/gcd(cell,16), so regions and
    // sub-tiles start on 16-pixel boundaries
    int g = 16;
    while (j.cell % g) g >>= 1;
    const int m = 16 / g;
    int rc = L.region / j.cell;
    rc = (rc + m - 1) / m * m;
    if (rc < m) rc = m;
    if (rc > MAX_RCELLS) rc = MAX_RCELLS / m * m;
    j.rcells = rc;
    j.rx = (j.gw + rc - 1) / rc;
    j.ry = (j.gh + rc - 1) / rc;
}

hipError_t fg_launch_pyramid(const fg_job &j, hipStream_t s) {
    for (int k = 1; k < j.levels; k += PYR_STEP) {
        PyrArgs A = {};
        A.src = j.lvl[k - 1];
        A.w = j.w[k - 1];
        A.h = j.h[k - 1];
        A.pitch = j.pitch[k - 1];
        A.n = j.levels - k < PYR_STEP ? j.levels - k : PYR_STEP;
        for (int i = 0; i < A.n; ++i) {
            A.lvl[i] = j.lvl[k + i];
            A.lw[i] = j.w[k + i];
            A.lh[i] = j.h[k + i];
            A.lpitch[i] = j.pitch[k + i];
        }
        hipLaunchKernelGGL(pyr_kernel, dim3((A.w + 255) / 256, (A.h + 31) / 32), dim3(64), 0, s, A);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The passes over levels MAX_FUSED.. of one frame, in order.
static hipError_t launch_upper(const fg_job &j, const fg_launch &L, bool scores, hipStream_t s) {
    const int c = fg_upper_cells(j.cell, j.rcells);
    const dim3 n((j.gw + c - 1) / c, (j.gh + c - 1) / c);
    if (j.levels > 3)
        hipLaunchKernelGGL((scores ? upper_plain_kernel<3, true> : upper_plain_kernel<3, false>), n,
                           dim3(L.block), fg_smem_bytes(L.block), s, j);
    if (j.levels > 6)
        hipLaunchKernelGGL((scores ? upper_plain_kernel<6, true> : upper_plain_kernel<6, false>), n,
                           dim3(L.block), fg_smem_bytes(L.block), s, j);
    return hipGetLastError();
}

// Whether every region of the frame is one fused sub-tile that one workgroup
// can stage at once (24 quads of 8 threads).
static bool single_regions(const fg_job &j, const fg_launch &L) { return j.rcells * j.cell <= SUB && L.block >= 256; }

// The kernel whose whole regions (Whole) are the frame's: 64 or 32 pixels a
// side, which the default rule gives, three levels and more or one.  Regions of
// another side or of two levels take the general set-up in it: 1920x1080 with two
// levels 12.0 us (12.8 in detect_plain_kernel, which they took before), with three
// and 48-pixel cells 14.3 (15.8), 640x480 with two 7.4 (8.0).
template <int SIDE>
static void (*single_kernel(int levels, bool scores))(fg_job) {
    if (levels == 1) return scores ? score_single_kernel<SIDE, 1> : detect_single_kernel<SIDE, 1>;
    return scores ? score_single_kernel<SIDE, 3> : detect_single_kernel<SIDE, 3>;
}

static hipError_t launch_frame(const fg_job &j, const fg_launch &L, bool scores, hipStream_t s) {
    const int side = j.rcells * j.cell;
    void (*kernel)(fg_job) = scores ? score_plain_kernel : detect_plain_kernel;
    if (single_regions(j, L)) kernel = side <= 32 ? single_kernel<32>(j.levels, scores) : single_kernel<SUB>(j.levels, scores);
    hipLaunchKernelGGL(kernel, dim3(j.rx * j.ry), dim3(L.block), fg_smem_bytes(L.block), s, j);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_upper(j, L, scores, s);
}

hipError_t fg_launch_plain(const fg_job &j, const fg_launch &L, hipStream_t s) { return launch_frame(j, L, false, s); }

hipError_t fg_launch_score_maps(const fg_job &j, const fg_launch &L, hipStream_t s) {
    return launch_frame(j, L, true, s);
}

hipError_t fg_launch_nms_grid(const fg_job &j, int radius, hipStream_t s) {
    const dim3 grid(j.rx * j.ry), block(NMS_THREADS);
    switch (radius) {
        case 1: hipLaunchKernelGGL(nms_grid_kernel<1>, grid, block, NmsTiles<1>::BYTES, s, j); break;
        case 2: hipLaunchKernelGGL(nms_grid_kernel<2>, grid, block, NmsTiles<2>::BYTES, s, j); break;
        case 3: hipLaunchKernelGGL(nms_grid_kernel<3>, grid, block, NmsTiles<3>::BYTES, s, j); break;
        default: hipLaunchKernelGGL(nms_grid_kernel<4>, grid, block, NmsTiles<4>::BYTES, s, j); break;
    }
    return hipGetLastError();
}

hipError_t fg_launch_batch(const fg_job *jobs_dev, const fg_item *items, const fg_batch_work &work, int total_upper,
                           int max_levels, unsigned *counter, const fg_launch &L, hipStream_t s) {
    int blocks = L.num_cu * L.blocks_per_cu;
    if (blocks > work.total) blocks = work.total;
    if (blocks < 1) blocks = 1;
    void (*kernel)(const fg_job *, const fg_item *, int, unsigned *) = nullptr;
    switch (fg_choose_batch(work, L)) {
        case fg_batch_kernel::WHOLE: kernel = detect_batch_kernel; break;
        case fg_batch_kernel::ANY: kernel = detect_batch_any_kernel; break;
        case fg_batch_kernel::GENERIC_WIDE: kernel = detect_batch_generic_kernel<true>; break;
        case fg_batch_kernel::GENERIC: kernel = detect_batch_generic_kernel<false>; break;
    }
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(L.block), fg_smem_bytes(L.block), s, jobs_dev, items, work.total,
                       counter);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || max_levels <= MAX_FUSED) return e;
    hipLaunchKernelGGL(upper_batch_kernel<3>, dim3(total_upper), dim3(L.block), fg_smem_bytes(L.block), s, jobs_dev,
                       items + work.total);
    if (max_levels > 2 * MAX_FUSED)
        hipLaunchKernelGGL(upper_batch_kernel<6>, dim3(total_upper), dim3(L.block), fg_smem_bytes(L.block), s,
                           jobs_dev, items + work.total);
    return hipGetLastError();
}
