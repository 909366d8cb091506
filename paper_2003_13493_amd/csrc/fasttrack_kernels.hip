// Lucas-Kanade feature tracking on gfx950 (Section II-E).
//
// The pyramidal, approximated simultaneous inverse compositional tracker:
// translation t = (tx, ty) plus affine illumination (alpha, beta), with the
// steepest-descent rows U(x) = [(1+alpha) dT/dx, (1+alpha) dT/dy, T(x), 1] and
// the Hessian H = sum U U^T fixed per level at the alpha the level starts with.
//
// One wave64 per feature, as the paper assigns one warp per feature: a 16x16
// patch is 4 pixels per lane, an 8x8 patch 1 pixel per lane, so every lane
// runs the same iterations and exits the same level.  The patch-wide sums
// (the entries of H once per level, the 4-vector sum of U r per iteration) are
// DPP reductions read from the wave's last lane, so every lane holds the same
// value and takes identical decisions.  Arithmetic is fp32.
//
// What bounds it: with 100 features the chain of the slowest one, a wave alone
// on its SIMD; with 10,000 the vector issue (2642 instructions a feature, 43
// of the 45 us).  With a patch's bytes all loaded before the first is used (four
// waits an iteration became one), a lane's 32-bit offsets to a scalar base, the
// sums reduced side by side, bytes and tests kept while the pixel position stays
// and an iteration's four sums in one register, 752x480, 3 levels: 100 features
// 18.7 -> 11.9 us, 1920x1080, 10,000 features 70.9 -> 44.6, every estimate bit for
// bit.
//
// Every sample of a patch sits at p + t + (integer offset), so all of them
// share one fractional part: positions are split into an integer base and a
// fraction in [0, 1), which keeps the bilinear weights exact to fp32 at any
// frame size and makes the border tests integer comparisons.
#include <hip/hip_runtime.h>

#include "fg_internal.h"

namespace {

// Features (waves) per workgroup.  One spreads a small feature set over the
// most compute units (100 features: 100 CUs instead of 25), which measured
// 2-3% faster than four at 100 and at 10,000 features.
constexpr int TRACK_WAVES = 1;

// v plus its DPP-permuted copy (one instruction, no LDS traffic); a lane the
// control gives nothing adds 0
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    const int p = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true);
    return v + __builtin_bit_cast(float, p);
}

__device__ __forceinline__ float lane_value(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// Sums over the wave of N values, wave-uniform: within each row of 16 lanes by
// swapping neighbours (quad_perm 1,0,3,2 and 2,3,0,1), halves of 8
// (row_half_mirror) and halves of the row (row_mirror), then each row's sum into
// the next row (row 3 holds r2 + r3, row 1 r0 + r1), then row 1's into row 3,
// whose last lane is read: (r0 + r1) + (r2 + r3).  The N chains run side by
// side, step by step, so no step waits for the one before it (a DPP operand
// needs two wait states).
template <int N>
__device__ __forceinline__ void wave_sums(float (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = dpp_add<0xB1>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = dpp_add<0x4E>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = dpp_add<0x141>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = dpp_add<0x140>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = dpp_add<0x142>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = dpp_add<0x143>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = lane_value(v[i], 63);
}

// v plus itself with even and odd rows of 16 lanes, or the wave's halves, swapped.
__device__ __forceinline__ float add_rows(float v) {
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float add_halves(float v) {
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Sums over quads of four values, value (lane & 3) in each lane: neighbours are
// added (quad_perm 1,0,3,2), even lanes keep one value of a pair and odd ones
// the other, and the same two lanes apart (2,3,0,1).
__device__ __forceinline__ float quad_sums(float a, float b, float c, float d) {
    const int lane = threadIdx.x & 63;
    a = dpp_add<0xB1>(a);
    b = dpp_add<0xB1>(b);
    c = dpp_add<0xB1>(c);
    d = dpp_add<0xB1>(d);
    const float ab = lane & 1 ? b : a, cd = lane & 1 ? d : c;
    const float abab = dpp_add<0x4E>(ab), cdcd = dpp_add<0x4E>(cd);
    return lane & 2 ? cdcd : abab;
}

// wave_sums of an iteration's four values, the same additions in 17 instructions
// instead of 24: once quads are summed one register holds all four.  Quads are
// added to the quad before (row_ror:4) and two before (row_ror:8), which in odd
// quads is (q0 + q1) + (q2 + q3), then rows and halves, (r0 + r1) + (r2 + r3).
// 10,000 features 46.7 -> 44.4 us, 100 alike.
__device__ __forceinline__ void wave_sums4(float (&b)[4]) {
    float v = dpp_add<0x124>(quad_sums(b[0], b[1], b[2], b[3]));
    v = add_halves(add_rows(dpp_add<0x128>(v)));
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = lane_value(v, 4 + i);
}

__device__ __forceinline__ float uniform(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// Between a and b, and the same with the other product rounded: which of the
// two a sample takes is written out, so that estimates do not depend on how the
// compiler fuses the sums around it.
__device__ __forceinline__ float lerp(float a, float b, float t) { return __builtin_fmaf(1.0f - t, a, t * b); }
__device__ __forceinline__ float lerp_b(float a, float b, float t) { return __builtin_fmaf(t, b, (1.0f - t) * a); }

// a * b, rounded before anything is added to it.
__device__ __forceinline__ float product(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}

// Bilinear sample of a b / c d at the shared fraction (ax, ay).
__device__ __forceinline__ float bilinear(float a, float b, float c, float d, float ax, float ay) {
    return lerp(lerp(a, b, ax), lerp(c, d, ax), ay);
}

__device__ __forceinline__ float byte_of(uint32_t w, int i) { return (float)((w >> (8 * i)) & 0xFFu); }

// Bytes at any address, through the global address space, at a uniform base
// plus a lane's 32-bit offset (scalar base, one vector register of address).
typedef uint16_t __attribute__((aligned(1))) u16_at1;
typedef uint32_t __attribute__((aligned(1))) u32_at1;
template <class T>
__device__ __forceinline__ uint32_t load_at(const uint8_t *base, uint32_t offset) {
    return *(const __attribute__((address_space(1))) T *)(base + offset);
}

// The correctly rounded square root and reciprocal of x in [2^-98, 2^120] by
// Newton steps with fused residuals (Markstein's method), 8 and 3 instructions
// where the compiler's, which also take zeros, infinities and subnormals, are 16
// and 10.  That they are correctly rounded is no property of the steps alone, which
// from some starting values miss by an ulp, but of the steps and gfx950's v_rsq_f32
// and v_rcp_f32: tests/test_gpu_rounding.py compares all mantissas.
__device__ __forceinline__ float sqrt_rounded(float x) {
    const float y = __builtin_amdgcn_rsqf(x);
    const float g = x * y, h = 0.5f * y, r = __builtin_fmaf(-h, g, 0.5f);
    const float g1 = __builtin_fmaf(g, r, g), h1 = __builtin_fmaf(h, r, h);
    return __builtin_fmaf(__builtin_fmaf(-g1, g1, x), h1, g1);
}
__device__ __forceinline__ float rcp_rounded(float x) {
    const float y = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(__builtin_fmaf(-x, y, 1.0f), y, y);
}

template <int S>
__device__ void track_level(const fg_track_args &A, int k, float pxf, int pxi, float pyf, int pyi, float &tkx,
                            float &tky, float &alpha, float &beta, int &total, int &status) {
    constexpr int NP = S * S / 64;   // pixels per lane: column lane % S, rows lane / S + 64 / S * m
    constexpr int HALF = S / 2;
    const int lane = threadIdx.x & 63;
    const uint8_t *T = A.tpl[k], *I = A.img[k];
    const int tp = A.tpitch[k], ip = A.ipitch[k], W = A.w[k], H = A.h[k];
    // the level's parameters in one wait: the compiler moves each load to its
    // first use, where the wave waits for it again
    asm volatile("" ::"s"(T), "s"(I), "s"(tp), "s"(ip), "s"(W), "s"(H));

    // template patch plus the gradient margin: x in [p-HALF-1, p+HALF] usable
    if (pxi - HALF - 1 < 0 || pyi - HALF - 1 < 0 || pxi + HALF > W - 2 || pyi + HALF > H - 2) {
        status = FAST_TRACK_TEMPLATE_OUTSIDE;
        return;
    }
    const float g = 1.0f + alpha;
    float tv[NP], ux[NP], uy[NP];
    float h[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};   // 00 01 02 03 11 12 13 22 23
    {
        // the 12 bytes behind a pixel's five samples: columns x-1 .. x+2 of
        // rows y and y+1, columns x and x+1 of rows y-1 and y+2, all in flight
        // before the first is used
        const uint8_t *base = T + (ptrdiff_t)(pyi - HALF - 1) * tp + (pxi - HALF - 1);
        uint32_t above[NP], here[NP], below[NP], under[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) {
            const uint32_t o = (uint32_t)((lane / S + 64 / S * m) * tp + lane % S);
            above[m] = load_at<u16_at1>(base + 1, o);
            here[m] = load_at<u32_at1>(base + tp, o);
            below[m] = load_at<u32_at1>(base + 2 * (ptrdiff_t)tp, o);
            under[m] = load_at<u16_at1>(base + 3 * (ptrdiff_t)tp + 1, o);
        }
#pragma unroll
        for (int m = 0; m < NP; ++m) {
            const float p0 = byte_of(here[m], 0), p1 = byte_of(here[m], 1), p2 = byte_of(here[m], 2),
                        p3 = byte_of(here[m], 3);
            const float q0 = byte_of(below[m], 0), q1 = byte_of(below[m], 1), q2 = byte_of(below[m], 2),
                        q3 = byte_of(below[m], 3);
            const float t = bilinear(p1, p2, q1, q2, pxf, pyf);
            const float gx = 0.5f * (bilinear(p2, p3, q2, q3, pxf, pyf) -
                                     lerp(lerp_b(p0, p1, pxf), lerp_b(q0, q1, pxf), pyf));
            const float gy = 0.5f * (bilinear(q1, q2, byte_of(under[m], 0), byte_of(under[m], 1), pxf, pyf) -
                                     bilinear(byte_of(above[m], 0), byte_of(above[m], 1), p1, p2, pxf, pyf));
            tv[m] = t;
            ux[m] = product(g, gx);
            uy[m] = product(g, gy);
            h[0] += ux[m] * ux[m];
            h[1] += ux[m] * uy[m];
            h[2] += ux[m] * t;
            h[3] += ux[m];
            h[4] += uy[m] * uy[m];
            h[5] += uy[m] * t;
            h[6] += uy[m];
            h[7] += t * t;
            h[8] += t;
        }
    }
    wave_sums(h);
    const bool gain = A.mode & FAST_TRACK_GAIN, offset = A.mode & FAST_TRACK_OFFSET;
    // Inactive parameters get an identity row and column and a zero right-hand
    // side, so their increment is 0 and the active block factors as it would
    // on its own.
    float M[4][4];
    M[0][0] = h[0];
    M[1][0] = h[1];
    M[1][1] = h[4];
    M[2][0] = gain ? h[2] : 0.0f;
    M[2][1] = gain ? h[5] : 0.0f;
    M[2][2] = gain ? h[7] : 1.0f;
    M[3][0] = offset ? h[3] : 0.0f;
    M[3][1] = offset ? h[6] : 0.0f;
    M[3][2] = gain && offset ? h[8] : 0.0f;
    M[3][3] = offset ? (float)(S * S) : 1.0f;
    // Cholesky factor, with the reciprocals of its diagonal kept so the
    // per-iteration solve has no divisions; singular when a pivot falls to
    // 1e-6 of its diagonal entry
    float L[4][4] = {}, inv[4];
    bool singular = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            float s = M[i][j];
#pragma unroll
            for (int q = 0; q < j; ++q) s -= L[i][q] * L[j][q];
            if (i == j) {
                singular |= !(s > 1e-6f * M[i][i]);
                if (s >= 0x1p-90f && s <= 0x1p+120f) {   // uniform
                    inv[i] = rcp_rounded(sqrt_rounded(s));
                } else {
                    const float l = sqrtf(fmaxf(s, 0.0f));
                    inv[i] = l > 0.0f ? 1.0f / l : 0.0f;
                }
            } else {
                L[i][j] = s * inv[j];
            }
        }
    }

    uint32_t io[NP];   // this lane's pixels in the image patch
#pragma unroll
    for (int m = 0; m < NP; ++m) io[m] = (uint32_t)((lane / S + 64 / S * m) * ip + lane % S);
    const float eps2 = A.eps * A.eps;
    float pa[NP], pb[NP], pc[NP], pd[NP];   // the image patch at the pixel (pxi + fpx, pyi + fpy)
    float fpx = __builtin_nanf(""), fpy = fpx;
    for (int it = 0; it < A.max_iter; ++it) {
        const float fx = pxf + tkx, fy = pyf + tky;
        const float flx = floorf(fx), fly = floorf(fy), ax = fx - flx, ay = fy - fly;
        // the patch's bytes, all in flight before the first is used, from a
        // scalar base and a lane's 32-bit offset (a global load of the same
        // bytes takes a 64-bit vector addition each).  Steps soon are fractions
        // of a pixel: the bytes of the last iteration mostly serve again, and
        // with them what was tested of their position (never for a NaN, which
        // equals nothing)
        if (!(flx == fpx && fly == fpy)) {
            // a non-finite or huge estimate is outside (keeps the integer parts small)
            if (!(fabsf(fx) < 65536.0f && fabsf(fy) < 65536.0f)) {
                status = FAST_TRACK_LOST_OUTSIDE;
                return;
            }
            const int x0 = pxi + __builtin_amdgcn_readfirstlane((int)flx) - HALF;
            const int y0 = pyi + __builtin_amdgcn_readfirstlane((int)fly) - HALF;
            // warped patch: x in [x0, x0+S-1] usable
            if (x0 < 0 || y0 < 0 || x0 + S - 1 > W - 2 || y0 + S - 1 > H - 2) {
                status = FAST_TRACK_LOST_OUTSIDE;
                return;
            }
            if (singular) {
                status = FAST_TRACK_SINGULAR;
                return;
            }
            fpx = flx;
            fpy = fly;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(I + (ptrdiff_t)y0 * ip + x0), (short)0, (S + 1) * ip, 0x00020000);
            uint32_t up[NP], down[NP];
#pragma unroll
            for (int m = 0; m < NP; ++m) {
                up[m] = __builtin_amdgcn_raw_buffer_load_b16(rs, io[m], 0, 0);
                down[m] = __builtin_amdgcn_raw_buffer_load_b16(rs, io[m], ip, 0);
            }
#pragma unroll
            for (int m = 0; m < NP; ++m) {
                pa[m] = byte_of(up[m], 0);
                pb[m] = byte_of(up[m], 1);
                pc[m] = byte_of(down[m], 0);
                pd[m] = byte_of(down[m], 1);
            }
        }
        float b[4] = {0, 0, 0, 0};
#pragma unroll
        for (int m = 0; m < NP; ++m) {
            const float r = bilinear(pa[m], pb[m], pc[m], pd[m], ax, ay) - (1.0f + alpha) * tv[m] - beta;
            b[0] += ux[m] * r;
            b[1] += uy[m] * r;
            b[2] += tv[m] * r;
            b[3] += r;
        }
        wave_sums4(b);
        const float rhs[4] = {b[0], b[1], gain ? b[2] : 0.0f, offset ? b[3] : 0.0f};
        float y[4], d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float s = rhs[i];
#pragma unroll
            for (int q = 0; q < i; ++q) s -= L[i][q] * y[q];
            y[i] = s * inv[i];
        }
#pragma unroll
        for (int i = 3; i >= 0; --i) {
            float s = y[i];
#pragma unroll
            for (int q = i + 1; q < 4; ++q) s -= L[q][i] * d[q];
            d[i] = s * inv[i];
        }
        ++total;
        tkx -= d[0];
        tky -= d[1];
        alpha += d[2];
        beta += d[3];
        if (d[0] * d[0] + d[1] * d[1] < eps2) break;
    }
}

// Track feature f of A from its initial estimate (A.q, or zero when
// zero_init) and write the estimate, status and iteration count.
__device__ void track_feature(const fg_track_args &A, int f, bool zero_init) {
    // wave-uniform, also where the list may change under the compiler's eyes
    // (a launch that reads the live count): the positions that follow stay in
    // scalar registers and the tests on them are scalar branches
    const float fx = uniform(A.feats[2 * f]), fy = uniform(A.feats[2 * f + 1]);
    float tx = 0.0f, ty = 0.0f, alpha = 0.0f, beta = 0.0f;
    if (!zero_init) {
        tx = uniform(A.q[4 * f]);
        ty = uniform(A.q[4 * f + 1]);
        alpha = uniform(A.q[4 * f + 2]);
        beta = uniform(A.q[4 * f + 3]);
    }
    int total = 0, status = FAST_TRACK_OK;
    for (int k = A.levels - 1; k >= 0; --k) {
        const float scale = ldexpf(1.0f, k);
        const float px = fx / scale, py = fy / scale;   // exact: a power-of-two divide
        if (!(px >= 0.0f && py >= 0.0f && px < 65536.0f && py < 65536.0f)) {   // also NaN
            status = FAST_TRACK_TEMPLATE_OUTSIDE;
            break;
        }
        const float pxfl = floorf(px), pyfl = floorf(py);
        const int pxi = (int)pxfl, pyi = (int)pyfl;
        const float pxf = px - pxfl, pyf = py - pyfl;
        float tkx = tx / scale, tky = ty / scale;
        if (k < 2)
            track_level<16>(A, k, pxf, pxi, pyf, pyi, tkx, tky, alpha, beta, total, status);
        else
            track_level<8>(A, k, pxf, pxi, pyf, pyi, tkx, tky, alpha, beta, total, status);
        if (status == FAST_TRACK_TEMPLATE_OUTSIDE) break;
        tx = tkx * scale;
        ty = tky * scale;
        if (status != FAST_TRACK_OK) break;
    }
    if ((threadIdx.x & 63) == 0) {
        A.q[4 * f] = tx;
        A.q[4 * f + 1] = ty;
        A.q[4 * f + 2] = alpha;
        A.q[4 * f + 3] = beta;
        A.status[f] = status;
        if (A.iters) A.iters[f] = total;
    }
}

__global__ void __launch_bounds__(64 * TRACK_WAVES) track_kernel(fg_track_args A) {
    // the wave's feature, provably uniform: its loads become scalar loads and
    // the tests and loops on its position become scalar branches
    const int f = __builtin_amdgcn_readfirstlane(blockIdx.x * TRACK_WAVES + (int)(threadIdx.x >> 6));
    if (f >= A.nfeat) return;   // whole waves leave together
    track_feature(A, f, false);
}

// ---------------------------------------------------------------------------
// The detect-and-track loop of many camera streams (Section III-D's tracker
// evaluation, one step per stream), with every feature list resident in
// device memory.
//
// track_batch_kernel: one wave per feature slot of every job; a slot past the
// job's live count (read from device memory) leaves at once.  Every track
// starts from a zero estimate.

// Atomic load of a counter another launch wrote (not through the scalar cache).
__device__ __forceinline__ int load_count(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void __launch_bounds__(64) track_batch_kernel(const fg_fe_job *__restrict__ jobs, int njobs) {
    const int b = (int)blockIdx.x;
    // the job whose slot range holds b: the last one with feat_base <= b
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].feat_base <= b) lo = mid;
        else hi = mid - 1;
    }
    const fg_fe_job &J = jobs[lo];
    const int f = b - J.feat_base;
    if (!J.has_prev || f >= J.capacity) return;
    const int n = __builtin_amdgcn_readfirstlane(load_count(J.count));
    if (f >= n) return;
    track_feature(J.A, f, true);
}

// frontend_update_kernel: one workgroup per job, after its tracking.
//   1. the tracked features (status OK) move by their estimate and are kept
//      in order; the others are dropped;
//   2. when fewer than redetect_below remain, the cells holding a kept
//      feature are marked taken, and the strongest cell winners of the other
//      cells (score descending, then cell index ascending) are appended up to
//      the capacity, at their level-0 positions (x << level, y << level);
//   3. the live count and (tracked, redetected, live) are written.
constexpr int FE_THREADS = 256;
constexpr int FE_MAX_SCORE = 4096;   // scores are at most 4080
static_assert(FAST_MAX_TRACKS <= 1024 && FAST_MAX_GRID_CELLS <= 65536, "LDS sizes below");

// Inclusive prefix sum over the workgroup of one int per thread; `tot`
// receives the total.  Uses wave DPP scans and one LDS word per wave.
__device__ int block_scan(int v, int *wsum, int &tot) {
    int x = v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int before = 0;
    tot = 0;
#pragma unroll
    for (int w = 0; w < FE_THREADS / 64; ++w) {
        const int s = wsum[w];
        before += w < wave ? s : 0;
        tot += s;
    }
    return x + before;
}

__global__ void __launch_bounds__(FE_THREADS) frontend_update_kernel(const fg_fe_job *__restrict__ jobs) {
    __shared__ float2 kept[FAST_MAX_TRACKS];
    __shared__ uint32_t taken[FAST_MAX_GRID_CELLS / 32];
    __shared__ int hist[FE_MAX_SCORE];
    __shared__ uint32_t sel[FAST_MAX_TRACKS];
    __shared__ int wsum[FE_THREADS / 64];
    __shared__ int s_nsel, s_all, s_sstar, s_at;
    const fg_fe_job &J = jobs[blockIdx.x];
    const int tid = threadIdx.x;
    const int cap = J.capacity;
    const int n = J.has_prev ? min(load_count(J.count), cap) : 0;
    // 1. keep the tracked features, in order, at their new positions
    int live = 0;
    for (int base = 0; base < n; base += FE_THREADS) {
        const int i = base + tid;
        const bool keep = i < n && J.A.status[i] == FAST_TRACK_OK;
        float2 p = make_float2(0.0f, 0.0f);
        if (keep) p = make_float2(J.A.feats[2 * i] + J.A.q[4 * i], J.A.feats[2 * i + 1] + J.A.q[4 * i + 1]);
        int tot;
        const int incl = block_scan(keep ? 1 : 0, wsum, tot);
        if (keep) kept[live + incl - 1] = p;
        live += tot;
    }
    // every thread has read the count and the kept list is complete before
    // anyone reads the list or thread 0 rewrites the count
    __syncthreads();
    const int tracked = live;
    const bool redetect = live < J.redetect_below;
    const int ncells = J.gw * J.gh;
    int nsel = 0;
    if (redetect && live < cap) {
        // 2a. taken cells and the score histogram of the free winners
        for (int i = tid; i < (ncells + 31) / 32; i += FE_THREADS) taken[i] = 0u;
        for (int i = tid; i < FE_MAX_SCORE; i += FE_THREADS) hist[i] = 0;
        if (tid == 0) {
            s_all = 1;
            s_sstar = 1;
            s_at = 0;
            s_nsel = 0;
        }
        __syncthreads();
        for (int i = tid; i < live; i += FE_THREADS) {
            const float2 p = kept[i];
            const long cx = (long)floorf(p.x / (float)J.cell), cy = (long)floorf(p.y / (float)J.cell);
            const long c = cy * J.gw + cx;
            if (c >= 0 && c < ncells) atomicOr(&taken[c >> 5], 1u << (c & 31));
        }
        __syncthreads();
        for (int i = tid; i < ncells; i += FE_THREADS) {
            const int sc = J.slots[i].score;
            if (sc > 0 && !((taken[i >> 5] >> (i & 31)) & 1u)) atomicAdd(&hist[sc], 1);
        }
        __syncthreads();
        // 2b. the score s* at which the count of free winners from the top
        // reaches k = capacity - live: every winner above s* is taken, and the
        // first ones in cell order at s*.  Thread i sums the 16 bins from
        // score 4095 - 16 i down; a scan over threads counts from the top.
        const int k = cap - live;
        constexpr int PER = FE_MAX_SCORE / FE_THREADS;
        const int top = FE_MAX_SCORE - 1 - tid * PER;
        int mine = 0;
        for (int j = 0; j < PER; ++j) mine += hist[top - j];
        int tot;
        const int incl = block_scan(mine, wsum, tot);
        const int excl = incl - mine;
        if (tot > k && excl < k && incl >= k) {   // exactly one thread
            int acc = excl;
            for (int j = 0; j < PER; ++j) {
                const int h = hist[top - j];
                if (acc + h >= k) {
                    s_sstar = top - j;
                    s_at = k - acc;
                    s_all = 0;
                    break;
                }
                acc += h;
            }
        }
        __syncthreads();
        const bool take_all = s_all != 0;
        const int sstar = s_sstar, at = s_at;
        // 2c. gather the chosen winners' keys (score << 16 | 0xFFFF - cell):
        // every free winner above s* (or every one), and the first `at` at
        // s* in cell order
        int eq_seen = 0;
        for (int base = 0; base < ncells; base += FE_THREADS) {
            const int i = base + tid;
            int sc = 0;
            if (i < ncells) {
                sc = J.slots[i].score;
                if ((taken[i >> 5] >> (i & 31)) & 1u) sc = 0;
            }
            const bool hi = sc > 0 && (take_all || sc > sstar);
            const bool eq = !take_all && sc > 0 && sc == sstar;
            int tot;
            const int incl = block_scan(eq ? 1 : 0, wsum, tot);
            const bool pick = hi || (eq && eq_seen + incl <= at);
            eq_seen += tot;
            if (pick) {
                const int slot = atomicAdd(&s_nsel, 1);
                sel[slot] = ((uint32_t)sc << 16) | (0xFFFFu - (uint32_t)i);
            }
        }
        __syncthreads();
        nsel = s_nsel;
        // 2d. order them: bitonic sort, descending, over the next power of two
        int m = 1;
        while (m < nsel) m <<= 1;
        for (int i = nsel + tid; i < m; i += FE_THREADS) sel[i] = 0u;
        __syncthreads();
        for (int size = 2; size <= m; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int i = tid; i < m; i += FE_THREADS) {
                    const int j = i ^ stride;
                    if (j > i) {
                        const uint32_t a = sel[i], b = sel[j];
                        const bool desc = (i & size) == 0;
                        if (desc ? a < b : a > b) {
                            sel[i] = b;
                            sel[j] = a;
                        }
                    }
                }
                __syncthreads();
            }
        }
    }
    // 3. write the list back: kept features, then the new ones (the list is
    // the job's own output; the tracking arguments only read it)
    float *const feats = const_cast<float *>(J.A.feats);
    for (int i = tid; i < live; i += FE_THREADS) {
        feats[2 * i] = kept[i].x;
        feats[2 * i + 1] = kept[i].y;
    }
    for (int r = tid; r < nsel; r += FE_THREADS) {
        const int cellidx = (int)(0xFFFFu - (sel[r] & 0xFFFFu));
        const fast_feature w = J.slots[cellidx];
        feats[2 * (live + r)] = (float)((int)w.x << w.level);
        feats[2 * (live + r) + 1] = (float)((int)w.y << w.level);
    }
    if (tid == 0) {
        *J.count = live + nsel;
        J.info[0] = tracked;
        J.info[1] = redetect ? 1 : 0;
        J.info[2] = live + nsel;
        J.info[3] = 0;
    }
}

}  // namespace

hipError_t fg_launch_frontend(const fg_fe_job *jobs_dev, int njobs, int total_slots, hipStream_t s) {
    if (total_slots > 0) {
        hipLaunchKernelGGL(track_batch_kernel, dim3(total_slots), dim3(64), 0, s, jobs_dev, njobs);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(frontend_update_kernel, dim3(njobs), dim3(FE_THREADS), 0, s, jobs_dev);
    return hipGetLastError();
}

hipError_t fg_launch_track(const fg_track_args &A, hipStream_t s) {
    if (A.nfeat <= 0) return hipSuccess;
    const int blocks = (A.nfeat + TRACK_WAVES - 1) / TRACK_WAVES;
    hipLaunchKernelGGL(track_kernel, dim3(blocks), dim3(64 * TRACK_WAVES), 0, s, A);
    return hipGetLastError();
}
