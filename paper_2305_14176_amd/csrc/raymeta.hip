// libraymeta: radar IF synthesis from ray meta data (Section II, Eqs. 1-7)
// for gfx950.  The C ABI is declared in include/raymeta.h.
//
// Kernels:
//   prep_kernel    once per call: each hit's triangle and vertex indices
//                  range-checked and reduced to a record; for rmd_if_cube also
//                  the largest weight (sets the fixed-point scale) and the
//                  spreading kernel's Fourier transform at the output
//                  frequencies (FP64 quadrature).
//   geometry_kernel Eq. 6 for every hit of a ray and the pair-independent
//                  part of its path (FP64), once per ray and chirp; in small
//                  calls also prep_kernel's work.
//   spread_kernel  Eqs. 7, 1, 2 (rmd_if_cube): per workgroup one antenna pair,
//                  one chirp and one partition of the rays; the antenna legs
//                  and phases per ray in FP64, then each ray's phasor spread
//                  onto an oversampled periodic grid in LDS (the sum over rays
//                  as a type-1 non-uniform FFT), in 64-bit fixed point.
//   finish_kernel  per (pair, chirp): the partitions' grids summed in FP64,
//                  their inverse DFT (FP64, LDS) and the deconvolved samples.
//   synth_kernel   the same sum evaluated directly (rmd_if_cube_direct): MFMA
//                  products of phasor tiles split into fp16 high and low parts
//                  (fast time factored into 32 rows x 16 columns).
//   reduce_kernel  sums synth_kernel's partition cubes in FP64, fixed order.
//   fft_kernel     FFT of lines, 8 elements a thread (Eq. 4, one axis a pass).
//   span_kernel    Eq. 5 rule masks, one thread per ray.
//   check_kernel   counts rays with out-of-range meta data.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>

#include "raymeta.h"

namespace rmd {

constexpr int kWave = 64;
constexpr int kWaves = 4;                 // waves per synthesis workgroup
constexpr int kThreads = kWave * kWaves;
constexpr int kRows = 32;                 // MFMA tile rows m: fast-time steps of kCols samples
constexpr int kCols = 16;                 // MFMA tile columns k: consecutive samples
constexpr int kBlock = kRows * kCols;     // samples of one pass (512)
constexpr int kGroup = 16;                // rays per operand table (two MFMA blocks of 8)
constexpr int kBlockRays = 8;             // rays per 32 x 32 x 16 fp16 MFMA (K = 2 components x 8 rays)
constexpr int kSlotWords = 4;             // one lane's operand: 8 fp16 values
// Word offset of lane slot L in operand block b.  Slots are permuted within
// each run of 8 by an XOR with bits 4 and 5 of the slot and the block, so that
// the 64 scattered 4-byte writes of each step of the build fall on 64 banks
// (rows: bit 3 of the slot picks the bank half, bits 4 and 5 and the block the
// run's eight slots; columns: bits 2 and 3 are the lane's quarter, bit 5 and
// the block the rest) and a lane's 16-byte reads stay within its run; the
// block needs no padding.  The build is bound by the LDS: an XOR with the run
// index put the rows' writes two and the columns' four to a bank, and with the
// shuffles and reads the LDS was active 90 % of the time (77 % now).  us per
// call before / after, rays x pairs x chirps x samples: 50001 x 12 x 16 x 512
// 341 / 314, 20000 x 3 x 12 x 400 57.4 / 52.2, 1000 x 1 x 4 x 64 23.2 / 21.5.
__host__ __device__ constexpr int slot_word(int L, int b) {
    return kSlotWords * (L ^ (((L >> 2) & 4) | ((L >> 4) & 2) | b));
}
constexpr int kBlockWords = kSlotWords * kWave;             // 256 words per block
constexpr int kArrayWords = (kGroup / kBlockRays) * kBlockWords;
constexpr int kTableWords = 4 * kArrayWords;                // A hi, A lo, B hi, B lo
static_assert(kWaves * kTableWords >= kWaves * 2 * kBlock, "wave sums must fit in the table memory");
static_assert(kRows / (kWave / kGroup) == 8 && kCols / (kWave / kGroup) == 4,
              "the build's step trees are written for 8 rows and 4 columns per lane");

typedef __fp16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr double kC0 = 299792458.0;

// Spreading method.  The sum s[n] = sum_i c_i e^{2 pi i n theta_i}, n < N, is
// a Fourier series at N integer frequencies with non-uniform positions
// theta_i (cycles per sample, modulo 1).  With the centre index n_c = N / 2,
//   s[n_c + m] = sum_i c'_i e^{2 pi i m theta_i},  c'_i = c_i e^{2 pi i n_c theta_i},
// for m in [-N/2, N/2).  Each c'_i is spread onto a periodic grid of M >= 2N
// cells around x_i = M theta_i with a kernel psi of kTaps cells; the grid's
// inverse DFT G[m] = sum_l g[l] e^{2 pi i m l / M} then equals
// psi_hat(m / M) s[n_c + m] up to the kernel's aliasing error, psi_hat being
// the continuous Fourier transform of psi (Poisson summation).  psi is the
// "exponential of semicircle" kernel e^{beta (sqrt(1 - z^2) - 1)}, z = 2 u /
// kTaps for an offset of u cells (Barnett, Magland and af Klinteberg, SIAM J.
// Sci. Comput. 41, 2019): at 2x oversampling and 8 cells its aliasing error
// is about 1e-7 relative.  Kernel values are evaluated as one polynomial per
// tap (degree kTapDeg, fitted on the host), which keeps their float32 error at
// a few ulp; exp() of a float32 argument near -beta would lose about 1e-6.
// Degree 8 interpolates the kernel at Chebyshev points to 7e-9 of its peak
// (degree 10: 5e-9), both below float32's spacing there (6e-8), with 8 fewer
// multiply-adds per ray and pair.
constexpr int kTaps = 8;
constexpr int kTapDeg = 8;
static_assert(kTapDeg % 2 == 0 && kTaps % 2 == 0, "taps come in mirrored pairs; even degree");
constexpr double kBeta = 2.30 * kTaps;
constexpr int kMinGridLog2 = 6;          // M >= 64
constexpr int kQuad = 256;               // trapezoid intervals of the psi_hat quadrature

struct SynthArgs {
    const int32_t* mesh_tri_off;
    const int32_t* tris;
    const double* verts;
    const int32_t* ray_off;
    const int32_t* hit_mesh;
    const int32_t* hit_tri;
    const float* hit_u;
    const float* hit_v;
    const double* pairs;
    const float* weights;
    double* geo;                // [7][chirp_count][n_rays]: inner path, first hit xyz, last hit xyz
    int4* hit_rec;              // [n_hits]: vertex indices i1, i2, i3 and the bits of u (i1 < 0: bad hit)
    float* hit_rec_v;           // [n_hits]: v
    float2* partial;            // [n_parts][n_pairs][chirp_count][n_samples]
    int64_t n_hits;
    int32_t n_meshes, n_tris, n_verts, n_rays;
    int32_t n_pairs, chirp0, chirp_count, n_samples;   // chirps [chirp0, chirp0 + chirp_count) of one batch
    int32_t n_parts, rays_per_part, n_passes;
    double cyc_per_m;           // f_c / c: carrier cycles per metre of path (Eq. 1 into Eq. 2)
    double step_per_m;          // mu / (c f_s): beat cycles per sample per metre (Eqs. 1-3)
    // spreading method: partial holds [n_parts][n_pairs][chirp_count][M] grids
    double* deconv;             // [n_samples]: 1 / psi_hat((n - center) / M)
    unsigned* wmax_bits;        // [n_wmax]: partial maxima of |w_i| as float bits
    int32_t n_wmax;             // at most kWave (0: every weight is 1)
    int32_t grid_log2, center;  // M = 2^grid_log2; center n_c = n_samples / 2
    // Tap t < kTaps / 2 has the polynomial P_t(s) = E_t(s^2) + s O_t(s^2), s in
    // [-1/2, 1/2); psi is even, so tap kTaps - 1 - t is P_t(-s) = E_t - s O_t.
    float tap_even[kTaps / 2][kTapDeg / 2 + 1];   // E_t coefficients, constant term first
    float tap_odd[kTaps / 2][kTapDeg / 2];        // O_t coefficients
};

// sqrt(x) for finite x >= 0 from the hardware reciprocal square root: one
// Newton step on y = 1/sqrt(x), then one correction of the root s = x y,
// s + (y / 2)(x - s^2) (Markstein's method): each step doubles the correct
// bits, so from the instruction's 2^-20 or better the result is within a few
// ulp, against about 25 instructions for a correctly rounded root.  The
// antenna legs (tens of metres at 257 carrier cycles per metre) need about
// 1e-13 relative, and so do the inner paths.  x = 0 gives 0.
__device__ inline double sqrt_leg(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double hy = 0.5 * y;
    y = fma(hy, fma(-x, y * y, 1.0), y);
    const double sr = x * y;
    const double r = fma(-sr, sr, x);
    const double out = fma(0.5 * y, r, sr);
    return x == 0.0 ? 0.0 : out;
}

__device__ inline double leg3(double ax, double ay, double az, double bx, double by, double bz) {
    const double dx = ax - bx, dy = ay - by, dz = az - bz;
    return sqrt_leg(dx * dx + dy * dy + dz * dz);
}

// Eq. 6 for hit k on the snapshot `v` (n_verts x 3); false if any index of
// the hit is out of range.
__device__ inline bool hit_point(const SynthArgs& a, const double* __restrict__ v, int64_t k,
                                 double& px, double& py, double& pz) {
    const int32_t m = a.hit_mesh[k];
    if (m < 0 || m >= a.n_meshes) return false;
    const int32_t t0 = a.mesh_tri_off[m], t1 = a.mesh_tri_off[m + 1];
    const int32_t b = a.hit_tri[k];
    if (b < 0 || t0 < 0 || t1 > a.n_tris || b >= t1 - t0) return false;
    const int32_t t = t0 + b;
    const int32_t i1 = a.tris[3 * t], i2 = a.tris[3 * t + 1], i3 = a.tris[3 * t + 2];
    if ((unsigned)i1 >= (unsigned)a.n_verts || (unsigned)i2 >= (unsigned)a.n_verts ||
        (unsigned)i3 >= (unsigned)a.n_verts)
        return false;
    const double u = a.hit_u[k], w = a.hit_v[k];
    const double g = 1.0 - u - w;
    const double* v1 = v + 3 * (int64_t)i1;
    const double* v2 = v + 3 * (int64_t)i2;
    const double* v3 = v + 3 * (int64_t)i3;
    px = g * v1[0] + u * v2[0] + w * v3[0];
    py = g * v1[1] + u * v2[1] + w * v3[1];
    pz = g * v1[2] + u * v2[2] + w * v3[2];
    return true;
}

// Hit k resolved: the vertex indices of its triangle and its barycentric u, or
// i1 = -1 if any index of the hit is out of range.
__device__ inline int4 resolve_hit(const SynthArgs& a, int64_t k) {
    int4 r = make_int4(-1, 0, 0, 0);
    const int32_t m = a.hit_mesh[k];
    if (m >= 0 && m < a.n_meshes) {
        const int32_t t0 = a.mesh_tri_off[m], t1 = a.mesh_tri_off[m + 1];
        const int32_t b = a.hit_tri[k];
        if (b >= 0 && t0 >= 0 && t1 <= a.n_tris && b < t1 - t0) {
            const int32_t t = t0 + b;
            const int32_t i1 = a.tris[3 * t], i2 = a.tris[3 * t + 1], i3 = a.tris[3 * t + 2];
            if ((unsigned)i1 < (unsigned)a.n_verts && (unsigned)i2 < (unsigned)a.n_verts &&
                (unsigned)i3 < (unsigned)a.n_verts)
                r = make_int4(i1, i2, i3, __float_as_int(a.hit_u[k]));
        }
    }
    return r;
}

// The tables of a call, by blocks of kPrepThreads threads: its deconvolution
// factors and its largest weight (spreading method only).
constexpr int kPrepThreads = 256;

// deconv[n] = 1 / psi_hat((n - center) / M), psi_hat(xi) the integral of
// psi(u) cos(2 pi xi u) over the kernel's support |u| <= kTaps / 2 (psi is
// even), by the trapezoid rule with kQuad intervals in FP64 (psi falls to
// e^{-beta} at the ends of its support, where the rule's error vanishes with
// it).  One wave per n; the lanes' partial sums are combined in a fixed order.
__device__ inline void deconv_block(const SynthArgs& a, int block) {
    const int n = block * (kPrepThreads / kWave) + (int)(threadIdx.x / kWave);
    const int lane = threadIdx.x & (kWave - 1);
    if (n >= a.n_samples) return;
    const double xi = (double)(n - a.center) / (double)(1 << a.grid_log2);
    const double h = (double)kTaps / kQuad;
    double acc = 0.0;
    for (int i = lane; i <= kQuad; i += kWave) {
        const double u = -0.5 * kTaps + i * h;
        const double z = 2.0 * u / kTaps;
        const double psi = exp(kBeta * (sqrt(fmax(0.0, 1.0 - z * z)) - 1.0));
        acc += ((i == 0 || i == kQuad) ? 0.5 * h : h) * psi * cospi(2.0 * xi * u);
    }
    for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) a.deconv[n] = 1.0 / acc;
}

// The float bits of max |w_i| over the block's share of the rays (nonnegative
// floats order like their bit patterns).
__device__ inline void wmax_block(const SynthArgs& a, int block) {
    __shared__ unsigned wave_max[kPrepThreads / kWave];
    unsigned m = 0u;
    const int64_t stride = (int64_t)a.n_wmax * kPrepThreads;
    int64_t i = (int64_t)block * kPrepThreads + threadIdx.x;
    for (; i + 7 * stride < a.n_rays; i += 8 * stride) {        // eight loads in flight
        float w[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) w[c] = a.weights[i + c * stride];
#pragma unroll
        for (int c = 0; c < 8; ++c) m = max(m, __float_as_uint(fabsf(w[c])));
    }
    for (; i < a.n_rays; i += stride) m = max(m, __float_as_uint(fabsf(a.weights[i])));
    for (int off = kWave / 2; off > 0; off >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, off));
    if ((threadIdx.x & (kWave - 1)) == 0) wave_max[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kPrepThreads / kWave; ++k) m = max(m, wave_max[k]);
        a.wmax_bits[block] = m;
    }
}

__device__ inline void table_block(const SynthArgs& a, int block) {
    if (block < a.n_wmax) wmax_block(a, block);
    else deconv_block(a, block - a.n_wmax);
}

// Once per call: every hit resolved, then the tables (blocks hit_blocks and up).
__global__ __launch_bounds__(kPrepThreads) void prep_kernel(SynthArgs a, int hit_blocks) {
    if ((int)blockIdx.x >= hit_blocks) {
        table_block(a, (int)blockIdx.x - hit_blocks);
        return;
    }
    const int64_t k = (int64_t)blockIdx.x * kPrepThreads + threadIdx.x;
    if (k >= a.n_hits) return;
    a.hit_rec[k] = resolve_hit(a, k);
    a.hit_rec_v[k] = a.hit_v[k];
}

// Eq. 6 for a resolved hit on the snapshot `v`.
__device__ inline void rec_point(const int4 r, float hv, const double* __restrict__ v, double& px, double& py,
                                 double& pz) {
    const double u = __int_as_float(r.w), w = hv;
    const double g = 1.0 - u - w;
    const double* v1 = v + 3 * (int64_t)r.x;
    const double* v2 = v + 3 * (int64_t)r.y;
    const double* v3 = v + 3 * (int64_t)r.z;
    px = g * v1[0] + u * v2[0] + w * v3[0];
    py = g * v1[1] + u * v2[1] + w * v3[1];
    pz = g * v1[2] + u * v2[2] + w * v3[2];
}

// The part of ray i's path that does not depend on the antenna pair, on the
// snapshot of chirp chirp0 + jj (Eq. 6 for every hit): the inner length from
// the first to the last hit and those two hit points.  One thread per (ray,
// chirp).  The hits' records are loaded kHitRun at a time before any vertex,
// so the common rays (up to kHitRun hits) wait for two dependent loads, not
// for one chain per hit.  The pair loop of the synthesis then only adds the
// two antenna legs.  A ray with no usable path (no hits, or out-of-range meta
// data) stores an inner length of -1.
//
// INLINE: small calls, where a launch costs more than resolving each hit once
// per chirp: the hits are resolved here, and the first n_tables blocks compute
// the call's tables (first, as they take the longest; the grid is
// one-dimensional, chirps slowest, so that they come once).
constexpr int kHitRun = 4;

template <bool INLINE>
__global__ __launch_bounds__(kPrepThreads) void geometry_kernel(SynthArgs a, int ray_blocks, int n_tables) {
    int block = blockIdx.x, jj = blockIdx.y;
    if constexpr (INLINE) {
        if (block < n_tables) {
            table_block(a, block);
            return;
        }
        jj = (block - n_tables) / ray_blocks;
        block = (block - n_tables) % ray_blocks;
    }
    const int ray = block * kPrepThreads + threadIdx.x;
    if (ray >= a.n_rays) return;
    const int64_t plane = (int64_t)a.chirp_count * a.n_rays;
    double* g = a.geo + (int64_t)jj * a.n_rays + ray;
    const int32_t b = a.ray_off[ray], e = a.ray_off[ray + 1];
    const double* v = a.verts + (int64_t)(a.chirp0 + jj) * a.n_verts * 3;
    double fx = 0, fy = 0, fz = 0, lx = 0, ly = 0, lz = 0, inner = -1.0;
    if (b >= 0 && e <= a.n_hits && e > b) {
        inner = 0.0;
        for (int64_t k0 = b; k0 < e && inner >= 0.0; k0 += kHitRun) {
            int4 r[kHitRun];
            float hv[kHitRun];
#pragma unroll
            for (int c = 0; c < kHitRun; ++c) {
                r[c] = make_int4(0, 0, 0, 0);
                hv[c] = 0.0f;
                if (k0 + c < e) {
                    if constexpr (INLINE) {
                        r[c] = resolve_hit(a, k0 + c);
                        hv[c] = a.hit_v[k0 + c];
                    } else {
                        r[c] = a.hit_rec[k0 + c];
                        hv[c] = a.hit_rec_v[k0 + c];
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < kHitRun; ++c) {
                if (k0 + c >= e) break;
                if (r[c].x < 0) {
                    inner = -1.0;
                    break;
                }
                double x, y, z;
                rec_point(r[c], hv[c], v, x, y, z);
                if (k0 + c == b) {
                    fx = x; fy = y; fz = z;
                } else {
                    inner += leg3(x, y, z, lx, ly, lz);
                }
                lx = x; ly = y; lz = z;
            }
        }
        if (inner < 0.0) fx = fy = fz = lx = ly = lz = 0.0;
    }
    g[0] = inner;
    g[plane] = fx;
    g[2 * plane] = fy;
    g[3 * plane] = fz;
    g[4 * plane] = lx;
    g[5 * plane] = ly;
    g[6 * plane] = lz;
}

// Pair-independent geometry of one ray on one batch chirp (see
// geometry_kernel) and its weight; w = 0 marks a ray that contributes nothing
// (outside the partition, or without a usable path).
struct Geo {
    double inner, fx, fy, fz, lx, ly, lz;
    float w;
};

__device__ inline Geo load_geo(const SynthArgs& a, int ray, int r1, int jj) {
    Geo g{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0f};
    if (ray >= r1) return g;
    const int64_t plane = (int64_t)a.chirp_count * a.n_rays;
    const double* p = a.geo + (int64_t)jj * a.n_rays + ray;
    g.inner = p[0];
    g.fx = p[plane];
    g.fy = p[2 * plane];
    g.fz = p[3 * plane];
    g.lx = p[4 * plane];
    g.ly = p[5 * plane];
    g.lz = p[6 * plane];
    g.w = a.weights ? a.weights[ray] : 1.0f;
    return g;
}

// Phases of a ray for pair pq, in cycles modulo 1: the path length is the
// inner path plus |p^f - x'_tx| + |p^l - x'_rx| (Eq. 7 with the traced pair's
// legs cancelled exactly); Eq. 1 turns it into the delay, Eq. 2 into
// phi = f_c tau and theta = mu tau / f_s (the phase step per sample).
struct Phases {
    double phi, theta;
    float w;
};

__device__ inline Phases ray_phases(const SynthArgs& a, const Geo& g, const double* __restrict__ pq) {
    Phases p{0.0, 0.0, 0.0f};
    if (!(g.inner >= 0.0) || g.w == 0.0f) return p;
    const double len = g.inner + leg3(g.fx, g.fy, g.fz, pq[0], pq[1], pq[2]) +
                       leg3(g.lx, g.ly, g.lz, pq[3], pq[4], pq[5]);
    const double ph = len * a.cyc_per_m;              // f_c tau
    const double th = len * a.step_per_m;             // mu tau / f_s
    p.phi = ph - floor(ph);
    p.theta = th - floor(th);
    p.w = g.w;
    return p;
}

__device__ inline double frac1(double x) { return x - floor(x); }

// e^{2 pi i x} for x in [0, 1) revolutions, hardware sine and cosine.
__device__ inline float2 cis(double x) {
    const float xf = (float)x;
    return make_float2(__builtin_amdgcn_cosf(xf), __builtin_amdgcn_sinf(xf));
}

__device__ inline float2 cmul(float2 p, float2 z) {
    return make_float2(fmaf(p.x, z.x, -p.y * z.y), fmaf(p.x, z.y, p.y * z.x));
}

// Split two float32 values into fp16 high parts (rounded toward zero) and
// fp16 low parts (the rounded remainders): x = hi + lo to about 2^-21 |x|.
// Returns the packed pairs (x in the low half, y in the high half).
__device__ inline void split2(float x, float y, uint32_t& hi, uint32_t& lo) {
    const f16x2 h = __builtin_amdgcn_cvt_pkrtz(x, y);
    const f16x2 l = __builtin_amdgcn_cvt_pkrtz(fmaf((float)h.x, -1.0f, x), fmaf((float)h.y, -1.0f, y));
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

// Workgroup (pair q, pass b, partition p, chirp j).  Fast time is split as
// n = 512 b + 16 m + k (pass b, row m < 32, column k < 16), so that
//   s[n] = sum_i A[m][i] B[i][k],  A[m][i] = w_i e^{2 pi i (phi_i + (32 b + m) 16 theta_i)},
//                                 B[i][k] = e^{2 pi i k theta_i}:
// a complex 32 x 16 product over the rays, in real form a 32 x 32 product
// with two K entries per ray: A' = (Re A, Im A) and B' = ([Re B | Im B],
// [-Im B | Re B]), which puts Re s in result columns 0-15 and Im s in
// columns 16-31.
//
// The product runs on the fp16 matrix path: every operand value is split into
// fp16 high and low parts (split2), and A'B' is formed as hi hi + hi lo + lo hi
// with float32 accumulation (the dropped lo lo term is below 2^-21 of the
// product).  One 32 x 32 x 16 MFMA takes 8 rays (K = 2 components x 8); its
// operand layout puts A'[m][kk] in lane m + 32 (kk / 8), element kk % 8, and
// B'[kk][col] in lane col + 32 (kk / 8), element kk % 8, with kk = 2 r + c for
// ray r of the block and component c.
//
// Each wave takes the partition's rays 64 at a time (one ray per lane;
// super-groups round-robin over the waves):
//   phases  lane l derives ray l's phases in FP64 (antenna legs, Eq. 1, the
//           reductions modulo one cycle) and the float32 phasor steps between
//           rows and columns;
// then, for each group of kGroup = 16 of these rays,
//   build   the four lanes r, r + 16, r + 32, r + 48 fetch ray r's phases
//           from its owner lane (cross-lane shuffles); quarter h of the wave
//           forms A rows [8 h, 8 h + 8) and B columns [4 h, 4 h + 4) from one
//           exact anchor each (phase reduced in FP64) and complex-multiply
//           steps (at most 7), splits them, and writes them into the
//           operand slots of the wave's LDS table;
//   sum     lanes run over operand slots: per 8-ray block four 16-byte LDS
//           reads and three MFMAs.
// The geometry of the next super-group is loaded before the groups run, so its
// global loads are in flight while the groups are summed.  The MFMA
// accumulates one super-group (64 rays); super-group sums are added into a
// second accumulator, which keeps the float32 sums short.  Waves combine through LDS in a fixed
// order.
//
// SIMD_WAVES: waves a SIMD, and workgroups a CU, that the registers have to
// leave room for: at 4 the kernel keeps within 128, at 3 it takes 132.
template <int SIMD_WAVES>
__global__ __launch_bounds__(kThreads, SIMD_WAVES) void synth_kernel(SynthArgs a) {
    __shared__ uint4 lds_raw[kWaves * kTableWords / 4];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // XCD-aware order: consecutive workgroup ids are dealt round-robin to the
    // 8 XCDs, so give each XCD a contiguous run of (pair, pass, partition,
    // chirp) blocks.  The pairs of one partition and chirp, which read the
    // same ray geometry, then run side by side on one XCD and share its L2.
    int g = (gridDim.x & 7) ? (int)blockIdx.x
                            : (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
    const int q = g % a.n_pairs;
    g /= a.n_pairs;
    const int pass = g % a.n_passes;
    g /= a.n_passes;
    const int part = g % a.n_parts;
    const int jj = g / a.n_parts;
    const double* pq = a.pairs + 6 * q;
    uint32_t* tw = reinterpret_cast<uint32_t*>(lds_raw) + wave * kTableWords;

    constexpr int kSplit = kWave / kGroup;           // lanes per ray in the build phase
    constexpr int kRowsPer = kRows / kSplit;         // A rows per lane (8)
    constexpr int kColsPer = kCols / kSplit;         // B columns per lane (4)
    const int ri = lane & (kGroup - 1);              // build: ray of the group
    const int h = lane / kGroup;                     // build: quarter of the rows and columns
    const int ma = pass * kRows + h * kRowsPer;      // first A row of the lane (global row index)
    const int ka = h * kColsPer;                     // first B column of the lane
    // build: where ray ri's operand values go (block, lane half, word in the slot)
    const int bk = ri / kBlockRays;
    const int hh = (ri % kBlockRays) / 4;
    const int rr = ri % 4;
    uint32_t* ahi = tw + bk * kBlockWords + rr;
    uint32_t* alo = ahi + kArrayWords;
    uint32_t* bhi = ahi + 2 * kArrayWords;
    uint32_t* blo = ahi + 3 * kArrayWords;
    const int la = h * kRowsPer + 32 * hh;           // slot of row h * 8 (+ t)
    const int lb = h * kColsPer + 32 * hh;           // slot of column h * 4 (+ t) ...
    const int lb2 = lb + kCols;                      // ... and of column 16 + h * 4 (+ t)

    f32x16 tot = {};
    const int r0 = part * a.rays_per_part;
    const int r1 = min(a.n_rays, r0 + a.rays_per_part);
    Geo gn = load_geo(a, r0 + wave * kWave + lane, r1, jj);
    for (int sbase = r0 + wave * kWave; sbase < r1; sbase += kThreads) {
        const Phases own = ray_phases(a, gn, pq);
        gn = load_geo(a, sbase + kThreads + lane, r1, jj);      // next super-group, in flight meanwhile
        const float2 own_s16 = cis(frac1(kCols * own.theta));   // step between rows
        const float2 own_s1 = cis(own.theta);                   // step between columns
        f32x16 acc[kGroup / kBlockRays] = {};   // one chain per block: consecutive MFMAs are independent
        for (int gq = 0; gq < kSplit && sbase + gq * kGroup < r1; ++gq) {
            const int src = gq * kGroup + ri;
            const double phi = __shfl(own.phi, src);
            const double theta = __shfl(own.theta, src);
            const float w = __shfl(own.w, src);
            const float2 s16 = make_float2(__shfl(own_s16.x, src), __shfl(own_s16.y, src));
            const float2 s1 = make_float2(__shfl(own_s1.x, src), __shfl(own_s1.y, src));
            {                                        // A rows ma + t: p_t = p_0 s^t
                float2 p = cis(frac1(phi + (double)ma * frac1(kCols * theta)));
                p.x *= w;
                p.y *= w;
#pragma unroll
                for (int t = 0; t < kRowsPer; ++t) {     // A'[m][0] = Re, A'[m][1] = Im
                    uint32_t hi, lo;
                    split2(p.x, p.y, hi, lo);
                    ahi[slot_word(la + t, bk)] = hi;
                    alo[slot_word(la + t, bk)] = lo;
                    p = cmul(p, s16);
                }
            }
            {                                        // B columns ka + t: q_t = q_0 s1^t
                float2 qv = cis(frac1((double)ka * theta));
#pragma unroll
                for (int t = 0; t < kColsPer; ++t) {
                    uint32_t hi, lo;
                    split2(qv.x, qv.y, hi, lo);
                    qv = cmul(qv, s1);
                    // column k: (B'[0][k], B'[1][k]) = (Re, -Im); column 16 + k: (Im, Re)
                    bhi[slot_word(lb + t, bk)] = hi ^ 0x80000000u;
                    blo[slot_word(lb + t, bk)] = lo ^ 0x80000000u;
                    bhi[slot_word(lb2 + t, bk)] = (hi >> 16) | (hi << 16);
                    blo[slot_word(lb2 + t, bk)] = (lo >> 16) | (lo << 16);
                }
            }
            __builtin_amdgcn_wave_barrier();
            // Every slot is written in every group; rays at or past the
            // partition end have A' = 0.
            constexpr int kB = kGroup / kBlockRays;
            f16x8 a_hi[kB], a_lo[kB], b_hi[kB], b_lo[kB];
#pragma unroll
            for (int b = 0; b < kB; ++b) {
                const uint32_t* base = tw + b * kBlockWords + slot_word(lane, b);
                a_hi[b] = *reinterpret_cast<const f16x8*>(base);
                a_lo[b] = *reinterpret_cast<const f16x8*>(base + kArrayWords);
                b_hi[b] = *reinterpret_cast<const f16x8*>(base + 2 * kArrayWords);
                b_lo[b] = *reinterpret_cast<const f16x8*>(base + 3 * kArrayWords);
            }
#pragma unroll
            for (int b = 0; b < kB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_hi[b], b_hi[b], acc[b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < kB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_hi[b], b_lo[b], acc[b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < kB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a_lo[b], b_hi[b], acc[b], 0, 0, 0);
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int b = 0; b < kGroup / kBlockRays; ++b) tot += acc[b];
    }

    // Result layout of the 32 x 32 MFMA: register r of lane l holds row
    // 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.  Row m, column col is
    // sample 16 m + col % 16 of the pass, real part for col < 16, imaginary
    // otherwise.  The wave sums reuse the table memory.
    __syncthreads();
    float* red = reinterpret_cast<float*>(lds_raw);
    const int c = lane >> 5, col = lane & 31;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int m = 8 * (r >> 2) + 4 * c + (r & 3);
        const int n = kCols * m + (col & (kCols - 1));
        red[wave * 2 * kBlock + 2 * n + (col >> 4)] = tot[r];
    }
    __syncthreads();
    float2* out = a.partial + (((int64_t)part * a.n_pairs + q) * a.chirp_count + jj) * (int64_t)a.n_samples;
    const int n_end = min(a.n_samples - pass * kBlock, kBlock);
    for (int n = threadIdx.x; n < n_end; n += kThreads) {
        float re = 0.f, im = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            re += red[w * 2 * kBlock + 2 * n];
            im += red[w * 2 * kBlock + 2 * n + 1];
        }
        out[pass * kBlock + n] = make_float2(re, im);
    }
}

// Workgroup (pair q, partition p, chirp j) of the spreading method.  The
// workgroup's grid of M complex cells sits in LDS as 64-bit fixed-point
// integers (real parts, then imaginary parts) with the scale 2^e chosen from
// the largest weight, 2^e max|w| in [2^29, 2^30): every contribution
// w e^{2 pi i phi'} psi is cut to an int32 multiple of 2^-e (toward zero, error
// below 2^-29 max|w|) and added with a 64-bit LDS integer atomic; a cell of a block
// receives at most n_rays contributions, so no sum exceeds 2^60.  Integer
// addition is exact and order-free, so all waves share the grid and the result
// does not depend on scheduling (LDS float atomics would not be, and on this
// chip they are several times slower than integer ones).
//
// What bounds it is the LDS: 16 atomics a ray, whose lanes meet in its banks.
// With two copies of the grid side by side, one for even and one for odd lanes,
// an atomic of 64 lanes took 13 cycles against 4 without conflicts, and the LDS
// was active 81 % of the time (vector instructions 71 %).  COPIES interleaved
// copies, lane l adding into copy l % COPIES of each cell, give each copy 32 /
// COPIES bank pairs of its own: fewer lanes can meet, on a cell or on a bank.
// us per call before / after, 12 pairs and 16 chirps: 2^20 rays, M = 1024
// 1901 / 1664; 400000 rays, M = 1024 828 / 718, 512 1002 / 662, 256 1194 / 656,
// 64 1172 / 594.  The sums are exact, so neither COPIES nor THREADS changes a bit.
//
// Each wave takes the partition's rays 64 at a time, one ray per lane (the
// same super-group order and geometry prefetch as synth_kernel): the lane forms
// the ray's phases in FP64, its grid position x = M theta, the first cell
// l0 = ceil(x - kTaps / 2) under the kernel and the offset
// s = l0 - x + (kTaps - 1) / 2 in [-1/2, 1/2), evaluates the kTaps kernel
// values by Horner's rule and adds the contributions into cells l0 .. l0 +
// kTaps - 1 (modulo M).  At the end the grid is scaled back and written as
// the partition's float32 grid.
template <int COPIES, int THREADS>
__global__ __launch_bounds__(THREADS) void spread_kernel(SynthArgs a) {
    extern __shared__ unsigned long long gq[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = 1 << a.grid_log2;
    // XCD-aware order as in synth_kernel: the pairs of one partition and chirp
    // run side by side on one XCD.
    int g = (gridDim.x & 7) ? (int)blockIdx.x
                            : (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
    const int q = g % a.n_pairs;
    g /= a.n_pairs;
    const int part = g % a.n_parts;
    const int jj = g / a.n_parts;
    const double* pq = a.pairs + 6 * q;
    // Each plane has kTaps cells of padding: padded cell i holds grid cell
    // (i - kTaps / 2) mod M, so a ray's taps are one address plus constant
    // offsets; the wrapped cells are folded back when the grid is written.
    // Lane l adds into copy l % COPIES of the grid; the copies of a cell are
    // neighbours, so each copy has 32 / COPIES of the bank pairs to itself.
    const int P = M + kTaps;
    for (int i = threadIdx.x; i < COPIES * 2 * P; i += THREADS) gq[i] = 0ull;
    // max|w| = m 2^e2, m in [1/2, 1), from the partial maxima (1 without weights)
    unsigned wbits = a.n_wmax ? (lane < a.n_wmax ? a.wmax_bits[lane] : 0u) : 0x3f800000u;
    for (int off = kWave / 2; off > 0; off >>= 1) wbits = max(wbits, (unsigned)__shfl_xor((int)wbits, off));
    int e2;
    frexpf(__uint_as_float(wbits), &e2);
    const int qexp = 30 - e2;                       // 2^qexp max|w| in [2^29, 2^30)
    __syncthreads();

    const int r0 = part * a.rays_per_part;
    const int r1 = min(a.n_rays, r0 + a.rays_per_part);
    const double fM = (double)M;
    Geo gn = load_geo(a, r0 + wave * kWave + lane, r1, jj);
    for (int sbase = r0 + wave * kWave; sbase < r1; sbase += THREADS) {
        const Phases own = ray_phases(a, gn, pq);
        gn = load_geo(a, sbase + THREADS + lane, r1, jj);      // next super-group, in flight meanwhile
        if (own.w != 0.0f) {
            const double x = own.theta * fM;                   // grid position in [0, M)
            const double l0 = ceil(x - 0.5 * kTaps);
            const float sv = (float)((l0 - x) + 0.5 * (kTaps - 1));
            float2 c = cis(frac1(own.phi + frac1((double)a.center * own.theta)));
            const float ws = ldexpf(own.w, qexp);             // weight in grid units (exact)
            c.x *= ws;
            c.y *= ws;
            // Kernel values, the mirrored taps t and kTaps - 1 - t from one
            // Horner pass over the even and odd parts in s^2.
            const float y = sv * sv;
            float k[kTaps];
#pragma unroll
            for (int t = 0; t < kTaps / 2; ++t) {
                float ev = a.tap_even[t][kTapDeg / 2];
#pragma unroll
                for (int d = kTapDeg / 2 - 1; d >= 0; --d) ev = fmaf(ev, y, a.tap_even[t][d]);
                float od = a.tap_odd[t][kTapDeg / 2 - 1];
#pragma unroll
                for (int d = kTapDeg / 2 - 2; d >= 0; --d) od = fmaf(od, y, a.tap_odd[t][d]);
                k[t] = fmaf(sv, od, ev);
                k[kTaps - 1 - t] = fmaf(-sv, od, ev);
            }
            // l0 is in [-kTaps / 2, M - kTaps / 2] for every finite theta in
            // [0, 1) (the clamp only guards non-finite pair coordinates), so
            // the taps' padded cells l0 + kTaps / 2 + t lie in [0, M + kTaps).
            const int base = min(max((int)l0, -kTaps / 2), M - kTaps / 2);
            unsigned long long* cr = gq + (base + kTaps / 2) * COPIES + (lane & (COPIES - 1));
            unsigned long long* ci = cr + P * COPIES;
#pragma unroll
            for (int t = 0; t < kTaps; ++t) {
                // |k c| < 2^31 by the choice of qexp; conversion rounds toward zero
                const long long vr = (int)(k[t] * c.x);
                const long long vi = (int)(k[t] * c.y);
                atomicAdd(cr + t * COPIES, (unsigned long long)vr);
                atomicAdd(ci + t * COPIES, (unsigned long long)vi);
            }
        }
    }
    __syncthreads();
    float2* out = a.partial + (((int64_t)part * a.n_pairs + q) * a.chirp_count + jj) * (int64_t)M;
    for (int i = threadIdx.x; i < M; i += THREADS) {
        const int h = i + kTaps / 2;                        // padded cell of grid cell i
        long long re = 0, im = 0;
#pragma unroll
        for (int cp = 0; cp < COPIES; ++cp) {
            const unsigned long long* g0 = gq + cp;
            re += (long long)g0[h * COPIES];
            im += (long long)g0[(P + h) * COPIES];
            if (i < kTaps / 2) {                            // wrapped past the end
                re += (long long)g0[(h + M) * COPIES];
                im += (long long)g0[(P + h + M) * COPIES];
            }
            if (i >= M - kTaps / 2) {                       // wrapped below the start
                re += (long long)g0[(h - M) * COPIES];
                im += (long long)g0[(P + h - M) * COPIES];
            }
        }
        out[i] = make_float2((float)ldexp((double)re, -qexp), (float)ldexp((double)im, -qexp));
    }
}

// Workgroup (pair q, batch chirp j): the partitions' grids of the block summed
// in FP64 in partition order, loaded bit-reversed; the inverse DFT
// G[m] = sum_l g[l] e^{2 pi i m l / M} by radix-2 decimation in time in FP64
// in LDS (twiddles from sincospi); then s[n] = G[(n - center) mod M] deconv[n]
// rounded once to float32 and written into the cube at chirp c0 + j.
//
// Bound by instructions, not by the sums' loads: they are mostly few, and the
// set-up of a loop with eight loads in flight costs each of the 16 waves more
// than its loads save.  us with four loads / with eight: 3072 blocks of one
// partition 43.5 / 66.5, 192 of one 6.9 / 7.4, 192 of 40 14.0 / 14.5, one of
// 118 18.9 / 20.2.
constexpr int kFinishThreads = 1024;     // one grid cell per thread at M = 1024

__global__ __launch_bounds__(kFinishThreads) void finish_kernel(SynthArgs a, float2* __restrict__ s, int n_chirps_out,
                                                              int c0) {
    extern __shared__ double2 fl[];
    const int logL = a.grid_log2, L = 1 << logL;
    double2* tw = fl;                    // L / 2 twiddles e^{+2 pi i k / L}
    double2* x = fl + L / 2;
    const int q = blockIdx.x % a.n_pairs, jj = blockIdx.x / a.n_pairs;
    for (int k = threadIdx.x; k < L / 2; k += blockDim.x) {
        double sn, cs;
        sincospi(2.0 * k / L, &sn, &cs);
        tw[k] = make_double2(cs, sn);
    }
    const int64_t stride = (int64_t)a.n_pairs * a.chirp_count * L;
    const float2* src = a.partial + ((int64_t)q * a.chirp_count + jj) * L;
    for (int l = threadIdx.x; l < L; l += blockDim.x) {
        double re = 0.0, im = 0.0;
#pragma unroll 4
        for (int p = 0; p < a.n_parts; ++p) {
            const float2 v = src[(int64_t)p * stride + l];
            re += v.x;
            im += v.y;
        }
        x[__brev((unsigned)l) >> (32 - logL)] = make_double2(re, im);
    }
    __syncthreads();
    for (int st = 0; st < logL; ++st) {
        const int half = 1 << st;
        for (int k = threadIdx.x; k < L / 2; k += blockDim.x) {
            const int pos = k & (half - 1);
            const int i0 = ((k >> st) << (st + 1)) + pos, i1 = i0 + half;
            const double2 w = tw[pos << (logL - 1 - st)];
            const double2 u = x[i0], v = x[i1];
            const double vr = v.x * w.x - v.y * w.y, vi = v.x * w.y + v.y * w.x;
            x[i0] = make_double2(u.x + vr, u.y + vi);
            x[i1] = make_double2(u.x - vr, u.y - vi);
        }
        __syncthreads();
    }
    float2* out = s + ((int64_t)q * n_chirps_out + c0 + jj) * a.n_samples;
    for (int n = threadIdx.x; n < a.n_samples; n += blockDim.x) {
        const double2 v = x[(n - a.center) & (L - 1)];
        const double f = a.deconv[n];
        out[n] = make_float2((float)(v.x * f), (float)(v.y * f));
    }
}

// Sample i of the cube: its partitions' values summed in FP64 and in order,
// eight loads in flight at a time, then four.  Bound by the latency of that
// chain.  us with four loads / with eight: 40 partitions of 98304 samples
// 13.5 / 6.2, 118 of 300 samples 29.0 / 7.5; 8 or fewer the same.
__global__ void reduce_kernel(const float2* __restrict__ partial, float2* __restrict__ s, int n_pairs, int nb,
                              int n_samples, int n_parts, int n_chirps_out, int c0) {
    const int64_t count = (int64_t)n_pairs * nb * n_samples;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    double re = 0.0, im = 0.0;
    int p = 0;
    for (; p + 8 <= n_parts; p += 8) {
        float2 v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = partial[(p + c) * count + i];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            re += v[c].x;
            im += v[c].y;
        }
    }
#pragma unroll 4
    for (; p < n_parts; ++p) {
        const float2 v = partial[p * count + i];
        re += v.x;
        im += v.y;
    }
    const int n = (int)(i % n_samples);
    const int64_t qj = i / n_samples;
    const int jj = (int)(qj % nb), q = (int)(qj / nb);
    s[((int64_t)q * n_chirps_out + c0 + jj) * n_samples + n] = make_float2((float)re, (float)im);
}

// FFT of lines of length L = 2^LOGL (Eq. 4, one axis a pass), in place or not:
// a Stockham autosort transform with E = min(8, L) elements of a line in each
// thread's registers.  The first stage (radix 2, 4 or 8, what L leaves over
// powers of 8) takes its elements straight from memory and the last one writes
// straight back, both in natural order; the radix-8 stages between them
// exchange through LDS, log8 L - 1 times.  Twiddles exp(-2 pi i k / L), k < L/2,
// are formed in FP64 and rounded once, after the loads are under way.
//
// What bounds it is latency, not the 16 bytes per sample and pass of traffic: a
// radix-2 transform in LDS paid two barriers and two LDS round trips for each of
// its log2 L stages and started from bit-reversed LDS writes.  12 x 128 x 512
// samples took 35 us for both passes of that and take 11.5 here (6.3 and 5.0 us
// of kernel: the loads, the FP64 twiddles, two exchanges and the stores one after
// another), 12 x 512 x 1024 133 and 46 (4.4 TB/s over both).
//
// STRIDED: the elements of a line are 2^lg apart and lines m, m + 1, ... are
// neighbours in memory (2^lg of them a group): lanes run over the lines, and the
// LDS holds a line's elements LB apart.  Otherwise lines are contiguous, lanes
// run along them, and the LDS pads every 8 elements by one (the stages' strides
// of 8 would fall on a quarter of the banks).
__device__ inline float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ inline float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ inline float2 mul_mi(float2 a) { return make_float2(a.y, -a.x); }   // times -i

__device__ inline void dft2(float2& a, float2& b) {
    const float2 t = csub(a, b);
    a = cadd(a, b);
    b = t;
}
__device__ inline void dft4(float2& a, float2& b, float2& c, float2& d) {     // outputs 0, 1, 2, 3 in a, b, c, d
    dft2(a, c);
    dft2(b, d);
    d = mul_mi(d);
    dft2(a, b);
    dft2(c, d);
    const float2 t = b;
    b = c;
    c = t;
}

template <int R>
__device__ inline void dft(float2 (&v)[R]) {
    if constexpr (R == 2) {
        dft2(v[0], v[1]);
    } else if constexpr (R == 4) {
        dft4(v[0], v[1], v[2], v[3]);
    } else if constexpr (R == 8) {
        dft4(v[0], v[2], v[4], v[6]);
        dft4(v[1], v[3], v[5], v[7]);
        constexpr float h = 0.70710678118654752f;
        v[3] = make_float2(h * (v[3].x + v[3].y), h * (v[3].y - v[3].x));
        v[5] = mul_mi(v[5]);
        v[7] = make_float2(h * (v[7].y - v[7].x), -h * (v[7].x + v[7].y));
#pragma unroll
        for (int k = 0; k < 8; k += 2) dft2(v[k], v[k + 1]);
        // (pairs k, k + 4) to natural order
        const float2 a1 = v[1], a2 = v[2], a3 = v[3], a4 = v[4], a5 = v[5], a6 = v[6];
        v[1] = a2; v[2] = a4; v[3] = a6; v[4] = a1; v[5] = a3; v[6] = a5;
    }
}

template <int LOGL>
struct FftPlan {
    static constexpr int L = 1 << LOGL;
    static constexpr int E = L < 8 ? L : 8;            // elements per thread
    static constexpr int TPL = L / E;                  // threads per line
    static constexpr int R0 = LOGL < 3 ? L : (LOGL % 3 == 0 ? 8 : LOGL % 3 == 1 ? 2 : 4);   // first radix
};

// The stages from NS = product of the radices done: v[q] holds element
// t + q TPL.  at(e): LDS place of the line's element e; put(e, v): the result.
template <int LOGL, int NS, int R, class At, class Put>
__device__ inline void fft_stages(float2 (&v)[FftPlan<LOGL>::E], float2* lds, const float2* tw, int t, At&& at,
                                  Put&& put) {
    using P = FftPlan<LOGL>;
    constexpr int NB = P::E / R;                       // butterflies of a thread
    constexpr bool last = NS * R == P::L;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int j = t + b * P::TPL;
        float2 u[R];
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = v[b + r * NB];
        if constexpr (NS > 1) {
            const int step = (j & (NS - 1)) * (P::L / (NS * R));
#pragma unroll
            for (int r = 1; r < R; ++r) {
                const int k = r * step;                // < L
                const float2 w = tw[k & (P::L / 2 - 1)];
                const float sg = (k & (P::L / 2)) ? -1.0f : 1.0f;
                u[r] = cmul(u[r], make_float2(sg * w.x, sg * w.y));
            }
        }
        dft<R>(u);
        const int d = (j / NS) * NS * R + (j & (NS - 1));
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (last) put(d + r * NS, u[r]);
            else lds[at(d + r * NS)] = u[r];
        }
    }
    if constexpr (!last) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < P::E; ++q) v[q] = lds[at(t + q * P::TPL)];
        if constexpr (NS * R * 8 < P::L) __syncthreads();   // the next stage writes these places again
        fft_stages<LOGL, NS * R, 8>(v, lds, tw, t, at, put);
    }
}

template <int LOGL, bool STRIDED>
__global__ __launch_bounds__(1024) void fft_kernel(const float2* in, float2* out, int lines, int lg) {
    using P = FftPlan<LOGL>;
    constexpr int L = P::L, E = P::E, TPL = P::TPL;
    extern __shared__ float2 lds[];
    float2* tw = lds;                                  // L / 2 twiddles (L > 8)
    float2* x = lds + (L > 8 ? L / 2 : 0);
    const int LB = blockDim.x / TPL;                   // lines per workgroup
    const int ln = STRIDED ? threadIdx.x % LB : threadIdx.x / TPL;
    const int t = STRIDED ? threadIdx.x / LB : threadIdx.x % TPL;
    const int m = blockIdx.x * LB + ln;
    const bool ok = m < lines;
    const int64_t base = STRIDED ? ((int64_t)(m >> lg) << (lg + LOGL)) + (m & ((1 << lg) - 1)) : (int64_t)m << LOGL;
    const int es = STRIDED ? lg : 0;                   // log2 of the element stride
    float2 v[E];
#pragma unroll
    for (int q = 0; q < E; ++q) v[q] = ok ? in[base + ((int64_t)(t + q * TPL) << es)] : make_float2(0.f, 0.f);
    if constexpr (L > 8) {
        for (int k = threadIdx.x; k < L / 2; k += blockDim.x) {
            double sn, cs;
            sincospi(-2.0 * k / L, &sn, &cs);
            tw[k] = make_float2((float)cs, (float)sn);
        }
        __syncthreads();
    }
    const int place = STRIDED ? ln : ln * (L + L / 8);
    auto at = [&](int e) { return STRIDED ? e * LB + place : place + e + (e >> 3); };
    auto put = [&](int e, float2 w) {
        if (ok) out[base + ((int64_t)e << es)] = w;
    };
    if constexpr (LOGL == 0) put(0, v[0]);
    else fft_stages<LOGL, 1, P::R0>(v, x, tw, t, at, put);
}

__global__ void span_kernel(rmd_scene sc, const uint8_t* __restrict__ in_set, rmd_span_rule rule,
                            const float* __restrict__ amp, float* __restrict__ weights) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= sc.n_rays) return;
    const int32_t b = sc.ray_off[i], e = sc.ray_off[i + 1];
    bool ok = b >= 0 && e <= sc.n_hits && e >= b;
    int inside = 0, n = 0;
    if (ok) {
        for (int64_t k = b; k < e; ++k) {
            const int32_t m = sc.hit_mesh[k];
            if (m < 0 || m >= sc.n_meshes) { ok = false; break; }
            inside += in_set[m] != 0;
            ++n;
        }
    }
    if (ok) {
        if (rule.mode == 0) ok = inside > 0;
        else if (rule.mode == 1) ok = inside == 0;
        else ok = inside == n;
        ok = ok && n >= rule.min_hits && n <= rule.max_hits;
    }
    weights[i] = ok ? (amp ? amp[i] : 1.0f) : 0.0f;
}

__global__ void zero_kernel(unsigned long long* p) { *p = 0ull; }

__global__ void check_kernel(SynthArgs a, unsigned long long* bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n_rays) return;
    const int32_t b = a.ray_off[i], e = a.ray_off[i + 1];
    bool ok = b >= 0 && e <= a.n_hits && e >= b;
    for (int64_t k = b; ok && k < e; ++k) {
        double x, y, z;
        ok = hit_point(a, a.verts, k, x, y, z);
    }
    if (!ok) atomicAdd(bad, 1ull);
}

}  // namespace rmd

// ------------------------------------------------------------------ C ABI

namespace {

thread_local std::string g_err;

rmd_status fail(rmd_status st, const std::string& msg) {
    g_err = msg;
    return st;
}

rmd_status hip_fail(hipError_t e, const char* what) {
    return fail(RMD_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

rmd_status check_scene_desc(const rmd_scene* sc) {
    if (!sc) return fail(RMD_EINVAL, "scene is NULL");
    if (sc->n_meshes <= 0 || sc->n_tris <= 0 || sc->n_verts <= 0 || sc->n_rays <= 0 || sc->n_hits < 0)
        return fail(RMD_EINVAL, "scene sizes must be positive (n_hits >= 0)");
    if (sc->n_hits > INT32_MAX) return fail(RMD_EINVAL, "n_hits above 2^31 - 1 (32-bit ray offsets)");
    if (sc->n_rays > RMD_MAX_RAYS) return fail(RMD_EINVAL, "n_rays above RMD_MAX_RAYS");
    if (!sc->mesh_tri_off || !sc->tris || !sc->verts || !sc->ray_off || !sc->hit_mesh || !sc->hit_tri ||
        !sc->hit_u || !sc->hit_v)
        return fail(RMD_EINVAL, "a scene array pointer is NULL");
    return RMD_OK;
}

// Work plan of one IF cube.  Chirps are processed in batches whose per-ray
// geometry (7 doubles per ray and chirp) fits in kGeoBudget bytes, at most
// kMaxBatch chirps.  Within a batch the rays are split into partitions so that
// the (pair, chirp, partition) workgroups fill the device several times over,
// each of four waves keeping at least four 64-ray super-groups (two, where the
// spreading takes eight waves a workgroup).  The workspace holds the
// batch's geometry, then the partition results of either method (direct:
// n_samples complex values per block; spreading: an M-cell grid per block and
// the deconvolution table), so one size serves both entry points.
constexpr int64_t kGeoBudget = int64_t(1) << 30;
constexpr int kMaxBatch = 16;

int grid_log2_for(int n_samples) {
    int l = rmd::kMinGridLog2;
    while ((1 << l) < 2 * n_samples) ++l;
    return l;
}

int64_t round256(int64_t b) { return (b + 255) / 256 * 256; }

struct Plan {
    int batch, parts, rays_per_part, grid_log2;
    int64_t geo_bytes, rec_bytes, partial_bytes, grid_bytes, deconv_bytes, total_bytes;
    int geo_sets;   // geometry buffers: 2 when there are several batches (the next one is built meanwhile)
};

Plan plan(int n_rays, int64_t n_hits, int n_pairs, int chirp_count, int n_samples) {
    Plan p{};
    const int64_t per_chirp = (int64_t)n_rays * 7 * (int64_t)sizeof(double);
    p.batch = (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)chirp_count, kMaxBatch, kGeoBudget / per_chirp}));
    const int64_t blocks = (int64_t)n_pairs * p.batch;
    const int64_t target = 8192;
    int64_t np = (target + blocks - 1) / blocks;
    const int64_t max_p = std::max<int64_t>(1, n_rays / (rmd::kThreads * 4));
    np = std::max<int64_t>(1, std::min(np, max_p));
    int64_t rpp = (n_rays + np - 1) / np;
    rpp = (rpp + rmd::kThreads - 1) / rmd::kThreads * rmd::kThreads;
    p.parts = (int)((n_rays + rpp - 1) / rpp);
    p.rays_per_part = (int)rpp;
    p.grid_log2 = grid_log2_for(n_samples);
    p.geo_bytes = round256(per_chirp * p.batch);
    p.rec_bytes = round256(n_hits * (int64_t)sizeof(int4)) + round256(n_hits * (int64_t)sizeof(float));
    p.partial_bytes = (int64_t)p.parts * blocks * n_samples * (int64_t)sizeof(float2);
    p.grid_bytes = round256((int64_t)p.parts * blocks * (int64_t(1) << p.grid_log2) * (int64_t)sizeof(float2));
    p.deconv_bytes = round256((int64_t)n_samples * (int64_t)sizeof(double)) + 256;   // + the largest weights' words
    p.geo_sets = chirp_count > p.batch ? 2 : 1;
    p.total_bytes = p.geo_sets * p.geo_bytes + p.rec_bytes + std::max(p.partial_bytes, p.grid_bytes + p.deconv_bytes);
    return p;
}

// Monomial coefficients (in s in [-1/2, 1/2]) of the degree-kTapDeg
// polynomials that interpolate the spreading kernel of taps t < kTaps / 2 at
// the kTapDeg + 1 Chebyshev points of that interval (tap t sits u = s + 1/2 -
// kTaps/2 + t cells from the ray; the nodes are symmetric, so the mirrored tap
// kTaps - 1 - t is the same polynomial at -s), split into even and odd parts.
// Solved once, in long double, by Gaussian elimination with partial pivoting.
struct TapPoly {
    float even[rmd::kTaps / 2][rmd::kTapDeg / 2 + 1];
    float odd[rmd::kTaps / 2][rmd::kTapDeg / 2];
};

const TapPoly& tap_poly() {
    static const TapPoly tp = [] {
        TapPoly r{};
        constexpr int n = rmd::kTapDeg + 1;
        const long double pi = 3.141592653589793238462643383279502884L;
        for (int t = 0; t < rmd::kTaps / 2; ++t) {
            long double A[n][n + 1];
            for (int i = 0; i < n; ++i) {
                const long double sn = 0.5L * cosl(pi * (i + 0.5L) / n);
                const long double z = (sn + 0.5L - 0.5L * rmd::kTaps + t) * 2.0L / rmd::kTaps;
                long double pw = 1.0L;
                for (int j = 0; j < n; ++j) {
                    A[i][j] = pw;
                    pw *= sn;
                }
                A[i][n] = expl((long double)rmd::kBeta * (sqrtl(fmaxl(0.0L, 1.0L - z * z)) - 1.0L));
            }
            for (int col = 0; col < n; ++col) {
                int piv = col;
                for (int i = col + 1; i < n; ++i)
                    if (fabsl(A[i][col]) > fabsl(A[piv][col])) piv = i;
                for (int j = 0; j <= n; ++j) std::swap(A[col][j], A[piv][j]);
                for (int i = col + 1; i < n; ++i) {
                    const long double f = A[i][col] / A[col][col];
                    for (int j = col; j <= n; ++j) A[i][j] -= f * A[col][j];
                }
            }
            for (int i = n - 1; i >= 0; --i) {      // back substitution; x_j kept in A[j][n]
                long double v = A[i][n];
                for (int j = i + 1; j < n; ++j) v -= A[i][j] * A[j][n];
                A[i][n] = v / A[i][i];
            }
            for (int j = 0; j < n; ++j) {
                if (j % 2 == 0)
                    r.even[t][j / 2] = (float)A[j][n];
                else
                    r.odd[t][j / 2] = (float)A[j][n];
            }
        }
        return r;
    }();
    return tp;
}

// Workspace of rmd_if_cube_static: a file-scope device array (each GPU the
// library runs on holds its own copy for the life of the process).  Host code
// must not pass the array's name to a kernel or a copy (on the host it is a
// stand-in, not a device address): static_scratch() looks up the device
// address of the current device's copy once and keeps it.
static __device__ __align__(256) unsigned char scratch[RMD_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;

rmd_status static_scratch(void** out) {
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(RMD_EINVAL, "device index beyond the static scratch table");
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p) return fail(RMD_EHIP, "hipGetSymbolAddress(scratch) gave NULL");
        addr[dev] = p;
    }
    *out = addr[dev];
    return RMD_OK;
}

rmd::SynthArgs synth_args(const rmd_scene* sc) {
    rmd::SynthArgs a{};
    a.mesh_tri_off = sc->mesh_tri_off;
    a.tris = sc->tris;
    a.verts = sc->verts;
    a.ray_off = sc->ray_off;
    a.hit_mesh = sc->hit_mesh;
    a.hit_tri = sc->hit_tri;
    a.hit_u = sc->hit_u;
    a.hit_v = sc->hit_v;
    a.n_hits = sc->n_hits;
    a.n_meshes = sc->n_meshes;
    a.n_tris = sc->n_tris;
    a.n_verts = sc->n_verts;
    a.n_rays = sc->n_rays;
    return a;
}

}  // namespace

extern "C" {

int32_t rmd_api_version(void) { return 2; }

const char* rmd_last_error(void) { return g_err.c_str(); }

rmd_status rmd_check_scene(const rmd_scene* scene, int32_t n_chirps, void* workspace, int64_t* n_bad_rays,
                           hipStream_t stream) {
    rmd_status st = check_scene_desc(scene);
    if (st != RMD_OK) return st;
    if (n_chirps <= 0) return fail(RMD_EINVAL, "n_chirps must be positive");
    if (!workspace || !n_bad_rays) return fail(RMD_EINVAL, "workspace and n_bad_rays must not be NULL");
    (void)n_chirps;   // indices are checked against the first snapshot's layout (the same for all)
    rmd::SynthArgs a = synth_args(scene);
    auto* bad = static_cast<unsigned long long*>(workspace);
    hipLaunchKernelGGL(rmd::zero_kernel, dim3(1), dim3(1), 0, stream, bad);
    hipLaunchKernelGGL(rmd::check_kernel, dim3((scene->n_rays + 255) / 256), dim3(256), 0, stream, a, bad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "check_kernel launch");
    unsigned long long h = 0;
    e = hipMemcpyAsync(&h, bad, sizeof(h), hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return hip_fail(e, "rmd_check_scene");
    *n_bad_rays = (int64_t)h;
    if (h) return fail(RMD_ESCENE, std::to_string(h) + " ray(s) with out-of-range meta data");
    return RMD_OK;
}

rmd_status rmd_workspace_bytes(const rmd_scene* scene, const rmd_radar* radar, int32_t n_pairs,
                               int32_t chirp_count, int64_t* bytes) {
    rmd_status st = check_scene_desc(scene);
    if (st != RMD_OK) return st;
    if (!radar || !bytes) return fail(RMD_EINVAL, "radar and bytes must not be NULL");
    if (n_pairs <= 0 || chirp_count <= 0 || radar->n_samples <= 0 || radar->n_samples > RMD_MAX_SAMPLES)
        return fail(RMD_EINVAL, "n_pairs, chirp_count must be positive; n_samples in [1, RMD_MAX_SAMPLES]");
    *bytes = plan(scene->n_rays, scene->n_hits, n_pairs, chirp_count, radar->n_samples).total_bytes;
    return RMD_OK;
}

}  // extern "C"

namespace {

// Checks shared by both IF entry points; fills the plan and the kernel
// arguments common to both methods.
rmd_status cube_setup(const rmd_scene* scene, const rmd_radar* radar, int32_t n_pairs, const double* pairs,
                      const float* weights, int32_t chirp0, int32_t chirp_count, float* s, void* workspace,
                      int64_t workspace_bytes, Plan& p, rmd::SynthArgs& a) {
    int64_t need = 0;
    rmd_status st = rmd_workspace_bytes(scene, radar, n_pairs, chirp_count, &need);
    if (st != RMD_OK) return st;
    if (!pairs || !s || !workspace) return fail(RMD_EINVAL, "pairs, s and workspace must not be NULL");
    if (workspace_bytes < need) return fail(RMD_EINVAL, "workspace smaller than rmd_workspace_bytes");
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(RMD_EINVAL, "workspace not 256-byte aligned");
    if (radar->n_chirps <= 0 || chirp0 < 0 || chirp0 + (int64_t)chirp_count > radar->n_chirps)
        return fail(RMD_EINVAL, "chirp range outside [0, n_chirps)");
    if (!(radar->f_s > 0) || !(radar->t_chirp > 0) || !std::isfinite(radar->f_c) || !std::isfinite(radar->bandwidth))
        return fail(RMD_EINVAL, "radar parameters must be finite, f_s and t_chirp positive");
    p = plan(scene->n_rays, scene->n_hits, n_pairs, chirp_count, radar->n_samples);
    if ((int64_t)n_pairs * p.batch * p.parts * 2 > INT32_MAX) return fail(RMD_EINVAL, "too many (pair, chirp) blocks");

    a = synth_args(scene);
    a.pairs = pairs;
    a.weights = weights;
    a.geo = static_cast<double*>(workspace);
    const int64_t geo_all = p.geo_sets * p.geo_bytes;
    a.hit_rec = reinterpret_cast<int4*>(static_cast<char*>(workspace) + geo_all);
    a.hit_rec_v = reinterpret_cast<float*>(static_cast<char*>(workspace) + geo_all +
                                           round256(scene->n_hits * (int64_t)sizeof(int4)));
    a.partial = reinterpret_cast<float2*>(static_cast<char*>(workspace) + geo_all + p.rec_bytes);
    a.n_pairs = n_pairs;
    a.n_samples = radar->n_samples;
    a.n_parts = p.parts;
    a.rays_per_part = p.rays_per_part;
    a.n_passes = (radar->n_samples + rmd::kBlock - 1) / rmd::kBlock;
    const double mu = radar->bandwidth / radar->t_chirp;               // Eq. 3
    a.cyc_per_m = radar->f_c / rmd::kC0;
    a.step_per_m = mu / (rmd::kC0 * radar->f_s);
    return RMD_OK;
}

// Helper stream of the current device (created once, default priority): the
// geometry of the next chirp batch is built on it while the current batch is
// synthesised on the caller's stream.
rmd_status helper_stream(hipStream_t* out) {
    static std::mutex mu;
    static hipStream_t streams[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(RMD_EINVAL, "device index beyond the helper stream table");
    std::lock_guard<std::mutex> lock(mu);
    if (!streams[dev]) {
        e = hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking);
        if (e != hipSuccess) return hip_fail(e, "hipStreamCreateWithFlags");
    }
    *out = streams[dev];
    return RMD_OK;
}

// The chirp batches of one IF cube: geometry_kernel of batch b into geometry
// set b mod geo_sets, then work(args, nb, c0) on `stream` (the batch's
// synthesis).  With two sets, batch b + 1's geometry runs on the helper stream
// while batch b is synthesised; events order each geometry after the
// synthesis that last read its set, and each synthesis after its geometry, so
// the helper stream's work is joined back into `stream` (also under graph
// capture).  The results are those of the serial order.
//
// Before them the call's hits are resolved and, where n_tables > 0, its tables
// computed: by prep_kernel, or in a call of one small batch (kInlineWork
// rays x chirps) of rays with few hits (kInlineHits on average) by the geometry
// kernel itself.  A ray then resolves its hits once per chirp, four loads that
// wait for one another in place of two, which costs less than the launch up to
// about that size: us per call, own launch and inline, 5003 rays x 8 chirps
// 22.5 / 21.1, 5003 x 4 20.7 / 18.3, 100000 x 8 59.8 / 62.2, 300000 x 8 133 /
// 143.  By hits a ray, 16000 rays x 4 chirps 1: 20.1 / 17.3, 6: 25.0 / 22.4, 16:
// 35.0 / 34.4, 32: 53 / 75; 65000 x 4 6: 45.7 / 40.4, 12: 72 / 97, 32: 179 / 565;
// 300 x 16 by the direct method 6: 18.3 / 18.1, 8: 19.9 / 20.6, 32: 36 / 47.  (The
// host knows the mean alone: where one ray in 61 has 16 hits and the others two,
// 300 x 16 takes 22.1 / 25.4, and 45 / 65 where it has 64.)
constexpr int64_t kInlineWork = int64_t(1) << 18;
constexpr int64_t kInlineHits = 6;

template <class Work>
rmd_status run_batches(const Plan& p, rmd::SynthArgs a, int32_t chirp0, int32_t chirp_count, int n_rays,
                       int n_tables, hipStream_t stream, Work&& work) {
    const int ray_blocks = (n_rays + rmd::kPrepThreads - 1) / rmd::kPrepThreads;
    const bool inline_prep = chirp_count <= p.batch && (int64_t)n_rays * chirp_count <= kInlineWork &&
                             a.n_hits <= kInlineHits * n_rays;
    if (!inline_prep) {
        const int hit_blocks = (int)((a.n_hits + rmd::kPrepThreads - 1) / rmd::kPrepThreads);
        if (hit_blocks + n_tables > 0)
            hipLaunchKernelGGL(rmd::prep_kernel, dim3((unsigned)(hit_blocks + n_tables)), dim3(rmd::kPrepThreads), 0,
                               stream, a, hit_blocks);
        hipError_t e0 = hipGetLastError();
        if (e0 != hipSuccess) return hip_fail(e0, "prep_kernel launch");
    }
    char* geo0 = reinterpret_cast<char*>(a.geo);
    auto geometry = [&](int b, hipStream_t st) {
        rmd::SynthArgs g = a;
        const int c0 = b * p.batch;
        g.chirp0 = chirp0 + c0;
        g.chirp_count = std::min(p.batch, chirp_count - c0);
        g.geo = reinterpret_cast<double*>(geo0 + (size_t)(b % p.geo_sets) * p.geo_bytes);
        if (inline_prep)
            hipLaunchKernelGGL(rmd::geometry_kernel<true>, dim3((unsigned)(n_tables + ray_blocks * g.chirp_count)),
                               dim3(rmd::kPrepThreads), 0, st, g, ray_blocks, n_tables);
        else
            hipLaunchKernelGGL(rmd::geometry_kernel<false>, dim3(ray_blocks, g.chirp_count), dim3(rmd::kPrepThreads), 0,
                               st, g, ray_blocks, 0);
    };
    auto batch_args = [&](int b) {
        rmd::SynthArgs w = a;
        const int c0 = b * p.batch;
        w.chirp0 = chirp0 + c0;
        w.chirp_count = std::min(p.batch, chirp_count - c0);
        w.geo = reinterpret_cast<double*>(geo0 + (size_t)(b % p.geo_sets) * p.geo_bytes);
        return w;
    };
    const int nbatch = (chirp_count + p.batch - 1) / p.batch;
    if (p.geo_sets == 1) {
        for (int b = 0; b < nbatch; ++b) {
            geometry(b, stream);
            const rmd::SynthArgs w = batch_args(b);
            work(w, w.chirp_count, b * p.batch);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return hip_fail(e, "IF cube launch");
        }
        return RMD_OK;
    }
    hipStream_t s2 = nullptr;
    rmd_status st = helper_stream(&s2);
    if (st != RMD_OK) return st;
    hipEvent_t ev[5] = {};   // start, geometry done (per set), synthesis done (per set)
    for (auto& x : ev) {
        hipError_t e = hipEventCreateWithFlags(&x, hipEventDisableTiming);
        if (e != hipSuccess) {
            for (auto& y : ev)
                if (y) (void)hipEventDestroy(y);
            return hip_fail(e, "hipEventCreateWithFlags");
        }
    }
    hipEvent_t* geo_done = ev + 1;
    hipEvent_t* work_done = ev + 3;
    hipError_t e = hipEventRecord(ev[0], stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(s2, ev[0], 0);      // after everything queued before the call
    if (e == hipSuccess) {
        geometry(0, s2);
        e = hipEventRecord(geo_done[0], s2);
    }
    for (int b = 0; b < nbatch && e == hipSuccess; ++b) {
        e = hipStreamWaitEvent(stream, geo_done[b & 1], 0);
        if (e != hipSuccess) break;
        const rmd::SynthArgs w = batch_args(b);
        work(w, w.chirp_count, b * p.batch);
        e = hipEventRecord(work_done[b & 1], stream);
        if (e != hipSuccess || b + 1 >= nbatch) break;
        // set (b + 1) % 2 was last read by batch b - 1
        if (b >= 1) e = hipStreamWaitEvent(s2, work_done[(b + 1) & 1], 0);
        if (e != hipSuccess) break;
        geometry(b + 1, s2);
        e = hipEventRecord(geo_done[(b + 1) & 1], s2);
    }
    if (e == hipSuccess) e = hipGetLastError();
    for (auto& x : ev) (void)hipEventDestroy(x);
    if (e != hipSuccess) return hip_fail(e, "IF cube launch");
    return RMD_OK;
}

// One pass of the range-Doppler transform over `lines` lines of 2^LOGL samples
// (lg: log2 of the element stride of a strided pass).  Workgroups of 256
// threads, or of 128 while that leaves compute units idle; strided lines want
// at least 8 neighbours in a workgroup (64 bytes of each row), up to 1024
// threads.
template <bool STRIDED, int LOGL>
void launch_fft_l(const float2* in, float2* out, int lines, int lg, hipStream_t stream) {
    using P = rmd::FftPlan<LOGL>;
    int threads = std::max(256, P::TPL);
    if (STRIDED) threads = std::min(1024, std::max(threads, 8 * P::TPL));
    else if (P::TPL <= 128 && (int64_t)lines * P::TPL < 512 * 256) threads = 128;
    const int lb = threads / P::TPL;
    const size_t words = (P::L > 8 ? P::L / 2 : 0) + (size_t)lb * (STRIDED ? P::L : P::L + P::L / 8);
    hipLaunchKernelGGL((rmd::fft_kernel<LOGL, STRIDED>), dim3((lines + lb - 1) / lb), dim3(threads),
                       P::L > 8 ? words * sizeof(float2) : 0, stream, in, out, lines, lg);
}

template <bool STRIDED, int LOGL = 0>
void launch_fft(const float2* in, float2* out, int logl, int lines, int lg, hipStream_t stream) {
    if (logl == LOGL) launch_fft_l<STRIDED, LOGL>(in, out, lines, lg, stream);
    else if constexpr ((1 << LOGL) < RMD_MAX_FFT) launch_fft<STRIDED, LOGL + 1>(in, out, logl, lines, lg, stream);
}

template <int COPIES, int THREADS>
void launch_spread_as(const rmd::SynthArgs& a, dim3 grid, int M, hipStream_t stream) {
    const size_t lds = (size_t)COPIES * 2 * (M + rmd::kTaps) * sizeof(unsigned long long);
    hipLaunchKernelGGL((rmd::spread_kernel<COPIES, THREADS>), grid, dim3(THREADS), lds, stream, a);
}

template <int THREADS>
void launch_spread_copies(const rmd::SynthArgs& a, dim3 grid, int M, int copies, hipStream_t stream) {
    if (copies >= 16) launch_spread_as<16, THREADS>(a, grid, M, stream);
    else if (copies == 8) launch_spread_as<8, THREADS>(a, grid, M, stream);
    else if (copies == 4) launch_spread_as<4, THREADS>(a, grid, M, stream);
    else launch_spread_as<2, THREADS>(a, grid, M, stream);
}

// Four workgroups a CU where the launch has them: with up to three a CU (of 256)
// all are resident either way, and the kernel is quicker with its registers.  us
// per launch at 3 / 4 waves a SIMD: 6 workgroups 20.5 / 21.9, 192 16.4 / 17.5,
// 768 37.2 / 38.0; 800 11.1 / 8.5, 1024 11.7 / 8.7, 3072 134 / 130, 6144 45.8 /
// 40.6, 7680 323 / 304, 9600 60.3 / 52.4.
void launch_synth(const rmd::SynthArgs& a, dim3 grid, hipStream_t stream) {
    if (grid.x <= 3 * 256) hipLaunchKernelGGL((rmd::synth_kernel<3>), grid, dim3(rmd::kThreads), 0, stream, a);
    else hipLaunchKernelGGL((rmd::synth_kernel<4>), grid, dim3(rmd::kThreads), 0, stream, a);
}

// Grid copies and threads of a spreading workgroup.  Copies spread the atomics
// over the banks but are cleared and summed once per workgroup: about 2048
// cells of them, and 4096 (with 512 threads, for the same LDS per wave) where a
// partition is long enough to pay for it.  512 threads also where a workgroup a
// CU or less is all there is, and where two copies of the largest grid leave
// room for two workgroups only.  us per call with 2048 cells / with 4096, 12
// pairs and 16 chirps, by M and rays per partition: 1024: 2560 rays 247 / 244,
// 4352 400 / 377, 6144 550 / 510; 512: 3072 280 / 287, 4352 366 / 356, 6144
// 513 / 475; 256: 4352 333 / 354, 6144 456 / 453, 9472 655 / 656; 128: 9472
// 615 / 603.  256 threads / 512: 8 and 16 workgroups a CU of M = 1024 147.5 /
// 154.7, one a CU 22.4 / 20.9; M = 2048 176 / 167.
//
// Fewer than 1024 rays are a single partition, too short to pay for as much:
// about 1024 cells, 512 below 96 rays, and 8 copies at most.  Time per call
// relative to 2 copies, 4 / 8 / 16, 9600 workgroups: M = 64: 64 rays 0.98 / 0.98
// / 1.09, 256 0.86 / 0.79 / 0.82, 1024 0.70 / 0.54 / 0.50; 128: 64 1.00 / 1.04 /
// 1.30, 256 0.94 / 0.88 / 1.03, 1024 0.82 / 0.67 / 0.70; 256: 64 1.02 / 1.15 /
// 1.74, 256 0.95 / 0.99 / 1.40, 1024 0.84 / 0.80 / 1.08; 512: 64 1.09, 256 1.04,
// 1024 0.96 (4 copies).
void launch_spread(const rmd::SynthArgs& a, dim3 grid, int M, int rays_per_part, hipStream_t stream) {
    const bool long_part = rays_per_part >= (M >= 512 ? 4096 : 8192);
    const int cells = long_part ? 4096 : a.n_rays >= 1024 ? 2048 : a.n_rays >= 96 ? 1024 : 512;
    const int copies = std::min(a.n_rays >= 1024 ? 16 : 8, std::max(2, cells / M));
    if (long_part || M >= 2048 || grid.x <= 256) launch_spread_copies<512>(a, grid, M, copies, stream);
    else launch_spread_copies<256>(a, grid, M, copies, stream);
}

}  // namespace

extern "C" {

rmd_status rmd_if_cube(const rmd_scene* scene, const rmd_radar* radar, int32_t n_pairs, const double* pairs,
                       const float* weights, int32_t chirp0, int32_t chirp_count, float* s, void* workspace,
                       int64_t workspace_bytes, hipStream_t stream) {
    Plan p;
    rmd::SynthArgs a;
    rmd_status st = cube_setup(scene, radar, n_pairs, pairs, weights, chirp0, chirp_count, s, workspace,
                               workspace_bytes, p, a);
    if (st != RMD_OK) return st;
    const int M = 1 << p.grid_log2;
    a.grid_log2 = p.grid_log2;
    a.center = radar->n_samples / 2;
    char* tail = static_cast<char*>(workspace) + p.geo_sets * p.geo_bytes + p.rec_bytes + p.grid_bytes;
    a.wmax_bits = reinterpret_cast<unsigned*>(tail);           // 256 bytes
    a.deconv = reinterpret_cast<double*>(tail + 256);
    a.n_wmax = weights ? (int)std::min<int64_t>(rmd::kWave, (scene->n_rays + 2047) / 2048) : 0;
    std::memcpy(a.tap_even, tap_poly().even, sizeof(a.tap_even));
    std::memcpy(a.tap_odd, tap_poly().odd, sizeof(a.tap_odd));
    const int n_tables = a.n_wmax + (radar->n_samples + rmd::kPrepThreads / rmd::kWave - 1) / (rmd::kPrepThreads / rmd::kWave);
    const size_t finish_lds = (size_t)(M / 2 + M) * sizeof(double2);
    // Chirp batches: the spreading and the transform of each batch after its
    // geometry (the partition count is the same for every batch: a shorter
    // last batch uses part of the buffers).
    return run_batches(p, a, chirp0, chirp_count, scene->n_rays, n_tables, stream,
                       [&](const rmd::SynthArgs& w, int nb, int c0) {
                           const dim3 grid((unsigned)((int64_t)n_pairs * nb * p.parts));
                           launch_spread(w, grid, M, p.rays_per_part, stream);
                           hipLaunchKernelGGL(rmd::finish_kernel, dim3((unsigned)(n_pairs * nb)),
                                              dim3(rmd::kFinishThreads), finish_lds, stream, w,
                                              reinterpret_cast<float2*>(s), chirp_count, c0);
                       });
}

rmd_status rmd_if_cube_static(const rmd_scene* scene, const rmd_radar* radar, int32_t n_pairs, const double* pairs,
                              const float* weights, int32_t chirp0, int32_t chirp_count, float* s,
                              hipStream_t stream) {
    int64_t need = 0;
    rmd_status st = rmd_workspace_bytes(scene, radar, n_pairs, chirp_count, &need);
    if (st != RMD_OK) return st;
    if (need > RMD_STATIC_SCRATCH_BYTES)
        return fail(RMD_EINVAL, "rmd_if_cube_static: these sizes need " + std::to_string(need) +
                                    " bytes of workspace, the static scratch holds " +
                                    std::to_string((long long)RMD_STATIC_SCRATCH_BYTES));
    void* ws = nullptr;
    st = static_scratch(&ws);
    if (st != RMD_OK) return st;
    return rmd_if_cube(scene, radar, n_pairs, pairs, weights, chirp0, chirp_count, s, ws, RMD_STATIC_SCRATCH_BYTES,
                       stream);
}

rmd_status rmd_if_cube_direct(const rmd_scene* scene, const rmd_radar* radar, int32_t n_pairs, const double* pairs,
                              const float* weights, int32_t chirp0, int32_t chirp_count, float* s, void* workspace,
                              int64_t workspace_bytes, hipStream_t stream) {
    Plan p;
    rmd::SynthArgs a;
    rmd_status st = cube_setup(scene, radar, n_pairs, pairs, weights, chirp0, chirp_count, s, workspace,
                               workspace_bytes, p, a);
    if (st != RMD_OK) return st;
    // Chirp batches: the synthesis and the partition sums of each batch after
    // its geometry.
    const int n_samples = radar->n_samples;
    return run_batches(p, a, chirp0, chirp_count, scene->n_rays, 0, stream,
                       [&](const rmd::SynthArgs& w, int nb, int c0) {
                           const dim3 grid((unsigned)((int64_t)n_pairs * w.n_passes * nb * p.parts));
                           launch_synth(w, grid, stream);
                           const int64_t count = (int64_t)n_pairs * nb * n_samples;
                           hipLaunchKernelGGL(rmd::reduce_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0,
                                              stream, w.partial, reinterpret_cast<float2*>(s), n_pairs, nb, n_samples,
                                              p.parts, chirp_count, c0);
                       });
}

rmd_status rmd_range_doppler(const float* s, float* S, int32_t n_pairs, int32_t n_chirps, int32_t n_samples,
                             hipStream_t stream) {
    if (!s || !S) return fail(RMD_EINVAL, "s and S must not be NULL");
    auto pow2 = [](int32_t n) { return n > 0 && (n & (n - 1)) == 0; };
    if (n_pairs <= 0 || !pow2(n_chirps) || !pow2(n_samples) || n_chirps > RMD_MAX_FFT || n_samples > RMD_MAX_FFT)
        return fail(RMD_EINVAL, "n_pairs > 0; n_chirps and n_samples powers of two <= RMD_MAX_FFT");
    if ((int64_t)n_pairs * n_chirps * n_samples > INT32_MAX) return fail(RMD_EINVAL, "cube too large");
    auto lg = [](int32_t n) { int l = 0; while ((1 << l) < n) ++l; return l; };
    const auto* in = reinterpret_cast<const float2*>(s);
    auto* out = reinterpret_cast<float2*>(S);
    // fast time: contiguous lines; slow time: lines n_samples apart, in place
    launch_fft<false>(in, out, lg(n_samples), n_pairs * n_chirps, 0, stream);
    launch_fft<true>(out, out, lg(n_chirps), n_pairs * n_samples, lg(n_samples), stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "fft_kernel launch");
    return RMD_OK;
}

rmd_status rmd_span_weights(const rmd_scene* scene, const uint8_t* in_set, const rmd_span_rule* rule,
                            const float* amp, float* weights, hipStream_t stream) {
    rmd_status st = check_scene_desc(scene);
    if (st != RMD_OK) return st;
    if (!in_set || !rule || !weights) return fail(RMD_EINVAL, "in_set, rule and weights must not be NULL");
    if (rule->mode < 0 || rule->mode > 2) return fail(RMD_EINVAL, "span mode must be 0, 1 or 2");
    hipLaunchKernelGGL(rmd::span_kernel, dim3((scene->n_rays + 255) / 256), dim3(256), 0, stream, *scene, in_set,
                       *rule, amp, weights);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "span_kernel launch");
    return RMD_OK;
}

}  // extern "C"
