// Phase-cell weights (Sec. 2, Eq. 7; Fibonacci lattice of Sec. 3) fused with the
// flux-matrix values (Eq. 6) and the direct-solar source (Eq. 9).
//
// One 64-lane wavefront per node l.  For every incoming propagation direction u
// (each in-edge, then the sunlight) the lattice is rotated so that its pole is u,
// each lattice point is owned by the out-edge direction s_m with the largest dot
// product (ties: lowest index), and the owners' phase weights are summed in 2^-52
// fixed point with LDS integer atomics (exact, so the sum is independent of the
// order).  Surface nodes use the unrotated lattice with cosine weights (Lambertian).
//
// The dot products of a direction are one contraction, R s_m (out-edges) by p_i (lattice
// points), and run on the matrix cores in FP16 halves of FP32 (see "The screen");
// the incoming directions are processed in groups of eight, two at a time.  Each
// direction's column of the node block (column-major) is one coalesced store.
//
// The ownership decision is an argmax over double-precision dot products; it is
// written with this exact operation sequence (also followed by the FP64 CPU
// reference):
//   s_m  = D_m / sqrt(Dx^2 + Dy^2 + Dz^2)             (exact integer sum; D_m = 0: below)
//   h    = 1 / (1 + u_z);  xy = (u_x u_y) h
//   R    = [[u_z + (u_y u_y) h, -xy, -u_x], [-xy, u_z + (u_x u_x) h, -u_y], [u_x, u_y, u_z]]
//          (R = diag(1, -1, -1) when 1 + u_z < 1e-12; the identity on the surface)
//   q_ik = fma(R_2k, p_i2, fma(R_1k, p_i1, R_0k p_i0))      (q_i = R^T p_i)
//   v_im = fma(q_i2, s_m2, fma(q_i1, s_m1, q_i0 s_m0))      (= p_i . R s_m)
// with no other contraction, hence the pragma below and -ffp-contract=off.
// Coupled nodes at one place (D_m = 0, an integer test) have no direction between them.  Such an
// out-edge owns nothing, unless no out-edge of the node has a direction (the first then owns
// all); as an incoming direction it counts as straight down (s_m = (0, 0, 1), u = -s_m).  No NaN
// arises, and this file is compiled as if there were none.
//
// The regular kernel finds that argmax through a screen with an error bound: every decision
// the screen cannot certify is taken by the FP64 sequence above, so each owner is the one
// the FP64 sequence gives.
#include "device.hpp"
#include "internal.hpp"

#pragma clang fp contract(off)

namespace sg {

namespace {

constexpr double kFix = 4503599627370496.0;  // 2^52
constexpr double kUnfix = 1.0 / 4503599627370496.0;
constexpr int kQMaxGroup = 8;  // incoming directions per group

// p / n for 0 <= p < 1024 and 1 <= n <= 128 with one FP32 multiply: (p + 1/2) / n is at
// least 1/(2n) >= 2^-8 away from an integer, far above the rounding error of the
// product (below 2^-12 here, also with a reciprocal a few ulp off)
__device__ __forceinline__ int small_div(int p, float inv_n) { return (int)(((float)p + 0.5f) * inv_n); }

// The screen.  The matrix cores multiply in FP16 and add in FP32, so each FP32 component
// (scaled by 2^10, which keeps the low halves normal) is split into a high half and a low half
// and the dot product takes 12 of the 16 products of v_mfma_f32_32x32x16_f16:
//   k     0..2     3..5     6..8     9..11    12
//   A     hi s     lo s     hi s     lo s     0, or -2^11 for a row past the last out-edge
//   B     hi p     hi p     lo p     lo p     2^10
// (lanes 0..31 hold k 0..7 of row or column lane, lanes 32..63 k 8..15 of row or column
// lane - 32).  A result holds 2^20 v for 32 out-edges (rows) and 32 lattice points
// (columns): lane l has column l mod 32 and the rows 8 (i / 4) + 4 (l / 32) + i mod 4 of its
// registers i < 16.  That row holds out-edge 2 i + l / 32 (+ 32 in a second row tile), so d
// out-edges fill about d / 2 registers and the others are left out.  The low bits of each
// value are replaced by 2 i (5 bits, 6 with two row tiles), and the two largest of a lane's
// values are kept; v_permlane32_swap brings the two halves of a column together, 64 columns
// (two tiles) a step, and the half is the out-edge's low bit.
// Error bound, in units of v (|v| <= 1): the rotation in FP32 (one multiply and two FMAs from
// the FP32 roundings of R and s) is off by at most 5 2^-24 per component, the halves of s
// (rounded toward zero) by 2^-22 and those of p by 1.5 2^-24 (2^-22 too where the points are rotated),
// together below sqrt(3) 13 2^-24 < 2^-19.5 in the dot product; the products are exact, and 16
// additions of partial sums below 2 are taken to be off by at most one unit of 2^-23 each, 2^-19
// (measured: 2^-22.3 in all); the index moves a value by less than 64 units in the last place, 2^-17.  So a value lies within 2^-16.1 of the
// FP64 sequence's, and if the largest exceeds the second by more than 2^-15 (kCertified), its
// out-edge is the FP64 argmax, with no tie.  The other slots (a few pairs in 10,000 on
// jittered grids) are queued, and the FP64 sequence decides them, one per lane.
// What bounds the kernel: vector issue.  Per tile of 32 points and d = 23 out-edges: 12 index
// inserts and 15 maxima and medians; the matrix product itself runs beside them (a probe: 32
// vector instructions 150 clocks, with one product 169).  FP32 FMAs with an index insert and 1.5
// maxima per product, the form before, took 9.1e8 vector instructions on plume 64x64x32 (now
// 5.5e8; issuing 93 % of the time): 1.27 -> 1.00 ms, cloud 128x128x48 7.6 -> 6.1 ms, plume
// 96x96x32 2.85 -> 2.22 ms.
// A node with an out-edge of no direction leaves all of its slots to the FP64 sequence.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
constexpr float kCertified = 32.0f;  // 2^-15 in units of 2^-20
constexpr float kHalfScale = 1024.0f;

struct Operand {  // four packed pairs of halves of a matrix operand
    unsigned w[4];
};
__device__ __forceinline__ float16v dot_tile(const Operand &a, const Operand &b) {
    const float16v zero = {};
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), zero, 0, 0,
                                                  0);
}

// (x, y, z), scaled, in halves rounded toward zero: (hi x, hi y), (hi z, lo x), (lo y, lo z)
__device__ __forceinline__ void split_halves(float x, float y, float z, unsigned (&p)[3]) {
    const auto h = __builtin_amdgcn_cvt_pkrtz(x, y);
    const float lx = x - (float)h[0], ly = y - (float)h[1];
    const auto m = __builtin_amdgcn_cvt_pkrtz(z, lx);
    const float lz = z - (float)m[0];
    p[0] = __builtin_bit_cast(unsigned, h);
    p[1] = __builtin_bit_cast(unsigned, m);
    p[2] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(ly, lz));
}

// u's low half beside v's low half, and u's high half beside v's (lanes 0..31, 32..63)
__device__ __forceinline__ void swap_halves(unsigned u, unsigned v, unsigned &low, unsigned &high) {
    const auto r = __builtin_amdgcn_permlane32_swap(u, v, false, false);
    low = r[0];
    high = r[1];
}
__device__ __forceinline__ void swap_halves(float u, float v, float &low, float &high) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(v), false, false);
    low = __uint_as_float(r[0]);
    high = __uint_as_float(r[1]);
}

// The two largest of a lane's first R values of a tile, with 2 i (from tag0 on) in their low
// bits, joined to (best, second) unless this is the first tile.  Three values a, b, c enter by
// their largest and their median (the smallest cannot be among the two), two such triples at
// a time: eight instructions for six values.
template <int R, int kMask>
__device__ __forceinline__ void fold_tile(const float16v &v, int tag0, bool first, float &best, float &second) {
    auto at = [&](int i) {
        return __uint_as_float((__float_as_uint(v[i]) & ~(unsigned)kMask) | (unsigned)(tag0 + 2 * i));
    };
    auto largest = [](float a, float b, float c) { return fmaxf(fmaxf(a, b), c); };
    int i = 0;
    if (first && R >= 3) {
        const float a = at(0), b = at(1), c = at(2);
        best = largest(a, b, c);
        second = __builtin_amdgcn_fmed3f(a, b, c);
        i = 3;
    } else if (first) {
        best = fmaxf(at(0), at(1));
        second = fminf(at(0), at(1));
        i = 2;
    }
#pragma unroll
    for (; i + 6 <= R; i += 6) {
        const float a = at(i), b = at(i + 1), c = at(i + 2), x = at(i + 3), y = at(i + 4), z = at(i + 5);
        const float g = largest(a, b, c), h = largest(x, y, z);
        const float mid = __builtin_amdgcn_fmed3f(best, g, h);
        second = largest(second, __builtin_amdgcn_fmed3f(a, b, c), __builtin_amdgcn_fmed3f(x, y, z));
        second = fmaxf(second, mid);
        best = largest(best, g, h);
    }
    if (i + 3 <= R) {
        const float a = at(i), b = at(i + 1), c = at(i + 2), g = largest(a, b, c);
        second = largest(second, __builtin_amdgcn_fmed3f(a, b, c), fminf(best, g));
        best = fmaxf(best, g);
        i += 3;
    }
    if (i + 2 <= R) {
        const float a = at(i), b = at(i + 1);
        second = fmaxf(second, __builtin_amdgcn_fmed3f(best, a, b));
        best = largest(best, a, b);
        i += 2;
    }
    if (i < R) {
        const float a = at(i);
        second = __builtin_amdgcn_fmed3f(best, second, a);
        best = fmaxf(best, a);
    }
}

// RT row tiles; R registers of the last (the first of two takes all 16)
template <int RT, int R>
struct Rows {
    static constexpr int kMask = RT == 1 ? 31 : 63;
    // the two largest values of every column against this lane's rows
    static __device__ __forceinline__ void column(const Operand (&a)[2], const Operand &b, float &best, float &second) {
        if constexpr (RT == 2) {
            fold_tile<16, kMask>(dot_tile(a[0], b), 0, true, best, second);
            fold_tile<R, kMask>(dot_tile(a[1], b), 32, false, best, second);
        } else {
            fold_tile<R, kMask>(dot_tile(a[0], b), 0, true, best, second);
        }
    }
    // Both halves of two tiles' columns: lanes 0..31 take tile X's columns, the others Y's.
    // The owner's out-edge, and whether it is certified.
    static __device__ __forceinline__ int owner(float bx, float sx, float by, float sy, bool &sure) {
        float b0, b1, s0, s1;
        swap_halves(bx, by, b0, b1);
        swap_halves(sx, sy, s0, s1);
        const float best = fmaxf(b0, b1), second = fmaxf(fmaxf(fminf(b0, b1), s0), s1);
        sure = best - second > kCertified;
        return (int)((__float_as_uint(best) & (unsigned)kMask) | (b1 > b0 ? 1u : 0u));
    }
};

// The unit vector of displacement (Dx, Dy, Dz); false (and straight up) where it is zero
__device__ __forceinline__ bool unit_vector(long long Dx, long long Dy, long long Dz, double &x, double &y, double &z) {
    const bool has = (Dx | Dy | Dz) != 0;
    const double nrm = has ? sqrt((double)(Dx * Dx + Dy * Dy + Dz * Dz)) : 1.0;
    x = (double)Dx / nrm;
    y = (double)Dy / nrm;
    z = has ? (double)Dz / nrm : 1.0;
    return has;
}

// q = R^T p for lattice point (x, y, z) (R row-major, 9 doubles)
__device__ __forceinline__ void rotate_point(const double *R, double x, double y, double z, double &q0, double &q1,
                                             double &q2) {
#pragma clang fp contract(off)
    q0 = fma(R[6], z, fma(R[3], y, R[0] * x));
    q1 = fma(R[7], z, fma(R[4], y, R[1] * x));
    q2 = fma(R[8], z, fma(R[5], y, R[2] * x));
}

// the rotation that takes direction u to the pole (row-major)
__device__ __forceinline__ void pole_rotation(double ux, double uy, double uz, double (&R)[9]) {
#pragma clang fp contract(off)
    if (1.0 + uz < 1e-12) {
        R[0] = 1.0; R[1] = 0.0; R[2] = 0.0; R[3] = 0.0; R[4] = -1.0; R[5] = 0.0; R[6] = 0.0; R[7] = 0.0; R[8] = -1.0;
    } else {
        const double h = 1.0 / (1.0 + uz);
        const double xy = (ux * uy) * h;
        R[0] = uz + (uy * uy) * h; R[1] = -xy; R[2] = -ux;
        R[3] = -xy; R[4] = uz + (ux * ux) * h; R[5] = -uy;
        R[6] = ux; R[7] = uy; R[8] = uz;
    }
}

// Dynamic LDS of a node in k_qbuild, for node degrees up to dm (a multiple of 8): the FP64
// sites [3][dm], bins [8][dm] (fixed point) and lattice weights [128] (fixed point), the
// rotations' rows in FP32 as float4 [dm + 1][3], and the queue of uncertified slots
constexpr int kQueue = kQMaxGroup * 128;
__host__ __device__ constexpr size_t qbuild_lds(int dm) {
    return 8 * (size_t)(3 * dm + kQMaxGroup * dm + 128) + 48 * (size_t)(dm + 1) + 2 * (size_t)kQueue;
}

// this lane's operand of lattice tile t
__device__ __forceinline__ Operand lattice_tile(const uint4 *__restrict__ lat_halves, int t, int lane) {
    const uint4 v = lat_halves[64 * t + lane];
    return {{v.x, v.y, v.z, v.w}};
}

// One group of ng directions from a0: their owners' weights into the bins, and the slots
// whose owner is not certified into the queue (point + 128 x direction of the group; returns
// their number).  Full tiles of 32 lattice points are taken two directions at a time, the out-edges
// rotated (A) against the lattice (B, the same for every direction); up to eight points past
// the last full tile are taken for all directions of the group at once, as columns (point,
// direction) with the points rotated instead (B) against the out-edges as they are (A).
template <int RT, int R>
__device__ __forceinline__ int group_owners(int a0, int ng, int n_in, int dm, int NF, int nt, int rest, bool screen,
                                            int lane, const float (&site)[2][3], const unsigned (&past)[2],
                                            const Operand (&pts)[4], const float4 *rows,
                                            const unsigned long long *wq, const double *__restrict__ lat,
                                            unsigned long long *bins, unsigned short *queue) {
    using T = Rows<RT, R>;
    int nq = 0;
    // lattice point pt's weight to its owner m for direction dl of the group, or the slot to the queue
    auto settle = [&](bool valid, int dl, int pt, int m, bool sure) {
        sure = sure && screen;
        if (valid && sure && SG_IN(dl * dm + m, kQMaxGroup * dm, 0x203)) atomicAdd(&bins[dl * dm + m], wq[pt]);
        const bool wait = valid && !sure;
        const unsigned long long open = __ballot(wait);
        if (open) {
            if (wait) queue[nq + __popcll(open & ((1ull << lane) - 1ull))] = (unsigned short)(dl * 128 + pt);
            nq += __popcll(open);
        }
    };
    const int half = lane >> 5, col = lane & 31;
    for (int dl = 0; dl < ng; dl += 2) {
        const int a = min(a0 + dl + half, n_in - 1);  // past the last direction: a repeat, not counted
        const float4 r0 = rows[3 * a], r1 = rows[3 * a + 1], r2 = rows[3 * a + 2];
        Operand op[2][2];  // [direction][row tile]
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const float x = site[t][0], y = site[t][1], z = site[t][2];
            unsigned p[3];
            split_halves(fmaf(r0.z, z, fmaf(r0.y, y, r0.x * x)), fmaf(r1.z, z, fmaf(r1.y, y, r1.x * x)),
                         fmaf(r2.z, z, fmaf(r2.y, y, r2.x * x)), p);
            swap_halves(p[0], p[1], op[0][t].w[0], op[1][t].w[0]);
            swap_halves(p[1], p[2], op[0][t].w[1], op[1][t].w[1]);
            swap_halves(p[2], past[t], op[0][t].w[2], op[1][t].w[2]);
            swap_halves(p[0], 0u, op[0][t].w[3], op[1][t].w[3]);
        }
        const bool two = dl + 1 < ng;
#pragma unroll
        for (int t = 0; t < 4; t += 2) {
            float b[2], s[2];
            bool sure;
            if (t + 1 < nt) {  // two tiles of each direction
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (q == 1 && !two) break;
                    T::column(op[q], pts[t], b[0], s[0]);
                    T::column(op[q], pts[t + 1], b[1], s[1]);
                    const int pt = 32 * t + lane, m = T::owner(b[0], s[0], b[1], s[1], sure);
                    if (32 * t + 64 <= NF) settle(true, dl + q, pt, m, sure);
                    else settle(pt < NF, dl + q, pt, m, sure);
                }
            } else if (t < nt) {  // the last tile of both directions
                T::column(op[0], pts[t], b[0], s[0]);
                T::column(op[1], pts[t], b[1], s[1]);
                const int pt = 32 * t + col, m = T::owner(b[0], s[0], b[1], s[1], sure);
                settle((half == 0 || two) && pt < NF, dl + half, pt, m, sure);
            }
        }
    }
    if (rest) {
        const int n = ng * rest;  // columns, at most 64
        const int dl = min(small_div(lane, 1.0f / (float)rest), ng - 1);
        const int pt = 32 * nt + lane - rest * small_div(lane, 1.0f / (float)rest);
        const float4 r0 = rows[3 * (a0 + dl)], r1 = rows[3 * (a0 + dl) + 1], r2 = rows[3 * (a0 + dl) + 2];
        const float x = (float)lat[3 * pt] * kHalfScale, y = (float)lat[3 * pt + 1] * kHalfScale,
                    z = (float)lat[3 * pt + 2] * kHalfScale;
        unsigned p[3];  // q = R^T p
        split_halves(fmaf(r2.x, z, fmaf(r1.x, y, r0.x * x)), fmaf(r2.y, z, fmaf(r1.y, y, r0.y * x)),
                     fmaf(r2.z, z, fmaf(r1.z, y, r0.z * x)), p);
        const unsigned one = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(kHalfScale, 0.0f));
        Operand q[2];  // (hx, hy) (hz, hx) (hy, hz) (lx, ly) | (lz, lx) (ly, lz) (2^10, 0) 0
        swap_halves(p[0], (p[2] >> 16) | (p[1] & 0xffff0000u), q[0].w[0], q[1].w[0]);
        swap_halves((p[1] & 0xffffu) | (p[0] << 16), p[2], q[0].w[1], q[1].w[1]);
        swap_halves((p[0] >> 16) | (p[1] << 16), one, q[0].w[2], q[1].w[2]);
        swap_halves((p[1] >> 16) | (p[2] << 16), 0u, q[0].w[3], q[1].w[3]);
        // the out-edges as they are; the second row tile's halves do not fit the registers and are made
        // group by group (the empty statement keeps the compiler from making them once and spilling them)
        Operand fixed[2];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            float sx = site[t][0];
            if (t == 1) asm volatile("" : "+v"(sx));
            split_halves(sx, site[t][1], site[t][2], p);
            fixed[t].w[0] = half ? p[1] : p[0];
            fixed[t].w[1] = half ? p[2] : p[1];
            fixed[t].w[2] = half ? past[t] : p[2];
            fixed[t].w[3] = half ? 0u : p[0];
        }
        float b0, s0, b1, s1;
        T::column(fixed, q[0], b0, s0);
        if (n > 32) T::column(fixed, q[1], b1, s1);
        else { b1 = b0; s1 = s0; }
        bool sure;
        const int m = T::owner(b0, s0, b1, s1, sure);
        settle(lane < n, dl, pt, m, sure);
    }
    return nq;
}

template <class Real, class BlkT, bool kWriteQ>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(5))) void k_qbuild(
    int N, int nvol, const long long *__restrict__ adj_ptr, const int *__restrict__ adj_idx,
    const int *__restrict__ pos, const double *__restrict__ lat, const uint4 *__restrict__ lat_halves,
    const double *__restrict__ tab, int NF, int n_phase, const float *__restrict__ frac, double sun_x, double sun_y,
    double sun_z, Real mu0, const Real *__restrict__ T, const Real *__restrict__ rho, const Real *__restrict__ Tsun,
    const long long *__restrict__ nodeoff, BlkT *__restrict__ val, Real *__restrict__ S, float *__restrict__ qsun,
    int dm, int per, long long wx, long long wy, int screen) {
#pragma clang fp contract(off)
    extern __shared__ double qb_lds[];
    double *sx = qb_lds, *sy = qb_lds + dm, *sz = qb_lds + 2 * dm;
    unsigned long long *bins = reinterpret_cast<unsigned long long *>(qb_lds + 3 * dm);
    unsigned long long *wq = bins + kQMaxGroup * dm;
    float4 *rows = reinterpret_cast<float4 *>(wq + 128);
    unsigned short *queue = reinterpret_cast<unsigned short *>(rows + 3 * (dm + 1));

    const int l = blockIdx.x;
    const int lane = threadIdx.x;
    const long long off = adj_ptr[l];
    const int d = (int)(adj_ptr[l + 1] - off);
    if (d == 0 || d > kWave) return;  // higher degree: k_qbuild_big
    const bool surf = l >= nvol;
    if (!SG_IN(nodeoff[l] + (long long)d * d - 1, nodeoff[N], 0x201)) return;

    bool none = false;
    if (lane < d) {
        const int j0 = adj_idx[off + lane];
        const int j = SG_IN(j0, N, 0x202) ? j0 : l;
        const long long Dx = min_image((long long)pos[3 * j] - pos[3 * l], wx, per & 1);
        const long long Dy = min_image((long long)pos[3 * j + 1] - pos[3 * l + 1], wy, per & 2);
        const long long Dz = (long long)pos[3 * j + 2] - pos[3 * l + 2];
        none = !unit_vector(Dx, Dy, Dz, sx[lane], sy[lane], sz[lane]);
    }
    const unsigned long long without = __ballot(none);  // the out-edges of no direction
    const bool screened = screen != 0 && without == 0ull;
    // phase weights of the lattice points in fixed point
    for (int i = lane; i < NF; i += 64) {
        double w;
        if (surf) {
            w = tab[n_phase * NF + i];
        } else {
            w = 0.0;
            for (int k = 0; k < n_phase; ++k) {
                const double f = frac ? (double)frac[(long long)k * nvol + l] : 1.0;
                w = w + f * tab[k * NF + i];
            }
        }
        wq[i] = (unsigned long long)llrint(w * kFix);
    }
    __syncthreads();
    // the rotations of all incoming directions, in FP32
    const int n_in = surf ? 1 : d + 1;
    for (int a = lane; a < n_in; a += 64) {
        double R[9] = {1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0};
        if (!surf) {
            if (a < d) pole_rotation(-sx[a], -sy[a], -sz[a], R);
            else pole_rotation(sun_x, sun_y, sun_z, R);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k)
            rows[3 * a + k] = make_float4((float)R[3 * k], (float)R[3 * k + 1], (float)R[3 * k + 2], 0.0f);
    }
    // this lane's out-edge of each row tile, and the lattice
    const unsigned below = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(-2.0f * kHalfScale, 0.0f));
    float site[2][3];
    unsigned past[2];
    Operand pts[4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int r = lane & 31, m = 32 * t + 2 * (4 * (r >> 3) + (r & 3)) + (r >> 2 & 1);
        const bool in = m < d;
        site[t][0] = in ? (float)sx[m] * kHalfScale : 0.0f;
        site[t][1] = in ? (float)sy[m] * kHalfScale : 0.0f;
        site[t][2] = in ? (float)sz[m] * kHalfScale : 0.0f;
        past[t] = in ? 0u : below;
    }
    // full tiles of lattice points; up to eight points past them are columns of their own, more
    // make another tile
    int nt = NF >> 5, rest = NF & 31;
    if (rest > 8) {
        ++nt;
        rest = 0;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) pts[t] = lattice_tile(lat_halves, t, lane);

    const float inv_d = 1.0f / (float)d;
    const Real rl = rho ? rho[l] : (Real)0;
    const Real tsun = Tsun ? Tsun[l] : (Real)0;
    BlkT *blk = val + nodeoff[l];  // column-major: element (row n, column m) at m d + n
    for (int a0 = 0; a0 < n_in; a0 += kQMaxGroup) {
        const int ng = min(kQMaxGroup, n_in - a0);
        for (int t = lane; t < ng * dm; t += 64) bins[t] = 0ull;
        __syncthreads();
        int nq;
#define SG_GROUP(RT, R)                                                                                            \
    nq = group_owners<RT, R>(a0, ng, n_in, dm, NF, nt, rest, screened, lane, site, past, pts, rows, wq, lat, \
                             bins, queue)
        if (d <= 8) SG_GROUP(1, 4);
        else if (d <= 16) SG_GROUP(1, 8);
        else if (d <= 20) SG_GROUP(1, 10);
        else if (d <= 24) SG_GROUP(1, 12);
        else if (d <= 28) SG_GROUP(1, 14);
        else if (d <= 32) SG_GROUP(1, 16);
        else if (d <= 48) SG_GROUP(2, 8);
        else SG_GROUP(2, 16);
#undef SG_GROUP
        __syncthreads();
        // the uncertified slots, one per lane, with the FP64 sequence; ties go to the lowest
        // index, the index moving only on a strict increase
        for (int t = lane; t < nq; t += 64) {
            const int slot = queue[t], dl = slot >> 7, i = slot & 127, a = a0 + dl;
            double R[9] = {1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0};
            if (!surf) {
                if (a < d) pole_rotation(-sx[a], -sy[a], -sz[a], R);
                else pole_rotation(sun_x, sun_y, sun_z, R);
            }
            double q0, q1, q2;
            rotate_point(R, lat[3 * i], lat[3 * i + 1], lat[3 * i + 2], q0, q1, q2);
            double best = -__builtin_inf();
            int o = 0;
            auto take = [&](int k) {
                const double v = fma(q2, sz[k], fma(q1, sy[k], q0 * sx[k]));
                o = v > best ? k : o;
                best = fmax(best, v);
            };
            if (without == 0ull) {
                for (int k = 0; k < d; ++k) take(k);
            } else {
                for (int k = 0; k < d; ++k)
                    if (!(without >> k & 1ull)) take(k);
            }
            if (SG_IN(dl * dm + o, kQMaxGroup * dm, 0x203)) atomicAdd(&bins[dl * dm + o], wq[i]);
        }
        __syncthreads();
        // this group's columns: pair t = (a - a0) d + m is column a, row m
        for (int t = lane; t < ng * d; t += 64) {
            const int al = small_div(t, inv_d), m = t - al * d, a = a0 + al;
            const double Q = (double)(long long)bins[al * dm + m] * kUnfix;
            const long long b = off + m;
            if (surf) {
                for (int c = 0; c < d; ++c) {
                    if (kWriteQ) blk[c * d + m] = (BlkT)Q;
                    else blk[c * d + m] = (BlkT)(T[off + c] * rl * (Real)Q);
                }
                if (!kWriteQ) S[b] = rl * mu0 * tsun * (Real)Q;
                qsun[b] = (float)Q;
            } else if (a < d) {
                if (kWriteQ) blk[a * d + m] = (BlkT)Q;
                else blk[a * d + m] = (BlkT)(T[off + a] * rl * (Real)Q);
            } else {
                if (!kWriteQ) S[b] = tsun * rl * (Real)Q;
                qsun[b] = (float)Q;
            }
        }
        __syncthreads();
    }
}

// Nodes of degree above 64 (graphs whose strongest couplings gather on the dense nodes): one
// workgroup of four wavefronts per (node, group of `group` incoming directions), wg =
// bigdir[b] + g.  The group's (direction, lattice point) pairs are the columns of the screen's
// matrix products, up to 1024, the points rotated by their direction; a wavefront keeps its
// pairs of column tiles in registers and the out-edges pass by as row tiles from LDS, so each
// is split into its halves once per group and read once per wavefront.
//
// Every lane keeps the largest value of a tile's 16 rows it holds (8 instructions), and of
// those the two largest with the largest one's tile (4 more): with hundreds of out-edges an
// index in every value, as k_qbuild inserts it, would cost 38.  The 16 rows of the best tile
// are then done again in FP32 with a 4-bit index.
// Error bound, in units of v: rotated point 5 2^-24 per component in FP32, its halves and the
// out-edge's 2^-22 each (rounded toward zero), the out-edge in FP32 from its integer offset 6
// 2^-24 relative: together below (sqrt(3) 13 + 6) 2^-24 < 2^-19.1; the additions of the matrix
// product 2^-19, or the FP32 ones 3 2^-24 with the index 2^-19.  Any two of these values
// together are off by less than 2^-17 (kBigCertified), so a larger gap between the best row and
// the largest of all others certifies the FP64 argmax.  The other columns (below a percent
// on jittered positions) are queued, and the workgroup scans all out-edges for them with the FP64
// sequence, several lanes per column while there are few.
//
// Bound: vector issue, 81 % of the time (plume 64x64x32 with its 11.5 strongest couplings per voxel,
// 1.3e9 cells: 35.6 ms with FP64 dot products for all out-edges, now 9.4 ms; four tenths of the
// vector instructions are the tiles', a sixth the best tiles' rows again).
constexpr int kBigPairs = 4;                    // pairs of 32-column tiles per wavefront
constexpr int kBigCols = 4 * kBigPairs * 64;    // columns per workgroup
constexpr int kBigGroup = 16;                   // most directions per workgroup (their rotations in LDS)
constexpr int kBigRows = 1024;                  // out-edges in LDS at a time, as halves
constexpr int kScanEdges = 256;                 // out-edges in LDS at a time, in FP64
constexpr int kBinRows = 512;                   // rows of a column summed at a time, per wavefront
constexpr float kBigCertified = 8.0f;           // 2^-17 in units of 2^-20
constexpr double kNoDirection = 2.0;            // x component, in LDS, of an out-edge of no direction

// A wavefront's first C pairs of column tiles against nt row tiles: per lane and tile the
// largest value of its rows, the second largest of the row tiles' largest, and the best's tile
template <int C>
__device__ __forceinline__ void pass_rows(const uint4 *rows, int nt, int col, const Operand (&pts)[2 * kBigPairs],
                                          float (&best)[2 * kBigPairs], float (&second)[2 * kBigPairs],
                                          int (&tile)[2 * kBigPairs]) {
    uint4 next = rows[col];
    for (int t = 0; t < nt; ++t) {
        const Operand a = {{next.x, next.y, next.z, next.w}};
        next = rows[32 * min(t + 1, nt - 1) + col];
#pragma unroll
        for (int j = 0; j < 2 * C; ++j) {
            const float16v v = dot_tile(a, pts[j]);
            auto largest = [](float x, float y, float z) { return fmaxf(fmaxf(x, y), z); };
            const float x = largest(v[0], v[1], v[2]), y = largest(v[3], v[4], v[5]), z = largest(v[6], v[7], v[8]);
            const float w = largest(v[9], v[10], v[11]), u = largest(v[12], v[13], v[14]);
            const float top = fmaxf(largest(x, y, z), largest(w, u, v[15]));
            second[j] = __builtin_amdgcn_fmed3f(best[j], second[j], top);
            tile[j] = top > best[j] ? t : tile[j];
            best[j] = fmaxf(best[j], top);
        }
    }
}

template <class Real, class BlkT, bool kWriteQ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_qbuild_big(
    int nbig, const int *__restrict__ big, const long long *__restrict__ bigdir, int nvol,
    const long long *__restrict__ adj_ptr, const int *__restrict__ adj_idx, const int *__restrict__ pos,
    const double *__restrict__ lat, const double *__restrict__ tab, int NF, int n_phase,
    const float *__restrict__ frac, double sun_x, double sun_y, double sun_z, Real mu0, const Real *__restrict__ T,
    const Real *__restrict__ rho, const Real *__restrict__ Tsun, const long long *__restrict__ nodeoff,
    BlkT *__restrict__ val, Real *__restrict__ S, float *__restrict__ qsun, int group, int per, long long wx,
    long long wy, int screen) {
#pragma clang fp contract(off)
    // out-edges as halves, then out-edges in FP64, then each wavefront's bins
    __shared__ uint4 pool[kBigRows];
    __shared__ float4 whole[kBigRows];  // the same out-edges in FP32
    static_assert(sizeof(pool) >= 3 * kScanEdges * sizeof(double), "FP64 out-edges");
    static_assert(sizeof(pool) >= 4 * kBinRows * sizeof(unsigned long long), "bins");
    __shared__ double Rg[kBigGroup * 9];
    __shared__ unsigned long long wq[128];
    __shared__ unsigned short owner[kBigCols], queue[kBigCols];
    // (flags in LDS, not __syncthreads_or: that keeps all three thread indices in a register through the
    // passes, the one that did not fit)
    __shared__ int queued, lost;  // columns without a certificate; whether an out-edge has no direction
    const long long wg = blockIdx.x;
    int lo = 0, hi = nbig;  // the node b with bigdir[b] <= wg < bigdir[b + 1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (bigdir[mid] <= wg) lo = mid; else hi = mid;
    }
    const int l = big[lo];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const long long off = adj_ptr[l];
    const int d = (int)(adj_ptr[l + 1] - off);
    const bool surf = l >= nvol;
    const int n_in = surf ? 1 : d + 1;
    const int a0 = (int)(wg - bigdir[lo]) * group;
    const int ng = min(group, n_in - a0);
    auto edge_offset = [&](int m, long long &Dx, long long &Dy, long long &Dz) {
        const int j = adj_idx[off + m];
        Dx = min_image((long long)pos[3 * j] - pos[3 * l], wx, per & 1);
        Dy = min_image((long long)pos[3 * j + 1] - pos[3 * l + 1], wy, per & 2);
        Dz = (long long)pos[3 * j + 2] - pos[3 * l + 2];
    };
    // the unit direction of out-edge m (the operation sequence of k_qbuild)
    auto edge_dir = [&](int m, double &ex, double &ey, double &ez) {
        long long Dx, Dy, Dz;
        edge_offset(m, Dx, Dy, Dz);
        return unit_vector(Dx, Dy, Dz, ex, ey, ez);
    };
    if (tid < NF) {
        double w;
        if (surf) {
            w = tab[n_phase * NF + tid];
        } else {
            w = 0.0;
            for (int k = 0; k < n_phase; ++k) {
                const double f = frac ? (double)frac[(long long)k * nvol + l] : 1.0;
                w = w + f * tab[k * NF + tid];
            }
        }
        wq[tid] = (unsigned long long)llrint(w * kFix);
    }
    if (tid == 0) queued = lost = 0;
    // rotations of this group's incoming directions
    if (tid >= 192 && tid - 192 < ng) {
        const int a = a0 + tid - 192;
        double R[9] = {1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0};
        if (!surf) {
            double ux = sun_x, uy = sun_y, uz = sun_z;
            if (a < d) {
                edge_dir(a, ux, uy, uz);
                ux = -ux; uy = -uy; uz = -uz;
            }
            pole_rotation(ux, uy, uz, R);
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) Rg[9 * (tid - 192) + k] = R[k];
    }
    __syncthreads();
    const int np = ng * NF;
    const float inv_nf = 1.0f / (float)NF;
    // column p's rotated point q = R^T p in FP32, scaled
    auto column = [&](int p, float &x, float &y, float &z) {
        const int al = small_div(p, inv_nf), i = p - al * NF;
        const double *R = Rg + 9 * al;
        const float u = (float)lat[3 * i] * kHalfScale, v = (float)lat[3 * i + 1] * kHalfScale,
                    w = (float)lat[3 * i + 2] * kHalfScale;
        x = fmaf((float)R[6], w, fmaf((float)R[3], v, (float)R[0] * u));
        y = fmaf((float)R[7], w, fmaf((float)R[4], v, (float)R[1] * u));
        z = fmaf((float)R[8], w, fmaf((float)R[5], v, (float)R[2] * u));
    };
    // this wavefront's pair j holds the columns 64 (wave + 4 j) + lane
    const int pairs = (np + 63) / 64;
    const int mine = pairs > wave ? (pairs - wave + 3) / 4 : 0;
    float run_best[kBigPairs], run_second[kBigPairs];
    int run_own[kBigPairs];
    if (screen) {
        Operand pts[2 * kBigPairs];
#pragma unroll
        for (int j = 0; j < kBigPairs; ++j) {
            float x, y, z;
            column(min(64 * (wave + 4 * j) + lane, np - 1), x, y, z);  // past the last: a repeat, not counted
            unsigned p[3];
            split_halves(x, y, z, p);
            // k 0..7 hi (x, y) (z, x) (y, z) (2^10, 0); k 8..15 lo (x, y) (z, x) (y, z) 0
            const unsigned one = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(kHalfScale, 0.0f));
            Operand &s = pts[2 * j], &t = pts[2 * j + 1];
            swap_halves(p[0], (p[1] >> 16) | (p[2] << 16), s.w[0], t.w[0]);
            swap_halves((p[1] & 0xffffu) | (p[0] << 16), (p[2] >> 16) | (p[1] & 0xffff0000u), s.w[1], t.w[1]);
            swap_halves((p[0] >> 16) | (p[1] << 16), p[2], s.w[2], t.w[2]);
            swap_halves(one, 0u, s.w[3], t.w[3]);
            run_best[j] = -8.0f * 0x1p20f;
            run_second[j] = -8.0f * 0x1p20f;
            run_own[j] = 0;
        }
        for (int m0 = 0; m0 < d; m0 += kBigRows) {
            const int nm = min(kBigRows, d - m0), nt = (nm + 31) / 32;
            if (m0) __syncthreads();
            // both k halves of a row read (hi x, y) (hi z, lo x) (lo y, z) (0 or -2^11 past the last, 0)
            for (int r = tid; r < 32 * nt; r += 256) {
                const float past = r < nm ? 0.0f : -2.0f * kHalfScale;
                float4 site = make_float4(0.0f, 0.0f, 0.0f, kHalfScale * past);
                if (r < nm) {
                    long long Dx, Dy, Dz;
                    edge_offset(m0 + r, Dx, Dy, Dz);
                    if ((Dx | Dy | Dz) == 0) lost = 1;
                    const float x = (float)Dx, y = (float)Dy, z = (float)Dz;  // whole: below 1 only if all zero
                    const float inv = __builtin_amdgcn_rsqf(fmaxf(fmaf(z, z, fmaf(y, y, x * x)), 1.0f)) * kHalfScale;
                    site.x = x * inv;
                    site.y = y * inv;
                    site.z = z * inv;
                }
                unsigned p[3];
                split_halves(site.x, site.y, site.z, p);
                pool[r] = make_uint4(p[0], p[1], p[2],
                                     __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(past, 0.0f)));
                whole[r] = site;
            }
            __syncthreads();
            float best[2 * kBigPairs], second[2 * kBigPairs];
            int tile[2 * kBigPairs];
#pragma unroll
            for (int j = 0; j < 2 * kBigPairs; ++j) {
                best[j] = -8.0f * 0x1p20f;
                second[j] = -8.0f * 0x1p20f;
                tile[j] = 0;
            }
            if (mine == 4) pass_rows<4>(pool, nt, lane & 31, pts, best, second, tile);
            else if (mine == 3) pass_rows<3>(pool, nt, lane & 31, pts, best, second, tile);
            else if (mine == 2) pass_rows<2>(pool, nt, lane & 31, pts, best, second, tile);
            else if (mine == 1) pass_rows<1>(pool, nt, lane & 31, pts, best, second, tile);
            // lanes take a column each (both halves of the rows), and its best tile's 16 rows again
#pragma unroll
            for (int j = 0; j < kBigPairs; ++j) {
                if (j >= mine) continue;
                float b0, b1, s0, s1;
                unsigned t0, t1;
                swap_halves(best[2 * j], best[2 * j + 1], b0, b1);
                swap_halves(second[2 * j], second[2 * j + 1], s0, s1);
                swap_halves((unsigned)tile[2 * j], (unsigned)tile[2 * j + 1], t0, t1);
                const bool upper = b1 > b0;
                const int r0 = 32 * (int)(upper ? t1 : t0) + (upper ? 4 : 0);
                float x, y, z;
                column(min(64 * (wave + 4 * j) + lane, np - 1), x, y, z);
                float top = -8.0f * 0x1p20f, next = fmaxf(fmaxf(fminf(b0, b1), s0), s1);
                auto again = [&](int i) {
                    const float4 a = whole[r0 + 8 * (i >> 2) + (i & 3)];
                    const float v = fmaf(a.z, z, fmaf(a.y, y, fmaf(a.x, x, a.w)));
                    return __uint_as_float((__float_as_uint(v) & ~15u) | (unsigned)i);
                };
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const float v = again(i), w = again(i + 1);
                    next = fmaxf(next, __builtin_amdgcn_fmed3f(top, v, w));
                    top = fmaxf(fmaxf(top, v), w);
                }
                const int i = (int)(__float_as_uint(top) & 15u);
                run_own[j] = top > run_best[j] ? m0 + r0 + 8 * (i >> 2) + (i & 3) : run_own[j];
                run_second[j] = fmaxf(fmaxf(run_second[j], next), fminf(run_best[j], top));
                run_best[j] = fmaxf(run_best[j], top);
            }
        }
    }
    __syncthreads();
    const bool sure = screen && !lost;
#pragma unroll
    for (int j = 0; j < kBigPairs; ++j) {
        const int p = 64 * (wave + 4 * j) + lane;
        const bool certain = sure && run_best[j] - run_second[j] > kBigCertified;
        if (p < np && certain) owner[p] = (unsigned short)run_own[j];
        const bool wait = p < np && !certain;
        const unsigned long long open = __ballot(wait);
        if (open) {
            int at = 0;
            if (lane == 0) at = atomicAdd(&queued, __popcll(open));
            at = __shfl(at, 0);
            if (wait) queue[at + __popcll(open & ((1ull << lane) - 1ull))] = (unsigned short)p;
        }
    }
    __syncthreads();
    // the queued columns: 256 / parts at a time, the out-edges m = part (mod parts) in a lane, with
    // the FP64 sequence; ties go to the lowest index
    const int nq = queued;
    int parts = 1;
    while (parts < 64 && 2 * parts * nq <= 256) parts *= 2;
    double *ex = reinterpret_cast<double *>(pool), *ey = ex + kScanEdges, *ez = ey + kScanEdges;
    for (int c0 = 0; c0 < nq; c0 += 256 / parts) {
        const int c = c0 + tid / parts, part = tid & (parts - 1);
        const int p = queue[min(c, nq - 1)], al = small_div(p, inv_nf), i = p - al * NF;
        double q0, q1, q2;
        rotate_point(Rg + 9 * al, lat[3 * i], lat[3 * i + 1], lat[3 * i + 2], q0, q1, q2);
        double best = -__builtin_inf();
        int own = 0;
        for (int m0 = 0; m0 < d; m0 += kScanEdges) {
            const int nm = min(kScanEdges, d - m0);
            if (tid < nm && !edge_dir(m0 + tid, ex[tid], ey[tid], ez[tid])) {
                ex[tid] = kNoDirection;
                lost = 1;
            }
            __syncthreads();
            if (c < nq && !lost) {
#pragma unroll 4
                for (int k = part; k < nm; k += parts) {
                    const double v = fma(q2, ez[k], fma(q1, ey[k], q0 * ex[k]));
                    own = v > best ? m0 + k : own;
                    best = fmax(best, v);
                }
            } else if (c < nq) {
                for (int k = part; k < nm; k += parts) {
                    const double x = ex[k], dot = fma(q2, ez[k], fma(q1, ey[k], q0 * x));
                    const double v = x == kNoDirection ? -__builtin_inf() : dot;
                    own = v > best ? m0 + k : own;
                    best = fmax(best, v);
                }
            }
            __syncthreads();  // the next edges overwrite these
        }
        for (int s = 1; s < parts; s <<= 1) {
            const double v = __shfl_xor(best, s);
            const int o = __shfl_xor(own, s);
            own = v > best || (v == best && o < own) ? o : own;
            best = fmax(best, v);
        }
        if (c < nq && part == 0) owner[p] = (unsigned short)own;
    }
    __syncthreads();
    // a wavefront per direction, kBinRows rows at a time: the weights summed by owner, then the
    // column filled with the value of an empty cell and the owners' rows written over it (at most
    // N_fib of the hundreds of rows; a read of every row's sum took a seventh of the kernel).  A
    // surface node has one direction, and its columns differ by T only: the wavefronts share them.
    const Real rl = rho ? rho[l] : (Real)0;
    const Real tsun = Tsun ? Tsun[l] : (Real)0;
    BlkT *blk = val + nodeoff[l];  // column-major: element (row n, column m) at m d + n
    unsigned long long *bins = reinterpret_cast<unsigned long long *>(pool) + kBinRows * wave;
    for (int al = surf ? 0 : wave; al < ng; al += 4) {
        const int a = a0 + al;
        for (int r0 = 0; r0 < d; r0 += kBinRows) {
            const int nr = min(kBinRows, d - r0);
            unsigned row[2];  // the owners of this lane's points, from r0
            double Q[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = lane + 64 * h;
                row[h] = i < NF ? (unsigned)(owner[al * NF + i] - r0) : ~0u;
                if (row[h] < (unsigned)nr) bins[row[h]] = 0ull;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (row[h] < (unsigned)nr) atomicAdd(&bins[row[h]], wq[lane + 64 * h]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int h = 0; h < 2; ++h) Q[h] = row[h] < (unsigned)nr ? (double)(long long)bins[row[h]] * kUnfix : 0.0;
            // rows r0.. of a column: value(Q) for every cell
            auto put = [&](auto *dst, auto value) {
                const auto empty = value(0.0);
                for (int r = lane; r < nr; r += 64) dst[r0 + r] = empty;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (row[h] < (unsigned)nr) dst[r0 + row[h]] = value(Q[h]);
            };
            auto put_column = [&](int c) {
                if (kWriteQ) put(blk + (long long)c * d, [](double q) { return (BlkT)q; });
                else {
                    const Real f = T[off + c] * rl;
                    put(blk + (long long)c * d, [f](double q) { return (BlkT)(f * (Real)q); });
                }
            };
            if (surf) {
                for (int c = wave; c < d; c += 4) put_column(c);
            } else if (a < d) {
                put_column(a);
            }
            if ((surf && wave == 0) || a == d) {
                const Real f = surf ? rl * mu0 * tsun : tsun * rl;
                if (!kWriteQ) put(S + off, [f](double q) { return f * (Real)q; });
                put(qsun + off, [](double q) { return (float)q; });
            }
        }
    }
}

// The paper's discretisation of Sigma (Sec. 3), for scenes that ask for it: per
// incoming direction, every out-edge direction colours its closest lattice point and
// the colours spread over the lattice by flood fill along the edges of its convex
// hull.  One 64-lane wavefront per node; two incoming directions at a time up to degree 32 (lane
// 32 dl + m: direction dl's out-edge m), one above (lane m).
//   seeds: for m = 0, 1, ...: the lattice point of largest v_im (the Voronoi
//   ownership's dot products, same operation sequence; ties to the lowest i) takes
//   colour m unless it was claimed with a value >= v_im by an earlier direction;
//   fill: in rounds, every uncoloured point takes the colour its lowest-index
//   coloured neighbour had at the start of the round, until all are coloured (the
//   hull graph is connected and there is at least one seed).
// Q(u -> m) is the fixed-point sum of the phase weights of colour m, as in k_qbuild.
// The largest v_im comes from k_qbuild's screen with the operands changed over (lattice points
// are the rows, out-edges the columns, 2^-15 certifies as there), its FP64 value from the FP64
// sequence at that point; a lane without a certificate scans all points in FP64.  In the fill
// the coloured points are two 64-bit masks and so are a point's neighbours (points lane and lane +
// 64): the lowest coloured neighbour is the first bit of their intersection, and one read gives
// its colour.
// Bound: vector issue.  FP64 dot products over all points and a fill that read up to 16
// neighbours' colours a round, the form before: plume 48x48x24 2.30 ms, now 1.04 ms.
// order-preserving 64-bit keys of doubles (for integer atomic max in LDS)
__device__ __forceinline__ unsigned long long order_key(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double order_value(unsigned long long k) {
    const unsigned long long b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
    return __longlong_as_double((long long)b);
}

template <class Real, class BlkT, bool kWriteQ>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(5))) void k_qcolour(
    int N, int nvol, const long long *__restrict__ adj_ptr, const int *__restrict__ adj_idx,
    const int *__restrict__ pos, const double *__restrict__ lat, const uint4 *__restrict__ lat_halves,
    const double *__restrict__ tab, int NF, int n_phase, const float *__restrict__ frac, double sun_x, double sun_y,
    double sun_z, Real mu0, const Real *__restrict__ T, const Real *__restrict__ rho, const Real *__restrict__ Tsun,
    const long long *__restrict__ nodeoff, BlkT *__restrict__ val, Real *__restrict__ S, float *__restrict__ qsun,
    const int *__restrict__ hull, int per, long long wx, long long wy, int screen) {
#pragma clang fp contract(off)
    __shared__ double sx[64], sy[64], sz[64];
    __shared__ unsigned long long wq[128], bins[2][64], bkey[2][128];
    __shared__ int col[2][128];
    __shared__ double rot[2][9];
    constexpr int kNone = 0x7fffffff;

    const int l = blockIdx.x;
    const int lane = threadIdx.x;
    const long long off = adj_ptr[l];
    const int d = (int)(adj_ptr[l + 1] - off);
    if (d == 0 || d > kWave) return;  // higher degree: k_qcolour_big
    const bool surf = l >= nvol;
    if (!SG_IN(nodeoff[l] + (long long)d * d - 1, nodeoff[N], 0x204)) return;
    bool none = false;
    if (lane < d) {
        const int j0 = adj_idx[off + lane];
        const int j = SG_IN(j0, N, 0x205) ? j0 : l;
        const long long Dx = min_image((long long)pos[3 * j] - pos[3 * l], wx, per & 1);
        const long long Dy = min_image((long long)pos[3 * j + 1] - pos[3 * l + 1], wy, per & 2);
        const long long Dz = (long long)pos[3 * j + 2] - pos[3 * l + 2];
        none = !unit_vector(Dx, Dy, Dz, sx[lane], sy[lane], sz[lane]);
    }
    const unsigned long long without = __ballot(none);  // the out-edges of no direction
    const bool screened = screen != 0 && without == 0ull;
    for (int i = lane; i < NF; i += 64) {
        double w;
        if (surf) {
            w = tab[n_phase * NF + i];
        } else {
            w = 0.0;
            for (int k = 0; k < n_phase; ++k) {
                const double f = frac ? (double)frac[(long long)k * nvol + l] : 1.0;
                w = w + f * tab[k * NF + i];
            }
        }
        wq[i] = (unsigned long long)llrint(w * kFix);
    }
    __syncthreads();

    const Real rl = rho ? rho[l] : (Real)0;
    const Real tsun = Tsun ? Tsun[l] : (Real)0;
    BlkT *blk = val + nodeoff[l];  // column-major: element (row n, column m) at m d + n
    const int n_in = surf ? 1 : d + 1;
    const int nd = d <= 32 ? 2 : 1;  // directions at a time
    const int dl = nd == 2 ? lane >> 5 : 0, m = nd == 2 ? lane & 31 : lane;
    const int mc = min(m, d - 1);  // lanes past d repeat the last out-edge, not counted
    const int nt = (NF + 31) >> 5, last = NF - 32 * (nt - 1);  // row tiles of lattice points
    unsigned long long near[2][2];  // the hull neighbours of points lane and lane + 64, as masks
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = lane + 64 * h;
        near[h][0] = near[h][1] = 0ull;
        if (i < NF) {
            const int nn = hull[NF * kHullNb + i];
            for (int t = 0; t < nn; ++t) {
                const int j = hull[i * kHullNb + t];
                near[h][0] |= j < 64 ? 1ull << j : 0ull;
                near[h][1] |= j < 64 ? 0ull : 1ull << (j & 63);
            }
        }
    }
    for (int a0 = 0; a0 < n_in; a0 += nd) {
        // the rotation of this lane's direction, in LDS
        const int a = min(a0 + dl, n_in - 1);  // past the last direction: a repeat, not counted
        {
            double R[9] = {1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0};
            if (!surf) {
                if (a < d) pole_rotation(-sx[a], -sy[a], -sz[a], R);
                else pole_rotation(sun_x, sun_y, sun_z, R);
            }
            if (m == 0) {
#pragma unroll
                for (int k = 0; k < 9; ++k) rot[dl][k] = R[k];
            }
        }
        __syncthreads();
        const double *R = rot[dl];
        const bool mine = m < d && a0 + dl < n_in, seeds = mine && !(without >> m & 1ull);
        // seeds: the screen's largest value over the lattice points of every (direction, out-edge)
        bool sure = false;
        int pt = 0;
        if (screened) {
            const float x = (float)sx[mc] * kHalfScale, y = (float)sy[mc] * kHalfScale, z = (float)sz[mc] * kHalfScale;
            unsigned p[3];
            split_halves(fmaf((float)R[2], z, fmaf((float)R[1], y, (float)R[0] * x)),
                         fmaf((float)R[5], z, fmaf((float)R[4], y, (float)R[3] * x)),
                         fmaf((float)R[8], z, fmaf((float)R[7], y, (float)R[6] * x)), p);
            // k 13: 2^10 against the -2^11 of the rows past the last point
            const unsigned one = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(0.0f, kHalfScale));
            Operand op[2], pts[4];
            // the lattice's operands are read anew (held from pair to pair they do not fit five wavefronts'
            // registers, and hoisted, which the empty statement prevents, they would be spilled)
            int at = lane;
            asm volatile("" : "+v"(at));
#pragma unroll
            for (int t = 0; t < 4; ++t) pts[t] = lattice_tile(lat_halves, t, at);
            swap_halves(p[0], p[1], op[0].w[0], op[1].w[0]);
            swap_halves(p[1], p[2], op[0].w[1], op[1].w[1]);
            swap_halves(p[2], one, op[0].w[2], op[1].w[2]);
            swap_halves(p[0], 0u, op[0].w[3], op[1].w[3]);
            float best[2], second[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {  // register i of tile t: 2 i + t mod 2 + 32 (t / 2)
                    if (t >= nt) break;
                    const int tag = 32 * (t >> 1) + (t & 1);
                    const float16v v = dot_tile(pts[t], op[q]);
                    if (t == nt - 1 && last <= 8) fold_tile<4, 63>(v, tag, t == 0, best[q], second[q]);
                    else fold_tile<16, 63>(v, tag, t == 0, best[q], second[q]);
                }
            }
            float b0, b1, s0, s1;
            swap_halves(best[0], best[1], b0, b1);
            swap_halves(second[0], second[1], s0, s1);
            const float top = fmaxf(b0, b1);
            sure = top - fmaxf(fmaxf(fminf(b0, b1), s0), s1) > kCertified;
            const int tag = (int)(__float_as_uint(top) & 63u), i = (tag & 31) >> 1;
            pt = 32 * (2 * (tag >> 5) + (tag & 1)) + 8 * (i >> 2) + (b1 > b0 ? 4 : 0) + (i & 3);
        }
        asm volatile("" ::: "memory");  // rotation and out-edge are read again: 24 registers less in the products
        double v = -__builtin_inf();
        if (seeds && sure) {
            double q0, q1, q2;
            rotate_point(R, lat[3 * pt], lat[3 * pt + 1], lat[3 * pt + 2], q0, q1, q2);
            v = fma(q2, sz[m], fma(q1, sy[m], q0 * sx[m]));
        } else if (seeds) {  // the lattice points in ascending order, strict >
            pt = 0;
            for (int i = 0; i < NF; ++i) {
                double q0, q1, q2;
                rotate_point(R, lat[3 * i], lat[3 * i + 1], lat[3 * i + 2], q0, q1, q2);
                const double w = fma(q2, sz[m], fma(q1, sy[m], q0 * sx[m]));
                pt = w > v ? i : pt;
                v = fmax(v, w);
            }
        }
        // claims: a point seeded by several out-edges goes to the largest value, ties to the
        // lowest m (claiming in order of m)
        for (int t = lane; t < 256; t += 64) {
            bkey[t >> 7][t & 127] = 0ull;
            col[t >> 7][t & 127] = kNone;
        }
        for (int q = 0; q < 2; ++q) bins[q][lane] = 0ull;
        __syncthreads();
        if (seeds) atomicMax(&bkey[dl][pt], order_key(v));
        __syncthreads();
        if (seeds && v == order_value(bkey[dl][pt])) atomicMin(&col[dl][pt], m);
        __syncthreads();
        // the fill, of both directions at once
        int c[2][2];
        bool ok[2][2];
        unsigned long long done[2][2];
        const bool unseeded = __popcll(without) == d;  // the first out-edge takes all
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                ok[q][h] = lane + 64 * h < NF && q < nd && a0 + q < n_in;
                c[q][h] = unseeded ? 0 : col[q][lane + 64 * h];
                done[q][h] = __ballot(ok[q][h] && c[q][h] != kNone);
            }
        }
        while (true) {
            bool fresh[2][2];
            unsigned long long news = 0ull;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const unsigned long long lo = near[h][0] & done[q][0], hi = near[h][1] & done[q][1];
                    fresh[q][h] = ok[q][h] && c[q][h] == kNone && (lo | hi) != 0ull;
                    const int from = lo ? __builtin_ctzll(lo) : 64 + __builtin_ctzll(hi | 1ull << 63);
                    if (fresh[q][h]) c[q][h] = col[q][from];
                }
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (fresh[q][h]) col[q][lane + 64 * h] = c[q][h];
                    const unsigned long long b = __ballot(fresh[q][h]);
                    done[q][h] |= b;
                    news |= b;
                }
            }
            __syncthreads();
            if (!news) break;
        }
        // cells: fixed-point sums per colour, then the directions' columns
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (ok[q][h] && c[q][h] != kNone && SG_IN(c[q][h], d, 0x206))
                    atomicAdd(&bins[q][c[q][h]], wq[lane + 64 * h]);
        }
        __syncthreads();
        if (mine) {
            const double Q = (double)(long long)bins[dl][m] * kUnfix;
            const long long b = off + m;
            if (surf) {
                for (int k = 0; k < d; ++k) {
                    if (kWriteQ) blk[k * d + m] = (BlkT)Q;
                    else blk[k * d + m] = (BlkT)(T[off + k] * rl * (Real)Q);
                }
                if (!kWriteQ) S[b] = rl * mu0 * tsun * (Real)Q;
                qsun[b] = (float)Q;
            } else if (a < d) {
                if (kWriteQ) blk[a * d + m] = (BlkT)Q;
                else blk[a * d + m] = (BlkT)(T[off + a] * rl * (Real)Q);
            } else {
                Real f = tsun;
                asm volatile("" : "+v"(f));  // keeps the product below from being held through the directions
                if (!kWriteQ) S[b] = f * rl * (Real)Q;
                qsun[b] = (float)Q;
            }
        }
        __syncthreads();
    }
}

// Cell sums by owner: a direction's lattice points have at most N_fib distinct owners among the d
// out-edges, so they go to a 256-slot open-addressing table in LDS (exact integer atomics), and a
// column is written by looking every row up (absent: 0).
constexpr int kCellHash = 256;  // above the most owners a direction can have (N_fib <= 128)

constexpr unsigned short kNoOwner = 0xffff;  // owners are below 4096
constexpr unsigned char kNoSeed = 0xff;      // lattice points are below 128

__device__ __forceinline__ int cell_find(const unsigned short *keys, int m) {
    int h = m & (kCellHash - 1);
    while (keys[h] != m && keys[h] != kNoOwner) h = (h + 1) & (kCellHash - 1);
    return keys[h] == m ? h : -1;
}

// The colouring for nodes of degree above 64: one 64-lane workgroup per (node, incoming
// direction), lattice points i and i + 64 in lane i, their rotated coordinates in LDS.
//   seeds: lanes run over the out-directions m; each scans the lattice points in
//   ascending order (strict >) for its seed and raises the point's best value (an
//   order-preserving 64-bit key, atomic max); then every m whose seed value equals its
//   point's best offers its index (atomic min): a point claimed several times goes to
//   the largest value, ties to the lowest m, as claiming in order of m gives.
//   fill and cells as in k_qcolour, the colours' sums in a hash table (at most N_fib
//   colours among the d out-edges), the column written by looking up every row.

// unit vector of node l's out-edge m (the shortest periodic image); false: it has none
__device__ __forceinline__ bool edge_unit(const long long *__restrict__ adj_ptr, const int *__restrict__ adj_idx,
                                          const int *__restrict__ pos, int l, int m, int per, long long wx,
                                          long long wy, double &ex, double &ey, double &ez) {
    const int j = adj_idx[adj_ptr[l] + m];
    const long long Dx = min_image((long long)pos[3 * j] - pos[3 * l], wx, per & 1);
    const long long Dy = min_image((long long)pos[3 * j + 1] - pos[3 * l + 1], wy, per & 2);
    const long long Dz = (long long)pos[3 * j + 2] - pos[3 * l + 2];
    return unit_vector(Dx, Dy, Dz, ex, ey, ez);
}

// seeds of S out-directions per lane (m0 + 64 s + lane, s < S): each scans the lattice
// points in ascending order (strict >), so every point read from LDS serves S dot products;
// then the point's best value is raised (order-preserving key, atomic max)
template <int S>
__device__ __forceinline__ void colour_seeds(int m0, int d, int NF, const double (*lq)[128],
                                             const long long *__restrict__ adj_ptr,
                                             const int *__restrict__ adj_idx, const int *__restrict__ pos, int l,
                                             int per, long long wx, long long wy, unsigned char *seed_pt,
                                             unsigned long long *bkey) {
#pragma clang fp contract(off)
    double tx[S], ty[S], tz[S], bv[S];
    int bi[S];
    bool has[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int m = min(m0 + 64 * s + (int)threadIdx.x, d - 1);
        has[s] = edge_unit(adj_ptr, adj_idx, pos, l, m, per, wx, wy, tx[s], ty[s], tz[s]);
        bv[s] = fma(lq[2][0], tz[s], fma(lq[1][0], ty[s], lq[0][0] * tx[s]));
        bi[s] = 0;
    }
    for (int i = 1; i < NF; ++i) {
        const double x = lq[0][i], y = lq[1][i], z = lq[2][i];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const double v = fma(z, tz[s], fma(y, ty[s], x * tx[s]));
            bi[s] = v > bv[s] ? i : bi[s];  // moves only on a strict increase
            bv[s] = fmax(bv[s], v);
        }
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int m = m0 + 64 * s + (int)threadIdx.x;
        if (m < d) {
            seed_pt[m] = has[s] ? (unsigned char)bi[s] : kNoSeed;
            if (has[s]) atomicMax(&bkey[bi[s]], order_key(bv[s]));
        }
    }
}

template <class Real, class BlkT, bool kWriteQ>
__global__ __launch_bounds__(64) void k_qcolour_big(
    int nbig, const int *__restrict__ big, const long long *__restrict__ bigdir, int nvol,
    const long long *__restrict__ adj_ptr, const int *__restrict__ adj_idx, const int *__restrict__ pos,
    const double *__restrict__ lat, const double *__restrict__ tab, int NF, int n_phase,
    const float *__restrict__ frac, double sun_x, double sun_y, double sun_z, Real mu0, const Real *__restrict__ T,
    const Real *__restrict__ rho, const Real *__restrict__ Tsun, const long long *__restrict__ nodeoff,
    BlkT *__restrict__ val, Real *__restrict__ S, float *__restrict__ qsun, const int *__restrict__ hull, int per,
    long long wx, long long wy) {
#pragma clang fp contract(off)
    __shared__ double lq[3][128];  // the rotated lattice; after the claims, the cells' hash table
    __shared__ unsigned long long bkey[128], wq[128];
    __shared__ int col[128], snap[128];
    __shared__ unsigned char seed_pt[kMaxDegree];
    static_assert(kCellHash * (sizeof(unsigned long long) + sizeof(unsigned short)) <= sizeof(lq), "hash in lq");
    unsigned long long *hval = reinterpret_cast<unsigned long long *>(&lq[0][0]);
    unsigned short *hkey = reinterpret_cast<unsigned short *>(hval + kCellHash);
    const long long wg = blockIdx.x;
    int lo = 0, hi = nbig;  // the node b with bigdir[b] <= wg < bigdir[b + 1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (bigdir[mid] <= wg) lo = mid; else hi = mid;
    }
    const int l = big[lo];
    const int a = (int)(wg - bigdir[lo]);
    const int lane = threadIdx.x;
    const long long off = adj_ptr[l];
    const int d = (int)(adj_ptr[l + 1] - off);
    const bool surf = l >= nvol;
    auto edge_dir = [&](int m, double &ex, double &ey, double &ez) {
        (void)edge_unit(adj_ptr, adj_idx, pos, l, m, per, wx, wy, ex, ey, ez);
    };
    double R[9];
    if (surf) {
        R[0] = 1.0; R[1] = 0.0; R[2] = 0.0; R[3] = 0.0; R[4] = 1.0; R[5] = 0.0; R[6] = 0.0; R[7] = 0.0; R[8] = 1.0;
    } else {
        double ux, uy, uz;
        if (a < d) {
            edge_dir(a, ux, uy, uz);
            ux = -ux; uy = -uy; uz = -uz;
        } else {
            ux = sun_x; uy = sun_y; uz = sun_z;
        }
        if (1.0 + uz < 1e-12) {
            R[0] = 1.0; R[1] = 0.0; R[2] = 0.0; R[3] = 0.0; R[4] = -1.0; R[5] = 0.0; R[6] = 0.0; R[7] = 0.0;
            R[8] = -1.0;
        } else {
            const double h = 1.0 / (1.0 + uz);
            const double xy = (ux * uy) * h;
            R[0] = uz + (uy * uy) * h; R[1] = -xy; R[2] = -ux;
            R[3] = -xy; R[4] = uz + (ux * ux) * h; R[5] = -uy;
            R[6] = ux; R[7] = uy; R[8] = uz;
        }
    }
    for (int i = lane; i < NF; i += 64) {
        const double x = lat[3 * i], y = lat[3 * i + 1], z = lat[3 * i + 2];
        lq[0][i] = fma(R[6], z, fma(R[3], y, R[0] * x));
        lq[1][i] = fma(R[7], z, fma(R[4], y, R[1] * x));
        lq[2][i] = fma(R[8], z, fma(R[5], y, R[2] * x));
        double w;
        if (surf) {
            w = tab[n_phase * NF + i];
        } else {
            w = 0.0;
            for (int k = 0; k < n_phase; ++k) {
                const double f = frac ? (double)frac[(long long)k * nvol + l] : 1.0;
                w = w + f * tab[k * NF + i];
            }
        }
        wq[i] = (unsigned long long)llrint(w * kFix);
        bkey[i] = 0ull;
        col[i] = 0x7fffffff;
    }
    int nn[2];  // this lane's lattice points' hull neighbours, four indices (< 128) a word
    unsigned nbw[2][kHullNb / 4];
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
        const int i = min(h2 ? lane + 64 : lane, NF - 1);
        nn[h2] = hull[NF * kHullNb + i];
#pragma unroll
        for (int w = 0; w < kHullNb / 4; ++w) {
            unsigned v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) v |= ((unsigned)hull[i * kHullNb + 4 * w + b] & 0xffu) << (8 * b);
            nbw[h2][w] = v;
        }
    }
    __syncthreads();
    // seeds: each out-direction's closest lattice point, and the points' best values
    for (int m0 = 0; m0 < d; m0 += 4 * 64) {
        const int left = d - m0;
        if (left > 3 * 64) colour_seeds<4>(m0, d, NF, lq, adj_ptr, adj_idx, pos, l, per, wx, wy, seed_pt, bkey);
        else if (left > 2 * 64) colour_seeds<3>(m0, d, NF, lq, adj_ptr, adj_idx, pos, l, per, wx, wy, seed_pt, bkey);
        else if (left > 64) colour_seeds<2>(m0, d, NF, lq, adj_ptr, adj_idx, pos, l, per, wx, wy, seed_pt, bkey);
        else colour_seeds<1>(m0, d, NF, lq, adj_ptr, adj_idx, pos, l, per, wx, wy, seed_pt, bkey);
    }
    __syncthreads();
    for (int m = lane; m < d; m += 64) {
        const int bi = seed_pt[m];
        if (bi == kNoSeed) continue;
        double tx, ty, tz;
        edge_dir(m, tx, ty, tz);
        const double v = fma(lq[2][bi], tz, fma(lq[1][bi], ty, lq[0][bi] * tx));
        if (v == order_value(bkey[bi])) atomicMin(&col[bi], m);
    }
    __syncthreads();
    for (int t = lane; t < kCellHash; t += 64) {  // lq is free now (the fill's barriers publish this)
        hkey[t] = kNoOwner;
        hval[t] = 0ull;
    }
    const int i0 = lane, i1 = lane + 64;
    const bool ok0 = i0 < NF, ok1 = i1 < NF;
    const bool unseeded = __ballot((ok0 && col[i0] != 0x7fffffff) || (ok1 && col[i1] != 0x7fffffff)) == 0ull;
    if (ok0 && col[i0] == 0x7fffffff) col[i0] = unseeded ? 0 : -1;  // each lane its own points
    if (ok1 && col[i1] == 0x7fffffff) col[i1] = unseeded ? 0 : -1;
    for (int round = 0; round < NF; ++round) {
        if (ok0) snap[i0] = col[i0];
        if (ok1) snap[i1] = col[i1];
        __syncthreads();
        bool missing = false;
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
            const int i = h2 ? i1 : i0;
            if (i >= NF || snap[i] >= 0) continue;
            int c = -1;
#pragma unroll
            for (int t = kHullNb - 1; t >= 0; --t) {
                if (t < nn[h2]) {
                    const int ct = snap[(nbw[h2][t >> 2] >> (8 * (t & 3))) & 0xffu];
                    c = ct >= 0 ? ct : c;
                }
            }
            col[i] = c;
            missing = missing || c < 0;
        }
        const bool any = __ballot(missing) != 0ull;
        __syncthreads();
        if (!any) break;
    }
    // cells: colour -> fixed-point sum
    for (int h2 = 0; h2 < 2; ++h2) {
        const int i = h2 ? i1 : i0;
        if (i >= NF || col[i] < 0) continue;
        const unsigned short key = (unsigned short)col[i];
        int h = col[i] & (kCellHash - 1);
        while (true) {
            const unsigned short old = atomicCAS(&hkey[h], kNoOwner, key);
            if (old == kNoOwner || old == key) break;
            h = (h + 1) & (kCellHash - 1);
        }
        atomicAdd(&hval[h], wq[i]);
    }
    __syncthreads();
    const Real rl = rho ? rho[l] : (Real)0;
    const Real tsun = Tsun ? Tsun[l] : (Real)0;
    BlkT *blk = val + nodeoff[l];  // column-major: element (row n, column m) at m d + n
    for (int m = lane; m < d; m += 64) {
        const int h = cell_find(hkey, m);
        const double Q = h < 0 ? 0.0 : (double)(long long)hval[h] * kUnfix;
        const long long b = off + m;
        if (surf) {
            for (int c = 0; c < d; ++c) {
                if (kWriteQ) blk[(long long)c * d + m] = (BlkT)Q;
                else blk[(long long)c * d + m] = (BlkT)(T[off + c] * rl * (Real)Q);
            }
            if (!kWriteQ) S[b] = rl * mu0 * tsun * (Real)Q;
            qsun[b] = (float)Q;
        } else if (a < d) {
            if (kWriteQ) blk[(long long)a * d + m] = (BlkT)Q;
            else blk[(long long)a * d + m] = (BlkT)(T[off + a] * rl * (Real)Q);
        } else {
            if (!kWriteQ) S[b] = tsun * rl * (Real)Q;
            qsun[b] = (float)Q;
        }
    }
}


}  // namespace

// directions per workgroup of k_qbuild_big: as many as fill its columns
int qbuild_group_big(int NF) { return std::min(kBigCols / NF, kBigGroup); }

template <class Real>
void launch_qbuild(Scene &s, hipStream_t st, int write_q) {
    const int dm = (std::min(s.dmax, kWave) + 7) / 8 * 8;
    const size_t qshm = qbuild_lds(dm);
    if (s.sigma_mode == SG_SIGMA_COLOUR) {
        if (write_q) {
            hipLaunchKernelGGL((k_qcolour<Real, float, true>), dim3(s.N), dim3(64), 0, st, s.N, s.n_vol, s.adj_ptr,
                               s.adj_idx, s.pos, s.lat, (const uint4 *)s.lat_halves, s.tab, s.n_fib, s.n_phase,
                               node_frac(s), s.sun_in[0], s.sun_in[1],
                               s.sun_in[2], (Real)s.mu0, (const Real *)nullptr, (const Real *)nullptr,
                               (const Real *)nullptr, s.nodeoff, s.q, (Real *)nullptr, s.qsun, s.hull, s.periodic,
                               (long long)s.nx * kFx, (long long)s.ny * kFx, s.qscreen);
        } else {
            hipLaunchKernelGGL((k_qcolour<Real, Real, false>), dim3(s.N), dim3(64), 0, st, s.N, s.n_vol, s.adj_ptr,
                               s.adj_idx, s.pos, s.lat, (const uint4 *)s.lat_halves, s.tab, s.n_fib, s.n_phase,
                               node_frac(s), s.sun_in[0], s.sun_in[1],
                               s.sun_in[2], (Real)s.mu0, (const Real *)s.T, (const Real *)s.rho,
                               (const Real *)s.Tsun, s.nodeoff, (Real *)s.val, (Real *)s.S, s.qsun, s.hull, s.periodic,
                               (long long)s.nx * kFx, (long long)s.ny * kFx, s.qscreen);
        }
        if (s.n_big) {  // nodes of degree above 64: one workgroup per (node, incoming direction)
            if (write_q)
                hipLaunchKernelGGL((k_qcolour_big<Real, float, true>), dim3(s.n_bigdir), dim3(64), 0, st, s.n_big,
                                   s.big, s.bigdir, s.n_vol, s.adj_ptr, s.adj_idx, s.pos, s.lat, s.tab, s.n_fib,
                                   s.n_phase, node_frac(s), s.sun_in[0], s.sun_in[1], s.sun_in[2], (Real)s.mu0,
                                   (const Real *)nullptr, (const Real *)nullptr, (const Real *)nullptr, s.nodeoff, s.q,
                                   (Real *)nullptr, s.qsun, s.hull, s.periodic, (long long)s.nx * kFx,
                                   (long long)s.ny * kFx);
            else
                hipLaunchKernelGGL((k_qcolour_big<Real, Real, false>), dim3(s.n_bigdir), dim3(64), 0, st, s.n_big,
                                   s.big, s.bigdir, s.n_vol, s.adj_ptr, s.adj_idx, s.pos, s.lat, s.tab, s.n_fib,
                                   s.n_phase, node_frac(s), s.sun_in[0], s.sun_in[1], s.sun_in[2], (Real)s.mu0,
                                   (const Real *)s.T, (const Real *)s.rho, (const Real *)s.Tsun, s.nodeoff,
                                   (Real *)s.val, (Real *)s.S, s.qsun, s.hull, s.periodic, (long long)s.nx * kFx,
                                   (long long)s.ny * kFx);
        }
        return;
    }
    if (s.n_big) {  // nodes of degree above 64
        if (write_q)
            hipLaunchKernelGGL((k_qbuild_big<Real, float, true>), dim3(s.n_bigdir), dim3(256), 0, st, s.n_big, s.big,
                               s.bigdir, s.n_vol, s.adj_ptr, s.adj_idx, s.pos, s.lat, s.tab, s.n_fib, s.n_phase, node_frac(s),
                               s.sun_in[0], s.sun_in[1], s.sun_in[2], (Real)s.mu0, (const Real *)nullptr,
                               (const Real *)nullptr, (const Real *)nullptr, s.nodeoff, s.q, (Real *)nullptr, s.qsun,
                               qbuild_group_big(s.n_fib), s.periodic, (long long)s.nx * kFx,
                               (long long)s.ny * kFx, s.qscreen);
        else
            hipLaunchKernelGGL((k_qbuild_big<Real, Real, false>), dim3(s.n_bigdir), dim3(256), 0, st, s.n_big, s.big,
                               s.bigdir, s.n_vol, s.adj_ptr, s.adj_idx, s.pos, s.lat, s.tab, s.n_fib, s.n_phase, node_frac(s),
                               s.sun_in[0], s.sun_in[1], s.sun_in[2], (Real)s.mu0, (const Real *)s.T,
                               (const Real *)s.rho, (const Real *)s.Tsun, s.nodeoff, (Real *)s.val, (Real *)s.S, s.qsun,
                               qbuild_group_big(s.n_fib), s.periodic, (long long)s.nx * kFx,
                               (long long)s.ny * kFx, s.qscreen);
    }
    if (write_q) {
        hipLaunchKernelGGL((k_qbuild<Real, float, true>), dim3(s.N), dim3(64), qshm, st, s.N, s.n_vol, s.adj_ptr,
                           s.adj_idx, s.pos, s.lat, (const uint4 *)s.lat_halves, s.tab, s.n_fib, s.n_phase, node_frac(s), s.sun_in[0], s.sun_in[1],
                           s.sun_in[2], (Real)s.mu0, (const Real *)nullptr, (const Real *)nullptr,
                           (const Real *)nullptr, s.nodeoff, s.q, (Real *)nullptr, s.qsun, dm, s.periodic,
                           (long long)s.nx * kFx, (long long)s.ny * kFx, s.qscreen);
    } else {
        hipLaunchKernelGGL((k_qbuild<Real, Real, false>), dim3(s.N), dim3(64), qshm, st, s.N, s.n_vol, s.adj_ptr,
                           s.adj_idx, s.pos, s.lat, (const uint4 *)s.lat_halves, s.tab, s.n_fib, s.n_phase, node_frac(s), s.sun_in[0], s.sun_in[1],
                           s.sun_in[2], (Real)s.mu0, (const Real *)s.T, (const Real *)s.rho, (const Real *)s.Tsun,
                           s.nodeoff, (Real *)s.val, (Real *)s.S, s.qsun, dm, s.periodic, (long long)s.nx * kFx,
                           (long long)s.ny * kFx, s.qscreen);
    }
}

template void launch_qbuild<float>(Scene &, hipStream_t, int);
template void launch_qbuild<double>(Scene &, hipStream_t, int);

}  // namespace sg
