// The sweep and residual kernels of many wavelengths and their launches, instantiated by
// three sources that compile side by side: the whole sweeps (batched.hip), the sweeps over
// the front (batched_front.hip) and the FP64 residual (batched_residual.hip).
#pragma once

#include "device.hpp"
#include "internal.hpp"

namespace sg {

namespace {

// One node per wavefront, lanes = wavelengths (tiles of 64).  The node's phase-cell
// block Q is staged, coalesced, in the wavefront's LDS slice and its entries are read
// as broadcasts (measured: reading the columns through scalar loads instead exposes
// their latency, 1.4x slower at 64 wavelengths); the in-edge list and optical depths
// are loaded once, coalesced, and broadcast with readlane; eight input gathers are in
// flight at a time (the FP64 residual of an FP32 iterate, at four wavefronts per SIMD, asks for the next
// eight before it uses these: 2.69 -> 2.04 ms at 96x96x32, 64 wavelengths; the FP32 sweep at seven loses
// 5 % with the registers this takes, and an FP64 iterate's do not fit); the node's rows are accumulated in registers, the row count
// rounded up to a multiple of 8 (DB) so the column reads are unguarded (the LDS slice
// is padded past the block by 64 floats).
// kResidual: FP64 residual r = S - x + K x of an FP64 iterate instead of a sweep.
// exp(-(tau_s + s tau_a)) as one hardware exp2; its relative error (~|tau| 1e-7) is
// below that of the FP32 path integral itself.  The sweep and the FP64 residual use
// the same function, so iterative refinement sees one matrix.
__device__ __forceinline__ float edge_T(float ts, float ta, float s) {
    return __builtin_amdgcn_exp2f(-(ts + s * ta) * 1.4426950408889634f);
}

// acc + q x.  In FP64 the FP32 entry q >= 0 is taken as the double of the same bits, moved to the
// double's places (two 32-bit shifts, its value 2^-896 q) and x carries 2^896: the product is
// exact either way.  (Cloud 71x53x29, 12 wavelengths: the residual 400 -> 248 us with this, three
// wavefronts per SIMD instead of spilled sums, and one division per node.)
constexpr double kResidualScale = 0x1p896;
__device__ __forceinline__ float add_q(float acc, float q, float x) { return acc + q * x; }
__device__ __forceinline__ double add_q(double acc, float q, double x) {
    const unsigned b = __float_as_uint(q);
    return fma(__hiloint2double((int)(b >> 3), (int)(b << 29)), x, acc);
}
__device__ __forceinline__ float column_input(float T, float x) { return T * x; }
__device__ __forceinline__ double column_input(double T, double x) { return T * x * kResidualScale; }

// The sum and the largest quotient num / den of a node's rows (num >= 0, den > 0): the
// quotients are compared across, so there is one division per node (one per row took 80 of
// the 240 us of a sweep of cloud 71x53x29, 12 wavelengths).  A num that is not finite
// makes the sum so, and the quotient infinite.
struct RowMeasures {
    double sum = 0.0, num = 0.0, den = 1.0;
    __device__ __forceinline__ void add(double n, double d) {
        sum += n;
        const bool more = n * den > num * d;
        num = more ? n : num;
        den = more ? d : den;
    }
    __device__ __forceinline__ float2 value() const {
        const double worst = sum < __builtin_huge_val() ? num / den : __builtin_huge_val();
        return make_float2((float)sum, (float)worst);
    }
};

// n passes of 64 consecutive block elements from t0 into the wavefront's LDS slice
template <int n>
__device__ __forceinline__ void stage_q(const float *__restrict__ qg, float *__restrict__ qs, int t0, int nq,
                                        int lane) {
    float v[n];
#pragma unroll
    for (int j = 0; j < n; ++j) v[j] = qg[min(t0 + j * 64 + lane, nq - 1)];
#pragma unroll
    for (int j = 0; j < n; ++j) qs[min(t0 + j * 64 + lane, nq - 1)] = v[j];
}

// kMark: the rows whose value moved for any wavelength mark their head node and this one for
// the next sweep over the front (as the single-wavelength sweep does).
template <int DB, class XT, class YT, class AccT, bool kResidual, bool kMark>
__device__ __forceinline__ float2 wide_node(int N, int l, int lane, int lam, bool lv, float s, int nl, int monitor,
                                            float *__restrict__ qs, const long long *__restrict__ adj_ptr,
                                            const long long *__restrict__ nodeoff, const int *__restrict__ rev,
                                            const float *__restrict__ q, const float *__restrict__ qsun,
                                            const float *__restrict__ tau_s, const float *__restrict__ tau_a,
                                            const float *__restrict__ brho, const float *__restrict__ bsrc,
                                            const float *__restrict__ rhs, const XT *__restrict__ x,
                                            YT *__restrict__ y, const int *__restrict__ adj_idx,
                                            unsigned char *__restrict__ mark) {
    constexpr int kU = 8;
    const long long off = adj_ptr[l];
    const int d = (int)(adj_ptr[l + 1] - off);
    const long long base = nodeoff[l];
    // per in-edge data in lane m (lanes past d repeat the last in-edge), then the node's
    // phase-cell block into this wavefront's LDS slice: as many 64-element passes as the
    // block needs, at most 16 at a time (a wave-uniform switch into straight-line copies,
    // so the loads are issued back to back; out-of-range lanes reload and rewrite the last
    // element)
    const long long em = off + min(lane, d - 1);
    const int rv = rev[em];
    const float ts = tau_s[em], ta = tau_a[em];
    constexpr bool kAhead = sizeof(AccT) == 8 && sizeof(XT) == 4;  // the next eight gathers before these are used
    auto inputs = [&](int m0, XT(&xv)[kU]) {
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const int m = min(m0 + j, 63);
            const int r = __builtin_amdgcn_readlane(rv, m);
            xv[j] = (m0 + j < d && lv) ? x[(long long)r * nl + lam] : (XT)0;
        }
    };
    XT xv[kU];
    if (kAhead) inputs(0, xv);
    {
        const int nq = d * d;
        for (int t0 = 0; t0 < nq; t0 += 64 * 16) {
            switch (min(16, (nq - t0 + 63) >> 6)) {
#define SG_STAGE_CASE(n) \
    case n: stage_q<n>(q + base, qs, t0, nq, lane); break;
                SG_STAGE_CASE(1) SG_STAGE_CASE(2) SG_STAGE_CASE(3) SG_STAGE_CASE(4) SG_STAGE_CASE(5)
                SG_STAGE_CASE(6) SG_STAGE_CASE(7) SG_STAGE_CASE(8) SG_STAGE_CASE(9) SG_STAGE_CASE(10)
                SG_STAGE_CASE(11) SG_STAGE_CASE(12) SG_STAGE_CASE(13) SG_STAGE_CASE(14) SG_STAGE_CASE(15)
                default: stage_q<16>(q + base, qs, t0, nq, lane);
#undef SG_STAGE_CASE
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    AccT acc[DB];
#pragma unroll
    for (int n = 0; n < DB; ++n) acc[n] = (AccT)0;
    for (int m0 = 0; m0 < d; m0 += kU) {
        XT next[kU];
        if (!kAhead) inputs(m0, xv);
        else if (m0 + kU < d) inputs(m0 + kU, next);
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const int m = m0 + j;
            if (m < d) {
                const float tsm = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ts), m));
                const float tam = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ta), m));
                const AccT xm = column_input((AccT)edge_T(tsm, tam, s), (AccT)xv[j]);
                const float *qm = qs + m * d;  // column m: Q[n][m], n contiguous (LDS, uniform address)
#pragma unroll
                for (int n = 0; n < DB; ++n) acc[n] = add_q(acc[n], qm[n], xm);
            }
        }
        if (kAhead)
#pragma unroll
            for (int j = 0; j < kU; ++j) xv[j] = next[j];
    }
    RowMeasures measures;
    unsigned long long rows = 0ull;  // the rows that moved for any wavelength
    if (lv) {
        const float rl = brho[(long long)l * nl + lam];
        const float sl = bsrc[(long long)l * nl + lam];
#pragma unroll
        for (int n = 0; n < DB; ++n) {
            if (n < d) {
                const long long b = off + n;
                const long long bi = b * nl + lam;
                if (kResidual) {
                    const double Sb = (double)(rl * sl * qsun[b]);
                    const double rb = (Sb - (double)x[bi]) + (double)rl * (double)acc[n];
                    y[bi] = (YT)rb;
                    measures.add(fabs(rb), fabs((double)x[bi]) + kRelFloor);
                } else {
                    const float src = rhs ? rhs[bi] : rl * sl * qsun[b];
                    const float yv = src + rl * (float)acc[n];
                    y[bi] = (YT)yv;
                    if (kMark && __ballot(moved(yv, (float)x[bi]))) rows |= 1ull << n;
                    if (monitor) measures.add(fabs((double)yv - (double)x[bi]), fabs((double)yv) + kRelFloor);
                }
            }
        }
    }
    if (kMark) {  // every lane with a wavelength holds the same mask, and lane 0 has one
        const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)rows);
        const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(rows >> 32));
        const unsigned long long m = ((unsigned long long)hi << 32) | lo;
        if (lane < d && (m >> lane & 1ull)) {
            const int head = adj_idx[em];
            if (SG_IN(head, N, 0x40b)) mark[head] = 1;
        }
        if (m && lane == 0) mark[l] = 1;
    }
    return measures.value();
}

// Occupancy hints: at the requested waves per SIMD the compiler fits each instantiation
// without spilling (the FP32 sweep: 72 VGPRs at D = 40 instead of 98; the FP64 residual up
// to D = 40: 124 of an FP32 iterate instead of 144, four waves per SIMD instead of three, where five
// would spill its accumulators, and 122 of an FP64 iterate, which leaves no room for the next gathers;
// the larger FP64 residuals keep their natural allocation, since their accumulators alone fill four
// waves' registers).  The marking sweeps hold the heads and moved rows too and fit six; the largest
// degrees fit four (64, and 56 over the front).
template <int D, bool kResidual, int kMode>
constexpr int wide_waves_per_eu() {
    if (kResidual) return D <= 40 ? 4 : 1;
    if (D <= 40) return kMode ? 6 : 7;
    return D <= 48 || (D <= 56 && kMode <= kFrontFirst) ? 5 : 4;
}

// kMode 0: every node; kFrontFirst: every node, marking the nodes of the next sweep;
// kFrontOn: the nodes marked in `now` only, marking those of the next (see k_spmv_front:
// the same marks, spread over the wavefronts by the same skewed stride; spent is cleared).
// 96x96x32, 64 wavelengths: whole sweeps 1.11 to 1.45 ms, the last six of ten 0.61 falling
// to 0.24 ms; a stream of the visited nodes' inputs and results, as a whole sweep.
enum { kFrontOn = kFrontFirst + 1 };
template <int D, class XT, class YT, class AccT, bool kResidual, int kMode>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(wide_waves_per_eu<D, kResidual, kMode>()))) void k_spmm_wide(
    int N, int nl, int groups, const long long *__restrict__ adj_ptr, const long long *__restrict__ nodeoff,
    const int *__restrict__ rev, const float *__restrict__ q, const float *__restrict__ qsun,
    const float *__restrict__ tau_s, const float *__restrict__ tau_a, const float *__restrict__ abs_scale,
    const float *__restrict__ brho, const float *__restrict__ bsrc, const float *__restrict__ rhs,
    const XT *__restrict__ x, YT *__restrict__ y, float2 *__restrict__ meas, int monitor, int dmax,
    const int *__restrict__ adj_idx, const unsigned char *__restrict__ now, unsigned char *__restrict__ next,
    unsigned long long *__restrict__ spent, int skew) {
    extern __shared__ float qs_all[];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lam = blockIdx.y * 64 + lane;
    const bool lv = lam < nl;
    const float s = lv ? abs_scale[lam] : 0.f;
    float *qs = qs_all + (size_t)w * (dmax * dmax + 64);  // + padding: whole-column reads past d
    const int waves = blockDim.x >> 6;
    auto node = [&](int l) {
        const int d = (int)(adj_ptr[l + 1] - adj_ptr[l]);
        if (d == 0) {  // an isolated node: no rows
            if (monitor && lv) meas[(long long)l * nl + lam] = make_float2(0.f, 0.f);
            return;
        }
#ifdef SG_DEBUG_BOUNDS
        {  // the node's Q block and its in-edges' reverse ids
            bool ok = SG_IN(nodeoff[l] + (long long)d * d - 1, nodeoff[N], 0x401);
            if (lane < d) ok = SG_IN(rev[adj_ptr[l] + lane], adj_ptr[N], 0x402) && ok;
            if (!__all(ok)) return;
        }
#endif
        const int bucket = (d + 7) >> 3;
        float2 part = make_float2(0.f, 0.f);
#define SG_NODE(DB)                                                                                               \
    part = wide_node<DB, XT, YT, AccT, kResidual, kMode != 0>(N, l, lane, lam, lv, s, nl, monitor, qs, adj_ptr, nodeoff, \
                                                              rev, q, qsun, tau_s, tau_a, brho, bsrc, rhs, x, y,   \
                                                              adj_idx, next)
        if (bucket <= 1) { SG_NODE(8); }
        else if (bucket == 2) { if constexpr (D >= 16) SG_NODE(16); }
        else if (bucket == 3) { if constexpr (D >= 24) SG_NODE(24); }
        else if (bucket == 4) { if constexpr (D >= 32) SG_NODE(32); }
        else if (bucket == 5) { if constexpr (D >= 40) SG_NODE(40); }
        else if (bucket == 6) { if constexpr (D >= 48) SG_NODE(48); }
        else if (bucket == 7) { if constexpr (D >= 56) SG_NODE(56); }
        else { if constexpr (D >= 64) SG_NODE(64); }
#undef SG_NODE
        if (monitor && lv) meas[(long long)l * nl + lam] = part;  // per node and wavelength
    };
    if constexpr (kMode == kFrontOn) {
        const int W = gridDim.x * waves, wv = blockIdx.x * waves + w;
        if (blockIdx.y == 0)
            for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < (N + 7) / 8; t += gridDim.x * blockDim.x) spent[t] = 0ull;
        for (int j0 = 0; j0 * (long long)W < N; j0 += 64) {
            const int mine = (j0 + lane) * (long long)W < N ? front_node(wv, j0 + lane, W, skew) : N;
            unsigned long long todo = __ballot(mine < N && now[min(mine, N - 1)]);
            for (; todo; todo &= todo - 1) node(__builtin_amdgcn_readlane(mine, __builtin_ctzll(todo)));
        }
    } else {
        for (int g = blockIdx.x; g < groups; g += gridDim.x) {
            const int l = __builtin_amdgcn_readfirstlane(g * waves + w);
            if (l >= N) break;
            node(l);
        }
    }
}

// ---- wavelength tiles narrower than a wavefront -------------------------------------
// For n_lambda <= 32 a wavefront holds 64 / W node slots of W wavelength lanes each, so
// a small wavelength count does not leave lanes idle.  Each slot's in-edge data (rev,
// tau_s, tau_a) goes to a small LDS slice.  The phase-cell columns pass through LDS a few
// at a time: a slot's lanes load them side by side, the next ones while these are used, and
// read them as 16-byte broadcasts (the slots' slices four words apart, so that their
// reads fall on different banks).  Read straight from memory with 16-byte loads, each lane of a
// slot took the same sixteen bytes through the vector memory path, and that path bound the
// sweep: cloud 71x53x29, 12 wavelengths, a whole sweep 331 -> 162 us, over the front 296 falling
// to 82 -> 166 falling to 34 us, the FP64 residual 427 -> 248 us.
// Per lane the arithmetic is exactly that of the full-wavefront kernel (same expressions,
// columns in the same order), so the two give the same bits.
typedef float f4u __attribute__((ext_vector_type(4)));

template <int W, int DB>
struct PackTile {
    static constexpr int kLoads = (DB + W - 1) / W;              // per lane and column
    static constexpr int kStride = kLoads * W;                   // rows of a staged column
    static constexpr int kCols = 4;                               // columns staged at a time
    static constexpr int kSlice = kCols * kStride + 4;           // words of a slot
};
// this lane's own row of the node's in-edges, read again after the columns (the empty statement keeps the
// compiler from holding it, two registers, through them)
__device__ __forceinline__ long long edges_from(const long long *__restrict__ adj_ptr, int l) {
    asm volatile("" : "+v"(l));
    return adj_ptr[l];
}
template <int W, int D>
constexpr int pack_slice() {  // the largest slice of the degree buckets up to D
    if constexpr (D <= 8) return PackTile<W, 8>::kSlice;
    else return PackTile<W, D>::kSlice > pack_slice<W, D - 8>() ? PackTile<W, D>::kSlice : pack_slice<W, D - 8>();
}

template <int W, int DB, class XT, class YT, class AccT, bool kResidual, bool kMark>
__device__ __forceinline__ float2 pack_node(int l, int lam, bool lv, float s, int nl, int monitor, 
                                            int d, long long base, int dw, const int *__restrict__ srv,
                                            const float *__restrict__ sts, const float *__restrict__ sta,
                                            float *__restrict__ qs, const long long *__restrict__ adj_ptr, const float *__restrict__ q,
                                            const float *__restrict__ qsun, const float *__restrict__ brho,
                                            const float *__restrict__ bsrc, const float *__restrict__ rhs,
                                            const XT *__restrict__ x, YT *__restrict__ y, unsigned long long &rows) {
    using P = PackTile<W, DB>;
    // one staged column less where four do not fit the registers
    constexpr int kCols = P::kCols - (W == 8 && (sizeof(XT) == 8 || (kMark && DB == 40)));
    AccT acc[DB];
#pragma unroll
    for (int n = 0; n < DB; ++n) acc[n] = (AccT)0;
    // columns m0.. of the block, rows lam, lam + W, .. in this lane, and their inputs.  Slots with
    // fewer in-edges repeat their last column with a zero input: adding Q * 0 leaves every
    // valid row's sum unchanged
    float qv[kCols * P::kLoads];
    XT xv[kCols];
    auto load = [&](int m0) {
#pragma unroll
        for (int j = 0; j < kCols; ++j) {
            const int mc = min(m0 + j, d - 1);
            const float *qm = q + base + mc * d;
#pragma unroll
            for (int k = 0; k < P::kLoads; ++k) qv[j * P::kLoads + k] = qm[lam + W * k];
            xv[j] = (m0 + j < d && lv) ? x[(long long)srv[mc] * nl + lam] : (XT)0;
        }
    };
    load(0);
    for (int m0 = 0; m0 < dw; m0 += kCols) {
        AccT xm[kCols];
#pragma unroll
        for (int j = 0; j < kCols; ++j) {
            const int mc = min(m0 + j, d - 1);
#pragma unroll
            for (int k = 0; k < P::kLoads; ++k) qs[j * P::kStride + lam + W * k] = qv[j * P::kLoads + k];
            xm[j] = column_input((AccT)edge_T(sts[mc], sta[mc], s), (AccT)xv[j]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (m0 + kCols < dw) load(m0 + kCols);
#pragma unroll
        for (int j = 0; j < kCols; ++j) {
            if (m0 + j >= dw) break;
            const f4u *qm = reinterpret_cast<const f4u *>(qs + j * P::kStride);
#pragma unroll
            for (int c = 0; c < DB / 4; ++c) {
                const f4u v = qm[c];
                acc[4 * c] = add_q(acc[4 * c], v.x, xm[j]);
                acc[4 * c + 1] = add_q(acc[4 * c + 1], v.y, xm[j]);
                acc[4 * c + 2] = add_q(acc[4 * c + 2], v.z, xm[j]);
                acc[4 * c + 3] = add_q(acc[4 * c + 3], v.w, xm[j]);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    RowMeasures measures;
    if (lv) {
        const long long off = edges_from(adj_ptr, l);
        const float rl = brho[(long long)l * nl + lam];
        const float sl = bsrc[(long long)l * nl + lam];
#pragma unroll
        for (int n = 0; n < DB; ++n) {
            if (n < d) {
                const long long b = off + n;
                const long long bi = b * nl + lam;
                if (kResidual) {
                    const double Sb = (double)(rl * sl * qsun[b]);
                    const double rb = (Sb - (double)x[bi]) + (double)rl * (double)acc[n];
                    y[bi] = (YT)rb;
                    measures.add(fabs(rb), fabs((double)x[bi]) + kRelFloor);
                } else {
                    const float src = rhs ? rhs[bi] : rl * sl * qsun[b];
                    const float yv = src + rl * (float)acc[n];
                    y[bi] = (YT)yv;
                    if (kMark && moved(yv, (float)x[bi])) rows |= 1ull << n;
                    if (monitor) measures.add(fabs((double)yv - (double)x[bi]), fabs((double)yv) + kRelFloor);
                }
            }
        }
    }
    return measures.value();
}

// Four waves per SIMD (the compiler would hoist the previous values of all rows and leave three);
// the FP64 residual's accumulators fit three from D = 32 to 40.  The rows beyond that keep the natural
// allocation.  No instantiation spills: the node's first edge is read again after the columns
// (edges_from), a slot's arrays lie behind one LDS address, and the sweep over the front recomputes its node.
// (Before, 2 to 10 spilled values; a wave less instead made 12 wavelengths on 71x53x29 7 % slower.)
template <int D, bool kResidual>
constexpr int pack_waves_per_eu() {
    return D > 40 ? 1 : kResidual && D > 24 ? 3 : 4;
}

// kMode: as k_spmm_wide.  Over the front, each slot of the wavefront takes the next of its
// marked nodes.
template <int W, int D, class XT, class YT, class AccT, bool kResidual, int kMode>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pack_waves_per_eu<D, kResidual>()))) void k_spmm_pack(
    int N, int nl, int groups, const long long *__restrict__ adj_ptr, const long long *__restrict__ nodeoff,
    const int *__restrict__ rev, const float *__restrict__ q, const float *__restrict__ qsun,
    const float *__restrict__ tau_s, const float *__restrict__ tau_a, const float *__restrict__ abs_scale,
    const float *__restrict__ brho, const float *__restrict__ bsrc, const float *__restrict__ rhs,
    const XT *__restrict__ x, YT *__restrict__ y, float2 *__restrict__ meas, int monitor,
    const int *__restrict__ adj_idx, const unsigned char *__restrict__ now, unsigned char *__restrict__ next,
    unsigned long long *__restrict__ spent, int skew) {
    constexpr int P = 64 / W;  // node slots per wavefront
    struct __align__(16) Slot {  // of one LDS address
        float qs[pack_slice<W, D>()];
        int rv[D];
        float ts[D], ta[D];
    };
    __shared__ Slot slots[4][P];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int k = lane / W, lam = lane - k * W;
    const bool lam_ok = lam < nl;
    const float s = lam_ok ? abs_scale[lam] : 0.f;
    Slot &slot = slots[w][k];
    int *srv = slot.rv;
    float *sts = slot.ts, *sta = slot.ta, *qs = slot.qs;
    auto slot_nodes = [&](int l) {  // node l per slot (l >= N: none)
        const bool node_ok = l < N;
        long long off = 0, base = 0;
        int d = 0;
        if (node_ok) {
            off = adj_ptr[l];
            d = (int)(adj_ptr[l + 1] - off);
            base = nodeoff[l];
        }
        for (int m = lam; m < d; m += W) {
            const long long e = off + m;
            srv[m] = SG_IN(rev[e], adj_ptr[N], 0x403) ? rev[e] : (int)e;
            sts[m] = tau_s[e];
            sta[m] = tau_a[e];
        }
        __builtin_amdgcn_wave_barrier();
        int dw = d;  // the wavefront's largest degree (uniform loop bound)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) dw = max(dw, __shfl_xor(dw, o, 64));
        dw = __builtin_amdgcn_readfirstlane(dw);
        const bool lv = node_ok && lam_ok && d > 0;
        float2 part = make_float2(0.f, 0.f);
        unsigned long long rows = 0ull;  // this lane's rows that moved
        if (dw > 0) {
            const int bucket = (dw + 7) >> 3;
#define SG_PACK(DB)                                                                                            \
    part = pack_node<W, DB, XT, YT, AccT, kResidual, kMode != 0>(l, lam, lv, s, nl, monitor, max(d, 1), base, dw,  \
                                                                 srv, sts, sta, qs, adj_ptr, q, qsun, brho, bsrc, rhs, x, \
                                                                 y, rows)
            if (bucket <= 1) { SG_PACK(8); }
            else if (bucket == 2) { if constexpr (D >= 16) SG_PACK(16); }
            else if (bucket == 3) { if constexpr (D >= 24) SG_PACK(24); }
            else if (bucket == 4) { if constexpr (D >= 32) SG_PACK(32); }
            else if (bucket == 5) { if constexpr (D >= 40) SG_PACK(40); }
            else if (bucket == 6) { if constexpr (D >= 48) SG_PACK(48); }
            else if (bucket == 7) { if constexpr (D >= 56) SG_PACK(56); }
            else { if constexpr (D >= 64) SG_PACK(64); }
#undef SG_PACK
        }
        if (kMode) {  // the rows that moved for any of the slot's wavelengths
            unsigned lo = (unsigned)rows, hi = (unsigned)(rows >> 32);
#pragma unroll
            for (int o = W / 2; o > 0; o >>= 1) {
                lo |= __shfl_xor(lo, o, 64);
                hi |= __shfl_xor(hi, o, 64);
            }
            const long long from = node_ok ? edges_from(adj_ptr, l) : 0;
            for (int m = lam; m < d; m += W)
                if ((m < 32 ? lo >> m : hi >> (m - 32)) & 1u) {
                    const int head = adj_idx[from + m];
                    if (SG_IN(head, N, 0x40c)) next[head] = 1;
                }
            if ((lo | hi) && lam == 0) next[l] = 1;
        }
        if (monitor && node_ok && lam_ok) meas[(long long)l * nl + lam] = part;
        __builtin_amdgcn_wave_barrier();  // the slices are rewritten by the next nodes
    };
    if constexpr (kMode == kFrontOn) {
        const int V = gridDim.x * 4, wv = blockIdx.x * 4 + w;
        for (int t = blockIdx.x * 256 + threadIdx.x; t < (N + 7) / 8; t += gridDim.x * 256) spent[t] = 0ull;
        for (int j0 = 0; j0 * (long long)V < N; j0 += 64) {
            const int mine = (j0 + lane) * (long long)V < N ? front_node(wv, j0 + lane, V, skew) : N;
            unsigned long long todo = __ballot(mine < N && now[min(mine, N - 1)]);
            while (todo) {
                unsigned long long m = todo;  // slot k: without its k lowest marks
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    m = i < k ? m & (m - 1) : m;
                    todo &= todo - 1;
                }
                slot_nodes(m ? front_node(wv, j0 + __builtin_ctzll(m), V, skew) : N);
            }
        }
    } else {
        for (int g = blockIdx.x; g < groups; g += gridDim.x) {
            const int l0 = __builtin_amdgcn_readfirstlane((g * 4 + w) * P);
            if (l0 >= N) break;
            slot_nodes(l0 + k);
        }
    }
}

}  // namespace

// front: which nodes (see front_of); kMode is its kind, one of the kernels' modes
template <int W, class XT, class YT, class AccT, bool kRes, int kMode>
static void launch_pack(Scene &s, hipStream_t st, int grid, const float *rhs, const XT *x, YT *y, int monitor, int front) {
    const int groups = batched_groups(s);
    static std::atomic<uint64_t> kept[8];  // per degree bucket
#define SG_PK(DD)                                                                                                  \
    if (kMode == kFrontOn)                                                                                         \
        grid = std::min(groups, resident_groups(k_spmm_pack<W, DD, XT, YT, AccT, kRes, kMode>, 256, 0, kept[DD / 8 - 1])); \
    hipLaunchKernelGGL((k_spmm_pack<W, DD, XT, YT, AccT, kRes, kMode>), dim3(grid), dim3(256), 0, st, s.N, s.n_lambda, \
                       groups, s.adj_ptr, s.nodeoff, s.rev, s.q, s.qsun, (const float *)s.tau_s, (const float *)s.tau_a, \
                       s.abs_scale_d, s.brho, s.bsrc, rhs, x, y, s.meas, monitor, s.adj_idx, front_marks_of(s, front), \
                       front_marks_of(s, front + 1), (unsigned long long *)front_marks_of(s, front + 2), front_skew(grid * 4))
    if (s.dmax <= 16) { SG_PK(16); }
    else if (s.dmax <= 24) { SG_PK(24); }
    else if (s.dmax <= 32) { SG_PK(32); }
    else if (s.dmax <= 40) { SG_PK(40); }
    else if (s.dmax <= 48) { SG_PK(48); }
    else if (s.dmax <= 56) { SG_PK(56); }
    else { SG_PK(64); }
#undef SG_PK
}

template <class XT, class YT, class AccT, bool kRes, int kMode>
static void launch_wide(Scene &s, hipStream_t st, int grid, const float *rhs, const XT *x, YT *y, int monitor, int front) {
    const int W = batched_tile(s);
    const int waves = wide_waves(s);
    grid = std::max(1, std::min(grid, batched_groups(s)));
    if (W == 8) return launch_pack<8, XT, YT, AccT, kRes, kMode>(s, st, grid, rhs, x, y, monitor, front);
    if (W == 16) return launch_pack<16, XT, YT, AccT, kRes, kMode>(s, st, grid, rhs, x, y, monitor, front);
    if constexpr (kMode == 0)  // (a 32-lane tile takes whole sweeps)
        if (W == 32) return launch_pack<32, XT, YT, AccT, kRes, kMode>(s, st, grid, rhs, x, y, monitor, front);
    const int groups = batched_groups(s);
    dim3 gr(grid, (s.n_lambda + 63) / 64);
    const size_t shm = (size_t)waves * (s.dmax * s.dmax + 64) * sizeof(float);
    static std::atomic<uint64_t> kept[8];  // per degree bucket
#define SG_WIDE(DD)                                                                                                 \
    if (kMode == kFrontOn)                                                                                          \
        gr.x = std::max(1, std::min(groups, resident_groups(k_spmm_wide<DD, XT, YT, AccT, kRes, kMode>, 64 * waves, shm, \
                                                            kept[DD / 8 - 1]) / (int)gr.y));                        \
    hipLaunchKernelGGL((k_spmm_wide<DD, XT, YT, AccT, kRes, kMode>), gr, dim3(64 * waves), shm, st, s.N, s.n_lambda,  \
                       groups, s.adj_ptr, s.nodeoff, s.rev, s.q, s.qsun, (const float *)s.tau_s, (const float *)s.tau_a, \
                       s.abs_scale_d, s.brho, s.bsrc, rhs, x, y, s.meas, monitor, s.dmax, s.adj_idx,                 \
                       front_marks_of(s, front), front_marks_of(s, front + 1),                                      \
                       (unsigned long long *)front_marks_of(s, front + 2), front_skew((int)gr.x * waves))
    if (s.dmax <= 16) { SG_WIDE(16); }
    else if (s.dmax <= 24) { SG_WIDE(24); }
    else if (s.dmax <= 32) { SG_WIDE(32); }
    else if (s.dmax <= 40) { SG_WIDE(40); }
    else if (s.dmax <= 48) { SG_WIDE(48); }
    else if (s.dmax <= 56) { SG_WIDE(56); }
    else { SG_WIDE(64); }
#undef SG_WIDE
}

}  // namespace sg
