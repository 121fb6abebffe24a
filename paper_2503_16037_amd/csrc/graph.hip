// The scattering graph G(R, L) (Sec. 2, Eq. 4) of a scene's nodes, built on the
// device: which node pairs are coupled.
//
// Relative positions (Sec. 3): node positions are centred and scaled to unit
// standard deviation per axis; their projection on the principal axes that
// follows is a rotation and leaves every distance, hence every coupling,
// unchanged, so the couplings are evaluated on the scaled coordinates q.  The
// coupling C = sqrt(mu_i mu_j) / |q_i - q_j| (Eq. 4) is ranked through its square
//   k = (mu_i * mu_j) / ((u*u + v*v) + w*w),   (u, v, w) = q_i - q_j,
// in FP64 with exactly this operation order (no contraction: the selection is an
// integer decision taken from these values); surface nodes couple with
// albedo x the largest mu_s (Sec. 3) and two surface nodes never couple.
//
// Pruning.  A pair with k >= t satisfies |q_i - q_j|^2 <= mu_i mu_max / t, so for a
// threshold t every partner of node i lies in an axis-aligned box of voxels around
// it (half-width sqrt(mu_i mu_max / t) standard deviations per axis; partners of higher
// id only, so its layers start at the node's own).  Box sizes
// differ by orders of magnitude (a strongly scattering node reaches far), so the
// cells of all boxes are flattened, node after node and within a box in increasing
// partner id (x fastest, then y, z, then the surface row), and evaluated one per
// thread; each thread finds its node by binary search in the prefix sum of the box
// sizes.  k is computed for the partners of higher id and the qualifying pairs are
// compacted in cell order (ballot and workgroup prefix, then the workgroups'
// prefix sum), so the candidate list is ordered by (i, j).
//   threshold mode: t = c_min^2, keep k > t;
//   top-n mode: t = the lowest threshold whose boxes hold at most a fixed budget
//   of cells; if at least n pairs have k >= t, the n best of them are the answer;
//   otherwise every pair is evaluated against a threshold taken from a sample of the
//   pairs (k_graph_all), so that only about n of them become candidates.
// General nodes (the path points of the lines of sight, Sec. 2) are not tied to voxels
// and always take the second way; its candidates are then sorted by (i, j).  Up to 2^23
// pairs are listed in order instead (k_graph_every), without a threshold.
// The n best of the candidates are selected, not sorted: a radix selection finds the
// n-th largest k, and a compaction in list order keeps the larger ones and the first of
// the equal ones (equal couplings: the smaller pair first).  The selected pairs are the
// forward half of the adjacency in row order; a stable sort by partner gives the other.
// Scans, the evaluated-pair sum and the sorts are this file's own: a three-phase
// exclusive scan, and a stable least-significant-digit radix sort (8-bit digits of the
// bits that node ids use, one wavefront per tile of 1024 keys, a key's rank among equal
// digits of its 64-key round from eight ballots).  A pair's code is i << 32 | j.
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <memory>
#include <string>
#include <vector>

#include "device.hpp"
#include "internal.hpp"

#pragma clang fp contract(off)

namespace sg {

namespace {

// Box cells a candidate pass may visit for the n strongest couplings: sixteen times n at
// first (one to five in ten cells of a box hold a candidate, by how much mu varies), then four
// times as many while the fitted threshold leaves fewer than n, up to 2^29
// (SG_GRAPH_CELL_BUDGET fixes a single budget, e.g. to exercise the ranking of every pair on
// small inputs).  64x64x32 plume, n = 1,507,328: 2^26 cells 0.60 ms of passes
// (2^25 0.40, 10 n 0.20 but then only 9 % more candidates than asked for, 16 n 0.29).
constexpr unsigned long long kMostBudget = 1ull << 29;
// candidates of all pairs that are listed, beyond four times as many as were expected, before the
// selection over all pairs takes over (a list costs a second pass, its sort and 32 bytes a pair, the
// selection thirteen passes: 16.2 M couplings equal, 13 ms by a list, 17.4 M 31 ms and 72 M 44 ms by
// selection; 2.2 G 0.5 s, which no list holds)
constexpr unsigned long long kMostListed = 1ull << 25;
// boxes of one voxel per node already beyond this are refused (with the default budgets)
constexpr unsigned long long kMostCells = 1ull << 26;

std::vector<unsigned long long> cell_budgets(unsigned long long n) {
    const char *v = std::getenv("SG_GRAPH_CELL_BUDGET");
    const unsigned long long fixed = v ? std::strtoull(v, nullptr, 10) : 0ull;
    if (fixed) return {fixed};
    std::vector<unsigned long long> b;
    for (unsigned long long k = std::max(16ull * n, 1ull << 22); k < kMostBudget; k *= 4) b.push_back(k);
    b.push_back(kMostBudget);
    return b;
}

struct Geo {
    int nx, ny, nz, surface;
    int general;               // 1: general volume nodes (every pair ranked), 0: one per voxel
    long long nvox, nvol, N;   // voxels, volume nodes, all nodes
    double mean[3], sd[3];  // per-axis centre and scale (sd = 0: the axis is ignored)
    double mu_max;
};

sg_status gfail(sg_status st, const std::string &msg) {
    set_error(msg);
    return st;
}

#define GHIP(call)                                                                                   \
    do {                                                                                             \
        hipError_t e_ = (call);                                                                      \
        if (e_ != hipSuccess) {                                                                      \
            ctx->sticky.store(1);                                                                    \
            return gfail(SG_E_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_));            \
        }                                                                                            \
    } while (0)
#define GTRY(x)                          \
    do {                                 \
        sg_status st_ = (x);             \
        if (st_ != SG_OK) return st_;    \
    } while (0)

// device blocks from the context pool, released on scope exit once the stream that uses
// them has drained (the pool serves other streams too)
struct Dev {
    Ctx *ctx;
    hipStream_t st;
    std::vector<void *> blocks;
    Dev(Ctx *c, hipStream_t s) : ctx(c), st(s) {}
    ~Dev() {
        if (!blocks.empty()) (void)hipStreamSynchronize(st);
        for (void *p : blocks) pool_free(ctx, p);
    }
    template <class T>
    sg_status get(T **p, size_t n) {
        void *q = nullptr;
        GTRY(pool_alloc(ctx, std::max<size_t>(n, 1) * sizeof(T), &q));
        blocks.push_back(q);
        *p = static_cast<T *>(q);
        return SG_OK;
    }
    // the blocks taken since there were `level` of them go back before the others, once the stream drained
    sg_status drop(size_t level) {
        GHIP(hipStreamSynchronize(st));
        for (; blocks.size() > level; blocks.pop_back()) pool_free(ctx, blocks.back());
        return SG_OK;
    }
};

// ---- kernels ---------------------------------------------------------------------------

// Checks and exact integer moments of the inputs, in one pass: sums of the positions and (in
// two halves: they pass 64 bits) of their squares per axis over all nodes, the largest mu_s,
// the first node outside its voxel (general nodes: outside the box; x = 0 and y = 0 allowed,
// a periodic wrap puts nodes there), and whether a mu_s or an albedo is out of range.
struct Moments {
    unsigned long long s1[3], lo[3], hi[3], bad_node;
    unsigned mu_max, bad_mu, bad_albedo, pad;
};
__global__ __launch_bounds__(256) void k_graph_moments(Geo g, const int *__restrict__ pos,
                                                       const float *__restrict__ mu_s,
                                                       const float *__restrict__ albedo, Moments *__restrict__ out) {
    unsigned long long v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, bad = ~0ull;
    unsigned top = 0u, bad_mu = 0u, bad_albedo = 0u;
    const long long n = max(g.N, g.nvox), stride = (long long)gridDim.x * 256;
    for (long long l = blockIdx.x * 256ll + threadIdx.x; l < n; l += stride) {
        if (l < g.nvox) {
            const float a = mu_s[l];
            if (a >= 0.0f && a < __builtin_inff()) top = max(top, __float_as_uint(a) & 0x7fffffffu);
            else bad_mu = 1u;
        }
        if (l >= g.N) continue;
        long long p[3];
        if (l < g.nvol) {
            const long long c[3] = {l % g.nx, (l / g.nx) % g.ny, l / ((long long)g.nx * g.ny)};
            const long long w[3] = {g.nx * kFx, g.ny * kFx, g.nz * kFx};
            bool in = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                p[a] = pos[3 * l + a];
                const long long lo = g.general ? (a < 2 ? -1 : 0) : c[a] * kFx;
                in = in && p[a] > lo && p[a] < (g.general ? w[a] : lo + kFx);
            }
            if (!in) bad = min(bad, (unsigned long long)l);
        } else {
            const long long c = l - g.nvol;
            p[0] = (c % g.nx) * kFx + kFx / 2;
            p[1] = (c / g.nx) * kFx + kFx / 2;
            p[2] = 0;
            const float a = albedo[c];
            if (!(a >= 0.0f && a <= 1.0f)) bad_albedo = 1u;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const unsigned long long sq = (unsigned long long)(p[a] * p[a]);
            v[a] += (unsigned long long)p[a];
            v[3 + a] += sq & 0xffffffffull;
            v[6 + a] += sq >> 32;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int a = 0; a < 9; ++a) v[a] += __shfl_xor(v[a], o, 64);
        bad = min(bad, __shfl_xor(bad, o, 64));
        top = max(top, __shfl_xor(top, o, 64));
        bad_mu |= __shfl_xor(bad_mu, o, 64);
        bad_albedo |= __shfl_xor(bad_albedo, o, 64);
    }
    // the wavefronts meet in LDS, and one thread per value takes it out (same-address atomics
    // from every wavefront took 0.2 ms)
    __shared__ unsigned long long sv[4][9], sbad[4];
    __shared__ unsigned stop[4], sflag[4];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int a = 0; a < 9; ++a) sv[w][a] = v[a];
        sbad[w] = bad;
        stop[w] = top;
        sflag[w] = bad_mu | bad_albedo << 1;
    }
    __syncthreads();
    if (threadIdx.x < 9) {
        unsigned long long t = 0ull;
        for (int k = 0; k < 4; ++k) t += sv[k][threadIdx.x];
        atomicAdd(&out->s1[0] + threadIdx.x, t);  // s1, lo and hi lie one after the other
    } else if (threadIdx.x == 9) {
        for (int k = 1; k < 4; ++k) {
            bad = min(k == 1 ? sbad[0] : bad, sbad[k]);
            top = max(k == 1 ? stop[0] : top, stop[k]);
        }
        const unsigned flag = sflag[0] | sflag[1] | sflag[2] | sflag[3];
        if (bad != ~0ull) atomicMin(&out->bad_node, bad);
        atomicMax(&out->mu_max, top);
        if (flag & 1u) atomicOr(&out->bad_mu, 1u);
        if (flag & 2u) atomicOr(&out->bad_albedo, 1u);
    }
}

// fixed-point position, coupling coefficient and scaled coordinates of every node; a
// general node couples with the mu_s of the voxel holding it
__global__ void k_graph_nodes(Geo g, const int *__restrict__ pos, const float *__restrict__ mu_s,
                              const float *__restrict__ albedo, long long *__restrict__ P, double *__restrict__ q,
                              double *__restrict__ mu) {
#pragma clang fp contract(off)
    const long long l = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (l >= g.N) return;
    long long p[3];
    if (l < g.nvol) {
        p[0] = pos[3 * l];
        p[1] = pos[3 * l + 1];
        p[2] = pos[3 * l + 2];
        const long long v =
            g.general ? p[0] / kFx + (long long)g.nx * (p[1] / kFx + (long long)g.ny * (p[2] / kFx)) : l;
        mu[l] = (double)mu_s[v];
    } else {
        const long long c = l - g.nvol;
        p[0] = (c % g.nx) * kFx + kFx / 2;
        p[1] = (c / g.nx) * kFx + kFx / 2;
        p[2] = 0;
        mu[l] = (double)albedo[c] * g.mu_max;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        P[3 * l + a] = p[a];
        q[3 * l + a] = g.sd[a] > 0.0 ? ((double)p[a] - g.mean[a]) / g.sd[a] : 0.0;
    }
}

__device__ __forceinline__ double pair_key(const double *__restrict__ q, const double *__restrict__ mu, long long i,
                                           long long j) {
#pragma clang fp contract(off)
    const double u = q[3 * i] - q[3 * j], v = q[3 * i + 1] - q[3 * j + 1], w = q[3 * i + 2] - q[3 * j + 2];
    const double d2 = (u * u + v * v) + w * w;
    return (mu[i] * mu[j]) / d2;
}

// The box of node i's possible partners at threshold t: voxel index ranges per axis
// (lo > hi: empty) and whether the surface row is inside.
struct Box {
    long long lo[3], hi[3];
    bool surf;
};

__device__ __forceinline__ Box node_box(const Geo &g, const long long *__restrict__ P, const double *__restrict__ mu,
                                        long long i, double t) {
    Box b;
    const double mi = mu[i];
    const long long n[3] = {g.nx, g.ny, g.nz};
    // k = 0 for every pair of this node, or a surface node (its pairs with volume
    // nodes are found from the volume side; two surface nodes never couple)
    if (!(mi > 0.0) || i >= g.nvol) {
        for (int a = 0; a < 3; ++a) { b.lo[a] = 1; b.hi[a] = 0; }
        b.surf = false;
        return b;
    }
    // radius in standard deviations; t = 0 (or an overflow): unbounded
    const double rho = t > 0.0 ? sqrt(mi * g.mu_max / t) * (1.0 + 1e-9) : __builtin_inf();
    bool low_z = false;
    for (int a = 0; a < 3; ++a) {
        const double r = g.sd[a] > 0.0 ? rho * g.sd[a] + 1.0 : __builtin_inf();  // fixed-point units
        const double pa = (double)P[3 * i + a];
        const double flo = floor((pa - r) / (double)kFx), fhi = floor((pa + r) / (double)kFx);
        // partners of higher id lie in the node's own layer (its voxel's) and above
        if (a == 2) b.lo[a] = i / ((long long)g.nx * g.ny);
        else b.lo[a] = flo < 0.0 ? 0 : (flo > (double)(n[a] - 1) ? n[a] : (long long)flo);
        b.hi[a] = fhi > (double)(n[a] - 1) ? n[a] - 1 : (fhi < 0.0 ? -1 : (long long)fhi);
        if (a == 2) low_z = pa - r <= 0.0;
    }
    b.surf = g.surface && low_z;
    return b;
}

// Total box cells of all nodes at the thresholds 2^((h0 + s dh) / 2), s < tests (dh = 0: of
// the unbounded boxes): one thread per node, a workgroup's sums in LDS and then one atomic per
// threshold.  The radius is taken in FP32 (a box may come out a voxel wider or narrower): the
// totals only choose the threshold, the boxes themselves are k_graph_boxes'.
// (In FP64, as node_box computes it, the launch took 88 us on the 64x64x32 plume, here 46.)
constexpr int kCellTests = 64;
inline double cell_threshold(int h) { return std::ldexp((h & 1) ? 1.4142135623730951 : 1.0, (h - (h & 1)) / 2); }
__global__ __launch_bounds__(256) void k_graph_cells(Geo g, const long long *__restrict__ P, const double *__restrict__ mu,
                                                     int h0, int dh, int tests, unsigned long long *__restrict__ total) {
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    __shared__ unsigned long long sum[kCellTests];
    if (threadIdx.x < kCellTests) sum[threadIdx.x] = 0ull;
    __syncthreads();
    const bool on = i < g.nvol && mu[i] > 0.0;
    const int n[3] = {g.nx, g.ny, g.nz};
    int vox[3] = {0, 0, 0};
    float f[3] = {0.f, 0.f, 0.f}, sd[3] = {0.f, 0.f, 0.f}, lg = 0.f;
    if (on) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            vox[a] = (int)(P[3 * i + a] >> 16);
            f[a] = (float)(P[3 * i + a] & 0xffff) * 0x1p-16f;
            sd[a] = (float)(g.sd[a] * 0x1p-16);
        }
        lg = (float)log2(mu[i] * g.mu_max);
    }
    const float huge = 4096.0f;  // voxels: beyond every grid
    for (int s = 0; s < tests; ++s) {
        unsigned long long v = 0ull;
        if (on) {
            const float rho = dh ? exp2f(fminf(0.5f * (lg - 0.5f * (float)(h0 + s * dh)), 100.0f)) : 0x1p100f;
            unsigned long long e[3];
            bool low = false;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float r = sd[a] > 0.0f ? fminf(rho * sd[a] + 0x1p-16f, huge) : huge;
                const int lo = a == 2 ? vox[2] : max(0, vox[a] + (int)floorf(f[a] - r));
                e[a] = (unsigned long long)(min(n[a] - 1, vox[a] + (int)floorf(f[a] + r)) - lo + 1);
                if (a == 2) low = (float)vox[2] + f[2] <= r;
            }
            v = e[0] * e[1] * (e[2] + (g.surface && low ? 1ull : 0ull));
        }
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0) atomicAdd(&sum[s], v);
    }
    __syncthreads();
    if (threadIdx.x < tests && sum[threadIdx.x]) atomicAdd(&total[threadIdx.x], sum[threadIdx.x]);
}

// Boxes of the nodes r < n at threshold t, stored as (lo x, lo y, lo z, extent
// x, y, z, surface row, 0), and their cell counts (volume cells + surface cells);
// cells[n] = 0 closes the array for the exclusive scan.
__global__ void k_graph_boxes(Geo g, const long long *__restrict__ P, const double *__restrict__ mu, double t,
                              long long n, int *__restrict__ box, unsigned long long *__restrict__ cells) {
    const long long r = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (r > n) return;
    if (r == n) {
        cells[n] = 0;
        return;
    }
    const Box b = node_box(g, P, mu, r, t);
    long long e[3];
    for (int a = 0; a < 3; ++a) e[a] = b.hi[a] >= b.lo[a] ? b.hi[a] - b.lo[a] + 1 : 0;
    const unsigned long long nv = (unsigned long long)e[0] * e[1] * e[2];
    const unsigned long long ns = b.surf ? (unsigned long long)e[0] * e[1] : 0ull;
    int *o = box + 8 * r;
    o[0] = (int)b.lo[0]; o[1] = (int)b.lo[1]; o[2] = (int)b.lo[2];
    o[3] = (int)e[0]; o[4] = (int)e[1]; o[5] = (int)e[2];
    o[6] = b.surf ? 1 : 0; o[7] = 0;
    cells[r] = nv + ns;
}

constexpr int kEvalRounds = 8;  // a workgroup covers kEvalRounds x 256 consecutive cells

// last r in [a, b) with coff[r] <= c (coff ascending, coff[a] <= c)
__device__ __forceinline__ long long owner(const unsigned long long *__restrict__ coff, long long a, long long b,
                                           unsigned long long c) {
    while (b - a > 1) {
        const long long m = (a + b) >> 1;
        if (coff[m] <= c) a = m;
        else b = m;
    }
    return a;
}

// The cells of all boxes, flattened in node order (a node's cells in increasing
// partner id), one thread per cell: the partner j > i is evaluated and the pairs
// with k >= t (strict: k > t), k > 0 are counted per workgroup (kFill = false:
// bcount) or written in cell order at the workgroup's offset (kFill = true), so the
// list stays ordered by (i, j).  bev: the evaluated pairs per workgroup (count pass).
template <bool kFill>
__global__ __launch_bounds__(256) void k_graph_eval(Geo g, const double *__restrict__ q,
                                                    const double *__restrict__ mu, double t, int strict, long long n,
                                                    const int *__restrict__ box,
                                                    const unsigned long long *__restrict__ coff, unsigned long long T,
                                                    unsigned long long *__restrict__ bcount,
                                                    const unsigned long long *__restrict__ boff,
                                                    double *__restrict__ keys, unsigned long long *__restrict__ codes,
                                                    unsigned long long *__restrict__ bev) {
    constexpr int kCells = kEvalRounds * 256;
    __shared__ unsigned int wcnt[4];
    __shared__ unsigned long long wev[4];
    __shared__ long long range[2];
    __shared__ unsigned long long scoff[kCells];  // box starts of the workgroup's nodes, when they fit
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const unsigned long long base = (unsigned long long)blockIdx.x * kCells;
    unsigned long long run = kFill ? boff[blockIdx.x] : 0ull, ev = 0ull;
    // the nodes owning this workgroup's cells: [fb, lb]
    if (threadIdx.x == 0) {
        const long long fb = owner(coff, 0, n, base);
        const unsigned long long cl = base + kCells - 1 < T ? base + kCells - 1 : T - 1;
        range[0] = fb;
        range[1] = owner(coff, fb, n, cl);
    }
    __syncthreads();
    const long long fb = range[0], lb = range[1];
    const bool staged = lb - fb + 1 <= kCells;
    if (staged)
        for (long long x = threadIdx.x; x <= lb - fb; x += blockDim.x) scoff[x] = coff[fb + x];
    __syncthreads();
    for (int rd = 0; rd < kEvalRounds; ++rd) {
        const unsigned long long c0 = base + (unsigned long long)rd * 256 + (unsigned long long)w * 64;
        const unsigned long long c = c0 + lane;
        bool ok = false, eval = false;
        double k = 0.0;
        long long i = 0, j = 0;
        if (c < T) {
            {
                long long r;
                if (staged) {  // last x with scoff[x] <= c, in LDS
                    long long a = 0, b = lb - fb + 1;
                    while (b - a > 1) {
                        const long long m2 = (a + b) >> 1;
                        if (scoff[m2] <= c) a = m2;
                        else b = m2;
                    }
                    r = fb + a;
                } else {
                    r = owner(coff, fb, lb + 1, c);
                }
                const int *o = box + 8 * r;
                // a box has at most 1024^3 + 1024^2 cells: 32-bit index arithmetic
                const unsigned bx = (unsigned)o[3], by = (unsigned)o[4], bz = (unsigned)o[5];
                const unsigned nv = bx * by * bz;
                const unsigned lc = (unsigned)(c - (staged ? scoff[r - fb] : coff[r]));
                i = r;
                if (lc < nv) {
                    const unsigned yz = lc / bx, cx = lc - yz * bx, cz = yz / by, cy = yz - cz * by;
                    j = ((long long)o[0] + cx) + (long long)g.nx * (((long long)o[1] + cy) + (long long)g.ny * ((long long)o[2] + cz));
                } else {
                    const unsigned sl = lc - nv, sy = sl / bx, sx = sl - sy * bx;
                    j = g.nvol + ((long long)o[0] + sx) + (long long)g.nx * ((long long)o[1] + sy);
                }
                eval = j > i && SG_IN(j, g.N, 0x701);
                if (eval) {
                    k = pair_key(q, mu, i, j);
                    ok = k > 0.0 && (strict ? k > t : k >= t);
                }
            }
        }
        const unsigned long long m = __ballot(ok);
        if (!kFill) ev += __popcll(__ballot(eval));
        if (lane == 0) wcnt[w] = (unsigned int)__popcll(m);
        __syncthreads();
        unsigned long long before = 0, total = 0;
        for (int v = 0; v < 4; ++v) {
            before += v < w ? wcnt[v] : 0u;
            total += wcnt[v];
        }
        if (kFill && ok) {
            const unsigned long long at = run + before + __popcll(m & ((1ull << lane) - 1ull));
            if (SG_IN(at, boff[gridDim.x], 0x702)) {
                keys[at] = k;
                codes[at] = (unsigned long long)i << 32 | (unsigned long long)j;
            }
        }
        run += total;
        __syncthreads();  // wcnt is rewritten by the next round
    }
    if (!kFill) {
        if (lane == 0) wev[w] = ev;
        __syncthreads();
        if (threadIdx.x == 0) {
            bcount[blockIdx.x] = run;
            bev[blockIdx.x] = wev[0] + wev[1] + wev[2] + wev[3];
        }
    }
}

// Radix selection of the n largest of 64-bit keys (couplings are positive, so their bit patterns
// order like them).  sel: [0] the chosen top bits of the n-th largest key, [1] how many keys with
// those top bits still belong to the n.
constexpr int kSelBits = 11, kSelBins = 1 << kSelBits, kSelPasses = 6;  // 5 x 11 bits, then 9

__device__ __forceinline__ int sel_shift(int pass) { return pass < 5 ? 64 - kSelBits * (pass + 1) : 0; }

// key k into a pass's bins, if its top bits are the chosen ones
__device__ __forceinline__ void sel_count(unsigned *bins, unsigned long long k, int pass, unsigned long long chosen) {
    const int up = pass ? sel_shift(pass - 1) : 0;
    if (pass && k >> up != chosen >> up) return;
    atomicAdd(&bins[(unsigned)(k >> sel_shift(pass)) & (pass < 5 ? kSelBins - 1u : 511u)], 1u);
}

// Every pair i < j (i a volume node) against threshold t: the candidates (k > 0 and k >= t,
// strict: k > t) appended to keys / codes in no fixed order, counted in *count also beyond
// cap.  A workgroup takes 512 nodes i, two per thread (each j read from LDS serves both), and
// the nodes j of every gridDim.y-th span of kAllSpan, staged in LDS kAllTile at a time.  The
// division is left to the pairs that mu_i mu_j >= t d2 (1 - 1e-9) lets through: the
// products, the differences and this test, eleven FP64 operations a pair, bound the kernel.
// The span is the launch's: 4096, or less where that leaves fewer than 2048 workgroups (9000 nodes
// 1.87 -> 0.68 ms by c_min).  Candidates are few: they collect in LDS and leave with one atomic per
// 512 and workgroup (a list that overflows within a tile goes out by one atomic per wavefront and node j).
// 119,958 nodes (7.2e9 pairs): 3.3 ms, 24 T lane-operations/s of the 30 that FP64 issues; its
// build 1440 -> 5.6 ms (every pair written out, sorted and merged into a best-n list before).
// Where far more pairs reach the threshold than are asked for (equal couplings), none is written:
// kAllKeys and kAllCodes count them for a pass of the radix selection (select_hist), by the coupling
// and then, among those equal to the n-th (kn), by the complement of the code, so that the n best are
// known in the order of their ids; kAllTake lists just these.
constexpr int kAllTile = 256, kAllSpan = 4096, kAllHits = 1024, kAllFlush = 512;
enum AllMode { kAllList, kAllKeys, kAllCodes, kAllTake };
template <AllMode kMode>
__global__ __launch_bounds__(256) void k_graph_all(Geo g, const double *__restrict__ q, const double *__restrict__ mu,
                                                   double t, int strict, unsigned long long cap,
                                                   unsigned long long *__restrict__ count, double *__restrict__ keys,
                                                   unsigned long long *__restrict__ codes, int span, int pass,
                                                   const unsigned long long *__restrict__ sel, unsigned long long kn) {
#pragma clang fp contract(off)
    constexpr bool kCount = kMode == kAllKeys || kMode == kAllCodes;
    __shared__ double2 jxy[kAllTile], jzm[kAllTile];
    __shared__ double hkey[kCount ? 1 : kAllHits];
    __shared__ unsigned long long hcode[kCount ? 1 : kAllHits], hbase;
    __shared__ unsigned nhit, bins[kCount ? kSelBins : 1];
    if (kCount)
        for (int b = threadIdx.x; b < kSelBins; b += 256) bins[b] = 0u;  // published by the loop's barriers
    const unsigned long long chosen = pass || kMode == kAllTake ? sel[0] : 0ull;
    const int lane = threadIdx.x & 63;
    const long long i0 = (long long)blockIdx.x * 512;
    double xi[2], yi[2], zi[2], mi[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const long long i = i0 + 256 * h + threadIdx.x, ic = min(i, g.N - 1);
        xi[h] = q[3 * ic];
        yi[h] = q[3 * ic + 1];
        zi[h] = q[3 * ic + 2];
        mi[h] = i < g.nvol ? mu[ic] : 0.0;
    }
    const double tl = t * (1.0 - 1e-9);
    auto candidate = [&](long long i, long long j, double mm, double d2) {
        const double k = mm / d2;
        if (!(j > i && k > 0.0 && (strict ? k > t : k >= t))) return;
        const unsigned long long code = (unsigned long long)i << 32 | (unsigned long long)j;
        const unsigned long long bits = (unsigned long long)__double_as_longlong(k);
        if (kCount) {
            if (kMode == kAllCodes && bits != kn) return;
            sel_count(bins, kMode == kAllKeys ? bits : ~code, pass, chosen);
            return;
        }
        if (kMode == kAllTake && (bits < kn || (bits == kn && ~code < chosen))) return;
        const unsigned at = atomicAdd(&nhit, 1u);
        if (at < (unsigned)kAllHits) {
            hkey[at] = k;
            hcode[at] = code;
            return;
        }
        const unsigned long long m = __ballot(true);  // the lanes that overflowed
        const int lead = __builtin_ctzll(m);
        unsigned long long b = 0ull;
        if (lane == lead) b = atomicAdd(count, (unsigned long long)__popcll(m));
        b = (unsigned long long)__shfl((long long)b, lead, 64) + __popcll(m & ((1ull << lane) - 1ull));
        if (b < cap) {
            keys[b] = k;
            codes[b] = code;
        }
    };
    auto flush = [&]() {  // by the whole workgroup, between barriers; the next one publishes nhit = 0
        const unsigned n = min(nhit, (unsigned)kAllHits);
        if (threadIdx.x == 0) hbase = n ? atomicAdd(count, (unsigned long long)n) : 0ull;
        __syncthreads();
        for (unsigned h = threadIdx.x; h < n; h += 256)
            if (hbase + h < cap) {
                keys[hbase + h] = hkey[h];
                codes[hbase + h] = hcode[h];
            }
        if (threadIdx.x == 0) nhit = 0u;
    };
    if (threadIdx.x == 0) nhit = 0u;
    for (long long jb = (long long)blockIdx.y * span; jb < g.N; jb += (long long)gridDim.y * span) {
        const long long je = min(g.N, jb + span);
        for (long long j0 = max(jb, i0); j0 < je; j0 += kAllTile) {  // none below every i
            const int nj = (int)min((long long)kAllTile, je - j0);
            __syncthreads();
            if (!kCount && nhit >= (unsigned)kAllFlush) flush();
            if ((int)threadIdx.x < nj) {
                const long long j = j0 + threadIdx.x;
                jxy[threadIdx.x] = make_double2(q[3 * j], q[3 * j + 1]);
                jzm[threadIdx.x] = make_double2(q[3 * j + 2], mu[j]);
            }
            __syncthreads();
            for (int a = 0; a < nj; ++a) {
                const double2 p = jxy[a], r = jzm[a];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const double u = xi[h] - p.x, v = yi[h] - p.y, w = zi[h] - r.x;
                    const double d2 = (u * u + v * v) + w * w;
                    const double mm = mi[h] * r.y;
                    if (mm > 0.0 && mm >= tl * d2) candidate(i0 + 256 * h + threadIdx.x, j0 + a, mm, d2);
                }
            }
        }
    }
    __syncthreads();
    if (kCount) {
        for (int b = threadIdx.x; b < kSelBins; b += 256)
            if (bins[b]) atomicAdd(&count[b], (unsigned long long)bins[b]);
        return;
    }
    flush();
}

// The coupling and code of every pair i < j (i a volume node) in order, 0 where it is no candidate (k > 0
// and k >= t, strict: k > t), and the candidates counted in *count: for few nodes, whose pairs
// are soon written and need no threshold, no atomics and no sort afterwards.  A workgroup takes 256
// nodes j and kEveryRows nodes i.
// Up to 2^23 pairs: 800 nodes 3.44 -> 0.27 ms (two workgroups of k_graph_all and an atomic per hit before),
// 3000 nodes with 8 couplings each 2.11 -> 0.43 ms.
constexpr unsigned long long kEveryPairs = 1ull << 23;
constexpr int kEveryRows = 8;
__global__ __launch_bounds__(256) void k_graph_every(Geo g, const double *__restrict__ q, const double *__restrict__ mu,
                                                     double t, int strict, unsigned long long *__restrict__ count,
                                                     double *__restrict__ keys, unsigned long long *__restrict__ codes) {
#pragma clang fp contract(off)
    const long long j = blockIdx.x * 256ll + threadIdx.x, i0 = (long long)blockIdx.y * kEveryRows;
    if (i0 >= blockIdx.x * 256ll + 255) return;  // no pair of this workgroup
    __shared__ unsigned sum[4];
    unsigned n = 0u;
    for (long long i = i0; i < min(i0 + kEveryRows, g.nvol); ++i) {
        double k = 0.0;
        if (j > i && j < g.N) {
            const double c = pair_key(q, mu, i, j);
            if (c > 0.0 && (strict ? c > t : c >= t)) k = c;
            const long long at = i * (2 * g.N - i - 1) / 2 + (j - i - 1);
            keys[at] = k;
            codes[at] = (unsigned long long)i << 32 | (unsigned long long)j;
        }
        n += (unsigned)__popcll(__ballot(k > 0.0));
    }
    if ((threadIdx.x & 63) == 0) sum[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        n = sum[0] + sum[1] + sum[2] + sum[3];
        if (n) atomicAdd(count, (unsigned long long)n);
    }
}

// The couplings of M pairs spread over all of them (a fixed hash of the sample's number, so
// a build is the same every time); 0 for a pair that cannot couple.
__global__ void k_graph_sample(Geo g, const double *__restrict__ q, const double *__restrict__ mu, long long M,
                               double *__restrict__ keys) {
#pragma clang fp contract(off)
    const long long s = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (s >= M) return;
    unsigned long long h = (unsigned long long)s * 0x9e3779b97f4a7c15ull;
    h ^= h >> 32;
    h *= 0xd6e8feb86659fd93ull;
    h ^= h >> 32;
    const long long i = (long long)(((h & 0xffffffffull) * (unsigned long long)g.N) >> 32);
    const long long j = (long long)(((h >> 32) * (unsigned long long)g.N) >> 32);
    double k = 0.0;
    if (i != j && !(i >= g.nvol && j >= g.nvol)) k = i < j ? pair_key(q, mu, i, j) : pair_key(q, mu, j, i);
    keys[s] = k > 0.0 ? k : 0.0;
}

// ---- selection of the n largest keys ---------------------------------------------------

__global__ __launch_bounds__(256) void k_sel_hist(const unsigned long long *__restrict__ keys, long long n, int pass,
                                                  const unsigned long long *__restrict__ sel,
                                                  unsigned long long *__restrict__ hist) {
    __shared__ unsigned h[kSelBins];
    for (int b = threadIdx.x; b < kSelBins; b += 256) h[b] = 0u;
    __syncthreads();
    const unsigned long long chosen = pass ? sel[0] : 0ull;
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += gridDim.x * 256ll) sel_count(h, keys[i], pass, chosen);
    __syncthreads();
    for (int b = threadIdx.x; b < kSelBins; b += 256)
        if (h[b]) atomicAdd(&hist[b], (unsigned long long)h[b]);
}

// one workgroup: the bin that holds the sel[1]-th largest (the n-th in the first pass), and the
// histogram cleared
__global__ __launch_bounds__(256) void k_sel_pick(int pass, unsigned long long n, unsigned long long *__restrict__ sel,
                                                  unsigned long long *__restrict__ hist) {
    __shared__ unsigned long long above[256];
    constexpr int kPer = kSelBins / 256;
    unsigned long long c[kPer];
    unsigned long long sum = 0ull;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        c[j] = hist[threadIdx.x * kPer + j];
        hist[threadIdx.x * kPer + j] = 0ull;
        sum += c[j];
    }
    above[threadIdx.x] = sum;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {  // sums over this thread's bins and all above
        const unsigned long long t = threadIdx.x + o < 256 ? above[threadIdx.x + o] : 0ull;
        __syncthreads();
        above[threadIdx.x] += t;
        __syncthreads();
    }
    const unsigned long long want = pass ? sel[1] : n;
    unsigned long long more = above[threadIdx.x] - sum;  // in the bins above this thread's
    __syncthreads();
    if (more < want && want <= above[threadIdx.x]) {
        int j = kPer - 1;
        while (more + c[j] < want) more += c[j--];
        sel[0] = (pass ? sel[0] : 0ull) | (unsigned long long)(threadIdx.x * kPer + j) << sel_shift(pass);
        sel[1] = want - more;
    }
}

constexpr int kPickItems = 8, kPickBlock = 256 * kPickItems;

// Counts of the keys above the n-th largest (low word) and equal to it (high word) per
// workgroup; with kWrite, their compaction in list order: a larger key, and the first sel[1]
// of the equal ones.
template <bool kWrite>
__global__ __launch_bounds__(256) void k_sel_take(const unsigned long long *__restrict__ keys,
                                                  const unsigned long long *__restrict__ codes, long long n,
                                                  const unsigned long long *__restrict__ sel,
                                                  unsigned long long *__restrict__ cnt,
                                                  const unsigned long long *__restrict__ off, long long n_sel,
                                                  unsigned long long *__restrict__ out) {
    __shared__ unsigned long long lds[4];
    const long long i0 = blockIdx.x * (long long)kPickBlock + (long long)threadIdx.x * kPickItems;
    const unsigned long long kn = sel[0], ties = sel[1];
    unsigned long long mine = 0ull;
    unsigned gt = 0u, eq = 0u;
#pragma unroll
    for (int j = 0; j < kPickItems; ++j) {
        const unsigned long long k = i0 + j < n ? keys[i0 + j] : 0ull;
        const bool in = i0 + j < n;
        if (in && k > kn) gt |= 1u << j;
        if (in && k == kn) eq |= 1u << j;
    }
    mine = (unsigned long long)__popc(gt) | (unsigned long long)__popc(eq) << 32;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned long long x = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[w] = x;
    __syncthreads();
    unsigned long long before = 0ull, total = 0ull;
    for (int k = 0; k < 4; ++k) {
        if (k < w) before += lds[k];
        total += lds[k];
    }
    if (!kWrite) {
        if (threadIdx.x == 0) cnt[blockIdx.x] = total;
        return;
    }
    const unsigned long long base = off[blockIdx.x] + before + x - mine;
    unsigned long long g = base & 0xffffffffull, e = base >> 32;
    for (int j = 0; j < kPickItems; ++j) {
        const bool is_gt = gt >> j & 1u, is_eq = eq >> j & 1u;
        if (is_gt || (is_eq && e < ties)) {
            const unsigned long long at = g + (e < ties ? e : ties);
            if (SG_IN(at, n_sel, 0x705)) out[at] = codes[i0 + j];
        }
        g += is_gt;
        e += is_eq;
    }
}

// the selected pairs with their ids swapped (j << 32 | i), to be sorted by j
__global__ void k_graph_swap(long long n, const unsigned long long *__restrict__ pair,
                             unsigned long long *__restrict__ rev) {
    const long long s = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (s < n) rev[s] = pair[s] << 32 | pair[s] >> 32;
}

// ptr[l] = first e with codes[e] >> 32 >= l
__device__ __forceinline__ long long first_of(const unsigned long long *__restrict__ codes, long long n, long long l) {
    const unsigned long long key = (unsigned long long)l << 32;
    long long a = 0, b = n;  // codes[0, a) < key <= codes[b, n)
    while (a < b) {
        const long long m = (a + b) >> 1;
        if (codes[m] < key) a = m + 1;
        else b = m;
    }
    return a;
}

// Row pointers: node l's row holds its partners of lower id (its run of rev) and then
// those of higher id (its run of pair), each ascending.
__global__ void k_graph_rowptr(long long N, long long n, const unsigned long long *__restrict__ pair,
                               const unsigned long long *__restrict__ rev, long long *__restrict__ up,
                               long long *__restrict__ down, long long *__restrict__ ptr) {
    const long long l = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (l > N) return;
    const long long u = first_of(pair, n, l), d = first_of(rev, n, l);
    up[l] = u;
    down[l] = d;
    ptr[l] = u + d;
}

__global__ void k_graph_heads(long long n, long long N, const unsigned long long *__restrict__ pair,
                              const unsigned long long *__restrict__ rev, const long long *__restrict__ up,
                              const long long *__restrict__ down, int *__restrict__ head) {
    const long long s = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (s >= n) return;
    const unsigned long long f = pair[s], r = rev[s];
    const long long i = (long long)(f >> 32), j = (long long)(r >> 32);
    if (SG_IN(i, N, 0x706) && SG_IN(s + down[i + 1], 2 * n, 0x707)) head[s + down[i + 1]] = (int)(f & 0xffffffffull);
    if (SG_IN(j, N, 0x708) && SG_IN(s + up[j], 2 * n, 0x709)) head[s + up[j]] = (int)(r & 0xffffffffull);
}

// ---- scans, sums and sorts of the builder -----------------------------------------------

constexpr int kScanItems = 8;                 // consecutive items per thread
constexpr int kScanBlock = 256 * kScanItems;  // items per workgroup

// exclusive prefix of v over the workgroup's 256 threads; total = the workgroup's sum
template <class T>
__device__ __forceinline__ T block_exclusive(T v, T *lds, T &total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    T x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[w] = x;
    __syncthreads();
    T before = 0;
    total = 0;
    for (int k = 0; k < 4; ++k) {
        if (k < w) before += lds[k];
        total += lds[k];
    }
    return before + x - v;
}

// pass 1: each workgroup's items scanned (exclusive, plus init), its total to tsum
template <class T>
__global__ __launch_bounds__(256) void k_scan_local(const T *__restrict__ in, T *__restrict__ out, long long n, T init,
                                                    T *__restrict__ tsum) {
    __shared__ T lds[4];
    const long long i0 = (long long)blockIdx.x * kScanBlock + (long long)threadIdx.x * kScanItems;
    T v[kScanItems];
    T sum = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        v[j] = i0 + j < n ? in[i0 + j] : (T)0;
        sum += v[j];
    }
    T total;
    T ex = block_exclusive(sum, lds, total) + init;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        if (i0 + j < n) out[i0 + j] = ex;
        ex += v[j];
    }
    if (tsum && threadIdx.x == 0) tsum[blockIdx.x] = total;
}

// pass 3: the workgroups' offsets added
template <class T>
__global__ void k_scan_add(T *__restrict__ out, long long n, const T *__restrict__ off) {
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i < n) out[i] += off[i / kScanBlock];
}

// sum of n values, one atomic per workgroup (integer: the order does not matter)
__global__ __launch_bounds__(256) void k_sum_u64(const unsigned long long *__restrict__ in, long long n,
                                                 unsigned long long *__restrict__ out) {
    __shared__ unsigned long long lds[4];
    unsigned long long v = 0;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        v += in[i];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(out, lds[0] + lds[1] + lds[2] + lds[3]);
}

constexpr int kRsItems = 16;             // keys per lane in a tile
constexpr int kRsTile = 64 * kRsItems;  // keys per tile (one wavefront; staged in LDS by the scatter)

// digit counts of each tile, digit-major: hist[digit * ntiles + tile]
__global__ __launch_bounds__(256) void k_rs_hist(const unsigned long long *__restrict__ keys, long long n, int bit,
                                                 long long ntiles, unsigned *__restrict__ hist) {
    __shared__ unsigned cnt[4][256];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long tile = (long long)blockIdx.x * 4 + w;
    for (int d = lane; d < 256; d += 64) cnt[w][d] = 0u;
    __syncthreads();
    if (tile < ntiles) {
        const long long base = tile * kRsTile;
        for (int r = 0; r < kRsItems; ++r) {
            const long long i = base + (long long)r * 64 + lane;
            if (i < n) atomicAdd(&cnt[w][(unsigned)(keys[i] >> bit) & 255u], 1u);
        }
    }
    __syncthreads();
    if (tile < ntiles)
        for (int d = lane; d < 256; d += 64) hist[(long long)d * ntiles + tile] = cnt[w][d];
}

// Stable scatter by one digit: tile t's keys with digit d go to off[d * ntiles + t] onward,
// in their order.  The tile is first sorted by digit in the wavefront's LDS (a stable
// counting sort: local digit starts from the tile's counts, then round r of the tile, keys
// base + 64 r + lane, ranked among the round's keys of its digit by the ballots of the
// digit's eight bits, after the digit's running count), then written out in that order, so
// the lanes holding one digit store to consecutive addresses.  Same order as placing every
// key straight at its global position.
__global__ __launch_bounds__(256) void k_rs_scatter(const unsigned long long *__restrict__ kin,
                                                    const unsigned long long *__restrict__ vin,
                                                    unsigned long long *__restrict__ kout,
                                                    unsigned long long *__restrict__ vout, long long n, int bit,
                                                    long long ntiles, const unsigned *__restrict__ off,
                                                    const unsigned *__restrict__ hist) {
    __shared__ unsigned gbase[4][256], lbase[4][256], run[4][256];
    __shared__ unsigned long long sk[4][kRsTile], sv[4][kRsTile];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long tile = (long long)blockIdx.x * 4 + w;
    if (tile >= ntiles) return;  // no barrier below: each wavefront works on its own LDS rows
    // the tile's digit counts, four consecutive digits per lane, and their exclusive scan
    unsigned c[4], sum = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int d = 4 * lane + j;
        c[j] = hist[(long long)d * ntiles + tile];
        gbase[w][d] = off[(long long)d * ntiles + tile];
        sum += c[j];
    }
    unsigned incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    unsigned start = incl - sum;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int d = 4 * lane + j;
        lbase[w][d] = start;
        run[w][d] = start;
        start += c[j];
    }
    __builtin_amdgcn_wave_barrier();
    const long long base = tile * kRsTile;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int r = 0; r < kRsItems; ++r) {
        const long long i = base + (long long)r * 64 + lane;
        const bool ok = i < n;
        const unsigned long long k = ok ? kin[i] : 0ull;
        const unsigned dg = (unsigned)(k >> bit) & 255u;
        unsigned long long peers = __ballot(ok);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const unsigned long long m = __ballot(ok && ((dg >> b) & 1u));
            peers &= ((dg >> b) & 1u) ? m : ~m;
        }
        const unsigned before = (unsigned)__popcll(peers & below);
        const unsigned p = ok ? run[w][dg] + before : 0u;
        __builtin_amdgcn_wave_barrier();
        if (ok && before == 0u) run[w][dg] = p + (unsigned)__popcll(peers);  // the digit's first lane
        if (ok && SG_IN(p, kRsTile, 0x703)) {
            sk[w][p] = k;
            if (vin) sv[w][p] = vin[i];
        }
        __builtin_amdgcn_wave_barrier();
    }
    // write-out in digit order: local position j holds the (j - lbase[digit])-th key of its
    // digit in this tile
    const int nk = (int)min((long long)kRsTile, n - base);
    for (int j = lane; j < nk; j += 64) {
        const unsigned long long k = sk[w][j];
        const unsigned dg = (unsigned)(k >> bit) & 255u;
        const unsigned g = gbase[w][dg] + ((unsigned)j - lbase[w][dg]);
        if (SG_IN(g, n, 0x704)) {
            kout[g] = k;
            if (vin) vout[g] = sv[w][j];
        }
    }
}

// The same of few nodes and voxels on the host: the device's answer is a round trip (8x8x8 nodes above a
// c_min: 221 -> 183 us).
constexpr long long kHostMoments = 4096;
void host_moments(const sg_graph_desc *d, const Geo &g, Moments &m) {
    m = Moments{};
    m.bad_node = ~0ull;
    for (long long v = 0; v < g.nvox; ++v) {
        unsigned bits;
        std::memcpy(&bits, d->mu_s + v, sizeof(bits));
        if (d->mu_s[v] >= 0.0f && std::isfinite(d->mu_s[v])) m.mu_max = std::max(m.mu_max, bits & 0x7fffffffu);
        else m.bad_mu = 1u;
    }
    const int *pos = g.general ? d->node_pos_fx : d->vol_pos_fx;
    for (long long l = 0; l < g.N; ++l) {
        long long p[3] = {0, 0, 0};
        if (l < g.nvol) {
            const long long c[3] = {l % g.nx, (l / g.nx) % g.ny, l / ((long long)g.nx * g.ny)};
            const long long w[3] = {g.nx * kFx, g.ny * kFx, g.nz * kFx};
            bool in = true;
            for (int a = 0; a < 3; ++a) {
                p[a] = pos[3 * l + a];
                const long long lo = g.general ? (a < 2 ? -1 : 0) : c[a] * kFx;
                in = in && p[a] > lo && p[a] < (g.general ? w[a] : lo + kFx);
            }
            if (!in) m.bad_node = std::min(m.bad_node, (unsigned long long)l);
        } else {
            const long long c = l - g.nvol;
            p[0] = (c % g.nx) * kFx + kFx / 2;
            p[1] = (c / g.nx) * kFx + kFx / 2;
            if (!(d->surf_albedo[c] >= 0.0f && d->surf_albedo[c] <= 1.0f)) m.bad_albedo = 1u;
        }
        for (int a = 0; a < 3; ++a) {
            const unsigned long long sq = (unsigned long long)(p[a] * p[a]);
            m.s1[a] += (unsigned long long)p[a];
            m.lo[a] += sq & 0xffffffffull;
            m.hi[a] += sq >> 32;
        }
    }
}

unsigned blocks_for(long long n, int threads) { return (unsigned)std::max<long long>(1, (n + threads - 1) / threads); }

// ---- host driver ---------------------------------------------------------------------

struct Builder {
    Ctx *ctx;
    hipStream_t st;
    Geo g;
    Dev dev;  // everything the build allocates, released when it ends
    long long *P = nullptr;
    double *q = nullptr, *mu = nullptr;
    unsigned long long *scal = nullptr;  // [0 .. kCellTests) cell totals, counters; then the selection's state
    unsigned long long *hist = nullptr;  // the selection's histogram (zero between passes)
    // build statistics: candidate passes, summed kernel times (HIP event pairs)
    int passes = 0;
    unsigned long long evals = 0;  // pairs evaluated by the candidate passes
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_pairs, ev_sort;
    Builder(Ctx *c, hipStream_t s) : ctx(c), st(s), dev(c, s) {}
    ~Builder() {
        for (auto &e : ev_pairs) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
        for (auto &e : ev_sort) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
    }
    // an event pair recording around whatever the caller enqueues next (its index; -1: none)
    int mark(std::vector<std::pair<hipEvent_t, hipEvent_t>> &v) {
        hipEvent_t a = nullptr, b = nullptr;
        if (hipEventCreate(&a) != hipSuccess) return -1;
        if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return -1; }
        v.push_back({a, b});
        (void)hipEventRecord(a, st);
        return (int)v.size() - 1;
    }
    void end(std::vector<std::pair<hipEvent_t, hipEvent_t>> &v, int e) {
        if (e >= 0) (void)hipEventRecord(v[e].second, st);
    }
    static double total_ms(const std::vector<std::pair<hipEvent_t, hipEvent_t>> &v) {
        double t = 0.0;
        for (auto &e : v) {
            float ms = 0.0f;
            if (hipEventElapsedTime(&ms, e.first, e.second) == hipSuccess) t += ms;
        }
        return t;
    }

    // box cells at the thresholds 2^((h0 + s dh) / 2), s < tests (dh = 0: of the unbounded boxes)
    sg_status cells(int h0, int dh, int tests, unsigned long long *out) {
        GHIP(hipMemsetAsync(scal, 0, tests * sizeof(unsigned long long), st));
        hipLaunchKernelGGL(k_graph_cells, dim3(blocks_for(g.N, 256)), dim3(256), 0, st, g, P, mu, h0, dh, tests, scal);
        GHIP(hipGetLastError());
        GHIP(hipMemcpyAsync(out, scal, tests * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
        GHIP(hipStreamSynchronize(st));
        return SG_OK;
    }

    // candidates of all nodes' boxes at threshold t, ordered by (i, j); only their number when
    // there are fewer than `least`
    sg_status pairs(double t, int strict, unsigned long long least, double *&keys, unsigned long long *&codes, unsigned long long &have) {
        const long long n = g.N;
        have = 0;
        int *box = nullptr;
        unsigned long long *cells = nullptr, *coff = nullptr;
        GTRY(dev.get(&box, 8 * n));
        GTRY(dev.get(&cells, n + 1));
        GTRY(dev.get(&coff, n + 1));
        hipLaunchKernelGGL(k_graph_boxes, dim3(blocks_for(n + 1, 256)), dim3(256), 0, st, g, P, mu, t, n, box, cells);
        GHIP(hipGetLastError());
        GTRY(scan<unsigned long long>(cells, coff, n + 1, 0ull));
        unsigned long long T = 0;
        GHIP(hipMemcpyAsync(&T, coff + n, sizeof(T), hipMemcpyDeviceToHost, st));
        GHIP(hipStreamSynchronize(st));
        if (T == 0) return SG_OK;
        const unsigned long long per = (unsigned long long)kEvalRounds * 256;
        const unsigned long long nb = (T + per - 1) / per;
        if (nb >= (1ull << 31)) return gfail(SG_E_NOMEM, "coupling boxes too large");
        unsigned long long *bcount = nullptr, *boff = nullptr, *bev = nullptr;
        GTRY(dev.get(&bcount, nb + 1));
        GTRY(dev.get(&boff, nb + 1));
        GTRY(dev.get(&bev, nb));
        GHIP(hipMemsetAsync(bcount + nb, 0, sizeof(unsigned long long), st));
        GHIP(hipMemsetAsync(scal, 0, sizeof(unsigned long long), st));
        ++passes;
        const int e0 = mark(ev_pairs);
        hipLaunchKernelGGL((k_graph_eval<false>), dim3((unsigned)nb), dim3(256), 0, st, g, q, mu, t, strict, n,
                           box, coff, T, bcount, nullptr, nullptr, nullptr, bev);
        end(ev_pairs, e0);
        GHIP(hipGetLastError());
        // boff = exclusive sum of the workgroup counts; boff[nb] = their total
        GTRY(scan<unsigned long long>(bcount, boff, (long long)nb + 1, 0ull));
        hipLaunchKernelGGL(k_sum_u64, dim3((unsigned)std::min<unsigned long long>((nb + 255) / 256, 1024)), dim3(256), 0,
                           st, bev, (long long)nb, scal);
        GHIP(hipGetLastError());
        unsigned long long total = 0, ev = 0;
        GHIP(hipMemcpyAsync(&total, boff + nb, sizeof(total), hipMemcpyDeviceToHost, st));
        GHIP(hipMemcpyAsync(&ev, scal, sizeof(ev), hipMemcpyDeviceToHost, st));
        GHIP(hipStreamSynchronize(st));
        evals += ev;
        if (total >= (1ull << 31)) return gfail(SG_E_NOMEM, "more than 2^31 coupling candidates");
        have = total;
        if (total && total >= least) {
            GTRY(dev.get(&keys, total));
            GTRY(dev.get(&codes, total));
            const int e1 = mark(ev_pairs);
            hipLaunchKernelGGL((k_graph_eval<true>), dim3((unsigned)nb), dim3(256), 0, st, g, q, mu, t, strict, n,
                               box, coff, T, nullptr, boff, keys, codes, nullptr);
            end(ev_pairs, e1);
            GHIP(hipGetLastError());
        }
        return SG_OK;
    }

    // candidates among all pairs at threshold t, ordered by (i, j); room for `expect` of them (more:
    // a second pass, or, when the `best` strongest of them are asked for and the list would be
    // long, these alone).  reached: the pairs at the threshold.
    sg_status all_pairs(double t, int strict, unsigned long long expect, unsigned long long best, double *&keys,
                        unsigned long long *&codes, unsigned long long &have, unsigned long long &reached) {
        unsigned long long cap = expect;
        while (true) {
            if (cap >= (1ull << 31)) return gfail(SG_E_NOMEM, "more than 2^31 coupling candidates");
            const size_t level = dev.blocks.size();
            GTRY(dev.get(&keys, cap));
            GTRY(dev.get(&codes, cap));
            GTRY(all_pass<kAllList>(t, strict, cap, scal, keys, codes, 0, 0ull));
            GHIP(hipMemcpyAsync(&have, scal, sizeof(have), hipMemcpyDeviceToHost, st));
            GHIP(hipStreamSynchronize(st));
            reached = have;
            if (have <= cap) break;
            GTRY(dev.drop(level));
            if (best && have > std::max(4 * cap, kMostListed)) {
                GTRY(best_pairs(t, strict, best, keys, codes));
                have = best;
                break;
            }
            cap = have;
        }
        const int e1 = mark(ev_sort);
        GTRY(sort_codes(codes, reinterpret_cast<unsigned long long *>(keys), (long long)have, true));
        end(ev_sort, e1);
        return SG_OK;
    }

    // one pass over all pairs (k_graph_all); out: the counter (cleared first) or the histogram
    template <AllMode kMode>
    sg_status all_pass(double t, int strict, unsigned long long cap, unsigned long long *out, double *keys,
                       unsigned long long *codes, int pass, unsigned long long kn) {
        const long long gx = (g.nvol + 511) / 512;
        const long long span = std::min<long long>(kAllSpan, (gx * g.N / 2048 / kAllTile + 1) * kAllTile);
        const dim3 grid((unsigned)gx, (unsigned)std::min<long long>((g.N + span - 1) / span, 65535));
        if (out == scal) GHIP(hipMemsetAsync(scal, 0, sizeof(unsigned long long), st));
        ++passes;
        const int e0 = mark(ev_pairs);
        hipLaunchKernelGGL(k_graph_all<kMode>, grid, dim3(256), 0, st, g, q, mu, t, strict, cap, out, keys, codes, (int)span,
                           pass, scal + kCellTests, kn);
        end(ev_pairs, e0);
        GHIP(hipGetLastError());
        evals += all();
        return SG_OK;
    }
    // the pairs i < j of a volume node i and any node j
    unsigned long long all() const { return (unsigned long long)g.nvol * (unsigned long long)(2 * g.N - g.nvol - 1) / 2; }

    // every pair in order (k_graph_every); have: the candidates among them
    sg_status every_pair(double t, int strict, double *&keys, unsigned long long *&codes, unsigned long long &have) {
        GTRY(dev.get(&keys, all()));
        GTRY(dev.get(&codes, all()));
        GHIP(hipMemsetAsync(scal, 0, sizeof(unsigned long long), st));
        ++passes;
        const int e0 = mark(ev_pairs);
        hipLaunchKernelGGL(k_graph_every, dim3(blocks_for(g.N, 256), (unsigned)((g.nvol + kEveryRows - 1) / kEveryRows)),
                           dim3(256), 0, st, g, q, mu, t, strict, scal, keys, codes);
        end(ev_pairs, e0);
        GHIP(hipGetLastError());
        GHIP(hipMemcpyAsync(&have, scal, sizeof(have), hipMemcpyDeviceToHost, st));
        GHIP(hipStreamSynchronize(st));
        evals += all();
        return SG_OK;
    }

    // the `best` strongest of more pairs than that at threshold t, by selection over all pairs; in no order
    sg_status best_pairs(double t, int strict, unsigned long long best, double *&keys, unsigned long long *&codes) {
        unsigned long long sel[2];
        for (int p = 0; p < kSelPasses; ++p) {
            GTRY(all_pass<kAllKeys>(t, strict, 0, hist, nullptr, nullptr, p, 0ull));
            hipLaunchKernelGGL(k_sel_pick, dim3(1), dim3(256), 0, st, p, best, scal + kCellTests, hist);
        }
        GHIP(hipMemcpyAsync(sel, scal + kCellTests, sizeof(sel), hipMemcpyDeviceToHost, st));
        GHIP(hipStreamSynchronize(st));
        for (int p = 0; p < kSelPasses; ++p) {
            GTRY(all_pass<kAllCodes>(t, strict, 0, hist, nullptr, nullptr, p, sel[0]));
            hipLaunchKernelGGL(k_sel_pick, dim3(1), dim3(256), 0, st, p, sel[1], scal + kCellTests, hist);
        }
        GTRY(dev.get(&keys, best));
        GTRY(dev.get(&codes, best));
        return all_pass<kAllTake>(t, strict, best, scal, keys, codes, 0, sel[0]);
    }

    // a threshold that about `want` pairs reach, from a sample (0: every pair)
    sg_status sampled_threshold(double want, double &t) {
        t = 0.0;
        const double pairs = 0.5 * (double)g.N * (double)(g.N - 1);
        if (pairs <= (double)(1 << 22)) return SG_OK;
        const long long M = want / pairs * (double)(1 << 21) < 1024.0 ? 1ll << 24 : 1ll << 21;
        const double m = std::max(64.0, std::ceil(want / pairs * (double)M));
        if (m >= (double)M) return SG_OK;
        const size_t level = dev.blocks.size();
        double *keys = nullptr;
        GTRY(dev.get(&keys, M));
        hipLaunchKernelGGL(k_graph_sample, dim3(blocks_for(M, 256)), dim3(256), 0, st, g, q, mu, M, keys);
        GHIP(hipGetLastError());
        GTRY(select(reinterpret_cast<unsigned long long *>(keys), M, (unsigned long long)m));
        unsigned long long bits = 0;
        GHIP(hipMemcpyAsync(&bits, scal + kCellTests, sizeof(bits), hipMemcpyDeviceToHost, st));
        GHIP(hipStreamSynchronize(st));
        std::memcpy(&t, &bits, sizeof(t));
        if (std::isinf(t)) t = std::numeric_limits<double>::max();  // coincident nodes
        return dev.drop(level);
    }

    // the n-th largest of have keys (n <= have) and the number of keys equal to it among the n
    // largest, to scal[kCellTests] and scal[kCellTests + 1]
    sg_status select(const unsigned long long *keys, long long have, unsigned long long n) {
        const unsigned nb = (unsigned)std::min<long long>((have + 2047) / 2048, 1024);
        for (int p = 0; p < kSelPasses; ++p) {
            hipLaunchKernelGGL(k_sel_hist, dim3(nb), dim3(256), 0, st, keys, have, p, scal + kCellTests, hist);
            hipLaunchKernelGGL(k_sel_pick, dim3(1), dim3(256), 0, st, p, n, scal + kCellTests, hist);
        }
        GHIP(hipGetLastError());
        return SG_OK;
    }

    // the codes of the n largest keys in list order (equal keys: the first ones)
    sg_status take(const double *keys, const unsigned long long *codes, long long have, long long n,
                   unsigned long long *&out) {
        const auto *k = reinterpret_cast<const unsigned long long *>(keys);
        GTRY(select(k, have, (unsigned long long)n));
        const long long nb = (have + kPickBlock - 1) / kPickBlock;
        unsigned long long *cnt = nullptr, *off = nullptr;
        GTRY(dev.get(&cnt, nb));
        GTRY(dev.get(&off, nb));
        GTRY(dev.get(&out, n));
        hipLaunchKernelGGL((k_sel_take<false>), dim3((unsigned)nb), dim3(256), 0, st, k, codes, have, scal + kCellTests,
                           cnt, nullptr, n, nullptr);
        GTRY(scan<unsigned long long>(cnt, off, nb, 0ull));
        hipLaunchKernelGGL((k_sel_take<true>), dim3((unsigned)nb), dim3(256), 0, st, k, codes, have, scal + kCellTests,
                           nullptr, off, n, out);
        GHIP(hipGetLastError());
        return SG_OK;
    }

    // out[i] = init + in[0] + ... + in[i - 1] for i < n (in and out distinct)
    template <class T>
    sg_status scan(const T *in, T *out, long long n, T init) {
        if (n <= 0) return SG_OK;
        const long long nb = (n + kScanBlock - 1) / kScanBlock;
        if (nb == 1) {
            hipLaunchKernelGGL((k_scan_local<T>), dim3(1), dim3(256), 0, st, in, out, n, init, (T *)nullptr);
            GHIP(hipGetLastError());
            return SG_OK;
        }
        T *tsum = nullptr, *toff = nullptr;
        GTRY(dev.get(&tsum, nb));
        GTRY(dev.get(&toff, nb));
        return scan_with(in, out, n, init, tsum, toff);
    }
    template <class T>
    sg_status scan_with(const T *in, T *out, long long n, T init, T *tsum, T *toff) {
        const long long nb = (n + kScanBlock - 1) / kScanBlock;
        hipLaunchKernelGGL((k_scan_local<T>), dim3((unsigned)nb), dim3(256), 0, st, in, out, n, (T)0, tsum);
        GHIP(hipGetLastError());
        GTRY(scan<T>(tsum, toff, nb, init));
        hipLaunchKernelGGL((k_scan_add<T>), dim3(blocks_for(n, 256)), dim3(256), 0, st, out, n, (const T *)toff);
        GHIP(hipGetLastError());
        return SG_OK;
    }

    // stable ascending sort of n codes (a << 32 | b, a and b node ids) by a, or by (a, b) with
    // both, with their values when vals is given, in place: passes of 8-bit digits of the bits
    // that ids use, through a second buffer
    sg_status sort_codes(unsigned long long *&keys, unsigned long long *vals, long long n, bool both) {
        if (n < 2) return SG_OK;
        int bits = 1;
        while (bits < 32 && (1ll << bits) < g.N) ++bits;
        std::vector<int> at;
        for (int h = both ? 0 : 1; h < 2; ++h)
            for (int b = 0; b < bits; b += 8) at.push_back(32 * h + b);
        const long long ntiles = (n + kRsTile - 1) / kRsTile, nh = 256 * ntiles;
        const long long sb = (nh + kScanBlock - 1) / kScanBlock;
        unsigned long long *k2 = nullptr, *v2 = nullptr;
        unsigned *hs = nullptr, *off = nullptr, *tsum = nullptr, *toff = nullptr;
        GTRY(dev.get(&k2, n));
        if (vals) GTRY(dev.get(&v2, n));
        GTRY(dev.get(&hs, nh));
        GTRY(dev.get(&off, nh));
        GTRY(dev.get(&tsum, sb));
        GTRY(dev.get(&toff, sb));
        const unsigned nblk = (unsigned)((ntiles + 3) / 4);
        unsigned long long *ka = keys, *va = vals, *kb = k2, *vb = v2;
        for (int bit : at) {
            hipLaunchKernelGGL(k_rs_hist, dim3(nblk), dim3(256), 0, st, ka, n, bit, ntiles, hs);
            GHIP(hipGetLastError());
            if (sb == 1) GTRY(scan<unsigned>(hs, off, nh, 0u));
            else GTRY(scan_with<unsigned>(hs, off, nh, 0u, tsum, toff));
            hipLaunchKernelGGL(k_rs_scatter, dim3(nblk), dim3(256), 0, st, ka, va, kb, vb, n, bit, ntiles,
                               (const unsigned *)off, (const unsigned *)hs);
            GHIP(hipGetLastError());
            std::swap(ka, kb);
            std::swap(va, vb);
        }
        if (ka != keys) {  // an odd number of passes: the result is in the second buffer
            if (vals) GHIP(hipMemcpyAsync(vals, va, sizeof(unsigned long long) * n, hipMemcpyDeviceToDevice, st));
            keys = ka;
        }
        return SG_OK;
    }
};

}  // namespace

sg_status graph_build(Ctx *ctx, const sg_graph_desc *d, hipStream_t st, int64_t *adj_ptr, int32_t *adj_idx,
                      int64_t cap, int64_t *n_edges, sg_graph_info *info) {
    const auto t_start = std::chrono::steady_clock::now();
    if (!d) return gfail(SG_E_INVALID, "desc is NULL");
    if (d->abi_version != SG_ABI_VERSION) return gfail(SG_E_ABI, "graph desc abi_version mismatch");
    if (!n_edges) return gfail(SG_E_INVALID, "n_edges is NULL");
    if (d->nx < 1 || d->ny < 1 || d->nz < 1 || d->nx > 1024 || d->ny > 1024 || d->nz > 1024)
        return gfail(SG_E_INVALID, "grid dimensions must be in 1..1024");
    const bool general = d->n_nodes > 0;
    if (d->n_nodes < 0) return gfail(SG_E_INVALID, "n_nodes must be >= 0");
    if (!d->mu_s || !(general ? d->node_pos_fx : d->vol_pos_fx) || (d->surface_nodes && !d->surf_albedo))
        return gfail(SG_E_INVALID, "a required array is NULL");
    if (d->n_pairs < 0) return gfail(SG_E_INVALID, "n_pairs must be >= 0");
    if (d->n_pairs == 0 && !(d->c_min >= 0.0 && std::isfinite(d->c_min)))
        return gfail(SG_E_INVALID, "c_min must be finite and >= 0");
    const long long nvox = (long long)d->nx * d->ny * d->nz;
    const long long nvol = general ? (long long)d->n_nodes : nvox;
    const long long N = nvol + (d->surface_nodes ? (long long)d->nx * d->ny : 0);
    if (N >= (1LL << 31)) return gfail(SG_E_INVALID, "too many nodes");
    Builder B(ctx, st);
    Geo &g = B.g;
    g.nx = d->nx;
    g.ny = d->ny;
    g.nz = d->nz;
    g.surface = d->surface_nodes ? 1 : 0;
    g.general = general ? 1 : 0;
    g.nvox = nvox;
    g.nvol = nvol;
    g.N = N;

    // the inputs, their checks and exact integer moments, then the node arrays
    int *pos = nullptr;
    float *mus = nullptr, *alb = nullptr;
    Moments *mom = nullptr;
    GTRY(B.dev.get(&pos, 3 * nvol));
    GTRY(B.dev.get(&mus, nvox));
    GTRY(B.dev.get(&alb, (long long)d->nx * d->ny));
    GTRY(B.dev.get(&mom, 1));
    GTRY(B.dev.get(&B.P, 3 * N));
    GTRY(B.dev.get(&B.q, 3 * N));
    GTRY(B.dev.get(&B.mu, N));
    GTRY(B.dev.get(&B.scal, kCellTests + 2));
    GTRY(B.dev.get(&B.hist, kSelBins));
    Moments m;
    const bool few = std::max(N, nvox) <= kHostMoments;
    if (few) host_moments(d, g, m);
    GHIP(hipMemsetAsync(B.hist, 0, sizeof(unsigned long long) * kSelBins, st));
    GHIP(hipMemcpyAsync(pos, general ? d->node_pos_fx : d->vol_pos_fx, sizeof(int) * 3 * nvol, hipMemcpyHostToDevice,
                        st));
    GHIP(hipMemcpyAsync(mus, d->mu_s, sizeof(float) * nvox, hipMemcpyHostToDevice, st));
    if (d->surface_nodes)
        GHIP(hipMemcpyAsync(alb, d->surf_albedo, sizeof(float) * d->nx * d->ny, hipMemcpyHostToDevice, st));
    if (!few) {
        GHIP(hipMemsetAsync(mom, 0, sizeof(Moments), st));
        GHIP(hipMemsetAsync(&mom->bad_node, 0xff, sizeof(mom->bad_node), st));
        hipLaunchKernelGGL(k_graph_moments, dim3(std::min(256u, blocks_for(std::max(N, nvox), 256))), dim3(256), 0, st, g,
                           pos, mus, alb, mom);
        GHIP(hipGetLastError());
        GHIP(hipMemcpyAsync(&m, mom, sizeof(m), hipMemcpyDeviceToHost, st));
        GHIP(hipStreamSynchronize(st));
    }
    if (m.bad_mu) return gfail(SG_E_INVALID, "mu_s must be finite and >= 0");
    if (m.bad_albedo) return gfail(SG_E_INVALID, "surf_albedo must be in [0, 1]");
    if (m.bad_node != ~0ull)
        return gfail(SG_E_INVALID, std::string(general ? "node position outside the box"
                                                       : "node position not strictly inside its voxel") +
                                       " (node " + std::to_string(m.bad_node) + ")");
    float mu_max;
    std::memcpy(&mu_max, &m.mu_max, sizeof(mu_max));
    g.mu_max = (double)mu_max;
    for (int a = 0; a < 3; ++a) {
        const __int128 s1 = (__int128)m.s1[a], s2 = ((__int128)m.hi[a] << 32) + (__int128)m.lo[a];
        g.mean[a] = (double)s1 / (double)N;
        const double var = (double)((__int128)N * s2 - s1 * s1) / ((double)N * (double)N);
        g.sd[a] = var > 0.0 ? std::sqrt(var) : 0.0;
    }
    hipLaunchKernelGGL(k_graph_nodes, dim3(blocks_for(N, 256)), dim3(256), 0, st, g, pos, mus, alb, B.P, B.q, B.mu);
    GHIP(hipGetLastError());

    // candidates and selection
    double *keys = nullptr;
    unsigned long long *codes = nullptr, have = 0, n_sel = 0, ranked = 0;
    unsigned long long listed = 0;  // keys and codes; `have` of them are candidates
    double t_used = 0.0;
    int streamed = 0;
    const unsigned long long n_want = (unsigned long long)d->n_pairs;
    if (d->n_pairs == 0) {
        t_used = d->c_min * d->c_min;
        if (general && B.all() <= kEveryPairs) {
            GTRY(B.every_pair(t_used, 1, keys, codes, have));
            listed = B.all();
        } else {
            if (general) GTRY(B.all_pairs(t_used, 1, 1ull << 20, 0ull, keys, codes, have, ranked));
            else GTRY(B.pairs(t_used, 1, 0ull, keys, codes, have));
            listed = have;
        }
        n_sel = ranked = have;
    } else {
        // the lowest threshold whose boxes fit the cell budget, to a factor of sqrt 2 (any
        // threshold within the budget gives the same selection, a tighter one only fewer
        // candidates): 64 thresholds a launch, over all exponents and then over one of the
        // 32-binade steps between; a larger budget when it leaves fewer than n candidates
        double t_fit = 0.0;
        bool enough = false;
        if (!general) {
            const std::vector<unsigned long long> budgets = cell_budgets(n_want);
            unsigned long long all_cells = 0, coarse[kCellTests], fine[kCellTests];
            GTRY(B.cells(0, 0, 1, &all_cells));
            const int h_lo = -2016, h_step = 64;  // thresholds 2^-1008, 2^-976, ..., 2^1008
            bool have_coarse = false;
            for (size_t k = 0; k < budgets.size(); ++k) {
                const unsigned long long bk = budgets[k];
                t_fit = 0.0;
                if (all_cells > bk) {
                    if (!have_coarse) GTRY(B.cells(h_lo, h_step, kCellTests, coarse));
                    have_coarse = true;
                    const unsigned long long least = coarse[kCellTests - 1];
                    if (least > bk) {
                        if (k + 1 < budgets.size() && least <= kMostCells) continue;
                        return gfail(SG_E_NOMEM, "coupling candidates exceed the cell budget");
                    }
                    int s = kCellTests - 1;
                    while (s > 0 && coarse[s - 1] <= bk) --s;
                    int h = h_lo + s * h_step;
                    if (s > 0) {  // between the last threshold above the budget and this one
                        GTRY(B.cells(h - h_step + 1, 1, kCellTests, fine));
                        int f = kCellTests - 1;
                        while (f > 0 && fine[f - 1] <= bk) --f;
                        h = h - h_step + 1 + f;
                    }
                    t_fit = cell_threshold(h);
                }
                const size_t level = B.dev.blocks.size();
                GTRY(B.pairs(t_fit, 0, t_fit > 0.0 ? n_want : 0ull, keys, codes, have));
                enough = have >= n_want || t_fit == 0.0;
                if (enough) break;
                GTRY(B.dev.drop(level));
            }
        }
        t_used = t_fit;
        ranked = listed = have;
        if (!enough && B.all() <= kEveryPairs) {
            streamed = 1;
            t_used = 0.0;
            B.evals = 0;
            GTRY(B.every_pair(0.0, 0, keys, codes, have));
            ranked = have;
            listed = B.all();
        } else if (!enough) {
            // every pair against a threshold from a sample, lower ones while too few reach it
            streamed = 1;
            t_used = 0.0;
            B.evals = 0;
            for (double more = 1.25;; more *= 4.0) {
                const double want = more * (double)n_want;
                double t = 0.0;
                GTRY(B.sampled_threshold(want, t));
                const double room = std::min({1.25 * want + 65536.0, (double)B.all(), 2147483647.0});
                const size_t level = B.dev.blocks.size();
                GTRY(B.all_pairs(t, 0, (unsigned long long)room, n_want, keys, codes, have, ranked));
                if (have >= n_want || !(t > 0.0)) break;
                GTRY(B.dev.drop(level));
            }
            listed = have;
        }
        n_sel = std::min(have, n_want);
    }

    // the selected pairs in (i, j) order: the forward half of the adjacency; the same pairs
    // sorted by j are the other half
    const long long E = 2 * (long long)n_sel;
    *n_edges = E;
    if (E >= (1LL << 31) - 1) return gfail(SG_E_INVALID, "too many edges");
    unsigned long long *rev = nullptr;
    int *head = nullptr;
    long long *ptr = nullptr, *up = nullptr, *down = nullptr;
    GTRY(B.dev.get(&rev, n_sel));
    GTRY(B.dev.get(&head, E));
    GTRY(B.dev.get(&ptr, N + 1));
    GTRY(B.dev.get(&up, N + 1));
    GTRY(B.dev.get(&down, N + 1));
    const int es = B.mark(B.ev_sort);
    if (n_sel && n_sel < listed) GTRY(B.take(keys, codes, (long long)listed, (long long)n_sel, codes));
    if (n_sel) {
        hipLaunchKernelGGL(k_graph_swap, dim3(blocks_for((long long)n_sel, 256)), dim3(256), 0, st, (long long)n_sel,
                           (const unsigned long long *)codes, rev);
        GHIP(hipGetLastError());
        GTRY(B.sort_codes(rev, nullptr, (long long)n_sel, false));
    }
    B.end(B.ev_sort, es);
    hipLaunchKernelGGL(k_graph_rowptr, dim3(blocks_for(N + 1, 256)), dim3(256), 0, st, N, (long long)n_sel,
                       (const unsigned long long *)codes, (const unsigned long long *)rev, up, down, ptr);
    GHIP(hipGetLastError());
    if (n_sel) {
        hipLaunchKernelGGL(k_graph_heads, dim3(blocks_for((long long)n_sel, 256)), dim3(256), 0, st, (long long)n_sel, N,
                           (const unsigned long long *)codes, (const unsigned long long *)rev, (const long long *)up,
                           (const long long *)down, head);
        GHIP(hipGetLastError());
    }
    if (adj_ptr) GHIP(hipMemcpyAsync(adj_ptr, ptr, sizeof(int64_t) * (N + 1), hipMemcpyDeviceToHost, st));
    if (adj_idx && cap >= E && E > 0)
        GHIP(hipMemcpyAsync(adj_idx, head, sizeof(int32_t) * E, hipMemcpyDeviceToHost, st));
    GHIP(hipStreamSynchronize(st));
    if (info) {
        info->candidates = (int64_t)ranked;
        info->pairs_evaluated = (int64_t)B.evals;
        info->threshold = t_used;
        info->streamed = streamed;
        info->passes = B.passes;
        info->ms_pairs = Builder::total_ms(B.ev_pairs);
        info->ms_sort = Builder::total_ms(B.ev_sort);
        info->ms_total =
            std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
    }
    return SG_OK;
}

}  // namespace sg

extern "C" sg_status sg_graph_build(sg_ctx *ctx, const sg_graph_desc *desc, void *hip_stream, int64_t *adj_ptr,
                                    int32_t *adj_idx, int64_t cap, int64_t *n_edges, sg_graph_info *info) {
    if (!ctx) return sg::gfail(SG_E_INVALID, "ctx is NULL");
    if (ctx->sticky.load()) return sg::gfail(SG_E_DEVICE, "context is in a failed state");
    if (hipSetDevice(ctx->device) != hipSuccess) return sg::gfail(SG_E_DEVICE, "hipSetDevice failed");
    const sg_status r = sg::graph_build(ctx, desc, hip_stream ? (hipStream_t)hip_stream : ctx->stream, adj_ptr,
                                        adj_idx, cap, n_edges, info);
    const sg_status b = sg::bounds_report();
    return b != SG_OK ? b : r;
}
