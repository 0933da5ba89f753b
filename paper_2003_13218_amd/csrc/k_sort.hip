// Stage a1/a2: wrap, leaf binning, Morton keys, stable counting sort by
// (key, original index), per-leaf ranges and the repack into sorted,
// leaf-local coordinates.  Integer work is bit-exact; the FP64 arithmetic
// that decides a leaf index uses explicitly rounded operations (no FMA
// contraction) so that it equals the plain definition
//   w = x - b floor(x / b)  (0 if that gives b),  c = floor(w * (2^L / b)).
#include "fmm_internal.h"
#include "morton.h"
#include "wrap.h"

namespace fmm {

__global__ void k_sort_begin(uint32_t *__restrict__ count, int64_t nleaf, int *__restrict__ flag) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nleaf;
         i += (int64_t)gridDim.x * blockDim.x)
        count[i] = 0u;
    if (blockIdx.x == 0 && threadIdx.x < kFlags) flag[threadIdx.x] = 0;
}

static inline unsigned grid_for(int64_t n, int bs) {
    int64_t g = (n + bs - 1) / bs;
    if (g > 65535 * 16) g = 65535 * 16;
    if (g < 1) g = 1;
    return (unsigned)g;
}

hipError_t launch_sort_begin(uint32_t *count, int64_t nleaf, int *flag, hipStream_t s) {
    int64_t g = (nleaf + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_sort_begin, dim3((unsigned)g), dim3(256), 0, s, count, nleaf, flag);
    return hipGetLastError();
}

// key[i], the per-leaf counts and every atom's slot in its leaf (in arrival
// order); flag |= 1 for a non-finite position or charge.
// Wave-aggregated increment of ctr[k]: the active lanes of a wavefront that
// share a key add their number once, and each lane gets the counter's old
// value plus its rank among them (its slot).  Neighbouring atoms usually
// share a leaf, so a wavefront's 64 increments become a few atomics, which the
// first lanes of all keys issue together: one round trip per wavefront.  Every
// pass finds the lanes of the first remaining key, so the loop ends after at
// most 64 passes.
__device__ inline uint32_t wave_agg_inc(uint32_t *ctr, uint32_t k) {
    const int lane = threadIdx.x & 63;
    int leader = lane;
    unsigned long long mine = 0;
    bool done = false;
    while (!done) {
        const uint32_t lk = __builtin_amdgcn_readfirstlane(k);
        const unsigned long long m = __ballot(k == lk);
        if (k == lk) {
            leader = __ffsll((long long)m) - 1;
            mine = m;
            done = true;
        }
    }
    uint32_t old = 0;
    if (lane == leader) old = atomicAdd(&ctr[k], (uint32_t)__popcll(mine));
    return __shfl(old, leader) + (uint32_t)__popcll(mine & ((1ull << lane) - 1ull));
}

__global__ void k_bin(int64_t n, const double *__restrict__ pos, const double *__restrict__ q,
                      double box, double scale, uint32_t nc, uint32_t *__restrict__ key,
                      uint32_t *__restrict__ slot, uint32_t *__restrict__ count, int *__restrict__ flag) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
        const double qi = q ? q[i] : 0.0;
        if (!isfinite(x) || !isfinite(y) || !isfinite(z) || !isfinite(qi)) {
            atomicOr(flag, 1);
            key[i] = 0;
            slot[i] = atomicAdd(&count[0], 1u);
            continue;
        }
        const uint32_t cx = leaf_coord(wrap_coord(x, box), scale, nc);
        const uint32_t cy = leaf_coord(wrap_coord(y, box), scale, nc);
        const uint32_t cz = leaf_coord(wrap_coord(z, box), scale, nc);
        const uint32_t k = morton3(cx, cy, cz);
        key[i] = k;
        slot[i] = wave_agg_inc(count, k);
    }
}

hipError_t launch_bin(int64_t n, const double *pos, const double *q, double box, int levels,
                      uint32_t *key, uint32_t *slot, uint32_t *count, int *flag, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const uint32_t nc = 1u << levels;
    const double scale = (double)nc / box;
    hipLaunchKernelGGL(k_bin, dim3(grid_for(n, 256)), dim3(256), 0, s, n, pos, q, box, scale, nc,
                       key, slot, count, flag);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Exclusive scan of uint32 counts into int32 starts (out has n + 1 entries).
// Three-phase: per-block scan of 1024 elements, recursive scan of block sums,
// add-back.  Deterministic integer arithmetic.
// ---------------------------------------------------------------------------
constexpr int kScanBlock = 1024;

__global__ void k_scan_block(const uint32_t *__restrict__ in, int32_t *__restrict__ out, int64_t n,
                             int32_t *__restrict__ block_sums) {
    __shared__ int32_t s[kScanBlock];
    const int64_t base = (int64_t)blockIdx.x * kScanBlock;
    for (int i = threadIdx.x; i < kScanBlock; i += blockDim.x) {
        int64_t g = base + i;
        s[i] = g < n ? (int32_t)in[g] : 0;
    }
    __syncthreads();
    // Hillis-Steele on 1024 elements with 256 threads (4 per thread)
    for (int off = 1; off < kScanBlock; off <<= 1) {
        int32_t v[4];
        for (int u = 0; u < 4; ++u) {
            int i = threadIdx.x * 4 + u;
            v[u] = i >= off ? s[i - off] : 0;
        }
        __syncthreads();
        for (int u = 0; u < 4; ++u) s[threadIdx.x * 4 + u] += v[u];
        __syncthreads();
    }
    for (int i = threadIdx.x; i < kScanBlock; i += blockDim.x) {
        int64_t g = base + i;
        if (g < n) out[g] = (i == 0 ? 0 : s[i - 1]);  // exclusive
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = s[kScanBlock - 1];
}

__global__ void k_scan_add(int32_t *__restrict__ out, int64_t n, const int32_t *__restrict__ offs) {
    const int64_t base = (int64_t)blockIdx.x * kScanBlock;
    const int32_t o = offs[blockIdx.x];
    for (int i = threadIdx.x; i < kScanBlock; i += blockDim.x) {
        int64_t g = base + i;
        if (g < n) out[g] += o;
    }
}

__global__ void k_set_total(int32_t *out, int64_t n, const uint32_t *in) {
    // out[n] = out[n-1] + in[n-1]
    if (threadIdx.x == 0 && blockIdx.x == 0) out[n] = (n > 0 ? out[n - 1] + (int32_t)in[n - 1] : 0);
}

int64_t scan_scratch_len(int64_t n) {
    int64_t total = 0;
    int64_t m = n;
    while (m > 1) {
        int64_t nb = (m + kScanBlock - 1) / kScanBlock;
        total += 2 * nb + 2;
        m = nb;
    }
    return total + 4;
}

// scratch: int32 buffer of scan_scratch_len(n)
static hipError_t scan_rec(const uint32_t *in_u, const int32_t *in_i, int32_t *out, int64_t n,
                           int32_t *scratch, hipStream_t s);

__global__ void k_scan_block_i(const int32_t *__restrict__ in, int32_t *__restrict__ out, int64_t n,
                               int32_t *__restrict__ block_sums) {
    __shared__ int32_t s[kScanBlock];
    const int64_t base = (int64_t)blockIdx.x * kScanBlock;
    for (int i = threadIdx.x; i < kScanBlock; i += blockDim.x) {
        int64_t g = base + i;
        s[i] = g < n ? in[g] : 0;
    }
    __syncthreads();
    for (int off = 1; off < kScanBlock; off <<= 1) {
        int32_t v[4];
        for (int u = 0; u < 4; ++u) {
            int i = threadIdx.x * 4 + u;
            v[u] = i >= off ? s[i - off] : 0;
        }
        __syncthreads();
        for (int u = 0; u < 4; ++u) s[threadIdx.x * 4 + u] += v[u];
        __syncthreads();
    }
    for (int i = threadIdx.x; i < kScanBlock; i += blockDim.x) {
        int64_t g = base + i;
        if (g < n) out[g] = (i == 0 ? 0 : s[i - 1]);
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = s[kScanBlock - 1];
}

static hipError_t scan_rec(const uint32_t *in_u, const int32_t *in_i, int32_t *out, int64_t n,
                           int32_t *scratch, hipStream_t s) {
    const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    int32_t *sums = scratch;
    int32_t *sums_scan = scratch + nb + 1;
    int32_t *rest = scratch + 2 * nb + 2;
    if (in_u)
        hipLaunchKernelGGL(k_scan_block, dim3((unsigned)nb), dim3(256), 0, s, in_u, out, n, sums);
    else
        hipLaunchKernelGGL(k_scan_block_i, dim3((unsigned)nb), dim3(256), 0, s, in_i, out, n, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nb == 1) return e;
    e = scan_rec(nullptr, sums, sums_scan, nb, rest, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(256), 0, s, out, n, sums_scan);
    return hipGetLastError();
}

hipError_t launch_scan(const uint32_t *in, int32_t *out, int64_t n, int32_t *scratch,
                       int64_t scratch_len, hipStream_t s) {
    if (scratch_len < scan_scratch_len(n)) return hipErrorInvalidValue;
    if (n > 0) {
        hipError_t e = scan_rec(in, nullptr, out, n, scratch, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_set_total, dim3(1), dim3(64), 0, s, out, n, in);
    return hipGetLastError();
}

// Leaf ranges of a tree of up to kOneScan leaves in one block: start (of the
// atoms) and pstart (of the near-field copy, every leaf padded to a multiple of
// G), each with its total.  A thread takes a run of leaves, the runs' sums are
// scanned in LDS.  One launch of a few microseconds against up to nine for the
// two scans of the general path (30,001 atoms, 4,096 leaves: 21 us of kernels and
// the gaps between them); beyond 32,768 leaves the runs of one block get longer
// than those launches.
constexpr int kOneScan = 32768;

// R leaves per thread (8^levels leaves: 1, 4 or 32), loaded together
template <int R>
__global__ __launch_bounds__(1024) void k_leaf_ranges(const uint32_t *__restrict__ count, int nleaf, uint32_t G,
                                                      int32_t *__restrict__ start, int32_t *__restrict__ pstart) {
    __shared__ int32_t wave[2][16];
    const int b = threadIdx.x * R;
    const bool on = b < nleaf;  // R > 1: every thread
    uint32_t c[R];
    if constexpr (R == 1) {
        c[0] = on ? count[b] : 0u;
    } else {
#pragma unroll
        for (int i = 0; i < R; i += 4) {
            const uint4 v = *reinterpret_cast<const uint4 *>(count + b + i);
            c[i] = v.x;
            c[i + 1] = v.y;
            c[i + 2] = v.z;
            c[i + 3] = v.w;
        }
    }
    int32_t s = 0, p = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        s += (int32_t)c[i];
        p += (int32_t)((c[i] + G - 1) / G * G);
    }
    int32_t is = s, ip = p;  // inclusive over the wavefront, then over wavefronts
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t us = __shfl_up(is, d), up = __shfl_up(ip, d);
        if (lane >= d) {
            is += us;
            ip += up;
        }
    }
    if (lane == 63) {
        wave[0][w] = is;
        wave[1][w] = ip;
    }
    __syncthreads();
    for (int k = 0; k < w; ++k) {
        is += wave[0][k];
        ip += wave[1][k];
    }
    if (threadIdx.x == 1023) {
        start[nleaf] = is;
        pstart[nleaf] = ip;
    }
    if (!on) return;
    is -= s;
    ip -= p;
    int32_t vs[R], vp[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        vs[i] = is;
        vp[i] = ip;
        is += (int32_t)c[i];
        ip += (int32_t)((c[i] + G - 1) / G * G);
    }
    if constexpr (R == 1) {
        start[b] = vs[0];
        pstart[b] = vp[0];
    } else {
#pragma unroll
        for (int i = 0; i < R; i += 4) {
            *reinterpret_cast<int4 *>(start + b + i) = make_int4(vs[i], vs[i + 1], vs[i + 2], vs[i + 3]);
            *reinterpret_cast<int4 *>(pstart + b + i) = make_int4(vp[i], vp[i + 1], vp[i + 2], vp[i + 3]);
        }
    }
}

// pcount: nleaf entries (used beyond kOneScan leaves only)
__global__ void k_pad_counts(int64_t nleaf, const uint32_t *__restrict__ count, uint32_t G,
                             uint32_t *__restrict__ pcount) {
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < nleaf;
         c += (int64_t)gridDim.x * blockDim.x)
        pcount[c] = (count[c] + G - 1) / G * G;
}

hipError_t launch_leaf_ranges(const uint32_t *count, int64_t nleaf, int G, int32_t *start, int32_t *pstart,
                              uint32_t *pcount, int32_t *scratch, int64_t scratch_len, hipStream_t s) {
    if (nleaf <= kOneScan) {
        auto k = nleaf <= 1024 ? k_leaf_ranges<1> : nleaf == 4096 ? k_leaf_ranges<4> : k_leaf_ranges<32>;
        if (nleaf > 1024 && nleaf != 4096 && nleaf != 32768) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k, dim3(1), dim3(1024), 0, s, count, (int)nleaf, (uint32_t)G, start, pstart);
        return hipGetLastError();
    }
    hipError_t e = launch_scan(count, start, nleaf, scratch, scratch_len, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pad_counts, dim3(grid_for(nleaf, 256)), dim3(256), 0, s, nleaf, count, (uint32_t)G, pcount);
    return launch_scan(pcount, pstart, nleaf, scratch, scratch_len, s);
}

// Original indices into their leaf segment (order inside a segment is then
// fixed by rank: k_cell_sort, k_sort_gather).
__global__ void k_scatter(int64_t n, const uint32_t *__restrict__ key, const uint32_t *__restrict__ slot,
                          const int32_t *__restrict__ start, int32_t *__restrict__ perm) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        perm[start[key[i]] + (int32_t)slot[i]] = (int32_t)i;
}

hipError_t launch_scatter(int64_t n, const uint32_t *key, const uint32_t *slot, const int32_t *start, int32_t *perm,
                          hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter, dim3(grid_for(n, 256)), dim3(256), 0, s, n, key, slot, start, perm);
    return hipGetLastError();
}

// Order each leaf segment by original index: makes the order (key, index),
// i.e. a stable sort, independent of atomic arrival order.  One wavefront
// per leaf: the segment is staged in LDS and every lane places its entries
// by rank (the number of smaller indices in the segment; indices are
// distinct), so the cost is n^2/64 compares per leaf instead of a serial
// insertion sort.  Segments longer than kSortCap (degenerate inputs) are
// sorted by lane 0 by insertion.
constexpr int kSortCap = 1024;

__device__ inline void insertion_sort(int32_t *perm, int32_t b, int32_t n) {
    for (int32_t i = b + 1; i < b + n; ++i) {
        const int32_t v = perm[i];
        int32_t j = i - 1;
        while (j >= b && perm[j] > v) {
            perm[j + 1] = perm[j];
            --j;
        }
        perm[j + 1] = v;
    }
}

__global__ __launch_bounds__(256) void k_cell_sort(int64_t nleaf, const int32_t *__restrict__ start,
                                                   int32_t *__restrict__ perm) {
    __shared__ int32_t buf[4][kSortCap];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int64_t c = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + w));
    if (c >= nleaf) return;  // whole wavefront; no block barriers below
    const int32_t b = start[c], n = start[c + 1] - b;
    if (n <= 1) return;
    if (n > kSortCap) {
        if (lane == 0) insertion_sort(perm, b, n);
        return;
    }
    int32_t *sb = buf[w];
    for (int32_t i = lane; i < n; i += 64) sb[i] = perm[b + i];
    // LDS accesses of one wavefront complete in order; the fence keeps the
    // compiler from moving the reads above the writes
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int32_t i = lane; i < n; i += 64) {
        const int32_t v = sb[i];
        int32_t r = 0;
        for (int32_t j = 0; j < n; ++j) r += sb[j] < v ? 1 : 0;
        perm[b + r] = v;
    }
}

hipError_t launch_cell_sort(int64_t nleaf, const int32_t *start, int32_t *perm, hipStream_t s) {
    if (nleaf <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cell_sort, dim3((unsigned)((nleaf + 3) / 4)), dim3(256), 0, s, nleaf, start, perm);
    return hipGetLastError();
}

// k_cell_sort and the repack in one pass, one wavefront per leaf: every lane
// places its entries by rank and writes them there at once:
//   xq   leaf-local coordinates (x - leaf centre) and charge in the mode's
//        precision;
//   xs   an FP64 copy of the wrapped position measured from the box centre and
//        the charge, which the correction terms, the energy reduction and the
//        solute-solvent pass read later (so they never touch the caller's
//        arrays again);
//   xqp  the near-field copy of xq, every leaf padded to its pstart range (a
//        multiple of the P2P source groups, so the P2P inner loop needs no
//        per-lane bounds test).  Padding atoms have q = 0 and sit far outside
//        the leaf (leaf-local coordinate `far` per axis), where their terms
//        vanish without forming 0/0.
// (Sort, repack and padded copy as three launches: 10 + 18 + 9 us on the
// 1M-atom box and three launches of a small box's fifteen before the far field.)
template <typename T>
__global__ __launch_bounds__(256) void k_sort_gather(int64_t nleaf, const int32_t *__restrict__ start,
                                                     const int32_t *__restrict__ pstart, int32_t *__restrict__ perm,
                                                     const double *__restrict__ pos, const double *__restrict__ q,
                                                     double box, double h, T far, T *__restrict__ xq,
                                                     double *__restrict__ xs, T *__restrict__ xqp) {
    __shared__ int32_t buf[4][kSortCap];
    typedef T V4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(w);
    if (c >= nleaf) return;  // whole wavefront; no block barriers below
    const int32_t b = start[c], n = start[c + 1] - b;
    const int32_t p0 = pstart[c], pn = pstart[c + 1] - p0;
    uint32_t lc[3];
    demorton3((uint32_t)c, lc[0], lc[1], lc[2]);
    const double hb = 0.5 * box;
    auto place = [&](int32_t i, int32_t r) {  // atom i at rank r of the leaf
        double wr[3], loc[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            wr[a] = wrap_coord(pos[3 * (int64_t)i + a], box);
            loc[a] = wr[a] - ((double)lc[a] + 0.5) * h;
        }
        const double qi = q[i];
        const V4 v = {(T)loc[0], (T)loc[1], (T)loc[2], (T)qi};
        reinterpret_cast<V4 *>(xq)[b + r] = v;
        reinterpret_cast<V4 *>(xqp)[p0 + r] = v;
        double *x = xs + 4 * (int64_t)(b + r);
        x[0] = wr[0] - hb;
        x[1] = wr[1] - hb;
        x[2] = wr[2] - hb;
        x[3] = qi;
    };
    for (int32_t i = n + lane; i < pn; i += 64) reinterpret_cast<V4 *>(xqp)[p0 + i] = V4{far, far, far, (T)0};
    if (n > kSortCap) {
        if (lane == 0) insertion_sort(perm, b, n);
        __threadfence();  // lane 0's stores before the wavefront's loads
        for (int32_t i = lane; i < n; i += 64) place(((volatile int32_t *)perm)[b + i], i);
        return;
    }
    int32_t *sb = buf[w];
    for (int32_t i = lane; i < n; i += 64) sb[i] = perm[b + i];
    // LDS accesses of one wavefront complete in order; the fence keeps the
    // compiler from moving the reads above the writes
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int32_t i = lane; i < n; i += 64) {
        const int32_t v = sb[i];
        int32_t r = 0;
        for (int32_t j = 0; j < n; ++j) r += sb[j] < v ? 1 : 0;
        perm[b + r] = v;
        place(v, r);
    }
}

hipError_t launch_sort_gather(int64_t nleaf, const int32_t *start, const int32_t *pstart, int32_t *perm,
                              const double *pos, const double *q, double box, int levels, bool fp64, double far,
                              void *xq, double *xs, void *xqp, hipStream_t s) {
    if (nleaf <= 0) return hipSuccess;
    const unsigned grid = (unsigned)((nleaf + 3) / 4);
    const double h = box / (double)(1u << levels);
    if (fp64)
        hipLaunchKernelGGL(k_sort_gather<double>, dim3(grid), dim3(256), 0, s, nleaf, start, pstart, perm, pos, q, box,
                           h, far, (double *)xq, xs, (double *)xqp);
    else
        hipLaunchKernelGGL(k_sort_gather<float>, dim3(grid), dim3(256), 0, s, nleaf, start, pstart, perm, pos, q, box,
                           h, (float)far, (float *)xq, xs, (float *)xqp);
    return hipGetLastError();
}

// Solute-only charges for the second far-field pass of the solute-solvent
// scheme: xq_u = xq with q multiplied by the solute flag of the atom.
template <typename T>
__global__ void k_mask_charges(int64_t n, const int32_t *__restrict__ perm, const uint8_t *__restrict__ mask,
                               const T *__restrict__ xq, T *__restrict__ xq_u) {
    for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < n;
         s += (int64_t)gridDim.x * blockDim.x) {
        const bool u = mask[perm[s]] != 0;
        xq_u[4 * s + 0] = xq[4 * s + 0];
        xq_u[4 * s + 1] = xq[4 * s + 1];
        xq_u[4 * s + 2] = xq[4 * s + 2];
        xq_u[4 * s + 3] = u ? xq[4 * s + 3] : (T)0;
    }
}

hipError_t launch_mask_charges(int64_t n, const int32_t *perm, const uint8_t *mask, bool fp64, const void *xq,
                               void *xq_u, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (fp64)
        hipLaunchKernelGGL(k_mask_charges<double>, dim3(grid_for(n, 256)), dim3(256), 0, s, n, perm, mask,
                           (const double *)xq, (double *)xq_u);
    else
        hipLaunchKernelGGL(k_mask_charges<float>, dim3(grid_for(n, 256)), dim3(256), 0, s, n, perm, mask,
                           (const float *)xq, (float *)xq_u);
    return hipGetLastError();
}

// out[i] = 1 - (mask[i] != 0): the solvent as the masked set
__global__ void k_invert_mask(int64_t n, const uint8_t *__restrict__ mask, uint8_t *__restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = mask[i] ? 0 : 1;
}

hipError_t launch_invert_mask(int64_t n, const uint8_t *mask, uint8_t *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_invert_mask, dim3(grid_for(n, 256)), dim3(256), 0, s, n, mask, out);
    return hipGetLastError();
}

}  // namespace fmm
