// Normalization (Sec. 5.1.1) and the octree build (Sec. 4.5) on the device.
//
// The octree over [-1,1]^3 with maximum depth D is the tree of Morton-code
// prefixes: quantize each coordinate to 15 bits, interleave into a 45-bit
// key, sort, and a node at depth d is a maximal run of sorted keys sharing
// their top 3d bits whose parent run holds more than one point.  With sorted
// keys this is decided locally: point i starts nodes at the depths
// L+1 .. min(max(L,R)+1, D), where L and R are the numbers of leading octal
// digits it shares with its left and right neighbours.  Numbering the nodes
// point by point, shallow to deep, yields a depth-first pre-order in which
// the first child of a node is the next node and a subtree is a contiguous
// index range.
#include <float.h>

#include <algorithm>
#include <utility>
#include <vector>

#include "common.h"
#include "internal.h"

namespace wnnc {

// ------------------------------------------------------------ normalize --
// Each cloud c (caller rows off[c] .. off[c+1]) is normalized on its own.

constexpr int kNormBlocksPerCloud = 32;

int64_t normalize_tmp_doubles(int64_t nclouds) {
    return nclouds * (kNormBlocksPerCloud * 6 + 4) + 8;
}

__device__ inline int cloud_of_row(const int64_t *off, int nclouds, int64_t i) {
    int lo = 0, hi = nclouds;  // off[lo] <= i < off[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= i)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// grid (kNormBlocksPerCloud, nclouds): per-block extremes of one cloud
__global__ __launch_bounds__(256) void k_minmax(const float *__restrict__ P,
                                                const int64_t *__restrict__ off,
                                                double *__restrict__ part) {
    const int c = blockIdx.y;
    const int64_t lo_i = off[c], hi_i = off[c + 1];
    float lo[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, hi[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
    for (int64_t i = lo_i + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi_i;
         i += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            float v = P[3 * i + k];
            lo[k] = fminf(lo[k], v);
            hi[k] = fmaxf(hi[k], v);
        }
    }
    __shared__ float s[6][256];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        s[k][threadIdx.x] = lo[k];
        s[3 + k][threadIdx.x] = hi[k];
    }
    __syncthreads();
    for (int d = 128; d > 0; d >>= 1) {
        if (threadIdx.x < d) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                s[k][threadIdx.x] = fminf(s[k][threadIdx.x], s[k][threadIdx.x + d]);
                s[3 + k][threadIdx.x] = fmaxf(s[3 + k][threadIdx.x], s[3 + k][threadIdx.x + d]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 6)
        part[((int64_t)c * kNormBlocksPerCloud + blockIdx.x) * 6 + threadIdx.x] = s[threadIdx.x][0];
}

// One thread per cloud: extremes -> centre and scale in FP64.
__global__ void k_norm_finalize(const double *__restrict__ part, int nclouds,
                                double *__restrict__ cs) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nclouds) return;
    double lo[3], hi[3];
    for (int k = 0; k < 3; ++k) {
        lo[k] = DBL_MAX;
        hi[k] = -DBL_MAX;
    }
    for (int b = 0; b < kNormBlocksPerCloud; ++b)
        for (int k = 0; k < 3; ++k) {
            lo[k] = fmin(lo[k], part[((int64_t)c * kNormBlocksPerCloud + b) * 6 + k]);
            hi[k] = fmax(hi[k], part[((int64_t)c * kNormBlocksPerCloud + b) * 6 + 3 + k]);
        }
    double half = 0.0;
    for (int k = 0; k < 3; ++k) {
        cs[4 * c + k] = (lo[k] + hi[k]) / 2.0;
        half = fmax(half, (hi[k] - lo[k]) / 2.0);
    }
    cs[4 * c + 3] = half > 0.0 ? (10.0 / 11.0) / half : 1.0;
}

__global__ __launch_bounds__(256) void k_norm_apply(const float *P, int64_t n3, float *Q,
                                                    const int64_t *__restrict__ off, int nclouds,
                                                    const double *__restrict__ cs) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n3) return;
    const int k = (int)(i % 3);
    const int c = nclouds == 1 ? 0 : cloud_of_row(off, nclouds, i / 3);
    Q[i] = (float)(((double)P[i] - cs[4 * c + k]) * cs[4 * c + 3]);
}

// tmp layout: [partials | centre/scale (4 per cloud)]; returns the offset of
// the centre/scale block in tmp.
int64_t launch_normalize(const float *P, int64_t n, const int64_t *d_off, int nclouds,
                         float *P_norm, double *tmp, hipStream_t st) {
    double *cs = tmp + (int64_t)nclouds * kNormBlocksPerCloud * 6;
    hipLaunchKernelGGL(k_minmax, dim3(kNormBlocksPerCloud, nclouds), dim3(256), 0, st, P, d_off, tmp);
    hipLaunchKernelGGL(k_norm_finalize, dim3((nclouds + 63) / 64), dim3(64), 0, st, tmp, nclouds, cs);
    const int64_t n3 = 3 * n;
    hipLaunchKernelGGL(k_norm_apply, dim3((unsigned)((n3 + 255) / 256)), dim3(256), 0, st, P, n3,
                       P_norm, d_off, nclouds, cs);
    return (int64_t)nclouds * kNormBlocksPerCloud * 6;
}

// ----------------------------------------------------------------- morton --

// Spread the low 15 bits of v so that bit b lands on bit 3b.
__device__ inline unsigned long long spread3(unsigned v) {
    unsigned long long x = v & 0x7fffu;
    x = (x | (x << 16)) & 0x00000000ff0000ffull;
    x = (x | (x << 8)) & 0x000000f00f00f00full;
    x = (x | (x << 4)) & 0x00000c30c30c30c3ull;
    x = (x | (x << 2)) & 0x0000249249249249ull;
    return x;
}

// Cell index of coordinate v along one axis at depth 15:
// floor((v + 1) 2^14) clamped to [0, 2^15 - 1], evaluated as
// floor(v 2^14) + 2^14, which is exact in FP32 (the scaling is by a power of
// two).  A coordinate on a split plane goes to the upper cell.
__device__ inline unsigned quantize15(float v) {
    float f = floorf(v * 16384.0f) + 16384.0f;
    f = fminf(fmaxf(f, 0.0f), 32767.0f);
    return (unsigned)f;
}

__global__ __launch_bounds__(256) void k_morton(const float *__restrict__ P, int64_t n,
                                                const int64_t *__restrict__ off, int nclouds,
                                                unsigned long long *__restrict__ keys,
                                                uint32_t *__restrict__ vals) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    unsigned qx = quantize15(P[3 * i]), qy = quantize15(P[3 * i + 1]), qz = quantize15(P[3 * i + 2]);
    const unsigned long long c = nclouds == 1 ? 0ull : (unsigned long long)cloud_of_row(off, nclouds, i);
    keys[i] = (c << kMortonBits) | (spread3(qx) << 2) | (spread3(qy) << 1) | spread3(qz);
    vals[i] = (uint32_t)i;
}

// Cloud index of every sorted point (clouds stay contiguous and in order).
__global__ __launch_bounds__(256) void k_point_cloud(const unsigned long long *__restrict__ keys,
                                                     int64_t n, int32_t *__restrict__ cloud) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) cloud[i] = (int32_t)(keys[i] >> kMortonBits);
}

// ------------------------------------------------------------ radix sort --
// Stable LSD radix sort of (45-bit key, uint32 value), 9 bits per pass: the
// 45 bits take five passes of three kernels (a tile's digit counts, their
// prefix sums over the tiles, the scatter).  It is bound by the latency of
// its launches and barriers, not by its 24 bytes per key and pass.  With 8
// bits, six passes of five kernels (the counts scanned as one array) and a
// barrier after every 256 keys, sorting 262k query points took 147 us; this
// takes 65 us (a scatter 7 us, 1.2 TB/s).

constexpr int kRsBits = 9;
constexpr int kRsBins = 1 << kRsBits;
constexpr int kRsThreads = kRsBins;  // one thread per digit
constexpr int kRsWaves = kRsThreads / kWave;
constexpr int kRsItems = 4;  // keys per thread; 2 and 8 build as fast at 2k to 3M points
constexpr int kRsTile = kRsThreads * kRsItems;

static inline int rs_tiles(int64_t n) { return (int)((n + kRsTile - 1) / kRsTile); }

int rs_passes(int key_bits) { return (key_bits + kRsBits - 1) / kRsBits; }

// Inclusive prefix sum over the wavefront's lanes.
__device__ inline uint32_t wave_scan_u32(uint32_t v, int lane) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(v, d);
        v += lane >= d ? o : 0u;
    }
    return v;
}

__global__ __launch_bounds__(kRsThreads) void k_rs_hist(const unsigned long long *__restrict__ keys,
                                                        int64_t n, int shift,
                                                        uint32_t *__restrict__ hist, int ntiles) {
    __shared__ uint32_t h[kRsBins];
    h[threadIdx.x] = 0;
    const int64_t base = (int64_t)blockIdx.x * kRsTile;
    unsigned long long key[kRsItems];
#pragma unroll
    for (int k = 0; k < kRsItems; ++k) {
        const int64_t i = base + k * kRsThreads + threadIdx.x;
        key[k] = i < n ? keys[i] : 0ull;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRsItems; ++k)
        if (base + k * kRsThreads + threadIdx.x < n)
            atomicAdd(&h[(unsigned)(key[k] >> shift) & (kRsBins - 1)], 1u);
    __syncthreads();
    hist[(int64_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

// One wavefront per digit: its tiles' counts become their exclusive prefix
// sums, total[digit] their sum.
__global__ __launch_bounds__(256) void k_rs_scan(uint32_t *__restrict__ hist, int ntiles,
                                                 uint32_t *__restrict__ total) {
    const int lane = threadIdx.x & (kWave - 1);
    const int bin = blockIdx.x * (256 / kWave) + threadIdx.x / kWave;
    uint32_t *row = hist + (int64_t)bin * ntiles;
    uint32_t carry = 0u;
    for (int t0 = 0; t0 < ntiles; t0 += 4 * kWave) {
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = t0 + k * kWave + lane;
            v[k] = t < ntiles ? row[t] : 0u;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = t0 + k * kWave + lane;
            const uint32_t inc = wave_scan_u32(v[k], lane);
            if (t < ntiles) row[t] = carry + inc - v[k];
            carry += __shfl(inc, kWave - 1);
        }
    }
    if (lane == 0) total[bin] = carry;
}

// A wavefront ranks its 64 * kRsItems consecutive keys by itself, counting the
// digits in its own row of LDS; one barrier then joins the rows.
__global__ __launch_bounds__(kRsThreads) void k_rs_scatter(
    const unsigned long long *__restrict__ kin, const uint32_t *__restrict__ vin,
    unsigned long long *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n, int shift,
    const uint32_t *__restrict__ offs, const uint32_t *__restrict__ total, int ntiles) {
    __shared__ uint32_t wc[kRsWaves][kRsBins];
    __shared__ uint32_t wsum[kRsWaves];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv = tid / kWave;
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int64_t first = ((int64_t)blockIdx.x * kRsWaves + wv) * kWave * kRsItems + lane;
    const uint32_t tot = total[tid];
    const uint32_t off = offs[(int64_t)tid * ntiles + blockIdx.x];
    unsigned long long key[kRsItems];
    uint32_t val[kRsItems], pos[kRsItems];
#pragma unroll
    for (int r = 0; r < kRsItems; ++r) {
        const int64_t i = first + r * kWave;
        key[r] = i < n ? kin[i] : 0ull;
        val[r] = i < n ? vin[i] : 0u;
    }
#pragma unroll
    for (int w = 0; w < kRsWaves; ++w) wc[w][tid] = 0u;
    const uint32_t inc = wave_scan_u32(tot, lane);
    if (lane == kWave - 1) wsum[wv] = inc;
    __syncthreads();
    volatile uint32_t *cnt = wc[wv];
#pragma unroll
    for (int r = 0; r < kRsItems; ++r) {
        const bool valid = first + r * kWave < n;
        const unsigned dig = (unsigned)(key[r] >> shift) & (kRsBins - 1);
        unsigned long long peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRsBits; ++b) {
            const bool bit = (dig >> b) & 1u;
            const unsigned long long m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t rank = (uint32_t)__popcll(peers & lt);
        const uint32_t before = cnt[dig];
        pos[r] = before + rank;
        if (valid && rank == 0u) cnt[dig] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {
        uint32_t b = off + inc - tot;
        for (int w = 0; w < wv; ++w) b += wsum[w];
#pragma unroll
        for (int w = 0; w < kRsWaves; ++w) {
            const uint32_t c = wc[w][tid];
            wc[w][tid] = b;
            b += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRsItems; ++r) {
        if (first + r * kWave < n) {
            const uint32_t p = wc[wv][(unsigned)(key[r] >> shift) & (kRsBins - 1)] + pos[r];
            kout[p] = key[r];
            vout[p] = val[r];
        }
    }
}

// ----------------------------------------------------------------- nodes --

// Number of leading octal digits (of 15) shared by two keys; -1 for keys of
// different clouds.
__device__ inline int lcp_digits(unsigned long long a, unsigned long long b) {
    unsigned long long x = a ^ b;
    if (x == 0ull) return 15;
    if (x >> kMortonBits) return -1;
    return (__clzll(x) - (64 - kMortonBits)) / 3;
}

__device__ inline void neighbour_lcp(const unsigned long long *keys, int64_t n, int64_t i, int D,
                                     int *L, int *R) {
    const unsigned long long k = keys[i];
    int l = i > 0 ? lcp_digits(keys[i - 1], k) : -1;
    int r = i + 1 < n ? lcp_digits(k, keys[i + 1]) : -1;
    *L = l > D ? D : l;
    *R = r > D ? D : r;
}

// First sorted position after i whose key leaves the depth-d cell of key i
// (at depth 0 the cell is the cloud: the shift keeps only the cloud bits).
__device__ inline int64_t run_end(const unsigned long long *keys, int64_t n, int64_t i, int d) {
    const int shift = 3 * (15 - d);
    const unsigned long long pre = keys[i] >> shift;
    int64_t lo = i, step = 1;
    while (lo + step < n && (keys[lo + step] >> shift) == pre) {
        lo += step;
        step <<= 1;
    }
    int64_t hi = lo + step < n ? lo + step : n;  // keys[hi] differs, or hi == n
    while (hi - lo > 1) {
        int64_t mid = lo + (hi - lo) / 2;
        if ((keys[mid] >> shift) == pre)
            lo = mid;
        else
            hi = mid;
    }
    return hi;
}

// First sorted position of the run of depth-d cells that holds i (the
// mirror of run_end).
__device__ inline int64_t run_start(const unsigned long long *keys, int64_t i, int d) {
    const int shift = 3 * (15 - d);
    const unsigned long long pre = keys[i] >> shift;
    int64_t hi = i, step = 1;
    while (hi - step >= 0 && (keys[hi - step] >> shift) == pre) {
        hi -= step;
        step <<= 1;
    }
    int64_t lo = hi - step >= 0 ? hi - step : -1;  // keys[lo] differs, or lo == -1
    while (hi - lo > 1) {
        int64_t mid = lo + (hi - lo) / 2;
        if ((keys[mid] >> shift) == pre)
            hi = mid;
        else
            lo = mid;
    }
    return hi;
}

// The nodes whose first point is i, outermost first (pre-order), as
// emit(depth, end, leaf).  A node at depth d >= 1 is there when its parent
// (the depth d-1 run holding i) holds more than K points; it is a leaf when
// it holds at most K points or d == D.  With K = 1 (Alg. 4's tree) these
// are the depths from one below the common prefix with the left neighbour
// down to where i is alone, with no search.  Returns the node count.
template <class Emit>
__device__ inline int node_chain(const unsigned long long *keys, int64_t n, int64_t i, int D,
                                 int K, Emit &&emit) {
    int L, R;
    neighbour_lcp(keys, n, i, D, &L, &R);
    if (L >= D) return 0;
    if (K <= 1) {
        int hi = (L > R ? L : R) + 1;
        if (hi > D) hi = D;
        for (int d = L + 1; d <= hi; ++d) {
            const int64_t end = run_end(keys, n, i, d);
            emit(d, end, (end - i == 1) || (d == D));
        }
        return hi - L;
    }
    int cnt = 0;
    for (int d = L + 1; d <= D; ++d) {
        if (d >= 1) {
            const int64_t pb = d - 1 == L ? run_start(keys, i, L) : i;
            if (run_end(keys, n, i, d - 1) - pb <= K) break;
        }
        const int64_t end = run_end(keys, n, i, d);
        const bool leaf = end - i <= K || d == D;
        emit(d, end, leaf);
        ++cnt;
        if (leaf) break;
    }
    return cnt;
}

__global__ __launch_bounds__(256) void k_count_nodes(const unsigned long long *__restrict__ keys,
                                                     int64_t n, int D, int K,
                                                     uint32_t *__restrict__ counts) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    if (i == n) {
        counts[n] = 0;
        return;
    }
    if (K <= 1) {  // no run boundaries needed for the count
        int L, R;
        neighbour_lcp(keys, n, i, D, &L, &R);
        int hi = (L > R ? L : R) + 1;
        if (hi > D) hi = D;
        counts[i] = L >= D ? 0u : (uint32_t)(hi - L);
        return;
    }
    counts[i] = (uint32_t)node_chain(keys, n, i, D, K, [](int, int64_t, bool) {});
}

__global__ __launch_bounds__(256) void k_emit_nodes(const unsigned long long *__restrict__ keys,
                                                    int64_t n, int D, int K,
                                                    const uint32_t *__restrict__ node_off,
                                                    int4 *__restrict__ topo,
                                                    uint32_t *__restrict__ strad_flag) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t idx = node_off[i];
    node_chain(keys, n, i, D, K, [&](int d, int64_t end, bool leaf) {
        topo[idx] = make_int4((int)node_off[end], (int)i, (int)end, d | ((leaf ? 1 : 0) << 4));
        strad_flag[idx] = ((i / kChunk) != ((end - 1) / kChunk)) ? 1u : 0u;
        ++idx;
    });
}

__global__ __launch_bounds__(256) void k_gather_roots(const uint32_t *__restrict__ node_off,
                                                      const int64_t *__restrict__ off, int nclouds,
                                                      int32_t *__restrict__ roots) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c <= nclouds) roots[c] = (int32_t)node_off[off[c]];
}

// Extract every third bit (bit 3b of x -> bit b), 15 bits.
__device__ inline unsigned compact3_15(unsigned long long x) {
    x &= 0x1249249249249ull;
    x = (x ^ (x >> 2)) & 0x10c30c30c30c3ull;
    x = (x ^ (x >> 4)) & 0x100f00f00f00full;
    x = (x ^ (x >> 8)) & 0x1f0000ff0000ffull;
    x = (x ^ (x >> 16)) & 0x1f00000000ffffull;
    x = (x ^ (x >> 32)) & 0x7fffull;
    return (unsigned)x;
}

// Static parts of the node records: the point range of every record (the
// moment passes write the rest), and the geometry of every node for
// searches by distance (the neighbour search, and the planning of the
// operators' walks): a single-point leaf holds its
// point (x, y, z, -1); any other node its cell (lower corner x, y, z, side),
// from the Morton key of its first point.
__global__ __launch_bounds__(256) void k_node_cells(const int4 *__restrict__ topo,
                                                    const unsigned long long *__restrict__ keys,
                                                    const float4 *__restrict__ pts, int64_t m,
                                                    float4 *__restrict__ cells,
                                                    float4 *__restrict__ mom) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= m) return;
    const int4 t = topo[k];
    // the parts of the record that no moment pass writes: flags,
    // skip pointer, point range; of a single-point leaf, whose representative
    // is its point whatever its attribute, also its position (hi = the
    // point, lo = 0) and threshold (-1: every target takes it)
    const bool single = (t.w & kRecLeaf) && t.z - t.y == 1;
    // the children of a node that is no leaf: the next node, then from each
    // child its skip pointer, up to the end of the node's subtree
    int nk = 0, wide = 0;
    float4 r3 = make_float4(__int_as_float(t.y), __int_as_float(t.z), 0.f, 0.f);
    if (!(t.w & kRecLeaf)) {
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        int c = (int)k + 1;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (c < t.x) {
                const uint32_t d = (uint32_t)(c - (int)k);
                if (d > 0xffffu) wide = kRecWideKids;
                if (q > 0) w[(q - 1) / 2] |= (d & 0xffffu) << (16 * ((q - 1) & 1));
                ++nk;
                c = topo[c].x;
            }
        }
        r3 = make_float4(__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]),
                         __uint_as_float(w[3]));
    }
    float4 r0 = make_float4(0.f, 0.f, 0.f,
                            __int_as_float((t.w & 31) | wide | (nk << kRecKidShift)));
    float4 r2 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (single) {
        const float4 q = pts[t.y];
        r0 = make_float4(q.x, q.y, q.z, __int_as_float((t.w & 31) | kRecSingle));
        r2.w = -1.0f;
    }
    const float4 r1 = make_float4(0.f, 0.f, 0.f, __int_as_float(t.x));
    float4 *ra = mom + kRecStride * k;
    ra[0] = r0, ra[1] = r1, ra[2] = r2, ra[3] = r3;
    if (single) {
        cells[k] = make_float4(r0.x, r0.y, r0.z, -1.0f);
        return;
    }
    const int depth = t.w & 15;
    const int sh = kMaxDepth - depth;
    const float w = ldexpf(1.0f, 1 - depth);
    const unsigned long long mk = keys[t.y] & ((1ull << kMortonBits) - 1ull);
    cells[k] = make_float4(-1.0f + (float)(compact3_15(mk >> 2) >> sh) * w,
                           -1.0f + (float)(compact3_15(mk >> 1) >> sh) * w,
                           -1.0f + (float)(compact3_15(mk) >> sh) * w, w);
}

__global__ __launch_bounds__(256) void k_gather_points(const float *__restrict__ P,
                                                       const uint32_t *__restrict__ perm,
                                                       int64_t n, float4 *__restrict__ pts) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t j = perm[i];
    pts[i] = make_float4(P[3 * (int64_t)j], P[3 * (int64_t)j + 1], P[3 * (int64_t)j + 2], 0.0f);
}

// Straddlers (nodes whose points cross a chunk boundary of the moment pass)
// are numbered wide ones first: a wide straddler has more chunks in between
// than a wavefront has lanes and is summed by a whole workgroup, the others
// by a wavefront each.  On entry flag marks the straddlers; on return flag
// marks the narrow ones and wflag the wide ones (both m + 1 entries, the
// last 0, for the exclusive scans that number them).
__global__ __launch_bounds__(256) void k_split_wide(const int4 *__restrict__ topo, int64_t m,
                                                    uint32_t *__restrict__ flag,
                                                    uint32_t *__restrict__ wflag) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= m || !flag[k]) return;
    const int4 t = topo[k];
    const bool wide = (t.z - 1) / kChunk - t.y / kChunk - 1 > kWave;
    flag[k] = wide ? 0u : 1u;
    wflag[k] = wide ? 1u : 0u;
}

// Slot of every straddler (wide ones 0 .. n_wide - 1, then the narrow ones)
// and the moment pass's view of every node.
__global__ __launch_bounds__(256) void k_strad_compact(const uint32_t *__restrict__ flag,
                                                       const uint32_t *__restrict__ slot,
                                                       const uint32_t *__restrict__ wflag,
                                                       const uint32_t *__restrict__ wslot,
                                                       const int4 *__restrict__ topo, int64_t m,
                                                       int32_t *__restrict__ node_strad,
                                                       int32_t *__restrict__ strad_node,
                                                       int4 *__restrict__ strad_topo,
                                                       int2 *__restrict__ mnode) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= m) return;
    const int4 t = topo[k];
    const int n_wide = (int)wslot[m];
    const int sl = wflag[k] ? (int)wslot[k] : (flag[k] ? n_wide + (int)slot[k] : -1);
    node_strad[k] = sl;
    if (sl >= 0) {
        strad_node[sl] = (int32_t)k;
        strad_topo[sl] = t;
        mnode[k] = make_int2(t.y, -1 - sl);
    } else {
        mnode[k] = make_int2(t.y, t.z | (topo_depth(t.w) << kMnodeEndBits));
    }
}

__global__ __launch_bounds__(256) void k_tail_count(const int32_t *__restrict__ strad_node,
                                                    const int4 *__restrict__ topo, int ns,
                                                    uint32_t *__restrict__ cnt) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= ns) return;
    const int e = topo[strad_node[s]].z;
    atomicAdd(&cnt[(e - 1) / kChunk], 1u);
}

// (straddler slot, end point) of every straddler, listed under the chunk
// its range ends in
__global__ __launch_bounds__(256) void k_tail_fill(const int32_t *__restrict__ strad_node,
                                                   const int4 *__restrict__ topo, int ns,
                                                   uint32_t *__restrict__ cursor,
                                                   int2 *__restrict__ list) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= ns) return;
    const int e = topo[strad_node[s]].z;
    const uint32_t q = atomicAdd(&cursor[(e - 1) / kChunk], 1u);
    list[q] = make_int2(s, e);
}

// ------------------------------------------------------------------- host --

static inline unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

// Builds the forest over the normalized points P (caller order); the cloud
// ranges are ctx->offsets (host) / ctx->d_offsets (device, already copied).
// Morton keys of the n caller-order points P (cloud index above the 45
// Morton bits when nclouds > 1) and a stable LSD sort, 9 bits per pass: on
// return ka holds the sorted keys and va the caller index of each.  An odd
// pass count leaves the result in the second buffer pair, which then becomes
// the first.  Uses ctx->hist and ctx->scan_tmp (sized here for n).
hipError_t morton_sort(wnnc_ctx_s *ctx, const float *P, int64_t n, int nclouds, int passes,
                       DevBuf<unsigned long long> &ka, DevBuf<unsigned long long> &kb,
                       DevBuf<uint32_t> &va, DevBuf<uint32_t> &vb) {
    hipStream_t st = ctx->stream;
    const int ntiles = rs_tiles(n);
    const int64_t hsize = (int64_t)kRsBins * (ntiles + 1);  // the digits' totals after the counts
    TRY(ka.ensure(n));
    TRY(kb.ensure(n));
    TRY(va.ensure(n));
    TRY(vb.ensure(n));
    TRY(ctx->hist.ensure(hsize));
    TRY(ctx->scan_tmp.ensure(scan_tmp_size(16 * (hsize > n + 1 ? hsize : n + 1) + 16)));
    hipLaunchKernelGGL(k_morton, dim3(blocks_for(n, 256)), dim3(256), 0, st, P, n,
                       ctx->d_offsets.p, nclouds, ka.p, va.p);
    unsigned long long *kin = ka.p, *kout = kb.p;
    uint32_t *vin = va.p, *vout = vb.p;
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = kRsBits * pass;
        uint32_t *hist = ctx->hist.p, *total = hist + (int64_t)kRsBins * ntiles;
        hipLaunchKernelGGL(k_rs_hist, dim3(ntiles), dim3(kRsThreads), 0, st, kin, n, shift, hist,
                           ntiles);
        hipLaunchKernelGGL(k_rs_scan, dim3(kRsBins * kWave / 256), dim3(256), 0, st, hist, ntiles,
                           total);
        hipLaunchKernelGGL(k_rs_scatter, dim3(ntiles), dim3(kRsThreads), 0, st, kin, vin, kout,
                           vout, n, shift, hist, total, ntiles);
        unsigned long long *tk = kin;
        kin = kout;
        kout = tk;
        uint32_t *tv = vin;
        vin = vout;
        vout = tv;
    }
    if (passes & 1) {
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    return hipGetLastError();
}

hipError_t build_tree(wnnc_ctx_s *ctx, const float *P) {
    const int64_t n = ctx->n;
    const int D = ctx->depth;
    const int nclouds = ctx->nclouds;
    hipStream_t st = ctx->stream;
    const int64_t nchunks = (n + kChunk - 1) / kChunk;
    const int ntiles = rs_tiles(n);
    const int64_t hsize = (int64_t)kRsBins * (ntiles + 1);  // the digits' totals after the counts
    int cloud_bits = 0;
    while ((1ll << cloud_bits) < nclouds) ++cloud_bits;
    const int passes = rs_passes(kMortonBits + cloud_bits);

    TRY(ctx->pts.ensure(n));
    TRY(ctx->perm.ensure(n));
    TRY(ctx->node_off.ensure(n + 1));
    TRY(ctx->keys_a.ensure(n));
    TRY(ctx->keys_b.ensure(n));
    TRY(ctx->vals_b.ensure(n));
    TRY(ctx->u32_tmp.ensure(n + 1));
    TRY(ctx->hist.ensure(hsize));
    TRY(ctx->tail_off.ensure(nchunks + 1));
    TRY(ctx->chunk_tot.ensure((int64_t)kMomSlots * nchunks));
    TRY(ctx->cloud_of.ensure(n));
    TRY(ctx->va.ensure(n));
    TRY(ctx->vb.ensure(n));
    TRY(ctx->vr.ensure(n));
    TRY(ctx->rho.ensure(n));
    TRY(ctx->scalars.ensure(nclouds));
    TRY(ctx->pair_ctr.ensure(kOpKinds));
    TRY(ctx->finite_flag.ensure(1));
    {
        int64_t big = hsize > n + 1 ? hsize : n + 1;
        TRY(ctx->scan_tmp.ensure(scan_tmp_size(16 * big + 16)));
    }

    TRY(morton_sort(ctx, P, n, nclouds, passes, ctx->keys_a, ctx->keys_b, ctx->perm,
                    ctx->vals_b));
    hipLaunchKernelGGL(k_point_cloud, dim3(blocks_for(n, 256)), dim3(256), 0, st, ctx->keys_a.p, n,
                       ctx->cloud_of.p);

    // nodes started per point -> pre-order offsets; M is read back once
    hipLaunchKernelGGL(k_count_nodes, dim3(blocks_for(n + 1, 256)), dim3(256), 0, st,
                       ctx->keys_a.p, n, D, ctx->leaf_cap, ctx->u32_tmp.p);
    TRY(exclusive_scan_u32(ctx->u32_tmp.p, ctx->node_off.p, n + 1, ctx->scan_tmp.p, st));
    // first node of every cloud (node_off at the cloud starts); the last
    // entry is M
    TRY(ctx->d_roots.ensure(nclouds + 1));
    hipLaunchKernelGGL(k_gather_roots, dim3((nclouds + 256) / 256), dim3(256), 0, st,
                       ctx->node_off.p, ctx->d_offsets.p, nclouds, ctx->d_roots.p);
    ctx->roots.resize(nclouds + 1);
    TRY(hipMemcpyAsync(ctx->roots.data(), ctx->d_roots.p, (size_t)(nclouds + 1) * sizeof(int32_t),
                       hipMemcpyDeviceToHost, st));
    TRY(hipStreamSynchronize(st));
    const int64_t m = ctx->roots[nclouds];
    if (m > kMaxNodes) return hipErrorNotSupported;  // beyond 32-bit record offsets
    ctx->m = m;

    TRY(ctx->topo.ensure(m));
    TRY(ctx->node_strad.ensure(m));
    TRY(ctx->mom.ensure(kRecStride * m));
    TRY(ctx->mnode.ensure(m));
    TRY(ctx->mflag.ensure(m + 1));
    TRY(ctx->mslot.ensure(m + 1));

    TRY(hipMemsetAsync(ctx->mflag.p, 0, (size_t)(m + 1) * sizeof(uint32_t), st));
    hipLaunchKernelGGL(k_emit_nodes, dim3(blocks_for(n, 256)), dim3(256), 0, st, ctx->keys_a.p,
                       n, D, ctx->leaf_cap, ctx->node_off.p, ctx->topo.p, ctx->mflag.p);
    hipLaunchKernelGGL(k_gather_points, dim3(blocks_for(n, 256)), dim3(256), 0, st, P,
                       ctx->perm.p, n, ctx->pts.p);
    TRY(ctx->cells.ensure(m));
    hipLaunchKernelGGL(k_node_cells, dim3(blocks_for(m, 256)), dim3(256), 0, st, ctx->topo.p,
                       ctx->keys_a.p, ctx->pts.p, m, ctx->cells.p, ctx->mom.p);
    TRY(ctx->wflag.ensure(m + 1));
    TRY(ctx->wslot.ensure(m + 1));
    TRY(hipMemsetAsync(ctx->wflag.p, 0, (size_t)(m + 1) * sizeof(uint32_t), st));
    hipLaunchKernelGGL(k_split_wide, dim3(blocks_for(m, 256)), dim3(256), 0, st, ctx->topo.p, m,
                       ctx->mflag.p, ctx->wflag.p);
    TRY(exclusive_scan_u32(ctx->mflag.p, ctx->mslot.p, m + 1, ctx->scan_tmp.p, st));
    TRY(exclusive_scan_u32(ctx->wflag.p, ctx->wslot.p, m + 1, ctx->scan_tmp.p, st));
    uint32_t nn32 = 0, nw32 = 0;
    TRY(hipMemcpyAsync(&nn32, ctx->mslot.p + m, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    TRY(hipMemcpyAsync(&nw32, ctx->wslot.p + m, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    TRY(hipStreamSynchronize(st));
    const int64_t ns = (int64_t)nn32 + nw32;
    ctx->n_strad = (int32_t)ns;
    ctx->n_wide = (int32_t)nw32;
    TRY(ctx->strad_node.ensure(ns + 1));
    TRY(ctx->strad_topo.ensure(ns + 1));
    TRY(ctx->tail_list.ensure(ns + 1));
    TRY(ctx->head.ensure((int64_t)kMomSlots * (ns + 1)));
    TRY(ctx->tail.ensure((int64_t)kMomSlots * (ns + 1)));
    hipLaunchKernelGGL(k_strad_compact, dim3(blocks_for(m, 256)), dim3(256), 0, st, ctx->mflag.p,
                       ctx->mslot.p, ctx->wflag.p, ctx->wslot.p, ctx->topo.p, m,
                       ctx->node_strad.p, ctx->strad_node.p, ctx->strad_topo.p, ctx->mnode.p);
    // chunk -> straddlers whose range ends inside it (CSR); counts reuse mflag
    uint32_t *tcnt = ctx->u32_tmp.p;  // n+1 >= chunks+1 entries
    TRY(hipMemsetAsync(tcnt, 0, (size_t)(nchunks + 1) * sizeof(uint32_t), st));
    if (ns > 0)
        hipLaunchKernelGGL(k_tail_count, dim3(blocks_for(ns, 256)), dim3(256), 0, st,
                           ctx->strad_node.p, ctx->topo.p, (int)ns, tcnt);
    TRY(exclusive_scan_u32(tcnt, ctx->tail_off.p, nchunks + 1, ctx->scan_tmp.p, st));
    uint32_t *cursor = ctx->mslot.p;  // free again: m+1 >= chunks+1 entries
    TRY(hipMemcpyAsync(cursor, ctx->tail_off.p, (size_t)(nchunks + 1) * sizeof(uint32_t),
                       hipMemcpyDeviceToDevice, st));
    if (ns > 0)
        hipLaunchKernelGGL(k_tail_fill, dim3(blocks_for(ns, 256)), dim3(256), 0, st,
                           ctx->strad_node.p, ctx->topo.p, (int)ns, cursor, ctx->tail_list.p);
    TRY(hipStreamSynchronize(st));
    TRY(hipMemsetAsync(ctx->pair_ctr.p, 0, kOpKinds * sizeof(unsigned long long), st));
    return hipGetLastError();
}

// The ancestors of each task's first node, from its cloud's root down: the
// nodes at which a part of a split walk re-evaluates its lanes' decisions
// (none for a walk that starts at the root).  At most one ancestor per
// depth and 8 children per node are examined, so the loops end.  A node's
// children are read from its record: one load per depth instead of one per
// child (17 us at 50k points, now less than 10).
__global__ __launch_bounds__(256) void k_task_chains(const int4 *__restrict__ tasks,
                                                     const int32_t *__restrict__ cloud,
                                                     const int32_t *__restrict__ roots,
                                                     const int4 *__restrict__ topo,
                                                     const float4 *__restrict__ mom, int ntasks,
                                                     int32_t *__restrict__ chain) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntasks) return;
    const int4 tk = tasks[t];
    const int nbeg = tk.z;
    int node = roots[cloud[tk.x]];
    int32_t *out = chain + (int64_t)t * kChainStride;
    int cnt = 0;
    for (int d = 0; d < kMaxDepth && node < nbeg; ++d) {
        out[1 + cnt++] = node;
        int ch = node + 1;  // the child whose subtree holds the first node
        const float4 *rec = mom + (int64_t)kRecStride * node;
        const int fl = __float_as_int(rec[0].w), nk = fl >> kRecKidShift;
        const float4 R3 = rec[3];
        if (fl & kRecWideKids) {
            for (int c = 0; c < 8; ++c) {
                const int sk = topo[ch].x;
                if (sk > nbeg) break;
                ch = sk;
            }
        } else {
            const uint32_t w[4] = {__float_as_uint(R3.x), __float_as_uint(R3.y),
                                   __float_as_uint(R3.z), __float_as_uint(R3.w)};
#pragma unroll
            for (int q = 1; q < 8; ++q) {
                const int kid = node + (int)((w[(q - 1) / 2] >> (16 * ((q - 1) & 1))) & 0xffffu);
                if (q < nk && kid <= nbeg) ch = kid;
            }
        }
        node = ch;
    }
    out[0] = cnt;
}

// ----------------------------------------------------------------- tasks --

// (first, last target; root, end node) of every group of `per` consecutive
// targets of one cloud: cloud c's groups are lo[c] .. lo[c+1]-1.
__global__ __launch_bounds__(256) void k_groups(const int32_t *__restrict__ lo,
                                                const int64_t *__restrict__ off,
                                                const int32_t *__restrict__ roots, int nclouds,
                                                int ngroups, int per, int4 *__restrict__ groups) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= ngroups) return;
    int a = 0, b = nclouds;  // lo[a] <= g < lo[b]
    while (b - a > 1) {
        const int mid = (a + b) >> 1;
        if (lo[mid] <= g)
            a = mid;
        else
            b = mid;
    }
    const int64_t first = off[a] + (int64_t)(g - lo[a]) * per, end = off[a + 1];
    groups[g] = make_int4((int)first, (int)(first + per < end ? first + per : end), roots[a],
                          roots[a + 1]);
}

// The plan of a group's walk: the nodes it visits are those whose parent some
// target opens.  One workgroup per group lists them breadth first, a node per
// thread (the distances from x_B of a constant attribute to the targets
// against Alg. 4's threshold, the boxes of kPlanPer targets first), and sorts
// them by index, which is the order of the walk.  Bound by the rounds of loads
// and LDS accesses, about a dozen, where a recording walk is a chain of up to
// 2,600 visits.  The list has to be exact: with the box of all 64 targets
// instead of the targets the A walk takes 132 instead of 74 us at 100k points,
// and with cell centres for x_B 341 instead of 332 us at 500k.
// The boxes are tested without a branch between them, and the sort shifts
// instead of dividing and meets a barrier only where pairs span wavefronts:
// 118 -> 80 us at 50k points, 207 -> 142 us at 164k.  The loops are unrolled
// little: with all of them in registers (119 instead of 35) a build of 3M
// points takes 4.9 instead of 3.5 ms.
constexpr int kPlanBlock = 256;
constexpr int kPlanPer = 8, kPlanBoxes = kWave / kPlanPer;

// A group's targets as a plan tests them (in LDS).
struct PlanTargets {
    float4 box[kPlanBoxes][2];  // lower corner, negated upper corner
    float4 tgt[kWave];
};

// Filled by the workgroup's first wavefront.
__device__ inline void plan_targets(PlanTargets &T, const int4 &G,
                                    const float4 *__restrict__ tpts, int lane) {
    // the group's last target in place of those it lacks
    const float4 p = tpts[min(G.x + lane, G.y - 1)];
    float v[6] = {p.x, p.y, p.z, -p.x, -p.y, -p.z};
    T.tgt[lane] = p;
#pragma unroll
    for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int d = 1; d < kPlanPer; d <<= 1) v[k] = fminf(v[k], __shfl_xor(v[k], d, kWave));
    if (lane % kPlanPer == 0) {
        T.box[lane / kPlanPer][0] = make_float4(v[0], v[1], v[2], 0.0f);
        T.box[lane / kPlanPer][1] = make_float4(v[3], v[4], v[5], 0.0f);
    }
}

// Whether some target does not accept the node at (x, y, z).
__device__ inline bool plan_opens(const PlanTargets &T, float x, float y, float z, float thr2) {
    unsigned near = 0u;
#pragma unroll 2
    for (int b = 0; b < kPlanBoxes; ++b) {
        const float4 bl = T.box[b][0], bh = T.box[b][1];
        const float dx = fmaxf(fmaxf(bl.x - x, x + bh.x), 0.f),
                    dy = fmaxf(fmaxf(bl.y - y, y + bh.y), 0.f),
                    dz = fmaxf(fmaxf(bl.z - z, z + bh.z), 0.f);
        near |= fmaf(dx, dx, fmaf(dy, dy, dz * dz)) > thr2 ? 0u : 1u << b;
    }
    bool open = false;
    while (near != 0u && !open) {
        const float4 *tb = T.tgt + kPlanPer * __builtin_ctz(near);
        near &= near - 1u;
#pragma unroll 4
        for (int t = 0; t < kPlanPer; ++t) {
            const float ex = tb[t].x - x, ey = tb[t].y - y, ez = tb[t].z - z;
            open |= fmaf(ex, ex, fmaf(ey, ey, ez * ez)) <= thr2;
        }
    }
    return open;
}

// The children of node nd (record words fl and R3), in order: see(q, kid).
template <class See>
__device__ inline void plan_kids(int nd, int fl, const float4 &R3, const int4 *__restrict__ topo,
                                 See &&see) {
    const int nk = fl >> kRecKidShift;
    const uint32_t w[4] = {__float_as_uint(R3.x), __float_as_uint(R3.y), __float_as_uint(R3.z),
                           __float_as_uint(R3.w)};
    int kid = nd + 1;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (q < nk) {
            if (q > 0)
                kid = (fl & kRecWideKids)
                          ? topo[kid].x
                          : nd + (int)((w[(q - 1) / 2] >> (16 * ((q - 1) & 1))) & 0xffffu);
            see(q, kid);
        }
    }
}

// Lists the nodes that the walk from `root` visits, a level per round: level
// by level until all are listed (returns -1; tail is their number) or a level
// does not fit into vis (returns the depth of the last level that did; *listed
// is the number of nodes down to it).  All threads of the workgroup call it.
__device__ inline int plan_list(const PlanTargets &T, int root, int *vis, int &tail,
                                const float4 *__restrict__ cells, const float4 *__restrict__ mom,
                                const int4 *__restrict__ topo, float c, int tid, int *listed) {
    if (tid == 0) {
        vis[0] = root;
        tail = 1;
    }
    int head = 0;
    for (int level = 0;; ++level) {
        __syncthreads();
        const int end = tail;
        __syncthreads();
        if (end > kPlanVisits) {
            *listed = head;
            return level - 1;
        }
        if (head >= end) break;
        for (int i = head + tid; i < end; i += kPlanBlock) {
            const int nd = vis[i];
            const float4 *rb = mom + (int64_t)kRecStride * nd;
            const float4 cb = cells[nd], R0 = rb[0], R3 = rb[3];
            if (cb.w < 0.0f) continue;  // a single-point leaf
            const int fl = __float_as_int(R0.w);
            const float thr2 = (c * cb.w) * (c * cb.w);
            if (!plan_opens(T, R0.x, R0.y, R0.z, thr2)) continue;
            const int nk = fl >> kRecKidShift;
            if (nk == 0) continue;  // a leaf
            const int o = atomicAdd(&tail, nk);
            plan_kids(nd, fl, R3, topo, [&](int q, int kid) {
                if (o + q < kPlanVisits) vis[o + q] = kid;
            });
        }
        head = end;
    }
    *listed = head;
    return -1;
}

// Bitonic sort of vis[0 .. n), padded to a power of two.
__device__ inline void plan_sort(int *vis, int n, int tid) {
    int m = 2;
    while (m < n) m <<= 1;
    for (int i = n + tid; i < m; i += kPlanBlock) vis[i] = INT32_MAX;
    __syncthreads();
    // (a wavefront's 64 pairs lie in 2 * 64 consecutive entries while their
    // distance j is at most 64: only the other steps need the whole block)
    for (int k = 2; k <= m; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int p = tid; p < m / 2; p += kPlanBlock) {
                const int lo = 2 * p - (p & (j - 1)), hi = lo + j;
                const int a = vis[lo], b = vis[hi];
                if ((a > b) == ((lo & k) == 0)) {
                    vis[lo] = b;
                    vis[hi] = a;
                }
            }
            if (j > kWave || (j == 1 && k > kWave)) {
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
    __syncthreads();
}

// Visits between two nodes that a plan holds: kPlanStep, doubled until a walk
// of n visits has no more than kPlanStride of them.
__device__ inline int plan_step(int n) {
    int step = kPlanStep;
    while ((int64_t)step * kPlanStride < n) step <<= 1;
    return step;
}

// sum[0] += the planned visits; a group of more than kPlanVisits is appended
// to `longs` instead (their number in sum[1]) and planned by k_plan_long.
__global__ __launch_bounds__(kPlanBlock) void k_plan(const int4 *__restrict__ groups,
                                                     const float4 *__restrict__ tpts,
                                                     const float4 *__restrict__ cells,
                                                     const float4 *__restrict__ mom,
                                                     const int4 *__restrict__ topo, float c,
                                                     int32_t *__restrict__ plan,
                                                     unsigned long long *__restrict__ sum,
                                                     int32_t *__restrict__ longs) {
    __shared__ int vis[kPlanVisits];
    __shared__ PlanTargets T;
    __shared__ int tail;
    const int tid = threadIdx.x;
    const int4 G = groups[blockIdx.x];
    if (tid < kWave) plan_targets(T, G, tpts, tid);
    int n;
    if (plan_list(T, G.z, vis, tail, cells, mom, topo, c, tid, &n) >= 0) {
        if (tid == 0) longs[atomicAdd(sum + 1, 1ull)] = (int32_t)blockIdx.x;
        return;
    }
    int32_t *out = plan + (int64_t)blockIdx.x * kPlanStride;
    plan_sort(vis, n, tid);
    for (int k = tid; k * kPlanStep < n; k += kPlanBlock) out[k] = k == 0 ? n : vis[k * kPlanStep];
    if (tid == 0) atomicAdd(sum, (unsigned long long)n);
}

// Plans of more than kPlanVisits visits (on a surface of 500k points those of
// some groups at c = 3, of nearly all at c = 5): the levels that fit are listed
// as in k_plan, and each node of the last one stands for all visits below it,
// which the workgroup counts with a stack of nodes in LDS, up to a node per
// thread at a time.  The plan is the listed node nearest to every plan_step-th
// visit.  (Finding the nodes between them as well, by a thread that walks below
// a listed one, makes no walk faster: A 1217 and 1202 us at 500k points and
// c = 4, the build 2750 and 2370 us.)  Bound by the rounds of the stack: loads,
// then three barriers.  Nodes at equal spacing over the cloud in place of this
// cut such walks very unevenly, as their visits are around their targets: the A
// walk took 388 us on a 100k-point sphere at c = 4, now 195; cutting up to visit
// 4,032 of a recorded walk and not beyond took 1555 us at 500k points and c = 4,
// now 1202 (the build 3280 and 2370 us; at c = 5 4340 and 3020).
constexpr int kPlanStack = 2048;  // a step leaves room for 8 entries per level below one node

__global__ __launch_bounds__(kPlanBlock) void k_plan_long(
    const int4 *__restrict__ groups, const float4 *__restrict__ tpts,
    const float4 *__restrict__ cells, const float4 *__restrict__ mom,
    const int4 *__restrict__ topo, float c, int32_t *__restrict__ plan,
    unsigned long long *__restrict__ sum, const int32_t *__restrict__ longs) {
    constexpr int kPer = kPlanVisits / kPlanBlock, kRoom = kPlanStack - 8 * kMaxDepth;
    __shared__ int vis[kPlanVisits], pos[kPlanVisits];
    __shared__ int stack[kPlanStack];
    __shared__ uint16_t owner[kPlanStack];  // the listed node above (kPlanVisits of them)
    __shared__ PlanTargets T;
    __shared__ int tail, sp, wsum[kPlanBlock / kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int g = longs[blockIdx.x];
    const int4 G = groups[g];
    if (tid < kWave) plan_targets(T, G, tpts, tid);
    int n;
    const int last = plan_list(T, G.z, vis, tail, cells, mom, topo, c, tid, &n);
    __syncthreads();
    plan_sort(vis, n, tid);
    // the visits of every listed node: its own, and of the last level those
    // below it
    for (int i = tid; i < kPlanVisits; i += kPlanBlock) pos[i] = i < n ? 1 : 0;
    if (tid == 0) sp = 0;
    int next = 0;  // the next listed node to look below
    for (;;) {
        __syncthreads();
        // nodes from the stack, then listed ones: never more than their
        // children fit; one at a time if need be, depth first
        const int s = sp;
        const int t = min(min(s, kPlanBlock), max(1, (kRoom - s) / 7));
        const int f = min(min(kPlanBlock - t, n - next), max(0, (kRoom - s - 7 * t) / 8));
        if (t + f == 0) break;
        int nd = -1, own = 0;
        if (tid < t) {
            nd = stack[s - 1 - tid];
            own = owner[s - 1 - tid];
        } else if (tid < t + f) {
            own = next + tid - t;
            nd = vis[own];
        }
        __syncthreads();
        if (tid == 0) sp = s - t;
        __syncthreads();
        if (nd >= 0) {
            const float4 *rb = mom + (int64_t)kRecStride * nd;
            const float4 R0 = rb[0], R3 = rb[3];
            const int fl = __float_as_int(R0.w), nk = fl >> kRecKidShift;
            const float cw = c * ldexpf(1.0f, 1 - (fl & 15));
            // (the children of a listed node above the last level are listed)
            if (nk > 0 && (fl & 15) >= last && plan_opens(T, R0.x, R0.y, R0.z, cw * cw)) {
                atomicAdd(&pos[own], nk);
                const int o = atomicAdd(&sp, nk);
                plan_kids(nd, fl, R3, topo, [&](int q, int kid) {
                    stack[o + q] = kid;
                    owner[o + q] = (uint16_t)own;
                });
            }
        }
        next += f;
    }
    __syncthreads();
    // the visits before every listed node: exclusive sums of the counts
    int own = 0;
    for (int k = 0; k < kPer; ++k) own += pos[tid * kPer + k];
    int inc = own;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(inc, d, kWave);
        inc += lane >= d ? o : 0;
    }
    if (lane == kWave - 1) wsum[wv] = inc;
    __syncthreads();
    int before = inc - own, total = 0;
    for (int w = 0; w < kPlanBlock / kWave; ++w) {
        before += w < wv ? wsum[w] : 0;
        total += wsum[w];
    }
    for (int k = 0; k < kPer; ++k) {
        const int w = pos[tid * kPer + k];
        pos[tid * kPer + k] = before;
        before += w;
    }
    __syncthreads();
    const int step = plan_step(total);
    int32_t *out = plan + (int64_t)g * kPlanStride;
    for (int i = tid; i < n; i += kPlanBlock) {
        const int v0 = pos[i], v1 = i + 1 < n ? pos[i + 1] : total;
        for (int q = max((v0 + step - 1) / step, 1); q * step < v1; ++q) {
            const bool up = i + 1 < n && q * step - v0 > v1 - q * step;  // nearer to the next
            out[q] = vis[up ? i + 1 : i];
        }
    }
    if (tid == 0) {
        out[0] = total;
        atomicAdd(sum, (unsigned long long)total);
    }
}

// The cuts of every group's walk into parts of at most about `split` visits
// (the first nodes of the parts after the first: nodes the plan reaches near
// equal numbers of visits, in walk order), and the number of its parts (0: a
// whole walk).  With step > 1, cuts are at multiples of step * kPlanStep visits
// only.
// One wavefront per group, a possible cut per lane: the plan is sorted, so a
// cut counts where its node is past the one before it.  (One thread per group
// was a chain of loads: 15 us at 50k points, now 3.)
__global__ __launch_bounds__(256) void k_cuts(const int4 *__restrict__ groups,
                                              const int32_t *__restrict__ plan, int ngroups,
                                              int split, int step, int32_t *__restrict__ cuts,
                                              uint32_t *__restrict__ nparts) {
    const int lane = threadIdx.x & (kWave - 1);
    const int g = blockIdx.x * (256 / kWave) + threadIdx.x / kWave;
    if (g >= ngroups) return;
    uint32_t cnt = 0;
    const int4 G = groups[g];
    const int32_t *pl = plan + (int64_t)g * kPlanStride;
    int32_t *out = cuts + (int64_t)g * kPlanStride;
    const int V = pl[0];
    const int ps = plan_step(V);
    const int per = max(kPlanStep * step / ps, 1);  // nodes of the plan from one possible cut
    const int visits = ps * per;                    // to the next, and the visits
    const int kmax = min((V - 1) / visits, kPlanStride / per - 1);
    const int P = min((V + split - 1) / split, kmax + 1);
    const auto node_at = [&](int q) {
        const int v = (int)((int64_t)V * q / P);
        return pl[per * min(max((v + visits / 2) / visits, 1), kmax)];
    };
    for (int q0 = 1; q0 < P; q0 += kWave) {
        const int q = q0 + lane;
        int nd = G.w, prev = G.z;
        if (q < P) {
            nd = node_at(q);
            if (q > 1) prev = max(prev, node_at(q - 1));
        }
        const bool cut = q < P && nd > prev && nd < G.w;
        const uint64_t m = __ballot(cut);
        if (cut) out[cnt + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = nd;
        cnt += (uint32_t)__popcll(m);
    }
    if (lane == 0) nparts[g] = cnt > 0 ? cnt + 1 : 0u;
}

// Exclusive sums over the groups of their parts and of the split groups, and
// the totals of both, by one workgroup.
constexpr int kPartScan = 1024;

__global__ __launch_bounds__(kPartScan) void k_part_scan(const uint32_t *__restrict__ nparts,
                                                         int n, uint32_t *__restrict__ part_off,
                                                         uint32_t *__restrict__ split_off,
                                                         uint32_t *__restrict__ count) {
    constexpr int kItems = 8, kWaves = kPartScan / kWave;
    __shared__ uint32_t wp[kWaves], ws[kWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    uint32_t cp = 0, cs = 0;
    for (int64_t base = 0; base < n; base += kPartScan * kItems) {
        uint32_t v[kItems], sp = 0, ss = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t i = base + (int64_t)tid * kItems + k;
            v[k] = i < n ? nparts[i] : 0u;
            sp += v[k];
            ss += v[k] ? 1u : 0u;
        }
        uint32_t ip = sp, is = ss;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t a = __shfl_up(ip, d, kWave), b = __shfl_up(is, d, kWave);
            if (lane >= d) ip += a, is += b;
        }
        if (lane == kWave - 1) wp[wv] = ip, ws[wv] = is;
        __syncthreads();
        uint32_t bp = cp, bs = cs;
        for (int w = 0; w < kWaves; ++w) {
            if (w < wv) bp += wp[w], bs += ws[w];
            cp += wp[w], cs += ws[w];
        }
        bp += ip - sp, bs += is - ss;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t i = base + (int64_t)tid * kItems + k;
            if (i < n) part_off[i] = bp, split_off[i] = bs;
            bp += v[k];
            bs += v[k] ? 1u : 0u;
        }
        __syncthreads();
    }
    if (tid == 0) count[0] = cp, count[1] = cs;
}

// The wavefront tasks of every group, in group order: group g's first task is
// the parts before it plus the whole walks before it (no nparts: all walks are
// whole).  One wavefront per group.
__global__ __launch_bounds__(256) void k_emit_tasks(
    const int4 *__restrict__ groups, const int32_t *__restrict__ cuts,
    const uint32_t *__restrict__ nparts, const uint32_t *__restrict__ part_off,
    const uint32_t *__restrict__ split_off, int ngroups, int4 *__restrict__ tasks,
    int32_t *__restrict__ slot, int4 *__restrict__ split_groups, int32_t *__restrict__ split_slot,
    int2 *__restrict__ gtab) {
    const int g = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kWave);
    const int lane = threadIdx.x & (kWave - 1);
    if (g >= ngroups) return;
    const int4 G = groups[g];
    const int P = nparts ? (int)nparts[g] : 0, po = nparts ? (int)part_off[g] : 0,
              so = nparts ? (int)split_off[g] : 0;
    const int t0 = po + (g - so);
    if (gtab && lane == 0) gtab[g] = P > 0 ? make_int2(po, po + P) : make_int2(0, 0);
    if (P == 0) {
        if (lane == 0) {
            tasks[t0] = G;
            slot[t0] = g;
        }
        return;
    }
    const int32_t *ct = cuts + (int64_t)g * kPlanStride;
    for (int q = lane; q < P; q += kWave) {
        tasks[t0 + q] = make_int4(G.x, G.y, q > 0 ? ct[q - 1] : G.z, q + 1 < P ? ct[q] : G.w);
        slot[t0 + q] = -1 - (po + q);
    }
    if (lane == 0) {
        split_groups[so] = make_int4(G.x, G.y, po, po + P);
        split_slot[so] = g;
    }
}

// Parts shorter than the split size where a cloud has too few of that size to
// fill the chip (8,192 wavefront slots), not below kPlanStep visits each.  A
// part's chain of visits is what a small cloud's walk takes; more of them add
// the visits of their ancestors.  Up to kOneRoundVisits visits per part, one
// round of wavefronts is best: just fewer parts than slots.  Longer parts leave
// slots idle behind the longest, and kFillParts of them even that out; so they
// do for leaves of several points (fewer nodes than points), whose visits
// differ.  An iteration (us) with parts of 256 visits / about 16,384 parts /
// one round: 254 / 174 / 154 at 20k points, 259 / 193 / 174 at 30k, 275 / 231 /
// 222 at 50k (parts of 94 visits), 303 / 272 / 289 at 70k (of 128), 354 / 343 /
// 352 at 100k, 429 / 172 / 189 at 20k with leaves of up to 8 points; a noisy 50k
// 259 with 16,384 parts, 238 with one round (of 117 visits); 2k points 229 with
// parts of 256 visits, 100 with parts of 16.
// Where kFillGroups whole walks nearly fill the slots by themselves (forests of
// small clouds), cutting them all only adds work, and the split size stands if
// it leaves most of them whole: G in forests of 8,192 x 64 / 4,096 x 128 /
// 3,072 x 128 points with the shorter parts 91 / 112 / 93 us, so 66 / 88 / 78 us.
// (Most walks cut in two take more rounds of wavefronts than either: 1,536 x 256
// points 119 us, with the shorter parts 109.)
constexpr unsigned long long kFillParts = 16384;
constexpr int64_t kFillGroups = 5120;
constexpr unsigned long long kOneRoundVisits = 120;
// Clouds that parts of kCoarseStep * kPlanStep visits (64) would fill are cut
// into parts of the split size at every kCoarseStep-th node of the plan: finer
// cuts balance them no better than 2 % (332 instead of 338 us at 500k points),
// and these keep the grouping, and so the bits, of the sums of large clouds
// independent of the plan's resolution.  Their sums are rounded to FP32, once
// per 64 visits or more.  All other parts keep FP64 sums: they also split walks
// that would otherwise be whole, whose sums meet FP32 only in the output.
constexpr int kCoarseStep = 4;

// How the current plan's walks are cut for a split size: parts of at most
// `visits` visits (0: not), at every step-th node of the plan.
struct CutRule {
    int visits, step;
};

// Groups of `per` consecutive targets of one cloud.
static int64_t group_count(const wnnc_ctx_s *ctx, int per) {
    int64_t g = 0;
    for (int c = 0; c < ctx->nclouds; ++c)
        g += (ctx->offsets[c + 1] - ctx->offsets[c] + per - 1) / per;
    return g;
}

static CutRule cut_rule(const wnnc_ctx_s *ctx, int tpl, int split) {
    if (split <= 0 || tpl != 1) return {0, 1};
    const unsigned long long fill = ctx->plan_visits / kFillParts;
    if (fill >= (unsigned long long)std::max(split, kPlanStep * kCoarseStep))
        return {split, kCoarseStep};
    const int64_t ng = group_count(ctx, kWave);
    if (ng >= kFillGroups && ctx->plan_visits <= (unsigned long long)ng * split) return {split, 1};
    unsigned long long visits = fill;
    if (ng < kFillGroups && ctx->m > ctx->n) {
        // (every group's last part is half full on average)
        const unsigned long long one = ctx->plan_visits / (kFillParts / 2 - ng / 2) + 1;
        if (one <= kOneRoundVisits) visits = one;
    }
    visits = std::max<unsigned long long>(visits, kPlanStep);
    return {(int)std::min<unsigned long long>(split, visits), 1};
}

// Wavefront tasks for tile shape tpl: each cloud's sorted targets cut into
// runs of 64 * tpl, in Morton order, cloud after cloud.
bool needs_plan(const wnnc_ctx_s *ctx, int tpl, int split) {
    return split > 0 && tpl == 1 && !ctx->plan_ok;
}

bool same_tasks(const wnnc_ctx_s *ctx, int tpl, int split_a, int split_b) {
    const CutRule a = cut_rule(ctx, tpl, split_a), b = cut_rule(ctx, tpl, split_b);
    return a.visits == b.visits && a.step == b.step;
}

hipError_t make_tasks(wnnc_ctx_s *ctx, int tpl, int split) {
    hipStream_t st = ctx->stream;
    // (no tasks until all of them are there)
    ctx->gtab_ok = false;
    ctx->ntasks = ctx->nparts = ctx->nsplit = ctx->ngroups = 0;
    const int per = kWave * tpl;
    // (kept: the copy may be under way when this returns)
    std::vector<int32_t> &lo = ctx->task_lo_host;
    lo.resize(ctx->nclouds + 1);
    int64_t g = 0;
    for (int c = 0; c < ctx->nclouds; ++c) {
        lo[c] = (int32_t)g;
        g += (ctx->offsets[c + 1] - ctx->offsets[c] + per - 1) / per;
    }
    lo[ctx->nclouds] = (int32_t)g;
    const int ng = (int)g;
    TRY(ctx->task_lo.ensure(ctx->nclouds + 1));
    TRY(ctx->groups.ensure(g));
    TRY(ctx->partial.ensure(3 * g));
    TRY(hipMemcpyAsync(ctx->task_lo.p, lo.data(), lo.size() * sizeof(int32_t),
                       hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_groups, dim3(blocks_for(g, 256)), dim3(256), 0, st, ctx->task_lo.p,
                       ctx->d_offsets.p, ctx->d_roots.p, ctx->nclouds, ng, per, ctx->groups.p);
    if (needs_plan(ctx, tpl, split)) {
        TRY(ctx->plan.ensure(g * kPlanStride));
        TRY(ctx->plan_sum.ensure(2));
        TRY(ctx->plan_longs.ensure(g));
        TRY(launch_zero_u64(ctx->plan_sum.p, 2, st));
        hipLaunchKernelGGL(k_plan, dim3((unsigned)ng), dim3(kPlanBlock), 0, st, ctx->groups.p,
                           ctx->pts.p, ctx->cells.p, ctx->mom.p, ctx->topo.p, ctx->c, ctx->plan.p,
                           ctx->plan_sum.p, ctx->plan_longs.p);
        unsigned long long sum[2];
        TRY(hipMemcpyAsync(sum, ctx->plan_sum.p, sizeof(sum), hipMemcpyDeviceToHost, st));
        TRY(hipStreamSynchronize(st));
        if (sum[1] > 0) {
            hipLaunchKernelGGL(k_plan_long, dim3((unsigned)sum[1]), dim3(kPlanBlock), 0, st,
                               ctx->groups.p, ctx->pts.p, ctx->cells.p, ctx->mom.p, ctx->topo.p,
                               ctx->c, ctx->plan.p, ctx->plan_sum.p, ctx->plan_longs.p);
            TRY(hipGetLastError());
            TRY(hipMemcpyAsync(sum, ctx->plan_sum.p, sizeof(sum), hipMemcpyDeviceToHost, st));
            TRY(hipStreamSynchronize(st));
        }
        ctx->plan_visits = sum[0];
        ctx->plan_ok = true;
    }
    const CutRule cut = cut_rule(ctx, tpl, split);
    const bool wide = cut.visits > 0 && cut.step == 1;
    uint32_t count[2] = {0, 0};  // parts, split groups
    if (cut.visits > 0) {
        TRY(ctx->cuts.ensure(g * kPlanStride));
        TRY(ctx->ncuts.ensure(g));
        TRY(ctx->part_off.ensure(g));
        TRY(ctx->split_off.ensure(g));
        TRY(ctx->part_count.ensure(2));
        hipLaunchKernelGGL(k_cuts, dim3(blocks_for(g, 256 / kWave)), dim3(256), 0, st,
                           ctx->groups.p, ctx->plan.p, ng, cut.visits, cut.step, ctx->cuts.p,
                           ctx->ncuts.p);
        hipLaunchKernelGGL(k_part_scan, dim3(1), dim3(kPartScan), 0, st, ctx->ncuts.p, ng,
                           ctx->part_off.p, ctx->split_off.p, ctx->part_count.p);
        TRY(hipMemcpyAsync(count, ctx->part_count.p, sizeof(count), hipMemcpyDeviceToHost, st));
        TRY(hipStreamSynchronize(st));
    }
    const uint32_t np = count[0], ns = count[1];
    const int64_t nt = (int64_t)np + (g - ns);
    // per group, its part range, when the groups are the 64-point blocks of
    // the sorted points (one group per wavefront, every cloud starting at a
    // multiple of 64): a moment pass can then combine the parts itself
    bool aligned = tpl == 1 && ns > 0;
    for (int c = 0; c < ctx->nclouds && aligned; ++c) aligned = ctx->offsets[c] % kWave == 0;
    if (aligned) TRY(ctx->gtab.ensure(g));
    TRY(ctx->tasks.ensure(nt));
    TRY(ctx->task_slot.ensure(nt));
    TRY(ctx->split_groups.ensure(ns > 0 ? ns : 1));
    TRY(ctx->split_slot.ensure(ns > 0 ? ns : 1));
    const int64_t nv = (int64_t)np * 3 * kWave;
    TRY(ctx->parts.ensure(std::max<int64_t>(wide ? nv : nv / 2, 1)));
    TRY(ctx->task_chain.ensure(nt * kChainStride));
    hipLaunchKernelGGL(k_emit_tasks, dim3(blocks_for(g * kWave, 256)), dim3(256), 0, st,
                       ctx->groups.p, ctx->cuts.p, ns > 0 ? ctx->ncuts.p : nullptr, ctx->part_off.p,
                       ctx->split_off.p, ng, ctx->tasks.p, ctx->task_slot.p, ctx->split_groups.p,
                       ctx->split_slot.p, aligned ? ctx->gtab.p : nullptr);
    hipLaunchKernelGGL(k_task_chains, dim3(blocks_for(nt, 256)), dim3(256), 0, st, ctx->tasks.p,
                       ctx->cloud_of.p, ctx->d_roots.p, ctx->topo.p, ctx->mom.p, (int)nt,
                       ctx->task_chain.p);
    TRY(hipGetLastError());
    ctx->gtab_ok = aligned;
    ctx->parts_wide = wide;
    ctx->ntasks = (int)nt;
    ctx->ngroups = ng;
    ctx->nparts = (int)np;
    ctx->nsplit = (int)ns;
    ctx->tpl = tpl;
    ctx->split = split;
    return hipSuccess;
}

hipError_t sort_queries(wnnc_ctx_s *ctx, const float *Q, int64_t M) {
    TRY(morton_sort(ctx, Q, M, 1, rs_passes(kMortonBits), ctx->qkeys_a, ctx->qkeys_b, ctx->qperm,
                    ctx->qvals_b));
    TRY(ctx->qpts.ensure(M));
    hipLaunchKernelGGL(k_gather_points, dim3(blocks_for(M, 256)), dim3(256), 0, ctx->stream, Q,
                       ctx->qperm.p, M, ctx->qpts.p);
    return hipGetLastError();
}

}  // namespace wnnc
