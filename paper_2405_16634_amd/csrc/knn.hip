// k = 16 nearest neighbours of every point within its cloud, on the octree,
// and the neighbourhood features of the learned warm start: the offsets to
// the 16 neighbours in increasing distance, divided by their RMS length.
//
// One wavefront per group of up to 64 Morton-consecutive points of one cloud,
// one point per lane.  Each lane keeps a candidate list in registers, sorted
// ascending, seeded with its Morton-order neighbours on both sides (a tight
// radius from the start).  The wavefront then searches the tree with a stack
// of nodes, 64 at a time, one per lane: a node goes on when its cell (built
// with the tree) is within the group's reach of the group's box, and when some
// lane's ball reaches it; the points of the leaves are offered to every lane.
// Ties are broken by sorted index, so the result does not depend on the order
// in which points are offered.
//
// What bounds it: instructions, and on clouds of very uneven density the
// longest search of one group.  A search that walked the nodes one by one, all
// lanes on the same node, with compare-and-select insertions, took 31,800
// vector instructions per wavefront and 836 us on a 164k-point sphere (VALU
// 89 % busy), 945 us on a 100k-point knot; keys and FP64 minima took that to
// 475 and 711 us, bound by the scalar unit and its loads, and nodes tested one
// per lane to 270 and 275 us (8,800 and 9,700 vector instructions per
// wavefront; VALU 86 and 58 % busy).
// Requires points inside [-1,1]^3 (normalized clouds).
#include <float.h>

#include "common.h"
#include "internal.h"

namespace wnnc {

constexpr int kK = 16;
constexpr int kSeedBatch = 8;  // seed points' loads in flight
constexpr int kHomePoints = 32;  // a search's first node holds at least so many points
// A search's stack of nodes.  A step leaves room for 8 entries per level, so
// that steps of one node, which go depth first, never overflow it.
constexpr int kKnnStack = 512;

// A candidate is one FP64 key: the squared distance's bits above the sorted
// index.  Distances are not negative, so the keys, read as doubles (finite
// ones: the upper half is a float's bits), order by distance and then index,
// and a list is kept with FP64 minima and maxima, which issue at the FP32
// rate.  The empty entry (FLT_MAX, index -1) is above every other; a NaN
// distance (of either sign) counts as an infinite one and is above it, so
// neither is ever taken.
__device__ inline double cand_key(float d, int j) {
    return __hiloint2double(__float_as_int(fminf(d, __builtin_huge_valf())), j);
}
__device__ inline float cand_d(double k) { return __int_as_float(__double2hiint(k)); }
__device__ inline int cand_j(double k) { return __double2loint(k); }

// Inserts key x into the sorted list (the last entry drops out), unless no
// lane has one: entry k becomes the smaller of itself and the larger of x and
// entry k - 1.  Two instructions per entry (compares and selects of distances
// and indices took about seven), written out with the branch around them:
// fmin and fmax quiet their operands first, and the list is copied where
// paths with and without an insertion meet.
__device__ inline void offer_if(double (&c)[kK], double x, uint64_t takers) {
    double s, t;
    static_assert(kK == 16, "the list below has 16 entries");
    // the sixteen entries are %0 .. %15
#define WNNC_PAIR(a, b, d)                  \
    "v_max_f64 %16, %" #b ", %18\n\t"       \
    "v_max_f64 %17, %" #d ", %18\n\t"       \
    "v_min_f64 %" #a ", %" #a ", %16\n\t"   \
    "v_min_f64 %" #b ", %" #b ", %17\n\t"
    asm("s_cmp_eq_u64 %19, 0\n\t"
        "s_cbranch_scc1 .Lskip%=\n\t"
        WNNC_PAIR(15, 14, 13) WNNC_PAIR(13, 12, 11) WNNC_PAIR(11, 10, 9)
        WNNC_PAIR(9, 8, 7) WNNC_PAIR(7, 6, 5) WNNC_PAIR(5, 4, 3)
        WNNC_PAIR(3, 2, 1)
        "v_max_f64 %16, %0, %18\n\t"
        "v_min_f64 %0, %0, %18\n\t"
        "v_min_f64 %1, %1, %16\n"
        ".Lskip%=:"
        : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]), "+v"(c[4]), "+v"(c[5]), "+v"(c[6]),
          "+v"(c[7]), "+v"(c[8]), "+v"(c[9]), "+v"(c[10]), "+v"(c[11]), "+v"(c[12]),
          "+v"(c[13]), "+v"(c[14]), "+v"(c[15]), "=&v"(s), "=&v"(t)
        : "v"(x), "s"(takers)
        : "scc");
#undef WNNC_PAIR
}

typedef int v4i_knn __attribute__((ext_vector_type(4)));
typedef float v4f_knn __attribute__((ext_vector_type(4)));

// Wave-uniform loads through the constant address space (scalar loads).
__device__ inline int4 knn_ld_i4(const int4 *p) {
    const v4i_knn v = *(const __attribute__((address_space(4))) v4i_knn *)p;
    return make_int4(v.x, v.y, v.z, v.w);
}
__device__ inline float4 knn_ld_f4(const float4 *p) {
    const v4f_knn v = *(const __attribute__((address_space(4))) v4f_knn *)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
// groups: per wavefront (first, last point; first, end node of the cloud),
// the 64-point groups of every cloud.
__device__ inline float lane_f(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Largest (MAX) or smallest value of the lanes.
template <bool MAX>
__device__ inline float wave_extreme(float v) {
#define WNNC_STEP(ctrl)                                                                     \
    {                                                                                       \
        const int b = __float_as_int(v);                                                    \
        const float o = __int_as_float(__builtin_amdgcn_update_dpp(b, b, ctrl, 0xf, 0xf, false)); \
        v = MAX ? fmaxf(v, o) : fminf(v, o);                                                \
    }
    WNNC_STEP(0x111) WNNC_STEP(0x112) WNNC_STEP(0x114) WNNC_STEP(0x118)  // row_shr 1 2 4 8
    WNNC_STEP(0x142) WNNC_STEP(0x143)                                    // row_bcast 15 31
#undef WNNC_STEP
    return lane_f(v, 63);
}

// Distance squared between the boxes [al, ah] and [bl, bh] along the axes,
// rounded as the distance of two points is: no larger than that of any two
// points in them.
__device__ inline float box_d2(float dx, float dy, float dz) {
    dx = fmaxf(dx, 0.0f), dy = fmaxf(dy, 0.0f), dz = fmaxf(dz, 0.0f);
    return fmaf(dx, dx, fmaf(dy, dy, dz * dz));
}

__global__ __launch_bounds__(kWave) void k_knn(const float4 *__restrict__ pts,
                                               const float4 *__restrict__ cells,
                                               const int4 *__restrict__ topo,
                                               const float4 *__restrict__ mom,
                                               const int4 *__restrict__ groups,
                                               const int64_t *__restrict__ off,
                                               const int32_t *__restrict__ cloud, int ngroups,
                                               int32_t *__restrict__ nbr,
                                               float *__restrict__ nd2) {
    __shared__ int stack[kKnnStack];
    const int g = blockIdx.x;
    if (g >= ngroups) return;
    const int lane = threadIdx.x;
    const int4 G = knn_ld_i4(groups + g);
    const int c = *(const __attribute__((address_space(4))) int *)(cloud + G.x);
    const int lo = (int)off[c], hi = (int)off[c + 1];
    const int t = G.x + lane;
    const bool valid = t < G.y;
    const float4 p = pts[min(t, G.y - 1)];
    const double none = cand_key(FLT_MAX, -1);
    // an idle lane's list takes nothing: no key is below 0
    double cd[kK];
#pragma unroll
    for (int k = 0; k < kK; ++k) cd[k] = valid ? none : 0.0;
    // seed with the kK Morton-order neighbours on each side (one side alone
    // fills the list, which bounds the radius also where the curve jumps);
    // the walk below skips them
    const int s_lo = max(lo, t - kK), s_hi = min(hi - 1, t + kK);
#pragma unroll 1
    for (int q0 = 0; q0 < 2 * kK; q0 += kSeedBatch) {
        float4 r[kSeedBatch];
#pragma unroll
        for (int u = 0; u < kSeedBatch; ++u) {
            const int q = q0 + u, j = t + (q < kK ? q - kK : q - kK + 1);
            r[u] = pts[min(max(j, lo), hi - 1)];
        }
#pragma unroll
        for (int u = 0; u < kSeedBatch; ++u) {
            const int q = q0 + u, j = t + (q < kK ? q - kK : q - kK + 1);
            const bool in = j >= s_lo && j <= s_hi;
            const float dx = r[u].x - p.x, dy = r[u].y - p.y, dz = r[u].z - p.z;
            offer_if(cd, in ? cand_key(fmaf(dx, dx, fmaf(dy, dy, dz * dz)), j) : none,
                     __ballot(in));
        }
    }
    // the group's box; the idle lanes repeat its last point
    const float glx = wave_extreme<false>(p.x), ghx = wave_extreme<true>(p.x);
    const float gly = wave_extreme<false>(p.y), ghy = wave_extreme<true>(p.y);
    const float glz = wave_extreme<false>(p.z), ghz = wave_extreme<true>(p.z);
    // A lane's bound: its last entry, or a distance within which some node has
    // more than kK points.  What is farther is not needed.
    float bound = cand_d(cd[kK - 1]), reach = wave_extreme<true>(bound);
    // Nearest first: the deepest node that holds the whole group and at least
    // kHomePoints points (its home), whose points give every lane a tight
    // radius; then, with that radius, the other children of the nodes above it.
    int home = G.z, sp = 0;
#pragma unroll 1
    for (int d = 0; d < kMaxDepth; ++d) {
        const int fl = knn_ld_i4((const int4 *)(mom + (int64_t)kRecStride * home)).w;
        const int nk = fl >> kRecKidShift;
        if (nk == 0) break;
        int kid = home + 1;
        if (fl & kRecWideKids) {
            for (int k = 1, ch = kid; k < nk; ++k) {
                ch = knn_ld_i4(topo + ch).x;
                if (lane == k) kid = ch;
            }
        } else if (lane > 0 && lane < nk) {
            kid = home + ((const uint16_t *)(mom + (int64_t)kRecStride * home + 3))[lane - 1];
        }
        const int4 tc = topo[kid];
        const uint64_t holds = __ballot(lane < nk && tc.y <= G.x && tc.z >= G.y &&
                                        tc.z - tc.y >= kHomePoints);
        if (holds == 0ull) break;
        const int at = __builtin_ctzll(holds);
        if (lane < nk && lane != at) stack[sp + lane - (lane > at ? 1 : 0)] = kid;
        sp += nk - 1;
        home = __builtin_amdgcn_readlane(kid, at);
    }
    if (lane == 0) stack[sp] = home;
    __syncthreads();
    int base = sp++;  // the home's subtree is searched before what lies below it
    // One step takes up to 64 nodes from the stack, one per lane: those whose
    // cells are within the reach of some box are opened: their children go to
    // the stack, or a leaf's points are offered to all lanes in turn.
#pragma unroll 1
    while (sp > 0) {
        base = sp > base ? base : 0;
        const int take_n = min(min(sp - base, kWave), max(1, (kKnnStack - 8 * kMaxDepth - sp) / 7));
        const bool on = lane < take_n;
        const int node = stack[sp - 1 - (on ? lane : 0)];
        sp -= take_n;
        __syncthreads();
        const int4 tp = topo[node];
        const float4 q = cells[node];
        const float4 *rec = mom + (int64_t)kRecStride * node;
        const int fl = __float_as_int(rec[0].w);
        const float4 R3 = rec[3];
        const bool single = q.w < 0.0f;
        const float h = single ? 0.0f : q.w;
        const float ux = q.x + h, uy = q.y + h, uz = q.z + h;
        const float d2 = box_d2(fmaxf(q.x - ghx, glx - ux), fmaxf(q.y - ghy, gly - uy),
                                fmaxf(q.z - ghz, glz - uz));
        const bool near = on && d2 <= reach;
        const bool leaf = (tp.w & kRecLeaf) != 0;
        // the points known to lie in the cell: points outside the tree's cube
        // and non-finite ones are in the cells along its faces
        const bool inner = fminf(fminf(q.x, q.y), q.z) > -1.0f &&
                           fmaxf(fmaxf(ux, uy), uz) < 1.0f;
        const int npts = inner ? tp.z - tp.y : 0;
        uint64_t offers = __ballot(near && leaf);
#pragma unroll 1
        while (offers) {
            const int s = __builtin_ctzll(offers);
            offers &= offers - 1ull;
            float x = lane_f(q.x, s), y = lane_f(q.y, s), z = lane_f(q.z, s);
            int j = __builtin_amdgcn_readlane(tp.y, s);
            const int je = __builtin_amdgcn_readlane(tp.z, s);
            if (lane_f(q.w, s) >= 0.0f) {
                const float4 r = knn_ld_f4(pts + j);
                x = r.x, y = r.y, z = r.z;
            }
            for (;;) {
                const float dx = x - p.x, dy = y - p.y, dz = z - p.z;
                const double key = cand_key(fmaf(dx, dx, fmaf(dy, dy, dz * dz)), j);
                // seeded (or the target itself) points were offered already
                const bool take =
                    ((uint32_t)(j - s_lo) > (uint32_t)(s_hi - s_lo)) & (key < cd[kK - 1]);
                offer_if(cd, take ? key : none, __ballot(take));
                if (++j >= je) break;
                const float4 r = knn_ld_f4(pts + j);
                x = r.x, y = r.y, z = r.z;
            }
        }
        bound = fminf(bound, cand_d(cd[kK - 1]));
        // of the other nodes, those that some lane's ball reaches
        uint64_t tests = __ballot(near && !leaf), open = tests;
#pragma unroll 1
        while (tests) {
            const int s = __builtin_ctzll(tests);
            tests &= tests - 1ull;
            const float x = lane_f(q.x, s), y = lane_f(q.y, s), z = lane_f(q.z, s);
            const float w = lane_f(q.w, s);
            const float lx = x - p.x, ly = y - p.y, lz = z - p.z;
            const float hx = p.x - (x + w), hy = p.y - (y + w), hz = p.z - (z + w);
            const float d = box_d2(fmaxf(lx, hx), fmaxf(ly, hy), fmaxf(lz, hz));
            if (__ballot(d <= bound) == 0ull) open &= ~(1ull << s);
            // the farthest corner: -min is the larger of the two extents
            const float f = box_d2(-fminf(lx, hx), -fminf(ly, hy), -fminf(lz, hz));
            const int np = __builtin_amdgcn_readlane(npts, s);
            bound = np > kK ? fminf(bound, f) : bound;
        }
        reach = wave_extreme<true>(bound);
        // the opened nodes' children, at the ranks of their counts' prefix sums
        const int nk = ((open >> lane) & 1ull) != 0ull ? fl >> kRecKidShift : 0;
        int at = sp;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint64_t m = __ballot((nk >> b) & 1);
            at += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))
                  << b;
            sp += __popcll(m) << b;
        }
        const uint32_t w[4] = {__float_as_uint(R3.x), __float_as_uint(R3.y), __float_as_uint(R3.z),
                               __float_as_uint(R3.w)};
        if (nk > 0) stack[at] = node + 1;
#pragma unroll
        for (int k = 1; k < 8; ++k)
            if (k < nk)
                stack[at + k] =
                    node + (int)((w[(k - 1) / 2] >> (16 * ((k - 1) & 1))) & 0xffffu);
        if (nk > 0 && (fl & kRecWideKids)) {
            int kid = node + 1;
            for (int k = 1; k < nk; ++k) {
                kid = topo[kid].x;
                stack[at + k] = kid;
            }
        }
        __syncthreads();
    }
    if (valid) {
#pragma unroll
        for (int k = 0; k < kK; ++k) {
            nbr[(int64_t)t * kK + k] = cand_j(cd[k]);
            nd2[(int64_t)t * kK + k] = cand_d(cd[k]);
        }
    }
}

// Features of sorted point t, written at its caller row: offsets to the 16
// neighbours (nearest first) divided by their RMS length; missing neighbours
// (clouds of fewer than 17 points) and zero RMS give zeros.  Optionally the
// neighbours' caller indices.
__global__ __launch_bounds__(256) void k_features(const float4 *__restrict__ pts,
                                                  const uint32_t *__restrict__ perm,
                                                  const int32_t *__restrict__ nbr, int n,
                                                  float *__restrict__ feat,
                                                  int32_t *__restrict__ nbr_caller) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const float4 p = pts[t];
    float o[3 * kK];
    double s2 = 0.0;
    int cnt = 0;
#pragma unroll
    for (int k = 0; k < kK; ++k) {
        const int j = nbr[(int64_t)t * kK + k];
        float ox = 0.f, oy = 0.f, oz = 0.f;
        if (j >= 0) {
            const float4 q = pts[j];
            ox = q.x - p.x, oy = q.y - p.y, oz = q.z - p.z;
            s2 += (double)ox * ox + (double)oy * oy + (double)oz * oz;
            ++cnt;
        }
        o[3 * k] = ox, o[3 * k + 1] = oy, o[3 * k + 2] = oz;
    }
    const double rms = cnt > 0 ? sqrt(s2 / cnt) : 0.0;
    const float inv = rms > 0.0 ? (float)(1.0 / rms) : 0.0f;
    const int64_t row = perm[t];
#pragma unroll
    for (int k = 0; k < 3 * kK; ++k) feat[row * (3 * kK) + k] = o[k] * inv;
    if (nbr_caller) {
#pragma unroll
        for (int k = 0; k < kK; ++k) {
            const int j = nbr[(int64_t)t * kK + k];
            nbr_caller[row * kK + k] = j >= 0 ? (int32_t)perm[j] : -1;
        }
    }
}

// Neighbour-search groups: runs of sorted points inside one octree cell of
// one depth (so of one cloud), cut every 64 points.  A wavefront walks the
// union of its lanes' search balls; capping the cell keeps that union small
// where points are sparse (64 Morton-consecutive isolated points can span
// much of the cloud's box), at the price of partly filled wavefronts there.
// The depth is the deepest whose cells hold kKnnMean points on average.  Areas
// of a 164k-point sphere / a 100k / a 500k-point knot: 412 / 413 / 1578 us with
// 10, 342 / 431 / 2017 us with 14 or 20 (one level up: longer searches where
// the knot is sparse); the largest cells of at most 64 points, whatever their
// depth: 397 / 723 / 2066 us.
constexpr int kKnnMean = 10;

// count[d] += the sorted points that share less than d octal digits with the
// point before them (the runs of depth d), d = 0 .. kMaxDepth.
__global__ __launch_bounds__(256) void k_knn_depths(const unsigned long long *__restrict__ keys,
                                                    int n, uint32_t *__restrict__ count) {
    __shared__ uint32_t h[kMaxDepth + 1];
    if (threadIdx.x <= kMaxDepth) h[threadIdx.x] = 0u;
    __syncthreads();
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) {
        const unsigned long long x = i > 0 ? keys[i] ^ keys[i - 1] : ~0ull;
        // the first depth at which the two points part
        int d = kMaxDepth + 1;
        if (x >> kMortonBits) d = 0;
        else if (x) d = (__clzll(x) - (64 - kMortonBits)) / 3 + 1;
        if (d <= kMaxDepth) atomicAdd(&h[d], 1u);
    }
    __syncthreads();
    if (threadIdx.x <= kMaxDepth && h[threadIdx.x]) atomicAdd(count + threadIdx.x, h[threadIdx.x]);
}

__global__ __launch_bounds__(256) void k_knn_brk(const unsigned long long *__restrict__ keys,
                                                 const uint32_t *__restrict__ count, int n,
                                                 uint32_t *__restrict__ brk) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    int depth = 0;
    uint32_t runs = count[0];
    for (int d = 1; d <= kMaxDepth; ++d) {
        runs += count[d];
        if ((int64_t)runs * kKnnMean > n) break;
        depth = d;
    }
    const int sh = 3 * (kMaxDepth - depth);  // the cloud index sits above the key
    brk[i] = (i == 0 || (keys[i] >> sh) != (keys[i - 1] >> sh)) ? 1u : 0u;
}

// run starts: runs[r] = first point of run r (rx = exclusive scan of brk)
__global__ __launch_bounds__(256) void k_knn_runs(const uint32_t *__restrict__ brk,
                                                  const uint32_t *__restrict__ rx, int n,
                                                  uint32_t *__restrict__ runs) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n && brk[i]) runs[rx[i]] = (uint32_t)i;
}

// group starts: every 64th point of its run
__global__ __launch_bounds__(256) void k_knn_gflag(const uint32_t *__restrict__ brk,
                                                   const uint32_t *__restrict__ rx,
                                                   const uint32_t *__restrict__ runs, int n,
                                                   uint32_t *__restrict__ gs) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t r = rx[i] + brk[i] - 1u;
    gs[i] = ((i - (int)runs[r]) & (kWave - 1)) == 0 ? 1u : 0u;
}

__global__ __launch_bounds__(256) void k_knn_groups(const uint32_t *__restrict__ brk,
                                                    const uint32_t *__restrict__ rx,
                                                    const uint32_t *__restrict__ runs,
                                                    const uint32_t *__restrict__ gs,
                                                    const uint32_t *__restrict__ gx, int n,
                                                    const int32_t *__restrict__ cloud,
                                                    const int32_t *__restrict__ roots,
                                                    int4 *__restrict__ groups,
                                                    uint32_t *__restrict__ count) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    if (i == n - 1) {
        count[0] = gx[i] + gs[i];
    }
    if (!gs[i]) return;
    const uint32_t r = rx[i] + brk[i] - 1u;
    const uint32_t nruns = rx[n - 1] + brk[n - 1];
    const int run_end = r + 1u < nruns ? (int)runs[r + 1] : n;
    const int c = cloud[i];
    groups[gx[i]] = make_int4(i, min(i + kWave, run_end), roots[c], roots[c + 1]);
}

static hipError_t knn_groups(wnnc_ctx_s *ctx) {
    const int n = (int)ctx->n;
    hipStream_t st = ctx->stream;
    static_assert((kMaxDepth + 1) % 2 == 0, "the depth counts are cleared in pairs");
    hipError_t e = ctx->knn_tmp.ensure(5 * (int64_t)n + 1);
    if (e != hipSuccess) return e;
    if ((e = ctx->knn_depths.ensure((kMaxDepth + 1) / 2)) != hipSuccess) return e;
    uint32_t *brk = ctx->knn_tmp.p, *rx = brk + n, *runs = rx + n, *gs = runs + n, *gx = gs + n;
    uint32_t *cnt = gx + n, *depths = (uint32_t *)ctx->knn_depths.p;
    const unsigned nb = (unsigned)((n + 255) / 256);
    if ((e = launch_zero_u64(ctx->knn_depths.p, (kMaxDepth + 1) / 2, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_knn_depths, dim3(nb), dim3(256), 0, st, ctx->keys_a.p, n, depths);
    hipLaunchKernelGGL(k_knn_brk, dim3(nb), dim3(256), 0, st, ctx->keys_a.p, depths, n, brk);
    if ((e = exclusive_scan_u32(brk, rx, n, ctx->scan_tmp.p, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_knn_runs, dim3(nb), dim3(256), 0, st, brk, rx, n, runs);
    hipLaunchKernelGGL(k_knn_gflag, dim3(nb), dim3(256), 0, st, brk, rx, runs, n, gs);
    if ((e = exclusive_scan_u32(gs, gx, n, ctx->scan_tmp.p, st)) != hipSuccess) return e;
    // at most one group per point
    if ((e = ctx->knn_groups.ensure(n)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_knn_groups, dim3(nb), dim3(256), 0, st, brk, rx, runs, gs, gx, n,
                       ctx->cloud_of.p, ctx->d_roots.p, ctx->knn_groups.p, cnt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    uint32_t ng = 0;
    if ((e = hipMemcpyAsync(&ng, cnt, sizeof(ng), hipMemcpyDeviceToHost, st)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    ctx->knn_ngroups = (int)ng;
    return hipSuccess;
}

hipError_t launch_knn(wnnc_ctx_s *ctx) {
    const int n = (int)ctx->n;
    hipError_t e = ctx->knn_idx.ensure((int64_t)n * kK);
    if (e != hipSuccess) return e;
    e = ctx->knn_d2.ensure((int64_t)n * kK);
    if (e != hipSuccess) return e;
    if (ctx->knn_ngroups == 0 && (e = knn_groups(ctx)) != hipSuccess) return e;
    if (ctx->knn_ngroups > 0)
        hipLaunchKernelGGL(k_knn, dim3((unsigned)ctx->knn_ngroups), dim3(kWave), 0, ctx->stream,
                           ctx->pts.p, ctx->cells.p, ctx->topo.p, ctx->mom.p,
                           ctx->knn_groups.p, ctx->d_offsets.p, ctx->cloud_of.p, ctx->knn_ngroups, ctx->knn_idx.p,
                           ctx->knn_d2.p);
    return hipGetLastError();
}

hipError_t launch_knn_features(wnnc_ctx_s *ctx, float *feat, int32_t *nbr_caller) {
    const int n = (int)ctx->n;
    hipError_t e = launch_knn(ctx);
    if (e != hipSuccess) return e;
    const unsigned nb = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_features, dim3(nb), dim3(256), 0, ctx->stream, ctx->pts.p, ctx->perm.p,
                       ctx->knn_idx.p, n, feat, nbr_caller);
    return hipGetLastError();
}

}  // namespace wnnc
