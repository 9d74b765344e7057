// Adjacency from a bare triangle list, on the device.
//
// What the smoothing pass takes as input -- the node->triangle and
// node->neighbour CSR and the boundary mask -- built the way the paper
// describes it (Sec. 3.3.2 finding of neighbours, Sec. 3.3.3 determining of
// constraints):
//   * a node's incident triangles are listed in index order;
//   * its neighbours are the other two vertices of those triangles, taken
//     triangle by triangle in index order and, inside a triangle, in stored
//     order (a triangle (v1,v2,v3) gives v1 the pair v2,v3; v2 the pair
//     v1,v3; v3 the pair v1,v2), each kept once where it first appears;
//   * a node is interior iff every neighbour was seen exactly twice (each
//     edge at the node lies in two triangles).
// Steps: the (node, triangle) incidences are binned by node range -- a
// histogram per work-group, a scan, a scatter -- and each bin is counted and
// placed by one work-group with its counters in LDS, which gives tri_ptr and
// the (unordered) rows of tri_idx; then one work-item per node sorts its
// incidences, deduplicates its neighbours in LDS and leaves row, degree and
// boundary flag; a scan of the degrees and one pass that writes the caller's
// arrays.
#include <algorithm>
#include <cstring>
#include <string>

#include "sl_common.h"
#include "sl_flow.h"

namespace sl {

namespace {

constexpr int kAB = 256;

constexpr uint32_t kAdjRange = 1u, kAdjRepeat = 2u;   // error bits

__device__ __forceinline__ uint32_t check_tri(int32_t a, int32_t b, int32_t c, int32_t n)
{
    if (a < 0 || b < 0 || c < 0 || a >= n || b >= n || c >= n) return kAdjRange;
    return a == b || b == c || a == c ? kAdjRepeat : 0u;
}

// ---- binning.  One device-wide counter per node (an atomic per incidence
// to count, another to place) ran at 21-26 G incidences/s on a shuffled
// million-node mesh: 520 us.  Through bins of consecutive nodes the random
// atomics stay in LDS and memory sees streams.

// Histogram of this work-group's triangles over the bins; checks the
// triangles.  hist[bin * groups + group].
__global__ __launch_bounds__(kAB) void k_adj_hist(const int32_t* __restrict__ tris, int32_t n_tris, int32_t n, int shift,
                                                  int bins, int32_t per, int32_t* __restrict__ hist,
                                                  uint32_t* __restrict__ err)
{
    extern __shared__ int32_t s_bin[];
    for (int q = threadIdx.x; q < bins; q += kAB) s_bin[q] = 0;
    __syncthreads();
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * per, t1 = min(t0 + per, static_cast<int64_t>(n_tris));
    uint32_t e = 0;
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kAB) {
        const int32_t a = tris[3 * t], b = tris[3 * t + 1], c = tris[3 * t + 2];
        const uint32_t f = check_tri(a, b, c, n);
        e |= f;
        if (f & kAdjRange) continue;
        atomicAdd(&s_bin[a >> shift], 1);
        atomicAdd(&s_bin[b >> shift], 1);
        atomicAdd(&s_bin[c >> shift], 1);
    }
    if (e) atomicOr(err, e);
    __syncthreads();
    for (int q = threadIdx.x; q < bins; q += kAB) hist[static_cast<int64_t>(q) * gridDim.x + blockIdx.x] = s_bin[q];
}

// The same triangles' incidences to their bins, as node-in-bin << 32 | triangle.
__global__ __launch_bounds__(kAB) void k_adj_scatter(const int32_t* __restrict__ tris, int32_t n_tris, int shift, int bins,
                                                     int32_t per, const int32_t* __restrict__ offs,
                                                     uint64_t* __restrict__ pairs, const uint32_t* __restrict__ err)
{
    extern __shared__ int32_t s_bin[];
    if (*err) return;
    for (int q = threadIdx.x; q < bins; q += kAB) s_bin[q] = offs[static_cast<int64_t>(q) * gridDim.x + blockIdx.x];
    __syncthreads();
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * per, t1 = min(t0 + per, static_cast<int64_t>(n_tris));
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kAB)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int32_t v = tris[3 * t + k], bin = v >> shift;
            pairs[atomicAdd(&s_bin[bin], 1)] =
                (static_cast<uint64_t>(v - (bin << shift)) << 32) | static_cast<uint32_t>(t);
        }
}

// One work-group per bin: counts per node in LDS, their scan (tri_ptr), and
// the triangles placed in their node's row, in no order.
constexpr int kBinBS = 512;
__global__ __launch_bounds__(kBinBS) void k_adj_bins(const uint64_t* __restrict__ pairs, const int32_t* __restrict__ offs,
                                                     int groups, int shift, int32_t n, int32_t* __restrict__ tri_ptr,
                                                     int32_t* __restrict__ tri_idx, const uint32_t* __restrict__ err)
{
    extern __shared__ int32_t s_cnt[];
    __shared__ int32_t s_wave[kBinBS / 64];
    if (*err) return;
    const int32_t v0 = static_cast<int32_t>(blockIdx.x) << shift, nv = min(1 << shift, n - v0);
    const int32_t b = offs[static_cast<int64_t>(blockIdx.x) * groups], e = offs[static_cast<int64_t>(blockIdx.x + 1) * groups];
    for (int q = threadIdx.x; q < nv; q += kBinBS) s_cnt[q] = 0;
    __syncthreads();
    for (int32_t k = b + threadIdx.x; k < e; k += kBinBS) atomicAdd(&s_cnt[static_cast<int32_t>(pairs[k] >> 32)], 1);
    __syncthreads();
    // exclusive scan of the counts, a contiguous segment per work-item
    const int per = (nv + kBinBS - 1) / kBinBS;
    const int q0 = min(static_cast<int>(threadIdx.x) * per, nv), q1 = min(q0 + per, nv);
    int32_t sum = 0;
    for (int q = q0; q < q1; ++q) sum += s_cnt[q];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int32_t x = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t t = __shfl_up(x, off);
        if (lane >= off) x += t;
    }
    if (lane == 63) s_wave[wv] = x;
    __syncthreads();
    int32_t run = b + x - sum;
    for (int w = 0; w < wv; ++w) run += s_wave[w];
    for (int q = q0; q < q1; ++q) {
        const int32_t c = s_cnt[q];
        s_cnt[q] = run;
        tri_ptr[v0 + q] = run;
        run += c;
    }
    if (v0 + nv == n && threadIdx.x == 0) tri_ptr[n] = e;
    __syncthreads();
    for (int32_t k = b + threadIdx.x; k < e; k += kBinBS) {
        const uint64_t w = pairs[k];
        tri_idx[atomicAdd(&s_cnt[static_cast<int32_t>(w >> 32)], 1)] = static_cast<int32_t>(static_cast<uint32_t>(w));
    }
}

// ---- beyond the bins' range (more than kBinNodes nodes): device-wide counters

__global__ __launch_bounds__(kAB) void k_adj_count(const int32_t* __restrict__ tris, int32_t n_tris, int32_t n,
                                                   int32_t* __restrict__ cnt, uint32_t* __restrict__ err)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * kAB + threadIdx.x;
    if (t >= n_tris) return;
    const int32_t a = tris[3 * t], b = tris[3 * t + 1], c = tris[3 * t + 2];
    const uint32_t f = check_tri(a, b, c, n);
    if (f) atomicOr(err, f);
    if (f & kAdjRange) return;
    atomicAdd(cnt + a, 1);
    atomicAdd(cnt + b, 1);
    atomicAdd(cnt + c, 1);
}

__global__ __launch_bounds__(kAB) void k_adj_fill(const int32_t* __restrict__ tris, int64_t m3,
                                                  const int32_t* __restrict__ tri_ptr, int32_t* __restrict__ cursor,
                                                  int32_t* __restrict__ tri_idx, const uint32_t* __restrict__ err)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kAB + threadIdx.x;
    if (*err || k >= m3) return;
    const int32_t v = tris[k];
    tri_idx[tri_ptr[v] + atomicAdd(cursor + v, 1)] = static_cast<int32_t>(k / 3);
}

__global__ __launch_bounds__(kAB) void k_adj_zero(int32_t* p, int64_t n)
{
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * kAB + threadIdx.x; k < n; k += static_cast<int64_t>(gridDim.x) * kAB)
        p[k] = 0;
}

// ---- rows

constexpr int kAdjInc = 16;   // incidences of a node handled in registers and LDS

// One node's incidences (1 <= c <= R of them) from registers: sorted by rank
// into tri_idx (when asked for), the two other vertices of each triangle to
// the node's LDS column in sorted order.  (The slots past c read triangle 0.)
template <int R>
__device__ __forceinline__ void adj_gather(int32_t v, int c, int32_t* __restrict__ row, const int32_t* __restrict__ tris,
                                           int32_t (*cand)[kAB], bool sorted)
{
    int32_t t[R];
#pragma unroll
    for (int q = 0; q < R; ++q) t[q] = q < c ? row[q] : INT32_MAX;
    int32_t a[R][3];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int k = 0; k < 3; ++k) a[q][k] = tris[q < c ? 3 * static_cast<int64_t>(t[q]) + k : 0];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (q >= c) continue;
        int rank = 0;   // (a node is in a triangle at most once: no two are equal)
#pragma unroll
        for (int k = 0; k < R; ++k) rank += t[k] < t[q];
        cand[2 * rank][threadIdx.x] = a[q][0] == v ? a[q][1] : a[q][0];
        cand[2 * rank + 1][threadIdx.x] = a[q][2] == v ? a[q][1] : a[q][2];
        if (sorted) row[rank] = t[q];
    }
}

// One node: its incidences sorted, its distinct neighbours in order of first
// appearance (into the scratch row at 2*tri_ptr[v]), their count and the
// boundary flag.  Without `rows` only the count.  Nodes in more than kAdjInc
// triangles work in the scratch rows in memory.
template <bool ROWS>
__global__ __launch_bounds__(kAB) void k_adj_rows(int32_t n, const int32_t* __restrict__ tris,
                                                  const int32_t* __restrict__ tri_ptr, int32_t* __restrict__ tri_idx,
                                                  int32_t* __restrict__ row, uint8_t* __restrict__ seen,
                                                  int32_t* __restrict__ deg, uint8_t* __restrict__ boundary,
                                                  const uint32_t* __restrict__ err)
{
    __shared__ int32_t cand[2 * kAdjInc][kAB];
    __shared__ uint8_t times[2 * kAdjInc][kAB];
    const int32_t v = static_cast<int32_t>(blockIdx.x) * kAB + threadIdx.x;
    if (v >= n || *err) return;
    const int32_t b = tri_ptr[v], c = tri_ptr[v + 1] - b;
    const int tid = threadIdx.x;
    int32_t L = 0;
    bool interior = c > 0;
    if (c <= kAdjInc) {
        // (a node in no triangle reads none: there may be no triangle at all)
        if (c > 8) adj_gather<kAdjInc>(v, c, tri_idx + b, tris, cand, ROWS);
        else if (c > 0) adj_gather<8>(v, c, tri_idx + b, tris, cand, ROWS);
        for (int k = 0; k < 2 * c; ++k) {
            const int32_t u = cand[k][tid];
            int q = 0;
            while (q < L && cand[q][tid] != u) ++q;
            if (q == L) {   // (the list never outruns the candidates it replaces)
                cand[L][tid] = u;
                times[L][tid] = 1;
                ++L;
            } else if (times[q][tid] < 255) {
                ++times[q][tid];
            }
        }
        for (int k = 0; k < L; ++k) {
            interior = interior && times[k][tid] == 2;
            if (ROWS) row[2 * static_cast<int64_t>(b) + k] = cand[k][tid];
        }
    } else {
        int32_t* const ti = tri_idx + b;
        for (int32_t i = 1; i < c; ++i) {   // insertion sort
            const int32_t x = ti[i];
            int32_t j = i - 1;
            while (j >= 0 && ti[j] > x) {
                ti[j + 1] = ti[j];
                --j;
            }
            ti[j + 1] = x;
        }
        int32_t* const r = row + 2 * static_cast<int64_t>(b);
        uint8_t* const s = seen + 2 * static_cast<int64_t>(b);
        for (int32_t q = 0; q < c; ++q) {
            const int64_t t = ti[q];
            const int32_t a0 = tris[3 * t], a1 = tris[3 * t + 1], a2 = tris[3 * t + 2];
            for (int h = 0; h < 2; ++h) {
                const int32_t u = h == 0 ? (a0 == v ? a1 : a0) : (a2 == v ? a1 : a2);
                int32_t k = 0;
                while (k < L && r[k] != u) ++k;
                if (k == L) {
                    r[L] = u;
                    s[L] = 1;
                    ++L;
                } else if (s[k] < 255) {
                    s[k] = static_cast<uint8_t>(s[k] + 1);
                }
            }
        }
        for (int32_t k = 0; k < L; ++k) interior = interior && s[k] == 2;
    }
    deg[v] = L;
    if (ROWS) boundary[v] = interior ? 0 : 1;
}

// Error bits and nbr_ptr[n] to pinned memory.
__global__ void k_adj_tell(const uint32_t* __restrict__ err, const int32_t* __restrict__ total, int32_t* __restrict__ out)
{
    out[0] = static_cast<int32_t>(*err);
    out[1] = *total;
}

// The results to their arrays: one work-item per node writes its row, then
// the offsets, flags and sorted incidences.
struct AdjOut {
    int32_t *nbr_ptr, *nbr_idx, *tri_ptr, *tri_idx;
    uint8_t* boundary;
};
__global__ __launch_bounds__(kAB) void k_adj_out(int32_t n, int64_t m3, const int32_t* __restrict__ tri_ptr,
                                                 const int32_t* __restrict__ tri_idx, const int32_t* __restrict__ row,
                                                 const int32_t* __restrict__ nbr_ptr, const uint8_t* __restrict__ boundary,
                                                 AdjOut o)
{
    const int64_t g = static_cast<int64_t>(blockIdx.x) * kAB + threadIdx.x, stride = static_cast<int64_t>(gridDim.x) * kAB;
    for (int64_t v = g; v < n; v += stride) {
        const int32_t tb = tri_ptr[v], b = nbr_ptr[v], L = nbr_ptr[v + 1] - b;
        const int32_t* const r = row + 2 * static_cast<int64_t>(tb);
        for (int32_t k = 0; k < L; ++k) o.nbr_idx[b + k] = r[k];
        o.nbr_ptr[v] = b;
        o.tri_ptr[v] = tb;
        o.boundary[v] = boundary[v];
        if (v == n - 1) {
            o.nbr_ptr[n] = nbr_ptr[n];
            o.tri_ptr[n] = tri_ptr[n];
        }
    }
    for (int64_t k = g; k < m3; k += stride) o.tri_idx[k] = tri_idx[k];
}

constexpr int64_t kBinNodes = int64_t(1) << 27;   // 4096 bins of 32768 nodes
constexpr int kBinGroups = 512;                   // work-groups of the histogram and the scatter

// Nodes per bin (a power of two): about 512 bins, so that the bins fill the
// device; at most 32768 nodes, whose counters take 128 KB of LDS.
int bin_shift(int32_t n)
{
    int s = 6;
    while (s < 15 && (static_cast<int64_t>(n) >> s) >= 512) ++s;
    return s;
}

}  // namespace

// Builds the adjacency of a device triangle list on `st` into device
// buffers of the library and hands it to the caller's arrays -- device
// arrays, written by the last kernel, or host arrays (to_host).  The
// caller's arrays are written only when everything succeeded; a null nbr_idx
// asks for *nnz only.
sl_status build_adjacency(const int32_t* d_tris, int32_t n_tris, int32_t n, int32_t* nbr_ptr, int32_t* nbr_idx,
                          int64_t nbr_capacity, int32_t* tri_ptr, int32_t* tri_idx, uint8_t* boundary, int64_t* nnz,
                          bool to_host, hipStream_t st)
{
    const int64_t m3 = 3 * static_cast<int64_t>(n_tris);
    const size_t un = static_cast<size_t>(n), um = static_cast<size_t>(std::max<int64_t>(m3, 1));
    const bool binned = n <= kBinNodes, build = nbr_idx != nullptr;
    const int shift = bin_shift(n), bins = binned ? div_up(n, 1 << shift) : 0;
    // a group takes at least 1024 triangles
    const int groups = std::max(1, std::min(kBinGroups, div_up(n_tris, 1024)));
    const int32_t per = div_up(n_tris, groups);
    const int64_t nh = static_cast<int64_t>(bins) * groups;
    const size_t bytes = Arena::piece(4) + 4 * Arena::piece(4 * (un + 1)) + Arena::piece(4 * um) + Arena::piece(8 * um) +
                         Arena::piece(2 * um) + Arena::piece(un) + 2 * Arena::piece(4 * static_cast<size_t>(nh + 1)) +
                         scan_bytes(std::max<int64_t>(n, nh)) +
                         (build && to_host ? 2 * Arena::piece(4 * (un + 1)) + Arena::piece(4 * um) + Arena::piece(8 * um) +
                                                 Arena::piece(un)
                                           : 0);
    PinnedPad pad;
    sl_status r = pad.init();
    if (r) return r;
    Arena ar;
    if ((r = ar.reserve(bytes, st))) return r;
    struct GiveBack {
        Arena& ar;
        hipStream_t st;
        ~GiveBack()
        {
            ar.release(st);
            (void)hipStreamSynchronize(st);
        }
    } give_back{ar, st};
    uint32_t* err = nullptr;
    int32_t *tp = nullptr, *ti = nullptr, *deg = nullptr, *np = nullptr, *hist = nullptr, *offs = nullptr, *cnt = nullptr;
    uint64_t* pairs = nullptr;   // later the scratch rows
    uint8_t *seen = nullptr, *bnd = nullptr;
    if ((r = ar.take(&err, 1)) || (r = ar.take(&tp, un + 1)) || (r = ar.take(&deg, un + 1)) || (r = ar.take(&np, un + 1)) ||
        (r = ar.take(&cnt, un + 1)) || (r = ar.take(&ti, um)) || (r = ar.take(&pairs, um)) || (r = ar.take(&seen, 2 * um)) ||
        (r = ar.take(&bnd, un)) || (r = ar.take(&hist, static_cast<size_t>(nh + 1))) ||
        (r = ar.take(&offs, static_cast<size_t>(nh + 1))))
        return r;
    int32_t* const row = reinterpret_cast<int32_t*>(pairs);
    const int gn = div_up(n, kAB);
    k_adj_zero<<<1, kAB, 0, st>>>(reinterpret_cast<int32_t*>(err), 1);
    if (m3 == 0) {
        k_adj_zero<<<std::min(gn, 1024), kAB, 0, st>>>(tp, static_cast<int64_t>(n) + 1);
    } else if (binned) {
        const size_t lds = sizeof(int32_t) * static_cast<size_t>(bins);
        const size_t blds = sizeof(int32_t) << shift;
        if (blds > 64 * 1024) {
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_adj_bins),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(blds));
            (void)hipGetLastError();
        }
        k_adj_hist<<<groups, kAB, lds, st>>>(d_tris, n_tris, n, shift, bins, per, hist, err);
        if ((r = scan_exclusive(hist, offs, nh, st, &ar))) return r;
        k_adj_scatter<<<groups, kAB, lds, st>>>(d_tris, n_tris, shift, bins, per, offs, pairs, err);
        k_adj_bins<<<bins, kBinBS, blds, st>>>(pairs, offs, groups, shift, n, tp, ti, err);
    } else {
        k_adj_zero<<<1024, kAB, 0, st>>>(cnt, n);
        k_adj_count<<<div_up(n_tris, kAB), kAB, 0, st>>>(d_tris, n_tris, n, cnt, err);
        if ((r = scan_exclusive(cnt, tp, n, st, &ar))) return r;
        k_adj_zero<<<1024, kAB, 0, st>>>(cnt, n);
        k_adj_fill<<<div_up(m3, kAB), kAB, 0, st>>>(d_tris, m3, tp, cnt, ti, err);
    }
    SL_HIP(hipGetLastError());
    if (build) k_adj_rows<true><<<gn, kAB, 0, st>>>(n, d_tris, tp, ti, row, seen, deg, bnd, err);
    else k_adj_rows<false><<<gn, kAB, 0, st>>>(n, d_tris, tp, ti, row, seen, deg, bnd, err);
    if ((r = scan_exclusive(deg, np, n, st, &ar))) return r;
    k_adj_tell<<<1, 1, 0, st>>>(err, np + n, static_cast<int32_t*>(pad.p));
    SL_HIP(hipGetLastError());
    SL_HIP(hipStreamSynchronize(st));
    int32_t told[2];
    std::memcpy(told, pad.p, sizeof(told));
    if (static_cast<uint32_t>(told[0]) & kAdjRange) return fail(SL_EINVAL, "triangle vertex id out of range");
    if (told[0]) return fail(SL_ETOPO, "triangle with a repeated vertex");
    const int32_t total = told[1];
    *nnz = total;
    if (!build) return SL_OK;
    if (total > nbr_capacity)
        return fail(SL_EINVAL, "nbr_idx holds " + std::to_string(nbr_capacity) + " entries, " +
                                   std::to_string(total) + " are needed");
    AdjOut o{nbr_ptr, nbr_idx, tri_ptr, tri_idx, boundary};
    if (to_host) {
        if ((r = ar.take(&o.nbr_ptr, un + 1)) || (r = ar.take(&o.tri_ptr, un + 1)) || (r = ar.take(&o.tri_idx, um)) ||
            (r = ar.take(&o.nbr_idx, 2 * um)) || (r = ar.take(&o.boundary, un)))
            return r;
    }
    k_adj_out<<<std::min(std::max(gn, div_up(um, kAB)), 8192), kAB, 0, st>>>(n, m3, tp, ti, row, np, bnd, o);
    SL_HIP(hipGetLastError());
    if (to_host) {
        const size_t n1 = un + 1;
        if ((r = copy_to_host(nbr_ptr, o.nbr_ptr, sizeof(int32_t) * n1, st)) ||
            (r = copy_to_host(nbr_idx, o.nbr_idx, sizeof(int32_t) * total, st)) ||
            (r = copy_to_host(tri_ptr, o.tri_ptr, sizeof(int32_t) * n1, st)) ||
            (r = copy_to_host(tri_idx, o.tri_idx, sizeof(int32_t) * m3, st)) ||
            (r = copy_to_host(boundary, o.boundary, un, st)))
            return r;
        return SL_OK;
    }
    SL_HIP(hipStreamSynchronize(st));
    return SL_OK;
}

namespace {

sl_status check_adj_args(const int32_t* tris, int32_t n_tris, int32_t n_nodes, const int32_t* nbr_ptr,
                         const int32_t* nbr_idx, int64_t nbr_capacity, const int32_t* tri_ptr,
                         const int32_t* tri_idx, const uint8_t* boundary, const int64_t* nnz)
{
    if (!nnz) return fail(SL_EINVAL, "null nnz");
    if (n_nodes <= 0) return fail(SL_EINVAL, "n_nodes must be >= 1");
    if (n_tris < 0) return fail(SL_EINVAL, "n_tris must be >= 0");
    if (n_tris > INT32_MAX / 6) return fail(SL_EINVAL, "n_tris too large");
    if (n_tris > 0 && !tris) return fail(SL_EINVAL, "null tris with n_tris > 0");
    if (nbr_idx && (!nbr_ptr || !tri_ptr || (n_tris > 0 && !tri_idx) || !boundary))
        return fail(SL_EINVAL, "null output array");
    if (nbr_capacity < 0) return fail(SL_EINVAL, "nbr_capacity must be >= 0");
    return SL_OK;
}

}  // namespace

}  // namespace sl

extern "C" {

sl_status sl_build_adjacency_device(const int32_t* tris, int32_t n_tris, int32_t n_nodes, int32_t* nbr_ptr,
                                    int32_t* nbr_idx, int64_t nbr_capacity, int32_t* tri_ptr, int32_t* tri_idx,
                                    uint8_t* boundary, int64_t* nnz, void* stream)
{
    using namespace sl;
    set_error("");
    sl_status r = check_adj_args(tris, n_tris, n_nodes, nbr_ptr, nbr_idx, nbr_capacity, tri_ptr, tri_idx, boundary,
                                 nnz);
    if (r) return r;
    keep_pool_warm();
    return build_adjacency(tris, n_tris, n_nodes, nbr_ptr, nbr_idx, nbr_capacity, tri_ptr, tri_idx, boundary, nnz,
                           false, static_cast<hipStream_t>(stream));
}

sl_status sl_build_adjacency(const int32_t* tris, int32_t n_tris, int32_t n_nodes, int32_t* nbr_ptr,
                             int32_t* nbr_idx, int64_t nbr_capacity, int32_t* tri_ptr, int32_t* tri_idx,
                             uint8_t* boundary, int64_t* nnz)
{
    using namespace sl;
    set_error("");
    sl_status r = check_adj_args(tris, n_tris, n_nodes, nbr_ptr, nbr_idx, nbr_capacity, tri_ptr, tri_idx, boundary,
                                 nnz);
    if (r) return r;
    keep_pool_warm();
    PooledStream ps;
    if ((r = ps.init())) return r;
    hipStream_t st = ps.s;
    Arena in;
    int32_t* d_tris = nullptr;
    const size_t m3 = 3 * static_cast<size_t>(n_tris);
    r = in.reserve(Arena::piece(sizeof(int32_t) * std::max<size_t>(m3, 1)), st);
    if (!r) r = in.take(&d_tris, std::max<size_t>(m3, 1));
    if (!r) r = copy_to_device(d_tris, tris, sizeof(int32_t) * m3, st);
    if (!r)
        r = build_adjacency(d_tris, n_tris, n_nodes, nbr_ptr, nbr_idx, nbr_capacity, tri_ptr, tri_idx, boundary, nnz,
                            true, st);
    in.release(st);
    (void)hipStreamSynchronize(st);
    return r;
}

}  // extern "C"
