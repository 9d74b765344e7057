// Mesh setup on the device: validation, node ordering, relabelling, fan
// build, coordinate buffers, and the inverse steps on the way out.
//
// The paper prepares a mesh in three procedures before iterating (Sec. 3.3.1
// initiating, Sec. 3.3.2 finding neighbours, Sec. 3.3.3 determining
// constraints).  Here the caller hands in the neighbour rows, incident
// triangles and the boundary mask; setup checks them and turns them into the
// layout the sweep kernels read:
//   - free nodes first, in Hilbert order of their position (or in the
//     caller's order), fixed nodes after them;
//   - neighbour rows relabelled, order inside a row kept (it is the
//     centroid's summation order);
//   - a 16-bit "fan" entry per (free node, incident triangle): the node's
//     position p in the triangle's stored order (bits 0-1) and the row slots
//     of the vertices at stored positions p+1 and p+2 mod 3 (bits 2-8, 9-15).
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "sl_common.h"
#include "sl_flow.h"

namespace sl {

namespace {

constexpr int kBS = 256;

// Order-preserving map of a double to uint64 (for atomic min/max).
__device__ __forceinline__ uint64_t ord_bits(double v)
{
    uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
    return (u & 0x8000000000000000ull) ? ~u : (u | 0x8000000000000000ull);
}
__host__ __device__ __forceinline__ double from_ord_bits(uint64_t u)
{
    u = (u & 0x8000000000000000ull) ? (u & 0x7FFFFFFFFFFFFFFFull) : ~u;
    double d;
    memcpy(&d, &u, sizeof(d));
    return d;
}

// ---------------------------------------------------------------- scan ----
//
// Reduce, then scan: one pass sums each tile of kScanTile values, and a
// second pass scans each tile from its offset.  Each work-item holds 16
// consecutive values, loaded and stored as four 16-byte vectors when the
// arrays allow it.

constexpr int kScanPer = 16;
constexpr int kScanTile = kBS * kScanPer;
constexpr int kSumsBS = 1024;

// This work-item's values of tile `b` (zeros past n).
__device__ __forceinline__ void scan_load(const int32_t* __restrict__ in, int64_t n, int64_t base, bool vec,
                                          int32_t (&v)[kScanPer])
{
    if (vec && base + kScanPer <= n) {
        const int4* p = reinterpret_cast<const int4*>(in + base);
#pragma unroll
        for (int q = 0; q < kScanPer / 4; ++q) {
            const int4 w = p[q];
            v[4 * q] = w.x;
            v[4 * q + 1] = w.y;
            v[4 * q + 2] = w.z;
            v[4 * q + 3] = w.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) v[j] = base + j < n ? in[base + j] : 0;
    }
}

// Exclusive scan of one value per work-item over a work-group of BS
// work-items (wave scans, then the wave totals); *total = the group's sum.
template <int BS>
__device__ __forceinline__ int32_t group_excl_scan(int32_t x, int32_t* s_wave, int32_t* total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int32_t inc = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t t = __shfl_up(inc, off, 64);
        if (lane >= off) inc += t;
    }
    if (lane == 63) s_wave[wv] = inc;
    __syncthreads();
    int32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < BS / 64; ++w) {
        const int32_t t = s_wave[w];
        before += w < wv ? t : 0;
        all += t;
    }
    __syncthreads();   // s_wave may be reused at once
    *total = all;
    return before + inc - x;
}

__global__ __launch_bounds__(kBS) void k_scan_sums(const int32_t* __restrict__ in, int64_t n, bool vec,
                                                   int32_t* __restrict__ sums)
{
    __shared__ int32_t s_wave[kBS / 64];
    int32_t v[kScanPer];
    scan_load(in, n, (static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x) * kScanPer, vec, v);
    int32_t x = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) x += v[j];
    int32_t total;
    (void)group_excl_scan<kBS>(x, s_wave, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Sum of sums[0..b) over a work-group of BS work-items (every one gets it).
template <int BS>
__device__ __forceinline__ int32_t sums_before(const int32_t* __restrict__ sums, int b, int32_t* s_wave)
{
    int32_t x = 0;
    for (int q = threadIdx.x; q < b; q += BS) x += sums[q];
    int32_t all;
    (void)group_excl_scan<BS>(x, s_wave, &all);
    return all;
}

// Exclusive scan of nb tile sums in place, by one work-group per row of nb.
__global__ __launch_bounds__(kSumsBS) void k_scan_offsets(int32_t* __restrict__ sums, int32_t nb)
{
    __shared__ int32_t s_wave[kSumsBS / 64];
    sums += static_cast<int64_t>(blockIdx.x) * nb;
    int32_t carry = 0;
    for (int32_t c0 = 0; c0 < nb; c0 += kSumsBS) {
        const int32_t b = c0 + static_cast<int32_t>(threadIdx.x), x = b < nb ? sums[b] : 0;
        int32_t all;
        const int32_t off = carry + group_excl_scan<kSumsBS>(x, s_wave, &all);
        if (b < nb) sums[b] = off;
        carry += all;
    }
}

// More tiles than this have their sums scanned before (k_scan_offsets).  Up to
// there each tile adds up the earlier tiles' sums itself, out of L2, which
// costs no more than the launch (adjacency of 130M nodes and a triangle 4.3 ms
// with, 4.2 without); but those reads grow with the square of the tiles (400M
// nodes 13.3 -> 10.3 ms, 10^9 47 -> 26).
constexpr int kSumsInPlace = 32768;

// Scans this work-group's tile from its offset: the sum of the earlier
// tiles' sums (scanned: already their scan).  The last tile also writes the
// total.
__device__ __forceinline__ void scan_tile(const int32_t* __restrict__ in, int32_t* __restrict__ out, int64_t n, bool vec,
                                          const int32_t* __restrict__ sums, bool scanned, int32_t* total, int32_t* s_wave)
{
    const int64_t base = (static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x) * kScanPer;
    int32_t v[kScanPer];
    scan_load(in, n, base, vec, v);
    int32_t x = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) x += v[j];
    const int32_t off = scanned ? sums[blockIdx.x] : sums_before<kBS>(sums, static_cast<int>(blockIdx.x), s_wave);
    int32_t all;
    int32_t run = off + group_excl_scan<kBS>(x, s_wave, &all);
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        const int32_t t = v[j];
        v[j] = run;
        run += t;
    }
    if (vec && base + kScanPer <= n) {
        int4* p = reinterpret_cast<int4*>(out + base);
#pragma unroll
        for (int q = 0; q < kScanPer / 4; ++q) p[q] = make_int4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    } else {
#pragma unroll
        for (int j = 0; j < kScanPer; ++j)
            if (base + j < n) out[base + j] = v[j];
    }
    if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) *total = off + all;
}

__global__ __launch_bounds__(kBS) void k_scan_tiles(const int32_t* __restrict__ in, int32_t* __restrict__ out,
                                                    int64_t n, bool vec, const int32_t* __restrict__ sums,
                                                    bool scanned, int32_t* __restrict__ total)
{
    __shared__ int32_t s_wave[kBS / 64];
    scan_tile(in, out, n, vec, sums, scanned, total, s_wave);
}

// Exclusive scan of a short in[0..n) by one work-group, kSumsBS*kScanPer
// values at a time with a running carry: one launch in place of two, for
// setups whose time goes into launches (a batch of small meshes).  In place
// (in == out) is allowed: every value is read and written by one work-item.
__global__ __launch_bounds__(kSumsBS) void k_scan_one(const int32_t* in, int32_t* out, int64_t n, bool vec,
                                                      int32_t* total)
{
    __shared__ int32_t s_wave[kSumsBS / 64];
    int32_t carry = 0;
    for (int64_t c0 = 0; c0 < n; c0 += static_cast<int64_t>(kSumsBS) * kScanPer) {
        const int64_t base = c0 + static_cast<int64_t>(threadIdx.x) * kScanPer;
        int32_t v[kScanPer];
        scan_load(in, n, base, vec, v);
        int32_t x = 0;
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) x += v[j];
        int32_t all;
        int32_t run = carry + group_excl_scan<kSumsBS>(x, s_wave, &all);
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            const int32_t t = v[j];
            v[j] = run;
            run += t;
        }
        if (vec && base + kScanPer <= n) {
            int4* p = reinterpret_cast<int4*>(out + base);
#pragma unroll
            for (int q = 0; q < kScanPer / 4; ++q) p[q] = make_int4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        } else {
#pragma unroll
            for (int j = 0; j < kScanPer; ++j)
                if (base + j < n) out[base + j] = v[j];
        }
        carry += all;
    }
    if (threadIdx.x == 0) *total = carry;
}

// Scans this long or shorter take the one-launch path (one pass of its loop:
// each further pass is a serial trip to memory, 28 us for 100K values
// against 8 us for the two launches).
constexpr int64_t kScanOneMax = int64_t(1) * kSumsBS * kScanPer;

// Exclusive scan of in[0..n) into out[0..n); *total = sum.  The tile sums
// come from `ar` when given, else from the allocator.
sl_status scan_rec(const int32_t* in, int32_t* out, int64_t n, int32_t* total, hipStream_t st, Arena* ar)
{
    if (n <= kScanOneMax) {
        const bool vec1 = ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
        k_scan_one<<<1, kSumsBS, 0, st>>>(in, out, n, vec1, total);
        SL_HIP(hipGetLastError());
        return SL_OK;
    }
    const int nb = div_up(n > 0 ? n : 1, kScanTile);
    int32_t* sums = nullptr;
    sl_status r = ar ? ar->take(&sums, static_cast<size_t>(nb)) : dalloc(&sums, static_cast<size_t>(nb), st);
    if (r) return r;
    const bool vec = ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
    k_scan_sums<<<nb, kBS, 0, st>>>(in, n, vec, sums);
    if (nb > kSumsInPlace) k_scan_offsets<<<1, kSumsBS, 0, st>>>(sums, nb);
    k_scan_tiles<<<nb, kBS, 0, st>>>(in, out, n, vec, sums, nb > kSumsInPlace, total);
    if (!ar) dfree(sums, st);
    SL_HIP(hipGetLastError());
    return SL_OK;
}

}  // namespace

// Arena bytes the temporaries of a scan of n values take.
size_t scan_bytes(int64_t n) { return Arena::piece(4 * static_cast<size_t>(div_up(n > 0 ? n : 1, kScanTile))); }

namespace {

// ----------------------------------------------------------- validation ---

struct ValArgs {
    const double* coords;
    int32_t n;
    const int32_t* nbr_ptr;
    const int32_t* nbr_idx;
    const int32_t* tri_ptr;
    const int32_t* tri_idx;
    const int32_t* tris;
    int32_t n_tris;
    const uint8_t* boundary;
    int64_t nnz, ninc;     // < 0: read from the ends of the offsets
    int check_symmetry;
    double coord_limit;    // coordinates must be below this in magnitude
};

constexpr int kRowRegs = 8;    // row entries, and incidences, of a node held in registers (k_rows_fans)
constexpr int kRowLds = 16;    // row entries held in LDS (k_validate_nodes)

__device__ __forceinline__ bool row_has(const int32_t* __restrict__ idx, int32_t b, int32_t e, int32_t v)
{
    for (int32_t k = b; k < e; ++k)
        if (idx[k] == v) return true;
    return false;
}

// Incidence rows that disagree (for the Form A tile path, which lists a
// triangle once per tile and scores it for every own vertex): a triangle
// listed by some of its free vertices but not by all of them.  One
// work-item per triangle looks for it in its free vertices' rows, the three
// rows' offsets and first kIncRegs entries loaded together.  Offsets out of
// order are left to the other checks.  Without `incidence` only the
// triangle's own vertices are checked.
constexpr int kIncRegs = 8;
__device__ __forceinline__ void check_triangle(int64_t t, const int32_t* __restrict__ tris, int32_t n,
                                               const uint8_t* __restrict__ bnd, const int32_t* __restrict__ tri_ptr,
                                               const int32_t* __restrict__ tri_idx, int64_t ninc, bool listed,
                                               ValStats* vs)
{
    int32_t v[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = tris[3 * t + k];
    uint32_t e = 0;
    if (v[0] == v[1] || v[1] == v[2] || v[0] == v[2]) e |= VE_TRIREP;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (v[k] < 0 || v[k] >= n) e |= VE_RANGE;
    if (e) atomicOr(&vs->err, e);
    if (!listed || (e & VE_RANGE)) return;
    int32_t ob[3], oe[3];
    uint8_t fl[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        fl[k] = bnd[v[k]];
        ob[k] = tri_ptr[v[k]];
        oe[k] = tri_ptr[v[k] + 1];
    }
    bool use[3];
    int32_t len[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        use[k] = fl[k] == 0 && 0 <= ob[k] && ob[k] <= oe[k] && oe[k] <= ninc;
        len[k] = use[k] ? oe[k] - ob[k] : 0;
    }
    int32_t x[3][kIncRegs];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int q = 0; q < kIncRegs; ++q) x[k][q] = tri_idx[len[k] > 0 ? ob[k] + min(q, len[k] - 1) : 0];
    int lists = 0, free_v = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (!use[k]) continue;
        ++free_v;
        bool found = false;
#pragma unroll
        for (int q = 0; q < kIncRegs; ++q) found |= q < len[k] && x[k][q] == static_cast<int32_t>(t);
        if (!found && len[k] > kIncRegs) found = row_has(tri_idx, ob[k] + kIncRegs, oe[k], static_cast<int32_t>(t));
        lists += found;
    }
    if (lists > 0 && lists < free_v) atomicOr(&vs->err, static_cast<uint32_t>(VI_INCIDENCE));
}

// What the fold found to need a check of its own.  Most inputs leave it
// nothing to do (4096^2: 550 us of random reads before that was seen; the
// symmetry test within the node checks 40-70 us at 2.2M nodes).
template <bool INCIDENCE>
__global__ __launch_bounds__(kBS) void k_validate_rest(const int32_t* __restrict__ tris, int32_t n_tris, int32_t n,
                                                       const uint8_t* __restrict__ bnd,
                                                       const int32_t* __restrict__ nbr_ptr,
                                                       const int32_t* __restrict__ nbr_idx,
                                                       const int32_t* __restrict__ tri_ptr,
                                                       const int32_t* __restrict__ tri_idx, int64_t ninc, ValStats* vs)
{
    if (vs->check_sym != 0) {
        // each neighbour of a free node that is free too lists the node
        const int64_t nnz = nbr_ptr[n];
        for (int64_t i64 = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x; i64 < n;
             i64 += static_cast<int64_t>(gridDim.x) * kBS) {
            const int32_t i = static_cast<int32_t>(i64), b = nbr_ptr[i], en = nbr_ptr[i + 1];
            if (bnd[i] != 0 || !(0 <= b && b <= en && en <= nnz)) continue;
            bool bad = false;
            for (int32_t k = b; k < en; ++k) {
                const int32_t j = nbr_idx[k];
                if (j < 0 || j >= n || bnd[j] != 0) continue;
                const int32_t jb = nbr_ptr[j], je = nbr_ptr[j + 1];
                bad |= !(0 <= jb && jb <= je && je <= nnz) || !row_has(nbr_idx, jb, je, i);
            }
            if (bad) atomicOr(&vs->err, static_cast<uint32_t>(VE_ASYM));
        }
    }
    if (vs->check_tris == 0) return;
    if (ninc < 0) ninc = tri_ptr[n];   // not known on the host
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x; t < n_tris;
         t += static_cast<int64_t>(gridDim.x) * kBS)
        check_triangle(t, tris, n, bnd, tri_ptr, tri_idx, ninc, INCIDENCE && ninc > 0, vs);
}

// Statistics of a wave or work-group, folded pairwise.
__device__ __forceinline__ void fold_stats(ValStats& a, const ValStats& b)
{
    a.err |= b.err;
    a.n_free += b.n_free;
    a.max_deg_free = max(a.max_deg_free, b.max_deg_free);
    a.max_inc_free = max(a.max_inc_free, b.max_inc_free);
    a.nnz_free += b.nnz_free;
    a.ninc_free += b.ninc_free;
    a.unordered |= b.unordered;
    a.uncovered |= b.uncovered;
    a.box[0] = min(a.box[0], b.box[0]);
    a.box[1] = min(a.box[1], b.box[1]);
    a.box[2] = max(a.box[2], b.box[2]);
    a.box[3] = max(a.box[3], b.box[3]);
}

// Over each N consecutive lanes of a wave.
template <int N>
__device__ __forceinline__ void fold_stats_lanes(ValStats& a)
{
#pragma unroll
    for (int off = N / 2; off > 0; off >>= 1) {
        ValStats b;
        b.err = __shfl_xor(a.err, off);
        b.n_free = __shfl_xor(a.n_free, off);
        b.max_deg_free = __shfl_xor(a.max_deg_free, off);
        b.max_inc_free = __shfl_xor(a.max_inc_free, off);
        b.nnz_free = __shfl_xor(a.nnz_free, off);
        b.ninc_free = __shfl_xor(a.ninc_free, off);
        b.unordered = __shfl_xor(a.unordered, off);
        b.uncovered = __shfl_xor(a.uncovered, off);
        for (int q = 0; q < 4; ++q)
            b.box[q] = static_cast<uint64_t>(__shfl_xor(static_cast<unsigned long long>(a.box[q]), off));
        fold_stats(a, b);
    }
}

// An empty set's statistics.
__device__ __forceinline__ ValStats empty_stats()
{
    return ValStats{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, {~0ull, ~0ull, 0ull, 0ull}, 0};
}

// LANES work-items per node, which share its neighbours and triangles; the
// work-groups take the nodes in strides and each leaves its statistics (with
// the bounding box of its nodes' coordinates, so that no pass of its own has
// to read them again) in a slot of its own.  Rows of up to kRowLds entries are
// held in an LDS column for the membership tests; longer ones are searched
// in memory.  The loops over the row and the incidences are kept rolled, a
// few loads in flight together: with the row in registers and every test
// unrolled the kernel was 26 KB of code, and on small meshes fetching that
// took most of its time (64 x 64 grid 16 us, 100K shuffled nodes 44 us).
template <int LANES>
__global__ __launch_bounds__(kBS) void k_validate_nodes(ValArgs a, ValStats* __restrict__ part)
{
    __shared__ int32_t s_row[kRowLds][kBS / LANES];
    constexpr int U = 4;   // entries whose loads are in flight together
    const int tid = threadIdx.x / LANES, sub = threadIdx.x % LANES;
    const int64_t nnz = a.nnz >= 0 ? a.nnz : a.nbr_ptr[a.n], ninc = a.ninc >= 0 ? a.ninc : a.tri_ptr[a.n];
    ValStats me = empty_stats();
    const uint64_t t0 = wall_clock64();
    if (blockIdx.x == 0 && threadIdx.x == 0 && (a.nbr_ptr[0] != 0 || a.tri_ptr[0] != 0)) me.err |= VE_PTR;
    for (int64_t i64 = static_cast<int64_t>(blockIdx.x) * (kBS / LANES) + tid; i64 < a.n;
         i64 += static_cast<int64_t>(gridDim.x) * (kBS / LANES)) {
        const int32_t i = static_cast<int32_t>(i64);
        uint32_t e = 0;
        int deg = 0, inc = 0;
        const double2 xy = reinterpret_cast<const double2*>(a.coords)[i];
        const uint64_t ox = ord_bits(xy.x), oy = ord_bits(xy.y);
        me.box[0] = min(me.box[0], ox);
        me.box[1] = min(me.box[1], oy);
        me.box[2] = max(me.box[2], ox);
        me.box[3] = max(me.box[3], oy);
        // finite and below the limit in magnitude (2^500 in double, 2^61 in
        // single precision): squared edge lengths, their sums and cross
        // products cannot overflow, so every quality is a finite number
        if (!(fabs(xy.x) < a.coord_limit) || !(fabs(xy.y) < a.coord_limit)) e |= VE_COORD;
        const int32_t b = a.nbr_ptr[i], en = a.nbr_ptr[i + 1];
        const bool row_ok = 0 <= b && b <= en && en <= nnz;
        const int32_t tb = a.tri_ptr[i], te = a.tri_ptr[i + 1];
        const bool trow_ok = 0 <= tb && tb <= te && te <= ninc;
        if (!row_ok || !trow_ok) e |= VE_PTR;
        const bool is_free = a.boundary[i] == 0;
        const bool in_lds = row_ok && en - b <= kRowLds;
        if (row_ok) {
            deg = en - b;
            if (is_free && deg == 0) e |= VE_EMPTY;
            if (is_free && deg > kMaxValence) e |= VE_VALENCE;
#pragma unroll 1
            for (int k0 = U * sub; k0 < deg; k0 += U * LANES) {
                int32_t j[U];
#pragma unroll
                for (int u = 0; u < U; ++u) j[u] = a.nbr_idx[b + min(k0 + u, deg - 1)];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (in_lds && k0 + u < deg) s_row[k0 + u][tid] = j[u];
                    if (j[u] < 0 || j[u] >= a.n) e |= VE_RANGE;
                    if (j[u] == i) e |= VE_SELF;
                }
            }
        }
        // (a node's lanes are of one wave: their LDS writes are in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint32_t covered = 0;   // the row entries found in the node's triangles
        if (trow_ok) {
            inc = te - tb;
            // incident triangles U at a time: their loads are in flight together
#pragma unroll 1
            for (int32_t k0 = tb + U * sub; k0 < te; k0 += U * LANES) {
                int32_t t[U], v[U][3];
#pragma unroll
                for (int u = 0; u < U; ++u) t[u] = a.tri_idx[min(k0 + u, te - 1)];
                int32_t before = k0 > tb ? a.tri_idx[k0 - 1] : -1;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (k0 + u < te && t[u] <= before) me.unordered = 1;
                    before = t[u];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool ok = t[u] >= 0 && t[u] < a.n_tris;
                    if (!ok) {
                        e |= VE_RANGE;
                        t[u] = -1;
                    }
#pragma unroll
                    for (int s3 = 0; s3 < 3; ++s3) v[u][s3] = ok ? a.tris[3 * static_cast<int64_t>(t[u]) + s3] : i;
                }
                bool f1[U], f2[U];
                int32_t o1[U], o2[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t v0 = v[u][0], v1 = v[u][1], v2 = v[u][2];
                    const bool has = v0 == i || v1 == i || v2 == i;
                    if (!has) e |= VE_NOTIN;
                    // the other two vertices, in stored cyclic order after i
                    o1[u] = v0 == i ? v1 : (v1 == i ? v2 : v0);
                    o2[u] = v0 == i ? v2 : (v1 == i ? v0 : v1);
                    f1[u] = f2[u] = !has || t[u] < 0 || !is_free || !row_ok;
                }
                if (in_lds) {
#pragma unroll 1
                    for (int k = 0; k < deg; ++k) {
                        const int32_t r = s_row[k][tid];
                        bool hit = false;
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            f1[u] |= r == o1[u];
                            f2[u] |= r == o2[u];
                            hit |= r == o1[u] || r == o2[u];
                        }
                        covered |= hit ? 1u << k : 0u;
                    }
                } else if (row_ok && is_free) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (!f1[u]) f1[u] = row_has(a.nbr_idx, b, en, o1[u]);
                        if (!f2[u]) f2[u] = row_has(a.nbr_idx, b, en, o2[u]);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (!f1[u] || !f2[u]) e |= VE_MISSING;
            }
        }
        me.err |= e;
#pragma unroll
        for (int off = LANES / 2; off > 0; off >>= 1) covered |= __shfl_xor(covered, off);
        if (is_free && (!in_lds || covered != (1u << deg) - 1u)) me.uncovered = 1;
        if (is_free && sub == 0) {
            me.n_free += 1;
            me.max_deg_free = max(me.max_deg_free, deg);
            me.max_inc_free = max(me.max_inc_free, inc);
            me.nnz_free += deg;
            me.ninc_free += inc;
        }
        // (the next node's row takes this one's place: program order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    fold_stats_lanes<64>(me);
    __shared__ ValStats s_part[kBS / 64];
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = me;
    __syncthreads();
    if (threadIdx.x < 64) {
        me = s_part[threadIdx.x & (kBS / 64 - 1)];
        fold_stats_lanes<kBS / 64>(me);
        if (threadIdx.x == 0) {
            me.t0 = t0;
            part[blockIdx.x] = me;
        }
    }
}

// Folds the per-block statistics into *vs (one work-group, no atomics), and
// decides whether the triangles need a check of their own.  They do not when
// every incidence row is strictly ascending (no entry twice), every entry
// names a triangle that holds its node, and the rows of all nodes have three
// entries per triangle between them: a triangle has at most one entry in the
// row of each of its distinct vertices, so it then has three distinct
// vertices, all in range, and is in all their rows.
__global__ __launch_bounds__(1024) void k_validate_fold(const ValStats* __restrict__ part, int32_t nb, ValArgs a,
                                                        ValStats* __restrict__ vs)
{
    __shared__ ValStats s_part[16];
    ValStats me = empty_stats();
    for (int32_t b = threadIdx.x; b < nb; b += 1024) fold_stats(me, part[b]);
    fold_stats_lanes<64>(me);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = me;
    __syncthreads();
    if (threadIdx.x < 64) {
        me = s_part[threadIdx.x & 15];
        fold_stats_lanes<16>(me);
        if (threadIdx.x == 0) {
            const int64_t ninc = a.ninc >= 0 ? a.ninc : a.tri_ptr[a.n];
            me.check_tris = (me.err & (VE_PTR | VE_RANGE | VE_NOTIN)) != 0 || me.unordered != 0 ||
                            ninc != 3 * static_cast<int64_t>(a.n_tris);
            // Rows are symmetric when nothing is wrong so far and every free
            // node's row holds vertices of its own triangles only: the
            // triangle that puts j into i's row is in j's list too (above),
            // and j's row holds its vertices.
            me.check_sym = a.check_symmetry != 0 && (me.err != 0 || me.check_tris != 0 || me.uncovered != 0);
            me.t0 = part[0].t0;
            *vs = me;
        }
    }
}

// ------------------------------------------------------------- ordering ---

// Hilbert index of cell (x, y) on a 2^bits x 2^bits grid.
__device__ __forceinline__ uint32_t hilbert_index(int bits, uint32_t x, uint32_t y)
{
    uint32_t d = 0;
    for (uint32_t s = 1u << (bits - 1); s > 0; s >>= 1) {
        const uint32_t rx = (x & s) ? 1u : 0u, ry = (y & s) ? 1u : 0u;
        d += s * s * ((3u * rx) ^ ry);
        if (ry == 0) {
            if (rx == 1) { x = (s - 1) ^ x; y = (s - 1) ^ y; }
            const uint32_t t = x; x = y; y = t;
        }
    }
    return d;
}

// Bucket of each free node: colour * 4^bits + Hilbert cell.  Fixed nodes:
// cells of their own, 4^fixed_bits of them from fixed_base on, or none
// (fixed_base < 0).
// Lanes of a wave that share a bucket count together, for up to
// kBucketShared buckets a wave: where many nodes fall into few buckets
// (strongly graded meshes), an atomic per node on one address is a queue
// (360K nodes, most of them in a handful of cells: setup 952 -> 243 us).
constexpr int kBucketShared = 4;
__global__ __launch_bounds__(kBS) void k_bucket(const double* __restrict__ coords, const uint8_t* __restrict__ bnd,
                                                const int32_t* __restrict__ color, int32_t n, int bits,
                                                int32_t fixed_base, int fixed_bits, const ValStats* __restrict__ vs, int32_t* __restrict__ key,
                                                int32_t* __restrict__ count, int32_t* __restrict__ rank)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (i >= n) return;
    const bool fixed = bnd[i] != 0;
    if (fixed && fixed_base < 0) return;
    if (fixed) bits = fixed_bits;
    uint32_t cell = 0;
    if (bits > 0) {
        const double x0 = from_ord_bits(vs->box[0]), y0 = from_ord_bits(vs->box[1]);
        const double ext = fmax(from_ord_bits(vs->box[2]) - x0, from_ord_bits(vs->box[3]) - y0);
        const double side = static_cast<double>(1u << bits);
        const double sc = ext > 0.0 ? side / ext : 0.0;
        const uint32_t lim = (1u << bits) - 1u;
        const double fx = (coords[2 * i] - x0) * sc, fy = (coords[2 * i + 1] - y0) * sc;
        const uint32_t cx = fx <= 0.0 ? 0u : (fx >= lim ? lim : static_cast<uint32_t>(fx));
        const uint32_t cy = fy <= 0.0 ? 0u : (fy >= lim ? lim : static_cast<uint32_t>(fy));
        cell = hilbert_index(bits, cx, cy);
    }
    const int32_t k = (fixed ? fixed_base : (color ? color[i] : 0) * (1 << (2 * bits))) + static_cast<int32_t>(cell);
    key[i] = k;
    const int lane = static_cast<int>(threadIdx.x & 63);
    int lead = lane, many = 1, at = 0;   // who counts for this lane, for how many, and the lane's place among them
    unsigned long long todo = __ballot(1);
#pragma unroll 1
    for (int r = 0; r < kBucketShared && todo != 0; ++r) {
        const int l = __builtin_ctzll(todo);
        const unsigned long long same = __ballot(k == __builtin_amdgcn_readlane(k, l)) & todo;
        if ((same >> lane) & 1ull) {
            lead = l;
            many = __popcll(same);
            at = __popcll(same & ((1ull << lane) - 1ull));
        }
        todo &= ~same;
    }
    int32_t base = 0;
    if (lead == lane) base = atomicAdd(count + k, many);
    rank[i] = __shfl(base, lead) + at;   // place inside the bucket (in no particular order)
}

__global__ __launch_bounds__(kBS) void k_bucket_scatter(int32_t n, const int32_t* __restrict__ key,
                                                        const int32_t* __restrict__ rank,
                                                        const int32_t* __restrict__ start,
                                                        int32_t* __restrict__ new_of_old, int32_t* __restrict__ perm)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (i >= n) return;
    const int32_t pos = start[key[i]] + rank[i];
    new_of_old[i] = pos;
    perm[pos] = static_cast<int32_t>(i);
}

// The same for the flow path, where fixed nodes have no place (-1).
__global__ __launch_bounds__(kBS) void k_flow_scatter(const uint8_t* __restrict__ bnd, int32_t n,
                                                      const int32_t* __restrict__ key, const int32_t* __restrict__ rank,
                                                      const int32_t* __restrict__ start,
                                                      int32_t* __restrict__ new_of_old, int32_t* __restrict__ perm)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (i >= n) return;
    if (bnd[i]) {
        new_of_old[i] = -1;
        return;
    }
    const int32_t pos = start[key[i]] + rank[i];
    new_of_old[i] = pos;
    perm[pos] = static_cast<int32_t>(i);
}

// flag[i] = (bnd[i] != 0) == want_fixed  (and, if color given, color[i] == c)
__global__ __launch_bounds__(kBS) void k_select(const uint8_t* __restrict__ bnd, const int32_t* __restrict__ color,
                                                int32_t c, int want_fixed, int32_t n, int32_t* __restrict__ flag)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (i >= n) return;
    int f = (bnd[i] != 0) == (want_fixed != 0);
    if (f && color) f = color[i] == c;
    flag[i] = f;
}

__global__ __launch_bounds__(kBS) void k_place(const int32_t* __restrict__ flag, const int32_t* __restrict__ pos,
                                               int32_t base, int32_t n, int32_t* __restrict__ new_of_old,
                                               int32_t* __restrict__ perm)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (i >= n || !flag[i]) return;
    const int32_t p = base + pos[i];
    new_of_old[i] = p;
    perm[p] = static_cast<int32_t>(i);
}

// ------------------------------------------------------------ colouring ---

// One round of greedy colouring in decreasing priority: a free node takes
// the smallest colour unused by its free neighbours once every free
// neighbour of higher priority has a colour.
// Appends v to list[] for every work-item of the group whose `keep` is set:
// one atomic per work-group reserves the group's places (one per wave, or
// per work-item, on a single counter would queue behind each other).  Every
// work-item of the group must call it.
constexpr int kColorBS = 256;
__device__ __forceinline__ void append_group(bool keep, int32_t v, int32_t* __restrict__ list,
                                             int32_t* __restrict__ count, int32_t* s_tmp /* [kColorBS/64 + 1] */)
{
    const int lane = static_cast<int>(threadIdx.x & 63), wv = static_cast<int>(threadIdx.x >> 6);
    const unsigned long long mask = __ballot(keep);
    if (lane == 0) s_tmp[wv] = __popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t tot = 0;
        for (int w = 0; w < kColorBS / 64; ++w) {
            const int32_t c = s_tmp[w];
            s_tmp[w] = tot;
            tot += c;
        }
        s_tmp[kColorBS / 64] = tot ? atomicAdd(count, tot) : 0;
    }
    __syncthreads();
    if (keep) list[s_tmp[kColorBS / 64] + s_tmp[wv] + __popcll(mask & ((1ull << lane) - 1ull))] = v;
}

constexpr int kColorRounds = 3;    // rounds between two looks of the host
constexpr int kColorTries = 80;    // tries of a node inside a round
constexpr int kColorWindow = 256 * 2048;   // listed nodes that are tried at the same time: the device's work-items

// One Jones-Plassmann round over the listed (uncoloured) free nodes: a node
// whose neighbours of higher priority are all coloured takes the smallest
// colour none of them has; the others go to the next list.  A node tries
// several times before it gives up, so that a chain of nodes that wait for
// each other is walked inside one launch as far as its nodes run at the same
// time (a bounded number of tries, no waiting: 2.2M nodes take 2 rounds
// instead of 21; small work-groups, whose places free up early).  A node does
// not wait for one that cannot get its colour in this round: one that has
// given up, which marks itself with the round's number, or one so far ahead
// in the numbering that its work-group has not begun (a list of n_list of
// the n nodes, in about their order, is n / n_list times as dense).  Without
// that a mesh in arbitrary numbering spent its rounds on tries in vain
// (2.2M shuffled nodes: setup 7.4 ms; 3.4 with, and 3.6 with one try a
// round; in grid numbering 0.93 either way, and 1.9 with one try).  The
// colour a node gets depends only on those neighbours' colours, so neither
// the rounds nor the list order change the result.
// cnt[0]: the list's length, cnt[1]: the next one's; top: the largest
// colour.  list null: the first round, over all n nodes.
__global__ __launch_bounds__(kColorBS) void k_color_round(const int32_t* __restrict__ nbr_ptr,
                                                     const int32_t* __restrict__ nbr_idx,
                                                     const uint8_t* __restrict__ bnd, int32_t* color,
                                                     const int32_t* __restrict__ list, int32_t n, int32_t round,
                                                     int32_t* cnt, int32_t* __restrict__ next, int32_t* top)
{
    constexpr int R = 8;
    __shared__ int32_t s_tmp[kColorBS / 64 + 1];
    const int32_t n_list = list ? cnt[0] : n;   // left by the previous round
    const int32_t t = static_cast<int32_t>(blockIdx.x * kColorBS + threadIdx.x);
    bool left = t < n_list && (list || !bnd[t]);
    int32_t i = -1, c = -1;
    if (left) {
        i = list ? list[t] : t;
        const uint64_t pi = splitmix64(static_cast<uint64_t>(i));
        const int32_t b = nbr_ptr[i], d = nbr_ptr[i + 1] - b;
        int32_t above[R];   // the first R neighbours that must have a colour first, else -1
#pragma unroll
        for (int j = 0; j < R; ++j) above[j] = j < d ? nbr_idx[b + j] : -1;
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (above[j] >= 0 && (bnd[above[j]] != 0 || splitmix64(static_cast<uint64_t>(above[j])) < pi)) above[j] = -1;
        uint64_t used0 = 0, used1 = 0;
        auto use = [&](int32_t cj) {
            if (cj < 64) used0 |= 1ull << cj;
            else used1 |= 1ull << (cj - 64);
        };
        const int32_t given_up = -2 - round;
        const int32_t reach = static_cast<int32_t>(
            min(static_cast<int64_t>(kColorWindow) * n / n_list, static_cast<int64_t>(INT32_MAX)));
        bool wait = true;
        for (int tries = 0; tries < kColorTries && left && wait; ++tries) {
            bool ready = true;
            int32_t cj[R];
#pragma unroll
            for (int j = 0; j < R; ++j) cj[j] = -1;
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (above[j] >= 0)
                    cj[j] = __hip_atomic_load(color + above[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (above[j] < 0) continue;
                if (cj[j] >= 0) {
                    use(cj[j]);
                    above[j] = -1;
                } else {
                    ready = false;
                    wait &= cj[j] != given_up && above[j] - i <= reach;
                }
            }
            if (d > R && ready)
                for (int32_t k = b + R; k < b + d; ++k) {
                    const int32_t j = nbr_idx[k];
                    if (bnd[j] || splitmix64(static_cast<uint64_t>(j)) < pi) continue;
                    const int32_t q = __hip_atomic_load(color + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (q >= 0) use(q);
                    else {
                        ready = false;
                        wait &= q != given_up && j - i <= reach;
                    }
                }
            if (ready) {
                c = (~used0) ? __builtin_ctzll(~used0) : 64 + __builtin_ctzll(~used1);
                __hip_atomic_store(color + i, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                left = false;
            }
        }
        if (left) __hip_atomic_store(color + i, given_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    append_group(left, i, next, cnt + 1, s_tmp);
    for (int off = 32; off > 0; off >>= 1) c = max(c, __shfl_xor(c, off));
    if ((threadIdx.x & 63) == 0 && c > __hip_atomic_load(top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(top, c);
}

__global__ void k_put_stats(ValStats* vs, ValStats h)
{
    if (threadIdx.x == 0) *vs = h;
}

// out[k] = in[k * stride] for k < n: a few words to pinned host memory.
__global__ void k_tell(const int32_t* __restrict__ in, int32_t n, int64_t stride, int32_t* __restrict__ out)
{
    for (int32_t k = threadIdx.x; k < n; k += blockDim.x) out[k] = in[k * stride];
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------ relabel -----

// Row lengths and incidence counts of the free nodes in device order, and
// their sums over each tile of kScanTile nodes (sums[b] and sums[nb + b]):
// the first pass of both offset scans, which k_offset_tiles finishes.
__global__ __launch_bounds__(kBS) void k_degree_sums(const int32_t* __restrict__ perm, int32_t n_free,
                                                     const int32_t* __restrict__ nbr_ptr,
                                                     const int32_t* __restrict__ tri_ptr, int32_t* __restrict__ deg,
                                                     int32_t* __restrict__ inc, int32_t* __restrict__ sums)
{
    __shared__ int32_t s_wave[kBS / 64];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x;
    int32_t x = 0, y = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        const int64_t k = base + j * kBS;
        if (k < n_free) {
            const int32_t o = perm[k];
            const int32_t d = nbr_ptr[o + 1] - nbr_ptr[o], c = tri_ptr[o + 1] - tri_ptr[o];
            deg[k] = d;
            inc[k] = c;
            x += d;
            y += c;
        }
    }
    int32_t tx, ty;
    (void)group_excl_scan<kBS>(x, s_wave, &tx);
    (void)group_excl_scan<kBS>(y, s_wave, &ty);
    if (threadIdx.x == 0) {
        sums[blockIdx.x] = tx;
        sums[gridDim.x + blockIdx.x] = ty;
    }
}

// Row offsets (blockIdx.y == 0) and incidence offsets (1).
__global__ __launch_bounds__(kBS) void k_offset_tiles(const int32_t* __restrict__ deg, const int32_t* __restrict__ inc,
                                                      int64_t n, const int32_t* __restrict__ sums, bool scanned,
                                                      int32_t* __restrict__ row_ptr, int32_t* __restrict__ fan_ptr)
{
    __shared__ int32_t s_wave[kBS / 64];
    int32_t* const out = blockIdx.y ? fan_ptr : row_ptr;
    // (arena pieces: 256-byte aligned)
    scan_tile(blockIdx.y ? inc : deg, out, n, true, sums + (blockIdx.y ? gridDim.x : 0), scanned, out + n,
              s_wave);
}

// The node path's rows in device labels and fan entries, p | slot << 2 |
// slot << 9: the node's position p in the triangle's stored order and the row
// slots of the vertices at p+1 and p+2 (mod 3).  GROUP: each node's entries
// grouped by p (0, then 1, then 2; incidence order inside a group) with the
// groups' bounds, c0 | (c0 + c1) << 16 for c_p entries of position p, so that
// the node kernel evaluates each group with the position fixed at compile
// time.  A minimum over a fan is exact, so the order of its entries changes
// no result.
// One work-item per node, its first kRowRegs entries and triangles in
// registers, every load of a stage in flight together and none in a branch.
// With 16 row entries in registers, loads and stores in branches (each waits
// for the last) and the grouping in a launch of its own it took 399 us on a
// 1500 x 1500 grid (now 194); at 4096 x 4096 the whole setup went from 6.31
// to 5.13 ms.  In arbitrary numbering it is bound by the cache lines it
// touches (2.4M nodes: 911 -> 790 us).
template <bool GROUP>
__global__ __launch_bounds__(kBS) void k_rows_fans(const int32_t* __restrict__ perm,
                                                   const int32_t* __restrict__ new_of_old, int32_t n_free,
                                                   const int32_t* __restrict__ nbr_ptr,
                                                   const int32_t* __restrict__ nbr_idx,
                                                   const int32_t* __restrict__ tri_ptr,
                                                   const int32_t* __restrict__ tri_idx,
                                                   const int32_t* __restrict__ tris,
                                                   const int32_t* __restrict__ row_ptr, int32_t* __restrict__ nbr,
                                                   const int32_t* __restrict__ fan_ptr, uint16_t* __restrict__ fan,
                                                   uint32_t* __restrict__ split)
{
    constexpr int U = kRowRegs;
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (k >= n_free) return;
    const int32_t o = perm[k];
    const int32_t b = nbr_ptr[o], d = nbr_ptr[o + 1] - b;   // d >= 1 for a free node
    const int32_t tb = tri_ptr[o], nt = tri_ptr[o + 1] - tb;
    const int32_t out = row_ptr[k], fo = fan_ptr[k];
    int32_t r[U];
#pragma unroll
    for (int j = 0; j < U; ++j) r[j] = nbr_idx[b + min(j, d - 1)];
    Corners v[U];
    if (nt > 0) {
        int32_t t[U];
#pragma unroll
        for (int q = 0; q < U; ++q) t[q] = tri_idx[tb + min(q, nt - 1)];
#pragma unroll
        for (int q = 0; q < U; ++q) v[q] = reinterpret_cast<const Corners*>(tris)[t[q]];
    }
    int32_t lab[U];
#pragma unroll
    for (int j = 0; j < U; ++j) lab[j] = new_of_old[r[j]];
#pragma unroll
    for (int j = 0; j < U; ++j) {
        if (j < d) nbr[out + j] = lab[j];
        else r[j] = -1;
    }
#pragma unroll 1
    for (int32_t j = U; j < d; ++j) nbr[out + j] = new_of_old[nbr_idx[b + j]];
    // a triangle's fan entry; a vertex that repeats in the row is its last entry
    auto entry = [&](const Corners& c) -> uint32_t {
        const uint32_t p = c.v0 == o ? 0u : (c.v1 == o ? 1u : 2u);
        const int32_t x = p == 0 ? c.v1 : (p == 1 ? c.v2 : c.v0), y = p == 0 ? c.v2 : (p == 1 ? c.v0 : c.v1);
        uint32_t sx = 0, sy = 0;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            sx = r[j] == x ? static_cast<uint32_t>(j) : sx;
            sy = r[j] == y ? static_cast<uint32_t>(j) : sy;
        }
#pragma unroll 1
        for (int32_t j = U; j < d; ++j) {
            const int32_t w = nbr_idx[b + j];
            sx = w == x ? static_cast<uint32_t>(j) : sx;
            sy = w == y ? static_cast<uint32_t>(j) : sy;
        }
        return p | (sx << 2) | (sy << 9);
    };
    uint32_t e[U];
    int32_t c0 = 0, c1 = 0;
#pragma unroll
    for (int q = 0; q < U; ++q) {
        e[q] = 3u;   // no entry
        if (q < nt) e[q] = entry(v[q]);
        c0 += (e[q] & 3u) == 0u;
        c1 += (e[q] & 3u) == 1u;
    }
    auto corners = [&](int32_t q) -> Corners { return reinterpret_cast<const Corners*>(tris)[tri_idx[tb + q]]; };
    if (GROUP)
#pragma unroll 1
        for (int32_t q = U; q < nt; ++q) {
            const Corners c = corners(q);
            c0 += c.v0 == o;
            c1 += c.v0 != o && c.v1 == o;
        }
    int32_t at0 = fo, at1 = fo + c0, at2 = fo + c0 + c1;
    auto put = [&](uint32_t w) {
        const uint32_t p = w & 3u;
        const int32_t at = !GROUP || p == 0u ? at0 : (p == 1u ? at1 : at2);
        fan[at] = static_cast<uint16_t>(w);
        at0 += !GROUP || p == 0u;
        at1 += p == 1u;
        at2 += p == 2u;
    };
#pragma unroll
    for (int q = 0; q < U; ++q)
        if (q < nt) put(e[q]);
#pragma unroll 1
    for (int32_t q = U; q < nt; ++q) put(entry(corners(q)));
    if (GROUP)
        split[k] = nt < 0xFFFF ? static_cast<uint32_t>(c0) | (static_cast<uint32_t>(c0 + c1) << 16) : kFanUngrouped;
}

// Both buffers of the ping-pong pair start at the caller's positions (X1
// from label x1_from on), rounded to R (float for the single-precision form).
template <typename R>
__global__ __launch_bounds__(kBS) void k_init_coords(const double* __restrict__ coords,
                                                     const int32_t* __restrict__ perm, int32_t n, int soa,
                                                     R* __restrict__ X0, R* __restrict__ X1, int32_t x1_from)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (k >= n) return;
    const int64_t o = perm[k];
    const double2 p = *reinterpret_cast<const double2*>(coords + 2 * o);
    const R x = static_cast<R>(p.x), y = static_cast<R>(p.y);
    const bool both = k >= x1_from;
    if (soa) {
        X0[k] = x; X0[n + k] = y;
        if (both) X1[k] = x, X1[n + k] = y;
    } else {
        X0[2 * k] = x; X0[2 * k + 1] = y;
        if (both) X1[2 * k] = x, X1[2 * k + 1] = y;
    }
}

// Buffer src = X[src], or X[sweeps run % 2] when `runs` is given (Form A,
// read on the device so that the host need not wait for the sweep loop).
template <typename R>
__global__ __launch_bounds__(kBS) void k_unpermute(const R* __restrict__ X0, int src, const MeshState* __restrict__ runs,
                                                   const int32_t* __restrict__ perm, int32_t n, int soa,
                                                   double* __restrict__ out)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (k >= n) return;
    const R* X = X0 + 2 * static_cast<int64_t>(n) * (runs ? (runs->s & 1) : src);
    const int64_t o = perm[k];
    const R x = soa ? X[k] : X[2 * k], y = soa ? X[n + k] : X[2 * k + 1];
    *reinterpret_cast<double2*>(out + 2 * o) = make_double2(static_cast<double>(x), static_cast<double>(y));
}

__global__ __launch_bounds__(kBS) void k_unpermute_flags(const uint64_t* __restrict__ bits, int64_t words,
                                                         const int32_t* __restrict__ new_of_old, int32_t n,
                                                         int32_t n_free, int32_t iterations,
                                                         const MeshState* __restrict__ state, uint8_t* __restrict__ out)
{
    const int64_t nbytes = (static_cast<int64_t>(n) + 7) / 8;
    const int64_t g = static_cast<int64_t>(blockIdx.x) * kBS + threadIdx.x;
    if (g >= nbytes * iterations) return;
    const int32_t runs = state->s;
    const int64_t s = g / nbytes, B = g % nbytes;
    uint32_t byte = 0;
    if (s < runs) {
        for (int q = 0; q < 8; ++q) {
            const int64_t i = 8 * B + q;
            if (i >= n) break;
            const int32_t k = new_of_old[i];
            if (static_cast<uint32_t>(k) < static_cast<uint32_t>(n_free) && ((bits[s * words + k / 64] >> (k % 64)) & 1ull)) byte |= 1u << q;
        }
    }
    out[g] = static_cast<uint8_t>(byte);
}

}  // namespace

// Bits per axis of the Hilbert cells of the counting sort for n_free free
// nodes in nc colour classes: grown while a class still has about two nodes
// per cell or more, at most 2^25 buckets.  The bucket count stays below
// max(4 nc, 2 n_free).
int hilbert_bits(int64_t n_free, int nc)
{
    int bits = 1;
    while (bits < 12 && (static_cast<int64_t>(nc) << (2 * bits)) < n_free / 2 &&
           (static_cast<int64_t>(nc) << (2 * (bits + 1))) <= (int64_t(1) << 25))
        ++bits;
    return bits;
}

namespace {

// Bits per axis of the fixed nodes' cells: 2^6 of the free nodes' cells each
// while they are few (a boundary), and few nodes a cell where most of a mesh
// is fixed (1.2M nodes, 400 of them free, the others in 4 cells: setup 13.7
// ms; so 0.21).
int fixed_bits(int64_t n_fixed, int bits) { return std::max({bits - 3, hilbert_bits(n_fixed, 1) - 1, 0}); }

// Scratch bytes make_order takes for n nodes (at most 128 colour classes).
size_t order_bytes(int64_t n)
{
    // (and the fixed nodes' buckets: a 64th of the free ones', or half the fixed nodes)
    const int64_t nbk = std::max<int64_t>(4 * 128, 2 * n) + n / 2 + 16;
    return 3 * Arena::piece(4 * static_cast<size_t>(n + 1)) + 2 * Arena::piece(4 * static_cast<size_t>(nbk + 1)) + scan_bytes(std::max<int64_t>(n, nbk));
}

sl_status make_order(const SetupArgs& a, const sl_options& o, const uint8_t* bnd, int32_t n_free, const ValStats* vs,
                     const int32_t* color, int32_t n_colors, DevMesh& m, hipStream_t st, Arena& scratch,
                     PinnedPad& pad)
{
    const int32_t n = a.n;
    const int gb = div_up(n, kBS);
    const size_t mk = scratch.mark();
    int32_t *flag = nullptr, *pos = nullptr;
    sl_status r;
    if ((r = scratch.take(&flag, n)) || (r = scratch.take(&pos, static_cast<size_t>(n) + 1))) return r;
    int32_t* cs = m.color_start_h;
    cs[0] = 0;
    if (o.reorder == SL_REORDER_HILBERT && n_free > 0) {
        // bucket counting sort: (colour, Hilbert cell); order inside a bucket is arbitrary,
        // which no result depends on (rows and triangles keep their order).
        const int nc = color ? n_colors : 1;
        const int bits = hilbert_bits(n_free, nc);
        // the fixed nodes' buckets follow
        const int64_t nfree_bk = static_cast<int64_t>(nc) << (2 * bits);
        const int fbits = fixed_bits(n - n_free, bits);
        const int64_t nbk = nfree_bk + (int64_t(1) << (2 * fbits));
        int32_t *count = nullptr, *start = nullptr, *key = nullptr;
        if ((r = scratch.take(&count, nbk)) || (r = scratch.take(&start, nbk + 1)) || (r = scratch.take(&key, n)))
            return r;
        k_fill_i32<<<div_up(nbk, 256), 256, 0, st>>>(count, nbk, 0);
        k_bucket<<<gb, kBS, 0, st>>>(a.coords, bnd, color, n, bits, static_cast<int32_t>(nfree_bk), fbits, vs, key, count, flag);
        if ((r = scan_exclusive(count, start, nbk, st, &scratch))) return r;
        if (color) {
            // nc <= 128: the class starts fit the mesh's table and the pad
            k_tell<<<1, 64, 0, st>>>(start, nc + 1, int64_t(1) << (2 * bits), static_cast<int32_t*>(pad.p));
            SL_HIP(hipGetLastError());
            SL_HIP(hipStreamSynchronize(st));
            std::memcpy(cs, pad.p, sizeof(int32_t) * static_cast<size_t>(nc + 1));
        } else {
            cs[1] = n_free;
        }
        k_bucket_scatter<<<gb, kBS, 0, st>>>(n, key, flag, start, m.new_of_old, m.perm);
    } else if (n_free > 0) {
        // stable: free nodes (by colour class when coloured) in caller order
        const int nc = color ? n_colors : 1;
        int32_t base = 0;
        for (int c = 0; c < nc; ++c) {
            k_select<<<gb, kBS, 0, st>>>(bnd, color, c, 0, n, flag);
            if ((r = scan_exclusive(flag, pos, n, st, &scratch))) return r;
            k_place<<<gb, kBS, 0, st>>>(flag, pos, base, n, m.new_of_old, m.perm);
            int32_t cnt = 0;
            SL_HIP(hipMemcpyAsync(&cnt, pos + n, sizeof(int32_t), hipMemcpyDeviceToHost, st));
            SL_HIP(hipStreamSynchronize(st));
            base += cnt;
            cs[c + 1] = base;
        }
    }
    if (n_free < n && (o.reorder != SL_REORDER_HILBERT || n_free == 0)) {
        k_select<<<gb, kBS, 0, st>>>(bnd, nullptr, 0, 1, n, flag);
        if ((r = scan_exclusive(flag, pos, n, st, &scratch))) return r;
        k_place<<<gb, kBS, 0, st>>>(flag, pos, n_free, n, m.new_of_old, m.perm);
    }
    scratch.rewind(mk);
    SL_HIP(hipGetLastError());
    return SL_OK;
}

}  // namespace

sl_status scan_exclusive(const int32_t* in, int32_t* out, int64_t n, hipStream_t st, Arena* scratch)
{
    const size_t mk = scratch ? scratch->mark() : 0;
    const sl_status r = scan_rec(in, out, n, out + n, st, scratch);
    if (scratch) scratch->rewind(mk);
    return r;
}

void devmesh_free(DevMesh& m, hipStream_t st)
{
    flow_mesh_free(m.flow, st);
    block_give(m.block, st);
    m.perm = m.new_of_old = m.row_ptr = m.nbr = m.fan_ptr = nullptr;
    m.fan = nullptr;
    m.X[0] = m.X[1] = nullptr;
    m.work = nullptr;
    m.tile_data = nullptr;
}

// Nodes per tile: Form A's tuned or default size; a colour-class tile
// (Form B) holds 256 unless asked otherwise (its halo is several times
// longer than a Form A tile's, and 512-node class tiles leave room for only
// two work-groups per CU).
// Colour-class tiles of 512 nodes from this many mesh nodes up, else 256.
// A larger class tile re-reads fewer halo positions per own node, but gives
// fewer tiles: on the 4096^2 grid 512 took 1.04 ms per sweep against 1.11
// (256) and 1.36 (128), on the 1024^2 grid 0.118 against 0.130 ms; on
// Delaunay meshes of 30K and 100K points 256 was faster (0.078 and 0.080
// against 0.096 and 0.100 ms).
constexpr int32_t kLargeClassMesh = 1 << 20;

// Form A tiles of 512 nodes from this many mesh nodes up, else 256, when
// neither the options nor sl_autotune fix the size (batches, servers and
// handles fix it before setup, so that one work list has one size).  A
// small mesh's sweep is one round of tiles, so smaller tiles finish sooner:
// Delaunay meshes of 10K, 30K and 100K points took 8.3, 9.4 and 11.2 us per
// sweep with 256 against 10.4, 10.8 and 12.1 with 512; the 1024^2 grid
// 0.033 ms with either.
constexpr int32_t kLargeTileMesh = 1 << 19;

int32_t tile_size_for(const sl_options& o, int32_t n)
{
    if (o.form == SL_JACOBI) {
        if (o.tile_nodes || tuned_shape().tile_nodes) return resolve_tile_nodes(o);
        return n >= kLargeTileMesh ? 512 : 256;
    }
    if (o.tile_nodes) return o.tile_nodes;
    return n >= kLargeClassMesh ? 512 : 256;
}

// Whether setup aims for the tile path, decided before validation as
// setup_mesh decides it.
static bool wants_tiles(const sl_options& o, bool resident, bool class_tiles_ok)
{
    if (o.kernel == SL_KERNEL_NODE || o.kernel == SL_KERNEL_LANES || resident) return false;
    // Form B takes its colour-class tiles on request only: the node kernel
    // sweeps it faster (each class phase gathers its neighbours through L2
    // instead of staging halos several times longer than the class tile)
    return o.form == SL_JACOBI || (o.kernel == SL_KERNEL_TILE && class_tiles_ok && o.precision == SL_F64);
}

size_t mesh_block_bytes(int32_t n, int64_t nnz, int64_t ninc, const sl_options& o, bool class_tiles_ok)
{
    // the same kernel choice as setup_mesh makes before validation
    const bool resident = o.kernel == SL_KERNEL_RESIDENT ||
                          (o.kernel == SL_KERNEL_AUTO && o.form == SL_INPLACE_COLORED &&
                           resident_fits(n, nnz, ninc, o.form == SL_INPLACE_COLORED));
    const bool want_tiles = wants_tiles(o, resident, class_tiles_ok);
    const size_t rb = o.precision == SL_F32 ? 4 : 8;
    const size_t un = static_cast<size_t>(n);
    size_t pb = 2 * Arena::piece(4 * un) + 2 * Arena::piece(4 * (un + 1)) + Arena::piece(4 * un * rb);
    pb += want_tiles ? tile_bytes(n, nnz, ninc, tile_size_for(o, n), o.form != SL_JACOBI)
                     : Arena::piece(4 * static_cast<size_t>(nnz)) + Arena::piece(2 * static_cast<size_t>(ninc)) +
                           Arena::piece(4 * un);
    return pb;
}

// Lanes per node of the node checks: on meshes that leave most of the device
// idle a node's checks are a serial chain of some twenty trips to memory,
// which four lanes shorten (4K nodes 12.5 -> 8.9 us, 46K refined ones 31 ->
// 14); with the device full, two lanes, and at many millions of nodes one
// (1M shuffled nodes 130 -> 125 us with two, 2.2M 198 -> 176; 16.8M 572 ->
// 579).
static int val_lanes(int32_t n) { return n <= (1 << 18) ? 4 : (n <= (1 << 22) ? 2 : 1); }

// Work-groups of the node checks, each with a slot for its statistics.
int val_groups(int32_t n) { return std::min(div_up(static_cast<int64_t>(n) * val_lanes(n), kBS), 8192); }

size_t setup_scratch_bytes(int32_t n)
{
    const size_t un = static_cast<size_t>(n);
    const size_t rows_bytes = 2 * Arena::piece(4 * un) + 2 * scan_bytes(n);
    return Arena::piece(sizeof(ValStats)) + Arena::piece(sizeof(ValStats) * static_cast<size_t>(val_groups(n))) +
           Arena::piece(4 * un) +
           std::max({order_bytes(n), rows_bytes, tile_scratch_bytes(),
                     2 * Arena::piece(4 * un) + Arena::piece(4 * (kColorRounds + 2))});   // the colouring's lists
}

// Queues the checks of one mesh's arrays; *vs receives the statistics, part a slot per work-group of k_validate_nodes.  incidence:
// also whether the incidence rows agree (VI_INCIDENCE).
static void queue_validation(const ValArgs& a, bool incidence, ValStats* vs, ValStats* part, hipStream_t st)
{
    const int gb = val_groups(a.n);
    const int lanes = val_lanes(a.n);
    if (lanes == 4) k_validate_nodes<4><<<gb, kBS, 0, st>>>(a, part);
    else if (lanes == 2) k_validate_nodes<2><<<gb, kBS, 0, st>>>(a, part);
    else k_validate_nodes<1><<<gb, kBS, 0, st>>>(a, part);
    k_validate_fold<<<1, 1024, 0, st>>>(part, gb, a, vs);
    const int gt = std::min(std::max(div_up(a.n_tris, kBS), div_up(a.n, kBS)), 8192);   // (n > 0)
    if (incidence && a.ninc != 0)
        k_validate_rest<true><<<gt, kBS, 0, st>>>(a.tris, a.n_tris, a.n, a.boundary, a.nbr_ptr, a.nbr_idx, a.tri_ptr,
                                                  a.tri_idx, a.ninc, vs);
    else
        k_validate_rest<false><<<gt, kBS, 0, st>>>(a.tris, a.n_tris, a.n, a.boundary, a.nbr_ptr, a.nbr_idx, a.tri_ptr,
                                                   a.tri_idx, a.ninc, vs);
}

// SL_OK, or the error that the validation's bits stand for.
sl_status validation_status(uint32_t err, const sl_options& o)
{
    if (err & (VE_PTR | VE_RANGE | VE_COORD)) {
        std::string msg = "invalid input:";
        if (err & VE_PTR) msg += " CSR offsets not monotone or out of range;";
        if (err & VE_RANGE) msg += " node or triangle id out of range;";
        if (err & VE_COORD)
            msg += o.precision == SL_F32 ? " coordinate not finite or of magnitude >= 2^61 (single precision);"
                                         : " coordinate not finite or of magnitude >= 2^500;";
        return fail(SL_EINVAL, msg);
    }
    if (err & kValErrors & ~(o.form == SL_JACOBI ? VE_ASYM : 0u)) {
        std::string msg = "invalid topology:";
        if (err & VE_SELF) msg += " node lists itself as a neighbour;";
        if (err & VE_TRIREP) msg += " triangle with a repeated vertex;";
        if (err & VE_NOTIN) msg += " incident triangle does not contain its node;";
        if (err & VE_MISSING) msg += " triangle vertex missing from the node's neighbour row;";
        if (err & VE_EMPTY) msg += " free node without neighbours;";
        if (err & VE_VALENCE) msg += " free node with more than 127 neighbours;";
        if (err & VE_ASYM) msg += " neighbour rows are not symmetric (needed by the coloured form);";
        return fail(SL_ETOPO, msg);
    }
    return SL_OK;
}

sl_status setup_mesh(const SetupArgs& a, const sl_options& o, DevMesh& m, int32_t mesh, hipStream_t st)
{
    const int32_t n = a.n;
    m.n = n;
    m.n_tris = a.n_tris;
    m.layout = o.layout;
    m.precision = o.precision;
    sl_status r;
    // the resident kernel when asked for, and automatically for Form B
    // (faster there than the node kernel's launch per colour class),
    // checked against bounds known before validation (check_options has
    // restricted it to f64; Form B is f64 only)
    const bool res_fit = resident_fits(n, a.nnz, a.ninc, o.form == SL_INPLACE_COLORED);
    if (o.kernel == SL_KERNEL_RESIDENT && !res_fit) return fail(SL_EINVAL, "mesh too large for the resident kernel");
    m.resident = o.kernel == SL_KERNEL_RESIDENT ||
                 (o.kernel == SL_KERNEL_AUTO && o.form == SL_INPLACE_COLORED && res_fit);
    m.lane_width = o.kernel == SL_KERNEL_LANES ? resolve_lane_width(o) : 0;
    const bool want_tiles = wants_tiles(o, m.resident, m.class_tiles_ok);
    const size_t un = static_cast<size_t>(n);
    // Two reservations: the mesh's own arrays, sized from bounds known before
    // validation (n >= free nodes, a.nnz and a.ninc >= their rows and fans),
    // and the setup's temporaries, given back when setup ends.
    Arena persist, scratch;
    const size_t pb = mesh_block_bytes(n, a.nnz, a.ninc, o, m.class_tiles_ok);
    const size_t sb = setup_scratch_bytes(n);
    const int gb = div_up(n, kBS);
    if (m.carve) {
        if (m.carve_bytes < pb) return fail(SL_EINVAL, "internal: mesh region smaller than its arrays");
        persist.adopt(m.carve, pb);
    } else {
        if ((r = persist.reserve(pb, st))) return r;
        m.block = persist.base;
    }
    if (m.scratch_carve) {
        if (m.scratch_carve_bytes < sb) return fail(SL_EINVAL, "internal: setup region smaller than its temporaries");
        scratch.adopt(m.scratch_carve, sb);
    } else if ((r = scratch.reserve(sb, st))) {
        return r;
    }
    struct GiveBack {
        Arena& ar;
        hipStream_t st;
        ~GiveBack() { ar.release(st); }
    } give_back{scratch, st};

    // ---- validation
    ValStats *vs = nullptr, *vpart = nullptr;
    if ((r = scratch.take(&vs, 1)) || (r = scratch.take(&vpart, val_groups(n)))) return r;
    ValArgs va{a.coords, n, a.nbr_ptr, a.nbr_idx, a.tri_ptr, a.tri_idx, a.tris, a.n_tris, a.boundary,
               a.nnz, a.ninc, o.form == SL_INPLACE_COLORED || m.want_flow, o.precision == SL_F32 ? 0x1p61 : 0x1p500};
    PinnedPad pad;   // what the host has to know, written by the kernels
    if ((r = pad.init())) return r;
    ValStats h{};
    if (m.checked) {
        h = *m.checked;
        k_put_stats<<<1, 64, 0, st>>>(vs, h);
        SL_HIP(hipGetLastError());
    } else {
        queue_validation(va, want_tiles && o.form == SL_JACOBI, vs, vpart, st);
        SL_HIP(hipGetLastError());
        k_tell<<<1, 64, 0, st>>>(reinterpret_cast<const int32_t*>(vs), sizeof(ValStats) / 4, 1, static_cast<int32_t*>(pad.p));
        SL_HIP(hipGetLastError());
        SL_HIP(hipStreamSynchronize(st));
        std::memcpy(&h, pad.p, sizeof(h));
    }
    if ((r = validation_status(h.err, o))) return r;
    m.n_free = h.n_free;
    m.t_setup = h.t0;
    m.max_deg = h.max_deg_free;
    m.max_inc = h.max_inc_free;

    if ((r = persist.take(&m.perm, n)) || (r = persist.take(&m.new_of_old, n))) return r;

    // ---- colouring (coloured form)
    int32_t* color = nullptr;
    m.n_colors = 0;
    if (o.form == SL_INPLACE_COLORED && m.n_free > 0) {
        if ((r = scratch.take(&color, n))) return r;
        // rounds over a shrinking list of the uncoloured free nodes; words:
        // the largest colour, then the lists' lengths, a place per round
        // between two looks
        const size_t cmark = scratch.mark();
        int32_t *list = nullptr, *next = nullptr, *words = nullptr;
        if ((r = scratch.take(&list, m.n_free)) || (r = scratch.take(&next, m.n_free)) ||
            (r = scratch.take(&words, kColorRounds + 2)))
            return r;
        k_fill_i32<<<1, 64, 0, st>>>(words, kColorRounds + 2, 0);
        k_fill_i32<<<div_up(n, 256), 256, 0, st>>>(color, n, -1);
        // rounds read their list's length on the device; the host looks at
        // it every kColorRounds rounds (rounds past the last are empty), and
        // sizes the launches by the last length it saw
        int32_t left = n, mx = -1;
        for (int round = 0; left > 0; round += kColorRounds) {
            if (round > m.n_free) return fail(SL_EDEVICE, "colouring made no progress");
            if (round > 0) {
                k_tell<<<1, 64, 0, st>>>(words + 1 + kColorRounds, 1, 1, words + 1);
                k_fill_i32<<<1, 64, 0, st>>>(words + 2, kColorRounds, 0);
            }
            for (int k = 0; k < kColorRounds; ++k) {
                k_color_round<<<div_up(left, kColorBS), kColorBS, 0, st>>>(a.nbr_ptr, a.nbr_idx, a.boundary, color,
                                                                          round + k > 0 ? list : nullptr, n,
                                                                          round + k, words + 1 + k, next, words);
                std::swap(list, next);
            }
            k_tell<<<1, 64, 0, st>>>(words, kColorRounds + 2, 1, static_cast<int32_t*>(pad.p));
            SL_HIP(hipGetLastError());
            SL_HIP(hipStreamSynchronize(st));
            left = static_cast<const int32_t*>(pad.p)[1 + kColorRounds];
            mx = static_cast<const int32_t*>(pad.p)[0];
        }
        scratch.rewind(cmark);
        m.n_colors = mx + 1;
        if (m.n_colors > 128) return fail(SL_ETOPO, "more than 128 colour classes");
        // the resident kernel holds a bounded number of classes: an automatic
        // choice falls back to the node kernel, an explicit one fails
        if (m.resident && m.n_colors > kResidentClasses) {
            if (o.kernel == SL_KERNEL_RESIDENT)
                return fail(SL_EINVAL, "the resident kernel holds at most " + std::to_string(kResidentClasses) +
                                           " colour classes");
            m.resident = false;
        }
    }

    // ---- node order
    if ((r = make_order(a, o, a.boundary, m.n_free, vs, color, m.n_colors, m, st, scratch, pad))) return r;

    // ---- rows and fans of free nodes
    if ((r = persist.take(&m.row_ptr, static_cast<size_t>(m.n_free) + 1)) ||
        (r = persist.take(&m.fan_ptr, static_cast<size_t>(m.n_free) + 1)))
        return r;
    const size_t mk = scratch.mark();
    int32_t *deg = nullptr, *inc = nullptr;
    if ((r = scratch.take(&deg, m.n_free)) || (r = scratch.take(&inc, m.n_free))) return r;
    const int gf = div_up(m.n_free > 0 ? m.n_free : 1, kBS);
    const int gt = div_up(m.n_free > 0 ? m.n_free : 1, kScanTile);
    int32_t* dsum = nullptr;
    if ((r = scratch.take(&dsum, 2 * static_cast<size_t>(gt)))) return r;
    k_degree_sums<<<gt, kBS, 0, st>>>(m.perm, m.n_free, a.nbr_ptr, a.tri_ptr, deg, inc, dsum);
    if (gt > kSumsInPlace) k_scan_offsets<<<2, kSumsBS, 0, st>>>(dsum, gt);
    k_offset_tiles<<<dim3(gt, 2), kBS, 0, st>>>(deg, inc, m.n_free, dsum, gt > kSumsInPlace, m.row_ptr, m.fan_ptr);
    SL_HIP(hipGetLastError());
    scratch.rewind(mk);
    m.nnz_free = h.nnz_free;     // the offsets' totals, counted by the validation
    m.ninc_free = h.ninc_free;
    // coordinate buffers: one block, X[1] right after X[0], in the sweep's precision
    const size_t n2 = 2 * un;
    const int32_t x1_from = m.one_buffer ? m.n_free : 0;
    if (m.precision == SL_F32) {
        float* xf = nullptr;
        if ((r = persist.take(&xf, 2 * n2))) return r;
        m.X[0] = xf;
        m.X[1] = xf + n2;
        k_init_coords<float><<<gb, kBS, 0, st>>>(a.coords, m.perm, n, o.layout == SL_SOA, xf, xf + n2, x1_from);
    } else {
        double* xd = nullptr;
        if ((r = persist.take(&xd, 2 * n2))) return r;
        m.X[0] = xd;
        m.X[1] = xd + n2;
        k_init_coords<double><<<gb, kBS, 0, st>>>(a.coords, m.perm, n, o.layout == SL_SOA, xd, xd + n2, x1_from);
    }
    // tile path for Form A (which needs consistent incidence rows: a tile
    // lists a triangle once and scores it for every own vertex) and, on
    // colour-class tiles, for Form B (each listed triangle has one own
    // vertex, whose row listed it); the node path's rows and fans otherwise
    const bool jacobi = o.form == SL_JACOBI;
    const bool tiles_ok = !jacobi || (h.err & VI_INCIDENCE) == 0;
    if (want_tiles && tiles_ok &&
        (r = build_tiles(a, m, tile_size_for(o, n), mesh, st, persist, scratch, !jacobi)))
        return r;
    // the flow path besides the tiles, for meshes whose rows are symmetric
    if (m.want_flow && m.tile_nodes > 0 && (h.err & VE_ASYM) == 0 && (r = flow_mesh_build(a, m, st))) return r;
    if (m.tile_nodes == 0 && m.precision == SL_F32 && m.n_free > 0)
        return fail(SL_EINVAL, tiles_ok ? "single precision needs the tile path, and this mesh does not fit it"
                                        : "single precision needs the tile path, which needs every free vertex of "
                                          "a listed triangle to list it too");
    if (m.tile_nodes == 0) {
        // (a mesh that did not fit the tile path gave the tile arrays' room back,
        // which bounds this)
        const bool group = m.n_free > 0 && m.n_free < kGroupFansBelow && m.max_deg <= 8 && !m.resident &&
                           m.lane_width == 0;
        if ((r = persist.take(&m.nbr, m.nnz_free)) || (r = persist.take(&m.fan, m.ninc_free)) ||
            (group && (r = persist.take(&m.fan_split, m.n_free))))
            return r;
        if (m.n_free > 0)
            (group ? k_rows_fans<true> : k_rows_fans<false>)<<<gf, kBS, 0, st>>>(
                m.perm, m.new_of_old, m.n_free, a.nbr_ptr, a.nbr_idx, a.tri_ptr, a.tri_idx, a.tris, m.row_ptr, m.nbr,
                m.fan_ptr, m.fan, m.fan_split);
    }
    SL_HIP(hipGetLastError());
    return SL_OK;
}

sl_status unpermute_coords(const DevMesh& m, int src, double* coords_out, hipStream_t st, const MeshState* runs)
{
    if (m.precision == SL_F32)
        k_unpermute<float><<<div_up(m.n, kBS), kBS, 0, st>>>(static_cast<const float*>(m.X[0]), src, runs, m.perm,
                                                              m.n, m.layout == SL_SOA, coords_out);
    else
        k_unpermute<double><<<div_up(m.n, kBS), kBS, 0, st>>>(static_cast<const double*>(m.X[0]), src, runs, m.perm,
                                                               m.n, m.layout == SL_SOA, coords_out);
    SL_HIP(hipGetLastError());
    return SL_OK;
}

sl_status unpermute_flags_raw(const uint64_t* bits, int64_t words, const int32_t* new_of_old, int32_t n, int32_t n_free,
                              int32_t iterations, const MeshState* state, uint8_t* out, hipStream_t st)
{
    const int64_t total = (static_cast<int64_t>(n) + 7) / 8 * iterations;
    if (total == 0) return SL_OK;
    k_unpermute_flags<<<div_up(total, kBS), kBS, 0, st>>>(bits, words, new_of_old, n, n_free, iterations, state, out);
    SL_HIP(hipGetLastError());
    return SL_OK;
}

sl_status unpermute_flags(const DevMesh& m, const uint64_t* bits, int32_t iterations, const MeshState* state,
                          uint8_t* out, hipStream_t st)
{
    return unpermute_flags_raw(bits, (static_cast<int64_t>(m.n_free) + 63) / 64, m.new_of_old, m.n, m.n_free,
                               iterations, state, out, st);
}

sl_status queue_flow_order(const SetupArgs& a, const sl_options& o, const FlowOrder& f, Arena& scratch, hipStream_t st)
{
    const int32_t n = a.n;
    const int gb = div_up(n, kBS);
    ValArgs va{a.coords, n, a.nbr_ptr, a.nbr_idx, a.tri_ptr, a.tri_idx, a.tris, a.n_tris, a.boundary,
               a.nnz, a.ninc, 1, 0x1p500};
    queue_validation(va, o.form == SL_JACOBI, f.vs, f.part, st);
    // (keys and ranks are in range whatever the checks find)
    k_bucket<<<gb, kBS, 0, st>>>(a.coords, a.boundary, nullptr, n, f.bits, -1, 0, f.vs, f.key, f.count, f.rank);
    sl_status r = scan_exclusive(f.count, f.start, int64_t(1) << (2 * f.bits), st, &scratch);
    if (r) return r;
    k_flow_scatter<<<gb, kBS, 0, st>>>(a.boundary, n, f.key, f.rank, f.start, f.new_of_old, f.perm);
    SL_HIP(hipGetLastError());
    return SL_OK;
}

}  // namespace sl
