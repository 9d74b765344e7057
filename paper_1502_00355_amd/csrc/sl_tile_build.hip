// Tile build of the tile sweeps.
//
// Form A (Jacobi): the free nodes (device order: Hilbert cells) are cut into
// tiles of T consecutive labels.  Form B (coloured, in place): each colour
// class (contiguous in device order, Hilbert cells inside) is cut into tiles
// of T consecutive labels.  The sweeps run one work-group per tile.  The
// tiles are built on the device: one work-group per tile collects the halo
// (every node an own node reads) in an LDS hash set and rewrites the rows in
// tile-local indices (own nodes 0..T-1, halo nodes T..T+H-1); a Form A tile
// lists its incident triangles in local indices, a colour-class tile gets
// one fan entry per incidence instead.
#include <algorithm>
#include <climits>
#include <cstdlib>
#include <cstring>

#include "sl_common.h"

namespace sl {

namespace {

constexpr int kTileMaxDeg = 16;   // row entries, and incidences, per own node on average over a tile
constexpr int kRowU = 8;          // row entries, and incidences, of a node held in registers by the tile build
constexpr int kClassBS = 512;
constexpr int kClassU = 4;        // entries a work-item of the class build takes per chunk: their loads are in flight together

// ------------------------------------------------------ block primitives --

template <int BS>
__device__ int block_excl_scan(int v, int* total, int* s_warp)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(x, off);
        if (lane >= off) x += t;
    }
    if (lane == 63) s_warp[w] = x;
    __syncthreads();
    int base = 0, tot = 0;
    for (int q = 0; q < BS / 64; ++q) {
        const int c = s_warp[q];
        if (q < w) base += c;
        tot += c;
    }
    __syncthreads();
    *total = tot;
    return base + x - v;
}

// Open-addressing set of caller node ids in LDS (-1 = empty slot), probed
// linearly from a multiplicative hash: the ids are runs of grid rows, ranges
// of a shuffled order, or anything else, and their low bits may all be alike.
// Probing stops after HS slots, so a full table reports failure (-1) instead
// of looping.
template <int HS>
__device__ __forceinline__ int set_home(int32_t key)
{
    return static_cast<int>((static_cast<uint32_t>(key) * 2654435761u) >> (32 - __builtin_ctz(HS)));
}

// *won: the key was not there before.
template <int HS>
__device__ __forceinline__ int set_insert(int32_t* tab, int32_t key, bool* won)
{
    int s = set_home<HS>(key);
    *won = false;
#pragma unroll 1
    for (int p = 0; p < HS; ++p) {
        const int32_t cur = tab[s];
        if (cur == key) return s;
        if (cur == -1) {
            const int32_t prev = atomicCAS(&tab[s], -1, key);
            *won = prev == -1;
            if (prev == -1 || prev == key) return s;
        }
        s = (s + 1) & (HS - 1);
    }
    return -1;
}

template <int HS>
__device__ int set_find(const int32_t* tab, int32_t key)
{
    int s = set_home<HS>(key);
#pragma unroll 1
    for (int p = 0; p < HS; ++p) {
        const int32_t cur = tab[s];
        if (cur == key) return s;
        if (cur == -1) return -1;
        s = (s + 1) & (HS - 1);
    }
    return -1;
}

// ------------------------------------------------------------ tile build --

struct TileBuildArgs {
    const int32_t* perm;
    const int32_t* new_of_old;
    const int32_t* nbr_ptr;
    const int32_t* nbr_idx;
    const int32_t* tri_ptr;
    const int32_t* tri_idx;
    const int32_t* tris;
    const int32_t* row_ptr;    // device-order rows of the free nodes
    const int32_t* fan_ptr;    // device-order incidence offsets of the free nodes
    int32_t n_free;
    int32_t mesh;              // MeshState index written into the descriptors
    int64_t n;
    const void* X;
    unsigned char* data;       // tile k's record at tile_record(k): row offsets, halo, rows, triangles
    TileWork* work;            // [n_tiles]
    int32_t* err;
    // 0: tile k holds free nodes [k T, k T + T).  Else colour-class tiles:
    // class c (device labels [cls_start[c], cls_start[c+1])) is cut into
    // tiles [cls_tile[c], cls_tile[c+1]) of T consecutive labels, the last
    // one of a class possibly shorter
    int32_t n_class;
    int32_t cls_start[kMaxTileClasses + 1];
    int32_t cls_tile[kMaxTileClasses + 1];
};

__host__ __device__ __forceinline__ int64_t align16(int64_t b) { return (b + 15) & ~int64_t(15); }

// Byte offset of tile k's record, from the row and incidence offsets of its
// first node.  A record holds T + 1 u16 row starts (node i's row is entries
// start[i] .. start[i+1] of the rows), then room for len halo ids (len = the
// tile's row entries; the halo is never longer), the rows (len rounded up to
// 4 u16), and flen triangle words (flen = its incidences, an upper bound of
// its triangles), each part 16-byte aligned: at most 2T + 6 len + 8 flen +
// 48 bytes, which the next record's offset leaves.  One record per tile
// keeps the static data a tile reads in one stream.
__host__ __device__ __forceinline__ int64_t tile_record(int32_t row_start, int32_t fan_start, int32_t tile, int T)
{
    return static_cast<int64_t>(tile) * (2 * T + 64) +
           align16(6 * static_cast<int64_t>(row_start) + 8 * static_cast<int64_t>(fan_start));
}
__host__ __device__ __forceinline__ int64_t halo_at(int T) { return align16(2 * static_cast<int64_t>(T) + 2); }

// A colour-class tile's record holds T + 1 u16 row starts, T + 1 u16 fan
// starts (node i's fan entries are start[i] .. start[i+1]), T u32 splits of
// each fan by stored position (low half: entries with p = 0, high half:
// those with p <= 1), room for len halo ids, the rows (len rounded up to 4
// u16) and flen u16 fan entries, each part 16-byte aligned: at most 8T +
// 6 len + 2 flen + 100 bytes.
__host__ __device__ __forceinline__ int64_t class_record(int32_t row_start, int32_t fan_start, int32_t tile, int T)
{
    return static_cast<int64_t>(tile) * (8 * T + 128) +
           align16(6 * static_cast<int64_t>(row_start) + 2 * static_cast<int64_t>(fan_start));
}
__host__ __device__ __forceinline__ int64_t class_halo_at(int T) { return 2 * halo_at(T) + align16(4 * static_cast<int64_t>(T)); }

// Writes the R words of s_w grouped by which of their vertices are own nodes
// (indices below T): all three first, then the patterns with two, then with
// one, in the order of s_w inside a group.  Each of the BS work-items takes a
// contiguous segment; its counts per group are packed 16 bits each (R is
// below 2^16).
template <int T, int BS>
__device__ __forceinline__ void group_words(const uint64_t* s_w, int R, uint64_t* __restrict__ out,
                                            uint64_t (*s_cnt)[BS / 64])
{
    // rank of each own-vertex pattern (bit r: vertex r is own)
    constexpr uint32_t kRank = (0u << 28) | (1u << 12) | (2u << 20) | (3u << 24) | (4u << 4) | (5u << 8) |
                               (6u << 16) | (7u << 0);
    auto rank = [&](uint64_t w) -> uint32_t {
        const uint32_t lo = static_cast<uint32_t>(w), hi = static_cast<uint32_t>(w >> 32);
        const uint32_t p = ((lo & 0xFFFFu) < T) | (((lo >> 16) < T) << 1) | ((hi < T) << 2);
        return (kRank >> (4u * p)) & 7u;
    };
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int per = (R + BS - 1) / BS, b = min(R, tid * per), e = min(R, b + per);
    uint64_t cnt[2] = {0, 0};
    for (int j = b; j < e; ++j) {
        const uint32_t k = rank(s_w[j]);
        const uint64_t one = 1ull << (16u * (k & 3u));
        cnt[0] += k < 4u ? one : 0;
        cnt[1] += k < 4u ? 0 : one;
    }
    uint64_t at[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        uint64_t x = cnt[c];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t y = static_cast<uint64_t>(__shfl_up(static_cast<unsigned long long>(x), off));
            if (lane >= off) x += y;
        }
        if (lane == 63) s_cnt[c][wv] = x;
        at[c] = x - cnt[c];
    }
    __syncthreads();
    uint64_t tot[2] = {0, 0};
#pragma unroll
    for (int q = 0; q < BS / 64; ++q)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint64_t x = s_cnt[c][q];
            if (q < wv) at[c] += x;
            tot[c] += x;
        }
    uint32_t base = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        at[k >> 2] += static_cast<uint64_t>(base) << (16 * (k & 3));
        base += static_cast<uint32_t>(tot[k >> 2] >> (16 * (k & 3))) & 0xFFFFu;
    }
    for (int j = b; j < e; ++j) {
        const uint64_t w = s_w[j];
        const uint32_t k = rank(w), sh = 16u * (k & 3u);
        out[((k < 4u ? at[0] : at[1]) >> sh) & 0xFFFFu] = w;
        at[0] += k < 4u ? 1ull << sh : 0;
        at[1] += k < 4u ? 0 : 1ull << sh;
    }
}

// One work-group per Form A tile, one work-item per own node, in one pass:
// every output of tile k goes to a place fixed by the row and incidence
// offsets of its first node, so no tile needs another's counts.
//   Halo: every neighbour of an own node that is not own, once, numbered by
//   the work-item that first put it into the LDS set: in the order of the own
//   nodes, so that neighbouring entries are neighbours in memory (local
//   index T + number).
//   Rows: the tile's neighbour rows in local indices, one segment padded to
//   4 entries.
//   Triangles: each triangle incident to an own node, listed once per tile,
//   by its own vertex of smallest label, grouped by which of its vertices are
//   own nodes (all three first, then the patterns with two, then with one),
//   in incidence order inside a group.  The sweep evaluates a vertex's
//   candidate quality only for own vertices; with the list grouped, the lanes
//   of a wave mostly agree on which of the three evaluations to skip.
// Neither the halo order nor the triangle order changes a result: sums run
// over rows, minima are exact.
// The set is keyed by caller ids, own nodes included, so only the halo's
// device labels are gathered; a triangle's vertices are found among the
// node's own row, of which kRowU entries are held in registers (two compares
// per entry), the others through the set.  A triangle then is 26 bits
// (position, two local indices) and kRowU of them wait in registers for the
// scan of the counts; longer fans, and triangles with a vertex beyond the
// row's registers, are read again in a rolled loop.  It is bound by its
// chains of dependent loads (node -> offsets -> row and fan -> triangles),
// which the 32 waves of a CU hide for each other, and on a mesh in arbitrary
// numbering by the cache lines those touch (1M nodes: about 10 lines a node,
// 7 TB/s).  With the label of every row entry and every triangle vertex
// gathered instead, entries walked as flat ranges and the grouping in a
// launch of its own it took 435 us on a shuffled 1024 x 1024 grid (now 135),
// 408 on a 3.1M-node annulus (169), 1727 on the 4096 x 4096 grid (924).  No
// global load or store stands in a branch that its neighbours' waits would
// serialise: the halo goes through LDS (970 us without that at 4096 x 4096).
template <int T>
__global__ __launch_bounds__(T) void k_tile_build(TileBuildArgs a)
{
    constexpr int HS = 8 * T, CAP = T * kTileMaxDeg, U = kRowU;
    __shared__ alignas(8) int32_t htab[HS];
    __shared__ uint16_t hidx[HS];        // the local index of each slot's node
    __shared__ int32_t s_warp[T / 64];
    __shared__ uint64_t s_cnt[2][T / 64];
    __shared__ int32_t s_halo[4 * T];    // the halo's caller ids
    __shared__ int32_t s_full;
    static_assert(5 * T <= 4096, "local indices of 12 bits");
    const int tid = threadIdx.x;
    const int tile = blockIdx.x;
    const int32_t k0 = tile * T;
    const int nown = min(T, a.n_free - k0);
    const int32_t rb = a.row_ptr[k0], fb = a.fan_ptr[k0];
    const int32_t len = a.row_ptr[k0 + nown] - rb, flen = a.fan_ptr[k0 + nown] - fb;
    if (len > CAP || flen > CAP) {   // denser than the halo set is meant for: the mesh takes the node path
        if (tid == 0) atomicOr(a.err, 2);
        return;
    }
    const bool live = tid < nown;
    const int own = min(tid, nown - 1);
    const int32_t o = a.perm[k0 + own];
    const int32_t rs = a.row_ptr[k0 + own] - rb, fs = a.fan_ptr[k0 + own] - fb;
    const int deg0 = a.row_ptr[k0 + own + 1] - rb - rs, deg = live ? deg0 : 0;   // (a free node's row is not empty)
    const int inc = live ? a.fan_ptr[k0 + own + 1] - fb - fs : 0;
    const int32_t* const row = a.nbr_idx + a.nbr_ptr[o];
    const int32_t* const fan = a.tri_idx + a.tri_ptr[o];
    for (int s = tid; s < HS; s += T) htab[s] = -1;
    if (tid == 0) s_full = 0;
    int32_t r[U];
#pragma unroll
    for (int q = 0; q < U; ++q) r[q] = row[min(q, deg0 - 1)];
    int32_t t[U];
    if (inc > 0) {
#pragma unroll
        for (int q = 0; q < U; ++q) t[q] = fan[min(q, inc - 1)];
    }
    __syncthreads();
    if (live) {
        bool won;
        hidx[set_insert<HS>(htab, o, &won)] = static_cast<uint16_t>(tid);
    }
    __syncthreads();

    // ---- node set: the slots of the entries beyond the registers are parked
    // in the row part of the record until the slots have local indices
    unsigned char* rec = a.data + tile_record(rb, fb, tile, T);
    uint16_t* rr = reinterpret_cast<uint16_t*>(rec);
    int32_t* halo = reinterpret_cast<int32_t*>(rec + halo_at(T));
    const int32_t len4 = (len + 3) & ~3;
    const int64_t seg_at = align16(halo_at(T) + 4 * static_cast<int64_t>(len));
    uint16_t* const seg = reinterpret_cast<uint16_t*>(rec + seg_at);
    constexpr uint32_t kWon = 0x8000u;   // in a parked slot: the entry is the halo node's first
    bool full = false;
    int wins = 0;
    uint32_t sl[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        sl[q] = 0;
        if (q >= deg) {
            r[q] = -1;
            continue;
        }
        bool won;
        const int s = set_insert<HS>(htab, r[q], &won);
        full |= s < 0;
        wins += won;
        sl[q] = static_cast<uint32_t>(s) | (won ? kWon : 0u);
    }
#pragma unroll 1
    for (int k = U; k < deg; ++k) {
        bool won;
        const int s = set_insert<HS>(htab, row[k], &won);
        full |= s < 0;
        wins += won;
        seg[rs + k] = static_cast<uint16_t>(static_cast<uint32_t>(s) | (won ? kWon : 0u));
    }
    if (full) s_full = 1;
    int H;
    int h = block_excl_scan<T>(wins, &H, s_warp);
    // more distinct nodes than the set holds, or own nodes with few
    // neighbours in common: the node path
    if (s_full || H > 4 * T) {
        if (tid == 0) atomicOr(a.err, 2);
        return;
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
        if (sl[q] & kWon) {
            s_halo[h] = r[q];
            hidx[sl[q] & (HS - 1)] = static_cast<uint16_t>(T + h++);
        }
#pragma unroll 1
    for (int k = U; k < deg; ++k)
        if (seg[rs + k] & kWon) {
            s_halo[h] = row[k];
            hidx[seg[rs + k] & (HS - 1)] = static_cast<uint16_t>(T + h++);
        }
    __syncthreads();
    for (int j = tid; j < H; j += T) halo[j] = a.new_of_old[s_halo[j]];

    // ---- rows in local indices, and their offsets
    uint32_t l[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        l[q] = hidx[sl[q] & (HS - 1)];
        if (q < deg) seg[rs + q] = static_cast<uint16_t>(l[q]);
    }
#pragma unroll 1
    for (int k = U; k < deg; ++k) seg[rs + k] = hidx[seg[rs + k] & (HS - 1)];
    if (tid < len4 - len) seg[len + tid] = 0;
    rr[tid] = static_cast<uint16_t>(live ? rs : len);
    if (tid == 0) rr[T] = static_cast<uint16_t>(len);

    // ---- triangles
    uint64_t* const tri = reinterpret_cast<uint64_t*>(rec + align16(seg_at + 2 * static_cast<int64_t>(len4)));
    const Corners* const corners = reinterpret_cast<const Corners*>(a.tris);
    constexpr uint32_t kNotListed = ~0u;
    // a triangle, as the node's position in its stored order and the local
    // indices of the vertices that follow it there: position | local << 2 |
    // local << 14; kNotListed if an own vertex with a smaller label lists it
    auto pack = [&](uint32_t p, uint32_t lx, uint32_t ly) -> uint32_t {
        return min(lx, ly) < static_cast<uint32_t>(tid) ? kNotListed : p | (lx << 2) | (ly << 14);
    };
    auto turn = [&](const Corners& v, int32_t& x, int32_t& y) -> uint32_t {
        const uint32_t p = v.v0 == o ? 0u : (v.v1 == o ? 1u : 2u);
        x = p == 0 ? v.v1 : (p == 1 ? v.v2 : v.v0);
        y = p == 0 ? v.v2 : (p == 1 ? v.v0 : v.v1);
        return p;
    };
    uint32_t w[U];
    uint32_t miss = 0;   // triangles with a vertex beyond the row's registers
    int listed = 0;
#pragma unroll
    for (int q = 0; q < U; ++q) w[q] = kNotListed;
    if (inc > 0) {
        Corners v[U];
#pragma unroll
        for (int q = 0; q < U; ++q) v[q] = corners[t[q]];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            int32_t x, y;
            const uint32_t p = turn(v[q], x, y);
            uint32_t lx = kNotListed, ly = kNotListed;
#pragma unroll
            for (int k = 0; k < U; ++k) {
                lx = r[k] == x ? l[k] : lx;
                ly = r[k] == y ? l[k] : ly;
            }
            if (q < inc) {
                if (max(lx, ly) == kNotListed) miss |= 1u << q;
                else w[q] = pack(p, lx, ly);
            }
            listed += w[q] != kNotListed;
        }
    }
    auto later = [&](int k) -> uint32_t {
        int32_t x, y;
        const uint32_t p = turn(corners[fan[k]], x, y);
        const int sx = set_find<HS>(htab, x), sy = set_find<HS>(htab, y);
        if (sx < 0 || sy < 0) {   // validation rules this out
            atomicOr(a.err, 1);
            return kNotListed;
        }
        return pack(p, hidx[sx], hidx[sy]);
    };
    // the triangles left for later: those of `miss`, then those from U on
    auto for_later = [&](auto&& f) {
#pragma unroll 1
        for (uint32_t m = miss, k = U;;) {
            uint32_t q;
            if (m != 0) {
                q = static_cast<uint32_t>(__builtin_ctz(m));
                m &= m - 1;
            } else if (static_cast<int>(k) < inc) {
                q = k++;
            } else {
                break;
            }
            f(later(static_cast<int>(q)));
        }
    };
    for_later([&](uint32_t w) { listed += w != kNotListed; });
    int R;
    int at = block_excl_scan<T>(listed, &R, s_warp);

    // ---- grouped through LDS, in the set's place; fans beyond the registers
    // still need the set, so their tile's list goes by way of its place in
    // the record.  (A list longer than the set is left in incidence order:
    // any order gives the same results.)
    uint64_t* const s_tri = reinterpret_cast<uint64_t*>(htab);
    if (inc > U || miss != 0) s_full = 1;
    __syncthreads();
    const bool direct = R <= HS / 2 && !s_full;
    uint64_t* const to = direct ? s_tri : tri;
    auto put = [&](uint32_t w) {
        if (w == kNotListed) return;
        const uint64_t me = static_cast<uint64_t>(tid), lx = (w >> 2) & 4095u, ly = w >> 14;
        const uint32_t p = w & 3u;
        const uint64_t v0 = p == 0 ? me : (p == 1 ? ly : lx), v1 = p == 0 ? lx : (p == 1 ? me : ly),
                       v2 = p == 0 ? ly : (p == 1 ? lx : me);
        to[at++] = v0 | (v1 << 16) | (v2 << 32);
    };
#pragma unroll
    for (int q = 0; q < U; ++q) put(w[q]);
    for_later(put);
    if (R <= HS / 2) {
        __syncthreads();
        if (!direct) {
            for (int j = tid; j < R; j += T) s_tri[j] = tri[j];
            __syncthreads();
        }
        group_words<T, T>(s_tri, R, tri, s_cnt);
    }
    if (tid == 0) {
        TileWork w;
        w.X = a.X;
        w.halo = halo;
        w.rows = reinterpret_cast<const uint64_t*>(seg);
        w.tris = tri;
        w.rr = rr;
        w.own_start = k0;
        w.nown = nown;
        w.halo_cnt = H;
        w.tri_cnt = R;
        w.row_words = len4 >> 2;
        w.mesh = a.mesh;
        w.n = a.n;
        a.work[tile] = w;
    }
}

// One work-group per colour-class tile, in one pass like the Form A build.
// Its nodes are spread out (no two adjacent), so its halo is every node of
// its rows; instead of triangle words it gets one fan entry per incidence,
// in incidence order: the node's position p in the triangle's stored order
// and the row slots of the vertices at p+1 and p+2 (mod 3),
// p | slot << 2 | slot << 9, with the fan starts.  The row entries and
// incidences are walked as flat ranges, a few per work-item at a time, so
// that a node with a long row is shared by many lanes (finding a vertex in
// its row is a search).  An entry's own node is found from the owner of its
// 16-entry block, stepping forward over the node offsets.
template <int T>
__global__ __launch_bounds__(kClassBS) void k_class_build(TileBuildArgs a)
{
    constexpr int HS = 8 * T;
    constexpr int BS = kClassBS, U = kClassU, CAP = T * kTileMaxDeg, SPT = HS / BS;
    __shared__ int32_t htab[HS];
    __shared__ uint16_t hidx[HS];        // the local index of each slot's node
    __shared__ uint16_t own[CAP / 16];   // owner of entries 16b, 16b+1, ... starts the search
    __shared__ int32_t s_id[T], s_nb[T], s_tb[T], s_rs[T + 1], s_fs[T + 1];
    __shared__ uint16_t s_seg[CAP];   // the rows in local indices, for the slot search
    __shared__ int32_t s_warp[BS / 64];
    __shared__ int32_t s_full;
    const int tid = threadIdx.x;
    const int tile = blockIdx.x;
    int cl = 0;
    while (cl + 1 < a.n_class && tile >= a.cls_tile[cl + 1]) ++cl;
    const int32_t k0 = a.cls_start[cl] + (tile - a.cls_tile[cl]) * T;
    const int nown = min(T, a.cls_start[cl + 1] - k0);
    const int32_t rb = a.row_ptr[k0], fb = a.fan_ptr[k0];
    const int32_t len = a.row_ptr[k0 + nown] - rb, flen = a.fan_ptr[k0 + nown] - fb;
    if (len > CAP || flen > CAP) {   // denser than the LDS maps hold: the mesh takes the node path
        if (tid == 0) atomicOr(a.err, 2);
        return;
    }
    for (int s = tid; s < HS; s += BS) htab[s] = -1;
    if (tid == 0) {
        s_full = 0;
        s_rs[nown] = len;
        s_fs[nown] = flen;
    }
    for (int i = tid; i < nown; i += BS) {
        const int32_t o = a.perm[k0 + i];
        s_id[i] = o;
        s_nb[i] = a.nbr_ptr[o];
        s_tb[i] = a.tri_ptr[o];
        s_rs[i] = a.row_ptr[k0 + i] - rb;
        s_fs[i] = a.fan_ptr[k0 + i] - fb;
    }
    __syncthreads();
    for (int i = tid; i < nown; i += BS)
        for (int b = (s_rs[i] + 15) >> 4; (b << 4) < s_rs[i + 1]; ++b) own[b] = static_cast<uint16_t>(i);
    __syncthreads();

    // ---- halo set (own nodes are in no row of the tile): the slot of each row entry is parked in the row part of
    // the record until the slots have local indices
    unsigned char* rec = a.data + class_record(rb, fb, tile, T);
    uint16_t* rr = reinterpret_cast<uint16_t*>(rec);
    const int64_t hat = class_halo_at(T);
    int32_t* halo = reinterpret_cast<int32_t*>(rec + hat);
    const int32_t len4 = (len + 3) & ~3;
    const int64_t seg_at = align16(hat + 4 * static_cast<int64_t>(len));
    uint16_t* seg = reinterpret_cast<uint16_t*>(rec + seg_at);
    bool full = false;
    for (int base = 0; base < len; base += BS * U) {
        int32_t id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(base + u * BS + tid, len - 1);
            int i = own[j >> 4];
            while (s_rs[i + 1] <= j) ++i;
            id[u] = a.nbr_idx[s_nb[i] + (j - s_rs[i])];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * BS + tid;
            if (j >= len) continue;
            bool won;
            const int s = set_insert<HS>(htab, id[u], &won);
            if (s < 0) full = true;
            else seg[j] = static_cast<uint16_t>(s);
        }
    }
    if (full) s_full = 1;
    __syncthreads();
    if (s_full) {   // more distinct nodes than the set holds: the node path
        if (tid == 0) atomicOr(a.err, 2);
        return;
    }
    int c = 0;
#pragma unroll
    for (int q = 0; q < SPT; ++q) c += htab[tid * SPT + q] != -1;
    int H;
    int h = block_excl_scan<BS>(c, &H, s_warp);
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        const int s = tid * SPT + q;
        const int32_t key = htab[s];
        if (key == -1) continue;
        halo[h] = a.new_of_old[key];
        hidx[s] = static_cast<uint16_t>(T + h++);
    }
    __syncthreads();
    auto local = [&](int32_t id) -> int {
        const int s = set_find<HS>(htab, id);
        if (s < 0) {
            atomicOr(a.err, 1);
            return T;
        }
        return hidx[s];
    };

    // ---- rows in local indices, and their offsets
    for (int j = tid; j < len; j += BS) {
        const uint16_t l = hidx[seg[j]];
        seg[j] = l;
        s_seg[j] = l;
    }
    for (int j = len + tid; j < len4; j += BS) seg[j] = 0;
    for (int i = tid; i <= T; i += BS) rr[i] = static_cast<uint16_t>(s_rs[min(i, nown)]);
    // the entry map is rebuilt for the incidences
    for (int i = tid; i < nown; i += BS)
        for (int b = (s_fs[i] + 15) >> 4; (b << 4) < s_fs[i + 1]; ++b) own[b] = static_cast<uint16_t>(i);
    __syncthreads();

    // ---- fan entries, one per incidence, and the fan starts
    uint64_t* tri = reinterpret_cast<uint64_t*>(rec + align16(seg_at + 2 * static_cast<int64_t>(len4)));
    uint16_t* fans = reinterpret_cast<uint16_t*>(tri);
    uint16_t* fr = rr + halo_at(T) / 2;
    for (int i = tid; i <= T; i += BS) fr[i] = static_cast<uint16_t>(s_fs[min(i, nown)]);
    for (int base = 0; base < flen; base += BS * U) {
        int32_t v[U][3], i_of[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = min(base + u * BS + tid, flen - 1);
            int i = own[f >> 4];
            while (s_fs[i + 1] <= f) ++i;
            i_of[u] = i;
            const int64_t t = a.tri_idx[s_tb[i] + (f - s_fs[i])];
#pragma unroll
            for (int q = 0; q < 3; ++q) v[u][q] = a.tris[3 * t + q];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = base + u * BS + tid;
            if (f >= flen) continue;
            const int32_t id = s_id[i_of[u]];
            const int p = v[u][0] == id ? 0 : (v[u][1] == id ? 1 : 2);
            const int la = local(v[u][(p + 1) % 3]), lb = local(v[u][(p + 2) % 3]);
            const int r0 = s_rs[i_of[u]], r1 = s_rs[i_of[u] + 1];
            int sa = -1, sb = -1;
            for (int j = r0; j < r1; ++j) {
                const int l = s_seg[j];
                if (l == la) sa = j - r0;
                if (l == lb) sb = j - r0;
            }
            if (sa < 0 || sb < 0) atomicOr(a.err, 1);   // validation rules this out
            fans[f] = static_cast<uint16_t>(p | (max(sa, 0) << 2) | (max(sb, 0) << 9));
        }
    }
    if (tid == 0) {
        TileWork w;
        w.X = a.X;
        w.halo = halo;
        w.rows = reinterpret_cast<const uint64_t*>(seg);
        w.tris = tri;
        w.rr = rr;
        w.own_start = k0;
        w.nown = nown;
        w.halo_cnt = H;
        w.tri_cnt = flen;
        w.row_words = len4 >> 2;
        w.mesh = a.mesh;
        w.n = a.n;
        a.work[tile] = w;
    }
}

// Colour-class tiles: each node's fan entries grouped by the node's stored
// position p (0, then 1, then 2), in incidence order inside a group, and the
// group bounds written beside the fan starts, so that the sweep evaluates
// each group with the stored order fixed at compile time.  The minima over a
// fan are exact, so the order of its entries changes no result.  One
// work-group per tile; the tile's entries (at most T * kTileMaxDeg, the
// build's limit) are read into LDS first and written back grouped.
template <int T>
__global__ __launch_bounds__(256) void k_class_fan_sort(const TileWork* __restrict__ work)
{
    __shared__ uint16_t s_f[T * kTileMaxDeg];
    const TileWork d = work[blockIdx.x];
    uint16_t* const rr = const_cast<uint16_t*>(d.rr);
    const uint16_t* const fr = rr + halo_at(T) / 2;
    uint32_t* const pc = reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(rr) + 2 * halo_at(T));
    uint16_t* const fans = reinterpret_cast<uint16_t*>(const_cast<uint64_t*>(d.tris));
    const int flen = d.tri_cnt;
    for (int j = threadIdx.x; j < flen; j += 256) s_f[j] = fans[j];
    __syncthreads();
    for (int i = threadIdx.x; i < d.nown; i += 256) {
        const int b = fr[i], e = fr[i + 1];
        int c[4] = {0, 0, 0, 0};
        for (int j = b; j < e; ++j) ++c[s_f[j] & 3u];
        int pos[4] = {b, b + c[0], b + c[0] + c[1], e};
        for (int j = b; j < e; ++j) {
            const uint16_t v = s_f[j];
            fans[pos[v & 3u]++] = v;
        }
        pc[i] = static_cast<uint32_t>(c[0]) | (static_cast<uint32_t>(c[0] + c[1]) << 16);
    }
}

// Largest halo, padded row segment and triangle list over the tiles
// (mx[0..2], zeroed before), 256 tiles per work-group.
__global__ __launch_bounds__(256) void k_tile_caps(const TileWork* __restrict__ work, int32_t nt, int32_t* mx)
{
    __shared__ int32_t s_m[3][4];
    const int32_t t = static_cast<int32_t>(blockIdx.x * 256 + threadIdx.x);
    int32_t m[3] = {0, 0, 0};
    if (t < nt) {
        m[0] = work[t].halo_cnt;
        m[1] = 4 * work[t].row_words;
        m[2] = work[t].tri_cnt;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        for (int off = 32; off > 0; off >>= 1) m[k] = max(m[k], __shfl_xor(m[k], off));
        if ((threadIdx.x & 63) == 0) s_m[k][threadIdx.x >> 6] = m[k];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int32_t* const w = s_m[threadIdx.x];
        atomicMax(mx + threadIdx.x, max(max(w[0], w[1]), max(w[2], w[3])));
    }
}

// The build's error bits and caps to pinned memory.
__global__ void k_tile_tell(const int32_t* __restrict__ flags, int32_t* __restrict__ out)
{
    if (threadIdx.x < 4) out[threadIdx.x] = flags[threadIdx.x];
}

__global__ void k_tile_zero(int32_t* flags)
{
    if (threadIdx.x < 4) flags[threadIdx.x] = 0;
}

}  // namespace

size_t tile_bytes(int64_t n, int64_t nnz, int64_t ninc, int tile_nodes, bool classes)
{
    // build_tiles takes nothing for other sizes
    if (tile_nodes != 256 && tile_nodes != 512 && !(classes && tile_nodes == 128)) return 0;
    // colour-class tiles: at most one short tile per class more
    const size_t nt = static_cast<size_t>(div_up(std::max<int64_t>(n, 1), tile_nodes)) +
                      (classes ? static_cast<size_t>(kMaxTileClasses) : 0);
    const size_t z = static_cast<size_t>(std::max<int64_t>(nnz, 1)), c = static_cast<size_t>(std::max<int64_t>(ninc, 1));
    const size_t rec = classes ? nt * (8 * tile_nodes + 128) + 6 * z + 2 * c + 16
                               : nt * (2 * tile_nodes + 64) + 6 * z + 8 * c + 16;
    return Arena::piece(sizeof(TileWork) * nt) + Arena::piece(rec);
}

size_t tile_scratch_bytes() { return Arena::piece(4 * sizeof(int32_t)); }

sl_status build_tiles(const SetupArgs& a, DevMesh& m, int tile_nodes, int mesh, hipStream_t st, Arena& persist,
                      Arena& scratch, bool classes)
{
    m.tile_nodes = 0;
    m.n_tile_classes = 0;
    if ((tile_nodes != 256 && tile_nodes != 512 && !(classes && tile_nodes == 128)) || m.n_free == 0) return SL_OK;
    if (classes && (m.n_colors < 1 || m.n_colors > kMaxTileClasses)) return SL_OK;
    const int T = tile_nodes;
    int nt = div_up(m.n_free, T);
    if (classes) {
        nt = 0;
        for (int c = 0; c < m.n_colors; ++c) {
            m.class_tile_h[c] = nt;
            nt += div_up(m.color_start_h[c + 1] - m.color_start_h[c], T);
        }
        m.class_tile_h[m.n_colors] = nt;
    }
    const size_t pmark = persist.mark(), smark = scratch.mark();
    sl_status r = SL_OK;
    int32_t* flags = nullptr;   // {err, largest halo, largest row segment, largest triangle list}
    if ((r = scratch.take(&flags, 4))) return r;
    PinnedPad pad;
    if ((r = pad.init())) return r;
    k_tile_zero<<<1, 64, 0, st>>>(flags);
    const size_t data_bytes =
        static_cast<size_t>(classes ? class_record(static_cast<int32_t>(m.nnz_free), static_cast<int32_t>(m.ninc_free), nt, T)
                                    : tile_record(static_cast<int32_t>(m.nnz_free), static_cast<int32_t>(m.ninc_free), nt, T));
    if ((r = persist.take(&m.work, nt)) || (r = persist.take(&m.tile_data, data_bytes))) return r;
    TileBuildArgs b{};
    b.perm = m.perm;
    b.new_of_old = m.new_of_old;
    b.nbr_ptr = a.nbr_ptr;
    b.nbr_idx = a.nbr_idx;
    b.tri_ptr = a.tri_ptr;
    b.tri_idx = a.tri_idx;
    b.tris = a.tris;
    b.row_ptr = m.row_ptr;
    b.fan_ptr = m.fan_ptr;
    b.n_free = m.n_free;
    b.mesh = mesh;
    b.n = m.n;
    b.X = m.X[0];
    b.data = m.tile_data;
    b.work = m.work;
    b.err = flags;
    b.n_class = classes ? m.n_colors : 0;
    for (int c = 0; classes && c <= m.n_colors; ++c) {
        b.cls_start[c] = m.color_start_h[c];
        b.cls_tile[c] = m.class_tile_h[c];
    }
    if (classes) {
        if (T == 128) k_class_build<128><<<nt, kClassBS, 0, st>>>(b);
        else if (T == 256) k_class_build<256><<<nt, kClassBS, 0, st>>>(b);
        else k_class_build<512><<<nt, kClassBS, 0, st>>>(b);
    } else {
        if (T == 256) k_tile_build<256><<<nt, 256, 0, st>>>(b);
        else k_tile_build<512><<<nt, 512, 0, st>>>(b);
    }
    k_tile_caps<<<div_up(nt, 256), 256, 0, st>>>(m.work, nt, flags + 1);
    k_tile_tell<<<1, 64, 0, st>>>(flags, static_cast<int32_t*>(pad.p));
    SL_HIP(hipGetLastError());
    SL_HIP(hipStreamSynchronize(st));
    int32_t h[4];
    std::memcpy(h, pad.p, sizeof(h));
    scratch.rewind(smark);
    if (h[0] & 1) return fail(SL_ETOPO, "triangle vertex outside its tile's neighbourhood");
    // a tile denser than the staging holds, or a halo or row segment too big
    // for LDS: the node path, whose arrays reuse the tile arrays' room
    const size_t lds = classes ? class_lds_bytes(T, h[1], h[2], h[3]) : tile_lds_bytes(T, h[1], h[2], m.precision);
    if ((h[0] & 2) || lds > kTileLdsLimit) {
        m.work = nullptr;
        m.tile_data = nullptr;
        persist.rewind(pmark);
        return SL_OK;
    }
    if (classes) {
        if (T == 128) k_class_fan_sort<128><<<nt, 256, 0, st>>>(m.work);
        else if (T == 256) k_class_fan_sort<256><<<nt, 256, 0, st>>>(m.work);
        else k_class_fan_sort<512><<<nt, 256, 0, st>>>(m.work);
    }
    SL_HIP(hipGetLastError());
    m.halo_max = h[1];
    m.rows_max = h[2];
    m.fans_max = h[3];
    m.n_tiles = nt;
    m.tile_nodes = T;
    m.n_tile_classes = classes ? m.n_colors : 0;
    return SL_OK;
}

}  // namespace sl
