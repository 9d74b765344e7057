// Small and medium meshes: every sweep of a mesh in one launch.
//
// A sweep of a mesh of at most a few hundred thousand nodes is a few
// microseconds of arithmetic; a launch per sweep (Form A), or per colour
// class (Form B), costs more than that in launch gaps, staging and drains
// (7-11 us a launch).  Here the free nodes (Hilbert order) are cut into
// tiles of T nodes, one work-group per tile, all resident on the device at
// once, and each keeps its tile's positions, rows and fans in LDS for the
// whole run.  Between sweeps (classes) a work-group needs from others only
// the new positions of its halo nodes.
//
// Exchange: a node that other tiles read is published, as two 8-byte
// device-scope stores, in ring[v % 4] for version v (the position after v
// sweeps).  A reader polls the node's own slot until neither half is the
// sentinel (a NaN pattern, which no position has: coordinates are finite),
// so one trip through memory carries data and signal together.  While
// version v is made, the node's slot for v + 2 is set back to the sentinel;
// that slot held version v - 2.  Every reader is done with it: tiles read
// each other both ways (neighbour rows are checked to be symmetric), the
// writer has seen version v - 1 of some node of the reader's tile, and the
// reader published that after it had read version v - 2 of all its halo.
// Every wave waits for its stores to memory at the head of each class (at
// that of each sweep in Form A), so the store that sets a slot back has been
// performed before the version ahead of it is published, and no reader finds
// the old value.
//
// Form A reads one LDS buffer and writes the other; Form B updates one in
// place, class by class, reading class c's halo nodes after its own class c.
//
// Waits end: a wait longer than the limit, or another group's failure, sets
// the abort word, every group leaves, the caller's positions are untouched
// and the call runs again on the one-launch-per-sweep kernels.  The groups
// of all flow launches that the process has in flight on a device are limited
// to what it holds at once (FlowSlots), so the limit is reached only if other
// work, such as another process's, keeps part of the device for that long;
// no run is begun there for a while then.
//
// With a tolerance one more work-group (the controller) folds the waves'
// displacement maxima of each sweep and publishes whether the next one runs;
// the tiles run at most kFlowLag sweeps ahead of its decisions and keep
// their last positions, so the result is that of the stopping sweep.
//
// The arithmetic of a node is the node kernel's, operation for operation;
// W lanes of a wave share a node's fan and fold their minima (exact in any
// order).
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "sl_common.h"
#include "sl_flow.h"
#include "sl_node_math.h"

namespace sl {

namespace {

using u64 = unsigned long long;

constexpr u64 kSent = 0xFFF8DEAD5EA15EA1ull;   // a quiet NaN: "not published yet"
constexpr int kFlowLag = 3;                    // sweeps a tile may run past the last decided one
constexpr int kFlowHist = 4;                   // positions kept per node with a tolerance (kFlowLag + 1)
// Sweeps whose displacement maxima have slots.  A wave sets the slot of sweep
// s + 2 back in sweep s, and waits for that at the head of s + 1, before it
// publishes the maximum ahead of it; what the slot held, that of s + 2 -
// kFlowSlots, has been decided on when the wave starts sweep s.
constexpr int kFlowSlots = 8;
static_assert(2 - kFlowSlots <= -kFlowLag, "a slot is free when it is set back");
constexpr uint32_t kOneCall = 1u;              // the number of a call's one run
constexpr uint32_t kDeclineColor = 8u;         // FlowState::decline: not coloured in time (1, 2, 4: the build)
constexpr int32_t kFixedKey = INT32_MIN;       // halo key of a fixed node: kFixedKey + its place in the positions

// Tile records in global memory and, with the same layout, in LDS.
struct FlowLayout {
    int hc, lc;   // halo nodes, and row (fan) entries, a tile may have
    int halo, hcls, cls, rs, fs, ord, flag, rows, fans, bytes;
    __host__ __device__ constexpr explicit FlowLayout(int T)
        : hc(T <= 64 ? 128 : (T <= 128 ? 192 : (T <= 256 ? 256 : 384))), lc(T <= 256 ? 10 * T : 8 * T), halo(32),
          hcls(halo + 4 * hc), cls(hcls + 80), rs(cls + 80), fs(rs + 2 * (T + 8)), ord(fs + 2 * (T + 8)),
          flag(ord + 2 * T), rows(flag + T), fans(rows + 2 * lc), bytes(fans + 4 * lc)
    {
    }
};
static_assert(2 * (kFlowClasses + 2) <= 80, "class tables");
static_assert(FlowLayout(64).bytes % 16 == 0 && FlowLayout(128).bytes % 16 == 0 && FlowLayout(256).bytes % 16 == 0 &&
                  FlowLayout(512).bytes % 16 == 0,
              "records are copied in 16-byte units");

__device__ __forceinline__ u64 ld_dev(const u64* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(u64* p, u64 v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_dev(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(uint32_t* p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The maximum over a wave (all lanes active; values >= 0).
__device__ __forceinline__ double wave_max(double v)
{
    const double m = -group_min<16>(-v);
    double r = 0.0;
#pragma unroll
    for (int l = 0; l < 64; l += 16) {
        const long long b = __double_as_longlong(m);
        const int lo = __builtin_amdgcn_readlane(static_cast<int>(b), l);
        const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), l);
        const double t = __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<uint32_t>(lo));
        r = t > r ? t : r;
    }
    return r;
}

// Whether the mesh is not for the flow kernels after all (every kernel after
// the checks asks; the host learns it with the report).  What it reads does
// not change while a kernel that asks runs, so a group's waves agree: the
// build, which sets the other decline bits, asks for the colouring's only.
__device__ __forceinline__ bool flow_off(const ValStats* vs, const FlowState* fs, uint32_t decline = ~0u)
{
    return vs->err != 0 || vs->n_free == 0 || (fs->decline & decline) != 0 || fs->n_colors > kFlowClasses;
}

// Bounded waiting: every 256 polls the abort word and the clock are looked
// at; with a limit of 0 nothing is waited for.  False: give up.
struct Waiter {
    FlowState* fs;
    u64 limit, t0;
    uint32_t run, polls;
    __device__ __forceinline__ Waiter(FlowState* f, u64 l, uint32_t r) : fs(f), limit(l), t0(0), run(r), polls(0) {}
    __device__ __forceinline__ bool again()
    {
        if ((++polls & 255u) != 0 && limit != 0) return true;
        if (ld_dev(&fs->abort) == run) return false;
        const u64 now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 <= limit && limit != 0) return true;
        st_dev(&fs->abort, run);
        return false;
    }
};

// Everything a call must find set before its kernels: counters and states
// zero, no node coloured, no version published, no maxima.
struct FlowInitArgs {
    ValStats* vs;        // nullable
    FlowState* fs;
    int32_t* count;
    int64_t n_count;
    int32_t* color;      // nullable
    int64_t n;
    u64* ring12;         // [2][2n]: the slots of versions 1 and 2
    u64* dmax;           // nullable, [n_dmax]
    int64_t n_dmax;
    u64* bits;           // nullable, [n_bits]
    int64_t n_bits;
};

__global__ __launch_bounds__(256) void k_flow_init(FlowInitArgs a)
{
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x, stride = static_cast<int64_t>(gridDim.x) * 256;
    if (blockIdx.x == 0) {
        if (a.vs)
            for (int q = threadIdx.x; q < static_cast<int>(sizeof(ValStats) / 4); q += 256)
                reinterpret_cast<uint32_t*>(a.vs)[q] = 0;
        for (int q = threadIdx.x; q < static_cast<int>(sizeof(FlowState) / 4); q += 256) reinterpret_cast<uint32_t*>(a.fs)[q] = 0;
        __syncthreads();
        if (threadIdx.x == 0) a.fs->t_begin = wall_clock64();
    }
    for (int64_t q = g; q < a.n_count; q += stride) a.count[q] = 0;
    for (int64_t q = g; q < 4 * a.n; q += stride) a.ring12[q] = kSent;
    if (a.color)
        for (int64_t q = g; q < a.n; q += stride) a.color[q] = -1;
    for (int64_t q = g; q < a.n_dmax; q += stride) a.dmax[q] = kSent;
    for (int64_t q = g; q < a.n_bits; q += stride) a.bits[q] = 0;
}

// ------------------------------------------------------------- colouring --

// Greedy colouring by dataflow: every free node's work-item waits for the
// colours of its free neighbours of higher priority and takes the smallest
// one none of them has (one launch instead of some twenty rounds; the
// highest uncoloured priority can always go on, so with all groups resident
// none waits for ever).
__global__ __launch_bounds__(256) void k_flow_color(const int32_t* __restrict__ nbr_ptr,
                                                    const int32_t* __restrict__ nbr_idx,
                                                    const uint8_t* __restrict__ bnd, int32_t* color, int32_t n,
                                                    const ValStats* __restrict__ vs, FlowState* fs, u64 wait)
{
    if (vs->err != 0) return;
    constexpr int R = 8;
    const int32_t i = static_cast<int32_t>(blockIdx.x * 256 + threadIdx.x);
    const bool mine = i < n && bnd[i] == 0;
    int32_t b = 0, d = 0;
    uint64_t pi = 0;
    if (mine) {
        b = nbr_ptr[i];
        d = nbr_ptr[i + 1] - b;
        pi = splitmix64(static_cast<uint64_t>(i));
    }
    int32_t above[R];   // the first R neighbours that must have a colour first, else -1
#pragma unroll
    for (int j = 0; j < R; ++j) above[j] = j < d ? nbr_idx[b + j] : -1;
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (above[j] >= 0 && (bnd[above[j]] != 0 || splitmix64(static_cast<uint64_t>(above[j])) < pi)) above[j] = -1;
    Waiter w(fs, wait, kOneCall);
    bool done = !mine;
    int32_t c = -1;
    uint64_t used0 = 0, used1 = 0;
    auto use = [&](int32_t cj) {
        if (cj < 64) used0 |= 1ull << cj;
        else used1 |= 1ull << (cj - 64);
    };
    const uint32_t* const col = reinterpret_cast<const uint32_t*>(color);
    for (;;) {
        if (!done) {
            bool ready = true;
            int32_t cj[R];
#pragma unroll
            for (int j = 0; j < R; ++j) cj[j] = -1;
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (above[j] >= 0) cj[j] = static_cast<int32_t>(ld_dev(col + above[j]));
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (above[j] < 0) continue;
                if (cj[j] >= 0) {
                    use(cj[j]);
                    above[j] = -1;
                } else {
                    ready = false;
                }
            }
            if (d > R && ready)
                for (int32_t k = b + R; k < b + d; ++k) {
                    const int32_t j = nbr_idx[k];
                    if (bnd[j] != 0 || splitmix64(static_cast<uint64_t>(j)) < pi) continue;
                    const int32_t q = static_cast<int32_t>(ld_dev(col + j));
                    if (q >= 0) use(q);
                    else ready = false;
                }
            if (ready) {
                c = (~used0) ? __builtin_ctzll(~used0) : 64 + __builtin_ctzll(~used1);
                st_dev(reinterpret_cast<uint32_t*>(color) + i, static_cast<uint32_t>(c));
                done = true;
            }
        }
        if (__ballot(!done) == 0ull) break;
        if (!w.again()) {
            if (!done) atomicOr(&fs->decline, kDeclineColor);   // not coloured: the mesh takes the other kernels
            break;
        }
    }
    for (int off = 32; off > 0; off >>= 1) c = max(c, __shfl_xor(c, off));
    if ((threadIdx.x & 63) == 0 && c >= 0 &&
        c + 1 > __hip_atomic_load(&fs->n_colors, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&fs->n_colors, c + 1);
}

// ----------------------------------------------------------------- build --

template <int BS>
__device__ __forceinline__ uint32_t block_excl(uint32_t v, uint32_t* total, uint32_t* s_warp)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(x, off);
        if (lane >= off) x += t;
    }
    if (lane == 63) s_warp[w] = x;
    __syncthreads();
    uint32_t base = 0, all = 0;
#pragma unroll
    for (int q = 0; q < BS / 64; ++q) {
        const uint32_t c = s_warp[q];
        base += q < w ? c : 0;
        all += c;
    }
    *total = all;
    return base + x - v;
}

struct FlowBuildArgs {
    const ValStats* vs;
    FlowState* fs;
    const int32_t* perm;
    const int32_t* new_of_old;   // fixed nodes: negative, or labels from the free nodes' count on
    const int32_t* nbr_ptr;
    const int32_t* nbr_idx;
    const int32_t* tri_ptr;
    const int32_t* tri_idx;
    const int32_t* tris;
    const int32_t* color;        // by caller node (Form B)
    unsigned char* rec;
};

// One work-group per tile writes the tile's record: the halo (free nodes by
// colour class, then fixed ones), rows in tile-local indices (own 0 .. T-1,
// halo from T), per incidence the local indices of the triangle's vertices
// that follow the node in stored order and the node's position, and the own
// nodes ordered by class and, inside a class, published nodes first.
// LPN = BS / T lanes share a node's entries.
template <int T, bool CLS>
__global__ __launch_bounds__((T > 256 ? T : 256)) void k_flow_build(FlowBuildArgs a)
{
    constexpr int BS = T > 256 ? T : 256, LPN = BS / T, HS = 4 * T, SPT = HS / BS, U = LPN > 1 ? 2 : 4;
    constexpr FlowLayout L(T);
    __shared__ int32_t htab[HS];
    __shared__ uint16_t hidx[HS];
    __shared__ int32_t s_row[L.lc];
    __shared__ int32_t s_hcnt[kFlowClasses + 2], s_ocnt[2 * kFlowClasses + 2];
    __shared__ uint8_t s_flag[T];
    __shared__ uint32_t s_warp[BS / 64];
    __shared__ int32_t s_full;
    if (flow_off(a.vs, a.fs, kDeclineColor)) return;
    const int tid = threadIdx.x, tile = blockIdx.x, n_free = a.vs->n_free, k0 = tile * T, nown = min(T, n_free - k0);
    if (nown <= 0) return;
    const int C = CLS ? a.fs->n_colors : 1;
    unsigned char* const rec = a.rec + static_cast<int64_t>(tile) * L.bytes;
    int32_t* const head = reinterpret_cast<int32_t*>(rec);
    int32_t* const halo = reinterpret_cast<int32_t*>(rec + L.halo);
    uint16_t* const hcls = reinterpret_cast<uint16_t*>(rec + L.hcls);
    uint16_t* const cls = reinterpret_cast<uint16_t*>(rec + L.cls);
    uint16_t* const rs = reinterpret_cast<uint16_t*>(rec + L.rs);
    uint16_t* const fo = reinterpret_cast<uint16_t*>(rec + L.fs);
    uint16_t* const ord = reinterpret_cast<uint16_t*>(rec + L.ord);
    uint16_t* const rows = reinterpret_cast<uint16_t*>(rec + L.rows);
    uint32_t* const fans = reinterpret_cast<uint32_t*>(rec + L.fans);

    const int i = tid / LPN, sub = tid % LPN;
    const bool own = i < nown;
    int32_t o = 0, nb = 0, d = 0, tb = 0, nt = 0, c_own = 0;
    if (own) {
        o = a.perm[k0 + i];
        nb = a.nbr_ptr[o];
        d = a.nbr_ptr[o + 1] - nb;
        tb = a.tri_ptr[o];
        nt = a.tri_ptr[o + 1] - tb;
        if (CLS) c_own = a.color[o];
    }
    for (int s = tid; s < HS; s += BS) htab[s] = -1;
    for (int s = tid; s < kFlowClasses + 2; s += BS) s_hcnt[s] = 0;
    for (int s = tid; s < 2 * kFlowClasses + 2; s += BS) s_ocnt[s] = 0;
    if (tid < T) s_flag[tid] = 0;
    if (tid == 0) s_full = 0;
    __syncthreads();
    if (nt > kMaxValence) s_full = 1;   // (an incidence list longer than any row: not for this path)
    // row and fan offsets, packed: at most 127 entries per node each
    uint32_t tot;
    const uint32_t at = block_excl<BS>(
        sub == 0 ? static_cast<uint32_t>(d) | (static_cast<uint32_t>(min(nt, kMaxValence)) << 16) : 0u, &tot, s_warp);
    const uint32_t at0 = __shfl(at, (tid & 63) / LPN * LPN);   // the node's first lane has its offsets
    const int r0 = static_cast<int>(at0 & 0xFFFFu), f0 = static_cast<int>(at0 >> 16);
    const int len = static_cast<int>(tot & 0xFFFFu), flen = static_cast<int>(tot >> 16);
    if (s_full || len > L.lc || flen > L.lc) {
        if (tid == 0) atomicOr(&a.fs->decline, 1u);
        return;
    }
    auto in_tile = [&](int32_t key) { return key >= k0 && key < k0 + nown; };
    auto key_of = [&](int32_t id) {
        const int32_t l = a.new_of_old[id];
        return l >= 0 && l < n_free ? l : kFixedKey + (l >= 0 ? l : id);
    };
    auto home = [&](int32_t key) {
        return static_cast<int>((static_cast<uint32_t>(key) * 2654435761u) >> (32 - __builtin_ctz(HS)));
    };
    // ---- rows as keys, and the halo set
    for (int j0 = sub; j0 < d; j0 += U * LPN) {
        int32_t key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = a.nbr_idx[nb + min(j0 + u * LPN, d - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = key_of(key[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + u * LPN < d) {
                s_row[r0 + j0 + u * LPN] = key[u];
                if (!in_tile(key[u])) {
                    int s = home(key[u]);
                    bool placed = false;
                    for (int p = 0; p < HS && !placed; ++p) {
                        const int32_t prev = atomicCAS(&htab[s], -1, key[u]);
                        placed = prev == -1 || prev == key[u];
                        s = (s + 1) & (HS - 1);
                    }
                    if (!placed) s_full = 1;
                }
            }
        }
    }
    __syncthreads();
    // ---- halo numbering: by class, fixed nodes last
    int hc[SPT], hr[SPT];
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        const int32_t key = htab[tid + q * BS];
        hc[q] = -1;
        hr[q] = 0;
        if (key != -1) {
            hc[q] = key < 0 ? C : (CLS ? a.color[a.perm[key]] : 0);
            hr[q] = atomicAdd(&s_hcnt[hc[q]], 1);
        }
    }
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int c = 0; c <= C; ++c) {
            const int t = s_hcnt[c];
            s_hcnt[c] = run;
            run += t;
        }
        s_hcnt[C + 1] = run;
    }
    __syncthreads();
    const int Hf = s_hcnt[C], H = s_hcnt[C + 1];
    if (s_full || H > L.hc) {
        if (tid == 0) atomicOr(&a.fs->decline, 2u);
        return;
    }
#pragma unroll
    for (int q = 0; q < SPT; ++q)
        if (hc[q] >= 0) {
            const int h = s_hcnt[hc[q]] + hr[q];
            hidx[tid + q * BS] = static_cast<uint16_t>(h);
            halo[h] = htab[tid + q * BS];
        }
    if (tid <= C) hcls[tid] = static_cast<uint16_t>(s_hcnt[tid]);
    __syncthreads();
    auto local = [&](int32_t key) -> uint32_t {
        if (in_tile(key)) return static_cast<uint32_t>(key - k0);
        int s = home(key);
        for (int p = 0; p < HS; ++p) {
            const int32_t cur = htab[s];
            if (cur == key) return static_cast<uint32_t>(T + hidx[s]);
            if (cur == -1) break;
            s = (s + 1) & (HS - 1);
        }
        atomicOr(&a.fs->decline, 4u);   // the checks rule this out
        return 0u;
    };
    // ---- rows in local indices; a node with a free neighbour in another tile is published
    bool border = false;
    for (int j = sub; j < d; j += LPN) {
        const int32_t key = s_row[r0 + j];
        rows[r0 + j] = static_cast<uint16_t>(local(key));
        border |= key >= 0 && !in_tile(key);
    }
    if (border) s_flag[i] = 1;
    // ---- fans
    for (int q0 = sub; q0 < nt; q0 += U * LPN) {
        int32_t t[U], v[U][3];
#pragma unroll
        for (int u = 0; u < U; ++u) t[u] = a.tri_idx[tb + min(q0 + u * LPN, nt - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < 3; ++q) v[u][q] = a.tris[3 * static_cast<int64_t>(t[u]) + q];
        int32_t ka[U], kb[U];
        uint32_t pp[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pp[u] = v[u][0] == o ? 0u : (v[u][1] == o ? 1u : 2u);
            ka[u] = key_of(pp[u] == 0 ? v[u][1] : (pp[u] == 1 ? v[u][2] : v[u][0]));
            kb[u] = key_of(pp[u] == 0 ? v[u][2] : (pp[u] == 1 ? v[u][0] : v[u][1]));
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (q0 + u * LPN < nt) fans[f0 + q0 + u * LPN] = local(ka[u]) | (local(kb[u]) << 12) | (pp[u] << 24);
    }
    if (own && sub == 0) {
        rs[i] = static_cast<uint16_t>(r0);
        fo[i] = static_cast<uint16_t>(f0);
    }
    if (tid == 0) {
        rs[nown] = static_cast<uint16_t>(len);
        fo[nown] = static_cast<uint16_t>(flen);
        head[0] = nown;
        head[1] = H;
        head[2] = Hf;
    }
    __syncthreads();
    // ---- own nodes by class, published ones first
    int rank = 0, bucket = 0;
    if (own && sub == 0) {
        bucket = 2 * c_own + (s_flag[i] ? 0 : 1);
        rank = atomicAdd(&s_ocnt[bucket], 1);
        rec[L.flag + i] = s_flag[i];
    }
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int c = 0; c < 2 * C; ++c) {
            const int t = s_ocnt[c];
            s_ocnt[c] = run;
            if ((c & 1) == 0) cls[c >> 1] = static_cast<uint16_t>(run);
            run += t;
        }
        cls[C] = static_cast<uint16_t>(run);
    }
    __syncthreads();
    if (own && sub == 0) ord[s_ocnt[bucket] + rank] = static_cast<uint16_t>(i);
}

// ----------------------------------------------------------------- sweep --

struct FlowArgs {
    const ValStats* vs;
    FlowState* fs;
    const int32_t* perm;        // place of each free node in `coords`; null: its label
    const double* coords;       // the start positions, read only
    const unsigned char* rec;
    u64* ring;                  // [4][2n]: published versions
    double* out;                // [2n] final positions, device order
    double* hist;               // [kFlowHist][2n] (with a tolerance)
    u64* dmax;                  // [kFlowSlots][tiles * waves]: displacement maxima per sweep (with a tolerance)
    FlowGroup* groups;          // [tiles]
    u64* bits;                  // nullable: accept bits, `words` per sweep
    int64_t words;
    int64_t n;
    int32_t T, tiles;           // tiles of n nodes (the free ones may fill fewer)
    int32_t iters;
    int32_t v0;                 // version of the start positions (mod 4)
    double tol2;
    u64 wait;                   // clock ticks a wait may take
    uint32_t run;               // the run's number: kOneCall, or a handle's count of its runs
    const int32_t *nbr_end, *tri_end;   // nbr_ptr + n, tri_ptr + n
};

// What a lane needs to know of its next node, read from the record ahead of
// its positions: the chain order -> offsets -> entries is off the path from
// an exchange to the next one.
constexpr int kRefRow = 8, kRefFan = 2;   // row entries, and fan entries of the lane
struct NodeRef {
    int i, r0, d, f, f1;          // node, row, the lane's first fan entry and the fan's end
    uint32_t row[kRefRow / 2];    // the first entries, two u16 each
    uint32_t fan[kRefFan];
    bool border;
};

struct FlowRec {
    const uint16_t *rs, *fo, *ord, *rows;
    const uint32_t* fans;
    const uint8_t* flag;
};

template <int W>
__device__ __forceinline__ void load_ref(NodeRef& n, const FlowRec& t, int q, int j)
{
    n.i = t.ord[q];
    n.r0 = t.rs[n.i];
    n.d = t.rs[n.i + 1] - n.r0;
    n.f = t.fo[n.i] + j;
    n.f1 = t.fo[n.i + 1];
    n.border = t.flag[n.i] != 0;
#pragma unroll
    for (int u = 0; u < kRefRow; u += 2)
        n.row[u / 2] = static_cast<uint32_t>(t.rows[n.r0 + min(u, n.d - 1)]) |
                       (static_cast<uint32_t>(t.rows[n.r0 + min(u + 1, n.d - 1)]) << 16);
#pragma unroll
    for (int u = 0; u < kRefFan; ++u) n.fan[u] = t.fans[max(min(n.f + u * W, n.f1 - 1), 0)];
    if (n.f1 == t.fo[n.i]) {   // a node in no triangle: its own position stands in
#pragma unroll
        for (int u = 0; u < kRefFan; ++u) n.fan[u] = static_cast<uint32_t>(n.i) | (static_cast<uint32_t>(n.i) << 12);
    }
}

// Candidate and worst qualities of node n by W lanes (this one is lane j).
template <int W>
__device__ __forceinline__ void flow_node(const NodeRef& n, const FlowRec& t, const double2* X, const double* recip,
                                          double2& o, double2& c, double& qo, double& qn)
{
    o = X[n.i];
    // the fan's vertices and the row's positions in flight together
    double2 va[kRefFan], vb[kRefFan];
    double2 p[kRefRow];
#pragma unroll
    for (int u = 0; u < kRefRow; ++u) p[u] = X[(n.row[u / 2] >> (16 * (u & 1))) & 0xFFFFu];
#pragma unroll
    for (int u = 0; u < kRefFan; ++u) {
        va[u] = X[n.fan[u] & 0xFFFu];
        vb[u] = X[(n.fan[u] >> 12) & 0xFFFu];
    }
    double sx = 0.0, sy = 0.0;
#pragma unroll
    for (int u = 0; u < kRefRow; ++u)
        if (u < n.d) {
            sx += p[u].x;
            sy += p[u].y;
        }
    for (int j0 = kRefRow; j0 < n.d; j0 += 4) {
        int l[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) l[u] = t.rows[n.r0 + min(j0 + u, n.d - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) p[u] = X[l[u]];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j0 + u < n.d) {
                sx += p[u].x;
                sy += p[u].y;
            }
    }
    const double dn = static_cast<double>(n.d), y = recip[n.d];
    c.x = div_small(sx, dn, y);
    c.y = div_small(sy, dn, y);
    const bool tiny = !(fabs(sx) >= kStepMin) || !(fabs(sy) >= kStepMin);
    if (__builtin_amdgcn_ballot_w64(tiny) != 0ull) {
        if (tiny) {
            c.x = sx / dn;
            c.y = sy / dn;
        }
    }
    qo = qn = INFINITY;
    for (int f = n.f, first = 1; f < n.f1; f += kRefFan * W, first = 0) {
        uint32_t e[kRefFan];
#pragma unroll
        for (int u = 0; u < kRefFan; ++u) e[u] = n.fan[u];
        if (!first) {
#pragma unroll
            for (int u = 0; u < kRefFan; ++u) {
                e[u] = t.fans[min(f + u * W, n.f1 - 1)];
                va[u] = X[e[u] & 0xFFFu];
                vb[u] = X[(e[u] >> 12) & 0xFFFu];
            }
        }
#pragma unroll
        for (int u = 0; u < kRefFan; ++u) {
            if (f + u * W < n.f1) {
                double v, w;
                fan_qualities(static_cast<int>(e[u] >> 24), o, c, va[u], vb[u], v, w);
                qo = v < qo ? v : qo;
                qn = w < qn ? w : qn;
            }
        }
    }
    qo = group_min<W>(qo);
    qn = group_min<W>(qn);
}

// The controller (with a tolerance): sweep after sweep, the largest
// displacement over all waves, then the decision.
__device__ void flow_control(const FlowArgs& a, int waves, int BS)
{
    constexpr int U = 8;
    __shared__ double s_m[8];
    __shared__ int s_bad;
    const int tid = threadIdx.x, n_slots = (a.vs->n_free + a.T - 1) / a.T * waves;
    const int64_t cap = static_cast<int64_t>(a.tiles) * waves;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    for (int s = 0; s < a.iters; ++s) {
        const u64* const slot = a.dmax + (s & (kFlowSlots - 1)) * cap;
        double m = 0.0;
        Waiter w(a.fs, a.wait, a.run);
        for (int q0 = tid; q0 < n_slots; q0 += U * BS) {
            u64 v[U];
            for (;;) {
                bool all = true;
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = q0 + u * BS < n_slots ? ld_dev(slot + q0 + u * BS) : 0ull;
#pragma unroll
                for (int u = 0; u < U; ++u) all = all && v[u] != kSent;
                if (all) break;
                if (!w.again()) {
                    s_bad = 1;
                    break;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double x = __longlong_as_double(static_cast<long long>(v[u]));
                m = x > m ? x : m;
            }
        }
        m = wave_max(m);
        if ((tid & 63) == 0) s_m[tid >> 6] = m;
        __syncthreads();
        if (s_bad) return;
        for (int q = 0; q < BS / 64; ++q) m = s_m[q] > m ? s_m[q] : m;
        const bool stop = s + 1 == a.iters || (a.tol2 > 0.0 && m < a.tol2);
        if (tid == 0) {
            if (stop) a.fs->maxd = static_cast<u64>(__double_as_longlong(m));
            st_dev(&a.fs->decided, static_cast<uint32_t>(s + 1) | (stop ? kFlowStop : 0u));
        }
        __syncthreads();   // s_m is free
        if (stop) return;
    }
}

template <bool B, int W, bool GT, bool TOL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_sweep_flow(FlowArgs a)
{
    extern __shared__ double2 flow_lds[];
    __shared__ double s_recip[kMaxValence + 1];
    __shared__ double s_d2[8];
    __shared__ u64 s_last[8], s_tot[8];
    // set in a phase before its barrier, read after it; two of each, so that
    // a wave already in the next phase does not write what others still read
    __shared__ int s_abort[2];
    __shared__ uint32_t s_stop[2];
    if (flow_off(a.vs, a.fs)) return;
    const int tid = threadIdx.x, BS = static_cast<int>(blockDim.x), lane = tid & 63, wv = tid >> 6, waves = BS >> 6;
    const int T = a.T;
    if (TOL && static_cast<int>(blockIdx.x) == a.tiles) {
        flow_control(a, waves, BS);
        return;
    }
    const int tile = static_cast<int>(blockIdx.x), k0 = tile * T;
    if (k0 >= a.vs->n_free) return;
    const FlowLayout L(T);
    const int span = T + L.hc;   // positions of one buffer: own, then halo
    double2* const buf = flow_lds;
    unsigned char* const rec = reinterpret_cast<unsigned char*>(flow_lds + (B ? 1 : 2) * span);
    {
        const uint4* src = reinterpret_cast<const uint4*>(a.rec + static_cast<int64_t>(tile) * L.bytes);
        uint4* dst = reinterpret_cast<uint4*>(rec);
        for (int q = tid; q < L.bytes / 16; q += BS) dst[q] = src[q];
        for (int q = tid; q <= kMaxValence; q += BS) s_recip[q] = q ? 1.0 / static_cast<double>(q) : 0.0;
        if (tid < 2) {
            s_abort[tid] = 0;
            s_stop[tid] = 0;
        }
    }
    __syncthreads();
    const int32_t* const head = reinterpret_cast<const int32_t*>(rec);
    const int32_t* const halo = reinterpret_cast<const int32_t*>(rec + L.halo);
    const uint16_t* const hcls = reinterpret_cast<const uint16_t*>(rec + L.hcls);
    const uint16_t* const cls = reinterpret_cast<const uint16_t*>(rec + L.cls);
    const uint16_t* const rs = reinterpret_cast<const uint16_t*>(rec + L.rs);
    const uint16_t* const fo = reinterpret_cast<const uint16_t*>(rec + L.fs);
    const uint16_t* const ord = reinterpret_cast<const uint16_t*>(rec + L.ord);
    const uint8_t* const flag = rec + L.flag;
    const uint16_t* const rows = reinterpret_cast<const uint16_t*>(rec + L.rows);
    const uint32_t* const fans = reinterpret_cast<const uint32_t*>(rec + L.fans);
    const int nown = head[0], H = head[1], C = B ? a.fs->n_colors : 1;
    const double2* const c2 = reinterpret_cast<const double2*>(a.coords);
    for (int i = tid; i < nown; i += BS) buf[i] = c2[a.perm ? a.perm[k0 + i] : k0 + i];
    for (int h = tid; h < H; h += BS) {
        const int32_t key = halo[h];
        const double2 p = c2[key < 0 ? key - kFixedKey : (a.perm ? a.perm[key] : key)];
        buf[T + h] = p;
        if (!B) buf[span + T + h] = p;   // fixed nodes stay in both buffers
    }
    __syncthreads();

    const FlowRec t{rs, fo, ord, rows, fans, flag};
    const int g = tid / W, j = tid % W, groups = BS / W;
    const int64_t n2 = 2 * a.n, dcap = static_cast<int64_t>(a.tiles) * waves;
    u64* const dslot = TOL ? a.dmax + static_cast<int64_t>(tile) * waves + wv : nullptr;
    int acc_total = 0, acc0 = 0, acc1 = 0, acc2 = 0, acc3 = 0;   // accepted: all, and the last four sweeps
    double d2 = 0.0;
    int s = 0, phase = 0;
    uint32_t stop = 0;
    NodeRef ref;   // the lane's first node of the class (Form A: of the tile) to come
    if (g < (B ? cls[1] : nown)) load_ref<W>(ref, t, g, j);
    if (tile == 0 && tid == 0) a.fs->t_sweep = wall_clock64();
    while (stop == 0 && (TOL || s < a.iters)) {
        const double2* const cur = buf + (!B && (s & 1) ? span : 0);
        double2* const nxt = buf + (!B && !(s & 1) ? span : 0);
        const int v = s + 1;   // the version this sweep makes
        u64* const ring_v = a.ring + ((a.v0 + v) & 3) * n2;
        u64* const ring_ahead = a.ring + ((a.v0 + v + 2) & 3) * n2;
        int acc = 0;
        bool whole = true;   // every class of the sweep done
        d2 = 0.0;
        for (int c = 0; c < C; ++c) {
            const int lo = B ? cls[c] : 0, hi = B ? cls[c + 1] : nown;
            const bool last_class = c + 1 == C;
            // what this wave has set back so far, before it publishes (stores
            // from before the barrier: they are as good as done)
            wait_stores();
            if (TOL && c == 0 && lane == 0) st_dev(dslot + ((s + 2) & (kFlowSlots - 1)) * dcap, kSent);
            for (int q = lo + g; q < hi; q += groups) {
                if (q != lo + g || (!B && groups < nown)) load_ref<W>(ref, t, q, j);
                const int i = ref.i;
                if (ref.border && j == 0) {
                    st_dev(ring_ahead + 2 * (k0 + i), kSent);
                    st_dev(ring_ahead + 2 * (k0 + i) + 1, kSent);
                }
                double2 o, cd;
                double qo, qn;
                flow_node<W>(ref, t, cur, s_recip, o, cd, qo, qn);
                const bool accepted = GT ? (qn > qo) : (qn >= qo);
                const double nx = accepted ? cd.x : o.x, ny = accepted ? cd.y : o.y;
                if (j == 0) {
                    if (ref.border) {
                        st_dev(ring_v + 2 * (k0 + i), static_cast<u64>(__double_as_longlong(nx)));
                        st_dev(ring_v + 2 * (k0 + i) + 1, static_cast<u64>(__double_as_longlong(ny)));
                    }
                    nxt[i] = make_double2(nx, ny);
                    if (TOL)
                        reinterpret_cast<double2*>(a.hist + (v & (kFlowHist - 1)) * n2)[k0 + i] = make_double2(nx, ny);
                    const double dx = nx - o.x, dy = ny - o.y;
                    const double e = dx * dx + dy * dy;
                    d2 = e > d2 ? e : d2;
                    acc += accepted ? 1 : 0;
                    if (a.bits != nullptr && accepted)
                        atomicOr(a.bits + s * a.words + ((k0 + i) >> 6), 1ull << ((k0 + i) & 63));
                }
            }
            if (B) {   // the next class's node, while this class's values travel
                const int cn = last_class ? 0 : c + 1, q = cls[cn] + g;
                if (q < cls[cn + 1]) load_ref<W>(ref, t, q, j);
            }
            // this class's halo nodes at the new version
            if (!(last_class && v == a.iters)) {
                Waiter w(a.fs, a.wait, a.run);
                const int hlo = B ? hcls[c] : 0, hhi = B ? hcls[c + 1] : head[2];
                for (int h = hlo + tid; h < hhi; h += BS) {
                    const u64* const p = ring_v + 2 * static_cast<int64_t>(halo[h]);
                    for (;;) {
                        const u64 x = ld_dev(p), y = ld_dev(p + 1);
                        if (x != kSent && y != kSent) {
                            nxt[T + h] = make_double2(__longlong_as_double(static_cast<long long>(x)),
                                                      __longlong_as_double(static_cast<long long>(y)));
                            break;
                        }
                        if (TOL) {
                            // the neighbour may have stopped for good
                            const uint32_t dec = ld_dev(&a.fs->decided);
                            if (dec & kFlowStop) {
                                s_stop[phase] = dec;
                                break;
                            }
                        }
                        if (!w.again()) {
                            s_abort[phase] = 1;
                            break;
                        }
                    }
                }
            }
            if (TOL && last_class) {
                const double m = wave_max(d2);
                if (lane == 0) st_dev(dslot + (s & (kFlowSlots - 1)) * dcap, static_cast<u64>(__double_as_longlong(m)));
            }
            if (TOL && last_class && tid == BS - 1) {   // (a wave that rarely has halo nodes to read)
                // sweep v runs once every sweep up to v - kFlowLag is decided;
                // after the last sweep the final decision is awaited
                const uint32_t need = static_cast<uint32_t>(max(v - kFlowLag + 1, 0));
                Waiter w(a.fs, a.wait, a.run);
                for (;;) {
                    const uint32_t dec = ld_dev(&a.fs->decided);
                    if (dec & kFlowStop) {
                        s_stop[phase] = dec;
                        break;
                    }
                    if (v < a.iters && dec >= need) break;
                    if (!w.again()) {
                        s_abort[phase] = 1;
                        break;
                    }
                }
            }
            __syncthreads();
            if (s_abort[phase]) return;   // the abort word is set: no result is taken
            if (TOL) stop = s_stop[phase];
            phase ^= 1;
            if (TOL && stop != 0) {
                whole = last_class;
                break;
            }
        }
        if (whole) {
            acc_total += acc;
            acc3 = acc2;
            acc2 = acc1;
            acc1 = acc0;
            acc0 = acc;
            ++s;
        }
    }
    if (TOL) {
        // the sweeps after the stopping one are taken back
        const int ran = static_cast<int>(stop & ~kFlowStop), lag = s - ran;
        const double2* const fin = reinterpret_cast<const double2*>(a.hist + (ran & (kFlowHist - 1)) * n2);
        for (int i = tid; i < nown; i += BS) reinterpret_cast<double2*>(a.out)[k0 + i] = fin[k0 + i];
        if (lag > 0) acc_total -= acc0;
        if (lag > 1) acc_total -= acc1;
        if (lag > 2) acc_total -= acc2;
        acc0 = lag == 0 ? acc0 : (lag == 1 ? acc1 : (lag == 2 ? acc2 : acc3));
    } else {
        const double2* const fin = buf + (!B && (s & 1) ? span : 0);
        for (int i = tid; i < nown; i += BS) reinterpret_cast<double2*>(a.out)[k0 + i] = fin[i];
    }
    u64 al = static_cast<u64>(acc0), at = static_cast<u64>(acc_total);
    for (int off = 32; off > 0; off >>= 1) {
        const double t = __shfl_xor(d2, off);
        d2 = t > d2 ? t : d2;
        al += __shfl_xor(al, off);
        at += __shfl_xor(at, off);
    }
    if (lane == 0) {
        s_d2[wv] = d2;
        s_last[wv] = al;
        s_tot[wv] = at;
    }
    __syncthreads();
    if (tid == 0) {
        for (int q = 1; q < waves; ++q) {
            d2 = s_d2[q] > d2 ? s_d2[q] : d2;
            al += s_last[q];
            at += s_tot[q];
        }
        a.groups[tile] = FlowGroup{static_cast<u64>(__double_as_longlong(d2)), al, at};
    }
}

// The groups' words folded by a work-group of BS work-items (work-item 0 has
// the result; non-negative doubles order as their bit patterns).
template <int BS>
__device__ __forceinline__ FlowGroup fold_groups(const FlowGroup* __restrict__ groups, int n)
{
    __shared__ FlowGroup s_f[BS / 64];
    u64 m = 0, al = 0, at = 0;
    for (int q = threadIdx.x; q < n; q += BS) {
        const FlowGroup g = groups[q];
        m = g.maxd > m ? g.maxd : m;
        al += g.acc_last;
        at += g.acc_total;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const u64 t = __shfl_xor(m, o);
        m = t > m ? t : m;
        al += __shfl_xor(al, o);
        at += __shfl_xor(at, o);
    }
    if ((threadIdx.x & 63) == 0) s_f[threadIdx.x >> 6] = FlowGroup{m, al, at};
    __syncthreads();
    if (threadIdx.x == 0)
        for (int q = 1; q < BS / 64; ++q) {
            m = s_f[q].maxd > m ? s_f[q].maxd : m;
            al += s_f[q].acc_last;
            at += s_f[q].acc_total;
        }
    return FlowGroup{m, al, at};
}

// Results to the caller's order -- nothing unless every group ran to its end
// -- and the report to the host.
__global__ __launch_bounds__(256) void k_flow_result(FlowArgs a, int tol, double* __restrict__ coords,
                                                     FlowReport* __restrict__ rep, MeshState* __restrict__ ms)
{
    const u64 t_end = wall_clock64();
    const bool gave_up = a.fs->abort == a.run, off = flow_off(a.vs, a.fs) || gave_up;
    const int n_free = a.vs->n_free, sweeps = tol ? static_cast<int>(a.fs->decided & ~kFlowStop) : a.iters;
    if (blockIdx.x == 0) {
        const FlowGroup f = fold_groups<256>(a.groups, off ? 0 : (n_free + a.T - 1) / a.T);
        if (threadIdx.x == 0) {
            rep->vs = *a.vs;
            rep->decline = a.fs->decline;
            rep->abort = gave_up ? 1u : 0u;
            rep->n_colors = a.fs->n_colors;
            rep->sweeps = sweeps;
            rep->maxd = tol ? a.fs->maxd : f.maxd;
            rep->acc_last = f.acc_last;
            rep->acc_total = f.acc_total;
            rep->nnz = a.nbr_end[0];
            rep->ninc = a.tri_end[0];
            rep->t[0] = a.fs->t_begin;
            rep->t[1] = a.fs->t_sweep;
            rep->t[2] = t_end;
            if (ms) ms->s = sweeps;
        }
    }
    if (off) return;
    const double2* const src = reinterpret_cast<const double2*>(a.out);
    const int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (k < n_free) reinterpret_cast<double2*>(coords)[a.perm[k]] = src[k];
}

// What a handle's runs leave on the host.
struct FlowCell {
    uint32_t done;       // the last run whose groups have all left the device
    uint32_t given_up;   // runs given up
};

// The end of a handle's run: the sweep state, from the groups' words (by the
// first work-group; the others find nothing to do).  A handle's call does not
// wait for the device, so when the run was given up (Waiter) the sweeps are
// made here, from the untouched start positions, by kFinishGroups
// work-groups: they take tile steps in order, sweep after sweep, and begin a
// sweep when all steps of the one before have been made.  A group waits only
// for steps dealt before its own, whose groups are running, so the wait ends
// with however few groups the device has room for.  (One group alone took 7 us
// a tile step: 600 sweeps of 100K nodes 842 ms; now 38, and 10 with a launch
// per sweep.)  Calls of very few tiles and
// sweeps (kSerialSteps) are made by one such group to begin with (serial): one
// launch.
// No two groups can be at different sweeps when one of them stops: the grid is
// at most a sweep's tiles, so the steps of the sweep that does not run are not
// all dealt before each group has taken one and left.
constexpr int kFinishBS = 512, kFinishGroups = 64;
template <bool GT>
__global__ __launch_bounds__(kFinishBS) void k_flow_finish(FlowArgs a, int tol, int serial, MeshState* ms, FlowCell* cell)
{
    extern __shared__ double2 flow_lds[];
    __shared__ double s_recip[kMaxValence + 1];
    __shared__ uint32_t s_item;
    __shared__ int s_stop;
    const int tid = threadIdx.x, T = a.T, n_free = a.vs->n_free;
    const int tiles = (n_free + T - 1) / T;
    const bool first = blockIdx.x == 0 && tid == 0, alone = gridDim.x == 1;
    const u64 t_begin = serial ? wall_clock64() : a.fs->t_sweep;
    if (!serial && first) __hip_atomic_store(&cell->done, a.run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    auto close = [&](int ran, u64 maxd, u64 acc_last, u64 acc_total) {
        MeshState m = *ms;
        m.iters = m.s + a.iters;
        m.s += ran;
        m.active = 0;
        m.tol2 = a.tol2;
        m.maxd_cur = m.acc_cur = 0;
        m.maxd_last = maxd;
        m.acc_last = acc_last;
        m.acc_total += acc_total;
        m.t_begin = t_begin;
        m.t_end = wall_clock64();
        *ms = m;
    };
    if (!serial && a.fs->abort != a.run) {   // (no group of the run is there any more)
        if (blockIdx.x != 0) return;
        const FlowGroup f = fold_groups<kFinishBS>(a.groups, tiles);
        if (tid == 0)
            close(tol ? static_cast<int>(a.fs->decided & ~kFlowStop) : a.iters, tol ? a.fs->maxd : f.maxd, f.acc_last,
                  f.acc_total);
        return;
    }
    if (!serial && first)   // (the one writer: no atomic over the bus)
        __hip_atomic_store(&cell->given_up,
                           __hip_atomic_load(&cell->given_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) + 1u,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    const FlowLayout L(T);
    double2* const X = flow_lds;
    unsigned char* const rec = reinterpret_cast<unsigned char*>(flow_lds + T + L.hc);
    for (int q = tid; q <= kMaxValence; q += kFinishBS) s_recip[q] = q ? 1.0 / static_cast<double>(q) : 0.0;
    double2* const buf[2] = {reinterpret_cast<double2*>(const_cast<double*>(a.coords)), reinterpret_cast<double2*>(a.out)};
    FlowState* const fs = a.fs;
    uint32_t next = 0;
    int whole = 0, ran = a.iters;   // sweeps known to be whole; sweeps run
    double m = 0.0;                 // (alone) the sweep's displacement maximum
    u64 acc = 0, total = 0;         // (alone) its accepted nodes, and all sweeps'
    for (;; ++next) {
        __syncthreads();   // s_item and the last tile's LDS are read
        if (tid == 0) s_item = alone ? next : atomicAdd(&fs->dealt, 1u);
        __syncthreads();
        const int s = static_cast<int>(s_item / static_cast<uint32_t>(tiles)),
                  tile = static_cast<int>(s_item % static_cast<uint32_t>(tiles));
        if (s > whole) {
            bool stop = tol && a.tol2 > 0.0;
            if (alone) {
                stop = stop && m < a.tol2;
                if (!stop && s < a.iters) {
                    m = 0.0;
                    acc = 0;
                }
            } else if (s < a.iters) {
                if (tid == 0) {
                    while (ld_dev(&fs->made) < static_cast<uint32_t>(s) * static_cast<uint32_t>(tiles))
                        __builtin_amdgcn_s_sleep(1);
                    s_stop = stop && __longlong_as_double(static_cast<long long>(ld_dev(&fs->r_maxd[(s - 1) & 3]))) < a.tol2;
                }
                __syncthreads();
                __threadfence();   // the other groups' positions
                stop = s_stop != 0;
            }
            whole = s;
            if (stop && s < a.iters) ran = s;
            if (stop) break;
        }
        if (s >= a.iters) break;
        const double2* const in = buf[s & 1];
        double2* const to = buf[(s & 1) ^ 1];
        const uint4* src = reinterpret_cast<const uint4*>(a.rec + static_cast<int64_t>(tile) * L.bytes);
        for (int q = tid; q < L.bytes / 16; q += kFinishBS) reinterpret_cast<uint4*>(rec)[q] = src[q];
        __syncthreads();
        const int32_t* const head = reinterpret_cast<const int32_t*>(rec);
        const int32_t* const halo = reinterpret_cast<const int32_t*>(rec + L.halo);
        const int k0 = tile * T, nown = head[0];
        for (int i = tid; i < nown; i += kFinishBS) X[i] = in[k0 + i];
        for (int h = tid; h < head[1]; h += kFinishBS) X[T + h] = in[halo[h] < 0 ? halo[h] - kFixedKey : halo[h]];
        __syncthreads();
        const FlowRec t{reinterpret_cast<const uint16_t*>(rec + L.rs),   reinterpret_cast<const uint16_t*>(rec + L.fs),
                        reinterpret_cast<const uint16_t*>(rec + L.ord),  reinterpret_cast<const uint16_t*>(rec + L.rows),
                        reinterpret_cast<const uint32_t*>(rec + L.fans), rec + L.flag};
        double d2 = 0.0;
        u64 n_acc = 0;
        for (int q = tid; q < nown; q += kFinishBS) {
            NodeRef ref;
            load_ref<1>(ref, t, q, 0);
            double2 o, c;
            double qo, qn;
            flow_node<1>(ref, t, X, s_recip, o, c, qo, qn);
            const bool accepted = GT ? (qn > qo) : (qn >= qo);
            const double nx = accepted ? c.x : o.x, ny = accepted ? c.y : o.y;
            to[k0 + ref.i] = make_double2(nx, ny);
            const double dx = nx - o.x, dy = ny - o.y, e = dx * dx + dy * dy;
            d2 = e > d2 ? e : d2;
            n_acc += accepted ? 1 : 0;
        }
        __threadfence();   // the next sweep reads these positions
        group_fold<kFinishBS>(d2, n_acc);
        if (alone) {
            m = d2 > m ? d2 : m;
            acc += n_acc;
            total += n_acc;
        } else if (tid == 0) {
            if (d2 > 0.0) atomicMax(&fs->r_maxd[s & 3], static_cast<u64>(__double_as_longlong(d2)));
            if (n_acc) {
                atomicAdd(&fs->r_acc[s & 3], n_acc);
                atomicAdd(&fs->r_total, n_acc);
            }
            if (tile == 0) {   // the next sweep's, which nobody reads or adds to before this step is made
                st_dev(&fs->r_maxd[(s + 1) & 3], 0ull);
                st_dev(&fs->r_acc[(s + 1) & 3], 0ull);
            }
            wait_stores();
            atomicAdd(&fs->made, 1u);
        }
    }
    if (!alone) {   // the last group to leave ends the run
        __syncthreads();
        if (tid == 0) s_item = atomicAdd(&fs->left, 1u);
        __syncthreads();
        if (s_item != gridDim.x - 1) return;
        __threadfence();
        m = __longlong_as_double(static_cast<long long>(ld_dev(&fs->r_maxd[(ran - 1) & 3])));
        acc = ld_dev(&fs->r_acc[(ran - 1) & 3]);
        total = ld_dev(&fs->r_total);
    }
    if ((ran & 1) == 0)   // the result belongs in `out`
        for (int k = tid; k < n_free; k += kFinishBS) buf[1][k] = buf[0][k];
    // after a run given up: the exchange as a new mesh finds it
    for (int64_t q = serial ? 8 * a.n : tid; q < 8 * a.n; q += kFinishBS) a.ring[q] = kSent;
    __syncthreads();
    if (tid == 0) {
        close(ran, static_cast<u64>(__double_as_longlong(m)), acc, total);
        if (!alone) {
            fs->dealt = fs->made = fs->left = 0;
            for (int k = 0; k < 4; ++k) fs->r_maxd[k] = fs->r_acc[k] = 0;
            fs->r_total = 0;
        }
    }
}

// ------------------------------------------------------------------ host --

// Work-groups of flow launches in flight per device: at most two per compute
// unit (each takes at most 80 KB of LDS, 512 work-items and 128 registers),
// so that all of them are resident together and none waits for a group that
// cannot start.  A call that finds too few left takes the other kernels.
// A handle's calls return before their work is done: it keeps its places
// between calls, and another taker gets them once the device has written the
// number of the last of them to the host.  (Not by asking an event: the
// runtime takes a query of an event whose stream is being captured meanwhile
// for an error of the capture.)
class FlowSlots {
public:
    ~FlowSlots() { give(); }
    // Places for `groups` work-groups (kept from before, or taken now).
    bool take(int groups)
    {
        std::lock_guard<std::mutex> lk(mu);
        if (held) {
            if (resting(dev)) return false;
            word = nullptr;   // in use: not to be taken back
            return true;
        }
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
        if (limit[dev] == 0) {
            int cus = 0;
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
                (void)hipGetLastError();
                return false;
            }
            limit[dev] = 2 * cus;
        }
        if (resting(dev)) return false;
        if (used[dev] + groups > limit[dev])
            for (size_t k = keepers.size(); k-- > 0;) {
                FlowSlots* const f = keepers[k];
                if (f->dev == dev && f->word && __atomic_load_n(f->word, __ATOMIC_ACQUIRE) == f->last) f->drop();
            }
        if (used[dev] + groups > limit[dev]) return false;
        used[dev] += groups;
        held = groups;
        return true;
    }
    // Kept until *w is `run`, or longer.
    void keep(const uint32_t* w, uint32_t run)
    {
        std::lock_guard<std::mutex> lk(mu);
        if (!held) return;
        word = w;
        last = run;
        if (std::find(keepers.begin(), keepers.end(), this) == keepers.end()) keepers.push_back(this);
    }
    void give()
    {
        std::lock_guard<std::mutex> lk(mu);
        if (held) drop();
    }
    // A run in these places has been given up: other work has the device
    // (another process that runs this path too, or a kernel that stays long).
    // No places are given out there for kRest, so that waits in vain take a
    // fiftieth of the time at most; calls take the other kernels meanwhile.
    void rest()
    {
        std::lock_guard<std::mutex> lk(mu);
        if (dev >= 0) until[dev] = Clock::now() + kRest;
    }
    static void wake()
    {
        std::lock_guard<std::mutex> lk(mu);
        for (auto& t : until) t = Clock::time_point();
    }

private:
    using Clock = std::chrono::steady_clock;
    static constexpr std::chrono::milliseconds kRest{100};
    static bool resting(int d) { return until[d] != Clock::time_point() && Clock::now() < until[d]; }
    void drop()
    {
        used[dev] -= held;
        held = 0;
        word = nullptr;
        keepers.erase(std::remove(keepers.begin(), keepers.end(), this), keepers.end());
    }
    static std::mutex mu;
    static int used[64], limit[64];
    static Clock::time_point until[64];
    static std::vector<FlowSlots*> keepers;
    int dev = -1, held = 0;
    const uint32_t* word = nullptr;   // set while kept between calls
    uint32_t last = 0;
};
std::mutex FlowSlots::mu;
int FlowSlots::used[64], FlowSlots::limit[64];
FlowSlots::Clock::time_point FlowSlots::until[64];
std::vector<FlowSlots*> FlowSlots::keepers;

// Tile size, lanes per node and work-group size for n nodes.  The smallest
// tiles that still give every compute unit at most one group win while they
// last (a group then takes one pass per sweep or class, with several lanes
// on a node's fan); beyond that, tiles of 512 nodes, two groups per compute
// unit at most.  Microseconds per sweep, the shape taken against the next:
//   Form A: 14.4K nodes 2.9 (T 64, 4 lanes) against 3.1 (T 128); 32.4K 3.2
//   (T 128, 4 lanes) against 3.4 (T 64); 98.6K 5.8 (T 512) against 6.2
//   (T 256, 2 lanes); 230K 10.0;
//   Form B: 14.4K 14.0 (T 64, 8 lanes) against 14.7; 32.4K 15.0 (T 128, 8
//   lanes) against 15.3; 98.6K 18.0 (T 512, 4 lanes) against 19.2; 230K 24.0.
struct FlowShape {
    int T, W, BS;
};

FlowShape flow_shape(int32_t n, bool b)
{
    if (n <= 64 * 256) return FlowShape{64, b ? 8 : 4, 256};
    if (n <= 128 * 256) return FlowShape{128, b ? 8 : 4, 512};
    if (n <= 256 * 256) return FlowShape{256, b ? 8 : 2, 512};
    return FlowShape{512, b ? 4 : 1, 512};
}
constexpr int32_t kFlowMaxNodes = 512 * 500;
constexpr int32_t kFlowMaxSweeps = 1 << 20;   // of one launch (times 500 tiles: within 32 bits)
// 2 ms of the 100 MHz clock: a thousand exchanges, and longer than most
// launches of this library keep a place.  (It was 2 s: two processes with a
// medium mesh each could hold half of the other's room for that long, and
// eight threads that run one-call smooths, handles, a batch, a server and
// adjacencies at once got through 0.3K smooths a second; 1.7K with 5 ms and a
// rest of 500, 1.8K with 2 and 100.)
constexpr u64 kFlowWait = 200000ull;

std::atomic<int64_t> g_counts[4];             // sl_one_launch_counts
enum { kCountRun, kCountDeclined, kCountGivenUp, kCountNoRoom };
void count(int what, int64_t by = 1) { g_counts[what].fetch_add(by, std::memory_order_relaxed); }

thread_local double t_wait_ms = -1.0;         // sl_one_launch_wait
u64 wait_limit() { return t_wait_ms < 0.0 ? kFlowWait : static_cast<u64>(t_wait_ms / kTickMs); }

// Automatic choices only, in double precision and the default order.
bool flow_options(const sl_options& o, int32_t n)
{
    return o.kernel == SL_KERNEL_AUTO && o.precision == SL_F64 && o.reorder == SL_REORDER_HILBERT && o.tile_nodes == 0 &&
           o.tile_wg_per_cu == 0 && o.block_size == 0 && n <= kFlowMaxNodes;
}

size_t flow_lds_bytes(const FlowShape& p, bool b)
{
    const FlowLayout L(p.T);
    return static_cast<size_t>(b ? 1 : 2) * static_cast<size_t>(p.T + L.hc) * 16 + static_cast<size_t>(L.bytes);
}

template <bool B, int W>
const void* flow_kernel(bool gt, bool tol)
{
    if (gt) return tol ? reinterpret_cast<const void*>(&k_sweep_flow<B, W, true, true>)
                       : reinterpret_cast<const void*>(&k_sweep_flow<B, W, true, false>);
    return tol ? reinterpret_cast<const void*>(&k_sweep_flow<B, W, false, true>)
               : reinterpret_cast<const void*>(&k_sweep_flow<B, W, false, false>);
}

sl_status launch_flow(const FlowArgs& a, const FlowShape& p, bool b, bool gt, bool tol, hipStream_t st)
{
    const void* fn = nullptr;
    if (b) fn = p.W == 8 ? flow_kernel<true, 8>(gt, tol) : flow_kernel<true, 4>(gt, tol);
    else fn = p.W == 4 ? flow_kernel<false, 4>(gt, tol)
                       : (p.W == 2 ? flow_kernel<false, 2>(gt, tol) : flow_kernel<false, 1>(gt, tol));
    const size_t lds = flow_lds_bytes(p, b);
    if (lds > 64 * 1024) {
        (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        (void)hipGetLastError();
    }
    FlowArgs args = a;
    void* argv[] = {&args};
    SL_HIP(hipLaunchKernel(fn, dim3(static_cast<unsigned>(a.tiles + (tol ? 1 : 0))), dim3(static_cast<unsigned>(p.BS)),
                           argv, lds, st));
    return SL_OK;
}

template <bool CLS>
void launch_build(const FlowBuildArgs& b, int T, int tiles, hipStream_t st)
{
    if (T == 64) k_flow_build<64, CLS><<<tiles, 256, 0, st>>>(b);
    else if (T == 128) k_flow_build<128, CLS><<<tiles, 256, 0, st>>>(b);
    else if (T == 256) k_flow_build<256, CLS><<<tiles, 256, 0, st>>>(b);
    else k_flow_build<512, CLS><<<tiles, 512, 0, st>>>(b);
}

}  // namespace

sl_status flow_run(const SetupArgs& a, const sl_options& o, int32_t iterations, double tol, sl_report* report,
                   double* coords, hipStream_t st, unsigned char* ws, size_t ws_bytes, bool* done, FlowSeen* seen)
{
    *done = false;
    seen->valid = false;
    const int32_t n = a.n;
    const bool b = o.form == SL_INPLACE_COLORED, tl = tol > 0.0;
    // automatic choices only, in double precision and the default order, for
    // meshes whose tiles the device holds all at once
    if (!flow_options(o, n) || iterations < 1 || iterations > kFlowMaxSweeps || a.n_tris <= 0 || !a.nbr_idx || !a.tri_idx || !a.tris)
        return SL_OK;
    const FlowShape p = flow_shape(n, b);
    const FlowLayout L(p.T);
    const int tiles = div_up(n, p.T), waves = p.BS / 64;
    FlowSlots slots;
    if (!slots.take(tiles + (tl ? 1 : 0))) {
        count(kCountNoRoom);
        return SL_OK;
    }

    const size_t un = static_cast<size_t>(n);
    FlowOrder f{};
    f.bits = hilbert_bits(n, 1);
    const int64_t nbk = int64_t(1) << (2 * f.bits);
    const int gb = div_up(n, 256);
    const int64_t words = (static_cast<int64_t>(n) + 63) / 64;
    const bool want_bits = o.flags_out != nullptr;
    const size_t n_bits = want_bits ? static_cast<size_t>(words) * static_cast<size_t>(iterations) : 0;
    const size_t n_dmax = tl ? static_cast<size_t>(kFlowSlots) * tiles * waves : 0;
    const size_t bytes = Arena::piece(sizeof(ValStats)) + Arena::piece(sizeof(ValStats) * static_cast<size_t>(val_groups(n))) +
                         Arena::piece(4 * static_cast<size_t>(nbk)) + Arena::piece(4 * static_cast<size_t>(nbk + 1)) +
                         scan_bytes(nbk) + 5 * Arena::piece(4 * un) + Arena::piece(sizeof(FlowState)) +
                         Arena::piece(static_cast<size_t>(tiles) * L.bytes) + Arena::piece(4 * 16 * un) +
                         Arena::piece(16 * un) + Arena::piece((tl ? kFlowHist : 0) * 16 * un) + Arena::piece(8 * n_dmax) +
                         Arena::piece(sizeof(FlowGroup) * static_cast<size_t>(tiles)) + Arena::piece(8 * n_bits) +
                         Arena::piece(sizeof(MeshState));
    if (ws && bytes > ws_bytes) return SL_OK;
    PinnedPad pad;
    sl_status r = pad.init();
    if (r) return r;
    static_assert(sizeof(FlowReport) <= kPadBytes, "report size");
    Arena ar;
    if (ws) {
        ar.adopt(ws, ws_bytes);
    } else if ((r = ar.reserve(bytes, st))) {
        if (r != SL_ENOMEM) return r;
        set_error("");
        return SL_OK;   // no room for it: the other kernels' arrays may still fit
    }
    struct GiveBack {
        Arena& ar;
        hipStream_t st;
        ~GiveBack()
        {
            ar.release(st);
            (void)hipStreamSynchronize(st);   // before the pad and the slots go back
        }
    } give_back{ar, st};

    FlowArgs fa{};
    FlowState* fs = nullptr;
    ValStats* vs = nullptr;
    int32_t *color = nullptr, *perm = nullptr;
    unsigned char* rec = nullptr;
    MeshState* ms = nullptr;
    uint64_t* bits = nullptr;
    if ((r = ar.take(&vs, 1)) || (r = ar.take(&f.part, val_groups(n))) || (r = ar.take(&f.count, nbk)) ||
        (r = ar.take(&f.start, nbk + 1)) || (r = ar.take(&f.key, un)) || (r = ar.take(&f.rank, un)) ||
        (r = ar.take(&f.new_of_old, un)) || (r = ar.take(&perm, un)) || (r = ar.take(&color, un)) ||
        (r = ar.take(&fs, 1)) || (r = ar.take(&rec, static_cast<size_t>(tiles) * L.bytes)) ||
        (r = ar.take(&fa.ring, 4 * 2 * un)) || (r = ar.take(&fa.out, 2 * un)) || (r = ar.take(&fa.hist, (tl ? kFlowHist : 0) * 2 * un)) ||
        (r = ar.take(&fa.dmax, n_dmax)) || (r = ar.take(&fa.groups, static_cast<size_t>(tiles))) ||
        (r = ar.take(&bits, n_bits)) || (r = ar.take(&ms, 1)))
        return r;
    f.vs = vs;
    f.perm = perm;
    fa.vs = vs;
    fa.fs = fs;
    fa.perm = perm;
    fa.coords = a.coords;
    fa.rec = rec;
    fa.bits = want_bits ? reinterpret_cast<u64*>(bits) : nullptr;
    fa.words = words;
    fa.n = n;
    fa.T = p.T;
    fa.tiles = tiles;
    fa.iters = iterations;
    fa.tol2 = tl ? tol * tol : 0.0;
    fa.wait = wait_limit();
    fa.run = kOneCall;
    fa.nbr_end = a.nbr_ptr + n;
    fa.tri_end = a.tri_ptr + n;

    const FlowInitArgs ia{vs, fs, f.count, nbk, b ? color : nullptr, n, fa.ring + 2 * un, fa.dmax,
                          static_cast<int64_t>(n_dmax), fa.bits, static_cast<int64_t>(n_bits)};
    k_flow_init<<<std::min(gb, 1024), 256, 0, st>>>(ia);
    if ((r = queue_flow_order(a, o, f, ar, st))) return r;
    if (b) k_flow_color<<<gb, 256, 0, st>>>(a.nbr_ptr, a.nbr_idx, a.boundary, color, n, vs, fs, fa.wait);
    const FlowBuildArgs ba{vs, fs, perm, f.new_of_old, a.nbr_ptr, a.nbr_idx, a.tri_ptr, a.tri_idx, a.tris, color, rec};
    if (b) launch_build<true>(ba, p.T, tiles, st);
    else launch_build<false>(ba, p.T, tiles, st);
    SL_HIP(hipGetLastError());
    if ((r = launch_flow(fa, p, b, o.accept == SL_ACCEPT_GT, tl, st))) return r;
    FlowReport* const rep = static_cast<FlowReport*>(pad.p);
    k_flow_result<<<gb, 256, 0, st>>>(fa, tl ? 1 : 0, coords, rep, want_bits ? ms : nullptr);
    SL_HIP(hipGetLastError());
    SL_HIP(hipStreamSynchronize(st));

    const FlowReport h = *rep;
    // (what the checks found wrong, the other path finds and reports too; it
    // takes rows that are not symmetric or incidences that disagree in Form A)
    *seen = FlowSeen{(h.vs.err & ~(b ? 0u : static_cast<uint32_t>(VE_ASYM) | VI_INCIDENCE)) == 0, h.vs, h.nnz, h.ninc};
    const bool late = h.abort != 0 || (h.decline & kDeclineColor) != 0;
    if (late || h.vs.err != 0 || h.vs.n_free == 0 || h.decline || h.n_colors > kFlowClasses) {
        count(late ? kCountGivenUp : kCountDeclined);
        if (late) slots.rest();
        return SL_OK;
    }
    count(kCountRun);
    if (want_bits) {
        if ((r = unpermute_flags_raw(bits, words, f.new_of_old, n, h.vs.n_free, iterations, ms, o.flags_out, st))) return r;
        SL_HIP(hipStreamSynchronize(st));
    }
    *done = true;
    if (report) {
        sl_report rp{};
        rp.iterations_run = h.sweeps;
        rp.n_colors = b ? h.n_colors : 0;
        std::memcpy(&rp.max_disp_sq_last, &h.maxd, sizeof(double));
        rp.accepted_last = static_cast<int64_t>(h.acc_last);
        rp.accepted_total = static_cast<int64_t>(h.acc_total);
        rp.setup_ms = static_cast<double>(h.t[1] - h.t[0]) * kTickMs;
        rp.sweep_ms = static_cast<double>(h.t[2] - h.t[1]) * kTickMs;
        // the kernel family of the mesh's size and form, as without this path
        rp.kernel_used = !b ? SL_KERNEL_TILE
                            : (resident_fits(n, h.nnz, h.ninc, true) ? SL_KERNEL_RESIDENT : SL_KERNEL_NODE);
        rp.tile_nodes = !b ? tile_size_for(o, n) : 0;
        *report = rp;
    }
    return SL_OK;
}

// -------------------------------------------------------------- handles --

struct FlowMesh {
    Arena ar, tol;          // (tol: what only runs with a tolerance need, from the first of them on)
    FlowShape p{};
    int tiles = 0;
    FlowArgs fa{};
    PinnedCell cell;        // (before the places, which look at it until they are given back)
    FlowSlots slots;
    uint32_t run = 0;       // runs queued
    uint32_t noted = 0;     // runs given up, as far as counted
    bool fresh = true;      // the exchange's slots are to be set up before the next run
    uint32_t version = 0;   // of the positions, as the exchange counts them
};

namespace {

__global__ void k_flow_mesh_begin(ValStats* vs, FlowState* fs, int32_t n_free)
{
    if (threadIdx.x == 0) {
        *vs = ValStats{};
        vs->n_free = n_free;
        *fs = FlowState{};
    }
}

__global__ void k_flow_mesh_tell(const FlowState* __restrict__ fs, uint32_t* __restrict__ out)
{
    if (threadIdx.x == 0) *out = fs->decline;
}

sl_status launch_finish(const FlowArgs& a, const FlowShape& p, int32_t n_free, bool gt, bool tol, bool serial,
                        MeshState* state, FlowCell* cell, hipStream_t st)
{
    const FlowLayout L(p.T);
    const size_t lds = static_cast<size_t>(p.T + L.hc) * 16 + static_cast<size_t>(L.bytes);
    const int groups = serial ? 1 : std::min(kFinishGroups, div_up(n_free, p.T));
    (gt ? k_flow_finish<true> : k_flow_finish<false>)<<<groups, kFinishBS, lds, st>>>(a, tol ? 1 : 0, serial ? 1 : 0, state,
                                                                                      cell);
    SL_HIP(hipGetLastError());
    return SL_OK;
}

// Tiles times sweeps up to which one work-group makes them all: 4 tile steps
// take some 15 us, about what the two launches of a run take before and
// after its sweeps.
constexpr int64_t kSerialSteps = 4;

}  // namespace

bool flow_wanted(const sl_options& o, int32_t n)
{
    return flow_options(o, n) && o.form == SL_JACOBI && o.layout == SL_AOS;
}

void flow_mesh_free(FlowMesh*& f, hipStream_t st)
{
    if (!f) return;
    f->ar.release(st);
    f->tol.release(st);
    delete f;
    f = nullptr;
}

sl_status flow_mesh_build(const SetupArgs& a, DevMesh& m, hipStream_t st)
{
    const size_t un = static_cast<size_t>(m.n);
    auto* f = new FlowMesh;
    f->p = flow_shape(m.n, false);
    f->tiles = div_up(m.n, f->p.T);
    const FlowLayout L(f->p.T);
    FlowArgs& fa = f->fa;
    unsigned char* rec = nullptr;
    ValStats* vs = nullptr;
    PinnedPad pad;
    sl_status r = pad.init();
    if (r || (r = f->cell.init()) || (r = f->ar.reserve(Arena::piece(sizeof(ValStats)) + Arena::piece(sizeof(FlowState)) +
                                    Arena::piece(static_cast<size_t>(f->tiles) * L.bytes) + Arena::piece(4 * 16 * un) +
                                    Arena::piece(sizeof(FlowGroup) * static_cast<size_t>(f->tiles)),
                                st)) ||
        (r = f->ar.take(&vs, 1)) || (r = f->ar.take(&fa.fs, 1)) ||
        (r = f->ar.take(&rec, static_cast<size_t>(f->tiles) * L.bytes)) || (r = f->ar.take(&fa.ring, 8 * un)) ||
        (r = f->ar.take(&fa.groups, static_cast<size_t>(f->tiles)))) {
        flow_mesh_free(f, st);
        if (r != SL_ENOMEM) return r;
        set_error("");
        return SL_OK;   // no room for it: the tile path
    }
    fa.vs = vs;
    fa.rec = rec;
    fa.n = m.n;
    fa.T = f->p.T;
    fa.tiles = f->tiles;
    *static_cast<FlowCell*>(f->cell.p) = FlowCell{};
    k_flow_mesh_begin<<<1, 64, 0, st>>>(vs, fa.fs, m.n_free);
    const FlowBuildArgs ba{vs, fa.fs, m.perm, m.new_of_old, a.nbr_ptr, a.nbr_idx, a.tri_ptr, a.tri_idx, a.tris, nullptr, rec};
    launch_build<false>(ba, f->p.T, f->tiles, st);
    k_flow_mesh_tell<<<1, 64, 0, st>>>(fa.fs, static_cast<uint32_t*>(pad.p));
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(st) != hipSuccess) {
        flow_mesh_free(f, st);
        return fail(SL_EDEVICE, "building the flow records failed");
    }
    if (*static_cast<const uint32_t*>(pad.p) != 0 || m.n_free == 0) {
        flow_mesh_free(f, st);   // does not fit: the tile path
        return SL_OK;
    }
    m.flow = f;
    return SL_OK;
}

sl_status flow_mesh_sweeps(const DevMesh& m, int cur, int32_t accept, int32_t iterations, double tol2, MeshState* state,
                           hipStream_t st, bool* done)
{
    *done = false;
    FlowMesh* const f = m.flow;
    const bool tl = tol2 > 0.0;
    // a captured stream's work may run any number of times, later: not with places taken now
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (!f || iterations < 2 || iterations > kFlowMaxSweeps) return SL_OK;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return SL_OK;
    }
    const bool gt = accept == SL_ACCEPT_GT;
    const int64_t n_dmax = static_cast<int64_t>(kFlowSlots) * f->tiles * (f->p.BS / 64);
    if (tl && !f->fa.hist) {
        const size_t n2 = static_cast<size_t>(kFlowHist) * 2 * static_cast<size_t>(m.n);
        sl_status r = f->tol.reserve(Arena::piece(8 * n2) + Arena::piece(8 * static_cast<size_t>(n_dmax)), st);
        if (r == SL_ENOMEM) {
            set_error("");
            return SL_OK;
        }
        if (r || (r = f->tol.take(&f->fa.dmax, static_cast<size_t>(n_dmax))) || (r = f->tol.take(&f->fa.hist, n2))) return r;
    }
    FlowArgs a = f->fa;
    a.coords = static_cast<const double*>(m.X[cur]);
    a.out = static_cast<double*>(m.X[cur ^ 1]);
    a.iters = iterations;
    a.tol2 = tol2;
    a.wait = wait_limit();
    if (static_cast<int64_t>(f->tiles) * iterations <= kSerialSteps) {
        *done = true;
        count(kCountRun);
        return launch_finish(a, f->p, m.n_free, gt, tl, true, state, nullptr, st);
    }
    if (!f->slots.take(f->tiles + 1)) {   // (+ 1: a run with a tolerance has a controller)
        count(kCountNoRoom);
        return SL_OK;
    }
    if (f->fresh || tl) {
        // (a run with a tolerance leaves groups some sweeps apart)
        f->version = 0;
        const FlowInitArgs ia{nullptr, a.fs, nullptr, 0, nullptr, m.n, a.ring + 2 * static_cast<int64_t>(m.n), a.dmax,
                              tl ? n_dmax : 0, nullptr, 0};
        k_flow_init<<<std::min(div_up(m.n, 256), 1024), 256, 0, st>>>(ia);
        SL_HIP(hipGetLastError());
    }
    a.v0 = static_cast<int32_t>(f->version & 3u);
    if (++f->run == 0) f->run = 1;
    a.run = f->run;
    sl_status r = launch_flow(a, f->p, false, gt, tl, st);
    FlowCell* const cell = static_cast<FlowCell*>(f->cell.p);
    if (r || (r = launch_finish(a, f->p, m.n_free, gt, tl, false, state, cell, st))) return r;
    f->slots.keep(&cell->done, f->run);
    count(kCountRun);
    f->fresh = tl;
    f->version += static_cast<uint32_t>(iterations);
    *done = true;
    return SL_OK;
}

void flow_mesh_note(FlowMesh* f)
{
    if (!f) return;
    const uint32_t n = __atomic_load_n(&static_cast<const FlowCell*>(f->cell.p)->given_up, __ATOMIC_ACQUIRE);
    if (n == f->noted) return;
    count(kCountGivenUp, static_cast<int32_t>(n - f->noted));
    f->noted = n;
    f->slots.rest();
}

}  // namespace sl

extern "C" {

void sl_one_launch_counts(int64_t counts[4])
{
    for (int k = 0; counts && k < 4; ++k) counts[k] = sl::g_counts[k].load(std::memory_order_relaxed);
}

void sl_one_launch_wait(double ms)
{
    sl::t_wait_ms = ms;
    if (ms < 0.0) sl::FlowSlots::wake();
}

}  // extern "C"
