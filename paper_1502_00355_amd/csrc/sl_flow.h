// The flow path: small and medium meshes, every sweep in one launch
// (sl_flow.hip), with the setup kernels it shares (sl_setup.hip).
#pragma once

#include "sl_common.h"

namespace sl {

constexpr int kFlowClasses = 32;               // colour classes at most (Form B)
constexpr uint32_t kFlowStop = 0x80000000u;    // FlowState::decided: no sweep after this count

// Device state of one call, zeroed before it.
struct FlowState {
    uint32_t decline;       // != 0: the mesh does not fit the tiles' limits
    uint32_t abort;         // number of the run (never 0) in which a wait took too long last
    int32_t n_colors;       // colour classes (Form B)
    uint32_t pad0[29];
    uint32_t decided;       // with a tolerance: sweeps decided, | kFlowStop with the last one
    uint32_t pad1[31];
    unsigned long long maxd;   // with a tolerance: displacement maximum of the last sweep
    unsigned long long t_begin, t_sweep;   // the device's clock at the call's first kernel and at the sweeps
    // zero but while k_flow_finish makes the sweeps of a run given up: tile
    // steps dealt and made, groups that have left, and displacement maxima and
    // accepted counts by sweep (mod 4) and in all
    uint32_t dealt, made, left, pad2;
    unsigned long long r_maxd[4], r_acc[4], r_total;
};

// What a tile's work-group leaves.
struct FlowGroup {
    unsigned long long maxd, acc_last, acc_total;
};

// What the host reads back, written by the last kernel into pinned memory.
struct FlowReport {
    ValStats vs;
    uint32_t decline, abort;
    int32_t n_colors, sweeps;
    unsigned long long maxd, acc_last, acc_total;
    unsigned long long t[3];     // clock: first kernel, first sweep, after the last
    int32_t nnz, ninc;           // nbr_ptr[n], tri_ptr[n]
};

// Arrays of the flow path's node order.
struct FlowOrder {
    ValStats *vs, *part;          // the mesh's statistics; one slot per work-group of the checks
    int32_t *count, *start;       // [buckets], [buckets + 1]
    int32_t *key, *rank;          // [n]
    int32_t *new_of_old, *perm;   // [n]; fixed nodes: -1; free nodes only
    int bits;
};

// Bits per axis of the Hilbert cells of a mesh of n free nodes in nc classes.
int hilbert_bits(int64_t n_free, int nc);
// Work-groups of the node checks (slots of FlowOrder::part).
int val_groups(int32_t n);
// Arena bytes of a scan's temporaries.
size_t scan_bytes(int64_t n);
// Queues the checks (with symmetry of the rows, and for Form A the incidence
// rows') and the Hilbert order of the free nodes; nothing is read back.
sl_status queue_flow_order(const SetupArgs& a, const sl_options& o, const FlowOrder& f, Arena& scratch, hipStream_t st);
// SL_OK, or the error that the checks' bits stand for.
sl_status validation_status(uint32_t err, const sl_options& o);
// Free nodes per tile that the tile path would take.
int32_t tile_size_for(const sl_options& o, int32_t n);
// Accept bits to the caller's layout: `words` 64-bit words per sweep.
sl_status unpermute_flags_raw(const uint64_t* bits, int64_t words, const int32_t* new_of_old, int32_t n, int32_t n_free,
                              int32_t iterations, const MeshState* state, uint8_t* out, hipStream_t st);

// Runs a whole call on the flow path when options, size and the device's
// free groups allow it.  *done = false (with SL_OK): not run, or the mesh
// turned out not to fit; the caller's arrays are untouched.  ws / ws_bytes:
// a region to carve every device array from, instead of allocating.  The
// CSR ends in `a` need not be known (-1).  *seen: what the checks found, when
// they ran and found nothing that the call will fail for.
struct FlowSeen {
    bool valid = false;
    ValStats vs;
    int32_t nnz, ninc;   // nbr_ptr[n], tri_ptr[n]
};
sl_status flow_run(const SetupArgs& a, const sl_options& o, int32_t iterations, double tol, sl_report* report,
                   double* coords, hipStream_t st, unsigned char* ws, size_t ws_bytes, bool* done, FlowSeen* seen);

// A set-up mesh's part of the flow path (mesh handles): its tile records and
// the exchange's slots.  Built by setup when DevMesh::want_flow is set; null
// when the mesh does not fit.
sl_status flow_mesh_build(const SetupArgs& a, DevMesh& m, hipStream_t st);
void flow_mesh_free(FlowMesh*& f, hipStream_t st);
// Whether handles of a mesh of n nodes with these (caller's) options have one.
bool flow_wanted(const sl_options& o, int32_t n);
// Queues `iterations` sweeps of m from buffer `cur` into the other one (the
// free nodes; *state counts them, as the per-sweep closes would) when the
// device has room for its groups now; *done tells.
sl_status flow_mesh_sweeps(const DevMesh& m, int cur, int32_t accept, int32_t iterations, double tol2, MeshState* state,
                           hipStream_t st, bool* done);
// Counts runs of f that were given up and have not been counted yet (when the
// host has waited for them, or some time later).
void flow_mesh_note(FlowMesh* f);

}  // namespace sl
