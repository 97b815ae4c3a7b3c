// sg_launch.h -- launch interface between the C ABI (host) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "sg_internal.h"

namespace sg {

struct ExpArgs {
    int64_t n;
    const int32_t* f;
    const float* b;
    const float* v;
    int32_t K;
    const float* W;
    int32_t* f_out;
    float* b_out;
    float* p_out;
    float* v_out;
    float* W_out;
    int32_t* status;
    int32_t* n_cross;
    uint64_t* seq_hash;
    int32_t max_steps;
    float snap;
    uint32_t debug;
    int32_t rays_per_lane;   // persistent walk: 1 or 2 rays per lane
};

struct BwdArgs {
    int64_t n;
    int32_t mode;           // 0 extrinsic proxy, 1 geodesic finite differences
    const int32_t* f;
    const float* b;
    const float* v;
    const int32_t* f_out;   // saved forward outputs (extrinsic proxy; vertex gradient and GFD without a re-walk)
    const float* b_out;
    const float* v_out;
    const int32_t* status_in;   // the forward's saved per-ray status, or null
    const float* g;         // dL/dp', or null (zero)
    const float* g_bo;      // dL/db' [n,3] (end barycentrics), or null
    const float* g_v;       // dL/dv' [n,3], or null
    const float* g_W;       // dL/dW' [n,K,3], or null
    int32_t K;              // transported vectors per query (g_W, grad_W)
    float* grad_v;
    float* grad_b;
    float* grad_W;          // dL/dW [n,K,3] (with g_W)
    float eps_v, eps_p;
    int32_t max_steps;
    float snap;
    double* grad_X;         // [n_verts, 3] accumulated vertex-position gradient, or null
    const int32_t* slot;    // position of each query in the walk arrays (set by the launcher), or null
    int32_t gx_records;     // grad-X records reserved per query for binned accumulation (<= 0: atomics only)
    int32_t gfd_saved;      // (set by the launcher) GFD takes the base geodesic's end from f_out, b_out, v_out
    const int32_t* vc_off;  // [n_verts + 1] vertex -> corner list offsets (the vertex gradient's gather)
    const int32_t* vc;      // [3 n_faces] corners 3 f + k (internal face f, corner k) of each vertex
    // (set by the launcher) the vertex gradient's start terms: nine floats per query,
    // each query's rank among those of its start face, the faces' list offsets, the lists
    const float* sterm;
    const int32_t* srank;
    const uint32_t* fstart;
    int32_t* qlist;
};

// Host-side result of packing a mesh (float64 work, rounded once).
struct PackedMesh {
    std::vector<FaceRec> face;
    std::vector<int32_t> F;           // internal (bisection) face order
    std::vector<int64_t> order;       // internal face id -> user face id
    std::vector<int32_t> perm;        // user face id -> internal face id
    int64_t part_start[kParts + 1];   // internal face ranges of the XCD parts
    std::vector<float> X;
    std::vector<int64_t> half;
    std::vector<int32_t> twin;        // half-edge across each edge (internal ids), -1 on the boundary
    std::vector<uint8_t> vbnd;        // vertex lies on a boundary edge
    std::vector<float> geo;           // [n_faces, 16]: per-face positions, lengths, corners, user id (DevMesh::geo)
    std::vector<int64_t> face_off;    // [n_meshes + 1] user face offsets of the batched meshes
    int64_t n_verts = 0, n_faces = 0;
    double mean_edge = 0.0;
    int64_t n_edges = 0;              // undirected edges
    int64_t n_boundary = 0;           // boundary edges
    int32_t has_flip = 0;
};

// Validates and packs a mesh on the host; returns SG_OK or an SG_E_* code.
int pack_mesh(const float* X_host, int64_t n_verts, const int32_t* F_host, int64_t n_faces,
              const int64_t* vert_offsets, const int64_t* face_offsets, int32_t n_meshes, PackedMesh& out);
// The position-dependent parts of a packed mesh (face records' lengths and
// corners, half_theta, X, mean_edge) for its connectivity, links and face order.
int pack_geometry(const float* X_host, PackedMesh& pm);

// Exclusive prefix sums of x[0, n) in place; tile: scan_tiles(n) words of scratch.
inline int64_t scan_tiles(int64_t n) { return (n + 4095) / 4096; }
hipError_t launch_scan(uint32_t* x, int64_t n, uint32_t* tile, hipStream_t s);

// The same for new positions, on the device.  ws (pos_workspace bytes) holds
// two error words (set to ~0 by the caller: the first non-finite vertex, the
// first face without area), the blocks' sums of edge lengths, and the positions.
inline int pos_blocks(int64_t n_verts, int64_t n_faces) { return (int)((std::max(n_verts, n_faces) + 255) / 256); }
inline float* pos_staging(void* ws, int64_t n_verts, int64_t n_faces) {
    return reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + 16 + 8 * (size_t)pos_blocks(n_verts, n_faces));
}
size_t pos_workspace(int64_t n_verts, int64_t n_faces);
hipError_t launch_pos_check(const DevMesh& M, void* ws, hipStream_t s);
hipError_t launch_pos_commit(const DevMesh& M, void* ws, const int32_t* vc_off, const int32_t* vc, hipStream_t s);

// Plain forward: one ray per lane, run to completion (Alg. gpu_parallel).
hipError_t launch_exp_plain(const DevMesh& M, const ExpArgs& a, hipStream_t s);

// Schedule of a persistent walk launch.
constexpr int kMaxQueues = 64;
// A ray crosses boundary edges at about 0.7 of their number per face and crossing:
// from one per hundred faces on, a good part of rays of some 50 crossings and more
// end early, in no order of their lengths.  The rays of one direction class, and a
// query's walks, then no longer end together (the walk order, GFD's long walks).
inline bool mesh_open(int64_t n_boundary, int64_t n_faces) { return 100 * n_boundary >= n_faces; }

// Hole avoidance: the steps that a lane waits at most for others to need an odd step
// too (meeting a boundary, or now and then a vertex).  Where these are rare it would
// end long after the others: us with 8, 16, 24 and 48 steps, boundary edges per
// thousand faces, for 5,000 rays in the plain kernel and 1,000,000 in the persistent:
// 0.4 on 81,920 faces 85, 86, 92, 104 and 527, 513, 511, 526; 1.1 92, 96, 94, 99 and
// 543, 535, 541, 545; 3.7 124, 114, 118, 124 and 656, 613, 592, 577; 11 174, 149, 148,
// 157 and 814, 777, 762, 757; 37 296, 212, 190, 190 and 1,141, 910, 829, 760; without
// boundaries 100,000 rays on 20,480 faces 48, 48, 49, 57.  Along a long boundary (a
// sheet's) a ray slides step after step: 200,000 rays on a sheet of 1.48 million
// faces with 3,440 boundary edges take 11.7 ms with 16 steps and 6.3 with 48.
inline int park_wait(int64_t n_boundary, int64_t n_faces) {
    return 300 * n_boundary >= n_faces || n_boundary >= 1000 ? 48 : 16;
}

struct WalkSched {
    int blocks;       // 256-lane blocks launched
    int refill_min;   // idle lanes (of 64 per ray slot) that trigger a refill
    int queues;       // ray queues: a multiple of 8, at most kMaxQueues
    bool one_mesh;    // the handle holds one mesh (the walk order's direction classes)
    bool open_mesh;   // many rays end at a boundary (mesh_open)
    // the backward's walks: their own block counts and refill thresholds, or those above
    bool own_blocks, own_refill;
    int cus, gfd_per_cu;   // CUs, and the most blocks of GFD's long-walk pass each holds
};

// Persistent forward: init kernel, persistent work-queue walk, finish kernel.
// ws must hold exp_persistent_workspace(n, K) bytes of device memory.
size_t exp_persistent_workspace(int64_t n, int32_t K);
// Device scratch of the allocation-free forward (one copy per device, held
// until the process ends): its size, the devices it is looked up for, and the
// current device's address (looked up with hipGetSymbolAddress on the first
// request from each device).
constexpr size_t kNoAllocScratchBytes = (size_t)128 << 20;
constexpr int kNoAllocMaxDevices = 64;
hipError_t noalloc_scratch(void** out);
// ev0/ev1 (nullable) are recorded on s around the walk kernel.
hipError_t launch_exp_persistent(const DevMesh& M, const ExpArgs& a, void* ws, const WalkSched& w, hipStream_t s,
                                 hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
int walk_blocks_per_cu();
int bwd_blocks_per_cu();
int part_blocks_per_cu();

// ---- projection integration (appendix "Projection Integration Exp Map")
// T: float for the ABI's arrays, double for the backward's internal stacks.
template <class T>
struct PiArgsT {
    int64_t n;
    const int32_t* f;   // user face ids
    const T* b;
    const T* v;
    int32_t K;
    const T* W;         // [n, K, 3] or null (K = 0)
    int32_t* f_out;
    T* b_out;
    T* p_out;
    T* v_out;
    T* W_out;
    int32_t* status;
    int32_t* n_steps;
    double step;        // s
    int32_t max_steps;
    int32_t scan;       // 1: scan every face of the mesh (the printed form), 0: grid search
    const int32_t* order;   // grid search: the order to take the rays in, or null
};
using PiArgs = PiArgsT<float>;
// ws: pi_order_workspace(n) bytes for a spatial order of the rays, or null (as
// they come).  The order pays once the face records exceed one L2 (4 MB) and
// there are rays for a wave per SIMD (below, a step waits for its own loads):
// 131,072 rays on 20,480 faces take 1.14 ms ordered, 1.07 not, on 327,680 faces
// 1.51 and 1.96; 65,536 rays on 81,920 faces 0.81 and 0.85, on 1,310,720 1.11 and
// 1.14; 40,000 rays there 1.06 and 1.03.
inline bool pi_ordered(int64_t rows, int64_t n_faces) {
    return rows >= 65536 && n_faces * (int64_t)sizeof(PiFace) >= ((int64_t)4 << 20);
}
size_t pi_order_workspace(int64_t n);
hipError_t launch_pi_exp(const PiMesh& P, const DevMesh& M, const PiArgs& a, void* ws, hipStream_t s);
// The projection data of a handle, in five parts.  Extents: kPiParts partial
// results per mesh (lowest and highest coordinates, sum of edge lengths, largest
// absolute coordinate of a share of all vertices).  The face records (slim: whether
// one of them is).  The numbers of cell entries that a choice of grids takes, and of
// faces with very many (sum[0], sum[1]; counting lists the latter in large, 1 +
// n_large words).  Counts: at cells[c] the entries before cell c (cells[total]: all
// of them; tile: scan_tiles(total + 1) words).  Fill: the entries; cells[c] moves to the end of cell c, so that
// cells - 1 (a zero word) are the cells' starts.
constexpr int kPiParts = 16, kPiExtent = 8;
hipError_t launch_pi_extents(const DevMesh& M, const int64_t* face_off, int n_meshes, double* out, hipStream_t s);
hipError_t launch_pi_faces(const DevMesh& M, PiFace* face, uint32_t* slim, hipStream_t s);
hipError_t launch_pi_entries(const PiMesh& P, unsigned long long* sum, double pad, hipStream_t s);
hipError_t launch_pi_count(const PiMesh& P, uint32_t* cells, int64_t total, double pad, uint32_t* tile, uint32_t* large,
                           int64_t n_large, hipStream_t s);
hipError_t launch_pi_fill(const PiMesh& P, uint32_t* cells, int32_t* cell_face, double pad, const uint32_t* large,
                          int64_t n_large, hipStream_t s);
// EP (saved f', v') or GFD (seven PI walks per query, stacked in two launches).
size_t pi_bwd_workspace(int64_t n, int32_t mode);
hipError_t launch_pi_backward(const PiMesh& P, const DevMesh& M, const BwdArgs& a, const PiArgs& pa, void* ws,
                              hipStream_t s);
// The extrinsic proxy from saved outputs (shared by both Exp maps).
hipError_t launch_ep_saved(const DevMesh& M, const BwdArgs& a, hipStream_t s);

// Backward of the exponential map (extrinsic proxy or geodesic finite differences).
// have_*: which of the forward's saved outputs (f', b', v', status) the call is given.
size_t bwd_workspace(int64_t n, int32_t mode, bool has_flip, bool vjp, bool gradx, int64_t n_faces,
                     int32_t gx_records, int walk_blocks, int cus, bool hole, bool have_f, bool have_b, bool have_v,
                     bool have_status);
hipError_t launch_backward(const DevMesh& M, const BwdArgs& a, void* ws, const WalkSched& w, hipStream_t s);

// Partitioned forward: the walk runs on the XCD whose L2 holds the ray's
// current part of the mesh; rays crossing parts are handed over through queues.
size_t exp_partitioned_workspace(int64_t n, int32_t K, bool hashes);
hipError_t launch_exp_partitioned(const DevMesh& M, const ExpArgs& a, void* ws, int grid_blocks, int refill_min,
                                  hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);

}  // namespace sg
