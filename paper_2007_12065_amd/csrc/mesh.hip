// Organized-point-cloud mesh extraction (Sec. 4.2, Alg. 1 and Alg. 2) as an
// ordered compaction over segments of 256 quads in GID order, one frame per
// call (the bodies are in tiles.h):
//   k_mesh_count : one workgroup per segment -> validity masks, the segment's
//                  triangle count
//   k_mesh_sums  : one workgroup, frames of more than kMeshSegMax segments:
//                  the counts become the triangles before each segment
//   k_mesh_emit  : one workgroup per segment -> T_map, T and HE of the
//                  segment, placed by the counts of the segments before it
// Indices come from prefix sums in GID order, so T is exactly Alg. 1's
// append order and every output is bit-exact and deterministic.
#include "tiles.h"

#include <mutex>

namespace pl {

namespace {

// each XCD takes a contiguous run of segments: the point row that two
// neighbouring quad rows share is then fetched once into one L2, and so are
// the masks of neighbouring rows in the emit
__global__ __launch_bounds__(kTileBlock) void k_mesh_count(MeshArgs m) {
    mesh_count_seg(m, xcd_remap((int)blockIdx.x, (int)gridDim.x));
}

__global__ __launch_bounds__(kMeshSumBlock) void k_mesh_sums(MeshArgs m) {
    mesh_scan_segs(m.seg, m.sums, mesh_segments((size_t)m.Q));
}

template <bool Summed> __global__ __launch_bounds__(kTileBlock) void k_mesh_emit(MeshArgs m) {
    mesh_emit_seg<Summed>(m, xcd_remap((int)blockIdx.x, (int)gridDim.x));
}

// Scratch of the allocation-free entry point (pl_mesh_opc_static): the
// validity masks and per-segment counts that pl_mesh_opc keeps in the
// caller's workspace.  Every device the library runs on holds one copy until
// the process ends.  Host code never passes this name to a kernel (in host
// code it is a host-side stand-in, not a device address): it uses the
// address hipGetSymbolAddress returns for the device in question.
constexpr size_t kMeshScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) uint8_t scratch[kMeshScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_addr[kMaxDevices];    // device address of `scratch` per device, once looked up

}  // namespace

size_t mesh_static_scratch_bytes() { return kMeshScratchBytes; }

pl_status mesh_static_scratch(hipStream_t s, void **out) {
    int cur = 0;
    if (pl_status st = hip_check(hipGetDevice(&cur), "hipGetDevice")) return st;
    int dev = cur;
    if (s) {
        hipDevice_t d;
        if (pl_status st = hip_check(hipStreamGetDevice(s, &d), "hipStreamGetDevice")) return st;
        dev = (int)d;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        set_error("device %d: the static mesh scratch serves devices 0..%d", dev, kMaxDevices - 1);
        return PL_ERR_ARG;
    }
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        // look the array up with its device current: each device holds its
        // own copy at its own address
        if (dev != cur)
            if (pl_status st = hip_check(hipSetDevice(dev), "hipSetDevice")) return st;
        void *p = nullptr;
        const pl_status st = hip_check(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)),
                                       "hipGetSymbolAddress(scratch)");
        if (dev != cur) (void)hipSetDevice(cur);
        if (st) return st;
        g_scratch_addr[dev] = p;
    }
    *out = g_scratch_addr[dev];
    return PL_OK;
}

// A byte per quad and an int per 256 quads of each row: the chunks (24 bytes
// per 64 quads) and the segments' counts need less (mesh_args).
size_t mesh_workspace(int M, int N) {
    const size_t Q = (size_t)(M - 1) * (N - 1);
    const size_t rows = (size_t)(M - 1) * ((size_t)(N - 1 + kMeshSeg - 1) / kMeshSeg);
    return align_up(Q, 256) + align_up(sizeof(int) * rows, 256);
}

MeshArgs mesh_args(const float *pts, int M, int N, uint8_t *tri_valid, int32_t *tri_map,
                   int32_t *triangles, int32_t *halfedges, int32_t cap, int32_t *n_tri, void *ws) {
    const size_t Q = (size_t)(M - 1) * (N - 1);
    char *w = static_cast<char *>(ws);
    const size_t o_seg = align_up(sizeof(MeshChunk) * mesh_chunks(Q), 256);
    const size_t o_sums = o_seg + align_up(sizeof(uint16_t) * (size_t)mesh_segments(Q), 256);
    return MeshArgs{pts, reinterpret_cast<MeshChunk *>(w), reinterpret_cast<uint16_t *>(w + o_seg),
                    reinterpret_cast<int *>(w + o_sums), tri_valid, tri_map, triangles, halfedges, n_tri, cap, N, (int)Q, QuadDiv::by(N - 1)};
}

pl_status launch_mesh_count(const MeshArgs &m, hipStream_t s) {
    k_mesh_count<<<mesh_segments((size_t)m.Q), kTileBlock, 0, s>>>(m);
    return hip_check(hipGetLastError(), "k_mesh_count");
}

pl_status launch_mesh_sums(const MeshArgs &m, hipStream_t s) {
    k_mesh_sums<<<1, kMeshSumBlock, 0, s>>>(m);
    return hip_check(hipGetLastError(), "k_mesh_sums");
}

pl_status launch_mesh_emit(const MeshArgs &m, hipStream_t s) {
    const int blocks = mesh_segments((size_t)m.Q);
    if (blocks > kMeshSegMax) k_mesh_emit<true><<<blocks, kTileBlock, 0, s>>>(m);
    else k_mesh_emit<false><<<blocks, kTileBlock, 0, s>>>(m);
    return hip_check(hipGetLastError(), "k_mesh_emit");
}

pl_status launch_mesh(const float *pts, int M, int N, uint8_t *tri_valid, int32_t *tri_map,
                      int32_t *triangles, int32_t *halfedges, int32_t cap, int32_t *n_tri,
                      void *ws, hipStream_t s) {
    const MeshArgs m = mesh_args(pts, M, N, tri_valid, tri_map, triangles, halfedges, cap, n_tri, ws);
    if (pl_status st = launch_mesh_count(m, s)) return st;
    if (mesh_segments((size_t)m.Q) > kMeshSegMax)
        if (pl_status st = launch_mesh_sums(m, s)) return st;
    return launch_mesh_emit(m, s);
}

}  // namespace pl
