// Bilateral triangle-normal filter on the organized mesh (Sec. 2.3 Eqs. 3-6;
// neighbourhood of Sec. 5.2) and the gather of the result onto T, one frame
// per call.  The tile body (LDS staging, fused sweeps, weight evaluation,
// underflow fallback, missing-data encoding) is bil_tile in tiles.h; this
// file launches it over the frame's tiles ceil(iterations / fuse) times with
// ping-pong buffers; the last launch gathers onto T.  Zero sweeps are a copy.
#include "tiles.h"
#include "tuning.h"

namespace pl {

namespace {

template <int R, typename NT>
__global__ __launch_bounds__(kTileBlock, bil_waves_per_simd(R, false)) void k_bilateral(
    const NT *__restrict__ nin, const float *__restrict__ cen, NT *__restrict__ nout, int Mq,
    int Nq, float ka, float kb, int F, int TQH, int TQW, int tiles_x, int ntiles,
    const int32_t *__restrict__ tri_map, NT *__restrict__ nT) {
    extern __shared__ float4 lds[];
    const int tile = xcd_remap(blockIdx.x, ntiles);
    bil_tile<R, NT, false, false, bil_frame_lanes<R>()>(nin, cen, nout, Mq, Nq, ka, kb, F, TQH, TQW,
                                                        (tile / tiles_x) * TQH,
                                                        (tile % tiles_x) * TQW, tri_map, nT, lds);
}

// Zero sweeps: the normals' bits into the output and gathered onto T.  Bound by
// its bytes; a thread takes 12 of them, a float32 triangle or a float16 quad.  As
// a pass of k_bilateral over no sweeps (strided streaming stores, the sums'
// registers and LDS) 720 x 1280 points took 25.5 us, here 12.2 (70 MB, 5.8 TB/s);
// 480 x 640 7.6 and 5.1.
template <typename NT>
__global__ __launch_bounds__(kTileBlock) void k_copy_normals(const NT *__restrict__ nin, int items,
                                                             NT *__restrict__ nout,
                                                             const int32_t *__restrict__ tri_map,
                                                             NT *__restrict__ nT) {
    constexpr int kTris = 4 / (int)sizeof(NT);           // triangles per item
    const int i = (int)(blockIdx.x * kTileBlock + threadIdx.x);
    if (i >= items) return;
    union {
        uint32_t w[3];
        uint16_t h[6];
    } v;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(nin) + 3 * (size_t)i;
    uint32_t *dst = reinterpret_cast<uint32_t *>(nout) + 3 * (size_t)i;
    int t[kTris];
#pragma unroll
    for (int k = 0; k < kTris; ++k) t[k] = tri_map ? tri_map[kTris * (size_t)i + k] : -1;
#pragma unroll
    for (int k = 0; k < 3; ++k) v.w[k] = src[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[k] = v.w[k];
#pragma unroll
    for (int k = 0; k < kTris; ++k) {
        if (t[k] < 0) continue;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if constexpr (kTris == 1) reinterpret_cast<uint32_t *>(nT)[3 * (size_t)t[k] + j] = v.w[j];
            else reinterpret_cast<uint16_t *>(nT)[3 * (size_t)t[k] + j] = v.h[3 * k + j];
        }
    }
}

template <typename NT>
pl_status copy_normals(const NT *nin, int M, int N, NT *nout, const int32_t *tri_map, NT *nT, hipStream_t s) {
    const int items = (M - 1) * (N - 1) * (int)sizeof(NT) / 2;       // quads have 6 normals' components
    k_copy_normals<<<(items + kTileBlock - 1) / kTileBlock, kTileBlock, 0, s>>>(nin, items, nout, tri_map, nT);
    return hip_check(hipGetLastError(), "k_copy_normals");
}

template <int R, typename NT>
pl_status run(const NT *nin, const float *cen, int M, int N, float sl, float sa, int iterations,
              NT *nout, const int32_t *tri_map, NT *nT, NT *tmp, hipStream_t s) {
    const TileCfg c = tile_cfg(frame_stage(false, M, N), R);
    const int Mq = M - 1, Nq = N - 1;
    const float log2e = 1.4426950408889634f;
    const float ka = log2e / (2.0f * sl * sl);
    const float kb = log2e / (2.0f * sa * sa);
    const int launches = (iterations + c.fuse - 1) / c.fuse;
    const NT *cur = nin;
    int left = iterations;
    for (int l = 0; l < launches; ++l) {
        const int F = left < c.fuse ? left : c.fuse;
        left -= F;
        const bool last = l == launches - 1;
        NT *dst = ((launches - 1 - l) % 2 == 0) ? nout : tmp;    // last launch lands in nout
        const TileCfg t = bil_frame_tile(R, c, F, Mq, Nq);
        const int tiles_x = (Nq + t.tw - 1) / t.tw;
        const int ntiles = tiles_x * ((Mq + t.th - 1) / t.th);
        const size_t lds = bil_lds_bytes(R, F, t.th, t.tw, bil_waves(R, false));
        if (pl_status st = allow_lds((const void *)k_bilateral<R, NT>, lds)) return st;
        k_bilateral<R, NT><<<ntiles, kTileBlock, lds, s>>>(cur, cen, dst, Mq, Nq, ka, kb, F,
                                                            t.th, t.tw, tiles_x, ntiles,
                                                            last ? tri_map : nullptr, nT);
        if (pl_status st = hip_check(hipGetLastError(), "k_bilateral")) return st;
        cur = dst;
    }
    return PL_OK;
}

template <typename NT>
pl_status dispatch(const NT *nin, const float *cen, int M, int N, int kernel, float sl, float sa,
                   int iterations, NT *nout, const int32_t *tri_map, NT *nT, NT *tmp,
                   hipStream_t s) {
    if (iterations == 0) return copy_normals(nin, M, N, nout, tri_map, nT, s);
    switch (kernel / 2) {
    case 1: return run<1, NT>(nin, cen, M, N, sl, sa, iterations, nout, tri_map, nT, tmp, s);
    case 2: return run<2, NT>(nin, cen, M, N, sl, sa, iterations, nout, tri_map, nT, tmp, s);
    case 3: return run<3, NT>(nin, cen, M, N, sl, sa, iterations, nout, tri_map, nT, tmp, s);
    default: return run<4, NT>(nin, cen, M, N, sl, sa, iterations, nout, tri_map, nT, tmp, s);
    }
}

}  // namespace

size_t bilateral_workspace(int M, int N, pl_dtype ndt, int iterations) {
    const size_t T = 2 * (size_t)(M - 1) * (N - 1);
    return iterations > 1 ? T * 3 * (ndt == PL_F32 ? 4 : 2) : 0;
}

pl_status launch_bilateral(const void *nin, const float *cen, pl_dtype ndt, int M, int N,
                           int kernel, float sigma_length, float sigma_angle, int iterations,
                           void *nout, const int32_t *tri_map, void *normals_T, void *ws,
                           hipStream_t s) {
    if (ndt == PL_F32)
        return dispatch<float>(static_cast<const float *>(nin), cen, M, N, kernel, sigma_length,
                               sigma_angle, iterations, static_cast<float *>(nout), tri_map,
                               static_cast<float *>(normals_T), static_cast<float *>(ws), s);
    return dispatch<__half>(static_cast<const __half *>(nin), cen, M, N, kernel, sigma_length,
                            sigma_angle, iterations, static_cast<__half *>(nout), tri_map,
                            static_cast<__half *>(normals_T), static_cast<__half *>(ws), s);
}

}  // namespace pl
