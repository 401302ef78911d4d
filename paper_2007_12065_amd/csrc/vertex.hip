// Vertex update from filtered normals: the second stage of the bilateral
// mesh denoising the paper cites with Eqs. (3)-(6) (Sun et al., 2007), which
// Polylidar3D skips (Sec. 5.2).  Each sweep moves every vertex by the mean,
// over the valid triangles of T_FC that contain it, of the correction that
// puts it on the plane through the triangle's centroid with the triangle's
// filtered normal:
//     x <- x + (1 / |F|) sum_f n_f (n_f . (c_f - x)).
//
// On the implicit right-cut mesh vertex (r, c) lies in at most six
// triangles: both triangles of quad (r, c) (as p1) and of quad (r-1, c-1)
// (as p3), the first triangle of quad (r, c-1) (as p2) and the second of
// quad (r-1, c) (as p4).  Their vertices are the point and six of its eight
// grid neighbours.  Sweeps are Jacobi: each reads the previous sweep's points.
//
// Up to kVuMaxSweeps sweeps run in one launch, temporally blocked in LDS: a
// tile's points with a halo of F points, and the normals of the quads between
// them.  Validity and the normals are fixed during the sweeps, so whether a
// triangle counts is settled once while staging (its normal is staged as zero
// if it does not), and a sweep has no branches and no NaN tests.  One launch
// per sweep (a thread per point, everything from L2) was bound by the launch
// and its memory latency: five sweeps of a 480 x 640 frame 28.2 us, now 19.2
// us, bound by the sweeps' LDS reads.  Two launches of 3 + 2 sweeps measured 22
// us, tiles of 8 x 32 or 32 x 32 points 26 us.
#include "tuning.h"
#include "vu.h"

namespace pl {

namespace {

constexpr int kVuBlock = 512;
constexpr int kVuTH = 16, kVuTW = 32;         // points per tile
constexpr int kVuMaxSweeps = 5;

struct P3 {
    float x, y, z;
};

__device__ __forceinline__ bool p_ok(P3 p) { return !any_nan(p.x, p.y, p.z); }

// s += the part of a triangle with corners (a, b, d) and normal n, if `in`
// (a triangle that does not count has n = 0, and its projection, which an
// infinite corner would make a NaN, is left out).
// The centroid through a multiply by the rounded 1/3 (within an ulp of the
// quotient; an IEEE division would cost ten instructions a component).
__device__ __forceinline__ void vu_add(P3 x, P3 a, P3 b, P3 d, P3 n, bool in, P3 &s) {
    constexpr float kThird = 1.0f / 3.0f;
    const float cx = fmaf(a.x + b.x + d.x, kThird, -x.x);
    const float cy = fmaf(a.y + b.y + d.y, kThird, -x.y);
    const float cz = fmaf(a.z + b.z + d.z, kThird, -x.z);
    const float p = fmaf(n.x, cx, fmaf(n.y, cy, n.z * cz));
    const float proj = in ? p : 0.f;
    s.x = fmaf(n.x, proj, s.x);
    s.y = fmaf(n.y, proj, s.y);
    s.z = fmaf(n.z, proj, s.z);
}

// LDS of a tile with its halo of F points.
__host__ __device__ constexpr size_t vu_lds_bytes(int F) {
    const size_t S = (size_t)(kVuTH + 2 * F) * (size_t)(kVuTW + 2 * F);
    return sizeof(P3) * S * 4 + S;            // two point buffers, two normals per quad, flags
}

template <typename NT>
__global__ __launch_bounds__(kVuBlock) void k_vertex_update(const float *__restrict__ in,
                                                            float *__restrict__ out, int M, int N,
                                                            const NT *__restrict__ normals, int F,
                                                            int tiles_x, int ntiles) {
    extern __shared__ float vu_lds[];
    const int tile = xcd_remap((int)blockIdx.x, ntiles);
    const int H = kVuTH + 2 * F, W = kVuTW + 2 * F, S = H * W;
    P3 *A = reinterpret_cast<P3 *>(vu_lds);
    P3 *B = A + S;
    P3 *n0 = B + S, *n1 = n0 + S;             // the quad whose p1 is point i
    uint8_t *ok = reinterpret_cast<uint8_t *>(n1 + S);
    const int ty0 = (tile / tiles_x) * kVuTH, tx0 = (tile % tiles_x) * kVuTW;
    const int oy = ty0 - F, ox = tx0 - F;
    const int Nq = N - 1;
    const DivBy byW(W);
    // points; missing and off-grid ones are staged as zeros with ok = 0
    for (int i = threadIdx.x; i < S; i += kVuBlock) {
        const int ly = byW.div(i), lx = i - ly * W;
        const int r = oy + ly, c = ox + lx;
        P3 p{0.f, 0.f, 0.f};
        bool v = false;
        if (r >= 0 && r < M && c >= 0 && c < N) {
            const float *q = in + 3 * ((size_t)r * N + c);
            const P3 g{q[0], q[1], q[2]};
            v = p_ok(g);
            if (v) p = g;
        }
        A[i] = p;
        B[i] = p;
        ok[i] = v;
    }
    __syncthreads();
    // normals of the quads inside the region, zero for a triangle that does
    // not count (a missing corner, a NaN normal)
    for (int i = threadIdx.x; i < S; i += kVuBlock) {
        const int ly = byW.div(i), lx = i - ly * W;
        P3 a{0.f, 0.f, 0.f}, b = a;
        bool ca = false, cb = false;
        if (ly + 1 < H && lx + 1 < W) {
            const bool v1 = ok[i] & 1, v2 = ok[i + 1] & 1, v3 = ok[i + W + 1] & 1, v4 = ok[i + W] & 1;
            if (v1 && v3 && (v2 || v4)) {     // the quad is on the grid
                const NT *q = normals + 6 * ((size_t)(oy + ly) * Nq + (ox + lx));
                const P3 a0{ld_f(q), ld_f(q + 1), ld_f(q + 2)};
                const P3 b0{ld_f(q + 3), ld_f(q + 4), ld_f(q + 5)};
                ca = v2 && p_ok(a0);
                cb = v4 && p_ok(b0);
                if (ca) a = a0;
                if (cb) b = b0;
            }
        }
        n0[i] = a;
        n1[i] = b;
        // bits 1, 2: whether the quad's triangles count (bit 0, the point's
        // validity, is read by other threads meanwhile and keeps its value)
        ok[i] = (uint8_t)((ok[i] & 1) | (ca ? 2 : 0) | (cb ? 4 : 0));
    }
    __syncthreads();
    for (int f = 1; f <= F; ++f) {
        // points still exact after f sweeps
        const int h = H - 2 * f, w = W - 2 * f;
        const DivBy byw(w);
        for (int k = threadIdx.x; k < h * w; k += kVuBlock) {
            const int ry = byw.div(k), ly = f + ry, lx = f + (k - ry * w);
            const int i = ly * W + lx;
            const int q11 = ok[i], q10 = ok[i - 1], q00 = ok[i - W - 1], q01 = ok[i - W];
            const int count = ((q11 >> 1) & 1) + ((q11 >> 2) & 1) + ((q10 >> 1) & 1) +
                              ((q00 >> 1) & 1) + ((q00 >> 2) & 1) + ((q01 >> 2) & 1);
            const P3 x = A[i];
            const P3 pr = A[i + 1], pl_ = A[i - 1], pd = A[i + W], pu = A[i - W];
            const P3 pdr = A[i + W + 1], pul = A[i - W - 1];
            P3 s{0.f, 0.f, 0.f};
            // triangle k = 0 of quad (u, v) is (p3, p2, p1), k = 1 is (p1, p4, p3)
            vu_add(x, pdr, pr, x, n0[i], q11 & 2, s);              // quad (r, c): x = p1
            vu_add(x, x, pd, pdr, n1[i], q11 & 4, s);
            vu_add(x, pd, x, pl_, n0[i - 1], q10 & 2, s);          // quad (r, c-1): x = p2
            vu_add(x, x, pu, pul, n0[i - W - 1], q00 & 2, s);      // quad (r-1, c-1): x = p3
            vu_add(x, pul, pl_, x, n1[i - W - 1], q00 & 4, s);
            vu_add(x, pu, x, pr, n1[i - W], q01 & 4, s);           // quad (r-1, c): x = p4
            if (count) {
                const float inv = __builtin_amdgcn_rcpf((float)count);   // count in 1..6
                B[i] = P3{fmaf(s.x, inv, x.x), fmaf(s.y, inv, x.y), fmaf(s.z, inv, x.z)};
            } else {
                B[i] = x;
            }
        }
        __syncthreads();
        P3 *t = A; A = B; B = t;
    }
    // one point per thread: the tile itself; a missing point keeps its bits
    for (int k = threadIdx.x; k < kVuTH * kVuTW; k += kVuBlock) {
        const int ty = k / kVuTW, tx = k % kVuTW;
        const int r = ty0 + ty, c = tx0 + tx;
        if (r >= M || c >= N) continue;
        const int i = (F + ty) * W + F + tx;
        const size_t o = 3 * ((size_t)r * N + c);
        P3 x = A[i];
        if (!(ok[i] & 1)) x = P3{in[o], in[o + 1], in[o + 2]};
        st_stream(&out[o], x.x);
        st_stream(&out[o + 1], x.y);
        st_stream(&out[o + 2], x.z);
    }
}

}  // namespace

size_t vertex_update_workspace(int M, int N, int iterations) {
    return iterations > 1 ? align_up(12 * (size_t)M * N, 256) : 0;
}

pl_status launch_vertex_update(const float *in, float *out, int M, int N, const void *normals,
                               pl_dtype ndt, int iterations, void *ws, hipStream_t s) {
    const size_t bytes = 12 * (size_t)M * N;
    if (iterations == 0)
        return hip_check(hipMemcpyAsync(out, in, bytes, hipMemcpyDeviceToDevice, s), "hipMemcpyAsync");
    const int tiles_x = (N + kVuTW - 1) / kVuTW;
    const int ntiles = tiles_x * ((M + kVuTH - 1) / kVuTH);
    // the fewest launches, their sweeps as even as they go
    const int launches = (iterations + kVuMaxSweeps - 1) / kVuMaxSweeps;
    const float *src = in;
    int left = iterations;
    for (int l = 0; l < launches; ++l) {
        const int F = (left + launches - l - 1) / (launches - l);
        left -= F;
        // the last launch lands in `out`; earlier ones alternate with the workspace
        float *dst = ((launches - 1 - l) % 2 == 0) ? out : static_cast<float *>(ws);
        const size_t lds = vu_lds_bytes(F);
        if (ndt == PL_F32) {
            if (pl_status st = allow_lds((const void *)k_vertex_update<float>, lds)) return st;
            k_vertex_update<float><<<ntiles, kVuBlock, lds, s>>>(
                src, dst, M, N, static_cast<const float *>(normals), F, tiles_x, ntiles);
        } else {
            if (pl_status st = allow_lds((const void *)k_vertex_update<__half>, lds)) return st;
            k_vertex_update<__half><<<ntiles, kVuBlock, lds, s>>>(
                src, dst, M, N, static_cast<const __half *>(normals), F, tiles_x, ntiles);
        }
        if (pl_status st = hip_check(hipGetLastError(), "k_vertex_update")) return st;
        src = dst;
    }
    return PL_OK;
}

}  // namespace pl
