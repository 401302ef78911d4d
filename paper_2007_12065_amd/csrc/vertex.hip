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
// Up to kVuMaxSweeps sweeps run in one launch: a workgroup takes a region of 32
// x 32 points, of which the inner 32 - 2 F squared are still exact after F
// sweeps.  A thread owns two points of it, one above the other, for all
// sweeps: their ten triangles' normals, which of them count and the points
// themselves stay in its registers, and a sweep reads the eight neighbouring
// points from LDS and writes its two.  Every read of LDS saved counts: with
// normals and flags in LDS as well, a point read 13 vectors and 4 bytes a
// sweep, and five sweeps of a 480 x 640 frame took 19.2 us, now 12.0 us (28.2
// us as five launches of a thread per point).
//
// Which triangles count is a matter of the sweep: a point that turns NaN in one
// (beside an infinite coordinate, or when one overflows) is a missing one from
// the next on.  A triangle that counted at the launch's start and has lost a
// corner makes each component of its sum NaN, so a thread that sees a NaN in
// its result, and no other, sums again with the corners looked at.  For the
// rest that is one comparison and a branch a sweep: 0.06 us of the 0.6 us one
// takes on a frame too small to fill the CUs, nothing measurable from 480 x 640.
//
// Frames whose regions would be mostly halo, and small frames' single sweeps,
// take a launch of a thread per point for each sweep (k_vertex_sweep).
#include "vu.h"

namespace pl {

namespace {

constexpr int kVuDim = 32;                    // points of a region, each way
constexpr int kVuBlock = kVuDim * kVuDim / 2;
constexpr int kVuMaxSweeps = 8;
// Register budget (80 VGPRs), for three workgroups per CU: with the rare second
// sum in registers beside the first (95) 1200 x 1944 points took 26.6 us a sweep.
constexpr int kVuWavesPerSimd = 6;

struct P3 {
    float x, y, z;
};

__device__ __forceinline__ bool p_ok(P3 p) { return !any_nan(p.x, p.y, p.z); }

__device__ __forceinline__ P3 vu_sum(P3 a, P3 b, P3 d) {
    return P3{a.x + b.x + d.x, a.y + b.y + d.y, a.z + b.z + d.z};
}

// s += the part of a triangle with corner sum t and normal n for vertex x, if
// `in` (a triangle that does not count has n = 0, and its projection, which an
// infinite corner would make a NaN, is left out).
// The centroid through a multiply by the rounded 1/3 (within an ulp of the
// quotient; an IEEE division would cost ten instructions a component).
__device__ __forceinline__ void vu_add(P3 x, P3 t, P3 n, bool in, P3 &s) {
    constexpr float kThird = 1.0f / 3.0f;
    const float cx = fmaf(t.x, kThird, -x.x);
    const float cy = fmaf(t.y, kThird, -x.y);
    const float cz = fmaf(t.z, kThird, -x.z);
    const float p = fmaf(n.x, cx, fmaf(n.y, cy, n.z * cz));
    const float proj = in ? p : 0.f;
    s.x = fmaf(n.x, proj, s.x);
    s.y = fmaf(n.y, proj, s.y);
    s.z = fmaf(n.z, proj, s.z);
}

__device__ __forceinline__ P3 vu_move(P3 x, P3 s, int count) {
    if (count == 0) return x;
    const float inv = __builtin_amdgcn_rcpf((float)count);   // count in 1..6
    return P3{fmaf(s.x, inv, x.x), fmaf(s.y, inv, x.y), fmaf(s.z, inv, x.z)};
}

// The point at `at` after a sweep, by triangles whose corners are valid now: of
// its six (normals and whether they counted at the launch's start: quad (r, c)'s
// two, the one of (r, c-1), (r-1, c-1)'s two, the one of (r-1, c)).  Points
// missing from the start are zero in LDS, and their triangles never counted.
__device__ __forceinline__ P3 vu_recheck(const P3 *buf, int at, P3 n0, bool k0, P3 n1, bool k1, P3 n2, bool k2,
                                         P3 n3, bool k3, P3 n4, bool k4, P3 n5, bool k5) {
    // an address the compiler cannot see through: kept from the first sum, the
    // points would not leave registers for it
    asm volatile("" : "+v"(at));
    const P3 *A = buf + at;
    const P3 x = A[0], a0 = A[-kVuDim - 1], a1 = A[-kVuDim], b0 = A[-1], b2 = A[1], c1 = A[kVuDim], c2 = A[kVuDim + 1];
    P3 s{0.f, 0.f, 0.f};
    int count = 0;
    auto add = [&](P3 t, P3 n, bool k, P3 p, P3 q) {
        k = (int)k & (int)p_ok(x) & (int)p_ok(p) & (int)p_ok(q);      // no branches
        vu_add(x, t, k ? n : P3{0.f, 0.f, 0.f}, k, s);
        count += (int)k;
    };
    add(vu_sum(c2, b2, x), n0, k0, c2, b2);
    add(vu_sum(x, c1, c2), n1, k1, c1, c2);
    add(vu_sum(c1, x, b0), n2, k2, c1, b0);
    add(vu_sum(x, a1, a0), n3, k3, a1, a0);
    add(vu_sum(a0, b0, x), n4, k4, a0, b0);
    add(vu_sum(a1, x, b2), n5, k5, a1, b2);
    return vu_move(x, s, count);
}

template <typename NT>
__global__ __launch_bounds__(kVuBlock, kVuWavesPerSimd) void k_vertex_update(
    const float *__restrict__ in, float *__restrict__ out, int M, int N,
    const NT *__restrict__ normals, int F, int tiles_x, int ntiles) {
    // a row and a point of slack on either side: the region's outer points
    // read past it (what they come to is not used)
    constexpr int kPad = kVuDim + 1, kSize = kVuDim * kVuDim + 2 * kPad;
    __shared__ P3 buf[2][kSize];
    __shared__ uint8_t ok[kSize];
    const int tile = xcd_remap((int)blockIdx.x, ntiles);
    const int inner = kVuDim - 2 * F;
    const int tx = (int)threadIdx.x % kVuDim, ty = 2 * ((int)threadIdx.x / kVuDim);
    const int r = (tile / tiles_x) * inner - F + ty, c = (tile % tiles_x) * inner - F + tx;
    const int at = kPad + ty * kVuDim + tx;      // the upper point
    const int Nq = N - 1;
    // both triangles' normals of quad (u, v); off the grid: zero
    struct Quad {
        NT n[6];
        bool in;
    };
    auto quad = [&](int u, int v) {
        Quad q;
        q.in = (unsigned)u < (unsigned)(M - 1) && (unsigned)v < (unsigned)Nq;
        if (q.in) {
            const NT *p = normals + 6 * ((size_t)u * Nq + v);
#pragma unroll
            for (int i = 0; i < 6; ++i) q.n[i] = p[i];
        }
        return q;
    };
    auto point = [&](int row) {
        P3 p{qnan(), 0.f, 0.f};
        if ((unsigned)row < (unsigned)M && (unsigned)c < (unsigned)N) {
            const float *q = in + 3 * ((size_t)row * N + c);
            p = P3{q[0], q[1], q[2]};
        }
        return p;
    };
    P3 x0 = point(r), x1 = point(r + 1);
    const Quad q00 = quad(r - 1, c - 1), q01 = quad(r - 1, c), q10 = quad(r, c - 1), q11 = quad(r, c),
               q20 = quad(r + 1, c - 1), q21 = quad(r + 1, c);
    const bool v0 = p_ok(x0), v1 = p_ok(x1);
    if (!v0) x0 = P3{0.f, 0.f, 0.f};
    if (!v1) x1 = P3{0.f, 0.f, 0.f};
    buf[0][at] = x0;
    buf[0][at + kVuDim] = x1;
    ok[at] = v0;
    ok[at + kVuDim] = v1;
    if (threadIdx.x < kPad) ok[threadIdx.x] = ok[kSize - 1 - threadIdx.x] = 0;   // the slack: no triangle
    __syncthreads();
    // which triangles count: corners valid, normal without a NaN.  Rows a, b,
    // c, d are r - 1 .. r + 2; b and c hold this thread's points.
    const uint8_t *o = ok + at;
    const bool a0 = o[-kVuDim - 1], a1 = o[-kVuDim], b0 = o[-1], b2 = o[1], c0 = o[kVuDim - 1],
               c2 = o[kVuDim + 1], d1 = o[2 * kVuDim], d2 = o[2 * kVuDim + 1];
    auto normal = [](const Quad &q, int k, bool corners, bool &counts) {
        const P3 n{ld_f(&q.n[3 * k]), ld_f(&q.n[3 * k + 1]), ld_f(&q.n[3 * k + 2])};
        counts = q.in && corners && p_ok(n);
        return counts ? n : P3{0.f, 0.f, 0.f};
    };
    // triangle 0 of quad (u, v) is (p3, p2, p1), triangle 1 is (p1, p4, p3)
    bool k00, k01, k11, k20, k21, k30, k31, k40, k41, k50;
    const P3 n00 = normal(q00, 0, v0 && a1 && a0, k00), n01 = normal(q00, 1, a0 && b0 && v0, k01);
    const P3 n11 = normal(q01, 1, a1 && v0 && b2, k11);
    const P3 n20 = normal(q10, 0, v1 && v0 && b0, k20), n21 = normal(q10, 1, b0 && c0 && v1, k21);
    const P3 n30 = normal(q11, 0, c2 && b2 && v0, k30), n31 = normal(q11, 1, v0 && v1 && c2, k31);
    const P3 n40 = normal(q21, 0, d2 && c2 && v1, k40), n41 = normal(q21, 1, v1 && d1 && d2, k41);
    const P3 n50 = normal(q20, 0, d1 && v1 && c0, k50);
    const int count0 = (int)k30 + (int)k31 + (int)k20 + (int)k00 + (int)k01 + (int)k11;
    const int count1 = (int)k40 + (int)k41 + (int)k50 + (int)k20 + (int)k21 + (int)k31;
    for (int f = 1; f <= F; ++f) {
        const P3 *A = buf[(f - 1) & 1] + at;
        const P3 pa0 = A[-kVuDim - 1], pa1 = A[-kVuDim], pb0 = A[-1], pb2 = A[1], pc0 = A[kVuDim - 1],
                 pc2 = A[kVuDim + 1], pd1 = A[2 * kVuDim], pd2 = A[2 * kVuDim + 1];
        const P3 t20 = vu_sum(x1, x0, pb0), t31 = vu_sum(x0, x1, pc2);      // of both points
        P3 s0{0.f, 0.f, 0.f}, s1 = s0;
        vu_add(x0, vu_sum(pc2, pb2, x0), n30, k30, s0);        // quad (r, c): p1
        vu_add(x0, t31, n31, k31, s0);
        vu_add(x0, t20, n20, k20, s0);                         // quad (r, c-1): p2
        vu_add(x0, vu_sum(x0, pa1, pa0), n00, k00, s0);        // quad (r-1, c-1): p3
        vu_add(x0, vu_sum(pa0, pb0, x0), n01, k01, s0);
        vu_add(x0, vu_sum(pa1, x0, pb2), n11, k11, s0);        // quad (r-1, c): p4
        vu_add(x1, vu_sum(pd2, pc2, x1), n40, k40, s1);
        vu_add(x1, vu_sum(x1, pd1, pd2), n41, k41, s1);
        vu_add(x1, vu_sum(pd1, x1, pc0), n50, k50, s1);
        vu_add(x1, t20, n20, k20, s1);
        vu_add(x1, vu_sum(pb0, pc0, x1), n21, k21, s1);
        vu_add(x1, t31, n31, k31, s1);
        x0 = vu_move(x0, s0, count0);
        x1 = vu_move(x1, s1, count1);
        if (__builtin_expect(__ballot(__builtin_isunordered(x0.x, x1.x)) != 0, 0)) {
            x0 = vu_recheck(buf[(f - 1) & 1], at, n30, k30, n31, k31, n20, k20, n00, k00, n01, k01, n11, k11);
            x1 = vu_recheck(buf[(f - 1) & 1], at + kVuDim, n40, k40, n41, k41, n50, k50, n20, k20, n21, k21,
                            n31, k31);
        }
        if (f < F) {
            P3 *B = buf[f & 1] + at;
            B[0] = x0;
            B[kVuDim] = x1;
            __syncthreads();
        }
    }
    // the exact points of the region; a missing point keeps its bits
    auto store = [&](int y, int row, P3 x, bool valid) {
        if (y < F || y >= kVuDim - F || tx < F || tx >= kVuDim - F || row >= M || c >= N) return;
        const size_t g = 3 * ((size_t)row * N + c);
        if (!valid) x = P3{in[g], in[g + 1], in[g + 2]};
        st_stream(&out[g], x.x);
        st_stream(&out[g + 1], x.y);
        st_stream(&out[g + 2], x.z);
    };
    store(ty, r, x0, v0);
    store(ty + 1, r + 1, x1, v1);
}

// One sweep, a thread per point, row-major over the frame: where a launch of
// fused sweeps has nothing to win (vu_by_points).  The 3 x 3 points around one
// and its normals come from cache.  Same bits: the same sums in the same order.
constexpr int kVuPointBlock = 256;

template <typename NT>
__global__ __launch_bounds__(kVuPointBlock) void k_vertex_sweep(const float *__restrict__ in,
                                                                float *__restrict__ out, int M, int N,
                                                                const NT *__restrict__ normals) {
    const long long idx =
        (long long)xcd_remap((int)blockIdx.x, (int)gridDim.x) * kVuPointBlock + threadIdx.x;
    if (idx >= (long long)M * N) return;
    const int r = (int)(idx / N), c = (int)(idx - (long long)r * N), Nq = N - 1;
    auto point = [&](int row, int col) {
        P3 p{qnan(), 0.f, 0.f};
        if ((unsigned)row < (unsigned)M && (unsigned)col < (unsigned)N) {
            const float *q = in + 3 * ((size_t)row * N + col);
            p = P3{q[0], q[1], q[2]};
        }
        return p;
    };
    const P3 x = point(r, c), a0 = point(r - 1, c - 1), a1 = point(r - 1, c), b0 = point(r, c - 1),
             b2 = point(r, c + 1), c1 = point(r + 1, c), c2 = point(r + 1, c + 1);
    P3 s{0.f, 0.f, 0.f};
    int count = 0;
    // triangle k of quad (u, v), p and q its corners beside x (all three on the
    // grid, so the quad is)
    auto add = [&](int u, int v, int k, P3 t, P3 p, P3 q) {
        if (!(p_ok(x) && p_ok(p) && p_ok(q))) return;
        const NT *m = normals + 3 * (2 * ((size_t)u * Nq + v) + k);
        const P3 n{ld_f(m), ld_f(m + 1), ld_f(m + 2)};
        if (!p_ok(n)) return;
        vu_add(x, t, n, true, s);
        ++count;
    };
    add(r, c, 0, vu_sum(c2, b2, x), c2, b2);               // quad (r, c): p1
    add(r, c, 1, vu_sum(x, c1, c2), c1, c2);
    add(r, c - 1, 0, vu_sum(c1, x, b0), c1, b0);           // quad (r, c-1): p2
    add(r - 1, c - 1, 0, vu_sum(x, a1, a0), a1, a0);       // quad (r-1, c-1): p3
    add(r - 1, c - 1, 1, vu_sum(a0, b0, x), a0, b0);
    add(r - 1, c, 1, vu_sum(a1, x, b2), a1, b2);           // quad (r-1, c): p4
    const P3 y = vu_move(x, s, count);
    float *o = out + 3 * idx;
    st_stream(&o[0], y.x);
    st_stream(&o[1], y.y);
    st_stream(&o[2], y.z);
}

}  // namespace

namespace {

// Launches for `iterations` sweeps over P points, their sweeps as even as they
// go: few of many sweeps recompute halos, many of few pay the launch and the
// points' and normals' way through memory.  In units of one point's sweep, a
// launch costs about 3.3 M + 2.5 P and F sweeps of it F P (32 / (32 - 2F))^2
// (measured: five sweeps in one launch and as 3 + 2: 480 x 640 11.9 and 15.2
// us, 1200 x 1944 64.5 and 66.0; six and 3 + 3: 480 x 640 13.3 and 15.9, 720 x
// 1280 34.2 and 33.9, 1200 x 1944 83.7 and 75.8).
int vu_launches(int iterations, double P) {
    auto sweeps = [P](int F) {
        const double inner = kVuDim - 2 * F;
        return F * P * (kVuDim * kVuDim / (inner * inner));
    };
    int best = iterations;
    double least = 1e300;
    for (int L = (iterations + kVuMaxSweeps - 1) / kVuMaxSweeps; L <= iterations; ++L) {
        const int F = iterations / L, more = iterations % L;      // `more` launches take F + 1
        const double cost = L * (3.3e6 + 2.5 * P) + (L - more) * sweeps(F) + (more ? more * sweeps(F + 1) : 0.0);
        if (cost >= least) break;
        least = cost;
        best = L;
    }
    return best;
}

// Whether a launch per sweep, a thread per point, is the faster way: a single
// sweep of a small frame, and frames so narrow that the regions' halo is most
// of the work.  In microseconds, a launch of F fused sweeps over t regions takes
// about 4.5 + 0.55 F + t (2.7 + 1.45 F) / 1000 where its points come from
// cache, and a sweep over P points 3.3 + 6.2 P / 10^6.  By points against
// regions: one sweep of 40 x 50 4.6, 5.2; 120 x 160 4.8, 5.4; 480 x 640 6.0, 6.6
// (720 x 1280: 12.8, 11.5); 70000 x 3 5.3, 15.2, and twenty 86, 162; 20000 x 16
// one 5.8, 7.3, and six as fused 18.2 (by points about 30).
bool vu_by_points(int M, int N, int iterations, int launches) {
    double fused = 0.0;
    for (int l = 0, left = iterations; l < launches; ++l) {
        const int F = (left + launches - l - 1) / (launches - l), inner = kVuDim - 2 * F;
        left -= F;
        fused += 4.5 + 0.55 * F +
                 (double)((M + inner - 1) / inner) * ((N + inner - 1) / inner) * (2.7 + 1.45 * F) * 1e-3;
    }
    return 1.0 + iterations * (3.3 + 6.2e-6 * M * N) < fused;
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
    int launches = vu_launches(iterations, (double)M * N);
    const bool by_points = vu_by_points(M, N, iterations, launches);
    if (by_points) launches = iterations;
    const float *src = in;
    int left = iterations;
    auto launch = [&](float *dst, int F, const auto *n) {
        if (by_points) {
            const unsigned grid = (unsigned)(((size_t)M * N + kVuPointBlock - 1) / kVuPointBlock);
            k_vertex_sweep<<<grid, kVuPointBlock, 0, s>>>(src, dst, M, N, n);
            return;
        }
        const int inner = kVuDim - 2 * F;
        const int tiles_x = (N + inner - 1) / inner;
        const int ntiles = tiles_x * ((M + inner - 1) / inner);
        k_vertex_update<<<ntiles, kVuBlock, 0, s>>>(src, dst, M, N, n, F, tiles_x, ntiles);
    };
    for (int l = 0; l < launches; ++l) {
        const int F = (left + launches - l - 1) / (launches - l);
        left -= F;
        // the last launch lands in `out`; earlier ones alternate with the workspace
        float *dst = ((launches - 1 - l) % 2 == 0) ? out : static_cast<float *>(ws);
        if (ndt == PL_F32)
            launch(dst, F, static_cast<const float *>(normals));
        else
            launch(dst, F, static_cast<const __half *>(normals));
        if (pl_status st = hip_check(hipGetLastError(), "k_vertex_update")) return st;
        src = dst;
    }
    return PL_OK;
}

}  // namespace pl
