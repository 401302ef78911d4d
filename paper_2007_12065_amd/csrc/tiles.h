// Per-tile device bodies shared by the single-frame kernels and the batched
// kernels, so that a frame gets bit-for-bit the same result
// whichever way it is launched.  Tile shapes and the number of fused sweeps
// are runtime values (LDS is dynamic), which lets the tuner pick them.
#pragma once

#include "common.h"

#include <float.h>
#include <type_traits>

namespace pl {

constexpr int kTileBlock = 256;        // threads per workgroup for every tile body

// ---------------------------------------------------------------------------
// Mesh (Sec. 4.2, Alg. 1 and Alg. 2), over the quads in GID order.
//
// Quads are numbered q = u Nq + v, whatever the frame's width, and dealt in
// chunks of 64, one per wave, four chunks (a segment) per workgroup.  A chunk's
// validity is two 64-bit masks (bit l: the first, the second triangle of quad
// 64 k + l is valid), so a triangle's place in T is the count of the segments
// before it, the chunk's place in its segment and a population count; the
// quads above, below and beside a chunk's are the masks 64 k -+ Nq and 64 k
// -+ 1 read across chunk borders.  A wave's emit is then scalar mask
// arithmetic and five stores, whose lanes write one contiguous run each: no
// LDS staging, no scan over the workgroup.  What bounds it is the outputs'
// bytes.  (With a byte of code per quad, shuffled scans and outputs staged in
// LDS, counting and emitting took 100 and 200 VALU instructions per 64 quads,
// now 60 and 110, and a 1200 x 1944 frame 11.7 + 39.2 us, now 13.1 + 26.6 us.)
// ---------------------------------------------------------------------------

constexpr int kMeshSeg = kTileBlock;           // quads per segment
constexpr int kMeshPerSeg = kMeshSeg / kWave;  // chunks per segment
// Segments per frame up to which an emit workgroup sums the counts before its
// segment itself; past it a launch of one workgroup does for all of them.  The
// workgroups' own sums grow with the square (9,101 segments take 26.6 us to
// emit, 22.8 us with the sums at hand), the launch takes 6 to 9 us.  A mesh by
// own sums against by a launch: 9,100 segments 38.3 and 40.9 us, 11,986 47.4
// and 49.5, 15,184 57.8 and 59.7, 16,304 61.8 and 62.2, 18,383 71.2 and 72.5
// (equal within its runs' spread); a batch is the same either way.
constexpr int kMeshSegMax = 16384;

struct MeshChunk {
    unsigned long long f, s;      // masks of the first and the second triangles
    int pre;                      // valid triangles of the segment before the chunk
    int unused;
};

__host__ __device__ constexpr int mesh_segments(size_t Q) { return (int)((Q + kMeshSeg - 1) / kMeshSeg); }
__host__ __device__ constexpr size_t mesh_chunks(size_t Q) { return (Q + kWave - 1) / kWave; }

// A frame's mesh buffers and outputs.
struct MeshArgs {
    const float *pts;
    MeshChunk *chunks;
    uint16_t *seg;                // [segments] valid triangles of each (at most 512)
    int *sums;                    // [segments + 1] triangles before each, and |T| (frames past kMeshSegMax)
    uint8_t *tri_valid;
    int32_t *tri_map, *tris, *he, *n_tri;
    int cap, N, Q;                // Q quads, N points per row
    QuadDiv by_row;               // by Nq = N - 1
};

// The arguments of a frame whose mesh buffers lie in `ws` (mesh_workspace).
MeshArgs mesh_args(const float *pts, int M, int N, uint8_t *tri_valid, int32_t *tri_map,
                   int32_t *triangles, int32_t *halfedges, int32_t cap, int32_t *n_tri, void *ws);
// pl_mesh_opc's launches (the sums for frames of more than kMeshSegMax segments).
pl_status launch_mesh_count(const MeshArgs &m, hipStream_t s);
pl_status launch_mesh_sums(const MeshArgs &m, hipStream_t s);
pl_status launch_mesh_emit(const MeshArgs &m, hipStream_t s);

// Masks and count of segment `sg`.
__device__ __forceinline__ void mesh_count_seg(const MeshArgs &m, int sg) {
    __shared__ int part[kMeshPerSeg];
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int k = sg * kMeshPerSeg + wave;
    const int Nq = m.by_row.d, q0 = k * kWave, q = q0 + lane;
    unsigned long long mf = 0, ms = 0;
    if (q0 < m.Q) {
        const int u0 = m.by_row.div(q0);
        // the lane's row: one step past the wave's first if rows are long
        const int t = q0 - u0 * Nq + lane;
        const int du = Nq >= kWave ? (t >= Nq ? 1 : 0) : m.by_row.div(t);
        const int v = t - du * Nq;
        const bool in = q < m.Q;
        const float *p1 = m.pts + 3 * (size_t)(in ? q + u0 + du : 0);
        const float *p4 = p1 + 3 * (size_t)m.N;
        const float ax = p1[0], ay = p1[1], az = p1[2], bx = p4[0], by = p4[1], bz = p4[2];
        // the right corners are the next lane's left ones, but for the wave's
        // last lane and a row's last quad
        bool right1 = false, right4 = false;
        const bool edge = in && (lane == kWave - 1 || v == Nq - 1);
        if (edge) {
            right1 = !any_nan(p1[3], p1[4], p1[5]);
            right4 = !any_nan(p4[3], p4[4], p4[5]);
        }
        const unsigned long long o1 = __ballot(in && !any_nan(ax, ay, az));
        const unsigned long long o4 = __ballot(in && !any_nan(bx, by, bz));
        const unsigned long long e = __ballot(edge), e1 = __ballot(right1), e4 = __ballot(right4);
        const unsigned long long o2 = ((o1 >> 1) & ~e) | e1, o3 = ((o4 >> 1) & ~e) | e4;
        mf = o1 & o2 & o3;              // first triangle (p3, p2, p1)
        ms = o1 & o3 & o4;              // second triangle (p1, p4, p3)
        if (m.tri_valid && in) {
            const unsigned f = lane_bit(mf), s = lane_bit(ms);
            *reinterpret_cast<uint16_t *>(m.tri_valid + 2 * (size_t)q) = (uint16_t)(f | (s << 8));
        }
    }
    if (lane == 0) part[wave] = __popcll(mf) + __popcll(ms);
    __syncthreads();
    int pre = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kMeshPerSeg; ++w) {
        const int c = part[w];
        pre += w < wave ? c : 0;
        all += c;
    }
    if (lane == 0 && q0 < m.Q) m.chunks[k] = MeshChunk{mf, ms, pre, 0};
    if (threadIdx.x == 0) m.seg[sg] = (uint16_t)all;
    __syncthreads();                    // `part` is reused by the next segment
}

// The triangles before each segment, and |T| behind them, from the segments'
// counts, by one workgroup of kMeshSumBlock threads.
constexpr int kMeshSumBlock = 1024;

__device__ __forceinline__ void mesh_scan_segs(const uint16_t *seg, int *sums, int n) {
    __shared__ int wsum[kMeshSumBlock / kWave];
    constexpr int kPer = 16;            // consecutive counts per thread and pass: 32 bytes
    const int lane = (int)threadIdx.x & (kWave - 1), wave = (int)threadIdx.x / kWave;
    int carry = 0;
    for (int base = 0; base < n; base += kPer * kMeshSumBlock) {
        const int i0 = base + kPer * (int)threadIdx.x;
        union {
            uint4 v[2];
            uint16_t c[kPer];
        } in = {{make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0)}};
        if (i0 + kPer <= n) {
            in.v[0] = reinterpret_cast<const uint4 *>(seg + i0)[0];
            in.v[1] = reinterpret_cast<const uint4 *>(seg + i0)[1];
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j) in.c[j] = i0 + j < n ? seg[i0 + j] : (uint16_t)0;
        }
        int sum = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) sum += in.c[j];
        const int incl = wave_inclusive_scan(sum);
        if (lane == kWave - 1) wsum[wave] = incl;
        __syncthreads();
        int run = carry + incl - sum;
#pragma unroll
        for (int w = 0; w < kMeshSumBlock / kWave; ++w) {
            const int t = wsum[w];
            run += w < wave ? t : 0;
            carry += t;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (i0 + j < n) sums[i0 + j] = run;
            run += in.c[j];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[n] = carry;
}

// The masks of the 64 quads from q on (q may lie outside the frame: quads
// there have none), and the valid triangles of q's segment before q.
struct MeshWindow {
    unsigned long long f, s;
    int before;
};

// Chunk k by scalar loads (constant while the reading kernel runs); none of
// its bits outside the frame.  The load is unconditional, so that several are
// in flight together.
__device__ __forceinline__ MeshChunk mesh_chunk(const MeshChunk *chunks, int K, int k) {
    typedef const __attribute__((address_space(4))) MeshChunk *Const;
    const Const p = (Const)chunks + min(max(k, 0), K - 1);
    const bool in = k >= 0 && k < K;
    const unsigned long long f = p->f, s = p->s;
    const int pre = p->pre;
    return MeshChunk{in ? f : 0ull, in ? s : 0ull, in ? pre : 0, 0};
}

// The window at q from its chunk c and the one after it.
__device__ __forceinline__ MeshWindow mesh_window(const MeshChunk &c, const MeshChunk &next, int q) {
    const int sh = q & (kWave - 1);
    const unsigned long long low = (1ull << sh) - 1;
    MeshWindow w{c.f >> sh, c.s >> sh, c.pre + (int)__popcll(c.f & low) + (int)__popcll(c.s & low)};
    if (sh) {
        w.f |= next.f << (kWave - sh);
        w.s |= next.s << (kWave - sh);
    }
    return w;
}

__device__ __forceinline__ int mesh_rank(const MeshWindow &w) { return bits_below(w.f) + bits_below(w.s); }

// This thread's share of the counts of segments 0 .. n - 1 (16-byte loads of
// eight, the rest one by one).
__device__ __forceinline__ int mesh_sum_segs(const uint16_t *__restrict__ seg, int n, int t, int threads) {
    int a = 0;
    for (int i = t; i < n / 8; i += threads) {
        const uint4 c = reinterpret_cast<const uint4 *>(seg)[i];
        a = __builtin_amdgcn_sad_u16(c.x, 0u, a);
        a = __builtin_amdgcn_sad_u16(c.y, 0u, a);
        a = __builtin_amdgcn_sad_u16(c.z, 0u, a);
        a = __builtin_amdgcn_sad_u16(c.w, 0u, a);
    }
    if (t < n % 8) a += seg[n - n % 8 + t];
    return a;
}

// T_map, T and HE of segment `sg`.  Summed: `sums` holds the triangles before
// each segment.  The last segment writes |T|.
template <bool Summed>
__device__ __forceinline__ void mesh_emit_seg(const MeshArgs &m, int sg) {
    __shared__ int part[kTileBlock / kWave];
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int Nq = m.by_row.d, K = (int)mesh_chunks((size_t)m.Q), S = mesh_segments((size_t)m.Q);
    const int q0 = (sg * kMeshPerSeg + wave) * kWave;
    // segments of the quads above and below this chunk's first
    const int qt = q0 - Nq, qb = q0 + Nq;
    const int st = max(qt, 0) / kMeshSeg, sb = qb < m.Q ? qb / kMeshSeg : sg;   // no row below: none to sum
    const int k0 = q0 / kWave, kt = qt >> 6, kb = qb >> 6;
    const MeshChunk c = mesh_chunk(m.chunks, K, k0), cl = mesh_chunk(m.chunks, K, k0 - 1),
                    cr = mesh_chunk(m.chunks, K, k0 + 1), ct = mesh_chunk(m.chunks, K, kt),
                    ct1 = mesh_chunk(m.chunks, K, kt + 1), cb = mesh_chunk(m.chunks, K, kb),
                    cb1 = mesh_chunk(m.chunks, K, kb + 1);
    int bt, b0, bb;                     // triangles before the segments st, sg and sb
    if constexpr (Summed) {
        bt = m.sums[st];
        b0 = m.sums[sg];
        bb = m.sums[sb];
        if (sg == S - 1 && threadIdx.x == 0) *m.n_tri = m.sums[S];
    } else {
        // the workgroup sums the segments before its first one above, each
        // wave the few between
        const int lo = max(sg * kMeshSeg - Nq, 0) / kMeshSeg;
        const int a = wave_sum(mesh_sum_segs(m.seg, lo, (int)threadIdx.x, kTileBlock));
        if (lane == 0) part[wave] = a;
        __syncthreads();
        int sum = 0;
#pragma unroll
        for (int w = 0; w < kTileBlock / kWave; ++w) sum += part[w];
        bt = b0 = bb = sum;
        for (int i = lo; i < sb; i += kWave) {
            const int c = i + lane < sb ? m.seg[i + lane] : 0;
            const int incl = wave_inclusive_scan(c);
            auto upto = [&](int x) {    // counts of i .. x - 1 within this pass
                const int d = min(x - i, kWave);
                return d > 0 ? __builtin_amdgcn_readlane(incl, d - 1) : 0;
            };
            bt += upto(st);
            b0 += upto(sg);
            bb += upto(sb);
        }
        if (sg == S - 1 && threadIdx.x == 0) *m.n_tri = b0 + m.seg[sg];
        __syncthreads();                // `part` is reused by the next segment
    }
    if (q0 >= m.Q) return;
    const MeshWindow top = mesh_window(ct, ct1, qt), bot = mesh_window(cb, cb1, qb);
    const unsigned long long left_f = (c.f << 1) | (cl.f >> 63), left_s = (c.s << 1) | (cl.s >> 63);
    const unsigned long long right_f = (c.f >> 1) | (cr.f << 63), right_s = (c.s >> 1) | (cr.s << 63);
    const int q = q0 + lane;
    if (q >= m.Q) return;
    const int u0 = m.by_row.div(q0);
    const int t = q0 - u0 * Nq + lane;
    const int du = Nq >= kWave ? (t >= Nq ? 1 : 0) : m.by_row.div(t);
    const int v = t - du * Nq;
    const int f = lane_bit(c.f), g = lane_bit(c.s);
    const int r0 = b0 + c.pre + mesh_rank(MeshWindow{c.f, c.s, 0});   // this quad's first triangle
    {
        // T_map: two entries per quad, -1 for an invalid triangle
        typedef int i2v __attribute__((ext_vector_type(2)));
        i2v w;
        w.x = f ? r0 : -1;
        w.y = g ? r0 + f : -1;
        __builtin_nontemporal_store(w, reinterpret_cast<i2v *>(m.tri_map + 2 * (size_t)q));
    }
    const bool wf = f && r0 < m.cap, wg = g && r0 + f < m.cap;
    // T: first triangle (p3, p2, p1), second (p1, p4, p3)
    const int i1 = q + u0 + du, i4 = i1 + m.N;
    // plain stores: a lane writes 12 of its 24 bytes at a time, which the L2
    // puts together (with streaming ones a 1200 x 1944 frame's emit took 48.9
    // us, where these take 22.2 us)
    int32_t *T0 = m.tris + 3 * (size_t)r0, *T1 = m.tris + 3 * (size_t)(r0 + f);
    if (wf) { T0[0] = i4 + 1; T0[1] = i1 + 1; T0[2] = i1; }
    if (wg) { T1[0] = i1; T1[1] = i4; T1[2] = i4 + 1; }
    // HE: Right = (u, v+1, 1), Top = (u-1, v, 1), Left = (u, v-1, 0),
    // Bottom = (u+1, v, 0)
    if (m.he) {
        const int rt = bt + top.before + mesh_rank(top), rb = bb + bot.before + mesh_rank(bot);
        const int lf = lane_bit(left_f), ls = lane_bit(left_s);
        const int rf = lane_bit(right_f), rs = lane_bit(right_s);
        const int right_t = rs && v + 1 < Nq ? 3 * (r0 + f + g + rf) : -1;
        const int left_t = lf && v > 0 ? 3 * (r0 - lf - ls) : -1;
        const int top_t = lane_bit(top.s) ? 3 * (rt + (int)lane_bit(top.f)) + 1 : -1;
        const int bot_t = lane_bit(bot.f) ? 3 * rb + 1 : -1;
        int32_t *H0 = m.he + 3 * (size_t)r0, *H1 = m.he + 3 * (size_t)(r0 + f);
        if (wf) { H0[0] = right_t; H0[1] = top_t; H0[2] = g ? 3 * (r0 + f) + 2 : -1; }
        if (wg) { H1[0] = left_t; H1[1] = bot_t; H1[2] = f ? 3 * r0 + 2 : -1; }
    }
}

// ---------------------------------------------------------------------------
// Laplacian (Sec. 2.3 Eqs. 1-2 on the image neighbourhood of Sec. 5.1):
// F Jacobi sweeps of one TH x TW tile, temporally blocked in LDS.
//
// The tile plus a halo of R*F pixels is staged as float4 (x, y, z, pad);
// sweep f updates the region that is still exact after f steps (shrinking by
// R per side) between two LDS buffers, and the centre is written back.
// Invalid pixels (any NaN coordinate) and pixels outside the image are staged
// as (0, 0, 0, +inf): the pad makes the squared distance +inf, whose
// reciprocal square root is exactly 0, so they drop out of both sums without
// a branch.  Pixels of the border band are staged with pad -0.0, which adds
// nothing to a distance: they are neighbours like any other, but only a +0.0
// pad (bits all zero) marks a pixel that is updated.  Invalid pixels and the
// border band are never updated; invalid pixels are written back from the
// input bits.  F = 0 copies the tile.
// LDS: 2 * (TH + 2RF) * (TW + 2RF) float4.
// ---------------------------------------------------------------------------

__host__ __device__ constexpr size_t lap_lds_bytes(int R, int F, int TH, int TW) {
    return 2 * sizeof(float4) * (size_t)(TH + 2 * R * F) * (size_t)(TW + 2 * R * F);
}

template <int R>
__device__ __forceinline__ void lap_tile(const float *__restrict__ src, float *__restrict__ dst,
                                         int M, int N, float lam, int F, int TH, int TW,
                                         int ty0, int tx0, float4 *lds) {
    const int halo = R * F;
    const int H = TH + 2 * halo, W = TW + 2 * halo;
    float4 *A = lds;
    float4 *B = lds + H * W;
    const int oy = ty0 - halo, ox = tx0 - halo;
    const float inf = __builtin_inff();

    // three points per thread and pass, their loads issued before the first is
    // used: a 16 x 16 tile with its halo of four waits for memory once
    constexpr int kU = 3;
    const DivBy byW(W);
    for (int base = threadIdx.x; base < H * W; base += kU * kTileBlock) {
        float4 p[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int idx = base + u * kTileBlock;
            const int ly = byW.div(idx), lx = idx - ly * W;
            const int gy = oy + ly, gx = ox + lx;
            p[u] = make_float4(qnan(), 0.f, 0.f, inf);
            if (idx < H * W && (unsigned)gy < (unsigned)M && (unsigned)gx < (unsigned)N) {
                const float *q = src + 3 * ((size_t)gy * N + gx);
                const bool inner = gy >= R && gy < M - R && gx >= R && gx < N - R;
                p[u] = make_float4(q[0], q[1], q[2], inner ? 0.f : -0.f);
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int idx = base + u * kTileBlock;
            if (idx >= H * W) break;
            if (any_nan(p[u].x, p[u].y, p[u].z)) p[u] = make_float4(0.f, 0.f, 0.f, inf);
            A[idx] = p[u];
        }
    }
    __syncthreads();

    for (int f = 1; f <= F; ++f) {
        const int lo = R * f;
        const int Hf = H - 2 * lo, Wf = W - 2 * lo;
        const DivBy byWf(Wf);
        for (int idx = threadIdx.x; idx < Hf * Wf; idx += kTileBlock) {
            const int ry = byWf.div(idx);
            const int ly = lo + ry, lx = lo + (idx - ry * Wf);
            const float4 c = A[ly * W + lx];
            float4 o = c;
            const bool active = __float_as_uint(c.w) == 0u;   // valid, not in the border band
            if (active) {
                float ws = 0.f, sx = 0.f, sy = 0.f, sz = 0.f;
                // The weighted sums; with `skip` set, coincident neighbours
                // (d2 = 0, weight 1/0) are left out.  Without the test such a neighbour makes ws
                // infinite -- nothing else can, every other weight being at
                // most 1/sqrt(the smallest float) -- so the point is summed
                // again with it (rare: duplicated points), and every result
                // is the same as with the test throughout.
                auto sums = [&](auto skip) {
                    ws = 0.f; sx = 0.f; sy = 0.f; sz = 0.f;
                    // 3x3: fully unrolled; larger windows: one row of the
                    // window per iteration, so only that row's neighbours are live
                    constexpr int kRowUnroll = R == 1 ? 3 : 1;
#pragma unroll kRowUnroll
                    for (int dy = -R; dy <= R; ++dy) {
#pragma unroll
                        for (int dx = -R; dx <= R; ++dx) {
                            if (dy == 0 && dx == 0) continue;
                            const float4 p = A[(ly + dy) * W + lx + dx];
                            const float ex = p.x - c.x, ey = p.y - c.y, ez = p.z - c.z;
                            const float d2 = fmaf(ex, ex, fmaf(ey, ey, fmaf(ez, ez, p.w)));
                            float w = __builtin_amdgcn_rsqf(d2);     // 1/||v_j - v_i||
                            if constexpr (decltype(skip)::value) w = d2 > 0.f ? w : 0.f;
                            ws += w;
                            sx = fmaf(w, ex, sx);
                            sy = fmaf(w, ey, sy);
                            sz = fmaf(w, ez, sz);
                        }
                    }
                };
                sums(std::false_type{});
                if (!(ws < inf)) sums(std::true_type{});
                if (ws > 0.f) {
                    const float k = lam * __builtin_amdgcn_rcpf(ws);
                    o.x = fmaf(k, sx, c.x);
                    o.y = fmaf(k, sy, c.y);
                    o.z = fmaf(k, sz, c.z);
                }
            }
            B[ly * W + lx] = o;
        }
        __syncthreads();
        float4 *t = A; A = B; B = t;
    }

    const DivBy byTW(TW);
    for (int idx = threadIdx.x; idx < TH * TW; idx += kTileBlock) {
        const int ry = byTW.div(idx), rx = idx - ry * TW;
        const int gy = ty0 + ry, gx = tx0 + rx;
        if (gy >= M || gx >= N) continue;
        const size_t off = 3 * ((size_t)gy * N + gx);
        const float4 c = A[(ry + halo) * W + rx + halo];
        if (c.w == 0.f) {                   // +0 or -0: a valid pixel
            dst[off] = c.x; dst[off + 1] = c.y; dst[off + 2] = c.z;
        } else {
            dst[off] = src[off]; dst[off + 1] = src[off + 1]; dst[off + 2] = src[off + 2];
        }
    }
    __syncthreads();                 // LDS is reused by the next tile
}

// ---------------------------------------------------------------------------
// Triangle centroids and normals (Sec. 5.2) of one quad.
// ---------------------------------------------------------------------------

struct V3 {
    float x, y, z;
};

__device__ __forceinline__ bool ok3(const V3 &a) { return !any_nan(a.x, a.y, a.z); }

// centroid (a + b + c) / 3 and unit normal of (b - a) x (c - a); NaN normal
// when the cross product vanishes.
__device__ __forceinline__ void tri_geom(const V3 &a, const V3 &b, const V3 &c, V3 &cen, V3 &nrm) {
    const float third = 1.0f / 3.0f;
    cen.x = (a.x + b.x + c.x) * third;
    cen.y = (a.y + b.y + c.y) * third;
    cen.z = (a.z + b.z + c.z) * third;
    const float e1x = b.x - a.x, e1y = b.y - a.y, e1z = b.z - a.z;
    const float e2x = c.x - a.x, e2y = c.y - a.y, e2z = c.z - a.z;
    // two rounded products and a difference (contraction is off, so the same
    // bits wherever this is inlined): when two corners coincide the edges are
    // equal and the products cancel exactly, so a zero-area triangle gets a
    // zero cross product and a NaN normal.  A fused form would leave the
    // rounding error of one product there instead.
    const float nx = e1y * e2z - e1z * e2y;
    const float ny = e1z * e2x - e1x * e2z;
    const float nz = e1x * e2y - e1y * e2x;
    const float l2 = fmaf(nx, nx, fmaf(ny, ny, nz * nz));
    if (l2 > 0.f) {
        const float k = __builtin_amdgcn_rsqf(l2);
        nrm = V3{nx * k, ny * k, nz * k};
    } else {
        nrm = V3{qnan(), qnan(), qnan()};
    }
}

// Centroids and normals of both triangles of a quad with corners p1 = (u, v),
// p2 = (u, v+1), p3 = (u+1, v+1), p4 = (u+1, v); NaN for a missing triangle.
__device__ __forceinline__ void quad_geom(const V3 &p1, const V3 &p2, const V3 &p3, const V3 &p4,
                                          V3 &c0, V3 &n0, V3 &c1, V3 &n1) {
    const bool v1 = ok3(p1), v2 = ok3(p2), v3 = ok3(p3), v4 = ok3(p4);
    const V3 nan3{qnan(), qnan(), qnan()};
    c0 = nan3; n0 = nan3; c1 = nan3; n1 = nan3;
    if (v1 & v2 & v3) tri_geom(p3, p2, p1, c0, n0);     // first triangle
    if (v1 & v3 & v4) tri_geom(p1, p4, p3, c1, n1);     // second triangle
}

// The corners of quad (qy, qx) of a frame with N points per row.
struct QuadPoints {
    V3 p1, p2, p3, p4;
};

__device__ __forceinline__ QuadPoints quad_points(const float *__restrict__ pts, int N, int qy, int qx) {
    const float *r0 = pts + 3 * ((size_t)qy * N + qx);
    const float *r1 = r0 + 3 * (size_t)N;
    return QuadPoints{{r0[0], r0[1], r0[2]}, {r0[3], r0[4], r0[5]}, {r1[3], r1[4], r1[5]}, {r1[0], r1[1], r1[2]}};
}

// Quad (qy, qx) of a frame with N points per row: centroids and normals.
__device__ __forceinline__ void quad_geom_at(const float *__restrict__ pts, int N, int qy, int qx,
                                             V3 &c0, V3 &n0, V3 &c1, V3 &n1) {
    const float *r0 = pts + 3 * ((size_t)qy * N + qx);
    const float *r1 = r0 + 3 * (size_t)N;
    quad_geom(V3{r0[0], r0[1], r0[2]}, V3{r0[3], r0[4], r0[5]}, V3{r1[3], r1[4], r1[5]},
              V3{r1[0], r1[1], r1[2]}, c0, n0, c1, n1);
}

// Up to kTileBlock consecutive quads [q0, q0 + nq), one per thread, q0 a
// multiple of kTileBlock.  Quad q = (u, v) has its top corners at point
// index q + u, so the block's top corners are one contiguous run of points
// and its bottom corners the run N points further; both runs are read with
// coalesced word loads into LDS (at most 2 kTileBlock points each, reached
// only when N = 2).  A quad's outputs (6 centroid floats, 6 normals) would be
// 24-byte strided per thread, so both are assembled in the same LDS and
// written with coalesced 8-byte (float32) or 4-byte (float16 pairs) stores.
struct NormalsStage {
    float f[2][3 * 2 * kTileBlock];
};

template <typename NT>
__device__ __forceinline__ void normals_block(const float *__restrict__ pts, int N, int Nq, size_t q0,
                                              int nq, NT *__restrict__ normals,
                                              float *__restrict__ centroids, NormalsStage &st) {
    // 6 Q < 2^31 (shape check): 32-bit index arithmetic
    const unsigned ua = (unsigned)q0 / (unsigned)Nq, ub = ((unsigned)q0 + nq - 1) / (unsigned)Nq;
    const size_t P0 = q0 + ua;                              // top-left corner of quad q0
    const int L = (int)(nq + 1 + (ub - ua));                // points per run
    const float *top = pts + 3 * P0, *bot = top + 3 * (size_t)N;
    constexpr int kLoads = 3 * 2 * kTileBlock / kTileBlock;   // all in flight at once
    float wt[kLoads], wb[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
        const int k = j * kTileBlock + threadIdx.x;
        wt[j] = k < 3 * L ? top[k] : 0.f;
        wb[j] = k < 3 * L ? bot[k] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
        const int k = j * kTileBlock + threadIdx.x;
        if (k < 3 * L) {
            st.f[0][k] = wt[j];
            st.f[1][k] = wb[j];
        }
    }
    __syncthreads();
    V3 c0, n0, c1, n1;
    if ((int)threadIdx.x < nq) {
        const unsigned q = (unsigned)q0 + threadIdx.x;
        const int o = 3 * (int)(q + q / (unsigned)Nq - (unsigned)P0);
        const float *t = st.f[0] + o, *b = st.f[1] + o;
        quad_geom(V3{t[0], t[1], t[2]}, V3{t[3], t[4], t[5]}, V3{b[3], b[4], b[5]},
                  V3{b[0], b[1], b[2]}, c0, n0, c1, n1);
    }
    __syncthreads();
    if ((int)threadIdx.x < nq) {
        float *co = st.f[0] + 6 * threadIdx.x;
        co[0] = c0.x; co[1] = c0.y; co[2] = c0.z;
        co[3] = c1.x; co[4] = c1.y; co[5] = c1.z;
        NT *no = reinterpret_cast<NT *>(st.f[1]) + 6 * threadIdx.x;
        st_f(no + 0, n0.x); st_f(no + 1, n0.y); st_f(no + 2, n0.z);
        st_f(no + 3, n1.x); st_f(no + 4, n1.y); st_f(no + 5, n1.z);
    }
    __syncthreads();
    float *gc = centroids + 6 * q0;
    for (int k = threadIdx.x; k < 3 * nq; k += kTileBlock)
        st_stream2(gc + 2 * k, st.f[0][2 * k], st.f[0][2 * k + 1]);
    if (sizeof(NT) == 4) {
        float *g = reinterpret_cast<float *>(normals + 6 * q0);
        for (int k = threadIdx.x; k < 3 * nq; k += kTileBlock)
            st_stream2(g + 2 * k, st.f[1][2 * k], st.f[1][2 * k + 1]);
    } else {
        const uint32_t *s1 = reinterpret_cast<const uint32_t *>(st.f[1]);
        uint32_t *g1 = reinterpret_cast<uint32_t *>(normals + 6 * q0);
        for (int k = threadIdx.x; k < 3 * nq; k += kTileBlock) st_stream(&g1[k], s1[k]);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Bilateral normal filter (Sec. 2.3 Eqs. 3-6; neighbourhood of Sec. 5.2):
// F Jacobi sweeps of one TQH x TQW tile of quads, temporally blocked in LDS.
//
// A thread owns a quad and filters both of its triangles, which share every
// neighbour load (the paper's unit of work).  With log2(e) folded into
//     ka = log2(e) / (2 sigma_l^2),  kb = log2(e) / (2 sigma_a^2),
// a neighbour's weight is w = 2^-e, e = ka ||c_i - c_j||^2 + kb ||n_i - n_j||^2.
// Both squared distances come from component differences (exact for nearby
// float32 values) before scaling; expanding them or pre-scaling the
// centroids saves instructions but costs ~1e-5 relative weight accuracy.
//
// Eq. 6 renormalises, so a common factor of the weights cancels: every
// weight is taken as w = 2^(48 - e) (the same value in exact arithmetic).
// The shift is a constant, so a pair's weight does not depend on which of
// its triangles is being filtered; with e >= 0 no weight exceeds 2^48, which
// keeps the sums and the squared norm of Eq. 6 finite for windows up to
// 9 x 9 (160 neighbours), and terms down to e = 174 stay normal floats.  If
// the weighted sum of normals drops below 2^-60 in norm (always when every
// neighbour is at e > 108; otherwise only where the normals nearly cancel),
// that triangle is recomputed with every exponent shifted by the smallest
// one, which puts the largest term at 1.
// Such triangles are isolated ones (about 7 per thousand on the LiDAR
// frames, 4 per 10^4 on the RGB-D ones), so instead of the lane
// redoing its window alone -- which held up its whole wave -- the lane
// queues the triangle in LDS, and after the sweep one wave per queued
// triangle takes its neighbours over the wave's lanes: the smallest exponent
// by a wave minimum, then the shifted weights and weighted normals summed
// over the lanes in a fixed tree.  The result depends on the triangle's
// window only, not on the tile.
//
// Summation order.  The window's displacements split into D+ (dy = 0 and
// dx > 0, or dy > 0) and their negatives; a triangle sums its terms in a
// fixed order: for each d of D+, the two triangles of quad a+d, then the two
// of quad a-d.  The order is the same for every tile shape and fusion depth,
// so float32 results are too.
//
// A staged quad is 12 floats (c0, c1, n0, n1) in three planes of float4: three
// 16-byte reads per neighbour, 48 bytes per quad (one float4 per vector, 64
// bytes, took four reads and a fourth address).  Off-grid quads and triangles
// with a NaN normal or centroid are staged with an infinite centroid and a
// zero normal: infinite exponent, weight exactly 0, contribution 0.  A triangle that is itself missing is copied through (its
// input bits).  Float16-stored normals produced by an intermediate sweep are
// re-rounded to float16, as if stored between launches, so results do not
// depend on F.  F = 0 copies the tile (and gathers).
// LDS: (TQH + 2RF) * (TQW + 2RF) quads of 48 bytes, twice with F > 1 unless
// the sweeps run in place (bil_in_place; else a sweep writes the second buffer,
// centroids along), a byte of flags per quad and the queue of underflowed
// triangles (16 bits per triangle of the region, and its counts).
// ---------------------------------------------------------------------------

constexpr float kBilUnderflow2 = 0x1p-120f;       // (2^-60)^2
// Register budget of the bilateral kernels, in waves per SIMD: 8 (<= 64 VGPRs)
// for 3x3 and 5x5 windows in the single-frame kernels, 6 (<= 80) elsewhere.  A
// 720 x 1280 frame takes 77.7 us at 8 (79.2 at 7), a 128 x 2048 one 80.8 us at
// 8 (81.8 at 6 and 7); the batch, whose lanes hold four partial sums at 5x5,
// 231.8 us at 6 (243.6 at 8), and its 3x3 kernels are the same at 6, 7 and 8.
// What it costs: at 64 VGPRs every 3x3 and 5x5 single-frame kernel spills 5 to 7
// (24 to 32 bytes of scratch a lane), at 80 the batch's 5x5 ones 2, its 7x7 and
// 9x9 ones 52 and 101 (no sensor's window; a budget of their own not tried).
constexpr int bil_waves_per_simd(int R, bool batch) { return batch || R > 2 ? 6 : 8; }
constexpr float kBilShift = 48.f;                 // every weight is 2^(48 - e)
constexpr int kBilMaxSweeps = 8;                  // fused sweeps per launch at most
#ifndef PL_BIL_PARTS_K3
#define PL_BIL_PARTS_K3 1
#endif
#ifndef PL_BIL_PARTS_K5
#define PL_BIL_PARTS_K5 4
#endif
#ifndef PL_BIL_FRAME_WAVES
#define PL_BIL_FRAME_WAVES 1
#endif
#ifndef PL_BIL_BATCH_WAVES
#define PL_BIL_BATCH_WAVES 0
#endif
// Whether a kernel runs the parts of a quad's sum on its waves (windows of
// 5x5 and up): the single-frame kernels do, the batched ones (many rounds
// of workgroups deep, where wave 0 closing the quads alone idles the others)
// keep them on lanes.
__host__ __device__ constexpr bool bil_waves(int R, bool batch) {
    return R >= 2 && (batch ? PL_BIL_BATCH_WAVES : PL_BIL_FRAME_WAVES) != 0;
}
// floats of the parts' exchange when the parts run on waves: the partial
// sums of parts 1.. of 64 quads
__host__ __device__ constexpr int bil_xch_floats(int R) {
    return R >= 2 ? (PL_BIL_PARTS_K5 - 1) * 6 * 64 : 0;
}
// Whether a launch of F sweeps runs the sweeps before the last in place: every
// quad of their regions has a thread of its own (3x3 windows), which keeps its
// result in registers until all have read.
__host__ __device__ constexpr bool bil_in_place(int R, int F, int TQH, int TQW) {
    return R == 1 && PL_BIL_PARTS_K3 == 1 && F > 1 &&
           (long)(TQH + 2 * (F - 1)) * (TQW + 2 * (F - 1)) <= kTileBlock;
}
__host__ __device__ constexpr size_t bil_lds_bytes(int R, int F, int TQH, int TQW, bool waves) {
    const size_t S = (size_t)(TQH + 2 * R * F) * (size_t)(TQW + 2 * R * F);
    return (F > 1 && !bil_in_place(R, F, TQH, TQW) ? 6 : 3) * sizeof(float4) * S +
           sizeof(int) * (kBilMaxSweeps + 1) + sizeof(uint16_t) * 2 * S +
           sizeof(int) * (size_t)TQH * TQW +    // T ranks of the tile (gather from the mesh masks)
           (waves ? sizeof(float) * (size_t)bil_xch_floats(R) : 0) + S;
}

// The mesh's chunks and per-segment counts (pl_mesh_opc's first pass): with
// them the gather finds each triangle's place in T itself instead of reading
// T_map, so the pass can run in the same launch as the mesh emit.
struct GatherCodes {
    const MeshChunk *chunks;
    const uint16_t *seg;
    int K;                      // chunks of the frame
};

// Output stores of the filter: streaming for float32 normals, plain for
// float16 (measured on float32 only).
__device__ __forceinline__ void bil_store(float *p, float v) { st_stream(p, v); }
__device__ __forceinline__ void bil_store(__half *p, __half v) { *p = v; }

template <typename NT> __device__ __forceinline__ float round_storage(float x);
template <> __device__ __forceinline__ float round_storage<float>(float x) { return x; }
template <> __device__ __forceinline__ float round_storage<__half>(float x) {
    return __half2float(__float2half_rn(f32_rounded(x)));
}

struct BilOwn {
    float cx, cy, cz;
    float nx, ny, nz;
    float ka, kb;
};

__device__ __forceinline__ float bil_pair_e(const BilOwn &o, const V3 &c, const V3 &n) {
    const float ax = o.nx - n.x, ay = o.ny - n.y, az = o.nz - n.z;
    const float dn2 = fmaf(ax, ax, fmaf(ay, ay, az * az));
    const float dx = o.cx - c.x, dy = o.cy - c.y, dz = o.cz - c.z;
    const float dc2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    return fmaf(dc2, o.ka, dn2 * o.kb);
}

// A quad's centroids and normals, and their place in LDS: floats 0..11 of
// (c0, c1, n0, n1) are plane i / 4, component i mod 4.
struct BilQuad {
    V3 c0, c1, n0, n1;
};

__device__ __forceinline__ BilQuad bil_read(const float4 *s, int a, int plane) {
    const float4 p = s[a], q = s[plane + a], r = s[2 * plane + a];
    return BilQuad{{p.x, p.y, p.z}, {p.w, q.x, q.y}, {q.z, q.w, r.x}, {r.y, r.z, r.w}};
}

__device__ __forceinline__ void bil_write(float4 *s, int a, int plane, const V3 &c0, const V3 &c1,
                                          const V3 &n0, const V3 &n1) {
    s[a] = make_float4(c0.x, c0.y, c0.z, c1.x);
    s[plane + a] = make_float4(c1.y, c1.z, n0.x, n0.y);
    s[2 * plane + a] = make_float4(n0.z, n1.x, n1.y, n1.z);
}

__device__ __forceinline__ void bil_write_normals(float4 *s, int a, int plane, const V3 &n0, const V3 &n1) {
    *reinterpret_cast<float2 *>(&s[plane + a].z) = make_float2(n0.x, n0.y);
    s[2 * plane + a] = make_float4(n0.z, n1.x, n1.y, n1.z);
}

// Vector v (0: c0, 1: c1, 2: n0, 3: n1) of the quad at a.
__device__ __forceinline__ float *bil_at(float4 *s, int a, int plane, int i) {
    return reinterpret_cast<float *>(s + (i >> 2) * plane + a) + (i & 3);
}
__device__ __forceinline__ V3 bil_vec(const float4 *s, int a, int plane, int v) {
    float4 *t = const_cast<float4 *>(s);
    return V3{*bil_at(t, a, plane, 3 * v), *bil_at(t, a, plane, 3 * v + 1), *bil_at(t, a, plane, 3 * v + 2)};
}

// Flags of a staged quad: bit k: triangle k is usable; bit 2 + k: it is not,
// and its normal as stored is the canonical NaN in every component (from the
// points: for a missing corner, where its centroid is that too).
constexpr int kBilUsable = 1, kBilCanonical = 4;

__device__ __forceinline__ bool is_qnan(float x) { return __float_as_uint(x) == 0x7fc00000u; }
__device__ __forceinline__ bool is_qnan(__half x) { return __half_as_ushort(x) == 0x7e00u; }

// Sum of weighted neighbour normals.  Eq. 6 renormalises it, so the sum of
// the weights is not needed; the underflow test uses the vector's norm,
// which never exceeds the total weight (unit normals).
struct BilAcc {
    float x, y, z;
};

// s += 2^(m - e) * n
__device__ __forceinline__ void bil_add(BilAcc &s, float m, float e, const V3 &n) {
    const float w = __builtin_amdgcn_exp2f(m - e);
    s.x = fmaf(w, n.x, s.x);
    s.y = fmaf(w, n.y, s.y);
    s.z = fmaf(w, n.z, s.z);
}

// The i-th displacement of D+: dy = 0, dx = 1..R, then dy = 1..R, dx = -R..R.
template <int R>
__device__ __forceinline__ void bil_dplus(int i, int &dy, int &dx) {
    if (i < R) {
        dy = 0;
        dx = i + 1;
    } else {
        const int j = i - R;
        dy = 1 + j / (2 * R + 1);
        dx = j % (2 * R + 1) - R;
    }
}
template <int R> constexpr int bil_ndplus() { return 2 * R * R + 2 * R; }

__device__ __forceinline__ float bil_norm2(const BilAcc &s) {
    return fmaf(s.x, s.x, fmaf(s.y, s.y, s.z * s.z));
}

template <typename NT>
__device__ __forceinline__ V3 bil_finish(BilAcc s, const V3 &cur) {
    const float l2 = bil_norm2(s);
    if (!(l2 > 0.f)) return cur;            // no usable neighbour
    const float k = __builtin_amdgcn_rsqf(l2);
    return V3{round_storage<NT>(s.x * k), round_storage<NT>(s.y * k), round_storage<NT>(s.z * k)};
}

// Exponent of a triangle pair's weight (Eqs. 4-5 with log2(e) folded into ka
// and kb), shifted by the constant 48: the weight is 2^(48 - e).  The value
// depends on the pair only: swapping the triangles changes the sign of every
// difference exactly and none of the squares.  A pair with an off-grid or missing
// triangle has e = +inf and weight 0 (NaN only when both are missing; no sum
// uses that).
__device__ __forceinline__ float bil_exponent(const V3 &ci, const V3 &ni, const V3 &cj, const V3 &nj,
                                              float ka, float kb) {
    const float ax = ni.x - nj.x, ay = ni.y - nj.y, az = ni.z - nj.z;
    const float dn2 = fmaf(ax, ax, fmaf(ay, ay, az * az));
    const float dx = ci.x - cj.x, dy = ci.y - cj.y, dz = ci.z - cj.z;
    const float dc2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    return -fmaf(dc2, ka, fmaf(dn2, kb, -kBilShift));
}

// s += w n
__device__ __forceinline__ void bil_acc(BilAcc &s, float w, const V3 &n) {
    s.x = fmaf(w, n.x, s.x);
    s.y = fmaf(w, n.y, s.y);
    s.z = fmaf(w, n.z, s.z);
}

// Eq. 6 for one triangle: a missing one (not ok) is copied through; pend:
// the weighted sum fell below 2^-60 in norm (the triangle goes to the queue
// and r is not set).  Every total weight below 2^-60 is caught, since the
// norm is at most the total weight.
template <typename NT>
__device__ __forceinline__ V3 bil_close(bool ok, const V3 &n, BilAcc s, bool &pend) {
    pend = ok && !(bil_norm2(s) >= kBilUnderflow2);
    return ok ? bil_finish<NT>(s, n) : n;
}

// Minimum and sum over the wave, every lane active, the same on every lane: the
// tree of pairs 1, 2, 4, 8, 16 and 32 lanes apart.  The first four steps are
// lane permutations within rows of 16 (by then every lane of a group of 4 or 8
// holds the group's value, so a mirror reaches the partner group), the four
// rows' values then meet as scalars.  (As six dependent trips through LDS each,
// the four reductions of a triangle took about 3,000 clocks at the end of a
// workgroup.)
template <int Ctrl> __device__ __forceinline__ float row_perm(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), Ctrl, 0xf, 0xf, true));
}
constexpr int kQuadXor1 = 0xb1, kQuadXor2 = 0x4e, kHalfMirror = 0x141, kRowMirror = 0x140;

__device__ __forceinline__ float row_value(float x, int row) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16 * row));
}

__device__ __forceinline__ float wave_min_f(float x) {
    x = fminf(x, row_perm<kQuadXor1>(x));
    x = fminf(x, row_perm<kQuadXor2>(x));
    x = fminf(x, row_perm<kHalfMirror>(x));
    x = fminf(x, row_perm<kRowMirror>(x));
    return fminf(fminf(row_value(x, 0), row_value(x, 1)), fminf(row_value(x, 2), row_value(x, 3)));
}

__device__ __forceinline__ float wave_sum_f(float x) {
    x += row_perm<kQuadXor1>(x);
    x += row_perm<kQuadXor2>(x);
    x += row_perm<kHalfMirror>(x);
    x += row_perm<kRowMirror>(x);
    return (row_value(x, 0) + row_value(x, 1)) + (row_value(x, 2) + row_value(x, 3));
}

// The underflowed triangle k of the quad at LDS index a, by one whole wave:
// lane l takes neighbours j = l, l + 64, ... in the main pass's order (j / 4
// the displacement of D+, bit 1 the side, bit 0 the triangle), the shift is
// the smallest exponent (a wave minimum, exact), and the shifted sums are
// added lane by lane in a fixed butterfly.  Every lane returns the result.
template <int R, typename NT>
__device__ __forceinline__ V3 bil_fallback_wave(const float4 *st, int a, int k, int pitch, int plane,
                                                float ka, float kb) {
    constexpr int kN = 4 * bil_ndplus<R>();               // neighbours
    constexpr int kPer = (kN + kWave - 1) / kWave;         // per lane
    const int lane = (int)threadIdx.x & (kWave - 1);
    const V3 c = bil_vec(st, a, plane, k), n = bil_vec(st, a, plane, 2 + k);
    const BilOwn o{c.x, c.y, c.z, n.x, n.y, n.z, ka, kb};
    const float inf = __builtin_inff();
    float e[kPer];
    V3 nj[kPer];
    float mn = inf;
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
        const int j = lane + t * kWave;
        e[t] = inf;
        nj[t] = V3{0.f, 0.f, 0.f};
        if (j < kN) {
            int dy, dx;
            bil_dplus<R>(j >> 2, dy, dx);
            const int off = dy * pitch + dx;
            const int b = ((j >> 1) & 1) ? a - off : a + off;
            const int kk = j & 1;
            const V3 cj = bil_vec(st, b, plane, kk);
            nj[t] = bil_vec(st, b, plane, 2 + kk);
            e[t] = bil_pair_e(o, cj, nj[t]);
            mn = fminf(mn, e[t]);
        }
    }
    mn = wave_min_f(mn);
    BilAcc s{0.f, 0.f, 0.f};
    if (mn < inf) {
#pragma unroll
        for (int t = 0; t < kPer; ++t) bil_add(s, mn, e[t], nj[t]);
    }
    s.x = wave_sum_f(s.x);
    s.y = wave_sum_f(s.y);
    s.z = wave_sum_f(s.z);
    return bil_finish<NT>(s, n);
}

// Queue of underflowed triangles in LDS: entries 2 a + k (at most two per
// quad of the staged region, so it cannot overflow) and one count per sweep
// (sweep f counts into count[f], so no count is reset in between).
struct BilQueue {
    uint16_t *entry;                 // 2 a + k fits: LDS holds under 3,500 quads
    int *count;
};

__device__ __forceinline__ void bil_push(const BilQueue &qu, int a, int k, int sweep) {
    const int i = atomicAdd(&qu.count[sweep], 1);
    qu.entry[i] = (uint16_t)(2 * a + k);
}

// Parts per quad: the displacements of D+ are dealt over P parts (part p
// takes i = p, p + P, ...), whose partial sums are then added in a fixed
// tree -- (s_0 + s_1) for P = 2, ((s_0 + s_1) + (s_2 + s_3)) for P = 4 --
// identical on every lane of the quad (addition commutes exactly).  Larger
// windows take more parts: a 5x5 window has 48 neighbours per triangle, and
// a LiDAR frame of 64 x 1024 quads filled only one wave per SIMD at one lane
// per quad.  A kernel runs the P parts on PP lanes (PP dividing P): a lane
// keeps the partial sums of its P / PP parts apart and adds them in the same
// tree, so every kernel gives the same bits whatever its PP.  The single-
// frame kernels put the four parts of a 5x5-and-up quad on the workgroup's
// four waves instead (bil_sweep_waves, same tree again); the batch, many
// rounds deep and bound by VALU issue, runs them on one lane, which needs no
// lane tree and closes and stores each quad once.
template <int R> constexpr int bil_parts() { return R == 1 ? PL_BIL_PARTS_K3 : PL_BIL_PARTS_K5; }
#ifndef PL_BIL_BATCH_LANES_K5
#define PL_BIL_BATCH_LANES_K5 1
#endif
// lanes per quad (0: parts on waves) of the single-frame kernels
template <int R> constexpr int bil_frame_lanes() {
    return bil_waves(R, false) ? 0 : bil_parts<R>();
}
// lanes per quad (0: parts on waves) of the batched kernels
template <int R> constexpr int bil_batch_lanes() {
    return bil_waves(R, true) ? 0 : (R == 1 ? bil_parts<1>() : PL_BIL_BATCH_LANES_K5);
}
static_assert(bil_ndplus<1>() % PL_BIL_PARTS_K3 == 0 && bil_ndplus<2>() % PL_BIL_PARTS_K5 == 0 &&
                  bil_ndplus<3>() % PL_BIL_PARTS_K5 == 0 && bil_ndplus<4>() % PL_BIL_PARTS_K5 == 0,
              "the parts of a quad share |D+| evenly");

// The tree over the P parts of a quad held as P / PP sets on PP lanes (part
// p = lane + k PP is set k): its steps with m < PP add across lanes, the
// rest across sets, each term its own value plus its partner's.
template <int P, int PP>
__device__ __forceinline__ BilAcc bil_reduce(BilAcc (&s)[P / PP]) {
    constexpr int NS = P / PP;
#pragma unroll
    for (int m = 1; m < PP; m <<= 1) {
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            s[k].x += __shfl_xor(s[k].x, m, kWave);
            s[k].y += __shfl_xor(s[k].y, m, kWave);
            s[k].z += __shfl_xor(s[k].z, m, kWave);
        }
    }
#pragma unroll
    for (int m = 1; m < NS; m <<= 1) {
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            if (k & m) continue;
            const int o = k ^ m;
            const BilAcc u{s[k].x + s[o].x, s[k].y + s[o].y, s[k].z + s[o].z};
            s[k] = u;
            s[o] = u;
        }
    }
    return s[0];
}

// The terms of the i-th displacement d of D+ for both triangles of the quad
// at LDS index a (own centroids c, normals n): the two triangles of quad
// a + d, then the two of quad a - d.
//
// Bound by VALU issue: about 48 clocks per pair and SIMD without the
// exponential, and an exponential among other instructions costs 15 to 24 more
// where a row of them takes 8 each.  The eight of a displacement are therefore
// kept together (the barriers stop the scheduler from spreading them): 128 x
// 2048 points at 5x5 81.1 to 78.6 us a frame, 64 x 1024 39.6 to 38.8, a batch of
// seven frames 232.5 to 225.3 us, 3x3 frames 0.1 to 0.2 us less.
template <int R>
__device__ __forceinline__ void bil_disp(const float4 *st, int a, int pitch, int plane, float ka,
                                         float kb, int i, const BilQuad &q, BilAcc &s0, BilAcc &s1) {
    int dy, dx;
    bil_dplus<R>(i, dy, dx);
    const int off = dy * pitch + dx;
    const BilQuad p = bil_read(st, a + off, plane), m = bil_read(st, a - off, plane);
    const V3 c[4] = {p.c0, p.c1, m.c0, m.c1}, n[4] = {p.n0, p.n1, m.n0, m.n1};
    float w[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        w[k] = bil_exponent(q.c0, q.n0, c[k], n[k], ka, kb);
        w[4 + k] = bil_exponent(q.c1, q.n1, c[k], n[k], ka, kb);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = __builtin_amdgcn_exp2f(w[k]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        bil_acc(s0, w[k], n[k]);
        bil_acc(s1, w[4 + k], n[k]);
    }
}

// Both triangles of the quad at LDS index a, in the fixed summation order:
// for each d of D+ (part p's share of them), the two triangles of quad
// a + d, then the two of quad a - d; the parts' partial sums are added in a
// fixed tree.  This lane (`lane` of PP) runs parts lane, lane + PP, ...: the
// i-th displacement belongs to part i mod P, whose set here is
// (i mod P) / PP.  Every lane of the quad returns the same r0, r1 and pending
// flags.
template <int R, typename NT, int PP>
__device__ __forceinline__ void bil_sum_quad(const float4 *st, int a, int pitch, int plane, float ka,
                                             float kb, int lane, const BilQuad &q, const uint8_t *flag,
                                             int &flags, V3 &r0,
                                             V3 &r1, bool &pend0, bool &pend1) {
    constexpr int ND = bil_ndplus<R>(), P = bil_parts<R>(), NS = P / PP;
    static_assert(P % PP == 0, "the lanes of a quad share its parts evenly");
    BilAcc s0[NS], s1[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        s0[k] = BilAcc{0.f, 0.f, 0.f};
        s1[k] = BilAcc{0.f, 0.f, 0.f};
    }
#pragma unroll 1
    for (int j0 = 0; j0 < ND / PP; j0 += NS) {
#pragma unroll
        for (int k = 0; k < NS; ++k)            // displacement j0 + k: set k
            bil_disp<R>(st, a, pitch, plane, ka, kb, (j0 + k) * PP + lane, q, s0[k], s1[k]);
    }
    flags = flag[a];
    r0 = bil_close<NT>(flags & 1, q.n0, bil_reduce<P, PP>(s0), pend0);
    r1 = bil_close<NT>(flags & 2, q.n1, bil_reduce<P, PP>(s1), pend1);
}

// One sweep over the OH x OW region at (oy0, ox0) of the staged tile;
// out(ry, rx, a, q, flags, pre(ry, rx), r0, r1, pend0, pend1) takes each quad's
// results (ry, rx within the region; q its staged values); pre is called
// before the sum if registers allow, so that what it loads arrives meanwhile.
// Ends with a barrier.
template <int R, typename NT, int PP, typename Pre, typename Out>
__device__ __forceinline__ void bil_sweep(const float4 *st, const uint8_t *flag, int pitch, int plane,
                                          int oy0, int ox0, int OH, int OW, float ka, float kb,
                                          Pre &&pre, Out &&out) {
    const int slot = (int)threadIdx.x / PP, lane = (int)threadIdx.x % PP;
    const DivBy byOW(OW);
    for (int idx = slot; idx < OH * OW; idx += kTileBlock / PP) {
        const int ry = byOW.div(idx), rx = idx - ry * OW;
        const int a = (oy0 + ry) * pitch + ox0 + rx;
        // a lane that holds several partial sums has no registers to spare for it
        constexpr bool kEarly = bil_parts<R>() == PP;
        int2 early = make_int2(-1, -1);
        if (kEarly) early = pre(ry, rx);
        const BilQuad q = bil_read(st, a, plane);
        int fl;
        V3 r0, r1;
        bool p0, p1;
        bil_sum_quad<R, NT, PP>(st, a, pitch, plane, ka, kb, lane, q, flag, fl, r0, r1, p0, p1);
        if (!kEarly) early = pre(ry, rx);
        out(ry, rx, a, q, fl, early, r0, r1, p0, p1);
    }
    __syncthreads();
}

// The same sweep with the P parts of a quad on the workgroup's P waves
// (wave w runs part w of 64 quads at a time): the displacement index is the
// same on every lane of a wave, so its decoding and the neighbour offsets
// are scalar work; waves 1.. leave their partial sums in `xch`, and wave 0
// adds them in the tree of bil_reduce -- ((s_0 + s_1) + (s_2 + s_3)) --
// closes the quad and calls out, alone.  Same bits as the lane form.
template <int R, typename NT, typename Pre, typename Out>
__device__ __forceinline__ void bil_sweep_waves(const float4 *st, const uint8_t *flag, int pitch,
                                                int plane, int oy0, int ox0, int OH, int OW,
                                                float ka, float kb, float *xch, Pre &&pre,
                                                Out &&out) {
    constexpr int ND = bil_ndplus<R>(), P = bil_parts<R>();
    static_assert(P == 4 && P == kTileBlock / kWave, "one wave per part, tree of four");
    static_assert(bil_xch_floats(R) == (P - 1) * 6 * kWave, "exchange size");
    const int part = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int lane = (int)threadIdx.x & (kWave - 1);
    const DivBy byOW(OW);
    const int n = OH * OW;
    for (int base = 0; base < n; base += kWave) {
        const int idx = base + lane;
        const bool have = idx < n;
        const int ry = have ? byOW.div(idx) : 0, rx = have ? idx - ry * OW : 0;
        const int a = (oy0 + ry) * pitch + ox0 + rx;
        BilAcc s0{0.f, 0.f, 0.f}, s1{0.f, 0.f, 0.f};
        BilQuad q;
        int2 early = make_int2(-1, -1);
        if (part == 0 && have) early = pre(ry, rx);
        if (have) {
            q = bil_read(st, a, plane);
#pragma unroll 1
            for (int j = 0; j < ND / P; ++j)
                bil_disp<R>(st, a, pitch, plane, ka, kb, j * P + part, q, s0, s1);
        }
        if (part != 0) {
            float *x = xch + (part - 1) * 6 * kWave + lane;
            x[0] = s0.x; x[kWave] = s0.y; x[2 * kWave] = s0.z;
            x[3 * kWave] = s1.x; x[4 * kWave] = s1.y; x[5 * kWave] = s1.z;
        }
        __syncthreads();
        if (part == 0 && have) {
            const float *x1 = xch + lane, *x2 = x1 + 6 * kWave, *x3 = x2 + 6 * kWave;
            const BilAcc t0{(s0.x + x1[0]) + (x2[0] + x3[0]),
                            (s0.y + x1[kWave]) + (x2[kWave] + x3[kWave]),
                            (s0.z + x1[2 * kWave]) + (x2[2 * kWave] + x3[2 * kWave])};
            const BilAcc t1{(s1.x + x1[3 * kWave]) + (x2[3 * kWave] + x3[3 * kWave]),
                            (s1.y + x1[4 * kWave]) + (x2[4 * kWave] + x3[4 * kWave]),
                            (s1.z + x1[5 * kWave]) + (x2[5 * kWave] + x3[5 * kWave])};
            const int fl = flag[a];
            bool p0, p1;
            const V3 r0 = bil_close<NT>(fl & 1, q.n0, t0, p0);
            const V3 r1 = bil_close<NT>(fl & 2, q.n1, t1, p1);
            out(ry, rx, a, q, fl, early, r0, r1, p0, p1);
        }
        if (base + kWave < n) __syncthreads();   // xch is reused by the next 64 quads
    }
    __syncthreads();
}

// T ranks of a tile's quads for the gather: rank[ty TQW + tx] is the index
// in T of quad (qy0 + ty, qx0 + tx)'s first valid triangle, with the quad's
// validity in bits 30..31 (T has fewer than 2^30 triangles).  T is the valid
// triangles in GID order, so the rank is the count of the segments before the
// quad's, plus the valid triangles before it in its segment (mesh_window):
// each wave takes tile rows.  Quads off the grid have no valid triangle.  No
// barrier: the caller's next one publishes the ranks.
__device__ __forceinline__ void bil_gather_ranks(const GatherCodes &gc, int Mq, int Nq, int qy0,
                                                 int qx0, int TQH, int TQW, int *rank) {
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    // segments before the tile's first row: the same for every row of it
    const int k0 = (int)(((long)qy0 * Nq + qx0) / kMeshSeg);
    const int before = wave_sum(mesh_sum_segs(gc.seg, k0, lane, kWave));
    for (int ty = wave; ty < TQH; ty += kTileBlock / kWave) {
        const int u = qy0 + ty;
        for (int t0 = 0; t0 < TQW; t0 += kWave) {
            const int tx = t0 + lane, v = qx0 + tx;
            int r = 0;
            if (u < Mq && qx0 + t0 < Nq) {
                const int q = u * Nq + qx0 + t0;
                int c = 0;
                for (int k = k0 + lane; k < q / kMeshSeg; k += kWave) c += gc.seg[k];
                const int base = before + wave_sum(c);
                const MeshWindow w = mesh_window(mesh_chunk(gc.chunks, gc.K, q >> 6),
                                                 mesh_chunk(gc.chunks, gc.K, (q >> 6) + 1), q);
                if (v < Nq)
                    r = (base + w.before + mesh_rank(w)) | ((int)lane_bit(w.f) << 30) |
                        (int)((unsigned)lane_bit(w.s) << 31);
            }
            if (tx < TQW) rank[ty * TQW + tx] = r;
        }
    }
}

// FromPts: the raw normals and centroids are not read but computed here from
// the (smoothed) points `pts` exactly as normals_block computes and stores
// them (normals rounded to NT), and the tile's centroids are written to
// `cen` -- the batched path's first pass, which then needs no normals
// stage.  Otherwise nin / cen are the stored raw normals and centroids.
// PP: lanes per quad for the parts of its sum (bil_parts); 0 puts the parts
// on the workgroup's waves instead (bil_sweep_waves; windows of 5x5 and up).
template <int R, typename NT, bool FromPts = false, bool ByCodes = false, int PP = bil_parts<R>()>
__device__ __forceinline__ void bil_tile(const NT *__restrict__ nin, const float *__restrict__ cen,
                                         NT *__restrict__ nout, int Mq, int Nq, float ka, float kb,
                                         int F, int TQH, int TQW, int qy0, int qx0,
                                         const int32_t *__restrict__ tri_map, NT *__restrict__ nT,
                                         float4 *lds, const float *__restrict__ pts = nullptr,
                                         float *__restrict__ cen_out = nullptr,
                                         GatherCodes gc = GatherCodes{}) {
    const int halo = R * F;
    const int H = TQH + 2 * halo, W = TQW + 2 * halo, S = H * W;
    const bool in_place = bil_in_place(R, F, TQH, TQW);
    float4 *st = lds;                   // [3][S] staged quads
    float4 *st2 = lds + 3 * S;          // [3][S] the next sweep's (F > 1, not in place)
    int *counts = reinterpret_cast<int *>(lds + (F > 1 && !in_place ? 6 : 3) * S);
    if (threadIdx.x < kBilMaxSweeps + 1) counts[threadIdx.x] = 0;
    // T ranks of the tile when the gather takes them from the mesh masks
    int *rank = counts + kBilMaxSweeps + 1;
    // the parts' exchange (parts on waves)
    float *xch = reinterpret_cast<float *>(rank + TQH * TQW);
    // queue of underflowed triangles: 2S entries, one count per sweep
    const BilQueue qu{reinterpret_cast<uint16_t *>(xch + (PP == 0 ? bil_xch_floats(R) : 0)), counts};
    uint8_t *flag = reinterpret_cast<uint8_t *>(qu.entry + 2 * S);   // [S]
    constexpr bool waves = PP == 0;
    static_assert(!waves || R >= 2, "parts on waves for windows of 5x5 and up");
    constexpr bool by_codes = ByCodes;
    if constexpr (by_codes) {
        bil_gather_ranks(gc, Mq, Nq, qy0, qx0, TQH, TQW, rank);
        if (F == 0) __syncthreads();
    }
    // indices in T of the two triangles of tile quad (ty, tx), -1 for none (or
    // no gather); read before the quad's sum, for the T_map of the launch
    // before this one comes from memory
    auto t_index = [&](int ty, int tx) -> int2 {
        int2 t = make_int2(-1, -1);
        if constexpr (by_codes) {
            const unsigned r = (unsigned)rank[ty * TQW + tx];
            const int code = (int)(r >> 30), base = (int)(r & 0x3fffffffu);
            if (code & 1) t.x = base;
            if (code & 2) t.y = base + (code & 1);
        } else if (tri_map && qy0 + ty < Mq && qx0 + tx < Nq) {
            t = *reinterpret_cast<const int2 *>(tri_map + 2 * ((size_t)(qy0 + ty) * Nq + qx0 + tx));
        }
        return t;
    };
    const float inf = __builtin_inff();
    const int oy = qy0 - halo, ox = qx0 - halo;

    struct RawPoints { QuadPoints p; };
    struct RawNormals {
        union { uint32_t w[6 * sizeof(NT) / 4]; NT n[6]; };
        float c[6];
    };
    using Raw = std::conditional_t<FromPts, RawPoints, RawNormals>;
    if (F > 0) {
        const DivBy byW(W);
        // two quads per thread and pass, the loads of both issued before
        // either is used (a tile has more quads with its halo than the
        // workgroup threads: one at a time waited for memory twice).  With
        // the leaner staging and the T_map read ahead of the sums, a 480 x 640
        // frame took 36.5 us (39.1 before), a 120 x 160 one 14.4 us (15.6), a
        // batch of seven mixed frames 247 us (264); VALU instructions of the
        // first bilateral launch of a 720 x 1280 frame 19.0 M (21.6 M)
        constexpr int kU = 2;
        for (int base = threadIdx.x; base < S; base += kU * kTileBlock) {
            Raw raw[kU];
            bool in[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int idx = base + u * kTileBlock;
                const int ly = byW.div(idx), lx = idx - ly * W;
                const int qy = oy + ly, qx = ox + lx;
                in[u] = idx < S && (unsigned)qy < (unsigned)Mq && (unsigned)qx < (unsigned)Nq;
                if (!in[u]) continue;
                if constexpr (FromPts) {
                    raw[u].p = quad_points(pts, Nq + 1, qy, qx);
                } else {
                    const size_t o = 6 * ((size_t)qy * Nq + qx);
                    // by words: six halves lie on a word's border as six floats do
                    // (half by half, one float16 sweep of 480 x 640 points took
                    // 11.9 us instead of 11.7, of 64 x 1024 6.3 instead of 6.2)
                    constexpr int kWords = 6 * (int)sizeof(NT) / 4;
                    const uint32_t *nw = reinterpret_cast<const uint32_t *>(nin + o);
#pragma unroll
                    for (int i = 0; i < kWords; ++i) raw[u].w[i] = nw[i];
#pragma unroll
                    for (int i = 0; i < 6; ++i) raw[u].c[i] = cen[o + i];
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int idx = base + u * kTileBlock;
                if (idx >= S) break;
                V3 c0{inf, inf, inf}, c1 = c0, n0{0.f, 0.f, 0.f}, n1 = n0;
                int fl = 0;
                if (in[u]) {
                    V3 d0, d1, m0, m1;
                    bool ok0, ok1, canon0, canon1;
                    if constexpr (FromPts) {
                        const QuadPoints &g = raw[u].p;
                        const bool diag = ok3(g.p1) && ok3(g.p3);
                        const bool has0 = diag && ok3(g.p2), has1 = diag && ok3(g.p4);
                        tri_geom(g.p3, g.p2, g.p1, d0, m0);
                        tri_geom(g.p1, g.p4, g.p3, d1, m1);
                        m0 = V3{round_storage<NT>(m0.x), round_storage<NT>(m0.y), round_storage<NT>(m0.z)};
                        m1 = V3{round_storage<NT>(m1.x), round_storage<NT>(m1.y), round_storage<NT>(m1.z)};
                        ok0 = has0 && ok3(d0) && ok3(m0);
                        ok1 = has1 && ok3(d1) && ok3(m1);
                        canon0 = !has0;
                        canon1 = !has1;
                    } else {
                        const NT *n = raw[u].n;
                        const float *c = raw[u].c;
                        d0 = V3{c[0], c[1], c[2]};
                        d1 = V3{c[3], c[4], c[5]};
                        m0 = V3{ld_f(n), ld_f(n + 1), ld_f(n + 2)};
                        m1 = V3{ld_f(n + 3), ld_f(n + 4), ld_f(n + 5)};
                        ok0 = ok3(d0) && ok3(m0);
                        ok1 = ok3(d1) && ok3(m1);
                        canon0 = is_qnan(n[0]) && is_qnan(n[1]) && is_qnan(n[2]);
                        canon1 = is_qnan(n[3]) && is_qnan(n[4]) && is_qnan(n[5]);
                    }
                    if (ok0) { c0 = d0; n0 = m0; }
                    if (ok1) { c1 = d1; n1 = m1; }
                    fl = (ok0 ? kBilUsable : 0) | (ok1 ? 2 * kBilUsable : 0) |
                         (canon0 ? kBilCanonical : 0) | (canon1 ? 2 * kBilCanonical : 0);
                }
                bil_write(st, idx, S, c0, c1, n0, n1);
                flag[idx] = (uint8_t)fl;
            }
        }
        __syncthreads();
    }

    const float4 *cur = st;
    float4 *nxt = st2;
    // PP lanes per quad: quad slot and lane within the quad; parts on
    // waves: the lane is the slot, the wave the part (only part 0 stores)
    constexpr int QL = waves ? 1 : PP;                       // lanes per quad
    const int slot = waves ? (int)threadIdx.x % kWave : (int)threadIdx.x / QL;
    const int part = waves ? (int)threadIdx.x / kWave : (int)threadIdx.x % QL;
    const int wave = (int)threadIdx.x / kWave, lane = (int)threadIdx.x & (kWave - 1);
    // one sweep over the OH x OW region at (o0, o0) of the staged tile
    auto sweep = [&](int o0, int OH, int OW, auto &&pre, auto &&out) {
        if constexpr (waves)
            bil_sweep_waves<R, NT>(cur, flag, W, S, o0, o0, OH, OW, ka, kb, xch, pre, out);
        else
            bil_sweep<R, NT, PP>(cur, flag, W, S, o0, o0, OH, OW, ka, kb, pre, out);
    };
    // Intermediate sweeps over the shrinking exact region, in place: a quad's
    // normals stay in its thread's registers until every thread has read, and a
    // wave sums the underflowed triangles of its own quads.  With one buffer eight
    // workgroups fit a CU where two buffers left four, so two sweeps fused beat two
    // launches on large frames too: the second launch's read of normals and
    // centroids and the first one's store of normals (66 of 240 MB on a 720 x 1280
    // frame) outweigh the halo computed twice.  480 x 640 frame 35.4 to 33.7 us,
    // 720 x 1280 83.3 to 77.7, a batch of seven frames 231 to 216 (between two
    // buffers such a tile took 91 us at 720 x 1280).
    if constexpr (R == 1 && PP == 1) {
        if (in_place) {
            for (int f = 1; f < F; ++f) {
                const int lo = R * f, OH = H - 2 * lo, OW = W - 2 * lo;
                const DivBy byOW(OW);
                const int idx = (int)threadIdx.x;
                const bool have = idx < OH * OW;
                const int ry = have ? byOW.div(idx) : 0, rx = have ? idx - ry * OW : 0;
                const int a = (lo + ry) * W + lo + rx;
                V3 r[2];
                bool pend[2] = {false, false};
                if (have) {
                    const BilQuad q = bil_read(st, a, S);
                    int fl;
                    bil_sum_quad<R, NT, PP>(st, a, W, S, ka, kb, 0, q, flag, fl, r[0], r[1], pend[0],
                                            pend[1]);
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    for (unsigned long long m = __ballot(pend[k]); m; m &= m - 1) {
                        const int l = __builtin_ctzll(m);
                        const V3 x = bil_fallback_wave<R, NT>(st, __builtin_amdgcn_readlane(a, l), k, W, S,
                                                              ka, kb);
                        if (lane == l) r[k] = x;
                    }
                }
                __syncthreads();
                if (have) bil_write_normals(st, a, S, r[0], r[1]);
                __syncthreads();
            }
        }
    }
    // else from one buffer to the other
    for (int f = in_place ? F : 1; f < F; ++f) {
        const int lo = R * f;
        sweep(lo, H - 2 * lo, W - 2 * lo, [](int, int) { return make_int2(-1, -1); },
              [&](int, int, int a, const BilQuad &q, int, int2, const V3 &r0, const V3 &r1, bool p0, bool p1) {
                  if (part != 0) return;
                  bil_write(nxt, a, S, q.c0, q.c1, r0, r1);   // a queued triangle's normal follows
                  if (p0) bil_push(qu, a, 0, f);
                  if (p1) bil_push(qu, a, 1, f);
              });
        const int nq = qu.count[f];
        for (int e = wave; e < nq; e += kTileBlock / kWave) {
            const int a = qu.entry[e] >> 1, k = qu.entry[e] & 1;
            const V3 r = bil_fallback_wave<R, NT>(cur, a, k, W, S, ka, kb);
            if (lane == 0) {
                *bil_at(nxt, a, S, 6 + 3 * k) = r.x;
                *bil_at(nxt, a, S, 7 + 3 * k) = r.y;
                *bil_at(nxt, a, S, 8 + 3 * k) = r.z;
            }
        }
        __syncthreads();
        float4 *t = const_cast<float4 *>(cur);
        cur = nxt;
        nxt = t;
    }

    // last sweep (or the copy when F = 0): the tile itself, to global memory
    auto emit = [&](int ty, int tx, int a, const BilQuad &g, int fl, int2 t, const V3 &r0,
                    const V3 &r1, bool p0, bool p1) {
        const int qy = qy0 + ty, qx = qx0 + tx;
        if (part != 0 || qy >= Mq || qx >= Nq) return;   // the quad's first lane stores
        const size_t q = (size_t)qy * Nq + qx;
        const V3 r[2] = {r0, r1};
        const bool pend[2] = {p0, p1};
        NT v[6];
        NT raw[6];                           // raw normals as stored (FromPts)
        if constexpr (FromPts) {
            // centroids as staged; a missing corner's and its normal are the
            // canonical NaN, and the rest (a triangle of no area) is computed
            // again, as everything is when nothing was staged
            const float nan = qnan();
            V3 c0{nan, nan, nan}, c1 = c0, n0 = c0, n1 = c0;
            if (fl & kBilUsable) c0 = g.c0;
            if (fl & (2 * kBilUsable)) c1 = g.c1;
            const bool odd = !(fl & (kBilUsable | kBilCanonical)) || !(fl & (2 * (kBilUsable | kBilCanonical)));
            if (F == 0 || odd) quad_geom_at(pts, Nq + 1, qy, qx, c0, n0, c1, n1);
            cen_out[6 * q + 0] = c0.x; cen_out[6 * q + 1] = c0.y; cen_out[6 * q + 2] = c0.z;
            cen_out[6 * q + 3] = c1.x; cen_out[6 * q + 4] = c1.y; cen_out[6 * q + 5] = c1.z;
            st_f(&raw[0], n0.x); st_f(&raw[1], n0.y); st_f(&raw[2], n0.z);
            st_f(&raw[3], n1.x); st_f(&raw[4], n1.y); st_f(&raw[5], n1.z);
        }
        // a triangle's normal as it came in: canonical NaN, or read again
        auto keep = [&](int k) {
            if constexpr (FromPts) {
#pragma unroll
                for (int i = 0; i < 3; ++i) v[3 * k + i] = raw[3 * k + i];
            } else {
                st_f(&v[3 * k], qnan());
                v[3 * k + 1] = v[3 * k];
                v[3 * k + 2] = v[3 * k];
                if (!(fl & (kBilCanonical << k))) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) v[3 * k + i] = nin[6 * q + 3 * k + i];
                }
            }
        };
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (pend[k]) {                 // queued: written after the sweep
                bil_push(qu, a, k, F);
            } else if (fl & (kBilUsable << k)) {
                st_f(&v[3 * k], r[k].x); st_f(&v[3 * k + 1], r[k].y); st_f(&v[3 * k + 2], r[k].z);
            } else {                       // missing triangle (or F = 0): input bits unchanged
                keep(k);
            }
        }
        // streaming stores (float32 normals): they write partial lines, about
        // 2 MB more per launch on a 480x640 frame, but the whole path gains
        // 2.4 us per frame.  A queued triangle is written after the sweep.
        const int t0 = t.x, t1 = t.y;
        if (!(pend[0] | pend[1])) {
#pragma unroll
            for (int i = 0; i < 6; ++i) bil_store(&nout[6 * q + i], v[i]);
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (!pend[0]) bil_store(&nout[6 * q + i], v[i]);
                if (!pend[1]) bil_store(&nout[6 * q + 3 + i], v[3 + i]);
            }
        }
        if (t0 >= 0 && !pend[0]) {
#pragma unroll
            for (int i = 0; i < 3; ++i) bil_store(&nT[3 * (size_t)t0 + i], v[i]);
        }
        if (t1 >= 0 && !pend[1]) {
#pragma unroll
            for (int i = 0; i < 3; ++i) bil_store(&nT[3 * (size_t)t1 + i], v[3 + i]);
        }
    };
    if (F > 0) {
        sweep(halo, TQH, TQW, t_index, emit);
    } else {
        const DivBy byTQW(TQW);
        const V3 z{0.f, 0.f, 0.f};
        for (int idx = slot; idx < TQH * TQW; idx += waves ? kWave : kTileBlock / QL) {
            const int ty = byTQW.div(idx), tx = idx - ty * TQW;
            emit(ty, tx, 0, BilQuad{z, z, z, z}, 0, t_index(ty, tx), z, z, false, false);
        }
    }
    if (F > 0) {
        // the queued triangles of the last sweep, one wave each (the sweep
        // ended with a barrier)
        const int nq = qu.count[F];
        for (int e = wave; e < nq; e += kTileBlock / kWave) {
            const int a = qu.entry[e] >> 1, k = qu.entry[e] & 1;
            const V3 r = bil_fallback_wave<R, NT>(cur, a, k, W, S, ka, kb);
            if (lane == 0) {
                const int ly = a / W, lx = a - ly * W;
                const size_t q = (size_t)(oy + ly) * Nq + (ox + lx);
                NT v[3];
                st_f(&v[0], r.x); st_f(&v[1], r.y); st_f(&v[2], r.z);
#pragma unroll
                for (int i = 0; i < 3; ++i) bil_store(&nout[6 * q + 3 * k + i], v[i]);
                const int2 tt = t_index(ly - halo, lx - halo);
                const int t = k ? tt.y : tt.x;
                if (t >= 0) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) bil_store(&nT[3 * (size_t)t + i], v[i]);
                }
            }
        }
    }
    __syncthreads();                 // LDS is reused by the next tile
}

}  // namespace pl
