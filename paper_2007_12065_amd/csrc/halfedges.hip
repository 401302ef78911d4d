// Half-edges of a user-provided mesh (Sec. 4.3) through a device hash table.
//
// Every half-edge (a, b) of T (3t + j runs from vertex j to vertex j+1 mod 3
// of triangle t) is keyed by its ordered point pair; its twin is the
// half-edge keyed (b, a).  Edges shared by more than two triangles keep the
// first pair (the paper's option 1): a half-edge is paired only if it has
// the lowest index among the half-edges with its key, and then with the
// lowest-index half-edge keyed (b, a).  Half-edges from a point to itself
// are never paired.
//
// Both ways below key an edge by its undirected point pair (lo, hi), lo < hi,
// and keep per key the first half-edge of each direction (lo -> hi and
// hi -> lo); a half-edge that is the first of its direction then takes the
// other direction's first, if any.  Minima are order-free, so the output is
// deterministic whatever the order of the threads.
//
// Partitioned (up to kHeMaxBuckets buckets, 5.6 M triangles): the keys are
// dealt to buckets by hash and every bucket is solved in the LDS of one
// workgroup, so the common case has no atomics on global memory.
//   k_he_count     per chunk of kHeChunk half-edges: how many fall in each
//                  bucket (LDS histogram), one row per chunk
//   k_he_offsets   per bucket, over the chunks: where each chunk's entries
//                  start in the bucket's region (a scan), and the total
//   k_he_scatter   every half-edge's key and index into its bucket's region
//                  (kHeRegion entries), staged in LDS in bucket order first
//                  so that each chunk writes one contiguous run per bucket;
//                  half-edges past a full region go to an overflow list, which
//                  only the buckets that overflowed read
//   k_he_solve     one workgroup per bucket: an LDS hash table of the
//                  bucket's keys (compare-and-swap on the key, atomic min of
//                  each direction's first index), then each entry takes its
//                  twin from the slot it found.  A bucket of more distinct
//                  keys than its LDS table has slots (only inputs built
//                  against the hash hold one) is solved by its workgroup in
//                  a table of its own in global memory
// A chunk past the mesh (a buffer may hold more triangles than |T|) is left by
// its workgroup at once: one triangle in a buffer of 5.5 M takes 145 us (370
// when its chunks were read and scanned, 147 before loads were kept in flight).
// All of a thread's loads of a pass are issued before the first is used (eight
// dependent rounds of memory latency were most of a pass before).  On 533 k
// triangles in a buffer for 612 k, count / offsets / scatter / solve take
// 4.9 / 4.9 / 12.8 / 20.2 us (8.2 / 6.0 / 22.9 / 30.0, and 4.7 for a launch that
// looked for full tables, before), 43.7 us a call (68.1); streaming stores of
// the twins: solve 47 us; 256 threads: 24 us.
// Buckets: the power of two nearest above 3 cap / kHeBucketMean; a
// bucket's keys are the top bits of the hash, its LDS slot the low bits.
//
// Global table (larger meshes): a slot (16 bytes, one cache line holds
// eight) keeps the key and both first indices.  Three launches:
//   k_he_clear    every slot of the table empty (a kernel, so the sequence
//                 can be captured into a graph)
//   k_he_insert   one thread per half-edge: it claims its edge's
//                 slot (64-bit compare-and-swap, linear probing), lowers its
//                 direction's value to its index (atomic min, in the same
//                 line as the key), so every slot ends with the first index
//                 of each direction whatever the order of the threads, and
//                 records the slot it found
//   k_he_lookup   one thread per half-edge: a half-edge that is the first of
//                 its direction takes the other direction's value from its
//                 recorded slot (one read, no probing)
// The table has 4 cap slots (rounded up to 64), at least 4/3 as many as
// half-edges (load <= 3/4), so every probe sequence meets its key or an
// empty slot.  Hash values are reduced to a slot by a 64 x 64-bit high
// product, which needs no power-of-two size.  Triangles are dealt to
// workgroups in contiguous runs per XCD, so the two triangles of an edge in
// an organized mesh, a row apart, usually run under the same L2.
//
// Probing reads a slot before it tries an atomic on it: only an empty slot
// or the edge's own key is worth a compare-and-swap.
#include "he.h"
#include "tuning.h"

#include <algorithm>
#include <climits>

namespace pl {

namespace {

constexpr int kHeBlock = 256;
constexpr unsigned long long kEmpty = ~0ull;   // (-1, -1): lo == hi, never inserted

struct alignas(16) HeSlot {
    unsigned long long key;
    int fwd, bwd;                    // first half-edge lo -> hi, hi -> lo
};

__device__ __forceinline__ unsigned long long he_key(int lo, int hi) {
    return ((unsigned long long)(unsigned)lo << 32) | (unsigned)hi;
}

// The 64-bit finaliser of MurmurHash3 (Appleby): every input bit reaches
// every output bit.
__device__ __forceinline__ unsigned long long he_mix(unsigned long long k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return k;
}

// hash in [0, 2^64) scaled to [0, slots)
__device__ __forceinline__ unsigned long long he_slot(unsigned long long key,
                                                      unsigned long long slots) {
    return __umul64hi(he_mix(key), slots);
}

size_t table_slots(int cap) {
    const size_t s = (4 * (size_t)cap + 63) / 64 * 64;
    return s < 256 ? 256 : s;
}

__global__ __launch_bounds__(kHeBlock) void k_he_clear(HeSlot *__restrict__ tab, size_t slots) {
    for (size_t i = (size_t)blockIdx.x * kHeBlock + threadIdx.x; i < slots;
         i += (size_t)gridDim.x * kHeBlock) {
        HeSlot e;
        e.key = kEmpty;
        e.fwd = INT_MAX;
        e.bwd = INT_MAX;
        tab[i] = e;
    }
}

__global__ __launch_bounds__(kHeBlock) void k_he_insert(const int32_t *__restrict__ tris,
                                                        const int32_t *__restrict__ n_tri,
                                                        int cap, HeSlot *__restrict__ tab,
                                                        unsigned long long slots,
                                                        int32_t *__restrict__ hslot) {
    // one thread per half-edge: the three of a triangle run side by side
    const int n = 3 * min(max(*n_tri, 0), cap);
    const int h = xcd_remap((int)blockIdx.x, (int)gridDim.x) * kHeBlock + (int)threadIdx.x;
    if (h >= n) return;
    const int t = h / 3, j = h - 3 * t;
    const int a = tris[h], b = tris[3 * t + (j == 2 ? 0 : j + 1)];
    int found = -1;
    if (a != b) {
        const int lo = min(a, b), hi = max(a, b);
        const unsigned long long key = he_key(lo, hi);
        unsigned long long slot = he_slot(key, slots);
        for (;;) {
            // a plain read first: only an empty slot or the key itself is
            // worth an atomic
            const unsigned long long seen = __hip_atomic_load(&tab[slot].key, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long prev =
                seen == kEmpty ? atomicCAS(&tab[slot].key, kEmpty, key) : seen;
            if (prev == kEmpty || prev == key) {
                atomicMin(a < b ? &tab[slot].fwd : &tab[slot].bwd, h);
                found = (int)slot;
                break;
            }
            slot = slot + 1 == slots ? 0 : slot + 1;
        }
    }
    hslot[h] = found;
}

__global__ __launch_bounds__(kHeBlock) void k_he_lookup(const int32_t *__restrict__ tris,
                                                        const int32_t *__restrict__ n_tri,
                                                        int cap, const HeSlot *__restrict__ tab,
                                                        const int32_t *__restrict__ hslot,
                                                        int32_t *__restrict__ he) {
    const int n = 3 * min(max(*n_tri, 0), cap);
    const int h = xcd_remap((int)blockIdx.x, (int)gridDim.x) * kHeBlock + (int)threadIdx.x;
    if (h >= n) return;
    const int sl = hslot[h];
    int twin = -1;
    if (sl >= 0) {
        const int t = h / 3, j = h - 3 * t;
        const int a = tris[h], b = tris[3 * t + (j == 2 ? 0 : j + 1)];
        const int2 f = *reinterpret_cast<const int2 *>(&tab[sl].fwd);
        const int own = a < b ? f.x : f.y, other = a < b ? f.y : f.x;
        if (own == h && other != INT_MAX) twin = other;
    }
    he[h] = twin;
}

// ---------------------------------------------------------------------------
// Partitioned way
// ---------------------------------------------------------------------------

constexpr int kHePartBlock = 1024;        // threads of the partitioned way's kernels
constexpr int kHeChunk = 4096;            // half-edges per row of the histogram
constexpr int kHePer = kHeChunk / kHePartBlock;   // half-edges of a chunk per thread
constexpr int kHeBucketMean = 2048;       // mean entries per bucket at n = 3 cap, at most
constexpr int kHeRegion = 3072;           // entries a bucket's region holds
constexpr int kHeSolvePer = kHeRegion / kHePartBlock;   // of them per thread
constexpr int kHeLdsSlots = 4096;         // LDS table of a bucket (64 KB)
constexpr int kHeMaxBuckets = 8192;       // LDS histogram of a chunk (32 KB)
constexpr int kHeScanBuckets = 16;        // buckets per offsets workgroup
constexpr int kHeScanParts = 64;          // parts splitting the chunks of a bucket
constexpr int kHeScanBlock = kHeScanBuckets * kHeScanParts;

// A half-edge in a bucket's region: its key's points and h | 2^31 when it
// runs hi -> lo.  Kept together: a chunk's run of a bucket, a few entries
// long, is then one piece of memory instead of two.
struct HeEntry {
    int lo, hi, hd;
};

int bucket_bits(int cap) {
    const long long want = (3LL * cap + kHeBucketMean - 1) / kHeBucketMean;
    int lg = 0;
    while ((1LL << lg) < want) ++lg;
    return lg;
}

// the half-edge h of T: from tris[h] to the next vertex of its triangle
__device__ __forceinline__ void he_ends(const int32_t *__restrict__ tris, int h, int &a, int &b) {
    const int t = h / 3, j = h - 3 * t;
    a = tris[h];
    b = tris[3 * t + (j == 2 ? 0 : j + 1)];
}

__device__ __forceinline__ int he_bucket(unsigned long long mix, int lg) {
    return lg == 0 ? 0 : (int)(mix >> (64 - lg));
}

// The half-edges of the mesh.
__device__ __forceinline__ int he_number(const int32_t *__restrict__ n_tri, int cap) {
    return 3 * min(max(*n_tri, 0), cap);
}

// A thread's half-edges base + i kHePartBlock + threadIdx.x of its chunk, all
// loads in flight at once.  Rows from n on hold whatever the buffer does, or
// (0, 0) past the capacity: the caller leaves them out by their index.
__device__ __forceinline__ void he_chunk_ends(const int32_t *__restrict__ tris, int cap, int base,
                                              int (&a)[kHePer], int (&b)[kHePer]) {
#pragma unroll
    for (int i = 0; i < kHePer; ++i) {
        const int h = base + i * kHePartBlock + (int)threadIdx.x;
        a[i] = 0;
        b[i] = 0;
        if (h < 3 * cap) he_ends(tris, h, a[i], b[i]);
    }
}

__global__ __launch_bounds__(kHePartBlock) void k_he_count(const int32_t *__restrict__ tris,
                                                           const int32_t *__restrict__ n_tri,
                                                           int cap, int lg,
                                                           int32_t *__restrict__ hist_out) {
    extern __shared__ int hist[];
    const int nb = 1 << lg;
    const int base = (int)blockIdx.x * kHeChunk, n = he_number(n_tri, cap);
    int32_t *row = hist_out + (size_t)blockIdx.x * nb;
    if (base >= n) {                     // a chunk past the mesh: no counts
        for (int i = threadIdx.x; i < nb; i += kHePartBlock) row[i] = 0;
        return;
    }
    int a[kHePer], b[kHePer];
    he_chunk_ends(tris, cap, base, a, b);
    for (int i = threadIdx.x; i < nb; i += kHePartBlock) hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kHePer; ++i) {
        const int h = base + i * kHePartBlock + (int)threadIdx.x;
        if (h < n && a[i] != b[i])
            atomicAdd(&hist[he_bucket(he_mix(he_key(min(a[i], b[i]), max(a[i], b[i]))), lg)], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += kHePartBlock) row[i] = hist[i];
}

// 16 buckets per workgroup of 1024 threads: lane l of wave w takes bucket
// l mod 16 and part 4 w + l / 16 of the chunks (kHeScanParts parts); each
// part sums its chunks, the parts are scanned (across the wave's four, then
// over the waves' sums in LDS), then each part writes its chunks' starts.
// Also clears the control words.
__global__ __launch_bounds__(kHeScanBlock) void k_he_offsets(
    const int32_t *__restrict__ hist, int chunks, int lg, int32_t *__restrict__ start,
    int32_t *__restrict__ total, int32_t *__restrict__ ctl) {
    constexpr int kWaves = kHeScanBlock / kWave;
    __shared__ int wave_total[kWaves][kHeScanBuckets];
    const int nb = 1 << lg;
    const int lane = (int)threadIdx.x & (kWave - 1), wave = (int)threadIdx.x / kWave;
    const int col = lane % kHeScanBuckets, part = (int)threadIdx.x / kHeScanBuckets;
    const int b = (int)blockIdx.x * kHeScanBuckets + col;
    if (blockIdx.x == 0 && threadIdx.x < 2) ctl[threadIdx.x] = 0;
    const int per = (chunks + kHeScanParts - 1) / kHeScanParts;
    const int c0 = part * per, c1 = min(c0 + per, chunks);
    int sum = 0;
    if (b < nb) {
#pragma unroll 8
        for (int c = c0; c < c1; ++c) sum += hist[(size_t)c * nb + b];
    }
    int incl = sum;                      // over the wave's parts of this bucket
#pragma unroll
    for (int d = kHeScanBuckets; d < kWave; d <<= 1) {
        const int y = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += y;
    }
    if (lane >= kWave - kHeScanBuckets) wave_total[wave][col] = incl;
    __syncthreads();
    int run = incl - sum, all = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const int v = wave_total[k][col];
        run += k < wave ? v : 0;
        all += v;
    }
    if (b >= nb) return;
    if (part == 0) total[b] = all;
#pragma unroll 8
    for (int c = c0; c < c1; ++c) {
        const int v = hist[(size_t)c * nb + b];
        start[(size_t)c * nb + b] = run;
        run += v;
    }
}

// Every half-edge's entry into its bucket's region.  The chunk's entries are first placed in LDS in bucket order (the chunk's
// counts, scanned), then written out: the chunk's entries of one bucket are
// one contiguous run of the bucket's region, written by consecutive lanes.
// LDS: the chunk's keys and entries (12 kHeChunk bytes), then per bucket a
// cursor and what takes a place in LDS to a place in the bucket's region
// (2 x 4 nb bytes).
__device__ __forceinline__ int block_exclusive_scan(int x, int *tmp, int *all) {
    const int lane = (int)threadIdx.x & (kWave - 1), w = (int)threadIdx.x / kWave;
    const int incl = wave_inclusive_scan(x);
    if (lane == kWave - 1) tmp[w] = incl;
    __syncthreads();
    int before = 0, sum = 0;
#pragma unroll
    for (int k = 0; k < kHePartBlock / kWave; ++k) {
        const int v = tmp[k];
        before += k < w ? v : 0;
        sum += v;
    }
    *all = sum;
    return before + incl - x;
}

__global__ __launch_bounds__(kHePartBlock) void k_he_scatter(
    const int32_t *__restrict__ tris, const int32_t *__restrict__ n_tri, int cap, int lg,
    const int32_t *__restrict__ hist, const int32_t *__restrict__ start,
    HeEntry *__restrict__ region, int32_t *__restrict__ ctl, int32_t *__restrict__ over,
    int32_t *__restrict__ he) {
    extern __shared__ unsigned long long lds_u64[];
    __shared__ int tmp[kHePartBlock / kWave];
    const int nb = 1 << lg;
    unsigned long long *skey = lds_u64;                                  // [kHeChunk]
    int *shd = reinterpret_cast<int *>(skey + kHeChunk);                 // [kHeChunk]
    int *lcur = shd + kHeChunk;                                          // [nb]
    int *ldelta = lcur + nb;                                             // [nb]
    const int base = (int)blockIdx.x * kHeChunk, n = he_number(n_tri, cap);
    if (base >= n) return;               // a chunk past the mesh
    const int32_t *crow = hist + (size_t)blockIdx.x * nb;
    const int32_t *srow = start + (size_t)blockIdx.x * nb;
    int a[kHePer], b[kHePer];
    he_chunk_ends(tris, cap, base, a, b);
    // the chunk's starts per bucket: each thread scans `per` consecutive
    // counts (nb < kHePartBlock: one or none)
    const int per = (nb + kHePartBlock - 1) / kHePartBlock;
    const int b0 = (int)threadIdx.x * per;
    int own = 0;
    for (int k = 0; k < per && b0 + k < nb; ++k) own += crow[b0 + k];
    int m;                                       // entries of the chunk
    int run = block_exclusive_scan(own, tmp, &m);
    for (int k = 0; k < per && b0 + k < nb; ++k) {
        lcur[b0 + k] = run;
        ldelta[b0 + k] = srow[b0 + k] - run;
        run += crow[b0 + k];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kHePer; ++i) {
        const int h = base + i * kHePartBlock + (int)threadIdx.x;
        if (h >= n) continue;
        if (a[i] == b[i]) {
            he[h] = -1;                  // from a point to itself: never paired
            continue;
        }
        const unsigned long long key = he_key(min(a[i], b[i]), max(a[i], b[i]));
        const int lp = atomicAdd(&lcur[he_bucket(he_mix(key), lg)], 1);
        skey[lp] = key;
        shd[lp] = a[i] < b[i] ? h : (h | INT_MIN);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kHePer; ++k) {
        const int i = k * kHePartBlock + (int)threadIdx.x;
        if (i >= m) continue;
        const unsigned long long key = skey[i];
        const int bk = he_bucket(he_mix(key), lg);
        const int pos = i + ldelta[bk];
        const HeEntry e{(int)(key >> 32), (int)key, shd[i]};
        if (pos < kHeRegion)
            region[(size_t)bk * kHeRegion + pos] = e;
        else
            over[atomicAdd(&ctl[0], 1)] = e.hd & INT_MAX;
    }
}

struct HeLdsTable {
    unsigned long long key[kHeLdsSlots];
    int2 first[kHeLdsSlots];             // first half-edge lo -> hi, hi -> lo
};

// Claims the key's slot and lowers its direction's first index: the slot, or
// -1 when the table is full of other keys.
__device__ __forceinline__ int he_lds_insert(HeLdsTable &t, unsigned long long key, int hd) {
    int slot = (int)(he_mix(key) & (kHeLdsSlots - 1));
    for (int p = 0; p < kHeLdsSlots; ++p) {
        const unsigned long long prev = atomicCAS(&t.key[slot], kEmpty, key);
        if (prev == kEmpty || prev == key) {
            atomicMin(hd < 0 ? &t.first[slot].y : &t.first[slot].x, hd & INT_MAX);
            return slot;
        }
        slot = (slot + 1) & (kHeLdsSlots - 1);
    }
    return -1;
}

// The slot of a key; -1 if it is not in the table (it always is once every
// insert succeeded: the probe is bounded all the same).
__device__ __forceinline__ int he_lds_find(const HeLdsTable &t, unsigned long long key) {
    int slot = (int)(he_mix(key) & (kHeLdsSlots - 1));
    for (int p = 0; p < kHeLdsSlots; ++p) {
        if (t.key[slot] == key) return slot;
        slot = (slot + 1) & (kHeLdsSlots - 1);
    }
    return -1;
}

// The twin of entry hd from its slot's first indices.
__device__ __forceinline__ int he_twin(int2 f, int hd) {
    const int own = hd < 0 ? f.y : f.x, other = hd < 0 ? f.x : f.y;
    return own == (hd & INT_MAX) && other != INT_MAX ? other : -1;
}

// A bucket with more distinct keys than the LDS table has slots, by its
// workgroup alone: its half-edges (the first m in its region, then its own of
// the overflow list's no) through a hash table of directed edges in global
// memory.  A slot is the first half-edge of its edge so far (-1: empty), whose
// points T holds: 4 bytes, of `slots` more than there are half-edges.  All
// accesses are atomic (they meet in L2).
__device__ void he_bucket_global(const int32_t *__restrict__ tris, const HeEntry *__restrict__ r, int m,
                                 const int32_t *__restrict__ over, int no, int bk, int lg, int *tab,
                                 int slots, int32_t *__restrict__ he) {
    for (int i = threadIdx.x; i < slots; i += kHePartBlock)
        __hip_atomic_store(&tab[i], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    // the i-th half-edge, from a to b; false for another bucket's
    auto take = [&](int i, int &h, int &a, int &b) {
        h = i < m ? r[i].hd & INT_MAX : over[i - m];
        he_ends(tris, h, a, b);
        return i < m || he_bucket(he_mix(he_key(min(a, b), max(a, b))), lg) == bk;
    };
    // the slot of a -> b, or the empty one where it belongs: the bucket's keys
    // share the mix's top bits, so the rest spreads them, either direction over
    // a half of its own; `v`: what it held
    auto find = [&](int a, int b, int &v) {
        unsigned long long x = he_mix(he_key(min(a, b), max(a, b))) << lg;
        if (a > b) x ^= 1ull << 63;
        int slot = (int)__umul64hi(x, (unsigned long long)slots);
        for (int p = 0; p < slots; ++p) {                     // a free slot is always left
            v = __hip_atomic_load(&tab[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v < 0) return slot;
            int c, d;
            he_ends(tris, v, c, d);
            if (c == a && d == b) return slot;
            slot = slot + 1 == slots ? 0 : slot + 1;
        }
        return -1;
    };
    for (int i = threadIdx.x; i < m + no; i += kHePartBlock) {
        int h, a, b;
        if (!take(i, h, a, b)) continue;
        for (;;) {
            int v;
            const int slot = find(a, b, v);
            if (slot < 0) break;
            if (v >= 0) {
                atomicMin(&tab[slot], h);
                break;
            }
            if (atomicCAS(&tab[slot], -1, h) == -1) break;    // else another took it: look again
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < m + no; i += kHePartBlock) {
        int h, a, b, own, other;
        if (!take(i, h, a, b)) continue;
        const bool in = find(a, b, own) >= 0 && own == h;
        he[h] = in && find(b, a, other) >= 0 ? other : -1;
    }
}

// One workgroup per bucket (two per CU, by the LDS of their tables).  Bound by
// the twins' scattered 4-byte writes (22.6 us for 1.6 M half-edges in random
// order, 9.4 without them; four workgroups per CU change nothing).  A thread holds its entries of the region in
// registers, loaded at once, and the slots they found: the twins then need
// neither a second read of the entries nor a second probe.
// ctl: [0] half-edges on the overflow list, [1] slots taken of the global table
// `tab`, whose 4 cap slots suffice: a bucket takes 4/3 of its half-edges, and all
// buckets together hold at most 3 cap.
__global__ __launch_bounds__(kHePartBlock) void k_he_solve(
    const int32_t *__restrict__ tris, const HeEntry *__restrict__ region,
    const int32_t *__restrict__ total, int32_t *ctl, const int32_t *__restrict__ over, int lg, int *tab,
    int32_t *__restrict__ he) {
    __shared__ HeLdsTable t;
    __shared__ int full, tab_base;
    const int bk = (int)blockIdx.x;
    const int tot = total[bk], m = min(tot, kHeRegion);
    // a bucket that overflowed also takes its entries from the overflow list
    const int no = tot > kHeRegion ? ctl[0] : 0;
    const HeEntry *r = region + (size_t)bk * kHeRegion;
    HeEntry e[kHeSolvePer];
    int slot[kHeSolvePer];
#pragma unroll
    for (int k = 0; k < kHeSolvePer; ++k) {
        const int i = k * kHePartBlock + (int)threadIdx.x;
        e[k] = i < m ? r[i] : HeEntry{0, 0, 0};
    }
    for (int i = threadIdx.x; i < kHeLdsSlots; i += kHePartBlock) {
        t.key[i] = kEmpty;
        t.first[i] = make_int2(INT_MAX, INT_MAX);
    }
    if (threadIdx.x == 0) full = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kHeSolvePer; ++k) {
        slot[k] = -1;
        if (k * kHePartBlock + (int)threadIdx.x < m) {
            slot[k] = he_lds_insert(t, he_key(e[k].lo, e[k].hi), e[k].hd);
            if (slot[k] < 0) full = 1;
        }
    }
    for (int i = threadIdx.x; i < no; i += kHePartBlock) {
        const int h = over[i];
        int a, b;
        he_ends(tris, h, a, b);
        const unsigned long long k = he_key(min(a, b), max(a, b));
        if (he_bucket(he_mix(k), lg) == bk && he_lds_insert(t, k, a < b ? h : (h | INT_MIN)) < 0) full = 1;
    }
    __syncthreads();
    if (full) {
        if (threadIdx.x == 0) tab_base = atomicAdd(&ctl[1], tot + tot / 3);
        __syncthreads();
        he_bucket_global(tris, r, m, over, no, bk, lg, tab + tab_base, tot + tot / 3, he);
        return;
    }
#pragma unroll
    for (int k = 0; k < kHeSolvePer; ++k)
        if (slot[k] >= 0) he[e[k].hd & INT_MAX] = he_twin(t.first[slot[k]], e[k].hd);
    for (int i = threadIdx.x; i < no; i += kHePartBlock) {
        const int h = over[i];
        int a, b;
        he_ends(tris, h, a, b);
        const unsigned long long k = he_key(min(a, b), max(a, b));
        if (he_bucket(he_mix(k), lg) != bk) continue;
        const int s = he_lds_find(t, k);
        if (s >= 0) he[h] = he_twin(t.first[s], a < b ? h : (h | INT_MIN));
    }
}

// Workspace of the partitioned way: the histogram rows and their starts,
// the bucket totals, two control words, the regions, the overflow list (a
// half-edge's index, 4 bytes; its points are T's) and the global table of
// buckets that outgrow their LDS table.
struct HeParts {
    int lg, nb, chunks;
    size_t hist, start, total, ctl, region, over, tab, end;
};

HeParts he_parts(int cap) {
    HeParts p{};
    p.lg = bucket_bits(cap);
    p.nb = 1 << p.lg;
    p.chunks = (int)((3 * (size_t)cap + kHeChunk - 1) / kHeChunk);
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += align_up(bytes, 256); return at; };
    p.hist = take(4 * (size_t)p.chunks * p.nb);
    p.start = take(4 * (size_t)p.chunks * p.nb);
    p.total = take(4 * (size_t)p.nb);
    p.ctl = take(8);
    p.region = take(sizeof(HeEntry) * (size_t)p.nb * kHeRegion);
    p.over = take(4 * 3 * (size_t)cap);
    p.tab = take(4 * 4 * (size_t)cap);
    p.end = o;
    return p;
}

bool partitioned(int cap) { return (1LL << bucket_bits(cap)) <= kHeMaxBuckets; }

}  // namespace

size_t user_halfedges_workspace(int cap) {
    if (partitioned(cap)) return he_parts(cap).end;
    return align_up(sizeof(HeSlot) * table_slots(cap), 256) + align_up(12 * (size_t)cap, 256);
}

pl_status launch_user_halfedges(const int32_t *tris, const int32_t *n_tri, int cap, int32_t *he,
                                void *ws, hipStream_t s) {
    if (cap == 0) return PL_OK;
    auto *w = static_cast<uint8_t *>(ws);
    if (partitioned(cap)) {
        const HeParts p = he_parts(cap);
        auto *hist = reinterpret_cast<int32_t *>(w + p.hist);
        auto *start = reinterpret_cast<int32_t *>(w + p.start);
        auto *total = reinterpret_cast<int32_t *>(w + p.total);
        auto *ctl = reinterpret_cast<int32_t *>(w + p.ctl);
        auto *region = reinterpret_cast<HeEntry *>(w + p.region);
        auto *over = reinterpret_cast<int32_t *>(w + p.over);
        const size_t hist_lds = 4 * (size_t)p.nb;
        k_he_count<<<p.chunks, kHePartBlock, hist_lds, s>>>(tris, n_tri, cap, p.lg, hist);
        if (pl_status st = hip_check(hipGetLastError(), "k_he_count")) return st;
        k_he_offsets<<<(p.nb + kHeScanBuckets - 1) / kHeScanBuckets, kHeScanBlock, 0, s>>>(
            hist, p.chunks, p.lg, start, total, ctl);
        if (pl_status st = hip_check(hipGetLastError(), "k_he_offsets")) return st;
        const size_t scatter_lds = 12 * (size_t)kHeChunk + 8 * (size_t)p.nb;
        if (pl_status st = allow_lds((const void *)k_he_scatter, scatter_lds)) return st;
        k_he_scatter<<<p.chunks, kHePartBlock, scatter_lds, s>>>(tris, n_tri, cap, p.lg, hist, start,
                                                                 region, ctl, over, he);
        if (pl_status st = hip_check(hipGetLastError(), "k_he_scatter")) return st;
        k_he_solve<<<p.nb, kHePartBlock, 0, s>>>(tris, region, total, ctl, over, p.lg,
                                                 reinterpret_cast<int *>(w + p.tab), he);
        return hip_check(hipGetLastError(), "k_he_solve");
    }
    const size_t slots = table_slots(cap);
    auto *tab = static_cast<HeSlot *>(ws);
    auto *hslot = reinterpret_cast<int32_t *>(w + align_up(sizeof(HeSlot) * slots, 256));
    const int clear_grid = (int)std::min<size_t>(4096, (slots + kHeBlock - 1) / kHeBlock);
    k_he_clear<<<clear_grid, kHeBlock, 0, s>>>(tab, slots);
    if (pl_status st = hip_check(hipGetLastError(), "k_he_clear")) return st;
    const int grid = (int)((3 * (size_t)cap + kHeBlock - 1) / kHeBlock);
    k_he_insert<<<grid, kHeBlock, 0, s>>>(tris, n_tri, cap, tab, slots, hslot);
    if (pl_status st = hip_check(hipGetLastError(), "k_he_insert")) return st;
    k_he_lookup<<<grid, kHeBlock, 0, s>>>(tris, n_tri, cap, tab, hslot, he);
    return hip_check(hipGetLastError(), "k_he_lookup");
}

}  // namespace pl
