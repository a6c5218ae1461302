// Small calls: all pairs instead of a grid.  (Kernels and their launch, compiled
// with hca_batch.hip.)
//
// A call of a few thousand points through the grid is some twenty to thirty
// launches of a few microseconds each, with one or two host round trips
// between them; the work in them hardly counts.  Here a call is five launches
// (six past eight axes) and one wait: the bounding box, all pair distances as
// a bit matrix with the neighbour counts, a first forest over the core points,
// the remaining unions with the border points' owners, and the labels.  The
// n^2 pair tests are cheap at this size (2-D, 10k points: 1e8 tests, 29 us;
// past eight axes the byte planes' matrix tiles take them: 27 axes, 5045
// points 14 us).  Bound: launches and the passes of a block over all points.
// 340 points x 16 axes 513 -> 49 us, 5045 x 27 785 -> 90, 10k x 2 162 -> 128.
//
// The box is not needed to lay anything out, only to tell which arithmetic is
// exact and which data the general path would refuse: the kernels read the
// box's partial extrema themselves, and the last one reports to the host.
#include <algorithm>

#include "hca_device.h"
#include "hca_kernels.h"

namespace hca {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

typedef __attribute__((address_space(4))) int32_t ConstInt;

constexpr uint32_t kSmallSlice = 256;          // candidates per wave of the pair tests
constexpr int kSmallBlock = 1024;
constexpr int kSmallWaves = kSmallBlock / kWave;

// ---------------------------------------------------------------------------
// Box partials [boxes][2][d]; counters cleared, every point its own parent.
// A thread keeps to one axis: the elements are taken in steps of a multiple
// of d.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_small_box(SmallArgs A)
{
    __shared__ int32_t s_lo[kBlock], s_hi[kBlock];
    const uint32_t d = (uint32_t)A.d, per = kBlock / d * d, t = threadIdx.x;
    for (uint32_t i = blockIdx.x * kBlock + t; i < A.np; i += gridDim.x * kBlock) {
        st_agent32(A.cnt + i, 0u);
        A.parent[i] = i;
    }
    int32_t lo = INT32_MAX, hi = INT32_MIN;
    const uint32_t total = A.n * d;
    if (t < per) {
        const uint32_t step = gridDim.x * per;
        uint32_t e = blockIdx.x * per + t;
        for (; e + 3 * step < total; e += 4 * step) {
            const int32_t v0 = A.pts[e], v1 = A.pts[e + step], v2 = A.pts[e + 2 * step], v3 = A.pts[e + 3 * step];
            lo = min(min(lo, min(v0, v1)), min(v2, v3));
            hi = max(max(hi, max(v0, v1)), max(v2, v3));
        }
        for (; e < total; e += step) {
            const int32_t v = A.pts[e];
            lo = min(lo, v);
            hi = max(hi, v);
        }
    }
    s_lo[t] = lo;
    s_hi[t] = hi;
    __syncthreads();
    if (t < d) {
        for (uint32_t k = t + d; k < per; k += d) {
            lo = min(lo, s_lo[k]);
            hi = max(hi, s_hi[k]);
        }
        A.partial[blockIdx.x * 2 * d + t] = lo;
        A.partial[blockIdx.x * 2 * d + d + t] = hi;
    }
}

// The box of the call from its partials, into s_box[0, d) and s_box[d, 2 d)
// (whole block; followed by a barrier).
__device__ __forceinline__ void small_box(const SmallArgs &A, int32_t *s_box)
{
    const uint32_t d = (uint32_t)A.d, t = threadIdx.x;
    if (t < 2 * d) s_box[t] = t < d ? INT32_MAX : INT32_MIN;
    __syncthreads();
    for (uint32_t e = t; e < A.boxes * 2 * d; e += blockDim.x) {
        const uint32_t k = e % (2 * d);
        const int32_t v = A.partial[e];
        if (k < d) atomicMin(s_box + k, v);
        else atomicMax(s_box + k, v);
    }
    __syncthreads();
}

// Up to eight axes: every squared distance below 2^31 with 24-bit differences.
__device__ __forceinline__ bool small_narrow(const SmallArgs &A, const int32_t *s_box)
{
    uint64_t span = 0;
    for (int k = 0; k < A.d; k++) span = max(span, (uint64_t)((int64_t)s_box[A.d + k] - s_box[k]));
    return span < (1u << 16) && (uint64_t)A.d * span * span < (1ull << 31);
}

// Can this path take the data?  Up to eight axes: spans below 2^30 and a
// packed cube key that surely fits 63 bits (a coordinate takes at most one
// bit more than its cube number, with search groups of at most eight cubes);
// past eight: data that byte planes hold.  Anything else is left to the
// general path, which refuses what it refuses.
__device__ __forceinline__ bool small_takes(const SmallArgs &A, const int32_t *s_box)
{
    uint64_t sum = 0, bits = 0;
    for (int k = 0; k < A.d; k++) {
        const uint64_t span = (uint64_t)((int64_t)s_box[A.d + k] - s_box[k]);
        if (span >= (A.d > kMaxDim ? 1ull << 15 : 1ull << 30)) return false;
        sum += span * span;
        if (A.d <= kMaxDim) bits += 1 + max(3, 64 - __clzll((long long)(span / A.side)));
    }
    if (A.d > kMaxDim) return sum < (1ull << 31);
    return bits <= 63;
}

// ---------------------------------------------------------------------------
// Past eight axes: byte planes of the rows (laid out as for the general
// path), negated norms, and the limit that 2 p.q - |q|^2 has to reach for a
// candidate p (nothing reaches that of a padding row).
// ---------------------------------------------------------------------------
template <int KS>
__global__ __launch_bounds__(kBlock) void k_small_planes(SmallArgs A)
{
    constexpr uint32_t C = 2 * KS;
    __shared__ int32_t s_box[2 * kMaxDimHigh];
    const uint32_t d = (uint32_t)A.d;
    small_box(A, s_box);
    const uint32_t c = threadIdx.x % C, half = c / KS, step = c % KS, a0 = 32u * step + 16u * half;
    const int32_t eps2 = (int32_t)min(A.eps2, (int64_t)INT32_MAX);
    // np is a multiple of 64, so whole waves take part
    for (uint32_t t = blockIdx.x * kBlock + threadIdx.x; t < A.np * C; t += gridDim.x * kBlock) {
        const uint32_t r = t / C;
        uint32_t hi[4] = {0, 0, 0, 0}, lo[4] = {0, 0, 0, 0}, norm = 0;
        if (r < A.n) {
            int32_t x[16];
#pragma unroll
            for (int i = 0; i < 16; i++) {
                const uint32_t a = a0 + i;
                x[i] = 0;
                if (a < d) x[i] = A.pts[r * d + a] - (int32_t)(((int64_t)s_box[a] + s_box[d + a]) >> 1);
            }
#pragma unroll
            for (int i = 0; i < 16; i++) {
                hi[i / 4] |= (uint32_t)(((x[i] + 128) >> 8) & 255) << (8 * (i % 4));
                lo[i / 4] |= (uint32_t)(x[i] & 255) << (8 * (i % 4));
                norm += (uint32_t)(x[i] * x[i]);
            }
        }
#pragma unroll
        for (uint32_t o = 1; o < C; o <<= 1) norm += __shfl_xor(norm, o);
        uint4 *row = reinterpret_cast<uint4 *>(A.planes) + (uint64_t)r * (2 * C) + half * (2 * KS);
        row[step] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        row[KS + step] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        if (c == 0) {
            A.nnorm[r] = -(int32_t)norm;
            A.lim[r] = r < A.n ? (int32_t)norm - eps2 : INT32_MAX;
        }
    }
}

// ---------------------------------------------------------------------------
// All pairs: word w of point i (adj[w * np + i], so that a wave's 64 points
// store and load whole lines) has bit k set when point 32 w + k is within
// eps of it; cnt[i] adds them up.  A wave takes 64 points and kSmallSlice
// candidates.
// ---------------------------------------------------------------------------
// Up to eight axes on the vector units: the points in the lanes, the
// candidates' coordinates wave-uniform.  A whole word's candidates lie one
// after the other, so they come in a few wide scalar loads; only the last
// word repeats the last point.  2 d + 3 vector instructions per 64 pairs.
template <int D, bool WIDE, bool WHOLE>
__device__ __forceinline__ uint32_t small_word(const SmallArgs &A, const Pt<D> &p, uint32_t jb)
{
    const ConstInt *pts = (const ConstInt *)(uintptr_t)A.pts + (uint64_t)jb * D;
    const int32_t lim = (int32_t)min(A.eps2, (int64_t)INT32_MAX);
    uint32_t word = 0;
    // (a whole word's coordinates fit the scalar registers up to three axes)
#pragma unroll D <= 3 && !WIDE ? 32 : 8
    for (int k = 31; k >= 0; k--) {
        const ConstInt *row = pts + (WHOLE ? (uint32_t)k : min((uint32_t)k, A.n - 1 - jb)) * D;
        bool hit;
        if constexpr (WIDE) {
            int64_t s = 0;
#pragma unroll
            for (int e = 0; e < D; e++) {
                const int64_t t = (int64_t)p.x[e] - row[e];
                s += t * t;
            }
            hit = s <= A.eps2;
        } else {
            int32_t s = 0;
#pragma unroll
            for (int e = 0; e < D; e++) {
                const int32_t t = p.x[e] - row[e];
                s += __mul24(t, t);
            }
            hit = s <= lim;
        }
        word |= hit ? 1u << k : 0u;
    }
    return WHOLE ? word : word & ((1u << (A.n - jb)) - 1u);
}

template <int D, bool WIDE>
__device__ __forceinline__ uint32_t small_words(const SmallArgs &A, const Pt<D> &p, uint32_t i, uint32_t j0)
{
    uint32_t cnt = 0, jb = j0;
    for (; jb + 32 <= min(j0 + kSmallSlice, A.n); jb += 32) {
        const uint32_t word = small_word<D, WIDE, true>(A, p, jb);
        A.adj[(uint64_t)(jb / 32) * A.np + i] = word;
        cnt += __popc(word);
    }
    if (jb < min(j0 + kSmallSlice, A.n)) {
        const uint32_t word = small_word<D, WIDE, false>(A, p, jb);
        A.adj[(uint64_t)(jb / 32) * A.np + i] = word;
        cnt += __popc(word);
    }
    return cnt;
}

template <int D>
__global__ __launch_bounds__(kBlock) void k_small_pairs(SmallArgs A)
{
    __shared__ int32_t s_box[2 * kMaxDimHigh];
    small_box(A, s_box);
    const uint32_t u = uniform(blockIdx.x * kWavesPerBlock + wave_in_block());
    const uint32_t slices = (A.n + kSmallSlice - 1) / kSmallSlice;
    const uint32_t i = u / slices * kWave + lane_id(), j0 = u % slices * kSmallSlice;
    if (u / slices * kWave >= A.n) return;
    Pt<D> p;
#pragma unroll
    for (int e = 0; e < D; e++) p.x[e] = A.pts[(uint64_t)min(i, A.n - 1) * D + e];
    const uint32_t cnt = small_narrow(A, s_box) ? small_words<D, false>(A, p, i, j0) : small_words<D, true>(A, p, i, j0);
    if (i < A.n && cnt) atomicAdd(A.cnt + i, cnt);
}

// Past eight axes on the matrix units: the wave's 64 points are the columns
// of two tiles, 32 candidates at a time the rows.  A lane has 16 of the 32
// rows of its column, the lane 32 further on the others.
template <int KS>
__global__ __launch_bounds__(kBlock, 2) void k_small_tiles(SmallArgs A)
{
    const uint32_t u = uniform(blockIdx.x * kWavesPerBlock + wave_in_block()), l = lane_id(), half = l >> 5;
    const uint32_t slices = (A.n + kSmallSlice - 1) / kSmallSlice;
    const uint32_t i0 = u / slices * kWave, j0 = u % slices * kSmallSlice;
    if (i0 >= A.n) return;
    const v4i *planes = reinterpret_cast<const v4i *>(A.planes);
    v4i b[2][2 * KS];
    int32_t nq[2];
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const uint32_t i = i0 + 32 * k + (l & 31u);
#pragma unroll
        for (int e = 0; e < 2 * KS; e++) b[k][e] = planes[(uint64_t)i * (4 * KS) + half * (2 * KS) + e];
        nq[k] = A.nnorm[i];
    }
    uint32_t cnt = 0;
    for (uint32_t jb = j0; jb < min(j0 + kSmallSlice, A.n); jb += 32) {
        v4i a[2 * KS];
#pragma unroll
        for (int e = 0; e < 2 * KS; e++) a[e] = planes[(uint64_t)(jb + (l & 31u)) * (4 * KS) + half * (2 * KS) + e];
        int32_t lim[16];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int4 t = *reinterpret_cast<const int4 *>(A.lim + jb + 8 * j + 4 * half);
            lim[4 * j] = t.x;
            lim[4 * j + 1] = t.y;
            lim[4 * j + 2] = t.z;
            lim[4 * j + 3] = t.w;
        }
        uint32_t word[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            v16i hh = {0}, hl = {0}, ll = {0};
#pragma unroll
            for (int st = 0; st < KS; st++) {
                hh = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[st], b[k][st], hh, 0, 0, 0);
                hl = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[st], b[k][KS + st], hl, 0, 0, 0);
                ll = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[KS + st], b[k][KS + st], ll, 0, 0, 0);
                hl = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[KS + st], b[k][st], hl, 0, 0, 0);
            }
            uint32_t m = 0;
#pragma unroll
            for (int r = 15; r >= 0; r--) {
                const uint32_t dot = ((((uint32_t)hh[r] << 8) + (uint32_t)hl[r]) << 8) + (uint32_t)ll[r];
                const int32_t v = (int32_t)((dot << 1) + (uint32_t)nq[k]);
                m = m + m + (v >= lim[r] ? 1u : 0u);
            }
            // result 4 a + c is row 8 a + c (+ 4 in the upper half)
            m = (m | m << 8) & 0x00FF00FFu;
            m = (m | m << 4) & 0x0F0F0F0Fu;
            m <<= 4 * half;
            word[k] = m | __shfl_xor(m, 32);
        }
        const uint32_t w = half ? word[1] : word[0];
        A.adj[(uint64_t)(jb / 32) * A.np + i0 + l] = w;
        cnt += __popc(w);
    }
    if (i0 + l < A.n && cnt) atomicAdd(A.cnt + i0 + l, cnt);
}

// ---------------------------------------------------------------------------
// Core points as a bit set in LDS (whole block; followed by a barrier).  Like
// every pass over all points by one block, it has all its loads in flight
// before the first is used.
// ---------------------------------------------------------------------------
constexpr int kSmallEach = kSmallMax / kSmallBlock;      // points per thread, at most

__device__ __forceinline__ void small_core_bits(const SmallArgs &A, uint32_t *s_core)
{
    uint32_t c[kSmallEach];
#pragma unroll
    for (int q = 0; q < kSmallEach; q++) {
        const uint32_t i = q * kSmallBlock + threadIdx.x;
        c[q] = i < A.n ? A.cnt[i] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kSmallEach; q++) {
        const uint32_t i = q * kSmallBlock + threadIdx.x;
        if (i >= A.np) break;
        const uint64_t m = __ballot(i < A.n && c[q] >= (uint32_t)A.min_pts);
        if (lane_id() == 0) {
            s_core[i / 32] = (uint32_t)m;
            s_core[i / 32 + 1] = (uint32_t)(m >> 32);
        }
    }
    __syncthreads();
}

// The forest from memory into LDS (followed by a barrier).
__device__ __forceinline__ void small_forest(const SmallArgs &A, uint32_t *s_root)
{
    uint32_t r[kSmallEach];
#pragma unroll
    for (int q = 0; q < kSmallEach; q++) {
        const uint32_t i = q * kSmallBlock + threadIdx.x;
        r[q] = i < A.np ? ld_agent32(A.parent + i) : 0u;
    }
#pragma unroll
    for (int q = 0; q < kSmallEach; q++) {
        const uint32_t i = q * kSmallBlock + threadIdx.x;
        if (i < A.np) s_root[i] = r[q];
    }
    __syncthreads();
}

// Root of x in the LDS forest: entries only ever move to ancestors.
__device__ __forceinline__ uint32_t small_root(volatile uint32_t *s_root, uint32_t x)
{
    uint32_t r = s_root[x];
    while (r != x) {
        x = r;
        r = s_root[x];
    }
    return r;
}

// Every point of the LDS forest under its root (whole block, after a barrier
// and followed by one).  An entry only moves up its path, so threads may read
// entries that others are moving; each step is written at once, so that the
// steps of the others grow with it: a chain of 12k points given in order, whose
// forest is as deep as that, takes some ten steps for each 1024 points instead
// of a thousand (2-D call 227 -> 158 us).  (Pointer jumping with a barrier per
// step was slower: 55 -> 72 us for the join of 10k points.)
__device__ __forceinline__ void small_flatten(uint32_t np, volatile uint32_t *s_root)
{
    for (uint32_t i = threadIdx.x; i < np; i += kSmallBlock) {
        uint32_t r = s_root[i];
        for (uint32_t up = s_root[r]; up != r; up = s_root[r]) {
            s_root[i] = up;
            r = up;
        }
    }
    __syncthreads();
}

// A first forest: every core point under its smallest core neighbour, with
// plain stores.  64 points per block, its 16 waves sharing the words.
// (Joining a sample of the neighbours here instead, with atomics, had all
// points of a cluster queue up at one root: 110 us at 4000 points, 6 this
// way.)
__global__ __launch_bounds__(kSmallBlock) void k_small_hook(SmallArgs A)
{
    __shared__ uint32_t s_core[kSmallMax / 32], s_first[kWave];
    const uint32_t w = wave_in_block(), l = lane_id(), i = blockIdx.x * kWave + l;
    if (threadIdx.x < (uint32_t)kWave) s_first[threadIdx.x] = kNone;
    small_core_bits(A, s_core);
    const bool core = (s_core[i / 32] >> (i % 32)) & 1u;
    uint32_t first = kNone;
    for (uint32_t k = w; 32 * k <= blockIdx.x * kWave + 63u && k * 32 < A.n; k += kSmallWaves) {
        if (!__ballot(core && first == kNone)) break;
        uint32_t m = A.adj[(uint64_t)k * A.np + i] & s_core[k];
        if (32 * k + 31 >= i) m = 32 * k >= i ? 0u : m & ((1u << (i - 32 * k)) - 1u);
        if (first == kNone && m) first = 32 * k + (uint32_t)__ffs(m) - 1;
    }
    if (core && first != kNone) atomicMin(&s_first[l], first);
    __syncthreads();
    if (w == 0 && core && s_first[l] != kNone) A.parent[i] = s_first[l];
}

// a and b joined in the LDS forest; true when they were two trees.
__device__ __forceinline__ bool small_union(uint32_t *s_root, uint32_t a, uint32_t b)
{
    while (true) {
        a = small_root(s_root, a);
        b = small_root(s_root, b);
        if (a == b) return false;
        if (a < b) { const uint32_t t = a; a = b; b = t; }
        if (atomicCAS(s_root + a, a, b) == a) return true;
    }
}

// The unions that are still missing, and the nearest core neighbour of every
// other point (ties to the smaller index).  Lane = point; a wave holds its
// sixteenth of the points' words in registers.  Where points have many
// neighbours, the members of one tree at a time are laid out as a bit set,
// which tells 32 neighbours per word apart from those of other trees (testing
// them one by one took 270 us at 16k points in dense blobs); where
// they have few, each neighbour's root is looked up.  The forest is kept
// in LDS and joined there; what joined two of its trees is noted and done in
// memory at the end, side by side, so that pairs between the same two trees
// cost one union there and no wave waits for one in the middle.
constexpr uint32_t kSmallPairs = 1024;         // unions noted; more go to memory at once
constexpr uint32_t kSmallFew = 24;             // neighbours per lane that are looked up one by one
__global__ __launch_bounds__(kSmallBlock) void k_small_join(SmallArgs A)
{
    __shared__ uint32_t s_core[kSmallMax / 32], s_root[kSmallMax], s_tree[kSmallMax / 32], s_most, s_noted, s_near[kWave];
    __shared__ uint2 s_pair[kSmallPairs];
    __shared__ unsigned long long s_dist[kWave];
    constexpr int W = kSmallMax / 32 / kSmallWaves;
    const uint32_t w = uniform(wave_in_block()), l = lane_id(), i = blockIdx.x * kWave + l, d = (uint32_t)A.d;
    const uint32_t words = (A.n + 31) / 32;
    uint32_t word[W];
#pragma unroll
    for (int x = 0; x < W; x++) {
        const uint32_t k = x * kSmallWaves + w;
        word[x] = k < words ? A.adj[(uint64_t)k * A.np + i] : 0u;
    }
    small_forest(A, s_root);
    if (threadIdx.x < (uint32_t)kWave) {
        s_near[threadIdx.x] = kNone;
        s_dist[threadIdx.x] = ~0ull;
    }
    if (threadIdx.x == 0) s_most = s_noted = 0;
    small_core_bits(A, s_core);
    small_flatten(A.np, s_root);
    const bool in = i < A.n, core = (s_core[i / 32] >> (i % 32)) & 1u;
    uint32_t bits = 0;
#pragma unroll
    for (int x = 0; x < W; x++) {
        const uint32_t k = x * kSmallWaves + w;
        if (k >= words) break;
        uint32_t m = in ? word[x] & s_core[k] : 0u;
        // a core point looks at smaller ones only
        if (core && 32 * k + 32 > i) m = 32 * k >= i ? 0u : m & ((1u << (i - 32 * k)) - 1u);
        word[x] = m;
        bits += core ? __popc(m) : 0u;
    }
    bits = wave_max(bits);
    if (l == 0) atomicMax(&s_most, bits);
    __syncthreads();
    uint32_t mine = s_root[i];
    auto join = [&](uint32_t j) {
        const uint32_t r = s_root[j];
        if (r == mine || !small_union(s_root, mine, r)) return;
        const uint32_t at = atomicAdd(&s_noted, 1u);
        if (at < kSmallPairs) s_pair[at] = make_uint2(mine, r);
        else uf_union<true>(A.parent, mine, r);
    };
    // a sample first, one neighbour per word: it connects nearly all of a
    // cluster, and the trees are flat again before the rest
#pragma unroll
    for (int x = 0; x < W; x++) {
        if ((uint32_t)(x * kSmallWaves) >= words) break;
        if (core && word[x]) join(32 * (x * kSmallWaves + w) + (uint32_t)__ffs(word[x]) - 1);
    }
    __syncthreads();
    small_flatten(A.np, s_root);
    mine = s_root[i];
    if (s_most <= kSmallFew) {
#pragma unroll
        for (int x = 0; x < W; x++) {
            if ((uint32_t)(x * kSmallWaves) >= words) break;
            for (uint32_t m = core ? word[x] : 0u; m; m &= m - 1) join(32 * (x * kSmallWaves + w) + (uint32_t)__ffs(m) - 1);
        }
    } else {
        // the trees of the block's points, one after the other (the same
        // order in every wave: the points' trees are read before any union)
        uint64_t left = __ballot(core);
        __syncthreads();
        while (left) {
            const uint32_t t = lane_value(mine, (uint32_t)__ffsll((unsigned long long)left) - 1);
            const uint64_t rows = __ballot(core && mine == t);
            left &= ~rows;
            uint32_t r[kSmallEach];
#pragma unroll
            for (int q = 0; q < kSmallEach; q++) {
                const uint32_t k = q * kSmallBlock + threadIdx.x;
                r[q] = k < A.np ? s_root[k] : kNone;
            }
#pragma unroll
            for (int q = 0; q < kSmallEach; q++) {
                const uint32_t k = q * kSmallBlock + threadIdx.x;
                if (k >= A.np) break;
                const uint64_t m = __ballot(r[q] == t);
                if (l == 0) {
                    s_tree[k / 32] = (uint32_t)m;
                    s_tree[k / 32 + 1] = (uint32_t)(m >> 32);
                }
            }
            __syncthreads();
#pragma unroll
            for (int x = 0; x < W; x++) {
                const uint32_t k = x * kSmallWaves + w;
                if (k >= words) break;
                for (uint32_t m = core && mine == t ? word[x] & ~s_tree[k] : 0u; m; m &= m - 1)
                    join(32 * k + (uint32_t)__ffs(m) - 1);
            }
            __syncthreads();
        }
    }
    uint32_t near = kNone;
    uint64_t best = ~0ull;
#pragma unroll
    for (int x = 0; x < W; x++) {
        const uint32_t k = x * kSmallWaves + w;
        if (k >= words) break;
        for (uint32_t m = core ? 0u : word[x]; m; m &= m - 1) {
            const uint32_t j = 32 * k + (uint32_t)__ffs(m) - 1;
            uint64_t t2 = 0;
#pragma unroll 8
            for (uint32_t e = 0; e < d; e++) {
                const int64_t t = (int64_t)A.pts[(uint64_t)i * d + e] - A.pts[(uint64_t)j * d + e];
                t2 += (uint64_t)(t * t);
            }
            if (t2 < best) {
                best = t2;
                near = j;
            }
        }
    }
    if (near != kNone) atomicMin(&s_dist[l], (unsigned long long)best);
    __syncthreads();
    if (near != kNone && s_dist[l] == best) atomicMin(&s_near[l], near);
    for (uint32_t k = threadIdx.x; k < min(s_noted, kSmallPairs); k += kSmallBlock)
        uf_union<true>(A.parent, s_pair[k].x, s_pair[k].y);
    __syncthreads();
    if (w == 0 && in) A.near[i] = core ? i : s_near[l];
}

// ---------------------------------------------------------------------------
// Labels, by one block: the forest flattened, every member offered to its
// root's smallest index, roots numbered in the order of those indices.  Also
// the verdict for the host: 0 labels written, 1 data for the general path.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kSmallBlock) void k_small_labels(SmallArgs A)
{
    __shared__ uint32_t s_root[kSmallMax], s_min[kSmallMax], s_bits[kSmallMax / 32], s_rank[kSmallMax / 64];
    __shared__ int32_t s_box[2 * kMaxDimHigh];
    const uint32_t t = threadIdx.x, l = lane_id(), n = A.n, np = A.np;
    small_box(A, s_box);
    for (uint32_t i = t; i < np; i += kSmallBlock) s_min[i] = kNone;
    const uint32_t verdict = small_takes(A, s_box) ? 0u : 1u;
    if (t < 2 * (uint32_t)A.d && A.d <= kMaxDim)
        __hip_atomic_store(A.report + 1 + t, (uint32_t)s_box[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (t == 0) __hip_atomic_store(A.report, verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (verdict) return;                                   // the same in every thread
    small_forest(A, s_root);
    small_flatten(np, s_root);
    // the root of each point's cluster (kNone: noise), in registers
    constexpr int Q = kSmallEach;
    uint32_t root[Q];
#pragma unroll
    for (int q = 0; q < Q; q++) root[q] = q * kSmallBlock + t < n ? A.near[q * kSmallBlock + t] : kNone;
#pragma unroll
    for (int q = 0; q < Q; q++)
        if (root[q] != kNone) {
            root[q] = s_root[root[q]];
            const uint32_t i = q * kSmallBlock + t;
            if (i < s_min[root[q]]) atomicMin(&s_min[root[q]], i);
        }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; q++) {
        const uint32_t i = q * kSmallBlock + t;
        if (i >= np) break;
        const uint64_t m = __ballot(root[q] != kNone && s_min[root[q]] == i);
        if (l == 0) {
            s_bits[i / 32] = (uint32_t)m;
            s_bits[i / 32 + 1] = (uint32_t)(m >> 32);
        }
    }
    __syncthreads();
    // smallest members before each 64 points: at most four words per lane of
    // the first wave
    if (t < (uint32_t)kWave) {
        constexpr uint32_t W = kSmallMax / 64 / kWave;
        uint32_t c[W], sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < W; q++) {
            const uint32_t word = t * W + q;
            c[q] = word * 64 < np ? (uint32_t)(__popc(s_bits[2 * word]) + __popc(s_bits[2 * word + 1])) : 0u;
            sum += c[q];
        }
        uint32_t at = wave_inclusive_scan(sum) - sum;
#pragma unroll
        for (uint32_t q = 0; q < W; q++) {
            s_rank[t * W + q] = at;
            at += c[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; q++) {
        const uint32_t i = q * kSmallBlock + t;
        if (i >= n) break;
        int32_t label = -1;
        if (root[q] != kNone) {
            const uint32_t f = s_min[root[q]];
            const uint64_t bits = (uint64_t)s_bits[f / 64 * 2 + 1] << 32 | s_bits[f / 64 * 2];
            label = (int32_t)(s_rank[f / 64] + (uint32_t)__popcll(bits & ((1ull << (f % 64)) - 1ull)));
        }
        A.labels[i] = label;
        if (A.core_out) A.core_out[i] = A.cnt[i] >= (uint32_t)A.min_pts;
    }
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
void launch_small(const SmallArgs &A, hipStream_t s)
{
    hipLaunchKernelGGL(k_small_box, dim3(A.boxes), dim3(kBlock), 0, s, A);
    const uint32_t blocks64 = A.np / kWave, slices = (A.n + kSmallSlice - 1) / kSmallSlice;
    const dim3 pairs((blocks64 * slices + kWavesPerBlock - 1) / kWavesPerBlock), threads(kBlock);
    switch (A.d) {
    case 1: hipLaunchKernelGGL(k_small_pairs<1>, pairs, threads, 0, s, A); break;
    case 2: hipLaunchKernelGGL(k_small_pairs<2>, pairs, threads, 0, s, A); break;
    case 3: hipLaunchKernelGGL(k_small_pairs<3>, pairs, threads, 0, s, A); break;
    case 4: hipLaunchKernelGGL(k_small_pairs<4>, pairs, threads, 0, s, A); break;
    case 5: hipLaunchKernelGGL(k_small_pairs<5>, pairs, threads, 0, s, A); break;
    case 6: hipLaunchKernelGGL(k_small_pairs<6>, pairs, threads, 0, s, A); break;
    case 7: hipLaunchKernelGGL(k_small_pairs<7>, pairs, threads, 0, s, A); break;
    case 8: hipLaunchKernelGGL(k_small_pairs<8>, pairs, threads, 0, s, A); break;
    default: {
        const int ks = A.d <= 32 ? 1 : 2;
        const dim3 rows((A.np * 2 * ks + kBlock - 1) / kBlock);
        if (ks == 1) {
            hipLaunchKernelGGL(k_small_planes<1>, rows, threads, 0, s, A);
            hipLaunchKernelGGL(k_small_tiles<1>, pairs, threads, 0, s, A);
        } else {
            hipLaunchKernelGGL(k_small_planes<2>, rows, threads, 0, s, A);
            hipLaunchKernelGGL(k_small_tiles<2>, pairs, threads, 0, s, A);
        }
    }
    }
    hipLaunchKernelGGL(k_small_hook, dim3(blocks64), dim3(kSmallBlock), 0, s, A);
    hipLaunchKernelGGL(k_small_join, dim3(blocks64), dim3(kSmallBlock), 0, s, A);
    hipLaunchKernelGGL(k_small_labels, dim3(1), dim3(kSmallBlock), 0, s, A);
}

}  // namespace hca
