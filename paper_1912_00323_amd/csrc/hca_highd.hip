// Data with more than eight axes (the paper's data sets reach 54; Table 1).
//
// The cube of side eps/sqrt(d) stays the unit that holds points within eps of
// each other (a cube with minPts points makes them all core, and a cube is
// the union-find node), but its stencil grows like (2 ceil(sqrt(d)) + 1)^d, so
// the neighbour search runs over search groups: boxes of side >= eps along at
// most eight key axes (those with the most groups), unbounded along the
// others.  Every point within eps of a point of group G lies in G or in a
// group at an offset in {-1, 0, 1} along each key axis; the neighbour lists
// keep the groups whose point boxes come within eps over all axes.
//
// Points are rows of sd int32 words (d padded with zeros to a multiple of 4),
// in sorted order.  A wave takes chunks of 8 consecutive points, stages them
// in LDS, and streams candidate rows through its lanes with 16-byte loads,
// each lane testing its candidate against all 8 staged points at once.
#include <algorithm>

#include "hca_device.h"
#include "hca_kernels.h"

namespace hca {

// A staged point in LDS: its int32 coordinates, then (packed form) its
// coordinates less the origin as int16 pairs.
constexpr int kOwnStride = kMaxDimHigh + kMaxDimHigh / 2;

typedef short short2_t __attribute__((ext_vector_type(2)));

// acc + (a.lo - b.lo)^2 + (a.hi - b.hi)^2 for two packed int16 pairs (their
// differences fit int16: every span is below 2^15).
__device__ __forceinline__ int32_t sq_dot16(uint32_t a, uint32_t b, int32_t acc)
{
    const short2_t d = __builtin_bit_cast(short2_t, a) - __builtin_bit_cast(short2_t, b);
    return __builtin_amdgcn_sdot2(d, d, acc, false);
}


// ---------------------------------------------------------------------------
// Byte planes.  When every span is below 2^15 and the squared spans add up to
// less than 2^31, a coordinate less its axis' centre is x = 256 h + l with
// signed bytes h in [-64, 64] and l in [-128, 127], so a product of two
// points is exact in four products of bytes,
//   p.q = 2^16 h.h' + 2^8 (h.l' + l.h') + l.l',
// each summed in 32 bits, and |p - q|^2 = |p|^2 + |q|^2 - 2 p.q (also below
// 2^31; the sums in between may wrap).  That makes the distances of a set of
// points from a set of candidates a contraction for the byte matrix units.
//
// A row holds two halves of KS chunks of high bytes and KS chunks of low ones
// (KS = 1 up to 32 axes, else 2): chunk (half, step) has the 16 axes from
// 32 step + 16 half on, which is what lane (column, half) feeds to step
// `step` of a 32x32x32 matrix instruction.
// ---------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// One thread per chunk: 16 axes of one row split into bytes, the row's norm
// summed over its 2 KS chunks (neighbouring lanes).
template <int KS>
__global__ __launch_bounds__(kBlock) void k_hd_planes(Plan P)
{
    constexpr uint32_t C = 2 * KS;
    const uint32_t sd = P.sd;
    const uint64_t total = (uint64_t)P.n * C;
    const uint32_t c = threadIdx.x % C, half = c / KS, step = c % KS, a0 = 32u * step + 16u * half;
    for (uint64_t b = (uint64_t)blockIdx.x * kBlock; b < total; b += (uint64_t)gridDim.x * kBlock) {
        const uint64_t t = b + threadIdx.x, r = min(t, total - 1) / C;
        uint32_t hi[4], lo[4], norm = 0;
#pragma unroll
        for (int w = 0; w < 4; w++) {
            const uint32_t a = a0 + 4 * w;
            int4 v = make_int4(0, 0, 0, 0), o = v;
            if (a < sd) {
                v = *reinterpret_cast<const int4 *>(P.spts + r * sd + a);
                o = *reinterpret_cast<const int4 *>(P.hd_centre + a);
            }
            const int32_t x[4] = {v.x - o.x, v.y - o.y, v.z - o.z, v.w - o.w};
            hi[w] = lo[w] = 0;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                hi[w] |= (uint32_t)(((x[i] + 128) >> 8) & 255) << (8 * i);
                lo[w] |= (uint32_t)(x[i] & 255) << (8 * i);
                norm += (uint32_t)(x[i] * x[i]);
            }
        }
#pragma unroll
        for (uint32_t o = 1; o < C; o <<= 1) norm += __shfl_xor(norm, o);
        if (t < total) {
            uint4 *row = reinterpret_cast<uint4 *>(P.planes) + r * (2 * C) + half * (2 * KS);
            row[step] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            row[KS + step] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            if (c == 0) P.nnorm[r] = -(int32_t)norm;
        }
    }
}

// ---------------------------------------------------------------------------
// Point box of every group over all axes.  Groups are very uneven (one point
// to tens of thousands), so the points are cut into chunks (box_chunk) and a
// wave takes the boxes of the stretches of groups in its chunk; a group that
// lies in several chunks is folded together with atomics.  (54 axes, 3.85M
// points: 5.3 ms with a wave per group, 0.38 ms this way.)
// ---------------------------------------------------------------------------
// Up to 2^15 points the chunks are of 16, so that there are waves enough for
// groups of one or two points (us, lists, with 64 and 16: 16 axes, 23k points
// 689 and 664, 27 axes, 9k 253 and 230; few large groups share more atomics: 12
// axes, 31k points in 6 groups 31 and 49).
__device__ __forceinline__ uint32_t box_chunk(const Plan &P) { return P.n < (1u << 15) ? 16u : (uint32_t)kWave; }

// Before it: backward list counters cleared, "no core cube yet" and "one
// root" for every group, and an empty box for the groups of several chunks.
__global__ __launch_bounds__(kBlock) void k_hd_group_init(Plan P)
{
    if (box_missed(P)) return;
    const uint32_t sd = P.sd, ng = ld_agent32(&P.ctr->n_groups), per = box_chunk(P);
    for (uint32_t g = blockIdx.x * kBlock + threadIdx.x; g < ng; g += gridDim.x * kBlock) {
        st_agent32(P.nbr_bcount + g, 0u);
        st_agent32(P.nbr_bcursor + g, 0u);
        st_agent32(P.gcube + g, kNone);
        P.unified[g] = 1;
        if (P.group_start[g] / per == (P.group_start[g + 1] - 1) / per) continue;
        uint32_t *box = (uint32_t *)(P.gbox + (uint64_t)g * 2 * sd);
        for (uint32_t e = 0; e < sd; e++) {
            st_agent32(box + e, (uint32_t)INT32_MAX);
            st_agent32(box + sd + e, (uint32_t)INT32_MIN);
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_hd_group_box(Plan P)
{
    if (box_missed(P)) return;
    // lane (row, axis): kWave / sd rows at a time
    const uint32_t l = lane_id(), sd = P.sd, rows = kWave / sd, row = l / sd, axis = l - row * sd;
    const bool in = row < rows;
    const uint32_t per = box_chunk(P), chunks = (P.n + per - 1) / per;
    const WaveRange hca_wr_ = wave_range(P.order);
    HCA_FOR_UNITS(u, chunks) {
        const uint32_t c0 = u * per, c1 = min(P.n, c0 + per);
        const uint32_t pg = P.group_of[P.cell_of[min(c0 + l, c1 - 1)]];
        const uint32_t pg0 = P.group_start[pg], pg1 = P.group_start[pg + 1];
        for (uint32_t s = c0; s < c1;) {
            const uint32_t g = lane_value(pg, s - c0), g0 = lane_value(pg0, s - c0), g1 = lane_value(pg1, s - c0);
            const uint32_t e = min(g1, c1);
            int32_t lo = INT32_MAX, hi = INT32_MIN;
            const int32_t *col = P.spts + axis;
            uint32_t q = s + row;
            // sixteen rows in flight per lane
            for (; in && q + 15 * rows < e; q += 16 * rows) {
                int32_t v[16];
#pragma unroll
                for (int i = 0; i < 16; i++) v[i] = col[(uint64_t)(q + i * rows) * sd];
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    lo = min(lo, v[i]);
                    hi = max(hi, v[i]);
                }
            }
            for (; in && q < e; q += rows) {
                const int32_t v = col[(uint64_t)q * sd];
                lo = min(lo, v);
                hi = max(hi, v);
            }
            int32_t l0 = lo, h0 = hi;
            for (uint32_t k = 1; k < rows; k++) {
                l0 = min(l0, __shfl(lo, axis + k * sd));
                h0 = max(h0, __shfl(hi, axis + k * sd));
            }
            if (l < sd) {
                int32_t *box = P.gbox + (uint64_t)g * 2 * sd;
                if (g0 / per == (g1 - 1) / per) {
                    box[l] = l0;
                    box[sd + l] = h0;
                } else {
                    atomicMin(box + l, l0);
                    atomicMax(box + sd + l, h0);
                }
            }
            s = e;
        }
    }
}

// Squared gap between two point boxes (rows [lo: sd][hi: sd]); stops once it
// exceeds eps2, so any value above eps2 only means "farther than eps".
__device__ __forceinline__ int64_t hd_box_gap2(const int32_t *a, const int32_t *b, uint32_t sd, int64_t eps2)
{
    int64_t acc = 0;
    for (uint32_t e = 0; e < sd && acc <= eps2; e++) {
        const int64_t gap = max((int64_t)b[e] - a[sd + e], (int64_t)a[e] - b[sd + e]);
        if (gap > 0) acc += gap * gap;
    }
    return acc;
}

// ---------------------------------------------------------------------------
// Neighbour lists over the key axes.  As for search groups in up to eight
// axes: the 3^kd offsets split into two halves of the key axes; the squared
// gaps between the group's point box and the neighbour group's slab add over
// axes, both halves are sorted, and for each first-half offset the valid
// second-half ones form a prefix.  Only offsets to a larger key are looked up
// (forward entries); a found group is kept when the two point boxes come
// within eps over all axes, and its backward counter is raised.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t hd_axis_gap2(const Plan &P, uint64_t gkey, int e, int o, int32_t lo, int32_t hi)
{
    const int64_t c = (int64_t)((gkey >> P.goff[e]) & ((1ull << P.gw[e]) - 1ull)) + o;
    if (c < 0 || c > (int64_t)P.gmax[e]) return -1;
    const int64_t glo = (int64_t)P.origin[e] + c * P.gside, ghi = glo + P.gside - 1;
    const int64_t gap = glo > hi ? glo - hi : (lo > ghi ? lo - ghi : 0);
    return gap * gap;
}

template <int FIRST, int K, int KD>
__device__ __forceinline__ int64_t hd_half_gap2(const Plan &P, uint64_t gkey, uint32_t idx, const int32_t *qlo,
                                                const int32_t *qhi)
{
    int64_t acc = 0;
#pragma unroll
    for (int e = 0; e < K; e++) {
        const int o = (int)(idx % 3u) - 1;
        idx /= 3u;
        const int64_t g2 = hd_axis_gap2(P, gkey, FIRST + e, o, qlo[FIRST + e], qhi[FIRST + e]);
        if (g2 < 0) return INT64_MAX;
        acc += g2;
    }
    return acc <= P.eps2 ? acc : INT64_MAX;
}

template <int FIRST, int K>
__device__ __forceinline__ int64_t hd_half_key_delta(const Plan &P, uint32_t idx)
{
    int64_t kd = 0;
#pragma unroll
    for (int e = 0; e < K; e++) {
        const int o = (int)(idx % 3u) - 1;
        idx /= 3u;
        kd += (int64_t)o * (int64_t)(1ull << P.goff[FIRST + e]);
    }
    return kd;
}

// Sign of the first non-zero component (the half's first axis most significant).
template <int K>
__device__ __forceinline__ int8_t hd_half_sign(uint32_t idx)
{
    int sg = 0;
#pragma unroll
    for (int e = 0; e < K; e++) {
        const int o = (int)(idx % 3u) - 1;
        idx /= 3u;
        if (sg == 0) sg = o;
    }
    return (int8_t)(sg > 0 ? 1 : (sg < 0 ? -1 : 0));
}

constexpr int kHdListBatch = 4;     // lookups in flight per lane
constexpr int kHdHalf = 81;         // 3^4 offset combinations per half, at most

template <int KD>
__global__ __launch_bounds__(kBlock) void k_hd_lists(Plan P)
{
    if (box_missed(P)) return;
    constexpr int DA = KD / 2, DB = KD - DA;
    constexpr int NA = DA == 0 ? 1 : DA == 1 ? 3 : DA == 2 ? 9 : DA == 3 ? 27 : 81;
    constexpr int NB = DB == 1 ? 3 : DB == 2 ? 9 : DB == 3 ? 27 : 81;
    __shared__ int64_t s_sa[kWavesPerBlock][kHdHalf], s_sb[kWavesPerBlock][kHdHalf];
    __shared__ int64_t s_ka[kWavesPerBlock][kHdHalf], s_kb[kWavesPerBlock][kHdHalf];
    __shared__ int64_t s_in[kWavesPerBlock][kHdHalf];
    __shared__ uint8_t s_ia[kWavesPerBlock][kHdHalf], s_ib[kWavesPerBlock][kHdHalf];
    __shared__ int8_t s_ga[kWavesPerBlock][kHdHalf], s_gb[kWavesPerBlock][kHdHalf];
    __shared__ uint32_t s_pre[kWavesPerBlock][kHdHalf + 1];
    const uint32_t w = wave_in_block(), l = lane_id(), sd = P.sd;
    const int64_t eps2 = P.eps2;
    const uint32_t ng = ld_agent32(&P.ctr->n_groups);
    const uint32_t waves = gridDim.x * kWavesPerBlock;
    const uint32_t slab = P.nbr_cap / waves;
    uint32_t at = (blockIdx.x * kWavesPerBlock + w) * slab;
    const uint32_t end = at + slab;
    uint32_t overflow = 0;
    const DynRange dr_ = dyn_range(P.ctr->dyn[kDynLists], P.order);
    HCA_FOR_UNITS_DYN(g, ng, dr_) {
        const uint64_t gkey = P.group_key[g];
        const int32_t *gb = P.gbox + (uint64_t)g * 2 * sd;
        int32_t qlo[KD], qhi[KD];
#pragma unroll
        for (int e = 0; e < KD; e++) {
            qlo[e] = gb[P.kdim[e]];
            qhi[e] = gb[sd + P.kdim[e]];
        }
        for (int i = l; i < NA; i += kWave) s_in[w][i] = hd_half_gap2<0, DA, KD>(P, gkey, i, qlo, qhi);
        __builtin_amdgcn_wave_barrier();
        bitonic_sort(s_in[w], NA, s_sa[w], s_ia[w]);
        __builtin_amdgcn_wave_barrier();
        for (int j = l; j < NB; j += kWave) s_in[w][j] = hd_half_gap2<DA, DB, KD>(P, gkey, j, qlo, qhi);
        __builtin_amdgcn_wave_barrier();
        bitonic_sort(s_in[w], NB, s_sb[w], s_ib[w]);
        __builtin_amdgcn_wave_barrier();
        for (int i = l; i < NA; i += kWave) s_ga[w][i] = hd_half_sign<DA>(s_ia[w][i]);
        for (int j = l; j < NB; j += kWave) s_gb[w][j] = hd_half_sign<DB>(s_ib[w][j]);
        // valid second-half offsets per first-half one (none when the first
        // half points backwards), then their prefix
        uint32_t tot = 0;
        for (int i0 = 0; i0 < NA; i0 += kWave) {
            const int i = i0 + (int)l;
            uint32_t c = 0;
            if (i < NA && s_sa[w][i] != INT64_MAX && s_ga[w][i] >= 0) {
                const int64_t lim = eps2 - s_sa[w][i];
                int lo = 0, hi = NB;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (s_sb[w][mid] <= lim) lo = mid + 1; else hi = mid;
                }
                c = (uint32_t)lo;
            }
            const uint32_t inc = wave_inclusive_scan(c);
            if (i < NA) s_pre[w][i] = tot + inc - c;
            tot += lane_value(inc, kWave - 1);
        }
        if (l == 0) s_pre[w][NA] = tot;
        for (int i = l; i < NA; i += kWave) s_ka[w][i] = hd_half_key_delta<0, DA>(P, s_ia[w][i]);
        for (int j = l; j < NB; j += kWave) s_kb[w][j] = hd_half_key_delta<DA, DB>(P, s_ib[w][j]);
        __builtin_amdgcn_wave_barrier();
        const uint32_t start = at;
        bool fits = true;
        for (uint32_t t0 = 0; t0 < tot; t0 += kWave * kHdListBatch) {
            uint64_t nk[kHdListBatch];
            uint32_t G[kHdListBatch];
#pragma unroll
            for (int b = 0; b < kHdListBatch; b++) {
                const uint32_t t = t0 + b * kWave + l;
                nk[b] = ~0ull;
                if (t < tot) {
                    int lo = 0, hi = NA;                  // last i with s_pre[i] <= t
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (s_pre[w][mid] <= t) lo = mid; else hi = mid;
                    }
                    const uint32_t j = t - s_pre[w][lo];
                    if (s_ga[w][lo] > 0 || s_gb[w][j] > 0) nk[b] = gkey + (uint64_t)(s_ka[w][lo] + s_kb[w][j]);
                }
            }
            group_lookup_n<kHdListBatch>(P, nk, G);
#pragma unroll
            for (int b = 0; b < kHdListBatch; b++) {
                if (G[b] != kNone && hd_box_gap2(gb, P.gbox + (uint64_t)G[b] * 2 * sd, sd, eps2) > eps2)
                    G[b] = kNone;
                const uint64_t m = __ballot(G[b] != kNone);
                const uint32_t k = (uint32_t)__popcll(m);
                if (at + k > end) fits = false;
                if (fits && G[b] != kNone) {
                    P.nbr[at + __popcll(m & __lanemask_lt())] = G[b];
                    atomicAdd(P.nbr_bcount + G[b], 1u);
                }
                if (fits) at += k;
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (l == 0) {
            P.nbr_start[g] = start;
            P.nbr_count[g] = fits ? at - start : kNone;
        }
        if (!fits) {
            at = start;
            overflow++;
        }
    }
    if (l == 0 && overflow) atomicAdd(&P.ctr->nbr_overflow, overflow);
}

// ---------------------------------------------------------------------------
// Walks over a group and its listed neighbours.
// ---------------------------------------------------------------------------
// Slot 0 is the group itself, then its forward entries, then (unless
// forward_only) its backward ones.
struct HdSrc {
    uint32_t start, fcount, bstart, slots;
};

__device__ __forceinline__ HdSrc hd_source(const Plan &P, uint32_t g, bool forward_only)
{
    HdSrc s;
    s.start = P.nbr_start[g];
    s.fcount = P.nbr_count[g];
    s.bstart = P.nbr_bstart[g];
    s.slots = 1 + s.fcount + (forward_only ? 0u : P.nbr_bcount[g]);
    return s;
}

__device__ __forceinline__ uint32_t hd_slot(const Plan &P, uint32_t g, const HdSrc &s, uint32_t j)
{
    if (j == 0) return g;
    return j <= s.fcount ? P.nbr[s.start + j - 1] : P.nbr_back[s.bstart + j - 1 - s.fcount];
}

// The 8 rows from sorted position pc (the last one repeated past np) into LDS.
__device__ __forceinline__ void hd_stage(const Plan &P, uint32_t pc, uint32_t np, int32_t (*own)[kOwnStride])
{
    const uint32_t sd = P.sd;
    __builtin_amdgcn_wave_barrier();
    for (uint32_t i = lane_id(); i < kPch * sd; i += kWave) {
        const uint32_t k = i / sd, e = i - k * sd;
        own[k][e] = P.spts[(uint64_t)(pc + min(k, np - 1)) * sd + e];
    }
    if (P.spts16) {
        const uint32_t hw = sd >> 1;
        for (uint32_t i = lane_id(); i < kPch * hw; i += kWave) {
            const uint32_t k = i / hw, e = i - k * hw;
            own[k][kMaxDimHigh + e] = (int32_t)P.spts16[(uint64_t)(pc + min(k, np - 1)) * hw + e];
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// The 8 rows at sorted positions pos[0..8) (wave-uniform) into LDS.
__device__ __forceinline__ void hd_stage_at(const Plan &P, const uint32_t *pos, int32_t (*own)[kOwnStride])
{
    const uint32_t sd = P.sd, l = lane_id();
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < kPch; k++) {
        if (l < sd) own[k][l] = P.spts[(uint64_t)pos[k] * sd + l];
        if (P.spts16 && l < (sd >> 1)) own[k][kMaxDimHigh + l] = (int32_t)P.spts16[(uint64_t)pos[k] * (sd >> 1) + l];
    }
    __builtin_amdgcn_wave_barrier();
}

// Box of the staged points flagged in mask, into qb[0, sd) and qb[sd, 2 sd).
__device__ __forceinline__ void hd_chunk_box(const Plan &P, const int32_t (*own)[kOwnStride], uint32_t mask,
                                             int32_t *qb)
{
    const uint32_t l = lane_id(), sd = P.sd;
    __builtin_amdgcn_wave_barrier();
    if (l < sd) {
        int32_t lo = INT32_MAX, hi = INT32_MIN;
#pragma unroll
        for (int k = 0; k < kPch; k++)
            if (mask & (1u << k)) {
                lo = min(lo, own[k][l]);
                hi = max(hi, own[k][l]);
            }
        qb[l] = lo;
        qb[sd + l] = hi;
    }
    __builtin_amdgcn_wave_barrier();
}

// Squared gap between a staged point and a group box; stops once above eps2.
__device__ __forceinline__ int64_t hd_point_box_gap2(const int32_t *p, const int32_t *b, uint32_t sd, int64_t eps2)
{
    int64_t acc = 0;
    for (uint32_t e = 0; e < sd && acc <= eps2; e++) {
        const int64_t gap = max((int64_t)b[e] - p[e], (int64_t)p[e] - b[sd + e]);
        if (gap > 0) acc += gap * gap;
    }
    return acc;
}

// Candidates of slots [first, first + 64): lane l resolves slot first + l.  A
// group is dropped when it has no core point (need_core), when its box is
// farther than eps from the query box qb (null: not looked at) or from every staged point in
// `mask`, or (skip_root != kNone) when all its core cubes already share the
// root skip_root.  Returns the candidate count.
__device__ __forceinline__ uint32_t hd_load_neighbours(const Plan &P, uint32_t g, const HdSrc &src, uint32_t first,
                                                       bool need_core, const int32_t *qb,
                                                       const int32_t (*own)[kOwnStride], uint32_t mask,
                                                       uint32_t skip_root, uint32_t *s_beg, uint32_t *s_pre)
{
    const uint32_t l = lane_id(), j = first + l, sd = P.sd;
    const int64_t eps2 = P.eps2;
    uint32_t a = 0, size = 0;
    if (j < src.slots) {
        const uint32_t G = hd_slot(P, g, src, j);
        const int32_t *gb = P.gbox + (uint64_t)G * 2 * sd;
        bool keep = !(need_core && P.gcube[G] == kNone);
        if (keep && skip_root != kNone && P.unified[G] && uf_find(P.parent, P.gcube[G]) == skip_root) keep = false;
        keep = keep && (!qb || hd_box_gap2(qb, gb, sd, eps2) <= eps2);
        if (keep && __popc(mask) > 1) {
            bool nearby = false;
#pragma unroll
            for (int k = 0; k < kPch; k++)
                if (!nearby && (mask & (1u << k))) nearby = hd_point_box_gap2(own[k], gb, sd, eps2) <= eps2;
            keep = nearby;
        }
        if (keep) {
            a = P.group_start[G];
            size = P.group_start[G + 1] - a;
        }
    }
    const uint32_t inc = wave_inclusive_scan(size);
    __builtin_amdgcn_wave_barrier();
    s_beg[l] = a;
    s_pre[l] = inc - size;
    __builtin_amdgcn_wave_barrier();
    return lane_value(inc, kWave - 1);
}

// Row forms, fixed per call by the host, one kernel instance each: 32-bit
// sums of int32 rows, 64-bit sums, or packed int16 rows.
constexpr int kRowNarrow = 0, kRowWide = 1, kRowPacked = 2;

__host__ __device__ inline int row_form(const Plan &P)
{
    return P.wide ? kRowWide : P.spts16 ? kRowPacked : kRowNarrow;
}

// Squared distances from the candidate row at sorted position pos to the 8
// staged points (exact: 64-bit, or 32-bit when the host has shown that every
// tested pair's sum fits).  The 32-bit form loads the whole row before any
// arithmetic; the 64-bit form, short of registers, goes 16 bytes at a time.
template <int ROW>
__device__ __forceinline__ void hd_dist(const Plan &P, const int32_t (*own)[kOwnStride], uint32_t pos, int64_t *dd)
{
    const int4 *row = reinterpret_cast<const int4 *>(P.spts + (uint64_t)pos * P.sd);
    const uint32_t n4 = P.sd >> 2;
    if constexpr (ROW == kRowWide) {
        int64_t acc[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) acc[k] = 0;
        for (uint32_t e = 0; e < n4; e++) {
            const int4 v = row[e];
#pragma unroll
            for (int k = 0; k < kPch; k++) {
                const int4 o = reinterpret_cast<const int4 *>(own[k])[e];
                const int64_t a = (int64_t)v.x - o.x, b = (int64_t)v.y - o.y;
                const int64_t c = (int64_t)v.z - o.z, f = (int64_t)v.w - o.w;
                acc[k] += a * a + b * b + c * c + f * f;
            }
        }
#pragma unroll
        for (int k = 0; k < kPch; k++) dd[k] = acc[k];
    } else if constexpr (ROW == kRowPacked) {
        // packed int16 coordinates: two axes per subtract and dot step
        const uint4 *prow = reinterpret_cast<const uint4 *>(P.spts16 + (uint64_t)pos * (P.sd >> 1));
        const uint32_t n8 = P.sd >> 3;
        uint4 v[kMaxDimHigh / 8];
#pragma unroll
        for (int e = 0; e < kMaxDimHigh / 8; e++) {
            v[e] = make_uint4(0, 0, 0, 0);
            if ((uint32_t)e < n8) v[e] = prow[e];
        }
        int32_t acc[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) acc[k] = 0;
#pragma unroll
        for (int e = 0; e < kMaxDimHigh / 8; e++) {
            if ((uint32_t)e >= n8) continue;
#pragma unroll
            for (int k = 0; k < kPch; k++) {
                const uint4 o = reinterpret_cast<const uint4 *>(own[k] + kMaxDimHigh)[e];
                acc[k] = sq_dot16(v[e].x, o.x, acc[k]);
                acc[k] = sq_dot16(v[e].y, o.y, acc[k]);
                acc[k] = sq_dot16(v[e].z, o.z, acc[k]);
                acc[k] = sq_dot16(v[e].w, o.w, acc[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < kPch; k++) dd[k] = acc[k];
    } else {
        // the whole row in flight at once (one memory latency per candidate)
        int4 v[kMaxDimHigh / 4];
#pragma unroll
        for (int e = 0; e < kMaxDimHigh / 4; e++) {
            v[e] = make_int4(0, 0, 0, 0);
            if ((uint32_t)e < n4) v[e] = row[e];
        }
        int32_t acc[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) acc[k] = 0;
#pragma unroll
        for (int e = 0; e < kMaxDimHigh / 4; e++) {
            if ((uint32_t)e >= n4) continue;
#pragma unroll
            for (int k = 0; k < kPch; k++) {
                const int4 o = reinterpret_cast<const int4 *>(own[k])[e];
                const int32_t a = v[e].x - o.x, b = v[e].y - o.y, c = v[e].z - o.z, f = v[e].w - o.w;
                acc[k] += __mul24(a, a) + __mul24(b, b) + __mul24(c, c) + __mul24(f, f);
            }
        }
#pragma unroll
        for (int k = 0; k < kPch; k++) dd[k] = acc[k];
    }
}

__device__ __forceinline__ uint32_t hd_candidate(uint32_t c, const uint32_t *s_beg, const uint32_t *s_pre)
{
    const uint32_t ln = candidate_lane(c, s_pre);
    return s_beg[ln] + (c - s_pre[ln]);
}

// ---------------------------------------------------------------------------
// Core marking (appendix, Definition 2), chunks of 8 sorted points: a point
// of a cube with at least minPts points is core; any other point counts the
// points within eps in its group and the listed neighbours, stopping at
// minPts.  Per cube: core points and the smallest core input index.
// ---------------------------------------------------------------------------
// Stops after `budget` candidates; *cut tells whether it stopped there with
// points left undecided.
// The first kRec neighbours found of staged point k (sorted position
// qpos[k]) are recorded for merging.
template <int ROW>
__device__ __forceinline__ uint32_t hd_count_walk(const Plan &P, uint32_t g, const int32_t (*own)[kOwnStride],
                                                  const uint32_t *qpos, uint32_t done, uint32_t *cnt, int32_t *qb,
                                                  uint32_t *s_beg, uint32_t *s_pre, uint32_t &lt, uint32_t budget,
                                                  bool *cut)
{
    const uint32_t l = lane_id(), minpts = (uint32_t)P.min_pts, all = (1u << kPch) - 1u;
    hd_chunk_box(P, own, ~done & all, qb);
    const HdSrc src = hd_source(P, g, false);
    uint32_t seen = 0;
    for (uint32_t oc = 0; oc < src.slots && done != all && seen < budget; oc += kWave) {
        const uint32_t total = hd_load_neighbours(P, g, src, oc, false, qb, own, ~done & all, kNone, s_beg, s_pre);
        for (uint32_t ci = 0; ci < total && done != all && seen < budget; ci += kWave, seen += kWave) {
            const uint32_t c = ci + l;
            const bool ok = c < total;
            const uint32_t pos = ok ? hd_candidate(c, s_beg, s_pre) : 0u;
            int64_t dd[kPch];
            hd_dist<ROW>(P, own, pos, dd);
#pragma unroll
            for (int k = 0; k < kPch; k++) {
                if (done & (1u << k)) continue;
                lt += ok;
                const bool hit = ok && dd[k] <= P.eps2;
                const uint64_t hm = __ballot(hit);
                if (hm && cnt[k] < (uint32_t)kRec) {
                    const uint32_t r = cnt[k] + __popcll(hm & __lanemask_lt());
                    if (hit && r < (uint32_t)kRec) P.rec[(uint64_t)qpos[k] * kRec + r] = pos;
                }
                cnt[k] += __popcll(hm);
                if (cnt[k] >= minpts) done |= 1u << k;
            }
            done = uniform(done);
        }
    }
    *cut = done != all && seen >= budget;
    return done;
}

// Per-cube tallies of a chunk's decided core points: one atomic per cube.
__device__ __forceinline__ void hd_tally(const Plan &P, bool in, uint32_t cell, bool core, uint32_t me)
{
    const uint32_t l = lane_id();
    uint64_t pend = __ballot(in && core);
    while (pend) {
        const uint32_t k0 = __ffsll((unsigned long long)pend) - 1;
        const uint32_t c = __shfl(cell, k0);
        const bool mine = in && core && cell == c;
        const uint64_t same = __ballot(mine);
        const uint32_t mn = wave_min(mine ? me : kNone);
        if (l == k0) {
            atomicAdd(P.ncore + c, (uint32_t)__popcll(same));
            atomicMin(P.cmin + c, mn);
        }
        pend &= ~same;
    }
}

// First pass: chunks of 8 consecutive sorted points, each point looking at
// up to P.hd_budget candidates; points still undecided are appended to
// the list of the second pass.
// The packed form is held to 96 registers (five waves per SIMD): some
// spill, and the walk still gains from the extra wave.
template <int ROW>
__global__ __launch_bounds__(kBlock, ROW == kRowPacked ? 5 : 1) void k_hd_core(Plan P)
{
    if (box_missed(P)) return;
    __shared__ __align__(16) int32_t s_own[kWavesPerBlock][kPch][kOwnStride];
    __shared__ int32_t s_qb[kWavesPerBlock][2 * kMaxDimHigh];
    __shared__ uint32_t s_beg[kWavesPerBlock][kWave], s_pre[kWavesPerBlock][kWave];
    const uint32_t w = wave_in_block(), l = lane_id();
    const uint32_t n = P.n, minpts = (uint32_t)P.min_pts, all = (1u << kPch) - 1u;
    uint32_t lt = 0;
    const DynRange dr_ = dyn_range(P.ctr->dyn[kDynCore], P.order);
    HCA_FOR_UNITS_DYN(u, (n + kPch - 1) / kPch, dr_) {
        const uint32_t pc = u * kPch, np = min((uint32_t)kPch, n - pc);
        uint32_t cell = kNone, grp = kNone;
        bool dense = true;
        if (l < np) {
            cell = P.cell_of[pc + l];
            grp = P.group_of[cell];
            dense = P.cell_start[cell + 1] - P.cell_start[cell] >= minpts;
        }
        uint32_t done = (uint32_t)__ballot(dense) & all, undec = 0;
        uint32_t cnt[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) cnt[k] = 0;
        uint32_t qpos[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) qpos[k] = pc + min((uint32_t)k, np - 1);
        if (done != all) {
            hd_stage(P, pc, np, s_own[w]);
            uint32_t left = ~done & all;
            while (left) {
                const uint32_t g = lane_value(grp, __ffs(left) - 1);
                const uint32_t run = (uint32_t)__ballot(grp == g) & left;
                left &= ~run;
                bool cut;
                const uint32_t got = hd_count_walk<ROW>(P, g, s_own[w], qpos, ~run & all, cnt, s_qb[w], s_beg[w],
                                                         s_pre[w], lt, P.hd_budget, &cut);
                done |= got & run;
                if (cut) undec |= run & ~got;
            }
        }
        uint32_t mine = 0;
#pragma unroll
        for (int k = 0; k < kPch; k++)
            if ((uint32_t)k == l) mine = cnt[k];
        const bool in = l < np, later = in && ((undec >> l) & 1u);
        const bool core = in && !later && (dense || mine >= minpts);
        if (in && !later) {
            P.core[pc + l] = core;
            P.nrec[pc + l] = (uint8_t)(dense ? 0u : rec_count(mine));
        }
        const uint64_t um = __ballot(later);
        if (um) {
            uint32_t base = 0;
            if (l == 0) base = atomicAdd(P.ctr->hd_left, (uint32_t)__popcll(um));
            base = __shfl(base, 0);
            if (later) P.hd_list[base + __popcll(um & __lanemask_lt())] = pc + l;
        }
        hd_tally(P, in, cell, core, core ? P.sidx[pc + l] : kNone);
    }
    flush_tests(P, kTestsCore, lt);
}

// Second pass: chunks of 8 points of the list, walked to the end.
template <int ROW>
__global__ __launch_bounds__(kBlock, ROW == kRowPacked ? 5 : 1) void k_hd_core_rest(Plan P)
{
    if (box_missed(P)) return;
    __shared__ __align__(16) int32_t s_own[kWavesPerBlock][kPch][kOwnStride];
    __shared__ int32_t s_qb[kWavesPerBlock][2 * kMaxDimHigh];
    __shared__ uint32_t s_beg[kWavesPerBlock][kWave], s_pre[kWavesPerBlock][kWave];
    const uint32_t w = wave_in_block(), l = lane_id();
    const uint32_t nl = ld_agent32(P.ctr->hd_left), minpts = (uint32_t)P.min_pts;
    const uint32_t all = (1u << kPch) - 1u;
    uint32_t lt = 0;
    const DynRange dr_ = dyn_range(P.ctr->dyn[kDynCoreRest], P.order);
    HCA_FOR_UNITS_DYN(u, (nl + kPch - 1) / kPch, dr_) {
        const uint32_t b0 = u * kPch, np = min((uint32_t)kPch, nl - b0);
        uint32_t pos[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) pos[k] = P.hd_list[b0 + min((uint32_t)k, np - 1)];
        uint32_t q = pos[0];
#pragma unroll
        for (int k = 1; k < kPch; k++)
            if ((uint32_t)k == l) q = pos[k];
        const bool in = l < np;
        const uint32_t cell = in ? P.cell_of[q] : kNone;
        const uint32_t grp = in ? P.group_of[cell] : kNone;
        hd_stage_at(P, pos, s_own[w]);
        uint32_t cnt[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) cnt[k] = 0;
        uint32_t left = (uint32_t)__ballot(in) & all;
        while (left) {
            const uint32_t g = lane_value(grp, __ffs(left) - 1);
            const uint32_t run = (uint32_t)__ballot(grp == g) & left;
            left &= ~run;
            bool cut;
            (void)hd_count_walk<ROW>(P, g, s_own[w], pos, ~run & all, cnt, s_qb[w], s_beg[w], s_pre[w], lt, ~0u,
                                      &cut);
        }
        uint32_t mine = 0;
#pragma unroll
        for (int k = 0; k < kPch; k++)
            if ((uint32_t)k == l) mine = cnt[k];
        const bool core = in && mine >= minpts;
        if (in) {
            P.core[q] = core;
            P.nrec[q] = (uint8_t)rec_count(mine);
        }
        hd_tally(P, in, cell, core, core ? P.sidx[q] : kNone);
    }
    flush_tests(P, kTestsCore, lt);
}

// ---------------------------------------------------------------------------
// Core marking on byte planes: a wave takes 64 points (two blocks of 32 rows
// of the matrix instruction) and streams candidates 32 at a time through the
// matrix units.
//
// Bound: the matrix and vector rates together.  A tile of 32 rows and columns
// costs four products per step of 32 axes (8 matrix instructions at 64 axes,
// 256 cycles) and four vector instructions per result (about as many cycles),
// which overlap between the two waves of a SIMD; the candidates' bytes (128
// per 64 rows) are the next limit.  Both operands are read as the rows lie in
// memory (a lane's chunk is 16 contiguous bytes) into registers one step of
// 64 candidates ahead.  Sharing each candidate between four waves through
// LDS, with a barrier per step, was slower (86 against 107 ms for the same
// passes).  54 axes, 3.85M points, 1e11 pair tests: 653 ms with two packed
// axes per vector dot product and 8 points per wave, 55 ms here.
//
// A row that needs no further neighbour (it reached minPts, or belongs to
// another run) gets a limit that nothing meets, so hits are met at most a few
// times per point and tile; each is counted through an LDS counter of its row.
// ---------------------------------------------------------------------------
constexpr int kTilePts = 64;
// A run of at most this many points takes its own box to the neighbour list;
// the box of more comes out close to the group's, which the list was built by.
constexpr uint32_t kHdBoxRun = 16;

// Box of the points at the lanes in `mask`, into qb[0, sd) and qb[sd, 2 sd).
__device__ __forceinline__ void hd_rows_box(const Plan &P, uint32_t qpos, uint64_t mask, int32_t *qb)
{
    const uint32_t l = lane_id(), sd = P.sd, col = min(l, sd - 1);
    int32_t lo = INT32_MAX, hi = INT32_MIN;
    while (mask) {
        const uint32_t q = (uint32_t)__ffsll((unsigned long long)mask) - 1;
        mask &= mask - 1;
        const int32_t v = P.spts[(uint64_t)lane_value(qpos, q) * sd + col];
        lo = min(lo, v);
        hi = max(hi, v);
    }
    __builtin_amdgcn_wave_barrier();
    if (l < sd) {
        qb[l] = lo;
        qb[sd + l] = hi;
    }
    __builtin_amdgcn_wave_barrier();
}

// Matrix row r of a lane's 16 results (its half of the wave gives the rest).
__device__ __forceinline__ uint32_t tile_row(uint32_t r, uint32_t half) { return (r & 3u) + 8u * (r >> 2) + 4u * half; }

// Candidates of two tiles of 32 columns: a lane holds its half of the row and
// the negated norm of column l % 32 of each; lane l has the position of
// candidate l of the 64.
template <int KS>
struct HdCols {
    v4i b[2][2 * KS];
    int32_t nq[2];
    uint32_t pos;
};

// The slot that the last looked-up candidate fell in (wave-uniform): its
// candidates [first, end) lie one after the other from sorted position beg.
struct HdSlot {
    uint32_t beg, first, end;
};

// Sorted positions of the candidates c0 .. c0 + 63 (the last one repeated).
__device__ __forceinline__ uint32_t hd_positions(uint32_t c0, uint32_t total, HdSlot &slot, const uint32_t *s_beg,
                                                 const uint32_t *s_pre)
{
    const uint32_t c = min(c0 + lane_id(), total - 1);
    if (min(c0 + kWave, total) <= slot.end) return slot.beg + (c - slot.first);
    const uint32_t ln = candidate_lane(c, s_pre);
    const uint32_t pos = s_beg[ln] + (c - s_pre[ln]);
    const uint32_t last = lane_value(ln, kWave - 1);
    slot.beg = uniform(s_beg[last]);
    slot.first = uniform(s_pre[last]);
    slot.end = last == kWave - 1 ? total : uniform(s_pre[last + 1]);
    return pos;
}

template <int KS>
__device__ __forceinline__ HdCols<KS> hd_cols(const Plan &P, uint32_t c0, uint32_t total, HdSlot &slot,
                                              const uint32_t *s_beg, const uint32_t *s_pre)
{
    const uint32_t l = lane_id();
    HdCols<KS> t;
    t.pos = hd_positions(c0, total, slot, s_beg, s_pre);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const uint32_t pos = __shfl(t.pos, 32 * k + (l & 31u));
        const v4i *row = reinterpret_cast<const v4i *>(P.planes) + (uint64_t)pos * (4 * KS) + (l >> 5) * (2 * KS);
#pragma unroll
        for (int e = 0; e < 2 * KS; e++) t.b[k][e] = row[e];
        t.nq[k] = P.nnorm[pos];
    }
    return t;
}

// 2 p.q - |q|^2 for the 32 x 32 points p (rows) and candidates q (columns):
// 16 results per lane.
template <int KS>
__device__ __forceinline__ void hd_tile(const v4i *a, const v4i *b, int32_t nq, int32_t *v)
{
    v16i hh = {0}, hl = {0}, ll = {0};
#pragma unroll
    for (int st = 0; st < KS; st++) {
        hh = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[st], b[st], hh, 0, 0, 0);
        hl = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[st], b[KS + st], hl, 0, 0, 0);
        ll = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[KS + st], b[KS + st], ll, 0, 0, 0);
        hl = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[KS + st], b[st], hl, 0, 0, 0);
    }
    // three shift-and-adds per result; the empty statements keep the compiler
    // from regrouping them into five instructions
#pragma unroll
    for (int r = 0; r < 16; r++) {
        uint32_t t = ((uint32_t)hh[r] << 8) + (uint32_t)hl[r];
        asm("" : "+v"(t));
        t = (t << 8) + (uint32_t)ll[r];
        asm("" : "+v"(t));
        v[r] = (int32_t)((t << 1) + (uint32_t)nq);
    }
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    return (uint64_t)uniform((uint32_t)(v >> 32)) << 32 | uniform((uint32_t)v);
}

// A wave's rows in LDS: neighbours found so far, the limit each row's results
// are compared with, and the rows' sorted positions.
struct HdRows {
    uint32_t cnt[kTilePts];
    int32_t lim[kTilePts];
    uint32_t pos[kTilePts];
};

// The limits of row block b: result r of a lane belongs to row tile_row(r,
// half), four consecutive rows for four consecutive results.
__device__ __forceinline__ void hd_limits(const HdRows &R, int b, uint32_t half, int32_t *thr)
{
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int4 t = *reinterpret_cast<const int4 *>(&R.lim[32 * b + 8 * j + 4 * half]);
        thr[4 * j] = t.x;
        thr[4 * j + 1] = t.y;
        thr[4 * j + 2] = t.z;
        thr[4 * j + 3] = t.w;
    }
}

// The hits of a tile of row block b, candidate `pos` per lane: every lane
// with a hit takes the next place of its row and records the candidate
// there; rows that reached minPts leave `act`.
__device__ __forceinline__ void hd_hits(const Plan &P, HdRows &R, int b, const int32_t *v, int32_t *thr, uint32_t pos,
                                        bool ok, uint64_t &act)
{
    const uint32_t l = lane_id(), half = l >> 5;
    uint32_t rank[16];
#pragma unroll
    for (int r = 0; r < 16; r++) {
        rank[r] = kNone;
        if (ok && v[r] >= thr[r]) rank[r] = atomicAdd(&R.cnt[32 * b + tile_row(r, half)], 1u);
    }
#pragma unroll
    for (int r = 0; r < 16; r++)
        if (rank[r] < (uint32_t)kRec) P.rec[(uint64_t)R.pos[32 * b + tile_row(r, half)] * kRec + rank[r]] = pos;
    __builtin_amdgcn_wave_barrier();
    const uint64_t done = __ballot(R.cnt[l] >= (uint32_t)P.min_pts) & act;
    if (done) {
        act &= ~done;
        if ((done >> l) & 1) R.lim[l] = INT32_MAX;
        __builtin_amdgcn_wave_barrier();
        hd_limits(R, b, half, thr);
    }
}

// The rows of a wave: counters, limits (INT32_MAX where the row is not in
// act) and positions.
__device__ __forceinline__ void hd_rows_init(HdRows &R, uint64_t act, int32_t lim, uint32_t qpos, uint32_t cnt)
{
    const uint32_t l = lane_id();
    __builtin_amdgcn_wave_barrier();
    R.cnt[l] = cnt;
    R.lim[l] = (act >> l) & 1 ? lim : INT32_MAX;
    R.pos[l] = qpos;
    __builtin_amdgcn_wave_barrier();
}

// The rows of a wave's 64 points as matrix operands.
template <int KS>
__device__ __forceinline__ void hd_load_rows(const Plan &P, uint32_t qpos, v4i (&a)[2][2 * KS])
{
    const uint32_t l = lane_id();
#pragma unroll
    for (int b = 0; b < 2; b++) {
        const uint32_t row = __shfl(qpos, 32 * b + (l & 31u));
        const v4i *src = reinterpret_cast<const v4i *>(P.planes) + (uint64_t)row * (4 * KS) + (l >> 5) * (2 * KS);
#pragma unroll
        for (int e = 0; e < 2 * KS; e++) a[b][e] = src[e];
    }
}

// The points of the lanes in `act` (all of group g) against the group and its
// neighbours, from candidate `from` to candidate `upto` of that list (both
// rounded up to where a step of 64 ends) or until each has minPts neighbours.
// own_box: the list is thinned by the points' own box (and walked whole).
// Returns the points that did not reach minPts; R.cnt has the neighbours.
template <int KS>
__device__ __forceinline__ uint64_t hd_tile_walk(const Plan &P, uint32_t g, uint64_t act, const v4i (&a)[2][2 * KS],
                                                 HdRows &R, bool own_box, int32_t *qb, uint32_t *s_beg,
                                                 uint32_t *s_pre, uint32_t &lt, uint32_t from, uint32_t upto,
                                                 bool *cut)
{
    const uint32_t l = lane_id(), half = l >> 5;
    int32_t thr[2][16];
    hd_limits(R, 0, half, thr[0]);
    hd_limits(R, 1, half, thr[1]);
    const HdSrc src = hd_source(P, g, false);
    uint32_t seen = 0;
    for (uint32_t oc = 0; oc < src.slots && act && seen < upto; oc += kWave) {
        const uint32_t total = uniform(hd_load_neighbours(P, g, src, oc, false, own_box ? qb : nullptr, nullptr, 0u,
                                                          kNone, s_beg, s_pre));
        const uint32_t skip = seen < from ? (from - seen + kWave - 1) / kWave * kWave : 0u;
        if (skip >= total) {
            seen += total;
            continue;
        }
        seen += skip;
        HdSlot slot = {0, 0, 0};
        HdCols<KS> nxt = hd_cols<KS>(P, skip, total, slot, s_beg, s_pre);
        for (uint32_t ci = skip; ci < total && act && seen < upto; ci += kWave) {
            const HdCols<KS> t = nxt;
            // the next 64 rows are on their way while these are tested
            if (ci + kWave < total) nxt = hd_cols<KS>(P, ci + kWave, total, slot, s_beg, s_pre);
            seen += min((uint32_t)kWave, total - ci);
            lt += ci + l < total ? (uint32_t)__popcll(act) : 0u;
#pragma unroll
            for (int k = 0; k < 2; k++) {
                if (ci + 32u * k >= total) break;
#pragma unroll
                for (int b = 0; b < 2; b++) {
                    if (!(uint32_t)(act >> (32 * b))) continue;
                    int32_t v[16];
                    hd_tile<KS>(a[b], t.b[k], t.nq[k], v);
                    // |p - q|^2 <= eps^2 as 2 p.q - |q|^2 >= |p|^2 - eps^2
                    bool any = false;
#pragma unroll
                    for (int r = 0; r < 16; r++) any |= v[r] >= thr[b][r];
                    if (!__ballot(any)) continue;
                    hd_hits(P, R, b, v, thr[b], __shfl(t.pos, 32 * k + (l & 31u)), ci + 32u * k + (l & 31u) < total, act);
                }
            }
        }
    }
    *cut = act && seen >= upto;
    return act;
}

// Core marking takes a few passes.  Each one takes its points to the next
// limit of P.hd_limit (candidates of the point's list); those still undecided
// are listed in order and go on from there in the next pass, so that the
// points of a tile are ones that still need it.
//
// Points a pass starts from: pass 0 all sorted positions, then the lists.
__device__ __forceinline__ uint32_t hd_pass_points(const Plan &P, uint32_t pass)
{
    return pass == 0 ? P.n : ld_agent32(P.ctr->hd_left + pass - 1);
}
__device__ __forceinline__ uint32_t *hd_pass_list(const Plan &P, uint32_t pass)
{
    return pass & 1u ? P.hd_list : P.blist;
}
__device__ __forceinline__ uint32_t hd_pass_point(const Plan &P, uint32_t pass, uint32_t i)
{
    return pass == 0 ? i : hd_pass_list(P, pass)[i];
}

// The units of a pass: runs of at most 64 consecutive points of one group
// within 256 places of the pass' order (pass 0 decides the points of dense
// cubes here).  Edge and noise points are often alone in their group: as
// units of their own they spread over all waves, where a unit of 64 such
// points would walk 64 lists one after the other.
__global__ __launch_bounds__(kBlock) void k_hd_runs(Plan P, uint32_t pass)
{
    if (box_missed(P)) return;
    __shared__ uint64_t s_first[kWavesPerBlock], s_todo[kWavesPerBlock + 1];
    __shared__ uint32_t s_grp[kWavesPerBlock];
    const uint32_t l = lane_id(), w = wave_in_block(), n = hd_pass_points(P, pass), minpts = (uint32_t)P.min_pts;
    const bool last = pass + 1 == P.hd_passes;
    for (uint32_t c0 = blockIdx.x * kBlock; c0 < n; c0 += gridDim.x * kBlock) {
        const uint32_t i = c0 + threadIdx.x, q = hd_pass_point(P, pass, min(i, n - 1));
        const bool in = i < n;
        const uint32_t cell = P.cell_of[q], grp = P.group_of[cell];
        const bool dense = pass == 0 && P.cell_start[cell + 1] - P.cell_start[cell] >= minpts;
        if (pass == 0) {
            if (in && dense) {
                P.core[q] = 1;
                P.nrec[q] = 0;
            }
            hd_tally(P, in, cell, dense, in && dense ? P.sidx[q] : kNone);
        }
        if (!last && l == 0 && in) st_agent(P.hd_mask + i / kWave, 0ull);
        if (l == kWave - 1) s_grp[w] = grp;
        __syncthreads();
        const uint32_t up = __shfl_up(grp, 1), before = l ? up : w ? s_grp[w - 1] : ~grp;
        const uint64_t firsts = __ballot(!in || grp != before), todo = __ballot(in && !dense);
        if (l == 0) {
            s_first[w] = firsts;
            s_todo[w] = todo;
            s_todo[kWavesPerBlock] = 0ull;
        }
        __syncthreads();
        // the group's stretch of these 256 places: its first and end
        uint64_t m = firsts & ((2ull << l) - 1ull);
        uint32_t e = w;
        while (!m && e > 0) m = s_first[--e];
        const uint32_t head = m ? e * kWave + 63u - (uint32_t)__clzll((long long)m) : 0u;
        m = l == kWave - 1 ? 0ull : firsts >> (l + 1) << (l + 1);
        e = w;
        while (!m && ++e < (uint32_t)kWavesPerBlock) m = s_first[e];
        const uint32_t end = m ? e * kWave + (uint32_t)__ffsll((unsigned long long)m) - 1 : (uint32_t)kBlock;
        // every 64th place of it starts a run
        const bool start = in && (threadIdx.x - head) % kTilePts == 0;
        const uint32_t len = min(end - threadIdx.x, (uint32_t)kTilePts);
        uint64_t need = (todo >> l) | (l ? s_todo[w + 1] << (kWave - l) : 0ull);
        if (len < (uint32_t)kTilePts) need &= (1ull << len) - 1ull;
        const bool take = start && need;
        const uint64_t hm = __ballot(take);
        uint32_t base = 0;
        if (l == 0 && hm) base = atomicAdd(P.ctr->hd_runs + pass, (uint32_t)__popcll(hm));
        base = uniform(base);
        if (take) {
            const uint32_t at = base + __popcll(hm & __lanemask_lt());
            P.hd_run_at[at] = i;
            P.hd_run_mask[at] = need;
        }
        __syncthreads();
    }
}

// Units are dealt to an XCD as one stretch of their order, so that its waves
// walk the lists of few groups at a time and share the candidates in its L2;
// a wave whose XCD has none left takes from the next one's.
struct HdQueue {
    uint32_t *cnt;
    uint32_t xcd, left;
};

__device__ __forceinline__ uint32_t hd_next(HdQueue &d, uint32_t units)
{
    while (d.left) {
        uint32_t i = 0;
        if (lane_id() == 0) i = atomicAdd(d.cnt + d.xcd * kCounterStride, 1u);
        i = uniform(i);
        const uint32_t lo = (uint32_t)((uint64_t)units * d.xcd / 8u), hi = (uint32_t)((uint64_t)units * (d.xcd + 1) / 8u);
        if (i < hi - lo) return lo + i;
        d.xcd = (d.xcd + 1) & 7u;
        d.left--;
    }
    return kNone;
}

template <int KS>
__global__ __launch_bounds__(kBlock, 2) void k_hd_core_tiles(Plan P, uint32_t pass)
{
    if (box_missed(P)) return;
    __shared__ __align__(16) HdRows s_rows[kWavesPerBlock];
    __shared__ int32_t s_qb[kWavesPerBlock][2 * kMaxDimHigh];
    __shared__ uint32_t s_beg[kWavesPerBlock][kWave], s_pre[kWavesPerBlock][kWave];
    const uint32_t w = wave_in_block(), l = lane_id(), minpts = (uint32_t)P.min_pts;
    const uint32_t runs = ld_agent32(P.ctr->hd_runs + pass);
    const uint32_t from = pass ? P.hd_limit[pass - 1] : 0u, upto = P.hd_limit[pass];
    const int32_t eps2 = (int32_t)min(P.eps2, (int64_t)INT32_MAX);
    uint32_t lt = 0;
    HdQueue queue = {P.ctr->dyn[pass & 1u ? kDynCoreRest : kDynCore], blockIdx.x & 7u, 8u};
    for (uint32_t u; (u = hd_next(queue, runs)) != kNone;) {
        u = unit_remap(u, runs, P.order);
        const uint32_t i0 = uniform(P.hd_run_at[u]);
        const uint64_t run = uniform64(P.hd_run_mask[u]);
        const bool in = (run >> l) & 1;
        // lanes past the run repeat its last point
        const uint32_t tail = 63u - (uint32_t)__clzll((long long)run);
        const uint32_t q = hd_pass_point(P, pass, i0 + min(l, tail));
        const uint32_t cell = P.cell_of[q], g = uniform(P.group_of[cell]);
        v4i a[2][2 * KS];
        hd_load_rows<KS>(P, q, a);
        HdRows &R = s_rows[w];
        hd_rows_init(R, run, -P.nnorm[q] - eps2, q, pass ? P.hd_cnt[q] : 0u);
        const bool own_box = pass == 0 && __popcll(run) <= kHdBoxRun;
        if (own_box) hd_rows_box(P, q, run, s_qb[w]);
        bool cut;
        const uint64_t rem = hd_tile_walk<KS>(P, g, run, a, R, own_box, s_qb[w], s_beg[w], s_pre[w], lt, from,
                                              own_box ? ~0u : upto, &cut);
        // decided points get their flags and join their cubes' tallies,
        // undecided ones are flagged, for k_hd_left to list in order
        const uint64_t undec = cut ? rem : 0ull;
        const bool later = (undec >> l) & 1;
        const uint32_t cnt = R.cnt[l];
        const bool core = in && cnt >= minpts;
        if (in && !later) {
            P.core[q] = core;
            P.nrec[q] = (uint8_t)rec_count(cnt);
        }
        if (later) P.hd_cnt[q] = cnt;
        if (undec && l == 0) {
            const uint32_t sh = i0 % kWave;
            unsigned long long *word = (unsigned long long *)P.hd_mask + i0 / kWave;
            if (undec << sh) atomicOr(word, (unsigned long long)(undec << sh));
            if (sh && undec >> (kWave - sh)) atomicOr(word + 1, (unsigned long long)(undec >> (kWave - sh)));
        }
        hd_tally(P, in, cell, core, core ? P.sidx[q] : kNone);
    }
    flush_tests(P, kTestsCore, lt);
}

// The points flagged by a pass, in its order, as the next pass' list.  A
// tile of 256 words per block, taken by ticket, with a look-back over earlier
// tiles; the pass' unit queues go back to zero for the pass after the next.
__global__ __launch_bounds__(kBlock) void k_hd_left(Plan P, uint32_t pass)
{
    if (box_missed(P)) return;
    __shared__ uint32_t s_scan[kWavesPerBlock], s_tile;
    __shared__ uint64_t s_base;
    if (blockIdx.x == 0 && threadIdx.x < 8)
        st_agent32(P.ctr->dyn[pass & 1u ? kDynCoreRest : kDynCore] + threadIdx.x * kCounterStride, 0u);
    const uint32_t n = hd_pass_points(P, pass), words = (n + kWave - 1) / kWave, tiles = (words + kBlock - 1) / kBlock;
    uint64_t *status = P.hd_status + (uint64_t)pass * (((uint64_t)P.n + kWave * kBlock - 1) / (kWave * kBlock));
    uint32_t *list = hd_pass_list(P, pass + 1);
    while (true) {
        if (threadIdx.x == 0) s_tile = atomicAdd(P.ctr->hd_tickets + pass, 1u);
        __syncthreads();
        const uint32_t tile = s_tile;
        if (tile >= tiles) return;
        const uint32_t word = tile * kBlock + threadIdx.x;
        uint64_t m = word < words ? ld_agent(P.hd_mask + word) : 0ull;
        uint32_t sum;
        const uint32_t pre = block_exclusive_scan<uint32_t>((uint32_t)__popcll(m), s_scan, &sum);
        if (threadIdx.x == 0) {
            s_base = scan_lookback(status, tile, sum);
            if (tile == tiles - 1) st_agent32(P.ctr->hd_left + pass, (uint32_t)s_base + sum);
        }
        __syncthreads();
        uint32_t at = (uint32_t)s_base + pre;
        while (m) {
            const uint32_t i = word * kWave + (uint32_t)__ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            list[at++] = hd_pass_point(P, pass, i);
        }
        __syncthreads();
    }
}

// First cube with a core point of every group (kNone: none).  A group's cubes
// are consecutive, so only the first of a wave's core cubes in each group is
// offered (an atomic per core cube had groups of 10^4 cubes queue up on one
// address: 2.8 ms at 3.4M core cubes, 0.07 ms this way).
__global__ __launch_bounds__(kBlock) void k_hd_gcore(Plan P)
{
    if (box_missed(P)) return;
    const uint32_t nc = ld_agent32(&P.ctr->n_cells);
    for (uint32_t base = blockIdx.x * kBlock; base < nc; base += gridDim.x * kBlock) {
        const uint32_t c = base + threadIdx.x;
        const bool core = c < nc && P.ncore[c] > 0;
        const uint32_t g = core ? P.group_of[c] : kNone;
        const uint64_t earlier = __ballot(core) & __lanemask_lt();
        const uint32_t prev = __shfl(g, earlier ? 63 - __clzll((long long)earlier) : 0);
        if (core && (!earlier || prev != g)) atomicMin(P.gcube + g, c);
    }
}

// ---------------------------------------------------------------------------
// Merging (Definitions 3-5): every pair of core points within eps joins its
// two cubes.  Each core point of a chunk walks its own group and the groups
// after it (the forward entries), so every pair of cubes is seen from the
// smaller one; roots are cached and a batch of candidates is skipped when no
// pair in it could join two different sets.
// ---------------------------------------------------------------------------
template <int ROW>
__device__ __forceinline__ void hd_link_walk(const Plan &P, uint32_t g, const int32_t (*own)[kOwnStride],
                                             uint32_t run, const uint32_t *ck, int32_t *qb, uint32_t *s_beg,
                                             uint32_t *s_pre, uint32_t &lt)
{
    const uint32_t l = lane_id();
    hd_chunk_box(P, own, run, qb);
    const HdSrc src = hd_source(P, g, true);
    uint32_t rk[kPch];
#pragma unroll
    for (int k = 0; k < kPch; k++) rk[k] = (run & (1u << k)) ? uf_find(P.parent, ck[k]) : kNone;
    for (uint32_t oc = 0; oc < src.slots; oc += kWave) {
        // the root all the walking points share, if they do
        uint32_t common = kNone;
        bool one = true;
#pragma unroll
        for (int k = 0; k < kPch; k++) {
            if (!(run & (1u << k))) continue;
            if (common == kNone) common = rk[k];
            else one = one && rk[k] == common;
        }
        if (!one) common = kNone;
        const uint32_t total = hd_load_neighbours(P, g, src, oc, true, qb, own, run, common, s_beg, s_pre);
        for (uint32_t ci = 0; ci < total; ci += kWave) {
            const uint32_t c = ci + l;
            bool ok = c < total;
            const uint32_t pos = ok ? hd_candidate(c, s_beg, s_pre) : 0u;
            ok = ok && P.core[pos];
            const uint32_t cq = ok ? P.cell_of[pos] : 0u;
            uint32_t rq = ok ? uf_find(P.parent, cq) : kNone;
            bool any = false;
#pragma unroll
            for (int k = 0; k < kPch; k++)
                if (run & (1u << k)) any |= ok && cq > ck[k] && rq != rk[k];
            if (!__ballot(any)) continue;
            int64_t dd[kPch];
            hd_dist<ROW>(P, own, pos, dd);
#pragma unroll
            for (int k = 0; k < kPch; k++) {
                if (!(run & (1u << k))) continue;
                lt += ok;
                const bool need = ok && cq > ck[k] && rq != rk[k] && dd[k] <= P.eps2;
                if (__ballot(need)) {
                    if (need) uf_union(P.parent, ck[k], cq);
                    rq = ok ? uf_find(P.parent, cq) : kNone;
#pragma unroll
                    for (int k2 = 0; k2 < kPch; k2++)
                        if (run & (1u << k2)) rk[k2] = uf_find(P.parent, ck[k2]);
                }
            }
        }
    }
}

// After the recorded pairs are joined: the whole walk, where a group whose
// core cubes all share the walking points' root is skipped without looking
// at its points.
template <int ROW>
__global__ __launch_bounds__(kBlock) void k_hd_merge(Plan P)
{
    if (box_missed(P)) return;
    __shared__ __align__(16) int32_t s_own[kWavesPerBlock][kPch][kOwnStride];
    __shared__ int32_t s_qb[kWavesPerBlock][2 * kMaxDimHigh];
    __shared__ uint32_t s_beg[kWavesPerBlock][kWave], s_pre[kWavesPerBlock][kWave];
    const uint32_t w = wave_in_block(), l = lane_id();
    const uint32_t n = P.n, all = (1u << kPch) - 1u;
    uint32_t lt = 0;
    const DynRange dr_ = dyn_range(P.ctr->dyn[kDynMerge], P.order);
    HCA_FOR_UNITS_DYN(u, (n + kPch - 1) / kPch, dr_) {
        const uint32_t pc = u * kPch, np = min((uint32_t)kPch, n - pc);
        bool core = l < np && P.core[pc + l];
        const uint32_t cell = core ? P.cell_of[pc + l] : kNone;
        const uint32_t grp = core ? P.group_of[cell] : kNone;
        core = core && P.groot[grp];
        const uint32_t live = (uint32_t)__ballot(core) & all;
        if (!live) continue;
        uint32_t ck[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) ck[k] = lane_value(cell, k);
        hd_stage(P, pc, np, s_own[w]);
        uint32_t left = live;
        while (left) {
            const uint32_t g = lane_value(grp, __ffs(left) - 1);
            const uint32_t run = (uint32_t)__ballot(grp == g) & left;
            left &= ~run;
            hd_link_walk<ROW>(P, g, s_own[w], run, ck, s_qb[w], s_beg[w], s_pre[w], lt);
        }
    }
    flush_tests(P, kTestsMerge, lt);
}

// The pairs recorded by core marking: each core point joins its cube with those of its
// recorded core neighbours (all within eps), no test needed.  The records,
// then the flags and cubes of all of them, are loaded before the first
// union, so their latencies overlap; the point's own root is carried from
// one union to the next.
template <bool TOP>
__device__ __forceinline__ void link_point(const Plan &P, uint32_t q)
{
    if (!P.core[q]) return;
    const uint32_t c = P.cell_of[q], nr = min((uint32_t)P.nrec[q], (uint32_t)kRec);
    if (!nr) return;
    uint32_t q2[kRec];
    const uint4 *rp = reinterpret_cast<const uint4 *>(P.rec + (uint64_t)q * kRec);
#pragma unroll
    for (int i = 0; i < kRec / 4; i++) {
        const uint4 v = rp[i];
        q2[4 * i] = v.x;
        q2[4 * i + 1] = v.y;
        q2[4 * i + 2] = v.z;
        q2[4 * i + 3] = v.w;
    }
    // cube of each recorded core neighbour (kNone: not core, or past nr,
    // where the record holds no position)
    uint32_t c2[kRec];
#pragma unroll
    for (int r = 0; r < kRec; r++) {
        c2[r] = kNone;
        if ((uint32_t)r < nr) {
            const bool cp = P.core[q2[r]];
            const uint32_t cc = P.cell_of[q2[r]];
            c2[r] = cp ? cc : kNone;
        }
    }
    uint32_t rc = kNone;
#pragma unroll
    for (int r = 0; r < kRec; r++) {
        if (c2[r] == kNone || c2[r] == c) continue;
        if (rc == kNone) rc = uf_find<TOP>(P.parent, c);
        // rc was c's root when found and stays an ancestor of c, so a
        // neighbour under rc is already in c's cluster
        const uint32_t r2 = uf_find<TOP>(P.parent, c2[r]);
        if (r2 == rc) continue;
        uf_union<TOP>(P.parent, rc, r2);
        rc = uf_find<TOP>(P.parent, rc);
    }
}

__global__ __launch_bounds__(kBlock) void k_link_recorded(Plan P)
{
    if (box_missed(P)) return;
    for (uint32_t q = blockIdx.x * kBlock + threadIdx.x; q < P.n; q += gridDim.x * kBlock) link_point<false>(P, q);
}

// The same over the points of sparse cubes, where core marking has listed
// them (the others have nothing recorded).  Cubes take the find that stores
// once per call, as in their merging (2-D, 4M points: 261 -> 189 us).
template <bool TOP>
__global__ __launch_bounds__(kBlock) void k_link_listed(Plan P)
{
    if (box_missed(P)) return;
    const uint32_t ns = ld_agent32(&P.ctr->n_sparse);
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < ns; i += gridDim.x * kBlock) link_point<TOP>(P, P.core_list[i]);
}

// Before the walk: whether all core cubes of each group share one root (a
// thread per cube; the flag starts as "yes").
__global__ __launch_bounds__(kBlock) void k_hd_unify(Plan P)
{
    if (box_missed(P)) return;
    const uint32_t nc = ld_agent32(&P.ctr->n_cells);
    for (uint32_t c = blockIdx.x * kBlock + threadIdx.x; c < nc; c += gridDim.x * kBlock) {
        if (!P.ncore[c]) continue;
        const uint32_t g = P.group_of[c], first = P.gcube[g];
        if (c != first && uf_find(P.parent, c) != uf_find(P.parent, first)) P.unified[g] = 0;
    }
}

// Then the groups whose points have to walk at all (groot = 1): not when the
// group's core cubes and those of every group after it in its list share one
// root.  On blobs the recorded pairs have joined nearly everything, and the
// walk is left with the few groups at the seams (54 axes, 3.85M points: merge
// 36.9 ms with every core point walking, 4.5 ms this way).
__global__ __launch_bounds__(kBlock) void k_hd_need(Plan P)
{
    if (box_missed(P)) return;
    const uint32_t l = lane_id(), ng = ld_agent32(&P.ctr->n_groups);
    const WaveRange hca_wr_ = wave_range(P.order);
    HCA_FOR_UNITS(g, ng) {
        const uint32_t first = uniform(P.gcube[g]);
        bool need = false;
        if (first != kNone) {
            need = !P.unified[g];
            const uint32_t r = uf_find(P.parent, first), at = P.nbr_start[g], cnt = P.nbr_count[g];
            for (uint32_t j = 0; j < cnt && !need; j += kWave) {
                bool other = false;
                if (j + l < cnt) {
                    const uint32_t G = P.nbr[at + j + l], f = P.gcube[G];
                    other = f != kNone && !(P.unified[G] && uf_find(P.parent, f) == r);
                }
                need = __ballot(other) != 0;
            }
        }
        if (l == 0) P.groot[g] = need;
    }
}

// ---------------------------------------------------------------------------
// Border points: each non-core point of a chunk takes the root of its nearest
// core point within eps (ties to the smaller input index); none -> noise.
// ---------------------------------------------------------------------------
template <int ROW>
__device__ __forceinline__ void hd_border_walk(const Plan &P, uint32_t g, const int32_t (*own)[kOwnStride],
                                               uint32_t todo, int64_t *bd, uint32_t *bi, uint32_t *bp, int32_t *qb,
                                               uint32_t *s_beg, uint32_t *s_pre, uint32_t &lt)
{
    const uint32_t l = lane_id();
    const int64_t eps2 = P.eps2;
    hd_chunk_box(P, own, todo, qb);
    const HdSrc src = hd_source(P, g, false);
    for (uint32_t oc = 0; oc < src.slots; oc += kWave) {
        const uint32_t total = hd_load_neighbours(P, g, src, oc, true, qb, own, todo, kNone, s_beg, s_pre);
        for (uint32_t ci = 0; ci < total; ci += kWave) {
            const uint32_t c = ci + l;
            bool ok = c < total;
            const uint32_t pos = ok ? hd_candidate(c, s_beg, s_pre) : 0u;
            ok = ok && P.core[pos];
            if (!__ballot(ok)) continue;
            int64_t dd[kPch];
            hd_dist<ROW>(P, own, pos, dd);
            bool near = false;
#pragma unroll
            for (int k = 0; k < kPch; k++) {
                if (todo & (1u << k)) lt += ok;
                near |= (todo & (1u << k)) && ok && dd[k] <= eps2 && dd[k] <= bd[k];
            }
            if (!near) continue;
            const uint32_t qi = P.sidx[pos];
#pragma unroll
            for (int k = 0; k < kPch; k++) {
                if (!(todo & (1u << k))) continue;
                if (ok && dd[k] <= eps2 && (dd[k] < bd[k] || (dd[k] == bd[k] && qi < bi[k]))) {
                    bd[k] = dd[k];
                    bi[k] = qi;
                    bp[k] = pos;
                }
            }
        }
    }
}

// Non-core points whose neighbours were all recorded: the nearest core point
// among them (exact 64-bit distances over the int32 rows), one thread per point.
__global__ __launch_bounds__(kBlock) void k_hd_border_rec(Plan P)
{
    if (box_missed(P)) return;
    const uint32_t sd = P.sd;
    for (uint32_t p = blockIdx.x * kBlock + threadIdx.x; p < P.n; p += gridDim.x * kBlock) {
        if (P.core[p] || !rec_complete(P, p)) continue;
        const int32_t *a = P.spts + (uint64_t)p * sd;
        int64_t bd = INT64_MAX;
        uint32_t bi = kNone, bq = kNone;
        for (uint32_t r = 0, nr = P.nrec[p]; r < nr; r++) {
            const uint32_t q = P.rec[(uint64_t)p * kRec + r];
            if (!P.core[q]) continue;
            const int32_t *b = P.spts + (uint64_t)q * sd;
            int64_t dd = 0;
            for (uint32_t e = 0; e < sd; e++) {
                const int64_t t = (int64_t)a[e] - b[e];
                dd += t * t;
            }
            const uint32_t qi = P.sidx[q];
            if (dd < bd || (dd == bd && qi < bi)) { bd = dd; bi = qi; bq = q; }
        }
        finish_owner(P, p, bq);
    }
}

// Chunks of 8 non-core points of the list.  Each takes the root of its
// nearest core point within eps (ties to the smaller input index) and offers
// its input index to that cluster's smallest member; none -> noise.
template <int ROW>
__global__ __launch_bounds__(kBlock) void k_hd_border(Plan P)
{
    if (box_missed(P)) return;
    __shared__ __align__(16) int32_t s_own[kWavesPerBlock][kPch][kOwnStride];
    __shared__ int32_t s_qb[kWavesPerBlock][2 * kMaxDimHigh];
    __shared__ uint32_t s_beg[kWavesPerBlock][kWave], s_pre[kWavesPerBlock][kWave];
    const uint32_t w = wave_in_block(), l = lane_id();
    const uint32_t nl = ld_agent32(&P.ctr->n_blist);
    const uint32_t *list = P.blist;
    // a short list: one point per wave, so that the walks run side by side
    const uint32_t per = nl >= (uint32_t)kPch * gridDim.x * kWavesPerBlock ? (uint32_t)kPch : 1u;
    uint32_t lt = 0;
    const DynRange dr_ = dyn_range(P.ctr->dyn[kDynBorder], P.order);
    HCA_FOR_UNITS_DYN(u, (nl + per - 1) / per, dr_) {
        const uint32_t b0 = u * per, np = min(per, nl - b0);
        uint32_t pos[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) pos[k] = list[b0 + min((uint32_t)k, np - 1)];
        uint32_t q = pos[0];
#pragma unroll
        for (int k = 1; k < kPch; k++)
            if ((uint32_t)k == l) q = pos[k];
        const bool in = l < np;
        const uint32_t todo = (uint32_t)__ballot(in) & ((1u << kPch) - 1u);
        const uint32_t grp = in ? P.group_of[P.cell_of[q]] : kNone;
        hd_stage_at(P, pos, s_own[w]);
        int64_t bd[kPch];
        uint32_t bi[kPch], bp[kPch];
#pragma unroll
        for (int k = 0; k < kPch; k++) { bd[k] = INT64_MAX; bi[k] = kNone; bp[k] = kNone; }
        uint32_t left = todo;
        while (left) {
            const uint32_t g = lane_value(grp, __ffs(left) - 1);
            const uint32_t run = (uint32_t)__ballot(grp == g) & left;
            left &= ~run;
            hd_border_walk<ROW>(P, g, s_own[w], run, bd, bi, bp, s_qb[w], s_beg[w], s_pre[w], lt);
        }
#pragma unroll
        for (int k = 0; k < kPch; k++) {
            if (!(todo & (1u << k))) continue;
            int64_t d0 = bd[k];
            uint32_t i0 = bi[k], q0 = bp[k];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const int64_t d1 = __shfl_xor(d0, o);
                const uint32_t i1 = __shfl_xor(i0, o), q1 = __shfl_xor(q0, o);
                if (d1 < d0 || (d1 == d0 && i1 < i0)) { d0 = d1; i0 = i1; q0 = q1; }
            }
            if (l == 0) {
                const uint32_t root = q0 == kNone ? kNone : ld_parent(P.parent + P.cell_of[q0]);
                P.owner[pos[k]] = root;
                if (root != kNone) {
                    const uint32_t me = P.sidx[pos[k]];
                    if (me < ld_agent32(P.minmem + root)) atomicMin(P.minmem + root, me);
                }
            }
        }
    }
    flush_tests(P, kTestsBorder, lt);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
void launch_link_recorded(const Plan &P, hipStream_t s)
{
    const int cb = (int)std::min<uint64_t>((P.n + kBlock - 1) / kBlock, 2048);
    if (P.core_list && P.m == 1) hipLaunchKernelGGL(k_link_listed<true>, dim3(cb), dim3(kBlock), 0, s, P);
    else if (P.core_list) hipLaunchKernelGGL(k_link_listed<false>, dim3(cb), dim3(kBlock), 0, s, P);
    else hipLaunchKernelGGL(k_link_recorded, dim3(cb), dim3(kBlock), 0, s, P);
}

void launch_hd_lists(const Plan &P, int blocks, hipStream_t s)
{
    const int ib = (int)std::min<uint64_t>((P.n + kBlock - 1) / kBlock, 1024);
    hipLaunchKernelGGL(k_hd_group_init, dim3(ib), dim3(kBlock), 0, s, P);
    hipLaunchKernelGGL(k_hd_group_box, dim3(blocks), dim3(kBlock), 0, s, P);
    switch (P.kd) {
    case 1: hipLaunchKernelGGL(k_hd_lists<1>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case 2: hipLaunchKernelGGL(k_hd_lists<2>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case 3: hipLaunchKernelGGL(k_hd_lists<3>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case 4: hipLaunchKernelGGL(k_hd_lists<4>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case 5: hipLaunchKernelGGL(k_hd_lists<5>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case 6: hipLaunchKernelGGL(k_hd_lists<6>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case 7: hipLaunchKernelGGL(k_hd_lists<7>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case 8: hipLaunchKernelGGL(k_hd_lists<8>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    }
    launch_lists_back(P, blocks, s);
}

template <int KS>
static void launch_hd_core_tiles(const Plan &P, hipStream_t s)
{
    const uint32_t words = (P.n + kTilePts - 1) / kTilePts;
    // two waves fit a SIMD: 512 workgroups of four fill the chip
    const int tb = (int)std::min<uint64_t>(512u, (((uint64_t)P.n + kWavesPerBlock - 1) / kWavesPerBlock + 7u) & ~7ull);
    const int lb = (int)std::min<uint32_t>((words + kBlock - 1) / kBlock, 256u);
    const int rb = (int)std::min<uint32_t>((P.n + kBlock - 1) / kBlock, 2048u);
    for (uint32_t pass = 0; pass < P.hd_passes; pass++) {
        hipLaunchKernelGGL(k_hd_runs, dim3(rb), dim3(kBlock), 0, s, P, pass);
        hipLaunchKernelGGL(k_hd_core_tiles<KS>, dim3(tb), dim3(kBlock), 0, s, P, pass);
        if (pass + 1 < P.hd_passes) hipLaunchKernelGGL(k_hd_left, dim3(lb), dim3(kBlock), 0, s, P, pass);
    }
}

static void launch_hd_planes(const Plan &P, hipStream_t s)
{
    const uint64_t chunks = (uint64_t)P.n * 2 * P.hd_steps;
    const int pb = (int)std::min<uint64_t>((chunks + kBlock - 1) / kBlock, 4096);
    if (P.hd_steps == 1) hipLaunchKernelGGL(k_hd_planes<1>, dim3(pb), dim3(kBlock), 0, s, P);
    else hipLaunchKernelGGL(k_hd_planes<2>, dim3(pb), dim3(kBlock), 0, s, P);
}

void launch_hd_core(const Plan &P, int blocks, hipStream_t s)
{
    if (P.planes && P.hd_tiles) {
        launch_hd_planes(P, s);
        if (P.hd_steps == 1) launch_hd_core_tiles<1>(P, s);
        else launch_hd_core_tiles<2>(P, s);
    } else {
        switch (row_form(P)) {
        case kRowWide:
            hipLaunchKernelGGL(k_hd_core<kRowWide>, dim3(blocks), dim3(kBlock), 0, s, P);
            hipLaunchKernelGGL(k_hd_core_rest<kRowWide>, dim3(blocks), dim3(kBlock), 0, s, P);
            break;
        case kRowPacked:
            hipLaunchKernelGGL(k_hd_core<kRowPacked>, dim3(blocks), dim3(kBlock), 0, s, P);
            hipLaunchKernelGGL(k_hd_core_rest<kRowPacked>, dim3(blocks), dim3(kBlock), 0, s, P);
            break;
        default:
            hipLaunchKernelGGL(k_hd_core<kRowNarrow>, dim3(blocks), dim3(kBlock), 0, s, P);
            hipLaunchKernelGGL(k_hd_core_rest<kRowNarrow>, dim3(blocks), dim3(kBlock), 0, s, P);
        }
    }
    const int cb = (int)std::min<uint64_t>((P.n + kBlock - 1) / kBlock, 1024);
    hipLaunchKernelGGL(k_hd_gcore, dim3(cb), dim3(kBlock), 0, s, P);
}

void launch_hd_merge(const Plan &P, int blocks, hipStream_t s)
{
    launch_link_recorded(P, s);
    const int cb = (int)std::min<uint64_t>((P.n + kBlock - 1) / kBlock, 2048);
    hipLaunchKernelGGL(k_hd_unify, dim3(cb), dim3(kBlock), 0, s, P);
    hipLaunchKernelGGL(k_hd_need, dim3(blocks), dim3(kBlock), 0, s, P);
    switch (row_form(P)) {
    case kRowWide: hipLaunchKernelGGL(k_hd_merge<kRowWide>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case kRowPacked: hipLaunchKernelGGL(k_hd_merge<kRowPacked>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    default: hipLaunchKernelGGL(k_hd_merge<kRowNarrow>, dim3(blocks), dim3(kBlock), 0, s, P);
    }
}

void launch_hd_border(const Plan &P, int blocks, hipStream_t s)
{
    const int cb = (int)std::min<uint64_t>((P.n + kBlock - 1) / kBlock, 2048);
    hipLaunchKernelGGL(k_hd_border_rec, dim3(cb), dim3(kBlock), 0, s, P);
    launch_border_list(P, s);
    switch (row_form(P)) {
    case kRowWide: hipLaunchKernelGGL(k_hd_border<kRowWide>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    case kRowPacked: hipLaunchKernelGGL(k_hd_border<kRowPacked>, dim3(blocks), dim3(kBlock), 0, s, P); break;
    default: hipLaunchKernelGGL(k_hd_border<kRowNarrow>, dim3(blocks), dim3(kBlock), 0, s, P);
    }
}

}  // namespace hca
