// Most-bound-particle halo centres (paper Sec. 2.2).
//
// For every particle of a halo, phi_i = -sum_{j in halo, j != i} m_j /
// sqrt(|x_j - x_i|^2 + eps^2), and per halo the particle with the smallest
// phi.  All pairs inside a halo, no cutoff: every evaluated pair is useful.
//
// Halos of more than kSymMin particles evaluate every pair once
// (k_centre_sym, below).  The others' work items are (halo, up to 128
// targets), heaviest first, pulled by
// persistent one-wave workgroups.  A wave stages 64 sources of its halo at a
// time in LDS (the next 64 are loaded into registers meanwhile) and every
// lane sums the staged sources for its targets: one target per lane, two
// per lane for items of more than 64 targets, or 2^lk lanes per target for
// halos of fewer than 64 particles.  Pair terms are float32; every 8 terms
// are added to a float64 accumulator, so the rounding does not grow with the
// halo size.  Each item also reduces its targets to a (phi, index) minimum,
// and a second pass takes the minimum over a halo's items.  The order of
// every sum is fixed by the item table, so results are bitwise reproducible.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "sr_internal.h"

namespace sr {
namespace {

constexpr float kFarAway = 1.0e18f;  // padding source: contributes m q = 0 * q
constexpr int kTargetsPerWave = 64;

// Workspace header: the condition word first (read by sr_ws_flags, like a
// force workspace's), the queue counter on its own 128-byte line.
struct CentreHeader {
    uint32_t flags;
    uint32_t pad0[31];
    uint32_t next;  // queue counter
    uint32_t pad1[31];
    uint32_t next_sym;  // queue counter of the pair-once items
    uint32_t pad2[31];
};

// Item: x = halo, y = first target, z = targets, w = lk | two << 4 | slot << 5.
__device__ __forceinline__ int4 uniform_item(const int4 *__restrict__ items, uint32_t g)
{
    const int4 it = items[g];
    return make_int4(__builtin_amdgcn_readfirstlane(it.x), __builtin_amdgcn_readfirstlane(it.y),
                     __builtin_amdgcn_readfirstlane(it.z), __builtin_amdgcn_readfirstlane(it.w));
}

// Source j of a halo as (x, y, z, m); past the end: far away and massless.
__device__ __forceinline__ float4 load_source(const float *__restrict__ pos,
                                              const float *__restrict__ mass, int j, int end)
{
    if (j < end) {
        const int64_t p = 3 * (int64_t)j;
        return make_float4(pos[p], pos[p + 1], pos[p + 2], mass[j]);
    }
    return make_float4(kFarAway, kFarAway, kFarAway, 0.f);
}

// m_j / sqrt(|d|^2 + eps^2), added to g.  Without softening a pair at zero
// distance (the target itself, or a coincident particle) adds nothing.
template <bool kSoft>
__device__ __forceinline__ float pot_term(const float4 s, float px, float py, float pz, float eps2,
                                          float g)
{
    const float dx = s.x - px, dy = s.y - py, dz = s.z - pz;
    const float t = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2)));
    float q = __builtin_amdgcn_rsqf(t);
    if (!kSoft) q = t > 0.f ? q : 0.f;
    return fmaf(s.w, q, g);
}

struct MinIdx {
    float v;
    int i;
};

__device__ __forceinline__ bool better(float v, int i, float w, int j)
{
    // smaller phi first, then the smaller index; a NaN never wins against a number
    if (v < w) return true;
    if (v == w) return i < j;
    return !(v == v) ? false : !(w == w);
}

__device__ __forceinline__ MinIdx wave_argmin(float v, int i)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const float w = __shfl_xor(v, o);
        const int j = __shfl_xor(i, o);
        if (better(w, j, v, i)) {
            v = w;
            i = j;
        }
    }
    return MinIdx{v, i};
}

// Sums over the 64 staged sources.  `self*` is the stage index of the
// target itself in this chunk, or -1.  Groups of 8 float32 terms go into the
// float64 accumulators.

// One target per lane.
template <bool kSoft, bool kSelf>
__device__ __forceinline__ void sum_dense(const float4 *stage, float px, float py, float pz,
                                          float eps2, int self, double &acc)
{
    for (int k = 0; k < kTargetsPerWave; k += 8) {
        // even and odd sources in two float32 partial sums: two independent
        // FMA chains instead of one
        float g0 = 0.f, g1 = 0.f;
#pragma unroll
        for (int u = 0; u < 8; u += 2) {
            const float t0 = pot_term<kSoft>(stage[k + u], px, py, pz, eps2, g0);
            const float t1 = pot_term<kSoft>(stage[k + u + 1], px, py, pz, eps2, g1);
            g0 = (kSelf && k + u == self) ? g0 : t0;
            g1 = (kSelf && k + u + 1 == self) ? g1 : t1;
        }
        acc += (double)(g0 + g1);
    }
}

// Two targets per lane: each staged source is read once for both.
template <bool kSoft, bool kSelf>
__device__ __forceinline__ void sum_two(const float4 *stage, float ax, float ay, float az, float bx,
                                        float by, float bz, float eps2, int self_a, int self_b,
                                        double &acc_a, double &acc_b)
{
    for (int k = 0; k < kTargetsPerWave; k += 8) {
        // per target, even and odd sources in two float32 partial sums
        float ga0 = 0.f, ga1 = 0.f, gb0 = 0.f, gb1 = 0.f;
#pragma unroll
        for (int u = 0; u < 8; u += 2) {
            const float4 s0 = stage[k + u], s1 = stage[k + u + 1];
            const float ta0 = pot_term<kSoft>(s0, ax, ay, az, eps2, ga0);
            const float tb0 = pot_term<kSoft>(s0, bx, by, bz, eps2, gb0);
            const float ta1 = pot_term<kSoft>(s1, ax, ay, az, eps2, ga1);
            const float tb1 = pot_term<kSoft>(s1, bx, by, bz, eps2, gb1);
            ga0 = (kSelf && k + u == self_a) ? ga0 : ta0;
            gb0 = (kSelf && k + u == self_b) ? gb0 : tb0;
            ga1 = (kSelf && k + u + 1 == self_a) ? ga1 : ta1;
            gb1 = (kSelf && k + u + 1 == self_b) ? gb1 : tb1;
        }
        acc_a += (double)(ga0 + ga1);
        acc_b += (double)(gb0 + gb1);
    }
}

// 2^lk lanes per target (lk >= 1): lane sub takes stage entries sub, sub + 2^lk, ...
template <bool kSoft, bool kSelf>
__device__ __forceinline__ void sum_sparse(const float4 *stage, int lk, int sub, float px,
                                           float py, float pz, float eps2, int self, double &acc)
{
    const int kl = 1 << lk;
    const int per = kTargetsPerWave >> lk;  // 1 .. 32
    for (int k = 0; k < per; k += 8) {
        float g = 0.f;
        for (int u = 0; u < 8 && k + u < per; ++u) {
            const int at = (k + u) * kl + sub;
            const float t = pot_term<kSoft>(stage[at], px, py, pz, eps2, g);
            g = (kSelf && at == self) ? g : t;
        }
        acc += (double)g;
    }
}

template <bool kSoft>
__global__ __launch_bounds__(64, 4) void k_centre_potential(
    const int4 *__restrict__ items, uint32_t n_items, const int *__restrict__ hoff,
    const float *__restrict__ pos, const float *__restrict__ mass, float eps2,
    float *__restrict__ phi, int2 *__restrict__ partial, CentreHeader *hdr, int64_t pull_limit)
{
    __shared__ float4 stage[kTargetsPerWave];
    const int lane = threadIdx.x;
    // Loop bound: the counter hands out increasing values, so one wave's
    // items increase strictly and it cannot pull more than exist.  A pull
    // that breaks either rule ends the loop and flags the workspace instead
    // of spinning; pull_limit below the item count (a test hook) ends every
    // wave early on purpose.
    const int64_t limit = min((int64_t)n_items, pull_limit);
    int64_t pulls = 0, last = -1;
    bool bad = false;
    for (;;) {
        // Lane 0 takes the next item; the loop body below ends with no other
        // lane-0-only branch, so the compiler cannot merge the two into one
        // region across the loop's back edge (which would let the other
        // lanes start the next iteration without lane 0's new item).
        uint32_t g = 0;
        if (lane == 0) g = atomicAdd(&hdr->next, 1u);
        g = __builtin_amdgcn_readfirstlane(g);
        if (g >= n_items) break;
        if ((int64_t)g <= last || ++pulls > limit) {
            bad = true;
            break;
        }
        last = g;
        const int4 it = uniform_item(items, g);
        const int h = it.x, t0 = it.y, nt = it.z, lk = it.w & 15;
        const bool two = (it.w >> 4) & 1;
        const int slot = it.w >> 5;
        const int s0 = __builtin_amdgcn_readfirstlane(hoff[h]);
        const int s1 = __builtin_amdgcn_readfirstlane(hoff[h + 1]);
        const int kl = 1 << lk;
        const int tsub = lane >> lk, sub = lane & (kl - 1);
        // targets of this lane: a = t0 + tsub (dense: tsub = lane), b = a + 64
        const bool va = tsub < min(nt, kTargetsPerWave);
        const bool vb = two && lane + kTargetsPerWave < nt;
        const int ia = t0 + tsub, ib = t0 + kTargetsPerWave + lane;
        float ax = 0.f, ay = 0.f, az = 0.f, bx = 0.f, by = 0.f, bz = 0.f;
        if (va) {
            ax = pos[3 * (int64_t)ia];
            ay = pos[3 * (int64_t)ia + 1];
            az = pos[3 * (int64_t)ia + 2];
        }
        if (vb) {
            bx = pos[3 * (int64_t)ib];
            by = pos[3 * (int64_t)ib + 1];
            bz = pos[3 * (int64_t)ib + 2];
        }
        double acc_a = 0.0, acc_b = 0.0;
        float4 next = load_source(pos, mass, s0 + lane, s1);
        // Chunks start at s0 + 64 m and items at s0 + 128 k, so the targets'
        // own entries are in the chunks starting at t0 (a) and t0 + 64 (b).
        for (int base = s0; base < s1; base += kTargetsPerWave) {
            __syncthreads();
            stage[lane] = next;
            __syncthreads();
            if (base + kTargetsPerWave < s1) next = load_source(pos, mass, base + kTargetsPerWave + lane, s1);
            const bool own_a = base == t0, own_b = base == t0 + kTargetsPerWave;
            if (two) {
                if (own_a || own_b)
                    sum_two<kSoft, true>(stage, ax, ay, az, bx, by, bz, eps2, own_a ? lane : -1,
                                         own_b ? lane : -1, acc_a, acc_b);
                else
                    sum_two<kSoft, false>(stage, ax, ay, az, bx, by, bz, eps2, -1, -1, acc_a, acc_b);
            } else if (lk == 0) {
                if (own_a)
                    sum_dense<kSoft, true>(stage, ax, ay, az, eps2, lane, acc_a);
                else
                    sum_dense<kSoft, false>(stage, ax, ay, az, eps2, -1, acc_a);
            } else {
                if (own_a)
                    sum_sparse<kSoft, true>(stage, lk, sub, ax, ay, az, eps2, tsub, acc_a);
                else
                    sum_sparse<kSoft, false>(stage, lk, sub, ax, ay, az, eps2, -1, acc_a);
            }
        }
        // combine the lanes of a target (sparse items), in a fixed order
        for (int o = 1; o < kl; o <<= 1) acc_a += __shfl_xor(acc_a, o);
        const float pa = (float)(-acc_a), pb = (float)(-acc_b);
        if (va && sub == 0) phi[ia] = pa;
        if (vb) phi[ib] = pb;
        // minimum of the item's targets
        float v = __builtin_inff();
        int idx = 0x7fffffff;
        if (va && sub == 0) {
            v = pa;
            idx = ia;
        }
        if (vb && better(pb, ib, v, idx)) {
            v = pb;
            idx = ib;
        }
        // every lane holds the same minimum: all store it (one address)
        const MinIdx m = wave_argmin(v, idx);
        partial[slot] = make_int2(__float_as_int(m.v), m.i);
    }
    if (bad && lane == 0) atomicOr(&hdr->flags, (uint32_t)SR_FLAG_QUEUE);
}

// ------------------------------------------------------- every pair once
//
// m_j q and m_i q of a pair share the distance, so a halo of n particles needs
// n^2 / 2 of them: its particles are cut into superblocks of B, and an item is
// a pair of superblocks I <= J.  For each window of kSymWin sources of J the
// item takes the target blocks of I, two targets per lane, and meets them with
// tiles of 64 sources: at step s lane l takes source (l + s) mod 64, and the
// running sum of the opposite terms moves one lane down after the step.  Each
// staged source serves two pairs per lane and each rotation two opposite
// terms.  Every four terms the float32 sums go into float64: a target's after
// four steps, in registers, a source's after two, in LDS (after four, eight
// terms, it was 3% faster but a halo of some hundred particles lay 3.0e-8 from
// the float64 sums instead of 2.7e-8 with both ends summed one by one).
// Inside a superblock a block meets only later sources, and itself from both
// ends.  Float64 partial sums go to rows of slots, one per partner superblock
// (row J of particle i: its sum over superblock J; the last row: what the
// blocks of its own superblock before its own added), and k_centre_sum adds
// the rows in a fixed order: results are bitwise reproducible.
// Bound by issue: 85 vector instructions (8 of them rsq) per 8 unordered pairs
// and lane, against 17 per pair for both ends one by one; and a halo's work is
// cut along both axes, where an item of 128 targets walked all its sources.
// 2,000 halos of 40 to 86,000 particles (1.65e10 ordered pairs): 7.1 -> 2.5 ms
// a run, 6.7e12 ordered pairs per second (2.3e12 before).
constexpr int kSymMin = 256;    // halos above this many particles (one superblock), where it pays: see pair_once_pays
constexpr int kSymWin = 512;    // sources per window: 4 KB of float64 sums
constexpr int kSymBlock = 2 * kWave;
constexpr int kSumThreads = 256;

// Tables of the pair-once halos, in plan order (largest first).
struct SymTables {
    int halos, B;
    const int *halo;          // [halos] the halo
    const int *first;         // [halos + 1] first item
    const int *chunk;         // [halos + 1] first chunk of kSumThreads particles
    const long long *slot;    // [halos] first slot (doubles)
};

// Largest k with first[k] <= x (x uniform).
__device__ __forceinline__ int table_find(const int *__restrict__ first, int n, int x)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <bool kSoft>
__device__ __forceinline__ float pair_q(const float4 s, float px, float py, float pz, float eps2)
{
    const float dx = s.x - px, dy = s.y - py, dz = s.z - pz;
    const float t = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2)));
    const float q = __builtin_amdgcn_rsqf(t);
    return kSoft ? q : (t > 0.f ? q : 0.f);
}

__device__ __forceinline__ float lane_down(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x134, 0xf, 0xf, false));
}

template <bool kSoft>
__global__ __launch_bounds__(64, 4) void k_centre_sym(SymTables tab, uint32_t n_items, const int *__restrict__ hoff,
                                                      const float *__restrict__ pos, const float *__restrict__ mass,
                                                      float eps2, double *__restrict__ slots, CentreHeader *hdr,
                                                      int64_t pull_limit)
{
    __shared__ float4 tile[2 * kWave];
    __shared__ double red[kSymWin];
    const int lane = threadIdx.x;
    const uint32_t limit = (uint32_t)min((int64_t)n_items, pull_limit);
    uint32_t pulls = 0, least = 0;
    bool bad = false;
    // the first item is the wave's own, the counter hands out those after them
    // (the loop bound and the lane-0 rule are those of k_centre_potential)
    for (uint32_t g = blockIdx.x;;) {
        if (pulls > 0) {
            uint32_t c = 0;
            if (lane == 0) c = atomicAdd(&hdr->next_sym, 1u);
            g = gridDim.x + __builtin_amdgcn_readfirstlane(c);
        }
        if (g >= n_items) break;
        if (g < least || ++pulls > limit) {
            bad = true;
            break;
        }
        least = g + 1u;
        const int k = table_find(tab.first, tab.halos, (int)g);
        const int h = tab.halo[k];
        const int s0 = hoff[h], n = hoff[h + 1] - s0;
        const int rows = (n + tab.B - 1) / tab.B;
        // item t of the halo: the pair I <= J with t = J (J + 1) / 2 + I
        const int t = (int)g - tab.first[k];
        int J = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
        while (J * (J + 1) / 2 > t) --J;
        while ((J + 1) * (J + 2) / 2 <= t) ++J;
        J = __builtin_amdgcn_readfirstlane(J);
        const int I = t - J * (J + 1) / 2;
        const bool diag = I == J;
        const int i0 = I * tab.B, i1 = min(n, i0 + tab.B), j0 = J * tab.B, j1 = min(n, j0 + tab.B);
        double *tout = slots + tab.slot[k] + (int64_t)J * n;
        double *sout = slots + tab.slot[k] + (int64_t)(diag ? rows : I) * n;
        for (int w0 = j0; w0 < j1; w0 += kSymWin) {
            const int w1 = min(j1, w0 + kSymWin);
            for (int i = lane; i < kSymWin; i += kWave) red[i] = 0.0;
            __syncthreads();
            for (int p = i0; p < i1; p += kSymBlock) {
                const int ia = p + lane, ib = ia + kWave;
                const float4 ta = load_source(pos, mass, s0 + ia, s0 + n), tb = load_source(pos, mass, s0 + ib, s0 + n);
                double acc_a = 0.0, acc_b = 0.0;
                if (diag && p >= w0 && p < w1) {
                    // the block against itself, both ends of every pair; s = 0 meets the lane's own entry
                    for (int c = 0; c < 2; ++c) {
                        __syncthreads();
                        tile[lane] = tile[lane + kWave] = c == 0 ? ta : tb;
                        __syncthreads();
                        const float4 *src = tile + lane;
                        for (int s = 0; s < kWave; s += 4) {
                            float ga = 0.f, gb = 0.f;
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const float4 sj = src[s + u];
                                const float na = fmaf(sj.w, pair_q<kSoft>(sj, ta.x, ta.y, ta.z, eps2), ga);
                                const float nb = fmaf(sj.w, pair_q<kSoft>(sj, tb.x, tb.y, tb.z, eps2), gb);
                                const bool own = s + u == 0;
                                ga = own && c == 0 ? ga : na;
                                gb = own && c == 1 ? gb : nb;
                            }
                            acc_a += (double)ga;
                            acc_b += (double)gb;
                        }
                    }
                }
                const int js = diag ? max(w0, p + kSymBlock) : w0;
                if (js < w1) {
                    float4 next = load_source(pos, mass, s0 + js + lane, s0 + w1);
                    for (int base = js; base < w1; base += kWave) {
                        __syncthreads();
                        tile[lane] = tile[lane + kWave] = next;
                        __syncthreads();
                        if (base + kWave < w1) next = load_source(pos, mass, s0 + base + kWave + lane, s0 + w1);
                        const float4 *src = tile + lane;
                        double *r = red + (base - w0);
                        int at = lane + 1;  // source whose sum the lane holds after two steps
                        for (int s = 0; s < kWave; s += 4) {
                            float ga = 0.f, gb = 0.f, b = 0.f;
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const float4 sj = src[s + u];
                                const float qa = pair_q<kSoft>(sj, ta.x, ta.y, ta.z, eps2);
                                const float qb = pair_q<kSoft>(sj, tb.x, tb.y, tb.z, eps2);
                                if (u & 1) b = lane_down(b);
                                ga = fmaf(sj.w, qa, ga);
                                gb = fmaf(sj.w, qb, gb);
                                b = fmaf(ta.w, qa, b);
                                b = fmaf(tb.w, qb, b);
                                if (u & 1) {
                                    // an LDS atomic, since other lanes add to the entry before and after;
                                    // one lane per entry and instruction, so the order of sums is fixed
                                    __hip_atomic_fetch_add(&r[at & (kWave - 1)], (double)b, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                                    b = 0.f;
                                    at += 2;
                                }
                            }
                            acc_a += (double)ga;
                            acc_b += (double)gb;
                        }
                    }
                }
                if (w0 == j0) {
                    if (ia < n) tout[ia] = acc_a;
                    if (ib < n) tout[ib] = acc_b;
                } else {
                    if (ia < n) tout[ia] += acc_a;
                    if (ib < n) tout[ib] += acc_b;
                }
            }
            __syncthreads();
            for (int i = lane; i < w1 - w0; i += kWave) sout[w0 + i] = red[i];
            __syncthreads();
        }
    }
    if (bad && lane == 0) atomicOr(&hdr->flags, (uint32_t)SR_FLAG_QUEUE);
}

// phi of a chunk of kSumThreads particles of a pair-once halo: its rows added
// in order; and the chunk's minimum.
__global__ __launch_bounds__(kSumThreads) void k_centre_sum(SymTables tab, const int *__restrict__ hoff,
                                                            const int *__restrict__ hbase,
                                                            const double *__restrict__ slots,
                                                            float *__restrict__ phi, int2 *__restrict__ partial)
{
    __shared__ int2 best[kSumThreads / kWave];
    const int k = table_find(tab.chunk, tab.halos, (int)blockIdx.x);
    const int c = (int)blockIdx.x - tab.chunk[k];
    const int h = tab.halo[k];
    const int s0 = hoff[h], n = hoff[h + 1] - s0;
    const int rows = (n + tab.B - 1) / tab.B + 1;
    const int i = c * kSumThreads + (int)threadIdx.x;
    float v = __builtin_inff();
    int idx = 0x7fffffff;
    if (i < n) {
        const double *p = slots + tab.slot[k] + i;
        double acc = 0.0;
        int r = 0;
        for (; r + 4 <= rows; r += 4, p += 4 * (int64_t)n) {
            const double x0 = p[0], x1 = p[(int64_t)n], x2 = p[2 * (int64_t)n], x3 = p[3 * (int64_t)n];
            acc = (((acc + x0) + x1) + x2) + x3;
        }
        for (; r < rows; ++r, p += n) acc += *p;
        v = (float)(-acc);
        idx = s0 + i;
        phi[idx] = v;
    }
    const MinIdx m = wave_argmin(v, idx);
    if ((threadIdx.x & (kWave - 1)) == 0) best[threadIdx.x / kWave] = make_int2(__float_as_int(m.v), m.i);
    __syncthreads();
    if (threadIdx.x != 0) return;
    int2 b = best[0];
    for (int w = 1; w < kSumThreads / kWave; ++w)
        if (better(__int_as_float(best[w].x), best[w].y, __int_as_float(b.x), b.y)) b = best[w];
    partial[hbase[h] + c] = b;
}

// Per halo: the best of its items' minima (one wave per halo).
__global__ __launch_bounds__(256) void k_centre_argmin(const int2 *__restrict__ partial,
                                                       const int *__restrict__ hbase, int n_halos,
                                                       int64_t *__restrict__ mbp,
                                                       float *__restrict__ phi_min)
{
    const int lane = threadIdx.x & 63;
    const int h = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (h >= n_halos) return;  // whole waves leave together
    const int a = hbase[h], b = hbase[h + 1];
    float v = __builtin_inff();
    int idx = 0x7fffffff;
    for (int s = a + lane; s < b; s += 64) {
        const int2 p = partial[s];
        const float w = __int_as_float(p.x);
        if (better(w, p.y, v, idx)) {
            v = w;
            idx = p.y;
        }
    }
    const MinIdx m = wave_argmin(v, idx);
    if (lane == 0) {
        const bool found = a < b && m.i != 0x7fffffff;  // none when every phi is NaN
        mbp[h] = found ? (int64_t)m.i : -1;
        if (phi_min) phi_min[h] = found ? m.v : 0.f;
    }
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace
}  // namespace sr

using namespace sr;

struct sr_centres_plan {
    int32_t H = 0;
    int64_t n = 0;
    int64_t n_items = 0;
    // pair-once halos: their number, superblock size, items and chunks
    int n_sym = 0, sym_block = 0;
    int64_t sym_items = 0, sym_chunks = 0;
    size_t off_hoff = 0, off_hbase = 0, off_items = 0, off_sym_halo = 0, off_sym_first = 0, off_sym_chunk = 0,
           off_sym_slot = 0, off_partial = 0, off_slots = 0, upload_bytes = 0, ws_bytes = 0;
    std::vector<char> image;  // header + hoff + hbase + items, uploaded by every run
    char *pinned = nullptr;   // its pinned copy, made by the first run
    int num_cu = 0;
};

namespace {

// The halos that evaluate every pair once, largest first, and their superblock
// size.  A smaller B cuts more items and keeps more slots, 8 B per particle and
// partner superblock, so B rises where the slots of 256 would be some 128 MB
// (4e9 ordered pairs) and those of 512 some 500 MB (3e10): each step halves
// them and costs up to a sixth of the time at its line, nothing well above it
// (256 / 512 / 1024, ms: 10 halos of 20,000 particles 0.60 / 0.67 / 0.95, 50 2.61
// / 2.64 / 3.2, 75 3.87 / 3.85 / 4.47, 150 7.49 / 7.49 / 8.0; one of 170,000 3.68 /
// 3.62 / 3.90, of 300,000 11.2 each).  Then it doubles (to kSymMaxBlock at most,
// items of a few ms) while the rows do not fit kSlotBytes, and then the halos are
// taken from the largest on as each fits; the others go to the one-sided items.
// A halo whose rows alone do not fit (more than 737,460 particles) is one-sided from the
// start, so that it does not decide the others' B.  Beside such a halo the
// others go pair-once only if that is clearly shorter, by a count of the time
// of both ways: its items of 128 targets against every source last long and
// leave waves idle (7,565 of 8,192 for 968,359 particles, 208 ms), which the
// others' one-sided items fill, whereas their pair-once items, at 0.7 of the
// time a pair, come before and have a tail of their own.  One-sided against
// pair-once, by the count's ratio: 968,359 with 300 of 20,000 particles 224 /
// 226 ms (1.04), with 30 of 100,000 254 / 259 (0.99), two of 800,000 with 400 of
// 30,000 325 / 328 (0.93), the node catalogue (968,359 the largest of 1,923)
// 347 / 328 ms (0.91).
constexpr double kSlotBytes = 1073741824.0;
constexpr int kSymMaxBlock = 4096;
constexpr double kSymPairTime = 0.7;
constexpr double kSymClear = 0.92;
constexpr double kOneSidedWaves = 8192.0;  // 32 per CU

// Whether the pair-once items of `fit` are worth their two launches in a
// catalogue whose one-sided items (at most one per wave) would be few: a count
// of the microseconds of both ways.  One-sided: the longest item, 47 ns a source
// while few waves share a SIMD, and the queue and the pairs of all items.
// Pair-once: two launches and the longest item of 256 targets and sources, some
// 35 us, the items beyond the first 1,280, and the halos of up to kSymMin in a
// launch of their own.  One-sided against pair-once, us: 300 halos of 20 to 300
// particles 31 / 54, of 20 to 2,000 192 / 119; 100 of 500 40 / 48, 500 of 500
// 90 / 63; one of 600 39 / 42, one of 800 48 / 42.  On 93 such catalogues the
// count takes the slower way by more than 2% once (600 halos of 20 to 700, 86 /
// 92).
bool pair_once_pays(int n_halos, const int64_t *offsets, const std::vector<int> &fit, int block)
{
    constexpr double kSource = 0.047, kItem = 0.015, kItemSource = 2.1e-5, kTwoLaunches = 35.0, kOnceItem = 0.02,
                     kOnceFree = 1280.0, kLaunch = 6.0;
    struct Cost {
        double longest = 0.0, items = 0.0, time = 0.0;
        void add(double n)
        {
            const double k = std::ceil(n / (2 * kTargetsPerWave));
            longest = std::max(longest, n);
            items += k;
            time += k * (kItem + kItemSource * n);
        }
        double us() const { return kSource * longest + time; }
    } all, rest;
    std::vector<char> once(n_halos, 0);
    double sym = 0.0;
    for (const int h : fit) {
        const double r = std::ceil((double)(offsets[h + 1] - offsets[h]) / block);
        once[h] = 1;
        sym += r * (r + 1.0) / 2.0;
    }
    for (int h = 0; h < n_halos; ++h) {
        const double n = (double)(offsets[h + 1] - offsets[h]);
        all.add(n);
        if (!once[h]) rest.add(n);
    }
    if (all.items > kOneSidedWaves) return true;
    const double split = kTwoLaunches + kOnceItem * std::max(0.0, sym - kOnceFree) +
                         (rest.items > 0.0 ? kLaunch + rest.us() : 0.0);
    return split < all.us();
}

std::vector<int> pair_once_halos(int n_halos, const int64_t *offsets, int &block)
{
    const auto rows = [&](int h, int B) { return (double)((offsets[h + 1] - offsets[h] + B - 1) / B); };
    const auto bytes = [&](int h, int B) { return 8.0 * (double)(offsets[h + 1] - offsets[h]) * (rows(h, B) + 1.0); };
    std::vector<int> sym;
    double pairs = 0.0, all_pairs = 0.0, longest = 0.0;  // longest: the items of halos that do not fit
    for (int h = 0; h < n_halos; ++h) {
        const double nh = (double)(offsets[h + 1] - offsets[h]);
        all_pairs += nh * nh;
        if (nh <= kSymMin) continue;
        if (bytes(h, kSymMaxBlock) > kSlotBytes) {
            longest = std::max(longest, 2.0 * kTargetsPerWave * nh);
            continue;
        }
        sym.push_back(h);
        pairs += nh * nh;
    }
    std::stable_sort(sym.begin(), sym.end(), [&](int a, int b) {
        return offsets[a + 1] - offsets[a] > offsets[b + 1] - offsets[b];
    });
    const auto all_bytes = [&](int B) {
        double b = 0.0;
        for (const int h : sym) b += bytes(h, B);
        return b;
    };
    block = pairs >= 3.0e10 ? 1024 : (pairs >= 4.0e9 ? 512 : 256);
    while (block < kSymMaxBlock && all_bytes(block) > kSlotBytes) block *= 2;
    // halos that fit, and items that fit 32-bit counters
    double used = 0.0, items = 0.0, once = 0.0;
    std::vector<int> fit;
    for (const int h : sym) {
        const double r = rows(h, block), b = bytes(h, block);
        const double it = r * (r + 1.0) / 2.0;
        if (used + b > kSlotBytes || items + it > 1.0e9) continue;
        used += b;
        items += it;
        once += (double)(offsets[h + 1] - offsets[h]) * (double)(offsets[h + 1] - offsets[h]);
        fit.push_back(h);
    }
    const auto one_sided = [&](double p) { return std::max(p / kOneSidedWaves, longest); };
    const double split = one_sided(all_pairs - once) + kSymPairTime * once / kOneSidedWaves;
    if (longest > 0.0 && split > kSymClear * one_sided(all_pairs)) fit.clear();
    if (!fit.empty() && !pair_once_pays(n_halos, offsets, fit, block)) fit.clear();
    return fit;
}

int device_cus()
{
    int dev = 0, cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cu;
}

}  // namespace

extern "C" {

sr_status sr_centres_plan_create(int32_t n_halos, const int64_t *offsets, sr_centres_plan **plan,
                                 size_t *ws_bytes)
{
    if (!plan || !ws_bytes || !offsets || n_halos < 1 || n_halos > (1 << 26)) return SR_E_ARG;
    *plan = nullptr;
    if (offsets[0] != 0) return SR_E_ARG;
    for (int h = 0; h < n_halos; ++h)
        if (offsets[h + 1] < offsets[h]) return SR_E_ARG;
    const int64_t n = offsets[n_halos];
    if (n > (int64_t(1) << 31) - 1) return SR_E_UNSUPPORTED;
    // an item's word holds its slot among the partial minima in 26 bits: every halo
    // counts as its one-sided items, at least as many as a pair-once halo has chunks
    int64_t most = 0;
    for (int h = 0; h < n_halos; ++h)
        most += (offsets[h + 1] - offsets[h] + 2 * kTargetsPerWave - 1) / (2 * kTargetsPerWave);
    if (most > (int64_t(1) << 26)) return SR_E_UNSUPPORTED;
    // items of each halo: up to 128 targets (two per lane), a last group of at
    // most 64 one per lane, halos under 64 with 2^lk lanes per target
    struct Item {
        int h, t0, nt, w;
        double cost;
    };
    std::vector<Item> items;
    std::vector<int> hbase(n_halos + 1, 0);
    int sym_block = 0;
    const std::vector<int> sym = pair_once_halos(n_halos, offsets, sym_block);
    std::vector<char> once(n_halos, 0);
    for (const int h : sym) once[h] = 1;
    for (int h = 0; h < n_halos; ++h) {
        const int64_t nh = offsets[h + 1] - offsets[h];
        if (once[h]) {  // one minimum per chunk of k_centre_sum
            hbase[h + 1] = hbase[h] + (int)((nh + kSumThreads - 1) / kSumThreads);
            continue;
        }
        int chunk = 0;
        for (int64_t t = 0; t < nh;) {
            const int64_t left = nh - t;
            const int nt = (int)std::min<int64_t>(left, left > kTargetsPerWave ? 2 * kTargetsPerWave
                                                                              : kTargetsPerWave);
            int lk = 0;
            while ((nt << (lk + 1)) <= kTargetsPerWave) ++lk;
            const int two = nt > kTargetsPerWave ? 1 : 0;
            items.push_back(Item{h, (int)(offsets[h] + t), nt, lk | (two << 4), 0.0});
            items.back().cost = (double)nh * (two ? 2.0 : 1.0) / (double)(1 << lk);
            t += nt;
            ++chunk;
        }
        hbase[h + 1] = hbase[h] + chunk;
    }
    // slot = position of the item inside its halo's range, fixed before sorting
    for (size_t k = 0, h = 0, c = 0; k < items.size(); ++k) {
        if ((int)h != items[k].h) {
            h = items[k].h;
            c = 0;
        }
        items[k].w |= (int)(hbase[h] + c) << 5;
        ++c;
    }
    std::stable_sort(items.begin(), items.end(), [](const Item &a, const Item &b) { return a.cost > b.cost; });
    auto *P = new sr_centres_plan;
    P->H = n_halos;
    P->n = n;
    P->n_items = (int64_t)items.size();
    size_t o = align256(sizeof(CentreHeader));
    P->off_hoff = o;
    o = align256(o + sizeof(int) * (n_halos + 1));
    P->off_hbase = o;
    o = align256(o + sizeof(int) * (n_halos + 1));
    P->off_items = o;
    o = align256(o + sizeof(int4) * std::max<size_t>(1, items.size()));
    P->n_sym = (int)sym.size();
    P->sym_block = sym_block;
    P->off_sym_halo = o;
    o = align256(o + sizeof(int) * (sym.size() + 1));
    P->off_sym_first = o;
    o = align256(o + sizeof(int) * (sym.size() + 1));
    P->off_sym_chunk = o;
    o = align256(o + sizeof(int) * (sym.size() + 1));
    P->off_sym_slot = o;
    o = align256(o + sizeof(long long) * (sym.size() + 1));
    P->upload_bytes = o;
    P->off_partial = o;
    o = align256(o + sizeof(int2) * std::max<size_t>(1, (size_t)hbase[n_halos]));
    P->off_slots = o;
    P->image.assign(P->upload_bytes, 0);
    {
        int *halo = reinterpret_cast<int *>(P->image.data() + P->off_sym_halo);
        int *first = reinterpret_cast<int *>(P->image.data() + P->off_sym_first);
        int *chunk = reinterpret_cast<int *>(P->image.data() + P->off_sym_chunk);
        long long *slot = reinterpret_cast<long long *>(P->image.data() + P->off_sym_slot);
        int64_t at = 0;
        for (size_t k = 0; k < sym.size(); ++k) {
            const int64_t nh = offsets[sym[k] + 1] - offsets[sym[k]], rows = (nh + sym_block - 1) / sym_block;
            halo[k] = sym[k];
            first[k] = (int)P->sym_items;
            chunk[k] = (int)P->sym_chunks;
            slot[k] = at;
            P->sym_items += rows * (rows + 1) / 2;
            P->sym_chunks += (nh + kSumThreads - 1) / kSumThreads;
            at += nh * (rows + 1);
        }
        o = align256(o + sizeof(double) * (size_t)at);
    }
    P->ws_bytes = o;
    int *hoff = reinterpret_cast<int *>(P->image.data() + P->off_hoff);
    for (int h = 0; h <= n_halos; ++h) hoff[h] = (int)offsets[h];
    std::memcpy(P->image.data() + P->off_hbase, hbase.data(), sizeof(int) * (n_halos + 1));
    int4 *it = reinterpret_cast<int4 *>(P->image.data() + P->off_items);
    for (size_t k = 0; k < items.size(); ++k) it[k] = make_int4(items[k].h, items[k].t0, items[k].nt, items[k].w);
    *plan = P;
    *ws_bytes = P->ws_bytes;
    return SR_OK;
}

sr_status sr_centres_plan_destroy(sr_centres_plan *P)
{
    if (!P) return SR_E_PLAN;
    if (P->pinned) (void)hipHostFree(P->pinned);
    delete P;
    return SR_OK;
}

sr_status sr_centres(sr_centres_plan *P, const float *pos, const float *mass, float eps, void *ws,
                     size_t ws_bytes, float *phi, int64_t *mbp, float *phi_min, void *stream)
{
    if (!P) return SR_E_PLAN;
    if (!(eps >= 0.f) || !std::isfinite(eps) || !mbp) return SR_E_ARG;
    if (P->n > 0 && (!pos || !mass || !phi)) return SR_E_ARG;
    if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 != 0 || ws_bytes < P->ws_bytes) return SR_E_WORKSPACE;
    if (P->num_cu <= 0 && (P->num_cu = device_cus()) <= 0) return SR_E_DEVICE;
    if (!P->pinned) {
        if (hipHostMalloc((void **)&P->pinned, P->upload_bytes, hipHostMallocDefault) != hipSuccess) {
            P->pinned = nullptr;
            return SR_E_DEVICE;
        }
        std::memcpy(P->pinned, P->image.data(), P->upload_bytes);
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *w = static_cast<char *>(ws);
    // tables and a zeroed queue counter, from pinned memory
    if (hipMemcpyAsync(w, P->pinned, P->upload_bytes, hipMemcpyHostToDevice, s) != hipSuccess)
        return SR_E_DEVICE;
    const int *hoff = reinterpret_cast<const int *>(w + P->off_hoff);
    const int *hbase = reinterpret_cast<const int *>(w + P->off_hbase);
    const int4 *items = reinterpret_cast<const int4 *>(w + P->off_items);
    int2 *partial = reinterpret_cast<int2 *>(w + P->off_partial);
    CentreHeader *hdr = reinterpret_cast<CentreHeader *>(w);
    const float eps2 = eps * eps;
    int64_t limit = INT64_MAX;
    if (const char *v = std::getenv("SR_PULL_LIMIT"))
        if (std::atoll(v) >= 0) limit = std::atoll(v);
    const SymTables tab{P->n_sym, P->sym_block, reinterpret_cast<const int *>(w + P->off_sym_halo),
                        reinterpret_cast<const int *>(w + P->off_sym_first),
                        reinterpret_cast<const int *>(w + P->off_sym_chunk),
                        reinterpret_cast<const long long *>(w + P->off_sym_slot)};
    double *slots = reinterpret_cast<double *>(w + P->off_slots);
    if (P->sym_items > 0) {
        const unsigned grid = (unsigned)std::min<int64_t>(P->sym_items, (int64_t)P->num_cu * 16);
        if (eps2 > 0.f)
            k_centre_sym<true><<<grid, 64, 0, s>>>(tab, (uint32_t)P->sym_items, hoff, pos, mass, eps2, slots, hdr, limit);
        else
            k_centre_sym<false><<<grid, 64, 0, s>>>(tab, (uint32_t)P->sym_items, hoff, pos, mass, 0.f, slots, hdr, limit);
        if (hipGetLastError() != hipSuccess) return SR_E_DEVICE;
        k_centre_sum<<<(unsigned)P->sym_chunks, kSumThreads, 0, s>>>(tab, hoff, hbase, slots, phi, partial);
        if (hipGetLastError() != hipSuccess) return SR_E_DEVICE;
    }
    if (P->n_items > 0) {
        const int64_t grid = std::min<int64_t>(P->n_items, (int64_t)P->num_cu * 32);
        if (eps2 > 0.f)
            k_centre_potential<true><<<(unsigned)grid, 64, 0, s>>>(items, (uint32_t)P->n_items, hoff, pos,
                                                                 mass, eps2, phi, partial, hdr, limit);
        else
            k_centre_potential<false><<<(unsigned)grid, 64, 0, s>>>(items, (uint32_t)P->n_items, hoff, pos,
                                                                  mass, 0.f, phi, partial, hdr, limit);
        if (hipGetLastError() != hipSuccess) return SR_E_DEVICE;
    }
    k_centre_argmin<<<(unsigned)((P->H + 3) / 4), 256, 0, s>>>(partial, hbase, P->H, mbp, phi_min);
    return hipGetLastError() == hipSuccess ? SR_OK : SR_E_DEVICE;
}

}  // extern "C"
