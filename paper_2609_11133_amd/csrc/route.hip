// Routing kernels of the MoE decode step: router logits, top-k softmax and the
// token-to-expert grouping.  One decode step of a MoE layer starts here (the decode
// lane of the paper's Background section; the MoE models of its Experimental Setup).
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>

#include <type_traits>

#include "fp8split.h"
#include "moe_internal.h"
#include "wave.h"

namespace moe {
namespace {

constexpr int kWave = 64;
constexpr int kThreads = 256;  // threads per workgroup of every routing kernel

// Values exchanged between workgroups of this kernel (logits, selected experts) are
// written and read with device-scope atomic stores and loads, which bypass the
// per-XCD L2 caches; a producer waits for its stores to complete before it bumps a
// counter.  This avoids whole-cache write-back / invalidate fences, which serialise
// per XCD.
template <typename T>
__device__ inline void st_dev(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ inline T ld_dev(const T *p) { return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// The memory clobber keeps the compiler from moving memory accesses across the wait,
// so every store issued before it has completed when the counter is bumped.
__device__ inline void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ------------------------------------------------------------------ router logits
//
// Canonical logit: one round-to-nearest-even to fp32 of the exact value of
// sum_h x[h] * w[h] + b.  Products of bf16 or fp32 operands are exact in fp64.
// Fast path: each lane sums its products in fp64 (one FMA each) together with
// sum |x*w|; the wave combines lanes by a butterfly.  Every product then passes
// through at most D roundings (D = products per lane + 6 butterfly levels + 1 for
// the bias), so |sum - exact| <= gamma_D * (sum|x*w| + |b|), gamma_D = D u/(1-D u),
// u = 2^-53.  If the interval sum +- bound (plus one fp64 ulp of slack) lies
// strictly between the two fp32 rounding midpoints around RNE(sum), every value in
// it rounds to the same fp32 number, which is then the canonical logit.  Otherwise
// the wave recomputes the sum in double-double (error-free TwoSum accumulation,
// about 106 significant bits) and rounds hi + lo with the tie resolved by lo.

__device__ inline double bf16_to_f64(uint32_t bits16) { return (double)__uint_as_float(bits16 << 16); }

__device__ inline void two_sum(double a, double b, double &s, double &e)
{
    s = a + b;
    double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// (h, l) += (h2, l2); symmetric in its operands, so butterfly partners agree.
__device__ inline void dd_add(double &h, double &l, double h2, double l2)
{
    double s, e;
    two_sum(h, h2, s, e);
    e += l + l2;
    h = s + e;
    l = e - (h - s);
}

// Round hi + lo (|lo| <= ulp(hi)/2) to fp32, nearest, ties to even.
__device__ inline float round_dd_to_f32(double hi, double lo)
{
    float r = (float)hi;
    double rd = (double)r;
    if (rd == hi) return r;
    float other = hi > rd ? nextafterf(r, INFINITY) : nextafterf(r, -INFINITY);
    double mid = 0.5 * (rd + (double)other);
    if (hi != mid || lo == 0.0) return r;  // not a tie, or an exact tie already resolved to even
    return ((lo > 0.0) == ((double)other > rd)) ? other : r;
}

// True if every real number within `bound` of v rounds to the same fp32 value r: rounding
// is monotonic, so it does if both ends of an interval that contains them do (the slack
// covers the ends' own fp64 rounding).
// `up` is the value that the upper end rounds to: at least every such number's.
__device__ inline bool certain_f32(double v, double bound, float &r, float &up)
{
    const double m = bound + fabs(v) * 0x1p-51;
    r = (float)(v - m);
    up = (float)(v + m);
    return r == up;
}

template <typename T>
__device__ inline void load8(const T *p, double (&v)[8]);

template <>
__device__ inline void load8<uint16_t>(const uint16_t *p, double (&v)[8])
{
    uint4 q = *reinterpret_cast<const uint4 *>(p);
    uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = bf16_to_f64(w[i] & 0xFFFFu);
        v[2 * i + 1] = bf16_to_f64(w[i] >> 16);
    }
}

template <>
__device__ inline void load8<float>(const float *p, double (&v)[8])
{
    float4 a = *reinterpret_cast<const float4 *>(p);
    float4 b = *reinterpret_cast<const float4 *>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// The lanes' double-double sums and the bias b, added and rounded.
__device__ __attribute__((always_inline)) inline float wave_dd_to_f32(double hi, double lo, double b)
{
    double nh = hi + lo;  // normalise the lane's pair before combining
    lo = lo - (nh - hi);
    hi = nh;
#pragma unroll
    for (int o = kWave / 2; o >= 1; o >>= 1) {
        double h2 = __shfl_xor(hi, o), l2 = __shfl_xor(lo, o);
        dd_add(hi, lo, h2, l2);
    }
    dd_add(hi, lo, b, 0.0);
    return round_dd_to_f32(hi, lo);
}

// Exact (double-double) logit of one (token, expert) pair, computed by one wave: the
// slow path taken when the fp64 sum cannot certify its fp32 rounding.
template <typename XT, typename WT>
__device__ __attribute__((always_inline)) inline float wave_logit_exact(const XT *__restrict__ xr, const WT *__restrict__ wrow, double b, int H,
                                         int lane)
{
    double hi = 0.0, lo = 0.0;
    for (int h = lane * 8; h < H; h += 512) {
        double xv[8], wv[8];
        load8<XT>(xr + h, xv);
        load8<WT>(wrow + h, wv);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            double p = xv[i] * wv[i], ss, ee;  // exact product
            two_sum(hi, p, ss, ee);
            hi = ss;
            lo += ee;
        }
    }
    return wave_dd_to_f32(hi, lo, b);
}

// Eight consecutive inputs of one lane, as raw bits (bf16: 4 words, fp32: 8 words).
template <typename T>
struct Chunk8 {
    uint32_t d[sizeof(T) == 2 ? 4 : 8];
};

template <typename T>
__device__ inline void ld_chunk(const T *p, Chunk8<T> &c)
{
#pragma unroll
    for (int q = 0; q < (int)(sizeof(c.d) / 16); ++q) {
        const uint4 u = reinterpret_cast<const uint4 *>(p)[q];
        c.d[4 * q] = u.x;
        c.d[4 * q + 1] = u.y;
        c.d[4 * q + 2] = u.z;
        c.d[4 * q + 3] = u.w;
    }
}

template <typename T>
__device__ inline double elem(const Chunk8<T> &c, int i)
{
    if constexpr (sizeof(T) == 2)
        return (double)__uint_as_float((i & 1) ? (c.d[i >> 1] & 0xFFFF0000u) : (c.d[i >> 1] << 16));
    else
        return (double)__uint_as_float(c.d[i]);
}

// wave_logit_exact with up to 4096 inputs of each row in flight at a time: where one wave's
// recomputation ends the step, the round trips are what it costs.  Routing stage with this,
// the bound without its slack and the biases loaded with the sums, us (96 experts of 3072
// inputs, Zipf-skewed): T=256 25.9 -> 24.8, T=512 36.5 -> 35.0.
template <typename XT, typename WT>
__device__ __attribute__((always_inline)) inline float wave_logit_exact_ahead(const XT *__restrict__ xr, const WT *__restrict__ wrow,
                                                                              double b, int H, int lane)
{
    constexpr int SEG = sizeof(XT) == 2 && sizeof(WT) == 2 ? 8 : 4;  // chunks of 512 inputs
    double hi = 0.0, lo = 0.0;
    for (int h0 = lane * 8; h0 < H; h0 += 512 * SEG) {
        Chunk8<XT> xc[SEG];
        Chunk8<WT> wc[SEG];
#pragma unroll
        for (int j = 0; j < SEG; ++j) {
            const int h = h0 + 512 * j < H ? h0 + 512 * j : h0;  // past the row: the first chunk again, not added
            ld_chunk<XT>(xr + h, xc[j]);
            ld_chunk<WT>(wrow + h, wc[j]);
        }
#pragma unroll
        for (int j = 0; j < SEG; ++j)
            if (h0 + 512 * j < H)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    double ss, ee;
                    two_sum(hi, elem<XT>(xc[j], i) * elem<WT>(wc[j], i), ss, ee);  // exact product
                    hi = ss;
                    lo += ee;
                }
    }
    return wave_dd_to_f32(hi, lo, b);
}

constexpr int kEPW = 4;  // experts per wave, at most

// One fp64 value moved by a DPP lane permutation (ctrl: an immediate DPP control).
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)u, CTRL, 0xF, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sum of v over the wave, the same in every lane: DPP quad permutes and the half-row
// and row mirrors give each 16-lane row its sum, and the four row sums are added from
// scalar registers.  Six additions deep, like a butterfly, so the recursive-summation
// bound of the caller holds.
__device__ inline double wave_sum_f64(double v)
{
    v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);  // row_half_mirror
    v += dpp_f64<0x140>(v);  // row_mirror
    double r[4];
#pragma unroll
    for (int row = 0; row < 4; ++row) {
        const uint64_t u = __double_as_longlong(v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 16 * row);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 16 * row);
        r[row] = __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    }
    return (r[0] + r[1]) + (r[2] + r[3]);
}

__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Canonical logits of one token row xr against router rows e0 .. e0+ne-1 (ne <= EPW),
// or the rows elist[0 .. ne-1],
// computed by one wave and written to lrow[e].  The lane's inputs are loaded once per
// segment and reused for every expert; the next expert's router row is in flight
// while the current one accumulates.  Returns the number of fallbacks taken.
//
// Each lane sums exact products in fp64 (two accumulators per expert) next to a bound
// on the sum of their magnitudes; the wave-reduced sum is certified against the fp32
// rounding midpoints with the recursive-summation error bound, else recomputed exactly.
// With bf16 inputs a product of two bf16 values is exact in fp32 (16-bit significand),
// so it is formed in fp32 and added in fp64, and the magnitude bound is summed in fp32
// and inflated by its own worst-case rounding; products below the fp32 subnormal grain
// add at most H*2^-149 in absolute error, which the margin covers.  fp32 inputs use
// fp64 fused multiply-adds throughout.
//
// EPW is the wave's expert capacity (ne <= EPW) and SEG the 8-input chunks per lane
// held at once: one expert per wave loads a 4096-input row in one round trip.
template <typename XT, typename WT, int EPW, int SEG>
__device__ __attribute__((always_inline)) inline int wave_logits(const XT *__restrict__ xr, const WT *__restrict__ wr, const float *bias, int H,
                                  int e0, int ne, int lane, float *lrow, const int *elist = nullptr)
{
    // expert i of the call: elist[i] if a list is given, else e0 + i
    int ex[EPW];
#pragma unroll
    for (int i = 0; i < EPW; ++i) ex[i] = elist ? elist[i < ne ? i : 0] : e0 + (i < ne ? i : 0);
    constexpr bool kBf16 = sizeof(XT) == 2 && sizeof(WT) == 2;
    const int nck = (H + 511) / 512;  // chunks of the lane with the most
    // Two accumulators per expert (even and odd chunks): each sums at most
    // ceil(nck/2)*8 products, then they are added and reduced over the wave.
    const int per_acc = ((nck + 1) / 2) * 8;
    const double gamma = (double)(per_acc + 1 + 6 + 1 + 2) * 0x1p-52;  // >= 2 gamma_D
    const double infl = 1.0 + (double)(per_acc + 2) * 0x1p-23;         // fp32 magnitude sums
    double s[EPW][2], a[EPW][2];
    float a32[EPW][2];
#pragma unroll
    for (int i = 0; i < EPW; ++i) {
        s[i][0] = s[i][1] = a[i][0] = a[i][1] = 0.0;
        a32[i][0] = a32[i][1] = 0.f;
    }
    for (int seg = 0; seg < nck; seg += SEG) {
        Chunk8<XT> xc[SEG];
        bool valid[SEG];
        int off[SEG];
#pragma unroll
        for (int j = 0; j < SEG; ++j) {
            const int h = lane * 8 + 512 * (seg + j);
            valid[j] = h < H;
            off[j] = valid[j] ? h : H - 8;  // clamped: an invalid chunk is loaded but its x is 0
            ld_chunk<XT>(xr + off[j], xc[j]);
            if (!valid[j])
#pragma unroll
                for (int q = 0; q < (int)(sizeof(xc[j].d) / 4); ++q) xc[j].d[q] = 0u;
        }
        float xf[SEG][8];
        if constexpr (kBf16)
#pragma unroll
            for (int j = 0; j < SEG; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    xf[j][2 * q] = bf16_lo(xc[j].d[q]);
                    xf[j][2 * q + 1] = bf16_hi(xc[j].d[q]);
                }
        // every expert's slice of this segment in flight at once (one memory latency)
        Chunk8<WT> wc[EPW][SEG];
#pragma unroll
        for (int i = 0; i < EPW; ++i)
#pragma unroll
            for (int j = 0; j < SEG; ++j)
                ld_chunk<WT>(wr + (size_t)ex[i] * H + off[j], wc[i][j]);
#pragma unroll
        for (int i = 0; i < EPW; ++i) {
            if (i < ne) {
#pragma unroll
                for (int j = 0; j < SEG; ++j)
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        if constexpr (kBf16) {
                            const uint32_t wd = wc[i][j].d[q >> 1];
                            const float wv = (q & 1) ? bf16_hi(wd) : bf16_lo(wd);
                            const float pv = xf[j][q] * wv;  // exact
                            s[i][j & 1] += (double)pv;
                            a32[i][j & 1] = fmaf(fabsf(xf[j][q]), fabsf(wv), a32[i][j & 1]);
                        } else {
                            const double xv = elem<XT>(xc[j], q), wv = elem<WT>(wc[i][j], q);
                            s[i][j & 1] = fma(xv, wv, s[i][j & 1]);
                            a[i][j & 1] = fma(fabs(xv), fabs(wv), a[i][j & 1]);
                        }
                    }
            }
        }
    }
    int nfb = 0;
#pragma unroll
    for (int i = 0; i < EPW; ++i) {
        if (i < ne) {
            const double si = wave_sum_f64(s[i][0] + s[i][1]);
            const double ai = wave_sum_f64(kBf16 ? ((double)a32[i][0] + (double)a32[i][1]) * infl : a[i][0] + a[i][1]);
            const int e = ex[i];
            const double b = bias ? (double)bias[e] : 0.0;
            const double slack = kBf16 ? (double)H * 0x1p-148 : 0.0;
            float r, up;
            if (!certain_f32(si + b, gamma * (ai + fabs(b)) + slack, r, up)) {
                r = wave_logit_exact<XT, WT>(xr, wr + (size_t)e * H, b, H, lane);
                ++nfb;
            }
            if (lane == 0) st_dev(&lrow[e], r + 0.0f);  // -0 -> +0
        }
    }
    return nfb;
}

// ------------------------------------------------------------------ top-k keys
//
// A key is (order-preserving integer image of the fp32 logit) << 32 | (~expert): the
// largest key is the largest logit, ties going to the lower expert index.

__device__ inline uint32_t ordered_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ inline float from_ordered(uint32_t o) { return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o); }

template <typename XT>
__device__ inline void load32_f32(const XT *p, float (&v)[32]);

template <>
__device__ inline void load32_f32<uint16_t>(const uint16_t *p, float (&v)[32])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint4 u = reinterpret_cast<const uint4 *>(p)[q];
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[8 * q + 2 * i] = __uint_as_float(w[i] << 16);
            v[8 * q + 2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
}

template <>
__device__ inline void load32_f32<float>(const float *p, float (&v)[32])
{
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float4 u = reinterpret_cast<const float4 *>(p)[q];
        v[4 * q] = u.x;
        v[4 * q + 1] = u.y;
        v[4 * q + 2] = u.z;
        v[4 * q + 3] = u.w;
    }
}

// ------------------------------------------------------------------ block scan

// Exclusive prefix sums of four counters over the 256 threads of a workgroup.
__device__ inline void block_exscan4(int (&v)[4], int (&tot)[4], int *sh /* [4 waves][4] */)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc[4] = {v[0], v[1], v[2], v[3]};
    int wt[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) wt[c] = wave_inclusive_scan(inc[c], lane);
    if (lane == 0)
        for (int c = 0; c < 4; ++c) sh[wave * 4 + c] = wt[c];
    __syncthreads();
    for (int c = 0; c < 4; ++c) {
        int before = 0, all = 0;
        for (int w = 0; w < 4; ++w) {
            const int s = sh[w * 4 + c];
            if (w < wave) before += s;
            all += s;
        }
        tot[c] = all;
        v[c] = before + inc[c] - v[c];
    }
    __syncthreads();
}

// Wave-wide maximum of 64-bit keys with DPP lane permutations: two quad permutes
// and the half-row and row mirrors leave every lane of a 16-lane row with the row's
// maximum; the four row maxima are combined in scalar registers.
__device__ inline uint64_t dpp_max64(uint64_t v, int ctrl_sel)
{
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32), olo, ohi;
    switch (ctrl_sel) {  // the DPP control is an immediate
    case 0:
        olo = __builtin_amdgcn_update_dpp(0u, lo, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
        ohi = __builtin_amdgcn_update_dpp(0u, hi, 0xB1, 0xF, 0xF, false);
        break;
    case 1:
        olo = __builtin_amdgcn_update_dpp(0u, lo, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
        ohi = __builtin_amdgcn_update_dpp(0u, hi, 0x4E, 0xF, 0xF, false);
        break;
    case 2:
        olo = __builtin_amdgcn_update_dpp(0u, lo, 0x141, 0xF, 0xF, false);  // row_half_mirror
        ohi = __builtin_amdgcn_update_dpp(0u, hi, 0x141, 0xF, 0xF, false);
        break;
    default:
        olo = __builtin_amdgcn_update_dpp(0u, lo, 0x140, 0xF, 0xF, false);  // row_mirror
        ohi = __builtin_amdgcn_update_dpp(0u, hi, 0x140, 0xF, 0xF, false);
        break;
    }
    const uint64_t o = ((uint64_t)ohi << 32) | olo;
    return o > v ? o : v;
}

__device__ inline uint64_t wave_max64(uint64_t v)
{
    v = dpp_max64(v, 0);
    v = dpp_max64(v, 1);
    v = dpp_max64(v, 2);
    v = dpp_max64(v, 3);
    uint64_t m = 0;
#pragma unroll
    for (int row = 0; row < 4; ++row) {
        // readlane returns a signed int: widen through uint32_t
        const uint64_t r = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), 16 * row) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 16 * row);
        m = r > m ? r : m;
    }
    return m;
}

// Top-k softmax of one token by one wave.  Keys are (ordered logit bits, complemented
// expert index): a larger logit wins, and among equal logits the lower index.  Lane
// owns keys of experts lane, lane+64, ... (V per lane, E <= 64V).  k rounds of a
// wave-wide argmax (DPP lane permutations, see wave_max64) each take the largest
// remaining key; lane j keeps choice j.  Weights are the softmax of the selected logits in
// fp32 relative to the largest, normalised by their butterfly sum, which every lane
// forms from the same pairs.
template <int V, bool MASK>
__device__ __attribute__((always_inline)) inline void wave_topk(const float *__restrict__ l, int E, int k, int32_t *ids, float *wts,
                                 int32_t *ids_user, float *wts_user, int lane, const uint32_t *cand)
{
    uint64_t key[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int e = 64 * v + lane;
        bool in = e < E;
        if constexpr (MASK) in = in && ((cand[e >> 5] >> (e & 31)) & 1u);
        key[v] = in ? ((uint64_t)ordered_bits(ld_dev(&l[e])) << 32) | (uint32_t)(~(uint32_t)e) : 0;
    }
    uint64_t mine = 0;  // lane j < k: key of choice j
    for (int j = 0; j < k; ++j) {
        uint64_t best = key[0];
#pragma unroll
        for (int v = 1; v < V; ++v) best = key[v] > best ? key[v] : best;
        best = wave_max64(best);
        if (lane == j) mine = best;
#pragma unroll
        for (int v = 0; v < V; ++v) key[v] = key[v] == best ? 0 : key[v];  // keys are unique
    }
    const float top = from_ordered((uint32_t)__shfl((uint32_t)(mine >> 32), 0));
    const float p = lane < k ? expf(from_ordered((uint32_t)(mine >> 32)) - top) : 0.f;
    float den = p;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) den += __shfl_xor(den, o);
    if (lane < k) {
        const int e = (int)(~(uint32_t)mine);
        const float w = p / den;
        st_dev(&ids[lane], e);
        wts[lane] = w;
        if (ids_user) ids_user[lane] = e;
        if (wts_user) wts_user[lane] = w;
    }
}

// MASK: only the experts of the bitmask `cand` may be selected (the others' logits need
// not be valid).
template <bool MASK = false>
__device__ __attribute__((always_inline)) inline void token_topk(const float *__restrict__ l, int E, int k, int32_t *ids, float *wts,
                                  int32_t *ids_user, float *wts_user, int lane, const uint32_t *cand = nullptr)
{
    if (E <= 64)
        wave_topk<1, MASK>(l, E, k, ids, wts, ids_user, wts_user, lane, cand);
    else if (E <= 128)
        wave_topk<2, MASK>(l, E, k, ids, wts, ids_user, wts_user, lane, cand);
    else if (E <= 256)
        wave_topk<4, MASK>(l, E, k, ids, wts, ids_user, wts_user, lane, cand);
    else if (E <= 512)
        wave_topk<8, MASK>(l, E, k, ids, wts, ids_user, wts_user, lane, cand);
    else
        wave_topk<16, MASK>(l, E, k, ids, wts, ids_user, wts_user, lane, cand);
}

// ------------------------------------------------------------------ fused routing kernel
//
// Grid = T x bpt workgroups of 4 waves.  Workgroup (t, q) computes the logits of token
// t for experts [4*q*epw, 4*(q+1)*epw).  The last workgroup of token t to finish (a
// device-scope counter) runs that token's top-k softmax in one wave while its other
// three waves write the token's 2-term FP8 activation split (when the MFMA path is
// on).  The last token to finish then groups all (token, choice) pairs by expert.  The
// counters are reset by the workgroup that consumes them, so they read zero at the
// start of every launch.


// No kernel reads more than this (256 bytes: four lines of argument memory, each a round
// trip to the host's memory when first touched): workgroup and grid sizes are constants or
// follow from it, since the dispatch's own would lie in a fifth line.
struct RouteArgs {
    const void *x;
    const void *wr;
    const float *bias;
    float *logits;
    int32_t *ids, *ids_user;
    float *wts, *wts_user;
    int32_t *meta, *slot_of, *tok_of;
    int32_t *cnt_tok;  // [Tmax][kCounterStride], one counter per 256-byte line
    int32_t *cnt_all;  // [1]
    int32_t *fb_acc;   // [1]
    uint8_t *xs_hi, *xs_lo, *xe_hi, *xe_lo;  // activation split (NULL: MFMA path off)
    _Float16 *x16;                           // f16 copy of x * 2^-k (NULL: none)
    int32_t *xk;                             // [T] the token's k
    int T, E, H, k, epw, bpt, mstar, do_group, max_chunks, chunk;
    uint32_t rk;  // ceil(2^32 / k): p / k = mulhi(p, rk) for k > 1, since T * k * k < 2^32
    int prefix, id_cache;  // the grouping keeps prefix counts / the choices in LDS (sized by the launch)
    // screened routing (large T): per K slice ks, partial sums part[ks][t][e] =
    // (sum x*w, sum |x*w|) and the slice's max |x[t,.]|, max |w[e,.]|
    double2 *part;
    float *xmax, *wmax;
    int KS, Tmax;
    int screened;  // screen_kernel and route_cand_kernel run (with KS > 0; else route_tile_kernel)
};
static_assert(sizeof(RouteArgs) <= 256);

// The 2-term FP8 split of one group of 32 inputs of token t (see fp8split.h).
template <typename XT>
__device__ __attribute__((always_inline)) inline void write_group(const RouteArgs &A, const XT *xr, int t, int g)
{
    const int H = A.H;
    float v[32], res[32];
    uint32_t qh[8], ql[8];
    load32_f32<XT>(xr + g * 32, v);
    const int ch = exp_for_group(amax_of(v));
    split_hi(v, ch, qh, res);
    const int cl = exp_for_group(amax_of(res));
    split_lo(res, cl, ql);
    const size_t o = (size_t)t * H + g * 32;
    reinterpret_cast<uint4 *>(A.xs_hi + o)[0] = make_uint4(qh[0], qh[1], qh[2], qh[3]);
    reinterpret_cast<uint4 *>(A.xs_hi + o)[1] = make_uint4(qh[4], qh[5], qh[6], qh[7]);
    reinterpret_cast<uint4 *>(A.xs_lo + o)[0] = make_uint4(ql[0], ql[1], ql[2], ql[3]);
    reinterpret_cast<uint4 *>(A.xs_lo + o)[1] = make_uint4(ql[4], ql[5], ql[6], ql[7]);
    A.xe_hi[(size_t)t * (H / 32) + g] = (uint8_t)ch;
    A.xe_lo[(size_t)t * (H / 32) + g] = (uint8_t)cl;
}

// The 2-term FP8 split of token t's activations (groups of 32 inputs, see fp8split.h),
// groups first, first + stride, ... written by the calling thread.
template <typename XT>
__device__ __attribute__((always_inline)) inline void write_split(const RouteArgs &A, const XT *xr, int t, int first, int stride)
{
    const int H = A.H, G = H / 32;
    for (int g = first; g < G; g += stride) write_group<XT>(A, xr, t, g);
}

// The token's bf16 x as f16 scaled by 2^-k, with k such that max|x| * 2^-k lies in
// [2^14, 2^15) (k = 0 for a zero row; k >= -112): every value at least 2^-31 of the
// row's maximum converts exactly.  Called by `nw` waves (wave index w), each of which
// takes the row maximum on its own (no barrier among them) and converts every nw-th
// chunk of 512 inputs.
__device__ __attribute__((always_inline)) inline void write_x16(const RouteArgs &A, const uint16_t *xr, int t, int w,
                                                                int nw, int lane)
{
    // eight chunks of 512 inputs in flight at a time; a row of one batch converts from registers
    constexpr int U = 8;
    const int H = A.H;
    float m = 0.f;
    uint4 c[U];
    auto load = [&](int h0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int h = h0 + 512 * u + lane * 8;
            c[u] = h < H ? *reinterpret_cast<const uint4 *>(xr + h) : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    auto value = [&](int u, float (&v)[8]) {
        const uint32_t wd[4] = {c[u].x, c[u].y, c[u].z, c[u].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(wd[i] << 16);
            v[2 * i + 1] = __uint_as_float(wd[i] & 0xFFFF0000u);
        }
    };
    for (int h0 = 0; h0 < H; h0 += 512 * U) {
        load(h0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float v[8];
            value(u, v);
#pragma unroll
            for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(v[i]));
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    const int ex = m > 0.f ? (int)((__float_as_uint(m) >> 23) & 0xFF) - 127 : 14;  // floor(log2 m) for normal m
    const int kk = max(ex - 14, -112);
    const float sc = __uint_as_float((uint32_t)(127 - kk) << 23);  // 2^-k
    for (int h0 = 0; h0 < H; h0 += 512 * U) {
        if (H > 512 * U) load(h0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int h = h0 + 512 * u + lane * 8;
            if (u % nw == w && h < H) {
                float v[8];
                value(u, v);
                _Float16 q[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) q[i] = (_Float16)(v[i] * sc);
                *reinterpret_cast<uint4 *>(A.x16 + (size_t)t * H + h) = __builtin_bit_cast(uint4, q);
            }
        }
    }
    if (w == 0 && lane == 0) A.xk[t] = kk;
}

// Last token of a step: group the T*k (token, choice) pairs by expert.  LDS holds one
// bit per (expert, token): expert e's tokens in token order.  counts = popcounts,
// offsets = exclusive prefix sum, slot of pair (t, j) choosing e = offsets[e] +
// (number of earlier tokens that chose e).  Experts with at least `mstar` tokens go
// to the MFMA list, the others to the GEMV list, each in expert order.  All threads
// of the workgroup call it.
__device__ __attribute__((always_inline)) inline void group_pairs(const RouteArgs &A, uint32_t *lds, int *s_scan)
{
    const int E = A.E;
    const int T = A.T, k = A.k, P = T * k;
    const int W = (T + 31) / 32;
    uint32_t *mask = lds;                        // [E][W]
    int32_t *offs = (int32_t *)(lds + E * W);    // [E]
    uint16_t *pre = (uint16_t *)(offs + E);      // [E][W] when the launch sized LDS for it: the expert's tokens in earlier words
    uint16_t *idc = pre + (A.prefix ? E * W : 0);  // [P] when the launch sized LDS for it: the choices, read once
    const bool cached = A.id_cache != 0;
    const MetaIdx mi{E, A.max_chunks};
    int nfb_total = 0, n_exact = A.T * E;
    if (threadIdx.x == 0) {  // in flight during the grouping; each counter is reset by its reader
        nfb_total = atomicExch(A.fb_acc, 0);
        if (A.KS) {  // screened: the logits computed exactly; tiled: the uncertain ones left out
            const int n = atomicExch(A.fb_acc + kCandCounterOff, 0);
            n_exact = A.screened ? n : n_exact - n;
        }
    }
    for (int i = threadIdx.x; i < E * W; i += kThreads) mask[i] = 0u;
    __syncthreads();
    // this thread's choices, eight loads in flight at a time (small loops: at small batches
    // this code is fetched cold, and 32 unrolled steps took 1.5 us longer)
    auto token = [&](int p) { return k == 1 ? p : (int)__umulhi((uint32_t)p, A.rk); };  // p / k
    for (int p0 = threadIdx.x; p0 < P; p0 += 8 * kThreads) {
        int e8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int p = p0 + u * kThreads;
            e8[u] = p < P ? ld_dev(&A.ids[p]) : 0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int p = p0 + u * kThreads;
            if (p < P) {
                const int tt = token(p);
                atomicOr(&mask[e8[u] * W + tt / 32], 1u << (tt % 32));
                if (cached) idc[p] = (uint16_t)e8[u];
            }
        }
    }
    __syncthreads();
    // each thread owns up to 4 consecutive experts
    const int per = (E + 255) / 256;
    const int eb = threadIdx.x * per;
    int cnt[4] = {0, 0, 0, 0};
    int v[4] = {0, 0, 0, 0};  // tokens, gemv experts, mfma experts, mfma token chunks
    for (int j = 0; j < per; ++j) {
        const int e = eb + j;
        if (e < E) {
            int c = 0;
            for (int w = 0; w < W; ++w) {
                if (A.prefix) pre[e * W + w] = (uint16_t)c;
                c += __popc(mask[e * W + w]);
            }
            cnt[j] = c;
            v[0] += c;
            if (c > 0) {
                if (A.mstar > 0 && c >= A.mstar) {
                    v[2]++;
                    v[3] += (c + A.chunk - 1) / A.chunk;
                } else {
                    v[1]++;
                }
            }
        }
    }
    int tot[4];
    block_exscan4(v, tot, s_scan);
    for (int j = 0; j < per; ++j) {
        const int e = eb + j;
        if (e < E) {
            const int c = cnt[j];
            offs[e] = v[0];
            A.meta[mi.counts() + e] = c;
            A.meta[mi.offsets() + e] = v[0];
            if (c > 0) {
                if (A.mstar > 0 && c >= A.mstar) {
                    int4 *cr = reinterpret_cast<int4 *>(A.meta + mi.chunk_rec());
                    for (int m0 = 0; m0 < c; m0 += A.chunk)
                        cr[v[3]++] = make_int4(e, v[0] + m0, min(A.chunk, c - m0), 0);
                    v[2]++;
                } else {
                    reinterpret_cast<int4 *>(A.meta + mi.gemv_rec())[v[1]++] = make_int4(e, v[0], c, 0);
                }
            }
            v[0] += c;
        }
    }
    if (threadIdx.x == 0) {
        A.meta[mi.offsets() + E] = tot[0];
        A.meta[mi.n_active()] = tot[1] + tot[2];
        A.meta[mi.n_gemv()] = tot[1];
        A.meta[mi.n_mfma()] = tot[2];
        A.meta[mi.n_fallback()] = nfb_total;
        A.meta[mi.n_mfma_chunks()] = tot[3];
        A.meta[mi.n_exact()] = n_exact;
        A.meta[mi.screened()] = A.screened;
        st_dev(A.cnt_all, 0);
        if (A.chunk != kMfmaChunk) A.fb_acc[kTicketOff] = A.fb_acc[kTicketOff + 1] = 0;
    }
    __syncthreads();
    for (int p = threadIdx.x; p < P; p += kThreads) {
        const int tt = token(p), e = cached ? idc[p] : ld_dev(&A.ids[p]);
        int rank = __popc(mask[e * W + tt / 32] & ((1u << (tt % 32)) - 1u));
        if (A.prefix)
            rank += pre[e * W + tt / 32];
        else
            for (int w = 0; w < tt / 32; ++w) rank += __popc(mask[e * W + w]);
        const int slot = offs[e] + rank;
        A.slot_of[p] = slot;
        A.tok_of[slot] = tt;
    }
}

template <typename XT, typename WT>
__global__ __launch_bounds__(256) void route_kernel(RouteArgs A)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ int s_flag;
    __shared__ int s_scan[16];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int t = blockIdx.x / A.bpt;
    const int q = blockIdx.x % A.bpt;
    const int E = A.E, H = A.H;
    const XT *xr = (const XT *)A.x + (size_t)t * H;

    // 1. logits of this workgroup's experts
    {
        const int e0 = (q * 4 + wave) * A.epw;
        const int ne = min(E, e0 + A.epw) - e0;
        if (ne > 0) {
            const WT *wr = (const WT *)A.wr;
            float *lrow = A.logits + (size_t)t * E;
            // one expert per wave: no loads for empty expert slots, and a row of up to
            // 4096 bf16 inputs in one round trip
            int nfb;
            if (A.epw > 1)
                nfb = wave_logits<XT, WT, kEPW, 4>(xr, wr, A.bias, H, e0, ne, lane, lrow);
            else if (sizeof(XT) == 2 && H <= 8 * 512)
                nfb = wave_logits<XT, WT, 1, 8>(xr, wr, A.bias, H, e0, ne, lane, lrow);
            else
                nfb = wave_logits<XT, WT, 1, 4>(xr, wr, A.bias, H, e0, ne, lane, lrow);
            if (lane == 0 && nfb) atomicAdd(A.fb_acc, nfb);
        }
    }
    // Publish this workgroup's logits, then count it; the last workgroup of the token
    // goes on.
    wait_stores();
    __syncthreads();
    if (threadIdx.x == 0) s_flag = atomicAdd(&A.cnt_tok[t * kCounterStride], 1) == A.bpt - 1;
    __syncthreads();
    if (!s_flag) return;

    // 2. last workgroup of token t: top-k softmax in wave 0 while waves 1-3 write the
    // token's 2-term activation split when the MFMA path is on (groups of 32 inputs), or
    // its scaled f16 copy for NVFP4 weights
    if (wave == 0) {
        token_topk(A.logits + (size_t)t * E, E, A.k, A.ids + (size_t)t * A.k, A.wts + (size_t)t * A.k,
                   A.ids_user ? A.ids_user + (size_t)t * A.k : nullptr,
                   A.wts_user ? A.wts_user + (size_t)t * A.k : nullptr, lane);
    } else if (A.xs_hi) {
        write_split<XT>(A, xr, t, threadIdx.x - kWave, kThreads - kWave);
    } else if constexpr (sizeof(XT) == 2) {
        if (A.x16) write_x16(A, xr, t, wave - 1, 3, lane);
    }
    if (threadIdx.x == 0) st_dev(&A.cnt_tok[t * kCounterStride], 0);
    if (!A.do_group) return;
    wait_stores();
    __syncthreads();
    // One token: its last workgroup is the step's last, without the second counter's
    // round trip (group_pairs leaves that counter at zero, where it already is).
    if (A.T > 1) {
        if (threadIdx.x == 0) s_flag = atomicAdd(A.cnt_all, 1) == A.T - 1;
        __syncthreads();
        if (!s_flag) return;
    }

    group_pairs(A, lds, s_scan);
}

// ------------------------------------------------------------------ screened routing
//
// At large T the exact logits of every (token, expert) pair are the step's largest
// vector-ALU cost.  Only the top-k of each token need them, so the screened path
// first brackets every logit and then computes exactly only the experts whose
// bracket can reach the top k:
//   screen_kernel    bf16 MFMA sums of x.w and |x|.|w| over 256-input chunks (fp32
//                    inside a chunk, fp64 across chunks), per K slice;
//   route_cand_kernel per token: the bracket [lo_e, hi_e] of every canonical logit
//                    l_e, LB = the k-th largest lo; e can be selected only if
//                    hi_e >= LB (k experts f have l_f >= lo_f >= LB > hi_e >= l_e
//                    otherwise); exact logits of those candidates (wave_logits), top-k
//                    among them by (l desc, e asc), softmax; the last token groups.
// Bracket.  A chunk of 256 exact products summed in fp32 in any order with any
// rounding is within g = 256u/(1-256u), u = 2^-23, of its exact sum times the sum of
// |products|; flushed denormal inputs, products or partial sums add at most
// 2^-126 (max|x| + max|w| + 2) per product; the fp64 sums across chunks and slices
// add at most 2^-40 of sum|products|; the bias add one fp64 rounding; the canonical
// rounding to fp32 at most 2^-23 relative plus 2^-149.

constexpr int kScreenChunk = 256;  // inputs per fp32 MFMA chunk
constexpr int kMaxE = 1024;
constexpr int kMaxKS = kScreenMaxKS;  // K slices of the screen at most
constexpr size_t kCandStaticLds = 12800;  // bytes, at least route_cand_kernel's static LDS

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kScreenOOR = 0x80000000u;  // buffer offset past every resource: zeros, no request

__device__ inline __amdgpu_buffer_rsrc_t screen_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}

// Grid (ceil(T/16), ceil(E/64), KS), 256 threads.  Wave w: experts e0 = 64y + 16w .. +16
// (MFMA rows: A = router rows), tokens 16x .. +16 (columns: B = x rows), chunks of
// slice z.  Writes part[z][t][e] = (sum x*w, sum |x*w|) and the slice's max |x|, max |w|.
__global__ __launch_bounds__(256) void screen_kernel(RouteArgs A)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, lg = lane >> 4;
    const int T = A.T, E = A.E, H = A.H;
    const int t0 = blockIdx.x * 16, e0 = blockIdx.y * 64 + wave * 16, ks = blockIdx.z;
    const int nch = H / kScreenChunk, cps = (nch + A.KS - 1) / A.KS;
    const int c0 = min(nch, ks * cps), c1 = min(nch, c0 + cps);
    const __amdgpu_buffer_rsrc_t xr = screen_rsrc(A.x, (uint32_t)T * H * 2u);
    const __amdgpu_buffer_rsrc_t wr = screen_rsrc(A.wr, (uint32_t)E * H * 2u);
    const uint32_t xo = t0 + r < T ? (uint32_t)(t0 + r) * H * 2u : kScreenOOR;
    const uint32_t wo = e0 + r < E ? (uint32_t)(e0 + r) * H * 2u : kScreenOOR;
    double S[4] = {0.0, 0.0, 0.0, 0.0}, Aa[4] = {0.0, 0.0, 0.0, 0.0};
    u16x2 mx = {0, 0}, mw = {0, 0};
    u32x4v xa[2][8], wa[2][8];
    auto load = [&](int b, int c) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t k2 = (uint32_t)(c * kScreenChunk + 32 * i + 8 * lg) * 2u;
            xa[b][i] = __builtin_amdgcn_raw_buffer_load_b128(xr, xo + k2, 0, 0);
            wa[b][i] = __builtin_amdgcn_raw_buffer_load_b128(wr, wo + k2, 0, 0);
        }
    };
    auto compute = [&](int b) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acca = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const u32x4v m = {0x7FFF7FFFu, 0x7FFF7FFFu, 0x7FFF7FFFu, 0x7FFF7FFFu};
            const u32x4v xabs = xa[b][i] & m, wabs = wa[b][i] & m;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[b][i]),
                                                          __builtin_bit_cast(bf16x8, xa[b][i]), acc, 0, 0, 0);
            acca = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wabs),
                                                           __builtin_bit_cast(bf16x8, xabs), acca, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {  // |bf16| bit patterns order like their values
                mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, xabs[q]));
                mw = __builtin_elementwise_max(mw, __builtin_bit_cast(u16x2, wabs[q]));
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            S[j] += (double)acc[j];
            Aa[j] += (double)acca[j];
        }
    };
    if (c0 < c1) {
        // chunk c sits in buffer (c - c0) % 2; loads of the next chunk are in flight
        // while one is multiplied (the last chunk is reloaded past the end)
        load(0, c0);
        int c = c0;
        for (; c + 2 <= c1; c += 2) {
            load(1, c + 1);
            compute(0);
            load(0, min(c + 2, c1 - 1));
            compute(1);
        }
        if (c < c1) compute(0);
    }
    // lane: experts e0 + 4lg + j (rows), token t0 + r (column)
    const int t = t0 + r;
    if (t < T) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = e0 + 4 * lg + j;
            if (e < E) A.part[((size_t)ks * A.Tmax + t) * E + e] = make_double2(S[j], Aa[j]);
        }
    }
    // slice maxima: lane (r, lg) saw row r of x and of the router block; combine the
    // four lane groups
    uint32_t m1 = max((uint32_t)mx.x, (uint32_t)mx.y), m2 = max((uint32_t)mw.x, (uint32_t)mw.y);
    m1 = max(m1, (uint32_t)__shfl_xor((int)m1, 16));
    m1 = max(m1, (uint32_t)__shfl_xor((int)m1, 32));
    m2 = max(m2, (uint32_t)__shfl_xor((int)m2, 16));
    m2 = max(m2, (uint32_t)__shfl_xor((int)m2, 32));
    if (lg == 0) {
        if (t < T) A.xmax[(size_t)ks * A.Tmax + t] = __uint_as_float(m1 << 16);
        if (e0 + r < E) A.wmax[(size_t)ks * E + e0 + r] = __uint_as_float(m2 << 16);
    }
}

// fp32 rounded down / up from fp64.
__device__ inline float f32_down(double v)
{
    float f = (float)v;
    return (double)f > v ? nextafterf(f, -INFINITY) : f;
}
__device__ inline float f32_up(double v)
{
    float f = (float)v;
    return (double)f < v ? nextafterf(f, INFINITY) : f;
}

// k-th largest of v[0 .. E-1] (E <= 64 V) in the key order of the top-k (value desc,
// index asc), by one wave: k rounds of the wave argmax.
template <int V>
__device__ __attribute__((always_inline)) inline float kth_largest(const float *v, int E, int k, int lane)
{
    uint64_t key[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const int e = 64 * i + lane;
        key[i] = e < E ? ((uint64_t)ordered_bits(v[e]) << 32) | (uint32_t)(~(uint32_t)e) : 0;
    }
    uint64_t best = 0;
    for (int j = 0; j < k; ++j) {
        best = key[0];
#pragma unroll
        for (int i = 1; i < V; ++i) best = key[i] > best ? key[i] : best;
        best = wave_max64(best);
#pragma unroll
        for (int i = 0; i < V; ++i) key[i] = key[i] == best ? 0 : key[i];
    }
    return from_ordered((uint32_t)(best >> 32));
}

// One workgroup per token (grid T), 256 threads; dynamic LDS as route_kernel's grouping.
__global__ __launch_bounds__(256) void route_cand_kernel(RouteArgs A)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ float s_lo[kMaxE], s_hi[kMaxE];
    __shared__ uint32_t s_cand[kMaxE / 32];
    __shared__ int s_list[kMaxE];
    __shared__ int s_n, s_flag;
    __shared__ int s_scan[16];
    static_assert(sizeof(float) * 2 * kMaxE + sizeof(uint32_t) * (kMaxE / 32) + sizeof(int) * (kMaxE + 2 + 16) <=
                  kCandStaticLds);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int t = blockIdx.x, E = A.E, H = A.H, k = A.k;
    const uint16_t *xr = (const uint16_t *)A.x + (size_t)t * H;
    const uint16_t *wr = (const uint16_t *)A.wr;

    // 1. brackets of every expert's canonical logit
    // (the slices' loads are issued together: KS <= kMaxKS, unrolled and predicated)
    float xm[kMaxKS];
#pragma unroll
    for (int s2 = 0; s2 < kMaxKS; ++s2) xm[s2] = s2 < A.KS ? A.xmax[(size_t)s2 * A.Tmax + t] : 0.f;
    float mxt = 0.f;
#pragma unroll
    for (int s2 = 0; s2 < kMaxKS; ++s2) mxt = fmaxf(mxt, xm[s2]);
    const double u = 0x1p-23, g = kScreenChunk * u / (1.0 - kScreenChunk * u);
    for (int e = threadIdx.x; e < E; e += kThreads) {
        double2 d[kMaxKS];
        float wm[kMaxKS];
#pragma unroll
        for (int s2 = 0; s2 < kMaxKS; ++s2) {
            d[s2] = s2 < A.KS ? A.part[((size_t)s2 * A.Tmax + t) * E + e] : make_double2(0.0, 0.0);
            wm[s2] = s2 < A.KS ? A.wmax[(size_t)s2 * E + e] : 0.f;
        }
        double S = 0.0, Aa = 0.0;
        float mwe = 0.f;
#pragma unroll
        for (int s2 = 0; s2 < kMaxKS; ++s2) {
            S += d[s2].x;
            Aa += d[s2].y;
            mwe = fmaxf(mwe, wm[s2]);
        }
        const double flush = (double)H * 0x1p-126 * ((double)mxt + (double)mwe + 2.0);
        const double Ab = (Aa * (1.0 + 0x1p-40) + flush) / (1.0 - g);
        const double Sb = S + (A.bias ? (double)A.bias[e] : 0.0);
        const double dsum = (g + 0x1p-40) * Ab + flush;
        const double D = dsum + fabs(Sb) * 0x1p-52 + (fabs(Sb) + dsum) * 0x1p-23 + 0x1p-149;
        s_lo[e] = f32_down(Sb - D);
        s_hi[e] = f32_up(Sb + D);
    }
    for (int i = threadIdx.x; i < kMaxE / 32; i += kThreads) s_cand[i] = 0u;
    __syncthreads();

    // 2. wave 0: LB = k-th largest lower bound, the candidates hi >= LB in expert
    // order; waves 1-3: the token's activation split (MFMA path)
    if (wave == 0) {
        const int V = (E + 63) / 64;
        const float LB = V <= 1   ? kth_largest<1>(s_lo, E, k, lane)
                         : V <= 2 ? kth_largest<2>(s_lo, E, k, lane)
                         : V <= 4 ? kth_largest<4>(s_lo, E, k, lane)
                         : V <= 8 ? kth_largest<8>(s_lo, E, k, lane)
                                  : kth_largest<16>(s_lo, E, k, lane);
        int n = 0;
        for (int v = 0; v < V; ++v) {
            const int e = 64 * v + lane;
            const bool c = e < E && !(s_hi[e] < LB);  // a NaN bracket or LB keeps e: n >= k always
            const uint64_t bal = __ballot(c);
            if (c) {
                s_list[n + __popcll(bal & ((1ull << lane) - 1ull))] = e;
                atomicOr(&s_cand[e >> 5], 1u << (e & 31));
            }
            n += __popcll(bal);
        }
        if (lane == 0) {
            s_n = n;
            atomicAdd(A.fb_acc + kCandCounterOff, n);
        }
    } else if (A.xs_hi) {
        write_split<uint16_t>(A, xr, t, threadIdx.x - kWave, kThreads - kWave);
    } else if (A.x16) {
        write_x16(A, xr, t, wave - 1, 3, lane);
    }
    __syncthreads();

    // 3. exact canonical logits of the candidates: an even share per wave, up to kEPW
    // router rows in flight per call; they go to LDS over the lower bounds, which are
    // no longer needed
    float *lrow = s_lo;
    int nfb = 0;
    const int n = s_n, per = (n + 3) / 4, i0 = wave * per, i1 = min(n, i0 + per);
    for (int i = i0; i < i1; i += kEPW)
        nfb += wave_logits<uint16_t, uint16_t, kEPW, 4>(xr, wr, A.bias, H, 0, min(kEPW, i1 - i), lane, lrow, s_list + i);
    if (lane == 0 && nfb) atomicAdd(A.fb_acc, nfb);
    __syncthreads();

    // 4. top-k among the candidates, softmax of the selected logits
    if (wave == 0)
        token_topk<true>(lrow, E, k, A.ids + (size_t)t * k, A.wts + (size_t)t * k,
                   A.ids_user ? A.ids_user + (size_t)t * k : nullptr, A.wts_user ? A.wts_user + (size_t)t * k : nullptr,
                   lane, s_cand);
    wait_stores();
    __syncthreads();
    if (threadIdx.x == 0) s_flag = atomicAdd(A.cnt_all, 1) == A.T - 1;
    __syncthreads();
    if (!s_flag) return;
    group_pairs(A, lds, s_scan);
}

// ------------------------------------------------------------------ tiled routing
//
// Where tile_routes says so, the logits come from fp64 matrix-core sums: workgroup (ks, y, z)
// forms the 16 x 16 products of experts 16y.. and tokens 16z.. over slice ks of the inputs
// (v_mfma_f64_16x16x4: products of bf16 or fp32 operands are exact in fp64), so each
// operand is converted once for sixteen products; converting and adding every product on
// the vector ALU bounded the logits of route_kernel, and the screen's two launches and
// dependent phases the large steps.  Each slice's sum goes out with a bound on its sum of
// |x*w| (the norms' product, by Cauchy-Schwarz).  The last workgroup of a token tile to
// arrive (a device-scope counter) finishes it while the others write its activation split:
// it adds the slices, certifies every fp32 rounding as route_kernel does, and runs the
// top-k softmax of the sixteen tokens, a token per 16-lane row, four to a wave.  The last
// token tile groups the pairs.
//
// What bounds it is that chain of dependent phases.  Device timestamps, us from the
// workgroup's start (480B-shaped T=64; 235B-shaped T=256): sums 6.8, 7.2; handed over 9.2,
// 9.7; certified 13.4, 12.3; top k 15.7, 14.2; written 16.8, 15.5; grouped 21, 25.  The whole
// kernel by rocprofv3, us: 23 and 25; 480B-shaped T=1000 92.  Step us, before / now:
// 235B-shaped NVFP4 T=127 282 / 274; 480B-shaped T=1000 1,854 / 1,753; T=64 even (908 / 906).

constexpr int kTileE = 256;  // experts at most (16 keys per lane)
constexpr int kTileK = 16;   // choices at most (one per lane of a row)
constexpr int kTileAcc = 4;  // accumulators per wave

// Where the tiled routing runs.  Its fixed phases (the slices' hand-off, a token tile's top-k
// in one workgroup, longer with more experts) cost more than the logits save on few (token,
// expert) pairs, and with bf16 inputs on short ones, whose products route_kernel forms in fp32.
// Step us against the other kernels (route_kernel, from 2^26 multiply-adds the screen),
// without a router bias / Zipf-skewed:
//   H 4096  128 experts T=51 +0.5 / +0.1, T=59 -2.0 / +1.3; 160 T=41 +0.7 / +3.7, T=54 -1.6 /
//           +1.5, T=75 -2.5 / +1.2; 256 T=34 -1.2 / +3.7, T=55 -4.8 / -0.9, T=129 -13 / -7.2
//   H 2048  64 experts T=102 +1.4 / +2.4, T=157 -1.4 / +1.4, T=219 -3.5 / -3.0; 128 T=94
//           +1.1 / +2.9, T=129 -2.3 / -0.5; 160 T=104 +1.0 / +1.6, T=157 -1.4 / -0.8; 256
//           T=129 +1.1 / +4.0, T=188 +2.7 / +7.2, T=258 -7.2 / -3.3
//   H 1024  32 experts T=204 +1.3 / +2.3, T=313 -0.5 / -0.6; 64 T=133 +1.3 / +1.6, T=219 -2.7 /
//           -2.8; 128 T=94 +2.1 / +4.4, T=129 -0.5 / 0.0; 256 T=65 +3.2 / +4.6, T=129 -2.8 / -3.4
bool tile_routes(const Layer &L, const RouteParams &P)
{
    const long pairs = (long)P.T * L.E;
    if (L.E > kTileE || P.k > kTileK || P.ks_max == 0 || pairs <= 6400) return false;
    if (!L.act_bf16 || !L.router_bf16) return true;
    if (L.H >= 3072) return P.T >= 50;
    return pairs >= 10000 && P.T >= (L.E > 192 && L.H >= 2048 ? 256 : 128);
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// This wave's LDS stores are done, and later reads are reads: lanes of one wave exchange
// values through LDS without a workgroup barrier.
__device__ inline void sync_wave() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Maximum / minimum over each 16-lane row, the same in all its lanes.
__device__ inline uint32_t row_max(uint32_t v)
{
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0u, v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0u, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0u, v, 0x140, 0xF, 0xF, false));  // row_mirror
}
__device__ inline int row_min(int v)
{
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false));
    return min(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false));
}

// The k largest logits of the token of each 16-lane row, ties to the lower expert: lane
// j < k of the row gets choice j (its logit and expert), every lane the last choice's
// logit.  Keys are the logits' ordered bits; 0
// stands for a chosen expert or none, below every logit's key, an infinity's and a NaN's
// too, so the choices are k different experts below E whatever the logits are (k <= E).
template <int V>
__device__ __attribute__((always_inline)) inline void tile_topk(const float *l, int E, int k, int j, float &lj, int &ej,
                                                                float &last)
{
    uint32_t key[V], m = 0u;
#pragma unroll
    for (int v = 0; v < V; ++v) key[v] = 16 * v + j < E ? max(ordered_bits(l[16 * v + j]), 1u) : 0u;
    lj = 0.f, ej = 0;
    for (int c = 0; c < k; ++c) {
        m = key[0];
#pragma unroll
        for (int v = 1; v < V; ++v) m = max(m, key[v]);
        m = row_max(m);
        int e = INT_MAX;
#pragma unroll
        for (int v = V - 1; v >= 0; --v) e = key[v] == m ? 16 * v + j : e;
        e = row_min(e);
        if (j == c) lj = from_ordered(m), ej = e;
#pragma unroll
        for (int v = 0; v < V; ++v) key[v] = 16 * v + j == e ? 0u : key[v];
    }
    last = from_ordered(m);
}

__device__ __attribute__((always_inline)) inline void tile_topk_any(const float *l, int E, int k, int j, float &lj, int &ej,
                                                                    float &last)
{
    if (E <= 64)
        tile_topk<4>(l, E, k, j, lj, ej, last);
    else if (E <= 128)
        tile_topk<8>(l, E, k, j, lj, ej, last);
    else if (E <= 192)
        tile_topk<12>(l, E, k, j, lj, ej, last);
    else
        tile_topk<16>(l, E, k, j, lj, ej, last);
}

// The slices' sums of token t against experts r, r + 16, ...: done(e, sum, bound, bias).  Up to 32
// 16-byte loads are in flight at a time, past the per-XCD L2 (the producers' stores went
// past theirs); one expert's at a time cost a memory round trip each.
template <int KS, class F>
__device__ __attribute__((always_inline)) inline void tile_sums(const RouteArgs &A, int t, int r, F done)
{
    constexpr int VG = KS == 1 ? 16 : 32 / KS, kDeviceScope = 16;  // experts per round; cache policy bit sc1
    const int E = A.E;
    const __amdgpu_buffer_rsrc_t pr = screen_rsrc(A.part, (uint32_t)KS * A.Tmax * E * 16u);
    for (int e0 = r; e0 < E; e0 += 16 * VG) {
        u32x4v u[VG][KS];
        float bias[VG];  // in flight with the sums
#pragma unroll
        for (int v = 0; v < VG; ++v) bias[v] = A.bias && e0 + 16 * v < E ? A.bias[e0 + 16 * v] : 0.f;
#pragma unroll
        for (int v = 0; v < VG; ++v)
#pragma unroll
            for (int q = 0; q < KS; ++q)
                u[v][q] = __builtin_amdgcn_raw_buffer_load_b128(
                    pr, t < A.T && e0 + 16 * v < E ? (((uint32_t)q * A.Tmax + t) * E + e0 + 16 * v) * 16u : kScreenOOR, 0,
                    kDeviceScope);
#pragma unroll
        for (int v = 0; v < VG; ++v)
            if (t < A.T && e0 + 16 * v < E) {
                double S = 0.0, B = 0.0;
#pragma unroll
                for (int q = 0; q < KS; ++q) {
                    S += __longlong_as_double((long long)(((uint64_t)u[v][q][1] << 32) | u[v][q][0]));
                    B += __longlong_as_double((long long)(((uint64_t)u[v][q][3] << 32) | u[v][q][2]));
                }
                done(e0 + 16 * v, S, B, (double)bias[v]);
            }
    }
}

template <typename XT, typename WT>
__global__ __launch_bounds__(256) void route_tile_kernel(RouteArgs A)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ double s_red[4][256];  // the waves' sums; then the list of uncertain logits (16 bits each)
    __shared__ double s_nx[4][16], s_nw[4][16];
    __shared__ int s_flag, s_nfb[4];
    __shared__ int s_width[16];
    __shared__ int s_scan[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int T = A.T, E = A.E, H = A.H, KS = A.KS;
    const int ks = blockIdx.x, e0 = blockIdx.y * 16, t0 = blockIdx.z * 16;
    constexpr uint32_t kX = sizeof(XT), kW = sizeof(WT);

    // 1. this wave's inputs: steps of 32, lane (r, g) the eight from 8g of row r
    const int nst = H / 32, per = (nst + 4 * KS - 1) / (4 * KS);
    const int s0 = min(nst, (ks * 4 + wave) * per), s1 = min(nst, s0 + per);
    const __amdgpu_buffer_rsrc_t xr = screen_rsrc(A.x, (uint32_t)T * H * kX), wr = screen_rsrc(A.wr, (uint32_t)E * H * kW);
    const uint32_t xo = t0 + r < T ? ((uint32_t)(t0 + r) * H + 8u * g) * kX : kScreenOOR;
    const uint32_t wo = e0 + r < E ? ((uint32_t)(e0 + r) * H + 8u * g) * kW : kScreenOOR;
    constexpr int B = kX == 2 && kW == 2 ? 4 : 2;  // steps loaded together
    Chunk8<XT> xc[2][B];
    Chunk8<WT> wc[2][B];
    auto load = [&](int b, int s) {
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const bool in = s + i < s1;  // past the slice: zeros
#pragma unroll
            for (int q = 0; q < (int)(kX / 2); ++q) {
                const u32x4v u = __builtin_amdgcn_raw_buffer_load_b128(xr, in ? xo + (uint32_t)(s + i) * 32u * kX + 16u * q : kScreenOOR, 0, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) xc[b][i].d[4 * q + c] = u[c];
            }
#pragma unroll
            for (int q = 0; q < (int)(kW / 2); ++q) {
                const u32x4v u = __builtin_amdgcn_raw_buffer_load_b128(wr, in ? wo + (uint32_t)(s + i) * 32u * kW + 16u * q : kScreenOOR, 0, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) wc[b][i].d[4 * q + c] = u[c];
            }
        }
    };
    f64x4 acc[kTileAcc];
#pragma unroll
    for (int i = 0; i < kTileAcc; ++i) acc[i] = (f64x4){0.0, 0.0, 0.0, 0.0};
    double nx = 0.0, nw = 0.0;
    auto compute = [&](int b) {
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double xv = elem<XT>(xc[b][i], q), wv = elem<WT>(wc[b][i], q);
                nx = fma(xv, xv, nx);
                nw = fma(wv, wv, nw);
                acc[q % kTileAcc] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv, xv, acc[q % kTileAcc], 0, 0, 0);
            }
    };
    load(0, s0);
    for (int s = s0; s < s1; s += 2 * B) {
        load(1, s + B);
        compute(0);
        load(0, s + 2 * B);
        compute(1);
    }
    // 2. the workgroup's sums.  Lane l holds experts 4i + l/16 (i < 4) of token l%16.
    nx += __shfl_xor(nx, 16);
    nx += __shfl_xor(nx, 32);
    nw += __shfl_xor(nw, 16);
    nw += __shfl_xor(nw, 32);
    if (g == 0) {
        s_nx[wave][r] = nx;
        s_nw[wave][r] = nw;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) s_red[wave][64 * i + lane] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
    __syncthreads();
    const XT *x = (const XT *)A.x;
    {
        const int e = 4 * wave + g, t = r;
        const double S = (s_red[0][tid] + s_red[1][tid]) + (s_red[2][tid] + s_red[3][tid]);
        const double x2 = (s_nx[0][t] + s_nx[1][t]) + (s_nx[2][t] + s_nx[3][t]);
        const double w2 = (s_nw[0][e] + s_nw[1][e]) + (s_nw[2][e] + s_nw[3][e]);
        if (t0 + t < T && e0 + e < E) {
            double *p = (double *)(A.part + ((size_t)ks * A.Tmax + t0 + t) * E + e0 + e);
            st_dev(p, S);
            st_dev(p + 1, sqrt(x2) * sqrt(w2) * (1.0 + 0x1p-30));
        }
    }
    wait_stores();
    __syncthreads();
    const int nwg = KS * ((E + 15) / 16), ntt = (T + 15) / 16;  // workgroups of a token tile, token tiles
    if (tid == 0) s_flag = atomicAdd(&A.cnt_tok[blockIdx.z * kCounterStride], 1);
    __syncthreads();
    const int wg = s_flag;  // order of arrival in the token tile
    if (wg < nwg - 1 || nwg == 1) {
        // the others share the token tile's activation split (MFMA path)
        const int n = nwg > 1 ? nwg - 1 : 1;
        if (A.xs_hi) {
            const int G = H / 32;
            for (int i = wg * 256 + tid; i < 16 * G; i += n * 256) {
                const int t = t0 + i / G;
                if (t < T) write_group<XT>(A, x + (size_t)t * H, t, i % G);
            }
        } else if constexpr (sizeof(XT) == 2) {
            if (A.x16)
                for (int i = wg * 4 + wave; i < 32; i += n * 4)  // two waves per token
                    if (t0 + i / 2 < T) write_x16(A, x + (size_t)(t0 + i / 2) * H, t0 + i / 2, i & 1, 2, lane);
        }
        if (wg < nwg - 1) return;
    }

    // 3. last workgroup of the token tile, a token per 16-lane row, four to a wave: logits,
    // top k.  A logit that the bound does not certify goes in at the lower end of its
    // interval, so the k-th largest value is a lower bound of the k-th largest logit, and the
    // logit matters only if its upper end reaches that value (ends equal to it may tie).
    // Under cancellation the two ends are many fp32 steps apart; s_width holds the token's
    // largest distance of them, rounded up, as float bits (ordered like the floats, a NaN
    // above all).  The logits that matter are recomputed exactly (every one where the logits
    // are asked for) and the top k taken again, all within the wave; the others stay below
    // the k largest.
    const int tk = 4 * wave + g, t = t0 + tk;
    float *l = (float *)lds + (size_t)tk * E;  // this row's logits
    uint16_t *fb = (uint16_t *)&s_red[wave][0];  // the wave's uncertain logits
    if (lane == 0) s_nfb[wave] = 0;
    if (r == 0) s_width[tk] = 0;
    if (tid == 0) st_dev(&A.cnt_tok[blockIdx.z * kCounterStride], 0);
    {
        // one accumulator's roundings (its MFMAs, four products each), the accumulators', the
        // waves' and the slices' additions and the bias; twice the recursive-summation bound
        // (the zeros that a slice's last batch is filled with are added without rounding)
        const int D = 4 * (per * 8 / kTileAcc) + 4 + 4 + KS + 1 + 2;
        const double gamma = (double)D * 0x1p-52;
        auto done = [&](int e, double S, double Bd, double bias) {
            float c, up;
            if (!certain_f32(S + bias, gamma * (Bd + fabs(bias)), c, up)) {
                fb[atomicAdd(&s_nfb[wave], 1)] = (uint16_t)(g * kTileE + e);
                const float wd = (float)((double)up - (double)c);
                atomicMax(&s_width[tk], (int)(__float_as_uint(nextafterf(wd, INFINITY)) & 0x7FFFFFFFu));
            }
            l[e] = c + 0.0f;  // -0 -> +0
        };
        if (KS == 1)
            tile_sums<1>(A, t, r, done);
        else if (KS == 2)
            tile_sums<2>(A, t, r, done);
        else
            tile_sums<4>(A, t, r, done);
    }
    sync_wave();
    float lj, last;
    int ej;
    for (int pass = 0;; ++pass) {
        tile_topk_any(l, E, A.k, r, lj, ej, last);
        if (pass) break;
        const int nfb = __builtin_amdgcn_readfirstlane(s_nfb[wave]);
        int nex = 0;
        for (int i = 0; i < nfb; ++i) {
            const int fg = __builtin_amdgcn_readfirstlane((int)fb[i] / kTileE);
            const int e = __builtin_amdgcn_readfirstlane((int)fb[i] % kTileE);
            float *lf = (float *)lds + (size_t)(4 * wave + fg) * E + e;
            const float up = (float)((double)*lf + (double)__int_as_float(s_width[4 * wave + fg]));
            if (A.do_group && up < __shfl(last, 16 * fg)) continue;
            const float c = wave_logit_exact_ahead<XT, WT>(x + (size_t)(t0 + 4 * wave + fg) * H, (const WT *)A.wr + (size_t)e * H,
                                                     A.bias ? (double)A.bias[e] : 0.0, H, lane);
            if (lane == 0) *lf = c + 0.0f;
            ++nex;
        }
        if (lane == 0 && nex < nfb) atomicAdd(A.fb_acc + kCandCounterOff, nfb - nex);
        if (!nex) break;
        if (lane == 0) atomicAdd(A.fb_acc, nex);
        sync_wave();
    }
    if (!A.do_group && t < T)
        for (int e = r; e < E; e += 16) A.logits[(size_t)t * E + e] = l[e];
    const float p = r < A.k ? expf(lj - __shfl(lj, lane & 48)) : 0.f;
    float den = p;
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) den += __shfl_xor(den, o);
    if (t < T && r < A.k) {
        const size_t o = (size_t)t * A.k + r;
        const float w = p / den;
        st_dev(&A.ids[o], ej);
        A.wts[o] = w;
        if (A.ids_user) A.ids_user[o] = ej;
        if (A.wts_user) A.wts_user[o] = w;
    }
    if (!A.do_group) return;
    wait_stores();
    __syncthreads();
    if (ntt > 1) {
        if (tid == 0) s_flag = atomicAdd(A.cnt_all, 1) == ntt - 1;
        __syncthreads();
        if (!s_flag) return;
    }
    group_pairs(A, lds, s_scan);
}

__global__ void zero_kernel(int32_t *p, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

}  // namespace

hipError_t launch_zero(int32_t *p, int n, hipStream_t st)
{
    zero_kernel<<<(n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024, 256, 0, st>>>(p, n);
    return hipGetLastError();
}

hipError_t launch_route(const Layer &L, const RouteParams &P, hipStream_t st)
{
    // Experts per wave: one up to 6400 (token, expert) pairs, four above.  Timed on the
    // 235B- and 480B-shaped routers with one to four experts per wave at 2048-12288
    // pairs: one is best or within 1.3 us up to 6400 pairs (480B-shaped, 32 tokens:
    // 16.5 us against 17.3 / 17.9 / 18.9 with two / three / four), four from 7168 pairs on
    // or within 0.8 us (235B-shaped, 64 tokens: 15.6 against 18.5 with one).
    const int epw = P.T * L.E <= 6400 ? 1 : kEPW;
    const int bpt = (L.E + 4 * epw - 1) / (4 * epw);
    RouteArgs A;
    A.x = P.x;
    A.wr = P.router_w;
    A.bias = P.bias;
    A.logits = P.logits;
    A.ids = P.ids;
    A.ids_user = P.ids_user;
    A.wts = P.wts;
    A.wts_user = P.wts_user;
    A.meta = P.meta;
    A.slot_of = P.slot_of;
    A.tok_of = P.tok_of;
    A.cnt_tok = P.cnt_tok;
    A.cnt_all = P.cnt_all;
    A.fb_acc = P.fb_acc;
    A.xs_hi = P.xs_hi;
    A.xs_lo = P.xs_lo;
    A.xe_hi = P.xe_hi;
    A.xe_lo = P.xe_lo;
    A.x16 = P.x16;
    A.xk = P.xk;
    A.T = P.T;
    A.E = L.E;
    A.H = L.H;
    A.k = P.k;
    A.epw = epw;
    A.bpt = bpt;
    A.mstar = P.mstar;
    A.do_group = P.do_group;
    A.max_chunks = P.max_chunks;
    A.chunk = P.chunk;
    A.part = (double2 *)P.part;
    A.xmax = P.xmax;
    A.wmax = P.wmax;
    A.Tmax = P.Tmax;
    A.KS = 0;
    A.screened = 0;
    A.rk = (uint32_t)((0x100000000ull + P.k - 1) / P.k);
    const int W = (P.T + 31) / 32;
    // grouping LDS: bitmasks [E][W] and offsets [E], then, in 16 bits, prefix counts [E][W]
    // and the choices [T*k], each while the whole stays within 48 KiB (64 KiB with the
    // kernels' static arrays)
    const size_t masks = (size_t)L.E * W, pairs = (size_t)P.T * P.k;
    size_t lds = sizeof(uint32_t) * (masks + L.E);
    A.prefix = W > 1 && lds + 2 * masks <= 49152 ? 1 : 0;
    if (A.prefix) lds += 2 * masks;
    A.id_cache = lds + 2 * pairs <= 49152 ? 1 : 0;
    if (A.id_cache) lds += 2 * pairs;
    if (!P.do_group) lds = 0;
    // Tiled routing, also where the screen was asked for; it needs H a multiple of 256 (ks_max
    // > 0: the workspace holds no partial sums otherwise).  As many slices of the inputs as
    // give one round of resident workgroups (two per CU), two up to 352 tiles of long inputs,
    // whose slices outweigh a second round.  Step us with 1 / 2 / 4 / 8 slices: 235B-shaped
    // NVFP4 layer, T=64 264 / 259 / 257 / 258, T=256 (128 tiles) 318 / 313 / 311 / 322;
    // 480B-shaped T=1000 (630) 1,768 / 1,767 / 1,783 / 1,804.  Against four slices up to 256
    // tiles and two up to 512: 160 experts of 2,048 inputs T=256 (160 tiles) -6.6, T=336
    // (210) -9.5; 256 of 2,048 T=256 (256) -12; 128 of 2,048 T=384 (192) -7.7; with one slice
    // from 257: 160 of 6,144 T=432 (270) +5.1, 256 of 6,144 T=336 (336) +5.9, T=432 (432) -3.4.
    if (tile_routes(L, P)) {
        const int tt = (P.T + 15) / 16, et = (L.E + 15) / 16;
        int ks = tt * et <= 128 ? 4 : (tt * et <= (L.H >= 4096 ? 352 : 256) ? 2 : 1);
        while (ks > 1 && (ks > P.ks_max || ks > L.H / 256)) ks /= 2;
        A.KS = ks;
        const size_t lf = (size_t)16 * L.E * sizeof(float), bytes = lds > lf ? lds : lf;
        dim3 grid(ks, et, tt), block(256);
        if (L.act_bf16 && L.router_bf16)
            route_tile_kernel<uint16_t, uint16_t><<<grid, block, bytes, st>>>(A);
        else if (L.act_bf16)
            route_tile_kernel<uint16_t, float><<<grid, block, bytes, st>>>(A);
        else if (L.router_bf16)
            route_tile_kernel<float, uint16_t><<<grid, block, bytes, st>>>(A);
        else
            route_tile_kernel<float, float><<<grid, block, bytes, st>>>(A);
        return hipGetLastError();
    }
    // screened routing: bf16 activations and router, H a multiple of 256, enough work
    if (P.do_group && P.screen && L.act_bf16 && L.router_bf16 && P.ks_max > 0 && L.E <= kMaxE) {
        const int tiles = (P.T + 15) / 16, groups = (L.E + 63) / 64;
        const int waves = tiles * groups * 4;
        int ks = (2048 + waves - 1) / waves;  // about two waves per SIMD
        ks = ks < 1 ? 1 : (ks > P.ks_max ? P.ks_max : ks);
        A.KS = ks;
        A.screened = 1;
        screen_kernel<<<dim3(tiles, groups, ks), 256, 0, st>>>(A);
        route_cand_kernel<<<dim3(P.T), 256, lds, st>>>(A);
        return hipGetLastError();
    }
    dim3 grid(P.T * bpt), block(256);
    if (L.act_bf16 && L.router_bf16)
        route_kernel<uint16_t, uint16_t><<<grid, block, lds, st>>>(A);
    else if (L.act_bf16)
        route_kernel<uint16_t, float><<<grid, block, lds, st>>>(A);
    else if (L.router_bf16)
        route_kernel<float, uint16_t><<<grid, block, lds, st>>>(A);
    else
        route_kernel<float, float><<<grid, block, lds, st>>>(A);
    return hipGetLastError();
}

}  // namespace moe
