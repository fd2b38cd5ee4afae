// MFMA path of the grouped expert FFN: experts that received enough tokens in a
// step run as real dense contractions on the CDNA4 scaled matrix cores
// (v_mfma_scale_f32_16x16x128_f8f6f4), consuming the stored FP8-E4M3 or E2M1
// weights directly.  Activations enter as a 2-term FP8 split (hi + lo, E8M0 scale
// per 32 inputs, see fp8split.h): two MFMAs per tile, with the same error as bf16.
//
// Operand layout of the 16x16x128 instruction on gfx950 (pinned by an on-device
// probe): lane l holds row/column l%16; with g = l/16 an FP8 operand holds K
// [16g, 16g+16) and [64+16g, 64+16g+16) (two 16-byte pieces), an E2M1 operand K
// [32g, 32g+32) (16 bytes, low nibble first); the operand scale of lane l covers
// (row/column l%16, K block [32g, 32g+32)); the 16x16 fp32 result gives lane l rows
// 4g..4g+3 of column l%16.
//
// Every wave streams two 16-row weight tiles per work item (see stream_tiles).
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "fp8split.h"
#include "moe_internal.h"
#include "own.h"
#include "wave.h"

namespace moe {
namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline uint4 ld16(const uint8_t *p) { return *reinterpret_cast<const uint4 *>(p); }

// FP8 operand fragment of K block kb (p = row start + kb*128).  Weight fragments use
// ordinary loads: on this path they measured faster than non-temporal ones.
__device__ inline i32x8 frag_fp8(const uint8_t *p, int g)
{
    const uint4 a = ld16(p + 16 * g);
    const uint4 b = ld16(p + 64 + 16 * g);
    return (i32x8){(int)a.x, (int)a.y, (int)a.z, (int)a.w, (int)b.x, (int)b.y, (int)b.z, (int)b.w};
}

// E2M1 operand fragment of K block kb (p = row start + kb*64).
__device__ inline i32x8 frag_fp4(const uint8_t *p, int g)
{
    const uint4 a = ld16(p + 16 * g);
    return (i32x8){(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
}

// acc += s * (A . (Bhi*2^eh + Blo*2^el)) for FP8 weights (fp32 block scale s);
// acc += A*2^ea . (...) for E2M1 weights (E8M0 scale ea in the instruction).
template <int FMT>
__device__ inline void mma2(f32x4 &acc, const i32x8 &a, int ea, float s, const i32x8 &bh, int eh, const i32x8 &bl,
                            int el)
{
    if constexpr (FMT == 0) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
        t = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, bh, t, 0, 0, 0, 127, 0, eh);
        t = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, bl, t, 0, 0, 0, 127, 0, el);
        acc += s * t;
    } else {
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, bh, acc, 4, 0, 0, ea, 0, eh);
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, bl, acc, 4, 0, 0, ea, 0, el);
    }
}

// Fragments of one K block: NA weight tiles and NT token tiles.
template <int NA, int NT>
struct Frags {
    i32x8 a[NA];
    int ea[NA];
    i32x8 bh[NT], bl[NT];
    int eh[NT], el[NT];
};

// K loop over KB blocks with an S-stage register ring: the loads of block kb+S-1 are
// issued before block kb is multiplied, so S-1 blocks stay in flight.  Neither the
// prologue nor the steady state has conditional loads: the compiler's wait counts
// are exact only when every path issues the same loads, and a guarded load before
// the loop makes every iteration wait for all outstanding loads.  So the prologue
// always fills S-1 slots, with block KB-1 standing in for blocks past the end, and
// issues them slot by slot: the wait at the top of the loop is one count for the
// path from the prologue and the path from the previous iteration, and a slot's
// loads scheduled after a later slot's (the scheduler likes to sink the byte loads)
// would make it wait for nearly all.
template <int S, typename FR, typename LoadF, typename CompF>
__device__ inline void k_pipeline(int KB, FR (&F)[S], LoadF load, CompF compute)
{
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {
        load(F[s], s < KB ? s : KB - 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    int kb = 0;
    for (; kb + 2 * S - 1 <= KB; kb += S) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            load(F[(s + S - 1) % S], kb + s + S - 1);
            compute(F[s], kb + s);
        }
    }
    // fewer than 2S-1 blocks remain; block kb+s sits in F[s % S]
#pragma unroll
    for (int s = 0; s < 2 * S - 2; ++s) {
        if (kb + s < KB) {
            if (kb + s + S - 1 < KB) load(F[(s + S - 1) % S], kb + s + S - 1);
            compute(F[s % S], kb + s);
        }
    }
}

// ------------------------------------------------------------------ activation operand
//
// Activation fragments are read through raw buffer resources sized to the step's
// data.  Lanes whose token column lies past the chunk use an offset beyond the
// resource, which the hardware answers with zeros and no memory request: the
// activation traffic through the L1 then scales with the chunk's real tokens, and
// no branch guards the loads (a branch around loads makes every K block wait for
// all outstanding loads).  An output column depends only on its own activation
// column, and columns past the chunk are never stored.

typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
constexpr uint32_t kOutOfRange = 0x80000000u;
constexpr int kRawBufferWord3 = 0x00020000;  // untyped 32-bit data format, no swizzle

__device__ inline __amdgpu_buffer_rsrc_t raw_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, kRawBufferWord3);
}

// FP8 fragment of a K block: bytes [16g, 16g+16) and [64+16g, 64+16g+16) at voff+soff.
__device__ inline i32x8 frag_buf(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    const u32x4v a = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    const u32x4v b = __builtin_amdgcn_raw_buffer_load_b128(r, voff + 64, soff, 0);
    return (i32x8){(int)a.x, (int)a.y, (int)a.z, (int)a.w, (int)b.x, (int)b.y, (int)b.z, (int)b.w};
}

// The four resources of a split activation buffer [rows][K] (hi, lo codes) and
// [rows][K/32] (hi, lo exponents) holding `rows` rows.
struct ActRsrc {
    __amdgpu_buffer_rsrc_t hi, lo, ehi, elo;
};

__device__ inline ActRsrc act_rsrc(const uint8_t *hi, const uint8_t *lo, const uint8_t *ehi, const uint8_t *elo,
                                   uint32_t rows, uint32_t K)
{
    return ActRsrc{raw_rsrc(hi, rows * K), raw_rsrc(lo, rows * K), raw_rsrc(ehi, rows * (K / 32)),
                   raw_rsrc(elo, rows * (K / 32))};
}

// Weight layouts.  Row-major (PK = false): a matrix [rows][K] with K contiguous.
// Packed 16-row tiles (PK = true): each tile of 16 rows keeps its place and size, and
// inside it each 128-input K block is one contiguous piece holding the operand
// fragments in lane order: FP8 2 KB, lane l's bytes K [16g, 16g+16) of row l%16 at
// 16l and K [64+16g, 64+16g+16) at 1024 + 16l (g = l/16); E2M1 1 KB, lane l's 16
// bytes (K [32g, 32g+32) of row l%16) at 16l.  A load instruction of a wave then reads
// 1 KB of contiguous bytes; on this GPU such a stream runs at 6.8-6.9 TB/s with
// non-temporal loads, against 6.0-6.2 TB/s for the row-major walk with either kind.
// The tile is the same for the whole wave, so packed fragments are read through a
// buffer resource on it (scalar registers), the lane's offset 16l and the block's
// offset as a scalar.  With packed E2M1 weights the E8M0 scales are packed too: inside
// each 16-row tile, per group of four K blocks, lane l's four scale bytes (K sub-block
// g of row l%16 in blocks 4q..4q+3) sit together at 4l of a 256-byte piece (a final
// group of two blocks: 2 bytes per lane, 128 bytes).  Read row by row, one byte per
// lane and block, the scales bound the E2M1 kernels.
constexpr int kNonTemporal = 2;  // cache policy of a non-temporal buffer load

// This lane's weight pointer for the 16-row tile starting at row `row0` (a multiple of
// 16) of a matrix with `rowb` bytes per row: its row (row-major) or the tile (packed).
template <bool PK>
__device__ inline const uint8_t *wlane(const uint8_t *mat, int row0, size_t rowb, int lane)
{
    return PK ? mat + (size_t)row0 * rowb : mat + (size_t)(row0 + (lane & 15)) * rowb;
}

__device__ inline __amdgpu_buffer_rsrc_t tile_rsrc(const uint8_t *tile)
{
    const uint64_t a = (uint64_t)tile;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)hi << 32) | lo), (short)0, -1, kRawBufferWord3);
}

// E8M0 scale byte of K block kb (of KB) from a packed tile's scales `et` (byte reads:
// the two-tile kernels; the staged ones read a word per four blocks).
__device__ inline int e8m0_packed(const uint8_t *et, int kb, int KB, int lane)
{
    const int q = kb >> 2, rem = min(4, KB - 4 * q);
    return et[256 * q + lane * rem + (kb & 3)];
}

// Weight operand fragment of K block kb from a pointer of wlane.
template <int FMT, bool PK>
__device__ inline i32x8 wfrag(const uint8_t *a, int kb, int g)
{
    if constexpr (PK) {
        const __amdgpu_buffer_rsrc_t r = tile_rsrc(a);
        const uint32_t v = 16u * (uint32_t)__lane_id();
        if constexpr (FMT == 0) {
            const u32x4v x = __builtin_amdgcn_raw_buffer_load_b128(r, v, kb * 2048, kNonTemporal);
            const u32x4v y = __builtin_amdgcn_raw_buffer_load_b128(r, v + 1024, kb * 2048, kNonTemporal);
            return (i32x8){(int)x.x, (int)x.y, (int)x.z, (int)x.w, (int)y.x, (int)y.y, (int)y.z, (int)y.w};
        } else {
            // ordinary loads for E2M1 tiles: an expert with several token chunks re-reads
            // its tiles, and the non-temporal policy made those re-reads miss the caches
            // (4-bit MXFP4 layer at 256 tokens per step: 1.31x its algorithmic bytes
            // fetched, 997k against 1,036k tokens/s with ordinary loads)
            const u32x4v x = __builtin_amdgcn_raw_buffer_load_b128(r, v, kb * 1024, 0);
            return (i32x8){(int)x.x, (int)x.y, (int)x.z, (int)x.w, 0, 0, 0, 0};
        }
    } else {
        if constexpr (FMT == 0)
            return frag_fp8(a + (size_t)kb * 128, g);
        else
            return frag_fp4(a + (size_t)kb * 64, g);
    }
}

// ------------------------------------------------------------------ two weight tiles
//
// A wave streams two 16-row weight tiles (this lane's rows arow[0], arow[1]) over KB
// K blocks against NT 16-token tiles, accumulating acc[t][j] (lane l: rows 4g..4g+3
// of token column l%16).  Two tiles per wave balance the two costs measured on this
// GPU: each extra concurrently streamed tile lowers the HBM rate (one: 6.3 TB/s,
// four: 5.2 TB/s), each activation fragment load is paid per tile pair.
//   arow[t]  weight row of this lane in tile t (FP8: KB*128 bytes, E2M1: KB*64 bytes)
//   erow[t]  E8M0 scales of that row (E2M1 only), one per 32 inputs
//   sblk[t]  fp32 block scale of tile t per K block (FP8 only)
//   voff[j], eoff[j]  this lane's byte offset of its token row in the code and
//                     exponent buffers (kOutOfRange past the chunk)
template <int FMT, int NT, int S, bool PK>
__device__ inline void stream_tiles(f32x4 (&acc)[2][NT], const uint8_t *const (&arow)[2],
                                    const uint8_t *const (&erow)[2], const float *const (&sblk)[2], int KB,
                                    const ActRsrc &B, const uint32_t (&voff)[NT], const uint32_t (&eoff)[NT], int g)
{
    auto load = [&](Frags<2, NT> &F, int kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            F.a[t] = wfrag<FMT, PK>(arow[t], kb, g);
            F.ea[t] = FMT == 0 ? 127 : (PK ? e8m0_packed(erow[t], kb, KB, __lane_id()) : erow[t][kb * 4 + g]);
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            F.bh[j] = frag_buf(B.hi, voff[j], kb * 128);
            F.bl[j] = frag_buf(B.lo, voff[j], kb * 128);
            F.eh[j] = __builtin_amdgcn_raw_buffer_load_b8(B.ehi, eoff[j], kb * 4, 0);
            F.el[j] = __builtin_amdgcn_raw_buffer_load_b8(B.elo, eoff[j], kb * 4, 0);
        }
    };
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto compute = [&](const Frags<2, NT> &F, int kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const float s = FMT == 0 ? sblk[t][kb] : 1.f;
#pragma unroll
            for (int j = 0; j < NT; ++j)
                mma2<FMT>(acc[t][j], F.a[t], F.ea[t], s, F.bh[j], F.eh[j], F.bl[j], F.el[j]);
        }
    };
    Frags<2, NT> F[S];
    k_pipeline<S>(KB, F, load, compute);
}

// stream_tiles for a block count KBC fixed at compile time and fully unrolled.  The
// activations' E8M0 exponents of the lane's token rows are read up front, 16 bytes
// (four K blocks) per load, instead of one byte load per block and token tile: on
// the 235B-shaped down projection (12 K blocks) the byte loads were a fifth of the
// K loop's memory instructions.
//   erow_off[j]  byte offset of the lane's token row in the exponent buffers
//                (kOutOfRange past the chunk)
template <int FMT, int NT, int S, int KBC, bool PK>
__device__ inline void stream_tiles_fixed(f32x4 (&acc)[2][NT], const uint8_t *const (&arow)[2],
                                          const uint8_t *const (&erow)[2], const float *const (&sblk)[2],
                                          const ActRsrc &B, const uint32_t (&voff)[NT],
                                          const uint32_t (&erow_off)[NT], int g)
{
    static_assert(KBC % 4 == 0 && S >= 2, "whole 16-byte exponent loads");
    constexpr int Q = KBC / 4;
    u32x4v exh[NT][Q], exl[NT][Q];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            exh[j][q] = __builtin_amdgcn_raw_buffer_load_b128(B.ehi, erow_off[j], q * 16, 0);
            exl[j][q] = __builtin_amdgcn_raw_buffer_load_b128(B.elo, erow_off[j], q * 16, 0);
        }
    auto load = [&](Frags<2, NT> &F, int kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            F.a[t] = wfrag<FMT, PK>(arow[t], kb, g);
            F.ea[t] = FMT == 0 ? 127 : (PK ? e8m0_packed(erow[t], kb, KBC, __lane_id()) : erow[t][kb * 4 + g]);
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            F.bh[j] = frag_buf(B.hi, voff[j], kb * 128);
            F.bl[j] = frag_buf(B.lo, voff[j], kb * 128);
        }
    };
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto compute = [&](const Frags<2, NT> &F, int kb) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const float sc = FMT == 0 ? sblk[t][kb] : 1.f;
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int eh = (int)__builtin_amdgcn_ubfe(exh[j][kb / 4][kb % 4], 8 * g, 8);
                const int el = (int)__builtin_amdgcn_ubfe(exl[j][kb / 4][kb % 4], 8 * g, 8);
                mma2<FMT>(acc[t][j], F.a[t], F.ea[t], sc, F.bh[j], eh, F.bl[j], el);
            }
        }
    };
    Frags<2, NT> F[S];
#pragma unroll
    for (int kb = 0; kb < S - 1; ++kb) load(F[kb], kb);
#pragma unroll
    for (int kb = 0; kb < KBC; ++kb) {
        if (kb + S - 1 < KBC) load(F[(kb + S - 1) % S], kb + S - 1);
        compute(F[kb % S], kb);
    }
}

// This lane's token-row offsets for the NT token tiles of a chunk.
template <int NT>
__device__ inline void token_offsets(uint32_t (&voff)[NT], uint32_t (&eoff)[NT], const int32_t *__restrict__ row_of,
                                     int slot0, int mc, int K, int r, int g)
{
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int m = 16 * j + r;
        const uint32_t row = m < mc ? (uint32_t)(row_of ? row_of[slot0 + m] : slot0 + m) : 0u;
        voff[j] = m < mc ? row * (uint32_t)K + 16u * g : kOutOfRange;
        eoff[j] = m < mc ? row * (uint32_t)(K / 32) + (uint32_t)g : kOutOfRange;
    }
}

// ------------------------------------------------------------------ gate/up + SiLU-gate
//
// Work item = (chunk of up to 32 tokens of one expert, rows [i0, i0+64) of the
// intermediate dimension) for a workgroup of four waves.  Wave w takes rows
// r0 = i0 + 16w .. r0+16 of both the gate and the up matrix, so h = silu(g)*u forms
// in its registers.  The 2-term split of h groups 32 rows (one E8M0 exponent per
// token and group): waves 2q and 2q+1 share group q and exchange their column
// maxima through LDS.

template <int FMT, int NT, int S, bool PK>
__device__ inline void w13_rows(int w, const uint8_t *__restrict__ we, const uint8_t *__restrict__ se, int H, int I,
                                int i0, int slot0, int mc, const int32_t *__restrict__ tok_of, const ActRsrc &X,
                                uint8_t *__restrict__ hs_hi, uint8_t *__restrict__ hs_lo,
                                uint8_t *__restrict__ he_hi, uint8_t *__restrict__ he_lo, float (&s_am)[4][2][16],
                                float (&s_rm)[4][2][16], int lane)
{
    const int r = lane & 15, g = lane >> 4;
    const int r0 = i0 + 16 * w;  // first row of this wave in the gate and in the up matrix
    const size_t rowb = FMT == 0 ? (size_t)H : (size_t)H / 2;
    const uint8_t *arow[2] = {wlane<PK>(we, r0, rowb, lane), wlane<PK>(we, I + r0, rowb, lane)};
    const int er = PK ? 0 : r;  // packed scales: the tile's
    const uint8_t *erow[2] = {se + (size_t)(r0 + er) * (H / 32), se + (size_t)(I + r0 + er) * (H / 32)};
    const float *sblk[2] = {(const float *)se + (size_t)(r0 / 128) * (H / 128),
                            (const float *)se + (size_t)((I + r0) / 128) * (H / 128)};
    uint32_t voff[NT], eoff[NT];
    token_offsets<NT>(voff, eoff, tok_of, slot0, mc, H, r, g);
    f32x4 acc[2][NT];
    stream_tiles<FMT, NT, S, PK>(acc, arow, erow, sblk, H / 128, X, voff, eoff, g);

    // epilogue: h = silu(g)*u for rows r0 + 4g + i of token column r of each tile
    float h[NT][4], res[NT][4];
    float am[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float gi = acc[0][j][i];
            h[j][i] = gi / (1.0f + expf(-gi)) * acc[1][j][i];
        }
        float m = amax_of(h[j]);
        m = fmaxf(m, __shfl_xor(m, 16));
        am[j] = fmaxf(m, __shfl_xor(m, 32));
        if (g == 0) s_am[w][j][r] = am[j];
    }
    __syncthreads();
    int ch[NT];
    uint32_t qh[NT][1], ql[NT][1];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        ch[j] = exp_for_group(fmaxf(am[j], s_am[w ^ 1][j][r]));
        split_hi(h[j], ch[j], qh[j], res[j]);
        float m = amax_of(res[j]);
        m = fmaxf(m, __shfl_xor(m, 16));
        am[j] = fmaxf(m, __shfl_xor(m, 32));
        if (g == 0) s_rm[w][j][r] = am[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int cl = exp_for_group(fmaxf(am[j], s_rm[w ^ 1][j][r]));
        split_lo(res[j], cl, ql[j]);
        if (16 * j + r < mc) {
            const size_t slot = (size_t)slot0 + 16 * j + r;
            *reinterpret_cast<uint32_t *>(hs_hi + slot * I + r0 + 4 * g) = qh[j][0];
            *reinterpret_cast<uint32_t *>(hs_lo + slot * I + r0 + 4 * g) = ql[j][0];
            if ((w & 1) == 0 && g == 0) {
                he_hi[slot * (I / 32) + r0 / 32] = (uint8_t)ch[j];
                he_lo[slot * (I / 32) + r0 / 32] = (uint8_t)cl;
            }
        }
    }
}

template <int FMT, bool PK>
__global__ __launch_bounds__(256) void w13_mfma_kernel(const uint8_t *__restrict__ ew, const uint8_t *__restrict__ es,
                                                       const int32_t *__restrict__ meta,
                                                       const int32_t *__restrict__ tok_of,
                                                       const uint8_t *__restrict__ xs_hi,
                                                       const uint8_t *__restrict__ xs_lo,
                                                       const uint8_t *__restrict__ xe_hi,
                                                       const uint8_t *__restrict__ xe_lo, uint8_t *__restrict__ hs_hi,
                                                       uint8_t *__restrict__ hs_lo, uint8_t *__restrict__ he_hi,
                                                       uint8_t *__restrict__ he_lo, int T, int H, int I, int E,
                                                       size_t ewb, size_t esb)
{
    __shared__ float s_am[4][2][16], s_rm[4][2][16];
    const MetaIdx mi{E};
    const int tiles = I / 64;
    const int n_items = meta[mi.n_mfma_chunks()] * tiles;
    const int4 *recs = reinterpret_cast<const int4 *>(meta + mi.chunk_rec());
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ActRsrc X = act_rsrc(xs_hi, xs_lo, xe_hi, xe_lo, (uint32_t)T, (uint32_t)H);
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int4 rec = recs[item / tiles];  // {expert, first slot, tokens, -}
        const int i0 = (item % tiles) * 64;
        const uint8_t *we = ew + (size_t)rec.x * ewb;
        const uint8_t *se = es + (size_t)rec.x * esb;
        if (rec.z > 16)
            w13_rows<FMT, 2, 2, PK>(wave, we, se, H, I, i0, rec.y, rec.z, tok_of, X, hs_hi, hs_lo, he_hi, he_lo, s_am,
                                s_rm, lane);
        else
            w13_rows<FMT, 1, 3, PK>(wave, we, se, H, I, i0, rec.y, rec.z, tok_of, X, hs_hi, hs_lo, he_hi, he_lo, s_am,
                                s_rm, lane);
    }
}

// ------------------------------------------------------------------ down projection
//
// Work item = (chunk of up to 32 tokens of one expert, 32 output rows [n0, n0+32)) for
// one wave; the four waves of a workgroup take consecutive row pairs of a chunk and
// so share its activation fragments through the L1 cache.  A chunk of at most 16
// tokens keeps three K blocks in flight on packed weights (the 480B TP4 shard's down
// projection: 81.7 -> 78.2 us at T=48), two on row-major ones.

template <int FMT, int NT, int S, bool PK>
__device__ inline void w2_rows(const uint8_t *__restrict__ we2, const uint8_t *__restrict__ se, int H, int I, int n0,
                               int slot0, int mc, const ActRsrc &Hs, float *__restrict__ obuf, int lane)
{
    const int r = lane & 15, g = lane >> 4;
    const size_t rowb = FMT == 0 ? (size_t)I : (size_t)I / 2;
    const uint8_t *sd8 = se + (size_t)2 * I * (H / 32);  // MXFP4 down scales
    const uint8_t *arow[2] = {wlane<PK>(we2, n0, rowb, lane), wlane<PK>(we2, n0 + 16, rowb, lane)};
    const int er = PK ? 0 : r;  // packed scales: the tile's
    const uint8_t *erow[2] = {sd8 + (size_t)(n0 + er) * (I / 32), sd8 + (size_t)(n0 + 16 + er) * (I / 32)};
    const float *sd = (const float *)se + (size_t)2 * (I / 128) * (H / 128);
    const float *sblk[2] = {sd + (size_t)(n0 / 128) * (I / 128), sd + (size_t)((n0 + 16) / 128) * (I / 128)};
    uint32_t voff[NT], eoff[NT];
    token_offsets<NT>(voff, eoff, nullptr, slot0, mc, I, r, g);
    f32x4 acc[2][NT];
    if (I == 12 * 128) {  // the 235B-shaped layer
        uint32_t erow_off[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) erow_off[j] = eoff[j] - (uint32_t)g;
        stream_tiles_fixed<FMT, NT, S, 12, PK>(acc, arow, erow, sblk, Hs, voff, erow_off, g);
    } else {
        stream_tiles<FMT, NT, S, PK>(acc, arow, erow, sblk, I / 128, Hs, voff, eoff, g);
    }
#pragma unroll
    for (int j = 0; j < NT; ++j)
        if (16 * j + r < mc) {
            const size_t slot = (size_t)slot0 + 16 * j + r;
#pragma unroll
            for (int t = 0; t < 2; ++t)
                *reinterpret_cast<f32x4 *>(obuf + slot * H + n0 + 16 * t + 4 * g) = acc[t][j];
        }
}

template <int FMT, bool PK>
__global__ __launch_bounds__(256) void w2_mfma_kernel(const uint8_t *__restrict__ ew, const uint8_t *__restrict__ es,
                                                      const int32_t *__restrict__ meta,
                                                      const uint8_t *__restrict__ hs_hi,
                                                      const uint8_t *__restrict__ hs_lo,
                                                      const uint8_t *__restrict__ he_hi,
                                                      const uint8_t *__restrict__ he_lo, float *__restrict__ obuf,
                                                      int P, int H, int I, int E, size_t ewb, size_t esb)
{
    const MetaIdx mi{E};
    const int tiles = H / 32;
    const int n_items = meta[mi.n_mfma_chunks()] * tiles;
    const int4 *recs = reinterpret_cast<const int4 *>(meta + mi.chunk_rec());
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t w2off = FMT == 0 ? (size_t)2 * I * H : (size_t)I * H;
    const ActRsrc Hs = act_rsrc(hs_hi, hs_lo, he_hi, he_lo, (uint32_t)P, (uint32_t)I);
    for (int item = blockIdx.x * 4 + wave; item < n_items; item += gridDim.x * 4) {
        const int4 rec = recs[item / tiles];
        const int n0 = (item % tiles) * 32;
        const uint8_t *we2 = ew + (size_t)rec.x * ewb + w2off;
        const uint8_t *se = es + (size_t)rec.x * esb;
        if (rec.z > 16)
            w2_rows<FMT, 2, 2, PK>(we2, se, H, I, n0, rec.y, rec.z, Hs, obuf, lane);
        else
            w2_rows<FMT, 1, PK ? 4 : 3, PK>(we2, se, H, I, n0, rec.y, rec.z, Hs, obuf, lane);
    }
}

// ------------------------------------------------------------------ LDS-staged activations
//
// When K spans a multiple of four 128-input blocks (every production shape), a work
// item is one workgroup of four waves over one chunk, and each wave streams exactly
// one 16-row weight tile with a four-deep register ring.  The chunk's split
// activations are staged once per workgroup in LDS, in double-buffered segments of
// four K blocks, and every wave reads its fragments from there.  Measured on this GPU,
// a wave streaming one tile reaches 6.3 TB/s and one streaming two 5.6 TB/s, but one
// tile per wave pays a full activation fragment per weight fragment when each wave
// fetches its own; staging removes that cost.

constexpr int kSegK = 4;                // K blocks per staged segment
constexpr int kSegBytes = kSegK * 128;  // activation bytes per token row and segment
constexpr int kStageTok = 32;           // token rows of a chunk

struct alignas(16) ActSeg {
    uint8_t code[2][kStageTok][kSegBytes];  // [hi, lo][token][16-byte pieces, swizzled]
    uint8_t ex[2][kStageTok][kSegK * 4];    // [hi, lo][token][E8M0 per 32 inputs]
    uint8_t sink[kSegK * 4];                // target of the threads that stage no exponents
};

// Piece c (16 bytes) of token t's 512-byte segment row is stored at piece swz(c, t):
// the low four bits of the piece index are XORed with the token, so the 16 tokens of a
// fragment read (one 16-lane group) fall on 16 distinct 16-byte bank groups of the
// 64-bank LDS.  A three-bit XOR left pairs of tokens on one bank group: the counters
// showed bank-conflict stalls in about 40 % of the LDS's active cycles.
__device__ inline int swz(int c, int t) { return (c & ~15) | ((c ^ t) & 15); }

__device__ inline void sync_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One thread's share of staging a segment for a workgroup of W waves: piece tid%32
// of token rows 2W*q + tid/32 (q < 8*NT/W) in both the hi and lo codes; threads
// tid < 32 also stage token tid's exponent bytes of each.  Every thread issues the
// same loads (tokens past the chunk read out of range), so the loads need no branch.
template <int NT, int W>
struct Stager {
    static_assert(W == 4 || W == 8, "four or eight waves per workgroup");
    static constexpr int Q = 8 * NT / W;
    uint32_t voff[Q];  // byte offset of this thread's piece in its token rows, segment 0
    uint32_t eoff;     // exponent offset of token tid, segment 0 (out of range if none)
    int tok[Q];
    int piece;
    u32x4v code[2][Q];
    u32x4v ex[2];

    __device__ void init(const int32_t *__restrict__ row_of, int slot0, int mc, int K, int tid)
    {
        piece = tid & 31;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int t = 2 * W * q + (tid >> 5);
            tok[q] = t;
            const uint32_t row = t < mc ? (uint32_t)(row_of ? row_of[slot0 + t] : slot0 + t) : 0u;
            voff[q] = t < mc ? row * (uint32_t)K + 16u * piece : kOutOfRange;
        }
        const uint32_t erow = tid < mc ? (uint32_t)(row_of ? row_of[slot0 + tid] : slot0 + tid) : 0u;
        eoff = (tid < 32 && tid < mc) ? erow * (uint32_t)(K / 32) : kOutOfRange;
    }
    // segment sg (callers clamp it to the last segment)
    __device__ void load(const ActRsrc &B, int sg)
    {
        const uint32_t d = (uint32_t)sg * kSegBytes, de = (uint32_t)sg * (kSegK * 4);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            code[0][q] = __builtin_amdgcn_raw_buffer_load_b128(B.hi, voff[q] + d, 0, 0);
            code[1][q] = __builtin_amdgcn_raw_buffer_load_b128(B.lo, voff[q] + d, 0, 0);
        }
        ex[0] = __builtin_amdgcn_raw_buffer_load_b128(B.ehi, eoff + de, 0, 0);
        ex[1] = __builtin_amdgcn_raw_buffer_load_b128(B.elo, eoff + de, 0, 0);
    }
    __device__ void store(ActSeg &S, int tid) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < Q; ++q)
                *reinterpret_cast<u32x4v *>(&S.code[h][tok[q]][swz(piece, tok[q]) * 16]) = code[h][q];
        uint8_t *e0 = tid < 32 ? &S.ex[0][tid][0] : S.sink;
        uint8_t *e1 = tid < 32 ? &S.ex[1][tid][0] : S.sink;
        *reinterpret_cast<u32x4v *>(e0) = ex[0];
        *reinterpret_cast<u32x4v *>(e1) = ex[1];
    }
};

// Streams this wave's NA weight tiles (this lane's rows arow[a]) over KB K blocks (KB a
// multiple of 4) against NT staged token tiles; acc[a][j] as in stream_tiles.  Each
// activation fragment read from LDS feeds the NA tiles' MFMAs.  All W waves of the
// workgroup call it together: it synchronises them once per staged segment (four K
// blocks).  On return no wave reads `seg` any more.
template <int FMT, int NT, int W, int NA, bool PK>
__device__ inline void stream_tile_lds(f32x4 (&acc)[NA][NT], const uint8_t *const (&arow)[NA],
                                       const uint8_t *const (&erow)[NA], const float *const (&sblk)[NA], int KB,
                                       const ActRsrc &B, Stager<NT, W> &st, ActSeg (&seg)[2], int lane, int tid)
{
    const int r = lane & 15, g = lane >> 4;
    const int nseg = KB / kSegK;
    i32x8 A[4][NA];
    int EA[4][NA];
    // packed E8M0 scales: one word per lane, tile and segment of four blocks, a segment ahead
    __amdgpu_buffer_rsrc_t er[NA];
    if constexpr (PK && FMT == 1) {
#pragma unroll
        for (int a = 0; a < NA; ++a) er[a] = tile_rsrc(erow[a]);
    }
    auto eword = [&](uint32_t (&w)[NA], int sg) {
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            if constexpr (PK && FMT == 1)
                w[a] = __builtin_amdgcn_raw_buffer_load_b32(er[a], 4u * lane, sg * 256, 0);
            else
                w[a] = 0u;
        }
    };
    // Packed E8M0 scales are taken from the segment's words when the block is multiplied,
    // not when its weights are loaded: the next segment's words arrive during this one,
    // and reading them at the load of the next segment's first block made every wave
    // wait there for all but its five newest loads (MXFP4 Zipf layer at T=256: gate/up
    // 120.0 -> 118.8 us in four-wave workgroups, 116.0 -> 115.5 us in eight-wave ones).
    uint32_t wc[NA], wn[NA];  // words of the segment being multiplied and of the next one
    auto loadA = [&](int slot, int kb) {
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            A[slot][a] = wfrag<FMT, PK>(arow[a], kb, g);
            if constexpr (FMT == 0)
                EA[slot][a] = 127;
            else if constexpr (!PK)
                EA[slot][a] = erow[a][kb * 4 + g];
        }
    };
    auto compute = [&](int slot, const ActSeg &S, int kk, int kb) {
        float sc[NA];
#pragma unroll
        for (int a = 0; a < NA; ++a) sc[a] = FMT == 0 ? sblk[a][kb] : 1.f;
        if constexpr (FMT == 1 && PK) {
#pragma unroll
            for (int a = 0; a < NA; ++a) EA[slot][a] = (int)__builtin_amdgcn_ubfe(wc[a], 8 * kk, 8);
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int t = 16 * j + r;
            const u32x4v h0 = *reinterpret_cast<const u32x4v *>(&S.code[0][t][swz(kk * 8 + g, t) * 16]);
            const u32x4v h1 = *reinterpret_cast<const u32x4v *>(&S.code[0][t][swz(kk * 8 + 4 + g, t) * 16]);
            const u32x4v l0 = *reinterpret_cast<const u32x4v *>(&S.code[1][t][swz(kk * 8 + g, t) * 16]);
            const u32x4v l1 = *reinterpret_cast<const u32x4v *>(&S.code[1][t][swz(kk * 8 + 4 + g, t) * 16]);
            const i32x8 bh = {(int)h0.x, (int)h0.y, (int)h0.z, (int)h0.w, (int)h1.x, (int)h1.y, (int)h1.z, (int)h1.w};
            const i32x8 bl = {(int)l0.x, (int)l0.y, (int)l0.z, (int)l0.w, (int)l1.x, (int)l1.y, (int)l1.z, (int)l1.w};
            const int eh = S.ex[0][t][kk * 4 + g], el = S.ex[1][t][kk * 4 + g];
#pragma unroll
            for (int a = 0; a < NA; ++a) mma2<FMT>(acc[a][j], A[slot][a], EA[slot][a], sc[a], bh, eh, bl, el);
        }
    };
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[a][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    eword(wc, 0);
    loadA(0, 0);
    loadA(1, 1);
    loadA(2, 2);
    st.load(B, 0);
    st.store(seg[0], tid);
    st.load(B, nseg > 1 ? 1 : 0);
    sync_lds();
    for (int kb = 0; kb < KB; kb += kSegK) {  // one staged segment per iteration
        const int sg = kb / kSegK;
        const ActSeg &cur = seg[sg & 1];
        eword(wn, min(sg + 1, nseg - 1));  // the last segment's past the end
#pragma unroll
        for (int u = 0; u < kSegK; ++u) {
            // block kb+3 is this segment's, kb+4.. the next one's; past the end: reload the last block.
            // The scheduling barrier keeps each block's loads here: left to itself the
            // scheduler sinks the next segment's loads to the end of the segment, and every
            // segment then starts with a full memory latency.
            loadA((u + 3) & 3, min(kb + u + 3, KB - 1));
            __builtin_amdgcn_sched_barrier(0);
            compute(u, cur, u, kb + u);
        }
#pragma unroll
        for (int a = 0; a < NA; ++a) wc[a] = wn[a];
        st.store(seg[(sg + 1) & 1], tid);
        st.load(B, min(sg + 2, nseg - 1));
        sync_lds();
    }
}

// gate/up: item = (chunk, NA*8W rows of the intermediate dimension) for W waves; wave w
// streams NA gate (w < W/2) or up (w >= W/2) tiles, rows i0 + 16*q for tiles
// q = NA*(w % (W/2)) + a.  The accumulators meet in LDS (over the staging buffer the
// last segment no longer needs) and wave w forms h and its 2-term split for the pairs
// e = w, w + W, ... < NT*NA*W/4 of token tile e % NT and 32-row group e / NT (32 rows are
// one E8M0 group per token).
template <int FMT, int NT, int W, int NA, bool PK>
__device__ inline void w13_item_lds(const uint8_t *__restrict__ we, const uint8_t *__restrict__ se, int H, int I,
                                    int i0, int slot0, int mc, const int32_t *__restrict__ tok_of, const ActRsrc &X,
                                    uint8_t *__restrict__ hs_hi, uint8_t *__restrict__ hs_lo,
                                    uint8_t *__restrict__ he_hi, uint8_t *__restrict__ he_lo, ActSeg (&seg)[2],
                                    int wave, int lane, int tid)
{
    constexpr int HW = W / 2;       // waves per projection
    constexpr int NQ = HW * NA;     // tiles per projection
    constexpr int NG = NQ / 2;      // 32-row groups per item
    const int r = lane & 15, g = lane >> 4;
    const size_t rowb = FMT == 0 ? (size_t)H : (size_t)H / 2;
    const uint8_t *arow[NA];
    const uint8_t *erow[NA];
    const float *sblk[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        const int row0 = (wave >= HW ? I : 0) + i0 + 16 * (NA * (wave % HW) + a);
        arow[a] = wlane<PK>(we, row0, rowb, lane);
        erow[a] = se + (size_t)(row0 + (PK ? 0 : r)) * (H / 32);
        sblk[a] = (const float *)se + (size_t)(row0 / 128) * (H / 128);
    }
    Stager<NT, W> st;
    st.init(tok_of, slot0, mc, H, tid);
    f32x4 acc[NA][NT];
    stream_tile_lds<FMT, NT, W, NA, PK>(acc, arow, erow, sblk, H / 128, X, st, seg, lane, tid);
    // red[(proj*NQ + q)*NT + j][lane]: 2*NQ*NT*64 f32x4.  Where they fit in seg[1].code,
    // which the next item first writes after its first barrier, no wave still reads red
    // by then; otherwise red starts at seg[0] and a barrier follows its last read.
    constexpr bool kRedAll = sizeof(f32x4) * 2 * NQ * NT * 64 > sizeof(seg[1].code);
    static_assert(sizeof(f32x4) * 2 * NQ * NT * 64 <= sizeof(seg), "reduction buffer");
    f32x4 *red = kRedAll ? reinterpret_cast<f32x4 *>(&seg[0]) : reinterpret_cast<f32x4 *>(&seg[1].code[0][0][0]);
    auto ridx = [&](int proj, int q, int j) { return ((proj * NQ + q) * NT + j) * 64 + lane; };
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int j = 0; j < NT; ++j) red[ridx(wave / HW, NA * (wave % HW) + a, j)] = acc[a][j];
    sync_lds();
    for (int e = wave; e < NG * NT; e += W) {  // one (group, token tile) per wave and pass
        const int j = e % NT, grp = e / NT;
        const f32x4 g0 = red[ridx(0, 2 * grp, j)], g1 = red[ridx(0, 2 * grp + 1, j)];
        const f32x4 u0 = red[ridx(1, 2 * grp, j)], u1 = red[ridx(1, 2 * grp + 1, j)];
        float h[8], res[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h[i] = g0[i] / (1.0f + expf(-g0[i])) * u0[i];
            h[4 + i] = g1[i] / (1.0f + expf(-g1[i])) * u1[i];
        }
        float am = amax_of(h);
        am = fmaxf(am, __shfl_xor(am, 16));
        am = fmaxf(am, __shfl_xor(am, 32));
        const int ch = exp_for_group(am);
        uint32_t qh[2], ql[2];
        split_hi(h, ch, qh, res);
        float rm = amax_of(res);
        rm = fmaxf(rm, __shfl_xor(rm, 16));
        rm = fmaxf(rm, __shfl_xor(rm, 32));
        const int cl = exp_for_group(rm);
        split_lo(res, cl, ql);
        if (16 * j + r < mc) {
            const size_t slot = (size_t)slot0 + 16 * j + r;
            const int c0 = i0 + 32 * grp;
            uint8_t *ph = hs_hi + slot * I + c0 + 4 * g;
            uint8_t *pl = hs_lo + slot * I + c0 + 4 * g;
            *reinterpret_cast<uint32_t *>(ph) = qh[0];
            *reinterpret_cast<uint32_t *>(ph + 16) = qh[1];
            *reinterpret_cast<uint32_t *>(pl) = ql[0];
            *reinterpret_cast<uint32_t *>(pl + 16) = ql[1];
            if (g == 0) {
                he_hi[slot * (I / 32) + c0 / 32] = (uint8_t)ch;
                he_lo[slot * (I / 32) + c0 / 32] = (uint8_t)cl;
            }
        }
    }
    if constexpr (kRedAll) sync_lds();
}

template <int FMT, int W, int NA, bool PK>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W == 8 ? (FMT == 1 ? 2 : 4) : 1))) void w13_mfma_lds_kernel(
    const uint8_t *__restrict__ ew, const uint8_t *__restrict__ es, const int32_t *__restrict__ meta,
    const int32_t *__restrict__ tok_of, const uint8_t *__restrict__ xs_hi, const uint8_t *__restrict__ xs_lo,
    const uint8_t *__restrict__ xe_hi, const uint8_t *__restrict__ xe_lo, uint8_t *__restrict__ hs_hi,
    uint8_t *__restrict__ hs_lo, uint8_t *__restrict__ he_hi, uint8_t *__restrict__ he_lo, int T, int H, int I,
    int E, size_t ewb, size_t esb)
{
    __shared__ ActSeg seg[2];
    const MetaIdx mi{E};
    const int tiles = I / (8 * W * NA);
    const int n_items = meta[mi.n_mfma_chunks()] * tiles;
    const int4 *recs = reinterpret_cast<const int4 *>(meta + mi.chunk_rec());
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ActRsrc X = act_rsrc(xs_hi, xs_lo, xe_hi, xe_lo, (uint32_t)T, (uint32_t)H);
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int4 rec = recs[item / tiles];  // {expert, first slot, tokens, -}
        const int i0 = (item % tiles) * 8 * W * NA;
        const uint8_t *we = ew + (size_t)rec.x * ewb;
        const uint8_t *se = es + (size_t)rec.x * esb;
        if (rec.z > 16)
            w13_item_lds<FMT, 2, W, NA, PK>(we, se, H, I, i0, rec.y, rec.z, tok_of, X, hs_hi, hs_lo, he_hi, he_lo,
                                            seg, wave, lane, tid);
        else
            w13_item_lds<FMT, 1, W, NA, PK>(we, se, H, I, i0, rec.y, rec.z, tok_of, X, hs_hi, hs_lo, he_hi, he_lo,
                                            seg, wave, lane, tid);
    }
}

// down: item = (chunk, rows [n0, n0+16*NA*W)) for W waves; wave w streams rows
// n0 + 16*(NA*w + a), a < NA.
template <int FMT, int NT, int W, int NA, bool PK>
__device__ inline void w2_item_lds(const uint8_t *__restrict__ we2, const uint8_t *__restrict__ se, int H, int I,
                                   int n0, int slot0, int mc, const ActRsrc &Hs, float *__restrict__ obuf,
                                   ActSeg (&seg)[2], int wave, int lane, int tid)
{
    const int r = lane & 15, g = lane >> 4;
    const size_t rowb = FMT == 0 ? (size_t)I : (size_t)I / 2;
    const uint8_t *arow[NA];
    const uint8_t *erow[NA];
    const float *sblk[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        const int row0 = n0 + 16 * (NA * wave + a);
        arow[a] = wlane<PK>(we2, row0, rowb, lane);
        erow[a] = se + (size_t)2 * I * (H / 32) + (size_t)(row0 + (PK ? 0 : r)) * (I / 32);
        sblk[a] = (const float *)se + (size_t)2 * (I / 128) * (H / 128) + (size_t)(row0 / 128) * (I / 128);
    }
    Stager<NT, W> st;
    st.init(nullptr, slot0, mc, I, tid);
    f32x4 acc[NA][NT];
    stream_tile_lds<FMT, NT, W, NA, PK>(acc, arow, erow, sblk, I / 128, Hs, st, seg, lane, tid);
#pragma unroll
    for (int j = 0; j < NT; ++j)
        if (16 * j + r < mc) {
            const size_t slot = (size_t)slot0 + 16 * j + r;
#pragma unroll
            for (int a = 0; a < NA; ++a)
                *reinterpret_cast<f32x4 *>(obuf + slot * H + n0 + 16 * (NA * wave + a) + 4 * g) = acc[a][j];
        }
}

template <int FMT, int W, int NA, bool PK>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W == 8 ? 4 : 1))) void w2_mfma_lds_kernel(
    const uint8_t *__restrict__ ew, const uint8_t *__restrict__ es, const int32_t *__restrict__ meta,
    const uint8_t *__restrict__ hs_hi, const uint8_t *__restrict__ hs_lo, const uint8_t *__restrict__ he_hi,
    const uint8_t *__restrict__ he_lo, float *__restrict__ obuf, int P, int H, int I, int E, size_t ewb, size_t esb)
{
    __shared__ ActSeg seg[2];
    const MetaIdx mi{E};
    const int tiles = H / (16 * W * NA);
    const int n_items = meta[mi.n_mfma_chunks()] * tiles;
    const int4 *recs = reinterpret_cast<const int4 *>(meta + mi.chunk_rec());
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t w2off = FMT == 0 ? (size_t)2 * I * H : (size_t)I * H;
    const ActRsrc Hs = act_rsrc(hs_hi, hs_lo, he_hi, he_lo, (uint32_t)P, (uint32_t)I);
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int4 rec = recs[item / tiles];
        const int n0 = (item % tiles) * 16 * W * NA;
        const uint8_t *we2 = ew + (size_t)rec.x * ewb + w2off;
        const uint8_t *se = es + (size_t)rec.x * esb;
        if (rec.z > 16)
            w2_item_lds<FMT, 2, W, NA, PK>(we2, se, H, I, n0, rec.y, rec.z, Hs, obuf, seg, wave, lane, tid);
        else
            w2_item_lds<FMT, 1, W, NA, PK>(we2, se, H, I, n0, rec.y, rec.z, Hs, obuf, seg, wave, lane, tid);
    }
}

// ------------------------------------------------------------------ wide chunks
//
// Large batches of FP8 layers: chunks of up to 128 tokens (kWideChunk), so that an
// expert's weights stream once for nearly all of its tokens; with 32-token chunks a batch
// of 50 tokens per expert streamed them twice.  HBM bounds these kernels.  One persistent
// workgroup of eight waves per CU; each wave streams two 16-row tiles (the gate and up
// rows of the same 16 rows, or two down tiles) against up to eight staged token tiles, so
// every activation fragment read from LDS feeds two tiles: at 128 tokens the fragment
// reads of a K block take 2,048 LDS cycles per CU, under the 2,900 that its 32 KB of
// weights take at the HBM rate.  Items come from a device counter (`ticket`, zeroed by the
// step's routing), drawn one item ahead, and the weight ring runs on into the next item,
// so only the first activations of an item are waited for.
//
// Measured, us (gate/up and down by the stage events, 32-token chunks -> these): the
// 480B-shaped layer with biased routing at T=1000 1,845 -> 1,038 and 1,013 -> 564 (6.4 GB
// and 3.1 GB fetched by the counters, with the writes 6.2 and 5.9 TB/s, where a read-only
// stream reaches 6.8); uniform routing T=600 1,179 -> 882 and
// 672 -> 498.  At T=600 the same kernel without its activation staging takes 810 and 454,
// and without MFMAs 867 and 491: what is left is the staging and, in the down projection,
// its shorter items.  Four-wave workgroups (two per CU) lost, 934 -> 1,287 at T=600: they
// stage twice the activations per weight byte.  Items of one expert kept on one XCD lost
// too (T=1000: down 564 -> 617).

constexpr int kWideW = 8;   // waves per workgroup
constexpr int kWideArea = 32 * kWideW;  // token rows x K blocks of a segment
constexpr int kWideNA = 2;  // weight tiles per wave
constexpr int kWideGrid = 256;  // persistent workgroups: one per CU

// A staged segment: K blocks x token rows = kWideArea,
// as [hi, lo][token][16-byte pieces, swizzled] codes and [hi, lo][token][E8M0] exponents.
struct alignas(16) WideSeg {
    uint8_t code[2][kWideArea * 128];
    uint8_t ex[2][kWideArea * 4];
};

// K blocks per segment for NT token tiles.
template <int NT>
constexpr int kWideSegK = NT * 16 * 4 <= kWideArea ? 4 : 2;

// Place of 16-byte piece p of token row t: the token XORed into the piece index so that
// the 16 rows of a fragment read fall on 16 distinct bank groups.
template <int SEGK>
__device__ inline int wide_place(int p, int t)
{
    return t * (SEGK * 128) + ((p & ~15) | ((p ^ t) & 15)) * 16;
}

// One thread's share of staging a segment: a 16-byte piece of NT*SEGK/4 token rows in both
// codes, and one 4-byte word of exponents (term tid/kWideArea).  Tokens past the chunk read out
// of range (zeros, no memory request).  A segment that runs past K stages bytes no block
// reads.
template <int NT>
struct WideStager {
    static constexpr int SEGK = kWideSegK<NT>, kTok = kWideArea / SEGK;
    static constexpr int kPieces = SEGK * 8;               // 16-byte pieces of a token row
    static constexpr int kRows = 64 * kWideW / kPieces;    // token rows per pass
    static constexpr int Q = 16 * NT / kRows;
    static_assert(16 * NT <= kTok && 16 * NT % kRows == 0, "a segment holds the tiles, in whole passes");
    static_assert(kRows % 16 == 0, "rows kRows apart have the same swizzle");
    uint32_t voff[Q], eoff;
    int tid, so;
    u32x4v code[2][Q];
    uint32_t ex;

    __device__ void init(const int32_t *__restrict__ row_of, int slot0, int mc, int K, int tid_)
    {
        tid = tid_;
        const int p = tid & (kPieces - 1), t0 = tid / kPieces;
        so = wide_place<SEGK>(p, t0);
        auto row = [&](int t) { return t < mc ? (uint32_t)(row_of ? row_of[slot0 + t] : slot0 + t) : 0u; };
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int t = kRows * q + t0;
            voff[q] = t < mc ? row(t) * (uint32_t)K + 16u * p : kOutOfRange;
        }
        const int te = (tid / SEGK) & (kTok - 1);
        eoff = te < mc ? row(te) * (uint32_t)(K / 32) + 4u * (tid & (SEGK - 1)) : kOutOfRange;
    }
    __device__ void load(const ActRsrc &B, int sg)
    {
        const uint32_t d = (uint32_t)sg * (SEGK * 128), de = (uint32_t)sg * (SEGK * 4);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            code[0][q] = __builtin_amdgcn_raw_buffer_load_b128(B.hi, voff[q] + d, 0, 0);
            code[1][q] = __builtin_amdgcn_raw_buffer_load_b128(B.lo, voff[q] + d, 0, 0);
        }
        ex = __builtin_amdgcn_raw_buffer_load_b32(__builtin_amdgcn_readfirstlane(tid) < kWideArea ? B.ehi : B.elo, eoff + de,
                                                  0, 0);  // the term is uniform over a wave
    }
    __device__ void store(WideSeg &S) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < Q; ++q)
                *reinterpret_cast<u32x4v *>(&S.code[h][0] + so + kRows * q * (SEGK * 128)) = code[h][q];
        reinterpret_cast<uint32_t *>(&S.ex[0][0])[tid] = ex;
    }
};

// A value that no kernel writes, at an address that is the same for the whole wave: a
// scalar load.  As a vector load (the compiler cannot prove either once pointers pass
// from item to item) the block scales made every fourth block wait for all loads in
// flight.
__device__ inline float wide_const(const float *p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return *(const float __attribute__((address_space(4))) *)(((uint64_t)hi << 32) | lo);
}

// Where a wave's two weight tiles of one item lie: the pointers of wlane and the block
// scales of its rows.
struct WideTiles {
    const uint8_t *arow[kWideNA];
    const float *sblk[kWideNA];
};

// The weight ring of a wave, carried from one item to the next.
struct WideRing {
    i32x8 A[4][kWideNA];
};

template <bool PK>
__device__ inline void wide_load(WideRing &R, int slot, const WideTiles &W, int kb, int g)
{
#pragma unroll
    for (int a = 0; a < kWideNA; ++a) R.A[slot][a] = wfrag<0, PK>(W.arow[a], kb, g);
}

// An item's first three blocks into ring slots 0..2.
template <bool PK>
__device__ inline void wide_fill(WideRing &R, const WideTiles &W, int KB, int lane)
{
#pragma unroll
    for (int u = 0; u < 3; ++u) wide_load<PK>(R, u, W, min(u, KB - 1), lane >> 4);
}

// Streams this wave's two weight tiles W over KB K blocks against NT staged token tiles;
// acc[a][j] as in stream_tiles.  All waves of the workgroup call it together; it
// synchronises them once per staged segment.  On entry the ring holds the item's first
// three blocks, on return those of the next item (tiles N), so the weight stream does not
// stop between items.  On return no wave reads `seg` any more.
template <int NT, bool PK>
__device__ inline void stream_wide(f32x4 (&acc)[kWideNA][NT], WideRing &R, const WideTiles &W, const WideTiles &N,
                                   int KB, const ActRsrc &B, WideStager<NT> &st, WideSeg (&seg)[2], int lane)
{
    constexpr int NA = kWideNA, SEGK = kWideSegK<NT>;
    const int r = lane & 15, g = lane >> 4;
    const int nseg = (KB + SEGK - 1) / SEGK;
    // block kb of this item, or of the next one past the end (reached only when KB is a
    // multiple of four, so the ring slots of the two items agree)
    auto loadA = [&](int slot, int kb) {
        const bool in = kb < KB;
        WideTiles S;
#pragma unroll
        for (int a = 0; a < NA; ++a) S.arow[a] = in ? W.arow[a] : N.arow[a];
        wide_load<PK>(R, slot, S, in ? kb : kb - KB, g);
    };
    // Token tile j+1's fragments are read from LDS while tile j is multiplied; the
    // scheduling barriers keep the compiler from hoisting all NT tiles' reads at once,
    // which does not fit the register file.
    struct BFrag {
        i32x8 h, l;
        int eh, el;
    };
    // LDS offsets of this lane's pieces of token row r (tile j adds 16 rows, the low term
    // half of the codes, a second pair of blocks 256 bytes), written so that only these
    // few registers hold addresses
    constexpr int kRow = SEGK * 128;
    int boff[2][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int q = 0; q < 2; ++q) boff[kk][q] = wide_place<SEGK>((8 * kk + 4 * q + g) & (8 * SEGK - 1), r);
    const int xoff = r * (SEGK * 4) + g;
    auto readB = [&](BFrag &f, const WideSeg &S, int kk, int j) {
        const uint8_t *c = &S.code[0][0] + 16 * j * kRow + (kk >> 1) * 256;
        const uint8_t *x = &S.ex[0][0] + xoff + 16 * j * (SEGK * 4) + 4 * kk;
        const u32x4v h0 = *reinterpret_cast<const u32x4v *>(c + boff[kk & 1][0]);
        const u32x4v h1 = *reinterpret_cast<const u32x4v *>(c + boff[kk & 1][1]);
        const u32x4v l0 = *reinterpret_cast<const u32x4v *>(c + boff[kk & 1][0] + sizeof(S.code[0]));
        const u32x4v l1 = *reinterpret_cast<const u32x4v *>(c + boff[kk & 1][1] + sizeof(S.code[0]));
        f.h = (i32x8){(int)h0.x, (int)h0.y, (int)h0.z, (int)h0.w, (int)h1.x, (int)h1.y, (int)h1.z, (int)h1.w};
        f.l = (i32x8){(int)l0.x, (int)l0.y, (int)l0.z, (int)l0.w, (int)l1.x, (int)l1.y, (int)l1.z, (int)l1.w};
        f.eh = x[0];
        f.el = x[sizeof(S.ex[0])];
    };
    auto compute = [&](int slot, const WideSeg &S, int kk, int kb) {
        float sc[NA];
#pragma unroll
        for (int a = 0; a < NA; ++a) sc[a] = wide_const(W.sblk[a] + kb);
        BFrag f[2];
        readB(f[0], S, kk, 0);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if (j + 1 < NT) readB(f[(j + 1) & 1], S, kk, j + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int a = 0; a < NA; ++a)
                mma2<0>(acc[a][j], R.A[slot][a], 127, sc[a], f[j & 1].h, f[j & 1].eh, f[j & 1].l, f[j & 1].el);
        }
    };
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[a][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    st.load(B, 0);
    st.store(seg[0]);
    st.load(B, min(1, nseg - 1));
    sync_lds();
    int kb = 0;
    for (; kb + 4 <= KB; kb += 4) {  // four blocks per iteration: 4 / SEGK segments
        const int sg = kb / SEGK;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            loadA((u + 3) & 3, KB % 4 ? min(kb + u + 3, KB - 1) : kb + u + 3);
            __builtin_amdgcn_sched_barrier(0);
            const int b = SEGK == 4 ? sg & 1 : (u / SEGK) & 1;  // the block's buffer
            compute(u, seg[b], u % SEGK, kb + u);
            if ((u + 1) % SEGK == 0) {
                st.store(seg[b ^ 1]);
                st.load(B, min(sg + 2 + u / SEGK, nseg - 1));
                sync_lds();
            }
        }
    }
    // Fewer than four blocks remain, in ring slots 0..2; their first segment is staged, the
    // next one sits in the stager's registers.
    if (kb < KB) {
        const int sg = kb / SEGK;
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (kb + u < KB) {
                const int b = SEGK == 4 ? sg & 1 : (u / SEGK) & 1;
                if (u && u % SEGK == 0) {
                    st.store(seg[b]);
                    st.load(B, min(sg + 1 + u / SEGK, nseg - 1));
                    sync_lds();
                }
                compute(u, seg[b], u % SEGK, kb + u);
            }
        }
        sync_lds();
        wide_fill<PK>(R, N, KB, lane);
    }
}

// gate/up: item = (chunk, 16 * kWideW rows of the intermediate dimension); wave w streams the
// gate and the up rows i0 + 16w .. +16, so silu(g)*u forms in its registers; waves 2q and
// 2q+1 share the 32-row group of h's split and exchange their column maxima through LDS
// (over seg[1], which the next item first writes after its first barrier).
template <bool PK>
__device__ inline void w13_wide_tiles(WideTiles &W, const uint8_t *__restrict__ we, const uint8_t *__restrict__ se,
                                      int H, int I, int r0, int lane)
{
    const size_t rowb = (size_t)H;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int row0 = a * I + r0;
        W.arow[a] = wlane<PK>(we, row0, rowb, lane);
        W.sblk[a] = (const float *)se + (size_t)(row0 / 128) * (H / 128);
    }
}

template <int NT, bool PK>
__device__ inline void w13_item_wide(WideRing &R, const WideTiles &W, const WideTiles &N, int H, int I, int r0,
                                     int slot0, int mc, const int *tok, const ActRsrc &X, uint8_t *__restrict__ hs_hi,
                                     uint8_t *__restrict__ hs_lo, uint8_t *__restrict__ he_hi,
                                     uint8_t *__restrict__ he_lo, WideSeg (&seg)[2], int wave, int lane, int tid)
{
    const int r = lane & 15, g = lane >> 4;
    WideStager<NT> st;
    st.init(tok, 0, mc, H, tid);
    f32x4 acc[2][NT];
    stream_wide<NT, PK>(acc, R, W, N, H / 128, X, st, seg, lane);
    float *s_am = reinterpret_cast<float *>(&seg[1].code[0][0]), *s_rm = s_am + kWideW * NT * 16;
    static_assert(sizeof(float) * 2 * kWideW * 8 * 16 <= sizeof(seg[1].code), "exchange buffers");
    auto ix = [&](int w, int j) { return (w * NT + j) * 16 + r; };
    float h[NT][4], res[NT][4], am[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float gi = acc[0][j][i];
            h[j][i] = gi / (1.0f + expf(-gi)) * acc[1][j][i];
        }
        float m = amax_of(h[j]);
        m = fmaxf(m, __shfl_xor(m, 16));
        am[j] = fmaxf(m, __shfl_xor(m, 32));
        if (g == 0) s_am[ix(wave, j)] = am[j];
    }
    sync_lds();
    int ch[NT];
    uint32_t qh[NT][1], ql[1];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        ch[j] = exp_for_group(fmaxf(am[j], s_am[ix(wave ^ 1, j)]));
        split_hi(h[j], ch[j], qh[j], res[j]);
        float m = amax_of(res[j]);
        m = fmaxf(m, __shfl_xor(m, 16));
        am[j] = fmaxf(m, __shfl_xor(m, 32));
        if (g == 0) s_rm[ix(wave, j)] = am[j];
    }
    sync_lds();
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int cl = exp_for_group(fmaxf(am[j], s_rm[ix(wave ^ 1, j)]));
        split_lo(res[j], cl, ql);
        if (16 * j + r < mc) {
            const size_t slot = (size_t)slot0 + 16 * j + r;
            *reinterpret_cast<uint32_t *>(hs_hi + slot * I + r0 + 4 * g) = qh[j][0];
            *reinterpret_cast<uint32_t *>(hs_lo + slot * I + r0 + 4 * g) = ql[0];
            if ((wave & 1) == 0 && g == 0) {
                he_hi[slot * (I / 32) + r0 / 32] = (uint8_t)ch[j];
                he_lo[slot * (I / 32) + r0 / 32] = (uint8_t)cl;
            }
        }
    }
}

// Calls go(integral_constant NT) with the token tiles of a chunk of mc tokens.
template <class F>
__device__ inline void wide_tiles_of(int mc, F go)
{
    if (mc > 96) go(std::integral_constant<int, 8>{});
    else if (mc > 64) go(std::integral_constant<int, 6>{});
    else if (mc > 32) go(std::integral_constant<int, 4>{});
    else go(std::integral_constant<int, 2>{});
}

template <bool PK>
__global__ __launch_bounds__(64 * kWideW) __attribute__((amdgpu_waves_per_eu(2))) void w13_wide_kernel(
    const uint8_t *__restrict__ ew, const uint8_t *__restrict__ es, const int32_t *__restrict__ meta,
    const int32_t *__restrict__ tok_of, const uint8_t *__restrict__ xs_hi, const uint8_t *__restrict__ xs_lo,
    const uint8_t *__restrict__ xe_hi, const uint8_t *__restrict__ xe_lo, uint8_t *__restrict__ hs_hi,
    uint8_t *__restrict__ hs_lo, uint8_t *__restrict__ he_hi, uint8_t *__restrict__ he_lo, int32_t *ticket, int T,
    int H, int I, int E, size_t ewb, size_t esb)
{
    __shared__ WideSeg seg[2];
    __shared__ int s_tok[2][kWideChunk];  // token rows of this item's chunk and the next one's
    __shared__ int s_next;
    const MetaIdx mi{E};
    const int tiles = I / (16 * kWideW);
    const int4 *recs = reinterpret_cast<const int4 *>(meta + mi.chunk_rec());
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ActRsrc X = act_rsrc(xs_hi, xs_lo, xe_hi, xe_lo, (uint32_t)T, (uint32_t)H);
    auto row0 = [&](int it) { return (it % tiles) * (16 * kWideW) + 16 * wave; };
    const int n_items = meta[mi.n_mfma_chunks()] * tiles;
    int item = blockIdx.x, nxt = item + gridDim.x;
    if (item >= n_items) return;  // uniform over the workgroup
    int4 rec = chunk_record(recs, item / tiles);  // {expert, first slot, tokens, -}
    WideTiles W, N;
    w13_wide_tiles<PK>(W, ew + (size_t)rec.x * ewb, es + (size_t)rec.x * esb, H, I, row0(item), lane);
    WideRing R;
    wide_fill<PK>(R, W, H / 128, lane);
    if (tid < kWideChunk) s_tok[0][tid] = tid < rec.z ? tok_of[rec.y + tid] : 0;
    __syncthreads();
    for (int p = 0;; p ^= 1) {
        const int after = tid == 0 ? atomicAdd(ticket, 1) + 2 * (int)gridDim.x : 0;
        const bool more = nxt < n_items;
        const int ni = more ? nxt : item;  // after the last item: its own blocks again
        const int4 nrec = chunk_record(recs, ni / tiles);
        const int ntok = tid < nrec.z && tid < kWideChunk ? tok_of[nrec.y + tid] : 0;
        w13_wide_tiles<PK>(N, ew + (size_t)nrec.x * ewb, es + (size_t)nrec.x * esb, H, I, row0(ni), lane);
        wide_tiles_of(rec.z, [&](auto nt) {
            w13_item_wide<decltype(nt)::value, PK>(R, W, N, H, I, row0(item), rec.y, rec.z, s_tok[p], X, hs_hi,
                                                        hs_lo, he_hi, he_lo, seg, wave, lane, tid);
        });
        if (!more) return;
        if (tid < kWideChunk) s_tok[p ^ 1][tid] = ntok;
        if (tid == 0) s_next = after;
        sync_lds();
        item = nxt;
        nxt = __builtin_amdgcn_readfirstlane(s_next);
        rec = nrec;
        W = N;
    }
}

// down: item = (chunk, 32 * kWideW output rows); wave w streams rows n0 + 32w .. +32 as two tiles.
template <bool PK>
__device__ inline void w2_wide_tiles(WideTiles &W, const uint8_t *__restrict__ we, const uint8_t *__restrict__ se,
                                     int H, int I, int r0, int lane)
{
    const size_t rowb = (size_t)I;
    const uint8_t *we2 = we + (size_t)2 * I * H;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int row0 = r0 + 16 * a;
        W.arow[a] = wlane<PK>(we2, row0, rowb, lane);
        W.sblk[a] = (const float *)se + (size_t)2 * (I / 128) * (H / 128) + (size_t)(row0 / 128) * (I / 128);
    }
}

template <bool PK>
__global__ __launch_bounds__(64 * kWideW) __attribute__((amdgpu_waves_per_eu(2))) void w2_wide_kernel(
    const uint8_t *__restrict__ ew, const uint8_t *__restrict__ es, const int32_t *__restrict__ meta,
    const uint8_t *__restrict__ hs_hi, const uint8_t *__restrict__ hs_lo, const uint8_t *__restrict__ he_hi,
    const uint8_t *__restrict__ he_lo, float *__restrict__ obuf, int32_t *ticket, int P, int H, int I, int E,
    size_t ewb, size_t esb)
{
    __shared__ WideSeg seg[2];
    __shared__ int s_next;
    const MetaIdx mi{E};
    const int tiles = H / (32 * kWideW);
    const int4 *recs = reinterpret_cast<const int4 *>(meta + mi.chunk_rec());
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ActRsrc Hs = act_rsrc(hs_hi, hs_lo, he_hi, he_lo, (uint32_t)P, (uint32_t)I);
    auto row0 = [&](int it) { return (it % tiles) * (32 * kWideW) + 32 * wave; };
    const int n_items = meta[mi.n_mfma_chunks()] * tiles;
    int item = blockIdx.x, nxt = item + gridDim.x;
    if (item >= n_items) return;  // uniform over the workgroup
    int4 rec = chunk_record(recs, item / tiles);
    WideTiles W, N;
    w2_wide_tiles<PK>(W, ew + (size_t)rec.x * ewb, es + (size_t)rec.x * esb, H, I, row0(item), lane);
    WideRing R;
    wide_fill<PK>(R, W, I / 128, lane);
    for (;;) {
        const int after = tid == 0 ? atomicAdd(ticket, 1) + 2 * (int)gridDim.x : 0;
        const bool more = nxt < n_items;
        const int ni = more ? nxt : item;  // after the last item: its own blocks again
        const int4 nrec = chunk_record(recs, ni / tiles);
        w2_wide_tiles<PK>(N, ew + (size_t)nrec.x * ewb, es + (size_t)nrec.x * esb, H, I, row0(ni), lane);
        wide_tiles_of(rec.z, [&](auto nt) {
            constexpr int NT = decltype(nt)::value;
            WideStager<NT> st;
            st.init(nullptr, rec.y, rec.z, I, tid);
            f32x4 acc[2][NT];
            stream_wide<NT, PK>(acc, R, W, N, I / 128, Hs, st, seg, lane);
#pragma unroll
            for (int j = 0; j < NT; ++j)
                if (16 * j + r < rec.z) {
                    const size_t slot = (size_t)rec.y + 16 * j + r;
#pragma unroll
                    for (int a = 0; a < 2; ++a)
                        *reinterpret_cast<f32x4 *>(obuf + slot * H + row0(item) + 16 * a + 4 * g) = acc[a][j];
                }
        });
        if (!more) return;
        if (tid == 0) s_next = after;
        sync_lds();
        item = nxt;
        nxt = __builtin_amdgcn_readfirstlane(s_next);
        rec = nrec;
        W = N;
    }
}

// ------------------------------------------------------------------ down projection with the combine
//
// Small batches: workgroup i owns output rows 16i .. +16 of every pair of the step, so it
// also combines them and writes y: no expert outputs in memory and no combine launch.  Its
// waves take the passes (up to eight tokens of one expert) in turn, and each wave's stream
// of weights (one 16-row tile per pass) runs through a four-slot ring without a break from
// one pass to the next, where a work item per tile paid a start of its own.  The token
// columns of the matrix instruction hold both terms of the activation split, the high codes
// of the pass's tokens in columns 0..7 and the low ones in 8..15, so a K block is one MFMA
// and one activation fragment; the two halves are added at the end of the pass.  All
// workgroups walk the experts in the same order, and together read each expert's matrix as
// one contiguous piece.
//
// Measured at one token on the 235B-shaped layer: 15.0 -> 13.0 us for the down projection and
// the combine together (of 44.1 us per step); rings of six and eight slots and workgroups of
// four and sixteen waves came out within 1 us.

constexpr int kOwnTok = 8;         // tokens per pass
constexpr int kOwnW = 8;           // waves per workgroup

template <int FMT, bool PK, bool OUTF32>
__global__ __launch_bounds__(64 * kOwnW) __attribute__((amdgpu_waves_per_eu(4))) void w2_own_kernel(
    const uint8_t *__restrict__ ew, const uint8_t *__restrict__ es, const int32_t *__restrict__ meta,
    const int32_t *__restrict__ slot_of, const float *__restrict__ wts, const uint8_t *__restrict__ hs_hi,
    const uint8_t *__restrict__ hs_lo, const uint8_t *__restrict__ he_hi, const uint8_t *__restrict__ he_lo,
    void *__restrict__ y, int T, int k, int H, int I, int E, size_t ewb, size_t esb)
{
    constexpr int W = kOwnW, R = 4;  // waves, ring slots
    extern __shared__ __attribute__((aligned(16))) float own_lds[];
    __shared__ int s_np;
    const int P = T * k;
    const OwnLds S(own_lds, P);
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = blockIdx.x * 16, KB = I / 128;
    const int np = own_passes<kOwnTok, W>(S, &s_np, meta, slot_of, wts, P, E, wave, tid);
    const int mine = np > wave ? (np - wave + W - 1) / W : 0;  // this wave's passes: wave, wave + W, ...

    const uint32_t lo_off = (uint32_t)(hs_lo - hs_hi), elo_off = (uint32_t)(he_lo - he_hi);
    const __amdgpu_buffer_rsrc_t hr = raw_rsrc(hs_hi, lo_off + (uint32_t)P * I);
    const __amdgpu_buffer_rsrc_t er = raw_rsrc(he_hi, elo_off + (uint32_t)P * (I / 32));
    const size_t rowb = FMT == 0 ? (size_t)I : (size_t)I / 2, w2off = FMT == 0 ? (size_t)2 * I * H : (size_t)I * H;
    struct {
        const uint8_t *arow, *erow;
        const float *sblk;
        uint32_t voff, eoff;
        int i, kb;
    } L;  // the pass whose blocks are being loaded
    auto pass = [&](int i) { return (uint32_t)__builtin_amdgcn_readfirstlane(S.pass[wave + W * i]); };
    auto open = [&](int i) {
        const uint32_t ps = pass(i);
        const int e = ps & 1023, mc = (ps >> 10) & 15, slot0 = ps >> 16;
        const uint8_t *we = ew + (size_t)e * ewb + w2off, *se = es + (size_t)e * esb;
        L.arow = wlane<PK>(we, row0, rowb, lane);
        L.erow = se + (size_t)2 * I * (H / 32) + (size_t)(row0 + (PK ? 0 : r)) * (I / 32);
        L.sblk = (const float *)se + (size_t)2 * (I / 128) * (H / 128) + (size_t)(row0 / 128) * (I / 128);
        const uint32_t row = slot0 + (r & 7);
        const bool live = (r & 7) < mc;
        L.voff = live ? (r < 8 ? 0u : lo_off) + row * (uint32_t)I + 16u * g : kOutOfRange;
        L.eoff = live ? (r < 8 ? 0u : elo_off) + row * (uint32_t)(I / 32) : kOutOfRange;
        L.i = i;
        L.kb = 0;
    };
    i32x8 A[R], Bf[R];
    int EA[R];
    uint32_t X[R];
    float sc[R];
    // the next block of the wave's stream into a ring slot (past its end: the last block again)
    auto load = [&](int slot) {
        A[slot] = wfrag<FMT, PK>(L.arow, L.kb, g);
        Bf[slot] = frag_buf(hr, L.voff, L.kb * 128);
        X[slot] = __builtin_amdgcn_raw_buffer_load_b32(er, L.eoff, L.kb * 4, 0);
        if constexpr (FMT == 0) {
            EA[slot] = 127;
            sc[slot] = wide_const(L.sblk + L.kb);
        } else {
            EA[slot] = PK ? e8m0_packed(L.erow, L.kb, KB, lane) : L.erow[L.kb * 4 + g];
        }
        if (L.kb + 1 < KB)
            ++L.kb;
        else if (L.i + 1 < mine)
            open(L.i + 1);
    };
    if (mine) {
        open(0);
#pragma unroll
        for (int u = 0; u < R - 1; ++u) {
            load(u);
            __builtin_amdgcn_sched_barrier(0);
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        int ci = 0, ckb = 0;
        const int nb = mine * KB;
        for (int n = 0; n < nb; n += R) {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                load((u + R - 1) % R);
                __builtin_amdgcn_sched_barrier(0);
                if (n + u < nb) {
                    const int eb = (int)__builtin_amdgcn_ubfe(X[u], 8 * g, 8);
                    if constexpr (FMT == 0) {
                        f32x4 t = {0.f, 0.f, 0.f, 0.f};
                        t = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A[u], Bf[u], t, 0, 0, 0, 127, 0, eb);
                        acc += sc[u] * t;
                    } else {
                        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A[u], Bf[u], acc, 4, 0, 0, EA[u], 0, eb);
                    }
                    if (++ckb == KB) {  // the pass is done: lane (r, g) has rows 4g.. of column r
                        const uint32_t ps = pass(ci);
                        f32x4 v;
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[c] = acc[c] + __shfl_xor(acc[c], 8);
                        if (r < (int)((ps >> 10) & 15)) S.o[((ps >> 16) + r) * 4 + g] = v;
                        acc = (f32x4){0.f, 0.f, 0.f, 0.f};
                        ckb = 0;
                        ++ci;
                    }
                }
            }
        }
    }
    __syncthreads();
    own_combine<W, OUTF32>(S, y, T, k, H, row0, tid);
}

// Waves per workgroup of the staged kernels.  FP8 weights stream at 4 waves and two
// workgroups per CU: eight waves per CU hold the HBM stream at its best, and more
// waves per CU slowed it (the 235B- and 480B-shaped layers lost 9-18%).  E2M1
// weights carry half the bytes per activation fragment, so the activation staging, not
// HBM, bounds them: 4 waves with several tiles each (kStagedTiles), and 8 waves for the
// three-tile gate/up (kThreeTileWaves), which stage each segment once for more rows.
// Eight-wave workgroups held to 128 VGPRs to run two per CU lost (the MXFP4 layer at
// T=256, one tile per wave: 570k against 604k tokens/s).
template <int FMT>
constexpr int kStagedWaves = 4;
// Weight tiles per wave of the staged kernels (NA).  E2M1 tiles: four on packed weights
// (each staged activation fragment then feeds four tiles; MXFP4 Zipf layer at T=256
// 1,035k -> 1,094k tokens/s), two on row-major ones (four need more than the 256
// registers two waves per SIMD allow there).
template <int FMT, bool PK>
constexpr int kStagedTiles = FMT == 0 ? 1 : (PK ? 4 : 2);
// Packed E2M1 gate/up takes three tiles per wave in eight-wave workgroups (one per CU,
// up to 256 VGPRs) where I is a multiple of 1536: an item then covers 192 rows, a chunk
// a multiple of 8 items, and since consecutive workgroups go round-robin over the 8
// XCDs, tile q of every chunk of one expert runs on one XCD, at about the same time, and
// its later chunks find the weights in that XCD's L2.  At four tiles (12 items per
// chunk at I = 1536) consecutive chunks land 4 XCDs apart.  MXFP4 Zipf layer at T=256:
// three tiles in four-wave workgroups (96 rows, 16 items per chunk) took gate/up fetch
// 760 -> 629 MB and 126.0 -> 120.0 us; eight waves, which stage each activation
// segment once for twice the rows, 120.0 -> 116.0 us (1,124k -> 1,140k tokens/s).
// Padding 12 items to a stride of 16 instead put twice the work on half the XCDs (126 ->
// 138 us).  The down projection stays at four waves (eight: 69.5 -> 72.4 us).
constexpr int kThreeTileWaves = 8;  // waves per workgroup of the three-tile gate/up
template <int FMT, bool PK>
constexpr bool w13_three_tiles(const Layer &L)
{
    return FMT == 1 && PK && L.I % (8 * kThreeTileWaves * 3 * 8) == 0;
}

// Workgroups for `items_per_chunk` items per chunk record, `per_block` items per workgroup.
int mfma_grid(const Layer &L, int T, int k, int items_per_chunk, int per_block)
{
    const long pairs = (long)T * k;
    const long recs = pairs < L.E ? pairs : L.E;
    const long chunks = recs + (pairs + kMfmaChunk - 1) / kMfmaChunk;  // >= number of chunk records
    const long blocks = (chunks * items_per_chunk + per_block - 1) / per_block;
    return blocks < 1 ? 1 : (blocks > 65535 ? 65535 : (int)blocks);
}

template <int FMT, bool PK, int NA, int W = kStagedWaves<FMT>>
hipError_t launch_w13_lds(const Layer &L, const uint8_t *ew, const uint8_t *es, int T, int k, const int32_t *meta,
                          const int32_t *tok_of, const Workspace &ws, hipStream_t st)
{
    dim3 grid(mfma_grid(L, T, k, L.I / (8 * W * NA), 1)), block(64 * W);
    w13_mfma_lds_kernel<FMT, W, NA, PK><<<grid, block, 0, st>>>(ew, es, meta, tok_of, ws.xs_hi, ws.xs_lo, ws.xe_hi, ws.xe_lo,
                                                        ws.hs_hi, ws.hs_lo, ws.he_hi, ws.he_lo, T, L.H, L.I, L.E,
                                                        L.expert_w_bytes, L.expert_s_bytes);
    return hipGetLastError();
}

template <int FMT, bool PK>
hipError_t launch_w2_lds(const Layer &L, const uint8_t *ew, const uint8_t *es, int T, int k, const int32_t *meta,
                         const Workspace &ws, hipStream_t st)
{
    constexpr int W = kStagedWaves<FMT>, NA = kStagedTiles<FMT, PK>;
    dim3 grid(mfma_grid(L, T, k, L.H / (16 * W * NA), 1)), block(64 * W);
    w2_mfma_lds_kernel<FMT, W, NA, PK><<<grid, block, 0, st>>>(ew, es, meta, ws.hs_hi, ws.hs_lo, ws.he_hi, ws.he_lo, ws.o,
                                                       T * k, L.H, L.I, L.E, L.expert_w_bytes, L.expert_s_bytes);
    return hipGetLastError();
}

template <int FMT, bool PK>
hipError_t w13_launch(const Layer &L, const uint8_t *ew, const uint8_t *es, int T, int k, const int32_t *meta,
                      const int32_t *tok_of, const Workspace &ws, hipStream_t st)
{
    if (FMT == 0 && chunk_tokens(L, T, k) == kWideChunk) {
        w13_wide_kernel<PK><<<kWideGrid, 64 * kWideW, 0, st>>>(
            ew, es, meta, tok_of, ws.xs_hi, ws.xs_lo, ws.xe_hi, ws.xe_lo, ws.hs_hi, ws.hs_lo, ws.he_hi, ws.he_lo,
            ws.tickets, T, L.H, L.I, L.E, L.expert_w_bytes, L.expert_s_bytes);
        return hipGetLastError();
    }
    if ((L.H / 128) % 4 == 0) {
        if constexpr (FMT == 1 && PK)
            if (w13_three_tiles<FMT, PK>(L))
                return launch_w13_lds<FMT, PK, 3, kThreeTileWaves>(L, ew, es, T, k, meta, tok_of, ws, st);
        return launch_w13_lds<FMT, PK, kStagedTiles<FMT, PK>>(L, ew, es, T, k, meta, tok_of, ws, st);
    }
    dim3 grid(mfma_grid(L, T, k, L.I / 64, 1)), block(256);
    w13_mfma_kernel<FMT, PK><<<grid, block, 0, st>>>(ew, es, meta, tok_of, ws.xs_hi, ws.xs_lo, ws.xe_hi, ws.xe_lo,
                                                     ws.hs_hi, ws.hs_lo, ws.he_hi, ws.he_lo, T, L.H, L.I, L.E,
                                                     L.expert_w_bytes, L.expert_s_bytes);
    return hipGetLastError();
}

template <int FMT, bool PK>
hipError_t w2_launch(const Layer &L, const uint8_t *ew, const uint8_t *es, int T, int k, const int32_t *meta,
                     const Workspace &ws, hipStream_t st)
{
    if (FMT == 0 && chunk_tokens(L, T, k) == kWideChunk) {
        w2_wide_kernel<PK><<<kWideGrid, 64 * kWideW, 0, st>>>(
            ew, es, meta, ws.hs_hi, ws.hs_lo, ws.he_hi, ws.he_lo, ws.o, ws.tickets + 1, T * k, L.H, L.I, L.E,
            L.expert_w_bytes, L.expert_s_bytes);
        return hipGetLastError();
    }
    // Staging pays a per-item prologue; with fewer than 16 K blocks per row (I < 2048)
    // the two-tile kernel measured faster for FP8 weights (235B-shaped layer: 155
    // against 160 us at T=64).  E2M1 weights carry half the bytes per activation
    // fragment, so they always take the staged kernel.
    if ((L.I / 128) % 4 == 0 && (L.I / 128 >= 16 || FMT == 1)) return launch_w2_lds<FMT, PK>(L, ew, es, T, k, meta, ws, st);
    dim3 grid(mfma_grid(L, T, k, L.H / 32, 4)), block(256);
    w2_mfma_kernel<FMT, PK><<<grid, block, 0, st>>>(ew, es, meta, ws.hs_hi, ws.hs_lo, ws.he_hi, ws.he_lo, ws.o, T * k,
                                                    L.H, L.I, L.E, L.expert_w_bytes, L.expert_s_bytes);
    return hipGetLastError();
}

// Row-major expert weights -> packed 16-row tiles (the layout above), one thread per
// 16-byte piece of the destination.  Per expert: the [2I][K = H] gate/up rows, then
// the [H][K = I] down rows; FP8 one byte per input, E2M1 half a byte.  fmt 0 FP8
// (128-input blocks), 1 MXFP4 (128-input blocks), 2 NVFP4 (256-input blocks of the
// bf16 kernels: lane l's bytes [32g, 32g+16) at 16l, [32g+16, 32g+32) at 1024 + 16l).
__global__ void pack_kernel(const uint8_t *__restrict__ src, uint8_t *__restrict__ dst, int64_t n_pieces, int H,
                            int I, int fmt, int64_t expert_bytes)
{
    const bool fp4 = fmt != 0;
    const int blk = fmt == 1 ? 1024 : 2048;     // bytes of a (16-row tile, K block) piece
    const int kbb = fmt == 1 ? 64 : 128;        // bytes of a row per K block
    const int64_t w13 = (int64_t)2 * I * H / (fp4 ? 2 : 1);  // gate/up bytes of an expert
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_pieces; p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t off = p * 16;                     // destination byte
        const int64_t e = off / expert_bytes, eo = off % expert_bytes;
        const bool down = eo >= w13;
        const int64_t mo = down ? eo - w13 : eo;        // byte within the matrix
        const int64_t rowb = (down ? I : H) / (fp4 ? 2 : 1);
        const int64_t tile = mo / (16 * rowb), to = mo % (16 * rowb);
        const int64_t kb = to / blk;
        const int q = (int)(to % blk) / 16;             // piece within the block
        const int half = fmt == 1 ? 0 : q / 64, l = q % 64;  // 2 KB pieces: two halves of 1 KB
        const int r = l & 15, g = l >> 4;
        const int lb = fmt == 2 ? 32 * g + 16 * half : 16 * g + 64 * half;  // byte within the row's block
        const int64_t so = e * expert_bytes + (down ? w13 : 0) + (tile * 16 + r) * rowb + kb * kbb + lb;
        *reinterpret_cast<uint4 *>(dst + off) = *reinterpret_cast<const uint4 *>(src + so);
    }
}

// MXFP4 E8M0 scales, row-major -> packed 16-row tiles (the layout above): per expert the
// [2I][H/32] gate/up scales, then the [H][I/32] down scales.  One thread per byte of the
// destination.
__global__ void pack_e8m0_kernel(const uint8_t *__restrict__ src, uint8_t *__restrict__ dst, int64_t n_bytes, int H,
                                 int I, int64_t expert_bytes)
{
    const int64_t w13 = (int64_t)2 * I * (H / 32);
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_bytes; p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = p / expert_bytes, eo = p % expert_bytes;
        const bool down = eo >= w13;
        const int64_t mo = down ? eo - w13 : eo;
        const int K = down ? I : H, KB = K / 128;
        const int64_t rowb = K / 32;
        const int64_t tile = mo / (16 * rowb);
        const int o = (int)(mo % (16 * rowb));
        const int nfull = KB / 4;
        int q, rem, oo;
        if (o < 256 * nfull) {
            q = o / 256, rem = 4, oo = o % 256;
        } else {
            q = nfull, rem = KB % 4, oo = o - 256 * nfull;
        }
        const int l = oo / rem, kb = 4 * q + oo % rem, r = l & 15, g = l >> 4;
        dst[p] = src[e * expert_bytes + (down ? w13 : 0) + (tile * 16 + r) * rowb + kb * 4 + g];
    }
}

// NVFP4 E4M3 scales, row-major -> packed 16-row tiles: per matrix [rows][K/16] bytes
// after each expert's 16 bytes of matrix scales.  Per (16-row tile, 256-input block) one
// 256-byte piece, lane l's 4 bytes (scales [4g, 4g+4) of row l%16) at 4l; where the
// matrix's block count K/256 is a multiple of four, per (16-row tile, group of four
// blocks) one 1 KB piece instead, lane l's 16 bytes (its 4 bytes of each block of the
// group, block by block) at 16l.  One thread per 4-byte word of the destination.
__global__ void pack_scales_kernel(const uint8_t *__restrict__ src, uint8_t *__restrict__ dst, int64_t n_words, int H,
                                   int I, int64_t expert_bytes)
{
    const int64_t w13 = (int64_t)2 * I * (H / 16);  // gate/up scale bytes of an expert
    const int64_t body = w13 + (int64_t)H * (I / 16);
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_words; p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t off = p * 4;                       // byte within the experts' scale bodies
        const int64_t e = off / body, eo = off % body;
        const bool down = eo >= w13;
        const int64_t mo = down ? eo - w13 : eo;
        const int K = down ? I : H;
        const int64_t rowb = K / 16;                     // scale bytes per row
        const int64_t tile = mo / (16 * rowb);
        const int w = (int)(mo % (16 * rowb)) / 4;       // word within the tile's scales
        int l, kb;
        if ((K / 256) % 4 == 0) {
            l = (w % 256) / 4, kb = 4 * (w / 256) + w % 4;
        } else {
            l = w % 64, kb = w / 64;
        }
        const int r = l & 15, g = l >> 4;
        const int64_t base = e * expert_bytes + 16 + (down ? w13 : 0);
        *reinterpret_cast<uint32_t *>(dst + base + mo) =
            *reinterpret_cast<const uint32_t *>(src + base + (tile * 16 + r) * rowb + kb * 16 + 4 * g);
    }
    // the 16 bytes of matrix scales of each expert, unchanged
    const int64_t n_e = n_words * 4 / body;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_e * 4; p += (int64_t)gridDim.x * blockDim.x)
        *reinterpret_cast<uint32_t *>(dst + (p / 4) * expert_bytes + (p % 4) * 4) =
            *reinterpret_cast<const uint32_t *>(src + (p / 4) * expert_bytes + (p % 4) * 4);
}

}  // namespace

// Token rows of a step's chunk records (MFMA experts): 128 for FP8 layers (64 for NVFP4, 32
// for MXFP4) once an expert has enough tokens on average for the weight streams saved to
// outweigh the wide kernels' item starts, which weigh more the shorter the down
// projection's rows (I) are.  Step us, 32-token chunks / wide, at pairs per expert:
//   FP8 packed     I 2560: 6.4 1,240 / 1,253, 12.8 1,338 / 1,279; I 1536: 12 468 / 473, 16
//                  503 / 485, 24 587 / 519; I 1024: 18 119 / 125, 24 142 / 138; I 640: 19
//                  453 / 470, 32 669 / 536; I 384: 32 70 / 85, 80 125 / 119
//   FP8 row-major  I 1536: 8 512 / 580, 16 600 / 608
//   NVFP4 packed   I 2560: 9.6 805 / 831; I 1536: 11.3 303 / 307, 13.1 313 / 312, 16 331 /
//                  317, 62 820 / 604; I 1024: 12 86 / 88, 16 95 / 92; I 512: 16 79 / 86, 32
//                  107 / 101
//   NVFP4 row-major (whose 32-token kernels read 16 bytes of scales per row)  I 1536: 2
//                  312 / 314, 4 357 / 334, 62 1,028 / 664; I 1024: 3 93 / 89; I 512: 8 76 /
//                  81, 16 94 / 94
// A chunk is I / 128 items of the gate/up projection and H / 256 of the down projection, for
// 256 workgroups; where all items are few, the 32-token kernels' many small workgroups fill
// the chip and the weights saved count only from more tokens.  So the wide kernels also need
// pairs * min(I / 128, H / 256) of 7680 (NVFP4 6144 packed, 4608 row-major), and where one
// chunk per expert gives under 1024 items 32 (30, 16) pairs per expert.  Speed against the
// 32-token kernels, mean of uniform and two Zipf-skewed routings, at pairs per expert:
//   FP8 packed     H 4096, 16 experts, I 768: 32 0.78, 64 1.01, 96 1.14; H 1024, 32 experts, I
//                  512: 40 0.84, 64 1.06; 16 experts, I 256: 109 0.7; H 4096, 8 experts, I 4096: 32
//                  0.92, 64 1.21; H 6144, 16 experts, I 2560: 16 0.79, 24 0.87, 32 1.03
//   NVFP4          H 4096, 16 experts, I 768: 32 0.90, 48 0.98, 64 1.03 packed, 24 0.80, 40 1.04
//                  row-major; H 1024, 32 experts, I 512: 40 0.95, 56 1.10 packed, 32 0.92, 48
//                  1.07 row-major; H 6144, 16 experts, I 2560: 24 0.96, 32 1.07 packed, 12 0.89,
//                  24 1.04 row-major
int chunk_tokens(const Layer &L, int T, int k)
{
    const long pairs = (long)T * k, E = L.E;
    const int t13 = L.I / 128, t2 = L.H / 256;
    const long units = pairs * (t13 < t2 ? t13 : t2);
    const bool few = E * (t13 + t2) < 1024, packed = L.wlayout != 0;
    if (L.wfmt == 0 && L.H % (32 * kWideW) == 0)
        return pairs * L.I > (packed ? 20000 : 26000) * E && units >= 7680 && pairs >= (few ? 32 : 0) * E ? kWideChunk
                                                                                                      : kMfmaChunk;
    if (L.wfmt == 2 && L.I % 128 == 0)
        return pairs > (packed ? 13 : 3) * E && pairs * L.I > (packed ? 13000 : 7000) * E &&
                       units >= (packed ? 6144 : 4608) && pairs >= (few ? (packed ? 30 : 16) : 0) * E
                   ? kWideChunk4
                   : kMfmaChunk;
    return kMfmaChunk;
}

hipError_t launch_w13_mfma(const Layer &L, const void *expert_w, const void *scales, int T, int k,
                           const int32_t *meta, const int32_t *tok_of, const Workspace &ws, hipStream_t st)
{
    const uint8_t *ew = (const uint8_t *)expert_w, *es = (const uint8_t *)scales;
    if (L.wfmt == 0)
        return L.wlayout ? w13_launch<0, true>(L, ew, es, T, k, meta, tok_of, ws, st)
                         : w13_launch<0, false>(L, ew, es, T, k, meta, tok_of, ws, st);
    return L.wlayout ? w13_launch<1, true>(L, ew, es, T, k, meta, tok_of, ws, st)
                     : w13_launch<1, false>(L, ew, es, T, k, meta, tok_of, ws, st);
}

hipError_t launch_w2_mfma(const Layer &L, const void *expert_w, const void *scales, int T, int k,
                          const int32_t *meta, const Workspace &ws, hipStream_t st)
{
    const uint8_t *ew = (const uint8_t *)expert_w, *es = (const uint8_t *)scales;
    if (L.wfmt == 0)
        return L.wlayout ? w2_launch<0, true>(L, ew, es, T, k, meta, ws, st)
                         : w2_launch<0, false>(L, ew, es, T, k, meta, ws, st);
    return L.wlayout ? w2_launch<1, true>(L, ew, es, T, k, meta, ws, st)
                     : w2_launch<1, false>(L, ew, es, T, k, meta, ws, st);
}

// The owner kernel saves a launch and the expert outputs' round trip, but a CU streams no
// more than about 24 GB/s through it, so it needs an even share of the rows on most CUs (192
// to 255 workgroups, or a multiple of 256), or so few pairs that launches and latency are the
// cost.  Step us, other kernels / this one: one token, 235B-shaped FP8 44.1 / 42.1, MXFP4 42.1 /
// 40.3, H 2048 28.3 / 26.2, H 1024 23.2 / 21.8, but 384 workgroups on 256 CUs (H 6144) 39.3 /
// 40.4; 24 pairs, H 2048 45.5 / 46.2, H 1024 28.2 / 29.6.
// FP8 weights, up to 8 tokens, one pass per expert: 235B-shaped T=4 106.0 / 104.7, T=8 163 / 159,
// Zipf-skewed T=8 86.9 / 86.0; 192 workgroups (H 3072, I 1280) T=4 51.5 / 48.8, 224 (H 3584, I
// 1024) T=8 93.9 / 90.5, 240 (H 3840, I 1536) T=8 150.0 / 147.1.  Row-major weights only on an
// even share: 192 workgroups T=6 63.2 / 67.0, 240 T=8 skewed 114.4 / 114.9, but 256 (I 2048) 149.5 /
// 143.7; rows above 2048 not: I 2560 on 208 workgroups packed T=6 skewed 60.2 / 62.6, row-major T=8
// 156 / 161, on 256 row-major skewed 113.8 / 119.0.  Above 8 tokens an expert's further passes
// stream its weights again: uniform T=32 343 / 339, but skewed T=12 98.3 / 101, T=16 103 / 108,
// T=64 209 / 234.  MXFP4 T=4 73.0 / 76.2.
// NVFP4 weights, whose conversion a second pass of an expert repeats: up to 12 tokens, where
// skewed routing is about even: 235B-shaped T=8 111.8 / 106.3 and Zipf-skewed 64.5 / 64.0, T=12
// 143.8 / 139.6 and 71.2 / 71.2, T=24 202.0 / 197.0 but skewed 97.5 / 99.0; row-major T=10 169.8 /
// 161.0 and skewed 82.2 / 84.0, T=12 204.8 / 193.2 and 94.2 / 96.3, T=24 skewed 120 / 130 (with all
// tokens on the same few experts it loses from T=6 row-major, 46.4 / 48.9, and T=10 packed, 48.4 /
// 50.6); 240 workgroups T=8 63.6 / 59.8, 208 T=3 32.2 / 29.3; 64 (H 1024) T=8 63.6 / 78.7, 384 (H
// 6144) T=8 246 / 253.
bool w2_combines(const Layer &L, int T, int k)
{
    const long pairs = (long)T * k, active = pairs < L.E ? pairs : L.E;
    if (pairs > kOwnPairs || active + (pairs + kMfmaChunk - 1) / kMfmaChunk > kOwnChunks ||
        chunk_tokens(L, T, k) != kMfmaChunk)
        return false;
    const int blocks = L.H / 16;
    if (pairs <= 8 && blocks <= 256) return true;
    const bool even = blocks % 256 == 0, most = blocks >= 192 && blocks < 256;
    if (L.wfmt == 2) return T <= 12 && (even || most);
    return L.wfmt == 0 && T <= 8 && L.I <= 2048 && (even || (most && L.wlayout));
}

template <int FMT, bool PK, bool OUTF32>
static hipError_t w2_own_launch(const Layer &L, const uint8_t *ew, const uint8_t *es, int T, int k, const int32_t *meta,
                                const Workspace &ws, void *y, hipStream_t st)
{
    const int P = T * k;
    w2_own_kernel<FMT, PK, OUTF32><<<L.H / 16, 64 * kOwnW, OwnLds::bytes(L.E, P, kOwnTok), st>>>(
        ew, es, meta, ws.slot_of, ws.wts, ws.hs_hi, ws.hs_lo, ws.he_hi, ws.he_lo, y, T, k, L.H, L.I, L.E, L.expert_w_bytes,
        L.expert_s_bytes);
    return hipGetLastError();
}

hipError_t launch_w2_combine(const Layer &L, const void *expert_w, const void *scales, int T, int k, const int32_t *meta,
                             const Workspace &ws, void *y, hipStream_t st)
{
    const uint8_t *ew = (const uint8_t *)expert_w, *es = (const uint8_t *)scales;
    if (L.wfmt == 2) return launch_w2_nvfp4_combine(L, expert_w, scales, T, k, meta, ws, y, st);
#define OWN(F, PK) (L.act_bf16 ? w2_own_launch<F, PK, false>(L, ew, es, T, k, meta, ws, y, st)     \
                               : w2_own_launch<F, PK, true>(L, ew, es, T, k, meta, ws, y, st))
    if (L.wfmt == 0) return L.wlayout ? OWN(0, true) : OWN(0, false);
    return L.wlayout ? OWN(1, true) : OWN(1, false);
#undef OWN
}

hipError_t launch_pack_scales(const Layer &L, const void *src, void *dst, int n_experts, hipStream_t st)
{
    if (L.wfmt == 1) {
        const int64_t bytes = (int64_t)n_experts * (int64_t)L.expert_s_bytes;
        const int64_t blocks = (bytes + 255) / 256;
        pack_e8m0_kernel<<<(unsigned)(blocks < 16384 ? blocks : 16384), 256, 0, st>>>(
            (const uint8_t *)src, (uint8_t *)dst, bytes, L.H, L.I, (int64_t)L.expert_s_bytes);
        return hipGetLastError();
    }
    const int64_t body = (int64_t)2 * L.I * (L.H / 16) + (int64_t)L.H * (L.I / 16);
    const int64_t words = (int64_t)n_experts * body / 4;
    const int64_t blocks = (words + 255) / 256;
    pack_scales_kernel<<<(unsigned)(blocks < 16384 ? blocks : 16384), 256, 0, st>>>(
        (const uint8_t *)src, (uint8_t *)dst, words, L.H, L.I, (int64_t)L.expert_s_bytes);
    return hipGetLastError();
}

hipError_t launch_pack_weights(const Layer &L, const void *src, void *dst, int n_experts, hipStream_t st)
{
    const int64_t pieces = (int64_t)n_experts * (int64_t)L.expert_w_bytes / 16;
    const int64_t blocks = (pieces + 255) / 256;
    pack_kernel<<<(unsigned)(blocks < 16384 ? blocks : 16384), 256, 0, st>>>(
        (const uint8_t *)src, (uint8_t *)dst, pieces, L.H, L.I, L.wfmt, (int64_t)L.expert_w_bytes);
    return hipGetLastError();
}

}  // namespace moe
