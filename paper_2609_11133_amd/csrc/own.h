// Shared parts of the down-projection kernels that also combine (w2_own_kernel in mfma.hip,
// w2_nvfp4_own_kernel in nvfp4.hip): workgroup i owns output rows 16i .. +16 of every pair
// of the step; its waves take the passes (up to TOK tokens of one expert) in turn.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "moe_internal.h"
#include "wave.h"

namespace moe {

typedef float own_f32x4 __attribute__((ext_vector_type(4)));

constexpr int kOwnChunks = 256;    // chunk records at most
constexpr int kOwnPairs = 512;     // (token, expert) pairs at most

// LDS of a workgroup: the pairs' 16 output rows, slots and weights, and the passes.
struct OwnLds {
    own_f32x4 *o;      // [P][4]: the pair's 16 rows
    int *slot;         // [P]
    float *wt;         // [P]
    uint32_t *pass;    // expert | tokens << 10 | first slot << 16
    __device__ OwnLds(float *lds, int P)
        : o(reinterpret_cast<own_f32x4 *>(lds)), slot(reinterpret_cast<int *>(lds) + 16 * P), wt(lds + 17 * P),
          pass(reinterpret_cast<uint32_t *>(lds) + 18 * P)
    {
    }
    // passes of a step at most: one per expert and one more per `tok` pairs
    static size_t bytes(int E, int P, int tok) { return sizeof(float) * (18 * (size_t)P + (P < E ? P : E) + (P + tok - 1) / tok + 1); }
};

// The step's passes in expert order (wave 0) and the combine's slots and weights (the other
// waves), into LDS; returns the number of passes after a barrier.
template <int TOK, int W>
__device__ inline int own_passes(const OwnLds &S, int *s_np, const int32_t *__restrict__ meta,
                                 const int32_t *__restrict__ slot_of, const float *__restrict__ wts, int P, int E,
                                 int wave, int tid)
{
    const MetaIdx mi{E};
    const int4 *recs = reinterpret_cast<const int4 *>(meta + mi.chunk_rec());
    const int lane = tid & 63;
    if (wave == 0) {
        const int n = meta[mi.n_mfma_chunks()], most = min(P, E) + (P + kMfmaChunk - 1) / kMfmaChunk;
        int4 rc[kOwnChunks / 64];  // records past the list's n are not used
#pragma unroll
        for (int u = 0; u < kOwnChunks / 64; ++u) rc[u] = recs[min(64 * u + lane, most - 1)];
        int before = 0;
#pragma unroll
        for (int u = 0; u < kOwnChunks / 64; ++u) {
            const int cnt = 64 * u + lane < n ? (rc[u].z + TOK - 1) / TOK : 0;
            int inc = cnt;
            const int tot = wave_inclusive_scan(inc, lane);
            for (int c = 0; c < cnt; ++c)
                S.pass[before + inc - cnt + c] =
                    (uint32_t)rc[u].x | (uint32_t)min(TOK, rc[u].z - TOK * c) << 10 | (uint32_t)(rc[u].y + TOK * c) << 16;
            before += tot;
        }
        if (lane == 0) *s_np = before;
    } else {
        for (int i = tid - 64; i < P; i += 64 * (W - 1)) {
            S.slot[i] = slot_of[i];
            S.wt[i] = wts[i];
        }
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*s_np);
}

// y of rows row0 .. +16: four rows of a token per thread, choices in rank order.
template <int W, bool OUTF32>
__device__ inline void own_combine(const OwnLds &S, void *__restrict__ y, int T, int k, int H, int row0, int tid)
{
    for (int i = tid; i < 4 * T; i += 64 * W) {
        const int t = i >> 2, q = i & 3;
        own_f32x4 a = {0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < k; ++j) {
            const own_f32x4 v = S.o[S.slot[t * k + j] * 4 + q];
            const float w = S.wt[t * k + j];
#pragma unroll
            for (int c = 0; c < 4; ++c) a[c] = fmaf(w, v[c], a[c]);
        }
        if constexpr (OUTF32) {
            *reinterpret_cast<own_f32x4 *>((float *)y + (size_t)t * H + row0 + 4 * q) = a;
        } else {
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            *reinterpret_cast<uint2 *>((uint16_t *)y + (size_t)t * H + row0 + 4 * q) =
                __builtin_bit_cast(uint2, __builtin_convertvector(a, bf16x4));
        }
    }
}

}  // namespace moe
