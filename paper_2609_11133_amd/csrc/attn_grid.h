// Which sequence a workgroup of the attention's split kernel takes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace attn {

// Workgroups go to the eight XCDs in turn, and within an XCD to its four shader engines in
// turn: one of 32 classes by the linear index modulo 32.  With the grid (Hkv, batch,
// splits) a row's splits lie Hkv * batch apart, so where that is a multiple of 16 they all
// fall into one class or two, and a class of long sequences queues while others idle.
// There each split index starts at another sequence: `step` is batch - 11 modulo 32, which
// puts consecutive splits of a sequence 11 * Hkv apart (odd: they go round all classes that
// the key/value heads leave; with 1, sequences sorted by length still collide).  Odd numbers
// up to 13 came out within 1 % over 46 mixes and draws.  Other products spread by themselves:
// 140 rows of chat contexts 15.2 us without, 15.9 with a rotation.
//
// Step us with cycled caches, without / with (and with the split index fastest in the grid;
// block tables as wide as the contexts): 24 agent contexts on 4 heads 20.7 / 19.5 (19.3), 48
// on 2 heads 20.3 / 19.6 (19.5); 64 chat contexts on 2 heads 18.1 / 14.9 (18.1), 40 on 4
// heads 20.4 / 15.8 (24.1).  Where every context has the same length there is nothing to
// even out: 96 rows of 2048 tokens 24.0 / 24.0 (28.0).
struct RowRotation {
    uint32_t step, recip, batch;  // recip = ceil(2^32 / batch): v / batch = mulhi(v, recip) while v * batch < 2^32
    __host__ __device__ RowRotation(uint32_t heads, uint32_t batch)
        : step(batch < 8 || heads * batch % 16 ? 0u : (batch - 11u) & 31u),
          recip(step ? (uint32_t)((0x100000000ull + batch - 1) / batch) : 0u), batch(batch)
    {
    }
    // The sequence of workgroup (., y, split): for each split a permutation of the batch.
    __host__ __device__ uint32_t sequence(uint32_t y, uint32_t split) const
    {
        const uint32_t v = y + step * split;
        return v - (uint32_t)(((uint64_t)v * recip) >> 32) * batch;
    }
};

}  // namespace attn
