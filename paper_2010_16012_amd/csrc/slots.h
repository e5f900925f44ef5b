// Walking the slots [b, e) of an adjacency row several ahead.  Positions are
// unsigned: e may be 2^31 - 1 (the most edges a graph may have), and a signed
// position that runs past it while the last slots are taken would wrap to a
// negative one, which is below every end.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define PP_SLOT_FN __host__ __device__ __forceinline__
#else
#define PP_SLOT_FN inline
#endif

namespace pp {

typedef uint32_t slot_t;

// The slot `ahead` after j, or the last one before e where that lies past it.
PP_SLOT_FN slot_t slot_at(slot_t j, slot_t ahead, slot_t e) { return j + ahead < e - 1 ? j + ahead : e - 1; }

// Whether there is a slot `ahead` after j.
PP_SLOT_FN bool slot_in(slot_t j, slot_t ahead, slot_t e) { return j + ahead < e; }

// End of the k-th piece of `len` slots of a row [b, e).
PP_SLOT_FN int32_t slot_piece_end(slot_t b, slot_t k, slot_t len, slot_t e) {
    const slot_t end = b + (k + 1) * len;
    return (int32_t)(end < e ? end : e);
}

}  // namespace pp
