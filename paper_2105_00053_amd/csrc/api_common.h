// Host-side helpers shared by the C ABI entry points: format codes, argument
// checks, status strings.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/positnn.h"

namespace pnn {

inline bool is_posit(int f) { return f >= PNN_POSIT8_0 && f <= PNN_POSIT12_2; }
inline bool is_standard(int f) { return (f >= PNN_POSIT8_0 && f <= PNN_POSIT32_2) || f == PNN_F32 || f == PNN_F64; }
inline bool is_float(int f) { return f == PNN_F32 || f == PNN_F64; }
inline size_t elem_size(int f) {
    switch (f) {
        case PNN_POSIT8_0: return 1;
        case PNN_POSIT16_1: return 2;
        case PNN_POSIT32_2: return 4;
        case PNN_POSIT8_1: case PNN_POSIT8_2: return 1;
        case PNN_POSIT10_1: case PNN_POSIT10_2: case PNN_POSIT12_1: case PNN_POSIT12_2: return 2;
        case PNN_F32: return 4;
        case PNN_F64: return 8;
    }
    return 0;
}
inline bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }
inline int hip_status(hipError_t e) { return e == hipSuccess ? PNN_OK : PNN_EHIP; }
// Entry points report their own launches through hipGetLastError(); an error left behind by an earlier, unrelated
// HIP call of this thread would otherwise be blamed on a call that launched fine.  Read (and so reset) it first.
inline void discard_stale_hip_error() { (void)hipGetLastError(); }

// Calls fn.template operator()<F>() ... with the format class of a posit code.
#define PNN_DISPATCH_POSIT(code, CALL)                    \
    switch (code) {                                        \
        case PNN_POSIT8_0: { typedef P8 F; CALL; } break;     \
        case PNN_POSIT16_1: { typedef P16 F; CALL; } break;   \
        case PNN_POSIT32_2: { typedef P32 F; CALL; } break;   \
        case PNN_POSIT8_1: { typedef P8_1 F; CALL; } break;   \
        case PNN_POSIT8_2: { typedef P8_2 F; CALL; } break;   \
        case PNN_POSIT10_1: { typedef P10_1 F; CALL; } break; \
        case PNN_POSIT10_2: { typedef P10_2 F; CALL; } break; \
        case PNN_POSIT12_1: { typedef P12_1 F; CALL; } break; \
        default: { typedef P12_2 F; CALL; } break;            \
    }

// Rounding and conversion beyond Table 1: a kernel with formats known at run time, one element a thread; formats as constants, 16 bytes a thread (rounding of
// binary32 and the narrowing copies of mixed-precision training); a table in LDS for 8-bit sources.  The last two start later -- a thread's four or eight elements in a row, the
// table -- and overtake where the first has more than the chip's threads.  us in a replayed graph, first and the other: f32 to (8,2), 100 elements 1.8 and 2.0,
// 50176 2.0 and 2.4, 300000 2.5 and 2.5, 10^6 4.0 and 3.0, 2^24 41 and 20; (12,2) to (8,2) 100 1.9 and 3.3, 200003 2.4 and 3.4, 700000 3.6 and 3.6, 2 x 10^6 6.8 and 5.0;
// (8,2) to (12,2) 100 1.9 and 2.1, 131072 2.2 and 2.2, 500000 3.1 and 2.3, 2^24 47 and 10.
enum MapChoice { MAP_RUNTIME, MAP_TYPED, MAP_TABLE };
inline MapChoice map_choice(int src, int dst, int64_t n) {
    const bool rounding = src == PNN_F32 && dst >= PNN_POSIT8_1 && dst <= PNN_POSIT12_2;
    const bool narrowing = (dst == PNN_POSIT8_1 && (src == PNN_POSIT12_1 || src == PNN_POSIT10_1)) || (dst == PNN_POSIT8_2 && (src == PNN_POSIT12_2 || src == PNN_POSIT10_2));
    if (rounding || narrowing) return n >= (rounding ? 393216 : 720896) ? MAP_TYPED : MAP_RUNTIME;
    return elem_size(src) == 1 && n >= 163840 ? MAP_TABLE : MAP_RUNTIME;
}

}  // namespace pnn
