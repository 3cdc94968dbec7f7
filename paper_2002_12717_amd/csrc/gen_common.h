// Block shapes, storage access and work-group order shared by the general-basis
// kernels (general.hip, pair.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"
#include "mfma.h"

template <int NB>
struct Shape {
    static constexpr int NT = NB / 16;
    static constexpr int TILES = NT * NT;
    static constexpr int WAVES = (TILES % 4 == 0) ? 4 : ((TILES % 3 == 0) ? 3 : 1);
    static constexpr int TPW = TILES / WAVES;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int LD = NB + 1;
};

template <typename T>
__device__ __forceinline__ void ldc(const cd* p, T& r, T& i) {
    cd v = *p;
    r = (T)v.x;
    i = (T)v.y;
}
template <typename T>
__device__ __forceinline__ void ldc(const float2* p, T& r, T& i) {
    float2 v = *p;
    r = (T)v.x;
    i = (T)v.y;
}
__device__ __forceinline__ void stc(cd* p, double r, double i) { *p = make_double2(r, i); }
__device__ __forceinline__ void stc(float2* p, double r, double i) { *p = make_float2((float)r, (float)i); }

// Work-groups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Logical block b of a grid of g work-groups (g a multiple of 8) is
// mapped so that each XCD owns a contiguous range of logical blocks, which
// keeps neighbouring blocks (adjacent output lines) in one L2.
__device__ __forceinline__ int xcd_block(int b, int g) { return (b & 7) * (g >> 3) + (b >> 3); }

template <typename T, typename S, int NB>
__device__ __forceinline__ void stage_block(const S* __restrict__ src, T* re, T* im) {
    constexpr int LD = Shape<NB>::LD;
    for (int idx = threadIdx.x; idx < NB * NB; idx += blockDim.x) {
        int r = idx / NB, c = idx % NB;
        T a, b;
        ldc(src + idx, a, b);
        re[r * LD + c] = a;
        im[r * LD + c] = b;
    }
}

// Nb = 64 runs eight waves of two tiles instead of four waves of four.  In
// gen_main (one work-group per compute unit) that is two waves per SIMD: 0.82
// instead of 1.11 ms per launch in binary64; holding a wave's rows of G> in
// registers as well gained nothing in binary64 and lost in binary32.  The
// quasi-Hamiltonians (gen_comm, two work-groups per compute unit) take the same
// shape.  Nb = 48 (75 KB of LDS in binary64, two work-groups per compute unit) runs
// nine waves of one tile instead of three of three, 95 registers each, so that both
// work-groups' waves fit: at 45 orbitals gen_main 331 -> 307 us, gen_vt 200 -> 192 us,
// and a mixed second Born step 1.73 -> 1.35 ms.
template <int NB>
struct MainShape : Shape<NB> {
    static constexpr int WAVES = NB == 64 ? 8 : NB == 48 ? 9 : Shape<NB>::WAVES;
    static constexpr int TPW = Shape<NB>::TILES / WAVES;
    static constexpr int THREADS = 64 * WAVES;
};
