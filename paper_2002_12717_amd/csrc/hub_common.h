// Per-cluster view of the Hubbard data and the types shared by the stage kernels
// (hubbard.hip, hub_tile.hip) and the adjoint.
#pragma once
#include <type_traits>

#include "ctx.h"

namespace hub {

struct Cl {
    int ns, zmax;
    double U, s_drive;   // U of the cluster at the stage time (switching applied)
    const int* __restrict__ nbr;    // [2][ns][zmax]
    const cd* __restrict__ hop;     // [2][ns][zmax]
    const double* __restrict__ d0;  // [2][ns]
    const double* __restrict__ xdrv;
    const cd* __restrict__ X;       // stage-input G^{<,up}
    const cd* __restrict__ Y;       // stage-input G^{<,down}
    const cd* __restrict__ hdg;     // [2][ns] diagonals of h^{HF} when precomputed, else unused
    const double* __restrict__ hopr; // [2][ns][zmax] real parts of hop when all hoppings are real, else unused
};

__device__ __forceinline__ Cl make_cl(const ClusterDesc& d, const int* nbr, const cd* hop,
                                      const double* d0, const double* xdrv, const cd* g1,
                                      double s_drive, double u_scale) {
    Cl a;
    a.ns = d.ns;
    a.zmax = d.zmax;
    a.U = d.U * u_scale;
    a.s_drive = s_drive;
    a.nbr = nbr + d.nbroff;
    a.hop = hop + d.nbroff;
    a.d0 = d0 + d.d0off;
    a.xdrv = xdrv + d.xoff;
    a.X = g1 + d.g1off;
    a.Y = a.X + d.ns * d.ns;
    a.hdg = nullptr;
    a.hopr = nullptr;
    return a;
}

// Diagonal of h^{HF,sigma} (Sec. III.D): h0_ii + v_i(t) - i U G^{<,-sigma}_ii.
__device__ __forceinline__ cd hf_diag(const Cl& a, int sig, int i) {
    const cd* other = sig ? a.X : a.Y;
    cd g = other[i * a.ns + i];
    double re = a.d0[sig * a.ns + i] + a.s_drive * a.xdrv[i];
    // -i U (g.x + i g.y) = U g.y - i U g.x
    return cmk(re + a.U * g.y, -a.U * g.x);
}

// Selfenergies of the stage kernels.  DSL (Sec. VI) is GW on the three
// channels with both ladders added on channel A.
enum { SE_SOA = 0, SE_TPP = 1, SE_TPH = 2, SE_GW = 3, SE_DSL = 4 };

__host__ __device__ constexpr bool has_pol(int se) { return se == SE_GW || se == SE_DSL; }
__host__ __device__ constexpr bool has_pp(int se) { return se == SE_TPP || se == SE_DSL; }
__host__ __device__ constexpr bool has_ph(int se) { return se == SE_TPH || se == SE_DSL; }

// G2 channels stored per cluster and diagonal tensors gathered per stage
// (GW's six layouts first, then the particle-hole ladder's two).
__host__ __device__ constexpr int n_channels(int se) { return has_pol(se) ? 3 : 1; }
__host__ __device__ constexpr int n_diag(int se) { return (has_pol(se) ? 6 : 0) + (has_ph(se) ? 2 : 0); }

struct StageArgs {
    const ClusterDesc* __restrict__ desc;
    const WorkItem* __restrict__ work;
    const int* __restrict__ nbr;
    const cd* __restrict__ hop;
    const double* __restrict__ d0;
    const double* __restrict__ xdrv;
    double s_drive;
    double u_scale;   // switching factor phi(t) of the stage
    const cd* in1;
    const cd* in2;
    const cd* y1;
    const cd* y2;
    cd* acc1;
    cd* acc2;
    cd* out1;
    cd* out2;
    double cb, cc;
    DivGuard guard;
    const cd* diag;   // per cluster: GW's six [ns]^3 layouts, then TPH's R and S (hub_diag_kernel)
};

// Storage of the G2 stage registers.  Mixed precision keeps the stage copies
// (the inputs of stages 2-4 and the outputs of stages 1-3) in binary32; y and
// acc, and every G1 register, stay binary64.
template <int MODE, bool MIXED>
struct StageTypes {
    using In = typename std::conditional<MIXED && (MODE == RK_MID || MODE == RK_LAST), float2, cd>::type;
    using Out = typename std::conditional<MIXED && (MODE == RK_FIRST || MODE == RK_MID), float2, cd>::type;
};

constexpr int NS_MAX_ROW = 64;
constexpr int Z_MAX_ROW = 4;

// A wave-uniform value moved to scalar registers.
__device__ __forceinline__ double wave_uniform(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b & 0xffffffffLL));
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ cd wave_uniform(cd v) { return cmk(wave_uniform(v.x), wave_uniform(v.y)); }
__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Element i of an array below 4 GiB, addressed as base + 32-bit byte offset:
// with a wave-uniform base the load takes the scalar-base + vector-offset form
// and needs no 64-bit address arithmetic per lane.
template <typename T>
__device__ __forceinline__ cd ldo(const T* __restrict__ p, unsigned i) {
    return ld_c(reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + i * (unsigned)sizeof(T)), 0);
}

// most G2 elements that one work item stages in LDS
constexpr int SLICE_ELEMS = 4096;

// n / d for n < 2^16 and 1 <= d <= 4096, with mg = slice_magic(d)
__host__ __device__ constexpr unsigned slice_magic(unsigned d) { return d == 1 ? 0u : 0xffffffffu / d + 1u; }
__device__ __forceinline__ int slice_div(int n, unsigned mg) {
    return mg == 0u ? n : (int)__umulhi((unsigned)n, mg);
}

}  // namespace hub

// Kernel arguments of one stage of the whole batch.
hub::StageArgs hub_make_stage(g1g2_ctx* c, double t, const Regs& in, const Regs& y, const Regs& acc, const Regs& out,
                              double cb, double cc);
