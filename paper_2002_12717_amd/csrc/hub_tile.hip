// Hubbard stage over one triangle of the pair matrix.
//
// G2 is Hermitian as a pair matrix, A_ijkl = conj(A_klij) (eq:Gsymm_b), and the
// right-hand side keeps it so (h0 Hermitian, G^< anti-Hermitian).  The stage
// kernels of hubbard.hip evaluate every element; here only the blocks (i,k),
// i >= k, of ns x ns elements (j,l) are evaluated and the block (k,i) is the
// conjugate transpose.  Per G2 element that halves the neighbour loads, which
// bound those kernels, the flops and the register traffic.
//
// A block is a tile of a work item: its ns rows A[i][j][k][:] are staged in LDS,
// where the j- and l-neighbours of the commutator lie; the i- and k-neighbours
// are rows of other blocks.  The source (eq:soa-cubic-scheme) at fixed (i,k) is
//     Psi_jl = Y_jl (alpha_j - beta_l) + gamma_j Y_il - delta_j Y_kl
// with alpha, beta, gamma, delta vectors of the tile, formed once per tile, so
// that one G1 element per G2 element is read from memory instead of ten.
//
// The transposed block is written where it is read: after the last stage
// always, in the other stages only where a neighbour across the diagonal or the
// caller (full) reads it.  The tile is read back, transposed through LDS and
// written in whole rows.  The last stage closes the blocks (i,i) in the same way,
// so that a step keeps the symmetry bit for bit: a restart from a saved state
// takes these kernels again.
//
// In binary64 the Runge-Kutta step keeps no running sum (rk_close); mixed
// precision stores the stage inputs in binary32 and keeps it.
//
// Condition: state with the symmetry to the last bit (checked when a state is set,
// hub_check_state: an asymmetry, however small, is evolved by the kernels that
// evaluate every element), real hoppings that are equal in both directions,
// ns <= 64, at most Z_MAX_ROW neighbours per site.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "ctx.h"
#include "hub_common.h"

using namespace hub;

namespace {

// Threads of a work-group and its waves per SIMD.  ROW: two work-groups per
// compute unit (a 64-site tile takes 64 KB of LDS in binary64); second Born has
// the registers for 12 waves each.  Mean stage at 8x8 sites with 8 / 12 waves:
// SOA 227 / 207 us, TPP 233 / 269, TPH 224 / 233, GW 643 / 638, DSL 771 / 995.
// Packed items of at most TILE_ELEMS elements leave the LDS for four work-groups
// (64 ragged TPP clusters, 9 to 36 sites: 413 us; 2,048 elements 485, 4,096 673).
constexpr int TILE_ELEMS = 1024;
__host__ __device__ constexpr int tile_threads(int se, bool row) { return row && se == SE_SOA ? 768 : 512; }
__host__ __device__ constexpr int tile_waves(int se, bool row) { return !row ? 8 : se == SE_SOA ? 6 : 4; }
// bits of a tile word: i, k, channel, and whether stages read the transposed block
constexpr int TW_NEED = 1 << 20;

struct TileArgs {
    const int* tiles;
    const cd* diag;              // per cluster: the diagonal tensors (hub_tdiag_kernel)
    const cd *r21, *r31;         // binary64, last stage: Y2 and Y3 of G1 ...
    const cd *r22, *r32;         // ... and of G2
    int full;                    // write every transposed block
};

// diagonal tensors: GW's six, TPH's R and S, TPP's E and F
__host__ __device__ constexpr int n_tdiag(int se) {
    return (has_pol(se) ? 6 : 0) + (has_ph(se) ? 2 : 0) + (has_pp(se) ? 2 : 0);
}
// per-tile vectors in LDS: alpha, gamma, delta, beta, Y_i, Y_k; X_i, X_k of a
// ladder; R_j.i and S_i k. of TPH; D1_ik. of GW
enum { V_AL = 0, V_GA = 1, V_DE = 2, V_BE = 3, V_YI = 4, V_YK = 5, V_XI = 6, V_XK = 7 };
__host__ __device__ constexpr int v_ph(int se) { return has_pp(se) || has_ph(se) ? 8 : 6; }
__host__ __device__ constexpr int v_pol(int se) { return v_ph(se) + (has_ph(se) ? 2 : 0); }
__host__ __device__ constexpr int n_vec(int se) { return v_pol(se) + (has_pol(se) ? 1 : 0); }

template <typename T>
__device__ __forceinline__ cd ld_herm(const T* __restrict__ A, int ns, int i, int j, int k, int l) {
    if (i >= k) return ld_c(A, (((long long)i * ns + j) * ns + k) * ns + l);
    return cconj(ld_c(A, (((long long)k * ns + l) * ns + i) * ns + j));
}

// Update of one element with slope f; av is the stage input at e.
template <int MODE, bool MIXED, typename TO>
__device__ __forceinline__ cd tile_update(unsigned e, cd f, cd av, const cd* __restrict__ y, cd* __restrict__ acc,
                                          const cd* __restrict__ r2, const cd* __restrict__ r3, double cb, double cc) {
    if (MODE == RK_FIRST) {
        if (MIXED) st_nt(acc + e, cmk(fma(cb, f.x, av.x), fma(cb, f.y, av.y)));
        return cmk(fma(cc, f.x, av.x), fma(cc, f.y, av.y));
    }
    if (MODE == RK_MID) {
        const cd yv = ld_nt(y + e);
        if (MIXED) {
            const cd a = ld_nt(acc + e);
            st_nt(acc + e, cmk(fma(cb, f.x, a.x), fma(cb, f.y, a.y)));
        }
        return cmk(fma(cc, f.x, yv.x), fma(cc, f.y, yv.y));
    }
    if (MIXED) {
        const cd a = ld_nt(acc + e);
        return cmk(fma(cb, f.x, a.x), fma(cb, f.y, a.y));
    }
    return rk_close(ld_nt(y + e), ld_nt(r2 + e), ld_nt(r3 + e), av, f, cb);
}

// G1 of one cluster (eq:eom_g1_hubbard); the collision integral's elements of A
// are read from the evaluated triangle.  The slopes of (i,j) and (j,i) are formed
// from the same sums, so that G^< stays anti-Hermitian bit for bit.
template <int MODE, bool MIXED, typename TI>
__device__ void tile_g1(const StageArgs& s, const TileArgs& t, const Cl& a, const ClusterDesc& d, int cluster,
                        const TI* __restrict__ A) {
    const int ns = a.ns, ns2 = ns * ns, z = a.zmax;
    const cd* y = s.y1 + d.g1off;
    cd* acc = s.acc1 + d.g1off;
    cd* out = s.out1 + d.g1off;
    if (MODE == RK_FIRST && cluster == 0 && threadIdx.x == 0) guard_begin_step(s.guard);
    const unsigned long long step = MODE == RK_LAST ? s.guard.div[0] : 0ull;
    for (int e = threadIdx.x; e < 2 * ns2; e += blockDim.x) {
        const int sig = e / ns2, r = e % ns2, i0 = r / ns, j0 = r % ns;
        const int i = max(i0, j0), j = min(i0, j0);
        const cd* G = sig ? a.Y : a.X;
        const int* nb = a.nbr + sig * ns * z;
        const cd* hp = a.hop + sig * ns * z;
        cd c = cmul(csub(hf_diag(a, sig, i), hf_diag(a, sig, j)), G[i * ns + j]);
        for (int q = 0; q < z; ++q) {
            const int p = nb[i * z + q];
            if (p >= 0) c = cfma(c, hp[i * z + q], G[p * ns + j]);
        }
        for (int q = 0; q < z; ++q) {
            const int p = nb[j * z + q];
            if (p >= 0) c = csub(c, cmul(G[i * ns + p], cconj(hp[j * z + q])));
        }
        // I^up_ij = -i U A_iiji, I^down_ij = -i U A_iiij
        const cd Iij = sig ? ld_herm(A, ns, i, i, i, j) : ld_herm(A, ns, i, i, j, i);
        const cd Iji = sig ? ld_herm(A, ns, j, j, j, i) : ld_herm(A, ns, j, j, i, j);
        c = cadd(c, cscale(cadd(cmul_mi(Iij), cconj(cmul_mi(Iji))), a.U));
        cd f = cmul_mi(c);
        if (i0 < j0) f.x = -f.x;
        if (i0 == j0) f.x = 0.0;
        const cd o = tile_update<MODE, MIXED, cd>((unsigned)e, f, G[r], y, acc, t.r21 + d.g1off, t.r31 + d.g1off,
                                                  s.cb, s.cc);
        out[e] = o;
        if (MODE == RK_LAST && guard_bad(o, i0 == j0)) guard_fire(s.guard, cluster, step);
    }
}

// ROW: an item is one tile and a wave takes a row (i,j,k) at a time, lane = l, so
// that everything indexed by i and k is uniform and the vectors over l stay in
// registers (one launch form for clusters that fill most of a wave's lanes).
// Otherwise an item packs the tiles of smaller clusters and every lane has an
// element of its own.
template <int MODE, int SE, bool MIXED, bool ROW>
__global__ __launch_bounds__(tile_threads(SE, ROW)) __attribute__((amdgpu_waves_per_eu(tile_waves(SE, ROW))))
void hub_tile_kernel(StageArgs s, TileArgs t) {
    constexpr bool TPP = has_pp(SE), TPH = has_ph(SE), GW = has_pol(SE);
    using TI = typename StageTypes<MODE, MIXED>::In;
    using TO = typename StageTypes<MODE, MIXED>::Out;
    constexpr int ZR = Z_MAX_ROW, TILE_THREADS = tile_threads(SE, ROW);
    extern __shared__ cd dyn[];
    // padded neighbour tables (a missing neighbour has offset 0 and hopping 0) for
    // the spins of (i,k) and (j,l) in the item's channel
    __shared__ int ofl[NS_MAX_ROW * ZR], ofj[NS_MAX_ROW * ZR];
    __shared__ int ofi[ROW ? 1 : NS_MAX_ROW * ZR], ofk[ROW ? 1 : NS_MAX_ROW * ZR];
    __shared__ double shj[NS_MAX_ROW * ZR], shi[ROW ? 1 : NS_MAX_ROW * ZR];
    __shared__ cd ejs[NS_MAX_ROW], eis[ROW ? 1 : NS_MAX_ROW];
    const WorkItem w = s.work[blockIdx.x];
    const ClusterDesc d = s.desc[w.cluster];
    const Cl a = make_cl(d, s.nbr, s.hop, s.d0, s.xdrv, s.in1, s.s_drive, s.u_scale);
    const int ns = d.ns, z = d.zmax, ns2 = ns * ns, ns3 = ns2 * ns;
    const TI* __restrict__ A = reinterpret_cast<const TI*>(s.in2) + d.g2off;
    const int tid = threadIdx.x;
    if (w.start < 0) {
        tile_g1<MODE, MIXED, TI>(s, t, a, d, w.cluster, A);
        return;
    }
    const int T = w.end - w.start;
    if (T <= 0) return;
    const int* __restrict__ tw = t.tiles + w.start;
    const int w0 = tw[0];
    const int ch = GW ? (w0 >> 16) & 3 : 0;   // items do not cross channels
    const int sI = ch == 2 ? 1 : 0, sJ = ch == 1 ? 0 : 1;
    const bool src = !GW || ch == 0;
    const long long n4 = (long long)ns2 * ns2;
    const TI* __restrict__ Ach = A + ch * n4;
    const cd* __restrict__ X = a.X;
    const cd* __restrict__ Y = a.Y;
    const cd* __restrict__ DG = t.diag + (long long)n_tdiag(SE) * d.doff;
    const cd* __restrict__ D1 = GW ? DG + (ch == 0 ? 4 : (ch == 1 ? 0 : 2)) * (long long)ns3 : nullptr;   // UB, UA, VA
    const cd* __restrict__ D2 = GW ? DG + (ch == 0 ? 5 : (ch == 1 ? 1 : 3)) * (long long)ns3 : nullptr;   // TC, TA, WA
    const cd* __restrict__ DR = TPH ? DG + (GW ? 6 : 0) * (long long)ns3 : nullptr;
    const cd* __restrict__ DS = TPH ? DR + ns3 : nullptr;
    const cd* __restrict__ DE = TPP ? DG + ((GW ? 6 : 0) + (TPH ? 2 : 0)) * (long long)ns3 : nullptr;
    const cd* __restrict__ DF = TPP ? DE + ns3 : nullptr;
    const cd* __restrict__ S1 = ch == 1 ? X : Y;
    const cd* __restrict__ S2 = ch == 2 ? Y : X;
    TI* const P = reinterpret_cast<TI*>(dyn);
    cd* const vec = reinterpret_cast<cd*>(P + ((T * ns2 + 1) & ~1));
    const unsigned mg2 = slice_magic((unsigned)ns2), mg1 = slice_magic((unsigned)ns);
    for (int q = tid; q < ns * ZR; q += TILE_THREADS) {
        const int site = q / ZR, qq = q - site * ZR;
        const int pj = qq < z ? a.nbr[(sJ * ns + site) * z + qq] : -1;
        ofl[q] = pj >= 0 ? pj - site : 0;
        ofj[q] = pj >= 0 ? (pj - site) * ns : 0;
        shj[q] = pj >= 0 ? a.hop[(sJ * ns + site) * z + qq].x : 0.0;
        if constexpr (!ROW) {
            const int pi = qq < z ? a.nbr[(sI * ns + site) * z + qq] : -1;
            ofi[q] = pi >= 0 ? (pi - site) * ns3 : 0;
            ofk[q] = pi >= 0 ? (pi - site) * ns : 0;
            shi[q] = pi >= 0 ? a.hop[(sI * ns + site) * z + qq].x : 0.0;
        }
    }
    for (int q = tid; q < ns; q += TILE_THREADS) {
        ejs[q] = hf_diag(a, sJ, q);
        if constexpr (!ROW) eis[q] = hf_diag(a, sI, q);
    }
    // the tiles and their vectors
    auto tile_ik = [&](int tl, int& i, int& k) {
        const int word = ROW ? w0 : tw[tl];
        i = word & 255;
        k = (word >> 8) & 255;
    };
    for (int m = tid; m < T * ns2; m += TILE_THREADS) {
        const int tl = ROW ? 0 : slice_div(m, mg2), r = m - tl * ns2, j = slice_div(r, mg1), l = r - j * ns;
        int i, k;
        tile_ik(tl, i, k);
        P[m] = Ach[((i * ns + j) * ns + k) * ns + l];
    }
    for (int q = tid; q < T * ns; q += TILE_THREADS) {
        const int tl = ROW ? 0 : slice_div(q, mg1), x = q - tl * ns;
        int i, k;
        tile_ik(tl, i, k);
        auto put = [&](int v, cd val) { vec[v * T * ns + q] = val; };
        if (src) {
            const cd xik = X[i * ns + k], xix = X[i * ns + x], xkx = X[k * ns + x];
            const cd yxi = Y[x * ns + i], yxk = Y[x * ns + k], xxk = X[x * ns + k];
            cd al = cscale(cmul_i(cmul(xix, xxk)), a.U), be = cscale(cmul_i(cmul(cmk(-xkx.x, xkx.y), xix)), a.U);
            if (x == i) al = cadd(al, cscale(xik, a.U));
            if (x == k) be = cadd(be, cscale(xik, a.U));
            put(V_AL, al);
            put(V_BE, be);
            put(V_GA, cscale(cmul_i(cmul(xik, yxi)), a.U));
            put(V_DE, cscale(cmul_i(cmul(xik, yxk)), a.U));
            put(V_YI, Y[i * ns + x]);
            put(V_YK, Y[k * ns + x]);
            if (TPP || TPH) {
                put(V_XI, xix);
                put(V_XK, xkx);
            }
            if (TPH) {
                put(v_ph(SE), DR[(x * ns + k) * ns + i]);
                put(v_ph(SE) + 1, DS[(i * ns + k) * ns + x]);
            }
        }
        if (GW) put(v_pol(SE), D1[(i * ns + k) * ns + x]);
    }
    __syncthreads();
    const cd* __restrict__ yr = s.y2 + d.g2off + ch * n4;
    cd* acc = s.acc2 + d.g2off + ch * n4;
    const cd* __restrict__ r2 = t.r22 + d.g2off + ch * n4;
    const cd* __restrict__ r3 = t.r32 + d.g2off + ch * n4;
    TO* out = reinterpret_cast<TO*>(s.out2) + d.g2off + ch * n4;
    // ROW: offsets and hoppings of i and k, and the vectors at l, in registers
    int oi[ZR], ok[ZR];
    double hi[ZR], hk[ZR];
    cd eik = cmk(0.0, 0.0);
    int ri = 0, rk = 0;
    if constexpr (ROW) {
        tile_ik(0, ri, rk);
#pragma unroll
        for (int q = 0; q < ZR; ++q) {
            const int pi = q < z ? a.nbr[(sI * ns + ri) * z + q] : -1, pk = q < z ? a.nbr[(sI * ns + rk) * z + q] : -1;
            oi[q] = wave_uniform(pi >= 0 ? (pi - ri) * ns3 : 0);
            ok[q] = wave_uniform(pk >= 0 ? (pk - rk) * ns : 0);
            hi[q] = wave_uniform(pi >= 0 ? a.hop[(sI * ns + ri) * z + q].x : 0.0);
            hk[q] = wave_uniform(pk >= 0 ? a.hop[(sI * ns + rk) * z + q].x : 0.0);
        }
        eik = wave_uniform(csub(hf_diag(a, sI, ri), hf_diag(a, sI, rk)));
    }
    auto element = [&](const int m, const int tl, const int i, const int k, const int j, const int l) {
        const unsigned e = ((i * ns + j) * ns + k) * ns + l;
        const cd av = ld_c(P, m);
        const cd ed = ROW ? eik : csub(eis[i], eis[k]);
        const cd ejl = csub(ejs[j], ejs[l]);
        cd c = cmul(cadd(ed, ejl), av);
        // h_jp A_ipkl - A_ijkp h_pl from the tile, h_ip A_pjkl - A_ijpl h_pk from other blocks
#pragma unroll
        for (int q = 0; q < ZR; ++q) {
            const cd vi = ldo(Ach, e + (ROW ? oi[q] : ofi[i * ZR + q]));
            const cd vk = ldo(Ach, e + (ROW ? ok[q] : ofk[k * ZR + q]));
            const double xi = ROW ? hi[q] : shi[i * ZR + q], xk = ROW ? hk[q] : shi[k * ZR + q];
            c.x = fma(xi, vi.x, fma(-xk, vk.x, c.x));
            c.y = fma(xi, vi.y, fma(-xk, vk.y, c.y));
        }
#pragma unroll
        for (int q = 0; q < ZR; ++q) {
            const cd vj = ld_c(P, m + ofj[j * ZR + q]), vl = ld_c(P, m + ofl[l * ZR + q]);
            const double xj = shj[j * ZR + q], xl = shj[l * ZR + q];
            c.x = fma(xj, vj.x, fma(-xl, vl.x, c.x));
            c.y = fma(xj, vj.y, fma(-xl, vl.y, c.y));
        }
        auto V = [&](int v, int x) { return vec[(v * T + tl) * ns + x]; };
        const cd yjl = ldo(S1, j * ns + l);   // Y_jl, or X_jl in GW's up-up channel
        if (GW) {   // Pi_1 - conj(Pi_2), see hub_slice_kernel
            const cd s2 = ldo(S2, k * ns + i);
            const cd p1 = cmul_mi(cmul(yjl, csub(V(v_pol(SE), j), V(v_pol(SE), l))));
            const cd p2 = cmul_mi(cmul(s2, csub(ldo(D2, (k * ns + j) * ns + l), ldo(D2, (i * ns + j) * ns + l))));
            c = cadd(c, cscale(csub(p1, cconj(p2)), a.U));
        }
        if (src) {
            const cd yil = V(V_YI, l), ykl = V(V_YK, l);
            c = cfma(c, yjl, csub(V(V_AL, j), V(V_BE, l)));
            c = cfma(c, V(V_GA, j), yil);
            const cd de = V(V_DE, j);
            c = cfma(c, cmk(-de.x, -de.y), ykl);
            if (TPP) {
                //   L_ijkl = delta_ij U A_iikl + i U (Y_ji A_iikl + X_ij A_jjkl), partner L_klij
                const cd yij = V(V_YI, j), dii = ld_c(P, tl * ns2 + i * ns + l), djj = ldo(DE, (k * ns + j) * ns + l);
                cd l1 = cmul_i(cadd(cmul(cmk(-yij.x, yij.y), dii), cmul(V(V_XI, j), djj)));
                if (i == j) l1 = cadd(l1, dii);
                const cd dkk = cconj(ld_c(P, tl * ns2 + j * ns + k)), dll = ldo(DF, (i * ns + j) * ns + l);
                cd l2 = cmul_i(cadd(cmul(cmk(-ykl.x, ykl.y), dkk), cmul(V(V_XK, l), dll)));
                if (k == l) l2 = cadd(l2, dkk);
                c = cadd(c, cscale(csub(l1, cconj(l2)), a.U));
            }
            if (TPH) {
                //   L_ijkl = i U (Y_il A_ijki - X_il A_ljkl), L_klij = i U (Y_kj A_klik - X_kj A_jlij)
                const cd rjkl = ldo(DR, (j * ns + k) * ns + l), sijl = ldo(DS, (i * ns + j) * ns + l);
                const cd l1 = cmul_i(csub(cmul(yil, V(v_ph(SE), j)), cmul(V(V_XI, l), rjkl)));
                const cd l2 = cmul_i(csub(cmul(V(V_YK, j), V(v_ph(SE) + 1, l)), cmul(V(V_XK, j), sijl)));
                c = cadd(c, cscale(csub(l1, cconj(l2)), a.U));
            }
        }
        st_c(out, e, tile_update<MODE, MIXED, TO>(e, cmul_mi(c), av, yr, acc, r2, r3, s.cb, s.cc));
    };
    if constexpr (ROW) {
        const int wid = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
        if (l < ns)
            for (int j = wid; j < ns; j += TILE_THREADS / 64) element(j * ns + l, 0, ri, rk, j, l);
    } else {
        for (int m = tid; m < T * ns2; m += TILE_THREADS) {
            const int tl = slice_div(m, mg2), r = m - tl * ns2, j = slice_div(r, mg1), l = r - j * ns;
            int i, k;
            tile_ik(tl, i, k);
            element(m, tl, i, k, j, l);
        }
    }
    // the transposed blocks; in the last stage also the blocks (i,i), whose elements
    // below the diagonal are the conjugates of those above
    auto wanted = [&](int word) {
        return MODE == RK_LAST || ((word & 255) != ((word >> 8) & 255) && (t.full || (word & TW_NEED)));
    };
    bool any = false;
    for (int tl = 0; tl < T; ++tl) any = any || wanted(tw[tl]);
    if (!any) return;
    __syncthreads();
    TO* const Q = reinterpret_cast<TO*>(dyn);
    for (int m = tid; m < T * ns2; m += TILE_THREADS) {
        const int tl = ROW ? 0 : slice_div(m, mg2), r = m - tl * ns2, j = slice_div(r, mg1), l = r - j * ns;
        if (!ROW && !wanted(tw[tl])) continue;
        int i, k;
        tile_ik(tl, i, k);
        Q[(tl * ns + j) * (ns + 1) + l] = out[((i * ns + j) * ns + k) * ns + l];
    }
    __syncthreads();
    for (int m = tid; m < T * ns2; m += TILE_THREADS) {
        const int tl = ROW ? 0 : slice_div(m, mg2), r = m - tl * ns2, l = slice_div(r, mg1), j = r - l * ns;
        if (!ROW && !wanted(tw[tl])) continue;
        int i, k;
        tile_ik(tl, i, k);
        if (MODE == RK_LAST && i == k && l < j) continue;
        TO v = Q[(tl * ns + j) * (ns + 1) + l];
        v.y = MODE == RK_LAST && i == k && l == j ? 0 : -v.y;
        out[((k * ns + l) * ns + i) * ns + j] = v;
    }
}

// Dynamic LDS of an item of T tiles of ns x ns: the staged tiles and vectors, or
// the padded tiles of the transposition.
template <int MODE, int SE, bool MIXED>
size_t tile_lds(int T, int ns) {
    using TI = typename StageTypes<MODE, MIXED>::In;
    using TO = typename StageTypes<MODE, MIXED>::Out;
    const size_t a = (((size_t)T * ns * ns + 1) & ~(size_t)1) * sizeof(TI) + (size_t)n_vec(SE) * T * ns * sizeof(cd);
    return std::max(a, (size_t)T * ns * (ns + 1) * sizeof(TO));
}

// The diagonal tensors of the stage input, from the evaluated triangle: those of
// hub_diag_kernel (GW's six, R, S), then for TPP
//   E[a][b][c] = A_bbac,  F[a][c][b] = A_bbac
template <typename TI, int SE>
__global__ __launch_bounds__(256) void hub_tdiag_kernel(const ClusterDesc* __restrict__ desc,
                                                       const WorkItem* __restrict__ dwork,
                                                       const cd* __restrict__ in2, cd* __restrict__ diag) {
    const WorkItem w = dwork[blockIdx.x];
    const ClusterDesc d = desc[w.cluster];
    const int ns = d.ns, ns2 = ns * ns, ns3 = ns2 * ns;
    const long long n4 = (long long)ns2 * ns2;
    const TI* A = reinterpret_cast<const TI*>(in2) + d.g2off;
    cd* D = diag + (long long)n_tdiag(SE) * d.doff;
    cd* DRS = D + (has_pol(SE) ? 6 * ns3 : 0);
    cd* DEF = DRS + (has_ph(SE) ? 2 * ns3 : 0);
    for (int t = w.start + threadIdx.x; t < w.end; t += blockDim.x) {
        const int x = t / ns2, y = (t / ns) % ns, z = t % ns;
        if (has_ph(SE)) {   // (x, y, z) = (a, b, c): A_cabc
            const cd v = ld_herm(A, ns, z, x, y, z);
            DRS[t] = v;
            DRS[ns3 + (y * ns + z) * ns + x] = v;
        }
        if (has_pp(SE)) {   // (a, b, c): A_bbac
            const cd v = ld_herm(A, ns, y, y, x, z);
            DEF[t] = v;
            DEF[ns3 + (x * ns + z) * ns + y] = v;
        }
        if (has_pol(SE)) {
            // (x, y, z) = (a, b, c): P_abcb of A, B, C
            const cd va = ld_herm(A, ns, x, y, z, y), vb = ld_herm(A + n4, ns, x, y, z, y),
                     vc = ld_herm(A + 2 * n4, ns, x, y, z, y);
            D[(x * ns + z) * ns + y] = va;                   // UA
            D[ns3 + (y * ns + z) * ns + x] = va;             // TA
            D[4 * ns3 + (x * ns + z) * ns + y] = vb;         // UB
            D[5 * ns3 + (y * ns + z) * ns + x] = vc;         // TC
            const cd vd = ld_herm(A, ns, x, y, x, z);        // A_abad
            D[2 * ns3 + (y * ns + z) * ns + x] = vd;         // VA
            D[3 * ns3 + (x * ns + z) * ns + y] = vd;         // WA
        }
    }
}

// Symmetry of a state: per block (i,k), i >= k, the maxima of |A_ijkl -
// conj(A_klij)| and |A|; the G1 item of a cluster those of |G + G^dagger| and |G|.
// res[0..1] and res[2..3] are the bits of these nonnegative numbers, ~0 for NaN.
__global__ __launch_bounds__(256) void hub_herm_kernel(StageArgs s, const int* __restrict__ tiles,
                                                      unsigned long long* __restrict__ res) {
    __shared__ double sh[2][4];
    const WorkItem w = s.work[blockIdx.x];
    const ClusterDesc d = s.desc[w.cluster];
    const int ns = d.ns, ns2 = ns * ns, tid = threadIdx.x;
    double md = 0.0, mx = 0.0;
    bool nan = false;
    auto take = [&](cd u, cd v) {   // |u - v|, |u|
        const double dx = fabs(u.x - v.x), dy = fabs(u.y - v.y);
        nan = nan || !(dx + dy < 1e300);
        md = fmax(md, fmax(dx, dy));
        mx = fmax(mx, fmax(fabs(u.x), fabs(u.y)));
    };
    const bool g1 = w.start < 0;
    if (g1) {
        const cd* G = s.in1 + d.g1off;
        for (int e = tid; e < 2 * ns2; e += 256) {
            const int sig = e / ns2, r = e - sig * ns2, i = r / ns, j = r - i * ns;
            const cd v = G[sig * ns2 + j * ns + i];
            take(G[e], cmk(-v.x, v.y));
        }
    } else {
        __shared__ cd P[NS_MAX_ROW][17];
        for (int tt = w.start; tt < w.end; ++tt) {
            const int word = tiles[tt], i = word & 255, k = (word >> 8) & 255, ch = (word >> 16) & 3;
            const cd* A = s.in2 + d.g2off + ch * (long long)ns2 * ns2;
            // strips of 16 j: rows of block (i,k) staged, columns of block (k,i) compared
            for (int j0 = 0; j0 < ns; j0 += 16) {
                const int nj = min(16, ns - j0);
                __syncthreads();
                for (int m = tid; m < ns * nj; m += 256) {
                    const int jj = m / ns, l = m - jj * ns;
                    P[l][jj] = A[((i * ns + j0 + jj) * ns + k) * ns + l];
                }
                __syncthreads();
                for (int m = tid; m < ns * nj; m += 256) {
                    const int l = m / nj, jj = m - l * nj;
                    take(P[l][jj], cconj(A[((k * ns + l) * ns + i) * ns + j0 + jj]));
                }
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        md = fmax(md, __shfl_xor(md, o, 64));
        mx = fmax(mx, __shfl_xor(mx, o, 64));
    }
    if (nan) atomicMax(res + (g1 ? 2 : 0), ~0ull);
    if ((tid & 63) == 0) {
        sh[0][tid >> 6] = md;
        sh[1][tid >> 6] = mx;
    }
    __syncthreads();
    if (tid < 2) {
        double m = 0.0;
        for (int q = 0; q < 4; ++q) m = fmax(m, sh[tid][q]);
        atomicMax(res + (g1 ? 2 : 0) + tid, (unsigned long long)__double_as_longlong(m));
    }
}

template <int MODE, int SE, bool MIXED>
void launch_tile(g1g2_ctx* c, const StageArgs& s, const TileArgs& t) {
    const HubbardData& H = c->hub;
    if (n_tdiag(SE) > 0) {
        using TI = typename StageTypes<MODE, MIXED>::In;
        hipLaunchKernelGGL((hub_tdiag_kernel<TI, SE>), dim3(H.ndwork), dim3(256), 0, c->stream, H.desc, H.dwork, s.in2,
                           const_cast<cd*>(t.diag));
    }
    if (H.ntrow > 0)
        hipLaunchKernelGGL((hub_tile_kernel<MODE, SE, MIXED, true>), dim3(H.ntrow), dim3(tile_threads(SE, true)),
                           (tile_lds<MODE, SE, MIXED>(1, H.row_ns)), c->stream, s, t);
    if (H.ntpack > 0) {
        size_t lds = 0;
        for (const auto& x : H.tile_shapes) lds = std::max(lds, tile_lds<MODE, SE, MIXED>(x.first, x.second));
        StageArgs sp = s;
        sp.work += H.ntrow;
        hipLaunchKernelGGL((hub_tile_kernel<MODE, SE, MIXED, false>), dim3(H.ntpack), dim3(tile_threads(SE, false)), lds,
                           c->stream, sp, t);
    }
}

template <int MODE, int SE>
void launch_tile_p(g1g2_ctx* c, const StageArgs& s, const TileArgs& t) {
    if (c->d.precision == G1G2_MIXED) launch_tile<MODE, SE, true>(c, s, t);
    else launch_tile<MODE, SE, false>(c, s, t);
}

template <int MODE>
void launch_tile_se(g1g2_ctx* c, const StageArgs& s, const TileArgs& t) {
    switch (c->d.selfenergy) {
        case G1G2_TPP: launch_tile_p<MODE, SE_TPP>(c, s, t); break;
        case G1G2_TPH: launch_tile_p<MODE, SE_TPH>(c, s, t); break;
        case G1G2_GW: launch_tile_p<MODE, SE_GW>(c, s, t); break;
        case G1G2_DSL: launch_tile_p<MODE, SE_DSL>(c, s, t); break;
        default: launch_tile_p<MODE, SE_SOA>(c, s, t); break;
    }
}

}  // namespace

// Least cluster, in sites, that the steps over one triangle pay for, per closure.  Below
// it the diagonal gather and the vectors of a tile weigh more than the half of the
// elements they save.  Batches of 1.2 x 2^20 elements in clusters of one size, 8 steps,
// slice kernel against this one, binary64 / mixed, in us:
//   TPP  5 sites 1271 / 1185 against 1476 / 1394, 7 sites 1138 / 1033 against 1200 / 1230,
//        8 sites 990 / 910 against 935 / 920
//   DSL  4 sites 4830 / 4680 against 6222 / 6280, 5 sites 0.99 and 1.00 of each other
//   GW   4 sites 5450 / 5280 against 5602 / 5390, 5 sites 1.10 and 1.15 times faster here
// Second Born and TPH gain at every size (1.06 to 2.3 times).
extern "C" int hub_tile_least(int selfenergy) {
    return selfenergy == G1G2_TPP ? 8 : selfenergy == G1G2_DSL || selfenergy == G1G2_GW ? 5 : 1;
}

// Whether a system of `elems` G2 elements per channel, `small` of them in clusters below
// hub_tile_least and `single` in clusters of 26 to 36 sites, and at most z neighbours per
// site takes the triangle: its larger part must pay.  In mixed TPP with more than two
// neighbours an item of one tile fills its 512 threads worse than the slice kernel's
// three or four slices do, which tells while the system is a few waves of work (8 steps,
// slice kernel against this one, in us: 12x3 sites 1326 against 1494, 6x6 1374 / 1484, two
// of 7x4 1062 / 1163; but three of 7x4 1817 / 1296, 13x3 2019 / 1852, a chain of 33 sites
// 1122 / 1048).  Host arithmetic with names that tests can find.
extern "C" int hub_tile_pays(int selfenergy, int mixed, int z, long long elems, long long small, long long single) {
    if (2 * small > elems) return 0;
    return !(selfenergy == G1G2_TPP && mixed && z > 2 && elems < (7LL << 18) && 2 * single > elems);
}

// Tiles of a work item of a cluster of ns sites that holds at most `most` elements: no
// more than the cluster has, since the launch takes the LDS of its largest item for
// all (a two-site cluster has three tiles, and room for 192 of them, 61 KB, took
// every work-group of its batch from four per compute unit to two), and in equal
// shares (seven sites: 14 and 14 tiles rather than 20 and 8).
extern "C" int hub_tile_per_item(int ns, int most) {
    if (ns >= TILE_ROW_MIN) return 1;
    const int fit = std::min(std::min(most, TILE_ELEMS) / (ns * ns), TILE_VEC / ns);
    const int nt = ns * (ns + 1) / 2, items = (nt + std::max(1, fit) - 1) / std::max(1, fit);
    return (nt + items - 1) / items;   // equal shares
}

// Tiles and work items of every cluster.  nbr: the host neighbour tables;
// per_item: the most G2 elements of an item per cluster.
void hub_tile_lists(g1g2_ctx* c, const std::vector<ClusterDesc>& desc, const std::vector<int>& nbr,
                    const std::vector<int>& per_item, std::vector<int>& tiles, std::vector<WorkItem>& work) {
    HubbardData& H = c->hub;
    const int sel = c->d.selfenergy;
    const int nch = sel == G1G2_GW || sel == G1G2_DSL ? 3 : 1;
    std::vector<WorkItem> items[2], g1[2];   // wave-per-row form, packed form
    std::vector<long long> cost[2];
    H.tile_shapes.clear();
    H.row_ns = 0;
    for (int cl = 0; cl < (int)desc.size(); ++cl) {
        const ClusterDesc& d = desc[cl];
        const int ns = d.ns, z = d.zmax, form = ns >= TILE_ROW_MIN ? 0 : 1;
        if (form == 0) H.row_ns = std::max(H.row_ns, ns);
        for (int ch = 0; ch < nch; ++ch) {
            // block (b,a) of the upper triangle, b < a, is read by a stage when it neighbours
            // an evaluated block: some neighbour of b is >= a, or one of a is <= b
            const int* nb = nbr.data() + d.nbroff + (ch == 2 ? ns * z : 0);
            std::vector<int> lo(ns), hi(ns);
            for (int q = 0; q < ns; ++q) {
                lo[q] = hi[q] = q;
                for (int u = 0; u < z; ++u)
                    if (nb[q * z + u] >= 0) {
                        lo[q] = std::min(lo[q], nb[q * z + u]);
                        hi[q] = std::max(hi[q], nb[q * z + u]);
                    }
            }
            const int per = hub_tile_per_item(ns, per_item[cl]);
            const size_t first = tiles.size();
            for (int i = 0; i < ns; ++i)
                for (int k = 0; k <= i; ++k)
                    tiles.push_back(i | k << 8 | ch << 16 | (hi[k] >= i || lo[i] <= k ? TW_NEED : 0));
            for (size_t t0 = first; t0 < tiles.size(); t0 += per) {
                const size_t t1 = std::min(tiles.size(), t0 + per);
                items[form].push_back({cl, (int)t0, (int)t1});
                cost[form].push_back((long long)(t1 - t0) * ns * ns);
            }
            const std::pair<int, int> shape(per, ns);
            if (form == 1 && std::find(H.tile_shapes.begin(), H.tile_shapes.end(), shape) == H.tile_shapes.end())
                H.tile_shapes.push_back(shape);
        }
        g1[form].push_back({cl, -1, -1});
    }
    // contiguous ranges per XCD: a block's i- and k-neighbours lie mostly in its range
    // (8x8 SOA 207 us; round-robin 222, ranges of 8x8 patches of blocks 214)
    work = xcd_order(items[0], cost[0], g1[0]);
    const std::vector<WorkItem> packed = xcd_order(items[1], cost[1], g1[1]);
    H.ntrow = (int)work.size();
    H.ntpack = (int)packed.size();
    work.insert(work.end(), packed.begin(), packed.end());
}

int hub_tile_diags(const g1g2_ctx* c) {
    switch (c->d.selfenergy) {
        case G1G2_TPP: return n_tdiag(SE_TPP);
        case G1G2_TPH: return n_tdiag(SE_TPH);
        case G1G2_GW: return n_tdiag(SE_GW);
        case G1G2_DSL: return n_tdiag(SE_DSL);
        default: return n_tdiag(SE_SOA);
    }
}

// G2 has to be symmetric bit for bit: what it lacks would be dropped.  Nothing of G1
// is dropped but the part of its asymmetry that enters the slopes, so that G1 may be
// anti-Hermitian to the rounding of its largest element (occupations formed as matrix
// products are to 2^-52), below the rounding of the source's own products.
g1g2_status hub_check_state(g1g2_ctx* c) {
    HubbardData& H = c->hub;
    c->herm = false;   // a state that is not checked does not take the triangle
    if (!H.tiles) return G1G2_OK;
    StageArgs s = hub_make_stage(c, 0.0, c->y, c->y, c->y, c->y, 0.0, 0.0);
    s.work = H.twork;
    HIP_OK(c, hipMemsetAsync(H.tsym, 0, 4 * sizeof(unsigned long long), c->stream));
    hipLaunchKernelGGL(hub_herm_kernel, dim3(H.ntrow + H.ntpack), dim3(256), 0, c->stream, s, H.tiles, H.tsym);
    HIP_OK(c, hipGetLastError());
    double r[4];
    HIP_OK(c, hipMemcpyAsync(r, H.tsym, sizeof(r), hipMemcpyDeviceToHost, c->stream));
    HIP_OK(c, hipStreamSynchronize(c->stream));
    // a NaN difference compares false
    c->herm = r[0] == 0.0 && r[2] <= 0x1p-51 * r[3];
    return G1G2_OK;
}

bool hub_tile_ok(const g1g2_ctx* c) { return c->d.basis == G1G2_HUBBARD && c->hub.tiles && c->herm; }

g1g2_status hub_tile_stage(g1g2_ctx* c, int mode, double t, const Regs& in, const Regs& y, const Regs& y2,
                           const Regs& y3, const Regs& acc, const Regs& out, double cb, double cc, bool full) {
    HubbardData& H = c->hub;
    StageArgs s = hub_make_stage(c, t, in, y, acc, out, cb, cc);
    s.work = H.twork;
    const TileArgs ta{H.tiles, H.diag, y2.g1, y3.g1, y2.g2, y3.g2, full ? 1 : 0};
    switch (mode) {
        case RK_FIRST: launch_tile_se<RK_FIRST>(c, s, ta); break;
        case RK_MID: launch_tile_se<RK_MID>(c, s, ta); break;
        default: launch_tile_se<RK_LAST>(c, s, ta); break;
    }
    HIP_OK(c, hipGetLastError());
    prof_mark(c, "hub_tile");
    return G1G2_OK;
}

// One step from y to out (which may be y), with stage registers Y2, Y3 and a third one: Y4 (binary64) or
// the running sum (mixed, where y4 may alias y2).
g1g2_status hub_tile_step(g1g2_ctx* c, double t, double dt, const Regs& y, const Regs& out, const Regs& y2,
                          const Regs& y3, const Regs& y4, const Regs& acc, bool full, bool last) {
    const bool mixed = c->d.precision == G1G2_MIXED;
    g1g2_status s;
    if ((s = hub_tile_stage(c, RK_FIRST, t, y, y, y, y, acc, y2, dt / 6.0, dt / 2.0, full)) != G1G2_OK) return s;
    if ((s = hub_tile_stage(c, RK_MID, t + 0.5 * dt, y2, y, y, y, acc, y3, dt / 3.0, dt / 2.0, full)) != G1G2_OK)
        return s;
    if ((s = hub_tile_stage(c, RK_MID, t + 0.5 * dt, y3, y, y, y, acc, y4, dt / 3.0, dt, full)) != G1G2_OK) return s;
    if (!last) return G1G2_OK;
    return hub_tile_stage(c, RK_LAST, t + dt, y4, y, mixed ? y : y2, mixed ? y : y3, acc, out, dt / 6.0, 0.0, full);
}
