// Polarization and ladder terms of the general basis (Secs. IV.C, V, VI) as
// products of reduced pair maps on the gfx950 matrix cores.
//
// Each term is one (Nb^2 x Nb^2 x Nb^2) complex product of a quasi-Hamiltonian
// and a permuted G2.  The symmetries of w (eq:wsymm_a/b, checked at init), of
// G^< (anti-Hermitian) and of G2 (eq:Gsymm_b) cut its 8 Nb^6 flops:
//
//  * GW (eq:gwpi) and TPH (eq:lambdaph).  With G^> = G^< - i,
//        h^eps_qjpl = i [G^<, M]_jl,  M_sr = w_sqrp,
//        h^ph_ipql = -i [G^<, M]_il,  M_sr = w_spqr
//    (block (p,q) of w), and every factor Z of the two products obeys
//    Z(ki,qp) = conj Z(ik,pq): it maps Hermitian matrices to Hermitian ones.  In
//    the coordinates (Re X_pq, Im X_pq, p < q; X_pp) such a map is a real
//    Nb^2 x Nb^2 matrix, and the product is a real one of 2 Nb^6 flops:
//        R = X Y,   X from G2 (gen_xop), Y from the commutators (gen_comm).
//    The term with its partner is i (Z + Z^T) for the map Z of R; the epilogue
//    of the product turns each 2x2 quad of R into complex elements and adds them
//    into D, so that the combine's D - D^dagger yields term and partner.
//  * TPP (eq:lambdapp).  h^pp = (1 + i (G^< x 1 + 1 x G^<)) w commutes with the
//    exchange of the pair, so the product splits into the exchange-even pairs
//    (Nb (Nb+1)/2) and the odd ones (Nb (Nb-1)/2): a quarter of the flops.
//
// The pairs (p,q), p < q, are numbered t by 8x8 blocks of p and q (table pt): the
// 64 pairs of a block are one edge of an output tile, so that a tile's elements
// form an 8^4 block of D and fill whole 128-byte lines at every index order the
// epilogues write.  Real coordinates are 2t (Re) and
// 2t + 1 (Im), then Nb (Nb-1) + p for (p,p); exchange-even pairs are t, then
// Nb (Nb-1)/2 + p.
//
// TPH and TPP also rest on the exchange symmetry of G2 (eq:Gsymm_a).  G2 is
// split into its exchange-even and -odd parts; where the odd part exceeds
// Nb 2^-54 of the largest element (a state that lacks the symmetry), its product is
// formed too.  Below that bound it is under the rounding of the even product: sums
// of Nb^2 terms of size t round to about 0.4 Nb^2 2^-53 t, and an odd part of that
// size contributes Nb 2^-54 Nb t.  Propagation keeps the symmetry to rounding: the odd
// part reaches 0.5 to 4.5 2^-53 after one step and 1 to 10 after 64 (3 to 64 orbitals,
// bounds 1.5 to 32), so that a long run may cross the bound and then costs the second
// product.  gen_xop measures both on the device and the later kernels of the stage
// read the result, so no synchronization is involved.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "ctx.h"
#include "gen_common.h"

namespace {

enum { K_GW = 0, K_PH = 1, K_PP = 2 };

struct PairTab {
    const int* pt;   // t -> p | q << 16, p < q
    int nb, nbp, nt, ld;
    unsigned long long* stat;   // bits of max |odd part| and max |G2| (nonnegative doubles)
};

__device__ __forceinline__ bool has_odd(const PairTab& tab) {
    const double o = __longlong_as_double((long long)tab.stat[0]);
    const double g = __longlong_as_double((long long)tab.stat[1]);
    return !(o <= tab.nb * 0x1p-54 * g);
}

template <typename T>
struct V2;
template <>
struct V2<double> {
    typedef double2 type;
};
template <>
struct V2<float> {
    typedef float2 type;
};
template <typename T>
__device__ __forceinline__ typename V2<T>::type mk2(double a, double b) {
    return typename V2<T>::type{(T)a, (T)b};
}

// pair number b of a launch over all pairs p <= q
__device__ __forceinline__ void pair_of(const PairTab& tab, int b, int& p, int& q) {
    if (b < tab.nt) {
        const int v = tab.pt[b];
        p = v & 0xffff;
        q = v >> 16;
    } else {
        p = q = b - tab.nt;
    }
}

// --------------------------------------------------------------------------- quasi-Hamiltonians
// One work-group per block (p,q), p <= q (the blocks p > q follow by symmetry),
// and kind.  K_GW / K_PH: C = G^< M - M G^< and the rows of Y of that pair;
// K_PP: H = M + i (G^< M + M G^<^T), M_rs = w_rspq, and the rows (p,q) of its
// even and odd parts, h[pq][ij] (the weight 2 of an unordered pair included).
// Two one-sided products per block of half the blocks; the sandwich forms they
// replace took 0.30 (h^eps) and 0.97 ms (h^pp, h^ph) per Nb = 64 launch.
struct CommArgs {
    const void* w[3];    // blocks of K_GW, K_PH, K_PP
    void* y[2];          // Y of K_GW, K_PH  [ld][ld]
    void* hs;            // K_PP even [lds][lds]
    void* ha;            // K_PP odd  [lda][lda]
    int lds, lda;
    int kind[3];         // kinds of the launch, by blockIdx.y
    double ws;
};

template <typename T, typename S, int NB>
__global__ __launch_bounds__(MainShape<NB>::THREADS) void gen_comm_kernel(CommArgs a, const cd* __restrict__ gl,
                                                                         PairTab tab) {
    typedef MainShape<NB> SH;
    typedef typename V2<T>::type CT;
    constexpr int LD = SH::LD;
    __shared__ T m_re[NB * LD], m_im[NB * LD];
    const int wave = threadIdx.x >> 6, kind = a.kind[blockIdx.y];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 2) tab.stat[threadIdx.x] = 0;
    int p, q;
    pair_of(tab, blockIdx.x, p, q);
    stage_block<T, S, NB>((const S*)a.w[kind] + (size_t)(p * NB + q) * NB * NB, m_re, m_im);
    __syncthreads();
    CAcc<T> acc[SH::TPW];
    T hr[SH::TPW][4], hi[SH::TPW][4];
    auto Gl = [&](int i, int k, T& r, T& m) { ldc(gl + i * NB + k, r, m); };
    auto Mkj = [&](int k, int j, T& r, T& m) {
        r = m_re[k * LD + j];
        m = m_im[k * LD + j];
    };
#pragma unroll
    for (int t = 0; t < SH::TPW; ++t) {
        const int tile = wave * SH::TPW + t, ti = tile / SH::NT, tj = tile % SH::NT;
        acc[t].clear();
        cgemm_tile<T, NB>(acc[t], Gl, Mkj, ti * 16, tj * 16);
        if (kind == K_PP)
            cgemm_tile<T, NB>(acc[t], Mkj, [&](int k, int j, T& r, T& m) { Gl(j, k, r, m); }, ti * 16, tj * 16);
        else
            cgemm_tile<T, NB>(
                acc[t],
                [&](int i, int k, T& r, T& m) {
                    r = -m_re[i * LD + k];
                    m = -m_im[i * LD + k];
                },
                Gl, ti * 16, tj * 16);
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int e = (ti * 16 + tile_row<T>(r4)) * LD + tj * 16 + tile_col();
            hr[t][r4] = kind == K_PP ? m_re[e] - acc[t].im(r4) : acc[t].re(r4);
            hi[t][r4] = kind == K_PP ? m_im[e] + acc[t].re(r4) : acc[t].im(r4);
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < SH::TPW; ++t) {
        const int tile = wave * SH::TPW + t, ti = tile / SH::NT, tj = tile % SH::NT;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int e = (ti * 16 + tile_row<T>(r4)) * LD + tj * 16 + tile_col();
            m_re[e] = (T)a.ws * hr[t][r4];
            m_im[e] = (T)a.ws * hi[t][r4];
        }
    }
    __syncthreads();
    const bool off = p < q;
    if (kind == K_PP) {
        const int row = blockIdx.x;
        CT* hs = (CT*)a.hs + (size_t)row * a.lds;
        CT* ha = (CT*)a.ha + (size_t)row * a.lda;
        for (int t = threadIdx.x; t < tab.nt; t += SH::THREADS) {
            const int v = tab.pt[t], j = v & 0xffff, l = v >> 16;
            const T ar = m_re[j * LD + l], ai = m_im[j * LD + l], br = m_re[l * LD + j], bi = m_im[l * LD + j];
            hs[t] = off ? CT{ar + br, ai + bi} : CT{ar, ai};
            if (off) ha[t] = CT{ar - br, ai - bi};
        }
        const T two = off ? (T)2 : (T)1;
        for (int j = threadIdx.x; j < tab.nb; j += SH::THREADS)
            hs[tab.nt + j] = CT{two * m_re[j * LD + j], two * m_im[j * LD + j]};
        return;
    }
    const int row = off ? 2 * blockIdx.x : 2 * tab.nt + p;
    const T sr = kind == K_GW ? (T)1 : (T)-1;
    T* y0 = (T*)a.y[kind] + (size_t)row * tab.ld;
    T* y1 = y0 + tab.ld;
    for (int t = threadIdx.x; t < tab.nt; t += SH::THREADS) {
        const int v = tab.pt[t], j = v & 0xffff, l = v >> 16;
        const T ar = m_re[j * LD + l], ai = m_im[j * LD + l], br = m_re[l * LD + j], bi = m_im[l * LD + j];
        *(CT*)(y0 + 2 * t) = CT{sr * (ar + br), sr * (ai - bi)};
        if (off) *(CT*)(y1 + 2 * t) = CT{ai + bi, br - ar};
    }
    for (int j = threadIdx.x; j < tab.nb; j += SH::THREADS) {
        y0[2 * tab.nt + j] = sr * m_re[j * LD + j];
        if (off) y1[2 * tab.nt + j] = m_im[j * LD + j];
    }
}

// --------------------------------------------------------------------------- G2 operands
// One work-group per pair (i,k), i <= k, and kind; the block of G2 is staged in
// LDS and its rows of the operand are written contiguously.
//   K_GW: the real map of G2_ipkq, row pair (i,k), column pair (p,q)
//   K_PH: the real map of G2_qjkp, row pair (j,k), column pair (p,q), its Im rows negated
//   K_PP: G2_pqkl, row pair (p,q), column pair (k,l), the even or odd combination
// K_PH and K_PP take the exchange-even part of G2, or with ODD the odd one (which
// in K_PH is i times a Hermitian map, and in K_PP has even rows and odd columns
// or the reverse).  Memory bound: G2 is read once (half of it for K_GW) and half
// its bytes are written.
struct XopArgs {
    const cd* g2;
    void* x[2];     // X of K_GW, K_PH [ld][ld]
    void* gs;       // K_PP: even rows [lds][lds], or with ODD [lds][lda]
    void* ga;       // K_PP: odd rows  [lda][lda], or with ODD [lda][lds]
    int lds, lda;
    int kind[3];
};

template <typename T, int NB, bool ODD>
__global__ __launch_bounds__(512) void gen_xop_kernel(XopArgs a, PairTab tab) {
    typedef typename V2<T>::type CT;
    constexpr int LD = NB + 1;
    __shared__ cd e[NB * LD];
    __shared__ double red[2][8];
    if (ODD && !has_odd(tab)) return;
    const int kind = a.kind[blockIdx.y], nb = tab.nb;
    int p0, q0;
    pair_of(tab, blockIdx.x, p0, q0);
    const bool off = p0 < q0;
    const size_t n1 = NB, n2 = NB * NB, n3 = (size_t)NB * NB * NB;
    double omax = 0.0, gmax = 0.0;
    for (int idx = threadIdx.x; idx < nb * NB; idx += 512) {
        const int r = idx / NB, c = idx % NB;
        if (c >= nb) continue;
        size_t src;
        if (kind == K_GW) src = p0 * n3 + r * n2 + q0 * n1 + c;          // [p][q] = G2_ipkq
        else if (kind == K_PH) src = r * n3 + p0 * n2 + q0 * n1 + c;     // [q][p] = G2_qjkp
        else src = p0 * n3 + q0 * n2 + r * n1 + c;                       // [k][l] = G2_pqkl
        e[r * LD + c] = a.g2[src];
    }
    __syncthreads();
    if (kind != K_GW) {
        // the partner block, G2_qkjp (conjugated) or G2_qpkl, transposed onto e
        for (int idx = threadIdx.x; idx < nb * NB; idx += 512) {
            const int r = idx / NB, c = idx % NB;
            if (c >= nb) continue;
            const size_t src = kind == K_PH ? r * n3 + q0 * n2 + p0 * n1 + c : q0 * n3 + p0 * n2 + r * n1 + c;
            cd v = a.g2[src];
            if (kind == K_PH) v.y = -v.y;
            const cd u = e[c * LD + r];
            const cd dif = csub(u, v);
            omax = fmax(omax, fmax(fabs(dif.x), fabs(dif.y)));
            gmax = fmax(gmax, fmax(fabs(u.x), fabs(u.y)));
            e[c * LD + r] = ODD ? cmk(0.5 * dif.x, 0.5 * dif.y) : cmk(0.5 * (u.x + v.x), 0.5 * (u.y + v.y));
        }
        if (!ODD) {   // largest odd and overall element of the work-group (NaN compares false: kept out)
            for (int o = 32; o > 0; o >>= 1) {
                omax = fmax(omax, __shfl_xor(omax, o, 64));
                gmax = fmax(gmax, __shfl_xor(gmax, o, 64));
            }
            if ((threadIdx.x & 63) == 0) {
                red[0][threadIdx.x >> 6] = omax;
                red[1][threadIdx.x >> 6] = gmax;
            }
        }
        __syncthreads();
        if (!ODD && threadIdx.x < 2) {
            double m = 0.0;
            for (int w = 0; w < 8; ++w) m = fmax(m, red[threadIdx.x][w]);
            if (threadIdx.x == 0) m *= 0.5;
            const unsigned long long b = (unsigned long long)__double_as_longlong(m);
            unsigned long long* s = tab.stat + threadIdx.x;
            if (b > __atomic_load_n(s, __ATOMIC_RELAXED)) atomicMax(s, b);
        }
    }
    if (kind == K_PP) {
        const int row = blockIdx.x;
        const int ldp = ODD ? a.lda : a.lds, ldm = ODD ? a.lds : a.lda;
        CT* gs = (CT*)a.gs + (size_t)row * ldp;
        CT* ga = (CT*)a.ga + (size_t)row * ldm;
        for (int t = threadIdx.x; t < tab.nt; t += 512) {
            const int v = tab.pt[t], k = v & 0xffff, l = v >> 16;
            const cd u = e[k * LD + l], w = e[l * LD + k];
            const cd pl = cscale(cadd(u, w), 0.5), mi = cscale(csub(u, w), 0.5);
            gs[t] = ODD ? mk2<T>(mi.x, mi.y) : mk2<T>(pl.x, pl.y);
            if (off) ga[t] = ODD ? mk2<T>(pl.x, pl.y) : mk2<T>(mi.x, mi.y);
        }
        for (int k = threadIdx.x; k < nb; k += 512) {
            const cd u = e[k * LD + k];
            if (!ODD) gs[tab.nt + k] = mk2<T>(u.x, u.y);
            else if (off) ga[tab.nt + k] = mk2<T>(u.x, u.y);
        }
        return;
    }
    // the odd part of K_PH is i b', b' = -i e a Hermitian map
    auto at = [&](int r, int c) {
        const cd v = e[r * LD + c];
        return kind == K_PH && ODD ? cmul_mi(v) : v;
    };
    const int row = off ? 2 * blockIdx.x : 2 * tab.nt + p0;
    T* x0 = (T*)a.x[kind] + (size_t)row * tab.ld;
    T* x1 = x0 + tab.ld;
    for (int t = threadIdx.x; t < tab.nt; t += 512) {
        const int v = tab.pt[t], p = v & 0xffff, q = v >> 16;
        if (kind == K_GW) {
            const cd u = at(p, q), w = at(q, p);
            const double wt = off ? 2.0 : 1.0;
            *(CT*)(x0 + 2 * t) = mk2<T>(wt * (u.x + w.x), wt * (w.y - u.y));
            if (off) *(CT*)(x1 + 2 * t) = mk2<T>(2.0 * (u.y + w.y), 2.0 * (u.x - w.x));
        } else {
            const cd u = at(q, p), w = at(p, q);
            if (off) {
                *(CT*)(x0 + 2 * t) = mk2<T>(2.0 * (u.x + w.x), 2.0 * (u.y - w.y));
                *(CT*)(x1 + 2 * t) = mk2<T>(2.0 * (u.y + w.y), 2.0 * (w.x - u.x));
            } else {
                *(CT*)(x0 + 2 * t) = mk2<T>(2.0 * u.x, 2.0 * u.y);
            }
        }
    }
    for (int p = threadIdx.x; p < nb; p += 512) {
        const cd u = at(p, p);
        x0[2 * tab.nt + p] = (T)(off ? 2.0 * u.x : u.x);
        if (off) x1[2 * tab.nt + p] = (T)(2.0 * u.y);
    }
}

// --------------------------------------------------------------------------- tile order
// Work-group -> tile of a grid of nr x nc tiles: each XCD takes a contiguous
// range of the order, which walks strips of eight tile rows column by column, so
// that the 64 tiles an XCD has in flight share eight row and eight column panels.
__device__ __forceinline__ void tile_order(int b, int nr, int nc, int& r, int& c) {
    const int tot = nr * nc, x = b & 7, per = tot >> 3, rem = tot & 7;
    const int l = x * per + (x < rem ? x : rem) + (b >> 3);
    const int strip = l / (8 * nc), r0 = strip * 8, h = nr - r0 < 8 ? nr - r0 : 8, in = l - r0 * nc;
    c = in / h;
    r = r0 + in % h;
}

// --------------------------------------------------------------------------- GW, TPH
// R = X Y, real, with the epilogue that adds the term into D.  Bound by the
// matrix cores: a 128x128 tile per work-group of four waves (64x64 each) reads
// 8 bytes of operands per compute unit and cycle, and two work-groups per
// compute unit cover each other's barriers.  Products too small to give every
// compute unit a 128x128 tile take 64x64 tiles, as does binary32, whose
// accumulators are added in binary64 every 64 K.
// ODD is the product with the exchange-odd part of G2 (K_PH).
template <typename T, int WT>
struct PairLds {
    static constexpr int TILE = 32 * WT, KS = 16;
    static constexpr int VN = WT == 1 ? 2 : 16 / sizeof(T);   // values per load
    static constexpr int LDA = KS + VN, LDB = TILE + 16;
    static constexpr int STAGE = 2 * (TILE * LDA + KS * LDB);
    static constexpr int EPI = 4 * 16 * 17 * (int)(sizeof(double) / sizeof(T));
    static constexpr int SIZE = STAGE > EPI ? STAGE : EPI;
};

template <typename T, int WT, int KIND, bool ODD>
__device__ __forceinline__ void pair_tile(const T* __restrict__ X, const T* __restrict__ Y, cd* __restrict__ D,
                                          double* __restrict__ dd, const PairTab& tab, int ntile, T* lds) {
    typedef PairLds<T, WT> L;
    constexpr int TILE = L::TILE, KS = L::KS, VN = L::VN, LDA = L::LDA, LDB = L::LDB;
    constexpr int PER = TILE * KS / (VN * 256);
    constexpr bool F32 = sizeof(T) == 4;
    typedef T V __attribute__((ext_vector_type(VN)));
    T* const as = lds;
    T* const bs = lds + 2 * TILE * LDA;
    int tr, tc;
    tile_order(blockIdx.x, ntile, ntile, tr, tc);
    const int bm = tr * TILE, bn = tc * TILE;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int wm = (wave >> 1) * (TILE / 2), wn = (wave & 1) * (TILE / 2);
    const int noff = 2 * tab.nt, n2 = noff + tab.nb, kend = (n2 + KS - 1) / KS * KS;
    const size_t ld = tab.ld;
    typename MF<T>::acc acc[WT][WT];
    double accd[F32 ? WT : 1][F32 ? WT : 1][4];
#pragma unroll
    for (int a = 0; a < WT; ++a)
#pragma unroll
        for (int b = 0; b < WT; ++b) {
            acc[a][b] = MF<T>::zero();
            if (F32)
                for (int r4 = 0; r4 < 4; ++r4) accd[a][b][r4] = 0.0;
        }
    V pa[PER], pb[PER];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int idx = threadIdx.x + u * 256;
            pa[u] = *(const V*)(X + (size_t)(bm + idx / (KS / VN)) * ld + k0 + idx % (KS / VN) * VN);
            pb[u] = *(const V*)(Y + (size_t)(k0 + idx / (TILE / VN)) * ld + bn + idx % (TILE / VN) * VN);
        }
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int idx = threadIdx.x + u * 256;
            *(V*)(as + buf * TILE * LDA + idx / (KS / VN) * LDA + idx % (KS / VN) * VN) = pa[u];
            *(V*)(bs + buf * KS * LDB + idx / (TILE / VN) * LDB + idx % (TILE / VN) * VN) = pb[u];
        }
    };
    fetch(0);
    __syncthreads();   // an earlier product's epilogue has left the LDS
    put(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < kend; k0 += KS, buf ^= 1) {
        const bool more = k0 + KS < kend;
        if (more) fetch(k0 + KS);
        const T* const ab = as + buf * TILE * LDA + (wm + li) * LDA + lk;
        const T* const bb = bs + buf * KS * LDB + lk * LDB + wn + li;
#pragma unroll
        for (int k4 = 0; k4 < KS; k4 += 4) {
            T av[WT], bv[WT];
#pragma unroll
            for (int a = 0; a < WT; ++a) av[a] = ab[a * 16 * LDA + k4];
#pragma unroll
            for (int b = 0; b < WT; ++b) bv[b] = bb[k4 * LDB + b * 16];
#pragma unroll
            for (int a = 0; a < WT; ++a)
#pragma unroll
                for (int b = 0; b < WT; ++b) acc[a][b] = MF<T>::mac(av[a], bv[b], acc[a][b]);
        }
        if (F32 && ((k0 + KS) % 64 == 0 || !more)) {
#pragma unroll
            for (int a = 0; a < WT; ++a)
#pragma unroll
                for (int b = 0; b < WT; ++b) {
                    for (int r4 = 0; r4 < 4; ++r4) accd[a][b][r4] += (double)acc[a][b][r4];
                    acc[a][b] = MF<T>::zero();
                }
        }
        if (more) put(buf ^ 1);
        __syncthreads();
    }
    // Epilogue, one 16x16 tile at a time through LDS; a lane takes one 2x2 quad.
    // r(A,B) and r(A,B~) (B~ the swapped pair) are the map's elements of row pair
    // A and column pair B.  The element of D - D^dagger at slot (A,B), slot =
    // [a1 b1][a2 b2] for GW and [a1 b1][b2 a2] for TPH, is i (r(A,B) + r(B,A)), for
    // the odd part r(A,B) - r(B,A), and equals the one at (B,A) up to that sign;
    // the quads (A,B) and (B,A) put their shares into slots that no other quad
    // writes: the quad of the later row pair into the slots themselves, the other
    // one into their Hermitian partners, where -conj of the share belongs.
    // The loads of a quad's four slots are issued together: one memory latency per
    // 16x16 tile.
    double* const ep = (double*)lds + wave * 16 * 17;
    const size_t n1 = tab.nbp;
    const int qr = 2 * (lane >> 3), qc = 2 * (lane & 7);
    int prow[WT], pcol[WT];
#pragma unroll
    for (int a = 0; a < WT; ++a) {
        const int r = bm + wm + a * 16 + qr, c = bn + wn + a * 16 + qc;
        prow[a] = r < noff ? tab.pt[r >> 1] : 0;
        pcol[a] = c < noff ? tab.pt[c >> 1] : 0;
    }
#pragma unroll
    for (int a = 0; a < WT; ++a)
#pragma unroll
        for (int b = 0; b < WT; ++b) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                ep[tile_row<T>(r4) * 17 + tile_col()] = F32 ? accd[F32 ? a : 0][F32 ? b : 0][r4] : (double)acc[a][b][r4];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // one wave's LDS accesses stay in order
            __builtin_amdgcn_wave_barrier();
            const double r00 = ep[qr * 17 + qc], r01 = ep[qr * 17 + qc + 1];
            const double r10 = ep[(qr + 1) * 17 + qc], r11 = ep[(qr + 1) * 17 + qc + 1];
            const int row = bm + wm + a * 16 + qr, col = bn + wn + b * 16 + qc;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (row >= n2 || col >= n2) continue;
            size_t slot[4];
            cd val[4];
            bool use[4] = {false, false, false, false};
            auto set = [&](int k, int a1, int a2, int b1, int b2, double vr, double vi) {
                slot[k] = KIND == K_GW ? ((a1 * n1 + b1) * n1 + a2) * n1 + b2 : ((a1 * n1 + b1) * n1 + b2) * n1 + a2;
                val[k] = cmk(vr, vi);
                use[k] = true;
            };
            // share c r of an element r: i r (even), r and -r for the two slots (odd)
            auto c1 = [&](double x, double y) { return ODD ? cmk(x, y) : cmk(-y, x); };
            auto c2 = [&](double x, double y) { return ODD ? cmk(-x, -y) : cmk(-y, x); };
            if (row < noff && col < noff) {
                const int va = prow[a], vb = pcol[b];
                const int a1 = va & 0xffff, a2 = va >> 16, b1 = vb & 0xffff, b2 = vb >> 16;
                const double xr = 0.25 * (r00 - r11), xi = 0.25 * (r10 + r01);
                const double yr = 0.25 * (r00 + r11), yi = 0.25 * (r10 - r01);
                const cd s1 = c1(xr, xi), s2 = c2(xr, xi), t1 = c1(yr, yi), t2 = c2(yr, yi);
                const bool lo = row < col;   // the Hermitian partners' slots
                if (row != col) {
                    set(0, lo ? b2 : a1, lo ? b1 : a2, lo ? a2 : b1, lo ? a1 : b2, lo ? -s1.x : s1.x, s1.y);
                    set(1, lo ? a2 : b1, lo ? a1 : b2, lo ? b2 : a1, lo ? b1 : a2, lo ? -s2.x : s2.x, s2.y);
                } else {
                    set(0, a1, a2, a1, a2, s1.x + s2.x, s1.y + s2.y);
                }
                set(2, a1, a2, b2, b1, t1.x, t1.y);
                set(3, b2, b1, a1, a2, t2.x, t2.y);
            } else if (row < noff) {          // B = (b,b)
                const int va = prow[a], a1 = va & 0xffff, a2 = va >> 16;
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const int bb = col + y - noff;
                    if (bb >= tab.nb) continue;
                    const double xr = 0.5 * (y ? r01 : r00), xi = 0.5 * (y ? r11 : r10);
                    const cd s1 = c1(xr, xi), s2 = c2(xr, xi);
                    set(2 * y, bb, bb, a2, a1, -s1.x, s1.y);
                    set(2 * y + 1, a2, a1, bb, bb, -s2.x, s2.y);
                }
            } else if (col < noff) {          // A = (a,a)
                const int vb = pcol[b], b1 = vb & 0xffff, b2 = vb >> 16;
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const int aa = row + y - noff;
                    if (aa >= tab.nb) continue;
                    const double xr = 0.5 * (y ? r10 : r00), xi = 0.5 * (y ? r11 : r01);
                    const cd s1 = c1(xr, xi), s2 = c2(xr, xi);
                    set(2 * y, aa, aa, b1, b2, s1.x, s1.y);
                    set(2 * y + 1, b1, b2, aa, aa, s2.x, s2.y);
                }
            } else {
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const int aa = row + (y >> 1) - noff, bb = col + (y & 1) - noff;
                    if (aa >= tab.nb || bb >= tab.nb) continue;
                    const double v = y == 0 ? r00 : y == 1 ? r01 : y == 2 ? r10 : r11;
                    // GW: slot [ab][ab] is its own partner, the combine adds both shares
                    const cd s1 = c1(v, 0.0);
                    if (KIND == K_GW) dd[aa * tab.nb + bb] = v;
                    else set(y, aa, aa, bb, bb, s1.x, s1.y);
                }
            }
            cd d[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (use[k]) d[k] = D[slot[k]];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (use[k]) D[slot[k]] = cadd(d[k], val[k]);
        }
}

// The odd product follows in the same work-group (64x64 tiles) or, ODD, as a
// launch of its own: both bodies in one 128x128 kernel exceed the registers.
template <typename T, int WT, int KIND, bool ODD = false>
__global__ __launch_bounds__(256, 2) void gen_pair_gemm_kernel(const T* __restrict__ X, const T* __restrict__ Xodd,
                                                              const T* __restrict__ Y, cd* __restrict__ D,
                                                              double* __restrict__ dd, PairTab tab, int ntile) {
    __shared__ __attribute__((aligned(16))) T lds[PairLds<T, WT>::SIZE];
    if constexpr (!ODD) pair_tile<T, WT, KIND, false>(X, Y, D, dd, tab, ntile, lds);
    if constexpr (KIND == K_PH && (ODD || WT <= 2))
        if (has_odd(tab)) pair_tile<T, WT, KIND, true>(Xodd, Y, D, dd, tab, ntile, lds);
}

// --------------------------------------------------------------------------- TPP
// Lambda of one exchange sector of the left pair, A^T B with A = h[K][rows] and
// B = G2[K][cols], complex.  Products that give every compute unit a 64x64 tile:
// four waves of 32x32, K staged in slices of 16.  A complex multiply-add takes three real products,
//   Re = Ar Br - Ai Bi,  Im = (Ar + Ai)(Br + Bi) - Ar Br - Ai Bi,
// the operand sums formed in registers.  Slices are kept as interleaved complex
// values, so an operand pair is one LDS access; two work-groups per compute unit.
// With T = float the products are accumulated in binary32 over 64-deep chunks and
// the chunk sums in binary64.  The epilogue adds the element at (ij,kl) to its
// exchange images in D with the signs of the sector: the images of the two
// sectors coincide, so each is a launch of its own.  Where G2 has an
// exchange-odd part, the tile's product with it (whose columns lie in the other
// sector) follows in the same work-group.
template <typename T, bool ODD>
__device__ __forceinline__ void pp_tile(const typename V2<T>::type* __restrict__ A,
                                    const typename V2<T>::type* __restrict__ B, cd* __restrict__ D,
                                    const PairTab& tab, bool even, int nr, int lds, int lda,
                                    typename V2<T>::type (*a_c)[65], typename V2<T>::type (*b_c)[65]) {
    constexpr int W = 2, TILE = 32 * W, KS = 16, PER = TILE * KS / 256;
    const int ns = tab.nt + tab.nb;
    const int ldr = even ? lds : lda;                  // rows and K of this sector
    const int kend = ((even ? ns : tab.nt) + KS - 1) / KS * KS;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int wm = (wave >> 1) * 16 * W, wn = (wave & 1) * 16 * W;
    int tr, tc;
    tile_order(blockIdx.x, nr, lds / TILE, tr, tc);
    const int bm = tr * TILE, bn = tc * TILE;
    const bool ceven = even != ODD;                // sector of the columns
    const int ldb = ceven ? lds : lda, ncol = ceven ? ns : tab.nt;
    if (bn >= ncol) return;
    constexpr bool F32 = sizeof(T) == 4;
    double accd[W][W][2][4];   // binary32 only
    typename MF<T>::acc p1[W][W], p2[W][W], p3[W][W];   // Ar Br, Ai Bi, (Ar + Ai)(Br + Bi)
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) {
            p1[a][b] = p2[a][b] = p3[a][b] = MF<T>::zero();
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) accd[a][b][0][r4] = accd[a][b][1][r4] = 0.0;
        }
    typedef T CV __attribute__((ext_vector_type(2)));
    CV pa[PER], pb[PER];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int idx = threadIdx.x + u * 256, k = idx / TILE, c = idx % TILE;
            pa[u] = *(const CV*)(A + (size_t)(k0 + k) * ldr + bm + c);
            pb[u] = *(const CV*)(B + (size_t)(k0 + k) * ldb + bn + c);
        }
    };
    fetch(0);
    for (int k0 = 0; k0 < kend; k0 += KS) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int idx = threadIdx.x + u * 256;
            *(CV*)&a_c[idx / TILE][idx % TILE] = pa[u];
            *(CV*)&b_c[idx / TILE][idx % TILE] = pb[u];
        }
        __syncthreads();
        if (k0 + KS < kend) fetch(k0 + KS);
        // raised wave priority over the matrix-core work: of the two work-groups of
        // a compute unit the one past its barrier goes first
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int k4 = 0; k4 < KS; k4 += 4) {
            T ar[W], ai[W], as[W], br[W], bi[W], bs[W];
#pragma unroll
            for (int a = 0; a < W; ++a) {
                const CV v = *(const CV*)&a_c[k4 + lk][wm + a * 16 + li];
                ar[a] = v.x;
                ai[a] = v.y;
                as[a] = ar[a] + ai[a];
            }
#pragma unroll
            for (int b = 0; b < W; ++b) {
                const CV v = *(const CV*)&b_c[k4 + lk][wn + b * 16 + li];
                br[b] = v.x;
                bi[b] = v.y;
                bs[b] = br[b] + bi[b];
            }
#pragma unroll
            for (int a = 0; a < W; ++a)
#pragma unroll
                for (int b = 0; b < W; ++b) {
                    p1[a][b] = MF<T>::mac(ar[a], br[b], p1[a][b]);
                    p2[a][b] = MF<T>::mac(ai[a], bi[b], p2[a][b]);
                    p3[a][b] = MF<T>::mac(as[a], bs[b], p3[a][b]);
                }
        }
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        if (F32 && ((k0 + KS) % 64 == 0 || k0 + KS >= kend)) {
#pragma unroll
            for (int a = 0; a < W; ++a)
#pragma unroll
                for (int b = 0; b < W; ++b) {
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const double d1 = p1[a][b][r4], d2 = p2[a][b][r4], d3 = p3[a][b][r4];
                        accd[a][b][0][r4] += d1 - d2;
                        accd[a][b][1][r4] += d3 - d1 - d2;
                    }
                    p1[a][b] = p2[a][b] = p3[a][b] = MF<T>::zero();
                }
        }
    }
    const size_t n1 = tab.nbp;
    const double sr = even ? 1.0 : -1.0, sc = ceven ? 1.0 : -1.0;
    int prow[W][4], pcol[W];   // pairs p | q << 16, -1 outside
    auto pair_at = [&](int x, int nx) {
        int p, q;
        if (x >= nx) return -1;
        pair_of(tab, x, p, q);
        return p | q << 16;
    };
#pragma unroll
    for (int a = 0; a < W; ++a) {
        pcol[a] = pair_at(bn + wn + a * 16 + tile_col(), ncol);
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) prow[a][r4] = pair_at(bm + wm + a * 16 + tile_row<T>(r4), even ? ns : tab.nt);
    }
    const double sg[4] = {1.0, sr, sc, sr * sc};
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) {
            // the exchange images of four elements, their loads issued together
            cd d[4][4];
            size_t x[4][4];
            bool use[4][4];
            const int k = pcol[b] & 0xffff, l = pcol[b] >> 16;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int i = prow[a][r4] & 0xffff, j = prow[a][r4] >> 16;
                const bool in = pcol[b] >= 0 && prow[a][r4] >= 0;
                x[r4][0] = ((i * n1 + j) * n1 + k) * n1 + l;
                x[r4][1] = ((j * n1 + i) * n1 + k) * n1 + l;
                x[r4][2] = ((i * n1 + j) * n1 + l) * n1 + k;
                x[r4][3] = ((j * n1 + i) * n1 + l) * n1 + k;
                use[r4][0] = in;
                use[r4][1] = in && i != j;
                use[r4][2] = in && k != l;
                use[r4][3] = in && i != j && k != l;
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    if (use[r4][m]) d[r4][m] = D[x[r4][m]];
            }
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const double vr = F32 ? accd[a][b][0][r4] : (double)(p1[a][b][r4] - p2[a][b][r4]);
                const double vi = F32 ? accd[a][b][1][r4] : (double)(p3[a][b][r4] - p1[a][b][r4] - p2[a][b][r4]);
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    if (use[r4][m]) D[x[r4][m]] = cmk(d[r4][m].x + sg[m] * vr, d[r4][m].y + sg[m] * vi);
            }
        }
}

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void gen_gemm_kernel(const typename V2<T>::type* __restrict__ A, const typename V2<T>::type* __restrict__ B,
                     const typename V2<T>::type* __restrict__ Bodd, cd* __restrict__ D, PairTab tab, bool even,
                     int nr, int lds, int lda) {
    __shared__ typename V2<T>::type a_c[16][65], b_c[16][65];
    pp_tile<T, false>(A, B, D, tab, even, nr, lds, lda, a_c, b_c);
    if (has_odd(tab)) pp_tile<T, true>(A, Bodd, D, tab, even, nr, lds, lda, a_c, b_c);
}

// Smaller products: 32x32 tiles of the pairs (t, t'), all four products of a tile at
// once.  The even and the odd sector number their pairs p < q alike, so that a tile
// of one and the same tile of the other share their exchange images in D, and one
// work-group owns them: group g of four waves takes the product g of
//   0: even rows, even columns   1: odd, odd   2: even, odd   3: odd, even
// (2 and 3 where G2 has an exchange-odd part), the results meet in LDS, and a thread
// adds one element's combinations into its four images.  Such a product is bound by the
// chain of its K slices on few compute units, so the products of a tile run beside
// each other.  Per stage, in us, against a launch per sector whose work-groups take
// the odd product after the even one: 16 orbitals 19 (30 there) in binary64, 26 (49) with
// the odd part, 21 (44) in mixed precision, which always has one; 32 orbitals 78 (84),
// 127 (154) and 87 (115).  64 registers and 67 KB of LDS (slices of 8 in binary64, 16 in
// binary32, two buffers) leave two work-groups per compute unit: at 32 orbitals there are
// 289; one per compute unit took 86, 138 and 99 us.
template <typename T>
struct PpSmall {
    typedef typename V2<T>::type CT;
    const CT *hs, *ha;            // h^pp [lds][lds], [lda][lda]
    const CT *gs, *ga, *gso, *gao;   // G2 [lds][lds], [lda][lda], [lds][lda], [lda][lds]
};

template <typename T>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void gen_pp_small_kernel(PpSmall<T> s, cd* __restrict__ D, PairTab tab, int nr,
                                                           int lds, int lda) {
    typedef typename V2<T>::type CT;
    typedef T CV __attribute__((ext_vector_type(2)));
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int TILE = 32, KS = F32 ? 16 : 8, LD = TILE + 1, PER = TILE * KS / 256, BUF = 2;
    // the slices of A and B per group, or the four results
    constexpr int STAGE = 4 * BUF * 2 * KS * LD, EPI = 4 * TILE * LD * (int)(sizeof(cd) / sizeof(CT));
    __shared__ __attribute__((aligned(16))) CT buf[STAGE > EPI ? STAGE : EPI];
    const bool odd = has_odd(tab);
    const int ns = tab.nt + tab.nb;
    const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), tid = threadIdx.x & 255;
    const int wave = tid >> 6, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wm = (wave >> 1) * 16, wn = (wave & 1) * 16;
    int tr, tc;
    tile_order(blockIdx.x, nr, nr, tr, tc);
    const int bm = tr * TILE, bn = tc * TILE;
    const bool reven = g == 0 || g == 2, ceven = g == 0 || g == 3;
    const CT* const A = reven ? s.hs : s.ha;
    const CT* const B = g == 0 ? s.gs : g == 1 ? s.ga : g == 2 ? s.gso : s.gao;
    const int ldr = reven ? lds : lda, ldb = ceven ? lds : lda;
    // odd sectors end at nt pairs; lda covers every tile that begins before that
    const bool on = (reven || bm < tab.nt) && (ceven || bn < tab.nt) && (g < 2 || odd);
    const int kend = on ? ((reven ? ns : tab.nt) + KS - 1) / KS * KS : 0, kall = (ns + KS - 1) / KS * KS;
    typename MF<T>::acc p1 = MF<T>::zero(), p2 = MF<T>::zero(), p3 = MF<T>::zero();
    double re[4] = {0, 0, 0, 0}, im[4] = {0, 0, 0, 0};
    CV pa[PER], pb[PER];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int idx = tid + u * 256, k = idx / TILE, c = idx % TILE;
            pa[u] = *(const CV*)(A + (size_t)(k0 + k) * ldr + bm + c);
            pb[u] = *(const CV*)(B + (size_t)(k0 + k) * ldb + bn + c);
        }
    };
    auto flush = [&]() {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const double d1 = p1[r4], d2 = p2[r4], d3 = p3[r4];
            re[r4] += d1 - d2;
            im[r4] += d3 - d1 - d2;
        }
        p1 = p2 = p3 = MF<T>::zero();
    };
    if (kend > 0) fetch(0);
    for (int k0 = 0; k0 < kall; k0 += KS) {
        CT* const as = buf + (k0 / KS % BUF * 4 + g) * 2 * KS * LD;
        CT* const bs = as + KS * LD;
        if (k0 < kend)
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int idx = tid + u * 256;
                *(CV*)(as + idx / TILE * LD + idx % TILE) = pa[u];
                *(CV*)(bs + idx / TILE * LD + idx % TILE) = pb[u];
            }
        __syncthreads();
        if (k0 + KS < kend) fetch(k0 + KS);
        if (k0 < kend)
#pragma unroll
        for (int k4 = 0; k4 < KS; k4 += 4) {
            const CV a = *(const CV*)(as + (k4 + lk) * LD + wm + li), b = *(const CV*)(bs + (k4 + lk) * LD + wn + li);
            p1 = MF<T>::mac(a.x, b.x, p1);
            p2 = MF<T>::mac(a.y, b.y, p2);
            p3 = MF<T>::mac(a.x + a.y, b.x + b.y, p3);
        }
        if (F32 && (k0 + KS) % 64 == 0) flush();
        if (BUF == 1) __syncthreads();
    }
    flush();
    __syncthreads();
    cd* const res = (cd*)buf;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
        res[(g * TILE + wm + tile_row<T>(r4)) * LD + wn + tile_col()] = cmk(re[r4], im[r4]);
    __syncthreads();
    const int r = threadIdx.x / TILE, c = threadIdx.x % TILE, row = bm + r, col = bn + c;
    if (row >= ns || col >= ns) return;
    int i, j, k, l;
    pair_of(tab, row, i, j);
    pair_of(tab, col, k, l);
    const cd ee = res[r * LD + c], oo = res[(TILE + r) * LD + c];
    const cd eo = res[(2 * TILE + r) * LD + c], oe = res[(3 * TILE + r) * LD + c];
    const cd sp = cadd(ee, oo), sm = csub(ee, oo), op = cadd(eo, oe), om = csub(eo, oe);
    const size_t n1 = tab.nbp;
    const size_t x0 = ((i * n1 + j) * n1 + k) * n1 + l, x1 = ((j * n1 + i) * n1 + k) * n1 + l;
    const size_t x2 = ((i * n1 + j) * n1 + l) * n1 + k, x3 = ((j * n1 + i) * n1 + l) * n1 + k;
    const bool u1 = i != j, u2 = k != l;
    const cd z = cmk(0.0, 0.0);
    const cd d0 = D[x0], d1 = u1 ? D[x1] : z, d2 = u2 ? D[x2] : z, d3 = u1 && u2 ? D[x3] : z;
    D[x0] = cadd(d0, cadd(sp, op));
    if (u1) D[x1] = cadd(d1, cadd(sm, om));
    if (u2) D[x2] = cadd(d2, csub(sm, om));
    if (u1 && u2) D[x3] = cadd(d3, csub(sp, op));
}

// --------------------------------------------------------------------------- host side
int round_up(int v, int m) { return (v + m - 1) / m * m; }

// Tile edges by size: the largest whose tiles give each of the 256 compute units
// one.  With fewer tiles than that the product is bound by the K loop of a
// work-group, which is proportional to the tile's area.
int tiles(int n, int edge) { return round_up(n, edge) / edge; }
bool fills(int n, int edge) { return tiles(n, edge) * tiles(n, edge) >= 256; }

template <typename T, typename S, int NB>
g1g2_status pair_run(g1g2_ctx* c, const Regs& in, double ws) {
    GeneralData& g = c->gen;
    typedef typename V2<T>::type CT;
    const bool mixed = sizeof(T) == 4;
    const int se = c->d.selfenergy;
    const bool gw = se == G1G2_GW || se == G1G2_DSL, pp = se == G1G2_TPP || se == G1G2_DSL,
               ph = se == G1G2_TPH || se == G1G2_DSL;
    const int nt = g.nb * (g.nb - 1) / 2, n2 = g.nb * g.nb, npair = nt + g.nb;
    const PairTab tab{g.pt, g.nb, g.nbp, nt, g.pld, g.pstat};
    CommArgs ca{};
    XopArgs xa{};
    int nk = 0;
    for (int k : {K_GW, K_PH, K_PP})
        if (k == K_GW ? gw : k == K_PH ? ph : pp) {
            ca.kind[nk] = xa.kind[nk] = k;
            ++nk;
        }
    ca.w[K_GW] = mixed ? (void*)g.w_gw32 : (void*)g.w_gw;
    ca.w[K_PH] = mixed ? (void*)g.w_ph32 : (void*)g.w_ph;
    ca.w[K_PP] = mixed ? (void*)g.w_pp32 : (void*)g.w_pp;
    for (int k = 0; k < 2; ++k) {
        ca.y[k] = g.py[k];
        xa.x[k] = g.px[k];
    }
    ca.hs = g.phs;
    ca.ha = g.pha;
    xa.g2 = in.g2;
    xa.gs = g.pgs;
    xa.ga = g.pga;
    ca.lds = xa.lds = g.plds;
    ca.lda = xa.lda = g.plda;
    ca.ws = ws;
    hipLaunchKernelGGL((gen_comm_kernel<T, S, NB>), dim3(npair, nk), dim3(MainShape<NB>::THREADS), 0, c->stream, ca,
                       in.g1, tab);
    HIP_OK(c, hipGetLastError());
    prof_mark(c, "gen_comm");
    hipLaunchKernelGGL((gen_xop_kernel<T, NB, false>), dim3(npair, nk), dim3(512), 0, c->stream, xa, tab);
    HIP_OK(c, hipGetLastError());
    prof_mark(c, "gen_xop");
    if (pp || ph) {   // the exchange-odd parts, into buffers of their own
        XopArgs xo = xa;
        int no = 0;
        for (int k : {K_PH, K_PP})
            if (k == K_PH ? ph : pp) xo.kind[no++] = k;
        xo.x[K_PH] = g.pxo;
        xo.gs = g.pgso;
        xo.ga = g.pgao;
        hipLaunchKernelGGL((gen_xop_kernel<T, NB, true>), dim3(npair, no), dim3(512), 0, c->stream, xo, tab);
        HIP_OK(c, hipGetLastError());
        prof_mark(c, "gen_xop_odd");
    }
    cd* const D = g.dmat;
    auto product = [&](auto kind) -> g1g2_status {
        constexpr int KIND = decltype(kind)::value;
        const T *x = (const T*)g.px[KIND], *xo = (const T*)g.pxo, *y = (const T*)g.py[KIND];
        auto launch = [&](auto wt, auto odd) -> g1g2_status {
            constexpr int WT = decltype(wt)::value;
            constexpr bool ODD = decltype(odd)::value;
            const int n = tiles(n2, 32 * WT);
            hipLaunchKernelGGL((gen_pair_gemm_kernel<T, WT, KIND, ODD>), dim3(n * n), dim3(256), 0, c->stream, x, xo, y,
                               D, g.pdd, tab, n);
            HIP_OK(c, hipGetLastError());
            prof_mark(c, ODD ? "gen_pair_gemm_odd" : "gen_pair_gemm");
            return G1G2_OK;
        };
        typedef std::integral_constant<bool, false> both;
        if constexpr (sizeof(T) == 8) {
            if (fills(n2, 128)) {
                const g1g2_status s = launch(std::integral_constant<int, 4>(), both());
                if constexpr (KIND == K_PH)
                    return s != G1G2_OK ? s
                                        : launch(std::integral_constant<int, 4>(), std::integral_constant<bool, true>());
                return s;
            }
        }
        if (fills(n2, 64)) return launch(std::integral_constant<int, 2>(), both());
        return launch(std::integral_constant<int, 1>(), both());
    };
    g1g2_status s;
    if (gw && (s = product(std::integral_constant<int, K_GW>())) != G1G2_OK) return s;
    if (ph && (s = product(std::integral_constant<int, K_PH>())) != G1G2_OK) return s;
    if (pp && fills(npair, 64)) {
        for (int even = 1; even >= 0; --even) {
            const int nr = tiles(even ? npair : nt, 64), nc = g.plds / 64;
            hipLaunchKernelGGL((gen_gemm_kernel<T>), dim3(nr * nc), dim3(256), 0, c->stream,
                               (const CT*)(even ? g.phs : g.pha), (const CT*)(even ? g.pgs : g.pga),
                               (const CT*)(even ? g.pgso : g.pgao), D, tab, even != 0, nr, g.plds, g.plda);
            HIP_OK(c, hipGetLastError());
            prof_mark(c, "gen_gemm");
        }
    } else if (pp) {
        const int nr = tiles(npair, 32);
        const PpSmall<T> ps{(const CT*)g.phs, (const CT*)g.pha,  (const CT*)g.pgs,
                            (const CT*)g.pga, (const CT*)g.pgso, (const CT*)g.pgao};
        hipLaunchKernelGGL((gen_pp_small_kernel<T>), dim3(nr * nr), dim3(1024), 0, c->stream, ps, D, tab, nr, g.plds,
                           g.plda);
        HIP_OK(c, hipGetLastError());
        prof_mark(c, "gen_gemm");
    }
    return G1G2_OK;
}

}  // namespace

g1g2_status pair_setup(g1g2_ctx* c, bool gw, bool pp, bool ph) {
    GeneralData& g = c->gen;
    const int nb = g.nb, nt = nb * (nb - 1) / 2, n2 = nb * nb;
    const size_t es = c->d.precision == G1G2_MIXED ? sizeof(float) : sizeof(double);
    std::vector<int> pt;
    const auto block = [&](int p0, int q0) {
        for (int p = p0; p < std::min(nb, p0 + 8); ++p)
            for (int q = std::max(q0, p + 1); q < std::min(nb, q0 + 8); ++q) pt.push_back(p | q << 16);
    };
    for (int full = 1; full >= 0; --full)
        for (int p0 = 0; p0 < nb; p0 += 8)
            for (int q0 = p0 + 8; q0 < nb; q0 += 8)
                if ((q0 + 8 <= nb) == (full == 1)) block(p0, q0);
    for (int p0 = 0; p0 < nb; p0 += 8) block(p0, p0);
    pt.push_back(0);
    HIP_OK(c, hipMalloc(&g.pt, pt.size() * sizeof(int)));
    HIP_OK(c, hipMemcpyAsync(g.pt, pt.data(), pt.size() * sizeof(int), hipMemcpyHostToDevice, c->stream));
    HIP_OK(c, hipMalloc(&g.pstat, 2 * sizeof(unsigned long long)));
    HIP_OK(c, hipMalloc(&g.pdd, (size_t)nb * nb * sizeof(double)));
    HIP_OK(c, hipMemsetAsync(g.pdd, 0, (size_t)nb * nb * sizeof(double), c->stream));
    g.pld = round_up(n2, es == sizeof(double) && fills(n2, 128) ? 128 : 64);
    g.plds = round_up(nt + nb, 64);
    g.plda = std::max(64, round_up(nt, 64));
    // the paddings stay zero: K paddings enter the products
    auto get = [&](void** p, size_t bytes) -> g1g2_status {
        HIP_OK(c, hipMalloc(p, bytes));
        HIP_OK(c, hipMemsetAsync(*p, 0, bytes, c->stream));
        return G1G2_OK;
    };
    const size_t rr = (size_t)g.pld * g.pld * es;
    const size_t ss = (size_t)g.plds * g.plds * 2 * es, aa = (size_t)g.plda * g.plda * 2 * es,
                 sa = (size_t)g.plds * g.plda * 2 * es;
    g1g2_status s;
    if (gw && ((s = get(&g.px[0], rr)) != G1G2_OK || (s = get(&g.py[0], rr)) != G1G2_OK)) return s;
    if (ph && ((s = get(&g.px[1], rr)) != G1G2_OK || (s = get(&g.py[1], rr)) != G1G2_OK ||
               (s = get(&g.pxo, rr)) != G1G2_OK))
        return s;
    if (pp && ((s = get(&g.phs, ss)) != G1G2_OK || (s = get(&g.pha, aa)) != G1G2_OK ||
               (s = get(&g.pgs, ss)) != G1G2_OK || (s = get(&g.pga, aa)) != G1G2_OK ||
               (s = get(&g.pgso, sa)) != G1G2_OK || (s = get(&g.pgao, sa)) != G1G2_OK))
        return s;
    HIP_OK(c, hipStreamSynchronize(c->stream));
    return G1G2_OK;
}

g1g2_status pair_add(g1g2_ctx* c, const Regs& in, double ws) {
    const bool mixed = c->d.precision == G1G2_MIXED;
    switch (c->gen.nbp) {
        case 16: return mixed ? pair_run<float, float2, 16>(c, in, ws) : pair_run<double, cd, 16>(c, in, ws);
        case 32: return mixed ? pair_run<float, float2, 32>(c, in, ws) : pair_run<double, cd, 32>(c, in, ws);
        case 48: return mixed ? pair_run<float, float2, 48>(c, in, ws) : pair_run<double, cd, 48>(c, in, ws);
        default: return mixed ? pair_run<float, float2, 64>(c, in, ws) : pair_run<double, cd, 64>(c, in, ws);
    }
}

void pair_free(g1g2_ctx* c) {
    GeneralData& g = c->gen;
    void* ptrs[] = {g.pt,    g.pstat, g.pdd, g.px[0], g.px[1], g.py[0], g.py[1], g.pxo,
                    g.phs,   g.pha,   g.pgs, g.pga,   g.pgso,  g.pgao};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
}
