// Discrete adjoint of the RK4 propagation of the driven Hubbard SOA system.
//
// Loss  L = sum_i a_i d_i(T) + sum_i b_i (n^up_ii(T) + n^dn_ii(T)),
// n_ii = Im G^<_ii (n = -i G^<), d_i = n^up_ii n^dn_ii - Re A_iiii.
// Parameters: drive coefficients c_m (through s(t) = sum_m c_m phi_m(t), which
// adds s(t) x_i to the diagonal of h0 for both spins) and U.
//
// Complex cotangents follow zbar = dL/dRe z + i dL/dIm z: for w = M z
// (complex linear) zbar += M^H wbar; for w = a b, abar += conj(b) wbar.
//
// One RK4 step y -> y + dt/6 (k1 + 2 k2 + 2 k3 + k4), k_s = f(Y_s, t_s), is
// reversed as
//   g4 = dt/6 l, m4 = J(Y4)^T g4, g3 = dt/3 l + dt m4, m3 = J(Y3)^T g3,
//   g2 = dt/3 l + dt/2 m3, m2 = J(Y2)^T g2, g1 = dt/6 l + dt/2 m2,
//   m1 = J(Y1)^T g1,  l <- l + m1 + m2 + m3 + m4,
// with y_n checkpointed every K steps; each segment is recomputed forward
// once, keeping y_n and the stage states Y2, Y3, Y4 of every step in device
// memory (four states per step of a segment).  The vector-Jacobian product of
// the right-hand side of eq:g2-hubbard / eq:eom_g1_hubbard is split into
//   adj_slice_red : in one pass over the cotangent, the G2 cotangent
//               (stencil of the commutator applied to the cotangent, plus the
//               collision-integral entries) and five of the six reductions of
//               the source Psi (eq:soa-cubic-scheme) differentiated with
//               respect to X and Y (per-slice partials),
//   adj_lane_red : the sixth reduction, reading contiguous rows,
//   adj_e, adj_g1e, adj_gsum : the G1 cotangents, the diagonal of h^HF,
//               dL/ds and dL/dU.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "ctx.h"
#include "hub_common.h"

using hub::Cl;
using hub::hf_diag;
using hub::make_cl;

namespace {

struct AdjArgs {
    Cl a;                       // stage state (X, Y) and model data
    const void* A;              // stage state G2: binary64, or binary32 (a32) for the
    int a32;                    // mixed-precision stage copies Y2, Y3, Y4
    const cd* gin1;             // cotangent of dG1 (scaled by gscale)
    const cd* gin2;             // cotangent of dG2
    double gscale;
    const cd* lam1;             // lambda (running cotangent of y_n)
    const cd* lam2;
    cd* lacc1;                  // lambda accumulator
    cd* lacc2;
    cd* gnext1;                 // next stage cotangent = alpha lambda + beta mu
    cd* gnext2;
    double alpha, beta;
    int init, has_next;
    cd* red;                    // reduction buffers (see adj_red)
    cd* part;                   // partial sums of the kind-3 lane reduction [nparts][ns][ns][2]
    int pairs_per_part, nparts;
    cd* spart;                  // per-slice partials of kinds 0, 2, 4, 5 [8][ns^3]
    cd* ebar;                   // [2][ns] cotangents of the h^HF diagonals
    double* gpart;              // [2 + blocks of adj_g1e]: partial dL/ds, dL/dU
    double* grads;              // [2]: dL/ds, dL/dU of this stage
};

// reduction buffer layout (each ns^2 complex): RX[6], RY[6], M02, M13, UPART
enum { R_X = 0, R_Y = 6, R_M02 = 12, R_M13 = 13, R_UP = 14, R_N = 15 };

__device__ __forceinline__ cd cmul3(cd a, cd b, cd c) { return cmul(cmul(a, b), c); }

// Element e of the stage state G2 (binary64 arithmetic whatever its storage).
__device__ __forceinline__ cd ld_a(const AdjArgs& s, long long e) {
    return s.a32 ? ld_c(static_cast<const float2*>(s.A), e) : ld_c(static_cast<const cd*>(s.A), e);
}

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ cd wsum(cd v) { return cmk(wsum(v.x), wsum(v.y)); }

// Reductions of the source term (eq:soa-cubic-scheme) differentiated with
// respect to X and Y, B = i gs g the scaled cotangent.  Each kind sums over the
// pair complementary to its free pair:
//   kind 0 free (i,k): X cotangent and M02 = sum conj(A) B
//   kind 1 free (i,j): X and Y cotangents and the U partial Re(conj(Psi/U) B)
//   kind 2 free (j,k), kind 3 free (k,l), kind 4 free (i,l): X and Y cotangents
//   kind 5 free (j,l): Y cotangent and M13 = sum conj(A) B
// Kinds 0, 1, 2, 4 and 5 come from one pass over the cotangent: one work-group
// per (i, j) slice, wave w over the rows k = w, w + ADJ_WAVES, ... with lane = l.
// At fixed (i, j) their weights are products of a factor in k and one in l, so
// the pass forms only the sums over l of a row,
//   s1 = sum conj(Y_jl) B, s2 = sum conj(Y_kl) B, s3 = sum conj(Y_il) B, s4 = sum conj(A) B,
// and the sums over k of a lane,
//   q1 = sum conj(X_lk) B, q2 = sum conj(X_ik) B, q3 = sum conj(X_jk) B, q4 = sum conj(A) B,
// eight complex multiply-adds per element instead of 25, and every kind follows
// from them once per row or lane.  The eight real row sums are reduced together,
// halving the number of values a lane holds in the first three exchanges: 10
// exchanges instead of 48, whose LDS permutes bound the pass.  Kind 1 is summed
// over the slice; kinds 0 and 2 leave partials per (i, j, k) that
// adj_slice_fin_kernel sums over j or i; kinds 4 and 5 partials per (i, j, l).
// Kind 3 is adj_lane_red_kernel.
//
// The same pass computes the G2 cotangent mu = i gs [conj(E) g + hop stencil
// applied to g] + collision entries (the commutator stencil is its own
// adjoint up to the conjugate of the diagonal) and updates the running sum and
// the next stage's cotangent: the l-neighbours of the stencil are other lanes
// (cross-lane permute), the other neighbours whole rows; neighbour tables are
// staged in LDS padded to four entries (a missing neighbour is the site itself
// with hopping 0).
// Four waves: 8x8 sites 473 us per pass, eight 493, and 635 before the sums were
// factored and the loads gathered ahead of the stores (the factored sums alone,
// loads between stores, 750: more waves in flight without more loads only widened
// what the L2 has to hold).
constexpr int ADJ_WAVES = 4;

// Sum of each of eight values over the 64 lanes; lane returns the sum of value
// lane / 8.
__device__ __forceinline__ double wsum8(const double (&v)[8], int lane) {
    double a[4], b[2];
    const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8;
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = (h5 ? v[q + 4] : v[q]) + __shfl_xor(h5 ? v[q] : v[q + 4], 32, 64);
#pragma unroll
    for (int q = 0; q < 2; ++q) b[q] = (h4 ? a[q + 2] : a[q]) + __shfl_xor(h4 ? a[q] : a[q + 2], 16, 64);
    double c = (h3 ? b[1] : b[0]) + __shfl_xor(h3 ? b[0] : b[1], 8, 64);
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    return c;
}

__global__ __launch_bounds__(64 * ADJ_WAVES) void adj_slice_red_kernel(AdjArgs s) {
    constexpr int ZR = 4;
    __shared__ cd sh4[ADJ_WAVES][5][64];   // per wave and lane: q1 .. q4 and the k = l term of q2
    __shared__ double srow[64][8];         // per row k: s1 .. s4
    __shared__ cd sdia[64];                // per row k: B at l = k
    __shared__ cd eu[64], ed[64];
    __shared__ int snb[2 * 64 * ZR];
    __shared__ cd shp[2 * 64 * ZR];
    const Cl& a = s.a;
    const int ns = a.ns, ns2 = ns * ns, ns3 = ns2 * ns, z = a.zmax;
    const int i = blockIdx.x / ns, j = blockIdx.x % ns;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool lane_ok = lane < ns;
    const int l = lane_ok ? lane : 0;
    const cd* X = a.X;
    const cd* Y = a.Y;
    const double U = a.U, gs = s.gscale;
    for (int q = tid; q < ns; q += blockDim.x) {
        eu[q] = hf_diag(a, 0, q);
        ed[q] = hf_diag(a, 1, q);
    }
    for (int q = tid; q < 2 * ns * ZR; q += blockDim.x) {
        const int row = q / ZR, qq = q - row * ZR, site = row % ns;
        const int p = qq < z ? a.nbr[row * z + qq] : -1;
        snb[q] = p >= 0 ? p : site;
        shp[q] = p >= 0 ? a.hop[row * z + qq] : cmk(0.0, 0.0);
    }
    __syncthreads();
    const int* nbu = snb;
    const int* nbd = snb + ns * ZR;
    const cd* hu = shp;
    const cd* hd = shp + ns * ZR;
    const cd* __restrict__ G = s.gin2;
    int src[ZR];
#pragma unroll
    for (int q = 0; q < ZR; ++q) src[q] = lane_ok ? nbd[l * ZR + q] : lane;
    const cd ei = eu[i], ej = ed[j], el = ed[l];
    const cd xij = X[i * ns + j], yji = Y[j * ns + i];
    const cd yjl = Y[j * ns + l], yil = Y[i * ns + l];
    cd q1 = cmk(0, 0), q2 = cmk(0, 0), q3 = cmk(0, 0), q4 = cmk(0, 0), qd = cmk(0, 0);
    cd* P = s.spart;
    for (int k = wave; k < ns; k += ADJ_WAVES) {
        double sv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const int e = ((i * ns + j) * ns + k) * ns + l;
        const cd g = lane_ok ? G[e] : cmk(0.0, 0.0);
        cd vl[ZR];
#pragma unroll
        for (int q = 0; q < ZR; ++q) {
            vl[q].x = __shfl(g.x, src[q], 64);
            vl[q].y = __shfl(g.y, src[q], 64);
        }
        if (lane_ok) {
            // G2 cotangent of this element
            const cd ek = eu[k];
            const cd E = cmk(ei.x + ej.x - ek.x - el.x, ei.y + ej.y - ek.y - el.y);
            cd hsum = cmul(cconj(E), g);
            // every load of the row before its stores
            cd vi[ZR], vj[ZR], vk[ZR];
#pragma unroll
            for (int q = 0; q < ZR; ++q) {
                vi[q] = G[e + (nbu[i * ZR + q] - i) * ns3];
                vj[q] = G[e + (nbd[j * ZR + q] - j) * ns2];
                vk[q] = G[e + (nbu[k * ZR + q] - k) * ns];
            }
            const cd av = ld_a(s, e);
            const cd base = ld_nt(s.init ? s.lam2 + e : s.lacc2 + e);
            const cd lv = s.has_next ? ld_nt(s.lam2 + e) : cmk(0.0, 0.0);
            const cd xkl = X[k * ns + l], ykl = Y[k * ns + l];
#pragma unroll
            for (int q = 0; q < ZR; ++q) {
                hsum = cfma(hsum, hu[i * ZR + q], vi[q]);
                hsum = cfma(hsum, hd[j * ZR + q], vj[q]);
                hsum = csub(hsum, cmul(vk[q], cconj(hu[k * ZR + q])));
                hsum = csub(hsum, cmul(vl[q], cconj(hd[l * ZR + q])));
            }
            cd mu = cscale(cmul_i(hsum), gs);
            if (j == i && l == i) {
                cd bxa = cscale(cmul_i(s.gin1[i * ns + k]), gs), bxb = cscale(cmul_i(s.gin1[k * ns + i]), gs);
                mu = cadd(mu, cscale(cmul_i(cadd(bxa, cconj(bxb))), a.U));
            }
            if (j == i && k == i) {
                const cd* gy = s.gin1 + ns2;
                cd bya = cscale(cmul_i(gy[i * ns + l]), gs), byb = cscale(cmul_i(gy[l * ns + i]), gs);
                mu = cadd(mu, cscale(cmul_i(cadd(bya, cconj(byb))), a.U));
            }
            st_nt(s.lacc2 + e, cadd(base, mu));
            if (s.has_next)
                st_nt(s.gnext2 + e, cmk(s.alpha * lv.x + s.beta * mu.x, s.alpha * lv.y + s.beta * mu.y));
            // sums of the source-term reductions; X_lk = -conj(X_kl) (G^< is anti-Hermitian, as
            // the forward stage reads it), so conj(X_lk) = -X_kl
            const cd B = cscale(cmul_i(g), gs);
            const cd cav = cconj(av);
            const cd xik = X[i * ns + k], xjk = X[j * ns + k];
            const cd m4 = cmul(cav, B), m2 = cmul(cconj(xik), B);
            const cd m1 = cmul(cconj(yjl), B), n2 = cmul(cconj(ykl), B), n3 = cmul(cconj(yil), B);
            q1 = csub(q1, cmul(xkl, B));
            q2 = cadd(q2, m2);
            q3 = cfma(q3, cconj(xjk), B);
            q4 = cadd(q4, m4);
            if (k == l) {
                qd = m2;
                sdia[k] = B;
            }
            sv[0] = m1.x;
            sv[1] = m1.y;
            sv[2] = n2.x;
            sv[3] = n2.y;
            sv[4] = n3.x;
            sv[5] = n3.y;
            sv[6] = m4.x;
            sv[7] = m4.y;
        }
        const double t = wsum8(sv, lane);
        if ((lane & 7) == 0) srow[k][lane >> 3] = t;
    }
    sh4[wave][0][lane] = q1;
    sh4[wave][1][lane] = q2;
    sh4[wave][2][lane] = q3;
    sh4[wave][3][lane] = q4;
    sh4[wave][4][lane] = qd;
    __syncthreads();
    if (wave != 0) return;
    // lane = k: the rows' partials of kinds 0 and 2, the terms of kind 1 and of dL/dU
    const double dij = i == j ? 1.0 : 0.0;
    auto iU = [&](cd v) { return cscale(cmul_i(v), U); };   // i U v
    cd x1 = cmk(0, 0), y1 = cmk(0, 0);
    double up = 0.0;
    if (lane_ok) {
        const int k = lane;
        const cd s1 = cmk(srow[k][0], srow[k][1]), s2 = cmk(srow[k][2], srow[k][3]);
        const cd s3 = cmk(srow[k][4], srow[k][5]), s4 = cmk(srow[k][6], srow[k][7]), Bkk = sdia[k];
        const cd xik = X[i * ns + k], xjk = X[j * ns + k], yjk = Y[j * ns + k];
        cd r0 = csub(cscale(s1, U * dij), cscale(cmul(cconj(yjk), Bkk), U));
        r0 = cadd(r0, iU(csub(cmul(cconj(yjk), s2), cmul(cconj(yji), s3))));
        const size_t o = ((size_t)i * ns + j) * ns + k;
        P[0 * (size_t)ns3 + o] = r0;
        P[1 * (size_t)ns3 + o] = s4;
        const cd c2 = iU(cmul(cconj(xij), s1));
        P[2 * (size_t)ns3 + o] = cmk(-c2.x, -c2.y);
        P[3 * (size_t)ns3 + o] = iU(cmul(cconj(xik), s2));
        const cd u1 = cmul(cconj(xjk), s1), u3 = cmul(cconj(xik), s3);
        x1 = iU(cmk(-u1.x, -u1.y));
        y1 = iU(cmk(-u3.x, -u3.y));
        // conj(Psi) B / U of the row, without its X_lk term
        cd t = csub(cscale(cmul(cconj(xik), s1), dij), cmul(cconj(cmul(xik, yjk)), Bkk));
        t = cadd(t, cmul_i(csub(cmul(cconj(cmul(yjk, xik)), s2),
                                cadd(cmul(cconj(xij), u1), cmul(cconj(yji), u3)))));
        up = t.x;
    }
    if (lane_ok) {   // lane = l: kinds 4 and 5
        cd v[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            v[q] = sh4[0][q][lane];
#pragma unroll
            for (int w = 1; w < ADJ_WAVES; ++w) v[q] = cadd(v[q], sh4[w][q][lane]);
        }
        const cd xil = X[i * ns + l];
        const size_t o = ((size_t)i * ns + j) * ns + l;
        P[4 * (size_t)ns3 + o] = iU(cmul(cconj(yjl), v[0]));
        const cd c4 = iU(cmul(cconj(yji), v[1]));
        P[5 * (size_t)ns3 + o] = cmk(-c4.x, -c4.y);
        cd a5 = cscale(csub(cscale(v[1], dij), v[4]), U);
        a5 = cadd(a5, iU(csub(cmul(cconj(xil), v[0]), cmul(cconj(xij), v[2]))));
        P[6 * (size_t)ns3 + o] = a5;
        P[7 * (size_t)ns3 + o] = v[3];
        const cd t = cmul_i(cmul(cconj(cmul(xil, yjl)), v[0]));
        up += t.x;
    }
    x1 = wsum(x1);
    y1 = wsum(y1);
    up = wsum(up);
    if (lane == 0) {
        cd* R = s.red;
        R[(R_X + 1) * ns2 + i * ns + j] = x1;
        R[(R_Y + 1) * ns2 + j * ns + i] = y1;
        R[R_UP * ns2 + i * ns + j] = cmk(up, 0.0);
    }
}

// Kinds 0, 2, 4, 5 from the per-slice partials: one thread per output pair;
// kinds 0 and 4 sum over j, kinds 2 and 5 over i (fixed order).  Threads
// 8 ns^2 .. 9 ns^2 - 1 add up the per-part sums of kind 3 (adj_lane_red).
__global__ __launch_bounds__(256) void adj_slice_fin_kernel(AdjArgs s) {
    const int ns = s.a.ns, ns2 = ns * ns, ns3 = ns2 * ns;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 9 * ns2) return;
    if (t >= 8 * ns2) {   // kind 3: the X cotangent at (l, k), the Y cotangent at (k, l)
        const int kl = t - 8 * ns2, k = kl / ns, l = kl % ns;
        cd v0 = cmk(0, 0), v1 = cmk(0, 0);
        for (int p = 0; p < s.nparts; ++p) {
            const cd* P = s.part + ((size_t)p * ns2 + kl) * 2;
            v0 = cadd(v0, P[0]);
            v1 = cadd(v1, P[1]);
        }
        s.red[(R_X + 3) * ns2 + l * ns + k] = v0;
        s.red[(R_Y + 3) * ns2 + k * ns + l] = v1;
        return;
    }
    const int q = t / ns2, o = t - q * ns2, p0 = o / ns, p1 = o - p0 * ns;
    const bool over_j = q == 0 || q == 1 || q == 4 || q == 5;
    const cd* P = s.spart + (size_t)q * ns3;
    cd v = cmk(0, 0);
    for (int r = 0; r < ns; ++r)
        v = cadd(v, over_j ? P[((size_t)p0 * ns + r) * ns + p1] : P[((size_t)r * ns + p0) * ns + p1]);
    static constexpr int slot[8] = {R_X + 0, R_M02, R_X + 2, R_Y + 2, R_X + 4, R_Y + 4, R_Y + 5, R_M13};
    s.red[slot[q] * ns2 + o] = v;
}

// Kind 3 of the source-term reductions (free (k,l)), with lane = l so that
// every load is a contiguous row.  Work-group (k, part): part a range of the
// summed pairs (i, j) split over the four waves; per-part sums go to s.part and
// adj_slice_fin_kernel adds them up.
__global__ __launch_bounds__(256) void adj_lane_red_kernel(AdjArgs s) {
    __shared__ cd sh[4][2][64];
    const Cl& a = s.a;
    const int ns = a.ns, ns2 = ns * ns;
    const int k = blockIdx.x % ns, part = blockIdx.x / ns;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool lane_ok = lane < ns;
    const int l = lane_ok ? lane : 0;
    const cd* X = a.X;
    const cd* Y = a.Y;
    const double U = a.U, gs = s.gscale;
    cd v0 = cmk(0, 0), v1 = cmk(0, 0);
    const int p0 = part * s.pairs_per_part, p1 = min(ns2, p0 + s.pairs_per_part);
    if (lane_ok) {
        for (int pr = p0 + wave; pr < p1; pr += 4) {
            const int i = pr / ns, j = pr % ns;
            const int e = ((i * ns + j) * ns + k) * ns + l;
            const cd B = cscale(cmul_i(s.gin2[e]), gs);
            v0 = cfma(v0, cscale(cmul_i(cconj(cmul(X[i * ns + l], Y[j * ns + l]))), U), B);
            v1 = cfma(v1, cscale(cmul_i(cconj(cmul(Y[j * ns + k], X[i * ns + k]))), U), B);
        }
    }
    sh[wave][0][lane] = v0;
    sh[wave][1][lane] = v1;
    __syncthreads();
    if (wave == 0 && lane_ok) {
        cd t0 = cadd(cadd(sh[0][0][lane], sh[1][0][lane]), cadd(sh[2][0][lane], sh[3][0][lane]));
        cd t1 = cadd(cadd(sh[0][1][lane], sh[1][1][lane]), cadd(sh[2][1][lane], sh[3][1][lane]));
        cd* P = s.part + ((size_t)part * ns2 + k * ns + l) * 2;
        P[0] = t0;
        P[1] = t1;
    }
}

// Cotangents of the h^HF diagonals (ebar), the drive and U parts that depend
// on them, and the sum of the U partials of the source (one work-group; four
// threads per site).
__global__ __launch_bounds__(256) void adj_e_kernel(AdjArgs s) {
    __shared__ double sh[2][256];
    const Cl& a = s.a;
    const int ns = a.ns, ns2 = ns * ns, t = threadIdx.x;
    const cd* R = s.red;
    const double gs = s.gscale;
    const cd* X = a.X;
    const cd* Y = a.Y;
    const cd* gx = s.gin1;
    const cd* gy = s.gin1 + ns2;
    double sbar = 0.0, ubar = 0.0;
    const int i = t >> 2, sub = t & 3;
    cd eu = cmk(0, 0), ed = cmk(0, 0);
    if (i < ns) {
        for (int p = sub; p < ns; p += 4) {
            // (BX X^H - X^H BX)_ii with BX = i gs gX
            cd bx_ip = cscale(cmul_i(gx[i * ns + p]), gs), bx_pi = cscale(cmul_i(gx[p * ns + i]), gs);
            eu = cadd(eu, csub(cmul(bx_ip, cconj(X[i * ns + p])), cmul(cconj(X[p * ns + i]), bx_pi)));
            cd by_ip = cscale(cmul_i(gy[i * ns + p]), gs), by_pi = cscale(cmul_i(gy[p * ns + i]), gs);
            ed = cadd(ed, csub(cmul(by_ip, cconj(Y[i * ns + p])), cmul(cconj(Y[p * ns + i]), by_pi)));
            eu = cadd(eu, csub(R[R_M02 * ns2 + i * ns + p], R[R_M02 * ns2 + p * ns + i]));
            ed = cadd(ed, csub(R[R_M13 * ns2 + i * ns + p], R[R_M13 * ns2 + p * ns + i]));
        }
    }
    // sum the four partial sums of a site (lanes 4i .. 4i+3)
    for (int o = 1; o < 4; o <<= 1) {
        eu.x += __shfl_xor(eu.x, o, 64);
        eu.y += __shfl_xor(eu.y, o, 64);
        ed.x += __shfl_xor(ed.x, o, 64);
        ed.y += __shfl_xor(ed.y, o, 64);
    }
    if (i < ns && sub == 0) {
        s.ebar[i] = eu;
        s.ebar[ns + i] = ed;
        sbar = a.xdrv[i] * (eu.x + ed.x);
        // e^up_i = ... - i U Y_ii, e^dn_i = ... - i U X_ii: Ubar += Re(conj(-i Y_ii) ebar)
        cd myi = cmul_mi(Y[i * ns + i]), mxi = cmul_mi(X[i * ns + i]);
        ubar = myi.x * eu.x + myi.y * eu.y + mxi.x * ed.x + mxi.y * ed.y;
    }
    for (int q = t; q < ns2; q += blockDim.x) ubar += R[R_UP * ns2 + q].x;
    sh[0][t] = sbar;
    sh[1][t] = ubar;
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if (t < st) {
            sh[0][t] += sh[0][t + st];
            sh[1][t] += sh[1][t + st];
        }
        __syncthreads();
    }
    if (t == 0) {
        s.gpart[0] = sh[0][0];
        s.gpart[1] = sh[1][0];
    }
}

// G1 cotangents, one thread per element of [X | Y]; partial dL/dU of the
// collision integral per work-group into s.gpart[2 + block].
__global__ __launch_bounds__(256) void adj_g1e_kernel(AdjArgs s) {
    __shared__ double sh[256];
    const Cl& a = s.a;
    const int ns = a.ns, ns2 = ns * ns, z = a.zmax;
    const cd* R = s.red;
    const double gs = s.gscale;
    const cd* gx = s.gin1;
    const cd* gy = s.gin1 + ns2;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    double ubar = 0.0;
    if (e < 2 * ns2) {
        const int sig = e / ns2, r = e % ns2, i = r / ns, j = r % ns;
        const cd* gg = sig ? gy : gx;
        const cd* eb = s.ebar + (sig ? 0 : ns);   // X_ii enters e^dn, Y_ii enters e^up
        const int* nb = a.nbr + sig * ns * z;
        const cd* hp = a.hop + sig * ns * z;
        // [h^H, B]_ij, B = i gs g
        cd ei = hf_diag(a, sig, i), ej = hf_diag(a, sig, j);
        cd bij = gg[r];
        cd c = csub(cmul(cconj(ei), bij), cmul(bij, cconj(ej)));
        for (int q = 0; q < z; ++q) {
            int p = nb[i * z + q];
            if (p >= 0) c = cfma(c, hp[i * z + q], gg[p * ns + j]);
        }
        for (int q = 0; q < z; ++q) {
            int p = nb[j * z + q];
            if (p >= 0) c = csub(c, cmul(gg[i * ns + p], cconj(hp[j * z + q])));
        }
        cd mu = cscale(cmul_i(c), gs);
        // source-term reductions: X receives kinds 0-4, Y kinds 1-5
        for (int kd = sig ? 1 : 0; kd < (sig ? 6 : 5); ++kd) mu = cadd(mu, R[((sig ? R_Y : R_X) + kd) * ns2 + r]);
        if (i == j) mu = cadd(mu, cscale(cmul_i(eb[i]), a.U));
        // collision-integral part of dL/dU: I_ij = -i U A..., Ibar_ij = B_ij + conj(B_ji)
        cd bb = cadd(cscale(cmul_i(gg[r]), gs), cconj(cscale(cmul_i(gg[j * ns + i]), gs)));
        cd av = sig == 0 ? ld_a(s, ((i * ns + i) * ns + j) * ns + i) : ld_a(s, ((i * ns + i) * ns + i) * ns + j);
        cd dI = cmul_mi(av);   // dI/dU
        ubar = dI.x * bb.x + dI.y * bb.y;
        cd base = s.init ? s.lam1[e] : s.lacc1[e];
        s.lacc1[e] = cadd(base, mu);
        if (s.has_next) {
            cd lv = s.lam1[e];
            s.gnext1[e] = cmk(s.alpha * lv.x + s.beta * mu.x, s.alpha * lv.y + s.beta * mu.y);
        }
    }
    sh[threadIdx.x] = ubar;
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) s.gpart[2 + blockIdx.x] = sh[0];
}

// dL/ds and dL/dU of the stage from the partials (fixed summation order).
__global__ void adj_gsum_kernel(AdjArgs s, int nblocks) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double u = s.gpart[1];
    for (int b = 0; b < nblocks; ++b) u += s.gpart[2 + b];
    s.grads[0] = s.gpart[0];
    s.grads[1] = u;
}

// Terminal cotangent of the loss and its value.
__global__ void adj_terminal_kernel(Cl a, const cd* __restrict__ A, const double* __restrict__ wa,
                                    const double* __restrict__ wb, cd* __restrict__ l1,
                                    cd* __restrict__ l2, double* __restrict__ loss) {
    const int ns = a.ns;
    double L = 0.0;
    for (int i = 0; i < ns; ++i) {
        const int ii = i * ns + i;
        const int e = ((i * ns + i) * ns + i) * ns + i;
        double nu = a.X[ii].y, nd = a.Y[ii].y;
        L += wa[i] * (nu * nd - A[e].x) + wb[i] * (nu + nd);
        l1[ii] = cmk(0.0, wa[i] * nd + wb[i]);            // dL/dIm X_ii
        l1[ns * ns + ii] = cmk(0.0, wa[i] * nu + wb[i]);  // dL/dIm Y_ii
        l2[e] = cmk(-wa[i], 0.0);                         // dL/dRe A_iiii
    }
    *loss = L;
}

}  // namespace

// ---------------------------------------------------------------------------- host
namespace {

// Stage states that the forward pass may keep when the library chooses the
// interval: with four states per step the reverse sweep recomputes nothing.  Up to
// this many, an eighth of the device's memory and, all buffers of the adjoint
// counted, a quarter of what is free of it (a program that already holds memory, or
// several contexts, keep checkpoints instead: the sweep then recomputes each step
// once, 7.5 instead of 36 GB for 32 steps of the 8x8 cluster).
constexpr int64_t ADJ_KEEP_STATES = 128;

struct AdjState {
    int64_t nsteps = 0;
    int64_t have_steps = 0;    // steps, interval and storage the buffers below were made for
    int have_interval = 0;
    size_t have_n1 = 0, have_n2 = 0;
    size_t have_bytes = 0;     // device memory of their states
    bool have_mixed = false, have_keep = false;
    bool ready = false;        // a forward pass has ended and its states are whole
    bool keep = false;         // one segment, whose states the forward pass kept
    bool herm = false;         // the symmetry check's result (ctx) for the states of the forward pass
    bool mixed = false;        // binary32 G2 stage copies (Y2, Y3, Y4), as the mixed forward stages
    int interval = 0;
    double dt = 0.0, t0 = 0.0;
    int nck = 0;
    std::vector<Regs> ckpt;
    // one segment of the forward pass, recomputed from its checkpoint: the
    // state y_n and the stage states Y2, Y3, Y4 of every step
    std::vector<Regs> seg, seg2, seg3, seg4;
    Regs LAM, LACC, CA, CB;
    cd* red = nullptr;
    cd* part = nullptr;        // kind-3 lane-reduction partials
    cd* spart = nullptr;       // per-slice partials of kinds 0, 2, 4, 5
    int nparts = 0, pairs_per_part = 0;
    cd* ebar = nullptr;
    double* gpart = nullptr;
    double* grads = nullptr;   // [4 nsteps][2]
    double* dev_ab = nullptr;  // weights a, b and the loss
};

constexpr int ADJ_PAIRS_PER_PART = 64;

AdjState* adj_of(g1g2_ctx* c) { return reinterpret_cast<AdjState*>(c->adj); }

// half32: the G2 part holds binary32 values only (a mixed-precision stage copy)
g1g2_status alloc_reg(g1g2_ctx* c, Regs& r, bool half32 = false) {
    HIP_OK(c, hipMalloc(&r.g1, c->n1 * sizeof(cd)));
    HIP_OK(c, hipMalloc(&r.g2, c->n2 * (half32 ? sizeof(float2) : sizeof(cd))));
    return G1G2_OK;
}

void free_reg(Regs& r) {
    if (r.g1) (void)hipFree(r.g1);
    if (r.g2) (void)hipFree(r.g2);
    r = Regs();
}

g1g2_status copy_reg(g1g2_ctx* c, const Regs& dst, const Regs& src) {
    HIP_OK(c, hipMemcpyAsync(dst.g1, src.g1, c->n1 * sizeof(cd), hipMemcpyDeviceToDevice, c->stream));
    HIP_OK(c, hipMemcpyAsync(dst.g2, src.g2, c->n2 * sizeof(cd), hipMemcpyDeviceToDevice, c->stream));
    prof_mark(c, "state_copy");
    return G1G2_OK;
}

// S32: the G2 of S holds binary32 values (a mixed-precision stage copy).
AdjArgs make_adj(g1g2_ctx* c, double t, const Regs& S, bool S32, const Regs& gin, double gscale,
                 const Regs& lam, const Regs& lacc, const Regs& gnext, double alpha, double beta, int init,
                 int has_next, double* grads) {
    HubbardData& H = c->hub;
    AdjState* st = adj_of(c);
    const ClusterDesc& d = H.hdesc[0];
    AdjArgs s;
    Cl a;
    a.ns = d.ns;
    a.zmax = d.zmax;
    a.U = d.U;
    a.s_drive = H.drive_value(t);
    a.nbr = H.nbr;
    a.hop = H.hop;
    a.d0 = H.d0;
    a.xdrv = H.xdrv;
    a.X = S.g1;
    a.Y = S.g1 + d.ns * d.ns;
    s.a = a;
    s.A = S.g2;
    s.a32 = S32 ? 1 : 0;
    s.gin1 = gin.g1;
    s.gin2 = gin.g2;
    s.gscale = gscale;
    s.lam1 = lam.g1;
    s.lam2 = lam.g2;
    s.lacc1 = lacc.g1;
    s.lacc2 = lacc.g2;
    s.gnext1 = gnext.g1;
    s.gnext2 = gnext.g2;
    s.alpha = alpha;
    s.beta = beta;
    s.init = init;
    s.has_next = has_next;
    s.red = st->red;
    s.part = st->part;
    s.spart = st->spart;
    s.pairs_per_part = st->pairs_per_part;
    s.nparts = st->nparts;
    s.ebar = st->ebar;
    s.gpart = st->gpart;
    s.grads = grads;
    return s;
}

g1g2_status vjp(g1g2_ctx* c, const AdjArgs& s) {
    const int ns = s.a.ns, ns2 = ns * ns;
    hipLaunchKernelGGL(adj_slice_red_kernel, dim3(ns2), dim3(64 * ADJ_WAVES), 0, c->stream, s);
    prof_mark(c, "adj_slice_red");
    hipLaunchKernelGGL(adj_lane_red_kernel, dim3(ns * s.nparts), dim3(256), 0, c->stream, s);
    prof_mark(c, "adj_lane_red");
    hipLaunchKernelGGL(adj_slice_fin_kernel, dim3((9 * ns2 + 255) / 256), dim3(256), 0, c->stream, s);
    prof_mark(c, "adj_slice_fin");
    HIP_OK(c, hipGetLastError());
    const int g1blocks = (2 * ns2 + 255) / 256;
    hipLaunchKernelGGL(adj_e_kernel, dim3(1), dim3(256), 0, c->stream, s);
    prof_mark(c, "adj_e");
    hipLaunchKernelGGL(adj_g1e_kernel, dim3(g1blocks), dim3(256), 0, c->stream, s);
    prof_mark(c, "adj_g1e");
    hipLaunchKernelGGL(adj_gsum_kernel, dim3(1), dim3(64), 0, c->stream, s, g1blocks);
    prof_mark(c, "adj_gsum");
    HIP_OK(c, hipGetLastError());
    return G1G2_OK;
}

// The buffers of a gradient of nsteps steps in segments of `interval`, in place of
// those of the last one.  After an error none are held.
g1g2_status adj_alloc(g1g2_ctx* c, int64_t nsteps, int interval, bool mixed, bool keep) {
    adj_free(c);
    AdjState* const st = new (std::nothrow) AdjState();
    if (!st) return set_error(c, G1G2_ENOMEM, "adjoint state");
    c->adj = st;
    const int ns = c->hub.hdesc[0].ns;
    const auto fill = [&]() -> g1g2_status {
        g1g2_status s;
        st->ckpt.resize((nsteps + interval - 1) / interval + 1);   // last slot keeps the final state
        for (auto& r : st->ckpt)
            if ((s = alloc_reg(c, r)) != G1G2_OK) return s;
        for (auto* v : {&st->seg, &st->seg2, &st->seg3, &st->seg4}) {
            v->resize(interval);
            for (auto& r : *v)
                if ((s = alloc_reg(c, r, mixed && v != &st->seg)) != G1G2_OK) return s;
        }
        for (Regs* r : {&st->LAM, &st->LACC, &st->CA, &st->CB})
            if ((s = alloc_reg(c, *r)) != G1G2_OK) return s;
        HIP_OK(c, hipMalloc(&st->red, (size_t)R_N * ns * ns * sizeof(cd)));
        st->pairs_per_part = ADJ_PAIRS_PER_PART;
        st->nparts = (ns * ns + ADJ_PAIRS_PER_PART - 1) / ADJ_PAIRS_PER_PART;
        HIP_OK(c, hipMalloc(&st->part, (size_t)st->nparts * ns * ns * 2 * sizeof(cd)));
        HIP_OK(c, hipMalloc(&st->spart, (size_t)8 * ns * ns * ns * sizeof(cd)));
        HIP_OK(c, hipMalloc(&st->ebar, (size_t)2 * ns * sizeof(cd)));
        HIP_OK(c, hipMalloc(&st->gpart, (size_t)(2 + (2 * ns * ns + 255) / 256) * sizeof(double)));
        HIP_OK(c, hipMalloc(&st->grads, (size_t)4 * nsteps * 2 * sizeof(double)));
        HIP_OK(c, hipMalloc(&st->dev_ab, (size_t)(2 * ns + 8) * sizeof(double)));
        return G1G2_OK;
    };
    const g1g2_status s = fill();
    if (s != G1G2_OK) {
        (void)hipGetLastError();   // reported here, not by a later launch check
        adj_free(c);
        return s;
    }
    st->have_steps = nsteps;
    st->have_interval = interval;
    st->have_n1 = c->n1;
    st->have_n2 = c->n2;
    st->have_bytes = (2 * st->ckpt.size() + (size_t)interval * (mixed ? 5 : 8) + 8) * c->n2 * (sizeof(cd) / 2);
    st->have_mixed = mixed;
    st->have_keep = keep;
    return G1G2_OK;
}

g1g2_status stage_fwd(g1g2_ctx* c, int mode, double t, const Regs& in, const Regs& y, const Regs& acc,
                      const Regs& out, double cb, double cc) {
    return hub_stage(c, mode, t, in, y, acc, out, cb, cc);
}

}  // namespace

void adj_free(g1g2_ctx* c) {
    AdjState* st = adj_of(c);
    if (!st) return;
    for (auto* v : {&st->ckpt, &st->seg, &st->seg2, &st->seg3, &st->seg4})
        for (auto& r : *v) free_reg(r);
    for (Regs* r : {&st->LAM, &st->LACC, &st->CA, &st->CB}) free_reg(*r);
    if (st->red) (void)hipFree(st->red);
    if (st->part) (void)hipFree(st->part);
    if (st->spart) (void)hipFree(st->spart);
    if (st->ebar) (void)hipFree(st->ebar);
    if (st->gpart) (void)hipFree(st->gpart);
    if (st->grads) (void)hipFree(st->grads);
    if (st->dev_ab) (void)hipFree(st->dev_ab);
    delete st;
    c->adj = nullptr;
}

extern "C" {

// Whether a run of nsteps steps keeps its states (ADJ_KEEP_STATES), given the size of
// a G2 register and the device's free and total memory.  Not part of the ABI; host
// arithmetic with a name that tests can find.
int adj_keeps_states(int64_t nsteps, size_t state_bytes, size_t free_bytes, size_t total_bytes) {
    if (nsteps < 1 || nsteps > ADJ_KEEP_STATES / 4) return 0;
    const size_t kept = 4 * (size_t)nsteps * state_bytes;
    const size_t all = kept + 6 * state_bytes;   // two checkpoints, four cotangents
    return kept <= total_bytes / 8 && all <= free_bytes / 4;
}

g1g2_status g1g2_forward_checkpointed(g1g2_ctx* c, double dt, int64_t nsteps, int32_t interval) {
    if (!c || nsteps < 1 || !(dt > 0.0)) return G1G2_EINVAL;
    if (c->d.basis != G1G2_HUBBARD || c->d.selfenergy != G1G2_SOA || c->hub.ncl != 1)
        return set_error(c, G1G2_EUNSUPPORTED, "the adjoint covers the single-cluster Hubbard SOA system");
    if (c->hub.hdesc[0].ns > 64) return set_error(c, G1G2_EUNSUPPORTED, "adjoint supports ns <= 64");
    if (c->has_switch())
        return set_error(c, G1G2_EUNSUPPORTED, "the adjoint takes a constant U (switching is set)");
    const bool mixed = c->d.precision == G1G2_MIXED;
    // default: the interval that minimizes checkpoints + four states per segment step
    const int def = std::max<int>(1, (int)std::ceil(std::sqrt((double)nsteps / 4.0)));
    const int group = interval > 0 ? interval : def;   // steps between divergence checks
    // the buffers of the last gradient serve again while its shape stays (allocating
    // and releasing the 8x8 cluster's 56 states took 9 ms of a 77 ms gradient)
    const auto same = [&](bool kept) {
        const AdjState* a = adj_of(c);
        return a && a->have_steps == nsteps && a->have_interval == (kept ? (int)nsteps : group) &&
               a->have_n1 == c->n1 && a->have_n2 == c->n2 && a->have_mixed == mixed && a->have_keep == kept;
    };
    g1g2_status s;
    bool keep = interval <= 0 && hub_tile_ok(c) && nsteps <= ADJ_KEEP_STATES / 4;
    if (keep && !same(true)) {
        size_t mfree = 0, mtotal = 0;
        HIP_OK(c, hipMemGetInfo(&mfree, &mtotal));
        const size_t held = adj_of(c) ? adj_of(c)->have_bytes : 0;
        keep = adj_keeps_states(nsteps, c->n2 * sizeof(cd), mfree + held, mtotal) != 0;
        if (keep && (s = adj_alloc(c, nsteps, (int)nsteps, mixed, true)) != G1G2_OK) {
            if (s != G1G2_ENOMEM) return s;
            keep = false;   // checkpoints need less
            c->err.clear();
        }
    }
    if (!keep && !same(false) && (s = adj_alloc(c, nsteps, group, mixed, false)) != G1G2_OK) return s;
    AdjState* const st = adj_of(c);
    st->ready = false;
    st->nsteps = nsteps;
    st->mixed = mixed;
    st->keep = keep;
    st->herm = c->herm;
    st->interval = keep ? (int)nsteps : group;
    st->dt = dt;
    st->t0 = c->t;
    st->nck = (int)((nsteps + st->interval - 1) / st->interval);
    const int ns = c->hub.hdesc[0].ns;
    HIP_OK(c, hipMemsetAsync(st->red, 0, (size_t)R_N * ns * ns * sizeof(cd), c->stream));
    if (keep) {
        // the steps themselves fill the segment: y_n, Y2, Y3, Y4 of step n, each step
        // writing the next y_n; checked for divergence as g1g2_step_rk4 does
        if ((s = copy_reg(c, st->seg[0], c->y)) != G1G2_OK) return s;
        for (int64_t n = 0; n < nsteps; n += group) {
            const int64_t m1 = std::min<int64_t>(nsteps, n + group);
            if ((s = step_begin(c)) != G1G2_OK) return s;
            for (int64_t m = n; m < m1; ++m) {
                const Regs& next = m + 1 < nsteps ? st->seg[m + 1] : st->ckpt[st->nck];
                if ((s = hub_tile_step(c, st->t0 + (double)m * dt, dt, st->seg[m], next, st->seg2[m], st->seg3[m],
                                       st->seg4[m], c->acc, true, true)) != G1G2_OK)
                    return s;
            }
            const Regs& done = m1 < nsteps ? st->seg[m1] : st->ckpt[st->nck];
            if ((s = copy_reg(c, c->y, done)) != G1G2_OK) return s;
            if ((s = step_end(c, c->t + (double)(m1 - n) * dt, m1 - n)) != G1G2_OK) return s;
        }
        st->ready = true;
        return G1G2_OK;
    }
    for (int q = 0; q < st->nck; ++q) {
        if ((s = copy_reg(c, st->ckpt[q], c->y)) != G1G2_OK) return s;
        const int64_t n = std::min<int64_t>(st->interval, nsteps - (int64_t)q * st->interval);
        if ((s = g1g2_step_rk4(c, dt, n)) != G1G2_OK) return s;
    }
    if ((s = copy_reg(c, st->ckpt[st->nck], c->y)) != G1G2_OK) return s;
    st->ready = true;
    return G1G2_OK;
}

g1g2_status g1g2_adjoint(g1g2_ctx* c, const double* wa, const double* wb, double* grad_c,
                         double* grad_U, double* loss) {
    if (!c || !wa || !wb) return G1G2_EINVAL;
    AdjState* st = adj_of(c);
    if (!st || !st->ready) return set_error(c, G1G2_ESTATE, "call g1g2_forward_checkpointed first");
    HubbardData& H = c->hub;
    const int ns = H.hdesc[0].ns;
    const double dt = st->dt;
    g1g2_status s;
    // terminal cotangent
    HIP_OK(c, hipMemcpyAsync(st->dev_ab, wa, ns * sizeof(double), hipMemcpyHostToDevice, c->stream));
    HIP_OK(c, hipMemcpyAsync(st->dev_ab + ns, wb, ns * sizeof(double), hipMemcpyHostToDevice, c->stream));
    HIP_OK(c, hipMemsetAsync(st->LAM.g1, 0, c->n1 * sizeof(cd), c->stream));
    HIP_OK(c, hipMemsetAsync(st->LAM.g2, 0, c->n2 * sizeof(cd), c->stream));
    prof_mark(c, "adj_init");
    {
        const Regs& fin = st->ckpt[st->nck];
        AdjArgs tmp = make_adj(c, st->t0 + st->nsteps * dt, fin, false, fin, 1.0, fin, fin, fin, 0, 0, 0, 0, nullptr);
        hipLaunchKernelGGL(adj_terminal_kernel, dim3(1), dim3(1), 0, c->stream, tmp.a, fin.g2, st->dev_ab,
                           st->dev_ab + ns, st->LAM.g1, st->LAM.g2, st->dev_ab + 2 * ns);
        HIP_OK(c, hipGetLastError());
        prof_mark(c, "adj_terminal");
    }
    Regs lam = st->LAM, lacc = st->LACC;
    for (int q = st->nck - 1; q >= 0; --q) {
        const int64_t n0 = (int64_t)q * st->interval;
        const int64_t n1 = std::min<int64_t>(n0 + st->interval, st->nsteps);
        // recompute the segment forward, keeping y_n and the stage states of every step;
        // the kernels are those of the forward pass, whatever state has been set since
        if (!st->keep) {
            c->herm = st->herm;
            if ((s = copy_reg(c, c->y, st->ckpt[q])) != G1G2_OK) return s;
        }
        for (int64_t n = n0; n < n1 && !st->keep; ++n) {
            const int m = (int)(n - n0);
            if ((s = copy_reg(c, st->seg[m], c->y)) != G1G2_OK) return s;
            const double t = st->t0 + (double)n * dt;
            const Regs &s2 = st->seg2[m], &s3 = st->seg3[m], &s4 = st->seg4[m];
            const bool last = n + 1 < n1;
            if (hub_tile_ok(c)) {   // the reverse sweep reads the stage states whole
                if ((s = hub_tile_step(c, t, dt, c->y, c->y, s2, s3, s4, c->acc, true, last)) != G1G2_OK) return s;
                continue;
            }
            if ((s = stage_fwd(c, RK_FIRST, t, c->y, c->y, c->acc, s2, dt / 6.0, dt / 2.0)) != G1G2_OK) return s;
            if ((s = stage_fwd(c, RK_MID, t + 0.5 * dt, s2, c->y, c->acc, s3, dt / 3.0, dt / 2.0)) != G1G2_OK) return s;
            if ((s = stage_fwd(c, RK_MID, t + 0.5 * dt, s3, c->y, c->acc, s4, dt / 3.0, dt)) != G1G2_OK) return s;
            if (last)
                if ((s = stage_fwd(c, RK_LAST, t + dt, s4, c->y, c->acc, c->y, dt / 6.0, 0.0)) != G1G2_OK) return s;
        }
        // reverse over the segment: Y2 = y + dt/2 k1, Y3 = y + dt/2 k2, Y4 = y + dt k3
        for (int64_t n = n1 - 1; n >= n0; --n) {
            const int m = (int)(n - n0);
            const Regs& y = st->seg[m];
            const double t = st->t0 + (double)n * dt;
            double* g = st->grads + (size_t)8 * n;
            const bool m32 = st->mixed;   // the stage copies Y2, Y3, Y4 are binary32 in mixed precision
            if ((s = vjp(c, make_adj(c, t + dt, st->seg4[m], m32, lam, dt / 6.0, lam, lacc, st->CA, dt / 3.0, dt, 1, 1, g + 6))) != G1G2_OK) return s;
            if ((s = vjp(c, make_adj(c, t + 0.5 * dt, st->seg3[m], m32, st->CA, 1.0, lam, lacc, st->CB, dt / 3.0, dt / 2.0, 0, 1, g + 4))) != G1G2_OK) return s;
            if ((s = vjp(c, make_adj(c, t + 0.5 * dt, st->seg2[m], m32, st->CB, 1.0, lam, lacc, st->CA, dt / 6.0, dt / 2.0, 0, 1, g + 2))) != G1G2_OK) return s;
            if ((s = vjp(c, make_adj(c, t, y, false, st->CA, 1.0, lam, lacc, st->CB, 0.0, 0.0, 0, 0, g + 0))) != G1G2_OK) return s;
            std::swap(lam, lacc);
        }
    }
    // restore the final state
    c->herm = st->herm;
    if ((s = copy_reg(c, c->y, st->ckpt[st->nck])) != G1G2_OK) return s;
    std::vector<double> gr((size_t)8 * st->nsteps);
    double L = 0.0;
    HIP_OK(c, hipMemcpyAsync(gr.data(), st->grads, gr.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIP_OK(c, hipMemcpyAsync(&L, st->dev_ab + 2 * ns, sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIP_OK(c, hipStreamSynchronize(c->stream));
    const double cs[4] = {0.0, 0.5, 0.5, 1.0};
    const int M = (int)H.drive_c.size();
    double gU = 0.0;
    if (grad_c)
        for (int m = 0; m < M; ++m) grad_c[m] = 0.0;
    for (int64_t n = 0; n < st->nsteps; ++n)
        for (int q = 0; q < 4; ++q) {
            const double sb = gr[8 * n + 2 * q], ub = gr[8 * n + 2 * q + 1];
            gU += ub;
            const double ts = st->t0 + ((double)n + cs[q]) * dt;
            if (grad_c)
                for (int m = 0; m < M; ++m) {
                    const double d = ts - H.drive_tc[m];
                    grad_c[m] += sb * std::exp(-d * d / (2.0 * H.drive_tau * H.drive_tau));
                }
        }
    if (grad_U) *grad_U = gU;
    if (loss) *loss = L;
    return G1G2_OK;
}

}  // extern "C"
