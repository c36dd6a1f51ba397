// Element-wise subgrid scale (Section 2.1.3): the subscale comes from an
// equation posed element by element -- the strong residual at the Gauss
// points times a diagonal stabilisation matrix -- evaluated in a plain loop
// over the elements with no system formed and nothing scattered. Read for
// the problems this library assembles:
//   utilde_q = tau_e (f_e + L(u_h)(x_q)),   tau_e = V_e^(2/3) / (4 k),
// L the Laplacian (Poisson, -Lap u = f, k = 1) or div sigma(u) =
// mu Lap u + (lam + mu) grad div u (linear elasticity, k = mu_e), u_h the
// interpolated nodal field, V_e = sum_q w_q detJ_q.
//
// Physical second derivatives: differentiating u(x(xi)) twice gives
//   H_xi(u) = J^T H_x(u) J + sum_k (du/dx_k) H_xi(x_k),
// so H_x(u) = J^-T M J^-1 with M = H_xi(u) - sum_k (du/dx_k) H_xi(x_k).
// Every shape function here is linear in each reference coordinate taken
// alone (tet4 linear, hex8 and the collapsed-hexahedron pyramid
// multilinear, pen6 linear in (r, s) times linear in t), so the pure
// second reference derivatives vanish and M has only its three mixed
// entries (xi eta, xi zeta, eta zeta). For tet4 all of them vanish:
// L(u_h) = 0 identically and u is not read.
//
// Work layout: the elements of a family in type-sorted order, one lane per
// (element, Gauss point). hex8 and the pyramid (a hexahedron whose top corners
// coincide) have as many Gauss points as corners: lane (b0, b1, b2) of an
// element gathers the corner with these coordinate signs, and the tensor
// products are formed one direction at a time by exchanges between lanes (see
// sub_tensor), without LDS and without a barrier. pen6: over the reference
// element every field is A(r, s) + t B(r, s) with A, B linear, as many
// coefficients as Gauss points; the element's lanes each gather one node into
// LDS, form one coefficient of every field from the node values and evaluate
// the fields at their Gauss point from the coefficients. tet4: one lane per
// element, no second derivatives.
//
// What bounds it: the vector instructions of a point (pyr5 and hex8 elasticity
// 496, 315 of them FP64, 23 of all only where an element has no stiffness) and the
// chain ids -> values -> results of a wave that lives for one group of elements. All
// global loads are therefore issued in two levels (ids; then coordinates,
// field, material, source and output place together), and material constants
// cost two divisions instead of three. Measured on MI355X, us a call,
// before -> after (before: coefficients of every field through LDS, five
// barriers, loads behind each other): elasticity, 96^3 cells of one family, pyr5
// (42M points) 996 -> 670, hex8 (7M) 179 -> 130, pen6 (11M) 237 -> 224, tet4 (5M)
// 128 -> 103; Poisson 489 -> 367, 96 -> 68, 116 -> 121, 86 -> 62; 16^3 cells, all
// families, 18.9 -> 7.2 (one launch for all, see run_sub). Issuing the pyramid's
// instructions takes 0.51 of its 0.67 ms (122 VGPRs: four waves per SIMD; at 138
// and three 0.73).
#include <algorithm>
#include <climits>

#include "elem.h"

namespace fea {

// Gauss coordinate of the two-point rule, as in the reference tables.
constexpr double kGauss = 0.57735026918962576451;

struct SubArgs {
    const double *x, *y, *z;
    const double *u;       // B values per node, node-major
    const double *young;   // per element, NULL = 1
    const double *nu;      // per element (elasticity)
    const double *source;  // B values per element
    const int32_t *perm;   // this family's element ids (type-sorted order)
    const int32_t *pnodes; // their node ids, NN per element
    const int64_t *gp_ptr; // Gauss-point offsets in element order
    int64_t n;             // elements in this launch
    double *out;           // out[(gp_ptr[e] + q) * B + c]
    int32_t *status;       // smallest element id with detJ <= 0
};

// SubArgs as the batched kernel reads them from its table: every pointer
// typed as addressing global memory, so that the compiler keeps global
// instead of flat accesses (see ElemArgsGlobal).
#define FEA_G(T) T __attribute__((address_space(1))) *
struct SubArgsGlobal {
    FEA_G(const double) x;
    FEA_G(const double) y;
    FEA_G(const double) z;
    FEA_G(const double) u;
    FEA_G(const double) young;
    FEA_G(const double) nu;
    FEA_G(const double) source;
    FEA_G(const int32_t) perm;
    FEA_G(const int32_t) pnodes;
    FEA_G(const int64_t) gp_ptr;
    int64_t n;
    FEA_G(double) out;
    FEA_G(int32_t) status;
};
#undef FEA_G
static_assert(sizeof(SubArgsGlobal) == sizeof(SubArgs) && offsetof(SubArgsGlobal, status) == offsetof(SubArgs, status),
              "SubArgsGlobal mirrors SubArgs");

__device__ __forceinline__ SubArgs from_global(const SubArgsGlobal &g)
{
    SubArgs a;
    a.x = (const double *)g.x;
    a.y = (const double *)g.y;
    a.z = (const double *)g.z;
    a.u = (const double *)g.u;
    a.young = (const double *)g.young;
    a.nu = (const double *)g.nu;
    a.source = (const double *)g.source;
    a.perm = (const int32_t *)g.perm;
    a.pnodes = (const int32_t *)g.pnodes;
    a.gp_ptr = (const int64_t *)g.gp_ptr;
    a.n = g.n;
    a.out = (double *)g.out;
    a.status = (int32_t *)g.status;
    return a;
}

// LDS of one workgroup (pen6 only): per element its nodes' values, then (same
// space) its coefficients. Strides padded to 2 (mod 4) doubles: the elements
// that a wave reads at once then start in distinct 16-byte bank slots.
template <int T, int MODEL>
struct SubSmem {
    static constexpr int NN = Fam<T>::NN, NQ = Fam<T>::NQ, EPW = 256 / NQ;
    static constexpr int B = MODEL == FEA_POISSON ? 1 : 3;
    static constexpr int NV = 3 + B;                                    // node values
    static constexpr int SE = NQ * NV + ((2 - (NQ * NV) % 4) + 4) % 4;
    double sNode[T == 2 ? EPW * SE : 1];
    double sWd[T == 2 ? 256 : 1];
};

// x of the lane whose index differs by the mask M, all lanes active.
template <int M>
__device__ __forceinline__ double lane_x(const double x)
{
    static_assert(M == 1 || M == 2 || M == 7, "one DPP move each");
    constexpr int CTRL = M == 1 ? 0xB1 : M == 2 ? 0x4E : 0x141;  // quad_perm 1 0 3 2, 2 3 0 1, half-row mirror
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)hi << 32 | (unsigned)lo);
}

// A trilinear field with value v at this lane's corner: its first (d) and
// mixed second (m2: pairs (0, 1), (0, 2), (1, 2)) derivatives at the Gauss point
// on the corner's side, with respect to reference coordinates that run from the
// opposite corner to this one over a length of 1 (xi_k = h_k eta_k, h_k = +-2:
// what follows from them does not depend on the scaling, but for det J, which
// is 8 times too large and has the sign of the corner's three signs).
// Neighbours in directions 0, 1, 2 are the lanes 1, 2 and 7 apart (three masks
// that one DPP move serves each, and that span the eight lanes); the difference
// v - v' is the derivative, v - (1 - g) / 2 (v - v') the interpolated value.
__device__ __forceinline__ void sub_tensor(const double v, double d[3], double m2[3])
{
    constexpr double C = 0.5 * (1.0 - kGauss);
    const double D = v - lane_x<1>(v), I = v - C * D;
    const double ID = I - lane_x<2>(I), II = I - C * ID;
    const double DD = D - lane_x<2>(D), DI = D - C * DD;
    d[2] = II - lane_x<7>(II);
    m2[2] = ID - lane_x<7>(ID);
    d[1] = ID - C * m2[2];
    m2[1] = DI - lane_x<7>(DI);
    d[0] = DI - C * m2[1];
    m2[0] = DD - C * (DD - lane_x<7>(DD));
}

// First and mixed second reference derivatives of field f at Gauss point q
// of pen6 from the element's six coefficients c[m * NV + f] (see sub_group):
// d[j] = df/dxi_j, m2 = the mixed pairs (0, 1), (0, 2), (1, 2).
template <int NV>
__device__ inline void sub_eval(const double *c, const int f, const int q, double d[3], double m2[3])
{
    // A(r, s) + t B(r, s): coefficients A0, A1, A2, B0, B1, B2
    constexpr double tr[3][2] = {{1.0 / 6, 1.0 / 6}, {2.0 / 3, 1.0 / 6}, {1.0 / 6, 2.0 / 3}};
    const double r = tr[q % 3][0], sc = tr[q % 3][1], t = q < 3 ? -kGauss : kGauss;
    const double A1 = c[1 * NV + f], A2 = c[2 * NV + f], B0 = c[3 * NV + f], B1 = c[4 * NV + f], B2 = c[5 * NV + f];
    d[0] = A1 + t * B1;
    d[1] = A2 + t * B2;
    d[2] = B0 + B1 * r + B2 * sc;
    m2[0] = 0.0;
    m2[1] = B1;
    m2[2] = B2;
}

// An element's material and source, and where its results go. tau (f + mu Lap
// u + (lam + mu) grad div u) with tau = h^2 / (4 mu) is h^2 / 2 (f / (2 mu) + (Lap
// u + grad div u / (1 - 2 nu)) / 2).
template <int B>
struct SubElem {
    double E, nu, f[B];
    int64_t gp;
};

template <int MODEL, int B>
__device__ __forceinline__ SubElem<B> sub_elem(const SubArgs &A, const int32_t e)
{
    SubElem<B> r;
    r.E = 1.0;
    r.nu = 0.0;
    if constexpr (MODEL != FEA_POISSON) {
        r.nu = A.nu[e];
        if (A.young) r.E = A.young[e];
    }
#pragma unroll
    for (int c = 0; c < B; ++c) r.f[c] = A.source[(int64_t)e * B + c];
    r.gp = A.gp_ptr[e];
    return r;
}

// J^-1 (columns scaled by 1 / det) and det J by the adjugate.
__device__ __forceinline__ double sub_inverse(const double J[3][3], double Ji[3][3])
{
    Ji[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    Ji[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
    Ji[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
    Ji[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    Ji[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
    Ji[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
    Ji[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    Ji[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
    Ji[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
    const double det = J[0][0] * Ji[0][0] + J[0][1] * Ji[1][0] + J[0][2] * Ji[2][0];
    const double id = 1.0 / det;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) Ji[i][j] *= id;
    return det;
}

// M^c on the mixed pairs, H_xi(u_c) - sum_k du_c/dx_k H_xi(x_k), from the
// reference derivatives of u_c (Gu, Du) and of the coordinates (Dx).
__device__ __forceinline__ void sub_mixed(const double Gu[3], const double Du[3], const double Ji[3][3],
                                          const double Dx[3][3], double M[3])
{
    double g[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) g[k] = Gu[0] * Ji[0][k] + Gu[1] * Ji[1][k] + Gu[2] * Ji[2][k];
#pragma unroll
    for (int m = 0; m < 3; ++m) M[m] = Du[m] - (g[0] * Dx[0][m] + g[1] * Dx[1][m] + g[2] * Dx[2][m]);
}

// L(u_h) / (2 k): half of Lap u (Poisson), of Lap u + grad div u / (1 - 2 nu)
// (elasticity; gd = 1 / (1 - 2 nu)).
template <int MODEL, int B>
__device__ __forceinline__ void sub_operator(const double M[B][3], const double Ji[3][3], const double gd, double L[B])
{
    constexpr int PJ[3] = {0, 0, 1}, PL[3] = {1, 2, 2};  // mixed pairs (j, l)
    // Lap u_c = tr(J^-T M^c J^-1) = 2 sum_m M^c_m (J^-1 J^-T)_(j_m, l_m)
    double S[3];
#pragma unroll
    for (int m = 0; m < 3; ++m)
        S[m] = Ji[PJ[m]][0] * Ji[PL[m]][0] + Ji[PJ[m]][1] * Ji[PL[m]][1] + Ji[PJ[m]][2] * Ji[PL[m]][2];
#pragma unroll
    for (int i = 0; i < B; ++i) L[i] = M[i][0] * S[0] + M[i][1] * S[1] + M[i][2] * S[2];
    if constexpr (MODEL != FEA_POISSON) {
        // (grad div u)_i = sum_k (H_x u_k)_ik = sum_j Ji[j][i] W_j with
        // W_j = sum_k sum_l M^k_jl Ji[l][k] (M^k symmetric, zero diagonal)
        double W[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            W[0] += M[k][0] * Ji[1][k] + M[k][1] * Ji[2][k];
            W[1] += M[k][0] * Ji[0][k] + M[k][2] * Ji[2][k];
            W[2] += M[k][1] * Ji[0][k] + M[k][2] * Ji[1][k];
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) W[j] *= 0.5 * gd;
#pragma unroll
        for (int i = 0; i < 3; ++i) L[i] += Ji[0][i] * W[0] + Ji[1][i] * W[1] + Ji[2][i] * W[2];
    }
}

// 1 / (2 k) and 1 / (1 - 2 nu) with one division (two where E (1 - 2 nu) has no
// reciprocal).
template <int MODEL, int B>
__device__ __forceinline__ void sub_material(const SubElem<B> &el, double &ik, double &gd)
{
    ik = 0.5;
    gd = 0.0;
    if constexpr (MODEL != FEA_POISSON) {
        const double s = 1.0 - 2.0 * el.nu, r = 1.0 / (el.E * s);
        ik = (1.0 + el.nu) * (s * r);
        gd = el.E * r;
        if (!__builtin_isnormal(r)) {  // no stiffness: tau is infinite, not its product with L undefined
            ik = (1.0 + el.nu) / el.E;
            gd = 1.0 / s;
        }
    }
}

// Writes Gauss point q's values: tau (f + k L) of an element of volume V.
template <int MODEL, int B>
__device__ __forceinline__ void sub_store(const SubArgs &A, const SubElem<B> &el, const double ik, const int q,
                                          const double V, const double L[B])
{
    const double h = cbrt(V), t = 0.5 * (h * h);
    double *o = A.out + (el.gp + q) * B;
#pragma unroll
    for (int c = 0; c < B; ++c) o[c] = t * (el.f[c] * ik + L[c]);
}

// One group of up to EPW consecutive elements of a family, type-sorted
// positions p0 .. min(p0 + EPW, pend), p0 < pend. Every lane of the workgroup
// calls it. Lanes without an element follow with the group's last one and
// write nothing (hex8 and the pyramid: the exchanges want all lanes). pen6
// starts with a barrier: the previous group's readers of S are done.
template <int T, int MODEL>
__device__ void sub_group(const SubArgs &A, int64_t p0, int64_t pend, SubSmem<T, MODEL> &S)
{
    using Sm = SubSmem<T, MODEL>;
    constexpr int NN = Sm::NN, NQ = Sm::NQ, EPW = Sm::EPW, B = Sm::B, NV = Sm::NV;
    const int tid = threadIdx.x;
    const int el = tid / NQ, q = tid - el * NQ;
    const bool act = el < EPW && p0 + el < pend;
    const int64_t p = act ? p0 + el : pend - 1;
    const int32_t e = A.perm[p];
    double J[3][3], Ji[3][3];
    if constexpr (T == 0) {
        int32_t v[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) v[a] = A.pnodes[p * 4 + a];
        double X[4][3];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            X[a][0] = A.x[v[a]];
            X[a][1] = A.y[v[a]];
            X[a][2] = A.z[v[a]];
        }
        const SubElem<B> se = sub_elem<MODEL, B>(A, e);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) J[i][j] = X[j + 1][i] - X[0][i];
        const double det = sub_inverse(J, Ji);
        if (act) {
            if (!(det > 0.0)) status_min(A.status, e);
            const double L[B] = {}, ik = MODEL == FEA_POISSON ? 0.5 : (1.0 + se.nu) / se.E;
            sub_store<MODEL, B>(A, se, ik, 0, Fam<T>::W * det, L);
        }
    } else if constexpr (T != 2) {
        const int b2 = q >> 2, b0 = (q & 1) ^ b2, b1 = ((q >> 1) & 1) ^ b2;  // corner signs (see sub_tensor)
        const int low = b0 | b1 << 1, node = (T == 1 && b2) ? 4 : (low ^ (low >> 1)) + 4 * b2;
        const int32_t v = A.pnodes[p * NN + node];
        const double X[3] = {A.x[v], A.y[v], A.z[v]};
        double U[B];
#pragma unroll
        for (int c = 0; c < B; ++c) U[c] = A.u[(int64_t)v * B + c];
        const SubElem<B> se = sub_elem<MODEL, B>(A, e);
        double ik, gd;
        sub_material<MODEL, B>(se, ik, gd);
        double Dx[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) sub_tensor(X[i], J[i], Dx[i]);
        const double det = sub_inverse(J, Ji) * ((b0 ^ b1 ^ b2) ? 0.125 : -0.125);
        if (act && !(det > 0.0)) status_min(A.status, e);
        double M[B][3];
#pragma unroll
        for (int c = 0; c < B; ++c) {
            double Gu[3], Du[3];
            sub_tensor(U[c], Gu, Du);
            sub_mixed(Gu, Du, Ji, Dx, M[c]);
        }
        double L[B];
        sub_operator<MODEL, B>(M, Ji, gd, L);
        double V = det;  // all weights are 1
        V += lane_x<1>(V);
        V += lane_x<2>(V);
        V += lane_x<7>(V);
        if (act) sub_store<MODEL, B>(A, se, ik, low + 4 * b2, V, L);
    } else {
        constexpr int SE = Sm::SE;
        double *sNode = S.sNode + (el < EPW ? el : 0) * SE;
        const int32_t v = A.pnodes[p * NN + q];
        const double X[3] = {A.x[v], A.y[v], A.z[v]};
        double U[B];
#pragma unroll
        for (int c = 0; c < B; ++c) U[c] = A.u[(int64_t)v * B + c];
        const SubElem<B> se = sub_elem<MODEL, B>(A, e);
        __syncthreads();
        if (act) {
#pragma unroll
            for (int i = 0; i < 3; ++i) sNode[q * NV + i] = X[i];
#pragma unroll
            for (int c = 0; c < B; ++c) sNode[q * NV + 3 + c] = U[c];
        }
        __syncthreads();
        // lane q forms coefficient q of every field: with P_k = (v_k + v_k+3) /
        // 2, Q_k = (v_k+3 - v_k) / 2 they are A0 = P0, A1 = P1 - P0, A2 = P2 - P0,
        // B0 = Q0, B1 = Q1 - Q0, B2 = Q2 - Q0
        double cf[NV];
        {
            const int k = q % 3, top = q / 3;
#pragma unroll
            for (int f = 0; f < NV; ++f) {
                const double v0 = sNode[0 * NV + f], v3 = sNode[3 * NV + f];
                const double vk = sNode[k * NV + f], vk3 = sNode[(k + 3) * NV + f];
                const double c0 = top ? 0.5 * (v3 - v0) : 0.5 * (v0 + v3);
                const double ck = top ? 0.5 * (vk3 - vk) : 0.5 * (vk + vk3);
                cf[f] = k == 0 ? c0 : ck - c0;
            }
        }
        __syncthreads();  // every lane has read the node values
        if (act) {
#pragma unroll
            for (int f = 0; f < NV; ++f) sNode[q * NV + f] = cf[f];
        }
        __syncthreads();
        double Dx[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) sub_eval<NV>(sNode, i, q, J[i], Dx[i]);
        const double det = sub_inverse(J, Ji);
        if (act && !(det > 0.0)) status_min(A.status, e);
        S.sWd[tid] = Fam<T>::W * det;
        double M[B][3];
#pragma unroll
        for (int c = 0; c < B; ++c) {
            double Gu[3], Du[3];
            sub_eval<NV>(sNode, 3 + c, q, Gu, Du);
            sub_mixed(Gu, Du, Ji, Dx, M[c]);
        }
        double L[B], ik, gd;
        sub_material<MODEL, B>(se, ik, gd);
        sub_operator<MODEL, B>(M, Ji, gd, L);
        __syncthreads();
        if (act) {
            double V = 0.0;
#pragma unroll
            for (int k = 0; k < NQ; ++k) V += S.sWd[el * NQ + k];
            sub_store<MODEL, B>(A, se, ik, q, V, L);
        }
    }
}

template <int T, int MODEL>
__global__ void __launch_bounds__(256) k_subscale(SubArgs A)
{
    __shared__ SubSmem<T, MODEL> S;
    sub_group(A, (int64_t)blockIdx.x * SubSmem<T, MODEL>::EPW, A.n, S);
}

// All families in one launch, family t's workgroups from first[t] on.
struct SubArgs4 {
    SubArgs a[4];
    uint32_t first[4];
};

template <int MODEL>
__global__ void __launch_bounds__(256) k_subscale4(SubArgs4 A)
{
    __shared__ union {
        SubSmem<0, MODEL> s0;
        SubSmem<1, MODEL> s1;
        SubSmem<2, MODEL> s2;
        SubSmem<3, MODEL> s3;
    } S;
    const uint32_t b = blockIdx.x;
    if (b < A.first[1])
        sub_group<0, MODEL>(A.a[0], (int64_t)b * SubSmem<0, MODEL>::EPW, A.a[0].n, S.s0);
    else if (b < A.first[2])
        sub_group<1, MODEL>(A.a[1], (int64_t)(b - A.first[1]) * SubSmem<1, MODEL>::EPW, A.a[1].n, S.s1);
    else if (b < A.first[3])
        sub_group<2, MODEL>(A.a[2], (int64_t)(b - A.first[2]) * SubSmem<2, MODEL>::EPW, A.a[2].n, S.s2);
    else
        sub_group<3, MODEL>(A.a[3], (int64_t)(b - A.first[3]) * SubSmem<3, MODEL>::EPW, A.a[3].n, S.s3);
}

// Batched form: persistent workgroups of one family dequeue work items
// (mesh, family, first type-sorted position, count) from the batch's queue
// of that family and run the item's elements group by group with the
// arguments of the item's mesh, margs[mesh] (its view of family T). Every
// workgroup reaches the exit test after each item.
template <int T, int MODEL>
__global__ void __launch_bounds__(256) k_subscale_batch(const SubArgs *__restrict__ margs, const int4 *items,
                                                        const int32_t *order, int32_t n_items, int32_t *head)
{
    constexpr int EPW = SubSmem<T, MODEL>::EPW;
    __shared__ SubSmem<T, MODEL> S;
    __shared__ int32_t s_item;
    for (;;) {
        __syncthreads();  // every lane has read the previous item
        if (threadIdx.x == 0) {
            const int32_t q = atomicAdd(head, 1);
            s_item = q < n_items ? order[q] : -1;
        }
        __syncthreads();
        const int32_t it = __builtin_amdgcn_readfirstlane(s_item);
        if (it < 0) break;
        const int4 w = items[it];
        const int32_t m = __builtin_amdgcn_readfirstlane(w.x);
        const int64_t first = __builtin_amdgcn_readfirstlane(w.z), count = __builtin_amdgcn_readfirstlane(w.w);
        const SubArgs A = from_global(reinterpret_cast<const SubArgsGlobal *>(margs)[m]);
        for (int64_t g0 = 0; g0 < count; g0 += EPW) sub_group(A, first + g0, first + count, S);
    }
}

__global__ void k_sub_status_init(int32_t *s) { *s = -1; }

// Gauss points per element, in element order, from the type segmentation.
template <int T>
__global__ void k_gp_counts(const int32_t *perm, int64_t n, uint8_t *cnt)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) cnt[perm[i]] = (uint8_t)Fam<T>::NQ;
}

struct SubTmp {
    void *p = nullptr;
    ~SubTmp() { dfree(p); }
};

static int gauss_points_prepare(fea_graph *g, hipStream_t s)
{
    if (g->gpready) return FEA_OK;
    int rc;
    const int64_t E = g->n_elems;
    if (!g->gp_ptr && (rc = dalloc((void **)&g->gp_ptr, sizeof(int64_t) * (E + 1)))) return rc;
    int64_t n_gp = 0;
    for (int t = 0; t < 4; ++t) {
        const int nq = t == 0 ? 1 : (t == 2 ? 6 : 8);
        n_gp += (g->seg[t + 1] - g->seg[t]) * nq;
    }
    if (E > 0) {
        SubTmp cnt, tmp;
        if ((rc = dalloc(&cnt.p, (size_t)E))) return rc;
        if ((rc = dalloc(&tmp.p, sizeof(int64_t) * (scan_tmp_elems(E) + 64)))) return rc;
        uint8_t *c = (uint8_t *)cnt.p;
        const int64_t n0 = g->seg[1] - g->seg[0], n1 = g->seg[2] - g->seg[1], n2 = g->seg[3] - g->seg[2],
                      n3 = g->seg[4] - g->seg[3];
        if (n0) k_gp_counts<0><<<grid_for(n0, 256), 256, 0, s>>>(g->perm + g->seg[0], n0, c);
        if (n1) k_gp_counts<1><<<grid_for(n1, 256), 256, 0, s>>>(g->perm + g->seg[1], n1, c);
        if (n2) k_gp_counts<2><<<grid_for(n2, 256), 256, 0, s>>>(g->perm + g->seg[2], n2, c);
        if (n3) k_gp_counts<3><<<grid_for(n3, 256), 256, 0, s>>>(g->perm + g->seg[3], n3, c);
        if ((rc = scan_to_ptr_u8(c, E, g->gp_ptr, (int64_t *)tmp.p, s))) return rc;
        FEA_HIP(hipGetLastError());
        // the temporaries are freed on return: wait for their readers
        FEA_HIP(hipStreamSynchronize(s));
    } else {
        FEA_HIP(hipMemsetAsync(g->gp_ptr, 0, sizeof(int64_t), s));
        FEA_HIP(hipStreamSynchronize(s));
    }
    g->n_gp = n_gp;
    g->gpready = true;
    return FEA_OK;
}

template <int T, int MODEL>
static void launch_sub(const SubArgs &a, hipStream_t s)
{
    constexpr int EPW = 256 / Fam<T>::NQ;
    if (a.n) k_subscale<T, MODEL><<<grid_for(a.n, EPW), 256, 0, s>>>(a);
}

// One launch for all families saves a launch and a partly empty last wave per
// family; its workgroups all have the registers of the pyramid's kernel (4
// waves in flight per SIMD where tet4 alone has 8), which costs more than that
// on a large mesh that is nearly all tet4 or pen6. Measured on MI355X, us a
// call, four launches -> one, elasticity / Poisson, n^3 cells in bands of the
// families: n = 8: 13.3 -> 6.2 / 11.4 -> 5.4, 16: 13.9 -> 7.2 / 11.9 -> 6.2, 32: 22 ->
// 16 / 15 -> 11, 48: 48 -> 37 / 32 -> 24, 64 (19000 workgroups): 93 -> 77 / 57 -> 48,
// 96 (64000): 287 -> 280 / 168 -> 152; hex8 and pyr5 in halves 56 (19200): 79 -> 82 /
// 42 -> 43; 98% tet4: 48 (2600): 19 -> 18 / 15 -> 13, 64 (6200): 34 -> 33 / 26 -> 23,
// 96 (20900): 114 -> 120 / 69 -> 69; 98% pen6: 48 (5200): 36 -> 32 / 21 -> 20, 96
// (41800): 220 -> 221 / 110 -> 115.
constexpr int64_t kSubFuse = 32768, kSubFuseLopsided = 4096;  // workgroups

template <int MODEL>
static void run_sub(const fea_graph *g, const SubArgs &a, hipStream_t s)
{
    SubArgs4 q;
    int64_t wgs = 0, most = 0;
    int fams = 0;
    for (int t = 0; t < 4; ++t) {
        const int epw = 256 / (t == 0 ? 1 : t == 2 ? 6 : 8);
        q.a[t] = a;
        q.a[t].n = g->seg[t + 1] - g->seg[t];
        q.a[t].perm = g->perm + g->seg[t];
        q.a[t].pnodes = g->pnodes + g->node_base[t];
        q.first[t] = (uint32_t)wgs;
        const int64_t w = (q.a[t].n + epw - 1) / epw;
        wgs += w;
        most = std::max(most, w);
        if (w) ++fams;
    }
    // lopsided: one family has more than three quarters of the workgroups
    if (fams > 1 && wgs <= (most > wgs / 4 * 3 ? kSubFuseLopsided : kSubFuse)) {
        k_subscale4<MODEL><<<(unsigned)wgs, 256, 0, s>>>(q);
        return;
    }
    // the costliest family first, so the cheap launches fill the tail
    launch_sub<1, MODEL>(q.a[1], s);
    launch_sub<3, MODEL>(q.a[3], s);
    launch_sub<2, MODEL>(q.a[2], s);
    launch_sub<0, MODEL>(q.a[0], s);
}

}  // namespace fea

using namespace fea;

extern "C" int fea_graph_gauss_points(const fea_graph *gc, int64_t *n_points, int64_t *gp_ptr, hipStream_t stream)
{
    clear_error();
    fea_graph *g = const_cast<fea_graph *>(gc);
    if (!g) return set_error(FEA_EINVAL, "graph is required");
    int dev = 0;
    FEA_HIP(hipGetDevice(&dev));
    if (dev != g->device) return set_error(FEA_EINVAL, "graph lives on device %d, current is %d", g->device, dev);
    int rc = gauss_points_prepare(g, stream);
    if (rc) return rc;
    if (n_points) *n_points = g->n_gp;
    if (gp_ptr)
        FEA_HIP(hipMemcpyAsync(gp_ptr, g->gp_ptr, sizeof(int64_t) * (g->n_elems + 1), hipMemcpyDeviceToDevice,
                               stream));
    return FEA_OK;
}

extern "C" int fea_subscale(const fea_graph *gc, const double *x, const double *y, const double *z,
                            const fea_material *mat, const double *u, const double *source,
                            hipStream_t stream, double *out, int32_t *status)
{
    clear_error();
    fea_graph *g = const_cast<fea_graph *>(gc);
    if (!g || !mat) return set_error(FEA_EINVAL, "graph and material are required");
    if (mat->model != FEA_POISSON && mat->model != FEA_ELASTIC)
        return set_error(FEA_EINVAL, "unknown model %d", mat->model);
    if (mat->nh_flag) return set_error(FEA_EINVAL, "the subgrid scale is defined for the linear models only");
    if (g->n_elems > 0) {
        if (!x || !y || !z || !u || !source || !out) return set_error(FEA_EINVAL, "NULL array argument");
        if (mat->model == FEA_ELASTIC && !mat->nu) return set_error(FEA_EINVAL, "nu is required");
    }
    int dev = 0;
    FEA_HIP(hipGetDevice(&dev));
    if (dev != g->device) return set_error(FEA_EINVAL, "graph lives on device %d, current is %d", g->device, dev);
    int rc;
    if ((rc = gauss_points_prepare(g, stream))) return rc;

    int32_t *st = status;
    if (!st) {
        static thread_local int32_t *own[64] = {nullptr};
        if (!own[dev] && (rc = dalloc((void **)&own[dev], sizeof(int32_t)))) return rc;
        st = own[dev];
    }
    k_sub_status_init<<<1, 1, 0, stream>>>(st);
    if (g->n_elems > 0) {
        SubArgs a = {};
        a.x = x; a.y = y; a.z = z;
        a.u = u;
        a.young = mat->young;
        a.nu = mat->nu;
        a.source = source;
        a.gp_ptr = g->gp_ptr;
        a.out = out;
        a.status = st;
        if (mat->model == FEA_POISSON)
            run_sub<FEA_POISSON>(g, a, stream);
        else
            run_sub<FEA_ELASTIC>(g, a, stream);
    }
    FEA_HIP(hipGetLastError());
    return FEA_OK;
}

// ------------------------------------------------------------------ //
// Batched subgrid scale: the batch's work items from its device queues. //
// ------------------------------------------------------------------ //
namespace fea {

__global__ void k_sub_batch_begin(int32_t *head, int32_t *status, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < 4) head[i] = 0;
    if (i < n) status[i] = -1;
}

// Resident workgroups of the batched kernel of family T on a device.
template <int T, int MODEL>
static int sub_batch_workers(int dev, int64_t *out)
{
    static int64_t cache[64] = {0};
    if (dev < 0 || dev >= 64) return set_error(FEA_EINVAL, "device index %d unsupported", dev);
    if (!cache[dev]) {
        int per = 0, cus = 0;
        FEA_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_subscale_batch<T, MODEL>, 256, 0));
        FEA_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        cache[dev] = (int64_t)std::max(per, 1) * std::max(cus, 1);
    }
    *out = cache[dev];
    return FEA_OK;
}

template <int T>
static int launch_sub_batch(const BatchView &v, const SubArgs *d_args, hipStream_t s)
{
    const int64_t n = v.foff[T + 1] - v.foff[T];
    if (n == 0) return FEA_OK;
    int64_t w = 0;
    int rc = sub_batch_workers<T, FEA_ELASTIC>(v.device, &w);
    if (rc) return rc;
    const unsigned grid = (unsigned)std::min<int64_t>(n, w);
    k_subscale_batch<T, FEA_ELASTIC><<<grid, 256, 0, s>>>(d_args + (size_t)T * v.n_meshes, v.items,
                                                          v.order + v.foff[T], (int32_t)n, v.head + T);
    return FEA_OK;
}

// Gauss-point layouts of every mesh of a batch; off[m] = first Gauss point
// of mesh m in the concatenated output (off[n_meshes] = total).
static int batch_gauss_offsets(const BatchView &v, hipStream_t s, std::vector<int64_t> &off)
{
    off.assign((size_t)v.n_meshes + 1, 0);
    for (int m = 0; m < v.n_meshes; ++m) {
        int rc = gauss_points_prepare(v.graphs[m], s);
        if (rc) return rc;
        off[m + 1] = off[m] + v.graphs[m]->n_gp;
    }
    return FEA_OK;
}

}  // namespace fea

namespace fea {

// The subgrid scale's work items: per family, runs of 4 element groups
// (1024 tet4, 128 pyr5, 168 pen6, 128 hex8 elements) of one mesh, so that
// only a mesh's last item of a family has a partial group; the order lists
// them family by family (mesh, then position), as the queues expect.
static int sub_items_prepare(BatchView &v)
{
    if (*v.items_owner) return FEA_OK;
    const int per[4] = {4 * 256, 4 * 32, 4 * 42, 4 * 32};
    std::vector<int32_t> items;
    std::vector<int32_t> order;
    int64_t foff[5] = {0, 0, 0, 0, 0};
    for (int t = 0; t < 4; ++t) {
        foff[t] = (int64_t)order.size();
        for (int m = 0; m < v.n_meshes; ++m) {
            const fea_graph *g = v.graphs[m];
            const int64_t n = g->seg[t + 1] - g->seg[t];
            for (int64_t s0 = 0; s0 < n; s0 += per[t]) {
                order.push_back((int32_t)(items.size() / 4));
                items.push_back(m);
                items.push_back(t);
                items.push_back((int32_t)s0);
                items.push_back((int32_t)std::min<int64_t>(per[t], n - s0));
            }
        }
    }
    foff[4] = (int64_t)order.size();
    const size_t ni = order.size();
    int rc;
    int4 *d_items = nullptr;
    int32_t *d_order = nullptr;
    if ((rc = dalloc((void **)&d_items, sizeof(int4) * std::max<size_t>(ni, 1)))) return rc;
    if ((rc = dalloc((void **)&d_order, sizeof(int32_t) * std::max<size_t>(ni, 1)))) {
        dfree(d_items);
        return rc;
    }
    if (ni) {
        hipError_t e1 = hipMemcpy(d_items, items.data(), sizeof(int4) * ni, hipMemcpyHostToDevice);
        hipError_t e2 = hipMemcpy(d_order, order.data(), sizeof(int32_t) * ni, hipMemcpyHostToDevice);
        if (e1 != hipSuccess || e2 != hipSuccess) {
            dfree(d_items);
            dfree(d_order);
            return set_error(FEA_EHIP, "uploading the subgrid-scale items failed");
        }
    }
    *v.items_owner = d_items;
    *v.order_owner = d_order;
    for (int t = 0; t < 5; ++t) v.foff_owner[t] = foff[t];
    v.items = d_items;
    v.order = d_order;
    for (int t = 0; t < 5; ++t) v.foff[t] = foff[t];
    return FEA_OK;
}

}  // namespace fea

extern "C" int fea_batch_gauss_points(fea_batch *b, int64_t *offsets, hipStream_t stream)
{
    clear_error();
    if (!b) return set_error(FEA_EINVAL, "batch is required");
    BatchView v;
    int rc = batch_view(b, &v);
    if (rc) return rc;
    std::vector<int64_t> off;
    if ((rc = batch_gauss_offsets(v, stream, off))) return rc;
    if (offsets) std::copy(off.begin(), off.end(), offsets);
    return FEA_OK;
}

extern "C" int fea_batch_subscale(fea_batch *b, hipStream_t stream, double *out, int32_t *status)
{
    clear_error();
    if (!b) return set_error(FEA_EINVAL, "batch is required");
    BatchView v;
    int rc = batch_view(b, &v);
    if (rc) return rc;
    if (v.model != FEA_ELASTIC) return set_error(FEA_EINVAL, "the batched subgrid scale is built for FEA_ELASTIC");
    if (!status && v.n_meshes > 0) return set_error(FEA_EINVAL, "status (one int32 per mesh) is required");
    for (int m = 0; m < v.n_meshes; ++m) {
        const fea_mesh_desc &d = v.desc[m];
        if (d.nh_flag) return set_error(FEA_EINVAL, "mesh %d: the subgrid scale is defined for linear elasticity only", m);
        if (d.n_elems > 0 && (!d.u || !d.nu || !d.source || !d.x || !d.y || !d.z))
            return set_error(FEA_EINVAL, "mesh %d: u, nu, source and coordinates are required", m);
    }
    int dev = 0;
    FEA_HIP(hipGetDevice(&dev));
    if (dev != v.device) return set_error(FEA_EINVAL, "batch lives on device %d, current is %d", v.device, dev);
    std::vector<int64_t> off;
    if ((rc = batch_gauss_offsets(v, stream, off))) return rc;
    if (off.back() > 0 && !out) return set_error(FEA_EINVAL, "NULL output");
    if ((rc = sub_items_prepare(v))) return rc;
    // per-(family, mesh) arguments, rebuilt when the outputs change
    const size_t na = (size_t)4 * std::max(v.n_meshes, 1);
    if (!(v.args_key[0] == out && v.args_key[1] == status && *v.args)) {
        std::vector<SubArgs> h(na);
        for (int t = 0; t < 4; ++t)
            for (int m = 0; m < v.n_meshes; ++m) {
                const fea_mesh_desc &d = v.desc[m];
                const fea_graph *g = v.graphs[m];
                SubArgs a = {};
                a.x = d.x; a.y = d.y; a.z = d.z;
                a.u = d.u;
                a.young = d.young;
                a.nu = d.nu;
                a.source = d.source;
                a.perm = g->perm + g->seg[t];
                a.pnodes = g->pnodes + g->node_base[t];
                a.gp_ptr = g->gp_ptr;
                a.n = g->seg[t + 1] - g->seg[t];
                a.out = out + off[m] * 3;
                a.status = status + m;
                h[(size_t)t * v.n_meshes + m] = a;
            }
        // a kernel still in flight may read the previous table
        FEA_HIP(hipStreamSynchronize(stream));
        if (*v.args_cap < na) {
            dfree(*v.args);
            *v.args = nullptr;
            *v.args_cap = 0;
            if ((rc = dalloc(v.args, sizeof(SubArgs) * na))) return rc;
            *v.args_cap = na;
        }
        FEA_HIP(hipMemcpy(*v.args, h.data(), sizeof(SubArgs) * na, hipMemcpyHostToDevice));
        v.args_key[0] = out;
        v.args_key[1] = status;
    }
    const SubArgs *d_args = (const SubArgs *)*v.args;
    const int nb = (int)grid_for(std::max(v.n_meshes, 4), 256);
    k_sub_batch_begin<<<nb, 256, 0, stream>>>(v.head, status, v.n_meshes);
    if ((rc = launch_sub_batch<1>(v, d_args, stream)) || (rc = launch_sub_batch<3>(v, d_args, stream)) ||
        (rc = launch_sub_batch<2>(v, d_args, stream)) || (rc = launch_sub_batch<0>(v, d_args, stream)))
        return rc;
    FEA_HIP(hipGetLastError());
    return FEA_OK;
}
