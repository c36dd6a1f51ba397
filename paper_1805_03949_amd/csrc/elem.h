// Element quadrature device code shared by the one-launch-per-family
// kernels and the persistent batched kernel.
//
//
// Element arithmetic (isoparametric, Gauss quadrature):
//   J = sum_a x_a (x) dN_a/dxi, G_a = J^-T dN_a/dxi, wd = w_q detJ
//   Poisson     K_ab    += wd G_a.G_b,            f_a   += wd N_a f
//   elasticity  K_ab,ij += wd [lam h_a,i h_b,j + c2 h_a,j h_b,i
//                              + mu delta_ij G_a.G_b],  f_a,i += wd N_a f_i
// with h = G and c2 = mu for linear elasticity, and for the compressible
// neo-Hookean tangent (Section 2.2, A = Jacobian of the first Piola-Kirchhoff
// stress) F = I + sum_a u_a (x) G_a, h_a = F^-T-applied gradient
// (h_a,j = sum_J G_a,J Finv_Jj) and c2 = mu - lam ln det F. That factored
// form is algebraically identical to contracting the 81-entry tangent
// AA_iJjL = mu d_ij d_JL + (mu - lam lnJ) Finv_Jj Finv_Li + lam Finv_Ji Finv_Lj.
//
// Work layout: one 256-thread workgroup holds a tile of EPB elements of one
// family. Upper-triangle forms: EPB = 256 / (n(n+1)/2), one thread per
// (element, pair a <= b) for the matrix; the others EPB = 256 / n^2, one thread per
// (element, block a-b). Each accumulates its b x b block over the Gauss points
// from the gradients in LDS; the right-hand side takes one thread per (element,
// node). The gradients come from the geometry, with three lanes per (element,
// Gauss point) where a tile has at most 84 points, one otherwise.
#pragma once
#include <climits>
#include <cstddef>
#include <cstring>
#include <mutex>

#include "fea_internal.h"

// Multiply-adds are fused within an expression, as the source writes them, and
// not across statements: the same element code then rounds alike in every
// kernel it is inlined into, and the forms that promise equal bits (batched
// and one-mesh) keep them whatever the compiler does around it.
#pragma clang fp contract(on)

namespace fea {

struct RefTables {
    double N[4][8][8];      // [family][gauss point][node]
    double dN[4][8][8][3];  // [family][gauss point][node][reference direction]
    double w[4][8];
    double flat[4][256];    // family's dN and N as [gauss point][node][4], back to back
};

// one copy per translation unit, uploaded by that unit's ensure_tables()
static __constant__ RefTables c_ref;

template <int T>
struct Fam {
    static constexpr int NN = 4 + T + (T == 3);
    static constexpr int NQ = T == 0 ? 1 : (T == 2 ? 6 : 8);
    // weight of every Gauss point (as in the reference tables)
    static constexpr double W = (T == 0 || T == 2) ? 1.0 / 6.0 : 1.0;
};

// Reference shape functions and Gauss rules (host side, uploaded once per
// device). hex8 / pyr5: 2x2x2 Gauss, xi fastest; pen6: 3-point triangle
// rule (weights 1/6) x 2-point Gauss in t, triangle point fastest; tet4:
// one point at the centroid, weight 1/6. The pyramid is the hexahedron with
// its top face collapsed into the apex.
static void shape_host(int t, const double p[3], double N[8], double dN[8][3])
{
    static const int sg[8][3] = {{-1, -1, -1}, {1, -1, -1}, {1, 1, -1}, {-1, 1, -1},
                                 {-1, -1, 1},  {1, -1, 1},  {1, 1, 1},  {-1, 1, 1}};
    if (t == 3 || t == 1) {
        double h[8], dh[8][3];
        for (int a = 0; a < 8; ++a) {
            double fx = 0.5 * (1 + sg[a][0] * p[0]), fy = 0.5 * (1 + sg[a][1] * p[1]),
                   fz = 0.5 * (1 + sg[a][2] * p[2]);
            h[a] = fx * fy * fz;
            dh[a][0] = 0.5 * sg[a][0] * fy * fz;
            dh[a][1] = 0.5 * sg[a][1] * fx * fz;
            dh[a][2] = 0.5 * sg[a][2] * fx * fy;
        }
        int nb = t == 3 ? 8 : 4;
        for (int a = 0; a < nb; ++a) {
            N[a] = h[a];
            for (int j = 0; j < 3; ++j) dN[a][j] = dh[a][j];
        }
        if (t == 1) {
            N[4] = h[4] + h[5] + h[6] + h[7];
            for (int j = 0; j < 3; ++j) dN[4][j] = dh[4][j] + dh[5][j] + dh[6][j] + dh[7][j];
        }
    } else if (t == 2) {
        double L[3] = {1 - p[0] - p[1], p[0], p[1]};
        double dL[3][2] = {{-1, -1}, {1, 0}, {0, 1}};
        for (int a = 0; a < 6; ++a) {
            int k = a % 3;
            double s = a < 3 ? -1.0 : 1.0;
            double g = 0.5 * (1 + s * p[2]);
            N[a] = L[k] * g;
            dN[a][0] = dL[k][0] * g;
            dN[a][1] = dL[k][1] * g;
            dN[a][2] = 0.5 * s * L[k];
        }
    } else {
        N[0] = 1 - p[0] - p[1] - p[2];
        N[1] = p[0];
        N[2] = p[1];
        N[3] = p[2];
        for (int a = 0; a < 4; ++a)
            for (int j = 0; j < 3; ++j) dN[a][j] = (a == 0) ? -1.0 : (a - 1 == j ? 1.0 : 0.0);
    }
}

// Gauss rule of family t (points as above); returns the number of points.
static int rule_host(int t, double pts[8][3], double w[8])
{
    const double g = 0.57735026918962576451;  // 1/sqrt(3)
    int nq = 0;
    if (t == 0) {
        pts[0][0] = pts[0][1] = pts[0][2] = 0.25;
        w[0] = 1.0 / 6.0;
        nq = 1;
    } else if (t == 2) {
        const double tr[3][2] = {{1.0 / 6, 1.0 / 6}, {2.0 / 3, 1.0 / 6}, {1.0 / 6, 2.0 / 3}};
        for (int k = 0; k < 2; ++k)
            for (int i = 0; i < 3; ++i, ++nq) {
                pts[nq][0] = tr[i][0];
                pts[nq][1] = tr[i][1];
                pts[nq][2] = k ? g : -g;
                w[nq] = 1.0 / 6.0;
            }
    } else {
        for (int k = 0; k < 2; ++k)
            for (int j = 0; j < 2; ++j)
                for (int i = 0; i < 2; ++i, ++nq) {
                    pts[nq][0] = i ? g : -g;
                    pts[nq][1] = j ? g : -g;
                    pts[nq][2] = k ? g : -g;
                    w[nq] = 1.0;
                }
    }
    return nq;
}

static void build_tables(RefTables *R)
{
    memset(R, 0, sizeof(*R));
    for (int t = 0; t < 4; ++t) {
        double pts[8][3], w[8];
        const int nq = rule_host(t, pts, w);
        for (int q = 0; q < nq; ++q) {
            double N[8] = {0}, dN[8][3] = {{0}};
            shape_host(t, pts[q], N, dN);
            R->w[t][q] = w[q];
            for (int a = 0; a < 8; ++a) {
                R->N[t][q][a] = N[a];
                for (int j = 0; j < 3; ++j) R->dN[t][q][a][j] = dN[a][j];
            }
            const int nn = nodes_of(t);
            for (int a = 0; a < nn; ++a)
                for (int j = 0; j < 4; ++j) R->flat[t][(q * nn + a) * 4 + j] = j < 3 ? dN[a][j] : N[a];
        }
    }
}

// Reference tables on the current device; flat (may be NULL) receives the
// device address of RefTables::flat.
static int ensure_tables(const double **flat = nullptr)
{
    static std::mutex mtx;
    static const double *done[64] = {nullptr};
    int dev = 0;
    FEA_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return set_error(FEA_EINVAL, "device index %d unsupported", dev);
    std::lock_guard<std::mutex> lock(mtx);
    if (!done[dev]) {
        RefTables R;
        build_tables(&R);
        FEA_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_ref), &R, sizeof(R), 0, hipMemcpyHostToDevice));
        void *p = nullptr;
        FEA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(c_ref)));
        done[dev] = reinterpret_cast<const RefTables *>(p)->flat[0];
    }
    if (flat) *flat = done[dev];
    return FEA_OK;
}

struct ElemArgs {
    const double *ref;  // RefTables::flat
    const double *x, *y, *z;
    const int64_t *conn_ptr;
    const int32_t *conn;
    const int32_t *elems;  // element ids handled by this launch
    int64_t n;             // number of ids
    const int64_t *map_ptr;
    const int32_t *e2nnz;
    // row-owner, indexed by the launch-local element index i (type-sorted
    // order): node ids [i][a], destination of slot (a,b) [i][a*n+b] and of
    // the right-hand-side entry of node a [i][a] in the sorted workspaces
    const int32_t *pnodes;
    const int32_t *pdest;
    const int32_t *prdest;
    const double *young, *nu;
    const uint8_t *nh_flag;
    const double *u;
    const double *source;
    double *vals;    // FP64 target of ATOMIC / COLOUR
    double *rhs;
    void *contrib;   // ROWOWNER slot workspace (compute type)
    void *rcontrib;  // right-hand-side workspace (ROWOWNER, TILECOL; ROWSYM with 1x1 blocks)
    int32_t *status;
    // upper-triangle form: tile-block ranges, indexed by the launch-local
    // tile index; per (element, pair) of the launch its staged place (see
    // sym_pair); per tile-block its entries' range and workspace slot
    const int64_t *ttb_ptr;
    const uint16_t *tpos;
    const uint16_t *tb_rng;
    const int32_t *tb_slot;
    // tile-coloured form: the launch's tiles (launch-local tile indices,
    // ntiles of them), every tile-block's block and every block's lower
    // partner (-1 if none)
    const int32_t *tiles;
    int64_t ntiles;
    const int32_t *tb_blk;
    const int32_t *lpart;
};

// The element arguments as the persistent kernels read them from their
// argument table: the same layout as ElemArgs, with every pointer typed as
// addressing global memory. Pointers loaded as plain (generic) pointers are
// accessed with flat instructions, which also count against the LDS wait
// counter, so that every wait for LDS data would wait for outstanding
// global loads and stores too; pointers typed global keep global
// instructions, as kernel arguments do.
#define FEA_G(T) T __attribute__((address_space(1))) *
struct ElemArgsGlobal {
    FEA_G(const double) ref;
    FEA_G(const double) x;
    FEA_G(const double) y;
    FEA_G(const double) z;
    FEA_G(const int64_t) conn_ptr;
    FEA_G(const int32_t) conn;
    FEA_G(const int32_t) elems;
    int64_t n;
    FEA_G(const int64_t) map_ptr;
    FEA_G(const int32_t) e2nnz;
    FEA_G(const int32_t) pnodes;
    FEA_G(const int32_t) pdest;
    FEA_G(const int32_t) prdest;
    FEA_G(const double) young;
    FEA_G(const double) nu;
    FEA_G(const uint8_t) nh_flag;
    FEA_G(const double) u;
    FEA_G(const double) source;
    FEA_G(double) vals;
    FEA_G(double) rhs;
    FEA_G(void) contrib;
    FEA_G(void) rcontrib;
    FEA_G(int32_t) status;
    FEA_G(const int64_t) ttb_ptr;
    FEA_G(const uint16_t) tpos;
    FEA_G(const uint16_t) tb_rng;
    FEA_G(const int32_t) tb_slot;
    FEA_G(const int32_t) tiles;
    int64_t ntiles;
    FEA_G(const int32_t) tb_blk;
    FEA_G(const int32_t) lpart;
};
#undef FEA_G
static_assert(sizeof(ElemArgsGlobal) == sizeof(ElemArgs), "ElemArgsGlobal mirrors ElemArgs");
static_assert(offsetof(ElemArgsGlobal, lpart) == offsetof(ElemArgs, lpart), "ElemArgsGlobal mirrors ElemArgs");
static_assert(offsetof(ElemArgsGlobal, ntiles) == offsetof(ElemArgs, ntiles), "ElemArgsGlobal mirrors ElemArgs");
static_assert(offsetof(ElemArgsGlobal, n) == offsetof(ElemArgs, n), "ElemArgsGlobal mirrors ElemArgs");

// ElemArgs from an argument-table entry (its pointers converted from the
// global address space, so that the compiler keeps global accesses).
__device__ __forceinline__ ElemArgs from_global(const ElemArgsGlobal &g)
{
    ElemArgs a;
    a.ref = (const double *)g.ref;
    a.x = (const double *)g.x;
    a.y = (const double *)g.y;
    a.z = (const double *)g.z;
    a.conn_ptr = (const int64_t *)g.conn_ptr;
    a.conn = (const int32_t *)g.conn;
    a.elems = (const int32_t *)g.elems;
    a.n = g.n;
    a.map_ptr = (const int64_t *)g.map_ptr;
    a.e2nnz = (const int32_t *)g.e2nnz;
    a.pnodes = (const int32_t *)g.pnodes;
    a.pdest = (const int32_t *)g.pdest;
    a.prdest = (const int32_t *)g.prdest;
    a.young = (const double *)g.young;
    a.nu = (const double *)g.nu;
    a.nh_flag = (const uint8_t *)g.nh_flag;
    a.u = (const double *)g.u;
    a.source = (const double *)g.source;
    a.vals = (double *)g.vals;
    a.rhs = (double *)g.rhs;
    a.contrib = (void *)g.contrib;
    a.rcontrib = (void *)g.rcontrib;
    a.status = (int32_t *)g.status;
    a.ttb_ptr = (const int64_t *)g.ttb_ptr;
    a.tpos = (const uint16_t *)g.tpos;
    a.tb_rng = (const uint16_t *)g.tb_rng;
    a.tb_slot = (const int32_t *)g.tb_slot;
    a.tiles = (const int32_t *)g.tiles;
    a.ntiles = g.ntiles;
    a.tb_blk = (const int32_t *)g.tb_blk;
    a.lpart = (const int32_t *)g.lpart;
    return a;
}

// V_ROWSYM: the row-owner scatter on the upper triangle. A symmetric
// element matrix has block (b, a) equal to block (a, b) transposed, so one
// thread per local pair a <= b computes block (a, b); the workgroup's tile
// of elements then sums, per distinct upper block it touches, its lanes'
// blocks (transposed where node a > node b) in ascending lane order and
// writes one value per (tile, block) to the workspace; the reduction adds
// the tile sums of each upper block and writes lower blocks as transposes.
// V_TILECOL: the same tiles and tile sums, coloured so that the tiles of a
// colour share no node (and so no block); a tile adds its sums, and their
// transposes for the lower partners, straight into FP64 block values, one
// colour at a time (the commutative tile accumulation of Algorithm 7).
enum { V_ROWOWNER = 0, V_ATOMIC = 1, V_COLOUR = 2, V_ROWSYM = 3, V_TILECOL = 4 };

// Kernel model codes: FEA_POISSON, FEA_ELASTIC (linear elements only) and
// M_ELASTIC_NH (some elements use the neo-Hookean tangent; only these
// kernels carry the displacement and pushed-gradient LDS arrays).
constexpr int M_ELASTIC_NH = 2;
// M_ELASTIC_RES: as M_ELASTIC_NH, and the right-hand side is the Newton
// residual f_ext - f_int(u) (its own instantiations: the internal-force
// code would otherwise raise every neo-Hookean kernel's register count)
constexpr int M_ELASTIC_RES = 3;


__device__ inline double det3(const double J[3][3])
{
    return J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
           J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
           J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
}

// inverse through the adjugate
__device__ inline void inv3(const double J[3][3], double d, double Ji[3][3])
{
    double r = 1.0 / d;
    Ji[0][0] = (J[1][1] * J[2][2] - J[1][2] * J[2][1]) * r;
    Ji[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * r;
    Ji[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * r;
    Ji[1][0] = (J[1][2] * J[2][0] - J[1][0] * J[2][2]) * r;
    Ji[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * r;
    Ji[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * r;
    Ji[2][0] = (J[1][0] * J[2][1] - J[1][1] * J[2][0]) * r;
    Ji[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * r;
    Ji[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * r;
}

// The hardware hands workgroup b to XCD b % 8. Renumbering tiles so that
// each XCD receives one contiguous range keeps neighbouring elements (which
// share nodes, coordinates and destination cache lines) in the same L2.
// The thread index as a value the compiler cannot treat as loop-invariant:
// inside a persistent loop this keeps per-thread index arithmetic from being
// hoisted out of the loop and held in registers across iterations.
__device__ inline int opaque_tid()
{
    int t;
    asm volatile("v_mov_b32 %0, %1" : "=v"(t) : "v"((int)threadIdx.x));
    return t;
}

__device__ inline int64_t xcd_tile(int64_t b, int64_t nblk)
{
    const int64_t q = nblk >> 3, rem = nblk & 7, x = b & 7, r = b >> 3;
    return x * q + (x < rem ? x : rem) + r;
}

// Gradients of one element at its Gauss points, optionally padded by one
// value (see ElemSmem).
template <typename CT, int NQ, int NN, bool PAD>
struct GradRecT {
    CT v[NQ][NN][3];
};
template <typename CT, int NQ, int NN>
struct GradRecT<CT, NQ, NN, true> {
    CT v[NQ][NN][3];
    CT pad;
};

template <int T, int MODEL, int VAR, typename CT_>
struct ElemDims {
    using CT = CT_;
    static constexpr int NN = Fam<T>::NN, NQ = Fam<T>::NQ, P = NN * NN;
    // threads per element: all n*n blocks, or the n(n+1)/2 pairs a <= b
    static constexpr int PW = (VAR == V_ROWSYM || VAR == V_TILECOL) ? NN * (NN + 1) / 2 : P;
    static constexpr int EPB = 256 / PW;
    static constexpr bool ELAS = MODEL != FEA_POISSON;
    static constexpr bool NHK = MODEL == M_ELASTIC_NH || MODEL == M_ELASTIC_RES;
    static constexpr int B = ELAS ? 3 : 1;
    static constexpr int BB = B * B;
    static constexpr bool RES = MODEL == M_ELASTIC_RES && sizeof(CT) == 8;  // Newton residual
    static constexpr int EU = NHK ? EPB : 1, ER = RES ? EPB : 1;
    static constexpr bool RO = VAR == V_ROWOWNER || VAR == V_ROWSYM || VAR == V_TILECOL;

    static constexpr bool SYM = VAR == V_ROWSYM || VAR == V_TILECOL;  // tile sums
    static constexpr bool TCOL = VAR == V_TILECOL;
    static_assert(!SYM || EPB == sym_epb(T), "tile size of the upper-triangle layout");
    // a tile holds one entry per lane (the graph rejects an element that
    // repeats a node, and the layout builder checks the count), and so at
    // most as many tile-blocks
    static constexpr int MAXENT = EPB * PW;
    static constexpr int NC = NHK ? 4 : 1;
    // lanes per Gauss point in the geometry: three where the tile's points fit
    // one round of the workgroup (four waves of 21 groups), one otherwise (the
    // upper-triangle pyr5 tile: two rounds of three lanes measured 0.53, one
    // lane 0.48 ms FP64, 0.37 and 0.34 mixed)
    static constexpr int GEO_LANES = EPB * NQ <= 84 ? 3 : 1;
    // Row-owner and upper-triangle stores are staged in LDS (BB consecutive
    // threads write one block's BB contiguous values; tile sums read them)
    static constexpr bool STAGE = RO;
    // physical gradients sG[EPB][NQ][NN][3], neo-Hookean gradients pushed
    // through F^-T sH[EU][NQ][NN][3], staged blocks sK[EPB * PW * BB].
    // Per-element gradient records are padded by one value where their size
    // is a multiple of the 64 LDS banks (hex8: 192 values): the lanes of a
    // wave span two elements, whose same-position reads would otherwise
    // fall in the same banks (36% of LDS cycles lost to conflicts).
    using GradRec = GradRecT<CT, NQ, NN, (NQ * NN * 3 * (int)sizeof(CT) / 4) % 64 == 0>;
    static constexpr int NG = EPB * (int)(sizeof(GradRec) / sizeof(CT)), NHG = EU * (int)(sizeof(GradRec) / sizeof(CT)),
                         NK = STAGE ? EPB * PW * BB : 1;
    // The staged blocks overwrite the gradients (one barrier more, after
    // every lane has read them) where the gradient records are large enough
    // for the shared space to decide occupancy, and always in FP64; FP32 tet4
    // blocks get a space of their own.
    static constexpr bool ALIAS = STAGE && ((NG + NHG) * (int)sizeof(CT) > 4096 || sizeof(CT) == 8);
    static constexpr int NBUF = ALIAS ? (NG + NHG > NK ? NG + NHG : NK) : NG + NHG + NK;
    static constexpr int KOFF = ALIAS ? 0 : NG + NHG;  // where sK starts in buf
    // FP64 upper-triangle form: the per-element inputs, Gauss-point
    // coefficients and reference tables are dead once the blocks are
    // staged, and share the staged blocks' space beyond the gradients where
    // they fit
    static constexpr int SRC = RO ? EPB : 1, NLM = ELAS ? EPB : 1;
    // reference table in LDS: [gauss point][node][4], padded per point so that
    // the points a wave reads at once start in different banks
    static constexpr int RQ = NN * 4 + 2;
    static constexpr int PRE_BYTES =
        (EPB * NN * 3 + EU * NN * 3 + NLM * 2 + SRC * B + NQ * RQ + ER * NQ * 9) * 8 +
        EPB * NQ * NC * (int)sizeof(CT) + 2 * EPB * 4;
    static constexpr bool PRE_ALIAS =
        ALIAS && sizeof(CT) == 8 && (NG + NHG) * (int)sizeof(CT) + PRE_BYTES <= NBUF * (int)sizeof(CT);
};

// The LDS arrays that the upper-triangle form may overlay on the staged
// blocks, apart or overlaid.
template <typename D>
struct ElemPreArrays {
    using CT = typename D::CT;
    double sX[D::EPB][D::NN][3];
    double sU[D::EU][D::NN][3];
    double sLM[D::NLM][2];        // lam, mu of every element (elasticity)
    double sSrc[D::SRC][D::B];    // source of every element (element-tile forms)
    double sRef[D::NQ][D::RQ];    // reference gradients and shape functions of this family
    double sP[D::ER][D::NQ][9];   // residual: w detJ times the stress (P or sigma) at every Gauss point
    CT sC[D::EPB][D::NQ][D::NC];  // wd, and for neo-Hookean wd*lam, wd*c2, wd*mu
    int32_t sE[D::EPB];
    int sNH[D::EPB];
};
template <typename D, bool OVERLAY = D::PRE_ALIAS>
struct ElemPre : ElemPreArrays<D> {
    alignas(16) typename D::CT buf[D::NBUF];
};
template <typename D>
struct ElemPre<D, true> {
    using CT = typename D::CT;
    union {
        alignas(16) CT buf[D::NBUF];
        struct {
            CT pre_gradients_[D::NG + D::NHG];
            double sX[D::EPB][D::NN][3];
            double sU[D::EU][D::NN][3];
            double sLM[D::NLM][2];
            double sSrc[D::SRC][D::B];
            double sRef[D::NQ][D::RQ];
            double sP[D::ER][D::NQ][9];
            CT sC[D::EPB][D::NQ][D::NC];
            int32_t sE[D::EPB];
            int sNH[D::EPB];
        };
    };
};

template <int T, int MODEL, int VAR, typename CT>
struct ElemSmem : ElemDims<T, MODEL, VAR, CT>, ElemPre<ElemDims<T, MODEL, VAR, CT>> {
    using D = ElemDims<T, MODEL, VAR, CT>;
    int64_t sM[D::RO ? 1 : D::EPB];   // first slot of each element
    int64_t sCP[D::RO ? 1 : D::EPB];  // first conn position of each element
    int32_t sD[D::STAGE && !D::SYM ? D::EPB * D::PW : 1];
    // per tile-block its workspace slot (tile-coloured: its block), its first
    // entry and entries - 1
    struct alignas(8) TileBlock {
        int32_t slot;
        uint32_t rng;
    } sTb[D::SYM ? D::MAXENT : 1];
    int32_t sLp[D::TCOL ? D::MAXENT : 1];    // tile-coloured: lower partner of every tile-block's block
};

// Waves per SIMD that the LDS of one 256-thread workgroup (one wave per
// SIMD) and the extra bytes of a kernel leave room for on a 160 KB CU, at
// most 8: the occupancy a kernel's register budget should not undercut.
template <typename Smem>
constexpr int lds_waves(int extra = 0)
{
    const int w = (160 * 1024) / (int)(sizeof(Smem) + extra);
    return w < 1 ? 1 : (w > 8 ? 8 : w);
}

// Minimum waves per SIMD asked of the element kernels: the FP64
// linear-elastic upper-triangle instances at their LDS occupancy (tet4,
// pen6 and hex8 eight waves: 64 VGPRs, which their one-tile code fits
// without spills, and their persistent code too; pyr5 six); in the
// persistent kernels also the FP64 neo-Hookean tet4 instance at five (96
// VGPRs instead of 102, no spills; hetero128 kernel 5.47 -> 5.27 ms); the
// others unbounded (a bound there spills, the FP32 hex8 and the other
// neo-Hookean instances included, and a seven-wave bound on the persistent
// pen6 and hex8 code as well: measured with the compiler's resource
// report).
template <int T, int MODEL, int VAR, typename CT>
constexpr int persistent_min_waves()
{
    using S = ElemSmem<T, MODEL, VAR, CT>;
    if (MODEL == FEA_ELASTIC && S::SYM && sizeof(CT) == 8) return lds_waves<S>(16);
    if (MODEL == M_ELASTIC_NH && S::SYM && T == 0 && sizeof(CT) == 8) return 5;
    return 1;
}

template <int T, int MODEL, int VAR, typename CT>
constexpr int one_tile_min_waves()
{
    using S = ElemSmem<T, MODEL, VAR, CT>;
    return (MODEL == FEA_ELASTIC && S::SYM && sizeof(CT) == 8) ? lds_waves<S>() : 1;
}

// Place in LDS of entry i of family T's reference table.
template <int T, int MODEL, int VAR, typename CT>
__device__ inline double &elem_ref(ElemSmem<T, MODEL, VAR, CT> &S, const int i)
{
    constexpr int R = Fam<T>::NN * 4;
    return S.sRef[i / R][i % R];
}

// Records element e in a status word, which holds the smallest element id
// recorded and, as an unsigned number, starts at its maximum: -1, the value for
// no element, so that nothing has to translate it afterwards.
__device__ inline void status_min(int32_t *status, const int32_t e)
{
    atomicMin(reinterpret_cast<uint32_t *>(status), (uint32_t)e);
}

// Lame parameters.
__device__ __forceinline__ void lame(const double E, const double nu, double lm[2])
{
    const double s = 1.0 + nu;
    lm[0] = E * nu / (s * (1.0 - 2.0 * nu));
    lm[1] = E / (2.0 * s);
}

// Lame parameters of element e (elasticity; e < 0: any).
__device__ inline void elem_lame(const ElemArgs &A, int32_t e, double lm[2])
{
    lame((e >= 0 && A.young) ? A.young[e] : 1.0, e >= 0 ? A.nu[e] : 0.25, lm);
}

// A Gauss point of family T in factored form: the 1D (hex8, pyr5) or triangle
// and 1D (pen6) factors of its shape functions. Derivatives of a field and
// gradients of the nodes then take sums over one direction after the other,
// in registers, instead of a table entry from LDS per node and direction.
template <int T>
struct GeoPoint {
    double fx[2], fy[2], fz[2];  // 1D shape functions at -1 and +1 (pen6: fz)
    double L[3];                 // pen6: triangle coordinates
};

template <int T>
__device__ __forceinline__ GeoPoint<T> geo_point(const int q)
{
    GeoPoint<T> p;
    constexpr double g = 0.57735026918962576451;  // 1/sqrt(3)
    constexpr double M = 0.5 * (1.0 - g), P = 0.5 * (1.0 + g);
    if constexpr (T == 1 || T == 3) {
        const bool bx = q & 1, by = q & 2, bz = q & 4;
        p.fx[0] = bx ? M : P;
        p.fx[1] = bx ? P : M;
        p.fy[0] = by ? M : P;
        p.fy[1] = by ? P : M;
        p.fz[0] = bz ? M : P;
        p.fz[1] = bz ? P : M;
    } else if constexpr (T == 2) {
        const bool bz = q >= 3;
        const int i = bz ? q - 3 : q;
        p.fz[0] = bz ? M : P;
        p.fz[1] = bz ? P : M;
#pragma unroll
        for (int k = 0; k < 3; ++k) p.L[k] = k == i ? 2.0 / 3.0 : 1.0 / 6.0;
    }
    return p;
}

// Reference derivatives d[j] = sum_a v(a) dN_a/dxi_j of a nodal field at the
// point.
template <int T, typename V>
__device__ __forceinline__ void geo_row(const GeoPoint<T> &p, const V &v, double d[3])
{
    if constexpr (T == 0) {
        const double v0 = v(0);
#pragma unroll
        for (int j = 0; j < 3; ++j) d[j] = v(j + 1) - v0;
    } else if constexpr (T == 2) {
        double c[3], t[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double lo = v(k), hi = v(k + 3);
            c[k] = p.fz[0] * lo + p.fz[1] * hi;
            t[k] = hi - lo;
        }
        d[0] = c[1] - c[0];
        d[1] = c[2] - c[0];
        d[2] = 0.5 * (p.L[0] * t[0] + p.L[1] * t[1] + p.L[2] * t[2]);
    } else {
        // corner (x, y) of the bottom face is node LO, of the top face LO + 4
        // (the apex for the collapsed pyramid)
        constexpr int LO[2][2] = {{0, 3}, {1, 2}};
        double vy[2], dy[2], tz[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            double c[2], t[2];
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const double lo = v(LO[x][y]), hi = v(T == 1 ? 4 : LO[x][y] + 4);
                c[y] = p.fz[0] * lo + p.fz[1] * hi;
                t[y] = hi - lo;
            }
            vy[x] = p.fy[0] * c[0] + p.fy[1] * c[1];
            dy[x] = c[1] - c[0];
            tz[x] = p.fy[0] * t[0] + p.fy[1] * t[1];
        }
        d[0] = 0.5 * (vy[1] - vy[0]);
        d[1] = 0.5 * (p.fx[0] * dy[0] + p.fx[1] * dy[1]);
        d[2] = 0.5 * (p.fx[0] * tz[0] + p.fx[1] * tz[1]);
    }
}

// out(a, sum_j c[j] dN_a/dxi_j) for every node a.
template <int T, typename Out>
__device__ __forceinline__ void geo_nodes(const GeoPoint<T> &p, const double c[3], const Out &out)
{
    if constexpr (T == 0) {
        out(0, -(c[0] + c[1] + c[2]));
#pragma unroll
        for (int j = 0; j < 3; ++j) out(j + 1, c[j]);
    } else if constexpr (T == 2) {
        const double m[3] = {-(c[0] + c[1]), c[0], c[1]}, h = 0.5 * c[2];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double t = p.L[k] * h;
            out(k, p.fz[0] * m[k] - t);
            out(k + 3, p.fz[1] * m[k] + t);
        }
    } else {
        constexpr int LO[2][2] = {{0, 3}, {1, 2}};
        const double h0 = 0.5 * c[0], h1 = 0.5 * c[1], h2 = 0.5 * c[2];
        double hx[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) hx[x] = h2 * p.fx[x];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const double m = (x ? h0 : -h0) * p.fy[y] + (y ? h1 : -h1) * p.fx[x], t = hx[x] * p.fy[y];
                out(LO[x][y], p.fz[0] * m - t);
                if constexpr (T == 3) out(LO[x][y] + 4, p.fz[1] * m + t);
            }
        if constexpr (T == 1) out(4, h2);
    }
}

// Row r of a 3x3 matrix, one row per lane of a group of three that starts at
// lane g0: column r of its cofactors, c[k] = cof(r, k) = det * inverse[k][r],
// and the determinant by this row's expansion.
__device__ __forceinline__ double geo_cofactors(const double row[3], const int g0, const int r, double c[3])
{
    const int l1 = g0 + (r == 2 ? 0 : r + 1), l2 = g0 + (r == 0 ? 2 : r - 1);
    double b[3], e[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        b[j] = __shfl(row[j], l1);
        e[j] = __shfl(row[j], l2);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) c[k] = b[(k + 1) % 3] * e[(k + 2) % 3] - b[(k + 2) % 3] * e[(k + 1) % 3];
    return row[0] * c[0] + row[1] * c[1] + row[2] * c[2];
}

// Geometry, in FP64, three lanes per (element, Gauss point), 21 such groups
// per wave (lane 63 idle, so that a group never spans two waves): lane r forms
// row r of J, takes the other two rows from its neighbours, and with them
// column r of J^-1 and component r of every node's gradient. A neo-Hookean
// point goes the same way once more: row r of F = I + (du/dxi) J^-1, column r
// of F^-1 and of J^-1 F^-1, component r of the gradients pushed through F^-T.
// For the Newton residual each point also leaves w detJ times its stress, so
// that a node's internal force is one 3x3 product per point; summed from the
// displacements at every node instead, it took a fifth of that kernel.
// (GEO_LANES = 1: the same with a point's three rows in one lane.)
// Writes the gradients and the Gauss-point coefficients.
// What bounds these kernels most is LDS: 79% of its cycles were busy for hex8
// when the reference derivatives were read from a table there and every
// lane formed the whole inverse. Per hex8 point the lanes now read 24
// coordinates and exchange 18 values, before 24 + 99 and 27. Measured on
// MI355X, element phase before -> after, ms, FP64 / mixed: tet4 (1.3M elements)
// 0.215 -> 0.194 / 0.19 -> 0.19, pen6 (1.0M) 0.55 -> 0.49 / 0.40 -> 0.38, hex8
// (885k) 0.83 -> 0.77 / 0.66 -> 0.63; Newton step of a 64^3-cell mesh with 30%
// neo-Hookean elements 0.60 -> 0.49; one lane per neo-Hookean point 0.50, and
// mixed tangent of 96^3 cells 0.95 against 0.89 with three.
template <int T, int MODEL, int VAR, typename CT>
__device__ inline void elem_geometry(const ElemArgs &A, ElemSmem<T, MODEL, VAR, CT> &S, const int tid)
{
    using Smem = ElemSmem<T, MODEL, VAR, CT>;
    constexpr int NQ = Fam<T>::NQ, EPB = Smem::EPB;
    constexpr bool NHK = Smem::NHK;
    using GradRec = typename Smem::GradRec;
    GradRec *sG = reinterpret_cast<GradRec *>(S.buf);
    GradRec *sH = reinterpret_cast<GradRec *>(S.buf + Smem::NG);
    if constexpr (Smem::GEO_LANES == 1) {
        for (int i = tid; i < EPB * NQ; i += 256) {
            const int el = i / NQ, q = i - el * NQ;
            const int32_t e = S.sE[el];
            if (e < 0) continue;
            const GeoPoint<T> pt = geo_point<T>(q);
            double J[3][3], Ji[3][3];
#pragma unroll
            for (int r = 0; r < 3; ++r) geo_row<T>(pt, [&](int a) { return S.sX[el][a][r]; }, J[r]);
            const double d = det3(J);
            if (!(d > 0.0)) status_min(A.status, e);
            inv3(J, d, Ji);
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const double c[3] = {Ji[0][r], Ji[1][r], Ji[2][r]};
                geo_nodes<T>(pt, c, [&](int a, double v) { sG[el].v[q][a][r] = (CT)v; });
            }
            const double wd = Fam<T>::W * d;
            S.sC[el][q][0] = (CT)wd;
            if constexpr (NHK) {
                const bool nh = S.sNH[el] != 0;
                if (nh || Smem::RES) {
                    const double lam = S.sLM[el][0], mu = S.sLM[el][1];
                    double H[3][3];  // du/dx
#pragma unroll
                    for (int r = 0; r < 3; ++r) {
                        double h[3];
                        geo_row<T>(pt, [&](int a) { return S.sU[el][a][r]; }, h);
#pragma unroll
                        for (int j = 0; j < 3; ++j) H[r][j] = h[0] * Ji[0][j] + h[1] * Ji[1][j] + h[2] * Ji[2][j];
                    }
                    if (nh) {
                        double Fi[3][3];
#pragma unroll
                        for (int j = 0; j < 3; ++j) H[j][j] += 1.0;  // F
                        const double jf = det3(H);
                        if (!(jf > 0.0)) status_min(A.status, e);
                        inv3(H, jf, Fi);
#pragma unroll
                        for (int r = 0; r < 3; ++r) {
                            double c[3];
#pragma unroll
                            for (int k = 0; k < 3; ++k)
                                c[k] = Ji[k][0] * Fi[0][r] + Ji[k][1] * Fi[1][r] + Ji[k][2] * Fi[2][r];
                            geo_nodes<T>(pt, c, [&](int a, double v) { sH[el].v[q][a][r] = (CT)v; });
                        }
                        const double c2 = mu - lam * log(jf);
                        S.sC[el][q][1] = (CT)(wd * lam);
                        S.sC[el][q][2] = (CT)(wd * c2);
                        S.sC[el][q][3] = (CT)(wd * mu);
                        if constexpr (Smem::RES) {
                            // P = mu F - (mu - lam ln J) F^-T
#pragma unroll
                            for (int i = 0; i < 3; ++i)
#pragma unroll
                                for (int j = 0; j < 3; ++j)
                                    S.sP[el][q][3 * i + j] = wd * (mu * H[i][j] - c2 * Fi[j][i]);
                        }
                    } else if constexpr (Smem::RES) {
                        // sigma = lam tr(H) I + mu (H + H^T)
                        const double t = lam * (H[0][0] + H[1][1] + H[2][2]);
#pragma unroll
                        for (int i = 0; i < 3; ++i)
#pragma unroll
                            for (int j = 0; j < 3; ++j)
                                S.sP[el][q][3 * i + j] = wd * ((i == j ? t : 0.0) + mu * (H[i][j] + H[j][i]));
                    }
                }
            }
        }
        return;
    }
    const int lane = tid & 63, r = lane % 3, g0 = lane - r;
    const int grp = (tid >> 6) * 21 + lane / 3;
    if (lane == 63 || grp >= EPB * NQ) return;
    const int el = grp / NQ, q = grp - el * NQ;
    const int32_t e = S.sE[el];
    if (e < 0) return;
    const GeoPoint<T> pt = geo_point<T>(q);
    double J[3], c[3], Ji[3];
    geo_row<T>(pt, [&](int a) { return S.sX[el][a][r]; }, J);
    const double d = geo_cofactors(J, g0, r, c);
    const double id = 1.0 / d;
#pragma unroll
    for (int k = 0; k < 3; ++k) Ji[k] = c[k] * id;
    geo_nodes<T>(pt, Ji, [&](int a, double v) { sG[el].v[q][a][r] = (CT)v; });
    const double wd = Fam<T>::W * d;
    if (r == 0) {
        if (!(d > 0.0)) status_min(A.status, e);
        S.sC[el][q][0] = (CT)wd;
    }
    if constexpr (NHK) {
        const bool nh = S.sNH[el] != 0;
        if (nh || Smem::RES) {
            const double lam = S.sLM[el][0], mu = S.sLM[el][1];
            double I[3][3];  // J^-1, column j from lane j of the group
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int j = 0; j < 3; ++j) I[k][j] = __shfl(Ji[k], g0 + j);
            double h[3], F[3];  // row r of du/dxi, of du/dx, then of F
            geo_row<T>(pt, [&](int a) { return S.sU[el][a][r]; }, h);
#pragma unroll
            for (int j = 0; j < 3; ++j) F[j] = h[0] * I[0][j] + h[1] * I[1][j] + h[2] * I[2][j];
            if (nh) {
                double Q[3], Fi[3];  // column r of J^-1 F^-1 and of F^-1
#pragma unroll
                for (int j = 0; j < 3; ++j) F[j] += r == j ? 1.0 : 0.0;
                const double jf = geo_cofactors(F, g0, r, c);
                const double ij = 1.0 / jf;
#pragma unroll
                for (int k = 0; k < 3; ++k) Fi[k] = c[k] * ij;
#pragma unroll
                for (int k = 0; k < 3; ++k) Q[k] = I[k][0] * Fi[0] + I[k][1] * Fi[1] + I[k][2] * Fi[2];
                geo_nodes<T>(pt, Q, [&](int a, double v) { sH[el].v[q][a][r] = (CT)v; });
                const double c2 = mu - lam * log(jf);
                if (r == 0) {
                    if (!(jf > 0.0)) status_min(A.status, e);
                    S.sC[el][q][1] = (CT)(wd * lam);
                    S.sC[el][q][2] = (CT)(wd * c2);
                    S.sC[el][q][3] = (CT)(wd * mu);
                }
                if constexpr (Smem::RES) {
                    // row r of P = mu F - (mu - lam ln J) F^-T
#pragma unroll
                    for (int j = 0; j < 3; ++j) S.sP[el][q][3 * r + j] = wd * (mu * F[j] - c2 * Fi[j]);
                }
            } else if constexpr (Smem::RES) {
                // row r of sigma = lam tr(H) I + mu (H + H^T)
                double t = 0.0, col[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double f0 = __shfl(F[0], g0 + k), f1 = __shfl(F[1], g0 + k), f2 = __shfl(F[2], g0 + k);
                    col[k] = r == 0 ? f0 : r == 1 ? f1 : f2;
                    t += k == 0 ? f0 : k == 1 ? f1 : f2;
                }
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    S.sP[el][q][3 * r + j] = wd * ((r == j ? lam * t : 0.0) + mu * (F[j] + col[j]));
            }
        }
    }
}

// Block (a, b) of element el of the tile, from the gradients in LDS.
template <int T, int MODEL, int VAR, typename CT>
__device__ inline void elem_block(const ElemSmem<T, MODEL, VAR, CT> &S, const int el, const int a, const int b,
                                  CT *K)
{
    using Smem = ElemSmem<T, MODEL, VAR, CT>;
    constexpr int NQ = Fam<T>::NQ;
    constexpr bool ELAS = Smem::ELAS, NHK = Smem::NHK;
    using GradRec = typename Smem::GradRec;
    const GradRec *sG = reinterpret_cast<const GradRec *>(S.buf);
    const GradRec *sH = reinterpret_cast<const GradRec *>(S.buf + Smem::NG);
    if constexpr (!ELAS) {
        CT acc = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            CT dot = sG[el].v[q][a][0] * sG[el].v[q][b][0] + sG[el].v[q][a][1] * sG[el].v[q][b][1] +
                     sG[el].v[q][a][2] * sG[el].v[q][b][2];
            acc += S.sC[el][q][0] * dot;
        }
        K[0] = acc;
    } else if (!NHK || !S.sNH[el]) {
        // linear: K = lam S + mu S^T + mu tr(S) I, S = sum_q wd G_a (x) G_b
        CT Sm[9];
#pragma unroll
        for (int c = 0; c < 9; ++c) Sm[c] = 0;
#pragma unroll 2
        for (int q = 0; q < NQ; ++q) {
            CT w = S.sC[el][q][0];
            CT ga[3] = {w * sG[el].v[q][a][0], w * sG[el].v[q][a][1], w * sG[el].v[q][a][2]};
            CT gb[3] = {sG[el].v[q][b][0], sG[el].v[q][b][1], sG[el].v[q][b][2]};
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) Sm[i * 3 + j] += ga[i] * gb[j];
        }
        const CT lam = (CT)S.sLM[el][0], mu = (CT)S.sLM[el][1];
        const CT tr = Sm[0] + Sm[4] + Sm[8];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                CT v = lam * Sm[i * 3 + j] + mu * Sm[j * 3 + i];
                if (i == j) v += mu * tr;
                K[i * 3 + j] = v;
            }
    } else if constexpr (NHK) {
        // neo-Hookean: K_ij = sum_q c1 h_a,i h_b,j + c2 h_a,j h_b,i + c0 d_ij G_a.G_b
        CT T1[9], T2[9], dsum = 0;
#pragma unroll
        for (int c = 0; c < 9; ++c) T1[c] = T2[c] = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            CT c1 = S.sC[el][q][1], c2 = S.sC[el][q][2], c0 = S.sC[el][q][3];
            CT ha[3] = {sH[el].v[q][a][0], sH[el].v[q][a][1], sH[el].v[q][a][2]};
            CT hb[3] = {sH[el].v[q][b][0], sH[el].v[q][b][1], sH[el].v[q][b][2]};
            CT dot = sG[el].v[q][a][0] * sG[el].v[q][b][0] + sG[el].v[q][a][1] * sG[el].v[q][b][1] +
                     sG[el].v[q][a][2] * sG[el].v[q][b][2];
            dsum += c0 * dot;
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    CT hh = ha[i] * hb[j];
                    T1[i * 3 + j] += c1 * hh;
                    T2[i * 3 + j] += c2 * hh;
                }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                CT v = T1[i * 3 + j] + T2[j * 3 + i];
                if (i == j) v += dsum;
                K[i * 3 + j] = v;
            }
    }
}

// Right-hand side of node a of element el: the body force (src, B values),
// minus, for the Newton residual, the internal force.
template <int T, int MODEL, int VAR, typename CT>
__device__ inline void elem_rhs(const ElemSmem<T, MODEL, VAR, CT> &S, const int el, const int a, const double *src,
                                CT *f)
{
    using Smem = ElemSmem<T, MODEL, VAR, CT>;
    constexpr int NQ = Fam<T>::NQ, B = Smem::B;
    using GradRec = typename Smem::GradRec;
    const GradRec *sG = reinterpret_cast<const GradRec *>(S.buf);
    CT wn = 0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) wn += S.sC[el][q][0] * (CT)S.sRef[q][a * 4 + 3];
#pragma unroll
    for (int i = 0; i < B; ++i) f[i] = wn * (CT)src[i];
    if constexpr (Smem::RES) {
        // f -= f_int_a = sum_q w detJ P grad N_a
#pragma unroll 2
        for (int q = 0; q < NQ; ++q) {
            const double *P = S.sP[el][q];
            const CT *g = sG[el].v[q][a];
#pragma unroll
            for (int i = 0; i < 3; ++i) f[i] -= P[3 * i] * g[0] + P[3 * i + 1] * g[1] + P[3 * i + 2] * g[2];
        }
    }
}

// Inputs of the cnt elements A.elems[first ..] of a position-ordered tile into
// LDS, for kernels with one wave group per kind of load. The loads form two
// levels that all waves go through together and without per-lane conditions
// (clamped indices): ids first (waves 0 and 1 an (element, node)'s node, waves 2
// and 3 an element) with the reference table, one value per thread; then
// three values behind the id: coordinates, material (wave 2), source (wave 3).
// Under per-lane conditions the compiler waits after every group of loads, and
// a wave goes through as many dependent loads as there are groups.
struct TileLevel1 {
    int32_t id;
    double ref;
};

template <int T, int MODEL, int VAR, typename CT>
__device__ __forceinline__ TileLevel1 tile_level1(const ElemArgs &A, const int64_t first, const int cnt, const int tid)
{
    using Smem = ElemSmem<T, MODEL, VAR, CT>;
    constexpr int NN = Fam<T>::NN, NQ = Fam<T>::NQ, EPB = Smem::EPB;
    static_assert(EPB * NN <= 128 && EPB <= 64 && NQ * NN * 4 <= 256, "one wave group per kind of load");
    const bool nodes = __builtin_amdgcn_readfirstlane(tid >> 6) < 2;
    const int32_t *p = nodes ? A.pnodes + first * NN : A.elems + first;
    const int l = tid & 63, lim = nodes ? cnt * NN : cnt, i = nodes ? tid : l;
    return {p[(unsigned)(i < lim ? i : 0)], A.ref[(unsigned)(T * 256 + (tid < NQ * NN * 4 ? tid : 0))]};
}

template <int T, int MODEL, int VAR, typename CT>
__device__ __forceinline__ void tile_level2(const ElemArgs &A, const int cnt, ElemSmem<T, MODEL, VAR, CT> &S,
                                            const TileLevel1 &in, const int tid)
{
    using Smem = ElemSmem<T, MODEL, VAR, CT>;
    constexpr int NN = Fam<T>::NN, NQ = Fam<T>::NQ, EPB = Smem::EPB, B = Smem::B;
    constexpr bool ELAS = Smem::ELAS, NHK = Smem::NHK;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const double *pa = A.x, *pb = A.y, *pc = A.z;
    int stride = 1;
    if (ELAS && wave == 2) {
        pa = pc = A.nu;
        pb = A.young ? A.young : A.nu;
    } else if (wave >= 2) {
        pa = A.source;
        pb = A.source + (B > 1 ? 1 : 0);
        pc = A.source + (B > 1 ? 2 : 0);
        stride = B;
    }
    const int64_t at = (int64_t)in.id * stride;
    const double va = pa[at], vb = pb[at], vc = pc[at];
    double u[3] = {0.0, 0.0, 0.0};
    int nh = 0;
    if constexpr (NHK) {
        if (wave < 2) {
#pragma unroll
            for (int c = 0; c < 3; ++c) u[c] = A.u[3 * (int64_t)in.id + c];
        } else if (A.nh_flag) {
            nh = (int)A.nh_flag[in.id];
        }
    }
    if (tid < NQ * NN * 4) elem_ref(S, tid) = in.ref;
    if (wave < 2) {
        const int el = tid / NN, a = tid - el * NN;
        if (el < cnt) {
            S.sX[el][a][0] = va;
            S.sX[el][a][1] = vb;
            S.sX[el][a][2] = vc;
            if constexpr (NHK) {
#pragma unroll
                for (int c = 0; c < 3; ++c) S.sU[el][a][c] = u[c];
            }
        }
    } else if (wave == 2) {
        if (l < EPB) {
            S.sE[l] = l < cnt ? in.id : -1;
            S.sNH[l] = nh;
            if constexpr (ELAS) lame(A.young ? vb : 1.0, va, S.sLM[l]);
        }
    } else if (l < EPB) {
        S.sSrc[l][0] = va;
        if constexpr (B == 3) {
            S.sSrc[l][1] = vb;
            S.sSrc[l][2] = vc;
        }
    }
}

// Row-owner, atomic and colour forms: the EPB elements A.elems[first ..
// first + EPB) (ids beyond A.n are skipped) with the calling workgroup's 256
// threads and LDS S; one thread per block (a, b) of every element.
template <int T, int MODEL, int VAR, typename CT>
__device__ void elem_tile_full(const ElemArgs &A, int64_t first, ElemSmem<T, MODEL, VAR, CT> &S, const int tid)
{
    using Smem = ElemSmem<T, MODEL, VAR, CT>;
    constexpr int NN = Fam<T>::NN, NQ = Fam<T>::NQ, P = NN * NN;
    constexpr int EPB = Smem::EPB, B = Smem::B, BB = Smem::BB;
    constexpr bool ELAS = Smem::ELAS, NHK = Smem::NHK, RO = Smem::RO, STAGE = Smem::STAGE;
    CT *sK = S.buf + Smem::KOFF;
    const int64_t left = A.n - first;
    const int cnt = __builtin_amdgcn_readfirstlane((int)(left < EPB ? left : EPB));  // elements of this tile
    const int pel = tid / P, p = tid - pel * P, nel = tid / NN, na = tid - nel * NN;
    const bool pact = pel < cnt, nact = nel < cnt;
    // destinations of this thread's block and right-hand-side entry
    int32_t dest = 0, rdest = 0;
    if constexpr (RO) {
        dest = A.pdest[first * P + (pact ? tid : 0)];
        rdest = A.prdest[first * NN + (nact ? tid : 0)];
        const TileLevel1 in = tile_level1<T, MODEL, VAR, CT>(A, first, cnt, tid);
        __syncthreads();  // the previous tile's readers of S are done
        tile_level2(A, cnt, S, in, tid);
        __syncthreads();
    } else {
        __syncthreads();
        if (tid < NQ * NN * 4) elem_ref(S, tid) = A.ref[T * 256 + tid];
        if (tid < EPB) {
            const int32_t e = tid < cnt ? A.elems[first + tid] : -1;
            S.sE[tid] = e;
            S.sM[tid] = e >= 0 ? A.map_ptr[e] : 0;
            S.sCP[tid] = e >= 0 ? A.conn_ptr[e] : 0;
            S.sNH[tid] = (ELAS && e >= 0 && A.nh_flag) ? (int)A.nh_flag[e] : 0;
            if constexpr (ELAS) elem_lame(A, e, S.sLM[tid]);
        }
        __syncthreads();
        if (pact) dest = A.e2nnz[S.sM[pel] + p];
        if (nact) {
            const int32_t v = A.conn[S.sCP[nel] + na];
            S.sX[nel][na][0] = A.x[v];
            S.sX[nel][na][1] = A.y[v];
            S.sX[nel][na][2] = A.z[v];
            if constexpr (NHK) {
                bool nh = S.sNH[nel] != 0 || MODEL == M_ELASTIC_RES;
                for (int c = 0; c < 3; ++c) S.sU[nel][na][c] = nh ? A.u[3 * (int64_t)v + c] : 0.0;
            }
        }
        __syncthreads();
    }

    elem_geometry(A, S, tid);
    __syncthreads();

    // element matrix: one thread per (element, block a-b)
    CT K[BB];
    if (pact) {
        elem_block(S, pel, p / NN, p % NN, K);
        if constexpr (!RO) {
            double *dst = A.vals + (int64_t)dest * BB;
#pragma unroll
            for (int c = 0; c < BB; ++c) {
                if constexpr (VAR == V_ATOMIC)
                    unsafeAtomicAdd(dst + c, (double)K[c]);
                else
                    dst[c] += (double)K[c];
            }
        }
    }

    // right-hand side: one thread per (element, node)
    if (nact) {
        double src[B];
#pragma unroll
        for (int i = 0; i < B; ++i) src[i] = RO ? S.sSrc[RO ? nel : 0][i] : A.source[(int64_t)S.sE[nel] * B + i];
        CT f[B];
        elem_rhs(S, nel, na, src, f);
        if constexpr (RO) {
            CT *dst = (CT *)A.rcontrib + (int64_t)rdest * B;
#pragma unroll
            for (int i = 0; i < B; ++i) dst[i] = f[i];
        } else {
            const int64_t v = A.conn[S.sCP[nel] + na];
            double *dst = A.rhs + v * B;
#pragma unroll
            for (int i = 0; i < B; ++i) {
                if constexpr (VAR == V_ATOMIC)
                    unsafeAtomicAdd(dst + i, (double)f[i]);
                else
                    dst[i] += (double)f[i];
            }
        }
    }

    if constexpr (STAGE) {
        // row-owner: the workspace is sorted by destination block; the blocks
        // go through LDS so that BB consecutive threads write one block
        if constexpr (Smem::ALIAS) __syncthreads();  // every lane has read what sK overwrites
        if (pact) {
            S.sD[tid] = dest;
#pragma unroll
            for (int c = 0; c < BB; ++c) sK[tid * BB + c] = K[c];
        }
        __syncthreads();
        CT *out = (CT *)A.contrib;
        // PB threads per block, W consecutive values each (see elem_tile_sym);
        // a division per value before: element phase of pure meshes, ms, FP64 /
        // mixed: tet4 0.32 -> 0.30 / 0.21 -> 0.20, pyr5 0.30 -> 0.29 / 0.21 -> 0.20,
        // pen6 0.48 -> 0.46 / 0.31 -> 0.29, hex8 0.51 -> 0.50 / 0.32 -> 0.30
        constexpr int W = sizeof(CT) == 4 ? B : 1, PB = BB / W, STEP = 256 / PB;
        typedef CT Out __attribute__((ext_vector_type(W), aligned(sizeof(CT))));
        const int b0 = tid / PB, c0 = (tid - b0 * PB) * W;
#pragma unroll 2
        for (int blk = b0 < STEP ? b0 : 256; blk < cnt * P; blk += STEP) {
            Out v;
#pragma unroll
            for (int c = 0; c < W; ++c) v[c] = sK[blk * BB + c0 + c];
            *reinterpret_cast<Out *>(out + (int64_t)S.sD[blk] * BB + c0) = v;
        }
    }
}

// Upper-triangle form (V_ROWSYM) and its tile-coloured variant (V_TILECOL):
// tile first / EPB, one thread per local pair a <= b of every element.
//
// What bounds it is latency and instruction issue, not HBM: a workgroup
// lives for a few dependent loads and a few hundred instructions. The global
// loads of a tile are therefore issued in two levels (see tile_level1), its
// pairs' places and tile-block records with the first, and nothing is loaded
// after them. With a condition around each group of loads the first wave
// went through eight dependent loads, a third to a half of the kernel's time
// (with tile sums, blocks and geometry left out, 0.34 of 1.06 ms for 885k
// hex8 and 0.24 of 0.62 ms for 1.3M pyr5).
//
// A pair's block is staged in LDS at its place in the order of the tile's
// (block, lane) entries, already transposed where node a > node b, so that the
// contributions to a tile-block are consecutive: its sum needs one read of
// the tile-block's record and then the values (before: its range, its
// entries, then the values, each read waiting for the one before).
// Measured on MI355X, element phase of pure meshes, before -> after, ms, FP64
// / mixed: tet4 (1.3M elements) 0.29 -> 0.22 / 0.25 -> 0.20, pyr5 (1.3M) 0.62
// -> 0.48 / 0.43 -> 0.37, pen6 (1.0M) 0.64 -> 0.54 / 0.48 -> 0.41, hex8 (885k)
// 1.06 -> 0.86 / 0.83 -> 0.70; 96^3-cell hybrid mesh 1.39 -> 1.12 / 1.09 ->
// 0.92 (with the factored geometry and the tile sums as they are now 1.00 /
// 0.76).
template <int T, int MODEL, int VAR, typename CT>
__device__ void elem_tile_sym(const ElemArgs &A, int64_t first, ElemSmem<T, MODEL, VAR, CT> &S, const int tid)
{
    using Smem = ElemSmem<T, MODEL, VAR, CT>;
    constexpr int NN = Fam<T>::NN;
    constexpr int PW = Smem::PW, EPB = Smem::EPB, B = Smem::B, BB = Smem::BB;
    constexpr bool TCOL = Smem::TCOL, ALIAS = Smem::ALIAS;
    // 3x3 blocks of the upper-triangle form: the right-hand side of node a
    // of an element rides in the strictly lower entries (3, 6, 7) of the
    // element's diagonal block (a, a), which symmetry makes redundant; the
    // tile sums then add it with the block values, and the block-value
    // kernel writes it out (no right-hand-side workspace, no reduction of
    // its own)
    constexpr bool RHSD = !TCOL && B == 3;
    CT *sK = S.buf + Smem::KOFF;
    const int64_t tl = first / EPB;
    const int64_t left = A.n - first;
    const int cnt = __builtin_amdgcn_readfirstlane((int)(left < EPB ? left : EPB));  // elements of this tile
    const int64_t d0 = A.ttb_ptr[tl];
    const int nd = (int)(A.ttb_ptr[tl + 1] - d0);
    const int pel = tid / PW;
    const bool pact = pel < cnt;  // this thread has a pair
    const int nel = tid / NN, na = tid - nel * NN;
    const bool nact = nel < cnt;  // and an (element, node)
    const uint16_t *tp = A.tpos + first * PW;
    const unsigned pos = tp[(unsigned)(pact ? tid : 0)];
    unsigned rpos = 0;
    int32_t rdest = 0;  // right-hand-side destination of (element, node) tid
    if constexpr (RHSD)
        rpos = tp[(unsigned)(nact ? nel * PW + ((na * (2 * NN + 1 - na)) >> 1) : 0)];  // pair (a, a)
    else
        rdest = A.prdest[first * NN + (nact ? tid : 0)];
    const TileLevel1 in = tile_level1<T, MODEL, VAR, CT>(A, first, cnt, tid);
    const unsigned td = (unsigned)(tid < nd ? tid : nd - 1);
    const uint32_t rng = (A.tb_rng + d0)[td];
    const int32_t slot = ((TCOL ? A.tb_blk : A.tb_slot) + d0)[td];
    __syncthreads();  // the previous tile's readers of S are done
    tile_level2(A, cnt, S, in, tid);
    if (tid < nd) S.sTb[tid] = {slot, rng};
    if constexpr (TCOL) {
        if (tid < nd) S.sLp[tid] = A.lpart[slot];
    }
    __syncthreads();

    elem_geometry(A, S, tid);
    __syncthreads();

    // blocks: one thread per (element, pair a <= b); right-hand side: one
    // thread per (element, node)
    CT Ks[BB];
#pragma unroll
    for (int c = 0; c < BB; ++c) Ks[c] = 0;
    const SymPair pr = sym_pair(pos);
    const bool diag = pr.a == pr.b;
    // the block at its place; a diagonal block with RHSD leaves the strictly
    // lower entries to the right-hand side
    auto stage = [&] {
        CT *k = sK + pr.place * BB;
#pragma unroll
        for (int c = 0; c < BB; ++c)
            if (c % B >= c / B) k[c] = Ks[c];
        if (!(RHSD && diag)) {
#pragma unroll
            for (int c = 0; c < BB; ++c)
                if (c % B < c / B) k[c] = Ks[c];
        }
    };
    if (pact) {
        elem_block(S, pel, pr.a, pr.b, Ks);
        if (!RHSD && diag) {
            // a diagonal block is symmetric; copying its upper entries
            // makes it so bitwise (the products G_i (w G_j) and
            // G_j (w G_i) round differently), and with it A (with
            // RHSD the block-value kernel writes the copies)
#pragma unroll
            for (int i = 0; i < B; ++i)
#pragma unroll
                for (int j = i + 1; j < B; ++j) Ks[j * B + i] = Ks[i * B + j];
        }
        if constexpr (!ALIAS) stage();
    }
    CT f[B];
    if (nact) {
        elem_rhs(S, nel, na, S.sSrc[nel], f);
        if constexpr (!RHSD) {
            CT *dst = (CT *)A.rcontrib + (int64_t)rdest * B;
#pragma unroll
            for (int i = 0; i < B; ++i) dst[i] = f[i];
        }
    }
    if constexpr (ALIAS) {
        __syncthreads();  // every lane has read the gradients that sK overwrites
        if (pact) stage();
    }
    if constexpr (RHSD) {
        if (nact) {
            CT *k = sK + sym_pair(rpos).place * BB;
            k[3] = f[0];
            k[6] = f[1];
            k[7] = f[2];
        }
    }
    __syncthreads();

    // tile sums, the block's entries added in ascending lane (element)
    // order, in FP64: PB threads per tile-block, each W consecutive values
    // written with one store, a step of the loop taking whole tile-blocks.
    // FP32: a row of the block, 12 bytes, so that a wave's store is contiguous
    // within a block (all nine by one thread left a quarter of the threads
    // idle and stored in nine passes: element phase of pure meshes, mixed, ms,
    // before -> after: hex8 0.62 -> 0.49, pen6 0.39 -> 0.35, tet4 0.19 -> 0.15,
    // pyr5 0.35 -> 0.34). FP64: one value; two or three a thread leave gaps
    // between the lanes of a store (hex8 0.77 -> 0.85 / 0.83).
    CT *out = (CT *)A.contrib;
    constexpr int W = sizeof(CT) == 4 ? B : 1, PB = BB / W, STEP = 256 / PB;
    typedef CT Out __attribute__((ext_vector_type(W), aligned(sizeof(CT))));
    const int d_first = tid / PB, c0 = (tid - d_first * PB) * W;
    for (int d = d_first < STEP ? d_first : nd; d < nd; d += STEP) {
        const auto t = S.sTb[d];
        const CT *k = sK + (t.rng & 255) * BB + c0;
        double acc[W];
#pragma unroll
        for (int c = 0; c < W; ++c) acc[c] = (double)k[c];
        for (int q = t.rng >> 8; q > 0; --q) {
            k += BB;
#pragma unroll
            for (int c = 0; c < W; ++c) acc[c] += (double)k[c];
        }
        const int64_t blk = t.slot;
        if constexpr (TCOL) {
            // blk is the block; no other tile of this colour touches it or
            // its partner
            const int64_t l = S.sLp[d];
#pragma unroll
            for (int c = 0; c < W; ++c) A.vals[blk * BB + c0 + c] += acc[c];
            if (l >= 0) {
#pragma unroll
                for (int c = 0; c < W; ++c) A.vals[l * BB + ((c0 + c) % B) * B + (c0 + c) / B] += acc[c];
            }
        } else {
            Out v;
#pragma unroll
            for (int c = 0; c < W; ++c) v[c] = (CT)acc[c];
            *reinterpret_cast<Out *>(out + blk * BB + c0) = v;
        }
    }
}

// One tile of elements in the form VAR.
template <int T, int MODEL, int VAR, typename CT>
__device__ inline void elem_tile(const ElemArgs &A, int64_t first, ElemSmem<T, MODEL, VAR, CT> &S,
                                 const int tid = threadIdx.x)
{
    if constexpr (ElemSmem<T, MODEL, VAR, CT>::SYM)
        elem_tile_sym(A, first, S, tid);
    else
        elem_tile_full(A, first, S, tid);
}

}  // namespace fea
