// Segmented sums over a destination-sorted workspace: the second phase of
// the row-owner scatter (the owner of a block adds every contribution to it,
// the distribution of Section 3.2 applied to block rows) and of its
// upper-triangle form.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>

namespace fea {

// Segment k of the workspace holds the W-value contributions to output k in
// ascending element order, segments back to back: ptr[k] .. ptr[k+1] (in
// slots of W values). The segments of a workgroup therefore form one
// contiguous range, which the workgroup streams into LDS a chunk at a time
// with coalesced loads of up to 16 bytes (data must be 16-byte aligned, as
// every device allocation is); each thread then adds its (segment,
// component) pairs, one per round, from LDS in ascending order, starting
// from 0, in FP64. The sums are bitwise those of a plain left-to-right loop over the
// segment.
//
// Launch shape per workspace type: bytes per load, rounds (segments per
// thread) and LDS bytes per chunk. It streams: 5 TB/s of tile contributions.
// Measured on MI355X over row-owner workspaces (pyr5 of 40^3 cells / hex8 of
// 60^3, ms): FP64 with 8-byte loads 0.20 / 0.35, 16-byte 0.20 / 0.33, two
// rounds 0.20 / 0.33, 8 KB chunks 0.21 / 0.34; FP32, whose segments are half as
// long, 16-byte loads with four rounds 0.095 / 0.160, three 0.093 / 0.166, two
// 0.097 / 0.192.
template <typename CT>
struct SegCfg {
    static constexpr int LOAD_BYTES = 16;
    static constexpr int ROUNDS = sizeof(CT) == 8 ? 1 : 4;
    static constexpr int CHUNK_BYTES = 16384;
};

// Bytes a workspace is allocated beyond its values: a workgroup reads whole
// vectors of up to 16 bytes.
constexpr size_t kSegPad = 16;

template <int W, typename CT, int LOAD_BYTES, int CHUNK_BYTES>
struct SegStage {
    static constexpr int VEC = LOAD_BYTES / (int)sizeof(CT);    // values per load
    static constexpr int CAPV = CHUNK_BYTES / (int)sizeof(CT);  // staged values per chunk
    static constexpr int NV = CAPV / VEC;
    static constexpr int LV = NV / 256;                         // loads per thread per chunk
    static constexpr int CAPS = (CAPV - 2 * VEC) / W;           // slots per chunk (room for the alignment shift)
    // (a struct of VEC values would go through scratch memory)
    using Vec = typename std::conditional<VEC == 1, CT, CT __attribute__((ext_vector_type(VEC == 1 ? 2 : VEC)))>::type;

    // Slots base .. base + ns (0 < ns <= CAPS) of the workspace into sv, by the
    // whole workgroup; returns the place of the first one's value 0 in sv.
    // Whole vectors are read, so up to VEC - 1 values on either side of the
    // range come along (the workspace is padded by one vector, see
    // kSegPad). Threads beyond the range load its last vector again and drop
    // it: every load of a chunk is issued before the first is waited for,
    // without branches inside a wave. again: the previous chunk's readers have
    // to be waited for.
    static __device__ inline int load(Vec *sv, const CT *data, int64_t base, int ns, bool again)
    {
        const int tid = threadIdx.x;
        const int64_t f0 = base * W, a0 = f0 & ~(int64_t)(VEC - 1);
        const int o = (int)(f0 - a0);
        const int nvec = __builtin_amdgcn_readfirstlane((o + ns * W + VEC - 1) / VEC);
        const char *src = reinterpret_cast<const char *>(data + a0);
        char *dst = reinterpret_cast<char *>(sv);
        const unsigned last = (unsigned)(nvec - 1) * sizeof(Vec);
        Vec v[LV];
#pragma unroll
        for (int q = 0; q < LV; ++q)
            if (q * 256 < nvec) {
                const unsigned off = min((unsigned)(tid + q * 256) * (unsigned)sizeof(Vec), last);
                v[q] = *reinterpret_cast<const Vec *>(src + off);
            }
        if (again) __syncthreads();
#pragma unroll
        for (int q = 0; q < LV; ++q)
            if (q * 256 < nvec) {
                const unsigned off = (unsigned)(tid + q * 256) * (unsigned)sizeof(Vec);
                if (off <= last) *reinterpret_cast<Vec *>(dst + off) = v[q];
            }
        __syncthreads();
        return o;
    }
};

template <int W, typename CT>
using RowStage = SegStage<W, CT, SegCfg<CT>::LOAD_BYTES, SegCfg<CT>::CHUNK_BYTES>;

// Workgroup b's segments.
template <int W, typename CT, typename OT>
__device__ __forceinline__ void segsum_range(const int64_t b, int64_t n, const int64_t *ptr, const CT *data, OT *out,
                                             typename RowStage<W, CT>::Vec *sv)
{
    constexpr int TPS = 256 / W;                // segments per round
    constexpr int R = SegCfg<CT>::ROUNDS;       // rounds per workgroup
    constexpr int BPW = TPS * R;                // segments per workgroup
    using Stage = RowStage<W, CT>;
    const CT *svs = reinterpret_cast<const CT *>(sv);
    const int tid = threadIdx.x;
    const int64_t m0 = b * BPW;
    const int64_t mend = m0 + BPW < n ? m0 + BPW : n;
    const int64_t s0 = ptr[m0], s1 = ptr[mend];
    const int lb = tid / W, c = tid - lb * W;
    int64_t j0[R], j1[R];
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t m = m0 + lb + r * TPS;
        const int64_t mc = m < mend ? m : mend - 1;
        j0[r] = ptr[mc];
        j1[r] = ptr[mc + 1];
        acc[r] = 0.0;
    }
    for (int64_t base = s0; base < s1; base += Stage::CAPS) {
        const int ns = __builtin_amdgcn_readfirstlane((int)(s1 - base < Stage::CAPS ? s1 - base : Stage::CAPS));
        const int o = Stage::load(sv, data, base, ns, base != s0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t d0 = j0[r] - base, d1 = j1[r] - base;
            const int lo = d0 > 0 ? (int)(d0 < ns ? d0 : ns) : 0, hi = d1 < ns ? (int)(d1 > 0 ? d1 : 0) : ns;
            const CT *v = svs + o + lo * W + c;
            for (int j = lo; j < hi; ++j, v += W) acc[r] += (double)*v;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t m = m0 + lb + r * TPS;
        if (lb < TPS && m < mend) out[m * W + c] = (OT)acc[r];
    }
}

template <int W, typename CT, typename OT>
__global__ void __launch_bounds__(256) k_segsum(int64_t n, const int64_t *ptr, const CT *data, OT *out)
{
    __shared__ typename RowStage<W, CT>::Vec sv[RowStage<W, CT>::NV];
    segsum_range<W, CT, OT>(blockIdx.x, n, ptr, data, out, sv);
}

// The upper-triangle form's block values: output m of the upper-block list
// is block blk[m] (an upper or diagonal block), its tile sums are slots
// uptr[m] .. uptr[m+1] of the workspace (segments of consecutive m are
// adjacent), and the sum is written to block blk[m] and, transposed, to its
// lower partner lp[m] when that is >= 0; lp[m] = -(v + 1) marks the
// diagonal block of row v. With RHSD (3x3 blocks) a diagonal block's
// strictly lower entries (3, 6, 7) carry row v's right-hand side: those
// sums go to rhs[3v .. 3v+2], and entries 1, 2, 5 are written to their
// mirror positions too, so that every diagonal block is symmetric
// bitwise. Every per-output index is read at position m, so a workgroup's
// index loads are contiguous and independent of each other, and its workspace
// range (uptr[m0] .. uptr[m0 + BPW]) is known after one load; R rounds of
// 256 / W outputs per workgroup.
// What bounds it is memory: the tile sums stream in (4.6 TB/s with the stores
// left out), the lower blocks go out as scattered 72-byte pieces. Two things
// cost time beyond that. The block and partner indices were waited for before
// the segment bounds were even loaded (three dependent loads where two do);
// and the pieces of one line of lower blocks were written by workgroups on
// different XCDs (see sym_run_tile). Measured on MI355X, before -> after, ms,
// FP64 / FP32 tile sums: 96^3-cell hybrid mesh (11.6M outputs) 0.92 -> 0.80 /
// 0.70 -> 0.49, 160^3 cells (50M) 4.01 -> 3.49 FP64. The first change alone
// gave 0.96 in FP64: without the runs it only brings the scattered writers
// closer together. FP64 with 16-byte loads 0.83, two rounds 0.84; runs of 16 /
// 128 / 512 / 1024 / 2048 / 8192 ranges 0.89 / 0.82 / 0.79 / 0.80 / 0.81 / 0.87
// (160^3: - / 3.77 / 3.54 / 3.49 / 3.51 / 3.62); non-temporal loads 0.88. FP32
// with one round 0.61, three or four 0.49 and 0.50.
template <typename CT>
struct SymSegCfg {
    static constexpr int LOAD_BYTES = sizeof(CT) == 8 ? 8 : 16;
    static constexpr int ROUNDS = sizeof(CT) == 8 ? 1 : 2;
    static constexpr int CHUNK_BYTES = 8192;
};

// Position of workgroup b's outputs: runs of kSymRun consecutive ranges go to
// one XCD (workgroup b runs on XCD b % 8), the XCDs taking turns; the last,
// shorter group is split into eight equal runs. A row's lower blocks are
// written, 72 bytes at a time, by the ranges of the rows next to it; within a
// run they meet in one L2 and leave it as whole lines.
constexpr int64_t kSymRun = 1024;
__device__ inline int64_t sym_run_tile(int64_t b, int64_t nblk)
{
    const int64_t g = b / (8 * kSymRun) * (8 * kSymRun), i = b - g, left = nblk - g;
    const int64_t x = i & 7, r = i >> 3;
    if (left >= 8 * kSymRun) return g + x * kSymRun + r;
    const int64_t q = left >> 3, rem = left & 7;
    return g + x * q + (x < rem ? x : rem) + r;
}

template <int W, typename CT>
using SymStage = SegStage<W, CT, SymSegCfg<CT>::LOAD_BYTES, SymSegCfg<CT>::CHUNK_BYTES>;

// Workgroup b of nblk.
template <int W, typename CT, typename OT, bool RHSD>
__device__ __forceinline__ void segsum_sym_range(const int64_t b, const int64_t nblk, int64_t n, const int32_t *blk,
                                                 const int32_t *lp, const int64_t *uptr, const CT *data, OT *out,
                                                 OT *rhs, typename SymStage<W, CT>::Vec *sv)
{
    constexpr int TPS = 256 / W;                                      // outputs per round
    constexpr int R = SymSegCfg<CT>::ROUNDS;                          // rounds per workgroup
    constexpr int BPW = TPS * R;                                      // outputs per workgroup
    using Stage = SymStage<W, CT>;
    const CT *svs = reinterpret_cast<const CT *>(sv);
    const int tid = threadIdx.x;
    const int64_t m0 = sym_run_tile(b, nblk) * BPW;
    const int64_t mend = m0 + BPW < n ? m0 + BPW : n;
    const int64_t s0 = uptr[m0], s1 = uptr[mend];
    const int lb = tid / W, c = tid - lb * W;
    const int ct = W == 9 ? (c % 3) * 3 + c / 3 : c;
    // unconditional loads at clamped positions, nothing derived from them
    // here: the workspace loads below are issued without waiting for them
    int32_t kb[R], lw[R];
    int64_t j0[R], j1[R];
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t m = m0 + lb + r * TPS;
        const int64_t mc = m < mend ? m : mend - 1;
        kb[r] = blk[mc];
        lw[r] = lp[mc];
        j0[r] = uptr[mc];
        j1[r] = uptr[mc + 1];
        acc[r] = 0.0;
    }
    for (int64_t base = s0; base < s1; base += Stage::CAPS) {
        const int ns = __builtin_amdgcn_readfirstlane((int)(s1 - base < Stage::CAPS ? s1 - base : Stage::CAPS));
        const int o = Stage::load(sv, data, base, ns, base != s0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t d0 = j0[r] - base, d1 = j1[r] - base;
            const int lo = d0 > 0 ? (int)(d0 < ns ? d0 : ns) : 0, hi = d1 < ns ? (int)(d1 > 0 ? d1 : 0) : ns;
            const CT *v = svs + o + lo * W + c;
            for (int j = lo; j < hi; ++j, v += W) acc[r] += (double)*v;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!(lb < TPS && m0 + lb + r * TPS < mend)) continue;
        const int32_t k = kb[r], l = lw[r];
        OT *p = out + (int64_t)k * W + c;       // this component's place
        OT *q = out + (int64_t)k * W + ct;      // and its mirror's: the lower partner's, or the diagonal block's own
        if (l >= 0) q = out + (int64_t)l * W + ct;
        if (RHSD && l < 0 && (c == 3 || c == 6 || c == 7)) {
            p = rhs + (int64_t)(-l - 1) * 3 + (c == 3 ? 0 : c - 5);
            q = p;
        }
        *p = (OT)acc[r];
        if (q != p) *q = (OT)acc[r];
    }
}

template <int W, typename CT, typename OT, bool RHSD>
__global__ void __launch_bounds__(256) k_segsum_sym(int64_t n, const int32_t *blk, const int32_t *lp,
                                                    const int64_t *uptr, const CT *data, OT *out, OT *rhs)
{
    __shared__ typename SymStage<W, CT>::Vec sv[SymStage<W, CT>::NV];
    segsum_sym_range<W, CT, OT, RHSD>(blockIdx.x, gridDim.x, n, blk, lp, uptr, data, out, rhs, sv);
}

// 1x1 blocks: the right-hand side's rows and the block values in one launch,
// the right-hand side's workgroups (the first nrb) first, while its workspace,
// just written, is still in the caches. A launch of its own costs as much as
// both sums take on a small mesh.
template <typename CT, typename OT>
__global__ void __launch_bounds__(256) k_segsum_rhs_sym(int64_t nrb, int64_t nr, const int64_t *ptr, const CT *rdata,
                                                        OT *rhs, int64_t n, const int32_t *blk, const int32_t *lp,
                                                        const int64_t *uptr, const CT *data, OT *out)
{
    __shared__ union {
        typename RowStage<1, CT>::Vec r[RowStage<1, CT>::NV];
        typename SymStage<1, CT>::Vec v[SymStage<1, CT>::NV];
    } S;
    const int64_t b = blockIdx.x;
    if (b < nrb)
        segsum_range<1, CT, OT>(b, nr, ptr, rdata, rhs, S.r);
    else
        segsum_sym_range<1, CT, OT, false>(b - nrb, gridDim.x - nrb, n, blk, lp, uptr, data, out, (OT *)nullptr, S.v);
}

template <typename CT, typename OT>
inline void launch_segsum_rhs_sym(int64_t nr, const int64_t *ptr, const CT *rdata, OT *rhs, int64_t n,
                                  const int32_t *blk, const int32_t *lp, const int64_t *uptr, const CT *data, OT *out,
                                  hipStream_t s)
{
    constexpr int RPW = 256 * SegCfg<CT>::ROUNDS, BPW = 256 * SymSegCfg<CT>::ROUNDS;
    const int64_t nrb = (nr + RPW - 1) / RPW, nvb = (n + BPW - 1) / BPW;
    if (nrb + nvb)
        k_segsum_rhs_sym<CT, OT><<<(unsigned)(nrb + nvb), 256, 0, s>>>(nrb, nr, ptr, rdata, rhs, n, blk, lp, uptr, data,
                                                                     out);
}

template <int W, typename CT, typename OT>
inline void launch_segsum_sym(int64_t n, const int32_t *blk, const int32_t *lp, const int64_t *uptr,
                              const CT *data, OT *out, OT *rhs, hipStream_t s)
{
    constexpr int BPW = (256 / W) * SymSegCfg<CT>::ROUNDS;
    const unsigned grid = (unsigned)((n + BPW - 1) / BPW);
    k_segsum_sym<W, CT, OT, W == 9><<<grid, 256, 0, s>>>(n, blk, lp, uptr, data, out, rhs);
}

// out[0 .. n) = 0: the right-hand side of rows that no element touches,
// which no diagonal block carries (a kernel rather than a memset, so that
// the sequence can be captured into a graph).
template <typename OT>
__global__ void __launch_bounds__(256) k_zero(int64_t n, OT *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = (OT)0;
}

// Launch over n segments (n > 0).
template <int W, typename CT, typename OT>
inline void launch_segsum(int64_t n, const int64_t *ptr, const CT *data, OT *out, hipStream_t s)
{
    constexpr int BPW = (256 / W) * SegCfg<CT>::ROUNDS;
    const unsigned grid = (unsigned)((n + BPW - 1) / BPW);
    k_segsum<W, CT, OT><<<grid, 256, 0, s>>>(n, ptr, data, out);
}

}  // namespace fea
