// Graph build: mesh validation, type segmentation, node incidence, block
// sparsity pattern, element-to-nonzero map, inverse map and greedy colouring.
//
// Definitions (paper Section 2.1.1, Algorithm 1; Section 3.2, Algorithm 5):
// a block (i, j) exists when nodes i and j share an element; e2nnz maps the
// element-matrix slot (e, a, b) to the block of (conn[e][a], conn[e][b]);
// the inverse map lists each block's slots in ascending element order;
// elements of one colour share no node.
#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstring>
#include <memory>
#include <thread>
#include <vector>

#include "fea_internal.h"
#include "host_graph.h"

namespace fea {

// ------------------------------------------------------------ validation
// Fingerprint of a validated mesh's connectivity: the sum over elements,
// modulo 2^64, of a SplitMix64-style mix of the element id, its family and
// its node ids in order (integer addition, so the result does not depend on
// the order the elements are visited in). Graph caches are checked against
// it.
__device__ inline uint64_t fp_mix(uint64_t z)
{
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// What the host needs to know of a mesh before it sizes anything.
struct MeshCheck {
    unsigned long long bad;     // first invalid element, ~0 if there is none
    unsigned long long fp;      // fingerprint (of a valid mesh)
    unsigned long long fam[4];  // elements of every family
};

// One thread per element: validity, fingerprint and family in one pass over
// the connectivity, with one addition per workgroup to each total (one per
// element to the fingerprint alone cost 0.63 ms on 0.9 M elements). fam_cnt
// (may be null): the workgroup's elements of family t at [t * gridDim + b].
__global__ void __launch_bounds__(256) k_mesh_check(int64_t n_nodes, int64_t n_elems, const uint8_t *types,
                                                    const int64_t *conn_ptr, const int32_t *conn, MeshCheck *out,
                                                    int32_t *fam_cnt)
{
    __shared__ unsigned long long part[4];
    __shared__ int wcnt[4][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    uint64_t h = 0;
    int t = 4;
    if (e < n_elems) {
        t = types[e];
        bool ok = t < 4;
        const int nn = ok ? nodes_of(t) : 0;
        const int64_t b = conn_ptr[e];
        ok = ok && (conn_ptr[e + 1] - b == nn) && b >= 0 && (e > 0 || b == 0);
        if (ok) {
            int32_t v[8];
#pragma unroll
            for (int a = 0; a < 8; ++a) v[a] = conn[b + (a < nn ? a : nn - 1)];
            h = fp_mix((uint64_t)e ^ ((uint64_t)t << 56));
#pragma unroll
            for (int a = 0; a < 8; ++a)
                if (a < nn) {
                    ok = ok && v[a] >= 0 && v[a] < n_nodes;
#pragma unroll
                    for (int c = 0; c < a; ++c) ok = ok && v[c] != v[a];
                    h = fp_mix(h ^ (uint64_t)(uint32_t)v[a]);
                }
        }
        if (!ok) atomicMin(&out->bad, (unsigned long long)e);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) h += (uint64_t)__shfl_xor((unsigned long long)h, o);
    if (lane == 0) part[wave] = h;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        const uint64_t m = __ballot(t == f);
        if (lane == 0) wcnt[wave][f] = __popcll(m);
    }
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(&out->fp, part[0] + part[1] + part[2] + part[3]);
    if (threadIdx.x < 4) {
        const int f = threadIdx.x, n = wcnt[0][f] + wcnt[1][f] + wcnt[2][f] + wcnt[3][f];
        if (n) atomicAdd(&out->fam[f], (unsigned long long)n);
        if (fam_cnt) fam_cnt[(int64_t)f * gridDim.x + blockIdx.x] = n;
    }
}

// ------------------------------------------------------ type segmentation
// Stable partition by family from the scanned per-workgroup counts (base:
// family-major, as k_mesh_check wrote them): every element's place in the
// type-sorted order (perm and its inverse epos) and, from the families'
// counts before it, its first element-matrix slot (map_ptr).
__global__ void __launch_bounds__(256) k_type_place(int64_t n_elems, const uint8_t *types, const int64_t *base,
                                                    int32_t *perm, int32_t *epos, int64_t *map_ptr)
{
    __shared__ int wcnt[4][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x, nb = gridDim.x;
    const int t = e < n_elems ? types[e] : 4;
    int before[4];  // same family, same wave, lower lane
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        const uint64_t m = __ballot(t == f);
        before[f] = __popcll(m & ((1ull << lane) - 1));
        if (lane == 0) wcnt[wave][f] = __popcll(m);
    }
    __syncthreads();
    if (e >= n_elems) return;
    int64_t slot = 0;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        int64_t p = base[f * nb + blockIdx.x] + before[f];
        for (int w = 0; w < wave; ++w) p += wcnt[w][f];
        slot += (p - base[f * nb]) * (nodes_of(f) * nodes_of(f));
        if (t == f) {
            perm[p] = (int32_t)e;
            epos[e] = (int32_t)p;
        }
    }
    map_ptr[e] = slot;
    if (e == n_elems - 1) map_ptr[n_elems] = slot + nodes_of(t) * nodes_of(t);
}

// --------------------------------------------------------- node incidence
// Per node the number of incident elements (high word) and the sum of their
// node counts, which is the number of element-matrix slots in the node's
// block row (low word); both totals stay below 2^31. The count before the
// addition is the incidence's place in the node's unsorted list.
__global__ void __launch_bounds__(256) k_node_count(int64_t n_elems, const int64_t *conn_ptr, const int32_t *conn,
                                                    unsigned long long *cnt, int32_t *place)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n_elems) return;
    const int64_t b = conn_ptr[e];
    const int nn = (int)(conn_ptr[e + 1] - b);
    int32_t v[8];
    unsigned long long old[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) v[a] = conn[b + (a < nn ? a : nn - 1)];
#pragma unroll
    for (int a = 0; a < 8; ++a)
        if (a < nn) old[a] = atomicAdd(&cnt[v[a]], (1ull << 32) | (unsigned)nn);
#pragma unroll
    for (int a = 0; a < 8; ++a)
        if (a < nn) place[b + a] = (int32_t)(old[a] >> 32);
}

__global__ void __launch_bounds__(256) k_node_fill(int64_t n_elems, const int64_t *conn_ptr, const int32_t *conn,
                                                   const int64_t *ptr2, const int32_t *place, int32_t *n2e,
                                                   uint8_t *n2a)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n_elems) return;
    const int64_t b = conn_ptr[e];
    const int nn = (int)(conn_ptr[e + 1] - b);
    int32_t q[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const int64_t p = b + (a < nn ? a : nn - 1);
        q[a] = (int32_t)(ptr2[conn[p]] >> 32) + place[p];
    }
#pragma unroll
    for (int a = 0; a < 8; ++a)
        if (a < nn) {
            n2e[q[a]] = (int32_t)e;
            n2a[q[a]] = (uint8_t)a;
        }
}

// ------------------------------------------------------- rows of the graph
// Type-sorted layout: element at place p of the type-sorted order, family t
// with n nodes, starts at node[t] + n p (node lists) and slot[t] + n^2 p
// (element-matrix slots).
struct RowBases {
    uint32_t node[4], slot[4];  // modulo 2^32 (the places themselves are in range)
};

// One row's outputs of k_rows, all but the incidence list of the node.
struct RowOut {
    const int64_t *conn_ptr;
    const int32_t *conn;
    const int64_t *map_ptr;
    const int32_t *epos;
    int32_t *vs;      // column of every slot of the row, sorted
    int32_t *inv;     // its slots, by column, then element
    int32_t *pdest;   // type-sorted slot -> place in inv
    int32_t *pnodes;  // type-sorted node lists
    int32_t *prdest;  // type-sorted node entry -> incidence index
};

// Element of a row: first connectivity entry, node count, first slot of its
// element-matrix row, and what takes a slot to its type-sorted place.
struct RowElem {
    int32_t c0, nn, s0, dq;
};

__device__ inline RowElem row_elem(const RowOut &o, const RowBases &bs, int32_t e, int a, int64_t row, int64_t inc)
{
    RowElem r;
    r.c0 = (int32_t)o.conn_ptr[e];
    r.nn = (int32_t)o.conn_ptr[e + 1] - r.c0;
    const uint32_t p = (uint32_t)o.epos[e], nn = (uint32_t)r.nn;
    r.s0 = (int32_t)o.map_ptr[e] + a * r.nn;
    const int t = r.nn == 8 ? 3 : r.nn - 4;
    r.dq = (int32_t)(bs.slot[t] + nn * nn * p + a * nn - (uint32_t)r.s0);
    const uint32_t n = bs.node[t] + nn * p + a;
    o.pnodes[n] = (int32_t)row;
    o.prdest[n] = (int32_t)inc;
    return r;
}

__device__ inline uint32_t lane_xor(uint32_t x, int mask)
{
    switch (mask) {  // constant after unrolling
    case 1: return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, true);   // quad_perm 1 0 3 2
    case 2: return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xf, 0xf, true);   // quad_perm 2 3 0 1
    case 4:                                                             // half-row mirror, then quad mirror
        return __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf, true);
    case 8: return __builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, true);  // row rotate by 8
    case 16: return __builtin_amdgcn_ds_swizzle(x, 0x401F);
    default: return __shfl_xor((int)x, 32);
    }
}

// The row's slots sorted by (column, element): candidate f = stride j + b is
// node b of the row's j-th element (stride: the largest node count in the
// row, so that rows of one family have no gaps), key (node id, f), K keys a
// lane, sorted across the wave by a bitonic network over lane exchanges.
// Returns the number of distinct columns.
template <int K>
__device__ inline int row_sort(const RowOut &o, const RowElem &el, int ne, int stride, int32_t r0, int len)
{
    constexpr uint64_t NONE = ~0ull;
    const int lane = threadIdx.x & 63;
    const int magic = 65536 / stride + 1;  // f / stride for f < 512
    uint64_t key[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int f = lane + 64 * k, j = (f * magic) >> 16, b = f - j * stride;
        const int nn = __shfl(el.nn, j & 63), c0 = __shfl(el.c0, j & 63);
        const bool in = j < ne && b < nn;
        const int32_t v = in ? o.conn[c0 + b] : 0;
        key[k] = in ? (uint64_t)(uint32_t)v << 9 | (uint32_t)f : NONE;
    }
#pragma unroll
    for (int size = 2; size <= 64 * K; size <<= 1)
#pragma unroll
        for (int st = size >> 1; st > 0; st >>= 1) {
            if (st >= 64) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int q = k ^ (st >> 6);
                    if (q > k) {
                        const bool up = ((k * 64) & size) == 0;
                        const uint64_t x = key[k], y = key[q];
                        const bool keep = (x < y) == up;
                        key[k] = keep ? x : y;
                        key[q] = keep ? y : x;
                    }
                }
            } else {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const bool up = size >= 64 ? ((k * 64) & size) == 0 : (lane & size) == 0;
                    const uint64_t x = key[k];
                    const uint64_t y = (uint64_t)lane_xor((uint32_t)(x >> 32), st) << 32 | lane_xor((uint32_t)x, st);
                    const bool low = (lane & st) == 0;
                    key[k] = (x < y) == (low == up) ? x : y;
                }
            }
        }
    int deg = 0, last = -1;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = lane + 64 * k, f = (int)(key[k] & 511), j = (f * magic) >> 16;
        const int32_t v = (int32_t)(key[k] >> 9);
        const int32_t s = __shfl(el.s0, j & 63) + (f - j * stride);
        const int32_t q = s + __shfl(el.dq, j & 63);
        int prev = __shfl_up(v, 1);
        if (lane == 0) prev = last;
        last = __shfl(v, 63);
        if (p < len) {
            o.vs[r0 + p] = v;
            o.inv[r0 + p] = s;
            o.pdest[q] = r0 + p;
        }
        deg += __popcll(__ballot(p < len && v != prev));
    }
    return deg;
}

// One 64-lane wave per row (node) sorts the row's slots by column and thereby
// makes everything that depends on the row alone: the incidence list by
// element, the columns, the inverse map and the type-sorted maps. Rows of up
// to 64 elements sort in registers: the incidence list by counting, the slots
// by a bitonic network (150 to 400 instructions; taking the smallest column
// above the last one, once per column, needs three times as many, and one
// thread per row waits for every scattered entry in turn). A row with more
// elements takes the columns one by one. Bound by the chain list ->
// connectivity and the scattered 4-byte stores. 96^3 hybrid mesh (0.9 M rows,
// 31 M slots), with k_row_blocks: 1.65 ms, where the one-thread-per-row
// and per-element kernels for the same maps took 17.5 ms.
__global__ void __launch_bounds__(256) k_rows(int64_t n_nodes, const int64_t *ptr2, RowOut o, RowBases bs,
                                              int64_t *n2e_ptr, int32_t *n2e, uint8_t *n2a, int32_t *deg)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_nodes) return;  // the whole wave
    const int64_t w0 = ptr2[i], w1 = ptr2[i + 1];
    const int32_t b = (int32_t)(w0 >> 32), ne = (int32_t)(w1 >> 32) - b;
    const int32_t r0 = (int32_t)(w0 & 0xffffffff), len = (int32_t)(w1 & 0xffffffff) - r0;
    if (lane == 0) {
        if (i == 0) n2e_ptr[0] = 0;
        n2e_ptr[i + 1] = w1 >> 32;
    }
    int d = 0;
    if (ne <= 64) {
        int32_t e = lane < ne ? n2e[b + lane] : INT_MAX;
        int a = lane < ne ? n2a[b + lane] : 0;
        int rank = lane < ne ? 0 : lane;
        for (int j = 0; j < ne; ++j) rank += __builtin_amdgcn_readlane(e, j) < e && lane < ne;
        e = __builtin_amdgcn_ds_permute(rank * 4, e);
        a = __builtin_amdgcn_ds_permute(rank * 4, a);
        RowElem el = {0, 0, 0, 0};
        if (lane < ne) {
            n2e[b + lane] = e;
            n2a[b + lane] = (uint8_t)a;
            el = row_elem(o, bs, e, a, i, b + lane);
        }
        const int stride = __ballot(el.nn == 8) ? 8 : __ballot(el.nn == 6) ? 6 : __ballot(el.nn == 5) ? 5 : 4;
        const int nc = ne * stride;
        if (nc <= 64) d = row_sort<1>(o, el, ne, stride, r0, len);
        else if (nc <= 128) d = row_sort<2>(o, el, ne, stride, r0, len);
        else if (nc <= 256) d = row_sort<4>(o, el, ne, stride, r0, len);
        else d = row_sort<8>(o, el, ne, stride, r0, len);
    } else {
        if (lane == 0)  // insertion sort by element
            for (int p = b + 1; p < b + ne; ++p) {
                const int32_t ke = n2e[p];
                const uint8_t ka = n2a[p];
                int q = p - 1;
                while (q >= b && n2e[q] > ke) {
                    n2e[q + 1] = n2e[q];
                    n2a[q + 1] = n2a[q];
                    --q;
                }
                n2e[q + 1] = ke;
                n2a[q + 1] = ka;
            }
        __threadfence_block();
        __builtin_amdgcn_wave_barrier();
        for (int j = lane; j < ne; j += 64) row_elem(o, bs, n2e[b + j], n2a[b + j], i, b + j);
        int32_t last = -1;
        int pos = 0;
        for (;;) {
            int32_t m = INT_MAX;  // smallest column above the last one
            for (int j = lane; j < ne; j += 64) {
                const int32_t e = n2e[b + j];
                for (int64_t p = o.conn_ptr[e]; p < o.conn_ptr[e + 1]; ++p) {
                    const int32_t v = o.conn[p];
                    m = v > last && v < m ? v : m;
                }
            }
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) {
                const int32_t y = __shfl_xor(m, x);
                m = y < m ? y : m;
            }
            if (m == INT_MAX) break;
            for (int j0 = 0; j0 < ne; j0 += 64) {  // its slots, one element per lane
                const int j = j0 + lane;
                int32_t s = -1, q = 0;
                if (j < ne) {
                    const int32_t e = n2e[b + j], a = n2a[b + j];
                    const int32_t c0 = (int32_t)o.conn_ptr[e], nn = (int32_t)o.conn_ptr[e + 1] - c0;
                    const int t = nn == 8 ? 3 : nn - 4;
                    for (int x = 0; x < nn; ++x)
                        if (o.conn[c0 + x] == m) {
                            s = (int32_t)o.map_ptr[e] + a * nn + x;
                            q = (int32_t)(bs.slot[t] + (uint32_t)(nn * nn) * (uint32_t)o.epos[e] + a * nn + x);
                        }
                }
                const uint64_t hit = __ballot(s >= 0);
                if (s >= 0) {
                    const int32_t p = r0 + pos + __popcll(hit & ((1ull << lane) - 1));
                    o.vs[p] = m;
                    o.inv[p] = s;
                    o.pdest[q] = p;
                }
                pos += __popcll(hit);
            }
            ++d;
            last = m;
        }
    }
    if (lane == 0) deg[i] = d;
}

// Of a sample of the nodes, one of every group of host::kMixedStep: how many
// belong to elements of different node counts (count[0]). The lists may come from
// a file: entries out of range are not followed (count[1] nodes have some).
static int64_t mixed_groups(int64_t n_nodes) { return (n_nodes + host::kMixedStep - 1) / host::kMixedStep; }
__global__ void __launch_bounds__(256) k_mixed_nodes(int64_t n_nodes, int64_t n_sampled, int64_t n_elems,
                                                     int64_t n_inc, const int64_t *n2e_ptr, const int32_t *n2e,
                                                     const int64_t *conn_ptr, unsigned long long *count)
{
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    bool mixed = false, bad = false;
    if (s < n_sampled) {
        const int64_t v = host::mixed_sample(s, n_nodes), b = n2e_ptr[v], e = n2e_ptr[v + 1];
        bad = b < 0 || b > e || e > n_inc;
        int64_t first = -1;
        for (int64_t p = b; p < e && !mixed && !bad; ++p) {
            const int32_t el = n2e[p];
            bad = el < 0 || el >= n_elems;
            if (bad) break;
            const int64_t nn = conn_ptr[el + 1] - conn_ptr[el];
            mixed = first >= 0 && nn != first;
            first = nn;
        }
    }
    const uint64_t m = __ballot(mixed), w = __ballot(bad);
    if (m && (threadIdx.x & 63) == 0) atomicAdd(count, (unsigned long long)__popcll(m));
    if (w && (threadIdx.x & 63) == 0) atomicAdd(count + 1, (unsigned long long)__popcll(w));
}

// With the rows' first blocks known: one wave per row turns its sorted
// columns into blocks (col, the start of every block's inverse-map list) and
// every slot's block (e2nnz).
__global__ void __launch_bounds__(256) k_row_blocks(int64_t n_nodes, const int64_t *ptr2, const int64_t *row_ptr,
                                                    const int32_t *vs, const int32_t *inv, int32_t *col,
                                                    int64_t *inv_ptr, int32_t *e2nnz)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_nodes) return;  // the whole wave
    const int32_t r0 = (int32_t)(ptr2[i] & 0xffffffff), len = (int32_t)(ptr2[i + 1] & 0xffffffff) - r0;
    int32_t k0 = (int32_t)row_ptr[i] - 1;
    for (int l0 = 0; l0 < len; l0 += 64) {
        const int l = l0 + lane;
        int32_t v = -1, prev = -1, s = 0;
        if (l < len) {
            v = vs[r0 + l];
            s = inv[r0 + l];
            if (l) prev = vs[r0 + l - 1];
        }
        const bool first = l < len && v != prev;
        const uint64_t m = __ballot(first);
        const int32_t k = k0 + __popcll(m & ((2ull << lane) - 1));
        if (first) {
            col[k] = v;
            inv_ptr[k] = r0 + l;
        }
        if (l < len) e2nnz[s] = k;
        k0 += __popcll(m);
    }
    if (i == n_nodes - 1 && lane == 0) inv_ptr[row_ptr[n_nodes]] = r0 + len;
}

// Scratch memory of one stream's work.
struct TmpBuf {
    hipStream_t s;
    void *p = nullptr;
    explicit TmpBuf(hipStream_t stream) : s(stream) {}
    ~TmpBuf()
    {
        if (p) pool_free(p, hipStreamSynchronize(s));
    }
};

// ---------------------------------------------- upper-triangle row-owner
// Block k = (i, j): its transposed partner (j, i) lies in row j (the
// pattern is structurally symmetric); upper blocks (j >= i) are their own.
// One wave per row, one lane per block, so that the binary searches of a row
// run side by side (one thread per row took them one after the other: 0.86 ms
// on a 96^3 hybrid mesh, 22 M blocks; now 0.50). flag: 1 for an upper block.
__global__ void __launch_bounds__(256) k_sym_partner(int64_t n_nodes, const int64_t *row_ptr, const int32_t *col,
                                                     int32_t *upart, int32_t *flag)
{
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_nodes) return;
    const int64_t e = row_ptr[i + 1];
    for (int64_t k = row_ptr[i] + (threadIdx.x & 63); k < e; k += 64) {
        const int32_t j = col[k];
        int32_t u = (int32_t)k;
        if (j < i) {
            int32_t lo = (int32_t)row_ptr[j], hi = (int32_t)row_ptr[j + 1] - 1;
            while (lo < hi) {
                const int32_t mid = lo + ((hi - lo) >> 1);
                if (col[mid] < i) lo = mid + 1;
                else hi = mid;
            }
            u = lo;
        }
        upart[k] = u;
        flag[k] = j >= i ? 1 : 0;
    }
}

// Lower partner of every upper block (-1 if none), and the upper blocks
// listed in CSR order (uoff = exclusive count of upper blocks before k).
__global__ void k_sym_lists(int64_t nnz, const int32_t *upart, const int64_t *uoff, int32_t *lpart,
                            int32_t *ublk)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nnz) return;
    const int32_t u = upart[k];
    if (u == k) ublk[uoff[k]] = (int32_t)k;
    else lpart[u] = (int32_t)k;
}

struct TileBases {
    int64_t seg[5], node[5], tile[5], pair[5];
};

// One workgroup per tile: the tile's contributions (one per lane) keyed by
// destination upper block, sorted by block then lane (a bitonic network over
// lane exchanges, through LDS only between waves: three stages of 36; with all
// of them in LDS, 72 barriers, a pass took 0.78 ms for the 260 k tiles of a 96^3
// hybrid mesh, now 0.53).
// Pass 1 (!WRITE) stores the distinct-block count; pass 2 writes every pair's
// place and the tile-blocks at the scanned offsets. (The graph build rejects
// an element that repeats a node, so a lane has exactly one destination.)
template <bool WRITE>
__global__ void __launch_bounds__(256) k_tile_entries(TileBases tb, const int32_t *perm, const int32_t *pnodes,
                                                      const int64_t *map_ptr, const int32_t *e2nnz,
                                                      int32_t *cnt_blk, const int64_t *ttb_ptr, uint16_t *tpos,
                                                      int32_t *tb_blk, uint16_t *tb_rng)
{
    constexpr int K = 256;
    constexpr uint64_t NONE = ~0ull;
    __shared__ uint64_t key[K];
    __shared__ int part[4];
    __shared__ uint16_t beg[K + 1];  // first entry of every tile-block
    __shared__ uint16_t word[K];     // lane -> its nodes, smaller id first
    const int tid = threadIdx.x;
    const int64_t tile = blockIdx.x;
    int t = 0;
    while (t < 3 && tile >= tb.tile[t + 1]) ++t;
    const int n = nodes_of(t), pw = n * (n + 1) / 2, epb = 256 / pw;
    const int64_t i0 = (tile - tb.tile[t]) * epb;  // first element, within the family
    const int el = tid / pw;
    const int64_t p = tb.seg[t] + i0 + el;
    uint64_t mine = NONE;
    if (el < epb && p < tb.seg[t + 1]) {
        int w = tid - el * pw, a = 0;
        while (w >= n - a) {
            w -= n - a;
            ++a;
        }
        const int b = a + w;
        const int32_t *pn = pnodes + tb.node[t] + (i0 + el) * n;
        const bool tr = pn[a] > pn[b];
        const int lo = tr ? b : a, hi = tr ? a : b;
        mine = (uint64_t)e2nnz[map_ptr[perm[p]] + lo * n + hi] << 8 | (uint64_t)tid;
        word[tid] = sym_pair_word(0, lo, hi);
    }
    uint64_t k = mine;
#pragma unroll
    for (int size = 2; size <= K; size <<= 1)
#pragma unroll
        for (int st = size >> 1; st > 0; st >>= 1) {
            uint64_t y;
            if (st >= 64) {
                __syncthreads();  // the previous exchange's readers are done
                key[tid] = k;
                __syncthreads();
                y = key[tid ^ st];
            } else {
                y = (uint64_t)lane_xor((uint32_t)(k >> 32), st) << 32 | lane_xor((uint32_t)k, st);
            }
            const bool low = (tid & st) == 0, up = (tid & size) == 0;
            k = (low == up) == (k < y) ? k : y;
        }
    __syncthreads();
    key[tid] = k;
    __syncthreads();
    // new-block flags and their scan
    const bool f = k != NONE && (tid == 0 || (k >> 8) != (key[tid - 1] >> 8));
    const uint64_t m = __ballot(f);
    const int lane = tid & 63, wave = tid >> 6;
    if (lane == 0) part[wave] = __popcll(m);
    const int nent = __syncthreads_count(k != NONE);
    int before = 0, nblk = 0;
    for (int q = 0; q < 4; ++q) {
        if (q < wave) before += part[q];
        nblk += part[q];
    }
    if constexpr (!WRITE) {
        if (tid == 0) cnt_blk[tile] = nblk;
    } else {
        const int d = before + __popcll(m & ((2ull << lane) - 1)) - 1;  // tile-block of entry tid
        if (f) beg[d] = (uint16_t)tid;
        if (tid == 0) beg[nblk] = (uint16_t)nent;
        __syncthreads();
        const int64_t d0 = ttb_ptr[tile];
        if (k != NONE) {
            const int l = (int)(k & 255);
            tpos[tb.pair[t] + i0 * pw + l] = (uint16_t)(word[l] | tid);
        }
        if (tid < nblk) {
            const int e = beg[tid];
            tb_blk[d0 + tid] = (int32_t)(key[e] >> 8);
            tb_rng[d0 + tid] = (uint16_t)(e | (beg[tid + 1] - e - 1) << 8);
        }
    }
}

// Per entry m of the upper-block list: its block's lower partner, or
// -(v + 1) for the diagonal block of row v, and the start of its workspace
// segment (uptr[nup] = the workspace length).
__global__ void k_sym_compact(int64_t nup, int64_t nnz, int64_t n_nodes, const int32_t *ublk, const int32_t *lpart,
                              const int64_t *ts_ptr, const int64_t *row_ptr, int32_t *ulp, int64_t *uptr)
{
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m < nup) {
        const int32_t k = ublk[m];
        int32_t l = lpart[k];
        if (l < 0) {
            int64_t lo = 0, hi = n_nodes - 1;  // the row holding block k
            while (lo < hi) {
                const int64_t mid = (lo + hi + 1) >> 1;
                if (row_ptr[mid] <= k) lo = mid; else hi = mid - 1;
            }
            l = -(int32_t)lo - 1;
        }
        ulp[m] = l;
        uptr[m] = ts_ptr[k];
    } else if (m == nup) {
        uptr[m] = ts_ptr[nnz];
    }
}

// Tile-blocks of every block, and each tile-block's place among them (in no
// particular order yet).
__global__ void k_tb_count(int64_t ntb, const int32_t *tb_blk, int32_t *cnt, int32_t *place)
{
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d < ntb) place[d] = atomicAdd(&cnt[tb_blk[d]], 1);
}

__global__ void k_tb_fill(int64_t ntb, const int32_t *tb_blk, const int64_t *ts_ptr, const int32_t *place, int32_t *lst)
{
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d < ntb) lst[ts_ptr[tb_blk[d]] + place[d]] = (int32_t)d;
}

// Each block's tile-blocks in ascending tile order (tile-blocks are numbered
// tile by tile), then every tile-block's workspace slot.
__global__ void k_tb_slots(int64_t nnz, const int64_t *ts_ptr, int32_t *lst, int32_t *tb_slot)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nnz) return;
    const int64_t b = ts_ptr[k], e = ts_ptr[k + 1];
    for (int64_t i = b + 1; i < e; ++i) {
        const int32_t v = lst[i];
        int64_t j = i - 1;
        while (j >= b && lst[j] > v) {
            lst[j + 1] = lst[j];
            --j;
        }
        lst[j + 1] = v;
    }
    for (int64_t i = b; i < e; ++i) tb_slot[lst[i]] = (int32_t)i;
}

int sym_prepare(fea_graph *g, hipStream_t s)
{
    constexpr int BS = 256;
    const int64_t N = g->n_nodes, nnz = g->nnz;
    int rc;
    if (g->mem[2]) {
        FEA_HIP(hipDeviceSynchronize());
        pool_free(g->mem[2], hipSuccess);
        g->mem[2] = nullptr;
    }
    g->nup = 0;
    g->ulen = 0;
    g->nent = 0;
    g->sready = false;
    g->tcready = false;
    TileBases tb;
    int64_t nt = 0, nent = 0;  // tiles; entries, one per (element, pair a <= b)
    for (int t = 0; t < 4; ++t) {
        tb.seg[t] = g->seg[t];
        tb.node[t] = g->node_base[t];
        tb.tile[t] = nt;
        tb.pair[t] = nent;
        const int epb = sym_epb(t);
        nt += (g->seg[t + 1] - g->seg[t] + epb - 1) / epb;
        nent += (g->seg[t + 1] - g->seg[t]) * (nodes_of(t) * (nodes_of(t) + 1) / 2);
    }
    tb.seg[4] = g->seg[4];
    tb.node[4] = g->node_base[4];
    tb.tile[4] = nt;
    tb.pair[4] = nent;
    for (int t = 0; t < 5; ++t) {
        g->tile_base[t] = tb.tile[t];
        g->pair_base[t] = tb.pair[t];
    }
    // upart[k] = block k itself if col >= row, else the block at the
    // transposed position; block k's tile sums are ts_ptr[k] .. ts_ptr[k+1]
    TmpBuf mem(s), big(s);
    int32_t *upart, *flag, *cblk;
    int64_t *ts_ptr, *uoff, *tptr, *tmp;
    const int64_t nscan = std::max<int64_t>(std::max<int64_t>(nnz, nt), 1);
    if ((rc = dalloc_arrays(&mem.p, {{(void **)&upart, sizeof(int32_t) * nnz},
                                     {(void **)&flag, sizeof(int32_t) * nnz},
                                     {(void **)&cblk, sizeof(int32_t) * nt},
                                     {(void **)&ts_ptr, sizeof(int64_t) * (nnz + 1)},
                                     {(void **)&uoff, sizeof(int64_t) * (nnz + 1)},
                                     {(void **)&tptr, sizeof(int64_t) * (nt + 1)},
                                     {(void **)&tmp, sizeof(int64_t) * (scan_tmp_elems(nscan) + 64)}})))
        return rc;
    // partners; tile-block counts and offsets
    int64_t nup = 0, ntb = 0;
    if (nnz) {
        k_sym_partner<<<grid_for(N, 4), 256, 0, s>>>(N, g->row_ptr, g->col, upart, flag);
        if ((rc = scan_to_ptr_i32(flag, nnz, uoff, tmp, s))) return rc;
        FEA_HIP(hipMemcpyAsync(&nup, uoff + nnz, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    }
    if (nt) {
        k_tile_entries<false><<<(unsigned)nt, 256, 0, s>>>(tb, g->perm, g->pnodes, g->map_ptr, g->e2nnz, cblk, nullptr,
                                                          nullptr, nullptr, nullptr);
        if ((rc = scan_to_ptr_i32(cblk, nt, tptr, tmp, s))) return rc;
        FEA_HIP(hipMemcpyAsync(&ntb, tptr + nt, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    } else {
        FEA_HIP(hipMemsetAsync(tptr, 0, sizeof(int64_t), s));
    }
    FEA_HIP(hipGetLastError());
    FEA_HIP(hipStreamSynchronize(s));
    if (ntb > INT32_MAX) return set_error(FEA_ERANGE, "%lld tile-blocks exceed the int32 slot range", (long long)ntb);
    if ((rc = dalloc_arrays(&g->mem[2], {{(void **)&g->lpart, sizeof(int32_t) * nnz},
                                         {(void **)&g->ublk, sizeof(int32_t) * nup},
                                         {(void **)&g->ulp, sizeof(int32_t) * nup},
                                         {(void **)&g->uptr, sizeof(int64_t) * (nup + 1)},
                                         {(void **)&g->ttb_ptr, sizeof(int64_t) * (nt + 1)},
                                         {(void **)&g->tpos, sizeof(uint16_t) * nent},
                                         {(void **)&g->tb_rng, sizeof(uint16_t) * ntb},
                                         {(void **)&g->tb_blk, sizeof(int32_t) * ntb},
                                         {(void **)&g->tb_slot, sizeof(int32_t) * ntb}})))
        return rc;
    FEA_HIP(hipMemcpyAsync(g->ttb_ptr, tptr, sizeof(int64_t) * (nt + 1), hipMemcpyDeviceToDevice, s));
    if (nnz) {
        FEA_HIP(hipMemsetAsync(g->lpart, 0xff, sizeof(int32_t) * nnz, s));
        k_sym_lists<<<grid_for(nnz, BS), BS, 0, s>>>(nnz, upart, uoff, g->lpart, g->ublk);
    }
    if (nt)
        k_tile_entries<true><<<(unsigned)nt, 256, 0, s>>>(tb, g->perm, g->pnodes, g->map_ptr, g->e2nnz, nullptr,
                                                         g->ttb_ptr, g->tpos, g->tb_blk, g->tb_rng);
    // workspace segments: per block its tile-blocks, ascending tile (listed
    // in uoff's memory, which nothing reads any more, where they fit)
    int32_t *lst = (int32_t *)uoff;
    if (ntb > 2 * (nnz + 1)) {
        if ((rc = dalloc_pool(&big.p, sizeof(int32_t) * ntb))) return rc;
        lst = (int32_t *)big.p;
    }
    if (nnz) {
        FEA_HIP(hipMemsetAsync(flag, 0, sizeof(int32_t) * nnz, s));
        // (tb_slot holds the places until k_tb_slots)
        if (ntb) k_tb_count<<<grid_for(ntb, BS), BS, 0, s>>>(ntb, g->tb_blk, flag, g->tb_slot);
        if ((rc = scan_to_ptr_i32(flag, nnz, ts_ptr, tmp, s))) return rc;
        if (ntb) {
            k_tb_fill<<<grid_for(ntb, BS), BS, 0, s>>>(ntb, g->tb_blk, ts_ptr, g->tb_slot, lst);
            k_tb_slots<<<grid_for(nnz, BS), BS, 0, s>>>(nnz, ts_ptr, lst, g->tb_slot);
        }
    } else {
        FEA_HIP(hipMemsetAsync(ts_ptr, 0, sizeof(int64_t), s));
    }
    k_sym_compact<<<grid_for(nup + 1, BS), BS, 0, s>>>(nup, nnz, N, g->ublk, g->lpart, ts_ptr, g->row_ptr, g->ulp,
                                                       g->uptr);
    FEA_HIP(hipGetLastError());
    FEA_HIP(hipStreamSynchronize(s));
    g->nup = nup;
    g->ulen = ntb;
    g->nent = nent;
    // every row an element touches has one diagonal block: nnz = 2 nup - rows
    g->sym_empty_rows = N - (2 * nup - nnz);
    g->sready = true;
    return FEA_OK;
}

// Colouring of the upper-triangle tiles, the GPU counterpart of the
// commutative multidependences of Algorithm 7: a tile's nodes are its
// elements' nodes, tiles sharing a node are neighbours, and a tile's
// priority is its neighbour count (nneig). Tiles are coloured greedily
// (first fit) in descending priority, so that the tiles of one colour
// share no node and no block, and each (family, colour) launch lists its
// tiles in descending priority too, so that the most connected tiles are
// dispatched first. On the host, one tile after the other.
int tile_colour_prepare(fea_graph *g, hipStream_t s)
{
    const int64_t N = g->n_nodes, C = g->conn_len;
    std::vector<int32_t> pn(std::max<int64_t>(C, 1));
    if (C) FEA_HIP(hipMemcpyAsync(pn.data(), g->pnodes, sizeof(int32_t) * C, hipMemcpyDeviceToHost, s));
    FEA_HIP(hipStreamSynchronize(s));
    const int64_t nt = g->tile_base[4];
    // node ranges of the tiles in pnodes (families and tiles are contiguous)
    std::vector<int64_t> ptr((size_t)nt + 1, 0);
    std::vector<uint8_t> fam((size_t)std::max<int64_t>(nt, 1), 0);
    for (int t = 0; t < 4; ++t) {
        const int n = nodes_of(t), epb = sym_epb(t);
        const int64_t ne = g->seg[t + 1] - g->seg[t];
        for (int64_t i = 0; i < g->tile_base[t + 1] - g->tile_base[t]; ++i) {
            ptr[(size_t)(g->tile_base[t] + i + 1)] = g->node_base[t] + std::min<int64_t>(ne, (i + 1) * epb) * n;
            fam[(size_t)(g->tile_base[t] + i)] = (uint8_t)t;
        }
    }
    std::vector<int32_t> nneig((size_t)std::max<int64_t>(nt, 1), 0);
    host::neighbour_counts(N, nt, ptr.data(), pn.data(), nneig.data());
    const std::vector<int64_t> order = host::priority_order(nt, nneig.data());
    std::vector<int16_t> colour((size_t)std::max<int64_t>(nt, 1), 0);
    const int64_t ncol = host::greedy_first_fit(N, nt, ptr.data(), pn.data(), order.data(), colour.data());
    if (ncol < 0)
        return set_error(FEA_ERANGE, "tile %lld needs more than %d colours", (long long)(-ncol - 1), host::kMaxColours);
    std::vector<int64_t> seg;
    std::vector<int32_t> ctile;
    host::buckets(nt, 4, fam.data(), colour.data(), (int)ncol, order.data(), g->tile_base, seg, ctile);
    dfree(g->ctile);
    g->ctile = nullptr;
    int rc;
    if ((rc = dalloc((void **)&g->ctile, sizeof(int32_t) * std::max<int64_t>(nt, 1)))) return rc;
    if (nt) FEA_HIP(hipMemcpyAsync(g->ctile, ctile.data(), sizeof(int32_t) * nt, hipMemcpyHostToDevice, s));
    FEA_HIP(hipStreamSynchronize(s));
    g->tc_colours = (int)ncol;
    g->tcseg = std::move(seg);
    g->tc_nneig = std::move(nneig);
    g->tcready = true;
    return FEA_OK;
}

// ------------------------------------------------------------- colouring
// Greedy first-fit in element order (the colouring of Algorithm 5; any
// valid colouring is correct, this one is deterministic). An element's colour
// needs those of its lower-numbered neighbours only, so some could be coloured
// side by side; this is the plain form, one element after the other on the host
// over per-node masks of used colours, on a thread of its own that starts once
// the mesh is validated and works while the device builds the pattern and the
// maps. The build waits for it: 1.5 ms of the 2.3 of a 48^3 hybrid mesh.
// It needs one element at a time, so a large mesh's connectivity comes in
// chunks through two small pinned buffers, the next one's copy beside this
// one's colouring: at 3.3 M elements 10 ms of colouring is then all there is,
// where copying everything first (pageable, and every page new) took 17 to 20 ms
// more before the device could go on.
struct HostColouring {
    static constexpr int64_t kChunk = 65536;  // elements
    int device = 0;
    int64_t N = 0, E = 0;
    const uint8_t *types_d = nullptr;
    const int32_t *conn_d = nullptr;
    std::unique_ptr<uint8_t[]> ty;
    std::unique_ptr<int32_t[]> cn;  // connectivity of a mesh of one chunk
    std::vector<int16_t> colour;
    std::vector<int64_t> cseg;
    std::vector<int32_t> cperm;
    int64_t ncol = 0;
    bool nomem = false;
    hipError_t err = hipSuccess;
    std::thread th;

    // Pinned buffers and a stream (open() on the colouring's thread)
    struct Feed {
        hipStream_t st = nullptr;
        int32_t *conn[2] = {nullptr, nullptr};
        uint8_t *types = nullptr;
        ~Feed()
        {
            if (st) {
                (void)hipStreamSynchronize(st);
                (void)hipStreamDestroy(st);
            }
            if (conn[0]) (void)hipHostFree(conn[0]);
        }
        hipError_t open()
        {
            const size_t cb = sizeof(int32_t) * 8 * kChunk;
            hipError_t e = hipHostMalloc((void **)&conn[0], 2 * cb + kChunk, hipHostMallocDefault);
            if (e != hipSuccess) return e;
            conn[1] = conn[0] + 8 * kChunk;
            types = (uint8_t *)(conn[0] + 2 * 8 * kChunk);
            return hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
        }
        // Device copy of pageable memory, through the two buffers.
        hipError_t put(void *dst, const void *src, size_t bytes)
        {
            const size_t cb = sizeof(int32_t) * 8 * kChunk;
            hipError_t e = hipSuccess;
            for (size_t off = 0, i = 0; off < bytes && e == hipSuccess; off += cb, ++i) {
                const size_t n = std::min(cb, bytes - off);
                if (i >= 2) e = hipStreamSynchronize(st);
                memcpy(conn[i & 1], (const char *)src + off, n);
                if (e == hipSuccess)
                    e = hipMemcpyAsync((char *)dst + off, conn[i & 1], n, hipMemcpyHostToDevice, st);
            }
            const hipError_t w = hipStreamSynchronize(st);
            return e == hipSuccess ? w : e;
        }
        hipError_t fetch(void *dst, const void *src, size_t bytes)
        {
            return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st);
        }
    };

    Feed f;

    ~HostColouring()
    {
        if (th.joinable()) th.join();
    }

    int64_t entries(int64_t e0, int64_t n) const
    {
        int64_t len = 0;
        for (int64_t e = e0; e < e0 + n; ++e) len += nodes_of(ty[e]);
        return len;
    }

    // Colours elements e0 .. e0 + n (their nodes at v): the first that finds
    // no colour, or -1.
    template <int W>
    int64_t place(host::FirstFit<W> &ff, int64_t e0, int64_t n, const int32_t *v)
    {
        for (int64_t e = e0; e < e0 + n; ++e) {
            const int nn = nodes_of(ty[e]);
            int c;
            switch (nn) {  // constant lengths
            case 4: c = ff.place(v, 4); break;
            case 5: c = ff.place(v, 5); break;
            case 6: c = ff.place(v, 6); break;
            default: c = ff.place(v, 8); break;
            }
            if (c < 0) return e;
            colour[(size_t)e] = (int16_t)c;
            v += nn;
        }
        return -1;
    }

    // Number of colours, or -(1 + e) when element e would need more than 64 W.
    template <int W>
    int64_t first_fit()
    {
        host::FirstFit<W> ff(N);
        int64_t bad = -1;
        if (cn) {
            bad = place(ff, 0, E, cn.get());
            return bad < 0 ? ff.colours() : -(1 + bad);
        }
        // chunk c's connectivity and chunk c + 1's types are on their way
        // while chunk c - 1 is coloured
        int64_t n = std::min(kChunk, E), pos = 0;
        if ((err = f.fetch(f.types, types_d, (size_t)n)) != hipSuccess) return 0;
        if ((err = hipStreamSynchronize(f.st)) != hipSuccess) return 0;
        memcpy(ty.get(), f.types, (size_t)n);
        int64_t len = entries(0, n);
        if ((err = f.fetch(f.conn[0], conn_d, sizeof(int32_t) * len)) != hipSuccess) return 0;
        int64_t n1 = std::min(kChunk, E - n);
        if (n1 && (err = f.fetch(f.types, types_d + n, (size_t)n1)) != hipSuccess) return 0;
        for (int64_t e0 = 0, c = 0; e0 < E; ++c) {
            if ((err = hipStreamSynchronize(f.st)) != hipSuccess) return 0;
            const int64_t e1 = e0 + n, next = n1;
            int64_t len1 = 0;
            if (next) {
                memcpy(ty.get() + e1, f.types, (size_t)next);
                len1 = entries(e1, next);
                if ((err = f.fetch(f.conn[(c + 1) & 1], conn_d + pos + len, sizeof(int32_t) * len1)) != hipSuccess)
                    return 0;
                n1 = std::min(kChunk, E - e1 - next);
                if (n1 && (err = f.fetch(f.types, types_d + e1 + next, (size_t)n1)) != hipSuccess) return 0;
            }
            if ((bad = place(ff, e0, n, f.conn[c & 1])) >= 0) return -(1 + bad);
            e0 = e1;
            n = next;
            pos += len;
            len = len1;
        }
        return ff.colours();
    }

    void run()
    {
        try {
            if (!cn && E) {
                if ((err = hipSetDevice(device)) != hipSuccess) return;
                if ((err = f.open()) != hipSuccess) return;
            }
            colour.assign((size_t)std::max<int64_t>(E, 1), 0);
            // one mask word per node first; with the full masks, in the same
            // order, only if an element needs a 65th colour
            if (E) ncol = first_fit<1>();
            if (ncol < 0) {
                if (f.st) (void)hipStreamSynchronize(f.st);
                ncol = first_fit<host::kMaxColours / 64>();
            }
            // stable buckets by (family, colour) of element ids
            if (err == hipSuccess && ncol >= 0)
                host::buckets(E, 4, ty.get(), colour.data(), (int)ncol, nullptr, nullptr, cseg, cperm);
        } catch (...) {
            nomem = true;
        }
    }
};

// Starts the colouring of the (validated) mesh.
static int colour_start(fea_graph *g, const int32_t *conn_d, const uint8_t *types_d, hipStream_t s, HostColouring &hc)
{
    const int64_t E = g->n_elems;
    hc.device = g->device;
    hc.N = g->n_nodes;
    hc.E = E;
    hc.types_d = types_d;
    hc.conn_d = conn_d;
    try {
        hc.ty.reset(new uint8_t[(size_t)std::max<int64_t>(E, 1)]);
        if (E <= HostColouring::kChunk) hc.cn.reset(new int32_t[(size_t)std::max<int64_t>(g->conn_len, 1)]);
    } catch (...) {
        return set_error(FEA_ENOMEM, "host allocation failed (colouring)");
    }
    if (hc.cn && E) {  // one chunk: without buffers and a stream for it
        FEA_HIP(hipMemcpyAsync(hc.ty.get(), types_d, (size_t)E, hipMemcpyDeviceToHost, s));
        FEA_HIP(hipMemcpyAsync(hc.cn.get(), conn_d, sizeof(int32_t) * g->conn_len, hipMemcpyDeviceToHost, s));
        FEA_HIP(hipStreamSynchronize(s));
    }
    try {
        hc.th = std::thread([&hc] { hc.run(); });
    } catch (...) {
        hc.run();  // no thread to be had: colour here
    }
    return FEA_OK;
}

// Waits for the colouring and uploads it.
static int colour_finish(fea_graph *g, HostColouring &hc, hipStream_t s)
{
    const int64_t E = g->n_elems;
    if (hc.th.joinable()) hc.th.join();
    if (hc.nomem) return set_error(FEA_ENOMEM, "host allocation failed (colouring)");
    if (hc.err != hipSuccess)
        return set_error(FEA_EHIP, "copy of the connectivity to the host failed: %s", hipGetErrorString(hc.err));
    if (hc.ncol < 0)
        return set_error(FEA_ERANGE, "element %lld needs more than %d colours", (long long)(-hc.ncol - 1),
                         host::kMaxColours);
    if (E && hc.cn) {
        FEA_HIP(hipMemcpyAsync(g->colour, hc.colour.data(), sizeof(int16_t) * E, hipMemcpyHostToDevice, s));
        FEA_HIP(hipMemcpyAsync(g->cperm, hc.cperm.data(), sizeof(int32_t) * E, hipMemcpyHostToDevice, s));
        FEA_HIP(hipStreamSynchronize(s));
    } else if (E) {
        FEA_HIP(hc.f.put(g->colour, hc.colour.data(), sizeof(int16_t) * E));
        FEA_HIP(hc.f.put(g->cperm, hc.cperm.data(), sizeof(int32_t) * E));
    }
    g->n_colours = (int)hc.ncol;
    g->cseg = std::move(hc.cseg);
    return FEA_OK;
}

// waited: result of the wait for all work on the graph's arrays.
static void destroy(fea_graph *g, hipError_t waited)
{
    if (!g) return;
    void *bufs[] = {g->mem[0], g->mem[1], g->mem[2], g->contrib, g->rcontrib, g->acc64,
                    g->gtile, g->gnodes, g->gdesc, g->ctile, g->gp_ptr};
    for (void *b : bufs) pool_free(b, waited);
    for (hipEvent_t e : g->ev)
        if (e) (void)hipEventDestroy(e);
    for (hipEvent_t e : g->gev)
        if (e) (void)hipEventDestroy(e);
    delete g;
}


// Checks a mesh (FEA_EMESH names the first bad element): its fingerprint,
// the elements of every family and, if fam_cnt is given (4 per workgroup of
// 256 elements), the workgroups' counts. out: device memory. Blocks on the
// stream.
static int mesh_check(int64_t N, int64_t E, const uint8_t *types, const int64_t *conn_ptr, const int32_t *conn,
                      MeshCheck *out, int32_t *fam_cnt, hipStream_t s, MeshCheck *mc)
{
    *mc = MeshCheck{~0ull, 0, {0, 0, 0, 0}};
    if (!E) return FEA_OK;
    FEA_HIP(hipMemcpyAsync(out, mc, sizeof(MeshCheck), hipMemcpyHostToDevice, s));
    k_mesh_check<<<grid_for(E, 256), 256, 0, s>>>(N, E, types, conn_ptr, conn, out, fam_cnt);
    FEA_HIP(hipGetLastError());
    FEA_HIP(hipMemcpyAsync(mc, out, sizeof(MeshCheck), hipMemcpyDeviceToHost, s));
    FEA_HIP(hipStreamSynchronize(s));
    if (mc->bad != ~0ull)
        return set_error(FEA_EMESH, "invalid element %lld (unknown type, wrong node count, node id out "
                         "of range or repeated node)", (long long)mc->bad);
    return FEA_OK;
}

// Where the families' elements, node entries and element-matrix slots start in
// the type-sorted order, from the elements of every family.
struct FamilyBases {
    int64_t seg[5] = {0}, node[5] = {0}, slot[5] = {0};
    explicit FamilyBases(const MeshCheck &mc)
    {
        for (int t = 0; t < 4; ++t) {
            const int64_t n = nodes_of(t), c = (int64_t)mc.fam[t];
            seg[t + 1] = seg[t] + c;
            node[t + 1] = node[t] + c * n;
            slot[t + 1] = slot[t] + c * n * n;
        }
    }
};

static int build(int64_t N, int64_t E, const uint8_t *types, const int64_t *conn_ptr,
                 const int32_t *conn, hipStream_t s, fea_graph *g)
{
    const int BS = 256;
    int rc;
    FEA_HIP(hipGetDevice(&g->device));
    g->n_nodes = N;
    g->n_elems = E;

    // validation, fingerprint, family counts: every size but the pattern's
    const int64_t nb = (E + 255) / 256;
    TmpBuf chk(s), tmp(s);
    MeshCheck *out, mc;
    int32_t *famc;
    if ((rc = dalloc_arrays(&chk.p, {{(void **)&out, sizeof(MeshCheck)}, {(void **)&famc, sizeof(int32_t) * 4 * nb}})))
        return rc;
    if ((rc = mesh_check(N, E, types, conn_ptr, conn, out, famc, s, &mc))) return rc;
    g->mesh_fp = mc.fp;
    const FamilyBases fb(mc);
    std::copy(fb.seg, fb.seg + 5, g->seg);
    std::copy(fb.node, fb.node + 5, g->node_base);
    std::copy(fb.slot, fb.slot + 5, g->slot_base);
    RowBases bs;
    for (int t = 0; t < 4; ++t) {
        const int64_t n = nodes_of(t);
        bs.node[t] = (uint32_t)(g->node_base[t] - g->seg[t] * n);
        bs.slot[t] = (uint32_t)(g->slot_base[t] - g->seg[t] * n * n);
    }
    g->conn_len = g->node_base[4];
    g->map_len = g->slot_base[4];
    HostColouring hc;  // joined on every return
    if ((rc = colour_start(g, conn, types, s, hc))) return rc;
    const int64_t C = g->conn_len, M = g->map_len;
    if (M > INT32_MAX || C > INT32_MAX)
        return set_error(FEA_ERANGE, "%lld element-matrix slots / %lld incidences exceed int32 maps", (long long)M,
                         (long long)C);
    int64_t *scan, *famp, *cnt, *ptr2;
    int32_t *epos, *deg, *vs;
    if ((rc = dalloc_arrays(&g->mem[0], {{(void **)&g->map_ptr, sizeof(int64_t) * (E + 1)},
                                         {(void **)&g->perm, sizeof(int32_t) * E},
                                         {(void **)&g->n2e_ptr, sizeof(int64_t) * (N + 1)},
                                         {(void **)&g->n2e, sizeof(int32_t) * C},
                                         {(void **)&g->n2a, sizeof(uint8_t) * C},
                                         {(void **)&g->pnodes, sizeof(int32_t) * C},
                                         {(void **)&g->prdest, sizeof(int32_t) * C},
                                         {(void **)&g->pdest, sizeof(int32_t) * M},
                                         {(void **)&g->inv, sizeof(int32_t) * M},
                                         {(void **)&g->e2nnz, sizeof(int32_t) * M},
                                         {(void **)&g->row_ptr, sizeof(int64_t) * (N + 1)},
                                         {(void **)&g->colour, sizeof(int16_t) * E},
                                         {(void **)&g->cperm, sizeof(int32_t) * E}})))
        return rc;
    if ((rc = dalloc_arrays(&tmp.p, {{(void **)&scan, sizeof(int64_t) * (scan_tmp_elems(std::max(4 * nb, N)) + 64)},
                                     {(void **)&famp, sizeof(int64_t) * (4 * nb + 1)},
                                     {(void **)&epos, sizeof(int32_t) * E},
                                     {(void **)&cnt, sizeof(int64_t) * N},
                                     {(void **)&ptr2, sizeof(int64_t) * (N + 1)},
                                     {(void **)&deg, sizeof(int32_t) * N},
                                     {(void **)&vs, sizeof(int32_t) * M}})))
        return rc;

    // type segmentation, first slots
    if (E) {
        if ((rc = scan_to_ptr_i32(famc, 4 * nb, famp, scan, s))) return rc;
        k_type_place<<<(unsigned)nb, 256, 0, s>>>(E, types, famp, g->perm, epos, g->map_ptr);
    } else {
        FEA_HIP(hipMemsetAsync(g->map_ptr, 0, sizeof(int64_t), s));
    }

    // node incidence (prdest holds the places in the unsorted lists meanwhile)
    if (N) FEA_HIP(hipMemsetAsync(cnt, 0, sizeof(int64_t) * N, s));
    if (E) k_node_count<<<grid_for(E, BS), BS, 0, s>>>(E, conn_ptr, conn, (unsigned long long *)cnt, g->prdest);
    if ((rc = scan_to_ptr_i64(cnt, N, ptr2, scan, s))) return rc;
    if (E) k_node_fill<<<grid_for(E, BS), BS, 0, s>>>(E, conn_ptr, conn, ptr2, g->prdest, g->n2e, g->n2a);

    // rows: sorted slots, degrees, prefix sum, then blocks
    const RowOut ro = {conn_ptr, conn, g->map_ptr, epos, vs, g->inv, g->pdest, g->pnodes, g->prdest};
    if (N)
        k_rows<<<grid_for(N, 4), 256, 0, s>>>(N, ptr2, ro, bs, g->n2e_ptr, g->n2e, g->n2a, deg);
    else
        FEA_HIP(hipMemsetAsync(g->n2e_ptr, 0, sizeof(int64_t), s));
    if ((rc = scan_to_ptr_i32(deg, N, g->row_ptr, scan, s))) return rc;
    FEA_HIP(hipMemcpyAsync(&g->nnz, g->row_ptr + N, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    // cnt is free again: its first two words take the counts (an array has at
    // least 256 bytes)
    unsigned long long mixed = 0;
    const int64_t sampled = mixed_groups(N);
    if (N) {
        FEA_HIP(hipMemsetAsync(cnt, 0, 2 * sizeof(int64_t), s));
        k_mixed_nodes<<<grid_for(sampled, 256), 256, 0, s>>>(N, sampled, E, C, g->n2e_ptr, g->n2e, conn_ptr,
                                                             (unsigned long long *)cnt);
        FEA_HIP(hipMemcpyAsync(&mixed, cnt, sizeof(mixed), hipMemcpyDeviceToHost, s));
    }
    FEA_HIP(hipStreamSynchronize(s));
    g->mixed = N > 0 && 2 * (int64_t)mixed >= sampled;
    if (g->nnz > INT32_MAX)
        return set_error(FEA_ERANGE, "%lld nonzero blocks exceed int32 block indices", (long long)g->nnz);
    if ((rc = dalloc_arrays(&g->mem[1], {{(void **)&g->col, sizeof(int32_t) * g->nnz},
                                         {(void **)&g->inv_ptr, sizeof(int64_t) * (g->nnz + 1)}})))
        return rc;
    if (N)
        k_row_blocks<<<grid_for(N, 4), 256, 0, s>>>(N, ptr2, g->row_ptr, vs, g->inv, g->col, g->inv_ptr, g->e2nnz);
    else
        FEA_HIP(hipMemsetAsync(g->inv_ptr, 0, sizeof(int64_t), s));
    FEA_HIP(hipGetLastError());
    FEA_HIP(hipStreamSynchronize(s));

    return colour_finish(g, hc, s);
}

}  // namespace fea

using namespace fea;

extern "C" int fea_graph_build(int64_t n_nodes, int64_t n_elems, const uint8_t *types,
                               const int64_t *conn_ptr, const int32_t *conn, hipStream_t stream,
                               fea_graph **out)
{
    clear_error();
    if (!out) return set_error(FEA_EINVAL, "out is NULL");
    *out = nullptr;
    if (n_nodes < 0 || n_elems < 0) return set_error(FEA_EINVAL, "negative size");
    if (n_elems > 0 && (!types || !conn_ptr || !conn))
        return set_error(FEA_EINVAL, "types, conn_ptr and conn are required");
    if (n_nodes > INT32_MAX || n_elems > INT32_MAX)
        return set_error(FEA_ERANGE, "more than 2^31-1 nodes or elements");
    fea_graph *g = new (std::nothrow) fea_graph();
    if (!g) return set_error(FEA_ENOMEM, "host allocation failed");
    int rc = build(n_nodes, n_elems, types, conn_ptr, conn, stream, g);
    if (rc == FEA_OK) rc = noalloc_setup();
    if (rc != FEA_OK) {
        // an error of the runtime may have left work on the colouring's stream too
        const hipError_t w = hipStreamSynchronize(stream);
        destroy(g, w == hipSuccess && rc == FEA_EHIP ? hipDeviceSynchronize() : w);
        return rc;
    }
    *out = g;
    return FEA_OK;
}

namespace {

// Graph cache file: header (magic, version, GPU architecture name, sizes,
// mesh fingerprint, family and colour offsets), then the graph's device
// arrays in a fixed order, each preceded by its byte count.
constexpr char kGraphMagic[8] = {'F', 'E', 'A', 'G', 'R', 'A', 'P', 'H'};
constexpr uint32_t kGraphVersion = 1;
constexpr size_t kStage = size_t(64) << 20;  // host staging buffer (bytes)

struct GraphHeader {
    char magic[8];
    uint32_t version;
    int32_t n_colours;
    char arch[64];
    int64_t n_nodes, n_elems, nnz, map_len, conn_len;
    uint64_t mesh_fp;
    int64_t seg[5], node_base[5], slot_base[5];
    int64_t cseg_len;
};

struct HostFile {
    FILE *f = nullptr;
    ~HostFile()
    {
        if (f) fclose(f);
    }
};

struct PinnedBuf {
    void *p = nullptr;
    ~PinnedBuf()
    {
        if (p) (void)hipHostFree(p);
    }
};

int device_arch(int dev, char *arch)
{
    hipDeviceProp_t prop;
    FEA_HIP(hipGetDeviceProperties(&prop, dev));
    memset(arch, 0, 64);
    strncpy(arch, prop.gcnArchName, 63);
    return FEA_OK;
}

// The graph's arrays that the cache holds, with their lengths in bytes.
std::vector<DevArray> graph_arrays(fea_graph *g)
{
    const size_t N = (size_t)g->n_nodes, E = (size_t)g->n_elems, nnz = (size_t)g->nnz,
                 ml = (size_t)g->map_len, cl = (size_t)g->conn_len;
    auto one = [](size_t n) { return n ? n : 1; };
    return {{(void **)&g->row_ptr, 8 * (N + 1)},   {(void **)&g->col, 4 * one(nnz)},
            {(void **)&g->map_ptr, 8 * (E + 1)},   {(void **)&g->e2nnz, 4 * one(ml)},
            {(void **)&g->inv_ptr, 8 * (nnz + 1)}, {(void **)&g->inv, 4 * one(ml)},
            {(void **)&g->pnodes, 4 * one(cl)},    {(void **)&g->pdest, 4 * one(ml)},
            {(void **)&g->prdest, 4 * one(cl)},    {(void **)&g->n2e_ptr, 8 * (N + 1)},
            {(void **)&g->n2e, 4 * one(cl)},       {(void **)&g->n2a, one(cl)},
            {(void **)&g->perm, 4 * one(E)},       {(void **)&g->colour, 2 * one(E)},
            {(void **)&g->cperm, 4 * one(E)}};
}

}  // namespace

extern "C" int fea_graph_save(const fea_graph *gc, const char *path)
{
    clear_error();
    if (!gc || !path) return set_error(FEA_EINVAL, "graph and path are required");
    fea_graph *g = const_cast<fea_graph *>(gc);
    GraphHeader h;
    memset(&h, 0, sizeof(h));
    memcpy(h.magic, kGraphMagic, 8);
    h.version = kGraphVersion;
    h.n_colours = g->n_colours;
    int rc = device_arch(g->device, h.arch);
    if (rc) return rc;
    h.n_nodes = g->n_nodes;
    h.n_elems = g->n_elems;
    h.nnz = g->nnz;
    h.map_len = g->map_len;
    h.conn_len = g->conn_len;
    h.mesh_fp = g->mesh_fp;
    memcpy(h.seg, g->seg, sizeof(h.seg));
    memcpy(h.node_base, g->node_base, sizeof(h.node_base));
    memcpy(h.slot_base, g->slot_base, sizeof(h.slot_base));
    h.cseg_len = (int64_t)g->cseg.size();
    HostFile f;
    f.f = fopen(path, "wb");
    if (!f.f) return set_error(FEA_EINVAL, "cannot write %s", path);
    bool ok = fwrite(&h, sizeof(h), 1, f.f) == 1 &&
              (h.cseg_len == 0 || fwrite(g->cseg.data(), 8, (size_t)h.cseg_len, f.f) == (size_t)h.cseg_len);
    PinnedBuf stage;
    FEA_HIP(hipHostMalloc(&stage.p, kStage, hipHostMallocDefault));
    FEA_HIP(hipDeviceSynchronize());
    for (const DevArray &a : graph_arrays(g)) {
        const uint64_t nb = a.bytes;
        ok = ok && fwrite(&nb, 8, 1, f.f) == 1;
        for (size_t off = 0; ok && off < a.bytes; off += kStage) {
            const size_t n = std::min(kStage, a.bytes - off);
            FEA_HIP(hipMemcpy(stage.p, (char *)*a.p + off, n, hipMemcpyDeviceToHost));
            ok = fwrite(stage.p, 1, n, f.f) == n;
        }
    }
    if (!ok) return set_error(FEA_EINVAL, "short write to %s", path);
    return FEA_OK;
}

extern "C" int fea_graph_load(const char *path, int64_t n_nodes, int64_t n_elems, const uint8_t *types,
                              const int64_t *conn_ptr, const int32_t *conn, hipStream_t stream, fea_graph **out)
{
    clear_error();
    if (!out || !path) return set_error(FEA_EINVAL, "path and out are required");
    *out = nullptr;
    if (n_nodes < 0 || n_elems < 0) return set_error(FEA_EINVAL, "negative size");
    if (n_elems > 0 && (!types || !conn_ptr || !conn))
        return set_error(FEA_EINVAL, "types, conn_ptr and conn are required");
    HostFile f;
    f.f = fopen(path, "rb");
    if (!f.f) return set_error(FEA_EINVAL, "cannot read %s", path);
    GraphHeader h;
    if (fread(&h, sizeof(h), 1, f.f) != 1 || memcmp(h.magic, kGraphMagic, 8) != 0)
        return set_error(FEA_EINVAL, "%s is not a graph cache", path);
    if (h.version != kGraphVersion)
        return set_error(FEA_EINVAL, "%s: graph cache version %u, this library reads %u", path, h.version,
                         kGraphVersion);
    int dev = 0;
    FEA_HIP(hipGetDevice(&dev));
    char arch[64];
    int rc = device_arch(dev, arch);
    if (rc) return rc;
    h.arch[63] = 0;
    if (strcmp(arch, h.arch) != 0)
        return set_error(FEA_EINVAL, "%s was written on %s, this device is %s", path, h.arch, arch);
    if (h.n_nodes != n_nodes || h.n_elems != n_elems)
        return set_error(FEA_EINVAL, "%s holds the graph of a mesh of %lld nodes and %lld elements, not %lld and %lld",
                         path, (long long)h.n_nodes, (long long)h.n_elems, (long long)n_nodes, (long long)n_elems);
    if (h.cseg_len < 0 || h.n_colours < 0 || h.nnz < 0 || h.map_len < 0 || h.conn_len < 0 ||
        h.cseg_len != 4 * ((int64_t)h.n_colours + 1))
        return set_error(FEA_EINVAL, "%s: inconsistent header", path);
    // the mesh must be the one the graph was built for
    MeshCheck mc;
    TmpBuf chk(stream);
    if ((rc = dalloc_pool(&chk.p, sizeof(MeshCheck)))) return rc;
    if ((rc = mesh_check(n_nodes, n_elems, types, conn_ptr, conn, (MeshCheck *)chk.p, nullptr, stream, &mc)))
        return rc;
    if (mc.fp != h.mesh_fp) return set_error(FEA_EINVAL, "%s was built for another mesh (connectivity differs)", path);
    const FamilyBases fb(mc);
    if (h.n_colours > host::kMaxColours || h.conn_len != fb.node[4] || h.map_len != fb.slot[4] || h.nnz > h.map_len ||
        memcmp(h.seg, fb.seg, sizeof(h.seg)) != 0 || memcmp(h.node_base, fb.node, sizeof(h.node_base)) != 0 ||
        memcmp(h.slot_base, fb.slot, sizeof(h.slot_base)) != 0)
        return set_error(FEA_EINVAL, "%s: inconsistent header", path);
    fea_graph *g = new (std::nothrow) fea_graph();
    if (!g) return set_error(FEA_ENOMEM, "host allocation failed");
    FEA_HIP(hipGetDevice(&g->device));
    g->n_nodes = h.n_nodes;
    g->n_elems = h.n_elems;
    g->nnz = h.nnz;
    g->map_len = h.map_len;
    g->conn_len = h.conn_len;
    g->n_colours = h.n_colours;
    g->mesh_fp = h.mesh_fp;
    memcpy(g->seg, h.seg, sizeof(h.seg));
    memcpy(g->node_base, h.node_base, sizeof(h.node_base));
    memcpy(g->slot_base, h.slot_base, sizeof(h.slot_base));
    g->cseg.resize((size_t)h.cseg_len);
    bool ok = h.cseg_len == 0 || fread(g->cseg.data(), 8, (size_t)h.cseg_len, f.f) == (size_t)h.cseg_len;
    PinnedBuf stage;
    if (ok) {
        hipError_t e = hipHostMalloc(&stage.p, kStage, hipHostMallocDefault);
        if (e != hipSuccess) {
            destroy(g, hipSuccess);
            return set_error(FEA_ENOMEM, "pinned staging buffer: %s", hipGetErrorString(e));
        }
    }
    const std::vector<DevArray> arrays = graph_arrays(g);
    // every array's byte count first: a file that does not match allocates
    // nothing (a pipe cannot seek: its counts are checked as they come)
    const long data = ftell(f.f);
    if (ok && data >= 0) {
        for (const DevArray &a : arrays) {
            uint64_t nb = 0;
            ok = ok && fread(&nb, 8, 1, f.f) == 1 && nb == a.bytes && fseek(f.f, (long)a.bytes, SEEK_CUR) == 0;
        }
        ok = ok && fseek(f.f, data, SEEK_SET) == 0;
    }
    if (ok && (rc = dalloc_arrays(&g->mem[0], arrays.data(), arrays.size()))) {
        destroy(g, hipSuccess);
        return rc;
    }
    for (const DevArray &a : arrays) {
        if (!ok) break;
        uint64_t nb = 0;
        ok = fread(&nb, 8, 1, f.f) == 1 && nb == a.bytes;
        if (!ok) break;
        for (size_t off = 0; ok && off < a.bytes; off += kStage) {
            const size_t n = std::min(kStage, a.bytes - off);
            ok = fread(stage.p, 1, n, f.f) == n;
            if (ok && hipMemcpy((char *)*a.p + off, stage.p, n, hipMemcpyHostToDevice) != hipSuccess) {
                destroy(g, hipDeviceSynchronize());
                return set_error(FEA_EHIP, "copy of %s to the device failed", path);
            }
        }
    }
    if (!ok) {
        destroy(g, hipSuccess);  // every copy was waited for
        return set_error(FEA_EINVAL, "%s is truncated or does not match its header", path);
    }
    if (n_nodes) {
        unsigned long long count[2] = {0, 0}, *cnt = (unsigned long long *)chk.p;
        const int64_t sampled = mixed_groups(n_nodes);
        hipError_t e = hipMemsetAsync(cnt, 0, sizeof(count), stream);
        if (e == hipSuccess) {
            k_mixed_nodes<<<grid_for(sampled, 256), 256, 0, stream>>>(n_nodes, sampled, n_elems, g->conn_len, g->n2e_ptr,
                                                                      g->n2e, conn_ptr, cnt);
            e = hipMemcpyAsync(count, cnt, sizeof(count), hipMemcpyDeviceToHost, stream);
        }
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) {
            destroy(g, hipDeviceSynchronize());
            return set_error(FEA_EHIP, "graph load: %s", hipGetErrorString(e));
        }
        if (count[1]) {
            destroy(g, hipSuccess);
            return set_error(FEA_EINVAL, "%s does not match its header (incidence lists out of range)", path);
        }
        g->mixed = 2 * (int64_t)count[0] >= sampled;
    }
    if ((rc = noalloc_setup())) {
        destroy(g, hipSuccess);  // every copy and kernel was waited for
        return rc;
    }
    *out = g;
    return FEA_OK;
}

extern "C" int fea_graph_tile_colouring(const fea_graph *g, int *n_colours, int64_t *bucket_ptr, int32_t *tiles,
                                        int32_t *nneig, hipStream_t stream)
{
    clear_error();
    if (!g) return set_error(FEA_EINVAL, "graph is NULL");
    if (!g->tcready) return set_error(FEA_EINVAL, "the tile colouring has not been built (no FEA_TILECOLOUR call yet)");
    if (n_colours) *n_colours = g->tc_colours;
    if (bucket_ptr) std::copy(g->tcseg.begin(), g->tcseg.end(), bucket_ptr);
    const int64_t nt = g->tile_base[4];
    if (nneig && nt) std::copy(g->tc_nneig.begin(), g->tc_nneig.begin() + nt, nneig);
    if (tiles && nt)
        FEA_HIP(hipMemcpyAsync(tiles, g->ctile, sizeof(int32_t) * nt, hipMemcpyDeviceToDevice, stream));
    return FEA_OK;
}

extern "C" int fea_graph_sizes(const fea_graph *g, int64_t *n_nodes, int64_t *n_elems,
                               int64_t *nnz_blocks, int64_t *map_len, int *n_colours)
{
    clear_error();
    if (!g) return set_error(FEA_EINVAL, "graph is NULL");
    if (n_nodes) *n_nodes = g->n_nodes;
    if (n_elems) *n_elems = g->n_elems;
    if (nnz_blocks) *nnz_blocks = g->nnz;
    if (map_len) *map_len = g->map_len;
    if (n_colours) *n_colours = g->n_colours;
    return FEA_OK;
}

extern "C" int fea_graph_sym_sizes(const fea_graph *g, int64_t *tiles, int64_t *entries, int64_t *tile_blocks,
                                   int64_t *upper_blocks)
{
    clear_error();
    if (!g) return set_error(FEA_EINVAL, "graph is NULL");
    if (!g->sready)
        return set_error(FEA_EINVAL, "the upper-triangle layout is built by the first FEA_ROWSYM assembly");
    if (tiles) *tiles = g->tile_base[4];
    if (entries) *entries = g->nent;
    if (tile_blocks) *tile_blocks = g->ulen;
    if (upper_blocks) *upper_blocks = g->nup;
    return FEA_OK;
}

extern "C" int fea_graph_export(const fea_graph *g, int64_t *row_ptr, int32_t *col,
                                int64_t *map_ptr, int32_t *e2nnz, int64_t *inv_ptr, int32_t *inv,
                                int16_t *colour, int32_t *type_perm, int64_t *type_seg,
                                hipStream_t s)
{
    clear_error();
    if (!g) return set_error(FEA_EINVAL, "graph is NULL");
    const hipMemcpyKind D2D = hipMemcpyDeviceToDevice;
    if (row_ptr) FEA_HIP(hipMemcpyAsync(row_ptr, g->row_ptr, sizeof(int64_t) * (g->n_nodes + 1), D2D, s));
    if (col && g->nnz) FEA_HIP(hipMemcpyAsync(col, g->col, sizeof(int32_t) * g->nnz, D2D, s));
    if (map_ptr) FEA_HIP(hipMemcpyAsync(map_ptr, g->map_ptr, sizeof(int64_t) * (g->n_elems + 1), D2D, s));
    if (e2nnz && g->map_len) FEA_HIP(hipMemcpyAsync(e2nnz, g->e2nnz, sizeof(int32_t) * g->map_len, D2D, s));
    if (inv_ptr) FEA_HIP(hipMemcpyAsync(inv_ptr, g->inv_ptr, sizeof(int64_t) * (g->nnz + 1), D2D, s));
    if (inv && g->map_len) FEA_HIP(hipMemcpyAsync(inv, g->inv, sizeof(int32_t) * g->map_len, D2D, s));
    if (colour && g->n_elems) FEA_HIP(hipMemcpyAsync(colour, g->colour, sizeof(int16_t) * g->n_elems, D2D, s));
    if (type_perm && g->n_elems) FEA_HIP(hipMemcpyAsync(type_perm, g->perm, sizeof(int32_t) * g->n_elems, D2D, s));
    if (type_seg) memcpy(type_seg, g->seg, sizeof(g->seg));
    return FEA_OK;
}

extern "C" void fea_graph_destroy(fea_graph *g)
{
    if (g) {
        int cur = 0;
        (void)hipGetDevice(&cur);
        (void)hipSetDevice(g->device);
        destroy(g, hipDeviceSynchronize());
        (void)hipSetDevice(cur);
    }
}
