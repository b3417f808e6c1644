// disco_stencil.hip -- the DISCO convolution with W folded into psi per call:
// every call of the axisymmetric and separable bases (Sec. 3.4), and depthwise
// channels (Sec. 4.2) with any basis.
//
// The paper writes the op as one sparse-dense product with
// Psi_ji = psi(R_j^{-1} w_i) (Sec. 4.1 eq. 7), psi the interpolated filter
// itself; with learnable node values p_k, psi = sum_k p_k psi_k, so for each
// (output channel, input channel) pair the stored per-entry basis values fold
// into one weight, c = sum_k W[co, ci, k] psi_k q.  With few channels (App. B
// times one channel; depthwise layers filter each channel alone) that costs
// one FMA per stored entry and output channel instead of a gather per basis
// function and a contraction.
//
// An entry stores the (at most four) basis values of its hat cell; the op's
// cell map names the basis function of each.  Per input channel the kernels
// stage a table T[j][cell][m] = W[co0 + j, ci, map[cell][m]] (0 where the map
// has no function) in LDS, and fold c = sum_m T[j][cell][m] v[m] while an
// entry is staged.
//
// Three kernels.  k_stencil_walk takes the one-channel items of stride-1 ops
// on every ring with narrow windows: it keeps input rings in LDS while it
// walks output rings.  k_stencil_blocked takes the wide rings beside it (the
// spectral path does in larger calls) and ops with several input channels
// and one output channel; k_stencil the rest.  Alone on one box, 2048 x
// 4096, eight separable channels, wide rings from 128 entries on: the blocked
// kernel over every ring 640 us, over the narrow rings 500 us, the walk over
// the narrow rings 183 us (512 MB at 2.8 TB/s; 107 us without its products,
// which occupy the fp32 matrix cores for about 70 us).
//
// k_stencil's layout and walk are the packed one of the fused kernel (disco_fused.hip):
// one workgroup = 256 consecutive output longitudes of one pattern (output
// ring, phase) of a work item, for one batch element and a tile of COT output
// channels.  For each input channel and each chunk of the pattern:
//   1. the chunk's spans of input-ring longitudes are copied into LDS
//      (coalesced along longitude, wrapping at the 0 / 2 pi seam, bf16 widened
//      to fp32), and each entry's offset and its COT folded weights;
//   2. lane q reads its input at (stride * q + offset) for every entry and
//      accumulates weight * x into its COT outputs.
// The accumulation order of a lane depends only on the pattern, never on q,
// so whole-pixel longitude shifts commute with the op bitwise.  Patterns cut
// into several segments write partial outputs that k_reduce_partials sums in
// a fixed order.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "disco_internal.h"

namespace disco {

namespace {

DISCO_BOUNDS_FLAG

constexpr int kBlock = kTileQ;

__device__ __forceinline__ float load_val(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float load_val(const uint16_t* p, int64_t i) {
    return __uint_as_float((uint32_t)p[i] << 16);
}
__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ void store_val(float* p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_val(uint16_t* p, int64_t i, float v) { p[i] = to_bf16(v); }

// Consecutive blocks go to the 8 XCDs in turn; remap so that each XCD walks a
// contiguous range of work items (neighbouring rings share input rings).
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    const int xcd = bid & 7, local = bid >> 3;
    const int per = nb >> 3, rem = nb & 7;
    return xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

// Fills T[j][cell][m] (64 floats per output channel j of the tile) for input
// channel ci.  dw_c > 0: depthwise, item b takes row b mod dw_c of a [C][K]
// W (Ci = Co = 1).
template <typename T, int COT, int NT>
__device__ __forceinline__ void fill_fold_table(float* wt, const int8_t* __restrict__ cmap,
                                                const T* __restrict__ w, int K, int b, int ci, int co0,
                                                int Ci, int Co, bool w_trans, int dw_c) {
    for (int idx = threadIdx.x; idx < COT * kCells * 4; idx += NT) {
        const int j = idx / (kCells * 4), cm = idx - j * (kCells * 4);
        const int k = cmap[cm];
        const int co = co0 + j;
        float v = 0.0f;
        if (k >= 0 && co < Co) {
            const int64_t base = dw_c > 0 ? (int64_t)(b % dw_c) * K
                                 : w_trans ? ((int64_t)ci * Co + co) * K
                                           : ((int64_t)co * Ci + ci) * K;
            v = load_val(w, base + k);
        }
        wt[idx] = v;
    }
}

// TQ: output longitudes (lanes) per workgroup, the width the op's spans were
// packed for (PackedDev::tile).
template <typename T, int COT, int TQ>
__global__ __launch_bounds__(TQ) void k_stencil(const PItem* __restrict__ items,
                                                    const PSeg* __restrict__ segs,
                                                    const PChunk* __restrict__ chunks,
                                                    const PSpan* __restrict__ spans,
                                                    const int32_t* __restrict__ offs,
                                                    const PVal* __restrict__ vals,
                                                    const int8_t* __restrict__ cmap, OpGeom g,
                                                    const T* __restrict__ x, const T* __restrict__ w,
                                                    T* __restrict__ y, float* __restrict__ partial,
                                                    int Ci, int Co, int K, int n_qtiles, int n_cotiles,
                                                    bool w_trans, int dw_c) {
    __shared__ float xs[kLdsCols];
    __shared__ __align__(16) int eoffs[kChunkEntries];
    __shared__ __align__(16) float ew[kChunkEntries * COT];  // [entry][j]
    __shared__ __align__(16) float wt[COT * kCells * 4];     // [j][cell][m]

    const int tid = threadIdx.x;
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int item = bid / n_qtiles;
    const int qt = bid - item * n_qtiles;
    const int b = blockIdx.y / n_cotiles;
    const int co0 = (blockIdx.y - b * n_cotiles) * COT;
    const int q0 = qt * TQ;
    const int q = q0 + tid;
    const int lane_col = g.stride * tid;
    const int64_t n_in = (int64_t)g.nlat_i * g.nlon_i;
    const int64_t n_out = (int64_t)g.nlat_o * g.nlon_o;
    const PItem it = items[item];

    for (int si = it.seg_begin; si < it.seg_end; ++si) {
        const PSeg sg = segs[si];
        float acc[COT];
#pragma unroll
        for (int j = 0; j < COT; ++j) acc[j] = 0.0f;
        for (int ci = 0; ci < Ci; ++ci) {
            // W[co0 + j][ci][.] (forward) or W[ci][co0 + j][.] (transposed op)
            // through the cell map.  The previous readers of the table (the
            // last chunk's staging) are behind that chunk's second barrier;
            // the next chunk's first barrier orders these writes before use.
            fill_fold_table<T, COT, TQ>(wt, cmap, w, K, b, ci, co0, Ci, Co, w_trans, dw_c);
            const T* xc = x + ((int64_t)b * Ci + ci) * n_in;
            for (int ch = sg.chunk_begin; ch < sg.chunk_end; ++ch) {
                const PChunk C = chunks[ch];
                __syncthreads();  // readers of the previous chunk (or channel) are done
                for (int sp = C.span_begin; sp < C.span_end; ++sp) {
                    const PSpan S = spans[sp];
                    int start = (g.stride * q0 + S.dstart) % g.nlon_i;
                    if (start < 0) start += g.nlon_i;
                    for (int j = tid; j < S.len; j += TQ) {
                        int idx = start + j;
                        if (idx >= g.nlon_i) idx = idx % g.nlon_i;
                        DISCO_CHECK(S.lds_base + j >= 0 && S.lds_base + j < kLdsCols);
                        xs[S.lds_base + j] = load_val(xc, (int64_t)S.row + idx);
                    }
                }
                const int ebase = C.cls[0], ne = C.cls[kCells] - C.cls[0];
                for (int i = tid; i < ne; i += TQ) {
                    eoffs[i] = offs[ebase + i];
                    const PVal pv = vals[ebase + i];
                    // Entries are sorted by cell: cls[c] is the first of cell c.
                    int cell = 0;
#pragma unroll
                    for (int c = 1; c < kCells; ++c) cell += ebase + i >= C.cls[c] ? 1 : 0;
#pragma unroll
                    for (int j = 0; j < COT; ++j) {
                        const float4 t = *(const float4*)(wt + (j * kCells + cell) * 4);
                        ew[i * COT + j] = t.x * pv.v[0] + t.y * pv.v[1] + t.z * pv.v[2] + t.w * pv.v[3];
                    }
                }
                __syncthreads();
                int e = 0;
                for (; e + 4 <= ne; e += 4) {
                    const int4 o = *(const int4*)(eoffs + e);
                    DISCO_CHECK(lane_col + o.x >= 0 && lane_col + o.x < kLdsCols && lane_col + o.y >= 0 && lane_col + o.y < kLdsCols &&
                                lane_col + o.z >= 0 && lane_col + o.z < kLdsCols && lane_col + o.w >= 0 && lane_col + o.w < kLdsCols);
                    const float x0 = xs[lane_col + o.x], x1 = xs[lane_col + o.y];
                    const float x2 = xs[lane_col + o.z], x3 = xs[lane_col + o.w];
#pragma unroll
                    for (int j = 0; j < COT; ++j) {
                        acc[j] = fmaf(ew[(e + 0) * COT + j], x0, acc[j]);
                        acc[j] = fmaf(ew[(e + 1) * COT + j], x1, acc[j]);
                        acc[j] = fmaf(ew[(e + 2) * COT + j], x2, acc[j]);
                        acc[j] = fmaf(ew[(e + 3) * COT + j], x3, acc[j]);
                    }
                }
                for (; e < ne; ++e) {
                    DISCO_CHECK(lane_col + eoffs[e] >= 0 && lane_col + eoffs[e] < kLdsCols);
                    const float xv = xs[lane_col + eoffs[e]];
#pragma unroll
                    for (int j = 0; j < COT; ++j) acc[j] = fmaf(ew[e * COT + j], xv, acc[j]);
                }
            }
        }
        if (q < g.nq) {
            const int to = sg.pattern / g.P, r = sg.pattern - (sg.pattern / g.P) * g.P;
            if (sg.slot < 0) {
                const int64_t pix = (int64_t)to * g.nlon_o + (int64_t)q * g.P + r;
#pragma unroll
                for (int j = 0; j < COT; ++j)
                    if (co0 + j < Co) store_val(y, ((int64_t)b * Co + co0 + j) * n_out + pix, acc[j]);
            } else {
                const int B = gridDim.y / n_cotiles;
#pragma unroll
                for (int j = 0; j < COT; ++j)
                    if (co0 + j < Co)
                        partial[(((int64_t)sg.slot * B + b) * Co + co0 + j) * g.nq + q] = acc[j];
            }
        }
    }
}

template <typename T, int COT, int TQ>
hipError_t stencil_launch_tq(const ExecArgs& a, const PackedDev& P, float* partial) {
    const OpGeom& g = a.op->g;
    const int n_qtiles = (g.nq + TQ - 1) / TQ;
    const int n_cot = (a.Co + COT - 1) / COT;
    dim3 grid((unsigned)(P.n_items * n_qtiles), (unsigned)(a.B * n_cot));
    const int tk = timing_begin("stencil", a.stream);
    hipLaunchKernelGGL((k_stencil<T, COT, TQ>), grid, dim3(TQ), 0, a.stream, P.items, P.segs, P.chunks,
                       P.spans, P.offs, P.vals, a.op->cmap_dev, g, (const T*)a.x, (const T*)a.w, (T*)a.y,
                       partial, a.Ci, a.Co, basis_size(a.op->basis), n_qtiles, n_cot, a.w_trans, a.dw_c);
    timing_end(tk, a.stream);
    return hipGetLastError();
}

template <typename T, int COT>
hipError_t stencil_launch(const ExecArgs& a, const PackedDev& P, float* partial) {
    if (P.n_items == 0) return hipSuccess;
    hipError_t e = P.tile == 64    ? stencil_launch_tq<T, COT, 64>(a, P, partial)
                   : P.tile == 128 ? stencil_launch_tq<T, COT, 128>(a, P, partial)
                                   : stencil_launch_tq<T, COT, kTileQ>(a, P, partial);
    if (e != hipSuccess) return e;
    return launch_reduce_partials(a, P, partial);
}

template <typename T>
hipError_t stencil_dispatch(const ExecArgs& a, const PackedDev& P, float* partial) {
    if (a.Co == 1) return stencil_launch<T, 1>(a, P, partial);
    if (a.Co <= 4) return stencil_launch<T, 4>(a, P, partial);
    return stencil_launch<T, 8>(a, P, partial);
}

// The blocked form for one output channel and longitude stride 1: lane l of
// a workgroup owns outputs q0 + 4l .. q0 + 4l + 3.  Entry i of a piece
// (offset dstart + i) adds c_i x[q + dstart + i] to output q, so for the
// block of entries 4b .. 4b + 3 the lane's four outputs need inputs
// x[q0 + 4l + dstart + 4b + m], m = 0..6: the aligned float4 V0 (m < 4) and
// V1 (m >= 4) at LDS columns 4l + 4b and 4l + 4b + 4 of the piece's span;
// V1 is the next block's V0.  Per block: one float4 of x and one float4 of
// folded weights (the same for every lane) from LDS for 16 FMAs.  TILE
// output longitudes per workgroup of TILE / 4 lanes; the chunk budgets scale
// with it, so every tile stages 16 columns and 2 entries per lane.
template <typename T, int TILE>
__global__ __launch_bounds__(TILE / 4) void k_stencil_blocked(const PItem* __restrict__ items,
                                                            const PSeg* __restrict__ segs,
                                                            const SChunk* __restrict__ chunks,
                                                            const SPiece* __restrict__ pieces,
                                                            const PVal* __restrict__ vals,
                                                            const uint8_t* __restrict__ cells,
                                                            const int8_t* __restrict__ cmap, OpGeom g,
                                                            const T* __restrict__ x,
                                                            const T* __restrict__ w, T* __restrict__ y,
                                                            float* __restrict__ partial, int Ci, int K,
                                                            int n_qtiles, int dw_c) {
    constexpr int NT = TILE / 4;
    constexpr int kCols = stencil_cols(TILE);
    constexpr int kEntries = stencil_entries(TILE);
    constexpr int kMaxPieces = kCols / TILE;  // every span is >= one tile
    constexpr int kColsPerThread = kCols / NT;
    constexpr int kEntriesPerThread = kEntries / NT;
    __shared__ float4 xs4[kCols / 4];
    __shared__ float4 ew4[kEntries / 4 + 1];
    __shared__ float4 wt4[kCells];  // [cell][m]
    float* xs = (float*)xs4;
    float* ew = (float*)ew4;

    const int tid = threadIdx.x;
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int item = bid / n_qtiles;
    const int qt = bid - item * n_qtiles;
    const int b = blockIdx.y;
    const int q0 = qt * TILE;
    const int64_t n_in = (int64_t)g.nlat_i * g.nlon_i;
    const int64_t n_out = (int64_t)g.nlat_o * g.nlon_o;
    const PItem it = items[item];

    for (int si = it.seg_begin; si < it.seg_end; ++si) {
        const PSeg sg = segs[si];
        float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
        for (int ci = 0; ci < Ci; ++ci) {
            // One output channel: W[0][ci][.] and the transposed op's
            // W[ci][0][.] are the same row (ordered as k_stencil's table).
            fill_fold_table<T, 1, NT>((float*)wt4, cmap, w, K, b, ci, 0, Ci, 1, false, dw_c);
            const T* xc = x + ((int64_t)b * Ci + ci) * n_in;
            for (int ch = sg.chunk_begin; ch < sg.chunk_end; ++ch) {
                const SChunk C = chunks[ch];
                // The chunk's spans fill LDS columns [0, used) back to back
                // (at most kCols / TILE pieces).  Every thread
                // first issues the loads of all its columns and entries, then
                // stores them, so that a chunk costs one memory latency.
                const int np = C.piece_end - C.piece_begin;
                int pbase[kMaxPieces], prow[kMaxPieces], pstart[kMaxPieces];
                int used = 0;
#pragma unroll
                for (int pp = 0; pp < kMaxPieces; ++pp) {
                    pbase[pp] = kCols;
                    prow[pp] = 0;
                    pstart[pp] = 0;
                    if (pp < np) {
                        const SPiece S = pieces[C.piece_begin + pp];
                        int st = (q0 + S.dstart) % g.nlon_i;
                        if (st < 0) st += g.nlon_i;
                        pbase[pp] = S.lds_base;
                        prow[pp] = S.row;
                        pstart[pp] = st;
                        used = S.lds_base + stencil_span(TILE, S.nblk);
                    }
                }
                float v[kColsPerThread];
#pragma unroll
                for (int u = 0; u < kColsPerThread; ++u) {
                    const int c = tid + u * NT;
                    v[u] = 0.0f;
                    if (c < used) {
                        int base = pbase[0], row = prow[0], st = pstart[0];
#pragma unroll
                        for (int pp = 1; pp < kMaxPieces; ++pp)
                            if (c >= pbase[pp]) { base = pbase[pp]; row = prow[pp]; st = pstart[pp]; }
                        int idx = st + (c - base);
                        while (idx >= g.nlon_i) idx -= g.nlon_i;
                        v[u] = load_val(xc, (int64_t)row + idx);
                    }
                }
                const int ne = C.ent_end - C.ent_begin;
                PVal pv[kEntriesPerThread];
                int pc[kEntriesPerThread];
#pragma unroll
                for (int u = 0; u < kEntriesPerThread; ++u) {
                    const int i = tid + u * NT;
                    pc[u] = 0;
                    if (i < ne) {
                        pv[u] = vals[C.ent_begin + i];
                        pc[u] = cells[C.ent_begin + i];
                    }
                }
                __syncthreads();  // readers of the previous chunk (or channel) are done
#pragma unroll
                for (int u = 0; u < kColsPerThread; ++u) {
                    const int c = tid + u * NT;
                    if (c < used) xs[c] = v[u];
                }
#pragma unroll
                for (int u = 0; u < kEntriesPerThread; ++u) {
                    const int i = tid + u * NT;
                    if (i < ne) {
                        const float4 t = wt4[pc[u]];
                        ew[i] = t.x * pv[u].v[0] + t.y * pv[u].v[1] + t.z * pv[u].v[2] + t.w * pv[u].v[3];
                    }
                }
                __syncthreads();
                int cb = 0;  // the piece's first weight block
                for (int p = C.piece_begin; p < C.piece_end; ++p) {
                    const SPiece S = pieces[p];
                    // lds_base is a multiple of 4, so the lane's blocks are
                    // float4 elements (16-byte aligned, conflict-free rows).
                    // The next block's x and weights are read one block
                    // ahead (the span and the weight table carry one spare
                    // block for the last).
                    const int xb = (S.lds_base >> 2) + tid;
                    DISCO_CHECK(xb >= 0 && xb + S.nblk + 1 < kCols / 4 && cb + S.nblk < kEntries / 4 + 1);
                    float4 V0 = xs4[xb], V1 = xs4[xb + 1];
                    float4 c = ew4[cb];
#pragma unroll 2
                    for (int bb = 0; bb < S.nblk; ++bb) {
                        const float4 V2 = xs4[xb + bb + 2];
                        const float4 cn = ew4[cb + bb + 1];
                        a0 = fmaf(c.x, V0.x, a0); a0 = fmaf(c.y, V0.y, a0); a0 = fmaf(c.z, V0.z, a0); a0 = fmaf(c.w, V0.w, a0);
                        a1 = fmaf(c.x, V0.y, a1); a1 = fmaf(c.y, V0.z, a1); a1 = fmaf(c.z, V0.w, a1); a1 = fmaf(c.w, V1.x, a1);
                        a2 = fmaf(c.x, V0.z, a2); a2 = fmaf(c.y, V0.w, a2); a2 = fmaf(c.z, V1.x, a2); a2 = fmaf(c.w, V1.y, a2);
                        a3 = fmaf(c.x, V0.w, a3); a3 = fmaf(c.y, V1.x, a3); a3 = fmaf(c.z, V1.y, a3); a3 = fmaf(c.w, V1.z, a3);
                        V0 = V1;
                        V1 = V2;
                        c = cn;
                    }
                    cb += S.nblk;
                }
            }
        }
        const int to = sg.pattern / g.P, r = sg.pattern - (sg.pattern / g.P) * g.P;
        const float av[4] = {a0, a1, a2, a3};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = q0 + 4 * tid + j;
            if (q >= g.nq) continue;
            if (sg.slot < 0)
                store_val(y, (int64_t)b * n_out + (int64_t)to * g.nlon_o + (int64_t)q * g.P + r, av[j]);
            else
                partial[((int64_t)sg.slot * gridDim.y + b) * g.nq + q] = av[j];
        }
    }
}

template <typename T, int TILE>
hipError_t stencil_blocked_launch(const ExecArgs& a, const StencilDev& S, float* partial) {
    const OpGeom& g = a.op->g;
    // With a ring walk only the wide patterns, whose items come last.
    PackedDev P = S.P;
    if (a.walk) {
        P.items += S.n_items_light;
        P.n_items -= S.n_items_light;
        P.red_pattern += S.n_split_light;
        P.red_ptr += S.n_split_light;
        P.n_split -= S.n_split_light;
    }
    if (P.n_items == 0) return hipSuccess;
    const int n_qtiles = (g.nq + TILE - 1) / TILE;
    dim3 grid((unsigned)(P.n_items * n_qtiles), (unsigned)a.B);
    const int tk = timing_begin("stencil_blocked", a.stream);
    hipLaunchKernelGGL((k_stencil_blocked<T, TILE>), grid, dim3(TILE / 4), 0, a.stream, P.items, P.segs,
                       S.chunks, S.pieces, S.vals, S.cells, a.op->cmap_dev, g, (const T*)a.x, (const T*)a.w,
                       (T*)a.y, partial, a.Ci, basis_size(a.op->basis), n_qtiles, a.dw_c);
    timing_end(tk, a.stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_reduce_partials(a, P, partial);
}

constexpr uint32_t kNoWeight = 0x80000000u;  // -0

// The folded weights of the ring walk: fw[c][i] = sum_m W[c][map[cell][m]]
// v[m] for every weight i and channel c (one row when dw_c is 0: Ci = Co = 1).
// grid: (ceil(n / 256), rows)
template <typename T>
__global__ __launch_bounds__(256) void k_fold_weights(const PVal* __restrict__ vals, const uint8_t* __restrict__ cells,
                                                      const int8_t* __restrict__ cmap, const T* __restrict__ w,
                                                      float* __restrict__ fw, int n, int K) {
    __shared__ float wt[kCells * 4];
    const int c = blockIdx.y;
    if (threadIdx.x < kCells * 4) {
        const int k = cmap[threadIdx.x];
        wt[threadIdx.x] = k >= 0 ? load_val(w, (int64_t)c * K + k) : 0.0f;
    }
    __syncthreads();
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const PVal v = vals[i];
    const float4 t = *(const float4*)(wt + 4 * cells[i]);
    // A weight without an entry is -0, any other zero +0: where inputs are not
    // finite the walk leaves the former out (kNoWeight).
    const bool none = v.v[0] == 0.0f && v.v[1] == 0.0f && v.v[2] == 0.0f && v.v[3] == 0.0f;
    fw[(int64_t)c * n + i] = none ? -0.0f : t.x * v.v[0] + t.y * v.v[1] + t.z * v.v[2] + t.w * v.v[3] + 0.0f;
}

// Raw buffer access (word 3 of the descriptor for gfx9 raw access): an offset
// at or past num_records reads 0 and drops a store, so that a step issues the
// same number of memory operations whatever it loads and stores, and a wait
// for the next rings' columns does not cover the stores issued after them.
constexpr int kRawBufferFlags = 0x00020000;
constexpr int kBufferOutOfRange = (int)0x80000000u;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, kRawBufferFlags);
}
// Element i, or the four from i on, of a buffer of T (i < 0: out of range).
__device__ __forceinline__ float buffer_load1(const float*, __amdgpu_buffer_rsrc_t r, int i) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, i < 0 ? kBufferOutOfRange : 4 * i, 0, 0));
}
__device__ __forceinline__ float buffer_load1(const uint16_t*, __amdgpu_buffer_rsrc_t r, int i) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, i < 0 ? kBufferOutOfRange : 2 * i, 0, 0) << 16);
}
__device__ __forceinline__ float4 buffer_load4(const float*, __amdgpu_buffer_rsrc_t r, int i) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, i < 0 ? kBufferOutOfRange : 4 * i, 0, 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ __forceinline__ void buffer_store1(float*, __amdgpu_buffer_rsrc_t r, int i, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, i < 0 ? kBufferOutOfRange : 4 * i, 0, 0);
}
__device__ __forceinline__ void buffer_store1(uint16_t*, __amdgpu_buffer_rsrc_t r, int i, float v) {
    __builtin_amdgcn_raw_buffer_store_b16(to_bf16(v), r, i < 0 ? kBufferOutOfRange : 2 * i, 0, 0);
}
__device__ __forceinline__ void buffer_store4(float*, __amdgpu_buffer_rsrc_t r, int i, const float (&v)[4]) {
    const u32x4 u = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
    __builtin_amdgcn_raw_buffer_store_b128(u, r, i < 0 ? kBufferOutOfRange : 4 * i, 0, 0);
}
__device__ __forceinline__ void buffer_store4(uint16_t*, __amdgpu_buffer_rsrc_t r, int i, const float (&v)[4]) {
    const u32x2 u = {(uint32_t)to_bf16(v[0]) | (uint32_t)to_bf16(v[1]) << 16,
                     (uint32_t)to_bf16(v[2]) | (uint32_t)to_bf16(v[3]) << 16};
    __builtin_amdgcn_raw_buffer_store_b64(u, r, i < 0 ? kBufferOutOfRange : 2 * i, 0, 0);
}

constexpr int kWalkLoads = (kWalkMaxPitch + 255) / 256;  // float4 columns per lane of one staged ring
constexpr int kWalkAhead = 4;                            // rings staged one step ahead, in registers
constexpr int kWalkW4 = kWalkPieces * kWalkPats * kWalkLags / 256;  // float4 weights per lane of a step
typedef float v4f __attribute__((ext_vector_type(4)));

enum { kColumns = 0, kInside = 1, kSeam = 2 };  // how a tile's columns are loaded

// Columns 4 lane + 256 k .. + 3 of ring t for the tile at q0 (start: the
// ring's ring_start), or nothing (zeros).  kInside: fp32 tiles away from the
// seam, four columns per load; kSeam: the same, the one lane whose columns
// straddle the seam taking the ring's last four and first four; kColumns:
// column by column (bf16, rings shorter than a slot).
template <typename T, int LOAD>
__device__ __forceinline__ void walk_load_ring(const T* __restrict__ x, __amdgpu_buffer_rsrc_t xr, const OpGeom& g,
                                               int q0, int t, int start, bool on, int pitch,
                                               float4 (&v)[kWalkLoads]) {
    int base = q0 + start;
    if (base >= g.nlon_i) base -= g.nlon_i;
    const int row = t * g.nlon_i;
#pragma unroll
    for (int k = 0; k < kWalkLoads; ++k) {
        const int c = 256 * k + 4 * (int)threadIdx.x;
        const bool in = on && c < pitch;
        if constexpr (LOAD == kInside) {
            v[k] = buffer_load4(x, xr, in ? row + base + c : -1);
        } else if constexpr (LOAD == kSeam) {
            const int i0 = base + c < g.nlon_i ? base + c : base + c - g.nlon_i;
            const int left = g.nlon_i - i0;  // columns before the seam
            const bool cut = left < 4;
            const float4 a = buffer_load4(x, xr, in ? row + (cut ? g.nlon_i - 4 : i0) : -1);
            const float4 b = buffer_load4(x, xr, in && cut ? row : -1);
            v[k].x = left >= 4 ? a.x : left == 3 ? a.y : left == 2 ? a.z : a.w;
            v[k].y = left >= 4 ? a.y : left == 3 ? a.z : left == 2 ? a.w : b.x;
            v[k].z = left >= 4 ? a.z : left == 3 ? a.w : left == 2 ? b.x : b.y;
            v[k].w = left >= 4 ? a.w : left == 3 ? b.x : left == 2 ? b.y : b.z;
        } else {
            float e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                int idx = base + c + u;
                if (idx >= g.nlon_i) idx -= g.nlon_i;
                if (g.nlon_i < kWalkMaxPitch) idx %= g.nlon_i;
                e[u] = buffer_load1(x, xr, in ? row + idx : -1);
            }
            v[k] = make_float4(e[0], e[1], e[2], e[3]);
        }
    }
}

// One piece in registers: the lane's columns from the piece's first one on,
// and the folded weights as A operand (lane i + 4 b: pattern i, lag b).
struct WalkPiece {
    float4 v[5];
    float w;
    int lags;
};
__device__ __forceinline__ void walk_fetch(WalkPiece& P, int piece, const float* __restrict__ wl,
                                           const float4* __restrict__ xl) {
    P.lags = piece & 31;
    P.w = *wl;
    const float4* xp = xl + (piece >> 7);
#pragma unroll
    for (int u = 0; u < 2; ++u) P.v[u] = xp[u];
    if (P.lags > 5) {
        P.v[2] = xp[2];
        if (P.lags > 9) {
            P.v[3] = xp[3];
            if (P.lags > 13) P.v[4] = xp[4];
        }
    }
}

// acc[o][pattern] += w[pattern][j] x[o + j] for lags j = J .. lags - 1: one
// v_mfma_f32_4x4x1_16b_f32 per lag and output o of the lanes (the A block of
// lag j broadcast to all sixteen 4-column blocks: CBSZ = 4, ABID = j).
template <int J>
__device__ __forceinline__ void walk_products(const WalkPiece& P, const float (&x)[20], v4f (&acc)[4]) {
    if constexpr (J < kWalkLags) {
        if (J < P.lags) {
#pragma unroll
            for (int o = 0; o < 4; ++o) acc[o] = __builtin_amdgcn_mfma_f32_4x4x1f32(P.w, x[J + o], acc[o], 4, J, 0);
            walk_products<J + 1>(P, x, acc);
        }
    }
}
__device__ __forceinline__ void walk_piece_products(const WalkPiece& P, v4f (&acc)[4]) {
    const float x[20] = {P.v[0].x, P.v[0].y, P.v[0].z, P.v[0].w, P.v[1].x, P.v[1].y, P.v[1].z,
                         P.v[1].w, P.v[2].x, P.v[2].y, P.v[2].z, P.v[2].w, P.v[3].x, P.v[3].y,
                         P.v[3].z, P.v[3].w, P.v[4].x, P.v[4].y, P.v[4].z, P.v[4].w};
    walk_products<0>(P, x, acc);
}

// The pieces of a step, the next one's columns and weights requested before
// the current one's products; two register sets swap roles.  Lane i of
// `desc` holds piece i; wl: this lane's weight of piece 0 in LDS.
__device__ __forceinline__ void walk_pieces(int n, int desc, const float* __restrict__ wl,
                                            const float4* __restrict__ xl, v4f (&acc)[4]) {
    if (n == 0) return;
    WalkPiece A, B;
    walk_fetch(A, __builtin_amdgcn_readlane(desc, 0), wl, xl);
    int i = 0;
    for (; i + 1 < n; i += 2) {
        walk_fetch(B, __builtin_amdgcn_readlane(desc, i + 1), wl + 64 * (i + 1), xl);
        __builtin_amdgcn_sched_barrier(0);
        walk_piece_products(A, acc);
        const int nx = i + 2 < n ? i + 2 : i + 1;
        walk_fetch(A, __builtin_amdgcn_readlane(desc, nx), wl + 64 * nx, xl);
        __builtin_amdgcn_sched_barrier(0);
        walk_piece_products(B, acc);
    }
    if (i < n) walk_piece_products(A, acc);
}

// The same sums where a staged input is not finite: the products are taken for
// the weights that have an entry only, so that an infinity or NaN reaches the
// outputs whose windows hold it and no others.
__device__ __forceinline__ void walk_pieces_checked(int n, int desc, const float* __restrict__ wlds,
                                                    const float* __restrict__ xl, v4f (&acc)[4]) {
    for (int i = 0; i < n; ++i) {
        const int piece = __builtin_amdgcn_readlane(desc, i);
        const float* x = xl + (piece >> 5);
        for (int j = 0; j < (piece & 31); ++j)
#pragma unroll
            for (int r = 0; r < kWalkPats; ++r) {
                const float w = wlds[kWalkPats * (kWalkLags * i + j) + r];
                if (__float_as_uint(w) == kNoWeight) continue;
#pragma unroll
                for (int o = 0; o < 4; ++o) acc[o][r] = fmaf(w, x[j + o], acc[o][r]);
            }
    }
}

struct WalkArgs {
    int n_steps, run_len, n_runs, n_tiles, n_slots, pitch, n_weights, dw_c, pat_end, back, ahead;
};

// The ring walk (layout: disco_internal.h).  One wave per workgroup: no
// barriers, LDS ordered by the wave's own program order; lane l owns outputs
// q0 + 4 l .. + 3 of the step's patterns.  The products run on the fp32 matrix
// cores, four patterns by 64 outputs per instruction; as VALU FMAs the
// weights would be scalar operands, at which the FMA rate halves.  VEC: four
// outputs per store (P <= 2, whole lanes, aligned rows).
template <typename T, bool VEC, int LOAD>
__device__ __forceinline__ void walk_run(float4* __restrict__ xs4, const WStep* __restrict__ steps,
                                         const int32_t* __restrict__ pieces, const int32_t* __restrict__ ring_start,
                                         const float* __restrict__ fw, const WalkArgs& W, const OpGeom& g,
                                         const T* __restrict__ x, T* __restrict__ y, int item, int q0, int s0, int s1) {
    const int lane = threadIdx.x;
    const int pitch = W.pitch, n_slots = W.n_slots;
    const float* wc = fw + (W.dw_c > 0 ? (int64_t)(item % W.dw_c) * W.n_weights : 0);
    const float4* xl = xs4 + lane;
    const int n_in = g.nlat_i * g.nlon_i, n_out = g.nlat_o * g.nlon_o;
    const __amdgpu_buffer_rsrc_t xr = buffer_of(x + (int64_t)item * n_in, n_in * (int)sizeof(T));
    const __amdgpu_buffer_rsrc_t yr = buffer_of(y + (int64_t)item * n_out, n_out * (int)sizeof(T));
    const int q = q0 + 4 * lane;

    auto load_ring = [&](int t, int start, bool on, float4 (&v)[kWalkLoads]) {
        walk_load_ring<T, LOAD>(x, xr, g, q0, t, start, on, pitch, v);
    };
    uint32_t odd = 0;  // slots with an infinity or NaN (or very large values)
    static_assert(kWalkMaxFloats / kWalkTile <= 32, "a bit for each slot");
    auto put_ring = [&](int slot, bool on, const float4 (&v)[kWalkLoads]) {
        float4* dst = xs4 + slot * (pitch >> 2) + lane;
        bool fine = true;
#pragma unroll
        for (int k = 0; k < kWalkLoads; ++k)
            fine &= fabsf(v[k].x) + fabsf(v[k].y) + fabsf(v[k].z) + fabsf(v[k].w) < INFINITY;
        if (on) odd = (odd & ~(1u << slot)) | (uint32_t)(__ballot(!fine) != 0) << slot;
#pragma unroll
        for (int k = 0; k < kWalkLoads; ++k)
            if (on && 256 * k + 4 * lane < pitch) {
                DISCO_CHECK(slot < n_slots && slot * pitch + 256 * k + 4 * lane + 3 < kWalkMaxFloats);
                dst[64 * k] = v[k];
            }
    };
    // A step's folded weights (n pieces of 64): float4 i of lane l is weights
    // 256 i + 4 l .. + 3.
    float* wlds = (float*)(xs4 + n_slots * (pitch >> 2));
    const __amdgpu_buffer_rsrc_t wr = buffer_of(wc, W.n_weights * 4);
    auto load_weights = [&](const WStep& S, float4 (&v)[kWalkW4]) {
#pragma unroll
        for (int k = 0; k < kWalkW4; ++k) {
            const int i = 256 * k + 4 * lane;
            v[k] = buffer_load4(wc, wr, i < 64 * S.n ? 64 * S.piece + i : -1);
        }
    };
    auto put_weights = [&](const float4 (&v)[kWalkW4]) {
#pragma unroll
        for (int k = 0; k < kWalkW4; ++k) ((float4*)wlds)[64 * k + lane] = v[k];
    };
    WStep S = steps[s0];
    int slot = S.lo % n_slots;  // the next ring's slot
    auto advance = [&](bool on) { slot = !on ? slot : slot + 1 < n_slots ? slot + 1 : 0; };
    {
        float4 wv[kWalkW4];
        load_weights(S, wv);
        for (int t = S.lo; t < S.hi; t += 4) {  // the first window, four rings' loads in flight
            float4 a[4][kWalkLoads];
#pragma unroll
            for (int u = 0; u < 4; ++u) load_ring(t + u, ring_start[t + u < S.hi ? t + u : t], t + u < S.hi, a[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                put_ring(slot, t + u < S.hi, a[u]);
                advance(t + u < S.hi);
            }
        }
        put_weights(wv);
    }
    // Step descriptors run two steps ahead of their use, a step's pieces
    // (lane i holds piece i), weights and new rings one step.
    WStep N = steps[s0 + 1 < s1 ? s0 + 1 : s0];
    // A step without entries has none, and may begin past the last one.
    int desc = lane < S.n ? pieces[S.piece + lane] : 0;
    for (int s = s0; s < s1; ++s) {
        const WStep N2 = steps[s + 2 < s1 ? s + 2 : s1 - 1];
        const int fresh = N.hi - S.hi;  // rings new to the next step's window
        const int desc_next = lane < N.n ? pieces[N.piece + lane] : 0;
        float4 wv[kWalkW4], pf[kWalkAhead][kWalkLoads];
        load_weights(N, wv);
#pragma unroll
        for (int k = 0; k < kWalkAhead; ++k)
            load_ring(S.hi + k, ring_start[S.hi + k < g.nlat_i ? S.hi + k : 0], k < fresh, pf[k]);
        __builtin_amdgcn_wave_barrier();  // the staged columns are written before the reads below
        v4f acc[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) acc[o] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        if (odd == 0) walk_pieces(S.n, desc, wlds + lane, xl, acc);
        else walk_pieces_checked(S.n, desc, wlds, (const float*)xl, acc);
        // Lane l of a product's column block holds its own output column.
        if (VEC && g.P == 2) {
            // The two phases of two output rings, interleaved in memory.
#pragma unroll
            for (int r = 0; r < kWalkPats; r += 2) {
                const int i = q < g.nq && S.pat + r < W.pat_end ? ((S.pat + r) >> 1) * g.nlon_o + 2 * q : -1;
                const float lo4[4] = {acc[0][r], acc[0][r + 1], acc[1][r], acc[1][r + 1]};
                const float hi4[4] = {acc[2][r], acc[2][r + 1], acc[3][r], acc[3][r + 1]};
                buffer_store4(y, yr, i, lo4);
                buffer_store4(y, yr, i < 0 ? i : i + 4, hi4);
            }
        } else if (VEC) {
#pragma unroll
            for (int r = 0; r < kWalkPats; ++r) {
                const float v[4] = {acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
                buffer_store4(y, yr, q < g.nq && S.pat + r < W.pat_end ? (S.pat + r) * g.nlon_o + q : -1, v);
            }
        } else {
#pragma unroll
            for (int r = 0; r < kWalkPats; ++r) {
                const int pat = S.pat + r, to = pat / g.P, ph = pat - to * g.P;
#pragma unroll
                for (int o = 0; o < 4; ++o)
                    buffer_store1(y, yr, q + o < g.nq && pat < W.pat_end ? to * g.nlon_o + (q + o) * g.P + ph : -1,
                                  acc[o][r]);
            }
        }
        __builtin_amdgcn_wave_barrier();  // the step's LDS reads are done before the next rings land
        put_weights(wv);
#pragma unroll
        for (int k = 0; k < kWalkAhead; ++k) {
            put_ring(slot, k < fresh, pf[k]);
            advance(k < fresh);
        }
        for (int t = S.hi + kWalkAhead; t < N.hi; ++t) {
            float4 a[kWalkLoads];
            load_ring(t, ring_start[t], true, a);
            put_ring(slot, true, a);
            advance(true);
        }
        S = N;
        N = N2;
        desc = desc_next;
    }
}

// grid: n_runs * n_tiles * items workgroups of 64 threads, dynamic LDS
// n_slots * pitch + 64 kWalkPieces floats.
template <typename T, bool VEC>
__global__ __launch_bounds__(64, 3) void k_stencil_walk(const WStep* __restrict__ steps, const int32_t* __restrict__ pieces,
                                                     const int32_t* __restrict__ ring_start,
                                                     const float* __restrict__ fw, WalkArgs W, OpGeom g,
                                                     const T* __restrict__ x, T* __restrict__ y) {
    extern __shared__ float4 xs4[];
    // Work item = (item, run, tile), tiles fastest: the workgroups of one XCD
    // share rings and halos in its L2.
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int item = bid / (W.n_runs * W.n_tiles), rt = bid - item * (W.n_runs * W.n_tiles);
    const int run = rt / W.n_tiles, q0 = (rt - run * W.n_tiles) * kWalkTile;
    const int s0 = run * W.run_len, s1 = s0 + W.run_len < W.n_steps ? s0 + W.run_len : W.n_steps;
    // Away from the seam every ring's columns q0 + lag lie in one turn.
    if constexpr (sizeof(T) == 4) {
        if (q0 >= W.back && q0 + W.ahead <= g.nlon_i)
            return walk_run<T, VEC, kInside>(xs4, steps, pieces, ring_start, fw, W, g, x, y, item, q0, s0, s1);
        if (g.nlon_i >= kWalkMaxPitch)
            return walk_run<T, VEC, kSeam>(xs4, steps, pieces, ring_start, fw, W, g, x, y, item, q0, s0, s1);
    }
    walk_run<T, VEC, kColumns>(xs4, steps, pieces, ring_start, fw, W, g, x, y, item, q0, s0, s1);
}

template <typename T>
hipError_t stencil_walk_launch(const ExecArgs& a, const StencilDev& S, float* fw) {
    const WalkDev& W = S.walk;
    const OpGeom& g = a.op->g;
    const int rows = a.dw_c > 0 ? a.dw_c : 1;
    int tk = timing_begin("fold_weights", a.stream);
    hipLaunchKernelGGL(k_fold_weights<T>, dim3((unsigned)((W.n_weights + 255) / 256), (unsigned)rows), dim3(256), 0,
                       a.stream, W.vals, W.cells, a.op->cmap_dev, (const T*)a.w, fw, W.n_weights,
                       basis_size(a.op->basis));
    timing_end(tk, a.stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int n_tiles = (g.nq + kWalkTile - 1) / kWalkTile;
    // Steps per run: long runs stage fewer rings twice, short ones keep more
    // waves in flight; about 8192 workgroups, 1 to 8 steps each.
    const int64_t all = (int64_t)W.n_steps * n_tiles * a.B;
    int run_len = (int)((all + 8191) / 8192);
    run_len = run_len < 1 ? 1 : run_len > 8 ? 8 : run_len;
    const int n_runs = (W.n_steps + run_len - 1) / run_len;
    // Four outputs of a lane in one access: whole lanes, aligned rows.
    const int align = a.dtype == 1 ? 8 : 16;
    const bool vec = g.P <= 2 && g.nq % 4 == 0 && g.nlon_o % 4 == 0 && (uintptr_t)a.y % align == 0;
    const dim3 grid((unsigned)((int64_t)n_runs * n_tiles * a.B));
    const size_t lds = sizeof(float) * ((size_t)W.n_slots * W.pitch + kWalkPats * kWalkLags * kWalkPieces);
    const WalkArgs wa{W.n_steps, run_len, n_runs, n_tiles, W.n_slots, W.pitch, W.n_weights, a.dw_c, W.pat_end, W.back, W.ahead};
    tk = timing_begin("stencil_walk", a.stream);
    if (vec)
        hipLaunchKernelGGL((k_stencil_walk<T, true>), grid, dim3(64), lds, a.stream, W.steps, W.pieces,
                           W.ring_start, (const float*)fw, wa, g, (const T*)a.x, (T*)a.y);
    else
        hipLaunchKernelGGL((k_stencil_walk<T, false>), grid, dim3(64), lds, a.stream, W.steps, W.pieces,
                           W.ring_start, (const float*)fw, wa, g, (const T*)a.x, (T*)a.y);
    timing_end(tk, a.stream);
    return hipGetLastError();
}

// The correlations of dy and x over the ring walk's layout (Sec. 4.2, the
// adjoint of the folded product): corr[split][c][w] = sum over the split's
// batch items and tiles and the outputs q of dy[pattern][q] x[ring][q + lag]
// for every weight w = (piece, lag, pattern) of a group.  One wave per
// (group, channel, split): per tile it stages the step's rings and holds 16
// dy operands (lane i + 4 b: pattern i, output 16 t + b), and one
// v_mfma_f32_4x4x1_16b_f32 takes four patterns by four lags at 16 outputs; the
// sixteen blocks' sums stay in registers until the end.  Rounding: a tile's
// products of one block are two chains of eight, the tiles (at most
// kFoldGradUnits, more are split between waves) are added to their sums; as
// one chain over everything the gradient was further from its 64-bit value than
// that of gathered sums (512 x 1024, 2 x 32 channels: 2.4e-7 against 2.0e-7;
// now 1.4e-7, at the same speed).  Per product one LDS
// read of 64 floats, which with the matrix cores bounds it.
// grid: splits * C * n_groups workgroups of 64, dynamic LDS n_slots * pitch floats.
template <typename T, int LOAD>
__global__ __launch_bounds__(64, 2) void k_walk_grad(const WGroup* __restrict__ groups, const WQuad* __restrict__ quads,
                                                     const WStep* __restrict__ steps,
                                                     const int32_t* __restrict__ ring_start, WalkArgs W, OpGeom g,
                                                     const T* __restrict__ x, const T* __restrict__ dy,
                                                     float* __restrict__ corr, int n_groups, int B, int C, int splits) {
    extern __shared__ float4 xs4[];
    const float* xs = (const float*)xs4;
    const int lane = threadIdx.x, pitch = W.pitch, n_slots = W.n_slots;
    // Work item = (channel, split, group), groups fastest.
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int grp = bid % n_groups, cs = bid / n_groups;
    const int split = cs % splits, c = cs / splits;
    const WGroup G = groups[grp];
    const WStep S = steps[G.step];
    const WQuad mine = quads[G.quad + (lane < G.n ? lane : 0)];  // lane i holds quad i
    const int n_in = g.nlat_i * g.nlon_i, n_out = g.nlat_o * g.nlon_o;
    // This lane's pattern of dy and column of a product.
    const int pat = S.pat + (lane & 3), to = pat / g.P, ph = pat - to * g.P;
    const bool pat_on = pat < W.pat_end;
    const int xcol = (lane >> 2) + (lane & 3);
    v4f acc[kWalkQuads];
#pragma unroll
    for (int k = 0; k < kWalkQuads; ++k) acc[k] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    for (int u = split; u < B * W.n_tiles; u += splits) {
        const int b = u / W.n_tiles, q0 = (u - b * W.n_tiles) * kWalkTile;
        const __amdgpu_buffer_rsrc_t xr = buffer_of(x + ((int64_t)b * C + c) * n_in, n_in * (int)sizeof(T));
        const __amdgpu_buffer_rsrc_t dr = buffer_of(dy + ((int64_t)b * C + c) * n_out, n_out * (int)sizeof(T));
        float A[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int q = q0 + 16 * t + (lane >> 2);
            A[t] = buffer_load1(dy, dr, pat_on && q < g.nq ? to * g.nlon_o + q * g.P + ph : -1);
        }
        int slot = S.lo % n_slots;
        __builtin_amdgcn_wave_barrier();  // the previous tile's reads are done
        for (int t = S.lo; t < S.hi; t += 4) {
            float4 v[4][kWalkLoads];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                walk_load_ring<T, LOAD>(x, xr, g, q0, t + k, ring_start[t + k < S.hi ? t + k : t], t + k < S.hi, pitch,
                                        v[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (t + k < S.hi) {
#pragma unroll
                    for (int l = 0; l < kWalkLoads; ++l)
                        if (256 * l + 4 * lane < pitch) xs4[slot * (pitch >> 2) + 64 * l + lane] = v[k][l];
                    slot = slot + 1 < n_slots ? slot + 1 : 0;
                }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < kWalkQuads; ++k) {
            if (k >= G.n) continue;  // the same for every lane
            const int col = __builtin_amdgcn_readlane(mine.col, k) + xcol;
            DISCO_CHECK(col >= 0 && col + 240 < n_slots * pitch);
            v4f even = {0.0f, 0.0f, 0.0f, 0.0f}, odd = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int t = 0; t < 16; t += 2) {
                even = __builtin_amdgcn_mfma_f32_4x4x1f32(A[t], xs[col + 16 * t], even, 0, 0, 0);
                odd = __builtin_amdgcn_mfma_f32_4x4x1f32(A[t + 1], xs[col + 16 * t + 16], odd, 0, 0, 0);
            }
            acc[k] += even + odd;
        }
    }
    // Lane j + 4 b holds block b's sums for lag j, patterns 0..3.
    float* out = corr + ((int64_t)split * C + c) * W.n_weights;
#pragma unroll
    for (int k = 0; k < kWalkQuads; ++k) {
        if (k >= G.n) continue;
        v4f v = acc[k];
#pragma unroll
        for (int off = 4; off < 64; off <<= 1)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] += __shfl_xor(v[r], off, 64);
        const int w = __builtin_amdgcn_readlane(mine.w, k);
        if (lane < 4) *(v4f*)(out + w + 4 * lane) = v;
    }
}

// partial[c][chunk][k] = sum over the chunk's weights of psi_k times their
// correlation (summed over splits), in 64 bits up to the stored sum.  A weight
// touches four of the K sums, so each thread keeps its own column of them in
// LDS (K selected additions in registers: 32 us for 512 x 1024, 32 channels,
// against 22).  Weights without an entry are left out, whatever their
// correlation holds.  grid: (kFoldGradChunks, C)
__global__ __launch_bounds__(256) void k_walk_grad_contract(const PVal* __restrict__ vals,
                                                            const uint8_t* __restrict__ cells,
                                                            const int8_t* __restrict__ cmap,
                                                            const float* __restrict__ corr, float* __restrict__ partial,
                                                            int n, int C, int splits, int chunks, int K) {
    __shared__ double sums[kSeparableBasis][256];
    __shared__ int map[kCells];
    const int c = blockIdx.y, tid = threadIdx.x;
    if (tid < kCells) {  // four basis functions per cell, a byte each
        int m = 0;
        for (int j = 0; j < 4; ++j) m |= (cmap[4 * tid + j] & 255) << (8 * j);
        map[tid] = m;
    }
#pragma unroll
    for (int k = 0; k < kSeparableBasis; ++k) sums[k][tid] = 0.0;
    __syncthreads();
    for (int i = blockIdx.x * 256 + tid; i < n; i += kFoldGradChunks * 256) {
        const PVal v = vals[i];
        if (v.v[0] == 0.0f && v.v[1] == 0.0f && v.v[2] == 0.0f && v.v[3] == 0.0f) continue;
        double s = 0.0;
        for (int sp = 0; sp < splits; ++sp) s += corr[((int64_t)sp * C + c) * n + i];
        const int m = map[cells[i]];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int kj = (m >> (8 * j)) & 255;
            if (kj < K) sums[kj][tid] += v.v[j] * s;
        }
    }
    __syncthreads();
    for (int k = tid >> 6; k < K; k += 4) {
        const double* row = sums[k] + (tid & 63);
        double v = (row[0] + row[64]) + (row[128] + row[192]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((tid & 63) == 0) partial[((int64_t)c * chunks + blockIdx.x) * K + k] = (float)v;
    }
}

template <typename T>
hipError_t fold_grad(const ExecArgs& a, const StencilDev& S, float* ws) {
    const WalkDev& W = S.walk;
    const OpGeom& g = a.op->g;
    const FoldGradPlan F = fold_grad_plan(a, S);
    float* corr = ws;
    float2* xh = (float2*)((char*)ws + F.corr);
    float2* dyh = (float2*)((char*)xh + F.xhat);
    float* partial = (float*)((char*)dyh + F.dyhat);
    const int C = a.dw_c > 0 ? a.dw_c : 1, B = a.B / C, K = basis_size(a.op->basis);
    const int n_tiles = (g.nq + kWalkTile - 1) / kWalkTile;
    hipError_t e = a.op->n_heavy_rings > 0 ? launch_spectral_fold_grad(a, xh, dyh, partial, F.chunks) : hipSuccess;
    if (e != hipSuccess) return e;
    const WalkArgs wa{W.n_steps, 0, 0, n_tiles, W.n_slots, W.pitch, W.n_weights, a.dw_c, W.pat_end, W.back, W.ahead};
    const dim3 grid((unsigned)((int64_t)F.splits * C * W.n_groups));
    const size_t lds = sizeof(float) * (size_t)W.n_slots * W.pitch;
    int tk = timing_begin("walk_grad", a.stream);
    bool done = false;
    if constexpr (sizeof(T) == 4)
        if (g.nlon_i >= kWalkMaxPitch) {
            hipLaunchKernelGGL((k_walk_grad<T, kSeam>), grid, dim3(64), lds, a.stream, W.groups, W.quads, W.steps,
                               W.ring_start, wa, g, (const T*)a.x, (const T*)a.dy, corr, W.n_groups, B, C, F.splits);
            done = true;
        }
    if (!done)
        hipLaunchKernelGGL((k_walk_grad<T, kColumns>), grid, dim3(64), lds, a.stream, W.groups, W.quads, W.steps,
                           W.ring_start, wa, g, (const T*)a.x, (const T*)a.dy, corr, W.n_groups, B, C, F.splits);
    timing_end(tk, a.stream);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    tk = timing_begin("walk_grad_contract", a.stream);
    hipLaunchKernelGGL(k_walk_grad_contract, dim3(kFoldGradChunks, C), dim3(256), 0, a.stream, W.vals, W.cells,
                       a.op->cmap_dev, corr, partial, W.n_weights, C, F.splits, F.chunks, K);
    timing_end(tk, a.stream);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_weight_grad_reduce_dw(partial, a.dw, a.dtype, C, F.chunks, K, a.stream);
}

template <typename T>
hipError_t stencil_blocked_parts(const ExecArgs& a, const StencilDev& S, float* ws) {
    float* partial = (float*)((char*)ws + walk_ws_bytes(a, S));
    hipError_t e = hipSuccess;
    if (!(a.walk && a.heavy_spectral))
        e = S.tile == kStencilSmallTile ? stencil_blocked_launch<T, kStencilSmallTile>(a, S, partial)
                                        : stencil_blocked_launch<T, kStencilTile>(a, S, partial);
    if (e != hipSuccess || !a.walk) return e;
    return stencil_walk_launch<T>(a, S, ws);
}

}  // namespace

DISCO_BOUNDS_READER(bounds_flag_stencil)

hipError_t launch_stencil_blocked(const ExecArgs& a, const StencilDev& S, float* ws) {
    if (S.tile != kStencilSmallTile && S.tile != kStencilTile) return hipErrorInvalidValue;
    if (a.dw) return a.dtype == 1 ? fold_grad<uint16_t>(a, S, ws) : fold_grad<float>(a, S, ws);
    return a.dtype == 1 ? stencil_blocked_parts<uint16_t>(a, S, ws) : stencil_blocked_parts<float>(a, S, ws);
}

hipError_t launch_stencil(const ExecArgs& a, const PackedDev& P, float* partial_ws) {
    return a.dtype == 1 ? stencil_dispatch<uint16_t>(a, P, partial_ws) : stencil_dispatch<float>(a, P, partial_ws);
}

}  // namespace disco
