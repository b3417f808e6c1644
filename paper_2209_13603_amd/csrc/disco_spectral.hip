// disco_spectral.hip -- the spectral path for heavy output rings.
//
// Near the poles an output ring's windows span whole input rings, so its sum
// over one input ring is a circular cross-correlation along longitude
// (Sec. 4.2: one pattern reused at every output longitude).  Three kernels
// evaluate it exactly through the DFT (ring lengths powers of two; Mi, Mo half
// the input and output ones, M the larger):
//   k_rfft_rings : Xhat of every input ring a heavy ring reads (real 2 Mi-point
//                  DFT as an Mi-point complex Stockham FFT in LDS + split),
//   k_spectral   : Yhat[co][m] = sum_{t_i, ci} Xhat[t_i][ci][m] sum_k W[co][ci][k]
//                  conj(Vhat_k[m]), using Vhat_{3a+2} = conj(Vhat_{3a}) and
//                  real Vhat_{3a+1} (9 stored floats per pair and frequency),
//   k_spectral_fold: the same for one-channel items of ops without a longitude
//                  stride, W folded into the tables' rows (every basis;
//                  depthwise channels),
//   k_irfft_rings: y of each heavy ring from Yhat (inverse real DFT); a ring
//                  whose Yhat is not finite is summed directly, so that an
//                  infinity or NaN of x reaches the outputs whose windows hold
//                  it and no others, as in the direct kernels.
// When the ring lengths differ (GEO) the longer one carries the tables: an
// upsampling op reads the input's spectrum repeated, a downsampling op sums
// the `alias` frequencies that fold onto each output frequency.
// Vhat is precomputed on the host in fp64 and scaled by 1 / (2 M); the device
// transforms are unnormalised.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "disco_internal.h"

namespace disco {

namespace {

constexpr int kFftBlock = 256;
constexpr int kFftBatch = 8;  // global loads per thread in flight while staging a ring

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

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float2 conjf2(float2 a) { return make_float2(a.x, -a.y); }

// Twiddles in LDS as two short tables, hi[t >> 6] = tw[64 (t >> 6)] and
// lo[t & 63] = tw[t & 63], whose product is tw[t] = exp(-2 pi i t / (2M))
// (t < M) to a few ulp: 33.5 KB of LDS per FFT workgroup at M = 2048
// instead of 48 KB with the whole table, so four workgroups share a CU.
constexpr int kTwLo = 64;
__host__ __device__ constexpr int tw_hi_len(int M) { return M > kTwLo ? M / kTwLo : 1; }

// Fills the two tables from the global table tw, every tws-th entry of it
// (the table is the longer ring's; t < M); all threads.
__device__ __forceinline__ void load_twiddles(const float2* __restrict__ tw, float2* __restrict__ thi,
                                              float2* __restrict__ tlo, int M, int tws) {
    for (int i = threadIdx.x; i < kTwLo + tw_hi_len(M); i += blockDim.x) {
        if (i < kTwLo) {
            if (i < M) tlo[i] = tw[i * tws];
        } else {
            thi[i - kTwLo] = tw[kTwLo * (i - kTwLo) * tws];
        }
    }
}

// Work item of a products' launch of nx blocks of bins, H rings and nz channel
// groups (grid nx H nz in x): consecutive workgroups go to the 8 XCDs in
// turn, so each XCD is given a contiguous run of rings, taken in turn from
// the two ends of the list: neighbouring rings share input rings, and rings
// mirrored about the equator their tables, in that XCD's L2.
__device__ __forceinline__ void spec_item(int nx, int H, int nz, int* ix, int* h, int* iz) {
    const int nb = (int)gridDim.x, xcd = (int)blockIdx.x & 7, local = (int)blockIdx.x >> 3;
    const int per = nb >> 3, rem = nb & 7;
    int b = xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
    *iz = b % nz;
    b /= nz;
    *ix = b % nx;
    b /= nx;
    *h = b & 1 ? H - 1 - (b >> 1) : b >> 1;
}

// Ring lengths of an op's products: tables over bins 0..M of the longer
// ring, Xhat over 0..Mi, Yhat over 0..Mo, `alias` = the downsampling factor.
struct SpecGeom { int M, Mi, Mo, alias; };

// Bin m of Yhat, alias j: the table bin mv and the input bin mx, and the
// signs of the imaginary parts of conj(Vhat) (sv) and Xhat (sx) there (both
// signals are real, so bins past the middle are conjugates).
__device__ __forceinline__ void spec_bins(const SpecGeom& S, int m, int j, int* mv, int* mx, float* sv, float* sx) {
    int f = m + 2 * j * S.Mo;  // < 2 M
    *sv = 1.0f;
    *sx = 1.0f;
    if (f > S.M) {
        f = 2 * S.M - f;
        *sv = -1.0f;
        *sx = -1.0f;
    }
    *mv = f;
    if (S.Mi < S.M) {  // upsampling: f <= M, the input's spectrum repeats
        f &= 2 * S.Mi - 1;
        if (f > S.Mi) {
            f = 2 * S.Mi - f;
            *sx = -1.0f;
        }
    }
    *mx = f;
}

// exp(-/+ 2 pi i t / (2M)) for t in [0, 2M) (the upper half is the negative
// of the lower).
__device__ __forceinline__ float2 tw_at(const float2* __restrict__ thi, const float2* __restrict__ tlo, int t,
                                        int M, bool inverse) {
    const bool upper = t >= M;
    const int tt = upper ? t - M : t;
    float2 w = cmul(thi[tt >> 6], tlo[tt & (kTwLo - 1)]);
    if (upper) w = make_float2(-w.x, -w.y);
    if (inverse) w.y = -w.y;
    return w;
}

// M-point complex FFT (M a power of two) in LDS, Stockham autosort between
// buffers a and b: radix-4 stages, then one radix-2 stage if log2 M is odd;
// sign -1 (forward) or +1 (inverse, unnormalised).  A stage combining
// sub-transforms of length Ls reads a[j + r M / R] (r < R), twiddles input
// r by exp(-/+ 2 pi i r k / (R Ls)) with k = j mod Ls, takes the R-point DFT
// and writes output s to b[R (j - k) + k + s Ls].  Returns the buffer with
// the result.
__device__ __forceinline__ float2* fft_lds(float2* a, float2* b, int M, const float2* __restrict__ thi,
                                          const float2* __restrict__ tlo, bool inverse) {
    int Ls = 1;
    const int q = M >> 2;
    for (; 4 * Ls <= M; Ls <<= 2) {
        const int tstep = M / (2 * Ls);
        for (int j = threadIdx.x; j < q; j += blockDim.x) {
            const int k = j & (Ls - 1);
            const int t = k * tstep;
            const float2 v0 = a[j];
            const float2 v1 = cmul(a[j + q], tw_at(thi, tlo, t, M, inverse));
            const float2 v2 = cmul(a[j + 2 * q], tw_at(thi, tlo, 2 * t, M, inverse));
            const float2 v3 = cmul(a[j + 3 * q], tw_at(thi, tlo, 3 * t, M, inverse));
            const float2 s02 = cadd(v0, v2), d02 = csub(v0, v2);
            const float2 s13 = cadd(v1, v3), d13 = csub(v1, v3);
            // -i d13 (forward) or +i d13 (inverse)
            const float2 jd13 = inverse ? make_float2(-d13.y, d13.x) : make_float2(d13.y, -d13.x);
            const int o = ((j - k) << 2) + k;
            b[o] = cadd(s02, s13);
            b[o + Ls] = cadd(d02, jd13);
            b[o + 2 * Ls] = csub(s02, s13);
            b[o + 3 * Ls] = csub(d02, jd13);
        }
        __syncthreads();
        float2* tmp = a;
        a = b;
        b = tmp;
    }
    if (2 * Ls == M) {
        const int half = M >> 1, tstep = M / Ls;
        for (int j = threadIdx.x; j < half; j += blockDim.x) {
            const int k = j & (Ls - 1);
            const float2 c0 = a[j];
            const float2 c1 = cmul(a[j + half], tw_at(thi, tlo, k * tstep, M, inverse));
            const int o = ((j - k) << 1) + k;
            b[o] = cadd(c0, c1);
            b[o + Ls] = csub(c0, c1);
        }
        __syncthreads();
        float2* tmp = a;
        a = b;
        b = tmp;
    }
    return a;
}

// Xhat[slot][b][ci][m], m in [0, M]: real DFT of ring slot_ring[slot] of x,
// the bins 0 < m < M multiplied by `interior` (2 gives the weights of a sum
// over the whole spectrum of a real signal, for Parseval's identity).
// grid: (n_slots, B * Ci)
template <typename T>
__global__ __launch_bounds__(kFftBlock) void k_rfft_rings(const int32_t* __restrict__ slot_ring,
                                                         const T* __restrict__ x, const float2* __restrict__ tw,
                                                         float2* __restrict__ xh, int B, int Ci, int nlat, int M,
                                                         int tws, float interior) {
    extern __shared__ float2 sm[];
    float2* a = sm;
    float2* bb = sm + M;
    float2* tlo = sm + 2 * M;
    float2* thi = tlo + kTwLo;
    const int slot = blockIdx.x;
    const int b = blockIdx.y / Ci, ci = blockIdx.y - (blockIdx.y / Ci) * Ci;
    const int N = 2 * M;
    const T* row = x + (((int64_t)b * Ci + ci) * nlat + slot_ring[slot]) * N;
    // Loads in batches of kFftBatch per thread, all issued before the LDS
    // writes (a loop with a run-time trip count would otherwise wait for
    // each load in turn).
    load_twiddles(tw, thi, tlo, M, tws);
    for (int j0 = threadIdx.x; j0 < M; j0 += kFftBatch * kFftBlock) {
        float2 v[kFftBatch];
#pragma unroll
        for (int u = 0; u < kFftBatch; ++u) {
            const int j = j0 + u * kFftBlock;
            if (j < M) v[u] = make_float2(load_val(row, 2 * j), load_val(row, 2 * j + 1));
        }
#pragma unroll
        for (int u = 0; u < kFftBatch; ++u) {
            const int j = j0 + u * kFftBlock;
            if (j < M) a[j] = v[u];
        }
    }
    __syncthreads();
    const float2* Z = fft_lds(a, bb, M, thi, tlo, false);
    float2* out = xh + (((int64_t)slot * B + b) * Ci + ci) * (M + 1);
    for (int m = threadIdx.x; m <= M; m += blockDim.x) {
        const float2 zm = Z[m & (M - 1)];
        const float2 zc = conjf2(Z[(M - m) & (M - 1)]);
        const float2 e = make_float2(0.5f * (zm.x + zc.x), 0.5f * (zm.y + zc.y));
        const float2 dif = csub(zm, zc);
        const float2 o = make_float2(0.5f * dif.y, -0.5f * dif.x);  // (zm - zc) / (2i)
        const float2 w = tw_at(thi, tlo, m, M, false);  // m = M gives -1
        const float2 v = cadd(e, cmul(w, o));
        const float sc = m == 0 || m == M ? 1.0f : interior;
        out[m] = make_float2(sc * v.x, sc * v.y);
    }
}

// One (ring pair, output bin)'s share of the per-pair sums of k_spectral and
// k_spectral_z for input channels ci0 .. ci0 + SC - 1: E, F, G[c][a] +=
// (Re Vhat_3a, Im Vhat_3a, Vhat_3a+1) X.  tb: the pair's table (bit 31: an
// equator mirror, rows a = 0 and a = 2 exchanged); xp: the input ring's Xhat.
template <bool GEO, int SC>
__device__ __forceinline__ void pair_sums(const SpecGeom& S, int m, int32_t tb, const float* __restrict__ vs,
                                          const float2* __restrict__ xp, int ci0, int Ci, float2 (&E)[SC][3],
                                          float2 (&F)[SC][3], float2 (&G)[SC][3]) {
    const int64_t vstride = (int64_t)(S.M + 1), xstride = GEO ? (int64_t)(S.Mi + 1) : vstride;
    const int r0 = tb < 0 ? 6 : 0;
    const float* vt = vs + (int64_t)(tb & 0x7fffffff) * 9 * vstride;
    for (int al = 0; al < (GEO ? S.alias : 1); ++al) {
        int mv = m, mx = m;
        float sv = 1.0f, sx = 1.0f;
        if constexpr (GEO) spec_bins(S, m, al, &mv, &mx, &sv, &sx);
        const float* v = vt + mv;
        float V[9];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            V[j] = v[(r0 + j) * vstride];
            V[3 + j] = v[(3 + j) * vstride];
            V[6 + j] = v[(6 - r0 + j) * vstride];
        }
        if constexpr (GEO) {
            V[1] *= sv;
            V[4] *= sv;
            V[7] *= sv;
        }
        const float2* xr = xp + mx;
#pragma unroll
        for (int c = 0; c < SC; ++c) {
            float2 X = ci0 + c < Ci ? xr[(int64_t)(ci0 + c) * xstride] : make_float2(0.0f, 0.0f);
            if constexpr (GEO) X.y *= sx;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                E[c][a].x = fmaf(V[3 * a + 0], X.x, E[c][a].x);
                E[c][a].y = fmaf(V[3 * a + 0], X.y, E[c][a].y);
                F[c][a].x = fmaf(V[3 * a + 1], X.x, F[c][a].x);
                F[c][a].y = fmaf(V[3 * a + 1], X.y, F[c][a].y);
                G[c][a].x = fmaf(V[3 * a + 2], X.x, G[c][a].x);
                G[c][a].y = fmaf(V[3 * a + 2], X.y, G[c][a].y);
            }
        }
    }
}

// Yhat[h][b][co][m] for heavy ring h.  grid: (ceil((Mo+1)/BLK), n_rings, B * n_cotiles)
template <typename T, int COT, int BLK, bool GEO>
__global__ __launch_bounds__(BLK) void k_spectral(const int32_t* __restrict__ pair_ptr,
                                                       const int32_t* __restrict__ pair_slot,
                                                       const int32_t* __restrict__ pair_tab,
                                                       const float* __restrict__ vs,
                                                       const float2* __restrict__ xh,
                                                       const T* __restrict__ w, float2* __restrict__ yh,
                                                       int B, int Ci, int Co, SpecGeom S, int n_cotiles,
                                                       bool w_trans) {
    // Input channels per accumulation pass.
    static_assert(COT <= 32, "output tiles of at most 32 channels");
    constexpr int SC = 4;
    // This pass's weights as (W_3a + W_3a+2, W_3a+2 - W_3a, W_3a+1) for each
    // (input channel, output channel, a), staged in LDS and read back by
    // broadcast (as uniform scalar loads they would need more SGPRs than
    // there are and spill).
    __shared__ float wsd[SC * COT * 9];
    const int m = blockIdx.x * BLK + threadIdx.x;
    const int h = blockIdx.y;
    const int b = blockIdx.z / n_cotiles;
    const int co0 = (blockIdx.z - b * n_cotiles) * COT;
    const bool active = m <= S.Mo;  // lanes past Mo still take part in the barriers
    const int p0 = pair_ptr[h], p1 = pair_ptr[h + 1];
    const int64_t vstride = (int64_t)(S.M + 1), xstride = GEO ? (int64_t)(S.Mi + 1) : vstride;
    const int64_t ystride = GEO ? (int64_t)(S.Mo + 1) : vstride;
    float2 Y[COT];
#pragma unroll
    for (int j = 0; j < COT; ++j) Y[j] = make_float2(0.0f, 0.0f);
    for (int ci0 = 0; ci0 < Ci; ci0 += SC) {
        __syncthreads();  // the previous pass's reads of wsd are done
        for (int idx = threadIdx.x; idx < SC * COT * 3; idx += BLK) {
            const int c = idx / (COT * 3), r = idx - c * (COT * 3), j = r / 3, a = r - j * 3;
            const int ci = ci0 + c < Ci ? ci0 + c : Ci - 1;  // E, F, G are zero past Ci
            const int co = co0 + j < Co ? co0 + j : Co - 1;
            const int64_t base = w_trans ? ((int64_t)ci * Co + co) * kBasis : ((int64_t)co * Ci + ci) * kBasis;
            const float w0 = load_val(w, base + 3 * a), w1 = load_val(w, base + 3 * a + 1),
                        w2 = load_val(w, base + 3 * a + 2);
            wsd[3 * idx + 0] = w0 + w2;
            wsd[3 * idx + 1] = w2 - w0;
            wsd[3 * idx + 2] = w1;
        }
        __syncthreads();
        if (!active) continue;
        float2 E[SC][3], F[SC][3], G[SC][3];
#pragma unroll
        for (int c = 0; c < SC; ++c)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                E[c][a] = make_float2(0.0f, 0.0f);
                F[c][a] = make_float2(0.0f, 0.0f);
                G[c][a] = make_float2(0.0f, 0.0f);
            }
        for (int p = p0; p < p1; ++p) {
            pair_sums<GEO, SC>(S, m, pair_tab[p], vs, xh + (((int64_t)pair_slot[p] * B + b) * Ci) * xstride, ci0, Ci, E,
                               F, G);
        }
        // Yhat[co] += sum_{c,a} (W_3a + W_3a+2) E + i (W_3a+2 - W_3a) F + W_3a+1 G
#pragma unroll
        for (int j = 0; j < COT; ++j) {
#pragma unroll
            for (int c = 0; c < SC; ++c) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float* wd = wsd + 3 * ((c * COT + j) * 3 + a);
                    const float S = wd[0], D = wd[1], w1 = wd[2];
                    Y[j].x = fmaf(S, E[c][a].x, fmaf(-D, F[c][a].y, fmaf(w1, G[c][a].x, Y[j].x)));
                    Y[j].y = fmaf(S, E[c][a].y, fmaf(D, F[c][a].x, fmaf(w1, G[c][a].y, Y[j].y)));
                }
            }
        }
    }
    if (!active) return;
#pragma unroll
    for (int j = 0; j < COT; ++j)
        if (co0 + j < Co) yh[(((int64_t)h * B + b) * Co + co0 + j) * ystride + m] = Y[j];
}

// The gathered sums of the heavy rings in the frequency domain: the products
// of k_spectral without the channel contraction, Zhat[h][b][ci * 9 + k][m] =
// sum over the ring's pairs of Xhat[slot][ci][m] conj(Vhat_k[pair][m]), the
// nine planes of each input channel from the same E, F, G sums (k = 3a:
// E - iF, 3a + 1: G, 3a + 2: E + iF in the conjugate convention of
// k_spectral).  grid: (ceil((Mo+1)/256), n_rings, B * ceil(Ci / 4))
template <bool GEO>
__global__ __launch_bounds__(kFftBlock) void k_spectral_z(const int32_t* __restrict__ pair_ptr,
                                                         const int32_t* __restrict__ pair_slot,
                                                         const int32_t* __restrict__ pair_tab,
                                                         const float* __restrict__ vs,
                                                         const float2* __restrict__ xh, float2* __restrict__ zh,
                                                         int B, int Ci, SpecGeom S, int n_cg) {
    constexpr int SC = 4;
    const int m = blockIdx.x * kFftBlock + threadIdx.x;
    if (m > S.Mo) return;  // no barriers below
    const int h = blockIdx.y;
    const int b = blockIdx.z / n_cg;
    const int ci0 = (blockIdx.z - b * n_cg) * SC;
    const int p0 = pair_ptr[h], p1 = pair_ptr[h + 1];
    const int64_t xstride = S.Mi + 1, ystride = S.Mo + 1;
    float2 E[SC][3], F[SC][3], G[SC][3];
#pragma unroll
    for (int c = 0; c < SC; ++c)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            E[c][a] = make_float2(0.0f, 0.0f);
            F[c][a] = make_float2(0.0f, 0.0f);
            G[c][a] = make_float2(0.0f, 0.0f);
        }
    for (int p = p0; p < p1; ++p)
        pair_sums<GEO, SC>(S, m, pair_tab[p], vs, xh + (((int64_t)pair_slot[p] * B + b) * Ci) * xstride, ci0, Ci, E, F,
                           G);
    const int Co = Ci * kBasis;
#pragma unroll
    for (int c = 0; c < SC; ++c) {
        if (ci0 + c >= Ci) continue;
        float2* zr = zh + (((int64_t)h * B + b) * Co + (int64_t)(ci0 + c) * kBasis) * ystride + m;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            zr[(3 * a + 0) * ystride] = make_float2(E[c][a].x + F[c][a].y, E[c][a].y - F[c][a].x);
            zr[(3 * a + 1) * ystride] = G[c][a];
            zr[(3 * a + 2) * ystride] = make_float2(E[c][a].x - F[c][a].y, E[c][a].y + F[c][a].x);
        }
    }
}

// Rows of a table (see disco_spectral_plan.cpp) per basis, which of them are
// imaginary parts, and the row an equator mirror reads instead.
template <int BASIS> struct FoldRows;
template <> struct FoldRows<DISCO_BASIS_BILINEAR_3X3> {
    static constexpr int K = 9;
    static constexpr bool imag(int r) { return r % 3 == 1; }
    static constexpr int mirror(int r) { return 3 * (2 - r / 3) + r % 3; }
    // The weight row r's value is multiplied with: conj(Vhat_3a) and Vhat_3a
    // = Re -/+ i Im pair up.
    template <class W> static __device__ float weight(W w, int r) {
        const int a = 3 * (r / 3);
        return r % 3 == 0 ? w(a) + w(a + 2) : r % 3 == 1 ? w(a + 2) - w(a) : w(a + 1);
    }
    // Basis function k's sum from the rows' sums (conj(Vhat_3a) against Q, then Vhat_3a).
    static __device__ float basis(const float (&g)[K], int k) {
        const int a = 3 * (k / 3);
        return k % 3 == 0 ? g[a] + g[a + 1] : k % 3 == 2 ? g[a] - g[a + 1] : g[a + 2];
    }
};
template <> struct FoldRows<DISCO_BASIS_AXISYMMETRIC_4> {
    static constexpr int K = 4;
    static constexpr bool imag(int) { return false; }
    static constexpr int mirror(int r) { return r; }
    template <class W> static __device__ float weight(W w, int r) { return w(r); }
    static __device__ float basis(const float (&g)[K], int k) { return g[k]; }
};
template <> struct FoldRows<DISCO_BASIS_SEPARABLE_4X4> {
    static constexpr int K = 16;
    static constexpr bool imag(int r) { return r % 4 == 2; }
    static constexpr int mirror(int r) { return r % 4 == 0 ? r + 3 : r % 4 == 3 ? r - 3 : r; }
    template <class W> static __device__ float weight(W w, int r) {
        const int a = r & ~3;
        return r % 4 == 0 ? w(a) : r % 4 == 1 ? w(a + 1) + w(a + 3) : r % 4 == 2 ? w(a + 3) - w(a + 1) : w(a + 2);
    }
    static __device__ float basis(const float (&g)[K], int k) {
        const int a = k & ~3;
        return k % 4 == 0 ? g[a] : k % 4 == 2 ? g[a + 3] : k % 4 == 1 ? g[a + 1] + g[a + 2] : g[a + 1] - g[a + 2];
    }
};

// One-channel items: Yhat[h][item][m] = sum over the ring's pairs of
// Xhat[slot][item][m] sum_k w[k] conj(Vhat_k[pair][m]), item b C + c taking
// row c of W (C = 1: row 0).  A wave takes 64 bins of CT channels and BT batch
// items: a table row is read once for all of them and the folded factor of a
// (channel, pair, bin) once for the BT items.  What bounds it: the tables and
// Xhat from L2 or HBM (4 K + 8 CT BT bytes per pair and bin), so fewer items
// per wave cost more (2048 x 4096, 8 channels: 74 us with eight, 105 us with
// four, the rings not ordered by XCD).
// GEO: an upsampling op (the ring walk beside it has no longitude stride).
// grid: nx H nz (spec_item), nx = ceil((Mo+1)/64), nz = ceil(C / CT) * ceil(B / BT)
template <typename T, int BASIS, int CT, int BT, bool GEO>
__global__ __launch_bounds__(64) void k_spectral_fold(const int32_t* __restrict__ pair_ptr,
                                                      const int32_t* __restrict__ pair_slot,
                                                      const int32_t* __restrict__ pair_tab,
                                                      const float* __restrict__ vs, const float2* __restrict__ xh,
                                                      const T* __restrict__ w, float2* __restrict__ yh, int B, int C,
                                                      SpecGeom S, int n_rings) {
    using R = FoldRows<BASIS>;
    constexpr int K = R::K;
    __shared__ float cw[CT * K];  // [channel][row]
    const int lane = threadIdx.x, nct = (C + CT - 1) / CT;
    int ix, h, iz;
    spec_item((S.Mo + 64) / 64, n_rings, nct * ((B + BT - 1) / BT), &ix, &h, &iz);
    const int c0 = (iz % nct) * CT, b0 = (iz / nct) * BT;
    const int mo = 64 * ix + lane, m = mo < S.Mo ? mo : S.Mo;  // lanes past Mo repeat it
    for (int i = lane; i < CT * K; i += 64) {
        const T* wr = w + (int64_t)(c0 + i / K < C ? c0 + i / K : C - 1) * K;
        cw[i] = R::weight([&](int k) { return load_val(wr, k); }, i % K);
    }
    __syncthreads();
    const int64_t vstride = (int64_t)(S.M + 1), xstride = GEO ? (int64_t)(S.Mi + 1) : vstride;
    const int64_t ystride = GEO ? (int64_t)(S.Mo + 1) : vstride;
    // Items past the tensor read its first one and are not stored.
    auto item = [&](int ct, int bt) { return c0 + ct < C && b0 + bt < B ? (b0 + bt) * C + c0 + ct : 0; };
    float2 Y[CT][BT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int bt = 0; bt < BT; ++bt) Y[ct][bt] = make_float2(0.0f, 0.0f);
    for (int p = pair_ptr[h]; p < pair_ptr[h + 1]; ++p) {
        const int32_t tb = pair_tab[p];
        const float* vt = vs + (int64_t)(tb & 0x7fffffff) * K * vstride;
        const float2* xp = xh + (int64_t)pair_slot[p] * B * C * xstride;
        int mv = m, mx = m;
        float sv = 1.0f, sx = 1.0f;  // mv = m <= M here, so sv = 1
        if constexpr (GEO) spec_bins(S, m, 0, &mv, &mx, &sv, &sx);
        float V[K];
        float2 X[CT][BT];
#pragma unroll
        for (int r = 0; r < K; ++r) V[r] = vt[(tb < 0 ? R::mirror(r) : r) * vstride + mv];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int bt = 0; bt < BT; ++bt) X[ct][bt] = xp[(int64_t)item(ct, bt) * xstride + mx];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            float fr = 0.0f, fi = 0.0f;
#pragma unroll
            for (int r = 0; r < K; ++r) {
                if (R::imag(r)) fi = fmaf(cw[ct * K + r], V[r], fi);
                else fr = fmaf(cw[ct * K + r], V[r], fr);
            }
#pragma unroll
            for (int bt = 0; bt < BT; ++bt) {
                float2 x = X[ct][bt];
                if constexpr (GEO) x.y *= sx;
                float2& y = Y[ct][bt];
                y.x = fmaf(fr, x.x, y.x);
                y.y = fmaf(fr, x.y, y.y);
                if constexpr (BASIS != DISCO_BASIS_AXISYMMETRIC_4) {
                    y.x = fmaf(-fi, x.y, y.x);
                    y.y = fmaf(fi, x.x, y.y);
                }
            }
        }
    }
    if (mo > S.Mo) return;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int bt = 0; bt < BT; ++bt)
            if (c0 + ct < C && b0 + bt < B)
                yh[((int64_t)h * B * C + (b0 + bt) * C + c0 + ct) * ystride + m] = Y[ct][bt];
}

// The weight gradient's share of ring h: with Q = sum_b Xhat conj(DYhat) of a
// (pair, bin), dW_k gains Re(Q conj(Vhat_k)), so each table row is summed
// against Re Q, or Im Q for imaginary parts, and the rows of one conjugate
// pair of basis functions are combined at the end.  DYhat: the real DFT of dy
// on the op's rings, interior bins doubled (Parseval).  A wave takes every
// kFoldGradSegments-th block of 64 bins of one ring for CT channels.
// partial: [C][chunks][K], chunk kFoldGradChunks + h kFoldGradSegments + segment.
// grid: kFoldGradSegments * n_rings * ceil(C / CT) (spec_item)
template <int BASIS, int CT, bool GEO>
__global__ __launch_bounds__(64) void k_spectral_fold_grad(const int32_t* __restrict__ pair_ptr,
                                                           const int32_t* __restrict__ pair_slot,
                                                           const int32_t* __restrict__ pair_tab,
                                                           const float* __restrict__ vs,
                                                           const float2* __restrict__ xh,
                                                           const float2* __restrict__ dyh, float* __restrict__ partial,
                                                           int B, int C, int chunks, SpecGeom S, int n_rings) {
    using R = FoldRows<BASIS>;
    constexpr int K = R::K;
    const int lane = threadIdx.x, nct = (C + CT - 1) / CT;
    int seg, h, iz;
    spec_item(kFoldGradSegments, n_rings, nct, &seg, &h, &iz);
    const int c0 = iz * CT;
    const int64_t vstride = (int64_t)(S.M + 1), xstride = (int64_t)(S.Mi + 1), ystride = (int64_t)(S.Mo + 1);
    float G[CT][K];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < K; ++r) G[ct][r] = 0.0f;
    for (int ix = seg; 64 * ix <= S.Mo; ix += kFoldGradSegments) {
        const int mo = 64 * ix + lane, m = mo < S.Mo ? mo : S.Mo;
        const float on = mo <= S.Mo ? 1.0f : 0.0f;
        for (int p = pair_ptr[h]; p < pair_ptr[h + 1]; ++p) {
            const int32_t tb = pair_tab[p];
            const float* vt = vs + (int64_t)(tb & 0x7fffffff) * K * vstride;
            const float2* xp = xh + (int64_t)pair_slot[p] * B * C * xstride;
            const float2* dp = dyh + (int64_t)h * B * C * ystride + m;
            int mv = m, mx = m;
            float sv = 1.0f, sx = 1.0f;
            if constexpr (GEO) spec_bins(S, m, 0, &mv, &mx, &sv, &sx);
            float V[K];
#pragma unroll
            for (int r = 0; r < K; ++r) V[r] = on * vt[(tb < 0 ? R::mirror(r) : r) * vstride + mv];
            float qr[CT], qi[CT];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) qr[ct] = qi[ct] = 0.0f;
            // Batch items in chains of sixteen.
            for (int b0 = 0; b0 < B; b0 += 16) {
                float cr[CT], ci[CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) cr[ct] = ci[ct] = 0.0f;
                for (int b = b0; b < (b0 + 16 < B ? b0 + 16 : B); ++b)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        const int64_t item = (int64_t)b * C + (c0 + ct < C ? c0 + ct : C - 1);
                        const float2 X = xp[item * xstride + mx], D = dp[item * ystride];
                        const float xy = GEO ? sx * X.y : X.y;
                        cr[ct] = fmaf(X.x, D.x, fmaf(xy, D.y, cr[ct]));
                        ci[ct] = fmaf(xy, D.x, fmaf(-X.x, D.y, ci[ct]));
                    }
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    qr[ct] += cr[ct];
                    qi[ct] += ci[ct];
                }
            }
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
                for (int r = 0; r < K; ++r) G[ct][r] = fmaf(V[r], R::imag(r) ? qi[ct] : qr[ct], G[ct][r]);
            }
        }
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
        for (int r = 0; r < K; ++r)
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) G[ct][r] += __shfl_xor(G[ct][r], off, 64);
        if (lane == 0 && c0 + ct < C) {
            float* out = partial + ((int64_t)(c0 + ct) * chunks + kFoldGradChunks + h * kFoldGradSegments + seg) * K;
#pragma unroll
            for (int k = 0; k < K; ++k) out[k] = R::basis(G[ct], k);
        }
    }
}

// What a ring's direct sums need: its entries (CSR over (ring, phase); none:
// no direct sums), the cells' basis functions, x and W.
template <typename T>
struct RingSums {
    const int32_t* ptr;
    const RingEntry* ent;
    const int8_t* cmap;
    const T *x, *w;
    int64_t n_in;
    int Ci, Co, K, dw_c, P, stride, nlon_i;
    bool w_trans;
};

// Ring h of batch item b and output channel co by direct sums, in 64 bits; all
// threads.  Only for data with infinities or NaN: nothing is staged.
template <typename T>
__device__ void ring_direct(const RingSums<T>& R, int h, int b, int co, T* __restrict__ yr, int nlon_o) {
    for (int o = threadIdx.x; o < nlon_o; o += blockDim.x) {
        const int q = o / R.P, r = o - q * R.P;
        const int e0 = R.ptr[h * R.P + r], e1 = R.ptr[h * R.P + r + 1];
        double acc = 0.0;
        for (int ci = 0; ci < R.Ci; ++ci) {
            const T* xr = R.x + ((int64_t)b * R.Ci + ci) * R.n_in;
            const T* w = R.w + (int64_t)R.K * (R.dw_c > 0 ? b % R.dw_c : R.w_trans ? ci * R.Co + co : co * R.Ci + ci);
            for (int e = e0; e < e1; ++e) {
                const RingEntry E = R.ent[e];
                float f = 0.0f;
                for (int m = 0; m < 4; ++m) {
                    const int k = R.cmap[4 * E.cell + m];
                    if (k >= 0) f = fmaf(load_val(w, k), E.v[m], f);
                }
                acc += (double)f * load_val(xr, E.row + (R.stride * q + E.d) % R.nlon_i);
            }
        }
        store_val(yr, o, (float)acc);
    }
}

// y[b][co][ring][:] = inverse real DFT of Yhat[h][b][co][:].  grid: (n_rings, B * Co)
template <typename T>
__global__ __launch_bounds__(kFftBlock) void k_irfft_rings(const int32_t* __restrict__ rings,
                                                          const float2* __restrict__ yh,
                                                          const float2* __restrict__ tw, T* __restrict__ y,
                                                          int B, int Co, int nlat_o, int M, int tws, RingSums<T> R) {
    extern __shared__ float2 sm[];
    float2* a = sm;
    float2* bb = sm + M;
    float2* tlo = sm + 2 * M;
    float2* thi = tlo + kTwLo;
    const int h = blockIdx.x;
    const int b = blockIdx.y / Co, co = blockIdx.y - (blockIdx.y / Co) * Co;
    const float2* Y = yh + (((int64_t)h * B + b) * Co + co) * (M + 1);
    load_twiddles(tw, thi, tlo, M, tws);
    bool fine = true;
    for (int m0 = threadIdx.x; m0 < M; m0 += kFftBatch * kFftBlock) {
        float2 xm[kFftBatch], xc[kFftBatch], twm[kFftBatch];
#pragma unroll
        for (int u = 0; u < kFftBatch; ++u) {
            const int m = m0 + u * kFftBlock;
            if (m < M) {
                xm[u] = Y[m];
                xc[u] = conjf2(Y[M - m]);
                twm[u] = tw[m * tws];
            }
        }
#pragma unroll
        for (int u = 0; u < kFftBatch; ++u) {
            const int m = m0 + u * kFftBlock;
            if (m < M) {
                const float2 e = cadd(xm[u], xc[u]);
                const float2 o = cmul(csub(xm[u], xc[u]), conjf2(twm[u]));
                fine &= fabsf(e.x) + fabsf(e.y) + fabsf(o.x) + fabsf(o.y) < INFINITY;
                a[m] = make_float2(e.x - o.y, e.y + o.x);  // e + i o
            }
        }
    }
    const int N = 2 * M;
    const int64_t base = (((int64_t)b * Co + co) * nlat_o + rings[h]) * N;
    if (R.ptr) {
        if (__syncthreads_or(!fine)) return ring_direct(R, h, b, co, y + base, N);
    } else {
        __syncthreads();
    }
    const float2* z = fft_lds(a, bb, M, thi, tlo, true);
    for (int j = threadIdx.x; j < M; j += blockDim.x) {
        const float2 v = z[j];
        store_val(y, base + 2 * j, v.x);
        store_val(y, base + 2 * j + 1, v.y);
    }
}

size_t fft_lds_bytes(int M) { return sizeof(float2) * (2 * (size_t)M + kTwLo + tw_hi_len(M)); }  // two FFT buffers, twiddles

template <typename T>
hipError_t spectral_rfft(const ExecArgs& a, float2* xh) {
    const SpectralDev& S = a.op->spectral;
    const int tk = timing_begin("spectral_rfft", a.stream);
    hipLaunchKernelGGL((k_rfft_rings<T>), dim3(S.n_slots, a.B * a.Ci), dim3(kFftBlock), fft_lds_bytes(S.Mi), a.stream,
                       S.slot_ring, (const T*)a.x, (const float2*)S.tw, xh, a.B, a.Ci, a.op->g.nlat_i, S.Mi,
                       S.M / S.Mi, 1.0f);
    timing_end(tk, a.stream);
    return hipGetLastError();
}

template <typename T>
hipError_t spectral_irfft(const ExecArgs& a, const float2* yh, bool z) {
    const SpectralDev& S = a.op->spectral;
    const OpGeom& g = a.op->g;
    // The planes of Z (no W) have none: what reads them sums over a ring anyway.
    const RingSums<T> R{z ? nullptr : S.ent_ptr, S.ents, a.op->cmap_dev, (const T*)a.x, (const T*)a.w,
                        (int64_t)g.nlat_i * g.nlon_i, a.Ci, a.Co, basis_size(a.op->basis), a.dw_c, g.P, g.stride,
                        g.nlon_i, a.w_trans};
    const int tk = timing_begin("spectral_irfft", a.stream);
    hipLaunchKernelGGL((k_irfft_rings<T>), dim3(S.n_rings, a.B * a.Co), dim3(kFftBlock), fft_lds_bytes(S.Mo), a.stream,
                       S.rings, yh, (const float2*)S.tw, (T*)a.y, a.B, a.Co, g.nlat_o, S.Mo, S.M / S.Mo, R);
    timing_end(tk, a.stream);
    return hipGetLastError();
}

SpecGeom spec_geom(const ExecArgs& a) {
    const SpectralDev& S = a.op->spectral;
    return SpecGeom{S.M, S.Mi, S.Mo, S.Mi / S.Mo > 1 ? S.Mi / S.Mo : 1};
}
bool same_rings(const SpecGeom& G) { return G.Mi == G.Mo; }

template <typename T, int COT, int BLK = kFftBlock>
hipError_t spectral_products(const ExecArgs& a, const float2* xh, float2* yh) {
    const SpectralDev& S = a.op->spectral;
    const SpecGeom G = spec_geom(a);
    const int n_cot = (a.Co + COT - 1) / COT;
    const dim3 grid((G.Mo + 1 + BLK - 1) / BLK, S.n_rings, a.B * n_cot);
    if (same_rings(G))
        hipLaunchKernelGGL((k_spectral<T, COT, BLK, false>), grid, dim3(BLK), 0, a.stream, S.pair_ptr, S.pair_slot,
                           S.pair_tab, S.vs, xh, (const T*)a.w, yh, a.B, a.Ci, a.Co, G, n_cot, a.w_trans);
    else
        hipLaunchKernelGGL((k_spectral<T, COT, BLK, true>), grid, dim3(BLK), 0, a.stream, S.pair_ptr, S.pair_slot,
                           S.pair_tab, S.vs, xh, (const T*)a.w, yh, a.B, a.Ci, a.Co, G, n_cot, a.w_trans);
    return hipGetLastError();
}

hipError_t spectral_z_products(const ExecArgs& a, const float2* xh, float2* yh) {
    // a.Co = a.Ci * 9: the planes of every input channel, no W.
    const SpectralDev& S = a.op->spectral;
    const SpecGeom G = spec_geom(a);
    const int n_cg = (a.Ci + 3) / 4;
    const dim3 grid((G.Mo + 1 + kFftBlock - 1) / kFftBlock, S.n_rings, a.B * n_cg);
    if (same_rings(G))
        hipLaunchKernelGGL(k_spectral_z<false>, grid, dim3(kFftBlock), 0, a.stream, S.pair_ptr, S.pair_slot,
                           S.pair_tab, S.vs, xh, yh, a.B, a.Ci, G, n_cg);
    else
        hipLaunchKernelGGL(k_spectral_z<true>, grid, dim3(kFftBlock), 0, a.stream, S.pair_ptr, S.pair_slot,
                           S.pair_tab, S.vs, xh, yh, a.B, a.Ci, G, n_cg);
    return hipGetLastError();
}

template <typename T, int BASIS, int CT, int BT>
hipError_t spectral_fold(const ExecArgs& a, const float2* xh, float2* yh) {
    const SpectralDev& S = a.op->spectral;
    const SpecGeom G = spec_geom(a);
    const int C = a.dw_c > 0 ? a.dw_c : 1, B = a.B / C;
    const int64_t blocks = (int64_t)((G.Mo + 64) / 64) * S.n_rings * ((C + CT - 1) / CT) * ((B + BT - 1) / BT);
    if (same_rings(G))
        hipLaunchKernelGGL((k_spectral_fold<T, BASIS, CT, BT, false>), dim3((unsigned)blocks), dim3(64), 0, a.stream,
                           S.pair_ptr, S.pair_slot, S.pair_tab, S.vs, xh, (const T*)a.w, yh, B, C, G, S.n_rings);
    else
        hipLaunchKernelGGL((k_spectral_fold<T, BASIS, CT, BT, true>), dim3((unsigned)blocks), dim3(64), 0, a.stream,
                           S.pair_ptr, S.pair_slot, S.pair_tab, S.vs, xh, (const T*)a.w, yh, B, C, G, S.n_rings);
    return hipGetLastError();
}

template <typename T, int BASIS>
hipError_t spectral_fold_sizes(const ExecArgs& a, const float2* xh, float2* yh) {
    // Eight (channel, batch item) pairs per wave, up to four of them a batch.
    const int C = a.dw_c > 0 ? a.dw_c : 1, B = a.B / C;
    if (a.B == 1) return spectral_fold<T, BASIS, 1, 1>(a, xh, yh);
    if (B == 1) return spectral_fold<T, BASIS, 8, 1>(a, xh, yh);
    if (B == 2) return spectral_fold<T, BASIS, 4, 2>(a, xh, yh);
    return spectral_fold<T, BASIS, 2, 4>(a, xh, yh);
}

template <typename T>
hipError_t spectral_mac(const ExecArgs& a, const float2* xh, float2* yh, int stages) {
    const int basis = a.op->basis;
    if (basis != DISCO_BASIS_BILINEAR_3X3 || a.dw_c > 0) {
        if (a.Ci != 1 || a.Co != 1) return hipErrorInvalidValue;
        return basis == DISCO_BASIS_AXISYMMETRIC_4  ? spectral_fold_sizes<T, DISCO_BASIS_AXISYMMETRIC_4>(a, xh, yh)
               : basis == DISCO_BASIS_SEPARABLE_4X4 ? spectral_fold_sizes<T, DISCO_BASIS_SEPARABLE_4X4>(a, xh, yh)
                                                    : spectral_fold_sizes<T, DISCO_BASIS_BILINEAR_3X3>(a, xh, yh);
    }
    if (stages & kSpectralZ) return spectral_z_products(a, xh, yh);
    if (a.Co <= 4) return spectral_products<T, 4>(a, xh, yh);
    if (a.Co <= 8) return spectral_products<T, 8>(a, xh, yh);
    // More output channels: one tile of up to 32 (the per-pair sums done
    // once), the frequencies in workgroups of 64 so that they still fill
    // the chip (512 x 1024, 32 -> 32 channels: tiles of 32 in workgroups of
    // 256 leave 240 of them; tiles of 8 redo the per-pair sums).
    if (a.Co <= 32) return spectral_products<T, 32, 64>(a, xh, yh);
    return spectral_products<T, 8>(a, xh, yh);
}

template <typename T>
hipError_t spectral_dispatch(const ExecArgs& a, float* ws, int stages) {
    float2* xh = (float2*)ws;
    float2* yh = spectral_yhat(a, ws);
    hipError_t e = stages & 1 ? spectral_rfft<T>(a, xh) : hipSuccess;
    if (e == hipSuccess && (stages & 2)) {
        const int tk = timing_begin("spectral_mac", a.stream);
        e = spectral_mac<T>(a, xh, yh, stages);
        timing_end(tk, a.stream);
    }
    if (e == hipSuccess && (stages & 4)) e = spectral_irfft<T>(a, yh, (stages & kSpectralZ) != 0);
    return e;
}

}  // namespace

size_t workspace_bytes_spectral(const ExecArgs& a) {
    const SpectralDev& S = a.op->spectral;
    if (S.n_rings == 0) return 0;
    return sizeof(float2) * (size_t)a.B * ((size_t)S.n_slots * a.Ci * (S.Mi + 1) + (size_t)S.n_rings * a.Co * (S.Mo + 1));
}

float2* spectral_yhat(const ExecArgs& a, float* ws) {
    const SpectralDev& S = a.op->spectral;
    return (float2*)ws + (size_t)S.n_slots * a.B * a.Ci * (S.Mi + 1);
}

size_t spectral_dyhat_bytes(const ExecArgs& a, int C) {
    const SpectralDev& S = a.op->spectral;
    return sizeof(float2) * (size_t)S.n_rings * a.B * C * (S.Mo + 1);
}

hipError_t launch_spectral_dyhat(const ExecArgs& a, const float* dy, int C, float2* dyh) {
    const SpectralDev& S = a.op->spectral;
    if (S.n_rings == 0) return hipSuccess;
    const int tk = timing_begin("spectral_rfft_dy", a.stream);
    hipLaunchKernelGGL((k_rfft_rings<float>), dim3(S.n_rings, a.B * C), dim3(kFftBlock), fft_lds_bytes(S.Mo), a.stream,
                       S.rings, dy, (const float2*)S.tw, dyh, a.B, C, a.op->g.nlat_o, S.Mo, S.M / S.Mo, 2.0f);
    timing_end(tk, a.stream);
    return hipGetLastError();
}

namespace {

template <int BASIS>
void spectral_fold_grad(const ExecArgs& a, const float2* xh, const float2* dyh, float* partial, int chunks) {
    const SpectralDev& S = a.op->spectral;
    const SpecGeom G = spec_geom(a);
    constexpr int CT = 4;
    const int C = a.dw_c > 0 ? a.dw_c : 1, B = a.B / C;
    const dim3 grid((unsigned)((int64_t)kFoldGradSegments * S.n_rings * ((C + CT - 1) / CT)));
    if (same_rings(G))
        hipLaunchKernelGGL((k_spectral_fold_grad<BASIS, CT, false>), grid, dim3(64), 0, a.stream, S.pair_ptr,
                           S.pair_slot, S.pair_tab, S.vs, xh, dyh, partial, B, C, chunks, G, S.n_rings);
    else
        hipLaunchKernelGGL((k_spectral_fold_grad<BASIS, CT, true>), grid, dim3(64), 0, a.stream, S.pair_ptr,
                           S.pair_slot, S.pair_tab, S.vs, xh, dyh, partial, B, C, chunks, G, S.n_rings);
}

template <typename T>
hipError_t spectral_fold_grad_all(const ExecArgs& a, float2* xh, float2* dyh, float* partial, int chunks) {
    const SpectralDev& S = a.op->spectral;
    hipError_t e = spectral_rfft<T>(a, xh);
    if (e != hipSuccess) return e;
    int tk = timing_begin("spectral_rfft_dy", a.stream);
    hipLaunchKernelGGL((k_rfft_rings<T>), dim3(S.n_rings, a.B), dim3(kFftBlock), fft_lds_bytes(S.Mo), a.stream, S.rings,
                       (const T*)a.dy, (const float2*)S.tw, dyh, a.B, 1, a.op->g.nlat_o, S.Mo, S.M / S.Mo, 2.0f);
    timing_end(tk, a.stream);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    tk = timing_begin("spectral_grad", a.stream);
    switch (a.op->basis) {
        case DISCO_BASIS_AXISYMMETRIC_4:
            spectral_fold_grad<DISCO_BASIS_AXISYMMETRIC_4>(a, xh, dyh, partial, chunks);
            break;
        case DISCO_BASIS_SEPARABLE_4X4:
            spectral_fold_grad<DISCO_BASIS_SEPARABLE_4X4>(a, xh, dyh, partial, chunks);
            break;
        default: spectral_fold_grad<DISCO_BASIS_BILINEAR_3X3>(a, xh, dyh, partial, chunks);
    }
    timing_end(tk, a.stream);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_spectral_fold_grad(const ExecArgs& a, float2* xh, float2* dyh, float* partial, int chunks) {
    return a.dtype == 1 ? spectral_fold_grad_all<uint16_t>(a, xh, dyh, partial, chunks)
                        : spectral_fold_grad_all<float>(a, xh, dyh, partial, chunks);
}

hipError_t launch_spectral(const ExecArgs& a, float* ws, int stages) {
    if (a.op->spectral.n_rings == 0) return hipSuccess;
    return a.dtype == 1 ? spectral_dispatch<uint16_t>(a, ws, stages) : spectral_dispatch<float>(a, ws, stages);
}

}  // namespace disco
