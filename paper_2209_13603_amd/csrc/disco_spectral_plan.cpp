// disco_spectral_plan.cpp -- host construction of the spectral data of heavy rings.
//
// The sum of one output ring over one input ring is, along longitude, a
// cyclic correlation with the ring's stored pattern (Sec. 4.2: the pattern is
// reused at every output longitude by a shift).  On the finer of the two
// longitude grids (Nf = max(nlon_i, nlon_o), both powers of two) an entry of
// phase r at offset d sits at lag n = P d - r (P = nlon_o / nlon_i phases of
// an upsampling op, 1 otherwise), the lags of all phases together form the
// Nf-periodic sequences v_k[n], and
//   same grid (P = stride = 1):  Yhat[m] = Xhat[m] conj(Vhat_k[m]);
//   upsampling (P > 1):  the input's spectrum repeats,
//     Yhat[m] = Xhat[m mod nlon_i] conj(Vhat_k[m]), m < nlon_o;
//   downsampling (stride s > 1):  every s-th output of the full-resolution
//     correlation is kept, so its spectrum folds,
//     Yhat[m] = sum_{j < s} Xhat[m + j nlon_o] conj(Vhat_k[m + j nlon_o]).
// This file computes Vhat_k in fp64 with its own radix-2 FFT, checks the
// east-west mirror symmetry of the lags that lets K floats per frequency
// describe all K basis functions (9, 4 or 16), and rounds to fp32.
//
// Rows of a table per frequency: 3x3 basis, for a = 0..2: Re Vhat_{3a},
// Im Vhat_{3a}, Vhat_{3a+1} (real), with Vhat_{3a+2} = conj(Vhat_{3a});
// axisymmetric: Vhat_0..3 (real); separable, for a = 0..3: Vhat_{4a} (real),
// Re Vhat_{4a+1}, Im Vhat_{4a+1}, Vhat_{4a+2} (real), with Vhat_{4a+3} =
// conj(Vhat_{4a+1}).
//
// The grids are symmetric about the equator: reflecting both rings of a pair
// (t_o -> nlat_o - 1 - t_o, t_i -> nlat_i - 1 - t_i) flips the sign of the
// local coordinate along the meridian and keeps the one along the parallel and
// the longitude offsets, so the reflected pair's psi rows are this pair's with
// the radial index a of psi_{3a+b} replaced by 2 - a (3x3) or the directions
// b = 0 (south) and 2 (north) exchanged (separable).  A pair whose stored
// entries show exactly that relation to an earlier pair reads that pair's
// table with those rows exchanged instead of holding its own.
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdlib>
#include <system_error>
#include <thread>

#include "disco.h"
#include "disco_internal.h"

namespace disco {

namespace {

using cd = std::complex<double>;

bool is_pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }

// In-place iterative radix-2 DFT, X[m] = sum_n x[n] exp(-2 pi i m n / N);
// w[t] = exp(-2 pi i t / N) for t < N / 2.
void fft(std::vector<cd>& a, const std::vector<cd>& w) {
    const size_t n = a.size();
    for (size_t i = 1, j = 0; i < n; ++i) {
        size_t bit = n >> 1;
        for (; j & bit; bit >>= 1) j ^= bit;
        j ^= bit;
        if (i < j) std::swap(a[i], a[j]);
    }
    for (size_t len = 2; len <= n; len <<= 1) {
        const size_t step = n / len;
        for (size_t i = 0; i < n; i += len)
            for (size_t k = 0; k < len / 2; ++k) {
                const cd u = a[i + k], v = a[i + k + len / 2] * w[k * step];
                a[i + k] = u + v;
                a[i + k + len / 2] = u - v;
            }
    }
}

}  // namespace

// A ring is wide when its outputs read min_entries inputs on average, as
// counted on the output's own spacing: a downsampling op of stride s reads
// s^2 times the inputs per output, and its products s times the pairs and s
// aliases, so the line scales with both.
std::vector<uint8_t> wide_patterns(const HostOp& op, int min_entries) {
    const OpGeom& g = op.g;
    std::vector<uint8_t> wide((size_t)g.n_patterns(), 0);
    for (int to = 0; to < g.nlat_o; ++to) {
        const int64_t n = (int64_t)op.pat_ptr[(size_t)(to + 1) * g.P] - op.pat_ptr[(size_t)to * g.P];
        if (n >= (int64_t)min_entries * g.P * g.stride * g.stride)
            for (int r = 0; r < g.P; ++r) wide[(size_t)to * g.P + r] = 1;
    }
    return wide;
}

int build_spectral(const HostOp& op, int min_entries, SpectralHost* sp, std::vector<uint8_t>* heavy,
                   std::string* err, bool phases, int64_t max_table_bytes) {
    const OpGeom& g = op.g;
    heavy->assign((size_t)g.n_patterns(), 0);
    *sp = SpectralHost{};
    const int Ni = g.nlon_i, No = g.nlon_o, N = std::max(Ni, No);
    // N <= 8192: the device FFTs keep two M-point buffers and two short
    // twiddle tables in LDS (about 16 M bytes, 65 KB at M = 4096).
    if ((g.P != 1 && !phases) || !is_pow2(Ni) || !is_pow2(No) || std::min(Ni, No) < 64 || N > 8192) return DISCO_OK;
    const int M = N / 2;
    const int K = basis_size(op.basis);
    const bool sep = op.basis == DISCO_BASIS_SEPARABLE_4X4, grid3 = op.basis == DISCO_BASIS_BILINEAR_3X3;

    const std::vector<uint8_t> wide = wide_patterns(op, min_entries);
    std::vector<int32_t> rings;
    for (int to = 0; to < g.nlat_o; ++to)
        if (wide[(size_t)to * g.P]) rings.push_back(to);
    if (rings.empty()) return DISCO_OK;

    // The entries of every heavy ring by input ring: lag and entry index.
    struct Lag { int32_t n, e; };
    struct Pair { int32_t to, ti, l0, l1; };
    std::vector<Lag> lags;
    std::vector<Pair> pe;
    for (int32_t to : rings) {
        std::vector<std::pair<int32_t, Lag>> byring;
        for (int r = 0; r < g.P; ++r)
            for (int32_t e = op.pat_ptr[(size_t)to * g.P + r]; e < op.pat_ptr[(size_t)to * g.P + r + 1]; ++e)
                byring.push_back({op.t_in[(size_t)e], Lag{((g.P * op.d[(size_t)e] - r) % N + N) % N, e}});
        std::stable_sort(byring.begin(), byring.end(),
                         [](const auto& a, const auto& b) { return a.first < b.first; });
        for (size_t i = 0; i < byring.size(); ++i) {
            if (i == 0 || byring[i].first != byring[i - 1].first)
                pe.push_back({to, byring[i].first, (int32_t)lags.size(), (int32_t)lags.size()});
            lags.push_back(byring[i].second);
            pe.back().l1 = (int32_t)lags.size();
        }
    }
    // All K basis values of an entry.
    const CellMap cm = cell_map(op.basis);
    auto basis_values = [&](int32_t e, double (&v)[kSeparableBasis]) {
        const double* s = &op.val64[(size_t)e * kBasis];
        for (int k = 0; k < kSeparableBasis; ++k) v[k] = 0.0;
        if (sep) {
            for (int m = 0; m < 4; ++m)
                if (const int k = cm.k[op.cell[(size_t)e]][m]; k >= 0) v[k] = s[m];
        } else {
            for (int k = 0; k < K; ++k) v[k] = s[k];
        }
    };
    // Basis function k of the point mirrored east-west, and about the equator.
    auto east_west = [&](int k) { return grid3 ? k / 3 * 3 + 2 - k % 3 : sep ? (k & ~3) + ((4 - (k & 3)) & 3) : k; };
    auto equator = [&](int k) { return grid3 ? 3 * (2 - k / 3) + k % 3 : sep ? (k & ~3) + ((6 - (k & 3)) & 3) : k; };

    // Mirror symmetry: the entry at lag n must match the entry at -n.  If the
    // stored pattern does not have it (it always should), the spectral path is
    // not used for this op.
    std::vector<int32_t> at((size_t)N, -1);
    std::vector<double> vmax(pe.size(), 0.0);
    double a[kSeparableBasis], b[kSeparableBasis];
    for (size_t p = 0; p < pe.size(); ++p)
        for (int32_t l = pe[p].l0; l < pe[p].l1; ++l) {
            basis_values(lags[(size_t)l].e, a);
            for (int k = 0; k < K; ++k) vmax[p] = std::max(vmax[p], std::fabs(a[k]));
        }
    for (size_t p = 0; p < pe.size(); ++p) {
        double ring_max = 0.0;  // over the output ring's pairs
        for (size_t q = p; q < pe.size() && pe[q].to == pe[p].to; ++q) ring_max = std::max(ring_max, vmax[q]);
        for (size_t q = p; q-- > 0 && pe[q].to == pe[p].to;) ring_max = std::max(ring_max, vmax[q]);
        for (int32_t l = pe[p].l0; l < pe[p].l1; ++l) at[(size_t)lags[(size_t)l].n] = lags[(size_t)l].e;
        bool same = true;
        for (int32_t l = pe[p].l0; l < pe[p].l1 && same; ++l) {
            basis_values(lags[(size_t)l].e, a);
            const int32_t f = at[(size_t)((N - lags[(size_t)l].n) % N)];
            if (f >= 0) basis_values(f, b);
            for (int k = 0; k < K; ++k)
                same &= std::fabs(a[k] - (f < 0 ? 0.0 : b[east_west(k)])) <= 1e-12 * ring_max;
        }
        for (int32_t l = pe[p].l0; l < pe[p].l1; ++l) at[(size_t)lags[(size_t)l].n] = -1;
        if (!same) return DISCO_OK;
    }

    // Input-ring slots and pairs.
    std::vector<int32_t> slot_of(g.nlat_i, -1);
    sp->Ni = Ni;
    sp->No = No;
    sp->N = N;
    sp->M = M;
    sp->nv = K;
    sp->rings = rings;
    sp->pair_ptr.assign(1, 0);
    for (size_t p = 0; p < pe.size(); ++p) {
        int32_t& sl = slot_of[(size_t)pe[p].ti];
        if (sl < 0) {
            sl = (int32_t)sp->slot_ring.size();
            sp->slot_ring.push_back(pe[p].ti);
        }
        sp->pair_slot.push_back(sl);
        if (p + 1 == pe.size() || pe[p + 1].to != pe[p].to) sp->pair_ptr.push_back((int32_t)p + 1);
    }
    // The table each pair reads: its own, or (bit 31) the equator mirror's
    // with its rows exchanged.
    const size_t n_pairs = pe.size();
    std::vector<int32_t> ring_first((size_t)g.nlat_o, -1);  // first pair of each spectral ring
    for (size_t p = n_pairs; p-- > 0;) ring_first[(size_t)pe[p].to] = (int32_t)p;
    sp->pair_tab.assign(n_pairs, -1);
    std::vector<int32_t> owners;  // pair whose entries make each table
    auto mirrors = [&](size_t p, size_t q) {
        const Pair &P = pe[p], &Q = pe[q];
        if (P.l1 - P.l0 != Q.l1 - Q.l0) return false;
        const double tol = 1e-12 * std::max(vmax[p], vmax[q]);
        for (int32_t l = Q.l0; l < Q.l1; ++l) at[(size_t)lags[(size_t)l].n] = lags[(size_t)l].e;
        bool same = true;
        for (int32_t l = P.l0; l < P.l1 && same; ++l) {
            const int32_t f = at[(size_t)lags[(size_t)l].n];
            if (f < 0) { same = false; break; }
            basis_values(lags[(size_t)l].e, a);
            basis_values(f, b);
            for (int k = 0; k < K; ++k) same &= std::fabs(a[k] - b[equator(k)]) <= tol;
        }
        for (int32_t l = Q.l0; l < Q.l1; ++l) at[(size_t)lags[(size_t)l].n] = -1;
        return same;
    };
    for (size_t p = 0; p < n_pairs; ++p) {
        const Pair& P = pe[p];
        // The mirror pair, if it is an earlier one with a table of its own.
        int32_t mq = -1;
        const int32_t mto = g.nlat_o - 1 - P.to, mti = g.nlat_i - 1 - P.ti;
        for (int32_t q = ring_first[(size_t)mto]; q >= 0 && q < (int32_t)p && pe[(size_t)q].to == mto; ++q)
            if (pe[(size_t)q].ti == mti) mq = q;
        if (mq >= 0 && sp->pair_tab[(size_t)mq] >= 0 && mirrors(p, (size_t)mq)) {
            sp->pair_tab[p] = sp->pair_tab[(size_t)mq] | (int32_t)0x80000000u;
        } else {
            sp->pair_tab[p] = (int32_t)owners.size();
            owners.push_back((int32_t)p);
        }
    }
    if (max_table_bytes > 0 && (int64_t)(owners.size() * (size_t)K * (size_t)(M + 1) * sizeof(float)) > max_table_bytes) {
        *sp = SpectralHost{};
        return DISCO_OK;
    }
    *heavy = wide;
    sp->ent_ptr.assign(1, 0);
    for (int32_t to : rings)
        for (int r = 0; r < g.P; ++r) {
            for (int32_t e = op.pat_ptr[(size_t)to * g.P + r]; e < op.pat_ptr[(size_t)to * g.P + r + 1]; ++e) {
                RingEntry E{};
                int cell = 0;
                if (!entry_cell_values(op, e, &cell, E.v)) {
                    if (err) *err = "internal: basis value outside its hat cell";
                    return DISCO_ERR_DEVICE;
                }
                E.row = op.t_in[(size_t)e] * Ni;
                E.d = op.d[(size_t)e];
                E.cell = cell;
                sp->ents.push_back(E);
            }
            sp->ent_ptr.push_back((int32_t)sp->ents.size());
        }
    // Vhat per table, scaled by 1/N (the inverse transform on the device is
    // unnormalised).  Two real sequences per complex FFT, the tables shared
    // out over a few host threads.
    sp->n_tables = (int32_t)owners.size();
    sp->vs.assign(owners.size() * (size_t)K * (size_t)(M + 1), 0.0f);
    std::vector<cd> wtab((size_t)M);
    for (int t = 0; t < M; ++t) {
        const double ang = -2.0 * 3.14159265358979323846 * (double)t / (double)N;
        wtab[(size_t)t] = cd(std::cos(ang), std::sin(ang));
    }
    auto make_tables = [&](std::vector<cd>& buf, size_t first, size_t step) {
        double v[kSeparableBasis];
        for (size_t tb = first; tb < owners.size(); tb += step) {
            const Pair& P = pe[(size_t)owners[tb]];
            float* dst = &sp->vs[tb * (size_t)K * (size_t)(M + 1)];
            // The DFTs of basis functions k0 and k1 as spectra of the real and
            // the imaginary part of one sequence; out(m, V_k0, V_k1).
            auto two = [&](int k0, int k1, auto out) {
                std::fill(buf.begin(), buf.end(), cd(0.0, 0.0));
                for (int32_t l = P.l0; l < P.l1; ++l) {
                    basis_values(lags[(size_t)l].e, v);
                    buf[(size_t)lags[(size_t)l].n] += cd(v[k0], v[k1]);
                }
                fft(buf, wtab);
                for (int m = 0; m <= M; ++m) {
                    const cd zm = buf[(size_t)m], zc = std::conj(buf[(size_t)((N - m) % N)]);
                    out(m, 0.5 * (zm + zc), cd(0.0, -0.5) * (zm - zc));
                }
            };
            auto put = [&](int row, int m, double x) { dst[(size_t)row * (M + 1) + m] = (float)(x / N); };
            if (grid3) {
                for (int ia = 0; ia < 3; ++ia)
                    two(3 * ia, 3 * ia + 1, [&](int m, cd v0, cd v1) {
                        put(3 * ia, m, v0.real());
                        put(3 * ia + 1, m, v0.imag());
                        put(3 * ia + 2, m, v1.real());
                    });
            } else if (sep) {
                for (int ia = 0; ia < 4; ++ia) {
                    two(4 * ia, 4 * ia + 2, [&](int m, cd v0, cd v2) {
                        put(4 * ia, m, v0.real());
                        put(4 * ia + 3, m, v2.real());
                    });
                    two(4 * ia + 1, 4 * ia + 1, [&](int m, cd v1, cd) {
                        put(4 * ia + 1, m, v1.real());
                        put(4 * ia + 2, m, v1.imag());
                    });
                }
            } else {
                for (int k = 0; k < 4; k += 2)
                    two(k, k + 1, [&](int m, cd v0, cd v1) {
                        put(k, m, v0.real());
                        put(k + 1, m, v1.real());
                    });
            }
        }
    };
    // About one thread per 4 ms of transforms, at most eight; buffers are
    // allocated here, so that nothing can throw inside a thread.
    const size_t want = std::min<size_t>(8, owners.size() * (size_t)K * (size_t)N / 500000);
    const size_t n_threads = std::max<size_t>(1, std::min<size_t>(want, std::thread::hardware_concurrency()));
    std::vector<std::vector<cd>> bufs(n_threads, std::vector<cd>((size_t)N));
    std::vector<std::thread> pool;
    pool.reserve(n_threads);
    try {
        for (size_t t = 1; t < n_threads; ++t)
            pool.emplace_back([&, t] { make_tables(bufs[t], t, n_threads); });
    } catch (const std::system_error&) {
        // Fewer threads than asked for: their shares are done below.
    }
    make_tables(bufs[0], 0, n_threads);
    for (size_t t = pool.size() + 1; t < n_threads; ++t) make_tables(bufs[t], t, n_threads);
    for (std::thread& t : pool) t.join();
    sp->tw.resize((size_t)N);
    for (int t = 0; t < M; ++t) {
        sp->tw[(size_t)2 * t] = (float)wtab[(size_t)t].real();
        sp->tw[(size_t)2 * t + 1] = (float)wtab[(size_t)t].imag();
    }
    return DISCO_OK;
}

}  // namespace disco
