// Device-resident Lanczos ground state for short chains (Sec. ed:sec:statics, by the Lanczos recurrence
// of Sec. ed:sec:krylov): with full reorthogonalisation and no restart, the whole recurrence runs in
// one cooperative launch instead of a dozen launches and a host round trip per product.
//
// G workgroups of kLT threads own consecutive slices of the state, one amplitude per thread. A
// product w = H v_j takes every term per amplitude (partners of the same slice from LDS), then
// classical Gram-Schmidt runs twice against v_0..v_j: each workgroup writes its partial dot
// products, and after a grid barrier every workgroup sums all of them in the same order (so all
// hold identical coefficients). beta_j = |w| comes the same way. One more workgroup tests
// convergence on T_m beside the others, after every kLCheck products (the lowest eigenvalue by
// multisection on Sturm counts, the last component of its eigenvector by inverse iteration).
// Every barrier and every wait is a bounded poll: a workgroup that waits too long flags an error and
// every workgroup leaves, so the launch always ends.
//
// What bounds it: latency, 37 us a product at 14 sites and a basis of 88 (88 us when every barrier
// flushed and dropped the caches, a fourth barrier and the tests stood in the products' way and every
// lane read the operator tables): 4 us in each pass's dot products, 5 us in each subtraction, 2.5 us in
// each sum over the workgroups, 2.7 us at each of three barriers, 2 us in the product.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <vector>

#include "ed_vec.h"
#include "hpsi_device.h"
#include "krylov_core.h"
#include "wave_ops.h"

namespace ed {
namespace {

constexpr int kLT = 256;                    // threads per workgroup
constexpr int kLCheck = 8;                  // products between convergence tests
constexpr unsigned kSpinLimit = 1u << 26;   // barrier polls before giving up
constexpr int kDevMaxVec = 512;             // basis vectors the kernel's LDS coefficients hold

struct DevLzArgs {
    int L;
    int64_t D;
    double2* V;     // basis slots 0..nmax (slot 0 holds the normalised start vector)
    int nmax;       // at most nmax products
    double2* p1;    // partial dots of the first pass [G][pld]
    double2* p2;    // partial dots of the second pass [G][pld]
    int pld;
    double* pn;     // partial squared norms [G]
    double* alpha;  // [nmax]
    double* beta;   // [nmax]
    unsigned* bar;  // barrier counter, zero at launch
    int* ctl;       // [0] error flag, [1] products at the first test that passed (0: none), [2] products
                    // done, [3] products at a breakdown (0: none)
    int* stop;      // set by workgroup 0 once it has seen ctl[1]
    double tol;
};

// What one workgroup writes and another reads within the launch (the partial sums, the new basis
// vector, the recurrence's scalars) goes through ld_shared and st_shared. The barriers then need no
// cache write-back or invalidation: a workgroup's own slices of the basis, which every sweep reads, stay
// in its XCD's L2. With plain accesses and a fence at each barrier a group of 16 vectors took 3.8 us to
// sum and a barrier 6 to 9 us.

// Grid barrier number gen + 1 of the G workgroups that own slices: the counter reaches (gen + 1) G
// once every one has arrived. It orders ld_shared and st_shared accesses and nothing else. Returns false
// (and flags the error) when the wait exceeds the limit or another workgroup failed.
__device__ bool grid_sync(const DevLzArgs& a, int G, unsigned& gen, int* bad) {
    drain();
    __syncthreads();
    if (threadIdx.x == 0) {
        *bad = 0;
        __hip_atomic_fetch_add(a.bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned target = (gen + 1) * unsigned(G);
        unsigned spins = 0;
        while (__hip_atomic_load(a.bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (++spins > kSpinLimit || (spins % 64 == 0 && ld_shared(a.ctl) != 0)) {
                st_shared(a.ctl, 1);
                *bad = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        drain();
    }
    ++gen;
    __syncthreads();
    return *bad == 0;
}

// part[i] (i < n) = sum over the workgroup's amplitudes of conj(V_i[x]) w, w from LDS. Wave wv takes
// the vectors i = wv, wv + 4, ..., eight at a time with four amplitudes a lane, so that a sum ends in
// one wave and its lane exchanges are shared by four amplitudes: the eight sums fold to one value a lane
// (each exchange keeps half of them), then over the remaining eight lanes.
__device__ void block_dots(const double2* V, int64_t D, int n, int64_t x0, const double2* w, double2* part) {
    constexpr int K = kLT / 64;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double2 wk[K];
#pragma unroll
    for (int k = 0; k < K; ++k) wk[k] = w[lane + 64 * k];
    for (int i0 = wv; i0 < n; i0 += 8 * K) {
        double2 r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            r[q] = make_double2(0.0, 0.0);
            const double2* v = V + int64_t(min(i0 + K * q, n - 1)) * D + x0;  // past n: a sum nobody takes
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const unsigned y = unsigned(lane + 64 * k);
                const double2 z = x0 + y < D ? v[y] : make_double2(0.0, 0.0);
                r[q].x = fma(z.x, wk[k].x, fma(z.y, wk[k].y, r[q].x));
                r[q].y = fma(z.x, wk[k].y, fma(-z.y, wk[k].x, r[q].y));
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = make_double2(pair_sum32(r[q].x, r[q + 4].x), pair_sum32(r[q].y, r[q + 4].y));
#pragma unroll
        for (int q = 0; q < 2; ++q) r[q] = make_double2(pair_sum16(r[q].x, r[q + 2].x), pair_sum16(r[q].y, r[q + 2].y));
        const bool up = (lane & 8) != 0;
        double2 s = up ? r[1] : r[0];
        const double2 o = up ? r[0] : r[1];
        s.x += dpp<kDppRor8>(o.x);
        s.y += dpp<kDppRor8>(o.y);
        s.x += dpp<kDppHalfMirror>(s.x);
        s.y += dpp<kDppHalfMirror>(s.y);
        s.x += dpp<kDppXor1>(s.x);
        s.y += dpp<kDppXor1>(s.y);
        s.x += dpp<kDppXor2>(s.x);
        s.y += dpp<kDppXor2>(s.y);
        // lane bits 5, 4, 3 are the vector's bits 2, 1, 0
        const int i = i0 + K * (lane >> 3);
        if ((lane & 7) == 0 && i < n) st_shared(part + i, s);
    }
}

// coef[i] (LDS, i < n) = sum over the G workgroups of part[b][i], the same sum on every workgroup:
// four lanes per coefficient take the rows b = k, k + 4, ... (their loads issued in groups of 16),
// and the four sums are added in one fixed tree.
__device__ void sum_partials(const double2* part, int pld, int G, int n, double2* coef) {
    const int t = threadIdx.x, k = t & 3;
    for (int i0 = 0; i0 < n; i0 += kLT / 4) {
        const int i = i0 + (t >> 2);
        double2 s = make_double2(0.0, 0.0);
        if (i < n) {
            for (int b0 = k; b0 < G; b0 += 64) {
                double2 v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = ld_shared(part + unsigned(min(b0 + 4 * u, G - 1) * pld + i));
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    if (b0 + 4 * u < G) {
                        s.x += v[u].x;
                        s.y += v[u].y;
                    }
                }
            }
        }
        s.x += dpp<kDppXor1>(s.x);
        s.y += dpp<kDppXor1>(s.y);
        s.x += dpp<kDppXor2>(s.x);
        s.y += dpp<kDppXor2>(s.y);
        if (k == 0 && i < n) coef[i] = s;
    }
    __syncthreads();
}

// w -= sum_{i < n} coef[i] V_i[x], the vectors in groups of 16 whose loads are issued together
__device__ void subtract(const double2* V, int64_t D, int n, unsigned x, const double2* coef, double2& w) {
    for (int i0 = 0; i0 < n; i0 += 16) {
        double2 v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = (V + int64_t(min(i0 + q, n - 1)) * D)[x];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            if (i0 + q < n) {
                const double2 c = coef[i0 + q];
                w.x -= c.x * v[q].x - c.y * v[q].y;
                w.y -= c.x * v[q].y + c.y * v[q].x;
            }
        }
    }
}

// Number of eigenvalues of the tridiagonal (d, e2 = squared off-diagonal) below x: negative
// pivots of LDL^T(T - x I), a pivot smaller in magnitude than pivmin taken as -pivmin.
__device__ int sturm_below(const double* d, const double* e2, int m, double x, double pivmin) {
    double q = d[0] - x;
    if (fabs(q) < pivmin) q = -pivmin;
    int c = q < 0.0;
#pragma unroll 4
    for (int i = 1; i < m; ++i) {
        q = (d[i] - x) - e2[i - 1] / q;
        if (fabs(q) < pivmin) q = -pivmin;
        c += q < 0.0;
    }
    return c;
}

// The testing workgroup's convergence test on T_m (diagonal al, off-diagonal be), the lowest Ritz value
// being at most hi0 (the previous test's, by interlacing; +inf at the first). theta = the lowest
// eigenvalue by multisection (kLT points per round); then y = (T - theta I)^{-1} applied twice to
// ones by elimination with partial pivoting (one thread), s_last = y[m-1] / |y|. Returns |s_last|
// (the residual estimate is beta_{m-1} |s_last|) and theta in *theta.
__device__ double ritz_last(const double* al, const double* be, int m, double hi0, double* sd, double* se,
                            double* se2, double* lu, int* first, double* theta) {
    const int t = threadIdx.x;
    for (int i = t; i < m; i += kLT) {
        sd[i] = ld_shared(al + i);
        se[i] = i + 1 < m ? ld_shared(be + i) : 0.0;
        se2[i] = se[i] * se[i];
    }
    __syncthreads();
    __shared__ double lo, hi, pivmin, slast;
    if (t == 0) {
        double l = HUGE_VAL, h = -HUGE_VAL, emax = 0.0;
        for (int i = 0; i < m; ++i) {
            const double r = (i > 0 ? fabs(se[i - 1]) : 0.0) + (i + 1 < m ? fabs(se[i]) : 0.0);
            l = fmin(l, sd[i] - r);
            h = fmax(h, sd[i] + r);
            if (i + 1 < m) emax = fmax(emax, se2[i]);
        }
        const double tn = fmax(fabs(l), fabs(h));
        pivmin = DBL_MIN * fmax(1.0, emax);
        const double pad = 2.1 * DBL_EPSILON * tn * m + 4.2 * pivmin;
        lo = l - pad;
        hi = fmin(h, hi0) + pad;
    }
    __syncthreads();
    for (int round = 0; round < 12; ++round) {
        const double l0 = lo, h0 = hi;
        if (!(h0 - l0 > 2.0 * DBL_EPSILON * fmax(fabs(l0), fabs(h0)) + pivmin)) break;
        const double step = (h0 - l0) / (kLT + 1);
        if (t == 0) *first = kLT;
        __syncthreads();
        if (sturm_below(sd, se2, m, l0 + (t + 1) * step, pivmin) >= 1) atomicMin(first, t);
        __syncthreads();
        if (t == 0) {
            const int f = *first;
            lo = f == 0 ? l0 : l0 + f * step;
            hi = f == kLT ? h0 : l0 + (f + 1) * step;
        }
        __syncthreads();
    }
    if (t == 0) {
        const double th = lo + 0.5 * (hi - lo);
        // rows of T - theta I: sub-diagonal se[i-1], diagonal c[i], super-diagonal u[i]; with row
        // swaps the eliminated rows keep at most two super-diagonals (u, u2)
        double* c = lu;
        double* u = lu + m;
        double* u2 = lu + 2 * m;
        double* y = lu + 3 * m;
        const double tiny = DBL_EPSILON * fmax(fabs(lo), fabs(hi)) + pivmin;
        for (int i = 0; i < m; ++i) y[i] = 1.0;
        for (int it = 0; it < 2; ++it) {
            for (int i = 0; i < m; ++i) {
                c[i] = sd[i] - th;
                u[i] = se[i];
                u2[i] = 0.0;
            }
            for (int i = 0; i + 1 < m; ++i) {
                const double b = se[i];  // entry (i+1, i)
                if (fabs(b) > fabs(c[i])) {
                    // swap rows i and i+1, then eliminate the old row i below the new pivot
                    const double ci = c[i], ui = u[i];
                    c[i] = b;
                    u[i] = c[i + 1];
                    u2[i] = u[i + 1];
                    const double ty = y[i];
                    y[i] = y[i + 1];
                    y[i + 1] = ty;
                    const double f = ci / b;
                    c[i + 1] = ui - f * u[i];
                    u[i + 1] = -f * u2[i];
                    y[i + 1] -= f * y[i];
                } else {
                    const double piv = c[i] != 0.0 ? c[i] : tiny;
                    c[i] = piv;
                    const double f = b / piv;
                    c[i + 1] -= f * u[i];
                    y[i + 1] -= f * y[i];
                }
            }
            if (c[m - 1] == 0.0) c[m - 1] = tiny;
            for (int i = m - 1; i >= 0; --i) {
                double r = y[i];
                if (i + 1 < m) r -= u[i] * y[i + 1];
                if (i + 2 < m) r -= u2[i] * y[i + 2];
                y[i] = r / c[i];
            }
            double nrm = 0.0;
            for (int i = 0; i < m; ++i) nrm = fmax(nrm, fabs(y[i]));
            for (int i = 0; i < m; ++i) y[i] /= nrm;
        }
        double n2 = 0.0;
        for (int i = 0; i < m; ++i) n2 += y[i] * y[i];
        slast = fabs(y[m - 1]) / sqrt(n2);
        *theta = th;
    }
    __syncthreads();
    return slast;
}

// The testing workgroup (the last of the grid; it owns no slice and takes no part in the barriers):
// after products kLCheck, 2 kLCheck, ... and nmax it tests T_n while the others go on, and leaves at the
// first n that passes, at a breakdown, or on an error. In the others' way a test cost its whole length
// (about 110 us); beside them it costs the one or two products begun before it ends, which are
// thrown away: the result is T_n and v_0..v_{n-1} either way.
__device__ void run_tests(const DevLzArgs& a, double* sd, double* se, double* se2, double* lu, int* first, int* go) {
    double theta_prev = HUGE_VAL;
    for (int n = min(kLCheck, a.nmax);; n = min(n + kLCheck, a.nmax)) {
        if (threadIdx.x == 0) {
            unsigned spins = 0;
            int ok = 1;
            while (ld_shared(a.ctl + 2) < n) {
                if (++spins > kSpinLimit) st_shared(a.ctl, 1);
                if (ld_shared(a.ctl) != 0 || ld_shared(a.ctl + 3) != 0) {
                    ok = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(32);
            }
            drain();
            const int brk = ld_shared(a.ctl + 3);  // written before the count of its product
            // a breakdown after product n leaves the test of T_n to be made: the count may have
            // passed n between the two reads
            if (!ok && ld_shared(a.ctl) == 0 && ld_shared(a.ctl + 2) >= n) ok = 1;
            if (brk != 0 && brk <= n) ok = 0;
            *go = ok;
        }
        __syncthreads();
        if (!*go) return;
        double th = 0.0;
        const double last = ritz_last(a.alpha, a.beta, n, theta_prev, sd, se, se2, lu, first, &th);
        theta_prev = th;
        if (ld_shared(a.beta + n - 1) * last <= a.tol) {
            if (threadIdx.x == 0) st_shared(a.ctl + 1, n);
            return;
        }
        if (n == a.nmax) return;
        __syncthreads();
    }
}

// The basis is kept unnormalised: u_{j+1} = w, v_{j+1} = u_{j+1} / beta_j, so the vector can be written
// before its norm is known and a product needs three grid barriers, not four. cs[i] = 1 / |u_i|.
template <unsigned CLS>
__global__ __launch_bounds__(kLT, 2) void lanczos_dev_kernel(DevLzArgs a, const double2* __restrict__ site,
                                                          const double2* __restrict__ bond,
                                                          const double2* __restrict__ dlo,
                                                          const double2* __restrict__ dmid,
                                                          const double2* __restrict__ dhi) {
    // one LDS area, laid out for the testing workgroup or for the others; under 32 KB, so that a CU can
    // hold two workgroups (the runtime counts 64 KB a CU) and 2^16 amplitudes still fit the chip
    __shared__ alignas(16) double sh[7 * kDevMaxVec];
    __shared__ double nred[kLT / 64];
    __shared__ int bad, first;
    const int t = threadIdx.x, g = blockIdx.x, G = gridDim.x - 1;
    if (g == G) {
        run_tests(a, sh, sh + kDevMaxVec, sh + 2 * kDevMaxVec, sh + 3 * kDevMaxVec, &first, &bad);
        return;
    }
    const int64_t x0 = int64_t(g) * kLT, x = x0 + t;
    const bool xok = x < a.D;
    unsigned gen = 0;
    double2* const hs = reinterpret_cast<double2*>(sh);  // h_i, both passes' sum
    double2* const ks = hs + kDevMaxVec;                 // this pass's coefficients
    double2* const wsh = ks + kDevMaxVec;                // the workgroup's slice of u_j, then of w
    double* const cs = reinterpret_cast<double*>(wsh + kLT);
    static_assert(4 * kDevMaxVec + 2 * kLT + kDevMaxVec <= 7 * kDevMaxVec, "LDS area");
    // one pass's sums <u_i|w> (in ks) become h_i = <v_i|w> = cs_i <u_i|w>, and the subtraction takes
    // cs_i h_i of u_i
    auto scale_coefs = [&](bool add, int n) {
        for (int i = t; i < n; i += kLT) {
            const double c = cs[i];
            const double2 h = make_double2(c * ks[i].x, c * ks[i].y);
            hs[i] = add ? make_double2(hs[i].x + h.x, hs[i].y + h.y) : h;
            ks[i] = make_double2(c * h.x, c * h.y);
        }
        __syncthreads();
    };
    if (t == 0) cs[0] = 1.0;
    wsh[t] = xok ? a.V[x] : make_double2(0.0, 0.0);
    __syncthreads();
    for (int j = 0; j < a.nmax; ++j) {
        const int n = j + 1;
        double2 w = make_double2(0.0, 0.0);
        if (xok) {
            const double2* u = a.V + int64_t(j) * a.D;
            // partners in the slice come from LDS
            const auto partner = [&](int mask) { return mask < kLT ? wsh[t ^ mask] : ld_shared(u + (unsigned(x) ^ unsigned(mask))); };
            w = dlo ? direct_entry<CLS>(partner, wsh[t], site, bond, dlo, dmid, dhi, a.L, int(x))
                    : small_entry<CLS, 2>(partner, site, bond, a.L, x);
            w.x *= cs[j];
            w.y *= cs[j];
        }
        __syncthreads();
        wsh[t] = w;
        __syncthreads();
        block_dots(a.V, a.D, n, x0, wsh, a.p1 + int64_t(g) * a.pld);
        if (!grid_sync(a, G, gen, &bad)) return;
        if (ld_shared(a.stop) != 0) return;
        // first pass: h1_i = <v_i|w>, w -= sum_i h1_i v_i
        sum_partials(a.p1, a.pld, G, n, ks);
        scale_coefs(false, n);
        if (xok) subtract(a.V, a.D, n, unsigned(x), ks, w);
        wsh[t] = w;
        __syncthreads();
        block_dots(a.V, a.D, n, x0, wsh, a.p2 + int64_t(g) * a.pld);
        if (!grid_sync(a, G, gen, &bad)) return;
        // second pass: u_{j+1} = w, and the partial of its squared norm
        sum_partials(a.p2, a.pld, G, n, ks);
        scale_coefs(true, n);
        double nn = 0.0;
        if (xok) {
            subtract(a.V, a.D, n, unsigned(x), ks, w);
            nn = w.x * w.x + w.y * w.y;
            st_shared(a.V + int64_t(n) * a.D + x, w);
        }
        wsh[t] = w;
        for (int o = 32; o > 0; o >>= 1) nn += __shfl_xor(nn, o, 64);
        if ((t & 63) == 0) nred[t >> 6] = nn;
        __syncthreads();
        if (t == 0) {
            double s = nred[0];
            for (int k = 1; k < kLT / 64; ++k) s += nred[k];
            st_shared(a.pn + g, s);
        }
        if (!grid_sync(a, G, gen, &bad)) return;
        // beta_j from every workgroup's partial norm, the same sum on every workgroup: lane l of each
        // wave loads rows l, l + 64, ..., and the wave sum follows a fixed butterfly
        double b2 = 0.0;
        for (int b = t & 63; b < G; b += 64) b2 += ld_shared(a.pn + b);
        for (int o = 32; o > 0; o >>= 1) b2 += __shfl_xor(b2, o, 64);
        const double beta = sqrt(b2);
        double hmax = 0.0;  // the same maximum on every thread
        for (int i = t & 63; i < n; i += 64) {
            hmax = fmax(hmax, sqrt(hs[i].x * hs[i].x + hs[i].y * hs[i].y));
        }
        for (int o = 32; o > 0; o >>= 1) hmax = fmax(hmax, __shfl_xor(hmax, o, 64));
        const bool brk = beta <= 1e-14 * fmax(hmax, 1e-300) || beta == 0.0;
        if (t == 0) cs[n] = brk ? 0.0 : 1.0 / beta;
        if (g == 0 && t == 0) {
            st_shared(a.alpha + j, hs[j].x);
            st_shared(a.beta + j, beta);
            if (brk) st_shared(a.ctl + 3, n);
            drain();
            st_shared(a.ctl + 2, n);
            // read by every workgroup after the next barrier, so that all stop together
            if (ld_shared(a.ctl + 1) != 0) st_shared(a.stop, 1);
        }
        if (brk) return;  // the same on every workgroup
        __syncthreads();
    }
}

template <unsigned CLS>
hipError_t launch_dev(const ed_model* m, const DevLzArgs& a, int G, hipStream_t s) {
    DevLzArgs args = a;
    const double2 *site = m->d_site, *bond = m->d_bond, *dlo = nullptr, *dmid = nullptr, *dhi = nullptr;
    if (m->L >= kTileBits) {
        dlo = m->d_diag_lo;
        dmid = m->d_diag_mid;
        dhi = m->d_diag_hi;
    }
    void* params[] = {&args, &site, &bond, &dlo, &dmid, &dhi};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&lanczos_dev_kernel<CLS>), dim3(G + 1), dim3(kLT),
                                      params, 0, s);
}

template <int I>
hipError_t dispatch_dev(const ed_model* m, const DevLzArgs& a, int G, hipStream_t s) {
    if constexpr (I >= kNumVariants) {
        return hipErrorInvalidValue;
    } else {
        if (variant_fits(kVariants[I], m->op_class)) return launch_dev<kVariants[I]>(m, a, G, s);
        return dispatch_dev<I + 1>(m, a, G, s);
    }
}

__global__ void clear_ints(int* p, int n) {
    const int i = int(threadIdx.x);
    if (i < n) p[i] = 0;
}

}  // namespace

bool lanczos_device_fits(const ed_model* m, int max_iter) {
    if (m->L > kDevLanczosMaxL || m->lr || m->lv_L > 0 || !m->far.empty()) return false;
    if (max_iter < 1 || max_iter > kDevMaxVec - 1) return false;
    const int64_t D = int64_t(1) << m->L;
    const int64_t G = (D + kLT - 1) / kLT;
    return 2 * G * int64_t(max_iter + 1) * int64_t(sizeof(double2)) <= int64_t(kPartBytes);
}

ed_status lanczos_device(const ed_model* m, const Workspace& w, int max_iter, double tol, int* m_out,
                         int* products, bool* converged, std::vector<double>* alpha, std::vector<double>* beta,
                         hipStream_t s) {
    const int64_t D = w.D;
    const int G = int((D + kLT - 1) / kLT);
    DevLzArgs a;
    a.L = m->L;
    a.D = D;
    a.V = w.V;
    a.nmax = max_iter;
    a.pld = max_iter + 1;
    a.p1 = w.part;
    a.p2 = w.part + int64_t(G) * a.pld;
    // device scalars after the ones the step kernels use: pn[G], alpha, beta, barrier and control
    double* sc = reinterpret_cast<double*>(w.scal + kObs);
    static_assert(kScalars - kObs >= 8, "scalar area");
    double* base = reinterpret_cast<double*>(w.scal + 1);  // the h1/h2 area is free on this path
    a.pn = base;
    a.alpha = base + G;
    a.beta = a.alpha + max_iter;
    unsigned* bar = reinterpret_cast<unsigned*>(sc);
    a.bar = bar;
    a.stop = reinterpret_cast<int*>(sc) + 1;
    a.ctl = reinterpret_cast<int*>(sc) + 4;
    a.tol = tol;
    if (size_t(G + 2 * max_iter) * sizeof(double) > size_t(2 * kMaxProj) * sizeof(double2))
        return fail(ED_ERR_UNSUPPORTED, "device Lanczos: too many scalars");
    hipLaunchKernelGGL(clear_ints, dim3(1), dim3(64), 0, s, reinterpret_cast<int*>(sc), 8);
    hipError_t e = dispatch_dev<0>(m, a, G, s);
    if (e == hipErrorCooperativeLaunchTooLarge) {
        // the workgroups cannot all be resident now: the caller runs the host-driven recurrence
        (void)hipGetLastError();
        *products = 0;
        return ED_ERR_UNSUPPORTED;
    }
    if (e != hipSuccess) return fail(ED_ERR_HIP, std::string("device Lanczos launch: ") + hipGetErrorString(e));
    int ctl[4] = {0, 0, 0, 0};
    ED_HIP_TRY(hipMemcpyAsync(ctl, a.ctl, sizeof(ctl), hipMemcpyDeviceToHost, s));
    ED_HIP_TRY(hipStreamSynchronize(s));
    if (ctl[0] != 0) return fail(ED_ERR_HIP, "device Lanczos: a grid barrier timed out");
    *converged = ctl[1] != 0 || ctl[3] != 0;
    *m_out = ctl[1] != 0 ? ctl[1] : ctl[3] != 0 ? ctl[3] : ctl[2];
    *products = *m_out;
    alpha->assign(size_t(*m_out), 0.0);
    beta->assign(size_t(*m_out), 0.0);
    if (*m_out > 0) {
        ED_HIP_TRY(hipMemcpy(alpha->data(), a.alpha, sizeof(double) * size_t(*m_out), hipMemcpyDeviceToHost));
        ED_HIP_TRY(hipMemcpy(beta->data(), a.beta, sizeof(double) * size_t(*m_out), hipMemcpyDeviceToHost));
    }
    return ED_OK;
}

}  // namespace ed
