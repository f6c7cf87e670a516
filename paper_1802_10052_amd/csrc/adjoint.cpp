// Gradient of a final-time observable with respect to piecewise-constant bond couplings, by
// costate (adjoint) back-propagation through the Krylov time evolution of Sec. ed:sec:krylov.
//
//   H_s = sum_b J[s][b] h_b + H_site    (h_b: the template's bond operator on bond b)
//   psi_s = exp(-i H_s Delta) psi_{s-1},  Loss = <psi_S|O|psi_S>,  O = sum_k w_k sigma^z_k
//   lam_S = O psi_S,  lam_{s-1} = exp(+i H_s Delta) lam_s
//   dLoss/dJ[s][b] = 2 int_0^Delta Im <mu(tau)| h_b |phi(tau)> dtau,
//       phi(tau) = exp(-i H_s tau) psi_{s-1},  mu(tau) = exp(-i H_s tau) lam_{s-1}.
// The forward pass stores psi_s at every slice boundary (checkpoints). The backward pass
// propagates the costate one slice back, then walks the slice in sub-steps: a Krylov basis of
// phi and of mu at the sub-step start gives both at every Gauss-Legendre node, and one fused
// pass per node returns Im<mu|h_b|phi> for every bond at once.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <vector>

#include "dense.h"
#include "ed_vec.h"
#include "hpsi_device.h"
#include "krylov_core.h"

namespace ed {

ed_status create_model(const ed_model_desc* desc, ed_model** out);
void destroy_model(ed_model* m);

namespace {

constexpr int kBT = 256;
constexpr int kAdjScal = 640;  // bond sums one copy fetches (scalars between the tickets and N at m_max = 64)
static_assert(kThreeTermFree + kAdjScal + 3 * 64 + 2 <= kObs, "scalar area");
constexpr int kBTile = 12;     // tile bits
constexpr int kBLow = 3;       // contiguous low bits of a window tile
constexpr int kBThr = 512;     // threads per tile, 8 amplitudes each
constexpr int kBSlots = (1 << kBTile) / kBThr;
constexpr int kBTb = 9;        // thread bits

// One pass over 12-bit tiles (the low bits, or c low bits and a window of 12 - c bits at h0):
// part[tile][p] = sum over the tile of conj(mu[x]) (h_p phi)[x] for the bonds on tile bits
// (q, q + 1), q0 <= q < q1, of global bit p. phi's tile sits in LDS, so a flipped partner costs an LDS
// read; both vectors are read once per pass. Bound by LDS and FP64: 40 us for both passes at L = 20, where
// gathering every partner from global memory took 139 us.
struct BondPass {
    int first, h0, c, tbits;
    int q0, q1;
};

__global__ __launch_bounds__(kBThr) void bond_expect_tile(const double2* __restrict__ mu, const double2* __restrict__ phi,
                                                          const double2* __restrict__ bond, BondPass bp,
                                                          double2* __restrict__ part, int part_ld) {
    __shared__ double2 s[1 << kBTile];
    __shared__ double red[kBThr / 64][2 * (kBTile - 1)];
    const int t = threadIdx.x;
    const int N = 1 << bp.tbits;
    const int64_t n = blockIdx.x;
    int64_t base;
    int hs;  // tile index i is base + (i & (2^c - 1)) + (i >> c) << hs
    if (bp.first) {
        base = n << bp.tbits;
        hs = bp.c;
    } else {
        const int lo_bits = bp.h0 - bp.c;
        base = ((n & ((int64_t(1) << lo_bits) - 1)) << bp.c) | ((n >> lo_bits) << (bp.h0 + kBTile - bp.c));
        hs = bp.h0;
    }
    double2 f[kBSlots], m[kBSlots];
#pragma unroll
    for (int k = 0; k < kBSlots; ++k) {
        const int i = t + kBThr * k;
        f[k] = m[k] = make_double2(0.0, 0.0);
        if (i < N) {
            const int64_t x = base + ((int64_t(i >> bp.c) << hs) | (i & ((1 << bp.c) - 1)));
            f[k] = phi[x];
            m[k] = mu[x];
        }
        s[i] = f[k];
    }
    __syncthreads();
    const int lane = t & 63, wv = t >> 6;
#pragma unroll
    for (int q = 0; q < kBTile - 1; ++q) {
        double ax = 0.0, ay = 0.0;
        if (q >= bp.q0 && q < bp.q1) {
            const int p = bp.first || q < bp.c ? q : bp.h0 + q - bp.c;
            const double2* B = bond + 16 * p;
            double2 hv[kBSlots];
            {
                const double2 d0 = B[0], d1 = B[5], d2 = B[10], d3 = B[15];
#pragma unroll
                for (int k = 0; k < kBSlots; ++k) {
                    const int l = ((t + kBThr * k) >> q) & 3;
                    hv[k] = cmul(sel4(l, d0, d1, d2, d3), f[k]);
                }
            }
#pragma unroll
            for (int mm = 1; mm < 4; ++mm) {
                const double2 b0 = B[0 + (0 ^ mm)], b1 = B[4 + (1 ^ mm)], b2 = B[8 + (2 ^ mm)], b3 = B[12 + (3 ^ mm)];
                const double any = fabs(b0.x) + fabs(b0.y) + fabs(b1.x) + fabs(b1.y) + fabs(b2.x) + fabs(b2.y) +
                                   fabs(b3.x) + fabs(b3.y);
                if (any == 0.0) continue;  // the same for all threads
#pragma unroll
                for (int k = 0; k < kBSlots; ++k) {
                    const int i = t + kBThr * k;
                    cfma<false>(hv[k], sel4((i >> q) & 3, b0, b1, b2, b3), s[i ^ (mm << q)]);
                }
            }
#pragma unroll
            for (int k = 0; k < kBSlots; ++k) {  // conj(m) * hv
                ax = fma(m[k].x, hv[k].x, fma(m[k].y, hv[k].y, ax));
                ay = fma(m[k].x, hv[k].y, fma(-m[k].y, hv[k].x, ay));
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                ax += __shfl_xor(ax, o, 64);
                ay += __shfl_xor(ay, o, 64);
            }
            if (lane == 0) {
                red[wv][2 * q] = ax;
                red[wv][2 * q + 1] = ay;
            }
        }
    }
    __syncthreads();
    const int q = t >> 1;
    if (q >= bp.q0 && q < bp.q1) {
        double v = 0.0;
        for (int w = 0; w < kBThr / 64; ++w) v += red[w][t];
        const int p = bp.first || q < bp.c ? q : bp.h0 + q - bp.c;
        reinterpret_cast<double*>(part + n * part_ld + p)[t & 1] = v;
    }
}

// out[x] = (sum_k w_k (1 - 2 bit_{L-k}(x))) psi[x]   (O = sum_k w_k sigma^z_k, diagonal)
__global__ __launch_bounds__(kBT) void apply_zobs(const double2* __restrict__ psi, double2* __restrict__ out, int L,
                                                 const double* __restrict__ w) {
    const int64_t D = int64_t(1) << L;
    const int64_t stride = int64_t(gridDim.x) * kBT;
    for (int64_t x = int64_t(blockIdx.x) * kBT + threadIdx.x; x < D; x += stride) {
        double o = 0.0;
        for (int k = 1; k <= L; ++k) o += ((x >> (L - k)) & 1) ? -w[k - 1] : w[k - 1];
        const double2 y = psi[x];
        out[x] = make_double2(o * y.x, o * y.y);
    }
}

// __global__ reduce of the partials lives in vec.hip; reuse through the public launchers
}  // namespace

hipError_t bond_expect(const double2* mu, const double2* phi, const double2* bond, int L, double2* out,
                       double2* part, hipStream_t s);

// Gauss-Legendre nodes x_q in (-1, 1) and weights, by Newton iteration on P_n (from the
// three-term recurrence of the Legendre polynomials).
void gauss_legendre(int n, std::vector<double>& x, std::vector<double>& w) {
    x.assign(n, 0.0);
    w.assign(n, 0.0);
    for (int i = 0; i < (n + 1) / 2; ++i) {
        double z = std::cos(M_PI * (i + 0.75) / (n + 0.5));
        double pp = 0.0;
        for (int it = 0; it < 100; ++it) {
            double p1 = 1.0, p2 = 0.0;
            for (int j = 1; j <= n; ++j) {
                const double p3 = p2;
                p2 = p1;
                p1 = ((2.0 * j - 1.0) * z * p2 - (j - 1.0) * p3) / j;
            }
            pp = n * (z * p1 - p2) / (z * z - 1.0);
            const double z1 = z;
            z = z1 - p1 / pp;
            if (std::fabs(z - z1) < 1e-16) break;
        }
        x[i] = -z;
        x[n - 1 - i] = z;
        w[i] = 2.0 / ((1.0 - z * z) * pp * pp);
        w[n - 1 - i] = w[i];
    }
}

namespace {

struct ModelSet {
    std::vector<ed_model*> m;
    ~ModelSet() {
        for (ed_model* x : m) destroy_model(x);
    }
};

// H_s from the template: its folded site operators unchanged, bond operator of bond b (sites
// b+1, b+2) scaled by J[s][b].
ed_status slice_models(const ed_model* tmpl, int S, const double* J, ModelSet* ms) {
    const int L = tmpl->L;
    std::vector<ed_c64> sop(4 * L), bop(16 * (L - 1));
    std::vector<double> scoef(size_t(L) * L, 0.0), bcoef(size_t(L - 1) * (L - 1), 0.0);
    for (int k = 1; k <= L; ++k) {
        const int p = L - k;
        for (int e = 0; e < 4; ++e) sop[4 * (k - 1) + e] = ed_c64{tmpl->site[4 * p + e].x, tmpl->site[4 * p + e].y};
        scoef[size_t(k - 1) * L + (k - 1)] = 1.0;
    }
    for (int k = 1; k <= L - 1; ++k) {
        const int p = L - k - 1;
        for (int e = 0; e < 16; ++e) bop[16 * (k - 1) + e] = ed_c64{tmpl->bond[16 * p + e].x, tmpl->bond[16 * p + e].y};
    }
    for (int s = 0; s < S; ++s) {
        for (int b = 0; b < L - 1; ++b) bcoef[size_t(b) * (L - 1) + b] = J[size_t(s) * (L - 1) + b];
        ed_model_desc d{L, 2, L, sop.data(), scoef.data(), L - 1, bop.data(), bcoef.data()};
        ed_model* m = nullptr;
        ED_TRY(create_model(&d, &m));
        ms->m.push_back(m);
    }
    return ED_OK;
}

struct Basis {
    Workspace w;
    ThreeTerm T;
    std::vector<xreal> d, Z;  // eigenpairs of the tridiagonal T (extended precision)
    int m = 0;
    double nrm = 0.0;
};

// Lanczos basis of psi under model (three-term recurrence with local re-projection, or fixed m); alias:
// psi itself is u_0 (it must then stay until the basis is no longer needed), else a copy is.
// Both projections are taken (local re-projection): the bases run at a fixed dimension well past
// convergence, where the gradient check needs the more orthogonal basis. The iterations of a fixed
// dimension are enqueued at once; adaptive ones in batches of the last basis's dimension.
ed_status build_basis(const ed_model* mod, const double2* psi, double dt_err, const ed_adjoint_params* p, Basis* B,
                      bool alias, hipStream_t s) {
    const int mmax = p->m_max;
    const int guess = B->m;
    ED_TRY(three_term_start(B->T, B->w, psi, alias, false, s));
    std::vector<double> a(mmax + 1), b(mmax + 1);
    std::vector<double2> hv(B->T.count());
    const double2 *hN = hv.data(), *hS = hN + (B->T.SP - B->T.N);
    int m = 0, enq = 0;
    bool stop = false;
    while (!stop) {
        int nb = p->m_fixed > 0 ? std::min(p->m_fixed, mmax) : std::max(guess - enq, 1);
        nb = std::min(nb, mmax - enq);
        ED_TRY(three_term_run(mod, B->T, B->w, enq, nb, true, s));
        enq += nb;
        ED_TRY(fetch_scalars(B->T.N, B->T.count(), hv.data(), s));
        for (; m < enq && !stop;) {
            const int j = m;
            if (j == 0) {
                if (!std::isfinite(hN[0].x)) return fail(ED_ERR_NUMERIC, "non-finite start vector");
                if (hN[0].x <= 0.0) return fail(ED_ERR_ARG, "start vector is zero");
                B->nrm = std::sqrt(hN[0].x);
            }
            if (!std::isfinite(hN[j + 1].x) || !std::isfinite(hS[2 * j].x))
                return fail(ED_ERR_NUMERIC, "non-finite value in the Krylov recurrence");
            const cplx h(hS[2 * j].x / hN[j].x, hS[2 * j].y / hN[j].x);
            const double hp =
                j > 0 ? std::hypot(hS[2 * j + 1].x, hS[2 * j + 1].y) / std::sqrt(hN[j - 1].x * hN[j].x) : 0.0;
            a[j] = h.real();
            bool brk = false;
            ED_TRY(three_term_beta(hN, j, std::max(std::abs(h), hp), &b[j], &brk));
            m = j + 1;
            stop = brk || m >= mmax;
            if (p->m_fixed > 0) {
                stop = brk || m >= std::min(p->m_fixed, mmax);
            } else if (!stop) {
                std::vector<xreal> dd(a.begin(), a.begin() + m), ee(m, 0.0L), Z(size_t(m) * m, 0.0L);
                for (int i = 0; i + 1 < m; ++i) ee[i] = b[i];
                for (int i = 0; i < m; ++i) Z[size_t(i) * m + i] = 1.0L;
                if (!tridiag_ql_ext(m, dd.data(), ee.data(), Z.data()))
                    return fail(ED_ERR_NUMERIC, "tridiagonal eigensolver did not converge");
                std::vector<cplx> u(m);
                expm_col_sym_ext(m, dd.data(), Z.data(), std::fabs(dt_err), u.data());
                stop = B->nrm * b[j] * std::abs(u[m - 1]) <= p->tol;
            }
        }
    }
    B->m = m;
    for (int i = 0; i < m; ++i) B->w.c[i] = 1.0 / std::sqrt(hN[i].x);
    B->d.assign(a.begin(), a.begin() + m);
    std::vector<xreal> ee(m, 0.0L);
    for (int i = 0; i + 1 < m; ++i) ee[i] = b[i];
    B->Z.assign(size_t(m) * m, 0.0L);
    for (int i = 0; i < m; ++i) B->Z[size_t(i) * m + i] = 1.0L;
    if (!tridiag_ql_ext(m, B->d.data(), ee.data(), B->Z.data()))
        return fail(ED_ERR_NUMERIC, "tridiagonal eigensolver did not converge");
    return ED_OK;
}

// out = nrm V exp(-i tau T) e_1
ed_status eval_basis(const Basis& B, double tau, double2* out, hipStream_t s) {
    std::vector<cplx> u(B.m);
    expm_col_sym_ext(B.m, B.d.data(), B.Z.data(), tau, u.data());
    std::vector<double2> c(B.m);
    for (int i = 0; i < B.m; ++i) c[i] = make_double2(B.nrm * u[i].real(), B.nrm * u[i].imag());
    return combine_basis(B.w, B.m, c.data(), out, s);
}

// out_q = nrm V exp(-i tau_q T) e_1 for up to kNodeOut times in one sweep of the basis; no output may
// be a basis vector
ed_status eval_nodes(const Basis& B, const std::vector<double>& tau, const std::vector<double2*>& out, hipStream_t s) {
    const int n = int(tau.size());
    std::vector<cplx> u(B.m);
    std::vector<double2> C(size_t(B.m) * n);
    for (int q = 0; q < n; ++q) {
        expm_col_sym_ext(B.m, B.d.data(), B.Z.data(), tau[q], u.data());
        for (int i = 0; i < B.m; ++i) {
            const double f = B.nrm * B.w.c[i];
            C[size_t(i) * n + q] = make_double2(f * u[i].real(), f * u[i].imag());
        }
    }
    if (combination_nodes(const_cast<const double2* const*>(B.w.u.data()), B.m, C.data(), out.data(), n, B.w.D, s) !=
        hipSuccess)
        return fail(ED_ERR_HIP, "node combination");
    return ED_OK;
}

// psi <- exp(-i H dt) psi through K sub-steps
ed_status propagate(const ed_model* mod, double2* psi, double dt, int K, const ed_adjoint_params* p, Basis* B,
                    hipStream_t s) {
    for (int k = 0; k < K; ++k) {
        ED_TRY(build_basis(mod, psi, dt / K, p, B, true, s));
        ED_TRY(eval_basis(*B, dt / K, psi, s));
    }
    return ED_OK;
}

size_t al(size_t x) { return (x + 255) & ~size_t(255); }

ed_status check_params(const ed_model* tmpl, int S, double Delta, const double* J, const ed_c64* psi0, const double* w,
                       const ed_adjoint_params* p) {
    if (tmpl && tmpl->lr) return fail(ED_ERR_UNSUPPORTED, "the adjoint does not take long-range (InfiniteFunc) terms");
    if (tmpl && tmpl->lv_L > 0) return fail(ED_ERR_UNSUPPORTED, "the adjoint does not take Liouvillian models");
    if (!tmpl || !J || !psi0 || !w || !p) return fail(ED_ERR_ARG, "null argument");
    if (S < 1 || !(Delta > 0.0)) return fail(ED_ERR_ARG, "n_slices >= 1 and slice_len > 0 required");
    if (tmpl->L > 24) return fail(ED_ERR_UNSUPPORTED, "the adjoint path supports L <= 24");
    if (p->substeps < 1 || p->quad_nodes < 1 || p->quad_nodes > 64) return fail(ED_ERR_ARG, "bad substeps / quad_nodes");
    if (p->m_max < 2 || p->m_max > 64) return fail(ED_ERR_ARG, "m_max must be in [2, 64]");
    if (p->m_fixed <= 0 && !(p->tol > 0.0)) return fail(ED_ERR_ARG, "tol must be > 0");
    for (int i = 0; i < S * (tmpl->L - 1); ++i)
        if (!std::isfinite(J[i])) return fail(ED_ERR_NUMERIC, "non-finite coupling");
    return ED_OK;
}

ed_status loss_of(const double2* psi, int L, const double* w, const Workspace& ws, double* loss, hipStream_t s) {
    std::vector<double> sz(L);
    double nrm = 0.0;
    ED_TRY(measure_state(psi, L, ws, sz.data(), &nrm, s));
    double acc = 0.0;
    for (int k = 0; k < L; ++k) acc += w[k] * sz[k];
    *loss = acc * nrm * nrm;
    return ED_OK;
}

}  // namespace
}  // namespace ed

using namespace ed;

extern "C" ed_status ed_adjoint_workspace(const ed_model* tmpl, int n_slices, const ed_adjoint_params* p, size_t* bytes) {
    if (!tmpl || !p || !bytes || n_slices < 1) return fail(ED_ERR_ARG, "bad argument");
    const int64_t D = int64_t(1) << tmpl->L;
    const size_t vec = size_t(D) * sizeof(double2);
    // two bases (phi, mu) of m_max + 1 vectors, checkpoints S + 1, lambda, 2 node vectors, w (L doubles)
    *bytes = 2 * (core_scratch_bytes() + al(size_t(p->m_max + 1) * vec)) + al(size_t(n_slices + 1) * vec) + 3 * al(vec) +
             al(64 * sizeof(double));
    return ED_OK;
}

extern "C" ed_status ed_evolve_adjoint(const ed_model* tmpl, int n_slices, double slice_len, const double* J,
                                      const ed_c64* psi0, const double* obs_w, const ed_adjoint_params* p,
                                      double* loss, double* grad, void* ws, size_t ws_bytes, void* stream) {
    ED_TRY(check_params(tmpl, n_slices, slice_len, J, psi0, obs_w, p));
    if (!loss || !grad) return fail(ED_ERR_ARG, "null output");
    size_t need = 0;
    ED_TRY(ed_adjoint_workspace(tmpl, n_slices, p, &need));
    if (!ws) return fail(ED_ERR_ARG, "workspace is null");
    if (ws_bytes < need) return fail(ED_ERR_WORKSPACE, "workspace too small");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int L = tmpl->L, S = n_slices, NB = L - 1;
    const int64_t D = int64_t(1) << L;
    const size_t vec = size_t(D) * sizeof(double2);
    char* c = static_cast<char*>(ws);
    Basis Bp, Bm;
    const size_t basis_bytes = core_scratch_bytes() + al(size_t(p->m_max + 1) * vec);
    ED_TRY(carve(c, basis_bytes, D, p->m_max + 1, &Bp.w));
    c += basis_bytes;
    ED_TRY(carve(c, basis_bytes, D, p->m_max + 1, &Bm.w));
    c += basis_bytes;
    double2* ck = reinterpret_cast<double2*>(c);
    c += al(size_t(S + 1) * vec);
    double2* lam = reinterpret_cast<double2*>(c);
    c += al(vec);
    double2* phin = reinterpret_cast<double2*>(c);
    c += al(vec);
    double2* mun = reinterpret_cast<double2*>(c);
    c += al(vec);
    double* dw = reinterpret_cast<double*>(c);
    ED_TRY(three_term_init(Bp.w, p->m_max, &Bp.T, s));
    ED_TRY(three_term_init(Bm.w, p->m_max, &Bm.T, s));

    ModelSet ms;
    ED_TRY(slice_models(tmpl, S, J, &ms));
    const int K = p->substeps;
    // forward with checkpoints
    ED_HIP_TRY(hipMemcpyAsync(ck, psi0, vec, hipMemcpyDeviceToDevice, s));
    for (int sl = 0; sl < S; ++sl) {
        double2* nxt = ck + int64_t(sl + 1) * D;
        ED_HIP_TRY(hipMemcpyAsync(nxt, ck + int64_t(sl) * D, vec, hipMemcpyDeviceToDevice, s));
        ED_TRY(propagate(ms.m[sl], nxt, slice_len, K, p, &Bp, s));
    }
    ED_TRY(loss_of(ck + int64_t(S) * D, L, obs_w, Bp.w, loss, s));
    // costate lam_S = O psi_S
    ED_HIP_TRY(hipMemcpyAsync(dw, obs_w, sizeof(double) * L, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(apply_zobs, dim3(unsigned(std::min<int64_t>((D + kBT - 1) / kBT, 4096))), dim3(kBT), 0, s,
                       ck + int64_t(S) * D, lam, L, dw);
    ED_HIP_TRY(hipGetLastError());
    std::vector<double> xq, wq;
    gauss_legendre(p->quad_nodes, xq, wq);
    const double delta = slice_len / K;
    std::vector<double2> z;
    double2* const zdev = Bp.w.scal + kThreeTermFree;  // free between the tickets and the recurrence's scalars
    for (int sl = S - 1; sl >= 0; --sl) {
        const ed_model* Hs = ms.m[sl];
        // lam_{s-1} = exp(+i H_s Delta) lam_s
        ED_TRY(propagate(Hs, lam, -slice_len, K, p, &Bm, s));
        // walk the slice: phi from the checkpoint, mu from lam_{s-1}
        ED_HIP_TRY(hipMemcpyAsync(phin, ck + int64_t(sl) * D, vec, hipMemcpyDeviceToDevice, s));
        ED_HIP_TRY(hipMemcpyAsync(mun, lam, vec, hipMemcpyDeviceToDevice, s));
        std::vector<double> g(NB, 0.0);
        for (int k = 0; k < K; ++k) {
            ED_TRY(build_basis(Hs, phin, delta, p, &Bp, false, s));
            ED_TRY(build_basis(Hs, mun, delta, p, &Bm, false, s));
            // the quadrature nodes, as many at a time as the slots behind both bases hold (always
            // one: slot m is free), the states at the end of the sub-step with the last of them
            const int room = std::min(std::min(p->m_max + 1 - Bp.m, p->m_max + 1 - Bm.m), kNodeOut - 1);
            const int zrows = std::max(1, kAdjScal / NB);
            int queued = 0, done = 0;  // node results waiting on the device, and read
            for (int q0 = 0; q0 < p->quad_nodes; q0 += room) {
                const int nq = std::min(room, p->quad_nodes - q0);
                const bool end = q0 + nq == p->quad_nodes;
                std::vector<double> tau(nq);
                for (int q = 0; q < nq; ++q) tau[q] = 0.5 * delta * (1.0 + xq[q0 + q]);
                if (end) tau.push_back(delta);
                std::vector<double2*> op, om;
                for (int q = 0; q < nq; ++q) {
                    op.push_back(Bp.w.slot(Bp.m + q));
                    om.push_back(Bm.w.slot(Bm.m + q));
                }
                if (end) {
                    op.push_back(phin);
                    om.push_back(mun);
                }
                ED_TRY(eval_nodes(Bp, tau, op, s));
                ED_TRY(eval_nodes(Bm, tau, om, s));
                for (int q = 0; q < nq; ++q) {
                    if (bond_expect(om[q], op[q], tmpl->d_bond, L, zdev + size_t(queued) * NB, Bp.w.part, s) != hipSuccess)
                        return fail(ED_ERR_HIP, "bond reduction");
                    ++queued;
                    if (queued == zrows || (end && q + 1 == nq)) {
                        z.resize(size_t(queued) * NB);
                        ED_TRY(fetch_scalars(zdev, queued * NB, z.data(), s));
                        // bond bit p = L - b - 2 for bond b (sites b+1, b+2)
                        for (int r = 0; r < queued; ++r, ++done)
                            for (int b = 0; b < NB; ++b)
                                g[b] += 0.5 * delta * wq[done] * 2.0 * z[size_t(r) * NB + L - b - 2].y;
                        queued = 0;
                    }
                }
            }
        }
        for (int b = 0; b < NB; ++b) grad[size_t(sl) * NB + b] = g[b];
    }
    ED_HIP_TRY(hipStreamSynchronize(s));
    return ED_OK;
}

extern "C" ed_status ed_evolve_loss_workspace(const ed_model* tmpl, const ed_adjoint_params* p, size_t* bytes) {
    if (!tmpl || !p || !bytes) return fail(ED_ERR_ARG, "bad argument");
    const int64_t D = int64_t(1) << tmpl->L;
    *bytes = core_scratch_bytes() + al(size_t(p->m_max + 1) * size_t(D) * sizeof(double2)) + al(size_t(D) * sizeof(double2));
    return ED_OK;
}

extern "C" ed_status ed_evolve_loss(const ed_model* tmpl, int n_slices, double slice_len, const double* J,
                                   const ed_c64* psi0, const double* obs_w, const ed_adjoint_params* p, double* loss,
                                   void* ws, size_t ws_bytes, void* stream) {
    ED_TRY(check_params(tmpl, n_slices, slice_len, J, psi0, obs_w, p));
    if (!loss) return fail(ED_ERR_ARG, "null output");
    size_t need = 0;
    ED_TRY(ed_evolve_loss_workspace(tmpl, p, &need));
    if (!ws) return fail(ED_ERR_ARG, "workspace is null");
    if (ws_bytes < need) return fail(ED_ERR_WORKSPACE, "workspace too small");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int L = tmpl->L;
    const int64_t D = int64_t(1) << L;
    Basis B;
    const size_t basis_bytes = core_scratch_bytes() + al(size_t(p->m_max + 1) * size_t(D) * sizeof(double2));
    ED_TRY(carve(ws, basis_bytes, D, p->m_max + 1, &B.w));
    double2* psi = reinterpret_cast<double2*>(static_cast<char*>(ws) + basis_bytes);
    ED_TRY(three_term_init(B.w, p->m_max, &B.T, s));
    ModelSet ms;
    ED_TRY(slice_models(tmpl, n_slices, J, &ms));
    ED_HIP_TRY(hipMemcpyAsync(psi, psi0, size_t(D) * sizeof(double2), hipMemcpyDeviceToDevice, s));
    for (int sl = 0; sl < n_slices; ++sl) ED_TRY(propagate(ms.m[sl], psi, slice_len, p->substeps, p, &B, s));
    ED_TRY(loss_of(psi, L, obs_w, B.w, loss, s));
    return ED_OK;
}

namespace ed {
hipError_t bond_expect(const double2* mu, const double2* phi, const double2* bond, int L, double2* out, double2* part,
                       hipStream_t s) {
    const int tbits = std::min(L, kBTile);
    const unsigned tiles = 1u << (L - tbits);
    BondPass bp{1, 0, std::min(kBLow, tbits), tbits, 0, std::min(L - 1, kBTile - 1)};
    hipLaunchKernelGGL(bond_expect_tile, dim3(tiles), dim3(kBThr), 0, s, mu, phi, bond, bp, part, kPartLd);
    // windows: each takes the bonds from the lowest one pending up to its own top
    for (int p = kBTile - 1; p < L - 1;) {
        const int w = kBTile - kBLow, h0 = std::min(p, L - w);
        const int top = std::min(h0 + w - 1, L - 1);  // bonds p .. top - 1
        bp = BondPass{0, h0, kBLow, kBTile, kBLow + p - h0, kBLow + top - h0};
        hipLaunchKernelGGL(bond_expect_tile, dim3(tiles), dim3(kBThr), 0, s, mu, phi, bond, bp, part, kPartLd);
        p = top;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce_partial_rows(part, int(tiles), L - 1, out, s);
}
}  // namespace ed
