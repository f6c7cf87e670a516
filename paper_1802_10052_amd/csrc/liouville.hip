// Liouville-space evolution (Sec. ed:sec:Liouville, Eqs. ed:eq:lioutrafo, ed:eq:liousuperket, App. F): the
// density matrix of an L-site system as the superket |rho>> of 2L digits (row-major vec(rho): the
// row index is the high L bits, the column index the low L bits), and
//   i Lcal = H_eff (x) 1 - 1 (x) H_eff^* + i sum_nu gamma_nu J_nu (x) J_nu^*,
//   H_eff = H - (i/2) sum_nu gamma_nu J_nu^dagger J_nu,
// so that exp(-i t (i Lcal)) = exp(t Lcal) and the Krylov time step applies unchanged (Arnoldi:
// i Lcal is not Hermitian). The first two terms are a local operator on the 2L-bit chain (site and
// bond terms on the row half and on the column half, nothing on the middle bond) and run through
// the streaming H psi passes; the jump sandwiches couple row bit L + (L - k) with column bit L - k
// of the same site k, L bits apart, and are applied here as far terms by a gather pass.
#include <algorithm>
#include <cmath>
#include <vector>

#include "ed_internal.h"

namespace ed {
namespace {

constexpr int kFarThreads = 256;
constexpr int kFarLow = 4;   // a cell: 2^4 rows j and 2^4 columns k, in 256-byte runs

// out[x] += sum_f sum_c K_f[r(x)][c] psi[x with bits (q_f, p_f) set to c], r(x) = 2 bit q + bit p,
// for terms that couple row bit p + Ls with column bit p (q = p + Ls).
// Bound by HBM: out is read and written once (32 B per entry) and psi should be read once (16 B), but
// each entry gathers up to one partner per term. A term flips the same bit of j and k, so the entries
// with one value of j XOR k never leave each other. A group (one value of the high bits of j XOR k) is
// 4 MiB of psi at L = 14; its cells run back to back on one XCD (workgroups are dealt to the 8 XCDs
// round-robin) and gather from its L2, while out streams past it: psi is then read once from HBM
// (counted: 8.6 GB for psi and out at L = 14). With ROWS = 4 a wave takes a cell; a thread's four rows
// share the term's row index, so four gathers are in flight and the per-term work is paid once; with
// one entry per thread the instructions bounded the pass (3.9 ms at L = 14). L = 14: 2.6 ms (4.9 TB/s
// of the 48 B per entry), 4.9 ms in index order. ROWS = 1 (a quarter of a cell per wave) fills the
// chip below 2^20 entries: L = 8 takes 21 us per product, 24 us with ROWS = 4.
template <int ROWS>
__global__ __launch_bounds__(kFarThreads) void far_terms(const double2* __restrict__ psi, double2* __restrict__ out,
                                                         const FarTerm* __restrict__ terms, int nterms, int Ls) {
    const int hb = Ls - kFarLow;  // high bits of j and of k
    const int lane = threadIdx.x & 63;
    constexpr int kCells = kFarThreads / 64 * ROWS / 4;  // cells per workgroup
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t cell = int64_t(blockIdx.x) * kCells + wave * ROWS / 4;
    int64_t group, jh;
    if (hb >= 4) {  // workgroups b, b + 8, ... take the cells of one group
        const int64_t b = blockIdx.x, i = (b >> 3) * kCells + wave * ROWS / 4;
        group = ((i >> hb) << 3) | (b & 7);
        jh = i & ((int64_t(1) << hb) - 1);
    } else {
        group = cell >> hb;
        jh = cell & ((int64_t(1) << hb) - 1);
    }
    const int64_t kh = jh ^ group;
    const int64_t j0 = (jh << kFarLow) | (ROWS == 4 ? 0 : 4 * (wave & 3)) | (lane >> kFarLow);
    const int64_t k = (kh << kFarLow) | (lane & 15);
    const int64_t x0 = (j0 << Ls) | k, row4 = int64_t(4) << Ls;  // rows j0, j0 + 4, ...
    double2 acc[ROWS];
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
        const double* o = reinterpret_cast<const double*>(out + x0 + e * row4);
        acc[e] = make_double2(__builtin_nontemporal_load(o), __builtin_nontemporal_load(o + 1));
    }
    for (int f = 0; f < nterms; ++f) {
        const int p = terms[f].p;
        const uint32_t mask = terms[f].mask;
        const int64_t step = (int64_t(1) << p) | (int64_t(1) << (p + Ls));
        if (p >= kFarLow) {  // both bits are the cell's own: one row index r for the wave
            const int r = int((((jh >> (p - kFarLow)) & 1) << 1) | ((kh >> (p - kFarLow)) & 1));
            const uint32_t row = (mask >> (4 * r)) & 15u;
            if (!row) continue;
            const int64_t base = x0 & ~step;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if ((row >> c) & 1u) {
                    const double2* y = psi + (base | (int64_t(c >> 1) << (p + Ls)) | (int64_t(c & 1) << p));
                    const double2 kk = terms[f].K[4 * r + c];
                    double2 v[ROWS];
#pragma unroll
                    for (int e = 0; e < ROWS; ++e) v[e] = y[e * row4];
#pragma unroll
                    for (int e = 0; e < ROWS; ++e) {
                        acc[e].x = fma(kk.x, v[e].x, fma(-kk.y, v[e].y, acc[e].x));
                        acc[e].y = fma(kk.x, v[e].y, fma(kk.y, v[e].x, acc[e].y));
                    }
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < ROWS; ++e) {
                const int64_t x = x0 + e * row4;
                const int r = int((((x >> (p + Ls)) & 1) << 1) | ((x >> p) & 1));
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if ((mask >> (4 * r + c)) & 1u) {
                        const double2 v = psi[(x & ~step) | (int64_t(c >> 1) << (p + Ls)) | (int64_t(c & 1) << p)];
                        const double2 kk = terms[f].K[4 * r + c];
                        acc[e].x = fma(kk.x, v.x, fma(-kk.y, v.y, acc[e].x));
                        acc[e].y = fma(kk.x, v.y, fma(kk.y, v.x, acc[e].y));
                    }
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
        double* o = reinterpret_cast<double*>(out + x0 + e * row4);
        __builtin_nontemporal_store(acc[e].x, o);
        __builtin_nontemporal_store(acc[e].y, o + 1);
    }
}

// The same for a superket of fewer than 4 + 4 bits (Ls < 4): one entry per thread.
__global__ __launch_bounds__(kFarThreads) void far_terms_small(const double2* __restrict__ psi,
                                                               double2* __restrict__ out,
                                                               const FarTerm* __restrict__ terms, int nterms, int Ls) {
    const int64_t x = threadIdx.x;
    if (x >= int64_t(1) << (2 * Ls)) return;
    double2 acc = out[x];
    for (int f = 0; f < nterms; ++f) {
        const int p = terms[f].p, q = p + Ls;
        const int r = int((((x >> q) & 1) << 1) | ((x >> p) & 1));
        const int64_t base = x & ~((int64_t(1) << p) | (int64_t(1) << q));
        for (int c = 0; c < 4; ++c) {
            if ((terms[f].mask >> (4 * r + c)) & 1u) {
                const double2 v = psi[base | (int64_t(c >> 1) << q) | (int64_t(c & 1) << p)];
                const double2 kk = terms[f].K[4 * r + c];
                acc.x = fma(kk.x, v.x, fma(-kk.y, v.y, acc.x));
                acc.y = fma(kk.x, v.y, fma(kk.y, v.x, acc.y));
            }
        }
    }
    out[x] = acc;
}

// one workgroup: res[0] = sum_j Re rho_jj, res[k] = sum_j Re rho_jj z_k(j) (site k at bit Ls - k of
// j, z = +1 for bit 0), in a fixed order
__global__ __launch_bounds__(256) void superket_diag_kernel(const double2* __restrict__ rho, int Ls,
                                                            double2* __restrict__ res) {
    __shared__ double red[256];
    const int64_t D = int64_t(1) << Ls;
    const int t = threadIdx.x;
    double acc[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) acc[i] = 0.0;
    for (int64_t j = t; j < D; j += 256) {
        const double v = rho[j * (D + 1)].x;
        acc[0] += v;
#pragma unroll
        for (int b = 0; b < 31; ++b)
            if (b < Ls) acc[1 + b] += ((j >> b) & 1) ? -v : v;
    }
    for (int i = 0; i <= Ls; ++i) {
        red[t] = acc[0];
#pragma unroll
        for (int b = 0; b < 31; ++b)
            if (i == 1 + b) red[t] = acc[1 + b];
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (t < h) red[t] += red[t + h];
            __syncthreads();
        }
        // bit b = i - 1 is site Ls - b
        if (t == 0) res[i == 0 ? 0 : Ls - (i - 1)] = make_double2(red[0], 0.0);
        __syncthreads();
    }
}

}  // namespace

ed_status launch_far_terms(const ed_model* m, const double2* psi, double2* out, hipStream_t s) {
    const int Ls = m->lv_L, nt = int(m->far.size());
    const int64_t cells = int64_t(1) << (2 * std::max(Ls - kFarLow, 0));
    if (Ls < kFarLow) {
        hipLaunchKernelGGL(far_terms_small, dim3(1), dim3(kFarThreads), 0, s, psi, out, m->d_far, nt, Ls);
    } else if (Ls < 10) {
        hipLaunchKernelGGL(far_terms<1>, dim3(unsigned(cells)), dim3(kFarThreads), 0, s, psi, out, m->d_far, nt, Ls);
    } else {
        hipLaunchKernelGGL(far_terms<4>, dim3(unsigned(cells / 4)), dim3(kFarThreads), 0, s, psi, out, m->d_far, nt,
                           Ls);
    }
    ED_HIP_TRY(hipGetLastError());
    return ED_OK;
}

ed_status superket_diag(const double2* rho, int Ls, double2* res, hipStream_t s) {
    hipLaunchKernelGGL(superket_diag_kernel, dim3(1), dim3(256), 0, s, rho, Ls, res);
    ED_HIP_TRY(hipGetLastError());
    return ED_OK;
}

}  // namespace ed
