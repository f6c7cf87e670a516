// The Hermitian three-term recurrence of a Krylov time step (Sec. ed:sec:krylov) with its scalars on the
// device, so that iterations run back to back: the host reads them once per batch, not once per
// product.
//
// The basis is kept unnormalised: u_{j+1} = s_j (H u_j - a_j u_j - b_j u_{j-1}), with
//   a_j = <u_j|H u_j> / N_j,   b_j = N_j / (s_{j-1} N_{j-1})   (N_j = |u_j|^2; the second is the previous
// step's norm, for a Hermitian H), or b_j = <u_{j-1}|H u_j> / N_{j-1} where both projections are taken.
// So alpha_j = a_j and beta_j = sqrt(N_{j+1} / N_j) / s_j, and every coefficient of a sweep comes
// from device scalars that earlier kernels of the same stream wrote. s_j (kept in N[j+1].y) is the power
// of two that brings |u_{j+1}| near 1 if beta_j is near beta_{j-1}, and s_0 = 1 / |u_0| to a factor of two.
// Scaling by it is exact. One factor for all steps, from a bound of |H|, would not do: the bound can be
// far above every beta (a uniform field that only turns the phase), and the norms then underflow.
#include <algorithm>
#include <cfloat>
#include <cmath>

#include "ed_vec.h"
#include "hpsi_device.h"
#include "krylov_core.h"

namespace ed {
namespace {

constexpr int kThr = 256;
constexpr int kSmallThr = 1024;
constexpr int kSmallBits = 12;          // one workgroup holds a state of up to 2^12 amplitudes
constexpr int kSmallAmps = (1 << kSmallBits) / kSmallThr;
constexpr int kTicketBlocks = 1024;     // sweeps of at most this many workgroups reduce in their own launch
constexpr int kTickets = 32;            // leaf counters of a sweep (and one root)
constexpr int kTicketStride = 16;       // unsigneds between counters: 64 bytes
constexpr int kOwnParts = 1024;         // per-tile partials that every workgroup of a sweep sums for itself

// floor(log2 v) of a positive normal v (-1023 for zero and subnormals, 1024 for infinity and NaN)
__device__ __forceinline__ int exponent_of(double v) {
    return int((__double_as_longlong(v) >> 52) & 0x7ff) - 1023;
}

// s_j from N_j and, past the first step, N_{j-1} and s_{j-1}: |H u_j - ...| is about beta_{j-1} sqrt(N_j) =
// N_j / (s_{j-1} sqrt(N_{j-1})).
__device__ __forceinline__ double step_scale(int j, double nj, double nm, double sm) {
    const int k = j == 0 ? -(exponent_of(nj) >> 1) : exponent_of(sm) - exponent_of(nj) + (exponent_of(nm) >> 1);
    return __longlong_as_double(static_cast<long long>(min(max(k, -1000), 1000) + 1023) << 52);
}

// Sums of NA values over a workgroup of W waves; every thread receives them (fixed order).
template <int NA, int W>
__device__ __forceinline__ void group_sums(double (&a)[NA], double (*lds)[NA]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) a[i] += __shfl_xor(a[i], o, 64);
    }
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) lds[wv][i] = a[i];
    }
    __syncthreads();
    // every W lanes of a wave add the W waves' sums by the same butterfly
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        a[i] = lds[lane & (W - 1)][i];
#pragma unroll
        for (int o = W / 2; o > 0; o >>= 1) a[i] += __shfl_xor(a[i], o, 64);
    }
    __syncthreads();
}

// End of a sweep: out[0..NA) = the sum over all workgroups of a[0..NA) (each thread holds its
// workgroup's sums). With a ticket the last workgroup to arrive adds all of them in workgroup
// order: the partials are agent-scope stores that have completed before their workgroup's ticket,
// and agent-scope loads. Arrivals count on one of 32 leaf counters, and the last of a leaf on the root:
// about 10 ns per arrival on one counter made a sweep of 1024 workgroups 10 us longer. Without a ticket
// (many workgroups) the partials stay in part for a reduction launch.
template <int NA>
__device__ __forceinline__ void sweep_sums(const double (&a)[NA], double* part, unsigned* ticket, double* out) {
    __shared__ int last;
    __shared__ double lds[kThr / 64][NA];
    const int t = threadIdx.x;
    if (t == 0) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
            __hip_atomic_store(part + int64_t(blockIdx.x) * NA + i, a[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = 0;
        if (ticket) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const unsigned G = gridDim.x, leaf = blockIdx.x % kTickets;
            const unsigned leaves = G < kTickets ? G : kTickets;
            const unsigned members = (G - leaf + kTickets - 1) / kTickets;  // workgroups b with b % 32 == leaf
            unsigned* lc = ticket + (1 + leaf) * kTicketStride;
            if (__hip_atomic_fetch_add(lc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == members - 1) {
                __hip_atomic_store(lc, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == leaves - 1;
            }
        }
    }
    __syncthreads();
    if (!last) return;
    double s[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) s[i] = 0.0;
    for (int b = t; b < int(gridDim.x); b += kThr) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
            s[i] += __hip_atomic_load(part + int64_t(b) * NA + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    group_sums<NA, kThr / 64>(s, lds);
    if (t == 0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) out[i] = s[i];
        __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ __launch_bounds__(kSmallThr) void zero_words(unsigned* p, int n) {
    if (int(threadIdx.x) < n) p[threadIdx.x] = 0u;
}

// out[i] = sum over rows b of part[b * n + i], workgroup i (fixed order)
__global__ __launch_bounds__(kSmallThr) void sum_rows(const double* __restrict__ part, int64_t rows, int n,
                                                      double* __restrict__ out) {
    __shared__ double lds[kSmallThr / 64][1];
    double s[1] = {0.0};
    for (int64_t b0 = threadIdx.x; b0 < rows; b0 += 8 * kSmallThr) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t b = b0 + u * kSmallThr;
            v[u] = b < rows ? part[b * n + blockIdx.x] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s[0] += v[u];
    }
    group_sums<1, kSmallThr / 64>(s, lds);
    if (threadIdx.x == 0) out[blockIdx.x] = s[0];
}

// N[0] = |src|^2, and dst = src where dst is given
__global__ __launch_bounds__(kThr) void start_sweep(const double2* __restrict__ src, double2* __restrict__ dst,
                                                    int64_t D, double* part, unsigned* ticket, double* out) {
    __shared__ double lds[kThr / 64][1];
    double a[1] = {0.0};
    const int64_t stride = int64_t(gridDim.x) * kThr;
    for (int64_t x = int64_t(blockIdx.x) * kThr + threadIdx.x; x < D; x += stride) {
        const double2 v = src[x];
        if (dst) dst[x] = v;
        a[0] = fma(v.x, v.x, fma(v.y, v.y, a[0]));
    }
    group_sums<1, kThr / 64>(a, lds);
    sweep_sums<1>(a, part, ticket, out);
}

struct SubArgs {
    const double2* um1;  // null for j = 0
    const double2* u;
    double2* y;
    int64_t D;
    double2 *N, *SP;  // N_j in N[j].x, s_{j-1} in N[j].y; SP[2 j] = <u_j|y>, SP[2 j + 1] = <u_{j-1}|y>
    int j, both;
    const double2* tiles;  // per-tile partials of <u_j|y> (and <u_{j-1}|y>), or null: SP holds the sums
    int ntiles;
    double* part;
    unsigned* ticket;
};

// y <- u_{j+1} in place, N_{j+1}. Bound by memory: 64 B per amplitude (13 us at L = 20, in the last-level
// cache). Up to kOwnParts per-tile partials of the product's projection are summed by every workgroup
// for itself, which costs less than a reduction launch (5 us).
template <bool NT>
__global__ __launch_bounds__(kThr) void three_term_sub(SubArgs A) {
    __shared__ double lds[kThr / 64][4];
    __shared__ double lds1[kThr / 64][1];
    const int t = threadIdx.x;
    // the norms come from HBM (another workgroup wrote them): asked for before the tiles are summed
    const double2 Nj = A.N[A.j], Nm = A.N[A.um1 ? A.j - 1 : A.j];
    double p[4] = {0.0, 0.0, 0.0, 0.0};
    if (A.tiles) {
        const int st = A.both ? 2 : 1;
        for (int b = t; b < A.ntiles; b += kThr) {
            const double2 v = A.tiles[b * st];
            p[0] += v.x;
            p[1] += v.y;
            if (A.both) {
                const double2 q = A.tiles[b * st + 1];
                p[2] += q.x;
                p[3] += q.y;
            }
        }
        group_sums<4, kThr / 64>(p, lds);
        if (blockIdx.x == 0 && t == 0) {
            A.SP[2 * A.j] = make_double2(p[0], p[1]);
            if (A.both) A.SP[2 * A.j + 1] = make_double2(p[2], p[3]);
        }
    } else {
        p[0] = A.SP[2 * A.j].x;
        p[1] = A.SP[2 * A.j].y;
        if (A.both) {
            p[2] = A.SP[2 * A.j + 1].x;
            p[3] = A.SP[2 * A.j + 1].y;
        }
    }
    const double nj = Nj.x, nm = Nm.x, sm = Nj.y;
    const double2 a = make_double2(p[0] / nj, p[1] / nj);
    double2 b = make_double2(0.0, 0.0);
    if (A.um1) b = A.both ? make_double2(p[2] / nm, p[3] / nm) : make_double2(nj / (sm * nm), 0.0);
    const double sj = step_scale(A.j, nj, nm, sm);
    if (blockIdx.x == 0 && t == 0) A.N[A.j + 1].y = sj;
    double n2[1] = {0.0};
    const int64_t chunk = (A.D + gridDim.x - 1) / gridDim.x;
    const int64_t lo = int64_t(blockIdx.x) * chunk;
    const int64_t hi = lo + chunk < A.D ? lo + chunk : A.D;
    constexpr int U = 4;
    for (int64_t x0 = lo + t; x0 < hi; x0 += U * kThr) {
        double2 y[U], v[U], w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t x = x0 + u * kThr < hi ? x0 + u * kThr : x0;
            y[u] = A.y[x];
            v[u] = load_vec<NT>(A.u + x);
            w[u] = A.um1 ? load_vec<NT>(A.um1 + x) : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (x0 + u * kThr >= hi) continue;
            double2 r = y[u];
            r.x -= a.x * v[u].x - a.y * v[u].y;
            r.y -= a.x * v[u].y + a.y * v[u].x;
            r.x -= b.x * w[u].x - b.y * w[u].y;
            r.y -= b.x * w[u].y + b.y * w[u].x;
            r.x *= sj;
            r.y *= sj;
            A.y[x0 + u * kThr] = r;
            n2[0] = fma(r.x, r.x, fma(r.y, r.y, n2[0]));
        }
    }
    group_sums<1, kThr / 64>(n2, lds1);
    sweep_sums<1>(n2, A.part, A.ticket, &A.N[A.j + 1].x);
}

struct SmallArgs {
    const double2* lr;  // long-range zz energy per basis state, or null
    int L, both;
    const double2* u0;
    double2* V;  // basis slots: u_j is slot j, but u_0 is u0
    int64_t D;
    double2 *N, *SP;
    int j0, nj;
};

// Iterations j0 .. j0 + nj - 1 for a state of at most 2^12 amplitudes in one workgroup: u_j sits in
// LDS, every other vector of the iteration in registers (up to four amplitudes per thread; the
// diagonal too, which all iterations share). Bound by latency: an iteration is one product from LDS and
// two workgroup sums, about 8 us for the XXZ chain at L = 12 (a ten-step quench: 1.63 ms), against 45 us
// in separate launches with a round trip each (4.79 ms).
template <unsigned CLS>
__global__ __launch_bounds__(kSmallThr) void three_term_small(SmallArgs A, const double2* __restrict__ site,
                                                              const double2* __restrict__ bond) {
    constexpr bool OFFR = CLS & kOffReal;
    constexpr int E = kSmallAmps;
    __shared__ double2 s[1 << kSmallBits];
    __shared__ double lds[kSmallThr / 64][4];
    __shared__ double lds1[kSmallThr / 64][1];
    const int t = threadIdx.x, D = int(A.D), L = A.L;
    double2 u[E], um1[E], diag[E];
    double nj, nm = 1.0, sm = 1.0;
    {
        const double2* src = A.j0 == 0 ? A.u0 : A.V + int64_t(A.j0) * A.D;
        const double2* prev = A.j0 == 1 ? A.u0 : A.V + int64_t(A.j0 - 1) * A.D;
        double n2[1] = {0.0};
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int x = (t + e * kSmallThr) & (D - 1);
            u[e] = src[x];
            um1[e] = A.j0 > 0 ? prev[x] : make_double2(0.0, 0.0);
            diag[e] = A.lr ? A.lr[x] : make_double2(0.0, 0.0);
        }
        // the diagonal; the loads of three bits of all amplitudes are issued together
        for (int p0 = 0; p0 < L; p0 += 3) {
            double2 ds[3][E], db[3][E];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int ps = p0 + k < L ? p0 + k : 0, pb = p0 + k + 1 < L ? p0 + k : 0;
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int x = (t + e * kSmallThr) & (D - 1);
                    ds[k][e] = site[4 * ps + 3 * ((x >> ps) & 1)];
                    db[k][e] = bond[16 * pb + 5 * ((x >> pb) & 3)];
                }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    if (p0 + k < L) {
                        diag[e].x += ds[k][e].x;
                        diag[e].y += ds[k][e].y;
                    }
                    if (p0 + k + 1 < L) {
                        diag[e].x += db[k][e].x;
                        diag[e].y += db[k][e].y;
                    }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int x = t + e * kSmallThr;
            if (x < D) {
                s[x] = u[e];
                n2[0] = fma(u[e].x, u[e].x, fma(u[e].y, u[e].y, n2[0]));
            } else {  // a place beyond the state: zero in every vector
                u[e] = um1[e] = diag[e] = make_double2(0.0, 0.0);
            }
        }
        if (A.j0 == 0) {
            group_sums<1, kSmallThr / 64>(n2, lds1);
            nj = n2[0];
            if (t == 0) A.N[0] = make_double2(nj, 0.0);
        } else {
            nj = A.N[A.j0].x;
            nm = A.N[A.j0 - 1].x;
            sm = A.N[A.j0].y;
            __syncthreads();
        }
    }
    for (int j = A.j0; j < A.j0 + A.nj; ++j) {
        double2 y[E];
#pragma unroll
        for (int e = 0; e < E; ++e) y[e] = cmul(diag[e], u[e]);
        // (unrolled over the bits, the LDS addresses of all flips stayed live and went to scratch memory)
#pragma unroll 1
        for (int p = 0; p < L; ++p) {
            if (CLS & kSiteOff) {
                const double2 c01 = site[4 * p + 1], c10 = site[4 * p + 2];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int x = t + e * kSmallThr;
                    cfma<OFFR>(y[e], sel2((x >> p) & 1, c01, c10), s[(x & (D - 1)) ^ (1 << p)]);
                }
            }
            if ((CLS & (kBondSingle | kBondDouble)) && p + 1 < L) {
                const double2* B = bond + 16 * p;
#pragma unroll
                for (int m = 1; m < 4; ++m) {
                    if (!(CLS & (m == 3 ? kBondDouble : kBondSingle))) continue;
                    const double2 b0 = B[0 + (0 ^ m)], b1 = B[4 + (1 ^ m)], b2 = B[8 + (2 ^ m)], b3 = B[12 + (3 ^ m)];
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const int x = t + e * kSmallThr;
                        cfma<OFFR>(y[e], sel4((x >> p) & 3, b0, b1, b2, b3), s[(x & (D - 1)) ^ (m << p)]);
                    }
                }
            }
        }
        double p[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < E; ++e) {
            p[0] = fma(u[e].x, y[e].x, fma(u[e].y, y[e].y, p[0]));
            p[1] = fma(u[e].x, y[e].y, fma(-u[e].y, y[e].x, p[1]));
            if (A.both) {
                p[2] = fma(um1[e].x, y[e].x, fma(um1[e].y, y[e].y, p[2]));
                p[3] = fma(um1[e].x, y[e].y, fma(-um1[e].y, y[e].x, p[3]));
            }
        }
        group_sums<4, kSmallThr / 64>(p, lds);  // (its first barrier also ends the reads of s)
        const double2 a = make_double2(p[0] / nj, p[1] / nj);
        double2 b = make_double2(0.0, 0.0);
        if (j > 0) b = A.both ? make_double2(p[2] / nm, p[3] / nm) : make_double2(nj / (sm * nm), 0.0);
        sm = step_scale(j, nj, nm, sm);
        double n2[1] = {0.0};
        double2* out = A.V + int64_t(j + 1) * A.D;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int x = t + e * kSmallThr;
            double2 r = x < D ? y[e] : make_double2(0.0, 0.0);
            r.x -= a.x * u[e].x - a.y * u[e].y;
            r.y -= a.x * u[e].y + a.y * u[e].x;
            r.x -= b.x * um1[e].x - b.y * um1[e].y;
            r.y -= b.x * um1[e].y + b.y * um1[e].x;
            r.x *= sm;
            r.y *= sm;
            n2[0] = fma(r.x, r.x, fma(r.y, r.y, n2[0]));
            um1[e] = u[e];
            u[e] = r;
            if (x < D) {
                out[x] = r;
                s[x] = r;
            }
        }
        group_sums<1, kSmallThr / 64>(n2, lds1);
        nm = nj;
        nj = n2[0];
        if (t == 0) {
            A.SP[2 * j] = make_double2(p[0], p[1]);
            A.SP[2 * j + 1] = make_double2(p[2], p[3]);
            A.N[j + 1] = make_double2(nj, sm);
        }
    }
}

// psi = sum_i c_i u_i over the first n basis vectors, in place on u_0 = psi, and its observables:
// res[0] = |psi|^2, res[1 + p] = sum |psi_x|^2 (1 - 2 bit_p(x)) (p = bit); one workgroup.
struct SmallComb {
    const double2* V;
    double2* psi;
    int64_t D;
    int L, n;
    double2* res;
    double2 c[kMaxComb];
};

__global__ __launch_bounds__(kSmallThr) void combine_measure_small(SmallComb A) {
    constexpr int NA = kSmallBits + 1;
    __shared__ double lds[kSmallThr / 64][NA];
    const int t = threadIdx.x, D = int(A.D);
    constexpr int E = kSmallAmps, H = 4;  // 16 loads in flight: amplitudes times vectors
    double2 r[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int x = t + e * kSmallThr;
        const double2 v = x < D ? A.psi[x] : make_double2(0.0, 0.0);
        r[e] = make_double2(A.c[0].x * v.x - A.c[0].y * v.y, A.c[0].x * v.y + A.c[0].y * v.x);
    }
    for (int i0 = 1; i0 < A.n; i0 += H) {
        double2 v[H][E];
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int x = t + e * kSmallThr;
                v[h][e] = A.V[int64_t(i0 + h < A.n ? i0 + h : i0) * A.D + (x < D ? x : 0)];
            }
#pragma unroll
        for (int h = 0; h < H; ++h)
            if (i0 + h < A.n) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    r[e].x = fma(A.c[i0 + h].x, v[h][e].x, fma(-A.c[i0 + h].y, v[h][e].y, r[e].x));
                    r[e].y = fma(A.c[i0 + h].x, v[h][e].y, fma(A.c[i0 + h].y, v[h][e].x, r[e].y));
                }
            }
    }
    double a[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) a[i] = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int x = t + e * kSmallThr;
        if (x >= D) continue;
        A.psi[x] = r[e];
        const double q = fma(r[e].x, r[e].x, r[e].y * r[e].y);
        a[0] += q;
#pragma unroll
        for (int p = 10; p < kSmallBits; ++p) a[1 + p] += ((x >> p) & 1) ? -q : q;
    }
    // bits 0..9 are the thread's: its sign for the sum of its amplitudes
#pragma unroll
    for (int p = 0; p < 10; ++p) a[1 + p] = ((t >> p) & 1) ? -a[0] : a[0];
    group_sums<NA, kSmallThr / 64>(a, lds);
    if (t == 0) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
            if (i <= A.L) A.res[i] = make_double2(a[i], 0.0);
    }
}

template <int I>
hipError_t launch_small(unsigned cls, const SmallArgs& a, const double2* site, const double2* bond, hipStream_t s) {
    if constexpr (I >= kNumVariants) {
        return hipErrorInvalidValue;
    } else {
        if (variant_fits(kVariants[I], cls)) {
            hipLaunchKernelGGL((three_term_small<kVariants[I]>), dim3(1), dim3(kSmallThr), 0, s, a, site, bond);
            return hipGetLastError();
        }
        return launch_small<I + 1>(cls, a, site, bond, s);
    }
}

unsigned sweep_blocks(int64_t D) {
    return unsigned(std::max<int64_t>(1, std::min<int64_t>(D / (4 * kThr), kRedBlocks)));
}

#define ED_L(expr)                                                                                        \
    do {                                                                                                  \
        hipError_t _e = (expr);                                                                           \
        if (_e != hipSuccess) return fail(ED_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(_e)); \
    } while (0)

}  // namespace

ed_status three_term_beta(const double2* N, int j, double hmax, double* beta, bool* brk) {
    const double n1 = std::max(N[j + 1].x, 0.0);
    *beta = std::sqrt(n1) / std::sqrt(N[j].x) / N[j + 1].y;
    *brk = *beta <= 1e-14 * std::max(hmax, 1e-300) || *beta == 0.0;
    if (!*brk && n1 < DBL_MIN) return fail(ED_ERR_NUMERIC, "a vector of the Krylov recurrence underflows");
    return ED_OK;
}

ed_status three_term_init(const Workspace& w, int mmax, ThreeTerm* T, hipStream_t s) {
    if (mmax > kThreeTermMax || kThreeTermFree + 3 * mmax + 2 > kObs) return fail(ED_ERR_UNSUPPORTED, "basis too large for device scalars");
    T->mmax = mmax;
    T->N = w.scal + kObs - T->count();
    T->SP = T->N + mmax + 2;
    static_assert((kTickets + 1) * kTicketStride * sizeof(unsigned) <= kThreeTermFree * sizeof(double2), "scalar area");
    T->ticket = reinterpret_cast<unsigned*>(w.scal);
    hipLaunchKernelGGL(zero_words, dim3(1), dim3(kSmallThr), 0, s, T->ticket, (kTickets + 1) * kTicketStride);
    ED_L(hipGetLastError());
    return ED_OK;
}

ed_status three_term_start(const ThreeTerm& T, const Workspace& w, const double2* psi, bool alias, bool have_norm,
                           hipStream_t s) {
    w.u.resize(std::max<size_t>(w.u.size(), size_t(T.mmax) + 1));
    w.c.resize(w.u.size());
    w.u[0] = alias ? const_cast<double2*>(psi) : w.slot(0);
    for (int i = 1; i <= T.mmax; ++i) w.u[i] = w.slot(i);
    if (w.D <= (int64_t(1) << kSmallBits) && alias) return ED_OK;  // the small kernel takes the norm itself
    if (have_norm && alias) return ED_OK;
    const unsigned G = sweep_blocks(w.D);
    const bool one = G <= unsigned(kTicketBlocks);
    double* part = reinterpret_cast<double*>(w.part);
    hipLaunchKernelGGL(start_sweep, dim3(G), dim3(kThr), 0, s, psi, alias ? nullptr : w.slot(0), w.D, part,
                       one ? T.ticket : nullptr, &T.N[0].x);
    if (!one) hipLaunchKernelGGL(sum_rows, dim3(1), dim3(kSmallThr), 0, s, part, int64_t(G), 1, &T.N[0].x);
    ED_L(hipGetLastError());
    return ED_OK;
}

bool three_term_small_fits(const ed_model* m) { return m->L <= kSmallBits; }

ed_status three_term_combine_small(const Workspace& w, int L, int n, const double2* c, double2* psi, double2* res,
                                   hipStream_t s) {
    SmallComb a;
    a.V = w.V;
    a.psi = psi;
    a.D = w.D;
    a.L = L;
    a.n = n;
    a.res = res;
    for (int i = 0; i < kMaxComb; ++i) a.c[i] = i < n ? c[i] : make_double2(0.0, 0.0);
    hipLaunchKernelGGL(combine_measure_small, dim3(1), dim3(kSmallThr), 0, s, a);
    ED_L(hipGetLastError());
    return ED_OK;
}

ed_status three_term_run(const ed_model* m, const ThreeTerm& T, const Workspace& w, int j0, int nj, bool both,
                         hipStream_t s) {
    const int64_t D = w.D;
    if (m->L <= kSmallBits) {
        SmallArgs a;
        a.lr = m->lr ? m->d_lr_low : nullptr;
        a.L = m->L;
        a.both = both ? 1 : 0;
        a.u0 = w.u[0];
        a.V = w.V;
        a.D = D;
        a.N = T.N;
        a.SP = T.SP;
        a.j0 = j0;
        a.nj = nj;
        ED_L(launch_small<0>(m->op_class, a, m->d_site, m->d_bond, s));
        return ED_OK;
    }
    const unsigned G = sweep_blocks(D);
    const bool one = G <= unsigned(kTicketBlocks);
    for (int j = j0; j < j0 + nj; ++j) {
        SubArgs a;
        a.um1 = j > 0 ? w.u[j - 1] : nullptr;
        a.u = w.u[j];
        a.y = w.u[j + 1];
        a.D = D;
        a.N = T.N;
        a.SP = T.SP;
        a.j = j;
        a.both = both && j > 0 ? 1 : 0;
        a.tiles = nullptr;
        a.ntiles = 0;
        // the product's projections per tile may fill the partial buffer (2^30 amplitudes do); the sweep's
        // partials take their place, or the buffer's end where the sweep itself reads the projections
        constexpr int64_t room = int64_t(kPartBytes / sizeof(double2));
        static_assert(2 * kOwnParts + kRedBlocks <= room, "partial buffer");
        a.part = reinterpret_cast<double*>(w.part);
        a.ticket = one ? T.ticket : nullptr;
        int64_t nparts = 0;
        ED_TRY(launch_apply_H_dot(m, a.u, a.y, w.part, room / (a.both ? 2 : 1), &nparts, s, a.both ? a.um1 : nullptr));
        if (nparts > 0 && nparts <= kOwnParts) {
            a.tiles = w.part;
            a.ntiles = int(nparts);
            a.part = reinterpret_cast<double*>(w.part + room - kRedBlocks);
        } else if (nparts > 0) {
            const int n = a.both ? 4 : 2;  // doubles per tile
            hipLaunchKernelGGL(sum_rows, dim3(unsigned(n)), dim3(kSmallThr), 0, s,
                               reinterpret_cast<const double*>(w.part), nparts, n,
                               reinterpret_cast<double*>(T.SP + 2 * j));
        } else {
            ED_L(dots_ptr(const_cast<const double2* const*>(&w.u[j]), 1, a.y, D, T.SP + 2 * j, w.part, s));
            if (a.both)
                ED_L(dots_ptr(const_cast<const double2* const*>(&w.u[j - 1]), 1, a.y, D, T.SP + 2 * j + 1, w.part, s));
        }
        hipLaunchKernelGGL(outgrows_cache(3, w.D) ? three_term_sub<true> : three_term_sub<false>, dim3(G), dim3(kThr), 0, s, a);
        if (!one) hipLaunchKernelGGL(sum_rows, dim3(1), dim3(kSmallThr), 0, s, a.part, int64_t(G), 1, &T.N[j + 1].x);
        ED_L(hipGetLastError());
    }
    return ED_OK;
}

}  // namespace ed
