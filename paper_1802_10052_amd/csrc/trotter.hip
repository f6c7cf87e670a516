// Suzuki-Trotter time evolution (Sec. ed:sec:trotter: Eqs. ed:eq:trotter1, ed:eq:trotter2,
// ed:eq:trotter4, constants Eq. ed:eq:trotter4c).
//
// H = H_o + H_e with H_o the bond terms (k, k+1) for odd k (1-based sites) and H_e those for even
// k; each site's terms are shared by the bonds that contain it (1/2 each, 1 for a site in a single
// bond). A layer exp(-i t H_o) (or H_e) is the product of the commuting two-site propagators
// exp(-i t h_k); the paper contracts each with two legs of the rank-L state tensor (tensordot plus
// a permutation). Here runs of kFuse consecutive layers stream the state through LDS tiles in a
// few in-place passes (the 12 low bits, then windows of 8 high bits above 4 contiguous low bits):
// a pass applies its gates layer by layer, and each gate goes to the first pass whose tile holds
// both of its bits and in which every gate of an earlier layer that shares one of its bits has
// already been applied (in an earlier pass, or earlier in the same pass). Gates of one layer act
// on disjoint bits and commute, so this keeps the order of the product wherever it matters; a
// tile is read completely before it is written, and tiles of a pass are disjoint, so the passes
// work in place.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "dense.h"
#include "ed_vec.h"
#include "krylov_core.h"

namespace ed {
namespace {

constexpr int kGTileBits = 12;
constexpr int kGThreads = 256;                           // 16 amplitudes (4 tile bits) per thread
constexpr int kGRegBits = 4;
constexpr int kGSlots = 1 << kGRegBits;
constexpr int kSmallThreads = 512;                       // tiles of fewer than 12 bits
constexpr int kGLow = 4;                                 // contiguous low bits of a window tile
constexpr int kFuse = 4;                                 // consecutive layers per run of passes
constexpr int kTableGates = 192;                         // gates one evolve call holds
// the gate table: 16 double2 (the matrix) per gate, then 2 ints per gate: the gates' codes, and as
// many slots for the rounds of all passes (a round holds a gate, or is one of a pass's two staging
// rounds, and a pass holds more rounds than one)
constexpr int kTableRounds = kTableGates;
constexpr size_t kGateTableBytes = size_t(kTableGates) * 16 * sizeof(double2) +
                                   size_t(kTableGates + kTableRounds) * sizeof(int);

// One pass: tile geometry and its gates, sorted by round, in device memory. Gate g of the pass maps
// the local pair index l = 2 bit(q+1) + bit(q) of the tile bits (q, q+1) (bit q+1 is the left site
// of the bond) by the 4x4 matrix U[16 g + 4 l + m]; its code G[g] is q, or for a 12-bit tile
// 1 << (q - a) of its round a, times kCross when the matrix couples 00 only with 11 and 01 only with
// 10. A round r of
// a 12-bit tile (code R[r]) holds the tile bits a..a+3 of 16 amplitudes in the registers of a
// thread and applies gates g0..g1-1 to them.
struct GatePass {
    int first;   // contiguous tile of the tbits low bits
    int c, h0;   // window tile: c low bits, window bits [h0, h0 + tbits - c)
    int tbits;   // tile bits (min(L, 12))
    int ngate;
    int nround;
    const double2* U;
    const int* G;
    const int* R;
};

constexpr int kCross = 8;
__host__ __device__ constexpr int round_code(int a, int g0, int g1) { return a | (g0 << 8) | (g1 << 18); }

// a = u a + c in a's own register (u uniform). Left to itself the compiler accumulates into c and
// copies every result back: 32 copies per gate beside its 256 multiply-adds.
__device__ __forceinline__ void fma_into(double& a, double u, double c) {
    asm("v_fma_f64 %0, %1, %0, %2" : "+v"(a) : "s"(u), "v"(c));
}

// One gate on register bits (R, R+1): slots k, k | 1 << R, k | 2 << R, k | 3 << R hold the pair
// indices l = 0..3 of one group (compile-time slot indices keep v in registers).
template <int R, bool CROSS>
__device__ __forceinline__ void reg_gate(double2 (&v)[kGSlots], const double2* __restrict__ U) {
    static_assert(R + 2 <= kGRegBits, "gate bits beyond the register slots");
#pragma unroll
    for (int k = 0; k < kGSlots; ++k) {
        if (((k >> R) & 3) != 0) continue;
        const double2 a[4] = {v[k], v[k | (1 << R)], v[k | (2 << R)], v[k | (3 << R)]};
        // the diagonal's real part last, into the amplitude's own register
        double2 acc[4];
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const double ui = U[5 * l].y;
            acc[l] = make_double2(-ui * a[l].y, ui * a[l].x);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                if (m == l || (CROSS && m != 3 - l)) continue;
                const double2 u = U[4 * l + m];
                acc[l].x = fma(u.x, a[m].x, fma(-u.y, a[m].y, acc[l].x));
                acc[l].y = fma(u.x, a[m].y, fma(u.y, a[m].x, acc[l].y));
            }
        }
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            fma_into(v[k | (l << R)].x, U[5 * l].x, acc[l].x);
            fma_into(v[k | (l << R)].y, U[5 * l].x, acc[l].y);
        }
    }
}

// LDS position of tile index i (doubles): the low five bits take the XOR of bits 4..8, so that 32
// neighbouring lanes hit 32 different 8-byte columns whatever four bits the registers hold
// (without it, a round on bits below 4 puts all lanes on one column).
__host__ __device__ constexpr int swz(int i) { return i ^ ((i >> 4) & 15) ^ ((i >> 4) & 16); }

// swz is linear over XOR: slot m of a round at bit a sits at swz(slot 0) ^ swz(m << a), the second
// part the same for all threads (scalar, in bytes)
__device__ __forceinline__ unsigned slot_bytes(int m, int a) {
    return unsigned(__builtin_amdgcn_readfirstlane(swz(m << a) * 8));
}
__device__ __forceinline__ double* lds_at(double* s, unsigned bytes) {
    return reinterpret_cast<double*>(reinterpret_cast<char*>(s) + bytes);
}

// A pass over 12-bit tiles. What a gate costs is FP64 arithmetic (16 complex multiply-adds per group
// of four amplitudes), a trip of the tile through LDS, and its share of the pass's trip through
// HBM. Holding four tile bits in registers lets a round apply the gates of up to three layers on
// those bits (three on average) for one LDS trip; the trip between two rounds goes component by
// component, so a tile takes 32 KiB of LDS and four tiles of 256 threads share a CU, one's loads and
// LDS trips under the others' arithmetic. The first round's registers are filled straight from
// the state and the last round's go straight back (their bits are above the low four, so 16 lanes
// cover 256 contiguous bytes).
// L = 27 TFIM, order 4 (14 passes, 143 gates): 16.4 ms per step, 23.5 ms with one gate per LDS trip;
// windows of 8 to 12 gates take 0.85-0.93 ms (4.6-5.0 TB/s), the low tiles' 16 to 20 gates
// 1.6-1.9 ms (FP64-bound). Measured besides: whole amplitudes through 64 KiB of LDS, two tiles per CU
// (16.8 ms); 512 threads of 8 amplitudes (17.9 ms).
__global__ __launch_bounds__(kGThreads) __attribute__((amdgpu_waves_per_eu(4)))
void gate_pass(double2* __restrict__ psi, GatePass gp, const double2* __restrict__ Utab, const int* __restrict__ G,
               const int* __restrict__ R) {
    __shared__ double s[1 << kGTileBits];
    const int t = threadIdx.x;
    const int64_t n = blockIdx.x;
    // global index of tile index i: base + (i & 15) + (i >> 4) << hs, for either geometry
    int64_t base;
    int hs;
    if (gp.first) {
        base = n << kGTileBits;
        hs = kGLow;
    } else {
        const int lo_bits = gp.h0 - gp.c;
        const int64_t nlo = n & ((int64_t(1) << lo_bits) - 1), nhi = n >> lo_bits;
        base = (nlo << gp.c) | (nhi << (gp.h0 + kGTileBits - gp.c));
        hs = gp.h0;
    }
    double2 v[kGSlots];
    for (int r = 0; r < gp.nround; ++r) {
        const int code = R[r];
        const int a = code & 255, g0 = (code >> 8) & 1023, g1 = code >> 18;
        const int b = (t & ((1 << a) - 1)) | ((t >> a) << (a + kGRegBits));  // slot 0 of this thread
        if (r == 0) {  // a >= kGLow
            const double2* p = psi + base + ((int64_t(b >> kGLow) << hs) | (b & ((1 << kGLow) - 1)));
            const int64_t st = int64_t(1) << (hs + a - kGLow);
#pragma unroll
            for (int m = 0; m < kGSlots; ++m) v[m] = p[m * st];
        }
        for (int g = g0; g < g1; ++g) {
            const double2* U = Utab + 16 * g;
            // one bit per body, tested one after the other (a switch, or tests that the compiler can
            // prove exclusive, made it copy all slots after every gate)
            const int code = G[g];
            if (code & 1) reg_gate<0, false>(v, U);
            if (code & 2) reg_gate<1, false>(v, U);
            if (code & 4) reg_gate<2, false>(v, U);
            if (code & (kCross << 0)) reg_gate<0, true>(v, U);
            if (code & (kCross << 1)) reg_gate<1, true>(v, U);
            if (code & (kCross << 2)) reg_gate<2, true>(v, U);
        }
        if (r + 1 == gp.nround) {  // a >= kGLow
            double2* p = psi + base + ((int64_t(b >> kGLow) << hs) | (b & ((1 << kGLow) - 1)));
            const int64_t st = int64_t(1) << (hs + a - kGLow);
#pragma unroll
            for (int m = 0; m < kGSlots; ++m) p[m * st] = v[m];
        } else {
            // to the next round's slots; a thread writes only positions that it read itself last, so no
            // barrier is needed before the first write
            const int a2 = R[r + 1] & 255;
            const int b2 = (t & ((1 << a2) - 1)) | ((t >> a2) << (a2 + kGRegBits));
            const unsigned pb = unsigned(swz(b)) * 8u, pb2 = unsigned(swz(b2)) * 8u;
#pragma unroll
            for (int m = 0; m < kGSlots; ++m) *lds_at(s, pb ^ slot_bytes(m, a)) = v[m].x;
            __syncthreads();
#pragma unroll
            for (int m = 0; m < kGSlots; ++m) v[m].x = *lds_at(s, pb2 ^ slot_bytes(m, a2));
            __syncthreads();
#pragma unroll
            for (int m = 0; m < kGSlots; ++m) *lds_at(s, pb ^ slot_bytes(m, a)) = v[m].y;
            __syncthreads();
#pragma unroll
            for (int m = 0; m < kGSlots; ++m) v[m].y = *lds_at(s, pb2 ^ slot_bytes(m, a2));
        }
    }
}

// A chain of fewer than 12 sites is one tile in one workgroup: latency counts, so every gate spreads
// its groups of four over 512 threads, in list order (by layer).
__global__ __launch_bounds__(kSmallThreads) void gate_pass_small(double2* __restrict__ psi, GatePass gp,
                                                                 const double2* __restrict__ Utab,
                                                                 const int* __restrict__ G) {
    __shared__ double2 s[1 << (kGTileBits - 1)];
    const int t = threadIdx.x;
    const int N = 1 << gp.tbits;
    for (int i = t; i < N; i += kSmallThreads) s[i] = psi[i];
    __syncthreads();
    for (int g = 0; g < gp.ngate; ++g) {
        const int q = G[g];
        const double2* U = Utab + 16 * g;
        const int lowm = (1 << q) - 1;
        for (int j = t; j < (N >> 2); j += kSmallThreads) {
            const int b = (j & lowm) | ((j >> q) << (q + 2));
            double2 a[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) a[m] = s[b | (m << q)];
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                double2 acc = make_double2(0.0, 0.0);
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const double2 u = U[4 * l + m];
                    acc.x = fma(u.x, a[m].x, fma(-u.y, a[m].y, acc.x));
                    acc.y = fma(u.x, a[m].y, fma(u.y, a[m].x, acc.y));
                }
                s[b | (l << q)] = acc;
            }
        }
        __syncthreads();
    }
    for (int i = t; i < N; i += kSmallThreads) psi[i] = s[i];
}

struct Geometry {
    int first, c, h0, tbits;
};

// Global bit of tile-local bit q in a pass.
int global_bit(const Geometry& ge, int q) { return ge.first ? q : (q < ge.c ? q : ge.h0 + (q - ge.c)); }

// The two-site Hamiltonian of the bond on bits (p, p+1) (sites k = L-p-1 and k+1), 4x4 with
// index 2 bit(p+1) + bit(p): bond terms plus the shared site terms.
void bond_hamiltonian(const ed_model* m, int p, cplx* h) {
    const int L = m->L;
    auto weight = [&](int bit) {
        const int k = L - bit;  // site
        const int nb = (k > 1 ? 1 : 0) + (k < L ? 1 : 0);
        return 1.0 / nb;
    };
    for (int e = 0; e < 16; ++e) h[e] = cplx(m->bond[16 * p + e].x, m->bond[16 * p + e].y);
    const double wl = weight(p + 1), wr = weight(p);
    for (int r = 0; r < 2; ++r)
        for (int c = 0; c < 2; ++c) {
            const cplx sl(m->site[4 * (p + 1) + 2 * r + c].x, m->site[4 * (p + 1) + 2 * r + c].y);
            const cplx sr(m->site[4 * p + 2 * r + c].x, m->site[4 * p + 2 * r + c].y);
            for (int o = 0; o < 2; ++o) {
                h[4 * (2 * r + o) + (2 * c + o)] += wl * sl;  // site k (x) I
                h[4 * (2 * o + r) + (2 * o + c)] += wr * sr;  // I (x) site k+1
            }
        }
}

// Host copy of a call's gate table and its place in device memory (null: only counting passes).
struct GateTable {
    std::vector<double2> U;
    std::vector<int> G, R;
    const double2* dev_U = nullptr;
    const int *dev_G = nullptr, *dev_R = nullptr;
};

// Rounds of a pass over a 12-bit tile. gates: (layer, q) by layer, then q; a_min: the lowest register
// bit a round may start at. Each round takes four adjacent tile bits and every gate on them that is
// free, layer by layer (no unapplied gate of an earlier layer shares a bit with it); the four bits
// with the most such gates come first. The first and the last round must start at bit kGLow or above
// (they move the tile from and to memory), so a round without gates is put before or after where
// that leaves no other choice. order: the gates by round; base: the round's first bit, per gate of
// order; R: the rounds' codes (appended).
void plan_rounds(const std::vector<std::pair<int, int>>& gates, int a_min, std::vector<int>* order,
                 std::vector<int>* base, std::vector<int>* R) {
    const int n = int(gates.size());
    const int a_max = kGTileBits - kGRegBits;
    std::vector<char> done(n, 0);
    auto take = [&](int a, std::vector<char> d) {
        std::vector<int> got;
        for (int g = 0; g < n; ++g) {
            if (d[g] || gates[g].second < a || gates[g].second + 1 >= a + kGRegBits) continue;
            bool free = true;
            for (int e = 0; e < n && free; ++e)
                free = d[e] || gates[e].first >= gates[g].first || std::abs(gates[e].second - gates[g].second) > 1;
            if (free) {
                d[g] = 1;
                got.push_back(g);
            }
        }
        return got;
    };
    bool first_round = true;
    int last_a = a_max;
    base->clear();
    while (int(order->size()) < n) {
        std::vector<int> best;
        int best_a = -1;
        for (int a = a_max; a >= (first_round ? kGLow : a_min); --a) {
            const std::vector<int> got = take(a, done);
            if (got.size() > best.size()) {
                best = got;
                best_a = a;
            }
        }
        if (best.empty()) {
            if (!first_round) return;  // no free gate: cannot happen for gates listed by layer
            best_a = a_max;            // all free gates sit below: a round without gates stages the tile
        }
        R->push_back(round_code(best_a, int(order->size()), int(order->size() + best.size())));
        for (int g : best) {
            done[g] = 1;
            order->push_back(g);
            base->push_back(best_a);
        }
        last_a = best_a;
        first_round = false;
    }
    if (last_a < kGLow) R->push_back(round_code(a_max, n, n));
}

// Passes of a run of consecutive layers (part, time): layer l holds the propagators exp(-i t_l h)
// of the bonds whose left site k has the layer's parity (1: odd k, H_o; 0: even k, H_e). The first
// pass is the contiguous tile of the 12 low bits; each later pass is a window of 8 bits above 4
// contiguous low bits, starting at the lowest bond still pending. A gate (l, p) on bits (p, p+1)
// is ready once every gate of an earlier layer on bonds p - 1, p, p + 1 has a pass; going through
// the layers in order, each pass takes the ready gates its tile holds. The matrices and codes go to
// tab; the passes point at its device copy. Returns false when a gate finds no pass or the table is
// full.
bool build_run(const ed_model* m, const std::vector<std::pair<int, double>>& run, double dt, GateTable* tab,
               std::vector<GatePass>* out) {
    const int L = m->L;
    const int F = int(run.size());
    const int T = std::min(L, kGTileBits);
    const int wb = kGTileBits - kGLow;
    auto is_bond = [&](int l, int p) { return p >= 0 && p + 1 < L && ((L - p - 1) & 1) == run[l].first; };
    std::vector<std::vector<int>> at(F, std::vector<int>(L, -1));  // pass of gate (l, p)
    int pending = 0;
    for (int l = 0; l < F; ++l)
        for (int p = 0; p + 1 < L; ++p) pending += is_bond(l, p);
    auto ready = [&](int l, int p) {
        for (int e = 0; e < l; ++e)
            for (int d = -1; d <= 1; ++d)
                if (is_bond(e, p + d) && at[e][p + d] < 0) return false;
        return true;
    };
    std::vector<Geometry> geo;
    std::vector<std::vector<std::pair<int, int>>> gates;  // (layer, p) of each pass, by layer then p
    auto fill = [&](const Geometry& ge, int lo, int hi) {  // gates with both bits in [lo, hi)
        const int pass = int(geo.size());
        std::vector<std::pair<int, int>> gs;
        for (int l = 0; l < F; ++l)
            for (int p = lo; p + 1 < hi; ++p)
                if (is_bond(l, p) && at[l][p] < 0 && ready(l, p)) {
                    at[l][p] = pass;
                    gs.push_back({l, p});
                    --pending;
                }
        geo.push_back(ge);
        gates.push_back(gs);
        return !gs.empty();
    };
    fill({1, T, T, T}, 0, T);
    while (pending > 0) {
        int h0 = L;
        for (int l = 0; l < F; ++l)
            for (int p = 0; p + 1 < L; ++p)
                if (is_bond(l, p) && at[l][p] < 0) h0 = std::min(h0, p);
        h0 = std::min(h0, L - wb);
        if (h0 < kGLow) return false;
        if (!fill({0, kGLow, h0, kGTileBits}, h0, h0 + wb)) return false;
    }
    for (size_t i = 0; i < geo.size(); ++i) {
        if (gates[i].empty()) continue;
        if (tab->U.size() / 16 + gates[i].size() > size_t(kTableGates)) return false;
        GatePass gp;
        std::memset(&gp, 0, sizeof(GatePass));
        gp.first = geo[i].first;
        gp.c = geo[i].c;
        gp.h0 = geo[i].h0;
        gp.tbits = geo[i].tbits;
        gp.U = tab->dev_U ? tab->dev_U + tab->U.size() : nullptr;  // null when only counting passes
        gp.G = tab->dev_G ? tab->dev_G + tab->G.size() : nullptr;
        gp.R = tab->dev_R ? tab->dev_R + tab->R.size() : nullptr;
        std::vector<std::pair<int, int>> local;  // (layer, tile bit q) in order of application
        for (const auto& lp : gates[i]) {
            const int l = lp.first, p = lp.second;
            const int q = geo[i].first ? p : geo[i].c + (p - geo[i].h0);
            if (global_bit(geo[i], q) != p || global_bit(geo[i], q + 1) != p + 1) return false;
            local.push_back({l, q});
        }
        std::vector<int> base(local.size(), 0);  // first register bit of each gate's round
        if (gp.tbits == kGTileBits) {
            std::vector<int> order;
            const size_t r0 = tab->R.size();
            plan_rounds(local, gp.first ? 0 : kGLow, &order, &base, &tab->R);
            if (order.size() != local.size() || tab->R.size() > size_t(kTableRounds)) return false;
            gp.nround = int(tab->R.size() - r0);
            std::vector<std::pair<int, int>> sorted;
            for (int g : order) sorted.push_back(local[g]);
            local = sorted;
        }
        for (size_t g = 0; g < local.size(); ++g) {
            const int l = local[g].first, q = local[g].second, p = global_bit(geo[i], q);
            cplx h[16], A[16], U[16];
            bond_hamiltonian(m, p, h);
            for (int e = 0; e < 16; ++e) A[e] = cplx(0.0, -run[l].second * dt) * h[e];
            expm_complex(4, A, U);
            bool cross = true;
            for (int r = 0; r < 4; ++r)
                for (int c = 0; c < 4; ++c)
                    if (c != r && c != 3 - r) cross = cross && U[4 * r + c] == cplx(0.0, 0.0);
            for (int e = 0; e < 16; ++e) tab->U.push_back(make_double2(U[e].real(), U[e].imag()));
            tab->G.push_back(gp.tbits < kGTileBits ? q : (1 << (q - base[g])) * (cross ? kCross : 1));
            ++gp.ngate;
        }
        out->push_back(gp);
    }
    return true;
}

hipError_t run_passes(const std::vector<GatePass>& passes, double2* psi, int L, hipStream_t s) {
    for (const GatePass& gp : passes) {
        const int64_t tiles = int64_t(1) << (L - gp.tbits);
        if (gp.tbits == kGTileBits)
            hipLaunchKernelGGL(gate_pass, dim3(unsigned(tiles)), dim3(kGThreads), 0, s, psi, gp, gp.U, gp.G, gp.R);
        else  // L < 12: one tile
            hipLaunchKernelGGL(gate_pass_small, dim3(1), dim3(kSmallThreads), 0, s, psi, gp, gp.U, gp.G);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The layers of one step (part, fraction of dt): Eq. ed:eq:trotter2 or Eq. ed:eq:trotter4 with
// the constants of Eq. ed:eq:trotter4c; part 0 = H_e (even k), 1 = H_o (odd k).
std::vector<std::pair<int, double>> step_layers(int order) {
    const double tau3 = 1.0 / (2.0 * (4.0 - std::cbrt(4.0)));
    const double tau1 = 1.0 - 8.0 * tau3, tau2 = 0.5 * (1.0 - 6.0 * tau3), tau4 = 2.0 * tau3;
    if (order == 2) return {{0, 0.5}, {1, 1.0}, {0, 0.5}};
    return {{0, tau3}, {1, tau4}, {0, tau4}, {1, tau4}, {0, tau2}, {1, tau1},
            {0, tau2}, {1, tau4}, {0, tau4}, {1, tau4}, {0, tau3}};
}

// The passes of one step: the step's layers in runs of kFuse, one set of passes per distinct run
// (runs), the run of each position (which), and the table of their gates.
struct StepPlan {
    std::vector<std::vector<GatePass>> runs;
    std::vector<int> which;
    GateTable table;
};

// dev: device memory of the gate table (kGateTableBytes), or null when only counting passes.
ed_status plan_step(const ed_model* m, int order, double dt, char* dev, StepPlan* sp) {
    if (dev) {
        sp->table.dev_U = reinterpret_cast<double2*>(dev);
        sp->table.dev_G = reinterpret_cast<int*>(dev + size_t(kTableGates) * 16 * sizeof(double2));
        sp->table.dev_R = sp->table.dev_G + kTableGates;
    }
    const std::vector<std::pair<int, double>> seq = step_layers(order);
    std::vector<std::vector<std::pair<int, double>>> keys;
    for (size_t i0 = 0; i0 < seq.size(); i0 += kFuse) {
        const std::vector<std::pair<int, double>> run(seq.begin() + i0, seq.begin() + std::min(seq.size(), i0 + kFuse));
        int found = -1;
        for (size_t j = 0; j < keys.size(); ++j)
            if (keys[j] == run) found = int(j);
        if (found < 0) {
            std::vector<GatePass> passes;
            if (!build_run(m, run, dt, &sp->table, &passes))
                return fail(ED_ERR_UNSUPPORTED, "internal error: no Trotter pass plan for L = " + std::to_string(m->L));
            keys.push_back(run);
            sp->runs.push_back(passes);
            found = int(keys.size()) - 1;
        }
        sp->which.push_back(found);
    }
    return ED_OK;
}

}  // namespace
}  // namespace ed

extern "C" ed_status ed_trotter_workspace(const ed_model* model, int with_energy, size_t* bytes) {
    if (!model || !bytes) return ed::fail(ED_ERR_ARG, "null argument");
    const int64_t D = int64_t(1) << model->L;
    // the scratch of the norm and energy kernels, two state vectors for the energy, the gate table
    *bytes = ed::core_scratch_bytes() + (with_energy ? size_t(2) * size_t(D) * sizeof(double2) + 256 : 0) +
             ed::kGateTableBytes;
    return ED_OK;
}

extern "C" ed_status ed_trotter_evolve(const ed_model* model, ed_c64* psi, double dt, int n_steps, int order,
                                       const ed_observe* obs, void* ws, size_t ws_bytes, void* stream) {
    using namespace ed;
    if (!model || !psi) return fail(ED_ERR_ARG, "null argument");
    if (order != 2 && order != 4) return fail(ED_ERR_ARG, "order must be 2 or 4");
    if (model->lr || model->lv_L > 0) return fail(ED_ERR_UNSUPPORTED, "the Trotter layers take site and bond rules only");
    if (n_steps < 0) return fail(ED_ERR_ARG, "n_steps must be >= 0");
    if (!std::isfinite(dt)) return fail(ED_ERR_ARG, "dt must be finite");
    const bool want_e = obs && obs->energy;
    size_t need = 0;
    ED_TRY(ed_trotter_workspace(model, want_e ? 1 : 0, &need));
    if (!ws) return fail(ED_ERR_ARG, "workspace is null");
    if (ws_bytes < need) return fail(ED_ERR_WORKSPACE, "workspace too small (energy needs with_energy = 1)");
    const int L = model->L;
    const int64_t D = int64_t(1) << L;
    Workspace w;
    ED_TRY(carve(ws, ws_bytes, D, want_e ? 2 : 0, &w));
    hipStream_t s = static_cast<hipStream_t>(stream);
    double2* v = reinterpret_cast<double2*>(psi);
    ObsStage stage;
    obs = stage.begin(obs, n_steps, L);

    // the step's passes; their gate matrices in the table at the end of the workspace
    const size_t vec_bytes = want_e ? (size_t(2) * size_t(D) * sizeof(double2) + 255) & ~size_t(255) : 0;
    const size_t table_off = core_scratch_bytes() + vec_bytes;  // after what carve hands out
    if (table_off + kGateTableBytes > ws_bytes) return fail(ED_ERR_WORKSPACE, "workspace too small for the gate table");
    char* const tab = static_cast<char*>(ws) + table_off;
    StepPlan sp;
    ED_TRY(plan_step(model, order, dt, tab, &sp));
    if (!sp.table.U.empty()) {
        auto upload = [&](const void* dst, const void* src, size_t bytes) {
            return bytes ? hipMemcpyAsync(const_cast<void*>(dst), src, bytes, hipMemcpyHostToDevice, s) : hipSuccess;
        };
        ED_HIP_TRY(upload(sp.table.dev_U, sp.table.U.data(), sp.table.U.size() * sizeof(double2)));
        ED_HIP_TRY(upload(sp.table.dev_G, sp.table.G.data(), sp.table.G.size() * sizeof(int)));
        ED_HIP_TRY(upload(sp.table.dev_R, sp.table.R.data(), sp.table.R.size() * sizeof(int)));
        ED_HIP_TRY(hipStreamSynchronize(s));  // the host tables are locals
    }
    auto record = [&](int step) -> ed_status {
        if (obs && (obs->sz || obs->norm)) {
            double nrm = 0.0;
            ED_TRY(measure_state(v, L, w, obs->sz ? obs->sz + size_t(step) * L : nullptr, &nrm, s));
            if (obs->norm) obs->norm[step] = nrm;
        }
        if (want_e) {
            double e = 0.0;
            ED_TRY(energy_of(model, w, v, &e, s));
            obs->energy[step] = e;
        }
        return ED_OK;
    };
    ED_TRY(record(0));
    for (int st = 0; st < n_steps; ++st) {
        for (int r : sp.which) {
            const hipError_t e = run_passes(sp.runs[r], v, L, s);
            if (e != hipSuccess) return fail(ED_ERR_HIP, std::string("Trotter layer launch: ") + hipGetErrorString(e));
        }
        ED_TRY(record(st + 1));
    }
    ED_HIP_TRY(hipStreamSynchronize(s));
    return stage.finish(s);
}

extern "C" ed_status ed_trotter_passes(const ed_model* model, int order, int* passes) {
    using namespace ed;
    if (!model || !passes) return fail(ED_ERR_ARG, "null argument");
    if (order != 2 && order != 4) return fail(ED_ERR_ARG, "order must be 2 or 4");
    if (model->lr || model->lv_L > 0) return fail(ED_ERR_UNSUPPORTED, "the Trotter layers take site and bond rules only");
    StepPlan sp;
    ED_TRY(plan_step(model, order, 0.0, nullptr, &sp));
    int n = 0;
    for (int r : sp.which) n += int(sp.runs[r].size());
    *passes = n;
    return ED_OK;
}
