// evolve_shared.h -- resident integration of small lattices: packs of whole
// trajectories (both spin blocks) in one workgroup, every stencil address in
// registers.  Included by evolve_shared_f32.hip and evolve_shared_f64.hip,
// which instantiate the kernel for one precision each.
//
// Equation of motion: Eq. (6) of arXiv:2212.04352,
//   f_ij = i [ t (sum_{k in nb(j)} rho_ik - sum_{k in nb(i)} rho_kj) + U (d_i - d_j) rho_ij ],
// d = diagonal of the other spin, classical RK4 in the fixed operation order
// of the other kernels (results are bitwise theirs).
//
// Layout.  The lattice is bipartite (sublattices A and B), so a spin block is
// AA and BB (the even class, Hermitian) and AB (the odd class; BA is its
// conjugate transpose).  LDS holds the stage input of a pack of K = 2^k
// trajectories: AA and BB as full squares, AB as a rectangle, rows S elements
// apart, the pack's trajectories of an element side by side in units of 16
// bytes: an element of both spins in FP32, of one in FP64 (the other spin's
// unit follows it).  A thread works on both spins of an FP32 element or on one
// (SPT), always on one of an FP64 element.  Nothing is
// ever read as its conjugate:
//   AB_ab:  col = sum_{k in nb(b)} AA_ak,  row = sum_{k in nb(a)} BB_kb;
//   AA_aa': col = sum_{k in nb(a')} AB_ak, conj(row) = R = sum_{k in nb(a)} AB_a'k;
//     with g = col - row: g.x = col.x - R.x, g.y = col.y + R.y;
//   BB_bb': the same form C = sum_{k in nb(b)} AB_kb', R = sum_{k in nb(b')} AB_kb
//     gives -g, so a BB element carries -f in place of f: its d_i - d_j is
//     taken as d_j - d_i and its Runge-Kutta coefficients enter negated (all
//     of it exact).
// The even elements are written twice (the element and its conjugate
// transpose).
//
// Bank conflicts.  LDS bandwidth bounds this kernel, and what it costs was
// measured (cycles per wave instruction): a 16-byte read 4.3 when each
// 16-lane group of a wave -- lanes 0-3, 12-15, 20-27 and 4-11, 16-19, 28-31 of
// either half -- reads 16 different units modulo 16, up to twice that for runs
// shorter than 32 lanes at arbitrary places; an 8-byte read 3.2, a 16-byte
// write 13 (eight lanes at a time over 128 bytes), an 8-byte write 6.3.  So
// FP32 reads both spins of a neighbour with one instruction, and I
// consecutive lanes (the trajectories, and the spins where SPT = 1) share an
// element: with I = 16 no access has a conflict; with fewer, the elements are
// dealt to lanes such that those of a group differ modulo M = 16 / I in every
// access.  With S odd (I = 1: S^2 = 1 modulo 16) every address of an element
// is own or S own plus a constant of its neighbourhood modulo M, so elements
// of equal neighbourhood shape and different own addresses are free of
// conflicts (shared_deal in lattice.cpp fills the groups).
//
// Threads.  I lanes own entries t / I + (NT / I) u, u < U, of the lattice's
// even list and of its odd list.  The addresses of an element's six
// neighbours, of itself and of the two diagonal values are computed once per
// table entry and stay in registers, so a stage touches nothing but LDS.
//
// With a general interaction the waves beyond the workers form the sums D_i
// of the next stage while the workers are at the odd elements: one lane per
// site and trajectory, each an ascending chain of N fused multiply-adds per
// spin.  (On the workers the chain's operands had no registers beside the
// state: 54 sites FP64 2.44e7 trajectory-steps/s, on
// waves of its own 2.56e7, the shared-block tiles 2.24e7.)
//
// A stage is two phases with a barrier after each: the even elements write
// the stage input they hold to AA and BB (nothing reads these in this phase),
// read AB and form their next values; then the odd elements read AA and BB
// and write their next values to AB.  The diagonal that the U term reads is a
// separate array of reals in two copies (stage parity), so the next diagonal
// is written in the first phase.  One wave per workgroup (NT = 64) needs no
// barrier: a wave's LDS operations complete in order.
#pragma once

#include <type_traits>

#include "device_common.h"
#include "ftwa_internal.h"

namespace ftwa {

struct SharedArgs {
    const ResidentInst* table;  // entries (instance windows), item0 ascending
    int n_entries;
    int kshift;                 // log2 of the trajectories per item
    int workers;                // threads that own elements (the others: see GINT)
    int64_t n_items;
    double dt;
    int64_t n_steps;
    int record_every;
};

// Hamiltonian variants: on-site U; with an external potential; with complex
// hopping; with a general interaction.
enum { kSharedPlain = 0, kSharedPot = 1, kSharedHop = 2, kSharedGint = 3 };

// Diagonal pairs (up, down) of a pack (N K) that the fixed diagonal areas
// hold.
constexpr int shared_diag_cap(int maxt) { return maxt == 64 ? 64 : 320; }

namespace shared_detail {

template <typename T> struct Vec;
template <> struct Vec<float> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct Vec<double> { typedef double type __attribute__((ext_vector_type(2))); };
template <typename T> using vec_t = typename Vec<T>::type;

#define FTWA_LDS __attribute__((address_space(3)))

// LDS accesses by byte address (the kernel declares no static LDS, so the
// dynamic block starts at address 0).
template <typename V> __device__ __forceinline__ V lds_get(uint32_t a) {
    return *(const FTWA_LDS V*)(uintptr_t)a;
}
template <typename V> __device__ __forceinline__ void lds_put(uint32_t a, V v) {
    *(FTWA_LDS V*)(uintptr_t)a = v;
}

// v with its sign bit toggled by mask (0 or 0x80000000).
__device__ __forceinline__ float flip(float v, uint32_t mask) {
    return __uint_as_float(__float_as_uint(v) ^ mask);
}
__device__ __forceinline__ double flip(double v, uint32_t mask) {
    return __hiloint2double(__double2hiint(v) ^ (int)mask, __double2loint(v));
}

template <typename T> __device__ __forceinline__ T scalar_real(double v) {
    if constexpr (sizeof(T) == 4) {
        const float f = (float)v;
        return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(f)));
    } else {
        const int lo = __builtin_amdgcn_readfirstlane(__double2loint(v));
        const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
        return __hiloint2double(hi, lo);
    }
}
__device__ __forceinline__ uint64_t scalar_ptr(const void* p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// A copy of v the compiler knows nothing about: index arithmetic on it is not
// shared with (and kept in registers since) an earlier use.
__device__ __forceinline__ int fresh(int v) {
    __asm__ volatile("" : "+v"(v));
    return v;
}

// Computes v here: without it the compiler keeps the slopes of three stages
// and forms the accumulator at the end.
template <typename V> __device__ __forceinline__ void settle(V& v) {
    __asm__ volatile("" : "+v"(v.x), "+v"(v.y));
}

// Orders the LDS accesses of the workgroup's phases.  Global stores (records)
// are not waited for: no thread reads them.
template <int MAXT> __device__ __forceinline__ void phase_barrier() {
    if constexpr (MAXT == 64)
        __asm__ volatile("" ::: "memory");
    else
        __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

}  // namespace shared_detail

// One instantiation set: U slots per class and thread, spt spins per slot, up
// to maxt threads per workgroup; the kernels by variant, general t and t = 1.
struct SharedShape {
    ftwa_dtype dtype;
    int U, spt, maxt;
    bool packed;    // addresses two to a register
    const void* fn[4];  // NULL: the shape has none
    const void* fn_t1[4];
};
constexpr int kSharedShapes = 6;  // of each precision
extern const SharedShape kSharedF32[kSharedShapes];
extern const SharedShape kSharedF64[kSharedShapes];

// LDS bytes before the blocks: two diagonal copies, then (potential) its
// profile in the same layout or (general interaction) two copies of D.
constexpr uint32_t shared_head(int tb, int maxt, int var) {
    return (uint32_t)((var == kSharedPot ? 3 : var == kSharedGint ? 4 : 2) *
                      shared_diag_cap(maxt) * 2 * tb);
}

template <typename T, int U, int SPT, int MAXT, int MINW, bool PF, bool PK, bool T1, int VAR>
__global__ __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(MINW, 8)))
void rk4_shared(SharedArgs A) {
    using namespace shared_detail;
    using C = vec_t<T>;
    using G = cplx_t<T>;
    constexpr bool F64 = sizeof(T) == 8;
    constexpr bool POT = VAR == kSharedPot, HOP = VAR == kSharedHop, GINT = VAR == kSharedGint;
    constexpr uint32_t CB = sizeof(C), TB = sizeof(T);
    constexpr uint32_t kDg = shared_diag_cap(MAXT) * 2 * TB;  // one diagonal copy
    constexpr uint32_t kHead = shared_head(TB, MAXT, VAR);
    static_assert(!F64 || SPT == 1, "an FP64 element's spins go to two lanes");
    extern __shared__ __align__(16) unsigned char smem[];  // dynamic LDS, at address 0
    (void)smem;
    const int tid = threadIdx.x;
    const int NT = MAXT == 64 ? 64 : A.workers;
    const int K = 1 << A.kshift;
    const int ishift = A.kshift + (SPT == 1 ? 1 : 0);  // lanes per entry
    const int lq = SPT == 1 ? (tid >> 1) & (K - 1) : tid & (K - 1);  // this lane's trajectory
    const int ls = SPT == 1 ? tid & 1 : 0;                           // and spin

    // Workgroups are dealt round-robin to the eight XCDs: a round's items go to
    // them in eight runs of consecutive ones (neighbouring trajectories, which
    // share cache lines of the state), a last round that is not full in eight
    // shorter runs, so that it is spread over the chip too.  (An eighth of all
    // items to each XCD instead is up to 2 % slower where the rounds are full.
    // Places within the round in 32 bits: in 64 bits they cost the occupancy of
    // the general interaction's kernel of one slot.)
    const bool runs = gridDim.x % 8 == 0;
    const unsigned xcd = runs ? blockIdx.x % 8 : 0, slot = runs ? blockIdx.x / 8 : blockIdx.x;

    C y[2 * U][SPT], acc[2 * U][SPT], Y[2 * U][SPT];  // even slots, then odd slots
    // addresses: kAddr fields per slot (six neighbours, the element and its
    // transpose, the two diagonal values), packed two to a register where PK
    enum { kC = 0, kR = 3, kOwn = 6, kOwn2 = 7, kDi = 8, kDj = 9, kAddr = 10 };
    uint32_t ad[2 * U][PK ? kAddr / 2 : kAddr], neg[U];
    // field f of slot v (constants once unrolled); PK: addresses in units of
    // 8 bytes (the diagonal offsets in bytes / 4)
    auto set_addr = [&](int v, int f, uint32_t a) {
        if constexpr (!PK) {
            ad[v][f] = a;
        } else {
            const uint32_t x = f >= kDi ? a >> 2 : a >> 3;
            ad[v][f / 2] = f % 2 ? ad[v][f / 2] | x << 16 : x;
        }
    };
    auto addr = [&](int v, int f) -> uint32_t {
        if constexpr (!PK) return ad[v][f];
        const uint32_t w = ad[v][PK ? f / 2 : 0];
        if (f >= kDi) return f % 2 ? hi16_shl<2>(w) : lo16_shl<2>(w);
        return f % 2 ? hi16_shl<3>(w) : lo16_shl<3>(w);
    };
    // slot 0 may hold a diagonal element: the place of its value in a diagonal
    // copy and (general interaction) of h, all ones otherwise
    uint32_t dg = 0xffffffffu, hg = 0;
    uint32_t wo[HOP ? 2 * U : 1];  // complex hopping: the two ratio triples' offsets
    int cur = -1;

    for (int64_t base = 0; base < A.n_items; base += gridDim.x) {
        const unsigned round = A.n_items - base < gridDim.x ? (unsigned)(A.n_items - base) : gridDim.x;
        const unsigned run = runs ? (round + 7) / 8 : round, place = xcd * run + slot;
        if (slot >= run || place >= round) break;
        const int64_t item = base + place;
        int ent = 0;
        while (ent + 1 < A.n_entries && A.table[ent + 1].item0 <= item) ++ent;
        ent = __builtin_amdgcn_readfirstlane(ent);
        const ResidentInst& E = A.table[ent];
        const int N = E.N, NA = E.n_a;
        const int P = E.P;
        // the dealt lists (shared_lists): [2 N] sites by position and their
        // neighbours' positions, then `room` even and `room` odd entries
        // a | b << 8, all ones: none
        const uint32_t* const site = E.stab;
        const uint32_t* const nbp = E.stab + N;
        const uint32_t* const list = E.stab + 2 * N;
        const int n_pass = NT >> ishift, room = shared_room(ishift);
        const int S = shared_stride(N, NA, 1 << ishift);
        const int o_bb = NA * S, o_ab = N * S;
        // elements of a block, then M that stay zero (missing neighbours) and
        // M of scratch (padding entries write there)
        const int M = ishift >= 4 ? 1 : 16 >> ishift;
        const int e_zero = ((N + NA) * S + M - 1) & -M, e_scr = e_zero + M;
        // LDS address of element e of this lane's trajectory (and spin)
        auto at = [&](int e) -> uint32_t {
            uint32_t unit = ((uint32_t)e << A.kshift) + (uint32_t)lq;
            if constexpr (F64) unit = 2 * unit + (uint32_t)ls;
            return kHead + (unit << 4) + (!F64 && SPT == 1 ? 8u * (uint32_t)ls : 0u);
        };
        const uint32_t tail =
            kHead + ((((uint32_t)(e_scr + M) << A.kshift) + 15u) & ~15u) * (F64 ? 32u : 16u);
        // complex hopping: two copies of the stage's ratio table, three per
        // position
        const uint32_t wtab = tail;
        // general interaction: h = d + 1/2 of both spins in site order, the
        // pack's trajectories side by side (zero from N up to the row count KU
        // of u's table), then u where the plan made room
        const int KU = umat_rows(N);
        const uint32_t hs = tail;
        const uint32_t hstr = (uint32_t)(KU + 2) * 2 * TB;  // trajectories apart in banks
        const uint32_t ulds = hs + (uint32_t)K * hstr;
        G* const rho = reinterpret_cast<G*>(scalar_ptr(E.rho));
        const int64_t Mc = E.Mc, ldr = E.ldr;
        const int64_t m0 = (item - E.item0) * K;
        double* const Xrec = E.X;

        // ---- addresses, once per table entry
        if (ent != cur && (!GINT || tid < NT)) {
            cur = ent;
#pragma unroll
            for (int v = 0; v < 2 * U; ++v) {
                const int x = (tid >> ishift) + n_pass * (v < U ? v : v - U);
                const uint32_t w = list[(v < U ? 0 : room) + x];
                const bool ok = w != 0xffffffffu;
                const int a = ok ? (int)(w & 0xffu) : 0, b = ok ? (int)(w >> 8 & 0xffu) : 0;
                const bool b_cls = v < U && a >= NA;  // BB
                const uint32_t pc = nbp[b_cls ? a : b], pr = nbp[b_cls ? b : a];
                uint32_t f[kAddr];
                int me, me2 = 0;
                if (v >= U) {
                    me = o_ab + a * S + b - NA;
                } else if (b_cls) {
                    me = o_bb + (a - NA) * S + b - NA;
                    me2 = o_bb + (b - NA) * S + a - NA;
                } else {
                    me = a * S + b;
                    me2 = b * S + a;
                }
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    const int kc = (int)((pc >> (8 * n)) & 0xffu), kr = (int)((pr >> (8 * n)) & 0xffu);
                    int c, r;
                    if (v >= U) {
                        c = a * S + kc;                       // AA_ak
                        r = o_bb + (kr - NA) * S + b - NA;    // BB_kb
                    } else if (!b_cls) {
                        c = o_ab + a * S + kc - NA;           // AB_ak
                        r = o_ab + b * S + kr - NA;           // AB_bk
                    } else {
                        c = o_ab + kc * S + b - NA;           // AB_kb
                        r = o_ab + kr * S + a - NA;           // AB_ka
                    }
                    // a missing neighbour: the zero element of this one's residue
                    f[kC + n] = at(ok && kc != 0xff ? c : e_zero + (me & (M - 1)));
                    f[kR + n] = at(ok && kr != 0xff ? r : e_zero + (me & (M - 1)));
                }
                const int pi = b_cls ? b : a, pj = b_cls ? a : b;  // d_i - d_j of the U term
                if (v == 0) {
                    dg = ok && a == b ? (uint32_t)(a * K + lq) * 2 * TB + ls * TB : 0xffffffffu;
                    if constexpr (GINT) hg = hs + (uint32_t)lq * hstr + (uint32_t)site[a] * 2 * TB + ls * TB;
                }
                const uint32_t spo = SPT == 1 ? (uint32_t)(ls ^ 1) * TB : 0u;  // the other spin's
                f[kDi] = (uint32_t)(pi * K + lq) * 2 * TB + spo;
                f[kDj] = (uint32_t)(pj * K + lq) * 2 * TB + spo;
                if constexpr (HOP) wo[v] = (uint32_t)(pj * 3 * CB) | (uint32_t)(pi * 3 * CB) << 16;
                f[kOwn] = at(ok ? me : e_scr + (x & (M - 1)));
                f[kOwn2] = at(ok ? me2 : e_scr + (x & (M - 1)));
                if (v < U) neg[v] = b_cls ? 0x80000000u : 0u;
#pragma unroll
                for (int n = 0; n < kAddr; ++n) set_addr(v, n, f[n]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // packed element of the state in HBM of slot v, spin index sp (false:
        // none); tr: its transpose
        auto state_at = [&](int v, int sp, int64_t& off, bool& tr) -> bool {
            const uint32_t w = list[(v < U ? 0 : room) + (fresh(tid) >> ishift) +
                                    n_pass * (v < U ? v : v - U)];
            const int64_t m = m0 + lq;
            if (w == 0xffffffffu || m >= Mc) return false;
            const int s = SPT == 1 ? ls : sp;
            const int sa = (int)site[w & 0xffu], sb = (int)site[w >> 8 & 0xffu];
            const int i = sa < sb ? sa : sb, j = sa < sb ? sb : sa;
            tr = sa > sb;
            off = ((int64_t)s * P + (int64_t)i * N - (int64_t)i * (i - 1) / 2 + (j - i)) * ldr + m;
            return true;
        };
        // element of slot address o from and to LDS, both spins where SPT = 2
        auto put = [&](uint32_t o, const C* v, bool cj) {
            C z[SPT];
#pragma unroll
            for (int s = 0; s < SPT; ++s) {
                z[s].x = v[s].x;
                z[s].y = cj ? -v[s].y : v[s].y;
            }
            if constexpr (SPT == 2) {
                typedef float F4 __attribute__((ext_vector_type(4)));
                lds_put<F4>(o, F4{z[0].x, z[0].y, z[SPT - 1].x, z[SPT - 1].y});
            } else {
                lds_put<C>(o, z[0]);
            }
        };
        auto get = [&](uint32_t o, C* v) {
            if constexpr (SPT == 2) {
                typedef float F4 __attribute__((ext_vector_type(4)));
                const F4 f = lds_get<F4>(o);
                v[0].x = f.x;
                v[0].y = f.y;
                v[SPT - 1].x = f.z;
                v[SPT - 1].y = f.w;
            } else {
                v[0] = lds_get<C>(o);
            }
        };
        // the diagonal element of slot 0 into a diagonal copy (and h = d + 1/2)
        auto put_diag = [&](uint32_t copy, const C* v) {
            if (dg == 0xffffffffu) return;
            if constexpr (SPT == 2) {
                lds_put<C>(copy + dg, C{v[0].x, v[SPT - 1].x});
                if constexpr (GINT) lds_put<C>(hg, C{v[0].x + (T)0.5, v[SPT - 1].x + (T)0.5});
            } else {
                lds_put<T>(copy + dg, v[0].x);
                if constexpr (GINT) lds_put<T>(hg, v[0].x + (T)0.5);
            }
        };

        phase_barrier<MAXT>();  // the previous item is done with LDS
        if constexpr (GINT) {
            if (tid >= NT) {
                // ---- the interaction's waves: u into LDS, then D of every
                // stage input, D_x = sum_k u_k,site(x) h_k of diagonal entry x,
                // both spins (an ascending fused chain each; the padded terms
                // k >= N are fma(0, 0, D) = D exactly: D starts at +0 and never
                // holds -0), the next 8 (FP64: 4) terms read ahead
                const int t0 = tid - NT, nd = (int)blockDim.x - NT;
                const T* const utab = reinterpret_cast<const T*>(scalar_ptr(E.umat));
                const bool u_lds = E.u_lds != 0;
                for (int x = t0; x < (KU - N) * K; x += nd)
                    lds_put<C>(hs + (uint32_t)(x & (K - 1)) * hstr +
                                   (uint32_t)(N + (x >> A.kshift)) * 2 * TB, C{0, 0});
                if (u_lds)
                    for (int x = t0; x < KU * N / 2; x += nd)
                        lds_put<C>(ulds + (uint32_t)x * 2 * TB, reinterpret_cast<const C*>(utab)[x]);
                auto interaction = [&](uint32_t dst) {
                    for (int x = t0; x < K * N; x += nd) {
                        const uint32_t i = site[x >> A.kshift];
                        uint32_t h = hs + (uint32_t)(x & (K - 1)) * hstr;
                        uint32_t e = 4 * i;
                        C D = {0, 0};
                        auto chain = [&](auto read) {
                            constexpr int CH = sizeof(T) == 8 ? 4 : 8;
                            C ub[2][CH / 2], hb[2][CH];
                            auto load = [&](int p) {
#pragma unroll
                                for (int k = 0; k < CH; k += 4, e += 4 * (uint32_t)N) {
                                    ub[p][k / 2] = read(e);
                                    ub[p][k / 2 + 1] = read(e + 2);
                                }
#pragma unroll
                                for (int k = 0; k < CH; ++k) hb[p][k] = lds_get<C>(h + k * 2 * TB);
                                h += CH * 2 * TB;
                            };
                            auto add = [&](int p) {
#pragma unroll
                                for (int k = 0; k < CH; ++k) {
                                    const T u = k % 2 ? ub[p][k / 2].y : ub[p][k / 2].x;
                                    D.x = fma_rn<T>(u, hb[p][k].x, D.x);
                                    D.y = fma_rn<T>(u, hb[p][k].y, D.y);
                                }
                            };
                            load(0);
                            for (int k0 = 0; k0 < N; k0 += 2 * CH) {
                                load(1);
                                add(0);
                                if (k0 + 2 * CH < N) load(0);
                                add(1);
                            }
                        };
                        if (u_lds)
                            chain([&](uint32_t e) { return lds_get<C>(ulds + e * TB); });
                        else
                            chain([&](uint32_t e) { return *reinterpret_cast<const C*>(utab + e); });
                        lds_put<C>(dst + (uint32_t)x * 2 * TB, D);
                    }
                };
                phase_barrier<MAXT>();
                interaction(2 * kDg);
                phase_barrier<MAXT>();
                for (int64_t stage = 0; stage < 4 * A.n_steps; ++stage) {
                    phase_barrier<MAXT>();
                    interaction(2 * kDg + (uint32_t)((stage & 1) ^ 1) * kDg);
                    phase_barrier<MAXT>();
                }
                continue;
            }
        }

        // ---- load the trajectories
#pragma unroll
        for (int v = 0; v < 2 * U; ++v) {
#pragma unroll
            for (int s = 0; s < SPT; ++s) {
                int64_t off;
                bool tr;
                C z = {0, 0};
                if (state_at(v, s, off, tr)) {
                    const G w = rho[off];
                    z.x = w.x;
                    z.y = tr ? -w.y : w.y;
                }
                __builtin_amdgcn_sched_barrier(0);
                y[v][s] = Y[v][s] = z;
                acc[v][s] = z;
            }
            if (v >= U) put(addr(v, kOwn), Y[v], false);
            if (v == 0) put_diag(0, Y[0]);
        }
        if ((tid >> ishift) < M) {
            const C z[2] = {C{0, 0}, C{0, 0}};
            put(at(e_zero + (tid >> ishift)), z, false);
        }

        // external potential: the profile in the diagonal's layout, the
        // envelope read one stage ahead
        const double* const venv = POT ? reinterpret_cast<const double*>(scalar_ptr(E.v_env)) : nullptr;
        const bool pot_on = POT && E.v_site != nullptr;
        T Anext = 0;
        if constexpr (POT) {
            const double* const vs = reinterpret_cast<const double*>(scalar_ptr(E.v_site));
            for (int x = tid; x < K * N; x += NT) {
                const T v = pot_on ? (T)vs[site[x >> A.kshift]] : (T)0;
                lds_put<C>(2 * kDg + (uint32_t)x * 2 * TB, C{v, v});
            }
            if (pot_on) Anext = scalar_real<T>(venv[0]);
        }
        // complex hopping: [2 n_steps + 1][N][3] ratios in site order; the
        // first table, in position order
        const T* const hop = HOP ? reinterpret_cast<const T*>(scalar_ptr(E.hop)) : nullptr;
        constexpr int kW = 3;  // reals of a table per thread (6 N <= kW NT)
        T wreg[kW];
        auto ratios_load = [&](int64_t half) {
#pragma unroll
            for (int k = 0; k < kW; ++k) {
                const int x = tid + NT * k;
                if (x < 6 * N) wreg[k] = hop[half * 6 * N + (int64_t)site[x / 6] * 6 + x % 6];
            }
        };
        auto ratios_store = [&](int buf) {
#pragma unroll
            for (int k = 0; k < kW; ++k) {
                const int x = tid + NT * k;
                if (x < 6 * N) lds_put<T>(wtab + (uint32_t)(buf * 6 * N + x) * TB, wreg[k]);
            }
        };
        if constexpr (HOP) {
            ratios_load(0);
            ratios_store(0);
        }
        if constexpr (GINT) phase_barrier<MAXT>();  // h complete; D formed before the next
        phase_barrier<MAXT>();

        auto record = [&](int64_t r) {
            if (dg == 0xffffffffu) return;
            const uint32_t w = list[fresh(tid) >> ishift];
            const int64_t m = m0 + lq;
            const int64_t row = r * 2 * N + (int64_t)site[w & 0xffu];
            if (m < Mc) {
#pragma unroll
                for (int s = 0; s < SPT; ++s)
                    Xrec[(row + (SPT == 2 ? s : ls) * N) * Mc + m] = (double)y[0][s].x;
            }
        };
        auto store_state = [&](G* out) {
#pragma unroll
            for (int v = 0; v < 2 * U; ++v)
#pragma unroll
                for (int s = 0; s < SPT; ++s) {
                    int64_t off;
                    bool tr;
                    if (state_at(v, s, off, tr)) {
                        G w;
                        w.x = y[v][s].x;
                        w.y = tr ? -y[v][s].y : y[v][s].y;
                        out[off] = w;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        record(0);

        const T tw = scalar_real<T>(E.t), Uw = GINT ? (T)1 : scalar_real<T>(E.U);
        const T c_half = scalar_real<T>(0.5 * A.dt), c_full = scalar_real<T>(A.dt);
        const T c_sixth = scalar_real<T>(A.dt / 6.0);
        int64_t step = 0;

        // an element's operands: its neighbours, the differences d_i - d_j and
        // v_i - v_j, the ratios of its two sites
        struct In {
            C c[3][SPT], r[3][SPT];
            C di, dj;
            T vi, vj;
            C wc[HOP ? 3 : 1], wr[HOP ? 3 : 1];
        };
        auto fetch = [&](int v, uint32_t dcopy, uint32_t wcopy) -> In {
            In in;
            const uint32_t di = addr(v, kDi), dj = addr(v, kDj);
            if constexpr (SPT == 2) {
                in.di = lds_get<C>(di + dcopy);
                in.dj = lds_get<C>(dj + dcopy);
            } else {
                in.di.x = lds_get<T>(di + dcopy);
                in.dj.x = lds_get<T>(dj + dcopy);
            }
            if constexpr (POT) {
                in.vi = lds_get<T>(di + 2 * kDg);
                in.vj = lds_get<T>(dj + 2 * kDg);
            }
            if constexpr (HOP) {
                const uint32_t oc = (wo[v] & 0xffffu) + wcopy, orr = (wo[v] >> 16) + wcopy;
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    in.wc[n] = lds_get<C>(oc + n * CB);
                    in.wr[n] = lds_get<C>(orr + n * CB);
                }
            }
#pragma unroll
            for (int n = 0; n < 3; ++n) {
                get(addr(v, kC + n), in.c[n]);
                get(addr(v, kR + n), in.r[n]);
            }
            return in;
        };
        // sum over three neighbours: (v0 + v1) + v2, with complex hopping of
        // w_n v_n (w already conjugated where needed)
        auto sum3 = [&](const C (*x)[SPT], const C* w, C* out) {
#pragma unroll
            for (int s = 0; s < SPT; ++s) {
                C v[3];
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    v[n] = x[n][s];
                    if constexpr (HOP) {
                        v[n].x = fma_rn<T>(w[n].x, x[n][s].x, -(w[n].y * x[n][s].y));
                        v[n].y = fma_rn<T>(w[n].x, x[n][s].y, w[n].y * x[n][s].x);
                    }
                }
                out[s].x = (v[0].x + v[1].x) + v[2].x;
                out[s].y = (v[0].y + v[1].y) + v[2].y;
            }
        };
        // one Runge-Kutta stage update (as rk_update of the other kernels)
        auto update = [&](auto stage_tag, T c, C k, C& yv, C& av) -> C {
            constexpr int STAGE = decltype(stage_tag)::value;
            if constexpr (STAGE == 1) {
                av = k;
            } else if constexpr (STAGE < 4) {
                av.x = fma_rn<T>((T)2, k.x, av.x);
                av.y = fma_rn<T>((T)2, k.y, av.y);
            } else {
                av.x = av.x + k.x;
                av.y = av.y + k.y;
            }
            C n;
            if constexpr (STAGE < 4) {
                n.x = fma_rn<T>(c, k.x, yv.x);
                n.y = fma_rn<T>(c, k.y, yv.y);
            } else {
                yv.x = fma_rn<T>(c, av.x, yv.x);
                yv.y = fma_rn<T>(c, av.y, yv.y);
                n = yv;
            }
            return n;
        };
        // slot v's next stage input into Y[v]
        auto element = [&](auto stage_tag, auto even_tag, int v, In& in, T c, T Aw) {
            constexpr bool EVEN = decltype(even_tag)::value;
            const uint32_t sgn = EVEN ? (uint32_t)fresh((int)neg[v < U ? v : 0]) : 0u;
            if constexpr (HOP) {
                // odd: w_b x and conj(w_a) x; even: conj(row) takes w_a too,
                // and a BB element the conjugates
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    if (EVEN) {
                        in.wc[n].y = flip(in.wc[n].y, sgn);
                        in.wr[n].y = flip(in.wr[n].y, sgn);
                    } else {
                        in.wr[n].y = -in.wr[n].y;
                    }
                }
            }
            T d[SPT];  // d_i - d_j of the other spin
            if constexpr (SPT == 2) {
                d[0] = in.di.y - in.dj.y;
                d[SPT - 1] = in.di.x - in.dj.x;
            } else {
                d[0] = in.di.x - in.dj.x;
            }
            C col[SPT], row[SPT];
            sum3(in.c, in.wc, col);
            sum3(in.r, in.wr, row);
#pragma unroll
            for (int s = 0; s < SPT; ++s) {
                T a = GINT ? d[s] : Uw * d[s];
                if constexpr (POT) {
                    if (pot_on) a = a + Aw * (in.vi - in.vj);
                }
                T gx = col[s].x - row[s].x;
                T gy = EVEN ? col[s].y + row[s].y : col[s].y - row[s].y;
                if constexpr (!T1) {
                    gx = tw * gx;
                    gy = tw * gy;
                }
                C k;
                k.y = fma_rn<T>(a, Y[v][s].x, gx);
                k.x = -fma_rn<T>(a, Y[v][s].y, gy);
                Y[v][s] = update(stage_tag, EVEN ? flip(c, sgn) : c, k, y[v][s], acc[v][s]);
                settle(acc[v][s]);
            }
        };

        auto run_stage = [&](auto stage_tag) {
            constexpr int STAGE = decltype(stage_tag)::value;
            constexpr uint32_t par = (STAGE - 1) & 1;
            const T c = STAGE <= 2 ? c_half : (STAGE == 3 ? c_full : c_sixth);
            const uint32_t dcopy = (GINT ? 2 * kDg : 0) + par * kDg;
            // the ratio tables of even half steps are in buffer 0, of odd ones in 1
            const uint32_t wcopy =
                HOP ? wtab + (STAGE == 2 || STAGE == 3 ? (uint32_t)(6 * N) * TB : 0u) : 0u;
            T Aw = 0;
            if constexpr (POT) {
                Aw = Anext;
                // next stage: t_n + h/2 (after 1 and 2), t_n + h (after 3 and 4)
                if (pot_on) Anext = scalar_real<T>(venv[2 * step + (STAGE <= 2 ? 1 : 2)]);
            }
            if constexpr (HOP) {
                if (STAGE == 1) ratios_load(2 * step + 1);
                if (STAGE == 3) ratios_load(2 * step + 2);
            }
            // ---- even elements
#pragma unroll
            for (int u = 0; u < U; ++u) {
                put(addr(u, kOwn), Y[u], false);
                put(addr(u, kOwn2), Y[u], true);
            }
            // (PF: the next slot's reads are issued before this one's arithmetic)
            In in = fetch(0, dcopy, wcopy);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                In nx = in;
                if (PF && u + 1 < U) nx = fetch(u + 1, dcopy, wcopy);
                __builtin_amdgcn_sched_barrier(0);
                element(stage_tag, std::true_type{}, u, in, c, Aw);
                if (u == 0) put_diag((par ^ 1) * kDg, Y[0]);
                __builtin_amdgcn_sched_barrier(0);
                if (!PF && u + 1 < U) nx = fetch(u + 1, dcopy, wcopy);
                in = nx;
            }
            phase_barrier<MAXT>();
            // ---- odd elements (GINT: D of the next stage meanwhile)
            in = fetch(U, dcopy, wcopy);
#pragma unroll
            for (int u = U; u < 2 * U; ++u) {
                In nx = in;
                if (PF && u + 1 < 2 * U) nx = fetch(u + 1, dcopy, wcopy);
                __builtin_amdgcn_sched_barrier(0);
                element(stage_tag, std::false_type{}, u, in, c, Aw);
                put(addr(u, kOwn), Y[u], false);
                __builtin_amdgcn_sched_barrier(0);
                if (!PF && u + 1 < 2 * U) nx = fetch(u + 1, dcopy, wcopy);
                in = nx;
            }
            if constexpr (HOP) {
                if (STAGE == 1) ratios_store(1);
                if (STAGE == 3) ratios_store(0);
            }
            phase_barrier<MAXT>();
        };

        int64_t rec = 0;
        int left = A.record_every;  // steps to the next record
        for (; step < A.n_steps; ++step) {
            run_stage(std::integral_constant<int, 1>{});
            run_stage(std::integral_constant<int, 2>{});
            run_stage(std::integral_constant<int, 3>{});
            run_stage(std::integral_constant<int, 4>{});
            if (--left == 0) {
                left = A.record_every;
                record(++rec);
                if constexpr (!T1) {
                    G* const dump = reinterpret_cast<G*>(scalar_ptr(E.dump));
                    if (dump) store_state(dump + (rec - 1) * E.dump_stride);
                }
            }
        }
        store_state(rho);
    }
}

// One wave has no room for the interaction's waves.
template <typename T, int U, int SPT, int MAXT, int MINW, bool PF, bool PK, bool T1>
constexpr const void* shared_gint_fn() {
    if constexpr (MAXT > 64)
        return (const void*)&rk4_shared<T, U, SPT, MAXT, MINW, PF, PK, T1, kSharedGint>;
    else
        return nullptr;
}

#define FTWA_SHARED_KERNELS(T, U, SPT, MAXT, MINW, PF, PK, T1)                       \
    {(const void*)&rk4_shared<T, U, SPT, MAXT, MINW, PF, PK, T1, kSharedPlain>,      \
     (const void*)&rk4_shared<T, U, SPT, MAXT, MINW, PF, PK, T1, kSharedPot>,        \
     (const void*)&rk4_shared<T, U, SPT, MAXT, MINW, PF, PK, T1, kSharedHop>,        \
     shared_gint_fn<T, U, SPT, MAXT, MINW, PF, PK, T1>()}
#define FTWA_SHARED(T, DT, U, SPT, MAXT, MINW, PF, PK)                               \
    SharedShape{DT, U, SPT, MAXT, PK, FTWA_SHARED_KERNELS(T, U, SPT, MAXT, MINW, PF, PK, false), \
                FTWA_SHARED_KERNELS(T, U, SPT, MAXT, MINW, PF, PK, true)}

}  // namespace ftwa
