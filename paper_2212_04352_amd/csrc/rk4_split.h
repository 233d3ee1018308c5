// rk4_split.h -- resident kernel of spin blocks too large for one CU.
#pragma once

#include "rk4_resident.h"

namespace ftwa {

// Pause between two looks at stale flags, in units of 64 cycles.
constexpr int kSplitSleep = 1;

// ---------------------------------------------------------------- split kernel
// A spin block too large for one CU (the 198-site block in FP64: 315 KB)
// spread over G workgroups ("parts") placed on one XCD: part p owns the stored
// elements of a strip of rows (sites in rank order, strips of nearly equal
// element count) and keeps, besides its own elements, the "halo" its stencils
// read from the neighbouring strips in LDS.  Every stage each part publishes
// the next values of its exported elements (those another part reads, and
// the diagonal, which the other spin's parts read for the U term) in a
// per-part area of global memory (two areas alternating by stage parity) and
// copies in its halo and the partner spin's diagonal.
//
// Every wave of every part has a flag per class: the last stage whose even
// (odd) exports it has published.  It raises the even flag a slot after its
// last export, when the stores have reached the L2 anyway, the odd flag at
// once, and no barrier is spent on it.  A reader looks at the flags of all members (one load, a
// flag per lane) a slot before it needs them, then reads the values, two
// 8-byte words each in FP64, while it computes the following slots.  The XCD's
// L2 is what the members share: they compare their XCDs once per launch, and
// where all are one, published words stop at the L2 (`near`) instead of being
// written through to memory.  That rests on this chip, not on the memory model
// (which asks for agent scope between workgroups): one L2 per XCD, first-level
// caches that write through to it, and a store counted off by vmcnt once the L2
// has it.  Otherwise the stores, the fences and the loads are those of the agent
// scope.
//
// No word is overwritten before it is read: a part publishes into an area
// again two stages later, after it has waited there for the odd flags of all
// parts of its spin for the stage between (by then these have landed both
// halos of the area's stage) and before that for the even flags of all
// members (the other spin's parts have then read the area's diagonal).
// Waits are bounded.
//
// The two-phase stage stays, with the waits placed where their data has had
// the most time to arrive: the even elements of a part are ordered interior
// (they read no other part's element) before boundary (the diagonal and the
// exported ones), exported odd elements come first in theirs.  The odd halo
// is read during the last interior slot and landed before the boundary ones;
// the even halo of the next stage and the partner's diagonal are read during
// the last odd slots and landed at the end of the stage.
//
// What bounds it: a stage's chain of element slots and exchanges, not the
// ALUs (VALU busy about 40 %).  198 sites, 512 trajectories, 50 steps: 14.2 ms,
// 1.8e6 trajectory-steps/s, 5.4 us a stage and group; 27.5 ms before, when
// every 32-bit word carried its stage number and was written through to
// memory (twice the bytes, four loads and stores an element, and a wait for
// the stores' round trip at every descriptor behind them).  150 sites, 500
// trajectories: 8.7 -> 7.2 ms.  Reading an element ahead spills (198 sites 17.7
// ms, 150 sites 13.8 ms).

template <int SH> __device__ __forceinline__ uint32_t b2_shl(uint32_t w) {
    uint32_t r;
    __asm__("v_lshlrev_b32_sdwa %0, %2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
            "src1_sel:BYTE_2" : "=v"(r) : "v"(w), "i"(SH));
    return r;
}
template <int SH> __device__ __forceinline__ uint32_t b3_shl(uint32_t w) {
    uint32_t r;
    __asm__("v_lshlrev_b32_sdwa %0, %2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
            "src1_sel:BYTE_3" : "=v"(r) : "v"(w), "i"(SH));
    return r;
}

// Compact descriptor of the split kernel: slot numbers x 2^SH bytes, diagonal
// positions x 2^DSH bytes; xp (constant once the slot loop is unrolled): the
// own field may carry the export flag (bit 15).
template <int SH, int DSH, bool GEN>
__device__ __forceinline__ Stencil decode_split(const uint4& w, bool xp) {
    Stencil e;
    const uint32_t f[3] = {w.x, w.y, w.z};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if constexpr (GEN) {
            e.n[2 * k] = ((f[k] & 0x7fffu) << SH) | ((f[k] & 0x8000u) << 16);
            e.n[2 * k + 1] = (((f[k] >> 16) & 0x7fffu) << SH) | (f[k] & 0x80000000u);
        } else {
            e.n[2 * k] = lo16_shl<SH>(f[k]);
            e.n[2 * k + 1] = hi16_shl<SH>(f[k]);
        }
    }
    e.own = xp ? (w.w & 0x7fffu) << SH : lo16_shl<SH>(w.w);
    e.di = b2_shl<DSH>(w.w);
    e.dj = b3_shl<DSH>(w.w);
    return e;
}

template <typename T, bool OWN_REG, bool T1, int SH, int DSH, bool POT = false, bool HOP = false>
__device__ __forceinline__ cplx_t<T> element_rhs_split(bool gen, bool xp, const unsigned char* Yb,
                                                       const unsigned char* Yd, const uint4& d,
                                                       T t, T U, cplx_t<T> own,
                                                       const unsigned char* Vd = nullptr,
                                                       T Aw = 0, bool pot_on = false,
                                                       HopTab Wt = {}) {
    return gen ? element_rhs<T, OWN_REG, true, T1, POT, HOP>(Yb, Yd, decode_split<SH, DSH, true>(d, xp),
                                                             t, U, own, Vd, Aw, pot_on, Wt)
               : element_rhs<T, OWN_REG, false, T1, POT, HOP>(Yb, Yd,
                                                              decode_split<SH, DSH, false>(d, xp),
                                                              t, U, own, Vd, Aw, pot_on, Wt);
}

// What an element's right-hand side reads from LDS, all of it issued before
// the first sum.
template <typename T> struct ElemIn {
    cplx_t<T> n[6], own;
    T di, dj, vi, vj;
};

template <typename T, bool OWN, int SH, int DSH, bool POT>
__device__ __forceinline__ void read_elem(ElemIn<T>& in, bool gen, bool xp, const unsigned char* Yb,
                                          const unsigned char* Yd, const unsigned char* Vd,
                                          const uint4& d) {
    const Stencil e = gen ? decode_split<SH, DSH, true>(d, xp) : decode_split<SH, DSH, false>(d, xp);
#pragma unroll
    for (int k = 0; k < 6; ++k)
        in.n[k] = gen ? lds_at<T>(Yb, e.n[k]) : *reinterpret_cast<const cplx_t<T>*>(Yb + e.n[k]);
    in.di = *reinterpret_cast<const T*>(Yd + e.di);
    in.dj = *reinterpret_cast<const T*>(Yd + e.dj);
    if constexpr (OWN) in.own = *reinterpret_cast<const cplx_t<T>*>(Yb + e.own);
    if constexpr (POT) {
        in.vi = *reinterpret_cast<const T*>(Vd + e.di);
        in.vj = *reinterpret_cast<const T*>(Vd + e.dj);
    }
}

// element_rhs of those values (the same operations in the same order).
template <typename T, bool T1, bool POT>
__device__ __forceinline__ cplx_t<T> rhs_elem(const ElemIn<T>& in, bool gen, const uint4& d, T t, T U,
                                              cplx_t<T> rho, T Aw, bool pot_on) {
    using C = cplx_t<T>;
    const C *c = in.n, *r = in.n + 3;
    C col, row;
    col.x = (c[0].x + c[1].x) + c[2].x;
    row.x = (r[0].x + r[1].x) + r[2].x;
    if (gen) {
        const uint32_t f[6] = {d.x << 16, d.x, d.y << 16, d.y, d.z << 16, d.z};
        T q[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) q[k] = conj_sign<T>(f[k]);
        col.y = fma_rn<T>(q[2], c[2].y, fma_rn<T>(q[1], c[1].y, q[0] * c[0].y));
        row.y = fma_rn<T>(q[5], r[2].y, fma_rn<T>(q[4], r[1].y, q[3] * r[0].y));
    } else {
        col.y = (c[0].y + c[1].y) + c[2].y;
        row.y = (r[0].y + r[1].y) + r[2].y;
    }
    T a = U * (in.di - in.dj);
    if constexpr (POT) {
        if (pot_on) a = a + Aw * (in.vi - in.vj);
    }
    if constexpr (T1) {
        C k;
        const T gr = fma_rn<T>(a, rho.x, col.x - row.x);
        const T gi = fma_rn<T>(a, rho.y, col.y - row.y);
        k.x = -gi;
        k.y = gr;
        return k;
    }
    return rhs_element<T>(col, row, rho, t, a);
}

// A value as published 64-bit words and back.
template <typename T> struct Payload {
    static constexpr int W = (int)sizeof(cplx_t<T>) / 8;
    uint64_t w[W];
};
template <typename T> __device__ __forceinline__ Payload<T> to_payload(cplx_t<T> v) {
    return __builtin_bit_cast(Payload<T>, v);
}
template <typename T> __device__ __forceinline__ cplx_t<T> from_payload(const Payload<T>& p) {
    return __builtin_bit_cast(cplx_t<T>, p);
}
// The real part from the first word.
__device__ __forceinline__ void real_of(uint64_t w, double& x) { x = __longlong_as_double((long long)w); }
__device__ __forceinline__ void real_of(uint64_t w, float& x) { x = __uint_as_float((uint32_t)w); }

// A published word: a wave-uniform base, opaque so that it stays in scalar
// registers, and a 32-bit byte offset; loads and stores take both as they are.
#if defined(__HIP_DEVICE_COMPILE__)
#define FTWA_GLOBAL __attribute__((address_space(1)))
#else
#define FTWA_GLOBAL  // host pass of the kernel source only
#endif
template <typename V> __device__ __forceinline__ FTWA_GLOBAL V* published(V* base, uint32_t at) {
    uint64_t b = uniform64((uint64_t)base);
    __asm__("" : "+s"(b));
    return (FTWA_GLOBAL V*)(b + at);
}
template <typename V> __device__ __forceinline__ V peek(V* base, uint32_t at) {
    return __hip_atomic_load(published(base, at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// `near`: every workgroup of the group runs on this XCD, so the word need go
// no further than the L2 they share (a round trip between two workgroups
// takes 0.6 of the one through memory).
template <typename V>
__device__ __forceinline__ void poke(V* base, uint32_t at, V v, bool near) {
    if (near)
        __hip_atomic_store(published(base, at), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else
        __hip_atomic_store(published(base, at), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The XCD this wave runs on.
__device__ __forceinline__ uint32_t xcc_id() {
    uint32_t v;
    __asm__ volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
    return v & 15u;
}

// Whether the 2G workgroups of a group run on one XCD, whose L2 they then
// share: each leaves its XCD in a word (zero before the launch) and reads the
// others'.  Bounded: a member that does not come counts as elsewhere.
template <int G>
__device__ __forceinline__ bool same_xcd(uint64_t* ids, int member, unsigned limit) {
    const uint32_t mine = xcc_id();
    const int lane = (int)(threadIdx.x & 63);
    if (threadIdx.x == 0)
        __hip_atomic_store(ids + member, (1ull << 32) | mine, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    uint64_t w = lane < 2 * G ? 0 : (1ull << 32) | mine;
    for (unsigned it = 0; w == 0 && it < limit; ++it) w = peek(ids, (uint32_t)lane * 8u);
    return __all(w == ((1ull << 32) | mine));
}

// T1: every instance of the launch has t = 1.  Even slots: interior elements
// in u < UB (the first GE1 slots read transposes), boundary elements from UB
// (the diagonal first; slots UB .. UB + GE2 - 1 read transposes); odd slots:
// the first GO read transposes, exported elements in the first XO.  KB: halo
// entries per thread and class whose reads are in flight at once.  POT: entries may
// carry an external potential (its profile after the two diagonal copies, in
// their layout; the element slots follow it).  GINT: every entry carries a
// general interaction u_ij (ResidentInst::umat, as the spin-split kernels
// read it): every part forms D_i = sum_k u_ki (d_k + 1/2) for all sites at
// the start of each stage from the partner's whole diagonal (which every
// part receives), into LDS after the diagonal copies, and the U factor of an
// element is D_i - D_j (U = 1 exactly).  HOP: every entry carries complex
// hopping (ResidentInst::hop, as the spin-split kernels read it); each stage
// keeps the whole ratio table of its time in LDS after the diagonal copies.
template <typename T, int G, int NTU, int UE, int UO, int UB, int GE1, int GE2, int GO, int XO,
          int KB, bool T1, bool POT = false, bool GINT = false, bool HOP = false>
__global__ __launch_bounds__(NTU) void rk4_split(ResidentArgs A) {
    using C = cplx_t<T>;
    constexpr int CB = (int)sizeof(C);
    constexpr int TB = (int)sizeof(T);
    constexpr int SH = CB == 8 ? 3 : 4;   // slot number -> byte offset
    constexpr int DSH = TB == 4 ? 2 : 3;  // diagonal position -> byte offset
    constexpr int W = Payload<T>::W;      // published words per element
    constexpr int NW = NTU / 64;          // waves
    constexpr int kEnt = NTU * (UE + UO); // descriptor entries of a part
    constexpr int kPlane = kEnt + kSplitPlanePad;  // published words of one kind (the first
                                                   // after kEnt takes what nobody reads)
    constexpr int kEvenPad = NTU * UE;
    constexpr uint32_t kDiagCopy = 256 * TB;
    static_assert(UB >= 2 && GE1 <= UB && UB < UE && UB + GE2 <= UE && GO <= UO && XO <= UO,
                  "slot groups within their class");
    static_assert((POT ? 1 : 0) + (GINT ? 1 : 0) + (HOP ? 1 : 0) <= 1,
                  "one of a potential, a general interaction and complex hopping");
    extern __shared__ __align__(16) unsigned char smem[];
    (void)smem;
    const int tid0 = threadIdx.x;
    // An earlier launch of this run gave up: nothing to wait for.  One thread
    // looks and the workgroup leaves as one, also where another group gives up
    // meanwhile.
    {
        int& gave_up = *reinterpret_cast<int*>(lds_ptr(A.tail_off + (NTU / 64) * 2 * 8));
        if (tid0 == 0)
            gave_up = __hip_atomic_load(A.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(gave_up)) return;
    }

    // groups of 2G workgroups on one XCD (blocks b = xcd + 8 k; members k =
    // 2G c .. 2G c + 2G - 1): spin = member / G, part = member % G; the
    // groups take items (trajectories) in the same order
    const int b = blockIdx.x, xcd = b % 8, k = b / 8;
    const int member = k % (2 * G);
    const int spin0 = member / G, part = member % G;
    const int group = (k / (2 * G)) * 8 + xcd;
    const int64_t n_groups = gridDim.x / (2 * G);
    // published words of this group: [2 spins][G parts][2 parities][W][kPlane],
    // the stage every wave of every member has published its even and its
    // odd elements of, then every member's XCD; a byte offset holds a member's
    // area and element (parity 0)
    static_assert(2 * G * NW <= 64, "a flag per lane");
    uint64_t* const xg = A.mailbox + (size_t)group * (2 * G * 2 * kPlane * W + kSplitSyncWords);
    uint32_t* const flags = reinterpret_cast<uint32_t*>(xg + (size_t)2 * G * 2 * kPlane * W);
    auto xbase = [&](uint32_t stamp) { return xg + (size_t)(stamp & 1) * kPlane * W; };
    auto xword = [&](int spin, uint32_t qs) {
        return ((uint32_t)((spin * G + (int)(qs >> 16)) * 2 * kPlane * W) + (qs & 0xffffu)) * 8u;
    };
    const bool near =
        !A.far && same_xcd<G>(xg + (size_t)2 * G * 2 * kPlane * W + 64, member, A.spin_limit);
    int64_t g = 0;  // stage counter (continues across items)

    C y[UE + UO], acc[UE + UO], hold[UE];

    for (int64_t item = group; item < A.n_items; item += n_groups) {
        const int t = tid0;
        const uint32_t toff = (uint32_t)t * 16u;
        int ent = 0;
        while (ent + 1 < A.n_entries && A.table[ent + 1].item0 <= item) ++ent;
        ent = __builtin_amdgcn_readfirstlane(ent);
        const ResidentInst& E = A.table[ent];
        const int N = E.N;
        const int P = E.P;
        const int pw = __builtin_amdgcn_readfirstlane(E.part_words);
        const int hmax = __builtin_amdgcn_readfirstlane(E.hmax);
        const uint32_t* const blob = reinterpret_cast<const uint32_t*>(uniform64((uint64_t)E.desc));
        const uint32_t* const pb = blob + (size_t)part * pw;
        const int n_own = __builtin_amdgcn_readfirstlane((int)pb[1]);
        const int n_ie = __builtin_amdgcn_readfirstlane((int)pb[2]);
        const int n_io = __builtin_amdgcn_readfirstlane((int)pb[3]);
        const int n_diag = __builtin_amdgcn_readfirstlane((int)pb[4]);
        gdesc_t desc = (gdesc_t)uniform64((uint64_t)(pb + 8));
        const uint32_t* const pord = pb + 8 + 4 * kEnt;
        const uint32_t* const imp = pord + kEnt;
        const uint32_t* const dsite = imp + hmax;
        const uint32_t* const dsrc = blob + (size_t)G * pw;
        // LDS: two copies of the partner's diagonal (sublattice-major), then
        // the potential's profile (POT) or D and two site-ordered copies of
        // h_k = d_k + 1/2, zero from N up to the u table's row count (GINT),
        // then the part's elements; HOP: the stage's ratio table (256 places)
        // in place of those
        constexpr uint32_t kYb = HOP ? 2 * kDiagCopy + 256 * 6 * TB : (GINT ? 5 : POT ? 3 : 2) * kDiagCopy;
        unsigned char* const Yb = lds_ptr(kYb);
        unsigned char* const dpart = lds_ptr(0);
        // byte offsets at which the halo elements are published: in LDS where
        // it has room for them (a stage's first reads then wait for no other
        // load), else formed from the table in global memory
        const uint32_t imp_at = kYb + (uint32_t)(n_own + n_ie + n_io + 33) * CB;
        uint32_t* const himp = reinterpret_cast<uint32_t*>(lds_ptr(imp_at));
        const bool imp_lds = imp_at + (uint32_t)(n_ie + n_io) * 4u <= A.tail_off;
        auto import_at = [&](int h) { return imp_lds ? himp[h] : xword(spin0, imp[h]); };
        auto hsite = [&](int c) { return reinterpret_cast<T*>(lds_ptr((3 + c) * kDiagCopy)); };
        int& abort_flag = *reinterpret_cast<int*>(lds_ptr(A.tail_off + (NTU / 64) * 2 * 8));
        const int64_t Mc = E.Mc;
        const int64_t m = item - E.item0;
        const bool active = m < Mc;
        C* const rho = reinterpret_cast<C*>(uniform64((uint64_t)E.rho));
        const int64_t ldr = E.ldr;
        double* const Xrec = E.X;
        auto own_slot_at = [&](gdesc_t dt, int e) -> uint32_t {
            return reinterpret_cast<const uint4*>((uint64_t)dt)[e].w & 0x7fffu;
        };
        // packed index of stored element a | b << 16 (conjugated when b < a)
        auto packed_ab = [&](uint32_t ab, bool& transposed) -> int64_t {
            const int a = (int)(ab & 0xffffu), bb = (int)(ab >> 16);
            const int i = a < bb ? a : bb, j = a < bb ? bb : a;
            transposed = a > bb;
            return (int64_t)i * N - (int64_t)i * (i - 1) / 2 + (j - i);
        };
        auto load_elem = [&](uint32_t ab) -> C {
            C v;
            v.x = 0;
            v.y = 0;
            if (active) {
                bool tr;
                const int64_t p = packed_ab(ab, tr);
                v = rho[((int64_t)spin0 * P + p) * ldr + m];
                if (tr) v.y = -v.y;
            }
            return v;
        };
        __syncthreads();  // the previous item is done with LDS

        // ---- the trajectory's own elements, the halo, the zero and scratch
        // slots, and the partner's diagonal
#pragma unroll
        for (int u = 0; u < UE + UO; ++u) {
            const int e = u < UE ? t + NTU * u : kEvenPad + t + NTU * (u - UE);
            const uint32_t own = own_slot_at(desc, e);
            C v;
            v.x = 0;
            v.y = 0;
            if (own < (uint32_t)n_own) v = load_elem(pord[own]);
            reinterpret_cast<C*>(Yb)[own] = v;
            y[u] = v;
            acc[u] = v;
            if (u < UE) hold[u] = v;
        }
        for (int h = t; h < n_ie + n_io; h += NTU) {
            const uint32_t qs = imp[h];
            const uint32_t* const pq = blob + (size_t)(qs >> 16) * pw + 8 + 4 * kEnt;
            reinterpret_cast<C*>(Yb)[n_own + h] = load_elem(pq[qs & 0xffffu]);
            if (imp_lds) himp[h] = xword(spin0, qs);
        }
        // this thread's site of the partner's diagonal: where it is published,
        // and its position
        const uint32_t dia_w = t < N ? xword(1 - spin0, dsrc[t]) : 0u;
        if (t < 33) {
            C z;
            z.x = 0;
            z.y = 0;
            reinterpret_cast<C*>(Yb)[n_own + n_ie + n_io + t] = z;
        }
        const int32_t* const dpos = reinterpret_cast<const int32_t*>(uniform64((uint64_t)E.dpos));
        for (int i = t; i < N; i += NTU) {
            const int64_t p = (int64_t)i * N - (int64_t)i * (i - 1) / 2;
            const int q = dpos[i];
            reinterpret_cast<T*>(dpart + (size_t)(g & 1) * kDiagCopy)[q] =
                active ? rho[((int64_t)(1 - spin0) * P + p) * ldr + m].x : (T)0;
            reinterpret_cast<T*>(dpart + (size_t)((g + 1) & 1) * kDiagCopy)[q] = (T)0;
            if constexpr (GINT) {
                hsite((int)(g & 1))[i] =
                    (active ? rho[((int64_t)(1 - spin0) * P + p) * ldr + m].x : (T)0) + (T)0.5;
                hsite((int)((g + 1) & 1))[i] = (T)0;
            }
        }
        if constexpr (GINT) {
            for (int i = N + t; i < umat_rows(N); i += NTU) {
                hsite(0)[i] = (T)0;
                hsite(1)[i] = (T)0;
            }
        }
        // general interaction: u in T, blocked by four along k
        const T* const utab = GINT ? reinterpret_cast<const T*>(uniform64((uint64_t)E.umat)) : nullptr;
        // complex hopping: the prepared ratio tables, [2 n_steps + 1][N][3]
        const unsigned char* const hop_tab =
            HOP ? reinterpret_cast<const unsigned char*>(uniform64((uint64_t)E.hop)) : nullptr;
        // external potential of this entry: the profile v (zero without one)
        // and the envelope, read per stage
        const double* const venv = POT ? reinterpret_cast<const double*>(uniform64((uint64_t)E.v_env))
                                       : nullptr;
        const bool pot_on = POT && E.v_site != nullptr;
        unsigned char* const vpart = lds_ptr(2 * kDiagCopy);
        if constexpr (POT) {
            const double* const vs = reinterpret_cast<const double*>(uniform64((uint64_t)E.v_site));
            for (int i = t; i < N; i += NTU)
                reinterpret_cast<T*>(vpart)[dpos[i]] = pot_on ? (T)vs[i] : (T)0;
        }
        int64_t cur_step = 0;  // index of the step being taken (the envelope's sample 2 cur_step)
        // records: boundary entry t < n_diag (slot UB) is the diagonal element
        // of site dsite[t]
        auto record = [&](int64_t r) {
            if (active && t < n_diag)
                Xrec[(r * 2 * N + (int64_t)spin0 * N + (int64_t)dsite[t]) * Mc + m] = (double)y[UB].x;
        };
        record(0);
        __syncthreads();

        const T tw = uniform_real<T>((T)E.t), Uw = uniform_real<T>((T)E.U);
        const T c_half = uniform_real<T>((T)(0.5 * A.dt));
        const T c_full = uniform_real<T>((T)A.dt);
        const T c_sixth = uniform_real<T>((T)(A.dt / 6.0));
        bool first = true;  // the item's first stage: its halo came from HBM

        // This wave has published its elements of class CLS for stage `stamp`:
        // its stores are in the L2 (in memory, where the group is not near).
        auto signal = [&](int cls, uint32_t stamp) {
            if (near) __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
            else __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            if ((t & 63) == 0) poke(flags, (uint32_t)(cls * 64 + member * NW + t / 64) * 4u, stamp, near);
        };
        // The flags of a class: of every member (even: the halo and the
        // partner's diagonal), of the members of this spin (odd).
        auto look = [&](int cls) { return peek(flags, (uint32_t)(cls * 64 + (t & 63)) * 4u); };
        auto await = [&](int cls, uint32_t seen, uint32_t want) {
            const int l = t & 63;
            const bool mine = cls == 0 ? l < 2 * G * NW
                                       : l >= spin0 * G * NW && l < (spin0 + 1) * G * NW;
            unsigned it = 0;
            while (!__all(!mine || (int32_t)(seen - want) >= 0)) {
                if (*reinterpret_cast<volatile int*>(&abort_flag)) break;
                if (++it >= A.spin_limit) {
                    abort_flag = 1;
                    if (l == 0) atomicExch(A.error, 1);
                    break;
                }
                __builtin_amdgcn_s_sleep(kSplitSleep);
                seen = look(cls);
            }
            if (near) __asm__ volatile("" ::: "memory");
            else __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        };

        // Halo copies: KB entries of [h0, h1) per thread at a time, read and
        // landed in their slots (further ones, if any, one after another).
        struct Batch {
            uint64_t w[KB][W];
        };
        auto fetch = [&](Batch& bt, int h0, int h1, uint32_t want) {
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                const int h = h0 + t + j * NTU;
                if (h < h1) {
                    const uint32_t at = import_at(h);
#pragma unroll
                    for (int kk = 0; kk < W; ++kk)
                        bt.w[j][kk] = peek(xbase(want) + (size_t)kk * kPlane, at);
                }
            }
        };
        auto land = [&](Batch& bt, int h0, int h1, uint32_t want) {
            for (;;) {
#pragma unroll
                for (int j = 0; j < KB; ++j) {
                    const int h = h0 + t + j * NTU;
                    if (h < h1) {
                        Payload<T> pl;
#pragma unroll
                        for (int kk = 0; kk < W; ++kk) pl.w[kk] = bt.w[j][kk];
                        reinterpret_cast<C*>(Yb)[n_own + h] = from_payload<T>(pl);
                    }
                }
                h0 += KB * NTU;
                if (h0 >= h1) return;
                fetch(bt, h0, h1, want);
            }
        };
        Batch be;  // the even halo of the next stage's input

        auto run_stage = [&](auto stage_tag) -> bool {
            constexpr int STAGE = decltype(stage_tag)::value;
            const T c = STAGE <= 2 ? c_half : (STAGE == 3 ? c_full : c_sixth);
            const unsigned char* dcur = dpart + ((STAGE - 1) & 1) * kDiagCopy;
            // envelope at this stage's time: t_n, t_n + h/2 (twice), t_n + h
            T Aw = 0;
            if constexpr (POT) {
                if (pot_on)
                    Aw = uniform_real<T>((T)venv[2 * cur_step + (STAGE == 1 ? 0 : STAGE == 4 ? 2 : 1)]);
            }
            // general interaction: D of this stage's input from the
            // site-ordered copy (complete: the previous stage ended with a
            // barrier after it landed), one ascending fused chain per site on
            // threads t < N; u blocked by four along k, two 16-byte loads per
            // lane and block (FP64), four blocks in flight; padded terms add
            // exactly +0 (the chain starts at +0 and never holds -0)
            // complex hopping: this stage's ratio table, all of it in LDS
            // (copied when the table changes: stages 2 and 4, and an item's
            // first stage; the previous stage ended with a barrier)
            const HopTab Wt{
                HOP ? hop_tab + (size_t)(2 * cur_step + (STAGE == 1 ? 0 : STAGE == 4 ? 2 : 1)) *
                                    (size_t)N * 3 * CB
                    : nullptr,
                N * 3 * CB, lds_ptr(2 * kDiagCopy), (uint32_t)N * TB};
            if constexpr (HOP) {
                if (STAGE == 2 || STAGE == 4 || cur_step == 0) {
                    const T* src = reinterpret_cast<const T*>(Wt.p);
                    for (int k = t; k < 6 * N; k += NTU)
                        reinterpret_cast<T*>(lds_ptr(2 * kDiagCopy))[k] = src[k];
                    __syncthreads();
                }
            }
            const unsigned char* Ud = dcur;
            T Uu = Uw;
            if constexpr (GINT) {
                if (t < N) {
                    constexpr int B = 4;
                    const int K = umat_rows(N);
                    const T* const hs = hsite((STAGE - 1) & 1);
                    const __amdgpu_buffer_rsrc_t urs = __builtin_amdgcn_make_buffer_rsrc(
                        (void*)utab, (short)0, (int)(K * N * TB), 0x00020000);
                    T accD = 0;
                    for (int k0 = 0; k0 < K; k0 += 4 * B) {
                        double2 ua[B], ub[B];
#pragma unroll
                        for (int b = 0; b < B; ++b) {
                            const int so = (k0 / 4 + b) * N * 32;
                            ua[b] = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(
                                                                    urs, (uint32_t)(t * 32), so, 0));
                            ub[b] = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(
                                                                    urs, (uint32_t)(t * 32 + 16), so, 0));
                        }
#pragma unroll
                        for (int b = 0; b < B; ++b) {
                            const double2 h0 = *reinterpret_cast<const double2*>(hs + k0 + 4 * b);
                            const double2 h1 = *reinterpret_cast<const double2*>(hs + k0 + 4 * b + 2);
                            accD = fma_rn<T>(ua[b].x, h0.x, accD);
                            accD = fma_rn<T>(ua[b].y, h0.y, accD);
                            accD = fma_rn<T>(ub[b].x, h1.x, accD);
                            accD = fma_rn<T>(ub[b].y, h1.y, accD);
                        }
                    }
                    reinterpret_cast<T*>(vpart)[dpos[t]] = accD;
                }
                __syncthreads();
                Ud = vpart;
                Uu = (T)1;
            }
            const uint32_t stamp = (uint32_t)(g + 1);
            uint64_t* const mine = xbase(stamp) + (size_t)(spin0 * G + part) * 2 * kPlane * W;
            desc = launder(desc);
            const __amdgpu_buffer_rsrc_t drs = __builtin_amdgcn_make_buffer_rsrc(
                (void*)desc, (short)0, (int)(kEnt * 16), 0x00020000);
            constexpr int KP = 3;  // descriptors in flight (2: 6 % slower)
            auto entry_of = [](int v) { return v < UE ? NTU * v : kEvenPad + NTU * (v - UE); };
            uint4 dq[KP];
#pragma unroll
            for (int v = 0; v < KP - 1; ++v) dq[v] = slot_desc_buf<uint4>(drs, entry_of(v), toff);
            auto next_desc = [&](int u) {
                if (u + KP - 1 < UE + UO)
                    dq[(u + KP - 1) % KP] = slot_desc_buf<uint4>(drs, entry_of(u + KP - 1), toff);
            };
            auto is_gen = [](int u) {
                return u < UE ? u < GE1 || (u >= UB && u < UB + GE2) : u - UE < GO;
            };
            auto is_xp = [](int u) { return u < UE ? u >= UB : u - UE < XO; };
            ElemIn<T> in;
            auto read = [&](int u) {
                if constexpr (!HOP) {
                    const uint4& d = dq[u % KP];
                    if (u >= UE && STAGE > 1)
                        read_elem<T, true, SH, DSH, POT>(in, is_gen(u), is_xp(u), Yb, Ud, vpart, d);
                    else
                        read_elem<T, false, SH, DSH, POT>(in, is_gen(u), is_xp(u), Yb, Ud, vpart, d);
                }
            };
            // every lane of an exporting slot stores (what is not exported to
            // the spare word), so the loads around it keep exact wait counts
            auto export_elem = [&](const uint4& d, C v) {
                const Payload<T> p = to_payload<T>(v);
                const uint32_t at = d.w & 0x8000u ? (d.w & 0x7fffu) * 8u : (uint32_t)kEnt * 8u;
                if (near) {
#pragma unroll
                    for (int k = 0; k < W; ++k) poke(mine + (size_t)k * kPlane, at, p.w[k], true);
                } else {
#pragma unroll
                    for (int k = 0; k < W; ++k) poke(mine + (size_t)k * kPlane, at, p.w[k], false);
                }
            };
            Batch bo;
            uint32_t fl = 0;
            if (!first) land(be, 0, n_ie, (uint32_t)g);
            // ---------------- phase 1: even elements (next values held)
#pragma unroll
            for (int u = 0; u < UE; ++u) {
                constexpr int UL = UB - 1;
                if (u == UL - 1) fl = look(1);
                if (u == UL && u < UB) {
                    // (also in an item's first stage: no member overwrites
                    // what another has still to read)
                    await(1, fl, (uint32_t)g);
                    if (!first) fetch(bo, n_ie, n_ie + n_io, (uint32_t)g);
                }
                if (u == UB) {
                    // the boundary elements read the odd halo
                    if (!first) land(bo, n_ie, n_ie + n_io, (uint32_t)g);
                    __syncthreads();
                }
                next_desc(u);
                const uint4 d = dq[u % KP];
                const C own = STAGE == 1 ? y[u] : hold[u];
                const bool xp = is_xp(u);
                const uint32_t ob = xp ? (d.w & 0x7fffu) << SH : lo16_shl<SH>(d.w);
                *reinterpret_cast<C*>(Yb + ob) = own;
                read(u);
                __builtin_amdgcn_sched_barrier(0);
                C kk;
                if constexpr (HOP)
                    kk = element_rhs_split<T, true, T1, SH, DSH, POT, HOP>(
                        is_gen(u), xp, Yb, Ud, d, tw, Uu, own, vpart, Aw, pot_on, Wt);
                else
                    kk = rhs_elem<T, T1, POT>(in, is_gen(u), d, tw, Uu, own, Aw, pot_on);
                hold[u] = rk_update<STAGE, T>(c, kk, y[u], acc[u]);
                pin(hold[u]);
                pin(acc[u]);
                if constexpr (STAGE == 4) pin(y[u]);
                if (xp) export_elem(d, hold[u]);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
            // ---------------- phase 2: odd elements (written straight to LDS);
            // the partner's diagonal of the next stage's input is read
            // meanwhile (into the copy this stage does not read)
            uint64_t dw = 0;
            // slots before the end at which the even flags are awaited: with few
            // slots the members' flags need the time (110 sites, (4, 4): one 6.6 ms,
            // two 7.5; 150 sites, (6, 6): 7.35 and 7.30)
            constexpr int AE = UO > 4 ? 2 : 1;
#pragma unroll
            for (int u = UE; u < UE + UO; ++u) {
                if (u == UE + 1) signal(0, stamp);
                if (u == UE + XO) signal(1, stamp);
                if (u == UE + UO - AE - 1) fl = look(0);
                if (u == UE + UO - AE) {
                    // every member is past its phase 1: the partner's diagonal
                    // and the even halo of the next stage's input
                    await(0, fl, stamp);
                    if (t < N) dw = peek(xbase(stamp), dia_w);
                    fetch(be, 0, n_ie, stamp);
                }
                next_desc(u);
                const uint4 d = dq[u % KP];
                const bool xp = is_xp(u);
                read(u);
                __builtin_amdgcn_sched_barrier(0);
                C kk;
                if constexpr (HOP)
                    kk = STAGE == 1
                        ? element_rhs_split<T, true, T1, SH, DSH, POT, HOP>(
                              is_gen(u), xp, Yb, Ud, d, tw, Uu, y[u], vpart, Aw, pot_on, Wt)
                        : element_rhs_split<T, false, T1, SH, DSH, POT, HOP>(
                              is_gen(u), xp, Yb, Ud, d, tw, Uu, y[u], vpart, Aw, pot_on, Wt);
                else
                    kk = rhs_elem<T, T1, POT>(in, is_gen(u), d, tw, Uu,
                                              STAGE == 1 ? y[u] : in.own, Aw, pot_on);
                const C nx = rk_update<STAGE, T>(c, kk, y[u], acc[u]);
                const uint32_t ob = xp ? (d.w & 0x7fffu) << SH : lo16_shl<SH>(d.w);
                *reinterpret_cast<C*>(Yb + ob) = nx;
                pin(acc[u]);
                if constexpr (STAGE == 4) pin(y[u]);
                if (xp) export_elem(d, nx);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (XO >= UO) signal(1, stamp);
            if (t < N) {
                T x;
                real_of(dw, x);
                reinterpret_cast<T*>(dpart + (STAGE & 1) * kDiagCopy)[dpos[t]] = x;
                if constexpr (GINT) hsite(STAGE & 1)[t] = x + (T)0.5;
            }
            __syncthreads();
            ++g;
            first = false;
            return abort_flag == 0;
        };

        auto store_state = [&](C* out) {
            const gdesc_t dl = launder(desc);
            out = reinterpret_cast<C*>(uniform64((uint64_t)out));
            if (!active) return;
#pragma unroll
            for (int u = 0; u < UE + UO; ++u) {
                const int e = u < UE ? t + NTU * u : kEvenPad + t + NTU * (u - UE);
                const uint32_t own = own_slot_at(dl, e);
                if (own < (uint32_t)n_own) {
                    bool tr;
                    const int64_t p = packed_ab(pord[own], tr);
                    C v = y[u];
                    if (tr) v.y = -v.y;
                    out[((int64_t)spin0 * P + p) * ldr + m] = v;
                }
            }
        };

        for (int64_t step = 1; step <= A.n_steps; ++step) {
            cur_step = step - 1;
            if (!run_stage(stage_c<1>{})) return;
            if (!run_stage(stage_c<2>{})) return;
            if (!run_stage(stage_c<3>{})) return;
            if (!run_stage(stage_c<4>{})) return;
            if (step % A.record_every == 0) {
                const int64_t r = step / A.record_every;
                record(r);
                if constexpr (!T1) {
                    C* const dump = reinterpret_cast<C*>(uniform64((uint64_t)E.dump));
                    if (dump) store_state(dump + (r - 1) * E.dump_stride);
                }
            }
        }
        store_state(rho);
    }
}

template <typename T, int G, int NTU, int UE, int UO, int UB, int GE1, int GE2, int GO, int XO,
          int KB>
constexpr const void* split_unit_hop_fn() {
    if constexpr (std::is_same<T, float>::value)
        return (const void*)&rk4_split<T, G, NTU, UE, UO, UB, GE1, GE2, GO, XO, KB, true>;
    else
        return nullptr;
}

#define FTWA_SPLIT_CFG(T, DT, G, NTU, UE, UO, UB, GE1, GE2, GO, XO, KB, AUTO)              \
    Config{DT, 1, NTU, 1, UE, UO, GE1, GO,                                                   \
           (const void*)&rk4_split<T, G, NTU, UE, UO, UB, GE1, GE2, GO, XO, KB, false>,     \
           split_unit_hop_fn<T, G, NTU, UE, UO, UB, GE1, GE2, GO, XO, KB>(), G, UB, GE2, XO, KB, \
           AUTO, (const void*)&rk4_split<T, G, NTU, UE, UO, UB, GE1, GE2, GO, XO, KB, false, true>, \
           nullptr,                                                                          \
           (const void*)&rk4_split<T, G, NTU, UE, UO, UB, GE1, GE2, GO, XO, KB, false, false, false, \
                                   true>,                                                    \
           nullptr,                                                                          \
           (const void*)&rk4_split<T, G, NTU, UE, UO, UB, GE1, GE2, GO, XO, KB, false, false, true>, \
           nullptr}

}  // namespace ftwa
