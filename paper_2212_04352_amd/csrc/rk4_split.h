// rk4_split.h -- resident kernel of spin blocks too large for one CU.
#pragma once

#include "rk4_resident.h"

namespace ftwa {

// ---------------------------------------------------------------- split kernel
// A spin block too large for one CU (the 198-site block in FP64: 315 KB)
// spread over G workgroups ("parts") placed on one XCD: part p owns the stored
// elements of a strip of rows (sites in rank order, strips of nearly equal
// element count) and keeps, besides its own elements, the "halo" its stencils
// read from the neighbouring strips in LDS.  Every stage each part publishes
// the next values of its exported elements (those another part reads, and
// the diagonal, which the other spin's parts read for the U term) into a
// per-part area of global memory, and copies in its halo and the partner
// spin's diagonal.  Every published 32-bit word travels with the number of
// the stage it belongs to in one 64-bit relaxed agent-scope atomic (two
// areas alternating by stage parity), so no fences are needed; a word is
// never overwritten before it is read because the stencil relation is
// symmetric (a part that reads a neighbour's element is read back by it in
// the other class) and the diagonal exchange is all-to-all, so no member of
// a group runs two stages ahead of a reader.  Waits are bounded.
//
// The two-phase stage stays, with the waits placed where their data has had
// the most time to arrive: the even elements of a part are ordered interior
// (they read no other part's element) before boundary (the diagonal and the
// exported ones).  The reads of both halos of a stage's input are issued at
// the start of the stage; the odd halo (published early in the producers'
// previous phase 2: exported odd elements come first) is needed only from the
// boundary slots on, after a barrier; the even halo (published in the
// producers' previous phase 1) before phase 2; the partner's diagonal of the
// next stage's input is read during phase 2.

// Sub-dword-select shifts with the shift as a template argument.
template <int SH> __device__ __forceinline__ uint32_t lo16_shl(uint32_t w) {
    uint32_t r;
    __asm__("v_lshlrev_b32_sdwa %0, %2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
            "src1_sel:WORD_0" : "=v"(r) : "v"(w), "i"(SH));
    return r;
}
template <int SH> __device__ __forceinline__ uint32_t hi16_shl(uint32_t w) {
    uint32_t r;
    __asm__("v_lshlrev_b32_sdwa %0, %2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD "
            "src1_sel:WORD_1" : "=v"(r) : "v"(w), "i"(SH));
    return r;
}
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

// A complex value as 32-bit payload words and back.
template <typename T> struct Payload {
    static constexpr int W = (int)sizeof(cplx_t<T>) / 4;
    uint32_t w[W];
};
template <typename T> __device__ __forceinline__ Payload<T> to_payload(cplx_t<T> v) {
    return __builtin_bit_cast(Payload<T>, v);
}
template <typename T> __device__ __forceinline__ cplx_t<T> from_payload(const Payload<T>& p) {
    return __builtin_bit_cast(cplx_t<T>, p);
}

// Publishes a value: every payload word with the stage number in the high
// half, each a relaxed agent-scope atomic (a reader sees the old or the new
// stage of a word, never a mixture); word k at dst + k * stride (word-major
// areas: the threads of a wave write consecutive words).
template <typename T>
__device__ __forceinline__ void publish(uint64_t* dst, int stride, cplx_t<T> v, uint32_t stamp) {
    const Payload<T> p = to_payload<T>(v);
#pragma unroll
    for (int k = 0; k < Payload<T>::W; ++k)
        __hip_atomic_store(dst + (size_t)k * stride, ((uint64_t)stamp << 32) | p.w[k],
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t peek(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until NW published words carry stage `want`: w[k] was read from
// src[k / WPE] + (k % WPE) * stride (WPE = NW / NP, null pointers are
// skipped); while any word is stale, all of them are read again (one round
// trip per retry).
// Bounded: false (abort flag and error word set) when the stage never comes
// or another wait of the workgroup gave up.
template <int NW, int NP>
__device__ __forceinline__ bool settle_words(const uint64_t* const* src, int stride, uint64_t* w,
                                             uint32_t want, int& abort_flag, int* error,
                                             unsigned limit) {
    constexpr int WPE = NW / NP;
    unsigned it = 0;
    while (true) {
        bool ok = true;
#pragma unroll
        for (int k = 0; k < NW; ++k)
            ok = ok && (src[k / WPE] == nullptr || (uint32_t)(w[k] >> 32) == want);
        if (ok) return true;
        if (*reinterpret_cast<volatile int*>(&abort_flag)) return false;
        if (++it >= limit) {
            abort_flag = 1;
            atomicExch(error, 1);
            return false;
        }
        // ~2000 cycles: polling less often leaves the memory system to the
        // producers (a shorter sleep is slower overall)
        __builtin_amdgcn_s_sleep(32);
#pragma unroll
        for (int k = 0; k < NW; ++k)
            if (src[k / WPE]) w[k] = peek(src[k / WPE] + (size_t)(k % WPE) * stride);
    }
}

// T1: every instance of the launch has t = 1.  Even slots: interior elements
// in u < UB (the first GE1 slots read transposes), boundary elements from UB
// (the diagonal first; slots UB .. UB + GE2 - 1 read transposes); odd slots:
// the first GO read transposes, exported elements in the first XO.  KB: halo
// entries per thread whose reads are issued a phase ahead.  POT: entries may
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
    constexpr int DW = TB / 4;            // words of the real part
    constexpr int kEnt = NTU * (UE + UO); // descriptor entries of a part
    constexpr int kEvenPad = NTU * UE;
    constexpr uint32_t kDiagCopy = 256 * TB;
    static_assert(GE1 <= UB && UB < UE && UB + GE2 <= UE && GO <= UO && XO <= UO,
                  "slot groups within their class");
    static_assert((POT ? 1 : 0) + (GINT ? 1 : 0) + (HOP ? 1 : 0) <= 1,
                  "one of a potential, a general interaction and complex hopping");
    extern __shared__ __align__(16) unsigned char smem[];
    (void)smem;
    const int tid0 = threadIdx.x;

    // groups of 2G workgroups on one XCD (blocks b = xcd + 8 k; members k =
    // 2G c .. 2G c + 2G - 1): spin = member / G, part = member % G; the
    // groups take items (trajectories) in the same order
    const int b = blockIdx.x, xcd = b % 8, k = b / 8;
    const int member = k % (2 * G);
    const int spin0 = member / G, part = member % G;
    const int group = (k / (2 * G)) * 8 + xcd;
    const int64_t n_groups = gridDim.x / (2 * G);
    if (tid0 == 0) *reinterpret_cast<int*>(lds_ptr(A.tail_off + (NTU / 64) * 2 * 8)) = 0;
    // published words of this group: [2 spins][G parts][2 parities][W][kEnt]
    uint64_t* const xg = A.mailbox + (size_t)group * 2 * G * 2 * kEnt * W;
    auto xslot = [&](int spin, int q, uint32_t stamp) {
        return xg + ((size_t)(spin * G + q) * 2 + (stamp & 1)) * kEnt * W;
    };
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
        unsigned char* const Yb =
            lds_ptr(HOP ? 2 * kDiagCopy + 256 * 6 * TB : (GINT ? 5 : POT ? 3 : 2) * kDiagCopy);
        unsigned char* const dpart = lds_ptr(0);
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
        }
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

        // Halo copies: the reads of this thread's first KB entries of [h0, h1)
        // are issued early (issue), the values land in their slots later
        // (land; further entries, if any, are read there).
        struct Batch {
            uint64_t w[KB * W];
            const uint64_t* src[KB];
        };
        auto issue = [&](Batch& bt, int h0, int h1, uint32_t want) {
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                const int h = h0 + t + j * NTU;
                bt.src[j] = nullptr;
                if (h < h1) {
                    const uint32_t qs = imp[h];
                    bt.src[j] = xslot(spin0, (int)(qs >> 16), want) + (qs & 0xffffu);
#pragma unroll
                    for (int kk = 0; kk < W; ++kk) bt.w[j * W + kk] = peek(bt.src[j] + (size_t)kk * kEnt);
                }
            }
        };
        auto land = [&](Batch& bt, int h0, int h1, uint32_t want) {
            for (int hb = h0;; ) {
                if (!settle_words<KB * W, KB>(bt.src, kEnt, bt.w, want, abort_flag, A.error,
                                              A.spin_limit))
                    return;
#pragma unroll
                for (int j = 0; j < KB; ++j) {
                    if (bt.src[j]) {
                        Payload<T> pl;
#pragma unroll
                        for (int kk = 0; kk < W; ++kk) pl.w[kk] = (uint32_t)bt.w[j * W + kk];
                        reinterpret_cast<C*>(Yb)[n_own + hb + t + j * NTU] = from_payload<T>(pl);
                    }
                }
                hb += KB * NTU;
                if (hb >= h1) return;
                issue(bt, hb, h1, want);
            }
        };

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
            uint64_t* const mine = xslot(spin0, part, stamp);
            desc = launder(desc);
            const __amdgpu_buffer_rsrc_t drs = __builtin_amdgcn_make_buffer_rsrc(
                (void*)desc, (short)0, (int)(kEnt * 16), 0x00020000);
            constexpr int KP = 2;
            auto entry_of = [](int v) { return v < UE ? NTU * v : kEvenPad + NTU * (v - UE); };
            uint4 dq[KP];
#pragma unroll
            for (int v = 0; v < KP; ++v) dq[v] = slot_desc_buf<uint4>(drs, entry_of(v < UE + UO ? v : UE + UO - 1), toff);
            // the halo of this stage's input (published in the producers'
            // previous stage): reads issued now, landed before the elements
            // that need them (the odd halo before the boundary, the even halo
            // before phase 2)
            Batch bo, be;
            if (!first) {
                issue(bo, n_ie, n_ie + n_io, (uint32_t)g);
                issue(be, 0, n_ie, (uint32_t)g);
            }
            // ---------------- phase 1: even elements (next values held)
#pragma unroll
            for (int u = 0; u < UE; ++u) {
                if (u == UB) {
                    // the boundary elements read the odd halo
                    if (!first) land(bo, n_ie, n_ie + n_io, (uint32_t)g);
                    __syncthreads();
                }
                const uint4 d = dq[u % KP];
                if (u + KP < UE + UO) dq[u % KP] = slot_desc_buf<uint4>(drs, entry_of(u + KP), toff);
                const C own = STAGE == 1 ? y[u] : hold[u];
                const bool xp = u >= UB;
                const bool gen = u < GE1 || (u >= UB && u < UB + GE2);
                const uint32_t ob = xp ? (d.w & 0x7fffu) << SH : lo16_shl<SH>(d.w);
                *reinterpret_cast<C*>(Yb + ob) = own;
                const C kk = element_rhs_split<T, true, T1, SH, DSH, POT, HOP>(
                    gen, xp, Yb, Ud, d, tw, Uu, own, vpart, Aw, pot_on, Wt);
                hold[u] = rk_update<STAGE, T>(c, kk, y[u], acc[u]);
                pin(hold[u]);
                pin(acc[u]);
                if constexpr (STAGE == 4) pin(y[u]);
                if (xp && (d.w & 0x8000u))
                    publish<T>(mine + (d.w & 0x7fffu), kEnt, hold[u], stamp);
                __builtin_amdgcn_sched_barrier(0);
            }
            // phase 2 reads the even halo
            if (!first) land(be, 0, n_ie, (uint32_t)g);
            __syncthreads();
            // ---------------- phase 2: odd elements (written straight to LDS);
            // the partner's diagonal of the next stage's input is read
            // meanwhile (into the copy this stage does not read)
            const uint64_t* dsrcp[1] = {nullptr};
            uint64_t dw[DW];
            if (t < N) {
                const uint32_t qs = dsrc[t];
                dsrcp[0] = xslot(1 - spin0, (int)(qs >> 16), stamp) + (qs & 0xffffu);
#pragma unroll
                for (int kk = 0; kk < DW; ++kk) dw[kk] = peek(dsrcp[0] + (size_t)kk * kEnt);
            }
#pragma unroll
            for (int u = UE; u < UE + UO; ++u) {
                const uint4 d = dq[u % KP];
                if (u + KP < UE + UO) dq[u % KP] = slot_desc_buf<uint4>(drs, entry_of(u + KP), toff);
                const bool xp = u - UE < XO;
                const bool gen = u - UE < GO;
                const C kk = STAGE == 1
                    ? element_rhs_split<T, true, T1, SH, DSH, POT, HOP>(gen, xp, Yb, Ud, d, tw, Uu,
                                                                        y[u], vpart, Aw, pot_on, Wt)
                    : element_rhs_split<T, false, T1, SH, DSH, POT, HOP>(gen, xp, Yb, Ud, d, tw, Uu,
                                                                         y[u], vpart, Aw, pot_on, Wt);
                const C nx = rk_update<STAGE, T>(c, kk, y[u], acc[u]);
                const uint32_t ob = xp ? (d.w & 0x7fffu) << SH : lo16_shl<SH>(d.w);
                *reinterpret_cast<C*>(Yb + ob) = nx;
                pin(acc[u]);
                if constexpr (STAGE == 4) pin(y[u]);
                if (xp && (d.w & 0x8000u)) publish<T>(mine + (d.w & 0x7fffu), kEnt, nx, stamp);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (t < N && settle_words<DW, 1>(dsrcp, kEnt, dw, stamp, abort_flag, A.error,
                                             A.spin_limit)) {
                Payload<T> pl;
#pragma unroll
                for (int kk = 0; kk < W; ++kk) pl.w[kk] = kk < DW ? (uint32_t)dw[kk] : 0u;
                reinterpret_cast<T*>(dpart + (STAGE & 1) * kDiagCopy)[dpos[t]] = from_payload<T>(pl).x;
                if constexpr (GINT) hsite(STAGE & 1)[t] = from_payload<T>(pl).x + (T)0.5;
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
