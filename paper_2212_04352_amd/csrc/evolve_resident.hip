// evolve_resident.hip -- host side of the resident path: which kernel
// configuration holds a lattice, its LDS and scratch, its grid and launch.
#include <algorithm>
#include <set>

#include "device_common.h"
#include "ftwa_internal.h"
#include "evolve_shared.h"
#include "resident_config.h"

namespace ftwa {

namespace {

// The public configuration index.  0-7 and 13-18: the first tiles with every
// slot general and with one general slot per class; 8-12: the spin split;
// 19-22 and 37: the split kernel; 23-24: FP64 tiles of 384 threads x 2 units with
// (2, 2) slots (the 768 entries per class of 256 x (3, 3) with two thirds of
// its registers per thread); 25-36: fewer units per workgroup (the per-stage
// barriers span fewer waves and more workgroups share a CU).  From 38 on: the
// shared-pack shapes, FP64 then FP32.
const Config* const kConfigTable[] = {
    &kConfigsF64Shared[0], &kConfigsF64Shared[1], &kConfigsF64Shared[2],
    &kConfigsF64Shared[3], &kConfigsF32Shared[0], &kConfigsF32Shared[1],
    &kConfigsF32Shared[2], &kConfigsF32Shared[3], &kConfigsF32Spin[0], &kConfigsF32Spin[1],
    &kConfigsF32Spin[2], &kConfigsF32Spin[3], &kConfigsF32Spin[4], &kConfigsF64Shared[4],
    &kConfigsF64Shared[5], &kConfigsF64Shared[6], &kConfigsF32Shared[4],
    &kConfigsF32Shared[5], &kConfigsF32Shared[6], &kConfigsF64Split[0],
    &kConfigsF64Split[1], &kConfigsF64Split[2], &kConfigsF64Split[3], &kConfigsF64Shared[7],
    &kConfigsF64Shared[8], &kConfigsF64Shared[9], &kConfigsF32Shared[7],
    &kConfigsF64Shared[10], &kConfigsF32Shared[8], &kConfigsF64Shared[11],
    &kConfigsF32Shared[9], &kConfigsF64Shared[12], &kConfigsF32Shared[10],
    &kConfigsF64Shared[13], &kConfigsF32Shared[11], &kConfigsF64Shared[14],
    &kConfigsF32Shared[12], &kConfigsF64Split[4]
};
constexpr int kNumConfigs = (int)(sizeof(kConfigTable) / sizeof(kConfigTable[0]));
inline const Config& config_at(int k) { return *kConfigTable[k]; }

// Order of preference of the first-fit choice (of tiles with the same slots,
// fewer units per workgroup first, then fewer general slots; indices are
// those of kConfigTable).
const int kPreference[] = {31, 29, 27, 25, 0, 33, 13, 1, 23, 24, 35, 14, 2, 15, 3,
                           32, 30, 28, 26, 4, 34, 16, 5, 36, 17, 6, 18, 7,
                           8, 9, 10, 11, 12, 37, 19, 22, 20, 21};
static_assert(sizeof(kPreference) == sizeof(kConfigTable) / sizeof(kConfigTable[0]) * sizeof(int),
              "every configuration has a place in the preference order");

constexpr size_t kMaxLds = 160 * 1024;  // the kernel declares no static LDS

// Dynamic LDS of a launch: the state blocks (S = 1: after two copies of the
// partner's diagonal, room for 256 reals each), then the per-wave record sums
// and the abort flag.
size_t lds_blocks(const Config& c, int N, int P) {
    (void)N;
    const size_t cb = c.dtype == FTWA_F64 ? 16 : 8;
    const size_t tail = c.S == 1 ? 33 : 2;  // zero slot(s) and scratch slot
    const size_t b = (size_t)c.UNITS * c.S * (P + tail) * cb + (c.S == 1 ? 2 * 256 * (cb / 2) : 0);
    return (b + 15) / 16 * 16;
}
size_t lds_tail(const Config& c) { return (size_t)(c.NTU * c.UNITS / 64) * 2 * c.S * 8 + 16; }
size_t lds_bytes(const Config& c, int N, int P) { return lds_blocks(c, N, P) + lds_tail(c); }
// The split kernel: two copies of the partner's diagonal, then the owned and
// halo elements, 32 zero slots and the scratch slot of the largest part.
size_t split_lds_bytes(const Config& c, int max_slots) {
    const size_t cb = c.dtype == FTWA_F64 ? 16 : 8;
    const size_t b = 2 * 256 * (cb / 2) + (size_t)(max_slots + 33) * cb;
    return (b + 15) / 16 * 16 + lds_tail(c);
}
// Published words per element of the split kernel, and per group of 2G
// workgroups: [2 spins][G parts][2 parities][entries][words], then its
// flags and the members' XCDs.
int64_t split_words(const Config& c) {
    const int64_t w = c.dtype == FTWA_F64 ? 2 : 1;
    const int64_t plane = (int64_t)c.NTU * (c.UE + c.UO) + kSplitPlanePad;
    return 2 * (int64_t)c.G * 2 * plane * w + kSplitSyncWords;
}

}  // namespace

namespace {

// Facts of a device that every plan asks for: its compute units, the
// configurations whose LDS limit is raised, and the workgroups of a
// configuration that a CU holds.  Asking the runtime again took 2.3 of the
// 6.5 us of a plan (a run plans twice: for its workspace and for itself) and as
// much again before the launches.
struct DeviceFacts {
    int cus = 0;
    std::set<int> prepared;
    std::map<std::tuple<int, int, size_t>, int> per_cu;  // configuration and variant, threads, LDS
    // the shared-pack plan of an ensemble that fills the chip, by what it
    // depends on (N, sites of the first sublattice, even elements, precision,
    // variant): two dozen candidates weighed take 6 us
    std::map<std::tuple<int, int, int64_t, int, int>, ResidentPlan> many;
};
constexpr size_t kMaxFacts = 4096;  // distinct launch shapes kept per device
std::mutex g_facts_mu;
std::map<int, DeviceFacts> g_facts;

int device_cus() {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess) return cus;
    std::lock_guard<std::mutex> lock(g_facts_mu);
    DeviceFacts& f = g_facts[dev];
    if (f.cus == 0 &&
        (hipDeviceGetAttribute(&f.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
         f.cus < 1)) {
        f.cus = 0;
        return cus;
    }
    return f.cus;
}

}  // namespace

namespace {

// The shared-pack shapes follow the tiles above in the configuration index:
// FP64, then FP32.
constexpr int kSharedF64At = kNumConfigs, kSharedF32At = kNumConfigs + kSharedShapes;

const SharedShape* shared_at(int config) {
    if (config >= kSharedF32At && config < kSharedF32At + kSharedShapes)
        return &kSharedF32[config - kSharedF32At];
    if (config >= kSharedF64At && config < kSharedF32At) return &kSharedF64[config - kSharedF64At];
    return nullptr;
}

int shared_variant(bool potential, bool hop, bool interaction) {
    return potential ? kSharedPot : hop ? kSharedHop : interaction ? kSharedGint : kSharedPlain;
}

// Dynamic LDS of a pack of K trajectories (evolve_shared.h's layout).
size_t shared_lds(int N, int n_a, int tb, int maxt, int var, int K, int spt, bool u_lds) {
    const int I = K * (3 - spt), M = I >= 16 ? 1 : 16 / I;
    const size_t el = (size_t)((N + n_a) * shared_stride(N, n_a, I) + M - 1) / M * M + 2 * M;
    size_t b = shared_head(tb, maxt, var) + (el * K + 15) / 16 * 16 * (tb == 8 ? 32 : 16);
    if (var == kSharedHop) b += (size_t)2 * 6 * N * tb;
    if (var == kSharedGint) b += (size_t)K * (umat_rows(N) + 2) * 2 * tb;
    if (u_lds) b += (size_t)umat_rows(N) * N * tb;
    return (b + 15) / 16 * 16;
}

// Shape `config` with packs of K trajectories: whether a lattice fits, and
// the plan (the fewest threads that hold it).
bool shared_fit(int config, int N, const DeviceTables& tab, int var, int K, ResidentPlan* plan) {
    const SharedShape& sh = *shared_at(config);
    const int tb = sh.dtype == FTWA_F64 ? 8 : 4;
    const int I = K * (3 - sh.spt);
    const int64_t most = std::max(tab.n_even, packed_count(N) - tab.n_even);
    // entries per pass: a U-th of the longer list, the diagonal (it sits in
    // slot 0), two groups of entries (the first lanes clear the zero elements)
    const int64_t need = std::max<int64_t>({(most + sh.U - 1) / sh.U, N, I < 16 ? 32 / I : 1});
    const int64_t nt = (need * I + 63) / 64 * 64;
    if (!sh.fn[var]) return false;
    // a general interaction: waves of their own for the sums D_i
    const int64_t nd = var == kSharedGint ? std::min<int64_t>((K * N + 63) / 64 * 64, 192) : 0;
    if (nt + nd > sh.maxt) return false;
    if (K * N > shared_diag_cap(sh.maxt)) return false;
    if (var == kSharedHop && 6 * N > 3 * nt) return false;
    bool u_lds = var == kSharedGint;
    size_t lds = shared_lds(N, tab.n_a, tb, sh.maxt, var, K, sh.spt, u_lds);
    if (u_lds && lds > kMaxLds) {
        u_lds = false;
        lds = shared_lds(N, tab.n_a, tb, sh.maxt, var, K, sh.spt, u_lds);
    }
    if (lds > kMaxLds) return false;
    *plan = ResidentPlan();
    plan->config = config;
    plan->variant = var;
    plan->threads = (int)(nt + nd);
    plan->workers = (int)nt;
    plan->units = K;
    plan->lanes = I;
    plan->even_slots = plan->odd_slots = (int64_t)sh.U * (nt / I);
    plan->lds = lds;
    plan->u_lds = u_lds;
    return true;
}

// How well a plan suits an ensemble that fills the chip: the share of its
// slots that hold elements, less where the resident waves of a CU fall short
// of the twelve that hide the LDS latency (20 sites FP32: two slots, packs of
// 8, 7 waves 5.0e8 trajectory-steps/s; one slot, packs of 4, 14 waves 6.0e8),
// where a pack of one leaves bank conflicts, for a single slot (the loads of
// an element's neighbours have no other element's arithmetic beside them), for
// packed addresses, and for interaction waves whose lanes have no site (30
// sites FP32: packs of one 683 us, of two 475, the tiles 527; 4000
// trajectories, 20 steps).  Against a sweep of every shape and pack at 25
// lattices of 16 to 96 sites, all variants, the choice is within 9 % of the
// fastest in 19 of 20 and within 21 % in all (the worst: 48 sites FP64 with a
// general interaction).
//
// Complex hopping spills in the packed shapes: three packed slots serve only
// where no other shape holds the lattice (66 sites FP64 7.8e6
// trajectory-steps/s, the tiles above 5.2e6; 40 sites FP64 2.0e7 against 4.1e7
// with two plain slots), the last shape never (66 sites FP64 4.3e6; 96 sites
// FP32 1.03e7, the tiles 1.02e7).
double shared_score(const ResidentPlan& rp, int N, int var) {
    const SharedShape& sh = *shared_at(rp.config);
    const int waves = rp.threads / 64, nd = rp.threads - rp.workers;
    const double groups = (double)resident_concurrency(rp.config, rp.lds, rp.threads, rp.units,
                                                       rp.variant) /
                          ((double)rp.units * device_cus());
    const double fill = (double)packed_count(N) * rp.lanes / (2.0 * sh.U * rp.workers);
    const double busy = 0.5 + 0.5 * std::min(1.0, groups * waves / 12.0);
    double shape = 1.0;
    if (sh.packed) shape = var == kSharedHop ? 0.5 : sh.U > 3 ? 0.88 : 0.89;
    else if (sh.U == 1) shape = 0.8;
    if (nd > 0) shape *= 0.5 + 0.5 * std::min(1.0, (double)rp.units * N / nd);
    return fill * busy * shape * (rp.units == 1 ? 0.95 : 1.0);
}

bool shared_allowed(int shape, int var) { return !(var == kSharedHop && shape == 5); }

bool shared_many_uncached(int N, ftwa_dtype dtype, const DeviceTables& tab, int var,
                          ResidentPlan* plan) {
    const bool f64 = dtype == FTWA_F64;
    const int at = f64 ? kSharedF64At : kSharedF32At;
    // Below 16 sites a stage is short and few waves per barrier matter more
    // than full slots: 12 sites, three slots, packs of 4 in one or two waves
    // 8.2e8 (FP64) and 1.59e9 (FP32) trajectory-steps/s, two slots, packs of
    // 16 in eleven 8.0e8 and 1.1e9; up to 11 sites one or two slots, packs of
    // 4 in two waves: 1.38e9 and 2.36e9 at 10.  From 13 sites three slots take
    // half as many waves more and fill them less than two (20000 trajectories,
    // 40 steps, 14 sites: FP64 2.08 ms on three, 1.37 on two, the tiles 1.50;
    // FP32 1.07, 0.69 and 0.88).  The waves of a general interaction want larger
    // packs (10 sites FP64: packs of 16 7.8e8, of 4 5.8e8; 12 sites: 6.0e8, of 4
    // on three slots 4.6e8; FP32 at 12: packs of 8 on one slot 1.14e9, of 4 on
    // three 8.8e8).
    if (N < 16) {
        const bool gint = var == kSharedGint;
        int shape, K = 4;
        if (N < 12) {
            shape = f64 ? 2 : 1;
            if (gint && f64) K = 16;
        } else {
            shape = !gint ? 3 : f64 ? 4 : 1;
            if (gint) K = f64 ? 16 : 8;
        }
        if (shape == 3 && (!shared_fit(at + 3, N, tab, var, K, plan) ||
                           plan->workers / plan->lanes > 16))
            shape = 2;
        if (shared_fit(at + shape, N, tab, var, K, plan)) return true;
    }
    double best = 0;
    for (int shape : {2, 1, 4, 5})
        for (int K = 16; K >= 1; K /= 2) {
            ResidentPlan rp;
            if (!shared_allowed(shape, var) || !shared_fit(at + shape, N, tab, var, K, &rp))
                continue;
            const double score = shared_score(rp, N, var);
            if (score > best) {
                best = score;
                *plan = rp;
            }
        }
    return best > 0;
}

// The plan for an ensemble that fills the chip (config -1: none).
bool shared_many(int N, ftwa_dtype dtype, const DeviceTables& tab, int var, ResidentPlan* plan) {
    int dev = 0;
    const auto key = std::make_tuple(N, tab.n_a, tab.n_even, (int)dtype, var);
    const bool known = hipGetDevice(&dev) == hipSuccess;
    if (known) {
        std::lock_guard<std::mutex> lock(g_facts_mu);
        const auto& many = g_facts[dev].many;
        const auto it = many.find(key);
        if (it != many.end()) {
            *plan = it->second;
            return plan->config >= 0;
        }
    }
    ResidentPlan rp;
    if (!shared_many_uncached(N, dtype, tab, var, &rp)) rp.config = -1;
    if (known) {
        std::lock_guard<std::mutex> lock(g_facts_mu);
        auto& many = g_facts[dev].many;
        if (many.size() >= kMaxFacts) many.clear();
        many[key] = rp;
    }
    *plan = rp;
    return rp.config >= 0;
}

// The plan for an ensemble of fewer trajectories than that plan keeps in
// flight: the smallest slots per thread that hold the lattice, packs of at
// most K, small enough to give every CU one (a stage's latency is what
// counts: 64 trajectories of 10 sites FP64 0.23 us per stage with one slot, 0.45
// with two, 0.66 with three, 0.74 on the tiles above).  wide: complex hopping with several
// packs to a CU, where two slots come before one (its registers let two waves
// of the one-slot kernel share a SIMD, three of the other: 13 sites FP32, 4000
// trajectories 293 us on two slots, 334 on one, the tiles 312).
bool shared_few(int N, ftwa_dtype dtype, const DeviceTables& tab, int var, int K, bool wide,
                ResidentPlan* plan) {
    const int at = dtype == FTWA_F64 ? kSharedF64At : kSharedF32At;
    for (int shape : {0, wide ? 2 : 1, wide ? 1 : 2, 4, 5}) {
        if (!shared_allowed(shape, var) || (shape == 0 && K != 1)) continue;
        for (int k = K; k >= 1; k /= 2)
            if (shared_fit(at + shape, N, tab, var, k, plan)) return true;
    }
    return false;
}

// Whether a plan keeps n_traj trajectories in flight at once.
bool shared_holds(const ResidentPlan& rp, int64_t n_traj) {
    return n_traj <= resident_concurrency(rp.config, rp.lds, rp.threads, rp.units, rp.variant);
}

// A forced shape that the rules do not choose: the largest pack up to 4 that
// leaves room for the variant.
bool shared_forced(int config, int N, const DeviceTables& tab, int var, ResidentPlan* plan) {
    for (int K = 4; K >= 1; K /= 2)
        if (shared_fit(config, N, tab, var, K, plan)) return true;
    return false;
}

}  // namespace

bool resident_is_shared(int config) { return shared_at(config) != nullptr; }

bool shared_plan(int N, ftwa_dtype dtype, const DeviceTables& tab, int64_t n_traj,
                 ResidentPlan* plan, int force_config, bool need_potential, bool need_hop,
                 bool need_interaction) {
    if (!tab.bipartite) return false;
    const int var = shared_variant(need_potential, need_hop, need_interaction);
    if (force_config >= 0) {
        // the plan of the rules, if that is its shape
        if (shared_at(force_config)->dtype == dtype &&
            shared_plan(N, dtype, tab, n_traj, plan, -1, need_potential, need_hop,
                        need_interaction) &&
            plan->config == force_config)
            return true;
        return shared_forced(force_config, N, tab, var, plan);
    }
    if (!shared_many(N, dtype, tab, var, plan)) return false;
    if (n_traj < resident_concurrency(plan->config, plan->lds, plan->threads, plan->units,
                                      plan->variant)) {
        const int64_t cus = device_cus();
        int K = 1;
        while (K < 4 && n_traj >= 2 * K * cus) K *= 2;
        ResidentPlan rp;
        if (!shared_few(N, dtype, tab, var, K, need_hop && N >= 12 && n_traj >= 4 * cus, &rp))
            return true;
        *plan = rp;
        // a general interaction that this plan takes in turns: in packs of four
        // if these are in flight all at once (30 sites FP64, 700 trajectories:
        // 198 us, 270 in turns, the tiles 232)
        if (need_interaction && !shared_holds(rp, n_traj))
            for (int shape : {1, 2, 4, 5})
                if (shared_fit((dtype == FTWA_F64 ? kSharedF64At : kSharedF32At) + shape, N, tab,
                               var, 4, &rp) &&
                    shared_holds(rp, n_traj)) {
                    *plan = rp;
                    break;
                }
    }
    return true;
}

bool shared_plan_like(const ResidentPlan& like, int N, const DeviceTables& tab,
                      ResidentPlan* plan) {
    if (!shared_fit(like.config, N, tab, like.variant, like.units, plan) ||
        plan->workers > like.workers)
        return false;
    plan->workers = like.workers;
    plan->threads = like.threads;
    plan->even_slots = plan->odd_slots =
        (int64_t)shared_at(like.config)->U * (like.workers / like.lanes);
    return true;
}

std::map<int, int> shared_passes(int N, const DeviceTables& tab, std::set<int>* configs) {
    std::map<int, int> passes;
    if (!tab.bipartite) return passes;
    for (int c = kSharedF64At; c < kSharedF32At + kSharedShapes; ++c)
        for (int var : {kSharedPlain, kSharedPot, kSharedHop, kSharedGint})
            for (int K = 16; K >= 1; K /= 2) {
                ResidentPlan rp;
                if (!shared_fit(c, N, tab, var, K, &rp)) continue;
                configs->insert(c);
                const int n_pass = rp.workers / rp.lanes;
                const auto it = passes.emplace(std::min(rp.lanes, 16), n_pass).first;
                it->second = std::min(it->second, n_pass);
            }
    return passes;
}

bool resident_plan(int N, ftwa_dtype dtype, const DeviceTables& tab, ResidentPlan* plan,
                   int force_config, bool allow_split, bool need_potential, bool need_hop,
                   bool need_interaction) {
    if (!tab.bipartite) return false;
    if (shared_at(force_config))
        return allow_split && shared_at(force_config)->dtype == dtype &&
               shared_plan(N, dtype, tab, 1, plan, force_config, need_potential, need_hop,
                           need_interaction);
    const int P = (int)packed_count(N);
    const int n_even = (int)tab.n_even, n_odd = P - n_even;
    const int n_cfg = kNumConfigs;
    for (int o = 0; o < n_cfg; ++o) {
        const int k = kPreference[o];
        if (force_config >= 0 && k != force_config) continue;
        const Config& c = config_at(k);
        bool u_lds = false;
        if (c.dtype != dtype) continue;
        if (!c.auto_pick && force_config < 0) continue;
        if (need_potential && !c.fn_pot) continue;
        if (need_hop && !c.fn_hop) continue;
        if (need_interaction && !c.fn_gint) continue;
        if (N > c.NTU) continue;  // the diagonal must sit in slot 0
        size_t lds;
        if (c.G > 1) {
            // the split kernel: every part must fit (no invariant sums)
            if (!allow_split || N > 256) continue;
            const SplitShape& sh = tab.split[c.G];
            const int64_t n = c.NTU;
            if (n * c.UE < sh.n_even || n * c.UO < sh.n_odd) continue;
            if (n * c.GE < sh.int_gen || n * (c.UE - c.UB) < sh.n_bnd || n * c.GE2 < sh.bnd_gen)
                continue;
            if (n * c.GO < sh.odd_gen || n * c.XO < sh.odd_x) continue;
            if (sh.max_slots + 33 > 0x7fff) continue;
            lds = split_lds_bytes(c, sh.max_slots);
            if (need_interaction) lds += 3 * 256 * (c.dtype == FTWA_F64 ? 8 : 4);  // D, h copies
            else if (need_hop) lds += 256 * 6 * (c.dtype == FTWA_F64 ? 8 : 4);  // ratio table
            else if (need_potential) lds += 256 * (c.dtype == FTWA_F64 ? 8 : 4);  // the profile
            // where the halo elements are published, a word each (the kernel
            // reads that from global memory where LDS has no room for it)
            const size_t imp = ((size_t)sh.max_halo * 4 + 15) / 16 * 16;
            if (lds + imp <= kMaxLds) lds += imp;
        } else {
            if (P + 33 > 0x7fff) continue;
            if ((int64_t)c.NTU * c.UE < n_even || (int64_t)c.NTU * c.UO < n_odd) continue;
            if ((int64_t)c.NTU * c.GE < tab.n_gen_even || (int64_t)c.NTU * c.GO < tab.n_gen_odd)
                continue;
            lds = lds_bytes(c, N, P);
            // spin split: the potential's profile, the general interaction's
            // D and two site-ordered copies of the partner's diagonal, or the
            // first kHopLds places of the complex-hopping stage table; shared
            // blocks: D of every unit and spin or the profile (one value per
            // site at the element stride), or the whole ratio table
            const size_t tb = c.dtype == FTWA_F64 ? 8 : 4;
            const size_t cbb = 2 * tb;
            if (need_interaction) {
                lds += c.S == 1 ? 3 * 256 * tb : ((size_t)c.UNITS * 2 * N * cbb + 15) / 16 * 16;
                // shared blocks: a copy of u and the units' h = d + 1/2 in
                // site order beside D where they fit (read there by the
                // per-stage chains instead of from L2 and the blocks)
                const size_t ub = (size_t)umat_rows(N) * N * tb +  // multiples of 16
                                  (size_t)c.UNITS * 2 * umat_rows(N) * tb;
                if (c.S == 2 && lds + ub <= kMaxLds) {
                    lds += ub;
                    u_lds = true;
                }
            }
            else if (need_hop)
                lds += c.S == 1 ? (size_t)kHopLds * 6 * tb : ((size_t)N * 3 * cbb + 15) / 16 * 16;
            else if (need_potential)
                lds += c.S == 1 ? 256 * tb : ((size_t)N * cbb + 15) / 16 * 16;
        }
        if (lds > kMaxLds) continue;
        plan->config = k;
        plan->spins_per_unit = c.S;
        plan->threads = c.NTU * c.UNITS;
        plan->units = c.UNITS;
        plan->even_slots = (int64_t)c.NTU * c.UE;
        plan->odd_slots = (int64_t)c.NTU * c.UO;
        plan->lds = lds;
        plan->bnd_entry = (int64_t)c.NTU * c.UB;
        plan->u_lds = u_lds;
        return true;
    }
    return false;
}

int resident_config_count() { return kNumConfigs + 2 * kSharedShapes; }

int resident_spins(int config) { return shared_at(config) ? 2 : config_at(config).S; }
int resident_parts(int config) { return shared_at(config) ? 1 : config_at(config).G; }
bool resident_has_potential(int config) {
    return shared_at(config) || config_at(config).fn_pot != nullptr;
}
bool resident_has_hop(int config) {
    return shared_at(config) || config_at(config).fn_hop != nullptr;
}
bool resident_has_interaction(int config) {
    return shared_at(config) || config_at(config).fn_gint != nullptr;
}


namespace {
ftwa_status raise_lds_limit(int config) {
    if (const SharedShape* sh = shared_at(config)) {
        for (int v = 0; v < 4; ++v)
            for (const void* f : {sh->fn[v], sh->fn_t1[v]})
                if (f)
                    FTWA_HIP_TRY(hipFuncSetAttribute(
                        f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds));
        return FTWA_OK;
    }
    FTWA_HIP_TRY(hipFuncSetAttribute(config_at(config).fn,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds));
    if (config_at(config).fn_t1)
        FTWA_HIP_TRY(hipFuncSetAttribute(config_at(config).fn_t1,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds));
    if (config_at(config).fn_pot)
        FTWA_HIP_TRY(hipFuncSetAttribute(config_at(config).fn_pot,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds));
    for (const void* f : {config_at(config).fn_pot_t1, config_at(config).fn_hop,
                          config_at(config).fn_hop_t1, config_at(config).fn_gint,
                          config_at(config).fn_gint_t1})
        if (f)
            FTWA_HIP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)kMaxLds));
    return FTWA_OK;
}
}  // namespace

ftwa_status resident_prepare(int config, size_t lds) {
    (void)lds;  // the limit is raised to the whole LDS once; launches use less
    int dev = 0;
    FTWA_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(g_facts_mu);
    DeviceFacts& f = g_facts[dev];
    if (f.prepared.count(config)) return FTWA_OK;
    const ftwa_status st = raise_lds_limit(config);
    if (st == FTWA_OK) f.prepared.insert(config);
    return st;
}

// Pairs of spin-split workgroups that are resident together: one workgroup
// per CU (LDS bound), pairs in groups of 8 (one per XCD).
int64_t resident_max_pairs() {
    const int64_t pairs = (int64_t)device_cus() / 2 / 8 * 8;
    return pairs < 8 ? 8 : pairs;
}

// Groups of 2G split workgroups resident together: whole groups per XCD.
int64_t split_max_groups(int G) {
    const int64_t per_xcd = (int64_t)device_cus() / 8 / (2 * G);
    return 8 * (per_xcd < 1 ? 1 : per_xcd);
}

// Trajectories (items) a spin-split launch runs at once, and its grid.
int64_t spin_split_slots(const Config& c) {
    return c.G > 1 ? split_max_groups(c.G) : resident_max_pairs();
}

// Workgroups of a kernel that a CU holds at once; false where the runtime does
// not say.  A workgroup of more than four waves starts only where every SIMD
// has room for its share rounded up, which the runtime's count leaves out (a
// kernel that does nothing but wait, by waves per workgroup at three a SIMD:
// 5 and 6 waves one workgroup, the runtime says two; at four a SIMD: 5 waves
// two, it says three).  A persistent grid of the runtime's count then ran its
// last third after the others had ended: 15 sites FP32, general interaction,
// 4000 trajectories 483 us, 259 with the grid that fits.
bool workgroups_per_cu(const void* fn, int threads, size_t lds, int* per_cu) {
    int n = 0, waves = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, threads, lds) != hipSuccess || n < 1)
        return false;
    if (threads > 256) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&waves, fn, 64, 0) != hipSuccess)
            return false;
        n = std::max(1, std::min(n, waves / 4 / ((threads / 64 + 3) / 4)));
    }
    *per_cu = n;
    return true;
}

int64_t resident_concurrency(int config, size_t lds, int threads, int units, int variant) {
    const SharedShape* sh = shared_at(config);
    if (!sh && config_at(config).S == 1) return spin_split_slots(config_at(config));
    // the occupancy query honours the dynamic-LDS limit of the kernel
    if (resident_prepare(config, kMaxLds) != FTWA_OK) return (int64_t)device_cus() * units;
    const int64_t cus = device_cus();
    int dev = 0, per_cu = 1;
    if (hipGetDevice(&dev) != hipSuccess) return cus * units;
    std::lock_guard<std::mutex> lock(g_facts_mu);
    auto& known = g_facts[dev].per_cu;
    const auto key = std::make_tuple(4 * config + variant, threads, lds);
    auto it = known.find(key);
    if (it != known.end()) return it->second * cus * units;
    if (sh) {
        int t1 = 1;
        if (!workgroups_per_cu(sh->fn[variant], threads, lds, &per_cu) ||
            !workgroups_per_cu(sh->fn_t1[variant], threads, lds, &t1))
            return cus * units;
        per_cu = std::min(per_cu, t1);
    } else if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, config_at(config).fn, threads,
                                                            lds) != hipSuccess ||
               per_cu < 1) {
        return cus * units;
    }
    if (known.size() >= kMaxFacts) known.clear();
    known.emplace(key, per_cu);
    return (int64_t)per_cu * cus * units;
}

int64_t resident_grid(int config, size_t lds, int64_t n_items, int threads, int units,
                      int variant) {
    if (!shared_at(config) && config_at(config).S == 1) {
        const Config& c = config_at(config);
        const int64_t n = std::min((n_items + 7) / 8 * 8, spin_split_slots(c));
        return 2 * (int64_t)c.G * n;
    }
    const int64_t cap = resident_concurrency(config, lds, threads, units, variant) / units;
    return std::max<int64_t>(1, std::min(n_items, cap));
}

// Spin-split scratch of one launch: the mailbox words (split kernel: the
// published words of every group).
size_t mailbox_words(const Config& c, int Nmax, int64_t grid) {
    if (c.G > 1) return (size_t)(grid / (2 * c.G)) * (size_t)split_words(c);
    return (size_t)(grid / 2) * 2 * 2 * Nmax;
}

size_t resident_mailbox_bytes(int config, int Nmax, int64_t n_items) {
    if (shared_at(config) || config_at(config).S != 1) return 0;
    const Config& c = config_at(config);
    return mailbox_words(c, Nmax, resident_grid(config, 0, n_items, 0, 1, 0)) * sizeof(uint64_t);
}


namespace {
// The ratio table of the complex-hopping variant: out[r][dpos[i]][n] = w[r][i][n]
// rounded once to T for n < deg(i), zero for a missing neighbour (whose
// caller-side value may be anything), r over the 2 n_steps + 1 half steps.
template <typename T>
__global__ __launch_bounds__(256) void hop_table_kernel(const double2* __restrict__ w,
                                                        const int32_t* __restrict__ nb,
                                                        const int32_t* __restrict__ dpos, int N,
                                                        int64_t n_rows, cplx_t<T>* __restrict__ out) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n_rows * N * 3) return;
    const int64_t r = x / (3 * N);
    const int i = (int)(x / 3 - r * N), n = (int)(x % 3);
    cplx_t<T> v;
    v.x = 0;
    v.y = 0;
    if (n < nb[i * 4 + 3]) {
        const double2 a = w[x];
        v.x = (T)a.x;
        v.y = (T)a.y;
    }
    out[(r * N + (dpos ? dpos[i] : i)) * 3 + n] = v;
}
}  // namespace

ftwa_status hop_table(const double* hop_w, const int32_t* nb, const int32_t* dpos, int N,
                      int64_t n_steps, ftwa_dtype dtype, void* out, hipStream_t stream) {
    const int64_t n_rows = 2 * n_steps + 1, n = n_rows * N * 3;
    const dim3 grid((unsigned)((n + 255) / 256));
    const double2* w = reinterpret_cast<const double2*>(hop_w);
    if (dtype == FTWA_F64)
        hipLaunchKernelGGL(hop_table_kernel<double>, grid, dim3(256), 0, stream, w, nb, dpos, N,
                           n_rows, static_cast<cplx_t<double>*>(out));
    else
        hipLaunchKernelGGL(hop_table_kernel<float>, grid, dim3(256), 0, stream, w, nb, dpos, N,
                           n_rows, static_cast<cplx_t<float>*>(out));
    FTWA_LAUNCH_CHECK("hop_table_kernel");
    return FTWA_OK;
}

namespace {
// u of the general-interaction variant rounded once to T, blocked by four
// along k: out[((k / 4) N + i) 4 + k % 4] = u_ki, rows k >= N zero.
template <typename T>
__global__ __launch_bounds__(256) void umat_table_kernel(const double* __restrict__ u, int N,
                                                         int64_t n, T* __restrict__ out) {
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n) return;
    const int64_t kb = x / (4 * (int64_t)N);
    const int64_t rem = x - kb * 4 * N;
    const int64_t i = rem / 4;
    const int64_t k = 4 * kb + (rem & 3);
    out[x] = k < N ? (T)u[k * N + i] : (T)0;
}
}  // namespace

ftwa_status umat_table(const double* u_mat, int N, ftwa_dtype dtype, void* out,
                       hipStream_t stream) {
    const int64_t n = (int64_t)umat_rows(N) * N;
    const dim3 grid((unsigned)((n + 255) / 256));
    if (dtype == FTWA_F64)
        hipLaunchKernelGGL(umat_table_kernel<double>, grid, dim3(256), 0, stream, u_mat, N, n,
                           static_cast<double*>(out));
    else
        hipLaunchKernelGGL(umat_table_kernel<float>, grid, dim3(256), 0, stream, u_mat, N, n,
                           static_cast<float*>(out));
    FTWA_LAUNCH_CHECK("umat_table_kernel");
    return FTWA_OK;
}

namespace {
// The flags and XCDs at the end of every split group's words.
__global__ __launch_bounds__(64) void clear_sync_kernel(uint64_t* words, int64_t per_group) {
    uint64_t* const sync = words + (blockIdx.x + 1) * per_group - kSplitSyncWords;
    for (int k = threadIdx.x; k < kSplitSyncWords; k += 64) sync[k] = 0;
}
}  // namespace

ftwa_status resident_launch(const ResidentLaunch& L, hipStream_t stream) {
    if (L.n_items <= 0) return FTWA_OK;
    if (const SharedShape* sh = shared_at(L.config)) {
        SharedArgs A;
        A.table = L.table;
        A.n_entries = L.n_entries;
        A.kshift = __builtin_ctz((unsigned)L.units);
        A.workers = L.workers;
        A.n_items = L.n_items;
        A.dt = L.dt;
        A.n_steps = L.n_steps;
        A.record_every = L.record_every;
        const int v = shared_variant(L.potential, L.hopping, L.interaction);
        const void* fn = L.unit_hop && !L.dumps ? sh->fn_t1[v] : sh->fn[v];
        void* args[] = {&A};
        FTWA_HIP_TRY(hipLaunchKernel(fn, dim3((unsigned)L.grid), dim3((unsigned)L.threads), args,
                                     (unsigned)L.lds, stream));
        return FTWA_OK;
    }
    const Config& c = config_at(L.config);
    ResidentArgs A;
    A.table = L.table;
    A.n_entries = L.n_entries;
    A.n_items = L.n_items;
    A.dt = L.dt;
    A.n_steps = L.n_steps;
    A.record_every = L.record_every;
    A.mailbox = static_cast<uint64_t*>(L.mailbox);
    A.Nmax = L.Nmax;
    A.tail_off = (uint32_t)(L.lds - lds_tail(c));
    A.error = L.error;
    A.spin_limit = L.spin_limit ? L.spin_limit : (c.G > 1 ? kSplitSpinLimit : kSpinLimit);
    A.far = L.inject == kInjectFarExchange;
    void* args[] = {&A};
    // fault injection for tests of the timeout path: only the up-spin
    // workgroups of eight trajectories run, so that each of them gives up its
    // first wait for the absent partners and exits
    const int64_t grid = L.inject == kInjectDropPartners && c.S == 1 ? 8 * c.G : L.grid;
    const bool t1 = L.unit_hop && !L.dumps;
    const void* fn = L.interaction ? (t1 && c.fn_gint_t1 ? c.fn_gint_t1 : c.fn_gint)
                     : L.hopping   ? (t1 && c.fn_hop_t1 ? c.fn_hop_t1 : c.fn_hop)
                     : L.potential ? (t1 && c.fn_pot_t1 ? c.fn_pot_t1 : c.fn_pot)
                                   : (t1 && c.fn_t1 ? c.fn_t1 : c.fn);
    if (!fn)
        return fail(FTWA_ENOTSUP, L.interaction ? "this configuration has no general-interaction variant"
                                  : L.hopping   ? "this configuration has no complex-hopping variant"
                                                : "this configuration has no external-potential variant");
    if (c.S == 1) {
        // (fill kernels, no memset node.)  Spin split: every word starts at stage
        // 0, which no wait accepts.  Split kernel: the flags at stage 0, no XCD;
        // the published words are read only behind flags raised in this launch,
        // so they keep what they hold (clearing them too, 0.8 MB a group, took
        // 15 of the 640 us of a record interval of one step at 150 sites with
        // 500 trajectories)
        ftwa_status st = FTWA_OK;
        if (c.G > 1) {
            const int64_t groups = L.grid / (2 * c.G);
            hipLaunchKernelGGL(clear_sync_kernel, dim3((unsigned)groups), dim3(64), 0, stream,
                               static_cast<uint64_t*>(L.mailbox), split_words(c));
            FTWA_LAUNCH_CHECK("clear_sync_kernel");
        } else {
            st = zero_words(static_cast<unsigned*>(L.mailbox),
                            (int64_t)mailbox_words(c, L.Nmax, L.grid) * 2, stream);
        }
        if (st != FTWA_OK) return st;
        // both workgroups of a pair must be resident at the same time: the
        // grid never exceeds one workgroup per CU; a cooperative launch checks
        // it (not available under graph capture, where the bounded waits
        // report a partner that never came)
        if (L.cooperative)
            FTWA_HIP_TRY(hipLaunchCooperativeKernel(fn, dim3((unsigned)grid),
                                                    dim3(c.NTU * c.UNITS), args,
                                                    (unsigned)L.lds, stream));
        else
            FTWA_HIP_TRY(hipLaunchKernel(fn, dim3((unsigned)grid), dim3(c.NTU * c.UNITS), args,
                                         (unsigned)L.lds, stream));
    } else {
        FTWA_HIP_TRY(hipLaunchKernel(fn, dim3((unsigned)grid), dim3(c.NTU * c.UNITS), args,
                                     (unsigned)L.lds, stream));
    }
    return FTWA_OK;
}

}  // namespace ftwa
