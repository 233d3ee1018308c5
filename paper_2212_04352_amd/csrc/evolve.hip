// evolve.hip -- ftwa_evolve and its batched forms: the plan of a run (which
// kernel path and configuration integrates each instance, how trajectories
// are split into passes, where every buffer sits in the workspace), the
// queueing of its launches, the HIP-graph form of the same launches, and the
// autotuner that picks resident configurations by timing them.
//
// Batching.  Instances whose resident configuration is the same form a group;
// each pass launches one persistent kernel per group over a device table of
// (instance, trajectory window) entries, so mixed lattice sizes and U values
// of a group run in one launch.  Instances that no resident configuration
// fits run on the stream path.  The per-element arithmetic does not depend on
// the grouping, the configuration or the pass split, so a batched run gives
// bitwise the same trajectories as one run per instance.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <set>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "ftwa_internal.h"

namespace ftwa {

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
size_t cplx_bytes(ftwa_dtype d) { return d == FTWA_F64 ? 16 : 8; }

constexpr size_t kRecordBudget = (size_t)4 << 30;  // FP64 record bytes per pass
constexpr int64_t kStreamChunk = 4096;

// Status block of a run at the start of its workspace (32-bit words): a
// marker, the timeout flag the multi-workgroup resident kernels set, the
// number of (instance, record) pairs whose invariant monitor counted a
// non-finite trajectory, and the first such pair as instance << 16 | record.
// Written only by kernels queued with the run, read by ftwa_evolve_check.
constexpr size_t kStatusBytes = 256;
constexpr uint32_t kStatusMagic = 0x46545741u;

__global__ __launch_bounds__(64) void status_nonfinite_kernel(const double* __restrict__ inv,
                                                              int64_t n_rec, uint32_t inst,
                                                              uint32_t* st) {
    for (int64_t r = threadIdx.x; r < n_rec; r += blockDim.x)
        if (inv[r * 4 + 3] > 0.0) {
            atomicAdd(st + 2, 1u);
            atomicMin(st + 3, (inst << 16) | (uint32_t)r);
        }
}

// Launch-table entries travel to the device as kernel arguments (no host
// buffer has to outlive the call, and the write can be captured in a graph).
constexpr int kTableChunk = 16;
struct TableChunk {
    int n;
    ResidentInst e[kTableChunk];
};
static_assert(sizeof(ResidentInst) % 4 == 0, "table entries are copied as 32-bit words");
static_assert(sizeof(TableChunk) <= 3072, "kernel argument size");

__device__ __forceinline__ void write_table(ResidentInst* dst, const TableChunk& c) {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(c.e);
    uint32_t* out = reinterpret_cast<uint32_t*>(dst);
    const int words = c.n * (int)(sizeof(ResidentInst) / 4);
    for (int w = threadIdx.x; w < words; w += blockDim.x) out[w] = src[w];
}
__global__ __launch_bounds__(256) void write_table_kernel(ResidentInst* dst, TableChunk c) {
    write_table(dst, c);
}

// What a run needs before its first kernel, in one launch (a launch each took
// 5 us of a 10-site run's 140): the status block, launch-table entries and the
// cleared moments.  More than fit go into further launches.
constexpr int kPrologueFills = 24;
struct Prologue {
    uint32_t* status;     // NULL: not in this launch
    ResidentInst* table;  // c.n entries from here
    int n_fill;
    struct {
        double* p;
        int64_t n;
    } fill[kPrologueFills];
    TableChunk c;
};
static_assert(sizeof(Prologue) <= 4000, "kernel argument size");

__global__ __launch_bounds__(256) void prologue_kernel(Prologue a) {
    if (blockIdx.x == 0) {
        if (a.status && threadIdx.x == 0) {
            a.status[0] = kStatusMagic;
            a.status[1] = 0u;
            a.status[2] = 0u;
            a.status[3] = 0xffffffffu;
        }
        write_table(a.table, a.c);
    }
    for (int k = 0; k < a.n_fill; ++k)
        for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < a.fill[k].n;
             e += (int64_t)gridDim.x * 256)
            a.fill[k].p[e] = 0.0;
}

struct InstPlan {
    ftwa_path path = FTWA_PATH_STREAM;
    ResidentPlan res;
    int group = -1;
    int64_t chunk = 0;             // stream: trajectories per chunk; resident: per pass window
    size_t off_x = 0, off_inv = 0; // resident: this instance's record regions
    size_t off_hop = 0;            // resident with complex hopping: its ratio table
    size_t off_umat = 0;           // resident with a general interaction: u in dtype
    bool by_record = false;        // resident: a launch per record interval (see plan_evolve)
};

struct LaunchDesc {                // one resident launch: a group in a pass
    int group = 0;
    int64_t first_entry = 0;       // into the uploaded table
    int n_entries = 0;
    int64_t n_items = 0;
    int64_t grid = 0;
    double work = 0;               // trajectory-steps
    double share = 1;              // of the workgroups that the chip holds at once
    bool unit_hop = true;          // every instance has t = 1
    bool potential = false;        // an instance carries an external potential
    bool hopping = false;          // every instance carries complex hopping
    bool interaction = false;      // every instance carries a general interaction
};

struct GroupPlan {
    int config = -1;
    int threads = 0, units = 1, workers = 0, variant = 0;
    size_t lds = 0;
    int Nmax = 0;
    bool by_record = false;        // one member, a launch per record interval
    std::vector<int> members;
    int64_t max_items = 0;
    size_t off_mb = 0;
    size_t off_mom = 0;            // scratch of its members' moments
};

struct Plan {
    int n_inst = 0;
    int64_t n_rec = 0, n_steps = 0;
    int record_every = 1;
    double dt = 0;
    ftwa_dtype dtype = FTWA_F64;
    int n_pass = 0;
    std::vector<InstPlan> inst;
    std::vector<GroupPlan> groups;
    std::vector<LaunchDesc> launches;  // pass-major
    // stream area
    size_t s_acc = 0, s_ya = 0, s_yb = 0, s_x = 0, s_mom = 0, s_inv = 0, s_D = 0, s_total = 0;
    size_t off_status = 0;  // the status block (kStatusBytes at the start of the workspace)
    // resident area
    size_t r_table = 0, r_total = 0;
    int64_t n_table = 0;
    size_t total = 0;
    // internal runs only (one instance): its state is stored at every record
    void* dump = nullptr;
    int64_t dump_stride = 0;
    // the launch table's entries, filled on the host by build_table and
    // written to r_table by kernels queued at the start of every run
    std::vector<ResidentInst> table;
    unsigned spin_limit = 0;   // 0: the kernels' default
    int inject = 0;            // ftwa_tuning's drop_partners
};

void window(const Plan& p, const ftwa_instance& in, int k, int j, int64_t* m0, int64_t* Mc) {
    const int64_t c = p.inst[k].chunk;
    *m0 = std::min<int64_t>((int64_t)j * c, in.n_traj);
    *Mc = std::min<int64_t>(c, in.n_traj - *m0);
}

// Whether a configuration's workgroups run independently of each other.
bool waits_for_none(int config) {
    return resident_is_shared(config) || resident_spins(config) == 2;
}

// Lattices of different sizes in one launch of the shared-pack kernel, in the
// shape of the largest, where that takes fewer rounds of its packs than the
// launches of their own would take together, a smaller lattice's round
// counted by its elements (a quarter off: small lattices take more than that):
// 54, 66, 72, 80 and 96 sites, 16 trajectories each, 40 steps: FP32 1.73 ms
// -> 0.66, FP64 2.41 -> 1.81.
void join_packs(const ftwa_instance* inst, Plan* p) {
    for (int var = 0; var < kSharedVariants; ++var) {
        std::vector<int> packs;
        int lead = -1;
        // the launches of their own: items, and the largest lattice
        std::map<std::tuple<int, int, int, int>, std::pair<int64_t, int>> own;
        for (int k = 0; k < p->n_inst; ++k) {
            const InstPlan& ip = p->inst[k];
            if (ip.path != FTWA_PATH_RESIDENT || !resident_is_shared(ip.res.config) ||
                ip.res.variant != var)
                continue;
            packs.push_back(k);
            auto& o = own[std::make_tuple(ip.res.config, ip.res.threads, ip.res.units,
                                          ip.res.workers)];
            o.first += (inst[k].n_traj + ip.res.units - 1) / ip.res.units;
            if (o.second == 0 || inst[k].lat->N > inst[o.second - 1].lat->N) o.second = k + 1;
            if (lead < 0 || inst[k].lat->N > inst[lead].lat->N) lead = k;
        }
        if (own.size() < 2) continue;
        std::vector<ResidentPlan> as(packs.size());
        const ResidentPlan& like = p->inst[lead].res;
        size_t lds = 0;
        int64_t items = 0;
        bool fit = true;
        for (size_t n = 0; n < packs.size() && fit; ++n) {
            const ftwa_instance& in = inst[packs[n]];
            fit = shared_plan_like(like, in.lat->N, host_tables(in.lat), &as[n]);
            lds = std::max(lds, as[n].lds);
            items += (in.n_traj + like.units - 1) / like.units;
        }
        if (!fit) continue;
        auto rounds = [&](int64_t n_items, const ResidentPlan& rp, size_t bytes) {
            const int64_t at_once = std::max<int64_t>(
                1, resident_concurrency(rp.config, bytes, rp.threads, rp.units, var) / rp.units);
            return (double)((n_items + at_once - 1) / at_once);
        };
        double apart = 0;
        for (const auto& [key, o] : own) {
            const InstPlan& ip = p->inst[o.second - 1];
            apart += rounds(o.first, ip.res, ip.res.lds) *
                     (double)packed_count(inst[o.second - 1].lat->N) /
                     (double)packed_count(inst[lead].lat->N);
        }
        if (rounds(items, like, lds) > 0.75 * apart) continue;
        for (size_t n = 0; n < packs.size(); ++n) p->inst[packs[n]].res = as[n];
    }
}

struct PlanMode {
    bool compact = false;  // as little workspace as possible (ftwa_evolve_static)
    bool join = false;     // lattices of different sizes share a launch where that is
                           // faster (not where the run's groups may run side by side)
    bool untuned = false;  // without the autotuner's choices
};
ftwa_status plan_evolve(const ftwa_instance* inst, int n_inst, double dt, int64_t n_steps,
                        int record_every, ftwa_dtype dtype, const ftwa_tuning* tune, Plan* out,
                        const PlanMode& mode = PlanMode()) {
    if (dtype != FTWA_F64 && dtype != FTWA_F32) return fail(FTWA_EINVAL, "unknown dtype");
    if (n_steps < 0) return fail(FTWA_EINVAL, "n_steps < 0");
    if (record_every < 1) return fail(FTWA_EINVAL, "record_every < 1");
    Plan p;
    p.n_inst = n_inst;
    p.n_steps = n_steps;
    p.record_every = record_every;
    p.dt = dt;
    p.dtype = dtype;
    p.n_rec = n_records(n_steps, record_every);
    if (p.n_rec > 65535) return fail(FTWA_EINVAL, "more than 65535 records");
    const ftwa_path want = tune ? tune->path : FTWA_PATH_AUTO;
    if (want != FTWA_PATH_AUTO && want != FTWA_PATH_STREAM && want != FTWA_PATH_RESIDENT)
        return fail(FTWA_EINVAL, "unknown path");
    const int force = tune ? tune->resident_config : -1;
    if (force >= resident_config_count()) return fail(FTWA_EINVAL, "resident_config out of range");
    const int64_t user_chunk = tune && tune->traj_chunk > 0 ? tune->traj_chunk : 0;
    p.spin_limit = tune ? tune->spin_limit : 0;
    p.inject = !tune || !tune->drop_partners ? 0
               : tune->drop_partners == kInjectFarExchange ? kInjectFarExchange
                                                           : kInjectDropPartners;

    // ---- path and configuration of every instance
    // Trajectories of the instances that would share a launch of the
    // shared-pack kernel (a scan of parameters on one lattice): whether an
    // ensemble fills the chip is asked of them together.
    std::map<std::tuple<int, int, int64_t, int>, int64_t> together;
    auto alike = [&](const ftwa_instance& in) {
        const DeviceTables& tab = host_tables(in.lat);
        return std::make_tuple(in.lat->N, tab.n_a, class_shape(tab),
                               (in.v_site ? 1 : 0) + (in.hop_w ? 2 : 0) + (in.u_mat ? 4 : 0));
    };
    for (int k = 0; k < n_inst; ++k)
        if (!inst[k].inv) together[alike(inst[k])] += inst[k].n_traj;
    for (int k = 0; k < n_inst; ++k) {
        InstPlan ip;
        const DeviceTables& tab = host_tables(inst[k].lat);
        const int N = inst[k].lat->N;
        int cfg = force;
        bool tuned_tile = false;  // a resident configuration was faster than the packs
        bool tuned_stream = false;
        Tuned tuned;
        if (cfg < 0 && want == FTWA_PATH_AUTO && !mode.untuned &&
            tuned_config(N, class_shape(tab), dtype, &tuned)) {
            // (a run that takes no packs where the tuned one would: one that is
            // fast with few trajectories may be slow with many, 72 sites FP64
            // with a general interaction tuned at 64 and run with 4000: 46.8
            // ms, untuned 22.9)
            if (!tuned.packs || together[alike(inst[k])] <= 2 * tuned.n_traj) cfg = tuned.config;
            tuned_stream = cfg < 0 && !tuned.packs;
            tuned_tile = cfg >= 0 && !tuned.packs;
        }
        // an external potential: the stream kernels, or a resident configuration
        // with the potential variant
        const bool pot = inst[k].v_site != nullptr;
        // a general interaction: the stream kernels, or a resident configuration
        // with the general-interaction variant (alone)
        const bool gint = inst[k].u_mat != nullptr;
        // complex hopping: the stream kernels, or a resident configuration with
        // the complex-hopping variant (alone)
        const bool hop = inst[k].hop_w != nullptr;
        const int n_var = (pot ? 1 : 0) + (hop ? 1 : 0) + (gint ? 1 : 0);
        if (n_var > 1 && (want == FTWA_PATH_RESIDENT || force >= 0))
            return fail(FTWA_ENOTSUP, "a potential, complex hopping and a general interaction "
                                      "together run on the stream path only");
        auto fits = [&](bool allow_split) {
            if (tuned_stream || n_var > 1 ||
                !resident_plan(N, dtype, tab, &ip.res, cfg, allow_split))
                return false;
            // the configuration chosen for the on-site U, real hopping and no
            // potential, if it has the instance's variant (else the stream path)
            const int c0 = ip.res.config;
            if ((gint && !resident_has_interaction(c0)) || (hop && !resident_has_hop(c0)) ||
                (pot && !resident_has_potential(c0)))
                return false;
            return n_var == 0 ||
                   resident_plan(N, dtype, tab, &ip.res, c0, allow_split, pot, hop, gint);
        };
        bool can_res = fits(inst[k].inv == nullptr);
        // The split configurations keep no invariant sums.  With monitors the
        // automatic path launches them once per record interval and sums the
        // stored state in between: a launch reads and writes the state once,
        // where the stream kernels do so several times a stage (150 sites
        // FP64, 500 trajectories, 50 steps, 6 records: 47.9 ms there, 9.3 ms
        // so; 20 steps with a record after each 20.8 and 12.3 ms, with 64
        // trajectories 3.8 and 3.3 ms).
        if (!can_res && inst[k].inv && !mode.compact && force < 0 && want == FTWA_PATH_AUTO)
            can_res = ip.by_record = fits(true);
        // Small lattices whose shared-pack form fits (with the instance's
        // variant) run there; whether the resident path takes the instance at
        // all was decided above.
        if (can_res && (force < 0 ? !tuned_tile && !inst[k].inv : resident_is_shared(force))) {
            ResidentPlan sp;
            if (shared_plan(N, dtype, tab, together[alike(inst[k])], &sp, force, pot, hop, gint))
                ip.res = sp;
        }
        if (force >= 0 && !can_res)
            return fail(FTWA_ENOTSUP, hop    ? "the forced resident configuration has no "
                                               "complex-hopping variant or does not fit"
                                      : gint ? "the forced resident configuration has no "
                                               "general-interaction variant or does not fit"
                                             : "the forced resident configuration does not fit");
        if (want == FTWA_PATH_RESIDENT && !can_res)
            return fail(FTWA_ENOTSUP, "no resident configuration fits this lattice and dtype");
        ip.path = (want == FTWA_PATH_STREAM || !can_res) ? FTWA_PATH_STREAM : FTWA_PATH_RESIDENT;
        p.inst.push_back(ip);
    }
    if (mode.join && force < 0) join_packs(inst, &p);

    // ---- groups: instances of one launch
    // (8 config + 4 (general interaction) + 2 (complex hopping) + (external
    // potential), threads, units, workers, 1 + the instance if it is launched
    // per record interval)
    std::map<std::tuple<int, int, int, int, int>, int> group_of_config;
    for (int k = 0; k < n_inst; ++k) {
        InstPlan& ip = p.inst[k];
        if (ip.path != FTWA_PATH_RESIDENT) continue;
        // instances with a potential form groups of their own: their
        // launches run the potential variant, whose LDS layout holds the
        // profile and is sized for it
        const auto key = std::make_tuple(
            8 * ip.res.config + (inst[k].u_mat ? 4 : 0) + (inst[k].hop_w ? 2 : 0) +
                (inst[k].v_site ? 1 : 0),
            ip.res.threads, ip.res.units, ip.res.workers, ip.by_record ? 1 + k : 0);
        auto it = group_of_config.find(key);
        if (it == group_of_config.end()) {
            it = group_of_config.emplace(key, (int)p.groups.size()).first;
            GroupPlan g;
            g.config = ip.res.config;
            g.threads = ip.res.threads;
            g.units = ip.res.units;
            g.workers = ip.res.workers;
            g.variant = ip.res.variant;
            g.by_record = ip.by_record;
            p.groups.push_back(g);
        }
        ip.group = it->second;
        GroupPlan& g = p.groups[ip.group];
        g.members.push_back(k);
        g.lds = std::max(g.lds, ip.res.lds);
        g.Nmax = std::max(g.Nmax, inst[k].lat->N);
    }

    // ---- stream instances: chunks of trajectories, one after another
    size_t s_state = 0, s_x = 0, s_mom = 0, s_inv = 0, s_D = 0;
    for (int k = 0; k < n_inst; ++k) {
        InstPlan& ip = p.inst[k];
        if (ip.path != FTWA_PATH_STREAM) continue;
        const int N = inst[k].lat->N;
        const int D = 2 * N;
        const int64_t traj = std::max<int64_t>(inst[k].n_traj, 1);
        const int64_t rec_cap = std::max<int64_t>(
            64, (int64_t)(kRecordBudget / ((size_t)p.n_rec * D * sizeof(double))));
        int64_t chunk = user_chunk > 0 ? user_chunk : kStreamChunk;
        chunk = std::max<int64_t>(1, std::min({chunk, traj, rec_cap}));
        ip.chunk = chunk;
        s_state = std::max(s_state, (size_t)2 * packed_count(N) * chunk * cplx_bytes(dtype));
        s_x = std::max(s_x, (size_t)p.n_rec * D * chunk * sizeof(double));
        s_mom = std::max(s_mom, moments_workspace_bytes(D, chunk, p.n_rec));
        if (inst[k].inv) s_inv = std::max(s_inv, (size_t)p.n_rec * 4 * chunk * sizeof(double));
        if (inst[k].u_mat) s_D = std::max(s_D, (size_t)2 * N * chunk * sizeof(double));
    }
    size_t off = kStatusBytes;  // the run's status block comes first
    p.s_acc = off; off = align_up(off + s_state);
    p.s_ya = off;  off = align_up(off + s_state);
    p.s_yb = off;  off = align_up(off + s_state);
    p.s_x = off;   off = align_up(off + s_x);
    p.s_mom = off; off = align_up(off + s_mom);
    p.s_inv = off; off = align_up(off + s_inv);
    p.s_D = off;   off = align_up(off + s_D);
    p.s_total = off;

    // ---- resident instances: passes over trajectory windows.  Their area
    // follows the stream area (no overlap: the launch tables are uploaded
    // before the stream-path instances run, and must survive them)
    size_t rec_bytes = 0;
    for (int k = 0; k < n_inst; ++k) {
        if (p.inst[k].path != FTWA_PATH_RESIDENT) continue;
        const int D = 2 * inst[k].lat->N;
        rec_bytes += (size_t)p.n_rec * (D + (inst[k].inv ? 4 : 0)) * inst[k].n_traj * sizeof(double);
    }
    int64_t n_pass_goal = std::max<int64_t>(1, (int64_t)((rec_bytes + kRecordBudget - 1) / kRecordBudget));
    p.n_pass = 0;
    for (int k = 0; k < n_inst; ++k) {
        InstPlan& ip = p.inst[k];
        if (ip.path != FTWA_PATH_RESIDENT) continue;
        const int64_t M = inst[k].n_traj;
        int64_t c;
        if (user_chunk > 0) {
            c = user_chunk;
        } else {
            // whole rounds of the trajectories the group runs at once
            const int64_t align = std::max<int64_t>(
                1, resident_concurrency(ip.res.config, p.groups[ip.group].lds, ip.res.threads,
                                        ip.res.units, ip.res.variant));
            c = (M + n_pass_goal - 1) / n_pass_goal;
            c = (c + align - 1) / align * align;
        }
        c = std::max<int64_t>(1, std::min(c, std::max<int64_t>(M, 1)));
        ip.chunk = c;
        p.n_pass = std::max<int>(p.n_pass, (int)((M + c - 1) / c));
    }
    off = p.s_total;
    for (int k = 0; k < n_inst; ++k) {
        InstPlan& ip = p.inst[k];
        if (ip.path != FTWA_PATH_RESIDENT) continue;
        const int D = 2 * inst[k].lat->N;
        ip.off_x = off; off = align_up(off + (size_t)p.n_rec * D * ip.chunk * sizeof(double));
        if (inst[k].hop_w) {
            ip.off_hop = off;
            off = align_up(off + (size_t)(2 * p.n_steps + 1) * inst[k].lat->N * 3 *
                                     cplx_bytes(p.dtype));
        }
        if (inst[k].u_mat) {
            ip.off_umat = off;
            off = align_up(off + (size_t)umat_rows(inst[k].lat->N) * inst[k].lat->N *
                                   cplx_bytes(p.dtype) / 2);
        }
        if (inst[k].inv) {
            ip.off_inv = off;
            off = align_up(off + (size_t)p.n_rec * 4 * ip.chunk * sizeof(double));
        }
    }
    size_t r_mom = 0;  // compact: one region for all groups
    for (GroupPlan& g : p.groups) {
        size_t need = 0;
        for (int k : g.members)
            need = std::max(need, moments_workspace_bytes(2 * inst[k].lat->N, p.inst[k].chunk, p.n_rec));
        g.off_mom = off;
        r_mom = std::max(r_mom, need);
        if (!mode.compact) off = align_up(off + need);
    }
    if (mode.compact) off = align_up(off + r_mom);
    // launches and their table entries
    int64_t entry = 0;
    for (int j = 0; j < p.n_pass; ++j)
        for (int gi = 0; gi < (int)p.groups.size(); ++gi) {
            GroupPlan& g = p.groups[gi];
            LaunchDesc L;
            L.group = gi;
            L.first_entry = entry;
            for (int k : g.members) {
                int64_t m0, Mc;
                window(p, inst[k], k, j, &m0, &Mc);
                if (Mc <= 0) continue;
                const int64_t per = g.units;
                L.n_items += (Mc + per - 1) / per;
                L.work += (double)Mc * n_steps;
                if (inst[k].lat->t != 1.0) L.unit_hop = false;
                if (inst[k].v_site) L.potential = true;
                if (inst[k].hop_w) L.hopping = true;
                if (inst[k].u_mat) L.interaction = true;
                ++L.n_entries;
            }
            entry += L.n_entries;
            g.max_items = std::max(g.max_items, L.n_items);
            L.grid = resident_grid(g.config, g.lds, std::max<int64_t>(L.n_items, 1), g.threads,
                                   g.units, g.variant);
            if (n_inst > 1 && waits_for_none(g.config))
                L.share = (double)L.grid * g.units /
                          (double)std::max<int64_t>(
                              1, resident_concurrency(g.config, g.lds, g.threads, g.units, g.variant));
            p.launches.push_back(L);
        }
    p.n_table = entry;
    for (GroupPlan& g : p.groups) {
        g.off_mb = off;
        off = align_up(off + resident_mailbox_bytes(g.config, g.Nmax, std::max<int64_t>(g.max_items, 1)));
    }
    p.r_table = off; off = align_up(off + (size_t)std::max<int64_t>(entry, 1) * sizeof(ResidentInst));
    p.r_total = off;
    p.total = p.r_total;
    *out = std::move(p);
    return FTWA_OK;
}

// The table of a resident plan (not of the shared packs').
TableShape table_shape(const ResidentPlan& rp, ftwa_dtype dtype) {
    TableShape sh;
    sh.G = resident_parts(rp.config);
    sh.even_slots = rp.even_slots;
    sh.odd_slots = rp.odd_slots;
    if (sh.G > 1) sh.bnd_entry = rp.bnd_entry;
    else sh.compact = resident_spins(rp.config) == 1;
    sh.elem_bytes = (int)cplx_bytes(dtype);
    return sh;
}

// Host work before the launches, nothing queued: the launch-table entries
// (their descriptor tables looked up; ftwa_lattice_upload created them) and
// the kernels' LDS limits.  Not under graph capture.
ftwa_status build_table(Plan& p, const ftwa_instance* inst, char* ws) {
    ftwa_status st;
    p.table.clear();
    p.table.reserve((size_t)p.n_table);
    for (int j = 0; j < p.n_pass; ++j)
        for (const GroupPlan& g : p.groups) {
            int64_t item0 = 0;
            const int64_t per = g.units;
            for (int k : g.members) {
                int64_t m0, Mc;
                window(p, inst[k], k, j, &m0, &Mc);
                if (Mc <= 0) continue;
                const InstPlan& ip = p.inst[k];
                ResidentInst e = {};
                e.N = inst[k].lat->N;
                e.P = (int)packed_count(e.N);
                e.Mc = Mc;
                e.rho = static_cast<char*>(inst[k].rho) + (size_t)m0 * cplx_bytes(p.dtype);
                e.ldr = inst[k].n_traj;
                e.part_words = 0;
                e.hmax = 0;
                if (resident_is_shared(g.config)) {
                    if ((st = shared_lists(inst[k].lat, ip.res.lanes, &e.stab)) != FTWA_OK)
                        return st;
                } else {
                    const TableShape sh = table_shape(ip.res, p.dtype);
                    st = sh.G > 1 ? split_tables(inst[k].lat, sh, &e.desc, &e.part_words, &e.hmax)
                                  : padded_descriptors(inst[k].lat, sh, &e.desc);
                    if (st != FTWA_OK) return st;
                }
                DeviceTables tab;
                if ((st = device_tables(inst[k].lat, &tab)) != FTWA_OK) return st;
                e.ord = tab.ord;
                e.nb = tab.nb;
                e.dpos = tab.dpos;
                e.n_a = tab.n_a;
                e.t = inst[k].lat->t;
                e.U = inst[k].U;
                e.X = reinterpret_cast<double*>(ws + ip.off_x);
                e.inv_parts = inst[k].inv && !ip.by_record
                                  ? reinterpret_cast<double*>(ws + ip.off_inv)
                                  : nullptr;
                e.item0 = item0;
                item0 += (Mc + per - 1) / per;
                e.dump = p.dump ? static_cast<char*>(p.dump) + (size_t)m0 * cplx_bytes(p.dtype)
                                : nullptr;
                e.dump_stride = p.dump_stride;
                e.v_site = inst[k].v_site;
                e.v_env = inst[k].v_env;
                e.hop = inst[k].hop_w ? ws + ip.off_hop : nullptr;
                e.umat = inst[k].u_mat ? ws + ip.off_umat : nullptr;
                e.u_lds = inst[k].u_mat && ip.res.u_lds ? 1 : 0;
                p.table.push_back(e);
            }
        }
    // the stream path's tables must be on this device as well
    for (int k = 0; k < p.n_inst; ++k) {
        DeviceTables tab;
        if ((st = device_tables(inst[k].lat, &tab)) != FTWA_OK) return st;
    }
    for (const GroupPlan& g : p.groups)
        if ((st = resident_prepare(g.config, g.lds)) != FTWA_OK) return st;
    return FTWA_OK;
}

// A resident launch per record interval, the invariant sums of the state
// before the first and after each full one.  L: the launch of the whole run,
// whose only table entry is rewritten for every interval (its records and its
// potential's envelope start where the interval does; monitors exclude complex
// hopping and a general interaction).
ftwa_status launch_by_record(const Plan& p, const ftwa_instance& in, int k, const LaunchDesc& Ld,
                             ResidentLaunch L, char* ws, hipStream_t stream, KernelTimer& timer) {
    ftwa_status st;
    const InstPlan& ip = p.inst[k];
    const ResidentInst& e = p.table[(size_t)Ld.first_entry];
    DeviceTables tab;
    if ((st = device_tables(in.lat, &tab)) != FTWA_OK) return st;
    StreamChunk c;
    c.N = e.N;
    c.P = e.P;
    c.Mc = e.Mc;
    c.y = e.rho;
    c.ldy = e.ldr;
    double* const parts = reinterpret_cast<double*>(ws + ip.off_inv);
    if ((st = record_inv(c, tab, p.dtype, parts, stream)) != FTWA_OK) return st;
    const int64_t every = p.record_every;
    for (int64_t r = 0, step = 0; step < p.n_steps || r == 0; ++r, step += every) {
        if (r > 0) {
            TableChunk t;
            t.n = 1;
            t.e[0] = e;
            t.e[0].X = e.X + r * 2 * e.N * e.Mc;
            if (e.v_env) t.e[0].v_env = e.v_env + 2 * step;
            hipLaunchKernelGGL(write_table_kernel, dim3(1), dim3(256), 0, stream,
                               reinterpret_cast<ResidentInst*>(ws + p.r_table) + Ld.first_entry, t);
            FTWA_LAUNCH_CHECK("write_table_kernel");
        }
        L.n_steps = std::min(every, p.n_steps - step);
        if ((st = timer.begin(stream)) != FTWA_OK) return st;
        if ((st = resident_launch(L, stream)) != FTWA_OK) return st;
        if ((st = timer.end(stream, 1, (double)e.Mc * L.n_steps)) != FTWA_OK) return st;
        if (L.n_steps == every &&
            (st = record_inv(c, tab, p.dtype, parts + (r + 1) * 4 * e.Mc, stream)) != FTWA_OK)
            return st;
    }
    return FTWA_OK;
}

// Side branches of a captured run: the nodes that the capturing stream's next
// launch follows, read and set (streams and events of their own for the
// branches took a third of a graph's creation).
constexpr int kBranches = 3;
using Nodes = std::vector<hipGraphNode_t>;
ftwa_status capture_tail(hipStream_t stream, Nodes* tail) {
    hipStreamCaptureStatus status;
    const hipGraphNode_t* at = nullptr;
    size_t n = 0;
    FTWA_HIP_TRY(hipStreamGetCaptureInfo_v2(stream, &status, nullptr, nullptr, &at, &n));
    tail->assign(at, at + n);
    return FTWA_OK;
}
ftwa_status capture_after(hipStream_t stream, Nodes tail) {
    FTWA_HIP_TRY(hipStreamUpdateCaptureDependencies(stream, tail.data(), tail.size(),
                                                    hipStreamSetCaptureDependencies));
    return FTWA_OK;
}

// Whether instances of different groups write to the same memory (slices of an
// ensemble whose moments meet in one S1 and S2, say): such groups keep their
// order on one stream.
bool groups_share_outputs(const Plan& p, const ftwa_instance* inst) {
    struct Range {
        const char *lo, *hi;
        int group;
    };
    std::vector<Range> all;
    for (int k = 0; k < p.n_inst; ++k) {
        const ftwa_instance& in = inst[k];
        const int N = in.lat->N;
        auto add = [&](const void* at, size_t bytes) {
            const char* lo = static_cast<const char*>(at);
            if (lo && bytes > 0) all.push_back({lo, lo + bytes, p.inst[k].group});
        };
        add(in.rho, (size_t)2 * packed_count(N) * in.n_traj * cplx_bytes(p.dtype));
        add(in.S1, (size_t)p.n_rec * 2 * N * sizeof(double));
        add(in.S2, (size_t)p.n_rec * s2_count(2 * N) * sizeof(double));
        add(in.inv, (size_t)p.n_rec * 4 * sizeof(double));
    }
    std::sort(all.begin(), all.end(), [](const Range& a, const Range& b) { return a.lo < b.lo; });
    Range far = {nullptr, nullptr, -1};  // the range so far that ends last
    for (const Range& r : all) {
        if (r.lo < far.hi && r.group != far.group) return true;
        if (r.hi > far.hi) far = r;
    }
    return false;
}

// Queues every launch of the run on `stream` (and nothing else: no host
// synchronisation), so that it can be captured into a graph.  fork (while the
// library captures `stream` only): the groups whose workgroups wait for no other run side by
// side once the spin-split and split groups are through (those fill the chip
// and need their workgroups resident together), if the chip holds all their
// workgroups at once, or nearly, or in fewer rounds than there are groups of
// one round each; otherwise persistent workgroups of several kernels share CUs
// for the whole run.  Groups that write to the same memory stay in order.
// Graphs of six lattices of 10 to 96 sites, 64 trajectories each, 100 steps:
// FP32 2.80 ms one after another, 1.55 so; FP64 5.09 and 3.21.  40, 54 and 66
// sites FP64, 96 trajectories each, which take somewhat more than the chip, 1.93
// and 1.37.  24, 54 and 96 sites FP64, 256 each, twice the chip: 3.8 and 5.4;
// FP32 with 4096 each, 20 steps: 6.0 and 9.0.  54 sites FP32, the four
// Hamiltonian variants, 128 trajectories each, half the chip (a CU holds one
// workgroup), 40 steps: 1.11 and 0.64.
constexpr double kForkShare = 1.25;
ftwa_status execute(const Plan& p, const ftwa_instance* inst, char* ws, hipStream_t stream,
                    KernelTimer& timer, bool cooperative, bool fork = false) {
    ftwa_status st;
    uint32_t* status = reinterpret_cast<uint32_t*>(ws + p.off_status);
    Prologue pro;
    pro.status = status;
    size_t e0 = 0;
    int64_t longest = 0;
    auto flush = [&]() -> ftwa_status {
        const size_t left = p.table.size() - e0;
        pro.table = reinterpret_cast<ResidentInst*>(ws + p.r_table) + e0;
        pro.c.n = (int)std::min<size_t>(kTableChunk, left);
        if (pro.c.n) std::memcpy(pro.c.e, p.table.data() + e0, (size_t)pro.c.n * sizeof(ResidentInst));
        const int64_t blocks = std::min<int64_t>(std::max<int64_t>((longest + 1023) / 1024, 1), 1024);
        hipLaunchKernelGGL(prologue_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, pro);
        FTWA_LAUNCH_CHECK("prologue_kernel");
        e0 += (size_t)pro.c.n;
        pro.status = nullptr;
        pro.n_fill = 0;
        longest = 0;
        return FTWA_OK;
    };
    pro.n_fill = 0;
    auto clear = [&](double* d, int64_t n) -> ftwa_status {
        if (n <= 0) return FTWA_OK;
        if (pro.n_fill == kPrologueFills && (st = flush()) != FTWA_OK) return st;
        pro.fill[pro.n_fill].p = d;
        pro.fill[pro.n_fill++].n = n;
        longest = std::max(longest, n);
        return FTWA_OK;
    };
    for (int k = 0; k < p.n_inst; ++k) {
        const ftwa_instance& in = inst[k];
        const int D = 2 * in.lat->N;
        if ((st = clear(in.S1, p.n_rec * D)) != FTWA_OK) return st;
        if ((st = clear(in.S2, p.n_rec * s2_count(D))) != FTWA_OK) return st;
        if (in.inv && (st = clear(in.inv, p.n_rec * 4)) != FTWA_OK) return st;
    }
    do {
        if ((st = flush()) != FTWA_OK) return st;
    } while (e0 < p.table.size());
    // ---- stream instances
    for (int k = 0; k < p.n_inst; ++k) {
        const InstPlan& ip = p.inst[k];
        if (ip.path != FTWA_PATH_STREAM) continue;
        const ftwa_instance& in = inst[k];
        DeviceTables tab;
        if ((st = device_tables(in.lat, &tab)) != FTWA_OK) return st;
        const int N = in.lat->N;
        const int D = 2 * N;
        double* X = reinterpret_cast<double*>(ws + p.s_x);
        double* parts = in.inv ? reinterpret_cast<double*>(ws + p.s_inv) : nullptr;
        for (int64_t m0 = 0; m0 < in.n_traj; m0 += ip.chunk) {
            const int64_t Mc = std::min(ip.chunk, in.n_traj - m0);
            StreamChunk c;
            c.N = N;
            c.P = packed_count(N);
            c.Mc = Mc;
            c.y = static_cast<char*>(in.rho) + (size_t)m0 * cplx_bytes(p.dtype);
            c.ldy = in.n_traj;
            c.acc = ws + p.s_acc;
            c.ya = ws + p.s_ya;
            c.yb = ws + p.s_yb;
            c.t = in.lat->t;
            c.U = in.U;
            c.dt = p.dt;
            c.v_site = in.v_site;
            c.v_env = in.v_env;
            c.u_mat = in.u_mat;
            c.D = in.u_mat ? ws + p.s_D : nullptr;
            c.hop_w = in.hop_w;
            if ((st = record_diag(c, tab, p.dtype, X, stream)) != FTWA_OK) return st;
            if (parts && (st = record_inv(c, tab, p.dtype, parts, stream)) != FTWA_OK) return st;
            int64_t open_steps = 0;
            for (int64_t step = 1; step <= p.n_steps; ++step) {
                if (open_steps == 0 && (st = timer.begin(stream)) != FTWA_OK) return st;
                c.step = step - 1;
                if ((st = stream_step(c, tab, p.dtype, stream)) != FTWA_OK) return st;
                ++open_steps;
                if (open_steps == 64 || step == p.n_steps) {
                    if ((st = timer.end(stream, 4 * open_steps, (double)Mc * open_steps)) != FTWA_OK)
                        return st;
                    open_steps = 0;
                }
                if (step % p.record_every == 0) {
                    const int64_t r = step / p.record_every;
                    if ((st = record_diag(c, tab, p.dtype, X + r * D * Mc, stream)) != FTWA_OK)
                        return st;
                    if (parts &&
                        (st = record_inv(c, tab, p.dtype, parts + r * 4 * Mc, stream)) != FTWA_OK)
                        return st;
                }
            }
            if ((st = moments_accumulate(D, Mc, p.n_rec, X, in.S1, in.S2, ws + p.s_mom, stream)) !=
                FTWA_OK)
                return st;
            if (parts && (st = invariants_accumulate(N, Mc, p.n_rec, in.lat->t, in.U, X, parts,
                                                     in.inv, stream)) != FTWA_OK)
                return st;
        }
    }
    // ---- resident groups, pass by pass
    // the ratio tables of the instances with complex hopping first
    for (int k = 0; k < p.n_inst; ++k) {
        const InstPlan& ip = p.inst[k];
        if (ip.path != FTWA_PATH_RESIDENT || !inst[k].hop_w) continue;
        DeviceTables tab;
        if ((st = device_tables(inst[k].lat, &tab)) != FTWA_OK) return st;
        // spin split: place order (the partner's diagonal); shared blocks:
        // site order
        const int32_t* const order = resident_spins(ip.res.config) == 1 ? tab.dpos : nullptr;
        if ((st = hop_table(inst[k].hop_w, tab.nb, order, inst[k].lat->N, p.n_steps, p.dtype,
                            ws + ip.off_hop, stream)) != FTWA_OK)
            return st;
    }
    for (int k = 0; k < p.n_inst; ++k) {
        const InstPlan& ip = p.inst[k];
        if (ip.path != FTWA_PATH_RESIDENT || !inst[k].u_mat) continue;
        if ((st = umat_table(inst[k].u_mat, inst[k].lat->N, p.dtype, ws + ip.off_umat, stream)) !=
            FTWA_OK)
            return st;
    }
    const ResidentInst* table = reinterpret_cast<const ResidentInst*>(ws + p.r_table);
    auto launch_group = [&](int j, size_t gi, hipStream_t q) -> ftwa_status {
        const LaunchDesc& Ld = p.launches[(size_t)j * p.groups.size() + gi];
        if (Ld.n_items == 0) return FTWA_OK;
        const GroupPlan& g = p.groups[gi];
        ResidentLaunch L;
        L.config = g.config;
        L.lds = g.lds;
        L.table = table + Ld.first_entry;
        L.n_entries = Ld.n_entries;
        L.n_items = Ld.n_items;
        L.grid = Ld.grid;
        L.threads = g.threads;
        L.units = g.units;
        L.workers = g.workers;
        L.Nmax = g.Nmax;
        L.dt = p.dt;
        L.n_steps = p.n_steps;
        L.record_every = p.record_every;
        L.mailbox = ws + g.off_mb;
        L.error = reinterpret_cast<int*>(status + 1);
        L.spin_limit = p.spin_limit;
        L.inject = p.inject;
        L.cooperative = cooperative;
        L.unit_hop = Ld.unit_hop;
        L.dumps = p.dump != nullptr;
        L.potential = Ld.potential;
        L.hopping = Ld.hopping;
        L.interaction = Ld.interaction;
        if (g.by_record)
            return launch_by_record(p, inst[g.members[0]], g.members[0], Ld, L, ws, q, timer);
        if ((st = timer.begin(q)) != FTWA_OK) return st;
        if ((st = resident_launch(L, q)) != FTWA_OK) return st;
        return timer.end(q, 1, Ld.work);
    };
    auto reduce_group = [&](int j, size_t gi, hipStream_t q) -> ftwa_status {
        for (int k : p.groups[gi].members) {
            const InstPlan& ip = p.inst[k];
            const ftwa_instance& in = inst[k];
            int64_t m0, Mc;
            window(p, in, k, j, &m0, &Mc);
            if (Mc <= 0) continue;
            const int N = in.lat->N;
            double* X = reinterpret_cast<double*>(ws + ip.off_x);
            if ((st = moments_accumulate(2 * N, Mc, p.n_rec, X, in.S1, in.S2,
                                         ws + p.groups[gi].off_mom, q)) != FTWA_OK)
                return st;
            if (in.inv &&
                (st = invariants_accumulate(N, Mc, p.n_rec, in.lat->t, in.U, X,
                                            reinterpret_cast<double*>(ws + ip.off_inv), in.inv,
                                            q)) != FTWA_OK)
                return st;
        }
        return FTWA_OK;
    };
    const bool may_fork = fork && p.groups.size() > 1 && !groups_share_outputs(p, inst);
    for (int j = 0; j < p.n_pass; ++j) {
        std::vector<size_t> apart;  // the groups that run side by side
        if (may_fork) {
            double share = 0;
            bool one_round = true;
            for (size_t gi = 0; gi < p.groups.size(); ++gi) {
                const LaunchDesc& Ld = p.launches[(size_t)j * p.groups.size() + gi];
                if (!waits_for_none(p.groups[gi].config) || Ld.n_items == 0) continue;
                apart.push_back(gi);
                share += Ld.share;
                one_round = one_round && Ld.grid >= Ld.n_items;
            }
            if (share > kForkShare && (!one_round || std::ceil(share) >= (double)apart.size()))
                apart.clear();
        }
        for (size_t gi = 0; gi < p.groups.size(); ++gi)
            if (std::find(apart.begin(), apart.end(), gi) == apart.end() &&
                (st = launch_group(j, gi, stream)) != FTWA_OK)
                return st;
        Nodes base, tail[kBranches];  // before the branches, and of each
        if (!apart.empty() && (st = capture_tail(stream, &base)) != FTWA_OK) return st;
        for (size_t n = 0; n < apart.size(); ++n) {
            Nodes& branch = tail[n % kBranches];
            if ((st = capture_after(stream, n < kBranches ? base : branch)) != FTWA_OK ||
                (st = launch_group(j, apart[n], stream)) != FTWA_OK ||
                (st = reduce_group(j, apart[n], stream)) != FTWA_OK ||
                (st = capture_tail(stream, &branch)) != FTWA_OK)
                return st;
        }
        if (!apart.empty() && (st = capture_after(stream, base)) != FTWA_OK) return st;
        for (size_t gi = 0; gi < p.groups.size(); ++gi)
            if (std::find(apart.begin(), apart.end(), gi) == apart.end() &&
                (st = reduce_group(j, gi, stream)) != FTWA_OK)
                return st;
        if (!apart.empty()) {
            Nodes all;
            if ((st = capture_tail(stream, &all)) != FTWA_OK) return st;
            if (all == base) all.clear();  // every branch follows it
            for (const Nodes& t : tail) all.insert(all.end(), t.begin(), t.end());
            if ((st = capture_after(stream, all)) != FTWA_OK) return st;
        }
    }
    // ---- non-finite trajectories counted by the invariant monitors
    for (int k = 0; k < p.n_inst; ++k) {
        if (!inst[k].inv) continue;
        hipLaunchKernelGGL(status_nonfinite_kernel, dim3(1), dim3(64), 0, stream, inst[k].inv,
                           p.n_rec, (uint32_t)std::min(k, 0xffff), status);
        FTWA_LAUNCH_CHECK("status_nonfinite_kernel");
    }
    return FTWA_OK;
}

// Waits for `stream` and reports what the status block of the last run in
// the workspace recorded: a bounded wait that gave up (FTWA_ETIMEOUT), then
// non-finite trajectories (FTWA_ENONFINITE).
ftwa_status check_status(const char* ws, hipStream_t stream) {
    uint32_t h[4] = {0, 0, 0, 0};
    FTWA_HIP_TRY(hipMemcpyAsync(h, ws, sizeof(h), hipMemcpyDeviceToHost, stream));
    FTWA_HIP_TRY(hipStreamSynchronize(stream));
    if (h[0] != kStatusMagic) return fail(FTWA_EINVAL, "no ftwa_evolve run recorded in this workspace");
    if (h[1] != 0)
        return fail(FTWA_ETIMEOUT,
                    "a workgroup of a resident run timed out waiting for the others of its "
                    "trajectory (were they resident together?)");
    if (h[2] != 0)
        return fail(FTWA_ENONFINITE, "instance " + std::to_string(h[3] >> 16) +
                                         ": a trajectory became non-finite by record " +
                                         std::to_string(h[3] & 0xffffu));
    return FTWA_OK;
}

// ---------------------------------------------------------------- static workspace
// The workspace of ftwa_evolve_static: a fixed array in device memory that
// the code object brings with it (each device the library runs on holds its
// own copy until the process ends).  Its name is only a host-side stand-in:
// host code uses the device address hipGetSymbolAddress returns, kept per
// device.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

std::mutex g_scratch_mu;
std::map<int, char*> g_scratch_ptr;  // device ordinal -> address of its copy

// The address of the current device's copy, looked up once per device.
ftwa_status static_scratch(char** out) {
    int dev = 0;
    FTWA_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    auto it = g_scratch_ptr.find(dev);
    if (it == g_scratch_ptr.end()) {
        void* ptr = nullptr;
        FTWA_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(FTWA_EHIP, "hipGetSymbolAddress returned no address");
        it = g_scratch_ptr.emplace(dev, static_cast<char*>(ptr)).first;
    }
    *out = it->second;
    return FTWA_OK;
}

// ---------------------------------------------------------------- tuning table
std::mutex g_tune_mu;
std::map<std::tuple<int, int, int64_t, int>, Tuned> g_tuned;

int current_device() {
    int d = 0;
    (void)hipGetDevice(&d);
    return d;
}

}  // namespace

// ---------------------------------------------------------------- stored-state runs
// Resident integration of one instance (rho updated in place) that also
// stores the state at every record: record r >= 1 (after r * record_every
// steps) goes to dump + (r - 1) * dump_stride elements, in the layout of rho
// (leading dimension in.n_traj).  For the adjoint's checkpoints and segment
// states.  With ws == NULL only *bytes is set; fails with FTWA_ENOTSUP when
// no resident configuration fits.
ftwa_status evolve_stored(const ftwa_instance& in, double dt, int64_t n_steps, int record_every,
                          ftwa_dtype dtype, void* dump, int64_t dump_stride, char* ws,
                          size_t* bytes, hipStream_t stream) {
    ftwa_tuning tune;
    std::memset(&tune, 0, sizeof(tune));
    tune.path = FTWA_PATH_RESIDENT;
    tune.resident_config = -1;
    // Packs of small lattices first, as in ordinary runs (whole gradients, 1024
    // trajectories, 200 steps: 54 sites FP32 stored every 50 steps 20.6 ms, on
    // the tiles 21.8, every 5 steps 22.8 and 25.2; FP64 37.0 and 38.7, 39.7 and
    // 42.0; 12 sites FP32 2.9 and 3.7, 3.2 and 4.5), but not in five slots per
    // thread, whose stores of a state take longer than its integration gains
    // (40 steps stored one by one and 1024 trajectories FP32: 96 sites, five
    // slots, 56.7 ms, on the tiles 49.3; 90 sites, three, 38.2 and 43.6).  Then
    // the shared-block tiles with several trajectories per workgroup (their
    // stores of neighbouring trajectories share cache lines; the single-unit
    // tiles that ordinary runs prefer took the 54-site checkpoint run from 0.24
    // to 0.38 s), then the usual first fit (spin split, split kernel).
    static const int kStoredPreference[] = {0, 13, 1, 23, 24, 14, 2, 15, 3,
                                            4, 16, 5, 17, 6, 18, 7};
    const DeviceTables& tab = host_tables(in.lat);
    ResidentPlan rp;
    const bool packs = !in.inv &&
                       shared_plan(in.lat->N, dtype, tab, in.n_traj, &rp, -1,
                                   in.v_site != nullptr, in.hop_w != nullptr,
                                   in.u_mat != nullptr) &&
                       rp.even_slots < 5 * (rp.workers / rp.lanes);
    for (int c : kStoredPreference) {
        if (packs) break;
        if (resident_plan(in.lat->N, dtype, tab, &rp, c, in.inv == nullptr)) {
            tune.resident_config = c;
            break;
        }
    }
    Plan plan;
    ftwa_status st = plan_evolve(&in, 1, dt, n_steps, record_every, dtype, &tune, &plan);
    if (st != FTWA_OK) return st;
    if (!ws) {
        *bytes = plan.total;
        return FTWA_OK;
    }
    if (*bytes < plan.total) return fail(FTWA_EINVAL, "stored-state run: workspace too small");
    plan.dump = dump;
    plan.dump_stride = dump_stride;
    if ((st = build_table(plan, &in, ws)) != FTWA_OK) return st;
    KernelTimer off(false);
    if ((st = execute(plan, &in, ws, stream, off, true)) != FTWA_OK) return st;
    return check_status(ws, stream);
}

bool tuned_config(int N, int64_t shape, ftwa_dtype dtype, Tuned* tuned) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    auto it = g_tuned.find(std::make_tuple(current_device(), N, shape, (int)dtype));
    if (it == g_tuned.end()) return false;
    *tuned = it->second;
    return true;
}

void set_tuned_config(int N, int64_t shape, ftwa_dtype dtype, const Tuned& tuned) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    g_tuned[std::make_tuple(current_device(), N, shape, (int)dtype)] = tuned;
}

}  // namespace ftwa

using namespace ftwa;

struct ftwa_graph_s {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    Plan plan;
    std::vector<ftwa_instance> inst;
    char* ws = nullptr;
};

extern "C" {

ftwa_status ftwa_lattice_upload(ftwa_lattice lat) {
    if (!lat) return fail(FTWA_EINVAL, "ftwa_lattice_upload: NULL lattice");
    int dev = 0;
    FTWA_HIP_TRY(hipGetDevice(&dev));
    if (uploaded(lat, dev)) return FTWA_OK;
    const DeviceTables& tab = host_tables(lat);
    ftwa_status st;
    std::vector<TableShape> shapes;
    std::set<int> configs;
    // every table a plan may look up: each configuration that holds the
    // lattice, in either precision, with and without the potential's layout
    // (a lattice that is not bipartite takes the stream path, which needs none)
    for (int c = 0; c < resident_config_count(); ++c)
        for (ftwa_dtype dtype : {FTWA_F64, FTWA_F32})
            for (bool pot : {false, true}) {
                ResidentPlan rp;
                if (resident_is_shared(c) ||
                    !resident_plan(lat->N, dtype, tab, &rp, c, true, pot))
                    continue;
                shapes.push_back(table_shape(rp, dtype));
                configs.insert(c);
            }
    const std::map<int, int> passes = shared_passes(lat->N, tab, &configs);
    for (int c : configs)
        if ((st = resident_prepare(c, 0)) != FTWA_OK) return st;
    return upload_tables(lat, dev, shapes, passes);
}

ftwa_status ftwa_evolve_workspace_size(const ftwa_instance* inst, int n_inst, int64_t n_steps,
                                       int record_every, ftwa_dtype dtype,
                                       const ftwa_tuning* tune, size_t* bytes) {
    ftwa_status st = check_instances(inst, n_inst, false, "ftwa_evolve_workspace_size");
    if (st != FTWA_OK) return st;
    if (!bytes) return fail(FTWA_EINVAL, "bytes is NULL");
    Plan plan;
    if ((st = plan_evolve(inst, n_inst, 0.0, n_steps, record_every, dtype, tune, &plan)) != FTWA_OK)
        return st;
    *bytes = plan.total;
    return FTWA_OK;
}

ftwa_status ftwa_evolve(const ftwa_instance* inst, int n_inst, double dt, int64_t n_steps,
                        int record_every, ftwa_dtype dtype, const ftwa_tuning* tune,
                        void* workspace, size_t workspace_bytes, void* stream_) {
    ftwa_status st = check_instances(inst, n_inst, true, "ftwa_evolve");
    if (st != FTWA_OK) return st;
    Plan plan;
    PlanMode mode;
    mode.join = true;
    if ((st = plan_evolve(inst, n_inst, dt, n_steps, record_every, dtype, tune, &plan, mode)) !=
        FTWA_OK)
        return st;
    // a joined launch's passes may be of other sizes than the ones asked for
    mode.join = false;
    if (workspace_bytes < plan.total &&
        (st = plan_evolve(inst, n_inst, dt, n_steps, record_every, dtype, tune, &plan, mode)) !=
            FTWA_OK)
        return st;
    if (workspace_bytes < plan.total || (!workspace && plan.total > 0))
        return fail(FTWA_EINVAL, "workspace smaller than ftwa_evolve_workspace_size");
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = static_cast<char*>(workspace);
    if ((st = build_table(plan, inst, ws)) != FTWA_OK) return st;
    KernelTimer timer(tune && tune->kernel_ms);
    if ((st = execute(plan, inst, ws, stream, timer, true)) != FTWA_OK) return st;
    if (tune && tune->kernel_ms)
        if ((st = timer.finish(tune->kernel_ms, tune->kernel_launches, tune->kernel_work)) != FTWA_OK)
            return st;
    return FTWA_OK;
}

ftwa_status ftwa_evolve_check(const void* workspace, void* stream) {
    if (!workspace) {
        // the last ftwa_evolve_static run on the current device
        char* ptr = nullptr;
        ftwa_status st = static_scratch(&ptr);
        if (st != FTWA_OK) return st;
        return check_status(ptr, (hipStream_t)stream);
    }
    return check_status(static_cast<const char*>(workspace), (hipStream_t)stream);
}

ftwa_status ftwa_evolve_static(const ftwa_instance* inst, int n_inst, double dt, int64_t n_steps,
                               int record_every, ftwa_dtype dtype, const ftwa_tuning* tune,
                               void* stream_) {
    ftwa_status st = check_instances(inst, n_inst, true, "ftwa_evolve_static");
    if (st != FTWA_OK) return st;
    if (tune && tune->kernel_ms)
        return fail(FTWA_EINVAL, "ftwa_evolve_static: kernel timing is not available");
    Plan plan;
    PlanMode mode;
    mode.join = true;
    if ((st = plan_evolve(inst, n_inst, dt, n_steps, record_every, dtype, tune, &plan, mode)) !=
        FTWA_OK)
        return st;
    // the split kernel's mailboxes are larger than a few trajectories' stream
    // chunks, and groups have scratch of their own
    mode.compact = true;
    mode.join = false;
    if (plan.total > kStaticScratchBytes &&
        (st = plan_evolve(inst, n_inst, dt, n_steps, record_every, dtype, tune, &plan, mode)) !=
            FTWA_OK)
        return st;
    if (plan.total > kStaticScratchBytes)
        return fail(FTWA_EINVAL, "ftwa_evolve_static: this run needs " + std::to_string(plan.total) +
                                     " bytes of workspace, more than the static " +
                                     std::to_string(kStaticScratchBytes) +
                                     " (use ftwa_evolve with a workspace, or fewer trajectories "
                                     "per call)");
    char* ws = nullptr;
    if ((st = static_scratch(&ws)) != FTWA_OK) return st;
    if ((st = build_table(plan, inst, ws)) != FTWA_OK) return st;
    KernelTimer off(false);
    return execute(plan, inst, ws, (hipStream_t)stream_, off, true);
}

ftwa_status ftwa_evolve_graph(const ftwa_instance* inst, int n_inst, double dt, int64_t n_steps,
                              int record_every, ftwa_dtype dtype, const ftwa_tuning* tune,
                              void* workspace, size_t workspace_bytes, void* stream_,
                              ftwa_graph* out) {
    ftwa_status st = check_instances(inst, n_inst, true, "ftwa_evolve_graph");
    if (st != FTWA_OK) return st;
    if (!out) return fail(FTWA_EINVAL, "out is NULL");
    if (tune && tune->kernel_ms) return fail(FTWA_EINVAL, "kernel timing is not available in a graph");
    auto* g = new (std::nothrow) ftwa_graph_s;
    if (!g) return fail(FTWA_ENOMEM, "graph handle");
    if ((st = plan_evolve(inst, n_inst, dt, n_steps, record_every, dtype, tune, &g->plan)) != FTWA_OK) {
        delete g;
        return st;
    }
    if (workspace_bytes < g->plan.total || (!workspace && g->plan.total > 0)) {
        delete g;
        return fail(FTWA_EINVAL, "workspace smaller than ftwa_evolve_workspace_size");
    }
    g->inst.assign(inst, inst + n_inst);
    g->ws = static_cast<char*>(workspace);
    (void)stream_;
    if ((st = build_table(g->plan, inst, g->ws)) != FTWA_OK) {
        delete g;
        return st;
    }
    hipStream_t cs = nullptr;
    if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) {
        delete g;
        return fail(FTWA_EHIP, "hipStreamCreateWithFlags");
    }
    KernelTimer off(false);
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        st = execute(g->plan, g->inst.data(), g->ws, cs, off, false, true);
        hipError_t e2 = hipStreamEndCapture(cs, &g->graph);
        if (st == FTWA_OK && e2 != hipSuccess) st = hip_fail(e2, "hipStreamEndCapture");
    } else {
        st = hip_fail(e, "hipStreamBeginCapture");
    }
    (void)hipStreamDestroy(cs);
    if (st == FTWA_OK) {
        e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
        if (e != hipSuccess) st = hip_fail(e, "hipGraphInstantiate");
    }
    if (st != FTWA_OK) {
        if (g->graph) (void)hipGraphDestroy(g->graph);
        delete g;
        return st;
    }
    *out = g;
    return FTWA_OK;
}

ftwa_status ftwa_graph_launch(ftwa_graph g, void* stream) {
    if (!g || !g->exec) return fail(FTWA_EINVAL, "invalid graph");
    FTWA_HIP_TRY(hipGraphLaunch(g->exec, (hipStream_t)stream));
    return FTWA_OK;
}

ftwa_status ftwa_graph_check(ftwa_graph g, void* stream) {
    if (!g) return fail(FTWA_EINVAL, "invalid graph");
    return check_status(g->ws, (hipStream_t)stream);
}

void ftwa_graph_free(ftwa_graph g) {
    if (!g) return;
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    delete g;
}

}  // extern "C"

// ---------------------------------------------------------------- autotuner
namespace ftwa {
namespace {

constexpr int kProbeReps = 3;

// The untuned automatic plan as a candidate: where it is a pack of the
// shared-pack kernel, whose size follows the ensemble and the Hamiltonian.
// Where it is the fastest, later plans choose their packs by the rules again;
// the best of the others serves the runs that have none.
constexpr int kAutomatic = -2;

struct Probe {
    std::vector<int> cands;  // resident configurations that fit (no packs), the automatic
                             // plan if it is a pack, then -1 (stream path)
    int pack = -1;           // the automatic plan's configuration, if it is a pack
    int64_t Mp = 0;          // trajectories timed
    size_t off_rho = 0, off_s1 = 0, off_s2 = 0, off_ws = 0, total = 0;
};

ftwa_tuning probe_tuning(int cand) {
    ftwa_tuning t;
    std::memset(&t, 0, sizeof(t));
    t.path = cand == kAutomatic ? FTWA_PATH_AUTO : cand < 0 ? FTWA_PATH_STREAM
                                                            : FTWA_PATH_RESIDENT;
    t.traj_chunk = 0;
    t.resident_config = std::max(cand, -1);
    return t;
}

ftwa_status plan_candidate(const ftwa_instance& q, ftwa_dtype dtype, int probe_steps, int cand,
                           Plan* out) {
    const ftwa_tuning t = probe_tuning(cand);
    PlanMode mode;
    mode.untuned = true;
    return plan_evolve(&q, 1, 0.01, probe_steps, probe_steps, dtype, &t, out, mode);
}

ftwa_instance probe_instance(const ftwa_instance& in, int64_t Mp, char* ws, const Probe& pr) {
    ftwa_instance q = in;
    q.n_traj = Mp;
    q.traj_offset = 0;
    q.rho = ws ? ws + pr.off_rho : nullptr;
    q.S1 = ws ? reinterpret_cast<double*>(ws + pr.off_s1) : nullptr;
    q.S2 = ws ? reinterpret_cast<double*>(ws + pr.off_s2) : nullptr;
    q.inv = nullptr;
    q.v_site = nullptr;  // the probes time the kernels without the potential term
    q.v_env = nullptr;
    q.u_mat = nullptr;   // and with the on-site interaction
    q.hop_w = nullptr;   // and real hopping
    return q;
}

ftwa_status plan_probe(const ftwa_instance& in, ftwa_dtype dtype, int probe_steps, Probe* out) {
    Probe pr;
    ftwa_status st;
    const DeviceTables& tab = host_tables(in.lat);
    const int N = in.lat->N;
    int64_t want = 0;
    for (int c = 0; c < resident_config_count(); ++c) {
        ResidentPlan rp;
        if (resident_is_shared(c) || !resident_plan(N, dtype, tab, &rp, c)) continue;
        pr.cands.push_back(c);
        want = std::max(want, 2 * resident_concurrency(c, rp.lds, rp.threads, rp.units, rp.variant));
    }
    {
        Plan p;
        const ftwa_instance q = probe_instance(in, std::max<int64_t>(in.n_traj, 1), nullptr, pr);
        if ((st = plan_candidate(q, dtype, probe_steps, kAutomatic, &p)) != FTWA_OK) return st;
        const ResidentPlan& rp = p.inst[0].res;
        if (p.inst[0].path == FTWA_PATH_RESIDENT && resident_is_shared(rp.config)) {
            pr.cands.push_back(kAutomatic);
            pr.pack = rp.config;
            want = std::max(want, 2 * resident_concurrency(rp.config, rp.lds, rp.threads, rp.units,
                                                           rp.variant));
        }
    }
    pr.cands.push_back(-1);
    if (want == 0) want = kStreamChunk;
    pr.Mp = std::max<int64_t>(1, std::min(in.n_traj, want));
    const int D = 2 * N;
    size_t off = 0;
    pr.off_rho = off; off = align_up(off + (size_t)2 * packed_count(N) * pr.Mp * cplx_bytes(dtype));
    pr.off_s1 = off;  off = align_up(off + (size_t)2 * D * sizeof(double));
    pr.off_s2 = off;  off = align_up(off + (size_t)2 * s2_count(D) * sizeof(double));
    pr.off_ws = off;
    size_t ews = 0;
    const ftwa_instance q = probe_instance(in, pr.Mp, nullptr, pr);
    for (int c : pr.cands) {
        Plan p;
        if ((st = plan_candidate(q, dtype, probe_steps, c, &p)) != FTWA_OK) return st;
        ews = std::max(ews, p.total);
    }
    pr.total = align_up(off + ews);
    *out = pr;
    return FTWA_OK;
}

}  // namespace
}  // namespace ftwa

extern "C" {

ftwa_status ftwa_autotune_workspace_size(const ftwa_instance* inst, int n_inst, ftwa_dtype dtype,
                                         int probe_steps, size_t* bytes) {
    ftwa_status st = check_instances(inst, n_inst, false, "ftwa_autotune_workspace_size");
    if (st != FTWA_OK) return st;
    if (!bytes || probe_steps < 1) return fail(FTWA_EINVAL, "bytes is NULL or probe_steps < 1");
    if (dtype != FTWA_F64 && dtype != FTWA_F32) return fail(FTWA_EINVAL, "unknown dtype");
    size_t total = 0;
    for (int k = 0; k < n_inst; ++k) {
        Probe pr;
        if ((st = plan_probe(inst[k], dtype, probe_steps, &pr)) != FTWA_OK) return st;
        total = std::max(total, pr.total);
    }
    *bytes = total;
    return FTWA_OK;
}

ftwa_status ftwa_autotune(const ftwa_instance* inst, int n_inst, ftwa_dtype dtype, int probe_steps,
                          void* workspace, size_t workspace_bytes, void* stream_, int* configs) {
    ftwa_status st = check_instances(inst, n_inst, false, "ftwa_autotune");
    if (st != FTWA_OK) return st;
    if (probe_steps < 1) return fail(FTWA_EINVAL, "probe_steps < 1");
    if (dtype != FTWA_F64 && dtype != FTWA_F32) return fail(FTWA_EINVAL, "unknown dtype");
    hipStream_t stream = (hipStream_t)stream_;
    char* ws = static_cast<char*>(workspace);
    std::map<std::pair<int, int64_t>, int> decided;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    FTWA_HIP_TRY(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail(FTWA_EHIP, "hipEventCreate");
    }
    auto done = [&](ftwa_status s) {
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        return s;
    };
    for (int k = 0; k < n_inst; ++k) {
        const ftwa_instance& in = inst[k];
        if (in.n_traj < 1 || !in.rho || !in.n0) return done(fail(FTWA_EINVAL, "instance without trajectories"));
        DeviceTables tab;
        if ((st = device_tables(in.lat, &tab)) != FTWA_OK) return done(st);
        const int N = in.lat->N;
        const auto key = std::make_pair(N, class_shape(tab));
        auto it = decided.find(key);
        if (it != decided.end()) {
            if (configs) configs[k] = it->second;
            continue;
        }
        Probe pr;
        if ((st = plan_probe(in, dtype, probe_steps, &pr)) != FTWA_OK) return done(st);
        if (!ws || workspace_bytes < pr.total)
            return done(fail(FTWA_EINVAL, "workspace smaller than ftwa_autotune_workspace_size"));
        const ftwa_instance q = probe_instance(in, pr.Mp, ws, pr);
        const size_t cb = cplx_bytes(dtype);
        const size_t P2 = (size_t)2 * packed_count(N);
        Tuned best;
        double best_ms = -1.0, pack_ms = -1.0;
        for (int c : pr.cands) {
            Plan p;
            if ((st = plan_candidate(q, dtype, probe_steps, c, &p)) != FTWA_OK) return done(st);
            char* ews = ws + pr.off_ws;
            if ((st = build_table(p, &q, ews)) != FTWA_OK) return done(st);
            // one warm-up run, then the fastest of kProbeReps timed runs
            float ms = -1.0f;
            for (int rep = 0; rep <= kProbeReps; ++rep) {
                FTWA_HIP_TRY(hipMemcpy2DAsync(ws + pr.off_rho, pr.Mp * cb, in.rho, in.n_traj * cb,
                                              pr.Mp * cb, P2, hipMemcpyDeviceToDevice, stream));
                KernelTimer off(false);
                FTWA_HIP_TRY(hipEventRecord(e0, stream));
                if ((st = execute(p, &q, ews, stream, off, true)) != FTWA_OK) return done(st);
                FTWA_HIP_TRY(hipEventRecord(e1, stream));
                FTWA_HIP_TRY(hipEventSynchronize(e1));
                float t = 0.0f;
                FTWA_HIP_TRY(hipEventElapsedTime(&t, e0, e1));
                if (rep > 0 && (ms < 0 || t < ms)) ms = t;
            }
            if ((st = check_status(ews, stream)) != FTWA_OK) return done(st);
            if (c == kAutomatic) {
                pack_ms = ms;
            } else if (best_ms < 0 || ms < best_ms) {
                best_ms = ms;
                best.config = c;
            }
        }
        best.packs = pack_ms >= 0 && pack_ms <= best_ms;
        best.n_traj = in.n_traj;
        set_tuned_config(N, class_shape(tab), dtype, best);
        decided[key] = best.packs ? pr.pack : best.config;
        if (configs) configs[k] = decided[key];
    }
    return done(FTWA_OK);
}

}  // extern "C"
