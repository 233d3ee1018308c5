// resident_config.h -- what the resident kernels and their host code share:
// the kernel arguments, the description of a kernel configuration, and the
// configuration tables of the files that instantiate the kernels.
#pragma once

#include "ftwa_internal.h"

namespace ftwa {

struct ResidentArgs {
    const ResidentInst* table;  // entries (instance windows), item0 ascending
    int n_entries;
    int64_t n_items;            // total items over the table
    double dt;
    int64_t n_steps;
    int record_every;
    uint64_t* mailbox;          // S = 1: [pairs][2 spins][2 slots][Nmax] stage-stamped words
    int Nmax;
    uint32_t tail_off;          // LDS byte offset of the record sums and the abort flag
    int* error;                 // set to 1 when a wait times out
    unsigned spin_limit;        // polls before a bounded wait gives up
    int far;                    // split kernel, nonzero: exchange as across XCDs
};

constexpr unsigned kSpinLimit = 1u << 26;  // default: ~2 s of polling
constexpr int kSplitPlanePad = 8;  // spare words at the end of a split part's published planes
constexpr int kSplitSyncWords = 80;  // words of a split group for its flags and its members' XCDs
constexpr unsigned kSplitSpinLimit = 6u << 20;  // default: ~2 s at the sleeps between looks

// Places whose complex-hopping ratios (three FP32 complex numbers, 24 bytes)
// a stage keeps in LDS: the most that fit beside a 198-site spin block (its
// elements, the two diagonal copies and the record sums leave 3,712 bytes of
// the 160 KB); the table's later places are read from global memory.
constexpr int kHopLds = 152;

// GE, GO: the leading even and odd slots that take the general path (the
// elements that read a transpose must fit in them).
// fn_t1: the variant for launches whose instances all have t = 1 (FP32).
struct Config {
    ftwa_dtype dtype;
    int S, NTU, UNITS, UE, UO, GE, GO;
    const void* fn;
    const void* fn_t1;
    // split kernel (G > 1 workgroups per spin block): GE = GE1; boundary
    // from slot UB, its first GE2 slots read transposes; exported odd
    // elements in the first XO odd slots; KB halo reads issued ahead
    int G = 1;
    int UB = 0, GE2 = 0, XO = 0, KB = 0;
    bool auto_pick = true;  // false: chosen only when forced or by the autotuner
    // variants (the FP32 spin split and the FP64 split kernel; _t1: the same
    // for launches with t = 1, FP32 only): external potential, complex
    // hopping, general interaction
    const void* fn_pot = nullptr;
    const void* fn_pot_t1 = nullptr;
    const void* fn_hop = nullptr;
    const void* fn_hop_t1 = nullptr;
    const void* fn_gint = nullptr;
    const void* fn_gint_t1 = nullptr;
};

// The configurations by the file that instantiates them (their order in the
// public configuration index: evolve_resident.hip).
extern const Config kConfigsF64Shared[];  // resident_f64_shared.hip
extern const Config kConfigsF32Shared[];  // resident_f32_shared.hip
extern const Config kConfigsF32Spin[];    // resident_f32_spin.hip
extern const Config kConfigsF64Split[];   // resident_f64_split.hip

}  // namespace ftwa
