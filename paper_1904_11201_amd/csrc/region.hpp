// region.hpp -- theta join over sorted sides (the paper's region pruning, taken to single rows).
#pragma once
#include "common.hpp"

namespace jl {

struct RegionPlan {
    int direct;                  // 1: both sides fit one workgroup's LDS sort, no partitioning
    int bits, B;                 // B = 2^bits value buckets shared by both sides (direct: 1)
    int binBits;                 // 2^binBits value bins, from which the buckets are made
    int64_t samples;             // rows sampled per side for the bins
    int64_t rows;                // R rows per unit
    int64_t U;                   // units: R blocks x Y
    int Y, tiled;                // shares of an R block's work, a power of two; 1: they are S tiles
    size_t off_zero, zero_words; // cleared first: bucket sizes, arrivals, counters
    size_t off_base, off_cur, off_extra, off_lut, off_split, off_sample, off_id;
    size_t off_pR, off_pS;       // bucketed rows
    size_t off_Ra, off_Rc, off_Rr, off_Sa, off_Sc, off_Sr;  // sorted columns
    size_t off_lo, off_hi;       // each R row's interval of sorted S rows
    size_t off_counts, off_wave, off_dbg, bytes;
    uint64_t stamp;              // signature of the fields above (plan_stamp)
};

// op_a JOIN_OP_NONE: unknown, sized for the largest layout.  knob: the theta.stash setting, which
// changes nothing here but is part of the plan's signature, so that changing it between the two
// passes is refused as it is for the nested loop.
RegionPlan region_plan(int64_t nR, int64_t nS, int op_a, int op_c, int num_cus, int64_t knob);

// Buckets, partition, sort, intervals, count pass and the scan of all counts.  Leaves the exact
// total at ws[0..8).
hipError_t region_count(const RegionPlan& pl, const join_rel_t& R, const join_rel_t& S,
                        const join_pred_t& p, char* ws, hipStream_t st, uint64_t* pub = nullptr);

// Write pass from the state region_count left in ws.
hipError_t region_write(const RegionPlan& pl, const join_rel_t& R, const join_rel_t& S,
                        const join_pred_t& p, char* ws, int32_t* pairs, uint64_t cap,
                        hipStream_t st);

}  // namespace jl
