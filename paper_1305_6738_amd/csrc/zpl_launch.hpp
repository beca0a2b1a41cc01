// zpl_launch.hpp -- host launchers of the kernels in zpl_kernels.hip.
#pragma once

#include <hip/hip_runtime.h>

#include "zpl_kernels.hpp"

namespace zpl {

// The context's constants: ln k for k = 0..kH+1 (doubles), ln k 2^53 as
// integers (uint64), then the MLE's start table (2 kGuessN doubles).
hipError_t launch_ln_table(double* ln, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, int n, uint32_t v, hipStream_t s);
// CDF tables (the truncated law's only when any_trunc: a cell with K > 0)
// and packed guides; the first table block also zeroes zero[0..n_zero).
hipError_t launch_tables(DevCell* cells, int n_cells, double* tables, uint16_t* guides,
                         const double* ln, hipStream_t s, bool any_trunc = true,
                         uint32_t* zero = nullptr, int n_zero = 0);
// Lane-form units and wave- and heavy-form ones in one launch; scratch: the lane
// form's slots (kLaneScratch int64 a wave) and the other waves' areas, as SimGrid
// places them.
hipError_t launch_simulate(const SimGrid& g, const DevCell* cells, const double* tables,
                           const uint16_t* guides, const double* ln, const Unit* lane_units,
                           int n_lane, const Unit* batch_units, int n_batch, uint32_t* lane_queue,
                           uint32_t* batch_queue, uint32_t* big_queue, Outputs out,
                           uint64_t* esc_list, uint32_t* esc_count, uint32_t esc_cap,
                           int64_t* scratch, uint32_t* err, hipStream_t s);
// The escalated replicates; scratch: grid * waves areas (waves <= kEscWaves) of `stride`
// int64, each for a replicate's every draw.  Grid 0 (no replicate can escalate): no launch.
hipError_t launch_escalated(int grid, const DevCell* cells, const double* tables,
                            const uint16_t* guides, const double* ln, uint32_t* queue, Outputs out,
                            uint64_t* esc_list, uint32_t* esc_count, uint32_t esc_cap,
                            int64_t* scratch, int waves, int64_t stride, uint32_t* err,
                            hipStream_t s);
// The units of cells with a lower cutoff, `waves` waves of each workgroup at
// work; scratch: grid * waves areas of `stride` int64.
hipError_t launch_cutoff(int grid, const DevCell* cells, const double* tables,
                         const uint16_t* guides, const double* ln, const Unit* units, int n_units,
                         uint32_t* queue, Outputs out, uint64_t* esc_list, uint32_t* esc_count,
                         uint32_t esc_cap, int64_t* scratch, int waves, int64_t stride,
                         uint32_t* err, hipStream_t s);
// Datasets of a batch, a workgroup each; scratch: grid areas of `stride` int64
// (heavy_stride of the largest).
hipError_t launch_fit(int grid, const int64_t* const* xs, const int64_t* ns, int n_sets,
                      const double* ln, int64_t* scratch, int64_t stride, double* ahat,
                      double* D, uint32_t* flags, uint32_t* status, hipStream_t s);
// One dataset (the truncated law on 1..K, or K = 0), or its fits with each of
// n_cand lower cutoffs; scratch: heavy_stride(n) int64.
hipError_t launch_fit_one(const int64_t* x, int64_t n, const double* ln, int64_t* scratch,
                          double* ahat, double* D, uint32_t* flags, uint32_t* status, uint32_t K,
                          hipStream_t s);
hipError_t launch_fit_scan(const int64_t* x, int64_t n, const int64_t* xmins, int n_cand,
                           const double* ln, int64_t* scratch, double* ahat, double* D,
                           int64_t* ntail, uint32_t* flags, uint32_t* status, hipStream_t s);
// Device address of the fixed scratch array of the allocation-free fit
// (kNoAllocStride int64) on the current device.
hipError_t noalloc_scratch_address(int64_t** p);
// gather: n_cells * kSelQ * gcap values, then n_cells * kSelQ * 32 bytes of
// per-(cell, quantile) state; maxR bounds every cell's R.
hipError_t launch_select(const double* D, const DevCell* cells, int n_cells, int n_q,
                         const uint32_t* qnum, const uint32_t* qden, double* qout,
                         uint64_t* gather, int64_t gcap, int64_t maxR, int n_cu, hipStream_t s);
hipError_t launch_count_ge(const double* Db, int64_t B, const double* Dobs,
                           unsigned long long* count, hipStream_t s);
hipError_t launch_count_cells(const double* D, const DevCell* cells, int n_cells,
                              const double* dobs, unsigned long long* counts, int64_t maxR,
                              hipStream_t s);
hipError_t launch_draws(const DevCell* cell, const double* table, const uint16_t* guide,
                        int64_t rep_lo, int64_t count, int64_t* x, uint32_t* flags,
                        int64_t total, hipStream_t s);

}  // namespace zpl
