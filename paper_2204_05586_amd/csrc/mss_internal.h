// Internal interface between the C-ABI layer (mss_api.hip) and the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <string>

#include "mss_device.h"

namespace mss {

// Scan tiling: one wave owns kScanTile consecutive matrices, each lane a
// run of kScanPerLane of them.
constexpr int kScanPerLane = 4;
constexpr int kScanTile = 64 * kScanPerLane;
// Largest level-1 tile count whose upper two levels run in one workgroup
// (scan_top_kernel, one wave per tile).  Eight waves leave each lane 256
// VGPRs (no spills); at sixteen the kernel spilled and the separate
// launches of the general path were faster.
constexpr int kTopWaves = 8;
// Largest tile count that is scanned whole in one workgroup
// (scan_small_kernel): one wave per SIMD of a CU.  With eight waves two share
// a SIMD and its registers (spin-1 spills) and wave 0's run over the totals
// grows: 10.4 us against 9.3 of the two launches at 2048 spin-1/2 operators,
// 21.5 against 15.2 at 2048 spin-1 ones; at four tiles 7.1 against 9.0 and
// 11.1 against 14.1.
constexpr int kSmallWaves = 4;

struct IntegrateArgs {
  FieldProgram fp;
  IntervalGrid g;
};

// host helpers shared by the C-ABI translation units (mss_api.hip)
mss_status api_fail(mss_status s, const char* fmt, ...);
mss_status api_fail_text(mss_status s, const std::string& msg);
mss_status api_ok();
mss_status api_hip_fail(hipError_t e, const char* what);
std::string api_last_error_copy();
mss_status api_validate_problem(const mss_problem* p);
// a spin-1 problem with a term on U_1, U_2, V_1 or V_2 (the full su(3) basis)
bool api_full_basis(const mss_problem* p);
// the term checks of api_validate_problem for a term list on its own
mss_status api_validate_terms(int spin_twice, const mss_term* terms, int n_terms, int n_params);
// a problem run with a sampler: its parameter vector covers what the
// sampler reads, and its spin suits the sampler's components
mss_status api_sampler_check_problem(mss_sampler s, const mss_problem* p);
int api_device_cu_count();
// lane-slices of a work set's items
int api_plan_slices(int64_t K, int32_t L, int cu);
int api_ilog2(int x);
// launch shape (lane-slices per interval, block size) of one simulation
mss_status api_resolve_launch(const mss_problem* p, const mss_launch* in, int* slices, int* block);
// Whether b, the term after a, takes the same phase 2 pi f t + phi at every
// time at which either is on, and the same segments: a circular drive's
// cosine and sine, evaluated once then.
bool same_phase(const mss_term& a, const mss_term& b);
// A term list in the order the interpreter walks it, into out[0 .. n): first
// the terms of components that depend on time (list order), then those of
// components all of whose terms are constant and always on, whose field is
// formed once per interval.  Components are summed apart, each in list
// order, so the field is the list's bit for bit.  Returns the count of the
// first kind.
int program_order(const mss_term* terms, int n, mss_term* out);
// work-queue integrator of a user sampler's module on the current device
// (loads the module there on first use); chained: the form that also forms
// the states (launch_work_chained)
mss_status api_sampler_work_function(mss_sampler s, hipFunction_t* fn, bool chained = false);
// True when s was generated by mss_sampler_create_for_terms from exactly
// these terms (compared byte for byte).
bool api_sampler_is_for_terms(mss_sampler s, const mss_term* terms, int32_t n_terms);

// mss_propagate (without <J>) on a caller-given workspace; api_ok() on success
mss_status api_propagate(int32_t spin_twice, int64_t n_samples, const double* U,
                         const double* psi0, double* psi, double* psi_final, void* ws,
                         size_t ws_bytes, void* stream);

hipError_t launch_integrate(int N, const IntegrateArgs& a, int block, hipStream_t st);
hipError_t launch_scan_reduce(int N, const double* M, int64_t n, double* agg, hipStream_t st);
hipError_t launch_scan_apply(int N, const double* M, int64_t n, const double* start, double* before,
                             double* after_last, hipStream_t st, double* spin = nullptr);

// levels 1 and 2 of a two-level single-sequence scan in one workgroup
// (n1 level-1 elements in at most kTopWaves tiles)
// level 0 of a one-level scan with the top level folded in (n1 = the level-0
// tile count, at most kScanTile)
hipError_t launch_scan_apply_fold(int N, const double* M, int64_t n, const double* A1, int64_t n1,
                                  const double* start, double* before, double* after_last,
                                  hipStream_t st, double* spin);
// a whole scan of at most kSmallWaves tiles
hipError_t launch_scan_small(int N, const double* M, int64_t n, const double* start,
                             double* before, double* after_last, hipStream_t st, double* spin);
hipError_t launch_scan_top(int N, const double* M1, int64_t n1, const double* start,
                           double* before1, hipStream_t st);

hipError_t launch_spin_projection(int N, const double* psi, int64_t K, double* out,
                                  hipStream_t st);

}  // namespace mss
