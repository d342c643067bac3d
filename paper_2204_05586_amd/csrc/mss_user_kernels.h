// Integrator kernels around a user-supplied field function.  This header is
// compiled at run time (hiprtc) by the sampler entry points, after the
// user's source, which defines
//
//   __device__ void mss_user_field(double t, const double* params, double* field);
//
// field arrives zeroed and receives f_x, f_y, f_z, f_q in Hz at time t (s);
// params is the simulation's parameter vector.  This is the counterpart of
// the paper's field function compiled into its integrator (Sec.
// "Compilation of integrator"): the user's code is inlined into the same
// interval operator as the field-program interpreter.
#pragma once

#include "mss_device.h"
#include "mss_work_device.h"

#ifndef MSS_TERMS_FIELD
__device__ void mss_user_field(double t, const double* params, double* field);
#endif

struct MssUserField {};

// Found by argument-dependent lookup from the interval operator's templates.
// Nothing is set apart as constant: the compiler moves what does not depend
// on time out of the loops by itself.
template <int C>
__device__ __forceinline__ void field_constant(const MssUserField&, const double* __restrict__,
                                               double (&fc)[C]) {
#pragma unroll
  for (int j = 0; j < C; ++j) fc[j] = 0.0;
}

// The field at M times: a generated program takes them all at once, a
// user's function is called for each.
template <int C, int M>
__device__ __forceinline__ void field_at(const MssUserField&, const double* __restrict__ params,
                                         const double (&)[C], const double (&t)[M],
                                         double (&f)[M][C], int = -1) {
#ifdef MSS_TERMS_FIELD
  mss_terms_field(t, params, f);
#else
#pragma unroll
  for (int i = 0; i < M; ++i) {
    f[i][0] = 0.0;
    f[i][1] = 0.0;
    f[i][2] = 0.0;
    f[i][3] = 0.0;
    mss_user_field(t[i], params, f[i]);
  }
#endif
}

// Two waves to a SIMD, 256 registers each, unless MSS_USER_ALL_REGISTERS says
// that the field function leaves too much in scratch memory that way
// (mss_sampler_create): then one wave with all 512.
#ifdef MSS_USER_ALL_REGISTERS
#define MSS_USER_BOUNDS __launch_bounds__(256)
#else
#define MSS_USER_BOUNDS __launch_bounds__(256, 2)
#endif

extern "C" __global__ void MSS_USER_BOUNDS mss_user_integrate_2(const mss::IntervalGrid g) {
  mss::integrate_lanes<2>(MssUserField{}, g);
}

extern "C" __global__ void MSS_USER_BOUNDS mss_user_integrate_3(const mss::IntervalGrid g) {
  mss::integrate_lanes<3>(MssUserField{}, g);
}

// Every descriptor of a batch takes its field from the user function.
struct MssUserSource {
  __device__ __forceinline__ MssUserField operator()(const mss::IntegrateWorkArgs&,
                                                     const mss::SimDesc&) const {
    return MssUserField{};
  }
};

extern "C" __global__ void MSS_USER_BOUNDS mss_user_work_integrate(
    const mss::IntegrateWorkArgs A) {
  mss::work_integrate_loop(A, MssUserSource{});
}

extern "C" __global__ void __launch_bounds__(256, 2) mss_user_work_chained(
    const mss::IntegrateWorkArgs A) {
  mss::chained_integrate_loop(A, MssUserSource{});
}
