// Group kernels: one work-group updates 16 elements, in FP64 or FP32.
//
// The matrix-core kernels of tuned_kern.hpp give a wavefront 16 elements and
// keep their state in its registers, which suits large ranges in 32 bits. A
// work-group of several wavefronts per 16 elements, with the state in LDS and
// the output tiles of every contraction shared out among the wavefronts, has
// room for FP64 (the matrix cores' v_mfma_f64_16x16x4), and finishes a small
// range in a fraction of the time. It is the FP64 form of the tuned kernels
// at orders 3..6 (the rows of order 7 exceed LDS) and the form of FP32 ranges
// below options.mc_min elements (orders 3..7); the smallest ranges of both take
// the plain kernels (launch_form in tuned.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <vector>

#include "device.hpp"
#include "model.hpp"

namespace seis {

template <typename T>
struct GroupArgs {
  T* Q;
  T* In;
  const T* G;
  const T* mat;
  const T* RCm;          // [E][4][12] own-trace flux coefficients
  const T* RCp;          // [E][4][12] neighbour-trace flux coefficients
  T* H2;                 // [n_half2][Bf][9] second-half traces
  T* gD;                 // stored time derivatives
  T* Ih;                 // [slot] tiled: half-step integrals of the 16-element groups with a finer neighbour
  const T* img;          // reference matrices in fragment order (group_image)
  const T* Et;           // [4][B][Bf] trace matrices, node-contiguous
  const int32_t* tgt;    // [E][4]
  const int32_t* mh4;    // [E]: byte f = mode | hperm << 2 of face f
  const int32_t* pinv;   // [6][Bf]
  const int32_t* half2;  // [E][4] writer: second-half slot, -1 none
  const int32_t* rhalf2; // [E][4] reader: second-half slot, -1 none
  const int32_t* dslot;  // [E] slot of the stored time derivatives, -1 none
  const int32_t* hslot;  // [groups] slot in Ih, -1 none
  const int32_t* fix_list;   // element * 4 + face of the faces handing over to a finer neighbour
  const int32_t* fix_group;  // [n][3] (group, first entry of fix_list, entries), by cluster
};

// degrees the group kernels are compiled for
template <typename T>
constexpr bool group_order(int N) {
  return N >= 2 && N <= (sizeof(T) == 8 ? 5 : 6);
}

// reference matrices in the fragment order of the FP64 or FP32 products
std::vector<double> group_image(const Model& M, bool fp64);

template <typename T>
hipError_t launch_predict_group(int N, const GroupArgs<T>& a, int64_t e0, int64_t e1, const Sched& sc,
                                hipStream_t s);
template <typename T>
hipError_t launch_correct_group(int N, const GroupArgs<T>& a, int64_t e0, int64_t e1, const Sched& sc,
                                hipStream_t s);
// Half-step traces of n entries of fix_group (after the predictor): the finer
// neighbour gets the first half in its inbox and the second in its slot.
template <typename T>
hipError_t launch_finer(int N, const GroupArgs<T>& a, int64_t first, int64_t n, hipStream_t s);

}  // namespace seis
