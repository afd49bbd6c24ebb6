// Host side of the matrix-core kernels: reference-matrix images, set-up,
// per-cluster launches (with the LTS half-step fix-ups) and the autotuner.
// The kernels are in tuned_kern.hpp and are instantiated per operand
// precision in tuned_f32.hip and tuned_bf16.hip.
#include "tuned_kern.hpp"

#include <sys/stat.h>

#include <fstream>
#include <sstream>

namespace seis {

namespace {

// Half-step fix-up of the faces handing over to a finer neighbour: the
// predictor wrote the full-step trace V; the finer neighbour needs the traces of
// the first and of the second half of this element's step, each over its own
// step: the first half h1 = E_f I~_h with I~_h = sum_k D~k 2^-k / (k+1) (from the
// stored derivatives) goes to the inbox, the second half 2 V - h1 to its slot.
// kFixElems elements share a work-group and its copy of the trace matrices; a
// wavefront forms the I~_h of whole elements (the non-zero rows of the
// derivatives, B_{N-k} of derivative k, requested together), then a thread sums
// all nine quantities of a node (one value of E_f and three wide broadcasts of
// I~_h per mode), V requested before. Bound by the memory traffic of the
// derivatives and the two traces, and the latency of their addresses.
// 248 832 elements at order 6 with four clusters (87 506 such faces): a pass of
// two macro steps took 12.15 ms with a work-group of one wavefront per face, which
// read all N + 1 full derivatives and its own copy of E_f, and 11.97 in this form.
constexpr int kFixElems = 4, kFixThreads = 256;

template <int N>
__global__ __launch_bounds__(kFixThreads) void k_finer_fixup(TArgs a, const float* Et, const int32_t* runs, int64_t n) {
  constexpr int B = nbasis(N), Bf = nface(N), FT = row_tiles(Bf), P = 12;  // P: a row of nine in three padded triples
  __shared__ __align__(16) float sE[4 * B * Bf], sIh[kFixElems][B * P];
  __shared__ int sOwner[4 * kFixElems], sId[4 * kFixElems], sSlot[kFixElems];
  const int64_t r0 = xcd_block() * kFixElems;
  const int ne = n - r0 < kFixElems ? int(n - r0) : kFixElems, tid = threadIdx.x;
  // faces of the elements: consecutive entries of the list
  const int f0 = runs[2 * r0], nf = runs[2 * (r0 + ne)] - f0;
  if (tid < ne) {
    sSlot[tid] = runs[2 * (r0 + tid) + 1];
    for (int u = runs[2 * (r0 + tid)] - f0; u < runs[2 * (r0 + tid + 1)] - f0; ++u) sOwner[u] = tid;
  }
  if (tid < nf) sId[tid] = a.fix_list[f0 + tid];
  for (int i = tid; i < 4 * B * Bf / 4; i += kFixThreads)
    reinterpret_cast<f4*>(sE)[i] = reinterpret_cast<const f4*>(Et)[i];
  __syncthreads();
  for (int r = tid >> 6; r < ne; r += kFixThreads / 64) {
    const float* D = a.gD + (int64_t)sSlot[r] * (N + 1) * B * 9;
#pragma unroll 4
    for (int j = tid & 63; j < B * 9; j += 64) {
      const int row = j / 9, q = j - row * 9;
      float d[N + 1], acc = 0.0f, w = 1.0f;
#pragma unroll
      for (int k = 0; k <= N; ++k) d[k] = row < nbasis(N - k) ? D[k * B * 9 + j] : 0.0f;
#pragma unroll
      for (int k = 0; k <= N; ++k) {
        acc = __builtin_fmaf(w / float(k + 1), d[k], acc);
        w *= 0.5f;
      }
      sIh[r][row * P + q / 3 * 4 + q % 3] = acc;
    }
  }
  __syncthreads();
  for (int i = tid; i < nf * Bf; i += kFixThreads) {
    const int u = i / Bf, m = i - u * Bf, id = sId[u], f = id & 3;
    const int32_t tg = a.tgt[id];
    const int mr = a.pinv[a.hperm[id] * Bf + m];
    float* out = a.H2 + ((int64_t)a.half2[id] * Bf + mr) * 9;
    float* blk = a.In + in_block(tg >> 2, tg & 3, mr, FT) * 576;
    const int l8 = in_lane(tg >> 2, mr);
    f4* in = reinterpret_cast<f4*>(blk + 8 * l8);
    const f4 v0 = in[0], v1 = in[1];
    const float v8 = blk[512 + l8];
    const float* E = sE + f * B * Bf + m;
    const f4* I = reinterpret_cast<const f4*>(sIh[sOwner[u]]);
    float h[9] = {};
#pragma unroll 4
    for (int l = 0; l < B; ++l) {
      const float x = E[l * Bf];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const f4 y = I[l * 3 + t];
#pragma unroll
        for (int j = 0; j < 3; ++j) h[t * 3 + j] = __builtin_fmaf(x, y[j], h[t * 3 + j]);
      }
    }
    in[0] = f4{h[0], h[1], h[2], h[3]};
    in[1] = f4{h[4], h[5], h[6], h[7]};
    blk[512 + l8] = h[8];
#pragma unroll
    for (int p = 0; p < 9; ++p) out[p] = 2.0f * (p < 4 ? v0[p & 3] : (p < 8 ? v1[p & 3] : v8)) - h[p];
  }
}

// Second-half traces into the inbox before the corrector of an odd sub-step
// (one work-group per face of list).
template <int N>
__global__ __launch_bounds__(64) void k_h2_to_in(TArgs a, const int32_t* list) {
  constexpr int Bf = nface(N), FT = row_tiles(Bf);
  const int id = list[xcd_block()];
  const int64_t e = id >> 2;
  const int f = id & 3;
  const int slot = a.rhalf2[e * 4 + f];
  for (int i = threadIdx.x; i < Bf * 9; i += 64) {
    const int m = i / 9, p = i % 9;
    a.In[inidx(e, f, m, p, FT)] = a.H2[((int64_t)slot * Bf + m) * 9 + p];
  }
}

template <int N>
hipError_t launch_fixup(const TunedData& t, int64_t first, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_finer_fixup<N>, dim3((unsigned)((n + kFixElems - 1) / kFixElems)), dim3(kFixThreads), 0, s, t.a,
                     t.d32.Et, t.fix_elem + 2 * first, n);
  return hipGetLastError();
}

template <int N>
hipError_t launch_h2(const TArgs& a, const int32_t* list, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_h2_to_in<N>, dim3((unsigned)n), dim3(64), 0, s, a, list);
  return hipGetLastError();
}

// elements [first, first + n) of fix_elem
hipError_t fixup_dispatch(int N, const TunedData& t, int64_t first, int64_t n, hipStream_t s) {
  switch (N) {
    case 2: return launch_fixup<2>(t, first, n, s);
    case 3: return launch_fixup<3>(t, first, n, s);
    case 4: return launch_fixup<4>(t, first, n, s);
    case 5: return launch_fixup<5>(t, first, n, s);
    case 6: return launch_fixup<6>(t, first, n, s);
  }
  return hipErrorInvalidValue;
}

hipError_t h2_dispatch(int N, const TArgs& a, const int32_t* list, int64_t n, hipStream_t s) {
  switch (N) {
    case 2: return launch_h2<2>(a, list, n, s);
    case 3: return launch_h2<3>(a, list, n, s);
    case 4: return launch_h2<4>(a, list, n, s);
    case 5: return launch_h2<5>(a, list, n, s);
    case 6: return launch_h2<6>(a, list, n, s);
  }
  return hipErrorInvalidValue;
}

template <typename X, typename Y>
hipError_t upload(std::vector<void*>& owned, int64_t& bytes, X** dst, const std::vector<Y>& src) {
  void* p = nullptr;
  const size_t n = std::max<size_t>(src.size(), 1);
  hipError_t st = hipMalloc(&p, n * sizeof(X));
  if (st != hipSuccess) return st;
  owned.push_back(p);
  bytes += int64_t(n * sizeof(X));
  *dst = static_cast<X*>(p);
  if (src.empty()) return hipSuccess;
  std::vector<X> tmp(src.size());
  for (size_t i = 0; i < src.size(); ++i) tmp[i] = (X)src[i];
  return hipMemcpy(p, tmp.data(), tmp.size() * sizeof(X), hipMemcpyHostToDevice);
}

// Host image of the LDS reference block (same layout as Lay<Op, N>).
template <class Op, int N>
std::vector<double> ref_image(const Model& M) {
  using L = Lay<Op, N>;
  const int B = L::B, Bf = L::Bf, B1 = L::B1;
  std::vector<double> r(L::total, 0.0);
  // position of state row k in the image: fragment order for BF16
  auto pos = [](int k) { return L::BF ? tile_perm(k) : k; };
  for (int d = 0; d < 3; ++d)
    for (int k = 0; k < B; ++k)
      for (int l = 0; l < B1; ++l) {
        const double v = M.ref.K[(d * B + k) * B + l];
        r[L::oK + (d * L::PB + pos(k)) * L::ldK + pos(l)] = v;
        if (L::BF) r[L::oT + (d * L::PB1 + pos(l)) * L::ldT + pos(k)] = v;
      }
  for (int f = 0; f < 4; ++f)
    for (int c = 0; c < 16 * L::FT; ++c) {
      const int m = node_of(c);
      if (m >= Bf) continue;  // padding slot: zero
      for (int k = 0; k < B; ++k) {
        r[L::oE + (f * 16 * L::FT + c) * L::ldE + pos(k)] = M.ref.E[(f * Bf + m) * B + k];
        r[L::oL + (f * L::PB + pos(k)) * L::ldL + c] = M.ref.L[(f * B + k) * Bf + m];
      }
    }
  return r;
}

template <class Op>
std::vector<double> ref_image_n(const Model& M, int& bytes) {
  switch (M.N) {
    case 2: bytes = Lay<Op, 2>::bytes; return ref_image<Op, 2>(M);
    case 3: bytes = Lay<Op, 3>::bytes; return ref_image<Op, 3>(M);
    case 4: bytes = Lay<Op, 4>::bytes; return ref_image<Op, 4>(M);
    case 5: bytes = Lay<Op, 5>::bytes; return ref_image<Op, 5>(M);
    default: bytes = Lay<Op, 6>::bytes; return ref_image<Op, 6>(M);
  }
}

}  // namespace

// matrix-core launches by precision: 1 FP32, 2 BF16, 3 split BF16
hipError_t pred_dispatch_any(int precision, int N, const LaunchCfg& c, const TArgs& a, int64_t e0, int64_t e1,
                             const Sched& sc, hipStream_t s) {
  if (precision == 1) return pred_dispatch_f32(N, c, a, e0, e1, sc, s);
  if (precision == 3) return pred_dispatch_bf16x3(N, c, a, e0, e1, sc, s);
  return pred_dispatch_bf16(N, c, a, e0, e1, sc, s);
}

hipError_t corr_dispatch_any(int precision, int N, const LaunchCfg& c, const TArgs& a, int64_t e0, int64_t e1,
                             hipStream_t s) {
  if (precision == 1) return corr_dispatch_f32(N, c, a, e0, e1, s);
  if (precision == 3) return corr_dispatch_bf16x3(N, c, a, e0, e1, s);
  return corr_dispatch_bf16(N, c, a, e0, e1, s);
}

// A launch of the wavefront form (mc_min) needs elements enough to fill the chip with a
// wavefront per 16; a smaller one takes a work-group per 16 elements (group) where that keeps more
// of the chip busy than a work-group per element (plain). Measured, us of one launch, plain - group:
//   corrector, from 256 elements on: FP32 288 elements 0.9 (order 3) .. 3.5 (order 6), 1920 2.8 .. 12; FP64
//     288 -0.3 .. 0.5, 1920 3 .. 22; 162 elements 0.2 .. -0.2 and -0.4 .. -5;
//   predictor, FP32 from 256 on: 162 elements -0.3 (order 3) .. -27 (order 7), 288 0.2, -0.4, 2.9, -0.8, -3.9
//     (orders 3..7), 720 0.6 .. 4.1, 1920 2.5 .. 67;
//   predictor, FP64 from 896 on: 720 elements -1.1 .. -3.8, 900 -0.5, -1.8, 0.2, 6.6 (orders 3..6), 1080 0.2 .. 35;
//   predictor with faces towards a finer neighbour, whose traces take a launch of their own, from
//     1536 on: LTS boxes of 576, 900, 1296 elements -4 .. -33, 1903 -4 .. 32, 2304 -0.4 .. 72.
// Small ranges of the BF16 precisions stay on the plain kernels: BF16 rounding amplifies another
// order of the FP32 sums (one ulp in a few elements of a small cluster becomes 3e-4 of the
// result in four steps).
namespace {
constexpr int64_t kGroupCorrect = 256, kGroupPredict32 = 256, kGroupPredict64 = 896, kGroupFiner = 1536;
}  // namespace

Form launch_form(int precision, int N, int64_t mc_min, int64_t n, bool predictor, bool finer) {
  if (precision != 0 && n >= mc_min) return Form::wave;
  if (precision > 1 || (precision == 0 && !group_order<double>(N))) return Form::plain;
  int64_t from = kGroupCorrect;
  if (predictor) from = finer ? kGroupFiner : (precision == 0 ? kGroupPredict64 : kGroupPredict32);
  return n >= from ? Form::group : Form::plain;
}

namespace {

// f(c0, c1) of every element range that a launch may cover: a cluster, or clusters 0..c
template <class F>
void launch_ranges(const Model& M, F f) {
  for (int c = 0; c < M.C; ++c) {
    if (M.cluster_start[c + 1] > M.cluster_start[c]) f(c, c);
    if (c > 0 && M.cluster_start[c + 1] > 0) f(0, c);
  }
}

Form range_form(const Model& M, int precision, int64_t mc_min, int c0, int c1, bool predictor) {
  return launch_form(precision, M.N, mc_min, M.cluster_start[c1 + 1] - M.cluster_start[c0], predictor,
                     M.fix_start[c1 + 1] > M.fix_start[c0]);
}

}  // namespace

int64_t plain_elements(const Model& M, int precision, int64_t mc_min) {
  int64_t end = 0;
  launch_ranges(M, [&](int c0, int c1) {
    for (bool predictor : {true, false})
      if (range_form(M, precision, mc_min, c0, c1, predictor) == Form::plain) end = std::max(end, M.cluster_start[c1 + 1]);
  });
  return end;
}

// Half-step hand-over of the clusters that some launch predicts on the group kernels: the
// groups with a face towards a finer neighbour (slot in Ih) and, per cluster, their runs of the
// model's fix_list (sorted by element).
struct FinerLists {
  std::vector<int32_t> hslot, runs;
  std::vector<int64_t> start;
  int32_t slots = 0;
};

FinerLists finer_lists(const Model& M, int precision, int64_t mc_min) {
  std::vector<char> grouped(M.C, 0);
  launch_ranges(M, [&](int c0, int c1) {
    if (range_form(M, precision, mc_min, c0, c1, true) == Form::group)
      for (int c = c0; c <= c1; ++c) grouped[c] = 1;
  });
  FinerLists r;
  r.hslot.assign((M.E + 15) / 16, -1);
  r.start.assign(M.C + 1, 0);
  for (int c = 0; c < M.C; ++c) {
    r.start[c] = (int64_t)r.runs.size() / 3;
    int32_t last = -1;
    for (int64_t i = M.fix_start[c]; grouped[c] && i < M.fix_start[c + 1]; ++i) {
      const int32_t grp = M.fix_list[i] >> 6;  // entries are element * 4 + face
      if (r.hslot[grp] < 0) r.hslot[grp] = r.slots++;
      if (grp != last) {
        r.runs.insert(r.runs.end(), {grp, int32_t(i), 0});
        last = grp;
      }
      ++r.runs.back();
    }
  }
  r.start[M.C] = (int64_t)r.runs.size() / 3;
  return r;
}

template <typename T>
hipError_t alloc(std::vector<void*>& owned, int64_t& bytes, T** dst, int64_t n) {
  void* p = nullptr;
  const int64_t b = std::max<int64_t>(n, 1) * (int64_t)sizeof(T);
  const hipError_t st = hipMalloc(&p, b);
  if (st != hipSuccess) return st;
  owned.push_back(p);
  bytes += b;
  *dst = static_cast<T*>(p);
  return hipSuccess;
}

// Arguments of the group kernels (the pointwise flux coefficients are filled by the assembly).
template <typename T>
hipError_t group_build(GroupArgs<T>& a, TunedData& t, const Model& M, const DevData<T>& d, std::vector<void*>& owned,
                       int64_t& bytes) {
  a.Q = d.Q;
  a.In = d.In;
  a.G = d.G;
  a.mat = d.mat;
  a.H2 = d.H2;
  a.gD = d.gD;
  a.tgt = d.tgt;
  a.half2 = d.half2;
  a.rhalf2 = d.rhalf2;
  const FinerLists fl = finer_lists(M, t.precision, t.mc_min);
  t.run_start = fl.start;
  // a group hands over from its slot of I~_h: derivatives only for gravity and fault faces
  std::vector<int32_t> mh(M.E, 0), ds(M.gslot.begin(), M.gslot.end());
  for (size_t k = 0; k < M.f_elem.size(); ++k)
    for (int64_t e : {int64_t(M.f_elem[k]), int64_t(M.f_pelem[k])}) ds[e] = M.dslot[e];
  for (int64_t e = 0; e < M.E; ++e)
    for (int f = 0; f < 4; ++f) mh[e] |= ((M.mode[e * 4 + f] & 3) | (M.hperm[e * 4 + f] & 7) << 2) << (8 * f);
  const int B = n_basis(M.N);
  T *rcm, *rcp, *ih, *img;
  int32_t *pinv, *dm, *dl, *hs, *fx, *runs;
  hipError_t st = alloc(owned, bytes, &rcm, M.E * 48);
  if (st == hipSuccess) st = alloc(owned, bytes, &rcp, M.E * 48);
  if (st == hipSuccess) st = alloc(owned, bytes, &ih, fl.slots * int64_t(row_tiles(B) * 36 * 64));
  if (st == hipSuccess) st = upload(owned, bytes, &img, group_image(M, sizeof(T) == 8));
  if (st == hipSuccess) st = upload(owned, bytes, &pinv, M.ref.pinv);
  if (st == hipSuccess) st = upload(owned, bytes, &dm, mh);
  if (st == hipSuccess) st = upload(owned, bytes, &dl, ds);
  if (st == hipSuccess) st = upload(owned, bytes, &hs, fl.hslot);
  if (st == hipSuccess) st = upload(owned, bytes, &fx, M.fix_list);
  if (st == hipSuccess) st = upload(owned, bytes, &runs, fl.runs);
  if (st != hipSuccess) return st;
  a.RCm = rcm;
  a.RCp = rcp;
  a.Ih = ih;
  a.Et = d.Et;
  a.img = img;
  a.pinv = pinv;
  a.mh4 = dm;
  a.dslot = dl;
  a.hslot = hs;
  a.fix_list = fx;
  a.fix_group = runs;
  return hipSuccess;
}

hipError_t tuned_build(TunedData& t, const Model& M, int precision, const DevData<double>& d64,
                       const DevData<float>& d32, int tile, int acoustic, std::vector<void*>& owned,
                       int64_t& bytes) {
  t.N = M.N;
  t.precision = precision;
  t.d64 = d64;
  t.d32 = d32;
  t.finer = M.fix_start;
  t.plain_end = plain_elements(M, precision, t.mc_min);
  t.fix_start.assign(M.C + 1, 0);
  t.h2_start = M.h2_start;
  if (tile > 0) {
    const int w = tile <= 32 ? 2 : 4;
    t.pc = LaunchCfg{w, 0, 0, 2};
    t.cc = LaunchCfg{w, 0, 0, 2};
    t.fixed = 1;
  }
  // The two product shapes of BF16 round differently, so the shape follows from the order, tuned
  // or not, and not from a timing (which chose the same in all but a few runs): 32 K entries
  // at a time where no product is half empty. SEIS_TUNE alone overrides it.
  if (precision == 2) t.pc.variant = row_tiles(n_basis(M.N)) % 2 == 0;
  t.run_start.assign(M.C + 1, 0);
  bool grouped = false;  // whether some launch takes the group kernels
  launch_ranges(M, [&](int c0, int c1) {
    for (bool predictor : {true, false})
      grouped = grouped || range_form(M, precision, t.mc_min, c0, c1, predictor) == Form::group;
  });
  if (precision == 0) {
    const hipError_t sg = grouped ? group_build(t.g64, t, M, d64, owned, bytes) : hipSuccess;
    t.ready = sg == hipSuccess;
    return sg;
  }
  hipError_t st = hipSuccess;
  if (grouped) st = group_build(t.g32, t, M, d32, owned, bytes);
  if (st != hipSuccess) return st;
  TArgs& a = t.a;
  a.Q = d32.Q;
  a.In = d32.In;
  a.G = d32.G;
  a.mat = d32.mat;
  a.tgt = d32.tgt;
  a.mode = d32.mode;
  a.hperm = d32.hperm;
  a.H2 = d32.H2;
  a.half2 = d32.half2;
  a.rhalf2 = d32.rhalf2;
  a.gD = d32.gD;
  {
    const int64_t nJ = q_size(M.E, row_tiles(n_basis(M.N)));
    void* pj = nullptr;
    hipError_t sj = hipMalloc(&pj, nJ * sizeof(float));
    if (sj != hipSuccess) return sj;
    owned.push_back(pj);
    bytes += nJ * int64_t(sizeof(float));
    a.Ib = static_cast<float*>(pj);
  }
  // pointwise flux coefficients: filled by the operator assembly (shared with the group kernels)
  float* rc[2] = {const_cast<float*>(t.g32.RCm), const_cast<float*>(t.g32.RCp)};
  for (int i = 0; i < 2 && !rc[i]; ++i) {
    void* p = nullptr;
    const int64_t n = M.E * 4 * 12;
    hipError_t sa = hipMalloc(&p, n * sizeof(float));
    if (sa != hipSuccess) return sa;
    owned.push_back(p);
    bytes += n * int64_t(sizeof(float));
    rc[i] = static_cast<float*>(p);
  }
  float *rcm = rc[0], *rcp = rc[1];
  int32_t* pinv;
  st = upload(owned, bytes, &pinv, M.ref.pinv);
  if (st != hipSuccess) return st;
  a.RCm = rcm;
  a.RCp = rcp;
  a.pinv = pinv;
  {
    std::vector<int32_t> mh(M.E, 0);
    for (int64_t e = 0; e < M.E; ++e)
      for (int f = 0; f < 4; ++f) mh[e] |= ((M.mode[e * 4 + f] & 3) | (M.hperm[e * 4 + f] & 7) << 2) << (8 * f);
    int32_t* dm;
    st = upload(owned, bytes, &dm, mh);
    if (st != hipSuccess) return st;
    a.mh4 = dm;
  }
  {
    int32_t *ds, *fl, *hl;
    st = upload(owned, bytes, &ds, M.dslot);
    if (st == hipSuccess) st = upload(owned, bytes, &fl, M.fix_list);
    if (st == hipSuccess) st = upload(owned, bytes, &hl, M.h2_list);
    if (st != hipSuccess) return st;
    a.dslot = ds;
    a.fix_list = fl;
    // fix_list by element: the first entry of each and its slot of derivatives, and the end
    std::vector<int32_t> fe;
    for (int c = 0; c < M.C; ++c) {
      t.fix_start[c] = (int64_t)fe.size() / 2;
      for (int64_t i = M.fix_start[c]; i < M.fix_start[c + 1]; ++i)
        if (i == M.fix_start[c] || M.fix_list[i] >> 2 != M.fix_list[i - 1] >> 2)
          fe.insert(fe.end(), {int32_t(i), M.dslot[M.fix_list[i] >> 2]});
    }
    t.fix_start[M.C] = (int64_t)fe.size() / 2;
    fe.insert(fe.end(), {int32_t(M.fix_list.size()), -1});
    int32_t* dfe;
    st = upload(owned, bytes, &dfe, fe);
    if (st != hipSuccess) return st;
    t.fix_elem = dfe;
    a.h2_list = hl;
  }
  {
    // 16-element groups of acoustic elements (mu = 0) run in the 4-quantity
    // form; element order puts the acoustic elements of a cluster together
    const int64_t ng = (M.E + 15) / 16;
    std::vector<int32_t> gac(ng, 0);
    t.n_acoustic_groups = 0;
    for (int64_t gi = 0; gi < ng && acoustic; ++gi) {
      bool all = true;
      for (int64_t e = gi * 16; e < std::min<int64_t>(M.E, gi * 16 + 16); ++e) all = all && M.a_lmr[e * 3 + 1] == 0.0;
      gac[gi] = all ? 1 : 0;
      t.n_acoustic_groups += gac[gi];
    }
    int32_t* dg;
    st = upload(owned, bytes, &dg, gac);
    if (st != hipSuccess) return st;
    a.gac = dg;
  }
  // LDS image of the reference matrices (layout of Lay<Op, N>), padded to 16 bytes
  int lbytes = 0;
  if (precision == 1) {
    std::vector<double> ref = ref_image_n<OpF32>(M, lbytes);
    ref.resize(lbytes / 4, 0.0);
    float* r;
    st = upload(owned, bytes, &r, ref);
    a.ref = r;
  } else {
    // BF16: one image rounded to BF16; split BF16 (precision 3): the image of
    // hi = bf16(x), then the image of lo = bf16(x - hi)
    const bool split = precision == 3;
    std::vector<double> ref = split ? ref_image_n<OpBF16X3>(M, lbytes) : ref_image_n<OpBF16>(M, lbytes);
    std::vector<unsigned short> rb(lbytes / 2, 0);
    const size_t one = split ? rb.size() / 2 : rb.size();
    for (size_t i = 0; i < ref.size() && i < one; ++i) {
      const float x = (float)ref[i];
      rb[i] = f2bf(x);
      if (split) {
        const uint32_t u = uint32_t(rb[i]) << 16;
        float hi;
        std::memcpy(&hi, &u, 4);
        rb[one + i] = f2bf(x - hi);
      }
    }
    unsigned short* r;
    st = upload(owned, bytes, &r, rb);
    a.ref = r;
  }
  a.ref_bytes = lbytes;
  if (st != hipSuccess) return st;
  t.ready = 1;
  return hipSuccess;
}

hipError_t tuned_predict(const TunedData& t, int precision, int N, int c0, int c1, int64_t e0, int64_t e1,
                         const Sched& sc, hipStream_t s) {
  if (e1 <= e0) return hipSuccess;
  const int64_t r0 = t.run_start[c0], nr = t.run_start[c1 + 1] - r0;
  const Form form = launch_form(precision, N, t.mc_min, e1 - e0, true, t.finer[c1 + 1] > t.finer[c0]);
  if (form == Form::group) {
    hipError_t st = precision == 0 ? launch_predict_group<double>(N, t.g64, e0, e1, sc, s)
                                   : launch_predict_group<float>(N, t.g32, e0, e1, sc, s);
    if (st != hipSuccess) return st;
    return precision == 0 ? launch_finer<double>(N, t.g64, r0, nr, s) : launch_finer<float>(N, t.g32, r0, nr, s);
  }
  if (form == Form::plain) {
    if (e1 > t.plain_end) return hipErrorInvalidValue;  // the flux matrices end there
    return precision == 0 ? launch_predict_plain<double>(N, t.d64, e0, e1 - e0, sc, s)
                          : launch_predict_plain<float>(N, t.d32, e0, e1 - e0, sc, s);
  }
  hipError_t st = pred_dispatch_any(precision, N, t.pc, t.a, e0, e1, sc, s);
  if (st != hipSuccess) return st;
  return fixup_dispatch(N, t, t.fix_start[c0], t.fix_start[c1 + 1] - t.fix_start[c0], s);
}

hipError_t tuned_correct(const TunedData& t, int precision, int N, int c0, int c1, int64_t e0, int64_t e1,
                         const Sched& sc, hipStream_t s) {
  if (e1 <= e0) return hipSuccess;
  const Form form = launch_form(precision, N, t.mc_min, e1 - e0, false, false);
  if (form == Form::group)
    return precision == 0 ? launch_correct_group<double>(N, t.g64, e0, e1, sc, s)
                          : launch_correct_group<float>(N, t.g32, e0, e1, sc, s);
  if (form == Form::plain) {
    if (e1 > t.plain_end) return hipErrorInvalidValue;
    return precision == 0 ? launch_correct_plain<double>(N, t.d64, e0, e1 - e0, sc, s)
                          : launch_correct_plain<float>(N, t.d32, e0, e1 - e0, sc, s);
  }
  // second-half traces into the inbox of the clusters on the second step of
  // their pair (h2_list is ordered by cluster): one launch per run of such
  // clusters
  for (int c = c0; c <= c1;) {
    if (!((sc.sub >> c) & 1)) {
      ++c;
      continue;
    }
    int c2 = c;
    while (c2 + 1 <= c1 && ((sc.sub >> (c2 + 1)) & 1)) ++c2;
    const int64_t h0 = t.h2_start[c], nh = t.h2_start[c2 + 1] - h0;
    hipError_t st = h2_dispatch(N, t.a, t.a.h2_list + h0, nh, s);
    if (st != hipSuccess) return st;
    c = c2 + 1;
  }
  return corr_dispatch_any(precision, N, t.cc, t.a, e0, e1, s);
}


namespace {

// ---------------------------------------------------------------------------
// Autotuner: candidate launch configurations are timed on the largest
// cluster's matrix-core range; the winner is kept per (kernel sources, device,
// order, precision, size class) in a text cache, one line per key:
//   <key> <waves> <cap> <remap> <waves> <cap> <remap> <split> <variant>
// (predictor, corrector, the corrector's passes over its output rows, the
// predictor's shape: FP32 LDS or HBM park of I~, timed; BF16 16x16x16 or 16x16x32
// products, by the order). The cache is $SEIS_TUNE_CACHE, else $HOME/.cache/seis/tune.txt.
// SEIS_TUNE=0 disables tuning; SEIS_TUNE=w,cap,remap,w,cap,remap[,split[,variant]]
// fixes the configuration.

std::string cache_path() {
  const char* e = std::getenv("SEIS_TUNE_CACHE");
  if (e && *e) return e;
  const char* home = std::getenv("HOME");
  if (!home || !*home) return "";
  const std::string dir = std::string(home) + "/.cache/seis";
  ::mkdir((std::string(home) + "/.cache").c_str(), 0755);
  ::mkdir(dir.c_str(), 0755);
  return dir + "/tune.txt";
}

std::string tune_key(const TunedData& t, int64_t ngroups) {
  int dev = 0;
  hipDeviceProp_t prop;
  std::string arch = "unknown";
  if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) arch = prop.gcnArchName;
  for (char& c : arch)
    if (c == ' ' || c == ':') c = '_';
  int lg = 0;
  while ((int64_t(1) << (lg + 1)) <= ngroups) ++lg;
  std::ostringstream k;
  k << "v4/" << SEIS_SOURCE_HASH << "/" << arch << "/cu" << num_cus() << "/N" << t.N << "/p" << t.precision
    << "/g" << lg;
  return k.str();
}

bool valid(const LaunchCfg& c) {
  return (c.waves == 2 || c.waves == 4) && c.cap >= 0 && c.cap <= 8 && (c.remap == 0 || c.remap == 1) &&
         (c.split == 1 || c.split == 2) && (c.variant == 0 || c.variant == 1);
}

bool parse_cfg(const std::string& txt, LaunchCfg& p, LaunchCfg& c) {
  std::string t = txt;
  std::replace(t.begin(), t.end(), ',', ' ');
  std::istringstream in(t);
  LaunchCfg a, b;
  if (!(in >> a.waves >> a.cap >> a.remap >> b.waves >> b.cap >> b.remap)) return false;
  int sp = 2, var = 0;
  if (in >> sp) {
    b.split = sp;
    if (in >> var) a.variant = var;
  }
  if (!valid(a) || !valid(b)) return false;
  p = a;
  c = b;
  return true;
}

// average ms of n launches of fn after one warm-up launch
template <class F>
hipError_t time_launch(F fn, hipStream_t s, int n, float& ms) {
  hipEvent_t a, b;
  hipError_t st = hipEventCreate(&a);
  if (st != hipSuccess) return st;
  st = hipEventCreate(&b);
  if (st != hipSuccess) {
    (void)hipEventDestroy(a);
    return st;
  }
  st = fn();
  if (st == hipSuccess) st = hipEventRecord(a, s);
  for (int i = 0; i < n && st == hipSuccess; ++i) st = fn();
  if (st == hipSuccess) st = hipEventRecord(b, s);
  if (st == hipSuccess) st = hipEventSynchronize(b);
  if (st == hipSuccess) st = hipEventElapsedTime(&ms, a, b);
  ms /= float(n);
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  return st;
}

}  // namespace

hipError_t tuned_autotune(TunedData& t, const Model& M, hipStream_t s) {
  if (t.precision == 0 || t.fixed) return hipSuccess;
  const char* env = std::getenv("SEIS_TUNE");
  if (env && std::strcmp(env, "0") == 0) return hipSuccess;
  if (env && *env && parse_cfg(env, t.pc, t.cc)) {
    t.source = 0;
    return hipSuccess;
  }
  // the largest cluster
  int cbest = -1;
  int64_t nbest = 0;
  for (int c = 0; c < M.C; ++c) {
    const int64_t n = M.cluster_start[c + 1] - M.cluster_start[c];
    if (n > nbest) {
      nbest = n;
      cbest = c;
    }
  }
  if (cbest < 0 || nbest < 16 || nbest < t.mc_min) return hipSuccess;
  const int64_t e0 = M.cluster_start[cbest], ei = M.cluster_start[cbest + 1];
  const int64_t ngroups = ((ei - 1) >> 4) - (e0 >> 4) + 1;
  const std::string key = tune_key(t, ngroups);
  const std::string path = cache_path();
  if (!path.empty()) {
    std::ifstream in(path);
    std::string line;
    LaunchCfg p, c;
    bool hit = false;
    while (std::getline(in, line)) {
      std::istringstream ls(line);
      std::string k;
      if (!(ls >> k) || k != key) continue;
      std::string rest;
      std::getline(ls, rest);
      if (parse_cfg(rest, p, c)) hit = true;
    }
    if (hit) {
      t.pc = p;
      t.cc = c;
      t.source = 2;
      return hipSuccess;
    }
  }
  struct Timed {
    LaunchCfg c;
    float ms;
  };
  auto predict = [&](const LaunchCfg& c, int reps, float& ms) {
    return time_launch([&]() { return pred_dispatch_any(t.precision, t.N, c, t.a, e0, ei, Sched{}, s); }, s, reps, ms);
  };
  auto correct = [&](const LaunchCfg& c, int reps, float& ms) {
    return time_launch([&]() { return corr_dispatch_any(t.precision, t.N, c, t.a, e0, ei, s); }, s, reps, ms);
  };
  std::vector<Timed> pred, corr;
  for (int w : {4, 2})
    for (int cap : {0, 1, 2, 4})
      for (int rm : {0, 1}) {
        LaunchCfg c{w, cap, rm, 2, 0};
        float ms = 0.0f;
        // predictor: both shapes of FP32, the one that set-up chose in BF16
        for (int var : {0, 1}) {
          if (cap > 2 || (t.precision != 1 && var != t.pc.variant)) continue;
          c.variant = var;
          const hipError_t st = predict(c, 2, ms);
          if (st != hipSuccess) return st;
          pred.push_back({c, ms});
        }
        c.variant = 0;
        for (int sp : {2, 1}) {
          c.split = sp;
          const hipError_t st = correct(c, 2, ms);
          if (st != hipSuccess) return st;
          corr.push_back({c, ms});
        }
      }
  // Two launches differ by 2% from one another: the configurations within 3% of the best are timed
  // again, four times as long (split BF16, 42 775 elements: 0.296 and 0.295 ms after two launches, in
  // either order; 0.297 and 0.291 after eight, and 11.1 and 10.8 ms for a pass over the whole box).
  auto best = [&](std::vector<Timed>& all, auto& time, LaunchCfg& c) {
    auto less = [](const Timed& x, const Timed& y) { return x.ms < y.ms; };
    const float lim = 1.03f * std::min_element(all.begin(), all.end(), less)->ms;
    all.erase(std::remove_if(all.begin(), all.end(), [&](const Timed& x) { return x.ms > lim; }), all.end());
    for (Timed& x : all) {
      if (all.size() == 1) break;
      const hipError_t st = time(x.c, 8, x.ms);
      if (st != hipSuccess) return st;
    }
    c = std::min_element(all.begin(), all.end(), less)->c;
    return hipSuccess;
  };
  LaunchCfg bp, bc;
  hipError_t st = best(pred, predict, bp);
  if (st == hipSuccess) st = best(corr, correct, bc);
  if (st != hipSuccess) return st;
  t.pc = bp;
  t.cc = bc;
  t.source = 1;
  if (!path.empty()) {
    std::ofstream out(path, std::ios::app);
    if (out) out << key << ' ' << bp.waves << ' ' << bp.cap << ' ' << bp.remap << ' ' << bc.waves << ' ' << bc.cap
                 << ' ' << bc.remap << ' ' << bc.split << ' ' << bp.variant << '\n';
  }
  return hipSuccess;
}

}  // namespace seis
