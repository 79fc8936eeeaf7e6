// Projections of a block of states onto the atom-centred functions
// (Sec. II.B: the integrals of every atom's functions, as for nonlocal
// projectors):
//
//   P[s][j] = dV * sum_x conj(phi_j(x)) y_s(x)                 (trapezoid rule)
//   Q[j][s] = sum_m' C_b[m][m'] P[s][j0+m']     (Q stored transposed for the scatter)
//
// with C_b = diag(gamma) for the KB channels and C_b = U (1/2 - D) for the
// Hubbard manifold (Eq. DerED).  The grid is cut into bricks of a few hundred
// neighbouring points; each brick's functions form a dense value tile, and
// a workgroup computes the brick's partial projections for 64 states as a
// small GEMM on the matrix cores, reading every point-state value once.  The
// partials are summed per function in a fixed order (deterministic), then
// the coupling is applied.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace hcu {

// Stage 2: P[s][j] = dV * sum of rows jrow[j] .. jrow[j+1] of part (fixed
// order).  One workgroup per (j, 64 states, job); its 16 waves take every 16th
// row and are combined in a fixed order.  JOBS: the pointers of job z instead
// of those given.  Bound by reading the partials: 41 us for the 126 MB of
// 72x72x96, 256 states (four rows under way per wave instead of two: 42 us).
template <typename T, bool JOBS>
__global__ __launch_bounds__(1024) void k_slot_sum(const TailJob* __restrict__ jobs, const T* __restrict__ part,
                                                   T* __restrict__ P, int ldp, int ncol,
                                                   const int64_t* __restrict__ jrow, int nproj, double dv) {
  using RT = typename real_of<T>::type;
  using D = double_of<T>;
  __shared__ __attribute__((aligned(16))) unsigned char red_raw[16 * 64 * sizeof(D)];
  D(*red)[64] = reinterpret_cast<D(*)[64]>(red_raw);
  if constexpr (JOBS) {
    part = (const T*)jobs[blockIdx.z].part;
    P = (T*)jobs[blockIdx.z].P;
  }
  const int j = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int s = blockIdx.x * 64 + lane;
  D x0 = D(0), x1 = D(0);
  if (s < ncol) {
    const int64_t r1 = jrow[j + 1];
    int64_t r = jrow[j] + wave;
    for (; r + 16 < r1; r += 32) {
      x0 += widen(part[r * ldp + s]);
      x1 += widen(part[(r + 16) * ldp + s]);
    }
    if (r < r1) x0 += widen(part[r * ldp + s]);
  }
  red[wave][lane] = x0 + x1;
  __syncthreads();
  if (wave == 0 && s < ncol) {
    D x = D(0);
    for (int w = 0; w < 16; ++w) x += red[w][lane];
    P[(int64_t)s * nproj + j] = narrow<T>(dv * x);
  }
}

// Q[j0+m][s] = sum_m' C_b[m][m'] P[s][j0+m'], one thread per (block, state, job).
template <typename T, bool JOBS>
__global__ __launch_bounds__(64) void k_couple(const TailJob* __restrict__ jobs, const T* __restrict__ P, const double* __restrict__ coup,
                         T* __restrict__ Q, const BlockDesc* __restrict__ blocks, int ncol, int nproj, int ldq) {
  if constexpr (JOBS) {
    P = (const T*)jobs[blockIdx.z].P;
    Q = (T*)jobs[blockIdx.z].Q;
    coup = jobs[blockIdx.z].coup;
  }
  const BlockDesc& b = blocks[blockIdx.y];
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= ncol) return;
  using RT = typename real_of<T>::type;
  // (full loops over kMaxNm with guards: the values stay in registers, and
  // their loads go out together from clamped addresses)
  const int nm = b.nm;
  const double* __restrict__ cb = coup + b.coup_off;
  T pv[kMaxNm];
  for (int m = 0; m < kMaxNm; ++m) pv[m] = P[(int64_t)s * nproj + b.j0 + min(m, nm - 1)];
  for (int m = 0; m < nm; ++m) {
    T qv = T(0);
    for (int mp = 0; mp < kMaxNm; ++mp) {
      const RT f = (RT)cb[m * nm + min(mp, nm - 1)];
      if (mp < nm) qv += f * pv[mp];
    }
    Q[(int64_t)(b.j0 + m) * ldq + s] = qv;
  }
}

// Several blocks of one context in one launch each: 16 complex FP32 blocks of
// 36x36x24, 32 states, block by block took 155 us per step (the SCF of two spins
// and 8 k-points 67 ms; 55 ms this way).
template <typename T>
static void launch_slot_sum(const Ctx& c, const TailJob* d_jobs, int njob, const TailJob& one, int ncol, hipStream_t st) {
  auto run = [&](auto k) {
    launch_k(k, dim3((ncol + 63) / 64, c.nproj, njob), 1024, 0, st, d_jobs, (const T*)one.part, (T*)one.P, c.p.ns, ncol,
             c.d_jrow, c.nproj, c.dv);
  };
  if (d_jobs) run(k_slot_sum<T, true>);
  else run(k_slot_sum<T, false>);
}
template <typename T>
static void launch_couple_jobs(const Ctx& c, const TailJob* d_jobs, int njob, const TailJob& one, int ncol,
                               hipStream_t st) {
  auto run = [&](auto k) {
    launch_k(k, dim3((ncol + 63) / 64, (unsigned)c.blocks.size(), njob), 64, 0, st, d_jobs, (const T*)one.P, one.coup,
             (T*)one.Q, c.d_blocks, ncol, c.nproj, c.p.ns);
  };
  if (d_jobs) run(k_couple<T, true>);
  else run(k_couple<T, false>);
}
template <typename T>
void launch_sum_couple(const Ctx& c, const TailJob* d_jobs, int njob, const TailJob& one, int ncol, hipStream_t st) {
  launch_slot_sum<T>(c, d_jobs, njob, one, ncol, st);
  launch_couple_jobs<T>(c, d_jobs, njob, one, ncol, st);
}
template void launch_sum_couple<double>(const Ctx&, const TailJob*, int, const TailJob&, int, hipStream_t);
template void launch_sum_couple<float>(const Ctx&, const TailJob*, int, const TailJob&, int, hipStream_t);
template void launch_sum_couple<cplx<double>>(const Ctx&, const TailJob*, int, const TailJob&, int, hipStream_t);
template void launch_sum_couple<cplx<float>>(const Ctx&, const TailJob*, int, const TailJob&, int, hipStream_t);

template <typename T>
bool scatter_project_ok(const Ctx& c) {
  if (c.nproj == 0 || c.pboff.empty()) return false;
  if constexpr (sizeof(T) == sizeof(typename real_of<T>::type)) return c.max_ptiles <= 8;
  else if constexpr (std::is_same<T, cplx<float>>::value) return c.max_ptiles <= 4;
  else return false;   // complex FP64: the accumulators do not fit the register budget
}

// part: 1 = the fused kernel only, 2 = the partial sums and coupling that
// follow it only, 3 = both (separate parts let the caller time the kernel)
template <typename T>
void launch_scatter_project(const Ctx& c, int ik, T* Y, int64_t ld, int ncol, const T* Qt, double alpha,
                            const double* coup, T* P, T* Q, hipStream_t st, int part_sel) {
  if constexpr (!std::is_same<T, cplx<double>>::value) {
    if (part_sel & 1)
      launch_brick_pass<T>(c, (const T*)c.d_bval[ik], (const T*)c.d_pbval[ik], Y, ld, ncol, Qt, alpha, true, true, st);
    if (part_sel & 2) launch_sum_couple<T>(c, nullptr, 1, TailJob{c.d_ppart, P, Q, coup}, ncol, st);
  }
}

template bool scatter_project_ok<double>(const Ctx&);
template bool scatter_project_ok<float>(const Ctx&);
template bool scatter_project_ok<cplx<double>>(const Ctx&);
template bool scatter_project_ok<cplx<float>>(const Ctx&);
template void launch_scatter_project<double>(const Ctx&, int, double*, int64_t, int, const double*, double,
                                             const double*, double*, double*, hipStream_t, int);
template void launch_scatter_project<float>(const Ctx&, int, float*, int64_t, int, const float*, double,
                                            const double*, float*, float*, hipStream_t, int);
template void launch_scatter_project<cplx<double>>(const Ctx&, int, cplx<double>*, int64_t, int,
                                                   const cplx<double>*, double, const double*, cplx<double>*,
                                                   cplx<double>*, hipStream_t, int);
template void launch_scatter_project<cplx<float>>(const Ctx&, int, cplx<float>*, int64_t, int, const cplx<float>*,
                                                  double, const double*, cplx<float>*, cplx<float>*, hipStream_t,
                                                  int);

// The job record of the fused pass of one block (the block's data, the
// projection partials of that block, its first workgroup).
template <typename T>
FusedJob fused_job_of(const Ctx& c, int ik, T* Y, int64_t ld, int ncol, const T* Qt, double alpha, void* part,
                      unsigned item0) {
  FusedJob j{};
  j.geo = c.geo;
  j.Y = Y; j.ld = ld; j.ncol = ncol; j.nst = (ncol + 63) / 64;
  j.boff = c.d_boff; j.bnj = c.d_bnj; j.bj = c.d_bj; j.bval = c.d_bval[ik];
  j.Qt = Qt; j.ldq = c.p.ns; j.alpha = alpha; j.nbrick = (int)c.boff.size() - 1;
  j.pboff = c.d_pboff; j.pbnj = c.d_pbnj; j.pbval = c.d_pbval[ik]; j.pdest = c.d_pdest;
  j.part = part; j.ldp = c.p.ns; j.nd = c.nd;
  j.item0 = item0;
  return j;
}

unsigned fused_job_items(const Ctx& c, int ncol) {
  return (unsigned)((c.pboff.size() - 1) * (size_t)((ncol + 63) / 64));
}

template <typename T>
void launch_scatter_project_batch(const FusedJob* d_jobs, int njob, unsigned items, int NT, int64_t ld, hipStream_t st) {
  if constexpr (!std::is_same<T, cplx<double>>::value) launch_brick_pass_batch<T>(d_jobs, njob, items, NT, ld, st);
}

#define INST_FUSED_JOB(T)                                                                                    \
  template FusedJob fused_job_of<T>(const Ctx&, int, T*, int64_t, int, const T*, double, void*, unsigned);  \
  template void launch_scatter_project_batch<T>(const FusedJob*, int, unsigned, int, int64_t, hipStream_t);
INST_FUSED_JOB(double)
INST_FUSED_JOB(float)
INST_FUSED_JOB(cplx<double>)
INST_FUSED_JOB(cplx<float>)

size_t project_partial_elems(const Ctx& c) {
  if (c.pboff.empty()) return 0;
  return (size_t)c.pboff.back() * c.p.ns;
}

// P = Phi^H Y dV with the function values of `table` (projection-brick
// layout: the context's orbitals/projectors at a k-point, or other functions
// on the same supports, e.g. their moments).
template <typename T>
void launch_project_table(const Ctx& c, const T* table, const T* Y, int ncol, int64_t ld, T* P, hipStream_t st) {
  if (c.nproj == 0) return;
  launch_brick_pass<T>(c, nullptr, table, const_cast<T*>(Y), ld, ncol, nullptr, 0.0, false, true, st);
  launch_slot_sum<T>(c, nullptr, 1, TailJob{c.d_ppart, P, nullptr, nullptr}, ncol, st);
}

template <typename T>
void launch_project_brick(const Ctx& c, int ik, const T* Y, int ncol, int64_t ld, const double* coup, T* P, T* Q,
                          hipStream_t st) {
  if (c.nproj == 0) return;
  launch_brick_pass<T>(c, nullptr, (const T*)c.d_pbval[ik], const_cast<T*>(Y), ld, ncol, nullptr, 0.0, false, true,
                       st);
  launch_sum_couple<T>(c, nullptr, 1, TailJob{c.d_ppart, P, Q, coup}, ncol, st);
}

template <typename T>
void launch_couple(const Ctx& c, const T* P, int ncol, const double* coup, T* Q, hipStream_t st) {
  if (c.nproj == 0) return;
  launch_couple_jobs<T>(c, nullptr, 1, TailJob{nullptr, const_cast<T*>(P), Q, coup}, ncol, st);
}
template void launch_couple<double>(const Ctx&, const double*, int, const double*, double*, hipStream_t);
template void launch_couple<float>(const Ctx&, const float*, int, const double*, float*, hipStream_t);
template void launch_couple<cplx<double>>(const Ctx&, const cplx<double>*, int, const double*, cplx<double>*,
                                          hipStream_t);
template void launch_couple<cplx<float>>(const Ctx&, const cplx<float>*, int, const double*, cplx<float>*,
                                         hipStream_t);

template void launch_project_table<double>(const Ctx&, const double*, const double*, int, int64_t, double*,
                                           hipStream_t);
template void launch_project_table<float>(const Ctx&, const float*, const float*, int, int64_t, float*, hipStream_t);
template void launch_project_table<cplx<double>>(const Ctx&, const cplx<double>*, const cplx<double>*, int, int64_t,
                                                 cplx<double>*, hipStream_t);
template void launch_project_table<cplx<float>>(const Ctx&, const cplx<float>*, const cplx<float>*, int, int64_t,
                                                cplx<float>*, hipStream_t);

template void launch_project_brick<double>(const Ctx&, int, const double*, int, int64_t, const double*, double*,
                                           double*, hipStream_t);
template void launch_project_brick<float>(const Ctx&, int, const float*, int, int64_t, const double*, float*,
                                          float*, hipStream_t);
template void launch_project_brick<cplx<double>>(const Ctx&, int, const cplx<double>*, int, int64_t, const double*,
                                                 cplx<double>*, cplx<double>*, hipStream_t);
template void launch_project_brick<cplx<float>>(const Ctx&, int, const cplx<float>*, int, int64_t, const double*,
                                                cplx<float>*, cplx<float>*, hipStream_t);

}  // namespace hcu
