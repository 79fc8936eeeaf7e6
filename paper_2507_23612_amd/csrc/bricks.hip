// Projector pass over a block of states on the matrix cores: the scatter of
// coupled projections, the projections of the result, or both at once,
//   Y_b += alpha Phi_b Q                              (64-point bricks)
//   part[pdest[slot]][s] = sum_{p in B} conj(Phi[slot][p]) Y[s][p]
//                                  (projection bricks B of four or ten bricks)
// (Sec. II.A potential section and Sec. II.B: the Hubbard orbitals are
// handled like nonlocal projectors).  Inside a Chebyshev step both run on the
// step's output: the projections are those of the next step's input.
#include "common.h"

#include <type_traits>

namespace hcu {

// A block's element as the kernels move it: a real number or the two parts
// of a complex one.
template <typename T>
struct El {
  using R = T;
  using E = T;
  static constexpr int C = 1;
};
template <typename S>
struct El<cplx<S>> {
  using R = S;
  using E = S __attribute__((ext_vector_type(2)));
  static constexpr int C = 2;
};
template <typename E>
__device__ __forceinline__ auto part_of(const E& v, int c) {
  if constexpr (std::is_arithmetic<E>::value) return v;
  else return c == 0 ? v.x : v.y;
}

// elements of one 16-byte access, consecutive in memory
template <typename T> constexpr int kPack = 16 / (int)sizeof(T);
template <typename E>
struct Pack {
  E v[kPack<E>];
};
template <typename E>
__device__ __forceinline__ Pack<E> ld_pack(const E* p) {
  Pack<E> r;
  __builtin_memcpy(&r, p, 16);
  return r;
}
using U4 = uint32_t __attribute__((ext_vector_type(4)));

// one block's share of a pass (pointers into global memory by type: a generic
// one from a job record would be read by flat loads, which LDS waits include)
template <typename P> using Glob = P __attribute__((address_space(1)));
template <typename T>
struct BrickArgs {
  using E = typename El<T>::E;
  Glob<E>* Y; int64_t ld; int ncol;
  const Glob<int64_t>* boff; const Glob<int>* bnj; const Glob<int>* bj; const Glob<E>* bval;
  const Glob<E>* Qt; int ldq; typename El<T>::R alpha; int nbrick;
  const Glob<int64_t>* pboff; const Glob<int>* pbnj; const Glob<E>* pbval; const Glob<int64_t>* pdest;
  Glob<E>* part; int ldp; int64_t nd;
};
template <typename T>
__host__ __device__ BrickArgs<T> brick_args(void* Y, int64_t ld, int ncol, const int64_t* boff, const int* bnj,
                                            const int* bj, const void* bval, const void* Qt, int ldq, double alpha,
                                            int nbrick, const int64_t* pboff, const int* pbnj, const void* pbval,
                                            const int64_t* pdest, void* part, int ldp, int64_t nd) {
  using E = typename El<T>::E;
  return {(Glob<E>*)Y, ld, ncol, (const Glob<int64_t>*)boff, (const Glob<int>*)bnj, (const Glob<int>*)bj,
          (const Glob<E>*)bval, (const Glob<E>*)Qt, ldq, (typename El<T>::R)alpha, nbrick, (const Glob<int64_t>*)pboff,
          (const Glob<int>*)pbnj, (const Glob<E>*)pbval, (const Glob<int64_t>*)pdest, (Glob<E>*)part, ldp, nd};
}

constexpr int kChunkFns = 16;                     // functions (slots) of one staged chunk
constexpr int kChunkVals = kChunkFns * kBrick;
template <typename T> constexpr int kTileRow = kBrick + kPack<T>;   // values of one state in the transposition tile
// A projection alone may load its values in the order in which the product
// takes them (lane (n, q): state n, points 4 i + q) instead of transposing
// them.  Done for 16-byte values, whose tile would leave room for one
// workgroup per compute unit: 112 instead of 121 us on 45x37x50, 75 states.
// (Elsewhere a load then meets four lines per quad of lanes: FP64 0.37
// instead of 0.33 ms on 72x72x96, 256 states.)
template <typename T, bool SC> constexpr bool kDirect = !SC && sizeof(T) == 16;
template <typename T, bool SC, bool PR>
constexpr int kBrickLds = (2 * kChunkVals + (PR && !kDirect<T, SC> ? 4 * 16 * kTileRow<T> : 0)) * (int)sizeof(T);

// A projection brick has up to 640 points, complex ones with two products
// each.  In 32 bits one chain of additions over all of them rounds at the size
// that its sum has reached, so each 64-point brick is summed from zero and
// joins the total once; the sum over the projection bricks runs in double
// precision (proj.hip).  Forces of 36 random blocks 0.9e-6 off 64 bits, complex
// ones 1.2e-6 (one chain: 1.3e-6 and 1.7e-6), in the same time; 1e-15 is left
// as it is in 64 bits, where this took 1 % of a complex filter.
template <typename T> constexpr bool kPieceSums = sizeof(typename El<T>::R) == 4;

// Waves per SIMD that the registers are allotted for: what the accumulators
// (a brick's values, as many requested ahead, NT slot tiles) leave room for.
// (FP64 with four tiles: two waves instead of three cost 0.72 instead of 0.65
// ms, complex FP32 0.94 instead of 0.87 ms on 72x72x96, 256 states.)
template <typename T, int NT>
constexpr int kBrickWaves = sizeof(T) == 16 ? 2 : sizeof(T) == 4 ? 4 : NT <= 4 ? 3 : 2;

// The workgroup's LDS writes are visible to all its waves (global loads and
// stores under way stay so).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A uniform address stays in scalar registers (the compiler would add it to
// the lanes' offsets, two vector additions per access).
template <typename P>
__device__ __forceinline__ P* scalar_base(P* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<P*>((uint64_t)hi << 32 | lo);
}

// One workgroup: the bricks k0 .. k1 - 1 (projection: brick b's), states
// swg .. swg + 63, wave w states swg + 16 w .. + 15.
//
//   scatter      D(16 states x 16 points) += alpha Q(16 x 4 functions) Phi(4 x 16 points)
//   projection   D(16 slots x 16 states)  += conj(Phi)(16 x 4 points) Y(4 x 16 states)
//
// (complex blocks: four real products each).  The tables pass through LDS in
// chunks of 16 functions x 64 points (both are stored in the order in which a
// chunk's operands are read), requested one chunk ahead by all four waves,
// one barrier per chunk; a brick's values are requested one brick ahead.
// Between the two products a wave transposes its values through an LDS tile
// of its own.
//
// Bound by the block's 64-byte runs and, from 4-byte values on, by the matrix
// cores about equally: 72x72x96, 256 states, FP64 both products 0.65 ms (read
// + write of the block 2.0 GB: 0.36 ms; products 0.2 ms), scatter alone 0.53,
// projection alone 0.29; 108x108x96, 640 states, FP32 2.59 ms (5.7 GB: 1.0
// ms; products 1.2 ms); 72x72x96, 256 states, complex FP32 0.87 ms.  The
// former kernels (tables staged behind two barriers per chunk, bricks that
// followed each other along x, every value requested where it was used) took
// 0.82, 0.58, 0.41, 3.25 and 1.09 ms.  One wave per 16 or 32 states without
// LDS was no faster than those: each table value then passes the vector cache
// once per wave, behind the block's own loads.  32 states per wave: 2.52
// instead of 2.39 ms in FP32 (half the waves).
template <typename T, typename OFF, int NT, bool SC, bool PR>
__device__ __forceinline__ void brick_pass(const BrickGeo& geo, const BrickArgs<T>& a, int b, int k0, int k1, int swg,
                                           unsigned char* lds) {
  using R = typename El<T>::R;
  using E = typename El<T>::E;
  using V = typename Mf<R>::V;
  constexpr int C = El<T>::C;
  constexpr bool DIR = kDirect<T, SC>;
  constexpr int G = kPack<E>, NG = 16 / G, RS = kTileRow<E>;
  constexpr int NL = kChunkVals / (256 * G);   // packs of a chunk that a thread stages
  E* const ring = reinterpret_cast<E*>(lds);
  const int lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  E* const yw = ring + 2 * kChunkVals + wave * (16 * RS);
  const int s0 = swg + 16 * wave;
  const bool wave_ok = s0 < a.ncol, full = s0 + 16 <= a.ncol;   // waves past the last state only stage
  const int njp = PR ? a.pbnj[b] : 0;
  if (PR && njp == 0) return;   // no function meets the brick
  const int64_t jop = PR ? a.pboff[b] : 0;
  // scatter chunks of the bricks (their lists follow each other, each padded
  // to whole chunks)
  int nsv = 0, left = 0;   // lane i: chunks of brick k0 + i; left: chunks not done yet
  const Glob<E>* sp = nullptr;
  const Glob<int>* ip = nullptr;
  if constexpr (SC) {
    nsv = (a.bnj[min(k0 + lane, k1 - 1)] + kChunkFns - 1) / kChunkFns;
    const int64_t jo = a.boff[k0];
    left = (int)((a.boff[k1] - jo) / kChunkFns);
    sp = a.bval + jo * kBrick;
    ip = a.bj + jo;
    if (!PR && left == 0) return;
  }
  auto chunks = [&](int k) { return SC ? __builtin_amdgcn_readlane(nsv, k - k0) : 0; };
  // lane (n, q) holds states s0 + q + 4 r at point n of every 16-point tile;
  // states past the last one repeat it (never stored)
  OFF voff[4];
  for (int r = 0; r < 4; ++r)
    voff[r] = ((OFF)(min(s0 + (DIR ? n : q + 4 * r), a.ncol - 1) - min(s0, a.ncol - 1)) * (OFF)a.ld +
               (OFF)geo.off(DIR ? q : n)) *
              (OFF)sizeof(E);
  const int sq = min(s0 + (sizeof(R) == 8 ? n : n / 4 + 4 * (n % 4)), a.ncol - 1);   // the state of operand row n
  Glob<E>* const Yw = a.Y + (int64_t)min(s0, a.ncol - 1) * a.ld;
  auto at = [&](Glob<E>* base, OFF o) -> Glob<E>& {
    return *reinterpret_cast<Glob<E>*>(reinterpret_cast<Glob<char>*>(base) + o);
  };

  V acc[C][4], pre[C][4];
  for (int c = 0; c < C; ++c)
    for (int pt = 0; pt < 4; ++pt)
      for (int r = 0; r < 4; ++r) pre[c][pt][r] = R(0);
  auto value = [&](int pt, int r) -> E {
    if constexpr (C == 1) return acc[0][pt][r];
    else return E{acc[0][pt][r], acc[1][pt][r]};
  };
  // brick k: its base, whether all its 64 points lie in the grid, and else how
  // far the lane's point of tile pt lies past the last one of its row (> 0: outside)
  auto place = [&](int k, bool* whole, int64_t* rem) {
    int w = 64;
    const int64_t p0 = geo.base(k, &w);
    *whole = geo.cube ? w == 1 << geo.lx : p0 + kBrick <= a.nd;
    *rem = geo.cube ? w : a.nd - p0;   // points left along x
    return p0;
  };
  // first point of the loads of (tile pt, r), and the lane's point in them
  auto first = [&](int pt, int r) { return DIR ? 16 * pt + 4 * r : 16 * pt; };
  auto past = [&](int64_t rem, int pt, int r) -> int64_t {
    return ((first(pt, r) + (DIR ? q : n)) & (geo.cube ? (1 << geo.lx) - 1 : 63)) - (rem - 1);
  };
  auto load_brick = [&](int k) {
    if (!wave_ok) return;
    bool whole;
    int64_t rem;
    const int64_t p0 = place(k, &whole, &rem);
    if (whole) {
      for (int pt = 0; pt < 4; ++pt)
        for (int r = 0; r < 4; ++r) {
          const E v = at(scalar_base(Yw + (p0 + geo.off(first(pt, r)))), voff[r]);
          for (int c = 0; c < C; ++c) pre[c][pt][r] = part_of(v, c);
        }
    } else {
      for (int pt = 0; pt < 4; ++pt)
        for (int r = 0; r < 4; ++r) {
          const int64_t d = past(rem, pt, r);   // outside: the last point, zeroed
          const E v = at(Yw + (p0 + geo.off(first(pt, r)) - (d > 0 ? d : 0)), voff[r]);
          for (int c = 0; c < C; ++c) pre[c][pt][r] = d > 0 ? R(0) : part_of(v, c);
        }
    }
  };
  auto store_brick = [&](int k) {
    bool whole;
    int64_t rem;
    const int64_t p0 = place(k, &whole, &rem);
    for (int pt = 0; pt < 4; ++pt) {
      Glob<E>* const base = scalar_base(Yw + (p0 + geo.off(16 * pt)));
      if (full && whole) {
        for (int r = 0; r < 4; ++r) at(base, voff[r]) = value(pt, r);
      } else if (past(rem, pt, 0) <= 0) {
        for (int r = 0; r < 4; ++r)
          if (s0 + q + 4 * r < a.ncol) at(base, voff[r]) = value(pt, r);
      }
    }
  };

  for (int t0 = 0; t0 == 0 || t0 * 16 < njp; t0 += NT) {   // more than NT slot tiles: projection only, one sweep each
    const int ntile = PR ? min((njp + 15) / 16 - t0, NT) : 0;
    const Glob<E>* const pp = PR ? a.pbval + (jop / 16 + t0) * (geo.pieces * kChunkVals) : nullptr;
    V pacc[NT][C];
    for (int t = 0; t < NT; ++t)
      for (int c = 0; c < C; ++c)
        for (int r = 0; r < 4; ++r) pacc[t][c][r] = R(0);

    U4 st[NL];
    E qn[4];
    int jv = 0, jvn = 0;   // function indices of the brick whose chunk is requested next (64 at a time), and of the next one
    auto request = [&](const Glob<E>* chunk) {
      const Glob<U4>* const base = (const Glob<U4>*)scalar_base(chunk);
      for (int i = 0; i < NL; ++i) st[i] = base[threadIdx.x + 256u * i];
    };
    auto request_scatter = [&](int c) {   // the next scatter chunk, number c of its brick, and its Q
      request(sp);
      if ((c & 3) == 0) jv = c == 0 ? jvn : ip[lane];   // (the array has a tail)
      for (int g = 0; g < 4; ++g) {
        const int j = __shfl(jv, (c & 3) * kChunkFns + 4 * g + q);
        qn[g] = a.Qt[(uint64_t)(unsigned)j * (unsigned)a.ldq + sq];
      }
      sp += kChunkVals;
      ip += kChunkFns;
    };
    auto stage = [&](int par) {
      for (int i = 0; i < NL; ++i) reinterpret_cast<U4*>(ring + par * kChunkVals)[threadIdx.x + 256 * i] = st[i];
    };
    int par = 0;
    if constexpr (SC) jvn = ip[lane];
    if (SC && (!PR || chunks(k0) > 0)) {
      request_scatter(0);
    } else {
      request(pp);
    }
    if (PR || chunks(k0) > 0) load_brick(k0);
    stage(0);
    for (int k = k0; k < k1; ++k) {
      for (int c = 0; c < C; ++c)
        for (int pt = 0; pt < 4; ++pt) acc[c][pt] = pre[c][pt];
      const int ns = chunks(k);
      // the next brick's values are requested behind the first chunk's request
      const bool fetch = k + 1 < k1 && (PR || chunks(k + 1) > 0);
      if constexpr (SC) {
        for (int ch = 0; ch < ns; ++ch) {
          lds_barrier();
          R qv[C][4];
          for (int g = 0; g < 4; ++g)
            for (int c = 0; c < C; ++c) qv[c][g] = a.alpha * part_of(qn[g], c);
          if (ch + 1 < ns) {
            request_scatter(ch + 1);
          } else if constexpr (!PR) {
            left -= ns;
            if (left > 0) {
              if (ns == 1 || !fetch) jvn = ip[lane];   // (else loaded with the next brick's values)
              request_scatter(0);
            }
          } else {
            request(pp + (k - k0) * kChunkVals);
          }
          if (ch == 0 && fetch) {
            if (PR || ns > 1) jvn = ip[kChunkFns * max(ns - 2, 0) + lane];   // (after the chunks requested so far)
            load_brick(k + 1);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (wave_ok) {
            const E* __restrict__ w = ring + par * kChunkVals + lane * G;
            for (int g = 0; g < 4; ++g) {
              E f[4];
              for (int i = 0; i < 4 / G; ++i) {
                const Pack<E> v = ld_pack(w + g * (4 * kBrick) + i * (64 * G));
                for (int e = 0; e < G; ++e) f[G * i + e] = v.v[e];
              }
              for (int pt = 0; pt < 4; ++pt)
                for (int c = 0; c < C; ++c) acc[c][pt] = Mf<R>::mfma(qv[0][g], part_of(f[pt], c), acc[c][pt]);
              if constexpr (C == 2)
                for (int pt = 0; pt < 4; ++pt) {
                  acc[0][pt] = Mf<R>::mfma(-qv[1][g], f[pt].y, acc[0][pt]);
                  acc[1][pt] = Mf<R>::mfma(qv[1][g], f[pt].x, acc[1][pt]);
                }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          par ^= 1;
          stage(par);
        }
        if (!PR && ns > 0 && wave_ok) store_brick(k);
        if (!PR && ns == 0 && fetch) load_brick(k + 1);   // (jvn is its list: a brick without functions adds none)
      }
      if constexpr (PR) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t >= ntile) break;   // uniform
          lds_barrier();
          if (t + 1 < ntile) {
            request(pp + ((t + 1) * geo.pieces + (k - k0)) * kChunkVals);
          } else if (k + 1 < k1) {
            if (SC && chunks(k + 1) > 0) request_scatter(0);
            else request(pp + (k + 1 - k0) * kChunkVals);
          }
          if (t == 0) {
            // (the stores and loads behind the request, whose wait would
            // include them otherwise)
            if (wave_ok) {
              if (SC && ns > 0) store_brick(k);
              if constexpr (!DIR) {
                for (int pt = 0; pt < 4; ++pt)
                  for (int r = 0; r < 4; ++r) yw[(q + 4 * r) * RS + 16 * pt + n] = value(pt, r);
                wave_lds_sync();
              }
            }
            if (ns == 0 && fetch) load_brick(k + 1);   // (jvn is its list, as above)
          }
          __builtin_amdgcn_sched_barrier(0);
          if (wave_ok) {
            const E* __restrict__ w = ring + par * kChunkVals + lane * G;
            const E* __restrict__ y = yw + n * RS + G * q;
            V sum[C];
            for (int c = 0; c < C; ++c)
              for (int r = 0; r < 4; ++r) sum[c][r] = kPieceSums<T> ? R(0) : pacc[t][c][r];
            for (int i = 0; i < NG; ++i) {
              const Pack<E> f = ld_pack(w + i * (64 * G));
              Pack<E> v;
              if constexpr (DIR) v.v[0] = value(i / 4, i % 4);
              else v = ld_pack(y + 4 * G * i);
              for (int e = 0; e < G; ++e) {
                for (int c = 0; c < C; ++c) sum[c] = Mf<R>::mfma(part_of(f.v[e], 0), part_of(v.v[e], c), sum[c]);
                if constexpr (C == 2) {
                  sum[0] = Mf<R>::mfma(f.v[e].y, v.v[e].y, sum[0]);
                  sum[1] = Mf<R>::mfma(-f.v[e].y, v.v[e].x, sum[1]);
                }
              }
            }
            for (int c = 0; c < C; ++c)
              for (int r = 0; r < 4; ++r) pacc[t][c][r] = kPieceSums<T> ? pacc[t][c][r] + sum[c][r] : sum[c][r];
          }
          __builtin_amdgcn_sched_barrier(0);
          par ^= 1;
          stage(par);
        }
      }
    }
    if constexpr (PR)
      if (wave_ok) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t >= ntile) break;
          int64_t dst[4];   // destination rows first (clamped), then the stores
          for (int r = 0; r < 4; ++r) dst[r] = a.pdest[jop + min((t0 + t) * 16 + Mf<R>::row(lane, r), njp - 1)];
          for (int r = 0; r < 4; ++r)
            if ((t0 + t) * 16 + Mf<R>::row(lane, r) < njp && s0 + n < a.ncol) {
              if constexpr (C == 1) a.part[dst[r] * a.ldp + s0 + n] = pacc[t][0][r];
              else a.part[dst[r] * a.ldp + s0 + n] = E{pacc[t][0][r], pacc[t][1][r]};
            }
        }
      }
    if (SC) break;
    lds_barrier();   // (before a next sweep restages the ring)
  }
}

// Order of the workgroups (brick group, 64 states): the groups of one row
// along x, then the state tiles.  Neighbours along x share cache lines of
// every state row, and a row's tables serve all state tiles, from the one L2
// (state tiles first: the FP32 pass of 108x108x96, 640 states 2.68 instead of
// 2.52 ms).
struct BrickItem {
  int b, s;
};
__device__ __forceinline__ BrickItem brick_item(const BrickGeo& geo, unsigned lw, unsigned nst) {
  const unsigned nb = geo.stacked() ? geo.nbx : 1, row = lw / (nb * nst), i = lw - row * (nb * nst);
  return {(int)(row * nb + i % nb), (int)(i / nb)};
}

template <typename T, typename OFF, int NT, bool SC, bool PR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kBrickWaves<T, NT>))) void k_brick_pass(
    const BrickArgs<T> a, int nst, int per, const BrickGeo geo) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kBrickLds<T, SC, PR>];
  const unsigned lw = xcd_linear();
  const BrickItem it = brick_item(geo, lw, nst);
  const int k0 = it.b * per;
  brick_pass<T, OFF, NT, SC, PR>(geo, a, it.b, k0, per == 1 ? k0 + 1 : k0 + geo.count(k0), it.s * 64, lds);
}

// One launch over the blocks of several (spin, k) problems: the workgroups of
// job i are item0_i .. item0_{i+1} - 1 (XCD-contiguous).
template <typename T, typename OFF, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kBrickWaves<T, NT>))) void k_brick_pass_batch(
    const FusedJob* __restrict__ jobs, int njob) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kBrickLds<T, true, true>];
  const unsigned lw = xcd_linear();
  // (a copy in scalar registers: read before any store)
  FusedJob J;
  {
    static_assert(sizeof(FusedJob) % 4 == 0, "copied by words");
    uint32_t w[sizeof(FusedJob) / 4];
    __builtin_memcpy(w, &fused_job(jobs, njob, lw), sizeof(FusedJob));
    for (uint32_t& x : w) x = __builtin_amdgcn_readfirstlane(x);
    __builtin_memcpy(&J, w, sizeof(FusedJob));
  }
  const BrickArgs<T> a = brick_args<T>(J.Y, J.ld, J.ncol, J.boff, J.bnj, J.bj, J.bval, J.Qt, J.ldq, J.alpha, J.nbrick,
                                       J.pboff, J.pbnj, J.pbval, J.pdest, J.part, J.ldp, J.nd);
  const BrickItem it = brick_item(J.geo, lw - J.item0, J.nst);
  const int k0 = it.b * J.geo.pieces;
  brick_pass<T, OFF, NT, true, true>(J.geo, a, it.b, k0, k0 + J.geo.count(k0), it.s * 64, lds);
}

// f(offset type): 32-bit byte offsets while a wave's 16 states span less than 4 GB
template <typename T, typename F>
void brick_offsets(int64_t ld, F f) {
  if (ld * (int64_t)sizeof(T) * 16 < (int64_t)1 << 32) f(uint32_t());
  else f(int64_t());
}

template <typename T>
void launch_brick_pass(const Ctx& c, const T* bval, const T* pbval, T* Y, int64_t ld, int ncol, const T* Qt,
                       double alpha, bool scatter, bool project, hipStream_t st) {
  const int nbrick = (int)c.boff.size() - 1, nst = (ncol + 63) / 64;
  const BrickArgs<T> a = brick_args<T>(Y, ld, ncol, c.d_boff, c.d_bnj, c.d_bj, bval, Qt, c.p.ns, alpha, nbrick, c.d_pboff,
                                       c.d_pbnj, pbval, c.d_pdest, c.d_ppart, c.p.ns, c.nd);
  // A scatter alone takes single bricks where groups of four would leave
  // compute units without a second workgroup
  const int per = !project && (size_t)nbrick * nst < (size_t)4 * 256 * c.geo.pieces ? 1 : c.geo.pieces;
  const unsigned items = (unsigned)((nbrick + per - 1) / per) * nst;
  brick_offsets<T>(ld, [&](auto off) {
    using OFF = decltype(off);
    using Y_ = std::true_type;
    using N_ = std::false_type;
    auto run = [&](auto nt, auto sc, auto pr) {
      launch_k(k_brick_pass<T, OFF, decltype(nt)::value, decltype(sc)::value, decltype(pr)::value>, items, 256, 0, st, a,
               nst, per, c.geo);
    };
    auto slots = [&](auto sc) {
      if (c.max_ptiles <= 4) run(std::integral_constant<int, 4>(), sc, Y_());
      else if constexpr (El<T>::C == 1) run(std::integral_constant<int, 8>(), sc, Y_());
      else if constexpr (!decltype(sc)::value) run(std::integral_constant<int, 4>(), sc, Y_());
    };
    if (!project) run(std::integral_constant<int, 1>(), Y_(), N_());
    else if (!scatter) slots(N_());
    else if constexpr (sizeof(T) < 16) slots(Y_());
  });
}

template <typename T>
void launch_brick_pass_batch(const FusedJob* d_jobs, int njob, unsigned items, int NT, int64_t ld, hipStream_t st) {
  brick_offsets<T>(ld, [&](auto off) {
    using OFF = decltype(off);
    if (El<T>::C == 2 || NT <= 4) launch_k(k_brick_pass_batch<T, OFF, 4>, items, 256, 0, st, d_jobs, njob);
    else if constexpr (El<T>::C == 1) launch_k(k_brick_pass_batch<T, OFF, 8>, items, 256, 0, st, d_jobs, njob);
  });
}
template void launch_brick_pass_batch<double>(const FusedJob*, int, unsigned, int, int64_t, hipStream_t);
template void launch_brick_pass_batch<float>(const FusedJob*, int, unsigned, int, int64_t, hipStream_t);
template void launch_brick_pass_batch<cplx<float>>(const FusedJob*, int, unsigned, int, int64_t, hipStream_t);

template <typename T>
void launch_nl_scatter(const Ctx& c, int ik, T* Y, int64_t ld, int ncol, const T* Qt, double alpha, hipStream_t st) {
  if (c.nproj > 0) launch_brick_pass<T>(c, (const T*)c.d_bval[ik], nullptr, Y, ld, ncol, Qt, alpha, true, false, st);
}

#define INST_BRICK(T)                                                                                             \
  template void launch_brick_pass<T>(const Ctx&, const T*, const T*, T*, int64_t, int, const T*, double, bool, bool, \
                                     hipStream_t);                                                                \
  template void launch_nl_scatter<T>(const Ctx&, int, T*, int64_t, int, const T*, double, hipStream_t);
INST_BRICK(double)
INST_BRICK(float)
INST_BRICK(cplx<double>)
INST_BRICK(cplx<float>)

}  // namespace hcu
