// Local part of H and the Chebyshev three-term step in one pass over the grid:
//
//   out = alpha * ( -1/2 Delta_h y + V y - c y ) - beta * yprev
//
// -1/2 Delta_h is the centred 2*n0-order stencil along each axis with
// periodic wrap and the Bloch factor e^{+-i k_a L_a} on wrapped values
// (Sec. II.B: off-grid indices are mapped back periodically with the Bloch
// factor).  The projector term alpha * sum_j phi_j Q_j is added afterwards by
// the projector pass (bricks.hip).
//
// Layout: y is one column of an nd x ncol column-major block, x fastest.  A
// workgroup owns a TX x TY tile of an x-y plane for one state and streams a
// range of z planes; each thread owns RY points stacked in y.  A plane is
// used up when it arrives: it is staged in LDS with its x/y halo (wrapped),
// its in-plane sum goes to its own output, and its values are added with the
// z weights to the running sums of the 2R outputs around it, which wait in
// registers (as many as a queue of z neighbours would take).
#include "common.h"
#include "stencil_tile.h"

#include <algorithm>
#include <type_traits>

namespace hcu {


template <typename RT>
struct KArgs {
  RT kx[kMaxR + 1], ky[kMaxR + 1], kz[kMaxR + 1];   // alpha times the weights
  RT center, center_lo;         // alpha (sum of the three centre weights - c) and what its rounding left (stencil_args)
  RT alpha, beta;
  RT ph_re[3], ph_im[3];        // Bloch factor per axis
  int n1, n2, n3;
  int tiles_x, tz;
  int has_prev;
  int64_t ld, ld_prev, ld_out;
};

template <typename RT>
struct SJob {
  const void* Yin;
  const void* Yprev;
  void* Yout;
  const RT* V;
  KArgs<RT> a;
  int ntiles, nzc;
  unsigned long long item_begin;
};

// One column of a block as a buffer resource: uniform base and size, a
// uniform byte offset of the plane and a 32-bit byte offset per lane.  Every
// access is range-checked by the hardware: reads at or past the size return
// 0 and writes there are dropped, so offset kNone stands for "no point" and a
// size of 0 for "no block", without a branch.
constexpr unsigned kNone = 0x80000000u;   // columns are smaller (2^22 points of 16 bytes)
template <typename T, int N>
struct Vec {   // N points consecutive in x
  T v[N];
  __device__ T& operator[](int i) { return v[i]; }
  __device__ const T& operator[](int i) const { return v[i]; }
};
struct Col {
  __amdgpu_buffer_rsrc_t r;
  __device__ Col(const void* p, unsigned bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000)) {}
  template <typename W>
  __device__ __forceinline__ W get(unsigned lane, unsigned plane) const {
    static_assert(sizeof(W) == 4 || sizeof(W) == 8 || sizeof(W) == 16, "one load");
    W v;
    if constexpr (sizeof(W) == 4) {
      const auto u = __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane, (int)plane, 0);
      __builtin_memcpy(&v, &u, 4);
    } else if constexpr (sizeof(W) == 8) {
      const auto u = __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane, (int)plane, 0);
      __builtin_memcpy(&v, &u, 8);
    } else {
      const auto u = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane, (int)plane, 0);
      __builtin_memcpy(&v, &u, 16);
    }
    return v;
  }
  // The plane goes into the lane offset: with a scalar offset the compiler
  // takes 16-byte stores as free to have their data registers overwritten by
  // the next instruction, and under load they then stored the new contents.
  template <typename W>
  __device__ __forceinline__ void put(W v, unsigned lane, unsigned plane) const {
    const unsigned at = lane + plane;
    using u2 = unsigned __attribute__((ext_vector_type(2)));
    using u4 = unsigned __attribute__((ext_vector_type(4)));
    if constexpr (sizeof(W) == 4) {
      unsigned u;
      __builtin_memcpy(&u, &v, 4);
      __builtin_amdgcn_raw_buffer_store_b32(u, r, (int)at, 0, 0);
    } else if constexpr (sizeof(W) == 8) {
      u2 u;
      __builtin_memcpy(&u, &v, 8);
      __builtin_amdgcn_raw_buffer_store_b64(u, r, (int)at, 0, 0);
    } else {
      u4 u;
      __builtin_memcpy(&u, &v, 16);
      __builtin_amdgcn_raw_buffer_store_b128(u, r, (int)at, 0, 0);
    }
  }
};
// Computed here, not later: sums are otherwise moved past the next branch,
// with every operand read before it waiting in registers.
__device__ __forceinline__ void pin(float& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin(double& v) { asm volatile("" : "+v"(v)); }
template <typename R>
__device__ __forceinline__ void pin(cplx<R>& v) { pin(v.re); pin(v.im); }

// acc plus the centre term (center + center_lo + alpha V) y.  In 32 bits the
// large part takes its own product: added to the others it would round them
// at its size.
template <typename T, typename RT>
__device__ __forceinline__ T add_centre(T acc, RT v, T y, const KArgs<RT>& a) {
  if constexpr (sizeof(RT) == 4) {
    acc += (a.alpha * v + a.center_lo) * y;
    acc += a.center * y;
  } else {
    acc += (a.center + a.alpha * v) * y;
  }
  return acc;
}

// an aligned vector of LDS values
template <typename W>
__device__ __forceinline__ W lds_get(const void* p) {
  W v;
  __builtin_memcpy(&v, __builtin_assume_aligned(p, sizeof(W)), sizeof(W));
  return v;
}
template <typename W>
__device__ __forceinline__ void lds_put(void* p, const W& v) {
  __builtin_memcpy(__builtin_assume_aligned(p, sizeof(W)), &v, sizeof(W));
}

// Bloch factor e^{i sum_d w_d k_d L_d} of a node reached with wrap counts w
// (1 for real blocks, which carry no factor).
template <typename T> struct Ph {
  static constexpr bool on = false;
  template <typename RT>
  __device__ static inline T of(int, int, int, const KArgs<RT>&) { return T(1); }
  __device__ static inline T mul(T v, T) { return v; }
};
template <typename R> struct Ph<cplx<R>> {
  static constexpr bool on = true;
  template <typename RT>
  __device__ static inline cplx<R> of(int wx, int wy, int wz, const KArgs<RT>& a) {
    cplx<R> ph(R(1), R(0));
    const int w[3] = {wx, wy, wz};
    for (int d = 0; d < 3; ++d) {
      const cplx<R> f(a.ph_re[d], w[d] > 0 ? a.ph_im[d] : -a.ph_im[d]);
      for (int t = 0; t < (w[d] > 0 ? w[d] : -w[d]); ++t) ph = ph * f;
    }
    return ph;
  }
  __device__ static inline cplx<R> mul(cplx<R> v, cplx<R> ph) { return v * ph; }
};

// periodic image of grid coordinate g: returns g - w n in [0, n), w = floor(g / n)
__device__ inline int wrap(int g, int n, int& w) {
  w = (g >= 0) ? g / n : -((n - 1 - g) / n);
  return g - w * n;
}

constexpr int kRingR = 6;   // shapes with the halo_ring flag: order-12 stencil

// Threads per workgroup a variant is built for: the light real ones (one
// FP64 or up to two FP32 points per thread) fit 128 registers, others get 256.
template <typename T, typename RT, int PT>
constexpr int kStencilThreads = (sizeof(T) == sizeof(RT) && PT * sizeof(T) <= 8) ? 1024 : 512;

// Waves per SIMD a variant is compiled for (512 registers shared): the
// running sums of VX x RY points take 2R words each, and left to itself the
// scheduler spends all registers of two waves on reading LDS ahead.
template <typename T, int VX, int RY>
constexpr int kStencilWaves = VX * RY * sizeof(T) <= 4 ? 8 : VX * RY * sizeof(T) <= 8 ? 5
                            : VX * RY * sizeof(T) <= 16 ? (sizeof(T) == 16 ? 3 : 4) : VX == 2 ? 3 : 2;

// Real points that are not side by side in vectors take the queue form.
template <typename T, int VX>
constexpr bool kQueue = VX == 1 && std::is_arithmetic<T>::value;
template <typename T, int VX, int RY>
constexpr int kWaves = kQueue<T, VX> ? 2 : kStencilWaves<T, VX, RY>;

// One work item: tile `tile` of the x-y plane, z chunk `zc`, state `s`.
//
// What bounds it: HBM streaming (3 words per point) as long as the y/x halo of
// a tile is found in L2.  Therefore the z direction is summed forwards: plane
// z is staged, its in-plane sum formed and its z weights applied all at the
// moment it is read, so a tile reads its halo rows of plane z while the
// neighbouring tiles read the same rows as their own.  (With a queue of z
// neighbours the halo of plane z is read R planes after the neighbours read
// those rows, when they have left L2: c2 FP64 fetched 3.75 GB per launch, the
// forward sum 2.5 GB.)  Second come LDS reads, which took 60 % of the cycles
// with one point per lane: VX points side by side share x windows and read
// their y neighbours in 16-byte accesses.  Measured, time of one step at the
// best tile shape, queue form and this one: c2 (72x72x96, 256 states) FP64
// 887 -> 630 us (4.85 TB/s of the 3 words), complex FP32 1485 -> 642 us, c3
// (108x108x96, 640 states) FP32 2811 -> 1871 us; 45x37x50, 75 states, complex
// FP64, order 8: 184 -> 87 us.
template <typename T, typename RT, int R, int VX, int RY, int NHS>
__device__ __forceinline__ void stencil_item(const T* __restrict__ Yin, const T* __restrict__ Yprev,
                                             T* __restrict__ Yout, const RT* __restrict__ V, const KArgs<RT>& a,
                                             int tile, int zc, int64_t s, unsigned char* smem) {
  using P = Ph<T>;
  using W = Vec<T, VX>;
  using WR = Vec<RT, VX>;
  constexpr int RM = (R + VX - 1) / VX * VX;   // x margin of the staged plane: whole vectors
  constexpr int ES = (int)sizeof(T);
  const int TXv = blockDim.x, TX = TXv * VX, TYt = blockDim.y, TY = TYt * RY;
  const int SW = TX + 2 * RM, SH = TY + 2 * R;
  const int row = SW * ES;                     // bytes of a staged row
  const int bufb = SW * SH * ES + 16;          // and of a staged plane; 16 take the unused halo slots
  const int tx = threadIdx.x * VX, ty = threadIdx.y;
  const int tid = ty * TXv + threadIdx.x, nthr = TXv * TYt;
  const int bx = tile % a.tiles_x, by = tile / a.tiles_x;
  const int x0 = bx * TX, y0 = by * TY;
  const int zbeg = zc * a.tz;
  const int zend = min(zbeg + a.tz, a.n3);
  const int n1 = a.n1, n2 = a.n2, n3 = a.n3;
  // x halo from the LDS row itself when the tile spans the whole x range
  const bool xfull = (TX == n1) && (n1 >= RM);
  const unsigned pb = (unsigned)(n1 * n2) * (unsigned)ES;    // bytes of a plane
  const unsigned pv = (unsigned)(n1 * n2) * (unsigned)sizeof(RT);
  const unsigned bytes = pb * (unsigned)n3;
  const Col Yi(Yin + s * a.ld, bytes), Yo(Yout + s * a.ld_out, bytes), Vc(V, pv * (unsigned)n3);
  const Col Yp(Yprev + s * a.ld_prev, a.has_prev ? bytes : 0u);

  unsigned off[RY], oout[RY];   // byte offsets of the thread's points in a plane, to read and to write
  T phc[RY];                    // Bloch factor of points past the grid (ragged tiles; never stored)
  for (int r = 0; r < RY; ++r) {
    int wx, wy;
    const int gx = wrap(x0 + tx, n1, wx), gy = wrap(y0 + ty * RY + r, n2, wy);
    off[r] = (unsigned)(gx + n1 * gy) * (unsigned)ES;
    oout[r] = x0 + tx < n1 && y0 + ty * RY + r < n2 ? off[r] : kNone;
    if constexpr (P::on) phc[r] = P::of(wx, wy, 0, a);
  }
  const bool ragged = x0 + TX > n1 || y0 + TY > n2;   // uniform

  // halo slots owned by this thread: y halo (2R rows x TX) then, unless
  // xfull, x halo (TY rows x 2RM), in vectors; slot k is vector tid + k * nthr
  const int nyh = 2 * R * TXv, nh = nyh + (xfull ? 0 : TY * (2 * RM / VX));
  unsigned h_off[NHS];
  int h_lds[NHS];
  T h_ph[NHS];
  for (int k = 0; k < NHS; ++k) {
    const int e = tid + k * nthr;
    h_lds[k] = bufb - 16;
    h_off[k] = kNone;
    if constexpr (P::on) h_ph[k] = T(1);
    if (e >= nh) continue;
    int hr, col, wx, wy;
    if (e < nyh) {
      const int rh = e / TXv;
      col = e % TXv * VX + RM;
      hr = rh < R ? rh : TY + rh;
    } else {
      const int e2 = e - nyh;
      const int cc = e2 % (2 * RM / VX) * VX;
      hr = e2 / (2 * RM / VX) + R;
      col = cc < RM ? cc : TX + cc;
    }
    const int hx = wrap(x0 + col - RM, n1, wx), hy = wrap(y0 + hr - R, n2, wy);
    h_lds[k] = hr * row + col * ES;
    h_off[k] = (unsigned)(hx + n1 * hy) * (unsigned)ES;
    if constexpr (P::on) h_ph[k] = P::of(wx, wy, 0, a);
  }
  T phx = T(1), phxm = T(1);
  if constexpr (P::on) { phx = P::of(1, 0, 0, a); phxm = P::of(-1, 0, 0, a); }
  auto mulv = [](W v, T ph) -> W {
    if constexpr (P::on)
      for (int e = 0; e < VX; ++e) v[e] = P::mul(v[e], ph);
    return v;
  };
  // Bloch factors of freshly read tile values of a plane with z wrap count w
  // (uniform branches: inside the cell there is nothing to do)
  auto phase_tile = [&](W* v, int w) {
    if constexpr (P::on) {
      if (ragged)
        for (int r = 0; r < RY; ++r) v[r] = mulv(v[r], phc[r]);
      if (w != 0) {
        const T pz = P::of(0, 0, w, a);
        for (int r = 0; r < RY; ++r) v[r] = mulv(v[r], pz);
      }
    }
  };
  const int own = (ty * RY + R) * row + (tx + RM) * ES;   // LDS offset of the thread's first vector
  auto stage = [&](unsigned char* buf, const W* v, const W* hv) {
    for (int r = 0; r < RY; ++r) {
      unsigned char* q = buf + own + r * row;
      lds_put(q, v[r]);
      if (xfull) {
        if (tx < RM) lds_put(q + n1 * ES, mulv(v[r], phx));
        if (tx >= n1 - RM) lds_put(q - n1 * ES, mulv(v[r], phxm));
      }
    }
    for (int k = 0; k < NHS; ++k) lds_put(buf + h_lds[k], mulv(hv[k], h_ph[k]));
  };

  // A[r][e][j]: running sum of the output R - j planes below the next plane
  // (j < R: planes already read, j >= R: planes to come)
  T A[RY][VX][2 * R];
  W cur[RY], nxt[RY], hal[NHS], yp[RY];
  WR vv[RY];
  int gz, wz;   // grid plane and wrap count of the next plane to read
  auto load_tile = [&](W* v) {
    for (int r = 0; r < RY; ++r) v[r] = Yi.template get<W>(off[r], pb * (unsigned)gz);
  };
  auto load_halo = [&] {
    for (int k = 0; k < NHS; ++k) hal[k] = Yi.template get<W>(h_off[k], pb * (unsigned)gz);
  };
  auto advance = [&] {
    if (++gz == n3) { gz = 0; ++wz; }
  };
  auto load_v = [&](int z) {   // plane n3 (after the last one) reads as 0
    for (int r = 0; r < RY; ++r)
      vv[r] = Vc.template get<WR>(off[r] / (unsigned)(sizeof(T) / sizeof(RT)), pv * (unsigned)z);
  };
  // planes before the chunk: past the end (no read, no write)
  auto out_plane = [&](int z) -> unsigned { return z >= zbeg ? pb * (unsigned)z : bytes; };
  auto load_prev = [&](int z, W* v) {
    for (int r = 0; r < RY; ++r) v[r] = Yp.template get<W>(off[r], out_plane(z));
  };

  // ---- planes zbeg - R .. zbeg - 1 (tile values only), then plane zbeg
  gz = wrap(zbeg - R, n3, wz);
  {
    W bv[R][RY];
    int bw[R];
    for (int i = 0; i < R; ++i) {
      bw[i] = wz;
      load_tile(bv[i]);
      advance();
    }
    load_tile(cur);
    load_halo();
    load_v(zbeg);
    for (int i = 0; i < R; ++i) phase_tile(bv[i], bw[i]);
    for (int r = 0; r < RY; ++r)
      for (int e = 0; e < VX; ++e)
        for (int j = 0; j < 2 * R; ++j) {
          T acc = T(0);
          // output zbeg + j - R from the planes zbeg - R + i within distance R
          for (int i = 0; i < R; ++i)
            if (j >= R && j - i <= R) acc += a.kz[j - i] * bv[i][r][e];
          A[r][e][j] = acc;
        }
    phase_tile(cur, wz);
    stage(smem, cur, hal);
    advance();
  }
  for (int r = 0; r < RY; ++r)
    for (int e = 0; e < VX; ++e) yp[r][e] = T(0);
  __syncthreads();

  int boff = 0;   // the staged plane's buffer
  for (int z = zbeg; z < zend; ++z) {
    W mid[RY];
    for (int r = 0; r < RY; ++r) {
      W o;
      for (int e = 0; e < VX; ++e) {
        T* S = A[r][e];
        const T c = cur[r][e];
        // the output R planes back is complete
        o[e] = S[0] + a.kz[R] * c;
        o[e] += (-a.beta) * yp[r][e];
        for (int j = 0; j < R - 1; ++j) S[j] = S[j + 1] + a.kz[R - 1 - j] * c;
        mid[r][e] = S[R];
        for (int j = R; j < 2 * R - 1; ++j) S[j] = S[j + 1] + a.kz[j + 1 - R] * c;
        S[2 * R - 1] = a.kz[R] * c;
      }
      Yo.put(o, oout[r], out_plane(z - R));
    }
    // the next plane's tile values (planes past the chunk end still enter its
    // last R outputs) and halo, and the next output's yprev
    const int wn = wz;
    load_tile(nxt);
    load_halo();
    load_prev(z + 1 - R, yp);
    // In-plane sums, in stages of a few neighbours, the small weights first
    // and the centre last, so that the in-plane additions round at the size of
    // the neighbour sums: 36x36x24, order 12, FP32, random blocks 7.7e-8 off
    // 64 bits, smooth ones 1.1e-6 (centre first: 1.16e-7 and 1.2e-6; the same
    // times).  The offset is opaque, or every row's address would be kept in a
    // register of its own.
    int at = boff + own;
    asm volatile("" : "+v"(at));
    for (int r = 0; r < RY; ++r) {
      constexpr int NV = RM / VX;
      T w[VX + 2 * RM];
      for (int i = 0; i < 2 * NV + 1; ++i) {
        const W t = i == NV ? cur[r] : lds_get<W>(smem + at + r * row + (i - NV) * (int)sizeof(W));
        for (int e = 0; e < VX; ++e) w[i * VX + e] = t[e];
      }
      for (int e = 0; e < VX; ++e) {
        for (int p = R; p >= 1; --p) mid[r][e] += a.kx[p] * (w[RM + e + p] + w[RM + e - p]);
        pin(mid[r][e]);
      }
    }
    int up = at + R * row, dn = at - R * row;
    for (int p = R; p >= 1; --p) {
      for (int r = 0; r < RY; ++r) {
        // y neighbours inside the thread's own RY rows are at hand
        const W u = (r + p < RY) ? cur[(r + p) % RY] : lds_get<W>(smem + up + r * row);
        const W d = (r - p >= 0) ? cur[(r - p + RY) % RY] : lds_get<W>(smem + dn + r * row);
        for (int e = 0; e < VX; ++e) {
          mid[r][e] += a.ky[p] * (u[e] + d[e]);
          if (p % 2 == 1) pin(mid[r][e]);
        }
      }
      up -= row;
      dn += row;
    }
    for (int r = 0; r < RY; ++r)
      for (int e = 0; e < VX; ++e) {
        A[r][e][R - 1] = add_centre(mid[r][e], vv[r][e], cur[r][e], a);
        pin(A[r][e][R - 1]);
      }
    load_v(z + 1);
    phase_tile(nxt, wn);
    boff = bufb - boff;
    stage(smem + boff, nxt, hal);
    for (int r = 0; r < RY; ++r) cur[r] = nxt[r];
    advance();
    __syncthreads();
  }
  // ---- planes zend .. zend + R - 1 (tile values only; cur holds the first)
  // complete the outputs zend - R .. zend - 1
  {
    W tv[R][RY], pr[R][RY];
    int tw[R];
    for (int r = 0; r < RY; ++r) {
      tv[0][r] = cur[r];
      pr[0][r] = yp[r];
    }
    for (int i = 1; i < R; ++i) {
      tw[i] = wz;
      load_tile(tv[i]);
      load_prev(zend - R + i, pr[i]);
      advance();
    }
    for (int i = 1; i < R; ++i) phase_tile(tv[i], tw[i]);
    for (int i = 0; i < R; ++i)
      for (int r = 0; r < RY; ++r) {
        W o;
        for (int e = 0; e < VX; ++e) {
          T acc = A[r][e][i];
          for (int m = 0; m <= i; ++m) acc += a.kz[R - i + m] * tv[m][r][e];
          o[e] = acc + (-a.beta) * pr[i][r][e];
        }
        Yo.put(o, oout[r], out_plane(zend - R + i));
      }
  }
}

// The same work item for real points without vectors (rows of odd length, or
// one point per thread): the 2R + 1 z neighbours of a thread's points wait in
// a register queue and one pass over the plane forms the sum.  Without vectors
// the forward sum's LDS reads are one point each as well, and its second pass
// over them costs more than the halo rows it finds in L2: 63x63x41, 192
// states, order 12, 132 us (FP32) and 219 us (FP64) in the queue, 268 and 401
// forwards; with vectors (64x62x40, order 8) 75 and 151 us forwards, 111 and
// 206 in the queue.
//
// FP32 tiles of odd checkerboard parity sweep their z range R planes behind
// the even ones (periodic in z), so that their own reads of a plane coincide
// with the neighbours' halo reads of it (9 % fewer bytes fetched).
template <typename T, int R, int RY, int NHS>
__device__ __forceinline__ void queue_item(const T* __restrict__ Yin, const T* __restrict__ Yprev, T* __restrict__ Yout,
                                           const T* __restrict__ V, const KArgs<T>& a, int tile, int zc, int64_t s,
                                           unsigned char* smem_raw) {
  using GC = const __attribute__((address_space(1))) T*;
  using GT = __attribute__((address_space(1))) T*;
  const int TX = blockDim.x, TYt = blockDim.y, TY = TYt * RY;
  const int SW = TX + 2 * R, SH = TY + 2 * R;
  T* const buf0 = reinterpret_cast<T*>(smem_raw);
  T* const buf1 = buf0 + SW * SH;
  const int tx = threadIdx.x, ty = threadIdx.y;
  const int tid = ty * TX + tx, nthr = TX * TYt;
  const int bx = tile % a.tiles_x, by = tile / a.tiles_x;
  const int x0 = bx * TX, y0 = by * TY;
  const int zbeg = zc * a.tz, zend = min(zbeg + a.tz, a.n3);
  const int n1 = a.n1, n2 = a.n2, n3 = a.n3;
  const int zsh = (sizeof(T) == 4 && ((bx + by) & 1) && n3 > R) ? n3 - R : 0;
  const GC Ys = (GC)(Yin + s * a.ld), Yp = (GC)(a.has_prev ? Yprev + s * a.ld_prev : Yin + s * a.ld), Vg = (GC)V;
  const GT Yo = (GT)(Yout + s * a.ld_out);
  const int64_t plane = (int64_t)n1 * n2;
  const bool xfull = (TX == n1) && (n1 >= R);   // x halo from the staged row itself
  int w;
  const int gx = wrap(x0 + tx, n1, w);
  int gy[RY];
  for (int r = 0; r < RY; ++r) gy[r] = wrap(y0 + ty * RY + r, n2, w);
  // halo values of this thread: y halo (2R rows x TX) then, unless xfull, x
  // halo (TY rows x 2R); unused slots read node 0 and stage nothing
  const int nyh = 2 * R * TX, nh = nyh + (xfull ? 0 : TY * 2 * R);
  int h_xy[NHS], h_lds[NHS];
  for (int k = 0; k < NHS; ++k) {
    const int e = tid + k * nthr;
    h_lds[k] = -1;
    h_xy[k] = 0;
    if (e >= nh) continue;
    int row, col;
    if (e < nyh) {
      const int rh = e / TX;
      col = e % TX + R;
      row = rh < R ? rh : TY + rh;
    } else {
      const int e2 = e - nyh, cc = e2 % (2 * R);
      row = e2 / (2 * R) + R;
      col = cc < R ? cc : TX + cc;
    }
    h_lds[k] = row * SW + col;
    h_xy[k] = wrap(x0 + col - R, n1, w) + n1 * wrap(y0 + row - R, n2, w);
  }
  T q[RY][2 * R + 1];
  for (int dz = -R; dz <= R; ++dz) {
    const int gz = wrap(zbeg + zsh + dz, n3, w);
    for (int r = 0; r < RY; ++r) q[r][dz + R] = Ys[gx + (int64_t)n1 * gy[r] + plane * gz];
  }
  auto stage = [&](T* buf, const T* hreg) {
    for (int r = 0; r < RY; ++r) {
      const int row = ty * RY + r + R;
      const T v = q[r][R];
      buf[row * SW + tx + R] = v;
      if (xfull) {
        if (tx < R) buf[row * SW + tx + n1 + R] = v;
        if (tx >= n1 - R) buf[row * SW + tx - n1 + R] = v;
      }
    }
    for (int k = 0; k < NHS; ++k)
      if (h_lds[k] >= 0) buf[h_lds[k]] = hreg[k];
  };
  T hreg[NHS];
  {
    const int gz = wrap(zbeg + zsh, n3, w);
    for (int k = 0; k < NHS; ++k) hreg[k] = Ys[h_xy[k] + plane * gz];
    stage(buf0, hreg);
  }
  __syncthreads();
  int cur = 0;
  for (int z = zbeg; z < zend; ++z) {
    const bool more = z + 1 < zend;
    T qn[RY];   // the next plane's queue head and halo, this plane's V and yprev
    if (more) {
      const int gz = wrap(z + 1 + R + zsh, n3, w), zh = wrap(z + 1 + zsh, n3, w);
      for (int r = 0; r < RY; ++r) qn[r] = Ys[gx + (int64_t)n1 * gy[r] + plane * gz];
      for (int k = 0; k < NHS; ++k) hreg[k] = Ys[h_xy[k] + plane * zh];
    }
    const int64_t zoff = plane * (z + zsh - (z + zsh >= n3 ? n3 : 0));
    T vv[RY], yp[RY];
    for (int r = 0; r < RY; ++r) {
      const int64_t p = gx + (int64_t)n1 * gy[r] + zoff;
      vv[r] = Vg[p];
      yp[r] = T(0);
      if (a.has_prev) yp[r] = Yp[p];
    }
    const T* B = cur ? buf1 : buf0;
    for (int r = 0; r < RY; ++r) {
      const T* L = B + (ty * RY + r + R) * SW + tx + R;
      T acc = T(0);
      for (int p = 1; p <= R; ++p) {
        acc += a.kx[p] * (L[p] + L[-p]);
        // y neighbours inside the thread's own rows come from the queue
        const T up = (r + p < RY) ? q[(r + p) % RY][R] : L[p * SW];
        const T dn = (r - p >= 0) ? q[(r - p + RY) % RY][R] : L[-p * SW];
        acc += a.ky[p] * (up + dn);
        acc += a.kz[p] * (q[r][R + p] + q[r][R - p]);
      }
      if ((x0 + tx < n1) && (y0 + ty * RY + r < n2)) {
        acc = add_centre(acc, vv[r], q[r][R], a);
        if (a.has_prev) acc += (-a.beta) * yp[r];
        Yo[gx + (int64_t)n1 * gy[r] + zoff] = acc;
      }
    }
    for (int r = 0; r < RY; ++r) {
      for (int t = 0; t < 2 * R; ++t) q[r][t] = q[r][t + 1];
      if (more) q[r][2 * R] = qn[r];
    }
    if (more) stage(cur ? buf0 : buf1, hreg);
    __syncthreads();
    cur ^= 1;
  }
}

template <typename T, typename RT, int R, int VX, int RY, int NHS>
__device__ __forceinline__ void run_item(const T* __restrict__ Yin, const T* __restrict__ Yprev, T* __restrict__ Yout,
                                         const RT* __restrict__ V, const KArgs<RT>& a, int tile, int zc, int64_t s,
                                         unsigned char* smem_raw) {
  if constexpr (kQueue<T, VX>) queue_item<T, R, RY, NHS>(Yin, Yprev, Yout, V, a, tile, zc, s, smem_raw);
  else stencil_item<T, RT, R, VX, RY, NHS>(Yin, Yprev, Yout, V, a, tile, zc, s, smem_raw);
}

template <typename T, typename RT, int R, int VX, int RY, int NHS>
__global__ __launch_bounds__((kStencilThreads<T, RT, VX * RY>))
__attribute__((amdgpu_waves_per_eu(kWaves<T, VX, RY>))) void k_stencil(const T* __restrict__ Yin,
                                                                          const T* __restrict__ Yprev,
                                                                          T* __restrict__ Yout,
                                                                          const RT* __restrict__ V,
                                                                          const KArgs<RT> a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  // logical order: tile fastest, then z chunk, then state; XCD-contiguous
  const unsigned lw = xcd_linear();
  const int tile = lw % gridDim.x;
  const int zc = (lw / gridDim.x) % gridDim.y;
  const int64_t s = lw / (gridDim.x * gridDim.y);
  run_item<T, RT, R, VX, RY, NHS>(Yin, Yprev, Yout, V, a, tile, zc, s, smem_raw);
}

// Form over a list of jobs (blocks of possibly different grids): one workgroup
// per work item (job, tile, z chunk, state), XCD-contiguous item order, the
// job found by bisection on the items' start indices; the hardware dispatcher
// balances.  first: the launch's first item (run_stencil_batch).
template <typename T, typename RT, int R, int VX, int RY, int NHS>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(kWaves<T, VX, RY>))) void k_stencil_multi(const SJob<RT>* __restrict__ jobs, int njobs,
                                                                    unsigned long long first) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const unsigned long long item = first + xcd_linear();
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (jobs[mid].item_begin <= item) lo = mid; else hi = mid - 1;
  }
  const int j = __builtin_amdgcn_readfirstlane(lo);
  const SJob<RT>& jb = jobs[j];
  const unsigned long long loc = item - jb.item_begin;
  const int tile = (int)(loc % jb.ntiles);
  const int zc = (int)((loc / jb.ntiles) % jb.nzc);
  const int64_t s = (int64_t)(loc / ((unsigned long long)jb.ntiles * jb.nzc));
  run_item<T, RT, R, VX, RY, NHS>((const T*)jb.Yin, (const T*)jb.Yprev, (T*)jb.Yout, jb.V, jb.a, tile, zc, s, smem_raw);
}

// Tile shape for a grid: TX threads along x, TYt thread rows, RY points per
// thread along y, tz planes per workgroup.  Tuned values (hcu_autotune) win.
struct StencilShape { int TX, TYt, RY, tz, ring = 0, vx = 1; };

// shapes above 512 threads: the light real variants (kStencilThreads)
static bool big_ok(const Ctx& c, int RY) {
  if (c.any_complex) return false;
  return c.mixed ? RY <= 2 : RY == 1;
}

// LDS of a workgroup: two staged planes with halo (x margin in whole
// vectors) and 16 spare bytes each
static size_t stencil_lds(int TX, int TYt, int RY, int R, size_t elem, int vx) {
  const int RM = (R + vx - 1) / vx * vx;
  return 2 * ((size_t)(TYt * RY + 2 * R) * (TX + 2 * RM) * elem + 16);
}
constexpr size_t kLdsPerWorkgroup = 160 * 1024;

static bool shape_ok(const Ctx& c, const StencilShape& sh, int R) {
  const int n1 = c.p.n[0], n2 = c.p.n[1];
  if (sh.TX < 1 || sh.TX > n1 || sh.TYt < 1 || sh.TX * sh.TYt > 1024) return false;
  if (sh.TX * sh.TYt > 512 && !big_ok(c, sh.RY)) return false;
  if (sh.RY != 1 && sh.RY != 2 && sh.RY != 4) return false;
  const int TY = sh.TYt * sh.RY;
  if (TY > n2) return false;
  if (halo_slots(n1, sh.TX, sh.TYt, TY, R) > kHaloSlots) return false;
  if (sh.ring) {   // the flag keeps its limits: order 12, 4 halo slots, 512 threads, R planes of halo in LDS
    if (sh.ring != 1 || R != kRingR || sh.TX * sh.TYt > 512) return false;
    if (halo_slots(n1, sh.TX, sh.TYt, TY, R) > kHaloSlotsSmall) return false;
    const size_t elem = c.any_complex ? (c.mixed ? 8 : 16) : (c.mixed ? 4 : 8);
    const size_t ring = (size_t)R * halo_values(n1, sh.TX, TY, R) * elem;
    if (stencil_lds(sh.TX, sh.TYt, sh.RY, R, elem, 1) + ring > kLdsPerWorkgroup) return false;
  }
  return sh.tz >= 1;
}

#if HCU_STENCIL_ELEM == 0
bool stencil_shape_ok(const Ctx& c, int TX, int TYt, int RY, int tz, int ring) {
  return shape_ok(c, StencilShape{TX, TYt, RY, tz, ring}, c.p.n0);
}
#endif

// Built-in shape, for ncol columns in one launch.  Whole rows of up to 128
// points, about 256 threads.  A tile re-reads 2R of its TY + 2R rows and R
// planes at either end of its z range, so many points per thread and whole z
// ranges are best as long as the launch fills the chip (c2, 256 states, FP64:
// 72 x 12 tiles over 96 planes 630 us, over 48 planes 712 us, 72 x 6 tiles
// 653 us); below two workgroups per CU it is split: shorter tiles first, then
// z until there are three per CU (c1, 32 states: 10.3 us with 768 workgroups
// of 3 planes, 34 us with 128 of 12).  Sixteen-byte values take one point per
// thread (their sums fill the registers), complex rows without whole vectors
// two.  Real points without vectors have their own rule (the queue form).
// Measured over 21 odd grids of 49 to 151 points, orders 2 to 12, FP32 and FP64,
// 8 to 300 states: 0.86 of the time of four points, whole rows of 256 threads
// and at least 2048 workgroups of 16 planes, at most 1.13.
static constexpr bool vectors_built(int R) { return R == 4 || R == kMaxR; }

static StencilShape pick_tiles(const Ctx& c, int64_t ncol, int elem) {
  const int n1 = c.p.n[0], n2 = c.p.n[1], n3 = c.p.n[2];
  const int R = c.p.n0;
  StencilShape sh{c.tile_x, c.tile_yt, c.ry, c.tile_z, c.halo_ring};
  // (a tuned shape is one of the block's type; Lanczos vectors may be wider)
  const bool own = elem == (c.mixed ? 4 : 8) * (c.any_complex ? 2 : 1);
  if (own && sh.TX > 0 && shape_ok(c, sh, R)) return sh;
  sh.ring = 0;
  sh.TX = n1 <= 128 ? n1 : 64;
  auto tiles = [&] {
    const int TY = sh.TYt * sh.RY;
    return (int64_t)((n1 + sh.TX - 1) / sh.TX) * ((n2 + TY - 1) / TY);
  };
  const bool vectors = vectors_built(R) && n1 % 2 == 0 && sh.TX % 2 == 0, queue = !vectors && !c.any_complex;
  auto set_rows = [&](int ry) {
    sh.RY = ry;
    while (sh.RY > 1 && sh.RY > n2) sh.RY /= 2;
    sh.TYt = std::max(1, std::min(256 / sh.TX, n2 / sh.RY));
    // few rows on a narrow grid: single rows keep enough threads for the halo
    if (halo_slots(n1, sh.TX, sh.TYt, sh.TYt * sh.RY, R) > kHaloSlots) {
      sh.RY = 1;
      sh.TYt = std::max(1, std::min(256 / sh.TX, n2));
    }
  };
  // halves in z until the launch has `want` workgroups, as long as chunks keep
  // `planes` planes; the number of workgroups
  auto split_z = [&](int64_t want, int planes) {
    int zs = 1;
    while (tiles() * ncol * zs < want && n3 / (2 * zs) >= planes) zs *= 2;
    sh.tz = (n3 + zs - 1) / zs;
    return tiles() * ncol * zs;
  };
  int64_t wgs = 0;
  if (queue) {
    // The queue's chunks read 2R planes more than their own, but eight
    // workgroups per CU are worth that down to 16 planes (75x75x60, 200 states,
    // FP32 order 12: 339 us whole, 292 in halves).  FP64 from order 8 on takes
    // two points (63x63x41, 192 states, order 12: 4 points 244 us, 2 points
    // 219), the shorter queues four (order 6: 202 us with 2, 192 with 4).
    set_rows(elem == 8 && R >= 4 ? 2 : 4);
    // Two rows of threads that leave a fifth of their waves' lanes idle give
    // way to 512 threads in a launch that fills the chip (99x99x85, 304 states,
    // order 12: FP32 1298 -> 919 us, FP64 2448 -> 1795).
    const int rows = 512 / sh.TX;
    if (sh.TX > 64 && sh.TYt <= 2 && 5 * sh.TX * sh.TYt < 4 * 64 * ((sh.TX * sh.TYt + 63) / 64) &&
        tiles() * ncol >= 2048 && rows * sh.RY <= n2)
      sh.TYt = rows;
    wgs = split_z(2048, 16);
  } else {
    // FP32 keeps four points, with no more rows of threads than its tiles
    // need, and z is split first, down to six planes (order 12: 60x60x40, 96
    // states, two points and whole z ranges 65 us, four points and halves 44;
    // 50x46x33, 160 states, tiles of 20 rows 64 us, of 16 rows 55).
    set_rows(elem > 8 ? 1 : vectors ? 4 : 2);
    if (elem == 4) {
      const int TY = sh.TYt * sh.RY, ny = (n2 + TY - 1) / TY;
      sh.TYt = (n2 + ny * sh.RY - 1) / (ny * sh.RY);
    }
    wgs = split_z(elem == 4 ? 768 : 0, 6);
  }
  if (wgs < (queue ? 384 : 512)) {
    if (sh.RY > 2) set_rows(2);
    split_z(768, 3);
  }
  while (!shape_ok(c, sh, R) && sh.TYt > 1) --sh.TYt;
  return sh;
}

// workgroups above 64 KB of LDS ask for it (gfx950 has 160 KB per CU)
template <typename K>
static void allow_lds(K kernel, size_t lds) {
  if (lds > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

// The points of a thread (PT of them, a shape's ry) lie side by side in x
// where the rows allow whole vectors, else stacked in y.  One vector access
// then moves up to 16 bytes of LDS and memory per lane, and the x neighbours
// of a vector overlap.  Built for the orders 8 and 12.
template <typename T>
static int vector_points(int R, int PT, int n1, int TX) {
  if (!vectors_built(R)) return 1;
  int vx = std::min(PT, (int)(16 / sizeof(T)));
  while (n1 % vx || TX % vx) vx /= 2;
  return vx;
}

// f(points per vector, rows of vectors per thread, few halo slots) as
// constants, for nh halo vectors per thread and plane
template <typename T, int R, typename F>
static void for_variant(int PT, int vx, int nh, F f) {
  auto slots = [&](auto v, auto ry) {
    if (nh <= kSlots<decltype(v)::value, true>) f(v, ry, std::true_type());
    else f(v, ry, std::false_type());
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I4 = std::integral_constant<int, 4>;
  if constexpr (vectors_built(R) && sizeof(T) <= 8) {
    if (vx == 2) return PT == 4 ? slots(I2(), I2()) : slots(I2(), I1());
    if constexpr (sizeof(T) == 4)
      if (vx == 4) return slots(I4(), I1());
  }
  if (PT == 4) slots(I1(), I4());
  else if (PT == 2) slots(I1(), I2());
  else slots(I1(), I1());
}

template <typename RT>
static KArgs<RT> stencil_args(const Ctx& c, int ik, double alpha, double cshift, double beta, bool prev) {
  StencilCoef sc;
  fill_stencil_coef(c, ik, sc);
  KArgs<RT> a{};
  // The weights cancel on smooth functions, so their rounding would shift the
  // whole spectrum: the centre takes the opposite of the neighbours' roundings
  // and keeps its own in a second word.
  double centre = alpha * (sc.center - cshift);
  auto weight = [&](double w, bool neighbour) {
    const RT r = (RT)(alpha * w);
    if (neighbour) centre += 2.0 * (alpha * w - (double)r);
    return r;
  };
  for (int p = 0; p <= kMaxR; ++p) {
    const bool nb = p >= 1 && p <= c.p.n0;
    a.kx[p] = weight(sc.kin[0][p], nb);
    a.ky[p] = weight(sc.kin[1][p], nb);
    a.kz[p] = weight(sc.kin[2][p], nb);
  }
  a.center = (RT)centre;
  a.center_lo = (RT)(centre - (double)a.center);
  a.alpha = (RT)alpha;
  a.beta = (RT)beta;
  for (int d = 0; d < 3; ++d) { a.ph_re[d] = (RT)sc.phase_re[d]; a.ph_im[d] = (RT)sc.phase_im[d]; }
  a.n1 = c.p.n[0]; a.n2 = c.p.n[1]; a.n3 = c.p.n[2];
  a.has_prev = (prev && beta != 0.0) ? 1 : 0;
  return a;
}

template <typename T, typename RT, int R>
static void launch_r(int RY, int vx, int nh, const KArgs<RT>& a, dim3 grid, dim3 block, size_t lds, const T* Yin,
                     const T* Yprev, T* Yout, const RT* V, hipStream_t st) {
  auto go = [&](auto kernel) {
    allow_lds(kernel, lds);
    launch_k(kernel, grid, block, lds, st, Yin, Yprev, Yout, V, a);
  };
  for_variant<T, R>(RY, vx, nh, [&](auto v, auto ry, auto small) {
    constexpr int VX = decltype(v)::value, NR = decltype(ry)::value;
    go(k_stencil<T, RT, R, VX, NR, kSlots<VX, decltype(small)::value>>);
  });
}

template <typename T>
void launch_stencil(const Ctx& c, int ik, const T* Yin, int64_t ld, const T* Yprev, int64_t ld_prev, T* Yout,
                    int64_t ld_out, int ncol, double alpha, double cshift, double beta, hipStream_t st) {
  using RT = typename real_of<T>::type;
  KArgs<RT> a = stencil_args<RT>(c, ik, alpha, cshift, beta, Yprev != nullptr);
  a.ld = ld;
  a.ld_prev = ld_prev;
  a.ld_out = ld_out;
  const StencilShape sh = pick_tiles(c, ncol, (int)sizeof(T));
  const int TX = sh.TX, TYt = sh.TYt, tz = sh.tz;
  const int TY = TYt * sh.RY;
  a.tiles_x = (a.n1 + TX - 1) / TX;
  a.tz = tz;
  dim3 grid(a.tiles_x * ((a.n2 + TY - 1) / TY), (a.n3 + tz - 1) / tz, ncol);
  const int R = c.p.n0;
  const int vx = vector_points<T>(R, sh.RY, a.n1, TX);
  dim3 block(TX / vx, TYt * vx);
  const size_t lds = stencil_lds(TX, TYt, sh.RY, R, sizeof(T), vx);
  const int nh = halo_vectors(a.n1, TX, TYt, TY, R, vx);
  const RT* V;
  if constexpr (sizeof(RT) == 4) V = c.d_Vf; else V = c.d_V;
  switch (R) {
    case 1: launch_r<T, RT, 1>(sh.RY, vx, nh, a, grid, block, lds, Yin, Yprev, Yout, V, st); break;
    case 2: launch_r<T, RT, 2>(sh.RY, vx, nh, a, grid, block, lds, Yin, Yprev, Yout, V, st); break;
    case 3: launch_r<T, RT, 3>(sh.RY, vx, nh, a, grid, block, lds, Yin, Yprev, Yout, V, st); break;
    case 4: launch_r<T, RT, 4>(sh.RY, vx, nh, a, grid, block, lds, Yin, Yprev, Yout, V, st); break;
    case 5: launch_r<T, RT, 5>(sh.RY, vx, nh, a, grid, block, lds, Yin, Yprev, Yout, V, st); break;
    default: launch_r<T, RT, 6>(sh.RY, vx, nh, a, grid, block, lds, Yin, Yprev, Yout, V, st); break;
  }
}

// Work items of one launch: a grid has fewer than 2^32 threads in x, and a
// batch may have more items than that (small tuned tiles of single planes).  A
// million workgroups keep the device busy for milliseconds, so a further
// launch costs nothing.
constexpr unsigned long long kLaunchItems = 1 << 20;

template <typename T, typename RT, int R>
static void launch_batch_r(int RY, int vx, int nh, unsigned long long items, dim3 block, size_t lds,
                           const SJob<RT>* jobs, int njobs, hipStream_t st) {
  for_variant<T, R>(RY, vx, nh, [&](auto v, auto ry, auto small) {
    constexpr int VX = decltype(v)::value, NR = decltype(ry)::value;
    constexpr auto kernel = k_stencil_multi<T, RT, R, VX, NR, kSlots<VX, decltype(small)::value>>;
    allow_lds(kernel, lds);
    for (unsigned long long i = 0; i < items; i += kLaunchItems)
      launch_k(kernel, dim3((unsigned)std::min(items - i, kLaunchItems)), block, lds, st, jobs, njobs, i);
  });
}

// Common tile shape for a set of grids: the autotuned shape of the first
// context if every grid admits it, else the largest admissible built-in one.
static bool batch_shape(const std::vector<const Ctx*>& cs, int64_t ncol, int elem, int& TX, int& TYt, int& RY, int* TZ) {
  const Ctx& c0 = *cs[0];
  StencilShape sh = pick_tiles(c0, ncol, elem);
  auto ok_all = [&](const StencilShape& t) {
    if (t.TX * t.TYt > 512) return false;   // the kernel over jobs is built for 512 threads
    for (const Ctx* c : cs)
      if (!shape_ok(*c, StencilShape{t.TX, t.TYt, t.RY, 1, t.ring}, c->p.n0)) return false;
    return true;
  };
  if (!ok_all(sh)) {
    int n1min = 1 << 30, n2min = 1 << 30;
    for (const Ctx* c : cs) { n1min = std::min(n1min, c->p.n[0]); n2min = std::min(n2min, c->p.n[1]); }
    bool found = false;
    for (int ry : {elem > 8 ? 2 : 4, 2, 1}) {
      for (int tx : {std::min(n1min, 128), 64, 32, 16}) {
        if (tx > n1min) continue;
        for (int tyt = std::max(1, 256 / tx); tyt >= 1 && !found; --tyt) {
          StencilShape t{tx, tyt, ry, 1};
          if (tyt * ry <= n2min && ok_all(t)) { sh = t; found = true; }
        }
        if (found) break;
      }
      if (found) break;
    }
    if (!found) return false;
  }
  TX = sh.TX; TYt = sh.TYt; RY = sh.RY;
  if (TZ) *TZ = sh.tz;
  return true;
}

// One stencil step for many blocks: the blocks are grouped by the tile shape
// their own grid prefers (tuned or built-in, at most 512 threads, the job's
// own z chunk), each group becoming one launch.
template <typename T>
hcu_status plan_stencil_batch(const std::vector<StencilJob>& jobs, std::vector<unsigned char>& host,
                              std::vector<BatchLaunch>& out) {
  using RT = typename real_of<T>::type;
  if (jobs.empty()) return HCU_OK;
  const int R = jobs[0].c->p.n0;
  for (const StencilJob& j : jobs)
    if (j.c->p.n0 != R) return HCU_INVALID_ARG;
  int64_t cols = 0;   // all blocks share the launch
  for (const StencilJob& j : jobs) cols += j.ncol;
  std::vector<StencilShape> shp(jobs.size());
  std::vector<int> gid(jobs.size());
  std::vector<StencilShape> groups;
  for (size_t i = 0; i < jobs.size(); ++i) {
    int TX, TYt, RY, TZ = 0;
    std::vector<const Ctx*> one{jobs[i].c};
    if (!batch_shape(one, cols, (int)sizeof(T), TX, TYt, RY, &TZ)) return HCU_INVALID_ARG;
    shp[i] = StencilShape{TX, TYt, RY, TZ, 0, vector_points<T>(R, RY, jobs[i].c->p.n[0], TX)};
    int g = -1;
    for (size_t k = 0; k < groups.size(); ++k)
      if (groups[k].TX == TX && groups[k].TYt == TYt && groups[k].RY == RY && groups[k].vx == shp[i].vx) g = (int)k;
    if (g < 0) {
      g = (int)groups.size();
      groups.push_back(shp[i]);
    }
    gid[i] = g;
  }
  size_t slot = host.size() / sizeof(SJob<RT>);
  host.resize(host.size() + jobs.size() * sizeof(SJob<RT>), 0);
  SJob<RT>* hj = reinterpret_cast<SJob<RT>*>(host.data());
  for (size_t g = 0; g < groups.size(); ++g) {
    const int TX = groups[g].TX, TYt = groups[g].TYt, RY = groups[g].RY;
    const int TY = TYt * RY;
    BatchLaunch L{slot, 0, 0, TX, TYt, RY, R, groups[g].vx, 0};
    for (size_t i = 0; i < jobs.size(); ++i) {
      if (gid[i] != (int)g) continue;
      const StencilJob& j = jobs[i];
      const Ctx& c = *j.c;
      L.halo_slots = std::max(L.halo_slots, halo_vectors(c.p.n[0], TX, TYt, TY, R, L.vx));
      KArgs<RT> a = stencil_args<RT>(c, j.ik, j.alpha, j.cshift, j.beta, j.Yprev != nullptr);
      a.ld = j.ld; a.ld_prev = j.ld_prev; a.ld_out = j.ld_out;
      a.tiles_x = (a.n1 + TX - 1) / TX;
      const int tiles = a.tiles_x * ((a.n2 + TY - 1) / TY);
      // the job's own z chunk (tuned or built-in); the fallback shape has none
      a.tz = shp[i].tz > 1 ? std::min(a.n3, shp[i].tz) : std::max(8, std::min(a.n3, 24));
      const int nzc = (a.n3 + a.tz - 1) / a.tz;
      SJob<RT>& h = hj[slot++];
      h.Yin = j.Yin; h.Yprev = j.Yprev; h.Yout = j.Yout;
      if constexpr (sizeof(RT) == 4) h.V = c.d_Vf; else h.V = c.d_V;
      h.a = a;
      h.ntiles = tiles;
      h.nzc = nzc;
      h.item_begin = L.total;
      L.total += (unsigned long long)tiles * nzc * j.ncol;
      ++L.njob;
    }
    out.push_back(L);
  }
  return HCU_OK;
}

template <typename T>
hcu_status run_stencil_batch(const BatchLaunch& L, const void* d_jobs, hipStream_t st) {
  using RT = typename real_of<T>::type;
  const size_t lds = stencil_lds(L.TX, L.TYt, L.RY, L.R, sizeof(T), L.vx);
  const dim3 block(L.TX / L.vx, L.TYt * L.vx);
  const unsigned long long n = L.total;
  const SJob<RT>* dj = reinterpret_cast<const SJob<RT>*>(d_jobs) + L.first;
  switch (L.R) {
    case 1: launch_batch_r<T, RT, 1>(L.RY, L.vx, L.halo_slots, n, block, lds, dj, L.njob, st); break;
    case 2: launch_batch_r<T, RT, 2>(L.RY, L.vx, L.halo_slots, n, block, lds, dj, L.njob, st); break;
    case 3: launch_batch_r<T, RT, 3>(L.RY, L.vx, L.halo_slots, n, block, lds, dj, L.njob, st); break;
    case 4: launch_batch_r<T, RT, 4>(L.RY, L.vx, L.halo_slots, n, block, lds, dj, L.njob, st); break;
    case 5: launch_batch_r<T, RT, 5>(L.RY, L.vx, L.halo_slots, n, block, lds, dj, L.njob, st); break;
    default: launch_batch_r<T, RT, 6>(L.RY, L.vx, L.halo_slots, n, block, lds, dj, L.njob, st); break;
  }
  return hipGetLastError() == hipSuccess ? HCU_OK : HCU_DEVICE;
}

#define INST_STENCIL(T)                                                                                 \
  template void launch_stencil<T>(const Ctx&, int, const T*, int64_t, const T*, int64_t, T*, int64_t, int, \
                                  double, double, double, hipStream_t);                                \
  template hcu_status plan_stencil_batch<T>(const std::vector<StencilJob>&, std::vector<unsigned char>&,   \
                                            std::vector<BatchLaunch>&);                                    \
  template hcu_status run_stencil_batch<T>(const BatchLaunch&, const void*, hipStream_t);
// built once per element type (HCU_STENCIL_ELEM), so the units compile side by side
#if HCU_STENCIL_ELEM == 0
INST_STENCIL(double)
#elif HCU_STENCIL_ELEM == 1
INST_STENCIL(float)
#elif HCU_STENCIL_ELEM == 2
INST_STENCIL(cplx<double>)
#else
INST_STENCIL(cplx<float>)
#endif

}  // namespace hcu
