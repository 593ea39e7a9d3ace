// gea_cgp.hip -- a whole Jacobi-PCG solve of a 2D system in one launch.
//
// A workgroup keeps its tile of the solve's vectors on the chip (registers,
// and LDS where the registers do not hold them) from the first iteration to
// the last, so an iteration moves no vector through memory.  The iterates are
// those of the iteration kernels in gea_cg.hip (same formulas, contractions
// and order of the operator's terms).  What is exchanged each iteration:
//  - the seven partial sums of the dot products, all workgroups to all;
//  - A p on the tile's border, to the four neighbours, which carry the
//    residual and direction of that one-cell halo along and update them as
//    the owner does.  So one exchange an iteration is enough.
// Every exchanged 32-bit half travels in a 64-bit word with the iteration's
// tag: a reader polls the word itself, and neither fences nor flags order
// anything (relaxed agent-scope accesses, which reach the other XCDs).  Words
// are double buffered by iteration parity: a workgroup writes parity
// j of iteration j + 2 only after it has read every workgroup's sums of
// j + 1, which each of them wrote after its last read of j.
//
// All workgroups of a launch must be on the card at once: the plan admits no
// more than the occupancy query allows, and a wait that outlasts its limit
// (another kernel holds the CUs) ends the launch with status kCgpAborted, on
// which the host takes the kernels of gea_cg.hip.
//
// What bounds it: on small meshes the exchange (store, then load, past the
// L2s: about 3 us an iteration up to 50 workgroups, 5 us at 250), on large
// ones the FP64 sums and the stencil on the vector units.  One iteration
// (with its share of the solve's set-up), us, one launch an iteration
// before / now: 64 x 32 FP64 25 / 4.5 (one workgroup, 2.4 without the set-up),
// 200 x 200 FP64 15.7 / 4.1, 333 x 251 15.9 / 4.4, 1024 x 1024 26.8 / 6.5,
// 2048 x 2048 FP32 33 / 11.4 (its 11 arrays a cell came from the last-level
// cache at 5.8 TB/s).  A workgroup's sums are one 128-byte line, read by
// coalesced loads of four: as 14 rows of one word a workgroup, which all
// workgroups polled at once, 1024 x 1024 took 11.5 us.  The registers decide
// how many rows a thread can hold (R = 32 in FP32 at two waves a SIMD): the
// face weights are formed anew from D each iteration, 2 R registers less
// than holding them.
#include "gea_reduce.h"

namespace gea {

namespace {

__device__ __forceinline__ uint64_t word_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void word_store(uint64_t* p, uint32_t tag, uint32_t half) {
  __hip_atomic_store(p, ((uint64_t)tag << 32) | half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the value of the lane below (above) in the wave; lane 0 (63) takes `edge`
__device__ __forceinline__ uint32_t lane_below(uint32_t edge, uint32_t v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t lane_above(uint32_t edge, uint32_t v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x130 /* wave_shl:1 */, 0xf, 0xf, false);
}
template <bool ABOVE>
__device__ __forceinline__ float lane_next(float edge, float v) {
  const uint32_t e = __float_as_uint(edge), a = __float_as_uint(v);
  return __uint_as_float(ABOVE ? lane_above(e, a) : lane_below(e, a));
}
template <bool ABOVE>
__device__ __forceinline__ double lane_next(double edge, double v) {
  const uint64_t e = __double_as_longlong(edge), a = __double_as_longlong(v);
  const uint32_t lo = ABOVE ? lane_above((uint32_t)e, (uint32_t)a) : lane_below((uint32_t)e, (uint32_t)a);
  const uint32_t hi = ABOVE ? lane_above((uint32_t)(e >> 32), (uint32_t)(a >> 32))
                            : lane_below((uint32_t)(e >> 32), (uint32_t)(a >> 32));
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ uint32_t half_of(float v, int) { return __float_as_uint(v); }
__device__ __forceinline__ uint32_t half_of(double v, int h) {
  return (uint32_t)(__double_as_longlong(v) >> (32 * h));
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

__device__ __forceinline__ double join(uint32_t lo, uint32_t hi) {
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
// lane ^ 8, ^ 2, ^ 1 within the wave by data-parallel primitives (CTRL)
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint32_t lo = half_of(v, 0), hi = half_of(v, 1);
  return join(__builtin_amdgcn_update_dpp(0u, lo, CTRL, 0xf, 0xf, false),
              __builtin_amdgcn_update_dpp(0u, hi, CTRL, 0xf, 0xf, false));
}
// a of lanes l and l ^ 32 (16) added in the lanes whose bit is clear, b in the
// others
template <int BIT>
__device__ __forceinline__ double halve(double a, double b) {
  const uint32_t al = half_of(a, 0), ah = half_of(a, 1), bl = half_of(b, 0), bh = half_of(b, 1);
  if constexpr (BIT == 32) {
    const auto lo = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return join(lo[0], hi[0]) + join(lo[1], hi[1]);
  } else {
    const auto lo = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return join(lo[0], hi[0]) + join(lo[1], hi[1]);
  }
}
// The sums over the wave of eight values, value l / 8 in lane l: each of the
// first three stages halves the values a lane holds.  No LDS, and the pairing
// and order of wave_sum.
__device__ __forceinline__ double wave_sum8(const double (&v)[8]) {
  const int lane = threadIdx.x & 63;
  double a[4], b[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) a[k] = halve<32>(v[k], v[k + 4]);
#pragma unroll
  for (int k = 0; k < 2; ++k) b[k] = halve<16>(a[k], a[k + 2]);
  const bool h3 = lane & 8;
  double c = (h3 ? b[1] : b[0]) + dpp<0x128 /* row_ror:8 */>(h3 ? b[0] : b[1]);
  const double up = dpp<0x12c /* row_ror:12 */>(c), dn = dpp<0x124 /* row_ror:4 */>(c);
  c += (lane & 4) ? dn : up;
  c += dpp<0x4e /* quad_perm 2 3 0 1 */>(c);
  c += dpp<0xb1 /* quad_perm 1 0 3 2 */>(c);
  return c;
}

// the sum over l / 8 of lane l's value, in every lane of the same l % 8
__device__ __forceinline__ double waves_sum(double v) {
  v += dpp<0x128>(v);
  v = halve<16>(v, v);
  return halve<32>(v, v);
}
__device__ __forceinline__ double lane_value(double v, int l) {
  return join(__builtin_amdgcn_readlane(half_of(v, 0), l), __builtin_amdgcn_readlane(half_of(v, 1), l));
}

// A wait that other workgroups end: polls are counted, and from the 64th on
// every 64th looks at the clock (100 MHz).
struct Wait {
  uint64_t end = 0;
  int polls = 0;
  __device__ bool over(uint64_t limit) {
    if (limit == 0) return true;
    if (++polls & 63) return false;
    __builtin_amdgcn_s_sleep(1);
    const uint64_t now = wall_clock64();
    if (end == 0) end = now + limit;
    return now > end;
  }
};

// T, CD: precision; D constant (CgVectors::D null).  R: rows a thread holds.
// NW: waves.  XL: x and c live in LDS.  The tile: 64 wx columns by R NW / wx
// rows; wave w holds columns 64 (w % wx) .. and rows R (w / wx) .. of it.
constexpr int kMaxCgpBlocks = 2 * kCus;  // workgroups of a launch, at most

template <typename T, bool CD, int R, int NW, bool XL>
__global__ __launch_bounds__(64 * NW) void k_cgp2(Geo G, Stencil<2, T> K, CgSolve<T> v, CgpGrid g,
                                                  CgScalars* sc) {
  constexpr int NT = 64 * NW, NH = sizeof(T) / 4;  // NH: 32-bit halves of a value
  // p around each wave's cells: the rows below and above, the cells left and right
  constexpr int kLo = 0, kHi = NW * 64, kLeft = 2 * NW * 64, kRight = kLeft + NW * R;
  __shared__ T ring[kRight + NW * R];
  // D of the cells right of a wave, weight of its left faces
  __shared__ T dr_edge[NW][CD ? 1 : R], wl_edge[NW][CD ? 1 : R];
  __shared__ T xs[XL ? R : 1][XL ? NT : 1], cs[XL ? R : 1][XL ? NT : 1];
  __shared__ double sh_w[NW][8], sh_s[NW][8];
  __shared__ int sh_dead;
  if (__hip_atomic_load(&sc->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) || sc->bb == 0.0) return;
  const int nx = G.nx, nz = G.nz, wx = g.wx, nwz = NW / wx;
  const int W = 64 * wx, TZ = R * nwz, EW = 2 * W + 2 * TZ;  // border cells of a tile
  const int tile = xcd_block(), bx = tile % g.nbx, bz = tile / g.nbx, nblk = gridDim.x;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);  // (a scalar)
  const int sx = w % wx, wz = w / wx;
  const int i = bx * W + sx * 64 + lane, k0 = bz * TZ + wz * R;
  const uint32_t base = (uint32_t)word_load(g.ex);  // (the previous launch left it)
  uint64_t* const edges = g.ex + 8;
  uint64_t* const sets = edges + 2L * nblk * EW * NH;
  const T kx = K.k[0], kz = K.k[1];
  const T wx0 = CD ? v.Dc * kx : T(0), wz0 = CD ? v.Dc * kz : T(0);
  const bool in = i < nx;
  if (t == 0) sh_dead = 0;
  for (int e = t; e < kRight + NW * R; e += NT) ring[e] = T(0);
  if (lane < (CD ? 1 : R)) dr_edge[w][lane] = wl_edge[w][lane] = T(0);

  // 1/diag of cell (ci, k) when D is constant (as k_cg_iter2 sums it)
  auto diag_inv = [&](T c, int ci, int k) {
    T dg = c;
    dg += ci + 1 < nx ? wx0 : T(0);
    dg += ci > 0 ? wx0 : T(0);
    dg += k + 1 < nz ? wz0 : T(0);
    dg += k > 0 ? wz0 : T(0);
    return T(1) / dg;
  };
  auto weight = [&](T a, T b, T k) { return T(0.5) * (a + b) * k; };

  // ---- the tile's vectors: cells outside the mesh hold zeros throughout
  T r[R], q[R], p[R], m[R];
  T x[XL ? 1 : R], c[XL ? 1 : R];
  T d[CD ? 1 : R + 1], wd0 = T(0);  // D of the rows and the one above; weight of row 0's lower face
  const T kxr = i + 1 < nx ? kx : T(0);  // (no face on the wall)
  const T wrc = CD && in && i + 1 < nx ? wx0 : T(0), wlc = CD && in && i > 0 ? wx0 : T(0);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int k = k0 + j;
    const bool ok = in && k < nz;
    const int P = (in ? i : nx - 1) + nx * (k < nz ? k : nz - 1);
    const T rv = v.r[P], cv = v.c[P], xv = v.x[P];
    r[j] = ok ? rv : T(0);
    q[j] = T(0);
    if constexpr (XL) {
      xs[j][t] = xv;
      cs[j][t] = ok ? cv : T(0);
    } else {
      x[j] = xv;
      c[j] = ok ? cv : T(0);
    }
    if constexpr (CD) {
      m[j] = ok ? diag_inv(cv, i, k) : T(0);
    } else {
      const T mv = v.dinv[P];
      m[j] = ok ? mv : T(0);
      d[j] = v.D[P];
      if (j == 0) {
        const T dd = v.D[ok && k > 0 ? P - nx : P];
        wd0 = ok && k > 0 ? weight(dd, d[0], kz) : T(0);
      }
      if (j == R - 1) d[R] = v.D[k + 1 < nz ? P + nx : P];
    }
    if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();  // (the zeros above)
  if constexpr (!CD) {
    if (lane < R) {
      const int k = k0 + lane, il = bx * W + sx * 64;
      if (il > 0 && il < nx && k < nz) {
        const int P = il + nx * k;
        wl_edge[w][lane] = weight(v.D[P - 1], v.D[P], kx);
      }
      if (il + 64 < nx && k < nz) dr_edge[w][lane] = v.D[il + 64 + nx * k];
    }
  }

  // ---- halo cells of this thread: below [0], above [1], side [2]
  T hr[3], hp[3], hm[3];
  int hw[3], hd[3];  // their owner's border words (parity 0); their place in the ring, -1: no cell
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    int hi = 0, hk = 0, owner = tile, e = 0;
    bool ok;
    if (s < 2) {
      hi = bx * W + t;
      hk = s == 0 ? bz * TZ - 1 : (bz + 1) * TZ;
      ok = t < W && hi < nx && hk >= 0 && hk < nz;
      owner = tile + (s == 0 ? -g.nbx : g.nbx);
      e = (s == 0 ? W : 0) + t;
      hd[s] = s == 0 ? kLo + t : kHi + (nwz - 1) * W + t;
    } else {
      const int side = t >= TZ, row = side ? t - TZ : t;
      hi = side ? (bx + 1) * W : bx * W - 1;
      hk = bz * TZ + row;
      ok = t < 2 * TZ && hi >= 0 && hi < nx && hk < nz;
      owner = tile + (side ? 1 : -1);
      e = 2 * W + (side ? 0 : TZ) + row;
      hd[s] = (side ? kRight + (wx - 1) * R : kLeft) + (row / R) * wx * R + row % R;
    }
    hr[s] = hp[s] = hm[s] = T(0);
    if (ok) {
      const int P = hi + nx * hk;
      hr[s] = v.r[P];
      hm[s] = CD ? diag_inv(v.c[P], hi, hk) : v.dinv[P];
    } else {
      hd[s] = -1;
    }
    hw[s] = (owner * EW + e) * NH;
  }
  const long epar = (long)nblk * EW * NH, spar = 16L * nblk;  // words of one parity
  const int lane_set = CD ? (t & 15) : (lane & 15);
  uint64_t* const my_edge = edges + (long)tile * EW * NH;
  const double tolbb = sc->tol2 * sc->bb;
  const int max_iter = sc->max_iter;

#pragma unroll
  for (int j = 0; j < R; ++j) p[j] = r[j] * m[j];
#pragma unroll
  for (int s = 0; s < 3; ++s) hp[s] = hr[s] * hm[s];
  T alpha, beta;
  double rr = 0.0;
  int iter = 0, status = 0;
  bool bad = false;
  for (;; ++iter) {
    const uint32_t tag = base + 1u + (uint32_t)iter;
#pragma unroll
    for (int s = 0; s < 3; ++s)
      if (hd[s] >= 0) ring[hd[s]] = hp[s];
    // borders between the workgroup's waves
    if (wz > 0) ring[kHi + (w - wx) * 64 + lane] = p[0];
    if (wz + 1 < nwz) ring[kLo + (w + wx) * 64 + lane] = p[R - 1];
    if (lane == 0 && sx > 0) {
#pragma unroll
      for (int j = 0; j < R; ++j) ring[kRight + (w - 1) * R + j] = p[j];
    }
    if (lane == 63 && sx + 1 < wx) {
#pragma unroll
      for (int j = 0; j < R; ++j) ring[kLeft + (w + 1) * R + j] = p[j];
    }
    lds_barrier();
    // A p, the dots, and the border of A p for the neighbours
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    uint64_t* const me = my_edge + (iter & 1) * epar;
    const T above = ring[kHi + t];
    T below = ring[kLo + t];
    T wdn = wd0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int k = k0 + j;
      const T pc = p[j];
      const T pr = lane_next<true>(ring[kRight + w * R + j], pc),
              pl = lane_next<false>(ring[kLeft + w * R + j], pc);
      const T pu = j + 1 < R ? p[j + 1] : above;
      T wrj, wlj, wuj;
      if constexpr (CD) {
        wrj = wrc;
        wlj = wlc;
        wuj = k + 1 < nz ? wz0 : T(0);
        wdn = k > 0 && k < nz ? wz0 : T(0);
      } else {
        // (formed anew each iteration: hoisted out of the loop they would not
        // fit the registers)
        asm volatile("" : "+v"(d[j]));
        wrj = weight(d[j], lane_next<true>(dr_edge[w][j], d[j]), kxr);
        wlj = lane_next<false>(wl_edge[w][j], wrj);
        wuj = weight(d[j], d[j + 1], k + 1 < nz ? kz : T(0));
      }
      T cj;
      if constexpr (XL)
        cj = cs[j][t];
      else
        cj = c[j];
      T a = cj * pc;
      a = fma_t(pc - pr, wrj, a);
      a = fma_t(pc - pl, wlj, a);
      a = fma_t(pc - pu, wuj, a);
      a = fma_t(pc - below, wdn, a);
      q[j] = a;
      asm volatile("" : "+v"(m[j]));  // (r m formed anew: kept from the update it is a register more a row)
      const T z = r[j] * m[j], mq = a * m[j];
      acc[0] += (double)pc * (double)a;
      acc[1] += (double)a * (double)z;
      acc[2] += (double)a * (double)mq;
      acc[3] += (double)r[j] * (double)r[j];
      acc[4] += (double)a * (double)r[j];
      acc[5] += (double)a * (double)a;
      acc[6] += (double)r[j] * (double)z;
      below = pc;
      wdn = wuj;
      if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if (nblk > 1) {
      // (rows 0 and R - 1 of the tile's first and last wave rows, its first and last columns)
      if (wz == 0) {
#pragma unroll
        for (int h = 0; h < NH; ++h) word_store(me + (sx * 64 + lane) * NH + h, tag, half_of(q[0], h));
      }
      if (wz == nwz - 1) {
#pragma unroll
        for (int h = 0; h < NH; ++h)
          word_store(me + (W + sx * 64 + lane) * NH + h, tag, half_of(q[R - 1], h));
      }
      if ((lane == 0 && sx == 0) || (lane == 63 && sx == wx - 1)) {
        uint64_t* const o = me + (2 * W + (lane == 0 ? 0 : TZ) + wz * R) * NH;
#pragma unroll
        for (int j = 0; j < R; ++j) {
#pragma unroll
          for (int h = 0; h < NH; ++h) word_store(o + j * NH + h, tag, half_of(q[j], h));
        }
      }
    }
    const double ws = wave_sum8(acc);
    if ((lane & 7) == 0) sh_w[w][lane >> 3] = ws;
    lds_barrier();
    uint64_t* const st = sets + (iter & 1) * spar + lane_set;
    double s7[7];
    bool late = false;
    if constexpr (CD) {
      // the tree of k_cg_iter2 and its sum over partials: the four waves in
      // order, then workgroup b in thread b (b - 256, ...) of four waves
      double sum[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      if (t < 16) {
        const double v8 = ((sh_w[0][t / 2] + sh_w[1][t / 2]) + sh_w[2][t / 2]) + sh_w[3][t / 2];
        word_store(st + 16L * blockIdx.x, tag, half_of(v8, t & 1));
      }
      for (int b = t; b < nblk; b += NT) {
        const uint64_t* const from = sets + (iter & 1) * spar + 16L * b;
        uint64_t dw[14];
        for (Wait wt;;) {
          bool ok = true;
#pragma unroll
          for (int u = 0; u < 14; ++u) dw[u] = word_load(from + u);
#pragma unroll
          for (int u = 0; u < 14; ++u) ok = ok && (uint32_t)(dw[u] >> 32) == tag;
          if (ok) break;
          if (wt.over(g.spin)) {
            late = true;
            break;
          }
        }
#pragma unroll
        for (int u = 0; u < 7; ++u) sum[u] += join((uint32_t)dw[2 * u], (uint32_t)dw[2 * u + 1]);
      }
      const double tot = wave_sum8(sum);
      if ((lane & 7) == 0) sh_s[w][lane >> 3] = tot;
      if (late) sh_dead = 1;
      lds_barrier();
#pragma unroll
      for (int u = 0; u < 7; ++u) s7[u] = ((sh_s[0][u] + sh_s[1][u]) + sh_s[2][u]) + sh_s[3][u];
    } else {
      static_assert(CD || NW == 8, "one value of one wave a lane");
      double tot = waves_sum(sh_w[lane >> 3][lane & 7]);  // value l % 8 in lane l
      if (nblk > 1) {
        // a workgroup's sums are one 128-byte line: lane l holds half l % 2
        // of value l % 16 / 2
        if (w == 0) {
          const double v8 = __shfl(tot, (lane & 15) >> 1, 64);
          if (lane < 16) word_store(st + 16L * blockIdx.x, tag, half_of(v8, lane & 1));
        }
        // every workgroup's sums: four lines a load, wave w the lines 4 w ..
        // of each 32, four such loads in flight
        double sum = 0.0;
        for (int b = w * 4 + (lane >> 4); b < nblk; b += 128) {
          const uint64_t* const from = st + 16L * b;
          uint64_t dw[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) dw[u] = word_load(from + (b + 32 * u < nblk ? 512 * u : 0));
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            for (Wait wt; (uint32_t)(dw[u] >> 32) != tag;
                 dw[u] = word_load(from + (b + 32 * u < nblk ? 512 * u : 0)))
              if (wt.over(g.spin)) {
                late = true;
                break;
              }
            // (even lanes: the other half is their neighbour's)
            const uint32_t own = (uint32_t)dw[u];
            const uint32_t other = __builtin_amdgcn_update_dpp(0u, own, 0xb1, 0xf, 0xf, false);
            if (b + 32 * u < nblk) sum += join(own, other);
          }
        }
        sum = halve<32>(sum, sum);
        sum = halve<16>(sum, sum);
        if (lane < 16 && (lane & 1) == 0) sh_s[w][lane >> 1] = sum;
        if (late) sh_dead = 1;
        lds_barrier();
        tot = waves_sum(sh_s[lane >> 3][lane & 7]);
      }
#pragma unroll
      for (int u = 0; u < 7; ++u) s7[u] = lane_value(tot, u);
    }
    if (sh_dead) {
      bad = true;
      status = kCgpAborted;
      break;
    }
    const StepScalars o = scalars_of(s7, iter, tolbb, max_iter);
    alpha = (T)o.alpha;
    beta = (T)o.beta;
    if (o.bad || o.fin) {
      status = o.status;
      bad = o.bad;
      rr = o.rr;
      break;
    }
    // the halo's A p while the own cells update
    uint64_t hv[3][NH];
    const long off = (iter & 1) * epar;
#pragma unroll
    for (int s = 0; s < 3; ++s)
      if (hd[s] >= 0) {
#pragma unroll
        for (int h = 0; h < NH; ++h) hv[s][h] = word_load(edges + off + hw[s] + h);
      }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if constexpr (XL)
        xs[j][t] = fma_t(p[j], alpha, xs[j][t]);
      else
        x[j] = fma_t(p[j], alpha, x[j]);
      r[j] = fma_t(-q[j], alpha, r[j]);
      p[j] = fma_t(p[j], beta, r[j] * m[j]);
      if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (bounds the LDS reads in flight)
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      if (hd[s] >= 0) {
        for (Wait wt;;) {
          bool ok = true;
#pragma unroll
          for (int h = 0; h < NH; ++h) ok = ok && (uint32_t)(hv[s][h] >> 32) == tag;
          if (ok) break;
          if (wt.over(g.spin)) {
            sh_dead = 1;
            break;
          }
#pragma unroll
          for (int h = 0; h < NH; ++h) hv[s][h] = word_load(edges + off + hw[s] + h);
        }
        T qh;
        if constexpr (NH == 1)
          qh = __uint_as_float((uint32_t)hv[s][0]);
        else
          qh = __longlong_as_double((hv[s][NH - 1] << 32) | (uint32_t)hv[s][0]);
        hr[s] = fma_t(-qh, alpha, hr[s]);
        hp[s] = fma_t(hp[s], beta, hr[s] * hm[s]);
      }
    }
  }
  // the last update (none after a non-finite value)
  if (in && status != kCgpAborted) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int k = k0 + j;
      if (k < nz) {
        const int P = i + nx * k;
        T xv;
        if constexpr (XL)
          xv = xs[j][t];
        else
          xv = x[j];
        if (!bad) xv = fma_t(p[j], alpha, xv);
        if (v.xo && !bad)
          v.xo[P] += (double)xv;
        else
          v.x[P] = xv;
      }
    }
  }
  if (t != 0) return;
  if (status == kCgpAborted) {  // (any workgroup may be the one that waited too long)
    __hip_atomic_store(&sc->status, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&sc->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (blockIdx.x == 0) {
    sc->iter = iter + 1;
    sc->rr = rr;
    sc->fin = bad ? 0 : 1;
    sc->done_iter = iter + 1;
    if (v.xo && !bad) sc->corrected = 1;
    sc->status = status;
    __hip_atomic_store(&sc->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    word_store(g.ex, 0u, base + 1u + (uint32_t)iter);
  }
}

// ---- plans -----------------------------------------------------------------------

template <typename T, bool CD, int R, int NW, bool XL>
void launch(hipStream_t s, const Geo& G, const CgSolve<T>& v, const CgpPlan& p, const CgpGrid& g,
            CgScalars* sc) {
  Stencil<2, T> K;
  for (int d = 0; d < 2; ++d) K.k[d] = (T)(G.S[d] / G.h[d]);
  hipLaunchKernelGGL((k_cgp2<T, CD, R, NW, XL>), dim3(p.blocks), dim3(64 * NW), 0, s, G, K, v, g, sc);
}

// the kernels: (precision, constant D, rows, waves, x and c in LDS)
template <typename T>
struct Variant {
  bool cd;
  int rows, waves;
  const void* fn;
  void (*run)(hipStream_t, const Geo&, const CgSolve<T>&, const CgpPlan&, const CgpGrid&, CgScalars*);
};
#define GEA_CGP(T, CD, R, NW, XL) \
  { CD, R, NW, (const void*)&k_cgp2<T, CD, R, NW, XL>, &launch<T, CD, R, NW, XL> }
const Variant<double> kV64[] = {
    GEA_CGP(double, true, 16, 4, false),
    GEA_CGP(double, false, 2, 8, false),
    GEA_CGP(double, false, 4, 8, false),
    GEA_CGP(double, false, 8, 8, false),
    GEA_CGP(double, false, 16, 8, true),
};
const Variant<float> kV32[] = {
    GEA_CGP(float, false, 2, 8, false),
    GEA_CGP(float, false, 4, 8, false),
    GEA_CGP(float, false, 8, 8, false),
    GEA_CGP(float, false, 16, 8, false),
    GEA_CGP(float, false, 32, 8, true),
};
template <typename T>
const Variant<T>* variants(int* n);
template <>
const Variant<double>* variants<double>(int* n) {
  *n = sizeof kV64 / sizeof kV64[0];
  return kV64;
}
template <>
const Variant<float>* variants<float>(int* n) {
  *n = sizeof kV32 / sizeof kV32[0];
  return kV32;
}

// the tiles of a variant on a mesh (blocks 0: too many); a tile is one, two or
// four waves wide, whichever leaves the fewest workgroups (the constant-D
// kernel's is four, as k_cg_iter2's)
template <typename T>
CgpPlan tiles(const Geo& G, const Variant<T>& V) {
  CgpPlan p{};
  long blocks = 0;
  int tz = 0;
  for (int wx = V.cd ? 4 : 1; wx <= 4; wx *= 2) {
    const int h = V.rows * V.waves / wx, nbx = (G.nx + 64 * wx - 1) / (64 * wx);
    const long n = (long)nbx * ((G.nz + h - 1) / h);
    if (blocks && n > blocks) continue;
    blocks = n;
    tz = h;
    p.wx = wx;
    p.nbx = nbx;
  }
  if (blocks > kMaxCgpBlocks) return p;
  p.blocks = (int)blocks;
  p.words = 8 + 2L * p.blocks * (2 * 64 * p.wx + 2 * tz) * (long)(sizeof(T) / 4) +
            2L * 16 * p.blocks;
  return p;
}

}  // namespace

// The plan of the one-launch solve: the variant with the fewest rows a thread
// whose workgroups are all on the card at once.  The constant-D system (the
// energy solves) has one variant, its tiles and sums those of k_cg_iter2.
template <typename T>
CgpPlan cgp_plan(const Geo& G, bool cd) {
  if (G.ndim != 2) return CgpPlan{};
  int dev = 0, cus = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return CgpPlan{};
  }
  const Variant<T>* V = variants<T>(&n);
  for (int k = 0; k < n; ++k) {
    if (V[k].cd != cd) continue;
    CgpPlan p = tiles(G, V[k]);
    int per = 0;
    if (p.blocks == 0) continue;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, V[k].fn, 64 * V[k].waves, 0) != hipSuccess) {
      (void)hipGetLastError();
      continue;
    }
    if (p.blocks > (long)cus * per) continue;
    // (a single workgroup exchanges nothing: worth twice the rows, not more)
    if (!cd && p.blocks > 1 && k + 1 < n && V[k + 1].rows <= 4 && tiles(G, V[k + 1]).blocks == 1) continue;
    p.variant = k + 1;
    return p;
  }
  return CgpPlan{};
}

// Words that the exchange area of any plan on the mesh can need (independent
// of the device).
template <typename T>
static long words_of(const Geo& G) {
  long most = 0;
  int n = 0;
  const Variant<T>* V = variants<T>(&n);
  for (int k = 0; k < n; ++k) {
    const CgpPlan p = tiles(G, V[k]);
    if (p.blocks > 0 && p.words > most) most = p.words;
  }
  return most;
}
long cgp_words(const Geo& G) {
  if (G.ndim != 2) return 0;
  const long a = words_of<double>(G), b = words_of<float>(G);
  return a > b ? a : b;
}
template CgpPlan cgp_plan<double>(const Geo&, bool);
template CgpPlan cgp_plan<float>(const Geo&, bool);

template <typename T>
void cgp_solve(hipStream_t s, const Geo& G, const CgVectors<T>& v, const CgpPlan& p, uint64_t* ex,
               uint64_t spin, CgScalars* sc) {
  int n = 0;
  const Variant<T>& V = variants<T>(&n)[p.variant - 1];
  const CgSolve<T> a{v.x, v.r, v.c, v.D, v.dinv, v.Dc, v.xo};
  const CgpGrid g{ex, spin, p.wx, p.nbx};
  V.run(s, G, a, p, g, sc);
}
template void cgp_solve<double>(hipStream_t, const Geo&, const CgVectors<double>&, const CgpPlan&, uint64_t*, uint64_t, CgScalars*);
template void cgp_solve<float>(hipStream_t, const Geo&, const CgVectors<float>&, const CgpPlan&, uint64_t*, uint64_t, CgScalars*);

}  // namespace gea
