// gea_cgp.hip -- a whole Jacobi-PCG solve in one launch.
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
// before / now: 64 x 32 FP64 25 / 4.5 (one workgroup: the launch takes 8 and
// 1.5 an iteration), 200 x 200 FP64 15.7 / 4.1, 333 x 251 15.9 / 4.4,
// 1024 x 1024 26.8 / 6.5, 2048 x 2048 FP32 33 / 11.4 (its 11 arrays a cell came
// from the last-level cache at 5.8 TB/s).  A workgroup's sums are one 128-byte line, read by
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
__device__ __forceinline__ float lane_value(float v, int l) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l) {
  return join(__builtin_amdgcn_readlane(half_of(v, 0), l), __builtin_amdgcn_readlane(half_of(v, 1), l));
}

// What a workgroup decides as one, whichever of its waves sees it first:
//  - go: whether there is work, read by one thread (another workgroup that
//    gives up sets the done flag while this one may still be starting);
//  - dead: the solve is given up.  It is read behind the second barrier of the
//    sums and changes only where a barrier lies between, so every wave leaves
//    the loop in the same iteration;
//  - late: what a wait for the halo sets that no barrier parts from those
//    reads (where A p is exchanged); it counts with the next sums.
struct Fate {
  int go, late, dead;
};
__device__ __forceinline__ void fate_set(const CgScalars* sc, Fate& fate) {
  if (threadIdx.x == 0) {
    fate.late = fate.dead = 0;
    fate.go = !__hip_atomic_load(&sc->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) && sc->bb != 0.0;
  }
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

// The sums of all workgroups' eight values from this workgroup's per wave
// (sh_w), in every thread: a workgroup's sums are one 128-byte line of `set`,
// lane l holds half l % 2 of value l % 16 / 2.  True when a wait, of this or
// for the halo before it (LATE), outlasted its limit.  (A barrier has made sh_w
// visible; eight waves.)
template <bool LATE>
__device__ __forceinline__ bool sums_of_all(const double (&sh_w)[8][8], double (&sh_s)[8][8],
                                            uint64_t* set, int nblk, uint32_t tag, uint64_t spin,
                                            Fate& fate, double (&s7)[7]) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double tot = waves_sum(sh_w[lane >> 3][lane & 7]);  // value l % 8 in lane l
  if (nblk > 1) {
    uint64_t* const st = set + (lane & 15);
    if (w == 0) {
      const double v8 = __shfl(tot, (lane & 15) >> 1, 64);
      if (lane < 16) word_store(st + 16L * blockIdx.x, tag, half_of(v8, lane & 1));
    }
    // every workgroup's sums: four lines a load, wave w the lines 4 w ..
    // of each 32, four such loads in flight
    double sum = 0.0;
    bool late = LATE && w == 0 && fate.late;
    for (int b = w * 4 + (lane >> 4); b < nblk; b += 128) {
      const uint64_t* const from = st + 16L * b;
      uint64_t dw[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) dw[u] = word_load(from + (b + 32 * u < nblk ? 512 * u : 0));
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        for (Wait wt; (uint32_t)(dw[u] >> 32) != tag;
             dw[u] = word_load(from + (b + 32 * u < nblk ? 512 * u : 0)))
          if (wt.over(spin)) {
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
    if (late) fate.dead = 1;
    lds_barrier();
    tot = waves_sum(sh_s[lane >> 3][lane & 7]);
  }
#pragma unroll
  for (int u = 0; u < 7; ++u) s7[u] = lane_value(tot, u);
  return fate.dead != 0;
}

// what a solve leaves (one thread a workgroup)
__device__ __forceinline__ void leave_scalars(CgScalars* sc, uint64_t* ex, int status, int iter,
                                              double rr, bool bad, bool corrects, uint32_t base) {
  // Any workgroup may be the one that waited too long, and workgroup 0 may end
  // well beside it: of the two the lesser status, given up, stays.
  if (status == kCgpAborted) {
    __hip_atomic_fetch_min(&sc->status, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&sc->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (blockIdx.x == 0) {
    sc->iter = iter + 1;
    sc->rr = rr;
    sc->fin = bad ? 0 : 1;
    sc->done_iter = iter + 1;
    if (corrects && !bad) sc->corrected = 1;
    __hip_atomic_fetch_min(&sc->status, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&sc->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    word_store(ex, 0u, base + 1u + (uint32_t)iter);
  }
}

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
  __shared__ Fate fate;
  fate_set(sc, fate);
  lds_barrier();
  if (!fate.go) return;
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
  // (half the constant: the same bits as 0.5 (a + b) k, a product less: 2048^2
  // FP32 steps 9.07 to 8.92 ms)
  const T hx = T(0.5) * kx, hz = T(0.5) * kz;
  auto weight = [](T a, T b, T half_k) { return (a + b) * half_k; };

  // ---- the tile's vectors: cells outside the mesh hold zeros throughout
  T r[R], q[R], p[R], m[R];
  T x[XL ? 1 : R], c[XL ? 1 : R];
  T d[CD ? 1 : R + 1], wd0 = T(0);  // D of the rows and the one above; weight of row 0's lower face
  const T kxr = i + 1 < nx ? hx : T(0);  // (no face on the wall)
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
        wd0 = ok && k > 0 ? weight(dd, d[0], hz) : T(0);
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
        wl_edge[w][lane] = weight(v.D[P - 1], v.D[P], hx);
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
  uint64_t* const my_edge = edges + (long)tile * EW * NH;
  const double tolbb = sc->tol2 * sc->bb;
  const int max_iter = min(sc->max_iter, g.cap);

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
        wuj = weight(d[j], d[j + 1], k + 1 < nz ? hz : T(0));
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
    double s7[7];
    if constexpr (CD) {
      uint64_t* const st = sets + (iter & 1) * spar + (t & 15);
      bool late = w == 0 && fate.late;
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
      if (late) fate.dead = 1;
      lds_barrier();
#pragma unroll
      for (int u = 0; u < 7; ++u) s7[u] = ((sh_s[0][u] + sh_s[1][u]) + sh_s[2][u]) + sh_s[3][u];
    } else {
      static_assert(CD || NW == 8, "one value of one wave a lane");
      if constexpr (!CD) sums_of_all<true>(sh_w, sh_s, sets + (iter & 1) * spar, nblk, tag, g.spin, fate, s7);
    }
    if (fate.dead) {
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
            fate.late = 1;
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
  if (t == 0) leave_scalars(sc, g.ex, status, iter, rr, bad, v.xo != nullptr, base);
}

// ---- 3D --------------------------------------------------------------------------
// The same solve of a 3D system.  A workgroup's tile is 64 x (8 RY) x RZ
// cells; wave w holds rows RY w .. of every plane, a thread a column of RZ
// cells in each of its RY rows.  The direction lives in LDS with a one-cell
// halo (the halo below and above in registers: those cells' thread is the
// column's own), r, A p and 1/diag in registers.  What holds the rest:
//  - MEM false: x and c in registers, D in LDS, nothing moves through memory;
//  - MEM true (64 cells a thread): D and c are read, x read and written each
//    iteration, 16 bytes a cell where the iteration kernel moves 44.
// And what the neighbours exchange:
//  - HQ true: A p, as in k_cgp2: the halo's r, p and 1/diag are kept by the
//    thread that stages it, and one exchange an iteration is enough;
//  - HQ false: the new direction, a second exchange behind the sums', where
//    the halo's vectors would not fit the registers.
template <typename T, int RY, int RZ, bool MEM, bool HQ>
__global__ __launch_bounds__(512) void k_cgp3(Geo G, Stencil<3, T> K, CgSolve<T> v, CgpGrid g,
                                              CgScalars* sc) {
  constexpr int NW = 8, NT = 512, NH = sizeof(T) / 4, TY = RY * NW, TZ = RZ, R = RY * RZ;
  constexpr int SX = 66, SY = TY + 2;
  constexpr int ZE = TY * 64, YE = TZ * 64, XE = TY * TZ;  // border cells of a z, y, x side
  constexpr int EW = 2 * (ZE + YE + XE);
  constexpr int NZ = 2 * RY, NY = (2 * YE + NT - 1) / NT, NHC = NZ + NY + (2 * XE + NT - 1) / NT;
  __shared__ T sp[TZ * SY * SX];
  __shared__ T sd[MEM ? 1 : TZ * SY * SX];
  __shared__ T zl[MEM ? NZ * NT : 1];
  __shared__ double sh_w[NW][8], sh_s[NW][8];
  __shared__ Fate fate;
  fate_set(sc, fate);
  const int nx = G.nx, ny = G.ny, nz = G.nz;
  const int tile = xcd_block(), nblk = gridDim.x;
  const int bx = tile % g.nbx, by = (tile / g.nbx) % g.nby, bz = tile / (g.nbx * g.nby);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int i0 = bx * 64, j0 = by * TY, k0 = bz * TZ, i = i0 + lane;
  const uint32_t base = (uint32_t)word_load(g.ex);  // (the previous launch left it)
  uint64_t* const edges = g.ex + 8;
  const long epar = (long)nblk * EW * NH, spar = 16L * nblk;  // words of one parity
  uint64_t* const sets = edges + 2 * epar;
  const bool in = i < nx;
  const T hx = T(0.5) * K.k[0], hy = T(0.5) * K.k[1], kz = T(0.5) * K.k[2];
  const T kxr = i + 1 < nx ? hx : T(0), kxl = in && i > 0 ? hx : T(0);
  // weights of the faces below the wave's rows and above the last (no face on the walls)
  T ky[RY + 1];
#pragma unroll
  for (int jy = 0; jy <= RY; ++jy) {
    const int gj = j0 + w * RY + jy;
    ky[jy] = gj > 0 && gj < ny ? hy : T(0);
  }
  // (half the constant: the same bits as 0.5 (a + b) k)
  auto weight = [](T a, T b, T half_k) { return (a + b) * half_k; };
  auto at = [](int k, int y, int x) { return (k * SY + y + 1) * SX + x + 1; };
  // the thread's own cell of plane 0 and its first row; other cells are
  // constants away.  (This, the thread index of the halo, the plane's size and
  // the tile's first plane are made opaque in each iteration: addresses kept from one to the next
  // would take the registers of the vectors.)
  int own = at(0, w * RY, lane), th = t, plane = nx * ny, kb = k0;
  auto off = [](int k, int y, int x) { return (k * SY + y) * SX + x; };
  for (int e = t; e < TZ * SY * SX; e += NT) {
    sp[e] = T(0);
    if constexpr (!MEM) sd[e] = T(0);
  }
  __syncthreads();
  if (!fate.go) return;

  // ---- halo cells of this thread: [0, NZ) below and above its columns, then
  // of the y sides, then of the x sides
  struct Halo {
    bool ok;
    int P, word, dst;  // cell; its owner's border word (parity 0); place in sp
  };
  auto halo = [&](int s) {
    Halo h;
    asm volatile("" : "+v"(th));  // (one cell's arithmetic after the other's)
    const int l = th & 63;
    int hi = i0 + l, hj, hk, owner, e;
    bool ok = true;
    if (s < NZ) {
      const int up = s / RY, y = w * RY + s % RY;
      hj = j0 + y;
      hk = up ? k0 + TZ : k0 - 1;
      owner = tile + (up ? 1 : -1) * g.nbx * g.nby;
      e = (up ? 0 : ZE) + y * 64 + l;
      h.dst = 0;
    } else if (s < NZ + NY) {
      const int e0 = th + NT * (s - NZ), up = e0 >= YE, rem = e0 - up * YE, k = rem >> 6;
      ok = e0 < 2 * YE;
      hj = up ? j0 + TY : j0 - 1;
      hk = k0 + k;
      owner = tile + (up ? 1 : -1) * g.nbx;
      e = 2 * ZE + (up ? 0 : YE) + rem;
      h.dst = at(k, up ? TY : -1, l);
    } else {
      const int e0 = th + NT * (s - NZ - NY), up = e0 >= XE, rem = e0 - up * XE, y = rem % TY, k = rem / TY;
      ok = e0 < 2 * XE;
      hi = up ? i0 + 64 : i0 - 1;
      hj = j0 + y;
      hk = k0 + k;
      owner = tile + (up ? 1 : -1);
      e = 2 * (ZE + YE) + (up ? 0 : XE) + rem;
      h.dst = at(k, y, up ? 64 : -1);
    }
    h.ok = ok && hi >= 0 && hi < nx && hj >= 0 && hj < ny && hk >= 0 && hk < nz;
    h.P = h.ok ? hi + nx * hj + plane * hk : 0;
    h.word = (h.ok ? owner * EW + e : tile * EW + l) * NH;  // (no cell: a word that is not waited for)
    return h;
  };

  // ---- the tile's vectors: cells outside the mesh hold zeros throughout
  T r[R], q[R], m[R], x[MEM ? 1 : R], c[MEM ? 1 : R];
  // direction below [0, RY) and above the thread's columns
  T zr[MEM ? 1 : NZ];
  auto zh_get = [&](int s) { return MEM ? zl[MEM ? s * NT + th : 0] : zr[MEM ? 0 : s]; };
  auto zh_put = [&](int s, T val) {
    if constexpr (MEM)
      zl[s * NT + th] = val;
    else
      zr[s] = val;
  };
  // weight of the lowest faces, D above the highest cells (MEM: read each iteration)
  T wz0[MEM ? 1 : RY], dt[MEM ? 1 : RY];
  const int ic = in ? i : nx - 1;
  // (uniform) start of the wave's row jy of plane k, clamped into the mesh
  int rows[RY + 2];
#pragma unroll
  for (int jy = -1; jy <= RY; ++jy) {
    const int gj = j0 + w * RY + jy;
    rows[jy + 1] = nx * (gj < 0 ? 0 : (gj < ny ? gj : ny - 1));
  }
  auto row_of = [&](int k, int jy) {
    const int gk = kb + k;
    return rows[jy + 1] + plane * (gk < 0 ? 0 : (gk < nz ? gk : nz - 1));
  };
  auto live_row = [&](int k, int jy) { return j0 + w * RY + jy < ny && kb + k < nz; };
  // a value of that row: scalar base, 32-bit offset of the lane
  uint32_t ib = (uint32_t)ic * sizeof(T);
  auto st = [&](T* f, int k, int jy, T val) {
    typedef __attribute__((address_space(1))) char* gchar;
    gchar row = (gchar)(f + row_of(k, jy));
    asm volatile("" : "+s"(row), "+v"(ib));
    *(__attribute__((address_space(1))) T*)(row + ib) = val;
  };
  auto ld = [&](const T* f, int k, int jy) {
    typedef const __attribute__((address_space(1))) char* gchar;
    gchar row = (gchar)(f + row_of(k, jy));
    asm volatile("" : "+s"(row), "+v"(ib));  // (or the address becomes a 64-bit vector sum)
    return *(const __attribute__((address_space(1))) T*)(row + ib);
  };
  double r_r = 0.0, r_z = 0.0;  // this thread's (r, r) and (r, z)
  // (in groups of GL cells, all of a group's loads ahead of their use, here and
  // at the solve's end: 12 us less a solve of 64 cells a thread than cell by
  // cell; the set-up takes 30 us of one on 256 x 256 x 128 cells)
  constexpr int GL = R < 8 ? R : 8;
#pragma unroll
  for (int n0 = 0; n0 < R; n0 += GL) {
    T rv[GL], mv[GL], cv[MEM ? 1 : GL], xv[MEM ? 1 : GL], dv[MEM ? 1 : GL];
#pragma unroll
    for (int u = 0; u < GL; ++u) {
      const int k = (n0 + u) / RY, jy = (n0 + u) % RY;
      rv[u] = ld(v.r, k, jy);
      mv[u] = ld(v.dinv, k, jy);
      if constexpr (!MEM) {
        cv[u] = ld(v.c, k, jy);
        xv[u] = ld(v.x, k, jy);
        dv[u] = ld(v.D, k, jy);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < GL; ++u) {
      const int n = n0 + u, k = n / RY, jy = n % RY, y = w * RY + jy;
      const bool ok = in && live_row(k, jy);
      r[n] = ok ? rv[u] : T(0);
      m[n] = ok ? mv[u] : T(0);
      q[n] = T(0);
      if constexpr (!MEM) {
        x[n] = xv[u];
        c[n] = ok ? cv[u] : T(0);
        sd[at(k, y, lane)] = dv[u];
      }
      const T z = r[n] * m[n];
      sp[at(k, y, lane)] = z;
      r_r += (double)r[n] * (double)r[n];
      r_z += (double)r[n] * (double)z;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (!MEM) {
#pragma unroll
    for (int jy = 0; jy < RY; ++jy) {
      wz0[jy] = k0 > 0 ? weight(ld(v.D, -1, jy), ld(v.D, 0, jy), kz) : T(0);
      dt[jy] = ld(v.D, TZ, jy);
    }
  }
  // (MEM) of plane k in lane k: D right of the tile's rows, weight of their left faces
  T er[RY], el[RY];
  if constexpr (MEM) {
    static_assert(RZ <= 64, "a plane a lane");
#pragma unroll
    for (int jy = 0; jy < RY; ++jy) {
      const T* const row = v.D + row_of(lane < RZ ? lane : 0, jy);
      er[jy] = row[i0 + 64 < nx ? i0 + 64 : nx - 1];
      el[jy] = i0 > 0 ? weight(row[i0 > 0 ? i0 - 1 : 0], row[i0], hx) : T(0);
    }
  }
  T hr[HQ ? NHC : 1], hp[HQ ? NHC : 1], hm[HQ ? NHC : 1];
  constexpr int GS = NHC < 7 ? NHC : 7;
#pragma unroll
  for (int s0 = 0; s0 < NHC; s0 += GS) {
    T rv[GS], mv[GS], dv[MEM ? 1 : GS];
#pragma unroll
    for (int s = s0; s < s0 + GS && s < NHC; ++s) {
      const Halo h = halo(s);
      rv[s - s0] = v.r[h.P];
      mv[s - s0] = v.dinv[h.P];
      if constexpr (!MEM) dv[s - s0] = v.D[h.P];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = s0; s < s0 + GS && s < NHC; ++s) {
      const Halo h = halo(s);
      const T pv = h.ok ? rv[s - s0] * mv[s - s0] : T(0);
      if constexpr (HQ) {
        hr[s] = rv[s - s0];
        hm[s] = mv[s - s0];
        hp[s] = pv;
      }
      if (s < NZ)
        zh_put(s, pv);
      else if (h.ok) {
        sp[h.dst] = pv;
        if constexpr (!MEM) sd[h.dst] = dv[s - s0];
      }
    }
  }
  __syncthreads();
  uint64_t* const my_edge = edges + (long)tile * EW * NH;
  // border words of the neighbours: scalar base, 32-bit offset
  auto edge_load = [&](int iter, int word) {
    typedef const __attribute__((address_space(1))) char* gchar;
    gchar from = (gchar)(edges + (iter & 1) * epar);
    uint32_t o = (uint32_t)word * 8u;
    asm volatile("" : "+s"(from), "+v"(o));
    return __hip_atomic_load((const __attribute__((address_space(1))) uint64_t*)(from + o), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  };
  auto publish = [&](uint64_t* o, int e, uint32_t tag, T val) {
#pragma unroll
    for (int h = 0; h < NH; ++h) word_store(o + e * NH + h, tag, half_of(val, h));
  };
  // (uniform) neighbours in z
  const bool zl_nb = bz > 0, zh_nb = k0 + TZ < nz;
  const double tolbb = sc->tol2 * sc->bb;
  const int max_iter = min(sc->max_iter, g.cap);
  constexpr int GX = R < 8 ? R : 8;  // x of these cells in flight (MEM)
  // (MEM) one load of a wave that names 64 of the 128-byte lines it reads later:
  // it brings them into the L2 in the meantime, for one register.  D and c of
  // WIN planes from plane k on, or x of 2 WIN planes.
  constexpr int WIN = 8;
  static_assert(!MEM || (RY * WIN * 4 == 64 && RZ == 4 * WIN && sizeof(T) == 4), "a line a lane");
  auto touch_row = [&](const T* f, int k, int n) {
    const int row = n % RY ? rows[RY] : rows[1], gk = kb + k + n / RY, gx = i0 + 32 * (th & 1);
    return f[row + plane * (gk < nz ? gk : nz - 1) + (gx < nx ? gx : nx - 1)];
  };
  auto touch = [&](int k) { return touch_row(th & 32 ? v.D : v.c, k, (th & 31) >> 1); };
  auto touch_x = [&](int k) { return touch_row(v.x, k, (th & 63) >> 1); };
  T line = T(0), line_x[2] = {T(0), T(0)};
  T alpha, beta;
  double rr = 0.0;
  int iter = 0, status = 0;
  bool bad = false;
  for (;; ++iter) {
    const uint32_t tag = base + 1u + (uint32_t)iter;
    asm volatile("" : "+v"(own), "+v"(th), "+s"(plane), "+s"(kb));
    // ---- A p and the dots, plane by plane
    // ((r, r) and (r, z) are summed where r is formed)
    double acc[8] = {0.0, 0.0, 0.0, r_r, 0.0, 0.0, r_z, 0.0};
    {
      // D and c around plane k that its step reads
      struct Set {
        T da[RY], dl[MEM ? 1 : RY], dr[MEM ? 1 : RY], c[RY], dlo, dhi;
      };
      auto load = [&](int k) {
        Set f;
#pragma unroll
        for (int jy = 0; jy < RY; ++jy) {
          if constexpr (MEM) {
            f.c[jy] = ld(v.c, k, jy);
            f.da[jy] = ld(v.D, k + 1, jy);
          } else {
            f.dl[jy] = sd[own + off(k, jy, -1)];
            f.dr[jy] = sd[own + off(k, jy, 1)];
            f.c[jy] = c[k * RY + jy];
            f.da[jy] = k + 1 < RZ ? sd[own + off(k + 1, jy, 0)] : dt[jy];
          }
        }
        if constexpr (MEM) {
          f.dlo = ld(v.D, k, -1);
          f.dhi = ld(v.D, k, RY);
        } else {
          f.dlo = sd[own + off(k, -1, 0)];
          f.dhi = sd[own + off(k, RY, 0)];
        }
        return f;
      };
      T pb[RY], pc[RY], dc[RY], wb[RY];
#pragma unroll
      for (int jy = 0; jy < RY; ++jy) {
        pb[jy] = zh_get(jy);
        pc[jy] = sp[own + off(0, jy, 0)];
        dc[jy] = MEM ? ld(v.D, 0, jy) : sd[MEM ? 0 : own + off(0, jy, 0)];
        wb[jy] = MEM ? weight(ld(v.D, -1, jy), dc[jy], k0 > 0 ? kz : T(0)) : wz0[MEM ? 0 : jy];
      }
      Set cur = load(0);
      int pl = own;  // (own cell of every eighth plane: LDS offsets are 16 bits)
#pragma unroll
      for (int k = 0; k < RZ; ++k) {
        if (k % 8 == 0 && k > 0) {
          pl += off(8, 0, 0);
          asm volatile("" : "+v"(pl));
        }
        Set nxt;
        if (k + 1 < RZ) nxt = load(k + 1);
        if constexpr (MEM) {
          if (k % WIN == 0 && k + WIN < RZ) line = touch(k + WIN);
        }
        const T kzu = kb + k + 1 < nz ? kz : T(0);
        const T plo = sp[pl + off(k % 8, -1, 0)], phi = sp[pl + off(k % 8, RY, 0)];
        T wlo = weight(cur.dlo, dc[0], ky[0]);
#pragma unroll
        for (int jy = 0; jy < RY; ++jy) {
          const int n = k * RY + jy;
          const T pr = sp[pl + off(k % 8, jy, 1)], pf = sp[pl + off(k % 8, jy, -1)];
          const T pu = jy + 1 < RY ? pc[jy + 1 < RY ? jy + 1 : 0] : phi;
          const T pd = jy > 0 ? pc[jy > 0 ? jy - 1 : 0] : plo;
          const T pa = k + 1 < RZ ? sp[pl + off(k + 1 < RZ ? k % 8 + 1 : 0, jy, 0)] : zh_get(RY + jy);
          T wr, wl;
          if constexpr (MEM) {
            wr = weight(dc[jy], lane_next<true>(lane_value(er[jy], k), dc[jy]), kxr);
            wl = lane_next<false>(lane_value(el[jy], k), wr);
          } else {
            wr = weight(dc[jy], cur.dr[jy], kxr);
            wl = weight(cur.dl[jy], dc[jy], kxl);
          }
          const T wu = weight(dc[jy], jy + 1 < RY ? dc[jy + 1 < RY ? jy + 1 : 0] : cur.dhi, ky[jy + 1]);
          const T wa = weight(dc[jy], cur.da[jy], kzu);
          const T p0 = pc[jy];
          T a = cur.c[jy] * p0;
          a = fma_t(p0 - pr, wr, a);
          a = fma_t(p0 - pf, wl, a);
          a = fma_t(p0 - pu, wu, a);
          a = fma_t(p0 - pd, wlo, a);
          a = fma_t(p0 - pa, wa, a);
          a = fma_t(p0 - pb[jy], wb[jy], a);
          q[n] = a;
          asm volatile("" : "+v"(m[n]));  // (r m formed anew: kept it is a register more a cell)
          const T z = r[n] * m[n], mq = a * m[n];
          acc[0] += (double)p0 * (double)a;
          acc[1] += (double)a * (double)z;
          acc[2] += (double)a * (double)mq;
          acc[4] += (double)a * (double)r[n];
          acc[5] += (double)a * (double)a;
          // (summed here, not gathered behind the planes)
          if constexpr (MEM)
            asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[4]), "+v"(acc[5]));
          wlo = wu;
          wb[jy] = wa;
          pb[jy] = pa;  // (swapped below: the row above still reads pc)
        }
#pragma unroll
        for (int jy = 0; jy < RY; ++jy) {
          const T up = pb[jy];
          pb[jy] = pc[jy];
          pc[jy] = up;
          dc[jy] = cur.da[jy];
        }
        if (k + 1 < RZ) cur = nxt;
        if constexpr (MEM) {
          if (k % WIN == WIN - 1) asm volatile("" ::"v"(line));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (HQ) {
      if (nblk > 1) {
        uint64_t* const me = my_edge + (iter & 1) * epar;
#pragma unroll
        for (int jy = 0; jy < RY; ++jy) {
          const int y = w * RY + jy;
          if (zl_nb) publish(me, y * 64 + lane, tag, q[jy]);
          if (zh_nb) publish(me, ZE + y * 64 + lane, tag, q[(RZ - 1) * RY + jy]);
        }
        if (w == 0 && by > 0) {
#pragma unroll
          for (int k = 0; k < RZ; ++k) publish(me, 2 * ZE + k * 64 + lane, tag, q[k * RY]);
        }
        if (w == NW - 1 && by + 1 < g.nby) {
#pragma unroll
          for (int k = 0; k < RZ; ++k) publish(me, 2 * ZE + YE + k * 64 + lane, tag, q[k * RY + RY - 1]);
        }
        if ((lane == 0 && bx > 0) || (lane == 63 && bx + 1 < g.nbx)) {
          const int side = lane == 0 ? 0 : XE;
#pragma unroll
          for (int n = 0; n < R; ++n)
            publish(me, 2 * (ZE + YE) + side + (n / RY) * TY + w * RY + n % RY, tag, q[n]);
        }
      }
    }
    // (MEM) the first x of the update, in flight while the sums arrive
    T xg[MEM ? GX : 1];
    if constexpr (MEM) {
      line_x[0] = touch_x(0);
      line_x[1] = touch_x(2 * WIN);
#pragma unroll
      for (int n = 0; n < GX; ++n) xg[n] = ld(v.x, n / RY, n % RY);
    }
    // ---- the sums of all workgroups
    const double ws = wave_sum8(acc);
    if ((lane & 7) == 0) sh_w[w][lane >> 3] = ws;
    lds_barrier();
    double s7[7];
    const bool late = sums_of_all<HQ>(sh_w, sh_s, sets + (iter & 1) * spar, nblk, tag, g.spin, fate, s7);
    if (late) {
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
    asm volatile("" : "+v"(own), "+v"(th), "+s"(plane), "+s"(kb));
    // ---- the update (every wave is past its reads of sp: the sums' barrier)
    uint64_t hv[HQ ? NHC : 1][NH];
    if constexpr (HQ) {  // the halo's A p meanwhile
#pragma unroll
      for (int s = 0; s < NHC; ++s) {
        const Halo h = halo(s);
#pragma unroll
        for (int u = 0; u < NH; ++u) hv[s][u] = edge_load(iter, h.word + u);
      }
    }
    uint64_t* const me = my_edge + (iter & 1) * epar;
    r_r = r_z = 0.0;
    int pl = own;  // (own cell of every eighth plane: LDS offsets are 16 bits)
#pragma unroll
    for (int n0 = 0; n0 < R; n0 += GX) {
      T xn[MEM ? GX : 1];
      if constexpr (MEM) {
        if (n0 + GX < R) {
#pragma unroll
          for (int u = 0; u < GX; ++u) {
            const int n = n0 + GX + u;
            xn[u] = ld(v.x, n / RY, n % RY);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < GX; ++u) {
        const int n = n0 + u, k = n / RY, jy = n % RY;
        if (n % (8 * RY) == 0 && n > 0) {
          pl += off(8, 0, 0);
          asm volatile("" : "+v"(pl));
        }
        const T pv = sp[pl + off(k % 8, jy, 0)];
        if constexpr (MEM) {
          const T xv = fma_t(pv, alpha, xg[u]);
          if (in && live_row(k, jy)) st(v.x, k, jy, xv);
        } else {
          x[n] = fma_t(pv, alpha, x[n]);
        }
        r[n] = fma_t(-q[n], alpha, r[n]);
        const T z = r[n] * m[n];
        r_r += (double)r[n] * (double)r[n];
        r_z += (double)r[n] * (double)z;
        asm volatile("" : "+v"(r_r), "+v"(r_z));  // (here, not gathered behind the update)
        const T pn = fma_t(pv, beta, z);
        sp[pl + off(k % 8, jy, 0)] = pn;
        if constexpr (!HQ) {  // what the neighbours below and above read
          if (k == 0 && zl_nb) publish(me, (w * RY + jy) * 64 + lane, tag, pn);
          if (k == RZ - 1 && zh_nb) publish(me, ZE + (w * RY + jy) * 64 + lane, tag, pn);
        }
      }
      if constexpr (MEM) {
#pragma unroll
        for (int u = 0; u < GX; ++u) xg[u] = xn[u];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("" : "+v"(own), "+v"(th), "+s"(plane), "+s"(kb));
    if constexpr (MEM) {
      asm volatile("" ::"v"(line_x[0]), "v"(line_x[1]));
      line = touch(0);
    }
    // ---- the halo
    if constexpr (!HQ) {
      lds_barrier();  // the own cells' new direction
      if (nblk > 1) {  // (by all waves: two of them alone took 14 us more for the y sides)
#pragma unroll
        for (int u = 0; u < NY; ++u) {
          const int e0 = th + NT * u, up = e0 >= YE, rem = e0 - up * YE;
          if (e0 < 2 * YE && (up ? by + 1 < g.nby : by > 0))
            publish(me, 2 * ZE + e0, tag, sp[at(rem >> 6, up ? TY - 1 : 0, th & 63)]);
        }
#pragma unroll
        for (int u = 0; u < NHC - NZ - NY; ++u) {
          const int e0 = th + NT * u, up = e0 >= XE, rem = e0 - up * XE;
          if (e0 < 2 * XE && (up ? bx + 1 < g.nbx : bx > 0))
            publish(me, 2 * (ZE + YE) + e0, tag, sp[at(rem / TY, rem % TY, up ? 63 : 0)]);
        }
      }
    }
    constexpr int GH = HQ ? NHC : 7;  // halo words in flight a thread
#pragma unroll
    for (int s0 = 0; s0 < NHC; s0 += GH) {
      uint64_t wv[HQ ? 1 : GH][NH];
      if constexpr (!HQ) {
#pragma unroll
        for (int s = s0; s < s0 + GH && s < NHC; ++s) {
          const Halo h = halo(s);
#pragma unroll
          for (int u = 0; u < NH; ++u) wv[s - s0][u] = edge_load(iter, h.word + u);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int s = s0; s < s0 + GH && s < NHC; ++s) {
        const Halo h = halo(s);
        if (!h.ok) continue;
        uint64_t(&hw)[NH] = HQ ? hv[HQ ? s : 0] : wv[HQ ? 0 : s - s0];
        for (Wait wt;;) {
          bool ok = true;
#pragma unroll
          for (int u = 0; u < NH; ++u) ok = ok && (uint32_t)(hw[u] >> 32) == tag;
          if (ok) break;
          if (wt.over(g.spin)) {
            (HQ ? fate.late : fate.dead) = 1;
            break;
          }
#pragma unroll
          for (int u = 0; u < NH; ++u) hw[u] = edge_load(iter, h.word + u);
        }
        T hval;
        if constexpr (NH == 1)
          hval = __uint_as_float((uint32_t)hw[0]);
        else
          hval = __longlong_as_double((hw[NH - 1] << 32) | (uint32_t)hw[0]);
        if constexpr (HQ) {
          hr[s] = fma_t(-hval, alpha, hr[s]);
          hp[s] = fma_t(hp[s], beta, hr[s] * hm[s]);
          hval = hp[s];
        }
        if (s < NZ)
          zh_put(s, hval);
        else
          sp[h.dst] = hval;
        if constexpr (!HQ) __builtin_amdgcn_sched_barrier(0);
      }
    }
    lds_barrier();
  }
  // the last update (none after a non-finite value)
  if (status != kCgpAborted) {
    const bool outer = v.xo != nullptr && !bad;
#pragma unroll
    for (int n0 = 0; n0 < R; n0 += GL) {
      T xv[MEM ? GL : 1];
      double xo[GL];
#pragma unroll
      for (int u = 0; u < GL; ++u) {
        const int k = (n0 + u) / RY, jy = (n0 + u) % RY;
        if constexpr (MEM) xv[u] = ld(v.x, k, jy);
        xo[u] = outer ? v.xo[row_of(k, jy) + ic] : 0.0;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < GL; ++u) {
        const int n = n0 + u, k = n / RY, jy = n % RY;
        T xn;
        if constexpr (MEM)
          xn = xv[u];
        else
          xn = x[n];
        if (!bad) xn = fma_t(sp[at(k, w * RY + jy, lane)], alpha, xn);
        if (in && live_row(k, jy)) {
          if (outer)
            v.xo[row_of(k, jy) + i] = xo[u] + (double)xn;
          else
            v.x[row_of(k, jy) + i] = xn;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (t == 0) leave_scalars(sc, g.ex, status, iter, rr, bad, v.xo != nullptr, base);
}

// ---- plans -----------------------------------------------------------------------

template <typename T, bool CD, int R, int NW, bool XL>
void launch(hipStream_t s, const Geo& G, const CgSolve<T>& v, const CgpPlan& p, const CgpGrid& g,
            CgScalars* sc) {
  Stencil<2, T> K;
  for (int d = 0; d < 2; ++d) K.k[d] = (T)(G.S[d] / G.h[d]);
  hipLaunchKernelGGL((k_cgp2<T, CD, R, NW, XL>), dim3(p.blocks), dim3(64 * NW), 0, s, G, K, v, g, sc);
}

template <typename T, int RY, int RZ, bool MEM, bool HQ>
void launch3(hipStream_t s, const Geo& G, const CgSolve<T>& v, const CgpPlan& p, const CgpGrid& g,
             CgScalars* sc) {
  Stencil<3, T> K;
  for (int d = 0; d < 3; ++d) K.k[d] = (T)(G.S[d] / G.h[d]);
  hipLaunchKernelGGL((k_cgp3<T, RY, RZ, MEM, HQ>), dim3(p.blocks), dim3(512), 0, s, G, K, v, g, sc);
}

// the kernels: (precision, constant D, rows, waves, x and c in LDS) in 2D,
// (precision, y rows, planes, vectors in memory, A p exchanged) in 3D
template <typename T>
struct Variant {
  int ndim;
  bool cd;
  int rows, waves;  // 2D: rows a thread; 3D: y rows of the tile, planes
  const void* fn;
  void (*run)(hipStream_t, const Geo&, const CgSolve<T>&, const CgpPlan&, const CgpGrid&, CgScalars*);
};
#define GEA_CGP(T, CD, R, NW, XL) \
  { 2, CD, R, NW, (const void*)&k_cgp2<T, CD, R, NW, XL>, &launch<T, CD, R, NW, XL> }
#define GEA_CGP3(T, RY, RZ, MEM, HQ) \
  { 3, false, 8 * RY, RZ, (const void*)&k_cgp3<T, RY, RZ, MEM, HQ>, &launch3<T, RY, RZ, MEM, HQ> }
const Variant<double> kV64[] = {
    GEA_CGP(double, true, 16, 4, false),
    GEA_CGP(double, false, 2, 8, false),
    GEA_CGP(double, false, 4, 8, false),
    GEA_CGP(double, false, 8, 8, false),
    GEA_CGP(double, false, 16, 8, true),
    GEA_CGP3(double, 1, 2, false, true),
    GEA_CGP3(double, 1, 4, false, true),
    GEA_CGP3(double, 1, 8, false, true),
    GEA_CGP3(double, 2, 8, false, false),
};
const Variant<float> kV32[] = {
    GEA_CGP(float, false, 2, 8, false),
    GEA_CGP(float, false, 4, 8, false),
    GEA_CGP(float, false, 8, 8, false),
    GEA_CGP(float, false, 16, 8, false),
    GEA_CGP(float, false, 32, 8, true),
    GEA_CGP3(float, 1, 2, false, true),
    GEA_CGP3(float, 1, 4, false, true),
    GEA_CGP3(float, 2, 8, false, true),
    GEA_CGP3(float, 2, 16, false, false),
    GEA_CGP3(float, 2, 32, true, false),
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
  if (G.ndim != V.ndim) return p;
  if (G.ndim == 3) {
    const int ty = V.rows, tz = V.waves;
    p.wx = 1;
    p.nbx = (G.nx + 63) / 64;
    p.nby = (G.ny + ty - 1) / ty;
    const long n = (long)p.nbx * p.nby * ((G.nz + tz - 1) / tz);
    // (tiles of 64 x 16 x 16 cells and more leave no LDS for a second workgroup)
    if (n > (ty * tz < 256 ? kMaxCgpBlocks : kCus)) return p;
    p.blocks = (int)n;
    p.words = 8 + 2L * n * 2 * (64 * ty + 64 * tz + ty * tz) * (long)(sizeof(T) / 4) + 2L * 16 * n;
    return p;
  }
  long blocks = 0;
  int tz = 0;
  p.nby = 1;
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

// The plan of the one-launch solve: the variant with the fewest cells a thread
// whose workgroups are all on the card at once.  (3D meshes of more than
// 256 tiles of 64 x 16 x 32 cells in FP32, 64 x 16 x 8 in FP64, have none.)  The constant-D system (the
// energy solves) has one variant, its tiles and sums those of k_cg_iter2.
template <typename T>
CgpPlan cgp_plan(const Geo& G, bool cd) {
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
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, V[k].fn, V[k].ndim == 3 ? 512 : 64 * V[k].waves, 0) != hipSuccess) {
      (void)hipGetLastError();
      continue;
    }
    if (p.blocks > (long)cus * per) continue;
    // (a single workgroup exchanges nothing: worth twice the rows, not more)
    if (!cd && G.ndim == 2 && p.blocks > 1 && k + 1 < n && V[k + 1].rows <= 4 && tiles(G, V[k + 1]).blocks == 1) continue;
    p.variant = k + 1;
    const int die = cus / 8 > 0 ? cus / 8 : 1, n8 = (p.blocks + 7) / 8;  // a die's compute units, what the launch takes of them
    p.share = p.blocks == 1 ? 0 : (n8 >= die ? kCardShares : (kCardShares * n8 + die - 1) / die);
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
  const long a = words_of<double>(G), b = words_of<float>(G);
  return a > b ? a : b;
}
template CgpPlan cgp_plan<double>(const Geo&, bool);
template CgpPlan cgp_plan<float>(const Geo&, bool);

template <typename T>
void cgp_solve(hipStream_t s, const Geo& G, const CgVectors<T>& v, const CgpPlan& p, uint64_t* ex,
               uint64_t spin, CgScalars* sc, int cap) {
  int n = 0;
  const Variant<T>& V = variants<T>(&n)[p.variant - 1];
  const CgSolve<T> a{v.x, v.r, v.c, v.D, v.dinv, v.Dc, v.xo};
  const CgpGrid g{ex, spin, cap, p.wx, p.nbx, p.nby};
  V.run(s, G, a, p, g, sc);
}
template void cgp_solve<double>(hipStream_t, const Geo&, const CgVectors<double>&, const CgpPlan&, uint64_t*, uint64_t, CgScalars*, int);
template void cgp_solve<float>(hipStream_t, const Geo&, const CgVectors<float>&, const CgpPlan&, uint64_t*, uint64_t, CgScalars*, int);

}  // namespace gea
