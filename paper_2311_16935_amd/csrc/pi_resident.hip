// The on-chip solve: Algorithm 1's whole loop in one kernel, the inner
// solve's vectors in registers.
//
// A CG pass of the streaming kernels (pi_kernels.hip) on a grid of a few
// million cells or less is bound by its launch (about 8 us from one graph
// node to the next) and, at 2048^2, by streaming vectors that fit the
// registers of 256 CUs (128 MB) several times over.  Here a workgroup owns a
// box of cells for the whole solve: a lane keeps p, r, q and the correction
// of R consecutive cells along the march axis in registers, the box's p
// (with a ring of one cell) goes through LDS once per pass, and workgroups
// exchange only what crosses box faces.
//
// What it gives (streaming before, this after): 64^2 to 1e-6 in 79.8 -> 15.0
// ms (one workgroup, 1.9 us a pass), 101^2 39 -> 14 ms, 2048^2 masked 609 ->
// 190 us per outer step of 20 passes (256 workgroups of 128 x 128 cells), the
// 128^3 fixed-point solve inside a coarse warm start 31 -> 9 ms.  What bounds
// it: with several workgroups, the exchange (about 2 us a hop from store to
// load across XCDs); in one, FP32 and FP64 vector issue (some 25 operations a
// cell, 7 of them FP64 sums).
//
// One synchronisation per CG pass.  The pass needs p_k in the ring.  Each
// workgroup keeps r, p and the correction of its ring cells as well and
// updates them with the owner's arithmetic, so the only ring input is the
// neighbours' q_k, and that travels together with the pass's partial sums:
// both are published after the stencil and awaited at once.  The outer step
// is the same with P (FP64) in place of p and the new residual in place of q.
//
// Exchange without fences.  A published value is an 8-byte word holding 32
// bits of data and a 32-bit tag, written and read with relaxed agent-scope
// atomics (coherent across the XCDs' L2s; 8-byte accesses do not tear), so a
// reader that sees the tag has the data.  Tags count the synchronisations of
// a solve; words alternate between two buffers by tag parity.  A workgroup
// overwrites a buffer only after every workgroup has published the sum of
// the synchronisation in between, which each does after it has read the
// buffer.  The buffers hold tag 0, which is never published, when a solve
// starts (k_init).
//
// Every workgroup adds all workgroups' partial sums in the same order, so
// all take the same scalars and decisions and results do not depend on
// scheduling.  Workgroups wait for each other: launches of more than one
// workgroup per grid are cooperative (all resident at once), and a wait that
// outlasts kPatience ends the solve with PI_ERR_DEVICE instead of spinning on,
// whichever workgroup waited (res_late).
//
// A published value with its tag in one word is how collective libraries send
// short messages (their low-latency protocols).
#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "pi_common.h"
#include "pi_device.h"
#include "pi_kernels.h"
#include "pi_resident.h"

namespace pi {

#define PI_G __attribute__((address_space(1)))

namespace {

constexpr int kRB = kResBlock;
constexpr int kRWaves = kRB / kWave;
constexpr uint64_t kPatience = 2000000000ull;  // 20 s of the 100 MHz constant clock

typedef unsigned long long u64;

__device__ inline void put(PI_G u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline u64 get(PI_G u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Rounds of one wait.  over() is true once it has lasted kPatience, or once
// another wait of the workgroup has (*abort).  Between rounds the wave sleeps
// 64 clocks: without that, the loads of the waiting waves queue up in front
// of the stores that others wait for.
struct Wait {
  uint32_t n = 0;
  u64 t0 = 0;
  __device__ bool over(volatile int *abort) {
    __builtin_amdgcn_s_sleep(1);
    if ((++n & 255u) != 0) return false;
    const u64 t = wall_clock64();
    if (t0 == 0) t0 = t;
    return t - t0 > kPatience || *abort != 0;
  }
};

// ---------------------------------------------------------------------------
// sums
// ---------------------------------------------------------------------------
// Sums of four values over a wave.  The first two levels fold the four
// values into one (each lane group keeps one of them), so that seven adds do
// instead of 24.  Row of lanes 0-15 gets sum 0, 16-31 sum 2, 32-47 sum 1, 48-63 sum 3.
__device__ inline double wave_sum4(const double (&v)[4]) {
  const D2 x = swap32(v[0], v[1]), y = swap32(v[2], v[3]);
  const D2 z = swap16(x.a + x.b, y.a + y.b);
  double s = z.a + z.b;
  s += ror16<8>(s);
  s += ror16<4>(s);
  s += ror16<2>(s);
  s += ror16<1>(s);
  return s;
}
__device__ inline int sum_of_row(int lane) { return ((lane >> 4) & 1) * 2 + (lane >> 5); }

// Sum over lanes of the same lane & 3, in every lane.
__device__ inline double sum_mod4(double v) {
  v += ror16<4>(v);
  v += ror16<8>(v);
  const D2 a = swap16(v, v);
  const double w = a.a + a.b;
  const D2 b = swap32(w, w);
  return b.a + b.b;
}

__device__ inline double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

struct Shared {
  double wred[kRWaves * 4];   // per-wave sums
  double lut[6][kStates];     // operator weights by direction and state (as T)
  double a[8];                // weights of the fixed point's operator
  double al, be;              // scalars of the next pass
  int end;                    // the inner solve (or, after an outer step, the solve) ends here
  int abort;                  // a wait has lasted kPatience
  State st;
};

template <typename T>
__device__ inline T fma_t(T a, T b, T c);
template <>
__device__ inline float fma_t<float>(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}
template <>
__device__ inline double fma_t<double>(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}

// A value the compiler cannot derive anything from ahead of its use: without
// it, the table addresses and masks of all of a lane's cells are computed
// before the loop over passes and kept there, in registers that spill.
template <typename V>
__device__ inline V fresh(V v) {
  asm volatile("" : "+v"(v));
  return v;
}
template <typename V>
__device__ inline V fresh_s(V v) {
  asm volatile("" : "+s"(v));
  return v;
}

// The four sums of `count` (at most 64) workgroups, eight words each from s
// on, added in a fixed order by one wave: sum lane & 3 in every lane.
__device__ inline double gather4(PI_G u64 *s, int count, uint32_t tag, int lane, volatile int *abort, bool &late) {
  const int first = lane >> 2;
  PI_G u64 *p = s + 2 * (lane & 3);
  u64 w[8];
  Wait wait;
  for (;;) {
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w[2 * k] = w[2 * k + 1] = (u64)tag << 32;
      if (16 * k < count && first + 16 * k < count) {
        w[2 * k] = get(p + 8 * (first + 16 * k));
        w[2 * k + 1] = get(p + 8 * (first + 16 * k) + 1);
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) ok &= (uint32_t)(w[k] >> 32) == tag;
    if (__all(ok)) break;
    if (wait.over(abort)) {
      late = true;
      break;
    }
  }
  double v = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) v += __hiloint2double((int)(uint32_t)w[2 * k + 1], (int)(uint32_t)w[2 * k]);
  return sum_mod4(v);
}
// Publish the sums that lanes 0-3 hold.
__device__ inline void put4(PI_G u64 *s, double v, uint32_t tag, int lane) {
  if (lane < 8) {
    const double w = __shfl(v, lane >> 1, kWave);
    put(s + lane, ((u64)tag << 32) | ((lane & 1) ? (uint32_t)__double2hiint(w) : (uint32_t)__double2loint(w)));
  }
}

// Values in the exchange buffers: one word for a float, two for a double.
template <typename T>
__device__ inline void put_value(PI_G u64 *x, int i, uint32_t tag, T v) {
  const u64 t = (u64)tag << 32;
  if constexpr (sizeof(T) == 4) {
    put(x + i, t | __float_as_uint(v));
  } else {
    put(x + 2 * i, t | (uint32_t)__double2loint(v));
    put(x + 2 * i + 1, t | (uint32_t)__double2hiint(v));
  }
}
template <typename T>
__device__ inline bool get_value(PI_G u64 *x, int i, uint32_t tag, T &v) {
  if constexpr (sizeof(T) == 4) {
    const u64 w = get(x + i);
    v = __uint_as_float((uint32_t)w);
    return (uint32_t)(w >> 32) == tag;
  } else {
    const u64 a = get(x + 2 * i), b = get(x + 2 * i + 1);
    v = __hiloint2double((int)(uint32_t)b, (int)(uint32_t)a);
    return (uint32_t)(a >> 32) == tag && (uint32_t)(b >> 32) == tag;
  }
}

// ---------------------------------------------------------------------------
// one workgroup's part of a solve: outer steps of about `syncs` synchronisations
// ---------------------------------------------------------------------------
// SCH: 2, 3 the face-crossing scheme's dimensions, 9 the cell-centred scheme (2-D, nine-point
// stencils); N: cells per lane, HJ: ring cells per lane, OPL: the fixed point's operator.
template <typename T, int SCH, int N, int HJ, bool OPL>
__device__ __forceinline__ void solve_box(const Inst &in, State *gst, int wg, int syncs, Shared &sh, double *dyn) {
  constexpr int ND = SCH == 3 ? 3 : 2, NB = SCH == 9 ? 8 : 2 * ND;
  constexpr bool CC = SCH == 9;
  constexpr bool kHold = N <= 4;  // P and S in registers as well
  constexpr int kBits = ND == 3 ? 5 : 3;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int TX = in.res_tx, TY = ND == 3 ? in.res_ty : 1, G = in.res_g, R = in.res_r, TM = G * R;
  const int SX = TX + 2, PS = ND == 3 ? SX * (TY + 2) : SX;
  const int nx = in.nx, ny = ND == 3 ? in.ny : 1, nm = in.nm, sm = (int)in.sm;
  const int nwg = in.res_nwg;
  const int bx = wg % in.res_bx, bq = wg / in.res_bx;
  const int by = ND == 3 ? bq % in.res_by : 0, bm = ND == 3 ? bq / in.res_by : bq;
  const int ox = bx * TX, oy = by * TY, om = bm * TM;
  T *tile = (T *)dyn;                             // p of the box and its ring
  const int spare = CC ? PS * (TM + 2) : 0;       // where lanes without a ring cell write (a corner, unless it is one)
  T *const qbox = tile + (size_t)PS * (TM + 2) + (CC ? kResSpare : 0);  // q of the box, [j][lane]
  T *const qown = qbox + threadIdx.x;
  double *tileP = dyn;                            // the outer step's P, over both

  // this lane's cells
  const int tx = t % TX, tr = t / TX;
  const int ty = ND == 3 ? tr % TY : 0, g = ND == 3 ? tr / TY : tr;
  const bool act = g < G;
  const int m0 = om + g * R;
  const bool inxy = act && ox + tx < nx && oy + ty < ny;
  const int c0 = inxy ? ox + tx + (oy + ty) * nx + m0 * sm : 0;
  const int i0 = act ? (g * R + 1) * PS + (ND == 3 ? (ty + 1) * SX : 0) + tx + 1
                     : PS + (ND == 3 ? SX : 0) + 1;  // lanes without cells read inside the tile and use nothing
  const PI_G uint32_t *gcode = (const PI_G uint32_t *)in.code;
  PI_G double *gP = (PI_G double *)in.P[gst->Pcur];
  const PI_G double *gS = (const PI_G double *)in.S64;
  PI_G u64 *const words = (PI_G u64 *)in.res_x;  // of the tag's parity: sums, then face cells
  const int64_t half = in.res_words;
  // counter codes: a 3-D one is a word, two 2-D ones share one
  constexpr int kPack = ND == 2 ? 2 : 1;
  uint32_t codes[N / kPack];
  auto code_of = [&](int j) -> uint32_t {
    const uint32_t c = fresh(codes[j / kPack]);
    return kPack == 1 ? c : (c >> (16 * (j & 1))) & 0xffffu;
  };
  // the cell-centred scheme's are numbers of the plan's distinct ring codes:
  // 0 no data, 1 all of the ring holds data
  constexpr uint32_t kData = CC ? 0xffffu : ND == 2 ? 1u << 15 : kValidBit;
  constexpr uint32_t kInterior = CC ? 1u : ND == 2 ? (interior_code<2>() & 0xfffu) | kData : interior_code<ND>();
  const PI_G uint16_t *gpat = (const PI_G uint16_t *)in.res_pat;
  uint32_t have = 0, usual_rows = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const bool e = inxy && j < R && m0 + j < nm;
    uint32_t cd = 0u;
    if (e) cd = CC ? (uint32_t)gpat[c0 + j * sm] : gcode[c0 + j * sm];
    if (ND == 2 && !CC) cd = (cd & 0xfffu) | (cd >> 31 << 15);
    if (kPack == 1 || (j & 1) == 0) codes[j / kPack] = cd;
    else codes[j / kPack] |= cd << 16;
    if (e) have |= 1u << j;
  }
  // a lane's usual code, that of its middle cell, and the rows of cells in
  // which the whole wave has it (cells without data get q = 0 whatever their
  // weights): inside the grid and along its x edges, all rows
  uint32_t usual = kInterior;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const uint32_t cd = code_of(j);
    if (j <= R / 2 && cd != 0u) usual = cd;
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const uint32_t cd = code_of(j);
    if (__all(cd == usual || cd == 0u)) usual_rows |= 1u << j;
  }
  usual_rows = __builtin_amdgcn_readfirstlane(usual_rows);

  // this lane's ring cells: faces along the march axis, then y (3-D), then x,
  // the lower of an axis first; ring cells outside the grid hold 0.  A box's
  // face cells lie in the exchange buffer in the same order, so a ring cell is
  // the word at its place on the opposite face of the box beyond.
  int hw[HJ];          // ring cell: word to read (-1: outside the grid)
  uint32_t hf[HJ];     // its place in the tile (16 bits; `spare`: none), the face cell's in qbox
                       // (14 bits), bit 31: the face cell is wanted
  const int ring0 = (t + kRB - 256) & (kRB - 1);  // first of this lane's ring cells, kRB apart
  const int word0 = wg * res_ring(in) + ring0;
  T rh[HJ], ph[HJ], dh[HJ];
  double Ph[HJ];
  {
    const int A = TX * TY, B = ND == 3 ? TX * TM : 0, C = TY * TM, H = res_ring(in);
#pragma unroll
    for (int i = 0; i < HJ; ++i) {
      const int h = ring0 + kRB * i;
      int lx = 0, ly = 0, lm = 0, u, size, stride;
      bool low;
      const int sides = 2 * (A + B + C);
      if (h < 2 * A) {
        low = h < A;
        u = low ? h : h - A;
        lx = u % TX;
        ly = u / TX;
        lm = low ? -1 : TM;
        size = A;
        stride = in.res_bx * (ND == 3 ? in.res_by : 1);
      } else if (h < 2 * (A + B)) {
        u = h - 2 * A;
        low = u < B;
        u = low ? u : u - B;
        lx = u % TX;
        lm = u / TX;
        ly = low ? -1 : TY;
        size = B;
        stride = in.res_bx;
      } else if (CC && h >= sides) {
        // corners, opposite ones three places apart in sum
        u = h - sides;
        low = true;
        lx = (u & 1) ? TX : -1;
        lm = (u & 2) ? TM : -1;
        size = 3 - 2 * u;
        stride = ((u & 1) ? -1 : 1) + ((u & 2) ? -in.res_bx : in.res_bx);
      } else {
        u = h - 2 * (A + B);
        low = u < C;
        u = low ? u : u - C;
        ly = u % TY;
        lm = u / TY;
        lx = low ? -1 : TX;
        size = C;
        stride = 1;
      }
      const bool ok = h < H;
      auto in_grid = [&](int x, int y, int m) {
        return ok && ox + x >= 0 && ox + x < nx && oy + y >= 0 && oy + y < ny && om + m >= 0 && om + m < nm;
      };
      const bool e = in_grid(lx, ly, lm);
      hw[i] = e ? (wg + (low ? -stride : stride)) * H + (low ? h + size : h - size) : -1;
      Ph[i] = e ? gP[ox + lx + (oy + ly) * nx + (om + lm) * sm] : 0.0;
      // the box's own cell next to it, wanted where the box beyond exists
      const int fx = min(max(lx, 0), TX - 1), fy = min(max(ly, 0), TY - 1), fm = min(max(lm, 0), TM - 1);
      const uint32_t at_tile = ok ? (lm + 1) * PS + (ND == 3 ? (ly + 1) * SX : 0) + lx + 1 : spare;
      const uint32_t at_q = ok ? (fm % R) * kRB + fx + TX * (fy + TY * (fm / R)) : 0;
      hf[i] = at_tile | at_q << 16 | (e && in_grid(fx, fy, fm) ? 1u << 31 : 0u);
      rh[i] = ph[i] = dh[i] = T(0);
    }
  }

  // weights: [W^{n+1}] from the plan's table, the fixed point's operator
  // from the face totals; state 0 (no data) has weight 0.  Cell-centred: both
  // by ring code, with a bit per neighbour that holds data.
  T(*lut)[kStates] = (T(*)[kStates])sh.lut;
  T(*pat)[8] = (T(*)[8])((char *)dyn + in.res_tab);
  uint8_t *has = (uint8_t *)(pat + in.res_npat);
  if constexpr (CC) {
    for (int i = t; i < in.res_npat * 8; i += kRB) pat[i / 8][i % 8] = (T)in.res_wt[i];
    for (int i = t; i < in.res_npat; i += kRB) has[i] = in.res_has[i];
    __syncthreads();
  } else {
    for (int i = t; i < 6 * kStates; i += kRB) {
      const int d = i / kStates, s = i % kStates;
      lut[d][s] = OPL ? (s ? (T)in.a[d] : T(0)) : (T)in.lut_np1[d][s];
    }
  }
  T wi[NB];
#pragma unroll
  for (int d = 0; d < NB; ++d) {
    if constexpr (CC) {
      wi[d] = pat[usual][d];
    } else {
      const int s = dstate(usual, d, kBits);
      wi[d] = OPL ? (s ? (T)in.a[d] : T(0)) : (T)in.lut_np1[d][s];
    }
  }
  if (t < NB) sh.a[t] = CC ? in.cc_a[t] : in.a[t];

  if (t == 0) {
    sh.st = *gst;
    sh.end = sh.abort = 0;
  }
  __syncthreads();
  bool resume = sh.st.have_delta != 0;  // a later launch of the same solve: its next residual has been judged
  uint32_t tag = (uint32_t)sh.st.tag;

  constexpr bool kQ = N * sizeof(T) <= 32;  // q in registers too
  T p[N], r[N], d[N], q[kQ ? N : 1];
  double Pr[kHold ? N : 1], Sr[kHold ? N : 1];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    p[j] = r[j] = d[j] = T(0);
    if constexpr (kHold) {
      const bool e = (have >> j) & 1u;
      Pr[j] = e ? gP[c0 + j * sm] : 0.0;
      Sr[j] = e ? gS[c0 + j * sm] : 0.0;
    }
  }

  // One synchronisation: partial sums v to totals, ring values of `tag`
  // into hv (if wanted), scalars by wave 0.  OUTER: the outer step's scalars.
  auto sync = [&](const double (&v)[4], bool ring, T (&hv)[HJ], auto outer) {
    PI_G u64 *const slots = words + ((tag & 1) ? half : 0), *const X = slots + 8 * (nwg + kResGroups);
    const double ws = wave_sum4(v);
    if ((lane & 15) == 0) sh.wred[wave * 4 + sum_of_row(lane)] = ws;
    __syncthreads();
    if constexpr (decltype(outer)::value) {
      // the residual on the box's faces, through the LDS that P has left
      if (ring) {
#pragma unroll
        for (int j = 0; j < N; ++j)
          if (j < fresh_s(R)) qown[j * kRB] = r[j];
        __syncthreads();
      }
    }
    bool late = false;
    if (ring) {
#pragma unroll
      for (int i = 0; i < HJ; ++i)
        if (hf[i] >> 31) put_value<T>(X, word0 + kRB * i, tag, qbox[hf[i] >> 16 & 0x3fff]);
    }
    if (wave == 0) {
      double tot = sum_mod4(sh.wred[lane]);
      if (nwg > 1) {
        put4(slots + wg * 8, tot, tag, lane);
        if (nwg <= 64) {
          tot = gather4(slots, nwg, tag, lane, &sh.abort, late);
        } else {
          // two hops: the first workgroup of every kResGroup adds its group's
          // sums and publishes them, all add the groups'
          const int g0 = wg / kResGroup * kResGroup;
          if (wg == g0) {
            tot = gather4(slots + g0 * 8, min(kResGroup, nwg - g0), tag, lane, &sh.abort, late);
            put4(slots + (nwg + wg / kResGroup) * 8, tot, tag, lane);
          }
          tot = gather4(slots + nwg * 8, (nwg + kResGroup - 1) / kResGroup, tag, lane, &sh.abort, late);
        }
      }
      double s[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] = lane_value(tot, i);
      if constexpr (decltype(outer)::value) {
        if (lane == 0) {
          if (!resume) outer_scalars(in, &sh.st, s);
          sh.end = sh.st.done;
        }
      } else {
        const CgScalars cs = cg_scalars(in, &sh.st, s);
        if (lane == 0) {
          sh.al = cs.al;
          sh.be = cs.be;
          if (OPL) sh.end = cs.stop ? 1 : 0;
        }
      }
    }
    if (ring) {
#pragma unroll
      for (int i = 0; i < HJ; ++i) {
        hv[i] = T(0);
        if (hw[i] < 0) continue;
        Wait wait;
        while (!get_value<T>(X, hw[i], tag, hv[i])) {
          if (wait.over(&sh.abort)) {
            late = true;
            break;
          }
        }
      }
    }
    if (late) sh.abort = 1;
    __syncthreads();
  };
  auto next_tag = [&] { tag = res_next_tag(tag); };

  bool pending = false;  // p, d and alpha of an inner solve wait to be added to P
  T at = T(0);
  const int K = in.inner_iters;
  const int chunk = max(1, syncs / (K + 1));
  int steps = 0;
  bool aborted = false;
  for (;;) {
    // outer step: P <- P + delta, r = S - (M - N) P (as k_outer)
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const uint32_t mine = fresh(have);
    const int Rn = fresh_s(R);
    const int io = fresh(i0), co = fresh(c0);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (j >= fresh_s(R)) continue;  // uniform
      const bool e = (mine >> j) & 1u;
      double P;
      if constexpr (kHold) P = Pr[j];
      else P = e ? gP[co + j * sm] : 0.0;
      const double dl = pending ? (double)fma_t(at, p[j], d[j]) : 0.0;
      P += dl;
      acc[2] += dl * dl;
      acc[3] += P * P;
      if constexpr (kHold) Pr[j] = P;
      else if (e && pending) gP[co + j * sm] = P;
      if (act) tileP[io + j * PS] = P;
    }
#pragma unroll
    for (int i = 0; i < HJ; ++i) {
      if (pending) Ph[i] += (double)fma_t(at, ph[i], dh[i]);
      tileP[hf[i] & 0xffff] = Ph[i];
    }
    __syncthreads();
    next_tag();
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (j >= fresh_s(R)) continue;
      const int o = io + j * PS;
      const uint32_t cd = code_of(j);
      double L = 0.0;
      const double vC = tileP[o], vB = tileP[o - PS], vF = tileP[o + PS];
      const double vW = tileP[o - 1], vE = tileP[o + 1];
      if constexpr (CC) {
        const uint32_t hb = has[cd];
        const double nb[8] = {vE, vW, vF, vB, tileP[o + PS + 1], tileP[o + PS - 1], tileP[o - PS + 1], tileP[o - PS - 1]};
#pragma unroll
        for (int k = 0; k < 8; ++k) L += ((hb >> k) & 1u ? sh.a[k] : 0.0) * (vC - nb[k]);
      } else {
        double w[2 * ND];
#pragma unroll
        for (int k = 0; k < 2 * ND; ++k) w[k] = dstate(cd, k, kBits) ? sh.a[k] : 0.0;
        L += w[DE] * (vC - vE);
        L += w[DW] * (vC - vW);
        if constexpr (ND == 3) {
          L += w[DN] * (vC - tileP[o + SX]);
          L += w[DS] * (vC - tileP[o - SX]);
          L += w[DF] * (vC - vF);
          L += w[DB] * (vC - vB);
        } else {
          L += w[DN] * (vC - vF);
          L += w[DS] * (vC - vB);
        }
      }
      double S;
      if constexpr (kHold) S = Sr[j];
      else S = ((mine >> j) & 1u) ? gS[co + j * sm] : 0.0;
      const double rr = (cd & kData) ? S - L : 0.0;
      r[j] = (T)rr;
      const double rt = (double)r[j];
      acc[0] += rr * rr;
      acc[1] += rt * rt;
      __builtin_amdgcn_sched_barrier(0);
    }
    T hv[HJ];
#pragma unroll
    for (int i = 0; i < HJ; ++i) hv[i] = T(0);  // a lone box's ring lies outside the grid
    sync(acc, nwg > 1, hv, std::true_type{});
    resume = false;
    if (sh.abort) {
      aborted = true;
      break;
    }
    if (__builtin_amdgcn_readfirstlane(sh.end) || steps >= chunk) break;
    ++steps;
    // inner CG from p_0 = r_0
#pragma unroll
    for (int j = 0; j < N; ++j) {
      p[j] = r[j];
      d[j] = T(0);
    }
#pragma unroll
    for (int i = 0; i < HJ; ++i) {
      rh[i] = ph[i] = hv[i];
      dh[i] = T(0);
    }
    int ran = 0;
    for (int k = 0;; ++k) {
      const int io = fresh(i0);
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (j < fresh_s(R) && act) tile[io + j * PS] = p[j];
#pragma unroll
      for (int i = 0; i < HJ; ++i)
        tile[hf[i] & 0xffff] = ph[i];
      __syncthreads();
      next_tag();
      const bool last = k + 1 >= K;
      const uint32_t rows = fresh_s(usual_rows);
      double s4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int j = 0; j < N; ++j) {
        if (j >= fresh_s(R)) continue;
        const int o = io + j * PS;
        const uint32_t cd = code_of(j);
        const T vC = p[j];
        const T vB = j > 0 ? p[j > 0 ? j - 1 : 0] : tile[o - PS];
        T vF = p[j + 1 < N ? j + 1 : j];
        if (j + 1 == N || j + 1 == fresh_s(R)) vF = tile[o + PS];
        const T vW = tile[o - 1], vE = tile[o + 1];
        T w[NB];
        if ((rows >> j) & 1u) {
#pragma unroll
          for (int n = 0; n < NB; ++n) w[n] = wi[n];
        } else {
#pragma unroll
          for (int n = 0; n < NB; ++n) {
            if constexpr (CC) w[n] = pat[cd][n];
            else w[n] = lut[n][dstate(cd, n, kBits)];
          }
        }
        T s = OPL ? T(0) : vC;
        auto term = [&](int n, T v) {
          if constexpr (OPL) s += w[n] * (vC - v);
          else s -= w[n] * v;
        };
        if constexpr (CC) {
          // E, W, N, S, then the diagonals
          term(0, vE);
          term(1, vW);
          term(2, vF);
          term(3, vB);
          term(4, tile[o + PS + 1]);
          term(5, tile[o + PS - 1]);
          term(6, tile[o - PS + 1]);
          term(7, tile[o - PS - 1]);
        } else if constexpr (ND == 3) {
          term(DE, vE);
          term(DW, vW);
          term(DN, tile[o + SX]);
          term(DS, tile[o - SX]);
          term(DF, vF);
          term(DB, vB);
        } else {
          term(DE, vE);
          term(DW, vW);
          term(DN, vF);
          term(DS, vB);
        }
        s = (cd & kData) ? s : T(0);
        if constexpr (kQ) q[j] = s;
        qown[j * kRB] = s;
        const double rd = (double)r[j], qd = (double)s;
        s4[0] += (double)vC * qd;
        s4[1] += rd * qd;
        s4[2] += qd * qd;
        s4[3] += rd * rd;
        if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // loads of four cells in flight, not of all: registers
      }
      sync(s4, nwg > 1 && !last, hv, std::false_type{});
      ++ran;
      at = (T)sh.al;
      const T be = (T)sh.be;
      if (last) break;
      if (OPL && __builtin_amdgcn_readfirstlane(sh.end)) break;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        T qj;
        if constexpr (kQ) qj = q[j];
        else qj = j < fresh_s(R) ? qown[j * kRB] : T(0);
        r[j] = fma_t(-at, qj, r[j]);
        d[j] = fma_t(at, p[j], d[j]);
        p[j] = fma_t(be, p[j], r[j]);
      }
#pragma unroll
      for (int i = 0; i < HJ; ++i) {
        rh[i] = fma_t(-at, hv[i], rh[i]);
        dh[i] = fma_t(at, ph[i], dh[i]);
        ph[i] = fma_t(be, ph[i], rh[i]);
      }
    }
    pending = true;
    if (t == 0) sh.st.stop_at = ran;
  }
  if constexpr (kHold) {
#pragma unroll
    for (int j = 0; j < N; ++j)
      if ((have >> j) & 1u) gP[c0 + j * sm] = Pr[j];
  }
  __syncthreads();
  if (aborted && t == 0) put(words + res_late_word(in), 1);
  if (wg == 0 && t == 0) {
    (void)res_late(sh.st, aborted);
    sh.st.tag = tag;
    *gst = sh.st;
  }
}

}  // namespace

template <typename T>
__global__ __launch_bounds__(kRB) void k_resident(const BlockEnt *tab, const Inst *__restrict__ insts, State *sts,
                                                  int syncs) {
  extern __shared__ double dyn[];
  __shared__ Shared sh;
  const BlockEnt e = tab[blockIdx.x];
  if (e.inst < 0) return;
  const Inst &in = insts[e.inst];
  State *st = sts + e.inst;
  if (st->done) return;  // the same for every workgroup of the grid: only its last launch sets it
  if (in.res_nwg > 1) {
    const u64 late = get((PI_G u64 *)in.res_x + res_late_word(in));
    if (late != 0) {  // of an earlier launch
      if (e.lb == 0 && threadIdx.x == 0) (void)res_late(*st, late);
      return;
    }
  }
  const bool opl = in.inner_op != 0;
#define PI_BOX(ND, N, HJ)                                                        \
  do {                                                                           \
    if (opl) solve_box<T, ND, N, HJ, true>(in, st, e.lb, syncs, sh, dyn);        \
    else solve_box<T, ND, N, HJ, false>(in, st, e.lb, syncs, sh, dyn);           \
  } while (0)
  if (in.cc) {
    if (in.res_n == 4) PI_BOX(9, 4, 1);
    else if (in.res_n == 8) PI_BOX(9, 8, 1);
    else if constexpr (sizeof(T) == 4) PI_BOX(9, 16, 1);
  } else if (in.ndim == 2) {
    if (in.res_n == 4) PI_BOX(2, 4, 1);
    else if (in.res_n == 8) PI_BOX(2, 8, 1);
    else if constexpr (sizeof(T) == 4) PI_BOX(2, 16, 1);
  } else {
    if (in.res_n == 4) PI_BOX(3, 4, kResRing3);
    else if constexpr (sizeof(T) == 4) PI_BOX(3, 8, kResRing3);
  }
#undef PI_BOX
}

hipError_t resident_setup() {
  static std::mutex mu;
  static bool ready[64] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> guard(mu);
  if (ready[dev]) return hipSuccess;
  for (const void *fn : {(const void *)k_resident<float>, (const void *)k_resident<double>})
    if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kResLds)) != hipSuccess) return e;
  // one empty cooperative launch: the runtime sets up its queue for them here
  // and not inside a solve
  BlockEnt none{-1, 0}, *tab = nullptr;
  if ((e = hipMalloc((void **)&tab, sizeof(none))) != hipSuccess) return e;
  e = hipMemcpy(tab, &none, sizeof(none), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = launch_resident(false, tab, nullptr, nullptr, 1, true, 0, 1, nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  (void)hipFree(tab);
  ready[dev] = e == hipSuccess;
  return e;
}

hipError_t launch_resident(bool fp64, const BlockEnt *tab, const Inst *insts, State *sts, int nwg, bool coop,
                           size_t lds, int syncs, hipStream_t s) {
  if (nwg <= 0) return hipSuccess;
  const void *fn = fp64 ? (const void *)k_resident<double> : (const void *)k_resident<float>;
  if (coop) {
    void *args[] = {(void *)&tab, (void *)&insts, (void *)&sts, (void *)&syncs};
    return hipLaunchCooperativeKernel(fn, dim3(nwg), dim3(kRB), args, (unsigned)lds, s);
  }
  if (fp64) k_resident<double><<<dim3(nwg), dim3(kRB), lds, s>>>(tab, insts, sts, syncs);
  else k_resident<float><<<dim3(nwg), dim3(kRB), lds, s>>>(tab, insts, sts, syncs);
  return hipGetLastError();
}

}  // namespace pi
