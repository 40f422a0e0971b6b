// Matrix-core kernels of the warm-start network's own layers for gfx950: the
// 3x3x3 convolution and its data gradient (k_conv3), its weight gradient
// (k_wgrad3), and the one-tap product of the transposed convolution (k_conv1).
// pi_unet.hip keeps the general kernels for every other shape of pu_conv and
// pu_conv_wgrad.
//
// A 3x3x3 layer reads every input 27 times.  The general kernel takes each
// tap's operand from memory anew (126 TFLOP/s on the last decoder stage of a
// 128^3 network); here a workgroup brings a box of positions with its rim of
// one cell into LDS once per 32 input channels and runs all taps from there.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pi_conv.h"

namespace pu {

namespace {

typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));

constexpr int kXcds = 8;

// Workgroup b runs on XCD b mod 8; logical block with every XCD sweeping one
// contiguous eighth of the boxes, so that rims are found in its own L2.
__device__ inline unsigned xcd_block(unsigned b, unsigned n) {
  const unsigned per = (n + kXcds - 1) / kXcds;
  return (b % kXcds) * per + b / kXcds;
}

// Boxes of positions: BZ x BY x BX of an (n, d, h, w) grid, x fastest.
struct Boxes {
  int tx, ty, tz, count;
};
inline Boxes boxes_of(int n, int d, int h, int w, int bz, int by, int bx) {
  Boxes b;
  b.tx = (w + bx - 1) / bx;
  b.ty = (h + by - 1) / by;
  b.tz = (d + bz - 1) / bz;
  b.count = n * b.tx * b.ty * b.tz;
  return b;
}
struct BoxAt {
  int n, z, y, x;
};
__device__ inline BoxAt box_at(const Boxes &b, int i) {
  BoxAt c;
  c.x = i % b.tx;
  i /= b.tx;
  c.y = i % b.ty;
  i /= b.ty;
  c.z = i % b.tz;
  c.n = i / b.tz;
  return c;
}
__device__ inline BoxAt box_after(const Boxes &b, BoxAt c) {
  if (++c.x < b.tx) return c;
  c.x = 0;
  if (++c.y < b.ty) return c;
  c.y = 0;
  if (++c.z < b.tz) return c;
  c.z = 0;
  ++c.n;
  return c;
}

// index in the caller's tap list of the tap (dz, dy, dx) in {-1, 0, 1}^3
struct TapList {
  int8_t of[27];
};
inline bool tap_list(const int8_t (*offs)[3], int taps, TapList &l) {
  if (taps != 27) return false;
  for (int i = 0; i < 27; ++i) l.of[i] = -1;
  for (int t = 0; t < 27; ++t) {
    for (int k = 0; k < 3; ++k)
      if (offs[t][k] < -1 || offs[t][k] > 1) return false;
    l.of[(offs[t][0] + 1) * 9 + (offs[t][1] + 1) * 3 + offs[t][2] + 1] = (int8_t)t;
  }
  for (int i = 0; i < 27; ++i)
    if (l.of[i] < 0) return false;
  return true;
}

// eight channels (16 bytes) of one cell, zero past c channels
template <bool VEC>
__device__ inline u4 load8(const uint16_t *p, int c) {
  if constexpr (VEC) return *(const u4 *)p;
  uint16_t t[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) t[e] = e < c ? p[e] : (uint16_t)0;
  u4 v;
  __builtin_memcpy(&v, t, 16);
  return v;
}

// ---------------------------------------------------------------------------
// 3x3x3 convolution
// ---------------------------------------------------------------------------
// y = act(sum over taps and channels of x w + b): D[co][pos] = W X with
// v_mfma_f32_16x16x32_bf16, so that a lane ends with four consecutive output
// channels of one position.  The 16 positions of a matrix tile are RY
// positions along y times RZ along z at ONE x: the tap's dx then selects
// another tile in registers instead of shifting one, and each tile read from
// LDS serves three taps (dx) and NF x 16 output channels.  A wave holds XF
// tiles along x, a workgroup four waves along z.
//
// Per (dz, dy) a wave reads XF + 2 tiles of 1 KB from LDS for 3 XF NF matrix
// instructions of 16 clocks: at XF = 8, NF = 2, 40 KB per CU for 3072 clocks
// of its four matrix cores.  Weights come from L1/L2 straight into registers,
// three taps (NF = 2) or one ahead.  Two workgroups share a CU, so one fills its box while
// the other computes.
//
// LDS: [z][x][y] cells of 32 channels (64 bytes), the 16-byte quarters of a
// cell permuted by its y so that eight consecutive y at one quarter touch
// every bank once.
struct Conv3 {
  ConvP c;
  TapList taps;
  Boxes boxes;
  int vec4;  // outputs are written four channels at a time
};

constexpr int kEnough = 200;  // workgroups: most of the 256 CUs

template <int NF, int XF, int RY>
__global__ __launch_bounds__(256, 2) void k_conv3(Conv3 a) {
  constexpr int RZ = 16 / RY, BZ = 4 * RZ;
  constexpr int XT = XF + 2, YT = RY + 2, ZT = BZ + 2, CELLS = XT * YT * ZT;
  __shared__ __attribute__((aligned(16))) unsigned char lds[CELLS * 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned blk = xcd_block(blockIdx.x, a.boxes.count);
  if (blk >= (unsigned)a.boxes.count) return;
  const BoxAt at_box = box_at(a.boxes, (int)blk);
  const int n = at_box.n, z0 = at_box.z * BZ, y0 = at_box.y * RY, x0 = at_box.x * XF;
  const int n0 = blockIdx.y * NF * 16;
  const Tens &X = a.c.x;
  const uint16_t *xs = X.p + (int64_t)n * X.d * X.h * X.w * X.ld + X.off;
  const int slabs = a.c.cin / 32;

  const int r = lane & 15, q = lane >> 4;  // position (or output channel) and channel quarter of this lane
  const int yl = r % RY, zl = wave * RZ + r / RY;
  int at[3];  // tile address of (dz = 0, dy, x = 0)
#pragma unroll
  for (int dy = 0; dy < 3; ++dy)
    at[dy] = (zl * XT * YT + yl + dy) * 64 + ((q ^ (((yl + dy) >> 1) & 3)) << 4);
  // weights [tap][cout][cin]: rows past cout repeat the last one, their results are not stored
  uint32_t wrow[NF];  // bytes
#pragma unroll
  for (int j = 0; j < NF; ++j) wrow[j] = 2u * (uint32_t)(min(n0 + 16 * j + r, a.c.cout - 1) * a.c.cin + 8 * q);
  const int wtap = a.c.cout * a.c.cin;
  auto weight = [&](int tap, int k0, int j) {
    // the tap and slab in a scalar base, the lane's row in a 32-bit offset
    const char *base = (const char *)(a.c.w + (int64_t)a.taps.of[tap] * wtap + k0);
    return __builtin_bit_cast(bf16x8, *(const u4 *)(base + wrow[j]));
  };

  f4 acc[XF][NF];
#pragma unroll
  for (int i = 0; i < XF; ++i)
#pragma unroll
    for (int j = 0; j < NF; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

  constexpr int AHEAD = NF == 2 ? 3 : 1;
  bf16x8 w[2 * AHEAD][NF];
  auto weights = [&](int t0, int k0) {
#pragma unroll
    for (int t = t0; t < t0 + AHEAD; ++t)
#pragma unroll
      for (int j = 0; j < NF; ++j) w[t % (2 * AHEAD)][j] = weight(t % 27, k0, j);
  };
  weights(0, 0);

  for (int s = 0; s < slabs; ++s) {
    const int k0 = 32 * s;
    if (s) __syncthreads();
    constexpr int CHUNKS = CELLS * 4, PER = (CHUNKS + 255) / 256, U = NF == 4 ? 6 : (PER + 1) / 2;
#pragma unroll 1
    for (int b = 0; b < PER; b += U) {
      u4 v[U];
      int dst[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = tid + 256 * (b + u);
        const int cell = i >> 2, c = i & 3;
        const int ly = cell % YT, lt = cell / YT, lx = lt % XT, lz = lt / XT;
        const int gz = z0 + lz - 1, gy = y0 + ly - 1, gx = x0 + lx - 1;
        dst[u] = i < CHUNKS ? cell * 64 + ((c ^ ((ly >> 1) & 3)) << 4) : -1;
        const bool in = i < CHUNKS && gz >= 0 && gz < X.d && gy >= 0 && gy < X.h && gx >= 0 && gx < X.w;
        v[u] = u4{0u, 0u, 0u, 0u};
        if (in) v[u] = *(const u4 *)(xs + ((gz * X.h + gy) * X.w + gx) * X.ld + k0 + 8 * c);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (dst[u] >= 0) *(u4 *)(lds + dst[u]) = v[u];
    }
    __syncthreads();
    // tiles of the next (dz, dy) are read while the matrix cores work on this one's
    bf16x8 xv[2][XT];
    auto tiles = [&](int g) {
#pragma unroll
      for (int i = 0; i < XT; ++i)
        xv[g & 1][i] = __builtin_bit_cast(bf16x8, *(const u4 *)(lds + at[g % 3] + (g / 3 * XT + i) * YT * 64));
    };
    tiles(0);
#pragma unroll
    for (int g = 0; g < 9; ++g) {
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const int t = 3 * g + dx;
        if (dx == 0 && g + 1 < 9) tiles(g + 1);
        if (t % AHEAD == 0 && t + AHEAD < 27) weights(t + AHEAD, k0);
        __builtin_amdgcn_sched_barrier(0);  // loads first, then the matrix instructions that hide them
#pragma unroll
        for (int i = 0; i < XF; ++i)
#pragma unroll
          for (int j = 0; j < NF; ++j)
            acc[i][j] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t % (2 * AHEAD)][j], xv[g & 1][i + dx], acc[i][j], 0, 0, 0);
      }
    }
    if (s + 1 < slabs) weights(0, k0 + 32);
  }

  const Tens &Y = a.c.y;
  const int gz = z0 + zl, gy = y0 + yl;
  if (gz >= a.c.md || gy >= a.c.mh) return;
  const int64_t yrow = (((int64_t)n * Y.d + gz) * Y.h + gy) * Y.w;
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    const int co = n0 + 16 * j + 4 * q;
    if (co >= a.c.cout) continue;
    float b[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = a.c.bias && co + e < a.c.cout ? a.c.bias[co + e] : 0.f;
#pragma unroll
    for (int i = 0; i < XF; ++i) {
      if (x0 + i >= a.c.mw) continue;
      const int64_t yi = (yrow + x0 + i) * Y.ld + Y.off + co;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = acc[i][j][e] + b[e];
        if (a.c.relu) v[e] = fmaxf(v[e], 0.f);
      }
      if (a.c.yfp32) {
        float *yf = (float *)Y.p + yi;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (co + e < a.c.cout) yf[e] = a.c.acc ? yf[e] + v[e] : v[e];
      } else if (a.vec4) {
        u2 *yp = (u2 *)(Y.p + yi);
        if (a.c.acc) {
          const u2 o = *yp;
          v[0] += bf2f((uint16_t)(o[0] & 0xffffu));
          v[1] += bf2f((uint16_t)(o[0] >> 16));
          v[2] += bf2f((uint16_t)(o[1] & 0xffffu));
          v[3] += bf2f((uint16_t)(o[1] >> 16));
        }
        *yp = u2{(uint32_t)f2bf(v[0]) | (uint32_t)f2bf(v[1]) << 16, (uint32_t)f2bf(v[2]) | (uint32_t)f2bf(v[3]) << 16};
      } else {
        uint16_t *yp = Y.p + yi;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (co + e < a.c.cout) yp[e] = f2bf(a.c.acc ? bf2f(yp[e]) + v[e] : v[e]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// one tap (the transposed convolution, one output parity at a time)
// ---------------------------------------------------------------------------
// Memory-bound (64 -> 32 channels at 64^3 into a 128^3 slice: 15 us a parity
// for 50 MB): 32 output channels' weights stay in registers, positions
// stream through them 16 at a time straight from memory (a position's 32
// channels are 64 contiguous bytes), kGroups groups in flight per wave.
constexpr int kGroups = 4;

template <int KS>
__global__ __launch_bounds__(256) void k_conv1(ConvP a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4, n0 = blockIdx.y * 32;
  bf16x8 w[KS][2];
#pragma unroll
  for (int k = 0; k < KS; ++k)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      w[k][j] = __builtin_bit_cast(
          bf16x8, *(const u4 *)(a.w + (int64_t)min(n0 + 16 * j + r, a.cout - 1) * a.cin + 32 * k + 8 * q));
  const int64_t p0 = ((int64_t)blockIdx.x * 4 + wave) * (16 * kGroups) + r;
  f4 acc[kGroups][2];
#pragma unroll
  for (int g = 0; g < kGroups; ++g)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[g][j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    u4 v[kGroups];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      const int64_t p = min(p0 + 16 * g, a.P - 1);
      v[g] = *(const u4 *)(a.x.p + p * a.x.ld + a.x.off + 32 * k + 8 * q);
    }
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[g][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[k][j], __builtin_bit_cast(bf16x8, v[g]), acc[g][j], 0, 0, 0);
  }
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int64_t p = p0 + 16 * g;
    if (p >= a.P) continue;
    int t = (int)p;  // fewer than 2^31 positions
    const int x = t % a.mw;
    t /= a.mw;
    const int y = t % a.mh;
    t /= a.mh;
    const int z = t % a.md, n = t / a.md;
    const int64_t cell = (((int64_t)n * a.y.d + z * a.sout + a.ooz) * a.y.h + y * a.sout + a.ooy) * a.y.w +
                         x * a.sout + a.oox;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int co = n0 + 16 * j + 4 * q;
      if (co >= a.cout) continue;  // cout is a multiple of 4
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = acc[g][j][e] + (a.bias ? a.bias[co + e] : 0.f);
        if (a.relu) v[e] = fmaxf(v[e], 0.f);
      }
      *(u2 *)(a.y.p + cell * a.y.ld + a.y.off + co) =
          u2{(uint32_t)f2bf(v[0]) | (uint32_t)f2bf(v[1]) << 16, (uint32_t)f2bf(v[2]) | (uint32_t)f2bf(v[3]) << 16};
    }
  }
}

// ---------------------------------------------------------------------------
// weight gradient of the 3x3x3 convolution
// ---------------------------------------------------------------------------
// dw[t][ci][co] = sum over positions of x[p + t][ci] g[p][co]: positions are
// the contraction, so both operands are read from LDS transposed
// (ds_read_b64_tr_b16: of a block of 4 positions x 16 channels each lane gets
// one channel's four positions), from cells stored channels-last as in
// memory; a tap is then an offset of whole cells.  A workgroup takes 32 input
// by 32 output channels and a part of the boxes, one wave for each of the
// nine (dz, dy); the 32 positions of a matrix step are RY along y times RZ
// along z at one x, so a column of x meets three columns of g (dx), and each
// operand is read from LDS once for all of them: 4 KB per 12 matrix
// instructions.  Accumulators stay in registers over all boxes of the part,
// and the next box's loads are on their way while this one is worked on.
//
// Measured, 64 x 32 channels over 2^20 positions (116 GFLOP), with the sums of
// the parts, calls back to back: 170 us (680 TFLOP/s); the general kernel took
// about 1.9 ms.  Two workgroups per CU with half the registers and no loads
// ahead took 17 % longer.
//
// LDS: cells of 64 bytes; their 32-byte halves are swapped by bit 3 of y (x)
// and of the position's number (g), so that the two groups of 16 lanes that
// are served together read different banks.
struct Wgrad3 {
  WgP g;
  TapList taps;
  Boxes boxes;
  int nsplit, cts;
};

typedef __attribute__((address_space(3))) s4 lds_s4;
__device__ inline bf16x8 read_tr(const unsigned char *p) {
  const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)p);
  const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(p + 4 * 64));
  const s8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, v);
}

constexpr int kWgThreads = 640;  // nine waves of taps, one for the bias

template <int RY, bool XVEC>
__global__ __launch_bounds__(kWgThreads, 3) void k_wgrad3(Wgrad3 a) {
  constexpr int RZ = 32 / RY, XF = 8, XT = XF + 2, YT = RY + 2, ZT = RZ + 2, CELLS = XT * YT * ZT;
  __shared__ __attribute__((aligned(16))) unsigned char xl[CELLS * 64];
  __shared__ __attribute__((aligned(16))) unsigned char gl[XF * 32 * 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int split = blockIdx.x, ci0 = (blockIdx.y / a.cts) * 32, co0 = (blockIdx.y % a.cts) * 32;
  const Tens &X = a.g.x, &G = a.g.g;
  const int dz = wave / 3, dy = wave % 3;
  const int j = lane & 15, q = lane >> 4;
  // position 8 q + j / 4 of a step (and the one four further), channels 4 (j % 4)
  const int k = 8 * q + (j >> 2), yk = k % RY, zk = k / RY;
  // four positions further along y the half may change: two addresses
  auto x_at = [&](int z, int y, int half) {
    return (z * XT * YT + y) * 64 + ((half ^ ((y >> 3) & 1)) << 5) + ((j & 3) << 3);
  };
  int xa[2][2];
  // Positions past the grid's end have g = 0, but an infinite x of a cell inside
  // it times that 0 would be NaN.  So past its last row and plane (zs, ys: those
  // of the box that are the grid's) a position reads x at its own place, where
  // it is 0, whatever the tap; and the grid's last column of x does not meet the
  // column of g after it.  This costs 0 to 2 % of the time; masking x in
  // registers instead cost 6 %.
  auto x_rows = [&](int zs, int ys) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const bool past = zk >= zs || yk + 4 * i >= ys;
      xa[0][i] = x_at(zk + (past ? 1 : dz), yk + 4 * i + (past ? 1 : dy), 0);
      xa[1][i] = xa[0][i] ^ 32;
    }
  };
  int ga[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) ga[h] = k * 64 + ((h ^ (q & 1)) << 5) + ((j & 3) << 3);
  auto read_x = [&](int h, int col) {
    const s4 u = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(xl + xa[h][0] + col * YT * 64));
    const s4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(xl + xa[h][1] + col * YT * 64));
    const s8 w = {u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]};
    return __builtin_bit_cast(bf16x8, w);
  };

  const int beg = (int)((int64_t)a.boxes.count * split / a.nsplit);
  const int end = (int)((int64_t)a.boxes.count * (split + 1) / a.nsplit);
  constexpr int XC = CELLS * 4, GC = XF * 32 * 4;  // 16-byte pieces of a box
  constexpr int XP = (XC + kWgThreads - 1) / kWgThreads, GP = (GC + kWgThreads - 1) / kWgThreads;
  u4 v[XP + GP];
  // a box into registers, zero outside the grid ...
  auto load = [&](BoxAt at) {
    const int n = at.n, z0 = at.z * RZ, y0 = at.y * RY, x0 = at.x * XF;
    const uint16_t *xs = X.p + (int64_t)n * X.d * X.h * X.w * X.ld + X.off + ci0;
    const uint16_t *gs = G.p + (int64_t)n * G.d * G.h * G.w * G.ld + G.off + co0;
    int ft = tid;  // opaque: otherwise every piece's place is kept in registers over the boxes
    asm volatile("" : "+v"(ft));
#pragma unroll
    for (int u = 0; u < XP; ++u) {
      const int i = ft + kWgThreads * u, cell = i >> 2, c = i & 3;
      const int ly = cell % YT, lt = cell / YT, lx = lt % XT, lz = lt / XT;
      const int gz = z0 + lz - 1, gy = y0 + ly - 1, gx = x0 + lx - 1;
      v[u] = u4{0u, 0u, 0u, 0u};
      if (i < XC && gz >= 0 && gz < X.d && gy >= 0 && gy < X.h && gx >= 0 && gx < X.w && ci0 + 8 * c < a.g.cin)
        v[u] = load8<XVEC>(xs + ((gz * X.h + gy) * X.w + gx) * X.ld + 8 * c, a.g.cin - ci0 - 8 * c);
    }
#pragma unroll
    for (int u = 0; u < GP; ++u) {
      const int i = ft + kWgThreads * u, cell = i >> 2, c = i & 3, kk = cell % 32;
      const int gz = z0 + kk / RY, gy = y0 + kk % RY, gx = x0 + cell / 32;
      v[XP + u] = u4{0u, 0u, 0u, 0u};
      if (i < GC && gz < G.d && gy < G.h && gx < G.w)
        v[XP + u] = *(const u4 *)(gs + ((gz * G.h + gy) * G.w + gx) * G.ld + 8 * c);
    }
  };
  // ... from there into LDS, and the loads of the next box on their way;
  // returns where the box in LDS is
  BoxAt ahead = box_at(a.boxes, beg);
  auto next = [&](int b) {
    const BoxAt at = ahead;
    if (b != beg) __syncthreads();
    int ft = tid;
    asm volatile("" : "+v"(ft));
#pragma unroll
    for (int u = 0; u < XP; ++u) {
      const int i = ft + kWgThreads * u, cell = i >> 2, c = i & 3, ly = cell % YT;
      if (i < XC) *(u4 *)(xl + cell * 64 + (((c >> 1) ^ ((ly >> 3) & 1)) << 5) + ((c & 1) << 4)) = v[u];
    }
#pragma unroll
    for (int u = 0; u < GP; ++u) {
      const int i = ft + kWgThreads * u, cell = i >> 2, c = i & 3, kk = cell % 32;
      if (i < GC) *(u4 *)(gl + cell * 64 + (((c >> 1) ^ ((kk >> 3) & 1)) << 5) + ((c & 1) << 4)) = v[XP + u];
    }
    __syncthreads();
    ahead = box_after(a.boxes, at);
    if (b + 1 < end) load(ahead);
    return at;
  };
  if (beg < end) load(ahead);

  if (wave == 9) {
    // g does not depend on the tap: the tenth wave sums it for the bias, as a product with ones
    const bool bias = a.g.bpart != nullptr && ci0 == 0;
    const s8 one_bits = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
    const bf16x8 ones = __builtin_bit_cast(bf16x8, one_bits);
    f4 sum[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
    for (int b = beg; b < end; ++b) {
      next(b);
      if (!bias) continue;
#pragma unroll 1
      for (int col = 0; col < XF; ++col)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          sum[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, read_tr(gl + col * 32 * 64 + ga[h]), sum[h], 0, 0, 0);
    }
    if (bias && q == 0) {
#pragma unroll
      for (int h = 0; h < 2; ++h) a.g.bpart[(int64_t)split * a.g.cout + co0 + 16 * h + j] = sum[h][0];
    }
    return;
  }
  f4 acc[3][2][2];
#pragma unroll
  for (int d = 0; d < 3; ++d)
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[d][m][h] = f4{0.f, 0.f, 0.f, 0.f};
  for (int b = beg; b < end; ++b) {
    const BoxAt at = next(b);
    const int last = G.w - 1 - at.x * XF;
    x_rows(G.d - at.z * RZ, G.h - at.y * RY);
    // column col of x (from -1) meets columns col - dx of g; one half of x's
    // channels at a time
    bf16x8 gw[3][2], xv[2];
    xv[0] = read_x(0, 0);
#pragma unroll
    for (int col = -1; col <= XF; ++col) {
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        // reads first: they land while the matrix cores work on what is there
        if (m == 0) xv[1] = read_x(1, col + 1);
        else if (col < XF) xv[0] = read_x(0, col + 2);
        if (m == 0 && col + 1 < XF) {
#pragma unroll
          for (int h = 0; h < 2; ++h) gw[(col + 1) % 3][h] = read_tr(gl + (col + 1) * 32 * 64 + ga[h]);
        }
#pragma unroll
        for (int dx = 1; dx >= -1; --dx) {
          const int gc = col - dx;
          if (gc < 0 || gc >= XF) continue;
          if (dx == -1 && col >= 0 && col == last) continue;  // uniform
#pragma unroll
          for (int h = 0; h < 2; ++h)
            acc[dx + 1][m][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[m], gw[gc % 3][h], acc[dx + 1][m][h], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  float *out = a.g.part + (int64_t)split * 27 * a.g.cin * a.g.cout;
#pragma unroll
  for (int dx = 0; dx < 3; ++dx) {
    float *ot = out + (int64_t)a.taps.of[dz * 9 + dy * 3 + dx] * a.g.cin * a.g.cout;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ci = ci0 + 16 * m + 4 * q + e;
        if (ci >= a.g.cin) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) ot[(int64_t)ci * a.g.cout + co0 + 16 * h + j] = acc[dx][m][h][e];
      }
  }
}

inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// offsets inside a sample stay below 2^31 elements
inline bool small_sample(const Tens &t) { return (int64_t)t.d * t.h * t.w * t.ld < (int64_t(1) << 31); }

}  // namespace

bool conv_fast(const ConvP &a, hipStream_t s) {
  if (a.cin % 32 || a.x.ld % 8 || a.x.off % 8 || !aligned16(a.x.p) || !aligned16(a.w) || !small_sample(a.x) ||
      (int64_t)a.taps * a.cin * a.cout >= (int64_t(1) << 31) || a.sin != 1)
    return false;
  const bool y4 = a.y.ld % 4 == 0 && a.y.off % 4 == 0 && a.cout % 4 == 0 && ((uintptr_t)a.y.p & 7) == 0;
  const bool same_x = a.x.d == a.md && a.x.h == a.mh && a.x.w == a.mw;
  if (a.taps == 1) {
    if (!same_x || a.offs[0][0] || a.offs[0][1] || a.offs[0][2] || !y4 || a.yfp32 || a.acc ||
        a.P >= (int64_t(1) << 31))
      return false;
    const dim3 grid((unsigned)((a.P + 64 * kGroups - 1) / (64 * kGroups)), (a.cout + 31) / 32);
    switch (a.cin) {
      case 32: k_conv1<1><<<grid, 256, 0, s>>>(a); return true;
      case 64: k_conv1<2><<<grid, 256, 0, s>>>(a); return true;
      case 128: k_conv1<4><<<grid, 256, 0, s>>>(a); return true;
      case 256: k_conv1<8><<<grid, 256, 0, s>>>(a); return true;
    }
    return false;
  }
  Conv3 c;
  if (!same_x || a.sout != 1 || a.ooz || a.ooy || a.oox || !tap_list(a.offs, a.taps, c.taps)) return false;
  c.c = a;
  c.vec4 = y4;
  // 16 or 8 positions along y per matrix tile: whichever leaves fewer lanes outside the grid
  auto padded = [&](int ry) {
    const int bz = 64 / ry;
    return (int64_t)((a.md + bz - 1) / bz * bz) * ((a.mh + ry - 1) / ry * ry);
  };
  const bool wide = padded(16) <= padded(8);
  const int ry = wide ? 16 : 8;
  // eight tiles along x and 64 output channels per wave reuse LDS and weights
  // most; smaller grids take fewer until there are enough workgroups
  auto groups = [&](int xf, int nf) {
    return (int64_t)boxes_of(a.x.n, a.md, a.mh, a.mw, 64 / ry, ry, xf).count * ((a.cout + 16 * nf - 1) / (16 * nf));
  };
  const int nf = a.cout > 32 && groups(8, 4) >= kEnough ? 4 : 2;
  const int xf = groups(8, nf) >= kEnough ? 8 : groups(4, nf) >= kEnough ? 4 : 2;
  c.boxes = boxes_of(a.x.n, a.md, a.mh, a.mw, 64 / ry, ry, xf);
  const dim3 grid((unsigned)((c.boxes.count + kXcds - 1) / kXcds * kXcds), (a.cout + 16 * nf - 1) / (16 * nf));
#define PU_GO(NF, XF)                                              \
  do {                                                             \
    if (wide) k_conv3<NF, XF, 16><<<grid, 256, 0, s>>>(c);         \
    else k_conv3<NF, XF, 8><<<grid, 256, 0, s>>>(c);               \
  } while (0)
  if (nf == 4) PU_GO(4, 8);
  else if (xf == 8) PU_GO(2, 8);
  else if (xf == 4) PU_GO(2, 4);
  else PU_GO(2, 2);
#undef PU_GO
  return true;
}

bool wgrad_fast(const WgP &a, int nsplit, hipStream_t s) {
  Wgrad3 w;
  const bool same = a.x.d == a.md && a.x.h == a.mh && a.x.w == a.mw && a.g.d == a.md && a.g.h == a.mh && a.g.w == a.mw;
  if (!same || a.sin != 1 || a.sout != 1 || a.ooz || a.ooy || a.oox || !tap_list(a.offs, a.taps, w.taps) ||
      a.cout % 32 || a.g.ld % 8 || a.g.off % 8 || !aligned16(a.g.p) || !small_sample(a.x) || !small_sample(a.g))
    return false;
  w.g = a;
  w.nsplit = nsplit;
  w.cts = a.cout / 32;
  const bool xvec = a.cin % 8 == 0 && a.x.ld % 8 == 0 && a.x.off % 8 == 0 && aligned16(a.x.p);
  auto padded = [&](int ry) {
    const int bz = 32 / ry;
    return (int64_t)((a.md + bz - 1) / bz * bz) * ((a.mh + ry - 1) / ry * ry);
  };
  const bool wide = padded(16) <= padded(8);
  const int ry = wide ? 16 : 8;
  w.boxes = boxes_of(a.x.n, a.md, a.mh, a.mw, 32 / ry, ry, 8);
  if (!wgrad_boxes_pay(w.boxes.count, a.P, nsplit, a.cin, a.cout)) return false;
  const dim3 grid((unsigned)nsplit, (unsigned)((a.cin + 31) / 32 * w.cts));
  if (wide && xvec) k_wgrad3<16, true><<<grid, kWgThreads, 0, s>>>(w);
  else if (wide) k_wgrad3<16, false><<<grid, kWgThreads, 0, s>>>(w);
  else if (xvec) k_wgrad3<8, true><<<grid, kWgThreads, 0, s>>>(w);
  else k_wgrad3<8, false><<<grid, kWgThreads, 0, s>>>(w);
  return true;
}

}  // namespace pu
