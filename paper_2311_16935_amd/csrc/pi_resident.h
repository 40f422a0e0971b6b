// Boxes of the on-chip solve (pi_resident.hip): sizes, and their choice.
#pragma once

#include <algorithm>
#include <vector>

#include "pi_common.h"

namespace pi {

// Tag of the synchronisation after that of tag t.  Words alternate between two
// buffers by tag parity, so after the last tag comes 2: 0 is never published,
// and 1 would use the last one's buffer again while others still read it.
__host__ __device__ inline uint32_t res_next_tag(uint32_t t) { return t == 0xffffffffu ? 2u : t + 1u; }

// A workgroup whose wait has lasted too long says so in the word after the
// exchange words of both parities (cleared with them when a solve starts).
// The next launch of the solve, and the sums of the gauge after the last, turn
// it into the solve's status: the workgroup that holds the state may have
// missed nothing itself and store any other.
inline __host__ __device__ int64_t res_late_word(const Inst &in) { return 2 * in.res_words; }
__host__ __device__ inline bool res_late(State &st, uint64_t word) {
  if (word == 0) return false;
  st.done = 1;
  st.status = 6;  // PI_ERR_DEVICE
  return true;
}

// Ring cells of a box: its faces along the march axis, y (3-D) and x, and its
// corners in the cell-centred scheme.
__host__ __device__ inline int res_ring(const Inst &in) {
  const int tm = in.res_g * in.res_r;
  return in.ndim == 3 ? 2 * (in.res_tx * in.res_ty + in.res_tx * tm + in.res_ty * tm)
                      : 2 * (in.res_tx + tm) + (in.cc ? 4 : 0);
}

// LDS bytes of a workgroup: the box and its ring of p followed by q of every
// lane's cells, or in their place P (FP64) of the box and its ring; after them
// the cell-centred scheme's weights and neighbour bits by ring code.
inline size_t res_boxes(const Inst &in, bool fp64) {
  const size_t sx = in.res_tx + 2, sy = in.ndim == 3 ? in.res_ty + 2 : 1;
  const size_t tile = sx * sy * ((size_t)in.res_g * in.res_r + 2) + (in.cc ? kResSpare : 0), t = fp64 ? 8 : 4;
  const size_t b = std::max(tile * sizeof(double), (tile + (size_t)kResBlock * in.res_r) * t);
  return in.cc ? (b + 15) / 16 * 16 : b;
}
inline size_t res_lds(const Inst &in, bool fp64) {
  return res_boxes(in, fp64) + (in.cc ? (size_t)in.res_npat * (8 * (fp64 ? 8 : 4) + 1) : 0);
}

// Microseconds of a pass of the on-chip solve, fitted to boxes of every shape:
// the cells of a lane (more each where they outgrow the registers), and the
// exchange -- one hop up to 64 workgroups, two beyond -- longer with the ring
// words a workgroup reads.
inline double res_cost(const Inst &in, int r, int ring, int nwg) {
  const double cell = (r > 8 ? 0.47 : 0.3) * (in.ndim == 3 || in.cc ? 1.3 : 1.0);
  const double wait = nwg == 1 ? 0.0 : nwg <= 64 ? 2.05 : 3.0 + 0.004 * nwg;
  return 0.45 + cell * r + wait + (nwg == 1 ? 0.0 : ring * (0.0004 + 0.0006 * nwg / 256.0));
}

// Boxes of a grid (the res_* sizes of Inst; res_nwg = 0 where it does not
// fit): the cheapest by res_cost of those that cut every axis into equal
// parts.  cus: CUs of the device.
inline void set_resident(Inst &in, bool fp64, int cus) {
  in.res_nwg = 0;
  if (in.bicg || (in.cc && in.res_npat == 0)) return;
  const int max_r = in.ndim == 2 ? (fp64 ? 8 : 16) : (fp64 ? 4 : 8);
  const int max_wg = std::min(cus, kResMaxWg);
  if (in.ncell > (int64_t)max_wg * kResBlock * max_r) return;
  const int ring_max = kResBlock * (in.ndim == 3 ? kResRing3 : 1);
  double best = 1e300;
  auto consider = [&](int tx, int ty, int g, int r) {
    const int64_t bx = (in.nx + tx - 1) / tx, by = (in.ndim == 3 ? (in.ny + ty - 1) / ty : 1);
    const int64_t tm = (int64_t)g * r, bm = (in.nm + tm - 1) / tm;
    if (bx * by * bm > max_wg) return;
    Inst c = in;
    c.res_tx = tx;
    c.res_ty = ty;
    c.res_g = g;
    c.res_r = r;
    const int ring = res_ring(c);
    if (ring > ring_max || res_lds(c, fp64) > (size_t)kResLds) return;
    const int nwg = (int)(bx * by * bm);
    const double cost = res_cost(in, r, ring, nwg);
    if (cost >= best) return;
    best = cost;
    in.res_nwg = nwg;
    in.res_n = r <= 4 ? 4 : r <= 8 ? 8 : 16;
    in.res_tx = tx;
    in.res_ty = ty;
    in.res_g = g;
    in.res_r = r;
    in.res_bx = (int)bx;
    in.res_by = (int)by;
    in.res_tab = (int)res_boxes(c, fp64);
  };
  for (int kx = 1; kx <= in.nx && kx <= max_wg; ++kx) {
    const int tx = (in.nx + kx - 1) / kx;
    if (tx > 256 || (tx < 16 && kx > 1)) continue;
    for (int ky = 1; ky <= (in.ndim == 3 ? in.ny : 1) && kx * ky <= max_wg; ++ky) {
      const int ty = in.ndim == 3 ? (in.ny + ky - 1) / ky : 1;
      if (tx * ty > kResBlock) continue;
      const int gmax = kResBlock / (tx * ty);
      for (int r = 1; r <= max_r; ++r) {
        // as few lane groups as cover the axis in the number of boxes that all groups would need
        const int bm = (in.nm + gmax * r - 1) / (gmax * r);
        const int g = (in.nm + bm * r - 1) / (bm * r);
        consider(tx, ty, g, r);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// batches: grids side by side on the chip, or streamed in one set of launches
// ---------------------------------------------------------------------------
// Grids that are solved on the chip, in the order they get there: the longest
// sides first (they take the most outer steps).
inline std::vector<int64_t> res_queue(const std::vector<Inst> &insts) {
  std::vector<int64_t> q;
  for (size_t i = 0; i < insts.size(); ++i)
    if (insts[i].res_nwg > 0) q.push_back((int64_t)i);
  auto side = [&](int64_t i) { return std::max({insts[i].nx, insts[i].ny, insts[i].nz}); };
  std::stable_sort(q.begin(), q.end(), [&](int64_t x, int64_t y) { return side(x) > side(y); });
  return q;
}

// Grids of a batch that go onto the chip next: from `todo` (in its order) into
// `on` whatever fits beside those there; wgs(i): workgroups of grid i.  False
// where nothing is on the chip then though grids wait.
template <class F>
inline bool res_admit(std::vector<int64_t> &todo, std::vector<int64_t> &on, int max_wg, F &&wgs) {
  int used = 0;
  for (int64_t i : on) used += wgs(i);
  for (auto it = todo.begin(); it != todo.end();) {
    if (used + wgs(*it) > max_wg) {
      ++it;
      continue;
    }
    used += wgs(*it);
    on.push_back(*it);
    it = todo.erase(it);
  }
  return !on.empty();
}

// Passes a grid is expected to take (their number enters both sides alike):
// about 16 outer steps per cell of the longest side, the fixed-point variant
// about 8 passes.
inline double batch_passes(const Inst &in) {
  const double side = std::max({in.nx, in.ny, in.nz}), per = in.inner_iters + 1.0;
  return std::min((double)in.max_iter * per, in.inner_op ? 8.0 * side : 16.0 * side * per);
}

// Microseconds of a pass on the chip as measured in batches: res_cost, which
// ranks one grid's boxes, is 20 % too high where two hops are taken, and too
// low for FP64, the cell-centred scheme and 3-D.
inline double batch_chip_us(const Inst &in, bool fp64) {
  return res_cost(in, in.res_r, res_ring(in), in.res_nwg) * (in.res_nwg > 64 ? 0.8 : 1.0) * (fp64 ? 1.2 : 1.0) *
         (in.cc ? 1.1 : in.ndim == 3 ? 1.1 : 1.0);
}

// Microseconds a grid adds to a streaming pass over many: per block, by cells
// per lane, for segments of four planes.  For every launch shape among the grids
// each pass takes kStreamUs besides, and the call kStreamStartUs to capture its
// graph.
constexpr double kStreamUs = 11.0, kStreamStartUs = 450.0;
inline double batch_stream_us(const Inst &in, bool fp64) {
  const int v = in.vw == 4 ? 2 : in.vw == 2 ? 1 : 0;
  constexpr double face[3] = {0.0065, 0.010, 0.020}, face64[3] = {0.009, 0.018, 0.045}, cell[3] = {0.0103, 0.018, 0.036};
  const double t = in.cc ? cell[v] * (fp64 ? 2.0 : 1.0) : fp64 ? face64[v] : face[v];
  return t * in.nblocks * in.mseg / 4.0;
}

// Where a batch had better stream than solve on the chip what fits there: every
// res_nwg is set to 0.  A grid's boxes are chosen for its own latency, with as
// few cells per lane as there are workgroups, so that grids of some 100^2 to
// 300^2 cells take turns on the device at one cell per lane, and many of them
// stream faster (24 outer steps, on the chip and streamed: 400 of 101^2 10.7
// and 7.0 ms, 300 of 300 x 200 78 and 53 ms, 300 of 1000 x 30 91 and 31 ms).
// Few of them, smaller ones (one workgroup each) and larger ones (more cells
// per lane) are faster on the chip (24 of 101^2 1.0 and 1.8 ms, 60 of 64^3 14
// and 49 ms), and so are batches of many launch shapes (200 with sides of 100 to
// 500: 43 and 54 ms).  Estimated, by the figures above, for the rounds on the
// chip and for passes over the same grids streamed (apart from those that
// stream anyway).  The estimates are rough (up to 40 % off); in each of some 60
// batches timed both ways they picked the faster one, or one 2 % slower at most.
inline void batch_routes(std::vector<Inst> &insts, bool fp64, int max_wg, int syncs) {
  std::vector<int64_t> todo = res_queue(insts), on;
  std::vector<double> left(insts.size());
  double longest = 0.0, stream = 0.0, chip = 0.0;
  bool shape[kShapes] = {};
  for (int64_t i : todo) {
    const Inst &in = insts[i];
    shape[shape_of(in.ndim, in.vw, in.gen, in.cc)] = true;
    left[i] = batch_passes(in);
    longest = std::max(longest, left[i]);
    stream += left[i] * batch_stream_us(in, fp64);
  }
  stream += (kStreamUs * longest + kStreamStartUs) * (double)std::count(shape, shape + kShapes, true);
  while (!todo.empty() || !on.empty()) {
    if (!res_admit(todo, on, max_wg, [&](int64_t i) { return insts[i].res_nwg; })) return;
    double us = 0.0;
    std::vector<int64_t> still;
    for (int64_t i : on) {
      const double run = std::min(left[i], (double)syncs);
      us = std::max(us, run * batch_chip_us(insts[i], fp64));
      left[i] -= run;
      if (left[i] > 0.0) still.push_back(i);
    }
    on.swap(still);
    chip += us + 40.0;  // a launch, and the host between two
    if (chip > stream) {
      for (Inst &in : insts) in.res_nwg = 0;
      return;
    }
  }
}

}  // namespace pi
