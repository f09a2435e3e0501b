// Post-transfer products of PPV cubes: Gaussian beam convolution over the two
// sky axes (paper, "Beam Convolution") and the l,v mean projection over one
// sky axis (the l,v panels of the paper's figures). Cubes are FP32
// [n1][n2][n_chan], channel fastest.
//
// The beam is separable. Up to kBeamFusedRadius pixels one kernel does both
// axes: it walks n1 row by row, convolves each row along n2 out of LDS and
// keeps the 2R + 1 output rows it reaches in registers, so the cube is read
// and written once. Wider beams, maps that leave it mostly halo (the rule is in
// iris_beam_convolve), and an output that overlaps the cube, take
// two passes, along n2 into a workspace and along n1 into the output: a lane
// computes a run of four consecutive positions along the pass axis for four
// channels (16-byte accesses when the rows allow it), so that the 2R + 1 taps
// of the run share 4 + 2R loads; each XCD takes a contiguous range of the
// work, so that rows re-read by neighbouring runs hit in its L2. Both ways are
// bound by HBM and sum the taps in the same order (equal results).

#include <hip/hip_runtime.h>

#include <cmath>

#include "device_util.h"
#include "host_common.h"

namespace iris {
namespace {

constexpr int kBeamMaxRadius = 128;

struct BeamArgs {
  const float* in;
  float* out;
  int64_t n1, n2, C;
  int32_t axis;  // 1: along n2 (stride C), 0: along n1 (stride n2 C)
  int32_t R;
  float w[kBeamMaxRadius + 1];  // w[|offset|], unit sum over -R..R
};

// Positions along the pass axis handled by one lane: the 2R + 1 taps of
// kBeamRun consecutive outputs share kBeamRun + 2R loads.
constexpr int kBeamRun = 4;

template <int V>
__global__ __launch_bounds__(256) void beam_pass_kernel(const BeamArgs a) {
  using T = typename std::conditional<V == 4, float4, float>::type;
  const int64_t nv = a.C / V;
  const int64_t n_axis = a.axis == 1 ? a.n2 : a.n1;
  const int64_t n_runs = (n_axis + kBeamRun - 1) / kBeamRun;
  const int64_t n_other = a.axis == 1 ? a.n1 : a.n2;
  const int64_t total = n_other * n_runs * nv;
  const int64_t stride = (a.axis == 1 ? a.C : a.n2 * a.C) / V;
  const T* in = (const T*)a.in;
  T* out = (T*)a.out;
  // One run of outputs per lane, columns fastest; each XCD takes a contiguous
  // range of the work, so that the rows a tap re-reads were loaded into the
  // same L2.
  const int64_t e = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int64_t col = e % nv, t = e / nv;
  const int64_t run = t % n_runs, other = t / n_runs;
  const int64_t pos0 = run * kBeamRun;
  // Element (p1, p2, col) sits at (p1 n2 + p2) nv + col.
  const int64_t e0 = (a.axis == 1 ? other * a.n2 + pos0 : pos0 * a.n2 + other) * nv + col;
  const int jlo = (int)max((int64_t)-a.R, -pos0);
  const int jhi = (int)min((int64_t)(kBeamRun - 1 + a.R), n_axis - 1 - pos0);
  float acc[kBeamRun][V] = {};
  for (int j = jlo; j <= jhi; ++j) {
    const T v = gload(in + e0 + j * stride);
#pragma unroll
    for (int m = 0; m < kBeamRun; ++m) {
      const int d = j - m < 0 ? m - j : j - m;
      if (d <= a.R) {
        const float w = a.w[d];
        if constexpr (V == 4) {
          acc[m][0] = fmaf(w, v.x, acc[m][0]);
          acc[m][1] = fmaf(w, v.y, acc[m][1]);
          acc[m][2] = fmaf(w, v.z, acc[m][2]);
          acc[m][3] = fmaf(w, v.w, acc[m][3]);
        } else {
          acc[m][0] = fmaf(w, v, acc[m][0]);
        }
      }
    }
  }
#pragma unroll
  for (int m = 0; m < kBeamRun; ++m) {
    if (pos0 + m < n_axis) {
      if constexpr (V == 4)
        gstore(out + e0 + m * stride, make_float4(acc[m][0], acc[m][1], acc[m][2], acc[m][3]));
      else
        gstore(out + e0 + m * stride, acc[m][0]);
    }
  }
}

// Both axes at once, R <= kBeamFusedRadius. A workgroup of nw wavefronts takes
// 32 channels (lane % 32), 8 nw positions along n2 (a run of four per half
// wavefront) and a segment of n1. Per row of n1 the 8 nw + 2R positions go to
// LDS, the next row's loads already in flight; each lane convolves its run
// along n2 (4 + 2R LDS reads for four outputs) and adds the result to the
// 2R + 1 output rows in reach, held oldest first: the sum of row k moves down
// to k - 1 in the multiply-add itself, so the window slides at no cost, and a
// finished row leaves at the bottom. Positions outside the map count as zero.
// Bound by HBM: 512 x 128 x 800, R = 5: two passes 320 us, this one 95 us
// (0.42 GB; the halos, (1 + 2R/64)(1 + 2R/segment), come from L2).
constexpr int kBeamFusedRadius = 12;
constexpr int kBeamCh = 32;     // channels of a workgroup
constexpr int kBeamPerWave = 8;  // positions along n2 per wavefront

// Wavefronts per SIMD that the window leaves: 2R + 1 rows of four FP32 sums
// (88, 124, 158 and 182 registers at R = 4, 7, 10 and 12).
__host__ __device__ constexpr int beam_waves(int R) {
  return R <= 4 ? 5 : R <= 7 ? 4 : R <= 10 ? 3 : 2;
}

template <int R>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(beam_waves(R)))) void
beam_fused_kernel(const BeamArgs a, int n_seg) {
  constexpr int kTaps = 2 * R + 1;
  extern __shared__ float rows[];  // [2][(positions + 2R)][kBeamCh]
  const int nw = (int)(blockDim.x >> 6);
  const int n1 = (int)a.n1, n2 = (int)a.n2, C = (int)a.C;
  const int t2 = nw * kBeamPerWave;  // positions of the workgroup
  const int held = t2 + 2 * R;       // with the halo
  const int n_ch = (C + kBeamCh - 1) / kBeamCh;
  // Channel blocks fastest: neighbouring workgroups share rows of the cube.
  const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
  const int cb = tile % n_ch, rest = tile / n_ch;
  const int seg = rest % n_seg, p2_0 = rest / n_seg * t2;
  const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
  const int ch = lane % kBeamCh, c = cb * kBeamCh + ch;
  const bool in_c = c < C;
  const int run = wave * kBeamPerWave + 4 * (lane / kBeamCh);  // first position of the lane's run
  // Segments differ by one row at most.
  const int m0 = (int)((int64_t)n1 * seg / n_seg), m1 = (int)((int64_t)n1 * (seg + 1) / n_seg);

  float w[R + 1];
#pragma unroll
  for (int i = 0; i <= R; ++i) w[i] = a.w[i];
  float acc[kTaps][4] = {};

  // Loads of one row by the whole workgroup: position h of the halo tile and
  // channel ch per lane, 2 nw positions per round.
  constexpr int kRounds = (kBeamPerWave + 2 * R + 1) / 2;  // nw >= 1
  float pre[kRounds];
  const int h0 = (int)threadIdx.x / kBeamCh, hs = 2 * nw;
  auto fetch = [&](int row) {
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
      if (k * hs >= held) break;  // wider workgroups take fewer rounds
      const int h = h0 + k * hs, p2 = p2_0 - R + h;
      const bool in = h < held && in_c && p2 >= 0 && p2 < n2;
      pre[k] = in ? gload(a.in + ((int64_t)row * n2 + p2) * C + c) : 0.f;
    }
  };
  // Rows before the map add nothing; those beyond it only move the window on.
  const int first = max(m0 - R, 0);
  fetch(first);
  for (int row = first, b = 0; row < m1 + R; ++row, b ^= 1) {
    // acc[k] is output row row - R + k after the shift: distance |R - k|.
    if (row < n1) {
      float* buf = rows + b * held * kBeamCh;
#pragma unroll
      for (int k = 0; k < kRounds; ++k) {
        if (k * hs >= held) break;
        const int h = h0 + k * hs;
        if (h < held) buf[h * kBeamCh + ch] = pre[k];
      }
      __syncthreads();  // also: the reads of this buffer two rows ago are done
      if (row + 1 < min(m1 + R, n1)) fetch(row + 1);
      float v[4] = {};
#pragma unroll
      for (int j = 0; j < 4 + 2 * R; ++j) {
        const float x = buf[(run + j) * kBeamCh + ch];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int d = j - R - m < 0 ? m + R - j : j - R - m;
          if (d <= R) v[m] = fmaf(w[d], x, v[m]);
        }
      }
#pragma unroll
      for (int k = 0; k < kTaps; ++k) {
        const float wk = w[k < R ? R - k : k - R];
#pragma unroll
        for (int m = 0; m < 4; ++m)
          acc[k][m] = fmaf(wk, v[m], k + 1 < kTaps ? acc[k + 1][m] : 0.f);
      }
    } else {
#pragma unroll
      for (int k = 0; k + 1 < kTaps; ++k)
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[k][m] = acc[k + 1][m];
    }
    const int o = row - R;
    if (o >= m0 && in_c) {
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (p2_0 + run + m < n2)
          gstore(a.out + ((int64_t)o * n2 + p2_0 + run + m) * C + c, acc[0][m]);
    }
  }
}

// Workgroups of the fused kernel: the positions along n2 in equal tiles of at
// most 64, and segments of n1, as many as stay resident together (a few more and
// the rest is a second round: 378 x 156 x 222, R = 11, 151 us by a count that
// overlooked whole workgroups, 83 us like this; a workgroup of more than four
// wavefronts puts two on one SIMD). A row costs a workgroup 0.6 + 0.08 R us on an
// idle device and the halo's rows as much as the segment's own, so small maps
// want many short segments (80 x 50 x 127, R = 7: 61 us in segments of 27 rows,
// 21 us in segments of 4). Where several workgroups share a CU, four rows are the
// shortest that pay (312 x 65 x 84, R = 5: 17 us in segments of four rows, 27 us
// of two); up to one workgroup a CU, one row (31 x 50 x 127, R = 6: 18.6 us in
// segments of five rows, 14.8 us of one).
struct BeamSplit {
  int nw = 0, segs = 0, seg_rows = 0;
  int64_t cols = 0;
};
BeamSplit beam_split(const BeamArgs& a) {
  constexpr int64_t kCUs = 256;
  BeamSplit s;
  const int64_t tiles = (a.n2 + 63) / 64;
  s.nw = (int)(((a.n2 + tiles - 1) / tiles + kBeamPerWave - 1) / kBeamPerWave);
  s.cols = tiles * ((a.C + kBeamCh - 1) / kBeamCh);
  const int waves = beam_waves(a.R);
  const int64_t resident = kCUs * (s.nw > 4 ? waves / 2 : 4 * waves / s.nw) / s.cols;
  const int64_t want = std::max<int64_t>(a.n1 / 4, std::min<int64_t>(a.n1, kCUs / s.cols));
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>(resident, want));
  s.seg_rows = (int)((a.n1 + most - 1) / most);
  s.segs = (int)((a.n1 + s.seg_rows - 1) / s.seg_rows);
  return s;
}

template <int R>
int launch_beam_fused(const BeamArgs& a, const BeamSplit& s, hipStream_t st) {
  if constexpr (R > 1)
    if (a.R < R) return launch_beam_fused<R - 1>(a, s, st);
  const size_t lds = (size_t)2 * (s.nw * kBeamPerWave + 2 * R) * kBeamCh * sizeof(float);
  hipLaunchKernelGGL(beam_fused_kernel<R>, dim3((unsigned)(s.cols * s.segs)), dim3(64 * s.nw), lds,
                     st, a, s.segs);
  return (int)hipGetLastError();
}

// Mean over sky axis `axis` of [n1][n2][C]: out [n_other][C], FP64 sums. A
// workgroup takes 64 columns (of V channels); its wavefronts each sum a
// contiguous part of the axis, eight loads in flight, and the parts are added
// in LDS. One lane per column left 400 to 1600 wavefronts waiting on one load
// each (512 x 128 x 800 over n2: 74 us; like this 35 us).
constexpr int kLvMaxParts = 16;

template <int V>
__global__ __launch_bounds__(64 * kLvMaxParts) void lv_mean_kernel(const float* cube, float* outp,
                                                                   int64_t n1, int64_t n2,
                                                                   int64_t C, int axis) {
  using T = typename std::conditional<V == 4, float4, float>::type;
  __shared__ double part[kLvMaxParts][V][64];
  const int64_t nv = C / V;
  const int64_t n_other = axis == 0 ? n2 : n1;
  const int64_t n_axis = axis == 0 ? n1 : n2;
  const int64_t total = n_other * nv;
  const T* in = (const T*)cube;
  T* out = (T*)outp;
  const int lane = (int)(threadIdx.x & 63), p = (int)(threadIdx.x >> 6);
  const int parts = (int)(blockDim.x >> 6);
  const int64_t e = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 64 + lane;
  double acc[V] = {};
  if (e < total) {
    const int64_t o = e / nv, k = e % nv;
    // Element (p1, p2, k) sits at (p1 n2 + p2) nv + k.
    const int64_t base = (axis == 0 ? o : o * n2) * nv + k;
    const int64_t step = (axis == 0 ? n2 : 1) * nv;
    const int64_t lo = n_axis * p / parts, hi = n_axis * (p + 1) / parts;
    auto add = [&](const T& v) {
      if constexpr (V == 4) {
        acc[0] += v.x;
        acc[1] += v.y;
        acc[2] += v.z;
        acc[3] += v.w;
      } else {
        acc[0] += v;
      }
    };
    constexpr int kU = 8;
    int64_t i = lo;
    for (; i + kU <= hi; i += kU) {
      T v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) v[u] = gload(in + base + (i + u) * step);
#pragma unroll
      for (int u = 0; u < kU; ++u) add(v[u]);
    }
    for (; i < hi; ++i) add(gload(in + base + i * step));
  }
  if (parts > 1) {
#pragma unroll
    for (int m = 0; m < V; ++m) part[p][m][lane] = acc[m];
    __syncthreads();
    if (p) return;
    for (int q = 1; q < parts; ++q)
#pragma unroll
      for (int m = 0; m < V; ++m) acc[m] += part[q][m][lane];
  }
  if (e >= total) return;
  const double s = 1.0 / (double)n_axis;
  if constexpr (V == 4)
    gstore(out + e, make_float4((float)(acc[0] * s), (float)(acc[1] * s), (float)(acc[2] * s),
                                (float)(acc[3] * s)));
  else
    gstore(out + e, (float)(acc[0] * s));
}

template <int V>
int launch_lv_mean(const float* cube, float* out, int64_t n1, int64_t n2, int64_t C, int axis,
                   hipStream_t st) {
  const int64_t n_other = axis == 0 ? n2 : n1, n_axis = axis == 0 ? n1 : n2;
  const int64_t blocks = (n_other * (C / V) + 63) / 64;
  // Parts of the axis: enough wavefronts to fill the GPU (16 per CU), at least
  // eight loads each.
  int64_t parts = std::min<int64_t>((4096 + blocks - 1) / blocks, n_axis / 8);
  parts = std::max<int64_t>(1, std::min<int64_t>(parts, kLvMaxParts));
  // A grid axis holds less than 2^32 threads: rows of at most 2^20 workgroups.
  const int64_t bx = std::min<int64_t>(blocks, 1 << 20), by = (blocks + bx - 1) / bx;
  hipLaunchKernelGGL(lv_mean_kernel<V>, dim3((unsigned)bx, (unsigned)by),
                     dim3((unsigned)(64 * parts)), 0, st, cube, out, n1, n2, C, axis);
  return (int)hipGetLastError();
}

bool overlap(const void* a, const void* b, size_t bytes) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + bytes && y < x + bytes;
}

bool aligned4(const void* p, int64_t C) { return ((uintptr_t)p & 15) == 0 && (C & 3) == 0; }

iris_status check_cube(const float* cube, const float* out, int32_t n1, int32_t n2,
                       int32_t n_chan) {
  if (!cube || !out) return host::fail(IRIS_E_INVALID_ARG, "cube or output is NULL");
  if (n1 < 1 || n2 < 1 || n_chan < 1)
    return host::fail(IRIS_E_INVALID_ARG, "need n1, n2, n_chan >= 1 (got %d, %d, %d)", n1, n2,
                      n_chan);
  return IRIS_OK;
}

}  // namespace
}  // namespace iris

using namespace iris;

extern "C" {

size_t iris_beam_workspace_bytes(int32_t n1, int32_t n2, int32_t n_chan) {
  if (n1 < 1 || n2 < 1 || n_chan < 1) return 0;
  return (size_t)n1 * n2 * n_chan * sizeof(float);
}

iris_status iris_beam_convolve(const float* cube, float* out, int32_t n1, int32_t n2,
                               int32_t n_chan, double fwhm_pix, void* workspace,
                               size_t workspace_bytes, void* stream) {
  host::clear_error();
  iris_status s = check_cube(cube, out, n1, n2, n_chan);
  if (s != IRIS_OK) return s;
  if (!(fwhm_pix > 0.0) || !std::isfinite(fwhm_pix))
    return host::fail(IRIS_E_INVALID_ARG, "fwhm_pix must be > 0");
  const double sigma = fwhm_pix / (2.0 * std::sqrt(2.0 * std::log(2.0)));
  const double rr = std::ceil(4.0 * sigma);
  if (rr > kBeamMaxRadius)
    return host::fail(IRIS_E_UNSUPPORTED, "beam radius %.0f pixels above %d (fwhm_pix %g)", rr,
                      kBeamMaxRadius, fwhm_pix);
  const size_t need = iris_beam_workspace_bytes(n1, n2, n_chan);
  if (!workspace || workspace_bytes < need)
    return host::fail(IRIS_E_WORKSPACE, "beam workspace needs %zu bytes, got %zu", need,
                      workspace_bytes);
  BeamArgs a{};
  a.n1 = n1;
  a.n2 = n2;
  a.C = n_chan;
  a.R = (int32_t)rr;
  double wsum = 0.0, wd[kBeamMaxRadius + 1];
  for (int i = 0; i <= a.R; ++i) {
    wd[i] = std::exp(-(double)i * i / (2.0 * sigma * sigma));
    wsum += i ? 2.0 * wd[i] : wd[i];
  }
  for (int i = 0; i <= a.R; ++i) a.w[i] = (float)(wd[i] / wsum);
  const hipStream_t st = (hipStream_t)stream;
  const bool v4 = aligned4(cube, n_chan) && aligned4(out, n_chan) && aligned4(workspace, n_chan);
  // One kernel for both axes up to kBeamFusedRadius (its output rows in reach
  // fill the registers beyond); it reads neighbours of what it writes, so an
  // output that overlaps the cube takes the two passes. So do wide beams on
  // maps that leave it short segments, mostly halo: from R = 7 with rows that
  // the passes load four channels at a time (148 x 96 x 468: segments of 9 rows
  // at R = 9, 74 us against 58; 208 x 74 x 260: of 15 at R = 10, 54 against 47;
  // 148 x 96 x 468: of 19 at R = 11, 64 against 66), from R = 8 with others (396
  // x 89 x 62, 4 rows at R = 9: 60 against 52; 207 x 91 x 255, 7 rows at R = 8:
  // 57 against 82). And so do strips of up to four positions, which leave half of
  // the smallest tile idle, under beams wider than they are, once they fill the
  // device (1065 x 4 x 1280, R = 6: 37 against 31; 243 x 3 x 2661, R = 3: 16
  // against 21).
  const BeamSplit split = beam_split(a);
  const bool short_segs = v4 ? a.R >= 7 && 2 * split.seg_rows <= 3 * a.R
                             : a.R >= 8 && 4 * split.seg_rows < 3 * a.R;
  const bool strip = n2 <= kBeamPerWave / 2 && a.R > n2 && split.cols * split.segs > 256;
  // The fused kernel's row and position numbers fit 32 bits, and a launch takes
  // less than 2^32 threads: maps of more positions than that go in two passes.
  const bool fits = a.n1 <= 0x7FFFFFFF - kBeamFusedRadius &&
                    split.cols * split.segs * split.nw * 64 < (1ll << 32);
  if (a.R <= kBeamFusedRadius && fits && !short_segs && !strip && !overlap(cube, out, need)) {
    a.in = cube;
    a.out = out;
    return host::hip_status(launch_beam_fused<kBeamFusedRadius>(a, split, st), "beam kernel");
  }
  const int V = v4 ? 4 : 1;
  // Work items of a pass: the other axis x runs of kBeamRun positions x columns.
  auto blocks_for = [&](int64_t n_axis, int64_t n_other) {
    return ((n_axis + kBeamRun - 1) / kBeamRun * n_other * (n_chan / V) + 255) / 256;
  };
  const int64_t b2 = blocks_for(n2, n1), b1 = blocks_for(n1, n2);
  if (std::max(b1, b2) > 0x7FFFFFFF)
    return host::fail(IRIS_E_UNSUPPORTED, "cube too large for one launch");
  // Along n2 into the workspace, then along n1 into the output.
  a.in = cube;
  a.out = (float*)workspace;
  a.axis = 1;
  if (v4) hipLaunchKernelGGL(beam_pass_kernel<4>, dim3((int)b2), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(beam_pass_kernel<1>, dim3((int)b2), dim3(256), 0, st, a);
  a.in = (const float*)workspace;
  a.out = out;
  a.axis = 0;
  if (v4) hipLaunchKernelGGL(beam_pass_kernel<4>, dim3((int)b1), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(beam_pass_kernel<1>, dim3((int)b1), dim3(256), 0, st, a);
  return host::hip_status((int)hipGetLastError(), "beam kernel");
}

iris_status iris_lv_mean(const float* cube, float* out, int32_t n1, int32_t n2, int32_t n_chan,
                         int32_t axis, void* stream) {
  host::clear_error();
  iris_status s = check_cube(cube, out, n1, n2, n_chan);
  if (s != IRIS_OK) return s;
  if (axis != 0 && axis != 1) return host::fail(IRIS_E_INVALID_ARG, "axis must be 0 or 1");
  const bool v4 = aligned4(cube, n_chan) && aligned4(out, n_chan);
  const hipStream_t st = (hipStream_t)stream;
  return host::hip_status(v4 ? launch_lv_mean<4>(cube, out, n1, n2, n_chan, axis, st)
                             : launch_lv_mean<1>(cube, out, n1, n2, n_chan, axis, st),
                          "l,v mean kernel");
}

}  // extern "C"
