// Conservative resize of threshold maps and block masks between resolutions
// (paper Sec. 4.3.1, Eq. 7).  Target block (u, v) samples the base map at
// x = u n_q / n_q', y = v n_k / n_k' (exact rationals: integer quotient and
// remainder); the bilinear neighbours with positive weight are base rows
// floor(x) and, if the remainder is non-zero, floor(x) + 1 (clamped to the
// last row), and likewise for columns.
//  * mask: the ceiling of the bilinear interpolation of a 0/1 mask is 1 iff a
//    positively weighted neighbour is 1, i.e. the OR of those <= 4 bits;
//  * threshold map: the minimum over the same neighbours, which makes
//    instantiation and resizing commute (1[T' <= p] is the resized 1[T <= p]).
// Both are streams over the target with cached reads of the base.  Upscaling,
// which the operation is meant for, has kernels of its own: neighbouring
// targets share their sources, so a base value is read once per strip of
// target rows (map) and a base bit is spread over all its targets of a word
// at once (mask).  A target smaller than the base takes the general kernels,
// which sample every target by itself.

#include <algorithm>

#include "device_common.h"
#include "launch.h"

namespace sa {

namespace {

struct AxisPt {
  int i0, i1;
  bool two;  // the second neighbour has a positive weight
};

// floor(t n_base / n_target) and whether the remainder is non-zero, without a
// division: all sizes are < 2^16, so t n_base < 2^32 (24-bit multiplies, which
// run at full rate) and the single-precision estimate num * (1 / n_target) is
// within 3 * 2^-24 * 2^16 < 0.02 of the true quotient; one remainder step,
// with the remainder modulo 2^32 as a signed number, fixes it.
__device__ __forceinline__ AxisPt axis_point(int t, int n_base, int n_target, float inv_target) {
  const uint32_t num = __umul24((uint32_t)t, (uint32_t)n_base);
  int q = (int)((float)num * inv_target);
  int rem = (int)(num - __umul24((uint32_t)q, (uint32_t)n_target));
  if (rem < 0) {
    --q;
    rem += n_target;
  } else if (rem >= n_target) {
    ++q;
    rem -= n_target;
  }
  return AxisPt{q, min(q + 1, n_base - 1), rem > 0};
}

constexpr int kMapRowsPerThread = 8;

// grid: (target columns / 256, target rows / 8, heads); each thread writes one
// column of eight consecutive target rows (few, well-filled workgroups).  The
// row sample points are uniform over the workgroup; all loads of the eight
// rows go out before the first minimum is formed, so their latencies overlap.
__global__ __launch_bounds__(256) void resize_map_kernel(const float* __restrict__ T, int nq,
                                                         int nk, float* __restrict__ out, int tq,
                                                         int tk) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= tk) return;
  const int h = blockIdx.z;
  const AxisPt b = axis_point(v, nk, tk, 1.0f / (float)tk);
  const float inv_tq = 1.0f / (float)tq;
  const float* Th = T + (int64_t)h * nq * nk;
  const int u0 = blockIdx.y * kMapRowsPerThread;
  float x[kMapRowsPerThread][4];
#pragma unroll
  for (int r = 0; r < kMapRowsPerThread; ++r) {
    const int u = min(u0 + r, tq - 1);  // rows past the end repeat the last (not stored)
    const AxisPt a = axis_point(u, nq, tq, inv_tq);
    const float* r0 = Th + (int64_t)a.i0 * nk;
    const float* r1 = Th + (int64_t)a.i1 * nk;
    x[r][0] = r0[b.i0];
    x[r][1] = r0[b.i1];
    x[r][2] = r1[b.i0];
    x[r][3] = r1[b.i1];
    x[r][3] = a.two ? x[r][3] : x[r][0];
    x[r][2] = a.two ? x[r][2] : x[r][0];
  }
#pragma unroll
  for (int r = 0; r < kMapRowsPerThread; ++r) {
    // fminf skips NaN; neighbours with zero weight are replaced by the first
    float m = fminf(x[r][0], b.two ? x[r][1] : x[r][0]);
    m = fminf(m, fminf(x[r][2], b.two ? x[r][3] : x[r][2]));
    if (u0 + r < tq) out[((int64_t)h * tq + u0 + r) * tk + v] = m;
  }
}

// Upscaling map kernel (tq >= nq).  Writing the target should bound the call
// (40 x 591 x 591 floats, 10 us, against 40 x 256 x 256 read); the general
// kernel above is bound by vector instructions instead, four loads, their
// minima and 64-bit sample points for every few floats stored.  Here a
// workgroup takes a strip of target rows and goes down the base rows under it:
// kStripRows rows lie on at most kStripRows + 1 base rows, since x = u nq / tq
// moves by at most one per row.  A lane reads its two column neighbours of
// every such base row once, all reads before the first use, and keeps their
// minimum in a register vector; a target row is then one minimum of two of its
// entries (uniform index) and a store.  The workgroup owns whole rows, one run
// of memory.  40 x 256^2 -> 591^2: 24.9 -> 15.0 us.  Tried first: 64-column
// pieces of the strips in workgroups of their own (30.8 us: most 128-byte lines
// are put together from two XCDs), and selecting the row entries with branches
// or conditional moves (24.5-26.5 us, vector instructions again).
// fminf of two values that hold no signalling NaN: the bare instruction
__device__ __forceinline__ float min_canonical(float x, float y) {
  float m;
  asm("v_min_f32 %0, %1, %2" : "=v"(m) : "v"(x), "v"(y));
  return m;
}

constexpr int kStripRows = 15;  // so that its base rows' values fit one 16-register vector
constexpr int kStripRowsFew = 7;
constexpr int kMapUpWaves = 8;
constexpr int kMapUpWavesFew = 16;

__global__ __launch_bounds__(64 * kMapUpWavesFew) void resize_map_up_kernel(
    const float* __restrict__ T, int nq, int nk, float* __restrict__ out, int tq, int tk,
    int strip) {
  const int h = blockIdx.y;
  const int u0 = blockIdx.x * strip;
  const int rows = min(strip, tq - u0);
  // the strip's row sample points: lane r holds target row u0 + r's
  const AxisPt a = axis_point(min(u0 + (int)(threadIdx.x & 63), tq - 1), nq, tq, 1.0f / (float)tq);
  const int first = a.i0, second = a.two ? a.i1 : a.i0;
  const int s0 = __builtin_amdgcn_readfirstlane(first);
  const int ns = __builtin_amdgcn_readlane(second, rows - 1) - s0 + 1;  // base rows under the strip
  const float* Th = T + ((int64_t)h * nq + s0) * nk;
  const float inv_tk = 1.0f / (float)tk;
  for (int v = threadIdx.x; v < tk; v += blockDim.x) {
    const AxisPt b = axis_point(v, nk, tk, inv_tk);
    float x0[16], x1[16];
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // base rows past the strip's last repeat it
      const float* row = Th + min(k, ns - 1) * nk;
      x0[k] = row[b.i0];
      x1[k] = row[b.i1];
    }
    if (ns > 8) {  // uniform; never with a scale of 7 / 15 or less between the sizes
#pragma unroll
      for (int k = 8; k < 16; ++k) {
        const float* row = Th + min(k, ns - 1) * nk;
        x0[k] = row[b.i0];
        x1[k] = row[b.i1];
      }
    } else {
#pragma unroll
      for (int k = 8; k < 16; ++k) x0[k] = x1[k] = 0.f;
    }
    f32x16 m;
    // a minimum skips NaN; a column neighbour with zero weight is left out
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float c0 = __builtin_canonicalizef(x0[k]);
      m[k] = b.two ? min_canonical(c0, __builtin_canonicalizef(x1[k])) : c0;
    }
    float* o = out + ((int64_t)h * tq + u0) * tk + v;
    for (int r = 0; r < rows; ++r) {  // uniform row indexes: register-indexed moves
      const float m0 = m[__builtin_amdgcn_readlane(first, r) - s0];
      const float m1 = m[__builtin_amdgcn_readlane(second, r) - s0];
      *o = min_canonical(m0, m1);
      o += tk;
    }
  }
}

constexpr int kResizeWaves = 4;
constexpr int kResizeRowsPerWave = 4;
// Target widths up to this many blocks keep their column sample points in a
// per-workgroup LDS table (32 KB); wider targets compute them per word.
constexpr int kResizeTableMax = 8192;

// A wavefront per target row, kResizeRowsPerWave rows per wavefront.  The
// target row's two base rows are ORed into one (the ceiling is the OR of the
// positively weighted neighbours, and the row and column choices combine
// independently), staged in LDS; the column sample points of the target
// width are shared by every row of the workgroup (TABLE: entry
// i0 | two << 31 per column).  Lane l of output word w takes target column
// 64 w + l; a ballot forms the word, and lane w keeps word w of a group of 64.
template <bool TABLE>
__global__ __launch_bounds__(64 * kResizeWaves) void resize_mask_kernel(
    const uint64_t* __restrict__ bits, int H, int nq, int nk, int W, uint64_t* __restrict__ out,
    int tq, int tk, int Wt) {
  extern __shared__ uint64_t lds_words[];  // [waves][W] ORed base rows, then the column table
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  uint32_t* table = (uint32_t*)(lds_words + kResizeWaves * W);
  const float inv_tk = 1.0f / (float)tk;
  if (TABLE) {
    for (int v = threadIdx.x; v < tk; v += 64 * kResizeWaves) {
      const AxisPt b = axis_point(v, nk, tk, inv_tk);
      table[v] = (uint32_t)b.i0 | (b.two ? 0x80000000u : 0u);
    }
    __syncthreads();
  }
  uint64_t* rr = lds_words + wave * W;
  const int64_t rows = (int64_t)H * tq;
  const int64_t row_first = ((int64_t)blockIdx.x * kResizeWaves + wave) * kResizeRowsPerWave;
  for (int k = 0; k < kResizeRowsPerWave; ++k) {
    const int64_t row = row_first + k;
    if (row >= rows) break;  // uniform per wavefront; no workgroup barrier below
    const int h = (int)(row / tq);
    const int u = (int)(row - (int64_t)h * tq);
    const AxisPt a = axis_point(u, nq, tq, 1.0f / (float)tq);
    const uint64_t* g0 = bits + ((int64_t)h * nq + a.i0) * W;
    const uint64_t* g1 = bits + ((int64_t)h * nq + a.i1) * W;
    __builtin_amdgcn_wave_barrier();  // the previous row's reads of rr are done
    for (int w = lane; w < W; w += 64) rr[w] = g0[w] | (a.two ? g1[w] : 0ull);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    uint64_t* orow = out + row * Wt;
    for (int w0 = 0; w0 < Wt; w0 += 64) {
      const int nw = min(64, Wt - w0);
      uint64_t mine = 0;
      for (int w = 0; w < nw; ++w) {
        const int v = (w0 + w) * 64 + lane;
        uint32_t on = 0;
        if (v < tk) {
          int i0;
          bool two;
          if (TABLE) {
            const uint32_t e = table[v];
            i0 = (int)(e & 0x7fffffffu);
            two = (e >> 31) != 0;
          } else {
            const AxisPt b = axis_point(v, nk, tk, inv_tk);
            i0 = b.i0;
            two = b.two;
          }
          const int i1 = min(i0 + 1, nk - 1);
          on = (uint32_t)(rr[i0 >> 6] >> (i0 & 63)) & 1u;
          if (two) on |= (uint32_t)(rr[i1 >> 6] >> (i1 & 63)) & 1u;
        }
        const uint64_t word = __ballot(on != 0);
        if (lane == w) mine = word;
      }
      if (lane < nw) orow[w0 + lane] = mine;
    }
  }
}

// Upscaling mask kernel (tk >= nk).  A base bit s is a positively weighted
// neighbour of the targets v with s - 1 < v nk / tk < s + 1, one run of
// columns, so a target word is the OR over the base bits under it of (bit ?
// its run in this word : 0).  The runs are the same for every row: lane l of a
// wavefront first stands for column 64 w + l, and two ballots give the run of
// each base bit as a scalar; then it stands for a target row, and one bit
// extract and two and-or instructions per base bit form 64 rows' words at
// once.  A word lies over at most 64 / (tk / nk) + 2 base bits, so a word costs
// (5 / 64) of that in vector instructions, against about 15 when every column
// of every row looks its two bits up; what is left is the latency of a few
// rounds of loads.  40 x 256^2 -> 591^2: 20.8 -> 6.3 us.
constexpr int kMaskUpWaves = 4;

__global__ __launch_bounds__(64 * kMaskUpWaves) void resize_mask_up_kernel(
    const uint32_t* __restrict__ bits, int rows, int nq, int nk, int W, uint64_t* __restrict__ out,
    int tq, int tk, int Wt) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = blockIdx.x * 64 + lane;
  const int r = min(row, rows - 1);
  const int h = r / tq;
  const AxisPt a = axis_point(r - h * tq, nq, tq, 1.0f / (float)tq);
  const uint32_t* g0 = bits + ((int64_t)h * nq + a.i0) * (2 * W);
  const uint32_t* g1 = a.two ? bits + ((int64_t)h * nq + a.i1) * (2 * W) : g0;
  const float inv_tk = 1.0f / (float)tk;
  for (int w = blockIdx.y * kMaskUpWaves + wave; w < Wt; w += kMaskUpWaves * gridDim.y) {
    const int v = 64 * w + lane;
    const AxisPt b = axis_point(min(v, tk - 1), nk, tk, inv_tk);
    const int e0 = v < tk ? b.i0 : -1;  // the column's neighbours; none past the end
    const int e1 = v < tk && b.two ? b.i1 : e0;
    // the base bits under the word: its first and last columns' neighbours
    const int s_lo = __builtin_amdgcn_readfirstlane(b.i0);
    const int s_hi = __builtin_amdgcn_readlane(b.two ? b.i1 : b.i0, 63);
    uint64_t word = 0;
    for (int d = s_lo >> 5; d <= s_hi >> 5; ++d) {  // at most three 32-bit words of the base row
      const uint32_t src = g0[d] | g1[d];
      uint32_t lo = 0, hi = 0;
      const int s_end = min(s_hi, 32 * d + 31);
      for (int s = max(s_lo, 32 * d); s <= s_end; ++s) {
        const uint64_t run = __ballot(e0 == s) | __ballot(e1 == s);
        const uint32_t on = (uint32_t)__builtin_amdgcn_sbfe((int)src, s & 31, 1);
        lo |= on & (uint32_t)run;
        hi |= on & (uint32_t)(run >> 32);
      }
      word |= ((uint64_t)hi << 32) | lo;
    }
    if (row < rows) out[(int64_t)row * Wt + w] = word;
  }
}

}  // namespace

hipError_t launch_resize_map(const float* T, int H, int nq, int nk, float* out, int tq, int tk,
                             hipStream_t stream) {
  if (tq >= nq) {  // a strip of target rows lies on few base rows
    // Where the strips would leave half of the compute units without one, the
    // time is that of a workgroup, and shorter strips and more wavefronts
    // shorten it.  Kernel in us, general / strips of 15 / of 7: 1 x 591^2 -> 600^2
    // 3.9 / 5.4 / 3.6, 1 x 20^2 -> 1200^2 5.5 / 7.1 / 5.3, 40 x (16, 600) -> (16, 640)
    // 3.9 / 5.4 / 3.7; of 4 3.5, 6.2 and 3.5.  At 192 strips (12 x 60^2 -> 240^2)
    // 15 and 7 rows take 3.5 both, at 400 (5 x 400^2 -> 450^2) 4.2 and 4.4.
    const bool few = (int64_t)H * ((tq + kStripRows - 1) / kStripRows) < 128;
    const int strip = few ? kStripRowsFew : kStripRows;
    // as few rounds of wavefronts over the columns as possible, and no more
    // wavefronts than these rounds need
    const int most = few ? kMapUpWavesFew : kMapUpWaves;
    const int pieces = (tk + 63) / 64;
    const int rounds = (pieces + most - 1) / most;
    hipLaunchKernelGGL(resize_map_up_kernel, dim3((tq + strip - 1) / strip, H),
                       dim3(64 * ((pieces + rounds - 1) / rounds)), 0, stream, T, nq, nk, out, tq,
                       tk, strip);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(resize_map_kernel,
                     dim3((tk + 255) / 256, (tq + kMapRowsPerThread - 1) / kMapRowsPerThread, H),
                     dim3(256), 0, stream, T, nq, nk, out, tq, tk);
  return hipGetLastError();
}

hipError_t launch_resize_mask(const uint64_t* bits, int H, int nq, int nk, uint64_t* out, int tq,
                              int tk, hipStream_t stream) {
  const int64_t rows = (int64_t)H * tq;
  const int W = (nk + 63) / 64, Wt = (tk + 63) / 64;
  const int64_t per_wg = (int64_t)kResizeWaves * kResizeRowsPerWave;
  const dim3 grid((unsigned)((rows + per_wg - 1) / per_wg));
  if (tk >= nk) {
    // 64 rows by kMaskUpWaves words a workgroup; fewer, longer workgroups once
    // there are enough to fill the chip several times over
    const int64_t gx = (rows + 63) / 64;
    const int64_t gy = std::min<int64_t>((Wt + kMaskUpWaves - 1) / kMaskUpWaves,
                                         std::max<int64_t>(1, 8192 / gx));
    hipLaunchKernelGGL(resize_mask_up_kernel, dim3((unsigned)gx, (unsigned)gy),
                       dim3(64 * kMaskUpWaves), 0, stream, (const uint32_t*)bits, (int)rows, nq, nk,
                       W, out, tq, tk, Wt);
    return hipGetLastError();
  }
  const size_t rows_bytes = (size_t)kResizeWaves * W * 8;
  if (tk <= kResizeTableMax)
    hipLaunchKernelGGL(resize_mask_kernel<true>, grid, dim3(64 * kResizeWaves),
                       rows_bytes + (size_t)tk * 4, stream, bits, H, nq, nk, W, out, tq, tk, Wt);
  else
    hipLaunchKernelGGL(resize_mask_kernel<false>, grid, dim3(64 * kResizeWaves), rows_bytes,
                       stream, bits, H, nq, nk, W, out, tq, tk, Wt);
  return hipGetLastError();
}

}  // namespace sa
