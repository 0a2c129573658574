// Mask instantiation from a threshold map (paper Sec. 4.1.2): the mask for a
// density threshold p is M_p = 1[T <= p], one comparison per block, stored in
// the CRM layout (LSB-first uint64 words per query-block row).
//
// One wavefront per row (h, u) and set of up to 16 thresholds, eight words at
// a time.  Lane l loads T[h][u][64 w + l] for the eight words of the group
// into registers (all loads in flight together); then for every threshold
// p[i][h] a wavefront ballot of the comparison is the word itself (ballot bit
// l is lane l's predicate, i.e. key block 64 w + l at bit l), lane k keeps
// word k, and the group's words leave in one 64-byte store.  The thresholds of
// a wavefront come in with one vector load, so no scalar load waits inside the
// threshold loop.  The map is read from memory once per 16 thresholds (a
// head's map serves every timestep of its layer; the re-reads hit in L2): 4
// bytes read per block, one bit written per block and threshold, three vector
// instructions per 64 bits (the compare and two lane writes).

#include <algorithm>

#include "device_common.h"
#include "launch.h"

namespace sa {

namespace {

constexpr int kInstWaves = 4;

constexpr int kGroup = 8;     // words whose map entries a lane holds in registers at once
constexpr int kInstThr = 16;  // thresholds per wavefront (grid.y splits larger sets)

// lo and hi hold the two halves of a wavefront-uniform 64-bit word in lane K,
// other lanes unchanged (v_writelane_b32).  The word is a ballot just written
// by a vector compare, and a vector read of a vector-written scalar needs two
// wait states first; one statement keeps the two writes behind the wait.
template <int K>
__device__ __forceinline__ void write_lane_k(uint32_t& lo, uint32_t& hi, uint64_t word) {
  asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
      : "+v"(lo), "+v"(hi)
      : "s"((uint32_t)word), "s"((uint32_t)(word >> 32)), "n"(K));
}
// The same for a k < kGroup that is a constant once the caller's loop is
// unrolled.
static_assert(kGroup <= 8, "write_lane covers lanes 0..7");
__device__ __forceinline__ void write_lane(uint32_t& lo, uint32_t& hi, uint64_t word, int k) {
  switch (k) {
    case 0: write_lane_k<0>(lo, hi, word); break;
    case 1: write_lane_k<1>(lo, hi, word); break;
    case 2: write_lane_k<2>(lo, hi, word); break;
    case 3: write_lane_k<3>(lo, hi, word); break;
    case 4: write_lane_k<4>(lo, hi, word); break;
    case 5: write_lane_k<5>(lo, hi, word); break;
    case 6: write_lane_k<6>(lo, hi, word); break;
    default: write_lane_k<7>(lo, hi, word); break;
  }
}

__global__ __launch_bounds__(64 * kInstWaves) void mask_inst_kernel(
    const float* __restrict__ T, const float* __restrict__ p, int n_p, int H, int n_qb, int n_kb,
    int W, uint64_t* __restrict__ bits) {
  const int lane = threadIdx.x & 63;
  const int64_t rows = (int64_t)H * n_qb;
  const int64_t row = (int64_t)blockIdx.x * kInstWaves + (threadIdx.x >> 6);
  if (row >= rows) return;  // uniform per wavefront
  const int h = (int)(row / n_qb);
  const int i_first = blockIdx.y * kInstThr;
  const int n_thr = min(kInstThr, n_p - i_first);
  // this wavefront's thresholds, lane k holding p[i_first + k][h], read once
  // with one vector load and handed to the comparisons by readlane
  const float p_lane = lane < n_thr ? p[(int64_t)(i_first + lane) * H + h] : 0.f;
  const float* trow = T + row * n_kb;
  for (int w0 = 0; w0 < W; w0 += kGroup) {
    const int nw = min(kGroup, W - w0);
    // all loads of the group first (independent, in flight together)
    float t[kGroup];
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      const int v = (w0 + k) * 64 + lane;
      t[k] = (k < nw && v < n_kb) ? trow[v] : __builtin_nanf("");  // NaN: never on
    }
    for (int i = 0; i < n_thr; ++i) {  // uniform trip count
      const float pi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, p_lane), i));
      uint32_t lo = 0, hi = 0;  // lane k ends up holding word w0 + k
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {
        if (k < nw) {  // uniform
          const uint64_t word = __ballot(t[k] <= pi);
          write_lane(lo, hi, word, k);
        }
      }
      if (lane < nw)
        bits[((int64_t)(i_first + i) * rows + row) * W + w0 + lane] =
            ((uint64_t)hi << 32) | lo;
    }
  }
}

// Many thresholds.  The comparisons bound the call: one vector compare per 64
// blocks and threshold at least, and in the kernel above two lane writes and
// their wait beside it, since a ballot is a scalar and stores take lanes.  Here
// a lane owns 32 consecutive blocks of a row (their map entries stay in
// registers for every threshold) and builds its half word by itself, a compare
// and an add-with-carry per block: acc = 2 acc + (t <= p).  That is two
// instructions per 64 blocks and threshold instead of five issue slots, at the
// price of a way through LDS for the map entries, so it takes sets of at least
// kInstManyMin thresholds, from where it is slower at no size measured: here
// and above, kernel in us, 4 thresholds 14.2 and 15.5 (40 x 591^2), 40 and 47
// (40 x 1200^2), but 3.6 and 3.4 (12 x 300^2); 6 16.9 and 18.6, 3.8 and 3.8; 8
// 18.9 and 22.1, 4.1 and 4.3.  Half words of consecutive lanes are consecutive in
// memory, whatever rows and heads they belong to; a lane reads its own head's
// threshold.  40 x 591^2 maps, 50 thresholds: 98.4 -> 63 us, of which the
// comparisons alone are 46 us; without the early requests 67 us (all
// wavefronts load, then all compare).
constexpr int kInstManyMin = 6;
constexpr int kInstManyWaves = 4;
constexpr int kInstManyResident = 4;  // wavefronts a SIMD

// For k = 15 .. 0: acc = 2 acc + (t[k] <= p).  A vector read of a vector-written
// scalar needs two wait states, so the compares rotate over three pairs of
// scalars and every carry is added two compares after its own; one statement,
// since that order is what keeps the distance.
__device__ __forceinline__ void push16(uint32_t& acc, const float* t, float p) {
  uint64_t c0, c1;
#define SA_CMP(c, n) "v_cmp_le_f32 " c ", %" #n ", %3\n\t"
#define SA_ADD(c) "v_addc_co_u32 %0, " c ", %0, %0, " c "\n\t"
#define SA_STEP(c, n) SA_ADD(c) SA_CMP(c, n)
  asm(SA_CMP("vcc", 19) SA_CMP("%1", 18) SA_CMP("%2", 17)
          SA_STEP("vcc", 16) SA_STEP("%1", 15) SA_STEP("%2", 14)
          SA_STEP("vcc", 13) SA_STEP("%1", 12) SA_STEP("%2", 11)
          SA_STEP("vcc", 10) SA_STEP("%1", 9) SA_STEP("%2", 8)
          SA_STEP("vcc", 7) SA_STEP("%1", 6) SA_STEP("%2", 5)
          SA_STEP("vcc", 4) SA_ADD("%1") SA_ADD("%2") SA_ADD("vcc")
      : "+&v"(acc), "=&s"(c0), "=&s"(c1)
      : "v"(p), "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]),
        "v"(t[7]), "v"(t[8]), "v"(t[9]), "v"(t[10]), "v"(t[11]), "v"(t[12]), "v"(t[13]),
        "v"(t[14]), "v"(t[15])
      : "vcc");
#undef SA_STEP
#undef SA_ADD
#undef SA_CMP
}

// Where lane l's half word f is in the map.
struct HalfWord {
  int64_t at;  // first entry of its 32
  int head;
  int down;  // places it is shifted down by
};

__device__ __forceinline__ HalfWord half_word(int64_t f, int n_qb, int n_kb, int W) {
  const int row = (int)(f / (2 * W));
  const int v0 = (int)(f - (int64_t)row * (2 * W)) * 32;  // first block of the half word
  // the 32 entries end with the row at the latest (n_kb >= 32); the half word
  // of a lane moved back so is shifted down again, which drops the entries of
  // earlier half words and leaves zeros past the row's end
  const int from = min(v0, n_kb - 32);
  return HalfWord{(int64_t)row * n_kb + from, row / n_qb, v0 - from};
}

// A wavefront takes groups of 64 half words g, g + n_waves, ... (with n_parts
// parts of the thresholds each) and requests the next one's entries before it
// compares, so that only the first group's loads are waited for.
__global__ __launch_bounds__(64 * kInstManyWaves) void mask_inst_many_kernel(
    const float* __restrict__ T, const float* __restrict__ p, int n_p, int per_part, int n_parts,
    int H, int n_qb, int n_kb, int W, uint32_t* __restrict__ bits) {
  // a wavefront's entries on their way from memory order to lane order, half
  // of each lane's at a time, in rows of 20 floats (16 lanes' 16-byte reads
  // lie in different banks); then the lanes' thresholds
  __shared__ __attribute__((aligned(16))) float stage_all[kInstManyWaves][64][20];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float(*stage)[20] = stage_all[wave];
  const int64_t n_half = (int64_t)H * n_qb * (2 * W);
  const int64_t n_units = (n_half + 63) / 64 * n_parts;
  const int64_t n_waves = (int64_t)gridDim.x * kInstManyWaves;
  int64_t unit = (int64_t)blockIdx.x * kInstManyWaves + wave;
  if (unit >= n_units) return;  // uniform; no workgroup barrier below

  // four lanes read 64 bytes of one half word's entries, 16 half words a load
  f32x4 x[2][4];
  HalfWord hw;
  int64_t f;
  auto request = [&](int64_t un) {
    f = min(un / n_parts * 64 + lane, n_half - 1);  // lanes past the end repeat the last
    hw = half_word(f, n_qb, n_kb, W);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t src = __shfl(hw.at, 16 * j + (lane >> 2), 64) + 4 * (lane & 3);
      __builtin_memcpy(&x[0][j], T + src, 16);  // 4-byte aligned
      __builtin_memcpy(&x[1][j], T + src + 16, 16);
    }
  };
  request(unit);
  while (true) {
    const int i0 = (int)(unit % n_parts) * per_part;
    const int i1 = min(n_p, i0 + per_part);
    const float* ph = p + hw.head;
    const int down = hw.down;
    uint32_t* o = bits + (int64_t)i0 * n_half + f;
    float t[32];
#pragma unroll
    for (int k0 = 0; k0 < 2; ++k0) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *(SA_LDS f32x4*)&stage[16 * j + (lane >> 2)][4 * (lane & 3)] = x[k0][j];
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
      for (int k = 0; k < 16; k += 4) {
        const f32x4 y = *(const SA_LDS f32x4*)&stage[lane][k];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[16 * k0 + k + e] = y[e];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    }
    // The lanes' thresholds take the stage's place, kStaged settings at a
    // time: read from memory inside the loop, each would wait for the store
    // before it (one counter for both), and LDS reads do not.
    constexpr int kStaged = 20;
    float* lane_p = &stage[0][0] + lane;
    const int64_t next = unit + n_waves;
    for (int c0 = i0; c0 < i1; c0 += kStaged) {
      const int n = min(kStaged, i1 - c0);
      __builtin_amdgcn_wave_barrier();
#pragma unroll 4
      for (int i = 0; i < n; ++i) lane_p[64 * i] = ph[(int64_t)(c0 + i) * H];
      if (c0 + kStaged >= i1 && next < n_units) request(next);
      float pn = lane_p[0];
      for (int i = 0; i < n; ++i) {
        const float pi = pn;
        pn = lane_p[64 * min(i + 1, n - 1)];
        uint32_t acc = 0;
        push16(acc, t + 16, pi);
        push16(acc, t, pi);
        *o = down < 32 ? acc >> (down & 31) : 0u;  // lanes past the end: the last one's, again
        o += n_half;
      }
    }
    if (next >= n_units) break;
    unit = next;
  }
}

}  // namespace

hipError_t launch_mask_instantiate(const float* T, const float* p, int n_p, int H, int n_qb,
                                   int n_kb, uint64_t* bits, hipStream_t stream) {
  const int64_t rows = (int64_t)H * n_qb;
  const int W = (n_kb + 63) / 64;
  if (n_p >= kInstManyMin && n_kb >= 32) {
    const int64_t groups = (rows * (2 * W) + 63) / 64;
    const int64_t places = 4 * 256 * kInstManyResident;
    // a group's thresholds are cut in parts until there are several units for
    // every place on the chip, but not below kInstManyMin, since each part
    // loads the entries again; until every SIMD has a unit, down to two (6 and 8
    // thresholds, kernel in us: 12 x 100^2 maps 3.7 and 4.0 -> 3.0 and 3.0, where
    // the kernel above takes 3.1 and 3.4; 1 x 591^2 3.7 and 4.0 -> 3.0 and 3.1)
    const int64_t cuts = std::max(std::min<int64_t>(std::max<int64_t>(1, 4 * places / groups),
                                                    n_p / kInstManyMin),
                                  std::min<int64_t>(4 * 256 / groups, n_p / 2));
    const int per_part = (int)((n_p + cuts - 1) / cuts);
    const int n_parts = (n_p + per_part - 1) / per_part;
    const int64_t waves = std::min<int64_t>(groups * n_parts, places);
    hipLaunchKernelGGL(mask_inst_many_kernel,
                       dim3((unsigned)((waves + kInstManyWaves - 1) / kInstManyWaves)),
                       dim3(64 * kInstManyWaves), 0, stream, T, p, n_p, per_part, n_parts, H, n_qb,
                       n_kb, W, (uint32_t*)bits);
    return hipGetLastError();
  }
  const int64_t grid = (rows + kInstWaves - 1) / kInstWaves;
  const int chunks = (n_p + kInstThr - 1) / kInstThr;
  if (chunks > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mask_inst_kernel, dim3((unsigned)grid, (unsigned)chunks), dim3(64 * kInstWaves),
                     0, stream, T, p, n_p, H, n_qb, n_kb, W, bits);
  return hipGetLastError();
}

}  // namespace sa
