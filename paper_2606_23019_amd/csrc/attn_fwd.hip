// Block-sparse attention forward for gfx950 (CDNA4).
//
// What it computes (paper Sec. 4.3.2): FlashAttention's forward pass with the
// dense key-block loop replaced by a walk over the key blocks enabled in the
// query block's Compressed Row Mask row.  Each executed block is a dense
// 128 x 128 (or 64 x 64) tile, so both contractions run on the matrix cores.
//
// Work item = (b, h, query block u), BQ / 32 wavefronts per item, each owning
// 32 query rows.  Items of 128 query rows, and the maskless path wherever
// the tiles fit in LDS, run 2 (or 4) items per 8-wavefront workgroup in
// ping-pong (bsattn_fwd_pp_kernel, described there); masked items of 64 rows
// run one item per workgroup (bsattn_fwd_kernel).  Per enabled key block kb:
//
//   1. the workgroup copies K[kb] and V[kb] (BK x D bf16, row-major) from
//      global memory into LDS (16-byte chunks, XOR-swizzled per row);
//   2. every wavefront computes S^T = K Q^T with v_mfma_f32_32x32x16_bf16:
//      Q^T (its 32 queries) stays in registers as the B operand (read once
//      per item, in the ping-pong kernel through LDS where the tiles are
//      square), K rows come from LDS as the A operand.  In the transposed product each lane owns
//      one query column, so the row statistics of the softmax are lane-local
//      apart from one exchange between the two half-wavefronts;
//   3. online softmax in fp32 in the log2 domain: running max m and sum l,
//      p = exp2(s * scale * log2(e) - m), the accumulator rescaled by
//      exp2(m_old - m_new);
//   4. O^T += V^T P^T, again 32x32x16 MFMA: P (rounded to bf16) is already
//      in the B-operand layout -- the K rows were fed to the first product
//      in an order that makes this so -- and V^T comes from LDS through the
//      gfx950 transposing read ds_read_b64_tr_b16.
//
// Epilogue: out = O / l rounded to bf16 (or kept in fp32 for the fp32-output
// entry points), lse = (m + log2 l) ln 2; the rows go out through the free
// K/V tiles in LDS so that stores write whole rows (store_rows_staged).
// The same kernels with DENSE = true are the maskless path (every key block).
// Keys past N (ragged last block) are loaded as zeros and get -inf logits.

#include <math.h>

#include "device_common.h"
#include "launch.h"

namespace sa {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

template <int BQ, int BK, int D>
struct Tile {
  static constexpr int kWaves = BQ / 32;
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kChunksPerRow = D / 8;  // 16-byte chunks
  // a tile is copied by wave-wide 1 KB direct-to-LDS loads (64 lanes x 16 B)
  static constexpr int kLoadsPerWave = BK * kChunksPerRow / 64 / kWaves;
  static_assert(BQ % 32 == 0 && BK % 32 == 0 && D % 32 == 0, "tile shape");
  static_assert((BK * kChunksPerRow) % (64 * kWaves) == 0, "copy split");
};

// XOR applied to the 16-byte chunk index of LDS row r (same for K and V
// tiles).  LDS is read 256 bytes (64 banks of 4 bytes) per cycle: 16 lanes of
// a 16-byte read, or 32 lanes of an 8-byte transposing read.
//  d = 128 (a row is one 256-byte bank line, 16 chunks): K operand reads put
//  16 different rows at one logical chunk per cycle -> the XOR must be a
//  bijection on r mod 16; V transposing reads put rows 4k .. 4k + 3 at 4
//  adjacent chunks -> the XORs of those rows must differ in bits 2..3.
//  d = 64 (two rows share a bank line, 8 chunks): the same conditions applied
//  separately to even and odd rows.
template <int D>
__device__ __forceinline__ int swz(int r) {
  static_assert(D == 64 || D == 128, "head dim");
  if constexpr (D == 128)
    return ((r & 3) << 2) | ((r >> 2) & 3);
  else
    return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
}

// Key (within a 32-key group) fed to MFMA row m: bits 2 and 3 of m swapped.
// With this order, register i of the S^T accumulator of lane l holds key
// 16 * (i / 8) + 8 * (l / 32) + (i % 8): eight consecutive keys per half
// wavefront, exactly the B-operand layout of the following P V product.
__device__ __forceinline__ int key_of_row(int m) {
  return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1);
}

// Workgroup barrier after this wave's LDS reads have completed.  Unlike
// __syncthreads() it does not wait for outstanding global->LDS copies.  The
// memory clobber keeps the compiler from moving memory accesses across it.
__device__ __forceinline__ void barrier_lds_reads_done() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Workgroup barrier once all but the VM most recent global->LDS copies of
// every wave have landed (copies complete in issue order).
template <int VM>
__device__ __forceinline__ void barrier_copies_landed() {
  static_assert(VM >= 0 && VM < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(VM) : "memory");
}

// Loads J .. J + COUNT - 1 of a group of four wave-wide direct-to-LDS copies: in
// load j lane l reads 16 bytes at base + off[j] + 1024 j and writes them to LDS
// byte address m0 + 1024 j + 16 l.  Issued as inline assembly so that the
// compiler does not add conservative vmcnt waits before unrelated LDS reads;
// completion is awaited explicitly with barrier_copies_landed().  The
// instruction's offset counts on both sides, so one write of m0 serves a group.
// A direct-to-LDS load needs one wait state after that write, which the compiler
// does not put ahead of inline assembly; with a write and a wait for every load
// masked items of 64 rows were 1-2 % slower (12 heads x 4000 tokens, d = 64,
// density 0.3: 43.5 -> 44.2 us, 41.1 in groups).
template <int J, int COUNT>
__device__ __forceinline__ void copy16_to_lds(uint32_t lds_byte_addr, const void* base,
                                              const uint32_t (&off)[4]) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_byte_addr);
  if constexpr (COUNT == 4)
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %4 offset:0\n\t"
                 "global_load_lds_dwordx4 %1, %4 offset:1024\n\t"
                 "global_load_lds_dwordx4 %2, %4 offset:2048\n\t"
                 "global_load_lds_dwordx4 %3, %4 offset:3072"
                 ::"v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base), "{m0}"(m0)
                 : "memory");
  else if constexpr (COUNT == 2)
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %2 offset:%4\n\t"
                 "global_load_lds_dwordx4 %1, %2 offset:%5"
                 ::"v"(off[J]), "v"(off[J + 1]), "s"(base), "{m0}"(m0), "n"(1024 * J),
                 "n"(1024 * J + 1024) : "memory");
  else
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3"
                 ::"v"(off[J]), "s"(base), "{m0}"(m0), "n"(1024 * J) : "memory");
}

// Per-lane byte offsets of a tile copy.  Lane l of load i writes the 16-byte
// LDS chunk 64 (i + kLoadsPerWave * wave) + l, i.e. row r = R (kLoadsPerWave
// wave + i) + l / C and physical chunk p = l mod C (C chunks per row, R = 64 / C
// rows per load); the XOR swizzle is applied by reading source chunk
// p ^ swz(r).  Source rows are sn elements apart (d for [B][H][N][d] tensors,
// H d for [B][N][H][d]).  The swizzle depends on r mod 16 only, so the lane's
// part of the offset repeats with period 4 in the load index n = kLoadsPerWave
// wave + i, and the rest, R n sn elements, is uniform over the wavefront:
// a plan holds 4 lane offsets, and each load adds its uniform row offset to
// the scalar base address.  (Every real row is congruent mod 16 to the row
// used for its swizzle: R (n - n mod 4) is a multiple of 16.)  The lane offsets
// also hold 3072 - 1024 (i mod 4), which with the kCopyShift elements that the
// base addresses given to the copies lie below their tensors takes back the
// 1024 (i mod 4) of the load instruction (copy16_to_lds).
constexpr int kCopyShift = 3072 / 2;
template <typename T, int D>
struct CopyPlan {
  static constexpr int kRowsPerLoad = 64 / T::kChunksPerRow;
  uint32_t lane_off[4];  // byte offset of the lane's chunk for loads with n mod 4 = m
  __device__ __forceinline__ void init(int wave, int lane, int sn) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = (wave * T::kLoadsPerWave + j) & 3;  // n mod 4 of load j, j + 4, ...
      const int lr = lane / T::kChunksPerRow;
      const int p = lane % T::kChunksPerRow;
      const int r = m * kRowsPerLoad + lr;  // row relative to load n - n mod 4
      lane_off[j] = (uint32_t)(r * sn + ((p ^ swz<D>(r)) << 3)) * 2u + 1024u * (3 - j);
    }
  }
  // wavefront-uniform byte offset of load i: rows R (n - n mod 4)
  __device__ __forceinline__ static int64_t row_off(int wave, int i, int sn) {
    const int n = wave * T::kLoadsPerWave + i;
    return (int64_t)((n & ~3) * kRowsPerLoad) * sn * 2;
  }
};

// Whether the loads of a group are issued one by one (one write of m0, but a
// wait each) instead of in one statement.  Masked items of 64 rows at d = 128
// stream the most tile bytes per flop, and where most of those miss in L2 a
// burst of four waits longer than four loads apart: 20 heads x 67609 tokens,
// unstructured masks, density 0.16, in bursts and one by one 11.22 and 10.96 ms
// (10.93 before copies waited for m0), 40 heads at 0.08 11.00 and 10.61 (10.63);
// 32768 tokens 2.68 and 2.69.  Elsewhere bursts are as fast or faster: 128 x 128
// 0.1-1 %.
template <typename T, int D>
constexpr bool kCopySpread = T::kWaves == 2 && D == 128;

// Loads i0 .. i0 + count - 1 of a copy of rows key0 .. key0 + BK - 1 (rows sn
// elements apart, row 0 at src + kCopyShift) into an LDS tile with global_load_lds_dwordx4 (no
// registers; completion is tracked by vmcnt).  count and i0 are compile-time
// constants wherever this is inlined into an unrolled loop.  In a ragged last
// block, rows past N repeat row N - 1: finite values whose logits are masked
// and whose probabilities are exactly zero.
template <typename T, int BK, int D>
__device__ __forceinline__ void issue_tile_slice(__bf16* lds, const __bf16* src, int key0, int N,
                                                 int sn, int wave_u, int lane,
                                                 const CopyPlan<T, D>& cp, int i0, int count) {
  const char* tile = (const char*)(src + (int64_t)key0 * sn);
  const uint32_t lds0 =
      (uint32_t)(uintptr_t)(SA_LDS void*)lds + (uint32_t)(wave_u * T::kLoadsPerWave * 1024);
  if (key0 + BK <= N) {
    const int step = count % 4 ? 2 : 4;  // slices begin at a multiple of their group's length
#pragma unroll
    for (int i = i0; i < i0 + count; i += step) {
      const char* from = tile + CopyPlan<T, D>::row_off(wave_u, i, sn);
      if (step == 4 && kCopySpread<T, D>) {
        copy16_to_lds<0, 1>(lds0 + i * 1024, from, cp.lane_off);
        copy16_to_lds<1, 1>(lds0 + i * 1024, from, cp.lane_off);
        copy16_to_lds<2, 1>(lds0 + i * 1024, from, cp.lane_off);
        copy16_to_lds<3, 1>(lds0 + i * 1024, from, cp.lane_off);
      } else if (step == 4)
        copy16_to_lds<0, 4>(lds0 + i * 1024, from, cp.lane_off);
      else if ((i & 3) == 0)
        copy16_to_lds<0, 2>(lds0 + i * 1024, from, cp.lane_off);
      else
        copy16_to_lds<2, 2>(lds0 + (i & ~3) * 1024, from, cp.lane_off);
    }
  } else {
    // Row R n + lr of the tile is read from row min(R n + lr, last), addressed
    // from the tile start: lane_off covers rows R (n mod 4) + lr, so the rows
    // still to add are min(R (n - n mod 4), last - R (n mod 4) - lr), which is
    // negative when the clamped row lies below row R (n - n mod 4).  The sum
    // is taken mod 2^32 and equals the true offset, which is non-negative and
    // inside the tile.  (Adding a negative row count to the uniform base of a
    // full-tile load instead would wrap the 32-bit lane offset.)
    const int last = N - 1 - key0;  // last real row of this tile
    int lr = lane / T::kChunksPerRow;
    // opaque to the optimiser: keeps the per-load row sums below from being
    // hoisted out of the block loop, where they would hold 4 registers
    asm volatile("" : "+v"(lr));
#pragma unroll
    for (int i = i0; i < i0 + count; ++i) {
      const int n = wave_u * T::kLoadsPerWave + i;
      constexpr int R = CopyPlan<T, D>::kRowsPerLoad;
      const int rows = min((n & ~3) * R, last - (n & 3) * R - lr);
      uint32_t off[4];
      off[i & 3] = cp.lane_off[i & 3] + (uint32_t)(rows * sn) * 2u;
      const uint32_t to = lds0 + (i & ~3) * 1024;
      switch (i & 3) {
        case 0: copy16_to_lds<0, 1>(to, tile, off); break;
        case 1: copy16_to_lds<1, 1>(to, tile, off); break;
        case 2: copy16_to_lds<2, 1>(to, tile, off); break;
        default: copy16_to_lds<3, 1>(to, tile, off);
      }
    }
  }
}

// A whole tile copy.
template <typename T, int BK, int D>
__device__ __forceinline__ void issue_tile_copy(__bf16* lds, const __bf16* src, int key0, int N,
                                                int sn, int wave_u, int lane,
                                                const CopyPlan<T, D>& cp) {
  issue_tile_slice<T, BK, D>(lds, src, key0, N, sn, wave_u, lane, cp, 0, T::kLoadsPerWave);
}

// Four consecutive outputs of a row: bf16 (round to nearest even) or fp32.
__device__ __forceinline__ void store_out4(__bf16* p, float a, float b, float c, float d) {
  *(bf16x4*)p = bf16x4{(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
}
__device__ __forceinline__ void store_out4(float* p, float a, float b, float c, float d) {
  *(f32x4*)p = f32x4{a, b, c, d};
}

// Output epilogue through LDS.  In the accumulator layout lane l holds 64
// values of query row l mod 32, so a direct store instruction writes 16
// bytes into each of 32 rows.  Here the wavefront's 32 rows, normalised and
// converted, go into a free LDS slice in row-major order (16-byte chunk c of
// row r at chunk c ^ (r mod C), C chunks per row, conflict-free both ways)
// and are read back so that each lane stores 16 contiguous bytes and a store
// instruction covers whole rows.  The slice is this wavefront's own and
// wavefront-local LDS accesses complete in order, so no barrier is needed.
// out0 is row 0 of the wavefront's rows (rows sn elements apart); rows at or
// past n_rows are not stored.
template <int D, typename OutT>
__device__ __forceinline__ void store_rows_staged(const f32x16 (&o)[D / 32], float inv,
                                                  char* slice, OutT* out0, int sn, int n_rows,
                                                  int lane) {
  constexpr int kChunk = 16 / (int)sizeof(OutT);  // elements per 16-byte chunk
  constexpr int C = D / kChunk;                   // chunks per row
  constexpr int kRowBytes = D * (int)sizeof(OutT);
  const int r = lane & 31;
  const int half = lane >> 5;
#pragma unroll
  for (int dg = 0; dg < D / 32; ++dg)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      // elements d = 32 dg + 8 r4 + 4 half + 0..3 of row r
      const float a = o[dg][4 * r4 + 0] * inv, b = o[dg][4 * r4 + 1] * inv;
      const float c = o[dg][4 * r4 + 2] * inv, d = o[dg][4 * r4 + 3] * inv;
      if constexpr (sizeof(OutT) == 2) {
        const int ch = 4 * dg + r4;
        *(SA_LDS bf16x4*)(slice + r * kRowBytes + ((ch ^ (r % C)) << 4) + 8 * half) =
            bf16x4{(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
      } else {
        const int ch = 8 * dg + 2 * r4 + half;
        *(SA_LDS f32x4*)(slice + r * kRowBytes + ((ch ^ (r % C)) << 4)) = f32x4{a, b, c, d};
      }
    }
  constexpr int kRowsPerStore = 64 / C;
  constexpr int kStores = 32 / kRowsPerStore;
  const int cl = lane % C;
  const int rl = lane / C;
  // All read-backs go out before the first store: the empty asm takes each
  // value where it is read, so the reads are not sunk into the guarded
  // stores below, where each would wait for its own LDS round trip.
  u32x4 v[kStores];
#pragma unroll
  for (int j = 0; j < kStores; ++j) {
    const int row = j * kRowsPerStore + rl;
    v[j] = *(const SA_LDS u32x4*)(slice + row * kRowBytes + ((cl ^ (row % C)) << 4));
  }
#pragma unroll
  for (int j = 0; j < kStores; ++j) asm volatile("" : "+v"(v[j]));
#pragma unroll
  for (int j = 0; j < kStores; ++j) {
    const int row = j * kRowsPerStore + rl;
    if (row < n_rows) *(u32x4*)(out0 + ((uint32_t)(row * sn) + (uint32_t)(cl * kChunk))) = v[j];
  }
}

// The staged epilogue needs 32 D sizeof(OutT) bytes per wavefront out of the
// item's K and V tiles (2 BK D bf16).
template <int BQ, int BK, int D, typename OutT>
constexpr bool kStagedStore = BQ * (int)sizeof(OutT) <= 4 * BK;

// DENSE = true is the maskless path: every key block 0 .. n_kb - 1 is enabled
// (counts, lists and order unused) and the items are laid out for the XCDs
// as the schedule lays them out, with the (b, h) groups in index order.
// Occupancy hint (waves per SIMD): two, except for 64 x 128 tiles with d = 128
// (two wavefronts own 128 keys of S and P each), which need more than 256
// registers per wave and run one.
template <int BQ, int BK, int D>
constexpr int kWavesPerSimd = (BQ == 64 && BK == 128 && D == 128) ? 1 : 2;

template <int BQ, int BK, int D, bool DENSE, typename OutT>
__global__ __launch_bounds__(BQ / 32 * 64, (kWavesPerSimd<BQ, BK, D>)) void bsattn_fwd_kernel(
    const __bf16* __restrict__ Q, const __bf16* __restrict__ K, const __bf16* __restrict__ V,
    const int32_t* __restrict__ counts, const int32_t* __restrict__ lists,
    const int32_t* __restrict__ order, OutT* __restrict__ O, float* __restrict__ LSE, int H,
    int N, int n_qb, int n_kb, float c_log2, int64_t sb, int64_t sh, int sn) {
  using T = Tile<BQ, BK, D>;
  constexpr int kL = T::kLoadsPerWave;
  __shared__ __attribute__((aligned(1024))) __bf16 Ks[BK * D];
  __shared__ __attribute__((aligned(1024))) __bf16 Vs[BK * D];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int half = lane >> 5;
  const int l32 = lane & 31;

  // Work item, row count and key blocks come from caller-visible buffers
  // (sa_bsattn_fwd_prepared): they are clamped into range, so malformed
  // input gives wrong values but never an access outside the tensors.
  const int n_items = (int)gridDim.x;
  int item;
  if (DENSE) {  // every group costs the same: the XCD layout of the schedule, groups in index order
    int uu;
    const int unit = xcd_slice(blockIdx.x, n_items / n_qb, n_qb, &uu);
    item = min(max(unit * n_qb + uu, 0), n_items - 1);
  } else {
    item = min(max(order[blockIdx.x], 0), n_items - 1);
  }
  const int bh = item / n_qb;
  const int u = item - bh * n_qb;
  const int h = bh % H;
  const int row = h * n_qb + u;
  const int cnt = DENSE ? n_kb : min(max(counts[row], 0), n_kb);
  const int32_t* list = DENSE ? nullptr : lists + (int64_t)row * n_kb;
  // key block of the t-th enabled block (ascending, as the CRM walk yields them)
  auto kblk = [&](int t) { return DENSE ? t : min(max(list[t], 0), n_kb - 1); };
  const int64_t base = (int64_t)(bh / H) * sb + (int64_t)h * sh;  // element (b, h, token 0, 0)
  const __bf16* Qb = Q + base;
  const __bf16* Kb = K + base - kCopyShift;  // read by tile copies only
  const __bf16* Vb = V + base - kCopyShift;

  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  CopyPlan<T, D> cp;
  cp.init(wave_u, lane, sn);
  if (cnt > 0) issue_tile_copy<T, BK, D>(Ks, Kb, kblk(0) * BK, N, sn, wave_u, lane, cp);

  // Q^T fragments (B operand): lane holds Q[qrow][16 dc + 8 half .. +7].
  // (Staging them through the V tile as the ping-pong kernel does measured
  // 0.2-0.6 % slower here: two more barriers against 16 KB of Q per item.)
  const int qrow = u * BQ + wave * 32 + l32;
  bf16x8 qf[D / 16];
#pragma unroll
  for (int dc = 0; dc < D / 16; ++dc) {
    if (qrow < N)
      qf[dc] = *(const bf16x8*)(Qb + (int64_t)qrow * sn + dc * 16 + half * 8);
    else
      qf[dc] = bf16x8{};
  }

  // Q and the first tiles have landed: the loop below starts with no
  // outstanding vector loads that the compiler would otherwise wait for.
  __builtin_amdgcn_s_waitcnt(0xF70);  // vmcnt(0)

  f32x16 o[D / 32];
#pragma unroll
  for (int dg = 0; dg < D / 32; ++dg) o[dg] = f32x16{};
  float m_run = -INFINITY;  // running max of the log2-domain logits
  float l_run = 0.f;        // this lane's share of the running sum

  const int g = lane >> 4;
  const int j = lane & 15;

  // Copies are issued in slices between compute steps rather than in one
  // burst per tile: V[t] in BK / 32 slices between the key groups of S[t]
  // (its buffer is free once P V[t-1] is done), K[t+1] in two halves inside
  // the softmax of block t (its buffer is free once S[t] is done).  Bursts of
  // copies queue behind each other at issue and hold up the wavefront.
  // A slice is at least a group of four loads, which take one write of m0 (64 x
  // 64 blocks, d = 64, slices of two and of four: 12 heads x 4000 tokens 44.3 and
  // 41.1 us, 10 x 16000 331 and 316, density 0.3; 43.7 and 327 with slices of two
  // before copies waited for m0).
  constexpr int kVSlice = kL / (BK / 32) < 4 ? 4 : kL / (BK / 32);
  constexpr int kKSlice = kL / 2 < 4 ? 4 : kL / 2;
  static_assert(kL % kVSlice == 0 && kL % kKSlice == 0, "copy slices");
  for (int t = 0; t < cnt; ++t) {
    const int key0 = kblk(t) * BK;
    const bool more = t + 1 < cnt;
    const int key1 = more ? kblk(t + 1) * BK : 0;

    barrier_copies_landed<0>();  // K[t] landed (no younger copy is in flight)

    // S^T = K Q^T, one 32-key group per accumulator.
    f32x16 s[BK / 32];
#pragma unroll
    for (int kg = 0; kg < BK / 32; ++kg) {
      s[kg] = f32x16{};
      const int kr = kg * 32 + key_of_row(l32);
#pragma unroll
      for (int dc = 0; dc < D / 16; ++dc) {
        const bf16x8 a = lds_read_b128(Ks + kr * D + (((2 * dc + half) ^ swz<D>(kr)) << 3));
        s[kg] = mfma32x32x16(a, qf[dc], s[kg]);
      }
      if (kg * kVSlice < kL)
        issue_tile_slice<T, BK, D>(Vs, Vb, key0, N, sn, wave_u, lane, cp, kg * kVSlice, kVSlice);
    }

    barrier_lds_reads_done();  // every wave is done with Ks

    if (key0 + BK > N) {  // ragged last block: keys >= N do not exist
#pragma unroll
      for (int kg = 0; kg < BK / 32; ++kg)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = key0 + kg * 32 + 16 * (i >> 3) + 8 * half + (i & 7);
          if (key >= N) s[kg][i] = -INFINITY;
        }
    }

    float mx = -INFINITY;
#pragma unroll
    for (int kg = 0; kg < BK / 32; ++kg)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[kg][i]);
    mx = pair_max(mx) * c_log2;
    if (more) issue_tile_slice<T, BK, D>(Ks, Kb, key1, N, sn, wave_u, lane, cp, 0, kKSlice);
    // Rescale only when some row's maximum grew.  Keeping the exact running
    // maximum (rather than a stale one) makes each row's largest probability
    // exactly 1, which bf16 represents without error.
    const bool grow = mx > m_run;  // always true on the first block
    if (__any(grow)) {
      const float m_new = grow ? mx : m_run;
      const float alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dg = 0; dg < D / 32; ++dg) o[dg] *= alpha;
    }

    bf16x8 pf[BK / 16];
    float lsum = 0.f;
#pragma unroll
    for (int kg = 0; kg < BK / 32; ++kg) {
#pragma unroll
      for (int j8 = 0; j8 < 2; ++j8)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float p = fast_exp2(fmaf(s[kg][8 * j8 + e], c_log2, -m_run));
          lsum += p;
          pf[2 * kg + j8][e] = (__bf16)p;
        }
      if (kg == (BK / 32 - 1) / 2 && kKSlice < kL && more)
        issue_tile_slice<T, BK, D>(Ks, Kb, key1, N, sn, wave_u, lane, cp, kKSlice, kKSlice);
    }
    l_run += lsum;

    if (more)
      barrier_copies_landed<kL>();  // V[t] landed; K[t+1] may still be in flight
    else
      barrier_copies_landed<0>();

    // O^T += V^T P^T.  Lane group g = lane / 16 covers d0 = 32 dg + 16 (g & 1)
    // and keys 16 c + 8 (g >> 1) + 0..7 (two transposing reads of 4 rows).
#pragma unroll
    for (int dg = 0; dg < D / 32; ++dg) {
      const int dd = dg * 32 + 16 * (g & 1) + (j & 3) * 4;
#pragma unroll
      for (int c = 0; c < BK / 16; ++c) {
        const int r0 = c * 16 + 8 * (g >> 1) + (j >> 2);
        const int r1 = r0 + 4;
        const bf16x4 lo = lds_read_tr16_b64(Vs + r0 * D + (((dd >> 3) ^ swz<D>(r0)) << 3) + (dd & 7));
        const bf16x4 hi = lds_read_tr16_b64(Vs + r1 * D + (((dd >> 3) ^ swz<D>(r1)) << 3) + (dd & 7));
        const bf16x8 a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        o[dg] = mfma32x32x16(a, pf[c], o[dg]);
      }
    }

    barrier_lds_reads_done();  // every wave is done with Vs
  }

  // Epilogue addresses are rebuilt from the wave-uniform row base and a lane
  // id recomputed here (mbcnt), so that nothing formed before the loop has to
  // stay live across it.
  const float l_tot = pair_sum(l_run);
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  const int lane_e = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int l32_e = lane_e & 31;
  const int half_e = lane_e >> 5;
  const int row0 = u * BQ + wave_u * 32;  // first query row of this wavefront
  if constexpr (kStagedStore<BQ, BK, D, OutT>) {
    // the loop's last barrier follows every wave's last LDS read, and no copy
    // is outstanding: wavefront w stages its rows in bytes [w S, (w + 1) S)
    // of [Ks | Vs], S = 32 D sizeof(OutT)
    if (half_e == 0 && row0 + l32_e < N)
      LSE[(int64_t)bh * N + row0 + l32_e] = l_tot > 0.f ? (m_run + fast_log2(l_tot)) * kLn2 : -INFINITY;
    constexpr int kSlice = 32 * D * (int)sizeof(OutT);
    constexpr int kTileBytes = BK * D * 2;
    const int off = wave_u * kSlice;
    char* slice = off < kTileBytes ? (char*)Ks + off : (char*)Vs + (off - kTileBytes);
    store_rows_staged<D, OutT>(o, inv, slice, O + base + (int64_t)row0 * sn, sn, N - row0, lane_e);
  } else if (row0 + l32_e < N) {
    if (half_e == 0)
      LSE[(int64_t)bh * N + row0 + l32_e] = l_tot > 0.f ? (m_run + fast_log2(l_tot)) * kLn2 : -INFINITY;
    OutT* orow = (O + base + (int64_t)row0 * sn) + (uint32_t)(l32_e * sn);
#pragma unroll
    for (int dg = 0; dg < D / 32; ++dg)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        store_out4(orow + dg * 32 + 8 * r4 + 4 * half_e, o[dg][4 * r4 + 0] * inv,
                   o[dg][4 * r4 + 1] * inv, o[dg][4 * r4 + 2] * inv, o[dg][4 * r4 + 3] * inv);
  }
}


// Ping-pong workgroups: 8 wavefronts in two groups of 4; a group holds
// 128 / BQ items (one of 128 query rows or two of 64), each item with its own
// K and V tiles in LDS.  Used where those tiles fit the 160 KB of LDS.
template <int BQ, int BK, int D>
struct PingPong {
  static constexpr int kItems = 8 / (BQ / 32);  // items per workgroup
  static constexpr int kLdsBytes = kItems * 2 * BK * D * 2;
  static constexpr bool kFits = kLdsBytes <= 160 * 1024;
};

// Where ping-pong is used: items of 128 query rows (two per workgroup), and
// the maskless path wherever the tiles fit.  Masked items of 64 rows keep one
// item per workgroup: four masked items in lockstep over the largest of their
// counts measured 7-10 % slower than separate workgroups at densities of 0.1
// and 0.25, while the maskless 64 x 64 path gained 5 %.
template <int BQ, int BK, int D, bool DENSE>
constexpr bool kUsePingPong = PingPong<BQ, BK, D>::kFits && (BQ == 128 || DENSE);

// Rows of up to this many key blocks are walked by their first part alone, and
// a workgroup with no others has nothing to put together, which takes 0.5-1.8
// us.  Kernels of rows of 1 / 2 / 3 / 4 blocks, us, without this rule -> with it
// (and not shared): 64 x 64, d = 128, 1 head x 512 tokens 7.4 / 7.5 / 8.3 / 8.5 ->
// 5.6 / 7.0 / 8.3 / 8.5 (5.0 / 6.4 / 7.7 / 9.1); 128 x 128, d = 128, 12 x 1024 7.9 /
// 9.3 / 11.1 / 12.7 -> 6.9 / 9.2 / 11.0 / 12.6 (9.1 / 11.8 / 14.8 / 17.9).  With
// rows of three walked alone too, those take 0.1-0.9 us more.
template <int PARTS>
constexpr int kAlone = PARTS > 1 ? 2 : 0;

// What stands for a maximum of -inf in the exponents of part `part`.  A walk
// over all blocks has a finite maximum when it comes to a block whose logits
// are all -inf, and gives it weights of 0, unless that is its first block,
// whose weights exp2(-inf + inf) are NaN.  So a first part keeps -inf, and the
// later ones, whose walk may begin with such a block, take the lowest finite
// value instead: -inf weighs 0, and NaN stays NaN.
template <int PARTS>
__device__ __forceinline__ float part_floor(int part) {
  return PARTS > 1 && part > 0 ? -3.402823466e+38f : -INFINITY;
}

// Puts together the PARTS parts of the workgroup's shared items: maxima, sums
// and accumulators of parts 1 .. go through LDS into those of part 0, which
// end up as the item's.  Every wavefront of the workgroup calls this, when the
// K and V tiles (KV bytes each) are free; `wave` numbers the WAVES wavefronts
// of a part, and equal lanes of equal wavefronts hold the same elements.  The
// accumulators take WAVES (PARTS - 1) times 128 D bytes; maxima and sums go
// behind them, or ahead of them in a round of their own where the tiles are
// too small for both.
template <int PARTS, int WAVES, int D, int KV>
__device__ __forceinline__ void merge_parts(f32x16 (&o)[D / 32], float& m, float& l, char* k_tiles,
                                            char* v_tiles, int part, int wave, int lane) {
  constexpr int kWaveBytes = 32 * D * 4;
  constexpr int kSums = (PARTS - 1) * WAVES * kWaveBytes;
  constexpr int kStats = (PARTS - 1) * WAVES * 512;
  static_assert(kSums <= 2 * KV && kStats <= KV && KV % kWaveBytes == 0, "the tiles hold the parts");
  constexpr bool kOneRound = kSums + kStats <= 2 * KV;
  auto at = [&](int off) { return off < KV ? k_tiles + off : v_tiles + (off - KV); };
  auto stats = [&](int p) {
    return (SA_LDS float*)(SA_LDS void*)(at((kOneRound ? kSums : 0) + ((p - 1) * WAVES + wave) * 512) +
                                         lane * 8);
  };
  auto sums = [&](int p) { return at(((p - 1) * WAVES + wave) * kWaveBytes) + lane * 16; };
  auto write_sums = [&]() {
#pragma unroll
    for (int i = 0; i < D / 8; ++i)
      *(SA_LDS f32x4*)(sums(part) + i * 1024) =
          f32x4{o[i / 4][4 * (i % 4)], o[i / 4][4 * (i % 4) + 1], o[i / 4][4 * (i % 4) + 2],
                o[i / 4][4 * (i % 4) + 3]};
  };
  if (part > 0) {
    stats(part)[0] = m;
    stats(part)[1] = l;
    if (kOneRound) write_sums();
  }
  barrier_lds_reads_done();
  float scale[PARTS];
  if (part == 0) {
    float mp[PARTS], lp[PARTS];
    mp[0] = m;
    lp[0] = l;
#pragma unroll
    for (int p = 1; p < PARTS; ++p) {
      mp[p] = stats(p)[0];
      lp[p] = stats(p)[1];
      m = fmaxf(m, mp[p]);
    }
    // A part of no key blocks, or of logits that are all -inf, has m = -inf and
    // sums of 0 (see part_floor): a weight of exp2(-inf) = 0 adds nothing.  A
    // part of NaN logits has m = -inf too and sums of NaN, which every weight
    // keeps, as the walk over all blocks in one would.
    l = 0.f;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
      scale[p] = mp[p] == m ? 1.f : fast_exp2(mp[p] - m);
      l = fmaf(scale[p], lp[p], l);
    }
  }
  if (!kOneRound) {
    barrier_lds_reads_done();
    if (part > 0) write_sums();
    barrier_lds_reads_done();
  }
  if (part == 0) {
#pragma unroll
    for (int dg = 0; dg < D / 32; ++dg)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dg][e] *= scale[0];
#pragma unroll
    for (int p = 1; p < PARTS; ++p)
#pragma unroll
      for (int i = 0; i < D / 8; ++i) {
        const f32x4 x = *(const SA_LDS f32x4*)(sums(p) + i * 1024);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[i / 4][4 * (i % 4) + e] = fmaf(scale[p], x[e], o[i / 4][4 * (i % 4) + e]);
      }
  }
  barrier_lds_reads_done();  // the tiles are free again
}

// Whether S requests the K operands of step dc + 1 before the MFMAs of step dc.
// Left to itself the compiler reads each pair just before its use, and every
// pair waits for LDS: an MFMA phase alone on a compute unit takes 3134 cycles
// (128 x 128, d = 128; its 64 MFMAs are 2048), 2712 with the early requests.
// Beside another group's softmax it is 3195 -> 3113, +1.4 % maskless; with
// masks and a full chip, clocked down by its power, it measured -1 to +0.5 %
// and the plain form stays.  Items of 64 rows have no registers to spare: at
// d = 64 it would cost maskless ones the second workgroup of a compute unit.
template <int BQ, bool DENSE, int PARTS>
constexpr bool kReadAhead = BQ == 128 && (DENSE || PARTS > 1);

// Ping-pong kernel.  An 8-wavefront workgroup runs 2 items of 128 query rows
// (or 4 of 64): wavefronts 0-3 and 4-7 form two groups, each item with its
// own K and V tiles in LDS (128 KB at 128 x 128, d = 128: one workgroup per
// CU).  Every SIMD holds one wavefront of each group.  A group's block loop
// alternates two phases separated by workgroup barriers:
//   MFMA phase t:    P V of block t - 1, then S of block t (the MFMAs of a
//                    step rotate over independent accumulators);
//   softmax phase t: copies of V[t] and K[t + 1] issued, then the softmax of
//                    block t; the phase ends once this group's copies landed.
// The second group starts one barrier later, so on every SIMD one group's
// softmax (vector ALU) runs beside the other group's MFMAs: gfx950 co-issues
// the two from different wavefronts, not from one wavefront whose softmax
// depends on its own S.  Both groups pass the same number of barriers: each
// runs max(counts) + 1 MFMA phases and max(counts) softmax phases over the
// workgroup's items, idle where its own item has no block, plus one offset
// barrier.  The items are neighbours in one XCD's sequence of the schedule,
// so they share most key blocks and have similar counts.
//
// PARTS > 1 (bsattn_split_kernel): kItems / PARTS items a workgroup, each
// shared by PARTS slots that take its key blocks in PARTS runs, put together at
// the end (merge_parts).  For problems with fewer items than the chip has
// places, see parts_of().  The two kernels have one body, included as text: as
// an inlined function it was scheduled otherwise (V operands read only when
// they are needed) and ran up to 5 % slower.
constexpr int kMaskWords = 8;  // words of a mask row that the kernel walks itself: 256 items a head at most, 128 x 64 blocks
#define SA_PP_PARAMS                                                                              \
  const __bf16 *__restrict__ Q, const __bf16 *__restrict__ K, const __bf16 *__restrict__ V,       \
      const int32_t *__restrict__ counts, const int32_t *__restrict__ lists,                      \
      const int32_t *__restrict__ order, OutT *__restrict__ O, float *__restrict__ LSE, int H,    \
      int N, int n_qb, int n_kb, float c_log2, int64_t sb, int64_t sh, int sn, int n_items,           \
      int place0, const uint64_t *__restrict__ mask

template <int BQ, int BK, int D, bool DENSE, typename OutT>
__global__ __launch_bounds__(512, 1) void bsattn_fwd_pp_kernel(SA_PP_PARAMS) {
  constexpr int PARTS = 1;
  constexpr bool FROM_MASK = false;
#include "attn_pp_body.h"
}

template <int BQ, int BK, int D, bool DENSE, typename OutT, int PARTS>
__global__ __launch_bounds__(512, 1) void bsattn_split_kernel(SA_PP_PARAMS) {
  constexpr bool FROM_MASK = false;
#include "attn_pp_body.h"
}

// One item a workgroup, its key blocks read off the mask row's words by a
// bit scan (a count of trailing zeros, the lowest bit cleared), which stays in
// scalar registers and takes the place of the list.  With every item on the
// chip at once an order has nothing to give either, so a one-shot call of such
// a shape is this one launch, with no pre-pass, schedule or workspace.
// Those three took longer than the attention: 1 x 1024 tokens, d = 64, blocks
// of 64 49.7 -> 19.0 us a call.
template <int BQ, int BK, int D, typename OutT, int PARTS>
__global__ __launch_bounds__(512, 1) void bsattn_mask_split_kernel(SA_PP_PARAMS) {
  constexpr bool DENSE = false;
  constexpr bool FROM_MASK = true;
#include "attn_pp_body.h"
}
#undef SA_PP_PARAMS

// Parts that an item of n_kb key blocks (where all are on) is shared in, for
// XCD sequences of up to `seq` items.  An XCD has kCus compute units with one
// ping-pong workgroup each, of two items of 128 query rows or four of 64
// (masked items of 64 rows: up to four workgroups of one).  A problem that
// does not fill them leaves units and groups idle, so its items are shared by
// the groups of a workgroup instead, as many to an item as there are compute
// units for.  The rule goes by the shape alone, so that every masked entry
// point and order gives the same bits, and so does the maskless one, up to the
// 512 items from which it has rules of its own (shared_rest, wide tiles).
// Measured, d = 128, start -> shared, us:
//   128 x 128, two parts: maskless 1 head x 16000 tokens 332 -> 175, 2 x 16000
//   337 -> 236; masked 2 x 8000 132 -> 75, 3 x 2000 39 -> 24;
//   64 x 64, four: maskless 1 x 16000 429 -> 156, masked 64 -> 32; two: 4 x
//   8000 228 -> 149 and 132 -> 98.
// One item a workgroup without sharing it gained 5-10 %; past the line sharing
// would cost two rounds of halves for one of pairs.  Rows of 8 key blocks are
// the shortest shared: kernels of a plan, not shared -> shared, us, at densities
// 0.1 / 0.3 / 0.6, 64 x 64, d = 64, 8 heads x 512 tokens 7.4 / 8.7 / 12.0 -> 6.2 /
// 6.8 / 7.4; d = 128, 1 x 512 6.2 / 9.0 / 11.8 -> 7.4 / 8.4 / 9.8 before kAlone, 1 x
// 1024 (16 blocks) 9.1 / 15.9 / 21.5 -> 8.5 / 11.4 / 13.3.  (Maskless tiles of 64
// with d = 64 leave room for a second workgroup on a compute unit, with 126
// registers a lane; masked ones take 146.  The rule counts on one.)
constexpr int kCus = 32;  // compute units of an XCD

inline int parts_of(int64_t seq, int slots, int n_kb) {
  int parts = n_kb >= 8 ? slots : 1;
  while (parts > 1 && seq * parts > kCus * slots) parts /= 2;
  return parts;
}

// Places at the end of every XCD's sequence whose maskless items are shared by
// two slots, in a launch of their own.  All items are of one length, so a
// sequence runs in rounds of kCus workgroups of two items, and a last round of
// up to kCus items leaves half of the compute units or more idle for as long as
// a full one takes; shared, it takes half as long (a fuller one would need two
// such rounds).  Measured start -> shared, us: d = 128, 5 heads x 32760 tokens
// (2.5 rounds) 2572 -> 2426, 5 x 14000 (1.1) 708 -> 577, 2 x 20 x 2000 (1.25)
// 118 -> 104, 40 x 1024 in batches of 2 (1.25, 8 key blocks) 72 -> 68, 20 x
// 33800 (10.4) 10827 -> 10582, 40 x 20000 (12.3) 7649 -> 7527; d = 64, 2 x 20 x
// 2000 81 -> 68.  Masked items differ in length, and those at the end of the
// order are the lightest: there the last round is short already.
inline int64_t shared_rest(int64_t seq, int n_kb) {
  const int64_t rest = seq % (2 * kCus);
  return n_kb >= 8 && seq > 2 * kCus && rest <= kCus ? rest : 0;
}

template <int BQ, int BK, int D, bool DENSE, typename OutT, int PARTS>
hipError_t launch_pp(const AttnArgs& a, int64_t n_items, int64_t place0, int64_t end,
                     hipStream_t stream) {
  // consecutive items of one XCD's sequence per workgroup, places place0 .. end - 1
  constexpr int kItems = PingPong<BQ, BK, D>::kItems / PARTS;
  const int64_t n_wg = kXcds * ((end - place0 + kItems - 1) / kItems);
  auto args = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)n_wg), dim3(512), 0, stream, (const __bf16*)a.q,
                       (const __bf16*)a.k, (const __bf16*)a.v, a.counts, a.lists, a.order,
                       (OutT*)a.out, a.lse, a.H, a.N, a.n_qb, a.n_kb, a.scale * kLog2e, a.sb, a.sh,
                       a.sn, (int)n_items, (int)place0, a.mask_bits);
  };
  if constexpr (kItems == 1 && !DENSE)
    if (a.mask_bits) {
      args(bsattn_mask_split_kernel<BQ, BK, D, OutT, PARTS>);
      return hipGetLastError();
    }
  if constexpr (PARTS == 1)
    args(bsattn_fwd_pp_kernel<BQ, BK, D, DENSE, OutT>);
  else
    args(bsattn_split_kernel<BQ, BK, D, DENSE, OutT, PARTS>);
  return hipGetLastError();
}

template <int BQ, int BK, int D, bool DENSE, typename OutT>
hipError_t launch_tile(const AttnArgs& a, hipStream_t stream) {
  const int64_t n_items = (int64_t)a.B * a.H * a.n_qb;
  const int64_t seq = (n_items + kXcds - 1) / kXcds;  // longest XCD sequence
  if constexpr (PingPong<BQ, BK, D>::kFits && !(DENSE && BQ != BK)) {  // maskless blocks are square
    constexpr int kSlots = PingPong<BQ, BK, D>::kItems;
    const int parts = parts_of(seq, kSlots, a.n_kb);
    if constexpr (kSlots == 4)
      if (parts == 4) return launch_pp<BQ, BK, D, DENSE, OutT, 4>(a, n_items, 0, seq, stream);
    if (parts == 2) return launch_pp<BQ, BK, D, DENSE, OutT, 2>(a, n_items, 0, seq, stream);
  }
  if constexpr (kUsePingPong<BQ, BK, D, DENSE>) {
    if constexpr (DENSE && BQ == 128 && BK == 128) {
      const int64_t rest = shared_rest(seq, a.n_kb);
      if (rest > 0) {
        const hipError_t e = launch_pp<BQ, BK, D, DENSE, OutT, 1>(a, n_items, 0, seq - rest, stream);
        if (e != hipSuccess) return e;
        return launch_pp<BQ, BK, D, DENSE, OutT, 2>(a, n_items, seq - rest, seq, stream);
      }
    }
    return launch_pp<BQ, BK, D, DENSE, OutT, 1>(a, n_items, 0, seq, stream);
  } else {
    hipLaunchKernelGGL((bsattn_fwd_kernel<BQ, BK, D, DENSE, OutT>), dim3((unsigned)n_items),
                       dim3(Tile<BQ, BK, D>::kThreads), 0, stream, (const __bf16*)a.q,
                       (const __bf16*)a.k, (const __bf16*)a.v, a.counts, a.lists, a.order,
                       (OutT*)a.out, a.lse, a.H, a.N, a.n_qb, a.n_kb, a.scale * kLog2e, a.sb,
                       a.sh, a.sn);
    return hipGetLastError();
  }
}

template <int BQ, int BK, bool DENSE, typename OutT>
hipError_t launch_d(const AttnArgs& a, hipStream_t stream) {
  if (a.d == 128) return launch_tile<BQ, BK, 128, DENSE, OutT>(a, stream);
  if (a.d == 64) return launch_tile<BQ, BK, 64, DENSE, OutT>(a, stream);
  return hipErrorInvalidValue;
}

template <bool DENSE, typename OutT>
hipError_t launch_any(const AttnArgs& a, hipStream_t stream) {
  if (a.blk_q == 128 && a.blk_k == 128) return launch_d<128, 128, DENSE, OutT>(a, stream);
  if (a.blk_q == 64 && a.blk_k == 64) return launch_d<64, 64, DENSE, OutT>(a, stream);
  if (a.blk_q == 128 && a.blk_k == 64) return launch_d<128, 64, DENSE, OutT>(a, stream);
  if (a.blk_q == 64 && a.blk_k == 128) return launch_d<64, 128, DENSE, OutT>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace

bool attention_reads_mask(int B, int H, int n_qb, int n_kb, int d, int blk_q, int blk_k) {
  const int slots = blk_q == 128 ? 2 : 4;
  if (slots * 4 * blk_k * d > 160 * 1024) return false;  // PingPong::kFits
  const int64_t seq = ((int64_t)B * H * n_qb + kXcds - 1) / kXcds;
  return n_kb <= 64 * kMaskWords && parts_of(seq, slots, n_kb) == slots;
}

hipError_t launch_attention(const AttnArgs& a, hipStream_t stream) {
  if (a.mask_bits && !attention_reads_mask(a.B, a.H, a.n_qb, a.n_kb, a.d, a.blk_q, a.blk_k))
    return hipErrorInvalidValue;
  return a.out_f32 ? launch_any<false, float>(a, stream) : launch_any<false, __bf16>(a, stream);
}

hipError_t launch_attention_dense(const AttnArgs& a, hipStream_t stream) {
  if (a.out_f32) return hipErrorInvalidValue;  // the maskless path writes bf16 only
  // Without a mask the block size is only a tile size.  Where tiles of 64 would
  // run unshared (parts_of), 128 x 128 tiles read half the K and V bytes per
  // query and are faster (12 heads x 4000 tokens, d = 128: 133 -> 116 us).  The
  // line is where no padding to 128 outweighs that: kernel in us, tiles of 64 and
  // of 128, d = 64, 65 x 512 20.5 and 15.4, 80 x 520 23.5 and 19.0, 60 x 580 23.9
  // and 18.5, d = 128 29.8 and 21.2, 35.5 and 27.8, 33.8 and 25.0; below it 100 x
  // 440 22.2 and 17.5, but 200 x 300 21.1 and 27.4 (d = 128 32.7 and 36.8).
  const int64_t items = (int64_t)a.B * a.H * a.n_qb;
  if (a.blk_q == 64 && a.N >= 512 && parts_of((items + kXcds - 1) / kXcds, 4, a.n_kb) == 1) {
    AttnArgs wide = a;
    wide.blk_q = wide.blk_k = 128;
    wide.n_qb = wide.n_kb = (a.N + 127) / 128;
    return launch_any<true, __bf16>(wide, stream);
  }
  return launch_any<true, __bf16>(a, stream);
}

}  // namespace sa
