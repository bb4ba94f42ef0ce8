// Down GEMM with per-group dequantization (Sec. 3.4) on 64 x 128 output tiles,
// for grids of at most one workgroup per CU (small row counts, small models).
// Such a grid is bound by how fast each CU can pull its own weights, not by the
// matrix cores, and a tile that stages weights in LDS has only two K-groups of
// them in flight. Here every weight row belongs to one wavefront, which takes
// it straight into registers, four K-groups ahead; only the 64 activation rows
// (8 KB per K-group), which all wavefronts read, pass through LDS.
//
//   * 8 wavefronts multiply: 64 rows x 16 output columns each, over one K split.
//   * 2 wavefronts copy the activation codes and row scales, direct to LDS, in
//     chunks of 4 K-groups into a ring of 3, with a barrier per chunk; the block
//     scales of the split go to LDS at the start.
//   * The weights (tile layout: two contiguous 1 KB halves per 16 rows and
//     K-group) are refilled in straight-line code, so that the compiler waits
//     for one K-group at a time. Activation operands are read from LDS a K-group
//     ahead (with two row groups ahead, in order, the whole FFN at M = 128 took
//     1.5 us more).
// The products, scales and the order of an element's K-groups are those of the
// tiled kernel: the same bits for the same K splits.
//
// Against the tiled kernel's 64 x 128 tiles over the same K splits, whole FFN in
// sequence with weights from memory, in us: H = 4096, I = 12288, M = 96 59.2 ->
// 57.9, 128 60.4 and 60.4, 256 72.5 -> 70.3; H = 3072, I = 8192, M = 180 40.9 ->
// 38.3, 512 60.9 -> 58.5; H = 2048, I = 6144, M = 256 31.8 -> 30.5; H = 7168, I =
// 2048, M = 190 51.9 -> 50.5; H = 1024, I = 3072, M = 150 25.8 -> 24.6. The same
// scheme for the gate/up GEMM (two slabs per wavefront) gained nothing: 100 MB
// over 96 column tiles stream in 24.7 us with no products at all (192 tiles that
// share no weights: 19.3), and the tiled kernel's loop hides under that.
#include "device.h"
#include "launch.h"

namespace lacache {
namespace {

constexpr int kRows = 64;        // activation rows per tile
constexpr int kMT = kRows / 16;  // row groups of an MFMA
constexpr int kMul = 8;          // wavefronts that multiply
constexpr int kCopiers = 2;      // wavefronts that copy
constexpr int kChunk = 4;        // K-groups per chunk
constexpr int kRing = 3;         // chunks in the ring
constexpr int kMaxGroups = 128;  // K-groups of a split, at most (block scales in LDS)
constexpr int kThreads = (kMul + kCopiers) * 64;

__global__ __launch_bounds__(kThreads) void down_rows64_kernel(
    const uint8_t* __restrict__ hq, const float* __restrict__ hs,  // [M x I] codes, [I/128 x M] scales
    const uint8_t* __restrict__ wq, const float* __restrict__ ws,  // [H x I] codes (tile layout), [H/128 x I/128] scales
    uint16_t* __restrict__ out, float* __restrict__ out_tap, float* __restrict__ part, int M, int64_t I, int64_t H,
    int KS) {
  __shared__ __align__(16) uint8_t ring[kRing][kChunk][kRows * 128];
  __shared__ __align__(16) float sXs[kRing][kChunk][kRows];
  __shared__ __align__(16) float sWs[kMaxGroups];
  const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
  const int q = lane >> 4, lr = lane & 15;
  const int KB = static_cast<int>(I / 128);
  // item: the (up to 4) row tiles of a column and K split, which share its
  // weights, one after the other on one XCD (with the splits among the row tiles,
  // as in the tiled kernel, 3 row tiles of a split fell on two XCDs: whole FFN at
  // H = 3072, I = 8192, M = 180 38.9 -> 38.1 us, H = 4096, I = 12288, M = 96 59.1
  // -> 58.3)
  const int R = (M + kRows - 1) / kRows, C = static_cast<int>(H / 128);
  int rt, vc;
  xcd_grouped_tile(static_cast<int>(blockIdx.x), R, C * KS, rt, vc);
  const int m0 = rt * kRows, ct = vc % C, split = vc / C;
  const int kb0 = split * KB / KS, nkb = (split + 1) * KB / KS - kb0;
  const int nch = (nkb + kChunk - 1) / kChunk;

  if (wave >= kMul) {
    // copier v: rows 32 v .. 32 v + 31 of each K-group, the row scales of K-groups
    // 2 v and 2 v + 1 of each chunk. Rows past M repeat the last (never stored);
    // K-groups past the end repeat the last (never used).
    const int cw = wave - kMul, alim = M - 1 - m0;
    uint32_t a_off[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = 8 * (4 * cw + u) + (lane >> 3);
      a_off[u] = static_cast<uint32_t>(row < alim ? row : alim) * static_cast<uint32_t>(I) +
                 (((lane & 7) ^ swz(row)) << 4);
    }
    const uint32_t x_off = static_cast<uint32_t>(lane < alim ? lane : alim) * 4;
    const uint8_t* a_base = hq + static_cast<int64_t>(m0) * I + static_cast<int64_t>(kb0) * 128;
    const float* x_base = hs + static_cast<int64_t>(kb0) * M + m0;
    auto copy_chunk = [&](int c) {
      const int slot = c % kRing;
#pragma unroll
      for (int k = 0; k < kChunk; ++k) {
        const int kb = c * kChunk + k < nkb ? c * kChunk + k : nkb - 1;
        const uint32_t lds = lds_u32(&ring[slot][k][0]) + 4 * cw * 1024;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          dma16s(a_base + static_cast<int64_t>(kb) * 128, a_off[u], wave_uniform(lds + u * 1024));
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int kk = 2 * cw + k, kb = c * kChunk + kk < nkb ? c * kChunk + kk : nkb - 1;
        dma4s(x_base + static_cast<int64_t>(kb) * M, x_off, wave_uniform(lds_u32(&sXs[slot][kk][0])));
      }
    };
    // the block scales, half of kMaxGroups by each copier
    const int kb = 64 * cw + lane;
    dma4s(ws + static_cast<int64_t>(ct) * KB + kb0, static_cast<uint32_t>(kb < nkb ? kb : nkb - 1) * 4,
          wave_uniform(lds_u32(&sWs[64 * cw])));
    copy_chunk(0);
    copy_chunk(1);
    for (int c = 0; c < nch; ++c) {
      wait_vm<kChunk * 4 + 2>();  // this wavefront's copies of chunk c (those of c + 1 may fly)
      bar();                      // ... and everyone's; chunk c - 1 is read by no one
      copy_chunk(c + 2);
    }
    wait_vm<0>();  // (no copy outlives its wavefront)
    return;
  }

  const int64_t row0 = static_cast<int64_t>(ct) * 128 + 16 * wave;  // this wavefront's weight rows
  const uint8_t* wp = wq + wtile_off(row0, 0, I) + static_cast<int64_t>(kb0) * 2048;
  const uint32_t w_off = static_cast<uint32_t>(lr * 64 + 16 * q);
  u4v wr[kChunk][2];
  auto load_w = [&](int j, int slot) {
    const uint8_t* base = wp + static_cast<int64_t>(j < nkb ? j : nkb - 1) * 2048;
    wr[slot][0] = *reinterpret_cast<const u4v*>(base + w_off);
    wr[slot][1] = *reinterpret_cast<const u4v*>(base + w_off + 1024);
  };
#pragma unroll
  for (int u = 0; u < kChunk; ++u) load_w(u, u);

  float acc[kMT][4];
#pragma unroll
  for (int i = 0; i < kMT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i][r] = 0.0f;
  // operands and scales of row group s % kMT of K-group s / kMT of a chunk
  constexpr int kAhead = kMT;
  v8i af[kAhead + 1];
  float xr[kAhead + 1];
  float w = 0.0f;
  auto read_a = [&](int slot, int s) {
    const int u = s / kMT, row = 16 * (s % kMT) + lr;
    const uint8_t* tile = &ring[slot][u][row * 128];
    af[s % (kAhead + 1)] = cat_frag(*reinterpret_cast<const u4v*>(tile + ((q ^ swz(row)) << 4)),
                               *reinterpret_cast<const u4v*>(tile + (((4 + q) ^ swz(row)) << 4)));
    xr[s % (kAhead + 1)] = sXs[slot][u][row];
  };
  auto group = [&](int c, int s) {
    const int u = s / kMT, i = s % kMT;
    if (i == 0) w = sWs[c * kChunk + u];
    if (s + kAhead < kChunk * kMT) read_a(c % kRing, s + kAhead);
    const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const v4f p = mfma_fp8_16x16x128(cat_frag(wr[u][0], wr[u][1]), af[s % (kAhead + 1)], zero);
    const float sc = xr[s % (kAhead + 1)] * w;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i][r] = __builtin_fmaf(p[r], sc, acc[i][r]);
    if (i == kMT - 1) __builtin_amdgcn_sched_barrier(0);
  };
  for (int c = 0; c + 1 < nch; ++c) {
    bar();
#pragma unroll
    for (int s = 0; s < kAhead; ++s) read_a(c % kRing, s);
#pragma unroll
    for (int s = 0; s < kChunk * kMT; ++s) {
      group(c, s);
      if (s % kMT == kMT - 1) load_w((c + 1) * kChunk + s / kMT, s / kMT);
    }
  }
  const int last = nch - 1;
  bar();
#pragma unroll
  for (int s = 0; s < kAhead; ++s) read_a(last % kRing, s);
#pragma unroll
  for (int u = 0; u < kChunk; ++u)
    if (last * kChunk + u < nkb) {
#pragma unroll
      for (int i = 0; i < kMT; ++i) group(last, u * kMT + i);
    }

  const int64_t col = row0 + 4 * q;
#pragma unroll
  for (int i = 0; i < kMT; ++i) {
    const int64_t m = m0 + 16 * i + lr;
    if (m >= M) continue;
    const float4 v = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    if (KS > 1) {
      *reinterpret_cast<float4*>(part + (static_cast<int64_t>(split) * M + m) * H + col) = v;
    } else {
      *reinterpret_cast<uint2*>(out + m * H + col) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
      if (out_tap != nullptr) *reinterpret_cast<float4*>(out_tap + m * H + col) = v;
    }
  }
}

}  // namespace

// One workgroup per CU at most: over several rounds the tiled kernel, whose
// workgroups walk several items with their copies running on, is the better one
// (whole FFN, tiled and this kernel: H = 16384, I = 24576, M = 156, three rounds
// 379.5 and 381.7 us; H = 3072, I = 8192, M = 435, two rounds 63.3 and 63.8, M =
// 404 65.0 and 64.4).
bool down_rows64_ok(int64_t M, int64_t H, int64_t I, int ks) {
  return (M + kRows - 1) / kRows * (H / 128) * ks <= device_cu_count() && (I / 128 + ks - 1) / ks <= kMaxGroups;
}

hipError_t launch_down_rows64(hipStream_t st, const uint8_t* hq, const float* hs, const uint8_t* wq, const float* ws,
                              uint16_t* out, float* out_tap, float* part, int64_t M, int64_t H, int64_t I, int ks) {
  const unsigned grid = static_cast<unsigned>((M + kRows - 1) / kRows * (H / 128) * ks);
  hipLaunchKernelGGL(down_rows64_kernel, dim3(grid), dim3(kThreads), 0, st, hq, hs, wq, ws, out, out_tap, part,
                     static_cast<int>(M), I, H, ks);
  return hipGetLastError();
}

}  // namespace lacache
