// Token-wise first-layer operators with EmbedCache and RoPECache (Sec. 3.3):
// inside a SAR block only the rows of the current block C change, so the
// embedding, the attention RMSNorm, the QKV projection and RoPE run on those
// rows only and write their results into the cached tensors (the embedding
// cache [N x H] and Q, K, V [heads x N x 128] in the attention layout). The
// first layer keeps 16-bit precision (Sec. 3.4): bf16 storage, fp32
// arithmetic.
//
//   embed_rmsnorm_kernel  one wavefront per row: gather the token's embedding
//                         row, write it to the embedding cache, RMSNorm (the
//                         fused FFN quantizer's arithmetic: fp64 sum of squares
//                         in the same fixed order) rounded to bf16;
//   linear_bf16_kernel    out = a W^T for a few rows: 16 or 48 weight rows per
//                         workgroup streamed from HBM once per 64 activation
//                         rows, K split over the 4 wavefronts (private
//                         direct-to-LDS rings), bf16 MFMAs into fp32, the four
//                         partials added in wavefront order, bf16 out;
//   linear_bf16_tiled_kernel  the same result for many rows, from 128 x 128,
//                         128 x 192 or 256 x 192 output tiles;
//   rope_scatter_kernel   rotate-half RoPE of the Q and K heads from fp32 cos /
//                         sin tables, V unrotated, scattered to each row's
//                         position in Q, K, V, as a stage of its own; the whole
//                         call does the same in the projection's epilogue.
// Token ids outside [0, vocab) and row indices outside [0, N) are skipped on
// the device (no access is made for them).
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace lacache {
namespace {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// A row belongs to 1 << wpr_log2 wavefronts of a workgroup: each reads the row
// and takes the whole sum (the fixed order is one chain of 8 T fp64 FMAs per
// lane), and normalizes and writes the passes t with t mod (1 << wpr_log2)
// equal to its index, which shortens a short call (the first layer at 32 rows of
// 4096: 26.4 us with one wavefront per row, 24.6 with four).
// dst (nullable) [R]: the row's position, or -1 where its token id or position is
// out of range (nothing else is written for it), for the projection's epilogue.
template <int T>
__global__ __launch_bounds__(256) void embed_rmsnorm_kernel(const int32_t* __restrict__ ids,
                                                            const int32_t* __restrict__ rows, int64_t R,
                                                            const uint16_t* __restrict__ embed, int64_t vocab,
                                                            const uint16_t* __restrict__ nw,
                                                            uint16_t* __restrict__ cache, int64_t N,
                                                            uint16_t* __restrict__ y, int H, int wpr_log2,
                                                            int32_t* __restrict__ dst) {
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int part = wave & ((1 << wpr_log2) - 1);
  const int64_t r = (static_cast<int64_t>(blockIdx.x) * 4 + wave) >> wpr_log2;
  if (r >= R) return;  // uniform per wavefront
  const int64_t id = ids[r], pos = rows[r];
  const bool ok = id >= 0 && id < vocab && pos >= 0 && pos < N;
  if (dst != nullptr && part == 0 && lane == 0) dst[r] = ok ? static_cast<int32_t>(pos) : -1;
  if (!ok) return;
  const int nchunk = H >> 3;
  const uint4* xr = reinterpret_cast<const uint4*>(embed + id * H);
  const uint4* wr = reinterpret_cast<const uint4*>(nw);
  uint4 xv[T], wv[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int c = t * 64 + lane;
    const int cc = c < nchunk ? c : nchunk - 1;
    xv[t] = xr[cc];
    wv[t] = wr[cc];
  }
  uint4* cw = reinterpret_cast<uint4*>(cache + pos * H);  // EmbedCache row
#pragma unroll
  for (int t = 0; t < T; ++t) {
    if (t * 64 + lane >= nchunk)
      xv[t] = make_uint4(0u, 0u, 0u, 0u);
    else if ((t & ((1 << wpr_log2) - 1)) == part)
      cw[t * 64 + lane] = xv[t];
  }
  // fp64 sum of squares: per-lane partials in increasing element index, then
  // a xor butterfly over offsets 32..1 (every lane ends with the same bits)
  double p = 0.0;
#pragma unroll
  for (int t = 0; t < T; ++t) p = sumsq8(p, xv[t]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) p = p + __shfl_xor(p, o, 64);
  const float rs = rms_inv(p, H);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int c = t * 64 + lane;
    if ((t & ((1 << wpr_log2) - 1)) != part || c >= nchunk) continue;
    float n[8];
    norm8(xv[t], wv[t], rs, n);
    uint32_t o[4];
    bool nan = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      nan |= __builtin_isunordered(n[2 * e], n[2 * e + 1]) != 0;
      o[e] = cvt_pk_bf16(n[2 * e], n[2 * e + 1]);
    }
    if (__builtin_expect(nan, 0)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = bf16x2_quiet(o[e]);
    }
    reinterpret_cast<uint4*>(y + r * H)[c] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// The RoPE + scatter of rope_scatter_kernel as the epilogue of the two
// projection kernels below (kRope; W is then w_qkv, N = 3 heads 128): the
// projection's rows are rounded to bf16, rotated and written to their places
// in q, k, v, and never go through memory. A tile's columns are then not
// consecutive: a pair (i, i + 64) of a head meets in one wavefront, so the
// tile takes P consecutive pairs of the 64 3 heads (pair p: head p / 64, i =
// p mod 64) and weight rows i and i + 64 for each. Rows whose position is
// outside [0, N) write nothing (the whole call passes the positions that the
// embedding kernel checked: the y of a row with a bad token id is never written).
struct RopeArgs {
  const int32_t* rows;
  const float* cs;
  const float* sn;
  uint16_t* q;
  uint16_t* k;
  uint16_t* v;
  int heads;
  int64_t N;
};
__device__ __forceinline__ uint16_t* rope_dst(const RopeArgs& ra, int head) {
  const int part = head / ra.heads;
  return (part == 0 ? ra.q : (part == 1 ? ra.k : ra.v)) + static_cast<int64_t>(head - part * ra.heads) * ra.N * 128;
}

// The four bf16 values that this lane stored at p, NaNs as 0x7FC0.
__device__ __forceinline__ void quiet_stored(uint2* p) {
  const uint2 v = *p;
  *p = make_uint2(bf16x2_quiet(v.x), bf16x2_quiet(v.y));
}

// out [M x N] = a [M x K] W[N x K]^T, bf16 in and out, fp32 accumulation.
// Workgroup (blockIdx.x, blockIdx.y): weight rows 16 NJ x .. (NJ slabs of
// 16), activation rows 64 y .. + 63 (MT slabs of 16 rows). Its 4 wavefronts
// take a quarter of the K range each; a K-step is 64 elements (128 bytes of a
// row), staged global -> LDS as [rows][128 B] with the 16-byte chunk c of
// row r at c ^ (r mod 8); each 16x16 tile gets two 16x16x32 bf16 MFMAs per
// K-step (the lanes' chunks q and 4 + q). Several weight slabs per workgroup
// share each staged activation row, so the activations (re-read from L2 by
// every workgroup) cost less of the CU's copy bandwidth than the weights.
constexpr int kLinSplit = 4;

template <int MT, int NJ>
struct LinCfg {
  static constexpr int RA = MT * 16;
  static constexpr int kA = RA * 128;
  static constexpr int kSlot = kA + NJ * 16 * 128;
  static constexpr int AI = RA / 8;  // 1 KB copies of activations per slot
  static constexpr int PER = AI + 2 * NJ;
  static constexpr int D0 = 160000 / (kLinSplit * kSlot);  // ring depth that fits the LDS
  static constexpr int D = D0 > 8 ? 8 : D0;
  static_assert(D >= 2, "ring depth");
};

__device__ __forceinline__ void lin_frag(const uint8_t* rows, int lr, int q, bf8& lo, bf8& hi) {
  const uint8_t* row = rows + lr * 128;
  lo = *reinterpret_cast<const bf8*>(row + ((q ^ (lr & 7)) << 4));
  hi = *reinterpret_cast<const bf8*>(row + (((4 + q) ^ (lr & 7)) << 4));
}

//
// kRope: a slab is 8 pairs, rows i .. i + 7 of a head and then i + 64 .. i + 71.
template <int MT, int NJ, bool kRope>
__global__ __launch_bounds__(kLinSplit * 64) void linear_bf16_kernel(const uint16_t* __restrict__ a,
                                                                     const uint16_t* __restrict__ w,
                                                                     uint16_t* __restrict__ out,
                                                                     float* __restrict__ out_tap, int64_t M,
                                                                     int64_t N, int64_t K, RopeArgs ra) {
  using C = LinCfg<MT, NJ>;
  constexpr int D = C::D, RA = C::RA, NC = 16 * NJ;
  __shared__ __align__(16) uint8_t ring[kLinSplit][D * C::kSlot];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = wave_uniform(t >> 6);
  const int q = lane >> 4, lr = lane & 15;
  const int64_t n0 = static_cast<int64_t>(blockIdx.x) * NC;
  const int64_t m0 = static_cast<int64_t>(blockIdx.y) * 64;
  const int64_t KS = K / 64;  // K-steps
  const int64_t ks0 = wave * KS / kLinSplit, ks1 = (wave + 1) * KS / kLinSplit;
  const int nks = static_cast<int>(ks1 - ks0);
  uint8_t* my = ring[wave];
  const uint8_t* ab = reinterpret_cast<const uint8_t*>(a);
  const uint8_t* wb = reinterpret_cast<const uint8_t*>(w);

  // copy plan: instruction u fills slot rows 8u..8u+7; lane l fills row
  // 8u + l/8, physical chunk l%8 (logical chunk (l%8) ^ (row & 7))
  const int crow = lane >> 3, pch = lane & 7;
  int64_t a_off[C::AI];
#pragma unroll
  for (int u = 0; u < C::AI; ++u) {
    const int row = 8 * u + crow;
    const int64_t gr = m0 + row < M ? m0 + row : M - 1;
    a_off[u] = gr * K * 2 + ((pch ^ (row & 7)) << 4);
  }
  int64_t w_off[2 * NJ];
#pragma unroll
  for (int u = 0; u < 2 * NJ; ++u) {
    const int row = 8 * u + crow;
    int64_t wrow = n0 + row;
    if (kRope) {  // 8 pairs of slab u / 2, the lower rows (u even) or the upper
      const int64_t p0 = n0 / 2 + 8 * (u >> 1);
      wrow = (p0 >> 6) * 128 + (p0 & 63) + 64 * (u & 1) + crow;
    }
    w_off[u] = wrow * K * 2 + ((pch ^ (row & 7)) << 4);
  }
  auto issue = [&](int s, int slot) {
    const int64_t kb = (ks0 + (s < nks ? s : nks - 1)) * 128;  // byte offset of the K-step
    const uint32_t base = lds_u32(my + slot * C::kSlot);
#pragma unroll
    for (int u = 0; u < C::AI; ++u) dma16(ab + a_off[u] + kb, wave_uniform(static_cast<int>(base) + u * 1024));
#pragma unroll
    for (int u = 0; u < 2 * NJ; ++u)
      dma16(wb + w_off[u] + kb, wave_uniform(static_cast<int>(base) + C::kA + u * 1024));
  };
  if (nks > 0) {
#pragma unroll
    for (int s = 0; s < D - 1; ++s) issue(s, s);
  }
  v4f acc[MT][NJ];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  for (int s = 0; s < nks; ++s) {
    wait_vm_lds<(D - 2) * C::PER>();  // step s has landed; slot (s-1) % D is read
    issue(s + D - 1, (s + D - 1) % D);
    const uint8_t* slot = my + (s % D) * C::kSlot;
    bf8 alo[MT], ahi[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) lin_frag(slot + i * 16 * 128, lr, q, alo[i], ahi[i]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      bf8 blo, bhi;
      lin_frag(slot + C::kA + j * 16 * 128, lr, q, blo, bhi);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo[i], blo, acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[i], bhi, acc[i][j], 0, 0, 0);
      }
    }
  }
  wait_vm<0>();
  __syncthreads();  // every ring is idle: reuse it for the partials
  float* red = reinterpret_cast<float*>(&ring[0][0]);
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[(wave * RA + 16 * i + 4 * q + r) * NC + 16 * j + lr] = acc[i][j][r];
  __syncthreads();
  if (kRope) {
    for (int e = t; e < RA * (NC / 2); e += kLinSplit * 64) {
      const int row = e / (NC / 2), p = e - row * (NC / 2);
      if (m0 + row >= M) continue;
      const int64_t pos = ra.rows[m0 + row];
      if (pos < 0 || pos >= ra.N) continue;
      const int lo = row * NC + 16 * (p >> 3) + (p & 7);  // the pair's upper row is 8 columns on
      float x = red[lo], y = red[lo + 8];
#pragma unroll
      for (int wv = 1; wv < kLinSplit; ++wv) {
        x += red[wv * RA * NC + lo];
        y += red[wv * RA * NC + lo + 8];
      }
      const int pair = static_cast<int>(n0 / 2) + p, head = pair >> 6, i = pair & 63;
      uint16_t* dst = rope_dst(ra, head) + pos * 128 + i;
      uint32_t xy = cvt_pk_bf16(x, y);
      if (head < 2 * ra.heads) {
        const float c = ra.cs[pos * 64 + i], s = ra.sn[pos * 64 + i], xb = bf16lo(xy), yb = bf16hi(xy);
        x = xb * c - yb * s;
        y = yb * c + xb * s;
        xy = cvt_pk_bf16(x, y);
      }
      if (__builtin_isunordered(x, y)) xy = bf16x2_quiet(xy);
      dst[0] = static_cast<uint16_t>(xy);
      dst[64] = static_cast<uint16_t>(xy >> 16);
    }
    return;
  }
  for (int e = t; e < RA * NC; e += kLinSplit * 64) {
    const int row = e / NC, col = e - row * NC;
    if (m0 + row >= M) continue;
    float sum = red[row * NC + col];
#pragma unroll
    for (int wv = 1; wv < kLinSplit; ++wv) sum += red[(wv * RA + row) * NC + col];
    out[(m0 + row) * N + n0 + col] = static_cast<uint16_t>(sum == sum ? cvt_pk_bf16(sum, 0.0f) : 0x7FC0u);
    if (out_tap != nullptr) out_tap[(m0 + row) * N + n0 + col] = sum;
  }
}

// out = a W^T for many rows: BM x BN output tiles, 8 wavefronts (4 bands of
// BM/4 activation rows x 2 bands of BN/2 weight rows), walked by a grid of at
// most one workgroup per CU in the XCD-grouped order (the row tiles that share
// a weight tile run on one L2). A K-step is 64 elements (128 bytes of a row:
// 64-byte row pieces would halve the rate at which a CU copies from L2, 65
// against 120-130 GB/s measured with 256 CUs copying). Wavefronts 0-3 copy the
// activation rows, wavefronts 4-7 the weight rows; separate wavefronts and
// rings, because a wavefront's copies retire in order and the weights, which
// come from HBM, need the deeper ring where the LDS does not hold both deep. Every output element gets exactly the arithmetic of
// linear_bf16_kernel: the same four K quarters, each a chain of the same
// 16x16x32 bf16 MFMAs in K order started from zero, and the quarter sums added
// in quarter order (the total starts from +0, which adds exactly: a chain that
// starts from +0 never ends in -0). So a row's result does not depend on which
// of the two kernels computed it, and a block update of the caches still
// equals a full recompute bit for bit.
//
// LDS operand reads bound the 128-row tiles: a wavefront reads MT + NT slabs
// (1 KB each) for MT NT MFMAs of 16 cycles, and the LDS gives 128 bytes per
// cycle, so half a K-step of 8 wavefronts needs 64 (MT + NT) LDS cycles beside
// 32 MT NT cycles of MFMA work per SIMD: 640 against 768 at 256 x 192, but 512
// against 384 at 128 x 192. The two accumulator sets of the 256 x 192 tile (192
// registers) leave no room to read a half step's operands ahead, so there the
// two wavefronts of a SIMD alternate (kPing): one reads its operands and
// issues copies while the other multiplies, a barrier between the phases.
constexpr int kLtWaves = 8;
#ifndef LACACHE_LIN_TILED_MIN_M
#define LACACHE_LIN_TILED_MIN_M 128
#endif
constexpr int64_t kLinTiledMinM = LACACHE_LIN_TILED_MIN_M;  // rows above which the tiled kernel runs

// kRope: a wavefront's NT slabs are NT/2 slabs of 16 pairs' lower rows, then
// the same pairs' upper rows (weight rows 64 on).
template <int BM, int BN, bool kPing, bool kRope>
__global__ __launch_bounds__(kLtWaves * 64) void linear_bf16_tiled_kernel(const uint16_t* __restrict__ a,
                                                                        const uint16_t* __restrict__ w,
                                                                        uint16_t* __restrict__ out,
                                                                        float* __restrict__ out_tap, int64_t M,
                                                                        int64_t N, int64_t K, int R, int C,
                                                                        RopeArgs ra) {
  constexpr int kA = BM * 128, kB = BN * 128;  // bytes of a K-step's activation and weight rows
  // steps in the two rings (a power of two of activations): 4 and 4, or 2 and 4 at 256 x 192
  constexpr int DA = 4 * (kA + kB) <= 163840 ? 4 : 2;
  constexpr int DB = (163840 - DA * kA) / kB > 4 ? 4 : (163840 - DA * kA) / kB;
  constexpr int MT = BM / 64, NT = BN / 32;
  constexpr int PA = BM / 32, PB = BN / 32;  // copies per step of an activation / a weight copy wavefront
  constexpr int PM = PA > PB ? PA : PB;
  static_assert(BM % 64 == 0 && BN % 32 == 0 && DB >= 3, "tile shape");
  __shared__ __align__(16) uint8_t sA[DA][kA];
  __shared__ __align__(16) uint8_t sB[DB][kB];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = wave_uniform(t >> 6);
  const int q = lane >> 4, lr = lane & 15;
  const int wm = wave >> 1, wn = wave & 1;
  const bool late = wave >= 4;  // copies weights; with kPing half a phase behind the others
  const int KS = static_cast<int>(K / 64);
  const uint32_t K2 = static_cast<uint32_t>(K) * 2u;
  // copy plan: copy u of wavefront v fills tile rows 8 g .. 8 g + 7, g = v % 4
  // + 4 u; lane l fills row l/8, physical chunk l%8, i.e. logical chunk (l%8) ^
  // ((row/2) mod 8), which spreads the 16 rows of an operand read over all banks
  const int crow = lane >> 3;
  const uint32_t cchunk = static_cast<uint32_t>(((lane & 7) ^ (4 * (wave & 1) + (crow >> 1))) << 4);
  const uint32_t coff = static_cast<uint32_t>(8 * (wave & 3) + crow) * K2;
  // this lane's operand bytes of a 16-row slab, first and second half of the K-step
  const int frag[2] = {lr * 128 + ((q ^ (lr >> 1)) << 4), lr * 128 + (((4 + q) ^ (lr >> 1)) << 4)};

  for (int item = blockIdx.x; item < R * C; item += gridDim.x) {
    int rt, ct;
    xcd_grouped_tile(item, R, C, rt, ct);
    const int64_t m0 = static_cast<int64_t>(rt) * BM, n0 = static_cast<int64_t>(ct) * BN;
    // rows past M fetch the last row; their results are never stored
    const uint8_t* base = late ? reinterpret_cast<const uint8_t*>(kRope ? w : w + n0 * K)
                               : reinterpret_cast<const uint8_t*>(a + m0 * K);
    const int64_t last = late ? BN - 1 : (M - 1 - m0 < BM - 1 ? M - 1 - m0 : BM - 1);
    const uint32_t lim = late && kRope ? 0xFFFFFFFFu : static_cast<uint32_t>(last) * K2;
    // byte offset of copy u's 8 rows from the first copy's (kRope: weight rows
    // by pair slab; below 2^32, as N K < 2^31)
    uint32_t uoff[kRope ? PM : 1];
    if (kRope) {
#pragma unroll
      for (int u = 0; u < PM; ++u) {
        const int g = (wave & 3) + 4 * u, slab = g >> 1, j = slab % NT;
        const int ps = ct * (BN / 32) + (slab / NT) * (NT / 2) + j % (NT / 2);
        const int row = (ps >> 2) * 128 + (ps & 3) * 16 + (j < NT / 2 ? 0 : 64) + 8 * (g & 1);
        uoff[u] = late ? static_cast<uint32_t>(row - 8 * (wave & 3)) * K2 : static_cast<uint32_t>(32 * u) * K2;
      }
    }
    auto issue = [&](int ks, uint8_t* dst, auto count) {
      constexpr int P = decltype(count)::value;
      const int lds = static_cast<int>(lds_u32(dst)) + (wave & 3) * 1024;
      // past the end the last step is copied again into an idle stage (never read)
      const uint8_t* g = base + static_cast<int64_t>(ks < KS ? ks : KS - 1) * 128;
#pragma unroll
      for (int u = 0; u < P; ++u) {
        const uint32_t o = coff + (kRope ? uoff[kRope ? u : 0] : static_cast<uint32_t>(32 * u) * K2);
        dma16s(g, (o < lim ? o : lim) + cchunk, wave_uniform(lds + u * 4096));
      }
    };
    auto issue_a = [&](int ks) { issue(ks, &sA[ks & (DA - 1)][0], std::integral_constant<int, PA>{}); };
    auto issue_b = [&](int ks, int slot) { issue(ks, &sB[slot][0], std::integral_constant<int, PB>{}); };
    // this wavefront's copies of the next step to be read have landed
    auto landed = [&]() {
      if (late)
        wait_vm<(DB - 2) * PB>();
      else
        wait_vm<(DA - 2) * PA>();
    };

    v4f acc[MT][NT], tot[MT][NT];
    const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) tot[i][j] = zero;
    if (late) {
#pragma unroll
      for (int s = 0; s < DB - 1; ++s) issue_b(s, s);
    } else {
#pragma unroll
      for (int s = 0; s < DA - 1; ++s) issue_a(s);
    }
    if (kPing) {
      landed();
      bar();  // K-step 0 is in LDS
      if (late) bar();
    }
    int ks = 0, cur = 0;
    for (int qq = 0; qq < kLinSplit; ++qq) {
      const int k1 = (qq + 1) * KS / kLinSplit;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = zero;
      for (; ks < k1; ++ks) {
        auto refill = [&]() {  // into the stages of step ks - 1, which every wavefront has read
          if (late)
            issue_b(ks + DB - 1, cur == 0 ? DB - 1 : cur - 1);
          else
            issue_a(ks + DA - 1);
        };
        if (!kPing) {
          landed();
          bar();  // ... and every wavefront's copies; the stages refilled next are read by no one
          refill();
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint8_t* pa = &sA[ks & (DA - 1)][0] + frag[h] + MT * wm * 2048;
          const uint8_t* pb = &sB[cur][0] + frag[h] + NT * wn * 2048;
          bf8 af[MT], bf[NT];
#pragma unroll
          for (int i = 0; i < MT; ++i) af[i] = *reinterpret_cast<const bf8*>(pa + i * 2048);
#pragma unroll
          for (int j = 0; j < NT; ++j) bf[j] = *reinterpret_cast<const bf8*>(pb + j * 2048);
          if (kPing) {
            if (h == 0) refill();
            if (h == 1 && late) landed();
            wait_lds();
            bar();
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
          }
          // weight rows first: a lane's four results are four consecutive columns of one row
#pragma unroll
          for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int i = 0; i < MT; ++i)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j], af[i], acc[i][j], 0, 0, 0);
          if (kPing) {
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            if (h == 1 && !late) landed();
            bar();
          }
        }
        cur = cur + 1 == DB ? 0 : cur + 1;
      }
      // the quarter's sum joins the total in quarter order
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) tot[i][j][r] = tot[i][j][r] + acc[i][j][r];
    }
    if (kPing && !late) bar();
    wait_vm<0>();  // the trailing repeat copies
    bar();         // every wavefront is done with the ring: the next item may refill it
    if (kRope) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int64_t row = m0 + 16 * (MT * wm + i) + lr;
        const int64_t pos = row < M ? ra.rows[row] : -1;
        if (pos < 0 || pos >= ra.N) continue;
        auto place = [&](int j, int& head, int& i0) {
          const int ps = ct * (BN / 32) + wn * (NT / 2) + j;
          head = ps >> 2;
          i0 = (ps & 3) * 16 + 4 * q;
          return rope_dst(ra, head) + pos * 128 + i0;
        };
        bool nan = false;
#pragma unroll
        for (int j = 0; j < NT / 2; ++j) {
          int head, i0;
          uint16_t* dst = place(j, head, i0);
          const v4f x = tot[i][j], y = tot[i][j + NT / 2];
          uint32_t lo[2] = {cvt_pk_bf16(x[0], x[1]), cvt_pk_bf16(x[2], x[3])};
          uint32_t hi[2] = {cvt_pk_bf16(y[0], y[1]), cvt_pk_bf16(y[2], y[3])};
          if (head < 2 * ra.heads) {
            const v4f c = *reinterpret_cast<const v4f*>(ra.cs + pos * 64 + i0);
            const v4f s = *reinterpret_cast<const v4f*>(ra.sn + pos * 64 + i0);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const float x0 = bf16lo(lo[e]), x1 = bf16hi(lo[e]), y0 = bf16lo(hi[e]), y1 = bf16hi(hi[e]);
              const float a0 = x0 * c[2 * e] - y0 * s[2 * e], a1 = x1 * c[2 * e + 1] - y1 * s[2 * e + 1];
              const float b0 = y0 * c[2 * e] + x0 * s[2 * e], b1 = y1 * c[2 * e + 1] + x1 * s[2 * e + 1];
              lo[e] = cvt_pk_bf16(a0, a1);
              hi[e] = cvt_pk_bf16(b0, b1);
              nan |= __builtin_isunordered(a0, a1) || __builtin_isunordered(b0, b1);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 4; e += 2) nan |= __builtin_isunordered(x[e], x[e + 1]) || __builtin_isunordered(y[e], y[e + 1]);
          }
          *reinterpret_cast<uint2*>(dst) = make_uint2(lo[0], lo[1]);
          *reinterpret_cast<uint2*>(dst + 64) = make_uint2(hi[0], hi[1]);
        }
        if (__builtin_expect(nan, 0)) {
          // a NaN is stored as 0x7FC0: this lane's values once more (rare, so not
          // worth the instructions for every value above)
#pragma unroll 1
          for (int j = 0; j < NT / 2; ++j) {
            int head, i0;
            uint2* dst = reinterpret_cast<uint2*>(place(j, head, i0));
            quiet_stored(dst);
            quiet_stored(dst + 16);
          }
        }
      }
      continue;  // the next item
    }
    const int64_t col0 = n0 + 16 * NT * wn + 4 * q;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int64_t row = m0 + 16 * (MT * wm + i) + lr;
      if (row >= M) continue;
      uint16_t* o = out + row * N + col0;
      bool nan = false;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        nan |= __builtin_isunordered(tot[i][j][0], tot[i][j][1]) || __builtin_isunordered(tot[i][j][2], tot[i][j][3]);
        *reinterpret_cast<uint2*>(o + 16 * j) =
            make_uint2(cvt_pk_bf16(tot[i][j][0], tot[i][j][1]), cvt_pk_bf16(tot[i][j][2], tot[i][j][3]));
      }
      if (__builtin_expect(nan, 0)) {  // (as in the RoPE epilogue)
#pragma unroll 1
        for (int j = 0; j < NT; ++j) quiet_stored(reinterpret_cast<uint2*>(o + 16 * j));
      }
    }
    if (out_tap != nullptr) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int64_t row = m0 + 16 * (MT * wm + i) + lr;
        if (row >= M) continue;
#pragma unroll
        for (int j = 0; j < NT; ++j) *reinterpret_cast<v4f*>(out_tap + row * N + col0 + 16 * j) = tot[i][j];
      }
    }
  }
}

// One thread per (row r, Q/K/V part, head, pair i < 64): the pair (i, i + 64)
// of the head's 128 values; Q and K rotated by the angle of the row's position.
__global__ __launch_bounds__(256) void rope_scatter_kernel(const uint16_t* __restrict__ qkv,
                                                           const int32_t* __restrict__ rows, int64_t R,
                                                           const float* __restrict__ cs, const float* __restrict__ sn,
                                                           uint16_t* __restrict__ q, uint16_t* __restrict__ k,
                                                           uint16_t* __restrict__ v, int64_t heads, int64_t N) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t per_row = 3 * heads * 64;
  if (e >= R * per_row) return;
  const int64_t r = e / per_row;
  const int64_t rem = e - r * per_row;
  const int part = static_cast<int>(rem / (heads * 64));
  const int64_t h = (rem / 64) % heads;
  const int i = static_cast<int>(rem & 63);
  const int64_t pos = rows[r];
  if (pos < 0 || pos >= N) return;
  const uint16_t* src = qkv + r * 3 * heads * 128 + (part * heads + h) * 128;
  uint16_t* dst = (part == 0 ? q : (part == 1 ? k : v)) + (h * N + pos) * 128;
  const uint16_t x1 = src[i], x2 = src[64 + i];
  if (part == 2) {
    dst[i] = x1;
    dst[64 + i] = x2;
    return;
  }
  const float a = bf16lo(x1), b = bf16lo(x2), c = cs[pos * 64 + i], s = sn[pos * 64 + i];
  dst[i] = static_cast<uint16_t>(f32_to_bf16(a * c - b * s));
  dst[64 + i] = static_cast<uint16_t>(f32_to_bf16(b * c + a * s));
}

}  // namespace

hipError_t launch_embed_rmsnorm(hipStream_t st, const int32_t* ids, const int32_t* rows, int64_t R,
                                const uint16_t* embed, int64_t vocab, const uint16_t* nw, uint16_t* cache, int64_t N,
                                uint16_t* y, int64_t H, int32_t* dst) {
  const int T = static_cast<int>((H + 511) / 512);
  // up to 1024 rows (4 wavefronts per SIMD): up to four wavefronts per row
  const int wl = R > 1024 ? 0 : (T >= 4 ? 2 : (T >= 2 ? 1 : 0));
  const dim3 grid(static_cast<unsigned>(((R << wl) + 3) / 4)), block(256);
  const int h = static_cast<int>(H);
#define ER(T_) \
  hipLaunchKernelGGL(embed_rmsnorm_kernel<T_>, grid, block, 0, st, ids, rows, R, embed, vocab, nw, cache, N, y, h, wl, dst)
  if (T <= 1) ER(1);
  else if (T <= 2) ER(2);
  else if (T <= 4) ER(4);
  else if (T <= 8) ER(8);
  else if (T <= 16) ER(16);
  else ER(32);
#undef ER
  return hipGetLastError();
}

namespace {

struct LinTile {
  int bm, bn;
};
// The tile of the least time for more than kLinTiledMinM rows: rounds of one
// workgroup per CU of a start and end and K/64 K-steps, and a K-step's time that
// grows with the work in flight. Fitted at 126 sizes, M = 129..4096, N x K = 1536 x
// 512 to 24576 x 8192 and 12288 x 128 to 4096, all tiles in turn in one process: on
// average 0.05 % slower than the best tile, 3.7 % at most (rounds times one cost per
// tile, as fitted at K = 4096 alone, 1.6 % and 37 %: N = 12288, K = 128, M = 1280 30.1
// us on 256 x 192 tiles, 22.0 on 128 x 128). At N = 12288, K = 4096, in us on 128 x
// 128, 128 x 192 and 256 x 192 tiles: M = 256 43, 54, 74; 512 78, 58, 75; 768 110,
// 104, 79; 1000 121, 115, 90.
LinTile lin_tile(int64_t M, int64_t N, int64_t K) {
  struct Tile {
    int bm, bn;
    double start, c0, c1;
  };
  constexpr Tile kTiles[3] = {{128, 128, 3.4, 0.43, 0.12}, {128, 192, 5.1, 0.60, 0.18}, {256, 192, 11.0, 0.75, 0.42}};
  const int64_t cus = device_cu_count();
  const double ks = static_cast<double>(K) / 64.0;
  LinTile pick{128, 128};
  double best = 0.0;
  for (int t = 0; t < 3; ++t) {
    const Tile& s = kTiles[t];
    if (N % s.bn != 0) continue;  // (N is a multiple of 128)
    const int64_t items = ((M + s.bm - 1) / s.bm) * (N / s.bn);
    const double rounds = static_cast<double>((items + cus - 1) / cus);
    const double us = rounds * (s.start + s.c0 * ks) + s.c1 * ks * static_cast<double>(items) / static_cast<double>(cus);
    if (t == 0 || us < best) pick = {s.bm, s.bn}, best = us;
  }
  return pick;
}

// Up to 128 rows: three weight slabs per workgroup when that still gives a
// workgroup per CU (few rows), else one.
bool lin_wide(int64_t M, int64_t N) { return M <= 32 && N % 48 == 0 && N / 48 >= 256; }

template <bool kRope>
hipError_t launch_linear(hipStream_t st, const uint16_t* a, const uint16_t* w, uint16_t* out, float* out_tap, int64_t M,
                         int64_t N, int64_t K, const RopeArgs& ra) {
  if (M > kLinTiledMinM) {
    const LinTile tile = lin_tile(M, N, K);
    const int64_t cus = device_cu_count();
#define LT(BM_, BN_, PING_)                                                                                       \
  do {                                                                                                           \
    const int r_ = static_cast<int>((M + BM_ - 1) / BM_), c_ = static_cast<int>(N / BN_);                        \
    hipLaunchKernelGGL((linear_bf16_tiled_kernel<BM_, BN_, PING_, kRope>),                                              \
                       dim3(static_cast<unsigned>(static_cast<int64_t>(r_) * c_ < cus ? r_ * c_ : cus)),         \
                       dim3(kLtWaves * 64), 0, st, a, w, out, out_tap, M, N, K, r_, c_, ra);                         \
  } while (0)
    if (tile.bm == 256)
      LT(256, 192, true);
    else if (tile.bn == 192)
      LT(128, 192, false);
    else
      LT(128, 128, false);
#undef LT
    return hipGetLastError();
  }
  // up to 64 rows per pass; the last pass may hold fewer slabs
  const unsigned passes = static_cast<unsigned>((M + 63) / 64);
  const int mt = static_cast<int>(M >= 64 ? 4 : (M + 15) / 16);
  const bool wide = lin_wide(M, N);
  const dim3 grid(static_cast<unsigned>(N / (wide ? 48 : 16)), passes), block(kLinSplit * 64);
#define LB(MT_, NJ_) hipLaunchKernelGGL((linear_bf16_kernel<MT_, NJ_, kRope>), grid, block, 0, st, a, w, out, out_tap, M, N, K, ra)
  if (wide) {
    if (mt <= 1) LB(1, 3);
    else LB(2, 3);
  } else if (mt <= 1) LB(1, 1);
  else if (mt == 2) LB(2, 1);
  else if (mt == 3) LB(3, 1);
  else LB(4, 1);
#undef LB
  return hipGetLastError();
}

}  // namespace

void linear_tile(int64_t M, int64_t N, int64_t K, int (&tile)[2]) {
  if (M > kLinTiledMinM) {
    const LinTile t = lin_tile(M, N, K);
    tile[0] = t.bm, tile[1] = t.bn;
  } else {
    tile[0] = 64, tile[1] = lin_wide(M, N) ? 48 : 16;
  }
}

hipError_t launch_linear_bf16(hipStream_t st, const uint16_t* a, const uint16_t* w, uint16_t* out, float* out_tap,
                              int64_t M, int64_t N, int64_t K) {
  return launch_linear<false>(st, a, w, out, out_tap, M, N, K, RopeArgs{});
}

hipError_t launch_linear_rope(hipStream_t st, const uint16_t* y, const uint16_t* w_qkv, const int32_t* rows, int64_t R,
                              const float* cs, const float* sn, uint16_t* q, uint16_t* k, uint16_t* v, int64_t heads,
                              int64_t N, int64_t H) {
  return launch_linear<true>(st, y, w_qkv, nullptr, nullptr, R, 3 * heads * 128, H,
                             RopeArgs{rows, cs, sn, q, k, v, static_cast<int>(heads), N});
}

hipError_t launch_rope_scatter(hipStream_t st, const uint16_t* qkv, const int32_t* rows, int64_t R, const float* cs,
                               const float* sn, uint16_t* q, uint16_t* k, uint16_t* v, int64_t heads, int64_t N) {
  const int64_t threads = R * 3 * heads * 64;
  hipLaunchKernelGGL(rope_scatter_kernel, dim3(static_cast<unsigned>((threads + 255) / 256)), dim3(256), 0, st, qkv,
                     rows, R, cs, sn, q, k, v, heads, N);
  return hipGetLastError();
}

}  // namespace lacache
