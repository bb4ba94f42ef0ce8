// Tiled FP8 MFMA GEMMs with per-group dequantization (Sec. 3.4):
//   gate/up: x[M x H] . Wgu[2I x H]^T, fused SwiGLU and 1x128 re-quantization
//   down:    h[M x I] . Wd[H x I]^T -> bf16
//
// Work items are BM-row x BNR-weight-row output tiles (BM 64 to 256 by the
// rules at the launchers; BNR 256, or 128 for the down GEMM's smaller tiles),
// times the K splits of the down GEMM. The grid is persistent: one workgroup
// per CU walks the items b, b + G, b + 2G, ... (G workgroups), and its copy
// ring runs straight across item boundaries, so the first K-groups of the next tile are already in LDS
// when a tile's epilogue ends and no workgroup launch or pipeline refill
// separates two tiles.
//
// A workgroup has 8 multiplying wavefronts (four of them also copy, or up to
// 128-row tiles four more only copy); wavefront (wm, wn) owns WR activation rows x
// WC weight rows (MT x NJ sub-tiles of 16 x 16). K is walked one 128-wide group
// at a time:
//   * the group's fp8 tiles (A: BM x 128 B, B: BNR x 128 B), the BM
//     activation scales and the tile's two weight-block scales go global ->
//     LDS with direct-to-LDS copies into a ring of stages, issued S - 1 groups
//     ahead, so no registers hold staging data;
//   * every 16x16 sub-tile gets one 16x16x128 FP8 MFMA (exactly one K-group)
//     whose fp32 result is added to the accumulator times
//     RN32(x_scale[row] * w_scale[block]): four VALU FMAs per MFMA, issued two
//     MFMAs later so that they find the result finished while the matrix core
//     works on the next ones.
// The MFMA takes the weight rows as its first operand, so a lane's four
// results are four consecutive output columns of one activation row: the
// epilogues pack e4m3 codes and bf16 values within a lane, and a row's max
// over the columns needs only two cross-lane steps.
//
// For gate/up the tile's 256 weight rows are the 128 gate rows and the 128
// matching up rows of one h-group; a wavefront's slabs are WC/2 gate rows and
// the WC/2 matching up rows, so SwiGLU pairs values held by one lane, and the
// row amax over the 128-wide h-group meets in LDS across the wavefronts of a
// row band. h never reaches memory.
#include <atomic>
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace lacache {
namespace {

__device__ __forceinline__ int lds_off(int row, int chunk) { return row * 128 + ((chunk ^ swz(row)) << 4); }

// MFMA operand for one 16-row slab: lane (q = l/16, r = l%16) takes row
// base + r, logical chunks q and 4 + q (the same K placement for A and B).
__device__ __forceinline__ v8i load_frag(const uint8_t* tile, int row, int q) {
  return cat_frag(*reinterpret_cast<const u4v*>(tile + lds_off(row, q)),
                  *reinterpret_cast<const u4v*>(tile + lds_off(row, 4 + q)));
}

// One LDS stage: A tile, B tile, BM activation scales, the two weight-block
// scales of the K-group (slots XR and XR + 1 of a 64-slot region written by
// one copy instruction), and 64 spare slots for duplicate scale copies.
template <int BM, int BNR>
struct Stage {
  static constexpr int XR = (BM + 63) / 64 * 64;  // activation scale slots (64 per copy instruction)
  uint8_t a[BM * 128];
  uint8_t b[BNR * 128];
  alignas(16) float xs[XR + 128];
};

// A work item: output tile (row tile, column tile) and its K range.
struct Item {
  int m0;   // first activation row
  int col;  // gate/up: h-group; down: 256-column tile
  int kb0, kb1;
  int split;
};

// Item w of R x C tiles x KS splits (R C KS < 2^31). The splits count as
// extra row tiles (split-major), so the XCD-grouped order keeps items that share
// an operand (the same K range of the same rows or columns) on one XCD.
__device__ __forceinline__ Item item_at(int w, int R, int C, int KS, int KB, int BM) {
  int vr, col;
  xcd_grouped_tile(w, R * KS, C, vr, col);
  Item it;
  it.col = col;
  it.split = vr / R;
  it.m0 = (vr - it.split * R) * BM;
  it.kb0 = it.split * KB / KS;
  it.kb1 = (it.split + 1) * KB / KS;
  return it;
}

}  // namespace

constexpr int kTileWaves = 8;  // wavefronts that multiply
constexpr int kCopyWaves = 4;  // wavefronts that copy (one per SIMD)
// Up to 128-row tiles the copies have wavefronts of their own (12 in all, at
// most 168 VGPRs each), so no multiplying wavefront waits for the memory
// pipeline to take its copies (H = 4096, I = 12288: down at 128 rows 20.9 ->
// 18.8 us, gate/up at 192 rows 32.9 -> 31.8); taller tiles need the registers.
constexpr bool tile_dedicated(int bm) { return bm <= 128; }
constexpr int tile_threads(int bm) { return (kTileWaves + (tile_dedicated(bm) ? kCopyWaves : 0)) * 64; }

template <bool kGateUp, int BM, int BNR>
__global__ __launch_bounds__(tile_threads(BM)) void gemm_tiled_kernel(
    const uint8_t* __restrict__ aq, const float* __restrict__ as,  // [M x K] codes, [K/128 x M] scales
    const uint8_t* __restrict__ bq, const float* __restrict__ bs,  // [N x K] codes, [N/128 x K/128] scales
    uint8_t* __restrict__ hq, float* __restrict__ hs, float* __restrict__ h_tap,
    uint16_t* __restrict__ out, float* __restrict__ out_tap, float* __restrict__ part,
    const float* __restrict__ col_s, int64_t M, int64_t K, int64_t N, int64_t I, int KS, int W) {
  constexpr bool kDed = tile_dedicated(BM);
  constexpr int NCW = BM > 128 ? 2 : 4;       // wavefronts along the weight rows
  constexpr int WC = BNR / NCW;               // weight rows (output columns) per wavefront
  constexpr int WR = BM * NCW / kTileWaves;   // activation rows per wavefront
  constexpr int MT = WR / 16, NJ = WC / 16;   // its 16 x 16 sub-tiles
  static_assert(MT * 16 * kTileWaves == BM * NCW && NJ * 16 * NCW == BNR && (!kGateUp || BNR == 256), "tile shape");
  using Stg = Stage<BM, BNR>;
  constexpr int XR = Stg::XR;
  // LDS ring: as many stages as fit (2 at BM = 256, 3 at BM = 64..128 x 256, 6 at 64 x 128)
  constexpr int kRoom = 163840 - NCW * BM * 4;
  constexpr int S = kRoom / static_cast<int>(sizeof(Stg)) > 6 ? 6 : kRoom / static_cast<int>(sizeof(Stg));
  __shared__ Stg stg[S];
  __shared__ float sRed[NCW][BM];

  const int t = threadIdx.x, lane = t & 63;
  // wavefront index made visibly uniform: LDS bases and item fields go scalar
  const int wave = wave_uniform(t >> 6);
  const int wm = wave / NCW, wn = wave % NCW;
  const int q = lane >> 4, lr = lane & 15;
  const int KB = static_cast<int>(K / 128);
  const int R = static_cast<int>((M + BM - 1) / BM);
  const int C = static_cast<int>(kGateUp ? I / 128 : (N + BNR - 1) / BNR);
  const int G = static_cast<int>(gridDim.x);
  const int cw = kDed ? wave - kTileWaves : wave;  // copy wavefront index

  // The copy wavefronts and the others run the same stream as two instances
  // of one loop: only the copy wavefronts' instance holds the copy cursor
  // (item, K-group, per-lane offsets) and issues the copies, so the other
  // wavefronts spend neither instructions nor registers on it.
  auto run = [&](auto copy_tag) {
    constexpr bool kCopy = decltype(copy_tag)::value;
    // ---- direct-to-LDS copy plan. Only the first kCopyWaves wavefronts (one
    // per SIMD) copy: a wavefront stalls while the memory pipeline takes its
    // copy instructions, and the other wavefront of its SIMD keeps the matrix
    // core busy meanwhile (all eight copying at once left it idle). A copy
    // instruction fills 64 consecutive 16-byte LDS slots (8 tile rows); lane l
    // fills slot l, i.e. row 8g + l/8, physical chunk l%8, so it fetches logical
    // chunk (l%8) ^ swz(row) of that row. Rows past M (or N) fetch a clamped
    // row; their results are never stored. Scales: each copy wavefront copies
    // the activation scales of rows 64 (w mod XR/64) .. + 63 (one float per
    // lane; copies beyond the first go to the spare slots) and the two
    // weight-block scales (lane 0 the first block, the others the second).
    constexpr int kAInst = BM / 8 / kCopyWaves;  // per copy wavefront
    constexpr int kBInst = BNR / 8 / kCopyWaves;
    constexpr int kPer = kAInst + kBInst + 2;  // copies per copy wavefront per K-group
    const int xband = cw % (XR / 64);
    const int xs_dst = cw < XR / 64 ? cw * 64 : XR + 64;

    // issue cursor: the item whose K-groups are being copied
    int iw = blockIdx.x, ikb = 0, ikb1 = 0;
    const uint8_t* a_base = aq;
    const uint8_t* b_base = bq;
    const uint8_t* b_base_hi = bq;
    const float* x_base = as;  // activation scales of the tile's rows (wave-uniform)
    uint32_t x_off = 0;        // ... this lane's byte offset (stride M floats per K-group)
    uint32_t w_off = 0;        // this lane's weight-block scale row, as a byte offset into bs
    uint32_t a_off[kCopy ? kAInst : 1], b_off[kCopy ? kBInst : 1];
    auto enter = [&](int w) {
      const Item it = item_at(w, R, C, KS, KB, BM);
      ikb = it.kb0;
      ikb1 = it.kb1;
      a_base = aq + static_cast<int64_t>(it.m0) * K;
      const int alim = static_cast<int>(M) - 1 - it.m0;  // last valid row of the tile
#pragma unroll
      for (int u = 0; u < (kCopy ? kAInst : 0); ++u) {
        const int row = (cw * kAInst + u) * 8 + (lane >> 3);
        const int r = row < alim ? row : alim;
        a_off[u] = static_cast<uint32_t>(r) * static_cast<uint32_t>(K) + ((lane & 7) ^ swz(row)) * 16;
      }
      // gate/up: tile rows 0..127 come from the gate block, 128..255 from the up
      // block (base b_base_hi); down: one contiguous 256-row block
      const int n0 = kGateUp ? 0 : it.col * BNR;
      const int blim = kGateUp ? BNR : static_cast<int>(N) - 1 - n0;
      b_base = kGateUp ? bq + static_cast<int64_t>(it.col) * 128 * K : bq + static_cast<int64_t>(n0) * K;
      b_base_hi = kGateUp ? bq + (I + static_cast<int64_t>(it.col) * 128 - 128) * K : b_base;
      // (weights in the tile layout of wtile_off: the slab bases above are the
      // same as row-major, the offsets within and the K-group step are not)
#pragma unroll
      for (int u = 0; u < (kCopy ? kBInst : 0); ++u) {
        const int row = (cw * kBInst + u) * 8 + (lane >> 3);
        const int r = row < blim ? row : blim;
        b_off[u] = static_cast<uint32_t>(wtile_off(r, ((lane & 7) ^ swz(row)) * 16, K));
      }
      {
        const int row = xband * 64 + lane;
        x_base = as + it.m0;
        x_off = static_cast<uint32_t>(row < alim ? row : alim) * 4u;
        // gate/up: {gate block, up block}; down: {block of columns n0.., the next
        // one (or the same past N)}
        const int r0 = kGateUp ? it.col : n0 / 128;
        const int r1 = kGateUp ? static_cast<int>(I / 128) + it.col : (n0 + 128 < N ? n0 / 128 + 1 : r0);
        w_off = static_cast<uint32_t>((lane == 0 ? r0 : r1) * KB) * 4u;
      }
    };
    // Copies of K-group kb of the cursor's item into stage dst (asynchronous).
    auto issue_group = [&](int kb, Stg* dst) {
      const int64_t ko = static_cast<int64_t>(kb) * 128;
      const int la = static_cast<int>(lds_u32(dst->a)), lb = static_cast<int>(lds_u32(dst->b));
#pragma unroll
      for (int u = 0; u < (kCopy ? kAInst : 0); ++u) dma16s(a_base + ko, a_off[u], wave_uniform(la + (cw * kAInst + u) * 1024));
#pragma unroll
      for (int u = 0; u < (kCopy ? kBInst : 0); ++u) {
        const uint8_t* base = (kGateUp && (cw * kBInst + u) * 8 >= 128) ? b_base_hi : b_base;
        dma16s(base + ko * 16, b_off[u], wave_uniform(lb + (cw * kBInst + u) * 1024));
      }
      const int lx = static_cast<int>(lds_u32(dst->xs));
      dma4s(x_base + static_cast<int64_t>(kb) * M, x_off, wave_uniform(lx + xs_dst * 4));
      dma4s(bs + kb, w_off, wave_uniform(lx + XR * 4));
    };
    // The next K-group in the workgroup's sequence. Past the last one the last
    // group is copied again into the idle stage (never read), so every step
    // waits for the same count.
    auto issue_next = [&](Stg* dst) {
      issue_group(ikb < ikb1 ? ikb : ikb1 - 1, dst);
      if (ikb < ikb1 && ++ikb == ikb1 && iw + G < W) {
        iw += G;
        enter(iw);
      }
    };

    float acc[MT][NJ][4];

    // Multiplies the K-group in stage cur into acc.
    auto compute = [&](const Stg* cur) {
      auto brow = [&](int j) {
        return kGateUp ? (j < NJ / 2 ? (WC / 2) * wn + 16 * j : 128 + (WC / 2) * wn + 16 * (j - NJ / 2)) : WC * wn + 16 * j;
      };
      // Every LDS read the first MFMAs and FMAs need is issued up front, in the
      // order they are needed (LDS reads complete in order): the first B slab,
      // the scales, then the four A slabs. MFMA i waits only for its own
      // operands, and the scale products are formed after MFMA 1, when the
      // first FMAs need them, instead of holding MFMA 0 back by a round trip.
      v8i bb[2];
      bb[0] = load_frag(cur->b, brow(0) + lr, q);
      __builtin_amdgcn_sched_barrier(0);
      float xv[MT];
#pragma unroll
      for (int i = 0; i < MT; ++i) xv[i] = cur->xs[WR * wm + 16 * i + lr];
      // gate/up: slabs 0..NJ/2-1 are gate rows (block scale in slot XR), the
      // rest the matching up rows (slot XR + 1); down: the wave's columns lie in
      // one block, slot XR + (WC wn) / 128
      const float w0 = cur->xs[XR + (kGateUp ? 0 : (WC * wn) / 128)];
      const float w1 = cur->xs[XR + 1];
      __builtin_amdgcn_sched_barrier(0);
      v8i af[MT];
#pragma unroll
      for (int i = 0; i < MT; ++i) af[i] = load_frag(cur->a, WR * wm + 16 * i + lr, q);
      __builtin_amdgcn_sched_barrier(0);
      float sc[kGateUp ? 2 : 1][MT];  // RN32(x_scale * w_scale) of this lane's row
      // Software pipeline over the MT NJ sub-tiles s = MT j + i: MFMA s, then the
      // scale FMAs of MFMA s - 2; the B operand of slab j + 1 is read while slab
      // j multiplies.
      v4f pr[3];
#pragma unroll
      for (int s = 0; s < MT * NJ; ++s) {
        const int j = s / MT, i = s % MT;
        if (i == 0 && j < NJ - 1) bb[(j + 1) & 1] = load_frag(cur->b, brow(j + 1) + lr, q);
        const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
        pr[s % 3] = mfma_fp8_16x16x128(bb[j & 1], af[i], zero);
        // keep MFMA s ahead of the FMAs below: they read a result two MFMAs
        // old, so they neither wait for the matrix core nor delay the next MFMA
        __builtin_amdgcn_sched_barrier(0);
        if (s == 1) {
#pragma unroll
          for (int i2 = 0; i2 < MT; ++i2) {
            sc[0][i2] = xv[i2] * w0;
            if (kGateUp) sc[kGateUp ? 1 : 0][i2] = xv[i2] * w1;
          }
        }
        if (s >= 2) {
          const int ps = s - 2, pj = ps / MT, pi = ps % MT;
          const int blk = (kGateUp && pj >= NJ / 2) ? 1 : 0;
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[pi][pj][r] = __builtin_fmaf(pr[ps % 3][r], sc[blk][pi], acc[pi][pj][r]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int ps = MT * NJ - 2; ps < MT * NJ; ++ps)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc[ps % MT][ps / MT][r] =
              __builtin_fmaf(pr[ps % 3][r], sc[kGateUp ? 1 : 0][ps % MT], acc[ps % MT][ps / MT][r]);
    };

    // ---- the stream: S - 1 K-groups ahead of the multiply, across items
    if (kCopy) {
      enter(iw);
#pragma unroll
      for (int s = 0; s < S - 1; ++s) issue_next(&stg[s]);
    }
    int cur = 0;  // stage of the K-group being multiplied

    for (int w = blockIdx.x; w < W; w += G) {
      const Item it = item_at(w, R, C, KS, KB, BM);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

      for (int kb = it.kb0; kb < it.kb1; ++kb) {
        // a copy wave's copies of the group have landed (later ones may still
        // fly; loads retire in issue order, so epilogue stores in between only
        // make the wait longer) ...
        if (kCopy)
          wait_vm_lds<(S - 2) * kPer>();
        else
          wait_lds();
        bar();  // ... and every wave's; and the stage of the previous group is read by no one
        if (kCopy) issue_next(&stg[cur == 0 ? S - 1 : cur - 1]);  // into the stage freed by the previous group
        if (!kDed || !kCopy) compute(&stg[cur]);
        cur = cur + 1 == S ? 0 : cur + 1;
      }
      if (kDed && kCopy) {
        if (kGateUp) bar();  // the epilogue's
        continue;
      }

      if (col_s != nullptr) {
        // per-channel weight scales: output column n times col_s[n]
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int64_t n = kGateUp ? (j < NJ / 2 ? 0 : I) + static_cast<int64_t>(it.col) * 128 + (WC / 2) * wn +
                                          16 * (j < NJ / 2 ? j : j - NJ / 2) + 4 * q
                                    : static_cast<int64_t>(it.col) * BNR + WC * wn + 16 * j + 4 * q;
          const float4 cs = (kGateUp || n < N) ? *reinterpret_cast<const float4*>(col_s + n) : make_float4(0, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < MT; ++i) {
            acc[i][j][0] *= cs.x;
            acc[i][j][1] *= cs.y;
            acc[i][j][2] *= cs.z;
            acc[i][j][3] *= cs.w;
          }
        }
      }
      if (kGateUp) {
        // ---- SwiGLU: h = SiLU(g) * u; lanes hold matching gate (j) and up
        // (j + NJ/2) values; h replaces g in acc
        float am[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          float a = 0.0f;
#pragma unroll
          for (int j = 0; j < NJ / 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float v = swiglu_fast(acc[i][j][r], acc[i][j + NJ / 2][r]);
              acc[i][j][r] = v;
              a = __builtin_fmaxf(a, __builtin_fabsf(v));
            }
          // over the four lanes that hold the row's other columns
          a = __builtin_fmaxf(a, __shfl_xor(a, 16, 64));
          a = __builtin_fmaxf(a, __shfl_xor(a, 32, 64));
          am[i] = a;
        }
        if (q == 0) {
#pragma unroll
          for (int i = 0; i < MT; ++i) sRed[wn][WR * wm + 16 * i + lr] = am[i];
        }
        wait_lds();
        bar();  // the row amax of every wavefront of the band is in LDS
        // ---- 1x128 quantization of each row's h-group (without hq: h only)
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          if (hq == nullptr) {
            const int64_t grow = static_cast<int64_t>(it.m0) + WR * wm + 16 * i + lr;
            if (grow < M) {
#pragma unroll
              for (int j = 0; j < NJ / 2; ++j)
                *reinterpret_cast<float4*>(h_tap + grow * I + static_cast<int64_t>(it.col) * 128 + (WC / 2) * wn +
                                           16 * j + 4 * q) =
                    make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            }
            continue;
          }
          const int row = WR * wm + 16 * i + lr;
          const int64_t grow = static_cast<int64_t>(it.m0) + row;
          float amax = sRed[0][row];
#pragma unroll
          for (int c = 1; c < NCW; ++c) amax = __builtin_fmaxf(amax, sRed[c][row]);
          const float s = amax / kE4M3Max;
          const FastQuant fq = fast_quant(s);
          const bool fast = scale_is_fast(s);
          const bool ok = grow < M;
#pragma unroll
          for (int j = 0; j < NJ / 2; ++j) {
            // E(RN32(h / s)) by the bracket where it decides, else by the division
            uint32_t code;
            const bool agree = enc4_bracket(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3], fq, code);
            if (s == 0.0f)
              code = 0u;
            else if (!(fast && agree))
              code = enc4_e4m3(qdiv(acc[i][j][0], s), qdiv(acc[i][j][1], s), qdiv(acc[i][j][2], s),
                               qdiv(acc[i][j][3], s));
            const int64_t col = static_cast<int64_t>(it.col) * 128 + (WC / 2) * wn + 16 * j + 4 * q;
            if (ok) {
              *reinterpret_cast<uint32_t*>(hq + grow * I + col) = code;
              if (h_tap != nullptr)
                *reinterpret_cast<float4*>(h_tap + grow * I + col) =
                    make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            }
          }
          if (wn == 0 && q == 0 && ok) hs[it.col * M + grow] = s;
        }
      } else {
        // ---- bf16 output (nearest-even from the fp32 accumulator), or the fp32
        // partial sum of this K split
        const int64_t n0 = static_cast<int64_t>(it.col) * BNR;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          const int64_t row = static_cast<int64_t>(it.m0) + WR * wm + 16 * i + lr;
          if (row >= M) continue;
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            const int64_t col = n0 + WC * wn + 16 * j + 4 * q;
            if (col >= N) continue;
            if (KS > 1) {
              *reinterpret_cast<float4*>(part + (it.split * M + row) * N + col) =
                  make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            } else {
              *reinterpret_cast<uint2*>(out + row * N + col) =
                  make_uint2(pack_bf16x2(acc[i][j][0], acc[i][j][1]), pack_bf16x2(acc[i][j][2], acc[i][j][3]));
              if (out_tap != nullptr)
                *reinterpret_cast<float4*>(out_tap + row * N + col) =
                    make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            }
          }
        }
      }
    }
    if (kCopy) wait_vm<0>();  // the trailing repeat copies
  };
  if (kDed ? wave >= kTileWaves : wave < kCopyWaves)
    run(std::true_type{});
  else
    run(std::false_type{});
}

// Compute units of the current device (the persistent grid's size), cached
// per device; 256 when the runtime cannot tell.
int device_cu_count() {
  static std::atomic<int> cached[64];  // 0: not looked up yet (zero-initialized)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

namespace {

// out = RNE_bf16(sum of the KS partials, in split order); 4 columns per thread.
__global__ __launch_bounds__(256) void split_reduce_kernel(const float* __restrict__ part, uint16_t* __restrict__ out,
                                                           float* __restrict__ out_tap, int64_t MN, int KS) {
  const int64_t e = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 4;
  if (e >= MN) return;
  float4 acc = *reinterpret_cast<const float4*>(part + e);
  for (int sp = 1; sp < KS; ++sp) {
    const float4 p = *reinterpret_cast<const float4*>(part + sp * MN + e);
    acc.x += p.x; acc.y += p.y; acc.z += p.z; acc.w += p.w;
  }
  *reinterpret_cast<uint2*>(out + e) = make_uint2(pack_bf16x2(acc.x, acc.y), pack_bf16x2(acc.z, acc.w));
  if (out_tap != nullptr) *reinterpret_cast<float4*>(out_tap + e) = acc;
}

template <bool kGateUp, int BM, int BNR>
hipError_t launch_tiled(hipStream_t st, const uint8_t* aq, const float* as, const uint8_t* bq, const float* bs,
                        uint8_t* hq, float* hs, float* h_tap, uint16_t* out, float* out_tap, float* part, int64_t M,
                        int64_t K, int64_t N, int64_t I, int KS, const float* col_s) {
  const int64_t ny = kGateUp ? I / 128 : (N + BNR - 1) / BNR;
  const int W = static_cast<int>(((M + BM - 1) / BM) * ny * KS);  // work items (< 2^31 by the size limits)
  // one workgroup per CU (the LDS ring allows no more)
  const int G = W < device_cu_count() ? W : device_cu_count();
  hipLaunchKernelGGL((gemm_tiled_kernel<kGateUp, BM, BNR>), dim3(static_cast<unsigned>(G)), dim3(tile_threads(BM)), 0,
                     st, aq, as, bq, bs, hq, hs, h_tap, out, out_tap, part, col_s, M, K, N, I, KS, W);
  return hipGetLastError();
}

// The split-K partials the workspace has room for: at 128 x 256 tiles as many
// splits as fit in one round of one workgroup per CU, each at least 16
// K-groups long (1 where 256-row tiles need fewer rounds).
int down_splits(int64_t M, int64_t H, int64_t I) {
  const int64_t ct = (H + 255) / 256, cus = device_cu_count(), tiles = ((M + 127) / 128) * ct;
  const int64_t r256 = (((M + 255) / 256) * ct + cus - 1) / cus, r128 = (tiles + cus - 1) / cus;
  if (r128 > r256 || tiles >= cus) return 1;
  int64_t ks = cus / tiles;
  const int64_t max_ks = (I / 128) / 16;
  if (ks > max_ks) ks = max_ks;
  return ks < 1 ? 1 : static_cast<int>(ks);
}

// Time of the K loops of a launch of `items` work items of n K-groups each, in
// us: rounds of one workgroup per CU, and a K-group's time c0 + c1 f on a
// device with a fraction f of its workgroup slots in use (the clock falls and
// the memory fills as more CUs work).
double loops_us(int64_t items, int64_t n, double c0, double c1) {
  const int64_t cus = device_cu_count(), rounds = (items + cus - 1) / cus;
  return static_cast<double>(rounds * n) * (c0 + c1 * static_cast<double>(items) / static_cast<double>(rounds * cus));
}

}  // namespace

size_t tiled_down_ws_bytes(int64_t M, int64_t H, int64_t I) {
  const int ks = down_splits(M, H, I);
  return ks > 1 ? static_cast<size_t>(ks) * static_cast<size_t>(M) * static_cast<size_t>(H) * 4 : 0;
}

namespace {

int gateup_height(int64_t M, int64_t H, int64_t I) {
  // Row-tile height: the least loop time. Every height gives the same bytes (an
  // element's K-groups are added in the same order). K-group times fitted to
  // sweeps at H = 512..8192, I = 6144..24576 and M = 65..2048; at H = 4096, I =
  // 12288 the kernel takes, at the height chosen and at the better of 128 and
  // 256 rows: M = 128 29 and 35 us (64 rows), 192 32 and 36 (96), 333 46 and 52
  // (192), 700 87 and 98 (192), 1536 138 and 160 (192).
  constexpr int kHeights[5] = {256, 192, 128, 96, 64};
  constexpr double kGroup[5][2] = {{1.1, 0.73}, {0.92, 0.55}, {0.72, 0.36}, {0.57, 0.33}, {0.43, 0.34}};
  int pick = 0;
  double best = 0.0;
  for (int t = 0; t < 5; ++t) {
    const double us = loops_us(((M + kHeights[t] - 1) / kHeights[t]) * (I / 128), H / 128, kGroup[t][0], kGroup[t][1]);
    if (t == 0 || us < best) pick = t, best = us;
  }
  return kHeights[pick];
}

}  // namespace

hipError_t launch_gateup_tiled(hipStream_t st, const uint8_t* xq, const float* xs, const uint8_t* wq,
                               const float* ws, uint8_t* hq, float* hs, float* h_tap, int64_t M, int64_t H,
                               int64_t I, const float* col_s) {
#define GU(BM_)                                                                                                    \
  return launch_tiled<true, BM_, 256>(st, xq, xs, wq, ws, hq, hs, h_tap, nullptr, nullptr, nullptr, M, H, 2 * I, I, 1, \
                                      col_s)
  switch (gateup_height(M, H, I)) {
    case 64: GU(64);
    case 96: GU(96);
    case 128: GU(128);
    case 192: GU(192);
    default: GU(256);
  }
#undef GU
}

namespace {

struct DownPlan {
  int shape;  // of kDownShapes
  int ks;     // K splits
  bool regs;  // 64 x 128 tiles by the kernel with the weights in registers
};
struct DownShape {
  int bm, bn;
  double start, c0, c1;
};
constexpr DownShape kDownShapes[4] = {
    {256, 256, 9.5, 0.85, 0.0}, {128, 256, 6.3, 0.55, 0.02}, {128, 128, 5.8, 0.32, 0.08}, {64, 128, 6.3, 0.26, 0.0}};
constexpr DownShape kDownRegs = {64, 128, 3.8, 0.24, 0.04};

// Tile shape and K splits (up to the partials the workspace holds): the least of
// start-up + loops + the partials' reduction (a launch, and writing and reading
// them). 64-row tiles take their weights into registers wherever that kernel fits
// one round (at M = 65..1024 and every split it was up to 4 us faster of the whole
// FFN, nowhere slower beyond noise). The constants are fitted to the whole FFN call at 188 sizes, M =
// 65..8192, H = 128..16384, I = 1024..16384, all shapes and splits in turn in one
// process; the chosen one is on average 0.13 % slower than the best, 4.8 % at most.
// 128 x 256 tiles over the workspace's splits stay unless another choice is more
// than 1 us less, about the fit's error: at H = 4096, I = 12288 the whole FFN
// takes, in us, with them, with the best other shape and split, and as chosen:
// M = 128 65.2, 59.6, 60.4; 256 73.6, 71.0, 71.0; 400 96.2, 96.5, 96.2; 512 98.8,
// 100.8, 98.8; at H = 3072, I = 8192, M = 400 59.3, 55.6, 55.6 (64 x 128 tiles
// without a split; 60.9 where the rule took them with three).
DownPlan down_plan(int64_t M, int64_t H, int64_t I, bool col_scales) {
  const int ks_max = down_splits(M, H, I);
  constexpr double kMargin = 1.0;
  DownPlan pick{1, ks_max, false};
  double best = 0.0;
  auto us = [&](int t, int k, bool regs) {
    const DownShape& s = regs ? kDownRegs : kDownShapes[t];
    const int64_t tiles = ((M + s.bm - 1) / s.bm) * ((H + s.bn - 1) / s.bn);
    return s.start + loops_us(tiles * k, (I / 128 + k - 1) / k, s.c0, s.c1) +
           (k > 1 ? 0.8 + (4.0 * k + 2.0) * static_cast<double>(M * H) / 3.5e6 : 0.0);
  };
  best = us(1, ks_max, false) - kMargin;
  for (int t = 0; t < 4; ++t)
    for (int k = 1; k <= (t == 0 ? 1 : ks_max); ++k) {
      if (t == 1 && k == ks_max) continue;
      const bool regs = t == 3 && !col_scales && down_rows64_ok(M, H, I, k);
      const double e = us(t, k, regs);
      if (e < best) pick = {t, k, regs}, best = e;
    }
  return pick;
}

}  // namespace

void tiled_plan(int64_t M, int64_t H, int64_t I, bool col_scales, int (&plan)[5]) {
  const DownPlan d = down_plan(M, H, I, col_scales);
  plan[0] = gateup_height(M, H, I);
  plan[1] = kDownShapes[d.shape].bm;
  plan[2] = kDownShapes[d.shape].bn;
  plan[3] = d.ks;
  plan[4] = d.regs ? 1 : 0;
}

hipError_t launch_down_tiled(hipStream_t st, const uint8_t* hq, const float* hs, const uint8_t* wq, const float* ws,
                             uint16_t* out, float* out_tap, int64_t M, int64_t H, int64_t I, void* ws_buf,
                             const float* col_s) {
  const DownPlan plan = down_plan(M, H, I, col_s != nullptr);
  const int ks = plan.ks;
  float* part = static_cast<float*>(ws_buf);
  hipError_t e = hipSuccess;
#define DN(BM_, BN_)                                                                                              \
  e = launch_tiled<false, BM_, BN_>(st, hq, hs, wq, ws, nullptr, nullptr, nullptr, out, out_tap, part, M, I, H, I, ks, \
                                    col_s)
  switch (plan.shape) {
    case 0: DN(256, 256); break;
    case 1: DN(128, 256); break;
    case 2: DN(128, 128); break;
    default:
      if (plan.regs)
        e = launch_down_rows64(st, hq, hs, wq, ws, out, out_tap, part, M, H, I, ks);
      else
        DN(64, 128);
      break;
  }
#undef DN
  if (e != hipSuccess || ks == 1) return e;
  const int64_t mn = M * H;
  hipLaunchKernelGGL(split_reduce_kernel, dim3(static_cast<unsigned>((mn / 4 + 255) / 256)), dim3(256), 0, st, part,
                     out, out_tap, mn, ks);
  return hipGetLastError();
}

}  // namespace lacache
