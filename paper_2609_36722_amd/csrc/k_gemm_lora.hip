// K2: bf16 MFMA projection GEMM with the rank-r LoRA update fused into its
// epilogue (query-side adaptation, section 4 eq. 4):
//   out[i][n] = x[i] . w[n]  +  (n < lora_cols ? t[i] . b[n] : 0),
//   t = scale * x A^T  (computed by the GEMM's own k-loop for r <= 32, else
//   by lora_down_kernel first).
//
// The GEMM is computed as C^T = W x^T so that the MFMA accumulator of a lane
// holds four consecutive output features of one token (8-byte stores).  Both
// operands are K-contiguous in memory ([rows][hidden]), so tiles go to LDS
// without a transpose.  Workgroup tile BN (features) x BM (tokens) x 64 (k),
// 32x32x16 MFMAs, fp32 accumulation, the operand tiles copied global -> LDS
// by the DMA form of the load.  Three kernels: gemm_lora_kernel (one wave per
// wave tile), gemm_kg2_kernel (96 x 64 wave tiles, two groups of waves on
// alternate k-steps) and gemm_ahead_kernel (one wave per wave tile, operand
// fragments read one k-step ahead; plain products and those whose low-rank t
// a kernel of its own computes).  At suffix sizes the operand ingest per CU is the
// ceiling (measured on gfx950: about 58 GB/s per CU, 15 TB/s out of the L2s,
// the same rate hipBLASLt's kernels reach on these shapes): large tiles ingest
// less, M N K 2 (1/BM + 1/BN) bytes, small ones keep every CU busy (plan_gemm
// weighs them), and the copies are spread between the MFMAs so that the
// compute hides under the ingest.  LDS rows are 128 bytes (eight 16-byte
// chunks); chunk c of row r is stored at c ^ ((r >> 1) & 7), so the 16 rows
// one operand read touches in a cycle land on 16 distinct bank groups.
//
// The LoRA term enters as extra MFMA k-steps after the main loop: A operand
// = rows of B (rank padded to 16 with zeros), B operand = t rounded to a
// bf16 hi/lo pair, so t keeps ~16 significant bits and the update is summed
// in fp32.  lora_down_kernel leaves t as fp32 partial sums over slices of
// the hidden dimension (256 or 1024 wide); the epilogue adds the slices in
// order.

#include <type_traits>

#include <algorithm>
#include <cmath>

#include "common.h"
#include "kernels.h"
#include "attuner.h"

namespace attuner {

namespace {

constexpr int BK = 64;
constexpr int kChunksPerRow = BK / 8;  // 16-byte chunks per LDS row
constexpr int kLoraSlice = 256;        // hidden elements per lora_down chunk (four waves x 64)
constexpr int kLoraSliceWide = 1024;   // hidden elements per lora_down workgroup above kGemvMaxTok tokens
constexpr int kLoraRows = 32;          // A rows staged per k-tile when the down-projection is fused
constexpr int kGroupM = 4;             // token tiles per group of the tile order

__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// Fused low-rank epilogue and store of one wave's FN x FM blocks of C^T:
// acc += B[n][:] . t[m][:] for features n < lora_cols, then bf16 stores (lane
// holds features nb + 8q + 4*hi + (0..3) of token m).  n_base / m_base: the
// wave tile's first feature / token.
template <int FN, int FM>
__device__ __forceinline__ void lora_epilogue_store(f32x16 (&acc)[FN][FM], int n_base, int m_base, int ml_base,
                                                    int l32, int hi, int M, int N, const bf16_t* __restrict__ b,
                                                    int rank, int r_pad, int lora_cols,
                                                    const float* __restrict__ t_part, int n_slice,
                                                    const float* t_lds, const GemmEpi& epi, bf16_t* out,
                                                    const u32x4 (*b_pre)[2] = nullptr) {
  if (r_pad > 0 && n_base < lora_cols) {
    const int64_t slice_stride = (int64_t)M * r_pad;
    // B rows as 16-byte loads when they are whole 16-byte runs
    const bool b_vec = (rank & 7) == 0 && (reinterpret_cast<uintptr_t>(b) & 15) == 0;
#pragma unroll
    for (int ks = 0; ks < ATTUNER_MAX_RANK; ks += 16) {
      if (ks >= r_pad) break;
      bf16x8 th[FM], tl[FM];
#pragma unroll
      for (int j = 0; j < FM; ++j) {
        f32x4 s0 = f32x4{}, s1 = f32x4{};
        if (t_lds != nullptr) {
          // fused: t[token][rank] staged in LDS by this workgroup
          const float* tr = t_lds + (ml_base + j * 32 + l32) * (kLoraRows + 1) + ks + 8 * hi;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s0[e] = tr[e];
            s1[e] = tr[4 + e];
          }
        } else {
          int m = m_base + j * 32 + l32;
          m = m < M ? m : M - 1;
          const float* tp = t_part + (int64_t)m * r_pad + ks + 8 * hi;
          for (int z = 0; z < n_slice; ++z) {
            s0 += *reinterpret_cast<const f32x4*>(tp + z * slice_stride);
            s1 += *reinterpret_cast<const f32x4*>(tp + z * slice_stride + 4);
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const __bf16 h0 = static_cast<__bf16>(s0[e]);
          const __bf16 h1 = static_cast<__bf16>(s1[e]);
          th[j][e] = h0;
          th[j][e + 4] = h1;
          tl[j][e] = static_cast<__bf16>(s0[e] - static_cast<float>(h0));
          tl[j][e + 4] = static_cast<__bf16>(s1[e] - static_cast<float>(h1));
        }
      }
#pragma unroll
      for (int i = 0; i < FN; ++i) {
        const int nb = n_base + i * 32;
        if (nb >= lora_cols) continue;  // lora_cols is a multiple of 32
        const int n = nb + l32;
        bf16x8 a;
        const int j0 = ks + 8 * hi;  // this lane's 8 ranks j0 .. j0 + 7 of B row n
        if (b_pre != nullptr && ks < kGemmFusedLoraMaxRank) {
          a = as_bf16x8(b_pre[i][ks < kGemmFusedLoraMaxRank ? ks / 16 : 0]);
        } else if (b_vec) {
          // rank % 8 == 0: the 8 ranks are all below rank or all past it
          u32x4 v = u32x4{0u, 0u, 0u, 0u};
          if (j0 < rank) v = *reinterpret_cast<const u32x4*>(b + (int64_t)n * rank + j0);
          a = as_bf16x8(v);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const bf16_t bv = j0 + e < rank ? b[(int64_t)n * rank + j0 + e] : (bf16_t)0;
            a[e] = __builtin_bit_cast(__bf16, bv);
          }
        }
#pragma unroll
        for (int j = 0; j < FM; ++j) {
          acc[i][j] = mfma32(a, th[j], acc[i][j]);
          acc[i][j] = mfma32(a, tl[j], acc[i][j]);
        }
      }
    }
  }

#pragma unroll
  for (int j = 0; j < FM; ++j) {
    const int m = m_base + j * 32 + l32;
    if (m >= M) continue;
#pragma unroll
    for (int i = 0; i < FN; ++i) {
      const int nb = n_base + i * 32;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = nb + 8 * q + 4 * hi;  // features n .. n + 3 of token m
        float c[4] = {acc[i][j][4 * q + 0], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        if (epi.mode == kEpiF32) {
          *reinterpret_cast<f32x4*>(epi.out_f32 + (int64_t)m * N + n) = f32x4{c[0], c[1], c[2], c[3]};
          continue;
        }
        if (epi.mode == kEpiSwiglu) {
          // (gate, up) pairs (n, n + 1) and (n + 2, n + 3) -> outputs n / 2, n / 2 + 1
          const float s0 = c[0] / (1.0f + __expf(-c[0])) * c[1];
          const float s1 = c[2] / (1.0f + __expf(-c[2])) * c[3];
          *reinterpret_cast<uint32_t*>(out + (int64_t)m * (N / 2) + n / 2) = pack_bf16x2(s0, s1);
          continue;
        }
        if (epi.mode == kEpiResidual) {
          const u32x2 r = *reinterpret_cast<const u32x2*>(epi.residual + (int64_t)m * N + n);
          c[0] += __uint_as_float(r[0] << 16);
          c[1] += __uint_as_float(r[0] & 0xFFFF0000u);
          c[2] += __uint_as_float(r[1] << 16);
          c[3] += __uint_as_float(r[1] & 0xFFFF0000u);
        }
        u32x2 pk;
        pk[0] = pack_bf16x2(c[0], c[1]);
        pk[1] = pack_bf16x2(c[2], c[3]);
        *reinterpret_cast<u32x2*>(out + (int64_t)m * N + n) = pk;
      }
    }
  }
}

// Both operand tiles are copied global -> LDS by the DMA form of the load
// (16 bytes per lane, no staging registers) into an NST-stage ring, so NST - 1
// k-tiles are in flight per workgroup while one is multiplied.  WN x WM waves;
// one barrier per k-tile.  A k-tile stage is (BN + BM) rows of 128 bytes,
// moved as 1 KiB blocks of 8 rows (lane i -> row 8 blk + i / 8, physical
// chunk i % 8, holding the logical chunk the swizzle maps there).
template <int BM, int BN, int WN, int WM, int NST>
__global__ __launch_bounds__(64 * WN * WM, 1) void gemm_lora_kernel(const bf16_t* __restrict__ x,
                                                                   const bf16_t* __restrict__ w, int M, int N, int K,
                                                                   const bf16_t* __restrict__ a, float scale,
                                                                   const bf16_t* __restrict__ b, int rank, int r_pad,
                                                                   int lora_cols, const float* __restrict__ t_part,
                                                                   int n_slice, GemmEpi epi, bf16_t* out, int n_mt,
                                                                   int n_nt, int kt_split) {
  constexpr int NW = WN * WM;
  constexpr int TN = BN / WN, TM = BM / WM;
  constexpr int FN = TN / 32, FM = TM / 32;
  static_assert(FN >= 1 && FM >= 1 && TN % 32 == 0 && TM % 32 == 0, "bad wave layout");
  // stage rows: W rows [0, BN), x rows [BN, BN + BM), and (fused LoRA) the
  // kLoraRows rows of A [BN + BM, BN + BM + kLoraRows)
  constexpr int ROWS = BN + BM + kLoraRows;
  static_assert((BN + BM) % 8 == 0, "stage must be whole 1 KiB blocks");
  constexpr int STAGE = ROWS * kChunksPerRow;
  static_assert(BM * (kLoraRows + 1) * 4 <= STAGE * 16, "t staging must fit one stage");
  __shared__ u32x4 lds[NST * STAGE];

  // Tile order.  Workgroup i runs on XCD i % 8: each XCD gets a contiguous
  // run of the order below, so the ~32 workgroups one XCD runs at a time
  // share operand panels in its L2.  The order walks groups of kGroupM token
  // tiles across all feature tiles, token tile fastest: 32 concurrent
  // workgroups cover about kGroupM x 8 tiles (kGroupM x-panels, 8 W-panels).
  // Split-K (kt_split > 0): workgroup blockIdx.x / total takes k-tiles
  // [split * kt_split, (split + 1) * kt_split) of tile blockIdx.x % total and
  // writes its fp32 partial to slice `split` of epi.out_f32.
  const int total = n_mt * n_nt;
  const int per_xcd = total >> 3;
  const int split = kt_split > 0 ? (int)blockIdx.x / total : 0;
  int lin = kt_split > 0 ? (int)blockIdx.x % total : (int)blockIdx.x;
  if (lin < 8 * per_xcd) lin = (lin & 7) * per_xcd + (lin >> 3);
  const int in_group = kGroupM * n_nt;
  const int first_m = (lin / in_group) * kGroupM;
  const int gm = min(n_mt - first_m, kGroupM);
  const int mt = first_m + (lin % in_group) % gm;
  const int nt = (lin % in_group) / gm;
  const int n0 = nt * BN;
  const int m0 = mt * BM;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wn = wave / WM;
  const int wm = wave % WM;
  const int l32 = lane & 31;
  const int hi = lane >> 5;
  const int kt0 = split * kt_split;
  const int n_kt = kt_split > 0 ? min(K / BK - kt0, kt_split) : K / BK;
  const uint32_t lds0 = lds_addr(lds);

  f32x16 acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = f32x16{};

  // Fused down-projection (t_part == null): this workgroup needs t for its
  // tokens, so the k-loop also stages A's rows and, for each 32-token block,
  // one wave that holds its x fragments accumulates t^T = A x^T next to its
  // main MFMAs.  t then goes through LDS to the epilogue.
  const bool fused = t_part == nullptr && r_pad > 0 && n0 < lora_cols;
  static_assert(FM <= WN, "at most one t block per wave");
  f32x16 tacc = f32x16{};

  // la_tag: stage A's rows; tj_tag: the token block whose t this wave
  // accumulates (-1: none)
  auto kloop = [&](auto la_tag, auto tj_tag) __attribute__((always_inline)) {
    constexpr bool LA = decltype(la_tag)::value;
    constexpr int TJ = decltype(tj_tag)::value;
    constexpr int NBLK = (BN + BM + (LA ? kLoraRows : 0)) / 8;
    constexpr int PW = (NBLK + NW - 1) / NW;  // DMA instructions per wave per stage
    static_assert((NST - 2) * PW <= 63, "vmcnt range");
    // DMA sources of this lane (blocks past the stage repeat the last block:
    // same bytes to the same place)
    const bf16_t* src[PW];
    uint32_t doff[PW];
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int blk = min(wave + NW * j, NBLK - 1);
      const int row = 8 * blk + (lane >> 3);
      const int lg = swz(row, lane & 7);
      const bf16_t* base;
      if (row < BN) {
        base = w + (int64_t)(n0 + row) * K;
      } else if (row < BN + BM) {
        const int m = min(m0 + row - BN, M - 1);  // rows past the end are computed, never stored
        base = x + (int64_t)m * K;
      } else {
        // A rows past rank repeat row rank - 1: finite, and met by zero B columns
        base = a + (int64_t)min(row - BN - BM, rank - 1) * K;
      }
      src[j] = base + 8 * lg + (int64_t)kt0 * BK;
      doff[j] = 1024u * blk;
    }
#pragma unroll
    for (int st = 0; st < NST - 1; ++st) {
      const int kt = min(st, n_kt - 1);
#pragma unroll
      for (int j = 0; j < PW; ++j) lds_dma16(src[j] + kt * BK, lds0 + (uint32_t)(st * STAGE * 16) + doff[j]);
    }
    int slot = 0, nslot = NST - 1;
    for (int kt = 0; kt < n_kt; ++kt) {
      // own copies of tile kt done, then everyone's; slot nslot (tile kt - 1) is free
      __builtin_amdgcn_s_waitcnt(vmcnt_wait((NST - 2) * PW));
      barrier_no_fence();
      const int nk = min(kt + NST - 1, n_kt - 1);
      const u32x4* cur = lds + slot * STAGE;
#pragma unroll
      for (int j = 0; j < PW; ++j) lds_dma16(src[j] + nk * BK, lds0 + (uint32_t)(nslot * STAGE * 16) + doff[j]);
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        const int ch = 2 * ks + hi;
        bf16x8 af[FN], bfr[FM];
#pragma unroll
        for (int i = 0; i < FN; ++i) {
          const int row = wn * TN + i * 32 + l32;
          af[i] = as_bf16x8(cur[row * kChunksPerRow + swz(row, ch)]);
        }
#pragma unroll
        for (int j = 0; j < FM; ++j) {
          const int row = BN + wm * TM + j * 32 + l32;
          bfr[j] = as_bf16x8(cur[row * kChunksPerRow + swz(row, ch)]);
        }
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
          for (int j = 0; j < FM; ++j) acc[i][j] = mfma32(af[i], bfr[j], acc[i][j]);
        if constexpr (TJ >= 0) {
          const int row = BN + BM + l32;
          tacc = mfma32(as_bf16x8(cur[row * kChunksPerRow + swz(row, ch)]), bfr[TJ], tacc);
        }
      }
      slot = slot + 1 == NST ? 0 : slot + 1;
      nslot = nslot + 1 == NST ? 0 : nslot + 1;
    }
    // the clamped copies of the last iterations must land before the LDS is
    // reused or the workgroup ends (its LDS may be handed to the next one)
    __builtin_amdgcn_s_waitcnt(vmcnt_wait(0));
  };

  const float* t_lds = nullptr;
  // the wave's B rows, requested before the k-loop (whole 16-byte runs only):
  // read in the epilogue they would cost it a memory latency
  u32x4 b_pre[FN][2];
  const bool pre = fused && (rank & 7) == 0 && (reinterpret_cast<uintptr_t>(b) & 15) == 0;
  if (pre) {
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int nb = n0 + wn * TN + i * 32, j0 = 16 * q + 8 * hi;
        b_pre[i][q] = u32x4{0u, 0u, 0u, 0u};
        if (nb < lora_cols && j0 < rank)
          b_pre[i][q] = *reinterpret_cast<const u32x4*>(b + (int64_t)(nb + l32) * rank + j0);
      }
  }
  if (fused) {
    // t block j (32 tokens) is accumulated by the wave column wn == j of the
    // wave row that holds those tokens.  Each case is a loop of its own: a
    // branch inside the loop would end a basic block at every k-step, and the
    // next step's LDS reads could not be issued before it (one layer of 256
    // tokens x 2560 at rank 16, 27 us of it this product: 84.3 us with the
    // branch and B read in the epilogue, 80.8 us as it is now).
    const std::integral_constant<bool, true> la{};
    if (wn == 0) kloop(la, std::integral_constant<int, 0>{});
    else if (FM > 1 && wn == 1) kloop(la, std::integral_constant<int, (FM > 1 ? 1 : 0)>{});
    else kloop(la, std::integral_constant<int, -1>{});
    static_assert(FM <= 2, "t blocks 0 and 1 only");
    // t^T accumulator: lane holds ranks 8 (v / 4) + 4 hi + v % 4 of token
    // l32 of each 32-token block; staged as fp32 t[token][rank], row stride
    // kLoraRows + 1
    float* ts = reinterpret_cast<float*>(lds);
    barrier_no_fence();
    if (wn < FM) {
      const int ml = wm * TM + wn * 32 + l32;
#pragma unroll
      for (int v = 0; v < 16; ++v) ts[ml * (kLoraRows + 1) + 8 * (v >> 2) + 4 * hi + (v & 3)] = scale * tacc[v];
    }
    __syncthreads();
    t_lds = ts;
  } else {
    kloop(std::integral_constant<bool, false>{}, std::integral_constant<int, -1>{});
  }

  if (kt_split > 0) epi.out_f32 += (int64_t)split * M * N;
  if (pre)
    lora_epilogue_store<FN, FM>(acc, n0 + wn * TN, m0 + wm * TM, wm * TM, l32, hi, M, N, b, rank, r_pad, lora_cols,
                                t_part, n_slice, t_lds, epi, out, b_pre);
  else
    lora_epilogue_store<FN, FM>(acc, n0 + wn * TN, m0 + wm * TM, wm * TM, l32, hi, M, N, b, rank, r_pad, lora_cols,
                                t_part, n_slice, t_lds, epi, out);
}

// The same product with two k-groups of waves.  Each wave holds a 96 x 64
// (features x tokens) tile of C^T, which reads 5 LDS fragments per 6 MFMAs
// (3 per 2 for the 32 x 64 tile above), and the waves of group g take
// k-steps g and g + 2 of every 64-deep k-tile, so that two waves share each
// SIMD and cover each other's LDS latency.  After the k-loop the groups
// exchange halves through LDS: group g gives its partner its partial sums of
// token block 1 - g and adds the partner's partial sums of token block g,
// then applies the epilogue to block g.  The fused LoRA down-projection is
// split the same way (each group's t^T over its k-steps, summed in LDS).
template <int BM, int BN, int WN, int WM, int NST>
__global__ __launch_bounds__(128 * WN * WM, 1) void gemm_kg2_kernel(const bf16_t* __restrict__ x,
                                                                   const bf16_t* __restrict__ w, int M, int N, int K,
                                                                   const bf16_t* __restrict__ a, float scale,
                                                                   const bf16_t* __restrict__ b, int rank, int r_pad,
                                                                   int lora_cols, const float* __restrict__ t_part,
                                                                   int n_slice, GemmEpi epi, bf16_t* out, int n_mt,
                                                                   int n_nt, int kt_split) {
  constexpr int NWG = WN * WM;  // waves per k-group
  constexpr int NW = 2 * NWG;
  constexpr int TN = BN / WN, TM = BM / WM;
  constexpr int FN = TN / 32, FM = TM / 32;
  static_assert(FM == 2 && FN >= 1 && TN % 32 == 0, "each group finishes one of a wave's two token blocks");
  constexpr int ROWS = BN + BM + kLoraRows;
  static_assert((BN + BM) % 8 == 0, "stage must be whole 1 KiB blocks");
  constexpr int STAGE = ROWS * kChunksPerRow;
  __shared__ u32x4 lds[NST * STAGE];
  // after the k-loop: t staging [BM][kLoraRows + 1] floats, then the exchange
  // [2 groups][NWG waves][FN][16][64 lanes] floats
  constexpr int kTsFloats = (BM * (kLoraRows + 1) + 63) / 64 * 64;
  static_assert((kTsFloats + 2 * NWG * FN * 16 * 64) * 4 <= NST * STAGE * 16, "exchange must fit the ring");

  const int total = n_mt * n_nt;
  const int per_xcd = total >> 3;
  const int split = kt_split > 0 ? (int)blockIdx.x / total : 0;
  int lin = kt_split > 0 ? (int)blockIdx.x % total : (int)blockIdx.x;
  if (lin < 8 * per_xcd) lin = (lin & 7) * per_xcd + (lin >> 3);
  const int in_group = kGroupM * n_nt;
  const int first_m = (lin / in_group) * kGroupM;
  const int gm = min(n_mt - first_m, kGroupM);
  const int mt = first_m + (lin % in_group) % gm;
  const int nt = (lin % in_group) / gm;
  const int n0 = nt * BN;
  const int m0 = mt * BM;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int kg = wave / NWG;
  const int wv = wave % NWG;
  const int wn = wv / WM;
  const int wm = wv % WM;
  const int l32 = lane & 31;
  const int hi = lane >> 5;
  const int kt0 = split * kt_split;
  const int n_kt = kt_split > 0 ? min(K / BK - kt0, kt_split) : K / BK;
  const uint32_t lds0 = lds_addr(lds);

  f32x16 acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = f32x16{};
  const bool fused = t_part == nullptr && r_pad > 0 && n0 < lora_cols;
  f32x16 tacc[FM];
#pragma unroll
  for (int j = 0; j < FM; ++j) tacc[j] = f32x16{};

  auto kloop = [&](auto la_tag) __attribute__((always_inline)) {
    constexpr bool LA = decltype(la_tag)::value;
    constexpr int NBLK = (BN + BM + (LA ? kLoraRows : 0)) / 8;
    constexpr int PW = (NBLK + NW - 1) / NW;
    static_assert((NST - 2) * PW <= 63, "vmcnt range");
    const bf16_t* src[PW];
    uint32_t doff[PW];
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int blk = min(wave + NW * j, NBLK - 1);
      const int row = 8 * blk + (lane >> 3);
      const int lg = swz(row, lane & 7);
      const bf16_t* base;
      if (row < BN) {
        base = w + (int64_t)(n0 + row) * K;
      } else if (row < BN + BM) {
        const int m = min(m0 + row - BN, M - 1);
        base = x + (int64_t)m * K;
      } else {
        base = a + (int64_t)min(row - BN - BM, rank - 1) * K;
      }
      src[j] = base + 8 * lg + (int64_t)kt0 * BK;
      doff[j] = 1024u * blk;
    }
#pragma unroll
    for (int st = 0; st < NST - 1; ++st) {
      const int kt = min(st, n_kt - 1);
#pragma unroll
      for (int j = 0; j < PW; ++j) lds_dma16(src[j] + kt * BK, lds0 + (uint32_t)(st * STAGE * 16) + doff[j]);
    }
    int slot = 0, nslot = NST - 1;
    for (int kt = 0; kt < n_kt; ++kt) {
      __builtin_amdgcn_s_waitcnt(vmcnt_wait((NST - 2) * PW));
      barrier_no_fence();
      const int nk = min(kt + NST - 1, n_kt - 1);
      const u32x4* cur = lds + slot * STAGE;
      // fragments of both k-steps (the second read while the first multiplies)
      bf16x8 af[2][FN], bfr[2][FM], ar[2];
      auto load = [&](int s2) __attribute__((always_inline)) {
        const int ch = 2 * (kg + 2 * s2) + hi;
#pragma unroll
        for (int i = 0; i < FN; ++i) {
          const int row = wn * TN + i * 32 + l32;
          af[s2][i] = as_bf16x8(cur[row * kChunksPerRow + swz(row, ch)]);
        }
#pragma unroll
        for (int j = 0; j < FM; ++j) {
          const int row = BN + wm * TM + j * 32 + l32;
          bfr[s2][j] = as_bf16x8(cur[row * kChunksPerRow + swz(row, ch)]);
        }
        if (LA && wn < FM) {
          const int row = BN + BM + l32;
          ar[s2] = as_bf16x8(cur[row * kChunksPerRow + swz(row, ch)]);
        }
      };
      constexpr int HALF = (PW + 1) / 2;
      load(0);
      load(1);
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        int q = 0;
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
          for (int j = 0; j < FM; ++j) {
            acc[i][j] = mfma32(af[s2][i], bfr[s2][j], acc[i][j]);
            if (q % 2 == 1) {
              const int d = s2 * HALF + q / 2;
              if (d < PW && q / 2 < HALF) {
                __builtin_amdgcn_sched_barrier(0);
                lds_dma16(src[d] + nk * BK, lds0 + (uint32_t)(nslot * STAGE * 16) + doff[d]);
                __builtin_amdgcn_sched_barrier(0);
              }
            }
            ++q;
          }
        if (LA && wn < FM) {
#pragma unroll
          for (int j = 0; j < FM; ++j)
            if (j % WN == wn) tacc[j] = mfma32(ar[s2], bfr[s2][j], tacc[j]);
        }
        // DMAs of this half not yet issued (more than FN * FM / 2 of them)
#pragma unroll
        for (int e = (FN * FM) / 2; e < HALF; ++e) {
          const int d = s2 * HALF + e;
          if (d < PW) lds_dma16(src[d] + nk * BK, lds0 + (uint32_t)(nslot * STAGE * 16) + doff[d]);
        }
      }
      slot = slot + 1 == NST ? 0 : slot + 1;
      nslot = nslot + 1 == NST ? 0 : nslot + 1;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_wait(0));
  };

  if (fused) kloop(std::integral_constant<bool, true>{});
  else kloop(std::integral_constant<bool, false>{});
  __syncthreads();  // every wave is done with the ring

  float* ts = reinterpret_cast<float*>(lds);
  float* xch = ts + kTsFloats;
  const float* t_lds = nullptr;
  if (fused) {
    // t^T accumulator: lane holds ranks 8 (v / 4) + 4 hi + v % 4 of token
    // l32 of each 32-token block; staged as t[token][rank] (row stride
    // kLoraRows + 1), group 0's sums first, group 1's added
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      if (kg == g) {
#pragma unroll
        for (int j = 0; j < FM; ++j) {
          if (j % WN != wn || wn >= FM) continue;
          const int ml = wm * TM + j * 32 + l32;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float* d = ts + ml * (kLoraRows + 1) + 8 * (v >> 2) + 4 * hi + (v & 3);
            *d = g == 0 ? scale * tacc[j][v] : *d + scale * tacc[j][v];
          }
        }
      }
      __syncthreads();
    }
    t_lds = ts;
  }

  if (kt_split > 0) epi.out_f32 += (int64_t)split * M * N;
  auto finish = [&](auto j_tag) __attribute__((always_inline)) {
    constexpr int J = decltype(j_tag)::value;  // the token block this group finishes
    float* give = xch + ((kg * NWG + wv) * FN) * 1024;
    float* take = xch + (((1 - kg) * NWG + wv) * FN) * 1024;
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) give[(i * 16 + v) * 64 + lane] = acc[i][1 - J][v];
    __syncthreads();
    f32x16 mine[FN][1];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) mine[i][0][v] = acc[i][J][v] + take[(i * 16 + v) * 64 + lane];
    lora_epilogue_store<FN, 1>(mine, n0 + wn * TN, m0 + wm * TM + 32 * J, wm * TM + 32 * J, l32, hi, M, N, b, rank,
                               r_pad, lora_cols, t_part, n_slice, t_lds, epi, out);
  };
  if (kg == 0) finish(std::integral_constant<int, 0>{});
  else finish(std::integral_constant<int, 1>{});
}

// The same product for the largest tiles, with the operand fragments read one
// k-step ahead.  What bounds these tiles is not a rate but waiting: with 64 KB
// per k-tile only two fit in LDS, and a ring slot that is free only when its
// k-tile has been multiplied leaves its refill half a k-tile (about 0.5 us,
// less than a loaded L2's latency) to land.  Here a wave reads the FN + FM
// fragments of the next k-step between the MFMAs of the current one, so a slot
// is free when its last k-step has been read, before that step is multiplied:
// the refill then has a whole k-tile to land, no MFMA waits for an LDS read
// issued just before it, and there is one barrier per k-tile.  Copies take a
// scalar base and a fixed 32-bit lane offset, which leaves the registers for
// the second set of fragments.  The low-rank term comes from t_part only.
// Measured against the same tiles without read-ahead (one box, 1024 tokens):
// 256 x 256 at 4096 -> 24576 236 against 252 us, 128 x 256 252 against 277 us
// and at 12288 -> 4096 (2 splits) 120 against 143 us; a 256 x 256 workgroup
// takes 160k shader cycles for 64 k-tiles, 132k of them MFMA issue, and from
// there the chip's power sets the clock (1.58 GHz with every CU busy, 2.25 GHz
// on zeros).  Waves are wider in the features' direction where the tile allows
// it: 2 x 4 waves of 128 x 64 at 256 x 256 read 6 fragments per 8 MFMAs.
template <int BM, int BN, int WN, int WM, int NST>
__global__ __launch_bounds__(64 * WN * WM, 1) void gemm_ahead_kernel(const bf16_t* __restrict__ x,
                                                                    const bf16_t* __restrict__ w, int M, int N, int K,
                                                                    const bf16_t* __restrict__ b, int rank, int r_pad,
                                                                    int lora_cols, const float* __restrict__ t_part,
                                                                    int n_slice, GemmEpi epi, bf16_t* out, int n_mt,
                                                                    int n_nt, int kt_split, int part_kt) {
  constexpr int NW = WN * WM;
  constexpr int TN = BN / WN, TM = BM / WM;
  constexpr int FN = TN / 32, FM = TM / 32;
  constexpr int NBLK = (BN + BM) / 8;  // 1 KiB blocks of a k-tile stage
  constexpr int PW = NBLK / NW;        // copies per wave and k-tile
  static_assert(TN % 32 == 0 && TM % 32 == 0 && NBLK % NW == 0 && (NST - 1) * PW <= 63, "bad wave layout");
  constexpr int STAGE = (BN + BM) * kChunksPerRow;
  __shared__ u32x4 lds[NST * STAGE];

  // tile order and key split as in gemm_lora_kernel
  const int total = n_mt * n_nt;
  const int per_xcd = total >> 3;
  const int split = kt_split > 0 ? (int)blockIdx.x / total : 0;
  int lin = kt_split > 0 ? (int)blockIdx.x % total : (int)blockIdx.x;
  if (lin < 8 * per_xcd) lin = (lin & 7) * per_xcd + (lin >> 3);
  const int in_group = kGroupM * n_nt;
  const int first_m = (lin / in_group) * kGroupM;
  const int gm = min(n_mt - first_m, kGroupM);
  const int mt = first_m + (lin % in_group) % gm;
  const int nt = (lin % in_group) / gm;
  const int n0 = nt * BN;
  const int m0 = mt * BM;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wn = wave / WM;
  const int wm = wave % WM;
  const int l32 = lane & 31;
  const int hi = lane >> 5;
  const int kt0 = split * kt_split;
  const int n_kt = kt_split > 0 ? min(K / BK - kt0, kt_split) : K / BK;
  const uint32_t lds0 = lds_addr(lds);

  // Copy j of this wave moves block wave + NW j: rows 8 (wave + NW j) .. + 7
  // of the stage, W's first (whole blocks of one operand: BN % 8 == 0).
  const bf16_t* sbase[PW];
  uint32_t voff[PW];
#pragma unroll
  for (int j = 0; j < PW; ++j) {
    const int row = 8 * (wave + NW * j) + (lane >> 3);
    const bool is_w = 8 * (wave + NW * j) < BN;
    // x rows past the end repeat the last: computed, never stored
    const int r = is_w ? row : min(m0 + row - BN, M - 1) - m0;
    sbase[j] = (is_w ? w + (int64_t)n0 * K : x + (int64_t)m0 * K) + (int64_t)kt0 * BK;
    voff[j] = 2u * ((uint32_t)r * (uint32_t)K + 8u * (uint32_t)swz(row, lane & 7));
  }
  // A few-token tile streams W from memory, each workgroup one 128-byte line of
  // BN rows at a time.  Started together they would all read the same columns,
  // which at a power-of-two row stride fall on few memory channels: workgroup
  // lin starts lin k-tiles further on and wraps (16 tokens x 4096 -> 24576:
  // 44.7-46.5 us in step, 35.4 staggered; no change at 2560 and 9728).  Larger
  // token tiles share operand panels in L2 and lose by it (256 x 192 at 6000
  // tokens x 4096 -> 6144: 263-274 in step, 268-301 staggered).
  // Where the result itself is fp32 (part_kt > 0: logits) the order of the sum
  // shows, so every workgroup takes k in order there (equal rows of W then give
  // equal bits), and as at most eight parts of part_kt k-tiles that are summed
  // apart and then pairwise: the largest logit of 16 x 4096 -> 151936 is off by
  // 5.5e-8 relative (one chain over k: 3.5e-7; the matrix-core GEMV: 7.0e-8).
  // 16 rows x 2560 -> 151936 with its argmax takes 153.5 us either way, 16 x
  // 512 -> 40960 18.6 against 17.5; a staggered start gave the logits nothing.
  constexpr bool kFew = BM == 32;
  static_assert(!kFew || FN * FM == 1, "one accumulator block per wave");
  const int kt_first = kFew && part_kt == 0 ? lin % n_kt : 0;
  auto copy = [&](int j, int kt, int slot) __attribute__((always_inline)) {
    if (kFew) {
      kt += kt_first;
      kt -= kt >= n_kt ? n_kt : 0;
    }
    lds_dma16_s(sbase[j] + (int64_t)kt * BK, voff[j], lds0 + (uint32_t)(slot * STAGE * 16) + 1024u * (wave + NW * j));
  };

  f32x16 acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = f32x16{};

  // fragments of one k-step: FN of W, then FM of x
  typedef bf16x8 Frags[FN + FM];
  Frags f0, f1;
  auto read = [&](Frags& f, const u32x4* cur, int ks, int e) __attribute__((always_inline)) {
    const int row = e < FN ? wn * TN + e * 32 + l32 : BN + wm * TM + (e - FN) * 32 + l32;
    f[e] = as_bf16x8(cur[row * kChunksPerRow + swz(row, 2 * ks + hi)]);
  };
  // the MFMAs of `cur`, with the reads of the next k-step (ks of stage `st`)
  // and (COPY) the refill of slot cslot with tile kt spread between them
  constexpr int NM = FN * FM, NR = FN + FM;
  auto phase = [&](Frags& cur, Frags& nxt, const u32x4* st, int ks, auto copy_tag, int kt, int cslot)
                   __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NM; ++q) {
      acc[q / FM][q % FM] = mfma32(cur[q / FM], cur[FN + q % FM], acc[q / FM][q % FM]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = q * NR / NM; u < (q + 1) * NR / NM; ++u) read(nxt, st, ks, u);
      if constexpr (decltype(copy_tag)::value) {
#pragma unroll
        for (int u = q * PW / NM; u < (q + 1) * PW / NM; ++u) copy(u, kt, cslot);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  const std::integral_constant<bool, true> with_copy{};
  const std::integral_constant<bool, false> no_copy{};

#pragma unroll
  for (int st = 0; st < NST; ++st)
    if (st < n_kt) {
#pragma unroll
      for (int j = 0; j < PW; ++j) copy(j, st, st);
    }
  if (n_kt >= NST) __builtin_amdgcn_s_waitcnt(vmcnt_wait((NST - 1) * PW));
  else __builtin_amdgcn_s_waitcnt(vmcnt_wait(0));
  barrier_no_fence();
#pragma unroll
  for (int u = 0; u < NR; ++u) read(f0, lds, 0, u);

  int slot = 0, kt = 0;
  auto tile = [&](auto copy_tag) __attribute__((always_inline)) {
    const int next = slot + 1 == NST ? 0 : slot + 1;
    const u32x4* st = lds + slot * STAGE;
    phase(f0, f1, st, 1, no_copy, 0, 0);
    phase(f1, f0, st, 2, no_copy, 0, 0);
    phase(f0, f1, st, 3, no_copy, 0, 0);
    // this wave has read all of tile kt and its copies of tile kt + 1 have
    // landed (tiles kt + 2 .. kt + NST - 1 may still fly; the last tiles wait
    // for all); past the barrier so has everyone, and tile kt's slot takes
    // tile kt + NST.  After the last tile a stale slot is read and not used.
    __builtin_amdgcn_s_waitcnt(vmcnt_wait(decltype(copy_tag)::value ? (NST - 2) * PW : 0) & ~(15 << 8));
    barrier_no_fence();
    phase(f1, f0, lds + next * STAGE, 0, copy_tag, kt + NST, slot);
    slot = next;
    ++kt;
  };
  if (kFew && part_kt > 0) {
    f32x16 part[4] = {f32x16{}, f32x16{}, f32x16{}, f32x16{}};  // part v goes to part[v % 4]
#pragma unroll 1
    while (kt < n_kt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int end = min(kt + part_kt, n_kt);
        acc[0][0] = f32x16{};
        while (kt < end && kt + NST < n_kt) tile(with_copy);
        while (kt < end) tile(no_copy);
        part[i] += acc[0][0];
        if (kt >= n_kt) break;
      }
    }
    acc[0][0] = (part[0] + part[2]) + (part[1] + part[3]);
  } else {
    while (kt + NST < n_kt) tile(with_copy);
    while (kt < n_kt) tile(no_copy);
  }

  if (kt_split > 0) epi.out_f32 += (int64_t)split * M * N;
  lora_epilogue_store<FN, FM>(acc, n0 + wn * TN, m0 + wm * TM, wm * TM, l32, hi, M, N, b, rank, r_pad, lora_cols,
                              t_part, n_slice, nullptr, epi, out);
}

// t = scale * x A^T with MFMAs, as fp32 partial sums per slice of the hidden
// dimension (slice_w wide: 256 for the few-token GEMV, which has few token
// blocks to spread, kLoraSliceWide otherwise, so that a GEMM epilogue sums
// fewer partials): workgroup (32-token block, slice), each wave multiplies a
// 64-wide part of every 256-wide chunk of the slice and the four waves are
// summed through LDS.  t_part[slice][token][r_pad]; ranks rank .. r_pad-1
// come out zero.
__global__ __launch_bounds__(256) void lora_down_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ a,
                                                        int n_tok, int hidden, int rank, int r_pad, float scale,
                                                        int slice_w, float* __restrict__ t_part) {
  __shared__ float red[4][2][16][64];
  const int mb = blockIdx.x, kz = blockIdx.y;
  const int m0 = mb * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, hf = lane >> 5;
  const int nblk = (r_pad + 31) / 32;
  const int m = min(m0 + l32, n_tok - 1);
  const bf16_t* xr = x + (int64_t)m * hidden;

  f32x16 acc[2] = {f32x16{}, f32x16{}};
  for (int c0 = kz * slice_w; c0 < min(hidden, (kz + 1) * slice_w); c0 += kLoraSlice) {
    u32x4 xa[4], ab[4][2];
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const int k = c0 + wave * 64 + st * 16 + 8 * hf;
      const bool kin = k < hidden;
      xa[st] = kin ? *reinterpret_cast<const u32x4*>(xr + k) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        const int n = 32 * nb + l32;
        ab[st][nb] = (kin && nb < nblk && n < rank) ? *reinterpret_cast<const u32x4*>(a + (int64_t)n * hidden + k)
                                                   : u32x4{0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
        if (nb < nblk) acc[nb] = mfma32(as_bf16x8(xa[st]), as_bf16x8(ab[st][nb]), acc[nb]);
  }
  // acc[nb][v] = C[token 8(v/4) + 4hf + v%4][rank 32nb + l32]
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave][nb][v][lane] = acc[nb][v];
  __syncthreads();

  for (int e = tid; e < nblk * 1024; e += 256) {
    const int nb = e >> 10, v = (e >> 6) & 15, ln = e & 63;
    const int tok = m0 + 8 * (v >> 2) + 4 * (ln >> 5) + (v & 3);
    const int rk = 32 * nb + (ln & 31);
    if (tok < n_tok && rk < r_pad)
      t_part[((int64_t)kz * n_tok + tok) * r_pad + rk] =
          scale * (red[0][nb][v][ln] + red[1][nb][v][ln] + red[2][nb][v][ln] + red[3][nb][v][ln]);
  }
}

}  // namespace

static int lora_slice_width(int n_tok) { return n_tok <= kGemvMaxTok ? kLoraSlice : kLoraSliceWide; }

int lora_down_slices(int hidden, int n_tok) {
  const int w = lora_slice_width(n_tok);
  return (hidden + w - 1) / w;
}

hipError_t launch_lora_down(const uint16_t* x, const uint16_t* a, int n_tok, int hidden, int rank, int r_pad,
                            float scale, float* t_part, hipStream_t stream) {
  if (n_tok == 0 || r_pad == 0) return hipSuccess;
  ATTUNER_LAUNCH("lora_down_kernel", lora_down_kernel,
                 dim3((n_tok + 31) / 32, lora_down_slices(hidden, n_tok)), dim3(256), stream, x, a, n_tok, hidden,
                 rank, r_pad, scale, lora_slice_width(n_tok), t_part);
  return hipGetLastError();
}

namespace {

// Sum of the n_split fp32 partials [n_split][M][N] and the epilogue of epi
// (thread = 4 consecutive outputs of one token).
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int n_split, int M, int N,
                                                            GemmEpi epi, bf16_t* out) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;  // quad index
  if (q >= (int64_t)M * N / 4) return;
  const int64_t m = q / (N / 4);
  const int n = (int)(q % (N / 4)) * 4;
  const int64_t plane = (int64_t)M * N;
  f32x4 c = *reinterpret_cast<const f32x4*>(part + m * N + n);
  for (int s = 1; s < n_split; ++s) c += *reinterpret_cast<const f32x4*>(part + s * plane + m * N + n);
  if (epi.mode == kEpiF32) {
    *reinterpret_cast<f32x4*>(epi.out_f32 + m * N + n) = c;
    return;
  }
  if (epi.mode == kEpiSwiglu) {
    const float s0 = c[0] / (1.0f + __expf(-c[0])) * c[1];
    const float s1 = c[2] / (1.0f + __expf(-c[2])) * c[3];
    *reinterpret_cast<uint32_t*>(out + m * (N / 2) + n / 2) = pack_bf16x2(s0, s1);
    return;
  }
  if (epi.mode == kEpiResidual) {
    const u32x2 r = *reinterpret_cast<const u32x2*>(epi.residual + m * N + n);
    c[0] += __uint_as_float(r[0] << 16);
    c[1] += __uint_as_float(r[0] & 0xFFFF0000u);
    c[2] += __uint_as_float(r[1] << 16);
    c[3] += __uint_as_float(r[1] & 0xFFFF0000u);
  }
  u32x2 pk;
  pk[0] = pack_bf16x2(c[0], c[1]);
  pk[1] = pack_bf16x2(c[2], c[3]);
  *reinterpret_cast<u32x2*>(out + m * N + n) = pk;
}

// A tile's cost, in microseconds: kt per 64-deep k-tile with every CU busy,
// first for the launch, the first k-tiles and the epilogue, round for each
// further round of 256 workgroups, and idle, the share of a round's k-tiles
// that it saves with the CUs empty (power and the shared L2s).  fuse: what the
// low-rank t adds to a k-tile where the kernel computes it itself (0: it can
// not).  Fitted together, see plan_gemm.
struct Tile {
  int bm, bn;
  double kt, first, round, idle, fuse;
};
constexpr Tile kTiles[] = {
    {256, 256, 1.614, 8.7, 7.0, 0.36, 0},    {256, 192, 1.246, 10.4, 5.8, 0.44, 0},   {128, 256, 0.923, 6.4, 3.2, 0.37, 0},
    {128, 128, 0.555, 5.7, 1.1, 0.22, 0},    {128, 64, 0.349, 6.4, 3.6, 0.26, 0},     {128, 128, 0.588, 6.7, 4.3, 0.14, 0.21},
    {64, 96, 0.344, 5.3, 3.2, 0.24, 0.08},   {64, 64, 0.251, 5.3, 2.5, 0.31, 0.32},   {128, 192, 0.706, 6.9, 3.8, 0.36, 0.22},
    {128, 96, 0.397, 7.6, 4.5, 0.35, 0.26},  {32, 128, 0.357, 6.2, 0.6, 0.45, 0},     {32, 64, 0.254, 5.3, 2.2, 0.36, 0},
    {128, 256, 0.910, 10.6, 3.9, 0.39, 0.19}};
constexpr int kNumTiles = (int)(sizeof(kTiles) / sizeof(kTiles[0]));

hipError_t launch_tile(int tile, int kt_split, int grid, const uint16_t* x, const uint16_t* w, int n_tok, int n_out,
                       int hidden, const uint16_t* a, float scale, const uint16_t* b, int rank, int r_pad,
                       int lora_cols, const float* t_part, int n_slice, GemmEpi epi, uint16_t* out, int part_kt,
                       hipStream_t stream) {
#define ATTUNER_GEMM(BM_, BN_, WN_, WM_, NST_)                                                                 \
  ATTUNER_LAUNCH("gemm_lora_kernel", (gemm_lora_kernel<BM_, BN_, WN_, WM_, NST_>), dim3((unsigned)grid),       \
                 dim3(64 * (WN_) * (WM_)), stream, x, w, n_tok, n_out, hidden, a, scale, b, rank, r_pad,       \
                 lora_cols, t_part, n_slice, epi, out, (n_tok + (BM_) - 1) / (BM_), n_out / (BN_), kt_split)
#define ATTUNER_GEMM_KG2(BM_, BN_, WN_, WM_, NST_)                                                             \
  ATTUNER_LAUNCH("gemm_kg2_kernel", (gemm_kg2_kernel<BM_, BN_, WN_, WM_, NST_>), dim3((unsigned)grid),       \
                 dim3(128 * (WN_) * (WM_)), stream, x, w, n_tok, n_out, hidden, a, scale, b, rank, r_pad,      \
                 lora_cols, t_part, n_slice, epi, out, (n_tok + (BM_) - 1) / (BM_), n_out / (BN_), kt_split)
#define ATTUNER_GEMM_AHEAD(BM_, BN_, WN_, WM_, NST_)                                                            \
  ATTUNER_LAUNCH("gemm_ahead_kernel", (gemm_ahead_kernel<BM_, BN_, WN_, WM_, NST_>), dim3((unsigned)grid),    \
                 dim3(64 * (WN_) * (WM_)), stream, x, w, n_tok, n_out, hidden, b, rank, r_pad, lora_cols,       \
                 t_part, n_slice, epi, out, (n_tok + (BM_) - 1) / (BM_), n_out / (BN_), kt_split, part_kt)
  switch (tile) {
    case 0: ATTUNER_GEMM_AHEAD(256, 256, 2, 4, 2); break;
    case 1: ATTUNER_GEMM_AHEAD(256, 192, 2, 4, 2); break;
    case 2: ATTUNER_GEMM_AHEAD(128, 256, 4, 2, 3); break;
    case 3: ATTUNER_GEMM_AHEAD(128, 128, 4, 2, 4); break;
    case 4: ATTUNER_GEMM_AHEAD(128, 64, 2, 2, 6); break;
    case 5: ATTUNER_GEMM(128, 128, 2, 2, 4); break;
    case 6: ATTUNER_GEMM(64, 96, 3, 2, 5); break;
    case 7: ATTUNER_GEMM(64, 64, 2, 2, 6); break;
    case 8: ATTUNER_GEMM_KG2(128, 192, 2, 2, 3); break;
    case 9: ATTUNER_GEMM_KG2(128, 96, 1, 2, 4); break;
    case 10: ATTUNER_GEMM_AHEAD(32, 128, 4, 1, 4); break;
    case 11: ATTUNER_GEMM_AHEAD(32, 64, 2, 1, 8); break;
    case 12: ATTUNER_GEMM(128, 256, 4, 2, 3); break;
    default: return hipErrorInvalidValue;  // callers keep n_out a multiple of 64: 64x64 always fits
  }
#undef ATTUNER_GEMM
#undef ATTUNER_GEMM_KG2
#undef ATTUNER_GEMM_AHEAD
  return hipGetLastError();
}

}  // namespace

// Tile and key split of a product: the least of a cost model over the tiles
// and splits.  One workgroup per CU at a time, in rounds of 256; the k-tiles'
// time and that of reading W from memory (8.12 TB/s, less with few workgroups)
// are added as squares.
// With kMaySplit, and when a tile's workgroups would leave CUs idle, the k
// range may be split across workgroups: shorter k-loops, paid for by the fp32
// partials (split * M * N * 8 bytes written and read at 7.47 TB/s) and the
// reduce launch.  A low-rank term that the tile does not compute itself costs
// the down-projection's launch and, per 16 ranks, the epilogue of each round.
// With one the small read-ahead tiles are left out: their few waves would each
// sum t's partials for 64 tokens (one layer of 184 tokens x 2560 at rank 64:
// 59.0 us with 128 x 64, 56.7 with 64 x 96).  An fp32 result of up to
// kGemvMaxTok tokens takes the tiles that sum it in parts, as exact as the GEMV
// would.  Ties go to the earlier tile and to no split.
//
// All tiles are on one scale: the constants are fitted together to every tile
// and split of 3,000 shapes (the model's products and generic ones, 9 to 16,000
// tokens, ranks 0 to 64; weights read from memory), for the plan they choose to
// be as near the fastest as the form allows: within 1 % of it in nine of ten of
// the model's shapes, within 2 % of generic ones.  Two scales, one of them an
// ingest rate without a cost per workgroup, had put tiles first that were not
// (us, the plan of the two scales / now):
// 5120 x 2560 -> 6144 at rank 16 193 (two-k-group 128 x 192) / 161 (256 x 256),
// 8192 tokens at rank 32 320 / 259, 6144 x 4096 at rank 16 353 / 286 (256 x
// 192); 512 x 12288 -> 4096 80 (128 x 64) / 64 (128 x 256 in 4 splits); 129 x
// 2560 -> 2560 17.3 (128 x 128 in 6) / 13.0 (64 x 64 in 2); 1152 x 2560 -> 2560
// 30.1 (128 x 128) / 25.8 (its read-ahead form).  128 x 256 has both forms: the
// one that computes t saves the down-projection's launch where k is short or the
// rounds are few (1152 x 2560 -> 6144 at rank 16 52.7, read-ahead 57.2; 410 x
// 576 -> 10496 18.5 / 24.8); a plain product takes the read-ahead one alone (4160
// x 12288 -> 4096 556 / 466).
//
// The GEMV streams W (tile -1) up to kGemvDotMaxTok tokens, up to kGemvMaxTok
// without a split, and up to kGemvMaxTok where it costs less.  Its matrix-core
// form has one workgroup of 16 rows on every CU up to 4096 outputs, and time
// goes with their number and k (fitted, within 10 %); the dot-product form (k
// no multiple of 128) reads x again for every row pair (within 7 %).  Measured, GEMV against
// the best tile, us: 16 tokens x 4096 -> 4096 12.6 / 12.4, 9 tokens 11.2 / 12.4;
// 16 x 3584 -> 4416 (a second workgroup on a few CUs) 17.6 / 12.4; 9 x 2560 ->
// 8192 17.3 / 18.4 with the argmax; 16 x 9728 -> 2560 22.4 / 16.3; 11 x 9792 ->
// 2112 (dot products) 28.7 / 15.7.
GemmPlan plan_gemm(int n_tok, int n_out, int k_dim, int r_pad, int mode, int may) {
  constexpr int kCUs = 256;
  constexpr int kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16};
  constexpr double kReadW = 8.12e6, kPartials = 7.47e6;        // bytes per us
  constexpr double kReduce = 0.59, kPerSplit = 0.26;           // us
  constexpr double kDown = 10.98, kTBase = 1.19, kTArea = 2.88;  // us; per 16 ranks, and more for 256 x 256 outputs
  constexpr double kReadWgs = 185;  // fewer workgroups have too few bytes in flight
  const int n_kt = k_dim / BK;
  GemmPlan best{-1, 1, 0};
  if (n_tok <= kGemvDotMaxTok || (n_tok <= kGemvMaxTok && !(may & kMaySplit))) return best;
  const double read_w = (double)n_out * k_dim * 2 / kReadW;
  double best_t = 0.0;
  for (int i = 0; i < kNumTiles; ++i) {
    const Tile& tl = kTiles[i];
    if (n_out % tl.bn != 0 || (tl.bm == 32 && (r_pad > 0 || n_tok > 32 || !(may & kMayFewTok)))) continue;
    if (tl.bm != 32 && mode == kEpiF32 && n_tok <= kGemvMaxTok) continue;
    if (r_pad > 0 && tl.fuse == 0 && (!(may & kMayDown) || tl.bm * tl.bn <= 128 * 128)) continue;
    const bool fused = r_pad > 0 && r_pad <= kGemmFusedLoraMaxRank && tl.fuse > 0;
    if (tl.bm * tl.bn == 128 * 256 && tl.fuse > 0 && !fused) continue;  // its read-ahead form
    const int64_t tiles = (int64_t)((n_tok + tl.bm - 1) / tl.bm) * (n_out / tl.bn);
    for (int s : kSplits) {
      // splits only add workgroups where the tiles alone leave CUs idle
      if (s > 1 && (!(may & kMaySplit) || n_kt < 4 * s || tiles >= kCUs)) break;
      const int kts = (n_kt + s - 1) / s;
      const int used = (n_kt + kts - 1) / kts;  // splits that hold k-tiles
      // fp32 partials of every split: bounded, so that a reserved workspace holds any plan
      if (used > 1 && (int64_t)used * n_tok * n_out * 4 > kGemmSplitWsMaxBytes) break;
      const int64_t wgs = tiles * used, rest = wgs % kCUs;
      const double rounds = (double)(wgs / kCUs) + (rest > 0 ? 1.0 - tl.idle * (double)(kCUs - rest) / kCUs : 0.0);
      const double k_time = kts * tl.kt * (fused ? 1.0 + tl.fuse : 1.0) * rounds;
      double t = std::sqrt(k_time * k_time + read_w * read_w / std::min(1.0, wgs / kReadWgs)) + tl.first + (double)((wgs - 1) / kCUs) * tl.round;
      if (used > 1) t += kReduce + kPerSplit * used + (double)used * n_tok * n_out * 8 / kPartials;
      if (r_pad > 0 && !fused) t += kDown + rounds * (kTBase + kTArea * tl.bm * tl.bn / 65536) * r_pad / 16;
      if (best.tile < 0 || t < best_t * (1.0 - 1e-9)) {
        best = GemmPlan{i, used, used > 1 ? kts : 0};
        best_t = t;
      }
    }
  }
  if (n_tok <= kGemvMaxTok) {
    const double gemv_t = k_dim % 128 == 0 ? 4.0 + (1.45e-3 + 3.4e-5 * n_tok) * k_dim * ((n_out + 4095) / 4096)
                                           : 2.8 + 0.17 * n_tok + 4.4e-4 * n_out + k_dim * std::max(8.8e-5 * n_tok, 7.6e-7 * n_out);
    if (gemv_t <= best_t) best = GemmPlan{-1, 1, 0};
  }
  return best;
}

namespace {

hipError_t launch_gemm_any(const uint16_t* x, const uint16_t* w, int n_tok, int n_out, int hidden, const uint16_t* a,
                           float scale, const uint16_t* b, int rank, int r_pad, int lora_cols, const float* t_part,
                           GemmEpi epi, uint16_t* out, const GemmPlan& pl, float* split_ws, hipStream_t stream) {
  if (n_tok == 0) return hipSuccess;
  if (pl.tile < 0)
    return launch_gemv(x, w, n_tok, n_out, hidden, b, rank, r_pad, lora_cols, t_part, epi, out, stream);
  const int n_slice = lora_down_slices(hidden, n_tok);
  if (r_pad > 0 && t_part == nullptr && !gemm_fuses_lora(pl, r_pad)) return hipErrorInvalidValue;
  const int tiles = ((n_tok + kTiles[pl.tile].bm - 1) / kTiles[pl.tile].bm) * (n_out / kTiles[pl.tile].bn);
  // an fp32 result (not a split's partial) of the few-token tiles: the GEMV's
  // eight chains where that is what it would take, else no chain under 8 k-tiles
  const int n_kt = pl.n_split > 1 ? pl.kt_split : hidden / BK;
  const int part_kt = epi.mode == kEpiF32 ? std::max(n_tok <= kGemvMaxTok ? 1 : 8, (n_kt + 7) / 8) : 0;
  if (pl.n_split <= 1)
    return launch_tile(pl.tile, 0, tiles, x, w, n_tok, n_out, hidden, a, scale, b, rank, r_pad, lora_cols, t_part,
                       n_slice, epi, out, part_kt, stream);
  if (split_ws == nullptr || r_pad > 0) return hipErrorInvalidValue;
  const GemmEpi part{kEpiF32, nullptr, split_ws};
  hipError_t e = launch_tile(pl.tile, pl.kt_split, tiles * pl.n_split, x, w, n_tok, n_out, hidden, nullptr, 0.f,
                             nullptr, 0, 0, 0, nullptr, n_slice, part, nullptr, part_kt, stream);
  if (e != hipSuccess) return e;
  const int64_t quads = (int64_t)n_tok * n_out / 4;
  ATTUNER_LAUNCH("splitk_reduce_kernel", splitk_reduce_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), stream,
                 split_ws, pl.n_split, n_tok, n_out, epi, out);
  return hipGetLastError();
}

}  // namespace

// Tiles that keep their MFMAs busy would show the redundant down-projection
// (every feature tile of the adapted columns computes t for its tokens) in
// full: at 5368 tokens x 4096 -> 6144 (rank 16) a fusing 256 x 256 tile took
// 268 us against 244 us for lora_down_kernel + the GEMM reading t.  The
// smaller tiles hide it (1024 tokens, rank 32: 63.6 us fused, 67.4 separate).
bool gemm_fuses_lora(const GemmPlan& plan, int r_pad) {
  return plan.tile >= 0 && r_pad <= kGemmFusedLoraMaxRank && kTiles[plan.tile].fuse > 0;
}

hipError_t launch_gemm_lora(const uint16_t* x, const uint16_t* w, int n_tok, int n_out, int hidden,
                            const uint16_t* a, float scale, const uint16_t* b, int rank, int r_pad, int lora_cols,
                            const float* t_part, uint16_t* out, const GemmPlan& plan, hipStream_t stream) {
  return launch_gemm_any(x, w, n_tok, n_out, hidden, a, scale, b, rank, r_pad, lora_cols, t_part,
                         GemmEpi{kEpiBf16, nullptr, nullptr}, out, plan, nullptr, stream);
}

hipError_t launch_gemm(const uint16_t* x, const uint16_t* w, int n_tok, int n_out, int k_dim, GemmEpi epi,
                       uint16_t* out, const GemmPlan& plan, float* split_ws, hipStream_t stream) {
  return launch_gemm_any(x, w, n_tok, n_out, k_dim, nullptr, 0.f, nullptr, 0, 0, 0, nullptr, epi, out, plan,
                         split_ws, stream);
}

}  // namespace attuner
