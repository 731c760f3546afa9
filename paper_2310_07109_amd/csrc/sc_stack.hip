// Projections and normalisation of the attention-only encoder stack
// (SparseCoder, arXiv 2310.07109, Sec. 4.2 / Fig. 5: the encoder layer around
// the sparse attention; RoBERTa shapes).
//
// k_gemm_bf16   Y[rows, N] = X[rows, K] . W[K, N], bf16 operands, fp32
//               accumulation on v_mfma_f32_16x16x32_bf16.  Workgroup tile
//               128 x 128, 4 waves of 64 x 64, K step 32.  W is row-major
//               [K, N] (as stored by the caller), so its tile is transposed
//               while it is written to LDS to give each lane 8 consecutive k.
//               Rows of sequence b at or beyond len[b] are skipped: the GEMM
//               runs on the surviving tokens only.  Epilogue: bf16 store,
//               fp32 store, or GELU (x * Phi(x), erf by Abramowitz & Stegun 7.1.26) then bf16 store
//               for the first feed-forward product.
// k_gemm_v3     the same product when K % 32 == 0 and N % 128 == 0 (the
//               encoder's shapes), on packed rows: the surviving rows of all
//               sequences are numbered in order on the device (prefix sum of
//               the lengths) and cut into shared tiles, so that the product
//               runs on ceil(R / BM) tiles of the R surviving rows instead of
//               one partly empty tile per sequence.  Tiles of 256 x 128 rows x
//               columns once R >= 8192 (4 waves of 128 x 64, two stage
//               buffers), else 128 x 128 (4 waves of 64 x 64, three buffers):
//               48 KB either way, three workgroups per CU.  K stages of 32
//               arrive by gfx950's direct global->LDS loads.  X rows are stored
//               as 64-byte rows whose 16-byte units are XOR-swizzled by bits 2-3
//               of the row and read as 16-byte A fragments; W stays row-major
//               ([k][n], 256-byte rows, units swizzled by twice the row's low
//               3 bits) and the B fragments (8 consecutive k of one column) come
//               from transposing LDS reads (ds_read_b64_tr_b16).  Those reads
//               hand each lane the rows 4g..4g+3 and 16+4g..16+4g+3 of a 32-row
//               chunk, so W's rows are loaded into that order and the lane
//               receives k = 8g..8g+7.  Items (tile, N tile, K range) go to the
//               XCDs in contiguous ranges.
//               Split reduction for small float32 products: when the packed
//               rows fill few tiles (after pruning), S blocks per output tile
//               each take K / S of the reduction and write float32 partial
//               sums into slabs; the residual LayerNorm adds the slabs in the
//               fixed order s = 0 .. S-1.  Both kernels derive the packing and
//               S from the lengths, so the host needs no synchronisation.
// k_gemm_v4     the same product for calls of few rows (kV4Rows), laid out for
//               latency: see below.
// k_residual_ln y = bf16(LayerNorm(x + t)), one wavefront per packed row, fp32
//               statistics (biased variance), gamma = 1, beta = 0.
#include <algorithm>

#include "sc_device.h"
#include "sc_internal.h"

namespace sc {
namespace {

constexpr int kBM = 128, kBN = 128, kBKg = 32;
constexpr int kGPitch = kBKg + 8;  // 80-byte rows: 16 consecutive rows hit distinct banks

// GELU, x Phi(x) = x (1 + erf(x / sqrt 2)) / 2, with erfc(z) for z = |x| / sqrt 2
// from Abramowitz & Stegun, Handbook of Mathematical Functions, eq. 7.1.26
// (erfc(z) = (a1 t + ... + a5 t^5) exp(-z^2), t = 1 / (1 + p z), absolute
// error <= 1.5e-7): for x >= 0 the result is x (1 - erfc / 2), for x < 0
// x erfc / 2.  Evaluated in float32 it stays within 6e-7 of the exact GELU
// (1.7e-4 relative where |GELU| >= 1e-3), far inside the bf16 rounding of the
// stored activation; one reciprocal, one exponential and five FMAs instead
// of the library erff.
SC_DEV float gelu_exact(float v) {
  const float z = fabsf(v) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
  const float poly =
      t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
  const float ec = poly * fast_exp2(-z * z * kLog2e);
  return v >= 0.f ? v * fmaf(-0.5f, ec, 1.0f) : 0.5f * v * ec;
}

__global__ __launch_bounds__(256) void k_gemm_bf16(const __bf16* __restrict__ X, const __bf16* __restrict__ W,
                                                   void* __restrict__ Y, int mode, int n, int K, int N,
                                                   const int* __restrict__ len, const int* __restrict__ xidx) {
  __shared__ __attribute__((aligned(16))) __bf16 sX[kBM * kGPitch];
  __shared__ __attribute__((aligned(16))) __bf16 sW[kBN * kGPitch];  // transposed: [col][k]
  const int b = blockIdx.z;
  const int m0 = blockIdx.y * kBM, n0 = blockIdx.x * kBN;
  const int rows = len ? clampi(len[b], 0, n) : n;
  if (m0 >= rows) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, lr = lane & 15;
  const int wm = (w >> 1) * 64, wn = (w & 1) * 64;
  const __bf16* Xb = X + (long long)b * n * K;
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int k0 = 0; k0 < K; k0 += kBKg) {
    __syncthreads();
    // X tile: 128 rows x 4 chunks of 8
#pragma unroll
    for (int c = tid; c < kBM * 4; c += 256) {
      const int row = c >> 2, part = c & 3;
      const int m = m0 + row;
      __bf16* d = sX + row * kGPitch + 8 * part;
      if (m < rows && k0 + 8 * part < K)
        copy16(d, Xb + (long long)(xidx ? clampi(xidx[(long long)b * n + m], 0, n - 1) : m) * K + k0 + 8 * part);
      else
        zero16(d);
    }
    // W tile: 32 k-rows x 128 cols, two k-rows per thread, transposed
    {
      const int kp = tid >> 4, part = tid & 15;
      const int kk = k0 + 2 * kp, col = n0 + 8 * part;
      uint4 a = make_uint4(0, 0, 0, 0), c = make_uint4(0, 0, 0, 0);
      if (col < N) {
        if (kk < K) a = *reinterpret_cast<const uint4*>(W + (long long)kk * N + col);
        if (kk + 1 < K) c = *reinterpret_cast<const uint4*>(W + (long long)(kk + 1) * N + col);
      }
      const uint32_t av[4] = {a.x, a.y, a.z, a.w}, cv[4] = {c.x, c.y, c.z, c.w};
      uint32_t* base = reinterpret_cast<uint32_t*>(sW);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t lo = (av[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
        const uint32_t hi = (cv[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
        base[((8 * part + j) * kGPitch + 2 * kp) >> 1] = lo | (hi << 16);
      }
    }
    __syncthreads();
    bf16x8 af[4], bfr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) af[i] = *reinterpret_cast<const bf16x8*>(sX + (wm + 16 * i + lr) * kGPitch + 8 * g);
#pragma unroll
    for (int j = 0; j < 4; ++j) bfr[j] = *reinterpret_cast<const bf16x8*>(sW + (wn + 16 * j + lr) * kGPitch + 8 * g);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
  }
  // result (row wm + 16i + 4g + e, col wn + 16j + lr)
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + wm + 16 * i + 4 * g + e;
      if (m >= rows) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = n0 + wn + 16 * j + lr;
        if (col >= N) continue;
        const long long off = ((long long)b * n + m) * N + col;
        if (mode == kGemmF32)
          static_cast<float*>(Y)[off] = acc[i][j][e];
        else if (mode == kGemmGeluBf16)
          static_cast<__bf16*>(Y)[off] = (__bf16)gelu_exact(acc[i][j][e]);
        else
          static_cast<__bf16*>(Y)[off] = (__bf16)acc[i][j][e];
      }
    }
}

// ---------------------------------------------------------------------------
// Packed rows.  The surviving rows of all sequences are numbered in sequence
// order (packed row p of sequence b is its row p - pre[b], pre = exclusive
// prefix sum of the lengths), so that the products run on ceil(R / BM) tiles
// of R = sum of the lengths rows instead of one partly empty tile per
// sequence and 128 rows.  Every workgroup derives the numbering from the
// lengths itself: the host never learns them.

// Wave 0 writes pre[0 .. B] (pre[B] = R); lengths clamped to [0, n], all n
// without lengths.
SC_DEV void pack_prefix(int* pre, const int* len, int B, int n) {
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  int carry = 0;
  for (int c = 0; c < B; c += 64) {
    const int b = c + lane;
    const int v = b < B ? (len ? clampi(len[b], 0, n) : n) : 0;
    const int incl = prefix_sum(v);
    if (b < B) pre[b] = carry + incl - v;
    carry += __builtin_amdgcn_readlane(incl, 63);
  }
  if (lane == 0) pre[B] = carry;
}

// The sequence holding packed row p < pre[B]: the largest b with pre[b] <= p
// (empty sequences share their start with the next one).
SC_DEV int pack_seq(const int* pre, int B, int p) {
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Tiles of the packed product.  R rows in tiles of bm rows: 256 once the
// rows fill at least kBigRows (the taller tile's lower traffic per flop
// pays); 64 when the 64-row tiles of an unsplit product still fit one round
// of kOneRound workgroups (few rows: more, smaller tiles keep more CUs busy,
// and each CU pulls (64 + 128) / (128 + 128) of the bytes); 128 otherwise.
// Split reduction (float32 outputs with slabs only, 128-row tiles): S
// blocks per output tile each take K / S of the reduction; S doubles while
// the partial sums stay within kGemmSplitRows rows, the launch within
// kSplitBlocks workgroups and every range keeps at least 3 stages.  The
// product and the residual LayerNorm that adds its slabs compute the same
// plan from the same lengths.
constexpr int kBigRows = 8192, kOneRound = 256, kSplitMax = 8, kSplitBlocks = 1024;
struct GemmPlan {
  int bm, T, S;
};
SC_DEV GemmPlan gemm_plan(int R, int Nt, int nk, bool split) {
  GemmPlan p;
  p.S = 1;
  if (R >= kBigRows) {
    p.bm = 256;
    p.T = (R + 255) / 256;
    return p;
  }
  if (!split && (R + 63) / 64 * Nt <= kOneRound) {
    p.bm = 64;
    p.T = (R + 63) / 64;
    return p;
  }
  p.bm = 128;
  p.T = (R + 127) / 128;
  if (split)
    while (2 * p.S <= kSplitMax && p.T * 2 * p.S * 128 <= kGemmSplitRows && p.T * Nt * 2 * p.S <= kSplitBlocks &&
           nk % (2 * p.S) == 0 && nk / (2 * p.S) >= 3)
      p.S *= 2;
  return p;
}

// k per stage; W tile 32 x 128 per stage.
constexpr int kGK = 32;
constexpr int kXUnits = kGK / 8;  // 16-byte units per X row
constexpr int kStageBytes = 49152;  // stage buffers: 4 x (64 + 128), 3 x (128 + 128) or 2 x (256 + 128) x 32 bf16

// X rows of 4 units (32 k) swizzle by bits 2-3 of the row, so that 16
// consecutive rows read at one unit hit 16 distinct 16-byte bank groups
SC_DEV int gx_off(int row, int unit) { return row * kGK + 8 * (unit ^ ((row >> 2) & 3)); }
// s_waitcnt vmcnt(n) alone (expcnt and lgkmcnt at their no-wait maxima)
template <int N>
SC_DEV void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
SC_DEV int gw_off(int row, int unit) { return row * kBN + 8 * (unit ^ (2 * (row & 7))); }
// W row held by LDS row r of a stage: within each 32-row chunk, LDS row
// 4g + t holds k = 8g + t and LDS row 16 + 4g + t holds k = 8g + 4 + t.
SC_DEV int gw_krow(int r) { return (r & ~31) + 8 * ((r & 15) >> 2) + 4 * ((r >> 4) & 1) + (r & 3); }

// Four consecutive columns (off a multiple of 4).
template <int kMode>
SC_DEV void gemm_store4(void* Y, long long off, f32x4 v) {
  if constexpr (kMode == kGemmF32) {
    *reinterpret_cast<f32x4*>(static_cast<float*>(Y) + off) = v;
  } else {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (__bf16)(kMode == kGemmGeluBf16 ? gelu_exact(v[e]) : v[e]);
    *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(Y) + off) = o;
  }
}

// One output tile of BM x 128 (4 waves of BM/2 x 64, BM = 64, 128, 256) over this block's
// stages s0 .. s1-1, kNBuf stage buffers with kNBuf - 1 stages in flight;
// grow[r] = global row of tile row r (-1: past the packed rows), xrow[r] = the
// row of X it comes from (any valid row past the packed ones).  slab: the
// split's partial sums of this tile (row r at slab + r N), else NULL.
template <int BM, int kNBuf, int kMode>
SC_DEV void gemm_tile(const __bf16* __restrict__ X, const __bf16* __restrict__ W, void* __restrict__ Y,
                      char* stage, const int* grow, const int* xrow, int K, int N, int n0, int s0, int s1,
                      float* slab) {
  constexpr int FI = BM / 32;        // 16-row fragments per wave (wave tile BM/2 x 64)
  constexpr int XL = BM / 64;        // X loads per wave and stage (16 rows each)
  constexpr int kDmaPerStage = XL + 2;
  constexpr int kXBytes = BM * kGK * 2, kWBytes = kGK * kBN * 2;
  static_assert(kNBuf * (kXBytes + kWBytes) <= kStageBytes, "stage buffers");
  __bf16* sxb = reinterpret_cast<__bf16*>(stage);
  __bf16* swb = reinterpret_cast<__bf16*>(stage + kNBuf * kXBytes);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4,
            lr = lane & 15;
  const int wm = (w >> 1) * (BM / 2), wn = (w & 1) * 64;
  const unsigned xrow_b = 2u * (unsigned)K, wrow_b = 2u * (unsigned)N;  // byte offsets fit in 32 bits (host)
  // this lane's X rows
  unsigned xoff[XL];
#pragma unroll
  for (int t = 0; t < XL; ++t) {
    const int R = (BM / 4) * w + 16 * t + lane / kXUnits;
    xoff[t] = (unsigned)xrow[R] * xrow_b;
  }
  auto issue = [&](int k0, int bf) {
    const int ln = opaque_lane();
#pragma unroll
    for (int t = 0; t < XL; ++t) {  // X: wave w fills rows BM/4 w .. , 16 rows per load
      const int R0 = (BM / 4) * w + 16 * t, R = R0 + ln / kXUnits;
      const int u = (ln % kXUnits) ^ ((R >> 2) & 3);
      lds_dma16(X, xoff[t] + 2u * (unsigned)(k0 + 8 * u), lds_addr(sxb + (bf * BM + R0) * kGK));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {  // W: wave w fills rows 8w .., 4 rows per load
      const int R0 = 8 * w + 4 * t, R = R0 + (ln >> 4);
      const int u = (ln & 15) ^ (2 * (R & 7));
      lds_dma16(W, (unsigned)(k0 + gw_krow(R)) * wrow_b + 2u * (unsigned)(n0 + 8 * u),
                lds_addr(swb + (bf * kGK + R0) * kBN));
    }
  };
  f32x4 acc[FI][4];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int jn = 0; jn < 4; ++jn) acc[i][jn] = f32x4{0.f, 0.f, 0.f, 0.f};
  // stages s0 .. s0 + kNBuf - 2 in flight; stage s + kNBuf - 1 is issued into
  // the buffer read in stage s - 1 once the barrier of stage s has passed
#pragma unroll
  for (int p = 0; p < kNBuf - 1; ++p)
    if (s0 + p < s1) issue((s0 + p) * kGK, p);
  for (int s = s0; s < s1; ++s) {
    const int later = min(s1 - 1 - s, kNBuf - 2);  // stages issued after s, still in flight
    if constexpr (kNBuf == 4) {
      if (later >= 2) wait_vm<2 * kDmaPerStage>();
      else if (later == 1) wait_vm<kDmaPerStage>();
      else wait_vm<0>();
    } else if constexpr (kNBuf == 3) {
      if (later >= 1) wait_vm<kDmaPerStage>();
      else wait_vm<0>();
    } else {
      static_assert(kNBuf == 2, "two to four stage buffers");
      wait_vm<0>();
    }
    __syncthreads();
    if (s + kNBuf - 1 < s1) issue((s + kNBuf - 1) * kGK, (s - s0 + kNBuf - 1) % kNBuf);
    const int bf = (s - s0) % kNBuf;
    const __bf16* sx = sxb + bf * BM * kGK;
    const __bf16* sw = swb + bf * kGK * kBN;
    bf16x8 af[FI], bfr[4];
#pragma unroll
    for (int i = 0; i < FI; ++i) af[i] = *reinterpret_cast<const bf16x8*>(sx + gx_off(wm + 16 * i + lr, g));
    const int vr = 4 * g + (lr >> 2), bsel = (lr >> 1) & 1, e = 4 * (lr & 1);
#pragma unroll
    for (int jn = 0; jn < 4; ++jn) {
      const int U = 2 * ((wn >> 4) + jn) + bsel;
      const i16x4 a0 = lds_read_tr16(sw + gw_off(vr, U) + e);
      const i16x4 a1 = lds_read_tr16(sw + gw_off(vr + 16, U) + e);
      bfr[jn] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
    }
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int jn = 0; jn < 4; ++jn)
        acc[i][jn] = kMode == kGemmF32
                         ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[jn], acc[i][jn], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[jn], af[i], acc[i][jn], 0, 0, 0);
  }
  if constexpr (kMode == kGemmF32) {
    // result (tile row wm + 16i + 4g + e, col wn + 16jn + lr): 64-byte runs of
    // four rows per store.  (Staged through LDS like the bf16 results, W2 at
    // 12 288 rows took 98 us instead of 88; four columns of 16 rows per store
    // cost the whole layer 7 %.)
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = wm + 16 * i + 4 * g + e;
        const int gr = grow[r];
        if (gr < 0) continue;
        float* d = (slab ? slab + (long long)r * N : static_cast<float*>(Y) + (long long)gr * N) + n0 + wn + lr;
#pragma unroll
        for (int jn = 0; jn < 4; ++jn) d[16 * jn] = acc[i][jn][e];
      }
  } else {
    // W's fragment is the first operand, so that a lane holds four consecutive
    // columns of a row (row wm + 16i + lr, cols wn + 16jn + 4g ..).  The wave's
    // 64 columns go through its quarter of the stage buffers, kRows rows at a
    // time (16-byte units swizzled by the row), and leave as whole 128-byte
    // lines, 16 bytes a lane, instead of 2-byte stores of 32-byte runs: QKV at
    // 24 576 rows, D 768, 104.9 -> 100.4 us, W1 149.4 -> 143.8.
    constexpr int kRows = FI < 4 ? 32 : 64;
    static_assert(kRows * 128 <= kStageBytes / 4 && (BM / 2) % kRows == 0, "staging rows");
    char* st = stage + w * (kStageBytes / 4);
    __syncthreads();  // every wave has read the last stage
#pragma unroll
    for (int c = 0; c < BM / 2 / kRows; ++c) {
#pragma unroll
      for (int i = 0; i < kRows / 16; ++i)
#pragma unroll
        for (int jn = 0; jn < 4; ++jn) {
          const f32x4 v = acc[c * (kRows / 16) + i][jn];
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (__bf16)(kMode == kGemmGeluBf16 ? gelu_exact(v[e]) : v[e]);
          *reinterpret_cast<bf16x4*>(st + (16 * i + lr) * 128 + 16 * ((2 * jn + (g >> 1)) ^ (lr & 7)) + 8 * (g & 1)) = o;
        }
#pragma unroll
      for (int x = 0; x < kRows / 8; ++x) {
        const int row = 8 * x + (lane >> 3), gr = grow[wm + c * kRows + row];
        const uint4 v = *reinterpret_cast<const uint4*>(st + row * 128 + 16 * ((lane ^ row) & 7));
        if (gr < 0) continue;
        *reinterpret_cast<uint4*>(static_cast<__bf16*>(Y) + (long long)gr * N + n0 + wn + 8 * (lane & 7)) = v;
      }
    }
  }
}

// Y[row, N] = X[row, K] . W[K, N] over the surviving rows of the B
// sequences (row j of sequence b at b n + j, j < len[b]); with xidx, row j of
// sequence b reads X at row b n + xidx[b n + j] (the survivors of a pruning,
// not compacted).  part: float32
// slabs of a split reduction (kGemmF32 only), NULL for none.  Items (packed
// tile t, N tile, K range ks), ks fastest, are dealt to the XCDs in
// contiguous ranges (workgroup i runs on XCD i % 8): an XCD keeps its tiles'
// X rows in its L2 and sweeps the N tiles.
// At most 168 VGPRs: three waves per SIMD, which the three workgroups per
// CU that the stage buffers allow need.
template <int kMode>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_gemm_v3(
    const __bf16* __restrict__ X, const __bf16* __restrict__ W, void* __restrict__ Y, int B, int n, int K, int N,
    const int* __restrict__ len, const int* __restrict__ xidx, float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) char stage[kStageBytes];
  __shared__ int grow[256], xrow[256];
  int* pre = reinterpret_cast<int*>(stage);  // until the first stage lands
  pack_prefix(pre, len, B, n);
  __syncthreads();
  const int R = pre[B], Nt = N / kBN, nk = K / kGK;
  const GemmPlan pl = gemm_plan(R, Nt, nk, kMode == kGemmF32 && part != nullptr);
  const long long items = (long long)pl.T * Nt * pl.S;
  const int x = blockIdx.x & 7;
  const long long item = items * x / 8 + (blockIdx.x >> 3);
  if (item >= items * (x + 1) / 8) return;
  const int ks = (int)(item % pl.S), nt = (int)(item / pl.S % Nt), t = (int)(item / pl.S / Nt);
  const int m0 = t * pl.bm;
  if ((int)threadIdx.x < pl.bm) {
    const int p = min(m0 + (int)threadIdx.x, R - 1);  // rows past the packed ones read the last row
    const int b = pack_seq(pre, B, p);
    const int gr = b * n + (p - pre[b]);
    grow[threadIdx.x] = m0 + (int)threadIdx.x < R ? gr : -1;
    xrow[threadIdx.x] = xidx ? b * n + clampi(xidx[gr], 0, n - 1) : gr;
  }
  __syncthreads();  // the prefix table is dead from here: the stages overwrite it
  const int per = nk / pl.S, s0 = ks * per, s1 = s0 + per;
  float* slab = pl.S > 1 ? part + ((long long)ks * pl.T * 128 + m0) * N : nullptr;
  if (pl.bm == 256)
    gemm_tile<256, 2, kMode>(X, W, Y, stage, grow, xrow, K, N, nt * kBN, s0, s1, nullptr);
  else if (pl.bm == 128)
    gemm_tile<128, 3, kMode>(X, W, Y, stage, grow, xrow, K, N, nt * kBN, s0, s1, slab);
  else
    gemm_tile<64, 4, kMode>(X, W, Y, stage, grow, xrow, K, N, nt * kBN, s0, s1, nullptr);
}

// ---------------------------------------------------------------------------
// k_gemm_v4: the packed product for calls of few rows (kV4Rows, kV4Tiles).  Few rows
// make few tiles, and a tile's time is then the round trips of its loads, a
// microsecond or more each (the weights come from beyond the L2): k_gemm_v3
// keeps 36 KB of stages in flight per workgroup.  Here one workgroup of 512
// threads has a CU's LDS to itself, 144 KB of stage buffers all but one in
// flight, K stages of 64 (whole 128-byte rows of X), and tiles down to 64 x 64
// put more CUs to work.  One file of 512 tokens, D 768, FFN 3072, us per launch
// before -> after: QKV 15.0 -> 12.0, W1 16.3 -> 12.7, and with 64 rows left 14.2 ->
// 9.3 and 15.4 -> 8.8.
struct Plan4 {
  int mode, bm, T, Nt, S;
};
constexpr int kModes4 = 3;
constexpr int kBm4[kModes4] = {128, 64, 64}, kBn4[kModes4] = {128, 128, 64};
constexpr int kGK4 = 64;
constexpr int kStage4 = 147456;  // stage buffers: 4 x 32 KB, 6 x 24 KB or 9 x 16 KB
constexpr int kMaxB4 = 2048;     // sequences whose prefix table fits beside them
constexpr int kWgs4 = 256;       // one workgroup per CU, each taking items in turn
// Padded rows (B n), and 128 x 128 tiles of them, up to which k_gemm_v4 takes the
// product: at most two rounds of its workgroups.  us with k_gemm_v3 and v4,
// weights of 8 layers in turn, every row kept, tiles in brackets: QKV at D 768
// 1536 rows (216) 17.3 and 14.0, 2048 (288) 18.5 and 23.2, 4096 (576) 26.2 and 32.8;
// W1 there 1024 rows (192) 18.8 and 15.0, 2048 (384) 22.6 and 24.4, 4096 (768) 31.9
// and 37.1; Wo with its LayerNorm 4096 rows (192) 27.3 and 23.5, W2 42.4 and 39.0.
// Between one and two rounds v4 loses with every row kept and gains once a
// layer has pruned (the rows left are known on the device only): 12 layers of
// B1 n2048 D 1024 FFN 4096 with pruning, us with v3, v4 up to 256, 512 and any
// number of tiles: 1548, 1420, 1369, 1368; 4 unpruned layers of B4 n1024 there
// 772, -, 779, 838.  Larger tiles of this kernel (256 x 128, 256 x 256) did not beat
// k_gemm_v3's three workgroups per CU at 24 576 rows (620 against 572 per layer).
// A workgroup takes its CU's whole LDS, but several calls at once still gain:
// the 12-layer encoder of B1 n512 on 1, 2 and 4 streams 1106, 609 and 367 us per
// call with k_gemm_v3, 864, 504 and 340 with this kernel.
constexpr int kV4Rows = 4096, kV4Tiles = 2 * kWgs4;
// Hundredths of a microsecond of a K stage per mode, and of an item beside its
// stages, fitted to measured launches; the plan takes the cheapest mode and
// split by rounds x (stages x stage + 200).  Splits (float32 outputs with slabs)
// as in k_gemm_v3: S workgroups take K / S each, the LayerNorm adds the slabs,
// which costs it about 0.1 us per 1024 rows of slab.  The product and the
// LayerNorm price the plan each for itself, so it is priced in whole numbers:
// two modes may cost the same, and both kernels have to settle it alike.
SC_DEV int stage_cost4(int m) { return m == 0 ? 33 : m == 1 ? 21 : 15; }
SC_DEV Plan4 gemm_plan4(int R, int N, int nk, bool split) {
  // lane 4 m + s prices mode m with S = 2^s; the cheapest wins (ties: the lower lane)
  const int lane = threadIdx.x & 63, m = (lane >> 2) & 3, S = 1 << (lane & 3);
  const int bm = m == 0 ? 128 : 64, bn = m == 2 ? 64 : 128;
  const int T = (R + bm - 1) / bm, per = nk >> (lane & 3);
  bool ok = m < kModes4 && (N & (bn - 1)) == 0 && per >= 2 && per << (lane & 3) == nk;
  ok = ok && (S == 1 || split);
  ok = ok && (S == 1 || (long long)T * bm * S <= kGemmSplitRows);
  const int rounds = (T * (N / bn) * S + kWgs4 - 1) / kWgs4;
  // in eighths of a hundredth: 0.4 us per 4096 rows of slab are 5 per 64
  int t = 8 * rounds * (per * stage_cost4(m) + 200) + (S > 1 ? 5 * S * (T * bm / 64) : 0);
  if (!ok) t = 0x7fffffff;
  int best = lane & 15;
  auto meet = [&](int to, int bo) {
    const bool take = to < t || (to == t && bo < best);
    t = take ? to : t;
    best = take ? bo : best;
  };
  meet(dpp<kDppXor1>(t), dpp<kDppXor1>(best));
  meet(dpp<kDppXor2>(t), dpp<kDppXor2>(best));
  meet(dpp<kDppHalfMirror>(t), dpp<kDppHalfMirror>(best));
  meet(dpp<kDppMirror>(t), dpp<kDppMirror>(best));
  best = __builtin_amdgcn_readfirstlane(best);
  Plan4 p;
  p.mode = best >> 2;
  p.bm = p.mode == 0 ? 128 : 64;
  p.T = (R + p.bm - 1) / p.bm;
  p.Nt = N / (p.mode == 2 ? 64 : 128);
  p.S = 1 << (best & 3);
  return p;
}

// Row tables of packed tile t: the rows of Y it writes (-1: past the packed
// ones) and of X it reads (the last packed row past them).
SC_DEV void tile_rows4(int* grow, int* xrow, const int* pre, const int* xidx, int B, int n, int R, int m0, int bm) {
  if ((int)threadIdx.x >= bm) return;
  const int q = m0 + threadIdx.x, p = min(q, R - 1);
  const int b = pack_seq(pre, B, p);
  const int gr = b * n + (p - pre[b]);
  grow[threadIdx.x] = q < R ? gr : -1;
  xrow[threadIdx.x] = xidx ? b * n + clampi(xidx[gr], 0, n - 1) : gr;
}

// Waits until at most `later` (< kNBuf) stages of kPer loads are in flight.
template <int kNBuf, int kPer, int kL = kNBuf - 1>
SC_DEV void wait_stages(int later) {
  if constexpr (kL == 0) {
    wait_vm<0>();
  } else {
    if (later >= kL) wait_vm<kL * kPer>();
    else wait_stages<kNBuf, kPer, kL - 1>(later);
  }
}

template <int kM, int kMode>
SC_DEV void gemm_run4(const __bf16* __restrict__ X, const __bf16* __restrict__ W, void* __restrict__ Y, char* stage,
                      int* rows, const int* pre, const int* __restrict__ xidx, int B, int n, int R, int K, int N,
                      const Plan4& pl, float* part) {
  constexpr int BM = kBm4[kM], BN = kBn4[kM];
  constexpr int WGM = kM == 2 ? 4 : 2, WGN = 8 / WGM;  // waves along M and N
  constexpr int WM = BM / WGM, WN = BN / WGN, FI = WM / 16, FJ = WN / 16;
  constexpr int XL = BM / 64, WL = BN / 64;  // loads per wave and stage
  constexpr int kPer = XL + WL;
  constexpr int kXB = BM * kGK4 * 2, kWB = kGK4 * BN * 2;
  constexpr int kNBuf = kStage4 / (kXB + kWB);
  static_assert(kNBuf >= 2 && kNBuf <= 9, "stage buffers");
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4,
            lr = lane & 15;
  const int wm = (w / WGN) * WM, wn = (w % WGN) * WN;
  const int nk = K / kGK4, per = __builtin_amdgcn_readfirstlane(nk / pl.S);
  const int items = pl.T * pl.Nt * pl.S;
  const int xcd = blockIdx.x & 7, hi = (int)((long long)items * (xcd + 1) / 8);
  const int step = gridDim.x >> 3;
  int item = (int)((long long)items * xcd / 8) + (blockIdx.x >> 3);
  if (item >= hi) return;
  // this lane's W offset per load (stage k0 = 0, n0 = 0)
  constexpr int kUr = BN / 8, kRi = 64 / kUr;  // units per W row, rows per load
  constexpr int kWx = BN == 64 ? 1 : 2;        // W rows swizzle by kWx times their low 3 bits
  unsigned woff[WL];
#pragma unroll
  for (int t = 0; t < WL; ++t) {
    const int r = 8 * w + kRi * t + lane / kUr;
    woff[t] = (unsigned)gw_krow(r) * 2u * (unsigned)N + 16u * ((lane % kUr) ^ (kWx * (r & 7)));
  }
  unsigned xoff[XL];
  int n0 = 0, s0 = 0, cur = 0;
  const unsigned lds0 = lds_addr(stage);
  auto setup = [&](int it, int buf) {  // tables and offsets of an item (its tables' barrier included)
    const int ks = it % pl.S, nt = it / pl.S % pl.Nt, t = it / pl.S / pl.Nt;
    int* grow = rows + 512 * buf;
    tile_rows4(grow, grow + 256, pre, xidx, B, n, R, __builtin_amdgcn_readfirstlane(t * BM), BM);
    n0 = __builtin_amdgcn_readfirstlane(nt * BN);
    s0 = __builtin_amdgcn_readfirstlane(ks * per);
    __syncthreads();
#pragma unroll
    for (int x = 0; x < XL; ++x)
      xoff[x] = (unsigned)grow[256 + (BM / 8) * w + 8 * x + (lane >> 3)] * 2u * (unsigned)K +
                16u * ((lane & 7) ^ (lane >> 3));
  };
  auto issue = [&](int s, int bf) {  // stage s of the item into buffer bf
    const __bf16* xb = X + (size_t)(s0 + s) * kGK4;
    const __bf16* wb = W + (size_t)(s0 + s) * kGK4 * N + n0;
    const unsigned lx = lds0 + (unsigned)bf * (kXB + kWB), lw = lx + kXB;
#pragma unroll
    for (int x = 0; x < XL; ++x) lds_dma16(xb, xoff[x], lx + ((BM / 8) * w + 8 * x) * 128u);
#pragma unroll
    for (int t = 0; t < WL; ++t) lds_dma16(wb, woff[t], lw + (8 * w + kRi * t) * (2u * BN));
  };
  // LDS addresses of the lane's fragments in buffer 0: A (unit of k-chunk kc:
  // xor 64 kc), B (row chunk kc: + 32 rows)
  const unsigned aa = lds0 + (wm + lr) * 128u + 16u * (g ^ (lr & 7));
  const int vr = 4 * g + (lr >> 2);
  unsigned ba[FJ];
#pragma unroll
  for (int j = 0; j < FJ; ++j)
    ba[j] = lds0 + kXB + vr * (2u * BN) + 16u * ((2 * ((wn >> 4) + j) + ((lr >> 1) & 1)) ^ (kWx * (vr & 7))) + 8u * (lr & 1);
  bf16x8 af[2][FI], bq[2][FJ];  // fragments of the two k-chunks of 32
  auto frags = [&](unsigned ob, int kc) {
#pragma unroll
    for (int j = 0; j < FJ; ++j) {
      const i16x4 a0 = lds_read_tr16(ba[j] + ob + 32u * kc * (2u * BN));
      const i16x4 a1 = lds_read_tr16(ba[j] + ob + (32u * kc + 16u) * (2u * BN));
      bq[kc][j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
    }
#pragma unroll
    for (int i = 0; i < FI; ++i) af[kc][i] = lds_read16((aa ^ (64u * kc)) + ob + i * 2048u);
  };
  setup(item, cur);
#pragma unroll
  for (int p = 0; p < kNBuf; ++p)
    if (p < per) issue(p, p);
  wait_stages<kNBuf, kPer>(min(per, kNBuf) - 1);
  while (true) {
    f32x4 acc[FI][FJ];
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int j = 0; j < FJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](int kc) {
#pragma unroll
      for (int i = 0; i < FI; ++i)
#pragma unroll
        for (int j = 0; j < FJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bq[kc][j], af[kc][i], acc[i][j], 0, 0, 0);
    };
    // One barrier per stage, between its two k-chunks: the second chunk's
    // fragments are in flight during the first chunk's products, the next
    // stage's first ones during the second's, and a stage's buffer is
    // refilled as soon as every wave has read it.
    __syncthreads();
    int bf = 0;
    frags(0u, 0);
    for (int s = 0; s < per; ++s) {
      const int bn = bf == kNBuf - 1 ? 0 : bf + 1;
      frags((unsigned)bf * (kXB + kWB), 1);
      mul(0);
      if (s + 1 < per) {
        wait_stages<kNBuf, kPer>(min(per - 2 - s, kNBuf - 2));
        __syncthreads();
        if (s + kNBuf < per) issue(s + kNBuf, bf);
        frags((unsigned)bn * (kXB + kWB), 0);
      }
      mul(1);
      bf = bn;
    }
    // the next item's first stages load while this item's results are stored
    const int on0 = n0, ot = item / pl.S / pl.Nt, oks = item % pl.S, ocur = cur;
    item += step;
    const bool more = item < hi;
    __syncthreads();  // every wave has read the last stage
    if (more) {
      cur ^= 1;
      setup(item, cur);
#pragma unroll
      for (int p = 0; p < kNBuf; ++p)
        if (p < per) issue(p, p);
    }
    const int* grow = rows + 512 * ocur;
    float* slab = pl.S > 1 ? part + ((size_t)oks * pl.T * BM + (size_t)ot * BM) * N : nullptr;
#pragma unroll
    for (int i = 0; i < FI; ++i) {
      const int r = wm + 16 * i + lr, gr = grow[r];
      if (gr >= 0) {
        const int col = on0 + wn + 4 * g;
#pragma unroll
        for (int j = 0; j < FJ; ++j) {
          if (slab)
            *reinterpret_cast<f32x4*>(slab + (size_t)r * N + col + 16 * j) = acc[i][j];
          else
            gemm_store4<kMode>(Y, (long long)gr * N + col + 16 * j, acc[i][j]);
        }
      }
    }
    if (!more) break;
    wait_vm<0>();  // the next item's first stages, and the stores, which share the counter
  }
}

template <int kMode>
__global__ __launch_bounds__(512) void k_gemm_v4(const __bf16* __restrict__ X, const __bf16* __restrict__ W,
                                                 void* __restrict__ Y, int B, int n, int K, int N,
                                                 const int* __restrict__ len, const int* __restrict__ xidx,
                                                 float* __restrict__ part) {
  __shared__ __attribute__((aligned(1024))) char sm4[kStage4];
  __shared__ int rows[1024], pre[kMaxB4 + 1];  // two pairs of row tables; prefix table
  pack_prefix(pre, len, B, n);
  __syncthreads();
  const int R = __builtin_amdgcn_readfirstlane(pre[B]);
  if (R == 0) return;
  const Plan4 pl = gemm_plan4(R, N, K / kGK4, kMode == kGemmF32 && part != nullptr);
  if (pl.mode == 0)
    gemm_run4<0, kMode>(X, W, Y, sm4, rows, pre, xidx, B, n, R, K, N, pl, part);
  else if (pl.mode == 1)
    gemm_run4<1, kMode>(X, W, Y, sm4, rows, pre, xidx, B, n, R, K, N, pl, part);
  else
    gemm_run4<2, kMode>(X, W, Y, sm4, rows, pre, xidx, B, n, R, K, N, pl, part);
}

// v[4u + q] = x[c + q] + t[c + q] for the columns c = 4 lane + 256 u .. +3
// (D a multiple of 64), t being the sum of S partial sums that lie `stride`
// floats apart, added in the order s = 0 .. S-1; 16-byte loads of t.
template <int S, int kPer>
SC_DEV void ln_load(float (&v)[kPer], const __bf16* xp, const float* tp, long long stride, int D, int lane) {
#pragma unroll
  for (int u = 0; u < kPer / 4; ++u) {
    const int c = 4 * lane + 256 * u;
    if (c < D) {
      float4 a = *reinterpret_cast<const float4*>(tp + c);
#pragma unroll
      for (int k = 1; k < S; ++k) {
        const float4 e = *reinterpret_cast<const float4*>(tp + k * stride + c);
        a.x += e.x;
        a.y += e.y;
        a.z += e.z;
        a.w += e.w;
      }
      const bf16x4 xv = *reinterpret_cast<const bf16x4*>(xp + c);
      v[4 * u] = a.x + (float)xv[0];
      v[4 * u + 1] = a.y + (float)xv[1];
      v[4 * u + 2] = a.z + (float)xv[2];
      v[4 * u + 3] = a.w + (float)xv[3];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[4 * u + q] = 0.f;
    }
  }
}

// One row of the residual LayerNorm: y = bf16(LayerNorm(x + t)) at global
// row `row`, packed index p (where a split product left its partial sums), x
// being row xrow of xr.
template <int kMaxPer>
SC_DEV void ln_row(const __bf16* __restrict__ xr, const float* __restrict__ t, __bf16* __restrict__ y, int D,
                   float eps, const float* __restrict__ part, int S, long long srows, long long row, long long xrow,
                   int p, int lane) {
  const __bf16* xp = xr + xrow * D;
  __bf16* yp = y + row * D;
  float v[kMaxPer];
  if (S == 1) {
    ln_load<1, kMaxPer>(v, xp, t + row * D, 0, D, lane);
  } else {  // the row's partial sums sit at its packed index in each slab
    const float* tp = part + (long long)p * D;
    const long long stride = srows * D;
    if (S == 2)
      ln_load<2, kMaxPer>(v, xp, tp, stride, D, lane);
    else if (S == 4)
      ln_load<4, kMaxPer>(v, xp, tp, stride, D, lane);
    else
      ln_load<8, kMaxPer>(v, xp, tp, stride, D, lane);
  }
  float s = 0.f;
#pragma unroll
  for (int u = 0; u < kMaxPer; ++u) s += v[u];
  s = butterfly_sum(s);
  const float mean = s / (float)D;
  float q = 0.f;
#pragma unroll
  for (int u = 0; u < kMaxPer; ++u) {
    const int c = 4 * lane + 256 * (u / 4);
    const float dv = c < D ? v[u] - mean : 0.f;
    q += dv * dv;
  }
  q = butterfly_sum(q);
  const float inv = 1.0f / sqrtf(q / (float)D + eps);
#pragma unroll
  for (int u = 0; u < kMaxPer / 4; ++u) {
    const int c = 4 * lane + 256 * u;
    if (256 * u < D && c < D) {
      bf16x4 o;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) o[q4] = (__bf16)((v[4 * u + q4] - mean) * inv);
      *reinterpret_cast<bf16x4*>(yp + c) = o;
    }
  }
}

// part, K: the slabs and reduction length of the product that wrote t, when
// it may have split its reduction (t itself is then unused).  One wavefront
// per packed row, rows dealt round-robin over the launch's waves.  kMaxPer =
// elements per lane (D <= 64 kMaxPer).  pre: dynamic LDS of B + 1 ints.
template <int kMaxPer>
__global__ __launch_bounds__(256) void k_residual_ln(const __bf16* __restrict__ xr, const float* __restrict__ t,
                                                     __bf16* __restrict__ y, int B, int n, int D, float eps,
                                                     const int* __restrict__ len, const int* __restrict__ xidx,
                                                     const float* __restrict__ part, int K, int v4) {
  extern __shared__ int pre[];
  pack_prefix(pre, len, B, n);
  __syncthreads();
  const int R = pre[B];
  const int lane = threadIdx.x & 63;
  // ranges of the product's split, and rows per slab
  int S = 1, srows = 0;
  if (v4) {
    const Plan4 pl = gemm_plan4(max(R, 1), D, K / kGK4, part != nullptr);
    S = pl.S;
    srows = pl.T * pl.bm;
  } else {
    const GemmPlan pl = gemm_plan(R, D / kBN, K / kGK, part != nullptr);
    S = pl.S;
    srows = pl.T * 128;
  }
  for (int p = blockIdx.x * 4 + (threadIdx.x >> 6); p < R; p += gridDim.x * 4) {
    const int b = pack_seq(pre, B, p);
    const long long row = (long long)b * n + (p - pre[b]);
    const long long xrow = xidx ? (long long)b * n + clampi(xidx[row], 0, n - 1) : row;
    ln_row<kMaxPer>(xr, t, y, D, eps, part, S, srows, row, xrow, p, lane);
  }
}

}  // namespace

namespace {
// Shapes of the packed product: K and N whole stages and tiles, 32-bit byte
// offsets over all B n rows of X and over W, the prefix table in the stage
// buffers.
bool gemm_v3_ok(int B, int n, int K, int N) {
  return K % kGK == 0 && N % kBN == 0 && K > 0 && N > 0 && B <= kPackMaxB &&
         (long long)B * n * K * 2 < (1LL << 32) && (long long)K * N * 2 < (1LL << 32);
}
}  // namespace

// Shapes of k_gemm_v4: as k_gemm_v3 with K whole stages of 64 (two at least),
// few rows, and a batch whose prefix table fits beside the stage buffers.
static bool gemm_v4_ok(int B, int n, int K, int N) {
  return gemm_v3_ok(B, n, K, N) && K % kGK4 == 0 && K >= 2 * kGK4 && B <= kMaxB4 && (long long)B * n <= kV4Rows &&
         ((long long)B * n + 127) / 128 * (N / kBN) <= kV4Tiles;
}

template <int kMode>
static hipError_t launch_v4(const __bf16* x, const __bf16* w, void* y, int B, int n, int K, int N, const int* len,
                            const int* xidx, float* part, hipStream_t s) {
  hipLaunchKernelGGL(k_gemm_v4<kMode>, dim3(kWgs4), dim3(512), 0, s, x, w, y, B, n, K, N, len, xidx, part);
  return hipGetLastError();
}

hipError_t launch_gemm_bf16(const void* x, const void* w, void* y, int mode, int B, int n, int K, int N,
                            const int* len, const int* xidx, float* part, hipStream_t s) {
  if (gemm_v4_ok(B, n, K, N)) {
    const __bf16* xb = static_cast<const __bf16*>(x);
    const __bf16* wb = static_cast<const __bf16*>(w);
    if (mode == kGemmF32) return launch_v4<kGemmF32>(xb, wb, y, B, n, K, N, len, xidx, part, s);
    if (mode == kGemmGeluBf16) return launch_v4<kGemmGeluBf16>(xb, wb, y, B, n, K, N, len, xidx, nullptr, s);
    return launch_v4<kGemmBf16>(xb, wb, y, B, n, K, N, len, xidx, nullptr, s);
  }
  if (gemm_v3_ok(B, n, K, N)) {
    // items: at most ceil(B n / 128) 128-row tiles x N tiles, kSplitBlocks for
    // a split, kOneRound for 64-row tiles
    const long long tiles = ((long long)B * n + 127) / 128 * (N / kBN);
    if (!(part && mode == kGemmF32)) part = nullptr;
    const long long items = std::max<long long>(tiles, part ? kSplitBlocks : kOneRound);
    const dim3 grid((unsigned)(8 * ((items + 7) / 8))), block(256);
    const __bf16* xb = static_cast<const __bf16*>(x);
    const __bf16* wb = static_cast<const __bf16*>(w);
    if (mode == kGemmF32)
      hipLaunchKernelGGL(k_gemm_v3<kGemmF32>, grid, block, 0, s, xb, wb, y, B, n, K, N, len, xidx, part);
    else if (mode == kGemmGeluBf16)
      hipLaunchKernelGGL(k_gemm_v3<kGemmGeluBf16>, grid, block, 0, s, xb, wb, y, B, n, K, N, len, xidx, nullptr);
    else
      hipLaunchKernelGGL(k_gemm_v3<kGemmBf16>, grid, block, 0, s, xb, wb, y, B, n, K, N, len, xidx, nullptr);
    return hipGetLastError();
  }
  dim3 grid((N + kBN - 1) / kBN, (n + kBM - 1) / kBM, B);
  hipLaunchKernelGGL(k_gemm_bf16, grid, dim3(256), 0, s, static_cast<const __bf16*>(x),
                     static_cast<const __bf16*>(w), y, mode, n, K, N, len, xidx);
  return hipGetLastError();
}

hipError_t launch_residual_layernorm(const void* x_res, const float* t, void* y, int B, int n, int D, float eps,
                                     const int* len, const int* xidx, const float* part, int K, hipStream_t s) {
  const long long rows = (long long)B * n;
  if (!gemm_v3_ok(B, n, K, D)) part = nullptr;  // the product took the path without a split
  auto* kern = D <= 1024 ? k_residual_ln<16> : k_residual_ln<32>;  // D <= 2048 (checked by the caller)
  // one wave per row, at most 1024 workgroups (later rows loop; with the
  // grid sized by the lengths' upper bound n, a pruned layer's few rows would
  // otherwise come with thousands of workgroups that only build the prefix
  // table: 7.5 -> 6.3 us in the stack's late layers)
  const long long blocks = std::min<long long>((rows + 3) / 4, 1024);
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), sizeof(int) * (B + 1), s,
                     static_cast<const __bf16*>(x_res), t, static_cast<__bf16*>(y), B, n, D, eps, len, xidx, part, K,
                     gemm_v4_ok(B, n, K, D) ? 1 : 0);
  return hipGetLastError();
}

}  // namespace sc
