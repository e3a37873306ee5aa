// bf16 matrix products of wide models (d = 512), where a row tile can no longer afford to stream a
// whole weight matrix through its compute unit:
//   C = epi(A W + bias),  A [R][K] bf16 (row stride lda), W packed in the fragment order of
//   v_mfma_f32_32x32x16_bf16 (block (nb, ks) = output columns 32nb.., inputs 16ks..; 1 KiB, lane l
//   holding W[16ks + 8(l/32) + j][32nb + l%32]).
// Products are formed transposed (C^T = W^T A^T) as in the other kernels, so a lane holds four
// consecutive output columns of one row.  Epilogues: bf16 store (+ bias, optional ReLU), or fp32
// residual add (the residual fp32 or bf16; it may alias the output).  Rows >= R and padding rows
// (r % rows_per_batch >= nvalid[r / rows_per_batch]) are not stored; their A rows are read from
// the tile's first row instead.
#include <type_traits>

#include "fe_common.h"

namespace {

// ------------------------------------------------------------------------------------------
// 64 x 128 output tiles, four waves of 64 x 32.
//
// A wave owns its 32 output columns for every row of the tile, so each weight fragment is read by
// exactly one wave and goes straight from memory to its registers (1 KiB, fully coalesced); only
// A passes through LDS, which the matrix units would otherwise wait for: with both operands in LDS
// and 32 x 64 per wave, a 16-deep step read 12 KiB of LDS (96 cycles at 128 B/clk) for 64 cycles
// of products.  A is staged 64 columns at a time as whole 128-byte row segments: eight lanes a
// row, 16-byte segment g of row r at position g ^ ((r / 2) % 8), which leaves both the writes and
// the fragment reads free of bank conflicts.  The rows go through registers and not through the
// direct LDS load: the compiler waits for every outstanding LDS copy before the next LDS read,
// which put a whole memory latency into each stage.  Rows are requested two stages and weights one
// stage ahead, in loops without branches, so that every wait counts only what it needs.  The
// output leaves through LDS as 64-byte (bf16) or 128-byte (fp32) row segments; stored from the
// accumulators it made one 16-byte write request per row and four columns.
//
// Bound by: the latency of the weight loads at few tiles, matrix issue and L2 at many (124 VGPRs:
// four workgroups per compute unit).  R = 8192, one MI355X, before (64 x 128 tiles, both operands
// by direct LDS load) -> now: K 512 N 1536 33.9 -> 20.4 us (633 TFLOP/s); K 512 N 2048 41.3 -> 24.3;
// K 2048 N 512 34.6 -> 26.4; K 512 N 512 16.2 -> 11.1; K 512 N 4096 83.1 -> 55.0.  Tiles of 128 x
// 128, 64 x 256 (2 workgroups per compute unit) and 128 x 256 were 5-15% slower at these sizes.
// ------------------------------------------------------------------------------------------
constexpr int BK = 64, KSS = BK / 16, RBW = 2, NW = 4, BM = 32 * RBW, BN = 32 * NW;

template <int EPI>
__global__ __launch_bounds__(64 * NW, 4) void k_gemm_tiled(GemmArgs a) {
  constexpr int SA = BM * BK, DPW = BM / 8 / NW;          // elements of a stage; row loads per lane and stage
  constexpr int SLD = EPI == EPI_RESID ? 32 + 4 : 32 + 8, ESZ = EPI == EPI_RESID ? 4 : 2;
  constexpr int STG = NW * 32 * SLD * ESZ / 2, SMEM = STG > 2 * SA ? STG : 2 * SA;
  __shared__ __attribute__((aligned(16))) bf16 smem[SMEM];
  __shared__ int s_valid[BM];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_nt = a.N / BN, id = xcd_tile(blockIdx.x, gridDim.x);
  const int mt = id / n_nt, nt = id % n_nt;             // column tiles vary fastest: an XCD's rows of A stay in its L2
  const int row0 = mt * BM, cb = nt * NW + wave;        // cb: this wave's 32-column block
  const int KS = a.K / 16, nst = a.K / BK;

  int v = 0;
  if (threadIdx.x < BM) {
    const int r = row0 + threadIdx.x;
    v = r < a.R;
    if (v && a.nvalid) v = (r % a.rows_per_batch) < a.nvalid[r / a.rows_per_batch];
    s_valid[threadIdx.x] = v;
  }
  if (!block_any<NW>(v)) return;                        // a tile made only of padding rows

  if (a.zero && blockIdx.x == 0)
    for (int i = threadIdx.x; i < a.zero_n; i += 64 * NW) a.zero[i] = 0;
  const bf16* src[DPW];
  int dst[DPW];
#pragma unroll
  for (int i = 0; i < DPW; ++i) {
    const int rr = (wave * DPW + i) * 8 + (lane >> 3);
    src[i] = static_cast<const bf16*>(a.A) + (long long)(s_valid[rr] ? row0 + rr : row0) * a.lda + (lane & 7) * 8;
    dst[i] = rr * BK + (((lane & 7) ^ ((rr >> 1) & 7)) * 8);
  }
  auto load_rows = [&](bf16x8 (&r)[DPW], int s) {
#pragma unroll
    for (int i = 0; i < DPW; ++i) r[i] = *reinterpret_cast<const bf16x8*>(src[i] + s * BK);
  };
  auto put_rows = [&](const bf16x8 (&r)[DPW], int s) {
#pragma unroll
    for (int i = 0; i < DPW; ++i) *reinterpret_cast<bf16x8*>(smem + (s & 1) * SA + dst[i]) = r[i];
  };
  const bf16x8* Wl = static_cast<const bf16x8*>(a.Wt) + (long long)cb * KS * 64 + lane;
  auto load_w = [&](bf16x8 (&w)[KSS], int s) {
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk) w[kk] = Wl[(s * KSS + kk) * 64];
  };
  f32x16 acc[RBW];
#pragma unroll
  for (int i = 0; i < RBW; ++i) acc[i] = f32x16{};

  // Stage s: its rows are in LDS buffer s & 1, its weights in wc and the rows of stage s + 1 in rc.
  // left: how many stages follow (0, 1, or 2 for "at least two").  Buffer (s + 1) & 1, written at
  // the end, was last read in stage s - 1, before that stage's barrier.
  auto stage = [&](int s, bf16x8 (&wc)[KSS], bf16x8 (&wx)[KSS], bf16x8 (&rc)[DPW], bf16x8 (&rx)[DPW], auto left_) {
    constexpr int left = decltype(left_)::value;
    if constexpr (left > 0) load_w(wx, s + 1);
    if constexpr (left > 1) load_rows(rx, s + 2);
    const bf16* buf = smem + (s & 1) * SA;
    bf16x8 af[2][RBW];
    auto load_a = [&](int kk) {
#pragma unroll
      for (int i = 0; i < RBW; ++i)
        af[kk & 1][i] = *reinterpret_cast<const bf16x8*>(
            buf + (i * 32 + (lane & 31)) * BK + (((2 * kk + (lane >> 5)) ^ ((lane >> 1) & 7)) * 8));
    };
    __builtin_amdgcn_sched_barrier(0);                  // the requests above go out first
    load_a(0);
#pragma unroll
    for (int kk = 0; kk < KSS; ++kk) {
      if (kk + 1 < KSS) load_a(kk + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < RBW; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wc[kk], af[kk & 1][i], acc[i], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (left > 0) put_rows(rc, s + 1);
    lds_barrier();
  };
  using More = std::integral_constant<int, 2>;
  bf16x8 w0[KSS], w1[KSS], r0[DPW], r1[DPW];            // nst is even and at least 2
  load_rows(r0, 0);
  load_w(w0, 0);
  load_rows(r1, 1);
  put_rows(r0, 0);
  lds_barrier();
  for (int s = 0; s < nst - 2; s += 2) {
    stage(s, w0, w1, r1, r0, More{});
    stage(s + 1, w1, w0, r0, r1, More{});
  }
  stage(nst - 2, w0, w1, r1, r0, std::integral_constant<int, 1>{});
  stage(nst - 1, w1, w0, r0, r1, std::integral_constant<int, 0>{});

  // Epilogue, one 32-row block at a time through this wave's part of smem (past the last barrier
  // nobody reads the stages any more): written as the accumulators lie (lane holds row lane % 32,
  // columns 8q + 4 (lane / 32) + e), read back as whole row segments.
  char* st = reinterpret_cast<char*>(smem) + wave * 32 * SLD * ESZ;
  const int n0 = cb * 32;
  if constexpr (EPI == EPI_RESID) {
    float* sf = reinterpret_cast<float*>(st);
    const int c4 = (lane & 7) * 4;
    const float4 bb = a.bias ? *reinterpret_cast<const float4*>(a.bias + n0 + c4) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(&sf[(lane & 31) * SLD + 8 * q + 4 * (lane >> 5)]) =
            make_float4(acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int rr = it * 8 + (lane >> 3);
        if (!s_valid[i * 32 + rr]) continue;
        const long long r = row0 + i * 32 + rr;
        const float4 o = *reinterpret_cast<const float4*>(&sf[rr * SLD + c4]);
        float4 rv;
        if (a.res_f32) {
          rv = *reinterpret_cast<const float4*>(static_cast<const float*>(a.res) + r * a.ldr + n0 + c4);
        } else {
          const bf16x4 t = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(a.res) + r * a.ldr + n0 + c4);
          rv = make_float4((float)t[0], (float)t[1], (float)t[2], (float)t[3]);
        }
        *reinterpret_cast<float4*>(static_cast<float*>(a.C) + r * a.ldc + n0 + c4) =
            make_float4(rv.x + (o.x + bb.x), rv.y + (o.y + bb.y), rv.z + (o.z + bb.z), rv.w + (o.w + bb.w));
      }
      __builtin_amdgcn_wave_barrier();
    }
  } else {
    bf16* sh = reinterpret_cast<bf16*>(st);
    float4 bb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      bb[q] = a.bias ? *reinterpret_cast<const float4*>(a.bias + n0 + 8 * q + 4 * (lane >> 5)) : make_float4(0.f, 0.f, 0.f, 0.f);
    const int c8 = (lane & 3) * 8;                       // a 32-column block lies within one column slab (col_block % 32 == 0)
    bf16* y = static_cast<bf16*>(a.C) + (long long)(n0 / a.col_block) * a.col_block_stride + n0 % a.col_block + c8;
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float o0 = acc[i][4 * q] + bb[q].x, o1 = acc[i][4 * q + 1] + bb[q].y;
        float o2 = acc[i][4 * q + 2] + bb[q].z, o3 = acc[i][4 * q + 3] + bb[q].w;
        if constexpr (EPI == EPI_RELU) {
          o0 = fmaxf(o0, 0.f); o1 = fmaxf(o1, 0.f); o2 = fmaxf(o2, 0.f); o3 = fmaxf(o3, 0.f);
        }
        bf16x4 o;
        o[0] = (bf16)o0; o[1] = (bf16)o1; o[2] = (bf16)o2; o[3] = (bf16)o3;
        *reinterpret_cast<bf16x4*>(&sh[(lane & 31) * SLD + 8 * q + 4 * (lane >> 5)]) = o;
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int rr = it * 16 + (lane >> 2);
        if (s_valid[i * 32 + rr])
          *reinterpret_cast<bf16x8*>(y + (long long)(row0 + i * 32 + rr) * a.ldc) = *reinterpret_cast<const bf16x8*>(&sh[rr * SLD + c8]);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// ------------------------------------------------------------------------------------------
// Products of few rows (the cross-sequence set of a text batch: B K = 128 rows): one wave per 32 x 32
// block, K in the order of the tiles above, so that a row's result is the same however many rows
// share the launch.
//
// Bound by latency: at 128 rows a product has a few dozen tiles, and a tiled loop of K / 64 stages
// waits for memory once a stage.  Here both operands go straight to registers, four batches of eight
// 16-deep steps in flight, after the bias and residual that the epilogue adds.
// R = 128, 64 x 64 tiles through LDS -> this kernel: K 512 N 512 5.9 -> 3.4 us, K 512 N 2048 6.0 ->
// 3.4, K 2048 N 512 12.9 -> 6.6.  Four waves per block, each over a quarter of K with the parts added
// in LDS, took 3.5, 3.7 and 6.7 us, and their sums differ from the tiles'.
// ------------------------------------------------------------------------------------------
template <int EPI>
__global__ __launch_bounds__(64) void k_gemm_thin(GemmArgs a) {
  constexpr int NB = 8, NBUF = 4;                        // 16-deep steps per batch of loads; batches in flight
  const int lane = threadIdx.x;
  const int n_nt = a.N / 32, id = xcd_tile(blockIdx.x, gridDim.x);
  const int row0 = (id / n_nt) * 32, nt = id % n_nt, row = row0 + (lane & 31);
  bool ok = row < a.R;
  if (ok && a.nvalid) ok = (row % a.rows_per_batch) < a.nvalid[row / a.rows_per_batch];
  if (!__any(ok)) return;
  if (a.zero && blockIdx.x == 0)
    for (int i = lane; i < a.zero_n; i += 64) a.zero[i] = 0;
  const int nb = a.K / (16 * NB);                        // at least 1: K is a multiple of 128
  // Batches past the last get offsets past the buffers (zeros, no traffic), so that no branch separates
  // the loads and every wait counts only the batch it needs.
  const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(static_cast<const bf16*>(a.A)) + (long long)row0 * a.lda, 0,
                                                    32 * a.lda * 2, 0x00027000);
  const auto rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(static_cast<const bf16*>(a.Wt)) + (long long)nt * a.K * 32, 0,
                                                    a.K * 32 * 2, 0x00027000);
  constexpr unsigned OUT = 0x80000000u;
  const unsigned a0 = ((ok ? row - row0 : 0) * a.lda + 8 * (lane >> 5)) * 2u, w0 = lane * 16u;
  // what the epilogue adds (the lane holds columns n0 + 8q + 0..3 of its row), requested first of all
  const int n0 = nt * 32 + 4 * (lane >> 5);
  f32x4 bias[4], res[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    bias[q] = a.bias ? *reinterpret_cast<const f32x4*>(a.bias + n0 + 8 * q) : f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (EPI == EPI_RESID) {
      const long long at = (long long)(ok ? row : row0) * a.ldr + n0 + 8 * q;
      if (a.res_f32) {
        res[q] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.res) + at);
      } else {
        const bf16x4 t = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(a.res) + at);
        res[q] = f32x4{(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
      }
    }
  }
  f32x16 acc = f32x16{};
  u32x4 af[NBUF][NB], wf[NBUF][NB];
  auto load = [&](int t, int b) {
    const unsigned ao = t < nb ? a0 + t * (NB * 32u) : OUT, wo = t < nb ? w0 + t * (NB * 1024u) : OUT;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      af[b][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, ao + i * 32u, 0, 0);
      wf[b][i] = __builtin_amdgcn_raw_buffer_load_b128(rw, wo + i * 1024u, 0, 0);
    }
  };
#pragma unroll
  for (int b = 0; b < NBUF; ++b) {
    load(b, b);
    __builtin_amdgcn_sched_barrier(0);                   // in this order: the waits below count on it
  }
  for (int t = 0; t < nb; t += NBUF) {
#pragma unroll
    for (int b = 0; b < NBUF; ++b) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[b][i]), __builtin_bit_cast(bf16x8, af[b][i]), acc,
                                                        0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      load(t + b + NBUF, b);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (!ok) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int n = n0 + 8 * q;
    const f32x4 o = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]} + bias[q];
    if constexpr (EPI == EPI_RESID) {
      *reinterpret_cast<f32x4*>(static_cast<float*>(a.C) + (long long)row * a.ldc + n) = res[q] + o;
    } else {
      bf16x4 h;
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = (bf16)(EPI == EPI_RELU ? fmaxf(o[e], 0.f) : o[e]);
      *reinterpret_cast<bf16x4*>(static_cast<bf16*>(a.C) + (long long)(n / a.col_block) * a.col_block_stride + (long long)row * a.ldc +
                                 n % a.col_block) = h;
    }
  }
}

template <int EPI>
hipError_t launch_epi(const GemmArgs& a, hipStream_t s) {
  // Up to 256 blocks (one wave per compute unit) the thin form is ahead at every K and N measured (K 384
  // to 4096, N 384 to 4096: 3.4 to 11.3 us, tiles 5.1 to 24 us).  With more, two waves of a compute
  // unit share its L1 and it takes half as long again: at 257 to 512 blocks it is ahead in the
  // residual products (N = 512, few tiles; K 512 R 768: 5.3 against 6.4 us, K 2048: 11.7 against
  // 13.2) and level in the others (K 512, N 2048, R 256: 5.1 against 5.2).  Beyond, the tiles are ahead (K
  // 512, N 1536, R 384: 5.2 against 6.7; K 2048, N 512, R 2048: 13.7 against 22).  Tiles of 64 x 64 were 5%
  // ahead of these at K 384 to 640, N 512, R 2048 (6.4 against 6.7 us at K 512) and behind elsewhere.
  const long long blocks = (long long)((a.R + 31) / 32) * (a.N / 32);
  if (blocks <= 512)
    hipLaunchKernelGGL((k_gemm_thin<EPI>), dim3((unsigned)blocks), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL((k_gemm_tiled<EPI>), dim3((unsigned)(((a.R + BM - 1) / BM) * (a.N / BN))), dim3(64 * NW), 0, s, a);
  return hipGetLastError();
}

}  // namespace

bool gemm_tiled_fits(int K, int N) { return K % 128 == 0 && N % 128 == 0 && K >= 128; }

hipError_t launch_gemm_tiled(const GemmArgs& a, hipStream_t s) {
  if (a.R <= 0) return hipSuccess;
  if (!gemm_tiled_fits(a.K, a.N) || a.ln_g || a.a_f32 || (a.lda % 8)) return hipErrorInvalidValue;
  if (a.epi == EPI_RESID) {
    if (!a.c_f32 || !a.res || (a.ldc % 4) || (a.ldr % 4)) return hipErrorInvalidValue;
  } else if (a.c_f32 || (a.col_block % 32) || (a.ldc % 8) || (a.col_block_stride % 8)) {
    return hipErrorInvalidValue;
  }
  switch (a.epi) {
    case EPI_STORE: return launch_epi<EPI_STORE>(a, s);
    case EPI_RELU: return launch_epi<EPI_RELU>(a, s);
    case EPI_RESID: return launch_epi<EPI_RESID>(a, s);
    default: return hipErrorInvalidValue;
  }
}
