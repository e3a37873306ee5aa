// fp32 row-tile matrix product with a LayerNorm prologue and bias / ReLU / residual epilogues,
// plus the standalone row LayerNorm used by both model types.
//
// On fp32 models every projection of the joint pass (q|k|v, attention output, FFN up and down,
// the context-side key/value cache) is one call of k_gemm: C = epi(LN(A) x W + b), on the
// v_mfma_f32_16x16x4_f32 matrix cores.  (bf16 models use the fused kernels of fused.hip.)
#include "fe_common.h"

namespace {

FE_DEV void load4(const void* p, bool f32, float* v) {
  if (f32) {
    float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
    bf16x4 t = *reinterpret_cast<const bf16x4*>(p);
    v[0] = (float)t[0]; v[1] = (float)t[1]; v[2] = (float)t[2]; v[3] = (float)t[3];
  }
}

// A workgroup of four waves owns GM x GN outputs, each wave 16 rows by two 16 x 16 blocks; k is
// staged through LDS in steps of up to GKC.  fp32 models answer small requests (a launch has one to
// a few tiles, K = d or 4d), so a launch is its chain of memory round trips: a step loads its whole
// A and W slices at once (buffer loads, bounds checked by the hardware), the next step's loads run
// behind this step's products, the LayerNorm statistics come from the staged registers where a row
// fits one step (K <= GKC), and the epilogue requests the residual before the first store.
// Measured, before and after: one tile, K = 32 with LayerNorm 20.9 -> 5.7 us, without (K = 32 and
// 128) 7.9 -> 3.8 us; a pass of the smallest model (d 32, one layer per module) 305 -> 132 us, of
// fp32 models at d 128, B 4, T 256 1129 -> 521 us and at d 512, B 2, T 100 1218 -> 458 us.
constexpr int GM = 64, GN = 32, GKC = 128, GLD = GKC + 4;

template <bool LN>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs a) {
  constexpr int QA = GM * GKC / 4 / 256, QW = GN * GKC / 4 / 256;   // 16-byte loads per thread and step
  __shared__ __attribute__((aligned(16))) float As[GM * GLD];
  __shared__ __attribute__((aligned(16))) float Bs[GN * GLD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row0 = blockIdx.x * GM, col0 = blockIdx.y * GN;
  // this thread's loads: k 4*(tid % 32) of rows tid / 32 + 8 q, so a row lies in one wave half
  const int kk = 4 * (tid & 31), rq = tid >> 5;
  const float* A = static_cast<const float*>(a.A) + (long long)row0 * a.lda;
  const float* W = static_cast<const float*>(a.Wt) + (long long)col0 * a.K;
  const int rows = min(GM, a.R - row0);
  // rows from `rows` on lie past the buffer; columns from K on get an offset that does
  const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A), 0, rows * a.lda * 4, 0x00027000);
  const auto rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W), 0, GN * a.K * 4, 0x00027000);
  constexpr unsigned OUT = 0x80000000u;
  u32x4 va[QA], vw[QW];
  auto load_a = [&](int k0) {
#pragma unroll
    for (int q = 0; q < QA; ++q)
      va[q] = __builtin_amdgcn_raw_buffer_load_b128(ra, k0 + kk < a.K ? ((rq + 8 * q) * a.lda + k0 + kk) * 4u : OUT, 0, 0);
  };
  auto load_w = [&](int k0) {
#pragma unroll
    for (int q = 0; q < QW; ++q)
      vw[q] = __builtin_amdgcn_raw_buffer_load_b128(rw, k0 + kk < a.K ? ((rq + 8 * q) * a.K + k0 + kk) * 4u : OUT, 0, 0);
  };
  load_a(0);
  load_w(0);

  // validity of this thread's rows (padding rows: not stored; a tile of padding only: skipped)
  unsigned valid = 0;
#pragma unroll
  for (int q = 0; q < QA; ++q) {
    const int r = row0 + rq + 8 * q;
    bool ok = r < a.R;
    if (ok && a.nvalid) ok = (r % a.rows_per_batch) < a.nvalid[r / a.rows_per_batch];
    valid |= (unsigned)ok << q;
  }
  if (a.nvalid && !block_any<4>(valid != 0)) return;

  float mean[QA], rstd[QA];
  if constexpr (LN) {
    // two-pass mean / biased variance in fp32; values past K are zero and left out of the squares
    const float inv = 1.f / (float)a.K;
#pragma unroll
    for (int q = 0; q < QA; ++q) mean[q] = rstd[q] = 0.f;
    auto sums = [&]() {
#pragma unroll
      for (int q = 0; q < QA; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c) mean[q] += __uint_as_float(va[q][c]);
    };
    auto squares = [&](int k0) {
      if (k0 + kk >= a.K) return;
#pragma unroll
      for (int q = 0; q < QA; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float t = __uint_as_float(va[q][c]) - mean[q];
          rstd[q] += t * t;
        }
    };
    auto means = [&]() {
#pragma unroll
      for (int q = 0; q < QA; ++q) mean[q] = half_sum(mean[q]) * inv;
    };
    if (a.K <= GKC) {
      sums();
      means();
      squares(0);
    } else {
      for (int k0 = 0; k0 < a.K; k0 += GKC) {
        if (k0) load_a(k0);
        sums();
      }
      means();
      for (int k0 = 0; k0 < a.K; k0 += GKC) {
        load_a(k0);
        squares(k0);
      }
      load_a(0);
    }
#pragma unroll
    for (int q = 0; q < QA; ++q) rstd[q] = rsqrtf(half_sum(rstd[q]) * inv + 1e-5f);
  }

  f32x4 acc[2] = {};
  for (int k0 = 0; k0 < a.K; k0 += GKC) {
    if (k0) lds_barrier();   // the previous step is no longer read
    const bool inside = k0 + kk < a.K;
    float4 g4 = make_float4(0.f, 0.f, 0.f, 0.f), b4 = g4;
    if constexpr (LN)
      if (inside) {
        g4 = *reinterpret_cast<const float4*>(a.ln_g + k0 + kk);
        b4 = *reinterpret_cast<const float4*>(a.ln_b + k0 + kk);
      }
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      float4 v = make_float4(__uint_as_float(va[q][0]), __uint_as_float(va[q][1]), __uint_as_float(va[q][2]), __uint_as_float(va[q][3]));
      if constexpr (LN) {
        const float mu = mean[q], rs = rstd[q];
        v = make_float4((v.x - mu) * rs * g4.x + b4.x, (v.y - mu) * rs * g4.y + b4.y, (v.z - mu) * rs * g4.z + b4.z,
                        (v.w - mu) * rs * g4.w + b4.w);
      }
      if (!(valid >> q & 1)) v = make_float4(0.f, 0.f, 0.f, 0.f);
      *reinterpret_cast<float4*>(&As[(rq + 8 * q) * GLD + kk]) = v;
    }
#pragma unroll
    for (int q = 0; q < QW; ++q) *reinterpret_cast<u32x4*>(&Bs[(rq + 8 * q) * GLD + kk]) = vw[q];
    lds_barrier();
    if (k0 + GKC < a.K) {
      load_a(k0 + GKC);
      load_w(k0 + GKC);
    }
    // K is a multiple of 32; product c of a group of 16 takes k = 4 (lane / 16) + c of both operands
    const int kn = min(GKC, a.K - k0);
    for (int ks = 0; ks < kn; ks += 32) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int ko = ks + 16 * u + 4 * (lane >> 4);
        const float4 af = *reinterpret_cast<const float4*>(&As[(wave * 16 + (lane & 15)) * GLD + ko]);
        const float4 b0 = *reinterpret_cast<const float4*>(&Bs[(lane & 15) * GLD + ko]);
        const float4 b1 = *reinterpret_cast<const float4*>(&Bs[(16 + (lane & 15)) * GLD + ko]);
        const float fa[4] = {af.x, af.y, af.z, af.w}, f0[4] = {b0.x, b0.y, b0.z, b0.w}, f1[4] = {b1.x, b1.y, b1.z, b1.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[c], f0[c], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[c], f1[c], acc[1], 0, 0, 0);
        }
      }
    }
  }

  // ---- epilogue: lane holds rows wave*16 + 4 (lane / 16) + i of columns lane % 16 and + 16.  The tile
  // lies inside one column block (both are multiples of 32).
  const int n = col0 + (lane & 15);
  const long long cb = (long long)(col0 / a.col_block) * a.col_block_stride + n % a.col_block;
  float bias[2] = {0.f, 0.f};
  if (a.bias) {
    bias[0] = a.bias[n];
    bias[1] = a.bias[n + 16];
  }
  float* C = static_cast<float*>(a.C);
  const int rl = wave * 16 + 4 * (lane >> 4);
  float v[4][2], res[4][2] = {};
  bool ok[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = row0 + rl + i;
    ok[i] = r < a.R;
    if (a.nvalid) {
      const int rc = min(r, a.R - 1);
      ok[i] = ok[i] && (rc % a.rows_per_batch) < a.nvalid[rc / a.rows_per_batch];
    }
    if (a.epi == EPI_RESID) {
      const float* rp = static_cast<const float*>(a.res) + (long long)min(r, a.R - 1) * a.ldr + n;
      res[i][0] = rp[0];
      res[i][1] = rp[16];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      v[i][x] = acc[x][i] + bias[x];
      if (a.epi == EPI_RESID) v[i][x] = res[i][x] + v[i][x];
      if (a.epi == EPI_RELU) v[i][x] = fmaxf(v[i][x], 0.f);
    }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!ok[i]) continue;
    float* c = C + cb + (long long)(row0 + rl + i) * a.ldc;
    c[0] = v[i][0];
    c[16] = v[i][1];
  }
}

// Row r of a wide model (d = 512 NC): each lane holds 8 consecutive values of every 512-column
// chunk (16- or 32-byte loads and stores), all indices compile-time.
template <typename T, int NC>
FE_DEV void ln_row_wide(const void* X, int x_f32, long long x_rs, int r, const float* g, const float* b, void* Y,
                        int y_f32, long long y_rs, bool valid, int lane) {
  constexpr int D = 512 * NC;
  // gains and offsets are requested with the row, so their latency overlaps the row's
  float4 gv[NC][2], bv[NC][2];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int k = c * 512 + lane * 8;
    gv[c][0] = *reinterpret_cast<const float4*>(g + k);
    gv[c][1] = *reinterpret_cast<const float4*>(g + k + 4);
    bv[c][0] = *reinterpret_cast<const float4*>(b + k);
    bv[c][1] = *reinterpret_cast<const float4*>(b + k + 4);
  }
  float v[8 * NC];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int k = c * 512 + lane * 8;
    if (x_f32 || sizeof(T) == 4) {
      const float4* src = reinterpret_cast<const float4*>(static_cast<const float*>(X) + (size_t)r * x_rs + k);
      const float4 t0 = src[0], t1 = src[1];
      v[8 * c] = t0.x; v[8 * c + 1] = t0.y; v[8 * c + 2] = t0.z; v[8 * c + 3] = t0.w;
      v[8 * c + 4] = t1.x; v[8 * c + 5] = t1.y; v[8 * c + 6] = t1.z; v[8 * c + 7] = t1.w;
    } else {
      const bf16x8 t = *reinterpret_cast<const bf16x8*>(static_cast<const bf16*>(X) + (size_t)r * x_rs + k);
#pragma unroll
      for (int j = 0; j < 8; ++j) v[8 * c + j] = (float)t[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) sum += v[8 * c + j];
  }
  const float mean = wave_sum(sum) * (1.f / D);
  float sq = 0.f;
#pragma unroll
  for (int t = 0; t < 8 * NC; ++t) { const float dl = v[t] - mean; sq += dl * dl; }
  const float rstd = rsqrtf(wave_sum(sq) * (1.f / D) + 1e-5f);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int k = c * 512 + lane * 8;
    const float4 g0 = gv[c][0], g1 = gv[c][1], b0 = bv[c][0], b1 = bv[c][1];
    const float gg[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    const float bb[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
    float y[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = valid ? (v[8 * c + j] - mean) * rstd * gg[j] + bb[j] : 0.f;
    if (y_f32) {
      float4* dst = reinterpret_cast<float4*>(static_cast<float*>(Y) + (size_t)r * y_rs + k);
      dst[0] = make_float4(y[0], y[1], y[2], y[3]);
      dst[1] = make_float4(y[4], y[5], y[6], y[7]);
    } else if constexpr (sizeof(T) == 2) {
      bf16x8 o;
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = (bf16)y[j];
      *reinterpret_cast<bf16x8*>(static_cast<bf16*>(Y) + (size_t)r * y_rs + k) = o;
    } else {
      float4* dst = reinterpret_cast<float4*>(static_cast<float*>(Y) + (size_t)r * y_rs + k);
      dst[0] = make_float4(y[0], y[1], y[2], y[3]);
      dst[1] = make_float4(y[4], y[5], y[6], y[7]);
    }
  }
}

// One wave per row: Y = LN(X), padding rows (per nvalid) written as zeros.  NC > 0: d = 512 NC
// (ln_row_wide); NC = 0: any d <= 1024.  Separate instances, so that the general form's registers
// do not lower the occupancy of the wide one.
template <typename T, int NC>
__global__ __launch_bounds__(256) void k_layernorm(const void* X, int x_f32, long long x_rs, int R, int d,
                                                   const float* g, const float* b, void* Y, int y_f32,
                                                   long long y_rs, const int32_t* nvalid, int rpb) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= R) return;
  const bool valid = !nvalid || (r % rpb) < nvalid[r / rpb];
  if constexpr (NC > 0) {
    ln_row_wide<T, NC>(X, x_f32, x_rs, r, g, b, Y, y_f32, y_rs, valid, lane);
    return;
  }
  // up to four 4-column groups per lane (d <= 1024), all loads -- the row, the gains and the
  // offsets -- requested before the first use; compile-time indices keep everything in registers
  float vals[16];
  float4 gv[4], bv[4];
  float sum = 0.f;
  x_f32 = x_f32 || sizeof(T) == 4;
  const size_t xs = x_f32 ? 4 : sizeof(T);
  const char* xr = static_cast<const char*>(X) + (size_t)r * x_rs * xs;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int k = lane * 4 + c * 256;
    if (k >= d) continue;
    float v4[4];
    load4(xr + (size_t)k * xs, x_f32, v4);
    gv[c] = *reinterpret_cast<const float4*>(g + k);
    bv[c] = *reinterpret_cast<const float4*>(b + k);
#pragma unroll
    for (int j = 0; j < 4; ++j) { vals[c * 4 + j] = v4[j]; sum += v4[j]; }
  }
  const float mean = wave_sum(sum) / (float)d;
  float sq = 0.f;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (lane * 4 + c * 256 >= d) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) { const float dl = vals[c * 4 + j] - mean; sq += dl * dl; }
  }
  const float rstd = rsqrtf(wave_sum(sq) / (float)d + 1e-5f);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int k = lane * 4 + c * 256;
    if (k >= d) continue;
    const float gg[4] = {gv[c].x, gv[c].y, gv[c].z, gv[c].w}, bb[4] = {bv[c].x, bv[c].y, bv[c].z, bv[c].w};
    float y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = valid ? (vals[c * 4 + j] - mean) * rstd * gg[j] + bb[j] : 0.f;
    if (y_f32) {
      *reinterpret_cast<float4*>(static_cast<float*>(Y) + (size_t)r * y_rs + k) = make_float4(y[0], y[1], y[2], y[3]);
    } else {
      T o[4];
      for (int j = 0; j < 4; ++j) o[j] = from_f32<T>(y[j]);
      if constexpr (sizeof(T) == 2) *reinterpret_cast<bf16x4*>(static_cast<T*>(Y) + (size_t)r * y_rs + k) = *reinterpret_cast<const bf16x4*>(o);
      else *reinterpret_cast<float4*>(static_cast<T*>(Y) + (size_t)r * y_rs + k) = *reinterpret_cast<const float4*>(o);
    }
  }
}

}  // namespace

hipError_t launch_gemm(const GemmArgs& a, bool bf16_model, hipStream_t s) {
  if (a.R <= 0) return hipSuccess;
  if (bf16_model) return hipErrorInvalidValue;   // bf16 weights are packed for k_proj / k_ffn
  // rows of fp32 values in whole groups of 32; 32-bit byte offsets inside a tile
  if (a.K % 32 || a.N % GN || a.col_block % GN || a.lda % 4 || a.lda > (1 << 22) || a.K > (1 << 22)) return hipErrorInvalidValue;
  dim3 grid((a.R + GM - 1) / GM, a.N / GN);
  if (a.ln_g) hipLaunchKernelGGL(k_gemm<true>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_gemm<false>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_layernorm_masked(const void* X, int x_f32, long long x_rs, int R, int d, const float* g,
                                   const float* b, void* Y, int y_f32, long long y_rs, const int32_t* nvalid,
                                   int rpb, bool bf16_model, hipStream_t s) {
  if (R <= 0) return hipSuccess;
  if (d > 1024 || d % 4) return hipErrorInvalidValue;
  const dim3 grid((R + 3) / 4);
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, X, x_f32, x_rs, R, d, g, b, Y, y_f32, y_rs, nvalid, rpb); };
  if (bf16_model) {
    if (d == 512) go(k_layernorm<bf16, 1>);
    else if (d == 1024) go(k_layernorm<bf16, 2>);
    else go(k_layernorm<bf16, 0>);
  } else {
    if (d == 512) go(k_layernorm<float, 1>);
    else if (d == 1024) go(k_layernorm<float, 2>);
    else go(k_layernorm<float, 0>);
  }
  return hipGetLastError();
}

hipError_t launch_layernorm(const void* X, int x_f32, long long x_rs, int R, int d, const float* g, const float* b,
                            void* Y, int y_f32, long long y_rs, bool bf16_model, hipStream_t s) {
  return launch_layernorm_masked(X, x_f32, x_rs, R, d, g, b, Y, y_f32, y_rs, nullptr, 1, bf16_model, s);
}
