// fp32 kernels of the training step (Section 4.5): the forward with saved activations and its
// backward: a strided product, attention per (sequence, head), row-wise LayerNorm, all with their
// backward passes, elementwise steps, row gathers and their scatter-add backward, and the losses
// with the label construction of Appendix B.1.
#include "fe_common.h"
#include "train_kernels.h"

#include <algorithm>
#include <initializer_list>

namespace {

// ------------------------------------------------------------------------------------------
// C = alpha * op(A) op(B) + beta * C (+ bias[j]); element (i, k) of A at A + i*a_rs + k*a_cs (likewise
// B with (k, j), C with (i, j) and unit column stride).
//
// fp32 matrix cores: a workgroup of four waves owns a (32 WM) x (32 WN) output tile, each wave one
// 32 x 32 block accumulated by v_mfma_f32_32x32x2_f32 (lane l feeds A[l%32][l/32] and
// B[l/32][l%32] of a 32x32x2 step and holds D[8q + 4(l/32) + e][l%32] in accumulator 4q + e).
// k advances in steps of 32 through LDS.  AK / BK: the operand's k index is its contiguous one, so
// consecutive lanes load along k (else along i or j), which keeps the global loads coalesced for
// both orientations.
// ------------------------------------------------------------------------------------------
constexpr int GK = 32;

// One operand's tile of T rows (i or j) by GK k values, through registers into LDS.
//   KC:  k contiguous in memory -> LDS [row][k], each group of eight k values as 0 2 4 6 1 3 5 7, rows of
//        GK + 4 floats (a wave half's 16-byte reads of 32 rows fall on every bank group once);
//   !KC: rows contiguous        -> LDS [k][row], rows of T + 8 floats.
// Either way the store keeps the orientation of the load (VEC: four values of it at a time).  MFMA c
// of the group of eight k values from 8s takes k = 8s + 2c + (l/32): k ascends over the MFMAs.
template <int T, bool KC, bool VEC>
struct TOperand {
  static constexpr int N = GK * T / 256;                    // values per thread and step
  static constexpr int LD = KC ? GK + 4 : T + 8, SIZE = KC ? T * LD : GK * LD;
  static constexpr int W = VEC ? 4 : 1, NG = N / W;         // values per load, loads
  static constexpr unsigned OUT = 0x80000000u;              // past every buffer below: such a load gives zeros
  const float* base;                                        // row 0 of the tile at k = 0 (uniform)
  unsigned off[NG];                                         // this thread's byte offsets at a step's first k
  long long ks;                                             // stride of k
  float r[N];
  // rows of the tile at row0 .. rows - 1; base0 is the matrix.  Rows past the last get OUT.
  FE_DEV void init(const float* base0, int row0, int rows, long long rs, long long ks_) {
    base = base0 + row0 * rs;
    ks = ks_;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int e = threadIdx.x + 256 * q;
      const int row = KC ? e / (GK / W) : W * (e % (T / W)), kk = KC ? W * (e % (GK / W)) : e / (T / W);
      off[q] = row0 + row < rows ? 4u * (unsigned)(row * (int)rs + kk * (int)ks_) : OUT;
    }
  }
  // the values of step k0, k < kend (a group of W lies inside or outside as a whole: the launcher
  // checks that the contiguous extent is a multiple of W).  Loads only: no branch between them, so
  // all of a step's are in flight together.
  FE_DEV void load(int k0, int kend) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + k0 * ks), 0, 0x7ffffffc, 0x00027000);
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int e = threadIdx.x + 256 * q;
      const int kk = KC ? W * (e % (GK / W)) : e / (T / W);
      const unsigned o = k0 + kk < kend ? off[q] : OUT;
      if constexpr (VEC) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, o, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) r[4 * q + c] = __uint_as_float(v[c]);
      } else {
        r[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, o, 0, 0));
      }
    }
  }
  FE_DEV void store(float* S) const {
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int e = threadIdx.x + 256 * q;
      if constexpr (KC) {
        const int k = W * (e % (GK / W));
        float* d = S + (e / (GK / W)) * LD + k / 8 * 8 + k % 2 * 4 + k % 8 / 2;
        if constexpr (VEC) {
          *reinterpret_cast<float2*>(d) = make_float2(r[4 * q], r[4 * q + 2]);
          *reinterpret_cast<float2*>(d + 4) = make_float2(r[4 * q + 1], r[4 * q + 3]);
        } else {
          *d = r[q];
        }
      } else {
        float* d = S + (e / (T / W)) * LD + W * (e % (T / W));
        if constexpr (VEC) *reinterpret_cast<float4*>(d) = make_float4(r[4 * q], r[4 * q + 1], r[4 * q + 2], r[4 * q + 3]);
        else *d = r[q];
      }
    }
  }
  // the lane's operands of the four MFMAs of k group s, for the 32 rows from w
  static FE_DEV void frag(const float* S, int w, int s, float (&v)[4]) {
    const int lr = threadIdx.x & 31, lk = (threadIdx.x >> 5) & 1;
    if constexpr (KC) {
      const float4 t = *reinterpret_cast<const float4*>(&S[(w + lr) * LD + 8 * s + 4 * lk]);
      v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = S[(8 * s + 2 * c + lk) * LD + w + lr];
    }
  }
};

// What bounds it: at K = d = 128 a tile has four k steps, so the latencies around them count as much
// as the products.  Hence: operands by buffer loads whose bounds the hardware checks (no branch
// between them, so a step's loads share one latency), LDS in two buffers (the next step's loads run
// behind this step's products, one barrier per step), the epilogue's residual / mask / old-C
// values all requested before the first store (C may alias them as far as the compiler knows, so
// loads written between the stores are waited for one by one), and the tiles numbered so that one
// XCD's L2 serves the column tiles of a row tile.  Measured, before and after: a 385 x 64 x 64
// product 9.3 -> 4.2 us; 16384 x 384 x 128 25.8 -> 23.2 us (67 TFLOP/s; its output alone is 25 MB);
// a training step of 385 context rows (d 64) 1984 -> 1390 us, of 16384 (d 128) 5632 -> 4962 us.
template <int WM, int WN, bool AK, bool BK, bool VA, bool VB>
__global__ __launch_bounds__(256) void k_gemm(TGemm g, int kc0, int tiles_n, int tiles) {
  static_assert(WM * WN == 4, "four waves");
  constexpr int TM = 32 * WM, TN = 32 * WN;
  using OA = TOperand<TM, AK, VA>;
  using OB = TOperand<TN, BK, VB>;
  __shared__ __align__(16) float As[2][OA::SIZE];
  __shared__ __align__(16) float Bs[2][OB::SIZE];
  const int id = xcd_tile(blockIdx.x, gridDim.x);   // tiles of one k chunk are neighbours
  const int kc = kc0 + id / tiles, tile = id % tiles;
  const int kbeg = g.ksplit > 0 ? kc * g.ksplit : 0;
  const int kend = g.ksplit > 0 ? min(g.K, kbeg + g.ksplit) : g.K;
  const int ti = tile / tiles_n, tj = tile % tiles_n;
  const int i0 = ti * TM, j0 = tj * TN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wi = (wave / WN) * 32, wj = (wave % WN) * 32;
  const int lr = lane & 31, lk = lane >> 5;
  OA a;
  OB b;
  a.init(g.A, i0, g.M, g.a_rs, g.a_cs);
  b.init(g.B, j0, g.N, g.b_cs, g.b_rs);
  auto load = [&](int k0) {
    a.load(k0, kend);
    b.load(k0, kend);
  };
  f32x16 acc = {};
  // first row tile: column sums of B, 256 / TN threads per column
  const bool csum = g.colsum && ti == 0;
  float cs = 0.f;
  load(kbeg);
  a.store(As[0]);
  b.store(Bs[0]);
  lds_barrier();
  int cur = 0;
  for (int k0 = kbeg; k0 < kend; k0 += GK, cur ^= 1) {
    const bool more = k0 + GK < kend;
    if (more) load(k0 + GK);
    const float *Ac = As[cur], *Bc = Bs[cur];
    float av[2][4], bv[2][4];                       // group s + 1 is read behind the products of group s
    OA::frag(Ac, wi, 0, av[0]);
    OB::frag(Bc, wj, 0, bv[0]);
#pragma unroll
    for (int s = 0; s < GK / 8; ++s) {
      if (s + 1 < GK / 8) {
        OA::frag(Ac, wi, s + 1, av[(s + 1) & 1]);
        OB::frag(Bc, wj, s + 1, bv[(s + 1) & 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s & 1][c], bv[s & 1][c], acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (csum) {
      const int jj = threadIdx.x % TN, part = threadIdx.x / TN;
      constexpr int KP = GK * TN / 256;
#pragma unroll
      for (int t = 0; t < KP; ++t) cs += BK ? Bc[jj * OB::LD + part * KP + t] : Bc[(part * KP + t) * OB::LD + jj];   // in either order of k
    }
    if (more) {
      a.store(As[cur ^ 1]);   // last read one step ago, before the barrier that ended it
      b.store(Bs[cur ^ 1]);
    }
    lds_barrier();
  }
  if (csum) {
    As[0][threadIdx.x] = cs;
    lds_barrier();
    if (threadIdx.x < TN && j0 + (int)threadIdx.x < g.N) {
      float t = 0.f;
#pragma unroll
      for (int p = 0; p < 256 / TN; ++p) t += As[0][p * TN + threadIdx.x];
      atomicAdd(&g.colsum[j0 + threadIdx.x], g.alpha * t);
    }
  }
  const int j = j0 + wj + lr;
  if (j >= g.N) return;
  const int ib = i0 + wi + 4 * lk;                  // row of accumulator 4q + e: ib + 8q + e
  float* C = g.C + j;
  if (g.ksplit > 0) {
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int i = ib + 8 * (t >> 2) + (t & 3);
      if (i < g.M) atomicAdd(C + i * g.c_rs, g.alpha * acc[t]);
    }
    return;
  }
  // rows past M read row M - 1, so every load is unconditional
  auto at = [&](int t) { return min(ib + 8 * (t >> 2) + (t & 3), g.M - 1) * g.c_rs; };
  float r[16];
  const float bias = g.bias ? g.bias[j] : 0.f;
#pragma unroll
  for (int t = 0; t < 16; ++t) r[t] = g.alpha * acc[t] + bias;
  if (g.R) {
    float v[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) v[t] = g.R[j + at(t)];
#pragma unroll
    for (int t = 0; t < 16; ++t) r[t] += v[t];
  }
  if (g.relu)
#pragma unroll
    for (int t = 0; t < 16; ++t) r[t] = fmaxf(r[t], 0.f);
  if (g.mask) {
    float v[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) v[t] = g.mask[j + at(t)];
#pragma unroll
    for (int t = 0; t < 16; ++t) r[t] = v[t] > 0.f ? r[t] : 0.f;
  }
  if (g.beta != 0.f) {
    float v[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) v[t] = C[at(t)];
#pragma unroll
    for (int t = 0; t < 16; ++t) r[t] += g.beta * v[t];
  }
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int i = ib + 8 * (t >> 2) + (t & 3);
    if (i < g.M) C[i * g.c_rs] = r[t];
  }
}

// ------------------------------------------------------------------------------------------
// Attention of the training step, forward and backward, per (sequence, head): scores and
// probabilities stay on chip.  The forward keeps each query's maximum m and 1 / l of its normaliser
// l = sum exp(score - m) (infinity and 0 for a query that attends to nothing), from which the
// backward forms the forward's probabilities again: the same products in the same order, the score
// scaled, the maximum taken off and the exponential scaled by 1 / l with a rounding each.
//
// Everything is a product of TS x TS blocks on the fp32 matrix cores (TS = 32: 32x32x2, TS = 16:
// 16x16x4; NS = 64 / TS k slots).  Accumulator a of a lane in slot g is block row
// 4 NS (a / 4) + 4 g + a % 4 of column lane % TS.  A product's left rows are fed in the order that
// makes it row NS a + g of the LDS tile: read as a k index, that is what a lane of slot g feeds to
// product a of a following contraction over the block's rows, so a block of probabilities goes into
// the next product from its registers.  Contractions over the head's columns take column
// 4 NS s + NS c + g for product (s, c), which a tile's column order (pos) makes 16-byte reads.
//
// The forward's sums run in a fixed order whatever the tiling (k ascending over the products; the
// normaliser as a tree over the key index: 64-strided partial sums, then bits 5 to 0), with the
// maximum known before the first exponential: a ReLU further on turns a rounding difference at zero
// into a jump of the gradient, so the order is part of the result.
//
// A wave owns TS queries (forward, dQ: blocks are [key][query]) or TS keys (dK and dV: blocks are
// [query][key]) and walks the other side in tiles that the workgroup stages in LDS, the next tile's
// loads in flight; sequences of up to TS rows (SMALL) take one wave each instead.  Bound by the fp32
// matrix rate (2 products forward up to 256 keys, 4 beyond, where the scores are formed anew for the
// maximum, the sum and the probabilities; 7 backward: S and dP are formed in both orientations, which
// costs less than moving dS through memory or adding dQ atomically).  Measured, before (probabilities
// through memory, a launch per product) and after: 256 x 256, 256 heads of 32: forward 69 -> 32 us,
// backward 117 -> 79 us; 11 x 11, 12800 heads of 32: forward 62 -> 18 us, backward 118 -> 32 us; 77 x
// 77, 10 heads of 32: forward 16 -> 12 us, backward 33 -> 15 us.
// ------------------------------------------------------------------------------------------
// LDS written before it by any lane of the wave is visible to the wave's reads after it.
FE_DEV void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int TS>
FE_DEV float slot_max(float v) {
  if constexpr (TS == 16) return rows_max(v);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
template <int TS>
FE_DEV float slot_sum(float v) {
  if constexpr (TS == 16) return rows_sum(v);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Sum over the keys of a column: p0 and p1 hold the sums over the even and odd tiles (accumulator i,
// slot g: key NS i + g of a tile; TS = 16 has one tile, whose bits 5 and 4 add nothing).
template <int TS, class Acc>
FE_DEV float tree_sum(const Acc& p0, const Acc& p1) {
  constexpr int NA = TS * TS / 64;
  float x[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) x[i] = p0[i] + p1[i];
#pragma unroll
  for (int h = NA / 2; h > 0; h >>= 1)
#pragma unroll
    for (int i = 0; i < h; ++i) x[i] += x[i + h];
  x[0] = slot_sum<32>(x[0]);                        // lanes l, l ^ 32
  if constexpr (TS == 16) {
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[0]), __float_as_uint(x[0]), false, false);
    x[0] = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  }
  return x[0];
}

template <int TS, int DH>
struct AttnTile {
  static constexpr int NS = 64 / TS, NA = TS * TS / 64, NQ = DH / (4 * NS), NB = DH / TS, LD = DH + 4, SIZE = TS * LD;
  typedef float acc_t __attribute__((ext_vector_type(NA)));
  static FE_DEV acc_t mfma(float a, float b, acc_t c) {
    if constexpr (TS == 32) return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static FE_DEV int col() { return threadIdx.x % TS; }
  static FE_DEV int slot() { return (threadIdx.x & 63) / TS; }
  static FE_DEV int row(int a) { return NS * a + slot(); }                 // tile row of accumulator a
  static FE_DEV int pos(int c) { return c / (4 * NS) * (4 * NS) + c % NS * 4 + c % (4 * NS) / NS; }   // of column c in a tile row
  // the operands of products (s, c), c = 0..3, from one row of DH values in memory
  static FE_DEV void row_frag(const float* p, float4 (&f)[NQ]) {
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
      const float* x = p + 4 * NS * s + slot();
      f[s] = make_float4(x[0], x[NS], x[2 * NS], x[3 * NS]);
    }
  }
  // ... from row r of an LDS tile
  static FE_DEV void tile_frag(const float* L, int r, float4 (&f)[NQ]) {
#pragma unroll
    for (int s = 0; s < NQ; ++s) f[s] = *reinterpret_cast<const float4*>(&L[r * LD + 4 * NS * s + 4 * slot()]);
  }
  // block [i][j] = rows i of the LDS tile L times the rows j held as fragments
  static FE_DEV acc_t rows_by(const float* L, const float4 (&f)[NQ]) {
    acc_t c = {};
    float4 t[NQ];
    const int i = col();
    tile_frag(L, NS * (4 * (i / (4 * NS)) + i % 4) + i % (4 * NS) / 4, t);
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
      c = mfma(t[s].x, f[s].x, c);
      c = mfma(t[s].y, f[s].y, c);
      c = mfma(t[s].z, f[s].z, c);
      c = mfma(t[s].w, f[s].w, c);
    }
    return c;
  }
  // out [column of L][j] += sum over the tile's rows i of L[i][.] times block [i][j]
  static FE_DEV void cols_by(const float* L, const acc_t& p, acc_t (&out)[NB]) {
    int at[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) at[b] = slot() * LD + pos(b * TS + col());
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) out[b] = mfma(L[NS * a * LD + at[b]], p[a], out[b]);
  }
  // the lane's row of DH values = out, or zeros
  static FE_DEV void put(const acc_t (&out)[NB], float* xrow, bool ok = true) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int a = 0; a < NA; a += 4)
        *reinterpret_cast<float4*>(xrow + b * TS + NS * a + 4 * slot()) =
            ok ? make_float4(out[b][a], out[b][a + 1], out[b][a + 2], out[b][a + 3]) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
};

// TS rows from row r0 of X (row stride rs, rows from n on read as zeros; n >= 1) by NT threads:
// requested by load(), written to an LDS tile by store().
template <int TS, int DH, int NT>
struct AttnStage {
  using T = AttnTile<TS, DH>;
  static constexpr int V = TS * DH / 4 / NT, TPR = DH / 4;
  static_assert(TS * DH % (4 * NT) == 0, "whole loads per thread");
  float4 r[V];
  bool ok[V];
  static FE_DEV int row(int p) { return (threadIdx.x % NT + p * NT) / TPR; }
  static FE_DEV int col() { return 4 * (threadIdx.x % TPR); }
  FE_DEV void load(const float* X, long long rs, int r0, int n) {
#pragma unroll
    for (int p = 0; p < V; ++p) {
      const int i = r0 + row(p);
      ok[p] = i < n;
      r[p] = *reinterpret_cast<const float4*>(X + min(i, n - 1) * rs + col());
    }
  }
  FE_DEV void store(float* L) const {
#pragma unroll
    for (int p = 0; p < V; ++p) {
      const float4 v = ok[p] ? r[p] : make_float4(0.f, 0.f, 0.f, 0.f);
      float* d = &L[row(p) * T::LD + T::pos(col())];
      if constexpr (TS == 32) {
        *reinterpret_cast<float2*>(d) = make_float2(v.x, v.z);
        *reinterpret_cast<float2*>(d + 4) = make_float2(v.y, v.w);
      } else {
        d[0] = v.x;
        d[4] = v.y;
        d[8] = v.z;
        d[12] = v.w;
      }
    }
  }
};

// Sequence, head and lengths of a (sequence, head) pair.
struct AttnPair {
  int z, h, nq, nk;
  FE_DEV AttnPair(const TAttn& a, int pair) {
    z = pair / a.H;
    h = pair % a.H;
    nq = a.qlen ? min(a.Sq, a.qlen[z]) : a.Sq;
    nk = a.klen ? min(a.Sk, a.klen[z]) : a.Sk;
  }
};

// NT > 0: keys of up to NT tiles, whose scores stay in registers between the maximum, the sum and
// the products with the values; NT = 0: any number, the scores formed anew for each of the three.
template <int TS, int DH, int NT, bool SMALL>
__global__ __launch_bounds__(256, 2) void k_attn_fwd(TAttn a) {
#pragma clang fp contract(off)
  constexpr int NK = NT > 0 ? NT : 1;
  using T = AttnTile<TS, DH>;
  using St = AttnStage<TS, DH, SMALL ? 64 : 256>;
  static_assert(!SMALL || NT == 1, "a wave per sequence holds one tile");
  constexpr int NBUF = SMALL ? 8 : 2;               // two tiles (K, V) per wave, or two buffers of the workgroup
  __shared__ __align__(16) float Xs[NBUF][T::SIZE];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int id = xcd_tile(blockIdx.x, gridDim.x);
  const int groups = SMALL ? 1 : (a.Sq + 4 * TS - 1) / (4 * TS);
  const int pair = SMALL ? 4 * id + wave : id / groups;
  if (SMALL && pair >= a.nseq * a.H) return;        // waves share nothing
  const AttnPair P(a, pair);
  const int q = (SMALL ? 0 : (id % groups * 4 + wave) * TS) + T::col();
  const float* K = a.k + P.z * a.k_bs + P.h * DH;
  const float* Vv = a.v + P.z * a.v_bs + P.h * DH;
  float4 qf[T::NQ];
  T::row_frag(a.q + P.z * a.q_bs + P.h * DH + min(q, a.Sq - 1) * a.q_rs, qf);
  St st;
  int cur = SMALL ? 2 * wave : 0;
  // The next staged tile, and the request for the one after it (null: none).  Storing to a buffer
  // follows every read of it: those precede the last barrier but one of the wave that read.
  auto next = [&](const float* X, long long rs, int r0) -> const float* {
    const float* tile = Xs[cur];
    st.store(Xs[cur]);
    if constexpr (SMALL) wave_sync();
    else lds_barrier();
    if (X) st.load(X, rs, r0, P.nk);
    cur ^= 1;
    return tile;
  };
  float m = -INFINITY, inv = 0.f;
  typename T::acc_t s[NK], o[T::NB] = {};
  if (P.nk > 0) st.load(K, a.k_rs, 0, P.nk);        // with no key at all every loop below is empty
  if constexpr (NT > 0) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t * TS >= P.nk) {
        s[t] = typename T::acc_t{};
        continue;
      }
      const bool last = (t + 1) * TS >= P.nk;
      const float* tile = last ? next(Vv, a.v_rs, 0) : next(K, a.k_rs, (t + 1) * TS);
      s[t] = T::rows_by(tile, qf);
#pragma unroll
      for (int i = 0; i < T::NA; ++i) {
        s[t][i] = t * TS + T::row(i) < P.nk ? s[t][i] * a.scale : -INFINITY;
        m = fmaxf(m, s[t][i]);
      }
    }
    m = slot_max<TS>(m);
    typename T::acc_t part[2] = {};
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (t * TS < P.nk)
#pragma unroll
        for (int i = 0; i < T::NA; ++i) {
          s[t][i] = expf(s[t][i] - m);
          part[t & 1][i] += s[t][i];
        }
    inv = 1.f / tree_sum<TS>(part[0], part[1]);
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (t * TS < P.nk) {
        const bool more = (t + 1) * TS < P.nk;
        const float* tile = next(more ? Vv : nullptr, a.v_rs, (t + 1) * TS);
#pragma unroll
        for (int i = 0; i < T::NA; ++i) s[t][i] *= inv;
        T::cols_by(tile, s[t], o);
      }
  } else {
    for (int k0 = 0; k0 < P.nk; k0 += TS) {
      const bool more = k0 + TS < P.nk;
      const float* tile = next(K, a.k_rs, more ? k0 + TS : 0);
      s[0] = T::rows_by(tile, qf);
#pragma unroll
      for (int i = 0; i < T::NA; ++i)
        if (k0 + T::row(i) < P.nk) m = fmaxf(m, s[0][i] * a.scale);
    }
    m = slot_max<TS>(m);
    auto probs = [&](const float* tile, int k0) {
      s[0] = T::rows_by(tile, qf);
#pragma unroll
      for (int i = 0; i < T::NA; ++i) s[0][i] = k0 + T::row(i) < P.nk ? expf(s[0][i] * a.scale - m) : 0.f;
    };
    typename T::acc_t part[2] = {};
    for (int k0 = 0; k0 < P.nk; k0 += TS) {
      const bool more = k0 + TS < P.nk;
      probs(next(K, a.k_rs, more ? k0 + TS : 0), k0);
      if ((k0 / TS) & 1) part[1] += s[0];
      else part[0] += s[0];
    }
    inv = 1.f / tree_sum<TS>(part[0], part[1]);
    for (int k0 = 0; k0 < P.nk; k0 += TS) {
      const bool more = k0 + TS < P.nk;
      probs(next(Vv, a.v_rs, k0), k0);
#pragma unroll
      for (int i = 0; i < T::NA; ++i) s[0][i] *= inv;
      T::cols_by(next(more ? K : nullptr, a.k_rs, k0 + TS), s[0], o);
    }
  }
  if (q >= a.Sq) return;
  const bool ok = q < P.nq && P.nk > 0;             // other queries attend to nothing: zero rows
  T::put(o, a.o + P.z * a.o_bs + P.h * DH + q * a.o_rs, ok);
  if (T::slot() == 0) a.stat[((long long)P.z * a.H + P.h) * a.Sq + q] = ok ? make_float2(m, inv) : make_float2(INFINITY, 0.f);
}

// dK and dV of the wave's TS keys (fragments kf, vf; kok: this lane's key exists) from one tile of
// queries Qt, output gradients Ot, and their statistics and D = rowsum(dO O).
template <int TS, int DH>
FE_DEV void attn_kv_tile(const float* Qt, const float* Ot, const float2* stat, const float* Dr, float scale, bool kok,
                         const float4 (&kf)[AttnTile<TS, DH>::NQ], const float4 (&vf)[AttnTile<TS, DH>::NQ],
                         typename AttnTile<TS, DH>::acc_t (&dk)[AttnTile<TS, DH>::NB],
                         typename AttnTile<TS, DH>::acc_t (&dv)[AttnTile<TS, DH>::NB]) {
#pragma clang fp contract(off)   // the forward's probabilities
  using T = AttnTile<TS, DH>;
  typename T::acc_t p = T::rows_by(Qt, kf), ds = T::rows_by(Ot, vf);
#pragma unroll
  for (int i = 0; i < T::NA; ++i) {
    const float2 st = stat[T::row(i)];
    p[i] = kok ? expf(p[i] * scale - st.x) * st.y : 0.f;
    ds[i] = scale * p[i] * (ds[i] - Dr[T::row(i)]);
  }
  T::cols_by(Ot, p, dv);
  T::cols_by(Qt, ds, dk);
}

// dQ of the wave's TS queries (fragments qf, of; their statistics and D) from one tile of keys and values
// whose first `nk` rows exist.
template <int TS, int DH>
FE_DEV void attn_q_tile(const float* Kt, const float* Vt, float2 st, float D, float scale, int nk,
                        const float4 (&qf)[AttnTile<TS, DH>::NQ], const float4 (&of)[AttnTile<TS, DH>::NQ],
                        typename AttnTile<TS, DH>::acc_t (&dq)[AttnTile<TS, DH>::NB]) {
#pragma clang fp contract(off)   // the forward's probabilities
  using T = AttnTile<TS, DH>;
  typename T::acc_t p = T::rows_by(Kt, qf), ds = T::rows_by(Vt, of);
#pragma unroll
  for (int i = 0; i < T::NA; ++i) ds[i] = T::row(i) < nk ? scale * (expf(p[i] * scale - st.x) * st.y) * (ds[i] - D) : 0.f;
  T::cols_by(Kt, ds, dq);
}

template <int TS, int DH>
FE_DEV float attn_dot(const float4 (&x)[AttnTile<TS, DH>::NQ], const float4 (&y)[AttnTile<TS, DH>::NQ]) {
  float t = 0.f;
#pragma unroll
  for (int s = 0; s < AttnTile<TS, DH>::NQ; ++s)
    t += x[s].x * y[s].x + x[s].y * y[s].y + x[s].z * y[s].z + x[s].w * y[s].w;
  return slot_sum<TS>(t);
}

// Long sequences: workgroups 0 .. n_kv - 1 (after the XCD order) form dK and dV of 4 TS keys each, the
// others dQ of 4 TS queries each.
template <int TS, int DH>
__global__ __launch_bounds__(256, DH == 32 ? 3 : 2) void k_attn_bwd(TAttn a, int n_kv) {
  using T = AttnTile<TS, DH>;
  using St = AttnStage<TS, DH, 256>;
  __shared__ __align__(16) float Xs[2][T::SIZE];
  __shared__ __align__(16) float Ys[2][T::SIZE];
  __shared__ __align__(16) float2 s_stat[2][TS];
  __shared__ __align__(16) float s_D[2][TS];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool is_kv = (int)blockIdx.x < n_kv;
  const int id = is_kv ? xcd_tile(blockIdx.x, n_kv) : xcd_tile(blockIdx.x - n_kv, gridDim.x - n_kv);
  const int groups = ((is_kv ? a.Sk : a.Sq) + 4 * TS - 1) / (4 * TS);
  const AttnPair P(a, id / groups);
  const int own = (id % groups * 4 + wave) * TS + T::col();   // this lane's key or query
  const float* Q = a.q + P.z * a.q_bs + P.h * DH;
  const float* K = a.k + P.z * a.k_bs + P.h * DH;
  const float* Vv = a.v + P.z * a.v_bs + P.h * DH;
  const float* O = a.o + P.z * a.o_bs + P.h * DH;
  const float* dO = a.dO + P.z * a.do_bs + P.h * DH;
  const float2* stat = a.stat + ((long long)P.z * a.H + P.h) * a.Sq;
  int cur = 0;
  if (is_kv) {
    float4 kf[T::NQ], vf[T::NQ];
    T::row_frag(K + min(own, a.Sk - 1) * a.k_rs, kf);
    T::row_frag(Vv + min(own, a.Sk - 1) * a.v_rs, vf);
    typename T::acc_t dk[T::NB] = {}, dv[T::NB] = {};
    St sq, sdo, so;
    float2 st = make_float2(INFINITY, 0.f);
    auto load = [&](int q0) {
      sq.load(Q, a.q_rs, q0, P.nq);
      sdo.load(dO, a.do_rs, q0, P.nq);
      so.load(O, a.o_rs, q0, P.nq);
      if (threadIdx.x < TS) st = q0 + (int)threadIdx.x < P.nq ? stat[q0 + threadIdx.x] : make_float2(INFINITY, 0.f);
    };
    const int nq = P.nk > 0 ? P.nq : 0;
    if (nq > 0) load(0);
    for (int q0 = 0; q0 < nq; q0 += TS, cur ^= 1) {
      sq.store(Xs[cur]);
      sdo.store(Ys[cur]);
#pragma unroll
      for (int p = 0; p < St::V; ++p) {             // D of the tile's rows: TPR neighbouring lanes hold one
        const float4 x = sdo.r[p], y = so.r[p];
        float t = x.x * y.x + x.y * y.y + x.z * y.z + x.w * y.w;
#pragma unroll
        for (int s = St::TPR / 2; s > 0; s >>= 1) t += __shfl_xor(t, s, 64);
        if (threadIdx.x % St::TPR == 0) s_D[cur][St::row(p)] = sdo.ok[p] ? t : 0.f;
      }
      if (threadIdx.x < TS) s_stat[cur][threadIdx.x] = st;
      lds_barrier();
      if (q0 + TS < nq) load(q0 + TS);
      attn_kv_tile<TS, DH>(Xs[cur], Ys[cur], s_stat[cur], s_D[cur], a.scale, own < P.nk, kf, vf, dk, dv);
    }
    if (own >= a.Sk) return;
    T::put(dk, a.dk + P.z * a.k_bs + P.h * DH + own * a.k_rs);
    T::put(dv, a.dv + P.z * a.v_bs + P.h * DH + own * a.v_rs);
    return;
  }
  float4 qf[T::NQ], of[T::NQ], oo[T::NQ];
  const int qc = min(own, a.Sq - 1);
  T::row_frag(Q + qc * a.q_rs, qf);
  T::row_frag(dO + qc * a.do_rs, of);
  T::row_frag(O + qc * a.o_rs, oo);
  const float2 st = stat[qc];
  St sk, sv;
  if (P.nk > 0) {
    sk.load(K, a.k_rs, 0, P.nk);
    sv.load(Vv, a.v_rs, 0, P.nk);
  }
  const float D = attn_dot<TS, DH>(of, oo);
  typename T::acc_t dq[T::NB] = {};
  for (int k0 = 0; k0 < P.nk; k0 += TS, cur ^= 1) {
    sk.store(Xs[cur]);
    sv.store(Ys[cur]);
    lds_barrier();
    if (k0 + TS < P.nk) {
      sk.load(K, a.k_rs, k0 + TS, P.nk);
      sv.load(Vv, a.v_rs, k0 + TS, P.nk);
    }
    attn_q_tile<TS, DH>(Xs[cur], Ys[cur], st, D, a.scale, P.nk - k0, qf, of, dq);
  }
  if (own < a.Sq) T::put(dq, a.dq + P.z * a.q_bs + P.h * DH + own * a.q_rs);
}

// Sequences of at most TS queries and keys: a wave per (sequence, head), all three gradients.
template <int TS, int DH>
__global__ __launch_bounds__(128) void k_attn_bwd_small(TAttn a) {
  using T = AttnTile<TS, DH>;
  using St = AttnStage<TS, DH, 64>;
  __shared__ __align__(16) float Qs[2][T::SIZE], Os[2][T::SIZE], Ks[2][T::SIZE], Vs[2][T::SIZE];
  __shared__ __align__(16) float2 s_stat[2][TS];
  __shared__ __align__(16) float s_D[2][TS];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pair = 2 * xcd_tile(blockIdx.x, gridDim.x) + wave;
  if (pair >= a.nseq * a.H) return;                 // waves share nothing
  const AttnPair P(a, pair);
  const int c = T::col();
  const float* O = a.o + P.z * a.o_bs + P.h * DH;
  float* dqp = a.dq + P.z * a.q_bs + P.h * DH + c * a.q_rs;
  float* dkp = a.dk + P.z * a.k_bs + P.h * DH + c * a.k_rs;
  float* dvp = a.dv + P.z * a.v_bs + P.h * DH + c * a.v_rs;
  typename T::acc_t dq[T::NB] = {}, dk[T::NB] = {}, dv[T::NB] = {};
  if (P.nq > 0 && P.nk > 0) {
    St sq, so, sk, sv;
    float4 of[T::NQ], oo[T::NQ], f0[T::NQ], f1[T::NQ];
    sq.load(a.q + P.z * a.q_bs + P.h * DH, a.q_rs, 0, P.nq);
    so.load(a.dO + P.z * a.do_bs + P.h * DH, a.do_rs, 0, P.nq);
    sk.load(a.k + P.z * a.k_bs + P.h * DH, a.k_rs, 0, P.nk);
    sv.load(a.v + P.z * a.v_bs + P.h * DH, a.v_rs, 0, P.nk);
    T::row_frag(O + min(c, P.nq - 1) * a.o_rs, oo);
    const float2 st = c < P.nq ? a.stat[((long long)P.z * a.H + P.h) * a.Sq + c] : make_float2(INFINITY, 0.f);
    sq.store(Qs[wave]);
    so.store(Os[wave]);
    sk.store(Ks[wave]);
    sv.store(Vs[wave]);
    wave_sync();
    T::tile_frag(Os[wave], c, of);
    const float D = attn_dot<TS, DH>(of, oo);
    if (T::slot() == 0) {
      s_stat[wave][c] = st;
      s_D[wave][c] = D;
    }
    wave_sync();
    T::tile_frag(Ks[wave], c, f0);
    T::tile_frag(Vs[wave], c, f1);
    attn_kv_tile<TS, DH>(Qs[wave], Os[wave], s_stat[wave], s_D[wave], a.scale, c < P.nk, f0, f1, dk, dv);
    T::tile_frag(Qs[wave], c, f0);
    attn_q_tile<TS, DH>(Ks[wave], Vs[wave], st, D, a.scale, P.nk, f0, of, dq);
  }
  if (c < a.Sq) T::put(dq, dqp);
  if (c < a.Sk) {
    T::put(dk, dkp);
    T::put(dv, dvp);
  }
}

// ------------------------------------------------------------------------------------------
// LayerNorm over rows of d values (biased variance, eps 1e-5): one wave per row.
// ------------------------------------------------------------------------------------------
template <int V>
FE_DEV void ldv(const float* p, float* v) {
  if constexpr (V == 4) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else if constexpr (V == 2) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    v[0] = t.x; v[1] = t.y;
  } else {
    v[0] = *p;
  }
}
template <int V>
FE_DEV void stv(float* p, const float* v) {
  if constexpr (V == 4) *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  else if constexpr (V == 2) *reinterpret_cast<float2*>(p) = make_float2(v[0], v[1]);
  else *p = v[0];
}

// Any d, one wave per row.
__global__ __launch_bounds__(256) void k_ln_fwd(const float* X, long long x_rs, int rows, int d, const float* g,
                                                const float* b, float* Y, long long y_rs, float* mean, float* rstd) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* x = X + row * x_rs;
  float s = 0.f;
  for (int j = lane; j < d; j += 64) s += x[j];
  const float mu = wave_sum(s) / d;
  float q = 0.f;
  for (int j = lane; j < d; j += 64) q += (x[j] - mu) * (x[j] - mu);
  const float rs = rsqrtf(wave_sum(q) / d + 1e-5f);
  float* y = Y + row * y_rs;
  for (int j = lane; j < d; j += 64) y[j] = (x[j] - mu) * rs * g[j] + b[j];
  if (lane == 0) { mean[row] = mu; rstd[row] = rs; }
}

// The same for d = 64 V NC, LN_ROWS rows per wave: a row and the vectors stay in registers (one
// memory round trip instead of one per pass over the row), and the rows' reductions overlap.  A lane
// sums its V adjacent columns of each chunk of 64 V (above: every 64th column) before the tree over
// the lanes, so the order of a row's sums depends on d, and on the alignment that picks the form, but
// not on the number of rows.  Measured, before and after: 35200 x 128 12.9 -> 8.7 us, 16384 x 128 7.4 ->
// 5.7 us.
constexpr int LN_ROWS = 4;
template <int V, int NC>
__global__ __launch_bounds__(256) void k_ln_fwd_rows(const float* X, long long x_rs, int rows, int d, const float* g,
                                                     const float* b, float* Y, long long y_rs, float* mean, float* rstd) {
  const int lane = threadIdx.x & 63, j0 = lane * V;
  const int row0 = (xcd_tile(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6)) * LN_ROWS;
  if (row0 >= rows) return;
  float v[LN_ROWS][NC][V], gv[NC][V], bv[NC][V];
#pragma unroll
  for (int r = 0; r < LN_ROWS; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c) ldv<V>(X + min(row0 + r, rows - 1) * x_rs + j0 + 64 * V * c, v[r][c]);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    ldv<V>(g + j0 + 64 * V * c, gv[c]);
    ldv<V>(b + j0 + 64 * V * c, bv[c]);
  }
  float mu[LN_ROWS], rs[LN_ROWS];
#pragma unroll
  for (int r = 0; r < LN_ROWS; ++r) {
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < V; ++e) s += v[r][c][e];
    mu[r] = wave_sum(s) / d;
  }
#pragma unroll
  for (int r = 0; r < LN_ROWS; ++r) {
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < V; ++e) q = fmaf(v[r][c][e] - mu[r], v[r][c][e] - mu[r], q);
    rs[r] = rsqrtf(wave_sum(q) / d + 1e-5f);
  }
#pragma unroll
  for (int r = 0; r < LN_ROWS; ++r) {
    const int row = row0 + r;
    if (row >= rows) break;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int e = 0; e < V; ++e) v[r][c][e] = fmaf((v[r][c][e] - mu[r]) * rs[r], gv[c][e], bv[c][e]);
      stv<V>(Y + row * y_rs + j0 + 64 * V * c, v[r][c]);
    }
    if (lane == 0) { mean[row] = mu[r]; rstd[row] = rs[r]; }
  }
}

// Backward, d = 64 V NC: dX (+)= rstd (dxh - mean(dxh) - xh mean(dxh xh)) with dxh = dY g and xh the
// normalised input, dg[j] += sum_rows dY xh, db[j] += sum_rows dY.  A wave takes rpw (a multiple of
// LN_ROWS) consecutive rows, LN_ROWS at a time, and keeps its columns' parameter sums in registers;
// the eight waves' sums meet in LDS, one atomic per column and workgroup.  One pass over X, dY and
// dX instead of two over X and dY; bound by memory (35200 x 128: 72 MB).  rpw makes at most 256
// workgroups: more atomics per column are what limits it beyond.  Measured, before (two kernels) and
// after: 35200 x 128 35.9 -> 17.9 us, 16384 x 128 20.7 -> 12.7 us, 385 x 64 8.8 -> 3.5 us.
template <int V, int NC>
__global__ __launch_bounds__(512) void k_ln_bwd(const float* X, long long x_rs, int rows, int d, const float* g,
                                                const float* mean, const float* rstd, const float* dY, long long dy_rs,
                                                float* dX, long long dx_rs, int accumulate, int rpw, float* dg, float* db) {
  constexpr int D = 64 * V * NC;
  __shared__ __align__(16) float part[8][2][D];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j0 = lane * V;
  const int first = (xcd_tile(blockIdx.x, gridDim.x) * 8 + wave) * rpw, last = min(rows, first + rpw);
  float gv[NC][V], sg[NC][V] = {}, sb[NC][V] = {};
#pragma unroll
  for (int c = 0; c < NC; ++c) ldv<V>(g + j0 + 64 * V * c, gv[c]);
  for (int row0 = first; row0 < last; row0 += LN_ROWS) {
    float xh[LN_ROWS][NC][V], dy[LN_ROWS][NC][V], ov[LN_ROWS][NC][V], mu[LN_ROWS], rs[LN_ROWS];
#pragma unroll
    for (int r = 0; r < LN_ROWS; ++r) {
      const int row = min(row0 + r, last - 1);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        ldv<V>(X + row * x_rs + j0 + 64 * V * c, xh[r][c]);
        ldv<V>(dY + row * dy_rs + j0 + 64 * V * c, dy[r][c]);
        if (accumulate) ldv<V>(dX + row * dx_rs + j0 + 64 * V * c, ov[r][c]);
        else
#pragma unroll
          for (int e = 0; e < V; ++e) ov[r][c][e] = 0.f;
      }
      mu[r] = mean[row];
      rs[r] = rstd[row];
    }
#pragma unroll
    for (int r = 0; r < LN_ROWS; ++r) {
      const bool live = row0 + r < last;
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < V; ++e) {
          xh[r][c][e] = (xh[r][c][e] - mu[r]) * rs[r];
          sg[c][e] += live ? dy[r][c][e] * xh[r][c][e] : 0.f;
          sb[c][e] += live ? dy[r][c][e] : 0.f;
          dy[r][c][e] *= gv[c][e];
          s1 += dy[r][c][e];
          s2 += dy[r][c][e] * xh[r][c][e];
        }
      s1 = wave_sum(s1) * (1.f / D);
      s2 = wave_sum(s2) * (1.f / D);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int e = 0; e < V; ++e) ov[r][c][e] += rs[r] * (dy[r][c][e] - s1 - xh[r][c][e] * s2);
        if (live) stv<V>(dX + (row0 + r) * dx_rs + j0 + 64 * V * c, ov[r][c]);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    stv<V>(&part[wave][0][j0 + 64 * V * c], sg[c]);
    stv<V>(&part[wave][1][j0 + 64 * V * c], sb[c]);
  }
  lds_barrier();
  for (int j = threadIdx.x; j < 2 * D; j += 512) {
    const int which = j >= D, col = j % D;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) t += part[w][which][col];
    atomicAdd(&(which ? db : dg)[col], t);
  }
}

// Any d: dX as above, one wave per row ...
__global__ __launch_bounds__(256) void k_ln_bwd_rows(const float* X, long long x_rs, int rows, int d, const float* g,
                                                     const float* mean, const float* rstd, const float* dY,
                                                     long long dy_rs, float* dX, long long dx_rs, int accumulate) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* x = X + row * x_rs;
  const float* dy = dY + row * dy_rs;
  const float mu = mean[row], rs = rstd[row];
  float s1 = 0.f, s2 = 0.f;
  for (int j = lane; j < d; j += 64) {
    const float xh = (x[j] - mu) * rs, dxh = dy[j] * g[j];
    s1 += dxh;
    s2 += dxh * xh;
  }
  s1 = wave_sum(s1) / d;
  s2 = wave_sum(s2) / d;
  float* dx = dX + row * dx_rs;
  for (int j = lane; j < d; j += 64)
    dx[j] = (accumulate ? dx[j] : 0.f) + rs * (dy[j] * g[j] - s1 - (x[j] - mu) * rs * s2);
}

// ... and dg, db: 64 columns x TRAIN_COL_ROWS rows per workgroup, its four waves every fourth row,
// one atomic per column and workgroup.
__global__ __launch_bounds__(256) void k_ln_bwd_params(const float* X, long long x_rs, int rows, int d,
                                                       const float* mean, const float* rstd, const float* dY,
                                                       long long dy_rs, float* dg, float* db) {
  __shared__ float part[2][4][64];
  const int c = threadIdx.x & 63, w = threadIdx.x >> 6, j = blockIdx.x * 64 + c;
  const int r0 = blockIdx.y * TRAIN_COL_ROWS, r1 = min(rows, r0 + TRAIN_COL_ROWS);
  float sg = 0.f, sb = 0.f;
  if (j < d)
    for (int r = r0 + w; r < r1; r += 4) {
      const float dy = dY[r * dy_rs + j];
      sg += dy * (X[r * x_rs + j] - mean[r]) * rstd[r];
      sb += dy;
    }
  part[0][w][c] = sg;
  part[1][w][c] = sb;
  __syncthreads();
  if (w == 0 && j < d) {
    atomicAdd(&dg[j], part[0][0][c] + part[0][1][c] + part[0][2][c] + part[0][3][c]);
    atomicAdd(&db[j], part[1][0][c] + part[1][1][c] + part[1][2][c] + part[1][3][c]);
  }
}

// ------------------------------------------------------------------------------------------
// Elementwise steps over n values.
// ------------------------------------------------------------------------------------------
__global__ void k_copy(const float* x, float* y, long long n) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[i] = x[i];
}
__global__ void k_fill(float* y, long long n, float v) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[i] = v;
}
// Y[b][r] = row idx[b][r] of table T + b*t_bs for r < n (n = nvalid ? nvalid[b] : rows); rows past
// n and ids outside [0, n_table) give zero rows.
__global__ void k_gather(const float* T, long long t_bs, int n_table, const int32_t* idx, int idx_bs,
                         const int32_t* nvalid, int rows, int d, float* Y) {
  const int b = blockIdx.y, r = blockIdx.x;
  const int n = nvalid ? nvalid[b] : rows;
  float* y = Y + ((long long)b * rows + r) * d;
  const int id = r < n ? idx[(long long)b * idx_bs + r] : -1;
  if (id < 0 || id >= n_table) {
    for (int j = threadIdx.x; j < d; j += blockDim.x) y[j] = 0.f;
    return;
  }
  const float* t = T + b * t_bs + (long long)id * d;
  for (int j = threadIdx.x; j < d; j += blockDim.x) y[j] = t[j];
}
// the gather's backward: dT row idx[b][r] += dY[b][r] for the rows the gather read
__global__ void k_scatter_add(const float* dY, const int32_t* idx, int idx_bs, const int32_t* nvalid, int rows,
                              int d, float* dT, long long t_bs, int n_table) {
  const int b = blockIdx.y, r = blockIdx.x;
  const int n = nvalid ? nvalid[b] : rows;
  if (r >= n) return;
  const int id = idx[(long long)b * idx_bs + r];
  if (id < 0 || id >= n_table) return;
  const float* dy = dY + ((long long)b * rows + r) * d;
  float* t = dT + b * t_bs + (long long)id * d;
  for (int j = threadIdx.x; j < d; j += blockDim.x) atomicAdd(&t[j], dy[j]);
}

// seq[b][k][0] = cls + pos[0]; seq[b][k][j+1] = H[b][slot[b][k][j]] + pos[j+1] (Section 4.3)
__global__ void k_assemble_f32(const float* H, int U_cap, const int32_t* slot, int K, int L, int d, const float* cls,
                               const float* pos, float* seq) {
  const int b = blockIdx.z, k = blockIdx.y, j = blockIdx.x;   // j = 0..L
  float* o = seq + (((long long)b * K + k) * (L + 1) + j) * d;
  const int sl = j == 0 ? 0 : slot[((long long)b * K + k) * L + j - 1];
  const float* src = j == 0 ? cls : H + ((long long)b * U_cap + sl) * d;
  // an entry outside the pool (slot -1) gives a zero row, as in the inference assembly
  for (int e = threadIdx.x; e < d; e += blockDim.x) o[e] = sl >= 0 ? src[e] + pos[(long long)j * d + e] : 0.f;
}
// the assembly's backward, element rows: dH[b][slot] += dseq rows (a distinct element's row receives
// the sum over its occurrences)
__global__ void k_assemble_bwd(const float* dseq, int U_cap, const int32_t* slot, int K, int L, int d, float* dH) {
  const int b = blockIdx.z, k = blockIdx.y, j = blockIdx.x + 1;
  const float* g = dseq + (((long long)b * K + k) * (L + 1) + j) * d;
  const int sl = slot[((long long)b * K + k) * L + j - 1];
  if (sl < 0) return;
  float* dst = dH + ((long long)b * U_cap + sl) * d;
  for (int e = threadIdx.x; e < d; e += blockDim.x) atomicAdd(&dst[e], g[e]);
}

// ... and positions and [CLS]: dpos[c] += sum over the B K sequences of dseq[.][c] for the (L+1) d
// entries c of a sequence, dcls[e] += the same sums of row 0; the zero rows of entries outside the
// pool (slot -1) carry no position and add nothing.  64 entries x TRAIN_COL_ROWS sequences per
// workgroup, one atomic per entry and workgroup.
__global__ __launch_bounds__(256) void k_assemble_bwd_pos(const float* dseq, const int32_t* slot, int L, int nseq,
                                                          int cols, int d, float* dpos, float* dcls) {
  __shared__ float part[4][64];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63), w = threadIdx.x >> 6;
  const int r0 = blockIdx.y * TRAIN_COL_ROWS, r1 = min(nseq, r0 + TRAIN_COL_ROWS);
  const int j = c / d;                                   // row of the sequence: 0 [CLS], 1..L entries
  float sum = 0.f;
  if (c < cols)
    for (int r = r0 + w; r < r1; r += 4)
      if (j == 0 || slot[(long long)r * L + j - 1] >= 0) sum += dseq[(long long)r * cols + c];
  part[w][threadIdx.x & 63] = sum;
  __syncthreads();
  if (w == 0 && c < cols) {
    const float t = part[0][threadIdx.x] + part[1][threadIdx.x] + part[2][threadIdx.x] + part[3][threadIdx.x];
    atomicAdd(&dpos[c], t);
    if (c < d) atomicAdd(&dcls[c], t);
  }
}

// Loss of request b (Section 4.5) with its labels (Appendix B.1): r_k = sum_j relevant[b][l_kj],
// y = min argmax r_k; MSE target r_k, BCE target r_k / L.  Adds loss_b / B to *loss and writes
// dscores[b][k] = (1/B) dloss_b / ds_k.  One workgroup per request, K <= 1024.
__global__ __launch_bounds__(256) void k_loss(const float* s, const int32_t* lists, const int32_t* relevant, int M,
                                              int B, int K, int L, int kind, float* loss, float* ds) {
  __shared__ int sr[1024];
  __shared__ float red[256];
  __shared__ int sy;
  const int b = blockIdx.x;
  const float* sb = s + (long long)b * K;
  for (int k = threadIdx.x; k < K; k += 256) {
    int r = 0;
    for (int j = 0; j < L; ++j) {
      const int e = lists[((long long)b * K + k) * L + j];
      r += (e >= 0 && e < M) ? relevant[(long long)b * M + e] : 0;
    }
    sr[k] = r;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int y = 0;
    for (int k = 1; k < K; ++k) if (sr[k] > sr[y]) y = k;
    sy = y;
  }
  __syncthreads();
  // CE needs max and sum of exp over the K scores
  float mx = -INFINITY;
  for (int k = threadIdx.x; k < K; k += 256) mx = fmaxf(mx, sb[k]);
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + o]);
    __syncthreads();
  }
  mx = red[0];
  __syncthreads();
  float part = 0.f;
  for (int k = threadIdx.x; k < K; k += 256) part += expf(sb[k] - mx);
  red[threadIdx.x] = part;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  const float sumexp = red[0];
  __syncthreads();
  float lpart = 0.f;
  for (int k = threadIdx.x; k < K; k += 256) {
    const float sk = sb[k];
    float l = 0.f, g = 0.f;
    if (kind == TRAIN_MSE) {
      const float t = (float)sr[k];
      l = (sk - t) * (sk - t) / K;
      g = 2.f * (sk - t) / K;
    } else if (kind == TRAIN_BCE) {
      const float t = (float)sr[k] / L;
      // t softplus(-s) + (1 - t) softplus(s), softplus(v) = max(v, 0) + log1p(exp(-|v|))
      const float sp_pos = fmaxf(sk, 0.f) + log1pf(expf(-fabsf(sk)));
      const float sp_neg = fmaxf(-sk, 0.f) + log1pf(expf(-fabsf(sk)));
      l = (t * sp_neg + (1.f - t) * sp_pos) / K;
      g = (1.f / (1.f + expf(-sk)) - t) / K;
    } else {
      const float p = expf(sk - mx) / sumexp;
      g = p - (k == sy ? 1.f : 0.f);
      if (k == sy) l = -(sk - mx - logf(sumexp));
    }
    lpart += l;
    ds[(long long)b * K + k] = g / B;
  }
  red[threadIdx.x] = lpart;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(loss, red[0] / B);
}

inline unsigned blocks(long long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

template <int WM, int WN, bool AK, bool BK, bool VA, bool VB>
void gemm_launch(const TGemm& g, int chunks, hipStream_t s) {
  constexpr int TM = 32 * WM, TN = 32 * WN;
  const int tiles_n = (g.N + TN - 1) / TN, tiles = tiles_n * ((g.M + TM - 1) / TM);
  const int per = std::max(1, (1 << 22) / tiles);   // k chunks per launch
  for (int c = 0; c < chunks; c += per)
    hipLaunchKernelGGL((k_gemm<WM, WN, AK, BK, VA, VB>), dim3((unsigned)(std::min(per, chunks - c) * tiles)), dim3(256), 0, s, g,
                       c, tiles_n, tiles);
}

// float4 loads of an operand are possible when its base and every stride but the contiguous one
// are multiples of four floats (so every group of four along the contiguous index is aligned) and so
// is the extent of the contiguous index (so no group is cut)
inline bool vec4(const float* p, long long other_stride, int extent) {
  return reinterpret_cast<uintptr_t>(p) % 16 == 0 && other_stride % 4 == 0 && extent % 4 == 0;
}

template <int WM, int WN, bool AK, bool BK>
void gemm_vec(const TGemm& g, int chunks, hipStream_t s) {
  const bool va = vec4(g.A, AK ? g.a_rs : g.a_cs, AK ? g.K : g.M) && (AK ? g.a_cs == 1 : g.a_rs == 1);
  const bool vb = vec4(g.B, BK ? g.b_cs : g.b_rs, BK ? g.K : g.N) && (BK ? g.b_rs == 1 : g.b_cs == 1);
  if (va && vb) gemm_launch<WM, WN, AK, BK, true, true>(g, chunks, s);
  else if (va) gemm_launch<WM, WN, AK, BK, true, false>(g, chunks, s);
  else if (vb) gemm_launch<WM, WN, AK, BK, false, true>(g, chunks, s);
  else gemm_launch<WM, WN, AK, BK, false, false>(g, chunks, s);
}

template <int WM, int WN>
void gemm_orient(const TGemm& g, int chunks, hipStream_t s) {
  const bool ak = g.a_cs == 1 && g.a_rs != 1, bk = g.b_rs == 1 && g.b_cs != 1;
  if (ak && bk) gemm_vec<WM, WN, true, true>(g, chunks, s);
  else if (ak) gemm_vec<WM, WN, true, false>(g, chunks, s);
  else if (bk) gemm_vec<WM, WN, false, true>(g, chunks, s);
  else gemm_vec<WM, WN, false, false>(g, chunks, s);
}

hipError_t t_gemm(const TGemm& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.ksplit > 0 && (g.beta != 1.f || g.bias || g.R || g.relu || g.mask || g.ksplit % GK)) return hipErrorInvalidValue;
  // a tile's byte offsets are 32-bit (at most 128 rows and 32 k values of either operand)
  for (long long st : {g.a_rs, g.a_cs, g.b_rs, g.b_cs})
    if (st < 0 || st > (1 << 21)) return hipErrorInvalidValue;
  const int chunks = g.ksplit > 0 ? (g.K + g.ksplit - 1) / g.ksplit : 1;
  if (g.N <= 32) {
    gemm_orient<4, 1>(g, chunks, s);                 // 128 x 32 tiles (the head)
  } else {
    gemm_orient<2, 2>(g, chunks, s);                 // 64 x 64 tiles
  }
  return hipGetLastError();
}

// d whose rows the register forms cover, with every pointer and row stride aligned to their loads:
// the values V per load (d = 64, 128, 256 in one, 512 in two), else 0
inline int ln_width(int d, std::initializer_list<const void*> ptrs, std::initializer_list<long long> strides) {
  const int V = d == 64 ? 1 : d == 128 ? 2 : d == 256 || d == 512 ? 4 : 0;
  if (!V) return 0;
  for (const void* p : ptrs)
    if (reinterpret_cast<uintptr_t>(p) % (4 * V)) return 0;
  for (long long st : strides)
    if (st % V) return 0;
  return V;
}

hipError_t t_ln_fwd(const float* X, long long x_rs, int rows, int d, const float* g, const float* b, float* Y,
                    long long y_rs, float* mean, float* rstd, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const dim3 grid((unsigned)((rows + 4 * LN_ROWS - 1) / (4 * LN_ROWS)));
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, X, x_rs, rows, d, g, b, Y, y_rs, mean, rstd); };
  switch (ln_width(d, {X, g, b, Y}, {x_rs, y_rs})) {
    case 1: go(k_ln_fwd_rows<1, 1>); break;
    case 2: go(k_ln_fwd_rows<2, 1>); break;
    case 4: if (d == 256) go(k_ln_fwd_rows<4, 1>); else go(k_ln_fwd_rows<4, 2>); break;
    default: hipLaunchKernelGGL(k_ln_fwd, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, X, x_rs, rows, d, g, b, Y, y_rs, mean, rstd);
  }
  return hipGetLastError();
}

hipError_t t_ln_bwd(const float* X, long long x_rs, int rows, int d, const float* g, const float* mean,
                    const float* rstd, const float* dY, long long dy_rs, float* dX, long long dx_rs, bool accumulate,
                    float* dg, float* db, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int V = ln_width(d, {X, g, dY, dX}, {x_rs, dy_rs, dx_rs});
  if (V) {
    const int rpw = (rows + 8 * 256 * LN_ROWS - 1) / (8 * 256 * LN_ROWS) * LN_ROWS;
    const dim3 grid((unsigned)((rows + 8 * rpw - 1) / (8 * rpw)));
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, grid, dim3(512), 0, s, X, x_rs, rows, d, g, mean, rstd, dY, dy_rs, dX, dx_rs, (int)accumulate, rpw, dg, db);
    };
    if (V == 1) go(k_ln_bwd<1, 1>);
    else if (V == 2) go(k_ln_bwd<2, 1>);
    else if (d == 256) go(k_ln_bwd<4, 1>);
    else go(k_ln_bwd<4, 2>);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_ln_bwd_rows, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, X, x_rs, rows, d, g, mean, rstd, dY, dy_rs, dX, dx_rs, (int)accumulate);
  hipLaunchKernelGGL(k_ln_bwd_params, dim3((unsigned)((d + 63) / 64), (unsigned)((rows + TRAIN_COL_ROWS - 1) / TRAIN_COL_ROWS)),
                     dim3(256), 0, s, X, x_rs, rows, d, mean, rstd, dY, dy_rs, dg, db);
  return hipGetLastError();
}

template <int DH>
hipError_t attn_fwd_dh(const TAttn& a, hipStream_t s) {
  const long long pairs = (long long)a.nseq * a.H;
  const dim3 grid((unsigned)(pairs * ((a.Sq + 127) / 128)));
  const dim3 small((unsigned)((pairs + 3) / 4));
  const int most = std::max(a.Sq, a.Sk);
  if (most <= 16) hipLaunchKernelGGL((k_attn_fwd<16, DH, 1, true>), small, dim3(256), 0, s, a);
  else if (most <= 32) hipLaunchKernelGGL((k_attn_fwd<32, DH, 1, true>), small, dim3(256), 0, s, a);
  else if (a.Sk <= 256) hipLaunchKernelGGL((k_attn_fwd<32, DH, 8, false>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_attn_fwd<32, DH, 0, false>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}
template <int DH>
hipError_t attn_bwd_dh(const TAttn& a, hipStream_t s) {
  const int most = std::max(a.Sq, a.Sk);
  const long long pairs = (long long)a.nseq * a.H;
  const dim3 small((unsigned)((pairs + 1) / 2));
  if (most <= 16) {
    hipLaunchKernelGGL((k_attn_bwd_small<16, DH>), small, dim3(128), 0, s, a);
  } else if (most <= 32) {
    hipLaunchKernelGGL((k_attn_bwd_small<32, DH>), small, dim3(128), 0, s, a);
  } else {
    const int n_kv = (int)(pairs * ((a.Sk + 127) / 128));
    hipLaunchKernelGGL((k_attn_bwd<32, DH>), dim3((unsigned)(n_kv + pairs * ((a.Sq + 127) / 128))), dim3(256), 0, s, a, n_kv);
  }
  return hipGetLastError();
}

// every row of every head at a 16-byte boundary
inline bool attn_ok(const TAttn& a) {
  for (long long st : {a.q_rs, a.k_rs, a.v_rs, a.o_rs, a.q_bs, a.k_bs, a.v_bs, a.o_bs})
    if (st % 4) return false;
  return (a.dh == 32 || a.dh == 64) && a.Sq > 0 && a.Sk > 0;
}

hipError_t t_attn_fwd(const TAttn& a, hipStream_t s) {
  if (a.nseq <= 0) return hipSuccess;
  if (!attn_ok(a)) return hipErrorInvalidValue;
  return a.dh == 32 ? attn_fwd_dh<32>(a, s) : attn_fwd_dh<64>(a, s);
}
hipError_t t_attn_bwd(const TAttn& a, hipStream_t s) {
  if (a.nseq <= 0) return hipSuccess;
  if (!attn_ok(a) || a.do_rs % 4 || a.do_bs % 4) return hipErrorInvalidValue;
  return a.dh == 32 ? attn_bwd_dh<32>(a, s) : attn_bwd_dh<64>(a, s);
}

hipError_t t_copy(const float* x, float* y, long long n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_copy, dim3(blocks(n)), dim3(256), 0, s, x, y, n);
  return hipGetLastError();
}
hipError_t t_fill(float* y, long long n, float v, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_fill, dim3(blocks(n)), dim3(256), 0, s, y, n, v);
  return hipGetLastError();
}
hipError_t t_gather(const float* T, long long t_bs, int n_table, const int32_t* idx, int idx_bs, const int32_t* nvalid,
                    int B, int rows, int d, float* Y, hipStream_t s) {
  if (B <= 0 || rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather, dim3((unsigned)rows, (unsigned)B), dim3(128), 0, s, T, t_bs, n_table, idx, idx_bs, nvalid,
                     rows, d, Y);
  return hipGetLastError();
}
hipError_t t_scatter_add(const float* dY, const int32_t* idx, int idx_bs, const int32_t* nvalid, int B, int rows, int d,
                         float* dT, long long t_bs, int n_table, hipStream_t s) {
  if (B <= 0 || rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_add, dim3((unsigned)rows, (unsigned)B), dim3(128), 0, s, dY, idx, idx_bs, nvalid, rows, d,
                     dT, t_bs, n_table);
  return hipGetLastError();
}
hipError_t t_assemble(const float* H, int B, int U_cap, const int32_t* slot, int K, int L, int d, const float* cls,
                      const float* pos, float* seq, hipStream_t s) {
  hipLaunchKernelGGL(k_assemble_f32, dim3((unsigned)(L + 1), (unsigned)K, (unsigned)B), dim3(128), 0, s, H, U_cap, slot, K,
                     L, d, cls, pos, seq);
  return hipGetLastError();
}
hipError_t t_assemble_bwd(const float* dseq, int B, int U_cap, const int32_t* slot, int K, int L, int d, float* dH,
                          float* dcls, float* dpos, hipStream_t s) {
  if (L > 0)
    hipLaunchKernelGGL(k_assemble_bwd, dim3((unsigned)L, (unsigned)K, (unsigned)B), dim3(128), 0, s, dseq, U_cap, slot, K,
                       L, d, dH);
  const int nseq = B * K, cols = (L + 1) * d;
  hipLaunchKernelGGL(k_assemble_bwd_pos, dim3((unsigned)((cols + 63) / 64), (unsigned)((nseq + TRAIN_COL_ROWS - 1) / TRAIN_COL_ROWS)),
                     dim3(256), 0, s, dseq, slot, L, nseq, cols, d, dpos, dcls);
  return hipGetLastError();
}
hipError_t t_loss(const float* scores, const int32_t* lists, const int32_t* relevant, int M, int B, int K, int L, int kind,
                  float* loss, float* dscores, hipStream_t s) {
  if (K > 1024) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_loss, dim3((unsigned)B), dim3(256), 0, s, scores, lists, relevant, M, B, K, L, kind, loss, dscores);
  return hipGetLastError();
}
