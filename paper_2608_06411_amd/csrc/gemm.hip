// Matrix-core GEMM for the predictor projections and the cosine Gram matrix.
//
// C = epilogue(A * B^T) with A [M][K] and B [N][K] both K-contiguous, which is
// the layout of every contraction on the path: token rows times weight rows
// (torch.nn.Linear layout) and token rows times token rows (the Gram matrix).
//
// Tiling for gfx950: a 256-thread workgroup computes a 128x128 tile; its four
// wave64s each own a 64x64 quarter made of 2x2 MFMA 32x32 blocks
// (v_mfma_f32_32x32x16_bf16 for bf16, v_mfma_f32_32x32x2_f32 for float32),
// accumulating in float32.  K advances in 128-byte slices (64 bf16 or 32
// floats per row) that are staged through LDS with a two-slot ring: the next
// slice is fetched into registers while the matrix cores consume the current
// one.  LDS rows are 8 chunks of 16 bytes, XOR-swizzled by (row >> 1) & 7 so that
// the 32 rows one MFMA operand read touches land in different banks.
//
// Several independent problems (for example the first layer of f_V, the
// first layer of f_T and the Gram matrix, which all stream the same visual
// tokens) run in one launch so that the 256 compute units are filled even at
// batch 1.  Workgroups are dispatched round-robin over the 8 XCDs; the block
// index is remapped so that consecutive tiles of a problem run on the same
// XCD and share its L2.
#include "internal.h"

namespace mapk {

namespace {

constexpr int BM = 128;
constexpr int BN = 128;
constexpr int NT = 256;
constexpr int kXcds = 8;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

template <typename T> struct Slice;
template <> struct Slice<bf16_t> { static constexpr int VEC = 8; static constexpr int BK = 64; };
template <> struct Slice<float> { static constexpr int VEC = 4; static constexpr int BK = 32; };

// LDS rows of a K slice are 8 chunks of 16 bytes; chunk c of row r sits at
// position c ^ swz(r).  Sixteen consecutive rows (the lanes one 16-byte LDS
// access serves together) then put a given chunk in 16 distinct 16-byte slots
// of the 256-byte bank window, so the operand reads are free of bank conflicts.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Block index -> tile index such that the tiles run by one XCD are contiguous.
__device__ __forceinline__ int xcd_remap(int b, int total) {
  const int per = total / kXcds, rem = total % kXcds;
  const int x = b % kXcds, local = b / kXcds;
  return x * per + min(x, rem) + local;
}

// erf by Abramowitz and Stegun, Handbook of Mathematical Functions, formula
// 7.1.26: for x >= 0, erf(x) = 1 - (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) e^(-x^2)
// with t = 1 / (1 + p x), absolute error at most 1.5e-7 (6e-7 in float32),
// far below the bfloat16 rounding of the layer's output; erf is odd.  One
// reciprocal, one exponential and five fused multiply-adds, no branches.
__device__ __forceinline__ float erf_as(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  const float poly =
      t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
  return copysignf(fmaf(-poly, __expf(-ax * ax), 1.0f), x);
}

__device__ __forceinline__ float gelu_erf(float x) {
  return 0.5f * x * (1.0f + erf_as(x * 0.70710678118654752f));
}

// d/dx [x Phi(x)] = Phi(x) + x phi(x), with Phi from the same erf.
__device__ __forceinline__ float gelu_erf_grad(float x) {
  return fmaf(x * 0.39894228040143268f, __expf(-0.5f * x * x), 0.5f * (1.0f + erf_as(x * 0.70710678118654752f)));
}

template <typename T>
__device__ __forceinline__ void mma_slice(const uint4 (*As)[8], const uint4 (*Bs)[8], int wm, int wn,
                                          int lane, f32x16_t (&acc)[2][2]);

template <>
__device__ __forceinline__ void mma_slice<bf16_t>(const uint4 (*As)[8], const uint4 (*Bs)[8], int wm,
                                                  int wn, int lane, f32x16_t (&acc)[2][2]) {
  // The operands of step s + 1 are read into the other register set before
  // the products of step s issue, so the LDS latency runs under them (the
  // scheduling barriers keep the two sets apart).
  const int lr = lane & 31, lh = lane >> 5;
  bf16x8_t a[2][2], b[2][2];
  auto read = [&](int s, int buf) {
    const int v = 2 * s + lh;  // 16-byte chunk: k = 16 s + 8 lh + (0..7)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = wm * 64 + i * 32 + lr;
      a[buf][i] = __builtin_bit_cast(bf16x8_t, As[r][v ^ swz(r)]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = wn * 64 + j * 32 + lr;
      b[buf][j] = __builtin_bit_cast(bf16x8_t, Bs[r][v ^ swz(r)]);
    }
  };
  read(0, 0);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s < 3) read(s + 1, (s + 1) & 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s & 1][i], b[s & 1][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <>
__device__ __forceinline__ void mma_slice<float>(const uint4 (*As)[8], const uint4 (*Bs)[8], int wm,
                                                 int wn, int lane, f32x16_t (&acc)[2][2]) {
  const int lr = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int v = 4 * lh + g;  // lane half lh covers k = 16 lh + 4 g + (0..3)
    float4 a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = wm * 64 + i * 32 + lr;
      a[i] = __builtin_bit_cast(float4, As[r][v ^ swz(r)]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = wn * 64 + j * 32 + lr;
      b[j] = __builtin_bit_cast(float4, Bs[r][v ^ swz(r)]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
  }
}

// Row and column of accumulator register r of lane `lane` in a 32x32 block.
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
__device__ __forceinline__ int acc_col(int lane) { return lane & 31; }

// The problem that holds `tile`, and the tile's number in it.
__device__ __forceinline__ int find_problem(const GemmBatch& args, int tile, int& local) {
  int pi = 0, begin = 0;
#pragma unroll
  for (int q = 1; q < kMaxGemmProblems; ++q)
    if (q < args.count && tile >= args.begin[q]) {
      pi = q;
      begin = args.begin[q];
    }
  local = tile - begin;
  return pi;
}

// Block index -> tile: the launch's classes of tiles (up to first_tiles, up to
// last_tiles, the rest) one after the other, each XCD-contiguous.
__device__ __forceinline__ int class_tile(const GemmBatch& args, int b) {
  const int f = args.first_tiles, h = args.last_tiles;
  const int lo = b < f ? 0 : b < h ? f : h, hi = b < f ? f : b < h ? h : args.total_tiles;
  return lo + xcd_remap(b - lo, hi - lo);
}

// Workgroup -> (problem, batch item, tile row, tile column).
// A problem split over K (ksplit > 1) runs its tiles once per K range kc,
// the ranges outermost, so that concurrent tiles read the same K columns.
__device__ __forceinline__ void decode_tile(const GemmBatch& args, int& pi, int& bt, int& tm, int& tn, int& kc,
                                            int& local) {
  const int tile = class_tile(args, blockIdx.x);
  pi = find_problem(args, tile, local);
  const GemmProblem& P = args.p[pi];
  bt = local / P.tiles_per_batch;
  int tt = local - bt * P.tiles_per_batch;
  kc = tt / P.tiles_tri;
  tt -= kc * P.tiles_tri;
  if (P.triangular) {  // upper triangle, row by row: row tm holds tiles_n - tm tiles
    tm = 0;
    while (tt >= P.tiles_n - tm) { tt -= P.tiles_n - tm; ++tm; }
    tn = tm + tt;
  } else {
    tm = tt / P.tiles_n;
    tn = tt - tm * P.tiles_n;
  }
}

// Epilogues on a tile of 64 IB x 64 JB, four waves (wm, wn) of 32 IB x 32 JB.
// The RoPE epilogue (128 x 128 tiles only) stages the tile through LDS: rows
// 0..63 in tile_lo, rows 64..127 in tile_hi (64 x 128 floats each).
// 128 x 128 tiles form row and column where they use them: with the wave's
// first row and column formed ahead, as 64 x 64 tiles have it, the compiler's
// register allocation makes the register-staged kernel's tiles slower (3 x 1225
// rows of 1160 with GELU 36 -> 40 us, 2880 of 4104 78 -> 84).
template <typename T, int IB, int JB>
__device__ __forceinline__ void epilogue(const GemmProblem& P, int bt, int tm, int tn, f32x16_t (&acc)[IB][JB],
                                         float* tile_lo, float* tile_hi, int tid, int lane, int wm, int wn) {
  const int M = P.M, N = P.N;
  const int m0 = tm * 64 * IB, n0 = tn * 64 * JB;
  const int wr = m0 + wm * 32 * IB, wc = n0 + wn * 32 * JB;  // this wave's first row and column
  auto row_at = [&](int i) { return IB == 1 ? wr : m0 + wm * (32 * IB) + i * 32; };
  auto col_at = [&](int j) { return JB == 1 ? wc : n0 + wn * (32 * JB) + j * 32; };
  if (epi_direct(P.epi)) {
    const int e = P.epi;
    const T* __restrict__ bias = static_cast<const T*>(P.bias);
    const long long base = bt * P.strideC;
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int col = col_at(j) + acc_col(lane);
      if (col >= N) continue;
      const float bv = (e == EPI_GELU2 && bias) ? to_f32<T>(bias[col]) : 0.0f;
#pragma unroll
      for (int i = 0; i < IB; ++i) {
        // the factor or residual of all 16 entries first (clamped rows), so
        // that no load waits behind this lane's stores
        float f[16];
        if (e == EPI_MUL || e == EPI_RESID) {
          const T* __restrict__ aux = static_cast<const T*>(P.aux) + base;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = min(row_at(i) + acc_row(r, lane), M - 1);
            f[r] = to_f32<T>(aux[(long long)row * P.ldc + col]);
          }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row_at(i) + acc_row(r, lane);
          if (row >= M) continue;
          const long long at = base + (long long)row * P.ldc + col;
          const float v = acc[i][j][r] + bv;
          if (e == EPI_F32) {
            static_cast<float*>(P.C)[at] = v;
          } else if (e == EPI_GELU2) {
            static_cast<T*>(P.C)[at] = from_f32<T>(gelu_erf(v));
            static_cast<T*>(P.aux)[at] = from_f32<T>(gelu_erf_grad(v));
          } else if (e == EPI_MUL) {
            static_cast<T*>(P.C)[at] = from_f32<T>(v * f[r]);
          } else {
            static_cast<T*>(P.C)[at] = from_f32<T>(v + f[r]);
          }
        }
      }
    }
  } else if (P.epi == EPI_BIAS_GELU || P.epi == EPI_BIAS) {
    T* __restrict__ C = static_cast<T*>(P.C) + bt * P.strideC;
    const T* __restrict__ bias = static_cast<const T*>(P.bias);
    const bool gelu = P.epi == EPI_BIAS_GELU;
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int col = col_at(j) + acc_col(lane);
      if (col >= N) continue;
      const float bv = bias ? to_f32<T>(bias[col]) : 0.0f;
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row_at(i) + acc_row(r, lane);
          if (row >= M) continue;
          float v = acc[i][j][r] + bv;
          if (gelu) v = gelu_erf(v);
          C[(long long)row * P.ldc + col] = from_f32<T>(v);
        }
    }
  } else if (P.epi == EPI_COSINE) {
    // Upper-triangle tiles only.  Each value is written to (row, col) and to
    // (col, row), so S is bitwise symmetric; inside a diagonal tile only the
    // entries with row <= col are taken from the accumulators.
    float* __restrict__ S = static_cast<float*>(P.C) + bt * P.strideC;
    const float* __restrict__ rs = P.rs + (long long)bt * M;
    const bool diag = tm == tn;
    const bool vec4 = (P.ldc & 3) == 0;
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int col = col_at(j) + acc_col(lane);
      if (col >= N) continue;
      const float sc = rs[col];
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row0 = row_at(i) + 8 * q + 4 * (lane >> 5);
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int row = row0 + e;
            v[e] = row < M ? acc[i][j][4 * q + e] * (rs[row] * sc) : 0.0f;
            if (row < M && (!diag || row <= col)) S[(long long)row * P.ldc + col] = v[e];
          }
          float* dst = S + (long long)col * P.ldc + row0;  // S[col][row0 .. row0 + 3]
          if (!diag && vec4 && row0 + 3 < M) {
            *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (row0 + e < M && (!diag || row0 + e < col)) dst[e] = v[e];
          }
        }
    }
  } else if constexpr (IB == 2 && JB == 2) {  // EPI_ROPE: stage the tile (plus the bias) in LDS so each thread sees both halves of a pair
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int cl = wn * 64 + j * 32 + acc_col(lane);
      const float bv = (P.rope_bias && n0 + cl < N) ? P.rope_bias[n0 + cl] : 0.0f;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int rl = wm * 64 + i * 32 + acc_row(r, lane);
          (rl < 64 ? tile_lo : tile_hi)[(rl & 63) * BN + cl] = acc[i][j][r] + bv;
        }
    }
    __syncthreads();
    float* __restrict__ out = static_cast<float*>(P.C) + bt * P.strideC;
    const int half = N >> 1;
    if ((half & 3) == 0 && (P.ldc & 3) == 0) {
      // four pairs per item; each thread issues all its cos/sin loads first
      const int q4 = half >> 2, items = BM * q4;
      for (int e0 = tid; e0 < items; e0 += 8 * NT) {
        float4 cs[8][2];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int e = e0 + u * NT, rl = e / q4, c = 4 * (e - rl * q4);
          const bool ok = e < items && m0 + rl < M;
          const float4* src = reinterpret_cast<const float4*>(P.rope_cs + (long long)(ok ? m0 + rl : 0) * half + c);
          cs[u][0] = ok ? src[0] : make_float4(0.f, 0.f, 0.f, 0.f);
          cs[u][1] = ok ? src[1] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int e = e0 + u * NT, rl = e / q4, c = 4 * (e - rl * q4);
          const int row = m0 + rl;
          if (e >= items || row >= M) continue;
          const float* tr = (rl < 64 ? tile_lo : tile_hi) + (rl & 63) * BN;
          const float4 a = *reinterpret_cast<const float4*>(tr + c);
          const float4 b = *reinterpret_cast<const float4*>(tr + c + half);
          const float4 c0 = cs[u][0], c1 = cs[u][1];  // (cos, sin) of pairs c, c+1 | c+2, c+3
          float* o = out + (long long)row * P.ldc + c;
          *reinterpret_cast<float4*>(o) = make_float4(a.x * c0.x - b.x * c0.y, a.y * c0.z - b.y * c0.w,
                                                      a.z * c1.x - b.z * c1.y, a.w * c1.z - b.w * c1.w);
          *reinterpret_cast<float4*>(o + half) = make_float4(b.x * c0.x + a.x * c0.y, b.y * c0.z + a.y * c0.w,
                                                             b.z * c1.x + a.z * c1.y, b.w * c1.z + a.w * c1.w);
        }
      }
      return;
    }
    for (int e = tid; e < BM * half; e += NT) {
      const int rl = e / half, c = e - rl * half;
      const int row = m0 + rl;
      if (row >= M) continue;
      const float* tr = (rl < 64 ? tile_lo : tile_hi) + (rl & 63) * BN;
      const float a = tr[c], b = tr[c + half];
      const float2 cs = P.rope_cs[(long long)row * half + c];
      out[(long long)row * P.ldc + c] = a * cs.x - b * cs.y;
      out[(long long)row * P.ldc + c + half] = b * cs.x + a * cs.y;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(NT) void gemm_kernel(const GemmBatch args) {
  // One contiguous 64 KiB block: A slices in [0, 2), B slices in [2, 4); the
  // RoPE epilogue reuses all of it as a 128 x 128 float tile.
  __shared__ uint4 smem[4][BM][8];
  uint4 (*As)[BM][8] = smem;
  uint4 (*Bs)[BM][8] = smem + 2;
  constexpr int VEC = Slice<T>::VEC;
  constexpr int BK = Slice<T>::BK;

  int pi, bt, tm, tn, kc, local;
  decode_tile(args, pi, bt, tm, tn, kc, local);
  const GemmProblem& P = args.p[pi];
  if (P.run_if && P.run_if[bt] == 0) return;  // (index maps and K ranges: direct-load kernel only)
  const int M = P.M, N = P.N, K = P.K;
  const T* __restrict__ A = static_cast<const T*>(P.A) + bt * P.strideA;
  const T* __restrict__ B = static_cast<const T*>(P.B) + bt * P.strideB;
  const int m0 = tm * BM, n0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int lv = tid & 7;          // 16-byte chunk this thread moves
  const int lrow = tid >> 3;       // first row this thread moves (then +32, +64, +96)

  uint4 ra[4], rb[4];
  auto fetch = [&](int k0) {
    const int gk = k0 + lv * VEC;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = lrow + 32 * j;
      const int gm = m0 + r, gn = n0 + r;
      ra[j] = (gm < M && gk < K) ? *reinterpret_cast<const uint4*>(A + (long long)gm * P.lda + gk)
                                 : make_uint4(0, 0, 0, 0);
      rb[j] = (gn < N && gk < K) ? *reinterpret_cast<const uint4*>(B + (long long)gn * P.ldb + gk)
                                 : make_uint4(0, 0, 0, 0);
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = lrow + 32 * j;
      As[buf][r][lv ^ swz(r)] = ra[j];
      Bs[buf][r][lv ^ swz(r)] = rb[j];
    }
  };

  f32x16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  const int nk = (K + BK - 1) / BK;
  fetch(0);
  stash(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const bool more = kt + 1 < nk;
    if (more) fetch((kt + 1) * BK);
    mma_slice<T>(As[kt & 1], Bs[kt & 1], wm, wn, lane, acc);
    if (more) stash((kt + 1) & 1);
    __syncthreads();
  }

  __syncthreads();  // the RoPE epilogue reuses the LDS tiles
  epilogue<T, 2, 2>(P, bt, tm, tn, acc, reinterpret_cast<float*>(&smem[0][0][0]),
              reinterpret_cast<float*>(&smem[2][0][0]), tid, lane, wm, wn);
}

// Staged epilogues of the direct-load kernel.  After the main loop the four
// 32 KiB stage arrays are free; the finished tile goes through them so that
// every global store moves 16 bytes per lane along a row.
//   q0, q1: the tile in row-major order (rows 0..63 in q0, 64..127 in q1),
//           128 floats per row;
//   t0, t1: the tile transposed (tile columns 0..63 in t0, 64..127 in t1),
//           one tile column per 128-float row whose 16-byte chunks are
//           XOR-swizzled by the column (chunk r/4 at position r/4 ^ (c & 31)),
//           so both the staging writes and the row reads avoid bank conflicts.
struct StagedTile {
  float* q0;
  float* q1;
  float* t0;
  float* t1;
  __device__ float* row(int r) const { return (r < 64 ? q0 : q1) + (r & 63) * BN; }
  // chunk holding tile entries (4 ch .. 4 ch + 3, c), i.e. rows 4 ch .. of column c
  __device__ float* col_chunk(int c, int ch) const { return (c < 64 ? t0 : t1) + (c & 63) * BM + 4 * (ch ^ (c & 31)); }
};

// The staged epilogues take a 128 x 128 tile from eight waves (wm, wn) of 64 x
// 32 (rows 64 wm + 32 i, columns 32 wn), 512 threads.  Here the accumulators go
// to LDS as they are; the element-wise part runs on the way out (store_rows,
// store_silu).
// IB = 1 (256 x 256 kernel only): the wave's first block alone, rows 32 wm.
template <int IB = 2>
__device__ __forceinline__ void stage_acc(const f32x16_t (&acc)[2][1], const StagedTile& L, int lane, int wm, int wn) {
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      L.row(wm * (32 * IB) + i * 32 + acc_row(r, lane))[wn * 32 + acc_col(lane)] = acc[i][0][r];
}

// The 128 x 128 kernel's tile with the bias, and GELU when asked, applied in
// registers on the way in: its eight waves hold 64 x 32 entries each, so this
// runs without the addresses and tests of the way out.  (In the loop on the way
// out one image's layer 1 took 42.2 us against 40.7 so, three of 1225 tokens
// 52.0 against 50.5.  The 256 x 256 kernel has it there: each of its four
// sub-tiles would hold a copy of this code.)
__device__ __forceinline__ void stage_bias(const GemmProblem& P, int n0, const f32x16_t (&acc)[2][1], const StagedTile& L,
                                           int lane, int wm, int wn) {
  const bf16_t* __restrict__ bias = static_cast<const bf16_t*>(P.bias);
  const bool gelu = P.epi == EPI_BIAS_GELU;
  const int cl = wn * 32 + acc_col(lane);
  const float bv = bias && n0 + cl < P.N ? bf16_to_f32(bias[n0 + cl]) : 0.0f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float v = acc[i][0][r] + bv;
      if (gelu) v = gelu_erf(v);
      L.row(wm * 64 + i * 32 + acc_row(r, lane))[cl] = v;
    }
}

__device__ __forceinline__ uint4 pack_bf16x8(const float (&f)[8]) {
  uint4 o;
  o.x = f32_to_bf16(f[0]) | (static_cast<uint32_t>(f32_to_bf16(f[1])) << 16);
  o.y = f32_to_bf16(f[2]) | (static_cast<uint32_t>(f32_to_bf16(f[3])) << 16);
  o.z = f32_to_bf16(f[4]) | (static_cast<uint32_t>(f32_to_bf16(f[5])) << 16);
  o.w = f32_to_bf16(f[6]) | (static_cast<uint32_t>(f32_to_bf16(f[7])) << 16);
  return o;
}

// The eight bf16 values at src (16 bytes when `vec`, else n of them, then zeros).
__device__ __forceinline__ void load_bf16x8(const bf16_t* src, bool vec, int n, float (&a)[8]) {
  if (vec) {
    const uint4 u = *reinterpret_cast<const uint4*>(src);
    const uint32_t w4[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[2 * k] = __uint_as_float(w4[k] << 16);
      a[2 * k + 1] = __uint_as_float(w4[k] & 0xffff0000u);
    }
  } else {
    for (int k = 0; k < 8; ++k) a[k] = k < n ? bf16_to_f32(src[k]) : 0.0f;
  }
}

__device__ __forceinline__ void store_bf16x8(bf16_t* dst, bool vec, int n, const float (&f)[8]) {
  if (vec) {
    *reinterpret_cast<uint4*>(dst) = pack_bf16x8(f);
  } else {
    for (int k = 0; k < n; ++k) dst[k] = f32_to_bf16(f[k]);
  }
}

// The row-wise epilogues over a staged tile of ROWS rows by W = 128 or 256
// columns (columns 0..127 in L0, 128.. in L1): bias (+ GELU), float32,
// GELU and GELU' of acc + bias, acc times or plus the bf16 aux entry; every
// global access moves 16 bytes along a row.  E: the epilogue where the caller
// knows it (kEpiAny: P.epi; kEpiFinal: the entries are final, only rounded).
constexpr int kEpiAny = -1, kEpiFinal = -2;
template <int W, int NTH, int ROWS = BM, int E = kEpiAny>
__device__ __forceinline__ void store_rows(const GemmProblem& P, int bt, int m0, int n0, const StagedTile& L0,
                                           const StagedTile& L1, int tid) {
  const int M = P.M, N = P.N, e = E == kEpiAny ? P.epi : E;
  const bf16_t* __restrict__ bias = static_cast<const bf16_t*>(P.bias);
  const long long base = bt * P.strideC;
  const bool aligned = (P.ldc & 7) == 0 && (reinterpret_cast<uintptr_t>(P.C) & 15) == 0 &&
                       (!P.aux || (reinterpret_cast<uintptr_t>(P.aux) & 15) == 0) && (base & 7) == 0;
  const bool biased = bias && (e == EPI_BIAS_GELU || e == EPI_BIAS || e == EPI_GELU2);
  // a thread's items share their columns (NTH is a multiple of W / 8)
  const int c8 = (tid % (W / 8)) * 8, col = n0 + c8;
  if (col >= N) return;
  const int n = min(8, N - col);
  const bool vec = aligned && n == 8;
  float bv[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) bv[k] = biased && k < n ? bf16_to_f32(bias[col + k]) : 0.0f;
#pragma unroll 4
  for (int r = tid / (W / 8); r < ROWS; r += NTH / (W / 8)) {
    const int row = m0 + r;
    if (row >= M) break;
    const float* src = W > BN && c8 >= BN ? L1.row(r) + (c8 - BN) : L0.row(r) + c8;
    const float4 x = *reinterpret_cast<const float4*>(src);
    const float4 y = *reinterpret_cast<const float4*>(src + 4);
    float f[8] = {x.x + bv[0], x.y + bv[1], x.z + bv[2], x.w + bv[3], y.x + bv[4], y.y + bv[5], y.z + bv[6], y.w + bv[7]};
    const long long at = base + (long long)row * P.ldc + col;
    if (e == EPI_F32) {
      float* dst = static_cast<float*>(P.C) + at;
      if (vec) {
        reinterpret_cast<float4*>(dst)[0] = x;
        reinterpret_cast<float4*>(dst)[1] = y;
      } else {
        for (int k = 0; k < n; ++k) dst[k] = f[k];
      }
      continue;
    }
    if (e == EPI_GELU2) {
      float g[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) g[k] = gelu_erf_grad(f[k]);
      store_bf16x8(static_cast<bf16_t*>(P.aux) + at, vec, n, g);
    }
    if (e == EPI_BIAS_GELU || e == EPI_GELU2) {
#pragma unroll
      for (int k = 0; k < 8; ++k) f[k] = gelu_erf(f[k]);
    } else if (e == EPI_MUL || e == EPI_RESID) {
      float a8[8];
      load_bf16x8(static_cast<const bf16_t*>(P.aux) + at, vec, n, a8);
#pragma unroll
      for (int k = 0; k < 8; ++k) f[k] = e == EPI_MUL ? f[k] * a8[k] : f[k] + a8[k];
    }
    store_bf16x8(static_cast<bf16_t*>(P.C) + at, vec, n, f);
  }
}

// EPI_SILU: SiLU(gate) * up of a staged tile whose gate columns are in L0 and
// whose up columns are in L1 (W = 128), or in L0's columns 0..63 and 64..127.
template <int W, int NTH, int ROWS = BM>
__device__ __forceinline__ void store_silu(const GemmProblem& P, int bt, int m0, int n0, const StagedTile& L0,
                                           const StagedTile& L1, int tid) {
  const long long base = bt * P.strideC;
  const int c8 = (tid % (W / 8)) * 8, col = n0 + c8;
  if (col >= P.N) return;
  const int n = min(8, P.N - col);
  const bool vec = n == 8 && (P.ldc & 7) == 0 && (reinterpret_cast<uintptr_t>(P.C) & 15) == 0 && (base & 7) == 0;
#pragma unroll 2
  for (int r = tid / (W / 8); r < ROWS; r += NTH / (W / 8)) {
    const int row = m0 + r;
    if (row >= P.M) break;
    const float* g = L0.row(r) + c8;
    const float* u = W == BN ? L1.row(r) + c8 : g + W;
    float f[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = g[k] / (1.0f + __expf(-g[k])) * u[k];
    store_bf16x8(static_cast<bf16_t*>(P.C) + base + (long long)row * P.ldc + col, vec, n, f);
  }
}

// Cosine: S[row][col] = acc * rs[row] * rs[col] (float32), written to both
// (row, col) and (col, row) from the same float, so S is bitwise symmetric.
// A diagonal tile takes the entries below its diagonal from the transposed
// copy (the mirror of the entries above it).
__device__ __forceinline__ void cosine_stage(f32x16_t (&acc)[2][1], const StagedTile& L, const float* rs_rows,
                                             const float* rs_cols, int lane, int wm, int wn) {
  const int cl = wn * 32 + acc_col(lane);
  const float sc = rs_cols[cl];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int rl0 = wm * 64 + i * 32 + 8 * q + 4 * (lane >> 5);
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = acc[i][0][4 * q + e] * (rs_rows[rl0 + e] * sc);
        L.row(rl0 + e)[cl] = v[e];
      }
      *reinterpret_cast<float4*>(L.col_chunk(cl, rl0 >> 2)) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

template <int NTH>
__device__ __forceinline__ void cosine_store(const GemmProblem& P, int bt, int tm, int tn, const StagedTile& L, int tid) {
  const int M = P.M, N = P.N, m0 = tm * BM, n0 = tn * BN;
  const bool diag = tm == tn;
  float* __restrict__ S = static_cast<float*>(P.C) + bt * P.strideC;
  const bool vec = (P.ldc & 3) == 0;
  // S[m0 + r][n0 + 4 ch ..]: row r of the tile (the mirror below a diagonal tile's diagonal)
  for (int e = tid; e < BM * (BN / 4); e += NTH) {
    const int r = e >> 5, ch = e & 31;
    const int row = m0 + r, col = n0 + 4 * ch;
    if (row >= M || col >= N) continue;
    float4 x = *reinterpret_cast<const float4*>(L.row(r) + 4 * ch);
    if (diag) {  // entry (r, c) with c < r is tile entry (c, r): rows 4 ch .. of column r
      const float4 t = *reinterpret_cast<const float4*>(L.col_chunk(r, ch));
      if (4 * ch + 0 < r) x.x = t.x;
      if (4 * ch + 1 < r) x.y = t.y;
      if (4 * ch + 2 < r) x.z = t.z;
      if (4 * ch + 3 < r) x.w = t.w;
    }
    float* dst = S + (long long)row * P.ldc + col;
    if (vec && col + 4 <= N) {
      *reinterpret_cast<float4*>(dst) = x;
    } else {
      const float f[4] = {x.x, x.y, x.z, x.w};
      for (int k = 0; k < 4 && col + k < N; ++k) dst[k] = f[k];
    }
  }
  if (diag) return;
  // S[n0 + c][m0 + 4 ch ..]: column c of the tile
  for (int e = tid; e < BN * (BM / 4); e += NTH) {
    const int c = e >> 5, ch = e & 31;
    const int row = n0 + c, col = m0 + 4 * ch;
    if (row >= N || col >= M) continue;
    const float4 x = *reinterpret_cast<const float4*>(L.col_chunk(c, ch));
    float* dst = S + (long long)row * P.ldc + col;
    if (vec && col + 4 <= M) {
      *reinterpret_cast<float4*>(dst) = x;
    } else {
      const float f[4] = {x.x, x.y, x.z, x.w};
      for (int k = 0; k < 4 && col + k < M; ++k) dst[k] = f[k];
    }
  }
}

// bf16 variant with a five-stage LDS ring filled by direct global->LDS loads
// (global_load_lds_dwordx4): four K slices are in flight while the matrix
// cores consume the fifth, with no register staging, and the five 32 KiB
// stages fill gfx950's 160 KiB of LDS.  Eight waves, two per SIMD (one
// wave's products run while the other waits on LDS or at the barrier):
// wave (wm, wn) = (w / 4, w % 4) forms 64 x 32 of the tile.  Each wave moves
// 16 rows of A and 16 rows of B per slice, one instruction per 8 rows: lane l lands at row
// 8j + l/8, chunk position l%8 of its instruction's 1 KiB, and fetches the
// chunk the XOR swizzle puts there.  The stages are separate LDS arrays
// addressed with compile-time stage numbers, so the only waits on those
// loads are the explicit counted ones before each barrier.
// Requirements (checked by the host): K % 64 == 0, K >= 256, lda and ldb multiples of
// 8, A and B 16-byte aligned, a staged epilogue (bias, cosine, direct) or
// EPI_PARTIAL.

// LDS byte address of a __shared__ object (the value M0 takes for a direct load).
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void*)p));
}

// One global_load_lds_dwordx4: lane l's 16 bytes at gsrc land at byte 16 l
// of the wave's 1 KiB at LDS address m (wave-uniform, passed in M0).  Issued
// from inline assembly so that the compiler adds no waits of its own for
// these loads: it tracks at most four destination arrays of direct loads
// and otherwise drains all of them before every LDS read.  Every read of a
// stage is preceded by the explicit counted wait and the barrier.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // M0 is written here and nowhere else in the kernel
__device__ __forceinline__ void dma16(const void* gsrc, uint32_t m) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gsrc), "s"(m) : "memory", "m0");
}
#pragma clang diagnostic pop

__device__ __forceinline__ void wait_vm_lgkm0(int outstanding) {
  // s_waitcnt encoding: vmcnt in bits [3:0] and [15:14], expcnt [6:4]
  // (7 = no wait), lgkmcnt [11:8]; here vmcnt = outstanding (0, 4, 8, 12,
  // 16 or 24; anything else waits for more) and lgkmcnt = 0
  if (outstanding >= 24) __builtin_amdgcn_s_waitcnt(0x4078);
  else if (outstanding >= 16) __builtin_amdgcn_s_waitcnt(0x4070);
  else if (outstanding >= 12) __builtin_amdgcn_s_waitcnt(0x007c);
  else if (outstanding >= 8) __builtin_amdgcn_s_waitcnt(0x0078);
  else if (outstanding >= 4) __builtin_amdgcn_s_waitcnt(0x0074);
  else __builtin_amdgcn_s_waitcnt(0x0070);
}

// One K slice of the eight-wave 128 x 128 tile: wave (wm, wn) forms rows
// 64 wm + (0..63) by columns 32 wn + (0..31), two 32x32 blocks sharing the B
// operand; the operands of step s + 1 are read before the products of
// step s issue.
__device__ __forceinline__ void mma_slice8(const uint4 (*As)[8], const uint4 (*Bs)[8], int wm, int wn, int lane,
                                           f32x16_t (&acc)[2][1]) {
  const int lr = lane & 31, lh = lane >> 5;
  bf16x8_t a[2][2], b[2];
  auto read = [&](int s, int buf) {
    const int v = 2 * s + lh;  // 16-byte chunk: k = 16 s + 8 lh + (0..7)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = wm * 64 + i * 32 + lr;
      a[buf][i] = __builtin_bit_cast(bf16x8_t, As[r][v ^ swz(r)]);
    }
    const int r = wn * 32 + lr;
    b[buf] = __builtin_bit_cast(bf16x8_t, Bs[r][v ^ swz(r)]);
  };
  read(0, 0);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s < 3) read(s + 1, (s + 1) & 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s & 1][i], b[s & 1], acc[i][0], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Row norms for the workgroups past the tiles: rows of one block spread over
// its waves, two rows per wave at a time.  Each row is summed as prep sums
// it: lane l squares 16-byte chunks l, l + 64, ... in that order, in groups
// of eight, then the wave adds its lanes by a butterfly.
__device__ __forceinline__ void norm_rows(const GemmBatch& args, int blk) {
  const int rows = args.norm_rows, D = args.norm_D, nb = args.norm_blocks;
  const int per = (rows + nb - 1) / nb, r0 = blk * per, r1 = min(rows, r0 + per);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  constexpr int VEC = 8, U = 8;
  const int nchunk = D / VEC;
  for (int r = r0 + 2 * wave; r < r1; r += 2 * nw) {
    const bf16_t* row0 = static_cast<const bf16_t*>(args.norm_V) + (long long)r * D;
    const bf16_t* row1 = static_cast<const bf16_t*>(args.norm_V) + (long long)min(r + 1, r1 - 1) * D;
    float acc[2] = {0.0f, 0.0f};
    for (int c0 = lane; c0 < nchunk; c0 += 64 * U) {
      uint4 uv[2][U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        uv[0][u] = *reinterpret_cast<const uint4*>(row0 + min(c0 + 64 * u, nchunk - 1) * VEC);
        uv[1][u] = *reinterpret_cast<const uint4*>(row1 + min(c0 + 64 * u, nchunk - 1) * VEC);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (c0 + 64 * u < nchunk) {
            // the chunk's eight values in order (low half of each word first)
            const uint32_t wv[4] = {uv[h][u].x, uv[h][u].y, uv[h][u].z, uv[h][u].w};
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
              const uint32_t bits = (k & 1) ? (wv[k >> 1] & 0xffff0000u) : (wv[k >> 1] << 16);
              const float x = __uint_as_float(bits);
              acc[h] = fmaf(x, x, acc[h]);
            }
          }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) acc[h] += __shfl_xor(acc[h], off);
      if (lane == 0 && r + h < r1) {
        const float n = sqrtf(acc[h]);
        args.norms[r + h] = n;
        args.ninv[r + h] = n > 0.0f ? 1.0f / n : 0.0f;
      }
    }
  }
}

constexpr int kDmaThreads = 512;

// SILU: every problem is EPI_SILU, 64 gate columns, then the same columns of up
// (rows N.. of B); else none is.
template <bool SILU>
__global__ __launch_bounds__(kDmaThreads) void gemm_dma_kernel(const GemmBatch args) {
  __shared__ uint4 st0[2][BM][8], st1[2][BM][8], st2[2][BM][8], st3[2][BM][8], st4[2][BM][8];  // 5 x 32 KiB
  if (static_cast<int>(blockIdx.x) >= args.total_tiles) {
    norm_rows(args, blockIdx.x - args.total_tiles);
    return;
  }
  int pi, bt, tm, tn, kc, local;
  decode_tile(args, pi, bt, tm, tn, kc, local);
  const GemmProblem& P = args.p[pi];
  if (P.run_if && P.run_if[bt] == 0) return;
  const int M = P.M, N = P.N;
  // this workgroup's K range: kc kl .. min(K, (kc + 1) kl), kl = kchunk (the
  // last range shorter) or K / ksplit
  const int kl = P.ksplit > 1 ? (P.kchunk > 0 ? P.kchunk : P.K / P.ksplit) : P.K;
  const bf16_t* __restrict__ A = static_cast<const bf16_t*>(P.A) + bt * P.strideA + (long long)kc * kl;
  const bf16_t* __restrict__ B = static_cast<const bf16_t*>(P.B) + bt * P.strideB + (long long)kc * kl;
  const int m0 = tm * BM, n0 = tn * (SILU ? BN / 2 : BN);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int nk = min(kl, P.K - kc * kl) / 64;
  float rs_mine = 0.0f;  // cosine epilogue: reciprocal norm of tile row tid, or of column tid - BM
  if (P.epi == EPI_COSINE && tid < BM + BN) {
    const float* rs = P.rs + (long long)bt * M;
    const int k = tid < BM ? m0 + tid : n0 + tid - BM;
    if (k < (tid < BM ? M : N)) rs_mine = rs[k];
  }

  // Per-lane global row pointers of this wave's 2 A rows and 2 B rows
  // (rows past the matrix read its last row; they are never stored), through
  // the index maps when there are any.
  const int32_t* mapA = P.mapA ? P.mapA + bt * P.mapStride : nullptr;
  const int32_t* mapB = P.mapB ? P.mapB + bt * P.mapStride : nullptr;
  const bf16_t* ga[2];
  const bf16_t* gb[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int r = 16 * wave + 8 * j + (lane >> 3);
    const int v = (lane & 7) ^ swz(r);  // the chunk the swizzle puts at position lane & 7 of row r
    const int ra = min(m0 + r, M - 1), rb = SILU ? (r < 64 ? min(n0 + r, N - 1) : N + min(n0 + r - 64, N - 1)) : min(n0 + r, N - 1);
    ga[j] = A + (long long)(mapA ? mapA[ra] : ra) * P.lda + 8 * v;
    gb[j] = B + (long long)(mapB ? mapB[rb] : rb) * P.ldb + 8 * v;
  }
  // this wave's first destination row inside a stage: 16 wave rows of 128 bytes
  const uint32_t wrow = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave)) * 16u * 128u;
  auto issue = [&](uint4 (*dst)[BM][8], int kt) {
    const int k0 = kt * 64;
    const uint32_t m = lds_addr(&dst[0][0][0]) + wrow;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      dma16(ga[j] + k0, m + 1024u * j);
      dma16(gb[j] + k0, m + BM * 128u + 1024u * j);
    }
  };

  f32x16_t acc[2][1];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][0][r] = 0.0f;

  // Step kt waits for slice kt (this wave's loads, then every wave's at the
  // barrier), refills the stage every wave finished reading in the previous
  // step with slice kt + 4, and runs the matrix cores on slice kt.  Slice kt
  // sits in stage kt % 5, a compile-time constant in the unrolled body; the
  // early exits are uniform scalar branches.
  auto mma = [&](uint4 (*cur)[BM][8]) { mma_slice8(cur[0], cur[1], wm, wn, lane, acc); };
  auto step = [&](uint4 (*cur)[BM][8], uint4 (*nxt)[BM][8], int kt) {
    wait_vm_lgkm0(4 * min(3, nk - 1 - kt));
    __builtin_amdgcn_s_barrier();
    if (kt + 4 < nk) issue(nxt, kt + 4);
    mma(cur);
  };
  issue(st0, 0);
  issue(st1, 1);
  issue(st2, 2);
  issue(st3, 3);
  step(st0, st4, 0);
  for (int kt = 1; kt < nk; kt += 5) {
    step(st1, st0, kt);
    if (kt + 1 >= nk) break;
    step(st2, st1, kt + 1);
    if (kt + 2 >= nk) break;
    step(st3, st2, kt + 2);
    if (kt + 3 >= nk) break;
    step(st4, st3, kt + 3);
    if (kt + 4 >= nk) break;
    step(st0, st4, kt + 4);
  }
  if (P.epi == EPI_PARTIAL) {
    // the raw sums of this K range in the four-wave layout the reductions
    // read: entries (i, j, 4 g .. 4 g + 3) of that layout's thread t (wave
    // 2 wm + wn / 2, j = wn % 2) as float4 q = (2 i + j) 4 + g at q * 256 + t
    // (every store of a wave contiguous)
    float4* dst = static_cast<float4*>(P.C) + (long long)local * (16 * 256);
    const int t4 = (2 * wm + (wn >> 1)) * 64 + lane, j4 = wn & 1;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        dst[((2 * i + j4) * 4 + g) * 256 + t4] =
            make_float4(acc[i][0][4 * g], acc[i][0][4 * g + 1], acc[i][0][4 * g + 2], acc[i][0][4 * g + 3]);
    return;
  }
  __syncthreads();  // the epilogues reuse the stage arrays
  float* rs_tile = reinterpret_cast<float*>(&st4[0][0][0]);
  if (P.epi == EPI_COSINE) {
    if (tid < BM + BN) rs_tile[tid] = rs_mine;
    __syncthreads();
  }
  const StagedTile L{reinterpret_cast<float*>(&st0[0][0][0]), reinterpret_cast<float*>(&st1[0][0][0]),
                     reinterpret_cast<float*>(&st2[0][0][0]), reinterpret_cast<float*>(&st3[0][0][0])};
  if constexpr (SILU) {
    stage_acc(acc, L, lane, wm, wn);
    __syncthreads();
    store_silu<BN / 2, kDmaThreads>(P, bt, m0, n0, L, L, tid);
    return;
  }
  if (P.epi == EPI_COSINE) {
    cosine_stage(acc, L, rs_tile, rs_tile + BM, lane, wm, wn);
    __syncthreads();
    cosine_store<kDmaThreads>(P, bt, tm, tn, L, tid);
  } else if (P.epi == EPI_BIAS_GELU || P.epi == EPI_BIAS) {
    stage_bias(P, n0, acc, L, lane, wm, wn);
    __syncthreads();
    store_rows<BN, kDmaThreads, BM, kEpiFinal>(P, bt, m0, n0, L, L, tid);
  } else {  // (the training step's 136 tiles of EPI_F32 and EPI_MUL: 11.5 us on one loop for all epilogues, 9.5 so)
    stage_acc(acc, L, lane, wm, wn);
    __syncthreads();
    if (P.epi == EPI_F32)
      store_rows<BN, kDmaThreads, BM, EPI_F32>(P, bt, m0, n0, L, L, tid);
    else if (P.epi == EPI_MUL)
      store_rows<BN, kDmaThreads, BM, EPI_MUL>(P, bt, m0, n0, L, L, tid);
    else if (P.epi == EPI_RESID)
      store_rows<BN, kDmaThreads, BM, EPI_RESID>(P, bt, m0, n0, L, L, tid);
    else
      store_rows<BN, kDmaThreads, BM, EPI_GELU2>(P, bt, m0, n0, L, L, tid);
  }
}

// ------------------------------------------------------------ float32 tiles
// 64 x 64 tiles for float32, and for bf16 launches too small to fill the chip
// with larger ones: eight waves in two groups of four; in a group each wave
// forms one 32 x 32 block, group g over the 128-byte K slices (32 floats, 64
// bf16) with kt % 2 = g, and the two sums are added in LDS at the end.  The
// slices come by direct loads through a ring of four pairs (32 KiB each).
// float32: the matrix rate bounds it (a slice's products take 1024 clocks on
// each SIMD, its operand reads 256 of LDS), so small tiles cost nothing and
// fill the chip, and two waves per SIMD hide the reads and the barriers of
// each other.  A 576 x 1024 x 4096 layer with its 576-token Gram matrix and
// the folds: 336 us on 128 x 128 tiles, 79 of them for 256 compute units, now
// about 75; 4096 x 4096 x 4096 1.21 ms (113 TFLOP/s of about 150 that products
// on registers alone reach).
// bf16: a compute unit takes in about 50 GB/s with the loads that LDS has
// room for in flight, so a tile's time is its operand bytes, half those of a
// 128 x 128 tile: the same bf16 launch 38 -> 22 us.
// Requirements (checked by the host): K a multiple of the slice, lda and ldb
// multiples of 16 bytes, A and B 16-byte aligned, no RoPE or SwiGLU
// epilogue, K range or index map.
constexpr int kTile = 64;
constexpr int kTilePairs = 4;
constexpr int kTileThreads = 512;

template <typename T>
__global__ __launch_bounds__(kTileThreads) void gemm_tile64_kernel(const GemmBatch args) {
  constexpr int BK = Slice<T>::BK, VEC = Slice<T>::VEC;
  __shared__ uint4 st[kTilePairs][2][2][kTile][8];  // per pair: slice of group 0, of group 1; each A rows, B rows
  int pi, bt, tm, tn, kc, local;
  decode_tile(args, pi, bt, tm, tn, kc, local);
  const GemmProblem& P = args.p[pi];
  if (P.run_if && P.run_if[bt] == 0) return;
  const int M = P.M, N = P.N, m0 = tm * kTile, n0 = tn * kTile, nk = P.K / BK;
  const T* __restrict__ A = static_cast<const T*>(P.A) + bt * P.strideA;
  const T* __restrict__ B = static_cast<const T*>(P.B) + bt * P.strideB;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, w4 = wave & 3, wm = w4 >> 1, wn = w4 & 1, lr = lane & 31, lh = lane >> 5;
  const int np = (nk + 1) / 2, own = (nk - grp + 1) / 2;  // pairs; this group's slices
  // wave w of a group moves rows 16 w .. 16 w + 15 of A and of B of its
  // group's slices, one instruction per 8 rows (rows past the matrix read
  // its last row; they are never stored)
  const T* ga[2];
  const T* gb[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int r = 16 * w4 + 8 * j + (lane >> 3), v = (lane & 7) ^ swz(r);
    ga[j] = A + (long long)min(m0 + r, M - 1) * P.lda + VEC * v + BK * grp;
    gb[j] = B + (long long)min(n0 + r, N - 1) * P.ldb + VEC * v + BK * grp;
  }
  const uint32_t wrow = lds_addr(&st[0][0][0][0][0]) + static_cast<uint32_t>(grp) * (2u * kTile * 128u) +
                        static_cast<uint32_t>(w4) * 16u * 128u;
  auto issue = [&](int p) {
    const uint32_t m = wrow + static_cast<uint32_t>(p % kTilePairs) * (4u * kTile * 128u);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      dma16(ga[j] + 2 * BK * p, m + 1024u * j);
      dma16(gb[j] + 2 * BK * p, m + kTile * 128u + 1024u * j);
    }
  };
  f32x16_t acc[1][1];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.0f;
  for (int p = 0; p < min(kTilePairs - 1, own); ++p) issue(p);
  for (int p = 0; p < np; ++p) {
    // this wave's part of its group's slice p (past its last one: nothing is outstanding)
    wait_vm_lgkm0(4 * max(0, min(kTilePairs - 2, own - 1 - p)));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();  // every wave's part, and every wave is done with pair p - 1
    asm volatile("" ::: "memory");
    if (p + kTilePairs - 1 < own) issue(p + kTilePairs - 1);
    if (p >= own) break;  // (the last pair of an odd count: group 1 has no slice)
    const uint4 (*As)[8] = st[p % kTilePairs][grp][0];
    const uint4 (*Bs)[8] = st[p % kTilePairs][grp][1];
    uint4 a[4], b[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      // float32: lane half lh covers k = 16 lh + 4 g + (0..3); bf16: 16 g + 8 lh + (0..7)
      const int v = (sizeof(T) == 4 ? 4 * lh + g : 2 * g + lh) ^ swz(lr);
      a[g] = As[32 * wm + lr][v];
      b[g] = Bs[32 * wn + lr][v];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if constexpr (sizeof(T) == 4) {
        const float4 af = __builtin_bit_cast(float4, a[g]), bf = __builtin_bit_cast(float4, b[g]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[e], bf[e], acc[0][0], 0, 0, 0);
      } else {
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a[g]),
                                                            __builtin_bit_cast(bf16x8_t, b[g]), acc[0][0], 0, 0, 0);
      }
    }
  }
  __syncthreads();  // the ring is read out: group 1's sums pass through it
  float* sums = reinterpret_cast<float*>(&st[0][0][0][0][0]) + w4 * 16 * 64 + lane;
  if (grp) {
#pragma unroll
    for (int r = 0; r < 16; ++r) sums[64 * r] = acc[0][0][r];
  }
  __syncthreads();
  if (grp) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] += sums[64 * r];
  epilogue<T, 1, 1>(P, bt, tm, tn, acc, nullptr, nullptr, tid, lane, wm, wn);
}

// ------------------------------------------------------------ 256 x 256 tiles
// Launches of several waves of workgroups (the first layer over a batch of
// images, the decoder layer's long products) run 256 x 256 tiles: per
// product a compute unit then moves half the bytes from L2 into LDS and
// reads half as many operand bytes from LDS as with 128 x 128 tiles, which
// is what bounds the smaller tile.  512 threads, eight wave64s, two per SIMD;
// wave (wm, wn) = (w / 4, w % 4) owns rows 128 i + 64 wm + (0..63) and columns
// 128 j + 32 wn + (0..31) for i, j = 0, 1: in each of the four 128 x 128
// sub-tiles (i, j) the layout of the 128 x 128 kernel, whose epilogues finish
// them one after the other.
//
// What bounds the loop: LDS moves 128 bytes per clock, and a 64-wide slice
// needs 192 KiB of operand reads and 64 KiB of direct-load writes there, 2048
// clocks, as many as its products take on a SIMD.  Neither may wait for the
// other, so the waves run in two groups (w / 4), half a phase apart: a SIMD
// holds one wave of each, and while one group's waves run the eight products
// of a phase the other group's read the operands of their next phase.  A
// slice has four phases, one per sub-tile; every phase is [operand reads,
// one half-tile's direct loads] barrier [products] barrier, and group 1 starts
// one barrier late.  Half-tiles (A or B, 128 rows by one slice, 16 KiB) sit
// in two buffers; each is reloaded as soon as both groups have read it, so
// 7 half-tiles (112 KiB) are in flight or waiting ahead of the reads.
// Against the former loop (one barrier per slice, all waves in step):
// 46080 x 1024 x 4096 461 -> 365 us, 8192 x 8192 x 8192 957 -> 808 us (1360
// TFLOP/s).  On operands that are all zero the latter takes 597 us: what is
// left is the clock that the power limit leaves.  (Reading every operand one
// phase ahead, with both halves of A and B in registers, is no faster: 905 us.)
// Tiles are ordered in groups of kBigRows tile rows, column by column inside
// a group (a triangular problem: its upper triangle row by row), each XCD
// taking a contiguous range.
constexpr int kBig = 256;
constexpr int kBigThreads = 512;
constexpr int kBigRows = 4;

// dma16 with a wave-uniform base and a 32-bit byte offset per lane.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // M0 is written here and in dma16 only
__device__ __forceinline__ void dma16_off(const void* base, uint32_t off, uint32_t m) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" : : "s"(base), "v"(off), "s"(m) : "memory", "m0");
}
#pragma clang diagnostic pop

// Barrier that neither the compiler's nor the scheduler's reordering crosses.
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Tile heights.  A launch whose tiles do not fill whole rounds of workgroups
// would leave compute units idle in its last one, so a problem's rows may also
// be cut into tiles of 192 or 128 rows (GemmProblem::th):
//   TM = 192: the lower half-tile of A is 64 rows (wave (wm, wn): rows 128 +
//       32 wm + (0..31)), the last two phases have half the products;
//   128 rows or fewer in a tile: two phases a slice (no lower half), the
//       slices in a ring of three.
// The rule (plan_big) counts a tile as its share of the products (0.75, 0.5)
// plus its start and epilogue.  2944 x 4096 x 4096: 192 tiles of 256 rows on
// 256 units 107 us, 256 tiles of 192 rows 96; 2944 x 12288 x 4096: 576 tiles
// 292 us, 768 of 192 rows 260; 36864 x 1024 x 3584 with its question rows
// and folds: 596 tiles (2.3 rounds) 320 us, 512 and 160 of 128 rows 287;
// 5760 x 1024 x 4096: 128 x 128 tiles 92 us, 180 of 128 x 256 74.
//
// NORMS: the launch has row norms to form (GemmProblem::norm_at).
template <bool NORMS, int TM>
__global__ __launch_bounds__(kBigThreads) void gemm_big_kernel(const GemmBatch args) {
  // Half-tile arrays.  More than 128 rows: 4 buffer + (A rows 0..127, A rows
  // 128.., B rows 0..127, B rows 128..), buffer = 0, 1; else 3 slot + (A, B
  // rows 0..127, B rows 128..), slot = 0, 1, 2.
  __shared__ uint4 half[9][BM][8];
  __shared__ float rs_big[2 * kBig];  // cosine: 1/norm of the tile's rows, then columns
  const int tile = class_tile(args, blockIdx.x);
  int local;
  const int pi = find_problem(args, tile, local);
  const GemmProblem& P = args.p[pi];
  const int bt = local / P.tiles_per_batch;
  int tt = local - bt * P.tiles_per_batch, tm, tn;
  if (P.triangular) {  // upper triangle, row by row: row tm holds tiles_n - tm tiles
    tm = 0;
    while (tt >= P.tiles_n - tm) { tt -= P.tiles_n - tm; ++tm; }
    tn = tm + tt;
  } else {
    const int grp = tt / (kBigRows * P.tiles_n), first = grp * kBigRows;
    const int rows = min(kBigRows, P.tiles_m - first), in = tt - grp * kBigRows * P.tiles_n;
    tm = first + in % rows;
    tn = in / rows;
  }
  if (P.run_if && P.run_if[bt] == 0) return;
  const int M = P.M, N = P.N, m0 = tm * P.th;
  const bool silu = P.epi == EPI_SILU;  // 128 gate columns, then the same columns of up (rows N.. of B)
  const int n0 = tn * (silu ? kBig / 2 : kBig);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int nk = P.K / 64;  // even (checked by the host)
  float rs_mine = 0.0f;     // cosine epilogue: 1/norm of tile row tid, or of column tid - 256
  if (P.epi == EPI_COSINE) {
    const int k = tid < kBig ? m0 + tid : n0 + tid - kBig;
    if (k < (tid < kBig ? M : N)) rs_mine = P.rs[(long long)bt * M + k];
  }
  // Wave w loads rows 16 w .. 16 w + 15 of every half-tile, one instruction
  // per 8 rows (rows past the matrix read its last row): byte offsets from
  // the tile's first row, or from the matrix with an index map.
  const int32_t* mapA = P.mapA ? P.mapA + bt * P.mapStride : nullptr;
  const int32_t* mapB = P.mapB ? P.mapB + bt * P.mapStride : nullptr;
  const char* baseA = reinterpret_cast<const char*>(static_cast<const bf16_t*>(P.A) + bt * P.strideA +
                                                    (mapA ? 0 : (long long)m0 * P.lda));
  const char* baseB = reinterpret_cast<const char*>(static_cast<const bf16_t*>(P.B) + bt * P.strideB +
                                                    (mapB ? 0 : (long long)n0 * P.ldb));
  uint32_t off[4][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = 16 * wave + 8 * j + (lane >> 3);
      const int v = (lane & 7) ^ swz(r);  // the chunk the swizzle puts at position lane & 7 of row r
      // (TM = 192: the lower half-tile has 8 rows per wave, one instruction)
      const int r1 = TM == 192 && x == 1 ? 8 * wave + (lane >> 3) : r, va = (lane & 7) ^ swz(r1);
      const int ra = min(128 * x + r1, M - 1 - m0), rb = silu ? min(r, N - 1 - n0) + x * N : min(128 * x + r, N - 1 - n0);
      off[x][j] = static_cast<uint32_t>(mapA ? mapA[m0 + ra] : ra) * static_cast<uint32_t>(2 * P.lda) + 16u * va;
      off[2 + x][j] = static_cast<uint32_t>(mapB ? mapB[n0 + rb] : rb) * static_cast<uint32_t>(2 * P.ldb) + 16u * v;
    }
  const uint32_t wrow = lds_addr(&half[0][0][0]) + static_cast<uint32_t>(wave) * 16u * 128u;
  auto issue_at = [&](int kt, int x, int at) {  // half-tile x of slice kt into array `at`
    const char* src = (x < 2 ? baseA : baseB) + 128LL * kt;
    const uint32_t m = wrow + static_cast<uint32_t>(at) * (BM * 128u);
    dma16_off(src, off[x][0], m);
    dma16_off(src, off[x][1], m + 1024u);
  };
  auto issue = [&](int kt, int buf, int x) {  // half-tile x of slice kt into buffer buf
    if (TM == 192 && x == 1)
      dma16_off(baseA + 128LL * kt, off[1][0],
                wrow + static_cast<uint32_t>(4 * buf + 1) * (BM * 128u) - static_cast<uint32_t>(wave) * 8u * 128u);
    else
      issue_at(kt, x, 4 * buf + x);
  };

  f32x16_t acc[2][2][2][1];  // [i][j][block]: rows 128 i + 64 wm + 32 block, columns 128 j + 32 wn
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][b][0][r] = 0.0f;
  const int lr = lane & 31, lh = lane >> 5;
  bf16x8_t a[2][4], b0[4], b1[4];  // [block][step of 16]
  constexpr int kLow = TM == 192 ? 1 : 2;  // blocks of a wave in the lower half-tile
  auto read_a = [&](int at, int i) {       // from array `at`: rows of the upper (i = 0) or lower half
    const int nb = i ? kLow : 2;
#pragma unroll
    for (int b = 0; b < nb; ++b)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = 32 * nb * wm + 32 * b + lr;
        a[b][s] = __builtin_bit_cast(bf16x8_t, half[at][r][(2 * s + lh) ^ swz(lr)]);
      }
  };
  auto read_b = [&](int at, bf16x8_t (&b)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int r = 32 * wn + lr;
      b[s] = __builtin_bit_cast(bf16x8_t, half[at][r][(2 * s + lh) ^ swz(lr)]);
    }
  };
  // Row norms (GemmProblem::norm_at).  Row block (i, b) = rows 128 i + 64 wm +
  // 32 b + (0..31) of both wm is summed by the tiles of column (2 i + b) mod
  // min(tiles_n, 4), wave wn taking step wn of 16 of every slice (lane l: row
  // l & 31, eight of the step's values), in float32, slice after slice; the
  // eight sums of a row meet at the end.  A wave then has 16 vector
  // instructions per slice, which fit beside the other group's products.
  // (With all of it on the first tile column, 64 instructions in half of its
  // waves, each of its slices took 9 % longer, and with it every round.)
  const int ncol = NORMS && P.norm_at ? min(P.tiles_n, 4) : 0;
  bool sq[2][2];
  float nacc[2][2] = {{0.0f, 0.0f}, {0.0f, 0.0f}};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int b = 0; b < 2; ++b) sq[i][b] = tn < ncol && (2 * i + b) % max(ncol, 1) == tn;
  auto squares = [&](int at, int i) {
    if constexpr (!NORMS) return;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (!sq[i][b]) continue;
      const uint4 u = half[at][64 * wm + 32 * b + lr][(2 * wn + lh) ^ swz(lr)];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read before this phase's barrier: see slice()
      const uint32_t wv[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float x = __uint_as_float((k & 1) ? (wv[k >> 1] & 0xffff0000u) : (wv[k >> 1] << 16));
        nacc[i][b] = fmaf(x, x, nacc[i][b]);
      }
    }
  };
  auto products = [&](int i, int j, const bf16x8_t (&b)[4]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < (i ? kLow : 2); ++c)
        acc[i][j][c][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[c][s], b[s], acc[i][j][c][0], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  // One slice kt in buffer buf (= kt % 2, a constant in the unrolled body).
  // Hazards: a half-tile is reloaded one phase or more after the phase that
  // read it, whose reads both groups have waited for by then.  Reads of an
  // array that is reloaded in the very next phase are waited for before their
  // own phase's first barrier, since the other group may start that phase
  // after it: B0's, and those that the row norms add (squares: the upper half
  // of A in the second phase, the lower half in the last).  The loads of
  // slice kt + 1 are waited for in the last phase, before the barrier that
  // lets either group read it.
  auto slice = [&](int kt, int buf) {
    const bool more1 = kt + 1 < nk, more2 = kt + 2 < nk;
    read_b(4 * buf + 2, b0);
    __builtin_amdgcn_sched_barrier(0);
    read_a(4 * buf, 0);
    if (more1) issue(kt + 1, buf ^ 1, 1);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(8)" ::: "memory");
    phase_barrier();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    products(0, 0, b0);
    phase_barrier();

    read_b(4 * buf + 3, b1);
    if (more2) issue(kt + 2, buf, 2);
    squares(4 * buf, 0);
    phase_barrier();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    products(0, 1, b1);
    phase_barrier();

    read_a(4 * buf + 1, 1);
    if (more2) issue(kt + 2, buf, 0);
    phase_barrier();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    products(1, 0, b0);
    phase_barrier();

    if (more2) {
      issue(kt + 2, buf, 3);
      squares(4 * buf + 1, 1);
      asm volatile("s_waitcnt vmcnt(6)" ::: "memory");  // all but the three half-tiles of slice kt + 2
    } else {
      squares(4 * buf + 1, 1);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    phase_barrier();
    products(1, 1, b1);
    phase_barrier();
  };
  // One slice of a tile of at most 128 rows, in ring slot kt % 3.  The slot
  // that slice kt + 2 goes to held slice kt - 1, whose last reads each group
  // waited for before a barrier that both have passed; slice kt + 1 has
  // landed before the barrier that lets either group read it.
  auto slice_low = [&](int kt, int slot, int refill) {
    const bool more = kt + 2 < nk;
    read_b(3 * slot + 1, b0);
    read_a(3 * slot, 0);
    if (more) {
      issue_at(kt + 2, 0, 3 * refill);
      issue_at(kt + 2, 2, 3 * refill + 1);
      issue_at(kt + 2, 3, 3 * refill + 2);
    }
    squares(3 * slot, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    phase_barrier();
    products(0, 0, b0);
    phase_barrier();

    read_b(3 * slot + 2, b1);
    if (more)
      asm volatile("s_waitcnt vmcnt(6)" ::: "memory");  // all but slice kt + 2
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    phase_barrier();
    products(0, 1, b1);
    phase_barrier();
  };
  const bool low = min(P.th, M - m0) <= 128;  // (uniform over the workgroup)
  if (low) {
    issue_at(0, 0, 0);
    issue_at(0, 2, 1);
    issue_at(0, 3, 2);
    issue_at(1, 0, 3);
    issue_at(1, 2, 4);
    issue_at(1, 3, 5);
    asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    phase_barrier();
    if (wm) phase_barrier();  // group 1 runs one barrier behind group 0
    int slot = 0;
#pragma unroll 1
    for (int kt = 0; kt < nk; ++kt) {
      slice_low(kt, slot, slot == 0 ? 2 : slot - 1);
      slot = slot == 2 ? 0 : slot + 1;
    }
  } else {
    issue(0, 0, 2);
    issue(0, 0, 0);
    issue(0, 0, 3);
    issue(0, 0, 1);
    issue(1, 1, 2);
    issue(1, 1, 0);
    issue(1, 1, 3);
    asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    phase_barrier();
    if (wm) phase_barrier();  // group 1 runs one barrier behind group 0
    for (int kt = 0; kt < nk; kt += 2) {
      slice(kt, 0);
      slice(kt + 1, 1);
    }
  }
  if (!wm) phase_barrier();
  __syncthreads();  // the buffers are free
  if (NORMS && tn < ncol) {
    float* sums = reinterpret_cast<float*>(&half[0][0][0]);  // [2 i + b][wm][wn][lh][32]
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (sq[q >> 1][q & 1]) sums[(8 * q + wave) * 64 + lane] = nacc[q >> 1][q & 1];
    __syncthreads();
    const int q = tid >> 6, row = 128 * (q >> 1) + 32 * (q & 1) + 64 * (lane >> 5) + lr;  // threads 0..255
    if (q < 4 && q % max(ncol, 1) == tn && row < P.th && m0 + row < M) {
      float t = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) t += sums[(8 * q + 4 * (lane >> 5)) * 64 + 32 * k + lr];
      const float n = sqrtf(t);
      args.norms[P.norm_at - 1 + m0 + row] = n;
      args.ninv[P.norm_at - 1 + m0 + row] = n > 0.0f ? 1.0f / n : 0.0f;
    }
    __syncthreads();
  }
  float* stage0 = reinterpret_cast<float*>(&half[0][0][0]);
  float* stage1 = reinterpret_cast<float*>(&half[4][0][0]);
  if (P.epi == EPI_COSINE) {
    rs_big[tid] = rs_mine;
    const StagedTile LC{stage0, stage0 + 64 * BN, stage1, stage1 + 64 * BM};
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      const int i = q >> 1, j = q & 1, tm1 = 2 * tm + i, tn1 = 2 * tn + j;  // the sub-tile in 128 x 128 tiles
      // (uniform over the workgroup; a diagonal tile's sub-tile below the
      // diagonal is the mirror of the one above it)
      if (tm1 > tn1 || tm1 * BM >= M || tn1 * BN >= N) continue;
      __syncthreads();  // the staging is free (and rs_big written)
      const float *rr = rs_big + 128 * i, *rc = rs_big + kBig + 128 * j;
      if (q == 0)
        cosine_stage(acc[0][0], LC, rr, rc, lane, wm, wn);
      else if (q == 1)
        cosine_stage(acc[0][1], LC, rr, rc, lane, wm, wn);
      else if (q == 2)
        cosine_stage(acc[1][0], LC, rr, rc, lane, wm, wn);
      else
        cosine_stage(acc[1][1], LC, rr, rc, lane, wm, wn);
      __syncthreads();
      cosine_store<kBigThreads>(P, bt, tm1, tn1, LC, tid);
    }
    return;
  }
  // 128 rows by 256 columns at a time (the lower half of TM = 192: 64)
  const StagedTile L0{stage0, stage0 + 64 * BN, nullptr, nullptr}, L1{stage1, stage1 + 64 * BN, nullptr, nullptr};
  stage_acc(acc[0][0], L0, lane, wm, wn);
  stage_acc(acc[0][1], L1, lane, wm, wn);
  __syncthreads();
  if (silu)
    store_silu<kBig / 2, kBigThreads>(P, bt, m0, n0, L0, L1, tid);
  else
    store_rows<kBig, kBigThreads>(P, bt, m0, n0, L0, L1, tid);
  if (low) return;
  __syncthreads();  // the staging is read out
  stage_acc<kLow>(acc[1][0], L0, lane, wm, wn);
  stage_acc<kLow>(acc[1][1], L1, lane, wm, wn);
  __syncthreads();
  if (silu)
    store_silu<kBig / 2, kBigThreads, 64 * kLow>(P, bt, m0 + 128, n0, L0, L1, tid);
  else
    store_rows<kBig, kBigThreads, 64 * kLow>(P, bt, m0 + 128, n0, L0, L1, tid);
}

// Projection to d_p <= 128 columns with the RoPE epilogue (the keys and
// queries of Eq. (3)): C = RoPE(A B^T + bias), A [M][K] and B [N][K] bf16
// (float32 inputs: the same with 32 x 32 x 2 float32 products).
// With N this small and rows for fewer than one wave of tiles, a 128 x 128
// tile leaves most compute units idle, each streaming the whole K with a
// few slices in flight.  Here a workgroup takes
// 32 rows and one of two groups of RoPE pairs: with half = N / 2 and
// PG = ceil(half / 2), group g holds pairs c = g PG .. (g + 1) PG - 1, i.e.
// columns c and c + half, so every rotation is local and each workgroup
// reads half of B.  Its eight waves split K: wave w takes the 64-wide chunks
// w, w + 8, ...  Lane l reads 64 contiguous bytes of row l & 31 per chunk, A
// and B alike, straight from global memory into registers, and the chunk's
// four products consume them in an order shared by both operands (any
// common order of k gives the same sum).  The eight partial tiles are summed
// in LDS in a fixed order.
// Requirements (checked by the host): N <= 128 and even, K, lda and ldb
// multiples of 8, A and B 16-byte aligned, one batch item.
constexpr int kPR = 32;   // rows per workgroup
constexpr int kPW = 8;    // waves per workgroup
constexpr int kPG = 2;    // groups of RoPE pairs per row block
constexpr int kPS = 68;   // LDS row stride of the partial tiles (floats)

typedef __attribute__((ext_vector_type(4))) float float4v;

template <typename T>
__global__ __launch_bounds__(kPW * 64) void proj_rope_kernel(const GemmBatch args) {
  __shared__ float part[kPW][kPR][kPS];
  const int t0 = args.p[0].tiles_m, pi = blockIdx.x < t0 ? 0 : 1;
  const GemmProblem& P = args.p[pi];
  const int local = blockIdx.x - (pi ? t0 : 0), g = local % kPG;
  const int m0 = (local / kPG) * kPR;
  const int M = P.M, K = P.K, half = P.N >> 1;
  const int PG = (half + kPG - 1) / kPG, c0 = g * PG, npg = min(PG, half - c0);
  if (npg <= 0) return;  // a group without pairs (half = 1)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const T* __restrict__ A = static_cast<const T*>(P.A);
  const T* __restrict__ B = static_cast<const T*>(P.B);

  const int r = lane & 31, h = lane >> 5;
  const T* arow = A + (long long)min(m0 + r, M - 1) * P.lda;
  const int pr = c0 + min(r, npg - 1);  // the pair of tile column r (32 + r: its partner)
  const T* brow[2] = {B + (long long)pr * P.ldb, B + (long long)(pr + half) * P.ldb};
  f32x16_t acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
  const int nchunk = (K + 63) >> 6;
  if constexpr (sizeof(T) == 4) {
    // float32: per 64-wide chunk lane l holds 32 contiguous k of its row
    // (half h = l >> 5 of the chunk), for A and B alike; the 32 x 32 x 2
    // products pair k = s of the first half with k = 32 + s of the second
    // (any common order of k gives the same sum)
    for (int kc = wave; kc < nchunk; kc += kPW) {
      const int kb = 64 * kc + 32 * h;
      float4v av[8], bv[2][8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int k = kb + 4 * q;
        const int off = k < K ? k : 0;  // past K: a valid address, zeroed below
        av[q] = *reinterpret_cast<const float4v*>(arow + off);
#pragma unroll
        for (int j = 0; j < 2; ++j) bv[j][q] = *reinterpret_cast<const float4v*>(brow[j] + off);
      }
      __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the products
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float4v z = {0.0f, 0.0f, 0.0f, 0.0f};
        const float4v a = kb + 4 * q < K ? av[q] : z;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], bv[j][q][e], acc[j], 0, 0, 0);
      }
    }
  } else
  for (int kc = wave; kc < nchunk; kc += 2 * kPW) {  // two chunks per pass, every load issued first
    uint4 av[2][4], bv[2][2][4];
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 64 * (kc + kPW * c2) + 32 * h + 8 * q;
        const int off = k < K ? k : 0;  // past K: a valid address, zeroed below
        av[c2][q] = *reinterpret_cast<const uint4*>(arow + off);
#pragma unroll
        for (int j = 0; j < 2; ++j) bv[c2][j][q] = *reinterpret_cast<const uint4*>(brow[j] + off);
      }
    __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the products
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 64 * (kc + kPW * c2) + 32 * h + 8 * q;
        const uint4 z = {0u, 0u, 0u, 0u};
        const bf16x8_t a = __builtin_bit_cast(bf16x8_t, k < K ? av[c2][q] : z);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8_t, bv[c2][j][q]), acc[j],
                                                           0, 0, 0);
      }
  }
  // the epilogue's (cos, sin) pairs and biases (item e = row e / npg, pair
  // c0 + e % npg; at most two per thread), in flight while the partials meet
  constexpr int EI = kPR * 32 / (kPW * 64);
  float2 cs[EI];
  float bl[EI], bh[EI];
#pragma unroll
  for (int u = 0; u < EI; ++u) {
    const int e = min(tid + kPW * 64 * u, kPR * npg - 1), rl = e / npg, c = c0 + e - rl * npg;
    cs[u] = P.rope_cs[(long long)min(m0 + rl, M - 1) * half + c];
    bl[u] = P.rope_bias ? P.rope_bias[c] : 0.0f;
    bh[u] = P.rope_bias ? P.rope_bias[c + half] : 0.0f;
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) part[wave][acc_row(e, lane)][32 * j + acc_col(lane)] = acc[j][e];
  __syncthreads();
  float* __restrict__ out = static_cast<float*>(P.C);
#pragma unroll
  for (int u = 0; u < EI; ++u) {
    const int e = tid + kPW * 64 * u, rl = e / npg, cl = e - rl * npg;
    if (e >= kPR * npg || m0 + rl >= M) continue;
    float s0[kPW], s1[kPW];
#pragma unroll
    for (int w = 0; w < kPW; ++w) {
      s0[w] = part[w][rl][cl];
      s1[w] = part[w][rl][32 + cl];
    }
    const float a = (((s0[0] + s0[1]) + (s0[2] + s0[3])) + ((s0[4] + s0[5]) + (s0[6] + s0[7]))) + bl[u];
    const float b = (((s1[0] + s1[1]) + (s1[2] + s1[3])) + ((s1[4] + s1[5]) + (s1[6] + s1[7]))) + bh[u];
    float* o = out + (long long)(m0 + rl) * P.ldc + c0 + cl;
    o[0] = a * cs[u].x - b * cs[u].y;
    o[half] = b * cs[u].x + a * cs[u].y;
  }
}

// The K ranges of a split problem summed in order kc = 0, 1, ...: workgroup
// (tile t, piece q, batch item) takes float4 q of every thread of the
// tile's partials, i.e. accumulator block (i, j) = (q / 8, q / 4 % 2), rows
// 4 (q % 4) .. + 3 of the thread's 32 x 32 block layout, and writes those
// entries of S and their mirror as the cosine epilogue does.
__global__ __launch_bounds__(NT) void gram_reduce_kernel(const GemmProblem P, float* out, int ldc,
                                                         const float* rs_all) {
  const int bt = blockIdx.y, t = blockIdx.x >> 4, q = blockIdx.x & 15;
  if (P.run_if && P.run_if[bt] == 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int ks = P.ksplit > 1 ? P.ksplit : 1;
  int tm = 0, tt = t;
  while (tt >= P.tiles_n - tm) {
    tt -= P.tiles_n - tm;
    ++tm;
  }
  const int tn = tm + tt;
  const float4* src = static_cast<const float4*>(P.C) + (long long)bt * P.tiles_per_batch * (16 * NT);
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 x[16];
#pragma unroll
  for (int kc = 0; kc < 16; ++kc)
    if (kc < ks) x[kc] = src[((long long)kc * P.tiles_tri + t) * (16 * NT) + q * NT + tid];
#pragma unroll
  for (int kc = 0; kc < 16; ++kc)
    if (kc < ks) {
      v.x += x[kc].x;
      v.y += x[kc].y;
      v.z += x[kc].z;
      v.w += x[kc].w;
    }
  for (int kc = 16; kc < ks; ++kc) {
    const float4 y = src[((long long)kc * P.tiles_tri + t) * (16 * NT) + q * NT + tid];
    v.x += y.x;
    v.y += y.y;
    v.z += y.z;
    v.w += y.w;
  }
  const int i = q >> 3, j = (q >> 2) & 1, g = q & 3;
  const int M = P.M, m0 = tm * BM, n0 = tn * BN;
  const bool diag = tm == tn;
  const int col = n0 + wn * 64 + j * 32 + acc_col(lane);
  const int row0 = m0 + wm * 64 + i * 32 + 8 * g + 4 * (lane >> 5);
  if (col >= M) return;
  const float* rs = rs_all + (long long)bt * M;
  float* S = out + (long long)bt * M * ldc;
  const float sc = rs[col];
  const float a[4] = {v.x, v.y, v.z, v.w};
  float w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = row0 + e;
    w[e] = row < M ? a[e] * (rs[row] * sc) : 0.0f;
    if (row < M && (!diag || row <= col)) S[(long long)row * ldc + col] = w[e];
  }
  float* dst = S + (long long)col * ldc + row0;  // S[col][row0 .. row0 + 3]
  if (!diag && (ldc & 3) == 0 && row0 + 3 < M) {
    *reinterpret_cast<float4*>(dst) = make_float4(w[0], w[1], w[2], w[3]);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (row0 + e < M && (!diag || row0 + e < col)) dst[e] = w[e];
  }
}

}  // namespace

// (tile t, piece q) of a plain (not triangular) problem split over K: the
// K ranges' float4 q of every thread summed in range order, plus the bf16
// residual at the same entries, stored as bf16 (the decoder layer's output
// projections).
__global__ __launch_bounds__(NT) void splitk_resid_kernel(const GemmProblem P, const bf16_t* __restrict__ res,
                                                          bf16_t* __restrict__ out, int ldc) {
  const int t = blockIdx.x >> 4, q = blockIdx.x & 15;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int ks = P.ksplit > 1 ? P.ksplit : 1;
  const int tm = t / P.tiles_n, tn = t - tm * P.tiles_n;
  const float4* src = static_cast<const float4*>(P.C);
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int kc0 = 0; kc0 < ks; kc0 += 8) {
    float4 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (kc0 + u < ks) x[u] = src[((long long)(kc0 + u) * P.tiles_tri + t) * (16 * NT) + q * NT + tid];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (kc0 + u < ks) {
        v.x += x[u].x;
        v.y += x[u].y;
        v.z += x[u].z;
        v.w += x[u].w;
      }
  }
  const int i = q >> 3, j = (q >> 2) & 1, g = q & 3;
  const int col = tn * BN + wn * 64 + j * 32 + acc_col(lane);
  const int row0 = tm * BM + wm * 64 + i * 32 + 8 * g + 4 * (lane >> 5);
  if (col >= P.N) return;
  const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = row0 + e;
    if (row < P.M) {
      const long long at = (long long)row * ldc + col;
      out[at] = f32_to_bf16(f[e] + bf16_to_f32(res[at]));
    }
  }
}

hipError_t launch_splitk_resid(const GemmProblem& P, const void* res, void* out, int ldc, hipStream_t s) {
  if (P.tiles_tri == 0) return hipSuccess;
  return launch_kernel("splitk_resid", splitk_resid_kernel, dim3(P.tiles_tri * 16), dim3(NT), 0, s, P,
                       static_cast<const bf16_t*>(res), static_cast<bf16_t*>(out), ldc);
}

hipError_t launch_gram_reduce(const GemmProblem& partial, float* out, int ldc, const float* rs, hipStream_t s,
                              const char* name) {
  if (partial.tiles_tri == 0 || partial.batch == 0) return hipSuccess;
  return launch_kernel(name, gram_reduce_kernel, dim3(partial.tiles_tri * 16, partial.batch), dim3(NT), 0,
                       s, partial, out, ldc, rs);
}

// Compute units of the current device (cached per device).
static int gemm_cus() {
  static int cached[16] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return 256;
  if (cached[dev] == 0) {
    int c = 0;
    cached[dev] = hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && c > 0 ? c : 256;
  }
  return cached[dev];
}

// Tiles of `wide` columns over a problem's columns (EPI_SILU: half of a
// tile's columns are gate columns, the other half their up columns).
static int col_tiles(const GemmProblem& p, int wide) {
  if (p.epi == EPI_SILU) wide /= 2;
  return (p.N + wide - 1) / wide;
}

// Tile counts and order of a problem list with tiles of p.th rows by `wide` columns.
static void count_tiles(GemmBatch& g, int wide) {
  int begin = 0;
  for (int i = 0; i < g.count; ++i) {
    GemmProblem& p = g.p[i];
    p.tiles_m = (p.M + p.th - 1) / p.th;
    p.tiles_n = col_tiles(p, wide);
    p.tiles_tri = p.triangular ? p.tiles_m * (p.tiles_m + 1) / 2 : p.tiles_m * p.tiles_n;
    p.tiles_per_batch = p.tiles_tri * (p.ksplit > 1 ? p.ksplit : 1);
    g.begin[i] = begin;
    begin += p.tiles_per_batch * p.batch;
  }
  g.total_tiles = begin;
  g.first_tiles = 0;
  g.last_tiles = begin;
}

static void finalize_tiles(GemmBatch& g, int tile) {
  for (int i = 0; i < g.count; ++i) g.p[i].th = tile;
  count_tiles(g, tile);
  // Classes of tiles, each spread evenly over the XCDs, one dispatched after
  // the other: trailing problems of at most half the first one's K (the weight
  // folds) come last.  Dealt out with the long ones, 16 short tiles on top of
  // 248 long ones left seven XCDs 33 long tiles for their 32 compute units, a
  // second wave of workgroups for one tile each (three 1225-token images: 69
  // us, now 52).  A Gram matrix before them, whose tiles take longer over their
  // epilogue, is a class of its own once the long tiles take more than one
  // round: with layer 1's in one class some XCDs get nothing but Gram tiles, two
  // rounds of them (three images of 1339 tokens, D_h = 512, 88.5 us, so 82.3;
  // in one round, 576 tokens on 64 x 64 tiles 22.0, so 22.3).
  int q = g.count;
  while (q > 1 && 2 * g.p[q - 1].K <= g.p[0].K) --q;
  if (q < g.count) g.last_tiles = g.begin[q];
  if (q > 1 && g.p[q - 1].epi == EPI_COSINE && g.last_tiles > gemm_cus()) g.first_tiles = g.begin[q - 1];
}

void gemm_finalize(GemmBatch& g) { finalize_tiles(g, BM); }

// K ranges of a split problem: equal ranges (K / ksplit) or kchunk-long ones
// with a shorter last range, each a multiple of 256 but the last, which is
// what K leaves: 256 at least, since the direct-load kernel starts with the
// loads of four slices of 64 whatever the range's length (K itself is a
// multiple of 64).
static bool k_ranges_ok(const GemmProblem& p) {
  if (p.ksplit <= 1) return true;
  if (p.kchunk > 0) return p.kchunk % 256 == 0 && p.K - (long long)(p.ksplit - 1) * p.kchunk >= 256;
  return p.K % p.ksplit == 0 && (p.K / p.ksplit) % 256 == 0;
}

// The epilogues of the direct-load kernel (the RoPE epilogue runs in the
// register-staged kernel or the projection kernel).
static bool dma_epilogue(int e) {
  return e == EPI_BIAS_GELU || e == EPI_BIAS || e == EPI_COSINE || e == EPI_PARTIAL || e == EPI_SILU || epi_direct(e);
}

static int silu_problems(const GemmBatch& g) {
  int n = 0;
  for (int i = 0; i < g.count; ++i) n += g.p[i].epi == EPI_SILU;
  return n;
}

bool gemm_direct_loads(map_dtype dt, const GemmBatch& g) {
  if (dt != MAP_BF16) return false;
  const int silu = silu_problems(g);  // all of a launch's problems or none
  bool dma = silu == 0 || silu == g.count;  // every problem meets the direct-load requirements
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    // (128 x 128 tiles: whole slices, four at least; K % 256 sent widths such
    // as 1152 to the register-staged kernel: 1450 x 2 tokens 59 us)
    dma = dma && dma_epilogue(p.epi) && p.K % 64 == 0 && p.K >= 256 && p.lda % 8 == 0 && p.ldb % 8 == 0 &&
          (reinterpret_cast<uintptr_t>(p.A) & 15) == 0 && (reinterpret_cast<uintptr_t>(p.B) & 15) == 0 &&
          p.strideA % 8 == 0 && p.strideB % 8 == 0 &&
          k_ranges_ok(p);
  }
  return dma;
}

// Costs of a tile, in hundredths of a 256 x 256 tile over the same K.
constexpr int kCost256 = 100, kCost192 = 79, kCost128 = 56;
// A 128 x 128 tile of the other kernel; over a short K a second round of them
// starts while the first one's rows are still on their way out (2 rounds over
// 256 take 14 to 18 us, one tile 9 to 12; large tiles of 192 rows 19 to 22).
static int cost_small(int K) { return K < 512 ? 36 : 43; }

// Cost c of a tile over the first problem's K, for a tile over K instead: a
// tile's start and epilogue take as long as about 800 of K (256 tiles of 256 x
// 256: 23 us at K = 256, 38 at 1024, 102 at 4096; of 128 x 128: 9, 17, 39).
static long long cost_at(long long c, int K, const GemmBatch& g) { return c * (K + 800) / (g.p[0].K + 800); }

// Time of `full` tiles of cost c, dispatched first, and `low` tiles of 128
// rows after them, one tile at a time on each of `cus` units.
static long long makespan(long long full, long long c, long long low, long long cus) {
  const long long rounds = full / cus, rem = full % cus;
  long long t = rounds * c;
  if (rem) {  // the units free in the last round of full tiles take low ones meanwhile
    t += c;
    low -= (cus - rem) * std::max(1LL, (c + c / 8) / kCost128);
  }
  return t + (low > 0 ? (low + cus - 1) / cus * kCost128 : 0);
}

// The tiles of 256 columns for a launch: whether they apply (row-wise
// epilogues and upper triangles with the cosine epilogue, no K split), their
// cost, and the launch's problem list q with tile heights `tm` or, dispatched
// after those, 128 rows.  The largest problem without an upper triangle is
// cut at the multiple of tm that lets the last round of workgroups end
// earliest; the others' tiles count as they are.
static long long plan_big(const GemmBatch& g, GemmBatch& q, int& tm) {
  if (g.norm_blocks) return -1;
  for (int i = 0; i < g.count; ++i)  // slices in pairs; its loads' 32-bit byte offsets (an index map reaches kSubsetMaxN rows)
    if (g.p[i].K % 128 != 0 || g.p[i].lda > (1 << 17) || g.p[i].ldb > (1 << 17) ||
        (g.p[i].epi == EPI_SILU && 2LL * g.p[i].ldb * (g.p[i].N + kBig) > INT32_MAX))
      return -1;
  if (g.norm_tiles > 0 && (g.norm_tiles > g.count || g.p[g.norm_tiles - 1].batch != 1)) return -1;
  int cut = -1, same = 0;  // the problem to cut; whether every problem has row-wise tiles
  long long most = 0;
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    const bool gram = p.epi == EPI_COSINE && p.triangular && p.M == p.N;
    if (!(p.epi == EPI_BIAS || p.epi == EPI_BIAS_GELU || p.epi == EPI_SILU || epi_direct(p.epi) || gram) || p.ksplit > 1 ||
        (p.triangular && !gram))
      return -1;
    same += !gram;
    const long long work = (long long)p.M * p.N * p.K;
    if (!gram && !p.mapA && p.batch == 1 && work > most) {
      most = work;
      cut = i;
    }
  }
  const long long cus = gemm_cus();
  long long best = -1;
  int best_tm = kBig, best_rows = 0;
  for (const int t : {256, 192}) {
    if (t == 192 && (same < g.count || g.norm_tiles)) continue;
    const long long c = t == 256 ? kCost256 : kCost192;
    long long full = 0, low = 0;  // of the problems that stay whole
    for (int i = 0; i < g.count; ++i) {
      const GemmProblem& p = g.p[i];
      const long long a = (p.M + t - 1) / t, b = col_tiles(p, kBig);
      if (i == cut) continue;
      if (p.triangular) full += a * (a + 1) / 2 * p.batch;
      else if (p.M <= 128 || 2 * p.K <= g.p[0].K) low += a * b * p.batch;
      else full += a * b * p.batch;
    }
    const int M = cut >= 0 ? g.p[cut].M : 0;
    const long long b = cut >= 0 ? col_tiles(g.p[cut], kBig) : 0;
    // f tile rows of t, the rest of 128.  Of the f with one number of rounds
    // of full tiles the largest is never the dearer: one row of them less
    // leaves units free for at most the tiles of 128 that take its place.
    for (long long f = M / t + (M % t > 128); f >= 0;) {
      const int rest = static_cast<int>(std::max(0LL, M - f * t));
      const long long cost = makespan(full + f * b, c, low + (rest + 127) / 128 * b, cus);
      if (best < 0 || cost < best) {
        best = cost;
        best_tm = t;
        best_rows = static_cast<int>(std::min<long long>(M, f * t));
      }
      const long long fewer = ((full + f * b + cus - 1) / cus - 1) * cus - full;  // full tiles in one round less
      f = cut < 0 || fewer < 0 ? -1 : fewer / b;
    }
  }
  // no launch is shorter than its longest tile (the training step's short
  // products: tiles over 1024 among those over 256, 152 large tiles 22.0 us, 400
  // of 128 x 128 20.6)
  for (int i = 0; i < g.count; ++i) {
    const bool late = i == cut ? best_rows == 0 : !g.p[i].triangular && g.p[i].M <= 128;
    const long long c = late ? kCost128 : best_tm == 256 ? kCost256 : kCost192;
    if (g.p[i].K > g.p[0].K) best = std::max(best, cost_at(c, g.p[i].K, g));
  }
  tm = best_tm;
  // the problem list: full tiles, then tiles of 128 rows and short sums
  q = g;
  q.count = 0;
  q.norm_tiles = g.norm_tiles;
  for (int late = 0; late < 2; ++late) {
    if (late) q.first_tiles = q.count;  // (a problem index until the tiles are counted)
    for (int i = 0; i < g.count; ++i) {
      GemmProblem p = g.p[i];
      p.norm_at = g.norm_tiles == i + 1 ? 1 : 0;
      p.th = best_tm;
      if (i == cut) {
        if (late ? best_rows == p.M : best_rows == 0) continue;
        if (late) {
          p.th = 128;
          p.A = static_cast<const bf16_t*>(p.A) + (long long)best_rows * p.lda;
          const long long at = (long long)best_rows * p.ldc;
          p.C = static_cast<char*>(p.C) + at * (p.epi == EPI_F32 ? 4 : 2);
          if (p.aux) p.aux = static_cast<char*>(p.aux) + at * 2;
          if (p.norm_at) p.norm_at += best_rows;
          p.M -= best_rows;
        } else {
          p.M = best_rows;
        }
      } else if (late != (!p.triangular && (p.M <= 128 || 2 * p.K <= g.p[0].K) ? 1 : 0)) {
        continue;
      }
      q.p[q.count++] = p;
    }
  }
  const int first = q.first_tiles;
  count_tiles(q, kBig);
  if (first > 0 && first < q.count) q.first_tiles = q.begin[first];
  return best;
}

// 128 x 128 tiles' time in the same units: rounds of the long tiles, then
// what the units free in the last one have not taken of the short sums.
static long long small_tiles_cost(const GemmBatch& g) {
  long long full = 0, brief = 0, kb = 1;
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    const long long a = (p.M + 127) / 128, b = col_tiles(p, BN), n = (p.triangular ? a * (a + 1) / 2 : a * b) * p.batch;
    const bool late = i > 0 && 2 * p.K <= g.p[0].K;
    (late ? brief : full) += n;
    if (late) kb = std::max<long long>(kb, p.K);
  }
  const long long cus = gemm_cus(), rounds = (full + cus - 1) / cus, k0 = std::max(1, g.p[0].K), c = cost_small(g.p[0].K);
  const long long left = std::max(0LL, brief - (rounds * cus - full) * (k0 / kb));
  long long t = rounds * c + (left + cus - 1) / cus * (c * kb / k0);
  for (int i = 0; i < g.count; ++i)
    if (g.p[i].K > g.p[0].K) t = std::max(t, cost_at(c, g.p[i].K, g));
  return t;
}

static bool big_tiles_pay(const GemmBatch& g, GemmBatch& q, int& tm) {
  const long long big = plan_big(g, q, tm);
  return big >= 0 && big < small_tiles_cost(g);
}

// Whether a launch meets the 64 x 64 tiles' requirements.
static bool tile64_fits(const GemmBatch& g, int vec, int bk) {
  if (g.norm_blocks || g.norm_tiles) return false;
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    if (p.epi == EPI_ROPE || p.epi == EPI_PARTIAL || p.epi == EPI_SILU || p.ksplit > 1 || p.mapA || p.mapB ||
        p.K % bk != 0 || p.lda % vec != 0 || p.ldb % vec != 0 || p.strideA % vec != 0 || p.strideB % vec != 0 ||
        (reinterpret_cast<uintptr_t>(p.A) & 15) != 0 || (reinterpret_cast<uintptr_t>(p.B) & 15) != 0)
      return false;
  }
  return true;
}

// 64 x 64 tiles for a bf16 launch when one round of workgroups holds all of
// its long ones: a round then takes half as long as one of 128 x 128 tiles;
// two rounds would take as long.
static bool tile64_pays(const GemmBatch& g) {
  long long n = 0;
  for (int i = 0; i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    const long long a = (p.M + kTile - 1) / kTile, b = (p.N + kTile - 1) / kTile;
    if (i == 0 || 2 * p.K > g.p[0].K) n += (p.triangular ? a * (a + 1) / 2 : a * b) * p.batch;
  }
  return n <= gemm_cus();
}

bool gemm_big_tiles(map_dtype dt, const GemmBatch& g) {
  GemmBatch q;
  int tm;
  return gemm_direct_loads(dt, g) && big_tiles_pay(g, q, tm);
}

bool gemm_small_tiles(map_dtype dt, const GemmBatch& g) {
  return gemm_direct_loads(dt, g) && !gemm_big_tiles(dt, g) && tile64_fits(g, 8, 64) && tile64_pays(g);
}

hipError_t launch_gemm(map_dtype dt, const GemmBatch& g, const char* name, hipStream_t s) {
  if (g.total_tiles == 0) return hipSuccess;
  if (dt == MAP_BF16) {
    const bool dma = gemm_direct_loads(dt, g);
    GemmBatch q;
    int tm;
    const bool big = dma && big_tiles_pay(g, q, tm);
    if (g.norm_tiles > 0 && !big) return hipErrorInvalidValue;  // the in-tile row norms exist there only
    if (big)
      return launch_kernel(name, g.norm_tiles ? gemm_big_kernel<true, 256> : tm == 192 ? gemm_big_kernel<false, 192> : gemm_big_kernel<false, 256>,
                           dim3(q.total_tiles), dim3(kBigThreads), 0, s, q);
    if (dma && tile64_fits(g, 8, 64) && tile64_pays(g)) {
      q = g;
      finalize_tiles(q, kTile);
      return launch_kernel(name, gemm_tile64_kernel<bf16_t>, dim3(q.total_tiles), dim3(kTileThreads), 0, s, q);
    }
    if (dma)
      return launch_kernel(name, silu_problems(g) > 0 ? gemm_dma_kernel<true> : gemm_dma_kernel<false>,
                           dim3(g.total_tiles + g.norm_blocks), dim3(kDmaThreads), 0, s, g);
    if (g.norm_blocks) return hipErrorInvalidValue;
    for (int i = 0; i < g.count; ++i)  // index maps and K ranges exist in the direct-load kernel only
      if (g.p[i].epi == EPI_PARTIAL || g.p[i].epi == EPI_SILU || g.p[i].mapA || g.p[i].mapB) return hipErrorInvalidValue;
    return launch_kernel(name, gemm_kernel<bf16_t>, dim3(g.total_tiles), dim3(NT), 0, s, g);
  }
  if (g.norm_tiles > 0) return hipErrorInvalidValue;
  if (tile64_fits(g, 4, 32)) {
    GemmBatch q = g;
    finalize_tiles(q, kTile);
    return launch_kernel(name, gemm_tile64_kernel<float>, dim3(q.total_tiles), dim3(kTileThreads), 0, s, q);
  }
  return launch_kernel(name, gemm_kernel<float>, dim3(g.total_tiles), dim3(NT), 0, s, g);
}

hipError_t launch_proj_rope(map_dtype dt, const GemmBatch& g, const char* name, hipStream_t s) {
  bool fits = (dt == MAP_BF16 || dt == MAP_F32) && g.count >= 1 && g.count <= 2;
  const int vec = dt == MAP_F32 ? 4 : 8;  // elements per 16-byte load
  for (int i = 0; fits && i < g.count; ++i) {
    const GemmProblem& p = g.p[i];
    fits = p.epi == EPI_ROPE && p.batch == 1 && p.N <= 128 && p.N % 2 == 0 && p.K % vec == 0 &&
           p.lda % vec == 0 && p.ldb % vec == 0 && (reinterpret_cast<uintptr_t>(p.A) & 15) == 0 &&
           (reinterpret_cast<uintptr_t>(p.B) & 15) == 0;
  }
  // With enough rows for a wave of 128 x 128 tiles, the tiled kernel reads
  // B once per tile instead of once per 32 rows.
  long long rows = 0;
  for (int i = 0; i < g.count; ++i) rows += g.p[i].M;
  if (!fits || rows >= 128LL * gemm_cus()) return launch_gemm(dt, g, name, s);
  GemmBatch q = g;
  int total = 0;
  for (int i = 0; i < q.count; ++i) {
    q.p[i].tiles_m = q.p[i].M > 0 ? kPG * ((q.p[i].M + kPR - 1) / kPR) : 0;
    total += q.p[i].tiles_m;
  }
  if (q.count == 1) q.p[1].tiles_m = 0;
  q.total_tiles = total;
  if (total == 0) return hipSuccess;
  if (dt == MAP_F32) return launch_kernel(name, proj_rope_kernel<float>, dim3(total), dim3(kPW * 64), 0, s, q);
  return launch_kernel(name, proj_rope_kernel<bf16_t>, dim3(total), dim3(kPW * 64), 0, s, q);
}

}  // namespace mapk
