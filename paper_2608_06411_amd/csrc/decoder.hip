// The language model's first layer over the pruned input (section
// "Inference-Time Token Pruning": after pruning, the model processes only
// the K kept visual tokens and the question tokens, which is where the
// prefill speedup comes from).  The layer is LLaMA's, in bf16 with float32
// arithmetic:
//
//   h = RMSNorm(x) g_attn;  qkv = h W_qkv^T;  RoPE on q and k per head;
//   o = causal softmax(q k^T / sqrt(d_h)) v;  x1 = x + o W_o^T;
//   y = x1 + (SiLU(h2 W_g^T) * (h2 W_u^T)) W_d^T,  h2 = RMSNorm(x1) g_ffn.
//
// The four products run on the matrix-core GEMM (gemm.hip); this file holds
// the kernels between them:
//   rmsnorm     one workgroup per row, 16-byte pieces, float32 sum of squares
//   rope_qkv    rotates q and k in place, angles pos * theta^(-2i/d_h) in float64
//   attention   one workgroup per (64 or 128 query rows, head, sequence): the
//               key blocks up to the diagonal through LDS on the bf16 matrix
//               cores with an online softmax; the causal mask follows the
//               rows' order in their sequence
//   silu_mul    SiLU(gate) * up, 8 entries per thread, where the product did not
//               form it in its epilogue (weights off a 16-byte boundary)
#include "internal.h"

namespace mapk {

namespace {

constexpr int NT = 256;
constexpr int DH = 128;  // head width (the 7B models' 4096 / 32)

union Bf8 {
  uint4 u;
  bf16_t e[8];
};

__device__ __forceinline__ float block_sum256(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const float r = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return r;
}

// out[r] = x[r] / sqrt(mean(x[r]^2) + eps) * g, rows of d bf16 (d % 8 == 0,
// d <= 8192: each thread holds up to four 16-byte pieces of its row).
__global__ __launch_bounds__(NT) void rmsnorm_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ g,
                                                     bf16_t* __restrict__ out, int d, float eps) {
  __shared__ float red[4];
  const int r = blockIdx.x, pieces = d >> 3;
  const uint4* src = reinterpret_cast<const uint4*>(x + (long long)r * d);
  Bf8 v[4];
  float ss = 0.0f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = threadIdx.x + u * NT;
    v[u].u = c < pieces ? src[c] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float f = bf16_to_f32(v[u].e[k]);
      ss = fmaf(f, f, ss);
    }
  }
  const float inv = 1.0f / sqrtf(block_sum256(ss, red) / static_cast<float>(d) + eps);
  const uint4* gp = reinterpret_cast<const uint4*>(g);
  uint4* dst = reinterpret_cast<uint4*>(out + (long long)r * d);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = threadIdx.x + u * NT;
    if (c >= pieces) continue;
    Bf8 w, o;
    w.u = gp[c];
#pragma unroll
    for (int k = 0; k < 8; ++k) o.e[k] = f32_to_bf16(bf16_to_f32(v[u].e[k]) * inv * bf16_to_f32(w.e[k]));
    dst[c] = o.u;
  }
}

// Row r: pair i (i, i + 64) of every head of q and of k turned by the angle
// pos[r] theta^(-2i/128): (a, b) -> (a cos - b sin, b cos + a sin).
__global__ __launch_bounds__(NT) void rope_qkv_kernel(const DecoderArgs a) {
  const int r = blockIdx.x, i = threadIdx.x & 63, hg = threadIdx.x >> 6;
  double sn, cs;
  sincos(static_cast<double>(a.pos[r]) * a.inv_freq[i], &sn, &cs);
  const float c = static_cast<float>(cs), s = static_cast<float>(sn);
  bf16_t* row = static_cast<bf16_t*>(a.qkv) + (long long)r * 3 * a.d;
  for (int h = hg; h < 2 * a.n_heads; h += 4) {  // q heads, then k heads
    bf16_t* p = row + h * DH;
    const float x = bf16_to_f32(p[i]), y = bf16_to_f32(p[i + DH / 2]);
    p[i] = f32_to_bf16(x * c - y * s);
    p[i + DH / 2] = f32_to_bf16(y * c + x * s);
  }
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

// Row and column of accumulator register r of lane `lane` in a 32 x 32
// matrix-core block.
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// One global_load_lds_dwordx4: lane l's 16 bytes at gsrc land at byte 16 l of
// the wave's 1 KiB at LDS address m (wave-uniform).  The wait before each
// block's barrier covers it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // M0 is written here and nowhere else in the file
__device__ __forceinline__ void dma16(const void* gsrc, uint32_t m) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gsrc), "s"(m) : "memory", "m0");
}
#pragma clang diagnostic pop

// Causal attention, flash-style on the bf16 matrix cores (32 x 32 x 16,
// float32 accumulation).  Workgroup (query block of 32 NW rows, head h,
// sequence b); wave w owns 32 query rows and their softmax.  Both products
// are formed transposed, S^T = K Q^T and O^T = V^T P^T, so that a lane holds
// one query (column lane & 31) throughout: the row maximum and sum are sums
// over its own registers and one exchange with lane ^ 32, the running
// statistics and the rescaling are per lane, and the scores become the
// second product's operand in place (its keys are taken in the order in
// which the lane holds them; V^T is stored in that order).  Nothing but K and V
// passes through LDS: 64 keys at a time, two buffers, one barrier per block,
// the next block's loads under this block's products.  Output rows are
// rescaled only when a row's maximum has grown by more than 2^6 (the sums
// carry the same factor, so the result is the same softmax).
// What bounds it: each block's 32 products of a wave (1024 clocks) and the
// about as long vector work of its softmax, on two waves per SIMD.  The
// scores took a trip through LDS and five barriers per block before:
// 2944 rows, 32 heads: 332 us, now 140 to 153 (fastest and median of 20); 224
// rows: 20 us, now 12 to 14.
constexpr int kKeys = 64;              // keys per block
constexpr int kKBytes = kKeys * DH * 2;  // one buffer of K, and of V^T
constexpr float kRescale = 6.0f;       // log2 of the growth that a row's factor may lag behind

// 16-byte chunk c of K row r sits at position c ^ (r & 15) of the row's 16;
// chunk c of V^T row (dim) r at c ^ vswz(r) of its 8.
__device__ __forceinline__ int vswz(int r) { return ((r >> 1) ^ (r >> 4)) & 7; }

template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void attention_kernel(const DecoderArgs a) {
  __shared__ __attribute__((aligned(1024))) uint4 lds[4 * kKBytes / 16];  // K, K, V^T, V^T
  constexpr int NTH = 64 * NW;
  constexpr int KI = 16 / NW;                // K: instructions of 4 rows per wave
  constexpr int VI = 32 * 16 / NTH;          // V: (pair of keys, 8 dims) items per thread
  const int h = blockIdx.y, b = blockIdx.z;
  const int s0 = a.seq_off[b], S = a.seq_off[b + 1] - s0;
  const int q0 = (gridDim.x - 1 - blockIdx.x) * 32 * NW;  // the longest first
  if (q0 >= S) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const long long ld = 3LL * a.d;
  const bf16_t* qkv = static_cast<const bf16_t*>(a.qkv) + s0 * ld + h * DH;
  const int nblk = (min(q0 + 32 * NW, S) + kKeys - 1) / kKeys;
  const int qw = q0 + 32 * wave, mine = qw < S ? (min(qw + 31, S - 1)) / kKeys + 1 : 0;  // this wave's blocks
  const int q = qw + lr;  // this lane's query

  bf16x8_t qf[8];  // the query's values 16 st + 8 lh + (0..7)
  {
    const bf16_t* row = qkv + min(q, S - 1) * ld + 8 * lh;
#pragma unroll
    for (int st = 0; st < 8; ++st) qf[st] = *reinterpret_cast<const bf16x8_t*>(row + 16 * st);
  }
  const uint32_t k_lds = static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void*)&lds[0]));
  auto load_k = [&](int kb) {  // rows past the sequence read its last row (masked below)
#pragma unroll
    for (int u = 0; u < KI; ++u) {
      const int r = 4 * (wave * KI + u) + (lane >> 4), c = (lane & 15) ^ (r & 15);
      dma16(qkv + min(kb * kKeys + r, S - 1) * ld + a.d + 8 * c,
            k_lds + static_cast<uint32_t>(kb & 1) * kKBytes + 1024u * (wave * KI + u));
    }
  };
  Bf8 va[VI], vb[VI];
  auto load_v = [&](int kb) {
#pragma unroll
    for (int u = 0; u < VI; ++u) {
      const int e = tid + NTH * u, c = e & 15, j = e >> 4;
      const int k = kb * kKeys + 2 * j;
      va[u].u = *reinterpret_cast<const uint4*>(qkv + min(k, S - 1) * ld + 2 * a.d + 8 * c);
      vb[u].u = *reinterpret_cast<const uint4*>(qkv + min(k + 1, S - 1) * ld + 2 * a.d + 8 * c);
    }
  };
  // V^T[dim][position]: key k of a block sits at position k with bits 2 and
  // 3 exchanged (within every 16: keys 0-3, 8-11, 4-7, 12-15)
  auto store_v = [&](int kb) {
    char* vt = reinterpret_cast<char*>(lds) + (2 + (kb & 1)) * kKBytes;
#pragma unroll
    for (int u = 0; u < VI; ++u) {
      const int e = tid + NTH * u, c = e & 15, k = 2 * (e >> 4);
      const int pos = (k & ~12) | ((k & 4) << 1) | ((k & 8) >> 1);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int dim = 8 * c + i;
        *reinterpret_cast<uint32_t*>(vt + dim * (2 * kKeys) + 16 * ((pos >> 3) ^ vswz(dim)) + 2 * (pos & 7)) =
            static_cast<uint32_t>(va[u].e[i]) | (static_cast<uint32_t>(vb[u].e[i]) << 16);
      }
    }
  };

  f32x16_t o[4];  // O^T: rows 32 d4 + acc_row = dims, column lr = the query
#pragma unroll
  for (int d4 = 0; d4 < 4; ++d4)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d4][r] = 0.0f;
  const float c2 = 1.4426950408889634f / sqrtf(static_cast<float>(DH));  // log2(e) / sqrt(d_h)
  // The row's factor 2^-m (both halves agree) and this half's sum.  m starts
  // below every finite score but finite, so that a row whose scores so far
  // are all -inf (products past float32's range) has zero probabilities there
  // and not 2^(-inf + inf).
  float m = -3.0e38f, l = 0.0f;

  load_k(0);
  load_v(0);
  for (int kb = 0; kb < nblk; ++kb) {
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's part of K; V below
    store_v(kb);
    __syncthreads();
    if (kb + 1 < nblk) {
      load_k(kb + 1);
      load_v(kb + 1);
    }
    if (kb >= mine) continue;  // (uniform over the wave; it still loads for the others)
    const uint4* K4 = lds + (kb & 1) * (kKBytes / 16);
    const uint4* V4 = lds + (2 + (kb & 1)) * (kKBytes / 16);
    f32x16_t sc[2];  // S^T: rows = keys 32 t + acc_row, column = the query
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[t][r] = 0.0f;
#pragma unroll
    for (int st = 0; st < 8; ++st)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int row = 32 * t + lr;
        sc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8_t, K4[row * 16 + ((2 * st + lh) ^ (row & 15))]), qf[st], sc[t], 0, 0, 0);
      }
    if (kb * kKeys + kKeys - 1 > qw) {  // the diagonal
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb * kKeys + 32 * t + acc_row(r, lane) > q) sc[t][r] = -INFINITY;
    }
    float mx = sc[0][0];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[t][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c2;
    if (__any(mx > m + kRescale)) {
      const float mn = fmaxf(m, mx), al = __builtin_amdgcn_exp2f(m - mn);  // (first finite block: 0)
      m = mn;
      l *= al;
#pragma unroll
      for (int d4 = 0; d4 < 4; ++d4)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d4][r] *= al;
    }
    bf16x8_t pf[4];  // the probabilities of steps of 16 keys
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float pv = __builtin_amdgcn_exp2f(fmaf(sc[st >> 1][8 * (st & 1) + k], c2, -m));
        l += pv;
        pf[st][k] = static_cast<__bf16>(pv);
      }
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int d4 = 0; d4 < 4; ++d4) {
        const int row = 32 * d4 + lr;
        o[d4] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8_t, V4[row * 8 + ((2 * st + lh) ^ vswz(row))]), pf[st], o[d4], 0, 0, 0);
      }
  }
  __syncthreads();  // K and V are read out: each wave's output rows through LDS, 128 + 8 values apart
  if (mine == 0) return;
  const float inv = 1.0f / (l + __shfl_xor(l, 32, 64));
  bf16_t* ot = reinterpret_cast<bf16_t*>(lds) + wave * 32 * (DH + 8);
#pragma unroll
  for (int d4 = 0; d4 < 4; ++d4)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      ushort4 w;
      w.x = f32_to_bf16(o[d4][4 * g] * inv);
      w.y = f32_to_bf16(o[d4][4 * g + 1] * inv);
      w.z = f32_to_bf16(o[d4][4 * g + 2] * inv);
      w.w = f32_to_bf16(o[d4][4 * g + 3] * inv);
      *reinterpret_cast<ushort4*>(ot + lr * (DH + 8) + 32 * d4 + 8 * g + 4 * lh) = w;
    }
  bf16_t* out = static_cast<bf16_t*>(a.o) + (long long)(s0 + qw) * a.d + h * DH;
#pragma unroll
  for (int u = 0; u < 8; ++u) {  // (this wave's own rows: no barrier)
    const int r = 4 * u + (lane >> 4), c = 8 * (lane & 15);
    if (qw + r < S) *reinterpret_cast<uint4*>(out + (long long)r * a.d + c) = *reinterpret_cast<const uint4*>(ot + r * (DH + 8) + c);
  }
}

// act[r][i] = SiLU(gu[r][i]) * gu[r][ff + i], 8 entries per thread.
__global__ __launch_bounds__(NT) void silu_mul_kernel(const DecoderArgs a) {
  const long long e = (long long)blockIdx.x * NT + threadIdx.x, per = a.ff >> 3;
  if (e >= (long long)a.R * per) return;
  const long long r = e / per, p = e - r * per;
  const bf16_t* gu = static_cast<const bf16_t*>(a.gu) + r * 2 * a.ff;
  Bf8 g, u, o;
  g.u = reinterpret_cast<const uint4*>(gu)[p];
  u.u = reinterpret_cast<const uint4*>(gu + a.ff)[p];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float x = bf16_to_f32(g.e[k]);
    o.e[k] = f32_to_bf16(x / (1.0f + __expf(-x)) * bf16_to_f32(u.e[k]));
  }
  reinterpret_cast<uint4*>(static_cast<bf16_t*>(a.act) + r * a.ff)[p] = o.u;
}

}  // namespace

hipError_t launch_rmsnorm(const DecoderArgs& a, const void* x, const void* g, void* out, hipStream_t s) {
  return launch_kernel("rmsnorm", rmsnorm_kernel, dim3(a.R), dim3(NT), 0, s, static_cast<const bf16_t*>(x),
                       static_cast<const bf16_t*>(g), static_cast<bf16_t*>(out), a.d, a.eps);
}

hipError_t launch_rope_qkv(const DecoderArgs& a, hipStream_t s) {
  return launch_kernel("rope_qkv", rope_qkv_kernel, dim3(a.R), dim3(NT), 0, s, a);
}

hipError_t launch_attention(const DecoderArgs& a, hipStream_t s) {
  // 128 query rows per workgroup share each block of K and V; with fewer of
  // them than two per compute unit, 64 rows, so that more units work.
  const long long wide = (long long)((a.max_len + 127) / 128) * a.n_heads * a.B;
  if (wide >= 512)
    return launch_kernel("attention", attention_kernel<4>, dim3((a.max_len + 127) / 128, a.n_heads, a.B), dim3(256), 0,
                         s, a);
  return launch_kernel("attention", attention_kernel<2>, dim3((a.max_len + 63) / 64, a.n_heads, a.B), dim3(128), 0, s, a);
}

hipError_t launch_silu_mul(const DecoderArgs& a, hipStream_t s) {
  const long long n = (long long)a.R * (a.ff >> 3);
  return launch_kernel("silu_mul", silu_mul_kernel, dim3(static_cast<unsigned>((n + NT - 1) / NT)), dim3(NT), 0, s, a);
}

}  // namespace mapk
