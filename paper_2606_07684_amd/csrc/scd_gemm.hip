// Generic MFMA kernel of the SCD codec: C[M, n] = prologue(A)[M, k] * B[n, k]^T, epilogue.
//
// One launch runs a table of jobs that share M.  Every Reuse-decode branch (Eq. decode_kv),
// every Patch branch (Eq. kv_from_patch) and every encode branch (Eq. encode_z_kv and the Patch
// code of Section 4.4.1) is one such product:
//   decode  A = codes [T*g, r]      B = W_dec [w, r]     epilogue + mu, RoPE on keys
//   patch   A = H_hat [T, d_model]  B = W_K|W_V [D, d]   epilogue + bias, RoPE on keys
//   encode  A = K|V  [T*g, w]       B = W_enc [r, w]     prologue deRoPE on keys, - mu
//
// A wave computes 32 x 64 or 32 x 32 outputs with both operands read straight from the caches into
// registers, one step ahead of use: no LDS staging and no barriers, so waves never wait for each
// other.  bf16 uses v_mfma_f32_16x16x32_bf16, fp32 v_mfma_f32_16x16x4_f32, both accumulating in fp32.
// The B rows (output columns) are the MFMA's first operand, so a lane ends with four consecutive
// outputs of one row (eight over two blocks) and stores them as one vector.  A lane holds 16 bytes of
// a row per block, so a load covers 16 rows x 64 bytes.  When the input needs deRoPE a step's two
// blocks are columns i and i + d_h/2 of one head; when the output is rotated a wave's column blocks are
// heads' first halves and their partners: every RoPE pair meets in one lane's registers.
//
// The shape follows the launch (generic_shape): four waves along the rows when there are enough of
// them to fill the chip; else one tile per workgroup whose waves split the contraction (their sums meet
// in LDS, added in wave order), so that short prefixes and thin codes do not wait on one wave's chain
// of loads.  fp32 is bound by the MFMA rate (32 cycles per 16 x 16 x 4), small launches by latency:
// the smallest model's codec (512 tokens, 4 layers) takes 32 us in four launches; on 128 x 128 tiles
// through LDS it took 193 us, three quarters of each 32-code tile computed for nothing.
#include <type_traits>

#include "scd_kernels.h"

namespace scd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kNumXcd = 8;

// Workgroups are dispatched round-robin over the XCDs.  Renumber them so each XCD receives a
// contiguous range of tiles: neighbouring tiles (which share A rows) then share one L2.
__device__ inline int xcd_remap(int bid, int nb) {
  const int q = nb / kNumXcd, rem = nb % kNumXcd;
  const int x = bid % kNumXcd, i = bid / kNumXcd;
  return (x < rem ? x * (q + 1) : rem * (q + 1) + (x - rem) * q) + i;
}

// Position of code row `row` (token row / g) within its own request.
__device__ inline int64_t row_position(const GemmParams& p, int64_t row) {
  if (row >= p.m) return 0;
  int64_t t = row / p.g;
  int b = 0;
  if (p.cu_seqlens != nullptr) {
    int lo = 0, hi = p.n_seqs - 1;  // largest b with cu[b] <= t
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (p.cu_seqlens[mid] <= t) lo = mid; else hi = mid - 1;
    }
    b = lo;
    t -= p.cu_seqlens[b];
  }
  return t + (p.pos0 != nullptr ? p.pos0[b] : 0);
}

__device__ inline int64_t table_row(const GemmParams& p, int64_t pos) {
  return pos < 0 ? 0 : (pos >= p.max_pos ? p.max_pos - 1 : pos);
}

template <bool BF16> struct Elem;
template <> struct Elem<true> {
  using T = uint16_t;
  static constexpr int kLane = 8;  // elements of a 16-byte vector
  __device__ static inline void unpack(const uint4& v, float* f) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  __device__ static inline uint32_t bits(float f) {
    return static_cast<uint32_t>(__builtin_bit_cast(uint16_t, static_cast<__bf16>(f)));
  }
  __device__ static inline uint4 pack(const float* f) {
    return make_uint4(bits(f[0]) | (bits(f[1]) << 16), bits(f[2]) | (bits(f[3]) << 16),
                      bits(f[4]) | (bits(f[5]) << 16), bits(f[6]) | (bits(f[7]) << 16));
  }
  __device__ static inline float load1(const void* p, int64_t i) {
    return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t*>(p)[i]) << 16);
  }
};
template <> struct Elem<false> {
  using T = float;
  static constexpr int kLane = 4;
  __device__ static inline void unpack(const uint4& v, float* f) {
    f[0] = __uint_as_float(v.x);
    f[1] = __uint_as_float(v.y);
    f[2] = __uint_as_float(v.z);
    f[3] = __uint_as_float(v.w);
  }
  __device__ static inline uint4 pack(const float* f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]),
                      __float_as_uint(f[3]));
  }
  __device__ static inline float load1(const void* p, int64_t i) {
    return static_cast<const float*>(p)[i];
  }
};

// Tag types that name each step's kernel.
struct ReuseDecode {};
struct PatchKV {};
struct EncodeKV {};
struct EncodeH {};
struct PatchAlign {};

// Four consecutive outputs of one row.
template <bool BF16>
__device__ inline void store4(void* base, int64_t i, const float* f) {
  if constexpr (BF16) {
    uint2 v;
    v.x = Elem<true>::bits(f[0]) | (Elem<true>::bits(f[1]) << 16);
    v.y = Elem<true>::bits(f[2]) | (Elem<true>::bits(f[3]) << 16);
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(base) + i) = v;
  } else {
    *reinterpret_cast<float4*>(static_cast<float*>(base) + i) = make_float4(f[0], f[1], f[2], f[3]);
  }
}

// Eight consecutive outputs of one row.
template <bool BF16>
__device__ inline void store8(void* base, int64_t i, const float* f, const float* g) {
  if constexpr (BF16) {
    const float y[8] = {f[0], f[1], f[2], f[3], g[0], g[1], g[2], g[3]};
    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(base) + i) = Elem<true>::pack(y);
  } else {
    store4<false>(base, i, f);
    store4<false>(base, i + 4, g);
  }
}

template <typename OP, bool BF16, int FM, int FN, int WM, int WK>
__global__ __launch_bounds__(WM * WK * 64, 2) void gemm_nt_kernel(GemmParams p) {
  using EL = Elem<BF16>;
  using T = typename EL::T;
  constexpr int VL = EL::kLane;  // contraction elements a lane holds of a block (16 bytes)
  constexpr int KB = 4 * VL;     // contraction of a block
  constexpr int BM = 16 * FM * WM, BN = 16 * FN, FP = FN / 2;
  constexpr bool kEnc = std::is_same<OP, EncodeKV>::value;  // the only step with an input prologue
  static_assert(FN % 2 == 0 && (WK == 1 || (WM == 1 && FM <= WK)), "block split");
  extern __shared__ __attribute__((aligned(16))) float4 red[];  // [WK][FM][FN][64] when WK > 1

  const int lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = WK > 1 ? wave : 0, wm = WK > 1 ? 0 : wave;

  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  int j = 0;
  while (j + 1 < p.n_jobs && bid >= p.jobs[j + 1].tile_begin) ++j;
  const GemmJob job = p.jobs[j];
  const int local = bid - job.tile_begin;
  const int K = job.k, N = job.n;
  const int64_t M = p.m;
  const int ntn = (N + BN - 1) / BN;
  const int64_t m0 = static_cast<int64_t>(local / ntn) * BM + wm * 16 * FM;
  const int n0 = (local % ntn) * BN;
  const bool derope = kEnc && (job.flags & kDeropeIn) != 0;
  const bool vec_in = kEnc && (job.flags & kVecIn) != 0 && job.vec != nullptr;
  const bool rope_out = (job.flags & kRopeOut) != 0;
  const bool vec_out = (job.flags & kVecOut) != 0 && job.vec != nullptr;
  const bool silu_out = (job.flags & kSiluOut) != 0;
  const int dh = p.head_dim, half = dh / 2;

  // Output columns: a lane's outputs of blocks 2q and 2q + 1 are the eight columns 8 (l / 16) + (0..7)
  // of a 32-column group (first column of the group: group_of), so that a bf16 store is 16 bytes.
  // When the output is rotated the first FN / 4 groups are columns of heads' first halves and the rest
  // their partners.  Two blocks, or heads of 32: single 16-column blocks instead (first column:
  // block_of).  -1: past the last column.
  const bool wide = FN == 4 && (!rope_out || half >= 32);
  auto group_of = [&](int q) {
    if (!rope_out) return n0 + 32 * q;
    const int per = half / 32, b = n0 / 64 + q % (FN / 4 > 0 ? FN / 4 : 1);
    return (b / per) * dh + (b % per) * 32 + (q / (FN / 4 > 0 ? FN / 4 : 1)) * half;
  };
  auto block_of = [&](int b) {
    if (!rope_out) return n0 + 16 * b;
    const int q = n0 / 32 + b % FP, per = half / 16;  // pair block, pair blocks per head
    return (q / per) * dh + (q % per) * 16 + (b / FP) * half;
  };
  // first of this lane's four columns of block b
  auto col_of = [&](int b) {
    const int c = wide ? group_of(b >> 1) + 8 * lq + 4 * (b & 1) : block_of(b) + 4 * lq;
    return c < N ? c : -1;
  };
  // rows past the ends read the last one (their results are never stored)
  const T* xrow[FM];
  const T* wrow[FN];
  const float2* csrow[FM];
#pragma unroll
  for (int a = 0; a < FM; ++a) {
    const int64_t m = m0 + 16 * a + lr < M ? m0 + 16 * a + lr : M - 1;
    xrow[a] = static_cast<const T*>(job.a) + m * K;
    if constexpr (kEnc) csrow[a] = derope ? p.rope + table_row(p, row_position(p, m)) * half : nullptr;
  }
#pragma unroll
  for (int b = 0; b < FN; ++b) {
    const int c = wide ? group_of(b >> 1) + 8 * (lr >> 2) + 4 * (b & 1) + (lr & 3) : block_of(b) + lr;
    wrow[b] = static_cast<const T*>(job.b) + static_cast<int64_t>(c < N ? c : 0) * K;
  }

  struct Step {
    uint4 x[FM][2], w[FN][2];
    float4 cs[kEnc ? FM : 1][kEnc ? VL / 2 : 1];
  };
  // This lane's contraction columns of step i: two blocks, or with deRoPE a block of first halves and
  // their partners.  Both operands take the same columns, so the order does not matter.
  const int hmask = half - 1;  // d_h is a power of two
  auto cols = [&](int i, int& c0, int& c1) {
    const int t = i * KB + VL * lq;
    if (derope) {
      c0 = 2 * (t & ~hmask) + (t & hmask);
      c1 = c0 + half;
    } else {
      c0 = t + i * KB;
      c1 = c0 + KB;
    }
  };
  auto load = [&](int i, Step& s) {
    int c0, c1;
    cols(i, c0, c1);
    // columns past the end read the row's first ones and are replaced by zero when used
    const int d0 = c0 < K ? c0 : 0, d1 = c1 < K ? c1 : 0;
#pragma unroll
    for (int a = 0; a < FM; ++a) {
      s.x[a][0] = *reinterpret_cast<const uint4*>(xrow[a] + d0);
      s.x[a][1] = *reinterpret_cast<const uint4*>(xrow[a] + d1);
      if constexpr (kEnc) {
        if (derope) {
          const float4* cs = reinterpret_cast<const float4*>(csrow[a] + (d0 & hmask));
#pragma unroll
          for (int e = 0; e < VL / 2; ++e) s.cs[a][e] = cs[e];
        }
      }
    }
#pragma unroll
    for (int b = 0; b < FN; ++b) {
      s.w[b][0] = *reinterpret_cast<const uint4*>(wrow[b] + d0);
      s.w[b][1] = *reinterpret_cast<const uint4*>(wrow[b] + d1);
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int i, Step& s) {
    int c[2];
    cols(i, c[0], c[1]);
    if constexpr (kEnc) {
      if (derope || vec_in) {
        float mu[2][VL];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < VL; ++e) mu[h][e] = 0.f;
        if (vec_in) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint4 v = *reinterpret_cast<const uint4*>(static_cast<const T*>(job.vec) +
                                                            (c[h] < K ? c[h] : 0));
            EL::unpack(v, mu[h]);
          }
        }
#pragma unroll
        for (int a = 0; a < FM; ++a) {
          float u[VL], v[VL];
          EL::unpack(s.x[a][0], u);
          EL::unpack(s.x[a][1], v);
          if (derope) {
            const float* cs = reinterpret_cast<const float*>(s.cs[a]);
#pragma unroll
            for (int e = 0; e < VL; ++e) {
              const float uu = u[e], vv = v[e];
              u[e] = uu * cs[2 * e] + vv * cs[2 * e + 1];
              v[e] = vv * cs[2 * e] - uu * cs[2 * e + 1];
            }
          }
#pragma unroll
          for (int e = 0; e < VL; ++e) {
            u[e] -= mu[0][e];
            v[e] -= mu[1][e];
          }
          s.x[a][0] = EL::pack(u);
          s.x[a][1] = EL::pack(v);
        }
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bool ok = c[h] < K;
      const uint4 zero = make_uint4(0, 0, 0, 0);
      uint4 x[FM], w[FN];
#pragma unroll
      for (int a = 0; a < FM; ++a) x[a] = ok ? s.x[a][h] : zero;
#pragma unroll
      for (int b = 0; b < FN; ++b) w[b] = ok ? s.w[b][h] : zero;
      if constexpr (BF16) {
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
          for (int b = 0; b < FN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, w[b]), __builtin_bit_cast(bf16x8, x[a]), acc[a][b], 0, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < VL; ++e)
#pragma unroll
          for (int a = 0; a < FM; ++a)
#pragma unroll
            for (int b = 0; b < FN; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                  __builtin_bit_cast(f32x4, w[b])[e], __builtin_bit_cast(f32x4, x[a])[e], acc[a][b],
                  0, 0, 0);
      }
    }
  };

  // steps wk, wk + WK, ...; each step's operands are loaded during the one before
  const int steps = (K + 2 * KB - 1) / (2 * KB);
  {
    Step s0, s1;
    int i = wk;
    if (i < steps) load(i, s0);
    for (; i < steps; i += 2 * WK) {
      if (i + WK < steps) load(i + WK, s1);
      compute(i, s0);
      if (i + WK >= steps) break;
      if (i + 2 * WK < steps) load(i + 2 * WK, s0);
      compute(i + WK, s1);
    }
  }

  // Lane holds, for blocks (a, b), row 16 a + lane % 16 and columns col_of(b) + (0..3).
  auto finish = [&](int a, const f32x4* y) {
    const int64_t m = m0 + 16 * a + lr;
    if (m >= M) return;
    float f[FN][4];
#pragma unroll
    for (int b = 0; b < FN; ++b) {
      const int c = col_of(b);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f[b][e] = y[b][e];
        if (vec_out && c >= 0) f[b][e] += EL::load1(job.vec, c + e);
      }
    }
    if (rope_out) {
      const float2* cs = p.rope + table_row(p, row_position(p, m)) * half;
#pragma unroll
      for (int b = 0; b < FP; ++b) {
        const int c = col_of(b);
        if (c < 0) continue;
        const float4* q = reinterpret_cast<const float4*>(cs + (c & hmask));
        const float4 q0 = q[0], q1 = q[1];
        const float co[4] = {q0.x, q0.z, q1.x, q1.z}, si[4] = {q0.y, q0.w, q1.y, q1.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float u = f[b][e], v = f[b + FP][e];
          f[b][e] = u * co[e] - v * si[e];
          f[b + FP][e] = v * co[e] + u * si[e];
        }
      }
    }
#pragma unroll
    for (int b = 0; b < FN; ++b) {
      const int c = col_of(b);
      if (c < 0) continue;
      if (silu_out) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[b][e] = f[b][e] / (1.f + expf(-f[b][e]));
      }
      if constexpr (FN == 4) {
        if (wide && (b & 1) == 0) continue;  // stored with the next block's
        if (wide) {
          store8<BF16>(job.c, m * N + c - 4, f[b - (b & 1)], f[b]);
          continue;
        }
      }
      store4<BF16>(job.c, m * N + c, f[b]);
    }
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int a = 0; a < FM; ++a) finish(a, acc[a]);
  } else {
    // the waves' partial sums, added in wave order; wave a finishes row block a
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int b = 0; b < FN; ++b)
        red[((wk * FM + a) * FN + b) * 64 + lane] = __builtin_bit_cast(float4, acc[a][b]);
    __syncthreads();
    if (wk >= FM) return;
    f32x4 y[FN];
#pragma unroll
    for (int b = 0; b < FN; ++b) {
      y[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < WK; ++w)
        y[b] += __builtin_bit_cast(f32x4, red[((w * FM + wk) * FN + b) * 64 + lane]);
    }
    finish(wk, y);
  }
}

__global__ void rope_table_kernel(float2* table, int64_t n, int half, int head_dim,
                                  double theta) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= n) return;
  const int64_t pos = idx / half;
  const int i = static_cast<int>(idx % half);
  const double omega = pow(theta, -2.0 * static_cast<double>(i) / static_cast<double>(head_dim));
  const double a = static_cast<double>(pos) * omega;
  double s, c;
  sincos(a, &s, &c);
  table[idx] = make_float2(static_cast<float>(c), static_cast<float>(s));
}

__global__ void positions_kernel(int32_t* out, int64_t n_tokens, int32_t n_seqs,
                                 const int32_t* cu, const int32_t* pos0) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n_tokens) return;
  int b = 0;
  int64_t local = t;
  if (cu != nullptr) {
    int lo = 0, hi = n_seqs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cu[mid] <= t) lo = mid; else hi = mid - 1;
    }
    b = lo;
    local = t - cu[b];
  }
  out[t] = static_cast<int32_t>(local + (pos0 != nullptr ? pos0[b] : 0));
}

}  // namespace

// Short contractions (the decode, thin head-shared encodes) are a load, a few MFMAs and a store per
// wave: 32 x 32 waves, more of them in flight (bf16 decode of 64-wide heads' shared basis, 8192 tokens
// x 14 layers: 254 us, 310 us as 32 x 64).  Longer ones take 32 x 64 waves, four to a workgroup once
// they give every SIMD one; below that the contraction is split so that the chip still has waves to
// run.  fp32, us on 128x64 / 32x64 split by 4 / 32x32 split by 8: encode of 4099 tokens x 8 layers
// (w = 512, 64 codes) 122 / 93 / 141; encode and Patch of 512 tokens x 4 layers 90 / 36 / 24; codec of
// 12,000 tokens x 24 layers 2140 / 3700 / 5400 (128 x 128 tiles through LDS took 3490).
GenericShape generic_shape(const GemmJob* jobs, size_t n_jobs, int64_t m) {
  int64_t waves = 0;  // of 32 x 64 outputs
  int k = 0;
  for (size_t i = 0; i < n_jobs; ++i) {
    waves += (m + 31) / 32 * ((jobs[i].n + 63) / 64);
    k = jobs[i].k > k ? jobs[i].k : k;
  }
  if (k <= 128) return GenericShape::k128x32;
  if (waves >= 1024) return GenericShape::k128x64;
  return waves >= 256 ? GenericShape::k32x64 : GenericShape::k32x32;
}

int generic_rows(GenericShape s) {
  constexpr int rows[] = {128, 128, 32, 32};
  return rows[static_cast<int>(s)];
}

int generic_cols(GenericShape s) {
  constexpr int cols[] = {64, 32, 64, 32};
  return cols[static_cast<int>(s)];
}

template <typename OP, bool BF16, int FM, int FN, int WM, int WK>
hipError_t launch_one(const GemmParams& p, hipStream_t stream) {
  const size_t lds = WK > 1 ? static_cast<size_t>(WK) * FM * FN * 64 * sizeof(float4) : 0;
  hipLaunchKernelGGL((gemm_nt_kernel<OP, BF16, FM, FN, WM, WK>), dim3(p.total_tiles),
                     dim3(64 * WM * WK), lds, stream, p);
  return hipGetLastError();
}

template <typename OP, bool BF16>
hipError_t launch_shape(GenericShape shape, const GemmParams& p, hipStream_t stream) {
  switch (shape) {
    case GenericShape::k128x64: return launch_one<OP, BF16, 2, 4, 4, 1>(p, stream);
    case GenericShape::k128x32: return launch_one<OP, BF16, 2, 2, 4, 1>(p, stream);
    case GenericShape::k32x64: return launch_one<OP, BF16, 2, 4, 1, 4>(p, stream);
    case GenericShape::k32x32: return launch_one<OP, BF16, 2, 2, 1, 8>(p, stream);
  }
  return hipErrorInvalidValue;
}

template <typename OP>
hipError_t launch_op(bool bf16, GenericShape shape, const GemmParams& p, hipStream_t stream) {
  return bf16 ? launch_shape<OP, true>(shape, p, stream) : launch_shape<OP, false>(shape, p, stream);
}

hipError_t launch_gemm(Op op, bool bf16, GenericShape shape, const GemmParams& p,
                       hipStream_t stream) {
  if (p.total_tiles <= 0) return hipSuccess;
  switch (op) {
    case Op::kReuseDecode: return launch_op<ReuseDecode>(bf16, shape, p, stream);
    case Op::kPatchKV: return launch_op<PatchKV>(bf16, shape, p, stream);
    case Op::kEncodeKV: return launch_op<EncodeKV>(bf16, shape, p, stream);
    case Op::kEncodeH: return launch_op<EncodeH>(bf16, shape, p, stream);
    case Op::kPatchAlign: return launch_op<PatchAlign>(bf16, shape, p, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_rope_table(float2* table, int64_t max_pos, int head_dim, double theta,
                             hipStream_t stream) {
  const int half = head_dim / 2;
  const int64_t n = max_pos * half;
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(rope_table_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream,
                     table, n, half, head_dim, theta);
  return hipGetLastError();
}

hipError_t launch_positions(int32_t* out, int64_t n_tokens, int32_t n_seqs,
                            const int32_t* cu_seqlens, const int32_t* pos0, hipStream_t stream) {
  if (n_tokens <= 0) return hipSuccess;
  const int64_t blocks = (n_tokens + 255) / 256;
  hipLaunchKernelGGL(positions_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream,
                     out, n_tokens, n_seqs, cu_seqlens, pos0);
  return hipGetLastError();
}

}  // namespace scd
