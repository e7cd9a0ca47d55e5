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
// outputs of one row per block, and eight over two blocks, which it stores as one vector.  A lane holds 16
// bytes of a row per block, so a load covers 16 rows x 64 bytes.  When the input needs deRoPE a step's two
// blocks are columns i and i + d_h/2 of one head; when the output is rotated a wave's column blocks are
// heads' first halves and their partners: every RoPE pair meets in one lane's registers.
//
// The shape follows the launch (generic_shape): four waves along the rows when there are enough of
// them to fill the chip; else one tile per workgroup whose waves split the contraction (their sums meet
// in LDS, added in wave order), so that short prefixes and thin codes do not wait on one wave's chain
// of loads.  fp32 is bound by the MFMA rate (32 cycles per 16 x 16 x 4), small launches by latency:
// the smallest model's codec (512 tokens, 4 layers) takes 32 us in four launches; on 128 x 128 tiles
// through LDS it took 193 us, three quarters of each 32-code tile computed for nothing.  Where tiles fill
// 128 x 128 and there are many of them, the bf16 decode and Patch run on such tiles all the same
// (gemm_staged_bf16_kernel).
#include <type_traits>

#include "scd_kernels.h"

namespace scd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kNumXcd = 8;
constexpr int kStagedTile = 128;  // rows and columns of a staged tile

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
  __device__ static inline float4 load4(const void* p, int64_t i) {  // i % 4 == 0
    const uint2 v = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(p) + i);
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                       __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
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
  __device__ static inline float4 load4(const void* p, int64_t i) {
    return *reinterpret_cast<const float4*>(static_cast<const float*>(p) + i);
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
  // of a 32-column group, so that a bf16 store is 16 bytes.  When the output is rotated a group counts
  // columns of heads' first halves (u, a head's half is a multiple of 8) and the groups past FN / 4 are
  // their partners; two blocks then are one 16-column block and its partner instead (first column:
  // block_of).  -1: past the last column.
  constexpr int FG = FN / 4 > 0 ? FN / 4 : 1;  // groups of first halves
  const bool wide = FN == 4 || !rope_out;
  const int hm = half - 1;
  auto group_col = [&](int q, int o) {
    if (!rope_out) return n0 + 32 * q + o;
    const int u = n0 / 2 + 32 * (q % FG) + o;
    return 2 * (u & ~hm) + (u & hm) + (q / FG) * half;
  };
  auto block_of = [&](int b) {
    const int q = n0 / 32 + b % FP, per = half / 16;  // pair block, pair blocks per head
    return (q / per) * dh + (q % per) * 16 + (b / FP) * half;
  };
  // first of this lane's four columns of block b
  auto col_of = [&](int b) {
    const int c = wide ? group_col(b >> 1, 8 * lq + 4 * (b & 1)) : block_of(b) + 4 * lq;
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
    const int c = wide ? group_col(b >> 1, 8 * (lr >> 2) + 4 * (b & 1) + (lr & 3)) : block_of(b) + lr;
    wrow[b] = static_cast<const T*>(job.b) + static_cast<int64_t>(c < N ? c : 0) * K;
  }

  struct Step {
    uint4 x[FM][2], w[FN][2];
  };
  // Rotation factors: loaded with the step's operands, or, where a second set is too many registers (51 of
  // them spilled), once the step before has used its own.
  constexpr bool kOneCs = BF16 && FN == 4 && WK > 1;
  struct Factors {
    float4 v[kEnc ? FM : 1][kEnc ? VL / 2 : 1];
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
  // steps wk, wk + WK, ...; each step's operands are loaded during the one before
  const int steps = (K + 2 * KB - 1) / (2 * KB);
  auto load = [&](int i, Step& s) {
    int c0, c1;
    cols(i, c0, c1);
    // columns past the end read the row's first ones and are replaced by zero when used
    const int d0 = c0 < K ? c0 : 0, d1 = c1 < K ? c1 : 0;
#pragma unroll
    for (int a = 0; a < FM; ++a) {
      s.x[a][0] = *reinterpret_cast<const uint4*>(xrow[a] + d0);
      s.x[a][1] = *reinterpret_cast<const uint4*>(xrow[a] + d1);
    }
#pragma unroll
    for (int b = 0; b < FN; ++b) {
      s.w[b][0] = *reinterpret_cast<const uint4*>(wrow[b] + d0);
      s.w[b][1] = *reinterpret_cast<const uint4*>(wrow[b] + d1);
    }
  };

  auto load_cs = [&](int i, Factors& cs) {
    if constexpr (kEnc) {
      if (derope && i < steps) {
        int c0, c1;
        cols(i, c0, c1);
#pragma unroll
        for (int a = 0; a < FM; ++a) {
          const float4* q = reinterpret_cast<const float4*>(csrow[a] + ((c0 < K ? c0 : 0) & hmask));
#pragma unroll
          for (int e = 0; e < VL / 2; ++e) cs.v[a][e] = q[e];
        }
      }
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int i, Step& s, Factors& cs) {
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
            const float* f = reinterpret_cast<const float*>(cs.v[a]);
#pragma unroll
            for (int e = 0; e < VL; ++e) {
              const float uu = u[e], vv = v[e];
              u[e] = uu * f[2 * e] + vv * f[2 * e + 1];
              v[e] = vv * f[2 * e] - uu * f[2 * e + 1];
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
        if constexpr (kOneCs) load_cs(i + WK, cs);
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

  {
    Step s0, s1;
    Factors f0, f1;
    Factors& g1 = kOneCs ? f0 : f1;
    auto ahead = [&](int i, Step& st, Factors& cs) {
      if (i >= steps) return;
      load(i, st);
      if constexpr (!kOneCs) load_cs(i, cs);
    };
    int i = wk;
    ahead(i, s0, f0);
    if constexpr (kOneCs) load_cs(i, f0);
    for (; i < steps; i += 2 * WK) {
      ahead(i + WK, s1, g1);
      compute(i, s0, f0);
      if (i + WK >= steps) break;
      ahead(i + 2 * WK, s0, f0);
      compute(i + WK, s1, g1);
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
      const float4 v = vec_out && c >= 0 ? EL::load4(job.vec, c) : make_float4(0.f, 0.f, 0.f, 0.f);
      f[b][0] = y[b][0] + v.x;
      f[b][1] = y[b][1] + v.y;
      f[b][2] = y[b][2] + v.z;
      f[b][3] = y[b][3] + v.w;
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
          f[b][e] = fmaf(-v, si[e], u * co[e]);  // as the staged kernel rounds
          f[b + FP][e] = fmaf(u, si[e], v * co[e]);
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
      if (wide) {
        if ((b & 1) == 1) store8<BF16>(job.c, m * N + c - 4, f[b - 1], f[b]);
        continue;
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

// The bf16 Reuse decode and Patch of all but small launches, staged through LDS: 256 threads (2 x 2 waves)
// compute a 128 x 128 tile of C, the contraction 32 at a time through double-buffered LDS, and the sums go
// through LDS too, so that a store instruction writes 256 contiguous bytes of 4 rows.  The decode is bound
// by its writes, for which the direct kernel's 64 bytes of 16 rows are too scattered, the Patch by its
// operands' way into the CU, of which a 128 x 128 tile takes a third of a 32 x 64 wave's per product.
// Decode of more than 256 requests, w = 1024, rank 128, 8192 tokens x 4 layers 82 us (198 direct); heads of
// 32, w = 512, rank 64, 8192 tokens x 8 layers 64 us (118 direct); Patch with heads of 32, d_model 2048, 512
// channels, 8192 tokens x 4 layers 207 us (685 direct).
template <typename OP>
__global__ __launch_bounds__(256) void gemm_staged_bf16_kernel(GemmParams p) {
  using EL = Elem<true>;
  constexpr int BM = kStagedTile, BN = kStagedTile, BK = 32, NT = 256;
  constexpr int LDK = BK + 8;  // LDS row, padded by 16 bytes
  constexpr int WT = 64, F = WT / 16;
  constexpr int LDC = BN + 4;
  constexpr int TP = BM * BK / 8 / NT;  // 16-byte pieces of an operand per thread and step
  constexpr size_t kAB = 2u * (BM + BN) * LDK * sizeof(uint16_t);
  constexpr size_t kC = static_cast<size_t>(BM) * LDC * sizeof(float);
  __shared__ __attribute__((aligned(16))) unsigned char smem[kAB > kC ? kAB : kC];
  __shared__ int s_pos[BM];
  uint16_t* As = reinterpret_cast<uint16_t*>(smem);  // [2][BM][LDK]
  uint16_t* Bs = As + 2 * BM * LDK;
  float* Cs = reinterpret_cast<float*>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  int j = 0;
  while (j + 1 < p.n_jobs && bid >= p.jobs[j + 1].tile_begin) ++j;
  const GemmJob job = p.jobs[j];
  const int local = bid - job.tile_begin;
  const int K = job.k, N = job.n;
  const int64_t M = p.m;
  const int ntn = (N + BN - 1) / BN;
  const int64_t m0 = static_cast<int64_t>(local / ntn) * BM;
  const int n0 = (local % ntn) * BN;
  const bool rope_out = (job.flags & kRopeOut) != 0;
  const bool vec_out = (job.flags & kVecOut) != 0 && job.vec != nullptr;
  const int dh = p.head_dim, half = dh / 2;
  const uint16_t* A = static_cast<const uint16_t*>(job.a);
  const uint16_t* B = static_cast<const uint16_t*>(job.b);
  if (rope_out)
    for (int r = tid; r < BM; r += NT) s_pos[r] = static_cast<int>(row_position(p, m0 + r));

  // step kc's pieces of this thread; pieces out of range read an in-bounds address and become zero
  uint4 ra[TP], rb[TP];
  auto gload = [&](int kc) {
#pragma unroll
    for (int t = 0; t < TP; ++t) {
      const int task = tid + t * NT, row = task / (BK / 8), col = kc * BK + 8 * (task % (BK / 8));
      const uint4 zero = make_uint4(0, 0, 0, 0);
      const int64_t gr = m0 + row;
      const int gn = n0 + row;
      const bool oka = gr < M && col < K, okb = gn < N && col < K;
      ra[t] = *reinterpret_cast<const uint4*>(A + (oka ? gr * K + col : 0));
      rb[t] = *reinterpret_cast<const uint4*>(B + (okb ? static_cast<int64_t>(gn) * K + col : 0));
      if (!oka) ra[t] = zero;
      if (!okb) rb[t] = zero;
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int t = 0; t < TP; ++t) {
      const int task = tid + t * NT, row = task / (BK / 8), q = task % (BK / 8);
      *reinterpret_cast<uint4*>(As + (buf * BM + row) * LDK + 8 * q) = ra[t];
      *reinterpret_cast<uint4*>(Bs + (buf * BN + row) * LDK + 8 * q) = rb[t];
    }
  };
  f32x4 acc[F][F];
#pragma unroll
  for (int a = 0; a < F; ++a)
#pragma unroll
    for (int b = 0; b < F; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int lr = lane & 15, lk = (lane >> 4) * 8;
  const int nk = (K + BK - 1) / BK;
  gload(0);
  sstore(0);
  __syncthreads();
  for (int kc = 0; kc < nk; ++kc) {
    const int cur = kc & 1;
    if (kc + 1 < nk) gload(kc + 1);
    bf16x8 af[F], bfr[F];
#pragma unroll
    for (int a = 0; a < F; ++a)
      af[a] = *reinterpret_cast<const bf16x8*>(As + (cur * BM + wm * WT + a * 16 + lr) * LDK + lk);
#pragma unroll
    for (int b = 0; b < F; ++b)
      bfr[b] = *reinterpret_cast<const bf16x8*>(Bs + (cur * BN + wn * WT + b * 16 + lr) * LDK + lk);
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
      for (int b = 0; b < F; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
    if (kc + 1 < nk) sstore(cur ^ 1);
    __syncthreads();
  }
  // sums -> LDS: a lane holds column lane % 16 and rows 4 (lane / 16) + e of a block
#pragma unroll
  for (int a = 0; a < F; ++a)
#pragma unroll
    for (int b = 0; b < F; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        Cs[(wm * WT + a * 16 + 4 * (lane >> 4) + e) * LDC + wn * WT + b * 16 + lr] = acc[a][b][e];
  __syncthreads();

  // eight columns of row `row` from tile column c, offset added
  auto take8 = [&](int row, int c, float* u) {
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (vec_out) EL::unpack(*reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(job.vec) + n0 + c), v);
    const float4* s = reinterpret_cast<const float4*>(Cs + row * LDC + c);
    const float4 x = s[0], y = s[1];
    const float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) u[e] = f[e] + v[e];
  };
  uint16_t* C = static_cast<uint16_t*>(job.c);
  if (rope_out) {
    const int gph = dh / 16;      // 8-wide groups in half a head
    constexpr int GPR = BN / 16;  // pair groups per tile row
    for (int task = tid; task < BM * GPR; task += NT) {
      const int row = task / GPR, cg = task % GPR;
      const int o = (cg % gph) * 8;
      const int c0 = (cg / gph) * dh + o, c1 = c0 + half;
      const int64_t gm = m0 + row;
      if (gm >= M || n0 + c0 >= N) continue;
      float u[8], v[8];
      take8(row, c0, u);
      take8(row, c1, v);
      const float2* cs = p.rope + table_row(p, s_pos[row]) * half + o;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float2 f = cs[e];
        const float x = u[e], y = v[e];
        u[e] = fmaf(-y, f.y, x * f.x);  // as the direct kernel rounds
        v[e] = fmaf(x, f.y, y * f.x);
      }
      *reinterpret_cast<uint4*>(C + gm * N + n0 + c0) = EL::pack(u);
      *reinterpret_cast<uint4*>(C + gm * N + n0 + c1) = EL::pack(v);
    }
  } else {
    constexpr int GPR = BN / 8;
    for (int task = tid; task < BM * GPR; task += NT) {
      const int row = task / GPR, c = (task % GPR) * 8;
      const int64_t gm = m0 + row;
      if (gm >= M || n0 + c >= N) continue;
      float u[8];
      take8(row, c, u);
      *reinterpret_cast<uint4*>(C + gm * N + n0 + c) = EL::pack(u);
    }
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

// One launch's workgroups, by what a CU has to do (figures: us).
// bf16 outputs wider than a 64-column tile are staged through LDS: decodes from 128 tiles of 128 x 128 on
// (128x64 / 128x32 / staged: w = 512, rank 32, 8 layers, 64 tokens, 64 tiles, 9.0 / 8.4 / 8.1, 200 tokens 9.3
// / 9.3 / 9.5, 500 tokens 10.7 / 11.6 / 10.2, 1000 tokens 18 / 19 / 12; w = 1024, rank 256, 4 layers, 64
// tokens, 64 tiles, 128x32 9.3, staged 10.4), the longer contractions of the Patch above 1024 tiles of
// 32 x 64, four a CU (split by 4 / staged: d_model 4128, 1024 channels, 4 layers, 200 tokens, 896 tiles, 67 /
// 102, 333 tokens, 1408 tiles, 98 / 102, 500 tokens 130 / 98; d_model 4096, 192 channels, 1000 tokens, 768
// tiles, 70 / 90, 1400 tokens, 1056 tiles, 112 / 91).
// Other contractions up to 128 are a load, a few MFMAs and a store per wave: 32 x 64 waves from 1536 of
// them on where the outputs fill them (128x64 / 128x32: fp32 w = 1024, rank 128, 16 layers, 200 tokens 45 / 43, 500 tokens 74 / 80, 8192
// tokens 966 / 1109; bf16 w = 64, rank 64, 16 heads x 4 layers, 8192 tokens 145 / 173, staged 136; with 32
// heads x 14 layers 943 / 1121, staged 1006; heads' shared rows of 32, 32 heads x 6 layers, 8192 tokens 251 /
// 195), 32 x 32 waves below.
// Decodes take those at every rank: the shapes that do not split the contraction add every sum in the same
// order, so a decode's bits do not depend on the layers it shares a launch with (the streamed receipt's groups).
// Longer ones take four 32 x 64 waves along the rows, or one such tile per workgroup whose waves split the
// contraction, or 32 x 32 tiles split by 8 below one 32 x 64 tile per CU (256 tokens of a d_model of 512 to
// 4096: a half to a third of the time).  The first two differ by the last round: a CU's share is whole
// workgroups, of four 32 x 64 tiles or of one, and one workgroup of the first kind alone hides less
// latency, while the split costs a sixth more per tile, in the bf16 key and value encode (deRoPE for every
// lane of four waves) almost half.  In units of a 32 x 64 tile a CU: 4 ceil(tiles / 1024) + 1 against
// 1.16 (1.45) ceil(tiles / 256) + 0.3.  128x64 / split by 4: fp32 K/V encode at w = 512, rank 64, 8 layers,
// 1000 tokens 48 / 26, 2000 tokens 49 / 45, 4099 tokens 102 / 86, 8192 tokens 148 / 161; code H of d_model
// 2048, rank 128, 4 layers, 4099 tokens 184 / 124, 8192 tokens 193 / 197; Patch of d_model 1024, 512
// channels, 2 layers, 4099 tokens 231 / 212, 8192 tokens 370 / 393; bf16 K/V encode of heads of 32, w = 1024,
// rank 128, 8 layers, 500 tokens 56 / 30, 2000 tokens 72 / 91, 4099 tokens 164 / 183.
GenericShape generic_shape(Op op, bool bf16, const GemmJob* jobs, size_t n_jobs, int64_t m) {
  int64_t tiles = 0, staged = 0;  // 32 x 64 and 128 x 128 tiles
  int k = 0, n = 0;
  for (size_t i = 0; i < n_jobs; ++i) {
    tiles += (m + 31) / 32 * ((jobs[i].n + 63) / 64);
    staged += (m + kStagedTile - 1) / kStagedTile * ((jobs[i].n + kStagedTile - 1) / kStagedTile);
    k = jobs[i].k > k ? jobs[i].k : k;
    n = jobs[i].n > n ? jobs[i].n : n;
  }
  if (bf16 && n > 64 &&
      ((op == Op::kReuseDecode && staged >= 128) || (op == Op::kPatchKV && tiles > 1024)))
    return GenericShape::kStaged;
  if (k <= 128 || op == Op::kReuseDecode)
    return n > 32 && tiles >= 1536 ? GenericShape::k128x64 : GenericShape::k128x32;
  if (tiles < 256) return GenericShape::k32x32;
  const int64_t rows4 = 4 * ((tiles + 1023) / 1024) + 1, split = (tiles + 255) / 256;
  const double cost = bf16 && op == Op::kEncodeKV ? 1.45 : 1.16;
  return static_cast<double>(rows4) <= cost * static_cast<double>(split) + 0.3 ? GenericShape::k128x64
                                                                                 : GenericShape::k32x64;
}

int generic_rows(GenericShape s) {
  constexpr int rows[] = {128, 128, 32, 32, kStagedTile};
  return rows[static_cast<int>(s)];
}

int generic_cols(GenericShape s) {
  constexpr int cols[] = {64, 32, 64, 32, kStagedTile};
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
    case GenericShape::kStaged: break;
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
  if (shape == GenericShape::kStaged) {
    if ((op != Op::kReuseDecode && op != Op::kPatchKV) || !bf16) return hipErrorInvalidValue;
    if (op == Op::kReuseDecode)
      hipLaunchKernelGGL(gemm_staged_bf16_kernel<ReuseDecode>, dim3(p.total_tiles), dim3(256), 0, stream, p);
    else
      hipLaunchKernelGGL(gemm_staged_bf16_kernel<PatchKV>, dim3(p.total_tiles), dim3(256), 0, stream, p);
    return hipGetLastError();
  }
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
