// Offline Reuse fit of the SCD codec (Section 4.3.1 "Joint Subspace Learning"; Appendix F.1
// "Reuse: Layer-wise Stack-SVD with Ridge Regression").
//
// For one branch (keys or values) of every Reuse layer, the producer's and the consumer's caches of
// the same calibration prefixes give rows A, B [N, w] (keys de-rotated first).  The fit needs only
// the joint Gram G = X^T X of X = [A B] (2w x 2w) and the column sums 1^T X:
//   * the truncated SVD of the (centred) X is the eigendecomposition of the (centred) G, whose top-r
//     eigenvectors V_r give the latents Z = X V_r;
//   * the ridge encoder E = (A^T A + lam I)^-1 A^T Z needs A^T A and A^T Z = G[0:w, :] V_r;
//   * the ridge decoder F = (Z^T Z + lam I)^-1 Z^T B needs Z^T Z = V_r^T G V_r and
//     Z^T B = (G[w:2w, :] V_r)^T.
// The O(N w^2) part (the Gram) streams the caches once on the matrix cores; the O(w^3) part runs in
// fp64 as a sequence of launches over all layers at once (Householder tridiagonalisation,
// bisection and inverse iteration for the top r eigenpairs, Cholesky solves).
#include "scd_device.h"

#include <mutex>

namespace scd {

using namespace dev;

// Device-resident scratch of the allocation-free solve (scd_fit_solve_noalloc): the solve's fp64
// matrices for as many layers as fit, reused launch after launch.  Each GPU the
// library runs on holds its own copy for the life of the process.  Host code must never pass this
// name to a kernel (in host code it is a stand-in, not a device address): fit_scratch() looks up
// the device address once per device.
static __device__ __align__(256) double scratch[kFitScratchBytes / sizeof(double)];

namespace {

constexpr int kTB = kFitTile;
constexpr int kTileFloats = kTB * kTB + kTB;  // one partial tile: Gram block + column sums

__device__ inline int fit_position(const FitGramParams& p, int64_t row) {
  const int64_t t = row / p.g;
  int b = 0;
  int64_t local = t;
  if (p.cu_seqlens != nullptr) {
    int lo = 0, hi = p.n_seqs - 1;  // largest b with cu[b] <= t
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (p.cu_seqlens[mid] <= t) lo = mid; else hi = mid - 1;
    }
    b = lo;
    local = t - p.cu_seqlens[b];
  }
  int64_t pos = local + (p.pos0 != nullptr ? p.pos0[b] : 0);
  pos = pos < 0 ? 0 : (pos >= p.max_pos ? p.max_pos - 1 : pos);
  return static_cast<int>(pos);
}

// Upper tiles (ti <= tj) of the nt x nt tile grid, numbered row by row.
__device__ inline void tile_of(int tile, int nt, int& ti, int& tj) {
  int rem = tile;
  ti = 0;
  while (rem >= nt - ti) {
    rem -= nt - ti;
    ++ti;
  }
  tj = ti + rem;
}

// First column (inside a 128-column block) of chunk pair cp: VEC columns of one head's first half;
// their RoPE partners sit d_h/2 further on.  A block holds 128 / d_h heads of d_h / (2 VEC) pairs.
template <int DH, int VEC>
__device__ inline int pair_col(int cp) {
  constexpr int PER_HEAD = DH / 2 / VEC;
  return (cp / PER_HEAD) * DH + (cp % PER_HEAD) * VEC;
}

// Loads through the global address space.  The row pointers come out of the job table through a
// select between two sources, which hides their address space from the compiler; as generic (flat)
// loads they would also count against the LDS counter, so every LDS wait would drain them.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 g_u32x4;
typedef __attribute__((address_space(1))) const f32x4 g_f32x4;
__device__ inline uint4 gload16(const char* p) {
  const u32x4 v = *(g_u32x4*)(p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ inline float4 gload_f4(const float2* p) {
  const f32x4 v = *(g_f32x4*)(p);
  return make_float4(v.x, v.y, v.z, v.w);
}

// Column sums of a staged dword (two bf16 values of one column): acc + lo + hi in one dot product.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ inline float add_bf16_pair(uint32_t v, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, v),
                                         __builtin_bit_cast(bf16x2_t, 0x3f803f80u), acc, false);
}

struct BlockSrc {
  const char* base;  // producer or consumer cache
  int col;           // column inside the w-wide row
};

// Source of the chunk pair starting at joint column jc (< 2w): columns [0, w) are the producer's,
// [w, 2w) the consumer's.  A head never straddles the two (w is a multiple of d_h).
__device__ inline BlockSrc block_src(const FitGramJob& j, int w, int jc, int eb) {
  BlockSrc s;
  s.base = static_cast<const char*>(jc < w ? j.a : j.b);
  s.col = (jc < w ? jc : jc - w) * eb;
  return s;
}

// ---------------------------------------------------------------------------------------------
// bf16 Gram: one workgroup of 4 waves per (job, upper 128 x 128 tile, row slice).  Each k-step
// stages 64 rows of the tile's two column blocks transposed in LDS ([column][row], so an MFMA
// operand fragment is 8 consecutive rows of one column) and runs v_mfma_f32_32x32x16_bf16 with the
// I block as A and the J block as B: C[m][n] = sum_rows X[row][I0+m] X[row][J0+n].  Keys are
// de-rotated in registers and rounded to bf16 once before the product (as the encoder does).
// Thread t stages row pair t % 32 and chunk pair t / 32 (8 columns + their RoPE partners).
//
// The step is bound by HBM latency, so rows travel two k-steps ahead in two register sets and the
// RoPE factors one step ahead; each is issued before the far data prefetch, so the in-order
// vector-memory counter never makes a step wait for rows it does not use yet.  The LDS tiles are
// double-buffered, which leaves one barrier per step, and that barrier waits for LDS only.
// PAIR: both rows of a thread's pair belong to one token (g even), so they share RoPE factors.
// ---------------------------------------------------------------------------------------------
//
// FULL (2w = 256 only): one workgroup owns the whole Gram of its (job, slice), so every row is read
// once.  Its two column blocks are the producer's (A) and the consumer's (B) columns; each wave
// computes one 128 x 128 tile (AA, AB, BB, and the mirror BA, which keeps the code uniform and is
// not stored), so a 64-row step is 64 MFMAs per wave against 32 KB of rows: about HBM speed.  The
// partial tiles keep the tile kernel's layout (AA, AB, BB), so the slice reduction is shared.
template <int DH, bool DEROPE, bool PAIR, bool FULL>
__device__ __forceinline__ void fit_gram_bf16_body(const FitGramParams& p) {
  constexpr int BK = kFitRowStep, S = BK + 8, HALF = DH / 2, NR = PAIR ? 1 : 2;
  constexpr int NA = FULL ? 4 : 2;  // accumulator blocks per wave and dimension
  __shared__ __attribute__((aligned(16))) uint16_t xt[2][2][kTB * S];  // [stage][block]

  const int nt = 2 * p.w / kTB, n_upper = nt * (nt + 1) / 2;
  // the tiles of one (job, slice) read the same rows: consecutive units on one XCD, so the second
  // read of a column block hits that XCD's L2
  int unit = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = FULL ? 0 : unit % n_upper;
  if (!FULL) unit /= n_upper;
  const int slice = unit % p.n_slices;
  const int job = unit / p.n_slices;
  int ti = 0, tj = 1;
  if (!FULL) tile_of(tile, nt, ti, tj);
  const bool diag = ti == tj;
  const int nblk = diag ? 1 : 2;
  const FitGramJob& jb = p.jobs[job];
  const int64_t r0 = static_cast<int64_t>(slice) * p.slice_rows;
  const int64_t r1 = r0 + p.slice_rows < p.n_rows ? r0 + p.slice_rows : p.n_rows;
  const int64_t row_bytes = static_cast<int64_t>(p.w) * 2;
  const int tj_src = diag ? ti : tj;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // eight consecutive lanes cover the eight chunk pairs of one row pair: a load instruction reads
  // 8 rows x 128 contiguous bytes
  const int cp = tid & 7, rp = tid >> 3;
  const int c = pair_col<DH, 8>(cp);
  const int ri = c % DH;  // RoPE pair index of the first column (< d_h / 2)
  BlockSrc src[2];
  src[0] = block_src(jb, p.w, ti * kTB + c, 2);
  src[1] = block_src(jb, p.w, tj_src * kTB + c, 2);

  uint4 la[2][2][2], lb[2][2][2];  // [block][row of the pair][first half / partner]
  float4 rc[NR][4];                // RoPE (cos, sin) of the next step's rows, pairs ri .. ri+7
  constexpr int NCS = FULL ? 32 : 16;  // column sums kept: one or both blocks
  float csum[NCS];
#pragma unroll
  for (int i = 0; i < NCS; ++i) csum[i] = 0.f;
  f32x16 acc[NA][NA];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  const uint4 zero4 = make_uint4(0, 0, 0, 0);
  // Every step issues the same loads on every path (rows past the slice read its last row and are
  // zeroed when staged; a diagonal tile's J block re-reads its I block from L1/L2), so the
  // compiler's counter waits can leave the far prefetch in flight.
  auto issue_rows = [&](uint4 (&ld)[2][2][2], int64_t k0) {
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
      int64_t n = k0 + 2 * rp + rr;
      n = n < r1 ? n : r1 - 1;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const char* rowp = src[b].base + n * row_bytes + src[b].col;
        ld[b][rr][0] = gload16(rowp);
        ld[b][rr][1] = gload16(rowp + HALF * 2);
      }
    }
  };
  auto issue_rope = [&](int64_t k0) {
    if constexpr (DEROPE) {
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int64_t n = k0 + 2 * rp + q;
        const float2* tab = p.rope + static_cast<int64_t>(n < r1 ? fit_position(p, n) : 0) * HALF + ri;
#pragma unroll
        for (int j = 0; j < 4; ++j) rc[q][j] = gload_f4(tab + 2 * j);
      }
    }
  };
  // de-rotate (keys), round, and write one k-step's rows into LDS stage sb; accumulate the diagonal
  // tile's column sums
  auto stage = [&](const uint4 (&ld)[2][2][2], int64_t k0, int sb) {
    if constexpr (!DEROPE) {
      // values: the staged dword of column j is the j-th bf16 of row 2rp (low half) and of row
      // 2rp + 1 (high half): one byte permute per dword, no conversions
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        if (b >= nblk) break;
        uint32_t* dst = reinterpret_cast<uint32_t*>(xt[sb][b]);
        const bool live0 = k0 + 2 * rp < r1, live1 = k0 + 2 * rp + 1 < r1;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint4 a0 = live0 ? ld[b][0][q] : zero4, a1 = live1 ? ld[b][1][q] : zero4;
          const uint32_t w0[4] = {a0.x, a0.y, a0.z, a0.w}, w1[4] = {a1.x, a1.y, a1.z, a1.w};
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const uint32_t v = __builtin_amdgcn_perm(w1[j >> 1], w0[j >> 1],
                                                     (j & 1) ? 0x07060302u : 0x05040100u);
            if (FULL) csum[16 * b + 8 * q + j] = add_bf16_pair(v, csum[16 * b + 8 * q + j]);
            else if (b == 0 && diag) csum[8 * q + j] = add_bf16_pair(v, csum[8 * q + j]);
            const int col = c + q * HALF + j;
            dst[col * (S / 2) + ((((rp >> 2) ^ (col >> 3)) & 7) << 2) + (rp & 3)] = v;
          }
        }
      }
      return;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (b >= nblk) break;
      float f[2][2][8];
#pragma unroll
      for (int rr = 0; rr < 2; ++rr) {
        const bool live = k0 + 2 * rp + rr < r1;
        unpack8(live ? ld[b][rr][0] : zero4, f[rr][0]);
        unpack8(live ? ld[b][rr][1] : zero4, f[rr][1]);
        if constexpr (DEROPE) {
          const int q = PAIR ? 0 : rr;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float4 cs = rc[q][j];
            const float u0 = f[rr][0][2 * j], v0 = f[rr][1][2 * j];
            const float u1 = f[rr][0][2 * j + 1], v1 = f[rr][1][2 * j + 1];
            // inverse rotation by the position's angle
            f[rr][0][2 * j] = u0 * cs.x + v0 * cs.y;
            f[rr][1][2 * j] = v0 * cs.x - u0 * cs.y;
            f[rr][0][2 * j + 1] = u1 * cs.z + v1 * cs.w;
            f[rr][1][2 * j + 1] = v1 * cs.z - u1 * cs.w;
          }
        }
      }
      uint32_t* dst = reinterpret_cast<uint32_t*>(xt[sb][b]);
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t v = pack_bf16x2(f[0][q][j], f[1][q][j]);  // rows 2rp (low), 2rp+1 (high)
          if (FULL) csum[16 * b + 8 * q + j] = add_bf16_pair(v, csum[16 * b + 8 * q + j]);
          else if (b == 0 && diag) csum[8 * q + j] = add_bf16_pair(v, csum[8 * q + j]);
          const int col = c + q * HALF + j;
          dst[col * (S / 2) + ((((rp >> 2) ^ (col >> 3)) & 7) << 2) + (rp & 3)] = v;
        }
    }
  };

  const int wy = wave >> 1, wx = wave & 1;
  const int h = lane >> 5;
  // LDS tile layout: row group kg (8 rows) of column col sits at slot kg ^ ((col >> 3) & 7) of the
  // column's padded row, so neither the transposed writes nor the fragment reads conflict
  const int jblk = diag ? 0 : 1;
  auto frag = [&](const uint16_t* base, int col, int kg) {
    return *reinterpret_cast<const bf16x8*>(base + col * S + (((kg ^ (col >> 3)) & 7) << 3));
  };
  // FULL: waves 0..3 multiply (A block, B block) = (0,0), (0,1), (1,1), (1,0): tiles AA, AB, BB
  // and the mirror BA, which is not stored
  const int fa_blk = (wave == 2 || wave == 3) ? 1 : 0;
  const int fb_blk = (wave == 1 || wave == 2) ? 1 : 0;
  auto products = [&](int sb) {
    if constexpr (FULL) {
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        bf16x8 fa[4], fb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          fa[i] = frag(xt[sb][fa_blk], i * 32 + (lane & 31), 2 * ks + h);
          fb[i] = frag(xt[sb][fb_blk], i * 32 + (lane & 31), 2 * ks + h);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        bf16x8 fa[2], fb[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          fa[i] = frag(xt[sb][0], wy * 64 + i * 32 + (lane & 31), 2 * ks + h);
          fb[i] = frag(xt[sb][jblk], wx * 64 + i * 32 + (lane & 31), 2 * ks + h);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
      }
    }
  };

  // prologue: rows of steps 0 and 1 in flight, RoPE of step 0 ahead of the step-1 rows.  Steps run
  // in pairs; a slice with an odd step count ends with a step of zeroed rows.
  // The scheduling fences keep each group of loads in issue order, so that the counter waits of a
  // step cover its own rows only.
  issue_rows(la, r0);
  __builtin_amdgcn_sched_barrier(0);
  issue_rope(r0);
  __builtin_amdgcn_sched_barrier(0);
  issue_rows(lb, r0 + BK);
  __builtin_amdgcn_sched_barrier(0);
  for (int64_t k0 = r0; k0 < r1; k0 += 2 * BK) {
    stage(la, k0, 0);
    __builtin_amdgcn_sched_barrier(0);
    issue_rope(k0 + BK);
    __builtin_amdgcn_sched_barrier(0);
    issue_rows(la, k0 + 2 * BK);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    products(0);
    __builtin_amdgcn_sched_barrier(0);
    stage(lb, k0 + BK, 1);
    __builtin_amdgcn_sched_barrier(0);
    issue_rope(k0 + 2 * BK);
    __builtin_amdgcn_sched_barrier(0);
    issue_rows(lb, k0 + 3 * BK);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    products(1);
    __builtin_amdgcn_sched_barrier(0);
  }

  float* out = p.partial + ((static_cast<int64_t>(job) * p.n_slices + slice) * n_upper + tile) *
                               static_cast<int64_t>(kTileFloats);
  if constexpr (FULL) {
    // waves 0, 1, 2 hold tiles AA, AB, BB (tile indices 0, 1, 2); wave 3's BA is the mirror of AB
    if (wave < 3) {
      float* to = out + wave * static_cast<int64_t>(kTileFloats);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int m = i * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
            const int n = j * 32 + (lane & 31);
            to[m * kTB + n] = acc[i][j][r];
          }
    }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = wy * 64 + i * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
          const int n = wx * 64 + j * 32 + (lane & 31);
          out[m * kTB + n] = acc[i][j][r];
        }
  }
  if (FULL) {
    // both blocks' column sums: block 0 is tile AA's, block 1 tile BB's
#pragma unroll
    for (int i = 0; i < 32; ++i)
#pragma unroll
      for (int o = 8; o <= 32; o <<= 1) csum[i] += __shfl_xor(csum[i], o, 64);
    __syncthreads();
    float* red = reinterpret_cast<float*>(&xt[0][0][0]);  // [wave][cp][32]
    if (lane < 8) {
#pragma unroll
      for (int i = 0; i < 32; ++i) red[(wave * 8 + cp) * 32 + i] = csum[i];
    }
    __syncthreads();
    {
      const int pc = tid >> 5, i = tid & 31;  // 8 chunk pairs x 32 sums
      const float v = red[(0 * 8 + pc) * 32 + i] + red[(1 * 8 + pc) * 32 + i] +
                      red[(2 * 8 + pc) * 32 + i] + red[(3 * 8 + pc) * 32 + i];
      const int b = i >> 4, e = i & 15;
      const int cc = pair_col<DH, 8>(pc) + (e >> 3) * HALF + (e & 7);
      out[(b == 0 ? 0 : 2) * static_cast<int64_t>(kTileFloats) + kTB * kTB + cc] = v;
    }
  } else if (diag) {
    // a chunk pair's rows are spread over the lanes tid % 8 == cp of every wave: reduce in the
    // wave, then over the four waves through LDS (the tiles are no longer read)
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int o = 8; o <= 32; o <<= 1) csum[i] += __shfl_xor(csum[i], o, 64);
    __syncthreads();
    float* red = reinterpret_cast<float*>(&xt[0][0][0]);  // [wave][cp][16]
    if (lane < 8) {
#pragma unroll
      for (int i = 0; i < 16; ++i) red[(wave * 8 + cp) * 16 + i] = csum[i];
    }
    __syncthreads();
    if (tid < 8 * 16) {
      const int pc = tid >> 4, i = tid & 15;
      const float v = red[(0 * 8 + pc) * 16 + i] + red[(1 * 8 + pc) * 16 + i] +
                      red[(2 * 8 + pc) * 16 + i] + red[(3 * 8 + pc) * 16 + i];
      const int cc = pair_col<DH, 8>(pc) + (i >> 3) * HALF + (i & 7);
      out[kTB * kTB + cc] = v;
    }
  }
}

template <int DH, bool DEROPE, bool PAIR>
__global__ __launch_bounds__(256, 2) void fit_gram_bf16_kernel(const FitGramParams p) {
  fit_gram_bf16_body<DH, DEROPE, PAIR, false>(p);
}

template <int DH, bool DEROPE, bool PAIR>
__global__ __launch_bounds__(256, 1) void fit_gram_full_bf16_kernel(const FitGramParams p) {
  fit_gram_bf16_body<DH, DEROPE, PAIR, true>(p);
}

// ---------------------------------------------------------------------------------------------
// fp32 Gram on the vector units (the fp32 path takes no reduced-precision products): 16-row
// k-steps staged row-major in LDS, each thread accumulates an 8 x 8 block of the tile.  Thread t
// stages row t % 16 and chunk pair t / 16 (4 columns + their RoPE partners).
// ---------------------------------------------------------------------------------------------
template <int DH, bool DEROPE>
__global__ __launch_bounds__(256) void fit_gram_f32_kernel(const FitGramParams p) {
  constexpr int BK = 16, LD = kTB + 4, HALF = DH / 2;
  __shared__ __attribute__((aligned(16))) float xs[2][BK * LD];

  const int nt = 2 * p.w / kTB, n_upper = nt * (nt + 1) / 2;
  // the tiles of one (job, slice) read the same rows: consecutive units on one XCD, so the second
  // read of a column block hits that XCD's L2
  int unit = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = unit % n_upper;
  unit /= n_upper;
  const int slice = unit % p.n_slices;
  const int job = unit / p.n_slices;
  int ti, tj;
  tile_of(tile, nt, ti, tj);
  const bool diag = ti == tj;
  const int nblk = diag ? 1 : 2;
  const FitGramJob& jb = p.jobs[job];
  const int64_t r0 = static_cast<int64_t>(slice) * p.slice_rows;
  const int64_t r1 = r0 + p.slice_rows < p.n_rows ? r0 + p.slice_rows : p.n_rows;
  const int64_t row_bytes = static_cast<int64_t>(p.w) * 4;

  const int tid = threadIdx.x;
  const int lr = tid & 15, cp = tid >> 4;
  const int c = pair_col<DH, 4>(cp);
  const int ri = c % DH;
  BlockSrc src[2];
  src[0] = block_src(jb, p.w, ti * kTB + c, 4);
  src[1] = block_src(jb, p.w, tj * kTB + c, 4);
  const int ty = tid >> 4, tx = tid & 15;

  float acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
  float csum[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) csum[i] = 0.f;

  for (int64_t k0 = r0; k0 < r1; k0 += BK) {
    const int64_t n = k0 + lr;
    float f[2][2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (b >= nblk) break;
      float4 u = make_float4(0.f, 0.f, 0.f, 0.f), v = u;
      if (n < r1) {
        const char* rowp = src[b].base + n * row_bytes + src[b].col;
        const uint4 ui = gload16(rowp), vi = gload16(rowp + HALF * 4);
        u = make_float4(__uint_as_float(ui.x), __uint_as_float(ui.y), __uint_as_float(ui.z),
                        __uint_as_float(ui.w));
        v = make_float4(__uint_as_float(vi.x), __uint_as_float(vi.y), __uint_as_float(vi.z),
                        __uint_as_float(vi.w));
      }
      f[b][0][0] = u.x; f[b][0][1] = u.y; f[b][0][2] = u.z; f[b][0][3] = u.w;
      f[b][1][0] = v.x; f[b][1][1] = v.y; f[b][1][2] = v.z; f[b][1][3] = v.w;
      if constexpr (DEROPE) {
        if (n < r1) {
          const float2* tab = p.rope + static_cast<int64_t>(fit_position(p, n)) * HALF + ri;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float2 cs = tab[j];
            const float a0 = f[b][0][j], b0 = f[b][1][j];
            f[b][0][j] = a0 * cs.x + b0 * cs.y;
            f[b][1][j] = b0 * cs.x - a0 * cs.y;
          }
        }
      }
      if (b == 0 && diag) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          csum[j] += f[0][0][j];
          csum[4 + j] += f[0][1][j];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (b >= nblk) break;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        xs[b][lr * LD + c + j] = f[b][0][j];
        xs[b][lr * LD + c + HALF + j] = f[b][1][j];
      }
    }
    __syncthreads();
    const float* xi = xs[0];
    const float* xj = xs[diag ? 0 : 1];
#pragma unroll 4
    for (int k = 0; k < BK; ++k) {
      float av[8], bv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        av[i] = xi[k * LD + ty + 16 * i];
        bv[i] = xj[k * LD + tx + 16 * i];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
    }
  }

  float* out = p.partial + ((static_cast<int64_t>(job) * p.n_slices + slice) * n_upper + tile) *
                               static_cast<int64_t>(kTileFloats);
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) out[(ty + 16 * i) * kTB + tx + 16 * j] = acc[i][j];
  if (diag) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int o = 8; o >= 1; o >>= 1) csum[i] += __shfl_xor(csum[i], o, 64);
    if (lr == 0) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        out[kTB * kTB + c + j] = csum[j];
        out[kTB * kTB + c + HALF + j] = csum[4 + j];
      }
    }
  }
}

// Sums each job's partial tiles over its slices in slice order (so the result does not depend on
// scheduling) and writes the full symmetric Gram and the column sums.  A workgroup owns one 32 x 32
// sub-block of an upper tile: it reads the partials coalesced, writes the block in place and its
// mirror image through an LDS transpose.  Inside a diagonal tile only sub-blocks on or above its
// diagonal run, and a diagonal sub-block takes element (min, max) for both (i, j) and (j, i), so the
// Gram is exactly symmetric.
__global__ __launch_bounds__(256) void fit_gram_reduce_kernel(const FitGramParams p) {
  const int n2 = 2 * p.w, nt = n2 / kTB, n_upper = nt * (nt + 1) / 2;
  const int job = blockIdx.y;
  const int tile = blockIdx.x / 16, sub = blockIdx.x % 16, sr = sub / 4, sc = sub % 4;
  int ti, tj;
  tile_of(tile, nt, ti, tj);
  const bool diag = ti == tj;
  if (diag && sr > sc) return;
  const FitGramJob& jb = p.jobs[job];
  const float* base = p.partial + (static_cast<int64_t>(job) * p.n_slices * n_upper + tile) *
                                      static_cast<int64_t>(kTileFloats);
  const int64_t slice_stride = static_cast<int64_t>(n_upper) * kTileFloats;
  __shared__ float blk[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ty + 8 * k;
    const int off = (sr * 32 + r) * kTB + sc * 32 + tx;
    float v = 0.f;
    for (int sl = 0; sl < p.n_slices; ++sl) v += base[sl * slice_stride + off];
    blk[r][tx] = v;
  }
  __syncthreads();
  const int i0 = ti * kTB + sr * 32, j0 = tj * kTB + sc * 32;
  const bool dsub = diag && sr == sc;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = ty + 8 * k;
    const float up = dsub && r > tx ? blk[tx][r] : blk[r][tx];
    jb.gram[static_cast<int64_t>(i0 + r) * n2 + j0 + tx] = up;      // G[i][j], i <= j
    if (!dsub) jb.gram[static_cast<int64_t>(j0 + r) * n2 + i0 + tx] = blk[tx][r];  // G[j][i]
  }
  if (diag && sub == 0 && threadIdx.x < kTB) {
    float v = 0.f;
    for (int sl = 0; sl < p.n_slices; ++sl) v += base[sl * slice_stride + kTB * kTB + threadIdx.x];
    jb.colsum[ti * kTB + threadIdx.x] = v;
  }
}

// ---------------------------------------------------------------------------------------------
// fp64 solve.  Every stage is one launch over all layers of the call (the last grid dimension is
// the layer), so each stage spreads over the whole GPU:
//   prep      the centred Gram G_c and the offsets;
//   tridiag   Householder reduction Q^T G_c Q = T (tridiagonal), one launch per column: the launch
//             for column k + 1 applies reflector k to the trailing block, forms reflector k + 1
//             from the updated column and the product p = tau A v that the next launch needs.  Two
//             matrix copies take turns as source and destination, so no workgroup reads what
//             another workgroup of the same launch writes; only every second launch writes.  The last steps (a trailing block of at
//             most 256 rows) run in one launch with the block in registers;
//   bisect    the r largest eigenvalues of T by multisection on Sturm counts, one wave each;
//   inverse   their eigenvectors of T by inverse iteration (three solves with T - lambda I, factored
//             once under partial pivoting); eigenvalues closer than 1e-7 ||T|| form a cluster, whose
//             vectors one thread computes in turn, each orthogonalised against the cluster's earlier
//             ones (the working vectors live in LDS);
//   back      V_r = Q Y, one wave per column, the column in registers, each column's largest-magnitude
//             entry then made positive;
//   project   P = G_c V_r;
//   normal    Z^T Z + lam I = V_r^T P + lam I and A^T A + lam I;
//   chol      Cholesky of both, 64 columns per panel and update launch;
//   out       the triangular solves for E and F, one wave per right-hand side in registers, and the
//             outputs, rounded once.
// ---------------------------------------------------------------------------------------------
constexpr int kSolveThreads = 256;
constexpr int kSolveRows = 16;  // rows per workgroup of the prep
// Rows per workgroup of 4 waves of a tridiagonal step: 4 while the launch has at most this many rows
// over its layers (three workgroups per CU), so that they spread over the chip; 8 above, where the vector
// part that every workgroup repeats costs more.  Above 1024 rows workgroups have 8 waves and twice the
// rows: the LDS holds one with a pair's five vectors.  Fit, ms, 4 / 8 rows: 1 layer at w = 1024 21.8 / 22.6, 2
// layers at w = 1024 29.7 / 28.3, 4 layers at w = 512 11.2 / 10.9, 16 layers at w = 256 6.1 / 5.9 (all
// with 4 waves and a write per launch).
constexpr int64_t kTridiagNarrow = 3072;
constexpr int kMaxN = 2 * kFitMaxSolveWidth;
constexpr int kInverseSolves = 3;
constexpr double kEps = 2.220446049250313e-16;  // 2^-52
constexpr double kClusterTol = 1e-7;            // relative to ||T||: eigenvalues closer cluster
constexpr double kNaN = __builtin_nan("");

// Per-layer table that the prep launch writes into the layer's workspace for the later launches
// (whose argument block stays small).
struct SolveJob {
  const float* gram;
  const float* colsum;
  void* w_enc;
  void* w_dec;
  void* mu_enc;
  void* mu_dec;
  int64_t rank;
  double tnorm;  // Gershgorin bound of ||T||, written by the bisection launch
};

struct SolveArgs {
  double* work;
  double rows;
  double lambda;
  int32_t w;
  int32_t step;
  int32_t center;
  int32_t bf16;
};

// One layer's workspace (fp64, n = 2w): four n x n matrices Z, X, Y, M, then 8n scalars.
struct Slots {
  double *z, *x, *y, *m;
  double *d, *e, *tau, *p0, *p1, *lam, *ldiag;
  SolveJob* job;
};

__device__ inline Slots slots(double* work, int w, int layer) {
  const int64_t n = 2 * w, n2 = n * n;
  double* b = work + layer * fit_solve_layer_doubles(w);
  Slots s;
  s.z = b;
  s.x = b + n2;
  s.y = b + 2 * n2;
  s.m = b + 3 * n2;
  double* v = b + 4 * n2;
  s.d = v;
  s.e = v + n;
  s.tau = v + 2 * n;
  s.p0 = v + 3 * n;
  s.p1 = v + 4 * n;
  s.lam = v + 5 * n;
  s.ldiag = v + 6 * n;  // Cholesky diagonals: A^T A block [w], then Z^T Z block [r]
  s.job = reinterpret_cast<SolveJob*>(v + 7 * n);
  return s;
}

// Centred Gram entry G[i][j] - s_i s_j / N in fp64 (inv = 1 / N rounded, or 0 without centring); every
// stage that needs G_c evaluates it with this one expression, so all see the same values.  The product
// of two fp32 sums is exact, and the quotient is its product with inv corrected by the exact remainder,
// which rounds as a division does (Markstein's theorem) at a quarter of its instructions.  A channel that is
// constant over the rows thus centres to exact zeros, as with a division; s_i s_j inv alone leaves
// rounding noise that the solve takes for a direction.
__device__ inline double centred(const float* gram, const float* cs, int n, int i, int j, double rows,
                                 double inv) {
  const double g = static_cast<double>(gram[static_cast<int64_t>(i) * n + j]);
  if (inv == 0.0) return g;
  const double s = static_cast<double>(cs[i]) * static_cast<double>(cs[j]), q = s * inv;
  return g - fma(fma(-q, rows, s), inv, q);
}

// Wave-wide fp64 sum without LDS: four DPP steps inside rows of 16 lanes, then the rows (halves)
// swapped against themselves.
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const int64_t b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double((static_cast<int64_t>(hi) << 32) | static_cast<uint32_t>(lo));
}
__device__ inline double row16_sum(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x140>(v);  // row_mirror
  return v;
}
// Sum over the four rows of 16 lanes (every lane keeps its column of the row).
__device__ inline double rows4_sum(double v) {
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = static_cast<uint32_t>(b), hi = static_cast<uint32_t>(b >> 32);
  auto join = [](uint32_t l, uint32_t h) {
    return __longlong_as_double((static_cast<int64_t>(h) << 32) | l);
  };
  const auto l16 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  v = join(l16[0], h16[0]) + join(l16[1], h16[1]);
  const int64_t c = __double_as_longlong(v);
  const uint32_t lo2 = static_cast<uint32_t>(c), hi2 = static_cast<uint32_t>(c >> 32);
  const auto l32 = __builtin_amdgcn_permlane32_swap(lo2, lo2, false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap(hi2, hi2, false, false);
  return join(l32[0], h32[0]) + join(l32[1], h32[1]);
}
__device__ inline double wave_sum_dpp(double v) { return rows4_sum(row16_sum(v)); }

__device__ inline void store_out(void* dst, int64_t i, double v, bool bf16) {
  if (bf16) static_cast<__bf16*>(dst)[i] = static_cast<__bf16>(static_cast<float>(v));
  else static_cast<float*>(dst)[i] = static_cast<float>(v);
}

// Where launch k of the tridiagonal steps writes (the matrix and reflector k+1): the two launches of a
// pair share a destination, pairs alternate between X and Y (launch -1: Y).
__device__ inline double* step_dst(const Slots& s, int k) { return ((k >> 1) & 1) ? s.y : s.x; }

// Reflector j lives in row j of the destination of launch j-1, entries j+1 .. n-1 (the first one 1).
__device__ inline double* reflector_rows(const Slots& s, int j) { return step_dst(s, j - 1); }

// ---- prep: G_c into Z, the offsets, the job table --------------------------------------------
__global__ __launch_bounds__(kSolveThreads) void fit_prep_kernel(const FitSolveParams p) {
  const int layer = blockIdx.y, n = 2 * p.w;
  const FitSolveJob& jb = p.jobs[layer];
  const Slots s = slots(p.work, p.w, layer);
  const double rows = static_cast<double>(p.n_rows);
  const bool center = p.center != 0, bf16 = p.bf16 != 0;
  const int i0 = blockIdx.x * kSolveRows;
  for (int e = threadIdx.x; e < kSolveRows * n; e += kSolveThreads) {
    const int i = i0 + e / n, j = e % n;
    if (i < n) s.z[static_cast<int64_t>(i) * n + j] = centred(jb.gram, jb.colsum, n, i, j, rows, center ? 1.0 / rows : 0.0);
  }
  if (blockIdx.x != 0) return;
  if (threadIdx.x == 0)
    *s.job = SolveJob{jb.gram, jb.colsum, jb.w_enc, jb.w_dec, jb.mu_enc, jb.mu_dec, jb.rank, 0.0};
  if (center) {
    for (int i = threadIdx.x; i < p.w; i += kSolveThreads) {
      store_out(jb.mu_enc, i, static_cast<double>(jb.colsum[i]) / rows, bf16);
      store_out(jb.mu_dec, i, static_cast<double>(jb.colsum[p.w + i]) / rows, bf16);
    }
  }
}

// ---- one Householder step ----------------------------------------------------------------------
// Launch k (k = -1 .. n-3), with A^(k) the matrix after reflectors 0 .. k-1 (A^(0) = G_c):
//   w_k = p_k - (tau_k / 2)(p_k . v_k) v_k;  A^(k+1) = A^(k) - v_k w_k^T - w_k v_k^T on the block
//   [k+1, n)^2 (launch -1 has no reflector to apply);
//   column k+1 of A^(k+1) gives d_{k+1}, and its part below the diagonal, x, gives reflector k+1:
//   beta = -sign(x_0) ||x||, tau = (beta - x_0) / beta, v = x / (x_0 - beta) with v_0 = 1, so that
//   (I - tau v v^T) x = beta e_0 (e_{k+1} = beta; x with nothing below x_0 takes tau = 0);
//   p_{k+1} = tau_{k+1} A^(k+1) v_{k+1} on rows [k+2, n), this workgroup's rows only.
// Launches run in pairs (k even, k + 1), and only the second writes the matrix: the first (which leaves
// its w in lam for the second) takes its updated rows no further than the registers, the second reads the
// same source and applies both reflectors, in the same order.  Above 1024 rows a step is bound by
// streaming the block, and a write less per pair took the fit of two layers at w = 1024 from 28.4 to 26.9
// ms, of one from 22.0 to 20.5.  Source: G_c (Z) for k <= 1, else the previous pair's destination
// (step_dst).  The last launch writes whatever its place, for the tail.  Reflector k+1 goes into row
// k+1 of the destination, a row no later launch writes; p alternates between two vectors.
// Every global load of a launch is issued at its start (the reflector, p and tau of the previous
// launch, row k+1 and this workgroup's rows of the source, in registers), so the launch waits on one
// round of loads and the rows arrive while the vector part's two barriers pass.  PRE: row entries per
// lane, n - k - 2 <= 64 PRE.  PAIR: the second of a pair.  write: store the matrix.  Every workgroup repeats the vector part (each thread keeps its own entries
// in registers).  Bound by launch latency and by streaming the block twice: with
// the rows loaded after the vector part, four barriers and shuffled sums, each of the 1792 steps at
// w = 1024 took about 10 us more (fit of two layers 46.3 ms, then 28.3).
template <int PRE, int ROWS, int THREADS, bool PAIR>
__global__ __launch_bounds__(THREADS, 2) void fit_tridiag_kernel(const SolveArgs a, int write) {
  constexpr int kVec = 64 * PRE + 1;  // entries k + 1 .. n - 1
  __shared__ double vk[kVec], wk[kVec], vn[kVec], vp[PAIR ? kVec : 1], wp[PAIR ? kVec : 1];
  __shared__ double red[2][THREADS / 64];
  const int layer = blockIdx.y, n = 2 * a.w, k = a.step, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kWaves = THREADS / 64, kRowsPerWave = ROWS / kWaves;
  constexpr int kOwn = (kVec + THREADS - 1) / THREADS;  // vector entries per thread
  static_assert(ROWS % kWaves == 0, "whole rows per wave");
  const Slots s = slots(a.work, a.w, layer);
  const double* src = k <= 1 ? s.z : step_dst(s, (k & ~1) - 1);
  double* dst = step_dst(s, k);
  double* p_next = ((k + 1) & 1) ? s.p1 : s.p0;
  // index x of the LDS vectors and of the block is row or column o + x
  const int o = k + 1, m = n - o;
  const int r0 = 1 + blockIdx.x * ROWS;
  // loads: reflector k, p_k and row k+1 of the source (own entries), own rows; the pair's first launch's
  // reflector and w
  double vo[kOwn], wo[kOwn], co[kOwn], tau_k = 0.0;
  double vpo[PAIR ? kOwn : 1], wpo[PAIR ? kOwn : 1], vp0 = 0.0, wp0 = 0.0;
#pragma unroll
  for (int u = 0; u < kOwn; ++u) vo[u] = wo[u] = 0.0;
  if (k >= 0) {
    const double* vrow = reflector_rows(s, k) + static_cast<int64_t>(k) * n + o;
    const double* p_cur = ((k & 1) ? s.p1 : s.p0) + o;
    tau_k = s.tau[k];
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
      const int i = tid + THREADS * u;
      if (i < m) {
        vo[u] = vrow[i];
        wo[u] = p_cur[i];
      }
    }
  }
  if constexpr (PAIR) {
    const double* vrow = reflector_rows(s, k - 1) + static_cast<int64_t>(k - 1) * n + o;
    const double* w_prev = s.lam + o;
    vp0 = vrow[0];
    wp0 = w_prev[0];
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
      const int i = tid + THREADS * u;
      vpo[u] = i < m ? vrow[i] : 0.0;
      wpo[u] = i < m ? w_prev[i] : 0.0;
    }
  }
  const double* row1 = src + static_cast<int64_t>(o) * n + o;
#pragma unroll
  for (int u = 0; u < kOwn; ++u) {
    const int i = tid + THREADS * u;
    co[u] = i < m ? row1[i] : 0.0;
  }
  double pre[kRowsPerWave][PRE];
#pragma unroll
  for (int q = 0; q < kRowsPerWave; ++q) {
    const int i = r0 + wave + kWaves * q;
    const double* arow = src + static_cast<int64_t>(o + (i < m ? i : 0)) * n + o;
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
      const int j = 1 + lane + 64 * u;
      pre[q][u] = arow[j < m ? j : m - 1];
    }
  }
  // w_k = p_k - (tau_k / 2)(p_k . v_k) v_k (zero for launch -1)
  double dot = 0.0;
#pragma unroll
  for (int u = 0; u < kOwn; ++u) dot += wo[u] * vo[u];
  dot = wave_sum_dpp(dot);
  if (lane == 0) red[0][wave] = dot;
  if (tid == 0) {
    vk[0] = vo[0];
    wk[0] = wo[0];
  }
  lds_barrier();
  double t = 0.0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) t += red[0][q];
  const double kk = 0.5 * tau_k * t;
  const double vk1 = vk[0], wk1 = wk[0] - kk * vk1;
  // column k+1 of A^(k+1) (row k+1, the matrix being symmetric) and w_k, own entries only
  double sig = 0.0;
#pragma unroll
  for (int u = 0; u < kOwn; ++u) {
    const int i = tid + THREADS * u;
    const double wi = wo[u] - kk * vo[u];
    if constexpr (PAIR) co[u] = co[u] - vp0 * wpo[u] - wp0 * vpo[u];
    co[u] = co[u] - vk1 * wi - wk1 * vo[u];
    if (i < m) {
      if constexpr (PAIR) {
        vp[i] = vpo[u];
        wp[i] = wpo[u];
      }
      vn[i] = co[u];
      if (i > 0) {  // entry 0 stays p_k's: every thread reads it above
        vk[i] = vo[u];
        wk[i] = wi;
      }
      if (i >= 2) sig += co[u] * co[u];
    }
  }
  sig = wave_sum_dpp(sig);
  if (lane == 0) red[1][wave] = sig;
  lds_barrier();
  double sigma = 0.0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) sigma += red[1][q];
  const double d_next = vn[0], alpha = vn[1];
  double tau = 0.0, beta = alpha, scale = 0.0;
  if (!(sigma == 0.0)) {
    const double norm = sqrt(alpha * alpha + sigma);
    beta = alpha >= 0.0 ? -norm : norm;
    tau = (beta - alpha) / beta;
    scale = 1.0 / (alpha - beta);
  }
  // this workgroup's rows of A^(k+1) and of p_{k+1}; v_{k+1} is the column scaled, its first entry 1
  // (entries past the end: zero)
  double acc[kRowsPerWave], vi[kRowsPerWave], wi[kRowsPerWave], vpi[kRowsPerWave], wpi[kRowsPerWave];
#pragma unroll
  for (int q = 0; q < kRowsPerWave; ++q) {
    const int i = r0 + wave + kWaves * q;
    acc[q] = 0.0;
    vi[q] = vk[i < m ? i : 0];
    wi[q] = wk[i < m ? i : 0];
    vpi[q] = PAIR ? vp[i < m ? i : 0] : 0.0;
    wpi[q] = PAIR ? wp[i < m ? i : 0] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < PRE; ++u) {
    const int j = 1 + lane + 64 * u;
    if (j < m) {
      const double wj = wk[j], vj = vk[j], nj = j == 1 ? 1.0 : vn[j] * scale;
#pragma unroll
      for (int q = 0; q < kRowsPerWave; ++q) {
        const int i = r0 + wave + kWaves * q;
        double v = pre[q][u];
        if constexpr (PAIR) v = v - vpi[q] * wp[j] - wpi[q] * vp[j];
        v = v - vi[q] * wj - wi[q] * vj;
        if (i < m) {
          if (write) dst[static_cast<int64_t>(o + i) * n + o + j] = v;
          acc[q] += v * nj;
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kRowsPerWave; ++q) {
    const int i = r0 + wave + kWaves * q;
    const double y = wave_sum_dpp(acc[q]);
    if (lane == 0 && i < m) p_next[o + i] = tau * y;
  }
  if (blockIdx.x == 0) {
    double* vrow = dst + static_cast<int64_t>(o) * n + o;
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
      const int i = tid + THREADS * u;
      if (i >= 1 && i < m) {
        vrow[i] = i == 1 ? 1.0 : co[u] * scale;
        if (!PAIR) s.lam[o + i] = wo[u] - kk * vo[u];
      }
    }
    if (tid == 0) {
      s.d[k + 1] = d_next;
      s.e[k + 1] = beta;
      s.tau[k + 1] = tau;
    }
  }
}

__device__ inline double readlane_f64(double v, int lane) {
  const int64_t b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(static_cast<int>(b), lane);
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), lane);
  return __longlong_as_double((static_cast<int64_t>(hi) << 32) | static_cast<uint32_t>(lo));
}

// The last steps, from step k0 on (trailing block of at most kTailN rows), in one launch: one
// workgroup per layer keeps the block [k0 + 1, n)^2 of A^(k0) in registers and applies the same steps
// as the per-column launches, the workgroup barriers standing in for the launch boundaries.
// k0 = -1 starts from G_c itself.
//
// The steps are a chain, so the layout keeps each one short.  The lower triangle (with whole 32 x 32
// blocks on the diagonal) is spread over 512 threads, thread (ty, tx) holding rows ty + 32 a and
// columns tx + 16 b; an element serves its row's sum and, below the diagonal blocks, its mirror's.  The
// threads' partial sums meet in LDS, where two threads add up each entry (lane reductions for 8 rows and
// 14 column blocks cost twice that).  The vector part of a step (w, the next column, its reflector) is
// one wave's work with four entries a lane, so it needs no barrier of its own: three barriers per
// step.  256 rows take 3.3 us a step on average; in LDS
// with a wave per row and six-step shuffles (128 rows at most) a step took 5.9 us, and the columns
// before that 9.6 us a launch.
constexpr int kTailN = 256, kTailThreads = 512;
__global__ __launch_bounds__(kTailThreads, 2) void fit_tridiag_tail_kernel(const SolveArgs a) {
  constexpr int kRB = kTailN / 32, kCB = kTailN / 16;
  // partial sums of A v: by thread row ty for the columns, by thread column tx for the rows (padded so
  // that the 64 lanes of a store hit distinct banks)
  constexpr int kRowLd = kTailN + 4;
  __shared__ double col[kTailN], vs[kTailN], ws[kTailN], ns[kTailN], ps[kTailN];
  __shared__ double cpart[32][kTailN], rpart[16][kRowLd];
  const int layer = blockIdx.x, n = 2 * a.w, k0 = a.step, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tx = tid & 15, ty = tid >> 4;
  const Slots s = slots(a.work, a.w, layer);
  const int o = k0 + 1;  // global index of local row / column 0
  const int m0 = n - o;  // rows of the block (<= kTailN)
  const double* src = k0 <= 0 ? s.z : step_dst(s, k0 - 1);
  double am[kRB][kCB];  // blocks b <= 2 row + 1
#pragma unroll
  for (int r = 0; r < kRB; ++r)
#pragma unroll
    for (int b = 0; b < 2 * r + 2; ++b) {
      const int i = ty + 32 * r, j = tx + 16 * b;
      am[r][b] = i < m0 && j < m0 ? src[static_cast<int64_t>(o + i) * n + o + j] : 0.0;
    }
  for (int i = tid; i < kTailN; i += kTailThreads)
    col[i] = i < m0 ? src[static_cast<int64_t>(o) * n + o + i] : 0.0;
  for (int i = tid; i < 32 * kTailN; i += kTailThreads) (&cpart[0][0])[i] = 0.0;
  for (int i = tid; i < 16 * kRowLd; i += kTailThreads) (&rpart[0][0])[i] = 0.0;
  // wave 0: p_k and v_k, entries lane + 64 q
  double pq[4] = {0.0, 0.0, 0.0, 0.0}, vq[4] = {0.0, 0.0, 0.0, 0.0}, tau = 0.0;
  if (wave == 0 && k0 >= 0) {
    const double* vrow = reflector_rows(s, k0) + static_cast<int64_t>(k0) * n;
    const double* p_cur = (k0 & 1) ? s.p1 : s.p0;
    tau = s.tau[k0];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = lane + 64 * q;
      if (i < m0) {
        vq[q] = vrow[o + i];
        pq[q] = p_cur[o + i];
      }
    }
  }
  __syncthreads();
  auto entry = [&](const double (&x)[4], int i) {  // entry i (uniform) of a wave-wide vector
    const int l = i & 63;
    const double y0 = readlane_f64(x[0], l), y1 = readlane_f64(x[1], l);
    const double y2 = readlane_f64(x[2], l), y3 = readlane_f64(x[3], l);
    return i < 128 ? (i < 64 ? y0 : y1) : (i < 192 ? y2 : y3);
  };
  for (int k = k0; k <= n - 3; ++k) {
    const int c = k + 1 - o;  // local index of global k + 1
    if (wave == 0) {
      double dot = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = lane + 64 * q;
        if (k > k0) pq[q] = tau * ps[i];
        if (i < c) pq[q] = vq[q] = 0.0;
        dot += pq[q] * vq[q];
      }
      const double kk = 0.5 * tau * wave_sum_dpp(dot);
      double wq[4], cq[4], sig = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) wq[q] = pq[q] - kk * vq[q];
      const double v1 = entry(vq, c), w1 = entry(wq, c);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = lane + 64 * q;
        cq[q] = col[i] - v1 * wq[q] - w1 * vq[q];
        if (i >= c + 2) sig += cq[q] * cq[q];
      }
      const double sigma = wave_sum_dpp(sig);
      const double d_next = entry(cq, c), alpha = entry(cq, c + 1);
      double beta = alpha, scale = 0.0;
      tau = 0.0;
      if (!(sigma == 0.0)) {
        // tau = (beta - alpha) / beta and scale = 1 / (alpha - beta), from one division unless their
        // common denominator comes near the smallest normal number (a column of about 1e-145)
        const double norm = sqrt(alpha * alpha + sigma);
        beta = alpha >= 0.0 ? -norm : norm;
        const double diff = alpha - beta, den = beta * diff;
        if (fabs(den) < 1e-290) {
          tau = -diff / beta;
          scale = 1.0 / diff;
        } else {
          const double inv = 1.0 / den;
          tau = -diff * diff * inv;
          scale = beta * inv;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = lane + 64 * q;
        vs[i] = i > c ? vq[q] : 0.0;
        ws[i] = i > c ? wq[q] : 0.0;
        vq[q] = i > c + 1 ? cq[q] * scale : (i == c + 1 ? 1.0 : 0.0);
        if (i >= m0) vq[q] = 0.0;
        ns[i] = vq[q];
      }
      if (lane == 0) {
        s.d[k + 1] = d_next;
        s.e[k + 1] = beta;
        s.tau[k + 1] = tau;
      }
    }
    lds_barrier();
    // reflector k + 1 where the per-column launches keep it
    if (tid < kTailN && tid > c && tid < m0)
      reflector_rows(s, k + 1)[static_cast<int64_t>(k + 1) * n + o + tid] = ns[tid];
    // A^(k+1) on [c + 1, m0)^2 and the sums of A^(k+1) v_{k+1}; column c + 1 for the next step
    double vi[kRB], wi[kRB], ni[kRB], rs[kRB];
#pragma unroll
    for (int r = 0; r < kRB; ++r) {
      vi[r] = vs[ty + 32 * r];
      wi[r] = ws[ty + 32 * r];
      ni[r] = ns[ty + 32 * r];
      rs[r] = 0.0;
    }
#pragma unroll
    for (int b = 0; b < kCB; ++b) {
      if (16 * b + 15 <= c || 16 * b >= m0) continue;  // columns all done, or past the end
      const double vj = vs[tx + 16 * b], wj = ws[tx + 16 * b], nj = ns[tx + 16 * b];
      double cs = 0.0;
#pragma unroll
      for (int r = b / 2; r < kRB; ++r) {
        am[r][b] = am[r][b] - vi[r] * wj - wi[r] * vj;
        rs[r] += am[r][b] * nj;
        if (r > b / 2) cs += am[r][b] * ni[r];
      }
      if (b / 2 + 1 < kRB) cpart[ty][tx + 16 * b] = cs;
      if (b == (c + 1) / 16 && tx == ((c + 1) & 15)) {
#pragma unroll
        for (int r = b / 2; r < kRB; ++r) col[ty + 32 * r] = am[r][b];
      }
    }
#pragma unroll
    for (int r = 0; r < kRB; ++r) rpart[tx][ty + 32 * r] = rs[r];
    lds_barrier();
    {
      // two threads per entry: half of its column's and half of its row's partial sums each
      const int i = tid >> 1, h = tid & 1;
      double t = 0.0;
#pragma unroll
      for (int m = 0; m < 16; ++m) t += cpart[16 * h + m][i];
#pragma unroll
      for (int m = 0; m < 8; ++m) t += rpart[8 * h + m][i];
      t += dpp_f64<0xB1>(t);
      if (h == 0) ps[i] = t;
    }
    lds_barrier();
  }
  if (tid == 0) s.d[n - 1] = col[m0 - 1];
}

// ---- bisection -------------------------------------------------------------------------------
// Number of eigenvalues of T below x (Sturm count of the LDL^T pivots of T - x I); a pivot smaller
// in magnitude than pivmin counts as -pivmin.  The pivots are a chain, so the quotient is the hardware
// reciprocal with two Newton steps (within an ulp; pivmin keeps the pivot normal) instead of an IEEE
// division, about half its latency.
__device__ inline int sturm_count(const double* d, const double* e2, int n, double x, double pivmin) {
  double q = d[0] - x;
  if (fabs(q) < pivmin) q = -pivmin;
  int c = q < 0.0 ? 1 : 0;
#pragma unroll 8
  for (int i = 1; i < n; ++i) {
    double r = __builtin_amdgcn_rcp(q);
    r = fma(fma(-q, r, 1.0), r, r);
    r = fma(fma(-q, r, 1.0), r, r);
    q = fma(-e2[i - 1], r, d[i] - x);
    if (fabs(q) < pivmin) q = -pivmin;
    c += q < 0.0 ? 1 : 0;
  }
  return c;
}

// Gershgorin interval of T, over the workgroup (64 threads, one wave).
__device__ inline void gershgorin(const double* d, const double* ae, int n, double& lo, double& hi) {
  lo = INFINITY;
  hi = -INFINITY;
  for (int i = threadIdx.x; i < n; i += 64) {
    const double rad = (i > 0 ? ae[i - 1] : 0.0) + (i < n - 1 ? ae[i] : 0.0);
    lo = fmin(lo, d[i] - rad);
    hi = fmax(hi, d[i] + rad);
  }
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o, 64));
    hi = fmax(hi, __shfl_xor(hi, o, 64));
  }
}

// One wave per eigenvalue: lam[j] = the (j+1)-th largest.  Every round the 64 lanes take Sturm counts
// at 64 evenly spaced interior points of the bracket, which then shrinks to the pair of neighbouring
// points (ends included) between which the count passes j's ascending index: a 65-fold cut per round (9
// rounds; 16 lanes need 13), until the bracket is below an absolute 2^-52 ||T|| plus a relative 2^-51.
constexpr int kSectionLanes = 64;
template <int N>  // n <= N: the LDS decides how many waves a CU holds
__global__ __launch_bounds__(64) void fit_bisect_kernel(const SolveArgs a) {
  __shared__ double d[N], e2[N], ae[N];
  const int layer = blockIdx.y, n = 2 * a.w;
  const Slots s = slots(a.work, a.w, layer);
  const int r = static_cast<int>(s.job->rank);
  for (int i = threadIdx.x; i < n; i += 64) {
    d[i] = s.d[i];
    const double e = i < n - 1 ? s.e[i] : 0.0;
    e2[i] = e * e;
    ae[i] = fabs(e);
  }
  __syncthreads();
  double lo0, hi0;
  gershgorin(d, ae, n, lo0, hi0);
  // a floor keeps the tolerances positive for an all-zero matrix
  const double tnorm = fmax(fmax(fabs(lo0), fabs(hi0)), 1e-280);
  if (blockIdx.x == 0 && threadIdx.x == 0) s.job->tnorm = tnorm;
  const int lane = threadIdx.x & (kSectionLanes - 1);
  const int j = blockIdx.x;
  const bool live = j < r;
  const double atol = kEps * tnorm, pivmin = kEps * tnorm;
  const int t = n - 1 - j;  // ascending index
  double lo = lo0 - atol, hi = hi0 + atol;
  for (int it = 0; it < 64; ++it) {
    if (hi - lo <= atol + 2.0 * kEps * fmax(fabs(lo), fabs(hi))) break;
    // point k = 1 .. 64 at lo + k step; the new ends are points (or the old ends), so the counts
    // already taken there hold for them
    const double step = (hi - lo) * (1.0 / (kSectionLanes + 1));
    const double x = lo + step * (lane + 1);
    const bool below = live && sturm_count(d, e2, n, x, pivmin) <= t;
    // lanes whose point lies below the eigenvalue (a prefix)
    const uint64_t m = __ballot(below);
    const int kb = __popcll(m);
    const double nlo = kb > 0 ? lo + step * kb : lo;
    const double nhi = kb < kSectionLanes ? lo + step * (kb + 1) : hi;
    lo = nlo;
    hi = nhi;
  }
  if (live && lane == 0) s.lam[j] = 0.5 * (lo + hi);
}

// ---- inverse iteration --------------------------------------------------------------------------
__device__ inline double start_entry(int i, int m) {
  uint32_t x = static_cast<uint32_t>(i) * 0x9E3779B1u ^ (static_cast<uint32_t>(m) + 0x7F4A7C15u) * 0x85EBCA77u;
  x ^= x >> 16;
  x *= 0x7FEB352Du;
  x ^= x >> 15;
  x *= 0x846CA68Bu;
  x ^= x >> 16;
  return static_cast<double>(x >> 8) * (1.0 / 16777216.0) - 0.5;
}

// A pivot smaller than tol in magnitude becomes +-tol (NaN stays NaN).
__device__ inline double guard_pivot(double c, double tol) {
  return !(fabs(c) <= tol) ? c : (c >= 0.0 ? tol : -tol);
}

// Strided view of one vector: entry i at p[i * stride].
struct Strided {
  double* p;
  int64_t stride;
  __device__ double& operator[](int i) const { return p[i * stride]; }
};

// What one eigenvector's inverse iteration works on: the vector, the LU factors of T - sigma I under
// partial pivoting (inverse diagonal, two superdiagonals, multipliers) and the row swaps.
struct InverseWork {
  Strided y, u0, u1, u2, mult;
  uint8_t* swap;
  int swap_stride;
};

// Inverse iteration for the cluster of eigenvalues lam[j .. last] (one thread).  Every finished vector m
// is stored at out(m) (Y[i][m] of the layer), which is also where the orthogonalisation reads the
// earlier members.  n is a multiple of kInvChunk.  The factors do not change between the solves of one
// eigenvalue, so they are formed once and no solve divides; the solves read kInvChunk entries ahead of
// the recurrence (which is one fma a step forward, two back), and the sums of a vector come out of its
// back substitution.
constexpr int kInvChunk = 8;
template <typename OutFn>
__device__ inline void inverse_cluster(const double* d, const double* e, int n, const double* lam,
                                       int j, int last, double tnorm, const InverseWork& wk, OutFn out) {
  const double pert = 10.0 * kEps * tnorm, ptol = kEps * tnorm;
  const Strided y = wk.y, u0 = wk.u0, u1 = wk.u1, u2 = wk.u2, mult = wk.mult;
  double sigma = 0.0;
  for (int m = j; m <= last; ++m) {
    // shifts inside a cluster step down by at least pert, so the solves stay independent
    sigma = m == j ? lam[m] : fmin(lam[m], sigma - pert);
    {
      // elimination of T - sigma I; a row holds (c0, c1) on the diagonal and the superdiagonal
      double c0 = d[0] - sigma, c1 = n > 1 ? e[0] : 0.0;
      for (int i = 0; i < n - 1; ++i) {
        const double sub = e[i], a1 = d[i + 1] - sigma, b1 = i + 1 < n - 1 ? e[i + 1] : 0.0;
        const bool keep = fabs(c0) >= fabs(sub);
        const double piv = keep ? guard_pivot(c0, ptol) : sub;
        const double inv = 1.0 / piv;
        const double ml = (keep ? sub : c0) / piv;
        u0[i] = inv;
        u1[i] = keep ? c1 : a1;
        u2[i] = keep ? 0.0 : b1;
        mult[i] = ml;
        wk.swap[i * wk.swap_stride] = keep ? 0 : 1;
        const double n0 = keep ? a1 - ml * c1 : c1 - ml * a1;
        c1 = keep ? b1 : -ml * b1;
        c0 = n0;
      }
      u0[n - 1] = 1.0 / guard_pivot(c0, ptol);
      u1[n - 1] = u2[n - 1] = mult[n - 1] = 0.0;
      wk.swap[(n - 1) * wk.swap_stride] = 0;
    }
    for (int i = 0; i < n; ++i) y[i] = start_entry(i, m);
    double sc = 2.0;  // the start vector's entries lie in [-1/2, 1/2)
    double ss = 0.0, mx = 0.0;
    for (int it = 0; it < kInverseSolves; ++it) {
      // forward: the right-hand side b / max|b| through the elimination
      double yc = y[0] * sc;
      for (int i0 = 0; i0 < n; i0 += kInvChunk) {
        double nb[kInvChunk], ml[kInvChunk], yo[kInvChunk];
        int sw[kInvChunk];
#pragma unroll
        for (int u = 0; u < kInvChunk; ++u) {
          nb[u] = y[i0 + u + 1 < n ? i0 + u + 1 : n - 1] * sc;
          ml[u] = mult[i0 + u];
          sw[u] = wk.swap[(i0 + u) * wk.swap_stride];
        }
#pragma unroll
        for (int u = 0; u < kInvChunk; ++u) {
          // the last row has nothing below it: its value is the running one
          yo[u] = sw[u] ? nb[u] : yc;
          yc = sw[u] ? yc - ml[u] * nb[u] : nb[u] - ml[u] * yc;
        }
#pragma unroll
        for (int u = 0; u < kInvChunk; ++u) y[i0 + u] = yo[u];
      }
      // back substitution, in place
      double x1 = 0.0, x2 = 0.0;
      ss = 0.0;
      mx = 0.0;
      for (int i0 = n - kInvChunk; i0 >= 0; i0 -= kInvChunk) {
        double v[kInvChunk], a0[kInvChunk], a1[kInvChunk], a2[kInvChunk];
#pragma unroll
        for (int u = 0; u < kInvChunk; ++u) {
          v[u] = y[i0 + u];
          a0[u] = u0[i0 + u];
          a1[u] = u1[i0 + u];
          a2[u] = u2[i0 + u];
        }
#pragma unroll
        for (int u = kInvChunk - 1; u >= 0; --u) {
          v[u] = (v[u] - a2[u] * x2 - a1[u] * x1) * a0[u];
          x2 = x1;
          x1 = v[u];
          ss += v[u] * v[u];
          mx = fmax(mx, fabs(v[u]));
        }
#pragma unroll
        for (int u = 0; u < kInvChunk; ++u) y[i0 + u] = v[u];
      }
      if (m > j) {
        // orthogonalise the normalised vector against the cluster's earlier ones
        const double inv = 1.0 / sqrt(ss);
        for (int i = 0; i < n; ++i) y[i] *= inv;
        for (int q = j; q < m; ++q) {
          const Strided yq = out(q);
          double dot = 0.0;
          for (int i = 0; i < n; ++i) dot += yq[i] * y[i];
          for (int i = 0; i < n; ++i) y[i] -= dot * yq[i];
        }
        ss = mx = 0.0;
        for (int i = 0; i < n; ++i) {
          ss += y[i] * y[i];
          mx = fmax(mx, fabs(y[i]));
        }
      }
      sc = mx > 0.0 ? 1.0 / mx : 1.0;
    }
    // a norm past fp64's range (only a zero matrix gets there, whose pivots are all the guard) leaves NaN:
    // dividing by it would pass a zero vector off as a direction
    const Strided o = out(m);
    const double inv = ss < INFINITY ? 1.0 / sqrt(ss) : kNaN;
    for (int i = 0; i < n; ++i) o[i] = y[i] * inv;
  }
}

// One thread per eigenvalue; only the first thread of a cluster works (it takes the whole
// cluster in order).  Returns false for threads with nothing to do.
__device__ inline bool cluster_of(const double* lam, int r, int j, double ctol, int* last) {
  if (j >= r || (j > 0 && !(lam[j - 1] - lam[j] > ctol))) return false;
  int l = j;
  while (l + 1 < r && !(lam[l] - lam[l + 1] > ctol)) ++l;
  *last = l;
  return true;
}

// Inverse iteration, one eigenvector per working thread: the thread keeps its vector and the LU
// factors of T - sigma I in LDS ([i][thread], THREADS interleaved, so the threads' accesses fall in
// distinct banks) and copies each finished vector to Y[i][m].  Two instances: 8 threads per workgroup
// for n <= 256, and one thread per workgroup (114 KiB of LDS) for larger n; the chain of dependent
// accesses would otherwise wait on global memory at each link.  28 layers x 64 vectors of 256 150 us, 2
// layers x 128 vectors of 2048 1.1 ms (a division per row in every solve, and the sums in passes of their
// own: 362 us and 2.9 ms).
constexpr int kInverseLdsN = 256, kInverseLdsThreads = 8;
template <int N, int THREADS>
__global__ __launch_bounds__(64) void fit_inverse_lds_kernel(const SolveArgs a) {
  __shared__ double d[N], e[N];
  __shared__ double vec[5 * N * THREADS];
  __shared__ uint8_t swap[N * THREADS];
  const int layer = blockIdx.y, n = 2 * a.w;
  const Slots s = slots(a.work, a.w, layer);
  const int r = static_cast<int>(s.job->rank);
  for (int i = threadIdx.x; i < n; i += 64) {
    d[i] = s.d[i];
    e[i] = i < n - 1 ? s.e[i] : 0.0;
  }
  __syncthreads();
  const int t = threadIdx.x;
  const int j = blockIdx.x * THREADS + t;
  if (t >= THREADS) return;
  const double tnorm = s.job->tnorm;
  int last;
  if (!cluster_of(s.lam, r, j, kClusterTol * tnorm, &last)) return;
  constexpr int64_t kPlane = static_cast<int64_t>(N) * THREADS;
  auto lds = [&](int q) { return Strided{vec + q * kPlane + t, THREADS}; };
  inverse_cluster(
      d, e, n, s.lam, j, last, tnorm,
      InverseWork{lds(0), lds(1), lds(2), lds(3), lds(4), swap + t, THREADS},
      [&](int m) { return Strided{s.z + m, r}; });
}

// ---- back-transformation and sign ---------------------------------------------------------------
// One wave per column of Y: the column stays in registers (entry lane + 64 q) while the reflectors
// n-3 .. 0 are applied in turn (y <- y - tau_j (v_j . y) v_j), each loaded while the one before is
// applied.  The n - 2 reflectors are a chain, and a wave's sum needs no barrier: n = 256, 28 layers x
// 64 columns 103 us, n = 2048, 2 layers x 128 columns 0.96 ms (8 columns per workgroup in LDS, three barriers
// per reflector: 330 us and 3.5 ms).  Then the column's first entry of largest magnitude is made
// positive.  NQ: entries per lane, n <= 64 NQ (MASK: n < 64 NQ).  The
// reflectors run in groups of 64 kGrp whose first live entry register is a constant, so the loops hold no
// tests of it.
template <int NQ, bool MASK, int Q0>
__device__ __forceinline__ void back_group(const Slots& s, int n, int j1, double (&y)[NQ]) {
  constexpr int kGrp = NQ >= 16 ? 4 : 1;
  if constexpr (Q0 >= 0) {
    // reflectors j1 .. 64 Q0 - 1 (down to 0 in the last group): entries past j, all in registers >= Q0
    const int j0 = Q0 == 0 ? 0 : 64 * Q0 - 1, lane = threadIdx.x;
    double cur[NQ], nxt[NQ], tnxt = 0.0;
    auto fetch = [&](int j) {
      tnxt = s.tau[j];
      const double* vrow = reflector_rows(s, j) + static_cast<int64_t>(j) * n;
#pragma unroll
      for (int q = Q0; q < NQ; ++q) {
        const int i = lane + 64 * q;
        const double v = vrow[MASK && i >= n ? n - 1 : i];
        nxt[q] = (q < Q0 + kGrp && i <= j) || (MASK && i >= n) ? 0.0 : v;
      }
    };
    if (j1 >= j0) fetch(j1);
    for (int j = j1; j >= j0; --j) {
      const double t = tnxt;
#pragma unroll
      for (int q = Q0; q < NQ; ++q) cur[q] = nxt[q];
      fetch(j > j0 ? j - 1 : j0);
      double dot = 0.0;
#pragma unroll
      for (int q = Q0; q < NQ; ++q) dot += cur[q] * y[q];
      const double f = t * wave_sum_dpp(dot);
      if (t == 0.0) continue;
#pragma unroll
      for (int q = Q0; q < NQ; ++q) y[q] -= f * cur[q];
    }
    back_group<NQ, MASK, Q0 - kGrp>(s, n, j0 - 1 < j1 ? j0 - 1 : j1, y);
  }
}

template <int NQ, bool MASK>
__global__ __launch_bounds__(64) void fit_back_kernel(const SolveArgs a) {
  const int layer = blockIdx.y, n = 2 * a.w, lane = threadIdx.x;
  const Slots s = slots(a.work, a.w, layer);
  const int r = static_cast<int>(s.job->rank), c = blockIdx.x;
  if (c >= r) return;
  double y[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = lane + 64 * q;
    y[q] = i < n ? s.z[static_cast<int64_t>(i) * r + c] : 0.0;
  }
  back_group<NQ, MASK, NQ - (NQ >= 16 ? 4 : 1)>(s, n, n - 3, y);
  double best = -1.0, val = 0.0;
  int bi = 0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = lane + 64 * q;
    if (i < n && fabs(y[q]) > best) {
      best = fabs(y[q]);
      val = y[q];
      bi = i;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64), ov = __shfl_xor(val, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (ob > best || (ob == best && oi < bi)) {
      best = ob;
      val = ov;
      bi = oi;
    }
  }
  const double sg = val < 0.0 ? -1.0 : 1.0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = lane + 64 * q;
    if (i < n) s.z[static_cast<int64_t>(i) * r + c] = sg * y[q];
  }
}

// ---- fp64 tiled products ------------------------------------------------------------------------
// 64 x 64 output tile per workgroup, 4 x 4 per thread, k-steps of 16 through LDS.  ta(kk, i) and
// tb(kk, j) give the operands' entries for reduction index kk (0 outside the matrix).
template <typename FA, typename FB, typename FC>
__device__ inline void tile_product(int kdim, FA ta, FB tb, FC out) {
  __shared__ double as[16][64 + 1], bs[16][64 + 1];
  const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
  double acc[4][4] = {};
  for (int k0 = 0; k0 < kdim; k0 += 16) {
    for (int e = tid; e < 16 * 64; e += kSolveThreads) {
      const int kk = e / 64, x = e % 64;
      as[kk][x] = k0 + kk < kdim ? ta(k0 + kk, x) : 0.0;
      bs[kk][x] = k0 + kk < kdim ? tb(k0 + kk, x) : 0.0;
    }
    __syncthreads();
    for (int kk = 0; kk < 16; ++kk) {
      double av[4], bv[4];
      for (int q = 0; q < 4; ++q) {
        av[q] = as[kk][ty + 16 * q];
        bv[q] = bs[kk][tx + 16 * q];
      }
      for (int q = 0; q < 4; ++q)
        for (int u = 0; u < 4; ++u) acc[q][u] += av[q] * bv[u];
    }
    __syncthreads();
  }
  for (int q = 0; q < 4; ++q)
    for (int u = 0; u < 4; ++u) out(ty + 16 * q, tx + 16 * u, acc[q][u]);
}

// P = G_c V_r [n, r] into M (grid: n / 64 x ceil(r_max / 64) tiles, layers)
__global__ __launch_bounds__(kSolveThreads) void fit_project_kernel(const SolveArgs a) {
  const int layer = blockIdx.z, n = 2 * a.w;
  const Slots s = slots(a.work, a.w, layer);
  const SolveJob jb = *s.job;
  const int r = static_cast<int>(jb.rank);
  const int i0 = blockIdx.x * 64, m0 = blockIdx.y * 64;
  if (m0 >= r) return;
  const double inv = a.center ? 1.0 / a.rows : 0.0;
  tile_product(
      n,
      // G_c is symmetric: its column i0 + x read as a row, so the loads run along rows
      [&](int kk, int x) { return centred(jb.gram, jb.colsum, n, kk, i0 + x, a.rows, inv); },
      [&](int kk, int x) {
        return m0 + x < r ? s.z[static_cast<int64_t>(kk) * r + m0 + x] : 0.0;
      },
      [&](int x, int y, double v) {
        if (m0 + y < r) s.m[static_cast<int64_t>(i0 + x) * r + m0 + y] = v;
      });
}

// Z^T Z + lam I = V_r^T P + lam I [r, r] into Y (grid.x = tiles of it), and A^T A + lam I [w, w]
// into X (grid.y = 1: w / 64 x w / 64 tiles over grid.x)
__global__ __launch_bounds__(kSolveThreads) void fit_normal_kernel(const SolveArgs a) {
  const int layer = blockIdx.z, n = 2 * a.w, w = a.w;
  const Slots s = slots(a.work, a.w, layer);
  const SolveJob jb = *s.job;
  const int r = static_cast<int>(jb.rank);
  if (blockIdx.y == 0) {
    const int nt = (r + 63) / 64;
    if (static_cast<int>(blockIdx.x) >= nt * nt) return;
    const int k0 = (blockIdx.x / nt) * 64, l0 = (blockIdx.x % nt) * 64;
    tile_product(
        n,
        [&](int i, int x) { return k0 + x < r ? s.z[static_cast<int64_t>(i) * r + k0 + x] : 0.0; },
        [&](int i, int x) { return l0 + x < r ? s.m[static_cast<int64_t>(i) * r + l0 + x] : 0.0; },
        [&](int x, int y, double v) {
          const int k = k0 + x, l = l0 + y;
          if (k < r && l < r) s.y[static_cast<int64_t>(k) * r + l] = v + (k == l ? a.lambda : 0.0);
        });
  } else {
    const int nt = w / 64;
    if (static_cast<int>(blockIdx.x) >= nt * nt) return;
    const int i0 = (blockIdx.x / nt) * 64, j0 = (blockIdx.x % nt) * 64;
    const double inv = a.center ? 1.0 / a.rows : 0.0;
    for (int e = threadIdx.x; e < 64 * 64; e += kSolveThreads) {
      const int i = i0 + e / 64, j = j0 + e % 64;
      s.x[static_cast<int64_t>(i) * w + j] =
          centred(jb.gram, jb.colsum, n, i, j, a.rows, inv) + (i == j ? a.lambda : 0.0);
    }
  }
}

// ---- Cholesky, 64 columns per pair of launches ------------------------------------------------------
// grid.y = 0: A^T A + lam I (X, size w), 1: Z^T Z + lam I (Y, size r).  Panel p holds columns
// [64 p, 64 p + 64).  The panel launch factors the panel's diagonal block (every workgroup for itself)
// and solves one 64-row block below it per workgroup in the same steps; the update launch takes
// the panel's part off the trailing lower triangle, a 64 x 64 tile per workgroup.  L[i][k] (i > k) is
// stored twice, in places nothing reads before the solves: at [k][i] in the upper triangle (column k of
// L as a row) and at [i][k] of a row-major copy of L just past the matrix; 1 / L[k][k] goes to ldiag.  A
// non-positive pivot leaves NaN, which reaches every output of the layer.  (One column per launch took
// 7.6 ms at w = 1024; one workgroup per matrix in LDS took 140 us at w = 128.)
constexpr int kPanel = 64;

__global__ __launch_bounds__(kSolveThreads) void fit_chol_panel_kernel(const SolveArgs a) {
  constexpr int LD = kPanel + 1;
  __shared__ double dg[kPanel][LD], xb[kPanel][LD];  // the diagonal block; this workgroup's rows below
  __shared__ double lt[kPanel][LD];                  // lt[k][j] = L[j][k], [k][k]: its inverse
  const int layer = blockIdx.z, w = a.w, tid = threadIdx.x;
  const Slots s = slots(a.work, a.w, layer);
  const int r = static_cast<int>(s.job->rank);
  const bool zz = blockIdx.y == 1;
  const int sz = zz ? r : w, k0 = a.step * kPanel;
  const int row0 = k0 + kPanel * static_cast<int>(blockIdx.x);  // first row of the block it stores
  if (row0 >= sz) return;
  const bool below = blockIdx.x > 0;
  const int kn = sz - k0 < kPanel ? sz - k0 : kPanel;  // columns of the panel
  double* mat = zz ? s.y : s.x;
  double* copy = mat + static_cast<int64_t>(sz) * sz;
  double* ldiag = s.ldiag + (zz ? w : 0);
  const int i = tid & 63, g = tid >> 6;  // row of both blocks; columns k + 1 + g, step 4
  // past the matrix's end: the identity, and rows of zeros
  for (int q = g; q < kPanel; q += 4) {
    dg[q][i] = q < kn && i < kn ? mat[static_cast<int64_t>(k0 + q) * sz + k0 + i] : (q == i ? 1.0 : 0.0);
    xb[q][i] = below && row0 + q < sz ? mat[static_cast<int64_t>(row0 + q) * sz + k0 + i] : 0.0;
  }
  __syncthreads();
  // column k of both blocks stays unscaled (every thread of a row reads it during step k)
  for (int k = 0; k < kPanel; ++k) {
    const double piv = dg[k][k];
    const double inv = piv > 0.0 ? 1.0 / sqrt(piv) : kNaN;
    const double l = dg[i][k] * inv, x = xb[i][k] * inv;
    if (g == 0) lt[k][i] = i == k ? inv : l;
    for (int j = k + 1 + g; j < kPanel; j += 4) {
      const double lj = dg[j][k] * inv;
      dg[i][j] -= l * lj;  // entries above the diagonal hold values nothing uses
      xb[i][j] -= x * lj;
    }
    __syncthreads();
  }
  if (!below) {
    for (int q = g; q < kn; q += 4) {
      if (i > q && i < kn) mat[static_cast<int64_t>(k0 + q) * sz + k0 + i] = lt[q][i];
      if (i < q) copy[static_cast<int64_t>(k0 + q) * sz + k0 + i] = lt[i][q];
    }
    if (tid < kn) ldiag[k0 + tid] = lt[tid][tid];
    return;
  }
  for (int q = g; q < kPanel; q += 4) {  // a panel with rows below is whole
    if (row0 + i < sz) mat[static_cast<int64_t>(k0 + q) * sz + row0 + i] = xb[i][q] * lt[q][q];
    if (row0 + q < sz) copy[static_cast<int64_t>(row0 + q) * sz + k0 + i] = xb[q][i] * lt[i][i];
  }
}

// Trailing update of panel a.step: tile (ti, tj), ti >= tj, of the rows and columns past the panel.
__global__ __launch_bounds__(kSolveThreads) void fit_chol_update_kernel(const SolveArgs a) {
  const int layer = blockIdx.z, w = a.w;
  const Slots s = slots(a.work, a.w, layer);
  const int r = static_cast<int>(s.job->rank);
  const bool zz = blockIdx.y == 1;
  const int sz = zz ? r : w, k0 = a.step * kPanel, first = k0 + kPanel;
  if (first >= sz) return;
  int ti = 0, rem = blockIdx.x;
  while (rem > ti) rem -= ++ti;  // tile ti (ti + 1) / 2 + tj
  const int i0 = first + ti * 64, j0 = first + rem * 64;
  if (i0 >= sz) return;
  double* mat = zz ? s.y : s.x;
  // L[i][k] is read from the upper triangle, where a panel column is a row
  tile_product(
      kPanel,
      [&](int kk, int x) {
        return i0 + x < sz ? mat[static_cast<int64_t>(k0 + kk) * sz + i0 + x] : 0.0;
      },
      [&](int kk, int x) {
        return j0 + x < sz ? mat[static_cast<int64_t>(k0 + kk) * sz + j0 + x] : 0.0;
      },
      [&](int x, int y, double v) {
        const int i = i0 + x, j = j0 + y;
        if (i < sz && j <= i) mat[static_cast<int64_t>(i) * sz + j] -= v;
      });
}

// ---- triangular solves and outputs --------------------------------------------------------------
// One wave solves (L L^T) x = b for one right-hand side in registers (entry lane + 64 q).  Forward
// L y = b column by column: y_i = b_i / L_ii, then b_j -= L[j][i] y_i for j > i with column i of L read
// as row i of the upper triangle (`lu`, contiguous).  Backward L^T x = y the same way from the bottom:
// x_i = y_i / L_ii, then y_j -= L[i][j] x_i for j < i with row i of L read from the row-major copy
// (`lr`).  The rows are loaded kAhead steps before use, so the chain of steps does not wait on a load
// at each link (28 layers, w = 128: 65 us, 2 layers, w = 1024: 0.59 ms; with the vector in LDS and each row
// loaded when its step came up, 204 us and 4.6 ms).
template <int NQ>
__device__ inline void wave_chol_solve(const double* lu, const double* lr, const double* inv, int sz,
                                       double (&x)[NQ]) {
  constexpr int kAhead = NQ <= 4 ? 4 : 2;
  const int lane = threadIdx.x & 63;
  // Steps run 64 at a time, so the registers a step touches are constants: q >= B going forward, q <= B
  // going back.  Entries past the size read the row's last one; their x is never used.
  auto block = [&](auto b_c, auto fwd_c) {
    constexpr int B = decltype(b_c)::value;
    constexpr bool FWD = decltype(fwd_c)::value != 0;
    constexpr int QA = FWD ? B : 0, QZ = FWD ? NQ : B + 1;
    const int i0 = 64 * B, i1 = sz < i0 + 64 ? sz : i0 + 64;  // steps [i0, i1), a multiple of 16 many
    if (i0 >= sz) return;
    const int first = FWD ? i0 : i1 - 1, dir = FWD ? 1 : -1, steps = i1 - i0;
    const double* m = FWD ? lu : lr;
    double row[kAhead][NQ], dg[kAhead];
    auto load = [&](int t, int u) {
      const int i = first + dir * (t < steps ? t : steps - 1);
      dg[u] = inv[i];
      const double* p = m + static_cast<int64_t>(i) * sz;
#pragma unroll
      for (int q = QA; q < QZ; ++q) {
        const int j = lane + 64 * q;
        row[u][q] = p[j < sz ? j : sz - 1];
      }
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load(u, u);
    for (int t = 0; t < steps; t += kAhead) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int i = first + dir * (t + u);
        const double yi = readlane_f64(x[B], i & 63) * dg[u];
        const double own = lane + i0 == i ? yi : x[B];
        x[B] = (FWD ? lane + i0 > i : lane + i0 < i) ? x[B] - row[u][B] * yi : own;
#pragma unroll
        for (int q = QA; q < QZ; ++q)
          if (q != B) x[q] -= row[u][q] * yi;
        load(t + u + kAhead, u);
      }
    }
  };
  auto all = [&](auto self, auto b_c) {
    constexpr int B = decltype(b_c)::value;
    if constexpr (B < NQ) {
      block(b_c, IntC<1>{});
      self(self, IntC<B + 1>{});
      block(b_c, IntC<0>{});
    }
  };
  all(all, IntC<0>{});
}

// One wave per right-hand side, four per workgroup.  ENC: encoder column m,
// E[:, m] = (A^T A + lam I)^-1 P[0:w, m] -> w_enc[m, :]; else decoder row j,
// F[:, j] = (Z^T Z + lam I)^-1 P[w + j, :]^T -> w_dec[j, :].
template <int NQ, bool ENC>
__global__ __launch_bounds__(kSolveThreads) void fit_out_kernel(const SolveArgs a) {
  const int layer = blockIdx.y, w = a.w, lane = threadIdx.x & 63;
  const Slots s = slots(a.work, a.w, layer);
  const SolveJob jb = *s.job;
  const int r = static_cast<int>(jb.rank);
  const int t = blockIdx.x * (kSolveThreads / 64) + (threadIdx.x >> 6);
  if (t >= (ENC ? r : w)) return;
  const int sz = ENC ? w : r;
  double x[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = lane + 64 * q;
    x[q] = i < sz ? (ENC ? s.m[static_cast<int64_t>(i) * r + t] : s.m[static_cast<int64_t>(w + t) * r + i])
                  : 0.0;
  }
  const double* l = ENC ? s.x : s.y;
  wave_chol_solve<NQ>(l, l + static_cast<int64_t>(sz) * sz, s.ldiag + (ENC ? 0 : w), sz, x);
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = lane + 64 * q;
    if (i < sz) store_out(ENC ? jb.w_enc : jb.w_dec, static_cast<int64_t>(t) * sz + i, x[q], a.bf16 != 0);
  }
}

template <int DH>
hipError_t launch_gram_dh(bool bf16, bool derope, const FitGramParams& p, dim3 grid,
                          hipStream_t stream) {
  if (bf16 && fit_full_gram(true, p.w)) {
    if (!derope) hipLaunchKernelGGL((fit_gram_full_bf16_kernel<DH, false, true>), grid, dim3(256), 0, stream, p);
    else if (p.g % 2 == 0) hipLaunchKernelGGL((fit_gram_full_bf16_kernel<DH, true, true>), grid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((fit_gram_full_bf16_kernel<DH, true, false>), grid, dim3(256), 0, stream, p);
  } else if (bf16) {
    if (!derope) hipLaunchKernelGGL((fit_gram_bf16_kernel<DH, false, true>), grid, dim3(256), 0, stream, p);
    else if (p.g % 2 == 0) hipLaunchKernelGGL((fit_gram_bf16_kernel<DH, true, true>), grid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((fit_gram_bf16_kernel<DH, true, false>), grid, dim3(256), 0, stream, p);
  } else {
    if (derope) hipLaunchKernelGGL((fit_gram_f32_kernel<DH, true>), grid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((fit_gram_f32_kernel<DH, false>), grid, dim3(256), 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace

int64_t fit_upper_tiles(int w) {
  const int64_t nt = 2 * static_cast<int64_t>(w) / kTB;
  return nt * (nt + 1) / 2;
}

bool fit_full_gram(bool bf16, int w) { return bf16 && 2 * w == 2 * kTB; }

int64_t fit_units_per_slice(bool bf16, int w, int n_jobs) {
  return static_cast<int64_t>(n_jobs) * (fit_full_gram(bf16, w) ? 1 : fit_upper_tiles(w));
}

hipError_t launch_fit_gram(bool bf16, const FitGramParams& p, hipStream_t stream) {
  const int64_t units = static_cast<int64_t>(p.n_jobs) * fit_units_per_slice(bf16, p.w, 1) *
                        p.n_slices;
  const dim3 grid(static_cast<unsigned>(units));
  hipError_t e;
  switch (p.head_dim) {
    case 32: e = launch_gram_dh<32>(bf16, p.derope != 0, p, grid, stream); break;
    case 64: e = launch_gram_dh<64>(bf16, p.derope != 0, p, grid, stream); break;
    case 128: e = launch_gram_dh<128>(bf16, p.derope != 0, p, grid, stream); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  const int64_t bx = fit_upper_tiles(p.w) * 16;  // 32 x 32 sub-blocks of every upper tile
  hipLaunchKernelGGL(fit_gram_reduce_kernel, dim3(static_cast<unsigned>(bx), p.n_jobs), dim3(256),
                     0, stream, p);
  return hipGetLastError();
}

hipError_t fit_scratch(double** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static double* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (addr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    addr[dev] = static_cast<double*>(p);
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t launch_fit_solve(const FitSolveParams& p, hipStream_t stream) {
  const int n = 2 * p.w, layers = p.n_jobs;
  int rmax = 0;
  for (int l = 0; l < layers; ++l) rmax = p.jobs[l].rank > rmax ? p.jobs[l].rank : rmax;
  const dim3 block(kSolveThreads), wave(64);
  SolveArgs a{p.work, static_cast<double>(p.n_rows), p.lambda, p.w, 0, p.center, p.bf16};
  hipLaunchKernelGGL(fit_prep_kernel, dim3((n + kSolveRows - 1) / kSolveRows, layers), block, 0,
                     stream, p);
  // steps k0 .. n-3 (a trailing block of n - k0 - 1 <= kTailN rows) in one launch
  const int k0 = n - 1 - kTailN > -1 ? n - 1 - kTailN : -1;
  for (int k = -1; k < k0; ++k) {
    a.step = k;
    const int rows = n - k - 2;
    const bool pair = k >= 0 && (k & 1) != 0;  // k0 is odd: the last launch is a pair's first
    const int write = pair || k == k0 - 1 ? 1 : 0;
    const int scale = rows > 1024 ? 2 : 1;
    const int rpw = (static_cast<int64_t>(rows) * layers > kTridiagNarrow ? 8 : 4) * scale;
    const dim3 grid((rows + rpw - 1) / rpw, layers), threads(kSolveThreads * scale);
#define SCD_FIT_TRIDIAG_ROWS(PRE, ROWS, THREADS)                                                  \
  do {                                                                                           \
    if (pair)                                                                                    \
      hipLaunchKernelGGL((fit_tridiag_kernel<PRE, ROWS, THREADS, true>), grid, threads, 0,       \
                         stream, a, write);                                                      \
    else                                                                                         \
      hipLaunchKernelGGL((fit_tridiag_kernel<PRE, ROWS, THREADS, false>), grid, threads, 0,      \
                         stream, a, write);                                                      \
  } while (0)
#define SCD_FIT_TRIDIAG(PRE, S)                                                                  \
  do {                                                                                           \
    if (rpw == 8 * S) SCD_FIT_TRIDIAG_ROWS(PRE, 8 * S, kSolveThreads * S);                       \
    else SCD_FIT_TRIDIAG_ROWS(PRE, 4 * S, kSolveThreads * S);                                    \
  } while (0)
    if (rows <= 512) SCD_FIT_TRIDIAG(8, 1);
    else if (rows <= 1024) SCD_FIT_TRIDIAG(16, 1);
    else if (rows <= 1536) SCD_FIT_TRIDIAG(24, 2);
    else SCD_FIT_TRIDIAG(32, 2);
#undef SCD_FIT_TRIDIAG
#undef SCD_FIT_TRIDIAG_ROWS
  }
  a.step = k0;
  hipLaunchKernelGGL(fit_tridiag_tail_kernel, dim3(layers), dim3(kTailThreads), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned rt = static_cast<unsigned>((rmax + 63) / 64);
  if (n <= 256) hipLaunchKernelGGL(fit_bisect_kernel<256>, dim3(rmax, layers), wave, 0, stream, a);
  else hipLaunchKernelGGL(fit_bisect_kernel<kMaxN>, dim3(rmax, layers), wave, 0, stream, a);
  if (n <= kInverseLdsN)
    hipLaunchKernelGGL((fit_inverse_lds_kernel<kInverseLdsN, kInverseLdsThreads>),
                       dim3((rmax + kInverseLdsThreads - 1) / kInverseLdsThreads, layers), wave, 0,
                       stream, a);
  else
    hipLaunchKernelGGL((fit_inverse_lds_kernel<kMaxN, 1>), dim3(rmax, layers), wave, 0, stream, a);
  const dim3 back(rmax, layers);
#define SCD_FIT_BACK(NQ)                                                                         \
  do {                                                                                           \
    if (n == 64 * NQ)                                                                            \
      hipLaunchKernelGGL((fit_back_kernel<NQ, false>), back, wave, 0, stream, a);                \
    else                                                                                         \
      hipLaunchKernelGGL((fit_back_kernel<NQ, true>), back, wave, 0, stream, a);                 \
  } while (0)
  if (n <= 256) SCD_FIT_BACK(4);
  else if (n <= 512) SCD_FIT_BACK(8);
  else if (n <= 1024) SCD_FIT_BACK(16);
  else SCD_FIT_BACK(32);
#undef SCD_FIT_BACK
  hipLaunchKernelGGL(fit_project_kernel, dim3(n / 64, rt, layers), block, 0, stream, a);
  const unsigned tw = static_cast<unsigned>(p.w / 64);
  hipLaunchKernelGGL(fit_normal_kernel, dim3(rt * rt > tw * tw ? rt * rt : tw * tw, 2, layers),
                     block, 0, stream, a);
  for (int k = 0; k * kPanel < p.w; ++k) {  // every rank is at most w
    a.step = k;
    const unsigned blocks = static_cast<unsigned>((p.w - k * kPanel + kPanel - 1) / kPanel);
    hipLaunchKernelGGL(fit_chol_panel_kernel, dim3(blocks, 2, layers), block, 0, stream, a);
    if (blocks > 1)
      hipLaunchKernelGGL(fit_chol_update_kernel, dim3((blocks - 1) * blocks / 2, 2, layers), block, 0,
                         stream, a);
  }
  constexpr int kWaves = kSolveThreads / 64;
  const dim3 enc((rmax + kWaves - 1) / kWaves, layers), dec((p.w + kWaves - 1) / kWaves, layers);
#define SCD_FIT_OUT(SZ, GRID, ENC)                                                             \
  if (SZ <= 128) hipLaunchKernelGGL((fit_out_kernel<2, ENC>), GRID, block, 0, stream, a);      \
  else if (SZ <= 256) hipLaunchKernelGGL((fit_out_kernel<4, ENC>), GRID, block, 0, stream, a); \
  else if (SZ <= 512) hipLaunchKernelGGL((fit_out_kernel<8, ENC>), GRID, block, 0, stream, a); \
  else hipLaunchKernelGGL((fit_out_kernel<16, ENC>), GRID, block, 0, stream, a)
  SCD_FIT_OUT(p.w, enc, true);
  SCD_FIT_OUT(rmax, dec, false);
#undef SCD_FIT_OUT
  return hipGetLastError();
}

}  // namespace scd
