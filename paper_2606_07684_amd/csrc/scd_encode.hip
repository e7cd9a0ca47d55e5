// Producer encode (Section 4.3.2, Eq. encode_z_kv; Section 4.4.1) on the bf16 path for gfx950:
//   Z_K = (rows(deRoPE(K)) - mu_K) W_enc,K^T,   Z_V = (rows(V) - mu_V) W_enc,V^T,   Z_H = H W_enc,H^T
// The step is bound by HBM reads of the K/V/H inputs (the codes are r/w of that traffic).
//
// A workgroup of 4 waves owns 128 input rows of one layer-branch and produces up to 128 code
// columns for them (RB*32; a rank above 128 takes two workgroups per row tile, so every instance
// keeps two waves per SIMD).  Every wave streams its 32 rows straight from HBM into registers, 128 input
// columns (one chunk) at a time, one chunk ahead of use.  With deRoPE each lane loads the same
// 8 columns of both halves of a head, so every rotation pair meets in one lane; the rotated values
// are rounded to bf16 and used directly as the B operand of v_mfma_f32_32x32x16_bf16 (without
// deRoPE the loaded bf16 values are the operand as they are).  Each lane keeps the cosines and
// sines of its row in registers for all heads.  The encoder weight chunk (all code rows x 128
// columns, rows permuted so each lane ends with 16 consecutive code columns of one row) is
// double-buffered in LDS and shared by the four waves.  Both operands visit the columns of a chunk
// in the same order, so the contraction is unchanged.
//
// The offset is folded into the product: (X - 1 mu^T) E^T = X E^T - 1 (E mu)^T.  With an offset a
// workgroup takes 127 rows and mu as its 128th, so E mu falls out of the same MFMAs (an extra product
// per k-step with mu broadcast, as before, was a fifth of the MFMAs and a third of the LDS reads); the
// workgroup shares it through LDS and every lane subtracts it from its fp32 accumulators, so the
// offset is never rounded.  Rank 256, 32,768 tokens: 2263 -> 2145 us; rank 128, 8192 tokens (with the
// Patch codes): 367 -> 358 us.
#include "scd_device.h"

namespace scd {
namespace {

using namespace dev;

constexpr int kThreads = 256;
constexpr int kChunk = 128;          // input columns per chunk
constexpr int kLdcPad = kChunk + 8;  // padded LDS row of a weight chunk (elements)

// Column (within a chunk) that lane half h supplies to MFMA k-step s (0..7).  With deRoPE, even
// steps take the first half of a head and odd steps the matching second half:
//   d_h = 128: step s -> offset o = 16*(s/2), half (s&1);  d_h = 64: two heads per chunk.
template <int DH>
__device__ constexpr int chunk_col(int s, int h, bool derope) {
  if (!derope) return 16 * s + 8 * h;
  constexpr int steps_per_head = DH / 16;
  const int hc = s / steps_per_head, sw = s % steps_per_head;
  return hc * DH + (sw & 1) * (DH / 2) + 16 * (sw >> 1) + 8 * h;
}

// RB = code blocks of 32 (rank <= 32*RB); DH = head_dim (64 or 128, used with deRoPE);
// DEROPE = key jobs; MU = every job of the launch has an offset.
template <int RB, int DH, bool DEROPE, bool MU, int DEPTH>
__global__ __launch_bounds__(kThreads) void encode_bf16_kernel(GemmParams p) {
  // With an offset a workgroup takes 127 rows and mu itself as its last one, which is not rotated: a
  // rotation by zero would turn an infinite entry's partner into NaN
  constexpr int kRows = MU ? kEncodeRowsMu : kEncodeRows;
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  // Weight chunk rows: padded (DEPTH 1) or swizzled without padding (DEPTH 2, where every wave must
  // issue a fixed number of copies so its waits can be counted).
  constexpr bool kSwz = DEPTH == 2;
  constexpr int kLdc = kSwz ? kChunk : kLdcPad;
  uint16_t* Es = lds;                               // [2][RB*32][kLdc]
  float* emu = reinterpret_cast<float*>(lds + 2 * RB * 32 * kLdc);  // [RB*32]: E mu

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int h = lane >> 5;

  const int unit = xcd_remap(blockIdx.x, gridDim.x);
  const GemmJob job = p.jobs[job_of(p, unit)];
  // A rank above RB*32 takes two workgroups per row tile, units 2i and 2i + 1, each producing
  // RB*32 (or the remaining) code columns of the same rows: consecutive units run on one XCD at
  // about the same time, so the second read of the rows mostly hits L2.
  const int n_split = (job.n + RB * 32 - 1) / (RB * 32);  // 1 or 2
  const int local = unit - job.tile_begin;
  const int code0 = (local % n_split) * RB * 32;
  const int R = job.n - code0 < RB * 32 ? job.n - code0 : RB * 32;  // code columns here
  const int K = job.k;
  const int64_t M = p.m;
  const int64_t row = static_cast<int64_t>(local / n_split) * kRows + wave * 32 + (lane & 31);
  const bool mu_row = MU && wave * 32 + (lane & 31) == kRows;
  const bool valid = row < M && !mu_row;
  constexpr bool derope = DEROPE;
  const uint16_t* X = static_cast<const uint16_t*>(job.a);
  const uint16_t* E = static_cast<const uint16_t*>(job.b) + static_cast<int64_t>(code0) * K;
  const uint16_t* mu = static_cast<const uint16_t*>(job.vec);
  const int nchunks = K / kChunk;

  // weight chunk c -> LDS buffer b, asynchronously; code rows beyond R read row 0 and only feed
  // accumulator blocks that are never stored.  Swizzled: RB*32 rows x 16 chunks of 16 bytes, chunk
  // q of row rho at q ^ (rho & 7), exactly 2*RB copies per wave.  Padded: rows of 17 slots, the
  // pad slot masked off.
  constexpr int kEDma = RB * 32 * (kChunk / 8) / kThreads;
  auto stage_weights = [&](int c, int b) {
    uint16_t* dst = Es + b * RB * 32 * kLdc;
    if constexpr (kSwz) {
#pragma unroll
      for (int j = 0; j < kEDma; ++j) {
        const int slot = (4 * j + wave) * 64 + lane;
        const int rho = slot >> 4, q = (slot & 15) ^ (rho & 7);
        const int r = row_of_lds(rho);
        __builtin_amdgcn_global_load_lds(
            E + static_cast<int64_t>(r < R ? r : 0) * K + c * kChunk + 8 * q,
            (lds_void_t)(dst + 8 * ((4 * j + wave) * 64)), 16, 0, 0);
      }
    } else {
      dma_rows(dst, RB * 32, kChunk / 8, kLdc / 8, wave, 4, lane, [&](int rho) {
        const int r = row_of_lds(rho);
        return E + static_cast<int64_t>(r < R ? r : 0) * K + c * kChunk;
      });
    }
  };
  // MFMA A fragment of weight block b at chunk column col (a multiple of 8) for this lane's row
  auto efrag = [&](const uint16_t* eb, int b, int col) {
    const int q = kSwz ? ((col >> 3) ^ (lane & 7)) : (col >> 3);
    return *reinterpret_cast<const bf16x8*>(eb + b * 32 * kLdc + 8 * q);
  };

  // this lane's rotation factors for every pair index it touches: i = 16*o + 8*h + e
  constexpr int kNo = DH / 32;  // 16-wide offsets per half head
  float cs_c[kNo][8], cs_s[kNo][8];
  if (derope) {
    const float2* cs_row = p.rope + static_cast<int64_t>(valid ? row_position(p, row) : 0) * (DH / 2);
#pragma unroll
    for (int o = 0; o < kNo; ++o)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float2 v = cs_row[16 * o + 8 * h + e];
        cs_c[o][e] = v.x;
        cs_s[o][e] = v.y;
      }
  }

  const uint16_t* xrow = mu_row ? mu : X + (valid ? row : 0) * K;
  // rows past the end read row 0 (always in bounds); their codes are never stored
  auto load_x = [&](int c, uint4* dst) {
#pragma unroll
    for (int s = 0; s < 8; ++s)
      dst[s] = *reinterpret_cast<const uint4*>(xrow + c * kChunk + chunk_col<DH>(s, h, derope));
  };

  f32x16 acc[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[b][e] = 0.f;

  // One chunk's MFMAs for input registers x (8 loads of this lane's row) against weight buffer buf.
  // The weight fragments of k-step s + 1 are read under the MFMAs of step s, so each LDS read has a
  // step to land instead of stalling the MFMA that needs it.  B operands come in (first half, second
  // half) pairs: deRoPE in fp32 and one bf16 rounding (keys), or the loaded values themselves.  Both
  // operands visit the chunk's columns in the same order, so the contraction is unchanged.
  auto compute_chunk = [&](int buf, const uint4* x) {
    const uint16_t* eb = Es + buf * RB * 32 * kLdc + (lane & 31) * kLdc;
    bf16x8 f[2][RB];
    auto read_step = [&](int s) {
      const int col = chunk_col<DH>(s, h, derope);
#pragma unroll
      for (int b = 0; b < RB; ++b) f[s & 1][b] = efrag(eb, b, col);
    };
    read_step(0);
    bf16x8 bu, bv;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if ((s & 1) == 0) {
        if constexpr (DEROPE) {
          float u[8], v[8];
          unpack8(x[s], u);
          unpack8(x[s + 1], v);
          constexpr int spH = DH / 16;
          const int o = (s % spH) >> 1;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float cc = cs_c[o][e], sn = cs_s[o][e];
            const float a = u[e], b = v[e];
            u[e] = a * cc + b * sn;
            v[e] = b * cc - a * sn;
          }
          bu = __builtin_bit_cast(bf16x8, mu_row ? x[s] : pack8(u));
          bv = __builtin_bit_cast(bf16x8, mu_row ? x[s + 1] : pack8(v));
        } else {
          bu = __builtin_bit_cast(bf16x8, x[s]);
          bv = __builtin_bit_cast(bf16x8, x[s + 1]);
        }
      }
      const bf16x8 bx = (s & 1) ? bv : bu;
      __builtin_amdgcn_sched_barrier(0);
      if (s + 1 < 8) read_step(s + 1);
#pragma unroll
      for (int b = 0; b < RB; ++b)
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s & 1][b], bx, acc[b], 0, 0, 0);
      if (s + 1 < 8) {
#pragma unroll
        for (int b = 0; b < RB; ++b) {
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  if constexpr (DEPTH == 1) {
  uint4 xc[8], xn[8];
  stage_weights(0, 0);
  load_x(0, xc);
  wait_vmem();
  lds_barrier();

  for (int c = 0; c < nchunks; ++c) {
    const int buf = c & 1;
    if (c + 1 < nchunks) {
      stage_weights(c + 1, buf ^ 1);
      load_x(c + 1, xn);
    }
    compute_chunk(buf, xc);
    wait_vmem();
    lds_barrier();
#pragma unroll
    for (int s = 0; s < 8; ++s) xc[s] = xn[s];
  }

  } else {
  // inputs two chunks ahead in a ring of three register sets; the chunk loop is unrolled by three
  // so every set keeps its registers (no copies of registers whose loads are in flight)
  constexpr int kWait8 = 8 | (0x7 << 4) | (0xF << 8);  // at most the 8 input loads of chunk c + 2
  uint4 x0[8], x1[8], x2[8];
  stage_weights(0, 0);
  load_x(0, x0);
  load_x(nchunks > 1 ? 1 : 0, x1);
  __builtin_amdgcn_s_waitcnt(kWait8);
  lds_barrier();
  const int last = nchunks - 1;
  auto step = [&](int c, uint4 (&xcur)[8], uint4 (&xfar)[8]) {
    const int buf = c & 1;
    // weights of chunk c + 1 and inputs of chunk c + 2 (past the end: in-bounds re-loads that are
    // never used, so every step issues the same loads and the compiler's counter waits can leave
    // the far inputs in flight)
    stage_weights(c + 1 < last ? c + 1 : last, buf ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    load_x(c + 2 < last ? c + 2 : last, xfar);
    __builtin_amdgcn_sched_barrier(0);
    if (c < nchunks) compute_chunk(buf, xcur);
    // chunk c + 1's weights and inputs have landed once only chunk c + 2's 8 input loads are
    // pending; the barrier makes that true for every wave and retires this chunk's LDS reads.  The
    // scheduling fences keep each step's loads on their side of the count.
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kWait8);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  // chunks run in threes; steps past the last chunk only keep the load pattern uniform
  for (int c = 0; c < nchunks; c += 3) {
    step(c, x0, x2);
    step(c + 1, x1, x0);
    step(c + 2, x2, x1);
  }
  wait_vmem();
  }
  if constexpr (MU) {
    // the last wave's last lanes of both halves hold E mu
    if (mu_row) {
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) emu[32 * b + 16 * h + e] = acc[b][e];
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[b][e] -= emu[32 * b + 16 * h + e];
  }
  if (!valid) return;
  // lane holds, for block b, code columns code0 + 32*b + 16*h + (0..15) of its row
  uint16_t* Zo = static_cast<uint16_t*>(job.c) + row * job.n + code0;
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int c0 = 32 * b + 16 * h;
    if (c0 >= R) continue;
    float y[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) y[e] = acc[b][e];
    uint4* d = reinterpret_cast<uint4*>(Zo + c0);
    d[0] = pack8(y);
    d[1] = pack8(y + 8);
  }
}

// ---- keys and values on resident weights ------------------------------------------------------------
// The same product with no weight traffic in the loop: a workgroup of 8 waves keeps its code block's
// whole encoder in LDS and every wave streams 32-row tiles on its own, inputs one or two chunks ahead
// across tiles, with no barrier until the share enters the next layer.  Fragments are read from LDS one
// k-step ahead and the next pair's deRoPE runs between MFMAs.  Bound by the mixed read/write stream of HBM
// and, above rank 64, by the products: w = 512, rank 128, 32,768 tokens x 24 layers 491 us, 4.1 TB/s (545 on
// the streamed kernel before; a plain copy moves 4.7 TB/s).  E mu is computed
// once per share and layer (chunks dealt to the waves) and subtracted from the accumulators.
constexpr int kCus = 256;
constexpr int kResWaves = 8, kResThreads = 64 * kResWaves;

// LDS of the resident kernel: RB * 32 code rows x K columns of the encoder, then E mu (partial sums of
// the waves, and their sum).
constexpr size_t resident_lds(int rb, int k) {
  return static_cast<size_t>(rb) * 32 * k * 2 + static_cast<size_t>(kResWaves + 1) * rb * 32 * 4;
}

template <int RB, int DH, bool DEROPE, bool MU>
__global__ __launch_bounds__(kResThreads, 2) void encode_kv_bf16_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  __shared__ LdsBatch lbatch;
  constexpr int CB = RB * 32;                    // codes of this workgroup
  const int K = p.jobs[0].k, nchunks = K / kChunk;
  uint16_t* Ws = lds;                            // [nchunks][CB][kChunk], 16-byte pieces swizzled
  float* part = reinterpret_cast<float*>(lds + static_cast<size_t>(CB) * K);  // [kResWaves][CB]
  float* emu = part + kResWaves * CB;            // [CB]

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t M = p.m;

  // workgroup -> (share of the wave tiles, code block); code block fastest, so that the workgroups
  // that read the same rows run on one XCD at the same time
  const int u = xcd_remap(blockIdx.x, gridDim.x);
  const int n = p.jobs[0].n;
  const int n_split = (n + CB - 1) / CB, n_share = gridDim.x / n_split;
  const int share = u / n_split, code0 = (u % n_split) * CB;
  const int R = n - code0 < CB ? n - code0 : CB;
  const int64_t per_job = (M + 31) / 32;         // wave tiles of 32 rows
  int64_t first, last;
  if (p.reserved > 0) {                          // whole jobs, `reserved` shares each
    const int j = share / p.reserved, q = share % p.reserved;
    first = j * per_job + per_job * q / p.reserved;
    last = j * per_job + per_job * (q + 1) / p.reserved;
  } else {                                       // one balanced list over all jobs
    const int64_t total = per_job * p.n_jobs;
    first = total * share / n_share;
    last = total * (share + 1) / n_share;
  }
  const bool lds_batch = p.n_seqs <= kMaxLdsSeqs;
  if (DEROPE && lds_batch) stage_batch(p, lbatch, tid, kResThreads);

  constexpr int kNo = DEROPE ? DH / 32 : 1;      // 16-wide offsets per half head
  // Two sets of input registers (loads one chunk ahead) where three and the factors are more than 256
  // registers: with three, rank 128 keys spilled 61 (w = 512, 24 layers: 4000 tokens 102 us, two sets 78;
  // 32,768 tokens 635, two sets 502).
  constexpr bool kTwoSets = DEROPE && (DH == 128 ? RB >= 3 : RB == 4 && MU);
  for (int64_t t = first; t < last;) {
    const int j = static_cast<int>(t / per_job);
    const int64_t t1 = last < (j + 1) * per_job ? last : (j + 1) * per_job;
    const int64_t job0 = j * per_job;
    const GemmJob& job = p.jobs[j];
    const uint16_t* X = static_cast<const uint16_t*>(job.a);
    const uint16_t* E = static_cast<const uint16_t*>(job.b) + static_cast<int64_t>(code0) * K;
    uint16_t* Z = static_cast<uint16_t*>(job.c);

    // Loads run two chunks (or one, kTwoSets) ahead of use, across the wave's tiles (t + wave, t + wave
    // + 8, ...).  Past the last tile they re-read the wave's first one; rows past the end read row 0.
    int64_t lt = t + wave;  // tile and chunk of the next load
    int lc = 0;
    const uint16_t* xrow;
    auto set_row = [&]() {
      const int64_t row = (lt < t1 ? lt : t) * 32 - job0 * 32 + (lane & 31);
      xrow = X + (row < M ? row : 0) * K;
    };
    set_row();
    auto load_x = [&](uint4 (&x)[8]) {
#pragma unroll
      for (int s = 0; s < 8; ++s)
        x[s] = *reinterpret_cast<const uint4*>(xrow + lc * kChunk + chunk_col<DH>(s, h, DEROPE));
      if (++lc == nchunks) {
        lc = 0;
        lt += kResWaves;
        set_row();
      }
    };
    uint4 x0[8], x1[8], x2[8];
    if (t != first) lds_barrier();  // every wave is done with the previous job's weights
    load_x(x0);
    if constexpr (!kTwoSets) load_x(x1);
    // the encoder -> LDS: chunk c of code row rho (permuted so that a lane ends with 16 consecutive
    // codes of one row), piece q at q ^ (rho & 7); rows past R repeat row 0 and are never stored
    for (int s = wave * 64; s < nchunks * CB * 16; s += kResThreads) {
      const int slot = s + lane, c = slot / (CB * 16), rho = (slot >> 4) % CB;
      const int q = (slot & 15) ^ (rho & 7), r = row_of_lds(rho);
      __builtin_amdgcn_global_load_lds(
          E + static_cast<int64_t>(r < R ? r : 0) * K + c * kChunk + 8 * q,
          (lds_void_t)(Ws + 8 * s), 16, 0, 0);
    }
    wait_vmem();
    lds_barrier();

    auto wfrag = [&](int c, int b, int col) {
      return *reinterpret_cast<const bf16x8*>(Ws + (c * CB + b * 32 + (lane & 31)) * kChunk +
                                              8 * ((col >> 3) ^ (lane & 7)));
    };
    if constexpr (MU) {
      // E mu: mu as the B operand in every column, chunks dealt out to the waves, partial sums added
      // in wave order
      const uint16_t* mu = static_cast<const uint16_t*>(job.vec);
      f32x16 am[RB];
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) am[b][e] = 0.f;
      for (int c = wave; c < nchunks; c += kResWaves) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const bf16x8 m = *reinterpret_cast<const bf16x8*>(mu + c * kChunk + 16 * s + 8 * h);
#pragma unroll
          for (int b = 0; b < RB; ++b)
            am[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfrag(c, b, 16 * s + 8 * h), m, am[b],
                                                            0, 0, 0);
        }
      }
      if ((lane & 31) == 0) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
          for (int e = 0; e < 16; ++e) part[wave * CB + 32 * b + 16 * h + e] = am[b][e];
      }
      lds_barrier();
      if (tid < CB) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kResWaves; ++w) v += part[w * CB + tid];
        emu[tid] = v;
      }
      lds_barrier();
    }

    // rotation factors of the row this lane works on, for every pair index it touches
    float cs_c[kNo][8], cs_s[kNo][8];
    auto load_rope = [&](int64_t tile) {
      if constexpr (DEROPE) {
        const int64_t row = (tile - job0) * 32 + (lane & 31);
        const int pos = row < M ? (lds_batch ? row_position_lds(p, lbatch, row) : row_position(p, row)) : 0;
        int off = 8 * h;  // opaque: hoisted out of the loop, the address took two registers too many
        asm volatile("" : "+v"(off));
        const float2* cs_row = p.rope + static_cast<int64_t>(pos) * (DH / 2) + off;
#pragma unroll
        for (int o = 0; o < kNo; ++o)
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const float4 v = *reinterpret_cast<const float4*>(cs_row + 16 * o + e);
            cs_c[o][e] = v.x;
            cs_s[o][e] = v.y;
            cs_c[o][e + 1] = v.z;
            cs_s[o][e + 1] = v.w;
          }
      }
    };
    f32x16 acc[RB];
    auto clear = [&]() {
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[b][e] = 0.f;
    };
    int64_t ct = t + wave;  // tile and chunk of the next product
    int cc = 0;
    clear();
    if (ct < t1) load_rope(ct);
    auto step = [&](uint4 (&x)[8], uint4 (&far)[8]) {
      load_x(far);
      __builtin_amdgcn_sched_barrier(0);
      // the B operand of steps sp and sp + 1: deRoPE in fp32 and one rounding, or the loaded values
      auto operand = [&](int sp, bf16x8& bu, bf16x8& bv) {
        if constexpr (DEROPE) {
          float a[8], b[8];
          unpack8(x[sp], a);
          unpack8(x[sp + 1], b);
          constexpr int spH = DH / 16;
          const int o = (sp % spH) >> 1;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float c = cs_c[o][e], sn = cs_s[o][e];
            const float uu = a[e], vv = b[e];
            a[e] = uu * c + vv * sn;
            b[e] = vv * c - uu * sn;
          }
          bu = __builtin_bit_cast(bf16x8, pack8(a));
          bv = __builtin_bit_cast(bf16x8, pack8(b));
        } else {
          bu = __builtin_bit_cast(bf16x8, x[sp]);
          bv = __builtin_bit_cast(bf16x8, x[sp + 1]);
        }
      };
      // Each step's fragments are read during the step before (read right before its MFMAs, an LDS
      // read's whole latency stands in front of every MFMA), and the next pair's deRoPE runs between
      // the MFMAs of the pair's second step.
      bf16x8 f[2][RB], bu[2], bv[2];
#pragma unroll
      for (int b = 0; b < RB; ++b) f[0][b] = wfrag(cc, b, chunk_col<DH>(0, h, DEROPE));
      operand(0, bu[0], bv[0]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        if (s + 1 < 8) {
#pragma unroll
          for (int b = 0; b < RB; ++b)
            f[(s + 1) & 1][b] = wfrag(cc, b, chunk_col<DH>(s + 1, h, DEROPE));
        }
        if ((s & 1) && s + 1 < 8) operand(s + 1, bu[((s + 1) >> 1) & 1], bv[((s + 1) >> 1) & 1]);
        const bf16x8 bx = (s & 1) ? bv[(s >> 1) & 1] : bu[(s >> 1) & 1];
#pragma unroll
        for (int b = 0; b < RB; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s & 1][b], bx, acc[b], 0, 0, 0);
        if (s + 1 < 8) __builtin_amdgcn_sched_group_barrier(0x100, RB, 0);
        if constexpr (DEROPE) {
          if ((s & 1) && s + 1 < 8) {
#pragma unroll
            for (int b = 0; b < RB; ++b) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x002, 64 / RB, 0);
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (++cc < nchunks) return;
      cc = 0;
      // the tile is complete: lane holds, for block b, codes code0 + 32 b + 16 h + (0..15) of its row
      const int64_t row = (ct - job0) * 32 + (lane & 31);
      ct += kResWaves;
      if (ct < t1) load_rope(ct);
      if (row < M) {
        uint16_t* zo = Z + row * n + code0;
#pragma unroll
        for (int b = 0; b < RB; ++b) {
          const int c0 = 32 * b + 16 * h;
          if (c0 >= R) continue;
          float y[16];
#pragma unroll
          for (int e = 0; e < 16; ++e) y[e] = MU ? acc[b][e] - emu[c0 + e] : acc[b][e];
          uint4* d = reinterpret_cast<uint4*>(zo + c0);
          d[0] = pack8(y);
          d[1] = pack8(y + 8);
        }
      }
      clear();
    };
    while (ct < t1) {
      if constexpr (kTwoSets) {
        step(x0, x1);
        if (ct >= t1) break;
        step(x1, x0);
      } else {
        step(x0, x2);
        if (ct >= t1) break;
        step(x1, x0);
        if (ct >= t1) break;
        step(x2, x1);
      }
    }
    t = t1;
  }
}

template <int RB>
hipError_t launch_resident(bool derope, bool mu, const GemmParams& p, int grid, hipStream_t stream) {
  const size_t lds = resident_lds(RB, p.jobs[0].k);
#define SCD_RESIDENT(DH, DEROPE, MU)                                                             \
  hipLaunchKernelGGL((encode_kv_bf16_kernel<RB, DH, DEROPE, MU>), dim3(grid), dim3(kResThreads), \
                     lds, stream, p)
  if (!derope) {
    if (mu) SCD_RESIDENT(128, false, true);
    else SCD_RESIDENT(128, false, false);
  } else if (p.head_dim == 128) {
    if (mu) SCD_RESIDENT(128, true, true);
    else SCD_RESIDENT(128, true, false);
  } else {
    if (mu) SCD_RESIDENT(64, true, true);
    else SCD_RESIDENT(64, true, false);
  }
#undef SCD_RESIDENT
  return hipGetLastError();
}

template <int RB, bool DEROPE, bool MU>
hipError_t launch_rb(int head_dim, const GemmParams& p, size_t lds, hipStream_t stream) {
  // long rows without deRoPE or offset (the H branch) prefetch two chunks ahead
  if constexpr (!DEROPE && !MU) {
    if (p.jobs[0].k >= 2048) {
      if (head_dim == 128)
        hipLaunchKernelGGL((encode_bf16_kernel<RB, 128, DEROPE, MU, 2>), dim3(p.total_tiles),
                           dim3(kThreads), lds, stream, p);
      else
        hipLaunchKernelGGL((encode_bf16_kernel<RB, 64, DEROPE, MU, 2>), dim3(p.total_tiles),
                           dim3(kThreads), lds, stream, p);
      return hipGetLastError();
    }
  }
  if (head_dim == 128)
    hipLaunchKernelGGL((encode_bf16_kernel<RB, 128, DEROPE, MU, 1>), dim3(p.total_tiles),
                       dim3(kThreads), lds, stream, p);
  else
    hipLaunchKernelGGL((encode_bf16_kernel<RB, 64, DEROPE, MU, 1>), dim3(p.total_tiles),
                       dim3(kThreads), lds, stream, p);
  return hipGetLastError();
}


template <int RB>
hipError_t launch_kind(bool derope, bool mu, int head_dim, const GemmParams& p, size_t lds,
                       hipStream_t stream) {
  if (derope)
    return mu ? launch_rb<RB, true, true>(head_dim, p, lds, stream)
              : launch_rb<RB, true, false>(head_dim, p, lds, stream);
  return mu ? launch_rb<RB, false, true>(head_dim, p, lds, stream)
            : launch_rb<RB, false, false>(head_dim, p, lds, stream);
}

}  // namespace

// Code blocks of 32 the kernel instance for `max_rank` computes (a template parameter); ranks
// above 128 take two workgroups of 4 blocks per row tile.
int encode_code_blocks(int max_rank) { return max_rank <= 64 ? 2 : 4; }

size_t encode_bf16_lds_bytes(int code_blocks, bool mu) {
  return static_cast<size_t>(2) * code_blocks * 32 * kLdcPad * 2 +
         (mu ? static_cast<size_t>(code_blocks) * 32 * 4 : 0);
}

// Code blocks of 32 per workgroup of the resident kernel.
static int resident_blocks(int k, int rank) {
  return rank <= 32 ? 1 : rank <= 64 || k > 512 ? 2 : rank <= 96 ? 3 : 4;
}

// Where one workgroup's LDS holds the encoder of every code the rows are read once, but a workgroup takes the
// whole CU and starts with its encoder.  So the kernel pays where the streamed kernel's chain of weight copies
// is what counts (a launch of few 32-row tiles a wave, of 256 x 8 waves) and where its products are (ranks
// above 64, long launches); in between, and for few codes, the streamed kernel's several workgroups per CU
// keep more loads in flight, above all on operands that are in no cache.  Keys and values, us streamed /
// resident, then the same on operands in no cache (in brackets: tiles a wave of one launch):
//   w = 1024, rank 64, 14 layers: 1000 tokens (0.22) 42 / 34, 56 / 51; 2000 (0.43) 43 / 42, 67 / 76; 16,384
//   (3.5) 239 / 244, 282 / 299
//   w = 512, 24 layers: rank 64, 1000 tokens (0.38) 32 / 30, 46 / 46; 4000 (1.5) 60 / 64, 105 / 112; 20,000
//   (7.3) 268 / 275, 297 / 317; rank 128, 4000 tokens 80 / 73, 118 / 123; 8192 (3) 159 / 143, 184 / 178;
//   20,000 329 / 314, 348 / 350
//   w = 256, 24 layers, rank 128: 4000 tokens (1.5) 51 / 52, 73 / 83; 16,384 (6) 173 / 160, 192 / 195
//   w = 128 (8 heads' shared basis), 16 layers: rank 64, 100 tokens (0.2) 17 / 19, 22 / 24; 1000 (2) 32 / 34,
//   48 / 55; 8192 (16) 208 / 199, 227 / 232; rank 32, 8192 tokens 176 / 155, 193 / 192; rank 128 286 / 268,
//   303 / 291
// Split over workgroups the rows are read once per 64 codes, which loses for large launches (w = 1024, rank
// 128, 8192 tokens: 315 / 330) and still wins while the launch is one tile per wave and bound by latency
// (rank 128, 40 tokens 49 / 29, 333 tokens 57 / 35).
bool encode_resident(int k, int rank, int64_t rows, int64_t n_jobs) {
  const int rb = resident_blocks(k, rank);
  if (resident_lds(rb, k) + sizeof(LdsBatch) > 160 * 1024) return false;
  const int n_split = (rank + 32 * rb - 1) / (32 * rb);
  const int64_t per_job = (rows + 31) / 32, waves = kCus * kResWaves, tiles = per_job * n_jobs;
  if (n_split > 1) return (per_job + kResWaves - 1) / kResWaves * n_jobs * n_split <= kCus;
  if (k == 128) return tiles >= 8 * waves;
  return 8 * tiles <= 3 * waves || (rank > 64 && (k >= 512 || tiles >= 2 * waves));
}

hipError_t launch_encode_kv_bf16(GemmParams p, hipStream_t stream) {
  if (p.m <= 0 || p.n_jobs < 1) return hipSuccess;
  const int k = p.jobs[0].k, n = p.jobs[0].n;
  const bool derope = (p.jobs[0].flags & kDeropeIn) != 0;
  const bool mu = p.jobs[0].vec != nullptr;
  for (int i = 0; i < p.n_jobs; ++i) {
    const GemmJob& j = p.jobs[i];
    if (j.k != k || j.n != n || ((j.flags & kDeropeIn) != 0) != derope || (j.vec != nullptr) != mu)
      return hipErrorInvalidValue;
  }
  const int rb = resident_blocks(k, n);
  if (resident_lds(rb, k) + sizeof(LdsBatch) > 160 * 1024) return hipErrorInvalidValue;
  const int n_split = (n + 32 * rb - 1) / (32 * rb);
  const int64_t shares = kCus / n_split > 0 ? kCus / n_split : 1;
  const int64_t per_job = (p.m + 31) / 32, wgs = (per_job + kResWaves - 1) / kResWaves;
  // a launch of at most one tile per wave: whole jobs, spread over as many workgroups as there are
  int64_t parts = 0;
  if (wgs * p.n_jobs <= shares) {
    parts = shares / p.n_jobs < per_job ? shares / p.n_jobs : per_job;
  }
  p.reserved = static_cast<int32_t>(parts);
  const int grid = static_cast<int>((parts > 0 ? parts * p.n_jobs : shares) * n_split);
  switch (rb) {
    case 1: return launch_resident<1>(derope, mu, p, grid, stream);
    case 2: return launch_resident<2>(derope, mu, p, grid, stream);
    case 3: return launch_resident<3>(derope, mu, p, grid, stream);
    default: return launch_resident<4>(derope, mu, p, grid, stream);
  }
}

hipError_t launch_encode_bf16(const GemmParams& p, hipStream_t stream) {
  if (p.total_tiles <= 0) return hipSuccess;
  // every job of a launch has the same width, the same deRoPE flag and an offset either on every
  // job or on none
  const int k = p.jobs[0].k;
  const bool derope = (p.jobs[0].flags & kDeropeIn) != 0;
  const bool mu = (p.jobs[0].flags & kVecIn) != 0 && p.jobs[0].vec != nullptr;
  int max_r = 0;
  for (int i = 0; i < p.n_jobs; ++i) {
    const GemmJob& j = p.jobs[i];
    if (j.k != k || ((j.flags & kDeropeIn) != 0) != derope ||
        (((j.flags & kVecIn) != 0 && j.vec != nullptr) != mu))
      return hipErrorInvalidValue;
    max_r = j.n > max_r ? j.n : max_r;
  }
  const int rb = encode_code_blocks(max_r);
  const size_t lds = encode_bf16_lds_bytes(rb, mu);
  if (rb == 2) return launch_kind<2>(derope, mu, p.head_dim, p, lds, stream);
  return launch_kind<4>(derope, mu, p.head_dim, p, lds, stream);
}

}  // namespace scd
