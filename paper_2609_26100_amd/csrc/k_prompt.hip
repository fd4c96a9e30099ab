// Embedding and causal attention of a prefill pass (bf16 mode, gfx950).
//
// A pass takes up to 2048 prompt tokens of one sequence through the decoder at
// once (the projections are k_tile's).  Token r sits at position and KV slot
// n0 + r and sees every slot up to its own; its K/V, like those of the context
// before it, are read back from the paged cache that the Q/K/V projection has
// just filled.
#include "tss_internal.h"

namespace tss {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// One workgroup per token: h = E[tok], the first norm's input h * gain, and
// the sums of h^2 per 16 columns.  A thread takes four adjacent columns, so a
// wave's residual stores are one KiB in a row (with 16 columns a thread they
// were 64 bytes apart: 512 tokens of the 7B shape 17 -> 10.8 us).
__global__ __launch_bounds__(256) void k_prompt_embed(PromptEmbedArgs a) {
  const int m = a.row0 + blockIdx.x, d = a.d;
  if (m == 0) {
    for (int i = threadIdx.x; i < kPromptCounters; i += 256) a.counters[i] = 0;
    if (threadIdx.x == 0) a.attn_split[2 * kAttnMaxItems] = 0;
  }
  const _Float16* row = (const _Float16*)a.embed + (size_t)a.tok[blockIdx.x] * d;
  for (int k = threadIdx.x * 4; k < d; k += 1024) {  // d is a multiple of 16, so a part's four lanes stay together
    const f16x4 e = *(const f16x4*)(row + k);
    const float4 g = *(const float4*)(a.gain + k);
    const float4 v = make_float4((float)e[0], (float)e[1], (float)e[2], (float)e[3]);
    *(float4*)(a.h + (size_t)m * d + k) = v;
    store_act4<_Float16>(a.xn, 0, act_index<_Float16>(m, k, d),
                         make_float4(v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w));
    float ss = (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
    ss += __shfl_xor(ss, 1);
    ss += __shfl_xor(ss, 2);
    if ((threadIdx.x & 3) == 0) a.ss_out[(size_t)m * a.ss_stride + (k >> 4)] = ss;
  }
}

// Causal attention, one workgroup per (head, 128 rows): four waves of two
// 16-row tiles walk the pages of 0 .. the last row's slot together, four pages
// (64 tokens) a step, staged through an LDS ring by global -> LDS loads (one
// page per wave and step, two steps in flight).
//   * S = K Q^T puts tokens on the MFMA rows and query rows on its columns, so
//     a lane holds 16 scores of one query row per step and the softmax needs
//     one exchange over the four lanes of that row for the maximum only (the
//     sums are kept per lane and added at the end).
//   * O^T = V^T P^T takes the scores' layout as its second operand without
//     moving them, two pages per 32-deep MFMA, and leaves each lane with
//     outputs of its own query row: rescaling needs no exchange, and a lane's
//     eight adjacent dimensions are one 16-byte store.
//   * K chunk c covers dims 32 c .. 32 c + 31 (16 tokens x 64 bytes of a page),
//     V chunk i dims 32 i .. 32 i + 31 of four token groups (4 x 256 bytes):
//     each is one KiB load, read back from LDS lane by lane in order.
// Row blocks are numbered from the last one (the longest walk) down.
constexpr int kPaWaves = 4, kPaTiles = 2, kPaPages = 4, kPaStages = 2;
constexpr int kPaRows = kPaWaves * kPaTiles * 16;
static_assert(kPromptRows <= kAttnMaxItems * kPaRows, "one report item per row block");
template <int HD>
constexpr size_t pa_lds() { return (size_t)kPaStages * kPaPages * HD * 64; }

template <int HD>
__global__ __launch_bounds__(kPaWaves * 64, 2) void k_prompt_attn(PromptAttnArgs a) {
  constexpr int NK = HD / 32;              // KiB of a K (or V) page block
  constexpr int PW = 2 * NK;               // loads of one wave per step: one page
  constexpr int STAGE = kPaPages * 2 * NK * 1024;
  extern __shared__ __align__(16) uint8_t ring[];
  const int head = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, grp = lane >> 4;
  const int rb = (int)(gridDim.y - 1 - blockIdx.y) * kPaRows;  // first row of the block
  const int M = a.M, n0 = a.n0;
  const int last = min(rb + kPaRows, M) - 1;                   // last row of the block
  const int n_pages = ((n0 + last) >> 4) + 1;
  const int n_st = (n_pages + kPaPages - 1) / kPaPages;
  if (head == 0 && threadIdx.x == 0) {  // the split this launch took (inspection)
    a.split_out[rb / kPaRows] = 1;
    a.split_out[kAttnMaxItems + rb / kPaRows] = last + 1 - rb;
    if (rb == 0) a.split_out[2 * kAttnMaxItems] = (int)gridDim.y;
  }
  const int wrow = rb + wave * kPaTiles * 16;                  // first row of the wave
  // steps that some row of the wave sees (none for a wave past the last row)
  const int my_st = wrow < M ? (((n0 + min(wrow + kPaTiles * 16, M) - 1) >> 4) / kPaPages) + 1 : 0;

  // this wave's page of step st: page st * 4 + wave (past the end: the last page)
  const size_t blk = 16 * (size_t)HD;
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)ring;
  const unsigned koff = (unsigned)(r16 * HD * 2 + grp * 16);          // + c * 64
  const unsigned voff = (unsigned)(grp * HD * 8 + r16 * 16);          // + i * 256
  int ids = 0;
  auto load_ids = [&](int st) {  // ids of the wave's pages of steps st .. st + 63, one per lane
    ids = a.page_table[min((st + lane) * kPaPages + wave, n_pages - 1)];
  };
  auto issue = [&](int st) {
    const int phys = __builtin_amdgcn_readlane(ids, st & 63);
    const uint8_t* kb = a.kv_pages + ((((size_t)a.layer * a.n_pages_pool + phys) * 2) * a.n_heads + head) * blk * 2;
    const uint8_t* vb = kb + (size_t)a.n_heads * blk * 2;
    const unsigned dst = lds0 + (unsigned)((st % kPaStages) * STAGE + wave * 2 * NK * 1024);
#pragma unroll
    for (int c = 0; c < NK; ++c) dma_kib(kb, koff + c * 64u, dst + c * 1024u);
#pragma unroll
    for (int c = 0; c < NK; ++c) dma_kib(vb, voff + c * 256u, dst + (NK + c) * 1024u);
  };

  // q tiles: lane (row r16, group grp) holds dims 32 c + 8 grp .. + 7 of its row
  f16x8 q[kPaTiles][NK];
#pragma unroll
  for (int t = 0; t < kPaTiles; ++t) {
    const float* qr = a.q + (size_t)min(wrow + t * 16 + r16, M - 1) * a.d + head * HD + grp * 8;
#pragma unroll
    for (int c = 0; c < NK; ++c) {
      const float4 x = *(const float4*)(qr + c * 32), y = *(const float4*)(qr + c * 32 + 4);
      q[t][c] = f16x8{(_Float16)x.x, (_Float16)x.y, (_Float16)x.z, (_Float16)x.w,
                      (_Float16)y.x, (_Float16)y.y, (_Float16)y.z, (_Float16)y.w};
    }
  }
  load_ids(0);
  f32x4 O[kPaTiles][2 * NK];  // [2 i + j]: dims 32 i + 8 grp + 2 v + j
  float m_run[kPaTiles], l_run[kPaTiles];
#pragma unroll
  for (int t = 0; t < kPaTiles; ++t) {
    m_run[t] = -1e30f;
    l_run[t] = 0.f;
#pragma unroll
    for (int n = 0; n < 2 * NK; ++n) O[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  issue(0);
  for (int st = 0; st < n_st; ++st) {
    if (st + 1 < n_st) {
      if (((st + 1) & 63) == 0) load_ids(st + 1);
      issue(st + 1);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PW) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();  // every wave's page of step st has landed
    asm volatile("" ::: "memory");
    if (st < my_st) {
      const uint8_t* base = ring + (st % kPaStages) * STAGE + lane * 16;
      const int tok0 = st * kPaPages * 16 + grp * 4;  // slot of page 0's v = 0
      f16x8 P[kPaTiles][2];
#pragma unroll
      for (int t = 0; t < kPaTiles; ++t) {
        f32x4 S[kPaPages];
#pragma unroll
        for (int p = 0; p < kPaPages; ++p) {
          S[p] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < NK; ++c)
            S[p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(*(const f16x8*)(base + (p * 2 * NK + c) * 1024), q[t][c],
                                                          S[p], 0, 0, 0);
        }
        // slots past the row's own are hidden; only the steps that reach past
        // the tile's first row hold any (uniform)
        const int pos = n0 + wrow + t * 16;
        if ((st + 1) * kPaPages * 16 > pos + 1) {
#pragma unroll
          for (int p = 0; p < kPaPages; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              S[p][v] = tok0 + p * 16 + v > pos + r16 ? -INFINITY : S[p][v];  // a select, no branch
        }
        float mx = -INFINITY;
#pragma unroll
        for (int p = 0; p < kPaPages; ++p)
#pragma unroll
          for (int v = 0; v < 4; ++v) mx = fmaxf(mx, S[p][v]);
        mx = fmaxf(m_run[t], mx * a.scale_log2);
        {
          const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
          mx = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
          const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
          mx = fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
        }
        const float alpha = __builtin_amdgcn_exp2f(m_run[t] - mx);
        m_run[t] = mx;
        float l = 0.f;
#pragma unroll
        for (int p = 0; p < kPaPages; ++p)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float e = __builtin_amdgcn_exp2f(S[p][v] * a.scale_log2 - mx);
            l += e;
            P[t][p >> 1][(p & 1) * 4 + v] = (_Float16)e;
          }
        l_run[t] = l_run[t] * alpha + l;
        // most steps raise no row's maximum (uniform branch)
        if (__any(alpha != 1.f)) {
#pragma unroll
          for (int n = 0; n < 2 * NK; ++n) O[t][n] *= alpha;
        }
      }
      // two pages per MFMA: k = 8 grp + 4 b + u is token 4 grp + u of page 2 h + b
#pragma unroll
      for (int h = 0; h < kPaPages / 2; ++h)
#pragma unroll
        for (int i = 0; i < NK; ++i) {
          const uint4 va = *(const uint4*)(base + (4 * h * NK + NK + i) * 1024);
          const uint4 vb = *(const uint4*)(base + ((4 * h + 2) * NK + NK + i) * 1024);
          const f16x8 v0 = __builtin_bit_cast(f16x8, uint4{va.x, va.y, vb.x, vb.y});
          const f16x8 v1 = __builtin_bit_cast(f16x8, uint4{va.z, va.w, vb.z, vb.w});
#pragma unroll
          for (int t = 0; t < kPaTiles; ++t) {
            O[t][2 * i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v0, P[t][h], O[t][2 * i], 0, 0, 0);
            O[t][2 * i + 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v1, P[t][h], O[t][2 * i + 1], 0, 0, 0);
          }
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // step st has been read: its slot may be refilled
    asm volatile("" ::: "memory");
  }

#pragma unroll
  for (int t = 0; t < kPaTiles; ++t) {
    const int row = wrow + t * 16 + r16;
    float l = l_run[t];
    {
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(l), __float_as_uint(l), false, false);
      l = __uint_as_float(r[0]) + __uint_as_float(r[1]);
      const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
      l = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    }
    if (row >= M) continue;
    const float inv = 1.f / l;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      f16x8 o;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        o[2 * v] = (_Float16)(O[t][2 * i][v] * inv);
        o[2 * v + 1] = (_Float16)(O[t][2 * i + 1][v] * inv);
      }
      *(f16x8*)((_Float16*)a.o + act_index<_Float16>(row, head * HD + 32 * i + 8 * grp, a.d)) = o;
    }
  }
}

hipError_t init_prompt_attributes() {
  hipError_t e = hipFuncSetAttribute((const void*)k_prompt_attn<128>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)pa_lds<128>());
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)k_prompt_attn<64>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)pa_lds<64>());
  return e;
}

hipError_t launch_prompt_embed(const PromptEmbedArgs& a, int rows, hipStream_t s) {
  if (rows < 1 || rows > kPromptToks) return hipErrorInvalidValue;
  TSS_LAUNCH(k_prompt_embed, dim3(rows), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_prompt_attn(int head_dim, const PromptAttnArgs& a, hipStream_t s) {
  if (a.M < 1 || a.M > kPromptRows) return hipErrorInvalidValue;
  const dim3 grid(a.n_heads, (a.M + kPaRows - 1) / kPaRows), block(kPaWaves * 64);
  if (head_dim == 128)
    TSS_LAUNCH(k_prompt_attn<128>, grid, block, pa_lds<128>(), s, a);
  else
    TSS_LAUNCH(k_prompt_attn<64>, grid, block, pa_lds<64>(), s, a);
  return hipGetLastError();
}

}  // namespace tss
