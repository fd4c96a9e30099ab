// Tiled projection GEMM for steps and prompts of many rows on gfx950 (fp16
// operands, fp32 accumulation).
//
// y[m][n] = sum_k x[m][k] * W[n][k], the same projections, operand layouts and
// fused epilogues as the weight-streaming kernel (k_gemm.hip), for the row
// counts where re-reading the activations in every wave, and not the weights'
// HBM stream, sets the pace: there each wave loads its own activation tiles
// from L2 and few of them are in flight; here a workgroup keeps a ring of K
// stages of both operands in LDS, filled by global -> LDS loads that need no
// registers, and its waves share every tile.
//   * Both operands are stored in 1 KiB tiles in MFMA lane order
//     (tss_internal.h), so a stage is a linear copy of tiles, each LDS read is
//     one conflict-free 16-byte read per lane, and no swizzle is needed.
//   * A workgroup takes MR x NC tiles of 16 x 16 outputs, its WM x WN waves
//     (MR / WM) x (NC / WN) each.  With the weights as the MFMA's first operand
//     a lane ends with four adjacent columns of one row, so the epilogues run
//     on the accumulators with 8- and 16-byte stores and no pass through LDS.
//   * The ring holds ST stages of KCH chunks (32 columns of K each); a wave
//     waits for its own loads of the stage with a counted wait, and one barrier
//     a stage both publishes the stage and frees the slot that is refilled
//     next, ST - 1 stages ahead.
//   * The next chunk's LDS reads are issued before the MFMAs of the current one.
//   * Column blocks are numbered row block first, in runs per XCD (block ids go
//     to the XCDs round robin), so the row blocks that share weight tiles meet
//     in one L2.
//
// Measured on the 7B shapes: gate/up of 2048 rows 331 us alone (1115 TFLOP/s
// with 16 x 16 tiles; a loop of the same MFMAs and LDS reads without loads or
// barriers runs at 1976), Q/K/V of 1024 rows 118 us in 16 x 12 tiles (130 in 16
// x 16, three quarters of a round), O / down of 1024 rows 53 / 125 us in 8 x 8.
// A prompt of 1024 tokens through four blocks and its first step: 9083 us in
// 64-row steps of k_gemm, 1961 us in one pass.  Steps: step_tiled.
//
// What bounds the shapes of up to 128 rows is the requests a CU keeps in
// flight to L2 and HBM: their time is the weights' at about 22-27 bytes per ns
// and CU plus the activations' at 60, whatever the depth of the ring (6 to 16
// stages), and loading waves of their own or weights and activations in
// rings of different depths change it by less than the runs differ (gate/up
// of 120 rows 44-49 us, Q/K/V 34-37, measured before a step's weights were
// loaded once and nontemporal: 44 and 34 since).
#include "tss_internal.h"

#include <type_traits>

namespace tss {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

// At most N of this wave's vector memory operations outstanding, and all its
// LDS reads done (the slot it has read may be refilled after the barrier).
template <int N>
__device__ __forceinline__ void wait_ring() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ float silu_f(float g) { return g / (1.0f + __expf(-g)); }

// Sum over the four lanes l, l^16, l^32, l^48 (every lane gets it).
__device__ __forceinline__ float sum4(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// (value, index) order of the greedy argmax: larger value first, NaN largest,
// lower index on ties.
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
  const bool nv = __builtin_isnan(v), nb = __builtin_isnan(bv);
  return (nv && !nb) || v > bv || ((v == bv || (nv && nb)) && i < bi);
}

}  // namespace

// PRE: the rows are a run of one sequence's prompt (row r at position and slot
// a.pre_n0 + r); otherwise they are a verification step's rows (a.sp).
template <int MR, int NC, int WM, int WN, int KCH, int ST, int EPI, bool PRE>
__global__ __launch_bounds__(WM* WN * 64, WM * WN <= 4 && ST * (MR + NC) * KCH <= 78 ? 2 : 1) void k_tile(GemmArgs a) {
  constexpr int W = WM * WN, TM = MR / WM, TN = NC / WN;
  constexpr int TT = MR + NC;              // tiles of one chunk
  constexpr int U = TT * KCH;              // KiB of one stage
  constexpr int PT = (TT + W - 1) / W;     // tiles that one wave loads per stage,
  constexpr int PW = PT * KCH;             // in PW loads
  constexpr int ROWS = MR * 16;
  static_assert(MR % WM == 0 && NC % WN == 0 && ST >= 2 && ST * PW < 63, "tile shape");
  static_assert(EPI != EPI_SWIGLU || TN % 2 == 0, "a wave owns whole gate/up pairs");
  static_assert(!PRE || EPI != EPI_RESID || TN == tile_wave_cols(TileShape{MR, NC, 1}), "partial sums of a prompt");
  extern __shared__ __align__(16) uint8_t ring[];  // [ST][U KiB]
  __shared__ float s_scale[ROWS];
  __shared__ int s_seq[EPI == EPI_RESID && !PRE ? ROWS : 1];
  __shared__ int s_pos[EPI == EPI_QKV ? ROWS : 1];   // rotary position
  __shared__ int s_phys[EPI == EPI_QKV ? ROWS : 1];  // pool page * 16 + token of the page

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, r16 = lane & 15, grp = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  const int M = a.M, nkc = a.nkc;
  const int rt_all = (M + 15) >> 4;        // row tiles of the launch
  const int ct_all = a.N >> 4;             // column tiles of the matrix
  const int mblocks = (rt_all + MR - 1) / MR;

  // block id -> (K split, row block, column block)
  const int ks = EPI == EPI_RESID ? a.ksplit : 1;
  const int total = mblocks * ((ct_all + NC - 1) / NC) * ks;
  const int per_xcd = (total + 7) >> 3;
  const int id = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
  if (((int)blockIdx.x >> 3) >= per_xcd || id >= total) return;
  const int mb = id % mblocks, rest = id / mblocks;
  const int split = rest % ks, cb = rest / ks;
  const int rt0 = mb * MR, ct0 = cb * NC;
  const int c_lo = split * nkc / ks, c_hi = (split + 1) * nkc / ks;
  const int n_st = (c_hi - c_lo + KCH - 1) / KCH;

  // This wave loads tiles wave + i * W of a stage, KCH KiB each: the chunks of
  // an activation or weight tile, or one half of the alternating chunks of a
  // gate/up pair (KiB r of a pair: chunk r / 2).  Tiles past the matrix
  // re-read its last tile, whose outputs are not stored.  Where W does not
  // divide the tiles, the last waves load the last tile again, from the caches,
  // in a prompt; in a step, where that fetched nontemporal weights again (7B
  // down of 48 rows 29.5 us, now 21.7), they issue one tile less (`full`) and
  // count their waits by it.
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)ring;
  const unsigned lane16 = lane * 16;
  const uint8_t* src[PT];
  bool pair[PT];   // gate/up weights: which half of the pair
  int half[PT];
  constexpr bool FEWER = !PRE && TT % W != 0;
  const bool full = !FEWER || wave < TT % W;  // this wave loads PT tiles a stage, else PT - 1
  const bool w_nt = !PRE && a.w_nt;
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int tl = min(wave + i * W, TT - 1);
    pair[i] = EPI == EPI_SWIGLU && tl >= MR;
    half[i] = (tl - MR) & 1;
    if (tl < MR)
      src[i] = (const uint8_t*)a.x + (size_t)min(rt0 + tl, rt_all - 1) * nkc * kTileBytes;
    else if (EPI == EPI_SWIGLU)
      src[i] = a.w + (size_t)min((ct0 + tl - MR) >> 1, (ct_all >> 1) - 1) * nkc * 2 * kTileBytes;
    else
      src[i] = a.w + (size_t)min(ct0 + tl - MR, ct_all - 1) * nkc * kTileBytes;
  }
  // Loads of stage st into slot; chunks past the range re-read its last one.
  // A step reads each weight tile once; where the model's weights do not fit
  // the memory-side cache they are nontemporal, as in k_gemm, and do not push
  // the K/V of the contexts out of it between steps (tile_weights_nt).  A
  // prompt's row blocks share the weights through L2.
  auto issue = [&](int st, int slot) {
    const int c0 = c_lo + st * KCH;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      if (FEWER && i == PT - 1 && !full) break;
      const int tl = min(wave + i * W, TT - 1);
      const unsigned dst = lds0 + (unsigned)(slot * U + tl * KCH) * 1024u;
      auto load = [&](auto nt) {
#pragma unroll
        for (int s = 0; s < KCH; ++s) {
          const int r = half[i] * KCH + s;
          const int kib = pair[i] ? 2 * min(c0 + (r >> 1), c_hi - 1) + (r & 1) : min(c0 + s, c_hi - 1);
          dma_kib<nt>(src[i], lane16 + (unsigned)kib * 1024u, dst + s * 1024u);
        }
      };
      if (!PRE && w_nt && tl >= MR)
        load(std::true_type{});
      else
        load(std::false_type{});
    }
  };
  // Row data of the epilogue and the partial sums of the RMSNorm row scales
  // are requested before the ring's first loads, behind which they would
  // otherwise complete: the threads of a row take 16-byte groups of its parts
  // in turn, up to SQ at a time.
  constexpr int TH = W * 64;
  constexpr int TPR = TH >= 4 * ROWS ? 4 : (TH >= 2 * ROWS ? 2 : 1);
  constexpr int SQ = 32;
  constexpr bool ROWDATA = EPI == EPI_QKV || (EPI == EPI_RESID && !PRE);
  static_assert(TH >= ROWS, "a thread per row");
  const int rl = threadIdx.x / TPR, rsub = threadIdx.x % TPR;
  const int rrow = min(rt0 * 16 + rl, M - 1);
  const bool ss_vec = EPI != EPI_RESID && a.ss_nparts % (4 * TPR) == 0 && a.ss_stride % 4 == 0;
  const int ss_groups = ss_vec ? a.ss_nparts / (4 * TPR) : 0;  // per thread
  const float* ss_row = EPI != EPI_RESID ? a.ss_in + (size_t)rrow * a.ss_stride : nullptr;
  float4 sq[EPI != EPI_RESID ? SQ : 1];
  if constexpr (EPI != EPI_RESID) {
    if (rl < ROWS) {
#pragma unroll
      for (int i = 0; i < SQ; ++i)
        if (i < ss_groups) sq[i] = *(const float4*)(ss_row + (i * TPR + rsub) * 4);
    }
  }
  int my_seq = 0, my_pos = 0, my_phys = 0;
  if (ROWDATA && (int)threadIdx.x < ROWS) {
    const int row = min(rt0 * 16 + (int)threadIdx.x, M - 1);
    if constexpr (PRE) {
      my_pos = a.pre_n0 + row;
      my_phys = a.page_table[my_pos >> 4] * 16 + (my_pos & 15);
    } else if constexpr (EPI == EPI_QKV) {
      my_pos = a.rows->pos[row];
      my_phys = a.rows->phys[row];
    } else {
      my_seq = a.n_seqs == 1 ? 0 : a.sp->row_seq[row];
    }
  }
#pragma unroll
  for (int st = 0; st < ST; ++st)
    if (st < n_st) issue(st, st);
  if (ROWDATA && (int)threadIdx.x < ROWS) {
    if constexpr (EPI == EPI_QKV) {
      s_pos[threadIdx.x] = my_pos;
      s_phys[threadIdx.x] = my_phys;
    } else {
      s_seq[threadIdx.x] = my_seq;
    }
  }
  if constexpr (EPI != EPI_RESID) {
    if (rl < ROWS) {
      float s = 0.f;
      if (ss_vec) {
#pragma unroll
        for (int i = 0; i < SQ; ++i)
          if (i < ss_groups) s += (sq[i].x + sq[i].y) + (sq[i].z + sq[i].w);
        for (int i = SQ; i < ss_groups; ++i) {
          const float4 v = *(const float4*)(ss_row + (i * TPR + rsub) * 4);
          s += (v.x + v.y) + (v.z + v.w);
        }
      } else {
        for (int q = rsub; q < a.ss_nparts; q += TPR) s += ss_row[q];
      }
#pragma unroll
      for (int off = 1; off < TPR; off <<= 1) s += __shfl_xor(s, off);
      if (rsub == 0) s_scale[rl] = rsqrtf(s / (float)a.norm_dim + a.eps);
    }
  }

  f32x4 acc[TM][TN];
#pragma unroll
  for (int t = 0; t < TM; ++t)
#pragma unroll
    for (int n = 0; n < TN; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Operand tiles of chunk c of the stage in `slot`, and their products.
  struct Frag {
    f16x8 x[TM], w[TN];
  };
  auto read = [&](Frag& f, int slot, int c) {
    const uint8_t* base = ring + (size_t)slot * U * 1024 + lane16;
#pragma unroll
    for (int n = 0; n < TN; ++n) {
      const int ct = wn * TN + n;
      const int at = EPI == EPI_SWIGLU ? (ct >> 1) * 2 * KCH + c * 2 + (ct & 1) : ct * KCH + c;
      f.w[n] = *(const f16x8*)(base + (MR * KCH + at) * 1024);
    }
#pragma unroll
    for (int t = 0; t < TM; ++t) f.x[t] = *(const f16x8*)(base + ((wm * TM + t) * KCH + c) * 1024);
  };
  auto mma = [&](const Frag& f) {
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int n = 0; n < TN; ++n) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f.w[n], f.x[t], acc[t][n], 0, 0, 0);
  };
  // Stage k + 1 is here once this wave's loads of it are done (stages up to
  // k + ST - 1 have been requested) and the others' are (the barrier), which
  // also says that every wave has read stage k out of `slot`.
  auto arrive = [&](int k) {
    if (k + ST - 1 < n_st) {
      if (full)
        wait_ring<(ST - 2) * PW>();
      else
        wait_ring<(ST - 2) * (PW - KCH)>();
    } else {
      wait_ring<0>();
    }
    barrier();
  };
  auto next = [&](int slot) { return slot + 1 == ST ? 0 : slot + 1; };

  // Each chunk's tiles are read one chunk ahead of their products, so the LDS
  // reads, the refill of the slot just freed and the wait of the next stage
  // overlap the MFMAs.
  Frag f0, f1;
  arrive(-1);
  read(f0, 0, 0);
  int slot = 0;
  if constexpr (KCH == 1) {
    for (int k = 0; k < n_st; k += 2) {
      int s1 = next(slot);
      if (k + 1 < n_st) {
        arrive(k);
        read(f1, s1, 0);
        if (k + ST < n_st) issue(k + ST, slot);
      }
      mma(f0);
      slot = next(s1);
      if (k + 2 < n_st) {
        arrive(k + 1);
        read(f0, slot, 0);
        if (k + 1 + ST < n_st) issue(k + 1 + ST, s1);
      }
      if (k + 1 < n_st) mma(f1);
    }
  } else {
    static_assert(KCH <= 2, "one or two chunks a stage");
    for (int k = 0; k < n_st; ++k) {
      const bool two = c_lo + k * KCH + 1 < c_hi;
      read(f1, slot, 1);
      mma(f0);
      const int s1 = next(slot);
      if (k + 1 < n_st) {
        arrive(k);
        read(f0, s1, 0);
        if (k + ST < n_st) issue(k + ST, slot);
      }
      slot = s1;
      if (two) mma(f1);
    }
  }

  // acc[t][n][v]: row (rt0 + wm TM + t) 16 + r16, column (ct0 + wn TN + n) 16 + 4 grp + v
  const int row_w = (rt0 + wm * TM) * 16 + r16;  // row of t = 0
  const int ct_w = ct0 + wn * TN;                // column tile of n = 0
  auto row_on = [&](int row) {
    return PRE || (((row < 64 ? a.row_on[0] : a.row_on[1]) >> (row & 63)) & 1ull);
  };

  if constexpr (EPI == EPI_RESID) {
    // h and the next norm's gain of one row tile; with few tiles per wave they
    // are requested before the merge of a K split
    const int N = a.N;
    constexpr bool EARLY = TM * TN <= 4;
    float4 h4[EARLY ? TM : 1][TN], g4[EARLY ? TM : 1][TN];
    auto operands = [&](int t, float4 (&h)[TN], float4 (&g)[TN]) {
      const int row = min(row_w + t * 16, M - 1);
      const float* gain = PRE || a.n_seqs == 1 ? a.g_next[0] : a.g_next[s_seq[row_w + t * 16 - rt0 * 16]];
#pragma unroll
      for (int n = 0; n < TN; ++n) {
        const int col = min(ct_w + n, ct_all - 1) * 16 + grp * 4;
        h[n] = *(const float4*)(a.h + (size_t)row * N + col);
        g[n] = *(const float4*)(gain + col);
      }
    };
    if constexpr (EARLY) {
#pragma unroll
      for (int t = 0; t < TM; ++t) operands(t, h4[t], g4[t]);
    }
    if (ks > 1) {
      // K split: publish the partial tiles (agent-scope stores, visible to
      // every XCD once acknowledged), count the arrival, and let the last of
      // the ks workgroups add them in split order.
      __shared__ int s_last;
      constexpr int kScopeAgent = 16;  // cache-policy operand: sc1 (agent scope)
      const int out = cb * mblocks + mb;
      const size_t slot_bytes = (size_t)MR * NC * 1024;
      const __amdgpu_buffer_rsrc_t pres = __builtin_amdgcn_make_buffer_rsrc(
          (uint8_t*)a.kpart + (size_t)out * ks * slot_bytes, (short)0, (int)(ks * slot_bytes), 0x00020000);
      const int off0 = wave * TM * TN * 1024 + lane * 16;
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int n = 0; n < TN; ++n)
          __builtin_amdgcn_raw_buffer_store_b128(acc[t][n], pres,
                                                 (int)(split * slot_bytes) + off0 + (t * TN + n) * 1024, 0,
                                                 kScopeAgent);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(a.kcount + out, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ks - 1;
      __syncthreads();
      if (!s_last) return;
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int n = 0; n < TN; ++n) {
          f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
          f32x4 v[kMaxKSplit];
#pragma unroll
          for (int k = 0; k < kMaxKSplit; ++k)
            if (k < ks && k != split)
              v[k] = __builtin_amdgcn_raw_buffer_load_b128(pres, (int)(k * slot_bytes) + off0 + (t * TN + n) * 1024, 0,
                                                           kScopeAgent);
#pragma unroll
          for (int k = 0; k < kMaxKSplit; ++k)
            if (k < ks) s += k == split ? acc[t][n] : v[k];
          acc[t][n] = s;
        }
      if (threadIdx.x == 0) a.kcount[out] = 0;
    }
    // residual add, the next norm's input h * gain, partial sums of h^2: one
    // per 16 columns in a step (the format every norm of a step reads), one
    // per wave (TN tiles) in a prompt
    constexpr int PN = PRE ? TN : 1;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int row = row_w + t * 16;
      const bool on = row < M && row_on(row);
      const int tt = EARLY ? t : 0;
      if constexpr (!EARLY) operands(t, h4[0], g4[0]);
      float ss = 0.f;
#pragma unroll
      for (int n = 0; n < TN; ++n) {
        const int col = (ct_w + n) * 16 + grp * 4;
        const bool st = on && ct_w + n < ct_all;
        const f32x4 y = acc[t][n];
        const float4 hn = make_float4(h4[tt][n].x + y[0], h4[tt][n].y + y[1], h4[tt][n].z + y[2], h4[tt][n].w + y[3]);
        if (st) {
          *(float4*)(a.h + (size_t)row * N + col) = hn;
          store_act4<_Float16>(a.xn, a.xn_plane, act_index<_Float16>(row, col, N),
                               make_float4(hn.x * g4[tt][n].x, hn.y * g4[tt][n].y, hn.z * g4[tt][n].z, hn.w * g4[tt][n].w));
          ss += (hn.x * hn.x + hn.y * hn.y) + (hn.z * hn.z + hn.w * hn.w);
        }
        if ((n + 1) % PN == 0) {
          const float s = sum4(ss);
          if (on && ct_w + n + 1 - PN < ct_all && grp == 0) a.ss_out[(size_t)row * a.ss_stride + (ct_w + n) / PN] = s;
          ss = 0.f;
        }
      }
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    const int F = a.N >> 1;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int row = row_w + t * 16;
      const float r = s_scale[row - rt0 * 16];
      if (row >= M) continue;
#pragma unroll
      for (int n = 0; n < TN; n += 2) {
        if (ct_w + n >= ct_all) break;
        const f32x4 g = acc[t][n] * r, u = acc[t][n + 1] * r;
        store_act4<_Float16>(a.act, a.act_plane, act_index<_Float16>(row, ((ct_w + n) >> 1) * 16 + grp * 4, F),
                             make_float4(silu_f(g[0]) * u[0], silu_f(g[1]) * u[1], silu_f(g[2]) * u[2],
                                         silu_f(g[3]) * u[3]));
      }
    }
  } else if constexpr (EPI == EPI_QKV) {
    const int HD = a.head_dim, d = a.d, half = HD >> 1;
    const int d16 = d >> 4, hd16 = HD >> 4;
#pragma unroll
    for (int n = 0; n < TN; ++n) {
      const int tile = ct_w + n;
      if (tile >= ct_all) break;
      const int sec = tile / d16, ts = tile % d16, head = ts / hd16, tt = ts % hd16;
      // the lane's four columns: adjacent dims of one half of the rotary pairs
      const int j = 8 * tt + (grp & 1) * 4;            // rotary index
      const int dim = (grp < 2 ? 0 : half) + j;
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        const int row = row_w + t * 16, rl = row - rt0 * 16;
        f32x4 y = acc[t][n] * s_scale[rl];
        if (sec < 2) {
          const float4* cs = (const float4*)(a.rope + (size_t)s_pos[rl] * half + j);
          const float4 a0 = cs[0], a1 = cs[1];         // (cos, sin) x 4
          f32x4 p;
#pragma unroll
          for (int v = 0; v < 4; ++v) p[v] = __shfl_xor(y[v], 32);
          if (grp < 2) {
            y = f32x4{y[0] * a0.x - p[0] * a0.y, y[1] * a0.z - p[1] * a0.w, y[2] * a1.x - p[2] * a1.y,
                      y[3] * a1.z - p[3] * a1.w};
          } else {
            y = f32x4{y[0] * a0.x + p[0] * a0.y, y[1] * a0.z + p[1] * a0.w, y[2] * a1.x + p[2] * a1.y,
                      y[3] * a1.z + p[3] * a1.w};
          }
        }
        if (row >= M) continue;
        if (sec == 0) {
          *(f32x4*)(a.q + (size_t)row * d + head * HD + dim) = y;
        } else if (row_on(row)) {
          const int tin = s_phys[rl] & 15;
          _Float16* blk =
              (_Float16*)a.kv_pages +
              ((((size_t)a.layer * a.n_pages_pool + (s_phys[rl] >> 4)) * 2 + (sec - 1)) * a.n_heads + head) * (16 * (size_t)HD);
          if (sec == 1) {
            typedef _Float16 h4 __attribute__((ext_vector_type(4)));
            *(h4*)(blk + tin * HD + dim) = h4{(_Float16)y[0], (_Float16)y[1], (_Float16)y[2], (_Float16)y[3]};
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) blk[(tin >> 2) * HD * 4 + (dim + v) * 4 + (tin & 3)] = (_Float16)y[v];
          }
        }
      }
    }
  } else {
    const int N = a.N;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int row = row_w + t * 16;
      const float r = s_scale[row - rt0 * 16];
#pragma unroll
      for (int n = 0; n < TN; ++n) {
        const int tile = ct_w + n;
        const f32x4 y = acc[t][n] * r;
        const int c0 = tile * 16 + grp * 4;
        const bool st = row < M && tile < ct_all;
        if (st) *(f32x4*)(a.logits + (size_t)row * N + c0) = y;
        // one (max, argmax) per 16 columns
        float bv = y[0];
        int bi = c0;
#pragma unroll
        for (int v = 1; v < 4; ++v)
          if (better(y[v], c0 + v, bv, bi)) {
            bv = y[v];
            bi = c0 + v;
          }
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
          const float ov = __shfl_xor(bv, off);
          const int oi = __shfl_xor(bi, off);
          if (better(ov, oi, bv, bi)) {
            bv = ov;
            bi = oi;
          }
        }
        if (st && grp == 0) {
          a.am_val[(size_t)row * a.am_stride + tile] = bv;
          a.am_idx[(size_t)row * a.am_stride + tile] = bi;
        }
      }
    }
  }
}

template <int MR, int NC, int KCH, int ST>
constexpr size_t tile_lds() { return (size_t)ST * (MR + NC) * KCH * 1024; }

template <int MR, int NC, int WM, int WN, int KCH, int ST, int EPI, bool PRE>
static hipError_t tile_attr() {
  return hipFuncSetAttribute((const void*)k_tile<MR, NC, WM, WN, KCH, ST, EPI, PRE>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)tile_lds<MR, NC, KCH, ST>());
}

template <int MR, int NC, int WM, int WN, int KCH, int ST, int EPI, bool PRE>
static hipError_t tile_go(const GemmArgs& a, hipStream_t s) {
  const int mblocks = ((a.M + 15) / 16 + MR - 1) / MR, cblocks = (a.N / 16 + NC - 1) / NC;
  const int total = mblocks * cblocks * a.ksplit;
  TSS_LAUNCH((k_tile<MR, NC, WM, WN, KCH, ST, EPI, PRE>), dim3((total + 7) / 8 * 8), dim3(WM * WN * 64),
             (tile_lds<MR, NC, KCH, ST>()), s, a);
  return hipGetLastError();
}

// Block shapes: MR, NC, waves WM x WN, KCH, ST.  Prompts: the large shapes and
// those of up to 128 rows; steps: exact row tiles for the residual projections
// (a K split's partial tiles grow with the rows), 6 or 8 for the others.
#define TSS_TILES_LARGE(F, E, P)  \
  F(16, 16, 2, 4, 2, 2, E, P)     \
  F(16, 8, 4, 2, 2, 3, E, P)      \
  F(8, 8, 2, 4, 2, 4, E, P)
#define TSS_TILES_QKV(F, E, P)    \
  F(6, 3, 2, 3, 2, 6, E, P)       \
  F(6, 4, 2, 2, 2, 6, E, P)       \
  F(6, 6, 2, 3, 2, 5, E, P)       \
  F(8, 3, 2, 3, 2, 6, E, P)       \
  F(8, 4, 2, 2, 2, 5, E, P)       \
  F(8, 6, 2, 3, 2, 4, E, P)
#define TSS_TILES_GATEUP(F, E, P) \
  F(6, 6, 2, 3, 2, 5, E, P)       \
  F(6, 8, 2, 4, 2, 5, E, P)       \
  F(6, 10, 2, 5, 2, 4, E, P)      \
  F(8, 6, 2, 3, 2, 4, E, P)       \
  F(8, 10, 2, 5, 2, 4, E, P)
#define TSS_TILES_RESID(F, E, P)  \
  F(6, 4, 3, 2, 2, 6, E, P)       \
  F(8, 4, 4, 2, 2, 6, E, P)

#define TSS_TRY(MR, NC, WM, WN, KCH, ST, E, P) \
  if (t.mr == MR && t.nc == NC) return tile_go<MR, NC, WM, WN, KCH, ST, E, P>(a, s);
#define TSS_ATTR(MR, NC, WM, WN, KCH, ST, E, P) \
  if (e == hipSuccess) e = tile_attr<MR, NC, WM, WN, KCH, ST, E, P>();

#define TSS_PROMPT_SHAPES(F)             \
  TSS_TILES_LARGE(F, EPI_QKV, true)      \
  F(16, 12, 2, 4, 1, 5, EPI_QKV, true)   \
  TSS_TILES_QKV(F, EPI_QKV, true)        \
  TSS_TILES_LARGE(F, EPI_SWIGLU, true)   \
  F(16, 12, 4, 2, 1, 5, EPI_SWIGLU, true) \
  TSS_TILES_GATEUP(F, EPI_SWIGLU, true)  \
  TSS_TILES_LARGE(F, EPI_RESID, true)    \
  TSS_TILES_RESID(F, EPI_RESID, true)
#define TSS_STEP_SHAPES(F)               \
  TSS_TILES_QKV(F, EPI_QKV, false)       \
  TSS_TILES_GATEUP(F, EPI_SWIGLU, false) \
  F(8, 8, 2, 4, 2, 4, EPI_SWIGLU, false) \
  F(6, 2, 3, 2, 2, 6, EPI_QKV, false)    \
  F(8, 2, 4, 2, 2, 6, EPI_QKV, false)    \
  F(6, 4, 3, 2, 2, 6, EPI_SWIGLU, false) \
  F(8, 4, 4, 2, 2, 6, EPI_SWIGLU, false) \
  TSS_TILES_RESID(F, EPI_RESID, false)   \
  F(2, 4, 2, 4, 2, 8, EPI_RESID, false)  \
  F(3, 4, 3, 2, 2, 8, EPI_RESID, false)  \
  F(4, 4, 4, 2, 2, 8, EPI_RESID, false)  \
  F(5, 4, 5, 2, 2, 6, EPI_RESID, false)  \
  F(7, 4, 7, 2, 2, 6, EPI_RESID, false)  \
  F(6, 8, 2, 4, 2, 5, EPI_LOGITS, false) \
  F(8, 8, 2, 4, 2, 4, EPI_LOGITS, false)

hipError_t init_tile_attributes() {
  hipError_t e = hipSuccess;
  TSS_PROMPT_SHAPES(TSS_ATTR)
  TSS_STEP_SHAPES(TSS_ATTR)
  return e;
}

static bool split_ok(int epi, const TileShape& t, const GemmArgs& a) {
  return a.ksplit == t.ks && t.ks >= 1 && t.ks <= kMaxKSplit &&
         (t.ks == 1 || (epi == EPI_RESID && a.nkc >= t.ks && a.kpart && a.kcount));
}

#define TSS_TRY_EPI(MR, NC, WM, WN, KCH, ST, E, P) \
  if (epi == E) TSS_TRY(MR, NC, WM, WN, KCH, ST, E, P)
hipError_t launch_tile_prompt(int epi, const TileShape& t, const GemmArgs& a, hipStream_t s) {
  if (!split_ok(epi, t, a) || a.M < 1 || a.M > kPromptRows || a.nkc < 1 || a.N % 16) return hipErrorInvalidValue;
  TSS_PROMPT_SHAPES(TSS_TRY_EPI)
  return hipErrorInvalidValue;
}

hipError_t launch_tile_step(int epi, const TileShape& t, const GemmArgs& a, hipStream_t s) {
  if (!split_ok(epi, t, a) || a.M < 1 || a.M > kMaxRows || a.M > t.mr * 16 || a.nkc < 1 || a.N % 16)
    return hipErrorInvalidValue;
  TSS_STEP_SHAPES(TSS_TRY_EPI)
  return hipErrorInvalidValue;
}

}  // namespace tss
