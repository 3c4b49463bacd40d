// Joint space-time flash attention over the tokens of one request
// (softmax(Q K^T / sqrt(64)) V per head, with an online softmax over key
// blocks), the dominant step of the recovery network.
//
// Each wave owns 32 queries.  Scores are computed transposed, S^T = K Q^T,
// so that the 32x32 MFMA accumulator puts one query per lane (lanes l and
// l+32 hold disjoint halves of the keys): the running max, the row sum and
// the rescale of the output stay lane-local, with one cross-half exchange
// (v_permlane32_swap) per key block.  The output is also accumulated
// transposed, O^T = V^T P^T, so the probabilities feed the MFMA straight
// from the score registers; V is stored transposed ([head][dim][token]) by
// the QKV epilogue for that.  Q arrives pre-scaled by log2(e)/8, so
// probabilities are exp2(s - m).
//
// The final division by the row sum makes the result independent of the
// max subtracted before exp2, so any max that keeps the probabilities finite
// will do.  The first block sets it; after that (BF16) the score products
// accumulate onto a register block holding -max, so they come out already
// shifted and the softmax is a bare exp2 per score.  BF16 rows first run a
// pass that never changes that max and takes no block max at all; if some
// row sum of the workgroup reaches 2^64 (or is not finite) the workgroup
// repeats its rows in a pass that raises the max lazily: a query keeps its
// max until a block's scores exceed it by more than 8 (in log2 units), so
// probabilities stay below 2^8 and the output rescale is skipped for almost
// every block.  FP32 rows (a kernel of their own, below) always use the lazy
// form.  Only the last key block of a request checks key bounds.
// K and V^T blocks of 64 keys are double-buffered in LDS and go there from HBM
// directly (buffer loads with an LDS destination, no registers in between)
// with swizzled, unpadded rows.  Loads take scalar per-block offsets, and the
// block loop runs two blocks per trip so both LDS buffers have fixed addresses.
#include <string.h>

#include "kernels.h"

namespace revo {

namespace {

constexpr int NT = 256;
constexpr int QT = 128;   // queries per workgroup (4 waves x 32)
constexpr int KB = 64;    // keys per block
constexpr float NEG_BIG = -1.0e30f;
constexpr float LAZY = 8.0f;

// One 16-byte-per-lane buffer load into LDS (lane L's bytes at lds + 16 L).
__device__ __forceinline__ void dma16_att(__amdgpu_buffer_rsrc_t rs, const void* lds, int vo, int so) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)lds, 16, vo, so, 0, 0);
}

// s_waitcnt vmcnt(N_): at most N_ of this wave's vector memory loads in flight.
template <int N_>
__device__ __forceinline__ void wait_vm_att() {
  static_assert(N_ >= 0 && N_ < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N_ & 15) | ((N_ >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// max / sum of a value and its partner lane (l ^ 32)
__device__ __forceinline__ float xhalf_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

constexpr int QCH = 4;  // 16-byte Q chunks per lane (BF16)

// BF16 K and V^T tiles: row r (a key of K, a dimension of V^T) holds its
// eight 16-byte chunks with chunk c at slot c ^ ((r >> 1) & 7), so the 16
// rows read by one 16-lane phase of a b128 read cover all 64 banks.
__device__ __forceinline__ int swz(int row, int chunk) { return row * 64 + ((chunk ^ ((row >> 1) & 7)) << 3); }

// One 64-key block for one wave: scores, online softmax, P V accumulation.
template <bool MASK, bool FIRST, bool FAST>
__device__ __forceinline__ void attn_block(const __bf16* __restrict__ kt, const __bf16* __restrict__ vt,
                                           const uint4 (&qf)[QCH], f32x16 (&oacc)[2], f32x16& negm, float& m_run,
                                           float& l_run, int lane, int kvalid) {
  typedef OpBF16 Op;
  const int half = lane >> 5, l32 = lane & 31;
  // after the first block the score products start from -m_run (all 16
  // registers of negm), so they come out already shifted by the max

  // S^T = K Q^T for two 32-key subtiles
  f32x16 sacc[2];
  if constexpr (!FIRST) {
    sacc[0] = negm;
    sacc[1] = negm;
  } else {
    sacc[0] = f32x16{};
    sacc[1] = f32x16{};
  }
  {
    // all eight K fragments in flight before the first product
    uint4 kf[QCH][2];
#pragma unroll
    for (int kc = 0; kc < QCH; ++kc)
#pragma unroll
      for (int st = 0; st < 2; ++st) kf[kc][st] = *reinterpret_cast<const uint4*>(kt + swz(st * 32 + l32, half * 4 + kc));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kc = 0; kc < QCH; ++kc)
#pragma unroll
      for (int st = 0; st < 2; ++st)
        Op::mma(sacc[st], __builtin_bit_cast(bf16x8, kf[kc][st]), __builtin_bit_cast(bf16x8, qf[kc]));
  }
  if constexpr (MASK) {
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (st * 32 + acc_row(i, lane) >= kvalid) sacc[st][i] = NEG_BIG;
  }

  // FAST (after the first block): the max stays where the first block put it
  // and no block max is taken; the caller checks the row sums after the last
  // block instead
  if constexpr (FIRST || !FAST) {
    // block max of this query
    float m0 = fmaxf(fmaxf(sacc[0][0], sacc[0][1]), sacc[0][2]);
    float m1 = fmaxf(fmaxf(sacc[1][0], sacc[1][1]), sacc[1][2]);
#pragma unroll
    for (int i = 3; i < 15; i += 2) {
      m0 = fmaxf(fmaxf(m0, sacc[0][i]), sacc[0][i + 1]);
      m1 = fmaxf(fmaxf(m1, sacc[1][i]), sacc[1][i + 1]);
    }
    float mloc = fmaxf(fmaxf(m0, sacc[0][15]), fmaxf(m1, sacc[1][15]));
    mloc = xhalf_max(mloc);
    if constexpr (FIRST) {
      // nothing accumulated yet: take this block's max as it is
      m_run = mloc;
#pragma unroll
      for (int i = 0; i < 16; ++i) negm[i] = -mloc;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int i = 0; i < 16; ++i) sacc[st][i] -= mloc;
    } else {
      // mloc is relative to m_run here
      const bool grow = mloc > LAZY;
      if (__any(grow)) {
        const float d = grow ? mloc : 0.0f;
        const float alpha = __builtin_amdgcn_exp2f(-d);
        m_run += d;
        l_run *= alpha;
        oacc[0] *= alpha;
        oacc[1] *= alpha;
#pragma unroll
        for (int i = 0; i < 16; ++i) negm[i] = -m_run;
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
          for (int i = 0; i < 16; ++i) sacc[st][i] -= d;
        // keep the rescale inside this (rarely taken) branch instead of letting
        // it become unconditional work with a selected factor
        asm volatile("" : "+v"(oacc[0]), "+v"(oacc[1]), "+v"(sacc[0]), "+v"(sacc[1]), "+v"(negm));
      }
    }
  }

  // O^T += V^T P^T, contraction over the block's keys
  // row sum from the bf16-rounded probabilities that also feed the MFMA
  const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
  float ls0 = l_run, ls1 = 0.0f;
#pragma unroll
  for (int st = 0; st < 2; ++st) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      // registers 8g..8g+7 hold keys st*32 + g*16 + {half*4 + 0..3, 8 + half*4 + 0..3};
      // V^T rows hold keys with bits 2 and 3 swapped, so those keys are the
      // 8 contiguous elements at st*32 + g*16 + half*8
      bf16x8 pf;
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[e] = (__bf16)__builtin_amdgcn_exp2f(sacc[st][8 * g + e]);
      ls0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pf[0], pf[1]}, one, ls0, false);
      ls1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pf[2], pf[3]}, one, ls1, false);
      ls0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pf[4], pf[5]}, one, ls0, false);
      ls1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pf[6], pf[7]}, one, ls1, false);
      const int pos = st * 32 + g * 16 + half * 8;
#pragma unroll
      for (int ds = 0; ds < 2; ++ds) {
        const uint4 vv = *reinterpret_cast<const uint4*>(vt + swz(ds * 32 + l32, pos >> 3));
        Op::mma(oacc[ds], __builtin_bit_cast(bf16x8, vv), pf);
      }
    }
  }
  l_run = ls0 + ls1;
}

// What a workgroup works on: head hd, queries q0 .. of the request of N tokens
// at row base (work entries: see AttnArgs).
struct AttnItem {
  int hd, N, base, q0, tile;
};
// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Remap so that XCD x runs a contiguous range of (head, q-tile) work:
// the q-tiles of one request and head then share its K/V in one L2.  False
// past the live work (grid sized for a capacity).
__device__ __forceinline__ bool attn_item(const AttnArgs& a, Prec p, AttnItem& it) {
  const int nwork = a.dyn_nwork ? *a.dyn_nwork : a.nwork;
  const int G = nwork * a.heads;
  const int L = blockIdx.x;
  if (L >= G) return false;
  const int xcd = L & 7, per = G >> 3, rem = G & 7;
  const int Lr = xcd * per + (xcd < rem ? xcd : rem) + (L >> 3);
  it.hd = Lr / nwork;
  const int i = Lr - it.hd * nwork;
  if (!a.work) {
    // one request of one_n tokens, tiles in order
    it.N = a.one_n;
    it.base = 0;
    it.tile = a.tile ? a.tile : attn_tile(p, it.N);
    it.q0 = i * it.tile;
    return true;
  }
  const int w = a.work[i];
  const ReqDesc& d = a.reqs[w >> 16];
  it.N = d.J * d.P;
  it.base = d.tok_off;
  // target-tubelet tiles (the last block, whose other queries feed nothing)
  it.tile = a.tile ? a.tile : attn_tile(p, it.N);
  it.q0 = ((w & ATTN_TARGET_TILE) ? (d.J - 1) * d.P : 0) + (w & (ATTN_TARGET_TILE - 1)) * it.tile;
  return true;
}

__global__ __launch_bounds__(NT, 3) void attn_kernel(const AttnArgs a) {
  // two K stages [key][dim], two V^T stages [dim][key], then a flag.  One
  // LDS object only: with a second one the compiler attaches alias scopes to
  // the stage loads and then waits for every prefetch before reading.
  __shared__ __attribute__((aligned(16))) __bf16 kv[4 * KB * 64 + 8];
  __bf16(*ks)[KB * 64] = reinterpret_cast<__bf16(*)[KB * 64]>(kv);
  __bf16(*vs)[KB * 64] = ks + 2;
  int& redo = *reinterpret_cast<int*>(kv + 4 * KB * 64);

  // The wave number as a scalar: the LDS destination of a stage load is a
  // scalar operand, and one per load and buffer was kept in vector registers
  // and read back at each block (24 heads x 10800 tokens 661 -> 657 us, 6 x 576
  // 8.0 -> 7.8)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  AttnItem it;
  if (!attn_item(a, P_BF16, it)) return;
  const int hd = it.hd, N = it.N, base = it.base, q0 = it.q0;
  const int q_local = q0 + wave * 32 + (lane & 31);
  const int q = base + q_local;

  const __bf16* __restrict__ Kg = (const __bf16*)a.k + ((size_t)hd * a.ldqk + base) * 64;
  const __bf16* __restrict__ Vg = (const __bf16*)a.vt + (size_t)hd * 64 * a.ldv + base;

  // Q^T fragment: this lane's query, dims [half*32, half*32 + 32); queries
  // past the request (ragged last tile) load row `base` and are never stored
  uint4 qf[QCH];
  {
    const __bf16* qp = (const __bf16*)a.q + ((size_t)hd * a.ldqk + (q_local < N ? q : base)) * 64 + half * 32;
#pragma unroll
    for (int i = 0; i < QCH; ++i) qf[i] = reinterpret_cast<const uint4*>(qp)[i];
  }

  const __amdgpu_buffer_rsrc_t krs =
      __builtin_amdgcn_make_buffer_rsrc((void*)Kg, (short)0, (a.ldqk - base) * 64 * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrs =
      __builtin_amdgcn_make_buffer_rsrc((void*)Vg, (short)0, (64 * a.ldv - base) * 2, 0x00020000);
  // Stage loads for key block kb_ into LDS buffer buf_: FETCH starts them,
  // LAND completes them (the caller then synchronises the workgroup).  Wave w
  // fills rows 16w .. 16w+15 of the K and V^T tiles, 8 rows (1 KB, 16 bytes per
  // lane) per load; lane L takes row 16w + 8j + L / 8 and the chunk whose
  // swizzled slot is L % 8.  V^T arrives with bits 2 and 3 of the key index
  // already swapped within each group of 16 keys (the QKV epilogue writes it
  // so; requests start on 16-key boundaries), so a lane's eight probabilities
  // meet one 16-byte read.
  int kvo[2], vvo[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int rr = wave * 16 + 8 * j + (lane >> 3);
    const int cc = (lane & 7) ^ ((rr >> 1) & 7);
    kvo[j] = (rr * 64 + cc * 8) * 2;
    vvo[j] = (rr * a.ldv + cc * 8) * 2;
  }
#define REVO_ATTN_DMA(rs_, lds_, vo_, so_)                                                            \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_, (__attribute__((address_space(3))) void*)(lds_), 16, \
                                           vo_, so_, 0, 0)
#define REVO_ATTN_FETCH(kb_, buf_)                                             \
  {                                                                            \
    REVO_ATTN_DMA(krs, &ks[buf_][(wave * 16) * 64], kvo[0], (kb_) * 64 * 2);   \
    REVO_ATTN_DMA(krs, &ks[buf_][(wave * 16 + 8) * 64], kvo[1], (kb_) * 64 * 2); \
    REVO_ATTN_DMA(vrs, &vs[buf_][(wave * 16) * 64], vvo[0], (kb_) * 2);        \
    REVO_ATTN_DMA(vrs, &vs[buf_][(wave * 16 + 8) * 64], vvo[1], (kb_) * 2);    \
  }
  // vmcnt(0): this wave's loads are in LDS
#define REVO_ATTN_LAND() __builtin_amdgcn_s_waitcnt(0x0F70)

  f32x16 oacc[2];
  f32x16 negm;
  float m_run, l_run;
  const int nkb = (N + KB - 1) / KB;
  const int nfull = N / KB;
  // One pass over the key blocks.  FAST passes keep the first block's max for
  // the whole row (see attn_block); SAFE passes update it lazily.  Written out
  // in the kernel body (not a called function) so that the compiler keeps
  // seeing the two LDS stages as distinct and does not wait for the prefetch
  // before reading the current stage.
#define REVO_ATTN_STEP(b_, buf_, fast_)                                                         \
  {                                                                                             \
    const int kn_ = (b_) + 1 < nkb ? ((b_) + 1) * KB : (b_) * KB;                               \
    REVO_ATTN_FETCH(kn_, buf_ ^ 1);                                                             \
    attn_block<false, false, fast_>(ks[buf_], vs[buf_], qf, oacc, negm, m_run, l_run, lane, KB); \
    REVO_ATTN_LAND();                                                                           \
    __syncthreads();                                                                            \
  }
#define REVO_ATTN_PASS(fast_)                                                                             \
  {                                                                                                       \
    oacc[0] = f32x16{};                                                                                   \
    oacc[1] = f32x16{};                                                                                   \
    m_run = 0.0f;                                                                                         \
    l_run = 0.0f;                                                                                         \
    REVO_ATTN_FETCH(0, 0);                                                                                \
    REVO_ATTN_LAND();                                                                                     \
    __syncthreads();                                                                                      \
    if (nfull == 0) {                                                                                     \
      /* a single, ragged block */                                                                        \
      attn_block<true, true, fast_>(ks[0], vs[0], qf, oacc, negm, m_run, l_run, lane, N);                 \
    } else {                                                                                              \
      /* the first block sets the max; the prefetch of the next block (or, at the end, a re-read of its   \
         own block into the idle buffer, which is then never read) overlaps it */                         \
      REVO_ATTN_FETCH(nkb > 1 ? KB : 0, 1);                                                               \
      attn_block<false, true, fast_>(ks[0], vs[0], qf, oacc, negm, m_run, l_run, lane, KB);               \
      REVO_ATTN_LAND();                                                                                   \
      __syncthreads();                                                                                    \
      int b = 1;                                                                                          \
      for (; b + 1 < nfull; b += 2) {                                                                     \
        REVO_ATTN_STEP(b, 1, fast_)                                                                       \
        REVO_ATTN_STEP(b + 1, 0, fast_)                                                                   \
      }                                                                                                   \
      if (b < nfull) REVO_ATTN_STEP(b, 1, fast_)                                                          \
      if (nfull < nkb) /* ragged last block, already in LDS */                                            \
        attn_block<true, false, fast_>(ks[nfull & 1], vs[nfull & 1], qf, oacc, negm, m_run, l_run, lane,  \
                                       N - nfull * KB);                                                   \
    }                                                                                                     \
  }
  // A FAST pass is exact as long as no probability overflowed: every
  // probability of a lane's keys is at most that lane's row sum, so row sums
  // below 2^64 bound them all (and the output by 2^64 max|v|).  Otherwise
  // (or on NaN) the whole workgroup repeats the row in a SAFE pass.
  if (tid == 0) redo = 0;  // ordered before any write by the pass's first barrier
  REVO_ATTN_PASS(true)
  if (__any(!(l_run < 0x1p64f)) && lane == 0) redo = 1;
  __syncthreads();
  if (redo) REVO_ATTN_PASS(false)  // every wave is past its last block
#undef REVO_ATTN_PASS
#undef REVO_ATTN_STEP
#undef REVO_ATTN_DMA
#undef REVO_ATTN_FETCH
#undef REVO_ATTN_LAND

  // The output goes through LDS (the K stages are free once every wave is
  // past its last block) so that whole 64-dim query rows are written in
  // 16-byte chunks rather than one short piece per query row.
  const float l_tot = xhalf_sum(l_run);
  const int ql = wave * 32 + (lane & 31);  // this lane's query within the tile
  uint8_t* st = reinterpret_cast<uint8_t*>(kv);
  __syncthreads();
  if (a.o_scale) {
    // FP8 output for an FP8 output projection
    constexpr int RB = 64 + 16;  // bytes per staged row
    const float inv = 1.0f / (l_tot * *a.o_scale);
#pragma unroll
    for (int ds = 0; ds < 2; ++ds)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int dim = ds * 32 + g * 8 + half * 4;
        *reinterpret_cast<uint32_t*>(st + ql * RB + dim) = e4m3x4(oacc[ds][4 * g] * inv, oacc[ds][4 * g + 1] * inv,
                                                                  oacc[ds][4 * g + 2] * inv, oacc[ds][4 * g + 3] * inv);
      }
    __syncthreads();
    for (int i = tid; i < QT * 4; i += NT) {
      const int row = i >> 2, c = (i & 3) * 16;
      const int qr = q0 + row;
      if (qr < N)
        *reinterpret_cast<uint4*>((uint8_t*)a.o + (size_t)(base + qr) * (a.heads * 64) + hd * 64 + c) =
            *reinterpret_cast<const uint4*>(st + row * RB + c);
    }
  } else {
    constexpr int RB = 64 * 2 + 16;
    static_assert(QT * RB <= (int)sizeof(kv), "output tile fits the K and V stages");
    const float inv = 1.0f / l_tot;
#pragma unroll
    for (int ds = 0; ds < 2; ++ds)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int dim = ds * 32 + g * 8 + half * 4;
        *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(st + ql * RB) + dim) =
            bf16x4{(__bf16)(oacc[ds][4 * g] * inv), (__bf16)(oacc[ds][4 * g + 1] * inv),
                   (__bf16)(oacc[ds][4 * g + 2] * inv), (__bf16)(oacc[ds][4 * g + 3] * inv)};
      }
    __syncthreads();
    for (int i = tid; i < QT * 8; i += NT) {
      const int row = i >> 3, c = (i & 7) * 8;
      const int qr = q0 + row;
      if (qr < N)
        *reinterpret_cast<uint4*>((__bf16*)a.o + (size_t)(base + qr) * (a.heads * 64) + hd * 64 + c) =
            *reinterpret_cast<const uint4*>(st + row * RB + c * 2);
    }
  }
}

// ---- FP32 form ---------------------------------------------------------------
//
// Q, K, V and the probabilities are split exactly into three BF16 parts each
// (common.h split3, scaled by 2^24 against subnormal parts) and every product
// of two FP32 values is the six largest of the nine products of their parts,
// accumulated in FP32 on the BF16 matrix cores: 6 products at 16 times the
// rate of the FP32 MFMA.  KG groups of QW waves (32 queries each) take every
// KG-th key block, each with its own running max, row sum and output, which
// are merged through LDS at the end.  K and V^T blocks go through registers
// (fetched one round ahead), are split once per group and lie in LDS as one
// BF16 plane per part.  Large requests take 4 waves x 2 groups (128 queries,
// two waves on every SIMD), small ones 1 wave x 6 groups (32 queries), whose
// waves share nothing until the merge and so need no barriers.
//
// The scores come out times 2^48, undone for free (the shift by the max is a
// multiply-add).  The probabilities are taken at their own size and then times
// 2^24, undone by the row sum, which has the same factor: 24 added to the
// exponent instead would save that product, but an exponent near 24 has only 19
// bits behind its point (a probability near 1 is then off by up to 6.6e-7; two
// keys 6e-8 -> 3e-7 against 64 bits, 576 with small scores 4.4e-7 -> 5.6e-7).  A row whose result is not finite (an
// infinity or NaN among its operands, or scores past 2^80) is computed again
// by FP32 MFMAs (attn_f32_row_tile).

// The rows of one wave (32 queries) with FP32 MFMAs on operands from global
// memory: scores, lazy max, probabilities, as in attn_block.
__device__ __forceinline__ void attn_f32_row_tile(const AttnArgs& a, int hd, int N, int base, int q, f32x16 (&oacc)[2],
                                               float& m_run, float& l_run) {
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const float* qp = (const float*)a.q + ((size_t)hd * a.ldqk + q) * 64;
  const float* kp = (const float*)a.k + ((size_t)hd * a.ldqk + base) * 64;
  const float* vp = (const float*)a.vt + (size_t)hd * 64 * a.ldv + base;
  oacc[0] = f32x16{};
  oacc[1] = f32x16{};
  m_run = 0.0f;
  l_run = 0.0f;
#pragma unroll 1
  for (int kb = 0; kb < N; kb += 32) {
    f32x16 s = {};
    const int kr = kb + l32 < N ? kb + l32 : N - 1;  // rows past the request are masked below
#pragma unroll 1
    for (int d = 0; d < 64; d += 2) OpF32::mma(s, kp[(size_t)kr * 64 + d + half], qp[d + half]);
    float mloc = NEG_BIG;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (kb + acc_row(i, lane) >= N) s[i] = NEG_BIG;
      mloc = fmaxf(mloc, s[i]);
    }
    mloc = xhalf_max(mloc);
    const bool grow = kb == 0 || mloc > m_run + LAZY;
    const float m_new = grow ? mloc : m_run;
    const float alpha = kb == 0 ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
    if (kb > 0 && grow) {
      l_run *= alpha;
    }
    m_run = m_new;
#pragma unroll
    for (int ds = 0; ds < 2; ++ds)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[ds][i] = kb > 0 && grow ? oacc[ds][i] * alpha : oacc[ds][i];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = __builtin_amdgcn_exp2f(s[i] - m_run);
      l_run += s[i];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int key = kb + acc_row(i, lane);
      const int kc = key < N ? key : N - 1;
      const float p = key < N ? s[i] : 0.0f;
#pragma unroll
      for (int ds = 0; ds < 2; ++ds) {
        const float v = key < N ? vp[(size_t)(ds * 32 + l32) * a.ldv + kc] : 0.0f;
        OpF32::mma(oacc[ds], v, p);
      }
    }
  }
}

// byte of 16-byte chunk c of row r of a plane with rows of KB BF16 values
template <int KBF>
__device__ __forceinline__ int f32_plane(int r, int c) {
  static_assert(KBF == 32 || KBF == 64, "rows of 64 or 128 bytes");
  return KBF == 32 ? r * 64 + ((c ^ ((r >> 2) & 3)) << 4) : r * 128 + ((c ^ ((r >> 1) & 7)) << 4);
}

constexpr int F32_NT = 512;       // threads per workgroup
constexpr int F32_LDS = 147456;   // K and V^T planes of one block per key group

template <int QW, int KG, int KBF>
__device__ __forceinline__ void attn_f32_tile(const AttnArgs& a, const AttnItem& it, uint8_t* smem) {
  static_assert(64 * QW * KG <= F32_NT, "at most eight waves (the others only join the barriers)");
  constexpr int GT = 64 * QW;               // threads of a key group
  constexpr int KP = KBF * 128, VP = 64 * KBF * 2;  // bytes per K / V^T plane
  constexpr int GB = 3 * (KP + VP);
  static_assert(KG * GB <= F32_LDS, "LDS");
  constexpr int LC = KBF * 16 / GT;         // 16-byte chunks per thread of K and of V^T
  constexpr int NST = KBF / 32;             // 32-key subtiles per block
  const int tid = threadIdx.x, lane = tid & 63;
  // (scalar, so that the block offsets of the loads and the bounds checks are)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int kg = wave / QW, qw = wave % QW, gt = tid - kg * GT;
  const int hd = it.hd, N = it.N, base = it.base, q0 = it.q0;
  const int q_local = q0 + qw * 32 + l32;
  const int q = base + (q_local < N ? q_local : 0);  // queries past the request are never stored
  uint8_t* ks = smem + kg * GB;
  uint8_t* vs = ks + 3 * KP;

  const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const float*)a.k + ((size_t)hd * a.ldqk + base) * 64), (short)0, (a.ldqk - base) * 64 * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const float*)a.vt + (size_t)hd * 64 * a.ldv + base), (short)0, (64 * a.ldv - base) * 4, 0x00020000);

  // this lane's query: dims 8 c .. 8 c + 7, c = 2 s + half, for step s
  bf16x8 qf[3][4];
  {
    const float4* qp = reinterpret_cast<const float4*>((const float*)a.q + ((size_t)hd * a.ldqk + q) * 64);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uint2 lo[3], hi[3];
      split3x4(qp[2 * (2 * s + half)], lo);
      split3x4(qp[2 * (2 * s + half) + 1], hi);
#pragma unroll
      for (int j = 0; j < 3; ++j) qf[j][s] = __builtin_bit_cast(bf16x8, make_uint4(lo[j].x, lo[j].y, hi[j].x, hi[j].y));
    }
  }
  // stage chunks: K row c / 16, dims 4 (c % 16) ..; V^T row c / (KBF / 4), keys
  // 4 (c % (KBF / 4)) .., stored with bits 2 and 3 of the key swapped (the
  // order in which a lane's eight probabilities meet one 16-byte read)
  float4 kr[LC], vr[LC];
  auto fetch = [&](int kb) {
#pragma unroll
    for (int i = 0; i < LC; ++i) {
      const int c = gt + i * GT;
      kr[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(krs, c * 16, kb * 256, 0));
      vr[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(
                                             vrs, ((c / (KBF / 4)) * a.ldv + (c % (KBF / 4)) * 4) * 4, kb * 4, 0));
    }
  };
  auto land = [&]() {
#pragma unroll
    for (int i = 0; i < LC; ++i) {
      const int c = gt + i * GT;
      uint2 p[3];
      split3x4(kr[i], p);
      const int ko = f32_plane<64>(c / 16, (c % 16) >> 1) + (c & 1) * 8;
#pragma unroll
      for (int j = 0; j < 3; ++j) *reinterpret_cast<uint2*>(ks + j * KP + ko) = p[j];
      split3x4(vr[i], p);
      const int u = c % (KBF / 4), up = (u & ~3) | ((u & 1) << 1) | ((u >> 1) & 1);
      const int vo = f32_plane<KBF>(c / (KBF / 4), up >> 1) + (up & 1) * 8;
#pragma unroll
      for (int j = 0; j < 3; ++j) *reinterpret_cast<uint2*>(vs + j * VP + vo) = p[j];
    }
  };
  constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};  // smallest products first

  f32x16 oacc[2];
  oacc[0] = f32x16{};
  oacc[1] = f32x16{};
  float m_run = NEG_BIG, l_run = 0.0f;
  // a group of one wave orders its LDS stores and reads by itself
  auto group_sync = [&]() {
    if constexpr (QW == 1) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    } else {
      __syncthreads();
    }
  };
  static_assert(QW == 1 || 64 * QW * KG == F32_NT, "barriers need every wave in the loop");
  const int nkb = (N + KBF - 1) / KBF, rounds = kg < KG ? (nkb + KG - 1) / KG : 0;
  if (rounds > 0) fetch(kg * KBF);
  for (int t = 0; t < rounds; ++t) {
    const int kb = (t * KG + kg) * KBF;
    if (t > 0) group_sync();  // the previous block is consumed
    land();
    group_sync();
    if (t + 1 < rounds) fetch(kb + KG * KBF);
    if (kb >= N) continue;  // the last round of a group without a block (the barriers above still meet)
    // S^T = K Q^T
    f32x16 s[NST];
#pragma unroll
    for (int st = 0; st < NST; ++st) s[st] = f32x16{};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      bf16x8 kf[3][NST];
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int st = 0; st < NST; ++st)
          kf[j][st] = *reinterpret_cast<const bf16x8*>(ks + j * KP + f32_plane<64>(st * 32 + l32, 2 * c + half));
#pragma unroll
      for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int st = 0; st < NST; ++st) OpBF16::mma(s[st], kf[PA[p]][st], qf[PB[p]][c]);
    }
    if (kb + KBF > N) {
#pragma unroll
      for (int st = 0; st < NST; ++st)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kb + st * 32 + acc_row(i, lane) >= N) s[st][i] = -INFINITY;
    }
    // lazy max (true scores are 2^-48 s)
    float mx = s[0][0];
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[st][i]);
    const float mloc = xhalf_max(mx) * 0x1p-48f;
    const bool grow = mloc > m_run + LAZY;
    if (__any(grow)) {
      const float m_new = grow ? mloc : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
      oacc[0] *= alpha;
      oacc[1] *= alpha;
      asm volatile("" : "+v"(oacc[0]), "+v"(oacc[1]));
    }
    // probabilities times 2^24, row sum, O^T += V^T P^T
    const float sh = -m_run;
    float l0 = 0.0f, l1 = 0.0f;
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        uint32_t pw[3][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(s[st][8 * g + 2 * e], 0x1p-48f, sh)) * 0x1p24f;
          const float p1 = __builtin_amdgcn_exp2f(fmaf(s[st][8 * g + 2 * e + 1], 0x1p-48f, sh)) * 0x1p24f;
          l0 += p0;
          l1 += p1;
          split3(p0, p1, pw[0][e], pw[1][e], pw[2][e]);
        }
        bf16x8 pf[3], vf[3][2];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          pf[j] = __builtin_bit_cast(bf16x8, make_uint4(pw[j][0], pw[j][1], pw[j][2], pw[j][3]));
#pragma unroll
          for (int ds = 0; ds < 2; ++ds)
            vf[j][ds] =
                *reinterpret_cast<const bf16x8*>(vs + j * VP + f32_plane<KBF>(ds * 32 + l32, st * 4 + g * 2 + half));
        }
#pragma unroll
        for (int p = 0; p < 6; ++p)
#pragma unroll
          for (int ds = 0; ds < 2; ++ds) OpBF16::mma(oacc[ds], vf[PA[p]][ds], pf[PB[p]]);
      }
    l_run += l0 + l1;
  }
  l_run = xhalf_sum(l_run);

  // the other groups' maxima, sums and outputs into the first's, in order
  // (O of group g, wave qw: 32 floats per lane at [i][lane])
  float* red = reinterpret_cast<float*>(smem);
  constexpr int RW = 34 * 64;
  static_assert((KG - 1) * QW * RW * 4 <= F32_LDS, "merge buffer");
  __syncthreads();  // every wave is past its last block
  if (kg > 0 && kg < KG) {
    float* r = red + ((kg - 1) * QW + qw) * RW;
    r[lane] = m_run;
    r[64 + lane] = l_run;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      r[(2 + i) * 64 + lane] = oacc[0][i];
      r[(18 + i) * 64 + lane] = oacc[1][i];
    }
  }
  __syncthreads();
  if (kg == 0) {
#pragma unroll
    for (int g = 0; g < KG - 1; ++g) {
      const float* r = red + (g * QW + qw) * RW;
      const float m2 = r[lane], l2 = r[64 + lane];
      const float m_new = fmaxf(m_run, m2);
      const float a1 = __builtin_amdgcn_exp2f(m_run - m_new), a2 = __builtin_amdgcn_exp2f(m2 - m_new);
      m_run = m_new;
      l_run = l_run * a1 + l2 * a2;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        oacc[0][i] = oacc[0][i] * a1 + r[(2 + i) * 64 + lane] * a2;
        oacc[1][i] = oacc[1][i] * a1 + r[(18 + i) * 64 + lane] * a2;
      }
    }
  }
  __syncthreads();  // the merge buffer has been read: LDS takes the output tile
  constexpr int RB = 64 * 4 + 16;
  static_assert(32 * QW * RB <= F32_LDS, "output tile");
  if (kg == 0) {
    float t = l_run * 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t = fmaf(oacc[0][i], 0.0f, fmaf(oacc[1][i], 0.0f, t));
    float inv;
    if (__any(!(t == 0.0f) || !(l_run > 0.0f))) {
      attn_f32_row_tile(a, hd, N, base, q, oacc, m_run, l_run);
      l_run = xhalf_sum(l_run);
      inv = 1.0f / l_run;
    } else {
      inv = 0x1p-24f / l_run;  // O holds 2^48, the row sum 2^24 times its value
      l_run *= 0x1p-24f;
    }
    if (a.lse && lane < 32 && q_local < N)
      a.lse[(size_t)hd * a.ldqk + q] = m_run + log2f(l_run);  // P = exp2(s - lse)
#pragma unroll
    for (int ds = 0; ds < 2; ++ds)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4*>(smem + (qw * 32 + l32) * RB + (ds * 32 + g * 8 + half * 4) * 4) =
            f32x4{oacc[ds][4 * g] * inv, oacc[ds][4 * g + 1] * inv, oacc[ds][4 * g + 2] * inv, oacc[ds][4 * g + 3] * inv};
  }
  __syncthreads();
  for (int i = tid; i < 32 * QW * 16; i += F32_NT) {
    const int row = i >> 4, c = (i & 15) * 4;
    const int qr = q0 + row;
    if (qr < N)
      *reinterpret_cast<uint4*>((float*)a.o + (size_t)(base + qr) * (a.heads * 64) + hd * 64 + c) =
          *reinterpret_cast<const uint4*>(smem + row * RB + c * 4);
  }
}

// One workgroup per work entry and head.  What bounds it at full load is the
// matrix cores: 6 heads of 10800 tokens take 921 us, 195 TFLOP/s of FP32 work or
// 1170 TFLOP/s of BF16 products (FP32 MFMAs: 1357 us); 6 heads of 3600 tokens,
// 174 workgroups on 256 CUs, 243 -> 139 us; 6 heads of 576 42.7 -> 17.2 us, three
// rounds of a wave's block at 3.3 us, its splits and products one after the
// other.  Errors against 64 bits, relative rms, FP32 MFMAs first: 1.35e-6 and
// 8.1e-7 at 3600 tokens, 7.6e-7 and 4.8e-7 at 576, 2.0e-7 and 1.5e-7 at 8; two
// tokens 8.2e-8 and 9.2e-8.
__global__ __launch_bounds__(F32_NT, 2) void attn_f32_kernel(const AttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[F32_LDS];
  AttnItem it;
  if (!attn_item(a, P_FP32, it)) return;
  if (it.tile == 32) attn_f32_tile<1, 6, 32>(a, it, smem);
  else attn_f32_tile<4, 2, 64>(a, it, smem);
}

// ---- FP8 form ----------------------------------------------------------------
//
// Q, K and V^T are OCP E4M3 with per-head power-of-two scales 2^eq, 2^ek,
// 2^ev, applied exactly by the scaled 32x32x64 FP8 MFMA (E8M0 block scales),
// so the score products come out in the BF16 kernel's units (log2 scale,
// onto the -max register block).  The probabilities are E4M3 with unit
// scale; the max is raised lazily as in the safe pass above, which keeps
// them at most 2^8 (E4M3 holds up to 448).  The row sums are those of the
// E4M3 probabilities, taken by one more product per block (a ones row
// against P^T) instead of VALU adds.  A head dimension of 64 is one product
// step: per 64-key block a wave issues 2 score, 2 P V and 1 row-sum products.  K rows and V^T rows are
// 64 bytes in LDS, 16-byte chunk c of row r at slot c ^ ((r >> 2) & 3), so
// the 16 rows one read phase touches cover all banks.  V^T columns are in
// fp8_vt_col order within each group of 64 keys (requests start on
// 64-token boundaries), so a lane's probabilities are its 32 consecutive k.

__device__ __forceinline__ int swz8(int row, int chunk) { return row * 64 + ((chunk ^ ((row >> 2) & 3)) << 4); }

// E8M0 exponents of an attn_fp8_kernel launch: a device array (the network's
// calibration) or, for the one-request entry point, values in the launch
struct Fp8Exps {
  const int* dev;
  uint8_t val[3 * ATTN_MAX_OP_HEADS];
};

__device__ __forceinline__ f32x16 mfma_fp8(const i32x8& a, const i32x8& b, const f32x16& c, int sa, int sb) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, sa, 0, sb);
}

__device__ __forceinline__ i32x8 load_frag8(const uint8_t* __restrict__ t, int row, int half) {
  const uint4 lo = *reinterpret_cast<const uint4*>(t + swz8(row, 2 * half));
  const uint4 hi = *reinterpret_cast<const uint4*>(t + swz8(row, 2 * half + 1));
  return i32x8{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
}

// Probabilities of one lane (byte j = 16 st + i of its 32, fp8_vt_col order)
// from the scores relative to the running max, without saturation: an
// exponent past 8.8 gives the E4M3 NaN (0x7F) or 448 (0x7E).
__device__ __forceinline__ i32x8 fp8_probs(const f32x16 (&sacc)[2]) {
  i32x8 pf;
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float p[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(sacc[st][4 * g + e]);
      int v = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], 0, false);
      pf[st * 4 + g] = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], v, true);
    }
  return pf;
}

template <bool MASK, bool FIRST>
__device__ __forceinline__ void fp8_block(const uint8_t* __restrict__ kt, const uint8_t* __restrict__ vt,
                                          const i32x8& qf, const i32x8& ones, f32x16 (&oacc)[2], f32x16& lacc,
                                          f32x16& negm, float& m_run, int lane, int kvalid, int eqk_q, int eqk_k,
                                          int ev) {
  const int half = lane >> 5, l32 = lane & 31;
  i32x8 kf[2];
#pragma unroll
  for (int st = 0; st < 2; ++st) kf[st] = load_frag8(kt, st * 32 + l32, half);
  __builtin_amdgcn_sched_barrier(0);
  f32x16 sacc[2];
#pragma unroll
  for (int st = 0; st < 2; ++st) sacc[st] = mfma_fp8(kf[st], qf, FIRST ? f32x16{} : negm, eqk_k, eqk_q);
  if constexpr (MASK) {
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (st * 32 + acc_row(i, lane) >= kvalid) sacc[st][i] = NEG_BIG;
  }
  auto block_max = [&]() {
    float m0 = fmaxf(fmaxf(sacc[0][0], sacc[0][1]), sacc[0][2]);
    float m1 = fmaxf(fmaxf(sacc[1][0], sacc[1][1]), sacc[1][2]);
#pragma unroll
    for (int i = 3; i < 15; i += 2) {
      m0 = fmaxf(fmaxf(m0, sacc[0][i]), sacc[0][i + 1]);
      m1 = fmaxf(fmaxf(m1, sacc[1][i]), sacc[1][i + 1]);
    }
    return xhalf_max(fmaxf(fmaxf(m0, sacc[0][15]), fmaxf(m1, sacc[1][15])));
  };
  i32x8 pf;
  if constexpr (FIRST) {
    const float mloc = block_max();
    m_run = mloc;
#pragma unroll
    for (int i = 0; i < 16; ++i) negm[i] = -mloc;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int i = 0; i < 16; ++i) sacc[st][i] -= mloc;
    pf = fp8_probs(sacc);
  } else {
    // The max is raised only past LAZY, that is when a probability exceeds
    // 2^8: first the probabilities as they are, then a look at their bytes (one
    // of 0x78 = 256 or above carries into bit 7 when 8 is added: 12 operations
    // where the block max takes 23), and only then the block max itself.  24
    // heads x 10800 tokens: 453 -> 441 us, bit-identical (VALU-bound: 32 exp2 a
    // block and lane are about 2/3 of that).
    static_assert(LAZY == 8.0f, "0x78 is 2^8");
    pf = fp8_probs(sacc);
    unsigned big = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) big |= (unsigned)pf[j] + 0x08080808u;
    if (__any((big & 0x80808080u) != 0)) {
      const float mloc = block_max();  // relative to m_run
      const bool grow = mloc > LAZY;
      if (__any(grow)) {
        const float d = grow ? mloc : 0.0f;
        const float alpha = __builtin_amdgcn_exp2f(-d);
        m_run += d;
        oacc[0] *= alpha;
        oacc[1] *= alpha;
        lacc *= alpha;
#pragma unroll
        for (int i = 0; i < 16; ++i) negm[i] = -m_run;
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
          for (int i = 0; i < 16; ++i) sacc[st][i] -= d;
        pf = fp8_probs(sacc);
        asm volatile("" : "+v"(oacc[0]), "+v"(oacc[1]), "+v"(lacc), "+v"(negm), "+v"(pf));
      }
    }
  }
#pragma unroll
  for (int ds = 0; ds < 2; ++ds) oacc[ds] = mfma_fp8(load_frag8(vt, ds * 32 + l32, half), pf, oacc[ds], ev, 127);
  // row sums of the E4M3 probabilities on the matrix core: a block whose
  // row 0 is all ones (the other rows zero) times P^T
  lacc = mfma_fp8(ones, pf, lacc, 127, 127);
}

__global__ __launch_bounds__(NT, 3) void attn_fp8_kernel(const AttnArgs a, const Fp8Exps exps) {
  constexpr int TB = KB * 64;  // bytes per K or V^T tile
  __shared__ __attribute__((aligned(16))) uint8_t kv[4 * TB];
  uint8_t* ks = kv;
  uint8_t* vs = kv + 2 * TB;
  // scalar wave number, as in attn_kernel (24 heads x 10800 tokens 434 -> 427 us)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  AttnItem it;
  if (!attn_item(a, P_FP8, it)) return;
  const int hd = it.hd, N = it.N, base = it.base, q0 = it.q0;
  const int q_local = q0 + wave * 32 + (lane & 31);
  const int q = base + q_local;
  // E8M0 scale operands (127 + e)
  const int sq = exps.dev ? exps.dev[hd] : exps.val[hd];
  const int sk = exps.dev ? exps.dev[a.heads + hd] : exps.val[a.heads + hd];
  const int sv = exps.dev ? exps.dev[2 * a.heads + hd] : exps.val[2 * a.heads + hd];

  const uint8_t* Kg = (const uint8_t*)a.k + ((size_t)hd * a.ldqk + base) * 64;
  const uint8_t* Vg = (const uint8_t*)a.vt + (size_t)hd * 64 * a.ldv + base;
  i32x8 qf;
  {
    const uint4* qp = reinterpret_cast<const uint4*>((const uint8_t*)a.q + ((size_t)hd * a.ldqk + (q_local < N ? q : base)) * 64 + half * 32);
    const uint4 lo = qp[0], hi = qp[1];
    qf = i32x8{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
  }
  const __amdgpu_buffer_rsrc_t krs =
      __builtin_amdgcn_make_buffer_rsrc((void*)Kg, (short)0, (a.ldqk - base) * 64, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrs =
      __builtin_amdgcn_make_buffer_rsrc((void*)Vg, (short)0, 64 * a.ldv - base, 0x00020000);
  // wave w fills rows 16w .. 16w+15 of the K and V^T tiles (1 KB, 16 bytes
  // per lane); lane L takes row 16w + L / 4 and the chunk whose swizzled
  // slot is L % 4
  const int rr = wave * 16 + (lane >> 2);
  const int cc = (lane & 3) ^ ((rr >> 2) & 3);
  const int kvo = rr * 64 + cc * 16;
  const int vvo = rr * a.ldv + cc * 16;
  auto fetch = [&](int kb, int buf) {
    dma16_att(krs, ks + buf * TB + wave * 16 * 64, kvo, kb * 64);
    dma16_att(vrs, vs + buf * TB + wave * 16 * 64, vvo, kb);
  };
  f32x16 oacc[2], lacc, negm;
  oacc[0] = f32x16{};
  oacc[1] = f32x16{};
  lacc = f32x16{};
  negm = f32x16{};
  float m_run = 0.0f;
  // row 0 of the row-sum block: E4M3 ones (0x38) from lanes 0 and 32
  const int one8 = (lane & 31) == 0 ? 0x38383838 : 0;
  const i32x8 ones = {one8, one8, one8, one8, one8, one8, one8, one8};
  const int nkb = (N + KB - 1) / KB;
  const int nfull = N / KB;
  fetch(0, 0);
  wait_vm_att<0>();
  __syncthreads();
  if (nfull == 0) {
    fp8_block<true, true>(ks, vs, qf, ones, oacc, lacc, negm, m_run, lane, N, sq, sk, sv);
  } else {
    fetch(nkb > 1 ? KB : 0, 1);
    fp8_block<false, true>(ks, vs, qf, ones, oacc, lacc, negm, m_run, lane, KB, sq, sk, sv);
    wait_vm_att<0>();
    __syncthreads();
    int b = 1;
    for (; b + 1 < nfull; b += 2) {
      fetch((b + 1) * KB, 0);
      fp8_block<false, false>(ks + TB, vs + TB, qf, ones, oacc, lacc, negm, m_run, lane, KB, sq, sk, sv);
      wait_vm_att<0>();
      __syncthreads();
      fetch(b + 2 < nkb ? (b + 2) * KB : (b + 1) * KB, 1);
      fp8_block<false, false>(ks, vs, qf, ones, oacc, lacc, negm, m_run, lane, KB, sq, sk, sv);
      wait_vm_att<0>();
      __syncthreads();
    }
    if (b < nfull) {
      fetch(b + 1 < nkb ? (b + 1) * KB : b * KB, 0);
      fp8_block<false, false>(ks + TB, vs + TB, qf, ones, oacc, lacc, negm, m_run, lane, KB, sq, sk, sv);
      wait_vm_att<0>();
      __syncthreads();
    }
    if (nfull < nkb)  // ragged last block, already in LDS
      fp8_block<true, false>(ks + (nfull & 1) * TB, vs + (nfull & 1) * TB, qf, ones, oacc, lacc, negm, m_run, lane,
                             N - nfull * KB, sq, sk, sv);
  }
  // output through LDS in whole 64-dim rows (the tiles are free once every
  // wave is past its last block)
  // the row sum of query l % 32 sits in register 0 of lane l % 32 (row 0 of
  // the block); lanes 32..63 hold rows 4..7, all zero
  const float l_tot = xhalf_sum(lane < 32 ? lacc[0] : 0.0f);
  const int ql = wave * 32 + (lane & 31);
  uint8_t* st = kv;
  __syncthreads();
  if (a.o_scale) {
    constexpr int RB = 64 + 16;
    static_assert(QT * RB <= 4 * TB, "output tile fits the stages");
    const float inv = 1.0f / (l_tot * *a.o_scale);
#pragma unroll
    for (int ds = 0; ds < 2; ++ds)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int dim = ds * 32 + g * 8 + half * 4;
        *reinterpret_cast<uint32_t*>(st + ql * RB + dim) = e4m3x4(oacc[ds][4 * g] * inv, oacc[ds][4 * g + 1] * inv,
                                                                  oacc[ds][4 * g + 2] * inv, oacc[ds][4 * g + 3] * inv);
      }
    __syncthreads();
    for (int i = tid; i < QT * 4; i += NT) {
      const int row = i >> 2, c = (i & 3) * 16;
      const int qr = q0 + row;
      if (qr < N)
        *reinterpret_cast<uint4*>((uint8_t*)a.o + (size_t)(base + qr) * (a.heads * 64) + hd * 64 + c) =
            *reinterpret_cast<const uint4*>(st + row * RB + c);
    }
  } else {
    // BF16 output: two passes of 64 queries through the 16 KB of stages
    constexpr int RB = 64 * 2 + 16;
    const float inv = 1.0f / l_tot;
    for (int pass = 0; pass < 2; ++pass) {
      if ((wave >> 1) == pass) {
        const int qp = ql - pass * 64;
#pragma unroll
        for (int ds = 0; ds < 2; ++ds)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int dim = ds * 32 + g * 8 + half * 4;
            *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(st + qp * RB) + dim) =
                bf16x4{(__bf16)(oacc[ds][4 * g] * inv), (__bf16)(oacc[ds][4 * g + 1] * inv),
                       (__bf16)(oacc[ds][4 * g + 2] * inv), (__bf16)(oacc[ds][4 * g + 3] * inv)};
          }
      }
      __syncthreads();
      for (int i = tid; i < 64 * 8; i += NT) {
        const int row = i >> 3, c = (i & 7) * 8;
        const int qr = q0 + pass * 64 + row;
        if (qr < N)
          *reinterpret_cast<uint4*>((__bf16*)a.o + (size_t)(base + qr) * (a.heads * 64) + hd * 64 + c) =
              *reinterpret_cast<const uint4*>(st + row * RB + c * 2);
      }
      __syncthreads();
    }
  }
}

}  // namespace

int launch_attention(Prec prec, const AttnArgs& a, hipStream_t s, const uint8_t* exps) {
  if (a.nwork <= 0) return 0;
  dim3 grid(a.nwork * a.heads);
  if (prec == P_FP8 && (a.qkv_exp || exps)) {
    Fp8Exps e;
    e.dev = a.qkv_exp;
    if (!a.qkv_exp) {
      if (a.heads > ATTN_MAX_OP_HEADS) return -22;
      memcpy(e.val, exps, 3 * a.heads);
    }
    attn_fp8_kernel<<<grid, NT, 0, s>>>(a, e);
  } else if (prec == P_BF16 || prec == P_FP8) {
    attn_kernel<<<grid, NT, 0, s>>>(a);  // uncalibrated FP8 form: BF16
  } else if (prec == P_FP32 && !a.o_scale) {
    attn_f32_kernel<<<grid, F32_NT, 0, s>>>(a);
  } else {
    return -95;
  }
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

int launch_attention_one(Prec prec, const void* q, const void* k, const void* vt, void* o, int heads, int ntok, int ld,
                         const uint8_t* exps, hipStream_t s) {
  AttnArgs a;
  memset(&a, 0, sizeof(a));
  a.q = q; a.k = k; a.vt = vt; a.o = o; a.heads = heads; a.ldqk = ld; a.ldv = ld;
  a.one_n = ntok;
  a.tile = attn_tile_all(prec, ntok, heads);
  a.nwork = cdiv(ntok, a.tile);
  return launch_attention(prec, a, s, exps);
}

}  // namespace revo
