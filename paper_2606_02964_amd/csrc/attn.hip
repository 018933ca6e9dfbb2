// attn.hip -- gfx950 kernels of Multi-Segment Attention.
//
// msa_attn: workgroups of W waves (W = 4 or 8: 128 or 256 rows, 32 rows per
// wave), each running its own list of work items (the launch is persistent;
// the plan deals the items out).  A work item is query rows of one sequence
// sharing one KV head, over one key range.  Each 64-key step:
//   - paged gather: the step's 4 cache blocks are looked up in the block
//     table (ids preloaded one lane per step, read with v_readlane) and
//     copied straight into LDS (global_load_lds,
//     16 bytes a lane, no staging registers): K as [key][d] rows, V as the
//     cache's channel-major [d][16 keys] pages, 16-byte chunks XOR-swizzled
//     so that every operand read is free of bank conflicts.  K runs one step
//     ahead of V in rings of two stages.  The copies are inline assembly
//     (see dma16 for why);
//   - S^T = K Q^T on v_mfma_f32_32x32x16_bf16.  K is the A operand, so each
//     lane holds one query row (a column of S^T) and 16 of the 32 keys: the
//     row max and row sum need one exchange with the lane 32 apart only;
//   - per-row causal limit: key j is visible to the row at absolute position
//     p iff j <= p (only on steps that reach past the wave's smallest
//     position; a wave stops computing after the step holding its largest
//     position, while it keeps copying its share and meeting the barriers);
//   - online softmax in fp32 in the exp2 domain: scale * log2(e) enters one
//     FMA per score against a reference max that only moves (and O is only
//     rescaled) when a row's max grows by more than 2^8.  The row max itself
//     is only taken when a step's weights may have outgrown the reference
//     (see settle); the row sum adds the fp32 weights with plain adds (a
//     v_dot2 of the packed weights stalls the MFMA stream on gfx950);
//   - O^T += V^T P^T on the same MFMA, P packed to bf16 straight from the
//     score registers.  The A-operand row order of K is permuted (bits 2 and 3
//     of the row index swapped) so that the 8 scores a lane feeds to one PV
//     step are 8 consecutive keys, a single 16-byte LDS read of V^T.  On the
//     step holding a row's own position (its latest keys, and all keys of a
//     row near the start of a sequence) its weights enter as two bf16 terms,
//     hi = bf16(w) and lo = bf16(w - hi), with a second PV pass on lo, and
//     its row sum adds them in fp32: rows whose weight sits on a few keys
//     then carry their weights to about 2^-18 instead of 2^-9.
// Steps that need no mask run software-pipelined, in pairs and then up to two
// singly: the QK MFMAs of step j+1 are interleaved with the exponentials of
// step j, so that each of them is followed by independent vector work.  The
// diagonal steps and a wave's last one (with precise weights also the one
// before a diagonal step) run the same operations without overlap.
// msa_decode: 32-row tiles of decode-like plans and 32-row items of plans with
// few short tiles; the four waves of a workgroup split the tile's keys, read K
// and V straight into registers and merge their softmax states through LDS
// (see the kernel); the half-steps of a row's diagonal step carry its weights
// as hi + lo terms, as above.
// Both kernels also come in a precise-weights form (kPrecise, selected by
// the plan): every step, or half-step, carries every row's weights as
// hi + lo terms.
// msa_merge: combines the per-split partials of a split tile by log-sum-exp.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>

#include "msa_internal.h"

namespace msa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLn2 = 0.69314718055994531f;
constexpr float kLog2e = 1.4426950408889634f;

// LDS layout of one stage (no padding; 16-byte chunks XOR-swizzled so that
// every 16-lane group of an operand read hits 16 distinct bank groups):
//   K tile: 64 keys x D channels, row = key (2*D bytes); chunk c of row k is
//           stored at chunk c ^ ((k / rows per 256 bytes) mod chunks per row)
//   V tile: page-major, 4 blocks x D channels x 16 keys (32 bytes per channel
//           row); the two 16-byte halves of channel d swap when bit 3 of d is set
template <int D>
struct Tile {
  static constexpr int kBytesK = kKvStep * D * 2;
  static constexpr int kBytesV = kKvStep * D * 2;
  static constexpr int kPage = kBlockSize * D * 2;  // bytes of one block of K or V
  static constexpr int kDmaPerPage = kPage / 1024;  // 1 KB per wave-wide 16-byte copy
};

__device__ __forceinline__ int swap_bits23(int m) {
  return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1);
}

// max / sum of x over the lane pair (l, l ^ 32)
__device__ __forceinline__ float pair_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// bf16 pair (a, b) packed into one register, round to nearest even
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}

typedef __attribute__((address_space(3))) void lds_void_t;

// 16 bytes per lane from global memory (wave-uniform base + per-lane 32-bit
// byte offset) straight into LDS at lds + 16 * lane (a wave copies 1 KB; M0
// holds the wave's LDS base); completion is tracked by vmcnt.  The base goes
// in scalar registers, so the copy needs no vector address arithmetic.
// Issued as inline assembly: when the compiler sees these copies it treats
// the LDS counter as unordered and waits for every outstanding LDS read
// (lgkmcnt(0)) before each MFMA, which cancels the operand read-ahead.  The
// kernel itself waits for the copies (wait_dma) before the barrier that
// publishes them; the compiler's own vmcnt waits stay correct because vector
// loads complete in issue order, so extra loads it does not count only make
// those waits stricter.  The s_nop covers the M0-write-to-LDS-DMA hazard.
__device__ __forceinline__ void dma16(const void* base, uint32_t off, void* lds) {
  const uint32_t l = (uint32_t)(uintptr_t)(lds_void_t*)lds;
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "{m0}"(l) : "memory");
}
// wait until at most n copies issued by this wave are outstanding
template <int n>
__device__ __forceinline__ void wait_dma() {
  static_assert(n >= 0 && n < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
}
// workgroup barrier that orders LDS accesses only: the compiler's
// __syncthreads() would also drain every outstanding global->LDS copy
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// running-max threshold of the lazy rescale: the reference max only moves
// when a row's max grows by more than this (log2 units), so the unnormalised
// weights stay <= 2^8
constexpr float kRescaleLog2 = 8.0f;
// a lane's step sum of weights at which the row max is taken (see settle)
constexpr float kSettleSum = 128.0f;

// r / G for a tile row r < 256 (r * (G * group_inv - 2^16) < 2^16, so exact)
__device__ __forceinline__ int div_group(int r, const AttnParams& p) {
  return (int)((uint32_t)r * (uint32_t)p.group_inv >> 16);
}

// One work item of msa_attn.  smem: the K ring (2 steps) then the V ring
// (2 steps).  Every wave leaves through the barrier that ends the item's
// last step before its epilogue (registers only), so the next item may
// refill the rings at once.
template <int D, int W, bool kPrecise, bool kHelp>
__device__ __forceinline__ void attn_item(const AttnParams& p, const WorkItem w, char* smem) {
  using T = Tile<D>;
  constexpr int kRows = 32 * W;  // tile rows
  if (w.nrows == 0) return;  // (uniform over the workgroup)

  // lane-dependent set-up is computed per item (an opaque copy of the
  // thread id keeps it from being hoisted and held across items)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int lane = tid & 63, hl = lane >> 5, ln = lane & 31;
  const int G = p.group;
  const int r = wave * 32 + ln;  // tile row
  const int t = div_group(r, p), hh = r - t * G;
  const bool valid = t < w.nrows;
  const int tok = w.row0 + t;
  const int head = w.kv_head * G + hh;

  // Block ids: every page a wave copies belongs to block slot wave & 3 of
  // its step, so a wave needs one id per step.  Lane i of idv holds the id of
  // step id_base + i, idv_next those of the next 64 steps; both load before
  // everything else of the item, since the first copies wait for them.
  const int32_t* bt = p.block_table + (int64_t)w.seq * p.max_blocks;
  const int bslot = wave & 3;
  const int n = (w.kv_hi - w.kv_lo + kKvStep - 1) / kKvStep;
  auto load_ids = [&](int s0) -> int32_t {
    const int st = s0 + lane;
    const int kb = w.kv_lo + st * kKvStep + bslot * kBlockSize;
    return (st < n && kb < w.kv_hi) ? bt[kb >> 4] : 0;
  };
  int32_t idv = load_ids(0), idv_next = n > 64 ? load_ids(64) : 0;

  const int pos = valid ? p.row_pos[tok] : -1;

  // Q fragments (B operand): row r, channels kk*16 + hl*8 .. +8
  bf16x8 qf[D / 16];
  {
    const uint16_t* qrow = p.q + (int64_t)tok * p.q_st + (int64_t)head * p.q_sh + hl * 8;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      if (valid) {
        qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + kk * 16);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) qf[kk][j] = (__bf16)0.0f;
      }
    }
  }

  // Gather geometry: a page (one block of K or V) is kDmaPerPage wave-wide
  // 16-byte copies (see the layout note above); lane offsets inside a block:
  constexpr int kChunksPerRow = 2 * D / 16;            // 16-byte chunks per K row
  constexpr int kRowsPerCopy = 64 / kChunksPerRow;     // K rows per 1 KB copy
  constexpr int kRowsPer256 = 256 / (2 * D);           // K rows sharing one 256-byte bank row
  auto kswz = [](int k) { return (k / kRowsPer256) & (kChunksPerRow - 1); };
  uint32_t kgo[T::kDmaPerPage];                       // byte offsets inside a cache block
#pragma unroll
  for (int q = 0; q < T::kDmaPerPage; ++q) {
    const int kin = q * kRowsPerCopy + lane / kChunksPerRow;
    const int lc = (lane % kChunksPerRow) ^ kswz(kin);
    kgo[q] = (uint32_t)(kin * p.k_st + lc * 8) * 2u;
  }
  // V copy q moves channels q*32 .. q*32+31: the same lane pattern, shifted
  // by 32 channels (bit 3 of the channel, hence the half swap, is unchanged)
  const uint32_t vgo0 = (uint32_t)((lane >> 1) * p.v_sd + (((lane & 1) ^ ((lane >> 4) & 1)) * 8)) * 2u;
  const uint32_t vgq = (uint32_t)(32 * p.v_sd) * 2u;
  const int64_t ksb = p.k_sb * 2, vsb = p.v_sb * 2;  // bytes per block
  const char* kbase = reinterpret_cast<const char*>(p.k + (int64_t)w.kv_head * p.k_sh);
  const char* vbase = reinterpret_cast<const char*>(p.v + (int64_t)w.kv_head * p.v_sh);
  auto kbuf = [&](int s) -> char* { return smem + __builtin_amdgcn_readfirstlane((s & 1) * T::kBytesK); };
  auto vbuf = [&](int s) -> char* {
    return smem + __builtin_amdgcn_readfirstlane(2 * T::kBytesK + (s & 1) * T::kBytesV);
  };
  // A step has 8 pages: the K and the V page of each of its 4 blocks; a
  // copying wave copies both pages of its block slot.  With 8 waves (256-row
  // tiles, and the helpers of kHelp) only waves 4-7 copy, one on each SIMD,
  // while waves 0-3 go straight to their MFMAs:
  // issuing a wave's copies takes it 40-80 cycles each, in which a SIMD whose
  // two waves both copy issues nothing else (338 of a step's 3360 cycles; with
  // four copying waves the 8 x 8192 workload takes 1389 us, not 1404, and
  // 2 x 32768 7628 us, not 7700).
  // Iteration j copies the K of step j+2 and the V of step j+1, so the id read
  // for a K page serves the V page of the next iteration.  A block at or past
  // kv_hi is not read; its V page is zero-filled instead (its K page keeps old
  // values: those keys are masked by selection, so never meet arithmetic).
  const bool copier = wave >= 4 || (W == 4 && !kHelp);  // wave-uniform
  const char *kpage, *vpage;  // pages of the next copies
  int32_t id_cur = 0;
  // Reads the ids of K step s and V step s - 1 and takes their page
  // addresses; called for s = 0, 1, 2, ... in turn, one iteration before the
  // copies, where the address arithmetic runs beside MFMAs.  (Taken at the
  // start of the iteration, with the range checks of both pages, it held up
  // every wave before its first MFMA: a step of a lone workgroup took 1.07 us
  // with 4 waves, d = 128, and now takes 0.90 us.)
  auto next_pages = [&](int s) __attribute__((always_inline)) {
    const int32_t id_prev = id_cur;
    id_cur = __builtin_amdgcn_readlane(idv, s & 63);
    // pinned to scalar registers here: left to itself the compiler moves the
    // products to the copies and spills 130 vector registers
    kpage = kbase + (int64_t)id_cur * ksb;
    vpage = vbase + (int64_t)id_prev * vsb;
    asm volatile("" : "+s"(kpage), "+s"(vpage));
  };
  // before next_pages(s) at multiples of 64: the next 64 ids move in
  auto move_ids = [&](int s) __attribute__((always_inline)) {
    if ((s & 63) == 0) {
      idv = idv_next;
      if (s + 64 < n) idv_next = load_ids(s + 64);
    }
  };
  auto copy_k = [&](const char* src, int s) __attribute__((always_inline)) {
    char* kd = kbuf(s) + bslot * T::kPage;
#pragma unroll
    for (int q = 0; q < T::kDmaPerPage; ++q) dma16(src, kgo[q], kd + q * 1024);
  };
  auto copy_v = [&](const char* src, int s) __attribute__((always_inline)) {
    char* vd = vbuf(s) + bslot * T::kPage;
#pragma unroll
    for (int q = 0; q < T::kDmaPerPage; ++q) dma16(src + q * vgq, vgo0, vd + q * 1024);
  };
  // copies of iteration j, both steps whole
  auto copy_whole = [&](int j) __attribute__((always_inline)) {
    if (!copier) return;
    copy_k(kpage, j + 2);
    copy_v(vpage, j + 1);
  };
  // K of step sk and V of step sv where either may end inside the step or lie past the end
  auto copy_any = [&](const char* ksrc, int sk, const char* vsrc, int sv) {
    if (!copier) return;
    const int kb = w.kv_lo + bslot * kBlockSize;
    if (kb + sk * kKvStep < w.kv_hi) copy_k(ksrc, sk);
    if (sv < n) {
      if (kb + sv * kKvStep < w.kv_hi) {
        copy_v(vsrc, sv);
      } else {
#pragma unroll
        for (int q = 0; q < T::kDmaPerPage; ++q)
          *reinterpret_cast<uint4*>(vbuf(sv) + bslot * T::kPage + q * 1024 + lane * 16) = make_uint4(0, 0, 0, 0);
      }
    }
  };

  const float c = p.scale_log2;  // > 0
  float m_ref = -__builtin_inff(), l_run = 0.0f;
  f32x16 oacc[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.0f;
  const int krow_m = swap_bits23(ln);                 // key row of MFMA row ln (tile kt adds 32)
  const int vsw = (hl ^ ((ln >> 3) & 1)) * 16;        // V half swizzle of channel dt*32 + ln
  constexpr int kQk = 2 * (D / 16);                   // QK MFMAs per step, ordered (kk, kt)
  constexpr int kPv = 4 * (D / 32);                   // PV MFMAs per step, ordered (ks, dt)
  constexpr int kElPerQk = 32 / kQk;                  // scores handled per QK MFMA
  constexpr int kElPerPv = 32 / kPv;                  // scores handled per V operand
  constexpr int kAhead = 3;                           // operand reads issued ahead of their MFMA

  // K operand of QK MFMA i of step s (register i of a lane: key row kt*32 + krow_m)
  auto kread_at = [&](const char* kb, int i) -> bf16x8 {
    const int kk = i >> 1, kt = i & 1;
    const int row = kt * 32 + krow_m;
    return *reinterpret_cast<const bf16x8*>(kb + row * (2 * D) + (((kk * 2 + hl) ^ kswz(row)) * 16));
  };
  auto vread_at = [&](const char* vb, int i) -> bf16x8 {
    const int ks = i / (D / 32), dt = i % (D / 32);
    return *reinterpret_cast<const bf16x8*>(vb + ks * T::kPage + (dt * 32 + ln) * 32 + vsw);
  };
  auto kread = [&](int s, int i) { return kread_at(kbuf(s), i); };
  auto vread = [&](int s, int i) { return vread_at(vbuf(s), i); };
  // the same with the ring stage known at compile time: its offset then
  // folds into the reads' immediate offsets
  auto kread_c = [&](auto st, int i) { return kread_at(smem + decltype(st)::value * T::kBytesK, i); };
  auto vread_c = [&](auto st, int i) {
    return vread_at(smem + 2 * T::kBytesK + decltype(st)::value * T::kBytesV, i);
  };
  // score e (0..31) of a lane sits in tile e/16, register e%16

  f32x16 sbuf[2][2];

  // QK of step s into sbuf[b] (no interleaving; prologue only)
  auto qk_plain = [&](int b, int s) {
#pragma unroll
    for (int i = 0; i < kQk; ++i) {
      const bf16x8 a = kread(s, i);
      const int kk = i >> 1, kt = i & 1;
      if (kk == 0) {
        const f32x16 zero = {};
        sbuf[b][kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[0], zero, 0, 0, 0);
      } else {
        sbuf[b][kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], sbuf[b][kt], 0, 0, 0);
      }
    }
  };
  // causal mask of step s applied to the scores in sbuf[b]
  auto mask_plain = [&](int b, int s) {
    const int lim = pos - (w.kv_lo + s * kKvStep) - hl * 8;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      const float x = sbuf[b][e >> 4][e & 15];
      sbuf[b][e >> 4][e & 15] = ((e >> 4) * 32 + ((e & 15) >> 3) * 16 + (e & 7)) <= lim ? x : -__builtin_inff();
    }
  };
  // weights of the scores in sbuf[b] against the reference max, packed to
  // bf16; ls gets the fp32 sum of the unrounded weights.  (The sum is taken
  // with plain adds: a v_dot2 of the packed weights against (1, 1) would be
  // one instruction per pair, but on gfx950 every dot2 stalls the matrix
  // core's MFMA stream for many cycles, while adds issue beside it.)
  // keep(e, w0, w1) gets each pair of unrounded weights.
  auto weights_plain = [&](int b, uint32_t (&pk)[16], float& ls, auto&& keep) {
    const float nm = m_ref == -__builtin_inff() ? 0.0f : -m_ref;
    ls = 0.0f;
#pragma unroll
    for (int e = 0; e < 32; e += 2) {
      const float w0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sbuf[b][e >> 4][e & 15], c, nm));
      const float w1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sbuf[b][(e + 1) >> 4][(e + 1) & 15], c, nm));
      pk[e >> 1] = pack_bf16x2(w0, w1);
      ls += w0 + w1;
      keep(e, w0, w1);
    }
  };
  // On the step that holds a row's own position (its diagonal step) the
  // row's weights are carried as two bf16 terms: the fp32 weights w are kept
  // (in sbuf[1]; with precise weights in place of the scores) and the PV
  // product runs on hi = bf16(w) and on lo = bf16(w - hi)
  // (w - hi is exact in fp32), so hi + lo is within 2^-18 of w.  The
  // diagonal step holds a row's latest keys, and a row near the start of
  // the sequence has all its keys there: few keys then carry all the
  // weight, and a bf16 weight alone would move such a row's output by up to
  // about 2^-9 |v_i - v_j|.  Which steps do this depends on the row's own
  // position only (not on the rows sharing its wave), so a row's result
  // does not depend on its tile.
  auto weights_inplace = [&](int b) {
    const float nm = m_ref == -__builtin_inff() ? 0.0f : -m_ref;
#pragma unroll
    for (int e = 0; e < 32; ++e)
      sbuf[b][e >> 4][e & 15] = __builtin_amdgcn_exp2f(__builtin_fmaf(sbuf[b][e >> 4][e & 15], c, nm));
  };
  // packed bf16 lo terms of the weights e, e+1 held in sbuf[b], given their
  // hi terms (zero for a row off its diagonal step: own = false)
  auto lo_pair = [&](int b, int e, uint32_t hi, bool own) {
    const bf16x2 h = __builtin_bit_cast(bf16x2, hi);
    const uint32_t lo =
        pack_bf16x2(sbuf[b][e >> 4][e & 15] - (float)h[0], sbuf[b][(e + 1) >> 4][(e + 1) & 15] - (float)h[1]);
    return own ? lo : 0u;
  };
  // packed bf16 hi and lo terms of the weights e, e+1 held in sbuf[b]
  auto hi_lo_pair = [&](int b, int e, uint32_t& hi, uint32_t& lo) {
    hi = pack_bf16x2(sbuf[b][e >> 4][e & 15], sbuf[b][(e + 1) >> 4][(e + 1) & 15]);
    lo = lo_pair(b, e, hi, true);
  };
  // largest score of a lane in sbuf[b]
  auto step_max = [&](int b) {
    float mx = -__builtin_inff();
#pragma unroll
    for (int e = 0; e < 32; ++e) mx = fmaxf(mx, sbuf[b][e >> 4][e & 15]);
    return mx;
  };
  // moves the reference of the rows whose max (mx: a lane's) exceeds it by
  // more than 2^8 and rescales their sums; whether any did (wave-uniform)
  auto move_reference = [&](float mx) -> bool {
    const float m_blk = pair_max(mx) * c;
    const bool grow = m_blk > m_ref + kRescaleLog2;
    if (!__any(grow)) return false;
    const float alpha = grow ? __builtin_amdgcn_exp2f(m_ref - m_blk) : 1.0f;
    m_ref = grow ? m_blk : m_ref;
    l_run *= alpha;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) oacc[dt] *= alpha;
    return true;
  };
  // The row max is only taken when the weights of a step may have outgrown
  // the reference: a lane's step sum reached 2^7, or the row has no
  // reference yet.  A row whose max exceeds the reference by more than 2^8
  // (in log2 units) holds a weight >= 2^8, so its lane's sum passes 2^7:
  // the reference moves exactly as if the max were taken every step.  The
  // weights are then recomputed against the new reference.
  // (reweigh recomputes the step's weights and their sum ls.)
  auto settle = [&](int b, float ls, auto&& reweigh) {
    if (__any(!(ls < kSettleSum) || m_ref == -__builtin_inff())) {  // wave-uniform
      if (move_reference(step_max(b))) reweigh();
    }
  };

  // One step j < nw - 1 that needs no mask, its scores in sbuf[B].  Step j+1
  // may need one (not with precise weights, which take its row max here): its
  // scores leave unmasked and the caller masks them.
  //   block 1: QK of step j+1 into sbuf[1-B], interleaved with the weights of
  //            step j; then settle the weights of step j (rarely does work)
  //   block 2: PV of step j, with the page addresses of the next copies
  // The source order is fixed with scheduling fences.  j has the parity of
  // B (the paired loop starts at step 0), so step j+1's K sits in ring stage
  // 1-B and step j's V in stage B.
  // With precise weights the fp32 weights stay in sbuf[B] in place of the
  // scores, so the reference must be settled before them: block 2 takes the
  // row max of step j+1 beside its MFMAs, and every V operand it reads feeds
  // the hi and the lo product (the lo terms of the next 16 keys are formed
  // meanwhile).  Against unpipelined steps with a second pass over V: the
  // 8 x 8192 workload 2042 -> 1947 us, 32-token segments at 4K 1510 -> 1408 us;
  // at d = 64, where vector instructions bound the step, 299 -> 298 us.
  auto fused = [&](auto bsel, auto&& addresses) {
    constexpr int B = decltype(bsel)::value, NB = 1 - B;
    const float nm = m_ref == -__builtin_inff() ? 0.0f : -m_ref;
    uint32_t pk[16];
    float ls = 0.0f;
    // block 1.  The vector work of a score is spread over three MFMAs (its FMA
    // beside MFMA i - 1, its exponential beside i, pack and sum beside i + 1),
    // so that no instruction waits for the one before it; the last slots read
    // the first V operands.  (Suffix recompute at 1K 20.4 -> 19.8 us, 256-row
    // tiles +0.3 to +1.1%.  Two 4-wave workgroups on a CU, free to drift apart,
    // fill each other's gaps and lose up to 1% by it: they keep the scores of a
    // slot together.)
    constexpr bool kSpread = W == 8 || kHelp;
    bf16x8 ka[kQk], va[kPv];
    float x[32];
    auto scale_score = [&](int e) { x[e] = __builtin_fmaf(sbuf[B][e >> 4][e & 15], c, nm); };
    auto finish_pair = [&](int e) {
      if constexpr (kPrecise) {
        sbuf[B][e >> 4][e & 15] = x[e];
        sbuf[B][(e + 1) >> 4][(e + 1) & 15] = x[e + 1];
      } else {
        pk[e >> 1] = pack_bf16x2(x[e], x[e + 1]);
      }
      ls += x[e] + x[e + 1];
    };
#pragma unroll
    for (int a = 0; a < kAhead; ++a) ka[a] = kread_c(std::integral_constant<int, NB>{}, a);
#pragma unroll
    for (int i = 0; i < kQk; ++i) {
      if (i + kAhead < kQk) ka[i + kAhead] = kread_c(std::integral_constant<int, NB>{}, i + kAhead);
      else if (kSpread) va[i + kAhead - kQk] = vread_c(std::integral_constant<int, B>{}, i + kAhead - kQk);
      const int kk = i >> 1, kt = i & 1;
      if (kk == 0) {
        const f32x16 zero = {};
        sbuf[NB][kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i], qf[0], zero, 0, 0, 0);
      } else {
        sbuf[NB][kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i], qf[kk], sbuf[NB][kt], 0, 0, 0);
      }
      const int e0 = i * kElPerQk;
      if (kSpread && i > 0) {
#pragma unroll
        for (int u = 0; u < kElPerQk; u += 2) finish_pair(e0 - kElPerQk + u);
      }
#pragma unroll
      for (int u = 0; u < kElPerQk; ++u) {
        if (!kSpread || i == 0) scale_score(e0 + u);
        x[e0 + u] = __builtin_amdgcn_exp2f(x[e0 + u]);
        if (!kSpread && (u & 1)) finish_pair(e0 + u - 1);
      }
      if (kSpread && i + 1 < kQk) {
#pragma unroll
        for (int u = 0; u < kElPerQk; ++u) scale_score(e0 + kElPerQk + u);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (kSpread) {
#pragma unroll
      for (int e = 32 - kElPerQk; e < 32; e += 2) finish_pair(e);
    }
    if constexpr (!kPrecise) settle(B, ls, [&]() { weights_plain(B, pk, ls, [](int, float, float) {}); });
    l_run += ls;
    // block 2
    constexpr int kPairs = 4 / (D / 32);  // hi and lo pairs of the next 16 keys formed per V operand
    uint32_t pl[16];
    float mx = -__builtin_inff();
    if constexpr (kPrecise) {
#pragma unroll
      for (int u = 0; u < 4; ++u) hi_lo_pair(B, 2 * u, pk[u], pl[u]);
    }
    if (!kSpread) {
#pragma unroll
      for (int a = 0; a < kAhead; ++a) va[a] = vread_c(std::integral_constant<int, B>{}, a);
    }
#pragma unroll
    for (int i = 0; i < kPv; ++i) {
      if (i + kAhead < kPv) va[i + kAhead] = vread_c(std::integral_constant<int, B>{}, i + kAhead);
      const int ks = i / (D / 32), dt = i % (D / 32);
      // P sub-step ks = keys 16*ks + hl*8 .. +8 = packed weights 4*ks .. 4*ks+3
      // (precise: the pairs of sub-step ks + 1 are formed beside the MFMAs of ks)
      const bf16x8 pb = __builtin_bit_cast(bf16x8, make_uint4(pk[4 * ks], pk[4 * ks + 1], pk[4 * ks + 2], pk[4 * ks + 3]));
      oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], pb, oacc[dt], 0, 0, 0);
      if constexpr (kPrecise) {
        const bf16x8 pc = __builtin_bit_cast(bf16x8, make_uint4(pl[4 * ks], pl[4 * ks + 1], pl[4 * ks + 2], pl[4 * ks + 3]));
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], pc, oacc[dt], 0, 0, 0);
        if (ks < 3) {
#pragma unroll
          for (int u = 4 * (ks + 1) + dt * kPairs; u < 4 * (ks + 1) + (dt + 1) * kPairs; ++u) hi_lo_pair(B, 2 * u, pk[u], pl[u]);
        }
#pragma unroll
        for (int e = i * kElPerPv; e < (i + 1) * kElPerPv; ++e) mx = fmaxf(mx, sbuf[NB][e >> 4][e & 15]);
      }
      if (i == 0) addresses();
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kPrecise) move_reference(mx);
  };

  // Step s's K sits in K buffer s % 2 and its V in V buffer s % 2; in
  // iteration j the copies of K_{j+2} and V_{j+1} are issued after the
  // barrier that ended iteration j-1 (the buffers' previous contents K_j and
  // V_{j-1} were last read before it) and waited for before the barrier that
  // ends iteration j.
  next_pages(0);
  copy_any(kbase + (int64_t)id_cur * ksb, 0, vbase + (int64_t)id_cur * vsb, 0);
  next_pages(1);
  copy_any(kpage, 1, vbase, n);
  next_pages(2);
  // wave-wide smallest and largest causal limit: a tile's rows are in
  // ascending position, so those of its first and last row
  const int nvalid = __builtin_popcountll(__ballot(valid)) >> 1;  // rows (both lane halves hold them)
  const int pmin = nvalid > 0 ? __builtin_amdgcn_readfirstlane(pos) : INT_MAX;
  const int pmax = nvalid > 0 ? __builtin_amdgcn_readlane(pos, nvalid - 1) : -1;
  // (>=: a step whose last key is some row's position counts too, so that
  // every row's diagonal step runs through the masked path)
  auto need_mask = [&](int s) { return w.kv_lo + s * kKvStep + kKvStep - 1 >= pmin; };
  // steps this wave computes: keys up to its largest position.  A wave past
  // them still copies its share of every step and meets every barrier.
  const int nw = pmax >= w.kv_lo ? min(n, (pmax - w.kv_lo) / kKvStep + 1) : 0;
  wait_dma<0>();
  lds_barrier();
  if (nw > 0) {
    qk_plain(0, 0);
    if (need_mask(0)) mask_plain(0, 0);
    if constexpr (kPrecise) move_reference(step_max(0));
  }
  lds_barrier();  // every wave is done with K_0 before K_2 replaces it

  // Iterations run in three parts.  The first handles two steps per trip
  // while both steps and their successors need no mask (the scores of step j
  // alternate between sbuf[0] and sbuf[1], so a trip starts and ends with
  // them in sbuf[0]).  The second pipelines the one or two steps without a
  // mask that may remain.  The third handles the diagonal steps and the last
  // one at a time, with every step's scores in sbuf[0].  Waves may split their
  // steps differently between the parts; every step still ends with exactly
  // one barrier.
  auto tail = [&]() {
    wait_dma<0>();
    lds_barrier();
  };
  int j = 0;
  const int whole = (w.kv_hi - w.kv_lo) / kKvStep;  // steps without a missing block
  for (; j + 2 < nw && !need_mask(j + 2); j += 2) {
    copy_whole(j);  // step j+2 is not masked, hence whole
    fused(std::integral_constant<int, 0>{}, [&]() { next_pages(j + 3); });
    tail();
    if (j + 3 < whole) copy_whole(j + 1);
    else copy_any(kpage, j + 3, vpage, j + 2);
    move_ids(j + 4);
    fused(std::integral_constant<int, 1>{}, [&]() { next_pages(j + 4); });
    tail();
  }
  // One or two steps without a mask may remain before the diagonal ones: the
  // same, with the next step's mask after its scores.  (With precise weights
  // the pipelined step takes the next step's row max, so that one must need no
  // mask either.)  A 3-step item of a helped workgroup 9.9 -> 8.9 us.
  if (j + 1 < nw && !need_mask(kPrecise ? j + 1 : j)) {
    copy_any(kpage, j + 2, vpage, j + 1);
    fused(std::integral_constant<int, 0>{}, [&]() { next_pages(j + 3); });
    if (!kPrecise && need_mask(j + 1)) mask_plain(1, j + 1);
    tail();
    ++j;
    if (!kPrecise && j + 1 < nw && !need_mask(j)) {
      copy_any(kpage, j + 2, vpage, j + 1);
      move_ids(j + 3);
      fused(std::integral_constant<int, 1>{}, [&]() { next_pages(j + 3); });
      if (need_mask(j + 1)) mask_plain(0, j + 1);
      tail();
      ++j;
    } else {
      sbuf[0][0] = sbuf[1][0];
      sbuf[0][1] = sbuf[1][1];
    }
  }
  // Remaining steps (the diagonal ones and the last) run without overlap:
  // weights of step j, PV of step j, then QK + mask of step j+1 into the
  // same score registers.  Same copy schedule as the pipelined loop.
  // On a masked step (split: the diagonal step of some row of the wave) the
  // rows whose diagonal step it is also enter their weights' bf16 lo terms
  // (other rows: zeros), in a second PV pass after the usual one on pk.
  // With precise weights every row enters them on every step, V operand by V
  // operand as in the pipelined loop (the same sums in the same order).
  auto plain_precise = [&](int jj) {
    weights_inplace(0);
    float ls = 0.0f;
#pragma unroll
    for (int e = 0; e < 32; e += 2) ls += sbuf[0][e >> 4][e & 15] + sbuf[0][(e + 1) >> 4][(e + 1) & 15];
    l_run += ls;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      uint32_t ph[4], pl[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) hi_lo_pair(0, 8 * ks + 2 * u, ph[u], pl[u]);
      const bf16x8 pb = __builtin_bit_cast(bf16x8, make_uint4(ph[0], ph[1], ph[2], ph[3]));
      const bf16x8 pc = __builtin_bit_cast(bf16x8, make_uint4(pl[0], pl[1], pl[2], pl[3]));
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) {
        const bf16x8 a = vread(jj, ks * (D / 32) + dt);
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb, oacc[dt], 0, 0, 0);
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pc, oacc[dt], 0, 0, 0);
      }
    }
    if (jj + 1 < nw) {
      qk_plain(0, jj + 1);
      if (need_mask(jj + 1)) mask_plain(0, jj + 1);
      move_reference(step_max(0));
    }
  };
  auto plain = [&](int jj, bool split) {
    uint32_t pk[16];
    float ls;
    auto weigh = [&]() {
      weights_plain(0, pk, ls, [&](int e, float w0, float w1) {  // the fp32 weights stay in sbuf[1]
        sbuf[1][e >> 4][e & 15] = w0;
        sbuf[1][(e + 1) >> 4][(e + 1) & 15] = w1;
      });
    };
    weigh();
    settle(0, ls, weigh);
    const int s_lo = w.kv_lo + jj * kKvStep;
    const bool own = pos >= s_lo && pos < s_lo + kKvStep;  // this is the row's diagonal step
    l_run += ls;
#pragma unroll
    for (int i = 0; i < kPv; ++i) {
      const int ks = i / (D / 32), dt = i % (D / 32);
      const bf16x8 pb = __builtin_bit_cast(bf16x8, make_uint4(pk[4 * ks], pk[4 * ks + 1], pk[4 * ks + 2], pk[4 * ks + 3]));
      oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vread(jj, i), pb, oacc[dt], 0, 0, 0);
    }
    if (split) {
#pragma unroll
      for (int i = 0; i < kPv; ++i) {
        const int ks = i / (D / 32), dt = i % (D / 32);
        uint32_t pl[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) pl[u] = lo_pair(1, 8 * ks + 2 * u, pk[4 * ks + u], own);
        const bf16x8 pc = __builtin_bit_cast(bf16x8, make_uint4(pl[0], pl[1], pl[2], pl[3]));
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vread(jj, i), pc, oacc[dt], 0, 0, 0);
      }
    }
    if (jj + 1 < nw) {
      qk_plain(0, jj + 1);
      if (need_mask(jj + 1)) mask_plain(0, jj + 1);
    }
  };
  for (; j < n; ++j) {
    copy_any(kpage, j + 2, vpage, j + 1);
    move_ids(j + 3);
    next_pages(j + 3);
    if (j < nw) {
      if constexpr (kPrecise) plain_precise(j);
      else plain(j, need_mask(j));
    }
    tail();
  }

  // epilogue: lane (hl, ln) holds row r, channels dt*32 + (i/4)*8 + hl*4 + i%4
  const float l_tot = pair_sum(l_run);
  if (!valid) return;
  if (w.out_slot < 0) {
    const float inv = 1.0f / l_tot;
    uint16_t* orow = p.o + (int64_t)tok * p.o_st + (int64_t)head * p.o_sh;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const uint2 v = make_uint2(pack_bf16x2(oacc[dt][g4 * 4 + 0] * inv, oacc[dt][g4 * 4 + 1] * inv),
                                   pack_bf16x2(oacc[dt][g4 * 4 + 2] * inv, oacc[dt][g4 * 4 + 3] * inv));
        *reinterpret_cast<uint2*>(orow + dt * 32 + g4 * 8 + hl * 4) = v;
      }
    if (p.lse && hl == 0)
      p.lse[(int64_t)tok * p.num_q_heads + head] = (m_ref + __log2f(l_tot)) * kLn2;
  } else {
    float* slot = p.ws + (int64_t)w.out_slot * kRows * (D + 1);
    const bool empty = !(l_tot > 0.0f);  // no visible key in this split
    const float inv = empty ? 0.0f : 1.0f / l_tot;
    float* orow = slot + r * D;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        f32x4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = oacc[dt][g4 * 4 + q] * inv;
        *reinterpret_cast<f32x4*>(orow + dt * 32 + g4 * 8 + hl * 4) = v;
      }
    if (hl == 0)
      slot[kRows * D + r] = empty ? -__builtin_inff() : (m_ref + __log2f(l_tot)) * kLn2;
  }
}

// Persistent launch: workgroup i runs its first item, which lies in its head
// so that no second load has to wait for the list's bounds, then the items
// heads[i].rest .. heads[i].end-1.
template <int D, int W, bool kPrecise>
__global__ __launch_bounds__(64 * W, 2) void msa_attn_kernel(AttnParams p) {
  using T = Tile<D>;
  // K ring (2 steps) then V ring (2 steps); K runs one step ahead of V
  __shared__ __attribute__((aligned(1024))) char smem[2 * T::kBytesK + 2 * T::kBytesV];
  const WgHead head = p.heads[blockIdx.x];
  WorkItem w = head.first;
  for (int it = head.rest;; w = p.work[it++]) {
    attn_item<D, W, kPrecise, false>(p, w, smem);
    if (it >= head.end) break;
  }
}

// The same for 128-row tiles in a launch of no more workgroups than CUs: four
// further waves that only copy.  Alone on its CU, a 4-wave workgroup issues its
// copies (402 of a step's 2430 cycles) with nothing to run beside them; the
// helpers need the registers of a second workgroup, which such a launch does
// not place.  Suffix recompute at 1K, 144 tiles: 22.3 -> 20.4 us; 192 tiles at
// 0.8K keys 20.4 -> 18.7 us.
template <int D, bool kPrecise>
__global__ __launch_bounds__(512, 2) void msa_helped_kernel(AttnParams p) {
  using T = Tile<D>;
  __shared__ __attribute__((aligned(1024))) char smem[2 * T::kBytesK + 2 * T::kBytesV];
  const WgHead head = p.heads[blockIdx.x];
  WorkItem w = head.first;
  for (int it = head.rest;; w = p.work[it++]) {
    attn_item<D, 4, kPrecise, true>(p, w, smem);
    if (it >= head.end) break;
  }
}

// msa_decode: tiles of up to 32 rows (decode-like plans).  Every wave of the
// 4-wave workgroup holds the same 32 rows; wave w takes the 32-key
// half-steps w, w + 4, w + 8, ... of the item's key range and reads their K
// and V straight from the cache into MFMA operand registers.  A tile this
// small gains nothing from sharing K/V between waves through LDS, and
// registers hold more bytes in flight: each wave keeps the K of its next
// half-step and the V of its current one loading while it computes.  The
// four partial softmax states (max, sum, O) are merged through LDS at the
// end.  Arithmetic per half-step is that of the main kernel: S^T = K Q^T
// with K's rows permuted (bits 2 and 3 swapped), the lazy reference max,
// bf16 weights for the PV product and a row sum of the fp32 weights.
template <int D>
struct DecodeLds {
  static constexpr int kWaves = 4;
  static constexpr int kOPad = D + 4;  // row stride of the partial O (bank spread)
  float mo[kWaves][32][kOPad];
  float mm[kWaves][32], ml[kWaves][32];
};

// One work item of msa_decode; the LDS merge area is reused by the next item
// only after the barrier the caller places between items.
template <int D, bool kPrecise>
__device__ __forceinline__ void decode_item(const AttnParams& p, const WorkItem w, DecodeLds<D>& lds) {
  constexpr int kWaves = DecodeLds<D>::kWaves, kHalf = 32;
  auto& mo = lds.mo;
  auto& mm = lds.mm;
  auto& ml = lds.ml;
  if (w.nrows == 0) return;  // (uniform over the workgroup)

  // lane-dependent set-up is computed per item (an opaque copy of the
  // thread id keeps it from being hoisted and held across items)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, hl = lane >> 5, ln = lane & 31;
  const int G = p.group;
  const int t = div_group(ln, p), hh = ln - t * G;  // tile row ln <-> token t, head hh of the group
  const bool valid = t < w.nrows;
  const int tok = w.row0 + t;
  const int head = w.kv_head * G + hh;

  // The two blocks of half-step h.  The second one is only read when it
  // holds a key of the range; otherwise the first one stands in (its keys
  // are then past every row's position, hence masked).  The ids of this
  // wave's first 64 half-steps (h = wave + 4i) are loaded once, lane i
  // holding those of half-step i, so that no half-step waits for a table
  // read, and before everything else of the item; later half-steps read the
  // table directly.
  const int32_t* bt = p.block_table + (int64_t)w.seq * p.max_blocks;
  const int nh = (w.kv_hi - w.kv_lo + kHalf - 1) / kHalf;  // (an item's keys end at its last row's position or before)
  auto table_blocks = [&](int h, int32_t& id0, int32_t& id1) {
    const int k0 = w.kv_lo + h * kHalf;
    id0 = bt[k0 >> 4];
    id1 = k0 + kBlockSize < w.kv_hi ? bt[(k0 >> 4) + 1] : id0;
  };
  int32_t idv0 = 0, idv1 = 0;
  if (wave + kWaves * lane < nh) table_blocks(wave + kWaves * lane, idv0, idv1);

  const int pos = valid ? p.row_pos[tok] : -1;
  bf16x8 qf[D / 16];
  {
    const uint16_t* qrow = p.q + (int64_t)tok * p.q_st + (int64_t)head * p.q_sh + hl * 8;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      if (valid) {
        qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + kk * 16);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) qf[kk][j] = (__bf16)0.0f;
      }
    }
  }

  const char* kbase = reinterpret_cast<const char*>(p.k + (int64_t)w.kv_head * p.k_sh);
  const char* vbase = reinterpret_cast<const char*>(p.v + (int64_t)w.kv_head * p.v_sh);
  const int64_t ksb = p.k_sb * 2, vsb = p.v_sb * 2;  // bytes per block
  const int krow = swap_bits23(ln);                   // key (0..31 in the half-step) of MFMA row ln
  // per-lane byte offsets inside a block: K row krow % 16 at channel hl*8
  // (+ kk*16 per fragment); V^T row (channel) ln at keys hl*8 (+ dt*32 rows)
  const uint32_t koff = (uint32_t)((krow & 15) * p.k_st + hl * 8) * 2u;
  const uint32_t voff = (uint32_t)(ln * p.v_sd + hl * 8) * 2u;
  const uint32_t vdt = (uint32_t)(32 * p.v_sd) * 2u;

  auto blocks = [&](int h, int64_t& id0, int64_t& id1) __attribute__((always_inline)) {
    const int i = (h - wave) / kWaves;  // wave-uniform
    if (i < 64) {
      id0 = __builtin_amdgcn_readlane(idv0, i);
      id1 = __builtin_amdgcn_readlane(idv1, i);
    } else {
      int32_t a, b;
      table_blocks(h, a, b);
      id0 = a;
      id1 = b;
    }
  };
  constexpr int kQk = D / 16;       // QK MFMAs per half-step
  constexpr int kPv = 2 * (D / 32); // PV MFMAs per half-step, ordered (ks, dt)
  bf16x8 ka[2][kQk], va[kPv];
  auto load_k = [&](auto bsel, int h) __attribute__((always_inline)) {
    constexpr int b = decltype(bsel)::value;
    int64_t id0, id1;
    blocks(h, id0, id1);
    const char* kb = kbase + (krow >= 16 ? id1 : id0) * ksb + koff;
#pragma unroll
    for (int kk = 0; kk < kQk; ++kk) ka[b][kk] = *reinterpret_cast<const bf16x8*>(kb + kk * 32);
  };
  auto load_v = [&](int h) __attribute__((always_inline)) {
    int64_t id0, id1;
    blocks(h, id0, id1);
#pragma unroll
    for (int i = 0; i < kPv; ++i) {
      const int ks = i / (D / 32), dt = i % (D / 32);
      va[i] = *reinterpret_cast<const bf16x8*>(vbase + (ks ? id1 : id0) * vsb + voff + dt * vdt);
    }
  };

  const float c = p.scale_log2;
  float m_ref = -__builtin_inff(), l_run = 0.0f;
  f32x16 oacc[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[dt][i] = 0.0f;

  int pmin = 0;  // position of the tile's first row, the smallest (set below, once loads are under way)
  // one half-step h of this wave, its K in buffer b
  auto half = [&](auto bsel, int h) __attribute__((always_inline)) {
    constexpr int b = decltype(bsel)::value;
    load_v(h);
    if (h + kWaves < nh) load_k(std::integral_constant<int, 1 - b>{}, h + kWaves);
    f32x16 sc = {};
#pragma unroll
    for (int kk = 0; kk < kQk; ++kk) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[b][kk], qf[kk], sc, 0, 0, 0);
    // score e (0..15) of a lane is key (e / 8) * 16 + hl * 8 + e % 8 of the half-step
    const int k0 = w.kv_lo + h * kHalf;
    // On the two half-steps of a row's diagonal 64-key step (split) the row
    // also enters its weights' bf16 lo terms, as in the main kernel: a
    // second PV pass on them follows (with precise weights: on every
    // half-step, for every row).
    const bool masked = k0 + kHalf - 1 >= pmin;  // holds some row's position, or passes one
    const bool split = (k0 | (kKvStep - 1)) >= pmin || kPrecise;
    if (masked) {
      const int lim = pos - k0 - hl * 8;
#pragma unroll
      for (int e = 0; e < 16; ++e) sc[e] = ((e >> 3) * 16 + (e & 7)) <= lim ? sc[e] : -__builtin_inff();
    }
    uint32_t pk[8];
    uint32_t plo[kPrecise ? 8 : 1];  // precise weights: the lo terms, taken with the hi ones
    float ls;
    auto weights = [&]() {
      const float nm = m_ref == -__builtin_inff() ? 0.0f : -m_ref;
      ls = 0.0f;
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float w0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e], c, nm));
        const float w1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e + 1], c, nm));
        pk[e >> 1] = pack_bf16x2(w0, w1);
        if constexpr (kPrecise) {
          const bf16x2 hv = __builtin_bit_cast(bf16x2, pk[e >> 1]);
          plo[e >> 1] = pack_bf16x2(w0 - (float)hv[0], w1 - (float)hv[1]);
        }
        ls += w0 + w1;  // fp32 sum (no v_dot2: it stalls the MFMA stream)
      }
    };
    weights();
    // the lazy reference max of the main kernel
    if (__any(!(ls < kSettleSum) || m_ref == -__builtin_inff())) {
      float mx = -__builtin_inff();
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sc[e]);
      const float m_blk = pair_max(mx) * c;
      const bool grow = m_blk > m_ref + kRescaleLog2;
      if (__any(grow)) {
        const float alpha = grow ? __builtin_amdgcn_exp2f(m_ref - m_blk) : 1.0f;
        m_ref = grow ? m_blk : m_ref;
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) oacc[dt] *= alpha;
        weights();
      }
    }
    const bool own = (pos | (kKvStep - 1)) == (k0 | (kKvStep - 1));  // the row's diagonal step
    if (split && !kPrecise) {  // the same weights in fp32, in place of the scores; hi(w) == pk
      const float nm = m_ref == -__builtin_inff() ? 0.0f : -m_ref;
#pragma unroll
      for (int e = 0; e < 16; ++e) sc[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e], c, nm));
    }
    l_run += ls;
#pragma unroll
    for (int i = 0; i < kPv; ++i) {
      const int ks = i / (D / 32), dt = i % (D / 32);
      const bf16x8 pb = __builtin_bit_cast(bf16x8, make_uint4(pk[4 * ks], pk[4 * ks + 1], pk[4 * ks + 2], pk[4 * ks + 3]));
      oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], pb, oacc[dt], 0, 0, 0);
    }
    if (split) {
#pragma unroll
      for (int i = 0; i < kPv; ++i) {
        const int ks = i / (D / 32), dt = i % (D / 32);
        uint32_t pl[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if constexpr (kPrecise) {
            pl[u] = plo[4 * ks + u];
          } else {
            const bf16x2 hv = __builtin_bit_cast(bf16x2, pk[4 * ks + u]);
            pl[u] = own ? pack_bf16x2(sc[8 * ks + 2 * u] - (float)hv[0], sc[8 * ks + 2 * u + 1] - (float)hv[1]) : 0u;
          }
        }
        const bf16x8 pc = __builtin_bit_cast(bf16x8, make_uint4(pl[0], pl[1], pl[2], pl[3]));
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], pc, oacc[dt], 0, 0, 0);
      }
    }
  };
  if (wave < nh) load_k(std::integral_constant<int, 0>{}, wave);
  pmin = __builtin_amdgcn_readfirstlane(pos);
  for (int h = wave; h < nh; h += 2 * kWaves) {
    half(std::integral_constant<int, 0>{}, h);
    if (h + kWaves < nh) half(std::integral_constant<int, 1>{}, h + kWaves);
  }

  // merge the waves' partial states: lane (hl, ln) holds row ln, channels
  // dt*32 + (i/4)*8 + hl*4 + i%4
  const float l_tot = pair_sum(l_run);
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      f32x4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = oacc[dt][g4 * 4 + q];
      *reinterpret_cast<f32x4*>(&mo[wave][ln][dt * 32 + g4 * 8 + hl * 4]) = v;
    }
  if (hl == 0) {
    mm[wave][ln] = m_ref;
    ml[wave][ln] = l_tot;
  }
  __syncthreads();
  constexpr int kCh = D / 8;  // channels per thread: 32 rows x 8 threads
  const int row = tid >> 3, c0 = (tid & 7) * kCh;
  const int rt = div_group(row, p), rh = row - rt * G;
  if (rt >= w.nrows) return;
  float M = -__builtin_inff();
#pragma unroll
  for (int u = 0; u < kWaves; ++u) M = fmaxf(M, mm[u][row]);
  float L = 0.0f, acc[kCh];
#pragma unroll
  for (int q = 0; q < kCh; ++q) acc[q] = 0.0f;
#pragma unroll
  for (int u = 0; u < kWaves; ++u) {
    const float f = mm[u][row] == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(mm[u][row] - M);
    L += f * ml[u][row];
#pragma unroll
    for (int q = 0; q < kCh; q += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&mo[u][row][c0 + q]);
#pragma unroll
      for (int z = 0; z < 4; ++z) acc[q + z] += f * v[z];
    }
  }
  const int otok = w.row0 + rt, ohead = w.kv_head * G + rh;
  if (w.out_slot < 0) {
    const float inv = 1.0f / L;
    uint16_t* orow = p.o + (int64_t)otok * p.o_st + (int64_t)ohead * p.o_sh + c0;
#pragma unroll
    for (int q = 0; q < kCh; q += 4)
      *reinterpret_cast<uint2*>(orow + q) = make_uint2(pack_bf16x2(acc[q] * inv, acc[q + 1] * inv),
                                                       pack_bf16x2(acc[q + 2] * inv, acc[q + 3] * inv));
    if (p.lse && c0 == 0) p.lse[(int64_t)otok * p.num_q_heads + ohead] = (M + __log2f(L)) * kLn2;
  } else {
    const int R = p.slot_rows;
    float* slot = p.ws + (int64_t)w.out_slot * R * (D + 1);
    const bool empty = !(L > 0.0f);  // no visible key in this split
    const float inv = empty ? 0.0f : 1.0f / L;
#pragma unroll
    for (int q = 0; q < kCh; q += 4) {
      f32x4 v;
#pragma unroll
      for (int z = 0; z < 4; ++z) v[z] = acc[q + z] * inv;
      *reinterpret_cast<f32x4*>(slot + row * D + c0 + q) = v;
    }
    if (c0 == 0) slot[(int64_t)R * D + row] = empty ? -__builtin_inff() : (M + __log2f(L)) * kLn2;
  }
}

template <int D, bool kPrecise>
__global__ __launch_bounds__(256, 2) void msa_decode_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(16))) DecodeLds<D> lds;
  const WgHead head = p.heads[blockIdx.x];
  WorkItem w = head.first;
  for (int it = head.rest;; w = p.work[it++]) {
    decode_item<D, kPrecise>(p, w, lds);
    if (it >= head.end) break;
    __syncthreads();  // the item's merge reads are done
  }
}

// msa_merge: one workgroup per (split tile, chunk of kRows rows), D / 4 threads
// to a row, 4 channels each.  Bound by reading the partials; a tile's rows are
// spread over workgroups because a plan may split few tiles into many pieces
// (58 tiles of 128 rows x 29 pieces, d = 128: 212 us with one workgroup per
// tile, about 16 us in this form; 688 tiles x 2-5 pieces: 71 us and 34 us).
// The lse and O of kBatch pieces load together, so that up to
// kBatch pieces cost one memory round trip.
template <int D>
__global__ __launch_bounds__(256) void msa_merge_kernel(MergeParams p) {
  constexpr int kThreadsPerRow = D / 4;
  constexpr int kRows = 256 / kThreadsPerRow;
  constexpr int kBatch = 8;
  const MergeItem mi = p.merge[blockIdx.x];
  const int G = p.group;
  const int r = blockIdx.y * kRows + threadIdx.x / kThreadsPerRow;
  if (r >= mi.nrows * G) return;
  const int sub = threadIdx.x % kThreadsPerRow;
  const int R = p.tile_rows;
  const int64_t slot_f = (int64_t)R * (D + 1);
  const int t = r / G, hh = r - t * G;
  const int tok = mi.row0 + t, head = mi.kv_head * G + hh;
  const float* base = p.ws + (int64_t)mi.slot0 * slot_f;
  float mx = -__builtin_inff(), L = 0.0f;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int s0 = 0; s0 < mi.nsplit; s0 += kBatch) {
    float ls[kBatch];
    f32x4 os[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float* slot = base + (int64_t)min(s0 + u, mi.nsplit - 1) * slot_f;
      ls[u] = slot[(int64_t)R * D + r];
      os[u] = *reinterpret_cast<const f32x4*>(slot + r * D + sub * 4);
    }
    float m_new = mx;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) m_new = fmaxf(m_new, ls[u]);
    const float mu = m_new == -__builtin_inff() ? 0.0f : m_new;
    const float alpha = __builtin_amdgcn_exp2f((mx - mu) * kLog2e);  // 0 on the first batch
    L *= alpha;
    acc *= alpha;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float wgt = s0 + u < mi.nsplit ? __builtin_amdgcn_exp2f((ls[u] - mu) * kLog2e) : 0.0f;
      L += wgt;
      acc += wgt * os[u];
    }
    mx = m_new;
  }
  const float inv = L > 0.0f ? 1.0f / L : 0.0f;
  bf16x4 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = (__bf16)(acc[j] * inv);
  *reinterpret_cast<bf16x4*>(p.o + (int64_t)tok * p.o_st + (int64_t)head * p.o_sh + sub * 4) = v;
  if (p.lse && sub == 0)
    p.lse[(int64_t)tok * p.num_q_heads + head] = (mx == -__builtin_inff() ? 0.0f : mx) + __logf(L);
}

// The precise-weights forms are separate instantiations, so that the
// default kernels carry no test of the flag.
template <bool kPrecise>
int launch_attn_form(const AttnParams& p, int head_dim, int item_rows, int num_wg, hipStream_t s) {
  if (item_rows == kTileRowsNarrow && num_wg <= kCUs && head_dim == 128)
    hipLaunchKernelGGL((msa_helped_kernel<128, kPrecise>), dim3(num_wg), dim3(512), 0, s, p);
  else if (item_rows == kTileRowsNarrow && num_wg <= kCUs && head_dim == 64)
    hipLaunchKernelGGL((msa_helped_kernel<64, kPrecise>), dim3(num_wg), dim3(512), 0, s, p);
  else if (head_dim == 128 && item_rows == kTileRowsNarrow)
    hipLaunchKernelGGL((msa_attn_kernel<128, 4, kPrecise>), dim3(num_wg), dim3(256), 0, s, p);
  else if (head_dim == 128 && item_rows == kTileRowsWide)
    hipLaunchKernelGGL((msa_attn_kernel<128, 8, kPrecise>), dim3(num_wg), dim3(512), 0, s, p);
  else if (head_dim == 64 && item_rows == kTileRowsNarrow)
    hipLaunchKernelGGL((msa_attn_kernel<64, 4, kPrecise>), dim3(num_wg), dim3(256), 0, s, p);
  else if (head_dim == 64 && item_rows == kTileRowsWide)
    hipLaunchKernelGGL((msa_attn_kernel<64, 8, kPrecise>), dim3(num_wg), dim3(512), 0, s, p);
  else if (head_dim == 128 && item_rows == kTileRowsDecode)
    hipLaunchKernelGGL((msa_decode_kernel<128, kPrecise>), dim3(num_wg), dim3(256), 0, s, p);
  else if (head_dim == 64 && item_rows == kTileRowsDecode)
    hipLaunchKernelGGL((msa_decode_kernel<64, kPrecise>), dim3(num_wg), dim3(256), 0, s, p);
  else
    return (int)hipErrorInvalidValue;
  return (int)hipGetLastError();
}

}  // namespace

int launch_attn(const AttnParams& p, int head_dim, int item_rows, int num_wg, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (num_wg <= 0) return 0;
  return p.precise ? launch_attn_form<true>(p, head_dim, item_rows, num_wg, s)
                   : launch_attn_form<false>(p, head_dim, item_rows, num_wg, s);
}

int launch_merge(const MergeParams& p, int head_dim, int num_merge, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (num_merge <= 0) return 0;
  const int rows_per_wg = 1024 / head_dim;  // kRows of msa_merge_kernel
  const dim3 grid(num_merge, (p.max_rows + rows_per_wg - 1) / rows_per_wg);
  if (head_dim == 128)
    hipLaunchKernelGGL(msa_merge_kernel<128>, grid, dim3(256), 0, s, p);
  else if (head_dim == 64)
    hipLaunchKernelGGL(msa_merge_kernel<64>, grid, dim3(256), 0, s, p);
  else
    return (int)hipErrorInvalidValue;
  return (int)hipGetLastError();
}

}  // namespace msa
