// Causal attention of bf16 prompt chunks (kernels_attn.hip has the decode attention and the fp32 prompt kernel, and
// describes the cache layout).
//
// One workgroup of eight waves per (block of rows of a sequence, kv head); wave w works for q-head kvh * grp + w % grp
// on a tile of 32 rows.  Two forms:
//  rows: wave group g = w / grp takes a row tile of the block and all its keys.  Half of a block's tiles count from the
//    sequence's first row and half from its last, so that all blocks have about the same number of keys to visit
//    (rows 0..2047 of 32 heads of 128: 112 us with neighbouring tiles, 99 so);
//  keys: groups 2 t and 2 t + 1 share row tile t and take every other key block; they merge their softmax states
//    through LDS at the end.  Twice the workgroups, each with half the serial chain, for twice the loads and barriers
//    per product: for launches that would leave CUs idle.
// Both products are 32x32x16 matrix instructions with the query row in the lane index:
//   S^T = K Q^T (A = K rows, B = Q rows)  and  O^T = V^T P^T (A = V^T rows, B = P rows),
// so a lane (row l & 31, half l >> 5) holds scores, probabilities, softmax state and output columns of one row and
// only the other half shares it.  K rows are read in an order (bits 2 and 3 of the slot swapped) that leaves a lane's
// scores in the registers where the second product needs its probabilities.
//
// What bounds it: the matrix cores (4 x 2 products per slot, hi and lo halves of q and p) and, nearly as much, the
// vector instructions of the softmax.  Those are kept to about 11 per score: scale and maximum enter one fused
// multiply-add before exp2; the running maximum only moves (and rescales the output rows) when some score exceeds it
// by more than 8 powers of two (the conditional rescaling published with FlashAttention-4), so most blocks need no
// exchange between lanes; sums stay in the lane until the end; masks and the zeroing of values past the end run only in
// blocks that reach past the wave's first row.  8B shape,
// 2,048 rows in the prefill of 4 x 32K tokens (kernel trace): at slots 30,720..32,767 2,279 -> 1,833 us, 1,160 TFLOP/s
// executed (16x16x32 products, about 25 vector instructions per score and two exchanges per block before), at slots
// 0..2,047 154 -> 101 us; by counters the matrix cores are busy 0.58 of the cycles there, at 1.94 GHz.
#include "device_common.h"
#include "gemm_epilogue.h"
#include "ham_internal.h"
#include "launch_rules.h"
#include "rows.h"

namespace ham {

typedef float f16v __attribute__((ext_vector_type(16)));

// Key blocks of 32 slots land in LDS straight from memory, two per stage in a ring of NS stages (NS - 1 in flight),
// in whole contiguous 1 KB pieces.  K keeps its rows (16-byte chunk c of slot r at chunk c ^ (r mod row's chunks)),
// V its tile rows (chunk c of row d at c ^ (d / 4 % 4)): the swizzles spread a wave's operand reads over all banks.
template <int HD> struct PA {
  static constexpr int NW = PROMPT_ATTN_WAVES, KB = 32, NBL = 2, NS = 4;
  static constexpr int KC = HD / 8, KU = KB * KC;       // 16-byte chunks per K row, per block
  static constexpr int VU = HD * 4, BU = KU + VU;       // chunks of a V tile, of a block
  static constexpr int PIECES = NBL * BU / 64, LPW = PIECES / NW;  // 1 KB pieces per stage, per wave
  static constexpr int NF = HD / 16, ND = HD / 32;
};

// One block of 32 slots from `base` for this wave's 32 rows.  MASK: slots at or past `limit` (the lane's row) count
// as -inf and values at or past `vlimit` as 0, whatever they hold.
// `load(j)`, j < NLD, issues this wave's loads of a later stage, spread among the products (at the head of a stage they
// would hold back its LDS reads until the address path has taken those of all waves).
template <int HD, bool MASK, int NLD, typename Load>
__device__ __forceinline__ void pa_block(const u4* blk, int base, int limit, int vlimit, const u4* qh, const u4* ql,
                                         float sc, float& mrun, float& lrun, f16v* o, const Load& load) {
  using P = PA<HD>;
  const int lane = threadIdx.x & 63, h = lane >> 5, r = lane & 31;
  f16v s;
#pragma unroll
  for (int e = 0; e < 16; ++e) s[e] = 0.f;
  const int slot = (r & 19) | ((r & 4) << 1) | ((r & 8) >> 1);  // operand row r holds the slot with bits 2, 3 swapped
  __builtin_amdgcn_s_setprio(1);  // products before the other wave's softmax
  const u4* kr = blk + slot * P::KC;
#pragma unroll
  for (int f = 0; f < P::NF; ++f) {
    const bf16x8 k = __builtin_bit_cast(bf16x8, kr[(2 * f + h) ^ (slot % P::KC)]);
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, __builtin_bit_cast(bf16x8, qh[f]), s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, __builtin_bit_cast(bf16x8, ql[f]), s, 0, 0, 0);
    if (f % (P::NF / NLD) == 0) {
      __builtin_amdgcn_sched_barrier(0);
      load(f / (P::NF / NLD));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __builtin_amdgcn_s_setprio(0);
  if constexpr (MASK) {
#pragma unroll
    for (int e = 0; e < 16; ++e)  // score e: slot 16 (e / 8) + 8 h + e % 8
      if (base + 16 * (e >> 3) + 8 * h + (e & 7) >= limit) s[e] = -INFINITY;
  }
  float bm = s[0];
#pragma unroll
  for (int e = 1; e < 16; ++e) bm = fmaxf(bm, s[e]);
  bm *= sc;  // sc > 0
  if (__any(bm > mrun + 8.f)) {
    bm = fmaxf(bm, __shfl_xor(bm, 32, WAVE));
    const float mnew = fmaxf(mrun, bm);
    const float alpha = mnew == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(mrun - mnew);  // 0 from the initial -inf
    lrun *= alpha;
#pragma unroll
    for (int d = 0; d < P::ND; ++d)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[d][e] *= alpha;
    mrun = mnew;
  }
  const float mref = mrun == -INFINITY ? 0.f : mrun;  // no score above -inf yet: probabilities 0
  float p[16], ps = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(s[e], sc, -mref));
#pragma unroll
  for (int e = 0; e < 16; ++e) ps += p[e];
  lrun += ps;
  u4 ph[2], pl[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    ph[t] = pack_frag_bf16(p + 8 * t);
    float lo[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      lo[e] = p[8 * t + e] - __uint_as_float((e & 1) ? (ph[t][e >> 1] & 0xFFFF0000u) : (ph[t][e >> 1] << 16));
    pl[t] = pack_frag_bf16(lo);
  }
  __builtin_amdgcn_s_setprio(1);
  const u4* vr = blk + P::KU;
#pragma unroll
  for (int d = 0; d < P::ND; ++d)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      u4 v = vr[(d * 32 + r) * 4 + ((2 * t + h) ^ ((r >> 2) & 3))];
      if constexpr (MASK) {
        const int keep = vlimit - (base + 16 * t + 8 * h);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e >= keep) v[e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
      }
      o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, ph[t]), o[d], 0, 0, 0);
      o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pl[t]), o[d], 0, 0, 0);
    }
}

template <int HD, bool KEYS>
__global__ __launch_bounds__(512, 2) void k_attn_prompt(AttnArgs a) {
  using P = PA<HD>;
  constexpr int NS = P::NS, LPW = P::LPW, KB = P::KB;
  __shared__ u4 lds[NS][P::NBL * P::BU];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kvh = blockIdx.y;
  const int grp = a.H / a.Hkv, nrg = P::NW / grp / (KEYS ? 2 : 1);
  const int jh = w % grp, rg = w / grp / (KEYS ? 2 : 1), kg = KEYS ? w / grp % 2 : 0;
  const int head = kvh * grp + jh;
  // rows [lo, hi) of the launch belong to sequence b; the blocks with the most keys start first
  const int b = a.rm.b0 + blockIdx.z;
  const int first = (int)blockIdx.z * a.rm.T - a.rm.s0;  // launch row of the sequence's slot 0
  const int lo = max(first, 0), hi = min(first + a.rm.T, a.R);
  const int slot0 = lo - first;                       // slot of row lo
  const int nt = (hi - lo + 31) / 32;                 // row tiles
  int tile, last;                                     // this wave's tile (-1: none), the last of the workgroup
  if constexpr (KEYS) {
    const int t0 = (int)(gridDim.x - 1 - blockIdx.x) * nrg;  // the blocks with the most keys start first
    if (t0 >= nt) return;                             // the same for every wave of the workgroup
    tile = t0 + rg < nt ? t0 + rg : -1;
    last = min(t0 + nrg, nt) - 1;
  } else {
    const int half = nrg / 2, t0 = (int)blockIdx.x * half, t = t0 + rg % half;
    if (2 * t0 >= nt) return;
    tile = rg < half ? (2 * t < nt ? t : -1) : (2 * t < nt - 1 ? nt - 1 - t : -1);
    last = nt - 1 - t0;
  }
  const bool rows_ok = rg < nrg && tile >= 0;         // waves past the q-heads or the rows only load
  const int row0 = lo + max(tile, 0) * 32;
  const int wslot = slot0 + (row0 - lo);              // slot of the wave's first row
  const int wave_end = rows_ok ? wslot + min(32, hi - row0) : 0;
  const int wg_end = slot0 + min((last + 1) * 32, hi - lo);  // keys [0, wg_end)
  const bf16* Kb = (const bf16*)a.K + b * a.sb + kvh * a.sh;
  const bf16* Vb = (const bf16*)a.VT + b * a.sb + kvh * a.sh;

  // this lane's row; rows past the end see slot 0 alone and are not stored
  const int qrow = row0 + (lane & 31);
  const bool qok = rows_ok && qrow < hi;
  const int limit = qok ? wslot + (lane & 31) + 1 : 1;
  u4 qh[P::NF], ql[P::NF];
  const bf16* qp = (const bf16*)a.q + (size_t)(qok ? qrow : 0) * a.ldq * 2 + (size_t)head * HD + (lane >> 5) * 8;
#pragma unroll
  for (int f = 0; f < P::NF; ++f) {
    qh[f] = qok ? ld16(qp + f * 16) : zero16();
    ql[f] = qok ? ld16(qp + a.ldq + f * 16) : zero16();
  }

  const int nblk = (wg_end + KB - 1) / KB, nst = (nblk + P::NBL - 1) / P::NBL;
  // this wave's pieces of a stage: piece w + NW i of 64 chunks; chunk u of a block is K slot u / KC, or V row (u - KU) / 4
  int off[LPW], bl[LPW];
  bool isk[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int u0 = (w + P::NW * i) * 64;
    bl[i] = u0 / P::BU;
    const int u = u0 % P::BU + lane;
    isk[i] = u0 % P::BU < P::KU;
    if (isk[i]) {
      const int sl = u / P::KC, c = u % P::KC;
      off[i] = sl * HD + ((c ^ (sl % P::KC)) * 8);
    } else {
      const int d = (u - P::KU) / 4, c = u % 4;
      off[i] = d * VT_TILE + ((c ^ ((d >> 2) & 3)) * 8);
    }
  }
  // every wave issues exactly LPW loads per stage (blocks past the end re-read the last block, never used), so vmcnt
  // counts stages
  auto issue1 = [&](int st, int i) {
    const int blk = min(st * P::NBL + bl[i], nblk - 1);
    const bf16* src = (isk[i] ? Kb : Vb) + (size_t)blk * KB * HD + off[i];  // a K block and a V tile are as long
    __builtin_amdgcn_global_load_lds((const void*)src,
                                     (__attribute__((address_space(3))) void*)(lds[st % NS] + (w + P::NW * i) * 64), 16, 0, 0);
  };

  f16v o[P::ND];
#pragma unroll
  for (int d = 0; d < P::ND; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[d][e] = 0.f;
  float mrun = -INFINITY, lrun = 0.f;
  const float sc = 1.44269504088896341f / sqrtf((float)HD);  // scores in powers of two
#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < nst) {
#pragma unroll
      for (int i = 0; i < LPW; ++i) issue1(st, i);
    }
  for (int st = 0; st < nst; ++st) {
    // stage st has landed once at most the loads of the stages issued after it are pending
    if (st + NS - 2 < nst) wait_vm_lgkm0<(NS - 2) * LPW>();
    else wait_vm_lgkm0<0>();
    asm volatile("s_barrier" ::: "memory");
    // every wave is past stage st - 1: its slot takes stage st + NS - 1
    constexpr int NB = KEYS ? 1 : P::NBL, NLD = LPW / NB;  // blocks of this wave, loads issued in each
    const bool more = st + NS - 1 < nst;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int bi = KEYS ? kg : i, base = (st * P::NBL + bi) * KB;
      const u4* blk = lds[st % NS] + bi * P::BU;
      const auto load = [&](int j) {
        if (more) issue1(st + NS - 1, i * NLD + j);
      };
      if (rows_ok && base + KB <= wslot + 1) {  // every slot visible to every row
        pa_block<HD, false, NLD>(blk, base, limit, wave_end, qh, ql, sc, mrun, lrun, o, load);
      } else if (base < wave_end) {
        pa_block<HD, true, NLD>(blk, base, limit, wave_end, qh, ql, sc, mrun, lrun, o, load);
      } else {  // blocks past this wave's last row hold nothing it sees
#pragma unroll
        for (int j = 0; j < NLD; ++j) load(j);
      }
    }
  }
  lrun += __shfl_xor(lrun, 32, WAVE);
  if constexpr (KEYS) {  // merge the two waves of a row tile: the second leaves its state in LDS
    constexpr int OV = P::ND * 16;  // output values per lane
    static_assert((size_t)P::NW / 2 * (OV + 2) * 64 * 4 <= sizeof(lds), "merge records");
    __syncthreads();  // every wave is past its last key block
    float* rec = reinterpret_cast<float*>(&lds[0][0]) + (size_t)(rg * grp + jh) * (OV + 2) * 64 + lane;
    if (kg == 1 && rows_ok) {
      rec[0] = mrun;
      rec[64] = lrun;
#pragma unroll
      for (int d = 0; d < P::ND; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) rec[(2 + d * 16 + e) * 64] = o[d][e];
    }
    __syncthreads();
    if (kg == 1 || !rows_ok) return;  // waves without rows (two of eight at three q-heads a kv head) have no record
    {
      const float m1 = rec[0], mnew = fmaxf(mrun, m1);
      const float a0 = mrun == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrun - mnew);
      const float a1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m1 - mnew);
      lrun = lrun * a0 + rec[64] * a1;
#pragma unroll
      for (int d = 0; d < P::ND; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[d][e] = o[d][e] * a0 + rec[(2 + d * 16 + e) * 64] * a1;
    }
  }
  if (!qok) return;
  const float inv = lrun > 0.f ? 1.0f / lrun : 0.f;
  bf16* op = (bf16*)a.o + (size_t)qrow * a.ldo * 2 + (size_t)head * HD + 4 * (lane >> 5);
#pragma unroll
  for (int d = 0; d < P::ND; ++d)
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {  // columns 32 d + 8 e4 + 4 (lane >> 5) + 0..3
      float v[4], l[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = o[d][4 * e4 + e] * inv;
      const uint2 hw = uint2{f2bf2(v[0], v[1]), f2bf2(v[2], v[3])};
      l[0] = v[0] - __uint_as_float(hw.x << 16);
      l[1] = v[1] - __uint_as_float(hw.x & 0xFFFF0000u);
      l[2] = v[2] - __uint_as_float(hw.y << 16);
      l[3] = v[3] - __uint_as_float(hw.y & 0xFFFF0000u);
      *reinterpret_cast<uint2*>(op + d * 32 + e4 * 8) = hw;
      *reinterpret_cast<uint2*>(op + a.ldo + d * 32 + e4 * 8) = uint2{f2bf2(l[0], l[1]), f2bf2(l[2], l[3])};
    }
}

int launch_attn_prompt(const AttnArgs& a, Stream s) {
  if (a.H % a.Hkv != 0 || a.H / a.Hkv > 4 || a.S % 64 != 0 || a.rm.mode != ROWS_PREFILL || a.rm.T < 1 || a.R < 1) return -1;
  const PromptAttnGrid pg = prompt_attn_grid(a.R, a.rm.s0, a.rm.T, a.H, a.Hkv);
  const dim3 grid(pg.blocks, a.Hkv, pg.seqs);
  if (a.hd == 64) {
    if (pg.keys) launch_k((k_attn_prompt<64, true>), grid, dim3(512), 0, s, a);
    else launch_k((k_attn_prompt<64, false>), grid, dim3(512), 0, s, a);
  } else if (a.hd == 128) {
    if (pg.keys) launch_k((k_attn_prompt<128, true>), grid, dim3(512), 0, s, a);
    else launch_k((k_attn_prompt<128, false>), grid, dim3(512), 0, s, a);
  } else {
    return -1;
  }
  return 0;
}

}  // namespace ham
