// The weight GEMM of bf16 prompt chunks: C[m][n] = sum_k X[m][k] * W[n][k] over many rows m (kernels_gemm.hip has
// the other GEMMs and describes the layouts they share).
//
// A 128 x BN output tile per workgroup of eight waves in two groups of four.  Each group covers the whole tile
// (64 x BN/2 per wave, 32x32x16 matrix instructions) over every other k-fragment of the range, one phase apart: in
// phase p group p % 2 reads the operands of stage p from LDS into registers while the matrix instructions of stage
// p - 1, from the other group, run on the same SIMDs.  The groups' accumulators are added through LDS at the end.
//
// What bounds it: the matrix cores at the clock that the power limit leaves them.  The tile costs 64 KB of operand
// reads and 32 KB of arriving operands per stage of 1024 matrix cycles, so a schedule in which all waves read, then
// all multiply (the 128 x 256 tile of four waves before this one) adds the two times: 1,850 cycles per stage at
// 2.25 GHz.  Three things bring it to 1,310 cycles at 1.8 GHz (1,240 and 1.75 GHz with no loads in the loop at all):
// the two groups one phase apart; the loads of a later stage issued by the waves that multiply, one per four matrix
// instructions (issued together at the head of a phase they hold back its LDS reads and its products for the ~500
// cycles that the address path takes for them: 1,850 again); 32x32x16 products.  8B shape, 2,048 rows, in the prefill of
// 4 x 32K tokens against the four-wave tile (kernel trace): gate/up 1,027 -> 799 us, down 573 -> 392, o-projection
// 173 -> 121, q/k/v 222 -> 215; by counters the matrix cores are busy 0.63 of the cycles there, at 1.86 GHz.
#include <algorithm>

#include "device_common.h"
#include "gemm_epilogue.h"
#include "ham_internal.h"

namespace ham {

typedef float f16v __attribute__((ext_vector_type(16)));

// Operand fragments (1 KB in lane order) land in LDS straight from memory (global_load_lds_dwordx4), one k-fragment
// per stage in a ring of D stages.  Stage q is loaded by the waves of group (q + 1) % 2, LPG loads each, so that a
// wave's vmcnt counts the stages of its group.
template <int BN> struct PP {
  static constexpr int BM = 128, KB = 32, EPL = 8;
  static constexpr int NA = BM / 16 * 2, NBW = BN / 16, NL = NA + NBW, LPG = NL / 4;
  static constexpr int D = 5;                        // 160 KB (BN = 256) or 120 KB of LDS
  static constexpr int JT = BN / 64, JK = JT / 2;    // 32-column tiles per wave; kept by a group at the end
  static constexpr int FRAG = 64;                    // u4 per fragment
  static constexpr int CW = 32 * JK, CP = CW + 4;    // columns a wave stores, pitch of its rows in LDS
};

// Output tile of a workgroup (gx x gy tiles).  Workgroups go to the 8 XCDs in turn (linear id mod 8), and each XCD
// has its own L2: the grid is renumbered so that every XCD takes one contiguous range of tiles, ordered in groups of
// PP_GM M-tiles (M fastest), so the ~32 workgroups an XCD runs at once share their X and weight slices in its L2.
constexpr int PP_GM = 4;
__device__ __forceinline__ void pp_tile(int gx, int gy, int& mt, int& nt) {
  const int G = gx * gy;
  int L = blockIdx.x;
  if (G % 8 == 0) L = (L % 8) * (G / 8) + L / 8;
  const int per_group = PP_GM * gx, group = L / per_group, first_m = group * PP_GM;
  const int gsz = min(gy - first_m, PP_GM), r = L - group * per_group;
  mt = first_m + r % gsz;
  nt = r / gsz;
}

__device__ __forceinline__ void pp_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Rows past M read row M - 1 and tiles past N the last tile (never stored).  With gridDim.y > 1 the k-range is split
// and the result is fp32 partials [split][M][N] in a.part that the consumer sums.
template <int EPI, int BN>
__global__ __launch_bounds__(512, 2) void k_gemm_pp(GemmArgs a) {
  if (!any_flag(a.gate, a.gate_n)) return;
  using C = PP<BN>;
  constexpr int BM = C::BM, KB = C::KB, EPL = C::EPL, LPG = C::LPG, D = C::D, JT = C::JT, JK = C::JK, FRAG = C::FRAG;
  __shared__ u4 ring[D][C::NL * FRAG];
  static_assert(sizeof(ring) >= (size_t)8 * 2 * JK * 4 * 64 * 16, "accumulator exchange");
  static_assert((size_t)2 * JK * 4 * 64 * 16 >= (size_t)32 * C::CP * 4, "a wave's rows in LDS");
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = w >> 2, wi = w & 3, wm = wi >> 1, wn = wi & 1;
  const int gx = (a.N + BN - 1) / BN, gy = (a.M + BM - 1) / BM;
  int mt, nt;
  pp_tile(gx, gy, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  const int nfr = a.K / KB, ntile = a.N / 16;
  const int split = blockIdx.y, nsplit = gridDim.y;
  const int c0 = (int)((long)split * nfr / nsplit), n = (int)((long)(split + 1) * nfr / nsplit) - c0;
  // wave wi of a group loads fragments wi + 4 i of a stage: X fragments (tile q / 2, plane q % 2) for i < 4, then
  // weights; its first stage is the group's first
  const bf16* src[LPG];
#pragma unroll
  for (int i = 0; i < LPG; ++i) {
    const int q = wi + 4 * i;
    if (i < 4) {
      const int m = min(m0 + (q >> 1) * 16 + (lane & 15), a.M - 1);
      src[i] = (const bf16*)a.X + ((size_t)m * 2 + (q & 1)) * a.ldx + (size_t)(c0 + (grp ^ 1)) * KB + (lane >> 4) * EPL;
    } else {
      const int t = min(n0 / 16 + (q - C::NA), ntile - 1);
      src[i] = (const bf16*)a.W + ((size_t)t * nfr + c0 + (grp ^ 1)) * FRAG * EPL + (size_t)lane * EPL;
    }
  }
  int islot = grp ^ 1;  // ring slot of the next stage this group loads
  auto issue1 = [&](int i) {
    __builtin_amdgcn_global_load_lds((const void*)src[i],
                                     (__attribute__((address_space(3))) void*)(ring[islot] + (wi + 4 * i) * FRAG), 16, 0, 0);
    src[i] += i < 4 ? 2 * KB : 2 * FRAG * EPL;
  };
  auto slot_next = [](int s) { return s + 2 >= D ? s + 2 - D : s + 2; };
  f16v acc[2][JT];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < JT; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  // 32-row operand from two 16-row fragments: lane l holds row l & 31, k-slice 2 ks + (l >> 5)
  const int lb = (lane >> 5) * 16 + (lane & 15), hb = (lane >> 4) & 1;
  const int xoff = (wm * 4 + hb) * 2 * FRAG + lb, woff = (C::NA + wn * 2 * JT + hb) * FRAG + lb;

  for (int q = grp ^ 1; q < D - 1 && q < n; q += 2) {
#pragma unroll
    for (int i = 0; i < LPG; ++i) issue1(i);
    islot = slot_next(islot);
  }
  if (grp == 1) {  // stage 0 has landed once only this group's stage 2 is pending
    if (2 < n) wait_vm_lgkm0<LPG>();
    else wait_vm_lgkm0<0>();
  }
  pp_barrier();
  if (grp == 1) {  // phase 0 of group 1: loads only
    if (D - 1 < n) {
#pragma unroll
      for (int i = 0; i < LPG; ++i) issue1(i);
      islot = slot_next(islot);
    }
    pp_barrier();
  }
  int rslot = grp;
  for (int p = grp; p < n; p += 2) {
    // phase p: operands of stage p.  Its slot is free again after this phase's barrier (the reads have returned), and
    // stage p + D, loaded in phase p + 1, is the next one to use it.
    const u4* slot = ring[rslot];
    rslot = slot_next(rslot);
    u4 xf[2][2][2], wf[2][JT];  // [k-step][plane][row tile], [k-step][column tile]
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int i = 0; i < 2; ++i) xf[ks][pl][i] = slot[xoff + i * 4 * FRAG + pl * FRAG + ks * 32];
#pragma unroll
      for (int j = 0; j < JT; ++j) wf[ks][j] = slot[woff + j * 2 * FRAG + ks * 32];
    }
    // stage p + 1, which this group loaded, has landed once only its loads of stage p + 3 are pending
    if (p + 3 < n) wait_vm_lgkm0<LPG>();
    else wait_vm_lgkm0<0>();
    pp_barrier();
    // phase p + 1: products of stage p, the loads of stage p + D among them
    const bool more = p + D < n;
    constexpr int NM = 8 * JT, PER = NM / LPG;
#pragma unroll
    for (int q = 0; q < NM; ++q) {
      const int ks = q / (4 * JT), pl = q / (2 * JT) % 2, i = q / JT % 2, j = q % JT;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xf[ks][pl][i]),
                                                          __builtin_bit_cast(bf16x8, wf[ks][j]), acc[i][j], 0, 0, 0);
      if (q % PER == 0 && q / PER < LPG) {
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue1(q / PER);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (more) islot = slot_next(islot);
    pp_barrier();
  }
  // the group with one phase fewer waits for the other's last reads
  if (((n ^ grp) & 1) == 0) pp_barrier();

  // Add the groups: group g keeps column tiles [g JK, (g + 1) JK) of its wave's tile and sends the others through LDS.
  // The wave then passes its 32 x CW blocks through LDS once more (its own region) so that every lane stores 16 bytes
  // of a row; residual rows are loaded before the exchange.
  u4* ex = &ring[0][0];
  constexpr int CW = C::CW, CP = C::CP, XCH = 2 * JK * 256;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jj = 0; jj < JK; ++jj)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        f4 s;
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = grp == 0 ? acc[i][JK + jj][4 * e4 + e] : acc[i][jj][4 * e4 + e];
        ex[w * XCH + (i * JK + jj) * 256 + e4 * 64 + lane] = __builtin_bit_cast(u4, s);
      }
  const int nw = n0 + wn * (BN / 2) + grp * CW, mw = m0 + wm * 64;  // this wave's columns and rows
  constexpr int IT = 32 * CW / 4 / 64;                              // 16-byte pieces per lane of a 32-row block
  auto piece = [&](int i, int t, int& m, int& n, int& c) {
    const int q = t * 64 + lane;
    c = q % (CW / 4) * 4;
    m = mw + i * 32 + q / (CW / 4);
    n = nw + c;
  };
  f4 xr[2][IT];
  if (EPI == EPI_RESID && nsplit == 1) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < IT; ++t) {
        int m, col, c;
        piece(i, t, m, col, c);
        xr[i][t] = f4{0.f, 0.f, 0.f, 0.f};
        if (m < a.M && col < a.N) xr[i][t] = *reinterpret_cast<const f4*>((const float*)a.out + (size_t)m * a.ldo + col);
      }
  }
  lds_barrier();
  f4 v[2][JK][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jj = 0; jj < JK; ++jj)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const f4 o = __builtin_bit_cast(f4, ex[(w ^ 4) * XCH + (i * JK + jj) * 256 + e4 * 64 + lane]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[i][jj][e4][e] = (grp == 0 ? acc[i][jj][4 * e4 + e] : acc[i][JK + jj][4 * e4 + e]) + o[e];
      }
  float* tw = reinterpret_cast<float*>(ex + (w ^ 4) * XCH);  // read by this wave alone
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int jj = 0; jj < JK; ++jj)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          tw[(8 * e4 + 4 * (lane >> 5) + e) * CP + jj * 32 + (lane & 31)] = v[i][jj][e4][e];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (EPI == EPI_SWIGLU && nsplit == 1) {
      // a 16-column tile holds the gate columns of 8 features, then their up columns
#pragma unroll
      for (int t = 0; t < JK; ++t) {
        const int q = t * 64 + lane, c = q % (CW / 16) * 16, r = q / (CW / 16), m = mw + i * 32 + r;
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float gate = tw[r * CP + c + e], up = tw[r * CP + c + 8 + e];
          o[e] = gate / (1.0f + expf(-gate)) * up;
        }
        if (m < a.M && nw + c < a.N) {
          bf16* d = (bf16*)a.out + (size_t)m * 2 * a.ldo + (nw + c) / 2;
          const u4 hi = pack_frag_bf16(o);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] -= bf2f((bf16)(hi[e >> 1] >> (16 * (e & 1))));
          *reinterpret_cast<u4*>(d) = hi;
          *reinterpret_cast<u4*>(d + a.ldo) = pack_frag_bf16(o);
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < IT; ++t) {
        int m, col, c;
        piece(i, t, m, col, c);
        f4 o = *reinterpret_cast<const f4*>(tw + (m - mw - i * 32) * CP + c);
        if (m < a.M && col < a.N) {
          if (nsplit > 1) {
            *reinterpret_cast<f4*>(a.part + ((size_t)split * a.M + m) * a.N + col) = o;
          } else {
            if (EPI == EPI_RESID) o += xr[i][t];
            *reinterpret_cast<f4*>((float*)a.out + (size_t)m * a.ldo + col) = o;
          }
        }
      }
    }
  }
}

// Tile width and k-split of a launch: the pair with the least estimated time, in cycles at the 1.8 GHz that the matrix
// cores keep under load (256 workgroups run at once, one per CU):
//  rounds of workgroups x (stages x cycles per stage + a fixed cost for the first loads, the exchange and the stores),
//  at least what the weights take to arrive; split results are written and read again as fp32 partials.
// Measured: 1,310 cycles per stage of the 256-column tile, 850 of the 128-column tile, 12,000 fixed (from the times of
// k-ranges of 2,048 to 14,336), 3,000 bytes per cycle.
struct PromptPlan {
  int bn, nsplit;
};
static PromptPlan prompt_plan(int M, int N, int K, int most) {
  const double fixed = 12000, bytes_per_cycle = 3000;
  const int gy = (M + PP<256>::BM - 1) / PP<256>::BM, nfr = K / PP<256>::KB;
  PromptPlan best{256, 1};
  double best_t = 1e30;
  for (int bn = 256; bn >= 128; bn -= 128)
    for (int ns = 1; ns <= most; ++ns) {
      if (ns > 1 && nfr / ns < 8) break;
      const long wgs = (long)((N + bn - 1) / bn) * gy * ns;
      const double rounds = (double)((wgs + 255) / 256), stages = (double)((nfr + ns - 1) / ns);
      const double t = std::max(rounds * (stages * (bn == 256 ? 1310 : 850) + fixed), (double)N * K * 2 / bytes_per_cycle) +
                       (ns > 1 ? (double)M * N * 4 * 2 * ns / bytes_per_cycle : 0);
      if (t < best_t * 0.97) {  // a split or a narrow tile has to gain something
        best_t = t;
        best = PromptPlan{bn, ns};
      }
    }
  return best;
}

template <int EPI>
static int prompt_t(const GemmArgs& a, int max_split, Stream s, int* nsplit) {
  // a split needs room for its partials; SwiGLU needs whole sums
  const long room = a.part && a.part_cap > 0 ? a.part_cap / ((long)a.M * a.N) : 1;
  const int most = EPI == EPI_SWIGLU ? 1 : (int)std::max(1L, std::min((long)max_split, room));
  const PromptPlan p = prompt_plan(a.M, a.N, a.K, most);
  const int gy = (a.M + 127) / 128;
  *nsplit = p.nsplit;
  if (p.bn == 256) launch_k((k_gemm_pp<EPI, 256>), dim3((a.N + 255) / 256 * gy, p.nsplit), dim3(512), 0, s, a);
  else launch_k((k_gemm_pp<EPI, 128>), dim3((a.N + 127) / 128 * gy, p.nsplit), dim3(512), 0, s, a);
  return 0;
}

int launch_gemm_prompt(int epi, const GemmArgs& a, int max_split, Stream s, int* nsplit) {
  if (a.M < 1 || a.N % 32 != 0 || a.K % 32 != 0 || a.ldo % 4 != 0) return -1;
  switch (epi) {
    case EPI_F32: return prompt_t<EPI_F32>(a, max_split, s, nsplit);
    case EPI_RESID: return prompt_t<EPI_RESID>(a, max_split, s, nsplit);
    case EPI_SWIGLU: return prompt_t<EPI_SWIGLU>(a, max_split, s, nsplit);
    default: return -1;
  }
}

}  // namespace ham
