// Launch rules that depend on sizes alone, without a GPU or a HIP header, so that they can be checked by themselves.
#pragma once
#include <algorithm>

namespace ham {

constexpr int MAX_ATTN_SPLIT = 64;

// Slot splits of the filled-cache attention for R rows of Hk kv heads of which the longest has kv_max slots: none while
// the keys of a (row, kv head) are under 128 KB (one workgroup then reads them about as fast as the extra combine
// launch, 4 us, takes), else the count with the least estimated time for rows of equal length, two key blocks or more
// each.  One workgroup runs per CU, so R * Hk * splits workgroups take ceil(... / 256) rounds; a workgroup needs 3.4 us
// and, per 32 slots of head dim 128 in bf16 (16 KB), 0.42 us alone and 0.59 with all 256 at work.  That takes splits whose
// last round is full.  8 kv heads of 128 in bf16, us at 256 / (R * Hk) splits rounded down and at the splits here: 12 rows x
// 4,096 slots 44.3 / 42.8, 17 x 8,192 131 / 105, 20 x 4,096 72 / 64, 24 x 32K 540 / 476, 40 x 4,096 150 / 124, 48 x 8,192
// 287 / 257; the same where 256 workgroups come out even (1 x 2,048 10.4, 8 x 4,096 29, 32 x 4,096 87, 4 x 32K 89).
// A row's slots are shared by its own splits alone, so a long row among short ones is a serial chain.  From 2 MB of keys
// (8,192 such slots: 111 us unsplit) a row gets at least two rounds' share, up to 8 splits.  One row of 32K slots and the
// rest of 500: 8 rows 126 -> 75 us, 20 rows 444 -> 75, 40 rows 445 -> 129; where all are long this costs up to a tenth (10 x
// 8,192 61 -> 67 us, 5 x 8,192 35 -> 37, 16 x 8,192 89 -> 97, 32 x 8,192 165 -> 174, 8 x 32K 169 -> 177).
inline int attn_decode_splits(int dtype, int R, int Hk, int hd, int kv_max) {
  const int es = dtype == 1 ? 2 : 4, kb = dtype == 1 ? 32 : 16;
  const long long keys = (long long)kv_max * hd * es, pairs = (long long)R * Hk;
  if (keys < 128 * 1024) return 1;
  const int blocks = (kv_max + kb - 1) / kb, most = std::max(1, std::min((blocks + 1) / 2, MAX_ATTN_SPLIT));
  int least = 1;
  if (keys >= 2 * 1024 * 1024) least = (int)std::min({(512 + pairs - 1) / pairs, 8ll, (long long)most});
  int best = least;
  double best_t = 1e30;
  for (int s = least; s <= most; ++s) {
    const double rounds = (double)((pairs * s + 255) / 256), last = (double)(pairs * s) / 256 - (rounds - 1);
    const double units = (double)((blocks + s - 1) / s) * hd / 128;  // of 16 KB
    const double t = rounds * 3.4 + units * (0.59 * (rounds - 1) + 0.42 + 0.17 * last) + (s > 1 ? 4 : 0);
    if (t < best_t) {
      best_t = t;
      best = s;
    }
  }
  return best;
}

// Whether k_gemm_rows takes a bf16 projection of M rows and N columns (k range a multiple of 128).  It runs one workgroup
// of 128 columns per CU, so its time grows by rounds of 256 where k_gemm_wide's grows with the columns: a second round
// has to be an eighth full at up to 16 rows and a quarter full at 32, and at 32 rows a fourth does not pay.  Gate/up, us,
// k_gemm_wide with the reduction of its splits / k_gemm_rows: k 4,096, 32 rows: 224 groups of columns 51 / 45, 260 73 / 79,
// 288 76 / 80, 320 85 / 81, 520 131 / 125, 768 170 / 145, 780 173 / 174; 16 rows: 260 71 / 69, 288 76 / 71, 780 166 / 153;
// k 8,192, 32 rows: 260 130 / 150, 288 139 / 153, 320 152 / 154, 448 201 / 175, 780 316 / 334; 16 rows: 260 126 / 134,
// 288 140 / 134.
constexpr int ROWS_MAX_M = 32;
inline bool gemm_rows_takes(int M, int N) {
  if (M <= 8 || M > ROWS_MAX_M) return false;
  const int groups = (N + 127) / 128;
  if (groups > 256 && groups < 512) return groups >= (M <= 16 ? 288 : 320);
  return M <= 16 || groups <= 768;
}

// Grid of the bf16 prompt attention (kernels_attn_prompt.hip): `blocks` x kv heads x `seqs` workgroups of eight waves, for
// R rows from input s0 of a sequence on, through sequences of T inputs.  Tiles of 32 rows; `blocks` covers the longest share
// of a sequence.  The keys form while the rows form would give no more than every other CU a workgroup (one sequence,
// rows / keys form: 512 rows of the 1B shape 20.2 / 17.0 us, 1,024 rows 35.5 / 28.7 and of the 8B shape 54.7 / 46.1; above
// that the rows form wins: 2,048 rows 68.9 / 96.0 and 99.4 / 142.5).
constexpr int PROMPT_ATTN_WAVES = 8, PROMPT_ATTN_KEYS_MAX_WGS = 128;
struct PromptAttnGrid {
  int blocks, seqs;
  bool keys;
};
inline PromptAttnGrid prompt_attn_grid(int R, int s0, int T, int H, int Hkv) {
  const int seqs = (s0 + R - 1) / T + 1, tiles = (std::min(R, T) + 31) / 32;
  const int half = PROMPT_ATTN_WAVES / (H / Hkv) / 2;  // row tiles of a workgroup: 2 * half (rows form) or half
  const int rows_blocks = ((tiles + 1) / 2 + half - 1) / half;
  const bool keys = (long)rows_blocks * Hkv * seqs <= PROMPT_ATTN_KEYS_MAX_WGS;
  return PromptAttnGrid{keys ? (tiles + half - 1) / half : rows_blocks, seqs, keys};
}

}  // namespace ham
