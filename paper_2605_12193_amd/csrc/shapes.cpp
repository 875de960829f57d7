// Host-side shape predicates and workspace sizes of the kernels: which
// (head dim, block, group, GQA group) combinations are built, the address
// limits of the Stage-1 score tiles, and the tile-stage workspace layout.
// Kept apart from the kernel sources so the C ABI layer builds and runs
// without device code (the sanitizer build of the ABI links this file).
#include <algorithm>

#include "bfla_internal.h"

namespace bfla {

bool estimate_supported(int head_dim, int block, int group) {
  if (head_dim != 64 && head_dim != 128 && head_dim != 256) return false;
  if (group < 1 || block % group) return false;
  const int G = block / group;
  if (G != 1 && G != 2 && G != 4 && G != 8 && G != 16) return false;
  return ((int64_t)group * head_dim) % kScoreChunk == 0;
}

bool estimate_q_fits(int group, int head_dim, int64_t q_stride_tok) {
  // one score tile reads kScoreTileM query groups of g tokens through one
  // buffer descriptor with a signed 32-bit byte range
  return ((int64_t)kScoreTileM * group - 1) * q_stride_tok + head_dim < (int64_t(1) << 30);
}

bool estimate_pages_fit(int group, int page_size) {
  // a tile of kScoreTileN key groups covers kScoreTileN * g tokens: at most
  // kScoreTileN * g / page_size + 1 pages
  return ((int64_t)kScoreTileN * group + page_size - 1) / page_size + 1 <= kScorePagesMax;
}

EstimatePlan estimate_plan(const int32_t* n_q, const int32_t* n_kv, int batch, int h_q,
                           int h_kv, int head_dim, int block, int group) {
  EstimatePlan p{};
  const int G = block / group, m = h_q / h_kv;
  int64_t capacity_tiles = 0;   // 256 x 128 tiles of one query head each
  double loaded = 0, pairs = 0; // LDS rows loaded per stage, and group pairs stored, by all tiles
  for (int r = 0; r < batch; ++r) {
    const ScoreGrid tg(n_q[r], n_kv[r], group, m);
    const int64_t n_c = n_kv[r] - n_q[r];
    p.total_tiles += (int64_t)h_kv * tg.tiles();
    capacity_tiles += (int64_t)h_q * ((tg.nqg + kScoreTileM - 1) / kScoreTileM) * tg.nct;
    for (int64_t rt = 0; rt < tg.nrt; ++rt) {
      // a row tile's causal column tiles: those whose first KV block starts at
      // or before the end of its last query block
      const int64_t u1 = std::min<int64_t>(tg.nu, (rt + 1) * kScoreUnits);
      const int64_t blk = (u1 - 1) / m;
      const int64_t i_max = (std::min<int64_t>(tg.nqg, (blk + 1) * kScoreUnit) - 1) / G;
      const int64_t e_i = std::min(n_c + (i_max + 1) * block - 1, (int64_t)n_kv[r] - 1);
      const int64_t cols = std::min<int64_t>(tg.nkg, (e_i / block + 1) * G);
      const int64_t ct = (cols + kScoreTileN - 1) / kScoreTileN;
      const double rows =
          std::min<double>((double)(u1 - rt * kScoreUnits) * kScoreUnit, (double)m * tg.nqg);
      p.causal_tiles += h_kv * ct;
      loaded += (double)h_kv * (rows * (double)ct + (double)cols);
      pairs += (double)h_kv * rows * (double)cols;
    }
  }
  // Estimated time of split S (whole chains per part only): a launch of T
  // causal tiles runs ceil(S T / 256) rounds of workgroups (one per compute
  // unit of an MI355X), each about 3 us to fill and drain and n_stage / S
  // stages.  A stage takes about 0.45 us plus 0.7 us for the loads of a full
  // tile (384 rows; 128K: 1.15 us a stage, chunks of 64 rows and fewer over
  // long prefixes: 0.75 us).  A split also writes and re-reads 4 bytes per
  // group pair and part, at about 5 TB/s.
  constexpr int kCUs = 256;
  const int n_stage = group * head_dim / kScoreChunk;
  const double stage_us =
      0.45 + 0.7 * loaded / ((double)p.causal_tiles * (kScoreTileM + kScoreTileN));
  auto cost = [&](int s) {
    const double rounds = (double)((p.causal_tiles * s + kCUs - 1) / kCUs);
    return rounds * (n_stage / s * stage_us + 3.0) + (s > 1 ? s * pairs * 8.0 / 5e6 : 0.0);
  };
  // a split must save at least 10 % of the estimate to be taken, and its
  // partial sums (room for the tiles of every query head on its own) must
  // stay within 300 MB
  const size_t part_bytes = (size_t)capacity_tiles * kScoreTileM * kScoreTileN * sizeof(float);
  double best = 0.9 * cost(1);
  p.split = 1;
  for (int s = 2; s <= 16; s *= 2) {
    if (n_stage % (s * kScoreChain) != 0 || s * part_bytes > 300000000u) break;
    const double c = cost(s);
    if (c < best) {
      best = c;
      p.split = s;
    }
  }
  p.partial_bytes = p.split > 1 ? p.split * part_bytes : 0;
  return p;
}

// counts [n_rows rounded up to 64] + scan partials [64] (int32), then the
// keep ballots [n_rows][ceil(max_t_kv / 64)] (uint64, at a 256-byte offset)
size_t expand_workspace_bytes(int64_t n_rows, int64_t max_t_kv) {
  return (size_t)(((n_rows + 63) / 64) * 64 + 64) * sizeof(int32_t) +
         (size_t)n_rows * (size_t)((max_t_kv + 63) / 64) * sizeof(uint64_t);
}

bool prefill_supported(int head_dim, int m) {
  bool c_ok = head_dim == 64 || head_dim == 128 || head_dim == 256;
  bool m_ok = m >= 1 && m <= 8;
  return c_ok && m_ok;
}

}  // namespace bfla
