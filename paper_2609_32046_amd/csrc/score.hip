// Host side of the persistent score kernel: the work list, the plan and
// workspace carve-up of one call, and the dispatch to the per-dtype launch
// instantiations (score_impl.h, score_*.hip).
#include <math.h>

#include <algorithm>

#include "kernels.h"

namespace cb {

void make_work_list(int units, int nstages, const int* per_unit, int resident, WorkList* wl) {
  *wl = WorkList{};
  wl->nstages = nstages;
  wl->units = units;
  for (int s = 0; s < nstages; ++s) {
    wl->per_unit[s] = per_unit[s];
  }
  // P2 trails P1 by enough steps that about 1.5 x the resident workgroups'
  // worth of P1 items is taken in between (one P1 item time, so that the
  // statistics are normally complete when a P2 item is taken), but never by
  // more than the number of units (so no step is empty).
  wl->lag[0] = 0;
  for (int s = 1; s < nstages; ++s) {
    int64_t gap = (3LL * resident + 2LL * wl->per_unit[s - 1] - 1) / (2LL * wl->per_unit[s - 1]);
    if (gap < 1) gap = 1;
    if (gap > units) gap = units;
    wl->lag[s] = wl->lag[s - 1] + (int)gap;
  }
  // Segment boundaries: where some stage starts or ends.
  int b[2 * kMaxStages];
  int nb = 0;
  for (int s = 0; s < nstages; ++s) {
    b[nb++] = wl->lag[s];
    b[nb++] = wl->lag[s] + units;
  }
  std::sort(b, b + nb);
  nb = (int)(std::unique(b, b + nb) - b);
  int64_t item = 0;
  wl->nseg = 0;
  for (int i = 0; i + 1 < nb; ++i) {
    int size = 0;
    for (int s = 0; s < nstages; ++s)
      if (wl->lag[s] <= b[i] && b[i] < wl->lag[s] + units) size += wl->per_unit[s];
    if (size == 0) continue;
    wl->seg_step[wl->nseg] = b[i];
    wl->seg_size[wl->nseg] = size;
    wl->seg_item[wl->nseg] = item;
    ++wl->nseg;
    item += (int64_t)size * (b[i + 1] - b[i]);
  }
  wl->items = item;
}

bool make_score_plan(int L, int Hq, int Hkv, int D, int m, int S, int64_t T, int dtype,
                     float scale, bool position, ScorePlan* p) {
  if (L < 1 || Hq < 1 || Hkv < 1 || m < 1 || S < 1 || T < 1) return false;
  if (Hq % Hkv != 0 || (D != 64 && D != 128) || T > kMaxSeqLen) return false;
  if (!(scale >= 0.f) || !isfinite(scale)) return false;
  const int G = Hq / Hkv;
  if ((int64_t)G * m > kMaxRows) return false;
  p->T = T;
  p->L = L; p->Hq = Hq; p->Hkv = Hkv; p->G = G; p->m = m; p->R = G * m; p->D = D;
  p->dtype = dtype;
  p->S = S;
  p->units = S * L * Hkv;
  p->position = position;
  if (position) {
    if (G > 8) return false;
    p->Gp = G <= 4 ? 4 : 8;
    if ((int64_t)p->Gp * m > kMaxRows) return false;
    p->Rp = p->Gp * m;
  } else {
    p->Gp = G;
    p->Rp = p->R;
  }
  // Waves per workgroup (a power of two, so that workgroups spread evenly over
  // the four SIMDs) and 16-row MFMA blocks per wave: the smallest that hold
  // the rows, up to 512 rows a workgroup.  Rows padded to 64 per wave cost
  // as much as real ones: 36 x 8 units of 160 rows (three blocks in four waves
  // instead of four) 630 -> 493 us as a whole position-level call.
  static constexpr int kShapes[][2] = {{1, 1}, {1, 2}, {1, 3}, {1, 4}, {2, 3}, {2, 4}, {4, 3},
                                       {4, 4}, {4, 5}, {4, 6}, {4, 8}, {8, 4}};
  p->row_groups = (p->Rp + kRowsPerGroup - 1) / kRowsPerGroup;
  // 128 rows a wave only where there are more items of kMinChunkTokens than
  // 512: an item's queries take twice as long to load into half the waves.
  // Eight waves against four, whole calls of 512 rows: 16 x 1000 22, 26 us; 384
  // x 1000 127, 141; 192 x 2000 122, 138; 64 x 4096 84, 87; 256 x 2048 133,
  // 138; but 288 x 3001 (864 items) 281, 269; 800 x 512 165, 150; 32 x 65536 574,
  // 554; 288 x 16384 1312, 1190.
  const bool few = (int64_t)p->units * p->row_groups *
                       ((T + kMinChunkTokens - 1) / kMinChunkTokens) <= 512;
  for (const auto& sh : kShapes) {
    if ((dtype == 0 && (sh[1] == 3 || sh[1] > 5)) || (position && sh[1] > 4)) continue;
    if (sh[1] == 8 && few) continue;
    p->waves = sh[0];
    p->rb = sh[1];
    if (16 * sh[0] * sh[1] >= p->Rp) break;
  }
  // Chunks: as many as fill 2048 workgroups, of no fewer than kTileTokens
  // positions, or else those of kMinChunkTokens.
  {
    const int64_t groups = (int64_t)p->units * p->row_groups;
    const int64_t least = (T + kMinChunkTokens - 1) / kMinChunkTokens;
    int64_t c = (2048 + groups - 1) / groups;
    const int64_t most = (T + kTileTokens - 1) / kTileTokens;
    if (c > most) c = most;
    if (c > 512) c = 512;
    p->chunks = (int)(c > least ? c : least);
  }
  const float sc = scale > 0.f ? scale : (float)(1.0 / sqrt((double)D));
  p->c2 = (float)((double)sc * 1.4426950408889634);
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  size_t off = 0;
  p->off_partial = off; off = al(off + (size_t)p->units * p->chunks * p->Rp * sizeof(float2));
  // Row normalisers between the two launches: only calls small enough for
  // that form (launch_w) with many chunks a unit.
  p->off_lse2 = 0;
  if (p->chunks > 16 && (int64_t)p->units * p->row_groups * p->chunks <= 4096) {
    p->off_lse2 = off;
    off = al(off + (size_t)p->units * p->Rp * sizeof(float));
  }
  p->off_imp_partial = off;
  if (p->row_groups > 1) off = al(off + (size_t)p->row_groups * p->units * (size_t)T * sizeof(float));
  p->off_numer_partial = off;
  if (position && p->row_groups > 1)
    off = al(off + (size_t)p->row_groups * p->units * (size_t)T * sizeof(float));
  // cb_pipeline's selection of the same units: its arrival counters follow
  // the score kernel's synchronisation words (cleared by the same launch),
  // its digit counts come last.
  p->sel = SelectSplit{1, 0, 0, 0};
  if (!position) select_split_plan(p->units, T, &p->sel);
  p->off_sync = off;
  p->off_sel_counters = kSyncHeader + (size_t)p->units * p->row_groups;
  p->sync_words = p->off_sel_counters +
                  (p->sel.parts > 1 ? (size_t)p->units * kSplitCounterWords : 0);
  off = al(off + p->sync_words * sizeof(uint32_t));
  p->off_sel_data = off;
  if (p->sel.parts > 1)
    off = al(off + (size_t)p->units * p->sel.data_words_per_unit * sizeof(uint32_t));
  p->total_bytes = off;
  return true;
}

// Plain launches or the queue, and the positions per item: whichever is
// estimated to keep a workgroup busy for fewer positions, an item counting
// kItemTokens more than it holds (its queries, its first tiles and its statistics
// take as long).
//
// Launches: items that fill one to four rounds of the resident workgroups, or
// of 1024, 2048 or 4096 positions.  A round that is only partly filled counts as
// a whole one, but in bf16 workgroups of one or two waves, which are bound by
// K's bytes, three quarters of what it lacks (the workgroups that are there then
// share a compute unit with fewer others).  320 units x 4096 positions x 128 rows
// (1024 resident): items of 1024 (1.25 rounds) 141 us, 1408 (0.94) 141, 2048 156;
// 88 x 26679 x 20 (2304 resident): 1024 (1.03) 229 us, 2048 235, 4096 255; 320 x
// 4096 x 256 (512 resident): 1024 (2.5) 204 us, 1408 (1.9) 210, 2048 (1.25) 220,
// 4096 250.
//
// The queue packs the items of both passes, ends on part of one, and has its
// words cleared by a kernel first (7 x 33329 x 296, position-level, one round of
// items either way: 90, 79 us).  Whole calls,
// queue and launches in us (bf16, 128 wide): 288 x 8192 x 256 365, 361; 384 x
// 32768 x 320 2119, 2098; 96 x 44045 x 368 876, 882; 288 x 16384 x 512 1190, 1194;
// 320 x 4096 x 256 219, 204; 8 x 8192 x 256 73, 41; eight waves: 384 x 1000 x 512
// 127, 155; 144 x 837 x 441 66, 65; 28 x 87519 x 575 (fp32, 64 wide) 4213, 4729;
// position-level: 864 x 3001 x 160 410, 417; 600 x 3595 x 156 344, 350; 512 x 8192
// x 512 1343, 1292.
//
// For the calls bound by K's bytes an estimate says little: the queue's
// workgroups drift apart and read evenly, launches start the second pass on
// what the first read last.  Up to three rounds launches are no slower: 64 x
// 131072 x 16 (two rounds) 762, 759; 376 x 20655 x 36 (2.2) 801, 743; 288 x 32768 x
// 4 (2.3) 852, 856; 88 x 26679 x 20 256, 229; 1 x 131072 x 8 50, 24; beyond, the
// queue: 256 x 65536 x 64 (four) 1498, 1532; 256 x 65536 x 128 (four) 1594, 1630
// (position-level 1814, 2021); 100 x 300000 x 64 (seven) 2672, 2727; but 240 x
// 86801 x 44 (five) 1949, 1928.
//
// (32-bit divisions: the rule runs on every call, and seven candidates in 64
// bits were 0.4 us of a 10 us call.)
ScoreForm choose_form(const ScorePlan& p, int queue_resident, int resident) {
  constexpr uint32_t kItemTokens = 160;
  constexpr uint64_t kMaxItems = 1u << 24;   // plain launches count items in 32 bits
  static_assert(kMinChunkTokens == 1 << 10, "candidates by shifts");
  const uint32_t T = (uint32_t)p.T, res = (uint32_t)resident;
  const uint32_t groups = (uint32_t)p.units * (uint32_t)p.row_groups;
  const uint32_t tile = (uint32_t)tile_tokens(p.dtype == 0 ? 4 : 2, p.D, p.waves, false);
  const bool whole_rounds = p.waves >= 4 || p.dtype == 0;
  const uint64_t queue_items = (uint64_t)groups * ((T + kQueueTokens - 1) / kQueueTokens);
  ScoreForm f{true, kQueueTokens};
  // Costs are in positions times 2 * resident.
  uint64_t best = UINT64_MAX;
  if (whole_rounds) {
    // A last row group of up to four waves has a SIMD to each: half an item.
    const uint32_t last_rows = (uint32_t)p.Rp - (uint32_t)(p.row_groups - 1) * kRowsPerGroup;
    const bool half = p.row_groups > 1 && last_rows <= 4 * kRowsPerWave;
    // Smaller items only where a workgroup has its compute unit to itself, so
    // that nothing else fills what a long one leaves idle (192 x 2000 x 512: 122
    // us with items of 1024, 146 as one round of launches).
    for (uint32_t q = kQueueTokens; q >= kMinChunkTokens; q /= 2) {
      const uint64_t c = T < q ? (T + tile - 1) / tile * tile : q;
      const uint64_t items = (uint64_t)groups * ((T + q - 1) / q);
      const uint64_t work = half ? items * 3 / 4 : items;
      const uint64_t fill = work > (uint32_t)queue_resident ? work : (uint32_t)queue_resident;
      const uint64_t cost = 4 * fill * (c + kItemTokens) * res / (uint32_t)queue_resident +
                            (c / 4 + 2 * kItemTokens) * res;
      if (cost < best) {
        best = cost;
        f.chunk_tokens = (int)q;
      }
      if (p.waves < kMaxWaves) break;
    }
  } else if (queue_items > 3u * (uint32_t)queue_resident) {
    return f;
  }
  uint32_t last = 0;
  for (uint32_t i = 0; i < 7; ++i) {
    uint32_t n = i < 4 ? (i + 1) * res / groups
                       : (T + (kMinChunkTokens << (i - 4)) - 1) >> (10 + i - 4);
    if (n > (uint32_t)p.chunks) n = (uint32_t)p.chunks;   // what the workspace holds
    if (n < 1 || n == last) continue;
    last = n;
    const uint32_t c = ((T + n - 1) / n + tile - 1) & ~(tile - 1);
    if (c > (uint32_t)kMaxItemTokens) continue;
    n = (T + c - 1) / c;
    if ((uint64_t)groups * n > kMaxItems) continue;
    const uint32_t items = groups * n;
    const uint64_t full = (uint64_t)((items + res - 1) / res) * res;
    const uint64_t used = items > res ? items : res;
    const uint64_t cost = (whole_rounds ? 4 * full : used + 3 * full) * (c + kItemTokens) +
                          (n > 16 ? 2 * kItemTokens * res : 0);   // the statistics' launch
    if (cost <= best) {
      best = cost;
      f.queue = false;
      f.chunk_tokens = (int)c;
    }
  }
  return f;
}

hipError_t launch_persistent(const ScorePlan& p, PersistArgs& a, hipStream_t s, ScoreForm* only) {
  if (p.position) {
    if (p.dtype == 1)
      return p.D == 128 ? launch_position_d<2, 128>(p, a, s, only)
                        : launch_position_d<2, 64>(p, a, s, only);
    return p.D == 128 ? launch_position_d<4, 128>(p, a, s, only)
                      : launch_position_d<4, 64>(p, a, s, only);
  }
  if (p.dtype == 1)
    return p.D == 128 ? launch_score_d<2, 128>(p, a, s, only) : launch_score_d<2, 64>(p, a, s, only);
  return p.D == 128 ? launch_score_d<4, 128>(p, a, s, only) : launch_score_d<4, 64>(p, a, s, only);
}

}  // namespace cb
