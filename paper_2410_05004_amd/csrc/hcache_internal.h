// Internal declarations shared by the translation units of libhcache.so.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <map>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "hcache.h"

namespace hc {

// Tile geometry of the fused restoration kernel.  The weight matrix is re-ordered once
// (hc_set_layer_weights) so that the kernel's accumulator registers come out in a
// store-friendly order; the constants below define that order and are used by both the
// packing kernel and the restoration kernel.
constexpr int kPairGroup = 64;    // physical rows per RoPE pair group: 32 "first" + 32 "second" features
constexpr int kPartAlign = 128;   // the K part and the V part are each padded to this many rows
constexpr int kTileF = 256;       // physical weight rows (features) per workgroup
constexpr int kTileT = 256;       // tokens per workgroup
constexpr int kTileK = 32;        // d_model slice per main-loop step
constexpr int kWTileBytes = kTileF * kTileK * 2;   // one packed weight tile: 256 rows x 64 bytes

// LDS placement of the activations' 16-byte chunks: super-tiles have 128-byte rows (8 chunks),
// chunk c of row r sits at position c ^ swz_x(r).  A fragment read takes 16 consecutive rows per
// lane quarter, quarter q reading chunk q (+ 4 for odd steps), and is bank-conflict free
// (checked with the bank-conflict counter).  The packed weights need no swizzle: they are
// stored, and staged, in fragment order.
__host__ __device__ inline int swz_x(int row) { return (row >> 1) & 7; }

inline int round_up(int x, int m) { return (x + m - 1) / m * m; }
constexpr int kChipCUs = 256;     // one workgroup of the restoration kernel per CU at a time

// Tile scheduling.  Workgroup ids are handed to the 8 XCDs round-robin and every XCD has
// its own L2, so the tiles one XCD works on at the same time should share weight rows
// and token rows.  The tile grid is cut into super tiles of GF x GT tiles (powers of two,
// GF * GT <= 32 = the CUs of an XCD); super tile k belongs to XCD k % 8.  The host picks the
// shape that keeps the XCDs evenly loaded first and shares the most rows second.
// Workgroups that fall outside the grid exit at once.
struct TileGrid {
  int nf, nt;        // tiles along features / tokens
  int gf_shift;      // log2(GF)
  int g_shift;       // log2(GF * GT)
  int nsf;           // super tiles along features
};

// Tile of workgroup slot `wg` (0 .. slots per layer - 1) of a layer; false for a slot that is
// padding of the order.  `rot` is the layer's index within its launch: of every eight super
// tiles, the one XCD x works on moves on by one with every layer, so that when the number of
// super tiles is not a multiple of 8 (56 feature tiles x 8 token tiles = 14 super tiles of
// 4 x 8) the XCDs that go short in one layer are others in the next.
__host__ __device__ inline bool slot_to_tile(const TileGrid& g, int wg, int rot, int& tile_f, int& tile_t) {
  const int xcd = (wg + rot) & 7, li = wg >> 3;
  const int super = (li >> g.g_shift) * 8 + xcd, r = li & ((1 << g.g_shift) - 1);
  tile_f = (super % g.nsf) * (1 << g.gf_shift) + (r & ((1 << g.gf_shift) - 1));
  tile_t = ((super / g.nsf) << (g.g_shift - g.gf_shift)) + (r >> g.gf_shift);
  return tile_f < g.nf && tile_t < g.nt;
}

// Super-tile shape for a layer of nf x nt tiles: fewest rounds on the busiest XCD (an XCD runs 32
// workgroups at a time, one per CU), then the most row sharing (smallest 1/GF + 1/GT), then
// fewest slots.  Of two shapes that tie (GF x GT = 4 x 8 and 8 x 4 for 8 x 32 tiles) the one
// with fewer feature tiles is met first and kept: it measured 105.4 against 107.0 us per layer.
// Returns the workgroup slots per layer (a multiple of 8).
inline int choose_tile_grid(int nf, int nt, TileGrid& g) {
  g.nf = nf;
  g.nt = nt;
  int best_rounds = 1 << 30, best_slots = 1 << 30, best_share = 1 << 30;
  g.gf_shift = g.g_shift = 0;
  for (int fs = 0; fs <= 5; ++fs) {
    for (int ts = 0; fs + ts <= 5; ++ts) {
      const int gf = 1 << fs, gt = 1 << ts;
      const int n_super = ((nf + gf - 1) >> fs) * ((nt + gt - 1) >> ts);
      const int slots = (n_super + 7) / 8 * gf * gt;      // workgroup slots per XCD
      const int rounds = (slots + 31) / 32;
      const int share = (32 >> fs) + (32 >> ts);          // 32 * (1/GF + 1/GT)
      if (rounds < best_rounds || (rounds == best_rounds && share < best_share) ||
          (rounds == best_rounds && share == best_share && slots < best_slots)) {
        best_rounds = rounds; best_share = share; best_slots = slots;
        g.gf_shift = fs; g.g_shift = fs + ts;
      }
    }
  }
  g.nsf = (nf + (1 << g.gf_shift) - 1) >> g.gf_shift;
  return best_slots * 8;
}

// How the workgroups of a launch spread over the chip's 32 shader engines (four per XCD, eight CUs each).
// The ids of an XCD go round its engines in order, those that exit at once included, so an engine can have
// more than eight workgroups while others have CUs free, and the launch then takes another round:
// 3 layers of 1088 channels onto 1152 features, 714 tokens in tiles of 128 rows x 256, are 30 workgroups on the busiest XCD
// but 9 on one of its engines, and took 35.7 us instead of the 22 of one round.  Over 2000 measured launches of
// several layers, those of up to 32 workgroups on an XCD but more than 8 on an engine took 1.6 times
// the one round's time, the others 0.9.
struct ChipLoad {
  int part[9][32];         // workgroups of each engine (4 x XCD + engine) in the first m layers, m = 0 .. 8

  // `slots` of a layer as choose_tile_grid returns them; tiles from feature tile `live_nf` on exit at once
  ChipLoad(const TileGrid& g, int slots, int live_nf) : part{} {
    const int gf = 1 << g.gf_shift, gt = 1 << (g.g_shift - g.gf_shift), per_xcd = slots >> 3;
    int own[8][4] = {};                                    // one layer's, by super tile k % 8 and engine
    for (int t0 = 0, k = 0; t0 < g.nt; t0 += gt)
      for (int i = 0; i < g.nsf; ++i, ++k) {
        const int nf_here = live_nf - i * gf < gf ? live_nf - i * gf : gf, nt_here = g.nt - t0 < gt ? g.nt - t0 : gt;
        const int at = (k >> 3) << g.g_shift;
        if (gf >= 4)                                       // tile f of every row is on engine f % 4
          for (int e = 0; e < 4; ++e) own[k & 7][e] += nf_here > e ? (nf_here - e + 3) / 4 * nt_here : 0;
        else
          for (int t = 0; t < nt_here; ++t)
            for (int f = 0; f < nf_here; ++f) ++own[k & 7][(at + f + t * gf) & 3];
      }
    for (int m = 0; m < 8; ++m) {                          // layer m: its super tile k on XCD (k - m) % 8
      const int turn = m * per_xcd & 3;                    // and its first slot on engine `turn`
      for (int x = 0; x < 8; ++x) {
        const int* here = own[(x + m) & 7];
        if (turn == 0)
          for (int e = 0; e < 4; ++e) part[m + 1][4 * x + e] = part[m][4 * x + e] + here[e];
        else
          for (int e = 0; e < 4; ++e) part[m + 1][4 * x + e] = part[m][4 * x + e] + here[(e - turn) & 3];
      }
    }
  }
  // workgroups on the busiest engine, and XCD, in a launch of n layers; its rounds at eight an engine at a time
  int busiest(int n) const {
    int most = 0;
    for (int e = 0; e < 32; ++e) {
      const int here = n / 8 * part[8][e] + part[n % 8][e];
      if (here > most) most = here;
    }
    return most;
  }
  int busiest_xcd(int n) const {
    int most = 0;
    for (int x = 0; x < 32; x += 4) {
      int here = 0;
      for (int e = x; e < x + 4; ++e) here += n / 8 * part[8][e] + part[n % 8][e];
      if (here > most) most = here;
    }
    return most;
  }
  int rounds(int n) const { return (busiest(n) + 7) / 8; }
};

// Workgroups of a launch per CU of its busiest part (an XCD of a single layer, an engine of several, or an XCD
// too where a CU takes two workgroups, `shared`), for a layer of nf x nt tiles of which those from
// feature tile live_nf on exit at once.  Beyond sixteen rounds the parts differ by little.
inline float launch_load(int nf, int nt, int live_nf, int n_layers, bool shared = false) {
  const float all = (float)live_nf * nt * n_layers / kChipCUs;
  if (all > 16.f) return all;
  TileGrid g;
  const int slots = choose_tile_grid(nf, nt, g);
  if (n_layers > 1) {
    const ChipLoad load(g, slots, live_nf);
    return shared ? load.busiest_xcd(n_layers) / 32.f : load.busiest(n_layers) / 8.f;
  }
  const int gf = 1 << g.gf_shift, gt = 1 << (g.g_shift - g.gf_shift);
  const int supers = g.nsf * ((nt + gt - 1) / gt);
  return (float)((supers + 7) / 8 * (gf < nf ? gf : nf) * (gt < nt ? gt : nt)) / (kChipCUs / 8);
}

// Split d_model loops for a partly filled last round (paper Section 4.1.1, "Performance
// considerations": the projection's efficiency depends on how the token count fills the device).
// A single-layer launch of nf x nt tiles runs in rounds of one workgroup per CU, and a last
// round with few tiles takes as long as a full one.  The token tiles that do not fit the full
// rounds can instead be computed by n_split workgroups each, every one taking a contiguous
// share of the d_model loop and writing its fp32 accumulators and the tokens' partial sums (of
// squares, and plain for LayerNorm) to a slot of a workspace; a second launch adds the slots up
// in a fixed order and runs the ordinary epilogue, kFixupPerTile workgroups per tile (one token
// block of each wave's four).  The split workgroups follow the whole tiles in the same grid, so
// they also fill CUs that the whole tiles leave idle.
//
// Cost model (microseconds, from token sweeps of three shapes: a whole tile takes 1.2 - 1.7 per
// 64 channels depending on how many CUs are busy, 1.5 here; a split workgroup, on a chip that is
// otherwise idle, 1.0; the slots are written and read back at the HBM rate, 264 KB each, 0.143
// for both; the second launch, the gap before it and the split workgroups' prologues add about
// 15): a split in n ways of t tiles costs nm / n + 0.143 t n + 15 against 1.5 nm for the
// unsplit round.
// n is the cheapest of 2 .. min(256 / t, nm / 8, 16) (one round of split workgroups, shares of
// at least 512 channels); the plan is used when it is cheaper than the round, or on request.
constexpr int kSplitSlotFloats = kTileF * kTileT + 512;   // accumulators, 256 sums of squares, 256 plain sums
constexpr int kSplitMaxSlots = 256;                       // slots of the workspace (one round of workgroups)
constexpr int kSplitMinSuper = 8;                         // least share of the loop: 8 x 64 channels
constexpr int kSplitMaxWays = 16;
constexpr int kFixupPerTile = 4;
constexpr float kWholeStepUs = 1.5f, kSplitStepUs = 1.0f, kSplitSlotUs = 0.143f, kSplitFixedUs = 15.f;
struct SplitPlan {
  float* ws;             // device: kSplitMaxSlots slots of kSplitSlotFloats floats
  int32_t main_slots;    // workgroup slots of the tiles computed whole (first in the grid)
  int32_t nt_main;       // token tiles tile_t < nt_main are computed whole
  int32_t n_tail;        // tiles whose loop is split: nf * (nt - nt_main)
  int32_t n_split;       // workgroups per such tile
};
// Fills `sp` (but for ws) and the tile grid of the whole tiles for a layer of nf x nt tiles and
// nm 64-channel steps; false when the launch is better left unsplit (`force`: when it cannot
// be split at all).
inline bool plan_split(int nf, int nt, int nm, bool force, SplitPlan& sp, TileGrid& g_main) {
  const int tiles = nf * nt, rem = tiles % kChipCUs;
  if (rem == 0) return false;
  const int nt_main = (tiles - rem) / nf;                // whole rows of token tiles within the full rounds
  const int n_tail = (nt - nt_main) * nf;
  int cap = kSplitMaxSlots / n_tail;
  if (cap > nm / kSplitMinSuper) cap = nm / kSplitMinSuper;
  if (cap > kSplitMaxWays) cap = kSplitMaxWays;
  if (cap < 2) return false;
  int ways = 2;
  float best = 0.f;
  for (int n = 2; n <= cap; ++n) {
    const float t = kSplitStepUs * nm / n + kSplitSlotUs * n_tail * n;
    if (n == 2 || t < best) { best = t; ways = n; }
  }
  if (!force && best + kSplitFixedUs >= kWholeStepUs * nm) return false;
  sp.nt_main = nt_main;
  sp.n_tail = n_tail;
  sp.n_split = ways;
  sp.main_slots = choose_tile_grid(nf, nt_main, g_main);
  return true;
}
// Share of the loop (in 64-channel steps) of split workgroup s of n: [first, second).
__host__ __device__ inline void split_range(int nm, int n, int s, int& m_begin, int& m_end) {
  m_begin = (int)((long)nm * s / n);
  m_end = (int)((long)nm * (s + 1) / n);
}

// Few tokens (restore_small.inc): 32 packed rows x 16 nb tokens per workgroup, no cross-workgroup
// sums (nb 1..4).
//
// A launch is as long as the busiest CU takes to stream its operands: 64 bytes per channel for the
// rows and 32 nb for the tokens, per workgroup; up to nb = 2 two workgroups share a CU, so
// their load evens out.  The 64-row pair groups go round the XCDs and all token tiles of a group stay on
// its XCD, so the busiest CU is one of an XCD with ceil(pair groups / 8) of them (128 features are two
// pair groups, on two of the eight XCDs).
// Token sweeps (d_model 1024 .. 8192, 1 .. 56 heads, 1 .. 9000 tokens) fit
// 3.5 us + the hypotenuse of that (2.85e-5 us per channel and unit of 32 + 16 nb, and 3 us more for the
// lookups and the reduction of every further round of workgroups) and the time
// the weights take from memory (5.4 MB/us), to 20 %.  The other side of the comparison is what
// plan_split's figures give for the tiles, with the workspace traffic of the live token blocks only.
// Below d_model 1024 the large tiles' workgroups take too short for a second order of sums to
// be worth having: there every launch adds a token's channels up in the same order.
// Measured, this kernel against the tiles, us per call back to back, the layers (600 MB of weights) in turn: 16
// tokens 10.7 / 25.5 (d_model 4096, 8 heads), 15.8 / 34.8 (32 heads), 26.8 / 42.2 (5120, 40 heads); 64 tokens
// 10.2 / 27.1, 21.7 / 36.9; 256 tokens of 4096, 8 heads 16.1 / 35.7.  Narrow K/V: 1700 tokens of 4096 channels
// onto 128 features 24.4 / 32.8, 4000 tokens 47.8 / 39.8 (not taken), 9000 of 1024 channels 53.7 / 26.4 (not taken).
constexpr int kSmallMinModel = 1024;
constexpr float kSmallRoundUs = 3.f;

// Tiles of 128 rows x 64 nb tokens (restore_mid.inc).  They add a token's channels up in the order of the
// unsplit 256 x 256 tiles, so results do not depend on which of the two a launch takes.
//
// A launch takes as many rounds as its busiest XCD (several layers: its busiest shader engine, see ChipLoad), one
// workgroup per CU.  Cost of a round, fitted on the times of every kernel at 8600 random shapes (d_model
// 64 .. 8192, 1 .. 128 heads, 1 .. 32768 tokens, one layer or 2 .. 32): kMidStepUs per 64 channels and
// 2.5 + 0.75 nb for prologue and epilogue; nb = 1 beyond one workgroup per CU (two share one) 0.48 per 64 channels
// and workgroup, prologue and epilogue behind the other's loop; the large tiles 1.09 and up to 0.45 more as
// the CUs fill up, a tenth less where rounds follow each other, and 4.7.  The hypotenuse of that and the time of the
// weights (7.7 TB/s, in part from the caches) is the cost; single-layer calls of the large tiles come
// out without the weights, split ones 6 % above plan_split's figures.
// Not taken: nb = 5 in launches of several layers, where its ring of two stages does not cover the
// memory's latency (300 tokens, 8 layers of 5120 onto 10240: 368 us against 308), and with LayerNorm, whose extra matrix
// ops make it slower than the large tiles (558 tokens of 7168 onto 14336: 167 us against 153); nb = 1
// beyond two workgroups per CU in a single layer (the pairs lose step and with it the L2: those 558 tokens
// 259 us), six in several (24 layers of 1600 onto 6400, 266 tokens: 374 us against 261).
// The figures are good to 9 % or so, so these tiles have to promise that.  Over those shapes the choice
// takes 0.3 % (one layer) and 1.9 % (several) longer than the fastest kernel in the mean, and 22 are more than 4 %
// slower than the large tiles; workgroups counted over the whole chip instead of its busiest part
// made that 166 (20 layers of 4096 onto 2048, 179 tokens 136 us against 99; 8627 tokens of 7872 onto 128 108 against 65).
// Measured, these tiles against the large ones (whole or split), us per call back to back, the layers (600 MB of weights) in
// turn: 4096 onto 2048, 800 tokens 28.2 / 44.2, 4000 tokens 66.4 / 93.8; 5120 onto 10240, 300 tokens
// 58.2 / 70.1, 900 124.2 / 126.8 (99.4 / 125.0 with one layer's weights in the caches), 1200 147 / 123 (not
// taken); 32 layers of 4096 onto 2048, 40 tokens 113 / 144, 256 tokens 181 / 147 (not taken).
constexpr float kMidStepUs[6] = {0.f, 0.41f, 0.57f, 0.725f, 0.87f, 1.29f};
constexpr float kMidSharedStepUs = 0.48f;                // nb = 1, two workgroups on a CU
constexpr float kMidFixedUs = 2.5f, kMidBlockUs = 0.75f, kMidPromise = 1.09f;
constexpr float kTileStepUs = 1.09f, kTileStepBusyUs = 0.45f, kTileNextRounds = 0.91f, kTileFixedUs = 4.7f;
constexpr float kSplitPrice = 1.06f;
constexpr float kWeightsUsPerByte = 1.f / 7.7e6f;
constexpr float kFewWeightsUsPerByte = 1.f / 5.4e6f;     // as the few-token kernel and split tiles read them

// Tiles of 128 rows x 32 nb tokens with loader waves (restore_stream.inc), nb = 2 .. 6; the same sums in the same order again.
// Cost, fitted on the times of nb = 2 .. 6 at 2000 random single-layer shapes (d_model 1024 .. 8192, 192 .. 8192
// K/V features, 16 .. 16384 tokens; each with the weights from memory and from the caches, geometric mean; 8 %) and
// 2000 of two to eight layers (9 %): rounds as above, of step us per 64 channels, growing with nb and with how many of the
// CUs are busy (the clock falls), `more` of it for every further round of several layers, whose CUs have lost step; the
// hypotenuse of that and the operands' time from memory (the hidden states count 2.4 times: several XCDs fetch them).
// Over 2411 single-layer shapes and 2246 calls of two to four layers, each measured on every kernel, time under this rule against the
// one without these tiles: single layers 0.937 in the geometric mean (0.923 if every choice were the fastest), 5 more than 4 %
// slower; of the calls 1438 take these tiles, to 0.751, 18.
// Where the lines lie:
//  * d_model above 1024: below, up to 16 supersteps, a launch is mostly prologue, epilogue and its issue, and these tiles gain
//    a microsecond or two (700 shapes: 0.92 of the time in the median up to 256 channels, 0.87 at 512 .. 1024, 0.82 above);
//    the tiles of 64 n tokens stay.
//  * a single layer of up to two rounds: beyond, the gain is gone with the CUs' step (1601 tokens of 5120 onto 10240, 2.8
//    rounds of 192-token tiles: 187 us against 162 in split 256 x 256 tiles).
//  * two to four layers, where the loop takes longer than the operands (kStreamOverMemory): weights that stream from
//    memory come in faster through eight loading waves, or two workgroups on a CU (20 layers of 8192 channels onto 2048, 43 tokens:
//    160 us here, 144 with 64-token tiles), and in longer launches the CUs are out of step for most of the time (best of these
//    tiles over the earlier choice, median: 0.75 at two to four layers of 3000 channels and more, 0.90 .. 1.02 at five to
//    twelve, 1.00 .. 1.05 beyond).  Weights whose token tiles fall into different rounds are read again
//    (kStreamWeightsAgain): 2 layers of 5120 onto 10240, 228 tokens: 101 us in tiles of 96 tokens, 80 in those of 256.
//    A second round whose weights are not in the last-level cache (kLastCacheBytes) waits for memory: 3 layers of 5120 onto 10240, 161
//    tokens: 118 us here, 106 on the large tiles; of 1446 launches taken at two to four layers, 33 were more than 4 % slower than
//    the tiles they displaced, 17 with a fifth more for those (kStreamColdRounds).
//  * 192 K/V features or more: what the fit covers.
//  * against the few-token kernel a quarter more (kFewOverStream), which its own estimate is too high by for wide K/V (41
//    tokens of 5120 onto 10240: 27.4 us, these tiles 32.6); not where the tiles of 64 n tokens or the large ones are estimated
//    below it as well (995 tokens of 1664 onto 768: 15.9 us in the few-token kernel, 12.5 here).
constexpr int kStreamMinModel = 1024, kStreamMinKv = 192, kStreamMostLayers = 4;
struct StreamCost {
  float step, block, busy, busy_block, norm_block;        // us per 64 channels and round: idle chip, all CUs busy, LayerNorm
  float more, round, round_block, call, hidden_times, us_per_byte, promise;
};
constexpr StreamCost kStreamCost[2] = {                   // one layer, several
    {0.163f, 0.0364f, -0.0161f, 0.0362f, 0.0052f, 0.f, 2.1f, 0.47f, 1.3f, 2.3f, 1.f / 6.86e6f, 1.09f},
    {0.049f, 0.0477f, 0.0643f, 0.0177f, 0.0056f, 0.0378f, 1.9f, 0.32f, 5.4f, 2.4f, 1.f / 6.46e6f, 1.04f}};
constexpr float kStreamMostRounds = 2.f, kStreamOverMemory = 1.f, kStreamWeightsAgain = 0.8f, kFewOverStream = 1.25f;
constexpr float kStreamColdRounds = 1.2f, kLastCacheBytes = 2.56e8f;

// Least time of a launch of nf x nt tiles of 128 rows: that of filling the L2s (all layers' bytes).  Every super tile brings its rows of
// the weights into its XCD's L2, but for those that an XCD works on at once and that lie in one column (k and k + 8 do where 8 is a
// multiple of the columns), and the hidden states come into the L2 of each XCD that has a column.  6.6 TB/s and 2.5 us, fitted on the
// tiles with loader waves of 9925 launches: those that this bounds were estimated 25 % too low without it and are 3 % with it
// (7 % rms).  Super tiles of one token tile each, taken because no other shape fits the XCDs evenly, are the usual case: 853
// tokens of 4224 channels onto 7168 in nine tiles of 96 tokens bring in the weights nine times, 545 MB: 86 us, 65 in tiles of 64 n
// tokens.  Of 2411 single-layer shapes 76 go elsewhere by it, to 0.85 of the time, none more than 4 % slower in the mean of
// weights from memory and from the caches (with 3.5 us it is 94, 0.88 and 3, and 257 to 320 tokens of 5120 onto 10240 lose up to 14 %
// from memory).  No estimate of a kernel, so no promise on top.  Up to 1024 channels nothing was measured against it.
constexpr float kL2FillUsPerByte = 1.f / 6.6e6f, kL2FillUs = 2.5f;
inline float l2_fill_us(int nf, int nt, float weights, float hidden, float out) {
  TileGrid g;
  choose_tile_grid(nf, nt, g);
  const int gt_shift = g.g_shift - g.gf_shift, rows = (nt + (1 << gt_shift) - 1) >> gt_shift;
  int at_once = (g.nsf * rows + 7) / 8;                    // super tiles that an XCD works on at once
  if (at_once > 32 >> g.g_shift) at_once = 32 >> g.g_shift;
  const int columns = 8 % g.nsf == 0 ? 1 : at_once < g.nsf ? at_once : g.nsf;   // of those
  return (weights * rows * columns / at_once + hidden * (g.nsf < 8 ? g.nsf : 8) + out) * kL2FillUsPerByte + kL2FillUs;
}

// Rows of the hidden states that a tile with loader waves, T tokens at t0, reads: its own, and in the place of those past
// the end, whose results nothing uses, its own over again, or where fewer than eight are left sixteen of the tile before.  The last
// row for all of them is one line asked for up to T times by every workgroup of the tile in every superstep: 65 tokens of 7168
// channels onto 14336 took 52.8 us, weights from the caches, and 128 tokens 38.7; now 39.8 (58.8 -> 55 with weights from memory).
// Rows of the tile before for all of them are more lines to bring in: 37.6 and 61; tiles with eight live rows or more lost up to 8 % by it.
// tile_row is relative to tile_base_row, which keeps byte offsets of up to two tiles within 32 bits.
__host__ __device__ inline int tile_base_row(int t0, int n_tok, int T, int d_model) {
  return t0 > 0 && n_tok - t0 < 8 && d_model <= 1 << 22 ? t0 - T : t0;
}
__host__ __device__ inline int tile_row(int r, int t0, int base_row, int n_tok) {
  const int live = n_tok - t0;
  return r < live ? t0 - base_row + r : base_row < t0 ? r & 15 : r % live;
}

// LayerNorm's sums ahead of the 256 x 256 tiles (token_sums_kernel).  Every feature tile of a token tile works the same
// sums out, by 4 of its 36 matrix ops, and at the chip's power limit they cost as much as any other: 0.16 us per 64
// channels and round.  A pass over the hidden states ahead of the launch takes their time from memory (4.5 TB/s) and
// some 6 us.  Measured, sums in the tiles / ahead: eight layers of 2048 tokens, 7168 channels onto 14336 features 2515 / 2330 us (4.3
// times the pass in estimated savings), one layer of 4096 tokens 672 / 644 (3.3 times), of 2048 tokens 337 / 337 (2.5
// times: a last round that is three quarters full gets no shorter): the line lies at 2.8.  RMSNorm's sums are half as many
// ops: 8192 and 20000 tokens of 5120 onto 10240 took the same either way (603 / 602, 1530 / 1532 us).
// The sums go to one of kSumsSlots slots of a context, in turn, so that launches on different streams seldom wait for
// each other; a launch that does not fit a slot, or is being captured (it would have to wait for an event from
// outside the capture), works them out in its tiles, with the same results bit for bit.
constexpr int kSumsSlots = 4;
constexpr size_t kSumsTokens = 262144;                    // token rows (of all layers of a launch) per slot
constexpr float kSumsSaveUs = 0.16f, kSumsUsPerByte = 1.f / 4.5e6f, kSumsCallUs = 6.f, kSumsTimes = 2.8f;
inline bool sums_pay_ahead(int nf, int nt, int nm, int n_tok, int n_layers) {
  if ((size_t)n_tok * n_layers > kSumsTokens) return false;
  const float save = (float)nf * nt * n_layers / kChipCUs * nm * kSumsSaveUs;
  return save > kSumsTimes * ((float)n_tok * n_layers * nm * 128.f * kSumsUsPerByte + kSumsCallUs);
}

// Tiles of 256 rows x 288 or 320 tokens (restore_wide.inc); the same sums in the same order again.  Estimate: rounds as above, of so
// much per 64 channels, more as the CUs fill up, and a fixed part; the hypotenuse of that and the operands' time from memory.  One layer: fitted on
// 2000 shapes (5 % over 187 launches).  Several: on 3114 launches of 2048 channels and more (5 %; the one layer's figures were 6 % too high
// in the mean, 10 % where a launch leaves CUs idle, which hid that one launch of 20 layers of 300 tokens, 4096 channels onto 2048, takes
// 136 us and 16 + 4 on the 256-token tiles 162).  The other estimates are good to 9 % or so, so against them
// these tiles have to promise that, 12 % with several layers; against a whole call of other launches, whose errors even out, 4 %.  Of 5328
// measured calls of several layers 58 go elsewhere by this than with the one layer's figures for all, to 0.86 of the time, none
// more than 4 % slower (at 9 % four of 87 are).  LayerNorm, whose plain sums would need a register more per block, and d_model below
// 2048, where nothing was measured, stay with the others.
constexpr int kWideMinModel = 2048;
constexpr float kWideCallPromise = 1.04f;
struct WideCost { float step[2], busy, round, hidden_times, us_per_byte, promise; };   // step: 288, 320 tokens
constexpr WideCost kWideCost[2] = {                       // one layer, several
    {{1.34f, 1.5f}, 0.4f, 9.f, 1.f, 1.f / 4.8e6f, 1.09f}, {{1.09f, 1.27f}, 0.45f, 16.6f, 2.1f, 1.f / 6.06e6f, 1.12f}};
inline float wide_us(int d_kv, int d_model, int n_tok, int n_layers, int nb) {
  const WideCost& k = kWideCost[n_layers > 1];
  const int nf = 2 * round_up(d_kv, kPartAlign) / kTileF;
  const float bytes_us = (4.f * d_kv * d_model + k.hidden_times * 2.f * n_tok * d_model) * n_layers * k.us_per_byte;
  const float load = launch_load(nf, (n_tok + 32 * nb - 1) / (32 * nb), nf, n_layers), rounds = ceilf(load);
  const float loop_us = rounds * ((k.step[nb - 9] + k.busy * (load / rounds)) * (d_model / (2 * kTileK)) + k.round);
  return hypotf(loop_us, bytes_us);
}

struct Route {
  enum Kind { kTiles, kSmall, kMid, kStream, kWide } kind = kTiles;
  int nb = 0;              // tokens per workgroup of the others: in 16s (kSmall), 64s (kMid), 32s (kStream, kWide)
  float us = 0.f;          // what the launch is estimated to take
  bool sums_ahead = false; // kTiles: LayerNorm's sums ahead of the tiles
  bool split = false;      // kTiles: the launch is split by
  SplitPlan split_plan{};
  TileGrid grid{};         // kTiles: of the tiles computed whole
};
// Which kernel a launch of n_layers layers takes, decided once per launch.  `free_order`: the order of the
// sums may depend on the token count (split launches allowed); the few-token kernel and split plans need it.
inline Route plan_route(int d_kv, int d_model, int n_tok, int n_layers, bool layer_norm, bool free_order) {
  const int nm = d_model / (2 * kTileK);
  const float weights = 4.f * d_kv * d_model;              // bytes of a layer
  const float few_weights_us = weights * kFewWeightsUsPerByte, weights_us = weights * n_layers * kWeightsUsPerByte;
  Route route;

  // the 256 x 256 tiles, whole or split
  const int nf = 2 * round_up(d_kv, kPartAlign) / kTileF, nt = (n_tok + kTileT - 1) / kTileT;
  float best;
  if (n_layers == 1 && free_order) {
    SplitPlan& sp = route.split_plan;
    route.split = plan_split(nf, nt, nm, false, sp, route.grid);
    if (route.split) {
      const int rest = n_tok - sp.nt_main * kTileT;      // tokens of the split tiles
      const float live = (float)round_up(rest, 16) / ((nt - sp.nt_main) * kTileT);
      float loop = 1.1f * kSplitStepUs * nm / sp.n_split;   // with most CUs busy
      if (loop < few_weights_us) loop = few_weights_us;
      best = kSplitPrice * (kWholeStepUs * nm * (nf * nt / kChipCUs) + loop + kSplitSlotUs * sp.n_tail * sp.n_split * live + kSplitFixedUs + kTileFixedUs);
    }
  }
  if (!route.split) {
    const float load = launch_load(nf, nt, nf, n_layers), rounds = ceilf(load);
    const float step_us = (kTileStepUs + kTileStepBusyUs * (load / rounds)) * (rounds > 1.f ? kTileNextRounds : 1.f);
    best = rounds * (step_us * nm + kTileFixedUs);
    if (n_layers > 1) best = sqrtf(best * best + weights_us * weights_us);
  }

  const int groups = d_kv / kPairGroup, groups_pad = round_up(d_kv, kPartAlign) / kPairGroup;
  for (int b = 1; b <= (n_layers > 1 || layer_norm ? 4 : 5); ++b) {
    auto cost = [&](float wgs) {                           // workgroups per CU of the busiest part
      const float loop_us = b == 1 && wgs > 1.f ? ceilf(wgs) * kMidSharedStepUs * nm
                                                : ceilf(wgs) * (kMidStepUs[b] * nm + kMidFixedUs + kMidBlockUs * b);
      return kMidPromise * sqrtf(loop_us * loop_us + weights_us * weights_us);
    };
    const int nt_b = (n_tok + 64 * b - 1) / (64 * b);
    if (b > 1 && cost((float)groups * nt_b * n_layers / kChipCUs) >= best) continue;   // even if the parts were equally busy
    const float wgs = launch_load(groups_pad, nt_b, groups, n_layers, b == 1);
    if (b == 1 && wgs > (n_layers > 1 ? 6.f : 2.f)) continue;
    float t = cost(wgs);
    if (t < best && nt_b > 1 && d_model > kStreamMinModel) t = fmaxf(t, l2_fill_us(groups_pad, nt_b, weights * n_layers, 2.f * d_model * n_tok * n_layers, 4.f * d_kv * n_tok * n_layers));
    if (t < best) { best = t; route.kind = Route::kMid; route.nb = b; }
  }

  const float others = best;                               // the tiles above
  if (d_model > kStreamMinModel && d_kv >= kStreamMinKv && n_layers <= kStreamMostLayers) {
    const StreamCost& k = kStreamCost[n_layers > 1];
    const float bytes_us = (weights + k.hidden_times * 2.f * (float)n_tok * d_model) * n_layers * k.us_per_byte;
    float stream = best;
    int nb = 0;
    for (int b = 2; b <= 6; ++b) {
      float loop_us;
      auto cost = [&](float wgs) {                         // workgroups per CU of the busiest part
        const float rounds = ceilf(wgs);
        const float step_us = k.step + k.block * b + (k.busy + k.busy_block * b) * (wgs / rounds) + (layer_norm ? k.norm_block * b : 0.f);
        loop_us = rounds * (step_us * nm * (1.f + k.more * fminf(rounds - 1.f, 9.f)) + k.round + k.round_block * b) + k.call;
        const float again_us = n_layers > 1 && rounds > 1.f && n_tok > 32 * b ? kStreamWeightsAgain * weights * n_layers * k.us_per_byte : 0.f;
        return k.promise * hypotf(loop_us, bytes_us + again_us);
      };
      const int nt_b = (n_tok + 32 * b - 1) / (32 * b);
      if (cost((float)groups * nt_b * n_layers / kChipCUs) >= stream) continue;   // even if the parts were equally busy
      const float wgs = launch_load(groups_pad, nt_b, groups, n_layers);
      if (n_layers == 1 && wgs > kStreamMostRounds) continue;
      float t = cost(wgs);
      if (n_layers > 1 && nt_b == 1 && wgs > 1.f && route.kind == Route::kTiles && weights * n_layers > kLastCacheBytes) t *= kStreamColdRounds;
      if (t < stream && nt_b > 1) t = fmaxf(t, l2_fill_us(groups_pad, nt_b, weights * n_layers, 2.f * d_model * n_tok * n_layers, 4.f * d_kv * n_tok * n_layers));
      if (t < stream) { stream = t; nb = n_layers == 1 || bytes_us < kStreamOverMemory * loop_us ? b : 0; }
    }
    if (nb) { best = stream; route.kind = Route::kStream; route.nb = nb; }
  }

  if (n_layers == 1 && free_order && d_model >= kSmallMinModel) {
    const int units = (2 * d_kv / kPairGroup + 7) / 8 * 2;   // 32-row units of the busiest XCD
    int nb = 0;
    float stream_us = 0.f;
    for (int b = 1; b <= 4; ++b) {
      const float load = (float)units * ((n_tok + 16 * b - 1) / (16 * b)) / (kChipCUs / 8);   // workgroups per CU
      const float in_turn = b <= 2 ? (load > 1.f ? load : 1.f) : ceilf(load);
      const float rounds = b <= 2 ? (load > 2.f ? load / 2 : 1.f) : in_turn;
      const float t = 2.85e-5f * d_model * in_turn * (32 + 16 * b) + kSmallRoundUs * (rounds - 1.f);
      if (b == 1 || t < stream_us) { stream_us = t; nb = b; }
    }
    const float t = 3.5f + sqrtf(stream_us * stream_us + few_weights_us * few_weights_us);
    if (t < others && t < best * (route.kind == Route::kStream ? kFewOverStream : 1.f)) { best = t; route.kind = Route::kSmall; route.nb = nb; }
  }
  // One round of 288 tokens is the least that wide_us answers; its launch_load is host time of every call.
  const WideCost& wide = kWideCost[n_layers > 1];
  if (d_model >= kWideMinModel && !layer_norm && wide.promise * (wide.step[0] * nm + wide.round) < best) {
    for (int b = 9; b <= 10; ++b) {
      const float t = wide.promise * wide_us(d_kv, d_model, n_tok, n_layers, b);
      if (t < best) { best = t; route.kind = Route::kWide; route.nb = b; }
    }
  }
  route.us = best;
  if (route.kind != Route::kTiles) route.split = false;
  if (layer_norm && route.kind == Route::kTiles && !route.split) route.sums_ahead = sums_pay_ahead(nf, nt, nm, n_tok, n_layers);
  return route;
}

// Arguments of one restoration launch (device pointers unless noted).
struct RestoreArgs {
  const uint16_t* hidden;        // bf16 [n_tok, d_model]
  const uint16_t* wpack;         // bf16 packed weight tiles [n_phys/256][d_model/32][16 blocks][4 chunks][16 rows][8], gamma folded in
  const int32_t* positions;      // [n_tok] or nullptr: position = pos_base + row
  const int32_t* cu_seqlens;     // [n_seq + 1] or nullptr (single context)
  const int32_t* block_tables;   // [n_seq][max_blocks]
  const float2* rope;            // [max_position][head_dim/2] (cos, sin); unused when rope_style = 2
  const float2* affine;          // [n_phys] per packed row: (sum of the row, constant term); modes 1, 2
  uint16_t* pool;                // bf16 [num_pages][2][block_size][n_kv_heads][head_dim]
  int32_t* err;                  // sticky error word
  int64_t num_pages;
  int32_t pos_base;
  int32_t n_seq;
  int32_t max_blocks;
  int32_t max_position;
  int32_t n_tok;
  int32_t d_model;
  int32_t d_kv;
  int32_t d_kv_pad;              // d_kv rounded up to kPartAlign
  int32_t head_dim;
  int32_t block_shift;           // log2(block_size)
  int32_t rope_style;            // 0 half-split, 1 interleaved, 2 no rotation
  int32_t mode;                  // 0 RMSNorm, 1 RMSNorm + bias, 2 LayerNorm + bias
  float inv_d;                   // 1 / d_model
  float eps;
  const float2* token_sums;      // [n_layers][n_tok] sums of squares and plain sums worked out ahead, or nullptr: in the tiles
  float* split_ws;               // workspace of the split launch, or nullptr: never split (host side only)
  int32_t split_force;           // split whenever the shape allows it, whatever the cost model says (host side only)
};

// Per-layer pointers of a launch that covers several layers of one context (the shared
// fields of RestoreArgs apply to all of them; its hidden / wpack / affine / pool / num_pages
// are ignored).  Passed by value as a kernel argument.
struct LayerEntry {
  const uint16_t* hidden;
  const uint16_t* wpack;
  const float2* affine;
  uint16_t* pool;
  int64_t num_pages;
};
// Layers per launch.  8 when a layer fills a good part of the chip: enough rounds of
// workgroups to hide the gaps between kernels, few enough that the CUs of an XCD stay close
// together and keep sharing weights in its L2 (measured at 256 tiles per layer: 16 and 32
// layers per launch fetch 4 % and 37 % more, and are no faster).  When a layer has fewer than
// 32 tiles (a short context), up to as many layers as would fill one round of 256 workgroups, at most 32:
// a launch takes a round's time however few of the CUs it uses.  Such a layer's tiles lie on few XCDs,
// consecutive layers on consecutive ones, so a launch can take two rounds with CUs free elsewhere; the count
// is the one with the fewest rounds over all launches of the call, of those with the fewest launches, and
// of those a multiple of eight, which loads the XCDs evenly (24 layers of 20 tiles: three times eight, not
// 11 + 11 + 2), or else the largest.
// 32 layers of 4096 onto 2048, 600 tokens (24 tiles a layer): 578 us in tens, which take two rounds each
// but for the last two layers, 381 in eights, which take one; 10 layers of 640 onto 5632, 239 tokens (22
// tiles): 36.8 us in one launch of two rounds, 56.8 as 8 + 2; 20 of 128 onto 1536, 271 tokens: 27.1 in
// one launch, 36.2 as 16 + 4.
constexpr int kMaxLayersPerLaunch = 32;
inline int layers_per_launch(int nf, int nt, int n_layers) {
  int most = kChipCUs / (nf * nt);
  if (most > kMaxLayersPerLaunch) most = kMaxLayersPerLaunch;
  if (most > n_layers) most = n_layers;
  if (most <= 8) return 8;
  TileGrid g;
  const int slots = choose_tile_grid(nf, nt, g);
  const ChipLoad load(g, slots, nf);
  int best = 0, best_rounds = 0, best_launches = 0;
  for (int n = most; n >= 8; --n) {
    const int launches = (n_layers + n - 1) / n, rounds = n_layers / n * load.rounds(n) + load.rounds(n_layers % n);
    if (best == 0 || rounds < best_rounds || (rounds == best_rounds && launches <= best_launches && n % 8 == 0 && best % 8 != 0)) {
      best = n; best_rounds = rounds; best_launches = launches;
    }
  }
  return best;
}
// Layers per launch on the tiles of 288 or 320 tokens: as many as fill one round of the chip.
inline int wide_layers_per_launch(int d_kv, int n_tok, int nb, int n_layers) {
  const int tiles = 2 * round_up(d_kv, kPartAlign) / kTileF * ((n_tok + 32 * nb - 1) / (32 * nb));
  int n = kChipCUs / tiles;
  if (n > kMaxLayersPerLaunch) n = kMaxLayersPerLaunch;
  if (n > n_layers) n = n_layers;
  return n < 8 ? 8 : n;
}
struct LayerBatch {
  LayerEntry e[kMaxLayersPerLaunch];
  int32_t slots_per_layer;     // workgroups per layer (a multiple of 8); set by launch_restore
};

// Launchers implemented in the .hip files.  All are asynchronous on `stream`.
// `batch` null: one layer from `a`; else n_layers <= kMaxLayersPerLaunch layers in one launch.  `route` is
// restore_route's for the same arguments.
hipError_t launch_restore(const RestoreArgs& a, const Route& route, LayerBatch* batch, int n_layers, hipStream_t stream);
// Tiles of 128 packed rows x 64 nb tokens (nb 1..5), one launch; `batch` as in launch_restore.
hipError_t launch_restore_mid(const RestoreArgs& a, int nb, LayerBatch* batch, int n_layers, hipStream_t stream);
// Tiles of 128 packed rows x 32 nb tokens with loader waves (nb 2..6), one launch; `batch` as in launch_restore.
hipError_t launch_restore_stream(const RestoreArgs& a, int nb, LayerBatch* batch, int n_layers, hipStream_t stream);
// Tiles of 256 packed rows x 32 nb tokens (nb 9 or 10; not LayerNorm), one launch; `batch` as in launch_restore.
hipError_t launch_restore_wide(const RestoreArgs& a, int nb, LayerBatch* batch, int n_layers, hipStream_t stream);
hipError_t launch_restore_small(const RestoreArgs& a, int nb, hipStream_t stream);
// The kernel a launch of n_layers layers of `a` takes.  A context that asks for split launches gets the
// 256 x 256 tiles.
inline Route restore_route(const RestoreArgs& a, int n_layers) {
  Route r;
  if (!a.split_force) r = plan_route(a.d_kv, a.d_model, a.n_tok, n_layers, a.mode == 2, a.split_ws != nullptr);
  else if (a.split_ws)
    r.split = plan_split(2 * a.d_kv_pad / kTileF, (a.n_tok + kTileT - 1) / kTileT, a.d_model / (2 * kTileK), true, r.split_plan, r.grid);
  r.split_plan.ws = a.split_ws;
  return r;
}
// Layers in the first launch of a call over n_layers layers of `a` (layers_per_launch), and its route; or more of them on the tiles
// of 288 or 320 tokens where the whole call is estimated to take less that way.  A call is its full launches and the last one, of
// the layers that are left, which goes its own way: 33 layers of 257 tokens of 8192 channels onto 2048 take 337 us as 32 on those tiles
// and one, 477 as 16 + 16 + 1.  (Counting the last launch as a full one refused that, and 20 layers of 1153 tokens of 2112 onto 640
// went out as one launch of 300 workgroups: 117.5 us, as 16 of 320 tokens and 4 111.)
inline int plan_layers(const RestoreArgs& a, int n_layers, Route& route) {
  const int per = layers_per_launch(2 * a.d_kv_pad / kTileF, (a.n_tok + kTileT - 1) / kTileT, n_layers);
  int n = per < n_layers ? per : n_layers;
  route = restore_route(a, n);
  if (a.split_force || a.mode == 2 || a.d_model < kWideMinModel || n == n_layers) return n;
  float call_us = -1.f;                                  // of the choice so far; worked out where it is asked for
  auto last_us = [&](int per_launch) { const int rest = n_layers % per_launch; return rest ? restore_route(a, rest).us : 0.f; };
  for (int b = 9; b <= 10; ++b) {
    const int n_wide = wide_layers_per_launch(a.d_kv, a.n_tok, b, n_layers);
    if (n_wide <= per) continue;
    if (call_us < 0.f) call_us = route.us * (n_layers / n) + last_us(n);
    const float us = kWideCallPromise * wide_us(a.d_kv, a.d_model, a.n_tok, n_wide, b), full_us = us * (n_layers / n_wide);
    if (full_us >= call_us) continue;
    const float t = full_us + last_us(n_wide);
    if (t >= call_us) continue;
    call_us = t;
    n = n_wide;
    route = Route();
    route.kind = Route::kWide;
    route.nb = b;
    route.us = us;
  }
  return n;
}
// What a context's split mode asks of a launch: `several` layers in one launch never split, but they take
// the 256 x 256 tiles too when split launches are asked for.
inline void set_split_rule(RestoreArgs& a, int split_mode, float* split_ws, bool several) {
  a.split_ws = !several && split_mode ? split_ws : nullptr;
  a.split_force = split_mode == 2;
}
// The tokens' sums of squares and plain sums of n_layers layers (`batch`, or a.hidden) into `out` [n_layers][n_tok].
hipError_t launch_token_sums(const RestoreArgs& a, const LayerBatch* batch, int n_layers, float2* out, hipStream_t stream);
hipError_t launch_pack_weights(const uint16_t* wkv, const uint16_t* gamma, uint16_t* wpack,
                               int d_model, int d_kv, int head_dim, int rope_style,
                               hipStream_t stream);
// Per packed row n: (sum_c W'[n,c], sum_c W[n,c] * beta[c] + bias[n]) with W' the rounded,
// gain-folded weights the pack kernel writes; beta and bias may be null (zeros).
hipError_t launch_pack_affine(const uint16_t* wkv, const uint16_t* gamma, const uint16_t* beta,
                              const uint16_t* bias, float2* affine, int d_model, int d_kv,
                              int head_dim, int rope_style, hipStream_t stream);
hipError_t launch_rope_table(float2* table, int max_position, int head_dim, double theta,
                             hipStream_t stream);
hipError_t configure_mid();
hipError_t configure_stream();
hipError_t configure_wide();
hipError_t configure_kernels();   // one-time function attributes (dynamic LDS size)
// Measurement only: chip-wide matrix-op rate (TFLOP/s, as if all 256 CUs were busy) inside
// the busy windows of a duty-cycled burst pattern; allocates and frees its own buffers and
// synchronises the device.
hipError_t run_mfma_duty(double period_us, double duty, int half_phase, double total_us,
                         int zero_operands, int op_shape, double* out_tflops);

// One contiguous piece of a layer's hidden states in the host store and where it goes in
// the HBM staging buffer.  `bytes` is a multiple of 16.
struct CopySegment {
  const void* src;   // pinned host memory (device-readable)
  void* dst;         // HBM
  uint64_t bytes;
};
constexpr int kGatherBlocksPerSegment = 8;
// Copies n_seg segments with a kernel that reads the pinned host memory directly
// (kGatherBlocksPerSegment workgroups per segment); `segs` must be device-readable.
hipError_t launch_gather(const CopySegment* segs, int n_seg, hipStream_t stream);

// Token rows [n_tok][K | V] (2 * d_kv bf16) <-> pages of one layer's pool.
struct KvRowsArgs {
  uint16_t* rows;                // bf16 [n_tok][2 * d_kv]
  uint16_t* pool;                // bf16 [num_pages][2][block_size][d_kv]
  const int32_t* positions;      // [n_tok] or nullptr: position = pos_base + row
  const int32_t* block_table;    // [n_blocks]
  int32_t* err;                  // sticky error word
  int64_t num_pages;
  int32_t pos_base, n_tok, n_blocks, max_position, d_kv, block_shift;
};
hipError_t launch_kv_rows(const KvRowsArgs& a, bool to_pool, hipStream_t stream);

// Error plumbing: thread-local message + status.
hc_status fail(hc_status code, const std::string& msg);
hc_status fail_hip(hipError_t e, const char* what);
void clear_error();

#define HC_HIP(call)                                         \
  do {                                                       \
    hipError_t e_ = (call);                                  \
    if (e_ != hipSuccess) return ::hc::fail_hip(e_, #call);  \
  } while (0)

}  // namespace hc

struct hc_ctx;
namespace hc {
// Validated launch of the fused kernel for one layer (shared by every restore entry point).
// positions == nullptr means position = pos_base + row.
hc_status restore_layer(hc_ctx* ctx, int32_t layer, const void* d_hidden,
                        const int32_t* d_positions, int32_t pos_base, int32_t n_tok,
                        const int32_t* d_cu, int32_t n_seq, const int32_t* d_tables,
                        int32_t max_blocks, hipStream_t stream);
// The same for layers [layer_begin, layer_begin + n_layers) of one context, hidden states of
// layer layer_begin + i at d_hidden[i] (host array of device pointers); as few launches as
// kMaxLayersPerLaunch and equal kernel modes allow.
hc_status restore_layers(hc_ctx* ctx, int32_t layer_begin, int32_t n_layers,
                         const void* const* d_hidden, const int32_t* d_positions, int32_t pos_base,
                         int32_t n_tok, const int32_t* d_block_table, int32_t n_blocks,
                         hipStream_t stream);
// Validated launch of the KV row copy for one layer: rows -> pages (to_pool) or pages -> rows.
hc_status kv_rows_layer(hc_ctx* ctx, int32_t layer, void* d_rows, const int32_t* d_positions,
                        int32_t pos_base, int32_t n_tok, const int32_t* d_block_table,
                        int32_t n_blocks, bool to_pool, hipStream_t stream);
}  // namespace hc

struct hc_layer_state {
  uint16_t* wpack = nullptr;     // owned
  float2* affine = nullptr;      // owned; present when the layer has a shift or a bias, or LayerNorm
  uint16_t* pool = nullptr;      // borrowed
  int64_t num_pages = 0;
};

struct hc_ctx {
  hc_model_desc desc;
  int device = 0;
  int d_kv = 0, d_kv_pad = 0, n_phys = 0, block_shift = 0;
  float2* rope = nullptr;                 // owned, device
  int32_t* err_dev = nullptr;             // owned, device: sticky error word
  std::vector<hc_layer_state> layers;
  // staging for hc_restore_context
  uint16_t* stage[2] = {nullptr, nullptr};
  size_t stage_bytes = 0;
  hipEvent_t h2d_done[2] = {nullptr, nullptr};
  hipEvent_t buf_free[2] = {nullptr, nullptr};
  int loader_mode = 0;                    // 0 = copy engines (strided runs), 1 = gather kernel
  hipStream_t copy2 = nullptr;            // owned: second copy stream of hc_restore_context (odd layers)
  // workspace of split single-layer launches (owned, device; allocated with the context so that
  // no restore call allocates) and the event recorded behind its last reader: a split launch on
  // another stream waits for it
  float* split_ws = nullptr;
  hipEvent_t split_done = nullptr;
  // slots of the tokens' sums worked out ahead of a launch (behind the split workspace), used in turn, each guarded by an
  // event recorded behind its last reader
  float2* sums = nullptr;
  hipEvent_t sums_done[hc::kSumsSlots] = {};
  int sums_next = 0;
  std::mutex sums_mutex;
  int split_mode = 1;                     // 0 = never split, 1 = when plan_split's cost model says so, 2 = whenever possible
  // segment tables of the gather loader: pinned host memory the kernel reads directly; two of
  // them, used alternately, each guarded by an event recorded after its last reader
  hc::CopySegment* seg_tab[2] = {nullptr, nullptr};
  size_t seg_cap[2] = {0, 0};
  hipEvent_t seg_done[2] = {nullptr, nullptr};
  int seg_next = 0;
  // row offsets (cu_seqlens) of hc_restore_contexts: two pinned tables with device copies, used
  // alternately, each guarded by an event recorded after the last kernel that reads it
  int32_t* cu_host[2] = {nullptr, nullptr};
  int32_t* cu_dev[2] = {nullptr, nullptr};
  int cu_cap[2] = {0, 0};
  hipEvent_t cu_done[2] = {nullptr, nullptr};
  int cu_next = 0;
  // per-launch timing
  bool timing = false;
  std::vector<hipEvent_t> ev_pool;        // created on demand, reused
  int ev_used = 0;
};

struct hc_seq_state {
  std::vector<int64_t> rows;                  // arena row of each chunk index (shared by all layers)
  std::vector<std::vector<int64_t>> chunks;   // per layer: arena chunk slots, in token order
  std::vector<int64_t> tokens;                // per layer: rows stored
};

// The arena is cut into ROWS of n_layers chunk slots: chunk index c of a context takes one row,
// layer l's chunk sitting at slot row * n_layers + l.  A layer's chunks are therefore exactly
// n_layers slots apart wherever the context's rows are consecutive, however the appends of
// different contexts and layers interleave, and one strided transfer moves them all.  Rows are
// handed out one at a time, with no reservation: a context continues right behind its last row
// while that row is free; otherwise it starts a new run in the largest free extent -- at its
// start, or in its middle when another context is growing into that extent from below (one
// that took a row within the last kGrowthWindow allocations), so that contexts that arrive
// interleaved each keep long runs of their own.
constexpr int64_t kGrowthWindow = 64;
struct hc_store {
  int32_t n_layers = 0, d_model = 0, chunk_tokens = 0;
  int64_t capacity_chunks = 0;
  int64_t rows_total = 0, rows_free = 0;
  size_t row_bytes = 0, chunk_bytes = 0;
  unsigned char* arena = nullptr;
  bool pinned = false;
  std::map<int64_t, int64_t> free_extents;    // first row -> number of rows, maximal and disjoint
  std::unordered_map<int64_t, int64_t> growth;   // row behind a context's last row -> allocation count then
  int64_t alloc_count = 0;                    // rows handed out so far
  std::unordered_map<int64_t, hc_seq_state> seqs;
  // guards the index (seqs, free_extents, growth): appends, drops and the readers that copy
  // chunk lists out of it may run on different threads; row payloads are copied outside of it
  mutable std::mutex index_mutex;
};

namespace hc {
// One copy-engine transfer of a pipelined restore: `rows` pieces of `row_bytes` each, `pitch`
// bytes apart at the source (pinned arena) and back to back at the destination (HBM).
struct CopyRun { const unsigned char* src; unsigned char* dst; size_t row_bytes; size_t pitch; int rows; };

// Copy-engine runs that bring tokens [tok_begin, tok_begin + n_tok) of one (context, layer) to
// `dst` (row 0 of the range): partial first / last chunks on their own, full chunks grouped
// while their arena slots stay equally spaced (one strided copy per group).  `emit(run)` is
// called per run in token order and returns false to stop early; the result says whether
// every run was emitted.  Nothing is allocated here.
template <class Emit>
inline bool for_each_run(const hc_store* st, const std::vector<int64_t>& chunks, int tok_begin,
                         int n_tok, unsigned char* dst, Emit&& emit) {
  const int CT = st->chunk_tokens;
  const int c_first = tok_begin / CT, c_last = (tok_begin + n_tok - 1) / CT;
  auto dst_at = [&](int c, int lo) { return dst + (size_t)(c * CT + lo - tok_begin) * st->row_bytes; };
  auto full = [&](int cc) { return cc < c_last || tok_begin + n_tok - cc * CT == CT; };
  int c = c_first;
  while (c <= c_last) {
    const int lo = c == c_first ? tok_begin - c * CT : 0;
    const int hi = c == c_last ? tok_begin + n_tok - c * CT : CT;
    const unsigned char* src = st->arena + (size_t)chunks[c] * st->chunk_bytes + (size_t)lo * st->row_bytes;
    if (lo != 0 || hi != CT) {
      if (!emit(CopyRun{src, dst_at(c, lo), (size_t)(hi - lo) * st->row_bytes, 0, 1})) return false;
      ++c;
      continue;
    }
    int c_end = c;
    int64_t stride = 0;
    if (c + 1 <= c_last && full(c + 1)) {
      stride = chunks[c + 1] - chunks[c];
      if (stride > 0) {
        c_end = c + 1;
        while (c_end + 1 <= c_last && full(c_end + 1) && chunks[c_end + 1] - chunks[c_end] == stride) ++c_end;
      }
    }
    if (!emit(CopyRun{src, dst_at(c, 0), st->chunk_bytes, (size_t)stride * st->chunk_bytes, c_end - c + 1}))
      return false;
    c = c_end + 1;
  }
  return true;
}

// Every run goes out in the two-dimensional form, a single piece as one row: measured here, a
// plain hipMemcpyAsync of a few MiB from the pinned arena is served several times slower than
// the same bytes as a 2D copy while the restoration kernel occupies the CUs (256 tokens of the
// Llama-3-8B shape, one 2 MiB chunk per layer: 8.6 ms per restore against 1.8 ms).
inline hc_status enqueue_run(const CopyRun& r, hipStream_t xs) {
  const size_t pitch = r.rows == 1 ? r.row_bytes : r.pitch;
  HC_HIP(hipMemcpy2DAsync(r.dst, r.row_bytes, r.src, pitch, r.row_bytes, r.rows, hipMemcpyHostToDevice, xs));
  return HC_OK;
}

// Device-resident scratch of the entry point that allocates nothing (static_restore.hip):
// looks the array's address up and creates the handshake events once per device.
hc_status static_scratch_init();

// One contiguous destination of appended rows: `bytes` from offset `src_off` of the source.
struct StorePiece {
  unsigned char* dst;
  size_t src_off, bytes;
};
hc_status store_reserve(hc_store* st, int64_t seq_id, int32_t layer, int32_t n_tok,
                        std::vector<StorePiece>& pieces);
}  // namespace hc
