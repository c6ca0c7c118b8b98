// Kernel parameter blocks and launchers (host <-> device interface inside the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace mw {

// Element strides of a [B, H, T, D] tensor view (D contiguous): element
// (b, h, t, d) is at base + b * b_ + h * h_ + t * t_ + d.
struct Strides {
  long long b;
  long long h;
  long long t;
};

// Forward / cached attention.  Queries: [BH, Tq, D]; keys: the (virtual) key
// sequence of length vis.Tk described below; output O [BH, Tq, D], lse [BH, Tq].
struct FwdParams {
  const uint16_t* q;
  const uint16_t* k;  // training: [BH, Tk, D]; cached: the queued chunks' keys [BH, Tq, D]
  const uint16_t* v;
  uint16_t* o;
  float* lse;  // may be null (cached attention)
  int BH;
  int H;
  int Tq;
  int n_qtiles;   // set by the launcher from its tile configuration
  int vis_mode;  // VisMode
  int L;         // chunk length (training) / committed chunk length (cached)
  int Tk;        // keys in the (virtual) sequence
  int qlen;      // queued chunk length (cached)
  int wL;        // history tokens = sink_len + n_window * L (cached; 0 in training)
  float scale_log2;  // softmax scale * log2(e)
  float scale_ln;    // unused by the kernels; kept for the host's records
  // cached attention only: the window lives in ring slots
  const uint16_t* k_slots;
  const uint16_t* v_slots;
  const uint16_t* k_sink;  // [BH, sink_len, D], first in the key sequence
  const uint16_t* v_sink;
  int sink_len;
  long long slot_stride;  // elements per slot (B*H*L*D)
  int S;                  // ring capacity in slots
  int first_slot;         // slot of the oldest window chunk; chunk i of the window is in slot (first_slot+i)%S
  // key-range splitting (cached attention, n_splits > 1): the n_whole heaviest
  // (last) query tiles of each head run unsplit; each of the others is covered
  // by n_splits workgroups, one per 1/n_splits of its key tiles, which write
  // fp32 partials for a merge kernel (see attn_fwd.hip).  The split tiles are a
  // head's first ones: rows [0, split_rows), set by the launcher.
  int n_splits;
  int n_whole;
  int split_rows;
  float* part;  // [n_splits][BH][split_rows][D] unnormalised O, then [n_splits][BH][split_rows][2] (m, l)
  // views of q, k (training keys / queued keys), v and o; lse and the ring
  // are always contiguous
  Strides sq, sk, sv, so;
  // fp8 kernel only: q, k, v, the slots and the sink hold e4m3 bytes
  // (contiguous; element strides are byte strides) and O is multiplied by
  // o_scale (the V scale) before it is stored
  float o_scale;
  // fp8 kernel only: window keys rotated on load, [n_window][BH, L, 128] bytes
  // in window order (chunk w at w * slot_stride), or null (keys from the slots)
  const uint8_t* k_win;
};

struct BwdParams {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const uint16_t* o;
  const uint16_t* d_o;
  const float* lse;
  float* delta;  // workspace [BH, T]: -rowsum(dO * O)
  float* lse2;   // workspace [BH, T]: LSE * log2(e)
  uint16_t* dq;
  uint16_t* dk;
  uint16_t* dv;
  int BH;
  int H;
  int T;
  int L;
  float scale;
  float scale_log2;
  // views of the [B, H, T, D] tensors; lse, delta and lse2 are contiguous [B, H, T]
  Strides sq, sk, sv, so, sdo, sdq, sdk, sdv;
};


hipError_t launch_fwd_64(const FwdParams& p, bool cached, hipStream_t stream);
hipError_t launch_fwd_72(const FwdParams& p, bool cached, hipStream_t stream);
hipError_t launch_fwd_128(const FwdParams& p, bool cached, hipStream_t stream);
// cached attention at D = 128: the 256-row configuration, and the few-row ones
hipError_t launch_fwd_cached_128(const FwdParams& p, hipStream_t stream);
hipError_t launch_fwd_decode_128(const FwdParams& p, hipStream_t stream);
// the D = 128 tiles for grids that do not fill the card
enum class GridFill;
hipError_t launch_fwd_small_128(const FwdParams& p, GridFill fill, hipStream_t stream);
enum class UnsplitTile;
hipError_t launch_fwd_unsplit_128(const FwdParams& p, UnsplitTile tile, hipStream_t stream);
inline hipError_t launch_fwd(const FwdParams& p, int D, bool cached, hipStream_t stream) {
  return D == 64 ? launch_fwd_64(p, cached, stream)
                 : (D == 72 ? launch_fwd_72(p, cached, stream) : launch_fwd_128(p, cached, stream));
}
// Query rows per workgroup, keys per main-loop step and resident workgroups
// per CU (runtime occupancy; the value the kernel's register and LDS use gives
// as built where no device is present) of the tile configuration the launcher
// picks for a cached call of Tq queued rows.
struct FwdChoice {
  int bm;
  int bk;
  int wg_per_cu;
  // for the price of a call bound by streaming its keys:
  double lone_rate;  // share of a CU's streaming rate that one workgroup alone on it reaches
  double part_rate;  // rate of its partials, written and read back, against HBM's
};
FwdChoice fwd_choice(int D, int Tq);
FwdChoice fwd_choice_64(int Tq);
FwdChoice fwd_choice_72(int Tq);
FwdChoice fwd_choice_cached_128();
FwdChoice fwd_choice_decode_128(int Tq);
// How far a call without a key-range split fills the card, counted in 64-row
// tiles of the key sequence (in training also the query sequence) over all
// heads; the forward launchers pick their tile by it.  Measured on MI355X,
// training forward, us, as (256-row | 128 | 64 | 64 in four key groups) where
// a line was drawn:
//   sparse  one eight-wave workgroup per CU, or up to 1.5 (2 at D = 64) where
//           the sequence is long enough that half the tiles are light:
//           D = 128, 1 x 8000 (183 | 143 | 96 | 76), 8 x 2200 (60 | - | 33 | 30),
//           12 x 1500 (45 | - | 26 | 27); D = 64, 4 x 4000 (86 | 61 | 40 | 28).  A
//           short sequence does not repay merging four groups: D = 128,
//           8 x 600 (25 | - | 12 | 14); D = 64, 2 x 256 (13 | 7.5 | 5.4 | 5.9).
//   small   up to 1.5 rounds of resident 64-row workgroups, at D = 72 and 128 about
//           one where the sequence is short and its tiles of much the same weight:
//           D = 128, 24 x 2000 (56 | 47 | 47), against 128 rows 12 x 2800 +15%, 9 x
//           4800 +9%, 24 x 1500 +14%, 36 x 1000 +7%, 64 x 512 +14%, 40 x 1000 -4%, 96 x
//           330 -10%, 144 x 200 -13%; D = 72, 16 x 3000 (67 | 53 | 43), 24 x 3600
//           (94 | 90 | 90), 25 x 3000 +4%, 56 x 1000 +8%, 64 x 1000 -7%, 96 x 512 +5%, 112 x
//           512 -19%; D = 64, 24 x 3600 (89 | 76 | 69), 40 x 2048 +2%, 128 x 512 +8%.
//   mid     D = 128 up to 1.5 rounds of resident 128-row workgroups: 16 x 4800
//           (131 | 118 | 130), 12 x 7200 (198 | 179 | 208), 12 x 9600 (300 | 314 | -).
//   large   D = 64 from about two rounds of 256-row workgroups on, whose two row
//           blocks per wave halve the LDS reads of K and V: 16 x 42240 (3765 | 4025),
//           16 x 19200 (831 | 873), 7 x 42240 (1765 | 1837), 96 x 4800 (381 | 393);
//           below, their last round costs more: 24 x 10560 (468 | 464), 16 x 14400
//           (520 | 511), 4 x 42240 (1105 | 1090), 8 x 19200 (497 | 476).
enum class GridFill { sparse, small, mid, full, large };
inline GridFill grid_fill(int D, int BH, int Tk) {
  const long long tiles = (long long)BH * ((Tk + 63) / 64);
  if (tiles <= 256 && Tk >= (D == 128 ? 1536 : 512)) return GridFill::sparse;
  if (tiles <= (D == 64 ? 512 : 384) && Tk >= 2048) return GridFill::sparse;
  const int small = D == 64    ? 1536
                    : D == 72 ? (Tk < 768 ? 800 : Tk < 2500 ? 960 : 1152)
                              : (Tk < 256 ? 384 : Tk < 1000 ? 544 : Tk < 2048 ? 608 : 768);
  if (tiles <= small) return GridFill::small;
  if (D == 128 && tiles <= 1536) return GridFill::mid;
  return D == 64 && tiles > 4300 ? GridFill::large : GridFill::full;
}
// Tile of a cached call without a key-range split: that of the split plans
// (fwd_choice), whose whole tiles the call then gives bit for bit, or one of its
// own, as the training forward has for the same heads and keys.  `training_rows`:
// the call's rows see their keys as training rows do (queued-causal, or one queued
// chunk).  At D = 64 and 72, and at D = 128 for more than 512 rows, such a call then
// splits each key step among as many wave groups as the training forward, and over
// a whole history gives its rows bit for bit.  us against the split plans' tiles, D =
// 64 | 72: 24 heads x 600 rows over 1800 keys 24 for 44 | 27 for 37, 40 x 256 over
// 1456 21 for 29 | 24 for 32, 8 x 64 over 3664 31 for 45 | 36 for 57; for the rows'
// sake 64 x 64 over 3664 62 for 45 | 70 for 59.  Other calls of more than 64 rows have
// the groups up to 512 64-row tiles (two a CU).
enum class UnsplitTile { plan = 0, groups4, groups2, rows128 };
inline UnsplitTile unsplit_tile(int D, int BH, int Tq, int Tk, bool training_rows) {
  if (D == 128 && Tq <= 512) return UnsplitTile::plan;
  if (!training_rows && (Tq <= 64 || (long long)BH * ((Tk + 63) / 64) > 512)) return UnsplitTile::plan;
  const GridFill fill = grid_fill(D, BH, Tk);
  if (fill == GridFill::sparse) return UnsplitTile::groups4;
  // (64 rows of a split plan have the two groups too)
  if (fill == GridFill::small) return Tq <= 64 ? UnsplitTile::plan : UnsplitTile::groups2;
  return D != 128 && Tq <= 64 ? UnsplitTile::rows128 : UnsplitTile::plan;
}
// fp8 (e4m3) cached attention at D = 128: its tile configuration and launcher
// (FwdParams as described above), and the merge of split partials (D = 128).
FwdChoice fwd8_choice(int Tq);
hipError_t launch_combine(const FwdParams& p, int D, hipStream_t stream);
// bf16 view -> contiguous e4m3, code = RNE(clamp(x * inv_scale, +-448)); up to
// two jobs of the same shape in one launch.
struct QuantJob {
  const uint16_t* x;
  Strides sx;
  uint8_t* y;
  float inv_scale;
};
struct QuantJobs {
  QuantJob j[2];
};
hipError_t launch_quantize_fp8(const QuantJobs& jobs, int n_jobs, int B, int H, int T, int D, hipStream_t stream);
// Key-range split plan of a cached call: the n_whole heaviest query tiles of
// each head run unsplit, the others over n_splits key ranges (n_splits = 1:
// no split, n_whole = 0).
struct SplitPlan {
  int n_splits;
  int n_whole;
};
// Plan for a call run by the configuration `ch` at `flops` FLOP/s of
// sustained MFMA throughput, over K/V elements of `kv_bytes` bytes, with
// queued chunks of `qlen` rows (`isolated`: each sees only the history and
// itself), within `ws_bytes` of workspace.
SplitPlan fwd_plan_splits(const FwdChoice& ch, double flops, int kv_bytes, int D, int BH, int Tq, int Tk, int qlen,
                          bool isolated, size_t ws_bytes);
// The plan of the bf16 cached launcher (its configuration and sustained rate).
SplitPlan fwd_plan_cached(int D, int BH, int Tq, int Tk, int qlen, bool isolated, size_t ws_bytes);
// Rows per head covered by the split tiles (0 without a split), and the
// workspace bytes of their partials.
int fwd_split_rows(int bm, int Tq, const SplitPlan& sp);
size_t fwd_split_bytes(int D, int BH, int split_rows, int n_splits);
// Grid of a forward launch with `bm`-row tiles, after setting the split fields
// of p: n_qtiles, and for a split (cached attention only) the whole-tile count
// clamped to the tiles and the rows of the split tiles.
inline long long fwd_prepare(FwdParams& p, int bm, bool cached) {
  p.n_qtiles = (p.Tq + bm - 1) / bm;
  if (p.n_splits < 1 || !cached) p.n_splits = 1;
  p.n_whole = p.n_whole < 0 ? 0 : (p.n_whole > p.n_qtiles ? p.n_qtiles : p.n_whole);
  if (p.n_whole == p.n_qtiles) p.n_splits = 1;
  if (p.n_splits == 1) p.n_whole = 0;
  p.split_rows = fwd_split_rows(bm, p.Tq, SplitPlan{p.n_splits, p.n_whole});
  return (long long)p.BH * (p.n_whole + (long long)(p.n_qtiles - p.n_whole) * p.n_splits);
}
// Configuration of the gradient grid (attn_bwd.hip), by the 64-row tiles of the
// sequence over all heads and its length.  A wave walks about T / 64 steps of
// 1.3 us; a small grid is bound by that chain, so two or four wave groups split
// it, for the price of staging Q and dO (K and V) for half the keys (queries), and
// the merge.  Backward with its row terms, us, as (128 rows | 64 in two groups |
// 64 in four), on both sides of each line:
//   four groups: the longer the chain, the more tiles; a short one does not repay
//   the merge (D = 64: 4 x 512 +4% against two, 4 x 768 -1%; D = 128: 4 x 400 +7%,
//   4 x 512 -1%).  D = 64: 2 x 1024 (29 | 21 | 18),
//   12 x 1024 (- | 31 | 34), 4 x 2500 (55 | 39 | 31), 8 x 2048 (- | 40 | 44),
//   4 x 4096 (81 | 58 | 53), 5 x 4096 (84 | 62 | 69), 1 x 24000 (435 | 304 | 283),
//   1 x 30000 (564 | 405 | 444); D = 72: 9 x 1024 +3%, 5 x 2500 -3%, 3 x 6800 +2%
//   against two; D = 128: 12 x 1024 +7%, 8 x 1500 -2%, 6 x 3000 -1%, 3 x 8000
//   (310 | 210 | 216), 2 x 12000 (450 | 303 | 283), 2 x 16000 (618 | 429 | 475);
//   two groups: up to about one round of 128-row workgroups (512 to 576 64-row
//   tiles), fewer where the sequence is short and every tile of much the same
//   weight.  D = 64: 46 x 512 (360 tiles) -6%, 60 x 512 -1%, 68 x 512 +13%; 32 x
//   1000 (32 | 29), 36 x 1000 +9%; 18 x 2000 -2%, 20 x 2000 +2%; D = 72: 36 x 700
//   -1%, 40 x 700 +2%, 23 x 1500 -5%, 24 x 1500 (64 | 67); D = 128: 64 x 512 -5%, 68
//   x 512 +8%, 67 x 330 -2%, 80 x 330 +5%;
//   wide3 (D = 64; three waves per SIMD) where a third workgroup per CU does not
//   only add to the longest chain, us as (wide | wide3): 8 x 7200 (191 | 215), 1 x
//   60000 (1382 | 1639), 12 x 5120 (153 | 164), 4 x 18000 (563 | 591), 6 x 13000
//   (473 | 452), 8 x 12000 (527 | 510), 24 x 10560 (1268 | 1247), and with short
//   chains 24 x 2500 (103 | 96), 48 x 1280 (68 | 61), 20 x 3200 (116 | 115).
enum class BwdGrid { wide = 0, pairs = 2, wide3 = 3, quads = 4 };
inline BwdGrid bwd_grid(int D, int BH, int T) {
  const long long tiles = (long long)BH * ((T + 63) / 64);
  const double chain = std::log2((double)T) - 8;
  if (T >= (D == 128 ? 512 : 768) && tiles <= (D == 128 ? 75 * chain : std::min(440., 70 * chain))) return BwdGrid::quads;
  if (tiles <= (D == 128 ? std::min(576, 256 + T / 2) : std::min({576, 272 + T / 4, 480 + T / 20}))) return BwdGrid::pairs;
  if (D == 64 && (tiles > 1130 || (tiles > 900 && T <= 3200))) return BwdGrid::wide3;
  return BwdGrid::wide;
}
// The rules above and the training grids' work order (tile_item of mw_device.h), for
// the host tests.
int training_fwd_fill(int D, int BH, int T);
int cached_unsplit_tile(int D, int BH, int Tq, int Tk, int training_rows);
int training_bwd_grid(int D, int BH, int T);
void training_work_item(int bid, int BH, int& bh, int& rank);
hipError_t launch_bwd_64(const BwdParams& p, hipStream_t stream);
hipError_t launch_bwd_72(const BwdParams& p, hipStream_t stream);
hipError_t launch_bwd_128(const BwdParams& p, hipStream_t stream);
// cos/sin of the re-shift angle of each rope pair
struct RopeTable {
  float c[64];
  float s[64];
};
hipError_t launch_rope_shift(uint16_t* k_slots, long long slot_stride, int S, int first_slot, int n_live,
                             long long rows_per_slot, int D, int dim_offset, int n_pairs, const RopeTable& tab,
                             hipStream_t stream);
// Rotation on load of an e4m3 cache's window keys: window chunk w (in window
// order, in slot (first_slot + w) % S) is rotated by -pend[w] positions on the
// band [dim_offset, dim_offset + 2 n_pairs); c1[i], s1[i] are the cos and sin
// of pair i's frequency (its rotation per position).
struct RopeLoadArgs {
  long long pend[64];
  double c1[64];
  double s1[64];
};
// The same rotation done inside the e4m3 attention kernel's staging, on each
// staged K tile in LDS (calls with one query tile per head): pend[w] for the
// window chunks of the call, band as above; n_pairs = 0 rotates nothing.
struct RopeStage {
  RopeLoadArgs a;
  int n_pairs;
  int dim_offset;
};
// Window chunks one workgroup of the in-staging rotation can span (their
// cos/sin tables live in LDS).
constexpr int kRopeStageChunks = 8;
// Whether a call (Tq queued rows over Tk keys, window chunks of L keys, split
// plan sp) has one query tile per head and every workgroup's key range
// spans at most kRopeStageChunks window chunks, with chunks of at least half
// a staged tile, so that it can rotate its window keys in staging instead of
// in a separate pass.
bool fwd8_rotates_in_staging(int Tq, int Tk, int L, const SplitPlan& sp);
hipError_t launch_fwd_fp8(FwdParams p, const RopeStage& rs, hipStream_t stream);
hipError_t launch_rope_load_fp8(const uint8_t* k_slots, uint8_t* k_win, long long slot_bytes, int S, int first_slot,
                                int n_window, long long rows_per_slot, int dim_offset, int n_pairs,
                                const RopeLoadArgs& args, hipStream_t stream);
hipError_t launch_kv_copy(const uint16_t* k_src, const uint16_t* v_src, uint16_t* k_dst,
                          uint16_t* v_dst, long long n_elems, hipStream_t stream);
// Gather of a strided [B, H, L, D] K/V chunk into a contiguous slot.
hipError_t launch_kv_gather(const uint16_t* k_src, const uint16_t* v_src, Strides sk, Strides sv, uint16_t* k_dst,
                            uint16_t* v_dst, int B, int H, int L, int D, hipStream_t stream);

// Record the calling thread's status message (what mw_last_error returns)
// and return `code`; MW_OK clears it.
int set_error(int code, const char* msg);

}  // namespace mw
