// Host plan and device descriptors of one apack_prune_layer call.
#pragma once

#include <cstdint>
#include <vector>

#include "common.hpp"

namespace apack {

#ifndef APACK_KEY_TILE
#define APACK_KEY_TILE 128
#endif
#ifndef APACK_ROW_BLOCKS
#define APACK_ROW_BLOCKS 2
#endif
#ifndef APACK_TILE_TARGET
#define APACK_TILE_TARGET 256
#endif
constexpr int kKeyTile = APACK_KEY_TILE;       // keys per LDS stage of the score kernels
constexpr int kKeyBlock = 32;                  // keys per MFMA block
constexpr int kRB = APACK_ROW_BLOCKS;          // 32-row query blocks held by one wave
constexpr int kRowsPerWave = 32 * kRB;
constexpr int kMaxWaves = 8;                   // waves per score workgroup
constexpr int kSmallRows = 16384;              // rows of a sequence that one workgroup selects from
#ifndef APACK_MAX_CHUNK
#define APACK_MAX_CHUNK 4096
#endif
constexpr int kMaxChunk = APACK_MAX_CHUNK;    // keys per score workgroup, at most
// A call whose sequences all have at most kFewRows query rows per key head
// (the last query token of a grouped head, say) and kFewTotal over the heads
// stores its logits in pass 1 rather than reading K again in pass 2.
constexpr int kFewRows = 16;
constexpr int kFewTotal = 1024;
constexpr int kFewTarget = 512;   // workgroups that the few-row pass 1 aims at: two per CU
constexpr int kRowTile = 1024;   // rows per workgroup of the select and compaction kernels

// Per-sequence descriptor on the device (uploaded once per call).  The
// select kernel fills thr / need / all_eq for modalities it ranks.
struct SeqDev {
  int64_t tok_off;      // first packed row of the sequence in K / scores
  int64_t n_tokens;
  int64_t q_off;        // first packed query row
  int64_t out_off;      // first slot in kept_rows
  int64_t n_kept;       // kept rows of the sequence (bound on the scan's writes)
  int64_t tag_off;      // first byte of the sequence in the tag array
  int64_t stats_off;    // first (max, sum) partial: [g][chunk][rows_pad]
  int64_t colpart_off;  // first per-group column partial: [g*n_rg + rg][n_tokens]; of a few-row
                        // call the first stored logit: [g][row][n_tokens rounded up to 16]
  int32_t q_len;
  int32_t n_rg;         // query-row groups per KV head
  int32_t rows_per_rg;  // rows per group (multiple of 64)
  int32_t rows_pad;     // n_rg * rows_per_rg
  int32_t chunk;        // keys per score workgroup (whole tiles; in fp32 whole blocks)
  int32_t n_chunks;
  int32_t n_cand;
  int32_t k_sel[2];     // keep count per modality (audio, visual)
  int32_t n_mod[2];     // candidate count per modality
  int32_t select[2];    // 1 when a radix select is needed (0 < k < n)
  uint32_t thr[2];      // threshold bits: rows above are kept
  int32_t need[2];      // rows equal to thr kept, lowest rows first
  int32_t all_eq[2];    // every row equal to thr is kept
  uint32_t prefix[2];   // radix digits chosen so far
  uint32_t kk[2];       // rank of the k-th value inside the chosen bucket
  uint32_t done_cnt;    // row tiles finished in the current select pass
  int32_t n_ftiles;     // row tiles of the sequence
  int32_t ctr_off;      // arrival counters: [n_chunks key chunks][1 sequence]
};

// A run of rows [begin, end) of one tag (see apack_prune_layer's tags).
struct SpanDev {
  int32_t begin, end, tag;
};

// The descriptors of a call with one sequence of at most kInlineSpans spans,
// passed to the first score kernel by value: it needs no upload and no loads
// of descriptors, and writes what the later kernels read (the sequence, its
// tiles, tags and zeroed counters) into the workspace itself.  The upload
// kernel, its pinned block and two dependent loads had cost 3-5 us of a call
// (9454-row layers 61.3 -> 58.1 and 69.5 -> 66.9 us, the 1312-row fp32 layer
// 53.6 -> 49.8).  Longer span lists (each key tests every span) and batches
// are uploaded; n_spans is then -1.
constexpr int kInlineSpans = 16;
struct InlineCall {
  SeqDev seq;
  int32_t n_spans;
  int32_t n_ctr;        // arrival counters to clear
  SpanDev spans[kInlineSpans];
};

struct FTileDev {
  int32_t seq, idx;     // sequence and row tile within it (rows idx*kRowTile ...)
};

struct TileDev {
  int32_t seq, g, rg, chunk;
};

// How the score passes cut a call; the forms' results agree to fp32 rounding.
//   kGeneral    chunks of 128-key tiles.  Every call can take it, and its
//               workspace is the smallest.
//   kFineChunks chunks of 32-key blocks (fp32), with more partials per row.
//   kFewRows    the few-row kernels (bf16), with room for the logits.
// A call takes the form of its dtype and rows if the workspace holds it, and
// kGeneral otherwise, so that a workspace sized for a wider call serves it.
enum class ScoreForm { kGeneral, kFineChunks, kFewRows };

struct PrunePlan {
  std::vector<SeqDev> seqs;
  std::vector<TileDev> tiles;
  std::vector<FTileDev> ftiles;
  std::vector<int64_t> n_kept;
  int64_t total_tok = 0;    // sum of n_tokens (tag bytes)
  int64_t max_tokens = 0;   // longest sequence
  int64_t total_stats = 0;  // (max, sum) partials
  int64_t total_colpart = 0;  // column partials, or the logits of a few-row call
  int64_t total_kept = 0;
  int64_t total_ctr = 0;    // arrival counters (zeroed by the upload)
  int64_t weighted = 0;     // keys times row groups over the call, the score passes' work
  int waves = 1;
  bool any_select = false;
  int max_planes = 0;       // most per-group partials of a key (general score kernels)
  bool few_rows = false;    // every sequence has at most kFewRows query rows per key head
  ScoreForm form = ScoreForm::kGeneral;
  // Workspace layout (byte offsets).
  size_t off_seqs = 0, off_tiles = 0, off_ftiles = 0, off_tags = 0, off_ctr = 0, blob_bytes = 0;
  size_t off_stats = 0, off_colpart = 0, off_hist = 0, off_cnt = 0, ws_bytes = 0;
};

// What the scores' last steps -- the sum over a key's per-group partials, the
// count of the first radix digit -- are left to.  The score kernels do them in
// their last workgroups to arrive: two round trips of atomics over the XCDs
// (7 us of a 9390-row layer's 25).  Where one workgroup selects anyway it
// counts the digit itself: calls at 1312 fp32 rows 41.2 us against 46.1, at
// 9390 bf16 rows 66.0 against 66.9, with few query rows 42.9 against 45.1, at
// 15564 rows 86.4 against 85.8 -- up to kDigitRows, or with few query rows.
// It sums too where there are one or two partials per key and few of them: it
// takes them one after another, a round trip to memory each, where the score
// kernels read eight together in many workgroups.  64 query rows, bf16, head
// dim 128, us with the sums in the score kernels and in the selection: one
// partial, 1312 keys 32.4 and 31.1, 9000 44.5 and 43.9, 15000 52.8 and 53.1;
// two, 1312 keys 33.0 and 32.1, 5400 39.2 and 39.2 (fp32 74.7 and 75.7);
// three, 1312 and 5400 keys 26.7 and 26.7, 33.0 and 33.8; four, 1312 keys 32.0
// and 32.1; eight, 2048 keys 28.4 and 30.3; 32, 512 keys 27.4 and 36.9; 64,
// 256 keys 30.7 and 50.8.
enum ScoreTail { kTailInScores = 0, kDigitInSelect = 1, kSumInSelect = 2 };
constexpr int64_t kSumPlanes = 2, kSumPartials = 8192, kDigitRows = 12288;
inline ScoreTail score_tail(const PrunePlan& pl) {
  const bool few = pl.form == ScoreForm::kFewRows;   // its kernels store whole scores
  if (pl.max_tokens > (few ? kSmallRows : kDigitRows)) return kTailInScores;
  return !few && pl.max_planes <= kSumPlanes && pl.max_planes * pl.max_tokens <= kSumPartials ? kSumInSelect
                                                                                             : kDigitInSelect;
}

struct DevPtrs {
  SeqDev* seqs;
  TileDev* tiles;
  uint8_t* tags;
  FTileDev* ftiles;
  float2* stats;
  float* colpart;
  uint32_t* hist;       // [n_seq][2][2048] radix histograms
  uint32_t* cnt;        // [n_ftiles][3] per-tile keep counts
  uint32_t* ctr;        // arrival counters of the score kernels
};

// Validates the call and fills what no form changes.
apack_status build_prune_plan(int32_t n_seq, const apack_seq* seqs, int32_t hq, int32_t hkv, int32_t d,
                              PrunePlan& plan);
// Chunks, tiles and workspace layout of the plan in one form.
void lay_out_prune(PrunePlan& plan, ScoreForm form, int n_rep, int hkv);

int64_t select_hist_words(int64_t n_seq);   // radix histogram words of n_seq sequences

apack_status launch_select(const PrunePlan& pl, const DevPtrs& dp, int n_rep, int hkv, float* scores, int32_t* kept,
                           hipStream_t stream);

apack_status launch_prune(const PrunePlan& pl, const DevPtrs& dp, const InlineCall& in, apack_dtype dt, int d, int hq, int hkv,
                          const void* q, int64_t q_hs, const void* k, int64_t k_hs, float* scores,
                          int32_t* kept, hipStream_t stream);

}  // namespace apack
