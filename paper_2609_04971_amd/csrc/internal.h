// Internal interface between the C ABI (abi.hip) and the kernel files.
// Not installed; the public contract is include/bkv.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "bkv.h"

namespace bkv {

// ---- workspace --------------------------------------------------------------
// Control block (zeroed by init except the stamp; the score words are also
// reset by every score launch before it starts, the compaction words are
// left zero by every compaction), then data.
// The control block's size and offsets depend only on P = B*Hkv and budget,
// so one initialised workspace stays valid while N, W or C change.
constexpr uint32_t kWsMagic = 0x424b5631u;  // "BKV1"

enum HdrWord : int {
    kHdrMagic = 0,
    kHdrP = 1,
    kHdrBudget = 2,
    kHdrErr = 3,     // sticky device error bits, cleared only by init
    kHdrWords = 64   // header is 256 bytes
};

// One 128-byte control line per (batch, kv-head), so that work items of
// different heads never contend for one address.
enum HeadWord : int {
    kHcScTicket = 0,  // score: work ticket within the head
    kHcP1Count = 2,   // score: statistics items of the head finished
    kHcReady = 3,     // score: the head's row normalisers are published
    kHcCpTicket = 4,  // compaction: work ticket within the head
    kHcCpDone = 5,    // compaction: segments of the head finished
    // the fused eviction launch (score, select and compaction work items of
    // every head under the score ticket)
    kHcFcDone = 6,    // fused: compaction segments of the head finished
    kHcFDone = 7,     // fused: final-score items of the head finished
    kHcScReady = 8,   // fused: the head's scores are all stored
    kHcKept = 9,      // fused: the head's kept indices are stored
    kHcWords = 32
};

enum DevErr : int { kErrScoreWait = 1, kErrCompactWait = 2, kErrStamp = 4, kErrBadIndex = 8 };

constexpr int kSegRows = 128;  // compaction rows per work item
constexpr int kMaxFillKeep = 65536;  // hole-filling compaction: kept rows per head at most (LDS bitmap)

// Per-head row metadata written before scoring: word 0 = number of occupied
// beacon slots, words kMetaAct.. = those slots, ascending.
constexpr int kMetaAct = 16;
constexpr int kMetaWords = 128;

struct WsLayout {
    // control block
    size_t hctl;    // per-head control lines (int32 [P][kHcWords])
    size_t cflags;  // compaction: per-segment read-done flags (int32 [P][nseg])
    // selection split over several workgroups per head (0: not laid out)
    size_t tk_hist;  // int32 [P][4096] bin counts, left zero after each selection
    size_t tk_head;  // int32 [P][kTkHeadWords]
    size_t tk_cand;  // uint32 [P][512][2] threshold-bin (order key, token)
    size_t tk_cnt;   // int32 [P][kTkMaxSlices] per-slice counts
    size_t ctl_end;
    // data
    size_t part_m, part_z;  // score: per-chunk row statistics (fp32 [P][nch][R_pad_max])
    size_t lse2;            // score: row log2-normalisers (fp32 [P][R_pad_max])
    size_t rows;            // score: observation rows in MFMA operand order (bf16 [P][R_pad_max][D])
    size_t rmeta;           // score: per-head occupied-slot list (int32 [P][kMetaWords])
    size_t score_end;
    size_t scores;          // evict: scores when the caller passes none [P][N]
    size_t kept;            // evict: kept indices when the caller passes none [P][budget]
    size_t evict_end;
    int P, nseg, R_pad_max, nch, kgn, key_chunk;
    int nch_ws;  // score chunks per head whose statistics the workspace holds
    int rtg;  // score fast path: row tiles (16 rows) per row group; 0 selects the generic path
};

// The score fast path (bf16) holds the rows of one row group in registers:
// at most kFastTiles tiles per group and kFastRowGroups groups.
constexpr int kFastTiles = 9;
// The fast path's key chunks (work items).  A chunk costs about as much
// around its key loop (ticket, rows, count-in, hand-off) as 600 keys in it,
// so chunks are as long as LDS and the balance of the machine allow: as many
// as fill the compute units' two workgroups each (kScoreSlots items), and
// more only so that none is longer than the limits below.  Measured with R =
// 144 against chunks of 1024 keys (256 with fewer than 512 such chunks), us:
//   heads x keys    before  chunks a head, after
//   4608 x 4224     1882    3   1789
//   256 x 16384     430     10   376 (chunks of 2^10 keys also start all
//   128 x 32768     402     20   371  streams on the same memory channels)
//   128 x 4224      76.6    4    65.9
//   128 x 2048      62.8    4    47.6 (2 chunks: 54.8, 8: 62.8)
//   64 x 4096       59.4    8    47.1 (4: 54.3, 16: 58.8)
//   8 x 32768       66.2    64   46.7 (32: 57.0, 128: 67.1)
//   256 x 1024      62.6    2    46.6
// A layer of few tokens runs only a few rounds of items, so its last round
// counts for more than what an item costs around its loop: it takes chunks of
// at most 1152 keys (chunks a head, us, by row count; * the one taken):
//   66 x 12520, 48 rows    8  83    10  77    11* 76   13  76
//   48 x 30000, 48 rows    18 121   24  116   27* 116
//   148 x 5440, 48 rows    4  78    5*  74    6   74
//   100 x 6000, 144 rows   5  79    6*  74
//   100 x 17472, 96 rows   11 150   15  145   16* 147
//   and past that line  200 x 9000, 144 rows: 6* 174, 8 184, 9 177;
//   168 x 13617, 144 rows: 9* 215, 12 219, 14 220
// A chunk is at least 256 keys (60 x 486, 56 rows: 1 chunk 21.4, 2* 19.1,
// 4 19.5).
// Heads of several row groups take shorter chunks and more of them (192 to
// 544 rows, us by chunks a head; those taken are marked):
//   32 x 65536   47  585   52  582   57* 549   64  551
//   128 x 16384  12  509   13  493   15* 492   16  515
//   64 x 12000   9   151   10  148   11  142   12* 136   16  136
//   40 x 20000   15  146   16  139   18* 139   24  139
//   32 x 12345   13  102   14  97    18  91    20* 86    25  89
//   96 x 6000    5   165   6*  151
//   128 x 4224   3   162   4*  136   5   151
// which is chunks of at most 1152 keys, and kMultiScoreItems of them in all
// unless there are so many heads that the count a head gets would be a
// coarse one (128 x 4096: 4 chunks 127, 5 145, 6 143).
//
// The chunk's cost: these limits look at the length of a chunk, not at how
// full the last round of items is, which cost up to 13 % against 1024-key
// chunks (256 with fewer than 512 such) where a round was nearly empty, most
// of all in the mean form, whose items are longer, and in heads of few rows.
// There chunks of 1024, 896 and 768 keys are taken where rounds times length
// is less,
//     max(2 P nch / kScoreSlots + kChunkTail, kChunkRounds) (keys + kChunkFixed),
// fitted over 2500 measured shapes.  In the max form several row groups keep
// the limits above (5 of 900 shapes lose more than 1 % by them), and one group
// of more than kFewTiles tiles takes 1024 keys only, and only 2 % below.
// us, chunk by the limits -> by the cost (beside 1024 or 256 keys):
//   92 x 5282, 176 rows, mean   1152 120 -> 768 89 (113)
//   280 x 4148, 520 rows, mean  1152 438 -> 896 393 (405)
//   94 x 5248, 144 rows, mean   1152 85 -> 768 77 (83)
//   152 x 3413, 72 rows, mean   1152 51.6 -> 896 46.0 (45.6)
//   58 x 7522, 8 rows           1024 36.1 -> 768 31.3 (32.8)
//   12 x 46437, 48 rows         1152 58.6 -> 896 52.2 (56.3)
// The losses are smaller: 28 x 29678, 656 rows, mean 505 -> 527 (544).
// Over 900 other shapes 32 are more than 1 % behind 1024 or 256 keys, 5 more
// than 4 % (19 and 47 of 500, counted alike, before); 15 % ahead on average.
constexpr float kChunkTail = 0.25f, kChunkRounds = 2.5f, kChunkMargin = 0.98f;
constexpr int kChunkFixed = 150, kFewTiles = 5;
constexpr int kOneGroupKeyChunk = 1664;
constexpr int kFewKeyChunk = 1152;    // one row group, fewer than kFewTokens tokens in all
constexpr long long kFewTokens = 1750000;
constexpr int kShortKeyChunk = 256;
constexpr int kMultiKeyChunk = 1152;  // several row groups
constexpr int kKeyChunkUnit = 128;    // four waves of 32-key groups
constexpr int kScoreSlots = 512;
constexpr int kMultiScoreItems = 768;
constexpr int kMultiHeads = 64;

// Split selection: words per head, slices per head at most, heads at most
// for which the regions are laid out, and the shortest head it takes.
constexpr int kTkHeadWords = 4;
constexpr int kTkMaxSlices = 64;
constexpr int kTkMaxHeads = 64;
constexpr int kTkMinN = 8192;
constexpr int kFastRowGroups = 8;

// flags (BKV_SCORE_*) choose the score's key chunks only; every offset and
// size is the same for all of them.
WsLayout ws_layout(const bkv_dims& d, int flags = 0);

// ---- the whole eviction (bkv_evict_ex), split so that a caller can check the
// arguments before it enqueues anything of its own -----------------------------
bkv_status evict_check(const bkv_dims* d, int32_t flags, const void* K, const void* V, const void* q_win,
                       const float* beacons, const int32_t* counts, const float* rope_cos, const float* rope_sin,
                       float scale);
// Arguments already checked, N > 0 and B > 0, ws holds ws_layout(d).evict_end bytes.
bkv_status evict_enqueue(const bkv_dims* d, int32_t flags, void* K, void* V, const void* q_win, const float* beacons,
                         const int32_t* counts, const float* rope_cos, const float* rope_sin, float scale,
                         int32_t* kept, float* scores, float* row_lse, void* ws, hipStream_t stream);

// ---- launches (enqueue only; arguments already validated) --------------------

hipError_t launch_beacon_update(const bkv_dims& d, const void* q_new, int T, float* beacons,
                                int32_t* counts, int32_t* assign, hipStream_t s);

hipError_t launch_score(const bkv_dims& d, const WsLayout& L, int flags, const void* K, const void* q_win,
                        const float* beacons, const int32_t* counts, const float* rope_cos,
                        const float* rope_sin, float scale, float* scores, float* row_lse,
                        void* ws, hipStream_t s);

// The whole eviction in one launch (score, select and compact work items
// under one per-head ticket); only where evict_fusable (the bf16 fast path,
// large layers of 16K to 32K tokens, where it measured faster than the
// chained launches).  kept and scores are required (the workspace's own may
// be passed).
bool evict_fusable(const bkv_dims& d, const WsLayout& L);
hipError_t launch_evict_fused(const bkv_dims& d, const WsLayout& L, int flags, void* K, void* V, const void* q_win,
                              const float* beacons, const int32_t* counts, const float* rope_cos,
                              const float* rope_sin, float scale, float* scores, float* row_lse, int32_t* kept,
                              void* ws, hipStream_t s);

// Selection; with a workspace holding the split-selection regions (ws
// non-null, L.tk_hist set) a layer of few heads is split over several
// workgroups per head.
hipError_t launch_topk(const bkv_dims& d, const WsLayout& L, const float* scores, int32_t* kept, void* ws,
                       hipStream_t s);
hipError_t launch_compact_fill(const bkv_dims& d, void* K, void* V, const int32_t* kept, int32_t* src_of, void* ws,
                               hipStream_t s);

hipError_t launch_compact(const bkv_dims& d, const WsLayout& L, void* K, void* V,
                          const int32_t* kept, void* ws, hipStream_t s);

// FPS over H heads of src [H][src_rows][D], k = min(m, n) picks per head;
// dst (optional) receives the picked rows, counts (optional) the occupancy.
hipError_t launch_fps(int H, int n, int kmax, int D, int dtype, const void* src, int src_rows, int32_t* picks,
                      void* dst, int dst_dtype, int dst_rows, int32_t* counts, hipStream_t s);

}  // namespace bkv
