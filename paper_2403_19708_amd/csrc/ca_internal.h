// Internal declarations shared by the host side of the library and its kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ca {

constexpr int kMaxSeqsPerLaunch = 64;  // per-conversation arguments travel in the kernel-argument block
constexpr int kPageSize = 16;
constexpr int kXcds = 8;               // MI355X: 8 accelerator dies, workgroup i runs on die i % 8

// ---------------------------------------------------------------------------------------
// paged pool <-> contiguous rows (Section 3.2: layer-wise load / save are data movement)
// ---------------------------------------------------------------------------------------
// One entry per conversation handled by a launch.  "contig" is [token][n_kv_heads][head_dim];
// token (contig_tok0 + i) <-> context token (ctx_tok0 + i) for i < count.
struct MoveArgs {
    uint8_t *contig_k[kMaxSeqsPerLaunch];
    uint8_t *contig_v[kMaxSeqsPerLaunch];
    int64_t contig_tok0[kMaxSeqsPerLaunch];
    int32_t ctx_tok0[kMaxSeqsPerLaunch];
    int32_t count[kMaxSeqsPerLaunch];
    int32_t seq[kMaxSeqsPerLaunch];  // row of the block table
};

// Second contiguous destination of a launch that writes what it reads twice (the new turn's K/V go into the pool AND
// to the tier in one pass): new token i of the entry also lands at row i of dst.
struct MoveArgs2 {
    uint8_t *dst_k[kMaxSeqsPerLaunch];
    uint8_t *dst_v[kMaxSeqsPerLaunch];
};

constexpr int kMoveUnroll = 2;   // 16-byte loads in flight per lane of the move kernel (one pass = kMoveUnroll*256 vectors)

struct MoveShape {
    const int32_t *block_table;  // device [n_seqs][max_pages]
    const int32_t *n_keep;       // device [n_seqs]    } where the new turn of a conversation lies on either side
    const int32_t *cu_q;         // device [n_seqs+1]  } (append launches)
    int32_t max_pages;
    int32_t n_kv_heads;
    int32_t vec_shift;           // log2 of the 16-byte vectors per head and token (3 or 4)
    int32_t heads_per_wg;        // heads one workgroup moves (grid.x slices the heads, and K/V)
    int32_t n_in_launch;
    int32_t max_pages_touched;   // largest number of pages a range of this launch touches
};

// to_pool = true: contiguous -> pages (unpack / append); false: pages -> contiguous (pack).
hipError_t launch_move(bool to_pool, const MoveArgs &args, const MoveShape &shape, uint8_t *k_pool,
                       uint8_t *v_pool, hipStream_t stream);
// the same between the pool and pinned host memory, with at most `workgroups` workgroups
hipError_t launch_link(bool to_pool, const MoveArgs &args, const MoveShape &shape, int workgroups, uint8_t *k_pool, uint8_t *v_pool,
                       hipStream_t stream);
// the new turn of conversations [0, shape.n_in_launch): rows cu_q[c].. of new_k / new_v -> context tokens n_keep[c]..
hipError_t launch_append(const MoveShape &shape, const uint8_t *new_k, const uint8_t *new_v, uint8_t *k_pool, uint8_t *v_pool,
                         hipStream_t stream);
// the same for conversations [first, first + shape.n_in_launch), and every vector is also stored to the second destination
hipError_t launch_append_save(const MoveShape &shape, int first, const MoveArgs2 &second, const uint8_t *new_k, const uint8_t *new_v,
                              uint8_t *k_pool, uint8_t *v_pool, hipStream_t stream);

// One token per conversation (decode steps), with everything the kernel would look up in the plan worked out by the host:
// where token i lies in the pool (page * kPageSize + slot), and for a save its row outside.
struct TokenSlots {
    int32_t slot[kMaxSeqsPerLaunch];
};
struct TokenRows {
    uint8_t *k[kMaxSeqsPerLaunch];
    uint8_t *v[kMaxSeqsPerLaunch];
};
// row i of new_k / new_v -> slot i of the pool, i < n
hipError_t launch_append_tokens(const TokenSlots &slots, int n, const MoveShape &shape, const uint8_t *new_k, const uint8_t *new_v,
                                uint8_t *k_pool, uint8_t *v_pool, hipStream_t stream);
// slot i of the pool -> rows.k[i], rows.v[i]
hipError_t launch_save_tokens(const TokenSlots &slots, const TokenRows &rows, int n, const MoveShape &shape, const uint8_t *k_pool,
                              const uint8_t *v_pool, hipStream_t stream);

// ---------------------------------------------------------------------------------------
// Section 3.4: per-token metadata of the rebased plan
// ---------------------------------------------------------------------------------------
struct RebaseArgs {
    const uint8_t *image;        // the plan's arrays in pinned host memory, as the GPU addresses it
    uint8_t *meta;               // where they go in device memory
    int64_t image_vecs;          // 16-byte vectors to copy
    int64_t off_table, off_n_keep, off_cu_q, off_cu_k;   // byte offsets in the image: [n_seqs][max_pages], [n_seqs], [n_seqs+1] x 2
    int32_t n_seqs;
    int32_t max_pages;
    int32_t *q_pos;              // device [sum new]
    int32_t *q_seq;              // device [sum new]
    int32_t *slot_map;           // device [sum context]
    uint32_t *arrived[2];        // merge counters of the two attention entry points: the first n_merges of each are set to zero
    int32_t n_merges;
};
hipError_t launch_rebase(const RebaseArgs &args, hipStream_t stream);

// ---------------------------------------------------------------------------------------
// Sections 2.1 / 3.1 / 3.4: attention of the new tokens over [kept history | new tokens]
// ---------------------------------------------------------------------------------------
struct WorkItem {      // one tile of stacked query rows of one (conversation, kv head)
    int32_t seq;       // -1: padding, the workgroup exits
    int32_t kv_head;
    int32_t row0;      // first stacked row; row r <-> new token r / G, query head kv_head*G + r % G
    int32_t n_rows;
    int32_t key_begin; // the item's share of the keys: [key_begin, min(key_end, what its rows see));
    int32_t key_end;   // the whole range unless the row tile was split; cuts are multiples of 64
    int32_t part;      // -1: the item writes `out`; else index of its share in the partial-result buffer
    int32_t reserved;
};

struct CombineItem {   // a row tile whose keys were split: shares first_part .. first_part + n_parts - 1
    int32_t seq, kv_head, row0, n_rows;
    int32_t first_part, n_parts;
    int32_t reserved[2];
};

// What a workgroup of launch_attn_rows needs to start streaming an item, in one piece: the item, where its conversation lies,
// its merge, and the page ids of its first pages (nothing else has to be looked up before the first loads go out).
struct RowsItem {
    int32_t seq, kv_head, n_rows, key_begin, key_end, part;
    int32_t n_keep, cu_q;                  // of the conversation
    int32_t merge, first_part, n_parts;    // shares first_part .. of the unit; `merge` numbers its counter
    int32_t reserved[5];
    int32_t page[16];                      // page ids of the 16 pages from key_begin on, as far as the item has them
};

struct AttnArgs {
    const uint16_t *q;       // bf16 bits
    uint16_t *out;
    const uint16_t *k_pool;
    const uint16_t *v_pool;
    const int32_t *block_table;
    const int32_t *n_keep;
    const int32_t *cu_q;
    const int32_t *q_pos;    // [total_q] rebased position of every new token
    const int32_t *q_seq;    // [total_q] its conversation
    const WorkItem *items;
    const CombineItem *combine;   // row tiles to merge after the walk (n_combine of them)
    float *partial;          // shares of split row tiles: per part the sums ([head_dim/4][tile_rows][4] from the tile kernels,
                             // [tile_rows][head_dim] from the others), [tile_rows] maxima, [tile_rows] denominators (fp32)
    const float2 *rope;      // [max_positions][head_dim/2] (cos, sin)
    // keys rotated once per batch and layer instead of in every row tile (launch_attn_prerot, launch_attn_pp):
    uint16_t *k_rot;             // scratch copy of the keys, dense pages [n_dense_pages][n_kv_heads][16][head_dim]
    uint16_t *v_t;               // scratch copy of the values, same pages, each block transposed (pipelined != 0 only)
    const int32_t *rot_nvalid;   // [n_dense_pages] context tokens in the page (16 except a conversation's last page)
    int32_t pipelined;            // the scratch copies have the layouts of ca_attn_pp.hip and its kernel runs
    const int32_t *dense_page0;  // [n_seqs] first dense page of a conversation
    const int32_t *rot_src_page; // [n_dense_pages] pool page a dense page is rotated from
    const int32_t *rot_pos0;     // [n_dense_pages] position of its first token
    int32_t n_dense_pages;
    int32_t max_positions;
    int32_t n_items;
    const RowsItem *rows_items;  // launch_attn_rows
    const int32_t *wg_first;     // launch_attn_rows with runs
    uint32_t *arrived;           // launch_attn_rows: shares of each merge that are there already; zero between calls
    int32_t n_wgs;
    int32_t n_combine;
    int32_t total_q;
    int32_t max_pages;
    int32_t n_q_heads, n_kv_heads, head_dim;
    int32_t rope_style;
    int32_t tile_rows;       // stacked query rows per workgroup: 128 (4 wavefronts), 256 (8), launch_attn_rows 16 or 32
    float softmax_scale;
    int32_t wgs_per_cu;      // tile kernels: workgroups that run on a compute unit at a time, as the plan was laid out for
};

constexpr int kAttnTileRowsMin = 128;   // smallest tile of stacked query rows (4 wavefronts x 32)
constexpr int kRopeMinRows = 256;       // the kernels read table rows below this whatever the window

hipError_t launch_attn_ref(const AttnArgs &args, hipStream_t stream);
hipError_t launch_attn_dma(const AttnArgs &args, hipStream_t stream);
// keys rotated once per layer into a scratch copy first
hipError_t launch_attn_prerot(const AttnArgs &args, hipStream_t stream);
// head_dim 128, 256-row tiles, keys rotated and values transposed once per layer into scratch copies; inside every
// wavefront the matrix instructions of one key tile are pipelined with the softmax of the previous one
hipError_t launch_attn_pp(const AttnArgs &args, hipStream_t stream);
// merges the shares of split row tiles (args.combine) into args.out: those of the tile kernels, and those laid out row by row
hipError_t launch_combine_tiles(const AttnArgs &args, hipStream_t stream);
hipError_t launch_attn_combine(const AttnArgs &args, hipStream_t stream);
// decode steps: every item has at most kAttnDecodeMaxRows stacked rows starting at row 0; streams K/V through
// registers instead of matrix-core tiles
constexpr int kAttnDecodeMaxRows = 2;
hipError_t launch_attn_decode(const AttnArgs &args, int max_rows, hipStream_t stream);
// few rows: every item has at most kAttnRowsMax stacked rows starting at row 0 (tile_rows 16 or 32); the context is streamed
// once through LDS rings of single wavefronts; merges its shares itself
constexpr int kAttnRowsMax = 32;
// runs: workgroup w of four wavefronts takes items [wg_first[w], wg_first[w + 1]), else, of four or eight, item w
hipError_t launch_attn_rows(const AttnArgs &args, int wavefronts, bool runs, hipStream_t stream);
constexpr int kAttnMaxParts = 1024;           // shares of split row tiles per batch (sizes the partial-result buffer)
constexpr int kAttnMaxPartsPerTile = 16;
constexpr int kAttnMinPartKeys = 256;         // a share of the tile kernels, or of a run, is at least this many keys

}  // namespace ca
