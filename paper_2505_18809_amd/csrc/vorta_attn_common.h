// Work decomposition shared by the attention kernels.
//
// A launch covers some or all heads of the layer.  Its grid is up to four consecutive segments
// of work items, in the order that has the long ones first in a large layer, so that short ones fill the tail of the launch:
//   [ route 1: (slot, q-block over the text rows)         | keys: rows [0, N)                      ]
//   [ route 0: (head, q-block) over all N rows            | keys: rows [0, N) of the head          ]
//   [ route 2: (slot, q-block) over L_c + n_text rows     | keys: all rows of the core-set         ]
//   [ route 1: bf16 (slot, item of a list)                | keys: a box of tokens, then the text   ]
//   [          fp32 (slot, tile, q-block inside the tile) | keys: the tile's run list              ]
// (Not in every layer: with a window that covers most of the grid the window items are longer than the
// core-set items.)  A work item is up to BM query rows.  The text rows of a window head attend to every row, so their items
// cost as much as those of a full-attention head and sit with them at the front.
#pragma once

#include <cstdint>

#include "vorta_internal.h"

namespace vorta {

struct AttnArgs {
  // route 0: caller's tensors
  const void *q0, *k0, *v0;
  void* o0;
  long head_stride0, row_stride0;   // elements
  // route 2: [n_lr][Nc][d]
  const void *qc, *kc, *vc;
  void* oc;
  // Core-set index, or null: with it the rows of route 2 go to the caller's output instead of oc, every slot's row
  // to the tokens that read it (unpool).
  const int *keep_idx, *assign;     // [n_lr][Lc], [n_lr][L]
  const int2* slot_bucket;          // [Lc]: centre token and extents of the slot's bucket
  int Lc, grid_H, grid_W, bucket_max;      // bucket_max: tokens of an unclipped bucket
  // route 1: [n_win][N][d] in tile order
  const void *qt, *kt, *vt;
  void* ot;
  // route 1 without tile-ordered copies (qt == null, win_gather): rows of the caller's tensors are gathered
  // through tok_of (tile-order index -> token index; fp32); win_heads = head id of each window slot.
  // row_of is the inverse.
  const int *tok_of, *row_of;       // [N]
  const int* tile_row0;             // [n_tiles + 1]: first tile-order row of each tile (edge tiles may be clipped)
  int win_gather;
  const int* runs;                  // [n_tiles][max_runs][2]
  const int* n_runs;                // [n_tiles]
  int max_runs;
  int N, Nc, L, n_text;
  int n_tiles, tile_tokens;
  // Route 1, bf16: window tiles whose key sets are identical (under the clamped centre rule the first
  // floor(w/2) + 1 tiles of every axis end, under the block rule all tiles of a block) are computed
  // together, their rows cut into blocks across tile borders -- one key stream serves them all.
  // win_items: WIN_ITEM_INTS numbers for each of the win_count items of every window head; row r of an item
  // lies at win_row[first + r] (token, or tile-order row of the copies).  Null (fp32): one item per
  // (tile, q-block), by arithmetic.
  const int* win_items;
  const int* win_row;               // [L]
  int win_count;
  // The last work items of a launch leave most CUs idle while a few finish them.  Items with
  // index >= split_from are therefore issued as two items of BM / 2 rows each (grid index
  // split_from + 2 j + h -> rows [h BM / 2, (h + 1) BM / 2) of item split_from + j); a workgroup
  // whose upper wavefronts have no rows runs them as helpers (staging only), which takes about
  // half the time of a full item.  split_from = INT_MAX: no split.
  int split_from;
  // Split kernel: of the first `round` workgroups the first ones take the last items of that round (see launch_split).
  int round, round_shift;
  int qb_dense, qb_core, qb_tile, qb_text;   // q-blocks per head / core-set / tile / text part
  int end_text, end_dense, end_core, end_tile;   // cumulative item counts, in grid order; end_tile = all
  float scale;
  HeadIds dense_heads, win_heads, core_heads;
  // [key lists][WIN_KEY_INTS], bf16: never null.  Last: ahead of the numbers above it costs the fp32 kernels' first reads 0.2 us.
  const int* win_keys;
};

// Eq. 5 epilogue of a dense launch over all heads: the rows it writes are
//   a1 (its own result) + a2 (the sliding-tile result, already in `out`) + a3 (core-set result of
//   the slot the row is assigned to),
// the first still in registers / LDS, the other two read as bf16 rows.  Text rows see every key
// under the sliding-tile branch too, so for them the second term equals the first.
struct MixArgs {
  const void* oc;              // [heads][Nc][d]: core-set outputs of every head
  const int* assign;           // [heads][L]
  int Lc;
  float alpha[VORTA_MAX_HEADS][3];
};
struct NoMix {};

// Tables that are the same for every lane and that no kernel writes are read as constant memory: with a wave-uniform index that
// is a scalar load, whose result lands in a scalar register and whose wait does not include the vector loads in flight.
typedef const __attribute__((address_space(4))) int* const_int_ptr;

struct WorkItem {
  long q_off, kv_off, o_off;   // element offsets of the head's row 0 in q / k,v / o
  long row_stride;             // elements
  int head;                    // head id (dense segment), head slot (core-set segment)
  int seg;                     // 0 dense, 1 core-set, 2 window
  int row0, n_rows;            // query rows row0 .. row0 + n_rows - 1; listed: places of win_row instead of rows
  bool listed;
  const int* keys;             // what its keys are computed from (WindowKeys); not listed: some entry, not used (read without a branch)
  int n_runs;
  const int* runs;             // null: the single run {0, single_len}
  int single_len;
};

// The arguments that finding an item and its rows takes, read all at once.  Read where they are used they are some fifteen
// scalar loads, each waited for before the branch that needs it, all ahead of an item's first row.  13 layers, 11 of them small: 1.7 %
// (3 window heads of 3,072 tokens 15.3 -> 14.4 us, 4 dense ones of 1,024 13.4 -> 13.1), and head ids in words (HeadIds) another 0.5 %; two fp32
// heads of 256 tokens 16.9 -> 16.7; large layers are level, but where a few text rows of long streams beside thousands of short window
// items set the end: those start sooner and press harder on the memory that the streams wait for (16 window heads of 35,712 tokens with
// 20 text rows 605 -> 621 us).  The fp32 kernels read five arguments here that they have no use for: without those, and with
// six that they do use in their place, 21 layers of 128 to 3,072 tokens are level.  (An operand of the statement is a register that
// holds the argument there; it emits nothing.)
__device__ __forceinline__ void read_together(const AttnArgs& a) {
  asm volatile("" ::"s"(a.head_stride0), "s"(a.row_stride0), "s"(a.q0), "s"(a.k0), "s"(a.v0), "s"(a.qc), "s"(a.kc), "s"(a.vc), "s"(a.N),
               "s"(a.Nc), "s"(a.L), "s"(a.n_text), "s"(a.win_gather), "s"(a.win_items), "s"(a.win_row), "s"(a.win_count),
               "s"(a.win_keys), "s"(a.split_from), "s"(a.qb_dense), "s"(a.qb_core), "s"(a.qb_text), "s"(a.end_text), "s"(a.end_dense),
               "s"(a.end_core), "s"(a.scale), "s"(a.round), "s"(a.round_shift), "s"(a.o0));
}

template <int BM, int D>
__device__ __forceinline__ WorkItem decode_item(const AttnArgs& a, int item) {
  WorkItem w;
  w.runs = nullptr;
  w.n_runs = 1;
  w.head = 0;
  w.listed = false;
  w.keys = a.win_keys;
  int half = -1;
  if (item >= a.split_from) {
    half = (item - a.split_from) & 1;
    item = a.split_from + ((item - a.split_from) >> 1);
  }
  if (item < a.end_text) {
    const int slot = item / a.qb_text, qb = item - slot * a.qb_text;
    w.seg = a.win_gather ? 0 : 2;   // gathered: rows of the caller's tensors, like a dense head
    w.q_off = w.kv_off = w.o_off = a.win_gather ? a.win_heads[slot] * a.head_stride0 : (long)slot * a.N * D;
    w.row_stride = a.win_gather ? a.row_stride0 : D;
    w.row0 = a.L + qb * BM;
    w.n_rows = min(BM, a.n_text - qb * BM);
    w.single_len = a.N;
  } else if (item < a.end_dense) {
    item -= a.end_text;
    const int slot = item / a.qb_dense, qb = item - slot * a.qb_dense;
    w.seg = 0;
    w.head = a.dense_heads[slot];
    w.q_off = w.kv_off = w.o_off = a.dense_heads[slot] * a.head_stride0;
    w.row_stride = a.row_stride0;
    w.row0 = qb * BM;
    w.n_rows = min(BM, a.N - w.row0);
    w.single_len = a.N;
  } else if (item < a.end_core) {
    item -= a.end_dense;
    const int slot = item / a.qb_core, qb = item - slot * a.qb_core;
    w.seg = 1;
    w.head = slot;
    w.q_off = w.kv_off = w.o_off = (long)slot * a.Nc * D;
    w.row_stride = D;
    w.row0 = qb * BM;
    w.n_rows = min(BM, a.Nc - w.row0);
    w.single_len = a.Nc;
  } else if (a.win_items) {
    item -= a.end_core;
    const int slot = item / a.win_count, i = item - slot * a.win_count;
    const const_int_ptr it = (const_int_ptr)(uintptr_t)(a.win_items + WIN_ITEM_INTS * i);
    w.seg = 2;
    w.q_off = w.kv_off = w.o_off = a.win_gather ? a.win_heads[slot] * a.head_stride0 : (long)slot * a.N * D;
    w.row_stride = a.win_gather ? a.row_stride0 : D;
    w.row0 = it[0];
    w.n_rows = it[1];
    w.listed = true;
    w.keys = a.win_keys + (long)WIN_KEY_INTS * it[2];
    w.n_runs = 0;
    w.single_len = 0;
  } else {
    item -= a.end_core;
    const int per_head = a.n_tiles * a.qb_tile;
    const int slot = item / per_head, r = item - slot * per_head;
    const int tile = r / a.qb_tile, qb = r - tile * a.qb_tile;
    w.seg = 2;
    w.q_off = w.kv_off = w.o_off = a.win_gather ? a.win_heads[slot] * a.head_stride0 : (long)slot * a.N * D;
    w.row_stride = a.win_gather ? a.row_stride0 : D;
    const int first = a.tile_row0[tile];
    w.row0 = first + qb * BM;
    w.n_rows = min(BM, a.tile_row0[tile + 1] - first - qb * BM);   // <= 0 for a clipped tile with fewer q-blocks
    w.runs = a.runs + (long)tile * a.max_runs * 2;
    w.n_runs = a.n_runs[tile];
    w.single_len = 0;
  }
  if (half >= 0) {          // n_rows may come out <= 0 here too: the workgroup then has nothing to do
    w.row0 += half * (BM / 2);
    w.n_rows = min(BM / 2, w.n_rows - half * (BM / 2));
  }
  return w;
}

// Work item of a workgroup.  Consecutive workgroup ids are dealt round-robin to the 8 XCDs
// (each with its own L2); with chunked = true the ids are re-dealt so that every XCD gets one
// contiguous range of the n items instead -- neighbouring window tiles, whose key sets
// overlap, then run on the same XCD at about the same time and share its L2.  For launches whose
// items cost about the same: a contiguous deal of unequal items leaves some XCDs with all the long ones.  The half-row
// items at the end of a window launch are unequal, and all of them fall to the last XCDs; the launch rule counts with that.
__device__ __forceinline__ int xcd_item(int block, int n, bool chunked) {
  if (!chunked) return block;
  const int xcd = block & 7, loc = block >> 3, q = n >> 3, r = n & 7;
  return xcd * q + min(xcd, r) + loc;
}

// Run list of a work item, read as constant memory.
struct RunList {
  const_int_ptr runs;      // (start, length) pairs; null: the single run {0, single_len}
  int n_runs, single_len;
  __device__ __forceinline__ explicit RunList(const WorkItem& w)
      : runs((const_int_ptr)(uintptr_t)w.runs), n_runs(w.n_runs), single_len(w.single_len) {}
  __device__ __forceinline__ int start(int r) const { return runs ? runs[2 * r] : 0; }
  __device__ __forceinline__ int len(int r) const { return runs ? runs[2 * r + 1] : single_len; }
};

// Keys of a window item: the video tokens of a box of the grid, in raster order, then the text tokens.  The token of
// a key is computed: a dozen vector instructions a lane and block, two of them products of 32 bits, in place of a walk
// through the tile's runs.  Scalar instructions and branches of a wavefront and block with the walk and without: 54 and 23
// on the 4-wavefront instance, 66 and 26 on the other; all instructions per matrix instruction 11.8 and 10.0, 9.6 and 8.3
// (counters, 720p layer).  The numbers are the same for every lane and no kernel
// writes them: constant memory, like the run lists.  They are kept once for a sequence of window rows, not in each of its
// items: that read is level (window heads of 768 to 75,600 tokens within 0.5 %), and a plan of one-token tiles has 96 instead
// of 192 bytes a tile.
struct WindowKeys {
  int n_keys, n_box, t0, step, mult_a, shift_a, skip_a, mult_b, shift_b, skip_b, text;
  __device__ __forceinline__ explicit WindowKeys(const WorkItem& w) {
    const const_int_ptr at = (const_int_ptr)(uintptr_t)w.keys;
    int* const field[] = {&n_keys, &n_box, &t0, &step, &mult_a, &shift_a, &skip_a, &mult_b, &shift_b, &skip_b, &text};
#pragma unroll
    for (int i = 0; i < 11; ++i) *field[i] = at[i];
  }
  // read once: kept in scalar registers, not read again in every iteration
  __device__ __forceinline__ void keep() {
    asm volatile("" : "+s"(n_keys), "+s"(n_box), "+s"(t0), "+s"(step), "+s"(mult_a), "+s"(shift_a), "+s"(skip_a), "+s"(mult_b),
                      "+s"(shift_b), "+s"(skip_b), "+s"(text));
  }
  // token of key k >= 0; past the end, that of the last key
  __device__ __forceinline__ unsigned token(int k) const {
    const unsigned key = (unsigned)min(k, n_keys - 1);
    const unsigned a = __umulhi(key, (unsigned)mult_a) >> shift_a, b = __umulhi(a, (unsigned)mult_b) >> shift_b;
    const unsigned video = (unsigned)t0 + mul24(key, step) + mul24(a, skip_a) + mul24(b, skip_b);
    // no branch: the difference is the sign of key - n_box spread over all bits
    const unsigned in_box = (unsigned)((int)(key - (unsigned)n_box) >> 31), other = key + (unsigned)text;
    return other ^ ((other ^ video) & in_box);
  }
  static __device__ __forceinline__ unsigned mul24(unsigned x, int y) { return (x & 0xffffffu) * ((unsigned)y & 0xffffffu); }
};

// Rows of the keys k[i] (i < NR, per lane, 0 <= k[i] < bn) of the bn-key block that begins pos keys into run
// r, whose first row is s and whose length is len (r, pos, s, len wave-uniform).  A block
// that reaches past the end of run r continues in the following runs: they are walked with
// uniform control flow, each lane keeping the row of the run its key falls in.  Keys past the
// end of the last run repeat its last row (they are masked out of the softmax).
template <int NR>
__device__ __forceinline__ void block_rows(const RunList& rl, int r, int pos, int s, int len, int bn, int (&k)[NR],
                                           int (&rows)[NR]) {
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    k[i] += pos;
    rows[i] = s + min(k[i], len - 1);
  }
  int end = pos + bn;
  while (end > len && r + 1 < rl.n_runs) {
    end -= len;
#pragma unroll
    for (int i = 0; i < NR; ++i) k[i] -= len;
    ++r;
    s = rl.start(r);
    len = rl.len(r);
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (k[i] >= 0) rows[i] = s + min(k[i], len - 1);
  }
}

// Work of the window heads (route 1) that a launch includes.
enum WindowPart { WIN_NONE = 0, WIN_TEXT = 1, WIN_TILES = 2, WIN_ALL = 3 };

// Fills AttnArgs for a launch over the heads of rl with BM-row work items; win_part selects
// which items of the window heads it carries.  win_list: -1 = one item per (tile, q-block);
// 0 .. 3 = the plan's lists of window items (see vorta_plan).
int fill_attn_args(vorta_plan* p, const RouteLists& rl, const vorta_attn_io* io, const CoreIndex* core, int BM,
                   int win_part, AttnArgs* a, int win_list = -1);

int launch_attention_bf16(vorta_plan* p, const RouteLists& rl, const vorta_attn_io* io, const CoreIndex* core,
                          void* stream, const MixArgs* mix = nullptr, bool win_text = true);

// Token j (< 64) of the bucket whose centre token and packed extents are given; -1 past its end.  The
// quotients are taken in fp32, which is exact for such small numbers (see the selection kernels).
__device__ __forceinline__ int slot_bucket_token(const AttnArgs& a, int2 bucket, int j) {
  const int df = bucket.y & 255, dh = (bucket.y >> 8) & 255, dw = bucket.y >> 16;
  const int x = (int)(((float)j + 0.5f) * __builtin_amdgcn_rcpf((float)(dh * dw))), r = j - x * (dh * dw);
  const int y = (int)(((float)r + 0.5f) * __builtin_amdgcn_rcpf((float)dw)), z = r - y * dw;
  return j < df * dh * dw ? bucket.x + ((x - df / 2) * a.grid_H + y - dh / 2) * a.grid_W + z - dw / 2 : -1;
}

}  // namespace vorta
