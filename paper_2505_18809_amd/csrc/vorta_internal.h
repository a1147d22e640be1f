// Internal declarations shared by the translation units of libvorta.
#pragma once

#include <cstdint>
#include <mutex>
#include <vector>

#include "vorta.h"

namespace vorta {
constexpr int WIN_ITEM_INTS = 4, WIN_KEY_INTS = 12;   // of an entry of vorta_plan::win_list, of win_keys
}

struct vorta_plan {
  vorta_layer_desc d;
  int64_t L = 0, N = 0;          // video tokens, all tokens
  int nt[3] = {0, 0, 0};         // tile grid
  int n_tiles = 0, tile_tokens = 0;
  int nb[3] = {0, 0, 0};         // bucket grid (ceil)
  int n_buckets = 0;
  int64_t Lc = 0;                // core-set slots
  int max_runs = 0;
  int win_most_keys = 0;         // keys of the query tile that has most, text keys included
  int window_key_tiles = 0;
  int elem_bytes = 0;
  float scale = 0.f;
  // first row of every tile in tile order, [n_tiles + 1]: a tile that the grid clips (the tile
  // does not divide the axis) holds fewer rows than tile_tokens
  std::vector<int32_t> tile_row0;
  std::vector<int32_t> boxes;    // [n_tiles][6]
  std::vector<int32_t> runs;     // [n_tiles][max_runs][2]
  std::vector<int32_t> n_runs;   // [n_tiles]
  std::vector<int32_t> slot_base;  // [n_buckets + 1]
  // window work items of the bf16 kernels: the rows of all tiles with one key set are one sequence, cut into
  // blocks whatever the tile borders; win_tiles holds the tiles of these sequences one after the other.
  // An item is WIN_ITEM_INTS numbers: {first, n_rows, k, 0}, n_rows places of the sequences' rows from `first`, whose keys the
  // kernels compute from entry k of win_keys, one for each sequence:
  //   n_keys, n_box (the video tokens among them), t0, s, mult_a, shift_a, s_a - a s, mult_b, shift_b, s_b - b s_a, L - n_box, 0
  // List 0: blocks of 129 to 256 rows; list 1: what is left of a sequence, at most 128 rows; list 2: the
  // sequences cut into blocks of at most 64 rows instead; list 3: of at most 128 rows.
  std::vector<int32_t> win_tiles;  // [n_tiles]
  std::vector<int32_t> win_list[4], win_keys;      // bf16 plans only, like the next ones
  // of the items of a list, for the launch estimate: 64-key blocks of the items before each one ([n + 1]), blocks of
  // the longest, and 32-row wavefronts that have rows, on average
  std::vector<int64_t> win_sums[4];
  int win_most_blocks[4] = {0, 0, 0, 0};
  double win_waves[4] = {0, 0, 0, 0};
  // rotary embedding: (cos, sin) of position * rate for every position of every axis,
  // [F][pairs_F] then [H][pairs_H] then [W][pairs_W]; empty without rope_dims
  bool rope = false;
  std::vector<float> rope_cs;

  int force_form = 0, force_halves = -1;   // tests only, see vorta_test_force_form

  // device tables, all in one allocation, uploaded on first device use: copies of the tables above and those that
  // have one entry per token and are made for the upload only.  Run lists for fp32 plans, window items for bf16 ones.
  std::mutex mu;
  bool on_device = false;
  int device = -1;
  int n_cus = 256;               // compute units of that device
  int32_t* d_runs = nullptr;
  int32_t* d_n_runs = nullptr;
  int32_t* d_slot_base = nullptr;
  // [Lc][2]: the bucket of every core-set slot, as its centre token and its clipped extents (df | dh << 8 | dw << 16);
  // which slots a bucket owns depends on its size only, so this is known before any selection
  int32_t* d_slot_bucket = nullptr;
  int32_t* d_tok_of = nullptr;   // [N]: tile-order row -> token (identity for the text rows)
  int32_t* d_row_of = nullptr;   // [N]: token -> tile-order row, the inverse
  int32_t* d_win_rows = nullptr; // [L]: the tile-order rows of the sequences of win_tiles
  int32_t* d_win_tok = nullptr;  // [L]: their tokens
  int32_t* d_tile_row0 = nullptr;   // [n_tiles + 1]
  float* d_rope_cs = nullptr;
  int32_t* d_win_list[4] = {nullptr, nullptr, nullptr, nullptr};
  int32_t* d_win_keys = nullptr;
  void* d_tables = nullptr;      // the allocation
};

namespace vorta {

// Head ids as kernels take them: four to a word.  A byte at a computed index is a vector load from the arguments, ahead of every
// address that depends on it; a word is a scalar one.  Cleared from the start: set() reads the word that it puts an id into.
struct HeadIds {
  uint32_t word[VORTA_MAX_HEADS / 4] = {};
  constexpr int operator[](int i) const { return (int)(word[i >> 2] >> (8 * (i & 3)) & 255u); }
  constexpr void set(int i, int id) {
    const uint32_t at = 8u * (uint32_t)(i & 3);
    word[i >> 2] = (word[i >> 2] & ~(255u << at)) | (uint32_t)id << at;
  }
};

int fail(int code, const char* fmt, ...);        // records the thread-local message, returns code
void clear_error();

struct RouteLists {
  int count[3] = {0, 0, 0};
  int heads[3][VORTA_MAX_HEADS];                 // head ids per route, ascending
};
int split_routes(const vorta_plan* p, const uint8_t* routes, RouteLists* out);

int ensure_device_tables(vorta_plan* p);         // vorta_passes.hip
// set by the device side when it is linked in: frees the device tables of a plan
extern void (*g_release_device_tables)(vorta_plan* p);

// Launchers (each returns VORTA_OK / VORTA_EHIP).  Pointers are device memory.
struct UserTensor {                               // a tensor in the caller's layout
  const void* base;
  int64_t head_stride;                            // elements
  int64_t row_stride;                             // elements
};
UserTensor user_tensor(const vorta_plan* p, const void* base);

int launch_reorder(vorta_plan* p, const RouteLists& rl, const void* user, void* tiled, bool to_tiles,
                   void* stream);
// feat.head_stride == 0: one feature tensor shared by every head
int launch_bcs_index(vorta_plan* p, const RouteLists& rl, const UserTensor& feat, int32_t* keep_idx,
                     int32_t* assign, void* stream);
int launch_bcs_pool(vorta_plan* p, const RouteLists& rl, const void* src, const int32_t* keep_idx,
                    const int32_t* assign, bool rotate, void* dst, void* stream);
bool bcs_fused_applies(const vorta_plan* p);
// One or two (src[1] not null) tensors whose rows of the heads on routes 0 and 1 go to dst turned.
struct RopeCopies {
  const void* src[2];
  void* dst[2];
};
// copies: not null, the rotation of the heads on routes 0 and 1 rides in the same launch
int launch_bcs_select_pool(vorta_plan* p, const RouteLists& rl, const void* q, const void* k, const void* v,
                           int32_t* keep_idx, int32_t* assign, void* qc, void* kc, void* vc, const RopeCopies* copies,
                           void* stream);
int launch_rope_rows(vorta_plan* p, const RouteLists& rl, const RopeCopies& copies, void* stream);
int launch_unpool(vorta_plan* p, const RouteLists& rl, const void* o_c, const int32_t* assign, void* out,
                  void* stream);
// Core-set index of a layer call: with it the attention launch writes the rows of route 2 to the tokens that
// read them (unpool) instead of to io.o_c.
struct CoreIndex {
  const int32_t* keep_idx;   // [n_lr][L_c]
  const int32_t* assign;     // [n_lr][L]
};
// How a bf16 attention launch is cut.
constexpr int ATTN_ROWS_SPLIT = 64, ATTN_ROWS_LONG = 256;    // query rows of an item of the split and of the pipelined kernel
struct AttnForm {
  bool empty;              // no items at all
  bool split_all;          // everything on the split kernel, with `shares` key shares
  int shares;
  bool split_win;          // window rows on the split kernel (two shares), the rest on the pipelined one
  bool win_128;            // all window rows on the 4-wavefront kernel in 128-row items
  bool together;           // long and window items of more than 128 rows in one launch
  int n_long, half_long;   // 256-row items of dense, core-set and text rows; how many of them as half-row items
  int n_big, half_big;     // the same of the window items of more than 128 rows
};
AttnForm choose_attention_form(const vorta_plan* p, const RouteLists& rl, bool mix, bool win_text, int units);
int split_round_shift(const vorta_plan* p, const RouteLists& rl, bool longs, bool win_text, int units);
int launch_attention_f32(vorta_plan* p, const RouteLists& rl, const vorta_attn_io* io, const CoreIndex* core, void* stream);
int launch_router(const float* t_emb, const float* w_r, int n_steps, int d_t, int heads, float* alpha,
                  uint8_t* routes, void* stream);
int launch_blend3(vorta_plan* p, const void* o0, const void* o1, const void* o2, const float* alpha_host,
                  void* out, void* stream);

}  // namespace vorta
