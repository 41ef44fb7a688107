// Internal: host-side layout handle shared by the layout builder and the launch code.
#pragma once
#include <cstdint>
#include <vector>

#include "../../include/s2attn.h"

namespace s2 {

// Merged tile list: groups of `group` block rows (or block columns) share one list of partner
// blocks; each entry packs (partner_index << 16) | membership_bits, bit r set when member r of
// the group keeps that partner.  This is the Merge-Q idea of section 3.2 (one large tile serves
// several fine-grained mask rows) and its mirror image for key tiles.  Row groups are
// consecutive rows.  Column groups are formed from columns with similar partner sets (a stripe
// column is attended by every later row, its neighbours only by the local window), so members
// of a column group need not be adjacent: `members` names them.  A partner index takes all of the upper
// sixteen bits (with 16-token blocks there are up to 65536 of them): read entries unsigned.
constexpr int kMaxListUnits = 1 << 15;  // blocks of a layout, or pairs of 16-token blocks

struct TileList {
  int group = 0;                 // members per tile (1..8)
  int tiles_per_head = 0;        // ceil(B / group)
  std::vector<int32_t> ptr;      // [H*tiles_per_head + 1]
  std::vector<int32_t> ent;      // packed entries; partner ascending inside a row tile,
                                 // descending inside a column tile
  std::vector<int32_t> order;    // [H*tiles_per_head]: per head, tile ids by descending length
  std::vector<int32_t> members;  // [H*tiles_per_head*group]: block index of each member, -1 = none
  // Per head and rank what a workgroup needs to begin with, so that it comes in one load: kRowRec or kColRec words a tile, (row tile) its
  // number, (column tile) nothing; where its list begins in ent; the list's length; nothing; (column tile) its members, -1 = none
  std::vector<int32_t> rec;
  int32_t* d_rec = nullptr;
  int32_t* d_ptr = nullptr;      // device copies (owned by the layout)
  int32_t* d_ent = nullptr;
  int max_len = 0;
};

// How the dK/dV launch may cut its longest key tiles into parts that different workgroups walk (their sums
// are then added by whichever of them is done last).  The lengths of a head's tiles are sorted, so a way
// of cutting is: the first n_long tiles of every head's order, tile k into as many parts as keep it within
// `steps` steps for the head where it is longest.
struct SplitLevel {
  int steps = 0;    // 64-row steps a part has at most
  int n_long = 0;   // tiles that are cut
  int n_items = 0;  // parts they are cut into, over one head
  int offset = 0;   // first of the level's n_items codes: tile | part << 16 | parts << 24, longest tile first
};

}  // namespace s2

struct s2_layout {
  s2_layout_params p{};
  std::vector<int32_t> row_ptr, col_idx, col_ptr, row_idx;
  int64_t nnz = 0;
  int max_row_blocks = 0;
  int covers_all = 0;
  bool on_device = false;
  int device = -1;
  int32_t* d_row_ptr = nullptr;  // device copies of the compressed rows (decode reads one row of them)
  int32_t* d_col_idx = nullptr;
  s2::TileList q_tiles;   // row groups  -> kept KV blocks   (forward, dQ pass)
  s2::TileList kv_tiles;  // column groups -> attending Q blocks (dK/dV pass)
  // Of the key tiles the kernels walk: the ways to cut them, and what choosing one takes
  std::vector<s2::SplitLevel> kv_levels;
  std::vector<int32_t> kv_split_codes;
  int32_t* d_kv_split_codes = nullptr;
  int kv_max_steps = 0;       // longest tile
  double kv_head_steps = 0;   // steps of all tiles of a head, averaged over heads
  // Backward that keeps dS (64- and 128-token blocks): the dK/dV pass leaves dS in units of 64
  // queries x 64 keys, unit (2 * step + wavefront pair) of its walk over kv_tiles; dq_units names, for
  // every 64-key chunk of the q_tiles lists and either 64-row half of the query tile, the unit that
  // holds it (-1: the mask row drops the block, or no pair of the piece is causal).
  std::vector<int32_t> dq_units;
  int32_t* d_dq_units = nullptr;
  int64_t ds_units = 0;   // units per batch element (0: this layout does not support the path)
};

namespace s2 {
// Host-only construction (no HIP calls).  Returns an S2_* status.
int build_host(const s2_layout_params& p, s2_layout& L);
// The same from caller-supplied compressed rows (validated: ascending, causal, diagonal kept).
int build_from_csr(int num_heads, int num_blocks, int block_size, const int32_t* row_ptr,
                   const int32_t* col_idx, s2_layout& L);
// Kept block columns of block row i of local head `head`, ascending, in closed form (no layout
// needed, any i >= 0): writes at most `capacity` of them to out and returns how many there are.
int64_t row_blocks(const s2_layout_params& p, int head, int i, int32_t* out, int64_t capacity);
// Merge `group` consecutive rows (transpose=false) or columns (transpose=true).
void build_tiles(const s2_layout& L, int group, bool transpose, TileList& out);
// Fills kv_levels and what belongs to them from kv_tiles (entries of single blocks).
void build_splits(s2_layout& L);
// Fills dq_units / ds_units from q_tiles and kv_tiles (built before, with 128-row and 128-key tiles).
void build_ds_units(s2_layout& L);
}  // namespace s2
