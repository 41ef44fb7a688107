// C ABI of libs2attn.so: argument validation, the layout handle's device copies, and dispatch to
// the kernels.  See include/s2attn.h for the contract of every entry point.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <limits>
#include <new>

#include "../../include/s2attn.h"
#include "config.h"
#include "kernels.h"
#include "layout.h"

namespace {

thread_local int g_last_hip_error = 0;

inline bool hip_ok(hipError_t e) {
  if (e == hipSuccess) return true;
  g_last_hip_error = (int)e;
  return false;
}

bool upload(const std::vector<int32_t>& host, int32_t** dev) {
  *dev = nullptr;
  const size_t bytes = (host.empty() ? 1 : host.size()) * sizeof(int32_t);
  if (!hip_ok(hipMalloc(reinterpret_cast<void**>(dev), bytes))) return false;
  if (host.empty()) return true;
  return hip_ok(hipMemcpy(*dev, host.data(), host.size() * sizeof(int32_t), hipMemcpyHostToDevice));
}

bool upload_tiles(s2::TileList& t) {
  return upload(t.ptr, &t.d_ptr) && upload(t.ent, &t.d_ent) && upload(t.rec, &t.d_rec);
}

void free_tiles(s2::TileList& t) {
  if (t.d_ptr) (void)hipFree(t.d_ptr);
  if (t.d_ent) (void)hipFree(t.d_ent);
  if (t.d_rec) (void)hipFree(t.d_rec);
  t.d_ptr = t.d_ent = t.d_rec = nullptr;
}

void free_device_copies(s2_layout* L) {
  free_tiles(L->q_tiles);
  free_tiles(L->kv_tiles);
  if (L->d_row_ptr) (void)hipFree(L->d_row_ptr);
  if (L->d_col_idx) (void)hipFree(L->d_col_idx);
  if (L->d_dq_units) (void)hipFree(L->d_dq_units);
  if (L->d_kv_split_codes) (void)hipFree(L->d_kv_split_codes);
  L->d_row_ptr = L->d_col_idx = L->d_dq_units = L->d_kv_split_codes = nullptr;
}

s2::DevTiles dev_tiles(const s2::TileList& t) {
  s2::DevTiles d;
  d.ptr = t.d_ptr;
  d.ent = t.d_ent;
  d.rec = t.d_rec;
  d.tiles_per_head = t.tiles_per_head;
  d.group = t.group;
  return d;
}

// The lists the row-tile and key-tile kernels walk.
void set_tiles(s2::AttnParams& p, const s2_layout* L) {
  p.q_tiles = dev_tiles(L->q_tiles);
  p.kv_tiles = dev_tiles(L->kv_tiles);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// The split partials of s2_attn_decode_static live here instead of in a caller's workspace: device
// memory that belongs to the loaded library, one copy per GPU at that GPU's own address, held
// until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; the address found there, kept per device, is what the kernels are given.
constexpr size_t kStaticScratchBytes = S2_DECODE_STATIC_SCRATCH_BYTES;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kScratchMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kScratchMaxDevices];  // zero-initialised: not looked up yet

// Address of `scratch` on the current device, or nullptr (the hipError_t is kept for
// s2_last_hip_error).  The first call on a device asks the runtime; later calls read the slot.
void* scratch_on_current_device() {
  int dev = -1;
  if (!hip_ok(hipGetDevice(&dev))) return nullptr;
  if (dev < 0 || dev >= kScratchMaxDevices) {
    g_last_hip_error = (int)hipErrorInvalidDevice;
    return nullptr;
  }
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr) return ptr;
  if (!hip_ok(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) || !ptr) return nullptr;
  g_scratch_ptr[dev].store(ptr, std::memory_order_release);  // racing threads store the same address
  return ptr;
}

// Shape / alignment checks shared by forward and backward.  `need_bwd` also checks the
// gradient tensors.
int check_tensors(const s2_tensors* t, bool need_bwd, float scale) {
  if (!t) return S2_ERR_NULL;
  if (!t->q || !t->k || !t->v || !t->o || !t->lse) return S2_ERR_NULL;
  if (need_bwd && (!t->d_o || !t->dq || !t->dk || !t->dv)) return S2_ERR_NULL;
  if (!(scale > 0.f) || !std::isfinite(scale)) return S2_ERR_BAD_PARAM;
  if (t->batch < 1 || t->heads < 1 || t->seqlen < 1) return S2_ERR_SHAPE;
  if (t->head_dim != 64 && t->head_dim != 128) return S2_ERR_SHAPE;
  if ((int64_t)t->batch * t->heads * t->seqlen > (int64_t)1 << 40) return S2_ERR_SHAPE;
  const int64_t strides[6] = {t->q_stride_b, t->q_stride_h, t->q_stride_t,
                              t->kv_stride_b, t->kv_stride_h, t->kv_stride_t};
  for (int64_t s : strides)
    if (s < 0 || (s & 7) != 0) return S2_ERR_ALIGN;
  if (t->q_stride_t < t->head_dim || t->kv_stride_t < t->head_dim) return S2_ERR_ALIGN;
  // the kernels address the 16 rows of a piece with unsigned 32-bit byte offsets
  if (t->q_stride_t > (1 << 24) || t->kv_stride_t > (1 << 24)) return S2_ERR_SHAPE;
  const void* ptrs[9] = {t->q, t->k, t->v, t->o, t->lse, t->d_o, t->dq, t->dk, t->dv};
  for (int i = 0; i < (need_bwd ? 9 : 5); ++i)
    if (!aligned16(ptrs[i])) return S2_ERR_ALIGN;
  return S2_OK;
}

s2::AttnParams make_params(const s2_tensors* t, float scale) {
  s2::AttnParams p{};
  p.q = static_cast<const uint16_t*>(t->q);
  p.k = static_cast<const uint16_t*>(t->k);
  p.v = static_cast<const uint16_t*>(t->v);
  p.o = static_cast<uint16_t*>(t->o);
  p.lse = t->lse;
  p.d_o = static_cast<const uint16_t*>(t->d_o);
  p.dq = static_cast<uint16_t*>(t->dq);
  p.dk = static_cast<uint16_t*>(t->dk);
  p.dv = static_cast<uint16_t*>(t->dv);
  p.batch = t->batch;
  p.heads = t->heads;
  p.seqlen = t->seqlen;
  p.q_row0 = 0;
  p.q_rows = t->seqlen;
  p.head_dim = t->head_dim;
  p.q_sb = t->q_stride_b;
  p.q_sh = t->q_stride_h;
  p.q_st = t->q_stride_t;
  p.kv_sb = t->kv_stride_b;
  p.kv_sh = t->kv_stride_h;
  p.kv_st = t->kv_stride_t;
  p.scale = scale;
  p.scale_log2e = scale * 1.4426950408889634f;
  // The dK/dV kernel forms P as exp(s * (S - lse / s)).  s is the scale, but not below 2^-120, so that lse / s is finite; where it is not
  // the scale P is off by a factor of exp(S * (s - scale)), which is 1 to float32's precision for |S| up to 2^96.
  const float s = std::max(scale, 0x1p-120f);
  p.neg_inv_scale = -1.0f / s;
  p.p_scale_log2e = s * 1.4426950408889634f;
  return p;
}

// The layout's lists live on the device that was current when it was built.
bool layout_on_current_device(const s2_layout* L) {
  if (!L->on_device) return false;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return dev == L->device;
}

int check_layout_fits(const s2_layout* L, const s2_tensors* t) {
  if (!L) return S2_ERR_NULL;
  if (t->heads != L->p.num_heads) return S2_ERR_SHAPE;
  if ((int64_t)t->seqlen != (int64_t)L->p.num_blocks * L->p.block_size) return S2_ERR_SHAPE;
  return S2_OK;
}

}  // namespace

extern "C" {

namespace {
// Tile lists for the three passes, then the device copy when a GPU is visible.  Takes ownership
// of L: on failure it is deleted.
int finish_layout(s2_layout* L, int st, s2_layout** out) {
  if (st == S2_OK) {
    try {
      const int S = L->p.block_size;
      static_assert(s2::kFwdBM == s2::kBwdBM, "forward and dQ walk the same lists");
      s2::build_tiles(*L, s2::kBwdBM / S, false, L->q_tiles);
      s2::build_tiles(*L, s2::kBwdBN / S, true, L->kv_tiles);
      s2::build_splits(*L);
      s2::build_ds_units(*L);
    } catch (const std::bad_alloc&) {
      st = S2_ERR_OVERFLOW;
    }
  }
  if (st != S2_OK) {
    delete L;
    return st;
  }
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) == hipSuccess && ndev > 0) {
    int dev = 0;
    bool ok = hip_ok(hipGetDevice(&dev)) && upload_tiles(L->q_tiles) && upload_tiles(L->kv_tiles) && upload(L->row_ptr, &L->d_row_ptr) &&
              upload(L->col_idx, &L->d_col_idx) && upload(L->dq_units, &L->d_dq_units) &&
              upload(L->kv_split_codes, &L->d_kv_split_codes);
    if (!ok) {
      free_device_copies(L);
      delete L;
      return S2_ERR_HIP;
    }
    L->device = dev;
    L->on_device = true;
  } else {
    (void)hipGetLastError();  // no GPU: a host-only layout is still a valid result
  }
  *out = L;
  return S2_OK;
}
}  // namespace

int s2_layout_build(const s2_layout_params* params, s2_layout** out) {
  if (!params || !out) return S2_ERR_NULL;
  *out = nullptr;
  s2_layout* L = new (std::nothrow) s2_layout();
  if (!L) return S2_ERR_OVERFLOW;
  int st;
  try {
    st = s2::build_host(*params, *L);
  } catch (const std::bad_alloc&) {
    st = S2_ERR_OVERFLOW;
  }
  return finish_layout(L, st, out);
}

int s2_layout_from_csr(int32_t num_heads, int32_t num_blocks, int32_t block_size, const int32_t* row_ptr,
                       const int32_t* col_idx, s2_layout** out) {
  if (!row_ptr || !col_idx || !out) return S2_ERR_NULL;
  *out = nullptr;
  s2_layout* L = new (std::nothrow) s2_layout();
  if (!L) return S2_ERR_OVERFLOW;
  int st;
  try {
    st = s2::build_from_csr(num_heads, num_blocks, block_size, row_ptr, col_idx, *L);
  } catch (const std::bad_alloc&) {
    st = S2_ERR_OVERFLOW;
  }
  return finish_layout(L, st, out);
}

int s2_layout_destroy(s2_layout* layout) {
  if (!layout) return S2_ERR_NULL;
  if (layout->on_device) free_device_copies(layout);
  delete layout;
  return S2_OK;
}

int s2_layout_get(const s2_layout* L, s2_layout_view* out) {
  if (!L || !out) return S2_ERR_NULL;
  out->row_ptr = L->row_ptr.data();
  out->col_idx = L->col_idx.data();
  out->col_ptr = L->col_ptr.data();
  out->row_idx = L->row_idx.data();
  out->nnz = L->nnz;
  out->num_heads = L->p.num_heads;
  out->num_blocks = L->p.num_blocks;
  out->block_size = L->p.block_size;
  out->max_row_blocks = L->max_row_blocks;
  out->covers_all = L->covers_all;
  out->on_device = L->on_device ? 1 : 0;
  return S2_OK;
}

int s2_layout_get_tiles(const s2_layout* L, int which, s2_tile_view* out) {
  if (!L || !out) return S2_ERR_NULL;
  if (which != S2_TILES_FWD && which != S2_TILES_DQ && which != S2_TILES_DKDV) return S2_ERR_BAD_PARAM;
  const s2::TileList& t = which == S2_TILES_DKDV ? L->kv_tiles : L->q_tiles;
  out->ptr = t.ptr.data();
  out->ent = t.ent.data();
  out->order = t.order.data();
  out->members = t.members.data();
  out->tiles_per_head = t.tiles_per_head;
  out->group = t.group;
  out->blocks_per_unit = 1;
  return S2_OK;
}

int s2_layout_get_ds_units(const s2_layout* L, s2_ds_units_view* out) {
  if (!L || !out) return S2_ERR_NULL;
  out->dq_units = L->dq_units.data();
  out->count = (int64_t)L->dq_units.size();
  out->ds_units = L->ds_units;
  return S2_OK;
}

int s2_attn_fwd(const s2_layout* layout, const s2_tensors* t, float scale, void* stream) {
  if (!layout) return S2_ERR_NULL;
  int st = check_tensors(t, false, scale);
  if (st != S2_OK) return st;
  st = check_layout_fits(layout, t);
  if (st != S2_OK) return st;
  if (!layout_on_current_device(layout)) return S2_ERR_NO_DEVICE;
  s2::AttnParams p = make_params(t, scale);
  p.block_size = layout->p.block_size;
  set_tiles(p, layout);
  return hip_ok(s2::launch_fwd(p, false, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

namespace {

size_t round256(size_t bytes) { return (bytes + 255) / 256 * 256; }

// The backward's workspace: the row statistics -delta = -rowsum(dO * O) and -lse / scale; then dS, where it is kept;
// then, for launches of so few tiles that the longest ones may be cut, a counter per key tile and the sums of the
// parts.  Without the last nothing is cut, without room for dS it is not kept, and neither depends on the other.
struct BwdWorkspace {
  size_t stats;      // bytes of either of the first two arrays
  size_t count;      // of the counters
  size_t sums;       // of the sums
  int64_t slots;     // parts that there is room for
  size_t required() const { return 2 * stats; }
  size_t cut() const { return count + sums; }
};
BwdWorkspace bwd_workspace(int32_t batch, int32_t heads, int32_t seqlen, int32_t head_dim) {
  BwdWorkspace w{};
  const int64_t rows = (int64_t)batch * heads * seqlen;
  w.stats = round256((size_t)rows * sizeof(float));
  const int64_t per_head = (seqlen + s2::kBwdBN - 1) / s2::kBwdBN, tiles = (int64_t)batch * heads * per_head;
  // From 4096 tiles on (eight rounds of the chip's 512 workgroup slots) the longest tile no longer decides.  (head_dim
  // is not checked here: the query has never done so, and no call takes one that is neither 64 nor 128.)
  if (tiles < 4096 && head_dim > 0) {
    w.count = round256((size_t)tiles * sizeof(int32_t));
    // no tile is longer than all of its head's rows, two 64-row steps to a tile, and no part shorter than four steps
    w.slots = std::min<int64_t>(768, tiles * std::min<int64_t>(8, (2 * per_head + 3) / 4));
    w.sums = (size_t)w.slots * s2::kBwdBN * head_dim * 2 * sizeof(float);
  }
  return w;
}

}  // namespace

size_t s2_attn_bwd_workspace_bytes(int32_t batch, int32_t heads, int32_t seqlen, int32_t head_dim) {
  if (batch < 1 || heads < 1 || seqlen < 1) return 0;
  const BwdWorkspace w = bwd_workspace(batch, heads, seqlen, head_dim);
  return w.required() + w.cut();
}

namespace {

// Whether and how to cut the longest key tiles.  A stripe column is attended by every later row, so a head
// has a few tiles of up to N / 64 steps among many short ones.  With enough (batch, head) pairs the long
// ones are hidden behind the rest; with few the launch is as long as its longest tile while most
// of the chip idles.  `even`: the steps a workgroup slot would walk if all were shared out evenly (a tile
// costs about five steps besides its own, an XCD holds 64 workgroups of head_dim 128 and the
// equivalent of 80 of 64).  Measured, forward + backward with the longest tile / even = 4.4 (8 heads
// x 4096): 202 -> 89 us; 2.3 (2 x 16 x 3904): 255 -> 183; 3.0 (16 x 16384): 969 -> 637; 1.5 (2 x 20 x 8192,
// blocks of 128): 677 -> 616; 1.2 (3 x 16 x 8192): 791 -> 764; 0.88 (4 x 16 x 8192): 999 uncut, 1026 cut.  The
// best length of a part was 6 to 8, 24, 64, 48 to 64 and 64 steps, that is about 3/4 of `even` plus 3: a
// part's own cost (its start, 64 KB per 128 keys and 64 features written and read again) against the evenness of the launch.
// Where all tiles start at once they should still do so when cut: 52 heads x 800 x 128 in blocks of 32, 49 workgroups for
// an XCD's 64 slots uncut and 84 cut, forward and backward 78 us uncut, 90 cut; 42 heads, 42 and 54, 66 and 54.  Where no
// cut leaves it so, a second round still costs less than a tile much longer than a part: with longest tile / best = 10 (8 heads x
// 8192 x 128, 64 workgroups and 88) 311 us uncut and 109 cut, 4.7 (16 x 4096 x 128) 191 and 112, 2.7 (4 x 8 x 2048 x 128) 123 and 89, 8.9 (8 x
// 10240 x 64) 262 and 119, but with 2.4 (3 x 8 x 2560 x 128) 172 and 168, or 141 and 152 in the launch that has the dQ tiles too, and with
// 1.9 (4 x 8 x 2048 x 128) 139 and 146 there.
// (batch, head) pairs that are left over from a multiple of eight are shared by the XCDs.  They count as a whole pair for whether to cut and
// what starts at once, as the parts of one tile lie on XCDs next to each other; for the best length three quarters of what they lack of one are added. And a
// cut whose parts all start at once is then no good where they are half as long again as the best length, or two thirds of it.  Backward, us,
// with pairs / 8, with that rounded up and so: 7 heads x 8192 x 128 122, 105 and 102, 4 x 23 x 768 79, 72 and 72, 2 x 8192 x 64 38, 56 and 35, 9 x 8192 x 64 84, 66 and 67, 3 x 4
// x 3072 x 128, blocks of 128, 72, 57 and 57.  Over 332 shapes with pairs left over each is this much behind the best of all cuts: 4.0, 3.5 and 2.6 %.
void choose_split(s2::AttnParams& p, const s2_layout* L, const BwdWorkspace& w, unsigned char* room) {
  const double slots = p.head_dim == 128 ? 64 : 80;
  const int T = p.kv_tiles.tiles_per_head;
  const int pairs = (p.batch * p.heads + 7) / 8;  // of an XCD
  const double even = (L->kv_head_steps + 5.0 * T) / slots;  // of each of them
  if (L->kv_max_steps <= 1.1 * pairs * even) return;
  const double best = 0.75 * (3 * pairs + p.batch * p.heads / 8.0) / 4 * even + 3;
  double off;  // how far from the best length the parts are of the cut that `closest` has found
  auto closest = [&](bool one_round) {
    const s2::SplitLevel* use = nullptr;
    off = 0;
    for (const s2::SplitLevel& lv : L->kv_levels) {
      if ((int64_t)p.batch * p.heads * lv.n_items > w.slots || 2 * lv.steps > L->kv_max_steps) continue;
      if (one_round && pairs * (T + lv.n_items - lv.n_long) > slots) continue;
      const double o = std::max(lv.steps / best, best / lv.steps);
      if (use && o >= off) continue;
      use = &lv;
      off = o;
    }
    return use;
  };
  const bool one_round = pairs * T <= slots;
  const s2::SplitLevel* use = closest(one_round);
  const double far = p.batch * p.heads % 8 ? 1.5 : HUGE_VAL;
  if (one_round && (!use || off > far) && L->kv_max_steps > 2.4 * best) use = closest(false);
  if (!use) return;
  p.split_codes = L->d_kv_split_codes + use->offset;
  p.split_items = use->n_items;
  p.split_long = use->n_long;
  p.split_count = reinterpret_cast<int32_t*>(room);
  p.split_sums = reinterpret_cast<float*>(room + w.count);
}

// The backward that keeps dS covers head_dim 128, mask blocks of 64 or 128 tokens (the layout then
// carries the unit table) and whole 128-row tiles.
bool keeps_ds(const s2_layout* L, int32_t seqlen, int32_t head_dim) {
  return L->ds_units > 0 && head_dim == 128 && seqlen % s2::kBwdBM == 0 &&
         (int64_t)seqlen == (int64_t)L->p.num_blocks * L->p.block_size;
}
}  // namespace

size_t s2_attn_bwd_layout_workspace_bytes(const s2_layout* layout, int32_t batch, int32_t heads, int32_t seqlen,
                                          int32_t head_dim) {
  const size_t small = s2_attn_bwd_workspace_bytes(batch, heads, seqlen, head_dim);
  if (!layout || small == 0 || heads != layout->p.num_heads || !keeps_ds(layout, seqlen, head_dim)) return small;
  return small + (size_t)batch * (size_t)layout->ds_units * 8192;
}

int s2_attn_bwd(const s2_layout* layout, const s2_tensors* t, float scale, void* workspace,
                size_t workspace_bytes, void* stream) {
  return s2_attn_bwd_stages(layout, t, scale, workspace, workspace_bytes, S2_BWD_ALL, stream);
}

int s2_attn_fwd_rows(const s2_layout* layout, const s2_tensors* t, int32_t q_row_start, int32_t q_rows,
                     float scale, void* stream) {
  if (!layout) return S2_ERR_NULL;
  int st = check_tensors(t, false, scale);
  if (st != S2_OK) return st;
  if (t->heads != layout->p.num_heads) return S2_ERR_SHAPE;
  if ((int64_t)t->seqlen > (int64_t)layout->p.num_blocks * layout->p.block_size) return S2_ERR_SHAPE;
  if (q_row_start < 0 || q_rows < s2::kFwdBM || q_row_start % s2::kFwdBM != 0 || q_rows % s2::kFwdBM != 0)
    return S2_ERR_SHAPE;
  if ((int64_t)q_row_start + q_rows > t->seqlen) return S2_ERR_SHAPE;
  if (!layout_on_current_device(layout)) return S2_ERR_NO_DEVICE;
  s2::AttnParams p = make_params(t, scale);
  p.q_row0 = q_row_start;
  p.q_rows = q_rows;
  p.block_size = layout->p.block_size;
  set_tiles(p, layout);
  return hip_ok(s2::launch_fwd(p, false, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

int s2_attn_fwd_varlen(const s2_layout* layout, const s2_tensors* t, const int32_t* cu_seqlens,
                       int32_t num_seqs, int32_t max_seqlen, float scale, void* stream) {
  if (!layout || !cu_seqlens) return S2_ERR_NULL;
  int st = check_tensors(t, false, scale);
  if (st != S2_OK) return st;
  if (t->batch != 1 || t->heads != layout->p.num_heads) return S2_ERR_SHAPE;
  if (num_seqs < 1 || max_seqlen < 1) return S2_ERR_SHAPE;
  if ((int64_t)max_seqlen > (int64_t)layout->p.num_blocks * layout->p.block_size) return S2_ERR_SHAPE;
  if ((int64_t)num_seqs * t->heads > std::numeric_limits<int32_t>::max() / 2) return S2_ERR_SHAPE;
  if ((reinterpret_cast<uintptr_t>(cu_seqlens) & 3u) != 0) return S2_ERR_ALIGN;
  if (!layout_on_current_device(layout)) return S2_ERR_NO_DEVICE;
  s2::AttnParams p = make_params(t, scale);
  p.batch = num_seqs;
  p.q_rows = max_seqlen;
  p.cu_seqlens = cu_seqlens;
  p.block_size = layout->p.block_size;
  set_tiles(p, layout);
  // one grid slot per (sequence, head, 128-row tile of the longest length allowed)
  const int64_t slots = 8 * (((int64_t)num_seqs * t->heads + 7) / 8) * ((max_seqlen + s2::kFwdBM - 1) / s2::kFwdBM);
  if (slots > std::numeric_limits<int32_t>::max()) return S2_ERR_SHAPE;
  return hip_ok(s2::launch_fwd(p, false, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

size_t s2_attn_bwd_varlen_workspace_bytes(int32_t heads, int32_t rows, int32_t head_dim) {
  (void)head_dim;
  if (heads < 1 || rows < 1) return 0;
  // the two row statistics per (head, row), plus one chunk of slack each: the dK/dV kernel fetches the
  // statistics of a whole 64-row chunk even where a sequence ends inside it
  const size_t floats = (size_t)heads * rows + 64;
  return 2 * (((floats * sizeof(float) + 255) / 256) * 256);
}

int s2_attn_bwd_varlen(const s2_layout* layout, const s2_tensors* t, const int32_t* cu_seqlens,
                       int32_t num_seqs, int32_t max_seqlen, float scale, void* workspace,
                       size_t workspace_bytes, void* stream) {
  if (!layout || !cu_seqlens) return S2_ERR_NULL;
  int st = check_tensors(t, true, scale);
  if (st != S2_OK) return st;
  if (t->batch != 1 || t->heads != layout->p.num_heads) return S2_ERR_SHAPE;
  if (num_seqs < 1 || max_seqlen < 1) return S2_ERR_SHAPE;
  if ((int64_t)max_seqlen > (int64_t)layout->p.num_blocks * layout->p.block_size) return S2_ERR_SHAPE;
  if ((reinterpret_cast<uintptr_t>(cu_seqlens) & 3u) != 0) return S2_ERR_ALIGN;
  const size_t need = s2_attn_bwd_varlen_workspace_bytes(t->heads, t->seqlen, t->head_dim);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < need)
    return S2_ERR_WORKSPACE;
  if (!layout_on_current_device(layout)) return S2_ERR_NO_DEVICE;
  s2::AttnParams p = make_params(t, scale);
  p.batch = num_seqs;
  p.q_rows = max_seqlen;
  p.cu_seqlens = cu_seqlens;
  p.block_size = layout->p.block_size;
  set_tiles(p, layout);
  p.neg_delta = static_cast<float*>(workspace);
  p.neg_lse = p.neg_delta + need / 8;
  // one grid slot per (sequence, head, tile): query tiles of the longest length allowed, key tiles of the layout
  const int64_t pairs = 8 * (((int64_t)num_seqs * t->heads + 7) / 8);
  const int64_t slots = pairs * std::max<int64_t>((max_seqlen + s2::kBwdBM - 1) / s2::kBwdBM, layout->kv_tiles.tiles_per_head);
  if (slots > std::numeric_limits<int32_t>::max()) return S2_ERR_SHAPE;
  // (whole runs of key tiles can be a few more)
  if (s2::key_map(num_seqs * t->heads, layout->kv_tiles.tiles_per_head).grid() > std::numeric_limits<int32_t>::max()) return S2_ERR_SHAPE;
  return hip_ok(s2::launch_bwd(p, false, s2::kBwdAll, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

int s2_attn_bwd_stages(const s2_layout* layout, const s2_tensors* t, float scale, void* workspace,
                       size_t workspace_bytes, int stages, void* stream) {
  if (!layout) return S2_ERR_NULL;
  if (stages < 1 || stages > S2_BWD_ALL) return S2_ERR_BAD_PARAM;
  int st = check_tensors(t, true, scale);
  if (st != S2_OK) return st;
  st = check_layout_fits(layout, t);
  if (st != S2_OK) return st;
  const BwdWorkspace w = bwd_workspace(t->batch, t->heads, t->seqlen, t->head_dim);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < w.required())
    return S2_ERR_WORKSPACE;
  if (!layout_on_current_device(layout)) return S2_ERR_NO_DEVICE;
  s2::AttnParams p = make_params(t, scale);
  p.neg_delta = static_cast<float*>(workspace);
  p.neg_lse = p.neg_delta + w.stats / sizeof(float);
  p.block_size = layout->p.block_size;
  set_tiles(p, layout);
  unsigned char* const ws = static_cast<unsigned char*>(workspace);
  size_t used = w.required();
  // Room for dS selects the backward that computes nothing twice.  Where there is room for dS or for cutting
  // tiles but not for both, the workspace is of the size asked for cutting alone if that is the larger of the two.
  const size_t ds_bytes = (size_t)t->batch * (size_t)layout->ds_units * 8192;
  if (keeps_ds(layout, t->seqlen, t->head_dim) && workspace_bytes >= used + ds_bytes &&
      (workspace_bytes >= used + ds_bytes + w.cut() || workspace_bytes < used + w.cut() || ds_bytes > w.cut())) {
    p.ds_store = reinterpret_cast<uint16_t*>(ws + used);
    p.ds_units = layout->ds_units;
    p.dq_units = layout->d_dq_units;
    used += ds_bytes;
  }
  if (w.slots > 0 && workspace_bytes >= used + w.cut()) choose_split(p, layout, w, ws + used);
  return hip_ok(s2::launch_bwd(p, false, stages, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

static int dense_params(const s2_tensors* t, s2::AttnParams& p) {
  if (t->seqlen % 128 != 0) return S2_ERR_SHAPE;
  p.block_size = s2::kChunk;
  p.q_tiles.tiles_per_head = t->seqlen / s2::kBwdBM;
  p.q_tiles.group = s2::kBwdBM / s2::kChunk;
  p.kv_tiles.tiles_per_head = t->seqlen / s2::kBwdBN;
  p.kv_tiles.group = s2::kBwdBN / s2::kChunk;
  return S2_OK;
}

int s2_dense_causal_fwd(const s2_tensors* t, float scale, void* stream) {
  int st = check_tensors(t, false, scale);
  if (st != S2_OK) return st;
  s2::AttnParams p = make_params(t, scale);
  st = dense_params(t, p);
  if (st != S2_OK) return st;
  return hip_ok(s2::launch_fwd(p, true, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

int s2_dense_causal_bwd(const s2_tensors* t, float scale, void* workspace, size_t workspace_bytes,
                        void* stream) {
  int st = check_tensors(t, true, scale);
  if (st != S2_OK) return st;
  const BwdWorkspace w = bwd_workspace(t->batch, t->heads, t->seqlen, t->head_dim);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < w.required())
    return S2_ERR_WORKSPACE;
  s2::AttnParams p = make_params(t, scale);
  st = dense_params(t, p);
  if (st != S2_OK) return st;
  p.neg_delta = static_cast<float*>(workspace);
  p.neg_lse = p.neg_delta + w.stats / sizeof(float);
  return hip_ok(s2::launch_bwd(p, true, s2::kBwdAll, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

size_t s2_dense_causal_bwd_workspace_bytes(int32_t batch, int32_t heads, int32_t seqlen, int32_t head_dim) {
  if (batch < 1 || heads < 1 || seqlen < 1) return 0;
  return bwd_workspace(batch, heads, seqlen, head_dim).required();
}

int32_t s2_attn_decode_default_splits(int32_t nseq, int32_t heads, int32_t max_len) {
  if (nseq < 1 || heads < 1 || max_len < 1) return 1;
  // aim for a few workgroups per compute unit (256 CUs); never more splits than 1K-token pieces
  const int64_t pairs = (int64_t)nseq * heads;
  int64_t want = (4 * 256 + pairs - 1) / pairs;
  const int64_t cap = (max_len + 1023) / 1024;
  if (want > cap) want = cap;
  if (want < 1) want = 1;
  if (want > 64) want = 64;
  return (int32_t)want;
}

size_t s2_attn_decode_workspace_bytes(int32_t nseq, int32_t heads, int32_t head_dim, int32_t max_len,
                                      int32_t num_splits) {
  if (nseq < 1 || heads < 1 || head_dim < 1) return 0;
  if (num_splits <= 0) num_splits = s2_attn_decode_default_splits(nseq, heads, max_len);
  const size_t items = (size_t)nseq * heads * num_splits;
  return ((items * (head_dim + 2) * sizeof(float) + 255) / 256) * 256;
}

namespace {

bool good_block_size(int S) { return S == 16 || S == 32 || S == 64 || S == 128; }

// The pattern a decode call follows: the closed form of `lp`, or, when `layout` is given, the
// layout's own rows (then lp = &layout->p supplies S and the head count only).
int check_pattern(const s2_layout_params* lp, const s2_layout* layout, int heads, int64_t max_len) {
  if (!good_block_size(lp->block_size)) return S2_ERR_BAD_PARAM;
  if (heads != lp->num_heads) return S2_ERR_SHAPE;
  if (layout) {
    if (max_len > (int64_t)lp->num_blocks * lp->block_size) return S2_ERR_SHAPE;
    return layout_on_current_device(layout) ? S2_OK : S2_ERR_NO_DEVICE;
  }
  if (lp->dense != 0 && lp->dense != 1) return S2_ERR_BAD_PARAM;
  if (!lp->dense && (lp->local_blocks < 1 || lp->stride < 0 || lp->window_blocks < 0)) return S2_ERR_BAD_PARAM;
  if (lp->head_index_base < 0) return S2_ERR_BAD_PARAM;
  return S2_OK;
}

// Split count when the caller leaves it to the library; never more than the public default, which also
// sizes the workspace.  A trip of a workgroup's wavefronts, a unit each (64 tokens, or a block of 32), takes 1.5 to 2 us
// however few workgroups there are, the second launch that merges splits 2 to 3 us.  Three ranges:
//  - All of a call's workgroups are of eight wavefronts and fit the chip at once: one split is best up to three trips
//    (four at head_dim 64), then as many as still fit, down to one trip each: 32 pairs of 19 units 11.1 us in one
//    split, 11.5 in two; of 31 units 16.3 in one, 11.2 in four; 75 pairs of 34 units 14.2, 12.5 in three, 16.1 in four.
//    Where only one fits but leaves a third of the chip idle, three splits of four wavefronts share it better (160 pairs of 95
//    units 60.1 us in one, 55.4; of 47 units 29.8, 28.5; 192 pairs: 71.8, 78.6).  Long rows of many pairs are cut
//    into pieces of 24 units though not all fit: sequences of different lengths even out better, and equal ones lose
//    little.  From 384 units on where two fit (four in blocks of 32, whose units are half as large), from 512 where
//    one does: 96 pairs of 128 to 512 units x 128 179 us in two splits, 163 in eight, all of 384 203 and 206; 80 pairs of 256
//    to 1024 32-token units x 64 101 in three, 82 in twelve; 180 pairs of 128 to 512 x 128 370 in one, 350 in six.
//  - Above that (192 pairs, 256 in blocks of 16), up to 255 pairs: one split while rows are short, then pieces of a dozen units.  At
//    head_dim 128 from 256 units on (200 pairs of 64 to 256 units 204 us in one split, 179 in six, all of 384 411 and 414, but
//    all of 128 139 and 148), at 64 from 96 (all of 128 89 and 83, of 64 34 and 39), in blocks of 32 from 64 (of 64 x 128
//    47 in one, 39 in two; of 256 to 1024 x 64 470 in one, 176 in six).
//  - With more pairs the cache's bytes count, and splits must be worth their partials: a dozen units each at least (512
//    pairs, 19 units: 33.5 us in one split, 37.0 in two).
int choose_splits(const s2_layout_params* lp, const s2_layout* layout, int nseq, int heads, int head_dim, int max_len,
                  size_t workspace_bytes) {
  const int splits = s2_attn_decode_default_splits(nseq, heads, max_len);
  const int S = lp->block_size;
  const int64_t blocks = layout ? layout->max_row_blocks : s2::row_blocks(*lp, 0, (max_len - 1) / S, nullptr, 0);
  const int64_t units64 = blocks * S / 64;                // 64 tokens each
  const int64_t units = S == 32 ? blocks : units64;       // as the kernel counts them, in the longest row
  const int64_t pairs = (int64_t)nseq * heads;
  int64_t cap;
  const int64_t fit = s2::kDecodeWideGroups / pairs;  // splits of eight wavefronts that fit
  const int64_t few = S == 16 ? 256 : 192;                // the first range's pairs
  if (pairs >= 256 && pairs > few) {
    cap = units64 / 12;
  } else if (pairs > few) {
    cap = units >= (S == 32 ? 64 : head_dim == 64 ? 96 : 256) ? units / 12 : 1;
  } else if (units <= (head_dim == 128 ? 24 : 32)) {
    cap = 1;
  } else if (fit <= (S == 32 ? 4 : 2) && units >= (fit == 1 && S != 32 ? 512 : 384)) {
    cap = units / 24;
  } else {
    cap = std::min<int64_t>((units + 7) / 8, fit);
    if (cap == 1 && S != 16 && 3 * pairs <= 512) cap = 3;
  }
  int n = (int)std::max<int64_t>(1, std::min<int64_t>(splits, cap));
  // a workspace that holds the partials of a split to every 768 tokens is enough
  while (n > 1 && 12 * (int64_t)n > units64 && s2_attn_decode_workspace_bytes(nseq, heads, head_dim, max_len, n) > workspace_bytes) --n;
  return n;
}

void set_pattern(s2::DecodeParams& p, const s2_layout_params* lp, const s2_layout* layout) {
  p.block_size = lp->block_size;
  p.local_blocks = lp->local_blocks;
  p.stride = lp->stride;
  p.window_blocks = lp->window_blocks;
  p.dense = lp->dense;
  p.head_index_base = lp->head_index_base;
  if (layout) {
    p.row_ptr = layout->d_row_ptr;
    p.col_idx = layout->d_col_idx;
    p.num_blocks = lp->num_blocks;
  }
}

int decode_contiguous(const s2_layout_params* lp, const s2_layout* layout, const s2_decode_args* a, float scale,
                      void* workspace, size_t workspace_bytes, void* stream) {
  if (!a->q || !a->k_cache || !a->v_cache || !a->seq_lens || !a->o) return S2_ERR_NULL;
  if (!(scale > 0.f) || !std::isfinite(scale)) return S2_ERR_BAD_PARAM;
  if (a->nseq < 1 || a->heads < 1 || a->max_len < 1) return S2_ERR_SHAPE;
  if (a->head_dim != 64 && a->head_dim != 128) return S2_ERR_SHAPE;
  int st = check_pattern(lp, layout, a->heads, a->max_len);
  if (st != S2_OK) return st;
  if (a->num_splits < 0 || a->num_splits > 64) return S2_ERR_BAD_PARAM;
  const int64_t strides[3] = {a->kv_stride_seq, a->kv_stride_head, a->kv_stride_tok};
  for (int64_t s : strides)
    if (s < 0 || (s & 7) != 0) return S2_ERR_ALIGN;
  if (a->kv_stride_tok < a->head_dim) return S2_ERR_ALIGN;
  if (!aligned16(a->q) || !aligned16(a->k_cache) || !aligned16(a->v_cache) || !aligned16(a->o) ||
      (reinterpret_cast<uintptr_t>(a->seq_lens) & 3u) != 0)
    return S2_ERR_ALIGN;
  const int splits = a->num_splits > 0 ? a->num_splits : choose_splits(lp, layout, a->nseq, a->heads, a->head_dim, a->max_len, workspace_bytes);
  const size_t need = s2_attn_decode_workspace_bytes(a->nseq, a->heads, a->head_dim, a->max_len, splits);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < need)
    return S2_ERR_WORKSPACE;

  s2::DecodeParams p{};
  p.q = static_cast<const uint16_t*>(a->q);
  p.k_cache = static_cast<const uint16_t*>(a->k_cache);
  p.v_cache = static_cast<const uint16_t*>(a->v_cache);
  p.seq_lens = a->seq_lens;
  p.o = static_cast<uint16_t*>(a->o);
  p.lse = a->lse;
  const size_t items = (size_t)a->nseq * a->heads * splits;
  p.part_acc = static_cast<float*>(workspace);
  p.part_ml = p.part_acc + items * a->head_dim;
  p.nseq = a->nseq;
  p.heads = a->heads;
  p.head_dim = a->head_dim;
  p.max_len = a->max_len;
  p.num_splits = splits;
  p.kv_ss = a->kv_stride_seq;
  p.kv_sh = a->kv_stride_head;
  p.kv_st = a->kv_stride_tok;
  p.scale = scale;
  p.scale_log2e = scale * 1.4426950408889634f;
  set_pattern(p, lp, layout);
  return hip_ok(s2::launch_decode(p, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

int decode_paged(const s2_layout_params* lp, const s2_layout* layout, const s2_paged_decode_args* a, float scale,
                 void* workspace, size_t workspace_bytes, void* stream) {
  if (!a->q || !a->k_pages || !a->v_pages || !a->block_table || !a->seq_lens || !a->o) return S2_ERR_NULL;
  if (!(scale > 0.f) || !std::isfinite(scale)) return S2_ERR_BAD_PARAM;
  if (!good_block_size(lp->block_size)) return S2_ERR_BAD_PARAM;
  if (a->nseq < 1 || a->heads < 1 || a->max_blocks < 1 || a->num_pages < 1) return S2_ERR_SHAPE;
  if ((int64_t)a->max_blocks * lp->block_size > std::numeric_limits<int32_t>::max()) return S2_ERR_SHAPE;
  if (a->head_dim != 64 && a->head_dim != 128) return S2_ERR_SHAPE;
  const int max_len = a->max_blocks * lp->block_size;
  int st = check_pattern(lp, layout, a->heads, max_len);
  if (st != S2_OK) return st;
  if (a->num_splits < 0 || a->num_splits > 64) return S2_ERR_BAD_PARAM;
  if (a->page_stride < 0 || (a->page_stride & 7) != 0 || a->tok_stride < 0 || (a->tok_stride & 7) != 0)
    return S2_ERR_ALIGN;
  if (a->tok_stride < a->head_dim) return S2_ERR_ALIGN;
  if (!aligned16(a->q) || !aligned16(a->k_pages) || !aligned16(a->v_pages) || !aligned16(a->o) ||
      (reinterpret_cast<uintptr_t>(a->seq_lens) & 3u) != 0 ||
      (reinterpret_cast<uintptr_t>(a->block_table) & 3u) != 0 ||
      (reinterpret_cast<uintptr_t>(a->missing) & 3u) != 0)
    return S2_ERR_ALIGN;
  const int splits = a->num_splits > 0 ? a->num_splits : choose_splits(lp, layout, a->nseq, a->heads, a->head_dim, max_len, workspace_bytes);
  const size_t need = s2_attn_decode_workspace_bytes(a->nseq, a->heads, a->head_dim, max_len, splits);
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 || workspace_bytes < need)
    return S2_ERR_WORKSPACE;

  s2::DecodeParams p{};
  p.q = static_cast<const uint16_t*>(a->q);
  p.k_cache = static_cast<const uint16_t*>(a->k_pages);
  p.v_cache = static_cast<const uint16_t*>(a->v_pages);
  p.seq_lens = a->seq_lens;
  p.o = static_cast<uint16_t*>(a->o);
  p.lse = a->lse;
  const size_t items = (size_t)a->nseq * a->heads * splits;
  p.part_acc = static_cast<float*>(workspace);
  p.part_ml = p.part_acc + items * a->head_dim;
  p.nseq = a->nseq;
  p.heads = a->heads;
  p.head_dim = a->head_dim;
  p.max_len = max_len;
  p.num_splits = splits;
  p.kv_ss = a->page_stride;
  p.kv_sh = 0;
  p.kv_st = a->tok_stride;
  p.scale = scale;
  p.scale_log2e = scale * 1.4426950408889634f;
  set_pattern(p, lp, layout);
  p.block_table = a->block_table;
  p.missing = a->missing;
  p.max_blocks = a->max_blocks;
  p.num_pages = a->num_pages;
  return hip_ok(s2::launch_decode(p, static_cast<hipStream_t>(stream))) ? S2_OK : S2_ERR_HIP;
}

}  // namespace

int s2_attn_decode(const s2_layout_params* lp, const s2_decode_args* a, float scale, void* workspace,
                   size_t workspace_bytes, void* stream) {
  if (!lp || !a) return S2_ERR_NULL;
  return decode_contiguous(lp, nullptr, a, scale, workspace, workspace_bytes, stream);
}

int s2_attn_decode_static(const s2_layout_params* lp, const s2_decode_args* a, float scale, void* stream) {
  if (!lp || !a) return S2_ERR_NULL;
  // the size check comes first and needs no device: shapes whose partials do not fit are refused
  if (a->nseq < 1 || a->heads < 1 || a->max_len < 1) return S2_ERR_SHAPE;
  if (a->head_dim != 64 && a->head_dim != 128) return S2_ERR_SHAPE;
  if (a->num_splits < 0 || a->num_splits > 64) return S2_ERR_BAD_PARAM;
  // num_splits == 0: the call may pick fewer splits than this bound, never more
  const size_t need = s2_attn_decode_workspace_bytes(a->nseq, a->heads, a->head_dim, a->max_len, a->num_splits);
  if (need > kStaticScratchBytes) return S2_ERR_WORKSPACE;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) {
    (void)hipGetLastError();
    return S2_ERR_NO_DEVICE;
  }
  void* ptr = scratch_on_current_device();
  if (!ptr) return S2_ERR_HIP;
  return decode_contiguous(lp, nullptr, a, scale, ptr, kStaticScratchBytes, stream);
}

int s2_attn_decode_paged(const s2_layout_params* lp, const s2_paged_decode_args* a, float scale,
                         void* workspace, size_t workspace_bytes, void* stream) {
  if (!lp || !a) return S2_ERR_NULL;
  return decode_paged(lp, nullptr, a, scale, workspace, workspace_bytes, stream);
}

int s2_attn_decode_layout(const s2_layout* layout, const s2_decode_args* a, float scale, void* workspace,
                          size_t workspace_bytes, void* stream) {
  if (!layout || !a) return S2_ERR_NULL;
  return decode_contiguous(&layout->p, layout, a, scale, workspace, workspace_bytes, stream);
}

int s2_attn_decode_paged_layout(const s2_layout* layout, const s2_paged_decode_args* a, float scale,
                                void* workspace, size_t workspace_bytes, void* stream) {
  if (!layout || !a) return S2_ERR_NULL;
  return decode_paged(&layout->p, layout, a, scale, workspace, workspace_bytes, stream);
}

int s2_layout_resident_blocks(const s2_layout* L, int32_t head, int32_t length, int32_t* blocks,
                              int32_t capacity, int32_t* count) {
  if (!L || !count) return S2_ERR_NULL;
  if (capacity < 0 || (capacity > 0 && !blocks)) return S2_ERR_NULL;
  const int B = L->p.num_blocks, S = L->p.block_size;
  if (head < 0 || head >= L->p.num_heads || length < 1 || (int64_t)length > (int64_t)B * S)
    return S2_ERR_BAD_PARAM;
  // A block among 0..i (i = row of the newest token) stays while row i or any later row keeps it:
  // walk each such column's list of attending rows (ascending) and look at its last entry.
  const int i = (length - 1) / S;
  int64_t n = 0;
  for (int j = 0; j <= i; ++j) {
    const int32_t lo = L->col_ptr[(size_t)head * B + j], hi = L->col_ptr[(size_t)head * B + j + 1];
    if (hi > lo && L->row_idx[hi - 1] >= i) {
      if (n < capacity) blocks[n] = j;
      ++n;
    }
  }
  *count = (int32_t)n;
  return n > capacity ? S2_ERR_OVERFLOW : S2_OK;
}

int s2_kv_resident_blocks(const s2_layout_params* lp, int32_t head, int32_t length, int32_t* blocks,
                          int32_t capacity, int32_t* count) {
  if (!lp || !count) return S2_ERR_NULL;
  if (capacity < 0 || (capacity > 0 && !blocks)) return S2_ERR_NULL;
  if (!good_block_size(lp->block_size)) return S2_ERR_BAD_PARAM;
  if (lp->dense != 0 && lp->dense != 1) return S2_ERR_BAD_PARAM;
  if (!lp->dense && (lp->local_blocks < 1 || lp->stride < 0 || lp->window_blocks < 0)) return S2_ERR_BAD_PARAM;
  if (lp->head_index_base < 0 || lp->num_heads < 1) return S2_ERR_BAD_PARAM;
  if (head < 0 || head >= lp->num_heads || length < 1) return S2_ERR_BAD_PARAM;
  // Every block a later row keeps among blocks 0..i is also kept by row i = (length-1) div S
  // (the mask only loses columns as the row index grows: a local block drops out of the window,
  // a stripe block stays until the optional window passes it), so the answer is row i itself.
  const int i = (length - 1) / lp->block_size;
  const int64_t n = s2::row_blocks(*lp, head, i, blocks, capacity);
  *count = (int32_t)n;
  return n > capacity ? S2_ERR_OVERFLOW : S2_OK;
}

const char* s2_status_string(int status) {
  switch (status) {
    case S2_OK: return "ok";
    case S2_ERR_NULL: return "a required pointer is NULL";
    case S2_ERR_BAD_PARAM: return "parameter out of range";
    case S2_ERR_SHAPE: return "tensor shape does not fit";
    case S2_ERR_ALIGN: return "pointer or stride not aligned";
    case S2_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case S2_ERR_HIP: return "HIP runtime error";
    case S2_ERR_NO_DEVICE: return "layout has no device copy";
    case S2_ERR_OVERFLOW: return "size overflow or out of memory";
    default: return "unknown status";
  }
}

int s2_last_hip_error(void) { return g_last_hip_error; }
int s2_version(void) { return 100; }

}  // extern "C"
