// mx_abi.cpp -- host side of libmx: argument validation, batch planning,
// metadata upload and the orchestration of the gfx950 kernels behind the C ABI
// declared in include/mx.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <condition_variable>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "mx.h"
#include "mx_kernels.h"

#define MX_EXPORT extern "C" __attribute__((visibility("default")))

namespace {

using namespace mx;

thread_local std::string g_err;

mx_status fail(mx_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

mx_status hip_fail(hipError_t e, const char* what) {
  return fail(MX_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ------------------------------------------------------------------ validation
mx_status validate_shape(const mx_attn_shape* s) {
  if (!s) return fail(MX_ERR_NULL, "attention shape is NULL");
  if (s->n_q_heads <= 0 || s->n_kv_heads <= 0)
    return fail(MX_ERR_INVALID, "head counts must be positive (nq=%d, nkv=%d)", s->n_q_heads,
                s->n_kv_heads);
  if (s->n_q_heads % s->n_kv_heads != 0)
    return fail(MX_ERR_INVALID, "n_q_heads %d is not a multiple of n_kv_heads %d", s->n_q_heads,
                s->n_kv_heads);
  if (s->n_q_heads > 32767) return fail(MX_ERR_UNSUPPORTED, "more than 32767 q heads");
  if (s->head_dim != 64 && s->head_dim != 128)
    return fail(MX_ERR_UNSUPPORTED, "head_dim %d not supported (64 or 128)", s->head_dim);
  if (s->page_size != 16) return fail(MX_ERR_UNSUPPORTED, "page_size %d not supported (16)", s->page_size);
  if (s->pool_pages <= 0) return fail(MX_ERR_INVALID, "pool_pages must be positive");
  if (!(s->scale >= 0.f) || std::isinf(s->scale)) return fail(MX_ERR_INVALID, "invalid scale");
  return MX_OK;
}

// Whether the new tokens write distinct slots.  A request's new tokens fill runs
// of consecutive slots of the pages they touch, so a page and the 16-bit mask of
// the slots written in it stand for up to 16 of them: an open-addressed table of
// the touched pages, at most half full (sorting the slots instead took most of
// the host's time of a call that brings a few thousand new tokens).
bool slots_distinct(const mx_batch* b, int64_t touched) {
  if (b->num_reqs == 0) return true;
  int bits = 4;
  while (((int64_t)1 << bits) < 2 * touched) bits++;
  struct Entry {
    int32_t page;    // the page's id + 1 (0: free)
    uint32_t slots;
  };
  std::vector<Entry> table((size_t)1 << bits, Entry{0, 0});
  const size_t mask = table.size() - 1;
  for (int r = 0; r < b->num_reqs; r++) {
    const mx_request& q = b->reqs[r];
    const int end = q.ctx_len + q.n_new;
    for (int pos = q.ctx_len; pos < end;) {
      const int s0 = pos % 16, n = std::min(16 - s0, end - pos);
      const uint32_t slots = ((1u << n) - 1) << s0;
      const uint32_t key = (uint32_t)q.pages[pos / 16] + 1u;
      size_t i = (size_t)((key * 0x9E3779B97F4A7C15ull) >> (64 - bits));
      while (table[i].page != 0 && table[i].page != (int32_t)key) i = (i + 1) & mask;
      if (table[i].slots & slots) return false;
      table[i].page = (int32_t)key;
      table[i].slots |= slots;
      pos += n;
    }
  }
  return true;
}

// The error of a batch whose slots are not distinct: names the lowest one
// written twice.
mx_status duplicate_slot(const mx_batch* b, int64_t T) {
  std::vector<int64_t> slots;
  slots.reserve((size_t)T);
  for (int r = 0; r < b->num_reqs; r++)
    for (int64_t p = b->reqs[r].ctx_len, end = p + b->reqs[r].n_new; p < end; p++)
      slots.push_back((int64_t)b->reqs[r].pages[p / 16] * 16 + p % 16);
  std::sort(slots.begin(), slots.end());
  const auto it = std::adjacent_find(slots.begin(), slots.end());
  return fail(MX_ERR_INVALID, "two new tokens write the same KV slot %lld",
              it == slots.end() ? -1ll : (long long)*it);
}

mx_status validate_batch(const mx_batch* b, const mx_attn_shape* s, int64_t* T_out) {
  if (!b) return fail(MX_ERR_NULL, "batch is NULL");
  mx_status st = validate_shape(s);
  if (st != MX_OK) return st;
  if (b->num_reqs < 0) return fail(MX_ERR_INVALID, "num_reqs %d < 0", b->num_reqs);
  if (b->num_reqs > 0 && !b->reqs) return fail(MX_ERR_NULL, "reqs is NULL");
  int64_t T = 0, touched = 0;
  for (int r = 0; r < b->num_reqs; r++) {
    const mx_request& q = b->reqs[r];
    if (q.phase != MX_PREFILL && q.phase != MX_DECODE)
      return fail(MX_ERR_INVALID, "request %d: bad phase %d", r, q.phase);
    if (q.n_new < 1) return fail(MX_ERR_INVALID, "request %d: n_new %d < 1", r, q.n_new);
    if (q.ctx_len < 0) return fail(MX_ERR_INVALID, "request %d: ctx_len %d < 0", r, q.ctx_len);
    if (q.phase == MX_DECODE && (q.n_new != 1 || q.ctx_len < 1))
      return fail(MX_ERR_INVALID, "request %d: a decode needs n_new == 1 and ctx_len >= 1", r);
    const int64_t kv_len = (int64_t)q.ctx_len + q.n_new;
    if (kv_len > (int64_t)INT32_MAX - 16) return fail(MX_ERR_TOO_LARGE, "request %d: context too long", r);
    const int64_t need = ceil_div(kv_len, 16);
    if (q.n_pages < need)
      return fail(MX_ERR_NO_SPACE, "request %d: %d pages for %lld tokens (need %lld)", r, q.n_pages,
                  (long long)kv_len, (long long)need);
    if (!q.pages) return fail(MX_ERR_NULL, "request %d: pages is NULL", r);
    // one branch-free pass over the ids (a negative one is a large unsigned one)
    const uint32_t limit = (uint32_t)std::min<int64_t>(s->pool_pages, (int64_t)1 << 31);
    bool bad = s->pool_pages < 0;
    for (int i = 0; i < q.n_pages; i++) bad |= (uint32_t)q.pages[i] >= limit;
    if (bad)
      for (int i = 0; i < q.n_pages; i++)
        if (q.pages[i] < 0 || q.pages[i] >= s->pool_pages)
          return fail(MX_ERR_INVALID, "request %d: page id %d outside [0, %lld)", r, q.pages[i],
                      (long long)s->pool_pages);
    touched += (kv_len - 1) / 16 - q.ctx_len / 16 + 1;
    T += q.n_new;
    if (T > INT32_MAX / 2) return fail(MX_ERR_TOO_LARGE, "too many tokens");
  }
  if (!slots_distinct(b, touched)) return duplicate_slot(b, T);
  if (T_out) *T_out = T;
  return MX_OK;
}

mx_status validate_cfg(const mx_layer_cfg* c) {
  if (!c) return fail(MX_ERR_NULL, "layer cfg is NULL");
  mx_status st = validate_shape(&c->attn);
  if (st != MX_OK) return st;
  if (c->hidden <= 0 || c->hidden % 64)
    return fail(MX_ERR_UNSUPPORTED, "hidden %d must be a positive multiple of 64", c->hidden);
  if (c->ffn <= 0 || c->ffn % 64)
    return fail(MX_ERR_UNSUPPORTED, "ffn %d must be a positive multiple of 64", c->ffn);
  if (!(c->rms_eps >= 0.f) || !(c->rope_theta > 0.f))
    return fail(MX_ERR_INVALID, "invalid rms_eps or rope_theta");
  return MX_OK;
}

// ------------------------------------------------------------------ planning
constexpr int kXcds = 8;  // accelerator dies: workgroup b runs on die b % 8

// What a call needs to know of its batch before it lays out the workspace; the
// metadata itself is written where it goes (pack_meta).
struct Plan {
  const mx_batch* batch = nullptr;
  int R = 0, T = 0;
  std::vector<ReqDev> reqs;
  std::vector<MergeItem> merges;
  int64_t n_pages = 0, n_items = 0, n_parts = 0;
  int64_t n_tiles = 0;       // prefill tiles (work items: one per q head each)
  int split_pages = 16;
  int group = 1;
  bool has_prefill = false;  // some work item is a prefill tile
};

// Decode splits: about 1024 work items (the chip holds 512 attention
// workgroups at once), at least kMinSplitPages pages per split.
// Fewer, longer items pay the start of an item (item, request and page-table
// reads before its first keys arrive) less often, and a request that fits in
// one split needs no partials and no merge: 2048 items were 3% slower on every
// layer shape, 512 no faster.  The same holds where there is too little work
// for 1024 items: a batch whose decodes all have at most 32 pages runs them
// whole, up to 64 pages when that still is an item per CU (calls of the
// attention alone: 7B heads, one decode over 250 tokens 15.4 -> 12.4 us, 16 over
// 700 tokens 35.9 -> 32.7; Llama-3-8B heads, 32 over 300-1000: 24.7 -> 20.2; but one
// decode of 44 pages in one piece made the 7B layer 1% slower), and otherwise
// splits have at least 16 pages, not the shortest possible 8 (70B heads, 8
// decodes over 1000-2000 tokens: 18.8 -> 17.2 us).
constexpr int64_t kMinSplitPages = 16, kUnsplitPages = 32, kUnsplitPagesFull = 64, kCUs = 256;

int choose_split_pages(const mx_batch* b, const mx_attn_shape* s) {
  const int group = s->n_q_heads / s->n_kv_heads;
  const int64_t sub = s->n_kv_heads * ceil_div(group, 16);
  int64_t total = 0, longest = 0, decodes = 0;
  for (int r = 0; r < b->num_reqs; r++)
    if (b->reqs[r].phase == MX_DECODE) {
      const int64_t pages = ceil_div((int64_t)b->reqs[r].ctx_len + 1, 16);
      total += pages * sub;
      longest = std::max(longest, pages);
      decodes++;
    }
  const int64_t target_items = 1024;
  int64_t sp = ceil_div(std::max<int64_t>(total, 1), target_items);
  sp = std::max(kMinSplitPages, std::min<int64_t>(sp, 4096));
  const int64_t whole = decodes * sub >= kCUs ? kUnsplitPagesFull : kUnsplitPages;
  if (longest <= whole) sp = std::max(sp, longest);
  sp = (sp + 1) / 2 * 2;
  return (int)sp;
}

void build_plan(const mx_batch* b, const mx_attn_shape* s, bool with_items, Plan& p) {
  p.batch = b;
  p.R = b->num_reqs;
  p.group = s->n_q_heads / s->n_kv_heads;
  p.split_pages = choose_split_pages(b, s);
  p.reqs.resize(p.R);
  const int nq = s->n_q_heads;
  const int64_t sub = s->n_kv_heads * ceil_div(p.group, 16);  // decode items per split
  int tok = 0, pg = 0;
  for (int r = 0; r < p.R; r++) {
    const mx_request& q = b->reqs[r];
    ReqDev& d = p.reqs[r];
    d.tok_start = tok;
    d.n_new = q.n_new;
    d.ctx_len = q.ctx_len;
    d.kv_len = q.ctx_len + q.n_new;
    d.page_start = pg;
    d.n_pages = (int)ceil_div(d.kv_len, 16);
    d.phase = q.phase;
    d.n_split = 1;
    tok += q.n_new;
    pg += d.n_pages;
    if (!with_items) continue;
    if (d.phase == MX_PREFILL) {
      p.n_tiles += ceil_div(d.n_new, kPrefillTileRows);
    } else {
      d.n_split = (int)ceil_div(d.n_pages, p.split_pages);
      if (d.n_split > 1) {
        p.merges.push_back(MergeItem{r, (int32_t)p.n_parts});
        p.n_parts += (int64_t)nq * d.n_split;
      }
      p.n_items += d.n_split * sub;
    }
  }
  p.n_items += p.n_tiles * nq;
  p.has_prefill = p.n_tiles > 0;
  p.T = tok;
  p.n_pages = pg;
}

// The attention's work items, p.n_items of them, in launch order.
void write_items(const Plan& p, const mx_attn_shape* s, AttnItem* out) {
  const int nq = s->n_q_heads;
  // The hardware hands workgroups to free slots in list order, so the longest
  // items must not be left for the end: prefill tiles by the keys their last
  // rows scan, and the decode splits by page count, each longest first.
  struct Tile {
    int req, start, keys;
  };
  std::vector<Tile> tiles;
  tiles.reserve(p.n_tiles);
  for (int r = 0; r < p.R; r++) {
    const ReqDev& d = p.reqs[r];
    if (d.phase != MX_PREFILL) continue;
    for (int t = (d.n_new - 1) / kPrefillTileRows; t >= 0; t--) {
      const int start = t * kPrefillTileRows;
      tiles.push_back({r, start, d.ctx_len + std::min(start + kPrefillTileRows, d.n_new)});
    }
  }
  auto longer = [](const Tile& a, const Tile& b) { return a.keys > b.keys; };
  // (one prompt's tiles are generated in this order already)
  if (!std::is_sorted(tiles.begin(), tiles.end(), longer))
    std::stable_sort(tiles.begin(), tiles.end(), longer);
  auto prefill = [&](const Tile& t, int head) {
    return AttnItem{t.req, (int16_t)head, 1, 16, t.start, 0};
  };
  // Decode splits: the whole ones of every request, then the requests' last
  // parts by a stable counting sort on their page count (1 .. split_pages; a
  // last part may be whole), so equal lengths keep request, split and head order.
  const int64_t nD = p.n_items - p.n_tiles * nq;
  std::vector<AttnItem> dec(p.n_tiles ? nD : 0);
  AttnItem* dp = p.n_tiles ? dec.data() : out;
  int64_t part_base = 0;
  auto split = [&](int r, int sp, int64_t base) {
    const ReqDev& d = p.reqs[r];
    for (int g = 0; g < s->n_kv_heads; g++)
      for (int h0 = 0; h0 < p.group; h0 += 16) {
        const int head = g * p.group + h0;
        *dp++ = AttnItem{r, (int16_t)head, 0, (int8_t)std::min(16, p.group - h0),
                         sp * p.split_pages, (int32_t)(base + (int64_t)head * d.n_split + sp)};
      }
  };
  struct Last {
    int req;
    int64_t base;
  };
  std::vector<Last> last;
  std::vector<int> count(p.split_pages + 2, 0);  // by decreasing page count
  if (nD > 0) {
    std::vector<std::pair<int, Last>> unsorted;
    unsorted.reserve(p.R);
    for (int r = 0; r < p.R; r++) {
      const ReqDev& d = p.reqs[r];
      if (d.phase != MX_DECODE) continue;
      const int64_t base = d.n_split > 1 ? part_base : 0;
      const int rest = d.n_pages - (d.n_split - 1) * p.split_pages;
      const int whole = d.n_split - (rest < p.split_pages);
      for (int sp = 0; sp < whole; sp++) split(r, sp, base);
      if (rest < p.split_pages) {
        unsorted.push_back({p.split_pages - rest, Last{r, base}});
        count[p.split_pages - rest + 1]++;
      }
      if (d.n_split > 1) part_base += (int64_t)nq * d.n_split;
    }
    for (size_t i = 1; i < count.size(); i++) count[i] += count[i - 1];
    last.resize(unsorted.size());
    for (const auto& u : unsorted) last[count[u.first]++] = u.second;
    for (const Last& l : last) split(l.req, p.reqs[l.req].n_split - 1, l.base);
  }
  if (!p.n_tiles) return;
  if (nD == 0) {
    for (const Tile& t : tiles)
      for (int h = 0; h < nq; h++) *out++ = prefill(t, h);
    return;
  }
  // Prefill tiles (matrix-core bound) and decode splits (bound by HBM) are
  // interleaved in proportion to their counts, each list keeping its own
  // order: a CU then mostly holds one workgroup of each kind, whose demands
  // overlap, instead of all prefill tiles and then all decode splits.  At the
  // 70B shape with an 8192-token chunk the launch took 2.39 ms this way
  // against 2.83 ms with the prefill tiles first (and 2.85 ms with the decode
  // splits first).  The interleave runs per XCD: workgroup b runs on XCD
  // b % kXcds, so list position kXcds j + x is item j of XCD x's list, which
  // holds the prefill tiles of the KV heads h with h % kXcds == x and every
  // kXcds-th decode split.  The tiles of one KV head then read its keys and
  // values through one L2 instead of all eight, which leaves more of the
  // fabric to the decode stream beside them: the 70B launch at P = 8192 took
  // 2.10 ms against 2.24 ms with one list for all XCDs (same at P <= 4096).
  struct Lane {
    std::vector<int> heads;        // q heads of this XCD's prefill tiles
    int64_t n_pre, n_dec;          // items of either kind
    int64_t i = 0, j = 0;          // next of either
    size_t tile = 0, head = 0;     // the next prefill item
  } lane[kXcds];
  for (int h = 0; h < nq; h++) lane[(h / p.group) % kXcds].heads.push_back(h);
  int64_t longest = 0;
  for (int x = 0; x < kXcds; x++) {
    Lane& l = lane[x];
    l.n_pre = p.n_tiles * (int64_t)l.heads.size();
    l.n_dec = (nD - x + kXcds - 1) / kXcds;
    longest = std::max(longest, l.n_pre + l.n_dec);
  }
  for (int64_t k = 0; k < longest; k++)
    for (int x = 0; x < kXcds; x++) {
      Lane& l = lane[x];
      if (k >= l.n_pre + l.n_dec) continue;
      // the list that is behind in its fraction done goes next
      if (l.j >= l.n_dec ||
          (l.i < l.n_pre && (double)l.i * (double)l.n_dec <= (double)l.j * (double)l.n_pre)) {
        *out++ = prefill(tiles[l.tile], l.heads[l.head]);
        l.i++;
        if (++l.head == l.heads.size()) {
          l.head = 0;
          l.tile++;
        }
      } else {
        *out++ = dec[kXcds * l.j++ + x];
      }
    }
}

// ------------------------------------------------------------------ workspace layout
struct Layout {
  size_t reqs = 0, pages = 0, items = 0, merges = 0, meta_end = 0;
  size_t tok_req = 0, tok_pos = 0, tok_slot = 0, map_end = 0, rope_cs = 0;
  size_t part_o = 0, part_ml = 0;
  size_t h = 0, q = 0, o = 0, x1 = 0, a = 0, scratch = 0, scratch_floats = 0;
  size_t total = 0;
};

size_t gemm_scratch_bound(const mx_layer_cfg* c, int64_t T) {
  const int H = c->hidden, F = c->ffn, nq = c->attn.n_q_heads, nkv = c->attn.n_kv_heads,
            d = c->attn.head_dim;
  const int M = (int)T;
  size_t m = gemm_scratch_floats(M, (nq + 2 * nkv) * d, H);
  m = std::max(m, gemm_scratch_floats(M, H, nq * d));
  m = std::max(m, gemm_scratch_floats(M, 2 * F, H));
  m = std::max(m, gemm_scratch_floats(M, H, F));
  return m;
}

Layout make_layout(int64_t R, int64_t T, int64_t n_pages, int64_t n_items, int64_t n_merges,
                   int64_t n_parts, const mx_attn_shape* s, const mx_layer_cfg* c,
                   size_t scratch_floats) {
  Layout L;
  size_t o = 0;
  const int d = s->head_dim;
  L.reqs = o; o = align_up(o + R * sizeof(ReqDev));
  L.pages = o; o = align_up(o + n_pages * sizeof(int32_t));
  L.items = o; o = align_up(o + n_items * sizeof(AttnItem));
  L.merges = o; o = align_up(o + n_merges * sizeof(MergeItem));
  L.meta_end = o;
  L.tok_req = o; o = align_up(o + T * 4);
  L.tok_pos = o; o = align_up(o + T * 4);
  L.tok_slot = o; o = align_up(o + T * 8);
  L.map_end = o;
  L.part_o = o; o = align_up(o + n_parts * d * 4);
  L.part_ml = o; o = align_up(o + n_parts * 8);
  if (c) {
    const int64_t H = c->hidden, F = c->ffn, nq = s->n_q_heads;
    // h, o and a are projection inputs in the tile layout (whole tile rows)
    L.rope_cs = o; o = align_up(o + T * (d / 2) * 8);
    L.h = o; o = align_up(o + tile_elems(T, H) * 2);
    L.q = o; o = align_up(o + T * nq * d * 2);
    L.o = o; o = align_up(o + tile_elems(T, nq * d) * 2);
    L.x1 = o; o = align_up(o + T * H * 2);
    L.a = o; o = align_up(o + tile_elems(T, F) * 2);
    L.scratch = o; o = align_up(o + scratch_floats * 4);
    L.scratch_floats = scratch_floats;
  }
  L.total = o;
  return L;
}

Layout layout_for(const Plan& p, const mx_attn_shape* s, const mx_layer_cfg* c) {
  const size_t sc = c ? gemm_scratch_bound(c, p.T) : 0;
  return make_layout(p.R, p.T, p.n_pages, p.n_items, (int64_t)p.merges.size(), p.n_parts, s, c, sc);
}

// ------------------------------------------------------------------ per-device state
// Metadata staging: kRing pinned host buffers used in turn.  A call reserves one,
// fills it without the lock (calls of several threads plan side by side) and
// launches the kernel that reads it under the lock again (two threads, two
// streams, the host time of a call: 8B mixed 66 -> 43 us, 70B with an 8192-token
// chunk 152 -> 80; one thread 38 and 76 as before).  A buffer may be
// rewritten once that kernel (the upload, the layer's prologue or the KV append)
// has run.  A completion event costs the stream a few microseconds, so on the null
// stream one is recorded per group of up to kEvery consecutive launches, behind
// the group's last one, and covers the whole group: a group ends after kEvery
// launches, when the next launch is on another stream, or when one of its buffers
// is wanted again.  On any other stream every launch closes its own group in the
// same call: an event is never recorded on a stream the caller may have destroyed
// since (the null stream cannot be).  The event is that of the group's last
// buffer, and waiting for it frees every buffer it covers, so it is not recorded
// again while a buffer still counts on it.
struct DeviceState {
  std::mutex mu;
  std::condition_variable filled;
  bool init = false;
  static constexpr int kRing = 8;
  static constexpr int kEvery = 4;
  void* buf[kRing] = {};   // pinned host staging buffers
  void* dbuf[kRing] = {};  // the same buffers as the device reads them
  size_t cap[kRing] = {};
  hipEvent_t ev[kRing] = {};
  bool filling[kRing] = {};  // reserved by a call that has not launched yet
  bool used[kRing] = {};     // a kernel may still read it
  int cover[kRing] = {};     // used: the buffer whose event covers it (-1: in the open group)
  int next = 0;
  int open[kEvery] = {};     // the open group's buffers, in launch order
  int n_open = 0;
  hipStream_t open_stream = nullptr;
};

std::mutex g_dev_mu;
std::map<int, DeviceState*> g_devs;

mx_status device_state(DeviceState** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  DeviceState* ds;
  {
    std::lock_guard<std::mutex> g(g_dev_mu);
    auto it = g_devs.find(dev);
    if (it == g_devs.end()) {
      ds = new DeviceState();
      g_devs[dev] = ds;
    } else {
      ds = it->second;
    }
  }
  std::lock_guard<std::mutex> g(ds->mu);
  if (!ds->init) {
    e = gemm_init();
    if (e != hipSuccess) return hip_fail(e, "kernel attribute setup");
    for (int i = 0; i < DeviceState::kRing; i++) {
      e = hipEventCreateWithFlags(&ds->ev[i], hipEventDisableTiming);
      if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
    }
    ds->init = true;
  }
  *out = ds;
  return MX_OK;
}

// Records the open group's event behind its last launch; every buffer of the
// group is then covered by it.  Buffers whose event cannot be recorded are given
// up (never written or freed again): nothing would tell when their kernels are
// done.
hipError_t close_group(DeviceState* ds) {
  const int last = ds->open[ds->n_open - 1];
  const hipError_t e = hipEventRecord(ds->ev[last], ds->open_stream);
  for (int k = 0; k < ds->n_open; k++) {
    const int j = ds->open[k];
    ds->cover[j] = last;
    if (e != hipSuccess) {
      ds->buf[j] = ds->dbuf[j] = nullptr;
      ds->cap[j] = 0;
      ds->used[j] = false;
    }
  }
  ds->n_open = 0;
  return e;
}

// Reserves the next buffer that no other call is filling and waits until its
// last reader is done.
hipError_t reserve_buffer(DeviceState* ds, std::unique_lock<std::mutex>& lock, int* out) {
  int i;
  for (int k = 0;; k++) {
    if (k == DeviceState::kRing) {
      ds->filled.wait(lock);
      k = 0;
    }
    i = (ds->next + k) % DeviceState::kRing;
    if (!ds->filling[i]) break;
  }
  ds->next = (i + 1) % DeviceState::kRing;
  hipError_t e;
  if (ds->used[i] && ds->cover[i] < 0 && (e = close_group(ds)) != hipSuccess) return e;
  if (ds->used[i]) {
    const int c = ds->cover[i];
    if ((e = hipEventSynchronize(ds->ev[c])) != hipSuccess) return e;
    for (int j = 0; j < DeviceState::kRing; j++)
      if (ds->used[j] && ds->cover[j] == c) ds->used[j] = false;
  }
  ds->filling[i] = true;
  *out = i;
  return hipSuccess;
}

// Grows buffer i, which the caller has reserved, to at least `bytes`.
mx_status grow_buffer(DeviceState* ds, int i, size_t bytes) {
  if (ds->cap[i] >= bytes) return MX_OK;
  hipError_t e;
  if (ds->buf[i]) {
    e = hipHostFree(ds->buf[i]);
    ds->buf[i] = ds->dbuf[i] = nullptr;
    ds->cap[i] = 0;
    if (e != hipSuccess) return hip_fail(e, "hipHostFree");
  }
  const size_t cap = std::max<size_t>(bytes * 2, 1 << 16);
  e = hipHostMalloc(&ds->buf[i], cap, hipHostMallocMapped);
  if (e != hipSuccess) {
    ds->buf[i] = nullptr;
    return hip_fail(e, "hipHostMalloc");
  }
  e = hipHostGetDevicePointer(&ds->dbuf[i], ds->buf[i], 0);
  if (e != hipSuccess) {
    (void)hipHostFree(ds->buf[i]);  // the lookup's error is the one reported
    ds->buf[i] = ds->dbuf[i] = nullptr;
    return hip_fail(e, "hipHostGetDevicePointer");
  }
  ds->cap[i] = cap;
  return MX_OK;
}

// Rotary inverse frequencies theta^(-2 k / d), k < d / 2 (the last pair of
// (theta, d) is kept per thread: the powers cost as much as a launch).
const RopeFreqs& rope_freqs(float theta, int d) {
  thread_local float last_theta = 0.f;
  thread_local int last_d = 0;
  thread_local RopeFreqs f;
  if (theta != last_theta || d != last_d) {
    for (int k = 0; k < d / 2; k++) f.inv[k] = std::pow((double)theta, -2.0 * k / d);
    last_theta = theta;
    last_d = d;
  }
  return f;
}

// The token map of the batch: request, position and KV slot of every new token.
void pack_token_map(const Plan& p, const Layout& L, char* h) {
  int32_t* req = (int32_t*)(h + L.tok_req);
  int32_t* pos = (int32_t*)(h + L.tok_pos);
  int64_t* slot = (int64_t*)(h + L.tok_slot);
  for (int r = 0; r < p.R; r++) {
    const mx_request& q = p.batch->reqs[r];
    const int end = q.ctx_len + q.n_new;
    for (int i = q.ctx_len; i < end; i++) {
      *req++ = r;
      *pos++ = i;
      *slot++ = (int64_t)q.pages[i / 16] * 16 + i % 16;
    }
  }
}

// The metadata block [0, L.meta_end) of the workspace, as the kernels read it:
// request records, page tables, attention work items, merge items (the gaps
// between them are never read); the work items from `items` where they are given.
void pack_meta(const Plan& p, const Layout& L, const mx_attn_shape* s, char* h,
               const AttnItem* items = nullptr) {
  if (!p.reqs.empty()) memcpy(h + L.reqs, p.reqs.data(), p.reqs.size() * sizeof(ReqDev));
  int32_t* pages = (int32_t*)(h + L.pages);
  for (int r = 0; r < p.R; r++)
    memcpy(pages + p.reqs[r].page_start, p.batch->reqs[r].pages,
           (size_t)p.reqs[r].n_pages * sizeof(int32_t));
  if (items)
    memcpy(h + L.items, items, p.n_items * sizeof(AttnItem));
  else if (p.n_items)
    write_items(p, s, (AttnItem*)(h + L.items));
  if (!p.merges.empty()) memcpy(h + L.merges, p.merges.data(), p.merges.size() * sizeof(MergeItem));
}

// Runs pack(host) on a staging buffer of at least `bytes` and launch(device
// view of it), a kernel on `stream` that reads the buffer, under the ring's
// discipline.
template <typename Pack, typename Launch>
mx_status staged(size_t bytes, hipStream_t stream, Pack&& pack, Launch&& launch) {
  DeviceState* ds;
  mx_status st = device_state(&ds);
  if (st != MX_OK) return st;
  std::unique_lock<std::mutex> lock(ds->mu);
  int i;
  hipError_t e = reserve_buffer(ds, lock, &i);
  if (e != hipSuccess) return hip_fail(e, "staging buffer event");
  struct Reservation {  // given back on every way out
    DeviceState* ds;
    std::unique_lock<std::mutex>& lock;
    int i;
    ~Reservation() {
      if (!lock.owns_lock()) lock.lock();
      ds->filling[i] = false;
      ds->filled.notify_one();
    }
  } reservation{ds, lock, i};
  lock.unlock();
  if ((st = grow_buffer(ds, i, bytes)) != MX_OK) return st;
  pack((char*)ds->buf[i]);
  lock.lock();
  // the open group is on another stream: close it there first
  if (ds->n_open > 0 && ds->open_stream != stream && (e = close_group(ds)) != hipSuccess)
    return hip_fail(e, "hipEventRecord");
  // from here on the kernel may read the buffer, also where launch reports an
  // error (of the timing events around it, for one): the buffer joins a group first
  ds->used[i] = true;
  ds->cover[i] = -1;
  ds->open[ds->n_open++] = i;
  ds->open_stream = stream;
  const hipError_t launched = launch(ds->dbuf[i]);
  if (stream != nullptr || ds->n_open == DeviceState::kEvery) e = close_group(ds);
  if (launched != hipSuccess) return hip_fail(launched, "metadata launch");
  if (e != hipSuccess) return hip_fail(e, "hipEventRecord");
  return MX_OK;
}

mx_status upload_meta(const Plan& p, const Layout& L, const mx_attn_shape* s, void* ws,
                      hipStream_t stream) {
  return staged(
      L.meta_end, stream, [&](char* h) { pack_meta(p, L, s, h); },
      [&](const void* dev) { return launch_upload(dev, ws, L.meta_end, stream); });
}

template <typename T>
T* at(void* ws, size_t off) { return reinterpret_cast<T*>((char*)ws + off); }

float eff_scale(const mx_attn_shape* s) {
  return s->scale > 0.f ? s->scale : 1.0f / std::sqrt((float)s->head_dim);
}

AttnParams attn_params(const Plan& p, const Layout& L, const mx_attn_shape* s, void* ws,
                       const uint16_t* q, int64_t q_stride, const uint16_t* kp,
                       const uint16_t* vp, uint16_t* out) {
  AttnParams a;
  a.q = q;
  a.q_tok_stride = q_stride;
  a.k_pool = kp;
  a.v_pool = vp;
  a.out = out;
  a.out_tok_stride = (int64_t)s->n_q_heads * s->head_dim;
  a.out_tiled = 0;
  a.reqs = at<ReqDev>(ws, L.reqs);
  a.pages = at<int32_t>(ws, L.pages);
  a.items = at<AttnItem>(ws, L.items);
  a.part_o = at<float>(ws, L.part_o);
  a.part_ml = at<float>(ws, L.part_ml);
  a.nq = s->n_q_heads;
  a.nkv = s->n_kv_heads;
  a.group = p.group;
  a.split_pages = p.split_pages;
  a.scale_log2 = eff_scale(s) * 1.4426950408889634f;
  a.decode_only = p.has_prefill ? 0 : 1;
  return a;
}

// packed weight regions
struct WLayout {
  size_t g1, qkv, o, g2, gu, down, total;
};
WLayout wlayout(const mx_layer_cfg* c) {
  const size_t H = c->hidden, F = c->ffn, nq = c->attn.n_q_heads, nkv = c->attn.n_kv_heads,
               d = c->attn.head_dim;
  WLayout w;
  size_t o = 0;
  w.g1 = o; o = align_up(o + H * 2);
  w.qkv = o; o = align_up(o + (nq + 2 * nkv) * d * H * 2);
  w.o = o; o = align_up(o + H * nq * d * 2);
  w.g2 = o; o = align_up(o + H * 2);
  w.gu = o; o = align_up(o + 2 * F * H * 2);
  w.down = o; o = align_up(o + H * F * 2);
  w.total = o;
  return w;
}

// ------------------------------------------------------------------ launch timing
// Optional per-launch timing (hipEvents recorded on the caller's stream around
// each kernel launch).  Off by default; costs two event records per launch.
struct Profiler {
  std::mutex mu;
  bool on = false;
  struct Rec {
    const char* name;
    hipEvent_t a, b;
  };
  std::vector<Rec> pending;
  std::vector<hipEvent_t> free_events;
  std::vector<const char*> names;
  std::vector<double> total_ms;
  std::vector<int> counts;

  hipEvent_t get() {
    if (!free_events.empty()) {
      hipEvent_t e = free_events.back();
      free_events.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
};
Profiler g_prof;

template <typename F>
hipError_t timed(const char* name, hipStream_t stream, F&& launch) {
  bool on;
  {
    std::lock_guard<std::mutex> g(g_prof.mu);
    on = g_prof.on;
  }
  if (!on) return launch();
  hipEvent_t a, b;
  {
    std::lock_guard<std::mutex> g(g_prof.mu);
    a = g_prof.get();
    b = g_prof.get();
  }
  if (!a || !b) return launch();
  hipError_t e = hipEventRecord(a, stream);
  if (e != hipSuccess) return e;
  e = launch();
  if (e != hipSuccess) return e;
  e = hipEventRecord(b, stream);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> g(g_prof.mu);
  g_prof.pending.push_back({name, a, b});
  return hipSuccess;
}

}  // namespace

// ======================================================================= ABI
MX_EXPORT const char* mx_status_str(mx_status s) {
  switch (s) {
    case MX_OK: return "MX_OK";
    case MX_ERR_INVALID: return "MX_ERR_INVALID";
    case MX_ERR_NO_SPACE: return "MX_ERR_NO_SPACE";
    case MX_ERR_TOO_LARGE: return "MX_ERR_TOO_LARGE";
    case MX_ERR_UNSUPPORTED: return "MX_ERR_UNSUPPORTED";
    case MX_ERR_NULL: return "MX_ERR_NULL";
    case MX_ERR_HIP: return "MX_ERR_HIP";
  }
  return "MX_ERR_UNKNOWN";
}

MX_EXPORT const char* mx_last_error(void) { return g_err.c_str(); }

MX_EXPORT uint32_t mx_version(void) { return (1u << 16) | 0u; }

// Device tensors are read and written with 16-byte vector accesses.
static mx_status check_aligned(std::initializer_list<const void*> ptrs) {
  for (const void* q : ptrs)
    if ((uintptr_t)q & 15) return fail(MX_ERR_INVALID, "device pointer %p is not 16-byte aligned", q);
  return MX_OK;
}

MX_EXPORT mx_status mx_batch_validate(const mx_batch* batch, const mx_attn_shape* shape) {
  g_err.clear();
  return validate_batch(batch, shape, nullptr);
}

MX_EXPORT size_t mx_workspace_bytes_for(const mx_batch* batch, const mx_attn_shape* shape,
                                        const mx_layer_cfg* cfg) {
  g_err.clear();
  if (cfg) {
    if (validate_cfg(cfg) != MX_OK) return 0;
    shape = &cfg->attn;
  }
  if (validate_batch(batch, shape, nullptr) != MX_OK) return 0;
  Plan p;
  build_plan(batch, shape, true, p);
  return layout_for(p, shape, cfg).total;
}

MX_EXPORT size_t mx_workspace_bytes(const mx_layer_cfg* cfg, const mx_attn_shape* shape,
                                    int32_t max_tokens, int32_t max_reqs, int64_t max_pages) {
  g_err.clear();
  if (cfg) {
    if (validate_cfg(cfg) != MX_OK) return 0;
    shape = &cfg->attn;
  } else if (validate_shape(shape) != MX_OK) {
    return 0;
  }
  if (max_tokens < 0 || max_reqs < 0 || max_pages < 0) {
    fail(MX_ERR_INVALID, "negative bound");
    return 0;
  }
  const int64_t nq = shape->n_q_heads, nkv = shape->n_kv_heads, group = nq / nkv;
  // every split but a request's last has at least kMinSplitPages (more than 8)
  // pages, so splits <= pages / 8 + requests
  const int64_t splits = max_pages / 8 + max_reqs;
  const int64_t items =
      splits * nkv * ceil_div(group, 16) + (max_tokens / kPrefillTileRows + max_reqs) * nq;
  const int64_t parts = splits * nq;
  const size_t scratch = cfg ? kMaxSplitFloats : 0;
  return make_layout(max_reqs, max_tokens, max_pages, items, max_reqs, parts, shape, cfg, scratch)
      .total;
}

MX_EXPORT size_t mx_packed_weights_bytes(const mx_layer_cfg* cfg) {
  g_err.clear();
  if (validate_cfg(cfg) != MX_OK) return 0;
  return wlayout(cfg).total;
}

MX_EXPORT mx_status mx_pack_weights(const mx_layer_cfg* cfg, const mx_layer_weights* w,
                                    void* packed, size_t packed_bytes, hipStream_t stream) {
  g_err.clear();
  mx_status st = validate_cfg(cfg);
  if (st != MX_OK) return st;
  if (!w || !packed || !w->ln1_g || !w->w_qkv || !w->w_o || !w->ln2_g || !w->w_gate_up || !w->w_down)
    return fail(MX_ERR_NULL, "weight pointer is NULL");
  if ((st = check_aligned({packed, w->ln1_g, w->w_qkv, w->w_o, w->ln2_g, w->w_gate_up, w->w_down})) !=
      MX_OK)
    return st;
  const WLayout L = wlayout(cfg);
  if (packed_bytes < L.total)
    return fail(MX_ERR_TOO_LARGE, "packed buffer %zu bytes < %zu", packed_bytes, L.total);
  DeviceState* ds;
  st = device_state(&ds);
  if (st != MX_OK) return st;
  const size_t H = cfg->hidden, F = cfg->ffn, nq = cfg->attn.n_q_heads,
               nkv = cfg->attn.n_kv_heads, d = cfg->attn.head_dim;
  char* P = (char*)packed;
  hipError_t e;
#define MX_CP(off, src, bytes)                                                        \
  e = hipMemcpyAsync(P + (off), (src), (bytes), hipMemcpyDeviceToDevice, stream);    \
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync (pack)");
  MX_CP(L.g1, w->ln1_g, H * 2)
  MX_CP(L.g2, w->ln2_g, H * 2)
#undef MX_CP
  // the four matrices in the GEMMs' tiled layout (row permutation applied on the way)
#define MX_TILE(off, src, N, K, kind, what)                                                      \
  e = launch_pack_tiled((src), (uint16_t*)(P + (off)), (int)(N), (int)(K), (kind), (int)nq,      \
                        (int)nkv, (int)d, (int)F, stream);                                       \
  if (e != hipSuccess) return hip_fail(e, what);
  MX_TILE(L.qkv, w->w_qkv, (nq + 2 * nkv) * d, H, 1, "qkv packing launch")
  MX_TILE(L.o, w->w_o, H, nq * d, 0, "o packing launch")
  MX_TILE(L.gu, w->w_gate_up, 2 * F, H, 2, "gate/up packing launch")
  MX_TILE(L.down, w->w_down, H, F, 0, "down packing launch")
#undef MX_TILE
  return MX_OK;
}

static mx_status check_ws(const Layout& L, void* ws, size_t ws_bytes) {
  if (!ws) return fail(MX_ERR_NULL, "workspace is NULL");
  if (ws_bytes < L.total)
    return fail(MX_ERR_TOO_LARGE, "workspace %zu bytes < %zu needed", ws_bytes, L.total);
  return MX_OK;
}

MX_EXPORT mx_status mx_kv_append(const mx_batch* batch, const mx_attn_shape* shape,
                                 const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool,
                                 uint16_t* v_pool, void* ws, size_t ws_bytes, hipStream_t stream) {
  g_err.clear();
  int64_t T;
  mx_status st = validate_batch(batch, shape, &T);
  if (st != MX_OK) return st;
  if (T == 0) return MX_OK;
  if (!k_new || !v_new || !k_pool || !v_pool) return fail(MX_ERR_NULL, "tensor pointer is NULL");
  if ((st = check_aligned({k_new, v_new, k_pool, v_pool, ws})) != MX_OK) return st;
  // one run per page that a request's new tokens touch
  int64_t n_pages = 0, n_runs = 0;
  for (int r = 0; r < batch->num_reqs; r++) {
    const mx_request& q = batch->reqs[r];
    n_pages += ceil_div((int64_t)q.ctx_len + q.n_new, 16);
    n_runs += (q.ctx_len + q.n_new - 1) / 16 - q.ctx_len / 16 + 1;
  }
  const Layout L = make_layout(batch->num_reqs, T, n_pages, 0, 0, 0, shape, nullptr, 0);
  if ((st = check_ws(L, ws, ws_bytes)) != MX_OK) return st;
  return staged(
      n_runs * sizeof(AppendRun), stream,
      [&](char* h) {
        AppendRun* run = reinterpret_cast<AppendRun*>(h);
        int32_t tok = 0;
        for (int r = 0; r < batch->num_reqs; r++) {
          const mx_request& q = batch->reqs[r];
          const int end = q.ctx_len + q.n_new;
          for (int pos = q.ctx_len; pos < end;) {
            const int n = std::min(16 - pos % 16, end - pos);
            *run++ = AppendRun{tok, n, (int64_t)q.pages[pos / 16] * 16 + pos % 16};
            tok += n;
            pos += n;
          }
        }
      },
      [&](const void* dev) {
        return launch_kv_append(k_new, v_new, k_pool, v_pool, static_cast<const AppendRun*>(dev),
                                n_runs, shape->n_kv_heads, shape->head_dim, stream);
      });
}

MX_EXPORT mx_status mx_paged_attn(const mx_batch* batch, const mx_attn_shape* shape,
                                  const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool,
                                  uint16_t* out, void* ws, size_t ws_bytes, hipStream_t stream) {
  g_err.clear();
  int64_t T;
  mx_status st = validate_batch(batch, shape, &T);
  if (st != MX_OK) return st;
  if (T == 0) return MX_OK;
  if (!q || !k_pool || !v_pool || !out) return fail(MX_ERR_NULL, "tensor pointer is NULL");
  if ((st = check_aligned({q, k_pool, v_pool, out, ws})) != MX_OK) return st;
  Plan p;
  build_plan(batch, shape, true, p);
  const Layout L = layout_for(p, shape, nullptr);
  if ((st = check_ws(L, ws, ws_bytes)) != MX_OK) return st;
  if ((st = upload_meta(p, L, shape, ws, stream)) != MX_OK) return st;
  AttnParams a = attn_params(p, L, shape, ws, q, (int64_t)shape->n_q_heads * shape->head_dim,
                             k_pool, v_pool, out);
  hipError_t e = timed("paged_attn", stream, [&] {
    return launch_paged_attn(a, (int)p.n_items, at<MergeItem>(ws, L.merges),
                             (int)p.merges.size(), shape->head_dim, stream);
  });
  if (e != hipSuccess) return hip_fail(e, "attention launch");
  return MX_OK;
}

// ------------------------------------------------------------------ static scratch
// Device memory of mx_paged_attn_static: the metadata block and the split
// partials of one call, in a file-scope array of kStaticScratchBytes that
// every GPU the library runs on holds until the process ends.  Host code uses
// the array only through the device address hipGetSymbolAddress returns for
// the current device (the array's name is a host-side stand-in, not a device
// address); the address is taken once per device, on the entry point's first
// call there, and kept.
constexpr size_t kStaticScratchBytes = size_t(32) << 20;
static __device__ __align__(256) char scratch[kStaticScratchBytes];

std::mutex g_scratch_mu;
std::map<int, void*> g_scratch_ptr;

// Host side of the same calls: the metadata block is packed into this
// file-scope buffer (no allocation per call) and copied from it with
// hipMemcpyAsync.  From pageable memory HIP performs that copy synchronously
// (the source has been read when the call returns), so the buffer is free
// again on return; the lock keeps the calls of different threads apart while
// they pack and copy.
std::mutex g_static_host_mu;
alignas(64) char g_static_host[kStaticScratchBytes];

mx_status static_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::lock_guard<std::mutex> g(g_scratch_mu);
  auto it = g_scratch_ptr.find(dev);
  if (it != g_scratch_ptr.end()) {
    *out = it->second;
    return MX_OK;
  }
  void* ptr = nullptr;
  e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress (static scratch)");
  if (!ptr) return fail(MX_ERR_HIP, "hipGetSymbolAddress returned NULL for the static scratch");
  g_scratch_ptr[dev] = ptr;
  *out = ptr;
  return MX_OK;
}

MX_EXPORT size_t mx_paged_attn_static_max_bytes(void) { return kStaticScratchBytes; }

MX_EXPORT mx_status mx_paged_attn_static(const mx_batch* batch, const mx_attn_shape* shape,
                                         const uint16_t* q, const uint16_t* k_pool,
                                         const uint16_t* v_pool, uint16_t* out,
                                         hipStream_t stream) {
  g_err.clear();
  int64_t T;
  mx_status st = validate_batch(batch, shape, &T);
  if (st != MX_OK) return st;
  if (T == 0) return MX_OK;
  if (!q || !k_pool || !v_pool || !out) return fail(MX_ERR_NULL, "tensor pointer is NULL");
  if ((st = check_aligned({q, k_pool, v_pool, out})) != MX_OK) return st;
  Plan p;
  build_plan(batch, shape, true, p);
  const Layout L = layout_for(p, shape, nullptr);
  if (L.total > kStaticScratchBytes)
    return fail(MX_ERR_TOO_LARGE,
                "batch needs %zu bytes of scratch; the static scratch holds %zu (use mx_paged_attn "
                "with a workspace)",
                L.total, kStaticScratchBytes);
  void* ws = nullptr;
  if ((st = static_scratch(&ws)) != MX_OK) return st;
  // the metadata block, packed on the host and copied into the scratch in
  // stream order (nothing in the scratch needs to start at zero: every split
  // partial is written by its item before the merge reads it)
  hipError_t e;
  std::vector<AttnItem> items(p.n_items);  // listed before the lock is taken
  write_items(p, shape, items.data());
  {
    std::lock_guard<std::mutex> g(g_static_host_mu);
    pack_meta(p, L, shape, g_static_host, items.data());  // L.meta_end <= L.total, checked above
    e = hipMemcpyAsync(ws, g_static_host, L.meta_end, hipMemcpyHostToDevice, stream);
  }
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync (metadata)");
  AttnParams a = attn_params(p, L, shape, ws, q, (int64_t)shape->n_q_heads * shape->head_dim,
                             k_pool, v_pool, out);
  e = timed("paged_attn", stream, [&] {
    return launch_paged_attn(a, (int)p.n_items, at<MergeItem>(ws, L.merges),
                             (int)p.merges.size(), shape->head_dim, stream);
  });
  if (e != hipSuccess) return hip_fail(e, "attention launch");
  return MX_OK;
}

MX_EXPORT mx_status mx_layer_step(const mx_batch* batch, const mx_layer_cfg* cfg,
                                  const void* packed_weights, const uint16_t* x, uint16_t* y,
                                  uint16_t* k_pool, uint16_t* v_pool, void* ws, size_t ws_bytes,
                                  hipStream_t stream) {
  g_err.clear();
  mx_status st = validate_cfg(cfg);
  if (st != MX_OK) return st;
  const mx_attn_shape* s = &cfg->attn;
  int64_t T;
  if ((st = validate_batch(batch, s, &T)) != MX_OK) return st;
  if (T == 0) return MX_OK;
  if (!packed_weights || !x || !y || !k_pool || !v_pool)
    return fail(MX_ERR_NULL, "tensor pointer is NULL");
  if (x == y) return fail(MX_ERR_INVALID, "y must not alias x");
  if ((st = check_aligned({packed_weights, x, y, k_pool, v_pool, ws})) != MX_OK) return st;
  Plan p;
  build_plan(batch, s, true, p);
  const Layout L = layout_for(p, s, cfg);
  if ((st = check_ws(L, ws, ws_bytes)) != MX_OK) return st;
  const WLayout W = wlayout(cfg);
  const char* P = (const char*)packed_weights;
  const int H = cfg->hidden, F = cfg->ffn, nq = s->n_q_heads, nkv = s->n_kv_heads,
            d = s->head_dim;
  const int Nqkv = (nq + 2 * nkv) * d;
  const int M = p.T;
  uint16_t* h = at<uint16_t>(ws, L.h);
  uint16_t* q = at<uint16_t>(ws, L.q);
  uint16_t* o = at<uint16_t>(ws, L.o);
  uint16_t* x1 = at<uint16_t>(ws, L.x1);
  uint16_t* act = at<uint16_t>(ws, L.a);
  float* scratch = at<float>(ws, L.scratch);
  float2* rope_cs = at<float2>(ws, L.rope_cs);
  hipError_t e;
#define MX_CK(call, what) \
  if ((e = (call)) != hipSuccess) return hip_fail(e, what);
  // a0-a2: metadata upload (the token map in it), rotary table and RMSNorm 1, in
  // one launch
  st = staged(
      L.map_end, stream,
      [&](char* b) {
        pack_meta(p, L, s, b);
        pack_token_map(p, L, b);
      },
      [&](const void* dev) {
        return timed("token_map+rmsnorm_1", stream, [&] {
          return launch_prologue(dev, ws, L.map_end, (const int32_t*)((const char*)dev + L.tok_pos),
                                 p.T, rope_freqs(cfg->rope_theta, d), rope_cs, d / 2, x,
                                 (const uint16_t*)(P + W.g1), h, H, cfg->rms_eps, stream);
        });
      });
  if (st != MX_OK) return st;
  // a3-a5: QKV projection with RoPE and the KV append fused into its epilogue
  {
    GemmArgs g{h, (const uint16_t*)(P + W.qkv), nullptr, nullptr, scratch, M, Nqkv, H, H, H, 0, 0, EPI_QKV,
               QkvEpilogue{rope_cs, at<int64_t>(ws, L.tok_slot), q, k_pool, v_pool, nq, nkv, d}};
    set_b_tiled(g);
    g.a_tiled = 1;
    MX_CK(timed("gemm_qkv", stream, [&] { return launch_gemm(g, L.scratch_floats, stream); }),
          "qkv gemm launch")
  }
  // a6: paged attention, prefill and decode rows in one launch (+ split merge)
  {
    AttnParams a = attn_params(p, L, s, ws, q, (int64_t)nq * d, k_pool, v_pool, o);
    a.out_tiled = 1;  // o feeds the output projection
    MX_CK(timed("paged_attn", stream, [&] {
            return launch_paged_attn(a, (int)p.n_items, at<MergeItem>(ws, L.merges),
                                     (int)p.merges.size(), d, stream);
          }), "attention launch")
  }
  // a7 + a8: output projection + residual, then RMSNorm 2.  When (some rows
  // of) the projection are split over K, their reduce, the residual and the
  // norm of every row run as one kernel (timed as o_reduce+rmsnorm_2), which
  // reads the fp32 planes once and keeps each x1 row in registers for the norm.
  {
    GemmArgs g{o, (const uint16_t*)(P + W.o), x1, x, scratch, M, H, nq * d, nq * d, nq * d, H, H, EPI_RESIDUAL, {}};
    set_b_tiled(g);
    g.a_tiled = 1;
    const uint16_t* g2 = (const uint16_t*)(P + W.g2);
    const bool fuse = H <= kFusedNormMaxH;  // the fused kernel holds a row in registers
    int split_row = M, ks = 1;
    MX_CK(timed("gemm_o", stream, [&] {
            return fuse ? launch_gemm_unreduced(g, L.scratch_floats, &split_row, &ks, stream)
                        : launch_gemm(g, L.scratch_floats, stream);
          }), "o gemm launch")
    MX_CK(timed(ks > 1 ? "o_reduce+rmsnorm_2" : "rmsnorm_2", stream, [&] {
            return ks > 1 ? launch_reduce_residual_rmsnorm(scratch, ks, x, x1, g2, h, M, H,
                                                           cfg->rms_eps, split_row, stream)
                          : launch_rmsnorm(x1, g2, h, M, H, cfg->rms_eps, stream);
          }), "rmsnorm launch")
  }
  // a9: gate/up projection + SwiGLU
  {
    GemmArgs g{h, (const uint16_t*)(P + W.gu), act, nullptr, scratch, M, 2 * F, H, H, H, F, 0, EPI_SWIGLU, {}};
    set_b_tiled(g);
    g.a_tiled = 1;
    g.c_tiled = 1;  // act feeds the down projection
    MX_CK(timed("gemm_gate_up", stream, [&] { return launch_gemm(g, L.scratch_floats, stream); }),
          "gate/up gemm launch")
  }
  // a10: down projection + residual
  {
    GemmArgs g{act, (const uint16_t*)(P + W.down), y, x1, scratch, M, H, F, F, F, H, H, EPI_RESIDUAL, {}};
    set_b_tiled(g);
    g.a_tiled = 1;
    MX_CK(timed("gemm_down", stream, [&] { return launch_gemm(g, L.scratch_floats, stream); }),
          "down gemm launch")
  }
#undef MX_CK
  return MX_OK;
}

MX_EXPORT mx_status mx_layer_workspace_offsets(const mx_batch* batch, const mx_layer_cfg* cfg,
                                               size_t off[5]) {
  g_err.clear();
  mx_status st = validate_cfg(cfg);
  if (st != MX_OK) return st;
  if ((st = validate_batch(batch, &cfg->attn, nullptr)) != MX_OK) return st;
  if (!off) return fail(MX_ERR_NULL, "off is NULL");
  Plan p;
  build_plan(batch, &cfg->attn, true, p);
  const Layout L = layout_for(p, &cfg->attn, cfg);
  off[0] = L.h;
  off[1] = L.q;
  off[2] = L.o;
  off[3] = L.x1;
  off[4] = L.a;
  return MX_OK;
}

MX_EXPORT mx_status mx_debug_token_map(const mx_batch* batch, const mx_attn_shape* shape,
                                       int32_t* tok_req, int32_t* tok_pos, int64_t* tok_slot,
                                       void* ws, size_t ws_bytes, hipStream_t stream) {
  g_err.clear();
  int64_t T;
  mx_status st = validate_batch(batch, shape, &T);
  if (st != MX_OK) return st;
  if (T == 0) return MX_OK;
  if (!tok_req || !tok_pos || !tok_slot) return fail(MX_ERR_NULL, "output pointer is NULL");
  Plan p;
  build_plan(batch, shape, false, p);
  const Layout L = layout_for(p, shape, nullptr);
  if ((st = check_ws(L, ws, ws_bytes)) != MX_OK) return st;
  st = staged(
      L.map_end, stream,
      [&](char* h) {
        pack_meta(p, L, shape, h);
        pack_token_map(p, L, h);
      },
      [&](const void* dev) { return launch_upload(dev, ws, L.map_end, stream); });
  if (st != MX_OK) return st;
  hipError_t e;
  e = hipMemcpyAsync(tok_req, at<int32_t>(ws, L.tok_req), T * 4, hipMemcpyDeviceToDevice, stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(tok_pos, at<int32_t>(ws, L.tok_pos), T * 4, hipMemcpyDeviceToDevice, stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(tok_slot, at<int64_t>(ws, L.tok_slot), T * 8, hipMemcpyDeviceToDevice, stream);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync (token map)");
  return MX_OK;
}

MX_EXPORT mx_status mx_debug_gather(const mx_batch* batch, const mx_attn_shape* shape, int32_t req,
                                    const uint16_t* k_pool, const uint16_t* v_pool,
                                    uint16_t* k_out, uint16_t* v_out, void* ws, size_t ws_bytes,
                                    hipStream_t stream) {
  g_err.clear();
  mx_status st = validate_batch(batch, shape, nullptr);
  if (st != MX_OK) return st;
  if (req < 0 || req >= batch->num_reqs) return fail(MX_ERR_INVALID, "request %d out of range", req);
  if (!k_pool || !v_pool || !k_out || !v_out) return fail(MX_ERR_NULL, "tensor pointer is NULL");
  Plan p;
  build_plan(batch, shape, false, p);
  const Layout L = layout_for(p, shape, nullptr);
  if ((st = check_ws(L, ws, ws_bytes)) != MX_OK) return st;
  if ((st = upload_meta(p, L, shape, ws, stream)) != MX_OK) return st;
  const ReqDev& rq = p.reqs[req];
  hipError_t e = launch_gather(k_pool, v_pool, at<int32_t>(ws, L.pages) + rq.page_start, rq.kv_len,
                               shape->n_kv_heads, shape->head_dim, k_out, v_out, stream);
  if (e != hipSuccess) return hip_fail(e, "gather launch");
  return MX_OK;
}

MX_EXPORT size_t mx_debug_gemm_ws_bytes(int32_t M, int32_t N, int32_t K) {
  if (M < 0 || N <= 0 || K <= 0) return 0;
  return align_up(gemm_scratch_floats(M, N, K) * 4 + 4);
}

MX_EXPORT mx_status mx_debug_gemm(int32_t M, int32_t N, int32_t K, const uint16_t* A,
                                  const uint16_t* B, uint16_t* C, const uint16_t* R,
                                  int32_t epilogue, void* ws, size_t ws_bytes, hipStream_t stream) {
  return mx_debug_gemm_config(M, N, K, A, B, C, R, epilogue, -1, 0, ws, ws_bytes, stream);
}

namespace {
mx_status debug_gemm(int32_t M, int32_t N, int32_t K, const uint16_t* A, const uint16_t* B,
                     bool b_tiled, uint16_t* C, const uint16_t* R, int32_t epilogue,
                     int32_t tile_cfg, int32_t ksplit, void* ws, size_t ws_bytes,
                     hipStream_t stream) {
  g_err.clear();
  if (b_tiled && (N % 16 || K % 32))
    return fail(MX_ERR_UNSUPPORTED, "tiled weights need N %% 16 == 0 and K %% 32 == 0");
  if (M < 0 || N <= 0 || K <= 0) return fail(MX_ERR_INVALID, "bad GEMM shape %d x %d x %d", M, N, K);
  if (K % 64) return fail(MX_ERR_UNSUPPORTED, "K %d is not a multiple of 64", K);
  if (tile_cfg < -1 || tile_cfg >= gemm_num_configs())
    return fail(MX_ERR_INVALID, "tile config %d out of range", tile_cfg);
  if (tile_cfg >= 0 && (ksplit < 1 || ksplit > 64 || K / 64 < ksplit))
    return fail(MX_ERR_INVALID, "K split %d is not in [1, min(64, K / 64 = %d)]", ksplit, K / 64);
  if (epilogue < 0 || epilogue > 2) return fail(MX_ERR_INVALID, "bad epilogue %d", epilogue);
  if (epilogue == EPI_SWIGLU && N % 64) return fail(MX_ERR_UNSUPPORTED, "SwiGLU needs N % 64 == 0");
  if (M == 0) return MX_OK;
  if (!A || !B || !C || (epilogue == EPI_RESIDUAL && !R)) return fail(MX_ERR_NULL, "NULL operand");
  if (mx_status sa = check_aligned({A, B, C, R, ws}); sa != MX_OK) return sa;
  if (epilogue == EPI_RESIDUAL) {
    const size_t bytes = (size_t)M * N * 2;  // C and R are both [M][N]
    const char *c0 = (const char*)C, *r0 = (const char*)R;
    if (c0 < r0 + bytes && r0 < c0 + bytes) return fail(MX_ERR_INVALID, "R overlaps C");
  }
  const size_t need = tile_cfg >= 0 ? (ksplit > 1 ? (size_t)ksplit * M * N : 0)
                                    : gemm_scratch_floats(M, N, K);
  if (need && (!ws || ws_bytes < need * 4))
    return fail(MX_ERR_TOO_LARGE, "GEMM scratch %zu bytes < %zu", ws_bytes, need * 4);
  DeviceState* ds;
  mx_status st = device_state(&ds);
  if (st != MX_OK) return st;
  const int ldc = epilogue == EPI_SWIGLU ? N / 2 : N;
  GemmArgs g{A, B, C, R, (float*)ws, M, N, K, K, K, ldc, N, epilogue, {}};
  if (b_tiled) {  // the layer step's operand layouts
    set_b_tiled(g);
    g.a_tiled = 1;
    g.c_tiled = epilogue == EPI_SWIGLU;
  } else {
    set_b_row_major(g);
  }
  hipError_t e = launch_gemm_config(g, ws ? ws_bytes / 4 : 0, tile_cfg, ksplit, stream);
  if (e != hipSuccess) return hip_fail(e, "gemm launch");
  return MX_OK;
}
}  // namespace

MX_EXPORT mx_status mx_debug_gemm_config(int32_t M, int32_t N, int32_t K, const uint16_t* A,
                                         const uint16_t* B, uint16_t* C, const uint16_t* R,
                                         int32_t epilogue, int32_t tile_cfg, int32_t ksplit,
                                         void* ws, size_t ws_bytes, hipStream_t stream) {
  return debug_gemm(M, N, K, A, B, false, C, R, epilogue, tile_cfg, ksplit, ws, ws_bytes, stream);
}

MX_EXPORT mx_status mx_debug_gemm_tiled(int32_t M, int32_t N, int32_t K, const uint16_t* A,
                                        const uint16_t* B_tiled, uint16_t* C, const uint16_t* R,
                                        int32_t epilogue, int32_t tile_cfg, int32_t ksplit,
                                        void* ws, size_t ws_bytes, hipStream_t stream) {
  return debug_gemm(M, N, K, A, B_tiled, true, C, R, epilogue, tile_cfg, ksplit, ws, ws_bytes,
                    stream);
}

MX_EXPORT mx_status mx_debug_gemm_plan(int32_t M, int32_t N, int32_t K, int32_t plan[5]) {
  g_err.clear();
  if (M < 0 || N <= 0 || K <= 0 || K % 64) return fail(MX_ERR_INVALID, "bad GEMM shape %d x %d x %d", M, N, K);
  if (!plan) return fail(MX_ERR_NULL, "plan is NULL");
  int out[5];
  gemm_plan(M, N, K, out);
  for (int i = 0; i < 5; i++) plan[i] = out[i];
  return MX_OK;
}

MX_EXPORT mx_status mx_debug_gemm_rows(int32_t M, int32_t N, int32_t K, const uint16_t* A,
                                       const uint16_t* B_tiled, uint16_t* C, const uint16_t* R,
                                       int32_t epilogue, int32_t m_main, int32_t main_cfg,
                                       int32_t tail_cfg, int32_t tail_ksplit, void* ws,
                                       size_t ws_bytes, hipStream_t stream) {
  g_err.clear();
  if (M < 2 || N <= 0 || K <= 0) return fail(MX_ERR_INVALID, "bad GEMM shape %d x %d x %d", M, N, K);
  if (N % 16 || K % 64) return fail(MX_ERR_UNSUPPORTED, "tiled weights need N %% 16 == 0 and K %% 64 == 0");
  if (m_main < 1 || m_main >= M || m_main % 16)
    return fail(MX_ERR_INVALID, "m_main %d not a multiple of 16 in [1, M)", m_main);
  if (main_cfg < 0 || main_cfg >= gemm_num_configs() || tail_cfg < 0 || tail_cfg >= gemm_num_configs())
    return fail(MX_ERR_INVALID, "tile config out of range");
  if (tail_ksplit < 1 || tail_ksplit > 64 || K / 64 < tail_ksplit)
    return fail(MX_ERR_INVALID, "K split %d is not in [1, min(64, K / 64 = %d)]", tail_ksplit, K / 64);
  if (epilogue < 0 || epilogue > 2) return fail(MX_ERR_INVALID, "bad epilogue %d", epilogue);
  if (epilogue == EPI_SWIGLU && N % 64) return fail(MX_ERR_UNSUPPORTED, "SwiGLU needs N % 64 == 0");
  if (!A || !B_tiled || !C || (epilogue == EPI_RESIDUAL && !R)) return fail(MX_ERR_NULL, "NULL operand");
  if (mx_status sa = check_aligned({A, B_tiled, C, R, ws}); sa != MX_OK) return sa;
  if (epilogue == EPI_RESIDUAL) {
    const size_t bytes = (size_t)M * N * 2;
    const char *c0 = (const char*)C, *r0 = (const char*)R;
    if (c0 < r0 + bytes && r0 < c0 + bytes) return fail(MX_ERR_INVALID, "R overlaps C");
  }
  const size_t need = tail_ksplit > 1 ? (size_t)tail_ksplit * (M - m_main) * N : 0;
  if (need && (!ws || ws_bytes < need * 4))
    return fail(MX_ERR_TOO_LARGE, "GEMM scratch %zu bytes < %zu", ws_bytes, need * 4);
  DeviceState* ds;
  mx_status st = device_state(&ds);
  if (st != MX_OK) return st;
  const int ldc = epilogue == EPI_SWIGLU ? N / 2 : N;
  GemmArgs g{A, B_tiled, C, R, (float*)ws, M, N, K, K, K, ldc, N, epilogue, {}};
  set_b_tiled(g);
  g.a_tiled = 1;
  g.c_tiled = epilogue == EPI_SWIGLU;
  hipError_t e = launch_gemm_rows(g, ws ? ws_bytes / 4 : 0, m_main, main_cfg, tail_cfg, tail_ksplit,
                                  stream);
  if (e != hipSuccess) return hip_fail(e, "gemm launch");
  return MX_OK;
}

MX_EXPORT mx_status mx_debug_reduce_residual_rmsnorm(const float* partial, int32_t ksplit,
                                                     const uint16_t* R, uint16_t* x1,
                                                     const uint16_t* g, uint16_t* h, int32_t M,
                                                     int32_t H, float eps, int32_t split_row,
                                                     hipStream_t stream) {
  g_err.clear();
  if (M < 0 || H <= 0 || H % 32) return fail(MX_ERR_INVALID, "bad shape %d x %d", M, H);
  if (H > kFusedNormMaxH) return fail(MX_ERR_UNSUPPORTED, "H %d > %d", H, kFusedNormMaxH);
  if (ksplit < 1) return fail(MX_ERR_INVALID, "ksplit %d < 1", ksplit);
  if (split_row < 0 || split_row > M) return fail(MX_ERR_INVALID, "split_row %d not in [0, M]", split_row);
  if (M == 0) return MX_OK;
  if ((split_row < M && !partial) || !R || !x1 || !g || !h) return fail(MX_ERR_NULL, "NULL operand");
  if (mx_status sa = check_aligned({partial, R, x1, g, h}); sa != MX_OK) return sa;
  DeviceState* ds;
  mx_status st = device_state(&ds);
  if (st != MX_OK) return st;
  hipError_t e = launch_reduce_residual_rmsnorm(partial, ksplit, R, x1, g, h, M, H, eps, split_row,
                                                stream);
  if (e != hipSuccess) return hip_fail(e, "reduce launch");
  return MX_OK;
}

MX_EXPORT mx_status mx_profile_enable(int32_t on) {
  std::lock_guard<std::mutex> g(g_prof.mu);
  g_prof.on = on != 0;
  return MX_OK;
}

MX_EXPORT int32_t mx_profile_read(const char** names, float* total_ms, int32_t* counts,
                                  int32_t max_entries) {
  std::lock_guard<std::mutex> g(g_prof.mu);
  for (auto& r : g_prof.pending) {
    float ms = 0.f;
    if (hipEventSynchronize(r.b) == hipSuccess && hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
      size_t i = 0;
      while (i < g_prof.names.size() && strcmp(g_prof.names[i], r.name) != 0) i++;
      if (i == g_prof.names.size()) {
        g_prof.names.push_back(r.name);
        g_prof.total_ms.push_back(0.0);
        g_prof.counts.push_back(0);
      }
      g_prof.total_ms[i] += ms;
      g_prof.counts[i] += 1;
    }
    g_prof.free_events.push_back(r.a);
    g_prof.free_events.push_back(r.b);
  }
  g_prof.pending.clear();
  const int32_t n = (int32_t)std::min<size_t>(g_prof.names.size(), (size_t)std::max(0, max_entries));
  for (int32_t i = 0; i < n; i++) {
    if (names) names[i] = g_prof.names[i];
    if (total_ms) total_ms[i] = (float)g_prof.total_ms[i];
    if (counts) counts[i] = g_prof.counts[i];
  }
  g_prof.names.clear();
  g_prof.total_ms.clear();
  g_prof.counts.clear();
  return n;
}
