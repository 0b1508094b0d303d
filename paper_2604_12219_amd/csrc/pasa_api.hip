// C ABI of the PASA forward (see include/pasa.h): argument validation, workspace carving, launches.
// Nothing here allocates, frees or synchronises.
#include "pasa.h"
#include "pasa_kernels.hpp"

#include <math.h>

#include <atomic>
#include <mutex>

// Scratch of pasa_sparse_attn_fwd_static, the entry point that allocates nothing: the attention workspace
// (statistics tiles, group matrices, unit sums) lives in this array instead of a caller's buffer.  Every GPU the
// library runs on holds its own copy until the process ends.  In host code the name is only a handle for
// hipGetSymbolAddress; the device address it yields is kept per device and is what the kernels receive.
static __device__ __align__(256) unsigned char scratch[PASA_STATIC_SCRATCH_BYTES];

namespace {

constexpr size_t kAlign = 256;
constexpr int kMaxChunks = 8192;   // chunks of 32 key blocks per head (262,144 key blocks)
constexpr int kMaxGroups = 65535;  // first-order groups per head
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

int check_shape(const pasa_shape_t* s) {
  if (!s) return PASA_EINVAL;
  if (s->B < 1 || s->H < 1 || s->n < 1) return PASA_EINVAL;
  if ((int64_t)s->B * s->H > 65535) return PASA_EUNSUPPORTED;
  if (s->d != 64 && s->d != 128) return PASA_EUNSUPPORTED;
  if (s->block != 64 && s->block != 128) return PASA_EUNSUPPORTED;
  if (!(s->scale >= 0.f) || isinf(s->scale)) return PASA_EINVAL;
  if (s->stride_n < s->d || s->stride_h < 1 || s->stride_b < 1) return PASA_EINVAL;
  if ((s->stride_n % 8) || (s->stride_h % 8) || (s->stride_b % 8)) return PASA_EALIGN;
  if ((int64_t)s->n * s->stride_n * 2 >= ((int64_t)1 << 32)) return PASA_EUNSUPPORTED;  // 32-bit byte offsets inside a head
  return PASA_OK;
}

int num_blocks(const pasa_shape_t* s) { return (s->n + s->block - 1) / s->block; }

int check_group(int group, int nb) {
  if (group < 0) return PASA_EINVAL;
  if (group == 0 || group >= nb) return PASA_OK;
  if (group % 32 == 0) return PASA_OK;
  if (group < 32 && (group & (group - 1)) == 0) return PASA_OK;
  return PASA_EUNSUPPORTED;
}

float effective_scale(const pasa_shape_t* s) { return s->scale > 0.f ? s->scale : 1.0f / sqrtf((float)s->d); }

struct AttnWorkspace {
  // `required` bytes hold everything that later calls read; between `required` and `total` there is room for the sums of units
  // smaller than `slot_unit`, which the statistics use if the caller's workspace has it
  size_t st, hg, partial, kbar, part_o, part_ml, queue, bitmap, required, total;
  int n_groups, n_chunks, n_slices;
  int slot_unit, n_slots, slots_per_group;  // the unit that the room for unit sums at `partial` is made for, and its units
};

// Number of key-range slices of the sparse kernel.  K and V of one head should fit the 4 MB L2 of an
// XCD slice by slice; there are 8 XCDs, so slices come in multiples of 8.
int choose_slices(const pasa_shape_t* s) {
  if (s->kv_slices >= 1) return s->kv_slices;
  // kv_slices == 0: no slicing.  Slicing removes most of the fabric traffic, but the extra partial
  // results and the merge pass cost more than that buys while the kernel is not yet limited by the
  // fabric; callers can switch it on per shape.
  return 1;
}

int check_slices(const pasa_shape_t* s) {
  if (s->kv_slices < 0) return PASA_EINVAL;
  if (s->kv_slices <= 1) return PASA_OK;
  if (s->kv_slices % 8 != 0 || s->kv_slices > (num_blocks(s) + 31) / 32) return PASA_EUNSUPPORTED;
  return PASA_OK;
}

int units_of(int nb, int unit) { return (nb + unit - 1) / unit; }

// The unit that the workspace always has room for.  The size a caller needs is a function of this one alone, so that
// a workspace does for the same shapes whatever unit the rule below takes.
int slot_unit(int64_t bh, int nb, int group) {
  int unit = group < 32 ? group : 32;
  while (unit > 8 && bh * units_of(nb, unit) < 1024) unit /= 2;
  return unit;
}

// Blocks summed by one workgroup of the statistics kernel: a whole group, at most 32 blocks, or half of that, a quarter, ...
// (which divides the group, unless the group is the whole sequence).  512 workgroups run at a time at d = 128, at d = 64 768
// before the memory is what counts (registers would allow 1024); so the sweep takes as many rounds as there are 512 or 768 units, each as
// long as a unit and the writing of its sum, which is worth about 6 blocks.  Units smaller than the group cost a launch that
// puts them together, about 8 blocks.  kv_stats_kernel + hg_finish_kernel, us, units of 32 / 16 / 8 / 4:
//   d = 128: 12 heads of 512 blocks 73 / 58 / 65 / 81; 5 of 1182 72 / 58 / 65 / 79; 3 of 1857 in groups of 64 75 / 54 / 61 / 74;
//     14 of 1182 190 / 181 / 193; 20 of 256 72 / 56 / 60; 16 of 513 97 / 76 / 91 (the rule's 32 is not the best there: 528 units
//     of 16 are hardly a second round)
//   d = 64: 12 of 512 38 / 27 / 25 / 29; in groups of 16 - / 25 / 26; 16 of 513 44 / 37 / 34; 24 of 512 46 / 41 / 46;
//     32 of 512 54 / 56 / 64; 20 of 1182 91 / 101 / 103
// Below 8 blocks the unit sums are more bytes than the keys and values they come from; that pays only where even units of 8
// leave most compute units without one and the kernel's time is that of one workgroup's serial sweep: 65 blocks x 4 heads
// take 22.9 us with units of 8 and 15.1 us with units of 2.  Units below slot_unit need room_bytes behind the required part.
int stats_unit(int64_t bh, int nb, int group, int d, size_t room_bytes) {
  auto units = [&](int unit) { return bh * units_of(nb, unit); };
  const int round = d == 128 ? 512 : 768;
  auto cost = [&](int unit) { return (units(unit) + round - 1) / round * (unit + 6) + (unit < group ? 8 : 0); };
  int best = group < 32 ? group : 32;
  for (int unit = best / 2; unit >= 8 && units(2 * unit) < 1024; unit /= 2)  // (with 1024 units the sums are many already)
    if (cost(unit) < cost(best)) best = unit;
  const int slot = slot_unit(bh, nb, group);
  while (best > 1 && units(best) < 128 && (best / 2 >= slot || (size_t)units(best / 2) * d * d * 4 <= room_bytes)) best /= 2;
  return best;
}

// The same for the prior's kernel, which has no sums to write but fetches its group's matrix once per workgroup (as many bytes
// as two blocks): half a unit pays while that leaves fewer than 1024 workgroups.  us, units of 16 / 8 / 4: 12 heads of 512 blocks
// 100 / 82 / 91, 5 of 1182 100 / 81 / 89, 3 of 1857 100 / 80 / 84.
int prior_unit(int64_t bh, int nb, int group) {
  int unit = group < 32 ? group : 32;
  while (unit > 8 && bh * ((nb + unit - 1) / unit) < 1024) unit /= 2;
  while (unit > 1 && bh * ((nb + unit - 1) / unit) < 128) unit /= 2;
  return unit;
}

AttnWorkspace carve_attn(const pasa_shape_t* s) {
  AttnWorkspace w{};
  const int nb = num_blocks(s);
  const size_t bh = (size_t)s->B * s->H;
  w.n_chunks = (nb + 31) / 32;
  w.n_slices = choose_slices(s);
  size_t off = 0;
  if (w.n_slices > 1) {
    w.part_o = off; off = align_up(off + bh * w.n_slices * s->n * s->d * 4);
    w.part_ml = off; off = align_up(off + bh * w.n_slices * s->n * 2 * 4);
    w.queue = off; off = align_up(off + 8 * 4);
  }
  // room for a selection bitmap built from index lists (callers that pass no bitmap of their own)
  w.bitmap = off; off = align_up(off + bh * nb * (size_t)w.n_chunks * 4);
  if (s->group > 0) {
    const int group = s->group >= nb ? nb : s->group;
    w.n_groups = (nb + group - 1) / group;
    w.slot_unit = slot_unit((int64_t)bh, nb, group);
    w.n_slots = units_of(nb, w.slot_unit);
    w.slots_per_group = s->group >= nb ? w.n_slots : group / w.slot_unit;
    w.st = off; off = align_up(off + bh * w.n_chunks * 64 * s->d * 2);
    w.hg = off; off = align_up(off + bh * w.n_groups * s->d * s->d * 2);
    w.partial = off; off = align_up(off + bh * w.n_slots * s->d * s->d * 4);
    w.kbar = off; off = align_up(off + bh * nb * s->d * 4);  // block-mean keys as split bf16 pairs, for pasa_block_score_with_stats
  }
  w.required = w.total = off;
  if (s->group > 0) {
    // room for small units, unless it would keep the shape from the static scratch array (PASA_STATIC_SCRATCH_BYTES)
    const size_t room_most = w.required <= (size_t)PASA_STATIC_SCRATCH_BYTES ? (size_t)PASA_STATIC_SCRATCH_BYTES - w.required : ~(size_t)0;
    const int unit = stats_unit((int64_t)bh, nb, s->group >= nb ? nb : s->group, s->d, room_most);
    if (unit < w.slot_unit) w.total += align_up(bh * units_of(nb, unit) * s->d * s->d * 4);
  }
  return w;
}

// Whether the dense path halves the keys between two teams of waves of a workgroup.  Such a workgroup fills a compute unit (eight
// waves of 256 registers): it pays where no compute unit would get two workgroups -- query tiles of a head are dealt to the
// eight XCDs in runs, so it is the 32 compute units of the XCD with the most tiles that count -- and where the walk is long
// enough to make up for the handing over.  us, one team / two:
//   d = 128: 512 tokens, 1 head 14.1 / 14.3; 768, 4: 19.0 / 18.1; 1024, 31: 29.8 / 28.3; 4140, 4: 79.9 / 68.9; 9900, 3: 198 / 168;
//     32,760, 1: 559 / 516; two workgroups on some compute units: 4140, 7: 123 / 141; 9900, 4: 273 / 301
//   d = 64: 320 tokens, 8 heads 7.8 / 8.1; 512, 16: 10.7 / 10.3; 1365, 6: 22.3 / 19.0; 9900, 3: 128 / 103; 1365, 22: 34.2 / 38.1
bool dense_teams(const pasa_shape_t* s) {
  const int64_t q_tiles_per_xcd = ((int64_t)s->n + 1023) / 1024, key_tiles = ((int64_t)s->n + 63) / 64;
  return (int64_t)s->B * s->H * q_tiles_per_xcd <= 32 && key_tiles >= (s->d == 128 ? 12 : 8);
}

// Whether the dense path takes workgroups of 256 query rows (eight waves, a compute unit to themselves) instead of two of 128 on a
// compute unit.  Both keep a compute unit equally busy, but the wide one brings every K and V tile into LDS once instead of twice,
// and where the power limit sets the clock that is worth 3.5 %: 12 heads of 32,760 tokens 5512 -> 5325 us at d = 128.  It loses where its
// rounds (32 compute units of the XCD with the most tiles at a time) come out longer than those of half the size.  us, narrow / wide:
//   d = 128: 7 heads of 4140 (35 narrow / 21 wide tiles on an XCD) 113 / 111; 12 (60 / 36) 132 / 229; 24 (120 / 72) 257 / 357;
//     6 of 9900 (60 / 30) 291 / 281; 26 (260 / 130) 1273 / 1362; 2 of 32,760 (64 / 32) 976 / 936; 3 (96 / 48) 1475 / 1562
//   d = 64: 7 of 4140 82.5 / 80.0; 12 86.6 / 159; 6 of 9900 195 / 193; 2 of 32,760 616 / 594
// At d = 64 a tile's loads are half as much and what a round of wide workgroups takes to start and to end counts for more, while over several rounds the two
// narrow ones of a compute unit cover each other's: there it is left at one round, two where the walk is long.  us, the code before this path and its pipelined
// steps / narrow / wide: 16 heads of 4096 (1 round) 89.5 / - / 86.0; 64 of 2048 (2) 92.6 / - / 94.6; 8 of 16,384 (2) 619 / - / 602; 96 of 2048 (3) 139 / 137 /
// 142; 128 (4) 182 / 178 / 188; 64 of 8192 (8) 1250 / 1206 / 1287; 12 of 32,760 (6) 3532 / 3431 / 3461
bool dense_wide(const pasa_shape_t* s) {
  const int64_t bh = (int64_t)s->B * s->H, n = s->n;
  const int64_t wide = (bh * ((n + 2047) / 2048) + 31) / 32, narrow = (bh * ((n + 1023) / 1024) + 31) / 32;  // rounds; half rounds
  return 62 * wide <= 32 * narrow && (s->d == 128 || wide <= (n > 8192 ? 2 : 1));
}

// Whether the sparse path with blocks of 64 tokens takes a ring of eight tiles instead of four.  The workgroup then has a compute unit to itself, so
// only where no compute unit would get two (see dense_teams), and it pays where the walk is long enough: the blocks of one of the two query blocks then
// take one barrier a step, and shared tiles arrive three steps ahead.  Where nearly every block is selected there are hardly any blocks of one query block
// alone, and it gains nothing: 7/8 of them is the line.  us, four / eight:
//   d = 128: 4140 tokens, 4 heads, 3 of 65 blocks 18.6 / 19.4, 10: 30.3 / 29.4, 26: 52.4 / 49.8; 9900, 3 heads, 8 of 155: 32.5 / 31.8, 62: 102 / 97.5;
//     32,760, 1 head, 26 of 512: 76.4 / 72.3; 2048, 16 heads, 13 of 32: 32.5 / 34.6; 4140, 6 heads, 52: 79.4 / 77.1, 58: 83.9 / 84.3, 65: 88.3 / 89.3
//   d = 64: 4140, 4 heads, 3: 12.3 / 12.2, 10: 20.8 / 19.4, 26: 37.0 / 33.9; 9900, 3 heads, 62: 75.4 / 67.0; 32,760, 1 head, 77: 104 / 90.9;
//     4140, 6 heads, 52: 57.6 / 55.4, 61: 62.5 / 62.4, 65: 64.0 / 65.0
bool sparse_deep(const pasa_shape_t* s, int32_t k_sel) {
  const int nb = num_blocks(s);
  return s->block == 64 && s->kv_slices <= 1 && nb >= 64 && k_sel >= 8 && 8 * (int64_t)k_sel <= 7 * (int64_t)nb && (int64_t)s->B * s->H * (((int64_t)s->n + 1023) / 1024) <= 32;
}

// Whether the sparse path takes workgroups of four query blocks of 64 tokens (pasa_quad.hpp) instead of two: they fetch fewer tiles, but plan
// their steps first (15 us a workgroup, with the starts and ends of its runs of steps) and have a compute unit to themselves meanwhile.  What they save depends
// on how little neighbouring query blocks have in common and on the caches, and the host knows only sizes.  The covariance prior and smooth inputs
// make the selections alike; the rule is such that even then the four lose next to nothing (at worst 1.7 %: groups of 64, 24 heads of 118,800 tokens, 177
// blocks).  Attention alone, us, two / four: first with independent noise as strong as the smooth field and no prior, then with noise of 0.2 and the prior:
//   * the selection has to be long.  75,600 tokens, 40 heads: 130 of 1182 blocks 19,446 / 18,845, 17,903 / 18,033 (in groups of 64 18,151 / 17,668,
//     16,583 / 16,899); 177: 24,957 / 23,678, 22,361 / 22,376 (23,861 / 22,474, 21,031 / 21,253); 295: - , 32,847 / 32,605
//   * the keys and values of a head have to exceed the eight L2s (32 MB), which otherwise hold what the rows select alike: 32,760 tokens, 40 heads, 245 of 512
//     blocks 11,442 / 11,577, 10,628 / 10,959; 47,628, 24 heads, 168 of 745 8104 / 7878, 7189 / 7608; 60,480, 12 heads, 189 of 945 6157 / 5860, 5249 / 5578; just
//     above, 68,040, 12 heads, 177 of 1064: - , 6134 / 6302
//   * those of all heads have to exceed the memory-side cache (256 MB) by far: 5 heads of 118,800 (304 MB), 371 of 1857 11,111 / 9848, 8578 / 8720; 10 of
//     75,600 (387 MB), 200 of 1182 - , 6350 / 6433
//   * the last round of workgroups (32 compute units of the XCD with the most tiles at a time) must not be much emptier than that of twice as many: 20 heads
//     of 75,600 (23.1 and 46.2 rounds), 177 blocks - , 11,432 / 11,716; 40 (46.2, 92.5) as above.  Where a head is larger there is more to gain: 24 of 118,800
//     (44.2, 87.8), 278 blocks 42,038 / 35,884, 32,562 / 32,564; 20 of 147,600 (45.6, 90.6), 461 - , 52,136 / 51,158
// Blocks of 128 tokens: 147,600 tokens, 6 heads, 58 blocks 4780 / 4889, 173: 11,014 / 11,338 (not taken).
bool sparse_quad(const pasa_shape_t* s, int32_t k_sel) {
  const int nb = num_blocks(s);
  if (s->d != 128 || s->block != 64 || s->kv_slices > 1 || s->n / 64 > kQuadMaxTiles || (s->group > 0 && s->group < 32)) return false;
  const int64_t bh = (int64_t)s->B * s->H, n = s->n, head_bytes = n * (4 * s->d);
  const int64_t quad = (bh * ((n + 2047) / 2048) + 31) / 32, pair = (bh * ((n + 1023) / 1024) + 31) / 32;  // rounds; half rounds
  return k_sel >= 160 && k_sel <= nb && head_bytes > (36 << 20) && bh * head_bytes > (int64_t)(512 << 20) &&
         160 * quad <= (head_bytes > (56 << 20) ? 82 : 81) * pair;
}

// Whether a walk (dense: every tile; sparse, blocks of 128 tokens: the selected ones) is too short for pipelined steps (pipe_step): a run of them
// starts and ends with a half-empty one, and requests a tile that nobody needs.  `tiles` of 64 keys.  us, steps of one tile / pipelined:
//   dense, d = 128: 1 tile, 1 head 6.5 / 6.9; 5, 1 head 10.6 / 10.8; 8 14.1 / 14.0; 12 17.9 / 17.0 (64 heads, 8 28.6 / 29.0, 16 48.8 / 46.8; 300, 1 30.0 / 30.7)
//   dense, d = 64: 300 heads, 1 tile 17.0 / 18.8, 4 37.7 / 38.4; 1 head, 5 tiles 7.4 / 7.9; 8 9.5 / 9.7; 12 12.1 / 12.2; 16 14.8 / 14.8; 20 17.1 / 17.0
//   blocks of 128, d = 128: 200 heads of 1024 tokens, 2 of 8 blocks 74.5 / 77.3, 4 104 / 106, 6 135 / 135, 8 168 / 166; 4140, 2 heads, 2 of 33 16.3 / 16.5, 6 25.5 /
//     25.3, 16 50.4 / 48.6
//   blocks of 128, d = 64: 4140, 2 heads, 2 of 33 11.0 / 11.3, 8 21.6 / 22.2, 24 47.8 / 48.4, 33 61.2 / 61.4; 40 heads, 8 93.6 / 94.6, 12 130 / 130, 32 303 / 299;
//     32,760, 12 heads, 4 of 256 146 / 150, 16 342 / 340
bool short_walk(const pasa_shape_t* s, bool sparse, int64_t tiles) { return tiles < (sparse ? (s->d == 128 ? 12 : 64) : (s->d == 128 ? 9 : 16)); }

// The form of the attention kernel a call takes (k_sel: declared number of selected key blocks; dense: not looked at)
AttnVariant attn_variant(const pasa_shape_t* s, bool sparse, int32_t k_sel) {
  if (!sparse) {
    if (short_walk(s, false, ((int64_t)s->n + 63) / 64)) return dense_teams(s) ? kShortTeams : kShort;
    return dense_teams(s) ? kTeams : dense_wide(s) ? kWide : kWhole;
  }
  if (choose_slices(s) > 1) return kSliced;
  if (s->block == 128) return short_walk(s, true, 2 * (int64_t)k_sel) ? kShort : kWhole;
  return sparse_deep(s, k_sel) ? kDeep : sparse_quad(s, k_sel) ? kQuad : kWhole;
}

// Whether a whole forward runs statistics and scoring in two launches instead of four (pasa_fused.hip).  The pooling then runs with the two workgroups a
// compute unit of the statistics: enough for tensors that are in cache or nearly so, not for the rate of the memory.  us, four / two, by MB of Q:
//   d = 128: 1024 tokens, 16 heads (4) 21.9 / 16.6; 2048, 40 (21) 39.3 / 29.4; 4140, 12 (13) 30.0 / 23.9; 9900, 16 (41) 52.3 / 47.8; 32,760, 2 (17)
//     37.5 / 28.7; 75,600, 1 (19) 40.6 / 30.4; 118,800, 3 (91) 119 / 126; 75,600, 5 (97) 112 / 128; 32,760, 12 (101) 101 / 119
//   d = 64: 2048, 40 (10) 23.7 / 17.3; 9900, 12 (15) 26.5 / 19.2; 32,760, 4 (17) 27.5 / 20.8; 32,760, 12 (50) 48.1 / 47.7
// At d = 128 512 units of the statistics run at a time: where there are as many, nothing is idle that the pooling could fill, and it is only held back.  Whole
// forwards, us: 256 tokens, 256 heads (256 units) 92.0 / 88.6, 512 heads 155 / 159; 128 tokens, 1024 heads 266 / 272; 64 tokens, 2048 410 / 416; d = 64, 64
// tokens, 2048 heads 235 / 233.
bool stats_and_score_together(const StatsParams& t) {
  return (int64_t)t.bh * t.n * t.d <= ((int64_t)20 << 20) && (t.d == 64 || (int64_t)t.bh * t.n_units < 512);
}

constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, null until looked up
std::mutex g_scratch_mutex;

// Device address of the static scratch array on the current device (looked up once per device).
int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PASA_EHIP;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    ptr = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (!ptr) {
      if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
        (void)hipGetLastError();
        return PASA_EHIP;
      }
      g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    }
  }
  *out = ptr;
  return PASA_OK;
}

}  // namespace

extern "C" {

const char* pasa_strerror(int status) {
  switch (status) {
    case PASA_OK: return "ok";
    case PASA_EINVAL: return "invalid argument";
    case PASA_EUNSUPPORTED: return "unsupported head dimension, block size, group size or problem size";
    case PASA_EWORKSPACE: return "workspace too small";
    case PASA_EALIGN: return "pointer or stride not sufficiently aligned";
    case PASA_EHIP: return "HIP launch failure";
    case PASA_ESCRATCH: return "problem needs more scratch than the static buffer of the no-allocation entry point holds";
    default: return "unknown status";
  }
}

int32_t pasa_topk_count(int32_t n_blocks, double keep_ratio) {
  if (n_blocks < 1 || !(keep_ratio > 0.0) || keep_ratio > 1.0) return PASA_EINVAL;
  double x = floor(keep_ratio * (double)n_blocks + 0.5);
  if (x < 1.0) x = 1.0;
  if (x > (double)n_blocks) x = (double)n_blocks;
  return (int32_t)x;
}

int32_t pasa_num_blocks(const pasa_shape_t* shape) {
  const int rc = check_shape(shape);
  return rc != PASA_OK ? rc : num_blocks(shape);
}

int32_t pasa_mask_words(int32_t n_blocks) { return n_blocks < 1 ? PASA_EINVAL : (n_blocks + 31) / 32; }

size_t pasa_score_workspace_bytes(const pasa_shape_t* shape) {
  if (check_shape(shape) != PASA_OK) return 0;
  const size_t one = align_up((size_t)shape->B * shape->H * num_blocks(shape) * shape->d * 4);
  return 2 * one;
}

size_t pasa_attn_workspace_bytes(const pasa_shape_t* shape) {
  if (check_shape(shape) != PASA_OK) return 0;
  if (check_group(shape->group, num_blocks(shape)) != PASA_OK) return 0;
  if (check_slices(shape) != PASA_OK) return 0;
  return carve_attn(shape).total;  // never zero for a valid shape (it holds a bitmap), so that 0 always means "bad shape"
}

int32_t pasa_attn_variant(const pasa_shape_t* shape, int32_t k_sel) {
  const int rc = check_shape(shape);
  if (rc != PASA_OK) return rc;
  if (k_sel < 0 || k_sel > num_blocks(shape)) return PASA_EINVAL;
  if (k_sel > 0) {
    const int rg = check_group(shape->group, num_blocks(shape));
    if (rg != PASA_OK) return rg;
    const int rs = check_slices(shape);
    if (rs != PASA_OK) return rs;
  }
  return attn_variant(shape, k_sel > 0, k_sel);
}

static int score_params(const void* q, const void* k, const pasa_shape_t* shape, const float* key_bias, float* scores, void* ws, size_t ws_bytes,
                        const void* kbar_split, ScoreParams* out) {
  const int rc = check_shape(shape);
  if (rc != PASA_OK) return rc;
  if (!q || (!k && !kbar_split) || !scores || !ws) return PASA_EINVAL;
  if (!aligned16(q) || (k && !aligned16(k)) || !aligned16(scores) || !aligned16(ws)) return PASA_EALIGN;
  if (ws_bytes < pasa_score_workspace_bytes(shape)) return PASA_EWORKSPACE;
  ScoreParams& p = *out;
  p = ScoreParams{};
  p.q = static_cast<const uint16_t*>(q);
  p.k = static_cast<const uint16_t*>(k);
  p.stride_b = shape->stride_b; p.stride_h = shape->stride_h; p.stride_n = shape->stride_n;
  p.bh = shape->B * shape->H; p.H = shape->H; p.n = shape->n; p.nb = num_blocks(shape);
  p.block = shape->block; p.d = shape->d;
  p.scale = effective_scale(shape);
  p.key_bias = key_bias;
  p.qbar = static_cast<float*>(ws);
  p.pool_k = kbar_split ? 0 : 1;
  p.kbar = kbar_split ? const_cast<float*>(static_cast<const float*>(kbar_split))
                      : reinterpret_cast<float*>(static_cast<char*>(ws) + pasa_score_workspace_bytes(shape) / 2);
  p.scores = scores;
  return PASA_OK;
}

static int block_score_impl(const void* q, const void* k, const pasa_shape_t* shape, const float* key_bias, float* scores, void* ws, size_t ws_bytes,
                            const void* kbar_split, void* stream) {
  ScoreParams p;
  const int rc = score_params(q, k, shape, key_bias, scores, ws, ws_bytes, kbar_split, &p);
  if (rc != PASA_OK) return rc;
  return pasa_launch_block_score(p, static_cast<hipStream_t>(stream)) == hipSuccess ? PASA_OK : PASA_EHIP;
}

int pasa_block_score(const void* q, const void* k, const pasa_shape_t* shape, const float* key_bias, float* scores,
                     void* ws, size_t ws_bytes, void* stream) {
  return block_score_impl(q, k, shape, key_bias, scores, ws, ws_bytes, nullptr, stream);
}

static int route_params(const float* scores, int32_t BH, int32_t n_blocks, int32_t k_sel, uint64_t seed, float noise_amp, int gumbel, int32_t* idx,
                        uint32_t* mask, RouteParams* out) {
  if (!scores || !idx || BH < 1 || n_blocks < 1) return PASA_EINVAL;
  if (k_sel < 1 || k_sel > n_blocks) return PASA_EINVAL;
  if (!(noise_amp >= 0.f) || isinf(noise_amp)) return PASA_EINVAL;
  if (n_blocks > kRouteMaxBlocks) return PASA_EUNSUPPORTED;
  RouteParams& p = *out;
  p = RouteParams{};
  p.scores = scores;
  p.bh = BH; p.nb = n_blocks; p.k_sel = k_sel; p.mask_words = (n_blocks + 31) / 32;
  p.seed_lo = (uint32_t)(seed & 0xffffffffu); p.seed_hi = (uint32_t)(seed >> 32);
  p.amp = noise_amp;
  p.gumbel = gumbel;
  p.idx = idx; p.mask = mask;
  return PASA_OK;
}

static int route_impl(const float* scores, int32_t BH, int32_t n_blocks, int32_t k_sel, uint64_t seed, float noise_amp,
                      int gumbel, int32_t* idx, uint32_t* mask, void* stream) {
  RouteParams p;
  const int rc = route_params(scores, BH, n_blocks, k_sel, seed, noise_amp, gumbel, idx, mask, &p);
  if (rc != PASA_OK) return rc;
  return pasa_launch_route(p, static_cast<hipStream_t>(stream)) == hipSuccess ? PASA_OK : PASA_EHIP;
}

int pasa_route(const float* scores, int32_t BH, int32_t n_blocks, int32_t k_sel, uint64_t seed, float noise_amp,
               int32_t* idx, uint32_t* mask, void* stream) {
  return route_impl(scores, BH, n_blocks, k_sel, seed, noise_amp, 0, idx, mask, stream);
}

int pasa_route_gumbel(const float* scores, int32_t BH, int32_t n_blocks, int32_t k_sel, uint64_t seed, float temperature,
                      int32_t* idx, uint32_t* mask, void* stream) {
  return route_impl(scores, BH, n_blocks, k_sel, seed, temperature, 1, idx, mask, stream);
}

// validation shared by the statistics and attention entry points; fills `s` (group normalised)
static int check_attn_args(const pasa_shape_t* shape, bool sparse, const void* ws, size_t ws_bytes, pasa_shape_t* s) {
  const int rc = check_shape(shape);
  if (rc != PASA_OK) return rc;
  *s = *shape;
  if (!sparse) { s->group = 0; s->kv_slices = 1; }
  const int rg = check_group(s->group, num_blocks(s));
  if (rg != PASA_OK) return rg;
  const int rs = check_slices(s);
  if (rs != PASA_OK) return rs;
  {  // one workgroup per 128 query rows, counted in 32 bits (also the work items of key-range slicing)
    const int64_t q_tiles = ((int64_t)s->n + 127) / 128;
    const int64_t wgs = (int64_t)s->B * s->H * 8 * ((q_tiles + 7) / 8) * (s->kv_slices > 1 ? s->kv_slices / 8 : 1);
    if (wgs >= ((int64_t)1 << 31)) return PASA_EUNSUPPORTED;
  }
  if (sparse) {  // field widths of the approximation pass's tile descriptors (13 bits of chunk, 16 bits of group)
    const int nb = num_blocks(s);
    const int group = s->group >= nb ? nb : s->group;
    if ((nb + 31) / 32 > kMaxChunks) return PASA_EUNSUPPORTED;
    if (group > 0 && (nb + group - 1) / group > kMaxGroups) return PASA_EUNSUPPORTED;
  }
  if (!ws) return PASA_EINVAL;
  if (!aligned16(ws)) return PASA_EALIGN;
  if (ws_bytes < carve_attn(s).required) return PASA_EWORKSPACE;
  return PASA_OK;
}

int pasa_block_score_with_stats(const void* q, const pasa_shape_t* shape, const float* key_bias, float* scores, void* ws,
                                size_t ws_bytes, const void* stats_ws, size_t stats_ws_bytes, void* stream) {
  pasa_shape_t s;
  const int rc = check_attn_args(shape, true, stats_ws, stats_ws_bytes, &s);
  if (rc != PASA_OK) return rc;
  if (s.group == 0) return PASA_EUNSUPPORTED;  // pasa_kv_stats leaves nothing when the approximation is off
  const AttnWorkspace w = carve_attn(&s);
  return block_score_impl(q, nullptr, shape, key_bias, scores, ws, ws_bytes, static_cast<const char*>(stats_ws) + w.kbar, stream);
}

int pasa_check_selection(const int32_t* idx, const uint32_t* mask, int32_t BH, int32_t n_blocks, int32_t k_sel, int32_t* n_bad,
                         void* stream) {
  if ((!idx && !mask) || !n_bad || BH < 1 || n_blocks < 1 || k_sel < 1 || k_sel > n_blocks) return PASA_EINVAL;
  if ((idx && !aligned4(idx)) || (mask && !aligned4(mask)) || !aligned4(n_bad)) return PASA_EALIGN;
  return pasa_launch_check_selection(idx, mask, (int64_t)BH * n_blocks, n_blocks, k_sel, n_bad, static_cast<hipStream_t>(stream)) ==
                 hipSuccess ? PASA_OK : PASA_EHIP;
}

// idx not null: the same launch builds the selection bitmap in the workspace from these index lists of k_sel blocks.
// out->group stays 0 where the approximation is off and there is nothing to launch
static int stats_params(const void* k, const void* v, const pasa_shape_t* shape, const int32_t* idx, int32_t k_sel, void* ws, size_t ws_bytes,
                        StatsParams* out) {
  StatsParams& t = *out;
  t = StatsParams{};
  pasa_shape_t s;
  const int rc = check_attn_args(shape, true, ws, ws_bytes, &s);
  if (rc != PASA_OK) return rc;
  if (!k || !v) return PASA_EINVAL;
  if (!aligned16(k) || !aligned16(v)) return PASA_EALIGN;
  if (s.group == 0) return PASA_OK;
  const int nb = num_blocks(&s);
  const AttnWorkspace w = carve_attn(&s);
  char* base = static_cast<char*>(ws);
  t.k = static_cast<const uint16_t*>(k); t.v = static_cast<const uint16_t*>(v);
  t.stride_b = s.stride_b; t.stride_h = s.stride_h; t.stride_n = s.stride_n;
  t.bh = s.B * s.H; t.H = s.H; t.n = s.n; t.nb = nb; t.block = s.block; t.tail = s.n - (nb - 1) * s.block; t.d = s.d;
  t.group = s.group >= nb ? nb : s.group; t.n_groups = w.n_groups;
  t.unit = stats_unit(t.bh, nb, t.group, s.d, ws_bytes - w.required);
  t.n_units = units_of(nb, t.unit);
  t.units_per_group = t.n_groups == 1 ? t.n_units : t.group / t.unit;
  t.scale = effective_scale(&s);
  t.n_chunks = w.n_chunks;
  t.st = reinterpret_cast<uint16_t*>(base + w.st);
  t.hg = reinterpret_cast<uint16_t*>(base + w.hg);
  t.group_sum = reinterpret_cast<float*>(base + w.partial);
  t.sum_head = w.n_slots; t.sum_group = w.slots_per_group;
  if (t.unit >= w.slot_unit) {  // a unit takes the slot of its first block
    t.partial = t.group_sum; t.partial_head = t.sum_head; t.partial_step = t.unit / w.slot_unit;
  } else {
    t.partial = reinterpret_cast<float*>(base + w.required); t.partial_head = t.n_units; t.partial_step = 1;
  }
  t.kbar_split = reinterpret_cast<uint16_t*>(base + w.kbar);
  t.idx = idx; t.k_sel = k_sel; t.mask_words = (nb + 31) / 32;
  t.mask = reinterpret_cast<uint32_t*>(base + w.bitmap);
  return PASA_OK;
}

static int kv_stats_impl(const void* k, const void* v, const pasa_shape_t* shape, const int32_t* idx, int32_t k_sel, void* ws, size_t ws_bytes,
                         void* stream) {
  StatsParams t;
  const int rc = stats_params(k, v, shape, idx, k_sel, ws, ws_bytes, &t);
  if (rc != PASA_OK || t.group == 0) return rc;
  return pasa_launch_kv_stats(t, static_cast<hipStream_t>(stream)) == hipSuccess ? PASA_OK : PASA_EHIP;
}

int pasa_kv_stats(const void* k, const void* v, const pasa_shape_t* shape, void* ws, size_t ws_bytes, void* stream) {
  return kv_stats_impl(k, v, shape, nullptr, 0, ws, ws_bytes, stream);
}

int pasa_key_prior(const void* k, const void* v, const pasa_shape_t* shape, float eps, float* beta, void* ws,
                   size_t ws_bytes, void* stream) {
  pasa_shape_t s;
  const int rc = check_attn_args(shape, true, ws, ws_bytes, &s);
  if (rc != PASA_OK) return rc;
  if (!k || !v || !beta || !(eps >= 0.f)) return PASA_EINVAL;
  if (!aligned16(k) || !aligned16(v)) return PASA_EALIGN;
  if (s.group == 0) return PASA_EUNSUPPORTED;
  const int nb = num_blocks(&s);
  const AttnWorkspace w = carve_attn(&s);
  char* base = static_cast<char*>(ws);
  StatsParams t{};
  t.k = static_cast<const uint16_t*>(k); t.v = static_cast<const uint16_t*>(v);
  t.stride_b = s.stride_b; t.stride_h = s.stride_h; t.stride_n = s.stride_n;
  t.bh = s.B * s.H; t.H = s.H; t.n = s.n; t.nb = nb; t.block = s.block; t.tail = s.n - (nb - 1) * s.block; t.d = s.d;
  t.group = s.group >= nb ? nb : s.group; t.n_groups = w.n_groups;
  t.prior_unit = prior_unit(t.bh, nb, t.group);
  t.scale = effective_scale(&s);
  t.n_chunks = w.n_chunks;
  t.group_sum = reinterpret_cast<float*>(base + w.partial);
  t.sum_head = w.n_slots; t.sum_group = w.slots_per_group;
  return pasa_launch_key_prior(t, eps, beta, static_cast<hipStream_t>(stream)) == hipSuccess ? PASA_OK : PASA_EHIP;
}

// Everything but the launches: checks the arguments and fills what the attention kernel is launched with.
// *build: the bitmap that has to be built from the index lists first (the caller gave none), null if there is nothing to build
static int attn_params(const void* q, const void* k, const void* v, const pasa_shape_t* shape, const int32_t* idx, const uint32_t* mask, int32_t k_sel,
                       void* out, float* lse, void* ws, size_t ws_bytes, bool sparse, AttnParams* params, uint32_t** build) {
  pasa_shape_t s;
  const int rc = check_attn_args(shape, sparse, ws, ws_bytes, &s);
  if (rc != PASA_OK) return rc;
  const int nb = num_blocks(&s);
  if (!q || !k || !v || !out) return PASA_EINVAL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out)) return PASA_EALIGN;
  if (out == q || out == k || out == v) return PASA_EINVAL;
  if (sparse) {
    if ((!idx && !mask) || k_sel < 1 || k_sel > nb) return PASA_EINVAL;
    if ((idx && !aligned4(idx)) || (mask && !aligned4(mask))) return PASA_EALIGN;
  }
  const AttnWorkspace w = carve_attn(&s);
  char* base = static_cast<char*>(ws);
  AttnParams& a = *params;
  a = AttnParams{};
  *build = nullptr;
  a.q = static_cast<const uint16_t*>(q); a.k = static_cast<const uint16_t*>(k); a.v = static_cast<const uint16_t*>(v);
  a.o = static_cast<uint16_t*>(out); a.lse = lse;
  a.stride_b = s.stride_b; a.stride_h = s.stride_h; a.stride_n = s.stride_n;
  a.bh = s.B * s.H; a.H = s.H; a.n = s.n; a.nb = nb; a.block = s.block; a.tail = s.n - (nb - 1) * s.block;
  a.scale = effective_scale(&s);
  a.n_slices = 1;
  if (sparse) {
    if (!mask) {  // the caller has index lists only: the bitmap the kernel walks is built from them
      *build = reinterpret_cast<uint32_t*>(base + w.bitmap);
      mask = *build;
    }
    a.idx = idx; a.mask = mask; a.k_sel = k_sel; a.mask_words = (nb + 31) / 32;
    a.group = s.group >= nb ? nb : s.group;
    a.st = reinterpret_cast<const uint16_t*>(base + w.st);
    a.hg = reinterpret_cast<const uint16_t*>(base + w.hg);
    a.n_groups = w.n_groups;
    a.n_chunks = w.n_chunks;
    a.n_slices = w.n_slices;
    a.part_o = reinterpret_cast<float*>(base + w.part_o);
    a.part_ml = reinterpret_cast<float*>(base + w.part_ml);
    a.queue = reinterpret_cast<uint32_t*>(base + w.queue);
  }
  a.variant = attn_variant(&s, sparse, k_sel);
  return PASA_OK;
}

static int attn_common(const void* q, const void* k, const void* v, const pasa_shape_t* shape, const int32_t* idx,
                       const uint32_t* mask, int32_t k_sel, void* out, float* lse, void* ws, size_t ws_bytes,
                       void* stream, bool sparse, bool with_stats) {
  AttnParams a;
  uint32_t* build;
  const int rc = attn_params(q, k, v, shape, idx, mask, k_sel, out, lse, ws, ws_bytes, sparse, &a, &build);
  if (rc != PASA_OK) return rc;
  const bool mask_with_stats = with_stats && build && a.group > 0;  // (without the approximation there is no statistics launch)
  if (with_stats) {
    const int rs = kv_stats_impl(k, v, shape, mask_with_stats ? idx : nullptr, k_sel, ws, ws_bytes, stream);
    if (rs != PASA_OK) return rs;
  }
  if (build && !mask_with_stats &&
      pasa_launch_mask_from_idx(idx, (int64_t)a.bh * a.nb, a.nb, k_sel, build, static_cast<hipStream_t>(stream)) != hipSuccess)
    return PASA_EHIP;
  return pasa_launch_attn(a, sparse, shape->d, static_cast<hipStream_t>(stream)) == hipSuccess ? PASA_OK : PASA_EHIP;
}

int pasa_sparse_attn_fwd(const void* q, const void* k, const void* v, const pasa_shape_t* shape, const int32_t* idx,
                         const uint32_t* mask, int32_t k_sel, void* out, float* lse, void* ws, size_t ws_bytes,
                         void* stream) {
  return attn_common(q, k, v, shape, idx, mask, k_sel, out, lse, ws, ws_bytes, stream, true, true);
}

int pasa_sparse_attn_fwd_prepared(const void* q, const void* k, const void* v, const pasa_shape_t* shape,
                                  const int32_t* idx, const uint32_t* mask, int32_t k_sel, void* out, float* lse,
                                  void* ws, size_t ws_bytes, void* stream) {
  return attn_common(q, k, v, shape, idx, mask, k_sel, out, lse, ws, ws_bytes, stream, true, false);
}

int pasa_sparse_attn_fwd_static(const void* q, const void* k, const void* v, const pasa_shape_t* shape,
                                const int32_t* idx, const uint32_t* mask, int32_t k_sel, void* out, float* lse,
                                void* stream) {
  const int rc = check_shape(shape);
  if (rc != PASA_OK) return rc;
  pasa_shape_t s = *shape;
  s.kv_slices = 1;  // the partial results of key-range slicing do not fit a modest static buffer
  const size_t need = pasa_attn_workspace_bytes(&s);
  if (need == 0) return check_group(s.group, num_blocks(&s)) != PASA_OK ? check_group(s.group, num_blocks(&s)) : PASA_EINVAL;
  if (need > (size_t)PASA_STATIC_SCRATCH_BYTES) return PASA_ESCRATCH;
  if (!q || !k || !v || !out || (!idx && !mask) || k_sel < 1 || k_sel > num_blocks(&s)) return PASA_EINVAL;
  void* ws = nullptr;
  const int rp = static_scratch(&ws);
  if (rp != PASA_OK) return rp;
  return attn_common(q, k, v, &s, idx, mask, k_sel, out, lse, ws, (size_t)PASA_STATIC_SCRATCH_BYTES, stream, true, true);
}

// ---- the whole forward in one call ---------------------------------------------------------------
namespace {
struct ForwardWorkspace {
  size_t scores, idx, mask, score_ws, attn_ws, required, total;
  int nb, k_sel;
};

// 0 in `total` on invalid arguments
ForwardWorkspace carve_forward(const pasa_shape_t* s, double keep_ratio) {
  ForwardWorkspace f{};
  if (check_shape(s) != PASA_OK) return f;
  f.nb = num_blocks(s);
  const int32_t k = pasa_topk_count(f.nb, keep_ratio);
  if (k < 1) return f;
  f.k_sel = k;
  pasa_shape_t a = *s;
  const size_t attn = pasa_attn_workspace_bytes(&a), score = pasa_score_workspace_bytes(&a);
  if (attn == 0 || score == 0) return f;
  const size_t attn_required = carve_attn(&a).required;
  const size_t bh = (size_t)s->B * s->H;
  size_t off = 0;
  f.scores = off; off = align_up(off + bh * f.nb * f.nb * 4);
  f.idx = off; off = align_up(off + bh * f.nb * (size_t)k * 4);
  f.mask = off; off = align_up(off + bh * f.nb * (size_t)((f.nb + 31) / 32) * 4);
  f.score_ws = off; off = align_up(off + score);
  f.attn_ws = off;
  f.required = off + attn_required;
  f.total = off + attn;
  return f;
}
}  // namespace

// The stages of a whole forward.  Every argument of every stage is checked before the first launch.
// pool_k: the scores' block-mean keys are pooled as pasa_block_score does it, not taken from the statistics (the two differ in the last place)
static int forward_stages(const void* q, const void* k, const void* v, const pasa_shape_t* shape, int32_t k_sel, uint64_t seed, float noise_amp,
                          float* scores, int32_t* idx, uint32_t* mask, void* score_ws, size_t score_bytes, void* attn_ws, size_t attn_bytes, void* out,
                          float* lse, bool pool_k, void* stream) {
  StatsParams t;
  ScoreParams p;
  RouteParams r;
  AttnParams a;
  uint32_t* build;
  int rc = stats_params(k, v, shape, nullptr, 0, attn_ws, attn_bytes, &t);
  if (rc != PASA_OK) return rc;
  const bool approx = t.group > 0;  // otherwise there are no statistics, and no key means in them
  rc = score_params(q, k, shape, nullptr, scores, score_ws, score_bytes, pool_k || !approx ? nullptr : t.kbar_split, &p);
  if (rc != PASA_OK) return rc;
  rc = route_params(scores, shape->B * shape->H, num_blocks(shape), k_sel, seed, noise_amp, 0, idx, mask, &r);
  if (rc != PASA_OK) return rc;
  rc = attn_params(q, k, v, shape, idx, mask, k_sel, out, lse, attn_ws, attn_bytes, true, &a, &build);
  if (rc != PASA_OK) return rc;

  const hipStream_t on = static_cast<hipStream_t>(stream);
  if (approx && stats_and_score_together(t)) {
    if (pasa_launch_stats_and_score(t, p, on) != hipSuccess) return PASA_EHIP;
  } else {
    if (approx && pasa_launch_kv_stats(t, on) != hipSuccess) return PASA_EHIP;
    if (pasa_launch_block_score(p, on) != hipSuccess) return PASA_EHIP;
  }
  if (pasa_launch_route(r, on) != hipSuccess) return PASA_EHIP;
  return pasa_launch_attn(a, true, shape->d, on) == hipSuccess ? PASA_OK : PASA_EHIP;
}

size_t pasa_forward_workspace_bytes(const pasa_shape_t* shape, double keep_ratio) { return carve_forward(shape, keep_ratio).total; }

int pasa_forward(const void* q, const void* k, const void* v, const pasa_shape_t* shape, double keep_ratio, uint64_t seed,
                 float noise_amp, void* out, float* lse, void* ws, size_t ws_bytes, void* stream) {
  const int rc = check_shape(shape);
  if (rc != PASA_OK) return rc;
  if (!(keep_ratio > 0.0) || keep_ratio > 1.0) return PASA_EINVAL;
  const int rg = check_group(shape->group, num_blocks(shape));
  if (rg != PASA_OK) return rg;
  const int rs = check_slices(shape);
  if (rs != PASA_OK) return rs;
  const ForwardWorkspace f = carve_forward(shape, keep_ratio);
  if (f.total == 0) return PASA_EUNSUPPORTED;
  if (!q || !k || !v || !out || !ws) return PASA_EINVAL;
  if (!aligned16(ws)) return PASA_EALIGN;
  if (ws_bytes < f.required) return PASA_EWORKSPACE;
  if (f.nb > kRouteMaxBlocks) return PASA_EUNSUPPORTED;
  char* base = static_cast<char*>(ws);
  float* scores = reinterpret_cast<float*>(base + f.scores);
  int32_t* idx = reinterpret_cast<int32_t*>(base + f.idx);
  uint32_t* mask = reinterpret_cast<uint32_t*>(base + f.mask);
  return forward_stages(q, k, v, shape, f.k_sel, seed, noise_amp, scores, idx, mask, base + f.score_ws, pasa_score_workspace_bytes(shape),
                        base + f.attn_ws, ws_bytes - f.attn_ws, out, lse, /*pool_k=*/false, stream);
}

int pasa_forward_buffers(const void* q, const void* k, const void* v, const pasa_shape_t* shape, int32_t k_sel, uint64_t seed, float noise_amp,
                         float* scores, int32_t* idx, uint32_t* mask, void* score_ws, size_t score_ws_bytes, void* attn_ws, size_t attn_ws_bytes,
                         void* out, float* lse, void* stream) {
  const int rc = check_shape(shape);
  if (rc != PASA_OK) return rc;
  if (num_blocks(shape) > kRouteMaxBlocks) return PASA_EUNSUPPORTED;
  if (!mask) return PASA_EINVAL;
  return forward_stages(q, k, v, shape, k_sel, seed, noise_amp, scores, idx, mask, score_ws, score_ws_bytes, attn_ws, attn_ws_bytes, out, lse,
                        /*pool_k=*/true, stream);
}

int pasa_attn_dense_ref(const void* q, const void* k, const void* v, const pasa_shape_t* shape, void* out, float* lse,
                        void* ws, size_t ws_bytes, void* stream) {
  return attn_common(q, k, v, shape, nullptr, nullptr, 0, out, lse, ws, ws_bytes, stream, false, false);
}

}  // extern "C"
