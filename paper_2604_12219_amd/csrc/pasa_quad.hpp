// Exact passes of the sparse attention kernel for workgroups of 256 query rows (eight waves, a compute unit to themselves): four adjacent
// query blocks of 64 tokens, two waves each ("groups"), which share every key block that more than one of them selected.  d = 128.
//
// Why.  Where a head's keys are much larger than an L2, the reads that miss the L2s bound the sparse kernel (7.2 to 7.9 TB/s, whatever is in
// flight).  Two query blocks that stream the union of their selections fetch 257 key blocks for 354 selected ones (75,600 tokens, 15 %),
// four fetch 373 for 708.  Attention alone, us, workgroups of two query blocks / of four: 75,600 tokens, 40 heads, 177 of 1182 blocks
// 24,912 / 24,034; 5 heads 3228 / 2982, 414 blocks 6631 / 5732; 118,800 tokens, 3 heads, 279 of 1857 blocks 5210 / 4702, 650 blocks 10,541 / 8776.
// (What the rule, sparse_quad in pasa_api.hip, leaves to two query blocks of these: few heads, whose selections may be alike.)
// What is left of the time is power: with all-zero inputs 10 heads of the first take 6.3 / 5.0 ms, with random ones 6.5 / 6.0.
//
// Classes and runs.  A key block belongs to the class of the groups that selected it (15 classes of four groups).  One block each of some
// disjoint classes makes a step in which every group has a tile.  Taking the classes greedily (all four groups; three and the fourth; two
// and two; two and two single ones; four single ones) uses all of them up at the sizes above, in exactly as many steps as a query block
// selects blocks: no wave waits for tiles that others need.  What is left where the groups' numbers of blocks differ makes steps in which
// some groups are idle.  The steps are put into runs of one number of tiles each, but steps of four and of three tiles alternate
// with steps of one as far as there are any: four tiles a step are more than the memory delivers in the time.
// The plan is made at the start of the workgroup, in LDS: a list of the tiles, step by step.
//
// Steps.  Half steps of 32 keys (pasa_mfma_pipes.hpp): the logits run one tile ahead of P V.  Half h of step s consumes the halves h of
// the K tiles of step s + 1 and of the V tiles of step s: one batch, as large for all s of a run.  LDS holds 9 to 2 batches: one is consumed
// while the others land, one barrier per half step.  Every wave requests an eighth of
// every half tile, so that no wave is held up by more than the others, in the shadow of its MFMAs.
#pragma once
#include "pasa_device.hpp"
#include "pasa_kernels.hpp"
#include "pasa_mfma_pipes.hpp"

namespace {

constexpr int kQuadWaves = 8;
constexpr int kQuadGroups = 4;
constexpr int kQuadSlots = pipes::kQuadSlots;
constexpr int kQuadMaxTakes = 15;     // every take uses a class up
constexpr int kQuadMaxRuns = pipes::kQuadKinds + kQuadMaxTakes;
constexpr int kQuadDim = 128;         // the head dimension
constexpr int kQuadHalf = 8 * pipes::kQuadBlock;

struct QuadRun {
  int steps, even, odd, base;  // 64-key steps; tiles of an even and of an odd one; place of the first one in the list
};

struct QuadShared {
  __attribute__((aligned(1024))) char ring[kQuadSlots * kQuadHalf];
  uint16_t list[kQuadMaxTiles];  // tile number and, in bits 12.., the groups that want it: step by step, run by run
  int begin[16];                 // planner: where a class begins among the sorted tiles
  int4 parts[4 * kQuadMaxTakes]; // planner: class part of a take: place among the sorted tiles, tiles, first step among those of n tiles (idle groups:
                                 // number of the run), place in a step | n << 4 | idle << 7 | class << 8
  int n_parts, n_runs, alternating[2];  // steps of three and of four tiles that alternate with steps of one
  QuadRun runs[kQuadMaxRuns];
  // planner only, before the ring is in use: tiles of each class in the segments of 64 key blocks before each; the tiles by class
  PASA_DEVICE int* counts() { return reinterpret_cast<int*>(ring); }
  PASA_DEVICE uint16_t* sorted() { return reinterpret_cast<uint16_t*>(ring + kQuadMaxTiles / 64 * 16 * 4); }
};
static_assert(kQuadMaxTiles / 64 * 16 * 4 + kQuadMaxTiles * 2 <= kQuadSlots * kQuadHalf && kQuadMaxTiles <= 4096, "");

PASA_DEVICE int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
PASA_DEVICE const char* uniform(const void* x) {
  const uint64_t a = (uint64_t)x;
  return reinterpret_cast<const char*>((uint64_t)(uint32_t)uniform((int)(uint32_t)(a >> 32)) << 32 | (uint32_t)uniform((int)(uint32_t)a));
}

// rows[g]: bitmap row of group g.  n_whole: key blocks to be planned (at most kQuadMaxTiles).
PASA_DEVICE void quad_plan(QuadShared& sh, const uint32_t* const (&rows)[kQuadGroups], int n_whole, int wave, int lane) {
  constexpr int G = kQuadGroups, NC = (1 << G) - 1;  // classes 1..NC
  const int n_seg = (n_whole + 63) / 64;
  auto class_of = [&](int seg) -> int {  // of key block 64 seg + lane, 0: nobody's
    const int j = 64 * seg + lane;
    uint32_t m = 0u;
    if (j < n_whole) {
#pragma unroll
      for (int g = 0; g < G; ++g)
        m |= ((rows[g][j >> 5] >> (j & 31)) & 1u) << g;
    }
    return (int)m;
  };
  constexpr int kMine = kQuadMaxTiles / 64 / kQuadWaves;  // segments of a wave
  int mine[kMine];
#pragma unroll
  for (int i = 0; i < kMine; ++i) mine[i] = class_of(wave + kQuadWaves * i);
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    const int seg = wave + kQuadWaves * i;
    if (seg >= n_seg) break;
    int count = 0;
#pragma unroll
    for (int c = 1; c <= NC; ++c) {
      const int cnt = __popcll(__builtin_amdgcn_ballot_w64(mine[i] == c));
      if (lane == c) count = cnt;
    }
    if (lane < 16) sh.counts()[seg * 16 + lane] = count;
  }
  __syncthreads();
  int total = 0, begin = 0;
  if (wave == 0) {
    if (lane < 16)
      for (int seg = 0; seg < n_seg; seg += 8) {  // (counts beyond the last segment are not used)
        int t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = seg + i < n_seg ? sh.counts()[(seg + i) * 16 + lane] : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (seg + i < n_seg) sh.counts()[(seg + i) * 16 + lane] = total;
          total += t[i];
        }
      }
    int sum = total;  // inclusive prefix over the classes
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const int up = __shfl_up(sum, d);
      if (lane >= d) sum += up;
    }
    begin = sum - total;
    if (lane < 16) sh.begin[lane] = begin;
  }
  __syncthreads();
  if (wave == 0) {
    // the classes in the order in which they are taken: lane i stands for class number (order >> 4 i) & 15
    constexpr uint64_t order = 0x842169A5C3EDB7Full;
    auto class_at = [&](int i) -> int { return (int)(order >> (4 * i)) & 15; };
    const int c = lane < NC ? class_at(lane) : 0;
    int left = __shfl(total, c), at = __shfl(begin, c);
    int apart = 0;  // lanes whose class shares no group with this one
#pragma unroll
    for (int i = 0; i < NC; ++i)
      if ((class_at(i) & c) == 0) apart |= 1 << i;
    int steps_of[5] = {0, 0, 0, 0, 0}, parts = 0, idle_runs = 0;
    for (;;) {
      const uint32_t all = (uint32_t)__builtin_amdgcn_ballot_w64(lane < NC && left > 0);
      if (all == 0u) break;
      uint32_t taken = 0u;
      int steps = 0x7fffffff, n = 0, groups = 0;
      for (uint32_t may = all; may != 0u;) {
        const int i = __builtin_ctz(may);
        taken |= 1u << i;
        steps = min(steps, __builtin_amdgcn_readlane(left, i));
        groups |= class_at(i);
        ++n;
        may &= (uint32_t)__builtin_amdgcn_readlane(apart, i);
      }
      const bool full = groups == NC;
      int from = idle_runs;
#pragma unroll
      for (int k = 1; k <= 4; ++k)
        if (full && k == n) {
          from = steps_of[k];
          steps_of[k] += steps;
        }
      if (!full) {
        if (lane == 0) sh.runs[pipes::kQuadKinds + idle_runs] = QuadRun{steps, n, n, 0};
        ++idle_runs;
      }
      // single classes of a step in the order of the groups: with four of them a group's tile has the group's number
      const int j = __popc(taken & ((1u << (lane & 31)) - 1u));
      if (lane < NC && ((taken >> lane) & 1u)) {
        sh.parts[parts + j] = make_int4(at, steps, from, j | n << 4 | (full ? 0 : 1 << 7) | c << 8);
        left -= steps;
        at += steps;
      }
      parts += n;
    }
    if (lane == 0) {
      // steps of one tile alternate with those of four, then with those of three
      const int with4 = min(steps_of[4], steps_of[1]), with3 = min(steps_of[3], steps_of[1] - with4);
      const int steps[pipes::kQuadKinds] = {steps_of[1] - with4 - with3, steps_of[2], 2 * with3, 2 * with4, steps_of[3] - with3, steps_of[4] - with4};
      sh.alternating[0] = with3;
      sh.alternating[1] = with4;
      int base = 0;
#pragma unroll
      for (int k = 0; k < pipes::kQuadKinds; ++k) {
        sh.runs[k] = QuadRun{steps[k], pipes::kQuadEven[k], pipes::kQuadOdd[k], base};
        base += (pipes::kQuadEven[k] + pipes::kQuadOdd[k]) * steps[k] / 2;
      }
      for (int r = pipes::kQuadKinds; r < pipes::kQuadKinds + idle_runs; ++r) {
        sh.runs[r].base = base;
        base += sh.runs[r].steps * sh.runs[r].even;
      }
      sh.n_parts = parts;
      sh.n_runs = pipes::kQuadKinds + idle_runs;
    }
  }
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    const int seg = wave + kQuadWaves * i, m = mine[i];
    if (seg >= n_seg) break;
    int rank = 0;
#pragma unroll
    for (int c = 1; c <= NC; ++c) {
      const uint64_t same = __builtin_amdgcn_ballot_w64(m == c);
      if (m == c) rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
    }
    if (m) {
      sh.sorted()[sh.begin[m] + sh.counts()[seg * 16 + m] + rank] = (uint16_t)(64 * seg + lane);
    }
  }
  __syncthreads();
  const int with3 = sh.alternating[0], with4 = sh.alternating[1];
  for (int e = wave; e < sh.n_parts; e += kQuadWaves) {
    const int4 part = sh.parts[e];
    const int j = part.w & 15, n = (part.w >> 4) & 7, bits = (part.w >> 8) << 12;
    for (int i = lane; i < part.y; i += 64) {
      int k = part.z + i, to;  // k-th step of n tiles
      if ((part.w >> 7) & 1) to = sh.runs[pipes::kQuadKinds + part.z].base + i * n + j;
      else if (n == 1) to = k < with4 ? sh.runs[3].base + 5 * k + 4 : k < with4 + with3 ? sh.runs[2].base + 4 * (k - with4) + 3 : sh.runs[0].base + k - with4 - with3;
      else if (n == 2) to = sh.runs[1].base + 2 * k + j;
      else if (n == 3) to = k < with3 ? sh.runs[2].base + 4 * k + j : sh.runs[4].base + 3 * (k - with3) + j;
      else to = k < with4 ? sh.runs[3].base + 5 * k + j : sh.runs[5].base + 4 * (k - with4) + j;
      sh.list[to] = (uint16_t)(sh.sorted()[part.x + i] | bits);
    }
  }
  __syncthreads();
}

// All steps of the plan.
struct QuadPasses {
  QuadShared& sh;
  const char* const kb;
  const char* const vb;
  const uint32_t row_bytes;
  const int group, wave, lane;
  const float c;
  uint32_t ring;
  uint32_t kl[4], vl[4];  // lane offsets in a half slot of row and column fragments (see quad_loads in gen_mfma_pipes.py)
  uint32_t x;             // byte offset, in a half tile, of the lane's 16 bytes of the wave's load
  int steps, even, odd, base;  // the run

  PASA_DEVICE QuadPasses(QuadShared& sh, const uint16_t* kb, const uint16_t* vb, uint32_t row_bytes, int group, int wave, int lane, float c)
      : sh(sh), kb(uniform(kb)), vb(uniform(vb)), row_bytes((uint32_t)uniform((int)row_bytes)), group(uniform(group)), wave(uniform(wave)),
        lane(lane), c(c) {
    ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)sh.ring;
    const int h = lane >> 5, i = lane & 15, row = lane & 31, block = pipes::kQuadBlock;
    const uint32_t k0 = (uint32_t)((row >> 2) * block + (row & 3) * 256 + h * 16);
    const uint32_t v0 = (uint32_t)(h * block + (i >> 2) * 256 + ((lane >> 4) & 1) * 32 + (i & 3) * 8);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      kl[j] = k0 + (uint32_t)((j ^ (row & 3)) * 64);
      vl[j] = v0 + (uint32_t)((j ^ (i >> 2)) * 64);
    }
    x = (uint32_t)(wave * 4 + (lane >> 4)) * this->row_bytes + (uint32_t)((i ^ ((lane >> 4) << 2)) * 16);
  }

  PASA_DEVICE uint32_t list_addr(int entry) const {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(char*)(sh.list + base + entry);
  }
  // byte offset of the lane's part of the tile of a list entry
  PASA_DEVICE uint32_t tile(int entry) const { return (uint32_t)(entry & 0xfff) * (64u * row_bytes) + x; }

  PASA_DEVICE int tiles_of(int t) const { return (t & 1) ? odd : even; }
  PASA_DEVICE int first_of(int t) const { return (t >> 1) * (even + odd) + ((t & 1) ? even : 0); }
  PASA_DEVICE int entry(int e) const { return uniform((int)sh.list[base + e]); }
  // Requests batch g of the run into batch slot `slot`: K halves of step g / 2, V halves of the step before it.
  PASA_DEVICE void request(int g, int slot) {
    const int t = g >> 1;
    const uint32_t half = (g & 1) ? 32u * row_bytes : 0u;
    uint32_t dst = ring + (uint32_t)(slot * (even + odd) * kQuadHalf + wave * pipes::kQuadBlock);
    const int nk = tiles_of(t), nv = t > 0 ? tiles_of(t - 1) : 0, k0 = first_of(t), v0 = k0 - nv;
#pragma unroll 1
    for (int j = t < steps ? 0 : nk; j < nk + nv; ++j)
      dma_1k((j < nk ? kb : vb) + half, tile(entry(j < nk ? k0 + j : v0 + j - nk)), dst + (uint32_t)(j * kQuadHalf));
  }
  // place of the group's tile among those of step t, or -1
  PASA_DEVICE int own(int t) const {
    int found = -1;
    if (t < steps)
      for (int j = tiles_of(t) - 1; j >= 0; --j)
        if ((entry(first_of(t) + j) >> (12 + group)) & 1) found = j;
    return uniform(found);
  }

  PASA_DEVICE static void meet() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

  // All steps of one run.  Batch g: step g / 2 - 1, half g & 1; 2 steps + 2 of them.  Batches 0 and 1 have no V tiles, the last two no K tiles.
  PASA_DEVICE void run(int kind, const bf16x8 (&qf)[8], f32x16 (&o)[4], float& m, float& l) {
    const int width = even + odd, depth = kQuadSlots / width, last = 2 * steps + 2;
    const uint32_t batch = (uint32_t)(width * kQuadHalf), wp = (uint32_t)(wave * pipes::kQuadBlock);
    meet();  // every wave is done with the ring
    for (int i = 0; i < depth && i < last; ++i) request(i, i);
    const int mine0 = own(0), active = mine0 >= 0;  // (the groups of a run are the same in all of its steps)
    auto k_at = [&](int place) -> uint32_t { return (uint32_t)((active ? place : 0) * kQuadHalf); };
    pipes::QuadState st;
    st.s0 = st.s1 = f32x16{0};
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) st.p0[i][e] = st.p1[i][e] = (__bf16)0.f;
    st.corr = 1.f;
    meet();
    pipes::quad_start0(uniform(active), (uint32_t)uniform((int)(ring + k_at(mine0))), kl, qf, m, l, st, c);
    meet();
    if (depth < last) request(depth, 0);
    pipes::quad_start1(uniform(active), (uint32_t)uniform((int)(ring + batch + k_at(mine0))), kl, qf, m, l, st, c);
    int g = 2, slot = 2 % depth;
    // whole steps that request whole batches only (all that are in flight meanwhile are whole ones)
    {
      pipes::QuadSteady t;
      const int count = uniform(!active ? 0 : even == odd ? max(0, (2 * steps - 1 - depth) >> 1) : max(0, (2 * steps - 1 - depth) >> 2));
      t.count = count;
      // `have`: the step whose tiles the first request, or the one before it, needs
      const int have = ((g + depth - 1) >> 1) - (depth & 1);
      const int nk = tiles_of(have), nv = have > 0 ? tiles_of(have - 1) : 0, k0 = first_of(have);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        t.xk[j] = j < nk && count > 0 ? tile(entry(k0 + j)) : 0u;
        t.xv[j] = j < nv && count > 0 ? tile(entry(k0 - nv + j)) : 0u;
      }
      t.la = list_addr(k0 + nk);
      t.lc = list_addr(width);
      t.ko = (uint32_t)uniform((int)k_at(own(1)));
      t.vo = (uint32_t)uniform((int)(tiles_of(1) * kQuadHalf + k_at(mine0)));
      t.sb = (uint32_t)uniform((int)(ring + slot * batch));
      t.ld = (uint32_t)uniform((int)(ring + ((slot == 0 ? depth : slot) - 1) * batch + wp));
      const uint32_t half = 32u * row_bytes;
      pipes::quad_steady(uniform(kind), ring, (uint32_t)uniform((int)(ring + depth * batch)), wp, (uint32_t)(12 + group), (uint32_t)(group * kQuadHalf), kl, qf, vl, o,
                         m, l, st, c, kb, kb + half, vb, vb + half, x, 64u * row_bytes, t);
      g += (even == odd ? 2 : 4) * count;
      slot = g % depth;
    }
    auto next = [&]() {  // requests the batch that takes the slot of the one before
      if (g + depth - 1 < last) request(g + depth - 1, slot == 0 ? depth - 1 : slot - 1);
    };
    int k_own = own(g >> 1), v_own = own((g >> 1) - 1);
    auto sk = [&]() -> uint32_t { return (uint32_t)uniform((int)(ring + slot * batch + k_at(k_own))); };
    auto sv = [&]() -> uint32_t { return (uint32_t)uniform((int)(ring + slot * batch + tiles_of(g >> 1) * kQuadHalf + k_at(v_own))); };
    auto advance = [&]() {
      ++g;
      slot = slot + 1 == depth ? 0 : slot + 1;
    };
#pragma unroll 1
    while (g < 2 * steps) {
      meet();
      next();
      pipes::quad_half0(uniform(active), sk(), sv(), kl, qf, vl, o, m, l, st, c);
      advance();
      meet();
      next();
      pipes::quad_half1(uniform(active), sk(), sv(), kl, qf, vl, o, m, l, st, c);
      advance();
      v_own = k_own;
      k_own = own(g >> 1);
    }
    meet();
    next();
    pipes::quad_end0(uniform(active), sv(), vl, o, m, l, st, c);
    advance();
    meet();
    pipes::quad_end1(uniform(active), sv(), vl, o, m, l, st, c);
  }

  PASA_DEVICE void all(const bf16x8 (&qf)[8], f32x16 (&o)[4], float& m, float& l) {
    const int n_runs = uniform(sh.n_runs);
#pragma unroll 1
    for (int r = 0; r < n_runs; ++r) {
      steps = uniform(sh.runs[r].steps);
      even = uniform(sh.runs[r].even);
      odd = uniform(sh.runs[r].odd);
      base = uniform(sh.runs[r].base);
      // (a run with idle groups: as of its kind, were there none)
      if (steps > 0) run(r < pipes::kQuadKinds ? r : even == 1 ? 0 : even == 2 ? 1 : 4, qf, o, m, l);
    }
  }
};

}  // namespace
