// top_a and gsgd of a few workers on long rows in ONE pass over the state (compress-then-mix order, direct
// form).
//
// The two-pass forms read x, xhat and g for the candidates or the norms and, when the threshold or the
// norm of every row is known, read all three again for the update of xhat and the mix.  But where few
// entries are sent - the k largest, or those of a long vector whose level is not zero - xhat does not
// change in most columns, and these can be mixed at once: 16 bytes per entry instead of 28 (top_a) or 32
// (gsgd).  A column in which some worker may have something to send is recorded (x' after the local
// update and xhat of all workers) and done again from its record when the row's figure is known.
//   k_onepass_mix      the pass.  top_a: lists as candidates the entries at or above the guess and mixes
//                      with those kept that it expects to be (|v| at or above a threshold predicted from
//                      the steps before).  gsgd: adds up the norms, marks the entries whose level is not
//                      zero by a bound on s / ||v||
//   k_onepass_list     top_a: the candidate lists of the rows out of the records
//   k_onepass_restore  top_a, normally idle; where a row's list turns out not to hold its k largest entries:
//                      x' and xhat back as they were before the mix, for the fallback and its row scans
//   (top_a: the fallback and the exact select of the two-pass form, on the lists; gsgd: the upper levels of
//   the norm trees)
//   k_onepass_finish   top_a: the recorded columns whose kept set is not the expected one; tiles left unmixed
//   k_onepass_encode   gsgd: the recorded columns; tiles left unmixed; everything where a bound did not hold
// Every bit of the result is that of the two-pass form.  x' is x_mixed - gamma acc (acc is formed again from
// the same xhat) but for some units in the last place, in about |gamma acc / x'| of the entries; the pass
// tries it and stores the difference, a byte per entry, for the rows of a tile that have one, and records
// the columns where a byte does not hold it.  (n = 8, d = 28 M, xhat near x and apart by a few percent of it
// between workers forty steps before, us per step by gamma 0.002 | 0.02 | 0.1 | 0.3: top_a 675 | 693 | 767 | 770, two
// passes 1043-1049; gsgd 751 | 807 | 820 | 806, two passes 1168-1175.  Columns recorded instead filled the slots from
// gamma acc / x' of a percent on.)  A tile with more than kRecSlots columns to record is left unmixed and done by the last kernel
// (top_a: its candidates go to the lists one by one).
#pragma once

#include "choco_kernels.h"

namespace choco {

// What the one-pass kernels need beside the argument block of all.
struct OnePassState {
  uint32_t redo_all;    // top_a: X holds x - lr g everywhere: every tile is mixed by the last kernel
  uint32_t open_step;   // (low word of the) last step in which a tile was left unmixed
  uint32_t failures;    // of what the pass went by, lately (judge_step)
};
constexpr uint32_t kHeldFailures = 1, kHeldWide = 2;   // OnePassCtl::held
struct OnePass {
  float2* recs;         // tiles x kRecSlots x n: x' and xhat of all workers in the recorded columns
  uint32_t* cols;       // tiles x 8: which columns of the tile are recorded; all bits: the tile was left unmixed
  int8_t* ulps;         // n x ld: bits of x' less those of x_mixed - gamma acc, in the rows of tiles that are marked in
  uint8_t* uneven;      // tiles: bit r: row r of the tile has such differences
  OnePassState* state;
  float marked_per_row; // gsgd: columns of a tile that a row is expected to mark where the bound is s / ||v|| itself
};

// Slots per tile of 256 columns.  A slot is 8 n bytes, so the records are a quarter of an array of the
// state; at 5 expected columns per tile (n = 8, k / d = 0.001) no tile in 10^6 has more than 20.
constexpr int kRecSlots = 32;
// A row per wave, n lanes of a group of eight where records are read, a byte per row in a word of marks: the form ends
// at eight workers by this layout (wider ones, where n k / d is as small, have not been built or measured).
constexpr int kOnePassRows = 8;
constexpr int kRecTiles = 16;       // tiles whose records a wave goes through together
constexpr float kWide = 28.0f;      // gsgd: columns that a tile is expected to have marked above which all tiles are left open

// Columns of the lane's 4-vector that some wave marked (a byte per wave).
__device__ __forceinline__ uint32_t fold_marks(uint64_t m) {
  m |= m >> 32;
  m |= m >> 16;
  m |= m >> 8;
  return (uint32_t)m & 0xFu;
}

// (x', xhat) of worker 0 in a slot; worker i's is i further on.
__device__ __forceinline__ float2* record_of(const Args& A, const OnePass& P, int64_t tile, int slot) {
  return P.recs + (tile * kRecSlots + slot) * A.n;
}

// A tile that was left unmixed has all bits of its mask set (a recorded one no more than kRecSlots).
__device__ __forceinline__ bool left_open(uint2 w) { return (w.x & w.y) == 0xFFFFFFFFu; }
static_assert(kRecSlots < 64, "two full words of a mask mean an open tile");

// top_a: the step is the first after choco_init, there is no threshold to go by (the guess lies above every key;
// the rows get theirs all in the same step).  The device tells, not the host: a first step that was captured
// into a graph is an ordinary one when it is replayed (n = 8, d = 12 M: 1616 us a replay when each went as a
// first step, 361 as it is; two passes 478).
__device__ __forceinline__ bool no_guess_yet(uint32_t guess_key) { return guess_key == 0xFFFFFFFFu; }

// top_a, a tile left open: the row's candidates in it (bits `cand` of the lane's 4-vector v) straight to the list.
__device__ __forceinline__ void list_here(const Args& A, int r, int tile_no, uint32_t cand, vf4 v, int e) {
  const int seg = tile_no % kSegs;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if ((cand >> c) & 1u) {
      const uint32_t at = atomicAdd(seg_counter(A, r, seg), 1u);
      if (at < A.seg_cap) A.cand[((int64_t)r * kSegs + seg) * A.seg_cap + at] = make_uint2(__float_as_uint(v[c]), (uint32_t)(e + c));
    }
}

// A step whose threshold or bound fails costs the pass, its undoing and the second form; where that happens to
// about every other step it is better to leave all tiles unmixed and do them once (16 bytes per entry here and
// 16 in the last kernel, as many as two passes take).  A failure counts two and a step that went well takes one
// back, up to kHeldMost; tiles are left open from kHeldFrom on, down to kHeldTo.  gsgd also leaves them for one step
// when its bound is so wide that nearly as many columns are going to be marked as there are slots for (top_a's next
// list does not follow from this one's length).
//   us per step, n = 8, d = 12 M: two passes | one pass always | as here
//   gsgd, the gradient step to and fro (norms by 5)   503 | 788 | 590    every other pair of steps 503 | 517 | 473
//         to or fro by chance                         503 | 384 | 374    a tenth of the entries moving 507 | 364 | 358
//   top_a, the gradient step to and fro (all lists fail) 1773 | 1888 | 1657   by chance 1191 | 1317 | 1238
// (The last kernel's whole tiles are bound by the encoding's arithmetic, with Philox, and by two workgroups of its 95
// registers to a compute unit: 336 us for what k_dense_apply_mix does in 351 with the gradients to read again.)
// One thread calls it, after k_onepass_mix has read the state and before the next step's does.
constexpr int kHeldFrom = 6, kHeldTo = 2, kHeldMost = 12;
__device__ __forceinline__ void judge_step(const Args& A, OnePassState* S, bool failed, bool wide) {
  const int count = failed ? min((int)S->failures + 2, kHeldMost) : max((int)S->failures - 1, 0);
  S->failures = (uint32_t)count;
  const bool was = onepass_ctl(A)[0].held == kHeldFailures;
  const uint32_t held = count >= kHeldFrom || (was && count > kHeldTo) ? kHeldFailures : wide ? kHeldWide : 0u;
  for (int i = 0; i < A.n; ++i) onepass_ctl(A)[i].held = held;
}

// grid ceil(d / 256), block 64 n (wave r: row r), dynamic LDS n x 256 floats.
template <int COMP>
__global__ __launch_bounds__(64 * kOnePassRows) void k_onepass_mix(Args A, OnePass P) {
  extern __shared__ float tile[];
  __shared__ uint64_t marks[64];   // a byte per lane and wave
  __shared__ float2 recs[kRecSlots * kOnePassRows];
  const int r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tile_no = (int)blockIdx.x;   // (line_sharing_tile: top_a 612 against 604 us at n = 8, d = 28 M)
  const int e = tile_no * kChunk + lane * 4;
  const bool mine = e < A.d;
  const int64_t o = (int64_t)r * A.ld + e;
  const bool mom = A.G != nullptr && A.M != nullptr;
  vf4 x = {0.f, 0.f, 0.f, 0.f}, h = x, g = x, m = x;
  if (mine) {
    x = load4<true>(A.X + o);
    h = load4<true>(A.Xhat + o);
    if (A.G) g = load4<true>(A.G + o);
    if (mom) m = load4<true>(A.M + o);
  }
  const RowSpan span = nbr_span<1, kOnePassRows>(A, r, lane);
  const uint32_t guess = A.ctl[r].guess_key, expect = onepass_ctl(A)[r].expect_key;
  const float bound = onepass_ctl(A)[r].bound_r;
  const bool held = onepass_ctl(A)[r].held != 0u;
  if (r == 0) marks[lane] = 0u;    // (bytes of rows that there are not)
  uint4 words = make_uint4(0, 0, 0, 0);
  if (COMP == Q_QSGD) words = random_words(A, r, (uint32_t)(e >> 2), STREAM_DITHER);
  const RowNbrs nb = nbr_fetch(A, span, lane);
  if (mine && A.G) {
    x = local_update_regs(A, x, g, m);
    if (mom) store4<true>(A.M + o, m);
  }
  if (COMP == Q_TOPK && no_guess_yet(guess)) {   // the last kernel does all tiles
    if (mine && A.G) store4<true>(A.X + o, x);
    return;
  }
  vf4 hn = h;
  uint32_t cand = 0u, kept = 0u;
  if (mine) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float q = x[c] - h[c];
      if (COMP == Q_TOPK) {
        const uint32_t key = __float_as_uint(q) & 0x7fffffffu;
        if (e + c < A.d && key >= guess) {
          cand |= 1u << c;
          if (key >= expect) {
            kept |= 1u << c;
            hn[c] = h[c] + q;
          }
        }
      } else {
        // (rounding is monotonic: no level is above zero that is not by the larger factor; and adding
        // the zero that a level of zero stands for changes an xhat of -0)
        if (e + c < A.d && (fabsf(q) * bound + dither_of(pick(words, c)) >= 1.0f || __float_as_uint(h[c]) == 0x80000000u))
          cand |= 1u << c;
      }
    }
  }
  if (COMP == Q_QSGD) {
    const double t = wave_tree_sum_lds(mine ? lane_terms<Q_QSGD>(x - h, e, A.d) : 0.0);
    if (lane == 0) A.chunk_sums[(int64_t)r * A.nchunks + tile_no] = t;
  }
  if (held) {
    if (mine && A.G) store4<true>(A.X + o, x);
    if (COMP == Q_TOPK) list_here(A, r, tile_no, cand, x - h, e);
    if (r == 0 && (lane & 7) == 0) P.cols[(int64_t)tile_no * 8 + (lane >> 3)] = 0xFFFFFFFFu;
    if (tile_no == 0 && threadIdx.x == 0) P.state->open_step = A.t_lo;
    return;
  }
  lds_store4(tile + r * kChunk + lane * 4, hn);
  __syncthreads();
  vf4 xm = x;
  uint32_t lost = 0u, ulps = 0u;
  const vf4 acc = mix_sum_staged<0>(A, tile, r, lane, nb);
  if (mine) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float step = A.gamma * acc[c];
      xm[c] = x[c] + step;
      const float back = xm[c] - step;
      const int32_t off = (int32_t)(__float_as_uint(x[c]) - __float_as_uint(back));
      if (off != (int32_t)(int8_t)off) lost |= 1u << c;
      else ulps |= (uint32_t)(off & 0xFF) << (8 * c);
    }
  }
  const bool uneven = __ballot(ulps != 0u) != 0ull;
  if (uneven && mine) *reinterpret_cast<uint32_t*>(P.ulps + o) = ulps;
  reinterpret_cast<uint8_t*>(marks)[lane * 8 + r] = (uint8_t)(cand | lost | (uneven ? 0x10u : 0u));
  __syncthreads();
  const uint32_t dirty = fold_marks(marks[lane]);
  uint64_t db[4];
  int total = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    db[c] = __ballot((dirty >> c) & 1u);
    total += __popcll(db[c]);
  }
  const bool open = total > kRecSlots;     // the same in every wave
  if (mine) {
    store4<true>(A.X + o, open ? x : xm);
    if (COMP == Q_TOPK && kept && !open) store4<false>(A.Xhat + o, hn);
    if (COMP == Q_QSGD && A.codes) *reinterpret_cast<vi4*>(A.codes + o) = vi4{0, 0, 0, 0};
  }
  if (r == 0) {
    const uint32_t w = mask_word(open ? 0xFu : dirty, lane);
    if ((lane & 7) == 0) P.cols[(int64_t)tile_no * 8 + (lane >> 3)] = w;
    if (lane == 0)   // (bit 4 of the rows' bytes, side by side)
      P.uneven[tile_no] = (uint8_t)((((marks[0] >> 4) & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56);
    if (open && lane == 0) P.state->open_step = A.t_lo;
  }
  if (open) {
    if (COMP == Q_TOPK) list_here(A, r, tile_no, cand, x - h, e);
  } else if (mine && dirty != 0u) {
    const uint64_t below = (1ull << lane) - 1ull;
    int slot = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) slot += __popcll(db[c] & below);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if ((dirty >> c) & 1u) recs[slot++ * A.n + r] = make_float2(x[c], h[c]);
  }
  if (open) return;
  // (by way of LDS, whole records at a time: 616 against 623 us for gsgd at n = 8, d = 28 M, top_a 602 against 607)
  __syncthreads();
  for (int j = threadIdx.x; j < total * A.n; j += (int)blockDim.x) record_of(A, P, tile_no, 0)[j] = recs[j];
}

// The marked columns of the kRecTiles tiles from t0 on, to LDS as (tile of the sixteen x slots + slot,
// column in the tile); returns how many.  A whole wave calls it: four lanes to a tile, two words of its
// mask each.
__device__ __forceinline__ uint32_t list_marked(const OnePass& P, int t0, int ntiles, ushort2* out) {
  const int lane = threadIdx.x & 63;
  const int t = t0 + (lane >> 2);
  uint2 w = make_uint2(0u, 0u);
  if (t < ntiles) w = *reinterpret_cast<const uint2*>(P.cols + (int64_t)t * 8 + 2 * (lane & 3));
  if (left_open(w)) w = make_uint2(0u, 0u);
  const uint32_t cnt = (uint32_t)(__popc(w.x) + __popc(w.y));
  const uint32_t incl = wave_scan(cnt);
  uint32_t at = incl - cnt;
  uint32_t slot = at - __shfl(at, lane & ~3, 64);
  uint64_t bits = ((uint64_t)w.y << 32) | w.x;
  while (bits) {
    const int b = __ffsll((unsigned long long)bits) - 1;
    bits &= bits - 1;
    out[at++] = make_ushort2((unsigned short)((lane >> 2) * kRecSlots + slot++), (unsigned short)(64 * (lane & 3) + b));
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return __shfl(incl, 63, 64);
}

// Record f of the listed ones, as lane i of its group sees it.
struct Recorded {
  float x, h;
  int col;
  bool have;    // there is such a record, and the lane stands for a worker in it
};
__device__ __forceinline__ Recorded recorded(const Args& A, const OnePass& P, int t0, const ushort2* list, uint32_t f, uint32_t total, int i) {
  Recorded R{0.0f, 0.0f, 0, false};
  if (f < total) {
    const int ts = list[f].x, t = t0 + ts / kRecSlots;
    R.col = t * kChunk + list[f].y;
    R.have = i < A.n && R.col < A.d;
    if (R.have) {
      const float2 v = record_of(A, P, t, ts % kRecSlots)[i];
      R.x = v.x;
      R.h = v.y;
    }
  }
  return R;
}

// Eight lanes to a record, lane i of them for worker i, with its row of W in registers.
struct RecordLanes {
  int i, grp, lane, deg;
  uint32_t near;      // the workers that this one mixes with, itself among them
  bool row;
  int nc[kOnePassRows];
  float nw[kOnePassRows];
  __device__ __forceinline__ RecordLanes(const Args& A, int lane_) : i(lane_ & 7), grp(lane_ >> 3), lane(lane_) {
    row = i < A.n;
    const int pbeg = row ? A.row_ptr[i] : 0;
    deg = row ? A.row_ptr[i + 1] - pbeg : 0;
    near = 0;
#pragma unroll
    for (int j = 0; j < kOnePassRows; ++j) {
      nc[j] = j < deg ? A.col[pbeg + j] : 0;
      nw[j] = j < deg ? A.w[pbeg + j] : 0.0f;
      if (j < deg) near |= 1u << nc[j];
    }
  }
  // Does x of the lane's worker change with these lanes' xhat?  (A worker none of whose neighbours sent
  // anything else than the pass went by has its x already: on a ring five of eight, and the scattered
  // stores are what the last kernel takes its time for.)
  __device__ __forceinline__ bool concerned(uint64_t lanes) const {
    return (((uint32_t)(lanes >> (lane & ~7))) & near) != 0u;
  }
  // sum_p w_p (xhat_j - xhat_i) in a record whose lanes hold xhat; all lanes of the wave call it
  __device__ __forceinline__ float mix_sum(float h) const {
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < kOnePassRows; ++j) {
      const float other = __shfl(h, (lane & ~7) + nc[j], 64);
      if (j < deg) acc = acc + nw[j] * (other - h);
    }
    return acc;
  }
};

// The candidates among the recorded entries, to the rows' lists: each wave counts those of its sixteen
// tiles row by row, takes room with one addition per row and writes them.  grid any, block 256.
__global__ __launch_bounds__(256) void k_onepass_list(Args A, OnePass P, int32_t ntiles) {
  __shared__ ushort2 lists[4][kRecTiles * kRecSlots];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 7, grp = lane >> 3;
  ushort2* list = lists[wave];
  const uint32_t guess = A.ctl[i < A.n ? i : 0].guess_key;
  const int w0 = (int)blockIdx.x * 4 + wave, nwaves = (int)gridDim.x * 4;
  for (int t0 = w0 * kRecTiles; t0 < ntiles; t0 += nwaves * kRecTiles) {
    const uint32_t total = list_marked(P, t0, ntiles, list);
    auto is_candidate = [&](const Recorded& R) {
      return R.have && (__float_as_uint(R.x - R.h) & 0x7fffffffu) >= guess;
    };
    uint32_t mine = 0;
#pragma unroll 4
    for (uint32_t f = (uint32_t)grp; f < total; f += 8) mine += is_candidate(recorded(A, P, t0, list, f, total, i)) ? 1u : 0u;
    uint32_t incl = mine;     // over the eight lanes of a row
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) {
      const uint32_t up = __shfl_up(incl, off, 64);
      if (lane >= off) incl += up;
    }
    const int seg = (t0 / kRecTiles) % kSegs;
    uint32_t base = 0;
    if (grp == 7 && incl != 0u) base = atomicAdd(seg_counter(A, i, seg), incl);
    base = __shfl(base, 56 + i, 64) + incl - mine;
    if (mine != 0u) {
      uint2* out = A.cand + ((int64_t)i * kSegs + seg) * A.seg_cap;
#pragma unroll 4
      for (uint32_t f = (uint32_t)grp; f < total; f += 8) {
        const Recorded R = recorded(A, P, t0, list, f, total, i);
        if (is_candidate(R)) {
          if (base < A.seg_cap) out[base] = make_uint2(__float_as_uint(R.x - R.h), (uint32_t)R.col);
          ++base;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// x' and xhat of the lane's 4-vector as they were before k_onepass_mix mixed tile t (not an open one).  All
// waves of the workgroup call it, one row each; the LDS tile holds the old xhat afterwards.
__device__ __forceinline__ void take_back(const Args& A, const OnePass& P, float* tile, int t, int r, int lane, const RowNbrs& nb, vf4& x,
                                          vf4& h, bool& recorded_here) {
  const int e = t * kChunk + lane * 4;
  const bool mine = e < A.d;
  const int64_t o = (int64_t)r * A.ld + e;
  const uint32_t dirty = (P.cols[(int64_t)t * 8 + (lane >> 3)] >> (4 * (lane & 7))) & 0xFu;
  int slot = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) slot += __popcll(__ballot((dirty >> c) & 1u) & ((1ull << lane) - 1ull));
  vf4 xr = {0.f, 0.f, 0.f, 0.f};
  x = h = xr;
  if (mine) {
    x = load4<true>(A.X + o);
    h = load4<true>(A.Xhat + o);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if ((dirty >> c) & 1u) {
        const float2 v = record_of(A, P, t, slot++)[r];
        xr[c] = v.x;
        h[c] = v.y;
      }
  }
  recorded_here = mine && dirty != 0u;
  __syncthreads();                       // what the tile held before has been read
  lds_store4(tile + r * kChunk + lane * 4, h);
  __syncthreads();
  const vf4 acc = mix_sum_staged<0>(A, tile, r, lane, nb);
  uint32_t ulps = 0u;
  if (mine && ((P.uneven[t] >> r) & 1u)) ulps = *reinterpret_cast<const uint32_t*>(P.ulps + o);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float step = A.gamma * acc[c];
    const int32_t off = (int32_t)(int8_t)(ulps >> (8 * c));
    x[c] = ((dirty >> c) & 1u) ? xr[c] : __uint_as_float(__float_as_uint(x[c] - step) + (uint32_t)off);
  }
}

// Do all lists hold their row's k largest entries?  If not, what k_onepass_mix did to x and xhat is
// undone, tile by tile, so that X is x' everywhere.  Normally a launch of workgroups that read the
// lists' lengths and leave.  grid any, block 64 n, dynamic LDS n x 256 floats.
__global__ __launch_bounds__(64 * kOnePassRows) void k_onepass_restore(Args A, OnePass P, int32_t ntiles) {
  extern __shared__ float tile[];
  __shared__ uint32_t s_bad;
  const int r = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (threadIdx.x == 0) s_bad = 0u;
  const bool first = no_guess_yet(A.ctl[0].guess_key);
  __syncthreads();
  const uint32_t raw = lane < kSegs ? *seg_counter(A, r, lane) : 0u;
  unsigned long long sum = raw;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
  const bool fits = __ballot(raw > A.seg_cap) == 0ull;
  if (lane == 0 && (!fits || sum < (unsigned long long)A.k)) s_bad = 1u;
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    P.state->redo_all = s_bad;
    if (!first) judge_step(A, P.state, s_bad != 0u, false);
  }
  if (s_bad == 0u || first) return;   // (in the first step nothing has been mixed)
  const RowNbrs nb = nbr_fetch(A, nbr_span<1, kOnePassRows>(A, r, lane), lane);
  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const uint32_t* cols = P.cols + (int64_t)t * 8;
    if (left_open(make_uint2(cols[0], cols[1]))) continue;
    const int e = t * kChunk + lane * 4;
    const int64_t o = (int64_t)r * A.ld + e;
    vf4 x, h;
    bool changed;
    take_back(A, P, tile, t, r, lane, nb, x, h, changed);
    if (changed) store4<false>(A.Xhat + o, h);
    if (e < A.d) store4<true>(A.X + o, x);
  }
}

// The k kept entries of every row are known (composite key >= kstar).  Tiles that hold x' as a whole
// (all of them in a first step or after k_onepass_restore) get the update of xhat and the mix here; of
// the others the recorded columns whose kept set is not the one that k_onepass_mix went by.
// grid any, block 64 n, dynamic LDS n x 256 floats.
__global__ __launch_bounds__(64 * kOnePassRows) void k_onepass_finish(Args A, OnePass P, int32_t ntiles) {
  extern __shared__ float tile[];
  __shared__ ushort2 lists[kOnePassRows][kRecTiles * kRecSlots];
  const int r = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool all = P.state->redo_all != 0u;
  if (all || P.state->open_step == A.t_lo) {
    const RowNbrs nb = nbr_fetch(A, nbr_span<1, kOnePassRows>(A, r, lane), lane);
    const uint64_t kstar = A.ctl[r].kstar;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
      const uint32_t* cols = P.cols + (int64_t)t * 8;
      if (!all && !left_open(make_uint2(cols[0], cols[1]))) continue;
      const int e = t * kChunk + lane * 4;
      const bool mine = e < A.d;
      const int64_t o = (int64_t)r * A.ld + e;
      vf4 x = {0.f, 0.f, 0.f, 0.f}, h = x;
      if (mine) {
        x = load4<true>(A.X + o);
        h = load4<true>(A.Xhat + o);
        bool kept = false;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float q = x[c] - h[c];
          if (e + c < A.d && Digits<Q_TOPK>::composite(__float_as_uint(q), (uint32_t)(e + c)) >= kstar) {
            h[c] = h[c] + q;
            kept = true;
          }
        }
        if (kept) store4<false>(A.Xhat + o, h);
      }
      __syncthreads();
      lds_store4(tile + r * kChunk + lane * 4, h);
      __syncthreads();
      const vf4 acc = mix_sum_staged<0>(A, tile, r, lane, nb);
      if (mine) {
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = x[c] + A.gamma * acc[c];
        store4<true>(A.X + o, x);
      }
    }
    if (all) return;
  }
  const RecordLanes L(A, lane);
  const uint64_t kstar = A.ctl[L.row ? L.i : 0].kstar;
  const uint32_t expected = onepass_ctl(A)[L.row ? L.i : 0].expected_key;
  const int waves = (int)(blockDim.x >> 6), nwaves = (int)gridDim.x * waves;
  for (int t0 = ((int)blockIdx.x * waves + r) * kRecTiles; t0 < ntiles; t0 += nwaves * kRecTiles) {
    const uint32_t total = list_marked(P, t0, ntiles, lists[r]);
    constexpr int U = 4;       // records of a group in flight
    for (uint32_t f0 = 0; f0 < total; f0 += 8 * U) {
      Recorded R[U];
#pragma unroll
      for (int u = 0; u < U; ++u) R[u] = recorded(A, P, t0, lists[r], f0 + 8u * u + (uint32_t)L.grp, total, L.i);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float q = R[u].x - R[u].h;
        const uint32_t a = __float_as_uint(q);
        const bool now = R[u].have && Digits<Q_TOPK>::composite(a, (uint32_t)R[u].col) >= kstar;
        const bool was = R[u].have && Digits<Q_TOPK>::key32(a) >= expected;
        const uint64_t wrong = __ballot(now != was);
        if (wrong != 0ull) {                                    // (every lane takes part in the exchange)
          const float hn = now ? R[u].h + q : R[u].h;
          const float acc = L.mix_sum(hn);
          if (R[u].have && L.concerned(wrong)) {
            const int64_t o = (int64_t)L.i * A.ld + R[u].col;
            A.X[o] = R[u].x + A.gamma * acc;
            if (now != was) A.Xhat[o] = hn;
          }
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Zeros to the bit planes of the kRecTiles tiles from t0 on, but for open ones: a piece of 512 bytes per row
// and plane, two lanes to a tile.  (32 bytes per row, plane and tile out of k_onepass_mix
// made that kernel 75 us longer at n = 8, d = 28 M, five planes; here they take 37.)  The words belong to this wave alone
// until the kernel's end, so its bits need no more than the order among its own accesses.
__device__ __forceinline__ void clear_planes(const Args& A, const OnePass& P, int t0, int ntiles, int lane) {
  typedef uint32_t words4 __attribute__((ext_vector_type(4), aligned(4)));   // (a plane may have any number of words)
  const int t = t0 + ((lane & 31) >> 1);
  if (t >= ntiles) return;
  const uint32_t* cols = P.cols + (int64_t)t * 8;
  if (left_open(make_uint2(cols[0], cols[1]))) return;
  const int64_t word = (int64_t)t * 8 + 4 * (lane & 1), left = ((int64_t)A.d + 31) / 32 - word;
  for (int q = lane >> 5; q < A.n * A.nplanes; q += 2) {
    uint32_t* plane = A.planes + (int64_t)q * A.plane_words + word;
    if (left >= 4) *reinterpret_cast<words4*>(plane) = words4{0u, 0u, 0u, 0u};
    else
      for (int j = 0; j < left; ++j) plane[j] = 0u;
  }
}
__device__ __forceinline__ void set_bits(uint32_t* word, uint32_t bits) {
  (void)__hip_atomic_fetch_or(word, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// gsgd: the scales of every row are known.  Levels, xhat and bit planes of the recorded entries, and the mix
// of the columns in which a level is not zero.  Tiles left unmixed are done as a whole; all tiles are where
// the factor s / ||v|| came out above the bound that the pass went by, or ||v|| beyond fp32 (then even a
// level of zero has a value).  grid any, block 64 n, dynamic LDS n x 256 floats.
__global__ __launch_bounds__(64 * kOnePassRows) void k_onepass_encode(Args A, OnePass P, int32_t ntiles) {
  extern __shared__ float tile[];
  __shared__ ushort2 lists[kOnePassRows][kRecTiles * kRecSlots];
  const int r = threadIdx.x >> 6, lane = threadIdx.x & 63;
  bool all = false;
  float marked = 0.0f;   // columns of a tile that the next step is expected to mark
  for (int j = 0; j < A.n; ++j) {
    const float now = A.ctl[j].scale_r;
    all = all || !(now <= onepass_ctl(A)[j].bounded_r) || !(A.ctl[j].scale_step <= 3.402823466e38f);
    marked += P.marked_per_row * (now > 0.0f ? onepass_ctl(A)[j].bound_r / now : 0.0f);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) judge_step(A, P.state, all, marked > kWide);
  if (all || P.state->open_step == A.t_lo) {
    const RowNbrs nb = nbr_fetch(A, nbr_span<1, kOnePassRows>(A, r, lane), lane);
    RowScale<Q_QSGD> sc;
    sc.load(A.ctl + r);
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
      const uint32_t* cols = P.cols + (int64_t)t * 8;
      const bool open = left_open(make_uint2(cols[0], cols[1]));
      if (!all && !open) continue;
      const int e = t * kChunk + lane * 4;
      const bool mine = e < A.d;
      const int64_t o = (int64_t)r * A.ld + e;
      vf4 x = {0.f, 0.f, 0.f, 0.f}, h = x;
      if (!open) {
        bool changed;
        take_back(A, P, tile, t, r, lane, nb, x, h, changed);
      } else if (mine) {
        x = load4<true>(A.X + o);
        h = load4<true>(A.Xhat + o);
      }
      vf4 nh = h;
      vi4 code = {0, 0, 0, 0};
      if (mine) {
        nh = absorb<Q_QSGD>(x, h, sc, random_words(A, r, (uint32_t)(e >> 2), STREAM_DITHER), code);
        mask_padding(A.d - e < 4 ? A.d - e : 4, h, nh, code);
        store4<true>(A.Xhat + o, nh);
        if (A.codes) *reinterpret_cast<vi4*>(A.codes + o) = code;
      }
      emit_code_planes<Q_QSGD>(A, r, e, lane, code, 0);
      __syncthreads();
      lds_store4(tile + r * kChunk + lane * 4, nh);
      __syncthreads();
      const vf4 acc = mix_sum_staged<0>(A, tile, r, lane, nb);
      if (mine) {
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = x[c] + A.gamma * acc[c];
        store4<true>(A.X + o, x);
      }
    }
    if (all) return;
  }
  const RecordLanes L(A, lane);
  RowScale<Q_QSGD> sc;
  sc.load(A.ctl + (L.row ? L.i : 0));
  const int waves = (int)(blockDim.x >> 6), nwaves = (int)gridDim.x * waves;
  for (int t0 = ((int)blockIdx.x * waves + r) * kRecTiles; t0 < ntiles; t0 += nwaves * kRecTiles) {
    clear_planes(A, P, t0, ntiles, lane);
    const uint32_t total = list_marked(P, t0, ntiles, lists[r]);
    constexpr int U = 4;       // records of a group in flight
    for (uint32_t f0 = 0; f0 < total; f0 += 8 * U) {
      Recorded R[U];
#pragma unroll
      for (int u = 0; u < U; ++u) R[u] = recorded(A, P, t0, lists[r], f0 + 8u * u + (uint32_t)L.grp, total, L.i);
      if (f0 == 0) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");   // the zeros before the bits
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int32_t code = 0;
        float hn = R[u].h;
        if (R[u].have) {
          const uint4 words = random_words(A, L.i, (uint32_t)R[u].col >> 2, STREAM_DITHER);
          hn = R[u].h + encode<Q_QSGD>(R[u].x - R[u].h, sc, pick(words, R[u].col & 3), code);
        }
        const bool changed = __float_as_uint(hn) != __float_as_uint(R[u].h);
        const uint64_t any = __ballot(changed);
        if (any != 0ull) {                                       // (every lane takes part in the exchange)
          const float acc = L.mix_sum(hn);
          if (R[u].have && L.concerned(any)) {
            const int64_t o = (int64_t)L.i * A.ld + R[u].col;
            A.X[o] = R[u].x + A.gamma * acc;
            if (changed) A.Xhat[o] = hn;
          }
        }
        if (code != 0) {   // (sent whether or not xhat is too large to show it)
          if (A.codes) A.codes[(int64_t)L.i * A.ld + R[u].col] = code;
          const uint32_t bit = 1u << (R[u].col & 31);
          uint32_t* plane = A.planes + (int64_t)L.i * A.nplanes * A.plane_words + ((uint32_t)R[u].col >> 5);
          if (code < 0) set_bits(plane, bit);
          const int32_t mag = magnitude_sent(A, L.i, R[u].col, 0, code);
          for (int p = 0; p < A.mb; ++p)
            if ((mag >> p) & 1) set_bits(plane + (int64_t)(1 + p) * A.plane_words, bit);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

}  // namespace choco
