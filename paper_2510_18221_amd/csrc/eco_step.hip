// eco_step.hip -- world-dynamics kernels of one step, and the init kernels.
//
// Step order (the policy kernel in eco_forward.hip runs first and has already
// applied turns and made the forward-move claims on the pre-step occupancy):
//   k_move         winners move; EAT; step cost; death at energy <= 0; age
//                  (Sec. 3.2 "Resources and Agent Health", "Actions")
//   k_claim_cells  slot tiles: eligible parents claim the empty cell behind them
//                  (Sec. 3.2 "Actions": child placed directly behind the parent) and
//                  the winners are listed in slot order, the free slots are listed in ascending order (the recycled-slot
//                  free list), the survivors' sums; cell tiles: each empty cell
//                  regrows one unit with probability p (Sec. 3.2: energy slowly
//                  grows back) and the window channels of the next step
//   k_birth_commit births: child state + child weights = parent + sigma * N(0,1)
//                  (Sec. 3.3 mutation) into the recycled slot; slot tiles: the
//                  live list of the next step; the statistics record (App. E
//                  measurement interface) and the clock
// Each launch needs what the one before it wrote anywhere in the world, so three is
// the least without a barrier across the grid, and a launch of this size costs its
// chain of dependent loads (2 - 4 us, next to 1.7 us for an empty one) whatever
// little it does: the step after the policy kernel of the 256 x 256 ecology world
// with 4,213 agents took 35 us in seven launches (moves, claims + regrowth, two
// ranking passes, births, two compaction passes with the cell pass), 22 in four
// (a ranking pass between the claims and the births), 20 in three, and takes 18 us
// since the cell pass gives each thread one cell.
// Every contended write of a move is an atomicMin on a claim word; every other write
// goes to a unique slot or cell, so the integer state is independent of scheduling.
#include <algorithm>
#include <cstddef>
#include <mutex>

#include "eco_device.h"

namespace eco {

constexpr int kSlotTile = 256;   // slots per block in per-slot kernels
constexpr int kScanThreads = 1024;

// ---------------------------------------------------------------------------
// Small block helpers
// ---------------------------------------------------------------------------
// Wave-wide sums by DPP, the data-parallel lane moves of the VALU: lane i of
// each row of 16 lanes adds row lanes i - 1, i - 2, i - 4, i - 8 (taking 0 past
// the row's start), then rows 1 and 3 add the last lane of rows 0 and 2, and
// rows 2 and 3 the last lane of row 1.  Each step is a few VALU cycles where a
// lane shuffle goes through the LDS crossbar.  Every lane of the wave must be
// active.  64-bit values move as two 32-bit halves.
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dpp_move(T x) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(
        T, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)__builtin_bit_cast(uint32_t, x), CTRL, ROWS, 0xf, false));
  } else {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
  }
}

// Inclusive sum over lanes 0..lane of the wave (a fixed order for FP64).
template <typename T>
__device__ __forceinline__ T wave_scan(T x) {
  x += dpp_move<0x111, 0xf>(x);   // row_shr:1
  x += dpp_move<0x112, 0xf>(x);   // row_shr:2
  x += dpp_move<0x114, 0xf>(x);   // row_shr:4
  x += dpp_move<0x118, 0xf>(x);   // row_shr:8
  x += dpp_move<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
  x += dpp_move<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
  return x;
}

// x of lane l (the same l in every lane).
template <typename T>
__device__ __forceinline__ T lane_value(T x, int l) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_readlane((int)__builtin_bit_cast(uint32_t, x), l));
  } else {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
  }
}

template <int NT>
__device__ __forceinline__ unsigned long long block_sum_u64(unsigned long long v, unsigned long long* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_scan(v);
  if (lane == 63) red[wave] = v;
  __syncthreads();
  unsigned long long t = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) t += red[i];
  __syncthreads();
  return t;  // valid in thread 0
}

// Deterministic FP64 block sum: a fixed order within each wave, then waves in order.
template <int NT>
__device__ __forceinline__ double block_sum_f64(double v, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_scan(v);
  if (lane == 63) red[wave] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) t += red[i];
  __syncthreads();
  return t;  // valid in thread 0
}

// Exclusive scan of one u32 per thread over the block; returns the exclusive
// prefix, *total gets the block total (all threads).
template <int NT>
__device__ __forceinline__ uint32_t block_exscan(uint32_t v, uint32_t* red, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_scan(v);
  if (lane == 63) red[wave] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t run = 0;
    for (int i = 0; i < NT / 64; ++i) {
      const uint32_t t = red[i];
      red[i] = run;
      run += t;
    }
    red[NT / 64] = run;
  }
  __syncthreads();
  const uint32_t ex = red[wave] + inc - v;
  *total = red[NT / 64];
  __syncthreads();
  return ex;
}

// Sum of the per-wave values r_i (lane i of every wave holding r_i, i < NW,
// zero in the other lanes) over the waves before the calling one; *all gets the
// sum over all NW waves.  Every wave computes both the same way.
template <int NW, typename T>
__device__ __forceinline__ T waves_before(T r, T* all) {
  static_assert(NW >= 1 && NW <= 64, "at most 64 waves");
  const int wave = threadIdx.x >> 6;
  r = wave_scan(r);
  *all = lane_value(r, NW - 1);
  const T b = lane_value(r, wave > 0 ? wave - 1 : 0);
  return wave > 0 ? b : T(0);
}

// Exclusive scan of one u64 per thread over the block with one barrier: each
// wave reads the waves' totals from red itself.  red[NT / 64] must not be
// written again before every thread has returned (the caller's next barrier).
template <int NT>
__device__ __forceinline__ unsigned long long block_exscan_u64(unsigned long long v, unsigned long long* red,
                                                             unsigned long long* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long inc = wave_scan(v);
  if (lane == 63) red[wave] = inc;
  __syncthreads();
  const unsigned long long before = waves_before<NT / 64>(lane < NT / 64 ? red[lane] : 0ull, total);
  return before + inc - v;
}

// Block counters in LDS with one atomic per wave instead of one per lane (the
// atomics of a wave's lanes on one LDS address run one after another, several
// cycles each).  count_lanes: adds the number of the wave's active lanes to *c
// (called in the branch whose lanes are counted).  count_lanes_by<N>: adds, for
// each k < N, the number of active lanes whose v is k to c[k].  wave_add_u64:
// adds the sum of v over the wave to *c (every lane of the wave active).
__device__ __forceinline__ void count_lanes(uint32_t* c) {
  const uint64_t m = __ballot(1);
  if ((threadIdx.x & 63u) == (uint32_t)__builtin_ctzll(m)) atomicAdd(c, (uint32_t)__builtin_popcountll(m));
}

template <int N>
__device__ __forceinline__ void count_lanes_by(uint32_t* c, int v) {
  const uint32_t first = (uint32_t)__builtin_ctzll(__ballot(1));
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const uint64_t m = __ballot(v == k);
    if (m && (threadIdx.x & 63u) == first) atomicAdd(&c[k], (uint32_t)__builtin_popcountll(m));
  }
}

__device__ __forceinline__ void wave_add_u64(unsigned long long v, unsigned long long* c) {
  v = wave_scan(v);
  if ((threadIdx.x & 63u) == 63 && v) atomicAdd(c, v);
}

// Number of set bits of m below this lane.
__device__ __forceinline__ uint32_t lanes_before(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Slot tile i and cell tile i of the object, and the slot tiles of world w.  An
// object of one world computes them (one dependent load less in every launch).
__device__ __forceinline__ Tile slot_tile(const TileScratch& ts, uint32_t i) {
  if (ts.cap0) return Tile{0u, i * kSlotTile, min((uint32_t)kSlotTile, ts.cap0 - i * kSlotTile), 0u};
  return ts.slot_tiles[i];
}
__device__ __forceinline__ Tile cell_tile(const TileScratch& ts, uint32_t i) {
  if (ts.cap0) return Tile{0u, i * ts.cell_tile, min(ts.cell_tile, ts.cells0 - i * ts.cell_tile), 0u};
  return ts.cell_tiles[i];
}
// World w's slot and cell offsets (zero without a load where it is the only one).
__device__ __forceinline__ uint32_t slot_offset(const Dev& d, const TileScratch& ts, uint32_t w) {
  return ts.cap0 ? 0u : d.wp[w].slot_off;
}
__device__ __forceinline__ uint32_t first_slot_tile(const TileScratch& ts, uint32_t w) {
  return ts.cap0 ? 0u : ts.tile_rng[4 * w];
}
__device__ __forceinline__ uint32_t end_slot_tile(const TileScratch& ts, uint32_t w) {
  return ts.cap0 ? ts.n_slot_tiles : ts.tile_rng[4 * w + 1];
}

// ---------------------------------------------------------------------------
// Weight storage formats.
// A "unit" is 4 consecutive logical parameters = one 16-byte FP32 master block.
// ---------------------------------------------------------------------------
// Round-to-nearest-even FP32 -> BF16 of two finite values, a in the low half (one
// gfx950 instruction; equal to rounding the bit pattern for every FP32 but NaN).
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// FP32 -> OCP FP8 E4M3FN, round to nearest even, saturating at 448; values
// that round to zero give +0.  Works on the magnitude's bit pattern: the
// E4M3 exponent range is [-6, 8], subnormal step 2^-9.
__device__ __forceinline__ uint32_t fp8_rne_sat(float x) {
  const uint32_t sign = (__float_as_uint(x) >> 24) & 0x80u;
  const float a = fabsf(x);
  if (!(a < 448.0f)) return sign | 0x7Eu;
  uint32_t q;
  if (a < 0x1p-6f) {
    // subnormal range: q = RNE(a / 2^-9) in 0..8 (8 = smallest normal, code 0x08)
    const float t = a * 512.0f;        // exact (power-of-two scale)
    q = (uint32_t)__builtin_rintf(t);  // round half to even
  } else {
    const uint32_t u = __float_as_uint(a);
    const int e = (int)(u >> 23) - 127;               // -6 .. 8
    const uint32_t mant = u & 0x7FFFFFu;
    uint32_t m3 = mant >> 20;                         // top 3 mantissa bits
    const uint32_t rest = mant & 0xFFFFFu;            // 20 dropped bits
    const uint32_t half = 0x80000u;
    if (rest > half || (rest == half && (m3 & 1u))) ++m3;
    uint32_t ee = (uint32_t)(e + 7);
    if (m3 == 8) { m3 = 0; ++ee; }
    q = (ee << 3) | m3;
    if (q > 0x7Eu) q = 0x7Eu;
  }
  if (q == 0) return 0u;
  return sign | q;
}

// ---------------------------------------------------------------------------
// Step kernels
// ---------------------------------------------------------------------------
// Winners move, then EAT, step cost, death, age; per-tile counters.
// Three-resource ecology, one live agent after the moves (it touches only its own
// cell c, which no other agent touches in this launch): eat the chosen resource
// (up to the eat amount, the cell's content and the room under the stomach cap);
// pay energy (destroyed; rest costs least) and water (onto the cell); each
// resource that ran short, the agent's age and each of the `hits` strikes on its
// cell this step cost health; at zero health the agent dies and leaves water,
// energy and biomass on its cell (killed, when struck); otherwise energy heals
// it below full health and it ages.  Takes and returns its energy; alive says
// whether it survives.
__device__ __forceinline__ int ecology_agent(const Dev& d, const eco_ecology& e, const WorldParams& wp, uint32_t slot,
                                             uint32_t c, int a, uint32_t hits, int E, bool& alive, uint32_t* cnt) {
  int Wt = d.water[slot], B = d.biomass[slot], hp = d.hp[slot];
  int t = 0;
  if (a == EAT) {
    t = min(min(wp.e_eat, d.ce[c]), e.cap_energy - E);
    if (t > 0) { d.ce[c] -= t; E += t; }
  } else if (a == EAT_WATER) {
    t = min(min(e.eat_water, d.cw[c]), e.cap_water - Wt);
    if (t > 0) { d.cw[c] -= t; Wt += t; }
  } else if (a == EAT_BIOMASS) {
    t = min(min(e.eat_biomass, d.cb[c]), e.cap_biomass - B);
    if (t > 0) { d.cb[c] -= t; B += t; }
  }
  if (t > 0) count_lanes(&cnt[PC_EATEN]);
  int over = 0;
  E -= (a == REST) ? wp.e_cost : e.e_cost_move;
  if (E < 0) { E = 0; ++over; }
  const int spend = min(Wt, e.w_cost);
  Wt -= spend;
  d.cw[c] += spend;
  if (spend < e.w_cost) ++over;
  const long long damage =
      (long long)over * e.hp_overspend + (d.age[slot] >> e.age_shift) + (long long)hits * e.attack_damage;
  alive = (long long)hp - damage > 0;
  if (!alive) {
    d.cw[c] += Wt;
    d.ce[c] += E;
    d.cb[c] += B;
    E = Wt = B = hp = 0;
    d.flags[slot] = 0;
    d.occ[c] = -1;
    count_lanes(&cnt[PC_DEATHS]);
    if (hits) count_lanes(&cnt[PC_KILLED]);
  } else {
    hp -= (int)damage;
    if (hp < e.hp_max && E >= e.heal_energy) {
      hp = min(hp + e.hp_heal, e.hp_max);
      E -= e.heal_energy;
    }
    d.age[slot] += 1;
  }
  d.water[slot] = Wt;
  d.biomass[slot] = B;
  d.hp[slot] = hp;
  return E;
}

// One live agent's move (a FORWARD winner takes its claimed cell), then EAT, the
// step cost and death (Sec. 3.2), or with the ecology ecology_agent; counts into
// the LDS counters cnt.  a, cell, t, E: its action, position, target and energy;
// stamp: the attack stamp of this step (step + 1).
struct Moved {
  int cell, energy;
  bool alive;
};

__device__ __forceinline__ Moved move_agent(const Dev& d, const WorldParams& wp, uint32_t w, uint32_t slot,
                                            uint32_t local, uint32_t stamp, int a, int cell, int t, int E,
                                            uint32_t* cnt) {
  // the loads of the cells it stands on or claimed, issued before any store (no
  // other agent writes these cells in this pass: a claim targets a cell free at
  // step start)
  const uint32_t won = (a == FORWARD && t >= 0) ? d.claim[wp.cell_off + t] : ~0u;
  const uint8_t r0 = d.ep ? 0 : d.res[wp.cell_off + cell];
  const uint32_t m0 = (!d.ep && wp.attack) ? d.mark[wp.cell_off + cell] : 0u;
  const uint32_t m1 = (!d.ep && wp.attack && a == FORWARD && t >= 0) ? d.mark[wp.cell_off + t] : 0u;
  count_lanes_by<9>(&cnt[PC_HIST], a);
  bool moved = false, alive = true;
  if (a == FORWARD) {
    if (t >= 0 && won == slot) {
      d.claim[wp.cell_off + t] = 0xFFFFFFFFu;
      d.occ[wp.cell_off + cell] = -1;
      d.occ[wp.cell_off + t] = (int)local;
      cell = t;
      moved = true;
      d.pos[slot] = cell;
      count_lanes(&cnt[PC_MOVES_OK]);
    } else {
      count_lanes(&cnt[PC_MOVES_BLOCKED]);
    }
  }
  if (d.ep) {
    const uint32_t g = wp.cell_off + (uint32_t)cell;
    E = ecology_agent(d, d.ep[w], wp, slot, g, a, wp.attack ? d.mark[g] : 0u, E, alive, cnt);
  } else if (wp.attack && (moved ? m1 : m0) == stamp) {
    // struck after the moves: dies where it stands; its carried energy goes
    // back to the cell as one resource unit (cells hold 0 or 1 unit)
    d.flags[slot] = 0;
    d.occ[wp.cell_off + cell] = -1;
    d.res[wp.cell_off + cell] = 1;
    E = 0;
    alive = false;
    count_lanes(&cnt[PC_DEATHS]);
    count_lanes(&cnt[PC_KILLED]);
  } else {
    if (a == EAT && r0 > 0) {   // an eater did not move: cell is its own
      d.res[wp.cell_off + cell] = (uint8_t)(r0 - 1);
      E += wp.e_eat;
      count_lanes(&cnt[PC_EATEN]);
    }
    E -= wp.e_cost;
    if (E <= 0) {
      d.flags[slot] = 0;
      d.occ[wp.cell_off + cell] = -1;
      alive = false;
      count_lanes(&cnt[PC_DEATHS]);
    } else {
      d.age[slot] += 1;
    }
  }
  d.energy[slot] = E;
  return Moved{cell, E, alive};
}

// Blocks that share one child (a power of two, its logarithm): one where there are
// enough children to fill the chip, else up to eight, each with at least eight of the
// H rows of a hidden layer and one of the eight (sixteen) of the output layer.
__device__ __forceinline__ uint32_t child_split(const TileScratch& ts, uint32_t H, uint32_t births) {
  uint32_t lgp = 0;
  while (lgp < 3 && (16u << lgp) <= H && births << lgp < ts.split_below) ++lgp;
  return lgp;
}

// |theta|^2 of child j of the object's births (its slot global): from the blocks'
// shares where they shared the child or for the small-world kernel, else stored.
__device__ __forceinline__ double child_trait(const Dev& d, const TileScratch& ts, uint32_t lgp, bool shares, uint32_t j,
                                              uint32_t slot) {
  if (!shares) return d.trait[slot];
  double t = 0.0;
  for (uint32_t p = 0; p < 1u << lgp; ++p) t += ts.parts[(j << lgp) + p];
  return t;
}

// Completes the last step's record of world w with its children's traits: the
// population's moments are the survivors' and the children's combined about the
// common mean (NT threads).  Run by the launch after the births (the next step's
// first, or k_settle at the end of a call), since nothing in the births' own launch
// knows when all of them are done: a counter all blocks add to cost 40 us at 1,700
// blocks.  TRAITS: also store the traits of children that blocks shared.
template <int NT, bool TRAITS>
__device__ void settle_record(const Dev& d, const TileScratch& ts, uint32_t w, uint32_t H, bool small) {
  __shared__ double red[NT / 64];
  __shared__ uint32_t s_off[2][NT / 64];
  const WorldVar& v = d.wv[w];
  const uint32_t nb = v.n_births;
  if (nb == 0) return;
  // the object's births before this world's, and all of them
  uint32_t before = 0, total = 0;
  for (uint32_t i = threadIdx.x; i < d.n_worlds; i += NT) {
    const uint32_t b = d.wv[i].n_births;
    total += b;
    before += i < w ? b : 0u;
  }
  before = wave_scan(before);
  total = wave_scan(total);
  if ((threadIdx.x & 63u) == 63u) {
    s_off[0][threadIdx.x >> 6] = before;
    s_off[1][threadIdx.x >> 6] = total;
  }
  __syncthreads();
  before = total = 0;
  for (int i = 0; i < NT / 64; ++i) {
    before += s_off[0][i];
    total += s_off[1][i];
  }
  const uint32_t lgp = child_split(ts, H, total), slot_off = d.wp[w].slot_off, n = v.n0 + nb;
  const bool shares = small || lgp > 0;
  // In one pass, with deviations from the survivors' mean: with e = t - c, mean = c +
  // sum e / n, and the squared deviations about it are sum e^2 less n (mean - c)^2.  Every
  // child has a surviving parent of its own, so n0 >= nb, and that is (sum e)^2 / n <=
  // sum e^2 nb / n, at most half of what it is taken from.  Several
  // children a thread at once, the next ones' slots loaded with their traits, so that the
  // dependent loads overlap (a block for 6,600 children: two passes 17 us, now 13).
  constexpr int U = NT > 256 ? 2 : 8;
  const bool slots = TRAITS || !shares;
  auto load_slots = [&](uint32_t k0, uint32_t (&slot)[U]) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const uint32_t k = k0 + i * NT;
      slot[i] = (k < nb && slots) ? slot_off + (uint32_t)d.freel[slot_off + k] : 0u;
    }
  };
  const double c = v.mean;
  double s = 0.0, q = 0.0;
  uint32_t slot[U];
  load_slots(threadIdx.x, slot);
  for (uint32_t k = threadIdx.x; k < nb; k += U * NT) {
    double t[U];
    uint32_t next[U];
#pragma unroll
    for (int i = 0; i < U; ++i)
      t[i] = k + i * NT < nb ? child_trait(d, ts, lgp, shares, before + k + i * NT, slot[i]) : c;
    load_slots(k + U * NT, next);
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (TRAITS && shares && k + i * NT < nb) d.trait[slot[i]] = t[i];
      const double e = t[i] - c;
      s += e;
      q += e * e;
      slot[i] = next[i];
    }
  }
  s = block_sum_f64<NT>(s, red);
  q = block_sum_f64<NT>(q, red);
  if (threadIdx.x == 0) {
    const double shift = s / (double)n;   // mean - c; the survivors' deviations sum to zero about c
    eco_stats& st = d.ring[(uint64_t)w * kStatsRing + (v.step % kStatsRing)];
    st.trait_mean = c + shift;
    st.trait_var = (v.m2 + q - (double)n * shift * shift) / (double)n;
  }
}

// The end of a call: the last step's records and traits complete, no births pending
// (so that nothing of the step's scratch is read after the call).
__global__ __launch_bounds__(256) void k_settle(Dev d, TileScratch ts, uint32_t H, uint32_t small) {
  settle_record<256, true>(d, ts, blockIdx.x, H, small != 0);
  if (d.n_worlds > 1) return;   // (other worlds' blocks read this world's births: k_settled)
  __syncthreads();
  if (threadIdx.x == 0) d.wv[0].n_births = 0;
}
__global__ void k_settled(Dev d) {
  const uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w < d.n_worlds) d.wv[w].n_births = 0;
}

// Moves (slot tiles), the free slots of each tile, and the birth counter of each
// world cleared for the step; past the tiles, a block per world completes the last
// step's record.  Every field a slot's move can need first is loaded at
// once, live or not (a free slot's are not used).
__global__ __launch_bounds__(kSlotTile) void k_move(Dev d, TileScratch ts, uint32_t H) {
  __shared__ uint32_t cnt[kSlotPart];
  __shared__ uint32_t s_free[kSlotTile / 64];
  if (blockIdx.x >= ts.n_slot_tiles) {
    settle_record<kSlotTile, true>(d, ts, blockIdx.x - ts.n_slot_tiles, H, false);
    return;
  }
  if (threadIdx.x < kSlotPart) cnt[threadIdx.x] = 0;
  const Tile tl = slot_tile(ts, blockIdx.x);
  const WorldParams wp = d.wp[tl.world];
  const uint32_t stamp = (uint32_t)d.wv[tl.world].step + 1u;   // attack stamp of this step
  const bool in = threadIdx.x < tl.count;
  const uint32_t local = tl.start + threadIdx.x, slot = slot_offset(d, ts, tl.world) + local;
  uint8_t fl = 0;
  int a = 0, cell = 0, t = -1, E = 0;
  if (in) {
    fl = d.flags[slot];
    a = d.act[slot];
    cell = d.pos[slot];
    t = d.tgt[slot];
    E = d.energy[slot];
  }
  __syncthreads();
  bool alive = (fl & kAlive) != 0;
  if (alive) alive = move_agent(d, wp, tl.world, slot, local, stamp, a, cell, t, E, cnt).alive;
  const uint64_t fm = __ballot(in && !alive);
  if ((threadIdx.x & 63u) == 0) s_free[threadIdx.x >> 6] = (uint32_t)__builtin_popcountll(fm);
  __syncthreads();
  if (threadIdx.x < kSlotPart && threadIdx.x != PC_BB_CELL)   // that one: the birth claims
    ts.part_slot[blockIdx.x * kSlotPart + threadIdx.x] = cnt[threadIdx.x];
  if (threadIdx.x == 0) {
    uint32_t f = 0;
#pragma unroll
    for (int i = 0; i < kSlotTile / 64; ++i) f += s_free[i];
    ts.scan[blockIdx.x * 4 + 1] = f;
    if (tl.start == 0) d.wv[tl.world].n_win = 0;
  }
}

// Whether a live agent can be a parent this step (water, biomass: what it carries, in
// the ecology).
__device__ __forceinline__ bool may_bear(const Dev& d, const WorldParams& wp, uint32_t w, uint32_t n_actions, int act,
                                         int energy, int water, int biomass) {
  if (d.ep) {   // ecology: the eighth action, and spare biomass and water to give the child
    const eco_ecology& e = d.ep[w];
    return act == REPRODUCE_ECO && energy >= wp.e_repro && water >= e.w_child && biomass >= e.b_repro;
  }
  return energy >= wp.e_repro && (n_actions == 5 || act == REPRODUCE);
}

// One live agent's birth claim after the moves: a parent claims the cell directly
// behind it, which must be empty, and the lowest slot of its claimants wins.  The
// others can only be the agents on the cell's other three sides that face away from it,
// so each claimant looks at them itself: nothing in this pass changes what it reads.
// (An atomic minimum on a word per cell, read by the next launch, cost 2 - 3 us of this
// launch and that launch.)
enum ClaimResult { CLAIM_NONE, CLAIM_WON, CLAIM_BLOCKED };
__device__ __forceinline__ int birth_claim_agent(const Dev& d, const WorldParams& wp, uint32_t w, uint32_t slot,
                                                 uint32_t n_actions, int act, int pos, int facing, int energy,
                                                 int water, int biomass) {
  if (!may_bear(d, wp, w, n_actions, act, energy, water, biomass)) return CLAIM_NONE;
  const uint32_t t = neighbour(wp, (uint32_t)pos, facing, -1);
  const bool walled = wp.has_walls && d.wall[wp.cell_off + t];
  const int on = d.occ[wp.cell_off + t];
  int o[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) o[k] = d.occ[wp.cell_off + neighbour(wp, t, (facing + k + 1) & 3, +1)];
  if (on != -1 || walled) return CLAIM_BLOCKED;
  bool lost = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t other = wp.slot_off + (uint32_t)o[k];
    if (o[k] < 0 || other >= slot) continue;
    const int f = d.facing[other], a = d.act[other], e = d.energy[other];
    const int cw = d.ep ? d.water[other] : 0, cb = d.ep ? d.biomass[other] : 0;
    lost |= f == ((facing + k + 1) & 3) && may_bear(d, wp, w, n_actions, a, e, cw, cb);
  }
  if (lost) return CLAIM_BLOCKED;
  d.tgt[slot] = (int)t;
  return CLAIM_WON;
}

// Birth claims of one slot tile (its winners in slot order, as places in the tile, and
// their number to scan[0], with several worlds also to the world's n_win; one world's
// births are summed from scan[0], since the additions of some hundred tiles to one word
// cost 3 us), the free list of the tile (its free slots at
// their ranks among the world's, the earlier tiles' counts summed here) and the
// survivors' sums: count, energy, trait mean and squared deviations from it, and in
// the ecology what they carry (births move these from parent to child, so they
// are the totals after the births too).  One barrier: each wave reduces its 64
// slots, then every wave reads the four waves' results.
__device__ __forceinline__ void claim_tile(const Dev& d, const TileScratch& ts, uint32_t tile, uint32_t n_actions) {
  constexpr int NW = kSlotTile / 64;
  __shared__ uint32_t s_alive[NW], s_free[NW], s_before[NW], s_won[NW], s_blocked[NW];
  __shared__ unsigned long long s_e[NW], s_eco[3][NW];
  __shared__ double s_mean[NW], s_m2[NW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Tile tl = slot_tile(ts, tile);
  const uint32_t w = tl.world;
  const WorldParams wp = d.wp[w];
  const bool in = threadIdx.x < tl.count;
  const uint32_t slot_off = slot_offset(d, ts, w), local = tl.start + threadIdx.x, slot = slot_off + local;
  uint8_t fl = 0;
  int act = 0, pos = 0, facing = 0, energy = 0, water = 0, biomass = 0, hp = 0;
  double trait = 0.0;
  if (in) {
    fl = d.flags[slot];
    act = d.act[slot];
    pos = d.pos[slot];
    facing = d.facing[slot];
    energy = d.energy[slot];
    trait = d.trait[slot];
    if (d.ep) {
      water = d.water[slot];
      biomass = d.biomass[slot];
      hp = d.hp[slot];
    }
  }
  uint32_t before = 0;   // free slots of the world's earlier tiles
  for (uint32_t t = first_slot_tile(ts, w) + threadIdx.x; t < tile; t += kSlotTile) before += ts.scan[t * 4 + 1];
  const bool alive = (fl & kAlive) != 0;
  int claim = CLAIM_NONE;
  if (alive) claim = birth_claim_agent(d, wp, w, slot, n_actions, act, pos, facing, energy, water, biomass);
  const uint64_t am = __ballot(alive), fm = __ballot(in && !alive);
  const uint64_t wm = __ballot(claim == CLAIM_WON), bm = __ballot(claim == CLAIM_BLOCKED);
  const uint32_t n = (uint32_t)__builtin_popcountll(am);
  const unsigned long long es = wave_scan(alive ? (unsigned long long)(long long)energy : 0ull);
  const double mean = n ? lane_value(wave_scan(alive ? trait : 0.0), 63) / (double)n : 0.0;
  const double dv = alive ? trait - mean : 0.0, m2 = wave_scan(dv * dv);
  before = wave_scan(before);
  unsigned long long carried[3] = {0, 0, 0};
  if (d.ep) {
    carried[0] = wave_scan(alive ? (unsigned long long)water : 0ull);
    carried[1] = wave_scan(alive ? (unsigned long long)biomass : 0ull);
    carried[2] = wave_scan(alive ? (unsigned long long)hp : 0ull);
  }
  if (lane == 63) {
    s_alive[wave] = n;
    s_free[wave] = (uint32_t)__builtin_popcountll(fm);
    s_before[wave] = before;
    s_won[wave] = (uint32_t)__builtin_popcountll(wm);
    s_blocked[wave] = (uint32_t)__builtin_popcountll(bm);
    s_e[wave] = es;
    s_mean[wave] = mean;
    s_m2[wave] = m2;
#pragma unroll
    for (int k = 0; k < 3; ++k) s_eco[k][wave] = carried[k];
  }
  __syncthreads();
  uint32_t first = 0, tot_before = 0, won_before = 0;   // free rank of the wave's first free slot
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    tot_before += s_before[i];
    if (i < wave) {
      first += s_free[i];
      won_before += s_won[i];
    }
  }
  if (claim == CLAIM_WON) d.bparent[slot_off + tl.start + won_before + lanes_before(wm)] = (int)threadIdx.x;
  if (in && !alive) d.freel[slot_off + tot_before + first + lanes_before(fm)] = (int)local;
  if (threadIdx.x == 0) {
    uint32_t N = 0, F = 0, won = 0, B = 0;
    unsigned long long E = 0, cw = 0, cb = 0, ch = 0;
    double sum = 0.0, M2 = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      N += s_alive[i];
      F += s_free[i];
      won += s_won[i];
      B += s_blocked[i];
      E += s_e[i];
      cw += s_eco[0][i];
      cb += s_eco[1][i];
      ch += s_eco[2][i];
      sum += (double)s_alive[i] * s_mean[i];
    }
    const double mu = N ? sum / (double)N : 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) M2 += s_m2[i] + (double)s_alive[i] * (s_mean[i] - mu) * (s_mean[i] - mu);
    ts.part_slot[tile * kSlotPart + PC_BB_CELL] = B;
    ts.scan[tile * 4] = won;
    if (won && !ts.cap0) atomicAdd(&d.wv[w].n_win, won);
    ts.scan[tile * 4 + 2] = tot_before;
    ts.esum[tile] = (long long)E;
    ts.tmean[tile] = mu;
    ts.tm2[tile] = M2;
    if (d.ep) {
      ts.ecosum[3 * tile] = cw;
      ts.ecosum[3 * tile + 1] = cb;
      ts.ecosum[3 * tile + 2] = ch;
    }
    if (tile + 1 == end_slot_tile(ts, w)) {   // what the births need, beside the record that advances the clock
      d.wv[w].n_free = tot_before + F;
      d.draft[w].step = d.wv[w].step;
      d.draft[w].uid_next = d.wv[w].uid_next;
    }
  }
}

// floor(min(1, rate * b) * 2^32) in exact integer arithmetic, for a finite rate >= 0
// and b >= 1: rate = M 2^E with an integer M < 2^24, so rate * b * 2^32 is the
// integer M b (< 2^55) scaled by 2^(E + 32), floored.
__device__ __forceinline__ uint64_t photo_threshold(float rate, int b) {
  const uint32_t u = __float_as_uint(rate);
  const uint32_t ex = (u >> 23) & 0xFFu;
  const uint64_t M = ex ? ((u & 0x7FFFFFu) | 0x800000u) : (u & 0x7FFFFFu);
  const int k = (ex ? (int)ex - 150 : -149) + 32;   // rate = M 2^(k - 32)
  const uint64_t mb = M * (uint64_t)(uint32_t)b;
  constexpr uint64_t one = 1ull << 32;
  if (mb == 0) return 0;
  if (k >= 0) return (k >= 32 || mb >= (one >> k)) ? one : (mb << k);
  if (k <= -64) return 0;
  const uint64_t v = mb >> (-k);
  return v > one ? one : v;
}

// The regrowth (and photosynthesis) draws of local cells 4 q .. 4 q + 3 at `step`:
// one Philox block, output j for cell 4 q + j.
__device__ __forceinline__ uint4 regrow_draws(const WorldParams& wp, uint32_t q, uint32_t step) {
  return philox10(q, step, ST_REGROW, 0u, wp.key0, wp.key1);
}

__device__ __forceinline__ uint32_t word_of(const uint4& x, int j) {
  return j == 0 ? x.x : (j == 1 ? x.y : (j == 2 ? x.z : x.w));
}

// One regrowth pass over the resource bytes of local cells c0 .. c0 + n - 1 (n <= V,
// which divides 4, and c0 a multiple of V) held in the word v: each empty cell regrows one unit
// with probability p (its draw against floor(p 2^32)).  Returns the new word;
// adds the regrown cells and the resource total to grown and total.
template <int V>
__device__ __forceinline__ uint32_t regrow_word(const WorldParams& wp, uint32_t c0, uint32_t n, uint32_t v,
                                                uint32_t step, unsigned long long& grown, unsigned long long& total) {
  bool any = false;
#pragma unroll
  for (uint32_t j = 0; j < V; ++j) any |= j < n && ((v >> (8 * j)) & 0xFFu) == 0;
  uint32_t nv = v;
  if (any) {
    const uint4 x = regrow_draws(wp, c0 >> 2, step);
#pragma unroll
    for (uint32_t j = 0; j < V; ++j)
      if (j < n && ((v >> (8 * j)) & 0xFFu) == 0 && (uint64_t)word_of(x, V == 4 ? (int)j : (int)(c0 & 3u)) < wp.regrow_thr) {
        nv |= 1u << (8 * j);
        ++grown;
      }
  }
#pragma unroll
  for (uint32_t j = 0; j < V; ++j)
    if (j < n) total += (nv >> (8 * j)) & 0xFFu;
  return nv;
}

// V consecutive int32 cells from local cell c (four: c a multiple of 4; the cell
// allocation ends at a multiple of 64, so a ragged last group reads inside it), the
// first n of them stored, and V byte cells as the bytes of a word.
template <int V>
__device__ __forceinline__ void load_cells(const int32_t* p, int (&v)[V]) {
  if constexpr (V == 4) {
    const int4 x = *reinterpret_cast<const int4*>(p);
    v[0] = x.x;
    v[1] = x.y;
    v[2] = x.z;
    v[3] = x.w;
  } else {
    v[0] = p[0];
  }
}

template <int V>
__device__ __forceinline__ void store_cells(int32_t* p, uint32_t n, const int (&v)[V]) {
  if (V == 4 && n == 4) {
    if constexpr (V == 4) *reinterpret_cast<int4*>(p) = make_int4(v[0], v[1], v[2], v[3]);
  } else {
    for (uint32_t j = 0; j < n; ++j) p[j] = v[j];
  }
}

template <int V, typename T>
__device__ __forceinline__ uint32_t load_bytes(const T* p) {
  static_assert(sizeof(T) == 1, "byte cells");
  if constexpr (V == 4) return *reinterpret_cast<const uint32_t*>(p);
  else return (uint32_t)(uint8_t)p[0];
}

template <int V>
__device__ __forceinline__ void store_bytes(uint8_t* p, uint32_t n, uint32_t v) {
  if (V == 4 && n == 4) {
    *reinterpret_cast<uint32_t*>(p) = v;
  } else {
    for (uint32_t j = 0; j < n; ++j) p[j] = (uint8_t)(v >> (8 * j));
  }
}

__device__ __forceinline__ int byte_of(uint32_t v, int j) { return (int)(int8_t)(uint8_t)(v >> (8 * j)); }

// Terrain: the water on local cells c0 .. c0 + n - 1 after the flow (each cell's
// water moves one cell downhill, every cell at once): a cell keeps its own water if
// it has no way down, and takes that of each neighbour whose way down leads to it.
// own[] holds the cells' water before the flow, fd their direction bytes.  A group of
// one cell, or of four with W a multiple of 4, lies in one row, and the neighbours above
// and below are whole groups: flow_rows_load reads them (and the cells left and right
// of the group) so that the caller can issue these loads with its own, and returns
// false where the group takes the per-cell path instead.
template <int V>
struct FlowRows {
  int wu[V], wd[V];   // water of the cells above and below
  uint32_t fu, fdn;   // their direction bytes
  int wl, wr, fl, fr;   // water and direction of the cells left and right of the group
};

template <int V>
__device__ __forceinline__ bool flow_rows_load(const Dev& d, const WorldParams& wp, uint32_t c0, uint32_t n,
                                               FlowRows<V>& r) {
  if (V > 1 && ((wp.W & 3u) != 0 || n != V)) return false;
  const uint32_t off = wp.cell_off, W = wp.W, y0 = c0 / W, x0 = c0 - y0 * W, row = y0 * W;
  const uint32_t up = (y0 == 0 ? wp.H - 1 : y0 - 1) * W + x0, dn = (y0 + 1 == wp.H ? 0u : y0 + 1) * W + x0;
  const uint32_t lf = row + (x0 == 0 ? W - 1 : x0 - 1), rt = row + (x0 + V == W ? 0u : x0 + V);
  load_cells(d.cw + off + up, r.wu);
  load_cells(d.cw + off + dn, r.wd);
  r.fu = load_bytes<V>(d.flowdir + off + up);
  r.fdn = load_bytes<V>(d.flowdir + off + dn);
  r.wl = d.cw[off + lf];
  r.wr = d.cw[off + rt];
  r.fl = d.flowdir[off + lf];
  r.fr = d.flowdir[off + rt];
  return true;
}

template <int V>
__device__ __forceinline__ void flow_gather(const Dev& d, const WorldParams& wp, uint32_t c0, uint32_t n,
                                            const int (&own)[V], uint32_t fd, bool rows, const FlowRows<V>& r,
                                            int (&out)[V]) {
#pragma unroll
  for (int j = 0; j < V; ++j) out[j] = byte_of(fd, j) < 0 ? own[j] : 0;
  if (V == 1 || rows) {
#pragma unroll
    for (int j = 0; j < V; ++j) {
      // the neighbour above (facing 0) leads here if it flows down (2), the one to
      // the right (1) if it flows left (3), below (2) if up (0), left (3) if right (1)
      if (byte_of(r.fu, j) == 2) out[j] += r.wu[j];
      if ((j < V - 1 ? byte_of(fd, j + 1) : r.fr) == 3) out[j] += j < V - 1 ? own[j + 1 < V ? j + 1 : j] : r.wr;
      if (byte_of(r.fdn, j) == 0) out[j] += r.wd[j];
      if ((j > 0 ? byte_of(fd, j - 1) : r.fl) == 1) out[j] += j > 0 ? own[j > 0 ? j - 1 : 0] : r.wl;
    }
  } else {
    for (uint32_t j = 0; j < n; ++j) {
#pragma unroll
      for (int dd = 0; dd < 4; ++dd) {
        const uint32_t nb = wp.cell_off + neighbour(wp, c0 + j, dd, +1);
        if (d.flowdir[nb] == ((dd + 2) & 3)) out[j] += d.cw[nb];
      }
    }
  }
}

// Window channels of a cell at the start of a step (Sec. 3.2 sensors, App. F
// layout), one byte per cell: bit 0 agent present, bit 1 resource present, bit 2
// wall (worlds with walls only), bits 3..5 the occupant's energy bin
// min(floor(8 E / e_repro), 7).  Built by the cell pass of the step before (and by
// init and state writes), so that the policy kernel's window gather reads one byte
// per cell instead of the occupancy, resource and wall arrays plus a dependent read
// of each occupant's energy.
// The cell's resource and wall bits of its sense byte.
__device__ __forceinline__ uint32_t cell_sense(const WorldParams& wp, uint32_t r, uint32_t wl) {
  return (r != 0 ? 2u : 0u) | (wp.has_walls && wl != 0 ? 4u : 0u);
}

// An occupant's bits of the sense byte: the agent bit and its energy bin
// (the number of b in 1..7 with 8 E >= b e_repro).
__device__ __forceinline__ uint32_t agent_sense(const WorldParams& wp, int energy) {
  const long long e8 = (long long)energy * 8;
  uint32_t eb = 0;
#pragma unroll
  for (int b = 1; b < 8; ++b) eb += (e8 >= (long long)b * wp.e_repro) ? 1u : 0u;
  return 1u | (eb << 3);
}

// Colour vision: the cell as others see it (occupant's colour, else a resource
// unit in green, else a wall in grey, else black; 8 bits per channel), with the
// cell's agent / resource / wall bits in the top byte for the move claim.
// round(clamp(c, 0, 1) * 255) with ties up, in exact integer arithmetic: a c in
// (0, 1) is M 2^-s with an integer M < 2^24 and s >= 24, so the result is
// floor((255 M + 2^(s-1)) / 2^s).
__device__ __forceinline__ uint32_t colour_byte(float c) {
  if (!(c > 0.0f)) return 0u;   // also NaN
  if (c >= 1.0f) return 255u;
  const uint32_t u = __float_as_uint(c);
  const uint32_t ex = u >> 23;   // c > 0: sign bit clear
  const uint64_t M = ex ? ((u & 0x7FFFFFu) | 0x800000u) : (u & 0x7FFFFFu);
  const int s = ex ? 150 - (int)ex : 149;   // c = M 2^-s, s >= 24
  if (s >= 64) return 0u;
  return (uint32_t)((255ull * M + (1ull << (s - 1))) >> s);
}

__device__ __forceinline__ uint32_t colour_word(const float4 c) {
  return colour_byte(c.x) | (colour_byte(c.y) << 8) | (colour_byte(c.z) << 16);
}

__device__ __forceinline__ uint32_t sat255(int v) { return (uint32_t)min(max(v, 0), 255); }

// The cells of tile tl of a single-resource world, V consecutive cells per
// thread and pass (tiles start at multiples of 4 cells).
// GROW (a step): each empty cell regrows one unit with probability p, and the
// regrown cells and the resource total go to cnt[0], cnt[1] (LDS).  Then the
// cell's window channels, from the resources just grown and the occupants after the
// moves (a birth adds its own, place_child), so the grid is read once a step.  agent,
// col: the occupants' sense bits by cell and colour words by slot, where the caller
// has them in LDS; else they are read through the occupancy.
template <bool GROW, int V>
__device__ __forceinline__ void plain_cells(const Dev& d, const WorldParams& wp, uint32_t cell_off, const Tile tl, uint32_t step,
                                            unsigned long long* cnt, const uint8_t* agent, const uint32_t* col) {
  unsigned long long grown = 0, total = 0;
#pragma unroll 1
  for (uint32_t i = V * threadIdx.x; i < tl.count; i += V * blockDim.x) {
    const uint32_t c0 = tl.start + i, n = min((uint32_t)V, tl.count - i), g = cell_off + c0;
    const uint32_t v = load_bytes<V>(d.res + g);
    const uint32_t wl = wp.has_walls ? load_bytes<V>(d.wall + g) : 0u;
    int o[V], q[V];   // the occupants, their sense bits or colour words
#pragma unroll
    for (int j = 0; j < V; ++j) {
      o[j] = -1;
      q[j] = 0;
    }
    if (d.rgb || !agent) {
      load_cells(d.occ + g, o);
#pragma unroll
      for (uint32_t j = 0; j < V; ++j) {
        if (j >= n) o[j] = -1;   // past a ragged tail: no occupant read
        if (o[j] < 0) continue;
        const uint32_t slot = wp.slot_off + (uint32_t)o[j];
        if (d.rgb) q[j] = (int)(col ? col[o[j]] : colour_word(d.colour[slot]));
        else q[j] = (int)agent_sense(wp, d.energy[slot]);
      }
    } else {
      const uint32_t ag = load_bytes<V>(agent + c0);
#pragma unroll
      for (int j = 0; j < V; ++j) q[j] = (int)((ag >> (8 * j)) & 0xFFu);
    }
    uint32_t nv = v;
    if constexpr (GROW) {
      nv = regrow_word<V>(wp, c0, n, v, step, grown, total);
      if (nv != v) store_bytes<V>(d.res + g, n, nv);
    }
    if (d.rgb) {
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const uint32_t bits = cell_sense(wp, (nv >> (8 * j)) & 0xFFu, (wl >> (8 * j)) & 0xFFu);
        if (o[j] < 0) q[j] = (bits & 2u) ? 255 << 8 : ((bits & 4u) ? 0x808080 : 0);
        q[j] |= (int)(((o[j] >= 0 ? 1u : 0u) | bits) << 24);
      }
      store_cells(reinterpret_cast<int32_t*>(d.rgb + g), n, q);
    } else {
      uint32_t sv = 0;
#pragma unroll
      for (int j = 0; j < V; ++j)
        sv |= ((uint32_t)q[j] | cell_sense(wp, (nv >> (8 * j)) & 0xFFu, (wl >> (8 * j)) & 0xFFu)) << (8 * j);
      store_bytes<V>(d.sense + g, n, sv);
    }
  }
  if constexpr (GROW) {
    wave_add_u64(grown, &cnt[0]);
    wave_add_u64(total, &cnt[1]);
  }
}

// The cells of tile tl of an ecology, V consecutive cells per thread and pass.
// STEP: photosynthesis, one energy unit with probability min(1, rate * biomass) on
// cells holding biomass below the energy ceiling (the threshold in exact integers;
// the draws of four cells are the four outputs of one Philox block); the strikes of
// this step cleared (they have been counted); with terrain, the water's flow
// gathered into cw_next (copied back by the next pass, once every cell has read the
// old layer); the photosynthesised units and the grid totals of energy, water and
// biomass to cnt[0..3] (LDS).  Then the window word of each cell: its water (after
// the flow), energy and biomass levels (capped at 255), or with colour vision the
// cell as others see it (occupant's colour, wall grey, else energy / biomass / water
// as red / green / blue); the agent / wall bits and the rock height in the top byte.
// col: the live agents' colour words by slot, where the caller has them in LDS.
template <bool STEP, int V>
__device__ __forceinline__ void ecology_cells(const Dev& d, const WorldParams& wp, const eco_ecology& e,
                                              uint32_t cell_off, const Tile tl, uint32_t step, unsigned long long* cnt, const uint32_t* col) {
  unsigned long long grown = 0, total = 0, wsum = 0, bsum = 0;
#pragma unroll 1
  for (uint32_t i = V * threadIdx.x; i < tl.count; i += V * blockDim.x) {
    const uint32_t c0 = tl.start + i, n = min((uint32_t)V, tl.count - i), g = cell_off + c0;
    int b[V], en[V], wv[V], o[V], rk[V] = {}, q[V] = {};
    load_cells(d.occ + g, o);
    load_cells(d.cb + g, b);
    load_cells(d.ce + g, en);
    load_cells(d.cw + g, wv);
    if (d.rock) load_cells(d.rock + g, rk);
    const uint32_t wl4 = wp.has_walls ? load_bytes<V>(d.wall + g) : 0u;
    const uint32_t fd = (STEP && d.rock) ? load_bytes<V>(d.flowdir + g) : 0u;
    FlowRows<V> fr{};   // the flow's neighbour rows, loaded with the cells' own values
    const bool rows = STEP && d.rock && flow_rows_load(d, wp, c0, n, fr);
#pragma unroll
    for (uint32_t j = 0; j < V; ++j)
      if (j >= n) o[j] = -1;   // past a ragged tail: no occupant read
    if (d.colour) {
#pragma unroll
      for (int j = 0; j < V; ++j)
        if (o[j] >= 0) q[j] = (int)(col ? col[o[j]] : colour_word(d.colour[wp.slot_off + (uint32_t)o[j]]));
    }
    if constexpr (STEP) {
      bool any = false;
#pragma unroll
      for (uint32_t j = 0; j < V; ++j) any |= j < n && b[j] > 0 && en[j] < e.cell_energy_max;
      if (any) {
        const uint4 x = regrow_draws(wp, c0 >> 2, step);
        bool grew = false;
#pragma unroll
        for (uint32_t j = 0; j < V; ++j)
          if (j < n && b[j] > 0 && en[j] < e.cell_energy_max &&
              (uint64_t)word_of(x, V == 4 ? (int)j : (int)(c0 & 3u)) < photo_threshold(e.photo_rate, b[j])) {
            ++en[j];
            ++grown;
            grew = true;
          }
        if (grew) store_cells(d.ce + g, n, en);
      }
#pragma unroll
      for (uint32_t j = 0; j < V; ++j)
        if (j < n) {
          total += (unsigned long long)(uint32_t)en[j];
          wsum += (unsigned long long)(uint32_t)wv[j];
          bsum += (unsigned long long)(uint32_t)b[j];
        }
      if (wp.attack) {
        const int none[V] = {};
        store_cells(reinterpret_cast<int32_t*>(d.mark + g), n, none);
      }
      if (d.rock) {
        int nw[V];
        flow_gather(d, wp, c0, n, wv, fd, rows, fr, nw);
        store_cells(d.cw_next + g, n, nw);
#pragma unroll
        for (int j = 0; j < V; ++j) wv[j] = nw[j];
      }
    }
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const bool wl = ((wl4 >> (8 * j)) & 0xFFu) != 0;
      if (!d.colour) {
        q[j] = (int)(sat255(wv[j]) | (sat255(en[j]) << 8) | (sat255(b[j]) << 16));
      } else if (o[j] < 0) {
        q[j] = (int)(wl ? 0x808080u
                        : (sat255(16 * min(en[j], 1 << 20)) | (sat255(64 * min(b[j], 1 << 20)) << 8) |
                           (sat255(16 * min(wv[j], 1 << 20)) << 16)));
      }
      q[j] |= (int)(((o[j] >= 0 ? 1u : 0u) | (wl ? 4u : 0u) | ((uint32_t)rk[j] << 3)) << 24);
    }
    store_cells(reinterpret_cast<int32_t*>(d.rgb + g), n, q);
  }
  if constexpr (STEP) {
    wave_add_u64(grown, &cnt[0]);
    wave_add_u64(total, &cnt[1]);
    wave_add_u64(wsum, &cnt[2]);
    wave_add_u64(bsum, &cnt[3]);
  }
}

// Window channels of the cells of tile tl as they stand (init, state, colour and
// terrain writes).
__device__ __forceinline__ void window_cells(const Dev& d, const Tile tl) {
  const WorldParams wp = d.wp[tl.world];
  if (d.ep) ecology_cells<false, 4>(d, wp, d.ep[tl.world], wp.cell_off, tl, 0u, nullptr, nullptr);
  else plain_cells<false, 4>(d, wp, wp.cell_off, tl, 0u, nullptr, nullptr, nullptr);
}

// With terrain: the water after the flow becomes the water of the cells of tile tl
// (every cell has read the old layer).
__device__ __forceinline__ void settle_water(const Dev& d, const WorldParams& wp, const Tile tl) {
  for (uint32_t i = 4 * threadIdx.x; i < tl.count; i += 4 * blockDim.x) {
    const uint32_t n = min(4u, tl.count - i), g = wp.cell_off + tl.start + i;
    int wv[4];
    load_cells(d.cw_next + g, wv);
    store_cells(d.cw + g, n, wv);
  }
}

// Birth claims, free lists and the survivors' sums (slot tiles), and in the same
// launch the cell pass (cell tiles): independent work, since a claim changes neither
// the occupancy nor the resources.  V: consecutive cells per thread.
template <int V>
__global__ __launch_bounds__(256) void k_claim_cells(Dev d, TileScratch ts, uint32_t n_actions) {
  __shared__ unsigned long long cnt[kCellPart];
  if (blockIdx.x < ts.n_slot_tiles) {
    claim_tile(d, ts, blockIdx.x, n_actions);
    return;
  }
  const uint32_t tile = blockIdx.x - ts.n_slot_tiles;
  if (threadIdx.x < kCellPart) cnt[threadIdx.x] = 0;
  __syncthreads();
  const Tile tl = cell_tile(ts, tile);
  const uint32_t cell_off = ts.cap0 ? 0u : d.wp[tl.world].cell_off;   // (the only world's cells: no load to wait for)
  const WorldParams wp = d.wp[tl.world];
  const uint32_t step = (uint32_t)d.wv[tl.world].step;
  if (d.ep) ecology_cells<true, V>(d, wp, d.ep[tl.world], cell_off, tl, step, cnt, nullptr);
  else plain_cells<true, V>(d, wp, cell_off, tl, step, cnt, nullptr, nullptr);
  __syncthreads();
  if (threadIdx.x < kCellPart) ts.part_cell[tile * kCellPart + threadIdx.x] = cnt[threadIdx.x];
}

// The sums of world w's tiles for its statistics record (one block of NT threads,
// once the moves, the claims and the cell pass are done): the counters, the grid
// totals plus, in the ecology, what the survivors carry, and the survivors' trait
// moments combined from the tiles' (mean = sum n_i mean_i / N, then the squared
// deviations about it: M2 = sum (M2_i + n_i (mean_i - mean)^2); the slot tiles of a
// world hold 256 slots each but the last).
template <int NT>
__device__ __forceinline__ void world_draft(const Dev& d, const TileScratch& ts, uint32_t w, StepDraft* dr,
                                            uint32_t* winners) {
  constexpr int NW = NT / 64;
  __shared__ uint32_t s_cnt[kSlotPart + 2][NW];
  __shared__ unsigned long long s_sum[kCellPart + 4][NW];
  __shared__ double s_f[NW], s_m2[NW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t cap = ts.cap0 ? ts.cap0 : d.wp[w].cap;
  const uint32_t t0 = first_slot_tile(ts, w), t1 = end_slot_tile(ts, w);
  const uint32_t c0 = ts.cap0 ? 0u : ts.tile_rng[4 * w + 2], c1 = ts.cap0 ? ts.n_cell_tiles : ts.tile_rng[4 * w + 3];
  uint32_t c[kSlotPart + 2];   // the counters, survivors, claim winners
  unsigned long long u[kCellPart + 4];
#pragma unroll
  for (int k = 0; k < kSlotPart + 2; ++k) c[k] = 0;
#pragma unroll
  for (int k = 0; k < kCellPart + 4; ++k) u[k] = 0;
  double sum = 0.0;
  for (uint32_t t = t0 + threadIdx.x; t < t1; t += NT) {
    const uint4* pr = reinterpret_cast<const uint4*>(ts.part_slot + t * kSlotPart);
    const uint2 sc = *reinterpret_cast<const uint2*>(ts.scan + t * 4);   // winners, free slots
    const uint32_t n = min((uint32_t)kSlotTile, cap - (t - t0) * kSlotTile) - sc.y;
    c[kSlotPart + 1] += sc.x;
#pragma unroll
    for (int k = 0; k < kSlotPart / 4; ++k) {
      const uint4 v = pr[k];
      c[4 * k] += v.x;
      c[4 * k + 1] += v.y;
      c[4 * k + 2] += v.z;
      c[4 * k + 3] += v.w;
    }
    c[kSlotPart] += n;
    u[kCellPart] += (unsigned long long)ts.esum[t];
    sum += (double)n * ts.tmean[t];
    if (d.ep) {
#pragma unroll
      for (int k = 0; k < 3; ++k) u[kCellPart + 1 + k] += ts.ecosum[3 * t + k];
    }
  }
  for (uint32_t t = c0 + threadIdx.x; t < c1; t += NT) {
    const ulonglong2* pc = reinterpret_cast<const ulonglong2*>(ts.part_cell + t * kCellPart);
    const ulonglong2 a = pc[0], b = pc[1];
    u[0] += a.x;
    u[1] += a.y;
    u[2] += b.x;
    u[3] += b.y;
  }
  sum = wave_scan(sum);
  if (lane == 63) s_f[wave] = sum;
#pragma unroll
  for (int k = 0; k < kSlotPart + 2; ++k) {
    const uint32_t v = wave_scan(c[k]);
    if (lane == 63) s_cnt[k][wave] = v;
  }
#pragma unroll
  for (int k = 0; k < kCellPart + 4; ++k) {
    if (k >= kCellPart + 1 && !d.ep) break;
    const unsigned long long v = wave_scan(u[k]);
    if (lane == 63) s_sum[k][wave] = v;
  }
  __syncthreads();
  uint32_t N = 0;
  double S = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    N += s_cnt[kSlotPart][i];
    S += s_f[i];
  }
  const double mean = N ? S / (double)N : 0.0;
  double m2 = 0.0;
  for (uint32_t t = t0 + threadIdx.x; t < t1; t += NT) {
    const uint32_t n = min((uint32_t)kSlotTile, cap - (t - t0) * kSlotTile) - ts.scan[t * 4 + 1];
    const double dv = ts.tmean[t] - mean;
    m2 += ts.tm2[t] + (double)n * dv * dv;
  }
  m2 = wave_scan(m2);
  if (lane == 63) s_m2[wave] = m2;
  __syncthreads();
  if (threadIdx.x < kSlotPart) {
    uint32_t v = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) v += s_cnt[threadIdx.x][i];
    dr->count[threadIdx.x] = v;
  } else if (threadIdx.x == 32) {
    uint32_t v = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) v += s_cnt[kSlotPart + 1][i];
    *winners = v;
  } else if (threadIdx.x == 64) {
    unsigned long long v[kCellPart + 4];
#pragma unroll
    for (int k = 0; k < kCellPart + 4; ++k) {
      v[k] = 0;
      if (k >= kCellPart + 1 && !d.ep) continue;
#pragma unroll
      for (int i = 0; i < NW; ++i) v[k] += s_sum[k][i];
    }
    double M2 = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) M2 += s_m2[i];
    dr->regrown = v[0];
    dr->resource_total = v[1];
    dr->water = d.ep ? v[2] + v[kCellPart + 1] : 0ull;
    dr->biomass = d.ep ? v[3] + v[kCellPart + 2] : 0ull;
    dr->hp = d.ep ? v[kCellPart + 3] : 0ull;
    dr->energy = (long long)v[kCellPart];
    dr->mean = mean;
    dr->m2 = M2;
    dr->n0 = N;
    dr->step = d.wv[w].step;
    dr->uid_next = d.wv[w].uid_next;
  }
  __syncthreads();
}

// Births of a world this step: its winners, as far as free slots go (an object of
// several worlds, or winners ranked by the small-world kernel).
__device__ __forceinline__ uint32_t births_of(const WorldVar& v) { return min(v.n_win, v.n_free); }

// Prefixes of the per-world birth and winner counts in LDS (same scheme as the live offsets).
__device__ __forceinline__ void birth_offsets(const WorldVar* __restrict__ wv, uint32_t n, uint32_t* off,
                                              uint32_t* off_win) {
  const int tid = threadIdx.x;
  if (tid < 64) {
    const uint32_t per = (n + 63) / 64;
    const uint32_t lo = min(tid * per, n), hi = min(lo + per, n);
    uint32_t s = 0, sw = 0;
    for (uint32_t i = lo; i < hi; ++i) {
      s += births_of(wv[i]);
      sw += wv[i].n_win;
    }
    const uint32_t inc = wave_scan(s), incw = wave_scan(sw);
    uint32_t run = inc - s, runw = incw - sw;
    for (uint32_t i = lo; i < hi; ++i) {
      off[i] = run;
      off_win[i] = runw;
      run += births_of(wv[i]);
      runw += wv[i].n_win;
    }
    if (tid == 63) {
      off[n] = inc;
      off_win[n] = incw;
    }
  }
  __syncthreads();
}

constexpr int kMaxWorlds = ECO_MAX_WORLDS;

// Unit u of an agent's master (16 bytes, four consecutive logical parameters):
// its Philox block (= first logical parameter / 4), layer (0..2 weights, 3..5
// biases), output row (first row for biases), k-block (the column quad in layer
// 2) and the number of its parameters that exist.  H = H1 = H2 is a power of
// two, so every index is a shift or a mask.
struct UnitPos {
  uint32_t blk, row, kb, nvalid;
  int layer;
};

template <int H>
__device__ __forceinline__ UnitPos unit_pos(const Layout& L, uint32_t u) {
  constexpr uint32_t LG = H == 32 ? 5 : (H == 64 ? 6 : 7);
  UnitPos r;
  r.nvalid = 4;
  r.kb = 0;
  if (u < L.u_b1) {                   // W1 [kb][row]: first parameter row D + 4 kb
    r.layer = 0; r.row = u & (H - 1); r.kb = u >> LG; r.blk = r.row * L.KB1 + r.kb;
  } else if (u < L.u_w2) {            // b1
    const uint32_t e = u - L.u_b1;
    r.layer = 3; r.row = 4 * e; r.blk = (L.p_b1 >> 2) + e;
  } else if (u < L.u_b2) {            // W2 [kb][row]: p_w2 + row H + 4 kb
    const uint32_t e = u - L.u_w2;
    r.layer = 1; r.row = e & (H - 1); r.kb = e >> LG; r.blk = (L.p_w2 >> 2) + r.row * (H / 4) + r.kb;
  } else if (u < L.u_w3) {            // b2
    const uint32_t e = u - L.u_b2;
    r.layer = 4; r.row = 4 * e; r.blk = (L.p_b2 >> 2) + e;
  } else if (u < L.u_b3) {            // W3 [row][H]: p_w3 + row H + 4 kb (rows >= A are padding)
    const uint32_t e = u - L.u_w3;
    r.layer = 2; r.row = e >> (LG - 2); r.kb = e & (H / 4 - 1); r.blk = (L.p_w3 >> 2) + e;
    r.nvalid = r.row < L.A ? 4u : 0u;
  } else {                            // b3, then the log temperature in slot A when it evolves
    const uint32_t e = u - L.u_b3, n3 = L.A + L.temp;
    r.layer = 5; r.row = 4 * e; r.blk = (L.p_b3 >> 2) + e;
    r.nvalid = r.row < n3 ? min(4u, n3 - r.row) : 0u;
  }
  return r;
}

// Streaming accesses of the weight blocks a birth reads once and writes once
// (non-temporal: no cache line is kept for them).
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 stream_load4(const float4* p) {
  const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
// The child's FP32 master; cached when it is read back for FP8 row scales (WDT 2).
template <int WDT>
__device__ __forceinline__ void stream_store4(float4* p, float a, float b, float c, float d) {
  if (WDT == 2) *p = make_float4(a, b, c, d);
  else __builtin_nontemporal_store(f32x4{a, b, c, d}, reinterpret_cast<f32x4*>(p));
}

// Storage copy of one unit's four master values (BF16 round-to-nearest-even;
// FP8: biases as FP32 here, weights after the row scales are known).
template <int WDT, int H>
__device__ __forceinline__ void store_unit(const Layout& L, uint8_t* sc, int layer, uint32_t row, uint32_t kb,
                                           const float (&v)[4], uint32_t* s_amax) {
  if (WDT == 1) {
    const uint32_t lo = bf16_pair(v[0], v[1]);
    const uint32_t hi = bf16_pair(v[2], v[3]);
    uint64_t off;
    if (layer == 0) off = L.s_w1 + ((uint64_t)(kb >> 1) * H + row) * 16 + (kb & 1) * 8;
    else if (layer == 1) off = L.s_w2 + ((uint64_t)(kb >> 1) * H + row) * 16 + (kb & 1) * 8;
    else if (layer == 2) off = L.s_w3 + ((uint64_t)row * H + 4 * kb) * 2;
    else off = L.s_b1 + (layer >= 4 ? L.s_b2 - L.s_b1 : 0u) + (layer >= 5 ? L.s_b3 - L.s_b2 : 0u) + (uint64_t)row * 2;
    *reinterpret_cast<uint2*>(sc + off) = make_uint2(lo, hi);   // half of a 16-byte block: cached
  } else if (WDT == 2) {
    if (layer < 3) {
      const uint32_t r = layer == 0 ? row : (layer == 1 ? H + row : 2 * H + row);
      const float mx = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
      atomicMax(&s_amax[r], __float_as_uint(mx));
    } else {
      const uint32_t base = L.s_b1 + (layer >= 4 ? L.s_b2 - L.s_b1 : 0u) + (layer >= 5 ? L.s_b3 - L.s_b2 : 0u);
      *reinterpret_cast<float4*>(sc + base + (uint64_t)row * 4) = make_float4(v[0], v[1], v[2], v[3]);
    }
  }
}

// One part of an agent's units, for 2^lgp blocks working on one agent: rows
// [part H / parts, ...) of W1, W2 and the biases, R3 / parts rows of the output
// layer, its biases with part 0.  Rows, not columns, so that an FP8 row's scale is
// one block's; at least eight rows, so that a k-block of a part is a whole 128-byte
// line.
template <int H>
struct PartRows {
  uint32_t lgr;     // log2 of the rows of a part
  uint32_t row0;    // its first row
  uint32_t part, lgp;
};
template <int H>
__device__ __forceinline__ PartRows<H> part_rows(uint32_t part, uint32_t lgp) {
  constexpr uint32_t LG = H == 32 ? 5 : (H == 64 ? 6 : 7);
  return PartRows<H>{LG - lgp, part << (LG - lgp), part, lgp};
}
// Unit of W2 number q of the part, and the others: b1, b2 and W3 in turn, then b3.
template <int H>
__device__ __forceinline__ uint32_t part_w2_unit(const Layout& L, const PartRows<H>& pr, uint32_t q) {
  return L.u_w2 + (q >> pr.lgr) * H + pr.row0 + (q & ((1u << pr.lgr) - 1u));
}
template <int H>
__device__ __forceinline__ uint32_t part_rest_count(const Layout& L, const PartRows<H>& pr) {
  return ((2u * (H / 4) + L.R3 * (H / 4)) >> pr.lgp) + (pr.part == 0 ? L.R3 / 4 : 0u);
}
template <int H>
__device__ __forceinline__ uint32_t part_rest_unit(const Layout& L, const PartRows<H>& pr, uint32_t q) {
  const uint32_t nb = (H / 4) >> pr.lgp, n3 = (L.R3 * (H / 4)) >> pr.lgp;
  if (q < nb) return L.u_b1 + pr.part * nb + q;
  q -= nb;
  if (q < nb) return L.u_b2 + pr.part * nb + q;
  q -= nb;
  return q < n3 ? L.u_w3 + pr.part * n3 + q : L.u_b3 + (q - n3);
}

// Four weights divided by their row's scale and rounded to FP8 (fp8_rne_sat, the last one
// lowest).  inv: 1 / scale.  The division is the product with inv corrected twice by its
// residual, exact (and its second correction then rounds correctly, Markstein 1990)
// for scales away from the ends of the range; the rounding is the conversion
// instruction, which agrees with fp8_rne_sat on every float but for values that round
// to -0 (made +0 here) and NaN.  Other scales, and NaN, take the division and
// fp8_rne_sat themselves.  (These were some 120 of a unit's 310 instructions: the birth
// launch of a 61,003-agent world 36.0 -> 31.3 us, the step of a 65,536-agent world with
// 8,110 births 1,313 -> 1,244, a reset of 61,003 agents 6.15 -> 4.95 ms.)
__device__ __forceinline__ uint32_t fp8_quantise4(const float4 m, float scale, float inv) {
  const float any = m.x + m.y + m.z + m.w;   // NaN if one of them is
  if (!(scale >= 0x1p-60f && scale <= 0x1p100f && any == any))
    return fp8_rne_sat(m.x / scale) | (fp8_rne_sat(m.y / scale) << 8) | (fp8_rne_sat(m.z / scale) << 16) |
           (fp8_rne_sat(m.w / scale) << 24);
  auto quotient = [&](float a) {
    float q = a * inv;
    q = __builtin_fmaf(__builtin_fmaf(-q, scale, a), inv, q);
    q = __builtin_fmaf(__builtin_fmaf(-q, scale, a), inv, q);
    return __builtin_amdgcn_fmed3f(q, -448.0f, 448.0f);
  };
  int r = __builtin_amdgcn_cvt_pk_fp8_f32(quotient(m.x), quotient(m.y), 0, false);
  r = __builtin_amdgcn_cvt_pk_fp8_f32(quotient(m.z), quotient(m.w), r, true);
  const uint32_t q = (uint32_t)r;
  return q & ((((q & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) & 0x80808080u) | 0x7F7F7F7Fu);   // no sign without a magnitude
}

// FP8 storage, after store_unit has gathered each row's amax in s_amax: the row
// scales of the part (left in s_amax), then its weights quantised with them (each
// thread re-reads master units its block wrote).
template <int H, int NT>
__device__ __forceinline__ void fp8_finish(const Layout& L, const float4* __restrict__ mc, uint8_t* sc,
                                           uint32_t* s_amax, const PartRows<H>& pr, uint32_t tid) {
  auto row_scale = [&](uint32_t r) { return __uint_as_float(s_amax[r]); };
  const uint32_t rows = 1u << pr.lgr, rows3 = L.R3 >> pr.lgp;
  for (uint32_t i = tid; i < 2 * rows + rows3; i += NT) {
    const bool l1 = i < rows, l2 = !l1 && i < 2 * rows;
    const uint32_t r = l1 ? pr.row0 + i : (l2 ? pr.row0 + i - rows : pr.part * rows3 + i - 2 * rows);
    uint32_t* at = &s_amax[l1 ? r : (l2 ? H + r : 2 * H + r)];
    const float amax = __uint_as_float(*at), scale = amax > 0.0f ? amax / 448.0f : 1.0f;
    *at = __float_as_uint(scale);
    *reinterpret_cast<float*>(sc + (l1 ? L.s_sc1 : (l2 ? L.s_sc2 : L.s_sc3)) + (uint64_t)r * 4) = scale;
  }
  __syncthreads();
  // W1: the four k-blocks of one 16-byte storage block of a row (k-blocks 4j .. 4j + 3,
  // the missing ones of a row's last block zero) in one thread, written whole
  const uint32_t KB1 = L.KB1, nquads = ((KB1 + 3) >> 2) << pr.lgr;
#pragma unroll 1
  for (uint32_t q = tid; q < nquads; q += NT) {
    const uint32_t row = pr.row0 + (q & (rows - 1)), j = q >> pr.lgr;
    const float scale = row_scale(row), inv = 1.0f / scale;
    uint32_t wq[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t kb = 4 * j + t;
      wq[t] = kb < KB1 ? fp8_quantise4(mc[kb * H + row], scale, inv) : 0u;
    }
    typedef unsigned int u32x4s __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(u32x4s{wq[0], wq[1], wq[2], wq[3]},
                                reinterpret_cast<u32x4s*>(sc + L.s_w1 + ((uint64_t)j * H + row) * 16));
  }
  const uint32_t n2 = (H / 4) << pr.lgr;
  for (uint32_t q = tid; q < n2; q += NT) {
    const uint32_t u = part_w2_unit<H>(L, pr, q), e = u - L.u_w2, row = e & (H - 1), kb = e / H;
    *reinterpret_cast<uint32_t*>(sc + L.s_w2 + ((uint64_t)(kb >> 2) * H + row) * 16 + (kb & 3) * 4) =
        fp8_quantise4(mc[u], row_scale(H + row), 1.0f / row_scale(H + row));
  }
  const uint32_t n3 = (L.R3 * (H / 4)) >> pr.lgp;
  for (uint32_t q = tid; q < n3; q += NT) {
    const uint32_t e = pr.part * n3 + q, row = e / (H / 4);
    *reinterpret_cast<uint32_t*>(sc + L.s_w3 + (uint64_t)4 * e) =
        fp8_quantise4(mc[L.u_w3 + e], row_scale(2 * H + row), 1.0f / row_scale(2 * H + row));
  }
}

// The birth launch's arguments in one struct, which the kernel reads where it uses
// them: args() is the argument segment behind an empty asm statement the compiler
// cannot see through, so that what is read through one call is not kept in scalar
// registers beyond the next.  Held over the noise loops the pointers and sizes of
// the rest of the kernel push that loop's own constants and keys out (its body grew
// from 243 to 321 instructions, and the births of a 65,536-agent world with 840 of
// them a step from 79 to 116 us).
struct WeightArgs {   // the first members of both kernels' arguments that write weights
  Dev d;
  Layout L;
};
struct CommitArgs {
  Dev d;
  Layout L;
  TileScratch ts;
  uint32_t base, first_birth, n_birth_blocks, ranked;   // first_birth: the first birth block's number
};
static_assert(offsetof(CommitArgs, d) == offsetof(WeightArgs, d) && offsetof(CommitArgs, L) == offsetof(WeightArgs, L),
              "write_weights reads these through WeightArgs");
// (The segment's address is a kernel's own: whatever calls args() is always inlined.)
template <typename A = CommitArgs>
__device__ __forceinline__ const A& args() {
  typedef const __attribute__((address_space(4))) A* seg_ptr;
  seg_ptr p = (seg_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const A*)p;
}

// One part of an agent's weights, the storage copy quantised from the master.
//  BIRTH: master = parent master + sigma z (Sec. 3.3 mutation of every parameter), z
//    standard normal from the parent's Philox stream (parent slot, step, MUTATE, block).
//  INIT: N(0, sd^2) weights with the layer's sd, from (slot, step 0, WINIT), zero biases.
//  REQUANT: the master is there already.
// Returns the part's share of the agent's |theta|^2 (valid in thread 0).
enum WeightMode { W_BIRTH, W_INIT, W_REQUANT };
struct Noise {
  double sd[3];   // sigma, or the three layers' standard deviations
  uint32_t key0, key1, slot, step;
};
template <int WDT, int H, int NT, int MODE>
__device__ __forceinline__ double write_weights(uint32_t child, uint32_t parent, const Noise nz, const PartRows<H> pr,
                                const double2* tab, uint32_t* s_amax, double* s_red) {
  constexpr uint32_t stream = MODE == W_BIRTH ? ST_MUTATE : ST_WINIT;
  const uint32_t tid = threadIdx.x, key0 = nz.key0, key1 = nz.key1, rng_slot = nz.slot, step = nz.step;
  const WeightArgs& a0 = args<WeightArgs>();
  // the parameter from its normal and its parent's (or present) value
  auto param = [](double z, double sd, float from) {
    return MODE == W_BIRTH ? (float)__builtin_fma(sd, z, (double)from) : (MODE == W_INIT ? (float)(z * sd) : from);
  };
  auto from4 = [&](const float4* p) { return MODE == W_INIT ? make_float4(0.0f, 0.0f, 0.0f, 0.0f) : stream_load4(p); };
  auto normals = [&](uint32_t blk, double z[4]) {
    if (MODE != W_REQUANT) gauss4k(key0, key1, rng_slot, step, stream, blk, tab, z);
  };
  auto put = [&](float4* p, const float (&v)[4]) {
    if (MODE != W_REQUANT) stream_store4<WDT>(p, v[0], v[1], v[2], v[3]);
  };
  const float4* __restrict__ mp = reinterpret_cast<const float4*>(a0.d.master + (uint64_t)parent * a0.L.mstride);
  float4* __restrict__ mc = reinterpret_cast<float4*>(a0.d.master + (uint64_t)child * a0.L.mstride);
  uint8_t* sc = a0.d.store + (uint64_t)child * a0.L.sstride;
  if (WDT == 2) {
    for (uint32_t i = tid; i < 2 * H + a0.L.R3; i += NT) s_amax[i] = 0u;
    __syncthreads();
  }
  const double sd1 = nz.sd[0];
  double tsum = 0.0;
  // W1 (most of the units) without the layer decode, then the other layers
  const uint32_t KB1 = a0.L.KB1, s_w1 = a0.L.s_w1, lgr = pr.lgr, row0 = pr.row0, rmask = (1u << lgr) - 1u;
  if (WDT == 1) {
    // BF16: the two units of one 16-byte storage block (k-blocks 2j and 2j + 1 of a
    // row) in one thread, so that the block is written whole and, like the
    // master, streamed past the caches (the second half of a row's last block is
    // padding when the row has an odd number of k-blocks: zero)
    const uint32_t npairs = ((KB1 + 1) >> 1) << lgr;
#pragma unroll 1
    for (uint32_t q = tid; q < npairs; q += NT) {
      const uint32_t row = row0 + (q & rmask), j = q >> lgr, kb0 = 2 * j;
      const bool two = kb0 + 1 < KB1;
      const uint32_t u0 = kb0 * H + row, u1 = u0 + H;
      const float4 a = from4(mp + u0);
      const float4 b = two ? from4(mp + u1) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      const float pa[4] = {a.x, a.y, a.z, a.w}, pb[4] = {b.x, b.y, b.z, b.w};
      float va[4], vb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      double z[4] = {0.0, 0.0, 0.0, 0.0};
      normals(row * KB1 + kb0, z);
#pragma unroll
      for (int i = 0; i < 4; ++i) va[i] = param(z[i], sd1, pa[i]);
      if (two) {
        normals(row * KB1 + kb0 + 1, z);
#pragma unroll
        for (int i = 0; i < 4; ++i) vb[i] = param(z[i], sd1, pb[i]);
        put(mc + u1, vb);
      }
      put(mc + u0, va);
#pragma unroll
      for (int i = 0; i < 4; ++i) tsum += (double)va[i] * (double)va[i] + (double)vb[i] * (double)vb[i];
      typedef unsigned int u32x4s __attribute__((ext_vector_type(4)));
      const u32x4s blk = {bf16_pair(va[0], va[1]), bf16_pair(va[2], va[3]),
                          bf16_pair(vb[0], vb[1]), bf16_pair(vb[2], vb[3])};
      __builtin_nontemporal_store(blk, reinterpret_cast<u32x4s*>(sc + s_w1 + ((uint64_t)j * H + row) * 16));
    }
  } else {
    const uint32_t n1 = KB1 << lgr;
    auto unit_of = [&](uint32_t q) { return (q >> lgr) * H + row0 + (q & rmask); };
    float4 next = tid < n1 ? from4(mp + unit_of(tid)) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 1
    for (uint32_t q = tid; q < n1; q += NT) {
      const float4 p4 = next;   // this unit's parent values, loaded one unit ahead
      if (q + NT < n1) next = from4(mp + unit_of(q + NT));
      const uint32_t row = row0 + (q & rmask), kb = q >> lgr;
      const float pv[4] = {p4.x, p4.y, p4.z, p4.w};
      double z[4] = {0.0, 0.0, 0.0, 0.0};
      normals(row * KB1 + kb, z);
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = param(z[i], sd1, pv[i]);
      put(mc + kb * H + row, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) tsum += (double)v[i] * (double)v[i];
      store_unit<WDT, H>(a0.L, sc, 0, row, kb, v, s_amax);
    }
  }
  const Layout& L = args<WeightArgs>().L;
  const uint32_t n2 = (H / 4) << lgr, nrest = n2 + part_rest_count<H>(L, pr);
#pragma unroll 1
  for (uint32_t q = tid; q < nrest; q += NT) {
    const uint32_t u = q < n2 ? part_w2_unit<H>(L, pr, q) : part_rest_unit<H>(L, pr, q - n2);
    const UnitPos up = unit_pos<H>(L, u);
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (up.nvalid > 0 && !(MODE == W_INIT && up.layer >= 3)) {
      const float4 p4 = from4(mp + u);
      const float pv[4] = {p4.x, p4.y, p4.z, p4.w};
      double z[4] = {0.0, 0.0, 0.0, 0.0};
      normals(up.blk, z);
      const double sd = MODE == W_INIT ? (up.layer == 1 ? nz.sd[1] : nz.sd[2]) : sd1;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (i < (int)up.nvalid) ? param(z[i], sd, pv[i]) : 0.0f;
    }
    put(mc + u, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) tsum += (double)v[i] * (double)v[i];
    store_unit<WDT, H>(L, sc, up.layer, up.row, up.kb, v, s_amax);
  }
  if (WDT == 2) {
    __syncthreads();
    fp8_finish<H, NT>(L, mc, sc, s_amax, pr, tid);
  }
  return block_sum_f64<NT>(tsum, s_red);
}

// The integer part of birth k of world w (one thread a birth): the child's state, what the
// parent gives, its colour trait, and the window channels that the birth changes
// after the cell pass of the step: the child's cell (occupied now, the child's
// energy or colour) and, in the sense bytes, the parent's (its energy after the birth).
__device__ __forceinline__ void place_child(const Dev& d, uint32_t w, uint32_t k, uint32_t p_local, uint32_t c_local,
                                            const double2* tab) {
  const WorldParams& wp = d.wp[w];
  const uint32_t pg = wp.slot_off + p_local, cg = wp.slot_off + c_local;
  const int t = d.tgt[pg], E = d.energy[pg] - wp.e_child, pc = d.pos[pg];
  const uint8_t facing = d.facing[pg];
  const unsigned long long puid = d.uid[pg];
  const uint32_t gt = wp.cell_off + (uint32_t)t, gp = wp.cell_off + (uint32_t)pc;
  const uint32_t word = d.rgb ? d.rgb[gt] : d.sense[gt], own = d.rgb ? 0u : d.sense[gp];
  uint32_t colour = 0u;
  if (d.colour) {   // the parent's plus sigma N(0,1) per channel
    double z[4];
    gauss4k(wp.key0, wp.key1, p_local, (uint32_t)d.draft[w].step, ST_COLOUR_MUTATE, 0u, tab, z);
    const double sigma = (double)wp.sigma;
    const float4 p = d.colour[pg];
    const float4 c = make_float4((float)__builtin_fma(sigma, z[0], (double)p.x),
                                 (float)__builtin_fma(sigma, z[1], (double)p.y),
                                 (float)__builtin_fma(sigma, z[2], (double)p.z), 0.0f);
    d.colour[cg] = c;
    colour = colour_word(c);
  }
  d.energy[pg] = E;
  d.pos[cg] = t;
  d.occ[gt] = (int)c_local;
  d.facing[cg] = facing;
  d.energy[cg] = wp.e_child;
  d.age[cg] = 0;
  d.uid[cg] = d.draft[w].uid_next + k;
  d.puid[cg] = puid;
  if (d.ep) {   // ecology: the parent gives water and biomass; the child starts at hp_child
    const eco_ecology& e = d.ep[w];
    d.water[pg] -= e.w_child;
    d.biomass[pg] -= e.b_child;
    d.water[cg] = e.w_child;
    d.biomass[cg] = e.b_child;
    d.hp[cg] = e.hp_child;
  }
  if (d.rgb) {
    d.rgb[gt] = (d.colour ? (word & 0xFF000000u) | colour : word) | 1u << 24;
  } else {
    d.sense[gt] = (uint8_t)((word & 6u) | agent_sense(wp, wp.e_child));
    d.sense[gp] = (uint8_t)((own & 6u) | agent_sense(wp, E));
  }
}

// World w's statistics record and the clock advance (one block): its draft (made here,
// or by the small-world kernel) completed by the births.  With births, the trait moments follow once
// the children are written (settle_record).
__device__ __forceinline__ void world_record(const Dev& d, const TileScratch& ts, uint32_t w, bool ranked) {
  __shared__ StepDraft drafted;
  __shared__ uint32_t winners;
  if (!ranked) world_draft<kSlotTile>(d, ts, w, &drafted, &winners);
  const StepDraft& dr = ranked ? d.draft[w] : drafted;
  WorldVar& v = d.wv[w];
  const uint32_t nw = ranked ? v.n_win : winners, n_free = v.n_free;
  if (threadIdx.x != 0) return;
  const uint32_t nb = min(nw, n_free), n = dr.n0 + nb;
  eco_stats st = {};
  v.n_births = nb;
  v.n0 = dr.n0;
  v.mean = dr.mean;
  v.m2 = dr.m2;
  v.n_live = n;
  v.uid_next = dr.uid_next + nb;
  v.step = dr.step + 1;
  st.step = dr.step + 1;
  st.population = n;
  st.births = nb;
  st.deaths = dr.count[PC_DEATHS];
  st.killed = dr.count[PC_KILLED];
  st.eaten = dr.count[PC_EATEN];
  st.regrown = dr.regrown;
  st.moves_ok = dr.count[PC_MOVES_OK];
  st.moves_blocked = dr.count[PC_MOVES_BLOCKED];
  st.births_blocked_cell = dr.count[PC_BB_CELL];
  st.births_blocked_capacity = nw - nb;
  st.resource_total = dr.resource_total;
  for (int a = 0; a < 9; ++a) st.action_hist[a] = dr.count[PC_HIST + a];
  st.energy_total = (double)dr.energy;
  st.trait_mean = n ? dr.mean : 0.0;
  st.trait_var = n ? dr.m2 / (double)n : 0.0;
  if (d.ep) {
    st.water_total = dr.water;
    st.biomass_total = dr.biomass;
    st.hp_total = dr.hp + (unsigned long long)nb * (unsigned long long)d.ep[w].hp_child;
  }
  d.ring[(uint64_t)w * kStatsRing + (st.step % kStatsRing)] = st;
}

// The next step's live list of one slot tile: the survivors and the free slots
// whose rank is below the world's births, in slot order (the live slots before the
// tile are the slots that were not free there and the births among those that
// were), and the tile's flags.
__device__ __forceinline__ void live_tile(const Dev& d, const TileScratch& ts, uint32_t tile, bool ranked) {
  constexpr int NW = kSlotTile / 64;
  __shared__ uint32_t s_live[NW], s_free[NW], s_win[NW];
  const int wave = threadIdx.x >> 6;
  const Tile tl = slot_tile(ts, tile);
  const uint32_t w = tl.world;
  const uint32_t slot_off = slot_offset(d, ts, w);
  const uint32_t free_before = ts.scan[tile * 4 + 2], n_free = d.wv[w].n_free, n_win = d.wv[w].n_win;
  const bool summed = ts.cap0 && !ranked;
  uint32_t win = 0;
  if (summed)
    for (uint32_t i = threadIdx.x; i < ts.n_slot_tiles; i += kSlotTile) win += ts.scan[i * 4];
  const bool in = threadIdx.x < tl.count;
  const uint32_t local = tl.start + threadIdx.x, slot = slot_off + local;
  const uint8_t fl = in ? d.flags[slot] : (uint8_t)0;
  const bool survivor = (fl & kAlive) != 0;
  const uint64_t am = __ballot(survivor), fm = __ballot(in && !survivor);
  win = wave_scan(win);
  if ((threadIdx.x & 63u) == 63u) {
    s_live[wave] = (uint32_t)__builtin_popcountll(am);
    s_free[wave] = (uint32_t)__builtin_popcountll(fm);
    s_win[wave] = win;
  }
  __syncthreads();
  uint32_t surv = lanes_before(am), fr = free_before + lanes_before(fm), nw = summed ? 0u : n_win;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    if (i < wave) {
      surv += s_live[i];
      fr += s_free[i];
    }
    if (summed) nw += s_win[i];
  }
  const uint32_t nb = min(nw, n_free);
  const bool alive = survivor || (in && fr < nb);
  // live slots before this one: those of the earlier tiles, this tile's survivors, and
  // the births with a smaller free rank
  if (alive) d.live[slot_off + (tl.start - free_before) + surv + min(fr, nb)] = (int)local;
  const uint8_t nf = alive ? kAlive : (uint8_t)0;
  if (in && fl != nf) d.flags[slot] = nf;
}

// The last launch of a step.  The first blocks: the live list of a slot tile each,
// the record of a world each, and with terrain the settled water of a cell tile each
// (small worlds: k_step_small has settled it).  The other n_birth_blocks: births (persistent over all
// worlds' births), as many blocks as are resident at once.  One block per child where
// there are enough children to fill the chip, else 2^lgp blocks share a child, each a
// part of its rows (child_split), so that few births do not take as long as one child
// on four waves (a 1024 x 1024 world of 32,768 agents with 133,767 parameters and
// 210 births a step: 153 to 83 us).  The children's state is placed apart from their
// weights, a thread a birth.  A birth's parent is found from the tiles' winner counts
// (prefix sums over 256 runs of tiles in LDS, then the tiles of the run), or
// read from bparent where the small-world kernel has ranked the winners.
// base: the first block's number (the roles can be launched apart).
template <int WDT, int H>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WDT == 1 ? 6 : 7)))
void k_birth_commit(CommitArgs by_value) {
  __shared__ uint32_t off[kMaxWorlds + 1], off_win[kMaxWorlds + 1];
  __shared__ uint32_t run_win[256 + 1];
  __shared__ uint32_t red[4];
  __shared__ uint32_t s_amax[128 + 128 + 16];
  __shared__ double s_red[4];
  __shared__ double2 tab[kNoiseTable];
  static_assert(kNoiseTable == 512, "two table entries per thread");
  uint32_t first = blockIdx.x, lgp = 0;
  {
    const CommitArgs& a = args();
    const uint32_t T = a.ts.n_slot_tiles, block = first + a.base;
    if (block < T) {
      live_tile(a.d, a.ts, block, a.ranked);
      return;
    }
    if (block < T + a.d.n_worlds) {
      world_record(a.d, a.ts, block - T, a.ranked);
      return;
    }
    if (block < a.first_birth) {
      const Tile ct = cell_tile(a.ts, block - T - a.d.n_worlds);
      settle_water(a.d, a.d.wp[ct.world], ct);
      return;
    }
    first = block - a.first_birth;
    if (a.ranked && births_of(a.d.wv[0]) == 0) return;
    // the winners before each run of tiles, and the worlds' births
    const bool summed = a.ts.cap0 && !a.ranked;
    const uint32_t per = (T + 255) / 256;   // tiles per run
    uint32_t own = 0;
    if (!a.ranked)
      for (uint32_t t = threadIdx.x * per; t < min((threadIdx.x + 1) * per, T); ++t) own += a.ts.scan[t * 4];
    const uint32_t inc = wave_scan(own);
    if ((threadIdx.x & 63u) == 63u) red[threadIdx.x >> 6] = inc;
    if (!summed) birth_offsets(a.d.wv, a.d.n_worlds, off, off_win);
    else __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
      if (i < threadIdx.x >> 6) before += red[i];
      all += red[i];
    }
    const uint32_t total = summed ? min(all, a.d.wv[0].n_free) : off[a.d.n_worlds];
    lgp = child_split(a.ts, H, total);
    if (first >= (total << lgp) + (total + 255) / 256) return;   // nothing for this block (no block, without births)
    run_win[threadIdx.x] = before + inc - own;
    tab[threadIdx.x] = a.d.trig[threadIdx.x];
    tab[256 + threadIdx.x] = a.d.trig[256 + threadIdx.x];
    if (threadIdx.x == 255) {
      run_win[256] = all;
      if (summed) {
        off[0] = off_win[0] = 0;
        off[1] = total;
        off_win[1] = all;
      }
    }
    __syncthreads();
  }
  // items: 256 children's states each, then the children's parts
  const uint32_t n_place = (off[args().d.n_worlds] + 255) / 256, n_items = n_place + (off[args().d.n_worlds] << lgp);
  // the parent of the world's birth whose winner is number win of the object's
  auto parent_of = [&](const CommitArgs& a, uint32_t slot_off, uint32_t k, uint32_t win) {
    if (a.ranked) return (uint32_t)a.d.bparent[slot_off + k];
    const uint32_t T = a.ts.n_slot_tiles, per = (T + 255) / 256;
    const uint32_t r = find_world(run_win, 256, win), end = min((r + 1) * per, T);
    uint32_t rem = win - run_win[r], t = r * per;   // its place among the run's
    for (; t + 1 < end; ++t) {
      const uint32_t c = a.ts.scan[t * 4];
      if (rem < c) break;
      rem -= c;
    }
    const uint32_t start = slot_tile(a.ts, t).start;
    return start + (uint32_t)a.d.bparent[slot_off + start + rem];
  };
  auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
  for (uint32_t i = first; i < n_items; i += args().n_birth_blocks) {
    const CommitArgs& a = args();
    const Dev& d = a.d;
    if (i < n_place) {
      const uint32_t g = i * 256 + threadIdx.x;
      if (g < off[d.n_worlds]) {
        const uint32_t w = find_world(off, d.n_worlds, g), k = g - off[w], slot_off = d.wp[w].slot_off;
        place_child(d, w, k, parent_of(a, slot_off, k, off_win[w] + k), (uint32_t)d.freel[slot_off + k], tab);
      }
      continue;
    }
    const uint32_t j = i - n_place, g = j >> lgp, part = j & ((1u << lgp) - 1u);
    const uint32_t w = uniform(find_world(off, d.n_worlds, g)), k = g - uniform(off[w]);
    const WorldParams& wp = d.wp[w];
    const uint32_t slot_off = wp.slot_off, child = slot_off + uniform((uint32_t)d.freel[slot_off + k]);
    const uint32_t p_local = uniform(parent_of(a, slot_off, k, uniform(off_win[w]) + k));
    const Noise nz{{(double)wp.sigma, 0.0, 0.0}, wp.key0, wp.key1, p_local, (uint32_t)d.draft[w].step};
    const double t = write_weights<WDT, H, 256, W_BIRTH>(child, slot_off + p_local, nz, part_rows<H>(part, lgp), tab,
                                                         s_amax, s_red);
    if (threadIdx.x == 0) {
      const CommitArgs& b = args();
      if (lgp || b.ranked) b.ts.parts[j] = t;
      if (!lgp) b.d.trait[child] = t;
    }
  }
}

// Trait moments of a group of agents: count, mean and the sum of squared
// deviations from that mean.  Two groups combine by the pairwise update of
// Chan, Golub and LeVeque (1979): with delta = mean_b - mean_a and n = n_a + n_b,
// mean = mean_a + delta n_b / n and M2 = M2_a + M2_b + delta^2 n_a n_b / n, which
// never subtracts two large sums (the variance of the whole is M2 / n).
struct Moments {
  double n, mean, m2;
};

__device__ __forceinline__ Moments merge_moments(const Moments& a, const Moments& b) {
  if (b.n == 0.0) return a;
  if (a.n == 0.0) return b;
  const double n = a.n + b.n, delta = b.mean - a.mean;
  return Moments{n, a.mean + delta * (b.n / n), a.m2 + b.m2 + delta * delta * (a.n * b.n / n)};
}

// Merge of one Moments per thread over the block, in a fixed order (a tree within
// each wave, then the waves in order); the result is valid in thread 0.
template <int NT>
__device__ __forceinline__ Moments block_merge_moments(Moments m, double (*red)[3]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const Moments o{__shfl_down(m.n, d), __shfl_down(m.mean, d), __shfl_down(m.m2, d)};
    if (lane < d) m = merge_moments(m, o);
  }
  if (lane == 0) {
    red[wave][0] = m.n;
    red[wave][1] = m.mean;
    red[wave][2] = m.m2;
  }
  __syncthreads();
  Moments t{0.0, 0.0, 0.0};
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) t = merge_moments(t, Moments{red[i][0], red[i][1], red[i][2]});
  __syncthreads();
  return t;  // valid in thread 0
}

// Live list and statistics of init and state writes (a step's are written by
// k_birth_commit).  Pass 1 (slot tiles): live count, energy sum and the trait moments of
// the tile (its mean, then the squared deviations from it: two passes over the
// tile's values, which stay in registers).
__global__ __launch_bounds__(kSlotTile) void k_compact_count(Dev d, TileScratch ts, int only_world) {
  __shared__ unsigned long long red64[kSlotTile / 64];
  __shared__ double redf[kSlotTile / 64];
  __shared__ double bcastf;
  const Tile tl = ts.slot_tiles[blockIdx.x];
  if (only_world >= 0 && (int)tl.world != only_world) return;
  const WorldParams wp = d.wp[tl.world];
  bool alive = false;
  long long e = 0;
  double t = 0.0;
  if (threadIdx.x < tl.count) {
    const uint32_t slot = wp.slot_off + tl.start + threadIdx.x;
    alive = d.flags[slot] & kAlive;
    if (alive) {
      e = d.energy[slot];
      t = d.trait[slot];
    }
  }
  const unsigned long long n = block_sum_u64<kSlotTile>(alive ? 1ull : 0ull, red64);
  const unsigned long long es = block_sum_u64<kSlotTile>((unsigned long long)e, red64);
  const double s1 = block_sum_f64<kSlotTile>(t, redf);
  if (threadIdx.x == 0) bcastf = n ? s1 / (double)n : 0.0;
  __syncthreads();
  const double tile_mean = bcastf;
  const double dv = alive ? t - tile_mean : 0.0;
  const double m2 = block_sum_f64<kSlotTile>(dv * dv, redf);
  if (d.ep) {   // ecology: water, biomass and health carried by the tile's live agents
    const uint32_t slot = wp.slot_off + tl.start + threadIdx.x;
    const bool on = alive && threadIdx.x < tl.count;
    const unsigned long long ws = block_sum_u64<kSlotTile>(on ? (unsigned long long)d.water[slot] : 0ull, red64);
    const unsigned long long bs = block_sum_u64<kSlotTile>(on ? (unsigned long long)d.biomass[slot] : 0ull, red64);
    const unsigned long long hs = block_sum_u64<kSlotTile>(on ? (unsigned long long)d.hp[slot] : 0ull, red64);
    if (threadIdx.x == 0) {
      ts.ecosum[3 * blockIdx.x] = ws;
      ts.ecosum[3 * blockIdx.x + 1] = bs;
      ts.ecosum[3 * blockIdx.x + 2] = hs;
    }
  }
  if (threadIdx.x == 0) {
    ts.scan[blockIdx.x * 4 + 3] = (uint32_t)n;
    ts.esum[blockIdx.x] = (long long)es;
    ts.tmean[blockIdx.x] = tile_mean;
    ts.tm2[blockIdx.x] = m2;
  }
}

// The statistics record of world w as it stands once pass 1's counts are in (run by
// the block of the world's last slot tile, NT threads); the grid totals come from
// k_resource_total.
template <int NT>
__device__ void world_finalize(const Dev& d, const TileScratch& ts, uint32_t w) {
  __shared__ uint32_t red[NT / 64 + 1];
  __shared__ unsigned long long red64[NT / 64];
  __shared__ double redm[NT / 64][3];
  const uint32_t t0 = ts.tile_rng[4 * w], t1 = ts.tile_rng[4 * w + 1];
  const uint32_t nt = t1 - t0;
  const uint32_t per = (nt + NT - 1) / NT;
  const uint32_t lo = t0 + threadIdx.x * per, hi = min(lo + per, t1);
  uint32_t n = 0;
  long long es = 0;
  Moments tm{0.0, 0.0, 0.0};   // the trait moments of this thread's tiles, merged in tile order
  for (uint32_t t = lo; t < hi; ++t) {
    const uint32_t nl = ts.scan[t * 4 + 3];
    n += nl;
    es += ts.esum[t];
    tm = merge_moments(tm, Moments{(double)nl, ts.tmean[t], ts.tm2[t]});
  }
  uint32_t N;
  block_exscan<NT>(n, red, &N);
  const unsigned long long E = block_sum_u64<NT>((unsigned long long)es, red64);
  const Moments TM = block_merge_moments<NT>(tm, redm);
  unsigned long long eco_h = 0;   // ecology: health
  if (d.ep) {
    unsigned long long c = 0;
    for (uint32_t t = lo; t < hi; ++t) c += ts.ecosum[3 * t + 2];
    eco_h = block_sum_u64<NT>(c, red64);
  }
  if (threadIdx.x == 0) {
    WorldVar& v = d.wv[w];
    eco_stats st = {};
    if (d.ep) st.hp_total = eco_h;
    v.n_live = N;
    st.step = v.step;
    st.population = N;
    st.energy_total = (double)(long long)E;
    st.trait_mean = N ? TM.mean : 0.0;
    st.trait_var = N ? TM.m2 / (double)N : 0.0;
    d.ring[(uint64_t)w * kStatsRing + (v.step % kStatsRing)] = st;
  }
}

// Sum over the tiles [lo, hi) of scan[t][c]; all threads of the block get the sum.
template <int NT>
__device__ __forceinline__ uint32_t tiles_sum(const TileScratch& ts, uint32_t lo, uint32_t hi, int c,
                                              unsigned long long* red64, uint32_t* bcast) {
  uint32_t v = 0;
  for (uint32_t t = lo + threadIdx.x; t < hi; t += NT) v += ts.scan[t * 4 + c];
  const unsigned long long tot = block_sum_u64<NT>(v, red64);
  if (threadIdx.x == 0) *bcast = (uint32_t)tot;
  __syncthreads();
  const uint32_t r = *bcast;
  __syncthreads();
  return r;
}

// Pass 2.  Slot-tile blocks: the tile's live slots at their
// offsets in the world's live list (offset = live counts of the world's earlier
// tiles, summed here); the world's last tile also writes the statistics record.
// Blocks past the slot tiles build the window channels of one cell tile each.
// only_world >= 0 restricts both parts.
__global__ __launch_bounds__(kSlotTile) void k_compact_write(Dev d, TileScratch ts, int only_world) {
  __shared__ uint32_t red[kSlotTile / 64 + 1];
  __shared__ unsigned long long red64[kSlotTile / 64];
  __shared__ uint32_t bcast;
  if (blockIdx.x >= ts.n_slot_tiles) {
    const Tile ct = ts.cell_tiles[blockIdx.x - ts.n_slot_tiles];
    if (only_world < 0 || (int)ct.world == only_world) window_cells(d, ct);
    return;
  }
  const Tile tl = ts.slot_tiles[blockIdx.x];
  if (only_world >= 0 && (int)tl.world != only_world) return;
  const uint32_t w = tl.world;
  const WorldParams wp = d.wp[w];
  const uint32_t t0 = ts.tile_rng[4 * w], t1 = ts.tile_rng[4 * w + 1];
  const uint32_t ol = tiles_sum<kSlotTile>(ts, t0, blockIdx.x, 3, red64, &bcast);
  const bool in = threadIdx.x < tl.count;
  const uint32_t local = tl.start + threadIdx.x;
  const bool alive = in && (d.flags[wp.slot_off + local] & kAlive);
  uint32_t tot;
  const uint32_t r = ol + block_exscan<kSlotTile>(alive ? 1u : 0u, red, &tot);
  if (alive) d.live[wp.slot_off + r] = (int)local;
  if (blockIdx.x + 1 == t1) world_finalize<kSlotTile>(d, ts, w);
}

// ---------------------------------------------------------------------------
// The moves, claims, cell pass and ranking of a step for an object of one small
// world, in one block: the phases of k_move and k_claim_cells with the
// world's scans done inside the block, before the same last launch (k_birth_commit:
// births, live list, record).  A small world's step is bound by the latency of its
// launches, and this replaces two dependent launches by one.  A thread scans a
// contiguous range of slots, so every scan is one block-wide exclusive sum.  ECO: the
// world has the ecology (d.ep set); the single-resource instantiation carries none of
// the ecology's phases (behind a run-time test they made its step measurably slower).
// ---------------------------------------------------------------------------
template <bool ECO>
__global__ __launch_bounds__(1024) void k_step_small(Dev d, TileScratch ts, uint32_t n_actions, uint32_t H) {
  // threads; slots or cells per thread in one pass (one 4-byte load of bytes); passes over
  // the slots (the capacity is at most NT CH NP)
  constexpr int NT = 1024, CH = 4, NP = 2, NW = NT / 64;
  static_assert(NT * CH * NP == ECO_SMALL_STEP_MAX_SLOTS, "the slot passes cover the largest object taken");
  static_assert(NT * CH == ECO_SMALL_STEP_MAX_CELLS, "a group of four cells per thread");
  static_assert(64 * CH == kSlotTile, "one wave's slots of a pass are one slot tile");
  if (blockIdx.x == 1) {   // the second block completes the last step's record from the blocks' shares
    settle_record<NT, false>(d, ts, 0, H, true);
    return;
  }
  __shared__ uint32_t cnt[kSlotPart];              // step counters (PC_*)
  __shared__ unsigned long long ccnt[kCellPart];   // regrown units, resource total (the ecology: grid energy), grid water, biomass
  __shared__ unsigned long long rank_red[NW];        // the ranking scan's wave totals
  __shared__ uint32_t live_red[NW];                  // the waves' survivors
  __shared__ unsigned long long red64[NW];           // the waves' energy sums
  __shared__ double mean_red[NW], m2_red[NW];        // the waves' trait means and sums of squared deviations
  __shared__ unsigned long long eco_red[3][NW];      // the ecology: the waves' carried water, biomass, health
  // per cell: the agent bit and energy bin of its occupant after the moves (0: none),
  // written by the agents, read by the cell pass
  __shared__ __align__(16) uint8_t s_agent[ECO_SMALL_STEP_MAX_CELLS];
  // colour vision: the surviving agents' colour words by slot, written by the agents,
  // read by the cell pass (no occupant-then-colour lookup chain)
  __shared__ uint32_t s_col[ECO_SMALL_STEP_MAX_SLOTS];
  const uint32_t tid = threadIdx.x;
  const int lane = (int)(tid & 63u), wave = (int)(tid >> 6);
  // live-list entry tid, loaded together with the world's live count: the
  // thread's only agent when there are at most NT (the object's one world
  // starts at slot 0; the list's allocation holds total_slots entries)
  const int32_t live_tid = d.live[min(tid, d.total_slots - 1u)];
  if (tid < kSlotPart) cnt[tid] = 0;
  if (tid < kCellPart) ccnt[tid] = 0;
  constexpr uint32_t w = 0;
  const WorldParams wp = d.wp[w];
  const uint32_t step = (uint32_t)d.wv[w].step, n_live = d.wv[w].n_live, cap = wp.cap, cells = wp.cells;
  const int32_t* live = d.live + wp.slot_off;
  // each thread's contiguous range of the live list
  const uint32_t per_l = (n_live + NT - 1) / NT;
  const uint32_t l0 = min(tid * per_l, n_live), l1 = min(l0 + per_l, n_live);
  const bool sense_bytes = d.rgb == nullptr;   // window channels as sense bytes (else rendered words)
  if (sense_bytes)
    for (uint32_t c0 = tid * 16; c0 < cells; c0 += NT * 16) *reinterpret_cast<uint4*>(s_agent + c0) = make_uint4(0, 0, 0, 0);
  __syncthreads();

  // the traits of the last step's children
  const uint32_t n_children = d.wv[w].n_births;
  if (n_children) {
    const uint32_t lgp = child_split(ts, H, n_children);
    for (uint32_t k = NT - 1 - tid; k < n_children; k += NT)   // from the last threads on: the first have the agents
      d.trait[wp.slot_off + (uint32_t)d.freel[wp.slot_off + k]] = child_trait(d, ts, lgp, true, k, 0u);
  }
  // 1. moves, eating, costs and deaths of the step's live agents (what the thread's
  // first one is afterwards stays in registers for the next phase)
  Moved held{0, 0, false};
  int held_act = 0, held_facing = 0;
  for (uint32_t i = l0; i < l1; ++i) {
    const uint32_t local = (uint32_t)(i == tid ? live_tid : live[i]), slot = wp.slot_off + local;
    const int a = d.act[slot], pos = d.pos[slot], t = d.tgt[slot], E = d.energy[slot], facing = d.facing[slot];
    float4 cv = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (d.colour) cv = d.colour[slot];
    const Moved m = move_agent(d, wp, w, slot, local, step + 1u, a, pos, t, E, cnt);
    if (i == l0) {
      held = m;
      held_act = a;
      held_facing = facing;
    }
    if (m.alive) {
      if (sense_bytes) s_agent[m.cell] = (uint8_t)agent_sense(wp, m.energy);   // one agent per cell
      if (d.colour) s_col[local] = colour_word(cv);
    }
  }
  __syncthreads();
  // 2. birth claims of the agents still alive with their sums (count, energy, what they
  // carry, and the trait mean and sum of squared deviations by Welford's update), and
  // the cell pass
  static_assert(CH * NP <= 32, "a bit per agent of a thread");
  uint32_t wins = 0, nblk = 0, n_t = 0;   // wins: bit i - l0
  long long es = 0;
  double mean_t = 0.0, m2_t = 0.0;
  unsigned long long eco_w[3] = {0, 0, 0};
  for (uint32_t i = l0; i < l1; ++i) {
    const uint32_t slot = wp.slot_off + (uint32_t)(i == tid ? live_tid : live[i]);
    bool alive = held.alive;
    int act = held_act, pos = held.cell, facing = held_facing, energy = held.energy;
    if (i != l0) {
      alive = (d.flags[slot] & kAlive) != 0;
      act = d.act[slot];
      pos = d.pos[slot];
      facing = d.facing[slot];
      energy = d.energy[slot];
    }
    const int water = ECO ? d.water[slot] : 0, biomass = ECO ? d.biomass[slot] : 0, hp = ECO ? d.hp[slot] : 0;
    const double trait = d.trait[slot];
    if (!alive) continue;
    ++n_t;
    es += energy;
    const double dv = trait - mean_t;
    if (n_t == 1) {
      mean_t = trait;
    } else {
      mean_t += dv / (double)n_t;
      m2_t += dv * (trait - mean_t);
    }
    if constexpr (ECO) {
      eco_w[0] += (unsigned long long)water;
      eco_w[1] += (unsigned long long)biomass;
      eco_w[2] += (unsigned long long)hp;
    }
    const int r = birth_claim_agent(d, wp, w, slot, n_actions, act, pos, facing, energy, water, biomass);
    if (r == CLAIM_WON) wins |= 1u << (i - l0);
    nblk += r == CLAIM_BLOCKED ? 1u : 0u;
  }
  nblk = wave_scan(nblk);
  if (lane == 63 && nblk) atomicAdd(&cnt[PC_BB_CELL], nblk);
  const Tile all{w, 0u, cells, 0u};
  if constexpr (ECO) ecology_cells<true, 4>(d, wp, d.ep[w], wp.cell_off, all, step, ccnt, s_col);
  else plain_cells<true, 4>(d, wp, wp.cell_off, all, step, ccnt, s_agent, s_col);
  // the waves' sums (whole waves without agents have none), combined below
  {
    const uint32_t n_w = lane_value(wave_scan(n_t), 63);
    double mean_w = 0.0, m2_w = 0.0;
    unsigned long long ew = 0;
    if (n_w) {
      mean_w = lane_value(wave_scan((double)n_t * mean_t), 63) / (double)n_w;
      m2_w = wave_scan(m2_t + (double)n_t * (mean_t - mean_w) * (mean_t - mean_w));
      ew = wave_scan((unsigned long long)es);
      if constexpr (ECO) {
#pragma unroll
        for (int k = 0; k < 3; ++k) eco_w[k] = wave_scan(eco_w[k]);
      }
    }
    if (lane == 63) {
      live_red[wave] = n_w;
      red64[wave] = ew;
      mean_red[wave] = mean_w;
      m2_red[wave] = m2_w;
      if constexpr (ECO) {
#pragma unroll
        for (int k = 0; k < 3; ++k) eco_red[k][wave] = eco_w[k];
      }
    }
  }
  __syncthreads();
  if (ECO && d.rock) settle_water(d, wp, all);
  // 3. the free slots; a wave's 256 slots of a pass are a slot tile
  uint32_t fm[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const uint32_t b0 = (p * NT + tid) * CH;
    fm[p] = 0;
    if (b0 < cap) {
      const uint32_t v = *reinterpret_cast<const uint32_t*>(d.flags + wp.slot_off + b0);
#pragma unroll
      for (int j = 0; j < CH; ++j)
        if (b0 + j < cap && !((v >> (8 * j)) & kAlive)) fm[p] |= 1u << j;
    }
  }
  // 4. ranking: the claim winners in slot order (the live list's order) and the free
  // slots in ascending order (the recycled-slot free list; only its first Wn entries
  // are used), both ranked by one block scan of 16-bit counts packed in a u64
  // (winners, free slots of each pass; no field carries into the next: every total is
  // at most 8,192).
  const uint32_t nw = (uint32_t)__builtin_popcount(wins);
  static_assert(NP == 2, "the packed ranking scan holds two passes of free slots");
  unsigned long long rtot;
  const unsigned long long rex =
      block_exscan_u64<NT>((unsigned long long)nw | (unsigned long long)__builtin_popcount(fm[0]) << 16 |
                               (unsigned long long)__builtin_popcount(fm[1]) << 32,
                           rank_red, &rtot);
  const uint32_t Wn = (uint32_t)(rtot & 0xFFFFu);
  uint32_t k = (uint32_t)(rex & 0xFFFFu);
  for (uint32_t m = wins; m; m &= m - 1) {
    const uint32_t i = l0 + (uint32_t)__builtin_ctz(m);
    d.bparent[wp.slot_off + k++] = i == tid ? live_tid : live[i];
  }
  uint32_t F = 0;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const uint32_t b0 = (p * NT + tid) * CH;
    uint32_t f = F + (uint32_t)((rex >> (16 * (p + 1))) & 0xFFFFu);
    if (lane == 0 && b0 < cap) ts.scan[(b0 / kSlotTile) * 4 + 2] = f;   // free slots before the wave's tile
    for (uint32_t m = fm[p]; m && f < Wn; m &= m - 1) d.freel[wp.slot_off + f++] = (int)(b0 + __builtin_ctz(m));
    F += (uint32_t)((rtot >> (16 * (p + 1))) & 0xFFFFu);
  }
  // 5. the draft of the statistics record (the block scan's barrier is behind every sum)
  StepDraft* dr = d.draft + w;
  if (tid >= 64 && tid < 64 + kSlotPart) dr->count[tid - 64] = cnt[tid - 64];
  if (wave == 0) {   // lane i < NW holds wave i's sums
    const bool on = lane < NW;
    const uint32_t n_i = on ? live_red[lane] : 0u;
    const double mean_i = on ? mean_red[lane] : 0.0;
    const uint32_t N = lane_value(wave_scan(n_i), 63);
    const double mean = N ? lane_value(wave_scan((double)n_i * mean_i), 63) / (double)N : 0.0;
    const double M2 = wave_scan((on ? m2_red[lane] : 0.0) + (double)n_i * (mean_i - mean) * (mean_i - mean));
    const unsigned long long E = wave_scan(on ? red64[lane] : 0ull);
    unsigned long long carried[3] = {0, 0, 0};
    if constexpr (ECO) {
#pragma unroll
      for (int q = 0; q < 3; ++q) carried[q] = wave_scan(on ? eco_red[q][lane] : 0ull);
    }
    if (lane == 63) {
      dr->regrown = ccnt[0];
      dr->resource_total = ccnt[1];
      dr->water = ECO ? ccnt[2] + carried[0] : 0ull;
      dr->biomass = ECO ? ccnt[3] + carried[1] : 0ull;
      dr->hp = carried[2];
      dr->energy = (long long)E;
      dr->mean = mean;
      dr->m2 = M2;
      dr->n0 = N;
      WorldVar& v = d.wv[w];
      dr->step = v.step;
      dr->uid_next = v.uid_next;
      v.n_win = Wn;
      v.n_free = F;
    }
  }
}

// Rendered window words of one world's cells (after a colour write).
__global__ __launch_bounds__(256) void k_render(Dev d, const Tile* __restrict__ tiles, int only_world) {
  const Tile ct = tiles[blockIdx.x];
  if ((int)ct.world != only_world) return;
  window_cells(d, ct);
}

// Terrain: each cell's way down, the lowest 4-neighbour if strictly lower (the
// first of N, E, S, W among equals), else -1.
__global__ __launch_bounds__(256) void k_flowdir(Dev d, const Tile* __restrict__ tiles, int only_world) {
  const Tile tl = tiles[blockIdx.x];
  if (only_world >= 0 && (int)tl.world != only_world) return;
  const WorldParams wp = d.wp[tl.world];
  for (uint32_t i = threadIdx.x; i < tl.count; i += blockDim.x) {
    const uint32_t c = tl.start + i;
    int best = -1, bh = d.rock[wp.cell_off + c];
    for (int dd = 0; dd < 4; ++dd) {
      const int h = d.rock[wp.cell_off + neighbour(wp, c, dd, +1)];
      if (h < bh) { bh = h; best = dd; }
    }
    d.flowdir[wp.cell_off + c] = (int8_t)best;
  }
}

// Grid totals of the records of init and state writes, whose record has just been
// written with zeros there: first_world + blockIdx.y is the world, its blocks of 1,024
// cells (or slots, at 256 at least) a pass add their shares.
__global__ __launch_bounds__(256) void k_resource_total(Dev d, uint32_t first_world) {
  __shared__ unsigned long long cnt[3];
  const uint32_t w = first_world + blockIdx.y;
  if (threadIdx.x < 3) cnt[threadIdx.x] = 0;
  __syncthreads();
  const WorldParams wp = d.wp[w];
  unsigned long long s = 0, sw = 0, sb = 0;
  const uint32_t first = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
  if (d.ep) {   // ecology: energy on the grid; water and biomass on the grid and in live agents
    for (uint32_t c = first; c < wp.cells; c += stride) {
      const uint32_t g = wp.cell_off + c;
      s += (unsigned long long)d.ce[g];
      sw += (unsigned long long)d.cw[g];
      sb += (unsigned long long)d.cb[g];
    }
    for (uint32_t j = first; j < wp.cap; j += stride) {
      const uint32_t g = wp.slot_off + j;
      if (d.flags[g] & kAlive) {
        sw += (unsigned long long)d.water[g];
        sb += (unsigned long long)d.biomass[g];
      }
    }
  } else {
    for (uint32_t c = 4 * first; c < wp.cells; c += 4 * stride) {   // (the bytes past a ragged end: not counted)
      const uint32_t v = *reinterpret_cast<const uint32_t*>(d.res + wp.cell_off + c);
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j)
        if (c + j < wp.cells) s += (v >> (8 * j)) & 0xFFu;
    }
  }
  wave_add_u64(s, &cnt[0]);
  wave_add_u64(sw, &cnt[1]);
  wave_add_u64(sb, &cnt[2]);
  __syncthreads();
  eco_stats* rec = &d.ring[(uint64_t)w * kStatsRing + (d.wv[w].step % kStatsRing)];
  uint64_t* to = threadIdx.x == 0 ? &rec->resource_total : (threadIdx.x == 1 ? &rec->water_total : &rec->biomass_total);
  if (threadIdx.x < 3 && cnt[threadIdx.x]) atomicAdd(reinterpret_cast<unsigned long long*>(to), cnt[threadIdx.x]);
}

// ---------------------------------------------------------------------------
// Init kernels
// ---------------------------------------------------------------------------
// Terrain height of local cell (x, y): bilinear blend, in exact integers with
// floor division, of the four surrounding values (0..31) of a torus lattice of
// NX x NY seeded values, NX = max(1, W / terrain_scale).
__device__ __forceinline__ int terrain_height(const WorldParams& wp, const eco_ecology& e, uint32_t x, uint32_t y) {
  const uint64_t W = wp.W, H = wp.H, L = (uint64_t)e.terrain_scale;
  const uint64_t NX = W / L > 0 ? W / L : 1, NY = H / L > 0 ? H / L : 1;
  const uint64_t ax = (uint64_t)x * NX, ay = (uint64_t)y * NY;
  const uint64_t i = ax / W, j = ay / H, fx = ax % W, fy = ay % H;
  const uint64_t i1 = (i + 1) % NX, j1 = (j + 1) % NY;
  const uint64_t v00 = draw32(wp, (uint32_t)(i + j * NX), 0u, ST_TERRAIN) >> 27;
  const uint64_t v10 = draw32(wp, (uint32_t)(i1 + j * NX), 0u, ST_TERRAIN) >> 27;
  const uint64_t v01 = draw32(wp, (uint32_t)(i + j1 * NX), 0u, ST_TERRAIN) >> 27;
  const uint64_t v11 = draw32(wp, (uint32_t)(i1 + j1 * NX), 0u, ST_TERRAIN) >> 27;
  const uint64_t num = v00 * (W - fx) * (H - fy) + v10 * fx * (H - fy) + v01 * (W - fx) * fy + v11 * fx * fy;
  return (int)(num / (W * H));
}

// floor(p * 2^32) clamped to [0, 2^32]: a 32-bit draw x is a Bernoulli(p) success iff x < it.
__device__ __forceinline__ uint64_t density_threshold(float p) {
  double t = floor((double)p * 4294967296.0);
  t = t < 0.0 ? 0.0 : (t > 4294967296.0 ? 4294967296.0 : t);
  return (uint64_t)t;
}

// Cell keys (for placement), initial resources, empty occupancy and claims.
__global__ __launch_bounds__(256) void k_init_cells(Dev d, const Tile* __restrict__ tiles) {
  const Tile tl = tiles[blockIdx.x];
  const WorldParams wp = d.wp[tl.world];
  for (uint32_t i = threadIdx.x; i < tl.count; i += blockDim.x) {
    const uint32_t c = tl.start + i, g = wp.cell_off + c;
    const uint32_t key = draw32(wp, c, 0u, ST_CELLKEY);
    d.cellkeys[g] = ((unsigned long long)key << 32) | c;
    d.res[g] = ((uint64_t)draw32(wp, c, 0u, ST_RESINIT) < wp.density_thr) ? 1 : 0;
    if (d.ep) {   // ecology: water, energy, biomass sites from outputs 1..3 of the same block
      const eco_ecology& e = d.ep[tl.world];
      const uint4 x = philox10(c, 0u, ST_RESINIT, 0u, wp.key0, wp.key1);
      d.res[g] = 0;
      d.cw[g] = ((uint64_t)x.y < density_threshold(e.water_density)) ? e.water_site : 0;
      d.ce[g] = ((uint64_t)x.z < density_threshold(e.energy_density)) ? e.energy_site : 0;
      d.cb[g] = ((uint64_t)x.w < density_threshold(e.biomass_density)) ? e.biomass_site : 0;
      if (d.rock) {   // terrain: the rock layer, and the sea instead of water sites
        const int r = terrain_height(wp, e, c % wp.W, c / wp.W);
        d.rock[g] = r;
        d.cw[g] = r < e.sea_level ? (e.sea_level - r) * e.water_per_depth : 0;
      }
    }
    d.occ[g] = -1;
    d.claim[g] = 0xFFFFFFFFu;
    if (wp.attack) d.mark[g] = 0;
    d.wall[g] = 0;
  }
}

// Placement (Sec. 3.2: the initial population on distinct cells; slot j takes
// the cell with the j-th smallest (Philox key, cell) pair).  The keys are 32-bit
// uniform draws, so a world's cells are bucketed by the top bits of the key into
// 2^k buckets of about four cells each (counts, a per-world exclusive scan, a
// scatter), and each cell's rank is its bucket's start plus the number of cells
// of its bucket with a smaller (key, cell) pair.  Only ranks below n_init are
// written.  Init only, never on the step path.
struct PlaceInfo {
  uint32_t boff;    // first bucket of the world in the bucket arrays
  uint32_t shift;   // bucket = key >> shift (2^(32 - shift) buckets)
};

__device__ __forceinline__ uint32_t place_bucket(const PlaceInfo& pi, unsigned long long k64) {
  return pi.boff + (pi.shift >= 32 ? 0u : (uint32_t)(k64 >> 32) >> pi.shift);
}

// Bucket counts (cnt zeroed by the caller).
__global__ __launch_bounds__(256) void k_place_count(Dev d, const Tile* __restrict__ tiles,
                                                     const PlaceInfo* __restrict__ pinfo, uint32_t* cnt) {
  const Tile tl = tiles[blockIdx.x];
  const WorldParams wp = d.wp[tl.world];
  const PlaceInfo pi = pinfo[tl.world];
  for (uint32_t i = threadIdx.x; i < tl.count; i += blockDim.x)
    atomicAdd(&cnt[place_bucket(pi, d.cellkeys[wp.cell_off + tl.start + i])], 1u);
}

// start[b] = exclusive prefix of the counts over the world's buckets (start of world
// w's buckets at boff + w, one extra entry per world holding its total), and the
// counts cleared for the scatter's cursors.  Blocks (tile, world) of 4,096 buckets:
// first each tile's sum (at boff / 4,096 + w + tile, apart for every world), then each
// tile from the sums before it.  (One block for a whole world took 600 us at 262,144
// buckets.)
constexpr uint32_t kPlaceTile = 4096;
__device__ __forceinline__ uint32_t place_sum_at(const PlaceInfo& pi, uint32_t w) { return pi.boff / kPlaceTile + w; }

__device__ __forceinline__ uint4 place_counts(const uint32_t* cnt, uint32_t b, uint32_t hi) {
  uint4 v = make_uint4(0, 0, 0, 0);
  if (b < hi) v.x = cnt[b];
  if (b + 1 < hi) v.y = cnt[b + 1];
  if (b + 2 < hi) v.z = cnt[b + 2];
  if (b + 3 < hi) v.w = cnt[b + 3];
  return v;
}

__global__ __launch_bounds__(kScanThreads) void k_place_sums(const PlaceInfo* __restrict__ pinfo, const uint32_t* cnt,
                                                             uint32_t* sums) {
  __shared__ unsigned long long red[kScanThreads / 64];
  const uint32_t w = blockIdx.y;
  const PlaceInfo pi = pinfo[w];
  const uint32_t nb = pinfo[w + 1].boff - pi.boff;
  if (blockIdx.x * kPlaceTile >= nb) return;
  const uint4 v = place_counts(cnt, pi.boff + blockIdx.x * kPlaceTile + 4 * threadIdx.x, pi.boff + nb);
  const unsigned long long t = block_sum_u64<kScanThreads>(v.x + v.y + v.z + v.w, red);
  if (threadIdx.x == 0) sums[place_sum_at(pi, w) + blockIdx.x] = (uint32_t)t;
}

__global__ __launch_bounds__(kScanThreads) void k_place_scan(const PlaceInfo* __restrict__ pinfo, uint32_t* cnt,
                                                             const uint32_t* __restrict__ sums, uint32_t* start) {
  __shared__ uint32_t red[kScanThreads / 64 + 1];
  const uint32_t w = blockIdx.y;
  const PlaceInfo pi = pinfo[w];
  const uint32_t nb = pinfo[w + 1].boff - pi.boff, hi = pi.boff + nb;
  if (blockIdx.x * kPlaceTile >= nb) return;
  const uint32_t b = pi.boff + blockIdx.x * kPlaceTile + 4 * threadIdx.x;
  const uint4 v = place_counts(cnt, b, hi);
  uint32_t before = 0, total;
  for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kScanThreads) before += sums[place_sum_at(pi, w) + t];
  block_exscan<kScanThreads>(before, red, &before);   // (its total: the earlier tiles' sum)
  uint32_t run = before + block_exscan<kScanThreads>(v.x + v.y + v.z + v.w, red, &total);
  const uint32_t c[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j)
    if (b + j < hi) {
      start[b + j + w] = run;
      run += c[j];
      cnt[b + j] = 0;
    }
  if (threadIdx.x == 0 && (blockIdx.x + 1) * kPlaceTile >= nb) start[hi + w] = before + total;
}

// Each cell into its bucket (unordered within the bucket) of sorted[].
__global__ __launch_bounds__(256) void k_place_scatter(Dev d, const Tile* __restrict__ tiles,
                                                       const PlaceInfo* __restrict__ pinfo, uint32_t* cnt,
                                                       const uint32_t* __restrict__ start) {
  const Tile tl = tiles[blockIdx.x];
  const WorldParams wp = d.wp[tl.world];
  const PlaceInfo pi = pinfo[tl.world];
  for (uint32_t i = threadIdx.x; i < tl.count; i += blockDim.x) {
    const unsigned long long k = d.cellkeys[wp.cell_off + tl.start + i];
    const uint32_t b = place_bucket(pi, k);
    d.sorted[wp.cell_off + start[b + tl.world] + atomicAdd(&cnt[b], 1u)] = k;
  }
}

// Rank of each bucketed cell; ranks below n_init go to cellkeys[cell_off + rank].
__global__ __launch_bounds__(256) void k_place_rank(Dev d, const Tile* __restrict__ tiles,
                                                    const PlaceInfo* __restrict__ pinfo,
                                                    const uint32_t* __restrict__ start) {
  const Tile tl = tiles[blockIdx.x];
  const WorldParams wp = d.wp[tl.world];
  const PlaceInfo pi = pinfo[tl.world];
  for (uint32_t i = threadIdx.x; i < tl.count; i += blockDim.x) {
    const unsigned long long k = d.sorted[wp.cell_off + tl.start + i];
    const uint32_t b = place_bucket(pi, k) + tl.world;
    const uint32_t s0 = start[b], s1 = start[b + 1];
    if (s0 >= wp.n_init) continue;   // the whole bucket ranks past the initial population
    uint32_t r = s0;
    for (uint32_t q = s0; q < s1; ++q) r += d.sorted[wp.cell_off + q] < k ? 1u : 0u;
    if (r < wp.n_init) d.cellkeys[wp.cell_off + r] = k;
  }
}

// Slot j < n_init takes the j-th smallest (key, cell); all other slots are free.
__global__ __launch_bounds__(kSlotTile) void k_init_agents(Dev d, Layout L, const Tile* __restrict__ tiles) {
  const Tile tl = tiles[blockIdx.x];
  const WorldParams wp = d.wp[tl.world];
  if (threadIdx.x >= tl.count) return;
  const uint32_t j = tl.start + threadIdx.x, g = wp.slot_off + j;
  d.tgt[g] = -1;
  d.act[g] = 0;
  d.sampled[g] = 255;
  if (j < wp.n_init) {
    const uint32_t cell = (uint32_t)(d.cellkeys[wp.cell_off + j] & 0xFFFFFFFFull);   // ranked by placement
    d.flags[g] = kAlive;
    d.pos[g] = (int)cell;
    d.occ[wp.cell_off + cell] = (int)j;
    d.facing[g] = (uint8_t)(draw32(wp, j, 0u, ST_FACING) >> 30);
    d.energy[g] = wp.e_init;
    d.age[g] = 0;
    if (d.ep) {
      d.water[g] = d.ep[tl.world].w_init;
      d.biomass[g] = d.ep[tl.world].b_init;
      d.hp[g] = d.ep[tl.world].hp_max;
    }
    d.uid[g] = j;
    d.puid[g] = ~0ull;
  } else {   // a free slot: no field is left as the allocation had it (a state read back is written as a whole)
    d.flags[g] = 0;
    d.trait[g] = 0.0;
    // of its weights, which nothing reads before they are written, the first 16 bytes: all
    // zero there, a read asks for the trait too
    const uint4 none = make_uint4(0, 0, 0, 0);
    *reinterpret_cast<uint4*>(d.store + (uint64_t)g * L.sstride) = none;
    *reinterpret_cast<uint4*>(d.master + (uint64_t)g * L.mstride) = none;
    d.pos[g] = 0;
    d.facing[g] = 0;
    d.energy[g] = 0;
    d.age[g] = 0;
    if (d.ep) d.water[g] = d.biomass[g] = d.hp[g] = 0;
    d.uid[g] = 0;
    d.puid[g] = 0;
  }
  if (j == 0) {
    WorldVar v{};
    v.uid_next = wp.n_init;
    d.wv[tl.world] = v;
  }
}

// Weights of n agents, one block per agent (persistent): of every world's initial
// agents in turn (list null), or of the list's (world, local slot) pairs; MODE W_INIT
// (with the colour trait) or W_REQUANT.  Bound by the arithmetic of the noise, as the
// births, whose writer it shares; nothing is cleared beforehand, since every byte that
// is read is written here or by a birth.  With that clearing and one unit per thread
// and turn, the row found by division and the quantised weights taken in a second
// pass, a reset of 65,536 agents (64 wide layers) took 9.4 ms in FP32 and 11.6 in
// BF16, now 3.7 and 4.2; FP8, 61,000 agents: 12.5, now 4.9.
struct InitArgs {
  Dev d;
  Layout L;
  const uint32_t* list;
  uint32_t n;
  double sd[3];
};
static_assert(offsetof(InitArgs, d) == offsetof(WeightArgs, d) && offsetof(InitArgs, L) == offsetof(WeightArgs, L),
              "write_weights reads these through WeightArgs");
template <int WDT, int H, int MODE>
__global__ __launch_bounds__(256) void k_init_weights(InitArgs by_value) {
  __shared__ uint32_t off[kMaxWorlds + 1];
  __shared__ uint32_t s_amax[128 + 128 + 16];
  __shared__ double s_red[4];
  __shared__ double2 tab[kNoiseTable];
  {
    const InitArgs& a = args<InitArgs>();
    if (!a.list && threadIdx.x < 64) {   // prefix of the worlds' initial populations
      const uint32_t n = a.d.n_worlds, per = (n + 63) / 64, lo = min(threadIdx.x * per, n), hi = min(lo + per, n);
      uint32_t own = 0;
      for (uint32_t i = lo; i < hi; ++i) own += a.d.wp[i].n_init;
      const uint32_t inc = wave_scan(own);
      uint32_t run = inc - own;
      for (uint32_t i = lo; i < hi; ++i) {
        off[i] = run;
        run += a.d.wp[i].n_init;
      }
      if (threadIdx.x == 63) off[n] = inc;
    }
    load_trig(a.d.trig, tab);
  }
  auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
  for (uint32_t e = blockIdx.x; e < args<InitArgs>().n; e += gridDim.x) {
    const InitArgs& a = args<InitArgs>();
    const Dev& d = a.d;
    const uint32_t w = uniform(a.list ? a.list[2 * e] : find_world(off, d.n_worlds, e));
    const uint32_t j = uniform(a.list ? a.list[2 * e + 1] : e - off[w]);
    const WorldParams& wp = d.wp[w];
    const uint32_t g = wp.slot_off + j;
    if (MODE == W_INIT && d.colour && threadIdx.x == 0) {   // colour trait: U[0,1) per channel
      const uint4 x = philox10(j, 0u, ST_COLOUR_INIT, 0u, wp.key0, wp.key1);
      d.colour[g] = make_float4((float)(x.x >> 8) * 0x1p-24f, (float)(x.y >> 8) * 0x1p-24f,
                                (float)(x.z >> 8) * 0x1p-24f, 0.0f);
    }
    const Noise nz{{a.sd[0], a.sd[1], a.sd[2]}, wp.key0, wp.key1, j, 0u};
    const double t = write_weights<WDT, H, 256, MODE>(g, g, nz, part_rows<H>(0u, 0u), tab, s_amax, s_red);
    if (threadIdx.x == 0) args<InitArgs>().d.trait[g] = t;
    __syncthreads();
  }
}

// Parity mode: mark every slot "not evaluated" before the policy kernel runs.
__global__ __launch_bounds__(256) void k_prestep_fill(Dev d) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.total_slots) return;
  d.sampled[i] = 255;
  if (d.keep_logits) {
    const float nan = __builtin_nanf("");
    for (uint32_t a = 0; a < d.lgs; ++a) d.logits[(uint64_t)i * d.lgs + a] = nan;
  }
}

// Host transfers of small pieces: one launch that reads or writes the pinned host
// buffer over PCIe instead of one staged copy (10 - 17 us) for each array.  A gather
// reads whole 16-byte units (device arrays end at a multiple of 64 elements), a
// scatter writes exactly the segment's bytes.  blockIdx.y: the segment.
__global__ __launch_bounds__(256) void k_segments_out(Segments g, uint4* host) {
  const Segment s = g.s[blockIdx.y];
  const uint32_t n = (s.bytes + 15u) / 16u;
  const uint4* src = reinterpret_cast<const uint4*>(s.dev);
  for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) host[s.at + i] = src[i];
}
__global__ __launch_bounds__(256) void k_segments_in(Segments g, const uint4* host) {
  const Segment s = g.s[blockIdx.y];
  const uint32_t n = s.bytes / 16u;
  uint4* dst = reinterpret_cast<uint4*>(s.dev);
  for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) dst[i] = host[s.at + i];
  const uint32_t tail = s.bytes & 15u;
  if (blockIdx.x == 0 && threadIdx.x < tail)
    reinterpret_cast<uint8_t*>(dst + n)[threadIdx.x] = reinterpret_cast<const uint8_t*>(host + s.at + n)[threadIdx.x];
}

// The last step's record of worlds 0, 1, ... (one block each) to host[w].
__global__ __launch_bounds__(64) void k_records_out(Dev d, eco_stats* host) {
  const uint32_t w = blockIdx.x;
  const uint64_t* src = reinterpret_cast<const uint64_t*>(d.ring + (uint64_t)w * kStatsRing + d.wv[w].step % kStatsRing);
  for (uint32_t i = threadIdx.x; i < sizeof(eco_stats) / 8; i += 64) reinterpret_cast<uint64_t*>(host + w)[i] = src[i];
}

// Streaming-read probe (measurement only): every 16-byte block of p read once,
// grid-stride, 8 non-temporal loads in flight per lane; the XOR of the data
// goes to *sink only if it equals a constant, so the loads cannot be dropped.
typedef unsigned int probe_u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(512) void k_stream_read(const probe_u32x4* __restrict__ p, uint64_t n, uint32_t* sink) {
  constexpr int U = 8;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t acc = 0;
  for (; i + (U - 1) * stride < n; i += U * stride) {
    probe_u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(p + i + u * stride);
#pragma unroll
    for (int u = 0; u < U; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (; i < n; i += stride) {
    const probe_u32x4 v = __builtin_nontemporal_load(p + i);
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  if (acc == 0x9E3779B9u) *sink = acc;
}

// ---------------------------------------------------------------------------
// Static scratch of the allocation-free step (eco_world_step_static): the tile
// partials, birth lists and statistics drafts of one object live in this array
// instead of the object's own buffers.  Each GPU the library runs on holds one
// copy until the process ends; every call on that GPU shares it.
// ---------------------------------------------------------------------------
constexpr size_t kStaticScratchBytes = (size_t(16) << 20) + ECO_MAX_WORLDS * sizeof(StepDraft) +
                                       ECO_MAX_PARTS * sizeof(double) + ECO_SMALL_CELL_TILES * kCellPart * sizeof(uint64_t);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// This GPU's address of the array (the array's name in host code is only a host
// stand-in): looked up once per device, with that device current, and kept.
hipError_t static_scratch(void** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex lock;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(lock);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Host-side launchers (used by eco_runtime.cpp)
// ---------------------------------------------------------------------------
#define ECO_CHECK_LAUNCH() return hipGetLastError()

hipError_t launch_move(hipStream_t s, const Dev& d, const TileScratch& ts, uint32_t H) {
  if (ts.n_slot_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_move, dim3(ts.n_slot_tiles + d.n_worlds), dim3(kSlotTile), 0, s, d, ts, H);
  ECO_CHECK_LAUNCH();
}
// After a call's last step.
hipError_t launch_settle(hipStream_t s, const Dev& d, const TileScratch& ts, uint32_t H, uint32_t small) {
  hipLaunchKernelGGL(k_settle, dim3(d.n_worlds), dim3(256), 0, s, d, ts, H, small);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || d.n_worlds == 1) return e;
  hipLaunchKernelGGL(k_settled, dim3((d.n_worlds + 255) / 256), dim3(256), 0, s, d);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_claim_cells(hipStream_t s, const Dev& d, const TileScratch& ts, uint32_t A) {
  const uint32_t nb = ts.n_slot_tiles + ts.n_cell_tiles;
  if (nb == 0) return hipSuccess;
  if (ts.cell_tile == ECO_SMALL_CELL_TILE) hipLaunchKernelGGL(k_claim_cells<1>, dim3(nb), dim3(256), 0, s, d, ts, A);
  else hipLaunchKernelGGL(k_claim_cells<4>, dim3(nb), dim3(256), 0, s, d, ts, A);
  ECO_CHECK_LAUNCH();
}
// Resident blocks per CU of the birth-commit kernel for this layout (its register
// and LDS use), so that the persistent grid is exactly one wave of resident blocks.
template <int WDT>
const void* birth_commit_fn(uint32_t H) {
  if (H == 32) return reinterpret_cast<const void*>(&k_birth_commit<WDT, 32>);
  if (H == 64) return reinterpret_cast<const void*>(&k_birth_commit<WDT, 64>);
  return reinterpret_cast<const void*>(&k_birth_commit<WDT, 128>);
}
hipError_t birth_commit_blocks_per_cu(const Layout& L, int* blocks) {
  const void* f = L.wdtype == 0 ? birth_commit_fn<0>(L.H1) : (L.wdtype == 1 ? birth_commit_fn<1>(L.H1)
                                                                              : birth_commit_fn<2>(L.H1));
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, f, 256, 0);
}

hipError_t launch_step_small(hipStream_t s, const Dev& d, const TileScratch& ts, uint32_t A, uint32_t H) {
  if (d.ep) hipLaunchKernelGGL(k_step_small<true>, dim3(2), dim3(1024), 0, s, d, ts, A, H);
  else hipLaunchKernelGGL(k_step_small<false>, dim3(2), dim3(1024), 0, s, d, ts, A, H);
  ECO_CHECK_LAUNCH();
}
// roles: 1 births, 2 live list, 4 records and water; 7 all in one launch, or one of them.
template <int WDT, int H>
void launch_birth_commit_wh(hipStream_t s, const Dev& d, const Layout& L, const TileScratch& ts, uint32_t births,
                            uint32_t ranked, int roles) {
  const uint32_t rest = ts.n_slot_tiles + d.n_worlds + (d.rock && !ranked ? ts.n_cell_tiles : 0u);
  const uint32_t base = (roles & 2) ? 0u : ((roles & 4) ? ts.n_slot_tiles : rest);
  const uint32_t end = (roles & 1) ? rest + births : ((roles & 4) ? rest : ts.n_slot_tiles);
  hipLaunchKernelGGL((k_birth_commit<WDT, H>), dim3(end - base), dim3(256), 0, s,
                     (CommitArgs{d, L, ts, base, rest, births, ranked}));
}
template <int WDT>
void launch_birth_commit_w(hipStream_t s, const Dev& d, const Layout& L, const TileScratch& ts, uint32_t births,
                           uint32_t ranked, int roles) {
  if (L.H1 == 32) launch_birth_commit_wh<WDT, 32>(s, d, L, ts, births, ranked, roles);
  else if (L.H1 == 64) launch_birth_commit_wh<WDT, 64>(s, d, L, ts, births, ranked, roles);
  else launch_birth_commit_wh<WDT, 128>(s, d, L, ts, births, ranked, roles);
}
hipError_t launch_birth_commit(hipStream_t s, const Dev& d, const Layout& L, const TileScratch& ts, uint32_t births,
                               uint32_t ranked, int roles) {
  if (L.H1 != L.H2 || (L.H1 != 32 && L.H1 != 64 && L.H1 != 128)) return hipErrorInvalidValue;
  if (L.wdtype == 0) launch_birth_commit_w<0>(s, d, L, ts, births, ranked, roles);
  else if (L.wdtype == 1) launch_birth_commit_w<1>(s, d, L, ts, births, ranked, roles);
  else launch_birth_commit_w<2>(s, d, L, ts, births, ranked, roles);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_compact(hipStream_t s, const Dev& d, const TileScratch& ts, int only_world) {
  hipLaunchKernelGGL(k_compact_count, dim3(ts.n_slot_tiles), dim3(kSlotTile), 0, s, d, ts, only_world);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_compact_write, dim3(ts.n_slot_tiles + ts.n_cell_tiles), dim3(kSlotTile), 0, s, d, ts,
                     only_world);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_stream_read(hipStream_t s, const void* p, uint64_t n16, uint32_t* sink, uint32_t blocks,
                              uint32_t threads) {
  hipLaunchKernelGGL(k_stream_read, dim3(blocks), dim3(threads), 0, s, reinterpret_cast<const probe_u32x4*>(p), n16,
                     sink);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_segments(hipStream_t s, const Segments& g, uint32_t n, uint32_t most, void* host, bool out) {
  const dim3 grid(std::min<uint32_t>(64u, std::max<uint32_t>(1u, (most + 4095u) / 4096u)), n);
  if (out) hipLaunchKernelGGL(k_segments_out, grid, dim3(256), 0, s, g, reinterpret_cast<uint4*>(host));
  else hipLaunchKernelGGL(k_segments_in, grid, dim3(256), 0, s, g, reinterpret_cast<const uint4*>(host));
  ECO_CHECK_LAUNCH();
}
hipError_t launch_records_out(hipStream_t s, const Dev& d, uint32_t n, void* host) {
  hipLaunchKernelGGL(k_records_out, dim3(n), dim3(64), 0, s, d, reinterpret_cast<eco_stats*>(host));
  ECO_CHECK_LAUNCH();
}
hipError_t launch_prestep_fill(hipStream_t s, const Dev& d) {
  hipLaunchKernelGGL(k_prestep_fill, dim3((d.total_slots + 255) / 256), dim3(256), 0, s, d);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_flowdir(hipStream_t s, const Dev& d, const TileScratch& ts, int world) {
  if (ts.n_cell_tiles == 0 || !d.rock) return hipSuccess;
  hipLaunchKernelGGL(k_flowdir, dim3(ts.n_cell_tiles), dim3(256), 0, s, d, ts.cell_tiles, world);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_render(hipStream_t s, const Dev& d, const TileScratch& ts, int world) {
  if (ts.n_cell_tiles == 0 || !d.rgb) return hipSuccess;
  hipLaunchKernelGGL(k_render, dim3(ts.n_cell_tiles), dim3(256), 0, s, d, ts.cell_tiles, world);
  ECO_CHECK_LAUNCH();
}
// most_cells: of one of the worlds.
hipError_t launch_resource_total(hipStream_t s, const Dev& d, int only_world, uint32_t most_cells) {
  const dim3 grid(std::min<uint32_t>(256u, (most_cells + 1023u) / 1024u), only_world < 0 ? d.n_worlds : 1u);
  hipLaunchKernelGGL(k_resource_total, grid, dim3(256), 0, s, d, only_world < 0 ? 0u : (uint32_t)only_world);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_init_cells(hipStream_t s, const Dev& d, const Tile* tiles, uint32_t nt) {
  if (nt == 0) return hipSuccess;
  hipLaunchKernelGGL(k_init_cells, dim3(nt), dim3(256), 0, s, d, tiles);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_placement(hipStream_t s, const Dev& d, const Tile* cell_tiles, uint32_t nt, const void* pinfo,
                            uint32_t* cnt, uint32_t* sums, uint32_t* start, uint32_t most_buckets) {
  if (nt == 0) return hipSuccess;
  const PlaceInfo* pi = reinterpret_cast<const PlaceInfo*>(pinfo);
  hipLaunchKernelGGL(k_place_count, dim3(nt), dim3(256), 0, s, d, cell_tiles, pi, cnt);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 tiles((most_buckets + kPlaceTile - 1) / kPlaceTile, d.n_worlds);
  hipLaunchKernelGGL(k_place_sums, tiles, dim3(kScanThreads), 0, s, pi, cnt, sums);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_place_scan, tiles, dim3(kScanThreads), 0, s, pi, cnt, sums, start);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_place_scatter, dim3(nt), dim3(256), 0, s, d, cell_tiles, pi, cnt, start);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_place_rank, dim3(nt), dim3(256), 0, s, d, cell_tiles, pi, start);
  ECO_CHECK_LAUNCH();
}
hipError_t launch_init_agents(hipStream_t s, const Dev& d, const Layout& L, const Tile* tiles, uint32_t nt) {
  if (nt == 0) return hipSuccess;
  hipLaunchKernelGGL(k_init_agents, dim3(nt), dim3(kSlotTile), 0, s, d, L, tiles);
  ECO_CHECK_LAUNCH();
}
template <int WDT, int H>
hipError_t launch_init_weights_wh(hipStream_t s, const InitArgs& a, uint32_t n_cus, bool requant) {
  int per_cu = 1;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, reinterpret_cast<const void*>(&k_init_weights<WDT, H, W_INIT>), 256, 0);
  if (e != hipSuccess) return e;
  const dim3 grid(std::min<uint32_t>(a.n, n_cus * (uint32_t)std::max(1, per_cu)));
  if (requant) hipLaunchKernelGGL((k_init_weights<WDT, H, W_REQUANT>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_init_weights<WDT, H, W_INIT>), grid, dim3(256), 0, s, a);
  ECO_CHECK_LAUNCH();
}
// Initial (or, requant, re-quantised) weights of n agents: the list's, or without one
// every world's initial agents.
hipError_t launch_init_weights(hipStream_t s, const Dev& d, const Layout& L, const uint32_t* list, uint32_t n,
                               bool requant, double std1, double std2, double std3, uint32_t n_cus) {
  if (n == 0) return hipSuccess;
  if (L.H1 != L.H2 || (L.H1 != 32 && L.H1 != 64 && L.H1 != 128)) return hipErrorInvalidValue;
  const InitArgs a{d, L, list, n, {std1, std2, std3}};
#define ECO_INIT(WW)                                                              \
  if (L.H1 == 32) return launch_init_weights_wh<WW, 32>(s, a, n_cus, requant);    \
  else if (L.H1 == 64) return launch_init_weights_wh<WW, 64>(s, a, n_cus, requant); \
  else return launch_init_weights_wh<WW, 128>(s, a, n_cus, requant);
  if (L.wdtype == 0) { ECO_INIT(0) }
  if (L.wdtype == 1) { ECO_INIT(1) }
  ECO_INIT(2)
#undef ECO_INIT
}

}  // namespace eco
