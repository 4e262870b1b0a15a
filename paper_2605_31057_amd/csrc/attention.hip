// attention.hip -- block-sparse and dense flash-attention forward for gfx950.
//
// Computes Eq. 2 of the LVSA paper (softmax attention restricted to a key
// set) with the key set of every query block given by a block CSR, and Eq. 1
// (all keys) with the same kernel visiting every key block.
//
// Work decomposition
//   A whole tile is 256 query rows of one head (two query blocks at BLOCK =
//   128, four at 64), eight waves of 32 rows each.  The workgroup walks the
//   union of the query blocks' key lists, 128 keys per step (one key block, or
//   two of 64), and every wave takes all keys of the step for its rows.
//   Adjacent query blocks mostly keep the same key blocks (they touch the same
//   frames), so each K/V tile brought from HBM/L2 into LDS serves 256 query
//   rows; a key block that only some of the query blocks keep is masked out
//   (no valid keys, V left out of the products) for the waves of the others.
//   Where whole tiles leave compute units idle (few tiles, or a last round that
//   is nearly empty), tiles are split over the key groups of a workgroup
//   (Split): 128 or 64 rows, the eight waves sharing the step's keys as well as
//   the rows, partial results combined in LDS at the end (combine_groups).  The
//   host plans which tiles run how (make_plan).
//   One persistent workgroup per compute unit takes items through atomic
//   counters (fetch_item); a launch with a workgroup for every item has no
//   counters.  A whole tile of four query blocks whose rows have little in common
//   is worked in its parts by the workgroup that took it (attn_tile).
//
// The merged walk
//   A tile's key blocks are the union of its query blocks' CSR rows, walked in
//   descending order, each key block once with a flag per query block.  At
//   the start of the tile the workgroup merges two rows in LDS (merge_pair):
//   every entry's position in the union is its index in its own row plus the
//   entries of the other row above it (a binary search) minus the entries
//   above it that both rows hold (a ballot count), and the step words are
//   written there; four rows are merged through bitmaps (merge_four), a tile
//   within one query block takes its row as it is (single_row).  The step loop
//   then reads its words three steps ahead (K tiles are loaded two steps
//   ahead).  The sparse modes take at most WALK_CAP key blocks (checked before
//   launch), so one merge covers any tile.  Dense attention up to WALK_CAP key
//   blocks runs the block mode with no CSR: the words are written directly
//   instead of merged.  The mask is only read, so any number of launches can
//   share it.
//
// Schedule ("ping-pong", 128 keys per step)
//   Waves w and w + 4 (which share a SIMD) run half a step apart: while one is
//   in its GEMM phase (O += P(j) V(j), S(j+1) = K(j+1) Q^T: MFMA with fragments
//   from LDS) the other is in its softmax phase (exponentials, P in bf16:
//   VALU), so the matrix core and the VALU of each SIMD are busy at the same
//   time.  A barrier ends every half step.  LDS holds two K stages and two V
//   stages (slab layout, see below); K(j+2) and V(j+1) stream from HBM/L2 into
//   the stages freed by step j-1 with buffer loads that write LDS directly,
//   issued by every wave in its softmax phase (in split tiles all in the step's
//   first half, StepLoads) and waited for at the end of the step.  The buffer
//   resource's size bound turns rows at or past N (ragged last block) into
//   zeros.
//   A whole key block per step keeps the per-step costs (two barriers, the
//   loop, the load set-up) small against the step's 136 MFMAs per wave; S
//   (64 registers) and P (32) then fill the register file, so the GEMM
//   phase finishes P(j) before it produces S(j+1), and masks run only in a
//   wave-uniform branch.
//
// Contractions (bf16 MFMA 16x16x32, fp32 accumulate)
//     S^T = K Q^T     A = K rows (LDS, ds_read_b128), B = Q rows (registers)
//     O^T += V^T P^T  A = V^T (LDS, ds_read_b64_tr_b16), B = P (registers)
//   The transposed products put a query row's scores in four lanes (l, l^16,
//   l^32, l^48), and P never leaves registers.
//   MFMA 16x16x32 lane layout (lane l, group g = l/16, i = l%16): A row i and B
//   column i carry k-slots 8g..8g+7; C register r holds row 4g + r, column i.
//   k-slot order only has to agree between A and B, so the keys held by S^T's
//   C registers of two 16-key tiles are paired with the V^T elements of those
//   keys (v_frag).
//   A wave's 32 query rows are two tiles of 16, and each K or V fragment is used
//   for both.
//
// What bounds it
//   Board power, then the VALU's issue slots.  The launch draws the board's
//   limit and the clock drops (2.4 GHz peak; 1.55 GHz with 32x32x16 MFMAs,
//   1.9 GHz with 16x16x32), so energy per step is time: a stream of 16x16x32
//   MFMAs on random data, four in a row into one accumulator, reaches 2.19
//   PFLOP/s at the limit, alternating accumulators 2.06, 32x32x16 1.75-1.84.
//   In cycles, an MFMA issue blocks the VALU for about 8 (an fma takes 8.3
//   cycles beside 16x16x32 MFMAs, 4.5 alone; an exponential 16.4 and 8.5), so
//   the softmax phase (112 VALU instructions and 64 exponentials a step beside
//   136 MFMAs, and 8 tile loads of about 67 cycles) takes 2,700 cycles, and the
//   GEMM phase (136 MFMAs of 16 cycles, 96 LDS reads of about 2.3) 2,600.
//   Wan-1.3B 6x, 12 heads, step 10: 31.4 ms with 32x32x16 MFMAs and a row
//   maximum per step, 28.3 ms now (1.42 PFLOP/s; a large bf16 matrix product
//   reaches 1.59), all on one board.
//
// Online softmax (fp32, base 2): p = exp2(s*log2(e)/sqrt(d) - m), l = sum p,
// with a reference m per row that is raised, and O and l rescaled, only when
// some p reaches 2 (softmax_phase); the result is exact either way because O
// and l always use the same m.
#include <atomic>

#include "internal.h"

namespace lvsa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int D = 128;             // head_dim
// Distance (log2) of a row's reference above the largest score it was set from,
// before and after the wave's first redo of a step, and the redos after which a
// wave takes the row maximum ahead of every step (softmax_phase).
constexpr float HEADROOM = 7.f;
constexpr float WIDE_HEADROOM = 39.f;
constexpr int MAX_REDOS = 12;

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base,
                                                            uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0,
                                           bytes, 0x00020000);
}

// Largest of x0 (and of x1) over the four lanes that hold one query row (l,
// l^16, l^32, l^48); every lane gets both results.  With 16-lane groups
// [0 1 2 3], permlane16_swap(a, b) gives [a0 b0 a2 b2] and [a1 b1 a3 b3], and
// permlane32_swap(a, b) gives [a0 a1 b0 b1] and [a2 a3 b2 b3].
__device__ __forceinline__ void row_max(float& x0, float& x1) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x0), __float_as_uint(x1),
                                                  false, false);
  const float y = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));   // x0 x1 x0 x1
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false,
                                                  false);
  const float z = fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
  const auto u = __builtin_amdgcn_permlane16_swap(__float_as_uint(z), __float_as_uint(z), false,
                                                  false);
  x0 = __uint_as_float(u[0]);
  x1 = __uint_as_float(u[1]);
}

// LDS tile layout ("slabs").  A BLOCK x 128 tile (one key block) is stored
// as 4 slabs of 32 columns; a slab row is 64 bytes (4 chunks of 16 bytes) and
// rows follow each other, so tile byte (slab, row, chunk) =
// slab*BLOCK*64 + row*64 + chunk*16.
// The chunk is XORed with x(row) = -(row/4) mod 4.  With 64 banks of 4 bytes:
//   - ds_read_b128 is served 16 lanes at a time, lanes 0-3, 12-15 and 20-27
//     together (then 4-11, 16-19 and 28-31; the same from lane 32 on): rows
//     0-3 and 12-15 at one logical chunk c and rows 4-11 at c ^ 1, which x
//     sends to four different bank quarters;
//   - ds_read_b64_tr_b16 (served 32 lanes at a time) reads 8 consecutive rows
//     x 2 chunks of a 32-byte half: rows 4..7 take the other half's banks.
// Both are free of bank conflicts, and every fragment address an unrolled loop
// needs is one of three per-lane bases plus an immediate offset.
constexpr int SLAB_ROW = 64;
__device__ __forceinline__ int xsw(int row) { return -(row >> 2) & 3; }

struct Tile {
  static constexpr int NW = 8;                      // waves
  static constexpr int NT = NW * 64;                // threads
  static constexpr int KEYS = 128;                  // keys per step
  static constexpr int SLAB = KEYS * SLAB_ROW;      // bytes per slab
  static constexpr int BYTES = 4 * SLAB;            // bytes per K or V tile
  static constexpr int LOADS = BYTES / 1024 / NW;   // 1 KiB wave loads per wave and tile
};

// How the eight waves share a tile: KG key groups of 8 / KG waves.  A wave
// holds 32 query rows of the tile's ROWS and takes NK of the step's 128 keys
// (key group kg: keys kg*NK .. kg*NK + NK - 1).  With KG > 1 several waves
// hold the same rows, each over its own share of the keys, and their partial
// results are combined at the end of the tile (combine_groups).
template <int KG>
struct Split {
  static constexpr int ROWS = 256 / KG;             // query rows per tile
  static constexpr int NRG = 8 / KG;                // waves per key group
  static constexpr int NK = Tile::KEYS / KG;        // keys per wave and step
  static constexpr int NU = NK / 32;                // 32-key groups per wave and step
};

// One wave load (1 KiB) of a K or V tile into LDS at byte address lds_dst:
// `rsrc` starts at the tile's first row, `voff` = the lane's part of the
// global byte offset plus the load's uniform part (LoadPlan).  Rows at or
// past N fall outside the buffer resource and read as zeros.  The loads are
// issued from inline assembly so the compiler does not track them: they are
// waited for explicitly (vmcnt(0) plus a barrier) at the end of the step, and
// no compiler-inserted wait can stall the phases in between.  The nop is the
// wait state gfx9 needs between an SALU write of M0 and an LDS-DMA
// instruction (the compiler cannot see into the statement to add it).
__device__ __forceinline__ void issue_load(uint32_t lds_dst, __amdgpu_buffer_rsrc_t rsrc,
                                           uint32_t voff, uint32_t soff) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %1, %2, %3 offen lds"
      :
      : "s"(lds_dst), "v"(voff), "s"(rsrc), "s"(soff)
      : "memory", "m0");
}

// Buffer resource over rows kb*BLOCK .. N-1 of one head of K or V; a key
// block index outside [0, nb) yields an empty resource (all loads read 0).
template <int BLOCK>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const __bf16* head_base,
                                                            int64_t row_elems,
                                                            uint32_t head_bytes,
                                                            int kb, int nb) {
  const bool ok = (uint32_t)kb < (uint32_t)nb;
  const int64_t skip = ok ? (int64_t)kb * BLOCK * row_elems : 0;
  const uint32_t bytes = ok ? head_bytes - (uint32_t)(skip * 2) : 0u;
  return make_rsrc(head_base + skip, bytes);
}

// Per-wave load plan: wave w's load j of a tile fills tile bytes
// 1024*(w + NW*j): slab j, rows 16*w + lane/4, physical chunk lane%4, which
// holds logical chunk (lane%4) ^ x(row).  Global
// offset: lane_off plus 64*j; LDS offset: lds_w plus 1024*NW*j.  With BLOCK =
// 64 a step's tile is two key blocks, rows 0..63 and 64..127, and the
// resource that waves 4..7 load through starts at the second one.
struct LoadPlan {
  uint32_t lane_off;   // (16*(w % (BLOCK/16)) + lane/4)*row_bytes + 16*((lane%4) ^ x(lane/4))
  uint32_t lds_w;      // 1024*w (uniform)
};

template <int BLOCK>
__device__ __forceinline__ LoadPlan load_plan(uint32_t row_bytes, int wave, int lane) {
  LoadPlan lp;
  lp.lane_off = (uint32_t)(16 * (wave % (BLOCK / 16)) + lane / 4) * row_bytes +
                16u * (uint32_t)((lane % 4) ^ xsw(lane / 4));
  lp.lds_w = (uint32_t)__builtin_amdgcn_readfirstlane(1024u * (uint32_t)wave);
  return lp;
}

__device__ __forceinline__ void issue_tile(uint32_t lds, __amdgpu_buffer_rsrc_t rsrc,
                                           const LoadPlan& lp) {
#pragma unroll
  for (int j = 0; j < Tile::LOADS; ++j)
    issue_load(lds + lp.lds_w + 1024u * Tile::NW * j, rsrc, lp.lane_off, 64u * j);
}

// The loads of one pipeline step: the next K tile and the next V tile.  A tile
// load costs its wave 40 to 70 cycles (the four waves of a half step share the
// CU's 64 bytes a cycle).  Whole tiles (KG = 1): every wave issues its share at the
// start of its softmax phase, which has the slack; the leaders' is the step's
// second half, so their loads have that phase to arrive before the step ends.
// Split tiles (KG > 1): a step's computation is a half or a quarter, its loads are
// the same, and what bounds it is their issue and arrival.  All waves issue
// them in the step's first half, spread over the phase they are in: the
// leaders' GEMM phase and the others' softmax phase.  In 64-row items, per
// step: 1.23 us with the leaders' loads at the start of their softmax phase,
// 1.16 this way (one head of 15,600 tokens: 149.7 and 141.9 us; 4,680 tokens:
// 46.8 and 44.4; 128-row items, one head of 32,760 tokens token-exact: 447.6 and
// 437.7; interleaved on one board).  Every wave's in its softmax phase with a
// whole step to arrive, the key halves of leaders and others loaded apart, was
// slower (1% to 8%): arrival alone is not the bound, bursts are.
// Near the end of a row the key-block indices repeat the last block and the loads
// land in slots no later step reads (in the last step the leaders of whole tiles
// issue none).
struct StepLoads {
  uint32_t k_dst, v_dst;                 // LDS tile addresses
  __amdgpu_buffer_rsrc_t rk, rv;         // resources starting at the tiles
  LoadPlan kp, vp;
};

__device__ __forceinline__ void issue_step_load(const StepLoads& sl, int i) {
  if (i < Tile::LOADS)
    issue_load(sl.k_dst + sl.kp.lds_w + 1024u * Tile::NW * i, sl.rk, sl.kp.lane_off, 64u * i);
  else
    issue_load(sl.v_dst + sl.vp.lds_w + 1024u * Tile::NW * (i - Tile::LOADS), sl.rv,
               sl.vp.lane_off, 64u * (i - Tile::LOADS));
}

__device__ __forceinline__ void issue_step_loads(const StepLoads& sl) {
#pragma unroll
  for (int i = 0; i < 2 * Tile::LOADS; ++i) issue_step_load(sl, i);
}

__device__ __forceinline__ void wait_loads_and_sync() {
  __builtin_amdgcn_s_waitcnt(0);  // vmcnt(0) expcnt(0) lgkmcnt(0)
  __syncthreads();
}

// Time of a part of 256 / KG rows, in percent of a whole tile's (256 rows) of the same
// walk (make_plan).
constexpr int PART_TIME[] = {0, 100, 60, 0, 42};
// What the parts of a tile take more in fixed times than the tile whole, in words of
// its walk (64 keys): a whole tile's fixed time is that of 2.5 steps of 128 keys, a part's
// 2.2 (64 rows) to 3.8 (128 rows), by the same measurements.
constexpr int PARTS_FIXED = 12;

// Scores of the wave's 32 query rows (two tiles of 16) against its keys, 16
// keys per tile: lane l holds query rows l%16 of both tiles and keys
// 16*kt + 4*(l/16) + r.
template <int NU>
struct Scores {
  f32x4 s[2 * NU][2];   // [key tile][query tile]
};

// Per-lane LDS byte offsets (within a tile) of the K and V fragments.
struct FragAddr {
  uint32_t k;               // K row of this lane
  uint32_t v_even, v_odd;   // V row, d tiles 2t / 2t+1 (transposing read)
};

// `key0`: the first key of the wave's share of the step.
__device__ __forceinline__ FragAddr frag_addr(int lane, int key0) {
  const int g = lane / 16, sl = lane % 16;
  FragAddr f;
  // K: row 16*kt + sl, d = 32*stp + 8*g: slab stp, logical chunk g.
  f.k = (key0 + sl) * SLAB_ROW + ((g ^ xsw(sl)) * 16);
  // V: the transposing read gives lane (group g = lane/16, j = lane%16)
  // element e of the group's chunk 4e + j/4, entry j%4.  Source lane
  // sl = 4e + q points at V row (key 4g + e) and columns 4q .. 4q+3 of the 16
  // of the d tile (slab dt/2, logical chunk 2*(dt%2) + q/2, byte half q%2).
  const int vrow = 4 * g + sl / 4;
  f.v_even = (key0 + vrow) * SLAB_ROW + ((((sl % 4) / 2) ^ xsw(vrow)) * 16) + (sl % 2) * 8;
  f.v_odd = f.v_even ^ 32u;
  return f;
}

// K fragment (16 keys x 32 d) and V^T fragment (16 d x 32 keys).  k-slot e < 4
// of lane group g is key 4g + e of the first 16, e >= 4 the same of the second
// 16: the order in which P's lanes hold their keys.
__device__ __forceinline__ bf16x8 k_frag(const char* lds_k, const FragAddr& fa, int kt, int stp) {
  return *(const bf16x8*)(lds_k + fa.k + stp * Tile::SLAB + kt * 16 * SLAB_ROW);
}
__device__ __forceinline__ i16x4 v_half(const char* lds_v, const FragAddr& fa, int dt, int u,
                                        int half) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (lds_i16x4*)(lds_v + ((dt & 1) ? fa.v_odd : fa.v_even) + (dt / 2) * Tile::SLAB +
                   (u * 32 + half * 16) * SLAB_ROW));
}
__device__ __forceinline__ bf16x8 join(i16x4 lo, i16x4 hi) {
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ bf16x8 v_frag(const char* lds_v, const FragAddr& fa, int dt, int u) {
  return join(v_half(lds_v, fa, dt, u, 0), v_half(lds_v, fa, dt, u, 1));
}

// S^T = K Q^T for the wave's keys of one step (K tile at lds_k).
template <int NU>
__device__ __forceinline__ void compute_scores(const char* lds_k, const bf16x8 (&qf)[4][2],
                                               Scores<NU>& sc, const FragAddr& fa) {
#pragma unroll
  for (int kt = 0; kt < 2 * NU; ++kt) {
    f32x4 acc[2] = {f32x4{}, f32x4{}};
#pragma unroll
    for (int stp = 0; stp < 4; ++stp) {
      const bf16x8 a = k_frag(lds_k, fa, kt, stp);
#pragma unroll
      for (int qt = 0; qt < 2; ++qt)
        acc[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[stp][qt], acc[qt], 0, 0, 0);
    }
    sc.s[kt][0] = acc[0];
    sc.s[kt][1] = acc[1];
  }
}

// Row sums l are taken on the matrix core, as a 16x16 MFMA accumulator that the
// GEMM phase adds each step's bf16 P into (register 0 of every lane holds its
// row's sum): 8 MFMAs a step instead of 64 adds in the softmax phase, whose VALU
// slots are the scarcer (fp32 sums on the VALU: Wan-1.3B 6x step 29.7 ms against
// 28.5; split tiles 3% slower, one head of 32,760 tokens 437 us against 419).
// They sum exactly the P that multiplies V, so the weights of a row add up to 1
// and P's rounding largely cancels: with d_i the relative rounding of p_i the
// result is off by sum d_i p_i (v_i - o) / l instead of sum d_i p_i v_i / l.
// Measured, 2-norm of the error against float64 relative to the result, fp32 sums
// (against the running maximum) and these: N(0, 1) inputs, 22 shapes in all forms,
// 2.29e-3 to 2.36e-3 and 2.25e-3 to 2.36e-3, not larger in any but one (token-exact,
// 4 heads, by 0.1%, in split tiles while those still summed on the VALU); with Q and
// K times 1, 2, 4, 8, 16, one head of 4,680 tokens, split tiles, 2.36e-3, 2.07e-3,
// 1.77e-3, 1.07e-3, 0.56e-3 and 2.36e-3, 1.82e-3, 1.51e-3, 0.93e-3, 0.49e-3, and 12
// heads of 5,460 tokens, whole tiles, 2.33e-3, 2.06e-3, 1.75e-3, 1.07e-3, 0.56e-3 and
// 2.33e-3, 1.88e-3, 1.54e-3, 0.94e-3, 0.49e-3.
constexpr int READY = 1, WIDE = 2, REDO = 4;
struct WaveState {
  f32x4 o[8][2];   // O^T tiles [d tile][query tile]: d = 16*dt + C row
  float m[2];      // reference of the exponentials (log2 domain), the same in a row's four lanes
  f32x4 l[2];      // row sums
  int flags;       // READY: every row has a finite m; WIDE: a step was redone; EAGER: REDO
                   // times the steps redone
};

// Keys at or past N (ragged last block) do not exist: their scores become
// -inf.  `valid` = N - the wave's first key (at most 0: no key is valid).  Per
// score one compare of a constant into VCC and one select, a scheduling
// barrier every 4 scores so that few compare results are live at once.
// For the 16-key tiles KT0 .. KT0 + KTN - 1, whose first key `valid` counts from.
template <int NU, int KT0 = 0, int KTN = 2 * NU>
__device__ __forceinline__ void mask_tail(Scores<NU>& sc, int lane, int valid) {
  if (valid < 16 * KTN) {
    const int lim = valid - 4 * (lane / 16);   // key 4*(lane/16) + c is valid iff c < lim
#pragma unroll
    for (int kt = 0; kt < KTN; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (r % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        const bool ok = 16 * kt + r < lim;
        sc.s[KT0 + kt][0][r] = ok ? sc.s[KT0 + kt][0][r] : -__builtin_inff();
        sc.s[KT0 + kt][1][r] = ok ? sc.s[KT0 + kt][1][r] : -__builtin_inff();
      }
  }
}

// Token-exact form: the 4-bit pattern of the wave's query block for this key
// block says which query-frame / key-frame parts are attended (bit 2a+b, a =
// the lane's query row lies in the query block's second frame, b = the key
// lies in the key block's second frame, which starts kfirst keys in; 0 = the
// query block does not keep the key block).  A row's kept keys are then one
// range [klo, khi) of the block, also clipped at `valid` = N minus the
// block's first key.  Scores outside the range become -inf.  Blocks whose
// every part is attended and that are not ragged skip the masking.
//
// Key kbase + c is kept iff the unsigned c + kbase - klo is below the range's
// width: per score one add of a constant, one compare into VCC and one
// select.  A scheduling barrier every 4 scores keeps the compiler from
// computing many compare results ahead (each holds an SGPR pair).
//
// The lane's query row lies in the second frame iff its row index within the
// wave's 32 rows reaches `sec_from` (wave-uniform); the lane index is
// recomputed here rather than held in a register through the loop.  `koff`
// is the wave's first key within the key block.
template <int BLOCK, int NU>
__device__ __forceinline__ void mask_exact(Scores<NU>& sc, uint32_t pat, int kfirst,
                                           int valid, int sec_from, int koff) {
  if (pat != 0xFu || valid < BLOCK) {
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      const uint32_t bits = 16 * qt + lane % 16 >= sec_from ? pat >> 2 : pat;
      const int klo = (bits & 1u) ? 0 : kfirst;
      const int khi = (bits & 2u) ? valid : min(kfirst, valid);
      const uint32_t shift = (uint32_t)(koff + 4 * (lane / 16) - klo);
      const uint32_t width = (uint32_t)max(khi - klo, 0);
#pragma unroll
      for (int kt = 0; kt < 2 * NU; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (r == 0) __builtin_amdgcn_sched_barrier(0);
          const uint32_t c = (uint32_t)(16 * kt + r);
          sc.s[kt][qt][r] = c + shift < width ? sc.s[kt][qt][r] : -__builtin_inff();
        }
    }
  }
}

// Probabilities in bf16: the B operands of the P V product.
template <int NU>
struct Probs {
  bf16x8 p[NU][2];   // [32-key group][query tile]
};

// Raises the reference m of every row whose largest score of the step lies
// above it, to `head` above that score, the others by `lift`, and rescales the rows'
// O and l.  FIRST: ahead of the step's probabilities, not because some are too large.
// EAGER: see softmax_phase.
template <int NU, bool FIRST, bool EAGER>
__device__ __forceinline__ void raise_max(const Scores<NU>& sc, WaveState& st,
                                          float scale_log2, float head, float lift) {
  float mx[2];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    mx[qt] = -__builtin_inff();
#pragma unroll
    for (int kt = 0; kt < 2 * NU; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx[qt] = fmaxf(mx[qt], sc.s[kt][qt][r]);
  }
  row_max(mx[0], mx[1]);
  if (!(FIRST && EAGER) ||
      __builtin_amdgcn_ballot_w64(mx[0] * scale_log2 > st.m[0] || mx[1] * scale_log2 > st.m[1])) {
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      const float top = mx[qt] * scale_log2;
      const float m = top > st.m[qt] ? top + head : st.m[qt] + lift;
      const float a = m == st.m[qt] ? 1.f : __builtin_amdgcn_exp2f(st.m[qt] - m);
      st.m[qt] = m;
      st.l[qt][0] *= a;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) st.o[dt][qt] *= a;
    }
  }
  const bool ready = __builtin_amdgcn_ballot_w64(st.m[0] == -__builtin_inff() ||
                                                 st.m[1] == -__builtin_inff()) == 0;
  st.flags = (st.flags & ~READY) |
             (ready && (!EAGER || st.flags < MAX_REDOS * REDO) ? READY : 0);
}

// P = 2^(s*scale - m) in bf16 from one step's scores, with the tile loads in `sl`
// issued along the way (LOADS).
// Returns the bits of all probabilities or-ed together.  Scheduling barriers
// every 8 scores keep the compiler from hoisting many exponentials at once
// (S, P, O and Q already fill the register file).
template <int NU, bool LOADS>
__device__ __forceinline__ uint32_t probabilities(const Scores<NU>& sc, Probs<NU>& pr,
                                                  const float (&m)[2], float scale_log2,
                                                  const StepLoads& sl) {
  constexpr int NLOADS = 2 * Tile::LOADS;
  constexpr int GROUPS = 4 * NU;                     // groups of 4 scores
  constexpr int PER = (NLOADS + GROUPS - 1) / GROUPS;
  constexpr int EVERY = GROUPS > NLOADS ? GROUPS / NLOADS : 1;
  int issued = 0;
  uint32_t bits = 0u;
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int grp = 4 * u + 2 * qt + t;
        if (t == 0) __builtin_amdgcn_sched_barrier(0);
        if (LOADS && grp % EVERY == 0)
          for (int i = 0; i < PER && issued < NLOADS; ++i) issue_step_load(sl, issued++);
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          const float a = __builtin_amdgcn_exp2f(
              __builtin_fmaf(sc.s[2 * u + t][qt][r], scale_log2, -m[qt]));
          const float b = __builtin_amdgcn_exp2f(
              __builtin_fmaf(sc.s[2 * u + t][qt][r + 1], scale_log2, -m[qt]));
          const bf16x2 pk = {(__bf16)a, (__bf16)b};
          bits |= __builtin_bit_cast(uint32_t, pk);
          pr.p[u][qt][4 * t + r] = pk[0];
          pr.p[u][qt][4 * t + r + 1] = pk[1];
        }
      }
  if (LOADS)
    for (; issued < NLOADS; ++issued) issue_step_load(sl, issued);
  return bits;
}

// Softmax phase of the ping-pong schedule: block j's scores (in `sc`) become
// its probabilities P (bf16, in `pr`), against the rows' reference m as it
// stands.  m is some headroom above the largest score it was set from, so p stays
// far below 2 until a score exceeds that one by the headroom + 1; then some p
// (rounded to bf16) is at least 2, which sets the top exponent bit of its half
// of the word (inf and NaN do too), and the wave raises m and does the step's
// probabilities again.  So a step usually takes no row maximum: one or3 per
// four scores instead of one max3 per two and the exchange between a row's
// lanes.  The result is exact either way because O and l always use the same
// m.  Until every row has an m (READY), m is raised first.
//
// The headroom is 7 at first: the result is then as precise as against the running
// maximum for V of any scale (measured down to 2^-120, where bf16 itself runs out).
// Logits so wide that a step is redone would cross it again and again (one redoing
// wave holds up the other seven at the half step's barrier), so a wave's first redo
// takes 39 from then on; products p v then lose bits for v below 2^-100 (measured,
// Q and K times 8: error 0.94e-3 down to 2^-95, 0.95e-3 at 2^-100, 7.8e-3 at 2^-105).
// Wan-1.3B 6x step with Q and K times 1, 2, 4, 8, ms, interleaved on one board: 27.8,
// 29.9, 31.0 and 30.0 with 7 throughout, 27.7, 28.5, 28.6 and 28.5 so (with a row
// maximum every step and 32x32x16 MFMAs 30.4, 31.8, 32.0 and 28.9).  Times 16 and
// more, where one key holds all of a row's weight, steps are redone even so: with
// EAGER a wave that has redone MAX_REDOS steps raises m ahead of every step from then
// on (READY stays off).  Wan-1.3B 1x, Q and K times 4, 8, 16, 32, ms, on one board:
// 4.55, 4.57, 4.73, 4.83 without, 4.59, 4.49, 4.47, 4.45 with (row maximum every step
// and 32x32x16 MFMAs: 5.13, 4.57, 4.48, 4.42).  Whole tiles of two query blocks only:
// split tiles and tiles of four are well ahead of the latter at any width and would
// pay 1% and up to 3% on ordinary inputs.
template <int NU, bool EAGER, bool LOADS>
__device__ __forceinline__ void softmax_phase(const Scores<NU>& sc, WaveState& st,
                                              Probs<NU>& pr, float scale_log2,
                                              const StepLoads& sl) {
  const int flags = __builtin_amdgcn_readfirstlane(st.flags);
  const bool first = !(flags & READY);
  if (first)
    raise_max<NU, true, EAGER>(sc, st, scale_log2, (flags & WIDE) ? WIDE_HEADROOM : HEADROOM,
                               0.f);
  float m[2];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) m[qt] = st.m[qt] == -__builtin_inff() ? 0.f : st.m[qt];
  const uint32_t bits = probabilities<NU, LOADS>(sc, pr, m, scale_log2, sl);
  if (__builtin_amdgcn_ballot_w64((bits & 0x40004000u) != 0u) && !first) {
    st.flags = EAGER ? (st.flags | WIDE) + REDO : st.flags | WIDE;
    raise_max<NU, false, EAGER>(sc, st, scale_log2, WIDE_HEADROOM,
                                (flags & WIDE) ? 0.f : WIDE_HEADROOM - HEADROOM);
    probabilities<NU, false>(sc, pr, st.m, scale_log2, sl);
  }
}

// GEMM phase of the ping-pong schedule: l += the row sums of P(j) (one MFMA per
// 32 keys and query tile, `ones` its A operand); then
// O += P(j) V(j) and S(j+1) = K(j+1) Q^T into `sc`, with K and V fragments
// read AHEAD fragments early.  The row-sum MFMAs come first: their operands are already in
// registers, so they run while the first fragments arrive from LDS.  LOADS: the
// step's tile loads `sl` are issued evenly over the phase.
//
// SUBS: the key blocks of a step (halves of the wave's key groups) that the wave's
// query block may or may not keep (0: it keeps all it walks); bit i of `keep` says
// whether it keeps key block i.  V of the others is left out, so that what a key
// block holds (inf, NaN) never reaches a query block that does not keep it; such a
// step issues none of the loads.
template <int NU, int SUBS, bool LOADS>
__device__ __forceinline__ void gemm_phase(const char* lds_k, const char* lds_v,
                                           const bf16x8 (&qf)[4][2], Scores<NU>& sc,
                                           const Probs<NU>& pr, WaveState& st,
                                           const FragAddr& fa, const bf16x8& ones, int keep,
                                           const StepLoads& sl) {
  if constexpr (SUBS > 0) {
    if (keep != (1 << SUBS) - 1) {
      if constexpr (SUBS > 1) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          if (!((keep >> (u / (NU / SUBS))) & 1)) continue;
#pragma unroll
          for (int qt = 0; qt < 2; ++qt)
            st.l[qt] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pr.p[u][qt], st.l[qt], 0, 0, 0);
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) {
            const bf16x8 f = v_frag(lds_v, fa, dt, u);
#pragma unroll
            for (int qt = 0; qt < 2; ++qt)
              st.o[dt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, pr.p[u][qt],
                                                                     st.o[dt][qt], 0, 0, 0);
          }
        }
      }
      compute_scores<NU>(lds_k, qf, sc, fa);
      return;
    }
  }
  constexpr int NS = 8 * NU;   // K fragments: (key tile, d-step)
  constexpr int NP = 8 * NU;   // V fragments: (d tile, 32-key group)
  constexpr int NF = NS + NP;
  constexpr int AHEAD = NU == 4 ? 8 : 4;
  // Fragment i < NP: V^T, d tile i/NU, key group i%NU.  Fragment NP + f: K, key
  // tile f/4, d-step f%4.  P(j) (with its row sums) is done before S(j+1) is
  // produced, so the two are never live together.
  auto frag = [&](int i) -> bf16x8 {
    return i < NP ? v_frag(lds_v, fa, i / NU, i % NU)
                  : k_frag(lds_k, fa, (i - NP) / 4, (i - NP) % 4);
  };
  bf16x8 fr[NF];
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) fr[i] = frag(i);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int qt = 0; qt < 2; ++qt)
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      st.l[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pr.p[u][qt], st.l[qt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  // What MFMA m of the phase's 2 * NF carries along: the read of half a V
  // fragment, or of a K fragment at every second one; a tile load at every
  // EVERY-th.
  constexpr int EVERY = 2 * NF / (2 * Tile::LOADS);
  i16x4 lo = i16x4{};
  auto carry = [&](int m) {
    if (LOADS && m % EVERY == EVERY - 1) issue_step_load(sl, m / EVERY);
    const int i = m / 2 + AHEAD;
    if (i < NF) {
      if (i >= NP) {
        if (m % 2 == 0) fr[i] = frag(i);
      } else if (m % 2 == 0) {
        lo = v_half(lds_v, fa, i / NU, i % NU, 0);
      } else {
        fr[i] = join(lo, v_half(lds_v, fa, i / NU, i % NU, 1));
      }
    }
  };
  // The fragments of one accumulator pair (NU for a d tile, 4 for a key tile)
  // one after the other into one query tile's accumulator, then in the other
  // order into the other's; the next pair starts with the query tile that the
  // last one ended with.  So consecutive MFMAs share the accumulator within a
  // chain and one operand between chains, which is what costs the least energy
  // (the launch is limited by power): chains instead of alternating
  // accumulators took 1-2% off the call, the order of the query tiles 0.6-1%.
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
      for (int i = 0; i < NU; ++i) {
        const int u = qt ? NU - 1 - i : i, q = qt ^ (dt & 1);
        carry((2 * dt + qt) * NU + i);
        st.o[dt][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[dt * NU + u], pr.p[u][q],
                                                               st.o[dt][q], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
  for (int kt = 0; kt < 2 * NU; ++kt)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int stp = qt ? 3 - i : i, q = qt ^ (kt & 1);
        carry(2 * NP + (2 * kt + qt) * 4 + i);
        sc.s[kt][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            fr[NP + 4 * kt + stp], qf[stp][q], i == 0 ? f32x4{} : sc.s[kt][q], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
}

// The thread's index, through an opaque move: what a tile derives from it is derived
// again by the next one instead of being kept, and spilled, across the tile.
__device__ __forceinline__ int fresh_tid() {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  return tid;
}

// LDS of the merged walk: the step words of the tile's query blocks (kept for
// the whole tile) and per-wave counts of the merge.  The merge's inputs, two CSR
// rows or the bitmaps of four, are staged in the K/V tile buffers, which are idle
// at the start of a tile.  The union of the rows has at most nb words, so nb <=
// WALK_CAP (checked before launch) lets one merge cover the tile.
constexpr int WALK_CAP = 8000;
struct WalkLds {
  uint32_t w[WALK_CAP];       // step words, in walk order
  int32_t cnt[2][16][5];      // per-wave counts of a merge pass (double-buffered)
};
static_assert(2 * WALK_CAP * 4 <= 4 * Tile::BYTES, "rows staged in the tile buffers");

// Step words of one or two rows (of four: merge_four).  Block form (row entries are
// key blocks): kb in bits 0..29, bit 30 / 31 set when row 0 / row 1 keeps kb.
// Token-exact form (row entries are entry words): bits 0..23 kb and kfirst, bits 24..27 / 28..31
// the patterns of row 0 / row 1, 0 where that row does not keep kb.  A key
// block outside [0, nb) gives a word that masks every key (and whose loads
// read zeros).
template <bool EXACT>
__device__ __forceinline__ int32_t entry_key(uint32_t e) {
  return EXACT ? (int32_t)(e & 0xFFFFu) : (int32_t)e;
}
template <bool EXACT>
__device__ __forceinline__ uint32_t step_word(uint32_t e0, uint32_t e1, bool in0, bool in1,
                                              int32_t nb) {
  const int32_t kb = entry_key<EXACT>(in0 ? e0 : e1);
  if (kb < 0 || kb >= nb) return EXACT ? 0xFFFFu : 0x3FFFFFFFu;
  if constexpr (EXACT)
    return ((in0 ? e0 : e1) & 0xFFFFFFu) | (in0 ? e0 & 0x0F000000u : 0u) |
           (in1 ? (e1 & 0x0F000000u) << 4 : 0u);
  return (uint32_t)kb | (in0 ? 1u << 30 : 0u) | (in1 ? 1u << 31 : 0u);
}

// Merges CSR rows 2p ("row 0": entries lo0 .. hi0-1) and 2p+1 ("row 1":
// lo1 .. hi1-1) into L.w, largest key first (every thread of the workgroup
// takes part; starts and ends with a barrier).  Both rows are staged in
// `stage` from their ends down; an entry's position in the union is its
// index in its own row, plus the entries of the other row with a larger key
// (a binary search), minus the keys above it that both rows hold (a count of
// its row's duplicates before it).  Returns the number of words.  Rows of up
// to WALK_CAP entries are merged whole (more are cut); rows that are not
// strictly ascending give some order of their entries, never a write outside
// L.w.
template <int NT, bool EXACT>
__device__ __forceinline__ int32_t merge_pair(WalkLds& L, uint32_t* stage,
                                              const uint32_t* __restrict__ rows,
                                              int32_t lo0, int32_t hi0, int32_t lo1,
                                              int32_t hi1, int32_t nb) {
  const int tid = fresh_tid(), lane = tid % 64, wave = tid / 64;
  constexpr int NWAVE = NT / 64;
  uint32_t* const sa = stage;              // row 0, largest key first
  uint32_t* const sb = stage + WALK_CAP;   // row 1
  const int na = max(0, min(hi0 - lo0, WALK_CAP));
  const int nc = max(0, min(hi1 - lo1, WALK_CAP));
  __syncthreads();   // the stage buffers are idle
  for (int t = tid; t < na; t += NT) sa[t] = rows[hi0 - 1 - t];
  for (int t = tid; t < nc; t += NT) sb[t] = rows[hi1 - 1 - t];
  __syncthreads();
  int dup_base0 = 0, dup_base1 = 0, words = 0;
  const int passes = (max(na, nc) + NT - 1) / NT;
  for (int ps = 0; ps < passes; ++ps) {
    const int t = ps * NT + tid;
    // Entries of the other row with a larger key: the first index whose key
    // is not larger (the staged rows descend), by binary search.
    int above0 = 0, above1 = 0;
    bool dup0 = false, dup1 = false;
    uint32_t e0 = 0u, e1 = 0u, p0 = 0u;
    if (t < na) {
      e0 = sa[t];
      const int32_t x = entry_key<EXACT>(e0);
      int lo = 0, hi = nc;
      while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (entry_key<EXACT>(sb[mid]) > x) lo = mid + 1; else hi = mid;
      }
      above0 = lo;
      if (lo < nc) {
        p0 = sb[lo];
        dup0 = entry_key<EXACT>(p0) == x;
      }
    }
    if (t < nc) {
      e1 = sb[t];
      const int32_t y = entry_key<EXACT>(e1);
      int lo = 0, hi = na;
      while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (entry_key<EXACT>(sa[mid]) > y) lo = mid + 1; else hi = mid;
      }
      above1 = lo;
      dup1 = lo < na && entry_key<EXACT>(sa[lo]) == y;
    }
    // Keys held by both rows above each entry: its row's duplicates before it.
    const uint64_t m0 = __ballot(dup0), m1 = __ballot(dup1);
    const uint64_t below = (1ull << lane) - 1ull;
    if (lane == 0) {
      L.cnt[ps & 1][wave][0] = __popcll(m0);
      L.cnt[ps & 1][wave][1] = __popcll(m1);
    }
    __syncthreads();
    int before0 = dup_base0 + __popcll(m0 & below), before1 = dup_base1 + __popcll(m1 & below);
    for (int w = 0; w < NWAVE; ++w) {
      const int v0 = L.cnt[ps & 1][w][0], v1 = L.cnt[ps & 1][w][1];
      before0 += w < wave ? v0 : 0;
      before1 += w < wave ? v1 : 0;
      dup_base0 += v0;
      dup_base1 += v1;
    }
    if (t < na) {
      const int r = t + above0 - before0;
      if (r >= 0 && r < WALK_CAP) L.w[r] = step_word<EXACT>(e0, p0, true, dup0, nb);
    }
    if (t < nc && !dup1) {
      const int r = t + above1 - before1;
      if (r >= 0 && r < WALK_CAP) L.w[r] = step_word<EXACT>(0u, e1, false, true, nb);
    }
    words = na + nc - dup_base1;
  }
  __syncthreads();   // the words are written; the stage buffers are free again
  return __builtin_amdgcn_readfirstlane(min(words, WALK_CAP));
}

// Merges four CSR rows (entries rp[i] .. rp[i+1]-1) into L.w, largest key first:
// a bitmap of every row's key blocks in `stage`, and a key block's position is
// the number of blocks above it in their union.  Words: kb in bits 0..27, bit
// 28 + i set when row i keeps kb; entries outside [0, nb) are skipped, and at
// most WALK_CAP entries of a row are read.  Returns the number of words (starts
// and ends with a barrier); `apart`: the words that parts of PART query blocks
// (1 or 2) would walk, all together.
template <int PART>
__device__ __forceinline__ int32_t merge_four(WalkLds& L, uint32_t* stage,
                                              const uint32_t* __restrict__ rows,
                                              const int32_t (&rp)[5], int32_t nb,
                                              int32_t& apart) {
  constexpr int WORDS = 256;                 // of 32 key blocks: WALK_CAP / 32, rounded up
  static_assert(WORDS * 32 >= WALK_CAP, "bitmap size");
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  uint32_t* const bm = stage;                // [row][word]
  uint32_t* const all = stage + 4 * WORDS;   // union
  int32_t* const above = (int32_t*)(stage + 5 * WORDS);   // blocks in the words after this one
  __syncthreads();   // the stage buffers are idle
  for (int t = tid; t < 4 * WORDS; t += Tile::NT) bm[t] = 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i)
    for (int t = max(rp[i], rp[i + 1] - WALK_CAP) + tid; t < rp[i + 1]; t += Tile::NT) {
      const uint32_t kb = rows[t];
      if (kb < (uint32_t)nb) atomicOr(&bm[i * WORDS + kb / 32], 1u << (kb % 32));
    }
  __syncthreads();
  // Threads 0..255 hold the words last to first; blocks before a thread's
  // word in that order are the blocks above it.
  const int w = WORDS - 1 - tid;
  // Counts of both kinds in one scan: the union's in the low half (at most 8192),
  // the parts' in the high half (at most 32768).
  uint32_t cnt = 0, incl = 0;
  if (tid < WORDS) {
    const uint32_t r0 = bm[w], r1 = bm[WORDS + w], r2 = bm[2 * WORDS + w], r3 = bm[3 * WORDS + w];
    const uint32_t u = r0 | r1 | r2 | r3;
    all[w] = u;
    const int ap = PART == 2 ? __popc(r0 | r1) + __popc(r2 | r3)
                             : __popc(r0) + __popc(r1) + __popc(r2) + __popc(r3);
    cnt = (uint32_t)__popc(u) | (uint32_t)ap << 16;
    incl = cnt;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    if (lane == 63) L.cnt[0][wave][0] = (int32_t)incl;
  }
  __syncthreads();
  uint32_t total = 0;
  for (int v = 0; v < WORDS / 64; ++v) {
    const uint32_t c = (uint32_t)L.cnt[0][v][0];
    if (v < wave) incl += c;
    total += c;
  }
  if (tid < WORDS) above[w] = (int32_t)((incl - cnt) & 0xFFFFu);
  __syncthreads();
  for (int kb = tid; kb < nb; kb += Tile::NT) {
    const uint32_t rest = all[kb / 32] >> (kb % 32);   // this block and those above it
    if (!(rest & 1u)) continue;
    uint32_t word = (uint32_t)kb;
#pragma unroll
    for (int i = 0; i < 4; ++i) word |= ((bm[i * WORDS + kb / 32] >> (kb % 32)) & 1u) << (28 + i);
    L.w[above[kb / 32] + __popc(rest >> 1)] = word;
  }
  __syncthreads();   // the words are written; the stage buffers are free again
  total = (uint32_t)__builtin_amdgcn_readfirstlane((int)total);
  apart = (int32_t)(total >> 16);
  return (int32_t)(total & 0xFFFFu);
}

// The step words of a tile that lies in one query block: its CSR row, largest
// key first.  Returns the number of words (ends with a barrier).
template <bool EXACT>
__device__ __forceinline__ int32_t single_row(WalkLds& L, const uint32_t* __restrict__ rows,
                                              int32_t lo, int32_t hi, int32_t nb) {
  const int n = max(0, min(hi - lo, WALK_CAP));
  for (int t = threadIdx.x; t < n; t += Tile::NT)
    L.w[t] = step_word<EXACT>(rows[hi - 1 - t], 0u, true, false, nb);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(n);
}

// Combines the key groups' partial results (KG > 1) and stores the tile's
// rows: each of the KG waves that hold the same rows keeps 8 / KG of the eight
// d tiles and takes the others' parts of them through LDS.  With m = max m_g,
// O = sum_g 2^(m_g - m) O_g and l = sum_g 2^(m_g - m) l_g, added in the order
// of the groups.  `xch`: the tile buffers, idle here; wave w's part of d tile
// dt is the 2 KB at 2048*(8*w + dt), and the slot of a d tile the wave keeps
// holds its rows' (m, l).
template <int KG>
__device__ __forceinline__ void combine_groups(char* xch, WaveState& st, const float (&lsum)[2],
                                               __bf16* oh, int64_t o_st, int qrow, int N,
                                               int wave, int lane) {
  using SP = Split<KG>;
  constexpr int KEEP = 8 / KG;
  const int rg = wave % SP::NRG, kg = wave / SP::NRG;
  auto slot = [&](int w, int dt) { return xch + 2048 * (8 * w + dt); };
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) {
    if (dt / KEEP == kg) continue;
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
      *(f32x4*)(slot(wave, dt) + 1024 * qt + 16 * lane) = st.o[dt][qt];
  }
  if (lane < 16) {
    float* const ml = (float*)(slot(wave, kg * KEEP) + 16 * lane);
    ml[0] = st.m[0];
    ml[1] = lsum[0];
    ml[2] = st.m[1];
    ml[3] = lsum[1];
  }
  __syncthreads();
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    float mg[KG], f[KG], m = -__builtin_inff(), l = 0.f;
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      mg[g] = *(const float*)(slot(g * SP::NRG + rg, g * KEEP) + 16 * (lane % 16) + 8 * qt);
      m = fmaxf(m, mg[g]);
    }
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      f[g] = mg[g] == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(mg[g] - m);
      l += f[g] *
           *(const float*)(slot(g * SP::NRG + rg, g * KEEP) + 16 * (lane % 16) + 8 * qt + 4);
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const bool ok = qrow + 16 * qt < N;
    __bf16* const orow = oh + (int64_t)(qrow + 16 * qt) * o_st + 4 * (lane / 16);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      if (dt / KEEP != kg) continue;
      f32x4 acc = f32x4{};
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        const f32x4 part = g == kg ? st.o[dt][qt]
                                   : *(const f32x4*)(slot(g * SP::NRG + rg, dt) + 1024 * qt +
                                                     16 * lane);
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[b] += part[b] * f[g];
      }
      bf16x4 w;
#pragma unroll
      for (int b = 0; b < 4; ++b) w[b] = (__bf16)(acc[b] * inv);
      if (ok) *(bf16x4*)(orow + 16 * dt) = w;
    }
  }
}

// MODE: ATTN_DENSE (every key block), ATTN_BLOCK (CSR rows of key blocks),
// ATTN_EXACT (CSR rows of token-exact entry words).
// One tile: rows row0 .. row0 + ROWS - 1 of head `head`, using the
// workgroup's LDS stages `lds` (K slots 0-1, V slots 0-1).  The tile lies in
// one query block or covers two or four whole ones.
// Returns false, with nothing done, where parts of KGP key groups (KGP > KG) take
// less time than the tile whole: a tile of four query blocks walks the union of their
// rows, and where these have little in common the walks of the parts, each at its
// share of a whole tile's time (PART_TIME), are the shorter ones.  Measured, 64-token
// blocks, 12 heads of 32,768 tokens, 10% of the blocks kept: rows alike in pairs and
// independent otherwise 0.75 ms against 0.98 with whole tiles only, all independent
// 1.19 and 1.69 ms, rows alike in fours (whole tiles) 0.60 either way.
template <int BLOCK, int MODE, int KG, int KGP>
__device__ __forceinline__ bool attn_tile(
    char* lds, WalkLds& walk, int head, int row0, const __bf16* __restrict__ qg,
    const __bf16* __restrict__ kg_, const __bf16* __restrict__ vg, __bf16* __restrict__ og,
    int64_t q_sh, int64_t q_st, int64_t k_sh, int64_t k_st, int64_t v_sh, int64_t v_st,
    int64_t o_sh, int64_t o_st, int32_t N, int32_t nb, const int32_t* __restrict__ row_ptr,
    const uint32_t* __restrict__ rows, int32_t P, float scale_log2) {
  using TL = Tile;
  using SP = Split<KG>;
  constexpr int NU = SP::NU;
  constexpr bool SPARSE = MODE != ATTN_DENSE;
  constexpr bool EXACT = MODE == ATTN_EXACT;
  constexpr bool QUAD = SP::ROWS == 4 * BLOCK;   // four query blocks
  constexpr bool PAIR = SP::ROWS == 2 * BLOCK;   // two of them, else (part of) one
  constexpr int SUBS = TL::KEYS / BLOCK;         // key blocks per step
  // Key blocks of a step that a wave's query block may not keep (gemm_phase): of a
  // tile in one query block none, of a wave whose keys lie in one key block one.
  constexpr int SKIP = !SPARSE ? 0 : QUAD ? 2 : PAIR ? 1 : 0;
  constexpr bool EAGER = KG == 1 && !QUAD;       // softmax_phase
  // Four query blocks only in the block form: four 4-bit patterns and a key
  // block do not fit the token-exact form's words.
  static_assert(QUAD ? MODE == ATTN_BLOCK && SUBS == 2 : SP::ROWS <= 2 * BLOCK, "tile rows");
  static_assert(QUAD || SP::NK <= BLOCK, "a wave's keys lie in one key block");
  constexpr uint32_t KB_MASK = EXACT ? 0xFFFFu : QUAD ? 0x0FFFFFFFu : 0x3FFFFFFFu;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void*)lds;

  const int tid = SPARSE ? fresh_tid() : (int)threadIdx.x;
  const int wave = tid / 64;
  const int lane = tid % 64;
  const int g16 = lane / 16;
  const int li = lane % 16;

  const int rg = wave % SP::NRG, kg = wave / SP::NRG;
  const bool upper = wave >= TL::NW / 2;        // follows half a step behind
  const int qb0 = row0 / BLOCK;                 // the tile's (first) query block
  const int wrow = row0 + 32 * rg;              // the wave's first row
  const int qb = wrow / BLOCK;
  // The wave's first key in its key block.
  const int koff = KG == 1 ? 0 : kg * SP::NK % BLOCK;
  // The wave's key block of a step (and the one it loads): word SUBS*j + sub.
  const int sub = SUBS == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave / (TL::NW / 2));

  const __bf16* qh = qg + head * q_sh;
  __bf16* oh = og + head * o_sh;
  const __bf16* const kh_base = kg_ + head * k_sh;
  const __bf16* const vh_base = vg + head * v_sh;
  const uint32_t k_bytes = (uint32_t)(((int64_t)(N - 1) * k_st + D) * 2);
  const uint32_t v_bytes = (uint32_t)(((int64_t)(N - 1) * v_st + D) * 2);
  const LoadPlan kp = load_plan<BLOCK>((uint32_t)(k_st * 2), wave, lane);
  const LoadPlan vp = load_plan<BLOCK>((uint32_t)(v_st * 2), wave, lane);
  // Step words: key block in bits 0..29 (block form; 0..27 with four query
  // blocks) or 0..15 (exact form).
  auto kb_of = [&](uint32_t w) { return (int)(w & KB_MASK); };
  auto rk_at = [&](uint32_t w) {
    return tile_rsrc<BLOCK>(kh_base, k_st, k_bytes, kb_of(w), nb);
  };
  auto rv_at = [&](uint32_t w) {
    return tile_rsrc<BLOCK>(vh_base, v_st, v_bytes, kb_of(w), nb);
  };
  const FragAddr fa = frag_addr(lane, KG == 1 ? 0 : kg * SP::NK);

  // Q fragments: rows qrow and qrow + 16, k-slots d = 32*stp + 8*g16 + 0..7.
  const int qrow = wrow + li;
  bf16x8 qf[4][2];
#pragma unroll
  for (int stp = 0; stp < 4; ++stp)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
      qf[stp][qt] = qrow + 16 * qt < N ? *(const bf16x8*)(qh + (int64_t)(qrow + 16 * qt) * q_st +
                                                          32 * stp + 8 * g16)
                                       : bf16x8{};

  // Exact mode: the first of the wave's 32 rows that lies in the query
  // block's second frame (the first frame holds the block's first qfirst
  // rows; P >= BLOCK, so there are at most two); wave-uniform.
  int sec_from = 32;
  if constexpr (EXACT) {
    const int qfirst = P - (int)(((int64_t)qb * BLOCK) % P);
    sec_from = __builtin_amdgcn_readfirstlane(qfirst - (wrow - qb * BLOCK));
  }
  // Masks the scores of the key block of step word w for this wave's query
  // block: a key block that block does not keep has no valid keys.
  // `second`: the wave holds rows of query block 2p + 1.
  // Returns whether the wave's query block keeps it.
  auto mask_block = [&](Scores<NU>& sc, uint32_t w, bool second) -> int {
    const int kb = kb_of(w);
    const uint32_t kept_bit = second ? 31u : 30u;      // block form
    const uint32_t pat_shift = second ? 28u : 24u;     // exact form
    if constexpr (EXACT) {
      const uint32_t pat = (w >> pat_shift) & 0xFu;
      mask_exact<BLOCK, NU>(sc, pat, (int)((w >> 16) & 0xFFu), N - kb * BLOCK, sec_from, koff);
      return pat != 0u;
    } else {
      const int kept = (int)((w >> kept_bit) & 1u);
      mask_tail<NU>(sc, lane, kept ? N - kb * BLOCK - koff : 0);
      return kept;
    }
  };

  // The walk (sparse modes) or the key blocks nb-1 .. 0 (dense): n steps.
  // Words of steps past the last one repeat it: their loads land in slots
  // that no later step reads.
  int words = nb;
  // Dense: the words nb-1 .. 0 (both query blocks keep every key block),
  // written to LDS and read from there like the merged walk's (timed faster
  // than computing them in the loop: 1.7% at the Wan-1.3B 6x shape and 2.9%
  // at 40 heads, interleaved on one board); steps past WALK_CAP compute
  // theirs.  The block mode runs dense attention this way when it is given
  // no CSR (row_ptr null, nb <= WALK_CAP): the same code as a full mask's
  // walk, without the merge.
  auto dense_word = [&](int i) {
    return i < nb ? (uint32_t)(nb - 1 - i) | ~KB_MASK : KB_MASK;
  };
  auto dense_words = [&]() {
    __syncthreads();
    for (int t = threadIdx.x; t < min(nb, WALK_CAP); t += TL::NT) walk.w[t] = dense_word(t);
    __syncthreads();
  };
  if constexpr (SPARSE) {
    if (EXACT || row_ptr != nullptr) {
      const int32_t r0 = __builtin_amdgcn_readfirstlane(row_ptr[qb0]);
      const int32_t r1 = __builtin_amdgcn_readfirstlane(row_ptr[qb0 + 1]);
      if constexpr (QUAD) {
        int32_t rp[5] = {r0, r1, 0, 0, 0};
#pragma unroll
        for (int i = 2; i < 5; ++i)
          rp[i] = __builtin_amdgcn_readfirstlane(row_ptr[min(qb0 + i, nb)]);
        int32_t apart = 0;
        words = merge_four<4 / KGP>(walk, (uint32_t*)lds, rows, rp, nb, apart);
        if (KGP > KG && 100 * (words - PARTS_FIXED) > PART_TIME[KGP] * apart) return false;
      } else if constexpr (PAIR) {
        const int32_t r2 =
            qb0 + 1 < nb ? __builtin_amdgcn_readfirstlane(row_ptr[qb0 + 2]) : r1;
        words = merge_pair<TL::NT, EXACT>(walk, (uint32_t*)lds, rows, r0, r1, r1, r2, nb);
      } else {
        words = single_row<EXACT>(walk, rows, r0, r1, nb);
      }
    } else {
      dense_words();
    }
  } else {
    dense_words();
  }
  if constexpr (SUBS == 2) {
    // An odd walk ends with a word that no query block keeps and whose loads
    // read zeros (words < WALK_CAP, which is even).
    if (words & 1) {
      if (tid == 0 && words < WALK_CAP) walk.w[words] = KB_MASK;
      __syncthreads();
    }
  }
  const int n = (words + SUBS - 1) / SUBS;
  uint32_t w0 = 0u, w1 = 0u, w2 = 0u;
  if (n > 0) {
    w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)walk.w[sub]);
    w1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)walk.w[SUBS * min(1, n - 1) + sub]);
    w2 = (uint32_t)__builtin_amdgcn_readfirstlane((int)walk.w[SUBS * min(2, n - 1) + sub]);
  }
  // With four query blocks a wave takes the keys of both key blocks of a step:
  // the words of the one it does not load.
  uint32_t o0 = 0u, o1 = 0u, o2 = 0u;
  if (QUAD && n > 0) {
    o0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)walk.w[1 - sub]);
    o1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)walk.w[SUBS * min(1, n - 1) + 1 - sub]);
    o2 = (uint32_t)__builtin_amdgcn_readfirstlane((int)walk.w[SUBS * min(2, n - 1) + 1 - sub]);
  }

  WaveState ws;
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) ws.o[dt][qt] = f32x4{};
    ws.m[qt] = -__builtin_inff();
    ws.l[qt] = f32x4{};
  }
  ws.flags = 0;
  // A operand of the row-sum MFMA: rows 0, 4, 8 and 12 (register 0 of every
  // lane of the result) take all 32 keys, the others none.
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = lane % 4 == 0 ? (__bf16)1.f : (__bf16)0.f;

  if (n > 0) {
    // LDS stages: K(b) in K slot b % 2, V(b) in V slot b % 2.
    const uint32_t k_slot0 = lds_base, v_slot0 = lds_base + 2 * TL::BYTES;
    const char* const k_lds = lds;
    const char* const v_lds = lds + 2 * TL::BYTES;

    // Ping-pong schedule.  Waves 0..3 ("leaders") run half a step ahead of
    // waves 4..7, so on each SIMD one wave is in its GEMM phase (O += P(j)
    // V(j), S(j+1) = K(j+1) Q^T: MFMA) while the other is in its softmax phase
    // (VALU): half-period 2j is the leaders' GEMM j and the others' softmax j,
    // half-period 2j+1 the leaders' softmax j+1 and the others' GEMM j.  A
    // barrier ends every half-period.  K(j+1) and V(j) stay resident through
    // half-periods 2j and 2j+1; K(j+2) and V(j+1) are issued in half-period 2j
    // (into the slots of K(j) and V(j-1), free since half-period 2j-1) and
    // waited for at the end of 2j+1.
    // (With KG = 1 the followers are the waves of the tile's second half: its second
    // query block, or the last two of four.)
    int lead_v = upper ? 0 : 1;
    asm("" : "+v"(lead_v));
    const bool lead = lead_v != 0;
    auto second = [&](bool follower) { return PAIR && (KG == 1 ? follower : qb > qb0); };
    // Masks a step's scores: its key block, or with four query blocks its two
    // (returns which of them the wave's query block keeps).
    auto mask_step = [&](Scores<NU>& sc, uint32_t w, uint32_t o, bool follower) -> int {
      if constexpr (QUAD) {
        const uint32_t wa = sub ? o : w, wb = sub ? w : o;
        const int bit = __builtin_amdgcn_readfirstlane(28 + qb - qb0);
        const int ka = (wa >> bit) & 1u, kb = (wb >> bit) & 1u;
        mask_tail<NU, 0, NU>(sc, lane, ka ? N - kb_of(wa) * BLOCK : 0);
        mask_tail<NU, NU, NU>(sc, lane, kb ? N - kb_of(wb) * BLOCK : 0);
        return ka | kb << 1;
      } else {
        return mask_block(sc, w, second(follower));
      }
    };
    issue_tile(k_slot0, rk_at(w0), kp);
    issue_tile(v_slot0, rv_at(w0), vp);
    issue_tile(k_slot0 + TL::BYTES, rk_at(w1), kp);
    wait_loads_and_sync();
    Scores<NU> sc;
    compute_scores<NU>(k_lds, qf, sc, fa);   // S(0)
    int keep = mask_step(sc, w0, o0, upper);
    Probs<NU> pr;
    if (lead) softmax_phase<NU, EAGER, false>(sc, ws, pr, scale_log2, StepLoads{});   // P(0)
    __syncthreads();
    for (int j = 0; j < n; ++j) {
      // Word of step j+3 from the walk's LDS, read now and used at the end of
      // the step (the last word again past the end of the walk; a sparse
      // walk never passes WALK_CAP words, nb <= WALK_CAP).
      const int g3 = SUBS * min(j + 3, n - 1) + sub;
      const uint32_t w3v = walk.w[min(g3, WALK_CAP - 1)];
      const uint32_t o3v = QUAD ? walk.w[min(g3 ^ 1, WALK_CAP - 1)] : 0u;
      const StepLoads sl{
          (uint32_t)__builtin_amdgcn_readfirstlane(k_slot0 + (uint32_t)(j & 1) * TL::BYTES),
          (uint32_t)__builtin_amdgcn_readfirstlane(v_slot0 + (uint32_t)((j + 1) & 1) * TL::BYTES),
          rk_at(w2), rv_at(w1), kp, vp};
      const char* const kj1 = k_lds + ((j + 1) & 1) * TL::BYTES;   // K(j+1)
      const char* const vj = v_lds + (j & 1) * TL::BYTES;          // V(j)
      // half-period 2j.  A leader whose query block does not keep the key block issues
      // its loads up front (gemm_phase).
      if (KG > 1 && SKIP && __builtin_amdgcn_readfirstlane(lead && !keep)) issue_step_loads(sl);
      if (lead) {
        gemm_phase<NU, SKIP, (KG > 1)>(kj1, vj, qf, sc, pr, ws, fa, ones, keep, sl);
        keep = mask_step(sc, w1, o1, false);
      } else {
        if constexpr (KG == 1) issue_step_loads(sl);
        softmax_phase<NU, EAGER, (KG > 1)>(sc, ws, pr, scale_log2, sl);
      }
      __syncthreads();
      // half-period 2j+1
      if (lead) {
        if (j + 1 < n) {
          if constexpr (KG == 1) issue_step_loads(sl);
          softmax_phase<NU, EAGER, false>(sc, ws, pr, scale_log2, sl);
        }
      } else {
        gemm_phase<NU, SKIP, false>(kj1, vj, qf, sc, pr, ws, fa, ones, keep, sl);
        keep = mask_step(sc, w1, o1, true);
      }
      wait_loads_and_sync();
      w1 = w2;
      if constexpr (QUAD) {
        o1 = o2;
        o2 = (uint32_t)__builtin_amdgcn_readfirstlane((int)o3v);
      }
      w2 = SPARSE || g3 < WALK_CAP ? (uint32_t)__builtin_amdgcn_readfirstlane((int)w3v)
                                   : dense_word(g3);
    }
    __syncthreads();
  }

  const float lsum[2] = {ws.l[0][0], ws.l[1][0]};   // whole in every lane
  if constexpr (KG > 1) {
    combine_groups<KG>(lds, ws, lsum, oh, o_st, qrow, N, wave, lane);
  } else {
    // Every wave holds whole rows: O / l, rounded to bf16.
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      const float inv = lsum[qt] > 0.f ? 1.f / lsum[qt] : 0.f;
      __bf16* const orow = oh + (int64_t)(qrow + 16 * qt) * o_st + 4 * g16;
      if (qrow + 16 * qt < N) {
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
          bf16x4 w;
#pragma unroll
          for (int b = 0; b < 4; ++b) w[b] = (__bf16)(ws.o[dt][qt][b] * inv);
          *(bf16x4*)(orow + 16 * dt) = w;
        }
      }
    }
  }
  return true;
}

// First item and item count of XCD x's share of `total` items: contiguous
// shares, the first total % 8 of them one item larger.
__device__ __forceinline__ int xcd_first(int x, int total) {
  const int per = total / 8, rem = total % 8;
  return x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per;
}
__device__ __forceinline__ int xcd_count(int x, int total) {
  return total / 8 + (x < total % 8 ? 1 : 0);
}

// A launch's items are `whole` whole tiles, then `split` parts of the tiles
// after them; an XCD's share is its share of the whole tiles followed by its
// share of the parts.  Item i of share x:
__device__ __forceinline__ int share_item(int x, int i, int whole, int split) {
  const int w = xcd_count(x, whole);
  return i < w ? xcd_first(x, whole) + i : whole + xcd_first(x, split) + (i - w);
}

// Next item for a workgroup on XCD `xcd`, or -1 when every item is handed
// out.  Items are dealt to the XCDs in shares; a workgroup takes the next
// item from the front of its own XCD's share and, once that share is handed
// out, the last one left at the back of another XCD's share, so XCDs that
// clock faster take on more items while each share is still worked from its
// front by its own XCD (neighbouring tiles, whose key lists overlap, stay
// together in that XCD's L2).  Counter word x holds in bits 0..31 the takes
// from the front of share x and in bits 32..63 those from its back; a take
// gets an item iff the two counts before it sum to less than the share's
// size, so each item goes out once.  Every call makes at most 8 atomic adds,
// so a workgroup's loop ends after at most items + 8 calls.
__device__ __forceinline__ int fetch_item(uint64_t* ctr, int xcd, int whole, int split) {
  for (int d = 0; d < 8; ++d) {
    const int x = (xcd + d) % 8;
    const uint64_t cnt = (uint64_t)(xcd_count(x, whole) + xcd_count(x, split));
    const uint64_t seen =
        __hip_atomic_load(&ctr[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((seen & 0xFFFFFFFFull) + (seen >> 32) >= cnt) continue;
    const uint64_t old = __hip_atomic_fetch_add(&ctr[x], d == 0 ? 1ull : 1ull << 32,
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t front = old & 0xFFFFFFFFull, back = old >> 32;
    if (front + back < cnt)
      return share_item(x, d == 0 ? (int)front : (int)(cnt - 1 - back), whole, split);
  }
  return -1;
}

// Kernel arguments, passed as one struct so that the persistent loop can
// read them again for every tile instead of holding them in registers.
struct KArgs {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  __bf16* o;
  int64_t q_sh, q_st, k_sh, k_st, v_sh, v_st, o_sh, o_st;
  const int32_t* row_ptr;
  const uint32_t* rows;
  uint64_t* counters;        // null: one item per workgroup
  int32_t N, nb, P;
  int32_t per_head;          // whole tiles of a head
  int32_t whole, split;      // items (share_item)
  float scale_log2;
};

template <int BLOCK, int MODE, int KG, int KGP>
__device__ __forceinline__ bool attn_tile_args(char* lds, WalkLds& walk, int head, int row0,
                                               const KArgs& a) {
  return attn_tile<BLOCK, MODE, KG, KGP>(lds, walk, head, row0, a.q, a.k, a.v, a.o, a.q_sh,
                                         a.q_st, a.k_sh, a.k_st, a.v_sh, a.v_st, a.o_sh, a.o_st,
                                         a.N, a.nb, a.row_ptr, a.rows, a.P, a.scale_log2);
}

// The kernel's arguments (its first), read through an offset that the compiler
// cannot see to be zero: every tile loads them afresh (scalar loads), so they are
// not live across tiles.
__device__ __forceinline__ const KArgs* fresh_args() {
  int zero = 0;
  asm volatile("" : "+v"(zero));
  zero = __builtin_amdgcn_readfirstlane(zero);
  return (const KArgs*)((const char*)__builtin_amdgcn_kernarg_segment_ptr() + zero);
}

// Persistent workgroups, at most one per CU, take items until all are done
// (fetch_item), through the launch's own counters, zeroed by
// zero_counters_kernel just before on the same stream; without counters
// there is a workgroup for every item (all whole or all split).  Whole tiles
// run with KGW key groups, the parts of split ones with KGS (KGS / KGW parts
// per tile).
template <int BLOCK, int MODE, int KGW, int KGS>
__global__ __launch_bounds__(Tile::NT) void attn_fwd_kernel(const KArgs args) {
  __shared__ __attribute__((aligned(1024))) char lds[4 * Tile::BYTES];
  __shared__ WalkLds walk;
  __shared__ int next_item;
  constexpr int PARTS = KGS / KGW;
  // attn_tile may refuse whole tiles of four query blocks.
  constexpr bool REFUSES = MODE == ATTN_BLOCK && Split<KGW>::ROWS == 4 * BLOCK && PARTS > 1;
  // Workgroups are dispatched round-robin over the 8 XCDs.
  const int xcd = blockIdx.x % 8;
  for (;;) {
    int item;
    if (args.counters) {
      if (threadIdx.x == 0)
        next_item = fetch_item(args.counters, xcd, args.whole, args.split);
      __syncthreads();
      item = __builtin_amdgcn_readfirstlane(next_item);
      __syncthreads();   // every wave has read next_item before it is rewritten
      if (item < 0) break;
    } else {
      item = __builtin_amdgcn_readfirstlane(
          share_item(xcd, (int)(blockIdx.x / 8), args.whole, args.split));
    }
    // Tiles of a head go last to first: rows that attend every key block (text
    // tokens, placed after the video tokens) are the longest tiles, and taking
    // them first keeps them out of the grid's tail (each row's key blocks are
    // then walked in descending order, which keeps neighbouring workgroups'
    // shared blocks in L2).
    if constexpr (REFUSES) {
      // First and last part to work: one part, all parts of a whole tile that was
      // refused (last to first), or none.
      const KArgs* ap = fresh_args();
      int i = -1, last = 0;
      if (item >= ap->whole) {
        i = last = PARTS - 1 - (item - ap->whole) % PARTS;
      } else {
        const int p = ap->per_head - 1 - item % ap->per_head;
        if (!attn_tile_args<BLOCK, MODE, KGW, KGS>(lds, walk, item / ap->per_head,
                                                   p * Split<KGW>::ROWS, *ap))
          i = PARTS - 1;
      }
      for (; i >= last; --i) {
        const KArgs* ap = fresh_args();
        const int tile = item < ap->whole ? item : ap->whole + (item - ap->whole) / PARTS;
        const int p = ap->per_head - 1 - tile % ap->per_head;
        const int row0 = p * Split<KGW>::ROWS + i * Split<KGS>::ROWS;
        if (row0 < ap->N)
          attn_tile_args<BLOCK, MODE, KGS, KGS>(lds, walk, tile / ap->per_head, row0, *ap);
      }
    } else {
      const KArgs* ap = fresh_args();
      if (item < ap->whole) {
        const int p = ap->per_head - 1 - item % ap->per_head;
        attn_tile_args<BLOCK, MODE, KGW, KGW>(lds, walk, item / ap->per_head,
                                              p * Split<KGW>::ROWS, *ap);
      } else if constexpr (PARTS > 1) {
        const int u = item - ap->whole;
        const int tile = ap->whole + u / PARTS;
        const int p = ap->per_head - 1 - tile % ap->per_head;
        const int row0 = p * Split<KGW>::ROWS + (PARTS - 1 - u % PARTS) * Split<KGS>::ROWS;
        if (row0 < ap->N)
          attn_tile_args<BLOCK, MODE, KGS, KGS>(lds, walk, tile / ap->per_head, row0, *ap);
      }
    }
    if (!args.counters) break;
  }
}

__global__ __launch_bounds__(64) void zero_counters_kernel(uint64_t* __restrict__ ctr) {
  if (threadIdx.x < kTileCounters) ctr[threadIdx.x] = 0;
}

// Compute units of the current device (cached per device).
int cu_count() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
      n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// How a launch's tiles are split (see Split): `whole` tiles of 256 / kgw rows,
// the rest in parts of 256 / kgs rows.
struct Plan {
  int kgw, kgs, whole;
};

int tiles_of(const AttnArgs& a, int kg) {
  const int rows = 256 / kg;
  return (int)(((int64_t)a.n_tokens + rows - 1) / rows) * a.heads;
}

// Rounds of whole tiles that the launch takes, by the plan: a CU works one
// tile at a time, so a last round that is nearly empty costs as much as a full
// one, and a launch of fewer tiles than CUs leaves CUs idle.  Splitting tiles
// over the key groups of a workgroup (Split) gives more, shorter items: a
// 128-row item takes 0.60 of a 256-row tile's time and a 64-row one 0.42
// (PART_TIME; not 0.5 and 0.25: each K/V tile brought into LDS serves fewer rows;
// measured with every CU busy, Wan-1.3B 1x and 6x: 4.48 and 28.7 ms whole, 5.28 and 33.3 ms in
// 128-row items, 7.69 and 43.1 ms in 64-row items; with 64-token blocks at 2x 9.34,
// 10.6 and 13.7 ms; walks of 16 steps 0.72 and 0.48, of 4 steps 0.94 and 0.61,
// where a tile's fixed times count: the plan they give is the same).  So whole
// tiles fill all rounds but the last one or two, and what remains is split if
// that ends earlier.
// 64-token blocks split the same way; in the token-exact form, whose step words
// hold two query blocks at most, 128-row tiles into 64-row ones.
Plan make_plan(const AttnArgs& a, int block, AttnMode mode, int cus) {
  struct Kind {
    int kgw, kgs;
    double part;   // time of a part, in whole tiles' times
  };
  static const Kind kinds[] = {{1, 2, 0.60}, {1, 4, 0.42}, {2, 4, 0.64}};
  const bool half = block == 64 && mode == ATTN_EXACT;
  const int from = half ? 2 : 0, to = half ? 3 : 2;
  const int tiles = tiles_of(a, kinds[from].kgw), rounds = tiles / cus;
  Plan best{kinds[from].kgw, kinds[from].kgs, tiles};
  // A split has to gain 1% to be taken.
  double best_cost = 0.99 * ((tiles + cus - 1) / cus);
  for (int i = from; i < to; ++i)
    for (int w = rounds; w >= 0 && w >= rounds - 1; --w) {
      const Kind& k = kinds[i];
      const int64_t parts = (int64_t)(tiles - w * cus) * (k.kgs / k.kgw);
      const double cost = w + (double)((parts + cus - 1) / cus) * k.part;
      if (cost < best_cost) {
        best_cost = cost;
        best = Plan{k.kgw, k.kgs, w * cus};
      }
    }
  return best;
}

// Items of a launch with that plan, and whether it runs a workgroup for every
// one of them (all whole or all parts): then it takes no counters.
int plan_items(const AttnArgs& a, const Plan& p) {
  return p.whole + (tiles_of(a, p.kgw) - p.whole) * (p.kgs / p.kgw);
}
bool plan_is_direct(const AttnArgs& a, const Plan& p, int cus) {
  const int items = plan_items(a, p);
  return items <= cus && (p.whole == 0 || p.whole == items);
}

template <int BLOCK, int MODE, int KGW, int KGS>
hipError_t launch_t(const AttnArgs& a, const Plan& p, hipStream_t stream) {
  const float scale_log2 = 1.4426950408889634f / __builtin_sqrtf((float)D);
  const int per_head = (int)(((int64_t)a.n_tokens + Split<KGW>::ROWS - 1) / Split<KGW>::ROWS);
  const int items = plan_items(a, p);
  // One persistent workgroup per CU (each takes 160 KB of LDS, so one fits a
  // CU), or one per item when there are fewer items.
  const int grid = items < cu_count() ? items : cu_count();
  KArgs k;
  k.q = (const __bf16*)a.q;
  k.k = (const __bf16*)a.k;
  k.v = (const __bf16*)a.v;
  k.o = (__bf16*)a.o;
  k.q_sh = a.q_sh; k.q_st = a.q_st; k.k_sh = a.k_sh; k.k_st = a.k_st;
  k.v_sh = a.v_sh; k.v_st = a.v_st; k.o_sh = a.o_sh; k.o_st = a.o_st;
  k.row_ptr = a.row_ptr;
  k.rows = a.rows;
  k.counters = plan_is_direct(a, p, cu_count()) ? nullptr : a.counters;
  k.N = a.n_tokens; k.nb = a.n_blocks; k.P = a.frame_tokens;
  k.per_head = per_head;
  k.whole = p.whole;
  k.split = items - p.whole;
  k.scale_log2 = scale_log2;
  if (k.counters)
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, stream, a.counters);
  hipLaunchKernelGGL((attn_fwd_kernel<BLOCK, MODE, KGW, KGS>), dim3(grid), dim3(Tile::NT), 0,
                     stream, k);
  return hipGetLastError();
}

}  // namespace

namespace {

// Dense attention over at most WALK_CAP key blocks runs the block mode's
// kernel without a CSR: the same code as the block-sparse kernel with a full
// mask, which it matched or beat only that way (a separate dense instantiation
// timed 0.6% slower than the full-mask launch at the Wan-1.3B 6x shape,
// interleaved on one board, for no difference in its step loop but the layout
// of its branches).
AttnMode kernel_mode(const AttnArgs& a, AttnMode mode) {
  return mode == ATTN_DENSE && a.n_blocks <= WALK_CAP ? ATTN_BLOCK : mode;
}

Plan plan_of(const AttnArgs& a, int32_t block, AttnMode mode) {
  // Past WALK_CAP key blocks: whole tiles only.
  if (mode == ATTN_DENSE) {
    const int kg = block == 128 ? 1 : 2;
    return Plan{kg, kg, tiles_of(a, kg)};
  }
  return make_plan(a, block, mode, cu_count());
}

}  // namespace

bool attention_uses_counters(const AttnArgs& a, int32_t block, AttnMode mode) {
  return !plan_is_direct(a, plan_of(a, block, kernel_mode(a, mode)), cu_count());
}

hipError_t launch_attention(const AttnArgs& a, int32_t block, AttnMode mode,
                            hipStream_t stream) {
  mode = kernel_mode(a, mode);
  const Plan p = plan_of(a, block, mode);
  if (mode == ATTN_DENSE)
    return block == 128 ? launch_t<128, ATTN_DENSE, 1, 1>(a, p, stream)
                        : launch_t<64, ATTN_DENSE, 2, 2>(a, p, stream);
  if (block == 64) {
    if (mode == ATTN_EXACT) return launch_t<64, ATTN_EXACT, 2, 4>(a, p, stream);
    if (p.kgs == 4) return launch_t<64, ATTN_BLOCK, 1, 4>(a, p, stream);
    return launch_t<64, ATTN_BLOCK, 1, 2>(a, p, stream);
  }
  if (mode == ATTN_EXACT) {
    if (p.kgs == 4) return launch_t<128, ATTN_EXACT, 1, 4>(a, p, stream);
    return launch_t<128, ATTN_EXACT, 1, 2>(a, p, stream);
  }
  if (p.kgs == 4) return launch_t<128, ATTN_BLOCK, 1, 4>(a, p, stream);
  return launch_t<128, ATTN_BLOCK, 1, 2>(a, p, stream);
}

}  // namespace lvsa
