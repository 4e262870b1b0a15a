// mask_device.hip -- LVSA mask builder on the GPU.
//
// Computes the same block CSR as the host builder (the LVSA frame sets of
// Sec. 2: Def. 2, Eq. 3, Alg. 1, expanded to blocks by the any-overlap rule)
// without a host round trip, so a denoising loop can rebuild the mask for
// step s on the stream that then runs attention.
//
// One launch.  What a row keeps has a closed form: the windows of a query
// block's frames each contain their own frame, so together they are one run of
// frames and its blocks one run [b0, b1] of key blocks; outside that run a key
// block is kept iff it touches an anchor frame or the text, the same for every
// row.  So every workgroup makes
//   - a table of the anchors below each frame and the windows of all frames
//     (Alg. 1, one frame per thread, the binary search on that table);
//   - a bitmap of the key blocks that touch an anchor or the text, and the
//     count of such blocks before each of its words,
// from which a row's length and the place of a kept block in its row are a few
// LDS reads.  Its rows start where the lengths of all rows before them add up
// to, which it sums itself; then it writes its rows, every thread its own key
// blocks.  The tables are small (a frame and a few key blocks per thread), so
// making them again in every workgroup costs less than a launch that would
// make them once: what bounds the builder is latency.  Wan 6x (1,475 blocks,
// 121 frames), block form then token-exact form: 167 us with three launches each
// (row lengths, scan, rows; every key block tested against every row, twice),
// 31 us now.
#include "internal.h"

namespace lvsa {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// Frames that two adjacent query blocks may touch (checked before launch): the
// interface's limit.  Nothing here is sized by it; one thread goes through a row's
// frames one by one (make_row), which is what such rows would cost.
constexpr int kMaxRowFrames = 1024;

// Key blocks: nb * nb fits in int32.
constexpr int kMaxBlocks = 46340;
constexpr int kMaxWords = (kMaxBlocks + 63) / 64;

// Rows per workgroup at most, and the number of workgroups aimed at (two per
// CU).
constexpr int kMaxRows = 128;
constexpr int kGroups = 512;
static_assert((kMaxBlocks + kGroups - 1) / kGroups <= kMaxRows, "rows per workgroup");

struct Tables {
  int16_t below[LVSA_MAX_FRAMES + 1];   // anchors among frames 0..f-1
  int16_t lo[LVSA_MAX_FRAMES];          // window of frame t
  int16_t hi[LVSA_MAX_FRAMES];
  uint64_t common[kMaxWords + 1];       // key blocks every row keeps
  int32_t rank[kMaxWords + 1];          // common blocks before word w
};

// One row: query segments f0..f1, the run of key blocks of their windows and
// the common blocks before it and up to its end, where the row starts.
struct Row {
  int32_t f0, f1, b0, b1, r0, r1, len;
};

// Common key blocks below b (0 <= b <= nb).
__device__ inline int32_t common_below(const Tables& tb, int32_t b) {
  const uint64_t w = tb.common[b / 64] & ((1ull << (b % 64)) - 1ull);
  return tb.rank[b / 64] + (int32_t)__popcll(w);
}

__device__ inline Row make_row(const Tables& tb, const FrameCfg& c, int32_t qb, int32_t P,
                               int32_t B, int32_t N, int32_t nb) {
  Row r;
  block_frame_range(qb, c.T, P, B, N, &r.f0, &r.f1);
  if (r.f1 == c.T) {   // text queries keep every block
    r.b0 = 0;
    r.b1 = nb - 1;
  } else {
    int32_t lo = tb.lo[r.f0], hi = tb.hi[r.f0];
    for (int32_t t = r.f0 + 1; t <= r.f1; ++t) {
      lo = imin(lo, tb.lo[t]);
      hi = imax(hi, tb.hi[t]);
    }
    r.b0 = lo * P / B;
    r.b1 = (hi * P + P - 1) / B;
  }
  r.r0 = common_below(tb, r.b0);
  r.r1 = common_below(tb, r.b1 + 1);
  r.len = (r.b1 - r.b0 + 1) + common_below(tb, nb) - (r.r1 - r.r0);
  return r;
}

// Sum over the workgroup, in every thread (`s_sum`: one word per wave).
__device__ inline int32_t block_sum(int32_t v, int32_t* s_sum) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if (threadIdx.x % 64 == 0) s_sum[threadIdx.x / 64] = v;
  __syncthreads();
  int32_t sum = 0;
  for (int w = 0; w < kWaves; ++w) sum += s_sum[w];
  return sum;
}

// Rows rows*g .. rows*g + rows - 1 of the mask (workgroup g); col_idx and
// entry may be null.
__global__ __launch_bounds__(kThreads) void build_rows_kernel(
    FrameCfg c, int32_t P, int32_t B, int32_t rows, int32_t* __restrict__ row_ptr,
    int32_t* __restrict__ col_idx, uint32_t* __restrict__ entry) {
  __shared__ Tables tb;
  __shared__ Row row[kMaxRows];
  __shared__ int32_t start[kMaxRows];
  __shared__ int32_t s_sum[kWaves];
  const int32_t tid = threadIdx.x, lane = tid % 64;
  const int32_t N = (int32_t)mask_tokens(c, P);
  const int32_t nb = ceil_div(N, B);
  const int32_t first = rows * (int32_t)blockIdx.x;
  const int32_t count = imin(rows, nb - first);

  for (int32_t f = tid; f <= c.T; f += kThreads) tb.below[f] = (int16_t)anchors_below(c, f);
  __syncthreads();
  for (int32_t t = tid; t < c.T; t += kThreads) {
    int32_t lo, hi;
    frame_window(c, t, [&](int32_t f) { return (int32_t)tb.below[f]; }, &lo, &hi);
    tb.lo[t] = (int16_t)lo;
    tb.hi[t] = (int16_t)hi;
  }
  const int32_t words = nb / 64 + 1;   // bit nb is in the last word
  for (int32_t base = 0; base < words * 64; base += kThreads) {
    const int32_t kb = base + tid;
    bool bit = false;
    if (kb < nb) {
      int32_t g0, g1;
      block_frame_range(kb, c.T, P, B, N, &g0, &g1);
      bit = g1 == c.T || tb.below[g1 + 1] > tb.below[g0];
    }
    const uint64_t bal = __ballot(bit);
    if (lane == 0 && kb / 64 < words) tb.common[kb / 64] = bal;
  }
  __syncthreads();
  if (tid < 64) {
    int32_t carry = 0;
    for (int32_t base = 0; base < words; base += 64) {
      const int32_t v = base + lane < words ? (int32_t)__popcll(tb.common[base + lane]) : 0;
      int32_t incl = v;
      for (int off = 1; off < 64; off <<= 1) {
        const int32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
      }
      if (base + lane < words) tb.rank[base + lane] = carry + incl - v;
      carry += __shfl(incl, 63);
    }
  }
  __syncthreads();

  int32_t before = 0;
  for (int32_t qb = tid; qb < first; qb += kThreads)
    before += make_row(tb, c, qb, P, B, N, nb).len;
  if (tid < count) row[tid] = make_row(tb, c, first + tid, P, B, N, nb);
  before = block_sum(before, s_sum);   // its barrier also covers row[]
  if (tid < count) {
    int32_t at = before;
    for (int32_t i = 0; i < tid; ++i) at += row[i].len;
    start[tid] = at;
    row_ptr[first + tid + 1] = at + row[tid].len;
    if (first + tid == 0) row_ptr[0] = 0;
  }
  __syncthreads();

  auto attends = [&](int32_t t, int32_t tau) {
    return t == c.T || tau == c.T || tb.below[tau + 1] > tb.below[tau] ||
           (tb.lo[t] <= tau && tau <= tb.hi[t]);
  };
  for (int32_t kb = tid; kb < nb; kb += kThreads) {
    const bool common = (tb.common[kb / 64] >> (kb % 64)) & 1ull;
    const int32_t rk = common_below(tb, kb);
    int32_t g0 = 0, g1 = 0;
    uint32_t kfirst = 0u;
    if (entry) key_block_split(kb, c.T, P, B, N, &g0, &g1, &kfirst);
    for (int32_t i = 0; i < count; ++i) {
      const Row r = row[i];
      const bool in_run = r.b0 <= kb && kb <= r.b1;
      if (!common && !in_run) continue;
      // Kept blocks of the row below kb.
      const int32_t at = start[i] + (kb < r.b0 ? rk
                                     : in_run  ? r.r0 + (kb - r.b0)
                                               : rk + (r.b1 - r.b0 + 1) - (r.r1 - r.r0));
      if (col_idx) col_idx[at] = kb;
      if (entry) entry[at] = exact_word(kb, g0, g1, kfirst, r.f0, r.f1, attends);
    }
  }
}

}  // namespace

bool device_mask_supported(const FrameCfg& c, int32_t P, int32_t B) {
  // A query-block pair touches at most min(T, 2B/P + 2) frames.
  return (int64_t)2 * B / P + 2 <= kMaxRowFrames || c.T <= kMaxRowFrames;
}

hipError_t launch_build_mask_device(const FrameCfg& c, int32_t P, int32_t B,
                                    int32_t* d_row_ptr, int32_t* d_col_idx,
                                    uint32_t* d_entry, hipStream_t stream) {
  const int32_t nb = (int32_t)((mask_tokens(c, P) + B - 1) / B);
  const int32_t rows = ceil_div(nb, kGroups);
  hipLaunchKernelGGL(build_rows_kernel, dim3(ceil_div(nb, rows)), dim3(kThreads), 0, stream, c, P,
                     B, rows, d_row_ptr, d_col_idx, d_entry);
  return hipGetLastError();
}

}  // namespace lvsa
