// Cache stage: per-page Mean / Max / Min key summaries (Sec. 3.1 Eq. 1; Sec. 3.2 Quest).
//
// Work decomposition: a task is 8 consecutive channels (16 bytes of bf16, 8 of fp8) of one
// (page, KV head) slice.  TS adjacent lanes share a task and take every TS-th valid token; quad DPP
// combines them (TS = 1 for a full pass over many pages, TS = 2 or 4 at a decode step where
// only one page per request changes).  Each lane loads up to 8 token rows per round trip (16 in a
// full pass, a whole page of 16).  A token row of a slice is D*2 contiguous bytes, so a load
// instruction reads whole rows of several slices.  HBM-bound: it reads page_size*D*2 bytes
// (page_size*D for an fp8 cache) and writes D*(4 + 2 + 2) bytes per (page, head).  A full pass
// streams both ways (non-temporal loads and stores), forms only the kinds of summary asked for and
// gives a workgroup one round of tasks, two in large launches over blocks of 16 (below): 16 prompts of
// 16k to 32k tokens on pages of 16, Mean and its bf16 copy (969 MB), 205 -> 189 us; 16 prompts of 131072
// tokens on pages of 32, Max and Min (4.6 GB), 967 -> 820 us.  (Of the first 16 us: wider batches and
// non-temporal loads 10, stores 6; with four rounds of tasks per workgroup 193 us, with sixteen 212.)
// fp8 caches: each code is converted exactly to fp32 and multiplied by the K scale (one fp32
// rounding), which is the cache value the summaries are taken over.
//
// Append mode (the decode step's cache stage fused into one launch): request i's new key and
// value rows are written at token L_i - 1, and the page holding it is summarised in the same
// pass.  The new key row is taken from the step's input, not read back, and enters the
// running sums last, exactly where a separate summarize pass over the page would add it, so
// the summaries are bit-identical to an append followed by vx_page_summarize.
//
// Blocks below the page size (r = ps / bs blocks per page): the unit is the block.  Logical
// block j of request i is block j % r of physical page indices[j / r], its summary row is
// (p * r + j % r), and every page count above is a block count.  r = 1 is the page case.
#include <type_traits>

#include "summary_task.h"
#include "vx_device.h"
#include "vx_internal.h"

namespace vx {
namespace {

constexpr int kThreads = 256;
using summ::AppendArgs;

template <int TS, int KT, bool APPEND, int KB, bool MEAN, bool ENV, bool STREAM>
__global__ __launch_bounds__(kThreads) void summarize_kernel(
    const void* __restrict__ kv, float k_scale, int num_phys, int H, int ps, int bs, int r, int D, int max_pages,
    const int32_t* __restrict__ indptr, const int32_t* __restrict__ indices,
    const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ first_page,
    float* __restrict__ mean, uint16_t* __restrict__ mean_bf, uint16_t* __restrict__ maxo,
    uint16_t* __restrict__ mino, int pages_per_block, int split_tasks, const AppendArgs app) {
  const int i = blockIdx.y;
  const int L = seq_lens[i];
  const int base = indptr[i];
  int P = num_pages(L, bs, (indptr[i + 1] - base) * r, max_pages);     // blocks
  int j0 = first_page ? first_page[i] : 0;
  if constexpr (APPEND) {
    j0 = (L - 1) / bs;                   // the block receiving token L - 1, and only that one
    P = min(P, j0 + 1);
  }
  j0 = j0 < 0 ? 0 : j0;
  const int chunks = D / 8;
  const int tasks_per_page = H * chunks;

  static_assert(TS == 1 || TS == 2 || TS == 4, "token slices per task");
  const int slice = (int)threadIdx.x % TS;
  // Decode-step launches (split_tasks): the x workgroups of a request share out the tasks of
  // each page from j0 on.  Full passes: workgroup x takes pages x*pages_per_block.. with stride.
  const int x_pg = split_tasks ? 0 : (int)blockIdx.x, n_pg = split_tasks ? 1 : (int)gridDim.x;
  const int t_first = split_tasks ? (int)blockIdx.x * (kThreads / TS) : 0;
  const int t_step = split_tasks ? (int)gridDim.x * (kThreads / TS) : kThreads / TS;
  for (int jb = j0 + x_pg * pages_per_block; jb < P; jb += n_pg * pages_per_block) {
    const int nj = min(pages_per_block, P - jb);
    const int ntask = nj * tasks_per_page;
    // t0 is uniform over the workgroup: every lane of a quad runs the same task count, so the
    // DPP combine sees full quads
    for (int t0 = t_first; t0 < ntask; t0 += t_step) {
      const int task = t0 + (int)threadIdx.x / TS;
      const bool active = task < ntask;
      const int tk = active ? task : 0;
      const int jj = tk / tasks_per_page;
      const int rem = tk - jj * tasks_per_page;
      const int h = rem / chunks;
      const int c8 = rem - h * chunks;
      const int j = jb + jj;                              // logical block
      summ::task<TS, KT, APPEND, KB, MEAN, ENV, STREAM>(kv, k_scale, num_phys, H, ps, bs, r, D, indices, base, L, i, j,
                                                        h, c8, active, slice, mean, mean_bf, maxo, mino, app);
    }
  }
}

// Workgroups per request at a decode step: one per 64 tasks (8-channel chunks of a page's
// heads), so each of a task's 4 lanes walks at most page_size / 4 token rows.
int step_wgs(const Geometry& g) {
  const int tasks_per_page = g.H * (g.Dqk / 8);
  return (tasks_per_page + kThreads / 4 - 1) / (kThreads / 4);
}

template <int TS, bool APPEND = false, int KB = summ::kBatch, bool MEAN = true, bool ENV = true,
          bool STREAM = TS == 1>
void dispatch(const Geometry& g, const int32_t* first_page, float* mean, uint16_t* mean_bf, uint16_t* maxo,
              uint16_t* mino, dim3 grid, int ppb, int split, hipStream_t stream, const AppendArgs& app = AppendArgs{}) {
#define VX_SUMMARIZE(KT)                                                                                        \
  hipLaunchKernelGGL((summarize_kernel<TS, KT, APPEND, KB, MEAN, ENV, STREAM>), grid, dim3(kThreads), 0, stream, g.k, g.k_scale, \
                     g.num_phys_pages, g.H, g.ps, g.bs, g.r, g.Dqk, g.max_pages, g.indptr, g.indices, g.seq_lens,  \
                     first_page,                                                                                 \
                     mean, mean_bf, maxo, mino, ppb, split, app)
  if (g.kv_dtype == kKvFp8E4M3) VX_SUMMARIZE(kKvFp8E4M3);
  else if (g.kv_dtype == kKvFp8E5M2) VX_SUMMARIZE(kKvFp8E5M2);
  else VX_SUMMARIZE(kKvBf16);
#undef VX_SUMMARIZE
}

}  // namespace

hipError_t launch_summarize(const Geometry& g, const int32_t* first_page, float* mean, uint16_t* mean_bf,
                            uint16_t* maxo, uint16_t* mino, hipStream_t stream) {
  if (g.batch == 0) return hipSuccess;
  const int tasks_per_page = g.H * (g.Dqk / 8);
  if (first_page) {
    // decode step: usually one new page per request, whose tasks are shared out over
    // step_wgs() workgroups of the request, 4 lanes per task splitting its tokens
    if (g.bs > 4 * summ::kBatch)   // blocks of 64 tokens: a lane's 16 rows in one round trip
      dispatch<4, false, 2 * summ::kBatch>(g, first_page, mean, mean_bf, maxo, mino, dim3(step_wgs(g), g.batch), 1,
                                           1, stream);
    else
      dispatch<4>(g, first_page, mean, mean_bf, maxo, mino, dim3(step_wgs(g), g.batch), 1, 1, stream);
  } else {
    // Blocks of 16 tokens are one round trip per task.  Once a launch is many rounds of workgroups
    // deep, two rounds of tasks per workgroup halve what each spends on its request's geometry (and
    // the workgroups past the ends of short requests); a small launch needs the workgroups, and a
    // bf16 Mean's stores keep them busy.  us at one / two rounds, by workgroups of one round per CU: 64
    // (16 prompts of 16k to 32k tokens) E4M3 Mean 129.7 / 121.1, envelope 116.1 / 109.9, bf16 Max 176.2 /
    // 173.0, envelope 184.2 / 182.9, Mean 189.6 / 193.0; 128 (16 of 4k to 64k, lognormal) E4M3 Mean 120.7 /
    // 107.5, bf16 Max 153.9 / 149.3, Mean 162.4 / 164.6; 32 (32 of 1k to 8k, lognormal) E4M3 Mean 38.9 / 39.7,
    // bf16 Max 48.0 / 49.5; 16 (64 of 256 to 2048) 30.6 / 34.7, 35.0 / 39.2.  Blocks of 64, E4M3 89.0 / 93.9.
    const int ppb1 = tasks_per_page >= kThreads ? 1 : kThreads / tasks_per_page;
    const long long wgs = ((long long)g.max_pages + ppb1 - 1) / ppb1 * g.batch;
    const bool two = g.bs <= 16 && (g.kv_dtype != kKvBf16 || (!mean && !mean_bf)) && wgs >= 48LL * device_cus();
    const int ppb = two ? 2 * ppb1 : ppb1;
    int gx = (g.max_pages + ppb - 1) / ppb;
    if (gx < 1) gx = 1;
    // a score kind reads the Mean or the Max / Min, so most callers ask for one of the two
    const dim3 grid(gx, g.batch);
    constexpr int KB = 2 * summ::kBatch;
    auto pass = [&](auto stream_loads) {
      constexpr bool S = decltype(stream_loads)::value;
      if (!maxo && !mino)
        dispatch<1, false, KB, true, false, S>(g, first_page, mean, mean_bf, maxo, mino, grid, ppb, 0, stream);
      else if (!mean && !mean_bf)
        dispatch<1, false, KB, false, true, S>(g, first_page, mean, mean_bf, maxo, mino, grid, ppb, 0, stream);
      else dispatch<1, false, KB, true, true, S>(g, first_page, mean, mean_bf, maxo, mino, grid, ppb, 0, stream);
    };
    // A token row shorter than a cache line (fp8 at 64 channels) shares its line with the next row's
    // load, which the non-temporal hint may fetch again: 32 prompts of 8k to 32k tokens, 2 KV heads,
    // E4M3 Mean 33.6 us with the hint, 30.9 without; with whole lines (128 channels) 126.1 / 129.9.
    if (g.Dqk * (g.kv_dtype == kKvBf16 ? 2 : 1) < 128) pass(std::false_type{});
    else pass(std::true_type{});
  }
  return hipGetLastError();
}

hipError_t launch_kv_append_summarize(const Geometry& g, const void* k_new, const void* v_new, float* mean,
                                      uint16_t* mean_bf, uint16_t* maxo, uint16_t* mino, hipStream_t stream) {
  if (g.batch == 0) return hipSuccess;
  const AppendArgs app{k_new, v_new, const_cast<void*>(g.k), const_cast<void*>(g.v)};
  // the launch shape of the decode step's incremental summary (same token slices, so the
  // summaries come out bit-identical)
  if (g.bs > 4 * summ::kBatch)     // blocks of 64 tokens: a lane's 16 rows in one round trip
    dispatch<4, true, 2 * summ::kBatch>(g, nullptr, mean, mean_bf, maxo, mino, dim3(step_wgs(g), g.batch), 1, 1,
                                        stream, app);
  else
    dispatch<4, true>(g, nullptr, mean, mean_bf, maxo, mino, dim3(step_wgs(g), g.batch), 1, 1, stream, app);
  return hipGetLastError();
}

}  // namespace vx
