// Batched estimation: many (graph, k, budget, seed) requests drained by one
// persistent kernel launch.
#include "batch.h"

#include <algorithm>
#include <chrono>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>

namespace moss {

namespace {
std::mutex g_tune_mu;
Tuning g_tuning;

std::mutex g_runner_mu;
std::map<int, std::unique_ptr<BatchRunner>> g_runners;

constexpr uint32_t kDefaultTile = 4096;

// Resident waves per CU of the persistent kernel.  Its tiles are drawn in lane order, so
// more waves hide latency on large graphs too: 12 / 16 / 20 / 24 / 28 waves on 256
// requests over 32 graphs (m to 5e6) 19.4 / 18.5 / 18.5 / 18.5 / 18.6 ms, on 64 requests over
// 8 graphs (m to 3e5) 1.78 / 1.64 / 1.58 / 1.57 / 1.56 ms, on 40 over 6 (m from 1e6 to
// 8e6) 8.67 / 8.28 / 8.50 / 8.55 / 8.68 ms.
constexpr int kBatchWaves = 24;

// Batched items drawn by grouped launches of their own: at least 2^18 samples on a graph
// whose sampled bytes are past 32 MB (the tuning's schedule overrides: PLAIN never, XCD
// always).  At 24 waves, from 2^17 / 2^18 / 2^19 / 2^20 samples: 18.24 / 18.30 / 18.34 /
// 18.48 ms on the first of those batches, 8.03 / 8.04 / 8.18 / 8.55 ms on the last; from 16
// or 64 MB on no faster.
constexpr uint64_t kBatchSortMinSamples = 1ull << 18;
constexpr uint64_t kBatchSortMinFootprint = 32ull << 20;
constexpr uint64_t kBatchSortChunk = 1ull << 25;

bool batch_sorted(const moss_graph* g, uint64_t n, const Tuning& t) {
  if (t.schedule == MOSS_SCHEDULE_PLAIN) return false;
  if (t.schedule == MOSS_SCHEDULE_XCD) return n > 0;
  const uint64_t min_n = t.group_min_samples_log2 ? 1ull << t.group_min_samples_log2 : kBatchSortMinSamples;
  const uint64_t min_fp = t.group_min_footprint_mb ? (uint64_t)t.group_min_footprint_mb << 20 : kBatchSortMinFootprint;
  return n >= min_n && sampling_footprint(g) >= min_fp;
}
}  // namespace

Tuning current_tuning() {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  return g_tuning;
}

uint32_t sort_window_for(const moss_graph* g) {
  const uint32_t w = current_tuning().sort_window;
  return w ? w : sort_window(sampling_footprint(g));
}

BatchRunner* batch_runner(int device) {
  std::lock_guard<std::mutex> lk(g_runner_mu);
  auto it = g_runners.find(device);
  if (it != g_runners.end()) return it->second.get();
  auto r = std::make_unique<BatchRunner>(device);
  BatchRunner* p = r.get();
  g_runners[device] = std::move(r);
  return p;
}

void result_header(const moss_graph* g, int32_t k, uint64_t n_samples, uint32_t flags, moss_result* r) {
  std::memset(r, 0, sizeof(*r));
  r->k = k;
  r->flags = flags;
  r->n_samples = n_samples;
  EstimatePlan plan;
  (void)plan_estimate(k, n_samples, flags, &plan);  // callers checked the request
  r->K[0] = plan.K[0];
  r->K[1] = plan.K[1];
  if (k == 4) {
    r->n_motifs = 6;
    r->gamma[0] = g->total[0];
    r->gamma[1] = plan.count == 2 ? g->total[3] : 0;
    r->lambda = g->lambda3;
  } else {
    r->n_motifs = 21;
    r->gamma[0] = g->total[1];
    r->gamma[1] = g->total[2];
    r->lambda = g->lambda4;
  }
}

BatchRunner::BatchRunner(int device) : device_(device) {}

BatchRunner::~BatchRunner() {
  // The per-device runners live until process exit, when the runtime may already be
  // gone; owners that end earlier (servers) call release() first.
}

void BatchRunner::release() {
  DeviceScope scope(device_);
  if (stream_) (void)hipStreamSynchronize(stream_);
  if (d_in_) (void)hipFree(d_in_);
  if (d_bins_) (void)hipFree(d_bins_);
  if (d_end_) (void)hipFree(d_end_);
  d_in_ = nullptr;
  d_bins_ = nullptr;
  d_end_ = nullptr;
  cap_in_ = cap_slots_ = 0;
  if (h_in_) (void)hipHostFree(h_in_);
  if (h_bins_) (void)hipHostFree(h_bins_);
  h_in_ = nullptr;
  h_bins_ = nullptr;
  if (ev_wait_) (void)hipEventDestroy(ev_wait_);
  if (ev_clear_) (void)hipEventDestroy(ev_clear_);
  for (int j = 0; j < 2; ++j) {
    if (ev_side_[j]) (void)hipEventDestroy(ev_side_[j]);
    ev_side_[j] = nullptr;
    if (side_[j]) {
      (void)hipStreamSynchronize(side_[j]);
      (void)hipStreamDestroy(side_[j]);
    }
    side_[j] = nullptr;
  }
  ev_wait_ = ev_clear_ = nullptr;
  if (stream_) (void)hipStreamDestroy(stream_);
  stream_ = nullptr;
}

// Room for `bytes` of views, items and control words and for `slots` histogram slots, on
// the device and in pinned host memory.
moss_status BatchRunner::reserve(size_t bytes, size_t slots) {
  auto device = [](auto** p, size_t size) {
    if (*p) (void)hipFree((void*)*p);
    *p = nullptr;
    return hipMalloc((void**)p, size) == hipSuccess || (*p = nullptr);
  };
  auto host = [](auto** p, size_t size) {
    if (*p) (void)hipHostFree((void*)*p);
    *p = nullptr;
    return hipHostMalloc((void**)p, size, hipHostMallocDefault) == hipSuccess || (*p = nullptr);
  };
  if (!d_end_ && !device(&d_end_, 2 * sizeof(unsigned long long))) return MOSS_E_NOMEM;
  if (bytes > cap_in_) {
    const size_t c = std::max<size_t>({bytes, 2 * cap_in_, 64 << 10});
    cap_in_ = 0;
    if (!device(&d_in_, c) || !host(&h_in_, c)) return MOSS_E_NOMEM;
    cap_in_ = c;
  }
  if (slots > cap_slots_) {
    const size_t c = std::max<size_t>({slots, 2 * cap_slots_, 512});
    cap_slots_ = 0;
    if (!device(&d_bins_, c * 22 * sizeof(unsigned long long)) ||
        !host(&h_bins_, (kBatchHostWords + c * 22) * sizeof(uint64_t)))
      return MOSS_E_NOMEM;
    cap_slots_ = c;
  }
  return MOSS_OK;
}

moss_status BatchRunner::run(const std::vector<WorkItem>& work, uint32_t n_slots, uint64_t* bins_out,
                             double* device_ms, hipStream_t wait_on, uint32_t tile_samples, uint32_t blocks_per_cu,
                             bool sort_large) {
  DeviceScope scope(device_);
  if (!scope.ok()) return MOSS_E_DEVICE;
  if (!stream_) {
    if (hipStreamCreateWithFlags(&stream_, hipStreamNonBlocking) != hipSuccess) return MOSS_E_DEVICE;
    if (hipEventCreateWithFlags(&ev_wait_, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ev_clear_, hipEventDisableTiming) != hipSuccess)
      return MOSS_E_DEVICE;
  }
  const Tuning tune = current_tuning();
  uint32_t T = tile_samples ? tile_samples : (tune.tile_samples ? tune.tile_samples : kDefaultTile);
  const int block = tune.threads_per_block ? (int)tune.threads_per_block : 256;
  int bpc = blocks_per_cu ? (int)blocks_per_cu : (int)tune.blocks_per_cu;
  if (bpc == 0) bpc = std::max(1, std::min(kBatchWaves / (block / 64), sample_kernel_blocks_per_cu(0, block)));
  const int grid = device_cus(device_) * bpc;

  // views: one per distinct (graph, sampler)
  std::vector<SamplerView> views;
  std::vector<const moss_graph*> view_graph;  // the graph of each view
  std::map<std::pair<const moss_graph*, int>, uint32_t> view_of;
  std::vector<BatchItem> items;
  std::vector<uint64_t> item_cost;
  // large items on large graphs run as grouped launches of their own (the plain path's
  // grouping passes and sorted sampling kernel, in two chains of chunks, each chain one
  // chunk at a time through a scratch block of its own), adding into their histogram slots
  struct SortChunk {
    int sampler;
    uint64_t seed, a, n;
    uint32_t slot, window;
    int grid, block;
    SamplerView view;
  };
  std::vector<SortChunk> chunks;
  uint64_t max_chunk = 0;
  for (const WorkItem& w : work) {
    if (!sort_large || w.k1 <= w.k0 || w.g->total[sampler_slot(w.sampler)] == 0) continue;
    if (!batch_sorted(w.g, w.k1 - w.k0, tune)) continue;
    const SamplerView view = sampler_view(w.g, w.sampler);
    const uint32_t window = sort_window_for(w.g);
    for (uint64_t a = w.k0; a < w.k1; a += kBatchSortChunk) {
      const uint64_t n = std::min<uint64_t>(kBatchSortChunk, w.k1 - a);
      SortChunk c{w.sampler, w.seed, a, n, w.slot, window, 0, 0, view};
      grouped_launch_shape(w.g, w.sampler, n, &c.grid, &c.block);
      chunks.push_back(c);
      max_chunk = std::max(max_chunk, n);
    }
  }
  // the costliest chunks first (samples times the Philox blocks a sample of the sampler
  // takes), each to the chain with less cost so far: the two chains then end together
  // (in request order by samples, one ended 0.8 ms after the other; 20.19 -> 19.91 ms on
  // a 256-request batch)
  auto chunk_cost = [](const SortChunk& c) {
    return c.n * ((c.sampler == kMoss4 || c.sampler == kMoss4Min) ? 2u : 3u);
  };
  std::stable_sort(chunks.begin(), chunks.end(),
                   [&](const SortChunk& x, const SortChunk& y) { return chunk_cost(x) > chunk_cost(y); });
  void* sort_scratch_block[2] = {nullptr, nullptr};
  struct Release {  // the blocks go back to the cache once the stream's work has finished
    hipStream_t s;
    void* (&a)[2];
    ~Release() {
      if (!a[0] && !a[1]) return;
      (void)hipStreamSynchronize(s);
      for (void*& p : a) device_block_free(s, p);
    }
  } release{stream_, sort_scratch_block};
  const int chains = chunks.size() > 1 ? 2 : 1;
  // the side streams exist once a run has needed them (a process holds few hardware
  // queues, and streams beyond them share one, so a runner without grouped launches,
  // such as the server's express path, keeps to its one stream)
  for (int j = 0; j < (chunks.empty() ? 0 : chains); ++j) {
    if (!side_[j] && hipStreamCreateWithFlags(&side_[j], hipStreamNonBlocking) != hipSuccess) {
      side_[j] = nullptr;
      return MOSS_E_DEVICE;
    }
    if (!ev_side_[j] && hipEventCreateWithFlags(&ev_side_[j], hipEventDisableTiming) != hipSuccess) {
      ev_side_[j] = nullptr;
      return MOSS_E_DEVICE;
    }
  }
  for (int j = 0; j < chains && max_chunk > 0; ++j)
    if (device_block_alloc(stream_, &sort_scratch_block[j], (size_t)grouped_scratch_bytes(max_chunk)) != MOSS_OK)
      return MOSS_E_NOMEM;
  for (const WorkItem& w : work) {
    if (w.k1 <= w.k0 || w.g->total[sampler_slot(w.sampler)] == 0) continue;
    if (sort_large && batch_sorted(w.g, w.k1 - w.k0, tune)) continue;  // a grouped launch
    auto key = std::make_pair((const moss_graph*)w.g, w.sampler);
    auto it = view_of.find(key);
    uint32_t vi;
    if (it == view_of.end()) {
      vi = (uint32_t)views.size();
      views.push_back(sampler_view(w.g, w.sampler));
      view_graph.push_back(w.g);
      view_of[key] = vi;
    } else {
      vi = it->second;
    }
    BatchItem b{};
    b.view = vi;
    b.sampler = (uint32_t)w.sampler;
    b.out = w.slot;
    b.seed = w.seed;
    b.k0 = w.k0;
    b.k1 = w.k1;
    items.push_back(b);
    item_cost.push_back((w.k1 - w.k0) * ((w.sampler == kMoss4 || w.sampler == kMoss4Min) ? 2 : 3));
  }
  // Graph-major order: the items of one (graph, sampler) view run together, so at any
  // moment the chip works on one graph's tables and they stay in L2 and the MALL
  // (interleaving the graphs of a batch measured about 15% slower per sample).  The
  // views of the graphs with the largest sampled footprint go first, then those with
  // the most work, and the largest items first within a view (256 requests over 32
  // graphs: largest footprint / most work / smallest footprint first 18.84 / 18.72 / 18.80
  // ms, no more apart than the runs of one).  The kernel cuts each item into tiles itself; the host hands over the
  // item list only.
  std::vector<uint64_t> view_cost(views.size(), 0), view_fp(views.size(), 0);
  for (size_t i = 0; i < items.size(); ++i) view_cost[items[i].view] += item_cost[i];
  for (size_t vi = 0; vi < views.size(); ++vi) view_fp[vi] = sampling_footprint(view_graph[vi]);
  std::vector<size_t> order(items.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) {
    const uint32_t vx = items[x].view, vy = items[y].view;
    if (vx != vy) {
      if (view_fp[vx] != view_fp[vy]) return view_fp[vx] > view_fp[vy];
      return view_cost[vx] != view_cost[vy] ? view_cost[vx] > view_cost[vy] : vx < vy;
    }
    return item_cost[x] > item_cost[y];
  });
  // A batch too small to give every block of the grid a tile gets smaller tiles (a
  // multiple of the block's threads, about its samples over the blocks): otherwise a
  // few blocks draw their lanes' samples one after another while the rest idle, and
  // a 10^4-sample request took 0.1-0.2 ms of kernel time instead of a few tens of µs.
  // The tiling does not change which samples are drawn, only which lanes draw them.
  uint64_t persistent = 0, tiles_at_T = 0;
  for (const BatchItem& b : items) {
    persistent += b.k1 - b.k0;
    tiles_at_T += (b.k1 - b.k0 + T - 1) / T;
  }
  if (tiles_at_T < (uint64_t)grid) {
    const uint64_t per_block = (persistent + (uint64_t)grid - 1) / (uint64_t)grid;
    const uint64_t t = std::max<uint64_t>((uint64_t)block, (per_block + block - 1) / block * block);
    if (t < T) T = (uint32_t)t;
  }
  uint64_t n_tiles = 0;
  for (size_t i : order) {
    items[i].first_tile = (uint32_t)n_tiles;
    n_tiles += (items[i].k1 - items[i].k0 + T - 1) / T;
    if (n_tiles >= 0xFFFFFFFFull) return MOSS_E_ARG;
  }
  // views | items | control words, staged in pinned memory in one piece
  auto pad = [](size_t n) { return (n + 15) / 16 * 16; };
  const size_t items_at = pad(views.size() * sizeof(SamplerView));
  const size_t ctl_at = items_at + pad(items.size() * sizeof(BatchItem)), bytes = ctl_at + pad(4 * sizeof(uint32_t));
  const uint64_t words = (uint64_t)n_slots * 22;
  moss_status st = reserve(bytes, n_slots);
  if (st != MOSS_OK) return st;
  std::memcpy(h_in_, views.data(), views.size() * sizeof(SamplerView));
  BatchItem* ip = (BatchItem*)(h_in_ + items_at);
  for (size_t i = 0; i < order.size(); ++i) ip[i] = items[order[i]];
  uint32_t* np = (uint32_t*)(h_in_ + ctl_at);
  np[kCtlTiles] = (uint32_t)n_tiles;
  np[kCtlCounter] = 0;
  np[kCtlItems] = (uint32_t)items.size();
  np[kCtlTileSize] = T;
  auto* host = (unsigned long long*)h_bins_;
  host[kBatchHostSeq] = 0;  // no launch of an earlier run still writes here
  const uint64_t seq = ++seq_;

  hipError_t e = hipSuccess;
  if (wait_on) {
    e = hipEventRecord(ev_wait_, wait_on);
    if (e == hipSuccess) e = hipStreamWaitEvent(stream_, ev_wait_, 0);
  }
  if (e == hipSuccess) e = launch_batch_stage(h_in_, d_in_, bytes, d_bins_, words, d_end_, stream_);
  // the grouped launches go to the side streams, free to start from the clear on.  They do
  // not run beside the persistent kernel, though: their first pass has blocks of 1024
  // threads, four wave places on every SIMD of a CU, of which the persistent kernel holds
  // six of eight until its list is drained.  So the two chains follow it and overlap one
  // another only; each chunk goes to the chain with less cost so far.  With one chain 256
  // requests over 32 graphs take 20.6 ms instead of 18.8, 40 over 6 7.45 instead of 6.32.
  const int side = chunks.empty() ? 0 : chains;
  if (e == hipSuccess && side) e = hipEventRecord(ev_clear_, stream_);
  for (int j = 0; j < side && e == hipSuccess; ++j) e = hipStreamWaitEvent(side_[j], ev_clear_, 0);
  if (e == hipSuccess && n_tiles > 0)
    e = launch_batch((const SamplerView*)d_in_, (const BatchItem*)(d_in_ + items_at), (uint32_t*)(d_in_ + ctl_at),
                     d_bins_, (int)std::min<uint64_t>((uint64_t)grid, n_tiles), block, stream_);
  uint64_t load[2] = {0, 0};
  for (const SortChunk& c : chunks) {
    if (e != hipSuccess) break;
    const int j = chains == 2 && load[1] < load[0] ? 1 : 0;
    load[j] += chunk_cost(c);
    const GroupChunk one{c.sampler, c.seed, c.a, c.n, sort_scratch_block[j], max_chunk};
    e = launch_group_chunks(&one, 1, nullptr, side_[j]);
    HitSink sink{};
    sink.add = d_bins_ + (uint64_t)c.slot * 22;
    if (e == hipSuccess)
      e = launch_sample_chunk(c.sampler, c.view, c.seed, c.a, c.n, sort_scratch_block[j], max_chunk, c.window, sink,
                              nullptr, c.grid, c.block, side_[j]);
  }
  for (int j = 0; j < side && e == hipSuccess; ++j) {
    e = hipEventRecord(ev_side_[j], side_[j]);
    if (e == hipSuccess) e = hipStreamWaitEvent(stream_, ev_side_[j], 0);
  }
  if (e == hipSuccess) e = launch_batch_collect(d_bins_, words, d_end_, host, seq, stream_);
  // the slots are in host memory once the sequence number is
  bool there = false;
  if (e == hipSuccess) {
    const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(1);
    do {
      for (int i = 0; i < 64 && !there; ++i) there = __atomic_load_n(&host[kBatchHostSeq], __ATOMIC_ACQUIRE) == seq;
    } while (!there && std::chrono::steady_clock::now() < until);
  }
  if (!there) {
    if (e == hipSuccess) e = hipStreamSynchronize(stream_);
    there = e == hipSuccess && __atomic_load_n(&host[kBatchHostSeq], __ATOMIC_ACQUIRE) == seq;
  }
  if (!there) {  // nothing of this batch left running
    (void)hipStreamSynchronize(stream_);
    for (int j = 0; j < side; ++j) (void)hipStreamSynchronize(side_[j]);
    return e == hipSuccess ? MOSS_E_DEVICE : status_of(e);
  }
  std::memcpy(bins_out, host + kBatchHostWords, (size_t)words * sizeof(uint64_t));
  if (device_ms) *device_ms = (double)host[kBatchHostTicks] / device_ticks_per_ms(device_);
  return MOSS_OK;
}

namespace {

std::mutex g_batch_mu;  // one batch at a time per process (the runner is shared)

moss_status batch_impl(const moss_request* reqs, int32_t n, moss_result* out, hipStream_t wait_on,
                       uint32_t tile_samples, uint32_t blocks_per_cu, double* device_ms) {
  if (n < 0 || (n > 0 && (!reqs || !out))) return MOSS_E_ARG;
  if (n == 0) return MOSS_OK;
  const int device = reqs[0].g ? reqs[0].g->device : -1;
  for (int32_t i = 0; i < n; ++i) {
    const moss_request& q = reqs[i];
    EstimatePlan plan;
    if (!q.g || q.g->device != device || plan_estimate(q.k, q.n_samples, q.flags, &plan) != MOSS_OK)
      return MOSS_E_ARG;
  }
  // build missing tables (each graph once)
  for (int32_t i = 0; i < n; ++i) {
    moss_graph* g = reqs[i].g;
    EstimatePlan plan;
    (void)plan_estimate(reqs[i].k, reqs[i].n_samples, reqs[i].flags, &plan);
    const uint32_t mask = plan.tables;
    if ((g->built & mask) == mask) continue;
    GraphClaim claim(g);
    if (!claim.ok()) return MOSS_E_BUSY;
    moss_status st = build_tables(g, mask);
    if (st != MOSS_OK) return st;
  }
  std::vector<WorkItem> work;
  work.reserve((size_t)n * 2);
  for (int32_t i = 0; i < n; ++i) {
    const moss_request& q = reqs[i];
    moss_result& r = out[i];
    result_header(q.g, q.k, q.n_samples, q.flags, &r);
    EstimatePlan plan;
    (void)plan_estimate(q.k, q.n_samples, q.flags, &plan);
    for (int s = 0; s < plan.count; ++s)
      work.push_back({q.g, plan.sampler[s], q.seed, 0, plan.K[s], (uint32_t)(2 * i + s)});
  }
  std::vector<uint64_t> bins((size_t)n * 2 * 22);
  std::lock_guard<std::mutex> lk(g_batch_mu);
  BatchRunner* runner = batch_runner(device);
  double ms = 0.0;
  moss_status st =
      runner->run(work, (uint32_t)(2 * n), bins.data(), &ms, wait_on, tile_samples, blocks_per_cu, true);
  if (st != MOSS_OK) return st;
  for (int32_t i = 0; i < n; ++i) {
    moss_result& r = out[i];
    std::memcpy(r.hits[0], &bins[(size_t)(2 * i) * 22], 22 * sizeof(uint64_t));
    std::memcpy(r.hits[1], &bins[(size_t)(2 * i + 1) * 22], 22 * sizeof(uint64_t));
    r.device_ms = ms;
    st = moss_finals(&r);
    if (st != MOSS_OK) return st;
  }
  if (device_ms) *device_ms = ms;
  return MOSS_OK;
}

}  // namespace
}  // namespace moss

using namespace moss;

extern "C" {

moss_status moss_estimate_batch(const moss_request* reqs, int32_t n, moss_result* out, void* hip_stream) {
  return batch_impl(reqs, n, out, (hipStream_t)hip_stream, 0, 0, nullptr);
}

moss_status moss_set_tuning(const moss_tuning* t) {
  if (!t) return MOSS_E_ARG;
  if (t->threads_per_block && (t->threads_per_block % 64 != 0 || t->threads_per_block > 256)) return MOSS_E_ARG;
  if (t->blocks_per_cu > 64 || t->schedule > MOSS_SCHEDULE_XCD) return MOSS_E_ARG;
  if (t->group_min_samples_log2 > 40 || t->group_min_footprint_mb > (1u << 20)) return MOSS_E_ARG;
  if (t->sort_window % 64 != 0 || t->sort_window > 512) return MOSS_E_ARG;
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tuning.tile_samples = t->tile_samples;
  g_tuning.blocks_per_cu = t->blocks_per_cu;
  g_tuning.threads_per_block = t->threads_per_block;
  g_tuning.schedule = t->schedule;
  g_tuning.group_min_samples_log2 = t->group_min_samples_log2;
  g_tuning.group_min_footprint_mb = t->group_min_footprint_mb;
  g_tuning.sort_window = t->sort_window;
  return MOSS_OK;
}

moss_status moss_get_tuning(moss_tuning* t) {
  if (!t) return MOSS_E_ARG;
  std::lock_guard<std::mutex> lk(g_tune_mu);
  t->tile_samples = g_tuning.tile_samples;
  t->blocks_per_cu = g_tuning.blocks_per_cu;
  t->threads_per_block = g_tuning.threads_per_block;
  t->schedule = g_tuning.schedule;
  t->group_min_samples_log2 = g_tuning.group_min_samples_log2;
  t->group_min_footprint_mb = g_tuning.group_min_footprint_mb;
  t->sort_window = g_tuning.sort_window;
  return MOSS_OK;
}

moss_status moss_autotune(const moss_request* reqs, int32_t n, moss_tuning* best, double* best_ms) {
  if (!reqs || n <= 0 || !best) return MOSS_E_ARG;
  static const uint32_t kTiles[] = {2048, 4096, 16384, 65536};
  static const uint32_t kBpc[] = {2, 3, 4, 5, 6, 8};
  static const uint32_t kGroupLog2[] = {17, 18, 19, 20, 21, 22};
  static const uint32_t kGroupMb[] = {4, 8, 16, 32, 64};
  static const uint32_t kWindows[] = {128, 256, 512};
  const moss_tuning before = [] {
    moss_tuning t{};
    (void)moss_get_tuning(&t);
    return t;
  }();
  std::vector<moss_result> ref((size_t)n), cur((size_t)n);
  moss_status st = batch_impl(reqs, n, ref.data(), nullptr, kDefaultTile, 4, nullptr);  // warm-up, reference
  if (st != MOSS_OK) return st;
  // the whole call, best of two (host time included: item list, staging, copies)
  auto timed = [&](uint32_t T, uint32_t bpc, double* ms) -> moss_status {
    *ms = 1e300;
    for (int rep = 0; rep < 2; ++rep) {
      const auto t0 = std::chrono::steady_clock::now();
      moss_status s = batch_impl(reqs, n, cur.data(), nullptr, T, bpc, nullptr);
      const double t = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
      if (s != MOSS_OK) return s;
      for (int32_t i = 0; i < n; ++i)
        if (std::memcmp(cur[i].hits, ref[i].hits, sizeof(ref[i].hits)) != 0) return MOSS_E_DEVICE;
      *ms = std::min(*ms, t);
    }
    return MOSS_OK;
  };
  double best_t = 1e300;
  moss_tuning b = before;
  b.threads_per_block = 256;
  // 1. tile size and occupancy of the persistent kernel, at the default grouping
  moss_tuning c = b;
  c.group_min_samples_log2 = c.group_min_footprint_mb = c.sort_window = 0;
  for (uint32_t T : kTiles) {
    for (uint32_t bpc : kBpc) {
      c.tile_samples = T;
      c.blocks_per_cu = bpc;
      if ((st = moss_set_tuning(&c)) != MOSS_OK) break;
      double ms;
      if ((st = timed(T, bpc, &ms)) != MOSS_OK) break;
      if (ms < best_t) {
        best_t = ms;
        b = c;
      }
    }
    if (st != MOSS_OK) break;
  }
  // 2. which items leave the persistent kernel for grouped launches of their own: the
  // fewest samples per item and the smallest sampled footprint of its graph
  for (uint32_t lg : kGroupLog2) {
    if (st != MOSS_OK) break;
    for (uint32_t mb : kGroupMb) {
      c = b;
      c.group_min_samples_log2 = lg;
      c.group_min_footprint_mb = mb;
      if ((st = moss_set_tuning(&c)) != MOSS_OK) break;
      double ms;
      if ((st = timed(c.tile_samples, c.blocks_per_cu, &ms)) != MOSS_OK) break;
      if (ms < best_t) {
        best_t = ms;
        b = c;
      }
    }
  }
  // 3. the window of the grouped launches' sorted kernel (by footprint, or fixed)
  for (uint32_t w : kWindows) {
    if (st != MOSS_OK) break;
    c = b;
    c.sort_window = w;
    if ((st = moss_set_tuning(&c)) != MOSS_OK) break;
    double ms;
    if ((st = timed(c.tile_samples, c.blocks_per_cu, &ms)) != MOSS_OK) break;
    if (ms < best_t) {
      best_t = ms;
      b = c;
    }
  }
  if (st != MOSS_OK) {
    (void)moss_set_tuning(&before);
    return st;
  }
  st = moss_set_tuning(&b);
  if (st != MOSS_OK) return st;
  *best = b;
  if (best_ms) *best_ms = best_t;
  return MOSS_OK;
}

}  // extern "C"
