// bsim_api_internal.h -- host-side objects behind the opaque ABI handles.
#pragma once

#include <unistd.h>

#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "bsim_internal.h"

namespace bsim {

// Host memory of results that were freed, kept for later ones up to kKeep
// bytes: touching fresh pages takes longer than the copy into them.  Blocks
// come back on any thread.  The contexts of a server share one pool; the end
// of the last context frees what is kept, and blocks still out then are freed
// as they come.
class BlockPool {
  public:
    static constexpr size_t kKeep = 512ull << 20;
    // A block of at least `bytes`; *cap: its size, for give().
    void* take(size_t bytes, size_t* cap);
    void give(void* p, size_t cap);
    void open();   // one more context
    void close();  // one less

  private:
    std::mutex mu_;
    std::vector<std::pair<void*, size_t>> free_;
    size_t kept_ = 0;
    int contexts_ = 0;
    const pid_t owner_ = getpid();  // (a forked process frees its copies)
};

// The host arrays of a result: ordinary memory, which a caller may hold as long
// and as much of as it likes, and which a forked process finds where it was.
// Pinned memory, which the device could write itself, is not inherited.
struct HostBlock {
    std::shared_ptr<BlockPool> pool;
    size_t cap = 0;
    void* p = nullptr;
    HostBlock(const std::shared_ptr<BlockPool>& from, size_t bytes) : pool(from), p(from->take(bytes, &cap)) {}
    ~HostBlock() { pool->give(p, cap); }
    HostBlock(const HostBlock&) = delete;
    HostBlock& operator=(const HostBlock&) = delete;
};

// Pinned memory of a context that its calls move host arrays through, taken at
// the first call that needs it: one small block, and a large one as two halves,
// of which the device fills one while host threads empty the other.  A call
// that returns 265 MB takes 8.8 ms that way (16.4 with halves of 2 MiB, 11.5
// with 4, 9.0 with 16), 7.8 where the device wrote the result's own pinned
// memory, and 64 through the runtime's copies into fresh pageable arrays.
struct HostStaging {
    static constexpr size_t kSmall = 1u << 20;
    static constexpr size_t kHalf = 8u << 20;
    void* small = nullptr;
    char* large = nullptr;
    hipEvent_t full[2] = {nullptr, nullptr};
    void* get_small();  // nullptr when there is no pinned memory
    char* get_large();
    void release();
};

// What the device and the host tell each other during a call, in one pinned
// allocation.
struct CtxPinned {
    RunStatus status[4];
    StageHost stage;
    FinalHost fin;
    uint32_t count[64];
    uint64_t report[kReportRing];
};

}  // namespace bsim

struct bsim_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;
    bsim::CtxPinned* pinned = nullptr;
    bsim::RunStatus* status_host = nullptr;  // parts of *pinned: 4 entries
    bsim::StageHost* stage_host = nullptr;   // what staging copies back
    bsim::FinalHost* final_host = nullptr;   // what finalize copies back
    uint64_t* report_host = nullptr;         // kReportRing words, written by refinement launches
    bsim::HostStaging staging;
    std::shared_ptr<bsim::BlockPool> blocks;
    uint32_t chunk_max = 32;
    uint32_t time_launches = 0;
    uint32_t hub_table_slots = 8192;  // LDS slots per hub-bucket block on this device
    uint32_t frontier_limit_pct = 10;  // incremental: larger frontiers recompute the level for all vertices
    uint32_t frontier_edge_pct = 15;   // ... and so do frontiers with more than this share of the edges
    // 0: the stop test looks two levels back, so that one level past the last
    // is hashed; else it knows the level just hashed
    uint32_t tail_split_ppm = 100;
    uint32_t* count_host = nullptr;   // part of *pinned: scratch for counts, 64 entries
    // batched calls: schedules picked by the autotuner, per size class
    uint32_t autotune = 1;
    struct BatchTune {
        uint64_t small_edges;       // graphs of at most this many edges go to the small-graph launch
        uint32_t hub_table_slots;   // LDS slots of a hub-bucket block
    };
    std::map<uint64_t, BatchTune> batch_tune;
    BatchTune last_batch{0, 0};     // what the last batched call ran with
    uint64_t fixed_small_edges = ~0ull;  // the schedule when autotune is off
    // temporaries of summarize and batched calls: one device buffer, grown
    // to the largest demand of the earlier calls (keep_work = 0: every call
    // takes them from the stream-ordered pool and returns them)
    uint32_t keep_work = 1;
    void* work = nullptr;
    size_t work_cap = 0, work_want = 0;
};

namespace bsim {

// Arrays shared by several results (the per-graph results of one batched
// call are views into the batch's arrays); freed with the last holder.
struct SharedArrays {
    int device = 0;
    hipStream_t stream = nullptr;
    std::vector<void*> device_ptrs;
    std::shared_ptr<HostBlock> host;
    ~SharedArrays();
};

// Owner of a result's arrays.
struct ResultPriv {
    int device = 0;
    hipStream_t stream = nullptr;
    std::vector<void*> device_ptrs;
    std::shared_ptr<HostBlock> host;
    std::vector<uint32_t> blocks_per_iter;
    std::shared_ptr<SharedArrays> shared;
};

// Device copies of the caller's graph when it arrives in host memory, or
// the caller's device pointers as they are.
struct DeviceGraph {
    Staged g;
};

// Let ctx take the memory of its host results from the pool of `with`.
void share_blocks(bsim_ctx* ctx, const bsim_ctx* with);

// staging: pinned memory for the upload of a small graph (nullable), in use
// until the stream has run past the upload.
void upload_graph(const bsim_graph& in, Staged& g, Arena& arena, hipStream_t s, HostStaging* staging = nullptr);

// Queue up to 8 copies between arrays of the library's own, all visible to the
// device, in one launch where they are small (a copy apiece otherwise); bytes
// are multiples of 4, addresses 4-byte aligned.  Never with a caller's pointer:
// the kernel would fault where the runtime's copy returns an error.
void copy_ranges(void* const* dst, const void* const* src, const size_t* bytes, int n, hipStream_t s);

// The six result arrays copied from dev[] into one block of host memory;
// base[i] = their places.  Returns once they are there.
std::shared_ptr<HostBlock> host_arrays(bsim_ctx* ctx, void* const* dev, const size_t* bytes, void** base);

// Per-level hash storage handed to the refinement loop.  With `levels`
// empty the loop double-buffers; otherwise levels[k] receives h^k.
struct LevelSink {
    std::vector<uint64_t*> levels;
};

struct LoopResult {
    uint32_t k_done = 0;
    uint32_t fixpoint = 0;
    uint32_t launches = 0;
    uint32_t split_launches = 0;  // launches run as a split half and a hash half
    float ms_kernels = 0.f;      // refinement launches that did work
    float ms_hub_kernels = 0.f;  // hub launches of those iterations
    uint32_t n_timed = 0;        // launches the two sums cover
    std::vector<uint32_t> blocks_per_iter;
    const uint64_t* h_final = nullptr;
};

// Iterations 0..k_done on a staged graph.  rep_prev (nullable, n entries)
// receives the class representatives of level k_done - 1 (of level 0 when
// k_done = 0; at a fixpoint those of level k_done, the same partition).
// use_timers: bracket launches with HIP events when the ctx option asks for
// it (the allocation-free entry point passes false).
LoopResult run_refinement(bsim_ctx* ctx, const Staged& g, const bsim_params& p, RunBuffers& rb,
                          LevelSink* sink, Arena& arena, uint32_t* rep_prev = nullptr, bool use_timers = true);

// The allocation-free entry point's scratch: its device address on the
// current device, looked up once per device (bsim_ctx_create calls it).
int noalloc_scratch_init(int device, std::string* err);

// finalize with summary edges into the classes named by rep_prev (their
// first-occurrence block ids) instead of the final blocks.
void finalize_prev_level(const Staged& g, const uint32_t* rep, const uint32_t* rep_prev, bool want_edges,
                         FinalOut& out, FinalHost* host, Arena& arena, Arena& keep, hipStream_t s);

// Assemble a bsim_result from finalize output (takes ownership of `keep`);
// hashes_preset: an array of n entries in `keep` to receive the hashes.
bsim_result* make_result(bsim_ctx* ctx, const Staged& g, const LoopResult& lr, const uint64_t* h,
                         FinalOut& fo, Arena& keep, uint32_t flags, uint64_t* hashes_preset = nullptr);

// Whole batch path for one graph; labels = the kept label set of the label
// parameterization (nullptr: every edge).
bsim_result* summarize_graph(bsim_ctx* ctx, const bsim_graph& graph, const bsim_params& p,
                             const std::vector<uint32_t>* labels);

// Many independent graphs in one refinement run (a disjoint union); graphs
// of at most small_edges edges (0: none) that fit one workgroup go to the
// persistent small-graph launch.
void batch_summarize(bsim_ctx* ctx, const bsim_graph* graphs, uint32_t n_graphs, const bsim_params& p,
                     bsim_result** outs, uint64_t small_edges);

// Batch path that also returns a resident state for incremental updates.
int summarize_with_state(bsim_ctx* ctx, const bsim_graph& graph, const bsim_params& p,
                         bsim_state** state_out, bsim_result** out);

// directions: whether the caller takes BSIM_BACKWARD / BSIM_BOTH_DIRECTIONS
// (only the single-graph summarization does).
void validate_params(const bsim_graph& graph, const bsim_params& p, bool directions = false);

// Back `arena` with the ctx's work buffer, grown first to the largest
// demand of the ctx's earlier calls and to at_least bytes (what does not
// fit comes from the pool; a failed growth leaves the arena on the pool).
// ctx_note_demand records a finished call's demand; ctx_release_work frees
// the buffer.
void ctx_back_arena(bsim_ctx* ctx, Arena& arena, size_t at_least = 0);
void ctx_note_demand(bsim_ctx* ctx, const Arena& arena);
void ctx_release_work(bsim_ctx* ctx);

// Device bytes a resident state holds.
uint64_t state_bytes(const bsim_state* st);
// The context a state runs on.
bsim_ctx* state_ctx(const bsim_state* st);

}  // namespace bsim
