// pj_host_internal.h -- host-side runtime pieces of libpassjoin shared by the join, index and
// serving translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <exception>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/passjoin.h"
#include "pj_internal.h"

namespace pj {

struct Error {
    int code;
    std::string msg;
    Error(int c, const char* fmt, ...);
};

void hip_check(hipError_t e, const char* what);

// Device allocator interface: named buffers, so a workspace can reuse them across calls.
struct Alloc {
    long long budget = 0;   // 0 = unlimited
    size_t used = 0;        // bytes requested in the current call
    size_t aside = 0;       // scratch of the call that lies elsewhere and counts against the budget
    virtual ~Alloc() = default;
    virtual void* get(const char* name, size_t bytes) = 0;
    void set_aside(const char* name, size_t bytes);
};

// Grow-only named buffers cached per thread (scratch of one call at a time).
struct Workspace : Alloc {
    struct Buf {
        void* p = nullptr;
        size_t cap = 0;
    };
    std::unordered_map<std::string, Buf> bufs;
    ~Workspace() override;
    void* get(const char* name, size_t bytes) override;
    void begin_call(long long b) { budget = b; used = 0; }
    void release_all();
};

// hipMalloc which, when memory runs out, first gives back the blocks kept for reuse
hipError_t device_malloc(void** p, size_t bytes);

// Allocations owned by a long-lived object (an index); freed with it.  Small ones share chunks, and
// the blocks of one object serve the next: unmapping a block of some 20 MB takes 300-700 us.  `used`
// is what the blocks hold.  Under a budget every allocation is a block of its size.
struct Owned : Alloc {
    struct Block {
        void* p = nullptr;
        size_t cap = 0;
        int device = 0;
        uint64_t freed = 0;     // when it was given up (count of objects freed)
    };
    std::vector<Block> blocks;
    void* chunk = nullptr;      // of the last chunk for small ones: the free part
    size_t chunk_left = 0;
    ~Owned() override;
    void* get(const char* name, size_t bytes) override;

private:
    void* take(size_t bytes);
};

// Scratch counted against A's budget (in addition to what A holds) while the scope lasts.
struct AsideScope {
    Alloc& A;
    const size_t before;
    explicit AsideScope(Alloc& a) : A(a), before(a.aside) {}
    ~AsideScope() { A.aside = before; }
};

Workspace& thread_workspace();
int device_cus();
// candidates from which the batched path buckets its hits (tests set it by the environment)
uint64_t bucket_min_candidates();

// Values the host reads back from the device to size the next phase.  A self-join plan runs the join
// once recording them in order, then captures the same sequence of launches in a graph: while it
// captures, every read is served from the record, and nothing is read back or synchronised (the
// tables by length are made on the device, by the captured launches).
struct ReadTape {
    bool replay = false;
    std::vector<uint8_t> bytes;
    size_t pos = 0;
    std::vector<std::pair<void*, size_t>> pending;   // reads enqueued before the next sync
};
extern thread_local ReadTape* t_tape;
// device -> host read, complete after the next sync_readback on the stream
void readback(void* host, const void* dev, size_t bytes, hipStream_t st);
void sync_readback(hipStream_t st);
// forgets this thread's read-backs that no sync_readback completed (after waiting for their
// streams): their targets belong to a scope an exception is leaving
void drop_readbacks();
// declared in a function that issues read-backs into its own variables: when an exception
// leaves the function between a read-back and its sync, the read-back is dropped
struct ReadbackScope {
    int uncaught = std::uncaught_exceptions();
    ~ReadbackScope()
    {
        if (std::uncaught_exceptions() > uncaught) drop_readbacks();
    }
};
// device memory = 0 with a kernel (bytes a multiple of 4)
void zero_words(void* dev, size_t bytes, hipStream_t st);

// hipEvent marks on one stream (none while a plan's graph is captured).
struct Timer {
    hipStream_t st;
    std::vector<hipEvent_t> evs;
    explicit Timer(hipStream_t s);
    ~Timer();
    int mark();
    double ms(int a, int b);
};

// Launch parameters of the batched path that do not change results (chosen by the autotuner,
// pj_tune.cpp; these are the built-in defaults).
struct TuneParams {
    int verify_waves_per_cu = 32;   // persistent grid of the verification kernels
    int seg_chunk = 4;              // list segments (64 members each) per wave chunk; 4: by their
                                    // number (list_seg_chunk)
    int big_list = 32;              // lists with at least this many candidates: list-segment kernel
    int probe_blocks_per_cu = 8;    // grid of the probe kernel
    int lane_cands = 1;             // list-segment candidates per lane (1 or 2)
    int probe_map = 1;              // probe threads: 0 string-major, 1 pair-major (64 strings)
};

bool tune_params_valid(const TuneParams& p);
// Parameters for a call: the autotune table entry for (this GPU, tau, length bucket of the
// probe set's mean length), read from the cache file when one is named, else the defaults.
TuneParams tune_lookup(const char* cache, int tau, double mean_len);

struct JoinScratch {
    int mode = PJ_MODE_AUTO;
    TuneParams tp;
    unsigned long long* counters = nullptr;
    Hit* hits = nullptr;
    unsigned long long* prefix = nullptr;
    uint64_t nhits = 0, ncand = 0;
    uint64_t* out = nullptr;
    uint64_t naccepted = 0;
    uint64_t guard_misses = 0;
    struct Mark { int a, b, kind; };     // event pairs around kernel launches (0 probe, 1 verify)
    std::vector<Mark> kernel_marks;
};

// with_sym: also the symbol map of the set's bytes (sets to be indexed)
void build_set(const pj_strings* S, bool on_device, Alloc& A, const std::string& tag, DevSet& D,
               hipStream_t st, bool with_sym = false);
void build_index(const DevSet& D, int tau, Alloc& A, const std::string& tag, DevIndex& X,
                 hipStream_t st, bool with_inline = false, bool with_share = false);
// The hits of a query batch that has been probed: records, the probe's counters on the device and here
// ([0] hits, [1] candidates, [2] selected).
struct ProbedHits {
    Hit* hits = nullptr;
    const unsigned long long* counters = nullptr;
    uint64_t counts[3] = {};
};
// What to probe: a uniform tau against one index, or per-probe thresholds (q_tau, by sorted
// position of the probe set) against the per-tau indices in refs.
struct ProbeSpec {
    bool self = false;
    int tau = 0;                       // uniform tau, or the largest tau of the batch
    const DevIndex* X = nullptr;       // uniform index
    const int32_t* q_tau = nullptr;    // device, per sorted position (mixed batch)
    const IndexRef* refs = nullptr;    // device, [kTauMax + 1] (mixed batch)
    uint64_t bound = 0;                // selection bound for a mixed batch (computed by the caller)
    SymMap sym;                        // the indexed set's symbol map (index keys)
    bool has_entries = true;           // some index has entries
    int selection = 0;                 // PJ_SELECT_*
    int probe_min_len = 0;             // self-join: only strings at least this long probe
    const ProbedHits* probed = nullptr;   // a batch probed already: only the rest
};

void run_candidates(const DevSet& P, const DevSet& Y, const ProbeSpec& spec, JoinScratch& J,
                    pj_stats& stats, Timer& tm, hipStream_t st);
uint64_t finish_pairs(const DevSet& P, const DevSet& Y, bool self, const uint64_t* acc,
                      uint64_t m, int32_t** a_out, int32_t** b_out, hipStream_t st);
void emit_output(const int32_t* da, const int32_t* db, uint64_t M, bool to_device, pj_pairs* out,
                 hipStream_t st);

void validate_host_strings(const pj_strings* S, const char* what);
void run_query_batch(const pj_index* idx, const pj_strings* Q, const int32_t* taus,
                     std::vector<uint64_t>& pairs, pj_stats& stats, hipStream_t st,
                     const char* tune_cache);
int64_t query_footprint(const pj_index* idx, int n, int tau);
void index_taus(const pj_index* idx, int* lo, int* hi);
const DevSet& index_set(const pj_index* idx);
const IndexRef* index_refs(const pj_index* idx);
SymMap index_sym(const pj_index* idx);
bool index_has_entries(const pj_index* idx);
int index_device(const pj_index* idx);
int64_t query_selections(const pj_index* idx, int n, int tau);

// Fixed-capacity buffers of one mixed-tau query batch run by launch_graph_probe and
// launch_graph_verify: the layout of the batch tables (counters, zero | nx | lenstart | gbase | perm |
// q_tau | slen, packed on the host) and the arena, uploaded in one copy, and the device work buffers.
// Used by the serving slots' captured pipelines (allocated), by small pj_query calls (in the thread's
// workspace) and by pj_query_noalloc (carved out of a static device array).
struct BatchLayout {
    int64_t qcap = 0, bcap = 0;             // queries, arena bytes
    uint64_t hcap = 0, cand_cap = 0, acc_cap = 0;
    size_t off_lenstart = 0, off_gbase = 0, off_perm = 0, off_qtau = 0, off_slen = 0;
    size_t tables_bytes = 0, arena_bytes = 0;
    size_t first_words = 0;
    size_t result_bytes = 0;                // [counters 8 | bcounts 4 | out_n | out kGraphSortCap]
};
// Part of a result block read back at once: most batches have no more pairs (a larger one's rest
// is a second copy).
constexpr uint32_t kBatchFirstPairs = 1024;
constexpr size_t kBatchFirstBytes = sizeof(uint64_t) * (kBatchResultHead + kBatchFirstPairs);
struct BatchBuffers {
    uint8_t* tables = nullptr;
    uint8_t* arena = nullptr;
    Hit* hits = nullptr;
    unsigned long long* prefix = nullptr;
    uint32_t* first = nullptr;
    uint64_t* acc = nullptr;
    uint8_t* result = nullptr;
};
enum class PackStatus { kOk, kTooManyQueries, kTauOutOfRange, kTooManySelections, kTooManyBytes };
BatchLayout batch_layout(int max_queries, uint64_t hcap, uint64_t cand_cap, uint64_t acc_cap);
size_t batch_device_bytes(const BatchLayout& L);
BatchBuffers carve_batch_buffers(const BatchLayout& L, uint8_t* base);
// tau_max: the largest threshold a batch may hold; queries: the most queries (grid sizes)
void setup_graph_batch(const pj_index* idx, const BatchLayout& L, const BatchBuffers& B, int tau_max,
                       int queries, const TuneParams& tp, GraphBatch& G);
// Packs Q into the host mirror of the tables and, after them, the arena; *arena_used = its bytes.
PackStatus pack_query_batch(const pj_index* idx, const BatchLayout& L, const pj_strings* Q,
                            const int32_t* taus, uint8_t* h_tables, int64_t* arena_used);
// Reads the rest of a result block of m pairs after its first part has been read back to h_result.
void read_batch_rest(uint8_t* h_result, const uint8_t* result, uint32_t m, hipStream_t st);
// Reads a batch result block: adds its counters to stats, returns the number of sorted
// (query << 32 | indexed id) pairs at *pairs; *flags != 0 means a capacity overflowed.
uint32_t batch_result(const uint8_t* h_result, pj_stats& stats, const uint64_t** pairs,
                      unsigned long long* flags);

// A serving slot's captured query pipeline (pj_graph.cpp): fixed-capacity device buffers, one
// instantiated hipGraph of the device phases, pinned staging for the batch and its result.
struct GraphPlan;
GraphPlan* graph_plan_create(const pj_index* idx, int max_queries, hipStream_t st,
                             const char* tune_cache);
void graph_plan_destroy(GraphPlan* g);
int64_t graph_plan_device_bytes(int max_queries);
// Runs one batch through the graph; false when the batch does not fit the plan's capacities or
// a device-side capacity overflowed (the caller then runs it with run_query_batch).  pairs get
// (query << 32 | indexed id), sorted.
bool graph_plan_run(GraphPlan* g, const pj_strings* Q, const int32_t* taus,
                    std::vector<uint64_t>& pairs, pj_stats& stats);
void release_thread_workspace();

// pj_self_join with the launch parameters given (the autotuner's trial runs)
int self_join_with(const pj_strings* S, int32_t tau, const pj_options* opt, pj_pairs* out,
                   const TuneParams* force);

extern thread_local std::string t_last_error;
extern thread_local pj_stats t_stats;
extern thread_local pj_stats t_last_ok_stats;

}  // namespace pj
