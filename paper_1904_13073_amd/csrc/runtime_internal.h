// Host-side objects shared by the C ABI files: device arenas, executors (a
// HIP stream with its statistics buffers and timing events) and the stream
// object itself.
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <utility>
#include <string>
#include <vector>

#include "swgn.h"
#include "swgn_frame.h"

namespace swgn {
namespace rt {

constexpr int kMaxNodes = 32768;
// Untuned batches take fused PCG steps up to this many rows in all (where one
// launch per iteration beats two; above it the products' re-reads cost more).
constexpr int64_t kFusedRows = 8192;
constexpr int kPcgAuto = 0, kPcgSplit = 1, kPcgFused = 2;
constexpr int64_t kMaxSurfels = (int64_t)1 << 28;

struct HipFail {
    hipError_t e;
    std::string what;
};

// an argument found wrong on the device
struct BadInput {
    std::string what;
};

#define SWGN_HIP(x)                                                         \
    do {                                                                    \
        hipError_t _e = (x);                                                \
        if (_e != hipSuccess) throw ::swgn::rt::HipFail{_e, std::string(#x)}; \
    } while (0)

// Device allocations released together.
class Arena {
public:
    ~Arena() { release(); }
    // 256-byte aligned; carved from the current chunk of device memory or a new
    // one (chunks grow geometrically from 4 MiB, so an arena of many arrays
    // costs a few hipMalloc calls, not one per array)
    void* raw(size_t bytes);
    template <class T>
    T* alloc(size_t n) {
        return static_cast<T*>(raw(n * sizeof(T)));
    }
    void release();
    // hands the chunks out again from the start (no device memory is freed;
    // the caller makes sure no work still uses what they held)
    void reset();
    // one piece instead of everything handed out before: in the memory at hand
    // if it holds that and is not much larger, else in new memory with an
    // eighth to spare (a model that grows a little each frame)
    void* renew(size_t bytes);
    size_t held() const {                     // bytes of device memory, handed out or not
        size_t n = 0;
        for (const Chunk& c : chunks_) n += c.size;
        return n;
    }
    void swap(Arena& o) {
        chunks_.swap(o.chunks_);
        std::swap(cur_, o.cur_);
    }

private:
    struct Chunk {
        char* base;
        size_t size, used;
    };
    std::vector<Chunk> chunks_;
    size_t cur_ = 0;                      // chunk handed out from
};

// A HIP stream plus what a solve needs besides the streams' own memory: the
// pinned host slots the statistics are written to (kMaxBatch streams) and
// timing events.
struct Executor {
    hipStream_t st = nullptr;
    bool own_stream = false;
    void* stats_host = nullptr;
    char* stats_dev = nullptr;            // the device's address of stats_host
    std::vector<hipEvent_t> events;
    // launch variant per stage (kVarXcd | kVarWide bits), per shape bucket of
    // a batch; chosen by the autotuner, a size rule where it has not run
    std::map<uint64_t, std::vector<int>> tuned;
    uint64_t bucket = 0;                  // bucket of the batch being launched
    uint64_t tune_epoch = 0;              // bumped when a choice changes (captured graphs are stale)
    int variant_of(int stage, int64_t rows) const;
    // replay of a batch's iterations as one HIP graph
    bool graphs = false;
    int pcg_mode = 0;                     // kPcgAuto, kPcgSplit, kPcgFused
    // whole linear solves in one launch (pcg.hip): the device's CUs (0: never
    // used); whether the call being enqueued takes them, in how many
    // workgroups per launch at most (its lease; 0: as many as it likes, for
    // none waits for another), of how many waves, and whether one has a CU to
    // itself
    int device = 0;
    int pcg_cus = 0;
    bool pcg_whole = false;
    int pcg_lease = 0;
    int pcg_waves = 4;
    bool pcg_alone = false;
    int pcg_hold = 0;                     // leases refused before the next one is tried (after a wait given up)
    int pcg_backoff = 0, pcg_good = 0;    // the last such number; leases that ended well since
    void pcg_stalled(int leases_per_frame);
    std::vector<std::pair<sw_stream, uint64_t>> graph_key;   // (stream, generation) the graphs were captured for
    // one graph per way the linear solves are launched in (it follows from the
    // lease, which depends on what other executors hold), the latest first
    struct Graph {
        std::vector<int> launches;
        hipGraphExec_t exec;
    };
    std::vector<Graph> graph_execs;
    ~Executor();
    void init(void* hip_stream);
    hipEvent_t event(size_t i);
    void drop_graphs();
};

// The right to have a number of workgroups of whole solves on a device, held
// while launches that need them may run: they wait for each other, so all that
// are in flight in this process must find a place together (swgn_lease.h).
// Takes what the streams can use, at least their largest solve, or nothing
// (their linear solves then run step by step, with equal results). Other
// kernels of the process can hold the CUs too, but end by themselves; other
// processes are not known here: the kernel's waits are bounded.
class PcgLease {
public:
    PcgLease(Executor& ex, const std::vector<sw_stream>& ss);
    ~PcgLease() { release(); }
    PcgLease(const PcgLease&) = delete;
    PcgLease& operator=(const PcgLease&) = delete;
    // waits for the executor's stream and gives the workgroups back
    void release();

private:
    Executor& ex_;
};

inline sw_status fail(std::string& err, sw_status code, const std::string& msg) {
    err = msg;
    return code;
}

template <class F>
sw_status guarded(std::string& err, F&& f) {
    try {
        return f();
    } catch (const HipFail& h) {
        const sw_status code =
            (h.e == hipErrorOutOfMemory || h.e == hipErrorMemoryAllocation) ? SW_ENOMEM : SW_EHIP;
        return fail(err, code, h.what + ": " + hipGetErrorString(h.e));
    } catch (const BadInput& b) {
        return fail(err, SW_EINVAL, b.what);
    } catch (const std::bad_alloc&) {
        return fail(err, SW_ENOMEM, "host allocation failed");
    }
}

size_t carve_workspace(FrameDesc& h, char* base);

// Frames an executor solves step by step after a wait given up, doubled each
// time it happens again up to the second number (a wait is 100 ms, a frame about
// 1 ms: at worst 2.5% of the time), until as many have gone well.
constexpr int kPcgHoldFrames = 64, kPcgHoldMost = 4096;
// graphs an executor keeps of one batch (all whole, all in steps, and a few between)
constexpr size_t kGraphsKept = 4;
// longest wait of a whole solve's workgroup for the others before the frame
// is solved again step by step (100 ms, in 10 ns)
constexpr long long kPcgWait = 10000000;

}  // namespace rt
}  // namespace swgn

struct sw_stream_s {
    sw_config cfg{};
    swgn::Cam cam{};
    std::string err;
    swgn::rt::Executor exec;              // the stream's own HIP stream
    swgn::rt::Arena frame_mem, surf_mem, graph_mem, ws_mem;
    swgn::rt::Arena setup_mem;            // temporaries of the node-set build, kept for the next one
    swgn::rt::Arena geo_mem, spare_mem;   // geometry update: temporaries, and the surfels before it (the next update's)
    int64_t held_ns = 0;                  // the largest model since the arenas were last given back
    int held_nn = 0;
    uint64_t generation = 0;              // bumped whenever device buffers are replaced

    // surfels as given
    int64_t ns = 0;
    float* in_pos = nullptr;
    float* in_nrm = nullptr;
    float* in_rad = nullptr;              // attributes, caller order (kept current by fusion)
    float* in_conf = nullptr;
    int* in_tobs = nullptr;
    int* in_tinit = nullptr;
    int t_now = 0;                        // frame time (visibility of recent surfels)

    // depth-map fusion workspace, allocated on first use
    swgn::rt::Arena fuse_mem;
    unsigned long long* fz4 = nullptr;    // 4x super-sampled index map
    float* flive = nullptr;               // [6][pitch] live positions and normals of the last fusion
    int* fmatch = nullptr;                // [npx]
    int* fcount = nullptr;                // [2]
    int* fcount_host = nullptr;           // pinned, [8]: fusion counts, append counts
    bool fused = false;
    uint64_t depth_gen = 0;               // bumped by every depth preprocessing
    uint64_t fuse_gen = ~0ull;            // depth_gen of the last fusion
    // append-candidate workspace, allocated on first use
    swgn::rt::Arena append_mem;
    int *aflag = nullptr, *apos = nullptr, *ascan = nullptr, *acount = nullptr;
    float4 *asv = nullptr, *asn = nullptr, *aboxes = nullptr;
    int* apix = nullptr;                  // staging of host outputs, capacity npx
    float *apos3 = nullptr, *anrm3 = nullptr, *arad = nullptr, *aconf = nullptr;
    bool surfels_set = false;
    bool graph_set = false;
    // sets of local nodes the whole-solve kernel needs with workgroups of 4
    // and 8 waves (0: the node set does not fit it)
    int pcg_sets4 = 0, pcg_sets8 = 0;
    sw_solve_counts counts{};
    int64_t folds = 0;                    // since the exchange words were last cleared
    int pcg_sets(int waves) const { return waves == 4 ? pcg_sets4 : pcg_sets8; }
    sw_server server = nullptr;           // set while attached to a serving loop

    // descriptor: host copy, pinned staging copy and the device copy kernels read
    swgn::FrameDesc h{};
    swgn::FrameDesc* h_pinned = nullptr;
    swgn::FrameDesc* d_desc = nullptr;
    size_t ws_bytes = 0;
    int nsets = 0;                        // distinct node sets
    int64_t nent = 0;                     // block-fold entries

    // node numbering: the library keeps nodes in a spatially local order
    // (Morton order of their reference positions), so that a block row's
    // columns lie near it; every export is in the caller's order
    std::vector<int> node_perm;           // library index k -> caller index
    std::vector<int> node_inv;            // caller index -> library index
    int* d_node_id = nullptr;             // [nn] node_perm on the device
    int* d_node_inv = nullptr;            // [nn] node_inv on the device

    float* se3_host = nullptr;            // pinned, node transforms for the caller; room for se3_host_nodes
    size_t se3_host_nodes = 0;
    int* info_host = nullptr;             // pinned, [kInfo]: sizes a setup hands to the host

    // captured iteration (allocated only when the config asks for a capture)
    int* dbg_index = nullptr;
    float *dbg_H = nullptr, *dbg_g = nullptr, *dbg_x = nullptr, *dbg_J = nullptr;
    bool captured = false;

    ~sw_stream_s() {
        if (h_pinned) (void)hipHostFree(h_pinned);
        if (fcount_host) (void)hipHostFree(fcount_host);
        if (se3_host) (void)hipHostFree(se3_host);
        if (info_host) (void)hipHostFree(info_host);
    }
};

namespace swgn {
namespace rt {
// update: a PCG finish or fused step launch that also performs the node
// update of every stream whose last finish it holds (not for replays)
void run_stage(Executor& ex, int stage, const std::vector<sw_stream>& ss, const std::vector<int>& its, int pcg_it,
               const DepthIn* depth, bool timing, std::vector<int>& ev_stage, bool update = false);
void enqueue_depth(Executor& ex, const std::vector<sw_stream>& ss, const float* const* depths, int32_t on_device,
                   bool timing, std::vector<int>& ev);
void enqueue_rigid(Executor& ex, const std::vector<sw_stream>& ss, bool timing, std::vector<int>& ev);
void enqueue_iteration(Executor& ex, const std::vector<sw_stream>& ss, const std::vector<int>& its, bool timing,
                       std::vector<int>& ev, std::vector<char>& captured);
// counts the linear solves of one Gauss-Newton iteration as enqueue_iteration runs them
void count_solves(const Executor& ex, const std::vector<sw_stream>& ss, const std::vector<int>& its);
// before n folds of the stream are enqueued: clears the whole solve's exchange
// words if their tags could come again
void count_folds(Executor& ex, sw_stream s, int64_t n);
void enqueue_collect(Executor& ex, const std::vector<sw_stream>& ss);
sw_status collect_frames(Executor& ex, const std::vector<sw_stream>& ss, const float* stage_us,
                         sw_frame_stats* stats, sw_status* status, std::vector<char>* stalled = nullptr);
// stalled (or null): streams whose frame has to be solved again because a
// whole solve gave up waiting (their node state is the frame's start's)
sw_status finish_frames(Executor& ex, const std::vector<sw_stream>& ss, const float* stage_us,
                        sw_frame_stats* stats, sw_status* status, std::vector<char>* stalled = nullptr);
uint64_t shape_bucket(const std::vector<sw_stream>& ss);
void server_quiesce(sw_server sv, sw_stream s);
void server_forget(sw_server sv, sw_stream s);
sw_status solve_frames(Executor& ex, const std::vector<sw_stream>& ss, const float* const* depths,
                       int32_t on_device, bool timing, sw_frame_stats* stats, sw_status* status);
}  // namespace rt
}  // namespace swgn
