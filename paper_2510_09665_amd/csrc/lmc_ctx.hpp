// Internal to liblmc: the context behind lmc_ctx_t and what its translation units share
// (lmc_ctx.cpp: life cycle, index calls, waiting; lmc_pipeline.cpp: store / retrieve;
// lmc_streams.cpp: hardware queues; lmc_measure.cpp: measurement aids; lmc_static.cpp: the
// entry point that allocates nothing).  Not part of the C ABI (include/lmc.h).
#ifndef LMC_CTX_HPP
#define LMC_CTX_HPP
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "../../include/lmc.h"
#include "lmc_guard.hpp"
#include "lmc_index.hpp"
#include "lmc_kernels.hpp"

namespace lmci {

// Staging ring of one direction.  The memory is num_staging allocations of buf_bytes;
// it is handed out in slots of slot_bytes (bulk mode: one slot per allocation;
// layer-wise mode: many small slots, so that a call seldom has to wait for a slot).
// Each slot has a `filled` event (producer done) and a `drained` event (consumer done).
struct Ring {
    std::vector<uint8_t *> buf;
    uint64_t buf_bytes = 0, slot_bytes = 0;
    uint32_t slots_per_buf = 1;
    std::vector<hipEvent_t> filled, drained;
    std::vector<char> used;
    uint64_t pos = 0;
};

struct Op {
    uint64_t ticket = 0;
    hipEvent_t done = nullptr;       // null: nothing enqueued (yet) for this ticket
    hipStream_t final_stream = nullptr;  // the library stream `done` was recorded on
    // Not 0: finished when the word of host memory has reached this.  A load that tells (its kernels run on the
    // caller's own stream) has no event.
    uint64_t stored_target = 0, loaded_target = 0;
    bool on_caller = false;              // its kernels run on the caller's own stream ...
    hipStream_t caller = nullptr;        // ... this one
    std::vector<int64_t> slots;      // pool slots whose in-flight count this op holds
    // layer-wise operations (paper section 5.2)
    bool layerwise = false;
    bool pending = false;                 // a store whose layers have not all been submitted
    int32_t next_layer = 0;               // first layer not yet submitted
    int32_t steps = 0;                    // pending store: lmc_store_layers calls served so far
    std::vector<hipStream_t> ends_on;     // pending store: the streams its steps so far end on
    // pending store: not 0: its steps without staging on s_d2h2 are done when kStoreStepWord has reached this
    uint64_t second_target = 0;
    bool has_staged_steps = false;
    hipStream_t producer = nullptr;       // pending store: the stream its last step was handed in with
    bool began_idle = false;              // pending store: nothing was on the caller's stream when it began
    std::vector<int64_t> new_chunk;       // pending store: chunk numbers that are new
    const int64_t *slot_mapping = nullptr;  // pending store: the caller's slot mapping
    std::vector<hipEvent_t> layer_done;   // per layer: event after which the layer is in place
    // ... or, for steps of a store that count themselves off, the word and the value it has then (0: no such step)
    struct Count {
        int word = 0;
        uint64_t target = 0;
    };
    std::vector<Count> layer_count;
    std::vector<hipEvent_t> owned_events; // the distinct events behind layer_done
    // A layer-wise retrieve that runs as one launch (retrieve_in_steps) has words instead: the layers of
    // step i are in place when word i of the context has reached step_target[i].
    int32_t step_layers = 0;
    std::vector<uint64_t> step_target;
    // The last stream that was made to wait for a step of it, and how far: for the steps of a load (waited[0]: how
    // many), for the values of kStoreWord and kStoreStepWord.  Steps end in order, so a stream that waits for one
    // need not wait for it or an earlier one again: a wait takes the calling thread 3 us and the stream's queue as
    // long, 32 of them more than 4 MiB take to come.  (A stream that takes the handle of a destroyed one has nothing
    // to wait for: the destroyed one's wait was over, see launches_on_caller.)
    hipStream_t waiter = nullptr;
    uint64_t waited[2] = {0, 0};
    bool waits_last = false;              // the newest wait has no event behind it (event_behind_wait)
    bool has_waiting(hipStream_t s, int which, uint64_t upto) const {
        return s == waiter && upto <= waited[which] && s != hipStreamPerThread;
    }
    void made_wait(hipStream_t s, int which, uint64_t upto) {
        if (s != waiter) waited[0] = waited[1] = 0;
        waiter = s;
        waited[which] = upto;
        waits_last = true;
    }
};

// One timed step of a pipeline: a kernel launch (LMC_FLAG_TIMING, LMC_FLAG_TRACE) or the
// copies of one group (LMC_FLAG_TRACE), between two timing events.
struct Timing {
    hipEvent_t start, stop;
    int32_t stage;        // LMC_STAGE_*
    uint64_t ticket;      // the operation the step belongs to, 0 = none
    int32_t chunks;
    uint64_t bytes;
};

struct CopyTiming {   // a large device-to-host copy by the runtime, watched by the guard
    hipEvent_t start, stop;
    uint64_t bytes;
};

}  // namespace lmci

using lmci::CopyTiming;
using lmci::Op;
using lmci::Ring;
using lmci::Timing;

struct lmc_ctx {
    lmc_config_t cfg{};
    lmc::KernelGeom kg{};
    lmc::LaunchShape shape{};
    uint32_t link_groups = 64;  // groups of 256 lanes of a launch whose other side is the pinned pool; 0 = as for HBM
    // Which copies between staging and the pool the library's own link-paced copy kernel
    // makes instead of hipMemcpyAsync: bit 0 = to the host, bit 1 = from the host.  Off
    // by default: the runtime's copies leave the compute units to the engine (a product that
    // fills every compute unit once takes 1.4 to 1.7 times as long beside the kernel).  But for some seconds after tens
    // of GiB of device or pinned memory have been freed or allocated in the process, the
    // runtime's device-to-host copies inside a store ran at 31.5 GB/s instead of 57 on
    // the machine this was measured on (not with HSA_ENABLE_SDMA=0, which points at the
    // copy engines being busy with the driver's own work on that memory); the kernel's
    // 57 GB/s does not depend on that.
    uint32_t copy_kernel = 0;
    // ... and the guard that switches device-to-host copies to the kernel by itself while
    // the runtime's are slow (lmc_guard.hpp).  On unless switched off (lmc_tune "d2h_guard"):
    // in a mix of stores and retrieves of many requests the runtime's copies to the host
    // collapse now and then (whole stores at 12.7 GB/s), and the mix runs in 3.2 s with the
    // guard against 4.4-5.2 s without; on the one-way 10 GiB request it costs nothing when
    // the runtime is healthy (one pair of event markers per group) and lifts a fresh
    // process's slow first seconds from 44.5 to 54.5 GB/s.
    bool d2h_guard_on = true;
    uint64_t pieces_by_kernel_below = uint64_t(2) << 20;   // bytes per transfer; see copy_group
    int32_t store_step_streams = 2;   // streams the steps of a layer-wise store take in turn, staged or not
    bool caller_waits = true;     // a bulk retrieve ends with the caller's stream waiting for it
    lmc::CopyEngineGuard d2h_guard;
    std::vector<CopyTiming> copy_timings;
    std::chrono::steady_clock::time_point born = std::chrono::steady_clock::now();
    int64_t edge_chunks = 1;  // size of the group at the exposed end of a pipeline; 0 = no special group
    // Scatter launches in the order of the destination (lmc_kernels.hpp): 0 = never, 1 = when
    // the launch fills enough pages per plane for neighbours to exist (ordered_min_pages pages
    // and at least one block in ordered_min_density_inv of the plane), 2 = whenever possible.
    // Off: measured on MI355X it loses to the plain order at every density tried (2048 of
    // 8192, 6480 of 16384, 4096 of 8192 blocks per plane: 2-6 % slower), because the jumps it
    // takes off the writes land on the reads of the staging buffer.  Kept as a switch so that
    // the benchmark can show the comparison.
    int32_t scatter_order = 0;
    int64_t ordered_min_pages = 1024, ordered_min_density_inv = 8;
    lmc::OrderScratch order{};         // device scratch of such launches, grown on demand
    uint64_t order_cap_tokens = 0;
    hipEvent_t order_free = nullptr;   // the last such launch has finished with the scratch
    std::vector<void *> order_retired; // outgrown scratch, freed with the context
    uint64_t use_calls = 0;         // number of the latest call that used chunks (recency of use)
    std::vector<uint64_t> evicted;  // LMC_FLAG_EVICT_LRU: ids evicted and not yet drained
    // Calls that move at most this many bytes skip staging and the copy engine: the kernel itself crosses the link.
    // That saves a small transfer launches and hand-overs and a long one 100 us, and takes 24 compute units for as
    // long as it lasts; staging makes two hardware queues (a load) or one (a store) besides the caller's stand still, and whatever
    // stream of the process happens to be in them.  So the lines depend on whether the caller has placed its streams
    // (lmc_probe_stream).  Figures: us for a transfer and products of 128, 512, 1536, 4096 rows by 4096 x 4096 beside
    // it, staged and direct.  lmc_tune "direct_store_below" / "direct_retrieve_below" set all lines of a direction; 0 = never.
    //
    // Stores, bulk: up to 64 MiB.  Alone 2-7 % faster; 96 and 128 MiB 3-4 %, but products over the four queues
    // they can be in 9-15 % slower.
    int64_t direct_store_below = int64_t(64) << 20;
    // Layer-wise stores: up to the same line (64 MiB in steps of 4, over the four queues: 9039, 9036, 10858, 14797
    // and 8678, 9060, 10866, 15002); if a stream has been found that stores do not hold up, steps of at most 2 MiB
    // (64 MiB there, in steps of 4: 2650, 1936, 2116, 3711 and 2313, 1711, 2252, 4384; of 2: 6075, 3204, 3233,
    // 3848 and 3139, 2312, 2565, 4143).
    int64_t direct_placed_store_below = 0;
    // Such steps up to 256 MiB (160 MiB in steps of 2 over the four queues: 15583, 15594, 19374, 28685 and 14302,
    // 15279, 19751, 28909; 192 MiB in steps of 6 would lose: 10085, 10105, 11891, 15773 and 9469, 10510, 12522, 16840),
    // and steps of any size where the producer has nothing on its stream and no other operation is under way, so
    // that there is nothing to slow down (86, 168, 224 MiB in steps of 6, 11, 7: 1878, 3339, 4544 and 1633, 3172, 4223).
    int64_t direct_store_steps_below = int64_t(256) << 20;
    static constexpr int64_t kDirectStoreStep = int64_t(2) << 20;
    static constexpr int64_t kStoreStepsInTurn = int64_t(512) << 10;   // see lmc_store_layers
    // Retrieves: up to 256 MiB (128 MiB over the four queues 4693, 4387, 4226, 4844 and 3626, 3833, 3795, 4046; the
    // load itself 2452 and 2341).
    int64_t direct_retrieve_below = int64_t(256) << 20;
    // Up to 64 MiB if a stream has been found that loads do not hold up: there, products beside 128 MiB take 3682,
    // 3360, 3123, 4168 and 3625, 3845, 3794, 4044, as much as 22 % more for a load that is 2-5 % faster.  And beside
    // a store that is under way: a kernel that reads the link while copies write it gets half of its rate (128 MiB
    // behind a store of 768 MiB 3.4 ms and 5.3, 64 MiB 2.0 and 4.2).
    int64_t direct_small_retrieve_below = int64_t(64) << 20;
    // Layer by layer a stage costs 10 us between two copies and 5-7 more for a rectangle besides, so small steps go
    // this way up to 512 MiB: of 8 MiB, or, where a stream has been found, of 3 (there, the consumer's products
    // between the layers, 96 MiB in steps of 3: 2931, 3054, 2484, 4234 and 2421, 2794, 2425, 4274; 128 in steps of
    // 4: 3907, 4052, 4168, 4387 and 3479, 3989, 4249, 4571; of 8: 3625, 3658, 3808, 3913 and 3463, 4003, 4235, 4454; in the
    // queues that a staged load holds up 4120-5700, 5730-6380 and 5560-6190 staged, and direct as above).
    int64_t direct_steps_below = int64_t(512) << 20;
    static constexpr int64_t kDirectRetrieveStep = int64_t(8) << 20, kPlacedRetrieveStep = int64_t(3) << 20;
    // Has lmc_probe_stream found a stream that staged loads, or stores, do not hold up?  Then the caller is taken to
    // have its other work there.  Not remembered: which.  Until the library's own streams are placed anew.
    bool loads_placed = false, stores_placed = false;
    int64_t chunk_bytes = 0;
    int64_t n_pool_slots = 0;
    uint8_t *pool = nullptr;
    uint8_t *pool_dev = nullptr;   // the pool's address as the GPU sees it (LMC_FLAG_DIRECT)
    bool has_device = false;
    lmc::ChunkIndex index;
    std::mutex mu;
    hipStream_t s_gather = nullptr, s_d2h = nullptr, s_h2d = nullptr, s_scatter = nullptr;
    // second copy streams: where consecutive transfers cannot be merged into one (layer
    // steps, scattered pool slots) they alternate between the two streams of their
    // direction, because back-to-back copies on one stream leave the link idle in between
    hipStream_t s_h2d2 = nullptr, s_d2h2 = nullptr;
    std::vector<hipStream_t> retired_streams;   // see arrange_streams; destroyed with the context, after the events
    Ring store_ring, load_ring;
    int32_t *bad_flag_host = nullptr, *bad_flag_dev = nullptr;
    // Words in device memory at which scatters from the pool count themselves off (lmc::Arrivals),
    // kWordStride bytes apart: kBulkWord for bulk retrieves, the others one for each step of a
    // layer-wise one.  The launches that use a word run one after the other, so a word only grows and
    // word_target[i], what it will have reached when everything launched so far is done, says
    // when the newest of them is.  Null where a stream cannot wait for a value.
    // kStoreWord is for bulk stores without staging, whose kernels pass its value on to
    // *stored_host: a thread that waits for such a store sees it there 5 us before the event
    // behind the kernel completes.
    // kStoreStepWord is for the steps of layer-wise stores that run on s_d2h2 (lmc_store_layers).
    // kFilledWord and kDoneWord are written by the streams themselves (hand_over) as groups of a bulk
    // retrieve reach the staging buffer, and as it ends.
    static constexpr int kBulkWord = LMC_MAX_LAYERS, kStoreWord = LMC_MAX_LAYERS + 1, kFilledWord = LMC_MAX_LAYERS + 2,
                         kDoneWord = LMC_MAX_LAYERS + 3, kStoreStepWord = LMC_MAX_LAYERS + 4, kWords = LMC_MAX_LAYERS + 5;
    // two words of host memory, kLoadedAt words apart, and their address on the GPU
    static constexpr int kLoadedAt = 8;
    uint64_t *stored_host = nullptr, *stored_dev = nullptr;
    bool is_stored(uint64_t target) const { return target != 0 && __atomic_load_n(stored_host, __ATOMIC_ACQUIRE) >= target; }
    // A bulk load that runs on the caller's stream tells the host likewise, at kBulkWord and the second word: nothing
    // of the library's then waits for it, on no stream, unless something else is to use the scatter stream meanwhile
    // (scatters_behind: the value that stream has been made to wait for).
    bool is_loaded(uint64_t target) const { return target != 0 && __atomic_load_n(stored_host + kLoadedAt, __ATOMIC_ACQUIRE) >= target; }
    uint64_t scatters_behind = 0;
    uint64_t *words = nullptr;
    uint64_t word_target[kWords] = {};
    // May a stream be made to wait for a word (lmc_tune "value_waits")?  The runtime waits for a value,
    // and writes one, by a kernel: one wavefront that stays until the word is there.  Where two kernels
    // may run at once that is harmless, since whatever brings the word about has been enqueued before the
    // wait.  A tool that lets the GPU run one kernel at a time may start the waiting one first, for
    // good: rocprofv3 does while it collects counters, which it tells the program by this variable.
    static bool kernels_run_one_by_one() {
        const char *v = std::getenv("ROCPROF_COUNTER_COLLECTION");
        return v != nullptr && *v != 0 && std::strcmp(v, "0") != 0;
    }
    bool value_waits = !kernels_run_one_by_one();
    bool can_wait_for_words() const { return words != nullptr && value_waits; }
    uint64_t *word(int i) const { return words + size_t(i) * (lmc::kWordStride / sizeof(uint64_t)); }
    std::deque<Op> ops;
    std::deque<Timing> timings;
    // LMC_FLAG_TRACE: finished steps, oldest first, at most kTraceCap; device time counts from trace_epoch
    std::deque<lmc_trace_rec_t> trace;
    uint64_t trace_dropped = 0;
    hipEvent_t trace_epoch = nullptr;
    uint64_t cur_ticket = 0;   // the operation whose steps are being enqueued (for the trace)
    uint64_t next_ticket = 1;
    std::vector<hipEvent_t> free_sync_events, free_time_events, all_events;
    // Threads that sleep in hipEventSynchronize with the mutex released.  While there are
    // any, events that become free are parked in held_events instead of going back to the
    // free list: an event somebody sleeps on is then never recorded anew under them.
    int waiters = 0;
    std::vector<hipEvent_t> held_events;
    // Test hook (lmc_tune "fail_hip_after"): the n-th checked HIP call from now is not made
    // and counts as failed.  Forces the error paths without any fault on the device.
    uint32_t fail_hip_after = 0;
    // and two others ("expect_stores_told", "expect_groups_staged"): stores that the host was told the end of by
    // the word, and groups of stores that went through a staging buffer
    uint64_t stores_told = 0, groups_staged = 0;
    lmc_stats_t stats{};
    int32_t last_hip_error = 0;
};

namespace lmci {

// A failed HIP call is reported through the library's own status and
// lmc_last_hip_error(); the runtime's per-thread "last error" is cleared so that it does
// not surface in the caller's next, unrelated HIP call.
inline bool injected_failure(lmc_ctx *c) {
    return c->fail_hip_after > 0 && --c->fail_hip_after == 0;
}

#define HIPCHK(ctx, expr)                                  \
    do {                                                   \
        hipError_t e_ = injected_failure(ctx) ? hipErrorUnknown : (expr); \
        if (e_ != hipSuccess) {                            \
            (ctx)->last_hip_error = int32_t(e_);           \
            (void)hipGetLastError();                       \
            return LMC_ERR_HIP;                            \
        }                                                  \
    } while (0)

// Makes the context's device current for the scope of one API call.
class DeviceScope {
public:
    explicit DeviceScope(const lmc_ctx *c) {
        if (c->has_device && hipGetDevice(&prev_) == hipSuccess && prev_ != c->cfg.device) {
            if (hipSetDevice(c->cfg.device) == hipSuccess) restore_ = true;
        }
    }
    ~DeviceScope() {
        if (restore_) (void)hipSetDevice(prev_);
    }

private:
    int prev_ = 0;
    bool restore_ = false;
};

// The mapped flag block holds 16 words: word 0 is set by the gather / scatter kernels on a
// slot outside the pages, word kCheckWord by the check kernel of LMC_FLAG_VALIDATE_SLOTS.
constexpr int kCheckWord = 8;
constexpr size_t kTraceCap = size_t(1) << 16;

// lmc_ctx.cpp
lmc_status_t get_event(lmc_ctx *c, bool timing, hipEvent_t *out);
lmc_status_t build_layer_ptrs(const lmc_ctx *c, void *const *kv_layers, lmc::LayerPtrs *out);
Op *find_op(lmc_ctx *c, uint64_t ticket);
double seconds_now(const lmc_ctx *c);
void recycle(lmc_ctx *c, hipEvent_t e);
void reap(lmc_ctx *c);
lmc_status_t order_after(lmc_ctx *c, hipStream_t waiter, hipStream_t stream);
bool caller_is_idle(hipStream_t user);
lmc_status_t order_after_caller(lmc_ctx *c, hipStream_t waiter, hipStream_t user);
bool other_direction_busy(lmc_ctx *c, bool for_store);
lmc_status_t validate_slots(lmc_ctx *c, const int64_t *slot_mapping, int64_t n_tokens,
                            hipStream_t stream);
lmc_status_t force_sync(lmc_ctx *c, hipStream_t s);
lmc_status_t trace_begin(lmc_ctx *c, hipStream_t stream, hipEvent_t *start);
lmc_status_t trace_end(lmc_ctx *c, hipStream_t stream, hipEvent_t start, int32_t stage, int64_t chunks, uint64_t bytes);
void begin_use(lmc_ctx *c, const uint64_t *ids, int64_t n);
void end_use(lmc_ctx *c, const uint64_t *ids, int64_t n);
int64_t take_slot(lmc_ctx *c, uint64_t id);
lmc_status_t free_ring(Ring &r);
lmc_status_t make_ring(lmc_ctx *c, Ring &r);
// lmc_pipeline.cpp
lmc_status_t timed_launch(lmc_ctx *c, bool gather, const lmc::LaunchView &view,
                          const lmc::LayerPtrs &ptrs, const int64_t *slots, uint32_t n_chunks,
                          uint8_t *staging, hipStream_t stream, const lmc::ChunkList *list = nullptr,
                          hipEvent_t stop = nullptr, lmc::Arrivals *arrivals = nullptr, uint32_t planes_per_step = 0,
                          lmc::HostWord *told = nullptr, uint32_t groups = 0);
lmc_status_t scatters_after_loads(lmc_ctx *c);
// lmc_streams.cpp
lmc_status_t shares_a_queue(lmc_ctx *c, hipStream_t busy, bool by_kernel, hipStream_t other, uint8_t *devbuf,
                            uint64_t nbytes, hipEvent_t a0, hipEvent_t a1, hipEvent_t k1, bool *shares);
void arrange_streams(lmc_ctx *c);
// lmc_static.cpp
hipError_t resolve_static_scratch(int device);
uint8_t *static_scratch_of(int device);

}  // namespace lmci

#endif  // LMC_CTX_HPP
