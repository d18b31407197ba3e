// liblmc: the store and retrieve pipelines (see include/lmc.h for the contract).
//
// Store  (paper sections 4 and 5.1): index probe -> per group of new chunks
//        gather kernel (stream G) -> event -> hipMemcpyAsync D2H into pool slots
//        (stream D) -> event that releases the staging buffer.
// Retrieve: hipMemcpyAsync H2D of the hit chunks (stream H) -> event -> scatter kernel
//        (stream S) -> event that releases the staging buffer.
// Each direction owns a ring of num_staging buffers, so the kernel of group k+1 runs
// while the copy of group k is on the link (section 1 (#1): storing and loading are
// batched and pipelined).  The host never waits inside store / retrieve; control
// crosses to the device once per group and direction, not once per page, which is
// the paper's argument for chunk-granular transfers (section 8.6, Table 5).
#include "lmc_ctx.hpp"

namespace lmci {

// Does this scatter launch go in the order of the destination?  It pays when the launch
// finds neighbours among its pages: many pages per plane, and a fair share of the plane.
static bool use_ordered_scatter(const lmc_ctx *c, const lmc::LaunchView &view, uint64_t n_tokens) {
    if (c->scatter_order == 0 || !lmc::ordered_scatter_fits(c->kg, view, c->shape, n_tokens)) return false;
    if (c->scatter_order >= 2) return true;
    const int64_t pages = int64_t(n_tokens) / c->cfg.geom.block_size;
    return pages >= c->ordered_min_pages && pages * c->ordered_min_density_inv >= int64_t(c->cfg.geom.num_blocks);
}

// The scratch of an ordered launch: allocated when first needed, grown when a launch has
// more tokens than any before (the outgrown arrays may still be in use by a launch under
// way and are kept until the context goes).  `stream` is made to wait for the previous
// ordered launch, which may have run on another stream: one set serves one launch at a time.
static lmc_status_t prepare_order_scratch(lmc_ctx *c, uint64_t n_tokens, hipStream_t stream) {
    auto alloc = [&](void **p, uint64_t bytes) -> lmc_status_t {
        const hipError_t e = injected_failure(c) ? hipErrorOutOfMemory : hipMalloc(p, bytes);
        if (e != hipSuccess) {
            *p = nullptr;
            c->last_hip_error = int32_t(e);
            (void)hipGetLastError();
            return e == hipErrorOutOfMemory ? LMC_ERR_NOMEM : LMC_ERR_HIP;
        }
        return LMC_OK;
    };
    lmc_status_t rc = LMC_OK;
    if (c->order.token_at == nullptr) {
        void *a = nullptr, *b = nullptr, *n = nullptr;
        rc = alloc(&a, lmc::order_table_words(c->kg) * 4);
        if (rc == LMC_OK) rc = alloc(&b, lmc::order_count_words(c->kg) * 4);
        if (rc == LMC_OK) rc = alloc(&n, 256);
        if (rc == LMC_OK) rc = get_event(c, false, &c->order_free);
        if (rc != LMC_OK) {
            for (void *p : {a, b, n})
                if (p) (void)hipFree(p);
            return rc;
        }
        c->order.token_at = static_cast<uint32_t *>(a);
        c->order.counts = static_cast<uint32_t *>(b);
        c->order.n_rows = static_cast<uint32_t *>(n);
    } else if (c->order_cap_tokens > 0) {
        HIPCHK(c, hipStreamWaitEvent(stream, c->order_free, 0));
    }
    if (n_tokens > c->order_cap_tokens) {
        void *p = nullptr;
        const uint64_t cap = std::max<uint64_t>(n_tokens, 2 * c->order_cap_tokens);
        if ((rc = alloc(&p, cap * 8)) != LMC_OK) return rc;
        if (c->order.pairs != nullptr) c->order_retired.push_back(c->order.pairs);
        c->order.pairs = static_cast<uint2 *>(p);
        c->order_cap_tokens = cap;
    }
    return LMC_OK;
}

lmc_status_t timed_launch(lmc_ctx *c, bool gather, const lmc::LaunchView &view,
                          const lmc::LayerPtrs &ptrs, const int64_t *slots, uint32_t n_chunks,
                          uint8_t *staging, hipStream_t stream, const lmc::ChunkList *list, hipEvent_t stop,
                          lmc::Arrivals *arrivals, uint32_t planes_per_step, lmc::HostWord *told, uint32_t groups) {
    // LMC_FLAG_TIMING: the launch itself carries a start and a stop event, which receive
    // the kernel's own begin / end time stamps; the stream gets no extra marker.
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (c->cfg.flags & (LMC_FLAG_TIMING | LMC_FLAG_TRACE)) {
        lmc_status_t rc = get_event(c, true, &e0);
        if (rc == LMC_OK) rc = get_event(c, true, &e1);
        if (rc != LMC_OK) return rc;
    }
    lmc::LaunchShape s = c->shape;
    // a launch that reads or writes the pinned pool itself is paced by the host link
    if (c->pool_dev != nullptr && staging >= c->pool_dev &&
        staging < c->pool_dev + uint64_t(c->n_pool_slots) * uint64_t(c->chunk_bytes))
        s.paced_groups = groups != 0 && c->link_groups != 0 ? groups : c->link_groups;
    // `stop` completes with the launch: as the launch's own stop event, which costs the GPU and
    // the calling thread 3 and 1 us less than an event recorded behind it, unless timing needs that
    // or the stream is being captured, where waits go by the events recorded on it
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    const bool own_stop = stop != nullptr && e1 == nullptr && hipStreamIsCapturing(stream, &capturing) == hipSuccess &&
                          capturing == hipStreamCaptureStatusNone;
    const hipEvent_t end = own_stop ? stop : e1;
    const uint64_t moved = uint64_t(n_chunks) * view.by_n_lp.d * c->kg.plane_bytes;
    const uint64_t n_tokens = uint64_t(n_chunks) * c->kg.chunk_tokens;
    const bool ordered = !gather && s.paced_groups == 0 && use_ordered_scatter(c, view, n_tokens);
    if (ordered) {
        const lmc_status_t rc = prepare_order_scratch(c, n_tokens, stream);
        if (rc != LMC_OK) {
            if (e0 != nullptr) {
                c->free_time_events.push_back(e0);
                c->free_time_events.push_back(e1);
            }
            return rc;
        }
    }
    hipError_t e =
        injected_failure(c) ? hipErrorUnknown
        : gather  ? lmc::launch_gather(c->kg, view, s, ptrs, slots, n_chunks, staging, c->bad_flag_dev, stream, e0, end, list, told)
        : ordered ? lmc::launch_scatter_ordered(c->kg, view, s, ptrs, slots, uint32_t(n_tokens), c->order, staging,
                                                c->bad_flag_dev, stream, e0, end)
                  : lmc::launch_scatter(c->kg, view, s, ptrs, slots, n_chunks, staging, c->bad_flag_dev, stream, e0, end, list,
                                        arrivals, planes_per_step);
    if (ordered && e == hipSuccess) e = hipEventRecord(c->order_free, stream);
    if (stop != nullptr && !own_stop && e == hipSuccess) e = hipEventRecord(stop, stream);
    if (e != hipSuccess) {
        if (e0 != nullptr) {
            c->free_time_events.push_back(e0);
            c->free_time_events.push_back(e1);
        }
        HIPCHK(c, e);
    }
    if (gather) {
        c->stats.gather_launches++;
        c->stats.bytes_gathered += moved;
    } else {
        c->stats.scatter_launches++;
        c->stats.bytes_scattered += moved;
    }
    if (e0 != nullptr)
        c->timings.push_back(Timing{e0, e1, gather ? LMC_STAGE_GATHER : LMC_STAGE_SCATTER, c->cur_ticket, int32_t(n_chunks), moved});
    return LMC_OK;
}

// Copies `width` bytes per chunk between staging (chunks `stride` bytes apart) and the
// pool (offset `pool_off` inside each slot), one transfer per run of consecutive pool
// slots: a plain copy when the extents are back to back on both sides (whole chunks),
// else a rectangle copy whose rows are the chunks (layer-wise mode).  With a second
// stream the runs go to the two streams in turn; *used_second says whether any did.
static lmc_status_t copy_group(lmc_ctx *c, bool to_host, uint8_t *staging, uint64_t stride,
                        const int64_t *pool_slots, int64_t k, uint64_t pool_off, uint64_t width,
                        hipStream_t first, hipStream_t second = nullptr, bool *used_second = nullptr) {
    const uint64_t cb = uint64_t(c->chunk_bytes);
    const hipMemcpyKind kind = to_host ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice;
    if (used_second) *used_second = false;
    // Many small pieces (a fragmented pool in layer-wise mode: one piece per chunk and step,
    // 1 MiB for one Llama layer): the runtime pays a fixed price per copy that a piece this
    // small does not cover (stores of 1 MiB pieces ran at 27-36 GB/s), so all pieces of the
    // group go in one launch of the library's copy kernel, which is told the slots.
    if (c->pool_dev != nullptr && k > 1 && width <= c->pieces_by_kernel_below &&
        ((width | stride | cb | pool_off | reinterpret_cast<uintptr_t>(staging)) % 16) == 0 &&
        c->n_pool_slots <= int64_t(INT32_MAX)) {
        int64_t runs = 1;
        for (int64_t j = 1; j < k; j++) runs += pool_slots[j] != pool_slots[j - 1] + 1;
        if (uint64_t(k) * width <= uint64_t(runs) * c->pieces_by_kernel_below && runs > 1) {
            const uint32_t groups = c->link_groups ? c->link_groups : 64u;
            for (int64_t j = 0; j < k; j += lmc::kMaxPieces) {
                const int64_t m = std::min<int64_t>(lmc::kMaxPieces, k - j);
                lmc::PieceSlots table;
                for (int64_t i = 0; i < m; i++) table.slot[i] = int32_t(pool_slots[j + i]);
                HIPCHK(c, lmc::launch_copy_pieces(c->pool_dev + pool_off, cb, staging + uint64_t(j) * stride, stride,
                                                  width, table, uint32_t(m), to_host, groups, c->shape.paced_lds, first));
            }
            if (to_host) c->stats.bytes_d2h += uint64_t(k) * width;
            else c->stats.bytes_h2d += uint64_t(k) * width;
            return LMC_OK;
        }
    }
    bool watched = false;
    int64_t run = 0;
    for (int64_t j = 0; j < k; run++) {
        int64_t m = 1;
        while (j + m < k && pool_slots[j + m] == pool_slots[j] + m) m++;
        hipStream_t stream = first;
        const bool wanted = ((c->copy_kernel >> (to_host ? 0 : 1)) & 1u) != 0 ||
                            (to_host && c->d2h_guard_on && c->d2h_guard.use_kernel(seconds_now(c)));
        const bool by_kernel = wanted && c->pool_dev != nullptr &&
                               ((width | stride | cb | pool_off | reinterpret_cast<uintptr_t>(staging)) % 16) == 0;
        if (by_kernel) {
            // launches follow each other without a gap: one stream is enough
            uint8_t *pool_at = c->pool_dev + uint64_t(pool_slots[j]) * cb + pool_off;
            uint8_t *stage_at = staging + uint64_t(j) * stride;
            const uint32_t groups = c->link_groups ? c->link_groups : 64u;
            if (to_host) HIPCHK(c, lmc::launch_copy_rect(pool_at, cb, stage_at, stride, width, uint64_t(m), true, groups, c->shape.paced_lds, stream));
            else HIPCHK(c, lmc::launch_copy_rect(stage_at, stride, pool_at, cb, width, uint64_t(m), false, groups, c->shape.paced_lds, stream));
            if (to_host) c->stats.bytes_d2h += uint64_t(m) * width;
            else c->stats.bytes_h2d += uint64_t(m) * width;
            j += m;
            continue;
        }
        if (second != nullptr && (run & 1)) {
            stream = second;
            if (used_second) *used_second = true;
        }
        uint8_t *host = c->pool + uint64_t(pool_slots[j]) * cb + pool_off;
        uint8_t *dev = staging + uint64_t(j) * stride;
        // one large copy to the host per group is timed for the guard (two markers around
        // milliseconds of copy; one per group, so that a group of many copies keeps its pace)
        CopyTiming watch{nullptr, nullptr, uint64_t(m) * width};
        if (to_host && c->d2h_guard_on && !watched && watch.bytes >= lmc::CopyEngineGuard::kMinBytes &&
            get_event(c, true, &watch.start) == LMC_OK) {
            if (get_event(c, true, &watch.stop) != LMC_OK) {
                c->free_time_events.push_back(watch.start);
                watch.start = nullptr;
            } else {
                HIPCHK(c, hipEventRecord(watch.start, stream));
            }
        }
        if (m == 1 || (width == cb && stride == cb)) {
            if (to_host) HIPCHK(c, hipMemcpyAsync(host, dev, size_t(uint64_t(m) * width), kind, stream));
            else HIPCHK(c, hipMemcpyAsync(dev, host, size_t(uint64_t(m) * width), kind, stream));
        } else {
            hipError_t e = to_host ? hipMemcpy2DAsync(host, cb, dev, stride, width, size_t(m), kind, stream)
                                   : hipMemcpy2DAsync(dev, stride, host, cb, width, size_t(m), kind, stream);
            if (e == hipErrorInvalidPitchValue || e == hipErrorInvalidValue) {
                // a pitch the runtime does not take: one plain copy per chunk instead
                (void)hipGetLastError();
                for (int64_t i = 0; i < m; i++) {
                    if (to_host) HIPCHK(c, hipMemcpyAsync(host + uint64_t(i) * cb, dev + uint64_t(i) * stride, size_t(width), kind, stream));
                    else HIPCHK(c, hipMemcpyAsync(dev + uint64_t(i) * stride, host + uint64_t(i) * cb, size_t(width), kind, stream));
                }
            } else {
                HIPCHK(c, e);
            }
        }
        if (watch.start != nullptr) {
            HIPCHK(c, hipEventRecord(watch.stop, stream));
            c->copy_timings.push_back(watch);
            watched = true;
        }
        if (to_host) c->stats.bytes_d2h += uint64_t(m) * width;
        else c->stats.bytes_h2d += uint64_t(m) * width;
        j += m;
    }
    return LMC_OK;
}

// True if the pool slots are not one run of consecutive numbers (more than one transfer).
static bool several_runs(const int64_t *pool_slots, int64_t k) {
    for (int64_t j = 1; j < k; j++)
        if (pool_slots[j] != pool_slots[j - 1] + 1) return true;
    return false;
}

// Registers the operation: from here on reap() gives back what it holds.  On an error
// nothing has been registered and `op` is still the caller's.
static lmc_status_t finish_op(lmc_ctx *c, Op &&op, hipStream_t last_stream, bool enqueued,
                       uint64_t *ticket_out) {
    if (enqueued) {
        lmc_status_t rc = get_event(c, false, &op.done);
        if (rc != LMC_OK) return rc;
        const hipError_t e = injected_failure(c) ? hipErrorUnknown : hipEventRecord(op.done, last_stream);
        if (e != hipSuccess) {
            c->free_sync_events.push_back(op.done);
            op.done = nullptr;
            HIPCHK(c, e);
        }
    }
    op.final_stream = last_stream;
    if (ticket_out) *ticket_out = op.ticket;
    c->ops.push_back(std::move(op));
    return LMC_OK;
}

// Switch the ring to slots of slot_bytes.  When the size changes, the producer stream
// first waits for everything the consumer stream has been given, so no slot of the old
// division is still being read when the new division is written.
static lmc_status_t ring_reslot(lmc_ctx *c, Ring &r, uint64_t slot_bytes, hipStream_t producer,
                         hipStream_t consumer, hipStream_t producer2 = nullptr, hipStream_t consumer2 = nullptr) {
    if (slot_bytes == r.slot_bytes) return LMC_OK;
    if (r.slot_bytes != 0) {
        lmc_status_t rc = order_after(c, producer, consumer);
        if (rc == LMC_OK && producer2 != nullptr) rc = order_after(c, producer2, consumer);
        if (rc == LMC_OK && consumer2 != nullptr) rc = order_after(c, producer, consumer2);
        if (rc != LMC_OK) return rc;
    }
    // the new division takes effect only when its events exist: a failure on the way
    // leaves the ring as it was
    const uint32_t per_buf = uint32_t(std::max<uint64_t>(1, std::min<uint64_t>(r.buf_bytes / slot_bytes, 32)));
    const size_t total = r.buf.size() * per_buf;
    while (r.filled.size() < total || r.drained.size() < total) {
        std::vector<hipEvent_t> &v = r.filled.size() < total ? r.filled : r.drained;
        hipEvent_t e;
        lmc_status_t rc = get_event(c, false, &e);
        if (rc != LMC_OK) return rc;
        v.push_back(e);
    }
    r.slot_bytes = slot_bytes;
    r.slots_per_buf = per_buf;
    r.used.assign(total, 0);
    r.pos = 0;
    return LMC_OK;
}

// Next slot in turn: its index (for the events) and its address.
static size_t ring_next(Ring &r, uint8_t **ptr) {
    const size_t total = r.buf.size() * r.slots_per_buf;
    const size_t idx = size_t(r.pos++ % total);
    *ptr = r.buf[idx / r.slots_per_buf] + uint64_t(idx % r.slots_per_buf) * r.slot_bytes;
    return idx;
}

// Layer-wise mode: how many chunks' share of `view` one group (one slot, one launch) takes.
static int64_t layer_group_chunks(const lmc_ctx *c, const Ring &r, const lmc::LaunchView &view, int64_t n_chunks) {
    const int64_t fit = int64_t(r.buf_bytes / view.chunk_stride);
    return std::max<int64_t>(1, std::min({n_chunks, fit, int64_t(lmc::max_chunks_per_launch(c->kg, view))}));
}

// A chunk whose store is still on its way to the pool must be loaded after that store:
// the loading stream waits for the event behind the copies of the store's group that holds
// the chunk (a staged bulk store records one per group, so that a retrieve issued right
// behind a store of the same chunks follows it group by group, both directions of the
// link at work), or else for the store's last event (stores end on different streams, the
// D2H stream or, without staging, the gather stream, so the newest alone says nothing
// about the others).  A layer-wise store that has not been submitted completely cannot
// be waited for on the device: LMC_ERR_BUSY.
static lmc_status_t after_stores(lmc_ctx *c, const int64_t *pool_slots, int64_t n, hipStream_t waiter) {
    std::vector<hipEvent_t> events;
    for (int64_t i = 0; i < n; i++) {
        const lmc::SlotMeta &m = c->index.meta(pool_slots[i]);
        if (m.ready_ticket == 0) continue;
        const Op *o = find_op(c, m.ready_ticket);
        if (o == nullptr) continue;  // finished
        if (o->pending) return LMC_ERR_BUSY;
        hipEvent_t e = m.ready_event != nullptr ? static_cast<hipEvent_t>(m.ready_event) : o->done;
        if (e != nullptr && std::find(events.begin(), events.end(), e) == events.end()) events.push_back(e);
    }
    for (hipEvent_t e : events) HIPCHK(c, hipStreamWaitEvent(waiter, e, 0));
    return LMC_OK;
}

// The part of n chunks that `view` describes, moved between the pages and the chunks' pool
// slots by kernels that cross the link themselves (no staging, no copy engine).  Chunk i is
// chunk `chunk[i]` of the slot mapping (null: i); one launch covers chunks that are
// consecutive there.  Where their pool slots are consecutive too the first one's address is
// all a launch needs; where they are not they are listed, so that a fragmented pool costs one
// launch for every kMaxListed chunks and not one for every run of slots.
// stop (may be null): completes with the last launch.  arrivals (may be null): the word at which the
// last launch of a scatter counts itself off, told (likewise) that of a gather; the others are over
// when it begins.
static lmc_status_t move_direct(lmc_ctx *c, bool gather, lmc::LaunchView view, uint64_t pool_off,
                                const lmc::LayerPtrs &ptrs, const int64_t *slot_mapping, const int64_t *chunk,
                                const int64_t *pool_slot, int64_t n, hipStream_t stream, hipEvent_t stop = nullptr,
                                lmc::Arrivals *arrivals = nullptr, lmc::HostWord *told = nullptr, uint32_t groups = 0) {
    const uint64_t cb = uint64_t(c->chunk_bytes);
    const int64_t CT = c->cfg.geom.chunk_tokens;
    view.chunk_stride = cb;  // chunks lie one pool slot apart
    const int64_t max_k = int64_t(lmc::max_chunks_per_launch(c->kg, view));
    // "link_groups" 0 asks for launches of one tile per workgroup, which take no list
    const bool may_list = c->link_groups > 0 && c->n_pool_slots <= INT32_MAX;
    int64_t map_end = 0;   // chunks i0 .. map_end - 1 are consecutive in the mapping; found once for all of them
    for (int64_t i0 = 0, k = 0; i0 < n; i0 += k) {
        if (map_end <= i0)
            for (map_end = i0 + 1; map_end < n && (!chunk || chunk[map_end] == chunk[map_end - 1] + 1);) map_end++;
        const int64_t in_map = std::min(max_k, map_end - i0);
        for (k = 1; k < in_map && pool_slot[i0 + k] == pool_slot[i0] + k;) k++;
        lmc::ChunkList list;
        const bool listed = may_list && k < in_map && k < lmc::kMaxListed;
        if (listed) {
            k = std::min<int64_t>(lmc::kMaxListed, in_map);
            for (int64_t i = 0; i < k; i++) list.slot[i] = int32_t(pool_slot[i0 + i]);
        }
        lmc_status_t rc = timed_launch(c, gather, view, ptrs, slot_mapping + (chunk ? chunk[i0] : i0) * CT, uint32_t(k),
                                       c->pool_dev + (listed ? 0 : uint64_t(pool_slot[i0]) * cb) + pool_off, stream,
                                       listed ? &list : nullptr, i0 + k == n ? stop : nullptr,
                                       i0 + k == n ? arrivals : nullptr, 0, i0 + k == n ? told : nullptr, groups);
        if (rc != LMC_OK) return rc;
        (gather ? c->stats.bytes_d2h : c->stats.bytes_h2d) += uint64_t(k) * view.by_n_lp.d * c->kg.plane_bytes;
        if ((rc = force_sync(c, stream)) != LMC_OK) return rc;
    }
    return LMC_OK;
}

static bool is_capturing(hipStream_t stream) {
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    const bool no = hipStreamIsCapturing(stream, &capturing) == hipSuccess && capturing == hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return !no;
}

// Can `stream` wait for a word of the context's (lmc_ctx::words)?  Not with "value_waits" 0, while it is
// being captured (the wait is no part of a graph), nor from another GPU.
static bool may_wait_for_word(const lmc_ctx *c, hipStream_t stream) {
    hipDevice_t dev = c->cfg.device;
    const bool ok = c->can_wait_for_words() && !is_capturing(stream) &&
                    (stream == nullptr || stream == hipStreamPerThread || hipStreamGetDevice(stream, &dev) == hipSuccess) &&
                    dev == c->cfg.device;
    (void)hipGetLastError();
    return ok;
}

// Does a store without staging tell the host through a word that it has ended?  Not where its launches
// are timed or traced: the word is there 5 us before a launch's stop event, and what a thread has waited
// for is to be in the statistics and the trace.
static bool tells_host(const lmc_ctx *c) {
    return c->words != nullptr && (c->cfg.flags & (LMC_FLAG_TIMING | LMC_FLAG_TRACE)) == 0 && !is_capturing(c->s_gather);
}

static lmc_status_t wait_for_word(lmc_ctx *c, hipStream_t stream, int word, uint64_t target) {
    HIPCHK(c, hipStreamWaitValue64(stream, c->word(word), target, hipStreamWaitValueGte, ~uint64_t(0)));
    return LMC_OK;
}

// Behind a wait for a value that may be the last entry of a caller's stream, an event: asked whether a stream has
// work whose last entry is such a wait, the runtime takes 16 us and says yes however long ago that was over, and the
// next call then waits for it by another event, 14 us more. 0.5 MiB loaded layer by layer, three contexts in
// turn: 45 -> 21 us; a store of 0.5 MiB behind the wait for the last layer of another, to its end, 58 -> 25.
// The wait is the newest of the ticket's, if that was made of this stream and there is no event yet.
static lmc_status_t event_behind_wait(lmc_ctx *c, Op *op, hipStream_t user) {
    if (!op->waits_last || op->waiter != user || is_capturing(user)) return LMC_OK;
    hipEvent_t e = nullptr;
    const lmc_status_t rc = get_event(c, false, &e);
    if (rc != LMC_OK) return rc;
    const hipError_t x = injected_failure(c) ? hipErrorUnknown : hipEventRecord(e, user);
    c->free_sync_events.push_back(e);
    HIPCHK(c, x);
    op->waits_last = false;
    return LMC_OK;
}

// Orders the scatter stream behind the bulk loads that run on a caller's stream and have not told yet.  They are all
// on one stream (launches_on_caller), so the newest's value is enough.
lmc_status_t scatters_after_loads(lmc_ctx *c) {
    uint64_t newest = 0;
    for (const Op &o : c->ops)
        if (!c->is_loaded(o.loaded_target)) newest = std::max(newest, o.loaded_target);
    if (newest <= c->scatters_behind) return LMC_OK;
    // What is outside a capture cannot be waited for inside.  No call gets here: a load tells only while the
    // scatter stream is not being captured, and the stream joins a capture behind this function; "value_waits"
    // is switched off behind it too.
    if (!may_wait_for_word(c, c->s_scatter)) return LMC_ERR_BUSY;
    const lmc_status_t rc = wait_for_word(c, c->s_scatter, lmc_ctx::kBulkWord, newest);
    if (rc == LMC_OK) c->scatters_behind = newest;
    return rc;
}

// Long waits of one stream for another.  A queue that stands waiting for an event polls a signal in
// host memory, over the link that the transfer it waits for is using: each such queue takes 0.6 % of
// the rate of a copy from the host and 0.25 % of one to it (1.25 GiB up: 57.2 GB/s with nobody waiting,
// 56.9, 56.55, 56.25 with one, two, three streams).  So the stream that is waited for writes a word in
// device memory behind its event, and the other waits for the word first and then for
// the event, which has completed by then: the event is what orders the two, the word only keeps the
// queue quiet.  What polls the word is a wavefront on a compute unit (lmc_ctx::value_waits), two of
// them for the length of a staged retrieve: on the scatter stream and on the caller's.  A word belongs to one stream, whose writes are in order.  Only retrieves use this: a
// store's gathers that wait for their buffers gain 0.1 % by it.
// hand_over: `stream` writes the word's next value, *at, or 0 where it cannot (capture).
static lmc_status_t hand_over(lmc_ctx *c, hipStream_t stream, int word, uint64_t *at) {
    *at = 0;
    if (!c->can_wait_for_words() || is_capturing(stream)) return LMC_OK;
    HIPCHK(c, hipStreamWriteValue64(stream, c->word(word), c->word_target[word] + 1, 0));
    *at = ++c->word_target[word];
    return LMC_OK;
}
static lmc_status_t wait_quietly(lmc_ctx *c, hipStream_t stream, int word, uint64_t at, hipEvent_t event) {
    if (at != 0 && may_wait_for_word(c, stream)) {
        lmc_status_t rc = wait_for_word(c, stream, word, at);
        if (rc != LMC_OK) return rc;
    }
    HIPCHK(c, hipStreamWaitEvent(stream, event, 0));
    return LMC_OK;
}

// All layers of n chunks into their pages, layers_per_step at a time, by one launch on the scatter
// stream (lmc::launch_scatter with planes_per_step); each step's layers are in place when its word says so.  *done:
// whether the transfer can go this way at all.  It cannot where the launch would have to be
// several (more chunks in scattered slots than a launch can list, "link_groups" 0), where each step
// is to have time stamps of its own or is to be waited for, or while the stream is being captured.
static lmc_status_t retrieve_in_steps(lmc_ctx *c, const lmc::LayerPtrs &ptrs, const int64_t *slot_mapping,
                                      const std::vector<int64_t> &pool_slots, int32_t layers_per_step, Op *op, bool *done) {
    const int64_t n = int64_t(pool_slots.size());
    const uint32_t planes = uint32_t(layers_per_step) * uint32_t(c->cfg.geom.num_planes);
    const lmc::LaunchView view = lmc::bulk_view(c->kg);
    const bool listed = several_runs(pool_slots.data(), n);
    *done = c->link_groups > 0 && n <= int64_t(lmc::max_chunks_per_launch(c->kg, view)) &&
            (!listed || (n <= lmc::kMaxListed && c->n_pool_slots <= INT32_MAX)) &&
            (c->cfg.flags & (LMC_FLAG_TIMING | LMC_FLAG_TRACE | LMC_FLAG_FORCE_SYNC)) == 0 && may_wait_for_word(c, c->s_scatter);
    if (!*done) return LMC_OK;
    lmc::ChunkList list;
    if (listed)
        for (int64_t i = 0; i < n; i++) list.slot[i] = int32_t(pool_slots[size_t(i)]);
    lmc::Arrivals arrivals{c->word(0), 0, nullptr, 0};
    const lmc_status_t rc = timed_launch(c, false, view, ptrs, slot_mapping, uint32_t(n),
                                         c->pool_dev + (listed ? 0 : pool_slots[0] * c->chunk_bytes), c->s_scatter,
                                         listed ? &list : nullptr, nullptr, &arrivals, planes);
    if (rc != LMC_OK) return rc;
    const int32_t steps = (c->cfg.geom.num_layers + layers_per_step - 1) / layers_per_step;
    op->step_layers = layers_per_step;
    for (int32_t i = 0; i < steps; i++) op->step_target.push_back(c->word_target[i] += arrivals.count);
    c->stats.scatter_launches += uint64_t(steps - 1);   // each step counts as a launch
    c->stats.bytes_h2d += uint64_t(n) * uint64_t(c->chunk_bytes);
    return LMC_OK;
}

// May the kernels of a bulk retrieve without staging be launched on the caller's own stream?
// They start after what is on it and it continues after them, which is the contract, and no
// event has to cross from that stream to the library's and back: those two hand-overs cost the
// calling thread 26 us (a query and a wait between streams are 12-14 us each on this runtime)
// and leave the link idle in between when one such retrieve follows another.  Call after call, three
// contexts in turn: 0.5 MiB 53 -> 36 us, 12 MiB in 256-byte rows 234 -> 223 us. The kernel tells the host
// when it is done; only where something of the library's has to wait for it on the device is the scatter
// stream made to wait for its word (scatters_after_loads), which else
// takes 4 us of the call and a hardware queue for as long as the transfer lasts (0.5 MiB 15.9 -> 9.5 us).
// What the runtime does for the first launch on a stream that has run nothing is done inside the call.
// Not while the stream is being captured, not for a stream of another GPU, and not where the caller's
// stream is not to wait ("caller_waits" 0), where the library itself waits before it launches
// (LMC_FLAG_VALIDATE_SLOTS) or where a launch leaves an event behind on its stream (timing,
// trace, and the scratch of ordered scatters, which "link_groups" 0 lets through).
// And not beside any transfer of the context's that is under way, other than retrieves that run
// on that same stream:
//   - retrieves into the same pages take effect in the order of the calls, which the scatter
//     stream sees to, and the caller's stream does not;
//   - the caller's stream may share a hardware queue with the gather stream or a copy stream of
//     a store, behind whose work the kernels would then wait: 8 MiB beside a store of 1 GiB that
//     takes 19 ms came back after 11-24 ms from such a stream, from the scatter stream after
//     0.2-1.1 ms, and whatever is issued next to the scatter stream would wait as long.
// hipStreamPerThread is one name for many streams, one a thread: the library's stream it is.
// A stream that is destroyed has finished its work (hipStreamDestroy blocks on this runtime), so a
// stream that takes the handle of a destroyed one has nothing to be ordered behind.
static lmc_status_t launches_on_caller(lmc_ctx *c, hipStream_t user, bool *yes) {
    *yes = false;
    if (!c->caller_waits || c->link_groups == 0 || user == hipStreamPerThread ||
        (c->cfg.flags & (LMC_FLAG_VALIDATE_SLOTS | LMC_FLAG_TIMING | LMC_FLAG_TRACE)) != 0)
        return LMC_OK;
    for (const Op &o : c->ops)   // what reap() has left
        if (!o.on_caller || o.caller != user) return LMC_OK;
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    const hipError_t e = injected_failure(c) ? hipErrorUnknown : hipStreamIsCapturing(user, &capturing);
    if (e == hipErrorStreamCaptureImplicit) {     // the null stream, while another is being captured
        (void)hipGetLastError();
        return LMC_OK;
    }
    HIPCHK(c, e);
    hipDevice_t dev = c->cfg.device;
    if (user != nullptr) HIPCHK(c, hipStreamGetDevice(user, &dev));
    *yes = capturing == hipStreamCaptureStatusNone && dev == c->cfg.device;
    return LMC_OK;
}

// Does a retrieve of this size skip staging (lmc_ctx::direct_retrieve_below and what follows it)?
static bool retrieves_directly(lmc_ctx *c, int64_t n_chunks, int32_t layers_per_step) {
    const int64_t bytes = n_chunks * c->chunk_bytes;
    const int64_t step = bytes / c->cfg.geom.num_layers * layers_per_step;
    const bool small_steps = layers_per_step > 0 && step <= (c->loads_placed ? lmc_ctx::kPlacedRetrieveStep : lmc_ctx::kDirectRetrieveStep);
    const int64_t line = c->loads_placed ? c->direct_small_retrieve_below : c->direct_retrieve_below;
    if (bytes > (small_steps ? std::max(c->direct_steps_below, line) : line)) return false;
    return bytes <= c->direct_small_retrieve_below || !other_direction_busy(c, false);
}

// Retrieve, bulk (layers_per_step == 0) or layer by layer (paper section 5.2).
static lmc_status_t do_retrieve(lmc_ctx *c, const uint64_t *ids, int64_t n_chunks,
                         const int64_t *slot_mapping, void *const *kv_layers, void *user_stream,
                         int32_t layers_per_step, uint64_t *ticket_out) {
    if (!c->has_device) return LMC_ERR_NODEVICE;
    DeviceScope dev(c);
    reap(c);
    std::vector<int64_t> pool_slots(size_t(n_chunks), 0);
    for (int64_t i = 0; i < n_chunks; i++) {
        pool_slots[size_t(i)] = c->index.find(ids[i]);
        if (pool_slots[size_t(i)] < 0) {
            c->stats.retrieve_misses++;
            return LMC_ERR_MISS;
        }
    }
    lmc::LayerPtrs ptrs;
    lmc_status_t rc = build_layer_ptrs(c, kv_layers, &ptrs);
    if (rc != LMC_OK) return rc;
    hipStream_t user = static_cast<hipStream_t>(user_stream);
    const lmc_kv_geom_t &geom = c->cfg.geom;
    const int64_t CT = geom.chunk_tokens;
    const bool direct = (c->cfg.flags & LMC_FLAG_DIRECT) != 0 || retrieves_directly(c, n_chunks, layers_per_step);
    bool on_caller = false;
    if (n_chunks > 0 && direct && layers_per_step == 0 && (rc = launches_on_caller(c, user, &on_caller)) != LMC_OK) return rc;
    hipStream_t scatters = on_caller ? user : c->s_scatter;
    // the pages may still be in use, and the slot mapping still be on its way, by work
    // already on the caller's stream
    if (n_chunks > 0 && !on_caller && (rc = scatters_after_loads(c)) != LMC_OK) return rc;
    if (n_chunks > 0 && !on_caller && (rc = order_after_caller(c, c->s_scatter, user)) != LMC_OK) return rc;
    rc = validate_slots(c, slot_mapping, n_chunks * CT, c->s_scatter);
    if (rc != LMC_OK) return rc;
    // without staging the scatters wait for every store at once; with staging each group's
    // copies wait for the stores of their own chunks (load_group)
    if ((rc = after_stores(c, pool_slots.data(), direct ? n_chunks : 0, scatters)) != LMC_OK) return rc;
    for (int64_t s : pool_slots) {
        const uint64_t t = c->index.meta(s).ready_ticket;
        const Op *o = t != 0 ? find_op(c, t) : nullptr;
        if (o != nullptr && o->pending) return LMC_ERR_BUSY;    // before anything is enqueued
    }
    begin_use(c, ids, n_chunks);   // a retrieve that is served is a use of its chunks
    end_use(c, ids, n_chunks);
    Op op;
    op.ticket = c->next_ticket++;
    c->cur_ticket = op.ticket;
    op.layerwise = layers_per_step > 0;
    op.on_caller = on_caller;
    op.caller = on_caller ? user : nullptr;
    if (n_chunks == 0) return finish_op(c, std::move(op), nullptr, false, ticket_out);

    Ring &ring = c->load_ring;
    const int64_t per = c->cfg.staging_chunks;
    // without staging (LMC_FLAG_DIRECT, or a small call): no copy, the scatter kernel reads the
    // pinned pool over the link
    auto load_direct = [&](const lmc::LaunchView &view, uint64_t pool_off, hipEvent_t stop, lmc::Arrivals *arrivals) {
        return move_direct(c, false, view, pool_off, ptrs, slot_mapping, nullptr, pool_slots.data(), n_chunks, scatters, stop,
                           arrivals);
    };
    // Long waits are quiet (hand_over) in bulk retrieves that have the link to themselves: the steps of a
    // layer-wise one are short, and take two copy streams in turn, and beside a store the write between
    // two copies costs more than the poll (5 GiB each way 96 GB/s in all with it, 99.9 without).  A store
    // that is issued behind the retrieve does not mind (99.4-99.6 with the words, 98.7-99.4 without).
    const bool two_copy_streams = !other_direction_busy(c, false);
    const bool quiet = !op.layerwise && two_copy_streams;
    bool by_word = false;   // the whole transfer is in place when the bulk word has reached its target
    // one group: copies into the next ring buffer on the H2D stream, scatter on the
    // scatter stream; the buffer is released when the scatter has read it
    auto load_group = [&](const lmc::LaunchView &view, uint64_t pool_off, int64_t i0, int64_t k,
                          hipStream_t copy_stream, hipStream_t second) -> lmc_status_t {
        uint8_t *buf;
        const size_t b = ring_next(ring, &buf);
        if (!several_runs(&pool_slots[size_t(i0)], k)) second = nullptr;
        lmc_status_t ra = after_stores(c, &pool_slots[size_t(i0)], k, copy_stream);
        if (ra == LMC_OK && second) ra = after_stores(c, &pool_slots[size_t(i0)], k, second);
        if (ra != LMC_OK) return ra;
        if (ring.used[b]) {
            HIPCHK(c, hipStreamWaitEvent(copy_stream, ring.drained[b], 0));
            if (second) HIPCHK(c, hipStreamWaitEvent(second, ring.drained[b], 0));
        }
        bool used_second = false;
        hipEvent_t traced = nullptr;
        lmc_status_t r = trace_begin(c, copy_stream, &traced);
        if (r != LMC_OK) return r;
        r = copy_group(c, false, buf, view.chunk_stride, &pool_slots[size_t(i0)], k,
                       pool_off, view.chunk_stride, copy_stream, second, &used_second);
        // the buffer is full when the copies of both streams are in
        if (r == LMC_OK && used_second) r = order_after(c, copy_stream, second);
        if (r != LMC_OK) {
            if (traced) c->free_time_events.push_back(traced);
            return r;
        }
        if ((r = trace_end(c, copy_stream, traced, LMC_STAGE_H2D, k, uint64_t(k) * view.by_n_lp.d * c->kg.plane_bytes)) != LMC_OK)
            return r;
        HIPCHK(c, hipEventRecord(ring.filled[b], copy_stream));
        // the copies of scattered chunks, two at a time, lose more to the write at the end of a group
        // than to the poll (20 x 8.6 MiB 3306 us without it, 3314 with it)
        uint64_t filled_at = 0;
        if (quiet && !used_second && (r = hand_over(c, copy_stream, lmc_ctx::kFilledWord, &filled_at)) != LMC_OK) return r;
        if ((r = force_sync(c, copy_stream)) != LMC_OK) return r;
        if ((r = wait_quietly(c, c->s_scatter, lmc_ctx::kFilledWord, filled_at, ring.filled[b])) != LMC_OK) return r;
        r = timed_launch(c, false, view, ptrs, slot_mapping + i0 * CT, uint32_t(k), buf, c->s_scatter);
        if (r != LMC_OK) return r;
        if (c->cfg.flags & LMC_FLAG_POISON_STAGING)
            HIPCHK(c, lmc::launch_fill(buf, 0xA5, uint64_t(k) * view.chunk_stride, c->s_scatter));
        HIPCHK(c, hipEventRecord(ring.drained[b], c->s_scatter));
        ring.used[b] = 1;
        return force_sync(c, c->s_scatter);
    };

    auto enqueue = [&]() -> lmc_status_t {
        if (direct && !op.layerwise) {
            lmc::Arrivals arrivals{nullptr, 0, nullptr, 0};
            hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
            HIPCHK(c, hipStreamIsCapturing(c->s_scatter, &capturing));
            const bool tells = c->can_wait_for_words() && c->link_groups > 0 && capturing == hipStreamCaptureStatusNone;
            if (tells) {
                arrivals.words = c->word(lmc_ctx::kBulkWord);
                arrivals.reached = c->word_target[lmc_ctx::kBulkWord];
                if (on_caller) arrivals.host = c->stored_dev + lmc_ctx::kLoadedAt;
            }
            rc = load_direct(lmc::bulk_view(c->kg), 0, nullptr, tells ? &arrivals : nullptr);
            c->word_target[lmc_ctx::kBulkWord] += arrivals.count;
            if (rc != LMC_OK) return rc;
            by_word = arrivals.count > 0;
            // an event is a matter of the library's own streams: the caller may
            // destroy its stream before the event is asked for
            if (on_caller && by_word) op.loaded_target = c->word_target[lmc_ctx::kBulkWord];
            else if (on_caller && (rc = order_after(c, c->s_scatter, user)) != LMC_OK) return rc;
        } else if (!op.layerwise) {
            const lmc::LaunchView view = lmc::bulk_view(c->kg);
            if ((rc = ring_reslot(c, ring, ring.buf_bytes, c->s_h2d, c->s_scatter, c->s_h2d2)) != LMC_OK) return rc;
            // The link is the bottleneck and every scatter but the last hides behind the next
            // copy, so the last group is a single chunk: only its scatter is exposed.
            const int64_t edge = std::min<int64_t>(c->edge_chunks, per);
            const int64_t body = (edge > 0 && n_chunks > edge) ? n_chunks - edge : n_chunks;
            for (int64_t i0 = 0, k = 0; i0 < n_chunks; i0 += k) {
                k = i0 < body ? std::min(per, body - i0) : n_chunks - i0;
                if ((rc = load_group(view, 0, i0, k, c->s_h2d, two_copy_streams ? c->s_h2d2 : nullptr)) != LMC_OK) return rc;
            }
        } else {
            if (direct) {
                bool done = false;
                if ((rc = retrieve_in_steps(c, ptrs, slot_mapping, pool_slots, layers_per_step, &op, &done)) != LMC_OK || done)
                    return rc;
            }
            // All chunks' share of a few layers at a time: one rectangle copy per run of pool
            // slots, one scatter launch, one event that says "these layers are in place".
            const int32_t L = geom.num_layers, P = geom.num_planes;
            const uint64_t layer_bytes = uint64_t(P) * c->kg.plane_bytes;
            op.layer_done.assign(size_t(L), nullptr);
            for (int32_t l0 = 0; l0 < L; l0 += layers_per_step) {
                const int32_t kk = std::min(layers_per_step, L - l0);
                const lmc::LaunchView view = lmc::layer_view(c->kg, uint32_t(P), uint32_t(l0), uint32_t(kk));
                hipEvent_t e;
                if ((rc = get_event(c, false, &e)) != LMC_OK) return rc;
                op.owned_events.push_back(e);
                if (direct) {
                    if ((rc = load_direct(view, uint64_t(l0) * layer_bytes, e, nullptr)) != LMC_OK) return rc;
                } else {
                    const int64_t cap = layer_group_chunks(c, ring, view, n_chunks);
                    if ((rc = ring_reslot(c, ring, (uint64_t(cap) * view.chunk_stride + 255) / 256 * 256, c->s_h2d,
                                          c->s_scatter, c->s_h2d2)) != LMC_OK)
                        return rc;
                    // Steps alternate between two copy streams: on one stream the runtime puts
                    // an event marker between consecutive copies, which costs the link about
                    // 20 us per step; with two streams the next step's copy is already running.
                    hipStream_t cs = (two_copy_streams && ((l0 / layers_per_step) & 1)) ? c->s_h2d2 : c->s_h2d;
                    for (int64_t i0 = 0; i0 < n_chunks; i0 += cap)
                        if ((rc = load_group(view, uint64_t(l0) * layer_bytes, i0, std::min(cap, n_chunks - i0), cs, nullptr)) != LMC_OK)
                            return rc;
                }
                if (!direct) HIPCHK(c, hipEventRecord(e, c->s_scatter));
                for (int32_t l = l0; l < l0 + kk; l++) op.layer_done[size_t(l)] = e;
            }
        }
        return LMC_OK;
    };
    op.slots = pool_slots;
    const bool layerwise = op.layerwise;
    if ((rc = enqueue()) == LMC_OK) rc = finish_op(c, std::move(op), c->s_scatter, op.loaded_target == 0, ticket_out);
    if (rc != LMC_OK) {
        // Part of the call may be enqueued and still read the pool slots, which nothing
        // protects (the in-flight counts belong to a registered operation): it is waited
        // for.  Pages the call was to fill are then in an unspecified state.
        for (hipStream_t s : {c->s_h2d, c->s_h2d2, c->s_scatter, scatters}) (void)hipStreamSynchronize(s);
        (void)hipGetLastError();
        for (hipEvent_t e : op.owned_events) recycle(c, e);
        return rc;
    }
    for (int64_t s : pool_slots) c->index.meta(s).inflight++;
    c->stats.chunks_retrieved += uint64_t(n_chunks);
    // bulk: the caller's stream continues when everything is in place; layer-wise: the
    // caller orders its streams per layer with lmc_wait_layer
    if (!layerwise && !on_caller && c->caller_waits) {
        if (by_word && may_wait_for_word(c, user))
            return wait_for_word(c, user, lmc_ctx::kBulkWord, c->word_target[lmc_ctx::kBulkWord]);
        uint64_t done_at = 0;
        if (quiet && (rc = hand_over(c, c->s_scatter, lmc_ctx::kDoneWord, &done_at)) != LMC_OK) return rc;
        return wait_quietly(c, user, lmc_ctx::kDoneWord, done_at, c->ops.back().done);
    }
    return LMC_OK;
}

// Token processor of a store: which chunks are new, and where they go.  Stops at the
// first chunk that finds no room.
static bool admit_new_chunks(lmc_ctx *c, const uint64_t *ids, int64_t n_chunks, Op *op,
                             std::vector<int64_t> *new_chunk) {
    bool fits = true;
    begin_use(c, ids, n_chunks);
    for (int64_t i = 0; i < n_chunks; i++) {
        if (c->index.find(ids[i]) >= 0) {
            c->stats.chunks_skipped_dup++;
            continue;
        }
        const int64_t s = take_slot(c, ids[i]);
        if (s < 0) {
            fits = false;
            break;
        }
        lmc::SlotMeta &m = c->index.meta(s);
        m.inflight = 1;
        m.ready_ticket = op->ticket;
        m.ready_event = nullptr;
        new_chunk->push_back(i);
        op->slots.push_back(s);
    }
    end_use(c, ids, n_chunks);
    return fits;
}

// A store that failed (a HIP error) after its chunks had been admitted.  What is already
// enqueued may still write the chunks' slots, so it is waited for; then the chunks leave
// the index again and their slots are free: no id stays behind that promises bytes which
// never arrived.  (Chunks that eviction removed to make room are not brought back.)
static void abort_store(lmc_ctx *c, const std::vector<int64_t> &slots) {
    for (hipStream_t s : {c->s_gather, c->s_d2h, c->s_d2h2}) (void)hipStreamSynchronize(s);
    (void)hipGetLastError();
    for (int64_t s : slots) c->index.erase(c->index.meta(s).id);
    c->stats.chunks_stored -= std::min<uint64_t>(c->stats.chunks_stored, slots.size());
    reap(c);
}

// Gather + D2H of the new chunks' part described by `view` (all layers, or a few),
// group by group through the store ring.
static lmc_status_t store_groups(lmc_ctx *c, const lmc::LaunchView &view, uint64_t pool_off,
                                 const lmc::LayerPtrs &ptrs, const int64_t *slot_mapping,
                                 const std::vector<int64_t> &new_chunk,
                                 const std::vector<int64_t> &new_slot, int64_t cap_chunks,
                                 bool edge_group, bool direct, bool layer_step = false, bool on_second_stream = false,
                                 std::vector<hipEvent_t> *group_events = nullptr, hipEvent_t stop = nullptr,
                                 lmc::HostWord *told = nullptr, uint32_t groups = 0) {
    Ring &ring = c->store_ring;
    const int64_t CT = c->cfg.geom.chunk_tokens;
    if (direct)   // no staging, no copy: the gather kernel writes the pinned pool over the link
        return move_direct(c, true, view, pool_off, ptrs, slot_mapping, new_chunk.data(), new_slot.data(),
                           int64_t(new_chunk.size()), on_second_stream ? c->s_d2h2 : c->s_gather, stop, nullptr, told, groups);
    const size_t per = size_t(cap_chunks);
    const bool two_copy_streams = !other_direction_busy(c, true);
    hipStream_t copies = on_second_stream ? c->s_d2h2 : c->s_d2h, other = on_second_stream ? c->s_d2h : c->s_d2h2;
    for (size_t j0 = 0; j0 < new_chunk.size();) {
        // one launch covers chunks that are consecutive in the caller's slot mapping.
        // Only the first gather is exposed (later ones hide behind the previous copy),
        // so the first group is a single chunk and the link starts working at once.
        const size_t edge = edge_group ? size_t(std::min<int64_t>(c->edge_chunks, int64_t(per))) : 0;
        const size_t cap = (j0 == 0 && edge > 0 && new_chunk.size() > edge) ? edge : per;
        size_t k = 1;
        while (k < cap && j0 + k < new_chunk.size() && new_chunk[j0 + k] == new_chunk[j0] + int64_t(k)) k++;
        uint8_t *buf;
        const size_t b = ring_next(ring, &buf);
        if (ring.used[b]) HIPCHK(c, hipStreamWaitEvent(c->s_gather, ring.drained[b], 0));
        lmc_status_t rc = timed_launch(c, true, view, ptrs, slot_mapping + new_chunk[j0] * CT, uint32_t(k),
                                       buf, c->s_gather);
        if (rc != LMC_OK) return rc;
        HIPCHK(c, hipEventRecord(ring.filled[b], c->s_gather));
        if ((rc = force_sync(c, c->s_gather)) != LMC_OK) return rc;
        HIPCHK(c, hipStreamWaitEvent(copies, ring.filled[b], 0));
        // a layer-wise step has the two streams step by step, not run by run (as the steps of a retrieve)
        hipStream_t second = (two_copy_streams && !(layer_step && c->store_step_streams == 2) && several_runs(&new_slot[j0], int64_t(k)))
                                 ? other : nullptr;
        if (second) HIPCHK(c, hipStreamWaitEvent(second, ring.filled[b], 0));
        bool used_second = false;
        hipEvent_t traced = nullptr;
        if ((rc = trace_begin(c, copies, &traced)) != LMC_OK) return rc;
        rc = copy_group(c, true, buf, view.chunk_stride, &new_slot[j0], int64_t(k), pool_off,
                        view.chunk_stride, copies, second, &used_second);
        // the group's copy stream stands for the whole group: it ends after the other stream's copies
        if (rc == LMC_OK && used_second) rc = order_after(c, copies, second);
        if (rc != LMC_OK) {
            if (traced) c->free_time_events.push_back(traced);
            return rc;
        }
        if ((rc = trace_end(c, copies, traced, LMC_STAGE_D2H, int64_t(k), uint64_t(k) * view.by_n_lp.d * c->kg.plane_bytes)) != LMC_OK)
            return rc;
        if (c->cfg.flags & LMC_FLAG_POISON_STAGING)
            HIPCHK(c, lmc::launch_fill(buf, 0xA5, uint64_t(k) * view.chunk_stride, copies));
        HIPCHK(c, hipEventRecord(ring.drained[b], copies));
        ring.used[b] = 1;
        c->groups_staged++;
        if (group_events != nullptr) {
            // "these chunks are in the pool": an event of the group's own (drained[b] is recorded
            // again whenever the buffer comes round), kept by the store until it is reaped
            hipEvent_t in_pool;
            if ((rc = get_event(c, false, &in_pool)) != LMC_OK) return rc;
            group_events->push_back(in_pool);
            HIPCHK(c, hipEventRecord(in_pool, copies));
            for (size_t j = j0; j < j0 + k; j++) c->index.meta(new_slot[j]).ready_event = in_pool;
        }
        if ((rc = force_sync(c, copies)) != LMC_OK) return rc;
        j0 += k;
    }
    return LMC_OK;
}

static lmc_status_t device_only(lmc_ctx_t *c, bool gather, void *const *kv_layers,
                                const int64_t *slot_mapping, int64_t n_chunks, uint8_t *staging,
                                void *stream) {
    if (!c || n_chunks < 0 || !kv_layers || (n_chunks > 0 && (!slot_mapping || !staging)))
        return LMC_ERR_INVAL;
    if (!c->has_device) return LMC_ERR_NODEVICE;
    if (reinterpret_cast<uintptr_t>(staging) % c->kg.align) return LMC_ERR_INVAL;
    std::lock_guard<std::mutex> lock(c->mu);
    c->cur_ticket = 0;
    DeviceScope dev(c);
    reap(c);
    lmc::LayerPtrs ptrs;
    lmc_status_t rc = build_layer_ptrs(c, kv_layers, &ptrs);
    if (rc != LMC_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t CT = c->cfg.geom.chunk_tokens;
    if ((rc = validate_slots(c, slot_mapping, n_chunks * CT, s)) != LMC_OK) return rc;
    const lmc::LaunchView view = lmc::bulk_view(c->kg);
    const int64_t per = int64_t(lmc::max_chunks_per_launch(c->kg, view));
    for (int64_t i0 = 0; i0 < n_chunks; i0 += per) {
        const int64_t k = std::min(per, n_chunks - i0);
        rc = timed_launch(c, gather, view, ptrs, slot_mapping + i0 * CT, uint32_t(k),
                          staging + i0 * c->chunk_bytes, s);
        if (rc != LMC_OK) return rc;
    }
    return LMC_OK;
}

}  // namespace lmci

using namespace lmci;

extern "C" {

lmc_status_t lmc_store(lmc_ctx_t *c, void *const *kv_layers, const int64_t *slot_mapping,
                       const uint64_t *ids, int64_t n_chunks, void *stream_to_wait_on,
                       uint64_t *ticket_out) {
    if (!c || n_chunks < 0 || !kv_layers || (n_chunks > 0 && (!slot_mapping || !ids)))
        return LMC_ERR_INVAL;
    if (!c->has_device) return LMC_ERR_NODEVICE;
    std::lock_guard<std::mutex> lock(c->mu);
    DeviceScope dev(c);
    reap(c);
    lmc::LayerPtrs ptrs;
    lmc_status_t rc = build_layer_ptrs(c, kv_layers, &ptrs);
    if (rc != LMC_OK) return rc;
    hipStream_t user = static_cast<hipStream_t>(stream_to_wait_on);
    const int64_t CT = c->cfg.geom.chunk_tokens;
    if (n_chunks > 0 && (rc = order_after_caller(c, c->s_gather, user)) != LMC_OK) return rc;
    if ((rc = validate_slots(c, slot_mapping, n_chunks * CT, c->s_gather)) != LMC_OK) return rc;

    Op op;
    op.ticket = c->next_ticket++;
    c->cur_ticket = op.ticket;
    std::vector<int64_t> new_chunk;
    const bool fits = admit_new_chunks(c, ids, n_chunks, &op, &new_chunk);
    c->stats.chunks_stored += new_chunk.size();
    const bool direct = (c->cfg.flags & LMC_FLAG_DIRECT) != 0 ||
                        int64_t(new_chunk.size()) * c->chunk_bytes <= c->direct_store_below;
    rc = direct ? LMC_OK : ring_reslot(c, c->store_ring, c->store_ring.buf_bytes, c->s_gather, c->s_d2h, nullptr, c->s_d2h2);
    if (rc == LMC_OK) {
        uint64_t &reached = c->word_target[lmc_ctx::kStoreWord];
        lmc::HostWord told{c->words ? c->word(lmc_ctx::kStoreWord) : nullptr, c->stored_dev, reached};
        const bool tells = direct && tells_host(c);
        rc = store_groups(c, lmc::bulk_view(c->kg), 0, ptrs, slot_mapping, new_chunk, op.slots,
                          c->cfg.staging_chunks, true, direct, false, false, &op.owned_events, nullptr, tells ? &told : nullptr);
        if (told.target != reached) op.stored_target = reached = told.target;
    }
    if (rc == LMC_OK)
        rc = finish_op(c, std::move(op), direct ? c->s_gather : c->s_d2h, !new_chunk.empty(), ticket_out);
    if (rc != LMC_OK) {
        abort_store(c, op.slots);   // finish_op registers as its last step: op is still whole
        for (hipEvent_t e : op.owned_events) recycle(c, e);
        return rc;
    }
    return fits ? LMC_OK : LMC_ERR_NOMEM;
}

lmc_status_t lmc_store_begin(lmc_ctx_t *c, const int64_t *slot_mapping, const uint64_t *ids,
                             int64_t n_chunks, void *stream_to_wait_on, uint64_t *ticket_out) {
    if (!c || n_chunks < 0 || (n_chunks > 0 && (!slot_mapping || !ids))) return LMC_ERR_INVAL;
    if (!c->has_device) return LMC_ERR_NODEVICE;
    std::lock_guard<std::mutex> lock(c->mu);
    DeviceScope dev(c);
    reap(c);
    lmc_status_t rc;
    hipStream_t user = static_cast<hipStream_t>(stream_to_wait_on);
    const int64_t CT = c->cfg.geom.chunk_tokens;
    const bool idle = n_chunks == 0 || caller_is_idle(user);
    if (!idle && (rc = order_after(c, c->s_gather, user)) != LMC_OK) return rc;
    if ((rc = validate_slots(c, slot_mapping, n_chunks * CT, c->s_gather)) != LMC_OK) return rc;
    Op op;
    op.ticket = c->next_ticket++;
    op.layerwise = true;
    const bool fits = admit_new_chunks(c, ids, n_chunks, &op, &op.new_chunk);
    c->stats.chunks_stored += op.new_chunk.size();
    op.pending = !op.new_chunk.empty();   // nothing new: the ticket is complete at once
    op.slot_mapping = slot_mapping;
    op.began_idle = idle;
    op.layer_done.assign(size_t(c->cfg.geom.num_layers), nullptr);
    op.layer_count.assign(size_t(c->cfg.geom.num_layers), Op::Count());
    if (ticket_out) *ticket_out = op.ticket;
    c->ops.push_back(std::move(op));
    return fits ? LMC_OK : LMC_ERR_NOMEM;
}

lmc_status_t lmc_store_layers(lmc_ctx_t *c, uint64_t ticket, int32_t first_layer, int32_t n_layers,
                              void *const *kv_layers, void *stream_to_wait_on) {
    if (!c || !kv_layers || n_layers < 1 || first_layer < 0) return LMC_ERR_INVAL;
    if (!c->has_device) return LMC_ERR_NODEVICE;
    std::lock_guard<std::mutex> lock(c->mu);
    DeviceScope dev(c);
    reap(c);
    const lmc_kv_geom_t &geom = c->cfg.geom;
    Op *op = find_op(c, ticket);
    if (op == nullptr) {
        // a layer-wise store with nothing new completes at once; its layers are accepted
        // and ignored so that the caller's per-layer loop needs no special case
        return (ticket != 0 && ticket < c->next_ticket && first_layer + n_layers <= geom.num_layers)
                   ? LMC_OK : LMC_ERR_INVAL;
    }
    if (!op->pending || first_layer != op->next_layer || first_layer + n_layers > geom.num_layers)
        return LMC_ERR_INVAL;
    c->cur_ticket = op->ticket;
    lmc::LayerPtrs ptrs;
    lmc_status_t rc = build_layer_ptrs(c, kv_layers, &ptrs);
    if (rc != LMC_OK) return rc;
    const lmc::LaunchView view = lmc::layer_view(c->kg, uint32_t(geom.num_planes), uint32_t(first_layer),
                                                 uint32_t(n_layers));
    const uint64_t layer_bytes = uint64_t(geom.num_planes) * c->kg.plane_bytes;
    const int64_t cap = layer_group_chunks(c, c->store_ring, view, int64_t(op->new_chunk.size()));
    const int64_t n_new = int64_t(op->new_chunk.size());
    const int64_t step_bytes = n_new * int64_t(layer_bytes) * n_layers;
    hipStream_t user = static_cast<hipStream_t>(stream_to_wait_on);
    const bool idle = caller_is_idle(user);
    // the producer has nothing more on its stream (nor had in front of the slot mapping), and nothing else is under way
    const bool undisturbed = idle && op->began_idle && c->ops.size() == 1;
    const int64_t bytes = n_new * c->chunk_bytes;
    const bool direct = (c->cfg.flags & LMC_FLAG_DIRECT) != 0 ||
                        bytes <= (c->stores_placed ? c->direct_placed_store_below : c->direct_store_below) ||
                        (bytes <= c->direct_store_steps_below && (step_bytes <= lmc_ctx::kDirectStoreStep || undisturbed));
    // Steps take the two copy streams in turn (as the steps of a layer-wise retrieve do):
    // between two copies of one stream the runtime leaves the link idle for some 20 us,
    // 7 % of a step of one Llama-3-8B layer, while on the other stream (another hardware
    // queue, see arrange_streams) the next step's copy is ready to start.  Not while a
    // retrieve is under way, whose kernels that stream would hold up.
    const bool on_second = !direct && (op->steps & 1) != 0 && c->store_step_streams == 2 && !other_direction_busy(c, true);
    // In an undisturbed store the steps without staging take the gather stream and the second copy stream to the
    // host in turn (which sits in the scatter stream's hardware queue, so that the library's kernels hold up no
    // third one), side by side with half of the groups each, so that one step's first slots and last stores do not
    // leave the link idle: kernels of one stream follow each other 1.4 us apart, and the first store of one and the last of
    // the other are some 3 more. On one stream and on two, steps of 0.6, 0.9, 1, 1.3 MiB: 34 MiB 809 and 760 us,
    // 22 490 and 461, 32 700 and 641, 105 2160 and 2020. Not for steps under 0.5 MiB (1.1 MiB in four 52 and 77
    // us, 10.7 in 61 of 0.2 528 and 645), whose launches take the thread longer than the link, nor beside other
    // operations, whose copies they might have to wait for. Behind a producer at work, which puts time between the
    // steps, there is nothing to gain, and a second hardware queue would wait (64 MiB in steps of 2, products of
    // 128 rows, over the four queues the producer's stream can be in, 5791 and 5905 us). The last step is on the
    // gather stream, behind the other's: what waits for the store waits for one stream.
    // All groups for a step that has the link to itself: the last one, and one that the last one follows if that is
    // as large. 16, 32, 64, 192 MiB in one call by half of them 310, 609, 1217, 3665 us, by all 306, 600, 1189,
    // 3550; in two 316, 612, 1219, 3664 and 309, 603, 1192, 3554; in four 315, 610, 1208, 3611 and 314, 606, 1195,
    // 3559. (Half also for one that only finds another still running on the second stream: four calls 3586.)
    const bool ends = first_layer + n_layers == geom.num_layers;
    const bool in_turn = undisturbed && direct && c->store_step_streams == 2 && step_bytes >= lmc_ctx::kStoreStepsInTurn &&
                         may_wait_for_word(c, c->s_gather);
    const bool beside = in_turn && !ends && (op->steps & 1) != 0;
    hipStream_t last = direct ? (beside ? c->s_d2h2 : c->s_gather) : on_second ? c->s_d2h2 : c->s_d2h;
    op->producer = user;
    // this layer's KV was produced by work already on the caller's stream
    rc = idle ? LMC_OK : order_after(c, c->s_gather, user);
    if (rc == LMC_OK && direct && ends && op->second_target != 0 && !op->has_staged_steps && may_wait_for_word(c, c->s_gather)) {
        rc = wait_for_word(c, c->s_gather, lmc_ctx::kStoreStepWord, op->second_target);
        op->ends_on.erase(std::remove(op->ends_on.begin(), op->ends_on.end(), c->s_d2h2), op->ends_on.end());
    }
    if (rc == LMC_OK && !direct)
        rc = ring_reslot(c, c->store_ring, (uint64_t(cap) * view.chunk_stride + 255) / 256 * 256, c->s_gather, c->s_d2h,
                         nullptr, c->s_d2h2);
    // A step without staging counts itself off at its stream's word, whose steps end in order: an event as the
    // launch's stop event takes the thread 2 us more, and whoever waits for it 10 us more.
    hipEvent_t e = nullptr;
    auto own_event = [&]() -> lmc_status_t {
        const lmc_status_t r = get_event(c, false, &e);
        if (r == LMC_OK) op->owned_events.push_back(e);
        return r;
    };
    const bool timed = (c->cfg.flags & (LMC_FLAG_TIMING | LMC_FLAG_TRACE)) != 0;
    const bool counts = direct && (beside || !timed) && may_wait_for_word(c, c->s_gather);
    if (rc == LMC_OK && !counts) rc = own_event();
    Op::Count count;
    if (rc == LMC_OK) {
        // the last step of a store whose steps all ran on the gather stream, or are waited for there, ends the store
        const bool tells = direct && ends && tells_host(c) &&
                           std::all_of(op->ends_on.begin(), op->ends_on.end(), [&](hipStream_t s) { return s == c->s_gather; });
        const int word = beside ? lmc_ctx::kStoreStepWord : lmc_ctx::kStoreWord;
        uint64_t &reached = c->word_target[word];
        lmc::HostWord told{counts || tells ? c->word(word) : nullptr, tells ? c->stored_dev : nullptr, reached};
        const bool shares = beside || (in_turn && int64_t(first_layer) + 2 * int64_t(n_layers) < geom.num_layers);
        const uint32_t groups = shares ? std::max(1u, c->link_groups / 2) : 0u;
        rc = store_groups(c, view, uint64_t(first_layer) * layer_bytes, ptrs, op->slot_mapping, op->new_chunk,
                          op->slots, cap, false, direct, true, on_second || beside, nullptr, e,
                          told.word != nullptr ? &told : nullptr, groups);
        if (told.target != reached) {
            reached = told.target;
            if (counts) count = Op::Count{word, reached};
            if (beside) op->second_target = reached;
            if (tells) op->stored_target = reached;
        } else if (beside) {
            op->has_staged_steps = true;     // rows that cannot count (lmc::HostWord): the end is left to the events
        }
        op->has_staged_steps = op->has_staged_steps || !direct;
        if (rc == LMC_OK && counts && count.target == 0 && (rc = own_event()) == LMC_OK)
            rc = [&]() -> lmc_status_t {
                HIPCHK(c, hipEventRecord(e, last));
                return LMC_OK;
            }();
    }
    if (rc == LMC_OK) {
        rc = [&]() -> lmc_status_t {
            if (!direct) HIPCHK(c, hipEventRecord(e, last));
            if (ends) {
                // the ticket is complete when the steps of every stream are
                lmc_status_t r = LMC_OK;
                for (hipStream_t s : op->ends_on)
                    if (r == LMC_OK && s != last) r = order_after(c, last, s);
                if (r == LMC_OK) r = get_event(c, false, &op->done);
                if (r != LMC_OK) return r;
                op->owned_events.push_back(op->done);   // given back with the others if the record fails
                HIPCHK(c, hipEventRecord(op->done, last));
                op->owned_events.pop_back();
                op->final_stream = last;
            }
            return LMC_OK;
        }();
    }
    if (rc != LMC_OK) {
        // the store cannot be completed any more: it is taken back as a whole
        const uint64_t t = op->ticket;
        auto it = std::find_if(c->ops.begin(), c->ops.end(), [t](const Op &o) { return o.ticket == t; });
        const Op gone = std::move(*it);
        c->ops.erase(it);
        abort_store(c, gone.slots);
        for (hipEvent_t x : gone.owned_events) recycle(c, x);
        return rc;
    }
    for (int32_t l = first_layer; l < first_layer + n_layers; l++) {
        op->layer_done[size_t(l)] = e;
        op->layer_count[size_t(l)] = count;
    }
    op->next_layer = first_layer + n_layers;
    op->steps++;
    if (std::find(op->ends_on.begin(), op->ends_on.end(), last) == op->ends_on.end()) op->ends_on.push_back(last);
    if (op->next_layer == geom.num_layers) op->pending = false;
    return LMC_OK;
}

lmc_status_t lmc_retrieve_layerwise(lmc_ctx_t *c, const uint64_t *ids, int64_t n_chunks,
                                    const int64_t *slot_mapping, void *const *kv_layers,
                                    int32_t layers_per_step, void *stream_to_wait_on,
                                    uint64_t *ticket_out) {
    if (!c || n_chunks < 0 || !kv_layers || layers_per_step < 1 ||
        (n_chunks > 0 && (!slot_mapping || !ids)))
        return LMC_ERR_INVAL;
    std::lock_guard<std::mutex> lock(c->mu);
    return do_retrieve(c, ids, n_chunks, slot_mapping, kv_layers, stream_to_wait_on,
                       std::min(layers_per_step, c->cfg.geom.num_layers), ticket_out);
}

lmc_status_t lmc_wait_layer(lmc_ctx_t *c, uint64_t ticket, int32_t layer, void *stream) {
    if (!c || ticket == 0 || layer < 0 || layer >= c->cfg.geom.num_layers) return LMC_ERR_INVAL;
    if (!c->has_device) return LMC_ERR_NODEVICE;
    std::lock_guard<std::mutex> lock(c->mu);
    DeviceScope dev(c);
    if (ticket >= c->next_ticket) return LMC_ERR_INVAL;
    Op *op = find_op(c, ticket);
    if (op == nullptr) return LMC_OK;                       // finished long ago
    if (!op->layerwise) return LMC_ERR_INVAL;
    if (!op->step_target.empty()) {
        if (hipEventQuery(op->done) == hipSuccess) return event_behind_wait(c, op, static_cast<hipStream_t>(stream));
        (void)hipGetLastError();   // "not ready" is an answer, not a failure
        const int32_t i = layer / op->step_layers;
        hipStream_t user = static_cast<hipStream_t>(stream);
        if (may_wait_for_word(c, user)) {
            if (op->has_waiting(user, 0, uint64_t(i) + 1)) return LMC_OK;
            const lmc_status_t rc = wait_for_word(c, user, i, op->step_target[size_t(i)]);
            if (rc != LMC_OK) return rc;
            op->made_wait(user, 0, uint64_t(i) + 1);
            return size_t(i) + 1 == op->step_target.size() ? event_behind_wait(c, op, user) : LMC_OK;
        }
        HIPCHK(c, hipStreamWaitEvent(static_cast<hipStream_t>(stream), op->done, 0));   // all layers
        return LMC_OK;
    }
    if (!op->layer_count.empty() && op->layer_count[size_t(layer)].target != 0) {
        const Op::Count &n = op->layer_count[size_t(layer)];
        hipStream_t user = static_cast<hipStream_t>(stream);
        if (!op->pending) {
            const bool ended = op->stored_target != 0 ? c->is_stored(op->stored_target)
                                                      : op->done != nullptr && hipEventQuery(op->done) == hipSuccess;
            (void)hipGetLastError();   // "not ready" is an answer, not a failure
            if (ended) return event_behind_wait(c, op, user);
        }
        if (may_wait_for_word(c, user)) {
            const int which = n.word == lmc_ctx::kStoreWord ? 0 : 1;
            if (op->has_waiting(user, which, n.target)) return LMC_OK;
            const lmc_status_t rc = wait_for_word(c, user, n.word, n.target);
            if (rc != LMC_OK) return rc;
            op->made_wait(user, which, n.target);
            // A store that is still being handed in asks the producer's stream next.  Others do without: 32 steps of
            // 0.125 MiB, each waited for by another stream, take 358 us, with an event behind each wait 446.
            const Op::Count &last = op->layer_count.back();
            const bool may_be_last = op->pending ? user == op->producer : n.word == last.word && n.target == last.target;
            return may_be_last ? event_behind_wait(c, op, user) : LMC_OK;
        }
        return order_after(c, user, n.word == lmc_ctx::kStoreWord ? c->s_gather : c->s_d2h2);
    }
    if (op->layer_done.empty() || (op->layer_done[size_t(layer)] == nullptr && !op->pending))
        return LMC_OK;                                      // nothing was enqueued for it
    if (op->layer_done[size_t(layer)] == nullptr) return LMC_ERR_BUSY;  // layer not submitted yet
    HIPCHK(c, hipStreamWaitEvent(static_cast<hipStream_t>(stream), op->layer_done[size_t(layer)], 0));
    return LMC_OK;
}

lmc_status_t lmc_retrieve(lmc_ctx_t *c, const uint64_t *ids, int64_t n_chunks,
                          const int64_t *slot_mapping, void *const *kv_layers,
                          void *stream_to_signal, uint64_t *ticket_out) {
    if (!c || n_chunks < 0 || !kv_layers || (n_chunks > 0 && (!slot_mapping || !ids)))
        return LMC_ERR_INVAL;
    std::lock_guard<std::mutex> lock(c->mu);
    return do_retrieve(c, ids, n_chunks, slot_mapping, kv_layers, stream_to_signal, 0, ticket_out);
}

lmc_status_t lmc_retrieve_batch(lmc_ctx_t *c, int64_t n_req, const int64_t *off,
                                const uint64_t *ids, const int64_t *slot_mapping,
                                void *const *kv_layers, void *stream_to_signal,
                                uint64_t *ticket_out) {
    if (!c || n_req < 0 || !off || !kv_layers || off[0] != 0) return LMC_ERR_INVAL;
    for (int64_t r = 0; r < n_req; r++)
        if (off[r + 1] < off[r]) return LMC_ERR_INVAL;
    const int64_t total = off[n_req];
    if (total > 0 && (!ids || !slot_mapping)) return LMC_ERR_INVAL;
    // The requests' chunks and slot mappings are already back to back, so the batch is
    // one stream of chunks: kernel launches and copies run across request borders.
    std::lock_guard<std::mutex> lock(c->mu);
    return do_retrieve(c, ids, total, slot_mapping, kv_layers, stream_to_signal, 0, ticket_out);
}

lmc_status_t lmc_gather(lmc_ctx_t *c, void *const *kv_layers, const int64_t *slot_mapping,
                        int64_t n_chunks, void *staging_dev, void *stream) {
    return device_only(c, true, kv_layers, slot_mapping, n_chunks, static_cast<uint8_t *>(staging_dev), stream);
}

lmc_status_t lmc_scatter(lmc_ctx_t *c, const void *staging_dev, const int64_t *slot_mapping,
                         int64_t n_chunks, void *const *kv_layers, void *stream) {
    return device_only(c, false, kv_layers, slot_mapping, n_chunks,
                       static_cast<uint8_t *>(const_cast<void *>(staging_dev)), stream);
}

}  // extern "C"
