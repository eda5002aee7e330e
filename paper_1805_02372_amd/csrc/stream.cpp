// Block-serial hashing (paper section 3, Fig. 1-3): the key is processed in
// blocks whose partial hashes are XOR-merged (Eq. 4-7), with the accumulator
// resident in device memory.  Each block is an ordinary job (planned as
// pa_hash plans it, on the block and its seed slice); its output lands in a
// scratch word array that a small kernel XORs into the accumulator.
//
// Blocks from host memory are pipelined over two staging slots: a feed copies
// its block into pinned memory and starts the DMA on a copy stream while the
// previous block's kernels still run, enqueues its own block behind them and its
// DMA, then checks the previous block's certificate (FP64 fallback as in
// pa_hash) and merges it.  The last block is checked by the next call on the
// stream (feed, state, resume or close).  The stream has its own GPU stream and
// workspace, so it runs beside the context's other calls.
#include <hip/hip_runtime.h>

#include <cstring>
#include <mutex>

#include "direct.hpp"
#include "engine.hpp"
#include "planner.hpp"

using namespace pa;

struct pa_stream {
    Ctx* c = nullptr;
    uint64_t n = 0, m = 0;
    uint32_t flags = 0;
    uint64_t fed = 0;
    DevBuf acc;                     // the accumulator
    StreamRes* r = nullptr;         // lanes, copy stream, staging slots
    int slot = 0;                   // slot of the next host block
    // the block in flight: its kernels enqueued on lane `lane`, its certificate
    // not yet read
    struct Block {
        bool live = false, fft = false;
        uint64_t len = 0;
        int lane = 0;
    } pending;
    bool ahead = true;              // a block may be enqueued before the last one is checked
    hipStream_t stream() const { return r->ln[0].stream; }
};

static uint64_t nwords(uint64_t bits) { return (bits + 63) >> 6; }

// Settle a block: wait for it, check its certificate (FP64 fallback of failed
// tiles) and merge it into the accumulator.  On an error the block is dropped
// (accumulator and fed count unchanged).
static pa_status settle(pa_stream* s, const pa_stream::Block& b) {
    if (!b.live) return PA_OK;
    if (b.fft) {
        pa_stats st{};
        const pa_status r = s->r->lane(b.lane).finish(s->c, s->flags & PA_NO_FALLBACK, &st, nullptr);
        if (r != PA_OK) return r;
        if (launch_xor_words((uint64_t*)s->acc.ptr, (const uint64_t*)s->r->part[b.lane].ptr, nwords(s->m), s->stream()))
            return PA_EDEVICE;
    }
    s->fed += b.len;
    return PA_OK;
}

static pa_status drain(pa_stream* s) {
    const pa_stream::Block b = s->pending;
    s->pending.live = false;
    return settle(s, b);
}

// Enqueue the partial hash of an FFT block on a lane.
static pa_status launch_fft(pa_stream* s, int lane, const uint64_t* dseed, const uint64_t* dkey, uint64_t len,
                            const TilePlan& plan) {
    auto launch = [&] {
        pa_stats st{};
        std::vector<JobDesc> jobs(1);
        fill_job(&jobs[0], dseed, dkey, (uint64_t*)s->r->part[lane].ptr, len, s->m, plan);
        return s->r->lane(lane).launch(s->c, plan.prec, plan.cls, jobs, false, true, &st);
    };
    const pa_status st = launch();
    if (st != PA_ENOMEM) return st;
    {
        std::lock_guard<std::mutex> lk(s->c->mu);   // the workspaces of idle calls
        if (!s->c->give_back(nullptr)) return st;
    }
    return launch();
}

// Enqueue the partial hash of one block (device pointers) and settle the block
// before it; a direct-product block is merged at once (it has no certificate),
// an FFT block when settled.  The previous block's error is returned, and this
// block is dropped.  An FFT block is enqueued before the previous one is checked,
// so that the device goes from one to the next without waiting for the host (8
// blocks of 16 Mbit, m = 10^6: 1.73 -> 1.54 ms); where the memory of a
// second output is not there, after it.
static pa_status launch_block(pa_stream* s, const uint64_t* dseed, const uint64_t* dkey, uint64_t len) {
    Ctx* c = s->c;
    const uint64_t m = s->m;
    const int policy = policy_of(s->flags);
    TilePlan plan;
    CostModel cm;
    const bool planned = c->plan_cached(len, m, policy, &plan);
    {
        std::lock_guard<std::mutex> pk(c->plan_mu);
        cm = c->cost;
    }
    const bool direct = planned && choose_direct(s->flags, len, m, cm, plan);
    if (planned && !direct && s->pending.live && s->pending.fft && s->ahead) {
        const int b = s->pending.lane ^ 1;
        if (s->r->part[b].ensure(c, nwords(m) * 8, s->stream()) == PA_OK &&
            launch_fft(s, b, dseed, dkey, len, plan) == PA_OK) {
            const pa_status st = drain(s);
            if (st != PA_OK) {
                (void)hipStreamSynchronize(s->stream());   // the dropped block's certificates are written
                return st;
            }
            s->pending = {true, true, len, b};
            return PA_OK;
        }
        (void)hipStreamSynchronize(s->stream());   // whatever part of it was enqueued
        s->ahead = false;
    }
    const int b = s->pending.lane;
    pa_status st = drain(s);
    if (st != PA_OK) return st;
    if (!planned) return PA_EINVAL;
    if (!s->ahead) s->r->part[b ^ 1].release(c);
    if (direct) {
        pa_stats stats{};
        uint64_t* out = (uint64_t*)s->r->part[b].ptr;
        st = s->r->lane(b).direct(c, dseed, dkey, len, m, out, false, &stats);
        if (st != PA_OK) return st;
        if (launch_xor_words((uint64_t*)s->acc.ptr, out, nwords(m), s->stream())) return PA_EDEVICE;
    } else {
        st = launch_fft(s, b, dseed, dkey, len, plan);
        if (st == PA_ENOMEM && s->ahead) {   // the second output's memory
            s->ahead = false;
            s->r->part[b ^ 1].release(c);
            st = launch_fft(s, b, dseed, dkey, len, plan);
        }
        while (st == PA_ENOMEM && smaller_plan(len, m, policy, cm, &plan)) st = launch_fft(s, b, dseed, dkey, len, plan);
        if (st != PA_OK) return st;
    }
    s->pending = {true, !direct, len, b};
    return PA_OK;
}

namespace pa {
void StreamRes::release(Ctx* c) {
    if (ln[0].stream) (void)hipStreamSynchronize(ln[0].stream);
    if (copy) (void)hipStreamSynchronize(copy);
    for (int b = 0; b < 2; ++b) {
        part[b].release(c);
        in[b].release(c);
        pin[b].release();
    }
    ln[1].release(c);
    ln[0].release(c);   // synchronises its stream (the frees above were queued on it) and destroys it
    if (copy) {
        (void)hipStreamSynchronize(copy);
        (void)hipStreamDestroy(copy);
    }
    copy = nullptr;
    for (int b = 0; b < 2; ++b) {
        if (staged[b]) (void)hipEventDestroy(staged[b]);
        if (used[b]) (void)hipEventDestroy(used[b]);
        staged[b] = used[b] = nullptr;
    }
}
}  // namespace pa

// Resources for a new stream: a closed stream's, else new ones.
static pa_status take_res(Ctx* c, uint64_t m, StreamRes** out) {
    StreamRes* r = nullptr;
    {
        std::lock_guard<std::mutex> lk(c->stream_mu);
        if (!c->idle_streams.empty()) {
            r = c->idle_streams.back();
            c->idle_streams.pop_back();
        }
    }
    pa_status st = PA_OK;
    if (!r) {
        r = new StreamRes();
        if (hipStreamCreateWithFlags(&r->ln[0].stream, hipStreamNonBlocking) != hipSuccess) st = PA_EDEVICE;
        r->ln[0].own_stream = r->ln[0].stream != nullptr;
        r->ln[1].stream = r->ln[0].stream;
        if (st == PA_OK && hipStreamCreateWithFlags(&r->copy, hipStreamNonBlocking) != hipSuccess) st = PA_EDEVICE;
        for (int b = 0; b < 2 && st == PA_OK; ++b)
            if (hipEventCreateWithFlags(&r->staged[b], hipEventDisableTiming) != hipSuccess ||
                hipEventCreateWithFlags(&r->used[b], hipEventDisableTiming) != hipSuccess ||
                hipEventRecord(r->staged[b], r->copy) != hipSuccess ||   // waits on them find them recorded
                hipEventRecord(r->used[b], r->ln[0].stream) != hipSuccess)
                st = PA_EDEVICE;
    }
    if (st == PA_OK) st = c->reserve_unlocked(r->part[0], nwords(m) * 8, r->ln[0].stream);
    if (st != PA_OK) {
        r->release(c);
        delete r;
        return st;
    }
    *out = r;
    return PA_OK;
}

// Close: keep one set of resources for the next stream, free the rest.
static void free_stream(pa_stream* s) {
    Ctx* c = s->c;
    (void)hipSetDevice(c->device);
    if (s->r) {
        (void)hipStreamSynchronize(s->stream());
        (void)hipStreamSynchronize(s->r->copy);
    }
    s->acc.release(c);
    if (s->r) {
        s->r->part[1].release(c);
        bool kept = false;
        {
            std::lock_guard<std::mutex> lk(c->stream_mu);
            if (c->idle_streams.empty()) {
                c->idle_streams.push_back(s->r);
                kept = true;
            }
        }
        if (!kept) {
            s->r->release(c);
            delete s->r;
        }
    }
    delete s;
}

extern "C" {

pa_status pa_stream_open(pa_ctx* ctx, uint64_t n, uint64_t m, uint32_t flags, pa_stream** out) {
    if (!ctx || !out || n == 0 || m == 0 || n > (1ull << 40) || m > (1ull << 40)) return PA_EINVAL;
    if (policy_of(flags) < 0) return PA_EINVAL;
    *out = nullptr;
    Ctx* c = reinterpret_cast<Ctx*>(ctx);
    if (hipSetDevice(c->device) != hipSuccess) return PA_EDEVICE;
    pa_stream* s = new pa_stream();
    s->c = c;
    s->n = n;
    s->m = m;
    s->flags = flags;
    pa_status st = take_res(c, m, &s->r);
    if (st == PA_OK) st = c->reserve_unlocked(s->acc, nwords(m) * 8, s->stream());
    // x ^ x = 0: clear the accumulator with the XOR kernel itself
    if (st == PA_OK &&
        launch_xor_words((uint64_t*)s->acc.ptr, (const uint64_t*)s->acc.ptr, nwords(m), s->stream()))
        st = PA_EDEVICE;
    if (st == PA_OK && hipStreamSynchronize(s->stream()) != hipSuccess) st = PA_EDEVICE;
    if (st != PA_OK) {
        free_stream(s);
        return st;
    }
    *out = s;
    return PA_OK;
}

pa_status pa_stream_feed(pa_stream* s, const uint64_t* key_block, uint64_t lo, uint64_t len,
                         const uint64_t* seed_block) {
    if (!s || !key_block || !seed_block || len == 0 || lo >= s->n || len > s->n - lo) return PA_EINVAL;
    Ctx* c = s->c;
    if (hipSetDevice(c->device) != hipSuccess) return PA_EDEVICE;
    const uint64_t kw = nwords(len), sw = nwords(len + s->m - 1);
    if (s->flags & PA_DEVICE_PTRS) {   // the caller's buffers, read before the call returns
        pa_status st = launch_block(s, seed_block, key_block, len);
        if (st == PA_OK) st = drain(s);
        if (hipStreamSynchronize(s->stream()) != hipSuccess && st == PA_OK) st = PA_EDEVICE;
        return st;
    }
    // Stage the block in slot b while the previous block runs: the slot's
    // pinned image is free once its last DMA is done, its device buffer once
    // the block that read it is done (the copy stream waits for that).
    const int b = s->slot;
    const size_t sbytes = sw * 8, off = (sbytes + 255) & ~(size_t)255, kbytes = kw * 8;
    if (hipEventSynchronize(s->r->staged[b]) != hipSuccess) return PA_EDEVICE;
    pa_status st = s->r->pin[b].ensure(off + kbytes);
    if (st == PA_OK && s->r->in[b].bytes < off + kbytes) {
        // a larger block: the old buffer may be freed only after its reader
        if (hipStreamWaitEvent(s->r->copy, s->r->used[b], 0) != hipSuccess) return PA_EDEVICE;
        st = c->reserve_unlocked(s->r->in[b], off + kbytes, s->r->copy);
    }
    if (st != PA_OK) return st;
    unsigned char* h = (unsigned char*)s->r->pin[b].ptr;
    unsigned char* d = (unsigned char*)s->r->in[b].ptr;
    c->copier.copy(h, seed_block, sbytes);
    if (hipStreamWaitEvent(s->r->copy, s->r->used[b], 0) != hipSuccess ||
        hipMemcpyAsync(d, h, sbytes, hipMemcpyHostToDevice, s->r->copy) != hipSuccess)
        return PA_EDEVICE;
    c->copier.copy(h + off, key_block, kbytes);   // while the seed's DMA runs
    if (hipMemcpyAsync(d + off, h + off, kbytes, hipMemcpyHostToDevice, s->r->copy) != hipSuccess ||
        hipEventRecord(s->r->staged[b], s->r->copy) != hipSuccess)
        return PA_EDEVICE;
    // this block behind the previous one, then the previous block's certificate,
    // fallback and merge; its error is this call's
    if (hipStreamWaitEvent(s->stream(), s->r->staged[b], 0) != hipSuccess) return PA_EDEVICE;
    const uint64_t* dseed = (const uint64_t*)s->r->in[b].ptr;
    const uint64_t* dkey = (const uint64_t*)(d + off);
    st = launch_block(s, dseed, dkey, len);
    if (hipEventRecord(s->r->used[b], s->stream()) != hipSuccess && st == PA_OK) st = PA_EDEVICE;
    s->slot ^= 1;
    return st;
}

pa_status pa_stream_state(pa_stream* s, uint64_t* acc, uint64_t* fed_bits) {
    if (!s) return PA_EINVAL;
    Ctx* c = s->c;
    if (hipSetDevice(c->device) != hipSuccess) return PA_EDEVICE;
    pa_status st = drain(s);
    if (st != PA_OK) return st;
    if (fed_bits) *fed_bits = s->fed;
    if (!acc) return PA_OK;
    const hipMemcpyKind kind = (s->flags & PA_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
    if (hipMemcpyAsync(acc, s->acc.ptr, nwords(s->m) * 8, kind, s->stream()) != hipSuccess ||
        hipStreamSynchronize(s->stream()) != hipSuccess)
        return PA_EDEVICE;
    return PA_OK;
}

pa_status pa_stream_resume(pa_stream* s, const uint64_t* acc, uint64_t fed_bits) {
    if (!s || !acc || fed_bits > s->n) return PA_EINVAL;
    Ctx* c = s->c;
    if (hipSetDevice(c->device) != hipSuccess) return PA_EDEVICE;
    (void)drain(s);   // a block in flight is replaced with the rest of the state
    const hipMemcpyKind kind = (s->flags & PA_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    if (hipMemcpyAsync(s->acc.ptr, acc, nwords(s->m) * 8, kind, s->stream()) != hipSuccess ||
        hipStreamSynchronize(s->stream()) != hipSuccess)
        return PA_EDEVICE;
    s->fed = fed_bits;
    return PA_OK;
}

pa_status pa_stream_close(pa_stream* s, uint64_t* out) {
    if (!s) return PA_EINVAL;
    (void)hipSetDevice(s->c->device);
    pa_status st = drain(s);
    if (st == PA_OK && out) st = s->fed == s->n ? pa_stream_state(s, out, nullptr) : PA_EINVAL;
    free_stream(s);
    return st;
}

}  // extern "C"
