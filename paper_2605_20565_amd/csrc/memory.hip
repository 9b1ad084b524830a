// Device memory kept in the process: blocks of trees that are gone, for the
// trees built next, and working memory of plain calls that sort their points.
#include <mutex>

#include "memory.h"
#include "ot_common.h"

namespace ot {
namespace {

// Memory of trees that are gone, for the trees built next: freeing a used
// buffer of some 20 MB costs the host 250 us or more (of the 2.4 ms in which a
// tree of 2.7 M leaves was built and destroyed, 1.4 ms went to hipFree).  At
// most kKeptBlocks blocks and kKeptBytes are kept, the oldest are freed first,
// and all of a device's are given back where an allocation of the library finds
// no room (give_back).  Blocks
// come here only when no work on them is left, so any stream may have them next.
constexpr size_t kKeptBlocks = 6, kKeptBytes = size_t(256) << 20;
// (a plain array: nothing here throws, and trees may be destroyed after the
// destructors of static objects)
std::mutex g_kept_lock;
Block g_kept[kKeptBlocks];   // oldest first
size_t g_n_kept = 0;

Block kept_remove(size_t i)
{
    const Block b = g_kept[i];
    for (--g_n_kept; i < g_n_kept; ++i) g_kept[i] = g_kept[i + 1];
    return b;
}

}  // namespace

Block block_take(size_t bytes)
{
    Block b;
    b.bytes = (bytes + 0xFFFF) & ~size_t(0xFFFF);
    (void)hipGetDevice(&b.device);
    {
        std::lock_guard<std::mutex> lock(g_kept_lock);
        size_t best = kKeptBlocks;
        for (size_t i = 0; i < g_n_kept; ++i) {
            const Block &c = g_kept[i];
            // not more than twice what is asked for
            if (c.device == b.device && c.bytes >= b.bytes && c.bytes / 2 <= b.bytes &&
                (best == kKeptBlocks || c.bytes < g_kept[best].bytes))
                best = i;
        }
        if (best < kKeptBlocks) return kept_remove(best);
    }
    if (device_malloc(&b.p, b.bytes) != hipSuccess) b.p = nullptr;
    return b;
}

void block_give(const Block &b)
{
    if (!b.p) return;
    std::lock_guard<std::mutex> lock(g_kept_lock);
    size_t kept = b.bytes;
    for (size_t i = 0; i < g_n_kept; ++i) kept += g_kept[i].bytes;
    while (g_n_kept && (kept > kKeptBytes || g_n_kept == kKeptBlocks)) {
        const Block old = kept_remove(0);
        kept -= old.bytes;
        (void)hipFree(old.p);
    }
    if (kept > kKeptBytes) (void)hipFree(b.p);
    else g_kept[g_n_kept++] = b;
}

namespace {

// Working memory of plain calls that sort their points, of all trees on a
// device (allocating it takes the host 100 us and more, the runtime's stream-
// ordered allocator ~50 us a call, and a program that adapts its mesh builds a
// tree every few calls).  A call takes a buffer nobody is using, waits on its
// stream for the event of the buffer's last call, and records the event anew
// when its kernels are enqueued: calls may come from several threads, streams
// and trees.  At most kScratchSlots buffers and kScratchKeep bytes are kept a
// device (a call that needs more allocates for itself), kKeptBytes when its
// last tree is gone.
constexpr int kScratchSlots = 4, kScratchDevices = 16;
constexpr size_t kScratchKeep = size_t(1) << 30;
struct ScratchSlot {
    void *p;
    size_t bytes;
    hipEvent_t done;     // the last call's kernels
    hipStream_t stream;  // and its stream
    bool busy;           // a call is enqueueing
    bool used;           // done has been recorded for this memory
};
struct DeviceScratch {
    std::mutex lock;
    ScratchSlot slot[kScratchSlots];
    int trees;
};
DeviceScratch g_scratch[kScratchDevices];

DeviceScratch *scratch_of(int device)
{
    return device >= 0 && device < kScratchDevices ? &g_scratch[device] : nullptr;
}

// A graph capture that another stream or thread has under way (in its default,
// global mode) forbids allocating and asking events; scratch memory never takes
// part in one, so the calls here are made in relaxed mode.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    bool set;
    RelaxedCapture() : set(hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {}
    ~RelaxedCapture()
    {
        if (set) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    RelaxedCapture(const RelaxedCapture &) = delete;
    RelaxedCapture &operator=(const RelaxedCapture &) = delete;
};

// Allocations and events of a tree's device, whatever device is current (a
// call's stream may belong to another one).
struct OnDevice {
    int before = -1;
    explicit OnDevice(int device)
    {
        if (hipGetDevice(&before) != hipSuccess || before == device || hipSetDevice(device) != hipSuccess) before = -1;
    }
    ~OnDevice()
    {
        if (before >= 0) (void)hipSetDevice(before);
    }
    OnDevice(const OnDevice &) = delete;
    OnDevice &operator=(const OnDevice &) = delete;
};

void slot_free(ScratchSlot &c)
{
    if (c.p) {
        if (c.used) (void)hipEventSynchronize(c.done);   // its last call
        (void)hipFree(c.p);
    }
    c.used = false;
    c.p = nullptr;
    c.bytes = 0;
}

size_t kept_bytes(const DeviceScratch &d)
{
    size_t b = 0;
    for (const ScratchSlot &c : d.slot) b += c.bytes;
    return b;
}

// What nobody is using of a device's memory: its blocks of gone trees, and (its
// lock held) its slots.
void give_back_blocks(int device)
{
    std::lock_guard<std::mutex> lock(g_kept_lock);
    for (size_t i = g_n_kept; i-- > 0;)
        if (g_kept[i].device == device) (void)hipFree(kept_remove(i).p);
}
void give_back_slots(DeviceScratch &d)
{
    for (ScratchSlot &c : d.slot)
        if (!c.busy) slot_free(c);
}
void give_back(int device)
{
    const OnDevice on(device);
    const RelaxedCapture relaxed;
    give_back_blocks(device);
    if (DeviceScratch *d = scratch_of(device)) {
        std::lock_guard<std::mutex> lock(d->lock);
        give_back_slots(*d);
    }
    (void)hipGetLastError();
}

// A slot with new memory of at least `bytes`, or null.  Buffers that nobody is
// using and that are too small for this call make room, the smallest first.
ScratchSlot *slot_grow(DeviceScratch &d, int device, size_t bytes)
{
    size_t want = (bytes + bytes / 4 + 0xFFFFF) & ~size_t(0xFFFFF);   // room for calls a little larger
    if (want > kScratchKeep) want = (bytes + 0xFFFFF) & ~size_t(0xFFFFF);
    if (want > kScratchKeep) return nullptr;
    for (;;) {
        ScratchSlot *empty = nullptr, *least = nullptr;
        for (ScratchSlot &c : d.slot) {
            if (c.busy) continue;
            if (!c.p) empty = &c;
            else if (c.bytes < bytes && (!least || c.bytes < least->bytes)) least = &c;
        }
        if (empty && kept_bytes(d) + want <= kScratchKeep) {
            if (!empty->done && hipEventCreateWithFlags(&empty->done, hipEventDisableTiming) != hipSuccess) {
                empty->done = nullptr;
                return nullptr;
            }
            hipError_t e = hipMalloc(&empty->p, want);
            if (e == hipErrorOutOfMemory) {
                (void)hipGetLastError();
                give_back_blocks(device);
                give_back_slots(d);
                want = bytes;
                e = hipMalloc(&empty->p, want);
            }
            if (e != hipSuccess) {
                empty->p = nullptr;
                return nullptr;
            }
            empty->bytes = want;
            return empty;
        }
        if (!least) return nullptr;
        slot_free(*least);
    }
}

}  // namespace

hipError_t device_malloc(void **p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        int device = 0;
        (void)hipGetDevice(&device);
        give_back(device);
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
    }
    return e;
}

hipError_t device_malloc_async(int device, void **p, size_t bytes, hipStream_t s)
{
    hipError_t e = hipMallocAsync(p, bytes, s);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        give_back(device);
        e = hipMallocAsync(p, bytes, s);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
    }
    return e;
}

Scratch scratch_take(int device, size_t bytes, hipStream_t s)
{
    const OnDevice on(device);
    const RelaxedCapture relaxed;
    if (DeviceScratch *d = scratch_of(device)) {
        std::lock_guard<std::mutex> lock(d->lock);
        ScratchSlot *best = nullptr;
        for (ScratchSlot &c : d->slot)
            if (!c.busy && c.bytes >= bytes && (c.stream == s || !c.used || hipEventQuery(c.done) == hipSuccess) &&
                (!best || c.bytes < best->bytes))
                best = &c;
        (void)hipGetLastError();   // an event not reached yet is no error
        if (best && best->used && hipStreamWaitEvent(s, best->done, 0) != hipSuccess) {
            (void)hipGetLastError();
            return {nullptr, -1};
        }
        if (!best) best = slot_grow(*d, device, bytes);
        (void)hipGetLastError();
        if (best) {
            best->stream = s;
            best->busy = true;
            return {best->p, (int)(best - d->slot)};
        }
    }
    void *p = nullptr;
    (void)device_malloc_async(device, &p, bytes, s);
    return {p, -1};
}

void scratch_give(int device, const Scratch &m, hipStream_t s)
{
    const OnDevice on(device);
    const RelaxedCapture relaxed;
    if (m.slot < 0) {
        if (m.p) (void)hipFreeAsync(m.p, s);
        return;
    }
    DeviceScratch &d = g_scratch[device];
    std::lock_guard<std::mutex> lock(d.lock);
    ScratchSlot &c = d.slot[m.slot];
    if (hipEventRecord(c.done, s) != hipSuccess) {
        // without the event the buffer cannot be handed on in order
        (void)hipGetLastError();
        (void)hipStreamSynchronize(s);
        c.used = false;
        slot_free(c);
    } else {
        c.used = true;
    }
    c.busy = false;
}

void scratch_trees(int device, int change)
{
    DeviceScratch *d = scratch_of(device);
    if (!d) return;
    const OnDevice on(device);
    std::lock_guard<std::mutex> lock(d->lock);
    d->trees += change;
    while (d->trees == 0 && kept_bytes(*d) > kKeptBytes) {
        ScratchSlot *most = nullptr;
        for (ScratchSlot &c : d->slot)
            if (c.p && !c.busy && (!most || c.bytes > most->bytes)) most = &c;
        if (!most) break;
        slot_free(*most);
    }
}

}  // namespace ot
