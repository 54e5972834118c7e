// General-case direct convolution: dispatch over filter side, tile shape and schedule, and
// the workspace that shared tiles are summed through.  The kernel is in general_kernel.h.
#include <cmath>
#include <map>
#include <memory>
#include <mutex>
#include <tuple>
#include <utility>
#include <vector>
#include "general_kernel.h"
#include "split_kernel.h"

namespace dconv {

// ---- workspace ---------------------------------------------------------------------------------
// One per (device, stream): launches on one stream run in order and may share it; launches on
// different streams may overlap and must not.  (hipStreamPerThread is one handle and another
// stream in every thread: each thread has a block of its own there, which passes to the next
// thread that needs one when it ends.)  It holds the partial sums of tiles shared by
// several workgroups and one arrival counter per workgroup.  The counters are zero between
// launches: the workgroup that completes a tile resets its counter.
//
// A block, once handed out, keeps its address until release_general_workspaces(): kernel
// arguments hold it by value, so a HIP graph captured on the stream refers to it for as long as
// the graph lives.  The first request on a (device, stream) therefore allocates what the
// largest launch on that device can need (a launch has at most OCC workgroups per CU, each with
// two partial tiles), and later requests find it large enough.  Should a request ever exceed it
// (a forced grid), a larger block is allocated beside the old one, which is kept until release.
//
// A graph may be replayed on another stream than the one it was captured on, beside calls on that
// one: the first captured launch takes the stream's block over, later captured launches share it,
// and the next call that is not captured is given a block of its own.
namespace {

// floats of partial sums and counters per CU that cover every compiled tile shape:
// 64 x 256 tiles at two workgroups per CU (2 * 2 * 16384), 64 x 128 or 32 x 256 at three
constexpr size_t kPartFloatsPerCu = 2 * 2 * 64 * 256;
constexpr size_t kCountersPerCu = 4;

struct WsBlock {
    float* part = nullptr;
    size_t part_floats = 0;
    int* cnt = nullptr;
    size_t ncnt = 0;
    bool holds(size_t floats, size_t counters) const { return part && part_floats >= floats && cnt && ncnt >= counters; }
};
struct WsEntry {
    std::mutex mutex;                // held while a call that uses the entry enqueues its kernels
    WsBlock eager, captured;         // for calls, and for launches that a graph holds
    hipEvent_t done = nullptr;       // hipStreamPerThread: recorded behind the last call that used `eager`
    std::vector<void*> retired;      // outgrown blocks: freed only by release_general_workspaces()
    void retire(WsBlock& b) noexcept
    {
        try {
            if (b.part) retired.push_back(b.part);
            if (b.cnt) retired.push_back(b.cnt);
        } catch (...) {}                                 // (never freed, but nobody's)
        b = WsBlock();
    }
    void free_all()
    {
        if (done) (void)hipEventDestroy(done);
        done = nullptr;
        for (WsBlock* b : {&eager, &captured}) retire(*b);
        for (void* q : retired) (void)hipFree(q);
        retired.clear();
    }
};
// (never destroyed: threads may end after the library's static objects have)
struct WsTable {
    std::mutex mutex;
    std::map<std::tuple<int, hipStream_t, uint64_t>, std::shared_ptr<WsEntry>> entries;     // device, stream, thread
    std::vector<std::pair<int, std::shared_ptr<WsEntry>>> left;                            // by threads that ended
};
WsTable& ws_table()
{
    static WsTable* t = new WsTable;
    return *t;
}

// The calling thread, for hipStreamPerThread; other streams are the same stream in every thread (0).
struct WsThread {
    uint64_t id = 0;
    ~WsThread()
    {
        if (id == 0) return;
        WsTable& t = ws_table();
        std::lock_guard<std::mutex> lock(t.mutex);
        for (auto it = t.entries.begin(); it != t.entries.end();) {
            if (std::get<2>(it->first) != id) { ++it; continue; }
            it->second->retire(it->second->captured);        // (graphs may outlive the thread)
            t.left.emplace_back(std::get<0>(it->first), std::move(it->second));
            it = t.entries.erase(it);
        }
    }
};
uint64_t ws_thread(hipStream_t st)
{
    static std::atomic<uint64_t> count{0};
    thread_local WsThread self;
    if (st != hipStreamPerThread) return 0;
    if (self.id == 0) self.id = ++count;
    return self.id;
}

__global__ void clear_counters_kernel(int* cnt, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) cnt[i] = 0;
}

// Clears the counters of a block before the calls that follow on the stream.  A capture that lets
// the allocation through (relaxed mode) would record the clearing instead of running it, and calls
// before the graph's first replay would find counters never cleared: there it runs on a stream
// of its own and is waited for.
bool clear_counters(int* cnt, size_t n, hipStream_t st)
{
    const bool apart = gen_capturing(st);
    hipStream_t on = st;
    if (apart && hipStreamCreateWithFlags(&on, hipStreamNonBlocking) != hipSuccess) return false;
    begin_launch();
    hipLaunchKernelGGL(clear_counters_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, on, cnt, (int)n);
    bool ok = launch_status() == DCONV_OK;
    if (apart) {
        ok = hipStreamSynchronize(on) == hipSuccess && ok;
        (void)hipStreamDestroy(on);
    }
    return ok;
}

}  // namespace

int gen_cus()
{
    static std::atomic<int> seen[64] = {};       // per device
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (dev >= 0 && dev < 64 && (cus = seen[dev].load(std::memory_order_relaxed)) > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (dev >= 0 && dev < 64) seen[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

bool gen_capturing(hipStream_t st)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) == hipSuccess) return cap != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

namespace {

// While it lives, this thread's allocations do not count as part of captures that go on elsewhere, which
// they would end as invalid.
class BesideCaptures {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    bool changed = false;
public:
    explicit BesideCaptures(bool apply) { changed = apply && hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess; }
    ~BesideCaptures() { if (changed) (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// The first request on a (device, stream) brings partial sums AND counters, whatever it asks for: a call
// that is captured later may take another kernel than the call that ran before it, and a capture
// does not allow an allocation.
GenWorkspace take_workspace(hipStream_t st, size_t part_floats, size_t ncnt)
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return {};
    const bool capturing = gen_capturing(st);
    const uint64_t thread = ws_thread(st);
    WsTable& table = ws_table();
    std::shared_ptr<WsEntry> e;
    bool taken_over = false;         // what another thread left: its launches may still run
    {
        std::lock_guard<std::mutex> lock(table.mutex);
        std::shared_ptr<WsEntry>& mine = table.entries[{dev, st, thread}];
        if (!mine && thread != 0 && !capturing) {
            const auto it = std::find_if(table.left.begin(), table.left.end(), [&](const auto& l) { return l.first == dev; });
            if (it != table.left.end()) {
                mine = std::move(it->second);
                table.left.erase(it);
                taken_over = true;
            }
        }
        if (!mine) mine = std::make_shared<WsEntry>();
        e = mine;
    }
    e->mutex.lock();
    const BesideCaptures beside(!capturing);
    const bool mark = thread != 0 && !capturing;
    // When the call has enqueued its kernels.  (Measured: a device synchronisation does not wait for the
    // per-thread stream of a thread that has ended.  An event on it tells when its calls are done.)
    auto unlock = [e, st, mark](void*) {
        if (mark && (!e->done || hipEventRecord(e->done, st) != hipSuccess)) {
            (void)hipGetLastError();
            e->retire(e->eager);
        }
        e->mutex.unlock();
    };
    std::shared_ptr<void> use(nullptr, unlock);
    if (taken_over && (!e->done || hipEventSynchronize(e->done) != hipSuccess)) {
        (void)hipGetLastError();
        e->retire(e->eager);
    }
    if (mark && !e->done && hipEventCreateWithFlags(&e->done, hipEventDisableTiming) != hipSuccess) {
        e->done = nullptr;
        (void)hipGetLastError();
        return {};
    }
    WsBlock& b = capturing ? e->captured : e->eager;
    if (!b.holds(part_floats, ncnt)) {
        if (capturing && e->eager.holds(part_floats, ncnt)) {
            e->retire(b);
            std::swap(b, e->eager);
        } else {
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return {};
            WsBlock fresh;
            fresh.part_floats = std::max(part_floats, std::max(kPartFloatsPerCu * (size_t)cus, kGenWorkspaceFloats));
            fresh.ncnt = std::max(ncnt, kCountersPerCu * (size_t)cus);
            if (hipMalloc((void**)&fresh.part, fresh.part_floats * sizeof(float)) != hipSuccess ||
                hipMalloc((void**)&fresh.cnt, fresh.ncnt * sizeof(int)) != hipSuccess || !clear_counters(fresh.cnt, fresh.ncnt, st)) {
                if (fresh.part) (void)hipFree(fresh.part);
                if (fresh.cnt) (void)hipFree(fresh.cnt);
                (void)hipGetLastError();
                return {};
            }
            e->retire(b);
            b = fresh;
        }
    }
    return {b.part, b.cnt, std::move(use)};
}

}  // namespace

GenWorkspace gen_workspace(hipStream_t st, size_t part_floats, size_t ncnt)
{
    try {
        return take_workspace(st, part_floats, ncnt);
    } catch (...) {                                  // (no memory for the table)
        return {};
    }
}

// Releases so far: what is remembered of a workspace from before one is void.
static std::atomic<uint64_t> ws_releases{1};

// A layer that the general kernel would share the tiles of, on a kernel without a workspace: the stream is given its
// block all the same, as programs run such a call before they capture others.  Once: the threads remember the last
// streams that they asked for (the lookup and the questions whether a stream captures cost a call of 8 us 0.4 us).
void bring_workspace(const Shape& s, hipStream_t st)
{
    if (!general_would_share_tiles(s)) return;
    struct Seen { hipStream_t st; int dev; uint64_t releases; };
    thread_local Seen seen[4] = {};
    thread_local unsigned at = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    const uint64_t releases = ws_releases.load(std::memory_order_acquire);      // (before the block is asked for)
    for (const Seen& e : seen)
        if (e.releases == releases && e.st == st && e.dev == dev) return;
    if (gen_capturing(st) || !gen_workspace(st, 0, 0).part) return;
    seen[at++ % 4] = Seen{st, dev, releases};
}

void release_general_workspaces()
{
    WsTable& table = ws_table();
    std::lock_guard<std::mutex> lock(table.mutex);
    auto free_all = [](WsEntry& e) {
        std::lock_guard<std::mutex> held(e.mutex);
        e.free_all();
    };
    for (auto& kv : table.entries) free_all(*kv.second);
    for (auto& l : table.left) free_all(*l.second);
    table.entries.clear();
    table.left.clear();
    ws_releases.fetch_add(1, std::memory_order_acq_rel);
}

// ---- the static scratch array of dconv_general_noalloc --------------------------------------------
// The same two things as the workspace above -- arrival counters, then partial sums -- in device
// memory that comes with the library's code object: every GPU the library runs on holds its own
// copy of the array, at its own address, from the moment the code object is loaded there until
// the process ends.  In host code the array's name only stands for the symbol; its address on
// the current device is looked up once per device and that pointer is what kernels are given.
// All calls on a device share the array (one call at a time, see dconv.h) and it keeps what the
// last call left: the counters a launch uses are cleared on its stream before it, by a kernel,
// so that the call can be captured into a graph.
namespace {

constexpr size_t kScratchCounters = 4096;               // ints: 16 KiB, then the partial sums
constexpr size_t kScratchPartFloats = kGenWorkspaceFloats; // 64 MiB: 512 workgroups x 2 x (64 x 256)
constexpr size_t kScratchBytes = 4 * (kScratchCounters + kScratchPartFloats);
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_scratch_mutex, g_scratch_use[kMaxDevices];  // (of the table below; of each device's array)
unsigned char* g_scratch_ptr[kMaxDevices] = {};         // device address of `scratch`, per device

}  // namespace

int gen_static_workspace(hipStream_t st, size_t part_floats, size_t ncnt, GenWorkspace* ws)
{
    if (part_floats > kScratchPartFloats || ncnt > kScratchCounters) return DCONV_SCRATCH_EXCEEDED;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return DCONV_LAUNCH_FAILED;
    unsigned char* base;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void* q = nullptr;
            if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) {
                (void)hipGetLastError();
                return DCONV_LAUNCH_FAILED;
            }
            g_scratch_ptr[dev] = (unsigned char*)q;
        }
        base = g_scratch_ptr[dev];
    }
    g_scratch_use[dev].lock();
    try {
        ws->use = std::shared_ptr<void>(nullptr, [dev](void*) { g_scratch_use[dev].unlock(); });
    } catch (...) {                                  // (unlocked by the deleter)
        return DCONV_LAUNCH_FAILED;
    }
    ws->cnt = (int*)base;
    ws->part = (float*)(base + 4 * kScratchCounters);
    if (ncnt == 0) return DCONV_OK;
    begin_launch();
    hipLaunchKernelGGL(clear_counters_kernel, dim3((unsigned)((ncnt + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, st, ws->cnt, (int)ncnt);
    return launch_status();
}

// ---- dispatch ----------------------------------------------------------------------------------

namespace {

// Tile configurations offered through the ABI: tile shape x schedule.
//   shape    0: 64 filters x 128 pixels, 1: 64 x 256, 2: 32 x 256
//   schedule 0: by shape, 1: whole tiles only, 2: tiles cut over channels wherever the even
//            split of the work falls, 3: the same on a grid of 7 workgroups (so that small
//            test shapes exercise every way a tile can be shared)
//   write-back: configurations 0 to 11 store straight from the accumulators, 12 to 23 are the
//            same twelve with tiles written back in whole 128-byte lines through LDS (the
//            reorganisation through on-chip memory that the paper leaves open, Sec. 4.2).
//            Measured against each other (paper_1705_10591_amd.tune writeback): the second is
//            never faster, so no shape gets it by itself.  Outputs that fit the 256 MB
//            memory-side cache do not care about line alignment at all; larger ones of narrow
//            maps break even at best, because every accumulator then passes the register file's
//            ports three times (to LDS, back, to memory) instead of once, and those ports are
//            what stores compete for with the matrix cores; wide maps lose up to 40 %, because
//            column strips cut every row into segments whose ends are partial lines anyway.
constexpr int kShapes = 3, kSchedules = 4, kWriteBacks = 2;

int launch_any(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st,
               int tile_cfg, const GenSched& sched, bool dry)
{
    switch (s.F) {
    case 1: return gen_launch_for_F<1>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 2: return gen_launch_for_F<2>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 3: return gen_launch_for_F<3>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 4: return gen_launch_for_F<4>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 5: return gen_launch_for_F<5>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 6: return gen_launch_for_F<6>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 7: return gen_launch_for_F<7>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 8: return gen_launch_for_F<8>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 9: return gen_launch_for_F<9>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 10: return gen_launch_for_F<10>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 11: return gen_launch_for_F<11>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 12: return gen_launch_for_F<12>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 13: return gen_launch_for_F<13>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 14: return gen_launch_for_F<14>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 15: return gen_launch_for_F<15>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 16: return gen_launch_for_F<16>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 17: return gen_launch_for_F<17>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 18: return gen_launch_for_F<18>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 19: return gen_launch_for_F<19>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 20: return gen_launch_for_F<20>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 21: return gen_launch_for_F<21>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 22: return gen_launch_for_F<22>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 23: return gen_launch_for_F<23>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 24: return gen_launch_for_F<24>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 25: return gen_launch_for_F<25>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 26: return gen_launch_for_F<26>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 27: return gen_launch_for_F<27>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 28: return gen_launch_for_F<28>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 29: return gen_launch_for_F<29>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 30: return gen_launch_for_F<30>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 31: return gen_launch_for_F<31>(in, filt, out, s, st, tile_cfg, sched, dry);
    case 32: return gen_launch_for_F<32>(in, filt, out, s, st, tile_cfg, sched, dry);
    default: return DCONV_UNSUPPORTED;
    }
}

// Tile shape by problem shape, from the tile search (paper_1705_10591_amd.tune) over forty layer
// shapes and from timing the three shapes on 630 layers drawn at random (3 to 512 channels, 16 to
// 512 filters of 1x1 to 7x7, 7 x 7 to 224 x 224 maps, 0.5 to 30 GFLOP); the rule below is within
// 1 % of the fastest shape on their average (4 % before it was refitted on them).
int shape_for(const Shape& s)
{
    const int64_t px = (int64_t)s.N * s.Ho * s.Wo;
    const int64_t wide_tiles = (px + 255) / 256, fblocks = (s.K + 63) / 64;
    const int64_t tiles = wide_tiles * fblocks;           // of the 64 x 256 shape
    const int taps = s.C * s.F * s.F;                      // multiply-adds per output element
    const int64_t chunks = ((int64_t)taps + 35) / 36;
    const bool tiny = (int64_t)s.Ho * s.Wo < 100;
    // Up to 32 filters: the 32 x 256 tile, so that half of every filter block is not padding
    // (1x1 filters on tiny maps, where a 256-pixel tile reaches over several images: 64 x 128).
    // (and 1x1 filters on 64 channels or more in a launch of under a hundred wide tiles: the
    // 64 x 128 tile's three workgroups per CU hide the barrier per chunk, which counts for more
    // than the padded half block -- kernel times from replayed graphs, 8 x 64 x 28 x 28 with 32
    // filters: 11.7 -> 8.8 us)
    if (s.K <= 32) return (s.F == 1 && (tiny || (s.C >= 64 && wide_tiles < 100))) ? 0 : 2;
    // Filter counts whose last block of 64 is at most half full (96, 160, 224, 288): the 32 x 256
    // tile computes 25, 17, 12, 10 % fewer padded filters and is 20, 10, 5, 4 % faster from 3x3
    // on (and for the smaller filters with few channels); on tiny maps only for 96.
    // (with few tiles only where a quarter is saved)
    if (s.K % 64 != 0 && s.K % 64 <= 32 && (s.F >= 3 || taps <= 64)) {
        const int k32 = (s.K + 31) / 32 * 32, k64 = (int)fblocks * 64;
        const bool quarter = k32 * 100 <= k64 * 76;
        if (tiles >= (quarter ? 20 : 100) && (quarter || (!tiny && k32 * 100 <= k64 * 91))) return 2;
    }
    // 1x1 filters: a chunk is sixteen channels, eight matrix-core steps and a barrier, whatever
    // the tile, and the 64 x 128 tile's three workgroups per CU hide that better than the four
    // matrix-core instructions per step of the 64 x 256 tile pay: 10-80 % faster from 128
    // channels on, and from 64 on maps up to 64 wide (14 x 14 .. 224 x 224 maps, 32 to 512
    // channels, 64 to 512 filters); with fewer channels or on wider maps the large tile's
    // fewer, longer output runs win by up to 30 %.
    // (a launch of a few tiles: the 32 x 256 tile, twice the tiles, 10-25 % faster in kernel
    // time on 7 x 7 .. 56 x 56 maps with 16 or 32 channels)
    if (s.F == 1) return (s.C >= 128 || (s.C >= 64 && s.Wo <= 64)) ? 0 : tiles < 64 ? 2 : 1;
    // Tiny maps (under a hundred outputs per image): a 256-pixel tile reaches over several
    // images, each with its halo rows in the image block; the 128-pixel tile is 20-35 % faster
    // (7 x 7 outputs, 64 to 512 channels and filters, hundreds of images).
    if (tiny) return 0;
    // 2x2 filters are like 1x1 ones: eight channels a chunk, and beyond 40 channels the small
    // tile is 13-34 % faster (maps up to 60 wide; a tie on the widest).
    if (s.F == 2 && taps > 160) return 0;
    // Few multiply-adds per output element (up to 160): the stores bound the time and the
    // 64 x 256 tile's longer runs win as soon as there are tiles enough for the CUs.
    const bool few_taps = taps <= 160;
    if (s.K <= 64) {
        // 64 x 256 when the work divides finely enough over the chip with it (many tiles, or so
        // many chunks per tile that sharing tiles is cheap), else 64 x 128, which doubles the
        // number of tiles and fits three workgroups per CU.  (With a few dozen wide tiles only,
        // sharing them leaves the chip unevenly loaded however many chunks they have: 512
        // channels, 64 filters of 5x5, 57 wide tiles: 9 % slower.)
        return (wide_tiles >= 1024 || (wide_tiles >= 200 && wide_tiles * chunks >= 12000) ||
                (few_taps && wide_tiles >= 300)) ? 1 : 0;
    }
    if (few_taps) return tiles >= 150 ? 1 : 0;
    return (tiles >= 400 || (tiles >= 100 && chunks >= 100)) ? 1 : 0;
}

}  // namespace

int general_tile_configs() { return kShapes * kSchedules * kWriteBacks; }

int general_auto_shape(const Shape& s) { return shape_for(s); }

namespace {

bool whole_batch_supported(const Shape& s)
{
    const GenSched sched{0, 0, false, false, 0};
    return launch_any(nullptr, nullptr, nullptr, s, nullptr, shape_for(s), sched, true) == DCONV_OK ||
           launch_any(nullptr, nullptr, nullptr, s, nullptr, 0, sched, true) == DCONV_OK;
}

// A batch whose images are so large that a tile reaching from one image into the next would need
// more than 32 bits of lane offset runs image by image (each launch is long: nothing is lost).
bool per_image_supported(const Shape& s, Shape* one)
{
    *one = s;
    one->N = 1;
    return s.N > 1 && whole_batch_supported(*one);
}

}  // namespace

bool general_tiled_supports(const Shape& s)
{
    Shape one;
    return whole_batch_supported(s) || per_image_supported(s, &one);
}

namespace {

int launch_split(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, const GenSched& sched)
{
    switch (s.F) {
    case 2: return split_launch_for_F<2>(in, filt, out, s, st, sched);
    case 3: return split_launch_for_F<3>(in, filt, out, s, st, sched);
    case 4: return split_launch_for_F<4>(in, filt, out, s, st, sched);
    case 5: return split_launch_for_F<5>(in, filt, out, s, st, sched);
    case 6: return split_launch_for_F<6>(in, filt, out, s, st, sched);
    case 7: return split_launch_for_F<7>(in, filt, out, s, st, sched);
    default: return DCONV_UNSUPPORTED;
    }
}

// When the split-operand kernel goes before the fp32 one, and whether its tiles are shared: by
// estimates of the three kernel times, fitted to 1000 layers drawn at random (8 to 512 channels,
// 17 to 512 filters of 2x2 to 7x7, 7 x 7 to 128 x 256 maps, 1 to 64 images, 0.3 to 60 GFLOP; rms
// 5 % whole tiles, 8 % shared, 15 % the fp32 kernel).  Split, per round of tiles over the CUs:
// 0.32 us a matrix-core step of a workgroup, 1.4 us a unit, 4.8 us a tile; 7.6 us for the launch with
// the small kernel in front.  Shared tiles cost 0.41 us a step and the parts of a tile meet at
// about 1.1 us each.  fp32: 133 TFLOP/s of what a block of 32 or 64 filters computes and 8 us, more on
// layers that do not fill the chip.  It has to promise a seventh: over those layers the chosen ones
// are 1.4 times faster on average and 6 of 1000 slower by 3 to 12 %; on 400 others 1.46 times and 1
// slower, by 7 % (profiles/rule_products_of_parts.txt).
// (0: no, 1: whole tiles, 2: shared)
int split_mode(const Shape& s)
{
    if (s.F < 2 || s.F > 7 || s.K < 17) return 0;
    const SplitPlan pl = make_split_plan(s, split_image_rows(s.F), 256, split_most_pixels(s.F));
    if (!pl.ok) return 0;
    constexpr int cus = 256;
    const double tiles = ((double)(pl.nstrips - 1) * pl.pt_full + pl.pt_last) * ((s.K + 63) / 64);
    const double nun = (double)((s.C + 15) / 16) * (s.F / split_image_rows(s.F));
    const double steps = (double)split_image_rows(s.F) * s.F;
    const double rounds = std::ceil(tiles / cus);
    const double taps = (double)s.C * s.F * s.F, px = (double)s.N * s.Ho * s.Wo;
    // (layers of one unit a tile and few taps are bound by their stores, in which the fp32 kernel is better)
    const double stores = nun == 1 && taps <= 160 ? 1.2 : 1.0;
    const double whole = stores * (7.6 + rounds * (nun * (0.319 * steps + 1.41) + 4.8));
    const double units = std::ceil(tiles * nun / cus);
    const double parts = tiles < cus ? std::min<double>(cus, tiles * nun) / tiles : 1.0;
    // (a few tiles of many parts each: the workgroup that adds them takes longer than the estimate)
    const double shared = tiles >= 24 && nun > 1 ? 15.2 + units * (0.413 * steps + 1.36) + 1.9 * rounds + 1.1 * parts : 1e30;
    const int k64 = (s.K + 63) / 64 * 64, k32 = (s.K + 31) / 32 * 32;
    const double mflop = 2e-6 * px * taps * (s.K <= 32 || s.F >= 3 ? k32 : k64);
    const double fp32 = 8.3 + 0.0075 * mflop + 0.278 * std::sqrt(mflop) - 0.33e-6 * px * s.K;
    if (std::min(whole, shared) > 0.86 * fp32) return 0;
    return whole <= shared ? 1 : 2;
}

// Runs the layer on the split-operand kernel; DCONV_UNSUPPORTED if the
// fp32 kernel has to.  A call that is being captured into a graph stays on the fp32 kernel unless
// its scratch memory is the static array: the workspace may have to be allocated, which a capture
// does not allow, and two graphs captured on one stream would share the split filters in it.
int try_split(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, bool static_ws, int mode)
{
    if (!static_ws && gen_capturing(st)) return DCONV_UNSUPPORTED;
    return launch_split(in, filt, out, s, st, GenSched{mode, 0, false, static_ws, 0});
}

}  // namespace

GeneralWay general_way_for(const Shape& s)
{
    Shape one;
    if (!whole_batch_supported(s) && per_image_supported(s, &one)) return general_way_for(one);
    return split_mode(s) != 0 ? GeneralWay::kParts : short_choice(s).time < 1e300 ? GeneralWay::kShort : GeneralWay::kTiled;
}

int launch_general_tiled(const float* in, const float* filt, float* out, const Shape& s, hipStream_t st, int cfg,
                         bool static_ws, GeneralWay way, const ShortChoice* small)
{
    if (cfg >= kShapes * kSchedules * kWriteBacks) return DCONV_UNSUPPORTED;
    Shape one;
    if (!whole_batch_supported(s) && per_image_supported(s, &one)) {
        const int64_t in_image = (int64_t)s.C * s.H * s.W, out_image = (int64_t)s.K * s.Ho * s.Wo;
        for (int n = 0; n < s.N; ++n) {
            const int rc = launch_general_tiled(in + n * in_image, filt, out + n * out_image, one, st, cfg,
                                                static_ws, way);
            if (rc != DCONV_OK) return rc;
        }
        return DCONV_OK;
    }
    switch (way) {
    case GeneralWay::kParts: {
        const int mode = split_mode(s);
        return try_split(in, filt, out, s, st, static_ws, mode ? mode : 1);
    }
    case GeneralWay::kShort: return launch_short(in, filt, out, s, st, short_choice(s).cfg);
    case GeneralWay::kAuto:
        if (const int mode = split_mode(s)) {
            const int rc = try_split(in, filt, out, s, st, static_ws, mode);
            if (rc != DCONV_UNSUPPORTED) return rc;
            break;
        }
        {
            const ShortChoice tiles = small ? *small : short_choice(s);
            if (tiles.time == 1e300) break;
            if (!static_ws) bring_workspace(s, st);
            const int rc = launch_short(in, filt, out, s, st, tiles.cfg);
            if (rc != DCONV_UNSUPPORTED) return rc;
        }
        break;
    case GeneralWay::kTiled: break;
    }
    if (cfg < 0) {
        const GenSched sched{0, 0, false, static_ws, 0};
        int rc = launch_any(in, filt, out, s, st, shape_for(s), sched, false);
        if (rc == DCONV_UNSUPPORTED)
            rc = launch_any(in, filt, out, s, st, 0, sched, false);
        return rc;
    }
    const int schedule = cfg / kShapes % kSchedules;
    const int wb = cfg / (kShapes * kSchedules) + 1;
    const GenSched sched{schedule == 3 ? 2 : schedule, schedule == 3 ? 7 : 0, false, static_ws, wb};
    return launch_any(in, filt, out, s, st, cfg % kShapes, sched, false);
}

}  // namespace dconv
