// router.hip -- C ABI of the gfx950 prefix-cache-aware router (see
// include/prefix_router.h for the contract of every entry point).
//
// Host side: per-peer snapshot copies, the union-forest build, device memory
// with spare capacity for merges, argument checks, the merge round loop and
// launches.  Device side: route_kernels.h (compiled in route.hip), merge_kernels.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <string>
#include <vector>

#include "forest_host.h"
#include "forest_layout.h"
#include "compact_kernels.h"
#include "export_kernels.h"
#include "lru_kernels.h"
#include "merge_kernels.h"
#include "prefix_router.h"
#include "route_launch.h"
#include "small_merge.h"
#include "tree_walk.h"

using pr::Node;

namespace {

thread_local std::string g_err;

pr_status fail(pr_status s, const std::string &msg) {
    g_err = msg;
    return s;
}

pr_status ok() {
    g_err.clear();
    return PR_OK;
}

// Device arrays of the forest.  Node ids and pool offsets never move: growing
// a capacity copies the arrays into larger ones.
struct DevImage {
    // nodes, ntok, nsep, mext and moved share one allocation (node_block)
    void *node_block = nullptr;
    size_t node_block_bytes = 0;
    Node *nodes = nullptr;
    int32_t *ntok = nullptr;
    int32_t *nsep = nullptr;
    uint64_t *mext = nullptr;
    int32_t *pool = nullptr;
    long long *moved = nullptr;
    unsigned long long *ltime = nullptr;  // local peer's access times (allocated while a local peer is set)
    uint16_t *pool16 = nullptr;  // low 16 bits of pool, which routes read while every label token fits 17 bits
    int64_t cap_pool16 = 0;
    uint32_t *hib = nullptr;     // bit 16 of pool token i: bit i % 32 of hib[i / 32] (hib_words(cap_pool16) words),
                                 // zero past the used pool
    int64_t cap_nodes = 0, cap_pool = 0;
    int64_t n_nodes = 0, n_pool = 0;  // host mirror of the device counters
};

// Scratch of one merge call, kept between calls and grown on demand.
struct MergeScratch {
    pr::InsState *st = nullptr;
    unsigned long long *keys_in = nullptr, *keys_out = nullptr;
    int32_t *vals_in = nullptr, *vals_out = nullptr;
    int32_t *grp_nw = nullptr, *grp_nb = nullptr, *win_tok = nullptr, *win_ins = nullptr;
    // add rounds: per sorted entry (cap + 1 entries)
    int32_t *win = nullptr, *widx = nullptr, *headv = nullptr, *hd = nullptr, *nch = nullptr, *cstart = nullptr;
    int32_t *addx = nullptr;   // per insert: parent of an ADD insert, else -1
    int32_t *arest = nullptr;  // per insert: tokens past the walk's end
    int64_t *rest = nullptr, *poff = nullptr, *grp_pool = nullptr, *grp_pb = nullptr;
    int64_t cap = 0;
    void *sort_tmp = nullptr;
    size_t sort_tmp_bytes = 0;
    // snapshot loads on the device path stage their host batch here
    int32_t *load_tok = nullptr;
    int64_t *load_off = nullptr;
    int64_t load_tok_cap = 0, load_seq_cap = 0;
};

// Scratch of snapshot exports, kept between calls and grown on demand.
struct ExportScratch {
    int64_t *depth = nullptr, *len1 = nullptr, *offs = nullptr;
    int32_t *parent = nullptr, *front = nullptr, *next = nullptr, *leaves = nullptr, *sorted = nullptr;
    int32_t *all = nullptr;  // every visited node (LRU eviction)
    int32_t *counts = nullptr;
    void *tmp = nullptr;
    size_t tmp_bytes = 0;
    int64_t cap = 0;  // node capacity of the per-node arrays
};

// Longest-first order of one route call: each query's length bucket, the
// per-workgroup bucket counts and the order itself.  One set per forest,
// grown on demand; `done` is recorded on the stream of the last route that
// used it, and a route on any stream waits for it before reusing the set.
struct RouteScratch {
    int32_t *order = nullptr;
    uint8_t *bkt = nullptr;
    int32_t *blockcnt = nullptr;
    int64_t cap = 0;
    hipEvent_t done = nullptr;
    bool pending = false;
};

}  // namespace

struct pr_forest {
    int32_t P = 0;
    int32_t W = 1;
    int device = -1;
    std::vector<pr::PeerSeqs> sets;
    bool dirty = true;            // host sets changed since the device image was built
    bool merged = false;          // the device image holds merges the host sets lack
    pr::HostImage host_img;
    bool host_img_valid = false;
    DevImage dev;
    bool has_dev = false;
    pr::MergeCounters *d_ctr = nullptr;
    void *h_stage = nullptr;      // pinned host staging for the small readbacks between device rounds
    uint32_t *d_stage = nullptr;  // h_stage as the device addresses it (nullptr: readbacks by DMA)
    unsigned long long *d_skipped = nullptr;  // inputs skipped by device calls
    pr::WalkStatus *d_walk = nullptr;         // what the last one-launch tree walk found
    pr::SizeState *d_size = nullptr;          // a tree size's sum over workgroups, zero between calls
    pr::CompactState *d_compact = nullptr;    // a compaction's ranges and totals
    DevImage spare;               // the arrays the last compaction replaced, for the next one (see retire_image)
    MergeScratch ms;
    ExportScratch xs;
    RouteScratch rs;
    long long stamp = 0;          // add-round counter (stamps of moved records)
    int64_t round_nodes = 0;      // records recent merges added at most (spare capacity kept for the next)
    int64_t round_pool = 0;       // pool tokens, likewise (0: no merge yet)
    int rounds[3] = {2, 2, 2};    // rounds the last batch took (a merge's, a snapshot's, a touch's), kMostRounds at
                                  // most
    int64_t refusals = 0;         // merge rounds repeated after running out of capacity
    int32_t local = -1;           // peer whose tree keeps access times (-1: none)
    int64_t now = 0;              // current time, set by the caller, never decreasing
    int64_t local_load_time = 0;  // time of the local peer's last host snapshot
    int64_t device_bytes = 0;
    int64_t layout_epoch = 0;     // advances whenever the device arrays the route reads move
    bool narrow = false;          // dev.pool16 and dev.hib mirror dev.pool[0, n_pool) (every label token in
                                  // [0, 131071])
    bool hi17 = false;            // some label token is in [65536, 131071]: routes need the bit plane
    bool wide_window = false;     // routes load the wide first-level window: at the last upload the root
                                  // had one child, with a label at least that long (a choice of speed
                                  // only: both windows give the same results)
    bool broken = false;          // a device update failed; only destroy is valid
};

namespace {

#ifndef PR_ROUTE_LONGEST_FIRST
#define PR_ROUTE_LONGEST_FIRST 1
#endif
// Batches of at most pr::kPlanMaxBatch inserts plan their add phase in one
// launch (0: always the multi-launch path, for comparisons).
#ifndef PR_MERGE_PLAN
#define PR_MERGE_PLAN 1
#endif

// Narrow (16- or 17-bit) label copies for routes; 0 keeps every forest on int32 labels.
#ifndef PR_NARROW_LABELS
#define PR_NARROW_LABELS 1
#endif

// Wide first-level window for forests whose root has one long-labelled child
// (0: always the narrow window, for comparisons).
#ifndef PR_WIDE_WINDOW
#define PR_WIDE_WINDOW 1
#endif

// Makes the forest's device current for the duration of a call.
class DeviceScope {
   public:
    explicit DeviceScope(pr_forest *f) {
        if (hipGetDevice(&prev_) != hipSuccess) {
            ok_ = false;
            return;
        }
        if (f->device < 0) f->device = prev_;
        if (f->device != prev_) ok_ = hipSetDevice(f->device) == hipSuccess;
        switched_ = f->device != prev_;
    }
    ~DeviceScope() {
        if (switched_) (void)hipSetDevice(prev_);
    }
    bool ok() const { return ok_; }

   private:
    int prev_ = -1;
    bool ok_ = true;
    bool switched_ = false;
};

constexpr size_t kStageBytes = 256;  // pinned readback staging per forest
constexpr size_t kEvictStage = 128;  // where in it an eviction's status goes (a walk's is at its start)
constexpr unsigned kExportBlocks = 2048;  // workgroups of an export's write when only the device knows its size
constexpr int kCompactLevels = 6;    // levels a compaction enqueues before it reads anything back
constexpr int kDeviceRounds = 2;     // merge rounds queued before each readback but the first
constexpr int kMostRounds = 4;       // ... before the first at most

unsigned grid_threads(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }
unsigned grid_waves(int64_t n) { return (unsigned)((n + pr::kMergeWavesPerBlock - 1) / pr::kMergeWavesPerBlock); }
unsigned grid_walk(int64_t n) { return (unsigned)((n + pr::kMergeWalkWaves - 1) / pr::kMergeWalkWaves); }
unsigned grid_split(int64_t n) { return (unsigned)((n + pr::kSplitWaves - 1) / pr::kSplitWaves); }

bool drop_spare(pr_forest *f);

// Device memory; when there is none left, what the forest keeps for its next
// compaction is given back first.  Every allocation of the library comes here.
bool malloc_or_drop(pr_forest *f, void **p, size_t n) {
    if (hipMalloc(p, n) == hipSuccess) return true;
    (void)hipGetLastError();
    if (drop_spare(f)) {
        if (hipMalloc(p, n) == hipSuccess) return true;
        (void)hipGetLastError();
    }
    *p = nullptr;
    return false;
}

// Device memory the forest keeps.
bool dev_malloc(pr_forest *f, void **p, size_t n) {
    if (!malloc_or_drop(f, p, n)) return false;
    f->device_bytes += (int64_t)n;
    return true;
}

template <typename T>
bool dalloc(pr_forest *f, T **p, int64_t count) {
    return dev_malloc(f, (void **)p, (size_t)std::max<int64_t>(count, 1) * sizeof(T));
}

template <typename T>
void dfree(pr_forest *f, T **p, int64_t count) {
    if (*p) {
        (void)hipFree(*p);
        f->device_bytes -= (int64_t)((size_t)std::max<int64_t>(count, 1) * sizeof(T));
    }
    *p = nullptr;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Words of the bit plane for a pool capacity of cap tokens: two per 64-token
// chunk (a wave writes a chunk's two words together).
int64_t hib_words(int64_t cap) { return 2 * ((cap + 63) / 64) + 2; }

// The per-node arrays of one capacity (records, first tokens, separators,
// extra mask words, move stamps) in one device allocation, each 256-byte
// aligned: growing the forest costs one hipMalloc and one hipFree instead of
// one per array.  Sets d's array pointers and d.cap_nodes.
bool alloc_node_arrays(pr_forest *f, DevImage &d, int64_t cap) {
    const size_t c = (size_t)std::max<int64_t>(cap, 1);
    const size_t o_ntok = align256(c * sizeof(Node));
    const size_t o_nsep = o_ntok + align256(c * sizeof(int32_t));
    const size_t o_mext = o_nsep + align256(c * sizeof(int32_t));
    const size_t o_moved = o_mext + align256(std::max<size_t>(c * (size_t)(f->W - 1), 1) * sizeof(uint64_t));
    const size_t bytes = o_moved + c * sizeof(long long);
    void *b = nullptr;
    if (!dev_malloc(f, &b, bytes)) return false;
    char *p = static_cast<char *>(b);
    d.node_block = b;
    d.node_block_bytes = bytes;
    d.nodes = reinterpret_cast<Node *>(p);
    d.ntok = reinterpret_cast<int32_t *>(p + o_ntok);
    d.nsep = reinterpret_cast<int32_t *>(p + o_nsep);
    d.mext = reinterpret_cast<uint64_t *>(p + o_mext);
    d.moved = reinterpret_cast<long long *>(p + o_moved);
    d.cap_nodes = (int64_t)c;
    return true;
}

void free_node_arrays(pr_forest *f, DevImage &d) {
    if (d.node_block) {
        (void)hipFree(d.node_block);
        f->device_bytes -= (int64_t)d.node_block_bytes;
    }
    d.node_block = nullptr;
    d.node_block_bytes = 0;
    d.nodes = nullptr;
    d.ntok = d.nsep = nullptr;
    d.mext = nullptr;
    d.moved = nullptr;
}

void free_arrays(pr_forest *f, DevImage &d) {
    free_node_arrays(f, d);
    dfree(f, &d.pool, d.cap_pool);
    dfree(f, &d.ltime, d.cap_nodes);
    dfree(f, &d.pool16, d.cap_pool16);
    dfree(f, &d.hib, hib_words(d.cap_pool16));
    d = DevImage();
}

void free_image(pr_forest *f) {
    free_arrays(f, f->dev);
    free_arrays(f, f->spare);
    f->has_dev = false;
    f->narrow = false;
    f->hi17 = false;
}

bool drop_spare(pr_forest *f) {
    const bool any = f->spare.node_block || f->spare.pool;
    free_arrays(f, f->spare);
    return any;
}

int64_t image_bytes(const DevImage &d) {
    return (int64_t)d.node_block_bytes + d.cap_pool * 4 + (d.ltime ? d.cap_nodes * 8 : 0) +
           (d.pool16 ? d.cap_pool16 * 2 + hib_words(d.cap_pool16) * 4 : 0);
}

// Bytes of the records and label tokens an image has in use.
int64_t used_bytes(const pr_forest *f, const DevImage &d) {
    return d.n_nodes * (int64_t)(sizeof(Node) + 2 * sizeof(int32_t) + 8 * f->W) + d.n_pool * (d.pool16 ? 6 : 4);
}

// The image a compaction replaces, nw the one that takes its place.  The old
// arrays are kept for the next compaction, which then allocates nothing (hipMalloc
// and hipFree of arrays of tens of MB take 0.3 to 0.6 ms each, more than the
// rebuild itself): up to 64 MB in any case, more as long as they are small beside
// the GPU's memory and the forest is one that merges fill and compactions empty in
// turn: at least half of what they held is still there, and the new arrays are at
// least a quarter as large (spare capacity grows fourfold).  A compaction that
// shrinks its forest by more gives them back.  At most one set is kept per forest.
constexpr int64_t kSpareBytes = 1ll << 30;
constexpr int64_t kSmallSpare = 64 << 20;
bool retire_image(pr_forest *f, const DevImage &nw) {
    free_arrays(f, f->spare);
    const int64_t bytes = image_bytes(f->dev);
    const bool keep = bytes <= kSmallSpare || (bytes <= kSpareBytes && bytes <= 4 * image_bytes(nw) &&
                                               used_bytes(f, f->dev) <= 2 * used_bytes(f, nw));
    if (keep)
        f->spare = f->dev;
    else
        free_arrays(f, f->dev);
    f->dev = DevImage();
    return keep;
}

// A capacity of at least n with 1/16 to 1/8 slack, so that needs that vary a
// little from one compaction to the next fit the same arrays.
int64_t slack_cap(int64_t n) {
    int64_t g = 1;
    while (g * 16 <= n) g *= 2;
    return (n + g - 1) / g * g;
}

// Node arrays (and access times, if wanted) for at least need records in nw, and
// extra if there is room: the spare's, unless they are too small or far too large.
bool new_node_arrays(pr_forest *f, DevImage &nw, int64_t need, int64_t extra, bool times) {
    const int64_t least = need;
    need += extra;
    DevImage &sp = f->spare;
    if (sp.node_block && sp.cap_nodes >= need && sp.cap_nodes <= 8 * need) {
        nw.node_block = sp.node_block;
        nw.node_block_bytes = sp.node_block_bytes;
        nw.nodes = sp.nodes;
        nw.ntok = sp.ntok;
        nw.nsep = sp.nsep;
        nw.mext = sp.mext;
        nw.moved = sp.moved;
        nw.cap_nodes = sp.cap_nodes;
        nw.ltime = sp.ltime;
        sp.node_block = nullptr;
        sp.node_block_bytes = 0;
        sp.ltime = nullptr;
    } else {
        free_node_arrays(f, sp);
        dfree(f, &sp.ltime, sp.cap_nodes);
        if (!alloc_node_arrays(f, nw, slack_cap(need)) && !alloc_node_arrays(f, nw, least)) return false;
    }
    if (times) return nw.ltime || dalloc(f, &nw.ltime, nw.cap_nodes);
    dfree(f, &nw.ltime, nw.cap_nodes);
    return true;
}

// The label pool (and its narrow copy, if wanted and there is memory for it)
// for at least need tokens in nw, and extra if there is room, in the same way.
constexpr int64_t kSmallPool = 8 << 20;  // tokens a pool may have however few are needed
bool new_pool(pr_forest *f, DevImage &nw, int64_t need, int64_t extra, bool narrow) {
    const int64_t least = need;
    need += extra;
    DevImage &sp = f->spare;
    if (sp.pool && sp.cap_pool >= need && sp.cap_pool <= std::max<int64_t>(2 * need, kSmallPool)) {
        nw.pool = sp.pool;
        nw.cap_pool = sp.cap_pool;
        sp.pool = nullptr;
        sp.cap_pool = 0;
        if (narrow && sp.pool16 && sp.hib && sp.cap_pool16 == nw.cap_pool) {
            nw.pool16 = sp.pool16;
            nw.hib = sp.hib;
            nw.cap_pool16 = sp.cap_pool16;
            sp.pool16 = nullptr;
            sp.hib = nullptr;
            sp.cap_pool16 = 0;
        }
    } else {
        free_arrays(f, sp);
        nw.cap_pool = std::min<int64_t>(slack_cap(need), (int64_t)UINT32_MAX);
        if (!dalloc(f, &nw.pool, nw.cap_pool)) {
            nw.cap_pool = std::min<int64_t>(least, (int64_t)UINT32_MAX);
            if (!dalloc(f, &nw.pool, nw.cap_pool)) return false;
        }
    }
    if (narrow && !nw.pool16) {
        nw.cap_pool16 = nw.cap_pool;
        if (!dalloc(f, &nw.pool16, nw.cap_pool) || !dalloc(f, &nw.hib, hib_words(nw.cap_pool))) {
            dfree(f, &nw.pool16, nw.cap_pool);
            nw.cap_pool16 = 0;
        }
    }
    return true;
}

void free_export_scratch(pr_forest *f) {
    ExportScratch &X = f->xs;
    dfree(f, &X.depth, X.cap);
    dfree(f, &X.len1, X.cap + 1);
    dfree(f, &X.offs, X.cap + 1);
    dfree(f, &X.parent, X.cap);
    dfree(f, &X.front, X.cap);
    dfree(f, &X.next, X.cap);
    dfree(f, &X.leaves, X.cap);
    dfree(f, &X.sorted, X.cap);
    dfree(f, &X.all, X.cap);
    dfree(f, &X.counts, 3);
    if (X.tmp) (void)hipFree(X.tmp);
    f->device_bytes -= (int64_t)X.tmp_bytes;
    X = ExportScratch();
}

void free_add_scratch(pr_forest *f) {
    MergeScratch &m = f->ms;
    const int64_t c = m.cap + 1;
    dfree(f, &m.win, c);
    dfree(f, &m.widx, c);
    dfree(f, &m.headv, c);
    dfree(f, &m.hd, c);
    dfree(f, &m.nch, c);
    dfree(f, &m.cstart, c);
    dfree(f, &m.rest, c);
    dfree(f, &m.poff, c);
    dfree(f, &m.grp_pool, c);
    dfree(f, &m.grp_pb, c);
    dfree(f, &m.arest, c);
    dfree(f, &m.addx, c);
}

void free_scratch(pr_forest *f) {
    MergeScratch &m = f->ms;
    dfree(f, &m.st, m.cap);
    dfree(f, &m.keys_in, m.cap);
    dfree(f, &m.keys_out, m.cap);
    dfree(f, &m.vals_in, m.cap);
    dfree(f, &m.vals_out, m.cap);
    dfree(f, &m.grp_nw, m.cap);
    dfree(f, &m.grp_nb, m.cap);
    dfree(f, &m.win_tok, m.cap);
    dfree(f, &m.win_ins, m.cap);
    free_add_scratch(f);
    if (m.sort_tmp) (void)hipFree(m.sort_tmp);
    f->device_bytes -= (int64_t)m.sort_tmp_bytes;
    dfree(f, &m.load_tok, m.load_tok_cap);
    dfree(f, &m.load_off, m.load_seq_cap + 1);
    m = MergeScratch();
    free_export_scratch(f);
}

// Buffers only (the event stays); callers make sure no route still uses them.
void free_route_buffers(pr_forest *f) {
    RouteScratch &R = f->rs;
    dfree(f, &R.order, R.cap);
    dfree(f, &R.bkt, R.cap);
    dfree(f, &R.blockcnt, (int64_t)pr::kOrderMaxBlocks * pr::kOrderBuckets);
    R.cap = 0;
}

pr_status ensure_host_image(pr_forest *f) {
    if (f->host_img_valid) return PR_OK;
    std::string err;
    pr::HostImage img;
    if (!pr::build_union_image(f->sets, f->W, &img, &err)) return fail(PR_ENOMEM, err);
    f->host_img = std::move(img);
    f->host_img_valid = true;
    return PR_OK;
}

void drop_pool16(pr_forest *f);

// Grow the node and pool capacities to hold at least the given totals.
pr_status ensure_capacity(pr_forest *f, int64_t need_nodes, int64_t need_pool, hipStream_t s) {
    DevImage &d = f->dev;
    if (need_pool > (int64_t)UINT32_MAX) return fail(PR_ENOMEM, "label pool would exceed 2^32 tokens");
    if (need_nodes > (int64_t)INT32_MAX) return fail(PR_ENOMEM, "node count would exceed 2^31");
    if (need_nodes > d.cap_nodes) {
        // rebuilt child blocks append records with every add round, so node
        // arrays grow fourfold: each growth (allocate, copy, wait for the
        // device, free) costs milliseconds of host time; where memory for that is
        // short, to what is needed
        const int64_t cap = std::min<int64_t>(std::max<int64_t>(need_nodes, 4 * d.cap_nodes), (int64_t)INT32_MAX);
        DevImage nd;
        if (!alloc_node_arrays(f, nd, cap) && !alloc_node_arrays(f, nd, need_nodes))
            return fail(PR_ENOMEM, "hipMalloc failed while growing the forest");
        const int64_t n = d.n_nodes;
        if (hipMemcpyAsync(nd.nodes, d.nodes, n * sizeof(Node), hipMemcpyDeviceToDevice, s) != hipSuccess ||
            hipMemcpyAsync(nd.ntok, d.ntok, n * sizeof(int32_t), hipMemcpyDeviceToDevice, s) != hipSuccess ||
            hipMemcpyAsync(nd.nsep, d.nsep, n * sizeof(int32_t), hipMemcpyDeviceToDevice, s) != hipSuccess ||
            (f->W > 1 && hipMemcpyAsync(nd.mext, d.mext, n * (f->W - 1) * sizeof(uint64_t), hipMemcpyDeviceToDevice,
                                        s) != hipSuccess) ||
            hipMemcpyAsync(nd.moved, d.moved, d.cap_nodes * sizeof(long long), hipMemcpyDeviceToDevice, s) !=
                hipSuccess ||
            hipMemsetAsync(nd.moved + d.cap_nodes, 0, (nd.cap_nodes - d.cap_nodes) * sizeof(long long), s) !=
                hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            free_node_arrays(f, nd);
            return fail(PR_EDEVICE, "device copy failed while growing the forest");
        }
        unsigned long long *lt = nullptr;
        if (d.ltime && (!dalloc(f, &lt, nd.cap_nodes) ||
                        hipMemcpyAsync(lt, d.ltime, n * sizeof(unsigned long long), hipMemcpyDeviceToDevice, s) !=
                            hipSuccess ||
                        hipStreamSynchronize(s) != hipSuccess)) {
            dfree(f, &lt, nd.cap_nodes);
            free_node_arrays(f, nd);
            return fail(PR_ENOMEM, "growing the access times failed");
        }
        // a route launched earlier on another stream may still read the old arrays
        if (hipDeviceSynchronize() != hipSuccess) {
            dfree(f, &lt, nd.cap_nodes);
            free_node_arrays(f, nd);
            return fail(PR_EDEVICE, "hipDeviceSynchronize failed while growing the forest");
        }
        if (lt) {
            dfree(f, &d.ltime, d.cap_nodes);
            d.ltime = lt;
        }
        free_node_arrays(f, d);
        d.node_block = nd.node_block;
        d.node_block_bytes = nd.node_block_bytes;
        d.nodes = nd.nodes;
        d.ntok = nd.ntok;
        d.nsep = nd.nsep;
        d.mext = nd.mext;
        d.moved = nd.moved;
        d.cap_nodes = nd.cap_nodes;
        f->layout_epoch++;
    }
    if (need_pool > d.cap_pool) {
        // like the node arrays, a pool that is still small grows fourfold
        const int64_t more = d.cap_pool < (16 << 20) ? 4 * d.cap_pool : d.cap_pool + d.cap_pool / 2;
        int64_t cap = std::min<int64_t>(std::max<int64_t>(need_pool, more), (int64_t)UINT32_MAX);
        int32_t *np = nullptr;
        if (!dalloc(f, &np, cap)) {
            cap = need_pool;
            if (!dalloc(f, &np, cap)) return fail(PR_ENOMEM, "hipMalloc failed while growing the label pool");
        }
        // the narrow copy grows with the pool, under the same wait (without
        // the memory, routes fall back to the int32 pool)
        uint16_t *n16 = nullptr;
        uint32_t *nhb = nullptr;
        const bool narrow = f->narrow && d.pool16 && d.hib;
        const bool keep16 = narrow && dalloc(f, &n16, cap) && dalloc(f, &nhb, hib_words(cap));
        // the tails are zeroed: the bit plane's, because words that two spans share
        // are ORed into it, and the pool's, so that tokens of a refused round, which
        // no label has, have a value
        if (hipMemcpyAsync(np, d.pool, d.n_pool * sizeof(int32_t), hipMemcpyDeviceToDevice, s) != hipSuccess ||
            hipMemsetAsync(np + d.n_pool, 0, (cap - d.n_pool) * sizeof(int32_t), s) != hipSuccess ||
            (keep16 &&
             (hipMemcpyAsync(n16, d.pool16, d.n_pool * sizeof(uint16_t), hipMemcpyDeviceToDevice, s) != hipSuccess ||
              hipMemsetAsync(nhb, 0, hib_words(cap) * sizeof(uint32_t), s) != hipSuccess ||
              hipMemcpyAsync(nhb, d.hib, hib_words(d.n_pool) * sizeof(uint32_t), hipMemcpyDeviceToDevice, s) !=
                  hipSuccess)) ||
            hipStreamSynchronize(s) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
            dfree(f, &np, cap);
            dfree(f, &n16, cap);
            dfree(f, &nhb, hib_words(cap));
            return fail(PR_EDEVICE, "device copy failed while growing the label pool");
        }
        dfree(f, &d.pool, d.cap_pool);
        d.pool = np;
        d.cap_pool = cap;
        if (keep16) {
            dfree(f, &d.pool16, d.cap_pool16);
            dfree(f, &d.hib, hib_words(d.cap_pool16));
            d.pool16 = n16;
            d.hib = nhb;
            d.cap_pool16 = cap;
        } else if (narrow) {
            dfree(f, &n16, cap);
            drop_pool16(f);
        }
        f->layout_epoch++;
    }
    return PR_OK;
}

// Room for the given totals where the ids and the memory allow it: what a merge
// may come to need.  What it does need is a refused round's request.
pr_status reserve_capacity(pr_forest *f, int64_t nodes, int64_t pool, hipStream_t s) {
    const pr_status r = ensure_capacity(f, std::min<int64_t>(nodes, (int64_t)INT32_MAX),
                                        std::min<int64_t>(pool, (int64_t)UINT32_MAX), s);
    return r == PR_ENOMEM ? PR_OK : r;
}

pr::DevForest dev_view(const pr_forest *f);

// The narrow label copy.  While every label token lies in [0, 131071], routes
// read labels from pool16 (the low 16 bits: half the label bytes) and, once
// some token is 65536 or more, from hib (bit 16, one bit per token) as well;
// otherwise from the int32 pool.  Labels are only ever appended to the pool
// (a split reuses a span of its label), and the kernels that append them write
// the copy too (copy_tokens_narrow).
void drop_pool16(pr_forest *f) {
    DevImage &d = f->dev;
    if (d.pool16 || d.hib) {
        // a route launched earlier on another stream may still read them
        (void)hipDeviceSynchronize();
        dfree(f, &d.pool16, d.cap_pool16);
        dfree(f, &d.hib, hib_words(d.cap_pool16));
        f->layout_epoch++;
    }
    d.cap_pool16 = 0;
    f->narrow = false;
    f->hi17 = false;
}

// Access times of the local peer: every node it holds gets time t, others 0.
pr_status init_local_times(pr_forest *f, int64_t t) {
    DevImage &d = f->dev;
    if (!d.ltime && !dalloc(f, &d.ltime, d.cap_nodes)) return fail(PR_ENOMEM, "hipMalloc failed for access times");
    hipLaunchKernelGGL(pr::lru_init_kernel, dim3(grid_threads(std::max<int64_t>(d.n_nodes, 1), 256)), dim3(256), 0,
                       nullptr, dev_view(f), d.n_nodes, (unsigned long long)t);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(nullptr) != hipSuccess)
        return fail(PR_EDEVICE, "access-time initialisation failed");
    return PR_OK;
}

// Rebuild and upload the device image if snapshots changed since the last one.
pr_status commit(pr_forest *f) {
    if (!f->dirty && f->has_dev) return PR_OK;
    pr_status s = ensure_host_image(f);
    if (s) return s;
    if (!f->d_skipped) {
        if (!dalloc(f, &f->d_walk, 1) || !dalloc(f, &f->d_compact, 1) || !dalloc(f, &f->d_ctr, 1) ||
            !dalloc(f, &f->d_size, 1) || !dalloc(f, &f->d_skipped, 1)) {
            dfree(f, &f->d_walk, 1);
            dfree(f, &f->d_size, 1);
            dfree(f, &f->d_compact, 1);
            dfree(f, &f->d_ctr, 1);
            return fail(PR_ENOMEM, "hipMalloc failed");
        }
        if (!f->h_stage && hipHostMalloc(&f->h_stage, kStageBytes, hipHostMallocDefault) != hipSuccess) {
            f->h_stage = nullptr;
            return fail(PR_ENOMEM, "hipHostMalloc failed for the readback staging");
        }
        void *dp = nullptr;
        if (hipHostGetDevicePointer(&dp, f->h_stage, 0) == hipSuccess)
            f->d_stage = static_cast<uint32_t *>(dp);
        else
            (void)hipGetLastError();  // readbacks fall back to DMA copies
        if (hipMemset(f->d_skipped, 0, sizeof(unsigned long long)) != hipSuccess ||
            hipMemset(f->d_size, 0, sizeof(pr::SizeState)) != hipSuccess)
            return fail(PR_EDEVICE, "hipMemset failed");
    }
    // earlier launches may still read the old image
    if (f->has_dev && hipDeviceSynchronize() != hipSuccess) return fail(PR_EDEVICE, "hipDeviceSynchronize failed");
    if (f->has_dev) free_image(f);
    const pr::HostImage &h = f->host_img;
    DevImage &d = f->dev;
    const int64_t n = (int64_t)h.nodes.size(), np = (int64_t)h.pool.size();
    // merges append records (rebuilt blocks move), so node capacity starts at
    // four times the image (a few merge batches before the first growth);
    // labels grow only by new leaves.  At least 1 MiB each: allocations up to
    // there cost a microsecond, each growth of a forest that starts empty and
    // takes its snapshots on the device some hundred
    const int64_t least = 1 << 20, node_bytes = sizeof(Node) + 2 * sizeof(int32_t) + 8 * (int64_t)f->W;
    d.cap_pool = std::max<int64_t>(np + np / 4, least / 4);
    if (!alloc_node_arrays(f, d, std::max<int64_t>(4 * n, least / node_bytes)) || !dalloc(f, &d.pool, d.cap_pool)) {
        free_image(f);
        return fail(PR_ENOMEM, "hipMalloc failed for the forest image");
    }
    if (hipMemcpy(d.nodes, h.nodes.data(), n * sizeof(Node), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(d.ntok, h.ntok.data(), n * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(d.nsep, h.nsep.data(), n * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess ||
        (f->W > 1 && hipMemcpy(d.mext, h.mext.data(), h.mext.size() * sizeof(uint64_t), hipMemcpyHostToDevice) !=
                         hipSuccess) ||
        (np > 0 && hipMemcpy(d.pool, h.pool.data(), np * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess) ||
        hipMemset(d.pool + np, 0, (d.cap_pool - np) * sizeof(int32_t)) != hipSuccess ||
        hipMemset(d.moved, 0, d.cap_nodes * sizeof(long long)) != hipSuccess) {
        free_image(f);
        return fail(PR_EDEVICE, "upload of the forest image failed");
    }
    d.n_nodes = n;
    d.n_pool = np;
    f->wide_window = PR_WIDE_WINDOW && n > 1 && h.nodes[0].ct_cnt == 1 &&
                     h.nodes[(size_t)h.nodes[0].ct_beg].lab_len >= pr::kWave * pr::kWideWinVectors;
    pr::MergeCounters c;
    std::memset(&c, 0, sizeof(c));
    c.n_nodes = (unsigned long long)n;
    c.n_pool = (unsigned long long)np;
    if (hipMemcpy(f->d_ctr, &c, sizeof(c), hipMemcpyHostToDevice) != hipSuccess)
        return fail(PR_EDEVICE, "counter upload failed");
    // narrow labels when every token fits 17 bits (else, or without the memory,
    // int32): the low 16 bits, and bit 16 as a plane once some token needs it
    f->narrow = PR_NARROW_LABELS &&
                std::all_of(h.pool.begin(), h.pool.end(), [](int32_t t) { return (uint32_t)t <= 0x1FFFFu; });
    f->hi17 = f->narrow && std::any_of(h.pool.begin(), h.pool.end(), [](int32_t t) { return (uint32_t)t > 0xFFFFu; });
    if (f->narrow) {
        std::vector<uint16_t> p16;
        std::vector<uint32_t> hb;
        try {
            p16.assign(h.pool.begin(), h.pool.end());  // the low 16 bits
            hb.assign((size_t)hib_words(np), 0u);
            for (int64_t i = 0; i < np; i++) hb[(size_t)(i >> 5)] |= (((uint32_t)h.pool[(size_t)i] >> 16) & 1u) << (i & 31);
        } catch (const std::bad_alloc &) {
            f->narrow = false;
        }
        if (f->narrow && dalloc(f, &d.pool16, d.cap_pool) && dalloc(f, &d.hib, hib_words(d.cap_pool))) {
            d.cap_pool16 = d.cap_pool;
            if ((np > 0 && hipMemcpy(d.pool16, p16.data(), np * sizeof(uint16_t), hipMemcpyHostToDevice) != hipSuccess) ||
                hipMemset(d.hib, 0, hib_words(d.cap_pool) * sizeof(uint32_t)) != hipSuccess ||
                hipMemcpy(d.hib, hb.data(), hb.size() * sizeof(uint32_t), hipMemcpyHostToDevice) != hipSuccess) {
                d.cap_pool16 = d.cap_pool;
                free_image(f);
                return fail(PR_EDEVICE, "upload of the narrow labels failed");
            }
        } else {
            dfree(f, &d.pool16, d.cap_pool);
            dfree(f, &d.hib, hib_words(d.cap_pool));
            f->narrow = false;
        }
    }
    if (!f->narrow) f->hi17 = false;
    f->has_dev = true;
    f->dirty = false;
    f->merged = false;
    f->layout_epoch++;
    if (f->local >= 0) {
        pr_status r = init_local_times(f, f->local_load_time);
        if (r) return r;
    }
    // the device image is the state of record now; drop the host copy of it
    f->host_img = pr::HostImage();
    f->host_img_valid = false;
    return PR_OK;
}

// Longest-first order: the dispatcher starts one wave per query in index
// order and refills a slot when its query ends, so with only a few long
// queries per slot the last long ones to start leave most slots idle at the
// end of the launch.  Taking the batch longest first removes that tail.  It
// pays where a wave slot of the chip (256 CUs x 32 waves) gets between one
// and eight queries of at least 4,096 tokens on average; elsewhere the order
// kernel (a few microseconds) costs more than the tail.
bool use_longest_first(int64_t nq, int64_t ntok) {
    const int64_t slots = 256 * 32;
    return PR_ROUTE_LONGEST_FIRST && nq > slots && nq <= 8 * slots && nq <= pr::kOrderMaxQueries &&
           ntok >= 4096 * nq;
}

// Fill f->rs.order with the queries longest first (two launches of at most 16
// workgroups) on stream s; length buckets are a quarter of the mean query wide.
pr_status route_order(pr_forest *f, const int64_t *q_offsets, int64_t nq, int64_t ntok, hipStream_t s,
                      const int32_t **order) {
    RouteScratch &R = f->rs;
    if (!R.done && hipEventCreateWithFlags(&R.done, hipEventDisableTiming) != hipSuccess) {
        R.done = nullptr;
        return fail(PR_EDEVICE, "hipEventCreate failed");
    }
    if (nq > R.cap) {
        // an earlier route, on any stream, may still read the old buffer
        if (R.pending && hipEventSynchronize(R.done) != hipSuccess)
            return fail(PR_EDEVICE, "waiting for an earlier route failed");
        R.pending = false;
        free_route_buffers(f);
        const int64_t cap = std::max<int64_t>(nq, std::min<int64_t>(2 * R.cap, pr::kOrderMaxQueries));
        R.cap = cap;  // sizes for free_route_buffers, also after a partial allocation
        if (!dalloc(f, &R.order, cap) || !dalloc(f, &R.bkt, cap) ||
            !dalloc(f, &R.blockcnt, (int64_t)pr::kOrderMaxBlocks * pr::kOrderBuckets)) {
            free_route_buffers(f);
            return fail(PR_ENOMEM, "hipMalloc failed for the route order");
        }
    }
    if (R.pending && hipStreamWaitEvent(s, R.done, 0) != hipSuccess)
        return fail(PR_EDEVICE, "hipStreamWaitEvent failed");
    if (pr::launch_route_order(q_offsets, nq, ntok, s, R.bkt, R.blockcnt, R.order) != hipSuccess)
        return fail(PR_EDEVICE, "route order launch failed");
    *order = R.order;
    return PR_OK;
}

// The forest as a route reads it: over the narrow labels when they are current.
pr::RouteForest route_view(const pr_forest *f) {
    const DevImage &d = f->dev;
    const bool narrow = f->narrow && d.pool16 && d.hib;
    return pr::RouteForest{d.nodes, d.ntok, d.nsep, d.mext, d.pool, narrow ? d.pool16 : nullptr,
                           narrow && f->hi17 ? d.hib : nullptr, f->P, f->W, f->wide_window};
}

// ---- routes without allocation ----------------------------------------------
// The longest-first order of one pr_route_noalloc call lives in one
// file-scope device array per GPU (`scratch`, held until the process ends):
// order (int32 per query), the per-workgroup bucket counts, then each query's
// length bucket (uint8).  On the host the array's name stands for no device
// address; its address on each device comes from hipGetSymbolAddress, taken
// once per device with that device current, and only that address is passed
// to kernels.
constexpr int64_t kNoAllocOrder = 0;
constexpr int64_t kNoAllocBlockcnt = kNoAllocOrder + 4 * (int64_t)pr::kOrderMaxQueries;
constexpr int64_t kNoAllocBkt = kNoAllocBlockcnt + 4 * (int64_t)pr::kOrderMaxBlocks * pr::kOrderBuckets;
constexpr int64_t kNoAllocBytes = kNoAllocBkt + (int64_t)pr::kOrderMaxQueries;
static_assert(PR_NOALLOC_MAX_QUERIES == pr::kOrderMaxQueries, "the header's limit is the order's capacity");
static_assert(kNoAllocBlockcnt % 256 == 0 && kNoAllocBkt % 256 == 0, "aligned sub-arrays");
constexpr int kNoAllocMaxDevices = 64;

}  // namespace

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {

std::mutex g_scratch_mu;
unsigned char *g_scratch_dev[kNoAllocMaxDevices] = {};

// The current device's address of `scratch` (dev must be current).
pr_status noalloc_scratch(int dev, unsigned char **out) {
    if (dev < 0 || dev >= kNoAllocMaxDevices) return fail(PR_EDEVICE, "device id beyond the scratch table");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return fail(PR_EDEVICE, std::string("hipGetSymbolAddress of the route scratch failed: ") +
                                        hipGetErrorString(e));
        }
        g_scratch_dev[dev] = static_cast<unsigned char *>(p);
    }
    *out = g_scratch_dev[dev];
    return PR_OK;
}

// ---- merge ------------------------------------------------------------------

pr_status ensure_merge_scratch(pr_forest *f, int64_t n, hipStream_t s) {
    MergeScratch &m = f->ms;
    if (n > m.cap) {
        const int64_t cap = std::max<int64_t>(n, m.cap * 2);
        dfree(f, &m.st, m.cap);
        dfree(f, &m.keys_in, m.cap);
        dfree(f, &m.keys_out, m.cap);
        dfree(f, &m.vals_in, m.cap);
        dfree(f, &m.vals_out, m.cap);
        dfree(f, &m.grp_nw, m.cap);
        dfree(f, &m.grp_nb, m.cap);
        dfree(f, &m.win_tok, m.cap);
        dfree(f, &m.win_ins, m.cap);
        free_add_scratch(f);
        m.cap = 0;
        const int64_t c1 = cap + 1;
        if (!dalloc(f, &m.st, cap) || !dalloc(f, &m.keys_in, cap) || !dalloc(f, &m.keys_out, cap) ||
            !dalloc(f, &m.vals_in, cap) || !dalloc(f, &m.vals_out, cap) || !dalloc(f, &m.grp_nw, cap) ||
            !dalloc(f, &m.grp_nb, cap) || !dalloc(f, &m.win_tok, cap) || !dalloc(f, &m.win_ins, cap) ||
            !dalloc(f, &m.win, c1) || !dalloc(f, &m.widx, c1) || !dalloc(f, &m.headv, c1) ||
            !dalloc(f, &m.hd, c1) || !dalloc(f, &m.nch, c1) || !dalloc(f, &m.cstart, c1) ||
            !dalloc(f, &m.rest, c1) || !dalloc(f, &m.poff, c1) || !dalloc(f, &m.grp_pool, c1) ||
            !dalloc(f, &m.grp_pb, c1) || !dalloc(f, &m.arest, c1) || !dalloc(f, &m.addx, c1)) {
            m.cap = cap;  // so that free_scratch releases the add arrays by their size
            free_scratch(f);
            return fail(PR_ENOMEM, "hipMalloc failed for merge scratch");
        }
        m.cap = cap;
    }
    // one temporary buffer serves the sort and the add round's scans
    size_t need = 0, q = 0;
    if (rocprim::radix_sort_pairs(nullptr, need, m.keys_in, m.keys_out, m.vals_in, m.vals_out, n, 0, 64, s) !=
        hipSuccess)
        return fail(PR_EDEVICE, "radix sort size query failed");
    if (rocprim::exclusive_scan(nullptr, q, m.win, m.widx, 0, (size_t)n, rocprim::plus<int32_t>(), s) != hipSuccess)
        return fail(PR_EDEVICE, "scan size query failed");
    need = std::max(need, q);
    if (rocprim::exclusive_scan(nullptr, q, m.rest, m.poff, (int64_t)0, (size_t)n, rocprim::plus<int64_t>(), s) !=
        hipSuccess)
        return fail(PR_EDEVICE, "scan size query failed");
    need = std::max(need, q);
    if (rocprim::inclusive_scan(nullptr, q, m.headv, m.hd, (size_t)n, rocprim::maximum<int32_t>(), s) != hipSuccess)
        return fail(PR_EDEVICE, "scan size query failed");
    need = std::max(need, q);
    if (rocprim::exclusive_scan(nullptr, q, m.nch, m.cstart, 0, (size_t)n + 1, rocprim::plus<int32_t>(), s) !=
        hipSuccess)
        return fail(PR_EDEVICE, "scan size query failed");
    need = std::max(need, q);
    if (need > m.sort_tmp_bytes) {
        if (m.sort_tmp) (void)hipFree(m.sort_tmp);
        f->device_bytes -= (int64_t)m.sort_tmp_bytes;
        m.sort_tmp_bytes = 0;
        m.sort_tmp = nullptr;
        if (!dev_malloc(f, &m.sort_tmp, need)) return fail(PR_ENOMEM, "hipMalloc failed for sort scratch");
        m.sort_tmp_bytes = need;
    }
    return PR_OK;
}

__global__ void reset_round_kernel(pr::MergeCounters *c) {
    c->n_add = 0;
    c->n_split = 0;
    c->pool_need = 0;
    c->node_need = 0;
    c->move_chunks = 0;
    c->plan_alloc = 0;
    c->plan_fallback = 0;
}

// The counters of a forest that was just compacted.
__global__ void compact_counters_kernel(pr::MergeCounters *c, const pr::CompactState *S) {
    if (S->bad) return;
    *c = pr::MergeCounters{};
    c->n_nodes = (unsigned long long)S->hi;
    c->n_pool = (unsigned long long)S->n_pool;
}

// The end of a merge: its skipped inputs are added up, and every counter but
// the used sizes is cleared for the next one.
__global__ void add_skipped_kernel(unsigned long long *acc, pr::MergeCounters *c) {
    *acc += c->skipped;
    pr::MergeCounters z{};
    z.n_nodes = c->n_nodes;
    z.n_pool = c->n_pool;
    *c = z;
}

// Counters after refused allocations: the used sizes the host clipped to the
// capacities, and no refusal pending.
__global__ void set_used_kernel(pr::MergeCounters *c, unsigned long long n_nodes, unsigned long long n_pool) {
    c->n_nodes = n_nodes;
    c->n_pool = n_pool;
    c->overflow = 0;
}

// One wave stores the words of a small readback straight into the pinned
// staging buffer, at system scope (past the GPU's caches).
__global__ void stage_copy_kernel(const uint32_t *src, uint32_t *dst, int words) {
    for (int i = (int)threadIdx.x; i < words; i += (int)blockDim.x)
        __hip_atomic_store(&dst[i], src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Copy `bytes` (<= kStageBytes) of device memory to the host through the
// forest's pinned staging buffer and wait.  Whole aligned words go through a
// one-wave kernel that writes the buffer directly (a DMA copy of a few bytes
// costs a blit launch several times as long); anything else by DMA.
bool read_small(pr_forest *f, void *out, const void *dsrc, size_t bytes, hipStream_t s) {
    if (bytes > kStageBytes || !f->h_stage) return false;
    if (f->d_stage && bytes % 4 == 0 && reinterpret_cast<uintptr_t>(dsrc) % 4 == 0) {
        hipLaunchKernelGGL(stage_copy_kernel, dim3(1), dim3(64), 0, s, static_cast<const uint32_t *>(dsrc),
                           f->d_stage, (int)(bytes / 4));
        if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return false;
    } else if (hipMemcpyAsync(f->h_stage, dsrc, bytes, hipMemcpyDeviceToHost, s) != hipSuccess ||
               hipStreamSynchronize(s) != hipSuccess) {
        return false;
    }
    std::memcpy(out, f->h_stage, bytes);
    return true;
}

static_assert(sizeof(pr::MergeCounters) <= kStageBytes && sizeof(pr::SmallStatus) <= kStageBytes && sizeof(pr::EvictPlan) <= kStageBytes &&
                  sizeof(pr::CompactState) <= kStageBytes,
              "readbacks fit the staging buffer");

// The counters only (the caller decides what the used sizes are).
pr_status read_counters_raw(pr_forest *f, pr::MergeCounters *c, hipStream_t s) {
    if (!read_small(f, c, f->d_ctr, sizeof(*c), s)) return fail(PR_EDEVICE, "reading merge counters failed");
    return PR_OK;
}

pr::DevForest dev_view(const pr_forest *f) {
    pr::DevForest F;
    F.nodes = f->dev.nodes;
    F.ntok = f->dev.ntok;
    F.nsep = f->dev.nsep;
    F.mext = f->dev.mext;
    F.pool = f->dev.pool;
    F.moved = f->dev.moved;
    F.ltime = f->local >= 0 ? f->dev.ltime : nullptr;
    F.local = f->local;
    F.now = (unsigned long long)f->now;
    F.cap_nodes = f->dev.cap_nodes;
    F.cap_pool = f->dev.cap_pool;
    F.W = f->W;
    return F;
}


// A batch of device sequences for run_merge: inserts into peer_of[i]'s trees,
// or into one peer's (peer_of nullptr), or touches of one peer's.
pr::Batch batch_of(const pr_forest *f, const int32_t *peer_of, int32_t peer, const int32_t *tokens,
                   int64_t num_tokens, const int64_t *offsets, int64_t n) {
    return pr::Batch{peer_of, tokens, offsets, num_tokens, n, f->P, peer, 0};
}

// What a merge's appended labels mean for the narrow copy: hi, wide count (or
// flag) tokens in [65536, 131071] and outside [0, 131071].
void narrow_seen(pr_forest *f, bool hi, bool wide) {
    if (wide)
        drop_pool16(f);
    else if (hi && f->narrow && !f->hi17) {
        f->hi17 = true;  // routes now read the bit plane too (a new kernel: the arrays stay)
        f->layout_epoch++;
    }
}

pr::NarrowDst narrow_dst(const pr_forest *f) {
    return pr::NarrowDst{f->narrow ? f->dev.pool16 : nullptr, f->dev.hib};
}

// One launch of the one-workgroup merge (small_merge.h) and one wait: a batch
// of at most pr::kSmallMax sequences (states nullptr), or what rounds left of a
// larger one (its states).
pr_status run_small_merge(pr_forest *f, const pr::Batch &B, const pr::InsState *states, hipStream_t s,
                          pr::SmallStatus *st) {
    DevImage &d = f->dev;
    hipLaunchKernelGGL(pr::small_merge_kernel, dim3(1), dim3(64 * pr::kSmallWaves), 0, s, dev_view(f), B,
                       narrow_dst(f), f->d_ctr, f->d_skipped, states, f->stamp + 1,
                       reinterpret_cast<pr::SmallStatus *>(f->d_stage));
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return fail(PR_EDEVICE, "merge failed");
    std::memcpy(st, f->h_stage, sizeof(*st));
    f->stamp += st->stamps;
    if (!st->overflow) {  // else refused requests advanced the counters (refused_round)
        d.n_nodes = (int64_t)st->n_nodes;
        d.n_pool = (int64_t)st->n_pool;
    }
    narrow_seen(f, st->hi != 0, st->wide != 0);
    f->merged = true;
    return PR_OK;
}

// A round ran out of capacity.  Every refused allocation wrote nothing and left
// its inserts to walk again, but the refused requests still advanced the
// counters (to asked_nodes and asked_pool).  The counters are clipped to the
// capacities (below them, what a refused request got is records that no peer
// holds, and tokens that no label has), and the forest grows before the round is
// repeated: to the records it asked for and to want_pool tokens, and, if there is
// room, to pool_need past the clipped ones.
pr_status refused_round(pr_forest *f, int64_t asked_nodes, int64_t asked_pool, int64_t want_pool, int64_t pool_need,
                        hipStream_t s) {
    f->refusals++;
    f->dev.n_nodes = std::min<int64_t>(asked_nodes, f->dev.cap_nodes);
    f->dev.n_pool = std::min<int64_t>(asked_pool, f->dev.cap_pool);
    hipLaunchKernelGGL(set_used_kernel, dim3(1), dim3(1), 0, s, f->d_ctr, (unsigned long long)f->dev.n_nodes,
                       (unsigned long long)f->dev.n_pool);
    if (hipGetLastError() != hipSuccess) return fail(PR_EDEVICE, "merge launch failed");
    asked_nodes = std::max<int64_t>(asked_nodes, f->dev.n_nodes + 1);
    const pr_status r = reserve_capacity(f, asked_nodes, std::max<int64_t>(want_pool, f->dev.n_pool + pool_need), s);
    return r ? r : ensure_capacity(f, asked_nodes, want_pool, s);
}

// Insert a device batch into the device forest (see merge_kernels.h), or touch
// the local peer's tree with it.
pr_status run_merge(pr_forest *f, const pr::Batch &B, hipStream_t s) {
    const int64_t pool0 = f->dev.n_pool;  // labels appended from here on
    const int64_t nodes0 = f->dev.n_nodes;
    const int64_t n = B.n;
    pr_status r;
    pr::SmallStatus ss;
    // one workgroup serves a batch up to a lane per sequence in about the time
    // of five launches, unless its sequences are long (the rounds below take
    // eleven launches)
    if (n <= pr::kSmallMax && f->d_stage) {
        if ((r = run_small_merge(f, B, nullptr, s, &ss))) return r;
        if (ss.done) return PR_OK;
    }
    if ((r = ensure_merge_scratch(f, n, s))) return r;
    MergeScratch &m = f->ms;
    const int bs = 256, wb = 64 * pr::kMergeWavesPerBlock;
    const unsigned plan_grid = (unsigned)pr::plan_blocks(n);
    const unsigned build_blocks = (unsigned)std::min<int64_t>(pr::kMoveBlocks, std::max<int64_t>(256, n / 4));
    int first = 1;  // the next walk is the first to look at the batch
    bool done = false;
    // Rounds the device drives: full rounds, each sized on the device (the add
    // phase planned there, the later steps striding over what it planned), then
    // one workgroup, which finishes up to pr::kSmallMax inserts that are left, and
    // one readback.  Most batches end there: the first round places every insert
    // but the losers of a slot or an edge, the second those, but for the losers
    // among them.  With more left, as when many sequences share a prefix the
    // forest does not have (a slot, then an edge, then the slots below it), more
    // rounds run.  As many are queued first as the last batch of the kind took (a
    // readback and its wait cost 25 us, a round with nothing to do 16): one for a
    // peer's next snapshot, most of which the forest still has, four for the first
    // ones of a cold start, three for 10,000 requests.  Anything else (a round too
    // large for the plan, a refused allocation) continues in the host-driven
    // rounds below, which read the counters back after every walk.
    int &taken = f->rounds[B.touch ? 2 : B.peer_of ? 0 : 1];
    int queued = 0;
    pr::MergeCounters c;
    std::memset(&c, 0, sizeof(c));
    // walk every unfinished insert, tally what the walks found and read it back
    auto walk_and_tally = [&](int round) {
        hipLaunchKernelGGL(reset_round_kernel, dim3(1), dim3(1), 0, s, f->d_ctr);
        hipLaunchKernelGGL(pr::merge_walk_kernel, dim3(grid_walk(n)), dim3(64 * pr::kMergeWalkWaves), 0, s, dev_view(f),
                           B, m.st, m.addx, m.arest, f->d_ctr, round);
        hipLaunchKernelGGL(pr::merge_tally_kernel,
                           dim3((unsigned)std::min<int64_t>(256, (n + pr::kTallyThreads - 1) / pr::kTallyThreads)),
                           dim3(pr::kTallyThreads), 0, s, B, m.st, f->d_ctr);
        return read_counters_raw(f, &c, s);
    };
    const bool device_rounds = PR_MERGE_PLAN && f->d_stage && n <= pr::kPlanMaxBatch;
    // A forest whose merges have not shown what they add, and a batch of more than
    // four times what its pool has left (prompts share most of their tokens): the
    // first round's walk is tallied, and the pool grows by that and, as at an
    // upload, a quarter, where a refused allocation would take a second set of
    // launches (first snapshot of 4,000 prompts of 2,000 tokens: 687 to 1,253 us
    // refused, 510 to 531 us).  Up to there the tally costs about what the
    // refusals do that it spares (500 prompts of 1,200 tokens, which do not fit:
    // 451 us with it, 473 without; 16 snapshots of 500, of which the first fits,
    // 2,864 with it, 2,812 without).
    bool walked = false;
    if (device_rounds && f->round_pool == 0 && !B.touch && B.num_tokens / 4 > f->dev.cap_pool - f->dev.n_pool) {
        if ((r = walk_and_tally(1)) ||
            (r = reserve_capacity(f, f->dev.n_nodes + n, f->dev.n_pool + (int64_t)(c.pool_need + c.pool_need / 4), s)))
            return r;
        walked = true;
        first = 0;
        queued = 1;
    }
    for (int k = 0; device_rounds && !done && k < 4; k++) {
        if ((r = reserve_capacity(f, f->dev.n_nodes + std::max<int64_t>(f->round_nodes, n),
                                  f->dev.n_pool + (B.touch ? 0 : f->round_pool), s)))
            return r;
        const pr::DevForest F = dev_view(f);
        const pr::NarrowDst N = narrow_dst(f);
        for (int left = k == 0 ? taken : kDeviceRounds; left > 0; left--, first = 0) {
            const long long stamp = ++f->stamp;
            if (!walked)
                hipLaunchKernelGGL(pr::merge_walk_kernel, dim3(grid_walk(n)), dim3(64 * pr::kMergeWalkWaves), 0, s, F,
                                   B, m.st, m.addx, m.arest, f->d_ctr, ++queued);
            walked = false;
            if (!B.touch) {  // touches add nothing
                hipLaunchKernelGGL(pr::add_plan_kernel, dim3(plan_grid), dim3(pr::kPlanThreads), 0, s, F, B, m.st,
                                   m.addx, m.arest, m.keys_out, m.vals_out, m.win, m.widx, m.hd, m.cstart, m.grp_nw,
                                   m.grp_nb, m.win_tok, m.rest, f->d_ctr);
                hipLaunchKernelGGL(pr::add_build_kernel, dim3(build_blocks), dim3(wb), 0, s, F, B, N, m.keys_out,
                                   m.vals_out, (int64_t)-1, m.st, m.win, m.widx, m.poff, m.hd, m.cstart, m.grp_nw,
                                   m.grp_nb, m.grp_pb, m.rest, m.win_tok, f->d_ctr, stamp);
            }
            hipLaunchKernelGGL(pr::add_finish_kernel, dim3(grid_threads(n, bs)), dim3(bs), 0, s, F, B, m.st,
                               m.keys_out, (int64_t)(B.touch ? 0 : -1), m.grp_nw, m.grp_nb, stamp, f->d_ctr);
            hipLaunchKernelGGL(pr::split_apply_kernel, dim3(grid_split(n)), dim3(64 * pr::kSplitWaves), 0, s, F, B, N,
                               m.st, f->d_ctr, stamp);
        }
        if (hipGetLastError() != hipSuccess) return fail(PR_EDEVICE, "merge launch failed");
        if ((r = run_small_merge(f, B, m.st, s, &ss))) return r;
        done = ss.done != 0;
        // (the next round's walk is tallied, which says what tokens are needed)
        if (ss.overflow && (r = refused_round(f, (int64_t)ss.n_nodes, (int64_t)ss.n_pool, 0, 0, s))) return r;
        if (ss.overflow || ss.fallback) break;
        // one more where the last workgroup had several inserts for a wave
        taken = std::min(std::max((int)ss.rounds + (ss.left > (uint32_t)pr::kSmallWaves), 1), kMostRounds);
    }
    const int max_rounds = 100000;
    int round = 0;
    int refusals = 0;
    const bool host_rounds = !done;
    for (; !done && round < max_rounds; round++, first = 0) {
        if ((r = walk_and_tally(first ? 1 : 0))) return r;
        if (c.overflow) {
            if (++refusals > 4) break;  // reported below
            if ((r = refused_round(f, (int64_t)c.n_nodes, (int64_t)c.n_pool, (int64_t)c.n_pool, (int64_t)c.pool_need,
                                   s)))
                return r;
            continue;
        }
        f->dev.n_nodes = (int64_t)c.n_nodes;
        f->dev.n_pool = (int64_t)c.n_pool;
        if (c.n_add == 0 && c.n_split == 0) break;
        // One round applies both kinds from the same walk: the add phase first
        // (rebuilt child blocks move records; the split phase finds them through
        // their move stamps), then the split phase.  The winners of either are
        // done; the losers (the same slot or the same edge as a winner) walk
        // again.  Allocations come from the device counters; one that does not
        // fit the capacity is refused (see refused_round), so no readback sits
        // between the phases.  A forest whose spare capacity is short of what the
        // last merges added grows first (the walk's tally bounds the pool tokens).
        const int64_t n_split = (int64_t)c.n_split, n_add = (int64_t)c.n_add;
        if ((r = reserve_capacity(f, f->dev.n_nodes + std::max<int64_t>(f->round_nodes, n),
                                  f->dev.n_pool + (int64_t)c.pool_need, s)))
            return r;
        const pr::DevForest F = dev_view(f);
        const pr::NarrowDst N = narrow_dst(f);
        long long add_stamp = 0;
        const bool plan = PR_MERGE_PLAN && n_add > 0 && n_add <= pr::kPlanMax && n <= pr::kPlanMaxBatch;
        if (n_add > 0) {
            if (plan) {
                // sort, marks, scans and groups in one launch
                hipLaunchKernelGGL(pr::add_plan_kernel, dim3(plan_grid), dim3(pr::kPlanThreads), 0, s, F, B, m.st,
                                   m.addx, m.arest, m.keys_out, m.vals_out, m.win, m.widx, m.hd, m.cstart, m.grp_nw,
                                   m.grp_nb, m.win_tok, m.rest, f->d_ctr);
            } else {
                hipLaunchKernelGGL(pr::add_keys_kernel, dim3(grid_threads(n, bs)), dim3(bs), 0, s, B, m.st, m.keys_in,
                                   m.vals_in);
                size_t tmp = m.sort_tmp_bytes;
                if (rocprim::radix_sort_pairs(m.sort_tmp, tmp, m.keys_in, m.keys_out, m.vals_in, m.vals_out, n, 0, 64,
                                              s) != hipSuccess)
                    return fail(PR_EDEVICE, "radix sort failed");
                // winners, group heads and chunks; their scans; per-group totals
                hipLaunchKernelGGL(pr::add_mark_kernel, dim3(grid_threads(n_add + 1, bs)), dim3(bs), 0, s, F, B,
                                   m.keys_out, m.vals_out, n_add, m.st, m.win, m.rest, m.headv, m.nch);
                size_t t1 = m.sort_tmp_bytes;
                if (rocprim::exclusive_scan(m.sort_tmp, t1, m.win, m.widx, 0, (size_t)n_add, rocprim::plus<int32_t>(),
                                            s) != hipSuccess)
                    return fail(PR_EDEVICE, "add scan failed");
                t1 = m.sort_tmp_bytes;
                if (rocprim::exclusive_scan(m.sort_tmp, t1, m.rest, m.poff, (int64_t)0, (size_t)n_add,
                                            rocprim::plus<int64_t>(), s) != hipSuccess)
                    return fail(PR_EDEVICE, "add scan failed");
                t1 = m.sort_tmp_bytes;
                if (rocprim::inclusive_scan(m.sort_tmp, t1, m.headv, m.hd, (size_t)n_add, rocprim::maximum<int32_t>(),
                                            s) != hipSuccess)
                    return fail(PR_EDEVICE, "add scan failed");
                t1 = m.sort_tmp_bytes;
                if (rocprim::exclusive_scan(m.sort_tmp, t1, m.nch, m.cstart, 0, (size_t)n_add + 1,
                                            rocprim::plus<int32_t>(), s) != hipSuccess)
                    return fail(PR_EDEVICE, "add scan failed");
                hipLaunchKernelGGL(reset_round_kernel, dim3(1), dim3(1), 0, s, f->d_ctr);
                hipLaunchKernelGGL(pr::add_group_kernel, dim3(grid_threads(n_add, bs)), dim3(bs), 0, s, F,
                                   m.keys_out, m.vals_out, n_add, m.st, m.win, m.rest, m.widx, m.poff, m.hd, m.cstart,
                                   m.grp_nw, m.grp_pool, m.win_tok, m.win_ins, f->d_ctr);
                hipLaunchKernelGGL(pr::add_alloc_kernel, dim3(grid_threads(n_add, bs)), dim3(bs), 0, s, F, m.keys_out,
                                   n_add, m.grp_nw, m.grp_pool, m.grp_nb, m.grp_pb, f->d_ctr);
            }
            add_stamp = ++f->stamp;
            hipLaunchKernelGGL(pr::add_build_kernel, dim3(std::max<unsigned>(pr::kMoveBlocks, grid_waves(n_add))),
                               dim3(wb), 0, s, F, B, N, m.keys_out, m.vals_out, plan ? -1 : n_add, m.st, m.win, m.widx, m.poff, m.hd, m.cstart,
                               m.grp_nw, m.grp_nb, m.grp_pb, plan ? m.rest : nullptr, m.win_tok, f->d_ctr, add_stamp);
        }
        hipLaunchKernelGGL(pr::add_finish_kernel, dim3(grid_threads(n, bs)), dim3(bs), 0, s, F, B, m.st, m.keys_out,
                           plan ? -1 : n_add, m.grp_nw, m.grp_nb, add_stamp, f->d_ctr);
        if (n_split > 0)
            hipLaunchKernelGGL(pr::split_apply_kernel, dim3(grid_split(n)), dim3(64 * pr::kSplitWaves), 0, s, F, B, N,
                               m.st, f->d_ctr, add_stamp);
        if (hipGetLastError() != hipSuccess) return fail(PR_EDEVICE, "merge launch failed");
    }
    if (round == max_rounds) return fail(PR_EDEVICE, "merge did not converge");
    // records and pool tokens the largest recent merge added: the spare
    // capacity the next one finds free (snapshot loads between two merge
    // batches, which add little, shrink it slowly).  A compaction leaves room
    // for two such merges, so that a period of loads, a merge and a compaction
    // settles on arrays that never grow
    f->round_nodes = std::max<int64_t>(f->dev.n_nodes - nodes0, f->round_nodes - f->round_nodes / 32);
    f->round_pool = std::max<int64_t>({f->dev.n_pool - pool0, f->round_pool - f->round_pool / 32, 1});
    if (!host_rounds) return PR_OK;
    // the last readback saw the last round's work; the counters are cleared for
    // the next call
    hipLaunchKernelGGL(add_skipped_kernel, dim3(1), dim3(1), 0, s, f->d_skipped, f->d_ctr);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return fail(PR_EDEVICE, "merge failed");
    if (c.overflow)
        return fail(PR_EDEVICE, "merge invariant broken (overflow " + std::to_string(c.overflow) + "); destroy the forest");
    narrow_seen(f, c.hi_tokens != 0, c.wide_tokens != 0);
    f->merged = true;
    return PR_OK;
}

// Snapshot load once merges have run: the host copies no longer describe the
// device forest, so the replacement happens on the device: clear the peer from
// every mask, then insert the snapshot for it.
pr_status device_load(pr_forest *f, int32_t peer, const pr::PeerSeqs &S) {
    MergeScratch &m = f->ms;
    const int64_t ns = S.count(), nt = (int64_t)S.tokens.size();
    hipStream_t s = nullptr;
    hipLaunchKernelGGL(pr::clear_peer_kernel, dim3(grid_threads(f->dev.n_nodes, 256)), dim3(256), 0, s,
                       dev_view(f), f->dev.n_nodes, peer);
    if (hipGetLastError() != hipSuccess) return fail(PR_EDEVICE, "snapshot kernels failed to launch");
    if (ns == 0) return hipStreamSynchronize(s) == hipSuccess ? PR_OK : fail(PR_EDEVICE, "sync failed");
    if (nt > m.load_tok_cap) {
        dfree(f, &m.load_tok, m.load_tok_cap);
        m.load_tok_cap = 0;
        if (!dalloc(f, &m.load_tok, nt)) return fail(PR_ENOMEM, "hipMalloc failed for the snapshot");
        m.load_tok_cap = nt;
    }
    if (ns > m.load_seq_cap) {
        dfree(f, &m.load_off, m.load_seq_cap + 1);
        m.load_seq_cap = 0;
        if (!dalloc(f, &m.load_off, ns + 1)) return fail(PR_ENOMEM, "hipMalloc failed for the snapshot");
        m.load_seq_cap = ns;
    }
    if ((nt > 0 && hipMemcpy(m.load_tok, S.tokens.data(), nt * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess) ||
        hipMemcpy(m.load_off, S.offsets.data(), (ns + 1) * sizeof(int64_t), hipMemcpyHostToDevice) != hipSuccess)
        return fail(PR_EDEVICE, "snapshot upload failed");
    return run_merge(f, batch_of(f, nullptr, peer, m.load_tok, nt, m.load_off, ns), s);
}

pr_status ensure_export_scratch(pr_forest *f, int64_t nn) {
    ExportScratch &X = f->xs;
    if (nn <= X.cap && X.counts) return PR_OK;
    const int64_t cap = std::max<int64_t>(nn, X.cap + X.cap / 2);
    free_export_scratch(f);
    if (!dalloc(f, &X.depth, cap) || !dalloc(f, &X.len1, cap + 1) || !dalloc(f, &X.offs, cap + 1) ||
        !dalloc(f, &X.parent, cap) || !dalloc(f, &X.front, cap) || !dalloc(f, &X.next, cap) ||
        !dalloc(f, &X.leaves, cap) || !dalloc(f, &X.sorted, cap) || !dalloc(f, &X.all, cap) ||
        !dalloc(f, &X.counts, 3)) {
        free_export_scratch(f);
        return fail(PR_ENOMEM, "hipMalloc failed for the export");
    }
    X.cap = cap;
    return PR_OK;
}

// Walk peer's nodes level by level from the root (export_kernels.h) into the
// forest's export scratch: depth and parent of every visited node, the leaves
// (counts[1]) and, if want_all, every visited node (counts[2]).
pr_status walk_peer(pr_forest *f, int32_t peer, bool want_all, hipStream_t s, int32_t counts[3]) {
    const int64_t nn = f->dev.n_nodes;
    pr_status r = ensure_export_scratch(f, nn);
    if (r) return r;
    ExportScratch &X = f->xs;
    const pr::DevForest F = dev_view(f);
    const int wb = 64 * pr::kExportWavesPerBlock;
    hipLaunchKernelGGL(pr::export_init_kernel, dim3(1), dim3(1), 0, s, X.front, X.depth, X.counts);
    int32_t n_front = 1;
    counts[0] = counts[1] = counts[2] = 0;
    while (n_front > 0) {
        hipLaunchKernelGGL(pr::export_reset_kernel, dim3(1), dim3(1), 0, s, X.counts);
        hipLaunchKernelGGL(pr::export_level_kernel,
                           dim3((unsigned)((n_front + pr::kExportWavesPerBlock - 1) / pr::kExportWavesPerBlock)),
                           dim3(wb), 0, s, F, nn, peer, X.front, n_front, X.next, X.leaves, X.depth, X.parent,
                           X.counts, want_all ? X.all : nullptr);
        if (hipGetLastError() != hipSuccess) return fail(PR_EDEVICE, "tree walk launch failed");
        if (!read_small(f, counts, X.counts, 3 * sizeof(int32_t), s))
            return fail(PR_EDEVICE, "tree walk readback failed");
        if (counts[0] > nn || counts[1] > nn || counts[2] > nn)
            return fail(PR_EDEVICE, "tree walk visited more nodes than exist");
        n_front = counts[0];
        std::swap(X.front, X.next);
    }
    return PR_OK;
}

// One-launch walk of peer's tree (tree_walk.h) with the outputs O asks for,
// enqueued; its status goes to f->d_walk and to the start of the pinned buffer.
bool enqueue_walk(pr_forest *f, int32_t peer, const pr::WalkOut &O, hipStream_t s) {
    hipLaunchKernelGGL(pr::tree_walk_kernel, dim3(1), dim3(pr::kWalkThreads), 0, s, dev_view(f), f->dev.n_nodes, peer,
                       O, f->d_walk, reinterpret_cast<pr::WalkStatus *>(f->d_stage));
    return hipGetLastError() == hipSuccess;
}

pr_status export_too_small(int64_t seqs, int64_t tokens) {
    return fail(PR_EINVAL, "export buffers too small: need " + std::to_string(seqs + 1) + " offsets and " +
                               std::to_string(tokens) + " tokens");
}

// sendTrie for one peer (see export_kernels.h).  Host-synchronous.  Writes the
// sizes always; the data only if both buffers are given and large enough.
pr_status export_impl(pr_forest *f, int32_t peer, int32_t *tokens, int64_t tokens_cap, int64_t *offsets,
                      int64_t seqs_cap, int64_t *num_seqs, int64_t *num_tokens, hipStream_t s) {
    const int64_t nn = f->dev.n_nodes;
    pr_status r = ensure_export_scratch(f, nn);
    if (r) return r;
    ExportScratch &X = f->xs;
    const pr::DevForest F = dev_view(f);
    const int wb = 64 * pr::kExportWavesPerBlock;
    if (f->d_stage) {
        // a tree that one workgroup walks: sizes, or sizes, order and offsets, in
        // one launch, the tokens in a second, and one wait
        const bool fill = offsets != nullptr;
        const pr::WalkOut O{X.depth, X.parent, nullptr, X.leaves, X.sorted, offsets, seqs_cap,
                            tokens ? tokens_cap : 0};
        if (!enqueue_walk(f, peer, O, s)) return fail(PR_EDEVICE, "tree walk launch failed");
        if (fill)
            hipLaunchKernelGGL(pr::export_write_kernel, dim3(kExportBlocks), dim3(wb), 0, s, F, X.sorted, 0, f->d_walk,
                               X.depth, X.parent, offsets, tokens);
        if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
            return fail(PR_EDEVICE, "export failed");
        pr::WalkStatus st;
        std::memcpy(&st, f->h_stage, sizeof(st));
        if (st.done) {
            *num_seqs = st.leaves;
            *num_tokens = (int64_t)st.leaf_tokens;
            if ((!tokens && !offsets) || (fill && st.fits)) return ok();
            return export_too_small(*num_seqs, *num_tokens);
        }
    }
    int32_t counts[3] = {0, 0, 0};
    r = walk_peer(f, peer, false, s, counts);
    if (r) return r;
    const int32_t n_leaves = counts[1];
    int64_t total = 0;
    if (n_leaves > 0) {
        size_t need = 0, need2 = 0;
        if (rocprim::radix_sort_keys(nullptr, need, X.leaves, X.sorted, (size_t)n_leaves, 0, 32, s) != hipSuccess ||
            rocprim::inclusive_scan(nullptr, need2, X.len1 + 1, X.offs + 1, (size_t)n_leaves,
                                    rocprim::plus<int64_t>(), s) != hipSuccess)
            return fail(PR_EDEVICE, "export sort / scan sizing failed");
        need = std::max(need, need2);
        if (need > X.tmp_bytes) {
            if (X.tmp) (void)hipFree(X.tmp);
            f->device_bytes -= (int64_t)X.tmp_bytes;
            X.tmp = nullptr;
            X.tmp_bytes = 0;
            if (!dev_malloc(f, &X.tmp, need)) return fail(PR_ENOMEM, "hipMalloc failed for the export");
            X.tmp_bytes = need;
        }
        size_t t1 = need;
        if (rocprim::radix_sort_keys(X.tmp, t1, X.leaves, X.sorted, (size_t)n_leaves, 0, 32, s) != hipSuccess)
            return fail(PR_EDEVICE, "export sort failed");
        hipLaunchKernelGGL(pr::export_lengths_kernel, dim3(grid_threads(n_leaves, 256)), dim3(256), 0, s, X.sorted,
                           n_leaves, X.depth, X.len1);
        size_t t2 = need;
        if (rocprim::inclusive_scan(X.tmp, t2, X.len1 + 1, X.offs + 1, (size_t)n_leaves, rocprim::plus<int64_t>(),
                                    s) != hipSuccess)
            return fail(PR_EDEVICE, "export scan failed");
        if (!read_small(f, &total, X.offs + n_leaves, sizeof(total), s))
            return fail(PR_EDEVICE, "export readback failed");
    }
    *num_seqs = n_leaves;
    *num_tokens = total;
    if (!tokens && !offsets) return ok();
    if (!offsets || (total > 0 && !tokens) || tokens_cap < total || seqs_cap < (int64_t)n_leaves + 1)
        return export_too_small(n_leaves, total);
    const int64_t zero = 0;
    if (hipMemcpyAsync(offsets, &zero, sizeof(zero), hipMemcpyHostToDevice, s) != hipSuccess)
        return fail(PR_EDEVICE, "export copy failed");
    if (n_leaves > 0) {
        if (hipMemcpyAsync(offsets + 1, X.offs + 1, (size_t)n_leaves * sizeof(int64_t), hipMemcpyDeviceToDevice,
                           s) != hipSuccess)
            return fail(PR_EDEVICE, "export copy failed");
        hipLaunchKernelGGL(pr::export_write_kernel,
                           dim3((unsigned)((n_leaves + pr::kExportWavesPerBlock - 1) / pr::kExportWavesPerBlock)),
                           dim3(wb), 0, s, F, X.sorted, n_leaves, (const pr::WalkStatus *)nullptr, X.depth, X.parent,
                           offsets, tokens);
        if (hipGetLastError() != hipSuccess) return fail(PR_EDEVICE, "export launch failed");
    }
    if (hipStreamSynchronize(s) != hipSuccess) return fail(PR_EDEVICE, "export failed");
    return ok();
}

// Device buffers of one touch or eviction call, released on every return path.
struct CallScratch {
    pr_forest *f;
    std::vector<void *> bufs;
    explicit CallScratch(pr_forest *f) : f(f) {}
    template <typename T>
    bool get(T **p, int64_t count) {
        if (!malloc_or_drop(f, (void **)p, (size_t)std::max<int64_t>(count, 1) * sizeof(T))) return false;
        bufs.push_back((void *)*p);
        return true;
    }
    ~CallScratch() {
        for (void *b : bufs) (void)hipFree(b);
    }
};

}  // namespace

extern "C" {

int32_t pr_abi_version(void) { return PR_ABI_VERSION; }

const char *pr_last_error(void) { return g_err.c_str(); }

pr_status pr_forest_create(int32_t num_peers, pr_forest **out) {
    if (!out) return fail(PR_EINVAL, "out is NULL");
    *out = nullptr;
    if (num_peers < 1 || num_peers > PR_MAX_PEERS)
        return fail(PR_EINVAL, "num_peers must be in [1, " + std::to_string(PR_MAX_PEERS) + "]");
    pr_forest *f = new (std::nothrow) pr_forest();
    if (!f) return fail(PR_ENOMEM, "host allocation failed");
    f->P = num_peers;
    f->W = pr::mask_words_for(num_peers);
    try {
        f->sets.resize((size_t)num_peers);
    } catch (const std::bad_alloc &) {
        delete f;
        return fail(PR_ENOMEM, "host allocation failed");
    }
    *out = f;
    return ok();
}

void pr_forest_destroy(pr_forest *f) {
    if (!f) return;
    if (f->device >= 0) {
        DeviceScope ds(f);
        (void)hipDeviceSynchronize();
        free_image(f);
        free_scratch(f);
        dfree(f, &f->d_skipped, 1);
        dfree(f, &f->d_ctr, 1);
        dfree(f, &f->d_walk, 1);
        dfree(f, &f->d_size, 1);
        dfree(f, &f->d_compact, 1);
        if (f->h_stage) (void)hipHostFree(f->h_stage);
        free_route_buffers(f);
        if (f->rs.done) (void)hipEventDestroy(f->rs.done);
    }
    delete f;
}

pr_status pr_load_snapshot(pr_forest *f, int32_t peer, const int32_t *tokens, const int64_t *offsets,
                           int64_t num_seqs) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (peer < 0 || peer >= f->P) return fail(PR_EINVAL, "peer out of range");
    if (num_seqs < 0) return fail(PR_EINVAL, "num_seqs < 0");
    if (!offsets) return fail(PR_EINVAL, "offsets is NULL");
    if (offsets[0] != 0) return fail(PR_EINVAL, "offsets[0] != 0");
    for (int64_t i = 0; i < num_seqs; i++)
        if (offsets[i + 1] < offsets[i]) return fail(PR_EINVAL, "offsets decrease at sequence " + std::to_string(i));
    if (offsets[num_seqs] > 0 && !tokens) return fail(PR_EINVAL, "tokens is NULL");
    if (num_seqs > (int64_t)INT32_MAX) return fail(PR_EINVAL, "too many sequences");
    const int64_t ntok = offsets[num_seqs];
    pr::PeerSeqs S;
    try {
        S.tokens.assign(tokens, tokens + ntok);
        S.offsets.assign(offsets, offsets + num_seqs + 1);
    } catch (const std::bad_alloc &) {
        return fail(PR_ENOMEM, "host allocation failed");
    }
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    if (f->has_dev && f->merged) {
        DeviceScope ds(f);
        if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
        pr_status r = device_load(f, peer, S);
        if (r) {
            f->broken = true;
            return r;
        }
        f->sets[(size_t)peer] = std::move(S);
        return ok();
    }
    f->sets[(size_t)peer] = std::move(S);
    f->dirty = true;
    f->host_img_valid = false;
    if (peer == f->local) f->local_load_time = f->now;
    return ok();
}

pr_status pr_merge(pr_forest *f, const int32_t *peer_of, const int32_t *tokens, int64_t num_tokens,
                   const int64_t *offsets, int64_t num_seqs, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (num_seqs < 0 || num_tokens < 0) return fail(PR_EINVAL, "negative count");
    if (num_seqs == 0) return ok();
    if (!peer_of || !offsets) return fail(PR_EINVAL, "NULL device pointer");
    if (num_tokens > 0 && !tokens) return fail(PR_EINVAL, "tokens is NULL");
    if (num_seqs > (int64_t)INT32_MAX) return fail(PR_EINVAL, "too many sequences");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    pr_status s = commit(f);
    if (s) return s;
    s = run_merge(f, batch_of(f, peer_of, 0, tokens, num_tokens, offsets, num_seqs), (hipStream_t)hip_stream);
    if (s) {
        f->broken = true;
        return s;
    }
    return ok();
}

pr_status pr_load_snapshot_device(pr_forest *f, int32_t peer, const int32_t *tokens, int64_t num_tokens,
                                  const int64_t *offsets, int64_t num_seqs, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (peer < 0 || peer >= f->P) return fail(PR_EINVAL, "peer out of range");
    if (num_seqs < 0 || num_tokens < 0) return fail(PR_EINVAL, "negative count");
    if (num_seqs > 0 && !offsets) return fail(PR_EINVAL, "offsets is NULL");
    if (num_tokens > 0 && !tokens) return fail(PR_EINVAL, "tokens is NULL");
    if (num_seqs > (int64_t)INT32_MAX) return fail(PR_EINVAL, "too many sequences");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    pr_status r = commit(f);
    if (r) return r;
    hipStream_t s = (hipStream_t)hip_stream;
    hipLaunchKernelGGL(pr::clear_peer_kernel, dim3(grid_threads(f->dev.n_nodes, 256)), dim3(256), 0, s,
                       dev_view(f), f->dev.n_nodes, peer);
    if (hipGetLastError() != hipSuccess) {
        f->broken = true;
        return fail(PR_EDEVICE, "snapshot kernels failed to launch");
    }
    if (num_seqs > 0) {
        r = run_merge(f, batch_of(f, nullptr, peer, tokens, num_tokens, offsets, num_seqs), s);
    } else {
        r = hipStreamSynchronize(s) == hipSuccess ? PR_OK : fail(PR_EDEVICE, "sync failed");
        f->merged = true;
    }
    if (r) {
        f->broken = true;
        return r;
    }
    f->sets[(size_t)peer] = pr::PeerSeqs();  // the host copy no longer describes the peer
    return ok();
}

pr_status pr_export_snapshot(pr_forest *f, int32_t peer, int32_t *tokens, int64_t tokens_cap, int64_t *offsets,
                             int64_t seqs_cap, int64_t *num_seqs, int64_t *num_tokens, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (peer < 0 || peer >= f->P) return fail(PR_EINVAL, "peer out of range");
    if (!num_seqs || !num_tokens) return fail(PR_EINVAL, "size outputs are NULL");
    if (tokens_cap < 0 || seqs_cap < 0) return fail(PR_EINVAL, "negative capacity");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    pr_status r = commit(f);
    if (r) return r;
    return export_impl(f, peer, tokens, tokens_cap, offsets, seqs_cap, num_seqs, num_tokens,
                       (hipStream_t)hip_stream);
}

pr_status pr_forest_compact(pr_forest *f, int64_t *nodes_before, int64_t *nodes_after, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    pr_status r = commit(f);
    if (r) return r;
    hipStream_t s = (hipStream_t)hip_stream;
    DevImage &d = f->dev;
    const int64_t n_old = d.n_nodes;
    if (nodes_before) *nodes_before = n_old;
    if ((r = ensure_export_scratch(f, n_old))) return r;
    ExportScratch &X = f->xs;
    // the new image: the old node count, 1/8 spare and what recent merges added;
    // labels sized once the live ones are known
    DevImage nw;
    auto fail_new = [&](pr_status st, const char *m) {
        free_arrays(f, nw);
        return fail(st, m);
    };
    if (!new_node_arrays(f, nw, std::max<int64_t>(n_old + n_old / 8, 1024), 2 * f->round_nodes, d.ltime != nullptr))
        return fail_new(PR_ENOMEM, "hipMalloc failed for the compacted forest");
    const pr::DevForest O = dev_view(f);
    pr::DevForest N = O;
    N.nodes = nw.nodes;
    N.ntok = nw.ntok;
    N.nsep = nw.nsep;
    N.mext = nw.mext;
    N.moved = nw.moved;
    N.ltime = d.ltime ? nw.ltime : nullptr;
    N.pool = nullptr;
    N.cap_nodes = nw.cap_nodes;
    const bool narrow = f->narrow && d.pool16 && d.hib;
    auto pool_need = [&](int64_t n) { return std::max<int64_t>(n + n / 8, 4096); };
    int32_t *old_of = X.front, *start = X.next;
    int64_t *off = X.len1, *blk = X.offs;
    pr::CompactState S;
    // a small forest's labels are bounded by the old pool's, so that it takes
    // one wait
    const bool small = n_old <= pr::kCompactSmall;
    const bool one_wait = small && d.n_pool <= (4 << 20);
    if (small) {
        hipLaunchKernelGGL(pr::compact_small_kernel, dim3(1), dim3(pr::kCompactThreads), 0, s, O, N, old_of, off,
                           n_old, f->d_compact);
    } else {
        hipLaunchKernelGGL(pr::compact_init_kernel, dim3(1), dim3(1), 0, s, O, N, old_of, f->d_compact);
        const unsigned g = (unsigned)std::min<int64_t>(2048, (n_old + pr::kCompactWaves - 1) / pr::kCompactWaves);
        do {
            for (int level = 0; level < kCompactLevels; level++) {
                hipLaunchKernelGGL(pr::compact_count_kernel, dim3(g), dim3(pr::kCompactThreads), 0, s, O, old_of,
                                   f->d_compact, start, blk);
                hipLaunchKernelGGL(pr::compact_scan_kernel, dim3(1), dim3(pr::kCompactThreads), 0, s, f->d_compact,
                                   blk, n_old);
                hipLaunchKernelGGL(pr::compact_copy_kernel, dim3(g), dim3(pr::kCompactThreads), 0, s, O, N, old_of,
                                   f->d_compact, start, blk);
            }
            hipLaunchKernelGGL(pr::compact_lab_kernel, dim3(g), dim3(pr::kCompactThreads), 0, s, N, f->d_compact, off,
                               blk);
            hipLaunchKernelGGL(pr::compact_lab_scan_kernel, dim3(1), dim3(pr::kCompactThreads), 0, s, f->d_compact,
                               blk);
            if (hipGetLastError() != hipSuccess || !read_small(f, &S, f->d_compact, sizeof(S), s))
                return fail_new(PR_EDEVICE, "compaction failed");
        } while (S.lo < S.hi && !S.bad);
    }
    if (small && !one_wait && !read_small(f, &S, f->d_compact, sizeof(S), s))
        return fail_new(PR_EDEVICE, "compaction failed");
    if (!one_wait) {
        if (S.bad) return fail_new(PR_EDEVICE, "compaction found more live nodes than exist");
        if (S.n_pool > (int64_t)UINT32_MAX) return fail_new(PR_EDEVICE, "compacted label pool exceeds 2^32 tokens");
    }
    const int64_t pool_from = one_wait ? 0 : S.n_pool;  // tokens past the used ones are zero
    if (!new_pool(f, nw, pool_need(one_wait ? d.n_pool : S.n_pool), 2 * f->round_pool, narrow))
        return fail_new(PR_ENOMEM, "hipMalloc failed for the compacted label pool");
    N.pool = nw.pool;
    N.cap_pool = nw.cap_pool;
    const unsigned gl = std::max(1u, grid_threads(one_wait ? d.n_pool : S.n_pool, pr::kCompactSeg));
    if (hipMemsetAsync(nw.pool + pool_from, 0, (nw.cap_pool - pool_from) * sizeof(int32_t), s) != hipSuccess ||
        (nw.pool16 && hipMemsetAsync(nw.hib, 0, hib_words(nw.cap_pool16) * sizeof(uint32_t), s) != hipSuccess) ||
        hipMemsetAsync(nw.moved, 0, nw.cap_nodes * sizeof(long long), s) != hipSuccess)
        return fail_new(PR_EDEVICE, "compaction memset failed");
    hipLaunchKernelGGL(pr::compact_labels_kernel, dim3(gl), dim3(pr::kCompactSegThreads), 0, s, O, N,
                       pr::NarrowDst{nw.pool16, nw.hib}, old_of, f->d_compact, off, small ? nullptr : blk);
    hipLaunchKernelGGL(compact_counters_kernel, dim3(1), dim3(1), 0, s, f->d_ctr, f->d_compact);
    if (hipGetLastError() != hipSuccess || !read_small(f, &S, f->d_compact, sizeof(S), s)) {
        f->broken = true;  // the counters may be the new image's already
        return fail_new(PR_EDEVICE, "compaction failed");
    }
    if (S.bad) return fail_new(PR_EDEVICE, "compaction found more live nodes than exist");
    // install the new image once no launch on another stream still reads the old one
    if (hipDeviceSynchronize() != hipSuccess) return fail_new(PR_EDEVICE, "hipDeviceSynchronize failed");
    nw.n_nodes = S.hi;
    nw.n_pool = S.n_pool;
    const bool kept = retire_image(f, nw);
    f->dev = nw;
    f->layout_epoch++;
    f->stamp = 0;  // no record carries a move stamp
    f->narrow = narrow && nw.pool16;
    f->hi17 = f->narrow && S.hi_tokens;  // the rebuilt pool holds only live labels
    if (f->narrow && S.wide_tokens) drop_pool16(f);
    f->host_img_valid = false;  // the host image no longer mirrors the device layout
    // scratch sized for far more records than are left goes back
    if (X.cap > (kept ? 4 : 2) * nw.n_nodes + (1 << 16)) free_export_scratch(f);
    if (nodes_after) *nodes_after = nw.n_nodes;
    return ok();
}

pr_status pr_tree_tokens(pr_forest *f, int32_t peer, int64_t *tokens, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (peer < 0 || peer >= f->P) return fail(PR_EINVAL, "peer out of range");
    if (!tokens) return fail(PR_EINVAL, "tokens is NULL");
    *tokens = 0;
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    pr_status r = commit(f);
    if (r) return r;
    hipStream_t s = (hipStream_t)hip_stream;
    if (f->d_stage && f->dev.n_nodes > pr::kSizeRecords) {
        if (!enqueue_walk(f, peer, pr::WalkOut{}, s) || hipStreamSynchronize(s) != hipSuccess)
            return fail(PR_EDEVICE, "tree walk failed");
        pr::WalkStatus st;
        std::memcpy(&st, f->h_stage, sizeof(st));
        if (st.done) {
            *tokens = (int64_t)st.tokens;
            return ok();
        }
    }
    if (f->d_stage) {
        const unsigned blocks = std::min(pr::kSizeBlocks, grid_threads(f->dev.n_nodes, pr::kSizeThreads * pr::kSizePer));
        hipLaunchKernelGGL(pr::tree_size_kernel, dim3(std::max(1u, blocks)), dim3(pr::kSizeThreads), 0, s, dev_view(f),
                           f->dev.n_nodes, peer, f->d_size, reinterpret_cast<unsigned long long *>(f->d_stage));
        if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
            return fail(PR_EDEVICE, "tree size failed");
        std::memcpy(tokens, f->h_stage, sizeof(*tokens));
        return ok();
    }
    int32_t counts[3];
    if ((r = walk_peer(f, peer, true, s, counts))) return r;
    if (counts[2] == 0) return ok();
    CallScratch X(f);
    unsigned long long *d = nullptr;
    if (!X.get(&d, 1)) return fail(PR_ENOMEM, "hipMalloc failed");
    unsigned long long h = 0;
    if (hipMemsetAsync(d, 0, sizeof(h), s) != hipSuccess) return fail(PR_EDEVICE, "hipMemsetAsync failed");
    hipLaunchKernelGGL(pr::tree_tokens_kernel, dim3(grid_threads(counts[2], 256)), dim3(256), 0, s, dev_view(f),
                       f->xs.all, counts[2], d);
    if (hipGetLastError() != hipSuccess || !read_small(f, &h, d, sizeof(h), s))
        return fail(PR_EDEVICE, "tree size failed");
    *tokens = (int64_t)h;
    return ok();
}

pr_status pr_set_local_peer(pr_forest *f, int32_t peer) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (peer < -1 || peer >= f->P) return fail(PR_EINVAL, "peer out of range");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    f->local = peer;
    f->local_load_time = f->now;
    if (!f->has_dev) return ok();
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    if (hipDeviceSynchronize() != hipSuccess) return fail(PR_EDEVICE, "hipDeviceSynchronize failed");
    if (peer < 0) {
        dfree(f, &f->dev.ltime, f->dev.cap_nodes);
        return ok();
    }
    if (f->dirty) return ok();  // the next rebuild initialises the times
    pr_status r = init_local_times(f, f->now);
    if (r) {
        f->broken = true;
        return r;
    }
    return ok();
}

pr_status pr_set_time(pr_forest *f, int64_t t) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (t < f->now) return fail(PR_EINVAL, "time must not decrease");
    f->now = t;
    return ok();
}

pr_status pr_touch(pr_forest *f, const int32_t *q_tokens, int64_t num_tokens, const int64_t *q_offsets,
                   int64_t num_queries, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (num_queries < 0 || num_tokens < 0) return fail(PR_EINVAL, "negative count");
    if (f->local < 0) return fail(PR_ESTATE, "no local peer is set");
    if (num_queries == 0) return ok();
    if (!q_offsets) return fail(PR_EINVAL, "NULL device pointer");
    if (num_tokens > 0 && !q_tokens) return fail(PR_EINVAL, "q_tokens is NULL");
    if (num_queries > (int64_t)INT32_MAX) return fail(PR_EINVAL, "too many queries");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    pr_status r = commit(f);
    if (r) return r;
    // the walk of a touch ends where the local tree does: it adds nothing but
    // node boundaries where a prefix ends inside a label, and stamps the paths
    pr::Batch B = batch_of(f, nullptr, f->local, q_tokens, num_tokens, q_offsets, num_queries);
    B.touch = 1;
    r = run_merge(f, B, (hipStream_t)hip_stream);
    if (r) {
        f->broken = true;
        return r;
    }
    return ok();
}

pr_status pr_evict_lru(pr_forest *f, int64_t max_tokens, int64_t *evicted, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (!evicted) return fail(PR_EINVAL, "evicted is NULL");
    *evicted = 0;
    if (max_tokens < 0) return fail(PR_EINVAL, "max_tokens < 0");
    if (f->local < 0) return fail(PR_ESTATE, "no local peer is set");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    if (max_tokens == 0) return ok();
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    pr_status r = commit(f);
    if (r) return r;
    if (!f->dev.ltime && (r = init_local_times(f, f->local_load_time))) return r;
    hipStream_t s = (hipStream_t)hip_stream;
    ExportScratch &W = f->xs;
    if (f->d_stage) {
        // among few records one launch finds the tree and evicts; a tree of at
        // most pr::kEvictNodes nodes takes a walk and a launch; one wait each
        if ((r = ensure_export_scratch(f, f->dev.n_nodes))) return r;
        pr::EvictStatus *out = reinterpret_cast<pr::EvictStatus *>(f->d_stage + kEvictStage / 4);
        for (int scan = f->dev.n_nodes <= pr::kEvictScan; scan >= 0; scan--) {
            if (scan) {
                hipLaunchKernelGGL((pr::evict_kernel<true>), dim3(1), dim3(pr::kWalkThreads), 0, s, dev_view(f),
                                   f->d_walk, W.all, W.depth, W.parent, max_tokens, f->d_ctr, out);
            } else {
                pr::WalkOut O{};
                O.depth = W.depth;
                O.parent = W.parent;
                O.all = W.all;
                if (!enqueue_walk(f, f->local, O, s)) return fail(PR_EDEVICE, "tree walk launch failed");
                hipLaunchKernelGGL((pr::evict_kernel<false>), dim3(1), dim3(pr::kWalkThreads), 0, s, dev_view(f),
                                   f->d_walk, W.all, W.depth, W.parent, max_tokens, f->d_ctr, out);
            }
            if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) {
                f->broken = true;
                return fail(PR_EDEVICE, "eviction failed");
            }
            pr::EvictStatus st;
            std::memcpy(&st, static_cast<const char *>(f->h_stage) + kEvictStage, sizeof(st));
            if (st.done) {
                f->dev.n_nodes = (int64_t)st.n_nodes;
                if (st.evicted == 0) return ok();
                f->merged = true;
                f->sets[(size_t)f->local] = pr::PeerSeqs();  // the host copy no longer describes the local peer
                *evicted = (int64_t)st.evicted;
                return ok();
            }
        }
    }
    int32_t counts[3];
    if ((r = walk_peer(f, f->local, true, s, counts))) return r;
    const int64_t V = counts[2];
    if (V == 0) return ok();
    CallScratch X(f);
    unsigned long long *keys = nullptr, *keys_s = nullptr;
    int32_t *vals = nullptr, *vals_s = nullptr;
    int64_t *cnt1 = nullptr, *cum = nullptr;
    pr::EvictPlan *d_plan = nullptr;
    if (!X.get(&keys, V) || !X.get(&keys_s, V) || !X.get(&vals, V) || !X.get(&vals_s, V) || !X.get(&cnt1, V + 1) ||
        !X.get(&cum, V + 1) || !X.get(&d_plan, 1))
        return fail(PR_ENOMEM, "hipMalloc failed for the eviction");  // nothing changed yet
    auto fail_dev = [&](const char *m) {
        f->broken = true;
        return fail(PR_EDEVICE, m);
    };
    // once a launch has changed the forest, a failed allocation leaves it
    // partly evicted: the forest is then broken, as after a device failure
    bool mutated = false;
    auto fail_nomem = [&](const char *m) {
        if (mutated) f->broken = true;
        return fail(PR_ENOMEM, m);
    };
    const pr::DevForest F = dev_view(f);
    hipLaunchKernelGGL(pr::lru_keys_kernel, dim3(grid_threads(V, 256)), dim3(256), 0, s, F, W.all, V, keys, vals);
    size_t need = 0, need2 = 0;
    if (rocprim::radix_sort_pairs(nullptr, need, keys, keys_s, vals, vals_s, (size_t)V, 0, 64, s) != hipSuccess ||
        rocprim::inclusive_scan(nullptr, need2, cnt1, cum, (size_t)V + 1, rocprim::plus<int64_t>(), s) != hipSuccess)
        return fail_dev("eviction sort sizing failed");
    char *tmp = nullptr;
    const size_t tmp_bytes = std::max(need, need2);
    if (!X.get(&tmp, (int64_t)tmp_bytes)) return fail_nomem("hipMalloc failed for the eviction");
    size_t t1 = tmp_bytes;
    if (rocprim::radix_sort_pairs(tmp, t1, keys, keys_s, vals, vals_s, (size_t)V, 0, 64, s) != hipSuccess)
        return fail_dev("eviction sort failed");
    hipLaunchKernelGGL(pr::lru_counts_kernel, dim3(grid_threads(V, 256)), dim3(256), 0, s, F, vals_s, V, cnt1);
    size_t t2 = tmp_bytes;
    if (rocprim::inclusive_scan(tmp, t2, cnt1, cum, (size_t)V + 1, rocprim::plus<int64_t>(), s) != hipSuccess)
        return fail_dev("eviction scan failed");
    hipLaunchKernelGGL(pr::lru_plan_kernel, dim3(1), dim3(1), 0, s, keys_s, cum, V, max_tokens, d_plan);
    pr::EvictPlan plan;
    if (!read_small(f, &plan, d_plan, sizeof(plan), s))
        return fail_dev("eviction readback failed");
    const int64_t n_evict = std::min<int64_t>(max_tokens, plan.total);
    if (plan.a > 0) {
        hipLaunchKernelGGL(pr::lru_clear_sorted_kernel, dim3(grid_threads(plan.a, 256)), dim3(256), 0, s, F, vals_s,
                           plan.a);
        mutated = true;
    }
    if (plan.r > 0) {
        const int64_t a = plan.a, b = plan.b, nc = b - a;
        hipLaunchKernelGGL(pr::lru_maxdepth_kernel, dim3(grid_threads(nc, 256)), dim3(256), 0, s, vals_s, a, b,
                           W.depth, d_plan);
        if (!read_small(f, &plan, d_plan, sizeof(plan), s))
            return fail_dev("eviction readback failed");
        const int32_t maxd = plan.maxd;
        long long *hist = nullptr, *cnt = nullptr, *rev = nullptr, *S = nullptr;
        int32_t *level = nullptr, *n_level = nullptr, *rank_of = nullptr, *cut_node = nullptr, *n_cut = nullptr;
        int32_t *cut_len = nullptr;
        if (!X.get(&hist, maxd + 2) || !X.get(&cnt, maxd + 2) || !X.get(&rev, maxd) || !X.get(&S, maxd) ||
            !X.get(&level, nc) || !X.get(&n_level, 1) || !X.get(&rank_of, f->dev.n_nodes) ||
            !X.get(&cut_node, nc) || !X.get(&n_cut, 1) || !X.get(&cut_len, nc))
            return fail_nomem("hipMalloc failed for the eviction");
        if (hipMemsetAsync(hist, 0, (maxd + 2) * sizeof(long long), s) != hipSuccess ||
            hipMemsetAsync(n_level, 0, sizeof(int32_t), s) != hipSuccess ||
            hipMemsetAsync(n_cut, 0, sizeof(int32_t), s) != hipSuccess)
            return fail_dev("eviction memset failed");
        hipLaunchKernelGGL(pr::lru_hist_kernel, dim3(grid_threads(nc, 256)), dim3(256), 0, s, F, vals_s, a, b,
                           W.depth, hist);
        size_t n3 = 0, n4 = 0;
        if (rocprim::inclusive_scan(nullptr, n3, hist, cnt, (size_t)maxd + 2, rocprim::plus<long long>(), s) !=
                hipSuccess ||
            rocprim::inclusive_scan(nullptr, n4, rev, S, (size_t)maxd, rocprim::plus<long long>(), s) != hipSuccess)
            return fail_dev("eviction scan sizing failed");
        char *tmp2 = nullptr;
        const size_t tb2 = std::max(n3, n4);
        if (!X.get(&tmp2, (int64_t)tb2)) return fail_nomem("hipMalloc failed for the eviction");
        size_t u3 = tb2, u4 = tb2;
        if (rocprim::inclusive_scan(tmp2, u3, hist, cnt, (size_t)maxd + 2, rocprim::plus<long long>(), s) !=
            hipSuccess)
            return fail_dev("eviction scan failed");
        hipLaunchKernelGGL(pr::lru_reverse_kernel, dim3(grid_threads(maxd, 256)), dim3(256), 0, s, cnt, maxd, rev);
        if (rocprim::inclusive_scan(tmp2, u4, rev, S, (size_t)maxd, rocprim::plus<long long>(), s) != hipSuccess)
            return fail_dev("eviction scan failed");
        hipLaunchKernelGGL(pr::lru_depth_plan_kernel, dim3(1), dim3(1), 0, s, S, d_plan);
        hipLaunchKernelGGL(pr::lru_level_nodes_kernel, dim3(grid_threads(nc, 256)), dim3(256), 0, s, F, vals_s, a, b,
                           W.depth, d_plan, level, n_level);
        int32_t h_level = 0;
        if (!read_small(f, &h_level, n_level, sizeof(h_level), s))
            return fail_dev("eviction readback failed");
        if (h_level > nc) return fail_dev("eviction level list overflow");
        hipLaunchKernelGGL(pr::lru_rank_kernel, dim3(grid_threads(h_level, 4)), dim3(256), 0, s, F, level, h_level,
                           W.parent, W.depth, rank_of);
        hipLaunchKernelGGL(pr::lru_apply_kernel, dim3(grid_threads(nc, 256)), dim3(256), 0, s, F, vals_s, a, b,
                           W.depth, rank_of, d_plan, cut_node, cut_len, n_cut);
        int32_t h_cut = 0;
        if (hipGetLastError() != hipSuccess ||
            !read_small(f, &h_cut, n_cut, sizeof(h_cut), s))
            return fail_dev("eviction failed");
        if (h_cut > 0) {
            const int64_t base = f->dev.n_nodes;
            if ((r = ensure_capacity(f, base + h_cut, f->dev.n_pool, s))) {
                f->broken = true;
                return r;
            }
            hipLaunchKernelGGL(pr::lru_cut_kernel, dim3(grid_threads(h_cut, 256)), dim3(256), 0, s, dev_view(f),
                               cut_node, cut_len, h_cut, base, f->d_ctr);
            f->dev.n_nodes = base + h_cut;
        }
    }
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return fail_dev("eviction failed");
    f->merged = true;
    f->sets[(size_t)f->local] = pr::PeerSeqs();  // the host copy no longer describes the local peer
    *evicted = n_evict;
    return ok();
}

static pr_status route_impl(pr_forest *f, const int32_t *q_tokens, int64_t num_tokens, const int64_t *q_offsets,
                            int64_t num_queries, const pr::Select &sel, int32_t *match_len, int32_t *chosen,
                            void *hip_stream) {
    if (num_queries > (int64_t)0x7fffffff * pr::kRouteWavesPerBlock) return fail(PR_EINVAL, "too many queries");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    hipStream_t st = (hipStream_t)hip_stream;
    // Under graph capture only the launch may be enqueued: no upload of a
    // changed forest (allocations, copies, waits) and no longest-first order
    // (its buffer, events and cross-stream wait); the batch goes in index
    // order, with the same results.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) return fail(PR_EDEVICE, "hipStreamIsCapturing failed");
    const bool capturing = cap != hipStreamCaptureStatusNone;
    if (capturing && (f->dirty || !f->has_dev))
        return fail(PR_ESTATE, "snapshots changed since the forest's last upload; route once outside graph capture");
    pr_status s = commit(f);
    if (s) return s;
    const int32_t *order = nullptr;
    if (!capturing && use_longest_first(num_queries, num_tokens) &&
        (s = route_order(f, q_offsets, num_queries, num_tokens, st, &order)))
        return s;
    const pr::RouteBatch batch{q_tokens, num_tokens, q_offsets, num_queries, match_len, chosen, order};
    const hipError_t e = pr::launch_route(route_view(f), batch, sel, st);
    if (e != hipSuccess) return fail(PR_EDEVICE, std::string("route launch failed: ") + hipGetErrorString(e));
    if (order) {
        // the order buffers are in use until the stream passes this launch
        if (hipEventRecord(f->rs.done, st) != hipSuccess) return fail(PR_EDEVICE, "hipEventRecord failed");
        f->rs.pending = true;
    }
    return ok();
}

pr_status pr_route(pr_forest *f, const int32_t *q_tokens, int64_t num_tokens, const int64_t *q_offsets,
                   int64_t num_queries, int32_t *match_len, int32_t *chosen, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (num_queries < 0 || num_tokens < 0) return fail(PR_EINVAL, "negative count");
    if (num_queries == 0) return ok();
    if (!q_offsets || !match_len || !chosen) return fail(PR_EINVAL, "NULL device pointer");
    if (num_tokens > 0 && !q_tokens) return fail(PR_EINVAL, "q_tokens is NULL");
    const pr::Select sel{nullptr, -1, 0, nullptr};
    return route_impl(f, q_tokens, num_tokens, q_offsets, num_queries, sel, match_len, chosen, hip_stream);
}

pr_status pr_route_noalloc(pr_forest *f, const int32_t *q_tokens, int64_t num_tokens, const int64_t *q_offsets,
                           int64_t num_queries, int32_t *match_len, int32_t *chosen, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (num_queries < 0 || num_tokens < 0) return fail(PR_EINVAL, "negative count");
    if (num_queries > PR_NOALLOC_MAX_QUERIES)
        return fail(PR_EINVAL, "pr_route_noalloc takes at most " + std::to_string(PR_NOALLOC_MAX_QUERIES) +
                                   " queries per call");
    if (num_queries == 0) return ok();
    if (!q_offsets || !match_len || !chosen) return fail(PR_EINVAL, "NULL device pointer");
    if (num_tokens > 0 && !q_tokens) return fail(PR_EINVAL, "q_tokens is NULL");
    if (f->broken) return fail(PR_ESTATE, "an earlier device update failed; destroy the forest");
    if (f->dirty || !f->has_dev)
        return fail(PR_ESTATE, "snapshots changed since the forest's last upload; call pr_route once first");
    DeviceScope ds(f);
    if (!ds.ok()) return fail(PR_EDEVICE, "cannot select the forest's device");
    hipStream_t st = (hipStream_t)hip_stream;
    unsigned char *sp = nullptr;
    pr_status r = noalloc_scratch(f->device, &sp);
    if (r) return r;
    const int32_t *order = nullptr;
    if (use_longest_first(num_queries, num_tokens)) {
        int32_t *ord = reinterpret_cast<int32_t *>(sp + kNoAllocOrder);
        if (pr::launch_route_order(q_offsets, num_queries, num_tokens, st, sp + kNoAllocBkt,
                                   reinterpret_cast<int32_t *>(sp + kNoAllocBlockcnt), ord) != hipSuccess)
            return fail(PR_EDEVICE, "route order launch failed");
        order = ord;
    }
    const pr::Select sel{nullptr, -1, 0, nullptr};
    const pr::RouteBatch batch{q_tokens, num_tokens, q_offsets, num_queries, match_len, chosen, order};
    const hipError_t e = pr::launch_route(route_view(f), batch, sel, st);
    if (e != hipSuccess) return fail(PR_EDEVICE, std::string("route launch failed: ") + hipGetErrorString(e));
    return ok();
}

pr_status pr_route_select(pr_forest *f, const int32_t *q_tokens, int64_t num_tokens, const int64_t *q_offsets,
                          int64_t num_queries, const uint64_t *eligible, int32_t local_peer, uint32_t flags,
                          int32_t *match_len, int32_t *best, int32_t *second, void *hip_stream) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (num_queries < 0 || num_tokens < 0) return fail(PR_EINVAL, "negative count");
    if (local_peer < -1 || local_peer >= f->P) return fail(PR_EINVAL, "local_peer out of range");
    if (flags & ~(uint32_t)PR_SELECT_PREFER_LOCAL) return fail(PR_EINVAL, "unknown flags");
    if (num_queries == 0) return ok();
    if (!q_offsets || !best) return fail(PR_EINVAL, "NULL device pointer");
    if (num_tokens > 0 && !q_tokens) return fail(PR_EINVAL, "q_tokens is NULL");
    const pr::Select sel{eligible, local_peer, (flags & PR_SELECT_PREFER_LOCAL) ? 1 : 0, second};
    return route_impl(f, q_tokens, num_tokens, q_offsets, num_queries, sel, match_len, best, hip_stream);
}

pr_status pr_forest_check(pr_forest *f) {
    if (!f) return fail(PR_EINVAL, "forest is NULL");
    if (f->device < 0 || !f->d_skipped) return ok();
    DeviceScope ds(f);
    unsigned long long n = 0;
    if (hipDeviceSynchronize() != hipSuccess) return fail(PR_EDEVICE, "hipDeviceSynchronize failed");
    if (hipMemcpy(&n, f->d_skipped, sizeof(n), hipMemcpyDeviceToHost) != hipSuccess)
        return fail(PR_EDEVICE, "hipMemcpy failed");
    if (!n) return ok();
    if (hipMemset(f->d_skipped, 0, sizeof(n)) != hipSuccess) return fail(PR_EDEVICE, "hipMemset failed");
    return fail(PR_EINVAL, std::to_string(n) + " device inputs were skipped");
}

pr_status pr_forest_info_get(pr_forest *f, pr_forest_info *out) {
    if (!f || !out) return fail(PR_EINVAL, "NULL argument");
    std::memset(out, 0, sizeof(*out));
    out->num_peers = f->P;
    out->mask_words = f->W;
    if (f->has_dev && !f->dirty) {
        out->num_nodes = f->dev.n_nodes;
        out->pool_tokens = f->dev.n_pool;
    } else if (f->host_img_valid) {
        out->num_nodes = (int64_t)f->host_img.nodes.size();
        out->pool_tokens = (int64_t)f->host_img.pool.size();
    }
    out->device_bytes = f->device_bytes;
    out->layout_epoch = f->layout_epoch;
    out->label_token_bytes = f->narrow ? 2 : 4;
    out->label_bits = f->narrow ? (f->hi17 ? 17 : 16) : 32;
    out->merge_refusals = f->refusals;
    out->first_window_tokens = (int64_t)pr::kWave * (f->wide_window ? pr::kWideWinVectors : pr::kWinVectors);
    int64_t t = 0;
    for (const auto &S : f->sets) t += (int64_t)S.tokens.size();
    out->host_seq_tokens = t;
    return ok();
}

pr_status pr_forest_host_image(pr_forest *f, pr_image_view *out) {
    if (!f || !out) return fail(PR_EINVAL, "NULL argument");
    if (f->merged) return fail(PR_ESTATE, "the device forest holds merges; the host copies do not describe it");
    pr_status s = ensure_host_image(f);
    if (s) return s;
    const pr::HostImage &h = f->host_img;
    out->mask_words = h.W;
    out->num_nodes = (int64_t)h.nodes.size();
    out->pool_tokens = (int64_t)h.pool.size();
    out->nodes = reinterpret_cast<const int32_t *>(h.nodes.data());
    out->ntok = h.ntok.data();
    out->nsep = h.nsep.data();
    out->mext = h.mext.data();
    out->pool = h.pool.data();
    return ok();
}

}  // extern "C"
