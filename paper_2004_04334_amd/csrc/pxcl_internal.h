// Internal layout shared by the device kernels and the host runtime of the
// pixel-clustering library.  Not part of the C ABI (include/pxcl.h is).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#if defined(__HIPCC__)
#define PXCL_HD __host__ __device__
#else
#define PXCL_HD
#endif

// Address space of the device pointers below as the kernels see them (global memory in
// their device compilation, nothing elsewhere): a pointer that the kernels read from
// memory would otherwise be a generic one, and every access through it a flat
// instruction, whose completion each wait for LDS includes.
#ifndef PXCL_G
#define PXCL_G
#endif

namespace pxcl {

typedef uint8_t u8;
typedef uint16_t u16;
typedef uint32_t u32;
typedef uint64_t u64;

// Module geometry.  Linear pixel index inside a module is column-major,
// lin = col*ROWS + row, so a column is 5 consecutive 32-bit bitmap words and a
// word never straddles two columns.
constexpr u32 ROWS = 160, COLS = 416, PIX = ROWS * COLS;
constexpr u32 WORDS = PIX / 32;          // 2080 bitmap words per module
constexpr u32 WPC = ROWS / 32;           // 5 words per column
constexpr u32 MAX_RUNS = PIX / 2;        // vertical runs in a module (alternating pixels)
constexpr u32 MAXB = 128;                // events per batch

// Kernel shapes.
constexpr u32 A_WG = 256;                                   // segmentation: ids per thread,
constexpr u32 A_PER_N = 8, A_PER_W = 32;                    // narrow chunks for launches that
                                                            // cannot fill the device, wide ones
                                                            // (fewer end-of-chunk atomics) else
constexpr u32 C_WG = 256;                                   // compaction: a wave per module
constexpr u32 K_SMALL = 8;                                  // digis per thread (small-module kernel)
constexpr u32 B_WG = 1024, K_BIG = 16;                      // big-module kernel
constexpr u32 BIG_RCAP = B_WG * K_BIG;                      // 16384: larger modules use scratch mode
constexpr u32 S_WG = 1024;                                  // its scratch mode

// Per-event control words (u32) at the start of an event workspace.
enum : u32 {
    CTL_ERR = 0,      // accumulated PXCL_ERRBIT_* of the launch in progress
    CTL_NCL = 2,      // kept clusters
    CTL_BIG = 4,      // modules on the big-module list (register mode)
    CTL_SCR = 3,      // modules on the scratch-mode list
    CTL_PRESENT = 5,  // words 5-6: modules on the present-module list, one count per
                      // launch parity (EventDesc::slot); a launch clears the other one
    CTL_DEFERRED = 7, // 1: a batch launch with LF_DEFER left this event to its second
                      // launch (set by the compaction, cleared by segmentation or grouping)
    CTL_CTR = 8,      // launch counters when the event is launched on its own; in a batch the
                      // first is one of the small kernel's tickets (zero between launches)
    CTL_WORDS = 64
};
// Launch counters: the small-module kernel's ticket (when it needs only one) and the
// big-module kernel's.
enum : u32 { S_TICK = 0, S_BIG = 1, N_CTR = 8 };
// Host status block (pinned) written by the compaction kernel.
enum : u32 { HS_EPOCH = 0, HS_ERR = 1, HS_NCL = 2, HS_WORDS = 16 };
constexpr u32 HS_BYTES = HS_WORDS * 4;

// Error bits (same values as PXCL_ERRBIT_*).
constexpr u32 EB_RANGE = 1, EB_ORDER = 2, EB_DUP = 4, EB_INTERNAL = 8, EB_HINT = 16;
// Not an error: a launch with LF_DEFER found modules above the small kernel's
// capacity, listed them and left the compaction to a second launch (big-module
// kernels, then the compaction), which the host queues.
constexpr u32 EB_DEFER = 32;

// Launch flags.
constexpr u32 LF_NO_BIG = 1;     // the big-module kernel is not launched (size hint)
constexpr u32 LF_SEG_WIDE = 2;   // segmentation in wide chunks
constexpr u32 LF_FUSED = 4;      // one event, no segmentation kernel: the small kernel
                                 // finds every module's digis by search
constexpr u32 LF_NO_SCRATCH = 8; // no module above BIG_RCAP digis (size hint): one is an EB_HINT
constexpr u32 LF_GROUP = 16;     // some event is in any order: the grouping kernels run first
constexpr u32 LF_NO_SEG = 32;    // no event is grouped by module: no segmentation kernel
constexpr u32 LF_DEFER = 64;     // with LF_NO_BIG | LF_NO_SCRATCH: modules above the small
                                 // kernel's capacity are listed as usual, and an event with
                                 // any is not compacted but reported with EB_DEFER
constexpr u32 LF_SECOND = 128;   // the second launch of a deferred batch: the compaction
                                 // takes only the events the first one left (CTL_DEFERRED)
PXCL_HD constexpr u32 seg_chunk(u32 flags) { return A_WG * ((flags & LF_SEG_WIDE) ? A_PER_W : A_PER_N); }

// Event flags (EventDesc::flags).
constexpr u32 EF_UNSORTED = 1;   // the digis are in any order: the grouping kernels read them
                                 // from r_* and write a copy grouped by module to the workspace
                                 // (grp: one word per digi, its input position in it), which
                                 // the other kernels read instead of module..adc
constexpr u32 EF_HITS = 2;       // hits fused into the clustering: every kept digi adds
                                 // adc*col and adc*row to its cluster's staging sums (hsum),
                                 // the compaction writes x and y beside each record and
                                 // zeroes the sums it read: they are zero between launches
                                 // (binding clears them, and so does the host after a
                                 // launch that failed or reported an error)

// One event as the kernels see it (144 bytes).
struct EventDesc {
    const u16 PXCL_G* module;   // digis grouped by module
    const u16 PXCL_G* row;
    const u16 PXCL_G* col;
    const u16 PXCL_G* adc;
    const u16 PXCL_G* r_module; // with EF_UNSORTED: the digis as given (any order)
    const u16 PXCL_G* r_row;
    const u16 PXCL_G* r_col;
    const u16 PXCL_G* r_adc;
    u8 PXCL_G* ws;              // event workspace (device)
    u32 PXCL_G* hstat;          // status block (pinned host memory or device memory)
    int32_t PXCL_G* o_digi;     // per-digi cluster ids [n], in input order
    int32_t PXCL_G* o_id;       // kept clusters (ascending id); room for n entries each, used as
    int32_t PXCL_G* o_charge;   // per-cluster temporaries of the big-module kernel's scratch mode
    int32_t PXCL_G* o_size;
    u32 n;               // digis
    u32 cap;             // workspace capacity in digis
    u32 epoch;           // launch tag of the module-table words
    u32 slot;            // launch parity: which present-module count this launch uses
    u32 flags;           // EF_*
    u32 pad[3];
};
static_assert(sizeof(EventDesc) == 144, "EventDesc is 144 bytes");

// A module's digis [first, end), each word tagged with the launch (epoch << 32):
// written by the digis at the module's boundaries, so an entry whose tags are not
// the current launch's belongs to an absent module and needs no clearing.
struct ModRange {
    u64 first, end;
};

// Batch header in device memory: u32 k, padding to 64 bytes, then EventDesc[k].
constexpr u32 HDR_EV_OFFSET = 64;
PXCL_HD inline size_t header_bytes(u32 max_events) { return HDR_EV_OFFSET + size_t(max_events) * sizeof(EventDesc); }

struct LaunchArgs {
    const u32 PXCL_G* hdr;   // batch header (device) or nullptr: then `single` is the only event
    u32 PXCL_G* ctr;         // N_CTR launch counters (device)
    u32 n_modules;
    u32 charge_cut;
    u32 dcap;           // largest module (digis) the small-module kernel takes
    u32 flags;          // LF_*
    EventDesc single;
};

// Arrays copied between pinned host memory and the device by one kernel: 8-byte aligned at
// both ends, whole 8-byte words and then a tail of 16-bit values.
constexpr u32 MAX_COPIES = 6;
struct CopyArgs {
    const u64 PXCL_G* src[MAX_COPIES];
    u64 PXCL_G* dst[MAX_COPIES];
    u32 first[MAX_COPIES + 1];   // words of the arrays before each one; the last: of all
    u32 tail[MAX_COPIES];        // 16-bit values after an array's words (at most 3)
    u32 n;
};

// What the runtime says of a host address: memory it allocated (pinned), coherent unless
// asked for otherwise, and where the device finds the address and the allocation around it.
struct HostMemory {
    bool pinned, coherent;
    u64 dev, base, size;
};
// The copy kernel may move `bytes` from or to `host`: 8-byte aligned, and every byte in one
// allocation that the device can address (the ends alone do not tell: two pinned blocks with
// anything between them have both).  Coherent, since the kernel's accesses make nothing else
// visible: the device may hold non-coherent memory in its caches across kernels, so the host's
// new values could be missed, and the results could reach the host after the callback.
inline bool copy_kernel_takes(u64 host, size_t bytes, const HostMemory& m) {
    return m.pinned && m.coherent && (host & 7u) == 0 && (m.dev & 7u) == 0 && m.dev >= m.base &&
           m.dev - m.base <= m.size && bytes <= m.size - (m.dev - m.base);
}

// Which of a server's batches defer the big-module kernel, when it may: all of them, until
// DEFER_LATE in a row needed their second launch; then one in DEFER_RETRY tries again, and the
// others launch everything at once.  A second launch is queued only when the completion thread
// has seen the first one end, and whether most batches need it depends on the small kernel's
// capacity at the shape in use.  10,000 requests of 10k-200k digis at 100 / 180 / 250 k/s, nearly
// all with a module above 2,048 digis, p50: at 256x1 (capacity 2,048) 185 / 238 / 350 us with
// every batch deferred, 137 / 190 / 290 with none; at 512x1 (4,096: none needs a second launch)
// 93 / 160 / 480 deferred, 113 / 250 / 1,400 not.
constexpr u32 DEFER_LATE = 3, DEFER_RETRY = 256;
struct DeferChoice {
    std::atomic<u32> late{0};   // deferred batches in a row that needed their second launch
    u32 whole = 0;              // batches since the last deferred one
    bool next() {               // of one thread
        if (late.load(std::memory_order_relaxed) < DEFER_LATE) return true;
        if (++whole < DEFER_RETRY) return false;
        whole = 0;
        return true;
    }
    void done(bool second) {    // of a deferred batch; of one thread
        const u32 n = late.load(std::memory_order_relaxed);
        late.store(second ? (n < DEFER_LATE ? n + 1 : n) : 0u, std::memory_order_relaxed);
    }
};

PXCL_HD constexpr size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

// Byte offsets of the arrays of an event workspace with capacity N digis and M
// modules per event.
struct EvLayout {
    size_t ctl, in_mod, in_row, in_col, in_adc;
    size_t digi, id, charge, size;           // outputs
    size_t tid, tcharge, tsize;              // cluster records before compaction
    size_t mtab;                             // per module: ModRange
    size_t kept;                             // per module: kept clusters
    size_t big;                              // module ids for the big-module kernel
    size_t scr;                              // module ids for the big-module kernel's scratch mode
    size_t present;                          // module ids of the modules present (any order)
    size_t off;                              // per module: its first cluster in the outputs
    size_t hit_x, hit_y;                     // hits (per kept cluster), when asked for
    size_t grp;                              // digis in any order: the grouped copy (u64[N])
    size_t gcnt;                             // digis in any order: per module, digis counted (zero between launches)
    size_t hsum;                             // fused hits: per staged record, sum(adc*col), sum(adc*row) (u64)
    size_t total;
};

// Every array starts at a multiple of 256 bytes, so the offsets are sums of a few rounded
// sizes (the kernels compute some of them for every module).
PXCL_HD constexpr EvLayout ev_layout(u32 N, u32 M) {
    EvLayout L{};
    const size_t n2 = al256(2 * size_t(N)), n4 = al256(4 * size_t(N)), n8 = al256(8 * size_t(N));
    const size_t m4 = al256(4 * size_t(M)), m16 = al256(16 * size_t(M));
    L.ctl = 0;
    const size_t in = al256(CTL_WORDS * 4);
    L.in_mod = in;
    L.in_row = in + n2;
    L.in_col = in + 2 * n2;
    L.in_adc = in + 3 * n2;
    const size_t out = in + 4 * n2;
    L.digi = out;
    L.id = out + n4;
    L.charge = out + 2 * n4;
    L.size = out + 3 * n4;
    L.tid = out + 4 * n4;
    L.tcharge = out + 5 * n4;
    L.tsize = out + 6 * n4;
    L.mtab = out + 7 * n4;
    const size_t mod = L.mtab + m16;
    L.kept = mod;
    L.big = mod + m4;
    L.scr = mod + 2 * m4;
    L.present = mod + 3 * m4;
    L.off = mod + 4 * m4;
    const size_t opt = mod + 5 * m4;
    L.hit_x = opt;
    L.hit_y = opt + n4;
    L.grp = opt + 2 * n4;
    L.gcnt = opt + 2 * n4 + n8;
    L.hsum = opt + 2 * n4 + n8 + m4;
    L.total = L.hsum + al256(16 * size_t(N));
    return L;
}

// Batch workspace: counters then the header.
constexpr size_t BW_CTR = 0;
constexpr size_t BW_HDR = 256;
PXCL_HD inline size_t batch_ws_bytes(u32 max_events) { return al256(BW_HDR + header_bytes(max_events)); }

}  // namespace pxcl
