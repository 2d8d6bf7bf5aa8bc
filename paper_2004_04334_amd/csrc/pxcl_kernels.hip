// Device kernels of the pixel-clustering path (gfx950 / CDNA4, wave64).
//
// One launch processes k >= 1 events through these kernels, in this order:
//
//   segment  (batches) streams the module ids; every digi at a module boundary
//            writes the module's entry of a per-module table (first digi, one past
//            the last, tagged with the launch), module starts go to a list of the
//            modules present; checks module range and order.  A single-event
//            launch has no segmentation kernel: the small kernel finds each
//            module's digis by search and checks the ids itself.
//   small    one module per group of threads (a single wave, or a whole
//            workgroup): fired-pixel bitmap in LDS, vertical runs, union-find over
//            runs, charge/size per cluster, charge cut; the module's kept clusters
//            go in ascending id to a staging area at the module's first digi, and
//            every digi gets its cluster id.  Modules above the group's capacity go
//            to the big-module or the scratch-mode list.  Groups take modules by
//            static rounds, then an atomic ticket, and prefetch the next module
//            while working on the current one.
//   big      one listed module per 1,024-thread workgroup: up to 16,384 digis in
//            register mode (digis held in registers), above that in scratch mode (the
//            digis re-read from memory in three passes).
//   compact  a wave per module: the offset of its clusters (the kept counts of the
//            modules before it) and a copy of its staged records to their final
//            position; a wave per event writes the status back to the host.
//
// On demand, after a launch: hits, the charge-weighted centroid of every kept
// cluster.
//
// The clustering: 8-connected components of fired pixels within a module; cluster
// id = smallest linear index module*66560 + col*160 + row; charge = sum of ADC
// (uint32); keep iff charge >= cut.  This is the "ClusterProducer" step of the
// paper's Figure 1 (Sec. 3).  Errors go to a device error word, never to device
// asserts, which would synchronise (Sec. 4.1).
//
// Memory ordering.  Workgroup barriers here order LDS only (global loads and stores
// stay in flight across them).  No workgroup reads what another workgroup of the same
// kernel writes: data crosses kernel boundaries, and the only device-scope atomics
// are counters whose returned values serve as indexes (tickets, list places).  No
// device-scope release/acquire fence is used: on gfx950 those write back and
// invalidate the L2.
#include <hip/hip_runtime.h>

#if defined(__AMDGCN__)
#define PXCL_G __attribute__((address_space(1)))
#define PXCL_C __attribute__((address_space(4)))   // constant: read-only while the kernel runs
// As flat accesses (163 of them in the 256x1 small kernel) instead of global ones the
// kernels took 1-4 % longer: one 320k-digi x 16 launch 421 us, now 414 us.
#else
#define PXCL_C
#endif
#include "pxcl_internal.h"

namespace pxcl {

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ u32 ld_wg(const u32* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void st_wg(u32* p, u32 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ u32 ld_ag(const u32* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_ag(u32* p, u32 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_sys(u32* p, u32 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Wait until every memory operation this thread issued has completed.
__device__ __forceinline__ void wait_all_mem() { __builtin_amdgcn_s_waitcnt(0); }

// Barrier over a group of G threads that orders LDS accesses only.  A group of 64
// is one wave: LDS requests of a wave are served in order, so only the compiler
// must be kept from moving accesses across the point.
template <u32 G>
__device__ __forceinline__ void gsync() {
    if constexpr (G == 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
}
__device__ __forceinline__ void lds_barrier() { gsync<128>(); }

__device__ __forceinline__ u32 num_events(const LaunchArgs& a) { return a.hdr ? a.hdr[0] : 1u; }
// Event e of the launch, in the header or in the kernel's own argument.  Neither is written
// while a kernel runs, so both are constant memory: with e the same for a whole wave the
// fields come by scalar loads, where they are needed.
__device__ __forceinline__ const EventDesc* event_at(const LaunchArgs& a, u32 e) {
#if defined(__AMDGCN__)
    const u8 PXCL_C* single = (const u8 PXCL_C*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(LaunchArgs, single);
#else
    const u8* single = reinterpret_cast<const u8*>(&a.single);
#endif
    const u8 PXCL_C* d = (const u8 PXCL_C*)(reinterpret_cast<uintptr_t>(a.hdr) + HDR_EV_OFFSET + sizeof(EventDesc) * e);
    return (const EventDesc*)(const EventDesc PXCL_C*)(a.hdr ? d : single);
}
__device__ __forceinline__ EventDesc get_event(const LaunchArgs& a, u32 e) { return *event_at(a, e); }
__device__ __forceinline__ u32* ticket(const LaunchArgs& a) { return (u32*)(a.ctr + S_TICK); }
__device__ __forceinline__ void reset_tickets(const LaunchArgs& a) {
    st_ag(ticket(a), 0u);
    st_ag((u32*)(a.ctr + S_BIG), 0u);
}
template <typename T>
__device__ __forceinline__ T* ws_ptr(const EventDesc& E, size_t off) {
    return (T*)(T PXCL_G*)(E.ws + off);         // generic again, but known to be global
}
// The digis of a module.  Given grouped by module they are the input's arrays; of an event in
// any order each is one word of the workspace's grouped copy: adc in bits 0-15, row in 16-23,
// column in 24-32 (255 and 511 for a pixel outside the module) and the input position, where
// its per-digi output goes, above.
__device__ __forceinline__ u64 pack_digi(u32 row, u32 col, u32 adc, u32 pos) {
    const u32 rc = row < ROWS && col < COLS ? row | (col << 8) : 0x1FFFFu;
    return u64(adc) | (u64(rc) << 16) | (u64(pos) << 33);
}
struct ModuleDigis {
    const u16 *row, *col, *adc;
    const u64* rec;              // nullptr: the arrays
    u32 st;
    static __device__ __forceinline__ u32 rc_of(u64 v) { return (u32(v >> 16) & 0xFFu) | ((u32(v >> 24) & 0x1FFu) << 16); }
    static __device__ __forceinline__ u32 pos_of(u64 v) { return u32(v >> 33); }
    // row | column << 16, adc and output position of the module's j-th digi
    __device__ __forceinline__ u32 rc(u32 j) const { return rec ? rc_of(rec[j]) : u32(row[j]) | (u32(col[j]) << 16); }
    __device__ __forceinline__ u32 adc_at(u32 j) const { return rec ? u32(rec[j]) & 0xFFFFu : u32(adc[j]); }
    __device__ __forceinline__ u32 pos(u32 j) const { return rec ? pos_of(rec[j]) : st + j; }
};
__device__ __forceinline__ ModuleDigis module_digis(const EventDesc& E, const EvLayout& L, u32 st) {
    ModuleDigis D;
    D.row = (const u16*)E.row + st;
    D.col = (const u16*)E.col + st;
    D.adc = (const u16*)E.adc + st;
    D.rec = (E.flags & EF_UNSORTED) ? ws_ptr<const u64>(E, L.grp) + st : nullptr;
    D.st = st;
    return D;
}

// Inclusive scan across the 64 lanes of a wave.
__device__ __forceinline__ u32 wave_incl_scan(u32 v) {
#if defined(__AMDGCN__)
    // six adds with their operand moved between lanes (data-parallel primitives), where
    // shuffles through the LDS take six round trips
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15, :31
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
#else
    const u32 lane = threadIdx.x & 63u;
#pragma unroll
    for (u32 d = 1; d < 64; d <<= 1) {
        const u32 y = __shfl_up(v, d, 64);
        if (lane >= d) v += y;
    }
    return v;
#endif
}

// Exclusive scan over a group of G threads (whole waves).  With G > 64 every thread
// of the workgroup must call it (it holds two LDS barriers); `wsum` has G/64 words
// private to the group.
template <u32 G>
__device__ __forceinline__ u32 group_excl_scan(u32 v, u32 lt, u32* wsum, u32& total) {
    const u32 inc = wave_incl_scan(v);
    if constexpr (G == 64) {
        total = __shfl(inc, 63, 64);
        return inc - v;
    } else {
        const u32 w = lt >> 6;
        if ((lt & 63u) == 63u) wsum[w] = inc;
        gsync<G>();
        u32 off = 0, tot = 0;
#pragma unroll
        for (u32 i = 0; i < G / 64; ++i) {
            const u32 s = wsum[i];
            off += (i < w) ? s : 0u;
            tot += s;
        }
        gsync<G>();
        total = tot;
        return off + inc - v;
    }
}

// The value of lane 0 in every lane (for values the whole wave holds alike: the
// compiler then keeps them in scalar registers and branches on them uniformly).
__device__ __forceinline__ u32 wave_uniform(u32 v) { return __builtin_amdgcn_readfirstlane(v); }

// Largest i in [0, k) with pref[i] <= t, given pref[0] <= t < pref[k], t the same for the
// whole wave: two ballots (k <= MAXB = 128) instead of a chain of LDS reads, and the event
// behind it then comes by scalar loads.  All lanes of the wave call it.
__device__ __forceinline__ u32 find_slot(const u32* pref, u32 k, u32 t) {
    const u32 lane = threadIdx.x & 63u;
    const bool in0 = lane < k && pref[lane] <= t, in1 = lane + 64 < k && pref[lane + 64] <= t;
    return wave_uniform(u32(__popcll(__ballot(in0 ? 1 : 0)) + __popcll(__ballot(in1 ? 1 : 0))) - 1u);
}

// What event_prefix counts per event: its work units, the digis of an event grouped by
// module (CNT_SORTED: zero for digis in any order) or in any order (CNT_ANY: zero for grouped
// ones).
constexpr u32 CNT_UNITS = 0xFFFFFFFEu, CNT_SORTED = 0xFFFFFFFDu, CNT_ANY = 0xFFFFFFFCu;

// Modules on the event's present-module list.
__device__ __forceinline__ u32 present_count(const LaunchArgs& a, const EventDesc& E) {
    return min(ld_ag(ws_ptr<const u32>(E, ev_layout(E.cap, a.n_modules).ctl) + CTL_PRESENT + (E.slot & 1u)), a.n_modules);
}

// Work units of the kernels after segmentation: when most modules are present, every
// module (unit j is module j; an absent one is recognised by its table entry), else
// the present-module list (unit j is its entry j, one more load away).
__device__ __forceinline__ bool dense_units(const LaunchArgs& a, u32 present) { return 2 * present > a.n_modules; }
__device__ __forceinline__ u32 unit_count(const LaunchArgs& a, const EventDesc& E) {
    if (!E.n) return 0u;
    const u32 p = present_count(a, E);
    return dense_units(a, p) ? a.n_modules : p;
}
__device__ __forceinline__ u32 unit_module(const LaunchArgs& a, const EventDesc& E, const EvLayout& L, u32 units,
                                           u32 j) {
    if (units == a.n_modules) return j;         // dense (a list as long as the module count is all of them)
    return min(ws_ptr<const u32>(E, L.present)[j], a.n_modules - 1);
}

// Prefix over the events of a launch of max(ceil(count / div), at_least) + plus,
// where count is one of the above or one of its control words (CTL_*, at most the modules
// per event); 0 for an empty event.  pref[k] = total.
// Every thread of the workgroup calls it; any k <= MAXB with any BS.
template <u32 BS>
__device__ __forceinline__ u32 event_prefix(const LaunchArgs& a, u32 k, u32* pref, u32* wsum, u32 which, u32 div,
                                            u32 at_least, u32 plus = 0) {
    u32 carry = 0;
    for (u32 base = 0; base < k; base += BS) {
        const u32 e = base + threadIdx.x;
        u32 v = 0;
        if (e < k) {
            const EventDesc E = get_event(a, e);
            u32 cnt = 0;
            if (E.n)
                cnt = which == CNT_SORTED  ? ((E.flags & EF_UNSORTED) ? 0u : E.n)
                      : which == CNT_ANY   ? ((E.flags & EF_UNSORTED) ? E.n : 0u)
                      : which == CNT_UNITS ? unit_count(a, E)
                                           : min(ld_ag(ws_ptr<u32>(E, ev_layout(E.cap, a.n_modules).ctl) + which), a.n_modules);
            v = max((cnt + div - 1) / div, at_least) + plus;
        }
        u32 tot;
        const u32 ex = group_excl_scan<BS>(v, threadIdx.x, wsum, tot);
        if (e < k) pref[e] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) pref[k] = carry;
    lds_barrier();
    return pref[k];
}

constexpr u32 NOPIX = 0xFFFFFFFFu;          // no pixel / no index

// ---------------------------------------------------------------------------
// bitmap helpers (column-major: 5 words per column; bit b of word w is row
// (w % 5)*32 + b of column w / 5)
// ---------------------------------------------------------------------------
// Union-find over runs in LDS: parent[x] <= x always; union hooks the larger root
// under the smaller with atomicMin; find halves paths with plain stores, which only
// ever point a node to one of its ancestors.  Both loops strictly decrease their
// index, so they terminate; the caps are a second guard.
__device__ __forceinline__ u32 uf_find(u32* par, u32 x) {
    for (u32 it = 0; it < 2 * MAX_RUNS; ++it) {
        const u32 p = ld_wg(&par[x]);
        if (p == x) return x;
        const u32 g = ld_wg(&par[p]);
        if (g == p) return p;
        st_wg(&par[x], g);
        x = g;
    }
    return x;
}

__device__ __forceinline__ void uf_unite(u32* par, u32 a, u32 b) {
    for (u32 it = 0; it < 2 * MAX_RUNS; ++it) {
        a = uf_find(par, a);
        b = uf_find(par, b);
        if (a == b) return;
        if (a < b) { const u32 t = a; a = b; b = t; }
        const u32 old = __hip_atomic_fetch_min(&par[a], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (old == a) return;
        a = old;
    }
}

// The same over the packed words of the register mode (RegModuleSmem::acc): the parent
// of run x is the top 16 bits of word x, the rest is zero while runs are united.
__device__ __forceinline__ u32* hi_word(u64* acc, u32 x) { return reinterpret_cast<u32*>(acc) + 2 * x + 1; }
__device__ __forceinline__ u32 parent_of(u64* acc, u32 x) { return ld_wg(hi_word(acc, x)) >> 16; }
__device__ __forceinline__ u32 find_packed(u64* acc, u32 x) {
    for (u32 it = 0; it < 2 * MAX_RUNS; ++it) {
        const u32 p = parent_of(acc, x);
        if (p == x) return x;
        const u32 g = parent_of(acc, p);
        if (g == p) return p;
        st_wg(hi_word(acc, x), g << 16);
        x = g;
    }
    return x;
}
__device__ __forceinline__ void unite_packed(u64* acc, u32 a, u32 b) {
    for (u32 it = 0; it < 2 * MAX_RUNS; ++it) {
        a = find_packed(acc, a);
        b = find_packed(acc, b);
        if (a == b) return;
        if (a < b) { const u32 t = a; a = b; b = t; }
        const u32 old = __hip_atomic_fetch_min(hi_word(acc, a), b << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >> 16;
        if (old == a) return;
        a = old;
    }
}

// Run index of row bit j of word w (fired), given the word's run starts s and the run
// starts before it r0: runs are numbered in column-major order of their first pixel.
__device__ __forceinline__ u32 run_at(u32 r0, u32 s, u32 j) { return r0 + __popc(s & ((2u << j) - 1u)) - 1u; }

// Which runs of neighbouring columns are united.  Rule B: every run start of column c+1
// is linked to the run of column c that holds the first fired pixel of the start's rows
// -1..+1.  Rule A: every run start q of column c is linked to the run of column c+1
// holding the first fired pixel of rows q-1..q+1, when rule B does not already make that
// link, which is when that pixel is at row q-1 and row q-2 is fired in either column.
// Every pair of touching runs X (column c+1), Y (column c) is linked this way: if X's
// start lies within Y's rows widened by one, rule B links X to Y, or to a run of column c
// ending right above X's start, and then Y starts just below X's start, within one row of
// it, and rule A links Y to X; otherwise Y starts inside X's rows widened by one, and
// rule A (or rule B for X, when X starts one row below Y's start) links them.  Runs are
// numbered in column-major order of their first pixel, so rule B links a run to a smaller
// one, and each run has at most one such link.

// The bitmap lies between words that stay zero, so that the columns on either side of
// the first and the last one read as not fired.
constexpr u32 BM_FRONT = WPC, BM_WORDS = BM_FRONT + WORDS + WPC + 3;

// Run numbers of a column: its first run in the low 16 bits, then one byte per bitmap
// word: the runs that start in the column before the word, less one when bit 0 of the
// word continues a run of the word above.  The run of row r (fired, in word k with bits b)
// is then first + byte k + the number of bits of b & ~(b << 1) up to r, less one: a lookup
// needs the entry and the one bitmap word.
__device__ __forceinline__ u32 runs_before(u64 e, u32 k) { return u32(e & 0xFFFFu) + (u32(e >> (16 + 8 * k)) & 255u); }
__device__ __forceinline__ u32 run_number(u64 e, u32 k, u32 word, u32 row) {
    return runs_before(e, k) + __popc(word & ~(word << 1) & ((2u << (row & 31u)) - 1u)) - 1u;
}

// Entry of column c but for its first run, and its number of runs.
__device__ __forceinline__ u64 col_entry(const u32* bm, u32 c, u32& n_runs) {
    u64 e = 0ull;
    u32 above = 0, runs = 0;
#pragma unroll
    for (u32 k = 0; k < WPC; ++k) {
        const u32 b = bm[BM_FRONT + c * WPC + k], cont = b & above;
        e |= u64(runs - cont) << (16 + 8 * k);
        runs += __popc(b & ~(b << 1)) - cont;
        above = b >> 31;
    }
    n_runs = runs;
    return e;
}

// Rows 32k..32k+31 of a column: bits, the rows above (row 32k-1 in bit 31) and below (row
// 32k+32 in bit 0), run starts, and the runs before the word.
struct ColWord {
    u32 b, above, below, st, r0;
};
__device__ __forceinline__ ColWord col_word(const u32* bm, const u64* col, u32 c, u32 k) {   // col[c + 1]: column c's entry
    const u32* w = &bm[BM_FRONT + c * WPC + k];
    ColWord x;
    x.b = w[0];
    x.above = k ? *(w - 1) : 0u;
    x.below = k + 1 < WPC ? w[1] : 0u;
    x.st = x.b & ~((x.b << 1) | (x.above >> 31));
    x.r0 = runs_before(col[c + 1], k) + (x.b & (x.above >> 31));
    return x;
}

// first(run, parent) for every run that starts in word k of column c: rule B's run, or the
// run itself.
template <typename F>
__device__ __forceinline__ void word_parents(const u32* bm, const u64* col, u32 c, u32 k, F first) {
    const ColWord x = col_word(bm, col, c, k);
    if (!x.st) return;
    u32 run = x.r0, m = x.st;
    ColWord l{};
    if (c) l = col_word(bm, col, c - 1, k);
    const u32 up = (l.b << 1) | (l.above >> 31), dn = (l.b >> 1) | (l.below << 31), touch = up | l.b | dn;
    const u32 next = c ? runs_before(col[c], k + 1 < WPC ? k + 1 : k) : 0u;   // the run of row 32k+32 (if it starts there)
    while (m) {
        const u32 i = __builtin_ctz(m);
        m &= m - 1u;
        u32 parent = run;
        if ((touch >> i) & 1u) {
            if ((up >> i) & 1u) parent = i ? run_at(l.r0, l.st, i - 1) : l.r0 - 1u;
            else if ((l.b >> i) & 1u) parent = run_at(l.r0, l.st, i);
            else parent = i < 31 ? run_at(l.r0, l.st, i + 1) : next;
        }
        first(run, parent);
        ++run;
    }
}

// link(run, run of column c + 1) for every rule A link of the runs that start in word k
// of column c.
template <typename F>
__device__ __forceinline__ void word_links(const u32* bm, const u64* col, u32 c, u32 k, F link) {
    if (c + 1 >= COLS) return;
    const u32* w = &bm[BM_FRONT + c * WPC + k];
    const u32 a = w[0], b = w[WPC];
    if (!a) return;
    const u32 pa = k ? *(w - 1) : 0u, pb = k ? w[WPC - 1] : 0u;      // rows 32k-32..32k-1
    const u32 sa = a & ~((a << 1) | (pa >> 31));
    u32 m = sa & ((b << 1) | (pb >> 31)) & (((a << 2) | (pa >> 30)) | ((b << 2) | (pb >> 30)));
    if (!m) return;
    const u32 ra0 = runs_before(col[c + 1], k) + (a & (pa >> 31)), rb0 = runs_before(col[c + 2], k) + (b & (pb >> 31));
    const u32 sb = b & ~((b << 1) | (pb >> 31));
    while (m) {
        const u32 i = __builtin_ctz(m);
        m &= m - 1u;
        link(run_at(ra0, sa, i), i ? run_at(rb0, sb, i - 1) : rb0 - 1u);
    }
}

// ---------------------------------------------------------------------------
// group (digis in any order): a counting sort by module ahead of the clustering,
// which then reads a grouped copy in the event workspace and writes every per-digi
// output at the digi's input position.  Three steps:
//   count    per chunk of G_CH digis an LDS histogram over the modules gives each
//            digi its rank among the chunk's digis of its module; one device atomic
//            per (chunk, module present in it) adds the chunk's count to the module's
//            total and returns the chunk's base, so a digi's rank in its module is
//            base + local rank.  The rank is parked in the per-digi output word (the
//            clustering overwrites it).  Module ids at or above the module count set
//            EB_RANGE and the digi takes no part.
//   table    an exclusive scan of the module totals gives each module its first grouped
//            position; module-table entries tagged with the launch, the present-module
//            list in ascending module order, kept counts cleared -- the segmentation
//            kernel's outputs.  Part of the scatter kernel, or a kernel of its own for
//            more than G_HMAX modules; the compaction clears the totals.
//   scatter  every digi goes to first[module] + rank of the grouped copy.  What bounds it is
//            the number of scattered stores (a wave's 64 digis go to dozens of modules), so a
//            digi is one word: 16 events of 64,000 digis 31.7 -> 15.5 us (row, column, adc,
//            module and input position stored one by one before).
// A digi's place within its module is not fixed (chunks take their bases in any
// order); the clustering does not depend on it.
// ---------------------------------------------------------------------------
constexpr u32 G_WG = 256, G_PER = 16, G_CH = G_WG * G_PER, G_HMAX = 4096, G_TPM = 8;
constexpr u32 G_SPER = 4, G_SCH = G_WG * G_SPER;   // scatter: smaller chunks, more workgroups

__global__ __launch_bounds__(G_WG) void k_group_count(LaunchArgs a) {
    __shared__ u32 hist[G_HMAX];
    __shared__ u32 s_pref[MAXB + 1];
    __shared__ u32 s_wsum[G_WG / 64];
    __shared__ u32 s_err;
    const u32 tid = threadIdx.x, k = num_events(a), M = a.n_modules;
    const bool lds = M <= G_HMAX;                 // else ranks straight from the totals
    const u32 total = event_prefix<G_WG>(a, k, s_pref, s_wsum, CNT_ANY, G_CH, 0);
    // the tickets start at zero (segmentation, which also resets them, is not launched
    // when every event of the launch is in any order)
    if (blockIdx.x == 0 && tid == 0) reset_tickets(a);
    for (u32 t = blockIdx.x; t < total; t += gridDim.x) {
        const u32 e = find_slot(s_pref, k, t), c = t - s_pref[e];
        const EventDesc E = get_event(a, e);
        const EvLayout L = ev_layout(E.cap, M);
        u32* gcnt = ws_ptr<u32>(E, L.gcnt);
        u32* rank = (u32*)E.o_digi;
        if (tid == 0) s_err = 0;
        if (lds)
            for (u32 m = tid; m < M; m += G_WG) hist[m] = 0u;
        lds_barrier();
        const u32 i0 = c * G_CH + tid;
        u32 mm[G_PER], lr[G_PER];
#pragma unroll
        for (u32 q = 0; q < G_PER; ++q) {
            const u32 i = i0 + q * G_WG;
            mm[q] = i < E.n ? u32(E.r_module[i]) : NOPIX;
        }
        u32 err = 0;
#pragma unroll
        for (u32 q = 0; q < G_PER; ++q) {
            lr[q] = 0u;
            if (mm[q] == NOPIX) continue;
            if (mm[q] >= M) {
                err |= EB_RANGE;
                mm[q] = NOPIX;
            } else {
                lr[q] = lds ? atomicAdd(&hist[mm[q]], 1u) : atomicAdd(&gcnt[mm[q]], 1u);
            }
        }
        lds_barrier();
        if (lds) {                                // the chunk's bases: independent atomics, all in flight
            constexpr u32 FL = G_HMAX / G_WG;
            u32 h[FL];
#pragma unroll
            for (u32 j = 0; j < FL; ++j) {
                const u32 m = tid + j * G_WG;
                h[j] = m < M ? hist[m] : 0u;
            }
#pragma unroll
            for (u32 j = 0; j < FL; ++j)
                if (h[j]) h[j] = atomicAdd(&gcnt[tid + j * G_WG], h[j]);
#pragma unroll
            for (u32 j = 0; j < FL; ++j)
                if (tid + j * G_WG < M) hist[tid + j * G_WG] = h[j];
        }
        lds_barrier();
#pragma unroll
        for (u32 q = 0; q < G_PER; ++q)
            if (mm[q] != NOPIX) rank[i0 + q * G_WG] = (lds ? hist[mm[q]] : 0u) + lr[q];
        if (err) atomicOr(&s_err, err);
        lds_barrier();
        if (tid == 0 && s_err) atomicOr(ws_ptr<u32>(E, L.ctl) + CTL_ERR, s_err);
        lds_barrier();                            // hist and s_err are reused by the next chunk
    }
}

// First grouped position of every module of event E: a scan of the module totals, by one
// workgroup.  The positions go to `first` (if given, in LDS); with `write` the segmentation
// kernel's outputs go to the event's workspace.
__device__ __forceinline__ void group_table(const EventDesc& E, const EvLayout& L, u32 M, u32* first, bool write, u32* wsum) {
    const u32 tid = threadIdx.x;
    const u32* gcnt = ws_ptr<const u32>(E, L.gcnt);
    u32* kept = ws_ptr<u32>(E, L.kept);
    u32* present = ws_ptr<u32>(E, L.present);
    u32* ctl = ws_ptr<u32>(E, L.ctl);
    ModRange* mt = ws_ptr<ModRange>(E, L.mtab);
    const u64 tag = u64(E.epoch) << 32;
    u32 carry = 0, pcarry = 0;
    for (u32 base = 0; base < M; base += G_WG * G_TPM) {
        const u32 m0 = base + tid * G_TPM;       // this thread's G_TPM consecutive modules
        u32 cnt[G_TPM], sum = 0, pres = 0;
#pragma unroll
        for (u32 j = 0; j < G_TPM; ++j) {
            cnt[j] = (m0 + j < M && E.n) ? gcnt[m0 + j] : 0u;
            sum += cnt[j];
            pres += cnt[j] ? 1u : 0u;
        }
        u32 tot, ptot = 0, pex = 0;
        const u32 ex = group_excl_scan<G_WG>(sum, tid, wsum, tot);
        if (write) pex = group_excl_scan<G_WG>(pres, tid, wsum, ptot);
        u32 pos = carry + ex, pp = pcarry + pex;
#pragma unroll
        for (u32 j = 0; j < G_TPM; ++j) {
            const u32 m = m0 + j;
            if (m >= M) break;
            if (first) first[m] = pos;
            if (write) {
                if (cnt[j]) {
                    const u32 end = pos + cnt[j];
                    if (end <= E.n) mt[m] = ModRange{tag | pos, tag | end};
                    else atomicOr(&ctl[CTL_ERR], EB_INTERNAL);   // totals left by a launch that did not finish
                    if (pp < M) present[pp] = m;
                    ++pp;
                }
                kept[m] = 0u;
            }
            pos += cnt[j];
        }
        carry += tot;
        pcarry += ptot;
    }
    if (write && tid == 0) {
        const u32 slot = E.slot & 1u;
        ctl[CTL_BIG] = 0u;
        ctl[CTL_SCR] = 0u;
        ctl[CTL_DEFERRED] = 0u;
        ctl[CTL_CTR] = 0u;                       // the small kernel's ticket of this event
        ctl[CTL_PRESENT + slot] = pcarry;
        ctl[CTL_PRESENT + (slot ^ 1u)] = 0u;
    }
}

__global__ __launch_bounds__(G_WG) void k_group_table(LaunchArgs a) {
    __shared__ u32 s_wsum[G_WG / 64];
    const u32 k = num_events(a);
    for (u32 e = blockIdx.x; e < k; e += gridDim.x) {
        const EventDesc E = get_event(a, e);
        if (!(E.flags & EF_UNSORTED)) continue;  // the same event for the whole workgroup
        group_table(E, ev_layout(E.cap, a.n_modules), a.n_modules, nullptr, true, s_wsum);
    }
}

// TABLE: the first positions come from k_group_table's table.  Else (at most G_HMAX modules)
// every workgroup scans the totals of its event itself, and the one with the event's first
// chunk also writes the table: reading 7 KB from the L2 and two scans (~2 us) take the place
// of a launch of one workgroup per event (6.4 us and the gap before it).
template <bool TABLE>
__global__ __launch_bounds__(G_WG) void k_group_scatter(LaunchArgs a) {
    __shared__ u32 s_pref[MAXB + 1];
    __shared__ u32 s_wsum[G_WG / 64];
    __shared__ u32 s_first[TABLE ? 1 : G_HMAX];
    const u32 tid = threadIdx.x, k = num_events(a), M = a.n_modules;
    const u32 total = event_prefix<G_WG>(a, k, s_pref, s_wsum, CNT_ANY, G_SCH, 0);
    u32 have = NOPIX;                            // the event whose positions s_first holds
    for (u32 t = blockIdx.x; t < total; t += gridDim.x) {
        const u32 e = find_slot(s_pref, k, t), c = t - s_pref[e];
        const EventDesc E = get_event(a, e);
        const EvLayout L = ev_layout(E.cap, M);
        const ModRange* mt = ws_ptr<const ModRange>(E, L.mtab);
        const u32* rank = (const u32*)E.o_digi;
        u64* rec = ws_ptr<u64>(E, L.grp);
        // every load first (module ids, then table entries, ranks and the digis), then
        // the stores: stores to the grouped copy could alias the input for the compiler,
        // which would otherwise keep each digi's loads behind the previous digi's stores
        const u32 i0 = c * G_SCH + tid;
        u32 mm[G_SPER], pos[G_SPER], rr[G_SPER], cc[G_SPER], aa[G_SPER];
#pragma unroll
        for (u32 q = 0; q < G_SPER; ++q) {
            const u32 i = i0 + q * G_WG;
            const u32 iv = i < E.n ? i : 0u;
            mm[q] = i < E.n ? u32(E.r_module[i]) : NOPIX;
            if constexpr (!TABLE) pos[q] = rank[iv];
            rr[q] = E.r_row[iv];
            cc[q] = E.r_col[iv];
            aa[q] = E.r_adc[iv];
        }
        if constexpr (!TABLE) {
            if (e != have) {
                lds_barrier();                   // every digi of the last chunk has its position
                group_table(E, L, M, s_first, c == 0, s_wsum);
                lds_barrier();
                have = e;
            }
        }
#pragma unroll
        for (u32 q = 0; q < G_SPER; ++q) {
            const u32 i = i0 + q * G_WG;
            const bool v = mm[q] < M;            // past the end, or out of range (flagged by count)
            if constexpr (TABLE) {
                const ModRange r = mt[v ? mm[q] : 0u];
                pos[q] = (v && u32(r.first >> 32) == E.epoch) ? u32(r.first) + rank[v ? i : 0u] : NOPIX;
                if (pos[q] != NOPIX && pos[q] >= u32(r.end)) pos[q] = NOPIX;   // only after an internal error
            } else {
                pos[q] = v ? s_first[mm[q]] + pos[q] : NOPIX;
            }
        }
#pragma unroll
        for (u32 q = 0; q < G_SPER; ++q)
            if (pos[q] < E.n) rec[pos[q]] = pack_digi(rr[q], cc[q], aa[q], i0 + q * G_WG);   // (not below only after one)
    }
}

// ---------------------------------------------------------------------------
// segment: every digi at a module boundary writes the module's entry of the module
// table (first digi, one past the last), tagged with the launch, and the digi that
// starts a module appends it to the present-module list (one atomic per chunk for
// the chunk's place in it); module ids must be non-decreasing (else EB_ORDER) and
// below the module count (else EB_RANGE).  The first chunk of an event also clears
// its kept counts (an absent module keeps nothing) and empties its big-module list.
// ---------------------------------------------------------------------------
template <u32 PER>
__global__ __launch_bounds__(A_WG) void k_segment(LaunchArgs a) {
    constexpr u32 CH = A_WG * PER;
    __shared__ u32 s_pref[MAXB + 1];
    __shared__ u32 s_wsum[A_WG / 64];
    __shared__ u32 s_err, s_base;
    const u32 tid = threadIdx.x;
    const u32 k = num_events(a);
    const u32 total = event_prefix<A_WG>(a, k, s_pref, s_wsum, CNT_SORTED, CH, 0);
    // The tickets start at zero in every launch: the compaction kernel of a finished
    // launch resets them, and this reset also covers a launch whose later kernels were
    // never queued.
    if (blockIdx.x == 0 && tid == 0) reset_tickets(a);

    for (u32 t = blockIdx.x; t < total; t += gridDim.x) {
        if (tid == 0) s_err = 0;
        const u32 e = find_slot(s_pref, k, t);
        const u32 c = t - s_pref[e];
        const EventDesc E = get_event(a, e);
        const EvLayout L = ev_layout(E.cap, a.n_modules);
        ModRange* mt = ws_ptr<ModRange>(E, L.mtab);
        const u32 n = E.n;
        const u32 i0 = c * CH + tid * PER;
        u32 m[PER];
        if ((reinterpret_cast<uintptr_t>(E.module) & 15u) == 0 && i0 + PER <= n) {
            uint4 v[PER / 8];                             // 16-byte loads, all in flight together
#pragma unroll
            for (u32 q = 0; q < PER / 8; ++q) v[q] = ((const uint4*)(E.module + i0))[q];
#pragma unroll
            for (u32 q = 0; q < PER / 8; ++q) {
                const u32 w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
                for (u32 j = 0; j < 8; ++j) m[8 * q + j] = (w[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
            }
        } else {
#pragma unroll
            for (u32 j = 0; j < PER; ++j) m[j] = E.module[min(i0 + j, n - 1)];
        }
        const u32 prev = E.module[i0 > 0 ? min(i0 - 1, n - 1) : 0];
        const u32 next = E.module[min(i0 + PER, n - 1)];
        u32* ctl = ws_ptr<u32>(E, L.ctl);
        const u32 slot = E.slot & 1u;
        if (c == 0) {                            // read by the kernels after this one
            if (tid == 0) {
                ctl[CTL_BIG] = 0u;
                ctl[CTL_SCR] = 0u;
                ctl[CTL_DEFERRED] = 0u;
                ctl[CTL_CTR] = 0u;                     // the small kernel's ticket of this event
                ctl[CTL_PRESENT + (slot ^ 1u)] = 0u;   // for the next launch (the last one's is done)
            }
            u32* kept = ws_ptr<u32>(E, L.kept);
            for (u32 q = tid; q < a.n_modules; q += A_WG) kept[q] = 0u;
        }
        u32 err = 0, starts = 0;
        const u64 tag = u64(E.epoch) << 32;
#pragma unroll
        for (u32 j = 0; j < PER; ++j) {
            const u32 i = i0 + j;
            if (i < n) {
                const u32 pm = (j == 0) ? prev : m[j - 1];
                const u32 nm = (j + 1 == PER) ? next : m[j + 1];
                if (i > 0 && m[j] < pm) err |= EB_ORDER;
                if (m[j] >= a.n_modules) {
                    err |= EB_RANGE;
                } else {
                    if (i == 0 || m[j] != pm) {
                        mt[m[j]].first = tag | i;
                        starts |= 1u << j;
                    }
                    if (i + 1 == n || m[j] != nm) mt[m[j]].end = tag | (i + 1);
                }
            }
        }
        u32 nstart;
        const u32 ex = group_excl_scan<A_WG>(__popc(starts), tid, s_wsum, nstart);   // also orders s_err
        if (tid == 0) s_base = nstart ? atomicAdd(&ctl[CTL_PRESENT + slot], nstart) : 0u;
        lds_barrier();
        u32* present = ws_ptr<u32>(E, L.present);
        u32 r = s_base + ex;
#pragma unroll
        for (u32 j = 0; j < PER; ++j)
            if (starts & (1u << j)) {
                if (r < a.n_modules) present[r] = m[j];
                else err |= EB_INTERNAL;         // a count left by a launch that did not finish
                ++r;
            }
        if (err) atomicOr(&s_err, err);
        lds_barrier();
        if (tid == 0 && s_err) atomicOr(&ctl[CTL_ERR], s_err);
        lds_barrier();                           // before s_err is cleared for the next chunk
    }
}

// ---------------------------------------------------------------------------
// clustering of one module with its digis in registers (K per thread, group of G)
// ---------------------------------------------------------------------------

template <u32 G, u32 K>
struct RegModuleSmem {
    static constexpr u32 RCAP = G * K, KBW = RCAP / 32;
    u32 bm[BM_WORDS];      // fired-pixel bitmap (clear between modules)
    u16 rpre[BM_WORDS];    // runs before each word, less one when the word's bit 0 continues a
                           // run of the word above (as in a column's entry, for each word)
    alignas(8) u64 acc[RCAP];   // per run: parent (16 bits) | size (16) | charge (32), charge and
                           // size at the roots only; then, at the roots, first pixel (17) |
                           // size (15) | charge (32)
    u32 kb[KBW];           // kept-root bits over run index
    u16 kpre[KBW];         // kept roots before each kb word
    u32 wsum[G / 64];
    u32 nlink;             // some pair of runs is left to unite
};

// A module as a group sees it.
struct Item {
    u32 e, it, st, n, mod;
    bool ok;
};

template <typename T>
__device__ __forceinline__ T PXCL_G* wave_uniform(T PXCL_G* p) {
    const u64 x = reinterpret_cast<u64>(p);
    return (T PXCL_G*)(u64(wave_uniform(u32(x))) | (u64(wave_uniform(u32(x >> 32))) << 32));
}
__device__ __forceinline__ Item wave_uniform(const Item& I) {
    return Item{wave_uniform(I.e), wave_uniform(I.it), wave_uniform(I.st), wave_uniform(I.n), wave_uniform(I.mod),
                wave_uniform(I.ok ? 1u : 0u) != 0};
}
__device__ __forceinline__ EventDesc wave_uniform(const EventDesc& E) {
    EventDesc U{};
    U.module = wave_uniform(E.module);
    U.row = wave_uniform(E.row);
    U.col = wave_uniform(E.col);
    U.adc = wave_uniform(E.adc);
    U.r_module = wave_uniform(E.r_module);
    U.r_row = wave_uniform(E.r_row);
    U.r_col = wave_uniform(E.r_col);
    U.r_adc = wave_uniform(E.r_adc);
    U.ws = wave_uniform(E.ws);
    U.hstat = wave_uniform(E.hstat);
    U.o_digi = wave_uniform(E.o_digi);
    U.o_id = wave_uniform(E.o_id);
    U.o_charge = wave_uniform(E.o_charge);
    U.o_size = wave_uniform(E.o_size);
    U.n = wave_uniform(E.n);
    U.cap = wave_uniform(E.cap);
    U.epoch = wave_uniform(E.epoch);
    U.slot = wave_uniform(E.slot);
    U.flags = wave_uniform(E.flags);
    return U;
}

// Issue the loads of the module's digis j = lt + q*G < n: row and column packed in
// one register (row | col << 16, half-word loads into each half), adc in another; the
// values are only used when the module is clustered, so the loads stay in flight
// meanwhile (those of an event in any order are unpacked here, and waited for).
template <u32 G, u32 K>
__device__ __forceinline__ void fetch_digis(const ModuleDigis& D, u32 n, u32 lt, u32* RC, u32* A) {
    if (D.rec) {
        u64 v[K];
#pragma unroll
        for (u32 q = 0; q < K; ++q)
            if (q * G < n && lt + q * G < n) v[q] = D.rec[lt + q * G];
#pragma unroll
        for (u32 q = 0; q < K; ++q) {
            const bool in = q * G < n && lt + q * G < n;
            RC[q] = in ? ModuleDigis::rc_of(v[q]) : NOPIX;
            A[q] = in ? u32(v[q]) & 0xFFFFu : 0u;
        }
        return;
    }
#pragma unroll
    for (u32 q = 0; q < K; ++q) {
        const u32 j = lt + q * G;
        RC[q] = NOPIX;
        A[q] = 0u;
        if (q * G < n && j < n) {
            RC[q] = u32(D.row[j]) | (u32(D.col[j]) << 16);
            A[q] = D.adc[j];
        }
    }
}

// f(q) for the digi slots q < nq (nq uniform over the group), in steps of U that the
// compiler may interleave (f must do nothing for a slot at or above nq).  The loop over the
// steps is not unrolled, so a large body appears once in the code (the register arrays it
// indexes with the uniform q stay in registers).
template <u32 K, u32 U, typename F>
__device__ __forceinline__ void for_slots(u32 nq, F f) {
    static_assert(K % U == 0, "whole steps");
#pragma unroll 1
    for (u32 q = 0; q < nq; q += U)
#pragma unroll
        for (u32 u = 0; u < U; ++u) f(q + u);
}

// Cluster module I (n <= G*K) whose raw digis are in RC/A (fetch_digis).  Every
// thread of the group calls it; with G > 64 all groups of the workgroup (SOLE: there is
// one) call it together.  `mid(stage)` runs at the end of phase 1, at the start of phase 3 and after
// phase 5 (the next module's prefetch).
//
// What bounds it is the number of instructions a wave issues (at four waves per SIMD its
// vector unit is busy half the time) and, for one module alone, their chain through the
// phases.  So the phases are few (8 barriers), a digi's LDS reads in a phase do not depend
// on each other where that can be had, and what is the same for a wave is kept scalar:
//   1  bitmap
//   2  run numbers of the bitmap words
//   3  every digi reads the four rows around it in three columns (three pairs of adjacent
//      words) and finds its run; a digi that starts a run stores the run's parent: the run
//      rule B links it to, or itself (a plain store: no other link decides the first parent)
//   4  only if some run has a rule A link: those unions
//   5  root of every digi's run, charge and size into the root's word
//   6  cut, one bit per kept root
//   7  outputs
template <u32 G, u32 K, bool SOLE, typename Mid>
__device__ __forceinline__ void cluster_regs(const LaunchArgs& a, const EventDesc& E, const EvLayout& L,
                                             const Item& I, RegModuleSmem<G, K>& gp, u32 lt, u32* RC, u32* A,
                                             Mid mid) {
    static_assert(G * K <= 16384, "sizes of up to 15 bits, run numbers of up to 16");
    constexpr u32 KBW = G * K / 32, CPT = (COLS + G - 1) / G;
    lt = (lt + (I.n >> 31)) & (G - 1u);                    // worked out anew for every module, as in thread_in_loop
    const bool act = I.ok;
    const u32 nq = act ? min((I.n + G - 1) / G, K) : 0u;   // slots that may hold a digi
    u32 err = 0, dup = 0, starts = 0;                      // starts, bit q: slot q starts its run
    auto has = [&](u32 mask, u32 q) { return ((mask >> q) & 1u) != 0; };
    // 1: the module's digis into the bitmap (RC becomes NOPIX for one out of range)
    if (lt == 0) {
        gp.nlink = 0u;
        gp.acc[0] = 0ull;                                  // run 0, its own root, also when no digi is in range
    }
    for (u32 w = lt; w < KBW; w += G) gp.kb[w] = 0u;
#pragma unroll
    for (u32 q = 0; q < K; ++q) {
        if (q < nq && lt + q * G < I.n) {
            const u32 row = RC[q] & 0xFFFFu, c = RC[q] >> 16, bit = 1u << (row & 31u);
            if (row < ROWS && c < COLS) {
                dup |= atomicOr(&gp.bm[BM_FRONT + c * WPC + (row >> 5)], bit) & bit;
            } else {
                err = EB_RANGE;
                RC[q] = NOPIX;
            }
        }
    }
    if (dup) err |= EB_DUP;
    mid(0);
    gsync<G>();
    // 2: run starts per word, prefix over the words in column order.  A thread takes CPT
    // consecutive columns.
    {
        u32 cnt = 0, n_before[CPT * WPC];
        const u32 c0 = lt * CPT;
#pragma unroll
        for (u32 i = 0; i < CPT; ++i) {
            u32 above = 0;
            const u32 c = min(c0 + i, COLS);               // past the last column: words that stay zero
#pragma unroll
            for (u32 k = 0; k < WPC; ++k) {
                const u32 b = gp.bm[BM_FRONT + c * WPC + k];
                cnt -= b & above;
                n_before[i * WPC + k] = cnt;
                cnt += __popc(b & ~(b << 1));
                above = b >> 31;
            }
        }
        const u32 inc = wave_incl_scan(cnt);
        u32 run = inc - cnt;
        if constexpr (G > 64) {
            if ((lt & 63u) == 63u) gp.wsum[lt >> 6] = inc;
            gsync<G>();
            const u32 wv = wave_uniform(lt >> 6);
            for (u32 i = 0; i < wv; ++i) run += gp.wsum[i];
        }
#pragma unroll
        for (u32 i = 0; i < CPT; ++i)
            if (c0 + i < COLS)
#pragma unroll
                for (u32 k = 0; k < WPC; ++k) gp.rpre[BM_FRONT + (c0 + i) * WPC + k] = u16(run + n_before[i * WPC + k]);
    }
    gsync<G>();
    mid(1);
    // 3: every digi's run (X: the run, above it the run a rule A link goes to), first parents
    u32 X[K];
    u32 link = 0;                                          // bit q: slot q has a rule A link
    for_slots<K, 2>(nq, [&](u32 q) {
        X[q] = 0u;
        if (RC[q] == NOPIX) return;
        const u32 row = RC[q] & 0xFFFFu, c = RC[q] >> 16;
        // rows s..s+3 of the columns c-1, c, c+1 lie in two adjacent words each
        const u32 s = row >= 2 ? row - 2 : 0u, ks = s >> 5, w0 = c * WPC + ks;   // in column c-1
        const u32* w = &gp.bm[w0];
        const u32 l0 = w[0], l1 = w[1], m0 = w[WPC], m1 = w[WPC + 1], r0 = w[2 * WPC], r1 = w[2 * WPC + 1];
        const u32 own = (row >> 5) - ks, before = gp.rpre[w0 + WPC + own];
        // bit i: row - 2 + i fired (above the first row and below the last one: not)
        const u32 up = row >= 2 ? 0u : 2u - row, mask = row + 1 < ROWS ? 15u : 7u;
        auto window = [&](u32 lo, u32 hi) { return (u32(((u64(hi) << 32) | lo) >> (s & 31u)) << up) & mask; };
        auto run_in = [&](u32 before, u32 word, u32 r) {   // run of row r, fired, of a word
            return before + __popc(word & ~(word << 1) & ((2u << (r & 31u)) - 1u)) - 1u;
        };
        const u32 wl = window(l0, l1), wm = window(m0, m1), wr = window(r0, r1);
        const u32 r = run_in(before, own ? m1 : m0, row);
        X[q] = r;
        if (wm & 2u) return;                               // not the first pixel of its run
        starts |= 1u << q;
        u32 parent = r;
        if (wl & 14u) {                                    // rule B
            const u32 f = row - 1u + __builtin_ctz((wl >> 1) & 7u), h = (f >> 5) - ks;
            parent = run_in(gp.rpre[w0 + h], h ? l1 : l0, f);
        }
        gp.acc[r] = u64(parent) << 48;
        if ((wr & 2u) && ((wm | wr) & 1u)) {               // rule A
            const u32 f = row - 1u, h = (f >> 5) - ks;
            X[q] |= run_in(gp.rpre[w0 + 2 * WPC + h], h ? r1 : r0, f) << 16;
            link |= 1u << q;
        }
    });
    if (link) st_wg(&gp.nlink, 1u);
    gsync<G>();
    // 4: rule A's unions (groups that share the workgroup's barrier all take it)
    const bool unions = ld_wg(&gp.nlink) != 0;
    if (unions) {
#pragma unroll 1
        for (u32 q = 0; q < nq; ++q)
            if (has(link, q)) unite_packed(gp.acc, X[q] & 0xFFFFu, X[q] >> 16);
    }
    if ((G > 64 && !SOLE) || unions) gsync<G>();
    // 5: roots (the walks of all slots step together), then charge and size per root.  Sums
    // touch the low 48 bits of roots only, walks read the parents.  Most trees are shallow:
    // a few plain steps; what is left points runs to ancestors as it goes.
    u32 more = 0;
#pragma unroll
    for (u32 q = 0; q < K; ++q)
        if (q < nq) {
            X[q] &= 0xFFFFu;                               // run 0 where there is no pixel
            const u32 p = parent_of(gp.acc, X[q]);
            if (p != X[q]) starts &= ~(1u << q);           // now: the digi starts its cluster
            X[q] = p;
        }
    for (u32 step = 0; step < 3; ++step) {
        more = 0;
#pragma unroll
        for (u32 q = 0; q < K; ++q)
            if (q < nq) {
                const u32 p = parent_of(gp.acc, X[q]);
                more |= p ^ X[q];
                X[q] = p;
            }
        if (!more) break;
    }
    if (more) {
#pragma unroll 1
        for (u32 q = 0; q < nq; ++q) X[q] = find_packed(gp.acc, X[q]);
    }
#pragma unroll
    for (u32 q = 0; q < K; ++q)
        if (q < nq && RC[q] != NOPIX) atomicAdd(&gp.acc[X[q]], (1ull << 32) | u64(A[q] & 0xFFFFu));
    mid(2);
    gsync<G>();
    // 6: charge cut, one bit per kept root; its word's upper half becomes the first pixel
    // and the size
#pragma unroll
    for (u32 q = 0; q < K; ++q)
        if (q < nq && has(starts, q)) {
            const u32 r = X[q];
            const u64 v = gp.acc[r];
            const u32 lin = (RC[q] >> 16) * ROWS + (RC[q] & 0xFFFFu);
            if (u32(v) >= a.charge_cut) atomicOr(&gp.kb[r >> 5], 1u << (r & 31u));
            st_wg(hi_word(gp.acc, r), (lin << 15) | (u32(v >> 32) & 0x7FFFu));
        }
    gsync<G>();
    // 7: kept roots before each kb word (every wave writes all of them, the same values, and
    // reads what it wrote), then the outputs: kept clusters -> staging records at
    // [st + position in the module], per-digi cluster ids; with fused hits every kept digi's
    // weighted coordinates go to its cluster's sums; the bitmap words used are cleared
    if (act) {
        constexpr u32 KPL = (KBW + 63) / 64;               // kb words per lane
        const u32 lane = lt & 63u;
        u32 pc[KPL], cnt = 0;
#pragma unroll
        for (u32 i = 0; i < KPL; ++i) {
            pc[i] = lane * KPL + i < KBW ? __popc(gp.kb[lane * KPL + i]) : 0u;
            cnt += pc[i];
        }
        const u32 inc = wave_incl_scan(cnt);
        u32 pre = inc - cnt;
#pragma unroll
        for (u32 i = 0; i < KPL; ++i) {
            if (lane * KPL + i < KBW) __hip_atomic_store(&gp.kpre[lane * KPL + i], u16(pre), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            pre += pc[i];
        }
        gsync<64>();
        if (lt == 63) ws_ptr<u32>(E, L.kept)[I.it] = inc;
        auto position = [&](u32 r) {                       // of the kept root r in the module
            return u32(__hip_atomic_load(&gp.kpre[r >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) +
                   __popc(gp.kb[r >> 5] & ((1u << (r & 31u)) - 1u));
        };
        const bool hits = (E.flags & EF_HITS) != 0;
        u64* hs = ws_ptr<u64>(E, L.hsum) + 2 * size_t(I.st);
        int32_t* tid_ = ws_ptr<int32_t>(E, L.tid) + I.st;
        int32_t* tch = ws_ptr<int32_t>(E, L.tcharge) + I.st;
        int32_t* tsz = ws_ptr<int32_t>(E, L.tsize) + I.st;
        const ModuleDigis D = module_digis(E, L, I.st);
        int32_t* od = (int32_t*)E.o_digi + (D.rec ? 0u : I.st);
        const u32 idbase = I.mod * PIX;
#pragma unroll
        for (u32 q = 0; q < K; ++q) {
            const u32 j = lt + q * G;
            if (q < nq && j < I.n) {
                int32_t id = -1;
                if (RC[q] != NOPIX) {
                    const u64 v = gp.acc[X[q]];
                    const u32 charge = u32(v), row = RC[q] & 0xFFFFu, c = RC[q] >> 16;
                    st_wg(&gp.bm[BM_FRONT + c * WPC + (row >> 5)], 0u);   // several digis may share a word
                    if (charge >= a.charge_cut) {
                        id = int32_t(idbase + u32(v >> 47));
                        if (has(starts, q)) {
                            const u32 p = position(X[q]);
                            tid_[p] = id;
                            tch[p] = int32_t(charge);
                            tsz[p] = int32_t(u32(v >> 32) & 0x7FFFu);
                        }
                        if (hits) {
                            const u32 p = position(X[q]);
                            const u64 w = D.adc_at(j);                 // A holds the next module's
                            atomicAdd(&hs[2 * p], w * c);
                            atomicAdd(&hs[2 * p + 1], w * row);
                        }
                    }
                }
                od[D.rec ? ModuleDigis::pos_of(D.rec[j]) : j] = id;
            }
        }
        if (err) atomicOr(ws_ptr<u32>(E, L.ctl) + CTL_ERR, err);
    }
    gsync<G>();
}

// ---------------------------------------------------------------------------
// XCD-aware order of workgroups: consecutive workgroup ids go to the eight XCDs in
// turn, so the order (id % 8, id / 8) gives each XCD a contiguous share of the work
// and the data its modules read and write stays in that XCD's L2.  A bijection on
// [0, n) for any n.
// ---------------------------------------------------------------------------
constexpr u32 N_XCD = 8;
__device__ __forceinline__ u32 xcd_order(u32 b, u32 n) {
    const u32 q = n / N_XCD, r = n % N_XCD, x = b % N_XCD, i = b / N_XCD;
    return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// ---------------------------------------------------------------------------
// Module ranges by search (launches without the segmentation kernel): with the
// module ids sorted, module m's digis are [lower bound of m, lower bound of m + 1).
// One wave finds both.  The first round probes 64 points SEARCH_STEP apart around
// where module m would start if the modules were evenly filled; when that brackets
// a bound, it is within SEARCH_STEP digis and the last round (up to 128 candidates,
// two per lane) finds it: two dependent loads.  Otherwise each further round probes
// 64 evenly spaced points of the remaining range and keeps the stretch the ballot
// points to (about 65 times shorter).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void narrow_range(u32& lo, u32& hi, u64 ge) {
    const u32 s = hi - lo;                      // > 64; probe l at lo + (l + 1) * s / 65
    if (ge) {
        const u32 f = __builtin_ctzll(ge);      // first probe at or above the key
        hi = lo + u32((u64(f) + 1) * s / 65);
        lo = f ? lo + u32(u64(f) * s / 65) + 1 : lo;
    } else {
        lo = lo + u32(u64(64) * s / 65) + 1;
    }
}

constexpr u32 SEARCH_STEP = 128, SEARCH_LAST = 128;

// Narrow [lo, hi] by a ballot over probes at q(l) = clamp(guess + (l - 32) * step),
// non-decreasing in l; the answer is the first index whose id is >= the key.
__device__ __forceinline__ void narrow_window(u32& lo, u32& hi, u64 ge, long long guess, u32 n) {
    auto q = [&](u32 l) -> u32 {
        const long long p = guess + (static_cast<long long>(l) - 32) * SEARCH_STEP;
        return u32(p < 0 ? 0 : (p >= (long long)n ? (long long)n - 1 : p));
    };
    if (ge) {
        const u32 f = __builtin_ctzll(ge);
        hi = q(f);
        if (f) lo = q(f - 1) + 1;
    } else {
        lo = q(63) + 1;
    }
}

// The search in three steps, each issuing the loads the next one looks at, so that a group
// can do other work in between: probe, narrow, finish.
struct RangeSearch {
    u32 v;                       // probe
    u32 lo0, hi0, lo1, hi1;      // each answer lies in [lo, hi]
    u32 p0, q0, p1, q1;          // last candidates (ids), NOPIX past hi
};
// Index where module `key` starts if the modules are evenly filled (any guess will do).
__device__ __forceinline__ long long range_guess(const EventDesc& E, u32 n_modules, u32 key) {
    return static_cast<long long>(float(key) * (float(E.n) / float(n_modules)));
}
__device__ __forceinline__ void range_probe(RangeSearch& S, const EventDesc& E, u32 n_modules, u32 key, u32 lane) {
    const long long n = E.n, p = range_guess(E, n_modules, key) + (static_cast<long long>(lane) - 32) * SEARCH_STEP;
    S.v = ((const u16*)E.module)[p < 0 ? 0u : u32(p >= n ? n - 1 : p)];
}
__device__ __forceinline__ void range_narrow(RangeSearch& S, const EventDesc& E, u32 n_modules, u32 key, u32 lane) {
    const u16* mod = (const u16*)E.module;
    const u32 n = E.n;
    const long long guess = range_guess(E, n_modules, key);
    u32 lo0 = 0, hi0 = n, lo1 = 0, hi1 = n;
    {
        const u64 b0 = __ballot(S.v >= key), b1 = __ballot(S.v >= key + 1);
        narrow_window(lo0, hi0, b0, guess, n);
        narrow_window(lo1, hi1, b1, guess, n);
    }
    while (hi0 - lo0 > SEARCH_LAST || hi1 - lo1 > SEARCH_LAST) {
        const bool w0 = hi0 - lo0 > SEARCH_LAST, w1 = hi1 - lo1 > SEARCH_LAST;
        const u32 q0 = lo0 + u32((u64(lane) + 1) * (hi0 - lo0) / 65);   // < hi0 <= n
        const u32 q1 = lo1 + u32((u64(lane) + 1) * (hi1 - lo1) / 65);
        const bool g0 = w0 && mod[q0] >= key;
        const bool g1 = w1 && mod[q1] >= key + 1;
        const u64 b0 = __ballot(g0), b1 = __ballot(g1);
        if (w0) narrow_range(lo0, hi0, b0);
        if (w1) narrow_range(lo1, hi1, b1);
    }
    S.lo0 = lo0; S.hi0 = hi0; S.lo1 = lo1; S.hi1 = hi1;
    // at most SEARCH_LAST = 128 candidates per bound: positions lo + lane, lo + 64 + lane
    S.p0 = S.q0 = S.p1 = S.q1 = NOPIX;
    if (lo0 + lane < hi0) S.p0 = mod[lo0 + lane];
    if (lo0 + 64 + lane < hi0) S.q0 = mod[lo0 + 64 + lane];
    if (lo1 + lane < hi1) S.p1 = mod[lo1 + lane];
    if (lo1 + 64 + lane < hi1) S.q1 = mod[lo1 + 64 + lane];
}
__device__ __forceinline__ void range_finish(const RangeSearch& S, u32 key, u32& first, u32& end) {
    auto at_least = [](u32 v, u32 k) { return v != NOPIX && v >= k; };
    const u64 b0 = __ballot(at_least(S.p0, key)), c0 = __ballot(at_least(S.q0, key));
    const u64 b1 = __ballot(at_least(S.p1, key + 1)), c1 = __ballot(at_least(S.q1, key + 1));
    first = b0 ? S.lo0 + u32(__builtin_ctzll(b0)) : c0 ? S.lo0 + 64 + u32(__builtin_ctzll(c0)) : S.hi0;
    end = b1 ? S.lo1 + u32(__builtin_ctzll(b1)) : c1 ? S.lo1 + 64 + u32(__builtin_ctzll(c1)) : S.hi1;
}

// Order and range checks of every digi's module id (launches without the
// segmentation kernel), one coalesced pass over the whole grid.  The first stride's
// ids are loaded by id_check_load (before the first range search, so that the two
// latencies overlap) and checked, with the rest, by id_check_finish.
struct IdCheck {
    u32 m0, m1;
};
template <u32 WG>
__device__ __forceinline__ IdCheck id_check_load(const EventDesc& E) {
    const u32 i = blockIdx.x * WG + threadIdx.x;
    IdCheck c{0u, 0xFFFFFFFFu};
    if (i < E.n) {
        c.m0 = E.module[i];
        if (i + 1 < E.n) c.m1 = E.module[i + 1];
    }
    return c;
}
template <u32 WG>
__device__ __forceinline__ void id_check_finish(const LaunchArgs& a, const EventDesc& E, IdCheck c) {
    u32 err = 0;
    for (u32 i = blockIdx.x * WG + threadIdx.x; i < E.n; i += gridDim.x * WG) {
        if (i >= gridDim.x * WG) {               // strides after the first
            c.m0 = E.module[i];
            c.m1 = i + 1 < E.n ? E.module[i + 1] : 0xFFFFFFFFu;
        }
        if (c.m0 >= a.n_modules) err |= EB_RANGE;
        if (c.m1 < c.m0) err |= EB_ORDER;
    }
    if (err) atomicOr(ws_ptr<u32>(E, ev_layout(E.cap, a.n_modules).ctl) + CTL_ERR, err);
}

// ---------------------------------------------------------------------------
// small: groups of G = WG/MPW threads, one module each, modules by ticket
// ---------------------------------------------------------------------------
template <u32 WG, u32 MPW, u32 K>
struct SmallSmem {
    static constexpr u32 G = WG / MPW;
    RegModuleSmem<G, K> grp[MPW];
    u32 pref[MAXB + 1];
    u32 wsum[WG / 64];
    u32 tick;                                 // the module after the current one (G > 64), once it is dynamic
};

// Waves per SIMD the shape's LDS allows, at most five (at most 96 registers): modules in
// flight bound throughput, so registers should not bound them first.  At 256x1 five fit
// (LDS for five groups a compute unit); six at 512x1 would spill 26 registers a lane.
template <u32 WG, u32 MPW, u32 K>
constexpr u32 small_waves_per_simd() {
    constexpr u32 lds_groups = 163840u / u32(sizeof(SmallSmem<WG, MPW, K>));
    constexpr u32 w = lds_groups * (WG / 64) / 4;
    return w < 1 ? 1 : (w > 5 ? 5 : w);
}
#ifndef PXCL_WAVES_PER_EU
#define PXCL_WAVES_PER_EU(...) __attribute__((amdgpu_waves_per_eu(__VA_ARGS__)))
#endif
template <u32 WG, u32 MPW, u32 K>
__global__ __launch_bounds__(WG) PXCL_WAVES_PER_EU(small_waves_per_simd<WG, MPW, K>()) void k_small(LaunchArgs a) {
    using S = SmallSmem<WG, MPW, K>;
    constexpr u32 G = S::G;
    constexpr bool WAVE = (G == 64);          // groups of one wave run independently
    constexpr u32 STEP = WAVE ? 1u : MPW;     // modules per ticket
    __shared__ S s;
    const u32 tid = threadIdx.x, g = tid / G, lt = tid % G;
    const u32 gofs = WAVE ? 0u : g;
    RegModuleSmem<G, K>& gp = s.grp[g];
    for (u32 w = lt; w < BM_WORDS; w += G) gp.bm[w] = 0u;
    const u32 k = num_events(a);
    // Without the segmentation kernel (one event): every module is a unit, its
    // digis found by search; this kernel then checks the module ids, writes the
    // module table entries of the modules present and sets the unit count the
    // kernels after it read.
    const bool fused = (a.flags & LF_FUSED) != 0 && k == 1;
    u32 total;
    IdCheck idc{0u, 0xFFFFFFFFu};
    if (k == 1) {                             // one event, alone or in a header
        const EventDesc E0 = get_event(a, 0);
        if (fused) {
            total = E0.n ? a.n_modules : 0u;
            idc = id_check_load<WG>(E0);
            if (blockIdx.x == 0 && tid == 0 && E0.n) {
                u32* ctl = ws_ptr<u32>(E0, ev_layout(E0.cap, a.n_modules).ctl);
                ctl[CTL_PRESENT + (E0.slot & 1u)] = a.n_modules;
                ctl[CTL_PRESENT + ((E0.slot & 1u) ^ 1u)] = 0u;
            }
        } else {
            total = unit_count(a, E0);
        }
        if (tid == 0) {
            s.pref[0] = 0;
            s.pref[1] = total;
        }
        lds_barrier();
    } else {
        total = event_prefix<WG>(a, k, s.pref, s.wsum, CNT_UNITS, 1, 0);
    }
    // Work unit t: unit t - pref[e] of event e.  Its module's range comes in three steps,
    // each issuing the loads the next one waits for: the module id, the module's table entry,
    // the item (without the table: the steps of the search).
    struct Next {
        const EventDesc* E;
        u32 e, mod;
        RangeSearch S;
        ModRange r;
    };
    const u32 lane = lt & 63u;
    auto step_module = [&](u32 t, Next& N) {
        N.e = k == 1 ? 0u : find_slot(s.pref, k, t);
        N.E = event_at(a, N.e);
        if (fused) {
            N.mod = t;
            range_probe(N.S, *N.E, a.n_modules, t, lane);
            return;
        }
        const u32 first = wave_uniform(s.pref[N.e]), units = wave_uniform(s.pref[N.e + 1]) - first;
        N.mod = t - first;                    // dense (a list as long as the module count is all of them)
        if (units != a.n_modules) N.mod = ws_ptr<const u32>(*N.E, ev_layout(N.E->cap, a.n_modules).present)[t - first];
    };
    auto step_range = [&](Next& N) {
        if (fused) {
            range_narrow(N.S, *N.E, a.n_modules, N.mod, lane);
            return;
        }
        N.mod = min(wave_uniform(N.mod), a.n_modules - 1);
        N.r = ws_ptr<const ModRange>(*N.E, ev_layout(N.E->cap, a.n_modules).mtab)[N.mod];
    };
    // I.n = 0 for an entry that is not this launch's (or inconsistent after an
    // ordering error); ok only for a present module the group can hold.
    auto step_item = [&](Next& N) {
        Item I{N.e, N.mod, 0, 0, N.mod, false};
        u32 st, en;
        bool mine = true;
        if (fused) {
            range_finish(N.S, N.mod, st, en);
            const u64 tag = u64(N.E->epoch) << 32;
            if (lt == 0 && en > st)           // for the big kernel, compaction, hits
                ws_ptr<ModRange>(*N.E, ev_layout(N.E->cap, a.n_modules).mtab)[N.mod] = ModRange{tag | st, tag | en};
        } else {
            st = u32(N.r.first);
            en = u32(N.r.end);
            mine = u32(N.r.first >> 32) == N.E->epoch && u32(N.r.end >> 32) == N.E->epoch;
        }
        if (mine && st < en && en <= N.E->n) {
            I.st = st;
            I.n = en - st;
        }
        I.ok = I.n > 0 && I.n <= G * K;
        return wave_uniform(I);               // one module per wave (or per group of waves)
    };
    // A module larger than the group goes to the big-module list, or above BIG_RCAP
    // digis to the scratch-mode list (or, when that kernel is not launched, keeps
    // nothing and flags the size hint; with LF_DEFER it is listed all the same, for
    // the second launch).  Other units not clustered (absent modules,
    // entries not of this launch) keep nothing: the segmentation kernel cleared the
    // kept counts, without it this kernel does.
    auto skip = [&](const EventDesc& Ev, const Item& Is) {
        const EvLayout L = ev_layout(Ev.cap, a.n_modules);
        u32* ctl = ws_ptr<u32>(Ev, L.ctl);
        const bool scr = Is.n > BIG_RCAP;
        const bool listed = (a.flags & LF_DEFER) || !(a.flags & (scr ? (LF_NO_BIG | LF_NO_SCRATCH) : LF_NO_BIG));
        if (Is.n > G * K && listed) {
            const u32 r = atomicAdd(&ctl[scr ? CTL_SCR : CTL_BIG], 1u);
            if (r < a.n_modules) ws_ptr<u32>(Ev, scr ? L.scr : L.big)[r] = Is.mod;
            else atomicOr(&ctl[CTL_ERR], EB_INTERNAL);
            return;
        }
        if (Is.n > G * K) atomicOr(&ctl[CTL_ERR], EB_HINT);
        if (fused || Is.n > G * K) ws_ptr<u32>(Ev, L.kept)[Is.mod] = 0u;
    };

    // Modules are assigned statically in rounds (round r: module r*per_round + the
    // group's index) for about three quarters of the work, the rest by ticket.  The ticket of
    // the module after next is drawn while the current one is clustered, and the next
    // module's table entry (or range, by search) and digis are loaded meanwhile.
    // Draws from one counter are served one after another, ~15 ns each, and all groups draw
    // their first one together: with one counter for 1,280 groups every first module of a
    // 16-event launch took 20-30 us instead of 6-10.  So the groups and the modules left are
    // dealt out to one counter per event (each in its event's control words), with at least
    // 16 groups at each.  One event has one counter, used only from three static rounds on:
    // with fewer, what a draw costs is more than what it balances.
    const u32 per_round = gridDim.x * MPW;
    u32 base = xcd_order(blockIdx.x, gridDim.x) * MPW + (WAVE ? wave_uniform(g) : 0u);
    const u32 ofs = wave_uniform(gofs);
    const EventDesc* E = event_at(a, 0);
    Item I{0, 0, 0, 0, 0, false};
    u32 RC[K], A[K];
    if (base + ofs < total) {
        Next N{};
        step_module(base + ofs, N);
        step_range(N);
        I = step_item(N);
        E = N.E;
        if (I.ok) fetch_digis<G, K>(module_digis(*E, ev_layout(E->cap, a.n_modules), I.st), I.n, lt, RC, A);
    }
    if (fused) id_check_finish<WG>(a, get_event(a, 0), idc);
    // (units of a launch: at most MAXB * PXCL_MAX_MODULES, so three times that fits 32 bits)
    u32 nrounds = per_round < total ? max(1u, 3u * total / (4u * per_round)) : 1u;         // static
    if (k == 1 && nrounds < 3) nrounds = (total + per_round - 1) / per_round;              // all of them
    const u32 nstatic = nrounds * per_round;
    const u32 parts = k == 1 ? 1u : max(1u, min(k, gridDim.x * (WAVE ? MPW : 1u) / 16u)), part = base / STEP % parts;
    u32* tick = parts == 1 ? ticket(a) : ws_ptr<u32>(*event_at(a, part), 0) + CTL_CTR;   // ctl is at offset 0
    auto draw_ticket = [&]() { return nstatic + (atomicAdd(tick, 1u) * parts + part) * STEP; };
    const bool dyn = nstatic < total;             // tickets needed at all
    const bool drawer = WAVE ? lt == 0 : tid == 0;
    u32 round = 0;                                // round of the current module (>= nrounds: dynamic)
    u32 nv = total;                               // ticket of the next dynamic module (in flight)
    if (dyn && nrounds == 1) {
        if (drawer) nv = draw_ticket();
        if constexpr (!WAVE) {                    // every wave reads it at its first module's first stage
            if (tid == 0) s.tick = nv;
            lds_barrier();
        }
    }

    while (base < total) {
        u32 nbase = total, nv2 = total;
        Next N{};
        N.E = E;
        bool have = false;
        Item In{0, 0, 0, 0, 0, false};
        u32 NRC[K];
        auto mid = [&](int stage) {
            if (stage == 0) {
                const bool snext = round + 1 < nrounds;            // next module static
                const bool draw = dyn && round + 2 >= nrounds;     // module after next dynamic
                if (snext) nbase = base + per_round;
                else if (dyn) nbase = WAVE ? wave_uniform(nv) : wave_uniform(s.tick);
                if (draw && drawer && nbase < total) nv2 = draw_ticket();
                have = nbase + ofs < total;
                if (have) step_module(nbase + ofs, N);
            } else if (stage == 1) {
                if (have) step_range(N);
            } else {
                // the drawn ticket, for the stage 0 of the next module (barriers lie between)
                if constexpr (!WAVE)
                    if (tid == 0) s.tick = nv2;
                if (have) {
                    In = step_item(N);
                    if (In.ok) fetch_digis<G, K>(module_digis(*N.E, ev_layout(N.E->cap, a.n_modules), In.st), In.n, lt, NRC, A);
                }
            }
        };
        if (base + ofs < total && !I.ok && lt == 0) skip(*E, I);
        if (!WAVE || I.ok) {
            cluster_regs<G, K, MPW == 1>(a, *E, ev_layout(E->cap, a.n_modules), I, gp, lt, RC, A, mid);
        } else {
            mid(0);
            mid(1);
            mid(2);
        }
        base = nbase;
        E = N.E;
        I = In;
        nv = nv2;
        ++round;
#pragma unroll
        for (u32 q = 0; q < K; ++q) RC[q] = NRC[q];
    }
}

// ---------------------------------------------------------------------------
// big: one module per 1,024-thread workgroup
// ---------------------------------------------------------------------------
// Register mode: up to BIG_RCAP digis, K per thread of a 1,024-thread workgroup.  At such
// occupancies most work is per digi, and one workgroup has the compute unit to itself (the
// words of up to BIG_RCAP runs take 128 KB), so what bounds it is the instructions its
// sixteen waves issue: run parents and links come from the bitmap, a word of 32 rows at a
// time, trees are flattened per run, and a digi looks its run up in one column entry and
// one bitmap word and adds to its root.  186 modules of 13,312 digis: 58 -> 34 us (512
// threads of 32 digis, links listed and united one by one, before).
template <u32 G, u32 K>
struct DenseSmem {
    static constexpr u32 RCAP = G * K, KBW = RCAP / 32;
    u32 bm[BM_WORDS];  // fired-pixel bitmap (clear between modules)
    u64 col[COLS + 2]; // entry c+1: column c's run numbers
    u64 acc[RCAP];     // per run, as RegModuleSmem::acc
    u32 kb[KBW];       // kept-root bits over run index
    u16 kpre[KBW];     // kept roots before each kb word
    u32 wsum[G / 64];
};

// This thread's index, worked out anew for every module (the second term is zero): addresses
// that depend on the index alone would be computed before the loop over the modules, for
// both modes, and spilled (21 registers, reloaded from memory between LDS phases; 12 still are,
// with the 128 a lane that sixteen waves of one compute unit can have).
template <u32 WG>
__device__ __forceinline__ u32 thread_in_loop(const Item& I) {
    return (threadIdx.x + (I.n >> 31)) & (WG - 1u);
}

template <u32 G, u32 K>
__device__ __forceinline__ void cluster_dense(const LaunchArgs& a, const EventDesc& E, const EvLayout& L, const Item& I,
                                              DenseSmem<G, K>& s) {
    constexpr u32 KBW = G * K / 32;
    static_assert(G >= COLS && KBW <= G, "a thread per column, and per word of kept bits");
    static_assert(G * K <= 16384, "sizes of up to 15 bits, run numbers of up to 16");
    const u32 tid = thread_in_loop<G>(I), n = I.n, st = I.st;
    const u32 nq = min((n + G - 1) / G, K);
    const ModuleDigis D = module_digis(E, L, st);
    const bool hits = (E.flags & EF_HITS) != 0;
    u32 RC[K], A[K], X[K], valid = 0, err = 0, dup = 0;
    fetch_digis<G, K>(D, n, tid, RC, A);
    if (tid < KBW) s.kb[tid] = 0u;
#pragma unroll
    for (u32 q = 0; q < K; ++q)
        if (q < nq && tid + q * G < n) {
            const u32 row = RC[q] & 0xFFFFu, c = RC[q] >> 16, bit = 1u << (row & 31u);
            if (row < ROWS && c < COLS) {
                dup |= atomicOr(&s.bm[BM_FRONT + c * WPC + (row >> 5)], bit) & bit;
                valid |= 1u << q;
            } else {
                err |= EB_RANGE;
            }
        }
    if (dup) err |= EB_DUP;
    lds_barrier();
    u32 nruns;
    {
        u32 cnt = 0;
        u64 e = 0ull;
        if (tid < COLS) e = col_entry(s.bm, tid, cnt);
        const u32 run = group_excl_scan<G>(cnt, tid, s.wsum, nruns);
        if (tid < COLS) s.col[tid + 1] = e | run;
    }
    lds_barrier();
    for (u32 u = tid; u < WORDS; u += G)                       // first parents (rule B), sums zero
        word_parents(s.bm, s.col, u / WPC, u % WPC, [&](u32 run, u32 parent) { s.acc[run] = u64(parent) << 48; });
    lds_barrier();
    for (u32 u = tid; u < WORDS; u += G)                       // rule A
        word_links(s.bm, s.col, u / WPC, u % WPC, [&](u32 x, u32 y) { unite_packed(s.acc, x, y); });
    lds_barrier();
    // every run points at its root: a thread moves only its own runs' parents, each to an
    // ancestor, so what it stores last (the root) stands; others' moves double the steps
    for (u32 base = 0; base < nruns; base += 4 * G) {
        u32 x[4], more, it = 0;
#pragma unroll
        for (u32 u = 0; u < 4; ++u) x[u] = min(base + u * G + tid, nruns - 1);
        do {
            u32 p[4];
            more = 0;
#pragma unroll
            for (u32 u = 0; u < 4; ++u) p[u] = parent_of(s.acc, x[u]);
#pragma unroll
            for (u32 u = 0; u < 4; ++u) {
                more |= p[u] ^ x[u];
                x[u] = p[u];
                if (base + u * G + tid < nruns) st_wg(hi_word(s.acc, base + u * G + tid), p[u] << 16);
            }
        } while (more && ++it < MAX_RUNS);
    }
    lds_barrier();
#pragma unroll
    for (u32 q = 0; q < K; ++q)                                // roots, charge and size
        if (q < nq && ((valid >> q) & 1u)) {
            const u32 row = RC[q] & 0xFFFFu, c = RC[q] >> 16, k = row >> 5;
            X[q] = parent_of(s.acc, run_number(s.col[c + 1], k, s.bm[BM_FRONT + c * WPC + k], row));
        }
#pragma unroll
    for (u32 q = 0; q < K; ++q)
        if (q < nq && ((valid >> q) & 1u)) atomicAdd(&s.acc[X[q]], (1ull << 32) | u64(A[q]));
    lds_barrier();
    for (u32 u = tid; u < WORDS; u += G) {                     // cut; first pixel and size of the roots
        const ColWord x = col_word(s.bm, s.col, u / WPC, u % WPC);
        u32 m = x.st, r = x.r0;
        while (m) {
            const u32 b = __builtin_ctz(m);
            m &= m - 1u;
            const u64 v = s.acc[r];
            if (u32(v >> 48) == r) {
                if (u32(v) >= a.charge_cut) atomicOr(&s.kb[r >> 5], 1u << (r & 31u));
                st_wg(hi_word(s.acc, r), (((u << 5) + b) << 15) | (u32(v >> 32) & 0x7FFFu));
            }
            ++r;
        }
    }
    lds_barrier();
    u32 Kc;
    {
        const u32 cnt = tid < KBW ? __popc(s.kb[tid]) : 0u;
        const u32 pre = group_excl_scan<G>(cnt, tid, s.wsum, Kc);
        if (tid < KBW) s.kpre[tid] = u16(pre);
    }
    lds_barrier();
    if (tid == 0) ws_ptr<u32>(E, L.kept)[I.it] = Kc;
    const u32 idbase = I.mod * PIX;
    // f(root, position) for the kept clusters
    auto kept_roots = [&](auto f) {
        for (u32 r = tid; r < nruns; r += G) {
            const u32 w = s.kb[r >> 5], bit = 1u << (r & 31u);
            if (w & bit) f(r, st + u32(s.kpre[r >> 5]) + __popc(w & (bit - 1u)));
        }
    };
    {
        int32_t* tid_ = ws_ptr<int32_t>(E, L.tid);
        int32_t* tch = ws_ptr<int32_t>(E, L.tcharge);
        int32_t* tsz = ws_ptr<int32_t>(E, L.tsize);
        kept_roots([&](u32 r, u32 p) {
            const u64 v = s.acc[r];
            tid_[p] = int32_t(idbase + u32(v >> 47));
            tch[p] = int32_t(u32(v));
            tsz[p] = int32_t(u32(v >> 32) & 0x7FFFu);
        });
    }
    int32_t* od = (int32_t*)E.o_digi;
    u32 keep = 0;
#pragma unroll
    for (u32 q = 0; q < K; ++q) {
        const u32 j = tid + q * G;
        if (q < nq && j < n) {
            int32_t id = -1;
            if ((valid >> q) & 1u) {
                const u64 v = s.acc[X[q]];
                if (u32(v) >= a.charge_cut) {
                    id = int32_t(idbase + u32(v >> 47));
                    keep |= 1u << q;
                }
            }
            od[D.pos(j)] = id;
        }
    }
    for (u32 w = tid; w < WORDS; w += G) s.bm[BM_FRONT + w] = 0u;
    if (err) atomicOr(ws_ptr<u32>(E, L.ctl) + CTL_ERR, err);
    lds_barrier();
    if (hits) {                                                // exact sums in LDS, columns, then rows
        u64* hs = ws_ptr<u64>(E, L.hsum);
        for (u32 axis = 0; axis < 2; ++axis) {
            kept_roots([&](u32 r, u32) { s.acc[r] = 0ull; });
            lds_barrier();
#pragma unroll
            for (u32 q = 0; q < K; ++q)
                if (q < nq && ((keep >> q) & 1u))
                    atomicAdd(&s.acc[X[q]], u64(A[q]) * (axis ? RC[q] & 0xFFFFu : RC[q] >> 16));
            lds_barrier();
            kept_roots([&](u32 r, u32 p) { hs[2 * p + axis] = s.acc[r]; });
            lds_barrier();
        }
    }
}

// Scratch mode (more than BIG_RCAP digis).  Connectivity is computed on the bitmap
// alone, with the parents of up to MAX_RUNS runs in LDS: every run starts under its rule B
// run (a chain along the columns, at most COLS long), pointer doubling flattens the chains,
// and only rule A's links need unions.  The roots, in run order (= order of their smallest
// linear index), number the clusters.  Three passes over the digis: bitmap; charge and
// size (LDS sums of the first LCAP clusters, device atomics into the module's slice of the
// event's final charge/size arrays, which the compaction kernel overwrites later, for the
// rest), leaving each digi's cluster in its output word; per-digi ids from that.  The passes
// take four digis per load and test the ranges of four at once.  Like register mode it is
// bound by the instructions of one workgroup: a serpentine alone in the launch 159 -> 71 us
// along rows, 49 us along columns (before: unions column by column, a lane per row, 60-85 us of
// it; one digi per load; runs looked up again for the ids).
template <u32 BW>
struct BigScratchSmem {
    u32 bm[BM_WORDS];
    alignas(8) u32 par[MAX_RUNS];   // its second half later holds 64-bit sums
    u32 rootb[MAX_RUNS / 32];   // root runs, then kept clusters (over cluster index)
    u64 col[COLS + 2];          // entry c+1: column c's run numbers
    u16 rootp[MAX_RUNS / 32];   // roots before each word, then kept clusters before each word
    u16 src[WPC * COLS];        // word k of column c: leftmost column of its stretch of like words
    u32 wsum[BW / 64];
};

constexpr u32 UNR = 4;                        // groups of 4 digis per thread fetched at once

// Four consecutive 16-bit values at any 2-byte address as one 8-byte load, four 32-bit
// ones at any 4-byte address as one 16-byte access (global memory takes both unaligned).
struct __attribute__((packed, aligned(2))) U16x4 {
    u64 v;
};
struct __attribute__((packed, aligned(4))) I32x4 {
    int32_t v[4];
};
__device__ __forceinline__ u64 load4(const u16* p) { return reinterpret_cast<const U16x4*>(p)->v; }
__device__ __forceinline__ u32 part(u64 v, u32 i) { return u32(v >> (16 * i)) & 0xFFFFu; }
// Some of the four values is `limit` (at most 2^15) or more.
__device__ __forceinline__ bool any_at_least(u64 v, u32 limit) {
    return ((v | (v + u64(0x8000u - limit) * 0x0001000100010001ull)) & 0x8000800080008000ull) != 0ull;
}

// Add `val` to base[key] for every lane with `valid`; one atomic per wave when all
// valid lanes share the key.  Called by all lanes of the wave.
template <typename T>
__device__ __forceinline__ void wave_add(T* base, u32 key, T val, bool valid) {
    const u64 vm = __ballot(valid);
    if (!vm) return;
    const u32 first = __ffsll((unsigned long long)vm) - 1;
    const u32 lead = __shfl(key, first, 64);
    const u64 same = __ballot(valid && key == lead);
    if (same == vm) {
        T sum = valid ? val : T(0);
#pragma unroll
        for (u32 d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
        if ((threadIdx.x & 63u) == first) atomicAdd(&base[lead], sum);
    } else if (valid) {
        atomicAdd(&base[key], val);
    }
}

template <u32 BW>
__device__ __forceinline__ void cluster_scratch(const LaunchArgs& a, const EventDesc& E, const EvLayout& L,
                                                const Item& I, BigScratchSmem<BW>& s) {
    constexpr u32 KW = MAX_RUNS / 32, KPT = (KW + BW - 1) / BW;
    constexpr u32 SPAN = 4 * UNR * BW;                     // digis per step
    static_assert(BW >= COLS, "a thread per column");
    const u32 tid = thread_in_loop<BW>(I), n = I.n, st = I.st;
    u32* cid = (u32*)E.o_id + st;       // per cluster: id (or -1 once cut)
    u32* cch = (u32*)E.o_charge + st;   // per cluster: charge
    u32* csz = (u32*)E.o_size + st;     // per cluster: size
    int32_t* od = (int32_t*)E.o_digi;
    const ModuleDigis D = module_digis(E, L, st);
    const bool hits = (E.flags & EF_HITS) != 0;
    u64* hs = ws_ptr<u64>(E, L.hsum);
    u32 err = 0;
    const u32 wv = tid >> 6, lane = tid & 63u;
    // A step: this thread's digis base + 4 * (u * BW + tid) + 0..3, u < UNR; quads past the
    // module's end are passed over by the whole workgroup.
    auto first_of = [&](u32 base, u32 u) { return base + 4u * (u * BW + tid); };
    auto some = [&](u32 base, u32 u) { return base + 4u * u * BW < n; };
    auto quad = [&](const u16* p, u32 base, u32 u) -> u64 {
        const u32 first = first_of(base, u);
        if (base + 4u * (u + 1) * BW <= n) return load4(p + first);
        u64 v = 0ull;
        for (u32 i = 0; i < 4; ++i)
            if (first + i < n) v |= u64(p[first + i]) << (16 * i);
        return v;
    };
    auto load = [&](u32 base, u32 u, u64& r, u64& c, u64* w) {     // rows, columns and, with w, adcs
        if (!D.rec) {
            r = quad(D.row, base, u);
            c = quad(D.col, base, u);
            if (w) *w = quad(D.adc, base, u);
            return;
        }
        const u32 first = first_of(base, u);
        u64 v[4];
        for (u32 i = 0; i < 4; ++i) v[i] = first + i < n ? D.rec[first + i] : 0ull;
        r = c = 0ull;
        if (w) *w = 0ull;
        for (u32 i = 0; i < 4; ++i) {
            const u32 rc = ModuleDigis::rc_of(v[i]);
            r |= u64(rc & 0xFFFFu) << (16 * i);
            c |= u64(rc >> 16) << (16 * i);
            if (w) *w |= (v[i] & 0xFFFFu) << (16 * i);
        }
    };
    // the wave's quads hold four pixels each (else each digi is looked at by itself)
    auto whole = [&](u32 base, u32 u, u64 r, u64 c) {
        return __ballot(first_of(base, u) + 4 > n || any_at_least(r, ROWS) || any_at_least(c, COLS)) == 0ull;
    };
    auto pixel = [&](u32 j, u32 row, u32 col) { return j < n && row < ROWS && col < COLS; };
    auto word_of = [&](u32 row, u32 col) { return BM_FRONT + col * WPC + (row >> 5); };
    auto cluster_of = [&](u32 run) {                      // of a flattened run (par[run] is its root)
        const u32 root = ld_wg(&s.par[run]);
        return u32(s.rootp[root >> 5]) + __popc(s.rootb[root >> 5] & ((1u << (root & 31u)) - 1u));
    };
    for (u32 base = 0; base < n; base += SPAN) {               // pass 1: bitmap
        u64 r[UNR], c[UNR];
#pragma unroll
        for (u32 u = 0; u < UNR; ++u)
            if (some(base, u)) load(base, u, r[u], c[u], nullptr);
        u32 dup = 0;
#pragma unroll
        for (u32 u = 0; u < UNR; ++u) {
            if (!some(base, u)) continue;
            const bool all = whole(base, u, r[u], c[u]);
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
                const u32 row = part(r[u], i), col = part(c[u], i), bit = 1u << (row & 31u);
                if (all || pixel(first_of(base, u) + i, row, col)) dup |= atomicOr(&s.bm[word_of(row, col)], bit) & bit;
                else if (first_of(base, u) + i < n) err |= EB_RANGE;
            }
        }
        if (dup) err |= EB_DUP;
    }
    lds_barrier();
    u32 nruns;
    {                                                           // runs
        u32 cnt = 0;
        u64 e = 0ull;
        if (tid < COLS) e = col_entry(s.bm, tid, cnt);
        const u32 run = group_excl_scan<BW>(cnt, tid, s.wsum, nruns);
        if (tid < COLS) s.col[tid + 1] = e | run;
    }
    lds_barrier();
    // Stretches of columns that hold the same 32 rows (and the same bit above them): their run
    // starts are the same too, and the runs that start at one row touch from column to column,
    // so each starts under the stretch's first one instead of its left neighbour.  A wave per
    // row of words, 1.3 us.  Chains along rows are as long as the module: 80 of them (a
    // serpentine along rows) took 24 us to flatten, now 17.
    for (u32 k = wv; k < WPC; k += BW / 64) {
        u32 carry = 0;
#pragma unroll
        for (u32 g = 0; g < (COLS + 63) / 64; ++g) {
            const u32 c = g * 64 + lane, cc = min(c, COLS - 1);
            const u32* w = &s.bm[BM_FRONT + cc * WPC + k];
            const u32 b = w[0], l = *(w - WPC), ab = k ? *(w - 1) >> 31 : 0u, al = k ? *(w - 1 - WPC) >> 31 : 0u;
            const u64 m = __ballot(c == 0 || b == 0u || b != l || ab != al ? 1 : 0), upto = m & ((2ull << lane) - 1ull);
            const u32 first = upto ? g * 64 + 63u - u32(__builtin_clzll(upto)) : carry;
            if (c < COLS) s.src[k * COLS + c] = u16(first);
            carry = m ? g * 64 + 63u - u32(__builtin_clzll(m)) : carry;
        }
    }
    lds_barrier();
    for (u32 u = tid; u < WORDS; u += BW) {                     // first parents
        const u32 c = u / WPC, k = u % WPC, src = s.src[k * COLS + c];
        if (src == c) {
            word_parents(s.bm, s.col, c, k, [&](u32 run, u32 parent) { st_wg(&s.par[run], parent); });
        } else {
            const ColWord x = col_word(s.bm, s.col, c, k);
            const u32 n_st = u32(__popc(x.st)), r0 = runs_before(s.col[src + 1], k) + (x.b & (x.above >> 31));
            for (u32 i = 0; i < n_st; ++i) st_wg(&s.par[x.r0 + i], r0 + i);
        }
    }
    lds_barrier();
    // Every run points at its root.  A thread moves only its own runs' parents, each to an
    // ancestor, so what it stores last (the root) stands; others' moves double the steps.
    // `last`: one bit per root too.
    auto flatten = [&](bool last) {
        constexpr u32 F = 4;
        for (u32 base = 0; base < nruns; base += F * BW) {
            u32 x[F], more;
#pragma unroll
            for (u32 u = 0; u < F; ++u) x[u] = min(base + u * BW + tid, nruns - 1);
            u32 it = 0;
            do {
                u32 p[F];
                more = 0;
#pragma unroll
                for (u32 u = 0; u < F; ++u) p[u] = ld_wg(&s.par[x[u]]);
#pragma unroll
                for (u32 u = 0; u < F; ++u) {
                    more |= p[u] ^ x[u];
                    x[u] = p[u];
                    if (base + u * BW + tid < nruns) st_wg(&s.par[base + u * BW + tid], p[u]);
                }
            } while (more && ++it < MAX_RUNS);
            if (last) {
#pragma unroll
                for (u32 u = 0; u < F; ++u) {
                    const u32 r = base + u * BW + tid;
                    const u64 m = __ballot(r < nruns && x[u] == r ? 1 : 0);
                    if (lane == 0 && r < nruns) {
                        s.rootb[r >> 5] = u32(m);
                        s.rootb[(r >> 5) + 1] = u32(m >> 32);
                    }
                }
            }
        }
        lds_barrier();
    };
    for (u32 w = tid; w < KW; w += BW) s.rootb[w] = 0u;
    flatten(false);
    for (u32 u = tid; u < WORDS; u += BW)                       // rule A
        word_links(s.bm, s.col, u / WPC, u % WPC, [&](u32 x, u32 y) { uf_unite(s.par, x, y); });
    lds_barrier();
    // the roots number the clusters in order of their smallest index
    flatten(true);
    u32 ncl;
    {
        u32 sw[KPT], cnt = 0;
#pragma unroll
        for (u32 i = 0; i < KPT; ++i) {
            const u32 w = tid * KPT + i;
            sw[i] = w < KW ? __popc(s.rootb[w]) : 0u;
            cnt += sw[i];
        }
        u32 run = group_excl_scan<BW>(cnt, tid, s.wsum, ncl);
#pragma unroll
        for (u32 i = 0; i < KPT; ++i) {
            const u32 w = tid * KPT + i;
            if (w < KW) s.rootp[w] = u16(run);
            run += sw[i];
        }
    }
    lds_barrier();
    // Every run's cluster as a u16 over the first half of the parents (each thread reads
    // its RPT consecutive runs before any is written); the second half then holds the
    // first LCAP clusters' charge | size << 44 (LDS atomics), the others' sums go to
    // device memory.
    constexpr u32 RPT = (MAX_RUNS + BW - 1) / BW, LCAP = MAX_RUNS * 2 / 8;
    static_assert((offsetof(BigScratchSmem<BW>, par) + size_t(MAX_RUNS) * 2) % 8 == 0, "64-bit LDS atomics need 8-byte alignment");
    u16* cl = reinterpret_cast<u16*>(s.par);
    u64* acc = reinterpret_cast<u64*>(reinterpret_cast<u8*>(s.par) + size_t(MAX_RUNS) * 2);
    {
        u32 cv[(RPT + 1) / 2];
#pragma unroll
        for (u32 i = 0; i < RPT; ++i) {
            const u32 r = tid * RPT + i;
            const u32 c = r < nruns ? cluster_of(r) : 0u;
            if (i & 1u) cv[i / 2] |= c << 16;
            else cv[i / 2] = c;
        }
        lds_barrier();
#pragma unroll
        for (u32 i = 0; i < RPT; ++i) {
            const u32 r = tid * RPT + i;
            if (r < nruns) cl[r] = u16(cv[i / 2] >> (16 * (i & 1u)));
        }
    }
    lds_barrier();
    // per cluster: id from the start of its root run; zero the sums
    for (u32 c = tid; c < min(ncl, LCAP); c += BW) acc[c] = 0ull;
    for (u32 u = tid; u < WORDS; u += BW) {
        const ColWord x = col_word(s.bm, s.col, u / WPC, u % WPC);
        u32 m = x.st, r = x.r0;
        while (m) {
            const u32 b = __builtin_ctz(m);
            m &= m - 1u;
            if (s.rootb[r >> 5] & (1u << (r & 31u))) {
                const u32 c = u32(s.rootp[r >> 5]) + __popc(s.rootb[r >> 5] & ((1u << (r & 31u)) - 1u));
                cid[c] = I.mod * PIX + (u << 5) + b;
                if (c >= LCAP) {
                    cch[c] = 0u;
                    csz[c] = 0u;
                }
            }
            ++r;
        }
    }
    wait_all_mem();
    lds_barrier();
    // Digi outputs at their own positions, and every cluster's sums in LDS: the usual case,
    // taken by the whole workgroup.
    const bool plain = !D.rec && ncl <= LCAP;
    auto cluster_at = [&](u32 row, u32 col) {
        return u32(cl[run_number(s.col[col + 1], row >> 5, s.bm[word_of(row, col)], row)]);
    };
    // A thread whose four digis belong to one cluster adds them to a running sum, which it
    // hands on when the cluster changes; of the last ones a wave whose threads all hold the
    // same cluster (a serpentine) makes one atomic.
    u32 run_c = 0;
    u64 run_sum = 0;
    for (u32 base = 0; base < n; base += SPAN) {               // pass 2: charge and size
        u64 r[UNR], c[UNR], w[UNR];
#pragma unroll
        for (u32 u = 0; u < UNR; ++u)
            if (some(base, u)) load(base, u, r[u], c[u], &w[u]);
#pragma unroll
        for (u32 u = 0; u < UNR; ++u) {
            if (!some(base, u)) continue;
            const u32 j = first_of(base, u);
            if (plain && whole(base, u, r[u], c[u])) {
                I32x4 cc;
                u32 sum = 0;
                bool one = true;
#pragma unroll
                for (u32 i = 0; i < 4; ++i) {
                    cc.v[i] = int32_t(cluster_at(part(r[u], i), part(c[u], i)));
                    one = one && cc.v[i] == cc.v[0];
                    sum += part(w[u], i);
                }
                *reinterpret_cast<I32x4*>(od + st + j) = cc;    // for pass 3
                if (one) {
                    if (u32(cc.v[0]) != run_c) {
                        if (run_sum) atomicAdd(&acc[run_c], run_sum);
                        run_c = u32(cc.v[0]);
                        run_sum = 0;
                    }
                    run_sum += (4ull << 44) | sum;
                } else {
#pragma unroll
                    for (u32 i = 0; i < 4; ++i) atomicAdd(&acc[cc.v[i]], (1ull << 44) | u64(part(w[u], i)));
                }
                continue;
            }
#pragma unroll 1
            for (u32 i = 0; i < 4; ++i) {
                const u32 row = part(r[u], i), col = part(c[u], i), x = part(w[u], i);
                const bool v = pixel(j + i, row, col);
                const u32 k = v ? cluster_at(row, col) : 0u;
                if (j + i < n) od[D.pos(j + i)] = v ? int32_t(k) : -1;
                wave_add<u64>(acc, k, (1ull << 44) | u64(x), v && k < LCAP);
                wave_add<u32>(cch, k, x, v && k >= LCAP);
                wave_add<u32>(csz, k, 1u, v && k >= LCAP);
            }
        }
    }
    wave_add<u64>(acc, run_c, run_sum, run_sum != 0);
    wait_all_mem();
    lds_barrier();
    // cut, one bit per kept cluster (64 at a time by ballot, so that lanes touch
    // consecutive words); kept clusters -> staging records in cluster (= ascending id) order
    for (u32 base = wv * 64; base < KW * 32; base += BW) {
        const u32 c = base + lane;
        u64 m = 0ull;
        if (base < ncl) m = __ballot(c < ncl && (c < LCAP ? u32(acc[c]) : ld_ag(&cch[c])) >= a.charge_cut ? 1 : 0);
        if (lane == 0) {
            s.rootb[base >> 5] = u32(m);
            s.rootb[(base >> 5) + 1] = u32(m >> 32);
        }
    }
    lds_barrier();
    u32 Kc;
    {
        u32 sw[KPT], cnt = 0;
#pragma unroll
        for (u32 i = 0; i < KPT; ++i) {
            const u32 w = tid * KPT + i;
            sw[i] = w < KW ? __popc(s.rootb[w]) : 0u;
            cnt += sw[i];
        }
        u32 run = group_excl_scan<BW>(cnt, tid, s.wsum, Kc);
        u32 keep_pre[KPT];
#pragma unroll
        for (u32 i = 0; i < KPT; ++i) {
            keep_pre[i] = run;
            run += sw[i];
        }
        int32_t* tid_ = ws_ptr<int32_t>(E, L.tid);
        int32_t* tch = ws_ptr<int32_t>(E, L.tcharge);
        int32_t* tsz = ws_ptr<int32_t>(E, L.tsize);
#pragma unroll
        for (u32 i = 0; i < KPT; ++i) {
            const u32 w = tid * KPT + i;
            if (w >= KW) continue;
            u32 pos = keep_pre[i];
            s.rootp[w] = u16(pos);                              // kept clusters before word w
            for (u32 b = 0; b < 32; ++b) {
                const u32 c = w * 32 + b;
                if (c >= ncl) break;
                const bool lds = c < LCAP;
                if (s.rootb[w] & (1u << b)) {
                    const u32 id = ld_ag(&cid[c]);
                    const u64 v = lds ? acc[c] : 0ull;
                    tid_[st + pos] = int32_t(id);
                    tch[st + pos] = int32_t(lds ? u32(v) : ld_ag(&cch[c]));
                    tsz[st + pos] = int32_t(lds ? u32(v >> 44) : ld_ag(&csz[c]));
                    ++pos;
                    if (lds) acc[c] = u64(id);                  // for the per-digi ids
                } else {
                    if (lds) acc[c] = u64(NOPIX);
                    st_ag(&cid[c], NOPIX);
                }
            }
        }
        if (tid == 0) ws_ptr<u32>(E, L.kept)[I.it] = Kc;
    }
    wait_all_mem();
    lds_barrier();
    if (hits) {
        // Weighted coordinates of the kept clusters: columns, then rows, in the LDS sums (the
        // records' device sums take them whole), those of clusters beyond them by device
        // atomics.  One device atomic per digi took 1.25 ms for a 33,423-pixel serpentine.
        for (u32 axis = 0; axis < 2; ++axis) {
            for (u32 c = tid; c < min(ncl, LCAP); c += BW) acc[c] = 0ull;
            lds_barrier();
            for (u32 j0 = 0; j0 < n; j0 += BW) {
                const u32 j = j0 + tid;
                const int32_t k = j < n ? od[D.pos(j)] : -1;
                const u64 x = k >= 0 ? u64(D.adc_at(j)) * (axis ? D.rc(j) & 0xFFFFu : D.rc(j) >> 16) : 0ull;
                const u32 c = k >= 0 ? u32(k) : 0u;
                const bool kept = k >= 0 && ((s.rootb[c >> 5] >> (c & 31u)) & 1u);
                wave_add<u64>(acc, c, x, kept && c < LCAP);
                if (kept && c >= LCAP) atomicAdd(&hs[2 * (st + s.rootp[c >> 5] + __popc(s.rootb[c >> 5] & ((1u << (c & 31u)) - 1u))) + axis], x);
            }
            lds_barrier();
            for (u32 c = tid; c < min(ncl, LCAP); c += BW)
                if ((s.rootb[c >> 5] >> (c & 31u)) & 1u)
                    hs[2 * (st + s.rootp[c >> 5] + __popc(s.rootb[c >> 5] & ((1u << (c & 31u)) - 1u))) + axis] = acc[c];
            lds_barrier();
        }
        for (u32 c = tid; c < min(ncl, LCAP); c += BW) acc[c] = u64(ld_ag(&cid[c]));
        lds_barrier();
    }
    for (u32 base = 0; base < n; base += SPAN) {               // pass 3: per-digi ids
#pragma unroll
        for (u32 u = 0; u < UNR; ++u) {                         // over what this thread left in pass 2
            if (!some(base, u)) continue;
            const u32 j = first_of(base, u);
            if (plain && __ballot(j + 4 > n) == 0ull) {
                I32x4 cc = *reinterpret_cast<const I32x4*>(od + st + j);
#pragma unroll
                for (u32 i = 0; i < 4; ++i) cc.v[i] = cc.v[i] >= 0 ? int32_t(u32(acc[cc.v[i]])) : -1;
                *reinterpret_cast<I32x4*>(od + st + j) = cc;
                continue;
            }
#pragma unroll 1
            for (u32 i = 0; i < 4; ++i) {
                if (j + i >= n) continue;
                const u32 q = D.pos(j + i);
                const int32_t k = od[q];
                if (k >= 0) od[q] = int32_t(u32(k) < LCAP ? u32(acc[k]) : ld_ag(&cid[k]));
            }
        }
    }
    if (err) atomicOr(ws_ptr<u32>(E, L.ctl) + CTL_ERR, err);
    lds_barrier();                                              // every thread is done with the bitmap
    for (u32 w = tid; w < WORDS; w += BW) s.bm[BM_FRONT + w] = 0u;
    lds_barrier();
}

// Entry t of the launch's big-module (or scratch-mode) lists (prefix s_pref): the
// module and its digis; ok when it is one the small kernel listed (above its
// capacity).
__device__ __forceinline__ Item big_item(const LaunchArgs& a, const u32* s_pref, u32 k, u32 t, bool scr) {
    Item I{0, 0, 0, 0, 0, false};
    I.e = find_slot(s_pref, k, t);
    const EventDesc E = get_event(a, I.e);
    const EvLayout L = ev_layout(E.cap, a.n_modules);
    I.mod = I.it = ws_ptr<const u32>(E, scr ? L.scr : L.big)[t - s_pref[I.e]];
    if (I.mod < a.n_modules) {
        const ModRange r = ws_ptr<const ModRange>(E, L.mtab)[I.mod];
        const u32 st = u32(r.first), en = u32(r.end);
        if (u32(r.first >> 32) == E.epoch && u32(r.end >> 32) == E.epoch && st < en && en <= E.n) {
            I.st = st;
            I.n = en - st;
            I.ok = scr ? I.n > BIG_RCAP : (I.n > a.dcap && I.n <= BIG_RCAP);
        }
    }
    if (!I.ok && threadIdx.x == 0) atomicOr(ws_ptr<u32>(E, L.ctl) + CTL_ERR, EB_INTERNAL);
    return I;
}

// Both modes in one launch: the modules of the scratch-mode list (above BIG_RCAP digis), which
// take longest, then those of the big-module list.  A workgroup's first module is given by its
// index, the others by ticket, so a workgroup busy with a scratch-mode module takes no more
// than that while the rest share the others.  16 events with a serpentine and 16-20 modules
// of 2,049 to 13,312 digis each: 92 us, where a launch per mode took 57 + 82 with the same code
// for the modules (118 us with tickets drawn when a module starts: those of the scratch-mode
// workgroups waited with them), 81 us since; launched for no module at all it costs one launch
// instead of two.
static_assert(B_WG == S_WG, "the modes share the workgroup");
__global__ __launch_bounds__(B_WG) void k_big(LaunchArgs a) {
    __shared__ union {
        DenseSmem<B_WG, K_BIG> d;
        BigScratchSmem<S_WG> x;
    } s;                                      // both start with the bitmap, clear between modules
    __shared__ u32 s_pref[MAXB + 1], s_xpref[MAXB + 1];
    __shared__ u32 s_wsum[B_WG / 64];
    __shared__ u32 s_tick;
    const u32 tid = threadIdx.x, k = num_events(a);
    if (k == 1) {                             // nothing listed for a single event: nothing else to set up
        const EventDesc& E = *event_at(a, 0);
        const u32* ctl = ws_ptr<const u32>(E, 0);
        if (!E.n || (ld_ag(ctl + CTL_SCR) | ld_ag(ctl + CTL_BIG)) == 0u) return;
    }
    for (u32 w = tid; w < BM_WORDS; w += B_WG) s.d.bm[w] = 0u;
    const u32 xtotal = event_prefix<B_WG>(a, k, s_xpref, s_wsum, CTL_SCR, 1, 0);
    const u32 total = xtotal + event_prefix<B_WG>(a, k, s_pref, s_wsum, CTL_BIG, 1, 0);
    for (u32 t = blockIdx.x; t < total;) {
        const bool scr = t < xtotal;
        const Item I = wave_uniform(big_item(a, scr ? s_xpref : s_pref, k, scr ? t : t - xtotal, scr));
        if (I.ok) {                           // the same for the whole workgroup
            const EventDesc& E = *event_at(a, I.e);
            const EvLayout L = ev_layout(E.cap, a.n_modules);
            if (scr) cluster_scratch<S_WG>(a, E, L, I, s.x);
            else cluster_dense<B_WG, K_BIG>(a, E, L, I, s.d);
        }
        if (total <= gridDim.x) break;
        if (tid == 0) s_tick = atomicAdd((u32*)(a.ctr + S_BIG), 1u) + gridDim.x;   // not before: it would wait with us
        lds_barrier();
        t = wave_uniform(s_tick);
        lds_barrier();                        // read by every wave before the next draw is stored
    }
}

// ---------------------------------------------------------------------------
// compact: S waves per block of C_BLK consecutive modules of an event (every module,
// present or not: an absent module keeps nothing).  The block's first output
// position is the sum of the kept counts of the modules before it, which each of its
// waves adds up (PS_UNR loads per lane in flight); a wave scan over the block's 64
// counts gives every module its position, and wave s of the block copies the s-th
// of S equal shares of the block's records, 64 at a time, each lane finding its
// record's module by a search over that scan.  S (a power of two, at most C_SPLIT)
// follows from the grid: launches of few blocks (one event of few modules) spread
// each block's copy over many waves, launches of many blocks keep one wave per
// block.  Wave 0 of an event's last block has the event's total and writes the
// status back to the host.  Loads per event grow as (modules / 64)^2 * 64 * S.
// ---------------------------------------------------------------------------
constexpr u32 CP_UNR = 4, PS_UNR = 16, C_WAVES = C_WG / 64, C_BLK = 64, C_SPLIT = 32;

__device__ __forceinline__ u32 compact_blocks(u32 n_modules) { return (n_modules + C_BLK - 1) / C_BLK; }

// Waves per block for a launch of `waves` waves over `blocks` blocks.
__host__ __device__ __forceinline__ u32 compact_split(u32 waves, u32 blocks) {
    u32 sp = 1;
    while (sp < C_SPLIT && u64(sp) * 2 * blocks <= waves) sp *= 2;
    return sp;
}

// Sum of kept[0, end) over the wave (end a multiple of 64).
__device__ __forceinline__ u32 kept_before(const u32* kept, u32 end, u32 lane) {
    u32 part = 0;
    for (u32 b = 0; b < end; b += 64 * PS_UNR) {
        u32 v[PS_UNR];
#pragma unroll
        for (u32 q = 0; q < PS_UNR; ++q) {
            const u32 i = b + q * 64 + lane;
            v[q] = i < end ? kept[i] : 0u;
        }
#pragma unroll
        for (u32 q = 0; q < PS_UNR; ++q) part += v[q];
    }
    return __shfl(wave_incl_scan(part), 63, 64);
}

__global__ __launch_bounds__(C_WG) void k_compact(LaunchArgs a) {
    const u32 tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
    const u32 k = num_events(a), M = a.n_modules, nblk = compact_blocks(M);
    if (blockIdx.x == 0 && tid == 0) reset_tickets(a);            // the kernels that draw them have finished
    const u32 sp = compact_split(gridDim.x * C_WAVES, k * nblk);
    const u32 total = k * nblk * sp;
    for (u32 u = wave_uniform(xcd_order(blockIdx.x, gridDim.x) * C_WAVES + wv); u < total; u += gridDim.x * C_WAVES) {
        const u32 eb = u / sp, part = u - eb * sp;
        const u32 e = eb / nblk, b = eb - e * nblk;
        const EventDesc E = wave_uniform(get_event(a, e));
        const EvLayout L = ev_layout(E.cap, M);
        u32* ctl = ws_ptr<u32>(E, L.ctl);
        const u32* kept = ws_ptr<const u32>(E, L.kept);
        // the module totals of digis in any order are zero between launches
        if ((E.flags & EF_UNSORTED) && part == 0 && b * C_BLK + lane < M) ws_ptr<u32>(E, L.gcnt)[b * C_BLK + lane] = 0u;
        if ((a.flags & LF_DEFER) && (ld_ag(ctl + CTL_BIG) | ld_ag(ctl + CTL_SCR)) != 0u) {
            // modules wait for the big-module kernels of a second launch: nothing is
            // compacted, the lists and error bits stay for it, the host learns why
            if (b + 1 == nblk && part == 0 && lane == 0) {
                ctl[CTL_DEFERRED] = 1u;
                ctl[CTL_CTR] = 0u;
                u32* hs = (u32*)E.hstat;
                st_sys(&hs[HS_ERR], ctl[CTL_ERR] | EB_DEFER);
                st_sys(&hs[HS_NCL], 0u);
                st_sys(&hs[HS_EPOCH], E.epoch);
            }
            continue;
        }
        if ((a.flags & LF_SECOND) && ld_ag(ctl + CTL_DEFERRED) == 0u) continue;   // finished by the first launch
        const u32 m = b * C_BLK + lane;
        // an empty event's kept counts were never written: it has no clusters
        const bool live = E.n != 0 && m < M;
        u32 cnt = live ? kept[m] : 0u;
        const u32 src = live ? u32(ws_ptr<const ModRange>(E, L.mtab)[m].first) : 0u;
        const u32 base = E.n ? wave_uniform(kept_before(kept, b * C_BLK, lane)) : 0u;
        if (cnt > E.n) cnt = 0u;                           // inconsistent (only after an input error)
        const u32 incl = wave_incl_scan(cnt), excl = incl - cnt;
        const u32 T = wave_uniform(__shfl(incl, 63, 64));
        const bool fits = base <= E.n && T <= E.n - base;  // every position below n
        if (b + 1 == nblk && part == 0 && lane == 0) {     // the event's status
            const u32 ncl = fits ? base + T : E.n;
            const u32 err = ctl[CTL_ERR];
            ctl[CTL_ERR] = 0u;
            ctl[CTL_CTR] = 0u;
            // an empty event has no segmentation, which clears this for the next launch
            if (!E.n) ctl[CTL_PRESENT + ((E.slot & 1u) ^ 1u)] = 0u;
            st_ag(ctl + CTL_BIG, 0u);                      // the big kernels have run (other waves
            st_ag(ctl + CTL_SCR, 0u);                      // of the event may read them atomically)
            ctl[CTL_NCL] = ncl;
            u32* hs = (u32*)E.hstat;
            st_sys(&hs[HS_ERR], err);
            st_sys(&hs[HS_NCL], ncl);
            st_sys(&hs[HS_EPOCH], E.epoch);
        }
        if (!fits || T == 0) continue;
        if (cnt && part == 0) ws_ptr<u32>(E, L.off)[m] = base + excl;
        const bool src_ok = cnt == 0 || src <= E.n - cnt;
        const int32_t* tid_ = ws_ptr<const int32_t>(E, L.tid);
        const int32_t* tch = ws_ptr<const int32_t>(E, L.tcharge);
        const int32_t* tsz = ws_ptr<const int32_t>(E, L.tsize);
        int32_t* oid = (int32_t*)E.o_id;
        int32_t* och = (int32_t*)E.o_charge;
        int32_t* osz = (int32_t*)E.o_size;
        const bool hits = (E.flags & EF_HITS) != 0;
        u64* hsm = ws_ptr<u64>(E, L.hsum);
        float* hx = ws_ptr<float>(E, L.hit_x);
        float* hy = ws_ptr<float>(E, L.hit_y);
        const u32 mod_src = src_ok ? src : NOPIX;          // a record of a bad module is skipped
        const u32 j_lo = u32(u64(T) * part / sp), j_hi = u32(u64(T) * (part + 1) / sp);
        for (u32 j0 = j_lo; j0 < j_hi; j0 += 64 * CP_UNR) {
            int32_t r0[CP_UNR], r1[CP_UNR], r2[CP_UNR];
            u64 sx[CP_UNR], sy[CP_UNR];
            u32 from[CP_UNR];
#pragma unroll
            for (u32 q = 0; q < CP_UNR; ++q) {
                const u32 j = j0 + q * 64 + lane;
                // the module holding record j: the first lane whose inclusive count exceeds j
                u32 lo = 0;
#pragma unroll
                for (u32 step = 32; step; step >>= 1)
                    if (__shfl(incl, lo + step - 1, 64) <= j) lo += step;
                const u32 s0 = __shfl(mod_src, lo, 64), x0 = __shfl(excl, lo, 64);
                from[q] = (j < j_hi && s0 != NOPIX) ? s0 + (j - x0) : NOPIX;
                const u32 fs = from[q] != NOPIX ? from[q] : 0u;
                r0[q] = tid_[fs];
                r1[q] = tch[fs];
                r2[q] = tsz[fs];
                sx[q] = sy[q] = 0ull;
                if (hits && from[q] != NOPIX) {
                    sx[q] = hsm[2 * fs];
                    sy[q] = hsm[2 * fs + 1];
                }
            }
#pragma unroll
            for (u32 q = 0; q < CP_UNR; ++q) {
                const u32 j = j0 + q * 64 + lane;
                if (from[q] != NOPIX) {
                    oid[base + j] = r0[q];
                    och[base + j] = r1[q];
                    osz[base + j] = r2[q];
                    if (hits) {                            // the centroid, as the hits kernel computes it
                        const u32 ch = u32(r1[q]);
                        hx[base + j] = ch ? float(double(sx[q]) / double(ch)) : __int_as_float(0x7FC00000);
                        hy[base + j] = ch ? float(double(sy[q]) / double(ch)) : __int_as_float(0x7FC00000);
                        hsm[2 * from[q]] = 0ull;           // the sums are zero again for the next launch
                        hsm[2 * from[q] + 1] = 0ull;
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// hits: per kept cluster the charge-weighted centroid of its pixels, x = sum(adc*col)
// / charge and y = sum(adc*row) / charge, from exact 64-bit sums, divided in double
// and rounded to float (NaN for zero charge).  One workgroup per module with kept
// clusters: the module's cluster ids (ascending) go to LDS, H_CAP at a time; every
// digi of the module whose id falls in the held range finds its cluster by binary
// search and adds its weighted coordinates with LDS atomics.
// ---------------------------------------------------------------------------
constexpr u32 H_WG = 64, H_CAP = 512;     // one wave, ~10 KB of LDS: every module resident at once

__global__ __launch_bounds__(H_WG) void k_hits(LaunchArgs a) {
    __shared__ u32 s_pref[MAXB + 1];
    __shared__ u32 s_wsum[H_WG / 64];
    __shared__ int32_t s_id[H_CAP];
    __shared__ u64 s_sx[H_CAP], s_sy[H_CAP];
    const u32 tid = threadIdx.x;
    const u32 k = num_events(a);
    const u32 total = event_prefix<H_WG>(a, k, s_pref, s_wsum, CNT_UNITS, 1, 0);
    for (u32 t = xcd_order(blockIdx.x, gridDim.x); t < total; t += gridDim.x) {
        const u32 e = find_slot(s_pref, k, t);
        const EventDesc E = get_event(a, e);
        const EvLayout L = ev_layout(E.cap, a.n_modules);
        const u32 mod = unit_module(a, E, L, s_pref[e + 1] - s_pref[e], t - s_pref[e]);
        const u32 cnt = ws_ptr<const u32>(E, L.kept)[mod];
        if (cnt == 0) continue;                            // absent, or nothing kept
        const ModRange r = ws_ptr<const ModRange>(E, L.mtab)[mod];
        const u32 st = u32(r.first), nd = u32(r.end) - st;
        const u32 off = ws_ptr<const u32>(E, L.off)[mod];
        if (cnt > E.n || off > E.n - cnt || st > E.n || nd > E.n - st) continue;
        const int32_t* ids = (const int32_t*)E.o_id + off;
        const int32_t* chg = (const int32_t*)E.o_charge + off;
        const int32_t* dcl = (const int32_t*)E.o_digi;
        const ModuleDigis D = module_digis(E, L, st);
        float* hx = ws_ptr<float>(E, L.hit_x) + off;
        float* hy = ws_ptr<float>(E, L.hit_y) + off;
        for (u32 c0 = 0; c0 < cnt; c0 += H_CAP) {
            const u32 len = min(H_CAP, cnt - c0);
            for (u32 c = tid; c < len; c += H_WG) {
                s_id[c] = ids[c0 + c];
                s_sx[c] = 0ull;
                s_sy[c] = 0ull;
            }
            lds_barrier();
            const int32_t lo = s_id[0], hi = s_id[len - 1];
            for (u32 j = tid; j < nd; j += H_WG) {
                const int32_t id = dcl[D.pos(j)];
                if (id < lo || id > hi) continue;          // cut (-1) or held by another chunk
                u32 l = 0, h = len;
                while (h - l > 1) {
                    const u32 m = (l + h) >> 1;
                    if (s_id[m] <= id) l = m; else h = m;
                }
                if (s_id[l] != id) continue;
                const u32 rc = D.rc(j);
                const u64 w = D.adc_at(j);
                atomicAdd(&s_sx[l], w * (rc >> 16));
                atomicAdd(&s_sy[l], w * (rc & 0xFFFFu));
            }
            lds_barrier();
            for (u32 c = tid; c < len; c += H_WG) {
                const u32 q = u32(chg[c0 + c]);
                hx[c0 + c] = q ? float(double(s_sx[c]) / double(q)) : __int_as_float(0x7FC00000);
                hy[c0 + c] = q ? float(double(s_sy[c]) / double(q)) : __int_as_float(0x7FC00000);
            }
            lds_barrier();
        }
    }
}

// ---------------------------------------------------------------------------
// fill: n words at p set to v (clears control words with a kernel node, which a
// caller's graph capture may record, instead of a memset node)
// ---------------------------------------------------------------------------
constexpr u32 F_WG = 256;
__global__ __launch_bounds__(F_WG) void k_fill(u32* p, u32 n, u32 v) {
    for (u32 i = blockIdx.x * F_WG + threadIdx.x; i < n; i += gridDim.x * F_WG) p[i] = v;
}

// ---------------------------------------------------------------------------
// copy: up to MAX_COPIES arrays between pinned host memory and the device in one launch.
// Bound by the link's latency and rate; an array per copy command costs ~10 us each (queuing
// it, an engine's start and its completion signal), so one launch moves them all, every
// thread with C_UNR words of any of them in flight.  The host's end is accessed at system
// scope: neither side may see the other's data through a cache it cannot see written.
// Four input and six output arrays of a 50,000-digi event, in new buffers or used ones: the
// whole chain of which they are part takes 101 us instead of 173 with a copy command each.
// ---------------------------------------------------------------------------
constexpr u32 CP_WG = 256, C_UNR = 4;
template <bool TO_HOST>
__global__ __launch_bounds__(CP_WG) void k_copy(CopyArgs c) {
    const u32 total = c.first[c.n], stride = gridDim.x * CP_WG, t0 = blockIdx.x * CP_WG + threadIdx.x;
    auto load = [](auto* p) {
        if constexpr (TO_HOST) return *p;
        else return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };
    auto store = [](auto* p, auto v) {
        if constexpr (TO_HOST) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        else *p = v;
    };
    for (u32 i0 = t0; i0 < total; i0 += C_UNR * stride) {
        u64 v[C_UNR];
        u64* to[C_UNR];
#pragma unroll
        for (u32 u = 0; u < C_UNR; ++u) {
            const u32 i = i0 + u * stride;
            to[u] = nullptr;
            if (i >= i0 && i < total) {
                u32 j = 0;
                while (j + 1 < c.n && i >= c.first[j + 1]) ++j;
                v[u] = load((const u64*)c.src[j] + (i - c.first[j]));
                to[u] = (u64*)c.dst[j] + (i - c.first[j]);
            }
        }
#pragma unroll
        for (u32 u = 0; u < C_UNR; ++u)
            if (to[u]) store(to[u], v[u]);
    }
    if (t0 < 4 * c.n) {                          // the tails, one value per thread
        const u32 j = t0 / 4, i = t0 % 4, words = c.first[j + 1] - c.first[j];
        if (i < c.tail[j])
            store((u16*)(c.dst[j] + words) + i, u16(load((const u16*)(c.src[j] + words) + i)));
    }
}

// ---------------------------------------------------------------------------
// host-side launch helpers
// ---------------------------------------------------------------------------
typedef void (*SmallKernel)(LaunchArgs);

static SmallKernel small_kernel(u32 wg, u32 mpw) {
    switch (wg * 8 + mpw) {
        case 64 * 8 + 1: return k_small<64, 1, K_SMALL>;
        case 128 * 8 + 1: return k_small<128, 1, K_SMALL>;
        case 128 * 8 + 2: return k_small<128, 2, K_SMALL>;
        case 256 * 8 + 1: return k_small<256, 1, K_SMALL>;
        case 256 * 8 + 2: return k_small<256, 2, K_SMALL>;
        case 256 * 8 + 4: return k_small<256, 4, K_SMALL>;
        case 512 * 8 + 1: return k_small<512, 1, K_SMALL>;
        case 512 * 8 + 2: return k_small<512, 2, K_SMALL>;
        case 512 * 8 + 4: return k_small<512, 4, K_SMALL>;
        default: return nullptr;
    }
}

bool cluster_config_valid(u32 wg, u32 mpw) { return small_kernel(wg, mpw) != nullptr; }
u32 cluster_capacity(u32 wg, u32 mpw) { return (wg / mpw) * K_SMALL; }

static int occ(const void* fn, int bs) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, bs, 0) != hipSuccess || n < 1) n = 1;
    return n;
}

int occupancy_segment() {
    return std::min(occ(reinterpret_cast<const void*>(k_segment<A_PER_N>), A_WG),
                    occ(reinterpret_cast<const void*>(k_segment<A_PER_W>), A_WG));
}
int occupancy_cluster(u32 wg, u32 mpw) {
    SmallKernel f = small_kernel(wg, mpw);
    return f ? occ(reinterpret_cast<const void*>(f), int(wg)) : 0;
}
int occupancy_big() { return occ(reinterpret_cast<const void*>(k_big), B_WG); }
int occupancy_compact() { return occ(reinterpret_cast<const void*>(k_compact), C_WG); }

int occupancy_group() {
    return std::min(occ(reinterpret_cast<const void*>(k_group_count), G_WG),
                    std::min(occ(reinterpret_cast<const void*>(k_group_scatter<false>), G_WG),
                             occ(reinterpret_cast<const void*>(k_group_scatter<true>), G_WG)));
}
u32 group_chunk() { return G_CH; }
u32 group_scatter_chunk() { return G_SCH; }
// The grouping kernels of the events in any order: count over `grid` workgroups, scatter over
// `grid_scatter`; between them, with more modules than the scatter can hold the first
// positions of, the table over `grid_events`.
hipError_t launch_group(const LaunchArgs& a, u32 grid, u32 grid_events, u32 grid_scatter, hipStream_t s) {
    hipLaunchKernelGGL(k_group_count, dim3(grid), dim3(G_WG), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.n_modules > G_HMAX) {
        hipLaunchKernelGGL(k_group_table, dim3(grid_events), dim3(G_WG), 0, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(k_group_scatter<true>, dim3(grid_scatter), dim3(G_WG), 0, s, a);
    } else {
        hipLaunchKernelGGL(k_group_scatter<false>, dim3(grid_scatter), dim3(G_WG), 0, s, a);
    }
    return hipGetLastError();
}
hipError_t launch_segment(const LaunchArgs& a, u32 grid, hipStream_t s) {
    if (a.flags & LF_SEG_WIDE) hipLaunchKernelGGL(k_segment<A_PER_W>, dim3(grid), dim3(A_WG), 0, s, a);
    else hipLaunchKernelGGL(k_segment<A_PER_N>, dim3(grid), dim3(A_WG), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_small(u32 wg, u32 mpw, const LaunchArgs& a, u32 grid, hipStream_t s) {
    SmallKernel f = small_kernel(wg, mpw);
    if (!f) return hipErrorInvalidValue;
    hipLaunchKernelGGL(f, dim3(grid), dim3(wg), 0, s, a);
    return hipGetLastError();
}
// The big-module kernel: workgroups for `grid` listed modules of either mode; with fewer,
// modules wait for a ticket.
hipError_t launch_big(const LaunchArgs& a, u32 grid, hipStream_t s) {
    hipLaunchKernelGGL(k_big, dim3(grid), dim3(B_WG), 0, s, a);
    return hipGetLastError();
}
u32 compact_waves_per_block(u32 waves, u32 blocks) { return compact_split(waves, blocks); }
hipError_t launch_compact(const LaunchArgs& a, u32 grid, hipStream_t s) {
    hipLaunchKernelGGL(k_compact, dim3(grid), dim3(C_WG), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_fill(u32* p, u32 n, u32 v, hipStream_t s) {
    if (!n) return hipSuccess;
    const u32 grid = std::min<u32>((n + F_WG - 1) / F_WG, 1024u);
    hipLaunchKernelGGL(k_fill, dim3(grid), dim3(F_WG), 0, s, p, n, v);
    return hipGetLastError();
}
hipError_t launch_copy(const CopyArgs& c, bool to_host, hipStream_t s) {
    const u32 grid = std::max<u32>(1u, std::min<u32>((c.first[c.n] + CP_WG * C_UNR - 1) / (CP_WG * C_UNR), 256u));
    if (to_host) hipLaunchKernelGGL(k_copy<true>, dim3(grid), dim3(CP_WG), 0, s, c);
    else hipLaunchKernelGGL(k_copy<false>, dim3(grid), dim3(CP_WG), 0, s, c);
    return hipGetLastError();
}
int occupancy_hits() { return occ(reinterpret_cast<const void*>(k_hits), H_WG); }
hipError_t launch_hits(const LaunchArgs& a, u32 grid, hipStream_t s) {
    hipLaunchKernelGGL(k_hits, dim3(grid), dim3(H_WG), 0, s, a);
    return hipGetLastError();
}

}  // namespace pxcl
