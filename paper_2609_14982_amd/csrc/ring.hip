// Level walk with the recent node values in LDS: one workgroup owns one
// (source, right-hand side) pair and walks the source's levels alone.
//
// Why.  Small and middle-sized problems are bound by the latency of a level,
// not by bytes: the node split pays a barrier between workgroups, a store to
// the L2 and a neighbour load from it in every level (about 2.3 us measured on
// a 101x101x51 grid), the rhs-group kernel store, barrier and load in its own
// CU plus the scattered accesses of one CU (4.4 us).  A workgroup that owns a
// level alone can keep the values of the last C positions of its walk in LDS
// (160 KB hold 15,300 to 19,100 FP64 values beside the far ones, five to ten
// levels of that grid), so that a level's chain is three LDS reads, three FMAs,
// one LDS write and a workgroup barrier, and everything it streams is known
// ahead of time:
//   - per node, in level order: the LDS slots of its neighbours, its node id,
//     its weights and its right-hand side q, permuted to level order by a pass
//     before the walk; all are loaded D batches ahead;
//   - neighbours that left the window ("far", 3-6 % there) are read back from
//     the node rows by waves of their own into a side window of F slots, so a
//     lane of the walk finds every operand in LDS, at a slot computed once
//     when the batch was created.
// A level wider than two batches of the narrow waves is walked in chunks, so
// that the window only has to hold the chunks a far value is late by and the
// level's own neighbours mostly stay in it.  Waves have one of three roles: CW
// waves take the chunk's nodes with at most three neighbours, OW waves the few
// with more (six slots and weights each), FW waves load far values and, for
// the transpose from receiver data, the receiver inputs.  All meet at one
// workgroup barrier per chunk that waits for LDS only; the node rows written
// to global memory are drained every K chunks, which is enough because any
// K + G + 1 consecutive chunks fit in the window and a far value is loaded
// G + 1 chunks before the chunk that reads it.  SCC blocks are solved by the
// whole workgroup at the end of their level.
//
// A node's sum is taken in the order of the other kernels (q, then its
// neighbours by ascending slot; unused slots add 0 * 0).
//
// Measured against the schedule it replaces, whole applies whose inputs change
// from pass to pass: 101x101x51, 8 sources x 16 right-hand sides, FP64: J 2.80 ->
// 1.12 ms, J^T summed 3.64 -> 1.62 ms; 121x97x57, 6 x 16, FP32: J to every node
// 5.52 -> 1.76 ms; 67x53x31, 5 x 5, FP64: J^T per source 1.28 -> 0.54 ms; 81x41, one
// pair: J 149 -> 40 us, J^T 199 -> 43 us; the same inputs again, 101x101x51, 8 x 1: J
// 3.50 -> 0.79 ms, J^T 2.89 -> 1.23 ms.  What bounds it now is the bytes one CU
// keeps in flight: 44 a node (36 with receiver input) arrive at some 32 GB/s
// however many batches are loaded ahead (3 to 8: the same time), and without the
// weights' load the walk takes half as long.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "devmem.h"
#include "ring.h"
#include "sweep.h"

namespace fm {

namespace {

constexpr uint32_t kCntMask = 1023u, kLast = 1u << 10, kBlk = 1u << 11, kDrain = 1u << 12;
constexpr uint32_t kStore = 1u << 31;      // ref word 0: the node row is read again from memory
constexpr uint32_t kRcvEntry = 1u << 31;   // far-list entry: receiver input instead of a node row

// One direction of one source.  Slots of the window (a value each):
// [0, C) position p at p mod C, C a zero, then F side slots.
struct RingDev {
    const uint2* ref;         // [N] slots 0 and 1, slot 2 and the input's slot
    const uint32_t* node;     // [N] node | kStore
    const void* wa;           // FP64: [N][2] w_1, w_2; FP32: [N][4] w_1, w_2, w_3, c
    const void* wb;           // FP64: [N] w_3
    const void* wc;           // FP64: [N] c (transpose)
    const uint32_t* wref;     // [nw][4] node | kStore, slots 0..5
    const void* wwt;          // [nw][8] V: c, w_1..w_6, then the input's slot as a uint32
    const uint2* nd;          // narrow batches: position, count | flags | slot << 16
    const uint4* wd;          // wide batches: position, count | flags | slot << 16, first wide record, levels
                              // passed over before it
    const uint4* fd;          // steps of the far waves, one per level and empty ones that fill the round
                              // after blocks: first far entry, count, flags, first side slot
    const uint32_t* far;      // far entries
    const int32_t* blk_w;     // [nblk] first wide record of each block's members
    int32_t n_nd, n_wd, n_fd;
    const int32_t* lev;       // [L] level of each chunk
};

struct RingArgs {
    const RingDev* dev;       // [S][2]
    const void* q;            // [S][B][N] inputs in level order, or receiver inputs [S][n_ent][B]
    int32_t C, F;
    int32_t stage_off;        // first byte of the block staging area in LDS
    int32_t store_all;        // every node row is an output
    int32_t n_ent;
    unsigned* xmask;          // XCDs seen per source (placement report), or nullptr
};

// A whole struct through one global-address-space load (see gld).
template <class T>
__device__ __forceinline__ T glv(const T* p) {
    typedef uint32_t vec __attribute__((ext_vector_type(sizeof(T) / 4), aligned(alignof(T))));
    typedef const __attribute__((address_space(1))) vec gvec;
    const vec x = *(gvec*)(p);
    T r;
    __builtin_memcpy(&r, &x, sizeof(T));
    return r;
}

// The same at a 32-bit byte offset from a uniform base (every array of one
// item spans less than 4 GiB): one scalar pair and one lane register.
template <class T>
__device__ __forceinline__ T ldo(const void* base, uint32_t off) {
    return glv(reinterpret_cast<const T*>(static_cast<const char*>(base) + off));
}

// LDS only: the level's window writes are visible to every wave after it
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// every load and store of this wave has completed (vmcnt(0) alone, as a
// builtin: the compiler then knows it too, and the waits after the branch stay
// those of the other path).  The wait names no memory: the clobbers keep the
// compiler from moving a store past it.  (A release fence waits for LDS as well:
// J^T of 101x101x51, 8 x 16, 1.51 -> 1.53 ms.)
__device__ __forceinline__ void drain() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70);
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ uint32_t uni(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

// A uniform pointer in scalar registers: read once before the walk (the
// barriers' memory clobber would have it loaded again in every step).
template <class T>
__device__ __forceinline__ const T* uptr(const T* p) {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint64_t lo = uni((uint32_t)v), hi = uni((uint32_t)(v >> 32));
    return (const T*)(uintptr_t)(hi << 32 | lo);
}

template <typename V>
struct WalkCtx {
    V* X;                     // node rows of this source, at this right-hand side
    V* outp;                  // per-source output rows of the transpose, or nullptr
    uint32_t xB, oB;          // values per row
    bool store_all;
    int C;
    int l;                    // level being walked
    bool blk;                 // it ends with blocks, after the round
    const SrcDev* sd;
    const RingDev* rd;
    const void* q;            // this item's inputs in level order, or nullptr
    const V* in;              // primal: rows of ds, at this right-hand side
    uint32_t lds;             // LDS address of the window
    int stage_off;
};

// The blocks of level l, by all TB threads: right-hand sides b from the window
// (summed in FP64 whatever the vector precision), then rows of A_C^{-1} b; the
// columns of a block are split over groups of whole waves when it has fewer
// rows than the workgroup has threads, and the partial sums added in column
// order.
template <int DIR, typename V, int TB, bool QS>
__device__ __forceinline__ void ring_blocks(const WalkCtx<V>& w) {
    typedef __attribute__((address_space(3))) V lds_v;
    typedef __attribute__((address_space(3))) double lds_d;
    lds_v* win = (lds_v*)(uintptr_t)w.lds;
    lds_d* sb = (lds_d*)(uintptr_t)(w.lds + (uint32_t)w.stage_off);
    const SrcDev& sd = *w.sd;
    const RingDev& rd = *w.rd;
    const V* q = (const V*)w.q;
    const int tid = (int)threadIdx.x;
    const int lev = gld(rd.lev + w.l);
    const int b0 = gld((DIR == kFwd ? sd.fblk_ptr : sd.rblk_ptr) + lev);
    const int b1 = gld((DIR == kFwd ? sd.fblk_ptr : sd.rblk_ptr) + lev + 1);
    const V* __restrict__ wwt = (const V*)rd.wwt;
    // member i's result: window slot, node row, per-source output
    auto put_member = [&](int w0, int i, int bp, double acc) {
        const uint32_t node = gld(rd.wref + (size_t)(w0 + i) * 4) & ~kStore;
        const V o = (V)acc;
        win[(bp + i) % w.C] = o;
        w.X[(size_t)node * w.xB] = o;
        if (DIR == kRev && w.outp) w.outp[(size_t)node * w.oB] = gld(wwt + (size_t)(w0 + i) * 8) * o;
    };
    for (int bi = b0; bi < b1; ++bi) {
        const int blk = gld((DIR == kFwd ? sd.fblk_id : sd.rblk_id) + bi);
        const int k = gld(sd.blk_k + blk);
        const int bp = gld((DIR == kFwd ? sd.blk_fpos : sd.blk_rpos) + blk);
        const int w0 = gld(rd.blk_w + blk);
        for (int m = tid; m < k; m += TB) {
            const uint32_t* rf = rd.wref + (size_t)(w0 + m) * 4;
            const V* wt = wwt + (size_t)(w0 + m) * 8;
            double acc;
            if constexpr (DIR == kFwd && sizeof(V) == 4)
                // (c ds is exact in FP64; the input pass has rounded it to FP32)
                acc = (double)gld(wt) * (double)gld(w.in + (size_t)(gld(rf) & ~kStore) * w.oB);
            else
                acc = (double)(QS ? win[gld(reinterpret_cast<const uint32_t*>(wt + 7))] : gld(q + bp + m));
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                const uint32_t s = (gld(rf + 1 + t / 2) >> (16 * (t & 1))) & 0xffffu;
                acc += (double)gld(wt + 1 + t) * (double)win[s];
            }
            sb[m] = acc;
        }
        wg_barrier();
        const int m_it = gld(sd.blk_it + 2 * blk + (DIR == kFwd ? 0 : 1));
        if (m_it) {
            // a large block solved by its Neumann series: x^0 = b,
            // x^j = b + W_CC x^{j-1} (transpose: W_CC^T), the iterates in two
            // more staging buffers, the last one straight to the node rows
            const int64_t sp = gld(sd.blk_sp + blk);
            const int32_t* __restrict__ rp = (DIR == kFwd ? sd.sp_ptr : sd.spt_ptr) + sp;
            const int32_t* __restrict__ cl = DIR == kFwd ? sd.sp_col : sd.spt_col;
            const double* __restrict__ wv = DIR == kFwd ? sd.sp_w : sd.spt_w;
            for (int j = 1; j <= m_it; ++j) {
                lds_d* cur = j == 1 ? sb : sb + k * (1 + ((j - 1) & 1));
                lds_d* nxt = sb + k * (1 + (j & 1));
                for (int i = tid; i < k; i += TB) {
                    double acc = sb[i];
                    const int e1 = gld(rp + i + 1);
                    for (int e = gld(rp + i); e < e1; ++e) acc += gld(wv + e) * cur[gld(cl + e)];
                    if (j < m_it) nxt[i] = acc;
                    else put_member(w0, i, bp, acc);
                }
                wg_barrier();
            }
            continue;
        }
        const int kw = (k + 63) & ~63;
        const int parts = kw < TB ? TB / kw : 1;
        lds_d* part = sb + k;             // [parts - 1][kw]
        const __attribute__((address_space(1))) double* __restrict__ Mx =
            gptr((DIR == kFwd ? sd.inv : sd.invt) + gld(sd.blk_inv + blk));
        for (int r0 = 0; r0 < k; r0 += TB) {
            const int pt = parts > 1 ? tid / kw : 0;
            const int i = parts > 1 ? tid - pt * kw : r0 + tid;
            const bool own = i < k && pt < parts;
            double acc = 0.0;
            if (own) {
                const int j1 = (int)((int64_t)k * (pt + 1) / parts);
                int j = (int)((int64_t)k * pt / parts);
                constexpr int G = 8;
                for (; j + G <= j1; j += G) {
                    double m[G];
#pragma unroll
                    for (int t = 0; t < G; ++t) m[t] = Mx[(size_t)(j + t) * k + i];
#pragma unroll
                    for (int t = 0; t < G; ++t) acc += m[t] * sb[j + t];
                }
                for (; j < j1; ++j) acc += Mx[(size_t)j * k + i] * sb[j];
                if (pt > 0) part[(pt - 1) * kw + i] = acc;
            }
            if (parts > 1) wg_barrier();
            if (own && pt == 0) {
                for (int p = 0; p + 1 < parts; ++p) acc += part[p * kw + i];
                put_member(w0, i, bp, acc);
            }
        }
        wg_barrier();   // the staging area is reused by the next block
    }
}

// End of a level: its rows drained where it asks for it, then its barrier,
// which orders the window.  A level with blocks ends after its round of steps
// (the rest of the round is empty), so that the steps hold no block code.
template <typename V>
__device__ __forceinline__ void level_end(uint32_t flags, WalkCtx<V>& w) {
    if (flags & kBlk) {
        w.blk = true;
        return;
    }
    if (flags & kDrain) drain();
    wg_barrier();
    ++w.l;
}

template <int DIR, typename V, int TB, bool QS>
__device__ __forceinline__ void round_end(WalkCtx<V>& w) {
    if (!w.blk) return;
    ring_blocks<DIR, V, TB, QS>(w);
    drain();
    wg_barrier();
    ++w.l;
    w.blk = false;
}

// A node's result: window slot, node row, per-source output.
template <bool PS, typename V>
__device__ __forceinline__ void put_node(const WalkCtx<V>& w, V* win, V o, uint32_t slot, uint32_t ref0, V c) {
    win[slot] = o;
    const uint32_t node = ref0 & ~kStore;
    if (w.store_all || (ref0 & kStore))
        *reinterpret_cast<V*>(reinterpret_cast<char*>(w.X) + node * (w.xB * (uint32_t)sizeof(V))) = o;
    if (PS) w.outp[(size_t)node * w.oB] = c * o;
}

// CW waves: nodes with at most three neighbours, one per lane.  Every stream
// is an array of its own, so that a wave's load takes whole cache lines and
// takes them once: the batches in flight are as large as the L1 (32 KB), which
// cannot hold a line for a second load (records of 32 bytes, two loads per
// line: 0.95 ms on the 101x101x51 grid against 0.72 ms with half the batches in
// flight).
template <int DIR, typename V, int TB, int D, bool QS, bool PS>
__device__ __forceinline__ void walk_narrow(const RingDev& rd, WalkCtx<V>& w, char* lds,
                                            const V* __restrict__ q, int lane) {
    constexpr bool F64 = sizeof(V) == 8;
    constexpr bool SC = F64 && PS;       // c is a stream of its own
    V* win = reinterpret_cast<V*>(lds);
    const void* __restrict__ wa = uptr(static_cast<const char*>(rd.wa));
    const void* __restrict__ wb = uptr(static_cast<const char*>(rd.wb));
    const void* __restrict__ wc = uptr(static_cast<const char*>(rd.wc));
    const uint2* __restrict__ ref = uptr(rd.ref);
    const uint32_t* __restrict__ node = uptr(rd.node);
    const uint2* __restrict__ nd = uptr(rd.nd);
    const int n_nd = (int)uni((uint32_t)rd.n_nd);
    struct Stage {
        uint2 rf;
        uint32_t nd, y;
        Pack<V, 16 / sizeof(V)> wa;
        V wb, wc, q;
    } s[D];
    uint2 ahead[D];
    // every lane loads a valid position (the batch's last one when it has no
    // node), so that a batch is the same number of loads for every wave
    auto fetch = [&](Stage& t, uint2 d) {
        const uint32_t p0 = uni(d.x);
        t.y = uni(d.y);
        const uint32_t last = max(t.y & kCntMask, 1u) - 1u;
        const uint32_t p = p0 + min((uint32_t)lane, last);
        t.rf = ldo<uint2>(ref, p * 8u);
        t.wa = ldo<Pack<V, 16 / sizeof(V)>>(wa, p * 16u);
        if (F64) t.wb = ldo<V>(wb, p * 8u);
        if (SC) t.wc = ldo<V>(wc, p * 8u);
        t.nd = ldo<uint32_t>(node, p * 4u);
        if (!QS) t.q = ldo<V>(q, p * (uint32_t)sizeof(V));
    };
    // the first two rounds of the loop only load the first batches (loads before
    // it would be in another order, and the memory counter is waited for by
    // position: the waits inside would be the shorter ones of both orders)
#pragma unroll
    for (int j = 0; j < D; ++j) {
        s[j] = Stage{};
        ahead[j] = uint2{0u, 0u};
    }
    wg_barrier();
    for (int n = -2 * D; n < n_nd; n += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const uint32_t y = s[j].y;
            if (lane < (int)(y & kCntMask)) {
                const V x0 = win[s[j].rf.x & 0xffffu], x1 = win[s[j].rf.x >> 16], x2 = win[s[j].rf.y & 0xffffu];
                V o = QS ? win[s[j].rf.y >> 16] : s[j].q;
                const V w3 = F64 ? s[j].wb : s[j].wa.v[F64 ? 0 : 2];
                const V c = F64 ? s[j].wc : s[j].wa.v[F64 ? 0 : 3];
                o += s[j].wa.v[0] * x0;
                o += s[j].wa.v[1] * x1;
                o += w3 * x2;
                uint32_t slot = (y >> 16) + (uint32_t)lane;
                if (slot >= (uint32_t)w.C) slot -= (uint32_t)w.C;
                put_node<PS, V>(w, win, o, slot, s[j].nd, c);
            }
            fetch(s[j], ahead[j]);
            ahead[j] = glv(nd + n + j + 2 * D);
            if (y & kLast) level_end(y, w);
        }
        round_end<DIR, V, TB, QS>(w);
    }
}

// OW waves: the level's nodes with four to six neighbours.
template <int DIR, typename V, int TB, int D, bool QS, bool PS>
__device__ __forceinline__ void walk_wide(const RingDev& rd, WalkCtx<V>& w, char* lds,
                                            const V* __restrict__ q, int lane) {
    V* win = reinterpret_cast<V*>(lds);
    const V* __restrict__ wwt = uptr((const V*)rd.wwt);
    const uint4* __restrict__ wref = uptr(reinterpret_cast<const uint4*>(rd.wref));
    const uint4* __restrict__ wd = uptr(rd.wd);
    const int n_wd = (int)uni((uint32_t)rd.n_wd);
    struct Stage {
        uint32_t y, skip;
        uint4 rf;
        Pack<V, 4> wa, wb;
        V q;
    } s[D];
    uint4 ahead[D];
    auto fetch = [&](Stage& t, uint4 d) {
        const uint32_t p0 = uni(d.x), w0 = uni(d.z);
        t.y = uni(d.y);
        t.skip = uni(d.w);
        const uint32_t i = min((uint32_t)lane, max(t.y & kCntMask, 1u) - 1u);
        t.rf = ldo<uint4>(wref, (w0 + i) * 16u);
        t.wa = ldo<Pack<V, 4>>(wwt, (w0 + i) * (uint32_t)(8 * sizeof(V)));
        t.wb = ldo<Pack<V, 4>>(wwt, (w0 + i) * (uint32_t)(8 * sizeof(V)) + (uint32_t)(4 * sizeof(V)));
        if (!QS) t.q = ldo<V>(q, (p0 + i) * (uint32_t)sizeof(V));
    };
#pragma unroll
    for (int j = 0; j < D; ++j) {
        s[j] = Stage{};
        ahead[j] = uint4{0u, 0u, 0u, 0u};
    }
    wg_barrier();
    for (int n = -2 * D; n < n_wd; n += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const uint32_t y = s[j].y;
            // levels without such nodes (and without blocks or a drain)
            for (uint32_t k = 0; k < s[j].skip; ++k) wg_barrier();
            w.l += (int)s[j].skip;
            if (lane < (int)(y & kCntMask)) {
                const uint32_t sl[6] = {s[j].rf.y & 0xffffu, s[j].rf.y >> 16, s[j].rf.z & 0xffffu,
                                        s[j].rf.z >> 16,     s[j].rf.w & 0xffffu, s[j].rf.w >> 16};
                const V wt[6] = {s[j].wa.v[1], s[j].wa.v[2], s[j].wa.v[3], s[j].wb.v[0], s[j].wb.v[1], s[j].wb.v[2]};
                V x[6];
#pragma unroll
                for (int t = 0; t < 6; ++t) x[t] = win[sl[t]];
                V o;
                if (QS) {
                    uint32_t qs;
                    const V tag = s[j].wb.v[3];
                    __builtin_memcpy(&qs, &tag, sizeof(qs));
                    o = win[qs];
                } else {
                    o = s[j].q;
                }
#pragma unroll
                for (int t = 0; t < 6; ++t) o += wt[t] * x[t];
                uint32_t slot = (y >> 16) + (uint32_t)lane;
                if (slot >= (uint32_t)w.C) slot -= (uint32_t)w.C;
                put_node<PS, V>(w, win, o, slot, s[j].rf.x, s[j].wa.v[0]);
            }
            fetch(s[j], ahead[j]);
            ahead[j] = glv(wd + n + j + 2 * D);
            if (y & kLast) level_end(y, w);
        }
        round_end<DIR, V, TB, QS>(w);
    }
}

// FW waves: far values and receiver inputs.  A level's entries are written to
// the side window one level ahead; its values are loaded G levels before that
// (no earlier, since they are results of the walk), its list entries E levels
// before the values and the list's place E before those (static data): each
// wait is for loads that are as many levels old, a load through the caches
// taking as long as several narrow levels.
template <int DIR, typename V, int TB, int FT, int G, int E, int U, bool QS>
__device__ __forceinline__ void walk_far(const RingDev& rd, WalkCtx<V>& w, char* lds, const V* __restrict__ rv, int B, int F,
                                         int lane) {
    static_assert(E % G == 0 && G < E, "the slots of the values repeat within a round; three rounds fill the pipeline");
    V* win = reinterpret_cast<V*>(lds);
    const uint32_t side = (uint32_t)w.C + 1u;
    const uint32_t* __restrict__ far = uptr(rd.far);
    const uint4* __restrict__ fd = uptr(rd.fd);
    const int L = (int)uni((uint32_t)rd.n_fd);
    auto value = [&](uint32_t e) {
        // (receiver entries have no use where the input is streamed)
        const bool rcv = (e & kRcvEntry) != 0u;
        if (!QS) return ldo<V>(w.X, (rcv ? 0u : e) * (w.xB * (uint32_t)sizeof(V)));
        const char* src = rcv ? reinterpret_cast<const char*>(rv) : reinterpret_cast<const char*>(w.X);
        return ldo<V>(src, (e & ~kRcvEntry) * ((rcv ? (uint32_t)B : w.xB) * (uint32_t)sizeof(V)));
    };
    auto put = [&](const uint4& d, int i, V x) {
        uint32_t s = d.w + (uint32_t)i;
        if (s >= (uint32_t)F) s -= (uint32_t)F;
        win[side + s] = x;
    };
    // entries past the lanes' registers: loaded and written at once
    auto rest = [&](const uint4& d, int from) {
        for (int i = from + lane; i < (int)d.y; i += FT) put(d, i, value(gld(far + d.x + i)));
    };
    auto whole = [&](const uint4& d) { return uint4{uni(d.x), uni(d.y), uni(d.z), uni(d.w)}; };
    uint4 dv[G], de[E], dd[E];
    V val[G][U];
    uint32_t ent[E][U];
    // a lane without an entry loads the last one (every step is the same
    // number of loads)
    auto entries = [&](uint32_t e[U], const uint4& d) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            e[u] = ldo<uint32_t>(far, (d.x + min((uint32_t)(lane + u * FT), max(d.y, 1u) - 1u)) * 4u);
    };
    // the first G + 2 E + 1 levels only fill the pipeline (the list of places
    // starts with E empty ones)
#pragma unroll
    for (int j = 0; j < E; ++j) {
        de[j] = dd[j] = uint4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int u = 0; u < U; ++u) ent[j][u] = 0u;
    }
#pragma unroll
    for (int j = 0; j < G; ++j) dv[j] = uint4{0u, 0u, 0u, 0u};
    uint32_t flags = 0u;
    for (int l = -3 * E; l < L; l += E) {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const uint4 d = dv[j % G];       // level l + j + 1
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (lane + u * FT < (int)d.y) put(d, lane + u * FT, val[j % G][u]);
            if ((int)d.y > FT * U) rest(d, FT * U);
            dv[j % G] = de[j];               // level l + j + 1 + G
#pragma unroll
            for (int u = 0; u < U; ++u) val[j % G][u] = value(ent[j][u]);
            de[j] = whole(dd[j]);            // level l + j + 1 + G + E
            entries(ent[j], de[j]);
            dd[j] = glv(fd + l + j + 1 + G + 2 * E + E);
            if (l + j == -1) wg_barrier();
            if (flags & kLast) level_end(flags, w);
            flags = d.z;
        }
        round_end<DIR, V, TB, QS>(w);
    }
}

// QS: the input is at a side slot (transpose from receiver data); otherwise
// it is streamed in level order.  PS: c lambda is written per source.
template <int DIR, typename V, int CW, int OW, int FW, int D, int DW, int G, int E, int U, bool QS, bool PS>
__global__ __launch_bounds__((CW + OW + FW) * 64) void k_ring(ApplyArgs a, RingArgs r) {
    constexpr int TB = (CW + OW + FW) * 64;
    const int wg = blockIdx.x;
    const int item = (wg % 8) * a.per_xcd + (wg / 8);
    if (item >= a.items) return;
    const int alpha = item / a.B, rhs = item - alpha * a.B;
    extern __shared__ char ring_lds[];
    WalkCtx<V> w;
    w.X = (V*)a.work + (size_t)alpha * a.N * a.xB + rhs;
    w.outp = DIR == kRev && a.out_mode == FM_JT_PER_SOURCE ? (V*)a.out + (size_t)alpha * a.N * a.B + rhs : nullptr;
    w.xB = (uint32_t)a.xB;
    w.oB = (uint32_t)a.B;
    w.store_all = r.store_all != 0;
    w.C = r.C;
    w.l = 0;
    w.blk = false;
    const V* q = QS ? nullptr : (const V*)r.q + (size_t)item * a.N;
    const V* rv = QS ? (const V*)r.q + (size_t)alpha * r.n_ent * a.B + rhs : nullptr;
    if (threadIdx.x == 0) {
        reinterpret_cast<V*>(ring_lds)[r.C] = (V)0;
        if (r.xmask) {
            unsigned x;
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
            __hip_atomic_fetch_or(r.xmask + (size_t)alpha * 32, 1u << (x & 0xfu), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    w.sd = a.src + alpha;
    w.rd = r.dev + 2 * alpha + (DIR == kFwd ? 0 : 1);
    w.q = q;
    w.in = DIR == kFwd ? (const V*)a.in + (a.in_mode == FM_DS_PER_PAIR ? (size_t)alpha * a.N * a.B : 0) + rhs : nullptr;
    w.lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring_lds;
    w.stage_off = r.stage_off;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (wave < CW)
        walk_narrow<DIR, V, TB, D, QS, PS>(*w.rd, w, ring_lds, q, (int)threadIdx.x);
    else if (wave < CW + OW)
        walk_wide<DIR, V, TB, DW, QS, PS>(*w.rd, w, ring_lds, q, (int)threadIdx.x - CW * 64);
    else
        walk_far<DIR, V, TB, FW * 64, G, E, U, QS>(*w.rd, w, ring_lds, rv, a.B, r.F, (int)threadIdx.x - (CW + OW) * 64);
}

// ---------------------------------------------------------------------------
// inputs in level order
// ---------------------------------------------------------------------------

constexpr int kPermRows = 256;

// q[alpha][b][p] = c ds (forward) or w (transpose) of the node at position p:
// CL columns of 256 rows at a time, rows read by CL lanes, transposed in LDS,
// written 256 values at a time.  Bound by the rows in flight: a lane has CL
// loads outstanding (with four of 64-row tiles the pass took 300 us for 8 x 16
// on 101x101x51, 1.07 GB).
template <int DIR, typename V, int CL>
__global__ __launch_bounds__(kPermRows) void k_ring_q(ApplyArgs a, RingArgs r, V* __restrict__ q) {
    __shared__ V tile[CL][kPermRows + 1];
    __shared__ uint32_t node[kPermRows];
    __shared__ V scale[kPermRows];
    constexpr int step = kPermRows / CL;       // rows of one load
    const int alpha = blockIdx.y, tid = (int)threadIdx.x;
    if (blockIdx.x == 0 && tid == 0 && r.xmask) r.xmask[(size_t)alpha * 32] = 0u;
    const SrcDev& sd = a.src[alpha];
    const uint64_t* __restrict__ meta = DIR == kFwd ? sd.fmeta : sd.rmeta;
    const bool per_source = DIR == kRev || a.in_mode == FM_DS_PER_PAIR;
    const V* __restrict__ in = (const V*)a.in + (per_source ? (size_t)alpha * a.N * a.B : 0);
    V* __restrict__ dst = q + (size_t)alpha * a.N * a.B;
    const int64_t p0 = (int64_t)blockIdx.x * kPermRows;
    const int rows = (int)min((int64_t)kPermRows, a.N - p0);
    // rows past the end repeat the last one
    const int64_t mine = p0 + min(tid, rows - 1);
    node[tid] = (uint32_t)(gld(meta + mine) & kNodeMask);
    if (DIR == kFwd) scale[tid] = gld((const V*)sd.fwts + (size_t)mine * 4);
    __syncthreads();
    const int c = tid % CL, i0 = tid / CL;
    for (int c0 = 0; c0 < a.B; c0 += CL) {
        const int col = min(c0 + c, a.B - 1);
        V x[CL];
#pragma unroll
        for (int k = 0; k < CL; ++k) x[k] = gld(in + (size_t)node[i0 + k * step] * a.B + col);
#pragma unroll
        for (int k = 0; k < CL; ++k) tile[c][i0 + k * step] = DIR == kFwd ? scale[i0 + k * step] * x[k] : x[k];
        __syncthreads();
        if (tid < rows)
#pragma unroll
            for (int k = 0; k < CL; ++k)
                if (c0 + k < a.B) dst[(size_t)(c0 + k) * a.N + p0 + tid] = tile[k][tid];
        __syncthreads();
    }
}

// Receiver inputs of the transpose: the entry that is first at its position
// holds the sum of the position's entries (in entry order).
template <typename V>
__global__ void k_ring_rcv(ApplyArgs a, RingArgs r, V* __restrict__ rv) {
    const int alpha = blockIdx.y;
    if (blockIdx.x == 0 && threadIdx.x == 0 && r.xmask) r.xmask[(size_t)alpha * 32] = 0u;
    const SrcDev& sd = a.src[alpha];
    const V* __restrict__ in = (const V*)a.in + (size_t)alpha * a.R * a.B;
    V* __restrict__ dst = rv + (size_t)alpha * r.n_ent * a.B;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < sd.n_ent * a.B; t += gridDim.x * blockDim.x) {
        const int e = t / a.B, b = t - e * a.B;
        const int pos = gld(sd.rcv_pos + e);
        if (e > 0 && gld(sd.rcv_pos + e - 1) == pos) continue;
        V acc = (V)0;
        for (int i = e; i < sd.n_ent && gld(sd.rcv_pos + i) == pos; ++i)
            acc = acc + (V)(gld(sd.rcv_ew + i) * (double)gld(in + (size_t)gld(sd.rcv_idx + i) * a.B + b));
        dst[(size_t)e * a.B + b] = acc;
    }
}

// ---------------------------------------------------------------------------
// tables
// ---------------------------------------------------------------------------

constexpr int kCand = 3;   // window sizes counted at once

struct BuildDev {          // one direction of one source
    const uint64_t* meta;
    const void* wts;
    const int32_t *lvl_ptr, *lvl_nsc, *lev;  // chunks: positions, singletons, level
    const int32_t *rcvlvl_ptr, *rcv_pos;   // transpose only
    const int32_t* rcv_node;               // forward only: rows read by the gather
    int32_t n_rcv_node;
    int32_t L;
    int32_t* pos;          // [N] position of each node, -1 outside the walk
    uint8_t* need;         // [N] the row is read again
    int32_t* cnt;          // [L][kCand + 2] far references per window size, receivers, nodes of <= 3 neighbours
    uint2* ref;
    uint32_t *node, *wref, *far;
    void *wa, *wb, *wc, *wwt;
    int32_t C, F;          // window chosen
    const int4* lv;        // [L + 1] first wide record, first far entry, first side slot, nodes of <= 3 neighbours
};

struct BuildArgs {
    const BuildDev* dev;
    int64_t N, st1, st2;
    int32_t C[kCand];
};

// (kernels: a memset costs the host 35 us)
__global__ void k_ring_clear(BuildArgs a) {
    const BuildDev& d = a.dev[blockIdx.y];
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < a.N; p += (int64_t)gridDim.x * blockDim.x) {
        d.pos[p] = -1;
        d.need[p] = 0;
    }
}

__global__ void k_ring_pos(BuildArgs a) {
    const BuildDev& d = a.dev[blockIdx.y];
    const int64_t n = d.lvl_ptr[d.L];
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x)
        d.pos[d.meta[p] & kNodeMask] = (int32_t)p;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < d.n_rcv_node;
         e += (int64_t)gridDim.x * blockDim.x)
        d.need[d.rcv_node[e]] = 1;
}

// a neighbour's position is in the window of a level that ends at p1
__device__ __forceinline__ bool in_window(int32_t pos, int32_t p1, int32_t C) { return pos >= 0 && p1 - pos <= C; }

// one workgroup per level: far references per window size, receiver nodes and
// nodes with at most three neighbours
__global__ __launch_bounds__(256) void k_ring_count(BuildArgs a) {
    const BuildDev& d = a.dev[blockIdx.y];
    const int l = blockIdx.x;
    if (l >= d.L) return;
    const int32_t p0 = d.lvl_ptr[l], p1 = d.lvl_ptr[l + 1], ps = p0 + d.lvl_nsc[l];
    __shared__ int32_t s[kCand + 2];
    if (threadIdx.x < kCand + 2) s[threadIdx.x] = 0;
    __syncthreads();
    int32_t far[kCand] = {0}, rcv = 0, few = 0;
    for (int32_t p = p0 + (int32_t)threadIdx.x; p < p1; p += 256) {
        const uint64_t m = d.meta[p];
        uint32_t mask = (uint32_t)(m >> kMaskShift);
        if (p < ps && __popc(mask) <= 3) ++few;
        if (d.rcv_pos && (m & kRcvFlag)) ++rcv;
        const int64_t node = (int64_t)(m & kNodeMask);
        for (; mask; mask &= mask - 1u) {
            const int32_t q = d.pos[node + slot_off(__ffs((int)mask) - 1, a.st1, a.st2)];
            for (int c = 0; c < kCand; ++c) far[c] += in_window(q, p1, a.C[c]) ? 0 : 1;
        }
    }
    for (int c = 0; c < kCand; ++c)
        if (far[c]) atomicAdd(&s[c], far[c]);
    if (rcv) atomicAdd(&s[kCand], rcv);
    if (few) atomicAdd(&s[kCand + 1], few);
    __syncthreads();
    if (threadIdx.x < kCand + 2) d.cnt[(size_t)l * (kCand + 2) + threadIdx.x] = s[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_ring_mark(BuildArgs a) {
    const BuildDev& d = a.dev[blockIdx.y];
    const int l = blockIdx.x;
    if (l >= d.L || d.C == 0) return;
    const int32_t p0 = d.lvl_ptr[l], p1 = d.lvl_ptr[l + 1];
    for (int32_t p = p0 + (int32_t)threadIdx.x; p < p1; p += 256) {
        const uint64_t m = d.meta[p];
        const int64_t node = (int64_t)(m & kNodeMask);
        for (uint32_t mask = (uint32_t)(m >> kMaskShift); mask; mask &= mask - 1u) {
            const int64_t u = node + slot_off(__ffs((int)mask) - 1, a.st1, a.st2);
            if (!in_window(d.pos[u], p1, d.C)) d.need[u] = 1;
        }
    }
}

// entries reserved for level l in the far list
__device__ __forceinline__ int32_t lv_end(const BuildDev& d, int l) { return d.lv[l + 1].y - d.lv[l].y; }

// slots, wide records and far lists of one level
template <typename V>
__global__ __launch_bounds__(256) void k_ring_fill(BuildArgs a) {
    const BuildDev& d = a.dev[blockIdx.y];
    const int l = blockIdx.x;
    if (l >= d.L || d.C == 0) return;
    const int32_t p0 = d.lvl_ptr[l], p1 = d.lvl_ptr[l + 1];
    const int4 lv = d.lv[l];
    const int32_t C = d.C;
    __shared__ int32_t n_far;
    if (threadIdx.x == 0) n_far = 0;
    __syncthreads();
    auto side = [&](uint32_t entry) {
        const int32_t i = atomicAdd(&n_far, 1);
        d.far[lv.y + i] = entry;
        int32_t s = lv.z + i;
        if (s >= d.F) s -= d.F;
        return (uint32_t)(C + 1 + s);
    };
    const V* wts = (const V*)d.wts;
    for (int32_t p = p0 + (int32_t)threadIdx.x; p < p1; p += 256) {
        const uint64_t m = d.meta[p];
        const int64_t node = (int64_t)(m & kNodeMask);
        uint32_t sl[6], qs = (uint32_t)C;
        int t = 0;
        for (uint32_t mask = (uint32_t)(m >> kMaskShift); mask; mask &= mask - 1u, ++t) {
            const int64_t u = node + slot_off(__ffs((int)mask) - 1, a.st1, a.st2);
            const int32_t q = d.pos[u];
            sl[t] = in_window(q, p1, C) ? (uint32_t)(q % C) : side((uint32_t)u);
        }
        const int deg = t;
        for (; t < 6; ++t) sl[t] = (uint32_t)C;
        if (d.rcv_pos && (m & kRcvFlag))
            for (int32_t e = d.rcvlvl_ptr[d.lev[l]]; e < d.rcvlvl_ptr[d.lev[l] + 1]; ++e)
                if (d.rcv_pos[e] == p) { qs = side((uint32_t)e | kRcvEntry); break; }
        const uint32_t w0 = (uint32_t)node | (d.need[node] ? kStore : 0u);
        const int32_t wide = p - (p0 + lv.w);
        if (wide < 0) {
            const V* rec = wts + (size_t)p * 4;
            d.ref[p] = uint2{sl[0] | sl[1] << 16, sl[2] | qs << 16};
            d.node[p] = w0;
            V* wa = (V*)d.wa + (size_t)p * (16 / sizeof(V));
            wa[0] = rec[1];
            wa[1] = rec[2];
            if (sizeof(V) == 8) {
                ((V*)d.wb)[p] = rec[3];
                if (d.wc) ((V*)d.wc)[p] = rec[0];
            } else {
                wa[2] = rec[3];
                wa[3] = rec[0];
            }
        } else {
            const size_t i = (size_t)lv.x + wide;
            uint32_t* rf = d.wref + i * 4;
            rf[0] = w0;
            for (int k = 0; k < 3; ++k) rf[1 + k] = sl[2 * k] | sl[2 * k + 1] << 16;
            V* o = (V*)d.wwt + i * 8;
            const V* rec = wts + (size_t)p * 4;
            const size_t ov = (size_t)a.N * 4 + (size_t)((m >> kOffShift) & kOffMask);
            for (int k = 0; k < 4; ++k) o[k] = rec[k];
            for (int k = 3; k < 6; ++k) o[1 + k] = k < deg ? wts[ov + (k - 3)] : (V)0;
            *reinterpret_cast<uint32_t*>(o + 7) = qs;
        }
    }
    // a counted receiver without entries leaves its place unused; lanes without
    // an entry load the one past the end
    if (l == d.L - 1 && threadIdx.x == 0) d.far[d.lv[d.L].y] = 0u;
    __syncthreads();
    for (int32_t i = n_far + (int32_t)threadIdx.x; i < lv_end(d, l); i += 256) d.far[lv.y + i] = 0u;
}

// Workgroup shapes: narrow, wide and far waves, narrow and wide batches in
// flight, levels that far values and their lists are loaded ahead, and far
// values per lane in flight.
struct Shape { int cw, ow, fw, d, dw, g, e, u; };
constexpr Shape kShapes[3] = {{2, 1, 1, 6, 5, 3, 6, 1}, {5, 1, 2, 6, 5, 2, 6, 2}, {8, 2, 2, 4, 4, 2, 4, 4}};

}  // namespace

struct RingPlan {
    int32_t shape = 0, n_ent = 0;
    int32_t C[2] = {0, 0}, F[2] = {0, 0};   // forward, transpose; C = 0: that direction has no window walk
    int32_t items = 0, per_xcd = 0;
    size_t lds = 0;
    int32_t stage_off = 0;
    bool pt = false;              // off-grid sources: the seed transposes read every row
    DevBlocks mem;                // the tables and q
    RingDev* dev = nullptr;       // [S][2]
    void* q = nullptr;            // inputs in level order
};

void ring_free(RingPlan* r) {
    if (!r) return;
    r->mem.release();
    delete r;
}

namespace {

template <int DIR, typename V, int SH, bool QS, bool PS>
const void* ring_fn() {
    constexpr Shape s = kShapes[SH];
    return (const void*)k_ring<DIR, V, s.cw, s.ow, s.fw, s.d, s.dw, s.g, s.e, s.u, QS, PS>;
}

template <typename V, int SH>
const void* ring_kind(int kind) {
    switch (kind) {
        case 0: return ring_fn<kFwd, V, SH, false, false>();
        case 1: return ring_fn<kRev, V, SH, false, false>();
        case 2: return ring_fn<kRev, V, SH, true, false>();
        case 3: return ring_fn<kRev, V, SH, false, true>();
    }
    return ring_fn<kRev, V, SH, true, true>();
}

template <typename V>
const void* ring_pick(int shape, int kind) {
    return shape == 0 ? ring_kind<V, 0>(kind) : shape == 1 ? ring_kind<V, 1>(kind) : ring_kind<V, 2>(kind);
}

// kind 0: primal; 1: transpose from nodes, summed; 2: from receivers, summed;
// 3, 4: the same per source
constexpr int kKinds = 5;
const void* ring_kernel(bool fp64, int shape, int kind) {
    return fp64 ? ring_pick<double>(shape, kind) : ring_pick<float>(shape, kind);
}

struct Bytes {
    size_t off = 0;
    size_t add(size_t n) {
        off = (off + 255) & ~size_t(255);
        const size_t at = off;
        off += n;
        return at;
    }
};

// The levels of one direction of one source in chunks of at most `most`
// singletons, the level's blocks with its last chunk: each is a step of the walk
// of its own, so that a wide level needs no more of the window than its own
// values and one chunk.
struct Chunks {
    std::vector<int32_t> pos, n, lev;   // first position of each and the end, singletons, level
    Chunks(const std::vector<int32_t>& ptr, const std::vector<int32_t>& nsc, int32_t most) {
        for (int32_t l = 0; l + 1 < (int32_t)ptr.size(); l++)
            for (int32_t o = 0; o == 0 || o < nsc[l]; o += most) {
                pos.push_back(ptr[l] + o);
                n.push_back(std::min(most, nsc[l] - o));
                lev.push_back(l);
            }
        pos.push_back(ptr.back());
    }
    int32_t size() const { return (int32_t)n.size(); }
    // any k consecutive chunks span at most c positions
    bool fit(int32_t k, int32_t c) const {
        const int32_t L = size();
        for (int32_t l = 0; l < L; l++)
            if (pos[std::min(l + k, L)] - pos[l] > c) return false;
        return true;
    }
};

// The walk's lists of one direction of one source.
struct Lists {
    std::vector<uint2> nd;
    std::vector<uint4> wd, fd;
    std::vector<int4> lv;      // (BuildDev::lv)
    std::vector<int32_t> bw;   // first wide record of each block's members
    int64_t n_far = 0, n_wide = 0;
};

constexpr int kPad = 16;       // half the empty batches past the end (the walk loads up to 3 D or 1 + G + 2 E ahead)

// cnt [chunks][kCand + 2] as counted, c the window taken.
Lists walk_lists(const Packed& pk, bool fwd, const Chunks& ch, const int32_t* cnt, int c, int32_t C, int32_t F,
                 const Shape& sh) {
    Lists t;
    const int NL = sh.cw * 64, OL = sh.ow * 64;
    const std::vector<int32_t>& bptr = fwd ? pk.fblk_ptr : pk.rblk_ptr;
    const std::vector<int32_t>& bid = fwd ? pk.fblk_id : pk.rblk_id;
    const std::vector<int32_t>& bpos = fwd ? pk.blk_fpos : pk.blk_rpos;
    const int32_t L = ch.size();
    t.fd.assign(sh.e, uint4{0u, 0u, 0u, 0u});
    // rows are drained every K chunks, as rarely as the window allows
    int32_t K = 16;
    while (K > 1 && !ch.fit(K + sh.g + 1, C)) --K;
    int32_t skip = 0;
    bool dirty = false;
    t.bw.assign(std::max<size_t>(pk.blk_k.size(), 1), 0);
    for (int32_t l = 0; l < L; l++, cnt += kCand + 2) {
        const int32_t p0 = ch.pos[l], p1 = ch.pos[l + 1], ns = ch.n[l];
        const int32_t few = cnt[kCand + 1], nw = ns - few, nf = cnt[c] + cnt[kCand];
        const bool blk = p1 - p0 > ns;       // members follow the singletons
        const uint32_t fl = (blk ? kBlk : 0u) | (l % K == K - 1 ? kDrain : 0u);
        t.lv.push_back(int4{(int)t.n_wide, (int)t.n_far, (int)(t.n_far % F), few});
        t.fd.push_back(uint4{(uint32_t)t.n_far, (uint32_t)nf, kLast | fl, (uint32_t)(t.n_far % F)});
        for (int32_t o = 0; o == 0 || o < few; o += NL) {
            const int32_t n = std::min(few - o, NL);
            t.nd.push_back(uint2{(uint32_t)(p0 + o),
                                 (uint32_t)n | (o + NL >= few ? kLast | fl : 0u) | (uint32_t)((p0 + o) % C) << 16});
        }
        // (a level where these waves have nothing to do is passed over: no
        // node, no block, and no store of theirs since the last drain)
        const int32_t q0 = p0 + few;
        dirty = dirty || nw > 0;
        if (nw == 0 && l + 1 < L && !(fl & kBlk) && !((fl & kDrain) && dirty)) {
            ++skip;
        } else {
            for (int32_t o = 0; o == 0 || o < nw; o += OL) {
                const int32_t n = std::min(nw - o, OL);
                t.wd.push_back(uint4{(uint32_t)(q0 + o),
                                     (uint32_t)n | (o + OL >= nw ? kLast | fl : 0u) | (uint32_t)((q0 + o) % C) << 16,
                                     (uint32_t)(t.n_wide + o), (uint32_t)skip});
                skip = 0;
            }
            if (fl & kDrain) dirty = false;
        }
        if (blk)
            for (int32_t b = bptr[ch.lev[l]]; b < bptr[ch.lev[l] + 1]; b++)
                t.bw[bid[b]] = (int32_t)(t.n_wide + nw + bpos[bid[b]] - (p0 + ns));
        // the rest of the round after a level with blocks is empty
        if (fl & kBlk) {
            while (t.nd.size() % sh.d) t.nd.push_back(uint2{0u, 0u});
            while (t.wd.size() % sh.dw) t.wd.push_back(uint4{0u, 0u, 0u, 0u});
            while (t.fd.size() % sh.e) t.fd.push_back(uint4{0u, 0u, 0u, 0u});
        }
        t.n_far += nf;
        t.n_wide += p1 - p0 - few;
    }
    t.lv.push_back(int4{(int)t.n_wide, (int)t.n_far, 0, 0});
    while (t.fd.size() % sh.e) t.fd.push_back(uint4{0u, 0u, 0u, 0u});
    // batches past the end load the first position again
    t.nd.insert(t.nd.end(), 2 * kPad, uint2{0u, 0u});
    t.wd.insert(t.wd.end(), 2 * kPad, uint4{0u, 0u, 0u, 0u});
    t.fd.insert(t.fd.end(), 2 * kPad, uint4{0u, 0u, 0u, 0u});
    return t;
}

}  // namespace

static int ring_build(const fm_batch* b, const std::vector<SrcDev>& src, RingPlan** out) {
    const int32_t S = b->S, B = b->B;
    const bool fp64 = b->prec == FM_FP64;
    const size_t vb = fp64 ? 8 : 4;
    const int64_t N = b->N;
    if (b->states[0]->stencil != 6) return FM_OK;        // up to 26 neighbours: no fixed record
    // 32-bit byte offsets inside one source's and one group's arrays
    if ((uint64_t)N * std::max<uint64_t>({(uint64_t)b->xB * vb, 64u}) >= (1ull << 32)) return FM_OK;
    int32_t minL = 1 << 30;
    int64_t stage_rows = 0;    // FP64 rows a block stages: b and partial sums, or b and two iterates
    size_t n_ent = 0;
    bool pt = false;
    for (const HostState* st : b->states) {
        const Packed& pk = st->pk;
        for (int32_t i = 0; i < pk.nblk; i++) {
            const int64_t rows = block_stage_rows(pk, i);
            stage_rows = std::max(stage_rows, pk.blk_it[2 * (size_t)i] ? rows : rows + 1024);
        }
        minL = std::min({minL, pk.L_f, pk.L_r});
        n_ent = std::max(n_ent, pk.rcv_node.size());
        pt = pt || !pk.seed_node.empty();
    }
    if (n_ent * B * vb >= (1ull << 32)) return FM_OK;
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b->device));
    // The workgroup by the mean level width: about two batches of the narrow
    // waves a level.  A barrier costs more the more waves meet at it, and a wave
    // without nodes only waits; 81x41 (width 48): 57 us with 4 waves, 67x53x31
    // (300): 335 us with 8, 101x101x51 (450): 1.03 ms with 12.
    const int64_t width = N / std::max(minL, 1);
    const int shape = width <= 160 ? 0 : width <= 400 ? 1 : 2;
    const Shape sh = kShapes[shape];
    // (several small workgroups share a CU: their LDS windows are a share of it)
    const int max_occ = shape == 0 ? 4 : shape == 1 ? 2 : 1;
    const int64_t pairs = (int64_t)S * B;
    const int occ = (int)std::min<int64_t>(std::max<int64_t>((pairs + cus - 1) / cus, 1), max_occ);
    // At most two rounds of workgroups.  J of the node split and of the walk,
    // then J^T, FP64, for each of the three workgroups; two rounds: 101x101x51, 32
    // sources x 16 right-hand sides, 3.23 and 2.62, 4.24 and 3.65 ms; 53x47x25,
    // 32 x 32, 1.31 and 1.00, 1.57 and 1.33; 401x201, 64 x 32, 3.32 and 1.81, 3.68
    // and 2.16.  Three rounds break even and take tables and inputs of their own:
    // 48 x 16, 4.25 and 3.97, 5.61 and 5.52; 48 x 32, 1.37 and 1.41, 1.69 and 1.82;
    // 96 x 32, 3.31 and 3.30, 3.90 and 3.77.
    if (pairs > (int64_t)cus * occ * 2) return FM_OK;
    const size_t budget = (size_t)160 * 1024 / occ - 512;
    const size_t stage = (size_t)stage_rows * sizeof(double);
    if (stage + 4096 > budget) return FM_OK;
    const int64_t slots = std::min<int64_t>((int64_t)((budget - stage) / vb) - 1, 65535 - 2);
    // side windows tried: 1/16, 1/8 and 1/4 of the slots
    int32_t C[kCand], F[kCand];
    for (int c = 0; c < kCand; c++) {
        F[c] = (int32_t)std::max<int64_t>(slots >> (4 - c), 1);
        C[c] = (int32_t)(slots - F[c]);
    }
    const int nd = 2 * S;
    // far references need the same positions in every direction of every
    // source: temporary buffers of the passes below
    Bytes tb;
    std::vector<BuildDev> bd(nd);
    std::vector<Chunks> ch;
    int32_t max_c = 0;
    for (int i = 0; i < nd; i++) {
        const Packed& pk = b->states[i / 2]->pk;
        if (i % 2 == 0) ch.emplace_back(pk.flvl_ptr, pk.flvl_nsc, 2 * sh.cw * 64);
        else ch.emplace_back(pk.rlvl_ptr, pk.rlvl_nsc, 2 * sh.cw * 64);
        // a far value is drained and loaded between its chunk and its reader's:
        // K + G + 1 chunks have to fit (K = 1 drains every chunk)
        if (!ch[i].fit(sh.g + 2, C[0])) return FM_OK;
        max_c = std::max(max_c, ch[i].size());
    }
    std::vector<size_t> o_cp(nd), o_cn(nd), o_cl(nd);
    for (int i = 0; i < nd; i++) {
        o_cp[i] = tb.add(sizeof(int32_t) * ch[i].pos.size());
        o_cn[i] = tb.add(sizeof(int32_t) * ch[i].n.size());
        o_cl[i] = tb.add(sizeof(int32_t) * ch[i].lev.size());
    }
    const size_t o_bd = tb.add(sizeof(BuildDev) * nd);
    const size_t head_end = tb.off;
    std::vector<size_t> o_cnt(nd);
    size_t n_cnt = 0;
    for (int i = 0; i < nd; i++) {
        o_cnt[i] = n_cnt;
        n_cnt += (kCand + 2) * ch[i].n.size();
    }
    struct Temp {
        DevBlocks mem;
        char* head = nullptr;
        int32_t *pos = nullptr, *cnt = nullptr;   // pos [nd][N]
        uint8_t* need = nullptr;                  // [nd][N]
        ~Temp() { mem.release(); }
    } temp;
    std::unique_ptr<RingPlan, void (*)(RingPlan*)> r(new RingPlan(), ring_free);
    // no window walk where its tables and inputs do not fit; other errors are reported
    auto give_up = [&](hipError_t err) -> int {
        if (err == hipSuccess || err == hipErrorOutOfMemory) { (void)hipGetLastError(); return FM_OK; }
        set_error("window tables of the batch failed: %s", hipGetErrorString(err));
        return FM_EHIP;
    };
    hipError_t e = temp.mem.take({{(void**)&temp.head, head_end}, {(void**)&temp.pos, sizeof(int32_t) * N * nd},
                                  {(void**)&temp.need, (size_t)N * nd}, {(void**)&temp.cnt, sizeof(int32_t) * n_cnt}});
    if (e != hipSuccess) return give_up(e);
    char* const tmp = temp.head;
    for (int i = 0; i < nd; i++) {
        const SrcDev& d = src[i / 2];
        const bool fwd = i % 2 == 0;
        BuildDev& x = bd[i];
        memset(&x, 0, sizeof(x));
        x.meta = fwd ? d.fmeta : d.rmeta;
        x.wts = fwd ? d.fwts : d.rwts;
        x.lvl_ptr = (const int32_t*)(tmp + o_cp[i]);
        x.lvl_nsc = (const int32_t*)(tmp + o_cn[i]);
        x.lev = (const int32_t*)(tmp + o_cl[i]);
        x.rcvlvl_ptr = fwd ? nullptr : d.rcvlvl_ptr;
        x.rcv_pos = fwd || d.n_ent == 0 ? nullptr : d.rcv_pos;
        x.rcv_node = d.rcv_node;
        x.n_rcv_node = fwd ? d.n_ent : 0;
        x.L = ch[i].size();
        x.pos = temp.pos + (size_t)i * N;
        x.need = temp.need + (size_t)i * N;
        x.cnt = temp.cnt + o_cnt[i];
    }
    BuildArgs ba{};
    ba.dev = (const BuildDev*)(tmp + o_bd);
    ba.N = N;
    ba.st1 = b->st1;
    ba.st2 = b->st2;
    for (int c = 0; c < kCand; c++) ba.C[c] = C[c];
    {
        std::vector<char> head(head_end);
        for (int i = 0; i < nd; i++) {
            memcpy(head.data() + o_cp[i], ch[i].pos.data(), sizeof(int32_t) * ch[i].pos.size());
            memcpy(head.data() + o_cn[i], ch[i].n.data(), sizeof(int32_t) * ch[i].n.size());
            memcpy(head.data() + o_cl[i], ch[i].lev.data(), sizeof(int32_t) * ch[i].lev.size());
        }
        memcpy(head.data() + o_bd, bd.data(), sizeof(BuildDev) * nd);
        e = hipMemcpy(tmp, head.data(), head_end, hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) return give_up(e);
    const int gx = (int)std::min<int64_t>((N + 255) / 256, 4096);
    hipLaunchKernelGGL(k_ring_clear, dim3(gx, nd), dim3(256), 0, nullptr, ba);
    hipLaunchKernelGGL(k_ring_pos, dim3(gx, nd), dim3(256), 0, nullptr, ba);
    hipLaunchKernelGGL(k_ring_count, dim3(max_c, nd), dim3(256), 0, nullptr, ba);
    std::vector<int32_t> cnt(n_cnt);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpy(cnt.data(), temp.cnt, sizeof(int32_t) * n_cnt, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return give_up(e);
    auto count = [&](int i, int32_t l, int c) {
        return cnt[o_cnt[i] + (size_t)l * (kCand + 2) + c];
    };
    // Per direction the smallest side window that holds the entries of any two
    // consecutive chunks, taken where few enough neighbours are far: a far value
    // is a row of its own from the L2 or memory for every pair.  Far values per
    // node, the time of the schedule that runs otherwise and of the walk, FP64.
    // Node split, J: 0.03 (101x101x51, 16 sources x 16 right-hand sides) 2.95 and
    // 1.38 ms, 0.13 (121x121x61, 8 x 8) 3.49 and 2.33, 0.36 (141x141x71, 8 x 16)
    // 5.55 and 5.31, 0.35 (201x201x51, 8 x 16) 6.65 and 7.79, 0.54 (161x161x81, 8 x
    // 16) 7.37 and 8.92; J^T: 0.10 3.69 and 1.85, 0.11 4.13 and 3.35, 0.13 and 0.23
    // (141x141x71, two placements of the sources) 4.9 and 3.7, 6.8 and 4.2, so that
    // the line is on the safe side there.  Right-hand-side groups, 8 x 1, J: 0.35
    // 17.1 and 8.5, 0.36 12.0 and 5.4, 0.54 17.5 and 9.5, 0.69 16.7 and 14.1; J^T: 0.13
    // 10.3 and 4.6, 0.20 14.5 and 6.7, 0.38 13.4 and 15.5.
    const double far_max[2] = {b->tun.split > 1 ? 0.2 : 0.5, b->tun.split > 1 ? 0.2 : 0.3};
    int pick[2] = {-1, -1};
    for (int dir = 0; dir < 2; dir++) {
        for (int c = 0; c < kCand && pick[dir] < 0; c++) {
            bool ok = true;
            int64_t far = 0;
            for (int i = dir; i < nd && ok; i += 2) {
                const int32_t L = bd[i].L;
                for (int32_t l = 0; l < L && ok; l++) {
                    int64_t two = 0;
                    for (int32_t m = l; m < std::min(l + 2, L); m++) two += count(i, m, c) + count(i, m, kCand);
                    far += count(i, l, c);
                    ok = two <= F[c];
                }
                ok = ok && ch[i].fit(sh.g + 2, C[c]);
            }
            if (ok && (double)far <= far_max[dir] * (double)S * (double)N) pick[dir] = c;
        }
        if (pick[dir] < 0) continue;
        r->C[dir] = C[pick[dir]];
        r->F[dir] = F[pick[dir]];
        for (int i = dir; i < nd; i += 2) {
            bd[i].C = r->C[dir];
            bd[i].F = r->F[dir];
        }
    }
    if (pick[0] < 0 && pick[1] < 0) return give_up(hipSuccess);
    r->shape = shape;
    r->n_ent = (int32_t)n_ent;
    r->items = S * B;
    r->per_xcd = (r->items + 7) / 8;
    r->pt = pt;
    const size_t win = (((size_t)(std::max(r->C[0] + r->F[0], r->C[1] + r->F[1]) + 1) * vb) + 15) & ~size_t(15);
    r->stage_off = (int32_t)win;
    r->lds = win + stage;
    std::vector<Lists> li(nd);
    for (int i = 0; i < nd; i++)
        if (bd[i].C)
            li[i] = walk_lists(b->states[i / 2]->pk, i % 2 == 0, ch[i], cnt.data() + o_cnt[i], pick[i % 2], bd[i].C,
                               bd[i].F, sh);
    Bytes pb;
    const size_t o_dev = pb.add(sizeof(RingDev) * nd), o_build = pb.add(sizeof(BuildDev) * nd);
    std::vector<size_t> o_nd(nd), o_wd(nd), o_fd(nd), o_lv(nd), o_bw(nd), o_lev(nd);
    for (int i = 0; i < nd; i++) {
        if (!bd[i].C) continue;
        o_nd[i] = pb.add(sizeof(uint2) * li[i].nd.size());
        o_wd[i] = pb.add(sizeof(uint4) * li[i].wd.size());
        o_fd[i] = pb.add(sizeof(uint4) * li[i].fd.size());
        o_lv[i] = pb.add(sizeof(int4) * li[i].lv.size());
        o_bw[i] = pb.add(sizeof(int32_t) * li[i].bw.size());
        o_lev[i] = pb.add(sizeof(int32_t) * ch[i].lev.size());
    }
    const size_t host_end = pb.add(0);
    // one array per stream over all sources (every source on a 256-byte boundary)
    Bytes st_ref, st_node, st_wa, st_wb, st_wc, st_wref, st_wwt, st_far;
    std::vector<size_t> o_ref(nd), o_node(nd), o_wa(nd), o_wb(nd), o_wc(nd), o_wref(nd), o_wwt(nd), o_far(nd);
    for (int i = 0; i < nd; i++) {
        if (!bd[i].C) continue;
        o_ref[i] = st_ref.add((size_t)N * 8);
        o_node[i] = st_node.add((size_t)N * 4);
        o_wa[i] = st_wa.add((size_t)N * 16);
        o_wb[i] = st_wb.add(fp64 ? (size_t)N * 8 : 0);
        o_wc[i] = st_wc.add(fp64 && i % 2 ? (size_t)N * 8 : 0);
        o_wref[i] = st_wref.add((size_t)(li[i].n_wide + 1) * 16);
        o_wwt[i] = st_wwt.add((size_t)(li[i].n_wide + 1) * 8 * vb);
        o_far[i] = st_far.add((size_t)(li[i].n_far + 1) * 4);
    }
    // at most a quarter of the free memory: a program that sized its own arrays
    // by a batch's scratch rows keeps its room
    const size_t q_bytes = std::max((size_t)S * N * B, (size_t)S * n_ent * B) * vb + 256;
    char *tab = nullptr, *ref = nullptr, *node = nullptr, *wa = nullptr, *wb = nullptr, *wc = nullptr, *wref = nullptr,
         *wwt = nullptr, *far = nullptr;
    const std::vector<Part> parts = {{(void**)&tab, host_end}, {(void**)&ref, st_ref.off}, {(void**)&node, st_node.off},
                                     {(void**)&wa, st_wa.off}, {(void**)&wb, st_wb.off}, {(void**)&wc, st_wc.off},
                                     {(void**)&wref, st_wref.off}, {(void**)&wwt, st_wwt.off},
                                     {(void**)&far, st_far.off}, {&r->q, q_bytes}};
    size_t all = 0;
    for (const Part& x : parts) all += x.bytes;
    size_t mem_free = 0, mem_total = 0;
    e = hipMemGetInfo(&mem_free, &mem_total);
    if (e != hipSuccess || all > mem_free / 4) return give_up(e);
    e = r->mem.take(parts);
    if (e != hipSuccess) return give_up(e);
    r->dev = (RingDev*)(tab + o_dev);
    std::vector<char> hb(host_end);
    std::vector<RingDev> rd(nd);
    for (int i = 0; i < nd; i++) {
        if (!bd[i].C) continue;
        memcpy(hb.data() + o_nd[i], li[i].nd.data(), sizeof(uint2) * li[i].nd.size());
        memcpy(hb.data() + o_wd[i], li[i].wd.data(), sizeof(uint4) * li[i].wd.size());
        memcpy(hb.data() + o_fd[i], li[i].fd.data(), sizeof(uint4) * li[i].fd.size());
        memcpy(hb.data() + o_lv[i], li[i].lv.data(), sizeof(int4) * li[i].lv.size());
        memcpy(hb.data() + o_bw[i], li[i].bw.data(), sizeof(int32_t) * li[i].bw.size());
        memcpy(hb.data() + o_lev[i], ch[i].lev.data(), sizeof(int32_t) * ch[i].lev.size());
        rd[i].ref = (const uint2*)(ref + o_ref[i]);
        rd[i].node = (const uint32_t*)(node + o_node[i]);
        rd[i].wa = wa + o_wa[i];
        rd[i].wb = wb + o_wb[i];
        rd[i].wc = wc + o_wc[i];
        rd[i].wref = (const uint32_t*)(wref + o_wref[i]);
        rd[i].wwt = wwt + o_wwt[i];
        rd[i].nd = (const uint2*)(tab + o_nd[i]);
        rd[i].wd = (const uint4*)(tab + o_wd[i]);
        rd[i].fd = (const uint4*)(tab + o_fd[i]);
        rd[i].far = (const uint32_t*)(far + o_far[i]);
        rd[i].blk_w = (const int32_t*)(tab + o_bw[i]);
        rd[i].n_nd = (int32_t)li[i].nd.size() - 2 * kPad;
        rd[i].n_wd = (int32_t)li[i].wd.size() - 2 * kPad;
        rd[i].n_fd = (int32_t)li[i].fd.size() - 2 * kPad - sh.e;
        rd[i].lev = (const int32_t*)(tab + o_lev[i]);
        bd[i].ref = (uint2*)(ref + o_ref[i]);
        bd[i].node = (uint32_t*)(node + o_node[i]);
        bd[i].wa = wa + o_wa[i];
        bd[i].wb = fp64 ? wb + o_wb[i] : nullptr;
        bd[i].wc = fp64 && i % 2 ? wc + o_wc[i] : nullptr;
        bd[i].wref = (uint32_t*)(wref + o_wref[i]);
        bd[i].wwt = wwt + o_wwt[i];
        bd[i].far = (uint32_t*)(far + o_far[i]);
        bd[i].lv = (const int4*)(tab + o_lv[i]);
    }
    memcpy(hb.data() + o_dev, rd.data(), sizeof(RingDev) * nd);
    memcpy(hb.data() + o_build, bd.data(), sizeof(BuildDev) * nd);
    e = hipMemcpy(tab, hb.data(), host_end, hipMemcpyHostToDevice);
    if (e != hipSuccess) return give_up(e);
    ba.dev = (const BuildDev*)(tab + o_build);
    hipLaunchKernelGGL(k_ring_mark, dim3(max_c, nd), dim3(256), 0, nullptr, ba);
    if (fp64) hipLaunchKernelGGL(k_ring_fill<double>, dim3(max_c, nd), dim3(256), 0, nullptr, ba);
    else hipLaunchKernelGGL(k_ring_fill<float>, dim3(max_c, nd), dim3(256), 0, nullptr, ba);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    for (int kind = 0; kind < kKinds && e == hipSuccess; kind++)
        e = hipFuncSetAttribute(ring_kernel(fp64, shape, kind), hipFuncAttributeMaxDynamicSharedMemorySize,
                                160 * 1024);
    if (e != hipSuccess) return give_up(e);
    *out = r.release();
    return FM_OK;
}

int ring_create(const fm_batch* b, const std::vector<SrcDev>& src, RingPlan** out) {
    *out = nullptr;
    try {
        return ring_build(b, src, out);
    } catch (const std::bad_alloc&) {
        return FM_OK;        // the other kernels need no tables
    }
}

template <typename V>
static void ring_inputs(const fm_batch* b, bool fwd, const ApplyArgs& a, const RingArgs& ra, const RingPlan* r) {
    if (!fwd && a.in_mode == FM_W_RECEIVERS) {
        const int g = (int)std::min<int64_t>(((int64_t)std::max(r->n_ent, 1) * a.B + 255) / 256, 1024);
        hipLaunchKernelGGL(k_ring_rcv<V>, dim3(g, a.S), dim3(256), 0, b->stream, a, ra, (V*)r->q);
        return;
    }
    const dim3 grid((unsigned)((a.N + kPermRows - 1) / kPermRows), a.S);
    // columns at a time: a whole row up to 16
    const auto fn = a.B > 8   ? (fwd ? k_ring_q<kFwd, V, 16> : k_ring_q<kRev, V, 16>)
                    : a.B > 4 ? (fwd ? k_ring_q<kFwd, V, 8> : k_ring_q<kRev, V, 8>)
                    : a.B > 1 ? (fwd ? k_ring_q<kFwd, V, 4> : k_ring_q<kRev, V, 4>)
                              : (fwd ? k_ring_q<kFwd, V, 1> : k_ring_q<kRev, V, 1>);
    hipLaunchKernelGGL(fn, grid, dim3(kPermRows), 0, b->stream, a, ra, (V*)r->q);
}

bool ring_has(const RingPlan* r, bool fwd) { return r && r->C[fwd ? 0 : 1] > 0; }

void ring_sizes(const RingPlan* r, bool fwd, int32_t* threads, int32_t* window, int32_t* side) {
    const Shape sh = kShapes[r->shape];
    *threads = (sh.cw + sh.ow + sh.fw) * 64;
    *window = r->C[fwd ? 0 : 1];
    *side = r->F[fwd ? 0 : 1];
}

hipError_t ring_walk(const fm_batch* b, bool fwd, const ApplyArgs& a0) {
    const RingPlan* r = b->ring;
    const bool fp64 = b->prec == FM_FP64;
    ApplyArgs a = a0;
    a.items = r->items;
    a.per_xcd = r->per_xcd;
    RingArgs ra{};
    ra.dev = r->dev;
    ra.q = r->q;
    ra.C = r->C[fwd ? 0 : 1];
    ra.F = r->F[fwd ? 0 : 1];
    ra.stage_off = r->stage_off;
    ra.n_ent = r->n_ent;
    // rows every node writes: the output itself, the source sum's input, and
    // the rows the seed transposes read; otherwise far targets and receivers
    ra.store_all = fwd ? a.out_mode == FM_OUT_NODES : a.out_mode == FM_JT_SUMMED || r->pt;
    ra.xmask = b->sync ? b->sync + (size_t)b->S * 32 : nullptr;
    if (fp64) ring_inputs<double>(b, fwd, a, ra, r);
    else ring_inputs<float>(b, fwd, a, ra, r);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int kind = fwd ? 0 : (a.in_mode == FM_W_RECEIVERS ? 2 : 1) + (a.out_mode == FM_JT_PER_SOURCE ? 2 : 0);
    const Shape sh = kShapes[r->shape];
    void* args[] = {&a, &ra};
    e = hipLaunchKernel(ring_kernel(fp64, r->shape, kind), dim3(8 * r->per_xcd), dim3((sh.cw + sh.ow + sh.fw) * 64),
                        args, r->lds, b->stream);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace fm
