// Direct-gather accumulators (kernels and their launchers, for one problem
// or, MULTI, a batch): expand-sort-compress (Section 4) of every output
// column, with the column's products gathered straight from A through its
// stored B entries, in two modes sharing one code path:
//   COUNT  (symbolic phase): the number of distinct rows of every column;
//   FILL   (numeric phase):  the rows in ascending order and their values,
//          each summed in Algorithm 1's order (B's stored order, starting from
//          zero, every product and sum rounded on its own), written
//          contiguously at the column's place in C.
// Nothing per product is kept between the phases.
//
// Wave buffer. A wavefront holds N = 64 KPL positions. The columns of a work
// item occupy aligned segments of S positions: S / KPL neighbouring lanes, KPL
// rows of them. A column's products fill its segment row by row in the order
// Algorithm 1 meets them (stored B entries in storage order, then the rows of
// the selected A column in storage order); the rest of the segment is padding
// that sorts last.
//
// Gather. A product's address in A is (start of its entry's A column) +
// (its position) - (the entry's first position). The wave writes that
// difference and the entry's B value (a "head") at the first position of every
// stored B entry, and of every further row the entry reaches; a position's head
// is the last one at or before it in its row, found from one ballot per row.
// All of a lane's loads of A are then independent and issued together, and
// neighbouring lanes read neighbouring entries of one A column.
//
// Sort and compress. Keys (row << 11 | position) are sorted inside every
// segment by a bitonic network on registers and lanes (DPP, ds_swizzle,
// ds_bpermute), or, where one column fills the buffer, by order-preserving
// buckets in LDS. Equal rows form runs whose positions are in Algorithm 1's
// order; a run's values are added in that order.
//
// Heavy columns (more products than a wave buffer holds) are cut into row
// windows of equal span, each an independent wave work item that compacts the
// window's products (from a per-column expansion into a scratch area) into its
// buffer; a window that still overflows is halved in row span.
#pragma once

#include <climits>

#include "devutil.h"

namespace spg {

constexpr int kKeyBits = 11;          // position bits of a key (N <= 2048)
constexpr int kHeavyBin = BIN_SORT2;  // first bin of the heavy columns (above 1024 products)
constexpr int kHeadNone = INT_MIN;    // no head at this position

// Device memory that no launch changes while this one runs (the header's bin
// positions, the problem table): read through the scalar cache, one load for
// the wavefront. The header's error words sit beside the positions; a flag
// raised while a kernel runs stops the kernels after it.
template <typename T>
using cmem = const __attribute__((address_space(4))) T;

struct BinRange {
    int first, count;  // positions in the bin list
    bool stop;         // an error (or, filling, too small a C): nothing to do
};
template <bool FILL>
__device__ __forceinline__ BinRange bin_range(const KArgs &a, int b0, int b1) {
    cmem<Hdr> *h = (cmem<Hdr> *)a.hdr;
    const int first = h->bin_start[b0], last = h->bin_start[b1] + h->bin_count[b1];
    return {first, last - first, (h->err | (FILL ? h->cap_over : 0)) != 0};
}

// Problem of global column g (the same in every lane): a single problem's
// arguments lie in scalar registers, a batch's in the device table.
template <bool MULTI>
__device__ __forceinline__ Prob prob_of(const KArgs &a, int g) {
    if constexpr (!MULTI) {
        return a.single;
    } else {
        cmem<int32_t> *c = (cmem<int32_t> *)a.col0s;
        const int gu = __builtin_amdgcn_readfirstlane(g);
        int lo = 0, hi = a.nprob;  // last problem that starts at or before g
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (c[mid] <= gu) lo = mid;
            else hi = mid;
        }
        cmem<Prob> *t = (cmem<Prob> *)a.table + lo;
        Prob d;
        d.m = t->m; d.k = t->k; d.n = t->n; d.col0 = t->col0;
        d.nnza = t->nnza; d.nnzb = t->nnzb; d.ebase = t->ebase;
        d.acp = t->acp; d.ari = t->ari; d.av = t->av;
        d.bcp = t->bcp; d.bri = t->bri; d.bv = t->bv;
        d.ccp = t->ccp; d.cri = t->cri; d.cv = t->cv;
        return d;
    }
}

__device__ __forceinline__ void wsync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename K>
struct KeyTraits;
template <>
struct KeyTraits<unsigned> {
    static constexpr unsigned kmax = ~0u;
};
template <>
struct KeyTraits<unsigned long long> {
    static constexpr unsigned long long kmax = ~0ull;
};

// Median of three unsigned 32-bit values where c is 0 (the smaller of x and
// y) or all ones (the larger): one v_med3_u32 takes a compare-exchange's side
// chosen per lane.
// (Written as the instruction itself: spelled as min and max, the network's
// chains of them send the compiler's combiner into a very long search.)
__device__ __forceinline__ unsigned med3u(unsigned x, unsigned y, unsigned c) {
    unsigned r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(c));
    return r;
}

// compare-exchange of two registers of one lane
__device__ __forceinline__ void minmax(unsigned &lo, unsigned &hi) {
    unsigned a, b;
    asm("v_min_u32 %0, %2, %3\n\tv_max_u32 %1, %2, %3" : "=&v"(a), "=v"(b) : "v"(lo), "v"(hi));
    lo = a;
    hi = b;
}
__device__ __forceinline__ void minmax(unsigned long long &lo, unsigned long long &hi) {
    const bool sw = lo > hi;
    const unsigned long long a = sw ? hi : lo, b = sw ? lo : hi;
    lo = a;
    hi = b;
}

// Four registers of a cross-lane stage whose exchange is a DPP move: each
// register takes the median of itself, the other lane's register (its own
// number, or with `flip` the mirrored one) and c. The moves, the wait that
// DPP reads need after a VALU write and the medians are one block: the
// compiler does not see the medians' writes as a hazard for its own moves.
#define SPG_DPP_BLOCK(CTRL, S0, S1, S2, S3)                                    \
    asm volatile(                                                              \
        "s_nop 1\n\t"                                                          \
        "v_mov_b32_dpp %4, " S0 " " CTRL " row_mask:0xf bank_mask:0xf\n\t"     \
        "v_mov_b32_dpp %5, " S1 " " CTRL " row_mask:0xf bank_mask:0xf\n\t"     \
        "v_mov_b32_dpp %6, " S2 " " CTRL " row_mask:0xf bank_mask:0xf\n\t"     \
        "v_mov_b32_dpp %7, " S3 " " CTRL " row_mask:0xf bank_mask:0xf\n\t"     \
        "v_med3_u32 %0, %0, %4, %8\n\t"                                        \
        "v_med3_u32 %1, %1, %5, %8\n\t"                                        \
        "v_med3_u32 %2, %2, %6, %8\n\t"                                        \
        "v_med3_u32 %3, %3, %7, %8"                                            \
        : "+v"(k0), "+v"(k1), "+v"(k2), "+v"(k3), "=&v"(t0), "=&v"(t1),        \
          "=&v"(t2), "=&v"(t3)                                                 \
        : "v"(c))

template <int MASK, bool FLIP>
__device__ __forceinline__ void dpp_block(unsigned &k0, unsigned &k1, unsigned &k2, unsigned &k3,
                                          unsigned c) {
    unsigned t0, t1, t2, t3;
    if constexpr (MASK == 1 && FLIP) SPG_DPP_BLOCK("quad_perm:[1,0,3,2]", "%3", "%2", "%1", "%0");
    else if constexpr (MASK == 1) SPG_DPP_BLOCK("quad_perm:[1,0,3,2]", "%0", "%1", "%2", "%3");
    else if constexpr (MASK == 2) SPG_DPP_BLOCK("quad_perm:[2,3,0,1]", "%0", "%1", "%2", "%3");
    else if constexpr (MASK == 3) SPG_DPP_BLOCK("quad_perm:[3,2,1,0]", "%3", "%2", "%1", "%0");
    else if constexpr (MASK == 7) SPG_DPP_BLOCK("row_half_mirror", "%3", "%2", "%1", "%0");
    else if constexpr (MASK == 15) SPG_DPP_BLOCK("row_mirror", "%3", "%2", "%1", "%0");
    else SPG_DPP_BLOCK("row_ror:8", "%0", "%1", "%2", "%3");  // exchange at distance 8
}
#undef SPG_DPP_BLOCK

// One compare-exchange stage across lanes: with the lane whose number differs
// in the bits of MASK, register r against register r, or (FLIP) KPL - 1 - r.
// The lane with the highest differing bit clear keeps the smaller keys.
template <typename K, int KPL, int MASK, bool FLIP>
__device__ __forceinline__ void lane_stage(K (&key)[KPL], int lane) {
    constexpr int TOP = FLIP ? (MASK + 1) / 2 : MASK;
    if constexpr (sizeof(K) == 4) {
        // all ones in the lanes with the bit set, else 0
        const unsigned c = (unsigned)(((int)((unsigned)lane << (31 - __builtin_ctz(TOP)))) >> 31);
        if constexpr (MASK <= 3 || MASK == 7 || MASK == 8 || MASK == 15) {
            static_assert(KPL % 4 == 0, "the exchange blocks take four registers");
#pragma unroll
            for (int r = 0; r < KPL / 2; r += 2) {
                if constexpr (FLIP)
                    dpp_block<MASK, true>(key[r], key[r + 1], key[KPL - 2 - r], key[KPL - 1 - r], c);
                else
                    dpp_block<MASK, false>(key[2 * r], key[2 * r + 1], key[2 * r + 2],
                                           key[2 * r + 3], c);
            }
        } else {
            unsigned o[KPL];
#pragma unroll
            for (int r = 0; r < KPL; ++r)
                o[r] = (unsigned)shfl_xor_c<MASK>((int)key[FLIP ? KPL - 1 - r : r]);
#pragma unroll
            for (int r = 0; r < KPL; ++r) key[r] = med3u(key[r], o[r], c);
        }
    } else {
        const bool take_max = (lane & TOP) != 0;
        K o[KPL];
#pragma unroll
        for (int r = 0; r < KPL; ++r) o[r] = shfl_xor_c64<MASK>(key[FLIP ? KPL - 1 - r : r]);
#pragma unroll
        for (int r = 0; r < KPL; ++r)
            key[r] = (key[r] < o[r]) != take_max ? key[r] : o[r];
    }
}

// Every aligned segment of S positions sorted ascending, position KPL lane + r
// in register r. Bitonic merges whose first stage compares a position with
// its mirror image in the merge (so every merge and every stage is ascending,
// a register exchange is one min and one max, and the first stage of a merge
// of 2, 4, 8 or 16 lanes is a DPP move).
template <typename K, int KPL, int S>
__device__ __forceinline__ void seg_sort(K (&key)[KPL], int lane_in) {
    // The masks below depend on the lane only: an opaque copy of the lane
    // number keeps them from being computed once outside the caller's loop
    // and held in registers for the whole kernel.
    int lane = lane_in;
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int k = 2; k <= S; k <<= 1) {
        if (k <= KPL) {
#pragma unroll
            for (int r = 0; r < KPL; ++r)
                if ((r & (k - 1)) < k / 2) minmax(key[r], key[r ^ (k - 1)]);
        } else {
            switch (k / KPL) {
                case 2: lane_stage<K, KPL, 1, true>(key, lane); break;
                case 4: lane_stage<K, KPL, 3, true>(key, lane); break;
                case 8: lane_stage<K, KPL, 7, true>(key, lane); break;
                case 16: lane_stage<K, KPL, 15, true>(key, lane); break;
                case 32: lane_stage<K, KPL, 31, true>(key, lane); break;
                default: lane_stage<K, KPL, 63, true>(key, lane); break;
            }
        }
#pragma unroll
        for (int j = k >> 2; j > 0; j >>= 1) {
            if (j < KPL) {
#pragma unroll
                for (int r = 0; r < KPL; ++r)
                    if (!(r & j)) minmax(key[r], key[r | j]);
            } else {
                switch (j / KPL) {
                    case 1: lane_stage<K, KPL, 1, false>(key, lane); break;
                    case 2: lane_stage<K, KPL, 2, false>(key, lane); break;
                    case 4: lane_stage<K, KPL, 4, false>(key, lane); break;
                    case 8: lane_stage<K, KPL, 8, false>(key, lane); break;
                    default: lane_stage<K, KPL, 16, false>(key, lane); break;
                }
            }
        }
    }
    // the caller's first move across lanes reads the last register, whose
    // write (inside an asm block) the compiler does not count as a hazard
    if constexpr (sizeof(K) == 4) asm volatile("s_nop 1" : "+v"(key[KPL - 1]), "+v"(key[0]));
}

// A buffer that is one segment, 32-bit keys: sorted by an order-preserving
// spread of the rows over as many buckets as the buffer has positions (counts
// by LDS atomics, their prefix sums, every key to its bucket), then as many
// odd-even exchanges of neighbours as the fullest bucket holds keys. For rows
// spread evenly over their span the fullest of 1024 buckets holds 5 or 6 keys,
// about 390 vector instructions against the 1216 of the bitonic network; a
// fuller bucket than kBucketMax (rows in a few clusters, or many products per
// row) leaves the keys as they were, for the network. The waves were bound by
// the network's vector instructions: 1024-product waves of a batch 384 -> 357
// us, counting 214 -> 172 us (with the smaller buffer below 341 and 140 us).
// What the attempt costs where it is given up, numeric phases, against the
// network alone: 20,000 columns of a band of 20, 23 and 30 (10 to 15 products a
// row) 42 and 37, 85 and 74, 86 and 77 us, blocks of 32 79 and 61, a 27-point
// stencil squared 114 and 100, rows drawn by u^4 26 and 24. What it gains where
// the rows spread: 10,000 columns of 22 24.3 and 25.4, 4096 of 40 64 and 68,
// windows on clusters, bands and blocks (narrow, so their rows spread) 104 and
// 112, 386 and 416, 496 and 527.
//   key: all ones where there is none; rows in [lo, lo + span); buf: 64 KPL
//   words.
constexpr int kBucketMax = 12;
template <int KPL>
__device__ __forceinline__ bool bucket_sort(unsigned (&key)[KPL], unsigned lo, unsigned span,
                                            int *buf, int lane) {
    constexpr int N = 64 * KPL;
    constexpr unsigned KMAX = ~0u;
    // (a float product rounds monotonically: larger rows, no smaller bucket)
    const float scale = (float)N * __builtin_amdgcn_rcpf((float)span);
#pragma unroll
    for (int r = 0; r < KPL; r += 4)
        *(int4 *)(buf + lane * KPL + r) = make_int4(0, 0, 0, 0);
    wsync();
    int b[KPL], at[KPL];
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        at[r] = 0;
        b[r] = min((int)((float)((key[r] >> kKeyBits) - lo) * scale), N - 1);
        if (key[r] != KMAX) at[r] = atomicAdd(&buf[b[r]], 1);
    }
    wsync();
    int cnt[KPL], sum = 0, most = 0;
#pragma unroll
    for (int r = 0; r < KPL; r += 4) {
        const int4 x = *(const int4 *)(buf + lane * KPL + r);
        cnt[r] = x.x;
        cnt[r + 1] = x.y;
        cnt[r + 2] = x.z;
        cnt[r + 3] = x.w;
    }
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        sum += cnt[r];
        most = max(most, cnt[r]);
    }
    const int inc = wave_incl_scan(sum);
    const int total = __builtin_amdgcn_readlane(inc, 63);
    const int fullest = __builtin_amdgcn_readlane(wave_incl_max(most), 63);
    if (fullest > kBucketMax) {
        wsync();
        return false;
    }
    int run = inc - sum;
#pragma unroll
    for (int r = 0; r < KPL; r += 4) {
        int4 x;
        x.x = run;
        x.y = x.x + cnt[r];
        x.z = x.y + cnt[r + 1];
        x.w = x.z + cnt[r + 2];
        run = x.w + cnt[r + 3];
        *(int4 *)(buf + lane * KPL + r) = x;
    }
    wsync();
#pragma unroll
    for (int r = 0; r < KPL; ++r) at[r] += buf[b[r]];
    wsync();  // every base is read before any key lands
#pragma unroll
    for (int r = 0; r < KPL; ++r)
        if (key[r] != KMAX) buf[at[r]] = (int)key[r];
    wsync();
#pragma unroll
    for (int r = 0; r < KPL; r += 4) {
        const int4 x = *(const int4 *)(buf + lane * KPL + r);
        key[r] = lane * KPL + r < total ? (unsigned)x.x : KMAX;
        key[r + 1] = lane * KPL + r + 1 < total ? (unsigned)x.y : KMAX;
        key[r + 2] = lane * KPL + r + 2 < total ? (unsigned)x.z : KMAX;
        key[r + 3] = lane * KPL + r + 3 < total ? (unsigned)x.w : KMAX;
    }
    wsync();
    // (b neighbours need b alternating rounds of exchanges, whichever pairs start)
    for (int p = fullest > 1 ? 0 : fullest; p < fullest; p += 2) {
#pragma unroll
        for (int r = 0; r < KPL; r += 2) minmax(key[r], key[r + 1]);
        // (the moves below read what the asm blocks above wrote)
        asm volatile("s_nop 1" : "+v"(key[0]), "+v"(key[KPL - 1]));
        const unsigned next = (unsigned)wave_shl1((int)key[0], -1);
        const unsigned prev = (unsigned)wave_shr1((int)key[KPL - 1], 0);
#pragma unroll
        for (int r = 1; r + 1 < KPL; r += 2) minmax(key[r], key[r + 1]);
        key[0] = max(key[0], prev);
        key[KPL - 1] = min(key[KPL - 1], next);
    }
    return true;
}

// Smallest and largest row of the keys (positions below n) of a buffer.
template <int KPL>
__device__ __forceinline__ void row_span(const unsigned (&key)[KPL], unsigned &lo, unsigned &span) {
    unsigned mn = ~0u, mx = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        mn = min(mn, key[r]);
        mx = max(mx, key[r] == ~0u ? 0u : key[r]);
    }
    // rows have 21 bits: signed comparisons order them
    const int l = -__builtin_amdgcn_readlane(wave_incl_max(-(int)(mn >> kKeyBits)), 63);
    const int h = __builtin_amdgcn_readlane(wave_incl_max((int)(mx >> kKeyBits)), 63);
    lo = (unsigned)l;
    span = (unsigned)(h - l + 1);
}

// ---------------------------------------------------------------- one buffer
// LDS of one wavefront. Groups: head offsets, then staged output rows (key),
// and head values, then the products by slot, then staged output values (val).
template <typename V, int N, bool FILL>
struct GroupLds {
    alignas(16) int key[N];
    V val[FILL ? N : 1];
    int colv[64];          // per column of the item: its place in C (-1: do not write)
    int seg_out[64];       // per column: output entries (run count)
};
// A buffer that is one segment holds in turn, in the same 8 bytes a position
// (4 counting): heads or compacted rows with their entries' or products'
// indices; the sort's buckets; the products by slot; the staged sums; the
// staged rows. Between those the products wait in registers: 8 KB for 1024
// positions let 4 waves per SIMD stand side by side (12 KB: 3).
template <int N, bool FILL>
struct OneLds {
    alignas(16) int mem[FILL ? 2 * N : N];
    int stk[2 * 48];       // window stack (heavy columns)
};

// Runs of equal rows inside every aligned segment of S positions of the sorted
// keys (position KPL lane + r in register r).
template <int KPL>
struct Runs {
    unsigned head;   // bit r: position r starts a run
    unsigned live;   // bit r: position r holds a product
    int run;         // run index (inside the segment) of the lane's first run start
    int total;       // runs of the segment
    bool first;      // the lane starts a segment
    bool dups;       // some run of the buffer has more than one product (uniform)
};

template <typename K, int KPL, int S>
__device__ __forceinline__ Runs<KPL> seg_runs(const K (&key)[KPL], int lane) {
    constexpr K KMAX = KeyTraits<K>::kmax;
    constexpr int LPS = S / KPL;  // lanes per segment
    static_assert(LPS >= 2, "a segment spans lanes");
    Runs<KPL> o;
    o.first = (lane & (LPS - 1)) == 0;
    // the last key of the lane below (the position before this lane's first)
    K prev;
    if constexpr (sizeof(K) == 4) {
        prev = (K)(unsigned)wave_shr1((int)key[KPL - 1], 0);
    } else {
        const int lo = wave_shr1((int)(unsigned)key[KPL - 1], 0);
        const int hi = wave_shr1((int)(unsigned)(key[KPL - 1] >> 32), 0);
        prev = ((K)(unsigned)hi << 32) | (unsigned)lo;
    }
    o.head = 0;
    o.live = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const K p = r == 0 ? prev : key[r - 1];
        const bool lv = key[r] != KMAX;
        const bool hd = lv && ((r == 0 && o.first) || (key[r] >> kKeyBits) != (p >> kKeyBits));
        o.live |= lv ? 1u << r : 0u;
        o.head |= hd ? 1u << r : 0u;
    }
    o.dups = ballot(o.live != o.head) != 0;
    const int cnt = __builtin_popcount(o.head);
    const int inc = wave_incl_scan(cnt);
    if constexpr (LPS == 64) {
        o.run = inc - cnt;
        o.total = __builtin_amdgcn_readlane(inc, 63);
    } else {
        const int first_lane = lane & ~(LPS - 1);
        const int base = __builtin_amdgcn_ds_bpermute(first_lane << 2, inc - cnt);
        o.run = inc - cnt - base;
        o.total = __builtin_amdgcn_ds_bpermute((first_lane + LPS - 1) << 2, inc) - base;
    }
    return o;
}

// Largest occurrence index of the sorted buffer: a product's distance to the
// head of its run (its position among the products Algorithm 1 adds into the
// same entry); raised into the header's later_maxk for the plan's statistics.
template <int KPL>
__device__ __forceinline__ void note_depth(const KArgs &a, const Runs<KPL> &o, int lane) {
    if (!o.dups) return;
    const int s0 = lane * KPL;
    // the last head of the lanes below (head positions increase with the lane)
    const int last = o.head ? s0 + 31 - __builtin_clz(o.head) : -1;
    int h = wave_shr1(wave_incl_max(last), -1);
    int k = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        if ((o.head >> r) & 1u) h = s0 + r;
        if ((o.live >> r) & 1u) k = max(k, s0 + r - h);
    }
    k = __builtin_amdgcn_readlane(wave_incl_max(k), 63);
    if (lane == 0 && k > __atomic_load_n(&a.hdr->later_maxk, __ATOMIC_RELAXED))
        atomicMax(&a.hdr->later_maxk, k);
}

// The sorted products' values (v[r] of position r) become the running sums of
// their runs in order, every run starting from zero: the last position of a
// run holds its sum. A run that crosses lanes hands its partial sum from lane
// to lane, which keeps the order of the additions.
template <typename V, int KPL>
__device__ __forceinline__ void run_sums(V (&v)[KPL], const Runs<KPL> &o) {
    if (!o.dups) {
#pragma unroll
        for (int r = 0; r < KPL; ++r) v[r] = V(0) + v[r];
        return;
    }
    const bool cont = (o.live & 1u) && !(o.head & 1u);  // starts inside a run of the lane below
    V carry = V(0);
    if (ballot(cont)) {
        // the sum of the lane's last run as far as this lane knows it
        V t = V(0);
#pragma unroll
        for (int r = 0; r < KPL; ++r)
            if ((o.live >> r) & 1u) t = ((o.head >> r) & 1u) ? V(0) + v[r] : t + v[r];
        // lanes wholly inside a run wait for the lane below, lane after lane
        int known = (o.head != 0 || !cont) ? 1 : 0;
        while (ballot(!known)) {
            const V c = wave_shr1_v(t);
            const int k = wave_shr1(known, 1);
            if (!known && k) {
                t = c;
#pragma unroll
                for (int r = 0; r < KPL; ++r)
                    if ((o.live >> r) & 1u) t = t + v[r];
                known = 1;
            }
        }
        carry = wave_shr1_v(t);
    }
    V t = carry;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        t = ((o.head >> r) & 1u) ? V(0) + v[r] : t + v[r];
        v[r] = t;
    }
}

// Bit r: position r is the last of its run.
template <int KPL, int S>
__device__ __forceinline__ unsigned run_tails(const Runs<KPL> &o, int lane) {
    constexpr int LPS = S / KPL;
    // the next lane's first position continues this lane's last run
    const bool next = (o.live & 1u) && !(o.head & 1u);
    const int go = wave_shl1(next ? 1 : 0, 0);
    const bool last_lane = (lane & (LPS - 1)) == LPS - 1;
    const unsigned cont = (o.live & ~o.head) >> 1;  // bit r: position r + 1 continues the run of r
    const unsigned high = (go && !last_lane) ? 1u << (KPL - 1) : 0u;
    return o.live & ~(cont | high);
}

// ---------------------------------------------------------------- one work item
// A work item: up to G = N / S columns of one problem (bin-list entry
// (global column, first stored B entry, B entries, products) in lane c), each
// in its segment. Lanes LPS seg .. LPS (seg + 1) - 1 hold segment seg, LPS =
// S / KPL; product i of a column is gathered in row r = i / LPS of its
// segment, lane i mod LPS, LDS slot 64 r + lane.
//
// What bounds it: the chain bin entry -> B entries -> A gathers -> stores, and
// between them the instructions of the scans, the sort and the sums. So the
// cross-lane steps are DPP moves rather than LDS permutes, a product finds its
// B entry from a ballot of the head flags (no fill over the lanes), the sort
// starts from the gathered layout (any start order sorts the same), and the
// runs are summed in registers.
template <typename K, typename V, int KPL, int S, bool FILL>
__device__ __forceinline__ void wave_item(const KArgs &a, const Prob &d,
                                          GroupLds<V, 64 * KPL, FILL> &L, int4 ent, int ncol,
                                          int lane_in, int &bad) {
    constexpr int N = 64 * KPL, G = N / S, LPS = S / KPL;
    constexpr K KMAX = KeyTraits<K>::kmax;
    int lane = lane_in;  // (opaque: see one_item)
    asm volatile("" : "+v"(lane));
    const int j = ent.x - d.col0;
    // the filling pass's column bounds in C (known before the kernel) load
    // with the entries; they are used after the sort
    int2a ccp = {0, 0};
    if (FILL && lane < ncol) ccp = load_pair(d.ccp, j);
    const int2 *__restrict__ Ep = a.E + d.ebase;
    const gmem<const V> *__restrict__ bvp = to_gmem((const V *)d.bv);
    // first entry and first product of every column in the item's list
    const int einc = wave_incl_scan(ent.z), oinc = wave_incl_scan(ent.w);
    const int es = einc - ent.z, ob = oinc - ent.w, bsd = ent.y - es;
    const int tot_entries = __builtin_amdgcn_readlane(einc, 63);
    const int tot_products = __builtin_amdgcn_readlane(oinc, 63);
#pragma unroll
    for (int r = 0; r < KPL; ++r) L.key[r * 64 + lane] = kHeadNone;
    wsync();
    // heads: at the slot of a stored B entry's first product (and of its first
    // product of every further row), A's index less the product's position
    bool ok = true;
    int run = 0;
    for (int x0 = 0; x0 < tot_entries; x0 += 64) {
        const int x = x0 + lane;
        int cc = 0;
#pragma unroll
        for (int c = 1; c < G; ++c)
            cc += x >= __builtin_amdgcn_readlane(es, c) ? 1 : 0;
        const int cbs = G == 1 ? __builtin_amdgcn_readlane(bsd, 0) : shfl_idx(bsd, cc);
        const int cob = G == 1 ? 0 : shfl_idx(ob, cc);
        const int ces = G == 1 ? 0 : shfl_idx(es, cc);
        int2 e = make_int2(0, 0);
        V bval = V(0);
        if (x < tot_entries) {
            e = Ep[cbs + x];
            if (FILL) bval = bvp[cbs + x];
        }
        const int inc = wave_incl_scan(e.y);
        // position of the entry's first product inside its column: the
        // products listed before it less those of the earlier columns
        const int o = run + inc - e.y - cob;
        if (x < tot_entries && x == ces && o != 0) ok = false;
        if (e.y > 0) {
            if (o < 0 || e.y > S - o) {
                ok = false;
            } else {
                const int end = o + e.y;
                int row = o / LPS;
                int slot = row * 64 + cc * LPS + o % LPS;
                L.key[slot] = e.x - o;
                if (FILL) L.val[slot] = bval;
                for (++row; row * LPS < end; ++row) {
                    slot = row * 64 + cc * LPS;
                    L.key[slot] = e.x - o;
                    if (FILL) L.val[slot] = bval;
                }
            }
        }
        run += __builtin_amdgcn_readlane(inc, 63);
    }
    if (ballot(!ok) != 0 || run != tot_products) {
        bad = 1;
        wsync();
        return;
    }
    wsync();
    // every product's head is the last one at or before its lane in its row
    const int seg = lane / LPS;
    const int opn = shfl_idx(ent.w, seg);
    const gmem<const int32_t> *__restrict__ ari = to_gmem(d.ari);
    const gmem<const V> *__restrict__ av = to_gmem((const V *)d.av);
    const unsigned long long le = mask_lt() | (1ull << lane);
    int q[KPL], from[KPL];
    unsigned live = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const unsigned long long m = ballot(L.key[r * 64 + lane] != kHeadNone) & le;
        const int i = r * LPS + (lane & (LPS - 1));
        const bool lv = i < opn && m != 0;
        from[r] = r * 64 + 63 - __builtin_clzll(m | 1ull);
        const int h = L.key[from[r]];
        q[r] = lv ? h + i : 0;  // (a product exists, so A's first entry does)
        live |= lv ? 1u << r : 0u;
    }
    int row[KPL];
    V v[KPL];
    // every gather of the lane issued before any is used
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        row[r] = ari[q[r]];
        if (FILL) v[r] = av[q[r]];
    }
    if (FILL) {
        // products by slot (a row's heads are read before its products land)
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
            const V b = L.val[from[r]];
            wsync();
            L.val[r * 64 + lane] = v[r] * b;
        }
    }
    K key[KPL];
    bool badrow = false;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const bool lv = (live >> r) & 1u;
        // a row outside A's row range is malformed input (reported; the
        // product takes no part)
        const bool in = row[r] >= 0 && row[r] < d.m;
        badrow |= lv && !in;
        key[r] = lv && in ? (((K)(unsigned)row[r] << kKeyBits) | (K)(unsigned)(r * 64 + lane)) : KMAX;
    }
    if (ballot(badrow) && lane == 0) atomicOr(&a.hdr->err, ERR_CSC);
    seg_sort<K, KPL, S>(key, lane);
    const Runs<KPL> o = seg_runs<K, KPL, S>(key, lane);
    if (!FILL || a.spec_fill) note_depth<KPL>(a, o, lane);
    if constexpr (!FILL) {
        // run count of every column, from its segment's lanes
        const int cnt = shfl_idx(o.total, (lane * LPS) & 63);
        if (lane < ncol) a.gnnz[ent.x] = cnt;
        wsync();
    } else {
        const int cnt = shfl_idx(o.total, (lane * LPS) & 63);
        if (lane < ncol) {
            // a count that differs from the symbolic phase's means other
            // inputs (nothing is written then)
            const int clen = ccp.y - ccp.x;
            L.colv[lane] = cnt == clen ? ccp.x : -1;
            L.seg_out[lane] = cnt;
            if (a.spec_fill) a.gnnz[ent.x] = cnt;
        }
        wsync();
#pragma unroll
        for (int r = 0; r < KPL; ++r)
            v[r] = L.val[(int)(key[r] & (K)(N - 1))];  // (of padding: any value)
        run_sums<V, KPL>(v, o);
        wsync();
        // a run's row and sum staged at segment start + run index
        const unsigned tails = run_tails<KPL, S>(o, lane);
        int at = seg * S + o.run - 1;
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
            at += (o.head >> r) & 1u;
            if ((tails >> r) & 1u) {
                L.key[at] = (int)(key[r] >> kKeyBits);
                L.val[at] = v[r];
            }
        }
        wsync();
        // consecutive lanes write consecutive entries of a column
        gmem<int32_t> *cri = to_gmem(d.cri);
        gmem<V> *cv = to_gmem((V *)d.cv);
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
            const int s = r * 64 + lane, c = s / S, i = s - c * S;
            if (c >= ncol) continue;
            const int c0 = L.colv[c];
            if (c0 < 0) {
                bad = 1;
                continue;
            }
            if (i < L.seg_out[c]) {
                cri[c0 + i] = L.key[s];
                cv[c0 + i] = L.val[s];
            }
        }
        wsync();
    }
}

// ---------------------------------------------------------------- one segment
// Sorts a buffer that is one segment (key: slot 64 r + lane in register r, all
// ones where there is none; rows in [lo, lo + span) when span > 0, else found
// here) and finds its runs.
template <typename K, int KPL, bool FILL>
__device__ __forceinline__ Runs<KPL> one_sort(const KArgs &a, K (&key)[KPL], unsigned lo,
                                              unsigned span, int *mem, int lane) {
    constexpr int N = 64 * KPL;
    bool sorted = false;
    if constexpr (sizeof(K) == 4) {
        if (span == 0) row_span<KPL>(key, lo, span);
        sorted = bucket_sort<KPL>(key, lo, span, mem, lane);
    }
    if (!sorted) seg_sort<K, KPL, N>(key, lane);
    const Runs<KPL> o = seg_runs<K, KPL, N>(key, lane);
    if (!FILL || a.spec_fill) note_depth<KPL>(a, o, lane);
    return o;
}

// The sorted buffer's runs to C at `at`: v holds the products by slot. The
// sums and then the rows pass through the LDS, so that consecutive lanes write
// consecutive entries.
template <typename K, typename V, int KPL>
__device__ __forceinline__ void one_emit(const Prob &d, const K (&key)[KPL], V (&v)[KPL],
                                         const Runs<KPL> &o, long long at, int *mem, int lane) {
    constexpr int N = 64 * KPL;
    V *val = (V *)mem;
#pragma unroll
    for (int r = 0; r < KPL; ++r) val[r * 64 + lane] = v[r];
    wsync();
#pragma unroll
    for (int r = 0; r < KPL; ++r) v[r] = val[(int)(key[r] & (K)(N - 1))];  // (of padding: any value)
    run_sums<V, KPL>(v, o);
    wsync();
    const unsigned tails = run_tails<KPL, N>(o, lane);
    int to = o.run - 1;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        to += (o.head >> r) & 1u;
        if ((tails >> r) & 1u) val[to] = v[r];
    }
    wsync();
    gmem<V> *cv = to_gmem((V *)d.cv) + at;
    for (int i = lane; i < o.total; i += 64) cv[i] = val[i];
    wsync();
    to = o.run - 1;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        to += (o.head >> r) & 1u;
        if ((tails >> r) & 1u) mem[to] = (int)(key[r] >> kKeyBits);
    }
    wsync();
    gmem<int32_t> *cri = to_gmem(d.cri) + at;
    for (int i = lane; i < o.total; i += 64) cri[i] = mem[i];
    wsync();
}

// One column per wavefront (`ent`: its bin-list entry, the same in every lane),
// its products gathered as in wave_item with one row of 64 slots per register.
template <typename K, typename V, int KPL, bool FILL>
__device__ __forceinline__ void one_item(const KArgs &a, const Prob &d,
                                         OneLds<64 * KPL, FILL> &L, int4 ent, int lane_in,
                                         int &bad) {
    constexpr int N = 64 * KPL;
    constexpr K KMAX = KeyTraits<K>::kmax;
    // opaque lane number: the slots' addresses are not kept in registers
    // outside the item
    int lane = lane_in;
    asm volatile("" : "+v"(lane));
    const int g = ent.x, bs = ent.y, nb = ent.z, op = ent.w;
    int2a ccp = {0, 0};
    if (FILL) ccp = load_pair(d.ccp, g - d.col0);
    const int2 *__restrict__ Ep = a.E + d.ebase + bs;
    int2 *head2 = (int2 *)L.mem;  // (A's index less the position, B entry); counting: the first only
    int *head1 = L.mem;
    int2 e = lane < nb ? Ep[lane] : make_int2(0, 0);
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        if (FILL) head2[r * 64 + lane] = make_int2(kHeadNone, 0);
        else head1[r * 64 + lane] = kHeadNone;
    }
    wsync();
    bool ok = true;
    int run = 0;
    for (int x0 = 0; x0 < nb; x0 += 64) {
        // the next entries load while these are placed
        const int2 next = x0 + 64 + lane < nb ? Ep[x0 + 64 + lane] : make_int2(0, 0);
        const int inc = wave_incl_scan(e.y), o = run + inc - e.y;
        if (e.y > 0) {
            if (o < 0 || e.y > N - o) {
                ok = false;
            } else {
                const int2 h = make_int2(e.x - o, bs + x0 + lane);
                int slot = o;
                do {  // its first product, and its first of every further row
                    if (FILL) head2[slot] = h;
                    else head1[slot] = h.x;
                    slot = (slot | 63) + 1;
                } while (slot < o + e.y);
            }
        }
        run += __builtin_amdgcn_readlane(inc, 63);
        e = next;
    }
    if (ballot(!ok) != 0 || run != op) {
        bad = 1;
        wsync();
        return;
    }
    wsync();
    const gmem<const int32_t> *__restrict__ ari = to_gmem(d.ari);
    const gmem<const V> *__restrict__ av = to_gmem((const V *)d.av);
    const gmem<const V> *__restrict__ bvp = to_gmem((const V *)d.bv);
    const unsigned long long le = mask_lt() | (1ull << lane);
    int row[KPL];
    V v[KPL];
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const int h = FILL ? head2[r * 64 + lane].x : head1[r * 64 + lane];
        const unsigned long long m = ballot(h != kHeadNone) & le;
        const int from = r * 64 + 63 - __builtin_clzll(m | 1ull);
        const bool lv = r * 64 + lane < op;  // (row r then starts with a head)
        int2 x = FILL ? head2[from] : make_int2(head1[from], 0);
        // a padding position reads A's and B's first entries
        const int q = lv ? x.x + r * 64 + lane : 0;
        row[r] = ari[q];
        if (FILL) v[r] = av[q] * bvp[lv ? x.y : 0];
    }
    // (the products are formed here: left to the compiler, both factors wait in
    // registers until the sort is over)
    if (FILL)
#pragma unroll
        for (int r = 0; r < KPL; ++r) asm volatile("" : "+v"(v[r]));
    K key[KPL];
    bool badrow = false;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
        const bool lv = r * 64 + lane < op;
        // a row outside A's row range is malformed input (reported; the
        // product takes no part)
        const bool in = row[r] >= 0 && row[r] < d.m;
        badrow |= lv && !in;
        key[r] = lv && in ? (((K)(unsigned)row[r] << kKeyBits) | (K)(unsigned)(r * 64 + lane)) : KMAX;
    }
    if (ballot(badrow)) {
        if (lane == 0) atomicOr(&a.hdr->err, ERR_CSC);
        return;
    }
    wsync();
    const Runs<KPL> o = one_sort<K, KPL, FILL>(a, key, 0u, 0u, L.mem, lane);
    if ((!FILL || a.spec_fill) && lane == 0) a.gnnz[g] = o.total;
    if constexpr (FILL) {
        // a count that differs from the symbolic phase's means other inputs
        // (nothing is written then)
        if (o.total != ccp.y - ccp.x) bad = 1;
        else one_emit<K, V, KPL>(d, key, v, o, ccp.x, L.mem, lane);
    }
    wsync();
}

template <typename K, typename V, int KPL, bool FILL, bool MULTI>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(KPL == 16 ? 4 : 1))) void k_acc_one(KArgs a, int bin) {
    __shared__ OneLds<64 * KPL, FILL> L;
    const BinRange br = bin_range<FILL>(a, bin, bin);
    if (br.stop) return;
    const int lane = threadIdx.x;
    int bad = 0;
    for (int i = blockIdx.x; i < br.count; i += gridDim.x) {
        const int4 e = a.binlist[br.first + i];
        const int4 ent = make_int4(
            __builtin_amdgcn_readfirstlane(e.x), __builtin_amdgcn_readfirstlane(e.y),
            __builtin_amdgcn_readfirstlane(e.z), __builtin_amdgcn_readfirstlane(e.w));
        if (ent.w > 64 * KPL || ent.z > 64 * KPL) {  // cannot happen for unchanged inputs
            bad = 1;
            break;
        }
        const Prob d = prob_of<MULTI>(a, ent.x);
        one_item<K, V, KPL, FILL>(a, d, L, ent, lane, bad);
    }
    if (ballot(bad != 0) && lane == 0)
        atomicOr(&a.hdr->err, a.spec_fill ? ERR_RETRY : ERR_GROUP);
}

// ---------------------------------------------------------------- wavefront groups
// Group gi of a bin of columns of at most S products: G = N / S of them.
template <typename K, typename V, int KPL, int S, bool FILL, bool MULTI>
__device__ __forceinline__ void group_item(const KArgs &a, GroupLds<V, 64 * KPL, FILL> &L,
                                           int bin_first, int bin_cols, int gi, int lane,
                                           int &bad) {
    constexpr int N = 64 * KPL, G = N / S;
    static_assert(S <= N && (N % S) == 0 && N <= (1 << kKeyBits), "segments tile the buffer");
    const int first = bin_first + gi * G, ncol = min(G, bin_cols - gi * G);
    int c0 = 0;
    do {
        // the columns from c0 on, lane c holding column c0 + c
        int4 ent = lane < ncol - c0 ? a.binlist[first + c0 + lane] : make_int4(0, 0, 0, 0);
        if (ballot(ent.w > S || ent.z > N)) {  // cannot happen for unchanged inputs
            bad = 1;
            break;
        }
        int nc = ncol - c0;
        const Prob d = prob_of<MULTI>(a, ent.x);
        if constexpr (MULTI) {
            // a group may cross problems (bins are filled problem by
            // problem): the columns of the first one's are an item
            const unsigned long long other =
                ballot(lane < nc && (ent.x < d.col0 || ent.x >= d.col0 + d.n));
            if (other) nc = __builtin_ctzll(other);
            if (lane >= nc) ent = make_int4(0, 0, 0, 0);
        }
        wave_item<K, V, KPL, S, FILL>(a, d, L, ent, nc, lane, bad);
        c0 += nc;
    } while (MULTI && c0 < ncol);
}

// ---------------------------------------------------------------- one column per lane
// Columns of at most L products and L stored B entries: every lane takes one
// column whole, in its own registers -- the paper's mapping of one column to
// one vector element (Section 3.1), with a sort-merge in place of its
// accumulator. No lane talks to another; each lane's values sit in its own
// LDS slots. Keys (row << LB | position) are 32-bit while rows stay below
// 2^(32 - LB) - 1.
template <typename K, typename V, int L, bool FILL, bool MULTI>
__device__ __forceinline__ void lane_item(const KArgs &a, V *sval, int start, int cnt, int gi,
                                          int lane, int &bad) {
    constexpr int LB = L <= 4 ? 2 : (L <= 8 ? 3 : 4);
    static_assert((1 << LB) == L, "L is 4, 8 or 16");
    constexpr K KMAX = KeyTraits<K>::kmax;
    int badrow = 0, kmax = 0;
    const int ci = gi * 64 + lane;
    do {  // (once; a lane that is done leaves it)
        if (ci >= cnt) break;
        const int4 ent = a.binlist[start + ci];
        const int g = ent.x, bs = ent.y, nb = ent.z, op = ent.w;
        if (op > L || nb > L) {  // cannot happen for unchanged inputs
            bad = 1;
            break;
        }
        // (the lanes' columns may belong to several problems)
        const Prob d = MULTI ? a.table[find_prob(a, g)] : a.single;
        // the C column's bounds (numeric phase) load together with the entries
        int c0 = 0, clen = 0;
        if (FILL) {
            const int j = g - d.col0;
            const int2a cp = load_pair(d.ccp, j);
            c0 = cp.x;
            clen = cp.y - c0;
        }
        const int2 *__restrict__ Ep = a.E + d.ebase;
        const gmem<const V> *__restrict__ bvp = to_gmem((const V *)d.bv);
        // the column's stored B entries: A column start, length, B value
        int as_[L], zs[L], oo[L];
        V bv_[L];
#pragma unroll
        for (int t = 0; t < L; ++t) {
            as_[t] = 0;
            zs[t] = 0;
            bv_[t] = V(0);
            if (t < nb) {
                const int2 e = Ep[bs + t];
                as_[t] = e.x;
                zs[t] = e.y;
                if (FILL) bv_[t] = bvp[bs + t];
            }
        }
        int run = 0;
#pragma unroll
        for (int t = 0; t < L; ++t) {
            oo[t] = run;
            run += zs[t];
        }
        if (run != op) {  // entries do not add up to the product count
            bad = 1;
            break;
        }
        // product p belongs to the entry after the ones ending at or before p
        int q[L];
        V bb[L];
#pragma unroll
        for (int p = 0; p < L; ++p) {
            int tp = 0;
#pragma unroll
            for (int t = 0; t < L; ++t) tp += (oo[t] + zs[t] <= p) ? 1 : 0;
            int qa = 0, qo = 0;
            V qv = V(0);
#pragma unroll
            for (int t = 0; t < L; ++t) {
                if (t == tp) {
                    qa = as_[t];
                    qo = oo[t];
                    if (FILL) qv = bv_[t];
                }
            }
            q[p] = qa + p - qo;
            bb[p] = qv;
        }
        const gmem<const int32_t> *__restrict__ ari = to_gmem(d.ari);
        const gmem<const V> *__restrict__ av = to_gmem((const V *)d.av);
        int row[L];
        V x[L];
#pragma unroll
        for (int p = 0; p < L; ++p) {
            row[p] = p < op ? ari[q[p]] : 0;
            if (FILL) x[p] = p < op ? av[q[p]] : V(0);
        }
        K key[L];
#pragma unroll
        for (int p = 0; p < L; ++p) {
            key[p] = KMAX;
            if (p < op) {
                if (row[p] < 0 || row[p] >= d.m) {
                    badrow = 1;
                } else {
                    key[p] = ((K)(unsigned)row[p] << LB) | (K)(unsigned)p;
                    if (FILL) sval[lane * L + p] = x[p] * bb[p];
                }
            }
        }
        // bitonic network over the lane's L keys
#pragma unroll
        for (int k = 2; k <= L; k <<= 1) {
#pragma unroll
            for (int jj = k >> 1; jj > 0; jj >>= 1) {
#pragma unroll
                for (int r = 0; r < L; ++r) {
                    if (r & jj) continue;
                    const int rp = r | jj;
                    const bool asc = (r & k) == 0;
                    const K u = key[r], w = key[rp];
                    const bool sw = asc ? (u > w) : (u < w);
                    key[r] = sw ? w : u;
                    key[rp] = sw ? u : w;
                }
            }
        }
        // runs of equal rows, each summed in position order (Algorithm 1's)
        int nd = 0, depth = 0, dcur = 0;
#pragma unroll
        for (int p = 0; p < L; ++p) {
            if (key[p] == KMAX) continue;
            const bool head = p == 0 || (key[p] >> LB) != (key[p - 1] >> LB);
            dcur = head ? 0 : dcur + 1;
            depth = max(depth, dcur);
            nd += head ? 1 : 0;
        }
        kmax = max(kmax, depth);
        if (!FILL || a.spec_fill) a.gnnz[g] = nd;
        if (FILL) {
            if (nd != clen) {
                bad = 1;
                break;
            }
            gmem<int32_t> *cri = to_gmem(d.cri);
            gmem<V> *cv = to_gmem((V *)d.cv);
            int u = 0;
            V acc = V(0);
#pragma unroll
            for (int p = 0; p < L; ++p) {
                if (key[p] == KMAX) continue;
                const V v = sval[lane * L + (int)(key[p] & (K)(L - 1))];
                const bool head = p == 0 || (key[p] >> LB) != (key[p - 1] >> LB);
                acc = head ? V(0) + v : acc + v;
                const bool last = p == L - 1 || key[p + 1 < L ? p + 1 : p] == KMAX ||
                                  (key[p + 1 < L ? p + 1 : p] >> LB) != (key[p] >> LB);
                if (last) {
                    cri[c0 + u] = (int32_t)(key[p] >> LB);
                    cv[c0 + u] = acc;
                    ++u;
                }
            }
        }
    } while (false);
    if (ballot(badrow) && lane == 0) atomicOr(&a.hdr->err, ERR_CSC);
    if ((!FILL || a.spec_fill) && ballot(kmax > 0)) {
        kmax = __builtin_amdgcn_readlane(wave_incl_max(kmax), 63);
        if (lane == 0 && kmax > __atomic_load_n(&a.hdr->later_maxk, __ATOMIC_RELAXED))
            atomicMax(&a.hdr->later_maxk, kmax);
    }
    wsync();
}

// ---------------------------------------------------------------- light columns
// Columns of at most 256 products: the bins of `mask` (bit i: ESC sub-bin i),
// largest first, in one launch. Sub-bins 0 and 1 (at most 4, 8 products) take
// 64 columns an item, one per lane; sub-bin i >= 2 (at most 4 << i products)
// 64 >> i columns in segments of 4 << i (measured: segments of 16 beat a lane
// per column by 16%, segments of 8 lose by 14%). One wavefront per workgroup:
// waves share nothing. The item's bin is found from the header's counts. With
// a launch per bin the chip drained between them and the host paid 4 to 5 us
// for each: whole product of a 1M-column power law 542 us, now 530, of a
// 300k-column one (f32) 223, now 214, numeric phase of a 400k one 205, now 192.
constexpr int kLightBins = kEscBins;
__host__ __device__ constexpr int light_columns(int i) { return i < kLaneSubBins ? 64 : 64 >> i; }

template <typename K, typename V, bool FILL, bool MULTI>
__global__ __launch_bounds__(64) void k_acc_light(KArgs a, unsigned mask) {
    __shared__ union {
        GroupLds<V, 256, FILL> g;
        V lanes[FILL ? 64 * 8 : 1];
    } L;
    cmem<Hdr> *h = (cmem<Hdr> *)a.hdr;
    if ((h->err | (FILL ? h->cap_over : 0)) != 0) return;
    const int lane = threadIdx.x;
    int bad = 0;
    for (int i = blockIdx.x;; i += gridDim.x) {
        int gi = i, bin = -1, first = 0, cols = 0;
#pragma unroll
        for (int b = kLightBins - 1; b >= 0; --b) {
            const int n = (mask >> b) & 1u ? h->bin_count[BIN_ESC0 + b] : 0;
            const int items = (n + light_columns(b) - 1) / light_columns(b);
            if (bin < 0) {
                if (gi < items) {
                    bin = b;
                    cols = n;
                    first = h->bin_start[BIN_ESC0 + b];
                } else {
                    gi -= items;
                }
            }
        }
        if (bin < 0) break;
        switch (bin) {
            case 0: lane_item<K, V, 4, FILL, MULTI>(a, L.lanes, first, cols, gi, lane, bad); break;
            case 1: lane_item<K, V, 8, FILL, MULTI>(a, L.lanes, first, cols, gi, lane, bad); break;
            case 2: group_item<K, V, 4, 16, FILL, MULTI>(a, L.g, first, cols, gi, lane, bad); break;
            case 3: group_item<K, V, 4, 32, FILL, MULTI>(a, L.g, first, cols, gi, lane, bad); break;
            case 4: group_item<K, V, 4, 64, FILL, MULTI>(a, L.g, first, cols, gi, lane, bad); break;
            case 5: group_item<K, V, 4, 128, FILL, MULTI>(a, L.g, first, cols, gi, lane, bad); break;
            default: group_item<K, V, 4, 256, FILL, MULTI>(a, L.g, first, cols, gi, lane, bad); break;
        }
    }
    // an output count other than the planned one: other inputs, or (a
    // numeric phase run at a previous structure's positions) a redo
    if (ballot(bad != 0) && lane == 0)
        atomicOr(&a.hdr->err, a.spec_fill ? ERR_RETRY : ERR_GROUP);
}

// ---------------------------------------------------------------- heavy columns
// The heavy column of every window (one thread per heavy column), written
// once the window scratch is in place; a launch planned with too small a
// scratch has been flagged for a redo and writes nothing.
template <bool MULTI>
__global__ __launch_bounds__(kBlock) void k_win_map(KArgs a) {
    const BinRange br = bin_range<false>(a, kHeavyBin, BIN_WSORT);
    if (br.stop) return;
    const int first = br.first, n = br.count;
    for (int li = blockIdx.x * kBlock + threadIdx.x; li < n; li += gridDim.x * kBlock) {
        const int w0 = a.wbase[li];
        const int w1 = w0 + (a.binlist[first + li].w - 1) / kWinTarget + 1;
        for (int w = w0; w < w1 && w < a.win_cap; ++w) a.winmap[w] = li;
    }
}

// Expansion of the heavy columns into the scratch: the row (and in FILL the
// value A(i,k) B(k,j)) of every product, in Algorithm 1's order. One workgroup
// per column of at most 4096 products, up to `split` per longer one (each a
// range of its stored B entries, kExpandEntries or more; its first product's
// position is the sum of the lengths before it), 256 entries at a time. On its
// own it is bound by the longest workgroup's rounds of gathers (10k-column
// power law, 21 heavy columns: 44 us; whole product 143, now 116), on a full
// chip by the 128-byte lines its short A columns touch.
constexpr int kExpandEntries = 64;
template <typename V, bool FILL, bool MULTI>
__global__ __launch_bounds__(kBlock) void k_heavy_expand(KArgs a, int split) {
    __shared__ int s_acp[kBlock], s_eoff[kBlock], scan_tmp[kBlock / 64 + 1];
    __shared__ V s_bv[FILL ? kBlock : 1];
    const BinRange br = bin_range<FILL>(a, kHeavyBin, BIN_WSORT);
    if (br.stop) return;  // the same in every thread
    const int first = br.first, n = br.count;
    const int tid = threadIdx.x;
    const int nlong = ((cmem<Hdr> *)a.hdr)->bin_count[BIN_WSORT];
    const int items = nlong * split + n - nlong;
    int bad = 0, rowbad = 0;
    // largest columns first (the heavy list runs from small to large bins):
    // the longest workgroups start before the short ones
    for (int it = blockIdx.x; it < items; it += gridDim.x) {
        const bool parted = it < nlong * split;
        const int lj = parted ? it / split : it - nlong * (split - 1);
        const int li = n - 1 - lj;
        const int4 ent = a.binlist[first + li];
        const int bs = ent.y, nb = ent.z;
        // its entries [b0, b1)
        int b0 = 0, b1 = nb;
        if (parted) {
            const int parts = min(split, (nb + kExpandEntries - 1) / kExpandEntries);
            const int per = (nb + parts - 1) / parts;
            b0 = min(nb, it % split * per);
            b1 = min(nb, b0 + per);
            if (b0 == b1) continue;
        }
        const Prob d = prob_of<MULTI>(a, ent.x);
        const long long base0 = a.hoff[li], end = base0 + ent.w;
        const int2 *__restrict__ Ep = a.E + d.ebase;
        const gmem<const int32_t> *__restrict__ ari = to_gmem(d.ari);
        const gmem<const V> *__restrict__ av = to_gmem((const V *)d.av);
        const gmem<const V> *__restrict__ bvp = to_gmem((const V *)d.bv);
        long long base = base0;
        if (b0 > 0) {
            int before = 0, sum;
            for (int t = tid; t < b0; t += kBlock) before += Ep[bs + t].y;
            block_excl_scan(before, scan_tmp, sum);
            base += sum;
            if (base < base0) {  // (the lengths do not add up to the product count)
                bad = 1;
                continue;
            }
        }
        for (int bw = b0; bw < b1; bw += kBlock) {
            const int t = bw + tid;
            int z = 0, as = 0;
            V bval = V(0);
            if (t < b1) {
                const int2 e = Ep[bs + t];
                as = e.x;
                z = e.y;
                if (FILL) bval = bvp[bs + t];
            }
            int Ew;
            const int ex = block_excl_scan(z, scan_tmp, Ew);
            s_acp[tid] = as;
            s_eoff[tid] = ex;
            if (FILL) s_bv[tid] = bval;
            __syncthreads();
            const int nbw = min(kBlock, b1 - bw);
            if (Ew < 0 || base + Ew > end) {  // more products than planned: inputs changed
                bad = 1;
                __syncthreads();
                break;
            }
            for (int e0 = 0; e0 < Ew; e0 += 4 * kBlock) {
                int rr[4];
                V xv[4];
                int tt[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = e0 + u * kBlock + tid;
                    const int ee = min(e, Ew - 1);
                    tt[u] = last_le(s_eoff, nbw, ee);
                    const int q = s_acp[tt[u]] + ee - s_eoff[tt[u]];
                    rr[u] = ari[q];
                    if (FILL) xv[u] = av[q];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = e0 + u * kBlock + tid;
                    if (e >= Ew) continue;
                    if (rr[u] < 0 || rr[u] >= d.m) {  // malformed input
                        rowbad = 1;
                        rr[u] = 0;
                    }
                    a.hrow[base + e] = rr[u];
                    if (FILL) ((V *)a.hval)[base + e] = xv[u] * s_bv[tt[u]];
                }
            }
            base += Ew;
            __syncthreads();
        }
    }
    if (bad && tid == 0) atomicOr(&a.hdr->err, ERR_GROUP);
    if (rowbad) atomicOr(&a.hdr->err, ERR_CSC);
}

// One window of a heavy column per wavefront (grid-stride over all windows):
// rows [m w / W, m (w + 1) / W) of the column's products, compacted in product
// order into the buffer, sorted, compressed. A window holding more products
// than the buffer is halved in row span (a stack, left half first); a window
// of a single row with more products than the buffer is one output entry,
// summed in product order by one lane.
template <typename K, typename V, bool FILL, bool MULTI>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_acc_window(KArgs a) {
    constexpr int KPL = kWinKpl, N = 64 * KPL;
    constexpr K KMAX = KeyTraits<K>::kmax;
    __shared__ OneLds<N, FILL> L;
    int *const prows = L.mem, *const pidx = L.mem + (FILL ? N : 0);  // compacted rows, indices
    const BinRange br = bin_range<FILL>(a, kHeavyBin, BIN_WSORT);
    if (br.stop) return;
    const int first = br.first;
    const int nwin = ((cmem<Hdr> *)a.hdr)->heavy_win;
    int bad = 0;
    // windows of the largest columns (the longest scans) first; workgroups go
    // to the 8 XCDs in turn and each XCD has its own L2, so every run of kRun
    // consecutive windows (mostly one column's, which all scan that column)
    // goes to one XCD: inside each block of kXcd kRun workgroups, XCD x takes
    // windows kRun x .. kRun x + kRun - 1 of the block (the ragged last block
    // keeps its order)
    constexpr int kXcd = 8, kRun = 16, kBlk = kXcd * kRun;
    const int full = nwin / kBlk * kBlk;
    for (int b = blockIdx.x; b < nwin; b += gridDim.x) {
        int lane = threadIdx.x;  // (opaque: see one_item)
        asm volatile("" : "+v"(lane));
        const int rb = b % kBlk;
        const int wj = b >= full ? b : b - rb + (rb % kXcd) * kRun + rb / kXcd;
        const int wi = nwin - 1 - wj;
        const int li = a.winmap[wi];
        const int4 ent = a.binlist[first + li];
        const int g = ent.x, op = ent.w;
        const int wb = a.wbase[li], w = wi - wb, W = (op - 1) / kWinTarget + 1;
        const Prob d = prob_of<MULTI>(a, g);
        const int j = g - d.col0;
        const long long hb = a.hoff[li];
        const int *__restrict__ prow = a.hrow + hb;
        const V *__restrict__ pval = FILL ? (const V *)a.hval + hb : nullptr;
        // output position of the window: the entries of the earlier windows
        int out = 0;
        if (FILL) {
            for (int q = lane; q < w; q += 64) out += a.wcnt[wb + q];
            out = wave_sum(out);
            // A launch at a previous structure's positions may meet windows that
            // no launch has counted, where any number stands: below zero it is
            // refused here, beyond the column where an entry would be written.
            if (out < 0) {
                bad = 1;
                continue;
            }
        }
        int c0 = 0;
        if (FILL) c0 = d.ccp[j];
        const int m = d.m;
        int sp = 0;
        if (lane == 0) {
            L.stk[0] = (int)((long long)m * w / W);
            L.stk[1] = (int)((long long)m * (w + 1) / W);
        }
        sp = 1;
        wsync();
        int total = 0;
        while (sp > 0) {
            --sp;
            const int x = L.stk[2 * sp], y = L.stk[2 * sp + 1];
            wsync();
            // compact the window's products (product order) into the buffer,
            // the next 8 rows per lane in flight while 8 are tested (the scan
            // waits on its loads: the kernel alone on a 1M power law 97 us, with
            // them ahead 87; the whole product 525, now 518)
            constexpr int U = 8;
            int cnt = 0;
            int ahead[U];
#pragma unroll
            for (int u = 0; u < U; ++u) ahead[u] = u * 64 + lane < op ? prow[u * 64 + lane] : -1;
            for (int e0 = 0; e0 < op; e0 += 64 * U) {
                int r[U], pos[U];
                bool in[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + (U + u) * 64 + lane;
                    r[u] = ahead[u];
                    ahead[u] = e < op ? prow[e] : -1;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    in[u] = r[u] >= x && r[u] < y;
                    const unsigned long long bm = ballot(in[u]);
                    pos[u] = cnt + popc64(bm & mask_lt());
                    cnt += popc64(bm);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (in[u] && pos[u] < N) {
                        prows[pos[u]] = r[u];
                        if constexpr (FILL) pidx[pos[u]] = e0 + u * 64 + lane;
                    }
                }
            }
            wsync();
            if (cnt > N && y - x > 1) {
                if (sp + 2 > 48) {  // cannot happen: the span halves every time
                    bad = 1;
                    break;
                }
                const int mid = x + (y - x) / 2;
                if (lane == 0) {
                    L.stk[2 * sp] = mid;
                    L.stk[2 * sp + 1] = y;
                    L.stk[2 * sp + 2] = x;
                    L.stk[2 * sp + 3] = mid;
                }
                sp += 2;
                wsync();
                continue;
            }
            if (cnt > N) {
                // one row, more products than the buffer: one entry
                if ((!FILL || a.spec_fill) && lane == 0 &&
                    cnt - 1 > __atomic_load_n(&a.hdr->later_maxk, __ATOMIC_RELAXED))
                    atomicMax(&a.hdr->later_maxk, cnt - 1);
                if (FILL && lane == 0) {
                    V acc = V(0);
                    bool firstp = true;
                    for (int e = 0; e < op; ++e) {
                        if (prow[e] != x) continue;
                        acc = firstp ? V(0) + pval[e] : acc + pval[e];
                        firstp = false;
                    }
                    if (total >= d.ccp[j + 1] - c0 - out) bad = 1;
                    else {
                        d.cri[c0 + out + total] = x;
                        ((V *)d.cv)[c0 + out + total] = acc;
                    }
                }
                total += 1;
                wsync();
                continue;
            }
            // keys by slot, and the values of the window's products in one batch
            // of gathers (the scan above waited on its rows only)
            K key[KPL];
            V v[KPL];
#pragma unroll
            for (int r = 0; r < KPL; ++r) {
                const int s = r * 64 + lane;
                const bool lv = s < cnt;
                key[r] = lv ? (((K)(unsigned)prows[s] << kKeyBits) | (K)(unsigned)s) : KMAX;
                if constexpr (FILL) v[r] = pval[lv ? pidx[s] : 0];
            }
            wsync();
            const Runs<KPL> o = one_sort<K, KPL, FILL>(a, key, (unsigned)x, (unsigned)(y - x),
                                                       L.mem, lane);
            const int runs = o.total;
            if constexpr (FILL) {
                const int clen = d.ccp[j + 1] - c0;
                if (total + runs > clen - out) bad = 1;
                else one_emit<K, V, KPL>(d, key, v, o, (long long)c0 + out + total, L.mem, lane);
            }
            total += runs;
        }
        if (!FILL && lane == 0) {
            a.wcnt[wb + w] = total;
            atomicAdd(&a.gnnz[g], total);
        }
        if (FILL && a.spec_fill && lane == 0) {
            // at a previous structure's positions: the window must have kept
            // its count
            if (total != a.wcnt[wb + w]) bad = 1;
            atomicAdd(&a.gnnz[g], total);
        }
        wsync();
    }
    if (__builtin_amdgcn_ballot_w64(bad != 0) && threadIdx.x == 0)
        atomicOr(&a.hdr->err, FILL && a.spec_fill ? ERR_RETRY : ERR_GROUP);
}

// ---------------------------------------------------------------- launchers
template <bool MULTI, typename K, typename V, bool FILL>
static hipError_t launch_light_k(const KArgs &a, unsigned mask, int items, hipStream_t s) {
    hipLaunchKernelGGL((k_acc_light<K, V, FILL, MULTI>), dim3(items), dim3(64), 0, s, a, mask);
    return hipGetLastError();
}
template <bool MULTI, typename K, typename V, bool FILL>
static hipError_t launch_one_k(const KArgs &a, int bin, int items, hipStream_t s) {
    if (bin == BIN_SORT0)
        hipLaunchKernelGGL((k_acc_one<K, V, 8, FILL, MULTI>), dim3(items), dim3(64), 0, s, a, bin);
    else
        hipLaunchKernelGGL((k_acc_one<K, V, 16, FILL, MULTI>), dim3(items), dim3(64), 0, s, a, bin);
    return hipGetLastError();
}

template <bool MULTI>
hipError_t launch_acc_light_t(const KArgs &a, unsigned mask, int items, bool wide, bool fill,
                              bool f64, hipStream_t s) {
    if (items <= 0) return hipSuccess;
    using W = unsigned long long;
    if (!fill)
        return wide ? launch_light_k<MULTI, W, float, false>(a, mask, items, s)
                    : launch_light_k<MULTI, unsigned, float, false>(a, mask, items, s);
    if (f64)
        return wide ? launch_light_k<MULTI, W, double, true>(a, mask, items, s)
                    : launch_light_k<MULTI, unsigned, double, true>(a, mask, items, s);
    return wide ? launch_light_k<MULTI, W, float, true>(a, mask, items, s)
                : launch_light_k<MULTI, unsigned, float, true>(a, mask, items, s);
}

template <bool MULTI>
hipError_t launch_acc_one_t(const KArgs &a, int bin, int items, bool wide, bool fill, bool f64,
                            hipStream_t s) {
    if (items <= 0) return hipSuccess;
    using W = unsigned long long;
    if (!fill)
        return wide ? launch_one_k<MULTI, W, float, false>(a, bin, items, s)
                    : launch_one_k<MULTI, unsigned, float, false>(a, bin, items, s);
    if (f64)
        return wide ? launch_one_k<MULTI, W, double, true>(a, bin, items, s)
                    : launch_one_k<MULTI, unsigned, double, true>(a, bin, items, s);
    return wide ? launch_one_k<MULTI, W, float, true>(a, bin, items, s)
                : launch_one_k<MULTI, unsigned, float, true>(a, bin, items, s);
}

template <bool MULTI>
hipError_t launch_heavy_t(const KArgs &a, int ncols, int nwin, bool wide, bool fill, bool f64,
                        hipStream_t s, bool radix, long long heavy_products, int rowbits,
                        int part, int nlong) {
    if (ncols <= 0) return hipSuccess;
    const bool expand = radix ? part == 0 : part == 1;
    if (expand) {
        // the long columns' workgroups end last where the heavy columns do not
        // fill the chip (8 workgroups on each of 256 CUs): split by 4 (400k
        // power law, 1.1k heavy columns, numeric phase: 190 us, split 172; by
        // 8: 180). Where they do, the parts only cost (1M, 3.7k heavy columns:
        // 532 us, split 534, by 8: 537)
        const int split = ncols <= 2048 ? 4 : 1;
        const int grid = ncols + nlong * (split - 1);
        if (!fill) hipLaunchKernelGGL((k_heavy_expand<float, false, MULTI>), dim3(grid), dim3(kBlock), 0, s, a,
                                      split);
        else if (f64) hipLaunchKernelGGL((k_heavy_expand<double, true, MULTI>), dim3(grid), dim3(kBlock), 0, s, a,
                                      split);
        else hipLaunchKernelGGL((k_heavy_expand<float, true, MULTI>), dim3(grid), dim3(kBlock), 0, s, a,
                                      split);
        return hipGetLastError();
    }
    if (radix) return part == 1 ? launch_esc_radix(a, heavy_products, rowbits, fill, f64, s) : hipSuccess;
    if (part == 0) {
        hipLaunchKernelGGL(k_win_map<MULTI>, dim3(ceil_div(ncols, kBlock)), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
    if (part != 2 || nwin <= 0) return hipSuccess;
    if (!fill) {
        if (wide) hipLaunchKernelGGL((k_acc_window<unsigned long long, float, false, MULTI>), dim3(nwin), dim3(64), 0, s, a);
        else hipLaunchKernelGGL((k_acc_window<unsigned, float, false, MULTI>), dim3(nwin), dim3(64), 0, s, a);
    } else if (f64) {
        if (wide) hipLaunchKernelGGL((k_acc_window<unsigned long long, double, true, MULTI>), dim3(nwin), dim3(64), 0, s, a);
        else hipLaunchKernelGGL((k_acc_window<unsigned, double, true, MULTI>), dim3(nwin), dim3(64), 0, s, a);
    } else {
        if (wide) hipLaunchKernelGGL((k_acc_window<unsigned long long, float, true, MULTI>), dim3(nwin), dim3(64), 0, s, a);
        else hipLaunchKernelGGL((k_acc_window<unsigned, float, true, MULTI>), dim3(nwin), dim3(64), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace spg
