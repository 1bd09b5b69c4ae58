// Planning kernels: per-column product count Op_j (Section 3.1), accumulator
// choice (the role of the paper's sort + hybrid switch, Sections 3.1-3.3),
// placement of columns into per-accumulator lists, and the column-pointer scan.
#include <cstddef>

#include "devutil.h"

namespace spg {

// the tile's problem and columns [j0, j1)
__device__ __forceinline__ void tile_columns(const KArgs &a, int &pid, int &j0, int &j1) {
    if (a.nprob == 1) {
        pid = 0;
        j0 = blockIdx.x * a.tile;
        j1 = min(a.single.n, j0 + a.tile);
    } else {
        const int4 tl = a.tiles[blockIdx.x];
        pid = tl.x;
        j0 = tl.y;
        j1 = tl.z;
    }
}

// row windows planned for a heavy column of op products
__device__ __forceinline__ int heavy_windows(int op) { return max(1, (op - 1) / kWinTarget + 1); }

// Totals of the heavy columns into the header; a planned launch whose scratch
// holds fewer products or windows is redone (set_err: the bit goes straight to
// the header, else it is returned).
__device__ __forceinline__ int heavy_totals(const KArgs &a, long long prod, long long win,
                                            bool set_err) {
    a.hdr->heavy_prod = (unsigned long long)prod;
    a.hdr->heavy_win = (int)min(win, 0x7fffffffll);
    const int err = a.direct && a.spec_total >= 0 && (prod > a.heavy_cap || win > a.win_cap) ? ERR_RETRY : 0;
    if (set_err && err) atomicOr(&a.hdr->err, err);
    return err;
}

// The whole header of a launch whose place kernel combines the tiles itself
// (one wavefront, lane b with bin b). With the product-space accumulators the
// header was cleared before and another stream may already raise error bits.
__device__ __forceinline__ void place_header(const KArgs &a, int err, const int *counts,
                                             unsigned long long total, int maxch, long long hprod,
                                             long long hwin) {
    Hdr *h = a.hdr;
    const int b = lane_id();
    const int n = b < NBINS ? counts[b] : 0;
    const int start = wave_incl_scan(n) - n;
    if (b < NBINS) {
        h->bin_count[b] = n;
        h->bin_start[b] = start;
    }
    err &= ERR_CSC | ERR_OPOVF;
    // a planned launch that does not cover a non-empty bin is redone
    if (ballot(n > 0 && !((a.spec_mask >> (b & 31)) & 1u)) && a.spec_total >= 0) err |= ERR_RETRY;
    // and one sized for another product count
    if (a.spec_total >= 0 && total != (unsigned long long)a.spec_total) err |= ERR_RETRY;
    if (b != 0) return;
    h->total_op = total;
    h->big_chunks = maxch;
    if (a.direct) {
        err |= heavy_totals(a, hprod, hwin, false);
        h->later_maxk = 0;
        h->cap_over = 0;
        h->err = err;
    } else if (err) {
        atomicOr(&h->err, err);
    }
}

// The header as (word, sequence number) pairs in mapped host memory, by the
// workgroup whose thread has just written it (see k_publish).
__device__ __forceinline__ void publish_header(const KArgs &a, const PubArgs &pub, int tid,
                                               int nthreads) {
    if (!pub.dst) return;
    __syncthreads();
    const uint32_t *src = (const uint32_t *)a.hdr;
    for (int i = tid; i < pub.nwords; i += nthreads)
        __hip_atomic_store(&pub.dst[i], (unsigned long long)src[i] | ((unsigned long long)pub.seq << 32),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------- classify
// One workgroup per tile of at most a.tile columns of one problem. The tile's
// stored B entries are contiguous; threads walk them flat (coalesced reads of
// B.rowidx, gathers of A.colptr), and add Z^A_k to the owning column's count.
// Every index read here is checked before it is used as an address.
//
// What bounds it: the chain of dependent loads (B's row, A's column pointers)
// of the tile with the most entries, so the tiles are cut fine (plan_tile) and
// a pass's gathers are in flight together with the next pass's row loads; then
// the work per entry, so a column's count is a difference of two prefix sums
// (an LDS search and a 64-bit LDS atomic per entry before). 4096 columns of 40
// entries: 76.5 us in 8 tiles of 512 columns, 6.1 us in 512 tiles of 8; 1000
// columns of 5: 15.5 -> 5.4 us; a million power-law columns (5 M gathers of
// A.colptr): 70 -> 62 us with the prefix sums, a squared grid operator of
// 250,000 columns 16.8 -> 12.0 us. (512 and 1024 threads per workgroup: 69 and
// 78 us before the prefix sums; the loads in flight set the rest.)
__global__ __launch_bounds__(kBlock) void k_classify(KArgs a) {
    constexpr int U = 4, STEP = U * kBlock, PER = kTile / kBlock;
    __shared__ int s_bcp[kTile + 1];
    __shared__ long long s_pre[STEP + 1];  // products before every entry of the pass
    __shared__ long long s_wave[kBlock / 64];
    __shared__ int s_hist[NBINS];
    __shared__ int s_err, s_maxch;
    __shared__ unsigned long long s_tot, s_hp[kHeavyBins];
    __shared__ int s_hw[kHeavyBins];

    int pid, j0, j1;
    tile_columns(a, pid, j0, j1);
    const Prob d = get_prob(a, pid);
    const int nt = j1 - j0;
    const int tid = threadIdx.x;

    for (int c = tid; c <= nt; c += kBlock) s_bcp[c] = d.bcp[j0 + c];
    if (tid < NBINS) s_hist[tid] = 0;
    if (tid < kHeavyBins) { s_hp[tid] = 0; s_hw[tid] = 0; }
    if (tid == 0) { s_err = 0; s_tot = 0; s_maxch = 0; }
    __syncthreads();

    // column pointers of B: monotone, inside [0, nnz], 0 first, nnz last
    int err = 0;
    for (int c = tid; c < nt; c += kBlock)
        if (s_bcp[c + 1] < s_bcp[c]) err = ERR_CSC;
    if (tid == 0) {
        if (s_bcp[0] < 0 || s_bcp[nt] > d.nnzb) err = ERR_CSC;
        if (j0 == 0 && s_bcp[0] != 0) err = ERR_CSC;
        if (j1 == d.n && s_bcp[nt] != d.nnzb) err = ERR_CSC;
        if (j0 == 0) {  // once per problem: A's first and last column pointer
            if (d.acp[0] != 0 || d.acp[d.k] != d.nnza) err = ERR_CSC;
        }
    }
    if (err) atomicOr(&s_err, err);
    __syncthreads();

    const int pb = s_bcp[0], pe = s_bcp[nt];
    const gmem<const int32_t> *__restrict__ bri = to_gmem(d.bri);
    err = 0;
    // with no A columns every stored B entry is out of range (and A.colptr
    // holds one entry: the pair loads below need two)
    if (d.k == 0 && pe > pb) err = ERR_CSC;
    unsigned long long op64[PER];  // products of column tid + kBlock v
#pragma unroll
    for (int v = 0; v < PER; ++v) op64[v] = 0;
    const bool sound = s_err == 0;
    __syncthreads();
    if (sound && d.k > 0 && pe > pb) {
        // Passes of STEP entries, U consecutive ones per thread. A slot past
        // the tile's end reads its last entry, an index out of range reads A's
        // first column pointers; neither result is used. Both column pointers
        // come in one 8-byte load (4-byte alignment is enough for a global
        // load): kc < k, so kc + 1 <= k.
        typedef int int4a __attribute__((ext_vector_type(4), aligned(4)));
        typedef int int4b __attribute__((ext_vector_type(4), aligned(8)));
        int kk[U], kn[U];
        int2a x[U];
        auto rows_at = [&](int p0, int (&k)[U]) {
            const int p = p0 + U * tid;
            if (p + U <= pe) {
                const int4a r = *(const gmem<const int4a> *)(bri + p);
#pragma unroll
                for (int u = 0; u < U; ++u) k[u] = r[u];
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) k[u] = bri[min(p + u, pe - 1)];
            }
        };
        rows_at(pb, kk);
        for (int p0 = pb; p0 < pe; p0 += STEP) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                x[u] = load_pair(d.acp, (kk[u] < 0 || kk[u] >= d.k) ? 0 : kk[u]);
            if (p0 + STEP < pe) rows_at(p0 + STEP, kn);  // in flight beside the gathers
            const int p = p0 + U * tid;
            int s0[U], z[U];
            long long sum = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = kk[u];
                const bool in = p + u < pe;
                const bool ok = k >= 0 && k < d.k && x[u].x >= 0 && x[u].y >= x[u].x && x[u].y <= d.nnza;
                s0[u] = ok ? x[u].x : 0;
                z[u] = (in && ok) ? x[u].y - x[u].x : 0;
                if (in && !ok) err = ERR_CSC;
                sum += z[u];
            }
            // the A column each stored B entry selects, for the accumulators
            int2 *E = a.E + d.ebase + p;
            if (p + U <= pe) {
                *(int4b *)(E) = int4b{s0[0], z[0], s0[1], z[1]};
                *(int4b *)(E + 2) = int4b{s0[2], z[2], s0[3], z[3]};
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (p + u < pe) E[u] = make_int2(s0[u], z[u]);
            }
            const long long inc = wave_incl_scan64(sum);
            if ((tid & 63) == 63) s_wave[tid >> 6] = inc;
            __syncthreads();
            long long run = inc - sum;
            for (int w = 0; w < tid >> 6; ++w) run += s_wave[w];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                s_pre[U * tid + u] = run;
                run += z[u];
            }
            if (tid == kBlock - 1) s_pre[STEP] = run;
            __syncthreads();
#pragma unroll
            for (int v = 0; v < PER; ++v) {
                const int c = tid + kBlock * v;
                if (c < nt) {
                    const int b = min(max(s_bcp[c] - p0, 0), STEP);
                    const int e = min(max(s_bcp[c + 1] - p0, 0), STEP);
                    op64[v] += (unsigned long long)(s_pre[e] - s_pre[b]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) kk[u] = kn[u];
        }
    }
    if (err) atomicOr(&s_err, err);
    __syncthreads();

    const int esc_max = 4 << (a.tune.esc_bins - 1);
    unsigned long long tot = 0;
    int maxch = 0;
    err = 0;
    if (!s_err) {
#pragma unroll
        for (int v = 0; v < PER; ++v) {
            const int c = tid + kBlock * v;
            if (c >= nt) continue;
            const int g = d.col0 + j0 + c;
            if (op64[v] > 0x7fffffffull) { err = ERR_OPOVF; op64[v] = 0x7fffffffull; }
            tot += op64[v];
            const int op = (int)op64[v];
            // the sort-merge bins take a column by its products or its stored B
            // entries, whichever is more (a work item holds both)
            const int size = max(op, s_bcp[c + 1] - s_bcp[c]);
            int bin;
            if (op == 0) bin = BIN_EMPTY;
            else if (size <= esc_max) bin = BIN_ESC0 + max(ceil_log2(size), 2) - 2;
            else if (op > a.tune.t_block) bin = BIN_BLK0 + blk_class(op);
            else if (size <= kSortMax) bin = BIN_SORT0 + max(ceil_log2(size), 9) - 9;
            else bin = BIN_WSORT;
            if (op > a.tune.t_split) maxch = max(maxch, ceil_div(s_bcp[c + 1] - s_bcp[c], kChunkB));
            a.op[g] = op;
            a.binw[g] = bin;
            a.gnnz[g] = 0;
            atomicAdd(&s_hist[bin], 1);
            if (bin >= BIN_SORT2 && bin <= BIN_WSORT) {
                atomicAdd(&s_hp[bin - BIN_SORT2], (unsigned long long)op);
                atomicAdd(&s_hw[bin - BIN_SORT2], heavy_windows(op));
            }
        }
    }
    // tile total of products
    if (err) atomicOr(&s_err, err);
    const long long wtot = wave_sum64((long long)tot);
    if ((tid & 63) == 0) atomicAdd(&s_tot, (unsigned long long)wtot);
    if (maxch) atomicMax(&s_maxch, maxch);
    __syncthreads();
    // the tile's tallies (no device atomics: k_place or k_tally combine them),
    // counts of at most kTile columns and the tile's error bits
    const int t = blockIdx.x;
    if (tid <= NBINS) {
        a.th[tid * a.tpitch + t] = (uint16_t)(tid < NBINS ? s_hist[tid] : s_err);
        if (t == a.ntiles - 1)  // zeros up to the pitch
            for (int x = a.ntiles; x < a.tpitch; ++x) a.th[tid * a.tpitch + x] = 0;
    }
    if (tid < kHeavyBins) {
        a.tprod[tid * a.tpitch + t] = (long long)s_hp[tid];
        a.twin[tid * a.tpitch + t] = s_hw[tid];
    }
    if (tid == 0) {
        a.ttot[t] = (long long)s_tot;
        a.tmax[t] = s_maxch;
        if (s_err) atomicOr(&a.hdr->err, s_err);
    }
}

// ---------------------------------------------------------------- tally
// With more than kSelfTiles tiles: workgroup b < NBINS scans bin b's per-tile
// counts (each tile's first position inside the bin) and writes the bin's
// total; workgroup NBINS the product total, the largest chunk count and the
// error bits; the kHeavyBins after it the heavy columns' products and windows
// per tile, over the heavy bins in bin-list order.
__global__ __launch_bounds__(256) void k_tally(KArgs a) {
    constexpr int T = 256, PT = 8;  // threads, consecutive tiles per thread
    __shared__ int tmp[T / 64 + 1];
    __shared__ long long tmp64[T / 64 + 1];
    __shared__ unsigned long long s_tot;
    __shared__ int s_max, s_err;
    const int tid = threadIdx.x, b = blockIdx.x, nt = a.ntiles;
    if (b < NBINS) {
        int carry = 0;
        for (int t0 = 0; t0 < nt; t0 += T * PT) {
            const int tb = t0 + tid * PT;
            int v[PT], sum = 0;
#pragma unroll
            for (int u = 0; u < PT; ++u) {
                v[u] = tb + u < nt ? a.th[b * a.tpitch + tb + u] : 0;
                sum += v[u];
            }
            int total;
            int run = carry + wg_excl_scan<T>(sum, tmp, total);
#pragma unroll
            for (int u = 0; u < PT; ++u) {
                if (tb + u < nt) a.tbase[b * a.tpitch + tb + u] = run;
                run += v[u];
            }
            carry += total;
        }
        if (tid == 0) {
            a.hdr->bin_count[b] = carry;
            // a planned launch that does not cover a non-empty bin is redone
            if (a.spec_total >= 0 && carry > 0 && !((a.spec_mask >> b) & 1u))
                atomicOr(&a.hdr->err, ERR_RETRY);
        }
    } else if (b == NBINS) {
        if (tid == 0) {
            s_tot = 0;
            s_max = 0;
            s_err = 0;
        }
        __syncthreads();
        unsigned long long tot = 0;
        int mx = 0, err = 0;
        for (int t = tid; t < nt; t += T) {
            tot += (unsigned long long)a.ttot[t];
            mx = max(mx, a.tmax[t]);
            err |= a.th[NBINS * a.tpitch + t];
        }
        atomicAdd(&s_tot, tot);
        atomicMax(&s_max, mx);
        if (err) atomicOr(&s_err, err);
        __syncthreads();
        if (tid == 0) {
            a.hdr->total_op = s_tot;
            a.hdr->big_chunks = s_max;
            // a planned launch sized for another product count is redone
            if (a.spec_total >= 0 && s_tot != (unsigned long long)a.spec_total) s_err |= ERR_RETRY;
            if (s_err) atomicOr(&a.hdr->err, s_err);
        }
    } else {
        // heavy bin c: its windows and products start after those of the
        // heavy bins before it
        const int c = b - NBINS - 1;
        long long pcarry = 0, wcarry = 0;
        for (int q = 0; q <= c; ++q) {
            for (int t0 = 0; t0 < nt; t0 += T * PT) {
                const int tb = t0 + tid * PT;
                long long pv[PT], wv[PT], psum = 0, wsum = 0;
#pragma unroll
                for (int u = 0; u < PT; ++u) {
                    const bool in = tb + u < nt;
                    pv[u] = in ? a.tprod[q * a.tpitch + tb + u] : 0;
                    wv[u] = in ? a.twin[q * a.tpitch + tb + u] : 0;
                    psum += pv[u];
                    wsum += wv[u];
                }
                long long ptot, wtot;
                long long prun = pcarry + wg_excl_scan64<T>(psum, tmp64, ptot);
                long long wrun = wcarry + wg_excl_scan64<T>(wsum, tmp64, wtot);
                if (q == c) {
#pragma unroll
                    for (int u = 0; u < PT; ++u) {
                        if (tb + u < nt) {
                            a.tpbase[c * a.tpitch + tb + u] = prun;
                            a.twbase[c * a.tpitch + tb + u] = (int)wrun;
                        }
                        prun += pv[u];
                        wrun += wv[u];
                    }
                }
                pcarry += ptot;
                wcarry += wtot;
            }
        }
        if (c == kHeavyBins - 1 && tid == 0) heavy_totals(a, pcarry, wcarry, true);
    }
}

hipError_t launch_tally(const KArgs &a, hipStream_t s) {
    if (a.ntiles <= kSelfTiles) return hipSuccess;
    hipLaunchKernelGGL(k_tally, dim3(NBINS + 1 + kHeavyBins), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------- place
// Same tiling. Each tile writes its columns to its range of every bin list in
// column order, so the columns that one wavefront of an accumulator takes lie
// close together (their per-column data and their output in C share cache
// lines). The rank of a column inside its bin is counted with wavefront
// ballots per bin, then the counts of the waves before it. The heavy columns
// (more than 1024 products) also get their first product in the heavy scratch
// (hoff), their first row window (wbase; windows of about kWinTarget products)
// and, in a planned launch, the map of windows to columns as far as its
// scratch holds them (more windows than it holds ask for a redo).
//
// SELF (at most kSelfTiles tiles): every workgroup adds up the tiles before
// its own from the tiles' records (38 bytes a tile, in the L2), which takes
// less than a tally launch before this one; a workgroup of its own writes the
// header. With the header's clearing, a tally, this kernel and a one-workgroup
// plan of the heavy columns as four launches: 6.2 + 5.0 + 2.7 us and the
// clearing for 1000 columns, 4.5 us now; 6.2 + 5.0 + 10.4 us for 4096 columns
// of 1600 products, 9.7 us now. What bounds it is the header's workgroup (one
// thread walking the bins took 5 us) and the chain of its loads. With more
// tiles each workgroup would read too much and k_tally scans the records first.
template <bool SELF>
__global__ __launch_bounds__(kTile) void k_place(KArgs a, PubArgs pub) {
    constexpr int T = kTile, NW = T / 64, ROWS = NBINS + 1;  // one column per thread
    __shared__ int s_base[ROWS], s_total[ROWS], s_start[NBINS];
    __shared__ int s_cnt[NW][NBINS];  // columns of every bin per wave
    __shared__ int s_at[NW][NBINS];   // the wave's first position in every bin
    __shared__ int s_w[NW][kHeavyBins];         // windows, then prefix
    __shared__ long long s_p[NW][kHeavyBins];   // products, then prefix
    __shared__ long long s_hpb[kHeavyBins], s_hpt[kHeavyBins];
    __shared__ long long s_hwb[kHeavyBins], s_hwt[kHeavyBins];
    __shared__ unsigned long long s_tot;
    __shared__ int s_max;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, mt = blockIdx.x;
    if (!SELF) {
        if (__syncthreads_or((__atomic_load_n(&a.hdr->err, __ATOMIC_RELAXED) & (ERR_CSC | ERR_OPOVF)) != 0))
            return;  // every thread takes the same branch
    }
    // one workgroup past the tiles (SELF) has no columns and writes the header
    const bool header = SELF && mt == a.ntiles;
    int pid = 0, j0 = 0, j1 = 0;
    if (!header) tile_columns(a, pid, j0, j1);
    const int col0 = a.nprob == 1 ? 0 : a.table[pid].col0;
    const int nt = j1 - j0;
    // column tid of the tile: its entries and product count load with its bin
    const int32_t *bcp = a.nprob == 1 ? a.single.bcp : a.table[pid].bcp;
    const bool in = tid < nt;
    // (a tile that found malformed input has written no bins: any number may
    // stand there, and it counts into the LDS before the error is known)
    const int bin = in ? (int)min((unsigned)a.binw[col0 + j0 + tid], (unsigned)NBINS - 1u) : -1;
    const int2a bse = in ? load_pair(bcp, j0 + tid) : int2a{0, 0};
    const int op = in ? a.op[col0 + j0 + tid] : 0;
    // row r of the records: bin r's columns per tile; the last row error bits.
    // Every load is issued before any is used.
    constexpr int RW = (ROWS + NW - 1) / NW, CH = (kSelfTiles + 8 * 64 - 1) / (8 * 64);
    uint4 v[SELF ? RW : 1][CH];
    unsigned long long ptot = 0;  // the header's product total and largest chunk count
    int pmax = 0;
    if (SELF) {
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int r = min(w + i * NW, ROWS - 1);
            const uint4 *row = (const uint4 *)(a.th + (size_t)r * a.tpitch);
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int q = c * 64 + lane;
                v[i][c] = 8 * q < a.tpitch ? row[q] : make_uint4(0, 0, 0, 0);
            }
        }
        if (header) {
            if (tid == 0) {
                s_tot = 0;
                s_max = 0;
            }
#pragma unroll
            for (int c = 0; c < (kSelfTiles + T - 1) / T; ++c) {
                const int t = c * T + tid;
                ptot += t < a.ntiles ? (unsigned long long)a.ttot[t] : 0ull;
                pmax = max(pmax, t < a.ntiles ? a.tmax[t] : 0);
            }
        }
    } else if (tid < NBINS) {
        s_base[tid] = a.tbase[tid * a.tpitch + mt];
        s_total[tid] = a.hdr->bin_count[tid];
    }
    // ranks inside the wave, one ballot per bin that occurs in it
    if (lane < NBINS) s_cnt[w][lane] = 0;
    int rank = 0;
    for (unsigned long long todo = ballot(in); todo;) {
        const int b = __builtin_amdgcn_readlane(bin, __builtin_ctzll(todo));
        const unsigned long long m = ballot(bin == b);
        if (bin == b) rank = popc64(m & mask_lt());
        if (lane == 0) s_cnt[w][b] = popc64(m);
        todo &= ~m;
    }
    if (SELF) {
        // a word holds two tiles' counts, summed as pairs of 16 bits (a lane
        // adds at most 24 tiles of kTile columns): all tiles (the pitch is
        // padded with zeros), and those before this one by a mask per word
        static_assert(8 * CH * kTile < 65536, "a lane's counts fit 16 bits");
        unsigned tot[RW], bef[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) tot[i] = bef[i] = 0;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int left = mt - 8 * (c * 64 + lane);  // the lane's tiles before this one
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const unsigned mb = left >= 2 * q + 2 ? ~0u : (left == 2 * q + 1 ? 0xffffu : 0u);
#pragma unroll
                for (int i = 0; i < RW; ++i) {
                    const unsigned x = (&v[i][c].x)[q];
                    // (a tile's error bits repeat at most 24 times in a lane's sum)
                    tot[i] += x;
                    bef[i] += x & mb;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int r = w + i * NW;
            const int total = wave_sum((int)((tot[i] & 0xffffu) + (tot[i] >> 16)));
            const int before = wave_sum((int)((bef[i] & 0xffffu) + (bef[i] >> 16)));
            if (lane == 0 && r < ROWS) {
                s_base[r] = before;
                s_total[r] = total;
            }
        }
    }
    __syncthreads();
    if (header) {
        const unsigned long long p = (unsigned long long)wave_sum64((long long)ptot);
        const int m = __builtin_amdgcn_readlane(wave_incl_max(pmax), 63);
        if (lane == 0) {
            atomicAdd(&s_tot, p);
            atomicMax(&s_max, m);
        }
    }
    if (SELF && s_total[NBINS] != 0) {
        // some tile has found an error: which one, tile by tile
        __shared__ int s_err;
        if (tid == 0) s_err = 0;
        __syncthreads();
        int e = 0;
        for (int t = tid; t < a.ntiles; t += T) e |= a.th[NBINS * a.tpitch + t];
        if (e) atomicOr(&s_err, e);
        __syncthreads();
        if (header) {
            if (w == 0) place_header(a, s_err, s_total, 0, 0, 0, 0);
            publish_header(a, pub, tid, T);
        }
        return;  // every thread takes the same branch
    }
    // exclusive prefix over the waves per bin, from the tile's first
    // position in the bin
    if (tid < NBINS) {
        int start = 0;
#pragma unroll
        for (int b = 0; b < NBINS; ++b) start += b < tid ? s_total[b] : 0;
        s_start[tid] = start;
        if (!SELF && mt == 0) a.hdr->bin_start[tid] = start;
        int run = start + s_base[tid];
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            s_at[x][tid] = run;
            run += s_cnt[x][tid];
        }
    }
    int heavy = 0, nheavy = 0;
    for (int b = BIN_SORT2; b <= BIN_WSORT; ++b) nheavy += s_total[b];
    if (a.direct && nheavy > 0)
        for (int b = BIN_SORT2; b <= BIN_WSORT; ++b)
#pragma unroll
            for (int x = 0; x < NW; ++x) heavy += s_cnt[x][b];
    // the heavy columns' products and windows before the tile
    const bool heavy_sums = a.direct && nheavy > 0 && (heavy || header);
    int wex = 0;
    long long pex = 0;
    if (heavy_sums) {
        if (SELF) {
            // one wave per heavy bin and kind of sum, every load issued first
            constexpr int PT = kSelfTiles / 64;
            const int q = w >> 1;
            if (q < kHeavyBins && (w & 1)) {
                int x[PT], before = 0, total = 0;
#pragma unroll
                for (int c = 0; c < PT; ++c)
                    x[c] = c * 64 + lane < a.ntiles ? a.twin[q * a.tpitch + c * 64 + lane] : 0;
#pragma unroll
                for (int c = 0; c < PT; ++c) {
                    total += x[c];
                    before += c * 64 + lane < mt ? x[c] : 0;
                }
                const long long wt = wave_sum64(total), wb = wave_sum64(before);
                if (lane == 0) {
                    s_hwt[q] = wt;
                    s_hwb[q] = wb;
                }
            } else if (q < kHeavyBins) {
                long long x[PT], before = 0, total = 0;
#pragma unroll
                for (int c = 0; c < PT; ++c)
                    x[c] = c * 64 + lane < a.ntiles ? a.tprod[q * a.tpitch + c * 64 + lane] : 0;
#pragma unroll
                for (int c = 0; c < PT; ++c) {
                    total += x[c];
                    before += c * 64 + lane < mt ? x[c] : 0;
                }
                const long long pt = wave_sum64(total), pb = wave_sum64(before);
                if (lane == 0) {
                    s_hpt[q] = pt;
                    s_hpb[q] = pb;
                }
            }
        } else if (tid < kHeavyBins) {
            s_hpb[tid] = a.tpbase[tid * a.tpitch + mt];
            s_hwb[tid] = a.twbase[tid * a.tpitch + mt];
            s_hpt[tid] = 0;
            s_hwt[tid] = 0;
        }
        if (heavy) {
            // prefix inside the wave over the columns of the same heavy bin
#pragma unroll 1
            for (int c = 0; c < kHeavyBins; ++c) {
                const bool mine = bin == BIN_SORT2 + c;
                int wt = 0;
                long long pt = 0;
                if (ballot(mine)) {
                    const int nw = mine ? heavy_windows(op) : 0;
                    const long long p = mine ? op : 0;
                    const int wi = wave_incl_scan(nw);
                    const long long pi = wave_incl_scan64(p);
                    if (mine) {
                        wex = wi - nw;
                        pex = pi - p;
                    }
                    wt = __builtin_amdgcn_readlane(wi, 63);
                    pt = wave_last64(pi);
                }
                if (lane == 0) {
                    s_w[w][c] = wt;
                    s_p[w][c] = pt;
                }
            }
        }
    }
    __syncthreads();
    if (header) {
        if (w == 0) {
            long long p = 0, q = 0;
            if (heavy_sums)
                for (int c = 0; c < kHeavyBins; ++c) {
                    p += s_hpt[c];
                    q += s_hwt[c];
                }
            place_header(a, 0, s_total, s_tot, s_max, p, q);
        }
        publish_header(a, pub, tid, T);
        return;
    }
    if (heavy) {
        if (tid < kHeavyBins) {
            long long p = s_hpb[tid], q = s_hwb[tid];
            if (SELF)
                for (int c = 0; c < tid; ++c) {  // the heavy bins before this one
                    p += s_hpt[c];
                    q += s_hwt[c];
                }
#pragma unroll 1
            for (int x = 0; x < NW; ++x) {
                const long long pv = s_p[x][tid];
                const int wv = s_w[x][tid];
                s_p[x][tid] = p;
                s_w[x][tid] = (int)q;
                p += pv;
                q += wv;
            }
        }
        __syncthreads();
    }
    if (!in) return;
    const int g = col0 + j0 + tid, at = s_at[w][bin] + rank;
    a.binlist[at] = make_int4(g, bse.x, bse.y - bse.x, op);
    if (heavy && bin >= BIN_SORT2 && bin <= BIN_WSORT) {
        const int h = bin - BIN_SORT2, li = at - s_start[BIN_SORT2];
        const int wr = s_w[w][h] + wex, we = wr + heavy_windows(op);
        a.hoff[li] = s_p[w][h] + pex;
        a.wbase[li] = wr;
        if (a.spec_total >= 0)
            for (int q = wr; q < we && q < a.win_cap; ++q) a.winmap[q] = li;
    }
}

// ---------------------------------------------------------------- scans
// Exclusive prefix sums in 64-bit, in two launches: per-block sums, then a
// down-sweep in which every block adds up the sums of the blocks before it
// itself (at most a few thousand values) and scans its kScanBlock elements.
// The product-space down-sweep also marks the tile starts.
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const int32_t *__restrict__ in, int n,
                                                        long long *__restrict__ bsum) {
    __shared__ long long s[kBlock / 64];
    const int base = blockIdx.x * kScanBlock;
    long long v = 0;
#pragma unroll
    for (int u = 0; u < kScanBlock / kBlock; ++u) {
        int i = base + u * kBlock + threadIdx.x;
        if (i < n) v += in[i];
    }
    v = wave_sum64(v);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int w = 0; w < kBlock / 64; ++w) t += s[w];
        bsum[blockIdx.x] = t;
    }
}

// Block-level scan of kScanBlock int32 values starting at `base` (zero past
// n). Returns, per thread, the exclusive prefixes of its PER consecutive
// elements (global: including the sums of the earlier blocks) and the total
// of all blocks up to this one.
struct ScanOut {
    static constexpr int PER = kScanBlock / kBlock;
    long long pre[PER];
    long long block_end;  // prefix after this block's last element
};

__device__ __forceinline__ void block_scan_down(const int32_t *__restrict__ in, int n,
                                                const long long *__restrict__ bsum,
                                                long long *s, ScanOut &o) {
    constexpr int PER = ScanOut::PER, NW = kBlock / 64;
    const int base = blockIdx.x * kScanBlock + threadIdx.x * PER;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    int v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u] = base + u < n ? in[base + u] : 0;
    // sums of the earlier blocks
    long long before = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kBlock) before += bsum[b];
    before = wave_sum64(before);
    long long run = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        o.pre[u] = run;
        run += v[u];
    }
    const long long inc = wave_incl_scan64(run);
    if (l == 63) {
        s[w] = inc;
        s[NW + w] = before;
    }
    __syncthreads();
    long long off = 0, all = 0, own = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        off += s[NW + q];
        if (q < w) own += s[q];
        all += s[q];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) o.pre[u] += off + own + inc - run;
    o.block_end = off + all;
}

// (word, sequence number) pairs of the header and totals to mapped host
// memory: see k_publish. Words the launch itself has set come from the caller.
__device__ __forceinline__ void publish_words(const uint32_t *src, const PubArgs &pub, int tid,
                                              int nthreads, int err, int cap_over,
                                              long long total) {
    constexpr int W_ERR = offsetof(Hdr, err) / 4, W_CAP = offsetof(Hdr, cap_over) / 4;
    constexpr int W_TOT = kHdrWords;
    for (int i = tid; i < pub.nwords; i += nthreads) {
        uint32_t v = src[i];
        if (i == W_ERR) v |= (uint32_t)err;
        if (i == W_CAP) v |= (uint32_t)cap_over;
        if (i == W_TOT) v = (uint32_t)total;
        if (i == W_TOT + 1) v = (uint32_t)((unsigned long long)total >> 32);
        __hip_atomic_store(&pub.dst[i], (unsigned long long)v | ((unsigned long long)pub.seq << 32),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// end of a single problem's scan (one thread): total, capacity and overflow
// flags, for the device's header and the published copy
__device__ __forceinline__ void scan_total(const KArgs &a, long long total, long long *totals,
                                           int &err, int &cap) {
    err = total > 0x7fffffffll ? ERR_NNZOVF : 0;
    a.single.ccp[a.ncols] = (int32_t)total;
    if (a.save) a.save[a.ncols] = (int32_t)total;
    totals[0] = total;
    // a numeric phase queued behind this scan must not write past the
    // caller's arrays
    cap = total > a.out_cap ? 1 : 0;
    if (cap) a.hdr->cap_over = 1;
    if (err) atomicOr(&a.hdr->err, err);
}

// A single problem of at most kScanSmall columns: column pointers, total and
// publication in one workgroup of one launch (three launches of 4 to 5 us
// each, and the gaps between them, otherwise).
constexpr int kScanSmallT = 1024, kScanSmallPer = 16;
constexpr int kScanSmall = kScanSmallT * kScanSmallPer;
__global__ __launch_bounds__(kScanSmallT) void k_scan_small(KArgs a, long long *totals,
                                                            PubArgs pub) {
    constexpr int PER = kScanSmallPer;
    __shared__ long long tmp[kScanSmallT / 64 + 1];
    __shared__ int s_err, s_cap;
    const int n = a.ncols, per = (n + kScanSmallT - 1) / kScanSmallT;
    const int base = threadIdx.x * per;
    int v[PER];
    long long sum = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        v[u] = u < per && base + u < n ? a.gnnz[base + u] : 0;
        sum += v[u];
    }
    long long total;
    long long run = wg_excl_scan64<kScanSmallT>(sum, tmp, total);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (u < per && base + u < n) {
            a.single.ccp[base + u] = (int32_t)run;
            if (a.save) a.save[base + u] = (int32_t)run;
        }
        run += v[u];
    }
    if (threadIdx.x == 0) scan_total(a, total, totals, s_err, s_cap);
    if (!pub.dst) return;
    __syncthreads();
    publish_words((const uint32_t *)a.hdr, pub, threadIdx.x, kScanSmallT, s_err, s_cap, total);
}

// C column pointers from the per-column counts. For one problem the int32 column pointers are written
// directly (with an overflow check); for several problems the 64-bit global
// prefix is kept in gcp and k_scan_finish cuts it per problem.
__global__ __launch_bounds__(kBlock) void k_scan_down(KArgs a, long long *__restrict__ gcp,
                                                      const long long *__restrict__ bsum,
                                                      long long *totals, PubArgs pub) {
    __shared__ long long s[2 * kBlock / 64];
    __shared__ int s_err, s_cap;
    const int n = a.ncols;
    ScanOut o;
    block_scan_down(a.gnnz, n, bsum, s, o);
#pragma unroll
    for (int u = 0; u < ScanOut::PER; ++u) {
        const int i = blockIdx.x * kScanBlock + threadIdx.x * ScanOut::PER + u;
        if (i >= n) break;
        if (a.nprob == 1) {
            a.single.ccp[i] = (int32_t)o.pre[u];  // the total is checked below
            if (a.save) a.save[i] = (int32_t)o.pre[u];
        } else {
            gcp[i] = o.pre[u];
        }
    }
    if (blockIdx.x != gridDim.x - 1) return;
    if (a.nprob > 1) {
        if (threadIdx.x == 0) gcp[n] = o.block_end;
        return;
    }
    if (threadIdx.x == 0) scan_total(a, o.block_end, totals, s_err, s_cap);
    if (!pub.dst) return;
    __syncthreads();
    publish_words((const uint32_t *)a.hdr, pub, threadIdx.x, kBlock, s_err, s_cap, o.block_end);
}

__global__ __launch_bounds__(kBlock) void k_scan_finish(KArgs a, const long long *__restrict__ gcp,
                                                        long long *__restrict__ totals) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < a.ncols) {
        const int pid = find_prob(a, i);
        const Prob &d = a.table[pid];
        long long v = gcp[i] - gcp[d.col0];
        d.ccp[i - d.col0] = (int32_t)v;  // per-problem total checked below
    }
    if (i < a.nprob) {
        const Prob &d = a.table[i];
        long long t = gcp[d.col0 + d.n] - gcp[d.col0];
        if (t > 0x7fffffffll) atomicOr(&a.hdr->err, ERR_NNZOVF);
        d.ccp[d.n] = (int32_t)(t > 0x7fffffffll ? 0x7fffffffll : t);
        totals[i] = t;
    }
}

// First product of every global column (exclusive scan of Op_j), and the
// product-balanced tiles: column g starts the tiles t with
// P(g - 1) < t * kProdTile <= P(g); the tiles after the last column's first
// product are empty.
__global__ __launch_bounds__(kBlock) void k_prod_down(KArgs a, const long long *__restrict__ bsum) {
    __shared__ long long s[2 * kBlock / 64];
    if (__syncthreads_or(__atomic_load_n(&a.hdr->err, __ATOMIC_RELAXED) != 0))
        return;  // every thread takes the same branch
    const int n = a.ncols;
    ScanOut o;
    block_scan_down(a.op, n, bsum, s, o);
    // a launch planned from an earlier call's sizes may run before the tally
    // has compared them: products beyond the product space carved for that
    // call stop the expansion here
    if (a.spec_total >= 0 && o.block_end > a.spec_total) {
        if (threadIdx.x == 0) atomicOr(&a.hdr->err, ERR_RETRY);
        return;
    }
#pragma unroll
    for (int u = 0; u < ScanOut::PER; ++u) {
        const int g = blockIdx.x * kScanBlock + threadIdx.x * ScanOut::PER + u;
        if (g >= n) break;
        const long long pg = o.pre[u];
        a.colprod[g] = pg;
        const long long t_hi = pg / kProdTile;
        const long long t_lo = g == 0 ? 0 : (pg - a.op[g - 1]) / kProdTile + 1;
        for (long long t = t_lo; t <= t_hi && t < a.nptiles; ++t) a.tilestart[t] = g;
        if (g == n - 1)
            for (long long t = t_hi + 1; t <= a.nptiles; ++t) a.tilestart[t] = n;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) a.colprod[n] = o.block_end;
}

// ---------------------------------------------------------------- launchers
hipError_t launch_prod_offsets(const KArgs &a, long long *bsum, int nbsum, hipStream_t s) {
    if (a.ncols <= 0) return hipSuccess;
    const int nblk = ceil_div(a.ncols, kScanBlock);
    if (nblk > nbsum) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_scan_reduce, dim3(nblk), dim3(kBlock), 0, s, (const int32_t *)a.op,
                       a.ncols, bsum);
    hipLaunchKernelGGL(k_prod_down, dim3(nblk), dim3(kBlock), 0, s, a, (const long long *)bsum);
    return hipGetLastError();
}

hipError_t launch_classify(const KArgs &a, hipStream_t s) {
    if (a.ntiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_classify, dim3(a.ntiles), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_place(const KArgs &a, const PubArgs &pub, hipStream_t s) {
    if (a.ntiles == 0) return hipSuccess;
    if (a.ntiles <= kSelfTiles)
        hipLaunchKernelGGL(k_place<true>, dim3(a.ntiles + 1), dim3(kTile), 0, s, a, pub);
    else
        hipLaunchKernelGGL(k_place<false>, dim3(a.ntiles), dim3(kTile), 0, s, a, pub);
    return hipGetLastError();
}

hipError_t launch_scan(const KArgs &a, long long *gcp, long long *bsum, int nblk,
                       long long *totals, const PubArgs &pub, hipStream_t s) {
    if (a.nprob == 1 && a.ncols > 0 && a.ncols <= kScanSmall) {
        hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(kScanSmallT), 0, s, a, totals, pub);
        return hipGetLastError();
    }
    if (a.ncols > 0) {
        hipLaunchKernelGGL(k_scan_reduce, dim3(nblk), dim3(kBlock), 0, s,
                           (const int32_t *)a.gnnz, a.ncols, bsum);
        hipLaunchKernelGGL(k_scan_down, dim3(nblk), dim3(kBlock), 0, s, a, gcp,
                           (const long long *)bsum, totals, pub);
    }
    if (a.nprob > 1) {
        int n = a.ncols > a.nprob ? a.ncols : a.nprob;
        hipLaunchKernelGGL(k_scan_finish, dim3(ceil_div(n, kBlock)), dim3(kBlock), 0, s, a,
                           (const long long *)gcp, totals);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- publish
// Copies the header and the per-problem totals (nwords 32-bit words) to mapped
// host memory, each word beside the call's sequence number in one 8-byte
// store, so the host can read them as soon as the symbolic phase ends while
// later work stays queued behind it. A word is current when its pair carries
// the current number: no fence or cache write-back is needed. (A single
// problem's scan publishes by itself.)
__global__ __launch_bounds__(64) void k_publish(const uint32_t *__restrict__ src, PubArgs pub) {
    for (int i = threadIdx.x; i < pub.nwords; i += 64)
        __hip_atomic_store(&pub.dst[i], (unsigned long long)src[i] | ((unsigned long long)pub.seq << 32),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_publish(const void *src, const PubArgs &pub, hipStream_t s) {
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, (const uint32_t *)src, pub);
    return hipGetLastError();
}

}  // namespace spg
