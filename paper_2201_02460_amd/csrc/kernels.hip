// gfx950 kernels of the exhaustive k-order epistasis scan.
//
// Paper mapping:
//   pack_kernel / singles_kernel  genotype tables of single SNPs (Section 2.1)
//   scan_persistent               enumeration (Algorithm 1), contingency
//                                 tables (Section 2.2), mutual information
//                                 (Section 2.3, Equations 1-3), best-K
//                                 retention (Section 2.4)
//   merge_part/final_kernel       final best-K selection (two stages)
//   finalize_kernel               combinations, scores and full 2 x 3^k
//                                 tables of the retained combinations
//
// Counting.  The paper intersects genotype rows with AND and counts bits.  A
// cell of a combination's table is popcount(AND of one row per SNP).  Here a
// lane counts the cells of one combination; the rows of SNPs shared by every
// lane of the wave (the prefix of Algorithm 1) are staged once per work item
// in the wave's LDS slot and read back with broadcast loads, so each cell of
// each 32-individual word costs one v_bitop3_b32 (three-input AND) and one
// v_bcnt_u32_b32 (popcount + accumulate).
//
// Reduced cells (kF2, kF3).  Only cells whose genotypes are all 0 or 1 are
// counted.  Every other cell follows exactly by inclusion-exclusion from
// counts of sub-combinations: the indicator of genotype 2 is 1 minus the
// indicators of genotypes 0 and 1, so a cell with genotype 2 at SNP t equals
// the table of the combination without SNP t minus the two cells with
// genotype 0 and 1 at t.  Order 2 needs the single-SNP counts, order 3 the
// pair sub-table (written by the kF2Emit variant) as well.  The integers are
// those of counting all 3^k cells.
//
// Score.  N * MI = sum_xy n_xy ln n_xy - sum_x n_x ln n_x - sum_y n_y ln n_y
// + N ln N (Equation 1 with p = n / N).  Each n ln n is read from a table of
// round(n ln n * 2^shift) and summed in int64, so the score of a combination
// is the same integer whatever kernel, tile or batch computes it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <type_traits>

#include "epi_internal.hpp"

namespace epi {

typedef __attribute__((address_space(4))) const v4u cv4u;  // wave-uniform rows: scalar loads
typedef __attribute__((address_space(1))) const v4u gv4u;  // per-lane rows: vector loads

#define EPI_DEV __device__ __forceinline__

// popcount(x) + acc as one v_bcnt_u32_b32 (the compiler would otherwise
// reassociate chains of popcounts into extra v_add3 instructions).
EPI_DEV unsigned bcnt_acc(unsigned x, unsigned acc) {
    unsigned r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
    return r;
}

// a + b + c as one v_add3_u32 (the compiler splits sums with a subtracted
// term into two-operand adds and subtracts).
EPI_DEV unsigned add3(unsigned a, unsigned b, unsigned c) {
    unsigned r;
    asm("v_add3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

EPI_DEV unsigned long long rfl64(unsigned long long v) {
    unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

EPI_DEV unsigned long long readlane64(unsigned long long v, int lane) {
    unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane);
    unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane);
    return ((unsigned long long)hi << 32) | lo;
}

EPI_DEV int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Orders this wave's LDS accesses (lane-0 writes before all-lane reads) without
// a workgroup barrier: the waves of a workgroup run independently.
EPI_DEV void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

EPI_DEV unsigned lane_prefix(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Pin a wave-uniform value to a scalar register (values decoded with VALU
// arithmetic, such as integer division, would otherwise stay in VGPRs and
// turn the uniform mask-row loads into vector loads).
EPI_DEV int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

EPI_DEV unsigned long long bias(long long v) { return (unsigned long long)v ^ 0x8000000000000000ull; }
EPI_DEV long long unbias(unsigned long long v) { return (long long)(v ^ 0x8000000000000000ull); }

EPI_DEV long long load_thr(unsigned long long *p) {
    return unbias(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

EPI_DEV bool better(long long an, unsigned long long ak, long long bn, unsigned long long bk) {
    return an > bn || (an == bn && ak < bk);
}

// ---------------------------------------------------------------------------
// Score histogram (layout in epi_internal.hpp).  A combination whose exact num
// enters a wave's list is counted once, in the bin of its leading bit and the
// next kHistFineBits bits; a bin's lower edge is at most the num of everything
// counted in it.  Each combination is scored by one wave only, so K counts at
// or above an edge are K distinct combinations at least that good: nothing
// below the edge can be in the best K.  Counts read while other waves add to
// them are never above the true ones, and leaving bins out only lowers a sum,
// so a bound taken from any part of the histogram is valid.
// ---------------------------------------------------------------------------
EPI_DEV int hist_bin(long long num) {  // num > 0
    const unsigned long long v = (unsigned long long)num;
    const int e = 63 - __builtin_clzll(v);
    const unsigned f = e >= kHistFineBits ? (unsigned)(v >> (e - kHistFineBits)) : (unsigned)(v << (kHistFineBits - e));
    return e * kHistFine + (int)(f & (kHistFine - 1));
}

EPI_DEV long long hist_edge(int bin) {
    const int e = bin / kHistFine;
    const unsigned long long top = (unsigned long long)(kHistFine + bin % kHistFine);
    return (long long)(e >= kHistFineBits ? top << (e - kHistFineBits) : top >> (kHistFineBits - e));
}

EPI_DEV unsigned wave_scan_incl(unsigned v) {
    const int lane = lane_id();
    #pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const unsigned o = __shfl_up(v, off);
        if (lane >= off) v += o;
    }
    return v;
}

// Largest lower edge with at least K counted combinations at or above it, or
// INT64_MIN.  The sum starts one leading-bit position above `top` (the
// highest bin this wave has counted) and runs down over at most two windows
// of 64 bins: a few round trips, however the scores are scaled.
EPI_DEV long long hist_bound(const unsigned *h, int K, int top) {
    const int lane = lane_id();
    int start = top + kHistFine;
    start = start < kHistTop ? start : kHistTop;
    unsigned carry = 0;
    #pragma unroll 1
    for (int w = 0; w < 2; ++w, start -= kWave) {
        const int b = start - lane;
        const unsigned c = b >= 0 ? __hip_atomic_load(h + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        const unsigned cs = wave_scan_incl(c) + carry;
        const unsigned long long m = __ballot(cs >= (unsigned)K);
        if (m) return hist_edge(start - (int)__builtin_ctzll(m));
        carry = (unsigned)__builtin_amdgcn_readlane((int)cs, kWave - 1);
        if (start < kWave) break;
    }
    return (long long)0x8000000000000000ull;
}

// The same over the whole histogram: each lane sums one leading-bit position
// (highest first), then the wave looks inside the one where the sum reaches K.
EPI_DEV long long hist_bound_all(const unsigned *h, int K) {
    const int lane = lane_id(), oct = 63 - lane;
    unsigned s = 0;
    if (oct < 63) {  // position 63 is never counted (its last word is the pilot counter)
        #pragma unroll
        for (int b = 0; b < kHistFine; ++b)
            s += __hip_atomic_load(h + oct * kHistFine + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const unsigned cs = wave_scan_incl(s);
    const unsigned long long m = __ballot(cs >= (unsigned)K);
    if (!m) return (long long)0x8000000000000000ull;
    const int src = (int)__builtin_ctzll(m);
    const unsigned above = (unsigned)__builtin_amdgcn_readlane((int)(cs - s), src);
    const int top = (63 - src) * kHistFine + kHistFine - 1;
    const unsigned c =
        lane < kHistFine ? __hip_atomic_load(h + top - lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    const unsigned long long m2 = __ballot(wave_scan_incl(c) + above >= (unsigned)K);
    return m2 ? hist_edge(top - (int)__builtin_ctzll(m2)) : hist_edge(top - kHistFine + 1);
}

// Rank of pair (x, y), x < y, in the lexicographic order of the pairs of M.
EPI_DEV unsigned long long lexpair(long long x, long long y, long long M) {
    return (unsigned long long)(x * (2 * M - x - 1) / 2 + (y - x - 1));
}

// Rank of pair (x, x + 1): x (2M - x - 1) / 2.  Both factors stay below 2^24
// (M < 2^23), which lets the product use the 24-bit multipliers.
EPI_DEV unsigned long long pair_row(int x, int M) {
    const unsigned a = (unsigned)x & 0xffffffu, b = (unsigned)(2 * M - x - 1) & 0xffffffu;
    return ((unsigned long long)a * (unsigned long long)b) >> 1;
}

// Valid-individual bits of words 4*w4 .. 4*w4+3 of a class of n individuals.
EPI_DEV v4u valid_mask(int n, int w4) {
    v4u v;
    #pragma unroll
    for (int q = 0; q < 4; ++q) {
        int left = n - 32 * (4 * w4 + q);
        v[q] = left >= 32 ? 0xffffffffu : (left <= 0 ? 0u : ((1u << left) - 1u));
    }
    return v;
}

// In-place inclusion-exclusion over a 3^2 / 3^3 table whose index 2 along an
// axis holds the marginal over that SNP on input and genotype 2 on output.
EPI_DEV void mobius2(int (&R)[9]) {
    #pragma unroll
    for (int e = 0; e < 3; ++e) R[6 + e] -= R[e] + R[3 + e];
    #pragma unroll
    for (int a = 0; a < 3; ++a) R[3 * a + 2] -= R[3 * a] + R[3 * a + 1];
}

EPI_DEV void mobius3(int (&R)[27]) {
    #pragma unroll
    for (int r = 0; r < 9; ++r) R[18 + r] -= R[r] + R[9 + r];
    #pragma unroll
    for (int a = 0; a < 3; ++a)
        #pragma unroll
        for (int e = 0; e < 3; ++e) R[9 * a + 6 + e] -= R[9 * a + e] + R[9 * a + 3 + e];
    #pragma unroll
    for (int ab = 0; ab < 9; ++ab) R[3 * ab + 2] -= R[3 * ab] + R[3 * ab + 1];
}

template <class T>
EPI_DEV void mobius4(T (&R)[81]) {
    #pragma unroll
    for (int st = 27; st >= 1; st /= 3)
        #pragma unroll
        for (int x = 0; x < 81; ++x)
            if ((x / st) % 3 == 2) R[x] -= R[x - 2 * st] + R[x - st];
}

// Cells whose base-3 index has an odd number of digits 2, held as B - 4n in
// the signed cell form.
constexpr bool odd_twos(int x) { return x == 0 ? false : ((x % 3 == 2) != odd_twos(x / 3)); }

// Sub-table passes keep no best-K list.
EPI_DEV bool is_emit(int variant) { return variant == kF2Emit || variant == kF3Emit; }

// Colex rank of x < y: C(y,2) + x.
EPI_DEV unsigned long long colex2(int x, int y) {
    const unsigned long long Y = (unsigned long long)y;
    return Y * (Y - 1) / 2 + (unsigned long long)x;
}

// Colex rank of x < y < z: C(z,3) + C(y,2) + x (z < 2^21).
EPI_DEV unsigned long long colex3(int x, int y, int z) {
    const unsigned long long Z = (unsigned long long)z, Y = (unsigned long long)y;
    return Z * (Z - 1) * (Z - 2) / 6 + Y * (Y - 1) / 2 + (unsigned long long)x;
}

// ---------------------------------------------------------------------------
// Per-wave best-K list in LDS (unsorted) with its current worst entry.
// ---------------------------------------------------------------------------
struct TopK {
    int n, K, wi;
    int cap;         // entries of the list in LDS (list_cap of the launch's largest K)
    long long wn;
    unsigned long long wk;
    unsigned *hist;  // the task's score histogram (null: none)
    int added;       // combinations counted since the bound was last taken
    int top;         // highest histogram bin this wave has counted (-1: none)
    unsigned long long dsum;  // checking launches: this lane's digest sum and count since the last flush
    unsigned dn;
    int xl;          // kX: SNP l of the wave's last item (a guess for the next)
    int nohist;      // the item's combinations are already in the histogram (a pilot item)
};

// ---------------------------------------------------------------------------
// Completeness check (checking launches only; definition in
// epi_internal.hpp): every scored combination adds mix64(h ^ s) to its
// lane's sum, flushed to the task's two counters when the wave leaves the
// task.
// ---------------------------------------------------------------------------
template <int K>
EPI_DEV unsigned long long combo_hash(const int (&c)[K]) {
    unsigned long long h = 0;
    #pragma unroll
    for (int t = 0; t < K; ++t) h = mix64(h + (unsigned long long)c[t] + 1ull);
    return h;
}

EPI_DEV void digest_add(TopK &t, bool valid, unsigned long long h, unsigned long long s) {
    if (valid) {
        t.dsum += mix64(h ^ s);
        t.dn += 1;
    }
}

// Weighted sum of a table held as plain counts F[class][x].
template <int CELLS, class T>
EPI_DEV unsigned long long table_sum(const T (&F0)[CELLS], const T (&F1)[CELLS]) {
    unsigned long long s = 0;
    #pragma unroll
    for (int x = 0; x < CELLS; ++x)
        s += (unsigned long long)(unsigned)F0[x] * cell_weight(0, x) + (unsigned long long)(unsigned)F1[x] * cell_weight(1, x);
    return s;
}

EPI_DEV void digest_flush(TopK &t, const Task &task) {
    unsigned long long s = t.dsum, n = t.dn;
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s += __shfl_xor(s, off);
        n += __shfl_xor(n, off);
    }
    if (lane_id() == 0 && task.digest) {
        atomicAdd(task.digest, n);
        atomicAdd(task.digest + 1, s);
    }
    t.dsum = 0;
    t.dn = 0;
}

// Count the combinations of the lanes with `counted` set: one atomic per
// distinct bin of the wave, with the number of its lanes in that bin.
EPI_DEV void hist_add(TopK &t, bool counted, long long num) {
    counted = counted && num > 0;
    unsigned long long pend = __ballot(counted);
    if (!pend) return;
    const int b = counted ? hist_bin(num) : -1;
    t.added = 1;
    while (pend) {
        const int src = (int)__builtin_ctzll(pend);
        const int bs = __builtin_amdgcn_readlane(b, src);
        const unsigned long long same = pend & __ballot(b == bs);
        if (lane_id() == src)
            __hip_atomic_fetch_add(t.hist + bs, (unsigned)__popcll(same), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        t.top = bs > t.top ? bs : t.top;
        pend &= ~same;
    }
}

EPI_DEV void tk_recompute(TopK &t, const Cand *list) {
    const int lane = lane_id();
    long long bn = 0;
    unsigned long long bk = 0;
    int bi = -1;
    for (int i = lane; i < t.n; i += kWave) {
        Cand c = list[i];
        if (bi < 0 || better(bn, bk, c.num, c.key)) {
            bn = c.num;
            bk = c.key;
            bi = i;
        }
    }
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        long long on = __shfl_xor(bn, off);
        unsigned long long ok = __shfl_xor(bk, off);
        int oi = __shfl_xor(bi, off);
        if (oi >= 0 && (bi < 0 || better(bn, bk, on, ok))) {
            bn = on;
            bk = ok;
            bi = oi;
        }
    }
    t.wn = (long long)rfl64((unsigned long long)bn);
    t.wk = rfl64(bk);
    t.wi = __builtin_amdgcn_readfirstlane(bi);
}

// Power of two a list of n entries is sorted in (at least 64).
EPI_DEV int tk_sort_size(int n) {
    int P = 64;
    while (P < n) P <<= 1;
    return P;
}

// Sort the first n entries of a wave's list best first, in place (entries
// n .. P - 1, P = tk_sort_size(n), hold the worst value meanwhile: the
// caller makes sure the list has P entries).  Bitonic network, each lane a
// pair per compare-exchange step.
EPI_DEV void tk_sort(Cand *a, int n) {
    const int P = tk_sort_size(n);
    for (int i = n + lane_id(); i < P; i += kWave) a[i] = Cand{(long long)0x8000000000000000ull, ~0ull};
    wave_sync();
    #pragma unroll 1
    for (int k = 2; k <= P; k <<= 1) {
        #pragma unroll 1
        for (int j = k >> 1; j > 0; j >>= 1) {
            #pragma unroll 1
            for (int q = lane_id(); q < P / 2; q += kWave) {
                const int i = ((q & ~(j - 1)) << 1) | (q & (j - 1));
                const int l = i | j;
                const Cand x = a[i], y = a[l];
                // best first where bit k of i is clear, worst first elsewhere
                const bool swap = (i & k) == 0 ? better(y.num, y.key, x.num, x.key) : better(x.num, x.key, y.num, y.key);
                if (swap) {
                    a[i] = y;
                    a[l] = x;
                }
            }
            wave_sync();
        }
    }
}

// Candidates wanted by a wave at once past which they go to the list as a
// batch (appended, then the list sorted and cut back to K) instead of one
// replacement and rescan each.  BATCH: the kernels whose waves see few
// combinations each (order 2); in the others
// the extra code costs the scoring loops registers.
constexpr int kBatchOffer = 8;

template <bool BATCH = false>
EPI_DEV void tk_offer(TopK &t, Cand *list, bool valid, long long num, unsigned long long key, long long gthr) {
    bool want = valid && num >= gthr && (t.n < t.K || better(num, key, t.wn, t.wk));
    unsigned long long mask = __ballot(want);
    // counted once the list is full or a bound exists: the unbounded filling
    // of the lists at the start would only add contention
    if (mask && t.hist && !t.nohist && (t.n == t.K || gthr != (long long)0x8000000000000000ull))
        hist_add(t, want, num);
    const int cnt = __popcll(mask);
    if (BATCH && cnt >= kBatchOffer && tk_sort_size(t.n + cnt) <= t.cap) {
        wave_sync();
        if (want) list[t.n + (int)lane_prefix(mask)] = Cand{num, key};
        const int n2 = t.n + cnt;
        wave_sync();
        if (n2 < t.K) {
            t.n = n2;
            return;
        }
        tk_sort(list, n2);
        // the best K stay, the K-th best is the entry the next better
        // candidate replaces
        t.n = t.K;
        const Cand w = list[t.K - 1];
        t.wn = (long long)rfl64((unsigned long long)w.num);
        t.wk = rfl64(w.key);
        t.wi = t.K - 1;
        return;
    }
    while (mask) {
        const int src = __builtin_ctzll(mask);
        const long long cn = (long long)readlane64((unsigned long long)num, src);
        const unsigned long long ck = readlane64(key, src);
        if (t.n < t.K) {
            if (lane_id() == 0) list[t.n] = Cand{cn, ck};
            t.n++;
            if (t.n == t.K) {
                wave_sync();
                tk_recompute(t, list);
            }
        } else if (better(cn, ck, t.wn, t.wk)) {
            if (lane_id() == 0) list[t.wi] = Cand{cn, ck};
            wave_sync();
            tk_recompute(t, list);
        }
        mask &= mask - 1;
        if (t.n == t.K) mask &= __ballot(want && better(num, key, t.wn, t.wk));
    }
}

// Append the list's entries that can still be in the final best K to the
// task's candidate buffer, then empty the list.
EPI_DEV void tk_flush(TopK &t, const Cand *list, const Task &task) {
    wave_sync();
    const long long g = load_thr(task.thr);
    for (int base = 0; base < t.n; base += kWave) {
        const int i = base + lane_id();
        Cand c{0, 0};
        bool keep = false;
        if (i < t.n) {
            c = list[i];
            keep = c.num >= g;
        }
        unsigned long long m = __ballot(keep);
        unsigned cnt = (unsigned)__popcll(m);
        unsigned off = 0;
        if (lane_id() == 0 && cnt) off = atomicAdd(task.cand_count, cnt);
        off = __builtin_amdgcn_readfirstlane(off);
        unsigned pos = off + lane_prefix(m);
        if (keep && pos < task.cand_cap) task.cand[pos] = c;
    }
    wave_sync();
    t.n = 0;
}

typedef __attribute__((address_space(1))) const long long glong;

// One cell's contribution T(n0) + T(n1) - T(n0 + n1) for counts derived by
// inclusion-exclusion.  The table holds 2N + 1 entries and each class count
// is clamped to N, so no value can index past it.
EPI_DEV long long cell_term(const long long *T, int n0, int n1, unsigned N) {
    const unsigned a = min((unsigned)n0, N);
    const unsigned b = min((unsigned)n1, N);
    glong *g = (glong *)T;
    return g[a] + g[b] - g[a + b];
}

// Same for counts that are popcounts of one class each (n0 + n1 <= N).
EPI_DEV long long cell_term_counted(const long long *T, unsigned n0, unsigned n1) {
    glong *g = (glong *)T;
    return g[n0] + g[n1] - g[n0 + n1];
}

// ---------------------------------------------------------------------------
// Score screening.  A combination can only enter a wave's best-K list if its
// score reaches te (the task's global bound, or the list's current worst once
// the list is full).  The same cell terms summed from the 32-bit table t(n) =
// round(n ln n 2^tq) (the workgroup's LDS copy, reloaded when a chunk of work
// starts a dataset whose table fits) give the score to within one unit of
// 2^-tq per table value read, so combinations whose sum is below the bound
// by more than that skip the exact int64 sum; the exact path is unchanged.
// The sums are taken modulo 2^32: only the result, at most 2^30 in size,
// needs to fit.  Datasets whose table is not in LDS take the exact path for
// every combination.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) const unsigned lu32;
typedef __attribute__((address_space(3))) v4u lv4u;

// The table sits at LDS address 0 (checked when it is loaded), so an entry's
// address is its byte offset with no base to add.  LDS reads cannot fault;
// the counts of valid lanes are always in range.
EPI_DEV unsigned ltab(unsigned byte) { return *(lu32 *)(uintptr_t)byte; }

// The per-combination kernels take the exact table round(n ln n 2^shift),
// n = 0 .. N, at LDS address 0 when it fits: entry n is at byte 8n.
typedef __attribute__((address_space(3))) const long long lli64;
EPI_DEV long long cell_term_lds(unsigned n0, unsigned n1) {
    return *(lli64 *)(uintptr_t)(8u * n0) + *(lli64 *)(uintptr_t)(8u * n1) - *(lli64 *)(uintptr_t)(8u * (n0 + n1));
}

// Stage the genotype-0/1 rows of `nsnp` wave-uniform SNPs (snp_of(r) for row
// pair r) over words [w0, w0 + wn) of class c into the wave's LDS slot:
// slot[(2 * r + g) * cw + w].  One coalesced pass by all lanes; the counting
// loop then reads them with broadcast LDS loads instead of scalar loads.
template <class SnpOf>
EPI_DEV void stage_rows(lv4u *slot, gv4u *gm, long long Mp, int wbase, int w0, int wn, int cw, int nsnp,
                        SnpOf snp_of) {
    wave_sync();
    const int n = 2 * nsnp * wn;
    for (int e = lane_id(); e < n; e += kWave) {
        const int r2 = e / wn;
        const int w = e - r2 * wn;
        const int r = r2 >> 1, g = r2 & 1;
        slot[r2 * cw + w] = gm[((long long)(wbase + w0 + w) * 2 + g) * Mp + snp_of(r)];
    }
    wave_sync();
}

// Screening sum of CELLS cells of plain counts (entry n at byte 4n).
template <int CELLS>
EPI_DEV int screen_sum(const int (&F0)[CELLS], const int (&F1)[CELLS]) {
    unsigned p = 0, q = 0, qh = 0;
    #pragma unroll
    for (int x = 0; x < CELLS; ++x) {
        p = add3(p, ltab(4u * (unsigned)F0[x]), ltab(4u * (unsigned)F1[x]));
        // the subtracted terms in pairs
        if (x & 1) q = add3(q, qh, ltab(4u * (unsigned)(F0[x] + F1[x])));
        else qh = ltab(4u * (unsigned)(F0[x] + F1[x]));
    }
    return (int)(p - q - ((CELLS & 1) ? qh : 0u));
}

// Same for the signed cell form (matrix-core order 3, order 4 by reduced
// cells); with REV the table's mirrored half is in LDS and a B - 4n cell is
// its address there, else it is turned back into 4n.
template <int CELLS, bool REV>
EPI_DEV int screen_sum_signed(const unsigned (&F0)[CELLS], const unsigned (&F1)[CELLS], unsigned B) {
    const unsigned nB = 0u - B;
    unsigned p = 0, q = 0, qh = 0;
    #pragma unroll
    for (int x = 0; x < CELLS; ++x) {
        unsigned a0 = F0[x], a1 = F1[x], s;
        if (odd_twos(x)) {
            if constexpr (REV) {
                s = add3(a0, a1, nB);  // B - 4 (n0 + n1)
            } else {
                a0 = B - a0;
                a1 = B - a1;
                s = a0 + a1;
            }
        } else {
            s = a0 + a1;
        }
        p = add3(p, ltab(a0), ltab(a1));
        // the subtracted terms in pairs
        if (x & 1) q = add3(q, qh, ltab(s));
        else qh = ltab(s);
    }
    return (int)(p - q - qh);
}

// Same for the packed cell form of order 4 by reduced cells (both classes of
// a cell in one register, 4 n(cases) | 4 n(controls) << 16: each half is its
// entry's byte address).
template <int CELLS>
EPI_DEV int screen_sum_packed(const unsigned (&F)[CELLS]) {
    unsigned p = 0, q = 0, qh = 0;
    #pragma unroll
    for (int x = 0; x < CELLS; ++x) {
        const unsigned a0 = F[x] & 0xffffu, a1 = F[x] >> 16;
        p = add3(p, ltab(a0), ltab(a1));
        // the subtracted terms in pairs
        if (x & 1) q = add3(q, qh, ltab(a0 + a1));
        else qh = ltab(a0 + a1);
    }
    return (int)(p - q - ((CELLS & 1) ? qh : 0u));
}

// Smallest screening sum of a combination whose num can reach te, for sums
// of `reads` table values.  Each table value and each exact term is within
// 1/2 of its scaled n ln n, so a sum and the num it screens for differ by at
// most reads units of 2^-tq (tq <= shift); one more unit covers the rounding
// of the scaled bound.
EPI_DEV int screen_bound(long long te, long long score_const, int shift, int tq, int reads) {
    if (te == (long long)0x8000000000000000ull) return (int)0x80000000u;
    const double v = ldexp((double)(te - score_const), tq - shift);
    return (int)floor(v) - reads - 1;
}

EPI_DEV long long entry_bound(const TopK &tk, long long gthr) {
    return tk.n < tk.K ? gthr : (tk.wn > gthr ? tk.wn : gthr);
}

// Pilot pass over an item: the wave's best screening sum S (best over its
// lanes' combinations; INT_MIN: none) becomes one histogram count, or each
// lane's best one count where the task has too few pilot items for K counts
// (pilot_lanes).  S is within `reads` units (2^-tq) of (num - score_const)
// 2^(tq - shift) (each table value within one unit of its n ln n, as in
// screen_bound), so score_const + (S - reads - 1) 2^(shift - tq) is below
// that combination's num; one atomic per wave, and the K-th best of such
// maxima is close to the K-th best of all the item's combinations.
EPI_DEV void pilot_count(TopK &tk, const Task &t, int best, int reads) {
    const bool lanes = t.pilot_lanes != 0;
    if (!lanes) {
        #pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const int o = __shfl_xor(best, off);
            best = o > best ? o : best;
        }
    }
    hist_add(tk, (lanes || lane_id() == 0) && best != (int)0x80000000u,
             t.score_const + (long long)(best - reads - 1) * (1ll << (t.ds.shift - t.ds.tq)));
}

// ---------------------------------------------------------------------------
// kF2 / kF2Emit / kF2Fold: order 2.  A work item is (block of NP SNPs i,
// block of 64 SNPs m > i); lane = m.  Reduced cells (a, d) in {0,1}^2 per
// class, scored (kF2), written to the pair sub-table (kF2Emit), or both
// (kF2Fold: a scan of all orders takes its order-2 results from the pair
// sub-table pass of its higher orders instead of counting the pairs twice).
// ---------------------------------------------------------------------------
template <int NP, bool EMIT, bool LDS, bool SCORE = !EMIT, bool CHECK = false, bool PILOT = false>
EPI_DEV void item_f2(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr, v4u *stage,
                     int stage_cap) {
    static_assert(!PILOT || (LDS && SCORE && !EMIT && !CHECK), "the pilot pass scores from the LDS table");
    const DsView d = t.ds;
    int pilot_best = (int)0x80000000u;  // PILOT: the lane's best screening sum
    const unsigned long long dsc = t.items[local];
    const int ib = uni((int)((dsc >> 20) & 0xfffffu));
    const int mb = uni((int)(dsc & 0xfffffu));
    const int i0 = ib * NP;
    const int lane = lane_id();
    const int m = i0 + 1 + mb * kWave + lane;
    const bool mv = m < d.M;
    const int m_ld = mv ? m : d.Mp - 1;
    int ip[NP];
    #pragma unroll
    for (int p = 0; p < NP; ++p) ip[p] = uni(min(i0 + p, d.M - 1));

    gv4u *gm = (gv4u *)d.masks;
    unsigned acc[NP][2][4];
    #pragma unroll
    for (int p = 0; p < NP; ++p)
        #pragma unroll
        for (int c = 0; c < 2; ++c)
            #pragma unroll
            for (int e = 0; e < 4; ++e) acc[p][c][e] = 0;

    const long long Mp = d.Mp;
    lv4u *slot = (lv4u *)stage;
    const int cw = stage_cap / (2 * NP);  // words (x4) per staged chunk
    #pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int W = d.w4[c];
        long long off = (long long)d.wbase[c] * 2 * Mp;
        v4u m0n = gm[off + m_ld];
        v4u m1n = gm[off + Mp + m_ld];
        for (int w0 = 0; w0 < W; w0 += cw) {
            const int wn = min(cw, W - w0);
            stage_rows(slot, gm, Mp, d.wbase[c], w0, wn, cw, NP, [&](int r) { return min(i0 + r, d.M - 1); });
        for (int w = 0; w < wn; ++w, off += 2 * Mp) {
            const v4u m0 = m0n;
            const v4u m1 = m1n;
            // next iteration's lane rows (the last iteration re-reads its own)
            const long long offn = w0 + w + 1 < W ? off + 2 * Mp : off;
            m0n = gm[offn + m_ld];
            m1n = gm[offn + Mp + m_ld];
            #pragma unroll
            for (int p = 0; p < NP; ++p) {
                const v4u a0 = slot[(2 * p + 0) * cw + w];
                const v4u a1 = slot[(2 * p + 1) * cw + w];
                #pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[p][c][0] = bcnt_acc(a0[q] & m0[q], acc[p][c][0]);
                    acc[p][c][1] = bcnt_acc(a0[q] & m1[q], acc[p][c][1]);
                    acc[p][c][2] = bcnt_acc(a1[q] & m0[q], acc[p][c][2]);
                    acc[p][c][3] = bcnt_acc(a1[q] & m1[q], acc[p][c][3]);
                }
            }
        }
        }
    }

    const v4u *single4 = (const v4u *)d.single;
    const v4u sm = single4[m_ld];
    #pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int i = i0 + p;
        const bool valid = mv && i < m && i <= d.M - 2;
        if constexpr (EMIT) {
            if (valid) {
                v4u *pv = (v4u *)t.pairs;
                const unsigned long long r = t.pair_colex ? colex2(i, m) : lexpair(i, m, d.M);
                if (t.pair_colex) {
                    // order 4 by reduced cells: one word per cell, both classes
                    // (4 n(cases) | 4 n(controls) << 16)
                    pv[r] = v4u{(acc[p][0][0] << 2) | (acc[p][1][0] << 18), (acc[p][0][1] << 2) | (acc[p][1][1] << 18),
                                (acc[p][0][2] << 2) | (acc[p][1][2] << 18), (acc[p][0][3] << 2) | (acc[p][1][3] << 18)};
                } else {
                const int sh = t.cell_shift;
                v4u c0 = v4u{acc[p][0][0] << sh, acc[p][0][1] << sh, acc[p][0][2] << sh, acc[p][0][3] << sh};
                v4u c1 = v4u{acc[p][1][0] << sh, acc[p][1][1] << sh, acc[p][1][2] << sh, acc[p][1][3] << sh};
                if (t.cell_neg) {
                    c0 = t.cell_bias - c0;
                    c1 = t.cell_bias - c1;
                } else {
                    c0 += t.cell_bias;
                    c1 += t.cell_bias;
                }
                pv[2 * r + 0] = c0;
                pv[2 * r + 1] = c1;
                }
            }
        }
        if constexpr (SCORE) {
            const v4u si = single4[ip[p]];
            int F[2][9];
            #pragma unroll
            for (int c = 0; c < 2; ++c) {
                F[c][0] = acc[p][c][0];
                F[c][1] = acc[p][c][1];
                F[c][3] = acc[p][c][2];
                F[c][4] = acc[p][c][3];
                F[c][2] = si[2 * c + 0];
                F[c][5] = si[2 * c + 1];
                F[c][6] = sm[2 * c + 0];
                F[c][7] = sm[2 * c + 1];
                F[c][8] = d.ncls[c];
                mobius2(F[c]);
            }
            if constexpr (PILOT) {
                if (valid) {
                    const int S = screen_sum<9>(F[0], F[1]);
                    pilot_best = S > pilot_best ? S : pilot_best;
                }
                continue;
            }
            if constexpr (CHECK) {
                const int cc[2] = {i, m};
                digest_add(tk, valid, combo_hash<2>(cc), table_sum<9>(F[0], F[1]));
            }
            bool pass = valid;
            if constexpr (LDS) {
                const int sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 27);
                pass = pass && screen_sum<9>(F[0], F[1]) >= sb;
            }
            if (__ballot(pass)) {
                long long num = t.score_const;
                #pragma unroll
                for (int x = 0; x < 9; ++x) num += cell_term(d.tlog, F[0][x], F[1][x], (unsigned)d.N);
                const unsigned long long key = ((unsigned long long)i << 32) | (unsigned long long)m;
                tk_offer<true>(tk, list, pass, num, key, gthr);
            }
        }
    }
    if constexpr (PILOT) pilot_count(tk, t, pilot_best, 27);
}

// ---------------------------------------------------------------------------
// kF3: order 3.  A work item is (j, block of NP SNPs i < j, block of 64 SNPs
// m > j); lane = m.  Reduced cells (a, b, d) in {0,1}^3 per class; every
// other cell comes from the pair sub-table and the single-SNP counts.
// ---------------------------------------------------------------------------
template <int NP, bool LDS, bool CHECK = false>
EPI_DEV void item_f3(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr, v4u *stage,
                     int stage_cap) {
    const DsView d = t.ds;
    const unsigned long long dsc = t.items[local];
    const int j = uni((int)((dsc >> 40) & 0xfffffu));
    const int ib = uni((int)((dsc >> 20) & 0xfffffu));
    const int mb = uni((int)(dsc & 0xfffffu));
    const int i0 = ib * NP;
    const int lane = lane_id();
    const int m = j + 1 + mb * kWave + lane;
    const bool mv = m < d.M;
    const int m_ld = mv ? m : d.Mp - 1;
    int ip[NP];
    #pragma unroll
    for (int p = 0; p < NP; ++p) ip[p] = uni(min(i0 + p, j - 1));

    // sub-table rows the epilogue needs, issued before the counting loop
    const v4u *single4 = (const v4u *)d.single;
    const v4u *pair4 = (const v4u *)t.pairs;
    const v4u sm = single4[m_ld];
    const unsigned long long rjm = mv ? lexpair(j, m, d.M) : 0ull;
    const v4u pjm0 = pair4[2 * rjm], pjm1 = pair4[2 * rjm + 1];
    unsigned long long rim = (mv && i0 < j) ? lexpair(i0, m, d.M) : 0ull;
    v4u pim_n0 = pair4[2 * rim], pim_n1 = pair4[2 * rim + 1];

    gv4u *gm = (gv4u *)d.masks;
    unsigned acc[NP][2][8];
    #pragma unroll
    for (int p = 0; p < NP; ++p)
        #pragma unroll
        for (int c = 0; c < 2; ++c)
            #pragma unroll
            for (int e = 0; e < 8; ++e) acc[p][c][e] = 0;

    const long long Mp = d.Mp;
    lv4u *slot = (lv4u *)stage;
    const int cw = stage_cap / (2 * (NP + 1));  // words (x4) per staged chunk
    #pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int W = d.w4[c];
        long long off = (long long)d.wbase[c] * 2 * Mp;
        v4u m0n = gm[off + m_ld];
        v4u m1n = gm[off + Mp + m_ld];
        for (int w0 = 0; w0 < W; w0 += cw) {
            const int wn = min(cw, W - w0);
            // row pair 0 = j, row pair 1 + p = i0 + p
            stage_rows(slot, gm, Mp, d.wbase[c], w0, wn, cw, NP + 1,
                       [&](int r) { return r == 0 ? j : min(i0 + r - 1, j - 1); });
        for (int w = 0; w < wn; ++w, off += 2 * Mp) {
            const v4u m0 = m0n;
            const v4u m1 = m1n;
            // next iteration's lane rows (the last iteration re-reads its own)
            const long long offn = w0 + w + 1 < W ? off + 2 * Mp : off;
            m0n = gm[offn + m_ld];
            m1n = gm[offn + Mp + m_ld];
            const v4u b0 = slot[0 * cw + w];
            const v4u b1 = slot[1 * cw + w];
            #pragma unroll
            for (int p = 0; p < NP; ++p) {
                const v4u a0 = slot[(2 * p + 2) * cw + w];
                const v4u a1 = slot[(2 * p + 3) * cw + w];
                #pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[p][c][0] = bcnt_acc(a0[q] & b0[q] & m0[q], acc[p][c][0]);
                    acc[p][c][1] = bcnt_acc(a0[q] & b0[q] & m1[q], acc[p][c][1]);
                    acc[p][c][2] = bcnt_acc(a0[q] & b1[q] & m0[q], acc[p][c][2]);
                    acc[p][c][3] = bcnt_acc(a0[q] & b1[q] & m1[q], acc[p][c][3]);
                    acc[p][c][4] = bcnt_acc(a1[q] & b0[q] & m0[q], acc[p][c][4]);
                    acc[p][c][5] = bcnt_acc(a1[q] & b0[q] & m1[q], acc[p][c][5]);
                    acc[p][c][6] = bcnt_acc(a1[q] & b1[q] & m0[q], acc[p][c][6]);
                    acc[p][c][7] = bcnt_acc(a1[q] & b1[q] & m1[q], acc[p][c][7]);
                }
            }
        }
        }
    }

    const v4u sj = single4[j];
    #pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int i = i0 + p;
        const bool valid = mv && i < j;
        const v4u pim0 = pim_n0, pim1 = pim_n1;
        if (p + 1 < NP) {
            // next prefix's pair row, in flight while this one is scored
            rim = (mv && i + 1 < j) ? lexpair(i + 1, m, d.M) : 0ull;
            pim_n0 = pair4[2 * rim];
            pim_n1 = pair4[2 * rim + 1];
        }
        const v4u si = single4[ip[p]];
        const unsigned long long rij = lexpair(ip[p], j, d.M);
        int F[2][27];
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            const v4u pij = pair4[2 * rij + c];
            const v4u pim = c == 0 ? pim0 : pim1;
            const v4u pjm = c == 0 ? pjm0 : pjm1;
            // F[a*9 + b*3 + e]; index 2 on an axis = marginal over that SNP
            #pragma unroll
            for (int a = 0; a < 2; ++a)
                #pragma unroll
                for (int b = 0; b < 2; ++b)
                    #pragma unroll
                    for (int e = 0; e < 2; ++e) F[c][9 * a + 3 * b + e] = acc[p][c][4 * a + 2 * b + e];
            #pragma unroll
            for (int a = 0; a < 2; ++a)
                #pragma unroll
                for (int b = 0; b < 2; ++b) F[c][9 * a + 3 * b + 2] = pij[2 * a + b];
            #pragma unroll
            for (int a = 0; a < 2; ++a)
                #pragma unroll
                for (int e = 0; e < 2; ++e) F[c][9 * a + 6 + e] = pim[2 * a + e];
            #pragma unroll
            for (int b = 0; b < 2; ++b)
                #pragma unroll
                for (int e = 0; e < 2; ++e) F[c][18 + 3 * b + e] = pjm[2 * b + e];
            F[c][9 * 0 + 8] = si[2 * c + 0];
            F[c][9 * 1 + 8] = si[2 * c + 1];
            F[c][18 + 2] = sj[2 * c + 0];
            F[c][18 + 5] = sj[2 * c + 1];
            F[c][24] = sm[2 * c + 0];
            F[c][25] = sm[2 * c + 1];
            F[c][26] = d.ncls[c];
            mobius3(F[c]);
        }
        if constexpr (CHECK) {
            const int cc[3] = {i, j, m};
            digest_add(tk, valid, combo_hash<3>(cc), table_sum<27>(F[0], F[1]));
        }
        bool pass = valid;
        if constexpr (LDS) {
            const int sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 81);
            pass = pass && screen_sum<27>(F[0], F[1]) >= sb;
        }
        if (__ballot(pass)) {
            long long num = t.score_const;
            #pragma unroll
            for (int x = 0; x < 27; ++x) num += cell_term(d.tlog, F[0][x], F[1][x], (unsigned)d.N);
            const unsigned long long key =
                ((unsigned long long)i << 42) | ((unsigned long long)j << 21) | (unsigned long long)m;
            tk_offer(tk, list, pass, num, key, gthr);
        }
    }
}

// ---------------------------------------------------------------------------
// kF3 with np = kNpMfma: order 3 counted by matrix cores.  A work item is
// (j, block of 16 SNPs i, block of 32 SNPs m); every (i, j, m) with i < j < m
// in it is one triplet.  Counts of individuals with genotypes (a, b, d) at
// (i, j, m) are dot products of 0/1 indicator rows, so the reduced cells of a
// class are the products (X_i . x_{j,b})^T X_m over its individuals, one
// matrix-core product per step of individuals, b and d: rows (i, a) are A,
// the rows of genotype b of SNP j mask A, rows (m, d) are B.  The 4-bit float
// operands (v_mfma_scale_f32_32x32x64_f8f6f4, 64 individuals a product) are
// kept as bit planes, 96 individuals per 16-byte entry: one AND (A with its
// mask, in the same instruction) turns a plane into floats, 0.5, 1.0 or 2.0
// for a set bit, and B's exponent scale evens that out.  The scales also put
// the sums at 4 x 2^-149 per count: below 2^24 such a float's bits are the
// integer 4 n, the byte offset of the count's entry in the screening table.
// Where both classes fit one accumulator (q3_pack_fits) the lane halves of
// the controls are scaled further and it holds 4 n(cases) + 2^T n(controls).
// 8-bit integer operands (v_mfma_i32_32x32x32_i8, 32 a step, B 4 for a set
// bit) give the same integers.
//
// Bound (M = 1000, N = 4000, times of the whole scan less 0.2 ms around it):
// the counting alone takes 2.1 ms (1.7 without its loads; its products 1.5),
// the scoring alone 2.0, the LDS time of its 81 table reads a triplet; two
// waves a SIMD overlap 0.8 of that.  Planes instead of whole 4-bit operands
// cut the operand loads from nine to three per 192 individuals, which bound
// the counting before: N = 15001, M = 1001: 15.2 -> 9.2 ms a scan; N = 4000:
// 4.1 -> 3.6.  Three waves a SIMD (168 registers, spills) took 3.9.  In the 32 x 32 result,
// lane l holds column l % 32 (SNP m) and rows 8 (r / 4) + 4 (l / 32) + r % 4
// of its 16 registers r, i.e. both genotypes a of eight SNPs i; the epilogue
// is that of the popcount kernel.
// ---------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// Descriptor word 3 of a raw (untyped, unswizzled) gfx9 buffer.
constexpr int kBufWord3 = 0x00020000;
// Steps in flight per operand stream of the 8-bit kernel.
constexpr int kQDepth = kQStepMultiple;

EPI_DEV v4u qload(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

typedef int v16i __attribute__((ext_vector_type(16)));

// Operand format of the matrix-core order-3 kernel.
//   I8 = false: 4-bit floats, 64 individuals per step, float32 sums;
//   I8 = true:  8-bit integers, 32 individuals per step, int32 sums.
template <bool I8>
struct QFmt;

template <>
struct QFmt<false> {
    typedef v16f acc_t;
    static EPI_DEV const v4u *qa(const DsView &d) { return d.qa; }
    static EPI_DEV const v4u *qb(const DsView &d) { return d.qb; }
    // sb, sa: exponent scales of the operands (E8M0, 127 = 2^0)
    static EPI_DEV acc_t mma(v4u a, v4u b, acc_t c, int sb = 127, int sa = 127) {
        const v8i a8 = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], 0, 0, 0, 0};
        const v8i b8 = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], 0, 0, 0, 0};
        // formats 4 / 4: e2m1 for both operands
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 4, 4, 0, sa, 0, sb);
    }
};

template <>
struct QFmt<true> {
    typedef v16i acc_t;
    static EPI_DEV const v4u *qa(const DsView &d) { return d.qa8; }
    static EPI_DEV const v4u *qb(const DsView &d) { return d.qb8; }
    static EPI_DEV int ks(const DsView &d, int c) { return d.ks8[c]; }
    static EPI_DEV acc_t mma(v4u a, v4u b, acc_t c, int = 127) {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(v4i, a), __builtin_bit_cast(v4i, b), c, 0, 0,
                                                     0);
    }
};

// Exponent scales of a step's three planes: A 2^-74, B this plus 2 - 2 p for
// plane p; e: log2 of a count's weight in the accumulator (2: 4 n).
constexpr int kScaleA = 127 - 74;
EPI_DEV int plane_scale(int e, int p) { return 127 - 75 + e + 2 - 2 * p; }
EPI_DEV unsigned plane_bits(int p) { return 0x11111111u << p; }

// ---------------------------------------------------------------------------
// kF2 with prefix block kNpMfma: order 2 on the matrix cores, the products of
// the order-3 kernel below without the middle SNP's mask.  A work item is
// (block ib of 32 SNPs i, block mb of 32 SNPs m); per step and class four
// products, A0 and A1 (32 rows each: the genotype-0 and -1 rows of the
// item's two 16-SNP blocks of i) times B0 and B1 (the 32 m's genotype-0 and
// -1 rows), 4 n per cell: four operand loads feed four products (two A
// blocks, so that the loads per product are those of the order-3 kernel).
// Lane l holds column m = 32 mb + l % 32 and both genotypes a of eight SNPs
// i of each A block (the layout of item_f3m); the epilogue is item_f2's.
// ---------------------------------------------------------------------------
template <bool LDS, bool PK, bool CHECK = false, bool PILOT = false>
EPI_DEV void item_f2m(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr) {
    static_assert(!PILOT || (LDS && !CHECK), "the pilot pass scores from the LDS table");
    typedef QFmt<false> Q;
    constexpr int NC = PK ? 1 : 2;  // accumulator sets: both classes in one, or one each
    int pilot_best = (int)0x80000000u;  // PILOT: the lane's best screening sum
    const DsView d = t.ds;
    const unsigned long long dsc = t.items[local];
    const int ib = uni((int)((dsc >> 20) & 0xfffffu));
    const int mb = uni((int)(dsc & 0xfffffu));
    const int lane = lane_id(), h = lane >> 5;
    const int m = mb * 32 + (lane & 31);
    const bool mv = m < d.M;
    const int m_ld = mv ? m : d.M - 1;
    const int S3 = d.xs, H0 = d.xh0, T = PK ? q3_pack_shift(d.ncls[0]) : 0;
    const int blk = S3 * 1024;  // bytes of one row block
    const v4u *qa = Q::qa(d), *qb = Q::qb(d);
    // the second 16-SNP block of i; past the operand copy's last block (its
    // SNPs would be M or more) the first block again, its lanes invalid
    const int nib = (d.M + 15) / 16;
    const int ib1 = 2 * ib + 1 < nib ? 2 * ib + 1 : 2 * ib;
    const __amdgpu_buffer_rsrc_t rA0 =
        __builtin_amdgcn_make_buffer_rsrc((void *)(qa + (long long)(2 * ib) * S3 * 64), 0, blk, kBufWord3);
    const __amdgpu_buffer_rsrc_t rA1 =
        __builtin_amdgcn_make_buffer_rsrc((void *)(qa + (long long)ib1 * S3 * 64), 0, blk, kBufWord3);
    const __amdgpu_buffer_rsrc_t rB0 =
        __builtin_amdgcn_make_buffer_rsrc((void *)(qb + (long long)(2 * mb) * S3 * 64), 0, blk, kBufWord3);
    const __amdgpu_buffer_rsrc_t rB1 =
        __builtin_amdgcn_make_buffer_rsrc((void *)(qb + (long long)(2 * mb + 1) * S3 * 64), 0, blk, kBufWord3);
    const int vo = lane * 16;
    typename Q::acc_t acc[NC][2][2];  // [class][A block][genotype of m]
    #pragma unroll
    for (int c = 0; c < NC; ++c)
        #pragma unroll
        for (int a = 0; a < 2; ++a)
            #pragma unroll
            for (int e = 0; e < 2; ++e) acc[c][a][e] = (typename Q::acc_t){};
    // the software pipeline of item_f3m
    struct Ops {
        v4u a0, a1, b0, b1;
    };
    auto load = [&](int s) __attribute__((always_inline)) {
        const int so = min(s, S3 - 1) * 1024;
        return Ops{qload(rA0, vo, so), qload(rA1, vo, so), qload(rB0, vo, so), qload(rB1, vo, so)};
    };
    auto mul = [&](const Ops &o, int e, auto cls) __attribute__((always_inline)) {
        constexpr int c = cls.value;
        #pragma unroll
        for (int p = 0; p < 3; ++p) {
            const unsigned pb = plane_bits(p);
            const int sb = plane_scale(e, p);
            const v4u a0 = o.a0 & pb, a1 = o.a1 & pb, b0 = o.b0 & pb, b1 = o.b1 & pb;
            acc[c][0][0] = Q::mma(a0, b0, acc[c][0][0], sb, kScaleA);
            acc[c][0][1] = Q::mma(a0, b1, acc[c][0][1], sb, kScaleA);
            acc[c][1][0] = Q::mma(a1, b0, acc[c][1][0], sb, kScaleA);
            acc[c][1][1] = Q::mma(a1, b1, acc[c][1][1], sb, kScaleA);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    Ops x = load(0);
    auto run = [&](int from, int to, auto cls) __attribute__((always_inline)) {
        #pragma unroll 1
        for (int s = from; s < to; s += 2) {
            const Ops y = load(s + 1);
            mul(x, PK && 2 * s + h >= H0 ? T : 2, cls);
            __builtin_amdgcn_sched_barrier(0);
            x = load(s + 2);
            if (s + 1 < to) mul(y, PK && 2 * s + 2 + h >= H0 ? T : 2, cls);
        }
    };
    if constexpr (PK) {
        run(0, S3, std::integral_constant<int, 0>{});
    } else {
        run(0, H0 / 2, std::integral_constant<int, 0>{});  // an even number of steps
        run(H0 / 2, S3, std::integral_constant<int, NC - 1>{});
    }
    const v4u *single4 = (const v4u *)d.single;
    const v4u sm = single4[m_ld];
    // the eight pairs of a lane in each A block (a function per block, so
    // that each loop over them unrolls and every accumulator index is a
    // constant)
    auto score_block = [&](const typename Q::acc_t (&c0)[2], const typename Q::acc_t (&c1)[2], int ab)
                           __attribute__((always_inline)) {
        const unsigned m0 = (1u << T) - 1u;
        const int i_base = ib * 32 + 16 * ab + 2 * h;
        #pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i_base + 4 * (u >> 1) + (u & 1);
            const int r0 = 4 * (u >> 1) + 2 * (u & 1);
            const bool valid = mv && i < m;
            const v4u si = single4[min(i, d.M - 1)];
            int F[2][9];
            #pragma unroll
            for (int c = 0; c < 2; ++c) {
                #pragma unroll
                for (int a = 0; a < 2; ++a)
                    #pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const unsigned w = __float_as_uint((c == 0 ? c0 : c1)[e][r0 + a]);
                        F[c][3 * a + e] = (int)(PK ? (c == 0 ? (w & m0) >> kQScaleShift : w >> T) : w >> kQScaleShift);
                    }
                F[c][2] = si[2 * c + 0];
                F[c][5] = si[2 * c + 1];
                F[c][6] = sm[2 * c + 0];
                F[c][7] = sm[2 * c + 1];
                F[c][8] = d.ncls[c];
                mobius2(F[c]);
            }
            if constexpr (PILOT) {
                if (valid) {
                    const int S = screen_sum<9>(F[0], F[1]);
                    pilot_best = S > pilot_best ? S : pilot_best;
                }
                continue;
            }
            if constexpr (CHECK) {
                const int cc[2] = {i, m};
                digest_add(tk, valid, combo_hash<2>(cc), table_sum<9>(F[0], F[1]));
            }
            bool pass = valid;
            if constexpr (LDS) {
                const int sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 27);
                pass = pass && screen_sum<9>(F[0], F[1]) >= sb;
            }
            if (__ballot(pass)) {
                long long num = t.score_const;
                #pragma unroll
                for (int x = 0; x < 9; ++x) num += cell_term(d.tlog, F[0][x], F[1][x], (unsigned)d.N);
                const unsigned long long key = ((unsigned long long)i << 32) | (unsigned long long)m;
                tk_offer<true>(tk, list, pass, num, key, gthr);
            }
        }
    };
    score_block(acc[0][0], acc[NC - 1][0], 0);
    score_block(acc[0][1], acc[NC - 1][1], 1);
    if constexpr (PILOT) pilot_count(tk, t, pilot_best, 27);
}

// PILOT: the histogram-only pass over an item (needs the screening table in
// LDS): lower bounds of the scores are counted, nothing is offered.
// PK: one accumulator per tile for both classes, where q3_pack_fits; always so
// with two middle SNPs.  (N = 4000: 3.6 ms against 3.7 with one per class,
// whose steps hold one class each.)
template <bool LDS, bool REV, bool I8, bool PK, bool EMIT = false, bool CHECK = false, int NJ = 1, bool PILOT = false>
EPI_DEV void item_f3m(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr, v4u *stage) {
    static_assert(NJ == 1 || (NJ == 2 && PK && !EMIT), "two middle SNPs per item: one accumulator for both classes");
    static_assert(!(PK && I8), "the 8-bit kernel keeps the classes apart");
    typedef QFmt<I8> Q;
    constexpr int NC = PK ? 1 : 2;
    const int T = PK ? q3_pack_shift(t.ds.ncls[0]) : 0;
    const DsView d = t.ds;
    const unsigned long long dsc = t.items[local];
    const int j = uni((int)((dsc >> 40) & 0xfffffu));
    const int ib = uni((int)((dsc >> 20) & 0xfffffu));
    const int mb = uni((int)(dsc & 0xfffffu));
    const int lane = lane_id(), h = lane >> 5;
    const int m = mb * 32 + (lane & 31);
    // The item's middle SNPs jv[0] = j and (NJ = 2) jv[1] = j + 1, which
    // share the i and m blocks and so every operand load of the counting
    // loop (jv[1] may be M - 1: no valid triplet).
    int jv[NJ];
    bool mv[NJ];
    #pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        jv[jj] = j + jj;
        mv[jj] = m > jv[jj] && m < d.M;
    }

    // Sub-table rows the epilogue needs, issued before the counting loop; all
    // counts below are 4 n, in the signed form of the epilogue (the pair
    // sub-table and the second half of `single` are written that way, the
    // class sizes are put in it here).  They are read through buffer
    // descriptors, at 32-bit offsets from the block's first row: a lane with
    // no valid triplet reads another entry, or zeros past the table's end,
    // and is left out by `valid`.
    const unsigned B = q3_bias(d.N);
    const unsigned nall[2] = {13u * B - ((unsigned)d.ncls[0] << kQScaleShift),
                              13u * B - ((unsigned)d.ncls[1] << kQScaleShift)};
    const __amdgpu_buffer_rsrc_t rS =
        __builtin_amdgcn_make_buffer_rsrc((void *)((const v4u *)d.single + d.Mp), 0, d.Mp * 16, kBufWord3);
    const unsigned long long pair_bytes = EMIT ? 0ull : pair_row(d.M - 1, d.M) * 32ull;
    auto pair_rows = [&](int first) {  // rows (first, first + 1) on
        const unsigned long long at = pair_row(min(first, d.M - 1), d.M) * 32ull, left = pair_bytes - at;
        return __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)t.pairs + at), 0,
                                                 (int)(left < 0x7fffffffull ? left : 0x7fffffffull), kBufWord3);
    };
    v4u sm, sj[NJ], pjm0[NJ], pjm1[NJ];
    if constexpr (!EMIT) {
        sm = qload(rS, m * 16, 0);
        #pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
            sj[jj] = ((cv4u *)d.single)[d.Mp + jv[jj]];  // uniform: a scalar load
            const __amdgpu_buffer_rsrc_t rj = pair_rows(jv[jj]);
            const int vj = (m - jv[jj] - 1) * 32;
            pjm0[jj] = qload(rj, vj, 0);
            pjm1[jj] = qload(rj, vj + 16, 0);
        }
    }

    // operands through buffer descriptors (scalar registers): a lane adds
    // its own constant byte offset and a step adds a scalar one, so a step
    // costs no vector address arithmetic
    const int KS = I8 ? d.ks8[0] + d.ks8[1] : d.xs;
    const int blk = KS * 1024;  // bytes of one row block
    const v4u *qa = Q::qa(d), *qb = Q::qb(d);
    const __amdgpu_buffer_rsrc_t rA =
        __builtin_amdgcn_make_buffer_rsrc((void *)(qa + (long long)ib * KS * 64), 0, blk, kBufWord3);
    __amdgpu_buffer_rsrc_t rJ[NJ];
    #pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
        rJ[jj] = __builtin_amdgcn_make_buffer_rsrc((void *)(qa + (long long)(jv[jj] >> 4) * KS * 64), 0, blk,
                                                   kBufWord3);
    const __amdgpu_buffer_rsrc_t rB0 =
        __builtin_amdgcn_make_buffer_rsrc((void *)(qb + (long long)(2 * mb) * KS * 64), 0, blk, kBufWord3);
    const __amdgpu_buffer_rsrc_t rB1 =
        __builtin_amdgcn_make_buffer_rsrc((void *)(qb + (long long)(2 * mb + 1) * KS * 64), 0, blk, kBufWord3);
    const int vo = lane * 16;
    typename Q::acc_t acc[NJ][NC][2][2];
    #pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
        #pragma unroll
        for (int c = 0; c < NC; ++c)
            #pragma unroll
            for (int b = 0; b < 2; ++b)
                #pragma unroll
                for (int e = 0; e < 2; ++e) acc[jj][c][b][e] = (typename Q::acc_t){};
    // The two mask rows of a middle SNP are the same for every lane of a half
    // wave: they are staged once per segment of kSeg steps in the wave's LDS
    // slot (entry jj 4 kSeg + 4 step + 2 h + b) and read back with broadcast
    // loads.
    constexpr int kSeg = I8 ? kQ8StageSteps : kQStageSteps;
    lv4u *slot = (lv4u *)stage;
    // mask rows of the segment [base, base + kSeg) of the stream
    auto stage_masks = [&](int base) __attribute__((always_inline)) {
        const int n = min(kSeg, KS - base);
        wave_sync();  // the slot's previous rows have been read
        // all loads issued at once, no branch between them (entries past the
        // segment repeat its last step's; the slot has room for them)
        #pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
            #pragma unroll
            for (int e0 = 0; e0 < 4 * kSeg; e0 += kWave) {
                const int e = min(e0 + lane, 4 * n - 1);
                const int vje = (((e >> 2) * 64) + 32 * ((e >> 1) & 1) + 2 * (jv[jj] & 15) + (e & 1)) * 16;
                slot[jj * 4 * kSeg + e0 + lane] = qload(rJ[jj], vje, base * 1024);
            }
        wave_sync();
    };
    int seg = 0;
    if constexpr (!I8) {
        // Both classes' steps form one stream; a step's operands are loaded
        // while the one before is multiplied (12 products of 32 cycles a
        // middle SNP against a load from L2, with another wave or two on the
        // SIMD), in two register sets taken in turn.
        const int H0 = d.xh0;
        struct Ops {
            v4u a, b0, b1;
        };
        auto load = [&](int s) __attribute__((always_inline)) {
            const int so = min(s, KS - 1) * 1024;
            return Ops{qload(rA, vo, so), qload(rB0, vo, so), qload(rB1, vo, so)};
        };
        auto mul = [&](int s, const Ops &o, int e, auto cls) __attribute__((always_inline)) {
            constexpr int c = cls.value;
            v4u J[NJ][2];
            #pragma unroll
            for (int jj = 0; jj < NJ; ++jj) {
                const int js = jj * 4 * kSeg + 4 * (s - seg) + 2 * h;
                J[jj][0] = slot[js];
                J[jj][1] = slot[js + 1];
            }
            #pragma unroll
            for (int p = 0; p < 3; ++p) {
                const unsigned pb = plane_bits(p);
                const int sb = plane_scale(e, p);
                const v4u b0 = o.b0 & pb, b1 = o.b1 & pb;
                #pragma unroll
                for (int jj = 0; jj < NJ; ++jj) {
                    const v4u A0 = o.a & J[jj][0] & pb, A1 = o.a & J[jj][1] & pb;
                    acc[jj][c][0][0] = Q::mma(A0, b0, acc[jj][c][0][0], sb, kScaleA);
                    acc[jj][c][0][1] = Q::mma(A0, b1, acc[jj][c][0][1], sb, kScaleA);
                    acc[jj][c][1][0] = Q::mma(A1, b0, acc[jj][c][1][0], sb, kScaleA);
                    acc[jj][c][1][1] = Q::mma(A1, b1, acc[jj][c][1][1], sb, kScaleA);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        Ops x = load(0);
        stage_masks(0);
        auto run = [&](int from, int to, auto cls) __attribute__((always_inline)) {
            #pragma unroll 1
            for (int s = from; s < to; s += 2) {
                if (s >= seg + kSeg) {
                    seg += kSeg;
                    stage_masks(seg);
                }
                const Ops y = load(s + 1);
                mul(s, x, PK && 2 * s + h >= H0 ? T : 2, cls);
                __builtin_amdgcn_sched_barrier(0);
                x = load(s + 2);
                if (s + 1 < to) mul(s + 1, y, PK && 2 * s + 2 + h >= H0 ? T : 2, cls);
            }
        };
        if constexpr (PK) {
            run(0, KS, std::integral_constant<int, 0>{});
        } else {
            run(0, H0 / 2, std::integral_constant<int, 0>{});  // an even number of steps
            run(H0 / 2, KS, std::integral_constant<int, NC - 1>{});
        }
    } else {
    // Software pipeline: the operands of kQDepth steps are in flight while a
    // step is multiplied (a step's products take far less time than a load
    // from L2).  The steps of both classes form one stream, class 0's first
    // as in the operand copies (each class has a multiple of kQDepth steps,
    // zero-padded), so the pipeline runs on across the class boundary and an
    // item waits for operands only at its start.  Scheduling barriers keep
    // the loads in step order, each step's refills right after its products:
    // left alone, the scheduler sinks all refills to the end of the unrolled
    // block, and the loop then waits for every load in flight at its top.
    const int ks0 = d.ks8[0];
    v4u bA[kQDepth], bB0[kQDepth], bB1[kQDepth];
    #pragma unroll
    for (int u = 0; u < kQDepth; ++u) {
        const int so = min(u, KS - 1) * 1024;
        bA[u] = qload(rA, vo, so);
        bB0[u] = qload(rB0, vo, so);
        bB1[u] = qload(rB1, vo, so);
        __builtin_amdgcn_sched_barrier(0);
    }
    stage_masks(0);
    #pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int c0 = c == 0 ? 0 : ks0;
        const int cn = d.ks8[c];
        #pragma unroll 1
        for (int k = 0; k < cn; k += kQDepth) {
            const int g = c0 + k;  // the group's first step in the stream
            if (g >= seg + kSeg) {
                seg += kSeg;
                stage_masks(seg);
            }
            #pragma unroll
            for (int u = 0; u < kQDepth; ++u) {
                const int js = 4 * (g - seg + u) + 2 * h;
                const v4u J0 = slot[js], J1 = slot[js + 1];
                const v4u A0 = bA[u] & J0, A1 = bA[u] & J1;
                acc[0][c][0][0] = Q::mma(A0, bB0[u], acc[0][c][0][0]);
                acc[0][c][0][1] = Q::mma(A0, bB1[u], acc[0][c][0][1]);
                acc[0][c][1][0] = Q::mma(A1, bB0[u], acc[0][c][1][0]);
                acc[0][c][1][1] = Q::mma(A1, bB1[u], acc[0][c][1][1]);
                // refill with the step kQDepth ahead in the stream (the last
                // steps re-read the stream's last step)
                const int so = min(g + u + kQDepth, KS - 1) * 1024;
                bA[u] = qload(rA, vo, so);
                bB0[u] = qload(rB0, vo, so);
                bB1[u] = qload(rB1, vo, so);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    }
    wave_sync();  // the slot's rows have been read

    // 4 n of a cell in class c (register r of tile (b, e) of middle SNP jj)
    const unsigned m0 = (1u << T) - 1u;
    auto count4 = [&](int jj, int c, int b, int e, int r) __attribute__((always_inline)) {
        if constexpr (I8) {
            return (unsigned)acc[jj][c][b][e][r];
        } else {
            const unsigned w = __float_as_uint(acc[jj][PK ? 0 : c][b][e][r]);
            return !PK ? w : (c == 0 ? w & m0 : (w >> (T - 2)) & ~3u);
        }
    };

    if constexpr (EMIT) {
        // triplet sub-table: the 8 cells 4a + 2b + d of the lane's eight
        // triplets at their colex ranks, both classes of a cell in one word
        // (the sums are 4n: 4 n(cases) | 4 n(controls) << 16, the packed form
        // of order 4 by reduced cells)
        gv4u *tv = (gv4u *)t.triples;
        #pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = ib * 16 + 2 * h + 4 * (u >> 1) + (u & 1);
            const int r0 = 4 * (u >> 1) + 2 * (u & 1);
            if (mv[0] && i < j) {
                v4u *dst = (v4u *)(tv + 2 * colex3(i, j, m));
                #pragma unroll
                for (int a = 0; a < 2; ++a) {
                    auto pk = [&](int b, int e) {
                        return count4(0, 0, b, e, r0 + a) | (count4(0, 1, b, e, r0 + a) << 16);
                    };
                    dst[a] = v4u{pk(0, 0), pk(0, 1), pk(1, 0), pk(1, 1)};
                }
            }
        }
        return;
    }

    // Cells F[c][9a + 3b + e] (digit 2: genotype 2, by inclusion-exclusion) in
    // the signed form: a cell with an odd number of digits 2 is held as B -
    // 4n, the others as 4n (B = q3_bias(N)).  Each inclusion-exclusion step is
    // then one three-input add, and both forms are byte addresses of the LDS table,
    // which holds t(n) at 4n and at B - 4n.  The marginal inputs come in the
    // forms that make the steps come out so: pair cells B - 4n (as the pair
    // pass writes them), single-SNP cells 4n - 4B, the class size 13B - 4n.
    // The lane's eight SNPs i: i_local = 4 (u / 2) + 2 h + u % 2, genotype a
    // in register 4 (u / 2) + 2 (u % 2) + a.
    const int i_base = ib * 16 + 2 * h;
    int pilot_best = (int)0x80000000u;  // PILOT: the lane's best screening sum
    int sb = 0;
    if constexpr (LDS) sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 81);
    // Byte offset of pair (i, m) from the block's first row: the entries of
    // SNP i0 + x start f(x) = x (2 A - x - 1) / 2 - x pairs on, A = M - i0;
    // for the upper lane half x is 2 more, f(x + 2) - f(x) = 2 A - 2 x - 5.
    const int i0 = ib * 16, A = d.M - i0;
    const __amdgpu_buffer_rsrc_t rI = pair_rows(i0);
    const int h64 = h * 64;
    auto f32 = [&](int x) { return 32 * (x * (2 * A - x - 1) / 2 - x); };
    #pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int jm = jv[jj];
        // the (j, m) table completed (genotype 2 of j, m, both): the marginals
        // over i, in the form the last inclusion-exclusion step takes
        // (B - 4n with an even number of digits 2, else 4n - 2B)
        unsigned P2[2][9];
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            const v4u p = c == 0 ? pjm0[jj] : pjm1[jj];
            P2[c][0] = p[0];
            P2[c][1] = p[1];
            P2[c][3] = p[2];
            P2[c][4] = p[3];
            P2[c][2] = sj[jj][2 * c] + p[0] + p[1];
            P2[c][5] = sj[jj][2 * c + 1] + p[2] + p[3];
            P2[c][6] = sm[2 * c] + p[0] + p[2];
            P2[c][7] = sm[2 * c + 1] + p[1] + p[3];
            P2[c][8] = nall[c] + sm[2 * c] + sm[2 * c + 1] + P2[c][2] + P2[c][5];
        }
        const int to_j = (jm - m) * 32;  // from pair (i, m) to pair (i, j)
        int off_n = (m - i0 - 1) * 32 + h * 32 * (2 * A - 5);
        v4u pim_n0 = qload(rI, off_n, 0), pim_n1 = qload(rI, off_n + 16, 0);
        #pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i_base + 4 * (u >> 1) + (u & 1);
            const bool valid = mv[jj] && i < jm;
            const v4u pim0 = pim_n0, pim1 = pim_n1;
            const v4u pij0 = qload(rI, off_n + to_j, 0), pij1 = qload(rI, off_n + to_j + 16, 0);
            const v4u si = qload(rS, i * 16, 0);
            if (u + 1 < 8) {
                // next SNP's pair row, in flight while this one is scored
                const int x = 4 * (u >> 1) + (u & 1), xn = 4 * ((u + 1) >> 1) + ((u + 1) & 1);
                off_n += (f32(xn) - f32(x)) - (xn - x) * h64;
                pim_n0 = qload(rI, off_n, 0);
                pim_n1 = qload(rI, off_n + 16, 0);
            }
            const int r0 = 4 * (u >> 1) + 2 * (u & 1);
            unsigned F[2][27];
            #pragma unroll
            for (int c = 0; c < 2; ++c) {
                const v4u pij = c == 0 ? pij0 : pij1;
                const v4u pim = c == 0 ? pim0 : pim1;
                #pragma unroll
                for (int a = 0; a < 2; ++a) {
                    unsigned *G = F[c] + 9 * a;
                    #pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        #pragma unroll
                        for (int e = 0; e < 2; ++e) G[3 * b + e] = count4(jj, c, b, e, r0 + a);
                        G[3 * b + 2] = pij[2 * a + b] + G[3 * b] + G[3 * b + 1];
                    }
                    #pragma unroll
                    for (int e = 0; e < 2; ++e) G[6 + e] = pim[2 * a + e] + G[e] + G[3 + e];
                    G[8] = si[2 * c + a] + pij[2 * a] + pij[2 * a + 1] + G[6] + G[7];
                }
                #pragma unroll
                for (int r = 0; r < 9; ++r) F[c][18 + r] = P2[c][r] + F[c][r] + F[c][9 + r];
            }
            if constexpr (PILOT) {
                static_assert(LDS && !CHECK && !EMIT, "the pilot pass reads the screening table from LDS");
                if (valid) {
                    const int S = screen_sum_signed<27, REV>(F[0], F[1], B);
                    pilot_best = S > pilot_best ? S : pilot_best;
                }
                continue;
            }
            if constexpr (CHECK) {
                unsigned long long sum = 0;
                #pragma unroll
                for (int x = 0; x < 27; ++x) {
                    const unsigned n0 = (odd_twos(x) ? B - F[0][x] : F[0][x]) >> kQScaleShift;
                    const unsigned n1 = (odd_twos(x) ? B - F[1][x] : F[1][x]) >> kQScaleShift;
                    sum += (unsigned long long)n0 * cell_weight(0, x) + (unsigned long long)n1 * cell_weight(1, x);
                }
                const int cc[3] = {i, jm, m};
                digest_add(tk, valid, combo_hash<3>(cc), sum);
            }
            bool pass = valid;
            if constexpr (LDS) pass = pass && screen_sum_signed<27, REV>(F[0], F[1], B) >= sb;
            if (__ballot(pass)) {
                long long num = t.score_const;
                #pragma unroll
                for (int x = 0; x < 27; ++x) {
                    const unsigned n0 = (odd_twos(x) ? B - F[0][x] : F[0][x]) >> kQScaleShift;
                    const unsigned n1 = (odd_twos(x) ? B - F[1][x] : F[1][x]) >> kQScaleShift;
                    num += cell_term(d.tlog, (int)n0, (int)n1, (unsigned)d.N);
                }
                const unsigned long long key =
                    ((unsigned long long)i << 42) | ((unsigned long long)jm << 21) | (unsigned long long)m;
                tk_offer(tk, list, pass, num, key, gthr);
                if constexpr (LDS) sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 81);
            }
        }
    }
    if constexpr (PILOT) pilot_count(tk, t, pilot_best, 81);
}

// ---------------------------------------------------------------------------
// kX: orders 5-8, all 3^K cells on the matrix cores.  The table of a
// combination is the product of the cell rows of its first xa(K) SNPs (A) and
// those of its last xb(K) (B): cell (x_A, x_B) = sum over the individuals of
// row x_A times row x_B, so no sub-table and no inclusion-exclusion.  A unit
// is 3 x 3 tiles of 32 x 32 products (27 cell rows and 5 spare ones a side):
// 27 combinations of order 5, 9 of order 6, 3 of order 7, one of order 8.
//
// A row is the AND of two entries of the dataset's cell rows (pairs and single
// SNPs), loaded at 96 individuals per lane entry, three bit planes that one
// AND with a constant each turns into a step of 4-bit floats: 0.5, 1.0 or 2.0
// for a set bit, evened out by the product's exponent scale.  The scales also
// put the sums at 2^-149 per unit, so that an accumulator's bits are the
// integer itself, and pack the classes into it (x_pack_fits).
//
// Per 192 individuals: 27 products (864 matrix-core cycles), mostly 7 or 8
// loads and 72 vector ANDs.  All cells of a combination are spread over the
// wave, so its screening sum is one wave reduction and its handling uniform.
// Bound by the sum of the products and of the scoring's vector and LDS work:
// two waves a SIMD overlap them only in part (products without the scoring
// 3.0 ms, scoring without the products 1.5, together 3.9 at order 8, M = 23,
// N = 2048, against 18.8 ms for the popcount kernel; order 5, M = 60,
// N = 2000: 1.8 ms against 6.7).
// ---------------------------------------------------------------------------
constexpr int pow3c(int k) { return k <= 0 ? 1 : 3 * pow3c(k - 1); }

// Colex unranking without the binomial table (K <= 4, rank < 2^31): index t
// from the t-th root of t! rank, corrected by its falling factorial.
template <int K>
EPI_DEV void colex_unrank_root(unsigned rank, int (&c)[K]) {
    #pragma unroll
    for (int t = K; t >= 1; --t) {
        if (t == 1) {
            c[0] = (int)rank;
            break;
        }
        const unsigned fact = t == 2 ? 2u : (t == 3 ? 6u : 24u);
        const unsigned long long want = (unsigned long long)rank * fact;
        auto fall = [&](int x) {  // x (x - 1) ... (x - t + 1)
            unsigned long long v = (unsigned long long)x * (unsigned)(x - 1);
            if (t > 2) v *= (unsigned)(x - 2);
            if (t > 3) v *= (unsigned)(x - 3);
            return v;
        };
        const float w = (float)want;
        int x = t == 2 ? (int)sqrtf(w) : (t == 3 ? (int)cbrtf(w) + 1 : (int)sqrtf(sqrtf(w)) + 1);
        x = max(x, t - 1);
        while (x > t - 1 && fall(x) > want) --x;
        while (fall(x + 1) <= want) ++x;
        c[t - 1] = x;
        rank = (unsigned)((want - fall(x)) / fact);
    }
}

// Inclusive scan over the wave in vector registers (row shifts and broadcasts).
EPI_DEV unsigned wave_scan_dpp(unsigned v) {
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}
EPI_DEV unsigned rl(unsigned v, int lane) { return (unsigned)__builtin_amdgcn_readlane((int)v, lane); }

EPI_DEV long long wave_sum64(long long v) {
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += (long long)__shfl_xor((unsigned long long)v, off);
    return (long long)rfl64((unsigned long long)v);
}

// The operand rows of one side of a unit: a lane's row c < 27 of tile t is the
// AND of an entry of its own tile (the SNP that runs fastest through the
// subsets, or the first pair of a quadruple) and one that the tiles mostly
// share (the rest of the subset); a pair's row is one entry.  An entry is at
// a lane constant + a scalar + step x stride; rows past the 27th repeat
// others (their products are left out of every sum).
template <int S, bool FIRST>  // FIRST: the subset's first SNP runs fastest (colex), else its last
struct XSide {
    static constexpr int kOwn = S == 3 ? kXSingle : kXPair;
    int vo[S == 2 ? 3 : 1], vs;  // lane constants
    int so[3], ss[3];            // scalars
    unsigned single0, pair0, S3;
    EPI_DEV int pair_at(int x, int y) const {
        return (int)(pair0 + ((unsigned)y * (unsigned)(y - 1) / 2u + (unsigned)x) * S3 * kXPair);
    }
    EPI_DEV void init(int c, int h, unsigned steps, int M) {
        S3 = steps;
        pair0 = (unsigned)M * S3 * kXSingle;
        c = c < 27 ? c : c - 9;
        if constexpr (S == 3 && FIRST) {
            vo[0] = (h * 4 + c / 9) * 16;
            vs = (h * 9 + c % 9) * 16;
        } else if constexpr (S == 3) {
            vo[0] = (h * 4 + c % 3) * 16;
            vs = (h * 9 + c / 3) * 16;
        } else {
            vo[0] = (h * 9 + (S == 4 ? c / 9 : c % 9)) * 16;
            vs = (h * 9 + c % 9) * 16;
        }
    }
    // tile t's subset: e wave-uniform (S = 2: the lane's own pair of the tile)
    EPI_DEV void set(int t, const int (&e)[S]) {
        if constexpr (S == 2) {
            if (t > 0) vo[t] = vo[0];
            so[t] = 0;
            ss[t] = pair_at(e[0], e[1]);  // added to the lane constant by finish()
        } else if constexpr (S == 3) {
            so[t] = (int)((unsigned)(FIRST ? e[0] : e[2]) * S3 * kXSingle);
            ss[t] = FIRST ? pair_at(e[1], e[2]) : pair_at(e[0], e[1]);
        } else {
            so[t] = pair_at(e[0], e[1]) + 3 * t * 16;
            ss[t] = pair_at(e[2], e[3]);
        }
    }
    EPI_DEV void finish() {
        if constexpr (S == 2)
            #pragma unroll
            for (int t = 0; t < 3; ++t) vo[t] += ss[t];
    }
    // whether the three tiles share their second entry
    EPI_DEV bool same() const { return S != 3 || (ss[1] == ss[0] && ss[2] == ss[0]); }
    template <int NS>  // second entries to load: none (pairs), 1 (shared) or 3
    EPI_DEV void load(__amdgpu_buffer_rsrc_t r, int step, v4u (&f1)[3], v4u (&f2)[3]) const {
        #pragma unroll
        for (int t = 0; t < NS; ++t) f2[t] = qload(r, vs, ss[t] + step * kXPair);
        #pragma unroll
        for (int t = 0; t < 3; ++t) f1[t] = qload(r, vo[S == 2 ? t : 0], so[t] + step * kOwn);
    }
};

// A unit's nine tiles over all steps; NA, NB: second entries per side.  The
// entries of the next step are in flight while one is multiplied: two sets of
// them where they fit the registers (each plane's operand is one three-input
// AND of them), else their two-input AND is formed first and the next step's
// are loaded behind it.
template <int NA, int NB, class SA, class SB>
EPI_DEV void x_count(const SA &sa, const SB &sb, __amdgpu_buffer_rsrc_t rx, int H0, int S3, int sh, int T, int h,
                     v16f (&acc)[3][3]) {
    #pragma unroll
    for (int ta = 0; ta < 3; ++ta)
        #pragma unroll
        for (int tb = 0; tb < 3; ++tb) acc[ta][tb] = (v16f){};
    // planes p of a step: products 4^(p - 1), evened out by B's exponent
    // scale, which also holds the lane half's class
    auto step = [&](int s, const v4u (&a1)[3], const v4u (&a2)[3], const v4u (&b1)[3], const v4u (&b2)[3], auto two)
                    __attribute__((always_inline)) {
        const int ex = 127 - 75 + (2 * s + h < H0 ? sh : T);
        #pragma unroll
        for (int p = 0; p < 3; ++p) {
            __builtin_amdgcn_sched_barrier(0);
            const unsigned plane = 0x11111111u << p;
            v4u b[3];
            #pragma unroll
            for (int x = 0; x < 3; ++x) {
                if constexpr (two.value && NB > 0) b[x] = b1[x] & b2[NB == 3 ? x : 0] & plane;
                else b[x] = b1[x] & plane;
            }
            #pragma unroll
            for (int ta = 0; ta < 3; ++ta) {
                v4u a;
                if constexpr (two.value && NA > 0) a = a1[ta] & a2[NA == 3 ? ta : 0] & plane;
                else a = a1[ta] & plane;
                #pragma unroll
                for (int tb = 0; tb < 3; ++tb)
                    acc[ta][tb] = QFmt<false>::mma(a, b[tb], acc[ta][tb], ex + 2 - 2 * p, 127 - 74);
            }
        }
    };
    v4u a1[3], a2[3], b1[3], b2[3];
    sa.template load<NA>(rx, 0, a1, a2);
    sb.template load<NB>(rx, 0, b1, b2);
    if constexpr (NA + NB <= 2) {
        v4u c1[3], c2[3], e1[3], e2[3];
        #pragma unroll 1
        for (int s = 0; s < S3; s += 2) {
            const int s1 = min(s + 1, S3 - 1), s2 = min(s + 2, S3 - 1);
            sa.template load<NA>(rx, s1, c1, c2);
            sb.template load<NB>(rx, s1, e1, e2);
            step(s, a1, a2, b1, b2, std::true_type{});
            __builtin_amdgcn_sched_barrier(0);
            sa.template load<NA>(rx, s2, a1, a2);
            sb.template load<NB>(rx, s2, b1, b2);
            if (s + 1 < S3) step(s + 1, c1, c2, e1, e2, std::true_type{});
        }
    } else {
        #pragma unroll 1
        for (int s = 0; s < S3; ++s) {
            v4u ra[3], rb[3];
            #pragma unroll
            for (int t = 0; t < 3; ++t) {
                ra[t] = NA > 0 ? a1[t] & a2[NA == 3 ? t : 0] : a1[t];
                rb[t] = NB > 0 ? b1[t] & b2[NB == 3 ? t : 0] : b1[t];
            }
            const int sn = min(s + 1, S3 - 1);
            sa.template load<NA>(rx, sn, a1, a2);
            sb.template load<NB>(rx, sn, b1, b2);
            step(s, ra, ra, rb, rb, std::false_type{});
        }
    }
}

template <int K, bool CHECK = false, bool PILOT = false>
EPI_DEV void item_x(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr) {
    constexpr int KA = xa(K), KB = xb(K), NA = xna(K), NB = xnb(K), READS = 3 * pow3c(K);
    const DsView d = t.ds;
    const int M = d.M, lane = lane_id(), h = lane >> 5, c = lane & 31;
    const int H0 = x_halves(d.ncls[0]), S3 = x_steps(d.ncls[0], d.ncls[1]);
    const int sh = x_pack_sh(d.ncls[0], d.ncls[1]), T = x_pack_shift(d.ncls[0], sh);
    const unsigned m0 = (1u << T) - 1u;
    // item -> (last SNP l below which A lies, group of B subsets, units); the
    // wave's previous item gives the first guess
    int lo = 0, hi = M - 1;
    if (tk.xl < M && t.items[tk.xl] <= local && local < t.items[tk.xl + 1]) lo = hi = tk.xl;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (t.items[mid] <= local) lo = mid; else hi = mid - 1;
    }
    const int l = uni(lo);
    tk.xl = l;
    const unsigned n_a = (unsigned)small_binom(l, KA), n_b = (unsigned)small_binom(M, KB);
    const unsigned units = (n_a + NA - 1) / NA, per_group = (units + (unsigned)t.np - 1) / (unsigned)t.np;
    const unsigned off = (unsigned)(local - t.items[l]);
    const unsigned grp = uni((int)(off / per_group));
    const unsigned u0 = uni((int)((off - grp * per_group) * (unsigned)t.np));
    unsigned n_u = min((unsigned)t.np, units - u0);
    if (PILOT && KA == 3) n_u = min(n_u, 2u);  // a unit holds several combinations
    const unsigned rb0 = ((unsigned)x_first_group(K, M, l) + grp) * NB;
    // lane s < NB: B subset s of the group (lexicographic, the mirror image of
    // the colex order); lane i < n_u NA: A subset i of the item
    int eb[KB], ea[KA];
    {
        const unsigned r = min(rb0 + (unsigned)min(lane, NB - 1), n_b - 1);
        int mc[KB];
        colex_unrank_root<KB>(n_b - 1 - r, mc);
        #pragma unroll
        for (int u = 0; u < KB; ++u) eb[u] = M - 1 - mc[KB - 1 - u];
        colex_unrank_root<KA>(min(u0 * NA + (unsigned)lane, n_a - 1), ea);
    }
    const unsigned nb = min((unsigned)NB, n_b - rb0);  // subsets of the group
    XSide<KB, false> sb_rows;
    sb_rows.init(c, h, (unsigned)S3, M);
    #pragma unroll
    for (int tb = 0; tb < 3; ++tb) {
        int e[KB];
        #pragma unroll
        for (int u = 0; u < KB; ++u)
            e[u] = KB == 2 ? __shfl(eb[u], 3 * tb + min(c / 9, 2)) : __builtin_amdgcn_readlane(eb[u], KB == 3 ? tb : 0);
        sb_rows.set(tb, e);
    }
    sb_rows.finish();
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc((void *)t.xrows, 0, (int)x_row_bytes(M, S3), kBufWord3);
    int sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, READS);
    int pilot_best = (int)0x80000000u;
    constexpr int NB1 = KB == 2 ? 0 : 1;
    XSide<KA, true> sa_rows;
    sa_rows.init(c, h, (unsigned)S3, M);
    // every combination of the item valid: whole groups and units, and all of
    // A below the group's first B subset
    const bool all_valid = nb == (unsigned)NB && (u0 + n_u) * NA <= n_a && l <= __builtin_amdgcn_readlane(eb[0], 0);
    #pragma unroll 1
    for (unsigned v = 0; v < n_u; ++v) {
        #pragma unroll
        for (int ta = 0; ta < 3; ++ta) {
            const int sub = (int)(v * NA) + (KA == 3 ? ta : 0);
            int e[KA];
            #pragma unroll
            for (int u = 0; u < KA; ++u) e[u] = __builtin_amdgcn_readlane(ea[u], sub);
            sa_rows.set(ta, e);
        }
        v16f acc[3][3];
        const bool a_same = sa_rows.same(), b_same = sb_rows.same();
        if (a_same && b_same) {
            x_count<1, NB1>(sa_rows, sb_rows, rx, H0, S3, sh, T, h, acc);
        } else {
            if constexpr (KA == 3 && KB == 3) {
                // (a third copy for shared A rows only cost 475 spilled
                // registers: M = 40, N = 1000 6.7 ms a scan, without 4.1)
                x_count<3, 3>(sa_rows, sb_rows, rx, H0, S3, sh, T, h, acc);
            } else if constexpr (KA == 3) {
                x_count<3, NB1>(sa_rows, sb_rows, rx, H0, S3, sh, T, h, acc);
            } else if constexpr (KB == 3) {
                x_count<1, 3>(sa_rows, sb_rows, rx, H0, S3, sh, T, h, acc);
            }
        }
        // a tile's part of the screening sum, per lane
        // (eight cells' table reads in flight at a time: with two waves per
        // SIMD nothing else hides the LDS latency)
        // rows past a tile's 27 (register 15, and 12 .. 14 of the upper half)
        // and its columns past 27 count as nothing
        const unsigned upper = h ? 0u : ~0u;
        auto cells = [&](const v16f &x, int r) __attribute__((always_inline)) {
            const unsigned w = __float_as_uint(x[r]);
            return r < 12 ? w : w & upper;
        };
        auto part_as = [&](const v16f &x, auto wide) __attribute__((always_inline)) {
            unsigned p = 0, q = 0;
            #pragma unroll
            for (int r0 = 0; r0 < 15; r0 += 5) {
                unsigned t0[5], t1[5], ts[5];
                #pragma unroll
                for (int r = 0; r < 5; ++r) {
                    const unsigned w = cells(x, r0 + r);
                    const unsigned a0 = wide.value ? (w & m0) << 2 : w & m0;
                    const unsigned a1 = wide.value ? (w >> T) << 2 : (w >> (T - 2)) & ~3u;
                    t0[r] = ltab(a0);
                    t1[r] = ltab(a1);
                    ts[r] = ltab(a0 + a1);
                }
                __builtin_amdgcn_sched_barrier(0);
                #pragma unroll
                for (int r = 0; r < 5; ++r) p = add3(p, t0[r], t1[r]);
                q = add3(q, ts[0], ts[1]);
                q = add3(q, ts[2], ts[3]);
                q += ts[4];
            }
            return c < 27 ? p - q : 0u;
        };
        auto part = [&](const v16f &x) __attribute__((always_inline)) {
            return sh ? part_as(x, std::false_type{}) : part_as(x, std::true_type{});
        };
        const unsigned ra0 = (u0 + v) * NA;  // rank of the unit's first A subset
        auto valid_at = [&](int a, int b) {   // A subset a of the unit with B subset b of the group
            return ra0 + (unsigned)a < n_a && (unsigned)b < nb &&
                   __builtin_amdgcn_readlane(ea[KA - 1], (int)(v * NA) + a) < __builtin_amdgcn_readlane(eb[0], b);
        };
        unsigned valid = 0, pass = 0;  // bit a NB + b
        auto judge = [&](int a, int b, unsigned sum) __attribute__((always_inline)) {
            const bool ok = all_valid || valid_at(a, b);
            const int q = a * NB + b;
            valid |= ok ? 1u << q : 0u;
            pass |= ok && (int)sum >= sb ? 1u << q : 0u;
            if constexpr (PILOT)
                if (ok && lane == q) pilot_best = (int)sum > pilot_best ? (int)sum : pilot_best;
        };
        if constexpr (KA == 3) {
            #pragma unroll
            for (int ta = 0; ta < 3; ++ta)
                #pragma unroll
                for (int tb = 0; tb < 3; ++tb) {
                    const unsigned sc = wave_scan_dpp(part(acc[ta][tb]));
                    if constexpr (KB == 2) {
                        // the nine columns of each of the tile's three pairs, in both halves
                        const unsigned e0 = rl(sc, 8), e1 = rl(sc, 17), e2 = rl(sc, 31);
                        const unsigned f0 = rl(sc, 40), f1 = rl(sc, 49), f2 = rl(sc, 63);
                        judge(ta, 3 * tb, e0 + (f0 - e2));
                        judge(ta, 3 * tb + 1, (e1 - e0) + (f1 - f0));
                        judge(ta, 3 * tb + 2, (e2 - e1) + (f2 - f1));
                    } else {
                        judge(ta, tb, rl(sc, 63));
                    }
                }
        } else if constexpr (KB == 3) {
            #pragma unroll
            for (int tb = 0; tb < 3; ++tb)
                judge(0, tb, rl(wave_scan_dpp(part(acc[0][tb]) + part(acc[1][tb]) + part(acc[2][tb])), 63));
        } else {
            unsigned sum = 0;
            #pragma unroll
            for (int ta = 0; ta < 3; ++ta)
                #pragma unroll
                for (int tb = 0; tb < 3; ++tb) sum += part(acc[ta][tb]);
            judge(0, 0, rl(wave_scan_dpp(sum), 63));
        }
        if constexpr (PILOT) continue;
        // combinations that can enter the list: exact score from the same counts
        unsigned todo = CHECK ? valid : pass;
        #pragma unroll 1
        while (todo) {
            const int q = (int)__builtin_ctz(todo), a = q / NB, b = q - a * NB;
            todo &= todo - 1;
            int cc[K];
            #pragma unroll
            for (int u = 0; u < KA; ++u) cc[u] = __builtin_amdgcn_readlane(ea[u], (int)(v * NA) + a);
            #pragma unroll
            for (int u = 0; u < KB; ++u) cc[KA + u] = __builtin_amdgcn_readlane(eb[u], b);
            long long num = 0;
            unsigned long long dsum = 0;
            #pragma unroll 1
            for (int tile = 0; tile < 9; ++tile) {
                const int ta = tile / 3, tb = tile - 3 * ta;
                if (KA == 3 && ta != a) continue;
                if (KB == 3 && tb != b) continue;
                if (KB == 2 && tb != b / 3) continue;
                v16f x = acc[0][0];
                #pragma unroll
                for (int k = 1; k < 9; ++k)
                    if (tile == k) x = acc[k / 3][k % 3];
                if (c >= 27 || (KB == 2 && c / 9 != b % 3)) continue;  // the lanes of its columns
                #pragma unroll
                for (int r = 0; r < 15; ++r) {
                    const unsigned w = cells(x, r);
                    const unsigned n0 = (w & m0) >> sh, n1 = w >> T;
                    num += cell_term_counted(d.tlog, n0, n1);
                    if constexpr (CHECK) {
                        const int row = 8 * (r / 4) + 4 * h + r % 4;
                        const int xA = KA == 3 ? row : 27 * ta + row;
                        const int xB = KB == 2 ? c % 9 : (KB == 3 ? c : 27 * tb + c);
                        const int cell = xA * pow3c(KB) + xB;
                        dsum += (unsigned long long)n0 * cell_weight(0, cell) +
                                (unsigned long long)n1 * cell_weight(1, cell);
                    }
                }
            }
            num = t.score_const + wave_sum64(num);
            if constexpr (CHECK) {
                digest_add(tk, lane == 0, combo_hash<K>(cc), (unsigned long long)wave_sum64((long long)dsum));
                if (!(pass >> q & 1u)) continue;
            }
            unsigned long long key = 0;
            #pragma unroll
            for (int u = 0; u < K; ++u) key = (key << t.key_bits) | (unsigned long long)cc[u];
            tk_offer(tk, list, lane == 0, num, key, gthr);
            sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, READS);
        }
    }
    if constexpr (PILOT) pilot_count(tk, t, pilot_best, READS);
}

// ---------------------------------------------------------------------------
// kGeneric: any order K (orders 4-8 where kR4 and kX do not fit).  A work item is 64 * kGenRanks consecutive colex
// ranks; lane l takes ranks l, l + 64, ...  Each lane counts all 3^K cells of
// its own combination, 27 cells (the last three SNPs) at a time for each
// genotype choice of the first K - 3 SNPs.
// ---------------------------------------------------------------------------
constexpr int kGenRanks = 4;

template <int K>
EPI_DEV void colex_unrank(unsigned long long rank, int M, const unsigned long long *binom, int bstride, int (&c)[K]) {
    #pragma unroll
    for (int t = K; t >= 1; --t) {
        const unsigned long long *row = binom + (long long)t * bstride;
        int lo = t - 1, hi = M - 1;
        while (lo < hi) {
            int mid = (lo + hi + 1) >> 1;
            if (row[mid] <= rank) lo = mid; else hi = mid - 1;
        }
        c[t - 1] = lo;
        rank -= row[lo];
    }
}

// The combinations of a wave's 64 consecutive colex ranks first .. first +
// 63: c enters as the combination of rank first (the same in every lane) and
// leaves as that of rank first + lane, by steps through the colex order,
// where the lowest index rises until it meets the next one, and the next
// combination then raises the lowest index that can grow and resets those
// below it to 0, 1, ...  A lane passes the loop once per run of its lowest
// index that it crosses, a few times at most.  Lanes past the last
// combination (valid false) get the first one, 0, 1, ..., K - 1.
template <int K>
EPI_DEV void colex_advance(int (&c)[K], int steps, bool valid) {
    if (!valid) {
        #pragma unroll
        for (int t = 0; t < K; ++t) c[t] = t;
        return;
    }
    #pragma unroll 1
    while (steps > 0) {
        const int room = c[1] - 1 - c[0];
        if (steps <= room) {
            c[0] += steps;
            break;
        }
        steps -= room + 1;
        int t = 1;
        #pragma unroll 1
        while (t < K - 1 && c[t] + 1 >= c[t + 1]) ++t;
        #pragma unroll
        for (int u = 0; u < K; ++u) {
            if (u == t) c[u] += 1;
            else if (u < t) c[u] = u;
        }
    }
}

// The combination after c in the colex order (wave-uniform values).
template <int K>
EPI_DEV void colex_next(int (&c)[K]) {
    int t = 0;
    #pragma unroll 1
    while (t < K - 1 && c[t] + 1 >= c[t + 1]) ++t;
    #pragma unroll
    for (int u = 0; u < K; ++u) {
        if (u == t) c[u] += 1;
        else if (u < t) c[u] = u;
    }
}

// Lane combinations of a per-combination work item, one block of 64 colex
// ranks after another: the item's first rank is unranked once, each block
// starts at the successor of the previous block's last combination, and the
// lanes step from there.
template <int K>
struct ColexWalk {
    int first[K];
    EPI_DEV void start(unsigned long long rank, int M, const unsigned long long *binom, int bstride) {
        colex_unrank<K>(rank, M, binom, bstride, first);
        #pragma unroll
        for (int t = 0; t < K; ++t) first[t] = uni(first[t]);
    }
    // this lane's combination of the block (c), then the next block's first
    EPI_DEV void lane(int (&c)[K], bool valid) {
        #pragma unroll
        for (int t = 0; t < K; ++t) c[t] = first[t];
        colex_advance<K>(c, lane_id(), valid);
        #pragma unroll
        for (int t = 0; t < K; ++t) first[t] = __builtin_amdgcn_readlane(c[t], kWave - 1);
        colex_next<K>(first);
    }
};

// Grouped counting for K >= 5: the three 27-cell chunks that differ only in
// the genotype of the last prefix SNP c[K-4] are counted in one pass over the
// words, so each word's rows and the AND of the other prefix rows are loaded
// and formed once for 81 cells instead of once per 27 (a third of the loads;
// per 32 individuals 81 AND + popcount pairs and 12 other operations).  The
// 81 class-0 counts wait for class 1 packed two to a register, so classes
// of up to 65535 individuals only.
template <int K>
EPI_DEV void g3_count(const DsView &d, const int (&c)[K], const int *dig, int cl, unsigned (&acc)[81]) {
    constexpr int NB = K - 4;
    gv4u *gm = (gv4u *)d.masks;
    const long long Mp = d.Mp;
    const int sp = c[NB];
    #pragma unroll
    for (int x = 0; x < 81; ++x) acc[x] = 0;
    const int W = d.w4[cl];
    long long off = (long long)d.wbase[cl] * 2 * Mp;
    for (int w = 0; w < W; ++w, off += 2 * Mp) {
        const v4u vm = valid_mask(d.ncls[cl], w);
        v4u X = vm;
        #pragma unroll
        for (int t = 0; t < NB; ++t) {
            const v4u r0 = gm[off + c[t]];
            const v4u r1 = gm[off + Mp + c[t]];
            X &= dig[t] == 0 ? r0 : (dig[t] == 1 ? r1 : vm & ~(r0 | r1));
        }
        const v4u p0 = gm[off + sp], p1 = gm[off + Mp + sp];
        v4u r0[3], r1[3];
        #pragma unroll
        for (int u = 0; u < 3; ++u) {
            r0[u] = gm[off + c[K - 3 + u]];
            r1[u] = gm[off + Mp + c[K - 3 + u]];
        }
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            unsigned rw[3][3];
            #pragma unroll
            for (int u = 0; u < 3; ++u) {
                rw[u][0] = r0[u][q];
                rw[u][1] = r1[u][q];
                rw[u][2] = vm[q] & ~(r0[u][q] | r1[u][q]);
            }
            #pragma unroll
            for (int g = 0; g < 3; ++g) {
                const unsigned xg = X[q] & (g == 0 ? p0[q] : (g == 1 ? p1[q] : vm[q] & ~(p0[q] | p1[q])));
                #pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const unsigned xa = xg & rw[0][a];
                    #pragma unroll
                    for (int b = 0; b < 3; ++b)
                        #pragma unroll
                        for (int e = 0; e < 3; ++e)
                            acc[27 * g + 9 * a + 3 * b + e] =
                                bcnt_acc(xa & rw[1][b] & rw[2][e], acc[27 * g + 9 * a + 3 * b + e]);
                }
            }
        }
    }
}

template <int K, bool STORE, bool LDT, bool DIG>
EPI_DEV long long generic_num_g3(const DsView &d, const int (&c)[K], long long score_const, uint32_t *out,
                                 int ostride, unsigned long long *dsum) {
    constexpr int NB = K - 4;       // prefix SNPs fixed within a group
    constexpr int NG = pow3c(NB);   // groups of 81 cells
    long long num = score_const;
    #pragma unroll 1
    for (int gi = 0; gi < NG; ++gi) {
        int dig[NB > 0 ? NB : 1];
        {
            int x = gi;
            #pragma unroll
            for (int t = NB - 1; t >= 0; --t) {
                dig[t] = x % 3;
                x /= 3;
            }
        }
        unsigned acc[81], pk[41];
        g3_count<K>(d, c, dig, 0, acc);
        #pragma unroll
        for (int x = 0; x < 41; ++x) pk[x] = acc[2 * x] | (2 * x + 1 < 81 ? acc[2 * x + 1] << 16 : 0u);
        g3_count<K>(d, c, dig, 1, acc);
        #pragma unroll
        for (int x = 0; x < 81; ++x) {
            const unsigned n0 = x & 1 ? pk[x >> 1] >> 16 : pk[x >> 1] & 0xffffu;
            if constexpr (DIG)
                *dsum += (unsigned long long)n0 * cell_weight(0, gi * 81 + x) +
                         (unsigned long long)acc[x] * cell_weight(1, gi * 81 + x);
            if constexpr (STORE) {
                out[(gi * 81 + x) * ostride] = n0;
                out[(pow3c(K) + gi * 81 + x) * ostride] = acc[x];
            } else {
                num += LDT ? cell_term_lds(n0, acc[x]) : cell_term_counted(d.tlog, n0, acc[x]);
            }
        }
    }
    return num;
}

// Counts every cell of combination c, 27 (order 2: 9) at a time.  The fused
// form (STORE false) scores each chunk as it is counted and returns the
// score; with STORE the counts go to out[x * ostride] (class 0) and
// out[(3^K + x) * ostride] (class 1) instead, x the cell's index in base 3
// with the genotype of c[0] as the leading digit.  With DIG the weighted sum
// of the counts (the table part of the completeness digest) is added to
// *dsum.
template <int K, bool STORE = false, bool LDT = false, bool DIG = false>
EPI_DEV long long generic_num(const DsView &d, const int (&c)[K], long long score_const, uint32_t *out = nullptr,
                              int ostride = kWave, unsigned long long *dsum = nullptr) {
    if constexpr (K >= 5)
        if (d.ncls[0] <= 0xffff) return generic_num_g3<K, STORE, LDT, DIG>(d, c, score_const, out, ostride, dsum);
    constexpr int NPRE = K > 3 ? K - 3 : 0;
    constexpr int NCH = pow3c(NPRE);
    constexpr int L = K >= 3 ? 3 : 2;
    constexpr int CELLS = L == 3 ? 27 : 9;
    gv4u *gm = (gv4u *)d.masks;
    const long long Mp = d.Mp;
    long long num = score_const;
    for (int ch = 0; ch < NCH; ++ch) {
        int dig[NPRE > 0 ? NPRE : 1];
        {
            int x = ch;
            #pragma unroll
            for (int t = NPRE - 1; t >= 0; --t) {
                dig[t] = x % 3;
                x /= 3;
            }
        }
        unsigned acc[2][CELLS];
        #pragma unroll
        for (int cl = 0; cl < 2; ++cl) {
            #pragma unroll
            for (int x = 0; x < CELLS; ++x) acc[cl][x] = 0;
            const int W = d.w4[cl];
            long long off = (long long)d.wbase[cl] * 2 * Mp;
            for (int w = 0; w < W; ++w, off += 2 * Mp) {
                const v4u vm = valid_mask(d.ncls[cl], w);
                v4u X = vm;
                #pragma unroll
                for (int t = 0; t < NPRE; ++t) {
                    const v4u r0 = gm[off + c[t]];
                    const v4u r1 = gm[off + Mp + c[t]];
                    const v4u r2 = vm & ~(r0 | r1);
                    X &= dig[t] == 0 ? r0 : (dig[t] == 1 ? r1 : r2);
                }
                v4u rows[L][3];
                #pragma unroll
                for (int u = 0; u < L; ++u) {
                    const int s = c[K - L + u];
                    rows[u][0] = gm[off + s];
                    rows[u][1] = gm[off + Mp + s];
                    rows[u][2] = vm & ~(rows[u][0] | rows[u][1]);
                }
                #pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (L == 3) {
                        #pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            const unsigned xa = X[q] & rows[0][a][q];
                            #pragma unroll
                            for (int b = 0; b < 3; ++b)
                                #pragma unroll
                                for (int e = 0; e < 3; ++e)
                                    acc[cl][9 * a + 3 * b + e] =
                                        bcnt_acc(xa & rows[1][b][q] & rows[2][e][q], acc[cl][9 * a + 3 * b + e]);
                        }
                    } else {
                        #pragma unroll
                        for (int a = 0; a < 3; ++a)
                            #pragma unroll
                            for (int b = 0; b < 3; ++b)
                                acc[cl][3 * a + b] = bcnt_acc(rows[0][a][q] & rows[1][b][q], acc[cl][3 * a + b]);
                    }
                }
            }
        }
        if constexpr (DIG) {
            #pragma unroll
            for (int x = 0; x < CELLS; ++x)
                *dsum += (unsigned long long)acc[0][x] * cell_weight(0, ch * CELLS + x) +
                         (unsigned long long)acc[1][x] * cell_weight(1, ch * CELLS + x);
        }
        if constexpr (STORE) {
            #pragma unroll
            for (int x = 0; x < CELLS; ++x) {
                out[(ch * CELLS + x) * ostride] = acc[0][x];
                out[(pow3c(K) + ch * CELLS + x) * ostride] = acc[1][x];
            }
        } else {
            #pragma unroll
            for (int x = 0; x < CELLS; ++x)
                num += LDT ? cell_term_lds(acc[0][x], acc[1][x]) : cell_term_counted(d.tlog, acc[0][x], acc[1][x]);
        }
    }
    return num;
}

template <int K, bool LDT, bool CHECK = false>
EPI_DEV void item_generic(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr,
                          const unsigned long long *binom, int bstride) {
    const DsView d = t.ds;
    const int bits = t.key_bits;
    ColexWalk<K> walk;
    walk.start(local * kGenRanks * kWave, d.M, binom, bstride);
    for (int rr = 0; rr < kGenRanks; ++rr) {
        const unsigned long long rank = (local * kGenRanks + rr) * kWave + lane_id();
        const bool valid = rank < t.n_combos;
        int c[K];
        walk.lane(c, valid);
        unsigned long long sum = 0;
        const long long num = generic_num<K, false, LDT, CHECK>(d, c, t.score_const, nullptr, kWave, &sum);
        if constexpr (CHECK) digest_add(tk, valid, combo_hash<K>(c), sum);
        unsigned long long key = 0;
        #pragma unroll
        for (int u = 0; u < K; ++u) key = (key << bits) | (unsigned long long)c[u];
        tk_offer(tk, list, valid, num, key, gthr);
    }
}

// ---------------------------------------------------------------------------
// kSeg: the segmented exploration of Section 3.4 (Algorithm 2) on a wave.  A
// block of b = 64 combinations (one per lane) first has all 2 x 3^K cells of
// its contingency tables counted, as kGeneric counts them, into the wave's
// slot of a device buffer (cell-major, 64 lanes contiguous); only then are
// the b tables read back and scored.  The item's kGenRanks blocks follow one
// another through the same slot.  A lane reads back only what it wrote, so
// program order is the only ordering needed.
// ---------------------------------------------------------------------------
template <int K, bool LDT, bool CHECK = false>
EPI_DEV void item_seg(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr,
                      const unsigned long long *binom, int bstride, uint32_t *slot) {
    constexpr int CELLS = pow3c(K);
    const DsView d = t.ds;
    const int bits = t.key_bits;
    const int lane = lane_id();
    uint32_t *mine = slot + lane;
    ColexWalk<K> walk;
    walk.start(local * kGenRanks * kWave, d.M, binom, bstride);
    #pragma unroll 1
    for (int rr = 0; rr < kGenRanks; ++rr) {
        const unsigned long long rank = (local * kGenRanks + rr) * kWave + lane;
        const bool valid = rank < t.n_combos;
        int c[K];
        walk.lane(c, valid);
        // phase 1: the block's tables
        (void)generic_num<K, true>(d, c, 0, mine);
        // phase 2: their scores
        long long num = t.score_const;
        unsigned long long sum = 0;
        #pragma unroll 9
        for (int x = 0; x < CELLS; ++x) {
            const unsigned n0 = mine[x * kWave], n1 = mine[(CELLS + x) * kWave];
            num += LDT ? cell_term_lds(n0, n1) : cell_term_counted(d.tlog, n0, n1);
            if constexpr (CHECK)
                sum += (unsigned long long)n0 * cell_weight(0, x) + (unsigned long long)n1 * cell_weight(1, x);
        }
        if constexpr (CHECK) digest_add(tk, valid, combo_hash<K>(c), sum);
        unsigned long long key = 0;
        #pragma unroll
        for (int u = 0; u < K; ++u) key = (key << bits) | (unsigned long long)c[u];
        tk_offer(tk, list, valid, num, key, gthr);
    }
}

// ---------------------------------------------------------------------------
// kR4: order 4 by reduced cells.  A work item is 64 * kGenRanks consecutive
// colex ranks; lane l takes ranks l, l + 64, ... (as kGeneric).  A lane counts
// the 16 cells of its combination whose four genotypes are all 0 or 1 (per 32
// individuals: 4 pair ANDs, then one three-input AND and one popcount per
// cell); every other cell follows by inclusion-exclusion from the triplet
// sub-table (written by the matrix-core kernel), the pair sub-table and the
// single-SNP counts, as for order 3; the sub-tables hold both classes of a
// cell in one register (4 n(cases) | 4 n(controls) << 16), and so do the
// lane's 81 cells.
// ---------------------------------------------------------------------------
// PILOT: the histogram-only pass (as for order 3).
template <bool LDS, bool CHECK = false, bool PILOT = false>
EPI_DEV void item_r4(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr,
                     const unsigned long long *binom, int bstride) {
    const DsView d = t.ds;
    int pilot_best = (int)0x80000000u;  // PILOT: the lane's best screening sum
    int sb = 0;
    if constexpr (LDS) sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 243);
    const int bits = t.key_bits;
    gv4u *gm = (gv4u *)d.masks;
    gv4u *single4 = (gv4u *)d.single;
    gv4u *pair4 = (gv4u *)t.pairs;
    gv4u *trip4 = (gv4u *)t.triples;
    const long long Mp = d.Mp;
    ColexWalk<4> walk;
    walk.start(local * kGenRanks * kWave, d.M, binom, bstride);
    #pragma unroll 1
    for (int rr = 0; rr < kGenRanks; ++rr) {
        const unsigned long long rank = (local * kGenRanks + rr) * kWave + lane_id();
        const bool valid = rank < t.n_combos;
        int c[4];
        walk.lane(c, valid);
        unsigned acc[2][16];
        // consecutive colex ranks share their two last SNPs almost always:
        // then their rows are wave-uniform scalar loads and their four
        // pairwise ANDs scalar operations, which halves the vector loads
        const int c2u = uni(c[2]), c3u = uni(c[3]);
        const bool u23 = __ballot(c[2] != c2u || c[3] != c3u) == 0ull;
        #pragma unroll
        for (int cl = 0; cl < 2; ++cl) {
            #pragma unroll
            for (int x = 0; x < 16; ++x) acc[cl][x] = 0;
            const int W = d.w4[cl];
            long long off = (long long)d.wbase[cl] * 2 * Mp;
            if (u23) {
                cv4u *sm = (cv4u *)d.masks;
                #pragma unroll 1
                for (int w = 0; w < W; ++w, off += 2 * Mp) {
                    v4u r[2][2];
                    #pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        r[u][0] = gm[off + c[u]];
                        r[u][1] = gm[off + Mp + c[u]];
                    }
                    const v4u s20 = sm[off + c2u], s21 = sm[off + Mp + c2u];
                    const v4u s30 = sm[off + c3u], s31 = sm[off + Mp + c3u];
                    #pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        unsigned p[4], y[4];
                        #pragma unroll
                        for (int ab = 0; ab < 4; ++ab) p[ab] = r[0][ab >> 1][q] & r[1][ab & 1][q];
                        y[0] = uni(s20[q] & s30[q]);
                        y[1] = uni(s20[q] & s31[q]);
                        y[2] = uni(s21[q] & s30[q]);
                        y[3] = uni(s21[q] & s31[q]);
                        #pragma unroll
                        for (int ab = 0; ab < 4; ++ab)
                            #pragma unroll
                            for (int ce = 0; ce < 4; ++ce)
                                acc[cl][4 * ab + ce] = bcnt_acc(p[ab] & y[ce], acc[cl][4 * ab + ce]);
                    }
                }
            } else {
                #pragma unroll 1
                for (int w = 0; w < W; ++w, off += 2 * Mp) {
                    v4u r[4][2];
                    #pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        r[u][0] = gm[off + c[u]];
                        r[u][1] = gm[off + Mp + c[u]];
                    }
                    #pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        unsigned p[4];
                        #pragma unroll
                        for (int ab = 0; ab < 4; ++ab) p[ab] = r[0][ab >> 1][q] & r[1][ab & 1][q];
                        #pragma unroll
                        for (int ab = 0; ab < 4; ++ab)
                            #pragma unroll
                            for (int ce = 0; ce < 4; ++ce)
                                acc[cl][4 * ab + ce] =
                                    bcnt_acc(p[ab] & r[2][ce >> 1][q] & r[3][ce & 1][q], acc[cl][4 * ab + ce]);
                    }
                }
            }
            // (keeps the scaling below out of the loop, where the compiler
            // would otherwise redo it every iteration)
            #pragma unroll
            for (int x = 0; x < 16; ++x) asm volatile("" : "+v"(acc[cl][x]));
        }
        // F[27 a + 9 b + 3 g + e]; digit 2 = marginal over that SNP, genotype
        // 2 once the inclusion-exclusion has run.  Packed cell form: a
        // register holds 4 n(cases) in its low half and 4 n(controls) in its
        // high half (classes of at most 16383 individuals), so one
        // subtraction steps both classes (no half ever goes below zero: a
        // marginal is at least the sum of its cells), and each half is the
        // byte address of its count's screening-table entry.  The
        // sub-table passes write their cells in this form.
        unsigned F[81];
        #pragma unroll
        for (int x = 0; x < 81; ++x) {
            const int a = x / 27, b = (x / 9) % 3, g = (x / 3) % 3, e = x % 3;
            if (a < 2 && b < 2 && g < 2 && e < 2) {
                const int i = 8 * a + 4 * b + 2 * g + e;
                F[x] = (acc[0][i] << kQScaleShift) | (acc[1][i] << (16 + kQScaleShift));
            }
        }
        // triplets: drop one SNP (its digit 2), cells 4a' + 2b' + d' of the rest
        #pragma unroll
        for (int drop = 0; drop < 4; ++drop) {
            int s3[3], k = 0;
            #pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u != drop) s3[k++] = c[u];
            const unsigned long long tr = colex3(s3[0], s3[1], s3[2]);
            const v4u lo = trip4[2 * tr], hi = trip4[2 * tr + 1];
            #pragma unroll
            for (int y = 0; y < 8; ++y) {
                int dig[4], k2 = 0;
                #pragma unroll
                for (int u = 0; u < 4; ++u) dig[u] = u == drop ? 2 : (y >> (2 - k2++)) & 1;
                F[27 * dig[0] + 9 * dig[1] + 3 * dig[2] + dig[3]] = y < 4 ? lo[y] : hi[y - 4];
            }
        }
        // pairs: keep two SNPs
        #pragma unroll
        for (int u0 = 0; u0 < 4; ++u0)
            #pragma unroll
            for (int u1 = u0 + 1; u1 < 4; ++u1) {
                const v4u pv = pair4[colex2(c[u0], c[u1])];  // the pair sub-table in colex order
                #pragma unroll
                for (int y = 0; y < 4; ++y) {
                    int dig[4];
                    #pragma unroll
                    for (int u = 0; u < 4; ++u) dig[u] = u == u0 ? (y >> 1) : (u == u1 ? (y & 1) : 2);
                    F[27 * dig[0] + 9 * dig[1] + 3 * dig[2] + dig[3]] = pv[y];
                }
            }
        // singles and the class sizes
        #pragma unroll
        for (int u = 0; u < 4; ++u) {
            const v4u sv = single4[c[u]];
            #pragma unroll
            for (int g = 0; g < 2; ++g) {
                int dig[4];
                #pragma unroll
                for (int v = 0; v < 4; ++v) dig[v] = v == u ? g : 2;
                F[27 * dig[0] + 9 * dig[1] + 3 * dig[2] + dig[3]] =
                    (sv[g] << kQScaleShift) | (sv[2 + g] << (16 + kQScaleShift));
            }
        }
        F[80] = ((unsigned)d.ncls[0] << kQScaleShift) | ((unsigned)d.ncls[1] << (16 + kQScaleShift));
        mobius4(F);
        if constexpr (PILOT) {
            static_assert(LDS && !CHECK, "the pilot pass reads the screening table from LDS");
            if (valid) {
                const int S = screen_sum_packed<81>(F);
                pilot_best = S > pilot_best ? S : pilot_best;
            }
            continue;
        }
        if constexpr (CHECK) {
            unsigned long long sum = 0;
            #pragma unroll
            for (int x = 0; x < 81; ++x)
                sum += (unsigned long long)((F[x] & 0xffffu) >> kQScaleShift) * cell_weight(0, x) +
                       (unsigned long long)(F[x] >> (16 + kQScaleShift)) * cell_weight(1, x);
            digest_add(tk, valid, combo_hash<4>(c), sum);
        }
        bool pass = valid;
        if constexpr (LDS) pass = pass && screen_sum_packed<81>(F) >= sb;
        if (__ballot(pass)) {
            long long num = t.score_const;
            #pragma unroll
            for (int x = 0; x < 81; ++x)
                num += cell_term_counted(d.tlog, (F[x] & 0xffffu) >> kQScaleShift, F[x] >> (16 + kQScaleShift));
            unsigned long long key = 0;
            #pragma unroll
            for (int u = 0; u < 4; ++u) key = (key << bits) | (unsigned long long)c[u];
            tk_offer(tk, list, pass, num, key, gthr);
            if constexpr (LDS) sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 243);
        }
    }
    if constexpr (PILOT) pilot_count(tk, t, pilot_best, 243);
}

// ---------------------------------------------------------------------------
// kR4M: order 4 by reduced cells, the cells counted on the matrix cores.  A
// work item is a middle pair j < k with 32 first SNPs i (B columns) and 16
// last SNPs l (A rows, two genotypes each).  The rows of l masked by j's
// (genotype b) and the columns of i's genotype a masked by k's (genotype c)
// give eight products a step: three loads feed 24 matrix instructions, both
// classes in one accumulator (q3_pack_fits).  Lane = SNP i; a lane holds all
// 16 reduced cells of its i with eight l's, so the scoring is that of kR4: the
// marginals come from the sub-tables, whose colex order puts consecutive i in
// consecutive lanes.
//
// Bound by the scoring: 81 cells are 243 reads of the screening table.  M =
// 200, N = 2000: a wave issues 341 LDS, 1346 vector and 57 matrix instructions
// of 32 cycles per 64 combinations (counters; 0.73 of the lanes hold one), the
// kernel takes 5.0 ms, 1.4 of it without the scoring and 3.5 without the table
// reads, against 7.5 ms for kR4.  A table of
// t(n0) + t(n1) - t(n0 + n1) for small counts, one read a cell, was slower
// (6.9): equal small counts share one read of the plain table.
// ---------------------------------------------------------------------------
template <bool CHECK = false, bool PILOT = false>
EPI_DEV void item_r4m(const Task &t, unsigned long long local, TopK &tk, Cand *list, long long gthr, v4u *stage) {
    static_assert(!PILOT || !CHECK, "the pilot pass only counts");
    typedef QFmt<false> Q;
    const DsView d = t.ds;
    const int M = d.M, lane = lane_id(), h = lane >> 5;
    // item -> group (block of i, block of l), then k and j
    int lo = 0, hi = r4_groups(M) - 1;
    if (tk.xl <= hi && t.items[tk.xl] <= local && local < t.items[tk.xl + 1]) lo = hi = tk.xl;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (t.items[mid] <= local) lo = mid; else hi = mid - 1;
    }
    tk.xl = uni(lo);
    const int nib = r4_iblocks(M), ib = tk.xl % nib, lb = tk.xl / nib;
    const unsigned off = (unsigned)(local - t.items[tk.xl]);
    // k's place r in the group, r (r + 1) / 2 <= off: a root, then corrected
    unsigned r = (unsigned)((sqrtf(8.0f * (float)off + 1.0f) - 1.0f) * 0.5f);
    while (r * (r + 1) / 2 > off) --r;
    while ((r + 1) * (r + 2) / 2 <= off) ++r;
    const int i0 = kR4I * ib, l0 = kR4L * lb;
    const int kk = uni(i0 + 2 + (int)r), j = uni(i0 + 1 + (int)(off - r * (r + 1) / 2));
    const int i = i0 + (lane & 31);

    // Sub-table rows are read through buffer descriptors, so that a lane
    // without a valid combination reads another entry, or zeros past the
    // table's end.
    auto C2 = [](int x) { return (long long)x * (x - 1) / 2; };
    auto C3 = [](int x) { return (long long)x * (x - 1) * (x - 2) / 6; };
    auto rows = [](const void *p, long long at, long long end) {
        const long long left = end - at;
        return __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)p + at), 0,
                                                 (int)(left < 0x7fffffffll ? left : 0x7fffffffll), kBufWord3);
    };
    const long long t_end = 32 * C3(M), p_end = 16 * C2(M);
    const __amdgpu_buffer_rsrc_t rTk = rows(t.triples, 32 * (C3(kk) + C2(j) + i0), t_end);
    const __amdgpu_buffer_rsrc_t rP = rows(t.pairs, 0, p_end);
    const __amdgpu_buffer_rsrc_t rS = __builtin_amdgcn_make_buffer_rsrc((void *)d.single, 0, d.Mp * 16, kBufWord3);

    const int KS = d.xs, H0 = d.xh0, T = q3_pack_shift(d.ncls[0]), blk = KS * 1024;
    const v4u *qa = Q::qa(d), *qb = Q::qb(d);
    auto block = [&](const v4u *q, int b) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)(q + (long long)b * KS * 64), 0, blk, kBufWord3);
    };
    const __amdgpu_buffer_rsrc_t rA = block(qa, lb), rB0 = block(qb, 2 * ib), rB1 = block(qb, 2 * ib + 1);
    const __amdgpu_buffer_rsrc_t rM[2] = {block(qa, j >> 4), block(qa, kk >> 4)};
    const int mrow[2] = {j & 15, kk & 15};
    const int vo = lane * 16;
    typename Q::acc_t acc[2][2][2];  // [b][c][a]
    #pragma unroll
    for (int x = 0; x < 8; ++x) acc[x >> 2][(x >> 1) & 1][x & 1] = (typename Q::acc_t){};
    // mask rows of j and k staged as those of the two middle SNPs of item_f3m
    constexpr int kSeg = kQStageSteps;
    lv4u *slot = (lv4u *)stage;
    auto stage_masks = [&](int base) __attribute__((always_inline)) {
        const int n = min(kSeg, KS - base);
        wave_sync();
        #pragma unroll
        for (int jj = 0; jj < 2; ++jj)
            #pragma unroll
            for (int e0 = 0; e0 < 4 * kSeg; e0 += kWave) {
                const int e = min(e0 + lane, 4 * n - 1);
                const int v = (((e >> 2) * 64) + 32 * ((e >> 1) & 1) + 2 * mrow[jj] + (e & 1)) * 16;
                slot[jj * 4 * kSeg + e0 + lane] = qload(rM[jj], v, base * 1024);
            }
        wave_sync();
    };
    struct Ops {
        v4u a, b0, b1;
    };
    auto load = [&](int s) __attribute__((always_inline)) {
        const int so = min(s, KS - 1) * 1024;
        return Ops{qload(rA, vo, so), qload(rB0, vo, so), qload(rB1, vo, so)};
    };
    int seg = 0;
    auto mul = [&](int s, const Ops &o, int e) __attribute__((always_inline)) {
        const int js = 4 * (s - seg) + 2 * h;
        const v4u J0 = slot[js], J1 = slot[js + 1], K0 = slot[4 * kSeg + js], K1 = slot[4 * kSeg + js + 1];
        #pragma unroll
        for (int p = 0; p < 3; ++p) {
            const unsigned pb = plane_bits(p);
            const int sb = plane_scale(e, p);
            const v4u A0 = o.a & J0 & pb, A1 = o.a & J1 & pb;
            #pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int c = x >> 1, a = x & 1;
                const v4u B = (a ? o.b1 : o.b0) & (c ? K1 : K0) & pb;
                acc[0][c][a] = Q::mma(A0, B, acc[0][c][a], sb, kScaleA);
                acc[1][c][a] = Q::mma(A1, B, acc[1][c][a], sb, kScaleA);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    Ops x = load(0);
    stage_masks(0);
    #pragma unroll 1
    for (int s = 0; s < KS; s += 2) {
        if (s >= seg + kSeg) {
            seg += kSeg;
            stage_masks(seg);
        }
        const Ops y = load(s + 1);
        mul(s, x, 2 * s + h >= H0 ? T : 2);
        __builtin_amdgcn_sched_barrier(0);
        x = load(s + 2);
        if (s + 1 < KS) mul(s + 1, y, 2 * s + 2 + h >= H0 ? T : 2);
    }
    wave_sync();  // the slot's rows have been read

    auto pack2 = [](unsigned n0, unsigned n1) __attribute__((always_inline)) {
        return (n0 << kQScaleShift) | (n1 << (16 + kQScaleShift));
    };
    const v4u pjk = ((cv4u *)t.pairs)[C2(kk) + j];
    const v4u sj = ((cv4u *)d.single)[j], sk = ((cv4u *)d.single)[kk];
    const unsigned nall = pack2((unsigned)d.ncls[0], (unsigned)d.ncls[1]);
    // triplets with l: from the block's first l on; C(l0 + x, 3) - C(l0, 3) =
    // x C(l0, 2) + C(x, 2) l0 + C(x, 3)
    const __amdgpu_buffer_rsrc_t rT = rows(t.triples, 32 * C3(l0), t_end);
    const int c2l = (int)C2(l0), cj = (int)C2(j) * 32, ck = (int)C2(kk) * 32;
    int pilot_best = (int)0x80000000u;  // PILOT: the lane's best screening sum
    int sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 243);
    // One genotype's 27 cells of a table over three SNPs, in the packed form
    // of kR4: reduced cells r, pair marginals p (cells of SNPs 1, 2), q (1, 3)
    // and s (2, 3), single ones x, y, z, all of them n.  Every difference is a
    // count of its own, so no half goes below zero.
    auto complete = [](unsigned (&G)[27], const unsigned (&p)[4], const unsigned (&q)[4], const unsigned (&s)[4],
                       const unsigned (&x)[2], const unsigned (&y)[2], const unsigned (&z)[2], unsigned n)
                        __attribute__((always_inline)) {
        unsigned y2[2];  // genotype 2 of SNP 1, f of SNP 2, any of SNP 3
        #pragma unroll
        for (int f = 0; f < 2; ++f) {
            #pragma unroll
            for (int g = 0; g < 2; ++g) {
                G[9 * f + 3 * g + 2] = p[2 * f + g] - G[9 * f + 3 * g] - G[9 * f + 3 * g + 1];
                G[9 * f + 6 + g] = q[2 * f + g] - G[9 * f + g] - G[9 * f + 3 + g];
            }
            G[9 * f + 8] = x[f] - p[2 * f] - p[2 * f + 1] - G[9 * f + 6] - G[9 * f + 7];
            y2[f] = y[f] - p[f] - p[2 + f];
        }
        #pragma unroll
        for (int f = 0; f < 2; ++f) {
            #pragma unroll
            for (int g = 0; g < 2; ++g) G[18 + 3 * f + g] = s[2 * f + g] - G[3 * f + g] - G[9 + 3 * f + g];
            G[18 + 3 * f + 2] = y2[f] - G[18 + 3 * f] - G[18 + 3 * f + 1];
        }
        #pragma unroll
        for (int g = 0; g < 2; ++g) G[24 + g] = z[g] - q[g] - q[2 + g] - G[18 + g] - G[21 + g];
        G[26] = n - x[0] - x[1] - y2[0] - y2[1] - G[24] - G[25];
    };
    const int li = (lane & 31) * 32, cij = (int)C2(j) * 16, cik = (int)C2(kk) * 16;
    // one loop body for all eight l's of a lane (its code in the instruction
    // cache, one copy of the exact path): only the accumulators are picked by
    // a branch
    #pragma unroll 1
    for (int u = 0; u < 8; ++u) {
        const int x0 = 4 * (u >> 1) + (u & 1), x2 = x0 + 2;  // l - l0 in the two lane halves
        const int l = l0 + x0 + 2 * h;
        const bool valid = i < j && l > kk && l < M;
        if (!__ballot(valid)) continue;
        unsigned W[16];  // the reduced cells 8 a + 4 b + 2 c + e
        auto pick = [&](auto uc) __attribute__((always_inline)) {
            constexpr int r0 = 4 * (uc.value >> 1) + 2 * (uc.value & 1);
            #pragma unroll
            for (int y = 0; y < 16; ++y)
                W[y] = __float_as_uint(acc[(y >> 2) & 1][(y >> 1) & 1][y >> 3][r0 + (y & 1)]);
        };
        switch (u) {
        case 0: pick(std::integral_constant<int, 0>{}); break;
        case 1: pick(std::integral_constant<int, 1>{}); break;
        case 2: pick(std::integral_constant<int, 2>{}); break;
        case 3: pick(std::integral_constant<int, 3>{}); break;
        case 4: pick(std::integral_constant<int, 4>{}); break;
        case 5: pick(std::integral_constant<int, 5>{}); break;
        case 6: pick(std::integral_constant<int, 6>{}); break;
        default: pick(std::integral_constant<int, 7>{}); break;
        }
        const int at0 = x0 * c2l + x0 * (x0 - 1) / 2 * l0 + x0 * (x0 - 1) * (x0 - 2) / 6;
        const int at2 = x2 * c2l + x2 * (x2 - 1) / 2 * l0 + x2 * (x2 - 1) * (x2 - 2) / 6;
        const int tl = (h ? at2 : at0) * 32, til = tl + i * 32;                                // triplets (., ., l)
        const int pl = (c2l + x0 * l0 + x0 * (x0 - 1) / 2 + h * (2 * l0 + 2 * x0 + 1)) * 16;  // pairs (., l)
        bool pass = valid;
        // The table is built for the screening sum and, for the few that pass,
        // once more for the exact score: 27 cells of one genotype of i at a
        // time, so that the registers hold them next to the accumulators.
        #pragma unroll 1
        for (int exact = 0; exact < 2; ++exact) {
            int zero = 0, sh = T;
            asm volatile("" : "+s"(zero), "+s"(sh));  // (nothing of the loop is kept for the second time)
            const unsigned m0 = (1u << sh) - 1u;
            unsigned G[27], R[27];
            unsigned S = 0;
            long long num = t.score_const;
            unsigned long long dig = 0;
            auto score = [&](auto exact_pass) __attribute__((always_inline)) {
                if (exact) {
                    // (one passing combination at a time, a cell per lane)
                    for (unsigned long long m = __ballot(pass); m; m &= m - 1) {
                        const int src = __builtin_ctzll(m);
                        unsigned w = 0;
                        #pragma unroll
                        for (int x = 0; x < 27; ++x) {
                            const unsigned g = (unsigned)__builtin_amdgcn_readlane((int)G[x], src);
                            w = lane == x ? g : w;
                        }
                        const long long sum = wave_sum64(
                            cell_term_counted(d.tlog, (w & 0xffffu) >> kQScaleShift, w >> (16 + kQScaleShift)));
                        if (lane == src) num += sum;  // (the spare lanes' terms are 0)
                    }
                } else {
                    if (valid) S += (unsigned)screen_sum_packed<27>(G);
                    if constexpr (CHECK) {
                        constexpr int base = 27 * exact_pass.value;
                        #pragma unroll
                        for (int x = 0; x < 27; ++x)
                            dig += (unsigned long long)((G[x] & 0xffffu) >> kQScaleShift) * cell_weight(0, base + x) +
                                   (unsigned long long)(G[x] >> (16 + kQScaleShift)) * cell_weight(1, base + x);
                    }
                }
            };
            const v4u pil = qload(rP, pl + i * 16, zero);
            const v4u pij = qload(rP, i * 16, cij + zero), pik = qload(rP, i * 16, cik + zero);
            const v4u si = qload(rS, i * 16, zero);
            auto slab = [&](auto ac) __attribute__((always_inline)) {
                constexpr int a = ac.value;
                const v4u jl = qload(rT, til + 16 * a, cj + zero), kl = qload(rT, til + 16 * a, ck + zero);
                const v4u jk = qload(rTk, li + 16 * a, zero);
                #pragma unroll
                for (int y = 0; y < 8; ++y) {
                    const int b = y >> 2, c = (y >> 1) & 1, e = y & 1;
                    const unsigned w = W[8 * a + y];
                    G[9 * b + 3 * c + e] = (w & m0) | ((w >> sh) << (16 + kQScaleShift));
                }
                const unsigned p[4] = {jk[0], jk[1], jk[2], jk[3]}, q[4] = {jl[0], jl[1], jl[2], jl[3]};
                const unsigned s[4] = {kl[0], kl[1], kl[2], kl[3]};
                const unsigned x[2] = {pij[2 * a], pij[2 * a + 1]}, y[2] = {pik[2 * a], pik[2 * a + 1]};
                const unsigned z[2] = {pil[2 * a], pil[2 * a + 1]};
                complete(G, p, q, s, x, y, z, pack2(si[a], si[2 + a]));
                #pragma unroll
                for (int v = 0; v < 27; ++v) R[v] = a ? R[v] + G[v] : G[v];
                score(ac);
            };
            slab(std::integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            slab(std::integral_constant<int, 1>{});
            __builtin_amdgcn_sched_barrier(0);
            {
                const v4u k0 = qload(rT, tl, ck + j * 32 + zero), k1 = qload(rT, tl + 16, ck + j * 32 + zero);
                const v4u sl = qload(rS, l * 16, zero);
                const v4u pjl = qload(rP, pl, j * 16 + zero), pkl = qload(rP, pl, kk * 16 + zero);
                #pragma unroll
                for (int y = 0; y < 8; ++y) G[9 * (y >> 2) + 3 * ((y >> 1) & 1) + (y & 1)] = y < 4 ? k0[y] : k1[y - 4];
                const unsigned p[4] = {pjk[0], pjk[1], pjk[2], pjk[3]}, q[4] = {pjl[0], pjl[1], pjl[2], pjl[3]};
                const unsigned s[4] = {pkl[0], pkl[1], pkl[2], pkl[3]};
                const unsigned x[2] = {pack2(sj[0], sj[2]), pack2(sj[1], sj[3])};
                const unsigned y[2] = {pack2(sk[0], sk[2]), pack2(sk[1], sk[3])};
                const unsigned z[2] = {pack2(sl[0], sl[2]), pack2(sl[1], sl[3])};
                complete(G, p, q, s, x, y, z, nall);
                #pragma unroll
                for (int v = 0; v < 27; ++v) G[v] -= R[v];
                score(std::integral_constant<int, 2>{});
            }
            const int cc[4] = {i, j, kk, l};
            if (exact) {
                unsigned long long key = 0;
                #pragma unroll
                for (int z = 0; z < 4; ++z) key = (key << t.key_bits) | (unsigned long long)cc[z];
                tk_offer(tk, list, pass, num, key, gthr);
                sb = screen_bound(entry_bound(tk, gthr), t.score_const, d.shift, d.tq, 243);
                break;
            }
            if constexpr (CHECK) digest_add(tk, valid, combo_hash<4>(cc), dig);
            if constexpr (PILOT) {
                if (valid && (int)S > pilot_best) pilot_best = (int)S;
                break;
            }
            pass = valid && (int)S >= sb;
            if (!__ballot(pass)) break;
        }
    }
    if constexpr (PILOT) pilot_count(tk, t, pilot_best, 243);
}

// ---------------------------------------------------------------------------
// Persistent scan kernel: four independent waves per workgroup.  The
// workgroup pops chunks of work items from a device queue that runs over the
// concatenated item spaces of all tasks of the launch, in task order; each
// wave keeps its own best-K list and prefix-row slot in LDS.
// ---------------------------------------------------------------------------
// Register budget per instantiation: enough waves per SIMD to hide load
// latency; the accumulators (16 per prefix for order 3, 8 for order 2, 128
// for the matrix-core order-3 kernels: two classes of one middle SNP, or one
// accumulator for both classes of each of two; 128 for order 2 on the
// matrix cores too) set the floor.
template <int NP2, int NP3, int GK>
constexpr int scan_waves_per_eu() {
    return is_mfma_np(NP3) || NP2 == kNpMfma || GK == kXGk + 4 ? 2
                           : (GK >= 4 ? 2 : (GK == 3 ? 3 : (NP3 >= 8 ? 2 : (NP3 >= 4 ? 3 : (NP3 >= 2 ? 4 : (NP2 >= 8 ? 3 : 4))))));
}

// Items of a task's pilot pass: pilot_n consecutive ones from pilot_first.
EPI_DEV bool is_pilot_item(const Task &t, unsigned long long local) {
    return local >= t.pilot_first && local - t.pilot_first < (unsigned long long)t.pilot_n;
}

// CHECK: the checking instantiation, which also adds every scored
// combination to its task's completeness digest (the same results otherwise).
template <int NP2, int NP3, int GK, bool CHECK>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(scan_waves_per_eu<NP2, NP3, GK>())))
scan_persistent(const Task *__restrict__ tasks, int n_tasks, unsigned long long total_items,
                unsigned long long *__restrict__ queue, const unsigned long long *__restrict__ binom, int bstride,
                int tab_cap, int kmax, int stage_cap) {
    // dynamic LDS (the kernel has no static LDS, so the screening table
    // starts at LDS address 0 and a count's byte offset is its address):
    //   [tab_cap floats: screening table of the current dataset]
    //   [4 x kmax best-K lists][4 x stage_cap uint4: staged rows][2 x u64: queue chunk]
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    unsigned *s_tab = (unsigned *)s_dyn;
    const int wave = uni((int)(threadIdx.x >> 6));  // wave index in the workgroup (uniform per wave)
    const long long lists_off = ((long long)tab_cap * 4 + 15) & ~15LL;
    const long long stage_off = lists_off + (long long)4 * kmax * sizeof(Cand);
    Cand *s_list = (Cand *)(s_dyn + lists_off) + wave * kmax;
    v4u *s_stage = (v4u *)(s_dyn + stage_off) + wave * stage_cap;
    unsigned long long *s_chunk = (unsigned long long *)(s_dyn + stage_off + (long long)4 * stage_cap * sizeof(v4u));
    TopK tk;
    tk.n = 0;
    tk.K = 1;
    tk.cap = kmax;
    tk.wi = 0;
    tk.wn = 0;
    tk.wk = 0;
    tk.hist = nullptr;
    tk.added = 0;
    tk.top = -1;
    tk.dsum = 0;
    tk.dn = 0;
    tk.nohist = 0;
    tk.xl = 0;
    int cur = -1;
    long long gthr = (long long)0x8000000000000000ull;
    const uint32_t *loaded = nullptr;  // dataset whose screening table is in s_tab
    bool loaded_rev = false;           // both halves of it (else the first)
    // Guided self-scheduling, one queue atomic per chunk of 4 x `per` items for
    // the whole workgroup; the chunk shrinks with the remaining work (estimated
    // from the last chunk).  Wave w takes items first + w, first + w + 4, ...
    // For the kernels of orders 4-8 on the matrix cores, which score from the
    // LDS screening table alone, a chunk that runs over several tasks is handed
    // out task by task, each with its dataset's table; what is left of it stays
    // in s_chunk (in registers it cost order 4, M = 200, N = 2000 1.9 %).  The
    // others take the items past the first task without a table: loading one
    // for them, and the other schedule of their loops that came with it, cost
    // batches of six small scans 2-4 %.
    constexpr bool by_task = GK > kXGk;
    const unsigned long long n_waves = (unsigned long long)gridDim.x * 4;
    unsigned long long est = 0;
    if (by_task && threadIdx.x == 0) s_chunk[1] = 0;
    #pragma unroll 1
    for (;;) {
        if (threadIdx.x == 0) {
            // by_task: s_chunk holds what is left of the chunk
            unsigned long long c0 = by_task ? s_chunk[0] : 0, n = by_task ? s_chunk[1] : 0;
            if (n == 0) {
                unsigned long long per = (total_items - min(est, total_items)) / (2 * n_waves);
                per = per < 1 ? 1 : (per > 32 ? 32 : per);
                c0 = atomicAdd(queue, 4 * per);
                n = by_task ? min(4 * per, total_items - min(c0, total_items)) : per;
            }
            s_chunk[0] = c0;
            s_chunk[1] = n;
        }
        __syncthreads();
        // values read back from LDS are wave-uniform: keep them in SGPRs
        const unsigned long long first = rfl64(s_chunk[0]);
        const unsigned long long n = by_task ? (unsigned)uni((int)s_chunk[1]) : rfl64(s_chunk[1]);
        __syncthreads();
        if (first >= total_items) break;
        unsigned long long end = by_task ? first + n : min(first + 4 * n, total_items);
        if constexpr (!by_task) est = end;
        // the first task's dataset takes the LDS screening table if it fits
        {
            int lo = 0, hi = n_tasks - 1;
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if (tasks[mid].item_base <= first) lo = mid; else hi = mid - 1;
            }
            if constexpr (by_task) {
                const unsigned long long all = end;
                if (lo + 1 < n_tasks) end = min(end, tasks[lo + 1].item_base);
                if (threadIdx.x == 0) {
                    s_chunk[0] = end;
                    s_chunk[1] = all - end;
                }
                est = end;
            }
            const Task &T0 = tasks[lo];
            // the screening reads address the table from LDS address 0; the
            // mirrored half too for the kernels in the signed cell form, when
            // it fits
            const int ent_fwd = T0.ds.N + 1, ent_rev = 2 * T0.ds.N + 2;
            const bool want = (T0.variant == kF2 || T0.variant == kF2Fold || T0.variant == kF3 || T0.variant == kR4 ||
                               T0.variant == kR4M || T0.variant == kX) &&
                              ent_fwd <= tab_cap &&
                              (unsigned)(uintptr_t)(lu32 *)s_tab == 0u;
            const bool sgn = T0.variant == kF3 && is_mfma_np(T0.np);
            const bool rev = want && sgn && ent_rev <= tab_cap;  // read only in the signed cell form
            if (want && (loaded != T0.ds.itab || (rev && !loaded_rev))) {
                const int ent = rev ? ent_rev : ent_fwd;
                #pragma unroll 1
                for (int x = threadIdx.x; x < ent; x += blockDim.x) s_tab[x] = T0.ds.itab[x];
                __syncthreads();
                loaded = T0.ds.itab;
                loaded_rev = rev;
            }
            // the per-combination kernels: the exact n ln n table, n <= N
            const int ent_tl = 2 * (T0.ds.N + 1);
            const bool want_tl = (T0.variant == kGeneric || T0.variant == kSeg) && ent_tl <= tab_cap &&
                                 (unsigned)(uintptr_t)(lu32 *)s_tab == 0u;
            if (want_tl && loaded != (const uint32_t *)T0.ds.tlog) {
                const uint32_t *src = (const uint32_t *)T0.ds.tlog;
                #pragma unroll 1
                for (int x = threadIdx.x; x < ent_tl; x += blockDim.x) s_tab[x] = src[x];
                __syncthreads();
                loaded = src;
                loaded_rev = false;
            }
        }
        #pragma unroll 1
        for (unsigned long long item = first + wave; item < end; item += 4) {
            int lo = 0, hi = n_tasks - 1;
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if (tasks[mid].item_base <= item) lo = mid; else hi = mid - 1;
            }
            if (lo != cur) {
                if (cur >= 0 && !is_emit(tasks[cur].variant)) {
                    if (tk.n == tk.K && tk.wn > gthr && lane_id() == 0) atomicMax(tasks[cur].thr, bias(tk.wn));
                    tk_flush(tk, s_list, tasks[cur]);
                    if constexpr (CHECK) digest_flush(tk, tasks[cur]);
                }
                cur = lo;
                tk.n = 0;
                tk.K = tasks[cur].top_k;
                tk.hist = is_emit(tasks[cur].variant) ? nullptr : tasks[cur].hist;
                tk.added = 0;
                tk.top = -1;
                gthr = (long long)0x8000000000000000ull;
                if (!is_emit(tasks[cur].variant)) {
                    // a new task starts from the bound published so far
                    long long g = 0;
                    if (lane_id() == 0) g = load_thr(tasks[cur].thr);
                    gthr = (long long)rfl64((unsigned long long)g);
                }
            }
            const Task &T = tasks[cur];
            // the bound other waves have published: read before every item,
            // taken up after it (the item's own waits cover the load)
            long long g_pub = (long long)0x8000000000000000ull;
            if (!is_emit(T.variant) && lane_id() == 0) g_pub = load_thr(T.thr);
            const unsigned long long local = item - T.item_base + T.first_item;
            const bool lds = loaded != nullptr && T.ds.itab == loaded;
            const bool ldt = loaded != nullptr && (const uint32_t *)T.ds.tlog == loaded;
            // the pilot pass has counted the combinations of its items
            tk.nohist = is_pilot_item(T, local);
            switch (T.variant) {
            case kF2:
                if constexpr (NP2 == kNpMfma) {
                    if (q3_pack_fits(T.ds.ncls[0], T.ds.ncls[1])) {
                        if (lds) item_f2m<true, true, CHECK>(T, local, tk, s_list, gthr);
                        else item_f2m<false, true, CHECK>(T, local, tk, s_list, gthr);
                    } else {
                        if (lds) item_f2m<true, false, CHECK>(T, local, tk, s_list, gthr);
                        else item_f2m<false, false, CHECK>(T, local, tk, s_list, gthr);
                    }
                } else if constexpr (NP2 > 0) {
                    if (lds) item_f2<NP2, false, true, true, CHECK>(T, local, tk, s_list, gthr, s_stage, stage_cap);
                    else item_f2<NP2, false, false, true, CHECK>(T, local, tk, s_list, gthr, s_stage, stage_cap);
                }
                break;
            case kF2Emit:
                if constexpr (NP2 > 0 && NP2 != kNpMfma)
                    item_f2<NP2, true, false>(T, local, tk, s_list, gthr, s_stage, stage_cap);
                break;
            case kF2Fold:
                if constexpr (NP2 > 0 && NP2 != kNpMfma) {
                    if (lds) item_f2<NP2, true, true, true, CHECK>(T, local, tk, s_list, gthr, s_stage, stage_cap);
                    else item_f2<NP2, true, false, true, CHECK>(T, local, tk, s_list, gthr, s_stage, stage_cap);
                }
                break;
            case kF3Emit:
                if constexpr (NP3 == kNpMfma) {
                    if (q3_pack_fits(T.ds.ncls[0], T.ds.ncls[1]))
                        item_f3m<false, false, false, true, true>(T, local, tk, s_list, gthr, s_stage);
                    else item_f3m<false, false, false, false, true>(T, local, tk, s_list, gthr, s_stage);
                }
                break;
            case kR4:
                if constexpr (GK == 4) {
                    if (lds) item_r4<true, CHECK>(T, local, tk, s_list, gthr, binom, bstride);
                    else item_r4<false, CHECK>(T, local, tk, s_list, gthr, binom, bstride);
                }
                break;
            case kF3:
                if constexpr (is_mfma_np(NP3)) {
                    constexpr bool i8 = NP3 == kNpMfmaI8;
                    constexpr int nj = NP3 == kNpMfma2 ? 2 : 1;
                    auto run = [&](auto pk) __attribute__((always_inline)) {
                        constexpr bool PK = pk.value;
                        if (lds && loaded_rev)
                            item_f3m<true, true, i8, PK, false, CHECK, nj>(T, local, tk, s_list, gthr, s_stage);
                        else if (lds)
                            item_f3m<true, false, i8, PK, false, CHECK, nj>(T, local, tk, s_list, gthr, s_stage);
                        else item_f3m<false, false, i8, PK, false, CHECK, nj>(T, local, tk, s_list, gthr, s_stage);
                    };
                    // one accumulator for both classes where they fit
                    if constexpr (NP3 == kNpMfma2 || NP3 == kNpMfmaP) run(std::true_type{});
                    else if constexpr (i8 || NP3 == kNpMfmaS) run(std::false_type{});
                    else if (q3_pack_fits(T.ds.ncls[0], T.ds.ncls[1])) run(std::true_type{});
                    else run(std::false_type{});
                } else if constexpr (NP3 > 0) {
                    if (lds) item_f3<NP3, true, CHECK>(T, local, tk, s_list, gthr, s_stage, stage_cap);
                    else item_f3<NP3, false, CHECK>(T, local, tk, s_list, gthr, s_stage, stage_cap);
                }
                break;
            case kX:
                // (its dataset's table is always in LDS: the host takes kX and
                // kR4M only where it fits)
                if constexpr (GK > kXGk + 4)
                    if (lds) item_x<GK - kXGk, CHECK>(T, local, tk, s_list, gthr);
                break;
            case kR4M:
                if constexpr (GK == kXGk + 4)
                    if (lds) item_r4m<CHECK>(T, local, tk, s_list, gthr, s_stage);
                break;
            case kSeg:
                if constexpr (GK > kSegGk && GK < kXGk) {
                    uint32_t *slot = T.seg + (size_t)(blockIdx.x * 4 + wave) * (2 * kWave * pow3c(GK - kSegGk));
                    if (ldt) item_seg<GK - kSegGk, true, CHECK>(T, local, tk, s_list, gthr, binom, bstride, slot);
                    else item_seg<GK - kSegGk, false, CHECK>(T, local, tk, s_list, gthr, binom, bstride, slot);
                }
                break;
            default:
                if constexpr (GK > 0 && GK < kSegGk) {
                    if (ldt) item_generic<GK, true, CHECK>(T, local, tk, s_list, gthr, binom, bstride);
                    else item_generic<GK, false, CHECK>(T, local, tk, s_list, gthr, binom, bstride);
                }
                break;
            }
            if (!is_emit(T.variant)) {
                const long long g = (long long)rfl64((unsigned long long)g_pub);
                gthr = g > gthr ? g : gthr;
            }
            if (tk.added) {
                // combinations were counted: raise and publish the bound
                tk.added = 0;
                const long long hb = hist_bound(tk.hist, tk.K, tk.top);
                if (hb > gthr) {
                    gthr = hb;
                    if (lane_id() == 0) atomicMax(T.thr, bias(hb));
                }
            }
        }
        if (cur >= 0 && !is_emit(tasks[cur].variant) && tk.n == tk.K && tk.wn > gthr) {
            if (lane_id() == 0) atomicMax(tasks[cur].thr, bias(tk.wn));
            gthr = tk.wn;
        }
    }
    if (cur >= 0 && !is_emit(tasks[cur].variant)) {
        tk_flush(tk, s_list, tasks[cur]);
        if constexpr (CHECK) digest_flush(tk, tasks[cur]);
    }
}

typedef void (*ScanKernelFn)(const Task *, int, unsigned long long, unsigned long long *, const unsigned long long *,
                             int, int, int, int);

struct ScanKernelEntry {
    int np2, np3, gk;
    ScanKernelFn fn;
};

// Every instantiation of the scan kernel, in one table per CHECK value: this
// file is compiled twice, once as is (everything but the checking
// instantiations) and once with EPI_SCAN_CHECK defined (only those), so the
// two large sets of instantiations compile in parallel.
#define EPI_SCAN_KERNELS(CK)                                                                                     \
    {2, 0, 0, scan_persistent<2, 0, 0, CK>}, {4, 0, 0, scan_persistent<4, 0, 0, CK>},                             \
        {8, 0, 0, scan_persistent<8, 0, 0, CK>}, /* order 2 / pair sub-table */                                  \
        {kNpMfma, 0, 0, scan_persistent<kNpMfma, 0, 0, CK>}, /* order 2, matrix cores */                         \
        {0, 1, 0, scan_persistent<0, 1, 0, CK>}, {0, 2, 0, scan_persistent<0, 2, 0, CK>},                         \
        {0, 4, 0, scan_persistent<0, 4, 0, CK>}, {0, 8, 0, scan_persistent<0, 8, 0, CK>}, /* order 3 */          \
        {0, 0, 4, scan_persistent<0, 0, 4, CK>}, {0, 0, 5, scan_persistent<0, 0, 5, CK>}, /* per combination */ \
        {0, 0, 6, scan_persistent<0, 0, 6, CK>}, {0, 0, 7, scan_persistent<0, 0, 7, CK>},                         \
        {0, 0, 8, scan_persistent<0, 0, 8, CK>},                                                                   \
        {0, 0, kSegGk + 2, scan_persistent<0, 0, kSegGk + 2, CK>}, /* segmented (two-phase) */                   \
        {0, 0, kSegGk + 3, scan_persistent<0, 0, kSegGk + 3, CK>},                                                 \
        {0, 0, kSegGk + 4, scan_persistent<0, 0, kSegGk + 4, CK>},                                                 \
        {0, 0, kSegGk + 5, scan_persistent<0, 0, kSegGk + 5, CK>},                                                 \
        {0, 0, kSegGk + 6, scan_persistent<0, 0, kSegGk + 6, CK>},                                                 \
        {0, 0, kSegGk + 7, scan_persistent<0, 0, kSegGk + 7, CK>},                                                 \
        {0, 0, kSegGk + 8, scan_persistent<0, 0, kSegGk + 8, CK>},                                                 \
        {0, 0, kXGk + 4, scan_persistent<0, 0, kXGk + 4, CK>}, /* order 4 on the matrix cores */                 \
        {0, 0, kXGk + 5, scan_persistent<0, 0, kXGk + 5, CK>}, /* all cells on the matrix cores */               \
        {0, 0, kXGk + 6, scan_persistent<0, 0, kXGk + 6, CK>},                                                     \
        {0, 0, kXGk + 7, scan_persistent<0, 0, kXGk + 7, CK>},                                                     \
        {0, 0, kXGk + 8, scan_persistent<0, 0, kXGk + 8, CK>},                                                     \
        {0, kNpMfma, 0, scan_persistent<0, kNpMfma, 0, CK>}, /* order 3, matrix cores */                         \
        {0, kNpMfmaP, 0, scan_persistent<0, kNpMfmaP, 0, CK>},                                                    \
        {0, kNpMfmaS, 0, scan_persistent<0, kNpMfmaS, 0, CK>},                                                    \
        {0, kNpMfmaI8, 0, scan_persistent<0, kNpMfmaI8, 0, CK>},                                                  \
        {0, kNpMfma2, 0, scan_persistent<0, kNpMfma2, 0, CK>},

#ifdef EPI_SCAN_CHECK
static const ScanKernelEntry kScanKernelsCheck[] = {EPI_SCAN_KERNELS(true)};

ScanKernelFn find_scan_kernel_check(int np2, int np3, int gk) {
    for (const auto &e : kScanKernelsCheck)
        if (e.np2 == np2 && e.np3 == np3 && e.gk == gk) return e.fn;
    return nullptr;
}
#else
// ---------------------------------------------------------------------------
// Pilot pass of a launch group's scans (order 2, order 3 on the matrix cores,
// order 4 by reduced cells, orders 5-8 on the matrix cores), launched before
// its main launch.  Each task with pilot_n > 0
// has pilot_n consecutive pilot items (from the middle of its scan, sharing
// operand blocks in L2 as the main launch's items do), numbered from
// pilot_base in the pilot launch; a workgroup takes 4 of them (one per wave,
// never two tasks).  A wave passes over its item counting the best lower
// bound of its scores into the task's histogram (one count, or one per lane
// where the task has few pilot items: pilot_lanes); the last wave of
// a task reads the bound the histogram gives (the K-th best of lower bounds
// of distinct combinations is at most the task's final K-th best) and
// publishes it.  Every wave of the main launch starts from that bound, and
// the main launch does not count the pilot items again.  Same launch shape
// and LDS layout as the scan kernel.
// ---------------------------------------------------------------------------
template <int NP2, int NP3, int GK>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(scan_waves_per_eu<NP2, NP3, GK>())))
scan_pilot(const Task *__restrict__ tasks, int n_tasks, unsigned long long total, const unsigned long long *binom,
           int bstride, int tab_cap, int kmax, int stage_cap) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    unsigned *s_tab = (unsigned *)s_dyn;
    // the screening reads address the table from LDS address 0
    if ((unsigned)(uintptr_t)(lu32 *)s_tab != 0u) return;
    const int wave = uni((int)(threadIdx.x >> 6));
    const long long lists_off = ((long long)tab_cap * 4 + 15) & ~15LL;
    const long long stage_off = lists_off + (long long)4 * kmax * sizeof(Cand);
    Cand *s_list = (Cand *)(s_dyn + lists_off) + wave * kmax;
    v4u *s_stage = (v4u *)(s_dyn + stage_off) + wave * stage_cap;
    TopK tk;
    tk.n = 0;
    tk.K = 1;
    tk.cap = kmax;
    tk.wi = 0;
    tk.wn = 0;
    tk.wk = 0;
    tk.hist = nullptr;
    tk.added = 0;
    tk.top = -1;
    tk.dsum = 0;
    tk.dn = 0;
    tk.nohist = 0;
    tk.xl = 0;
    constexpr bool i8 = NP3 == kNpMfmaI8;
    constexpr int nj = NP3 == kNpMfma2 ? 2 : 1;
    const long long none = (long long)0x8000000000000000ull;
    const uint32_t *loaded = nullptr;
    bool loaded_rev = false;
    #pragma unroll 1
    for (unsigned long long g = (unsigned long long)blockIdx.x * 4; g < total; g += (unsigned long long)gridDim.x * 4) {
        int lo = 0, hi = n_tasks - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tasks[mid].pilot_base <= g) lo = mid; else hi = mid - 1;
        }
        const Task &T = tasks[lo];
        // the task's screening table (the host takes only tasks whose table
        // fits), with its mirrored half for the signed cell form of order 3
        const int ent_fwd = T.ds.N + 1, ent_rev = 2 * T.ds.N + 2;
        const bool rev = NP3 != 0 && ent_rev <= tab_cap;
        if (ent_fwd <= tab_cap && (loaded != T.ds.itab || (rev && !loaded_rev))) {
            __syncthreads();  // every wave is done with the previous table
            const int ent = rev ? ent_rev : ent_fwd;
            #pragma unroll 1
            for (int x = threadIdx.x; x < ent; x += blockDim.x) s_tab[x] = T.ds.itab[x];
            __syncthreads();
            loaded = T.ds.itab;
            loaded_rev = rev;
        }
        const unsigned long long local = T.pilot_first + (g - T.pilot_base) + (unsigned long long)wave;
        tk.hist = T.hist;
        tk.K = T.top_k;
        tk.top = -1;
        tk.added = 0;
        if (ent_fwd <= tab_cap && local < T.n_items) {
            if constexpr (GK == kXGk + 4) {
                item_r4m<false, true>(T, local, tk, s_list, none, s_stage);
            } else if constexpr (GK > kXGk) {
                item_x<GK - kXGk, false, true>(T, local, tk, s_list, none);
            } else if constexpr (GK == 4) {
                item_r4<true, false, true>(T, local, tk, s_list, none, binom, bstride);
            } else if constexpr (NP2 == kNpMfma) {
                if (q3_pack_fits(T.ds.ncls[0], T.ds.ncls[1])) item_f2m<true, true, false, true>(T, local, tk, s_list, none);
                else item_f2m<true, false, false, true>(T, local, tk, s_list, none);
            } else if constexpr (NP2 > 0) {
                item_f2<NP2, false, true, true, false, true>(T, local, tk, s_list, none, s_stage, stage_cap);
            } else {
                auto run = [&](auto pk) __attribute__((always_inline)) {
                    constexpr bool PK = pk.value;
                    if (rev) item_f3m<true, true, i8, PK, false, false, nj, true>(T, local, tk, s_list, none, s_stage);
                    else item_f3m<true, false, i8, PK, false, false, nj, true>(T, local, tk, s_list, none, s_stage);
                };
                if constexpr (NP3 == kNpMfma2 || NP3 == kNpMfmaP) run(std::true_type{});
                else if constexpr (i8 || NP3 == kNpMfmaS) run(std::false_type{});
                else if (q3_pack_fits(T.ds.ncls[0], T.ds.ncls[1])) run(std::true_type{});
                else run(std::false_type{});
            }
        }
        // the task's last pilot wave takes the bound
        __threadfence();
        unsigned prev = 0;
        if (lane_id() == 0) prev = atomicAdd(T.hist + kPilotWord, 1u);
        prev = (unsigned)__builtin_amdgcn_readfirstlane((int)prev);
        if (prev + 1 == (unsigned)T.pilot_n) {
            __threadfence();
            const long long hb = hist_bound_all(T.hist, T.top_k);
            if (hb != none && lane_id() == 0) atomicMax(T.thr, bias(hb));
        }
    }
}

// ---------------------------------------------------------------------------
// Best-K selection over a task's candidate buffer: one 1024-thread workgroup
// per task; candidates below the task's final threshold are dropped, the rest
// are bitonic-sorted in LDS (best first) chunk by chunk.
// ---------------------------------------------------------------------------
EPI_DEV void bitonic_sort_best_first(Cand *buf, int P) {
    for (int k = 2; k <= P; k <<= 1) {
        for (int jj = k >> 1; jj > 0; jj >>= 1) {
            for (int i = threadIdx.x; i < P; i += blockDim.x) {
                const int ixj = i ^ jj;
                if (ixj > i) {
                    const Cand a = buf[i], b = buf[ixj];
                    const bool up = (i & k) == 0;
                    const bool sw = up ? better(b.num, b.key, a.num, a.key) : better(a.num, a.key, b.num, b.key);
                    if (sw) {
                        buf[i] = b;
                        buf[ixj] = a;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// Best K of src[lo, hi) (entries below g dropped) into out[0, K), best first.
EPI_DEV void merge_range(const Cand *src, unsigned lo, unsigned hi, long long g, int K, Cand *buf, int *s_ctr,
                         Cand *out) {
    const Cand sentinel{(long long)0x8000000000000000ull, ~0ull};
    for (int i = threadIdx.x; i < kMergeSlots; i += blockDim.x) buf[i] = sentinel;
    __syncthreads();
    int fill = K;
    for (unsigned base = lo; base < hi; base += blockDim.x) {
        const unsigned i = base + threadIdx.x;
        Cand c = sentinel;
        bool keep = false;
        if (i < hi) {
            c = src[i];
            keep = c.num >= g;
        }
        const int n = __syncthreads_count(keep);
        if (fill + n > kMergeSlots) {
            int P = 64;
            while (P < fill) P <<= 1;
            bitonic_sort_best_first(buf, P);
            for (int x = K + threadIdx.x; x < kMergeSlots; x += blockDim.x) buf[x] = sentinel;
            fill = K;
            __syncthreads();
        }
        if (threadIdx.x == 0) *s_ctr = fill;
        __syncthreads();
        if (keep) buf[atomicAdd(s_ctr, 1)] = c;
        __syncthreads();
        fill += n;
    }
    int P = 64;
    while (P < fill) P <<= 1;
    bitonic_sort_best_first(buf, P);
    for (int r = threadIdx.x; r < K; r += blockDim.x) out[r] = buf[r];
}

// Stage 1: workgroup (part, task) reduces its slice of the task's candidate
// buffer to the best K.
__global__ void __launch_bounds__(1024) merge_part_kernel(const Task *__restrict__ tasks, Cand *__restrict__ parts) {
    __shared__ Cand buf[kMergeSlots];
    __shared__ int s_ctr;
    const Task &t = tasks[blockIdx.y];
    unsigned count = *t.cand_count;
    count = count < t.cand_cap ? count : t.cand_cap;
    const unsigned lo = (unsigned)((unsigned long long)count * blockIdx.x / gridDim.x);
    const unsigned hi = (unsigned)((unsigned long long)count * (blockIdx.x + 1) / gridDim.x);
    merge_range(t.cand, lo, hi, load_thr(t.thr), t.top_k, buf, &s_ctr,
                parts + ((long long)blockIdx.y * gridDim.x + blockIdx.x) * kMaxTopK);
}

// Stage 2: one workgroup per task merges the stage-1 lists.
__global__ void __launch_bounds__(1024) merge_final_kernel(const Task *__restrict__ tasks, const Cand *__restrict__ parts,
                                                           int n_parts, Cand *__restrict__ results) {
    __shared__ Cand buf[kMergeSlots];
    __shared__ int s_ctr;
    const Task &t = tasks[blockIdx.x];
    const int K = t.top_k;
    const Cand *src = parts + (long long)blockIdx.x * n_parts * kMaxTopK;
    // gather the n_parts lists (K entries each, stride kMaxTopK) behind the best K
    const Cand sentinel{(long long)0x8000000000000000ull, ~0ull};
    for (int i = threadIdx.x; i < kMergeSlots; i += blockDim.x) buf[i] = sentinel;
    __syncthreads();
    const long long g = load_thr(t.thr);
    int fill = K;
    if (K + n_parts * K <= kMergeSlots) {
        // all lists at once, every load in flight together; only entries
        // that reach the task's bound are kept, packed behind the first K
        // slots, so the sort covers those alone
        if (threadIdx.x == 0) s_ctr = K;
        __syncthreads();
        for (int i = threadIdx.x; i < n_parts * K; i += blockDim.x) {
            const int p = i / K, r = i - p * K;
            const Cand c = src[(long long)p * kMaxTopK + r];
            if (c.num >= g) buf[atomicAdd(&s_ctr, 1)] = c;
        }
        __syncthreads();
        fill = s_ctr;
    } else
    for (int p = 0; p < n_parts; ++p) {
        if (fill + K > kMergeSlots) {
            int P = 64;
            while (P < fill) P <<= 1;
            bitonic_sort_best_first(buf, P);
            for (int x = K + threadIdx.x; x < kMergeSlots; x += blockDim.x) buf[x] = sentinel;
            fill = K;
            __syncthreads();
        }
        for (int r = threadIdx.x; r < K; r += blockDim.x) {
            const Cand c = src[(long long)p * kMaxTopK + r];
            buf[fill + r] = c.num >= g ? c : sentinel;
        }
        __syncthreads();
        fill += K;
    }
    int P = 64;
    while (P < fill) P <<= 1;
    bitonic_sort_best_first(buf, P);
    for (int r = threadIdx.x; r < K; r += blockDim.x) results[(long long)blockIdx.x * kMaxTopK + r] = buf[r];
}

// ---------------------------------------------------------------------------
// Result tables: a workgroup per (result, task, 256 cells) decodes the
// combination, converts the score, and counts its part of the full 2 x 3^k
// table straight from the masks.  It stages the rows of the k SNPs (genotype
// 2 = valid & ~(row0 | row1)) in LDS, kFinWords 128-individual words at a
// time; the threads that share a cell (tables of fewer than 256 cells) take
// every parts-th word of it and add their counts in LDS.  One wave that
// walked all cells of a result from global memory left the device idle: 2600
// us for the ten 6561-cell tables of an order-8 scan, now 14; a hundred of
// order 5 81 and 11, of order 4 36 and 7, of order 3 at N = 4000 25 and 8.
// Bound by the latency of its few loads.
// ---------------------------------------------------------------------------
constexpr int kFinThreads = 256, kFinWords = 16;

__global__ void __launch_bounds__(kFinThreads)
finalize_kernel(const Task *__restrict__ tasks, const Cand *__restrict__ results,
                const ResultLayout *__restrict__ layout, char *__restrict__ out) {
    __shared__ v4u s_rows[kMaxBinomOrder * 3][kFinWords];
    __shared__ unsigned s_cnt[2][kFinThreads];
    const int ti = blockIdx.y;
    const int r = blockIdx.x;
    const Task &t = tasks[ti];
    const int K = t.top_k, k = t.order, tid = (int)threadIdx.x;
    int cells = 1;
    for (int u = 0; u < k; ++u) cells *= 3;
    const int x0 = (int)blockIdx.z * kFinThreads;
    if (r >= K || x0 >= cells) return;
    const DsView d = t.ds;
    char *blk = out + layout[ti].offset;
    int32_t *combos = (int32_t *)(blk + 16);
    float *scores = (float *)(blk + 16 + (long long)K * k * 4);
    uint32_t *tables = (uint32_t *)(blk + 16 + (long long)K * k * 4 + (long long)K * 4);
    const Cand *res = results + (long long)ti * kMaxTopK;
    const unsigned long long sentinel_key = ~0ull;
    if (r == 0 && blockIdx.z == 0) {
        const int nv = __syncthreads_count(tid < K && res[tid < K ? tid : 0].key != sentinel_key);
        if (tid == 0) {
            int32_t *hdr = (int32_t *)blk;
            hdr[0] = nv;
            hdr[1] = *d.err;  // nonzero: the dataset's last packing had invalid input
        }
    }
    const Cand e = res[r];
    if (e.key == sentinel_key) return;
    const int bits = t.key_bits;
    const unsigned long long kmask = (1ull << bits) - 1ull;
    auto snp = [&](int u) { return min((int)((e.key >> (bits * (k - 1 - u))) & kmask), d.Mp - 1); };
    if (blockIdx.z == 0) {
        if (tid < k) combos[r * k + tid] = snp(tid);
        if (tid == 0) scores[r] = (float)(ldexp((double)e.num, -d.shift) / (double)d.N);
    }
    const int here = min(cells - x0, kFinThreads);  // cells of this workgroup
    const int parts = kFinThreads / here, part = tid / here, xl = tid - part * here;
    int row[kMaxBinomOrder];  // the cell's row of each SNP
    #pragma unroll
    for (int u = kMaxBinomOrder - 1, y = x0 + xl; u >= 0; --u) {
        row[u] = 3 * u + y % 3;
        if (u < k) y /= 3;
    }
    s_cnt[0][tid] = 0;
    s_cnt[1][tid] = 0;
    gv4u *gm = (gv4u *)d.masks;
    const long long Mp = d.Mp;
    #pragma unroll 1
    for (int cl = 0; cl < 2; ++cl) {
        unsigned cnt = 0;
        #pragma unroll 1
        for (int w0 = 0; w0 < d.w4[cl]; w0 += kFinWords) {
            const int n = min(kFinWords, d.w4[cl] - w0);
            __syncthreads();
            for (int i = tid; i < k * kFinWords; i += kFinThreads) {
                const int u = i / kFinWords, w = i % kFinWords;
                if (w < n) {
                    const long long off = ((long long)d.wbase[cl] + w0 + w) * 2 * Mp + snp(u);
                    const v4u r0 = gm[off], r1 = gm[off + Mp];
                    s_rows[3 * u][w] = r0;
                    s_rows[3 * u + 1][w] = r1;
                    s_rows[3 * u + 2][w] = valid_mask(d.ncls[cl], w0 + w) & ~(r0 | r1);
                }
            }
            __syncthreads();
            if (part < parts)
                for (int w = part; w < n; w += parts) {
                    v4u X = s_rows[row[0]][w];
                    #pragma unroll
                    for (int u = 1; u < kMaxBinomOrder; ++u)
                        if (u < k) X &= s_rows[row[u]][w];
                    cnt += __builtin_popcount(X[0]) + __builtin_popcount(X[1]) + __builtin_popcount(X[2]) +
                           __builtin_popcount(X[3]);
                }
        }
        if (part < parts) atomicAdd(&s_cnt[cl][xl], cnt);
    }
    __syncthreads();
    for (int i = tid; i < 2 * here; i += kFinThreads) {
        const int cl = i / here, x = i - cl * here;
        tables[((long long)r * 2 + cl) * cells + x0 + x] = s_cnt[cl][x];
    }
}

// ---------------------------------------------------------------------------
// The three steps of Section 2 as separate passes over a list of
// combinations (n x K int32 SNP indices): genotype tables (Section 2.1),
// contingency tables (Section 2.2) and mutual information (Section 2.3,
// Equation 1).  An index outside [0, M) or a table that does not fit the
// dataset sets *err and leaves that combination's output unwritten (tables,
// rows) or NaN (MI).
// ---------------------------------------------------------------------------

// Genotype rows, depth-first over the genotypes of SNPs T .. K-1: p is the
// AND of the rows chosen for SNPs 0 .. T-1 (Algorithm 1's combine step adds
// one SNP per level); leaves are written W words apart.
template <int T, int K>
EPI_DEV void gt_walk(const unsigned (&r)[K][3], unsigned p, uint32_t *&o, int W) {
    if constexpr (T + 2 >= K) {
        #pragma unroll
        for (int g = 0; g < 3; ++g) {
            const unsigned q = p & r[T][g];
            if constexpr (T + 1 == K) {
                *o = q;
                o += W;
            } else {
                gt_walk<T + 1, K>(r, q, o, W);
            }
        }
    } else {
        #pragma unroll 1
        for (int g = 0; g < 3; ++g) {
            const unsigned rg = g == 0 ? r[T][0] : (g == 1 ? r[T][1] : r[T][2]);
            gt_walk<T + 1, K>(r, p & rg, o, W);
        }
    }
}

// Leading SNPs whose genotypes split a combination's rows over threads.
template <int K>
constexpr int gt_split() { return K >= 5 ? 2 : 0; }

// One thread per (combination, genotypes of its first gt_split SNPs, 32-bit
// word of the two classes' rows): rows [i][x][w], W = 4 (w4[0] + w4[1])
// words, class 0 first.
template <int K>
__global__ void __launch_bounds__(256) gt_kernel(DsView d, const int32_t *__restrict__ combos, unsigned long long n,
                                                 uint32_t *__restrict__ rows, int *__restrict__ err) {
    constexpr int P = pow3c(K), S = gt_split<K>(), PS = pow3c(S);
    const int W0 = 4 * d.w4[0], W = W0 + 4 * d.w4[1];
    const unsigned *m = (const unsigned *)d.masks;
    const long long Mp = d.Mp;
    const unsigned long long total = n * PS * (unsigned long long)W;
    for (unsigned long long id = blockIdx.x * 256ull + threadIdx.x; id < total;
         id += (unsigned long long)gridDim.x * 256ull) {
        const unsigned long long rest = id / (unsigned)W;
        const int w = (int)(id - rest * (unsigned)W);
        const unsigned long long i = rest / PS;
        const int sub = (int)(rest - i * PS);
        const int cl = w < W0 ? 0 : 1;
        const int wc = w - (cl ? W0 : 0);
        const long long g4 = d.wbase[cl] + wc / 4;
        const int left = d.ncls[cl] - 32 * wc;
        const unsigned vm = left >= 32 ? ~0u : (left <= 0 ? 0u : ((1u << left) - 1u));
        unsigned r[K][3];
        bool bad = false;
        #pragma unroll
        for (int t = 0; t < K; ++t) {
            int sn = combos[i * K + t];
            bad |= sn < 0 || sn >= d.M;
            sn = sn < 0 || sn >= d.M ? 0 : sn;
            r[t][0] = m[((g4 * 2 + 0) * Mp + sn) * 4 + (wc & 3)];
            r[t][1] = m[((g4 * 2 + 1) * Mp + sn) * 4 + (wc & 3)];
            r[t][2] = vm & ~(r[t][0] | r[t][1]);
        }
        if (bad) {
            atomicOr(err, 1);
            continue;
        }
        unsigned p = ~0u;
        #pragma unroll
        for (int t = 0, x = sub, div = PS / 3; t < S; ++t, div /= 3) {
            const int g = x / div;
            x -= g * div;
            p &= g == 0 ? r[t][0] : (g == 1 ? r[t][1] : r[t][2]);
        }
        uint32_t *o = rows + (i * P + (unsigned long long)sub * (P / PS)) * (unsigned long long)W + w;
        gt_walk<S, K>(r, p, o, W);
    }
}

// Both classes' 3^K cells of combination c (K = 2, 3).
template <int K>
EPI_DEV void count_small(const DsView &d, const int (&c)[K], unsigned (&acc)[2 * pow3c(K)]) {
    constexpr int P = pow3c(K);
    gv4u *gm = (gv4u *)d.masks;
    #pragma unroll
    for (int cl = 0; cl < 2; ++cl) {
        #pragma unroll
        for (int x = 0; x < P; ++x) acc[cl * P + x] = 0;
        long long off = (long long)d.wbase[cl] * 2 * d.Mp;
        for (int w = 0; w < d.w4[cl]; ++w, off += 2 * d.Mp) {
            const v4u vm = valid_mask(d.ncls[cl], w);
            v4u r[K][3];
            #pragma unroll
            for (int u = 0; u < K; ++u) {
                r[u][0] = gm[off + c[u]];
                r[u][1] = gm[off + d.Mp + c[u]];
                r[u][2] = vm & ~(r[u][0] | r[u][1]);
            }
            #pragma unroll
            for (int q = 0; q < 4; ++q)
                #pragma unroll
                for (int x = 0; x < P; ++x) {
                    const int g0 = x / (P / 3), g1 = x / (P / 9) % 3, g2 = x % 3;
                    unsigned v = r[0][g0][q] & r[1][g1][q];
                    if constexpr (K == 3) v &= r[K - 1][g2][q];
                    acc[cl * P + x] = bcnt_acc(v, acc[cl * P + x]);
                }
        }
    }
}

// Contingency tables, tables[i][class][x]: a one-wave workgroup takes 64
// combinations, one per lane, and (orders 4 up) one class and 81 cells of
// their tables; the counts go through LDS, half the lanes at a time, so that
// the stores are runs of whole table parts.  Bound by the counting's vector
// instructions; 100000 combinations of order 4, N = 2048: 92 us with a
// thread per table (three passes over the rows, every lane of a store in a
// line of its own), now 63.
template <int K>
constexpr int ct_units() { return K < 4 ? 1 : 2 * pow3c(K > 4 ? K - 4 : 0); }
template <int K>
__global__ void __launch_bounds__(64) ct_kernel(DsView d, const int32_t *__restrict__ combos, unsigned long long n,
                                                uint32_t *__restrict__ tables, int *__restrict__ err) {
    constexpr int U = ct_units<K>(), C = K < 4 ? 2 * pow3c(K) : 81, ROW = C | 1;  // an odd stride
    __shared__ unsigned slot[32 * ROW];
    const int lane = threadIdx.x;
    const unsigned long long units = (n + 63) / 64 * U;
    for (unsigned long long id = blockIdx.x; id < units; id += gridDim.x) {
        const unsigned long long i0 = id / U * 64;
        const int sub = (int)(id % U), cl = sub & 1, gi = sub >> 1;
        const bool live = i0 + lane < n;
        int c[K];
        bool bad = false;
        #pragma unroll
        for (int t = 0; t < K; ++t) {
            const int sn = live ? combos[(i0 + lane) * K + t] : 0;
            bad |= sn < 0 || sn >= d.M;
            c[t] = sn < 0 || sn >= d.M ? 0 : sn;
        }
        if (bad) atomicOr(err, 1);
        const unsigned long long keep = __ballot(live && !bad);
        unsigned acc[C];
        if constexpr (K < 4) {
            count_small<K>(d, c, acc);
        } else {
            int dig[K > 4 ? K - 4 : 1], x = gi;
            #pragma unroll
            for (int t = K - 5; t >= 0; --t) {
                dig[t] = x % 3;
                x /= 3;
            }
            g3_count<K>(d, c, dig, cl, acc);
        }
        // first word of this part in the group's tables
        uint32_t *out = tables + i0 * (2ull * pow3c(K)) + (K < 4 ? 0 : cl * pow3c(K) + gi * 81);
        #pragma unroll
        for (int half = 0; half < 2; ++half) {
            __syncthreads();
            if (lane >> 5 == half) {
                #pragma unroll
                for (int x = 0; x < C; ++x) slot[(lane & 31) * ROW + x] = acc[x];
            }
            __syncthreads();
            #pragma unroll 4
            for (int e = lane; e < 32 * C; e += 64) {
                const int t = e / C, x = e - t * C, at = 32 * half + t;
                if ((keep >> at) & 1) out[(unsigned long long)at * (2 * pow3c(K)) + x] = slot[t * ROW + x];
            }
        }
    }
}

// N * MI of a table by Equation 1 from the exact n ln n table, as the scans
// score a combination, then MI = that / 2^shift / N; a table whose classes do
// not sum to the dataset's class sizes is rejected.  LANES lanes per table,
// neighbouring cells in neighbouring lanes, BATCH cells a lane loaded at
// once; their sums (integers, so in any order) meet in a butterfly.  With LDT
// the n ln n table (n = 0 .. N) is staged at LDS address 0 first.  Bound by
// the latency of a wave's loads and look-ups: 100000 tables of order 4, N =
// 2048: 82 us with a table per lane staged in LDS (1563 waves), now 24.
//
// Lanes per table, and cells a lane: as few as hold a table of order 2 or 3
// (a million tables of order 2, N = 128, counted and scored: 107 us, with 16
// lanes a table 196).
constexpr int mi_lanes(int order) { return order == 2 ? 4 : (order == 3 ? 8 : (order <= 5 ? 16 : 64)); }
constexpr int mi_batch(int order) { return order == 2 ? 3 : (order == 3 ? 4 : 6); }

template <int LANES, int BATCH, bool LDT>
__global__ void __launch_bounds__(256) mi_kernel(DsView d, int P, long long score_const,
                                                 const uint32_t *__restrict__ tables, unsigned long long n,
                                                 double *__restrict__ mi, int *__restrict__ err) {
    extern __shared__ __attribute__((aligned(16))) unsigned char s_mi[];  // LDT: 2 (N + 1) words
    unsigned *s_t = (unsigned *)s_mi;
    bool at0 = false;  // the lookups address the staged table from LDS address 0
    if constexpr (LDT) {
        const unsigned *src = (const unsigned *)d.tlog;
        for (int x = threadIdx.x; x < 2 * (d.N + 1); x += blockDim.x) s_t[x] = src[x];
        __syncthreads();
        at0 = (unsigned)(uintptr_t)(lu32 *)s_t == 0u;
    }
    const int sub = threadIdx.x % LANES;
    const unsigned n_case = (unsigned)d.ncls[0], n_ctrl = (unsigned)d.ncls[1];
    for (unsigned long long i = (blockIdx.x * 256ull + threadIdx.x) / LANES; i < n;
         i += gridDim.x * (256ull / LANES)) {
        const uint32_t *T = tables + i * 2ull * (unsigned)P;
        long long num = 0;
        unsigned long long s0 = 0, s1 = 0;
        bool ok = true;
        for (int x0 = sub; x0 < P; x0 += LANES * BATCH) {
            unsigned n0[BATCH], n1[BATCH];
            #pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int x = x0 + u * LANES;
                n0[u] = x < P ? T[x] : 0u;
                n1[u] = x < P ? T[P + x] : 0u;
            }
            #pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const bool in = n0[u] <= n_case && n1[u] <= n_ctrl;
                ok &= in;
                s0 += n0[u];
                s1 += n1[u];
                const unsigned a = in ? n0[u] : 0u, b = in ? n1[u] : 0u;  // (an empty cell's term is 0)
                num += LDT && at0 ? cell_term_lds(a, b) : cell_term_counted(d.tlog, a, b);
            }
        }
        #pragma unroll
        for (int off = LANES / 2; off > 0; off >>= 1) {
            num += (long long)__shfl_xor((unsigned long long)num, off, LANES);
            s0 += __shfl_xor(s0, off, LANES);
            s1 += __shfl_xor(s1, off, LANES);
            ok &= __shfl_xor((int)ok, off, LANES) != 0;
        }
        if (sub == 0) {
            ok &= s0 == (unsigned long long)n_case && s1 == (unsigned long long)n_ctrl;
            mi[i] = ok ? ldexp((double)(score_const + num), -d.shift) / (double)d.N : __builtin_nan("");
            if (!ok) atomicOr(err, 1);
        }
    }
}

template <int K>
static hipError_t launch_function_k(int fn, hipStream_t st, const DsView &d, const int32_t *combos,
                                    unsigned long long n, void *out, int *err, int grid) {
    if (fn == 0) {
        hipLaunchKernelGGL(gt_kernel<K>, dim3(grid), dim3(256), 0, st, d, combos, n, (uint32_t *)out, err);
    } else {
        if constexpr (K < 2) return hipErrorInvalidValue;  // tables start at order 2
        else {
            const unsigned long long units = (n + 63) / 64 * ct_units<K>();
            hipLaunchKernelGGL(ct_kernel<K>, dim3((unsigned)(units < (1u << 20) ? units : 1u << 20)), dim3(64), 0, st, d,
                               combos, n, (uint32_t *)out, err);
        }
    }
    return hipGetLastError();
}

hipError_t launch_function(int fn, int order, hipStream_t st, const DsView &d, const int32_t *combos,
                           const uint32_t *tables, unsigned long long n, void *out, int *err, int grid,
                           long long score_const) {
    if (fn == 2) {
        // the exact table in LDS when it fits beside two workgroups per CU
        const size_t tl = (size_t)8 * (d.N + 1);
        const bool ldt = tl <= 64 * 1024;
        auto pick = [&](auto oc) {
            constexpr int L = mi_lanes(oc.value), B = mi_batch(oc.value);
            return ldt ? mi_kernel<L, B, true> : mi_kernel<L, B, false>;
        };
        auto *fn2 = order == 2   ? pick(std::integral_constant<int, 2>{})
                    : order == 3 ? pick(std::integral_constant<int, 3>{})
                    : order <= 5 ? pick(std::integral_constant<int, 5>{})
                                 : pick(std::integral_constant<int, 8>{});
        // as many workgroups as a CU holds at once (each stages the table)
        const unsigned long long want = (n * (unsigned)mi_lanes(order) + 255) / 256;
        const size_t per_cu = ldt ? (size_t)160 * 1024 / tl : 8;
        grid = (int)(want < (unsigned long long)grid * (per_cu < 8 ? per_cu : 8) ? want : grid * (per_cu < 8 ? per_cu : 8));
        hipLaunchKernelGGL(fn2, dim3(grid), dim3(256), ldt ? tl : 0, st, d, pow3i(order), score_const, tables, n,
                           (double *)out, err);
        return hipGetLastError();
    }
    switch (order) {
    case 1: return launch_function_k<1>(fn, st, d, combos, n, out, err, grid);
    case 2: return launch_function_k<2>(fn, st, d, combos, n, out, err, grid);
    case 3: return launch_function_k<3>(fn, st, d, combos, n, out, err, grid);
    case 4: return launch_function_k<4>(fn, st, d, combos, n, out, err, grid);
    case 5: return launch_function_k<5>(fn, st, d, combos, n, out, err, grid);
    case 6: return launch_function_k<6>(fn, st, d, combos, n, out, err, grid);
    case 7: return launch_function_k<7>(fn, st, d, combos, n, out, err, grid);
    case 8: return launch_function_k<8>(fn, st, d, combos, n, out, err, grid);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// Packing (Section 2.1): a wave takes kPackSnps SNPs of one 128-individual
// group of a class.  idx lists the input position of each class's individuals
// (cases first, in input order), so a SNP's 64 genotypes of a load lie close
// together, and a ballot over the wave is two words of its row.  Genotypes
// outside {0,1,2} raise *err.
//
// Bound by the latency of the byte loads, which go eight at a time: M = 1000,
// N = 4000 43 us with a thread per SNP and group (each byte of a row another
// load of the same thread, a line per lane), now 8; M = 4000 82 and 19.
// ---------------------------------------------------------------------------
constexpr int kPackSnps = 16;
__global__ void __launch_bounds__(256) pack_kernel(const uint8_t *__restrict__ geno, long long ld,
                                                   const int32_t *__restrict__ idx, DsView d,
                                                   v4u *__restrict__ masks, int *__restrict__ err) {
    const int nsb = (d.Mp + kPackSnps - 1) / kPackSnps;
    const long long wid = (long long)blockIdx.x * 4 + uni((int)(threadIdx.x >> 6));
    if (wid >= (long long)(d.w4[0] + d.w4[1]) * nsb) return;
    const int g4 = uni((int)(wid / nsb)), s0 = uni((int)(wid % nsb)) * kPackSnps, lane = lane_id();
    const int cl = g4 < d.w4[0] ? 0 : 1;
    const int32_t *cidx = idx + (cl == 0 ? 0 : d.ncls[0]);
    int bad = 0;
    unsigned at[2];
    bool in[2];
    #pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int pos = 128 * (g4 - d.wbase[cl]) + 64 * q + lane;
        in[q] = pos < d.ncls[cl];
        at[q] = in[q] ? (unsigned)cidx[pos] : 0u;
        if (at[q] >= (unsigned)d.N) {
            bad |= 8;
            in[q] = false;
            at[q] = 0;
        }
    }
    v4u r0 = {0u, 0u, 0u, 0u}, r1 = {0u, 0u, 0u, 0u};
    #pragma unroll
    for (int x0 = 0; x0 < kPackSnps; x0 += 4) {
        unsigned g[4][2];
        #pragma unroll
        for (int x = 0; x < 4; ++x) {
            const uint8_t *row = geno + (long long)min(s0 + x0 + x, d.M - 1) * ld;
            g[x][0] = row[at[0]];
            g[x][1] = row[at[1]];
        }
        #pragma unroll
        for (int x = 0; x < 4; ++x) {
            const bool real = s0 + x0 + x < d.M, mine = lane == x0 + x;  // (rows past the last SNP are zero)
            #pragma unroll
            for (int q = 0; q < 2; ++q) {
                const bool v = real && in[q];
                const unsigned long long b0 = __ballot(v && g[x][q] == 0u), b1 = __ballot(v && g[x][q] == 1u);
                bad |= v && g[x][q] > 2u ? 1 : 0;
                r0[2 * q] = mine ? (unsigned)b0 : r0[2 * q];
                r0[2 * q + 1] = mine ? (unsigned)(b0 >> 32) : r0[2 * q + 1];
                r1[2 * q] = mine ? (unsigned)b1 : r1[2 * q];
                r1[2 * q + 1] = mine ? (unsigned)(b1 >> 32) : r1[2 * q + 1];
            }
        }
    }
    if (lane < kPackSnps && s0 + lane < d.Mp) {
        masks[((long long)g4 * 2 + 0) * d.Mp + s0 + lane] = r0;
        masks[((long long)g4 * 2 + 1) * d.Mp + s0 + lane] = r1;
    }
    if (bad) atomicOr(err, bad);
}

__global__ void singles_kernel(DsView d, uint32_t *__restrict__ single) {
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= d.Mp * 2) return;
    const int s = tid >> 1, cl = tid & 1;
    gv4u *gm = (gv4u *)d.masks;
    unsigned n0 = 0, n1 = 0;
    long long off = (long long)d.wbase[cl] * 2 * d.Mp;
    for (int w = 0; w < d.w4[cl]; ++w, off += 2 * d.Mp) {
        const v4u r0 = gm[off + s], r1 = gm[off + d.Mp + s];
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            n0 += __builtin_popcount(r0[q]);
            n1 += __builtin_popcount(r1[q]);
        }
    }
    single[(s * 2 + cl) * 2 + 0] = n0;
    single[(s * 2 + cl) * 2 + 1] = n1;
    // again in the signed cell form of the matrix-core order-3 kernels
    const unsigned B4 = 4u * q3_bias(d.N);
    single[(d.Mp + s) * 4 + cl * 2 + 0] = (n0 << kQScaleShift) - B4;
    single[(d.Mp + s) * 4 + cl * 2 + 1] = (n1 << kQScaleShift) - B4;
}

// Matrix-core operand copies of the genotype-0/1 rows: one thread per (SNP,
// genotype, step, half); an entry is three 32-individual mask words, one per
// bit plane.
EPI_DEV unsigned spread8(unsigned b) {  // bit t of a byte to bit 4 t
    b = (b | (b << 12)) & 0x000f000fu;
    b = (b | (b << 6)) & 0x03030303u;
    return (b | (b << 3)) & 0x11111111u;
}

EPI_DEV v4u planes_entry(unsigned p0, unsigned p1, unsigned p2) {
    v4u e;
    #pragma unroll
    for (int q = 0; q < 4; ++q)
        e[q] = spread8((p0 >> (8 * q)) & 0xffu) | (spread8((p1 >> (8 * q)) & 0xffu) << 1) |
               (spread8((p2 >> (8 * q)) & 0xffu) << 2);
    return e;
}

__global__ void qpack_kernel(DsView d, v4u *__restrict__ qa, v4u *__restrict__ qb) {
    const long long S3 = d.xs;
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= (long long)d.Mp * 2 * S3 * 2) return;
    const int s = (int)(tid % d.Mp);
    long long rest = tid / d.Mp;
    const int g = (int)(rest & 1);
    rest >>= 1;
    const int h = (int)(rest & 1);
    const long long step = rest >> 1;
    const int half = 2 * (int)step + h, c = half < d.xh0 ? 0 : 1;
    const int w0 = 3 * (half - (c ? d.xh0 : 0));  // the entry's first 32-bit word within the class
    const unsigned *m = (const unsigned *)d.masks;
    unsigned word[3];
    #pragma unroll
    for (int p = 0; p < 3; ++p) {
        const int w = w0 + p;
        word[p] = (w >> 2) < d.w4[c] ? m[(((long long)(d.wbase[c] + (w >> 2)) * 2 + g) * d.Mp + s) * 4 + (w & 3)] : 0u;
    }
    const v4u out = planes_entry(word[0], word[1], word[2]);
    qa[((long long)(s >> 4) * S3 + step) * 64 + 32 * h + 2 * (s & 15) + g] = out;
    qb[(((long long)(s >> 5) * 2 + g) * S3 + step) * 64 + 32 * h + (s & 31)] = out;
}

// Cell rows of the dataset's single SNPs and pairs (layout in
// epi_internal.hpp): one thread per (SNP or pair; step; half).
__global__ void __launch_bounds__(256) xrows_kernel(DsView d, v4u *__restrict__ out, unsigned long long total) {
    const int H0 = x_halves(d.ncls[0]), S3 = x_steps(d.ncls[0], d.ncls[1]);
    const unsigned long long id = blockIdx.x * 256ull + threadIdx.x;
    if (id >= total) return;
    const int h = (int)(id & 1);
    const unsigned long long rest = id >> 1;
    const unsigned long long sub = rest / (unsigned)S3;
    const int s = (int)(rest - sub * (unsigned)S3);
    v4u *o;
    int snp[2] = {0, 0}, n = 0;
    if (sub < (unsigned)d.M) {
        n = 1;
        snp[0] = (int)sub;
        o = out + ((long long)snp[0] * S3 + s) * (kXSingle / 16) + 4 * h;
    } else {
        n = 2;
        const unsigned p = (unsigned)(sub - (unsigned)d.M);
        int y = (int)((1.0f + sqrtf(1.0f + 8.0f * (float)p)) * 0.5f);
        while ((unsigned)y * (unsigned)(y - 1) / 2u > p) --y;
        while ((unsigned)y * (unsigned)(y + 1) / 2u <= p) ++y;
        snp[1] = y;
        snp[0] = (int)(p - (unsigned)y * (unsigned)(y - 1) / 2u);
        o = out + ((long long)d.M * S3 * kXSingle + ((long long)p * S3 + s) * kXPair) / 16 + 9 * h;
    }
    const int half = 2 * s + h, cl = half < H0 ? 0 : 1;
    const int w0 = 3 * (half - (cl ? H0 : 0));  // first 32-individual word in the class
    const unsigned *m = (const unsigned *)d.masks;
    unsigned g[2][3][3];  // [SNP][genotype][plane]
    #pragma unroll
    for (int p = 0; p < 3; ++p) {
        const int w = w0 + p, left = d.ncls[cl] - 32 * w;
        const unsigned vm = left >= 32 ? ~0u : (left <= 0 ? 0u : ((1u << left) - 1u));
        #pragma unroll
        for (int u = 0; u < 2; ++u) {
            unsigned g0 = 0, g1 = 0;
            if (left > 0) {
                const long long at = ((long long)(d.wbase[cl] + (w >> 2)) * 2 * d.Mp + snp[u]) * 4 + (w & 3);
                g0 = m[at];
                g1 = m[at + 4ll * d.Mp];
            }
            g[u][0][p] = g0;
            g[u][1][p] = g1;
            g[u][2][p] = vm & ~(g0 | g1);
        }
    }
    auto put = [&](int cell, unsigned p0, unsigned p1, unsigned p2) { o[cell] = planes_entry(p0, p1, p2); };
    if (n == 1) {
        #pragma unroll
        for (int a = 0; a < 3; ++a) put(a, g[0][a][0], g[0][a][1], g[0][a][2]);
    } else {
        #pragma unroll
        for (int a = 0; a < 3; ++a)
            #pragma unroll
            for (int b = 0; b < 3; ++b)
                put(3 * a + b, g[0][a][0] & g[1][b][0], g[0][a][1] & g[1][b][1], g[0][a][2] & g[1][b][2]);
    }
}

// Integer operand copies: one thread per (SNP, genotype, 32-individual step,
// half); each 16-individual half word becomes 16 bytes, 1 (qa8) or 4 (qb8)
// per set bit.
__global__ void qpack8_kernel(DsView d, v4u *__restrict__ qa8, v4u *__restrict__ qb8) {
    const long long KS = d.ks8[0] + d.ks8[1];
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= (long long)d.Mp * 2 * KS * 2) return;
    const int s = (int)(tid % d.Mp);
    long long rest = tid / d.Mp;
    const int g = (int)(rest & 1);
    rest >>= 1;
    const int h = (int)(rest & 1);
    const long long step = rest >> 1;
    const int c = step < d.ks8[0] ? 0 : 1;
    const int widx = (int)(step - (c == 0 ? 0 : d.ks8[0]));  // 32-bit word within the class
    unsigned word = 0;
    if ((widx >> 2) < d.w4[c]) {
        gv4u *gm = (gv4u *)d.masks;
        word = gm[((long long)(d.wbase[c] + (widx >> 2)) * 2 + g) * d.Mp + s][widx & 3];
    }
    const unsigned half = word >> (16 * h);
    v4u out;
    #pragma unroll
    for (int k = 0; k < 4; ++k) {
        unsigned x = 0;
        #pragma unroll
        for (int t = 0; t < 4; ++t) x |= ((half >> (4 * k + t)) & 1u) << (8 * t);
        out[k] = x;
    }
    qa8[((long long)(s >> 4) * KS + step) * 64 + 32 * h + 2 * (s & 15) + g] = out;
    qb8[(((long long)(s >> 5) * 2 + g) * KS + step) * 64 + 32 * h + (s & 31)] = out << 2;  // 4 per set bit
}

// Class index map: idx[0 .. n_case) = input positions of the cases in input
// order, idx[n_case .. N) = those of the controls.  One 1024-thread
// workgroup, the first kernel of a packing: it clears the dataset's error
// word, then a phenotype outside {0,1} raises bit 2 and a number of cases
// other than n_case bit 4 (some index then falls outside its class).
__global__ void __launch_bounds__(1024) classidx_kernel(const uint8_t *__restrict__ pheno, int N, int n_case,
                                                        int32_t *__restrict__ idx, int *__restrict__ err) {
    __shared__ int s_wave[2][16];  // cases of each wave of a chunk, two chunks in turn
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    if (tid == 0) *err = 0;
    __syncthreads();
    int bc = 0;  // cases before the chunk
    for (int base = 0, k = 0; base < N; base += 1024, k ^= 1) {
        const int s = base + tid;
        int f = 0;
        if (s < N) {
            const unsigned v = pheno[s];
            f = v == 1u ? 1 : 0;
            if (v > 1u) atomicOr(err, 2);
        }
        const unsigned long long m = __ballot(f);
        if (lane == 0) s_wave[k][wave] = (int)__popcll(m);
        __syncthreads();
        int before = (int)lane_prefix(m), all = 0;  // cases before s within the chunk, all of them
        #pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int n = s_wave[k][w];
            before += w < wave ? n : 0;
            all += n;
        }
        if (s < N) {
            if (f) {
                if (bc + before < n_case) idx[bc + before] = s;
                else atomicOr(err, 4);
            } else {
                const int pos = n_case + (base - bc) + (tid - before);
                if (pos < N) idx[pos] = s;
                else atomicOr(err, 4);
            }
        }
        bc += all;
    }
}

// After a merge: the best K (results) become the first entries of each
// task's candidate buffer, so later launches of the same task (serving
// rounds) add to a compact list.
__global__ void reseed_kernel(const Task *__restrict__ tasks, const Cand *__restrict__ results) {
    const Task &t = tasks[blockIdx.x];
    const Cand *res = results + (long long)blockIdx.x * kMaxTopK;
    int n = 0;
    for (int r = 0; r < t.top_k; ++r) n += res[r].key != ~0ull ? 1 : 0;
    for (int r = threadIdx.x; r < n; r += blockDim.x) t.cand[r] = res[r];
    if (threadIdx.x == 0) *t.cand_count = (unsigned)n;
}

// Work-item descriptor table of one shape (kinds and layouts in
// epi_internal.hpp), written by one workgroup: the groups go 1024 at a time,
// a scan of their sizes gives each its offset, and each thread writes the
// items of its group.  out holds exactly the sum of the group sizes, which
// the host counts with the same functions.
__global__ void __launch_bounds__(1024) items_kernel(int kind, int M, int np, unsigned long long *__restrict__ out) {
    __shared__ unsigned long long s_scan[1024];
    __shared__ unsigned long long s_base;
    const long long G = item_groups(kind, M, np);
    if (threadIdx.x == 0) s_base = 0;
    __syncthreads();
    for (long long g0 = 0; g0 < G; g0 += 1024) {
        const long long g = g0 + threadIdx.x;
        ItemGroup gr{0, 1, 0, 0};
        if (g < G) gr = item_group(kind, M, np, g);
        s_scan[threadIdx.x] = gr.count;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const unsigned long long v = (int)threadIdx.x >= off ? s_scan[threadIdx.x - off] : 0ull;
            __syncthreads();
            s_scan[threadIdx.x] += v;
            __syncthreads();
        }
        const unsigned long long start = s_base + s_scan[threadIdx.x] - gr.count;
        for (unsigned long long t = 0; t < gr.count; ++t) out[start + t] = item_at(gr, t);
        __syncthreads();
        if (threadIdx.x == 1023) s_base += s_scan[1023];
        __syncthreads();
    }
}

// kX, kR4M: first work item of each entry and the end (x_items summed), one
// workgroup.
__global__ void __launch_bounds__(1024) xbase_kernel(int order, int M, int u, unsigned long long *__restrict__ out) {
    __shared__ unsigned long long s_scan[1024];
    __shared__ unsigned long long s_base;
    if (threadIdx.x == 0) s_base = 0;
    __syncthreads();
    const int L = x_entries(order, M);
    for (int l0 = 0; l0 <= L; l0 += 1024) {
        const int l = l0 + (int)threadIdx.x;
        const unsigned long long n = l < L ? x_items(order, M, u, l) : 0ull;
        s_scan[threadIdx.x] = n;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            const unsigned long long v = (int)threadIdx.x >= off ? s_scan[threadIdx.x - off] : 0ull;
            __syncthreads();
            s_scan[threadIdx.x] += v;
            __syncthreads();
        }
        if (l <= L) out[l] = s_base + s_scan[threadIdx.x] - n;
        __syncthreads();
        if (threadIdx.x == 1023) s_base += s_scan[1023];
        __syncthreads();
    }
}

// Bytes carried to device memory in a kernel's arguments (the task array of
// a launch sequence that may not copy from host memory).
struct StoreChunk {
    unsigned char b[kStoreChunkBytes];
};

__global__ void store_kernel(StoreChunk payload, int n, unsigned char *__restrict__ dst) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = payload.b[i];
}

// A result block (layout in epi_internal.hpp) copied to separate buffers of
// the caller: combinations, scores and (tables non-null) tables of the
// n_valid results; *n receives n_valid, or -1 when the dataset's last packing
// had invalid input.
__global__ void scatter_kernel(const char *__restrict__ block, int top_k, int order, int32_t *__restrict__ combos,
                               float *__restrict__ scores, uint32_t *__restrict__ tables, int32_t *__restrict__ n) {
    const int32_t *hdr = (const int32_t *)block;
    const long long nv = hdr[0];
    const long long nc = nv * order, ns = nv, nt = tables ? nv * 2 * pow3c(order) : 0;
    const int32_t *src_c = (const int32_t *)(block + 16);
    const float *src_s = (const float *)(block + 16 + (long long)top_k * order * 4);
    const uint32_t *src_t = (const uint32_t *)(block + 16 + (long long)top_k * order * 4 + (long long)top_k * 4);
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nc + ns + nt;
         i += (long long)gridDim.x * blockDim.x) {
        if (i < nc) combos[i] = src_c[i];
        else if (i < nc + ns) scores[i - nc] = src_s[i - nc];
        else tables[i - nc - ns] = src_t[i - nc - ns];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *n = hdr[1] ? -1 : (int32_t)nv;
}

// Counters of a launch sequence: queues, candidate counts, thresholds.
__global__ void init_counters_kernel(unsigned long long *queues, int nq, unsigned *cand_counts,
                                     unsigned long long *thrs, int n_tasks, unsigned *hist) {
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid < nq) queues[tid] = 0;
    if (tid < n_tasks) {
        cand_counts[tid] = 0;
        thrs[tid] = 0;  // bias(INT64_MIN)
    }
    if (hist && tid < (long long)n_tasks * kHistWords) hist[tid] = 0;
}

// ---------------------------------------------------------------------------
// Host-side launchers (called by the runtime).
// ---------------------------------------------------------------------------
static const ScanKernelEntry kScanKernels[] = {EPI_SCAN_KERNELS(false)};

ScanKernelFn find_scan_kernel_check(int np2, int np3, int gk);  // the EPI_SCAN_CHECK build of this file

size_t scan_lds_bytes(int tab_cap, int kmax, int stage_cap) {
    return (((size_t)tab_cap * 4 + 15) & ~(size_t)15) + (size_t)4 * kmax * sizeof(Cand) +
           (size_t)4 * stage_cap * sizeof(v4u) + 2 * sizeof(unsigned long long);
}

ScanKernelFn find_scan_kernel(int np2, int np3, int gk) {
    for (const auto &e : kScanKernels)
        if (e.np2 == np2 && e.np3 == np3 && e.gk == gk) return e.fn;
    return nullptr;
}

// grid = number of 4-wave workgroups; check: the checking instantiation
hipError_t launch_scan(int np2, int np3, int gk, int grid, hipStream_t st, const Task *tasks, int n_tasks,
                       unsigned long long total_items, unsigned long long *queue, const unsigned long long *binom,
                       int bstride, int tab_cap, int kmax, int stage_cap, bool check) {
    ScanKernelFn fn = check ? find_scan_kernel_check(np2, np3, gk) : find_scan_kernel(np2, np3, gk);
    if (!fn) return hipErrorInvalidValue;
    const size_t lds = scan_lds_bytes(tab_cap, kmax, stage_cap);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(4 * kWave), lds, st, tasks, n_tasks, total_items, queue, binom, bstride,
                       tab_cap, kmax, stage_cap);
    return hipGetLastError();
}

hipError_t launch_pilot(int np2, int np3, int gk, int grid, hipStream_t st, const Task *tasks, int n_tasks,
                        unsigned long long total, const unsigned long long *binom, int bstride, int tab_cap, int kmax,
                        int stage_cap) {
    void (*fn)(const Task *, int, unsigned long long, const unsigned long long *, int, int, int, int) =
        gk == 4               ? scan_pilot<0, 0, 4>
        : gk == kXGk + 4      ? scan_pilot<0, 0, kXGk + 4>
        : gk == kXGk + 5      ? scan_pilot<0, 0, kXGk + 5>
        : gk == kXGk + 6      ? scan_pilot<0, 0, kXGk + 6>
        : gk == kXGk + 7      ? scan_pilot<0, 0, kXGk + 7>
        : gk == kXGk + 8      ? scan_pilot<0, 0, kXGk + 8>
        : np3 == kNpMfma      ? scan_pilot<0, kNpMfma, 0>
        : np3 == kNpMfmaP     ? scan_pilot<0, kNpMfmaP, 0>
        : np3 == kNpMfmaS     ? scan_pilot<0, kNpMfmaS, 0>
        : np3 == kNpMfmaI8    ? scan_pilot<0, kNpMfmaI8, 0>
        : np3 == kNpMfma2     ? scan_pilot<0, kNpMfma2, 0>
        : np2 == kNpMfma      ? scan_pilot<kNpMfma, 0, 0>
        : np2 == 2            ? scan_pilot<2, 0, 0>
        : np2 == 4            ? scan_pilot<4, 0, 0>
        : np2 == 8            ? scan_pilot<8, 0, 0>
                              : nullptr;
    if (!fn) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(4 * kWave), scan_lds_bytes(tab_cap, kmax, stage_cap), st, tasks, n_tasks,
                       total, binom, bstride, tab_cap, kmax, stage_cap);
    return hipGetLastError();
}

hipError_t launch_merge(int n_tasks, hipStream_t st, const Task *tasks, Cand *parts, Cand *results) {
    hipLaunchKernelGGL(merge_part_kernel, dim3(kMergeParts, n_tasks), dim3(1024), 0, st, tasks, parts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(merge_final_kernel, dim3(n_tasks), dim3(1024), 0, st, tasks, (const Cand *)parts, kMergeParts,
                       results);
    return hipGetLastError();
}

hipError_t scan_attributes(int np2, int np3, int gk, int *vgprs, int *lds_bytes) {
    ScanKernelFn fn = find_scan_kernel(np2, np3, gk);
    if (!fn) return hipErrorInvalidValue;
    hipFuncAttributes a;
    hipError_t e = hipFuncGetAttributes(&a, (const void *)fn);
    if (e != hipSuccess) return e;
    *vgprs = a.numRegs;
    *lds_bytes = (int)a.sharedSizeBytes;
    return hipSuccess;
}

hipError_t launch_finalize(int n_tasks, int max_k, int max_order, hipStream_t st, const Task *tasks,
                           const Cand *results, const ResultLayout *layout, char *out) {
    const int z = (pow3i(max_order) + kFinThreads - 1) / kFinThreads;
    hipLaunchKernelGGL(finalize_kernel, dim3(max_k, n_tasks, z), dim3(kFinThreads), 0, st, tasks, results, layout, out);
    return hipGetLastError();
}

hipError_t launch_init_counters(hipStream_t st, unsigned long long *queues, int nq, unsigned *cand_counts,
                                unsigned long long *thrs, int n_tasks, unsigned *hist) {
    long long n = nq > n_tasks ? nq : n_tasks;
    if (hist && (long long)n_tasks * kHistWords > n) n = (long long)n_tasks * kHistWords;
    hipLaunchKernelGGL(init_counters_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, queues, nq,
                       cand_counts, thrs, n_tasks, hist);
    return hipGetLastError();
}

hipError_t launch_xrows(hipStream_t st, const DsView &d, v4u *out) {
    const int S3 = x_steps(d.ncls[0], d.ncls[1]);
    const unsigned long long n = ((unsigned)d.M + (unsigned long long)d.M * (d.M - 1) / 2) * S3 * 2;
    hipLaunchKernelGGL(xrows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d, out, n);
    return hipGetLastError();
}

hipError_t launch_items(hipStream_t st, int kind, int M, int np, unsigned long long *out) {
    if (kind >= kItemsX) {
        hipLaunchKernelGGL(xbase_kernel, dim3(1), dim3(1024), 0, st, kind - kItemsX, M, np, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(items_kernel, dim3(1), dim3(1024), 0, st, kind, M, np, out);
    return hipGetLastError();
}

hipError_t launch_store(hipStream_t st, const void *src, size_t bytes, void *dst) {
    for (size_t off = 0; off < bytes; off += kStoreChunkBytes) {
        StoreChunk c;
        const size_t n = bytes - off < (size_t)kStoreChunkBytes ? bytes - off : (size_t)kStoreChunkBytes;
        memcpy(c.b, (const char *)src + off, n);
        hipLaunchKernelGGL(store_kernel, dim3(1), dim3(256), 0, st, c, (int)n, (unsigned char *)dst + off);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_scatter(hipStream_t st, const char *block, int top_k, int order, int32_t *combos, float *scores,
                          uint32_t *tables, int32_t *n) {
    const long long items = (long long)top_k * (order + 1 + (tables ? 2 * pow3i(order) : 0));
    const int grid = (int)((items + 255) / 256 + 1 < 1024 ? (items + 255) / 256 + 1 : 1024);
    hipLaunchKernelGGL(scatter_kernel, dim3(grid), dim3(256), 0, st, block, top_k, order, combos, scores, tables, n);
    return hipGetLastError();
}

hipError_t launch_reseed(int n_tasks, hipStream_t st, const Task *tasks, const Cand *results) {
    hipLaunchKernelGGL(reseed_kernel, dim3(n_tasks), dim3(64), 0, st, tasks, results);
    return hipGetLastError();
}

hipError_t launch_pack(hipStream_t st, const uint8_t *geno, long long ld, const int32_t *idx, const DsView &d,
                       v4u *masks, int *err) {
    const long long n = (long long)(d.w4[0] + d.w4[1]) * ((d.Mp + kPackSnps - 1) / kPackSnps);  // waves
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, geno, ld, idx, d, masks, err);
    return hipGetLastError();
}

hipError_t launch_classidx(hipStream_t st, const uint8_t *pheno, int N, int n_case, int32_t *idx, int *err) {
    hipLaunchKernelGGL(classidx_kernel, dim3(1), dim3(1024), 0, st, pheno, N, n_case, idx, err);
    return hipGetLastError();
}

hipError_t launch_qpack(hipStream_t st, const DsView &d, v4u *qa, v4u *qb) {
    const long long n = (long long)d.Mp * 2 * d.xs * 2;
    hipLaunchKernelGGL(qpack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d, qa, qb);
    return hipGetLastError();
}

hipError_t launch_qpack8(hipStream_t st, const DsView &d, v4u *qa8, v4u *qb8) {
    const long long n = (long long)d.Mp * 2 * (d.ks8[0] + d.ks8[1]) * 2;
    hipLaunchKernelGGL(qpack8_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d, qa8, qb8);
    return hipGetLastError();
}

hipError_t launch_singles(hipStream_t st, const DsView &d, uint32_t *single) {
    const int n = d.Mp * 2;
    hipLaunchKernelGGL(singles_kernel, dim3((n + 255) / 256), dim3(256), 0, st, d, single);
    return hipGetLastError();
}

#endif  // EPI_SCAN_CHECK

}  // namespace epi
