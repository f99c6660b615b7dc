// CSR <-> CMRS conversion kernels and the CSR validity check (gfx950).
//
// CSR -> CMRS follows Sec. 3 and 4 of Koza et al. (arXiv:1203.2946):
//   StripPtr[j] = RowPtr[j*height], StripPtr[strips] = nnz;
//   word[k] = (ColInd[k] << bits) | (row(k) mod height);
//   optionally every strip reordered by (column, RowInStrip), ties in CSR
//   order (Sec. 4, fourth optimisation).
// CMRS -> CSR is the inverse: per-row counts inside a strip give RowPtr (no
// global scan is needed, a strip's entries are exactly its rows' entries), and
// a stable scatter by RowInStrip restores row order.  One wave takes the
// whole strips of 32 consecutive rows and streams their entries (contiguous)
// with coalesced loads, counting, then scattering; at height 1 the
// conversion is a plain copy.
//
// Work split of CSR -> CMRS.  Without the reorder, entries keep their
// places: one wave takes the whole strips of 32 consecutive rows and streams
// their entries with coalesced loads, stepping through the row pointers to
// find each entry's row.  With the reorder, the main kernel gives each strip a
// group of G lanes (64/G strips per wave) and each lane up to E = 8 entries,
// all loaded before any is used, so a wave keeps 64*E entries of traffic in
// flight.  The row of an entry comes from a binary search over the strip's row
// pointers, which sit one per lane of the group (cross-lane reads, no memory
// traffic).
//
// Reorder: a strip of canonical CSR is `height` runs (its rows) that are
// already sorted by column, and within a strip (column, RowInStrip) order is
// the order of the packed words.  The runs are merged pairwise, log2(height)
// levels, in LDS: each entry counts the keys of the partner run below its own
// (binary search) and moves to its place in the merged run.  Keys are
// (word << 32 | position in strip), unique, so the result is the stable order.
// Matrices of longer strips (a mean of 450 to 3800 entries) give each strip to a
// workgroup, which merges the same way or sorts by buckets of columns.  Strips that
// are longer than that, or short ones whose rows are not sorted, go to a list in the workspace: strips of up to 1024
// entries are sorted by one wave (run merge, or a bitonic network for unsorted
// rows); of longer ones, few long rows among short ones are streamed against the
// short rows' sorted words, others are merged by a workgroup in LDS as far as that
// holds them, in the workspace beyond, unsorted rows by a bitonic network.
#include <limits.h>

#include <type_traits>

#include "cmrs_device.hpp"
#include "cmrs_internal.hpp"
#include "merge_search.hpp"

namespace cmrs {

constexpr int kConvWaves = 4;
constexpr int kConvThreads = kConvWaves * kWave;
// Threads of the listed-strip sort that are resident: its LDS and registers allow
// 1024 per CU, 256 CUs.
constexpr int kListThreads = 1024 * 256;

__global__ void set_ints_kernel(int32_t* p, int32_t n, int32_t v) {
    if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < n) p[threadIdx.x] = v;
}

// Largest t with rp_t <= e, where lane base+t holds rp_t = RowPtr[first row of
// the strip + t] (INT_MAX for rows the strip does not have): the RowInStrip of
// entry e (empty rows are skipped because their rp_t repeats).  All lanes of
// the wave must be active.
template <int HB>
__device__ inline int row_in_strip(int myrp, int e, int base) {
    int lo = 0;
#pragma unroll
    for (int step = HB / 2; step >= 1; step >>= 1) {
        const int v = __shfl(myrp, base + lo + step);
        if (v <= e) lo += step;
    }
    return lo;
}

struct StripRows {
    int r0, nr, myrp, s0, s1;
};

// Row pointers of strip `strip` spread over the lanes of the whole wave.
__device__ inline StripRows load_strip_rows(int strip, int rows, int height, const int* __restrict__ row_ptr,
                                            int lane) {
    StripRows s;
    s.r0 = strip * height;
    s.nr = min(height, rows - s.r0);
    s.myrp = lane <= s.nr ? row_ptr[s.r0 + lane] : INT_MAX;
    s.s0 = __shfl(s.myrp, 0);
    s.s1 = __shfl(s.myrp, s.nr);
    return s;
}

__device__ inline int pow2_at_least(int n) {
    int p = 1;
    while (p < n) p <<= 1;
    return n == 0 ? 0 : p;
}

// Ascending bitonic network over keys k[0..P), P a power of two, run by
// `nthreads` threads numbered `tid`; `sync` orders the passes.  The keys are
// elements base .. base + P of a larger network's: bitonic_merge runs the
// passes of one size from stride `from` down.
template <typename Key, typename Sync>
__device__ inline void bitonic_merge(Key* k, int P, int size, int from, int base, int tid, int nthreads, Sync sync) {
    for (int stride = from; stride > 0; stride >>= 1) {
        for (int t = tid; t < P / 2; t += nthreads) {
            const int i = ((t & ~(stride - 1)) << 1) | (t & (stride - 1));
            const int l = i + stride;
            const bool up = ((base + i) & size) == 0;
            const uint64_t a = k[i], b = k[l];
            if ((a > b) == up) {
                k[i] = b;
                k[l] = a;
            }
        }
        sync();
    }
}
template <typename Key, typename Sync>
__device__ inline void bitonic_sort(Key* k, int P, int base, int tid, int nthreads, Sync sync) {
    for (int size = 2; size <= P; size <<= 1) bitonic_merge(k, P, size, size >> 1, base, tid, nthreads, sync);
}

// ------------------------------------------------------------------ whole-wave paths

// Pointers into LDS.  Functions that are not inlined take their LDS this way:
// with a generic pointer their accesses are flat ones, which are slower, and
// whose address before the instruction's own offset has to lie in the LDS
// aperture, which an index with a negative part need not keep.
typedef __attribute__((address_space(3))) uint32_t LdsWord;
typedef __attribute__((address_space(3))) uint64_t LdsKey;
typedef __attribute__((address_space(3))) int LdsInt;

// The word at an LDS address: a signed number, so that one word before the
// first stays below it.
__device__ inline int lds_address(const LdsWord* p) { return static_cast<int>(reinterpret_cast<uintptr_t>(p)); }
__device__ inline uint32_t lds_word(int address) { return *reinterpret_cast<const LdsWord*>(static_cast<uintptr_t>(address)); }

// Largest value of v over the wave.
__device__ inline int wave_max(int v) {
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off));
    return uniform(v);
}

// Merge of the row runs of strips held in registers, G lanes per strip, slot u
// of lane q holding entry q + G*u: words (col << bits | RowInStrip) in wd and
// their current place in the strip in pos.  LDS
// buffers A and B (the group's words by place, A filled on entry) alternate
// per level, level k merging the runs of 2^k rows pairwise (ONE: every level
// leaves its words in A, the last one too, so that A ends sorted); the words of
// different runs never tie (their RowInStrip fields differ), so
// an entry's place after a level is its rank in its own run plus the number
// of partner-run words below it.  On return pos holds each entry's place in
// the sorted strip.  The caller has made A and rt visible to the wave; row_max
// bounds the rows' lengths and n_max the strips' (both uniform, n_max <= G*E).
//
// Bound by VALU issue: with a search loop per entry the sorted conversion of
// 2^20 Poisson(16) rows at height 8 issued VALU instructions on 99 % of its
// 154 us, 363 of them per 64 entries.  So the search is a fixed number of
// steps for the whole wave, four instructions each, on LDS addresses: cur is
// the last word known to be below the entry's own (one before the run at
// first), and a step moves it on by a power of two where that stays in the
// run and below.  A step may read past its run: up to 4 kWave E bytes past B,
// which the buffer holds behind the last wave's slice (merge_pad); with CLAMP it
// reads no further than one word before A.  sync orders the levels.  Conversions
// (fp64, us): 2^20 Poisson(16) rows at height 8 150 -> 131, at height 16 184 ->
// 141; 27-point stencil of 10^6 rows at height 8 233 -> 178; 5-point stencil in
// bf16 at height 32 70 -> 49.
template <int HB, int G, int E, bool MAIN, bool ONE = false, bool CLAMP = false, typename Sync>
__device__ inline void merge_runs_regs(LdsWord* A, LdsWord* B, const LdsInt* rt, const uint32_t (&wd)[E],
                                       int (&pos)[E], int umax, bool go, int n, int q, int row_max, int n_max,
                                       Sync sync) {
    const auto merge_level = [&](int k) {
        if (k > 0) sync();
        const int longest = min(row_max << k, n_max);
        const int top = merge_first_step(longest);
        const int first = lds_address(A) - 4;
        // Level k of the slots u0 .. u0 + C - 1, their searches in step.
        const auto level = [&](auto count, int u0) {
            constexpr int C = decltype(count)::value;
            int start[C], cur[C], last[C];
#pragma unroll
            for (int v = 0; v < C; ++v) {
                const int partner = (static_cast<int>(wd[u0 + v]) & (HB - 1) & -(1 << k)) ^ (1 << k);
                start[v] = cur[v] = first + 4 * rt[partner];
                last[v] = first + 4 * rt[partner + (1 << k)];
            }
            for (int step = top; step > 3; step >>= 1) {
                uint32_t x[C];
#pragma unroll
                for (int v = 0; v < C; ++v) x[v] = lds_word(CLAMP ? min(cur[v] + step, last[v]) : cur[v] + step);
#pragma unroll
                for (int v = 0; v < C; ++v) cur[v] = merge_step(cur[v], step, last[v], x[v] < wd[u0 + v]);
            }
#pragma unroll
            for (int v = 0; v < C; ++v) {
                const int u = u0 + v;
                // The partner's words in front of a left run's entry move it
                // back; a right run's entry already stands behind all of them.
                const bool right = (wd[u] >> k) & 1u;
                pos[u] += (cur[v] - (right ? last[v] : start[v])) >> 2;
                if (!ONE && (2 << k) < HB && go && q + G * u < n) B[pos[u]] = wd[u];
            }
        };
        // Four slots at a time; what is left of them in the main kernel by a set
        // of its own size (an empty slot costs as much as a full one).
#pragma unroll
        for (int u0 = 0; u0 < E; u0 += 4) {
            const int left = umax - u0;
            if (left <= 0) break;
            if (!MAIN || left >= 4)
                level(std::integral_constant<int, 4>(), u0);
            else if (left == 3)
                level(std::integral_constant<int, 3>(), u0);
            else if (left == 2)
                level(std::integral_constant<int, 2>(), u0);
            else
                level(std::integral_constant<int, 1>(), u0);
        }
        if constexpr (ONE) {
            sync();
#pragma unroll
            for (int u = 0; u < E; ++u)
                if (go && q + G * u < n) A[pos[u]] = wd[u];
        } else {
            LdsWord* tmp = A;
            A = B;
            B = tmp;
        }
    };
    // The listed strips' kernel runs a level's code a few times per wave only,
    // so there the levels share it: unrolled, it was mostly instruction fetch.
    if constexpr (MAIN) {
#pragma unroll
        for (int k = 0; (1 << k) < HB; ++k) merge_level(k);
    } else {
#pragma unroll 1
        for (int k = 0; (1 << k) < HB; ++k) merge_level(k);
    }
}


// 64-bit words a search may read past the last wave's slice of kWave*E.
constexpr int merge_pad(int E) { return kWave * E / 2; }

// Unsorted rows, bucketed by column (see from_csr_tall_kernel): most keys of a
// bucket, beyond which the strip goes through a bitonic network.
constexpr int kBucketMax = 64;

// Places (pos) in the sorted strip of the n words of a strip with unsorted rows
// that a wave of the group kernel holds, slot u of lane q entry q + kWave*u: the
// bucketing of from_csr_tall_kernel in the wave's LDS slice (A, B: kWave*E words
// each), where A takes the words by bucket and B the buckets' starts and the
// words' places in the strip, which order equal words.  Returns false, pos
// unchanged, if a bucket is too full.  Listed, as they are below kBucketHeight, such
// strips go through the list kernel's bitonic networks: 6*10^6 entries in strips of
// 430 to 448, height 16, 292 us against 60 to 82 here.
typedef __attribute__((address_space(3))) uint16_t LdsHalf;
template <int E>
__device__ inline bool bucket_places(LdsWord* A, LdsWord* B, const uint32_t (&wd)[E], int (&pos)[E], int n, int bits,
                                     int lane) {
    constexpr int NB = kWave * E / 4, PER = NB / kWave;
    static_assert(NB + 1 + kWave * E / 2 <= kWave * E && PER * kWave == NB, "starts and places fit B");
    LdsHalf* const place = reinterpret_cast<LdsHalf*>(B + kWave * E / 2);
    int cmin = INT_MAX, cmax = -1;
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if (lane + kWave * u < n) {
            cmin = min(cmin, static_cast<int>(wd[u] >> bits));
            cmax = max(cmax, static_cast<int>(wd[u] >> bits));
        }
    }
    cmin = -wave_max(-cmin);
    cmax = wave_max(cmax);
    int nbk = 1;
    while (nbk < NB && nbk * 4 < n) nbk <<= 1;
    const uint64_t scale = (static_cast<uint64_t>(nbk) << 32) / (static_cast<uint64_t>(cmax - cmin) + 1u);
#pragma unroll
    for (int k = 0; k < PER; ++k) B[lane * PER + k] = 0u;
    wave_lds_sync();
    uint32_t bs[E];  // bucket << 16 | slot in bucket
#pragma unroll
    for (int u = 0; u < E; ++u) {
        bs[u] = 0u;
        if (lane + kWave * u < n) {
            const uint32_t c = (wd[u] >> bits) - static_cast<uint32_t>(cmin);
            const uint32_t bk = static_cast<uint32_t>((static_cast<uint64_t>(c) * scale) >> 32);
            bs[u] = (bk << 16) | __hip_atomic_fetch_add(B + bk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    wave_lds_sync();
    int cnt[PER], sum = 0, most = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        cnt[k] = static_cast<int>(B[lane * PER + k]);
        sum += cnt[k];
        most = max(most, cnt[k]);
    }
    if (wave_max(most) > kBucketMax) return false;
    int run = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int t = __shfl_up(run, off);
        if (lane >= off) run += t;
    }
    run -= sum;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        B[lane * PER + k] = static_cast<uint32_t>(run);
        run += cnt[k];
    }
    if (lane == kWave - 1) B[NB] = static_cast<uint32_t>(run);
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < E; ++u) {
        const int i = lane + kWave * u;
        if (i < n) {
            const int at = static_cast<int>(B[bs[u] >> 16] + (bs[u] & 0xffffu));
            A[at] = wd[u];
            place[at] = static_cast<uint16_t>(i);
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < E; ++u) {
        const int i = lane + kWave * u;
        if (i < n) {
            int p = static_cast<int>(B[bs[u] >> 16]);
            const int end = static_cast<int>(B[(bs[u] >> 16) + 1]);
            for (int k = p; k < end; ++k) p += A[k] < wd[u] || (A[k] == wd[u] && place[k] < i) ? 1 : 0;
            pos[u] = p;
        }
    }
    return true;
}

// From this height (next power of two) on, a strip with unsorted rows is bucketed by
// the wave of the group kernel that holds it; lower ones go through the network.
constexpr int kBucketHeight = 16;

// Each entry and its value (read again) to its place.
template <int E, typename ET>
__device__ inline void scatter_strip(const uint32_t (&wd)[E], const int (&pos)[E], int umax, int n, int s0,
                                     const ET* __restrict__ val_in, uint32_t* __restrict__ col_word,
                                     ET* __restrict__ val_out, int lane) {
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if (u >= umax) break;
        const int i = lane + kWave * u;
        if (i < n && static_cast<unsigned>(pos[u]) < static_cast<unsigned>(n)) {
            col_word[s0 + pos[u]] = wd[u];
            val_out[s0 + pos[u]] = val_in[s0 + i];
        }
    }
}

// A strip of at most kWave*E entries with unsorted rows, its words in registers
// (slot u of lane l: entry l + kWave*u): with BUCKET by buckets of columns, else or
// where they don't divide, by a bitonic network over (word, position) keys.
template <int E, bool BUCKET, typename ET>
__device__ inline void sort_unsorted(LdsKey* slice, const uint32_t (&wd)[E], int n, int s0, int bits,
                                     const ET* __restrict__ val_in, uint32_t* __restrict__ col_word,
                                     ET* __restrict__ val_out, int lane) {
    wave_lds_sync();  // the slice's words are read above; buckets or keys overwrite them
    if constexpr (BUCKET) {
        LdsWord* A = reinterpret_cast<LdsWord*>(slice);
        int pos[E];
        if (bucket_places<E>(A, A + kWave * E, wd, pos, n, bits, lane)) {
            scatter_strip<E, ET>(wd, pos, uniform((n + kWave - 1) / kWave), n, s0, val_in, col_word, val_out, lane);
            return;
        }
        wave_lds_sync();
    }
    const int P = pow2_at_least(n);
#pragma unroll
    for (int u = 0; u < E; ++u) {
        const int i = lane + kWave * u;
        if (i < n)
            slice[i] = (static_cast<uint64_t>(wd[u]) << 32) | static_cast<uint32_t>(i);
        else if (i < P)
            slice[i] = ~0ull;
    }
    wave_lds_sync();
    bitonic_sort(slice, P, 0, lane, kWave, [] { wave_lds_sync(); });
    for (int i = lane; i < n; i += kWave) {
        const uint64_t kk = slice[i];
        col_word[s0 + i] = static_cast<uint32_t>(kk >> 32);
        val_out[s0 + i] = val_in[s0 + static_cast<int>(static_cast<uint32_t>(kk))];
    }
}

// sort_unsorted for the group kernel's wave, whose one strip's words lie in its
// slice; out of line, and the last thing that wave does: its registers would spill
// those of the kernel around it (Poisson(15) rows, fp64, height 12, 1.5*10^6 rows:
// 174 -> 271 us).
template <int E, typename ET>
__device__ __attribute__((noinline)) void sort_held_strip(LdsKey* slice, int n, int s0, int bits,
                                                          const ET* __restrict__ val_in,
                                                          uint32_t* __restrict__ col_word, ET* __restrict__ val_out,
                                                          int lane) {
    const LdsWord* A = reinterpret_cast<const LdsWord*>(slice);
    uint32_t wd[E];
#pragma unroll
    for (int u = 0; u < E; ++u) wd[u] = lane + kWave * u < n ? A[lane + kWave * u] : 0u;
    sort_unsorted<E, true, ET>(slice, wd, n, s0, bits, val_in, col_word, val_out, lane);
}

// Sorted conversion of one strip of at most kWave*E entries by the whole wave,
// words in registers (slot u of lane l: entry l + kWave*u), in its LDS slice
// of kWave*E 64-bit words: rows sorted by column, a merge of the row runs
// (merge_runs_regs), then each entry and its value (read again) to its place;
// otherwise a bitonic network over (word, position) keys.  KERNEL tells the callers
// apart: with a copy of its own, each list kernel has it inlined (a call there costs
// 7 us), while the group kernels share one out of line.
template <int HB, int E, int KERNEL, typename ET>
__device__ inline void sort_strip_mid(int strip, int rows, int height, int bits, const int* __restrict__ row_ptr,
                                      const int* __restrict__ col_ind, const ET* __restrict__ val_in,
                                      uint32_t* __restrict__ col_word, ET* __restrict__ val_out, LdsKey* slice,
                                      LdsInt* rt, int lane) {
    const StripRows sr = load_strip_rows(strip, rows, height, row_ptr, lane);
    const int n = sr.s1 - sr.s0;
    const int umax = uniform((n + kWave - 1) / kWave);
    const uint32_t mask = (1u << bits) - 1u;
    LdsWord* A = reinterpret_cast<LdsWord*>(slice);
    LdsWord* B = A + kWave * E;
    uint32_t wd[E];
    int pos[E];
#pragma unroll
    for (int u = 0; u < E; ++u) {
        wd[u] = 0u;
        pos[u] = lane + kWave * u;
        if (u < umax) {
            const int i = lane + kWave * u;
            const int r = row_in_strip<HB>(sr.myrp, sr.s0 + i, 0);
            if (i < n) {
                wd[u] = (static_cast<uint32_t>(col_ind[sr.s0 + i]) << bits) | static_cast<uint32_t>(r);
                A[i] = wd[u];
            }
        }
    }
    if (lane <= HB) rt[lane] = lane < sr.nr ? sr.myrp - sr.s0 : n;
    wave_lds_sync();
    bool bad = false;
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if (u >= umax) break;
        const int i = lane + kWave * u;
        if (i + 1 < n) {
            const uint32_t nw = A[i + 1];
            if ((nw & mask) == (wd[u] & mask) && (nw >> bits) < (wd[u] >> bits)) bad = true;
        }
    }
    if (ballot(bad) == 0ull) {
        const int next_row = __shfl_down(sr.myrp, 1);
        const int row_max = wave_max(lane < sr.nr ? next_row - sr.myrp : 0);
        merge_runs_regs<HB, kWave, E, false>(A, B, rt, wd, pos, umax, true, n, lane, row_max, n,
                                                 [] { wave_lds_sync(); });
        scatter_strip<E, ET>(wd, pos, umax, n, sr.s0, val_in, col_word, val_out, lane);
    } else {
        sort_unsorted<E, false, ET>(slice, wd, n, sr.s0, bits, val_in, col_word, val_out, lane);
    }
    wave_lds_sync();
}

// ------------------------------------------------------------------ group kernels

__device__ inline uint64_t group_mask(int gbase, int G) {
    return G == kWave ? ~0ull : (((1ull << G) - 1ull) << gbase);
}

// Number of per-lane slots any group of the wave uses: ceil(max n / G)
// (wave-uniform), so the slot loops stop at the longest strip of the wave.
template <int G>
__device__ inline int used_slots(int n) {
    int m = n;
#pragma unroll
    for (int off = kWave / 2; off >= G; off >>= 1) m = max(m, __shfl_xor(m, off));
    return uniform((m + G - 1) / G);
}

// Strips past a group's capacity of at most this many entries are sorted by
// the group kernel's wave itself, longer ones listed for the list kernels.
// (Listing every such strip spreads the work but costs a wave per strip;
// measured on the skewed 2*10^6-row workload, sorted conversion at height
// 2/4/8: 256/275/298 us inline up to 512 entries, 243/257/273 us up to 256,
// 383/289/272 us listing all; the benchmark matrix is unchanged.)
constexpr int kInlineSortMax = 256;

// CSR -> CMRS with the reorder, for strips of at most G*E entries, G lanes
// per strip.  Writes strip_ptr too.  Longer strips of at most kInlineSortMax
// entries (and no more than kWave*E), and strips with unsorted rows as short,
// are sorted by the whole wave afterwards in the wave's LDS slice; longer ones
// go to the workspace lists (ws_count[0] / ws_small: at most kWaveSortCap
// entries; ws_count[1] / ws_big: longer).  No output may alias an input.
template <int HB, int G, int E, typename ET>
__global__ __launch_bounds__(kConvThreads) __attribute__((amdgpu_waves_per_eu(8))) void from_csr_group_kernel(
    int rows, int strips, int height, int bits, int nnz, const int* __restrict__ row_ptr,
    const int* __restrict__ col_ind, const ET* __restrict__ val_in, int* __restrict__ strip_ptr,
    uint32_t* __restrict__ col_word, ET* __restrict__ val_out, int* __restrict__ ws_count,
    int* __restrict__ ws_small, int* __restrict__ ws_big) {
    static_assert(G >= HB && G <= kWave && G >= 2, "group width");
    constexpr int NG = kWave / G;
    constexpr int CAP = G * E;
    __shared__ uint64_t lds[kConvWaves * kWave * E + merge_pad(E)];
    __shared__ int rowtab[kConvWaves][NG * (HB + 1)];
    const int lane = lane_id();
    const int wave = uniform(static_cast<int>(threadIdx.x) / kWave);
    LdsKey* const slice = (LdsKey*)lds + wave * kWave * E;
    const int strip0 = (xcd_logical_block(blockIdx.x, gridDim.x) * kConvWaves + wave) * NG;
    if (strip0 >= strips) return;
    const int g = lane / G, q = lane % G, gbase = g * G;
    const int strip = strip0 + g;
    const bool valid = strip < strips;
    const int r0 = strip * height;
    const int nr = valid ? min(height, rows - r0) : 0;
    const int myrp = (valid && q < nr) ? row_ptr[r0 + q] : INT_MAX;
    const int s1 = valid ? row_ptr[r0 + nr] : 0;
    const int s0_lane = __shfl(myrp, gbase);
    const int s0 = valid ? s0_lane : 0;
    const int n = s1 - s0;
    if (valid && q == 0) {
        strip_ptr[strip] = s0;
        if (strip == strips - 1) strip_ptr[strips] = nnz;
    }
    bool special = valid && n > CAP;
    const int umax = used_slots<G>(valid && !special ? n : 0);

    int c[E], t[E];
    ET v[E];
#pragma unroll
    for (int u = 0; u < E; ++u) {
        c[u] = 0;
        t[u] = 0;
        v[u] = ET(0);
        if (u < umax) {
            const int j = s0 + q + G * u;
            const bool act = valid && !special && j < s1;
            if (act) {
                c[u] = col_ind[j];
                v[u] = val_in[j];
            }
            t[u] = row_in_strip<HB>(myrp, j, gbase);
        }
    }

    {
        // Words of every strip the group holds in LDS by place, and the
        // strip-relative row pointers of rows 0..HB (row_place).
        const bool fits = valid && !special;
        LdsWord* A = reinterpret_cast<LdsWord*>(slice) + gbase * E;
        LdsWord* B = A + kWave * E;
        LdsInt* rtab = (LdsInt*)&rowtab[wave][g * (HB + 1)];
        uint32_t wd[E];
        int pos[E];
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int p = q + G * u;
            wd[u] = (static_cast<uint32_t>(c[u]) << bits) | static_cast<uint32_t>(t[u]);
            pos[u] = p;
            if (u < umax && fits && p < n) A[p] = wd[u];
        }
        if (q < HB) rtab[q] = row_place(fits, q, nr, myrp - s0, n);
        if (q == 0) rtab[HB] = row_place(fits, HB, nr, 0, n);
        wave_lds_sync();
        // Rows must ascend (non-strictly) by column for the merge: an entry
        // and the next one of the strip, when they share the RowInStrip field
        // (the same row), must not descend.
        const uint32_t mask = (1u << bits) - 1u;
        bool bad = false;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            if (u >= umax) break;
            const int p = q + G * u;
            if (fits && p + 1 < n) {
                const uint32_t nw = A[p + 1];
                if ((nw & mask) == (wd[u] & mask) && (nw >> bits) < (wd[u] >> bits)) bad = true;
            }
        }
        const bool gbad = (ballot(bad) & group_mask(gbase, G)) != 0;
        special = special || (valid && gbad);
        // Uniform: the wave's one strip, sorted below from the words in A.
        const bool held = G == kWave && HB >= kBucketHeight && gbad;
        constexpr int WCAP = kWave * E;  // what sort_strip_mid<HB, E> holds
        constexpr int INLINE = kInlineSortMax < WCAP ? kInlineSortMax : WCAP;
        if (valid && special && !held && q == 0 && n > INLINE) {
            if (n <= kWaveSortCap)
                ws_small[atomicAdd(&ws_count[0], 1)] = strip;
            else
                ws_big[atomicAdd(&ws_count[1], 1)] = strip;
        }
        const bool go = valid && !special;
        const int next_row = __shfl_down(myrp, 1);
        const int row_end = q + 1 < nr ? next_row : s1;
        const int row_max = HB > 1 ? wave_max(go && q < nr ? row_end - myrp : 0) : 0;
        if (!held)
            merge_runs_regs<HB, G, E, true>(A, B, rtab, wd, pos, umax, go, n, q, row_max, umax * G,
                                             [] { wave_lds_sync(); });
        // Out from registers: each entry to its place in the sorted strip.
        // (Staging through LDS as the tall-strip kernel does was measured
        // slower here: 133 -> 137 us at height 2, 156 -> 164 us at height 4.)
#pragma unroll
        for (int u = 0; u < E; ++u) {
            if (u >= umax) break;
            if (go && q + G * u < n && static_cast<unsigned>(pos[u]) < static_cast<unsigned>(n)) {
                col_word[s0 + pos[u]] = wd[u];
                val_out[s0 + pos[u]] = v[u];
            }
        }
        wave_lds_sync();  // the wave's slice is reused below
        if constexpr (G == kWave && HB >= kBucketHeight) {
            if (held) sort_held_strip<E, ET>(slice, n, s0, bits, val_in, col_word, val_out, lane);
        }
        uint64_t mids = ballot(valid && special && !held && q == 0 && n <= INLINE);
        while (mids) {
            const int leader = __ffsll(static_cast<unsigned long long>(mids)) - 1;
            mids &= mids - 1;
            sort_strip_mid<HB, E, 0, ET>(strip0 + leader / G, rows, height, bits, row_ptr, col_ind, val_in, col_word,
                                         val_out, slice, (LdsInt*)rowtab[wave], lane);
        }
    }
}

// ------------------------------------------------------------------ tall strips

// The key (word << 32 | place) of entry i of a strip; all lanes of the wave
// must be active.
template <int HB>
__device__ inline uint64_t strip_key(const StripRows& sr, int n, int i, int bits, const int* __restrict__ col_ind) {
    const int r = row_in_strip<HB>(sr.myrp, sr.s0 + i, 0);
    if (i >= n) return ~0ull;
    const uint32_t w = (static_cast<uint32_t>(col_ind[sr.s0 + i]) << bits) | static_cast<uint32_t>(r);
    return (static_cast<uint64_t>(w) << 32) | static_cast<uint32_t>(i);
}

template <typename Key, typename ET>
__device__ inline void write_sorted_keys(const Key* K, const StripRows& sr, int n, const ET* __restrict__ val_in,
                                         uint32_t* __restrict__ col_word, ET* __restrict__ val_out, int tid, int NT) {
    for (int i = tid; i < n; i += NT) {
        const uint64_t k = K[i];
        col_word[sr.s0 + i] = static_cast<uint32_t>(k >> 32);
        val_out[sr.s0 + i] = val_in[sr.s0 + static_cast<int>(static_cast<uint32_t>(k))];
    }
}

// Sorted CSR -> CMRS for strips of several hundred to a few thousand entries, one
// workgroup of NT threads per strip of at most 8 NT entries (longer strips go to
// the workspace lists), words, values and places in registers.
//
// Rows sorted by column: a merge of the row runs (merge_runs_regs) in one LDS
// buffer, which then holds the sorted words; the values go through the same LDS.
// Both leave in order: a scatter into the strip's range would leave partly
// written lines (each reaching HBM more than once).  Bound by VALU issue like the
// group kernel, with six waves per SIMD (eight spilled registers: 188 us against
// 157 on 2^20 Poisson(16) rows, fp64, height 32; one wave per strip with 20
// entries per lane had four: 249 us).  Strips like these went to the lists or,
// bunched columns at height 16 and up, through the bitonic network: band of 129,
// fp32, height 8/16/32 1068/3252/3313 -> 212/221/426 us; 27-point stencil, fp64,
// height 32 640 -> 271 us; Poisson(48) rows, fp64, height 32 3840 -> 210 us.
//
// Rows not sorted: one bucketing pass, whatever the height: entries fall into NB
// buckets of about equal width over the strip's column range [cmin, cmax] (NB
// about n/4; the bucket is a multiply and a shift of c - cmin, non-decreasing in
// c), a count per bucket (LDS atomics) and a scan give each bucket's start, the
// keys (word << 32 | position in strip) are scattered by bucket, and an entry's
// place is its bucket's start plus the number of keys of its bucket below its own.
// Keys are unique and ordered as the reorder of Sec. 4 requires (column, then
// RowInStrip, then CSR order), so duplicates need no special path.  A strip whose
// largest bucket holds more than kBucketMax keys (columns bunched at a few values
// far apart) is sorted by a bitonic network over the same keys instead.
constexpr int kTallSlots = 8;
// Sorted rows from kBucketHeight (next power of two) on take the bucketing pass too,
// as long as no bucket then holds more than kSpreadBucketMax: the levels of merging
// cost more than it does.  At four levels every strip tries (40 000 strips, fp64,
// merged/bucketed: band of 81, height 16, 288/242 us; band of 129, height 12, 326/261;
// Poisson(30) rows, height 16, 190/161; 3000 strips of Poisson(48) rows, height 12,
// 28.8/22.6), at five only those whose columns range over at least kSpread times
// their entries (60 000 Poisson(15) rows, height 32: 23.9/18.6), since clustered
// columns, counted in vain or in full buckets, pay for it (40 000 strips, height 24,
// 27-point stencil 270/302, band of 41 255/282).
template <int HB>
constexpr int kSpread = HB > kBucketHeight ? 32 : 0;
constexpr int kSpreadBucketMax = 16;

template <int HB, int NT, typename ET>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(6))) void from_csr_tall_kernel(
    int rows, int strips, int height, int bits, int nnz, const int* __restrict__ row_ptr,
    const int* __restrict__ col_ind, const ET* __restrict__ val_in, int* __restrict__ strip_ptr,
    uint32_t* __restrict__ col_word, ET* __restrict__ val_out, int* __restrict__ ws_count,
    int* __restrict__ ws_small, int* __restrict__ ws_big) {
    constexpr int E = kTallSlots, CAP = E * NT, NBMAX = CAP / 4;
    // The bucket count doubles up to NBMAX, so NBMAX must be a power of two
    // (otherwise it would pass NBMAX and overrun start).
    static_assert((NBMAX & (NBMAX - 1)) == 0 && NBMAX % NT == 0, "bucket capacity");
    static_assert(HB + 1 <= kWave && NT >= 2 * kWave, "row table in one wave");
    // Words in the first half (a search reads at most CAP past them), then values
    // or keys in all of it.
    __shared__ __align__(16) uint64_t keys[CAP];
    __shared__ int start[NBMAX + 1];  // also the row table
    __shared__ int red[3][NT / kWave];
    const int tid = static_cast<int>(threadIdx.x);
    const int lane = lane_id();
    const int wave = uniform(tid / kWave);
    const int strip = xcd_logical_block(blockIdx.x, gridDim.x);
    const StripRows sr = load_strip_rows(strip, rows, height, row_ptr, lane);
    const int s0 = uniform(sr.s0);
    const int n = uniform(sr.s1) - s0;
    if (tid == 0) {
        strip_ptr[strip] = s0;
        if (strip == strips - 1) strip_ptr[strips] = nnz;
        if (n > CAP) {
            if (n <= kWaveSortCap)
                ws_small[atomicAdd(&ws_count[0], 1)] = strip;
            else
                ws_big[atomicAdd(&ws_count[1], 1)] = strip;
        }
    }
    if (n > CAP || n == 0) return;
    const int umax = (n + NT - 1) / NT;
    LdsWord* const A = (LdsWord*)reinterpret_cast<uint32_t*>(keys);
    const uint32_t rmask = (1u << bits) - 1u;
    uint32_t wd[E];
    ET v[E];
#pragma unroll
    for (int u = 0; u < E; ++u) {
        wd[u] = 0u;
        v[u] = ET(0);
        if (u < umax) {
            const int j = s0 + min(tid + NT * u, n - 1);
            wd[u] = static_cast<uint32_t>(col_ind[j]) << bits;
            v[u] = val_in[j];
        }
    }
    if (tid <= HB) start[tid] = tid < sr.nr ? sr.myrp - s0 : n;  // wave 0: lane == tid
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if (u >= umax) break;
        const int i = tid + NT * u;
        wd[u] |= static_cast<uint32_t>(row_in_strip<HB>(sr.myrp, s0 + min(i, n - 1), 0));
        if (i < n) A[i] = wd[u];
    }
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if (u >= umax) break;
        const int i = tid + NT * u;
        if (i + 1 < n) {
            const uint32_t nw = A[i + 1];
            if ((nw & rmask) == (wd[u] & rmask) && nw < wd[u]) bad = true;
        }
    }
    bad = __syncthreads_or(bad);
    int cmin = INT_MAX, cmax = -1;
    if (!bad && HB >= kBucketHeight) {  // uniform
        // The rows ascend: their first and last words, in every wave by itself.
        const int r0 = lane < sr.nr ? start[lane] : 0, r1 = lane < sr.nr ? start[lane + 1] : 0;
        if (r0 < r1) {
            cmin = static_cast<int>(A[r0] >> bits);
            cmax = static_cast<int>(A[r1 - 1] >> bits);
        }
        cmin = -wave_max(-cmin);
        cmax = wave_max(cmax);
    }
    if (bad) {
#pragma unroll
        for (int u = 0; u < E; ++u) {
            if (tid + NT * u < n) {
                const int c = static_cast<int>(wd[u] >> bits);
                cmin = min(cmin, c);
                cmax = max(cmax, c);
            }
        }
        cmin = -wave_max(-cmin);
        cmax = wave_max(cmax);
        if (lane == 0) {
            red[0][wave] = cmin;
            red[1][wave] = cmax;
        }
        __syncthreads();
        for (int w = 0; w < NT / kWave; ++w) {
            cmin = min(cmin, red[0][w]);
            cmax = max(cmax, red[1][w]);
        }
    }
    const bool spread = HB >= kBucketHeight && cmax - cmin >= kSpread<HB> * n;
    int pos[E];
#pragma unroll
    for (int u = 0; u < E; ++u) pos[u] = tid + NT * u;
    bool merge = !bad && !spread;
    if (!merge) {
        int nbk = 1;
        while (nbk < NBMAX && nbk * 4 < n) nbk <<= 1;
        __syncthreads();  // the row table is read above; the counts overwrite it
        for (int b = tid; b < NBMAX; b += NT) start[b] = 0;
        __syncthreads();
        // bucket(c) = ((c - cmin) * scale) >> 32 with scale = floor(2^32 nbk /
        // range): non-decreasing in c and below nbk for c <= cmax.
        const uint64_t range = static_cast<uint64_t>(cmax - cmin) + 1u;
        const uint64_t scale = (static_cast<uint64_t>(nbk) << 32) / range;
        int bs[E];  // bucket << 16 | slot in bucket
#pragma unroll
        for (int u = 0; u < E; ++u) {
            bs[u] = 0;
            if (tid + NT * u < n) {
                const uint32_t c = wd[u] >> bits;
                const int bk = static_cast<int>((static_cast<uint64_t>(c - static_cast<uint32_t>(cmin)) * scale) >> 32);
                bs[u] = (bk << 16) | atomicAdd(&start[bk], 1);
            }
        }
        __syncthreads();
        // Counts to starts: thread t takes PER buckets from t * PER.
        constexpr int PER = NBMAX / NT;
        int cnt[PER], sum = 0, most = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            cnt[k] = start[tid * PER + k];
            sum += cnt[k];
            most = max(most, cnt[k]);
        }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int t = __shfl_up(incl, off);
            if (lane >= off) incl += t;
        }
        most = wave_max(most);
        if (lane == kWave - 1) red[0][wave] = incl;
        if (lane == 0) red[2][wave] = most;
        __syncthreads();
        int run = incl - sum;
        for (int w = 0; w < NT / kWave; ++w) {
            if (w < wave) run += red[0][w];
            most = max(most, red[2][w]);
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            start[tid * PER + k] = run;
            run += cnt[k];
        }
        if (tid == NT - 1) start[NBMAX] = run;
        __syncthreads();
        if (most <= (bad ? kBucketMax : kSpreadBucketMax)) {
#pragma unroll
            for (int u = 0; u < E; ++u) {
                const int i = tid + NT * u;
                if (i < n)
                    keys[start[bs[u] >> 16] + (bs[u] & 0xffff)] =
                        (static_cast<uint64_t>(wd[u]) << 32) | static_cast<uint32_t>(i);
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < E; ++u) {
                const int i = tid + NT * u;
                if (i < n) {
                    const int bk = bs[u] >> 16;
                    const int b0 = start[bk], b1 = start[bk + 1];
                    const uint64_t key = (static_cast<uint64_t>(wd[u]) << 32) | static_cast<uint32_t>(i);
                    int p = b0;
                    for (int k = b0; k < b1; ++k) p += keys[k] < key ? 1 : 0;
                    pos[u] = p;
                }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < E; ++u)
                if (tid + NT * u < n) A[pos[u]] = wd[u];
        } else if (!bad) {
            merge = true;  // A still holds the words
            if (tid <= HB) start[tid] = tid < sr.nr ? sr.myrp - s0 : n;
        } else {
            const int P = pow2_at_least(n);
#pragma unroll
            for (int u = 0; u < E; ++u) {
                const int i = tid + NT * u;
                if (i < P) keys[i] = i < n ? (static_cast<uint64_t>(wd[u]) << 32) | static_cast<uint32_t>(i) : ~0ull;
            }
            __syncthreads();
            bitonic_sort(keys, P, 0, tid, NT, [] { __syncthreads(); });
            write_sorted_keys(keys, sr, n, val_in, col_word, val_out, tid, NT);
            return;
        }
        __syncthreads();
    }
    if (merge) {
        const int next_row = __shfl_down(sr.myrp, 1);
        const int row_max = wave_max(lane < sr.nr ? next_row - sr.myrp : 0);
        merge_runs_regs<HB, NT, E, true, true>(A, A, (LdsInt*)start, wd, pos, umax, true, n, tid, row_max, n,
                                               [] { __syncthreads(); });
        __syncthreads();
    }
    for (int i = tid; i < n; i += NT) col_word[s0 + i] = A[i];
    __syncthreads();
    ET* KV = reinterpret_cast<ET*>(keys);
#pragma unroll
    for (int u = 0; u < E; ++u)
        if (tid + NT * u < n) KV[pos[u]] = v[u];
    __syncthreads();
    for (int i = tid; i < n; i += NT) val_out[s0 + i] = KV[i];
}

// CMRS -> CSR at height 1: every strip is one row, so RowPtr is StripPtr and
// every entry keeps its place (column = word >> bits); a plain coalesced
// stream.  (A word with a non-zero RowInStrip is invalid input at height 1;
// it is copied like the others.)
template <typename ET>
__global__ __launch_bounds__(256) void to_csr_h1_kernel(int rows, int nnz, int bits, const int* __restrict__ strip_ptr,
                                                        const uint32_t* __restrict__ word, const ET* __restrict__ val,
                                                        int* __restrict__ row_ptr, int* __restrict__ col_ind,
                                                        ET* __restrict__ val_out) {
    constexpr int U = 4;
    const int64_t nthreads = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    for (int64_t i = tid; i <= rows; i += nthreads) row_ptr[i] = strip_ptr[i];
    for (int64_t b0 = static_cast<int64_t>(blockIdx.x) * blockDim.x * U; b0 < nnz; b0 += nthreads * U) {
        uint32_t w[U];
        ET v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t j = b0 + u * blockDim.x + threadIdx.x;
            w[u] = j < nnz ? word[j] : 0u;
            v[u] = j < nnz ? val[j] : ET(0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t j = b0 + u * blockDim.x + threadIdx.x;
            if (j < nnz) {
                col_ind[j] = static_cast<int>(w[u] >> bits);
                val_out[j] = v[u];
            }
        }
    }
}

// Strip of every lane's entry in one round of a wave's run of whole strips.
// Lane t <= nsw holds StripPtr[S + t] (INT_MAX past that); `tc` (uniform)
// enters as the last strip whose pointer is <= the round's first entry and
// leaves as that of the round's last entry `lim`, so the rounds of a run step
// through its strip pointers once, whatever the strip lengths.  Empty strips
// are passed over because their pointer repeats.
__device__ inline int round_strip(int myp, int j, int lim, int& tc) {
    int t = tc;
    for (;;) {
        const int nx = __builtin_amdgcn_readlane(myp, tc + 1);
        if (nx > lim) break;
        if (j >= nx) t = tc + 1;
        ++tc;
    }
    return t;
}

// Key of an entry of strip t of the run: t*height + RowInStrip, the row's
// offset from the run's first row; -1 for a word whose RowInStrip names no
// row of its strip (the entry is then neither counted nor written).
__device__ inline int run_row_key(int t, uint32_t r, int height, int nrow) {
    const int key = t * height + static_cast<int>(r);
    return (r < static_cast<uint32_t>(height) && key < nrow) ? key : -1;
}

// Rows per wave of the CMRS -> CSR kernel: lane k < kRunRows owns row k of
// the wave's run, and row keys fit in kRunKeyBits bits.
constexpr int kRunRows = 32;
constexpr int kRunKeyBits = 5;

// Lanes of `valid` whose key (< kRunRows) equals k, from kb[b] = ballot of bit
// b of every lane's key: a match over the wave without a loop over key values.
__device__ inline uint64_t key_match(int k, uint64_t valid, const uint64_t (&kb)[kRunKeyBits]) {
    uint64_t m = valid;
#pragma unroll
    for (int b = 0; b < kRunKeyBits; ++b) m &= ((k >> b) & 1) ? kb[b] : ~kb[b];
    return m;
}

// One round of 64 consecutive entries [b, b + 64) of a run: every lane's row
// key (-1: no entry or an invalid word), its key ballots and the valid mask.
struct RunRound {
    int key;
    uint64_t valid;
    uint64_t kb[kRunKeyBits];
};

__device__ inline RunRound run_round(int myp, int b, int e1, uint32_t w, uint32_t mask, int height, int nrow, int& tc) {
    RunRound rr;
    const int j = b + lane_id();
    const int t = round_strip(myp, j, min(b + kWave, e1) - 1, tc);
    rr.key = j < e1 ? run_row_key(t, w & mask, height, nrow) : -1;
#pragma unroll
    for (int k = 0; k < kRunKeyBits; ++k) rr.kb[k] = ballot(rr.key >= 0 && ((rr.key >> k) & 1));
    rr.valid = ballot(rr.key >= 0);
    return rr;
}

// Waves per workgroup of the CMRS -> CSR kernel, and the run length above
// which the workgroup's waves share a run.  (2 and 8 waves were measured
// slower on both the benchmark and the skewed-row matrices.)
constexpr int kToCsrWaves = 4;
constexpr int kToCsrThreads = kToCsrWaves * kWave;
constexpr int kLongRun = 2048;
constexpr int kToCsrStage = 640;

// One run of the CMRS -> CSR kernel: strips [S, S + nsw), rows [r0, r0 +
// nrow), entries [e0, e1); lane t <= nsw holds StripPtr[S + t] in myp.
struct ToCsrRun {
    int S, nsw, r0, nrow, e0, e1, myp;
};

__device__ inline ToCsrRun to_csr_run(int run, int ns, int strips, int rows, int height,
                                      const int* __restrict__ strip_ptr, int lane) {
    ToCsrRun R;
    R.S = run * ns;
    R.nsw = R.S < strips ? min(ns, strips - R.S) : 0;
    R.myp = (R.nsw > 0 && lane <= R.nsw) ? strip_ptr[R.S + lane] : INT_MAX;
    const int p0 = __shfl(R.myp, 0), p1 = __shfl(R.myp, R.nsw);
    R.e0 = R.nsw > 0 ? uniform(p0) : 0;
    R.e1 = R.nsw > 0 ? uniform(p1) : 0;
    R.r0 = R.S * height;
    R.nrow = R.nsw > 0 ? min(R.nsw * height, rows - R.r0) : 0;
    return R;
}

// CMRS -> CSR with one wave per run of `ns` whole strips (ns*height <=
// kRunRows consecutive rows, lane k owning row k of the run).  The run's
// entries are contiguous, so the wave streams them 64 at a time with
// coalesced loads whatever the strip lengths.  Pass 1 counts the entries of
// every row (the rows' CSR starts are then a prefix sum over the lanes); pass
// 2 scatters each entry to its row's start plus its rank, the number of
// earlier entries of the same row (earlier rounds: a per-row counter; this
// round: lanes below it with the same key).  The scatter keeps strip order
// inside every row, the stable order of the inverse conversion.  A run of at
// most FIT entries is loaded once and both passes work on the registers;
// longer runs are read twice.  A run of more than kLongRun entries is shared
// by the workgroup's waves after they have finished their own runs: each wave
// counts a contiguous slice, the per-row counts of earlier slices (LDS) start
// its ranks, and each wave scatters its slice.  Every wave reads the lengths
// of the workgroup's runs and so takes the same barrier-or-not decision; a
// workgroup without a long run has no barrier.
template <typename ET, bool STAGE>
__global__ __launch_bounds__(kToCsrThreads) __attribute__((amdgpu_waves_per_eu(STAGE ? 5 : 8))) void to_csr_rows_kernel(
    int rows, int strips, int height, int bits, int ns, const int* __restrict__ strip_ptr,
    const uint32_t* __restrict__ word, const ET* __restrict__ val, int* __restrict__ row_ptr,
    int* __restrict__ col_ind, ET* __restrict__ val_out) {
    constexpr int UF = 12, U = 8, FIT = UF * kWave;
    __shared__ int slice_cnt[kToCsrWaves][kRunRows];
    // STAGE: a run of at most kToCsrStage entries is scattered into LDS and
    // then written out in order (the run's CSR range is contiguous): with many
    // rows per strip the 64 lanes of a scatter would otherwise each write into
    // another line.  The LDS lowers the waves per SIMD from 8 to 5, which costs
    // more than it saves at small heights and on runs of very uneven length.
    constexpr int SCAP = STAGE ? kToCsrStage : 1;
    __shared__ int stage_col[kToCsrWaves][SCAP];
    __shared__ ET stage_val[kToCsrWaves][SCAP];
    const int lane = lane_id();
    const int wave = uniform(static_cast<int>(threadIdx.x) / kWave);
    const int run0 = xcd_logical_block(blockIdx.x, gridDim.x) * kToCsrWaves;
    const int nruns = (strips + ns - 1) / ns;
    const uint32_t mask = (1u << bits) - 1u;
    const uint64_t lt = lanemask_lt();

    // This wave's run, loaded before the lengths below so that both loads are
    // in flight together.
    const ToCsrRun Rw = to_csr_run(run0 + wave, ns, strips, rows, height, strip_ptr, lane);
    // Bit r: run run0 + r holds more than kLongRun entries (lanes r <
    // kToCsrWaves read the runs' first strip pointers, the next kToCsrWaves
    // lanes their last).
    uint64_t longs;
    {
        const int run = run0 + (lane & (kToCsrWaves - 1));
        const int sidx = min(run * ns + (lane >= kToCsrWaves ? ns : 0), strips);
        const int p = (lane < 2 * kToCsrWaves && run < nruns) ? strip_ptr[sidx] : 0;
        const int pend = __shfl(p, (lane & (kToCsrWaves - 1)) + kToCsrWaves);
        longs = ballot(lane < kToCsrWaves && run < nruns && pend - p > kLongRun);
    }

    // CSR starts of the run's rows from per-row counts (lane k: row k);
    // `write` stores them.
    auto row_starts = [&](const ToCsrRun& R, int cnt, bool write) {
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < kRunRows; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        const int start = R.e0 + incl - cnt;
        if (write && lane < R.nrow) row_ptr[R.r0 + lane] = start;
        if (write && R.S + R.nsw == strips && lane == 0) row_ptr[rows] = R.e1;
        return start;
    };
    // Scatter of one round; `next` (lane k): CSR position of the next entry of row k.
    auto scatter = [&](const ToCsrRun& R, const RunRound& rr, uint32_t w, ET v, int& next) {
        const int src = rr.key >= 0 ? rr.key : 0;
        const int pos = __shfl(next, src) + __popcll(key_match(src, rr.valid, rr.kb) & lt);
        // pos lies in [e0, e1) by construction; the check keeps a corrupt
        // strip from writing outside its run.
        if (rr.key >= 0 && static_cast<unsigned>(pos - R.e0) < static_cast<unsigned>(R.e1 - R.e0)) {
            col_ind[pos] = static_cast<int>(w >> bits);
            val_out[pos] = v;
        }
        next += __popcll(key_match(lane, rr.valid, rr.kb));
    };
    // Per-row counts (lane k: row k) of the run's entries [lo, hi).
    auto count_range = [&](const ToCsrRun& R, int lo, int hi) {
        int cnt = 0, tc = 0;
        for (int b0 = lo; b0 < hi; b0 += U * kWave) {
            uint32_t w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = b0 + u * kWave + lane;
                w[u] = j < hi ? word[j] : 0u;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (b0 + u * kWave >= hi) break;
                const RunRound rr = run_round(R.myp, b0 + u * kWave, hi, w[u], mask, height, R.nrow, tc);
                cnt += __popcll(key_match(lane, rr.valid, rr.kb));
            }
        }
        return cnt;
    };
    // Scatter of the run's entries [lo, hi).
    auto scatter_range = [&](const ToCsrRun& R, int lo, int hi, int& next) {
        int tc = 0;
        for (int b0 = lo; b0 < hi; b0 += U * kWave) {
            uint32_t w[U];
            ET v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = b0 + u * kWave + lane;
                w[u] = j < hi ? word[j] : 0u;
                v[u] = j < hi ? val[j] : ET(0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (b0 + u * kWave >= hi) break;
                const RunRound rr = run_round(R.myp, b0 + u * kWave, hi, w[u], mask, height, R.nrow, tc);
                scatter(R, rr, w[u], v[u], next);
            }
        }
    };

    // This wave's own run, unless it is long.
    if (run0 + wave < nruns && !((longs >> wave) & 1)) {
        const ToCsrRun& R = Rw;
        if (R.e1 - R.e0 <= FIT) {
            uint32_t w[UF];
            ET v[UF];
#pragma unroll
            for (int u = 0; u < UF; ++u) {
                const int j = R.e0 + u * kWave + lane;
                w[u] = j < R.e1 ? word[j] : 0u;
                v[u] = j < R.e1 ? val[j] : ET(0);
            }
            int cnt = 0, tc = 0;
#pragma unroll
            for (int u = 0; u < UF; ++u) {
                if (R.e0 + u * kWave >= R.e1) break;
                const RunRound rr = run_round(R.myp, R.e0 + u * kWave, R.e1, w[u], mask, height, R.nrow, tc);
                cnt += __popcll(key_match(lane, rr.valid, rr.kb));
            }
            int next = row_starts(R, cnt, true);
            tc = 0;
            const int n = R.e1 - R.e0;
            if (STAGE && n <= SCAP) {
                int* sc = stage_col[wave];
                ET* sv = stage_val[wave];
#pragma unroll
                for (int u = 0; u < UF; ++u) {
                    if (R.e0 + u * kWave >= R.e1) break;
                    const RunRound rr = run_round(R.myp, R.e0 + u * kWave, R.e1, w[u], mask, height, R.nrow, tc);
                    const int src = rr.key >= 0 ? rr.key : 0;
                    const int pos = __shfl(next, src) + __popcll(key_match(src, rr.valid, rr.kb) & lt) - R.e0;
                    if (rr.key >= 0 && static_cast<unsigned>(pos) < static_cast<unsigned>(n)) {
                        sc[pos] = static_cast<int>(w[u] >> bits);
                        sv[pos] = v[u];
                    }
                    next += __popcll(key_match(lane, rr.valid, rr.kb));
                }
                wave_lds_sync();
                // Every place of the run is written above (the rows' counts
                // add up to n) unless a word names no row of its strip; those
                // places keep what the stage held and are not valid output.
                for (int i = lane; i < n; i += kWave) {
                    col_ind[R.e0 + i] = sc[i];
                    val_out[R.e0 + i] = sv[i];
                }
                wave_lds_sync();
            } else {
#pragma unroll
                for (int u = 0; u < UF; ++u) {
                    if (R.e0 + u * kWave >= R.e1) break;
                    const RunRound rr = run_round(R.myp, R.e0 + u * kWave, R.e1, w[u], mask, height, R.nrow, tc);
                    scatter(R, rr, w[u], v[u], next);
                }
            }
        } else {
            int next = row_starts(R, count_range(R, R.e0, R.e1), true);
            scatter_range(R, R.e0, R.e1, next);
        }
    }

    // The workgroup's long runs, shared by all its waves (`longs` is the same
    // in every wave, so every wave meets the same barriers).
    if (longs) {
        for (int r = 0; r < kToCsrWaves; ++r) {
            if (!((longs >> r) & 1)) continue;
            const ToCsrRun R = to_csr_run(run0 + r, ns, strips, rows, height, strip_ptr, lane);
            const int n = R.e1 - R.e0;
            const int chunk = ((n + kToCsrWaves - 1) / kToCsrWaves + kWave - 1) / kWave * kWave;
            const int lo = min(R.e0 + wave * chunk, R.e1), hi = min(lo + chunk, R.e1);
            const int cnt = count_range(R, lo, hi);
            if (lane < kRunRows) slice_cnt[wave][lane] = cnt;
            __syncthreads();
            int tot = 0, before = 0;
            if (lane < kRunRows) {
                for (int w2 = 0; w2 < kToCsrWaves; ++w2) {
                    const int c = slice_cnt[w2][lane];
                    tot += c;
                    if (w2 < wave) before += c;
                }
            }
            int next = row_starts(R, tot, wave == 0) + before;
            scatter_range(R, lo, hi, next);
            __syncthreads();  // slice_cnt is reused by the next long run
        }
    }
}

// CSR -> CMRS without the reorder, one wave per run of `ns` whole strips
// (ns*height <= kRunRows consecutive rows); lane k <= nrow holds RowPtr of
// row k of the run.  Entries keep their places, so the wave streams the run's
// (contiguous) entries 64 at a time with coalesced loads: the row of every
// entry comes from stepping through the run's row pointers (`round_strip`),
// and word = col << bits | (row mod height).  Writes the strip pointers too.
// col_word may alias col_ind and val_out may alias val_in (each entry is read
// and written by the same lane).
template <typename ET>
__global__ __launch_bounds__(kConvThreads) void from_csr_rows_kernel(
    int rows, int strips, int height, int bits, int nnz, int ns, const int* __restrict__ row_ptr,
    const int* col_ind, const ET* val_in, int* __restrict__ strip_ptr, uint32_t* col_word, ET* val_out,
    int copy_val) {
    constexpr int U = 8;
    const int lane = lane_id();
    const int wave = uniform(static_cast<int>(threadIdx.x) / kWave);
    const int S = (xcd_logical_block(blockIdx.x, gridDim.x) * kConvWaves + wave) * ns;
    if (S >= strips) return;
    const int nsw = min(ns, strips - S);
    const int r0 = S * height;
    const int nrow = min(nsw * height, rows - r0);
    const int myrp = lane <= nrow ? row_ptr[r0 + lane] : INT_MAX;
    const int e0 = uniform(__shfl(myrp, 0)), e1 = uniform(__shfl(myrp, nrow));
    const int sfirst = __shfl(myrp, min(lane * height, kRunRows));  // first entry of strip S + lane
    if (lane < nsw) strip_ptr[S + lane] = sfirst;
    if (S + nsw == strips && lane == 0) strip_ptr[strips] = nnz;
    const bool pow2 = (height & (height - 1)) == 0;
    int tc = 0;
    for (int b0 = e0; b0 < e1; b0 += U * kWave) {
        int c[U];
        ET v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = b0 + u * kWave + lane;
            c[u] = j < e1 ? col_ind[j] : 0;
            v[u] = j < e1 ? val_in[j] : ET(0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (b0 + u * kWave >= e1) break;
            const int j = b0 + u * kWave + lane;
            const int k = round_strip(myrp, j, min(b0 + u * kWave + kWave, e1) - 1, tc);
            const int r = pow2 ? (k & (height - 1)) : k % height;
            if (j < e1) {
                col_word[j] = (static_cast<uint32_t>(c[u]) << bits) | static_cast<uint32_t>(r);
                if (copy_val) val_out[j] = v[u];
            }
        }
    }
}

// Entries [lo, lo + len) of a sorted LDS array below w, for C entries at
// once: the searches step together (binary lifting, as many steps as the
// longest of the C ranges needs) so their LDS reads are in flight together.
template <int C>
__device__ inline void count_below(const uint32_t* S, const uint32_t (&w)[C], const int (&lo)[C],
                                   const int (&len)[C], int (&cnt)[C]) {
    int top = 0;
#pragma unroll
    for (int v = 0; v < C; ++v) {
        top |= len[v];
        cnt[v] = 0;
    }
    top = top > 0 ? 1 << (31 - __clz(top)) : 0;
    for (int step = top; step > 0; step >>= 1) {
#pragma unroll
        for (int v = 0; v < C; ++v) {
            const bool ok = cnt[v] + step <= len[v];
            const uint32_t x = S[ok ? lo[v] + cnt[v] + step - 1 : 0];
            if (ok && x < w[v]) cnt[v] += step;
        }
    }
}

// Rows of at most kLightRow entries are light, the others heavy.  A listed strip
// of at most kHeavyMax heavy rows (kHeavyStaged where only the workspace could merge
// it) and kLightCap entries in light ones (a long row or few among short ones, as
// skewed matrices have them) is streamed.
constexpr int kLightRow = 64;
constexpr int kLightCap = 512;
constexpr int kHeavyMax = 2, kHeavyStaged = 4;

// The rows of a long strip, row x in lane x of every wave: its first entry in
// the strip and its length (rows past the strip: n, 0).
struct RunTable {
    int lo, len;
};
template <int HB>
__device__ inline RunTable run_table(const StripRows& sr, int n, int lane) {
    RunTable t;
    t.lo = lane < sr.nr ? sr.myrp - sr.s0 : n;
    const int next = __shfl(t.lo, min(lane + 1, kWave - 1));
    t.len = lane < HB ? next - t.lo : 0;
    return t;
}

// A long strip that a workgroup streams: returns whether an entry descends (the
// strip's output is then to be written again).  Thread t owns light entry t: its
// rank among the light words comes from comparing it with all of them in LW (the
// same words for every lane: no bank conflicts, no dependent loads), and SL takes
// the light words in order.  A heavy entry's place is its index in its row plus
// its count of light words below (a binary search over SL) plus one over each
// other heavy row; a light entry's is its rank plus, for each heavy row, the first
// entry that has counted it (H).  A heavy row's entries are read in order and
// leave in nearly that order, so nothing of it is held but, for the searches of
// another heavy row, the strip's columns where they fit (staged: HC, by place);
// otherwise those searches read global memory (150 strips of two rows of 4000 and
// 30 of 3, fp64, global / staged 71/65 us, and three such rows 124/103; the merge in
// the workspace takes 144 for those).  The strip costs few barriers, and two
// workgroups share a CU.  (With the whole
// strip's words in LDS, one workgroup of 1024 threads per CU, the listed strips of
// the skewed 2*10^6-row workload, fp32, height 16, took 152 us at a quarter of the
// VALU rate, 32 us a strip and workgroup, nearly all latency between barriers; now
// 12 to 25 us a strip, 127 us for both lists.)
template <int HB, int NT, typename ET>
__device__ inline bool stream_strip(const StripRows& sr, const RunTable& rows_of, uint64_t heavy, int m, int rls,
                                    int bits, const int* __restrict__ col_ind, const ET* __restrict__ val_in,
                                    uint32_t* __restrict__ col_word, ET* __restrict__ val_out, uint32_t* LW,
                                    uint32_t* SL, int* H, int* HC, bool staged, int tid, int lane) {
    static_assert(NT >= kLightCap, "one light entry per thread");
    constexpr int C = 4;  // entries of a heavy row searched together
    const uint32_t rmask = (1u << bits) - 1u;
    const int* __restrict__ col = col_ind + sr.s0;
    const ET* __restrict__ vin = val_in + sr.s0;
    bool bad = false;
    uint32_t w = 0;
    ET v = ET(0);
    int pos = 0;
    const bool mine = tid < m;
    if (staged) {
        const int n = sr.s1 - sr.s0;
        for (int i = tid; i < n; i += NT) HC[i] = col[i];
        __syncthreads();
        // Unsorted rows show here for little.
        for (uint64_t hm = heavy; hm; hm &= hm - 1) {  // uniform
            const int r = __ffsll(static_cast<unsigned long long>(hm)) - 1;
            const int lo = __shfl(rows_of.lo, r), len = __shfl(rows_of.len, r);
            for (int i = tid; i + 1 < len; i += NT) bad = bad || HC[lo + i + 1] < HC[lo + i];
        }
        if (__syncthreads_or(bad)) return true;
    }
    {
        const int r = row_in_strip<HB>(lane < HB ? rls : INT_MAX, tid, 0);
        const int lo = __shfl(rows_of.lo, r), first = __shfl(rls, r);
        if (mine) {
            const int i = lo + tid - first;
            w = (static_cast<uint32_t>(col[i]) << bits) | static_cast<uint32_t>(r);
            v = vin[i];
            LW[tid] = w;
        }
    }
    __syncthreads();
    if (mine) {
        if (tid + 1 < m) {
            const uint32_t nw = LW[tid + 1];
            bad = (nw & rmask) == (w & rmask) && nw < w;
        }
        const uint4* LW4 = reinterpret_cast<const uint4*>(LW);
        const auto add = [&](uint32_t a, int j) { pos += (a < w || (a == w && j < tid)) ? 1 : 0; };
        int j = 0;
#pragma unroll 1
        for (; j + 8 <= m; j += 8) {
            const uint4 p = LW4[j / 4], q = LW4[j / 4 + 1];
            add(p.x, j); add(p.y, j + 1); add(p.z, j + 2); add(p.w, j + 3);
            add(q.x, j + 4); add(q.y, j + 5); add(q.z, j + 6); add(q.w, j + 7);
        }
        for (; j < m; ++j) add(LW[j], j);
        SL[pos] = w;
    }
    const int rank = pos;
    __syncthreads();
    for (uint64_t hm = heavy; hm; hm &= hm - 1) {  // uniform
        const int r = __ffsll(static_cast<unsigned long long>(hm)) - 1;
        const int lo = __shfl(rows_of.lo, r), len = __shfl(rows_of.len, r);
        if (mine) H[tid] = len;
        __syncthreads();
#pragma unroll 1
        for (int i0 = 0; i0 < len; i0 += C * NT) {  // uniform
            int c[C], nc[C], at[C], from[C], upto[C], cnt[C];
            ET hv[C];
            uint32_t hw[C];
#pragma unroll
            for (int k = 0; k < C; ++k) {
                at[k] = i0 + k * NT + tid;
                const int i = lo + min(at[k], len - 1);
                c[k] = col[i];
                hv[k] = vin[i];
                // The next entry's column: the next lane's, or loaded by the last lane.
                nc[k] = lane == kWave - 1 ? col[lo + min(at[k] + 1, len - 1)] : 0;
            }
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const int shifted = __shfl_down(c[k], 1);
                if (at[k] + 1 < len && (lane == kWave - 1 ? nc[k] : shifted) < c[k]) bad = true;
                hw[k] = (static_cast<uint32_t>(c[k]) << bits) | static_cast<uint32_t>(r);
                from[k] = 0;
                upto[k] = m;
            }
            count_below<C>(SL, hw, from, upto, cnt);
            // The light words below this entry and not below the one before it
            // stand behind `at` entries of the row; noted at the last of them.
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const int before = __shfl_up(cnt[k], 1);
                if (at[k] < len && cnt[k] > 0 && (lane == 0 || before != cnt[k])) atomicMin(&H[cnt[k] - 1], at[k]);
            }
#pragma unroll 1
            for (uint64_t om = heavy & ~(1ull << r); om; om &= om - 1) {  // uniform
                const int x = __ffsll(static_cast<unsigned long long>(om)) - 1;
                const int xlo = __shfl(rows_of.lo, x), xlen = __shfl(rows_of.len, x);
                // Entries of the other heavy row that sort before this one:
                // columns below, or equal in an earlier row.
                int below[C];
#pragma unroll
                for (int k = 0; k < C; ++k) below[k] = 0;
                const auto search = [&](const int* row) {
#pragma unroll 1
                    for (int step = 1 << (31 - __clz(xlen)); step > 0; step >>= 1) {
                        int y[C];
#pragma unroll
                        for (int k = 0; k < C; ++k) y[k] = row[min(below[k] + step, xlen) - 1];
#pragma unroll
                        for (int k = 0; k < C; ++k)
                            if (below[k] + step <= xlen && (y[k] < c[k] || (x < r && y[k] == c[k]))) below[k] += step;
                    }
                };
                if (staged)
                    search(HC + xlo);
                else
                    search(col + xlo);
#pragma unroll
                for (int k = 0; k < C; ++k) cnt[k] += below[k];
            }
#pragma unroll
            for (int k = 0; k < C; ++k) {
                if (at[k] < len) {
                    col_word[sr.s0 + at[k] + cnt[k]] = hw[k];
                    val_out[sr.s0 + at[k] + cnt[k]] = hv[k];
                }
            }
        }
        __syncthreads();
        // Entries of this row before the light word of rank t: the least note
        // at t or behind it.
        if (mine) {
            int least = len;
            for (int j = rank; j < m; ++j) least = min(least, H[j]);
            pos += least;
        }
        __syncthreads();
    }
    if (mine && static_cast<unsigned>(pos) < static_cast<unsigned>(sr.s1 - sr.s0)) {
        col_word[sr.s0 + pos] = w;
        val_out[sr.s0 + pos] = v;
    }
    return bad;
}

// A long strip of at most NT*E entries by a merge of its row runs in LDS (A, B:
// its words by place; rt: the rows' first places, HB + 1 of them): returns
// whether an entry descends (nothing is written then).
template <int HB, int NT, int E, typename ET>
__device__ inline bool merge_strip_block(const StripRows& sr, int n, int row_max, int bits,
                                         const int* __restrict__ col_ind, const ET* __restrict__ val_in,
                                         uint32_t* __restrict__ col_word, ET* __restrict__ val_out, LdsWord* A,
                                         LdsWord* B, const LdsInt* rt, int tid) {
    const int umax = (n + NT - 1) / NT;
    const uint32_t rmask = (1u << bits) - 1u;
    uint32_t wd[E];
    int pos[E];
#pragma unroll
    for (int u = 0; u < E; ++u) {
        pos[u] = tid + NT * u;
        wd[u] = static_cast<uint32_t>(col_ind[sr.s0 + min(pos[u], n - 1)]) << bits;
    }
#pragma unroll
    for (int u = 0; u < E; ++u) {  // every lane runs the row lookup
        wd[u] |= static_cast<uint32_t>(row_in_strip<HB>(sr.myrp, sr.s0 + min(pos[u], n - 1), 0));
        if (pos[u] < n) A[pos[u]] = wd[u];
    }
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if (pos[u] + 1 < n) {
            const uint32_t nw = A[pos[u] + 1];
            if ((nw & rmask) == (wd[u] & rmask) && nw < wd[u]) bad = true;
        }
    }
    if (__syncthreads_or(bad)) return true;
    merge_runs_regs<HB, NT, E, false, false, true>(A, B, rt, wd, pos, umax, true, n, tid, row_max, n,
                                            [] { __syncthreads(); });
    ET v[E];
#pragma unroll
    for (int u = 0; u < E; ++u) v[u] = val_in[sr.s0 + min(tid + NT * u, n - 1)];
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if (tid + NT * u < n && static_cast<unsigned>(pos[u]) < static_cast<unsigned>(n)) {
            col_word[sr.s0 + pos[u]] = wd[u];
            val_out[sr.s0 + pos[u]] = v[u];
        }
    }
    return false;
}

// merge_strip_block for a strip of any length, keys in the strip's slice G
// (2 n of them) of the workspace, C entries of a thread searched together (four /
// eight: 150 strips of eight rows of 1500 and 24 of 3, fp64, 183/157 us; of three
// rows of 4000, 159/144).
template <int HB, int NT, typename ET>
__device__ inline bool merge_strip_global(const StripRows& sr, int n, int bits, const int* __restrict__ col_ind,
                                          const ET* __restrict__ val_in, uint32_t* __restrict__ col_word,
                                          ET* __restrict__ val_out, uint64_t* G, const int* rt, int tid) {
    constexpr int C = 8;
    const uint64_t rmask = (1ull << bits) - 1ull;
    const int n64 = (n + kWave - 1) / kWave * kWave;  // whole waves: the row lookup's cross-lane reads see all lanes
    for (int i = tid; i < n64; i += NT) {
        const uint64_t k = strip_key<HB>(sr, n, i, bits, col_ind);
        if (i < n) G[i] = k;
    }
    __syncthreads();
    bool bad = false;
    for (int i = tid; i + 1 < n; i += NT) {
        const uint32_t w = static_cast<uint32_t>(G[i] >> 32), nw = static_cast<uint32_t>(G[i + 1] >> 32);
        if ((nw & rmask) == (w & rmask) && nw < w) bad = true;
    }
    if (__syncthreads_or(bad)) return true;
    uint64_t *src = G, *dst = G + n;
    for (int k = 0; (1 << k) < HB; ++k) {
        for (int i0 = tid; i0 < n; i0 += C * NT) {
            uint64_t key[C];
            int lo[C], len[C], cnt[C], own[C];
            int top = 0;
#pragma unroll
            for (int v = 0; v < C; ++v) {
                const int i = min(i0 + v * NT, n - 1);
                key[v] = src[i];
                const int run = static_cast<int>((key[v] >> 32) & (HB - 1)) >> k;
                lo[v] = rt[(run ^ 1) << k];
                len[v] = rt[((run ^ 1) + 1) << k] - lo[v];
                own[v] = run & 1 ? i - len[v] : i;
                cnt[v] = 0;
                top |= len[v];
            }
            for (int step = top > 0 ? 1 << (31 - __clz(top)) : 0; step > 0; step >>= 1) {
                uint64_t x[C];
#pragma unroll
                for (int v = 0; v < C; ++v) x[v] = src[max(lo[v] + min(cnt[v] + step, len[v]) - 1, 0)];
#pragma unroll
                for (int v = 0; v < C; ++v)
                    if (cnt[v] + step <= len[v] && x[v] < key[v]) cnt[v] += step;
            }
#pragma unroll
            for (int v = 0; v < C; ++v)
                if (i0 + v * NT < n) dst[own[v] + cnt[v]] = key[v];
        }
        __syncthreads();
        uint64_t* t = src;
        src = dst;
        dst = t;
    }
    write_sorted_keys(src, sr, n, val_in, col_word, val_out, tid, NT);
    return false;
}

// A long strip with unsorted rows: a bitonic network over its keys, in the
// workgroup's LDS K (TILE of them) or, for more, tile by tile, with the passes
// between tiles in the strip's slice G of the workspace (its pow2(n) < 2 n keys).
template <int HB, int NT, int TILE, typename ET>
__device__ inline void bitonic_strip(const StripRows& sr, int n, int bits, const int* __restrict__ col_ind,
                                     const ET* __restrict__ val_in, uint32_t* __restrict__ col_word,
                                     ET* __restrict__ val_out, LdsKey* K, uint64_t* G, int tid) {
    const int P = pow2_at_least(n);
    const auto sync = [] { __syncthreads(); };
    const int tile = min(P, TILE);  // a multiple of 64, so the row lookup sees whole waves
    for (int t0 = 0; t0 < P; t0 += tile) {
        for (int i = tid; i < tile; i += NT) K[i] = strip_key<HB>(sr, n, t0 + i, bits, col_ind);
        __syncthreads();
        bitonic_sort(K, tile, t0, tid, NT, sync);
        if (P == tile) break;
        for (int i = tid; i < tile; i += NT) G[t0 + i] = K[i];
        __syncthreads();
    }
    if (P == tile) {
        write_sorted_keys(K, sr, n, val_in, col_word, val_out, tid, NT);
        return;
    }
    for (int size = 2 * tile; size <= P; size <<= 1) {
        // Strides of whole tiles in the workspace, the rest of the size in LDS.
        for (int stride = size >> 1; stride >= tile; stride >>= 1) {
            for (int t = tid; t < P / 2; t += NT) {
                const int i = ((t & ~(stride - 1)) << 1) | (t & (stride - 1));
                const uint64_t a = G[i], b = G[i + stride];
                if ((a > b) == ((i & size) == 0)) {
                    G[i] = b;
                    G[i + stride] = a;
                }
            }
            __syncthreads();
        }
        for (int t0 = 0; t0 < P; t0 += tile) {
            for (int i = tid; i < tile; i += NT) K[i] = G[t0 + i];
            __syncthreads();
            bitonic_merge(K, tile, size, tile >> 1, t0, tid, NT, sync);
            for (int i = tid; i < tile; i += NT) G[t0 + i] = K[i];
            __syncthreads();
        }
    }
    write_sorted_keys(G, sr, n, val_in, col_word, val_out, tid, NT);
}

// Row pointers of strip `strip` for lane <= rows of the strip (INT_MAX past
// them), as load_strip_rows reads them.
__device__ inline int strip_row_ptr(int strip, int rows, int height, const int* __restrict__ row_ptr, int lane) {
    const int r0 = strip * height;
    return lane <= min(height, rows - r0) ? row_ptr[r0 + lane] : INT_MAX;
}

// Sorted conversion of the listed strips, both lists in one launch.  First the
// short ones (at most kWaveSortCap entries), one wave each in its slice of the
// key buffer, at a fixed stride.  Then the long ones: a workgroup takes the list
// entry of its number, counted from the last workgroup (which has had the fewest
// short strips), then the next untaken entry of a shared counter (ws_count[2],
// zero at launch), so strips of very different lengths spread evenly.  (The other
// way round, the workgroups that had sorted long strips until late started on
// their short ones last: skewed 2*10^6 rows, fp32, height 16, 154 us against 127;
// short ones by a counter too: 129 us, and slower at heights 2 to 8.)  Few long
// rows among short ones are streamed, other strips are merged in LDS while they fit
// (CAP words twice), in the workspace beyond that, and strips with
// unsorted rows go through a bitonic network afterwards.  A strip costs a chain
// of dependent global loads (list entry, row pointers, then entries); the next
// strip's list entry and row pointers are loaded while the current one is sorted.
template <int HB, int NT, typename ET>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void sort_lists_kernel(
    int rows, int height, int bits, const int* __restrict__ row_ptr, const int* __restrict__ col_ind,
    const ET* __restrict__ val_in, uint32_t* __restrict__ col_word, ET* __restrict__ val_out,
    int* __restrict__ ws_count, const int* __restrict__ ws_small, const int* __restrict__ ws_big,
    uint64_t* __restrict__ gkeys) {
    constexpr int E = kWaveSortCap / kWave, CAP = NT * E, NWS = NT / kWave;
    // Behind the slices: what a search of the last one may read, and the light lists
    // of a streamed strip whose STAGE columns fill the rest.
    constexpr int PAD = std::max(merge_pad(E), 3 * kLightCap / 2), STAGE = 2 * CAP;
    // Eight bytes in front: a clamped search reads one word before the first.
    __shared__ __align__(16) uint64_t lds[2 + CAP + PAD];
    __shared__ int rt[HB + 1];
    __shared__ int taken[2];
    __shared__ int wrt[NWS][HB + 1];
    uint64_t* const skeys = lds + 2;
    const int tid = static_cast<int>(threadIdx.x);
    const int lane = lane_id();
    const int wave = uniform(tid / kWave);
    const int scount = ws_count[0], count = ws_count[1];
    for (int it = static_cast<int>(blockIdx.x) * NWS + wave; it < scount; it += static_cast<int>(gridDim.x) * NWS)
        sort_strip_mid<HB, E, NT, ET>(ws_small[it], rows, height, bits, row_ptr, col_ind, val_in, col_word, val_out,
                                      (LdsKey*)skeys + wave * kWaveSortCap, (LdsInt*)wrt[wave], lane);
    __syncthreads();  // the long strips use the slices
    int item = static_cast<int>(gridDim.x - 1 - blockIdx.x);
    if (item < count) {
        if (tid == 0) taken[0] = static_cast<int>(gridDim.x) + atomicAdd(&ws_count[2], 1);
        int strip = ws_big[item];
        int myrp = strip_row_ptr(strip, rows, height, row_ptr, lane);
        __syncthreads();
        int next = taken[0];
        for (int k = 1; item < count; ++k) {
            // The entry after `next` is taken now and read after this strip's
            // last barrier (taken[] alternates, so it is not overwritten early).
            if (tid == 0 && next < count) taken[k & 1] = static_cast<int>(gridDim.x) + atomicAdd(&ws_count[2], 1);
            StripRows sr;
            sr.r0 = strip * height;
            sr.nr = min(height, rows - sr.r0);
            sr.myrp = myrp;
            sr.s0 = __shfl(myrp, 0);
            sr.s1 = __shfl(myrp, sr.nr);
            const int n = sr.s1 - sr.s0;
            const int nstrip = next < count ? ws_big[next] : 0;
            const int nmyrp = next < count ? strip_row_ptr(nstrip, rows, height, row_ptr, lane) : INT_MAX;
            const RunTable rows_of = run_table<HB>(sr, n, lane);
            const bool light = lane < HB && rows_of.len <= kLightRow;
            int incl = light ? rows_of.len : 0;  // light entries up to and with this row
#pragma unroll
            for (int off = 1; off < HB; off <<= 1) {
                const int t = __shfl_up(incl, off);
                if (lane >= off) incl += t;
            }
            const int m = __shfl(incl, HB - 1);
            const int rls = incl - (light ? rows_of.len : 0);
            const uint64_t heavy = ballot(lane < HB && !light);
            uint64_t* const G = gkeys + 2 * static_cast<size_t>(sr.s0);
            bool bad;
            // Streamed: up to kHeavyMax long rows, and up to kHeavyStaged where their
            // columns fit LDS but a merge would not.  (With two long rows of a low
            // strip, a level or two of merging costs 1024 threads less.)
            const int nheavy = __popcll(heavy);
            const bool staged = HB > 1 && nheavy > 1 && n <= STAGE;
            const int most = n <= CAP ? (NT == 1024 && HB <= 4 ? 1 : kHeavyMax) : (staged ? kHeavyStaged : kHeavyMax);
            if (nheavy <= most && m <= kLightCap) {
                uint32_t* LW = reinterpret_cast<uint32_t*>(skeys);
                bad = __syncthreads_or(stream_strip<HB, NT, ET>(
                    sr, rows_of, heavy, m, rls, bits, col_ind, val_in, col_word, val_out, LW, LW + kLightCap,
                    reinterpret_cast<int*>(LW + 2 * kLightCap), reinterpret_cast<int*>(LW + 3 * kLightCap), staged, tid,
                    lane));
            } else {
                if (wave == 0 && lane <= HB) rt[lane] = lane < HB ? rows_of.lo : n;
                __syncthreads();
                LdsWord* A = (LdsWord*)reinterpret_cast<uint32_t*>(skeys);
                if (n <= CAP) {
                    bad = merge_strip_block<HB, NT, E, ET>(sr, n, wave_max(rows_of.len), bits, col_ind, val_in,
                                                           col_word, val_out, A, A + CAP, (LdsInt*)rt, tid);
                } else {
                    bad = merge_strip_global<HB, NT, ET>(sr, n, bits, col_ind, val_in, col_word, val_out, G, rt, tid);
                }
            }
            if (bad) {
                __syncthreads();
                bitonic_strip<HB, NT, CAP, ET>(sr, n, bits, col_ind, val_in, col_word, val_out,
                                                         (LdsKey*)skeys, G, tid);
            }
            __syncthreads();  // the next item reuses skeys and rt
            item = next;
            next = next < count ? taken[k & 1] : count;
            strip = nstrip;
            myrp = nmyrp;
        }
    }
}

__global__ void validate_csr_kernel(int rows, int cols, int nnz, const int* __restrict__ row_ptr,
                                    const int* __restrict__ col_ind, int* __restrict__ flag) {
    const int tid = static_cast<int>(blockIdx.x * blockDim.x + threadIdx.x);
    const int nth = static_cast<int>(gridDim.x * blockDim.x);
    int f = 0;
    if (tid == 0 && (row_ptr[0] != 0 || row_ptr[rows] != nnz)) f |= 1;
    for (int i = tid; i < rows; i += nth)
        if (row_ptr[i + 1] < row_ptr[i]) f |= 2;
    for (int k = tid; k < nnz; k += nth) {
        const int c = col_ind[k];
        if (c < 0 || c >= cols) f |= 4;
    }
    if (f) atomicOr(flag, f);
}

namespace {

// From this mean on every strip is listed.
constexpr double kTallEnd = 3800.0;

inline size_t align256(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }

struct Conv {
    int rows, strips, height, bits, nnz;
};

// Both lists of strips the first kernel could not sort (sort_lists_kernel), by as
// many workgroups as are resident, or fewer when the lists cannot be that long.
// Workgroups of 512 threads, two on a CU, suit a few long strips among short ones and
// strips of up to half an LDS.  Where every strip is listed, 1024 threads merge in LDS
// what 512 take to the workspace (750 strips of 8000 in four rows, 512 / 1024 threads,
// 183/113 us; 428 of 14 000 205/116), and while each has a CU to itself
// they are faster below that too (31 strips of 8000 in four rows 65/33, 41 of 6000
// with unsorted rows 108/89; but 1333 strips of 4500 with one long row, height 4,
// 112/157).  Longer strips fit neither (300 strips of 20 000 in sixteen rows 380/438).
constexpr double kWideLists = 7000.0, kWideListsEnd = 15000.0;
constexpr int kWideListsFew = 256;
template <int HB, int NT, typename ET>
void launch_sort_lists_nt(const Conv& cv, const FromCsrWorkspaceLayout& L, const int* row_ptr, const int* col_ind,
                          const ET* vin, uint32_t* col_word, ET* vout, int* ws_count, const int* ws_small,
                          const int* ws_big, uint64_t* gkeys, hipStream_t stream) {
    constexpr size_t NW = NT / kWave;
    const size_t want = std::max<size_t>(L.big_cap, (L.small_cap + NW - 1) / NW);
    const int g = static_cast<int>(std::max<size_t>(1, std::min<size_t>(want, kListThreads / NT)));
    hipLaunchKernelGGL((sort_lists_kernel<HB, NT, ET>), dim3(g), dim3(NT), 0, stream, cv.rows, cv.height, cv.bits,
                       row_ptr, col_ind, vin, col_word, vout, ws_count, ws_small, ws_big, gkeys);
}

template <int HB, typename ET>
void launch_sort_lists(const Conv& cv, const FromCsrWorkspaceLayout& L, const int* row_ptr, const int* col_ind,
                       const ET* vin, uint32_t* col_word, ET* vout, int* ws_count, const int* ws_small,
                       const int* ws_big, uint64_t* gkeys, hipStream_t stream) {
    const double mean = static_cast<double>(cv.nnz) / cv.strips;
    if (mean >= (cv.strips <= kWideListsFew ? kTallEnd : kWideLists) && mean < kWideListsEnd)
        launch_sort_lists_nt<HB, 1024, ET>(cv, L, row_ptr, col_ind, vin, col_word, vout, ws_count, ws_small, ws_big,
                                           gkeys, stream);
    else
        launch_sort_lists_nt<HB, 512, ET>(cv, L, row_ptr, col_ind, vin, col_word, vout, ws_count, ws_small, ws_big,
                                          gkeys, stream);
}

template <int G, int E, int HB, typename ET>
hipError_t from_csr_g(const Conv& cv, const int* row_ptr, const int* col_ind, const void* val_in,
                      int* strip_ptr, uint32_t* col_word, void* val_out, void* workspace, hipStream_t stream) {
    constexpr int NG = kWave / G;
    const int waves = (cv.strips + NG - 1) / NG;
    const int blocks = (waves + kConvWaves - 1) / kConvWaves;
    const auto* vin = static_cast<const ET*>(val_in);
    auto* vout = static_cast<ET*>(val_out);
    const FromCsrWorkspaceLayout L = from_csr_workspace_layout(cv.rows, cv.nnz, cv.height);
    auto* ws = static_cast<char*>(workspace);
    int* ws_count = reinterpret_cast<int*>(ws);
    int* ws_small = reinterpret_cast<int*>(ws + L.small_off);
    int* ws_big = reinterpret_cast<int*>(ws + L.big_off);
    auto* gkeys = reinterpret_cast<uint64_t*>(ws + L.global_off);
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, stream, ws_count, 4, 0);
    hipLaunchKernelGGL((from_csr_group_kernel<HB, G, E, ET>), dim3(blocks), dim3(kConvThreads), 0, stream,
                       cv.rows, cv.strips, cv.height, cv.bits, cv.nnz, row_ptr, col_ind, vin, strip_ptr, col_word,
                       vout, ws_count, ws_small, ws_big);
    launch_sort_lists<HB, ET>(cv, L, row_ptr, col_ind, vin, col_word, vout, ws_count, ws_small, ws_big, gkeys,
                              stream);
    return hipGetLastError();
}

// Tall strips (from_csr_tall_kernel), then the same list kernel for longer
// ones.
template <int HB, int NT, typename ET>
hipError_t from_csr_tall(const Conv& cv, const int* row_ptr, const int* col_ind, const void* val_in, int* strip_ptr,
                         uint32_t* col_word, void* val_out, void* workspace, hipStream_t stream) {
    const auto* vin = static_cast<const ET*>(val_in);
    auto* vout = static_cast<ET*>(val_out);
    const FromCsrWorkspaceLayout L = from_csr_workspace_layout(cv.rows, cv.nnz, cv.height);
    auto* ws = static_cast<char*>(workspace);
    int* ws_count = reinterpret_cast<int*>(ws);
    int* ws_small = reinterpret_cast<int*>(ws + L.small_off);
    int* ws_big = reinterpret_cast<int*>(ws + L.big_off);
    auto* gkeys = reinterpret_cast<uint64_t*>(ws + L.global_off);
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, stream, ws_count, 4, 0);
    hipLaunchKernelGGL((from_csr_tall_kernel<HB, NT, ET>), dim3(cv.strips), dim3(NT), 0, stream, cv.rows, cv.strips,
                       cv.height, cv.bits, cv.nnz, row_ptr, col_ind, vin, strip_ptr, col_word, vout, ws_count,
                       ws_small, ws_big);
    launch_sort_lists<HB, ET>(cv, L, row_ptr, col_ind, vin, col_word, vout, ws_count, ws_small, ws_big, gkeys,
                              stream);
    return hipGetLastError();
}

// The mean strips that a workgroup of 128, 256 or 512 threads takes one at a time
// (from_csr_tall_kernel): nearly up to its 1024, 2048 or 4096 entries, since a
// longer strip goes to the lists.  Below, a wave of the group kernel holds a strip
// (512 entries) and is faster: means of 384 to 432 entries 149/74/200 us against
// 185/112/248 (band of 81, fp32, height 8; band of 21, fp64, height 32; 27-point
// stencil, fp64, height 16).
constexpr double kTall128Mean = 450.0, kTall256Mean = 900.0, kTall512Mean = 1850.0;
// Up to four strips per CU, where a strip's latency is the kernel's time, take twice
// the threads (128 / 256 threads, height 32: 98 Poisson(15) strips, fp64, 18.7/13.9 us,
// 625 strips 19.1/14.8, 625 27-point stencil strips, fp32, 22.5/17.0; 1875 strips
// 23.9/25.1; 256 / 512 threads, 98 Poisson(40) strips 20.4/15.1).
constexpr int kTallFew = 1024;
// From kBucketHeight on, strips that are all resident at once as workgroups of 128
// (12 on a CU) go that way from a lower mean on: their latency counts, not their
// issue (group kernel / one workgroup each: 2500 strips of Poisson(15) rows, fp64,
// height 24, 23.0/18.8 us; 543 strips of one row of 368 and 31 of 2, height 32,
// 21.8/15.0; but 3750 strips, band of 41, height 16, 24.4/25.7).
constexpr int kTallResident = 3072;
constexpr double kTallMeanFew = 320.0;

template <int HB, typename ET>
hipError_t from_csr_hb(const Conv& cv, const int* row_ptr, const int* col_ind, const void* val_in,
                       int* strip_ptr, uint32_t* col_word, void* val_out, void* workspace, hipStream_t stream) {
    const double mean = static_cast<double>(cv.nnz) / cv.strips;
    const bool few = cv.strips <= kTallFew;
    const double from = HB >= kBucketHeight && cv.strips <= kTallResident ? kTallMeanFew : kTall128Mean;
    if (mean >= from && mean < kTallEnd) {
        if (mean < kTall256Mean && !few)
            return from_csr_tall<HB, 128, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace,
                                              stream);
        if (mean < (few ? kTall256Mean : kTall512Mean))
            return from_csr_tall<HB, 256, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace,
                                              stream);
        return from_csr_tall<HB, 512, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace,
                                          stream);
    }
    const ConvShape sh = conv_shape(cv.nnz, cv.strips, HB);
#define CMRS_FROM_G(GG, EE)                                                                                      \
    if constexpr (GG >= HB) {                                                                                    \
        if (sh.g == GG && sh.e == EE)                                                                            \
            return from_csr_g<GG, EE, HB, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, \
                                              workspace, stream);                                                \
    }
    CMRS_FROM_G(2, 8)
    CMRS_FROM_G(4, 8)
    CMRS_FROM_G(8, 8)
    CMRS_FROM_G(16, 8)
    CMRS_FROM_G(32, 8)
    CMRS_FROM_G(64, 8)
#undef CMRS_FROM_G
    return hipErrorInvalidValue;
}

template <typename ET>
hipError_t from_csr_typed(const Conv& cv, uint32_t flags, const int* row_ptr, const int* col_ind,
                          const void* val_in, int* strip_ptr, uint32_t* col_word, void* val_out, void* workspace,
                          hipStream_t stream) {
    if (!(flags & CMRS_SORT)) {
        const int ns = kRunRows / cv.height;
        const int waves = (cv.strips + ns - 1) / ns;
        const int blocks = (waves + kConvWaves - 1) / kConvWaves;
        hipLaunchKernelGGL((from_csr_rows_kernel<ET>), dim3(blocks), dim3(kConvThreads), 0, stream, cv.rows,
                           cv.strips, cv.height, cv.bits, cv.nnz, ns, row_ptr, col_ind, static_cast<const ET*>(val_in),
                           strip_ptr, col_word, static_cast<ET*>(val_out), val_out != val_in ? 1 : 0);
        return hipGetLastError();
    }
    switch (next_pow2(cv.height)) {
        case 1: return from_csr_hb<1, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
        case 2: return from_csr_hb<2, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
        case 4: return from_csr_hb<4, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
        case 8: return from_csr_hb<8, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
        case 16: return from_csr_hb<16, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
        default: return from_csr_hb<32, ET>(cv, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
    }
}

template <typename ET>
hipError_t to_csr_typed(const cmrs_mat_t* A, int* row_ptr, int* col_ind, void* val_out, hipStream_t stream) {
    if (A->height == 1) {
        const int64_t work = static_cast<int64_t>(A->nnz > A->rows + 1 ? A->nnz : A->rows + 1);
        const int64_t want = (work + 1023) / 1024;
        const int blocks = static_cast<int>(want < 4096 ? want : 4096);
        hipLaunchKernelGGL((to_csr_h1_kernel<ET>), dim3(blocks), dim3(256), 0, stream, A->rows, A->nnz, A->bits,
                           A->strip_ptr, A->col_word, static_cast<const ET*>(A->val), row_ptr, col_ind,
                           static_cast<ET*>(val_out));
        return hipGetLastError();
    }
    const int strips = (A->rows + A->height - 1) / A->height;
    // Whole strips per wave: as many as fit in kRunRows rows (height <= 32).
    const int ns = kRunRows / A->height;
    const int runs = (strips + ns - 1) / ns;
    const int blocks = (runs + kToCsrWaves - 1) / kToCsrWaves;
    // Staged output from height 8 on, for runs of at least kToCsrStage/2.5
    // entries on average (measured: 2^20 rows of Poisson(16), height 32: 160
    // -> 107 us; height 2 and the skewed rows of up to 10^4 entries are faster
    // without).
    const bool stage = A->height >= 8 && static_cast<double>(A->nnz) >= kToCsrStage / 2.5 * runs;
    auto kern = stage ? to_csr_rows_kernel<ET, true> : to_csr_rows_kernel<ET, false>;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kToCsrThreads), 0, stream, A->rows, strips,
                       A->height, A->bits, ns, A->strip_ptr, A->col_word, static_cast<const ET*>(A->val), row_ptr,
                       col_ind, static_cast<ET*>(val_out));
    return hipGetLastError();
}

}  // namespace

FromCsrWorkspaceLayout from_csr_workspace_layout(int32_t rows, int32_t nnz, int32_t height) {
    FromCsrWorkspaceLayout L;
    const size_t strips = height > 0 ? (static_cast<size_t>(rows) + height - 1) / height : 0;
    L.small_off = 256;
    L.small_cap = strips > 0 ? strips : 1;
    L.big_off = align256(L.small_off + 4 * L.small_cap);
    L.big_cap = static_cast<size_t>(nnz) / (kWaveSortCap + 1) + 1;
    L.global_off = align256(L.big_off + 4 * L.big_cap);
    L.total = L.global_off + 16 * static_cast<size_t>(nnz);
    return L;
}

hipError_t launch_from_csr(int32_t rows, int32_t cols, int32_t nnz, const int32_t* row_ptr, const int32_t* col_ind,
                           const void* val_in, cmrs_dtype_t dtype, int32_t height, int32_t bits, uint32_t flags,
                           int32_t* strip_ptr, uint32_t* col_word, void* val_out, void* workspace,
                           hipStream_t stream) {
    (void)cols;
    const int strips = (rows + height - 1) / height;
    if (strips == 0) {
        hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, stream, strip_ptr, 1, nnz);
        return hipGetLastError();
    }
    const Conv cv{rows, strips, height, bits, nnz};
    // No entries: nothing to pack or sort (and the sorted path's workspace is
    // then zero bytes); the group kernel only writes the strip pointers.
    if (nnz == 0) flags &= ~CMRS_SORT;
    switch (dtype_bytes(dtype)) {
        case 8: return from_csr_typed<uint64_t>(cv, flags, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
        case 4: return from_csr_typed<uint32_t>(cv, flags, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
        default: return from_csr_typed<uint16_t>(cv, flags, row_ptr, col_ind, val_in, strip_ptr, col_word, val_out, workspace, stream);
    }
}

hipError_t launch_to_csr(const cmrs_mat_t* A, int32_t* row_ptr, int32_t* col_ind, void* val_out,
                         hipStream_t stream) {
    if (A->rows == 0) {
        hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, stream, row_ptr, 1, 0);
        return hipGetLastError();
    }
    switch (dtype_bytes(A->val_dtype)) {
        case 8: return to_csr_typed<uint64_t>(A, row_ptr, col_ind, val_out, stream);
        case 4: return to_csr_typed<uint32_t>(A, row_ptr, col_ind, val_out, stream);
        default: return to_csr_typed<uint16_t>(A, row_ptr, col_ind, val_out, stream);
    }
}

hipError_t launch_validate_csr(int32_t rows, int32_t cols, int32_t nnz, const int32_t* row_ptr,
                               const int32_t* col_ind, int32_t* flag, hipStream_t stream) {
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, stream, flag, 1, 0);
    int work = rows > nnz ? rows : nnz;
    int g = (work + 255) / 256;
    if (g < 1) g = 1;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(validate_csr_kernel, dim3(g), dim3(256), 0, stream, rows, cols, nnz, row_ptr, col_ind, flag);
    return hipGetLastError();
}

}  // namespace cmrs
