// Dense packing (Sec. 4.3): window-based greedy selection of the retained sequences into
// rows of `capacity` tokens. The placement is sequential by definition (each one changes the
// remaining space and refills the pool), so ONE workgroup does everything: 16 wavefronts compact
// and validate the kept items, one wavefront places them, and all 16 turn the order into offsets.
// Integer work only; the result is a bit-exact function of the inputs.
//
// What bounds it is the latency of one placement: a wavefront alone on its compute unit issues an
// instruction about every 7 cycles, and reading the pool from memory costs 600 to 2000 cycles. The placing wavefront therefore keeps
// the pool in registers, oldest item in the lowest lane: a ballot finds the oldest item that fits (first-fit
// reading) or a DPP max the longest one (best-fit), and no memory is touched between two placements.
// A taken branch, or a VALU result that the scalar unit waits for, costs several instructions more, so first-fit's loop over rows is straight-line code with one look (at the slots, the
// stream and the row ends together) per row.
// Measured (8 500 prompts, pool of 32, about 2 950 rows): first-fit 0.51 ms (3.07 with the pool in global memory and one wavefront for
// everything; 0.75 with a branch for each of those looks, in every row and around every search), best-fit 1.28 ms.
// Compaction and offsets, spread over 16 wavefronts: 18 us.
#include "dppo_internal.h"

namespace dppo {
namespace {

constexpr int WAVE = 64;
constexpr int PACK_THREADS = 1024, PACK_WAVES = PACK_THREADS / WAVE;
constexpr int EMPTY = -1;                         // length of a placed or absent item: as unsigned, larger than any space left
// Stream lengths held in LDS up to this many items (60 KB: no attribute needed for the dynamic LDS of a
// launch); longer streams keep them in the caller's cu array, read through the L2.
constexpr int LDS_ITEMS = 15360;
// With at most this many loss positions the packing workgroup writes them itself; beyond, a grid-wide
// kernel does (its launch costs about 5 us, which one workgroup needs for 30 K positions).
constexpr int64_t INLINE_LOSS_POS = 16384;

__device__ __forceinline__ int64_t wave_sum64(int64_t v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    return v;
}

__device__ __forceinline__ int64_t wave_max64(int64_t v) {
    for (int off = 32; off > 0; off >>= 1) {
        int64_t o = __shfl_xor(v, off, WAVE);
        v = o > v ? o : v;
    }
    return v;
}

// Wave-wide maximum and inclusive prefix sum by DPP moves (registers only; a shuffle goes through the LDS unit).
// The maximum takes every row's broadcast in every row behind it: taking a value twice does no harm.
__device__ __forceinline__ uint32_t wave_max_dpp(uint32_t v) {
    auto step = [&](uint32_t o) { v = o > v ? o : v; };
    step(__builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true));   // row_shr:1
    step(__builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true));   // row_shr:2
    step(__builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true));   // row_shr:4
    step(__builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true));   // row_shr:8
    step(__builtin_amdgcn_update_dpp(0, v, 0x142, 0xf, 0xf, true));   // row_bcast:15
    step(__builtin_amdgcn_update_dpp(0, v, 0x143, 0xf, 0xf, true));   // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ uint32_t wave_scan_dpp(uint32_t v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

__device__ __forceinline__ bool fits_in(int len, int rem) { return (uint32_t)len <= (uint32_t)rem; }

// Set bits of m below this lane.
__device__ __forceinline__ int bits_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

__device__ __forceinline__ uint64_t mask_below(int n) { return n >= 64 ? ~0ull : (1ull << n) - 1ull; }
// Mask of the lanes below n (any integer), by one compare.
__device__ __forceinline__ uint64_t lanes_below(int n) { return __ballot((int)(threadIdx.x & (WAVE - 1)) < n); }

// Window-based greedy placement by one wavefront, pool of n_win <= 64 R - 32 items in registers.
// The pool occupies the slots 0, 1, ... (slot = 64 r + lane) in arrival order; a placed item leaves a
// hole and its slot remembers its position in the order. The slots behind the pool already hold the
// stream items that will be fetched next, so a refill only moves `limit`, the number of slots that
// count as fetched. Once the slots run out, the order is written and the pool closed up again (at least
// 32 placements later). order[] receives stream indices.
// First-fit begins a row with the run of oldest items whose lengths add up to at most the capacity; the
// prefix sums for that are kept up to date, so the whole run is one step, as dear as one
// placement in the search for later items that still fit.
// lens: stream lengths (LDS or global); moved: 64 R ints of LDS. Returns the number of rows.
template <int R, bool BEST>
__device__ __forceinline__ int place_pool(int S, int capacity, int n_win, const int32_t* lens, int32_t* moved, int32_t* order,
                                          int32_t* row_ptr) {
    const int lane = threadIdx.x & (WAVE - 1);
    constexpr int SLOTS = WAVE * R;
    int idx[R], at[R];                   // stream index, position in the order once placed
    uint32_t len[R], sum[R];             // length; lengths of the slots up to this one, less the placed ones that were out of turn
    uint64_t open[R];                    // slots with an item that is not placed
    uint32_t base = 0;                   // sum[] - base = lengths of the open slots up to here, for every open slot
    int cnt0 = 0, next0 = 0, pos0 = 0;   // at the last closing-up: kept items, first stream item behind them, items placed
    int limit = n_win, pos = 0, rows = 0;
    auto fill = [&](int kept) {
        base = 0;
        uint32_t before = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int q = r * WAVE + lane;
            idx[r] = q < kept ? moved[q] : next0 + (q - cnt0);
            int l = idx[r] < S ? lens[idx[r]] : 0;
            asm volatile("" : "+v"(l));  // waits for the load here, not (and for the stores to order[]) at every placement
            len[r] = l;
            at[r] = -1;
            open[r] = __ballot(idx[r] < S);
            if (!BEST) {
                sum[r] = before + wave_scan_dpp(l);
                before = __builtin_amdgcn_readlane(sum[r], WAVE - 1);
            }
        }
    };
    fill(0);
    auto write_order = [&]() {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (at[r] >= 0) order[at[r]] = idx[r];
    };
    auto fetched_slots = [&](int r) -> uint64_t { return open[r] & __ballot(r * WAVE + lane < limit); };
    auto close_up = [&]() {
        write_order();
        limit = limit < SLOTS ? limit : SLOTS;
        const int fetched = next0 + (limit - cnt0);
        int n = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t keep = fetched_slots(r);
            if (__builtin_amdgcn_inverse_ballot_w64(keep)) moved[n + bits_below(keep)] = idx[r];
            n += __popcll(keep);
        }
        __builtin_amdgcn_wave_barrier();
        cnt0 = n; next0 = fetched; pos0 = pos; limit = n_win;    // the pool holds n_win items while the stream lasts
        fill(n);
        __builtin_amdgcn_wave_barrier();
    };

    int row_end = 0;                     // lane i: items placed up to the end of row 64 k + i, written out 64 rows at a time
    if (lane == 0) row_ptr[0] = 0;
    auto end_row = [&]() __attribute__((always_inline)) {
        row_end = lane == (rows & (WAVE - 1)) ? pos : row_end;
        rows += 1;
    };
    auto write_rows = [&]() __attribute__((always_inline)) {
        if ((rows & (WAVE - 1)) == 0) row_ptr[rows - WAVE + 1 + lane] = row_end;
    };
    while (BEST && pos < S) {
        uint32_t rem = capacity;
        while (true) {
            uint64_t ok[R];
            uint32_t v = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                ok[r] = fetched_slots(r) & __ballot(len[r] <= rem);
                const uint32_t l = __builtin_amdgcn_inverse_ballot_w64(ok[r]) ? len[r] : 0;
                v = l > v ? l : v;
            }
            const uint32_t want = wave_max_dpp(v);       // the longest length that fits
            bool placed = false;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint64_t mm = ok[r] & __ballot(len[r] == want);
                if (placed || mm == 0) continue;
                const int f = __builtin_ctzll(mm);
                at[r] = lane == f ? pos : at[r];
                open[r] &= ~(1ull << f);
                placed = true;
            }
            if (!placed) break;
            rem -= want;
            pos += 1;
            limit += 1;
            if (limit > SLOTS) close_up();
        }
        end_row();
        write_rows();
    }
    // first-fit: places the run of oldest items (all slots before it are placed; its own refills follow in turn)
    uint32_t rem = 0;
    auto run_step = [&](bool may_be_empty) __attribute__((always_inline)) {
        const uint32_t top = base + rem;              // both below 2^31
        int n = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t in = __ballot(sum[r] <= top);              // sum[] never falls from slot to slot
            const uint64_t run = in & open[r];
            at[r] = __builtin_amdgcn_inverse_ballot_w64(run) ? bits_below(run) + (pos + n) : at[r];
            open[r] &= ~in;
            n += __popcll(run);
            const int here = __popcll(in);
            if ((r == 0 && !may_be_empty) || here > 0) base = __builtin_amdgcn_readlane(sum[r], here - 1);
        }
        pos += n;
        limit += n;
        rem = top - base;
    };
    // and the later items that still fit, oldest first
    auto later_items = [&]() __attribute__((always_inline)) {
        auto next_slots = [&](uint64_t (&ok)[R]) __attribute__((always_inline)) -> uint64_t {
            uint64_t any = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                ok[r] = __ballot(len[r] <= rem) & open[r] & lanes_below(limit - r * WAVE);
                any |= ok[r];
            }
            return any;
        };
        uint64_t ok[R];
        for (uint64_t any = next_slots(ok); any != 0; any = next_slots(ok)) {
            uint32_t l = 0;
            bool placed = false;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (placed) {                         // behind the placed item's register
                    sum[r] -= l;
                } else if (r == R - 1 || ok[r] != 0) {
                    const int f = __builtin_ctzll(ok[r]);
                    l = __builtin_amdgcn_readlane(len[r], f);
                    at[r] = lane == f ? pos : at[r];
                    open[r] &= ~(1ull << f);
                    sum[r] -= lane >= f ? l : 0;
                    placed = true;
                }
            }
            rem -= l;
            pos += 1;
            limit += 1;
        }
    };
    // Rows are ended one after the other, without a look at anything else, as long as neither the slots, nor the stream, nor
    // the 64 row ends of the register run out.
    while (!BEST && pos < S) {
        const int stop = S < pos0 + (SLOTS - n_win) ? S : pos0 + (SLOTS - n_win), last_row = rows | (WAVE - 1);
        while (true) {
            rem = capacity;
            run_step(false);                          // (a row begins with the oldest item, which fits)
            later_items();
            if (((pos - stop) & (rows - last_row)) >= 0) break;
            end_row();
        }
        // the search may have run past the last slot: the items it could not fetch are the newest, which the scan of this row
        // reaches last anyway
        while (pos < S && pos - pos0 >= SLOTS - n_win) {
            close_up();
            run_step(true);
            later_items();
        }
        end_row();
        write_rows();
    }
    write_order();
    if (lane < (rows & (WAVE - 1))) row_ptr[(rows & ~(WAVE - 1)) + 1 + lane] = row_end;
    return rows;
}

// The same for pools beyond the register window: the pool is the set of items not yet placed among the
// first `next` of the stream, `lens` (EMPTY once placed) is scanned 64 items at a time.
__device__ __forceinline__ int place_scan(int S, int capacity, int n_win, int policy, int32_t* lens_, int32_t* order, int32_t* row_ptr) {
    const int lane = threadIdx.x & (WAVE - 1);
    volatile int32_t* lens = lens_;
    int next = n_win < S ? n_win : S;
    int lo = 0;                         // every stream item below lo is placed
    int pos = 0, rows = 0;
    if (lane == 0) row_ptr[0] = 0;
    while (pos < S) {
        int rem = capacity;
        if (policy == DPPO_PACK_BEST_FIT) {
            // longest pool item that fits, oldest among equals; repeat until none fits
            while (true) {
                int64_t best = -1;
                for (int i0 = lo; i0 < next; i0 += WAVE) {
                    int i = i0 + lane;
                    int len = (i < next) ? lens[i] : EMPTY;
                    if (fits_in(len, rem)) {
                        int64_t key = ((int64_t)len << 32) | (int64_t)(0x7fffffff - i);
                        best = key > best ? key : best;
                    }
                }
                best = wave_max64(best);
                if (best < 0) break;
                const int sel = 0x7fffffff - (int)(best & 0xffffffffLL);
                if (lane == 0) {
                    order[pos] = sel;
                    lens[sel] = EMPTY;
                }
                __threadfence_block();   // the mark must be visible to the next scan
                rem -= (int)(best >> 32);
                pos += 1;
                if (next < S) next += 1;
            }
        } else
        for (int i0 = lo; i0 < next; i0 += WAVE) {
            int i = i0 + lane;
            int len = (i < S) ? lens[i] : EMPTY;
            uint64_t done = 0;                        // lanes already passed by the scan
            while (true) {
                bool fits = fits_in(len, rem) && i < next;
                uint64_t m = __ballot(fits) & ~done;
                if (m == 0) break;
                int f = __ffsll((unsigned long long)m) - 1;
                rem -= __builtin_amdgcn_readlane(len, f);
                if (lane == f) {
                    order[pos] = i;
                    lens[i] = EMPTY;
                    len = EMPTY;
                }
                pos += 1;
                if (next < S) next += 1;             // refill the pool from the stream
                done = mask_below(f + 1);
            }
        }
        rows += 1;
        if (lane == 0) row_ptr[rows] = pos;
        __threadfence_block();   // placed marks must be visible to the reloads below
        // advance lo past the placed prefix
        while (lo < S) {
            int i = lo + lane;
            bool unplaced = (i < S) && lens[i] != EMPTY;
            uint64_t m = __ballot(unplaced);
            if (m != 0) { lo += __ffsll((unsigned long long)m) - 1; break; }
            lo += WAVE;
        }
        if (lo > S) lo = S;
    }
    return rows;
}

__device__ __forceinline__ int place(int S, int capacity, int n_win, int policy, int32_t* lens, int32_t* moved, int32_t* order,
                                     int32_t* row_ptr) {
    const bool best = policy == DPPO_PACK_BEST_FIT;
    if (n_win <= WAVE - 32)
        return best ? place_pool<1, true>(S, capacity, n_win, lens, moved, order, row_ptr)
                    : place_pool<1, false>(S, capacity, n_win, lens, moved, order, row_ptr);
    if (n_win <= 2 * WAVE - 32)
        return best ? place_pool<2, true>(S, capacity, n_win, lens, moved, order, row_ptr)
                    : place_pool<2, false>(S, capacity, n_win, lens, moved, order, row_ptr);
    return place_scan(S, capacity, n_win, policy, lens, order, row_ptr);
}

__device__ void write_loss_pos(int s, const int32_t* order, const int32_t* prompt_len, const int32_t* cu, const int32_t* lcu,
                               int32_t* loss_pos, int t0, int step) {
    const int first = cu[s] + prompt_len[order[s]] - 1;
    const int a = lcu[s], b = lcu[s + 1];
    for (int t = a + t0; t < b; t += step) loss_pos[t] = first + (t - a);
}

__global__ __launch_bounds__(PACK_THREADS) void pack_kernel(
    int n_items, int capacity, int n_win, int policy, const int32_t* __restrict__ prompt_len,
    const int32_t* __restrict__ comp_len, const uint8_t* __restrict__ keep, int32_t* order,
    int32_t* row_ptr, int32_t* cu /* scratch: stream lengths of a stream beyond LDS_ITEMS */,
    int32_t* lcu /* scratch: stream item -> original index */, int32_t* loss_pos, int64_t loss_pos_capacity,
    int inline_loss_pos, int32_t* meta) {
    extern __shared__ int32_t s_len[];             // min(n_items, LDS_ITEMS) stream lengths
    __shared__ int64_t s_a[PACK_WAVES], s_b[PACK_WAVES], s_c[PACK_WAVES];
    __shared__ int s_n[PACK_WAVES], s_bad[PACK_WAVES], s_rows;
    __shared__ int32_t s_moved[2 * WAVE];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int32_t* lens = n_items <= LDS_ITEMS ? s_len : cu;

    // ---- compact the kept items into the stream, validate, total T and N: every wavefront takes one
    // contiguous range of items, counts its kept ones, and writes them behind those of the ranges before ----
    const int min_c = comp_len != nullptr ? 1 : 0;   // prompts alone: no completion part
    const int64_t per_wave = ((int64_t)n_items + PACK_THREADS - 1) / PACK_THREADS * WAVE;
    const int64_t j_lo = wave * per_wave, j_hi = j_lo + per_wave < n_items ? j_lo + per_wave : n_items;
    {
        int n = 0, bad = 0;
        int64_t T = 0, N = 0, longest = 1;
        for (int64_t j = j_lo + lane; j - lane < j_hi; j += WAVE) {
            const bool kept = j < j_hi && (keep == nullptr || keep[j] != 0);
            const int P = kept ? prompt_len[j] : 1;
            const int C = (kept && comp_len != nullptr) ? comp_len[j] : min_c;
            const int64_t len = (int64_t)P + (int64_t)C;
            if (kept) {
                if (P < 1 || C < min_c || len > 0x7fffffffLL) bad = 1;
                longest = len > longest ? len : longest;
                T += len;
                N += C;
            }
            n += __popcll(__ballot(kept));
        }
        T = wave_sum64(T); N = wave_sum64(N); longest = wave_max64(longest);
        bad = __any(bad) ? 1 : 0;
        if (lane == 0) { s_n[wave] = n; s_bad[wave] = bad; s_a[wave] = T; s_b[wave] = N; s_c[wave] = longest; }
    }
    __syncthreads();
    int S = 0, at = 0, bad = 0;
    int64_t T = 0, N = 0, longest = 1;
    for (int w = 0; w < PACK_WAVES; ++w) {
        if (w == wave) at = S;
        S += s_n[w];
        bad |= s_bad[w];
        T += s_a[w]; N += s_b[w];
        longest = s_c[w] > longest ? s_c[w] : longest;
    }
    if (capacity == 0) capacity = (int)(longest > 0x7fffffffLL ? 0x7fffffff : longest);   // L_max = longest item
    int status = 0;
    if (bad || longest > (int64_t)capacity) status = 1;
    else if (N > loss_pos_capacity) status = 2;
    else if (T > 0x7fffffffLL) status = 3;
    if (status != 0) {
        if (tid == 0) {
            meta[0] = 0; meta[1] = 0; meta[2] = 0; meta[3] = status;
            meta[4] = 0; meta[5] = capacity; meta[6] = 0; meta[7] = 0;
            row_ptr[0] = 0; cu[0] = 0; lcu[0] = 0;
        }
        return;
    }
    for (int64_t j = j_lo + lane; j - lane < j_hi; j += WAVE) {
        const bool kept = j < j_hi && (keep == nullptr || keep[j] != 0);
        const uint64_t m = __ballot(kept);
        if (kept) {
            const int p = at + bits_below(m);
            lens[p] = prompt_len[j] + (comp_len != nullptr ? comp_len[j] : 0);
            lcu[p] = (int32_t)j;
        }
        at += __popcll(m);
    }
    __syncthreads();   // the stream is read by other lanes below

    // ---- window-based greedy placement: order[] = stream indices ------------------------
    if (wave == 0) {
        int rows;
        // two copies, so that the lengths are read by LDS instructions where they are in LDS: a load through a
        // generic pointer would wait for the stores to order[] that are still under way
        if (n_items <= LDS_ITEMS) rows = place(S, capacity, n_win, policy, s_len, s_moved, order, row_ptr);
        else rows = place(S, capacity, n_win, policy, cu, s_moved, order, row_ptr);
        if (lane == 0) s_rows = rows;
    }
    __syncthreads();

    // ---- offsets of the packed sequences: every wavefront sums one contiguous range, then scans it ----
    const int64_t s_per_wave = ((int64_t)S + PACK_THREADS - 1) / PACK_THREADS * WAVE;
    const int64_t s_lo = wave * s_per_wave < S ? wave * s_per_wave : S;
    const int64_t s_hi = s_lo + s_per_wave < S ? s_lo + s_per_wave : S;
    {
        int64_t a = 0, b = 0;
        for (int64_t s = s_lo + lane; s < s_hi; s += WAVE) {
            const int j = lcu[order[s]];
            order[s] = j;                             // stream index -> original index
            const int C = comp_len != nullptr ? comp_len[j] : 0;
            a += prompt_len[j] + C;
            b += C;
        }
        a = wave_sum64(a); b = wave_sum64(b);
        if (lane == 0) { s_a[wave] = a; s_b[wave] = b; }
    }
    __syncthreads();                                  // (lcu is rewritten below)
    int tok = 0, ltok = 0;                            // totals fit int32 (status 3)
    for (int w = 0; w < wave; ++w) { tok += (int)s_a[w]; ltok += (int)s_b[w]; }
    for (int64_t s0 = s_lo; s0 < s_hi; s0 += WAVE) {
        const int64_t s = s0 + lane;
        const int j = s < s_hi ? order[s] : 0;
        const int C = (s < s_hi && comp_len != nullptr) ? comp_len[j] : 0;
        int a = s < s_hi ? prompt_len[j] + C : 0, b = C;
        for (int off = 1; off < WAVE; off <<= 1) {    // inclusive scan over the wave
            const int ta = __shfl_up(a, off, WAVE), tb = __shfl_up(b, off, WAVE);
            if (lane >= off) { a += ta; b += tb; }
        }
        if (s < s_hi) {
            cu[s + 1] = tok + a;
            lcu[s + 1] = ltok + b;
        }
        tok += __shfl(a, WAVE - 1, WAVE);
        ltok += __shfl(b, WAVE - 1, WAVE);
    }
    if (tid == 0) {
        cu[0] = 0; lcu[0] = 0;
        const int rows = s_rows;
        meta[0] = rows; meta[1] = (int32_t)T; meta[2] = (int32_t)N; meta[3] = 0;
        meta[4] = S; meta[5] = capacity;
        // fill density T / (rows * capacity) as the two halves of a double (low word first)
        const double dens = rows > 0 ? (double)T / ((double)rows * (double)capacity) : 0.0;
        const uint64_t bits = (uint64_t)__double_as_longlong(dens);
        meta[6] = (int32_t)(uint32_t)(bits & 0xffffffffull); meta[7] = (int32_t)(uint32_t)(bits >> 32);
    }
    if (!inline_loss_pos) return;
    __syncthreads();
    for (int s = wave; s < S; s += PACK_WAVES) write_loss_pos(s, order, prompt_len, cu, lcu, loss_pos, lane, WAVE);
}

// loss_pos of every packed sequence: one workgroup per sequence (grid-strided).
__global__ void loss_pos_kernel(const int32_t* __restrict__ meta, const int32_t* __restrict__ order,
                                const int32_t* __restrict__ prompt_len, const int32_t* __restrict__ cu,
                                const int32_t* __restrict__ lcu, int32_t* __restrict__ loss_pos) {
    const int S = meta[4];
    for (int s = blockIdx.x; s < S; s += gridDim.x)
        write_loss_pos(s, order, prompt_len, cu, lcu, loss_pos, threadIdx.x, blockDim.x);
}

__global__ void gather_f32_kernel(int64_t n, const int32_t* __restrict__ idx, const float* __restrict__ src,
                                  float* __restrict__ dst) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[idx[i]];
}

}  // namespace

void launch_pack(const dppo_pack_params& p, const int32_t* prompt_len, const int32_t* comp_len,
                 const uint8_t* keep, int32_t* order, int32_t* row_ptr, int32_t* cu, int32_t* lcu,
                 int32_t* loss_pos, int64_t loss_pos_capacity, int32_t* meta, hipStream_t st) {
    const size_t lds = (size_t)(p.n_items < LDS_ITEMS ? p.n_items : LDS_ITEMS) * 4;
    const int inline_pos = comp_len != nullptr && loss_pos_capacity <= INLINE_LOSS_POS ? 1 : 0;
    pack_kernel<<<1, PACK_THREADS, lds, st>>>(p.n_items, p.capacity, p.n_win, p.policy, prompt_len, comp_len, keep, order,
                                              row_ptr, cu, lcu, loss_pos, loss_pos_capacity, inline_pos, meta);
    if (comp_len == nullptr || inline_pos) return;   // prompts alone: no loss positions
    int blocks = p.n_items < 2048 ? p.n_items : 2048;
    loss_pos_kernel<<<blocks, 256, 0, st>>>(meta, order, prompt_len, cu, lcu, loss_pos);
}

void launch_gather_f32(int64_t n, const int32_t* idx, const float* src, float* dst, hipStream_t st) {
    if (n <= 0) return;
    gather_f32_kernel<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(n, idx, src, dst);
}

}  // namespace dppo
