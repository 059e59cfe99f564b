// Sub-graph construction (Algorithm 1 Step-2 with the intra-community probability knob of
// Section 4.2): per-layer fanout sampling, frontier de-duplication in first-appearance order,
// CSR blocks with local column ids and their transposes.  Integer arithmetic only; a whole group of
// mini-batches is sampled by one set of launches (blockIdx.y = batch within the group).
#include "cr_common.h"
#include <type_traits>

namespace cr {

constexpr uint64_t KEY_MAX = ~0ull;
constexpr uint64_t EMPTY = ~0ull;

// ---------------------------------------------------------------------------------------------
// integer exponential clock: E(r) = -log2((2r+1)/2^33) in Q24, one result bit per squaring
// ---------------------------------------------------------------------------------------------
// COMPACT: the squarings as a loop (for the rarely taken exact paths of kernels whose common path should keep its
// registers: unrolled, four of these chains side by side cost the weighted kernel half its occupancy)
template <bool COMPACT = false>
__device__ __forceinline__ uint32_t exp_clock_q24(uint32_t r)
{
    const uint64_t x = 2ull * r + 1ull;
    const int t = 63 - __clzll((long long)x);
    uint32_t y = (uint32_t)((x << (63 - t)) >> 32);
    uint32_t frac = 0;
    constexpr int UNROLL = COMPACT ? 1 : 24;
#pragma unroll UNROLL
    for (int i = 0; i < 24; ++i) {
        const uint32_t hi = __umulhi(y, y), lo = y * y;
        const bool top = (hi >> 31) != 0;
        y = top ? hi : ((hi << 1) | (lo >> 31));
        frac = (frac << 1) | (top ? 1u : 0u);
    }
    return ((uint32_t)(33 - t) << 24) - frac;
}

struct ScanArgs {
    const int32_t *prev_hdr;
    int64_t n_roots_total;
    int32_t batch_size;
    int32_t mode;          // 0: row counts -> indptr ; 1: new-node counts -> offsets ; 2: source counts -> t_indptr ;
                           // 3: n_fixed values per batch, no header involved ;
                           // 4: as 0, the counts min(fanout, degree) taken here (blocks of one tile)
    const int32_t *in;
    int64_t in_stride;
    int32_t *out;
    int64_t out_stride;
    int32_t *out_copy;     // mode 2: fill cursors
    int64_t copy_stride;
    int32_t *hdr;
    int32_t n_fixed;
    const int32_t *tile_before;   // optional (one batch only): sum of everything in front of each tile, computed beforehand
    int32_t cap_src;              // mode 1: entries the frontier array holds
    int64_t *async_status;        // mode 1: status words of the caller's context, or NULL
    const int64_t *g_indptr;      // mode 4
    const int32_t *dst_ids;
    int64_t dst_stride;
    int32_t fanout;
    int32_t *head_ids;            // mode 4, input-side block in global ids: takes the destination nodes too, or NULL
    int64_t head_stride;
    int32_t *zero;                // [G][n_zero] words to clear for a later kernel of the hop, or NULL
    int32_t n_zero;               // at most SCAN_THREADS
};

struct SelectArgs {
    const int64_t *g_indptr;
    const int32_t *g_indices;
    const int32_t *comm;
    const uint32_t *edge_intra;   // one bit per adjacency entry (same community), or NULL
    int64_t n_entries;
    const int32_t *dst_ids;   // roots, or the frontier of the layer above
    int64_t dst_stride;
    const int32_t *prev_hdr;  // header array of the layer above, NULL for the root layer
    int64_t n_roots_total;
    int32_t batch_size;
    int32_t fanout;
    uint32_t q_in, q_out;
    uint32_t strict_p1;       // drop inter-community picks (only meaningful when q_out == 0)
    uint32_t seed_lo, seed_hi, ctr3, first_batch;
    int32_t *sel;             // [G][cap_dst*fanout] chosen global neighbour ids, rows in slot order
    int64_t sel_stride;
    int32_t *cnt;             // [G][cap_dst]
    int64_t cnt_stride;
    uint32_t cand_target;     // long rows, uniform sampling: expected number of slots below the pre-filter threshold
    // Direct output (input-side block left in global ids, every row keeps min(fanout, degree) neighbours): the row
    // pointers are known before anything is selected, so the chosen ids go straight to their place in the block's
    // per-edge id array and the intermediate [row][fanout] array is not written at all.
    const int32_t *out_indptr;   // [G][out_indptr_stride] or NULL
    int64_t out_indptr_stride;
    int32_t *out_ids;            // [G][out_stride]
    int64_t out_stride;
    int32_t rows_per_wave;       // destination rows a wave of select_quad_kernel takes (at most QUAD_ROWS)
    uint32_t exact_select;       // verification aid: no pre-filter thresholds, every ranking on full (key, slot) pairs
    int32_t scan_here;           // 1: select_quad_kernel works out the row pointers itself (`scan`, as mode 4 of scan_kernel)
    ScanArgs scan;
};

// where the chosen neighbours of a row go, and (when they go to the intermediate array) the row's count
__device__ __forceinline__ int32_t *sel_row_ptr(const SelectArgs &a, int g, int row)
{
    if (a.out_indptr) return a.out_ids + (int64_t)g * a.out_stride + a.out_indptr[(int64_t)g * a.out_indptr_stride + row];
    return a.sel + (int64_t)g * a.sel_stride + (int64_t)row * a.fanout;
}
__device__ __forceinline__ void set_row_count(const SelectArgs &a, int g, int row, int n)
{
    if (!a.out_indptr) a.cnt[(int64_t)g * a.cnt_stride + row] = n;
}

__device__ __forceinline__ int group_n_dst(const int32_t *prev_hdr, int g, int64_t n_roots_total, int batch_size)
{
    if (prev_hdr) return prev_hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_N_SRC];
    const int64_t left = n_roots_total - (int64_t)g * batch_size;
    return (int)(left < 0 ? 0 : (left > batch_size ? batch_size : left));
}

__device__ __forceinline__ uint32_t rl32(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ uint64_t rl64(uint64_t v, int lane)
{
    return ((uint64_t)rl32((uint32_t)(v >> 32), lane) << 32) | rl32((uint32_t)v, lane);
}
__device__ __forceinline__ uint32_t push32(uint32_t v, int dst_lane) { return (uint32_t)__builtin_amdgcn_ds_permute(dst_lane << 2, (int)v); }
__device__ __forceinline__ uint64_t push64(uint64_t v, int dst_lane)
{
    return ((uint64_t)push32((uint32_t)(v >> 32), dst_lane) << 32) | push32((uint32_t)v, dst_lane);
}

__device__ __forceinline__ bool edge_is_intra(const SelectArgs &a, int64_t e) { return (a.edge_intra[e >> 5] >> (e & 31)) & 1u; }

__device__ __forceinline__ uint32_t pull32(uint32_t v, int src_lane) { return (uint32_t)__builtin_amdgcn_ds_bpermute(src_lane << 2, (int)v); }
__device__ __forceinline__ int lanes_below(uint64_t mask, int acc)      // acc + number of set bits below this lane
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, (uint32_t)acc));
}

// ordering key of slot j of node v given its random word: narrow mode (p = 0.5) uses the word itself
// MODE: 0 uniform (p = 0.5), 1 p = 1 (classes only, no clock), 2 weighted (0.5 < p < 1)
template <int MODE, bool COMPACT = false>
__device__ __forceinline__ uint64_t slot_key(const SelectArgs &a, uint32_t r, bool intra)
{
    if (MODE == 0) return r;
    if (MODE == 1) return (intra ? 0ull : (1ull << 62)) + (uint64_t)r;
    return (uint64_t)exp_clock_q24<COMPACT>(r) * (uint64_t)(intra ? a.q_out : a.q_in);
}

__device__ __forceinline__ uint32_t slot_word(const SelectArgs &a, int j, int32_t v, uint32_t batch)
{
    const u32x4 w = philox4x32_10((uint32_t)j >> 2, (uint32_t)v, batch, a.ctr3, a.seed_lo, a.seed_hi);
    const uint32_t pick = (uint32_t)j & 3u;
    return pick == 0 ? w.x : (pick == 1 ? w.y : (pick == 2 ? w.z : w.w));
}

// A row with more than 64 neighbours, handled by a whole wave.  A slot's ordering value is the pair
// (key, slot); with WIDE == false (p = 0.5, 32-bit keys) the pair is packed into one 64-bit word.
// Lanes 0..k-1 hold the k smallest pairs seen so far in ascending order: the first 64 slots are ranked
// by counting and permuted into place, later chunks of 64 slots are tested against the k-th pair and
// inserted by shifting.  Every pair is distinct, so the surviving set is unique.
template <int MODE, bool COMPACT = false>
__device__ __forceinline__ void select_big_row(const SelectArgs &a, int g, int row, int32_t *sel_row, int32_t v, int64_t base, int deg, int32_t cv,
                                            int lane)
{
    constexpr bool WIDE = MODE != 0;
    const int f = a.fanout;
    const int k = f;
    const uint32_t batch = a.first_batch + (uint32_t)g;
    auto less = [&](uint64_t ka, uint32_t sa, uint64_t kb, uint32_t sb) -> bool {
        if (!WIDE) return ka < kb;
        return ka < kb || (ka == kb && sa < sb);
    };
    auto make_key = [&](uint32_t r, int j, bool intra, uint64_t &ck, uint32_t &cs) {
        if (!WIDE) {
            ck = ((uint64_t)r << 32) | (uint32_t)j;
            cs = 0;
        } else {
            ck = slot_key<MODE, COMPACT>(a, r, intra);
            cs = (uint32_t)j;
        }
    };
    // neighbour class look-ups are clamped to the row, so they can be issued ahead unconditionally
    auto load_u = [&](int j) -> int32_t { return a.g_indices[base + min(j, deg - 1)]; };

    // first chunk: rank the first 64 slots by counting, then move rank r to lane r
    uint64_t ck = KEY_MAX;
    uint32_t cs = 0xFFFFFFFFu;
    // class of slot j (clamped to the row): one bit when the graph carries them, else two dependent look-ups
    auto cls = [&](int j) -> bool {
        if (a.edge_intra) return edge_is_intra(a, base + min(j, deg - 1));
        return a.comm[load_u(j)] == cv;
    };
    {
        bool intra = false;
        if (WIDE) intra = cls(lane);
        make_key(slot_word(a, lane, v, batch), lane, intra, ck, cs);
        int rank = 0;
        for (int j = 0; j < WAVE; ++j) {
            const uint64_t kj = rl64(ck, j);
            const uint32_t sj = WIDE ? rl32(cs, j) : 0u;
            rank += less(kj, sj, ck, cs) ? 1 : 0;
        }
        ck = push64(ck, rank);
        if (WIDE) cs = push32(cs, rank);
    }

    // later chunks: a slot that beats the current k-th pair is inserted by shifting the sorted lanes
    uint64_t tk = rl64(ck, k - 1);
    uint32_t ts = WIDE ? rl32(cs, k - 1) : 0u;
    auto offer = [&](bool have, uint64_t nk, uint32_t ns) {
        uint64_t pass = __ballot(have && less(nk, ns, tk, ts));
        while (pass) {
            const int src = __ffsll((long long)pass) - 1;
            pass &= pass - 1;
            const uint64_t xk = rl64(nk, src);
            const uint32_t xs = WIDE ? rl32(ns, src) : 0u;
            if (less(xk, xs, tk, ts)) {
                const int pos = __popcll(__ballot(lane < k && less(ck, cs, xk, xs)));
                const uint64_t upk = __shfl_up(ck, 1);
                const uint32_t ups = WIDE ? __shfl_up(cs, 1) : 0u;
                if (lane > pos) { ck = upk; cs = ups; }
                if (lane == pos) { ck = xk; cs = xs; }
                tk = rl64(ck, k - 1);
                ts = WIDE ? rl32(cs, k - 1) : 0u;
            }
        }
    };
    if (!WIDE) {
        // uniform sampling needs no neighbour data at all: one Philox block gives a lane the words of
        // four consecutive slots, so an iteration covers 256 slots with arithmetic only
        for (int j0 = WAVE; j0 < deg; j0 += 4 * WAVE) {
            const int jb = j0 + 4 * lane;
            const u32x4 w = philox4x32_10((uint32_t)jb >> 2, (uint32_t)v, batch, a.ctr3, a.seed_lo, a.seed_hi);
            const uint32_t wr[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) offer(jb + i < deg, ((uint64_t)wr[i] << 32) | (uint32_t)(jb + i), 0u);
        }
    } else if (a.edge_intra) {
        // biased sampling needs the class of every neighbour; here it is one bit, fetched one chunk ahead
        bool c1 = cls(WAVE + lane);
        for (int j0 = WAVE; j0 < deg; j0 += WAVE) {
            const bool c2 = cls(j0 + WAVE + lane);
            const int j = j0 + lane;
            uint64_t nk = KEY_MAX;
            uint32_t ns = 0xFFFFFFFFu;
            if (j < deg) make_key(slot_word(a, j, v, batch), j, c1, nk, ns);
            offer(j < deg, nk, ns);
            c1 = c2;
        }
    } else {
        // without the bits: ids are fetched two chunks ahead and classes one chunk ahead, so the dependent
        // look-ups overlap the arithmetic
        int32_t u1 = load_u(WAVE + lane);
        int32_t c1 = a.comm[u1];
        int32_t u2 = load_u(2 * WAVE + lane);
        for (int j0 = WAVE; j0 < deg; j0 += WAVE) {
            const int32_t c2 = a.comm[u2];
            const int32_t u3 = load_u(j0 + 2 * WAVE + lane);
            const int j = j0 + lane;
            uint64_t nk = KEY_MAX;
            uint32_t ns = 0xFFFFFFFFu;
            if (j < deg) make_key(slot_word(a, j, v, batch), j, c1 == cv, nk, ns);
            offer(j < deg, nk, ns);
            c1 = c2;
            u2 = u3;
        }
    }

    // emit in ascending slot order
    const uint32_t slot = WIDE ? cs : (uint32_t)ck;
    const bool valid = lane < k && !(WIDE && a.strict_p1 && ck >= (1ull << 62));
    int32_t cu = 0;
    if (valid) cu = a.g_indices[base + slot];
    int rank = 0;
    for (int i = 0; i < k; ++i) {
        const uint32_t si = rl32(slot, i);
        const uint32_t vi = rl32(valid ? 1u : 0u, i);
        rank += (vi && si < slot) ? 1 : 0;
    }
    const uint64_t vmask = __ballot(valid);
    if (valid) sel_row[rank] = cu;
    if (lane == 0) set_row_count(a, g, row, __popcll(vmask));
}

// Uniform sampling of a row with more than 64 neighbours, the common way: slots whose random word falls
// below a threshold chosen so that about cand_target of them do (far more than the fanout, far fewer than
// the wave's candidate buffer holds) are compacted in slot order into LDS, ranked among themselves by
// counting, and the fanout smallest (word, slot) pairs are emitted in slot order.  Exact whenever it
// applies: every slot left out has a word >= the threshold > every candidate's word.  Returns false when
// the candidates are fewer than the fanout or more than the buffer holds (then the caller takes the
// general path, which needs no threshold).
constexpr int CAND_CAP = 128;

// sum over the wave, the same in all lanes: operand modifiers inside rows of sixteen lanes, four lane reads across them (no LDS)
__device__ __forceinline__ int wave_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true);      // quad [1 0 3 2]
    x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true);      // quad [2 3 0 1]
    x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true);     // half mirror
    x += __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, true);     // mirror
    return (__builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16)) + (__builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48));
}

// (Rows of more than 256 neighbours ranked each of their ~50 to 100 candidates against all of them, about 150 issue slots, and when
// weighted reduced four extremes over the wave by shuffles.  A bound found by search, and one look for keys too near to it, in
// their place: reddit-like, 8 batches, p = 0.9, the call 343 -> 317 us; products-like, 32 batches, uniform 867 -> 835,
// p = 0.9 1309 -> 1236; papers-like 931 -> 895.)
// A bound with exactly k of the wave's words below it, searched as in the passes of short rows (see quad_pass): moved inside
// (0, hi) to where evenly spread words would put it.  count(T): words below the bound that x stands for; to_word(x): that bound.
// All arguments and results are the same in every lane.  false: no such bound found (equal words around it, or too many steps).
template <typename ToWord, typename Count>
__device__ __forceinline__ bool search_bound(int n, int k, float hi, ToWord &&to_word, Count &&count, uint32_t &T)
{
    float lo = 0.0f, at_lo = (float)k + 0.5f, at_hi = (float)(n - k) + 0.5f;
    for (int step = 0; step < 24; ++step) {
        const float x = lo + (hi - lo) * (at_lo * __builtin_amdgcn_rcpf(at_lo + at_hi));
        T = to_word(x);
        const int off = count(T) - k;
        if (off == 0) return true;
        if (off < 0) { lo = x; at_lo = 0.5f - (float)off; }
        else { hi = x; at_hi = 0.5f + (float)off; }
    }
    return false;
}

// INTRA_ONLY is the same for p = 1 when the graph carries its edge-class bits: the pool is the row's
// intra-community slots (counted from the bits first); with fewer of them than the fanout the caller's general
// path fills up with inter-community ones.
template <bool INTRA_ONLY>
__device__ __forceinline__ bool select_big_row_filtered(const SelectArgs &a, int g, int row, int32_t *sel_row, int32_t v, int64_t base, int deg,
                                                        int lane, uint32_t *ckey /*[CAND_CAP + 4]*/, uint32_t *cslot /*[CAND_CAP]*/)
{
    const int k = a.fanout;
    const uint32_t batch = a.first_batch + (uint32_t)g;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    int pool = deg;
    if (INTRA_ONLY) {
        const int64_t w_first = base >> 5, e_last = base + deg, w_last = (e_last - 1) >> 5;
        int n_in = 0;
        for (int64_t w = w_first + lane; w <= w_last; w += WAVE) {
            uint32_t bits = a.edge_intra[w];
            if (w == w_first) bits &= ~0u << (base & 31);
            if (w == w_last && (e_last & 31)) bits &= (1u << (e_last & 31)) - 1u;
            n_in += __popc(bits);
        }
        n_in = wave_sum(n_in);
        if (n_in < k) return false;
        pool = n_in;
    }
    const int64_t w_max = (a.n_entries - 1) >> 5;
    // (float arithmetic: the threshold only steers how many candidates there are, any value gives the same result)
    const float thr_f = (float)a.cand_target * 4294967296.0f / (float)pool;
    const bool keep_all = thr_f >= 4294967040.0f;                  // every slot of the pool is to be a candidate
    const uint32_t thr = keep_all ? 0xFFFFFFFFu : (uint32_t)thr_f;
    int n = 0;
    // 256 slots from j0 on; a slot is a candidate iff its word is below thr and it belongs to the pool (of the right class,
    // and, in the row's last stretch, not beyond its end).  false: more candidates than the list holds.
    auto stretch = [&](int j0, auto is_last) -> bool {
        constexpr bool LAST = decltype(is_last)::value;
        const int jb = j0 + 4 * lane;
        const u32x4 w = philox4x32_10((uint32_t)jb >> 2, (uint32_t)v, batch, a.ctr3, a.seed_lo, a.seed_hi);
        const uint32_t wr[4] = {w.x, w.y, w.z, w.w};
        uint32_t nib = 0xFu;          // which of the lane's four slots belong to the pool
        if (INTRA_ONLY) {
            const int64_t e = base + min(jb, deg - 1);
            const int64_t wi = e >> 5;
            const uint64_t win = (uint64_t)a.edge_intra[wi] | ((uint64_t)a.edge_intra[min(wi + 1, w_max)] << 32);
            nib = (uint32_t)(win >> (e & 31)) & 0xFu;
        }
        if (LAST) {
            const int left = deg - jb;
            nib &= left >= 4 ? 0xFu : (left > 0 ? (1u << left) - 1u : 0u);
        }
        bool c[4];
        uint64_t b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t t = (INTRA_ONLY || LAST) ? (((nib >> i) & 1u) ? thr : 0u) : thr;
            c[i] = wr[i] < t;
            b[i] = __ballot(c[i]);
        }
        if ((b[0] | b[1] | b[2] | b[3]) == 0) return true;             // (most stretches of a very long row)
        int before = n;
#pragma unroll
        for (int i = 0; i < 4; ++i) before = lanes_below(b[i], before);
        const int total = __popcll(b[0]) + __popcll(b[1]) + __popcll(b[2]) + __popcll(b[3]);
        if (n + total > CAND_CAP) return false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (c[i]) { ckey[before] = wr[i]; cslot[before] = (uint32_t)(jb + i); }
            before += c[i] ? 1 : 0;
        }
        n += total;
        return true;
    };
    int j0 = 0;
    for (; j0 + 4 * WAVE <= deg; j0 += 4 * WAVE)
        if (!stretch(j0, std::false_type{})) return false;
    if (j0 < deg && !stretch(j0, std::true_type{})) return false;
    // (a word of all ones is never below the threshold: with every slot wanted, leave such a row to the general path)
    if (keep_all && n != pool) return false;
    if (n < k) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // candidate t sits at index t in slot order; a lane owns candidates lane and lane + 64.  Words only are compared: with
    // equal words at the boundary there is no bound, and the caller's general path takes the row.
    const bool have0 = lane < n, have1 = lane + WAVE < n;
    const uint32_t w0 = have0 ? ckey[lane] : ~0u, w1 = have1 ? ckey[lane + WAVE] : ~0u;
    uint32_t T;
    const bool exact = search_bound(n, k, thr_f, [](float x) { return (uint32_t)x; },
                                    [&](uint32_t t) { return (int)__popcll(__ballot(w0 < t)) + (n > WAVE ? (int)__popcll(__ballot(w1 < t)) : 0); }, T);
    const bool s0 = w0 < T, s1 = w1 < T;
    const uint64_t m0 = __ballot(s0), m1 = __ballot(s1);
    if (exact) {
        if (s0) sel_row[__popcll(m0 & lt_mask)] = a.g_indices[base + cslot[lane]];
        if (s1) sel_row[__popcll(m0) + __popcll(m1 & lt_mask)] = a.g_indices[base + cslot[lane + WAVE]];
        if (lane == 0) set_row_count(a, g, row, k);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the buffers are reused by this wave's next long row
    return exact;
}

// Long rows for 0.5 < p < 1, with the graph's edge-class bits.  A slot's key is E(r) * m with m = 1-p for an
// intra-community slot and p for an inter-community one, E a non-increasing function of the random word r, so
// "key below kappa" is "r at or above a per-class threshold".  kappa is chosen (float arithmetic, a few Newton steps
// on the expected candidate count; its value only affects how many candidates there are) so that about cand_target
// slots pass; only those get the 24-squaring clock.  The result is exact iff the fanout-th smallest candidate key
// is below the smallest key any left-out slot can have, E(threshold - 1) * m per class in integer arithmetic: that is
// checked, and otherwise (or with too few / too many candidates) the caller takes the general path.
template <bool COMPACT = false>
__device__ __forceinline__ bool select_big_row_weighted(const SelectArgs &a, int g, int row, int32_t *sel_row, int32_t v, int64_t base, int deg,
                                                        int lane, uint2 *cand, unsigned long long *ckey)
{
    const int k = a.fanout;
    const uint32_t batch = a.first_batch + (uint32_t)g;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    const int64_t w_first = base >> 5, e_last = base + deg, w_last = (e_last - 1) >> 5;
    int n_in = 0;
    for (int64_t w = w_first + lane; w <= w_last; w += WAVE) {
        uint32_t bits = a.edge_intra[w];
        if (w == w_first) bits &= ~0u << (base & 31);
        if (w == w_last && (e_last & 31)) bits &= (1u << (e_last & 31)) - 1u;
        n_in += __popc(bits);
    }
#pragma unroll
    for (int o = 32; o; o >>= 1) n_in += __shfl_xor(n_in, o);
    const int n_out = deg - n_in;

    // per-class thresholds on the random word: candidate iff r >= t_class
    uint64_t t_in = 0, t_out = 0;
    if ((int)a.cand_target < deg) {
        const float ln2 = 0.69314718f, target = (float)a.cand_target;
        const float s_in = 1.0f / ((float)a.q_out * 16777216.0f), s_out = 1.0f / ((float)a.q_in * 16777216.0f);
        const float fi = (float)n_in, fo = (float)n_out;
        float kappa = target / (ln2 * (fi * s_in + fo * s_out));       // tangent at zero: never past the root
#pragma unroll
        for (int it = 0; it < 3; ++it) {
            const float ei = exp2f(-kappa * s_in), eo = exp2f(-kappa * s_out);
            const float gv = fi * (1.0f - ei) + fo * (1.0f - eo) - target;
            const float gd = ln2 * (fi * s_in * ei + fo * s_out * eo);
            if (gd > 0.0f) kappa -= gv / gd;
        }
        const float pi = exp2f(-kappa * s_in) * 4294967296.0f, po = exp2f(-kappa * s_out) * 4294967296.0f;
        t_in = pi >= 4294967296.0f ? 0x100000000ull : (uint64_t)(pi > 0.0f ? pi : 0.0f);
        t_out = po >= 4294967296.0f ? 0x100000000ull : (uint64_t)(po > 0.0f ? po : 0.0f);
    }
    // smallest key a slot that is left out can have (lane 0: intra, lane 1: inter), exact integers
    uint64_t bound;
    {
        const uint64_t t = lane == 0 ? t_in : t_out;
        const uint32_t m = lane == 0 ? a.q_out : a.q_in;
        const int pool = lane == 0 ? n_in : n_out;
        const uint64_t e = (uint64_t)exp_clock_q24<COMPACT>((uint32_t)(t > 0 ? t - 1 : 0)) * m;
        const uint64_t mine = (t == 0 || pool == 0) ? KEY_MAX : e;
        const uint64_t b0 = rl64(mine, 0), b1 = rl64(mine, 1);
        bound = b0 < b1 ? b0 : b1;
    }

    const int64_t w_max = (a.n_entries - 1) >> 5;
    int n = 0;
    for (int j0 = 0; j0 < deg; j0 += 4 * WAVE) {
        const int jb = j0 + 4 * lane;
        const u32x4 w = philox4x32_10((uint32_t)jb >> 2, (uint32_t)v, batch, a.ctr3, a.seed_lo, a.seed_hi);
        const uint32_t wr[4] = {w.x, w.y, w.z, w.w};
        const int64_t e = base + min(jb, deg - 1);
        const int64_t wi = e >> 5;
        const uint64_t win = (uint64_t)a.edge_intra[wi] | ((uint64_t)a.edge_intra[min(wi + 1, w_max)] << 32);
        const uint32_t nib = (uint32_t)(win >> (e & 31)) & 0xFu;
        bool c[4];
        uint64_t b[4];
        int before = n, total = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c[i] = jb + i < deg && (uint64_t)wr[i] >= (((nib >> i) & 1u) ? t_in : t_out);
            b[i] = __ballot(c[i]);
            before += __popcll(b[i] & lt_mask);
            total += __popcll(b[i]);
        }
        if (n + total > CAND_CAP) return false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (c[i]) cand[before] = make_uint2(wr[i], (uint32_t)(jb + i) | (((nib >> i) & 1u) << 31));
            before += c[i] ? 1 : 0;
        }
        n += total;
    }
    if (n < k) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // keys of the candidates only; candidate t sits at index t in slot order, a lane owns candidates lane and lane + 64
    const uint2 c0 = cand[min(lane, n - 1)], c1 = cand[min(lane + WAVE, n - 1)];
    const bool have0 = lane < n, have1 = lane + WAVE < n;
    const uint64_t key0 = (uint64_t)exp_clock_q24<COMPACT>(c0.x) * ((c0.y >> 31) ? a.q_out : a.q_in);
    uint64_t key1 = KEY_MAX;
    if (n > WAVE) key1 = (uint64_t)exp_clock_q24<COMPACT>(c1.x) * ((c1.y >> 31) ? a.q_out : a.q_in);
    if (have0) ckey[lane] = key0;
    if (have1) ckey[lane + WAVE] = key1;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int r0 = 0, r1 = 0;
    if (n <= WAVE) {
        for (int t = 0; t < n; ++t) {
            const uint64_t kt = ckey[t];
            r0 += (kt < key0 || (kt == key0 && t < lane)) ? 1 : 0;
        }
    } else {
        for (int t = 0; t < n; ++t) {
            const uint64_t kt = ckey[t];
            r0 += (kt < key0 || (kt == key0 && t < lane)) ? 1 : 0;
            r1 += (kt < key1 || (kt == key1 && t < lane + WAVE)) ? 1 : 0;
        }
    }
    // the fanout-th smallest candidate key must beat everything that was left out
    const uint64_t q0 = __ballot(have0 && r0 == k - 1), q1 = __ballot(have1 && r1 == k - 1);
    const uint64_t kth = q0 ? rl64(key0, __ffsll((long long)q0) - 1) : rl64(key1, __ffsll((long long)q1) - 1);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // both buffers are reused by this wave's next long row
    if (!(kth < bound)) return false;

    const bool s0 = have0 && r0 < k, s1 = have1 && r1 < k;
    const uint64_t m0 = __ballot(s0), m1 = __ballot(s1);
    if (s0) sel_row[__popcll(m0 & lt_mask)] = a.g_indices[base + (c0.y & 0x7FFFFFFFu)];
    if (s1) sel_row[__popcll(m0) + __popcll(m1 & lt_mask)] = a.g_indices[base + (c1.y & 0x7FFFFFFFu)];
    if (lane == 0) set_row_count(a, g, row, k);
    return true;
}

// A wave takes SEL_ROWS consecutive destination rows.  Rows with at most 64 neighbours are packed side
// by side into the wave's lanes (lane = one neighbour slot of one row; as many consecutive rows per pass
// as fit), so that the random words, the keys and the ranking of several short rows cost one pass of
// instructions: a row with deg <= fanout keeps every neighbour, otherwise the slots whose (key, slot)
// pair ranks below the fanout inside their row survive; output keeps slot order.  Longer rows go through
// select_big_row one at a time.
constexpr int SEL_ROWS = 8;

template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void select_kernel(SelectArgs a)
{
    constexpr bool WIDE = MODE != 0;
    __shared__ uint2 cand[4][CAND_CAP];
    __shared__ unsigned long long ckey[MODE == 2 ? 4 : 1][MODE == 2 ? CAND_CAP : 1];
    const int g = blockIdx.y;
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);
    const int row0 = (int)(blockIdx.x * 4 + threadIdx.x / WAVE) * SEL_ROWS;
    if (row0 >= n_dst) return;
    const int lane = lane_id();
    const int f = a.fanout;
    const uint32_t batch = a.first_batch + (uint32_t)g;

    // lanes 0..SEL_ROWS-1 fetch one row's node id, adjacency range and community each
    int32_t mv = 0, mcv = 0;
    int64_t mbase = 0;
    int mdeg = 0;
    if (lane < SEL_ROWS && row0 + lane < n_dst) {
        mv = a.dst_ids[(int64_t)g * a.dst_stride + row0 + lane];
        mbase = a.g_indptr[mv];
        const int64_t d = a.g_indptr[mv + 1] - mbase;
        mdeg = (int)(d > 0x7FFFFFFF ? 0x7FFFFFFF : d);
        if (WIDE) mcv = a.comm[mv];
        if (mdeg == 0) set_row_count(a, g, row0 + lane, 0);
    }
    int32_t v[SEL_ROWS], cv[SEL_ROWS];
    int deg[SEL_ROWS], start[SEL_ROWS], pass[SEL_ROWS];
    int64_t base[SEL_ROWS];
    int off = 0, last_pass = 0;
#pragma unroll
    for (int i = 0; i < SEL_ROWS; ++i) {
        v[i] = (int32_t)rl32((uint32_t)mv, i);
        cv[i] = WIDE ? (int32_t)rl32((uint32_t)mcv, i) : 0;
        deg[i] = (int)rl32((uint32_t)mdeg, i);
        base[i] = (int64_t)rl64((uint64_t)mbase, i);
        // greedy packing of the short rows into passes of at most 64 lanes
        pass[i] = -1;
        start[i] = 0;
        if (deg[i] > 0 && deg[i] <= WAVE) {
            if (off + deg[i] > WAVE) { ++last_pass; off = 0; }
            pass[i] = last_pass;
            start[i] = off;
            off += deg[i];
        }
    }

    for (int p = 0; p <= last_pass; ++p) {
        int ri = -1, my_start = 0, my_len = 0, maxlen = 0;
        int32_t my_v = 0, my_cv = 0;
        int64_t my_base = 0;
#pragma unroll
        for (int i = 0; i < SEL_ROWS; ++i) {
            if (pass[i] != p) continue;                       // uniform
            if (deg[i] > f) maxlen = max(maxlen, deg[i]);
            if (lane >= start[i] && lane < start[i] + deg[i]) {
                ri = i; my_start = start[i]; my_len = deg[i]; my_v = v[i]; my_cv = cv[i]; my_base = base[i];
            }
        }
        const bool active = ri >= 0;
        if (__ballot(active) == 0) continue;
        const int j = lane - my_start;
        int32_t u = 0;
        if (active) u = a.g_indices[my_base + j];
        bool intra = false;
        if (WIDE && active && (maxlen > 0 || a.strict_p1)) intra = a.edge_intra ? edge_is_intra(a, my_base + j) : a.comm[u] == my_cv;
        bool survivor = active && !(WIDE && a.strict_p1 && !intra);
        if (maxlen > 0) {
            // every lane computes its slot's key; lanes of rows that keep all their neighbours ignore it
            const uint64_t ck = slot_key<MODE>(a, slot_word(a, j, my_v, batch), intra);
            int rank = 0;
            for (int d0 = 0; d0 < maxlen; d0 += 4) {          // four independent lane exchanges in flight per step
                uint64_t ok[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int src = my_start + d0 + q;
                    if (WIDE) ok[q] = ((uint64_t)pull32((uint32_t)(ck >> 32), src) << 32) | pull32((uint32_t)ck, src);
                    else ok[q] = pull32((uint32_t)ck, src);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int d = d0 + q;
                    rank += (d < my_len && (ok[q] < ck || (ok[q] == ck && d < j))) ? 1 : 0;
                }
            }
            if (active && my_len > f) survivor = rank < f && !(WIDE && a.strict_p1 && ck >= (1ull << 62));
        }
        const uint64_t seg = (my_len >= WAVE ? ~0ull : ((1ull << my_len) - 1ull)) << my_start;
        const uint64_t smask = __ballot(survivor) & seg;
        if (active) {
            const int row = row0 + ri;
            if (survivor) sel_row_ptr(a, g, row)[__popcll(smask & ((1ull << lane) - 1ull))] = u;
            if (j == 0) set_row_count(a, g, row, __popcll(smask));
        }
    }

#pragma unroll
    for (int i = 0; i < SEL_ROWS; ++i)
        if (deg[i] > WAVE) {
            uint2 *buf = cand[threadIdx.x / WAVE];
            if (MODE == 2 && !a.exact_select && a.edge_intra &&
                select_big_row_weighted(a, g, row0 + i, sel_row_ptr(a, g, row0 + i), v[i], base[i], deg[i], lane, buf, ckey[threadIdx.x / WAVE])) continue;
            select_big_row<MODE>(a, g, row0 + i, sel_row_ptr(a, g, row0 + i), v[i], base[i], deg[i], cv[i], lane);
        }
}

// ---------------------------------------------------------------------------------------------
// Selection with four neighbour slots per lane: uniform sampling, and p = 1 on a graph that carries its edge-class bits
// ---------------------------------------------------------------------------------------------
// One Philox block yields the random words of four consecutive slots, so a lane owns a "quad" of slots and a pass of the
// wave covers 256 slots of consecutive destination rows laid side by side (a row of up to 256 slots never straddles two
// passes).  Both settings reduce to "keep the m smallest words of a pool of P slots, and all of the rest that is kept":
//   uniform        pool = the row, m = min(fanout, degree);
//   p = 1          with n_in >= fanout intra-community slots the pool is those and m = fanout; with fewer, all of them are
//                  kept and the pool is the inter-community slots with m = fanout - n_in (0 in strict mode).
// The kept slots are those below a bound T with exactly m words of the pool below it.  T is found by search: it is moved
// inside a bracket to where evenly spread words would put it, and the words below it are counted per row with four ballots
// and population counts under the row's mask of lanes (about 30 instructions a step, no LDS; simulated on random words: 3 to 4
// steps a row, 5 to 6 for the slowest row of a pass).  The kernel is bound by vector instruction issue; ranking every slot
// against a list of its row's candidates in LDS, which this replaces, took 426 M vector instructions in the input-side hop of a
// products-like group of 32 batches against 312 M.  Selection of that group (uniform, three hops): 792 -> 630 us; of a
// papers-like one 910 -> 804 us; weighted, a reddit-like group of 8: 222 -> 193 us.  Then three of a step's ballots added up as masks,
// the bracket's counts kept as distances and a quad's ids in one load: 647 -> 622 us for the first of these.  A row without such a bound in SEARCH_STEPS steps (equal words at the boundary) is
// redone with (word, slot) pairs compared in full, so the result is exact in every case.
//
// Weighted sampling (0.5 < p < 1) takes the same passes with single-precision keys: approx_clock(r) * m_class, compared
// through their bit patterns (all positive).  They decide only WHICH slots are kept (the output is in slot order), so the
// result is exact whenever no key lies within its error bound of T; that is checked per row, and a row that fails is redone
// with the exact integer keys.  A redone row costs its wave some 8000 instructions (counted in the code, not measured), as much
// as ten passes, and so a launch its tail: with T left wherever the search ended a reddit-like group's selection took 223 us,
// with T moved off the keys 193.
// The error bound: |approx_clock(r) * 2^24 - E(r)| <= CLOCK_ERR_ABS + CLOCK_ERR_REL * E(r), E in its Q24 units, for every one of
// the 2^32 words, with a factor of two to spare; cr_selftest_clock_approximation measures it on the device.
constexpr float CLOCK_ERR_ABS = 8.0f;             // Q24 units
constexpr float CLOCK_ERR_REL = 0x1p-17f;       // (measured: 3 units / 2^-19)

__device__ __forceinline__ float approx_clock(uint32_t r)
{
    // (2r+1) / 2^33 below one half: 33 - log2(2r+1), the argument rounded to 24 bits.  Above: the distance from one,
    // d = 2^33 - (2r+1), is converted instead, so that the small clocks -- the ones that get picked -- keep their
    // relative precision.
    // (one logarithm: the argument is chosen first; the instruction runs at a quarter of the rate of ordinary ones)
    const bool far = r < 0x80000000u;
    const float arg = far ? (float)(2u * r + 1u) : 1.0f - (float)(2u * ~r + 1u) * 0x1p-33f;
    const float lg = __builtin_amdgcn_logf(arg);
    return far ? 33.0f - lg : __builtin_fabsf(lg);
}

// Is every key of the kept side provably below every key of the left-out side?  hi = the largest approximate key kept
// (class weight m_hi), lo = the smallest approximate key left out (class weight m_lo; +infinity: nothing there).  A key's
// error: its clock's (CLOCK_ERR_ABS + CLOCK_ERR_REL * E, times the class weight) plus the rounding of the product; the
// last term covers the rounding of this comparison itself.
__device__ __forceinline__ bool keys_apart(float hi, float m_hi, float lo, float m_lo)
{
    if (!(lo < INFINITY)) return true;
    const float slack = (hi + lo) * (CLOCK_ERR_REL + 0x1p-21f) + CLOCK_ERR_ABS * 0x1p-24f * (m_hi + m_lo);
    return lo - hi > slack;
}

constexpr int QUAD_ROWS = 32;            // destination rows per wave, ...
constexpr int QUAD_MIN_ROWS = 2;         // ... and as few as this
constexpr int QUAD_FILL_WAVES = 8192;    // until there are this many waves (eight per SIMD)
constexpr int QUAD_MAX_DEG = 4 * WAVE;   // longest row a pass holds
constexpr int SEARCH_STEPS = 24;         // bounds tried before a row is ranked in full

// acc + number of set bits, in one instruction (the compiler takes two and an addition apart)
__device__ __forceinline__ uint32_t bits_onto(uint32_t bits, uint32_t acc)
{
    uint32_t n;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(n) : "v"(bits), "v"(acc));
    return n;
}

struct alignas(16) QuadRow {
    int32_t v, deg;                      // node, degree
    int64_t base;                        // first adjacency entry
    int64_t out;                         // where the row's chosen ids go, counted from the group's array
    int64_t pad;
};

// One pass over the rows packed into it: lane `lane` (below `used`) holds quad lane - first of the wave's r-th row.  Returns
// the rows that have to be redone exactly.
template <int MODE, bool EXACT>
__device__ __forceinline__ uint32_t quad_pass(const SelectArgs &a, int g, int row0, int r, int first, int used, const QuadRow *rows,
                                              int32_t *out, uint32_t *klist, unsigned long long *k64, int lane)
{
    const int f = a.fanout;
    const uint32_t batch = a.first_batch + (uint32_t)g;
    const QuadRow R = rows[r];
    const bool active = lane < used;
    const int qi = lane - first, nq = (R.deg + 3) >> 2;
    const int jb = 4 * qi;
    const int left = active ? R.deg - jb : 0;
    const uint32_t vmask = left >= 4 ? 0xFu : ((1u << left) - 1u);        // the quad's slots that exist
    const u32x4 w = philox4x32_10((uint32_t)qi, (uint32_t)R.v, batch, a.ctr3, a.seed_lo, a.seed_hi);
    const uint32_t wr[4] = {w.x, w.y, w.z, w.w};

    // the row's lanes of this pass; counts over a row are population counts of ballots under this mask: no LDS round trips
    const uint64_t row_lanes = active ? (nq >= WAVE ? ~0ull : ((1ull << nq) - 1ull) << first) : 0ull;
    // (three of the four ballots are first added up bit by bit, in scalar registers: two counted bits fewer per lane)
    const uint32_t lanes_lo = (uint32_t)row_lanes, lanes_hi = (uint32_t)(row_lanes >> 32);
    auto count4_onto = [&](int base, bool f0, bool f1, bool f2, bool f3) -> int {          // base + set flags in the whole row
        const uint64_t b0 = __ballot(f0), b1 = __ballot(f1), b2 = __ballot(f2), b3 = __ballot(f3);
        const uint64_t half = b0 ^ b1, ones = half ^ b2, twos = (b0 & b1) | (half & b2);
        auto onto = [&](uint64_t b, uint32_t acc) { return bits_onto((uint32_t)(b >> 32) & lanes_hi, bits_onto((uint32_t)b & lanes_lo, acc)); };
        return (int)((onto(twos, 0u) << 1) + onto(b3, onto(ones, (uint32_t)base)));
    };
    auto count4 = [&](bool f0, bool f1, bool f2, bool f3) -> int { return count4_onto(0, f0, f1, f2, f3); };
    auto before4 = [&](bool f0, bool f1, bool f2, bool f3) -> int {         // ... and in the row's lanes before this one
        const uint64_t b0 = __ballot(f0), b1 = __ballot(f1), b2 = __ballot(f2), b3 = __ballot(f3);
        const uint64_t half = b0 ^ b1, ones = half ^ b2, twos = (b0 & b1) | (half & b2);
        return 2 * lanes_below(twos & row_lanes, 0) + lanes_below(b3 & row_lanes, lanes_below(ones & row_lanes, 0));
    };
    auto count_bits = [&](uint32_t m4) { return count4(m4 & 1u, m4 & 2u, m4 & 4u, m4 & 8u); };
    auto before_bits = [&](uint32_t m4) { return before4(m4 & 1u, m4 & 2u, m4 & 4u, m4 & 8u); };

    uint32_t pool = vmask, take = 0u;
    int m = min(f, R.deg), P = R.deg, expect = m;
    uint32_t nib = 0u;
    int n_in = 0;
    if (MODE >= 1) {
        if (active) {
            const int64_t e = R.base + jb, wi = e >> 5, w_max = (a.n_entries - 1) >> 5;
            const uint64_t win = (uint64_t)a.edge_intra[wi] | ((uint64_t)a.edge_intra[min(wi + 1, w_max)] << 32);
            nib = (uint32_t)(win >> (e & 31)) & 0xFu;
        }
        n_in = count_bits(nib & vmask);
    }
    if (MODE == 1) {
        const uint32_t in4 = nib & vmask;
        if (n_in >= f) {
            pool = in4; m = f; P = n_in; expect = f;
        } else {
            take = in4; pool = vmask & ~nib; P = R.deg - n_in;
            m = a.strict_p1 ? 0 : min(f - n_in, P);
            expect = n_in + m;
        }
    }
    const bool ranked = active && m > 0 && m < P;
    if (!ranked) {
        if (m >= P) take |= pool;           // the whole pool is kept
        pool = 0u;
    }
    // the ordering words of the lane's four slots: the random words themselves, or (weighted) the bit patterns of the
    // single-precision keys
    uint32_t kw[4] = {wr[0], wr[1], wr[2], wr[3]};
    if (MODE == 2 && !EXACT) {
#pragma unroll
        for (int i = 0; i < 4; ++i) kw[i] = __float_as_uint(approx_clock(wr[i]) * (float)(((nib >> i) & 1u) ? a.q_out : a.q_in));
    }
    uint32_t emit;
    int epos;
    bool ok = true;
    if constexpr (!EXACT) {
        // slots kept without a ranking lie below every bound, slots outside the pool above every one
        const uint32_t none = ~(pool | take);
#pragma unroll
        for (int i = 0; i < 4; ++i) kw[i] = (kw[i] & (uint32_t)((int32_t)(pool << (31 - i)) >> 31)) | (uint32_t)((int32_t)(none << (31 - i)) >> 31);
        // A bound T with `expect` words of the row below it: T is moved inside a bracket to where evenly spread words would put it
        // (lo, hi: the bracket's ends; at_lo, at_hi: how many words, and half a word, their counts are off).  x is T itself
        // (weighted: the bound's place in a single exponential law of the row's mean rate); float arithmetic only steers T, the
        // counts are what decides.  A row that is done has lo = hi and keeps its T.
        float lo = 0.0f, at_lo = (float)m + 0.5f, hi = 4294967296.0f, at_hi = (float)(P - m) + 0.5f;
        float to_key = 1.0f;
        if (MODE == 2) {
            // the law's rate: the slots' mean rate for the first of them, that of the mean waiting time for the last (with the
            // mean rate alone, rows of few slots more than the fanout take 8 to 20 steps at p = 0.97, with this 3 to 5)
            const float fi = (float)n_in, fo = (float)(P - n_in), w_in = (float)a.q_out, w_out = (float)a.q_in;
            const float fr = at_lo * __builtin_amdgcn_rcpf((float)P + 1.0f), p_f = (float)P;
            const float rate = (fi * __builtin_amdgcn_rcpf(w_in) + fo * __builtin_amdgcn_rcpf(w_out)) * __builtin_amdgcn_rcpf(p_f);
            const float late = p_f * __builtin_amdgcn_rcpf(fi * w_in + fo * w_out);
            to_key = __builtin_amdgcn_rcpf(rate + fr * (late - rate));
            lo = 1.0f; hi = 0.0f;            // (weighted: x is what is left of the law, 1 at T = 0)
        }
        uint32_t T = 0u;
        uint64_t open = __ballot(ranked);
        for (int step = 0; step < SEARCH_STEPS && open != 0; ++step) {
            const float x = lo + (hi - lo) * (at_lo * __builtin_amdgcn_rcpf(at_lo + at_hi));
            T = MODE == 2 ? __float_as_uint(fmaxf(0.0f, -__builtin_amdgcn_logf(x) * to_key)) : (uint32_t)x;
            const int off = count4_onto(-expect, kw[0] < T, kw[1] < T, kw[2] < T, kw[3] < T);
            const float at = 0.5f + __builtin_fabsf((float)off);
            const bool above = off > 0, below = off < 0;
            lo = above ? lo : x;
            at_lo = above ? at_lo : at;
            hi = below ? hi : x;
            at_hi = below ? at_hi : at;
            open &= __ballot(above) | __ballot(below);
        }
        ok = ((open >> lane) & 1u) == 0;
        T = ranked ? T : 1u;
        if (MODE == 2) {
            // No key may lie within its error bound of T: then every kept slot's exact key is below every other's.  The bound's
            // absolute part goes with the slot's own class: with the larger class weight for all slots three times as many rows
            // were redone, 14 us of 222 on a reddit-like group.  T is anywhere in the gap around it, so a row that fails tries
            // again a few bounds higher and lower.  (Slots outside the pool hold a NaN: never near.)
            auto apart = [&](float t) -> bool {
                const float rel = t * (CLOCK_ERR_REL + 0x1p-20f);
                const float near_in = rel + (CLOCK_ERR_ABS + 0.25f) * 0x1p-24f * (float)a.q_out;
                const float near_out = rel + (CLOCK_ERR_ABS + 0.25f) * 0x1p-24f * (float)a.q_in;
                bool near[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    near[i] = __builtin_fabsf(__uint_as_float(kw[i]) - t) <= (((nib >> i) & 1u) ? near_in : near_out);
                return count4(near[0], near[1], near[2], near[3]) == 0;
            };
            const float tf = __uint_as_float(T);
            bool safe = !ranked || apart(tf);
            if (__ballot(ok && !safe) != 0) {
                const float shift = 2.5f * (tf * (CLOCK_ERR_REL + 0x1p-20f) + (CLOCK_ERR_ABS + 0.25f) * 0x1p-24f * (float)max(a.q_in, a.q_out));
#pragma unroll 1
                for (int s = 0; s < 2; ++s) {
                    const float t = fmaxf(0.0f, s ? tf - shift : tf + shift);
                    const uint32_t moved = __float_as_uint(t);
                    const bool as_many = count4(kw[0] < moved, kw[1] < moved, kw[2] < moved, kw[3] < moved) == expect;
                    if (apart(t) && as_many && !safe) { safe = true; T = moved; }
                }
            }
            ok = ok && safe;
        }
        const bool k0 = kw[0] < T, k1 = kw[1] < T, k2 = kw[2] < T, k3 = kw[3] < T;
        emit = (k0 ? 1u : 0u) | (k1 ? 2u : 0u) | (k2 ? 4u : 0u) | (k3 ? 8u : 0u);
        epos = before4(k0, k1, k2, k3);
    } else {
        const int cpos = before_bits(pool), nc_mine = ranked ? P : 0;
        int rk[4] = {0, 0, 0, 0};
        uint32_t below_m = 0u;               // slots of the pool with fewer than m of its slots in front
        if constexpr (MODE == 2) {
            // the exact integer keys, 64 bits each; (key, slot) pairs compared in full
            unsigned long long ek[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) ek[i] = (uint64_t)exp_clock_q24<true>(wr[i]) * (uint64_t)(((nib >> i) & 1u) ? a.q_out : a.q_in);
            unsigned long long *kl = k64 + 4 * first;
            if (ranked) {
                int k = cpos;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if ((pool >> i) & 1u) kl[k++] = ek[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int t = 0; __ballot(t < nc_mine) != 0; ++t) {
                if (t < nc_mine) {
                    const unsigned long long kt = kl[t];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        rk[i] += (kt < ek[i] || (kt == ek[i] && t < cpos + (int)__popc(pool & ((1u << i) - 1u)))) ? 1 : 0;
                }
            }
        } else {
            // the row's list: the pool's words in slot order
            uint32_t *kl = klist + 4 * first;
            if (ranked) {
                int k = cpos;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if ((pool >> i) & 1u) kl[k++] = kw[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int t = 0; __ballot(t < nc_mine) != 0; ++t) {
                if (t < nc_mine) {
                    const uint32_t kt = kl[t];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        rk[i] += (kt < kw[i] || (kt == kw[i] && t < cpos + (int)__popc(pool & ((1u << i) - 1u)))) ? 1 : 0;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) below_m |= rk[i] < m ? 1u << i : 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the lists are reused by the next pass
        emit = take | (pool & below_m);
        epos = before_bits(emit);
    }
    if (active && ok) {
        const int32_t *from = a.g_indices + R.base + jb;
        int32_t id[4] = {0, 0, 0, 0};
        if (R.base + jb + 4 <= a.n_entries) {            // the quad's ids in one load (four bytes of alignment are enough for it)
            if (emit) {
                struct __attribute__((packed, aligned(4))) Quad { int32_t x[4]; };
                const Quad v = *reinterpret_cast<const Quad *>(from);
#pragma unroll
                for (int i = 0; i < 4; ++i) id[i] = v.x[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if ((emit >> i) & 1u) id[i] = from[i];
        }
        int32_t *to = out + R.out + epos;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if ((emit >> i) & 1u) to[__popc(emit & ((1u << i) - 1u))] = id[i];
        if (qi == 0) set_row_count(a, g, row0 + r, expect);
    }
    uint64_t bad = __ballot(active && qi == 0 && !ok);
    uint32_t redo = 0u;
    while (bad) {
        redo |= 1u << rl32((uint32_t)r, __ffsll((long long)bad) - 1);
        bad &= bad - 1;
    }
    return redo;
}

// Long rows, weighted, with single-precision keys: the row's slots are filtered by per-class thresholds on the random word
// (chosen so that about cand_target keys lie below a common kappa), the candidates' keys approx_clock(r) * m_class are
// ranked through their bit patterns, and the result is accepted if the largest kept key and the smallest key left out
// (among the candidates, and the smallest a filtered-out slot can have) are further apart than the keys' error bounds.
// Returns false otherwise (too few or too many candidates, check failed): the caller goes on to the exact paths.
__device__ __forceinline__ bool select_big_row_weighted_f32(const SelectArgs &a, int g, int row, int32_t *sel_row, int32_t v, int64_t base, int deg,
                                                            int lane, uint32_t *ckey /*[CAND_CAP + 4]*/, uint32_t *cslot /*[CAND_CAP]*/)
{
    const int k = a.fanout;
    const uint32_t batch = a.first_batch + (uint32_t)g;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    const int64_t w_first = base >> 5, e_last = base + deg, w_last = (e_last - 1) >> 5;
    int n_in = 0;
    for (int64_t w = w_first + lane; w <= w_last; w += WAVE) {
        uint32_t bits = a.edge_intra[w];
        if (w == w_first) bits &= ~0u << (base & 31);
        if (w == w_last && (e_last & 31)) bits &= (1u << (e_last & 31)) - 1u;
        n_in += __popc(bits);
    }
    n_in = wave_sum(n_in);
    const int n_out = deg - n_in;
    const float m_in = (float)a.q_out, m_out = (float)a.q_in;       // an intra-community slot's clock is scaled by 1 - p

    // candidate iff r >= t_class; lo_non: the smallest key a slot below its class's threshold can have
    uint32_t t_in = 0u, t_out = 0u;
    float non_in = INFINITY, non_out = INFINITY, most = INFINITY;      // most: the candidates' keys end about here
    if ((int)a.cand_target < deg) {
        const float ln2 = 0.69314718f, target = (float)a.cand_target, fi = (float)n_in, fo = (float)n_out;
        const float s_in = __builtin_amdgcn_rcpf(m_in), s_out = __builtin_amdgcn_rcpf(m_out);
        float kp = target / (ln2 * (fi * s_in + fo * s_out));
#pragma unroll
        for (int it = 0; it < 3; ++it) {
            const float ei = __builtin_amdgcn_exp2f(-kp * s_in), eo = __builtin_amdgcn_exp2f(-kp * s_out);
            const float gv = fi * (1.0f - ei) + fo * (1.0f - eo) - target;
            const float gd = ln2 * (fi * s_in * ei + fo * s_out * eo);
            if (gd > 0.0f) kp -= gv / gd;
        }
        most = kp;
        const float pi = __builtin_amdgcn_exp2f(-kp * s_in) * 4294967296.0f, po = __builtin_amdgcn_exp2f(-kp * s_out) * 4294967296.0f;
        t_in = pi >= 4294967040.0f ? 0xFFFFFFFFu : (uint32_t)(pi > 0.0f ? pi : 0.0f);
        t_out = po >= 4294967040.0f ? 0xFFFFFFFFu : (uint32_t)(po > 0.0f ? po : 0.0f);
        if (t_in > 0u && n_in > 0) non_in = approx_clock(t_in - 1u) * m_in;
        if (t_out > 0u && n_out > 0) non_out = approx_clock(t_out - 1u) * m_out;
    }

    const int64_t w_max = (a.n_entries - 1) >> 5;
    int n = 0;
    // 256 slots from j0 on; a slot is a candidate iff its word is at or above its class's threshold (in the row's last
    // stretch: and it is not beyond the row's end).  false: more candidates than the list holds.
    auto stretch = [&](int j0, auto is_last) -> bool {
        constexpr bool LAST = decltype(is_last)::value;
        const int jb = j0 + 4 * lane;
        const u32x4 w = philox4x32_10((uint32_t)jb >> 2, (uint32_t)v, batch, a.ctr3, a.seed_lo, a.seed_hi);
        const uint32_t wr[4] = {w.x, w.y, w.z, w.w};
        const int64_t e = base + min(jb, deg - 1);
        const int64_t wi = e >> 5;
        const uint64_t win = (uint64_t)a.edge_intra[wi] | ((uint64_t)a.edge_intra[min(wi + 1, w_max)] << 32);
        const uint32_t nib = (uint32_t)(win >> (e & 31)) & 0xFu;
        bool c[4];
        uint64_t b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            c[i] = wr[i] >= (((nib >> i) & 1u) ? t_in : t_out);
            if (LAST) c[i] = c[i] && jb + i < deg;
            b[i] = __ballot(c[i]);
        }
        if ((b[0] | b[1] | b[2] | b[3]) == 0) return true;             // (most stretches of a very long row)
        int before = n;
#pragma unroll
        for (int i = 0; i < 4; ++i) before = lanes_below(b[i], before);
        const int total = __popcll(b[0]) + __popcll(b[1]) + __popcll(b[2]) + __popcll(b[3]);
        if (n + total > CAND_CAP) return false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (c[i]) {
                ckey[before] = wr[i];               // (the key is computed once per candidate, after the loop)
                cslot[before] = (uint32_t)(jb + i) | (((nib >> i) & 1u) << 31);
            }
            before += c[i] ? 1 : 0;
        }
        n += total;
        return true;
    };
    int j0 = 0;
    for (; j0 + 4 * WAVE <= deg; j0 += 4 * WAVE)
        if (!stretch(j0, std::false_type{})) return false;
    if (j0 < deg && !stretch(j0, std::true_type{})) return false;
    if (n < k || !(most < INFINITY)) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // candidate t sits at index t in slot order; a lane owns candidates lane and lane + 64 and turns their random words
    // into keys
    const bool have0 = lane < n, have1 = lane + WAVE < n, two = n > WAVE;
    const uint32_t q0 = cslot[min(lane, n - 1)], q1 = cslot[min(lane + WAVE, n - 1)];
    const bool in0 = q0 >> 31, in1 = q1 >> 31;
    const uint32_t w0 = have0 ? __float_as_uint(approx_clock(ckey[lane]) * (in0 ? m_in : m_out)) : 0x7F800000u;
    uint32_t w1 = 0x7F800000u;
    if (two && have1) w1 = __float_as_uint(approx_clock(ckey[lane + WAVE]) * (in1 ? m_in : m_out));
    // A bound with k candidates below it, and no key -- a candidate's, or one that a filtered-out slot can have -- within its error
    // bound of it: then every kept slot's exact key is below every other's.  A row that fails tries again a few bounds higher
    // and lower, as in the passes of short rows.
    auto below = [&](uint32_t t) { return (int)__popcll(__ballot(w0 < t)) + (two ? (int)__popcll(__ballot(w1 < t)) : 0); };
    auto apart = [&](float t) -> bool {
        const float rel = t * (CLOCK_ERR_REL + 0x1p-20f);
        const float near_in = rel + (CLOCK_ERR_ABS + 0.25f) * 0x1p-24f * m_in, near_out = rel + (CLOCK_ERR_ABS + 0.25f) * 0x1p-24f * m_out;
        const bool near0 = __builtin_fabsf(__uint_as_float(w0) - t) <= (in0 ? near_in : near_out);
        const bool near1 = __builtin_fabsf(__uint_as_float(w1) - t) <= (in1 ? near_in : near_out);
        return __ballot(near0 || near1) == 0 && keys_apart(t, m_in, non_in, m_in) && keys_apart(t, m_out, non_out, m_out);
    };
    uint32_t T;
    bool exact = search_bound(n, k, most, [](float x) { return __float_as_uint(x); }, below, T);
    if (exact && !apart(__uint_as_float(T))) {
        const float tf = __uint_as_float(T);
        const float shift = 2.5f * (tf * (CLOCK_ERR_REL + 0x1p-20f) + (CLOCK_ERR_ABS + 0.25f) * 0x1p-24f * fmaxf(m_in, m_out));
        exact = false;
#pragma unroll 1
        for (int i = 0; i < 2 && !exact; ++i) {
            T = __float_as_uint(fmaxf(0.0f, i ? tf - shift : tf + shift));
            exact = below(T) == k && apart(__uint_as_float(T));
        }
    }
    const bool s0 = w0 < T, s1 = w1 < T;
    const uint64_t m0 = __ballot(s0), m1 = __ballot(s1);
    if (exact) {
        if (s0) sel_row[__popcll(m0 & lt_mask)] = a.g_indices[base + (q0 & 0x7FFFFFFFu)];
        if (s1) sel_row[__popcll(m0) + __popcll(m1 & lt_mask)] = a.g_indices[base + (q1 & 0x7FFFFFFFu)];
        if (lane == 0) set_row_count(a, g, row, k);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the buffers are reused by this wave's next long row
    return exact;
}

// Row pointers of a block of few rows, worked out by the first wave of every workgroup of the selection (they need degrees only):
// a launch of their own is 4.5 us for 64 rows (a group of one batch of 64 roots: 32.8 -> 28.2 us, with its training step 74.5 ->
// 66.3).  Every workgroup reads all of the batch's degrees, so only where that is a few loads a lane.  pre: exclusive prefix sums;
// `writer` also writes what scan_kernel does in mode 4.
constexpr int SELECT_SCAN_ROWS = 512;
__device__ __forceinline__ void select_scan(const SelectArgs &a, int g, int n_dst, bool writer, int *pre)
{
    constexpr int CHUNKS = SELECT_SCAN_ROWS / WAVE;
    const int lane = lane_id();
    const ScanArgs &sc = a.scan;
    const int32_t *dst = a.dst_ids + (int64_t)g * a.dst_stride;
    int32_t node[CHUNKS];
    int cnt[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c)
        if (c * WAVE < n_dst) node[c] = dst[min(c * WAVE + lane, n_dst - 1)];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        cnt[c] = 0;
        if (c * WAVE < n_dst) {
            const int64_t d = a.g_indptr[node[c] + 1] - a.g_indptr[node[c]];
            cnt[c] = c * WAVE + lane < n_dst ? (int)(d < a.fanout ? d : a.fanout) : 0;
        }
    }
    int total = 0;
    int32_t *out = sc.out + (int64_t)g * sc.out_stride;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        if (c * WAVE >= n_dst) break;
        const int r = c * WAVE + lane;
        int incl = cnt[c];
#pragma unroll
        for (int off = 1; off < WAVE; off <<= 1) {
            const int y = __shfl_up(incl, off);
            if (lane >= off) incl += y;
        }
        const int before = total + incl - cnt[c];
        pre[r] = before;
        if (writer && r < n_dst) {
            out[r] = before;
            if (sc.head_ids) sc.head_ids[(int64_t)g * sc.head_stride + r] = node[c];
        }
        total += __builtin_amdgcn_readlane(incl, WAVE - 1);
    }
    if (!writer) return;
    if (sc.zero) {
        for (int i = lane; i < sc.n_zero; i += WAVE) sc.zero[(int64_t)g * sc.n_zero + i] = 0;
    }
    if (lane == 0) {
        int32_t *hdr = sc.hdr + (int64_t)g * CR_HDR_WORDS;
        out[n_dst] = total;
        hdr[CR_HDR_N_DST] = n_dst;
        hdr[CR_HDR_NNZ] = total;
        hdr[CR_HDR_STATUS] = sc.prev_hdr ? sc.prev_hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_STATUS] : 0;
        hdr[4] = hdr[5] = hdr[6] = hdr[7] = 0;
        if (sc.head_ids) hdr[CR_HDR_N_SRC] = -1;
    }
}

// (occupancy targets: the weighted instantiation takes 85 registers when left alone, which leaves five waves per SIMD and
// measures 5 % slower on a sampled group than 80 registers, six waves; the other two fit 64 registers, eight waves: 3 % on a group at p = 1)
template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MODE == 2 ? 6 : 8, 8))) void select_quad_kernel(SelectArgs a)
{
    __shared__ QuadRow rows_s[4][QUAD_ROWS];
    __shared__ __align__(16) uint32_t klist_s[4][4 * WAVE];
    __shared__ uint32_t cslot_s[4][CAND_CAP];              // long rows: candidates' slots
    __shared__ unsigned long long k64_s[MODE == 2 ? 4 : 1][MODE == 2 ? 4 * WAVE : 1];     // weighted: exact 64-bit keys
    const int wv = (int)threadIdx.x / WAVE;
    unsigned long long *k64 = k64_s[MODE == 2 ? wv : 0];
    const int g = blockIdx.y;
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);
    const int row0 = (int)(blockIdx.x * 4 + wv) * a.rows_per_wave;
    const int lane = lane_id();
    __shared__ int pre_s[SELECT_SCAN_ROWS];
    if (a.scan_here) {
        if (wv == 0) select_scan(a, g, n_dst, blockIdx.x == 0, pre_s);
        __syncthreads();
    }
    if (row0 >= n_dst) return;

    // lanes 0..QUAD_ROWS-1 fetch one row's node id, adjacency range and output place each
    int32_t mv = 0;
    int64_t mbase = 0;
    int mdeg = 0;
    int64_t mout = 0;
    int32_t *out = a.out_indptr ? a.out_ids + (int64_t)g * a.out_stride : a.sel + (int64_t)g * a.sel_stride;
    if (lane < a.rows_per_wave && row0 + lane < n_dst) {
        mv = a.dst_ids[(int64_t)g * a.dst_stride + row0 + lane];
        mbase = a.g_indptr[mv];
        const int64_t d = a.g_indptr[mv + 1] - mbase;
        mdeg = (int)(d > 0x7FFFFFFF ? 0x7FFFFFFF : d);
        mout = a.scan_here ? (int64_t)pre_s[row0 + lane]
                           : (a.out_indptr ? (int64_t)a.out_indptr[(int64_t)g * a.out_indptr_stride + row0 + lane] : (int64_t)(row0 + lane) * a.fanout);
        if (mdeg == 0) set_row_count(a, g, row0 + lane, 0);
    }
    const int mq = (mdeg > 0 && mdeg <= QUAD_MAX_DEG) ? (mdeg + 3) >> 2 : 0;
    if (lane < QUAD_ROWS) {
        QuadRow R;
        R.v = mv; R.deg = mdeg; R.base = mbase; R.out = mout; R.pad = 0;
        rows_s[wv][lane] = R;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // Packing of the rows' quads into passes of 64 (a row never straddles two passes): a pass takes, again and again, the
    // first row not yet placed that still fits (first fit over the rows; filling the passes with the rows in their own
    // order leaves them three quarters full on the degree mixes of sampled frontiers, this gets them to ~85 %).  Every lane
    // from the row's first one on notes the row as it is placed, so that the pass needs no search for it.
    auto run = [&](uint32_t waiting, auto exact) -> uint32_t {
        constexpr bool EXACT = decltype(exact)::value;
        uint32_t redo = 0u;
        while (waiting) {
            int room = WAVE, r = 0, first = 0;
            for (;;) {
                const uint32_t fits = (uint32_t)__ballot(mq <= room) & waiting;
                if (!fits) break;
                const int i = __builtin_ctz(fits), at = WAVE - room;
                r = lane >= at ? i : r;
                first = lane >= at ? at : first;
                room -= (int)rl32((uint32_t)mq, i);
                waiting &= ~(1u << i);
            }
            redo |= quad_pass<MODE, EXACT>(a, g, row0, r, first, WAVE - room, rows_s[wv], out, klist_s[wv], k64, lane);
        }
        return redo;
    };
    const uint32_t all_rows = (uint32_t)__ballot(mq > 0);       // (lanes from QUAD_ROWS on hold no row: mq = 0)
    const uint32_t exact_rows = a.exact_select ? all_rows : run(all_rows, std::false_type{});
    if (exact_rows) run(exact_rows, std::true_type{});

    // longer rows, one at a time
#pragma unroll 1
    for (int i = 0; i < QUAD_ROWS; ++i) {
        const int deg = (int)rl32((uint32_t)mdeg, i);
        if (deg <= QUAD_MAX_DEG) continue;
        const int32_t v = (int32_t)rl32((uint32_t)mv, i);
        const int64_t base = (int64_t)rl64((uint64_t)mbase, i);
        int32_t *sel_row = out + (int64_t)rl64((uint64_t)mout, i);
        if constexpr (MODE == 2) {
            if (!a.exact_select && select_big_row_weighted_f32(a, g, row0 + i, sel_row, v, base, deg, lane, klist_s[wv], cslot_s[wv])) continue;
            if (!a.exact_select &&
                select_big_row_weighted<true>(a, g, row0 + i, sel_row, v, base, deg, lane, reinterpret_cast<uint2 *>(klist_s[wv]), k64)) continue;
        } else {
            if (!a.exact_select && select_big_row_filtered<MODE == 1>(a, g, row0 + i, sel_row, v, base, deg, lane, klist_s[wv], cslot_s[wv])) continue;
        }
        select_big_row<MODE, true>(a, g, row0 + i, sel_row, v, base, deg, MODE >= 1 ? a.comm[v] : 0, lane);
    }
}

// rows of a block that keep min(fanout, degree) neighbours each (no strict mode): the counts need no selection
__global__ __launch_bounds__(256) void row_counts_kernel(const int64_t *__restrict__ g_indptr, const int32_t *__restrict__ dst_ids,
                                                         int64_t dst_stride, const int32_t *__restrict__ prev_hdr, int64_t n_roots_total,
                                                         int32_t batch_size, int32_t fanout, int32_t *__restrict__ cnt, int64_t cnt_stride)
{
    const int g = blockIdx.y;
    const int n_dst = group_n_dst(prev_hdr, g, n_roots_total, batch_size);
    const int row = (int)(blockIdx.x * 256 + threadIdx.x);
    if (row >= n_dst) return;
    const int32_t v = dst_ids[(int64_t)g * dst_stride + row];
    const int64_t d = g_indptr[v + 1] - g_indptr[v];
    cnt[(int64_t)g * cnt_stride + row] = (int32_t)(d < fanout ? d : fanout);
}

// Error of approx_clock against the integer clock over every 32-bit word: out[0] = largest |error| (Q24 units) among the
// words of the upper half (small clocks), out[1] = largest |error| / E over the lower half, out[2] = largest
// |error| / (CLOCK_ERR_ABS + CLOCK_ERR_REL * E) over all words (the selection relies on this being at most 1).
__global__ __launch_bounds__(256) void clock_selftest_kernel(float *out)
{
    float worst_abs = 0.f, worst_rel = 0.f, worst_ratio = 0.f;
    const uint32_t stride = gridDim.x * 256u;
    uint32_t r = blockIdx.x * 256u + threadIdx.x;
    for (uint64_t n = r; n < 0x100000000ull; n += stride, r += stride) {
        const uint32_t exact = exp_clock_q24(r);
        // (the single-precision value times 2^24 and the 30-bit integer are both exact in double precision)
        const float err = (float)fabs((double)approx_clock(r) * 16777216.0 - (double)exact);
        const float ef = (float)exact;
        const bool small_clock = r >= 0x80000000u;
        worst_abs = fmaxf(worst_abs, small_clock ? err : 0.f);
        worst_rel = fmaxf(worst_rel, small_clock ? 0.f : err / ef);
        worst_ratio = fmaxf(worst_ratio, err / (CLOCK_ERR_ABS + CLOCK_ERR_REL * ef));
    }
    // (non-negative floats order like their bit patterns)
    atomicMax(reinterpret_cast<unsigned int *>(out + 0), __float_as_uint(worst_abs));
    atomicMax(reinterpret_cast<unsigned int *>(out + 1), __float_as_uint(worst_rel));
    atomicMax(reinterpret_cast<unsigned int *>(out + 2), __float_as_uint(worst_ratio));
}

// out[0..n] = exclusive prefix sums of in[0..n) per batch (blockIdx.y).  A workgroup owns one tile of 256 x 16
// elements (blockIdx.x): it first adds up everything in front of its tile (the input is a few hundred KB at most and
// sits in L2, so the tiles of a batch need no hand-off between workgroups and all of them run at once), then scans
// its own tile.  The workgroup of the last tile also writes out[n] and the block header.
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

__global__ __launch_bounds__(SCAN_THREADS) void scan_kernel(ScanArgs a)
{
    __shared__ int lds[17];
    const int g = blockIdx.y;
    int32_t *hdr = a.hdr + (int64_t)g * CR_HDR_WORDS;
    if (a.zero && blockIdx.x == 0 && threadIdx.x < a.n_zero) a.zero[(int64_t)g * a.n_zero + threadIdx.x] = 0;
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);
    const int n = a.mode == 3 ? a.n_fixed : (a.mode == 2 ? hdr[CR_HDR_N_SRC] : n_dst);
    const int first = (int)blockIdx.x * SCAN_TILE;
    if (first >= n && blockIdx.x != 0) return;              // (the first workgroup also handles an empty batch)
    const int32_t *in = a.in + (int64_t)g * a.in_stride;
    int32_t *out = a.out + (int64_t)g * a.out_stride;
    int32_t *out_copy = a.out_copy ? a.out_copy + (int64_t)g * a.copy_stride : nullptr;

    int before = 0;                                          // sum of in[0..first)
    if (a.tile_before) {
        before = a.tile_before[blockIdx.x];
    } else if (first > 0) {
        int part = 0;
        int i0 = (int)threadIdx.x;                               // (first is a multiple of the tile size)
        // four tiles' loads in flight at a time: the loop is a chain of round trips to the L2, not of additions
        for (; i0 + 3 * SCAN_TILE < first; i0 += 4 * SCAN_TILE) {
            int x[4][SCAN_ITEMS];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < SCAN_ITEMS; ++k) x[u][k] = in[i0 + u * SCAN_TILE + k * SCAN_THREADS];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < SCAN_ITEMS; ++k) part += x[u][k];
        }
        for (; i0 < first; i0 += SCAN_TILE) {
            int x[SCAN_ITEMS];
#pragma unroll
            for (int k = 0; k < SCAN_ITEMS; ++k) x[k] = in[i0 + k * SCAN_THREADS];
#pragma unroll
            for (int k = 0; k < SCAN_ITEMS; ++k) part += x[k];
        }
        block_exclusive_scan<SCAN_THREADS / WAVE>(part, lds, before);
        __syncthreads();                                     // lds is reused below
    }
    // A thread scans sixteen consecutive elements, but the tile travels between memory and the threads through LDS, so
    // that a wave's loads and stores touch consecutive words (a thread reading its own sixteen words straight from memory
    // makes every load instruction touch 64 different cache lines).  Sixteen words are followed by one of padding: the
    // threads' stretches start 17 words apart, on different banks.
    __shared__ int tile[SCAN_TILE + SCAN_TILE / SCAN_ITEMS];
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        const int j = k * SCAN_THREADS + (int)threadIdx.x;
        int v = 0;
        if (a.mode != 4) {
            v = first + j < n ? in[first + j] : 0;
        } else if (j < n) {
            const int32_t node = a.dst_ids[(int64_t)g * a.dst_stride + j];
            const int64_t d = a.g_indptr[node + 1] - a.g_indptr[node];
            v = (int)(d < a.fanout ? d : a.fanout);
            if (a.head_ids) a.head_ids[(int64_t)g * a.head_stride + j] = node;
        }
        tile[j + j / SCAN_ITEMS] = v;
    }
    __syncthreads();
    int *mine = tile + (int)threadIdx.x * (SCAN_ITEMS + 1);
    int x[SCAN_ITEMS];
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) x[i] = mine[i];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) sum += x[i];
    int tile_total;
    int run = before + block_exclusive_scan<SCAN_THREADS / WAVE>(sum, lds, tile_total);
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        mine[i] = run;
        run += x[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        const int j = k * SCAN_THREADS + (int)threadIdx.x;
        if (first + j < n) {
            const int v = tile[j + j / SCAN_ITEMS];
            out[first + j] = v;
            if (out_copy) out_copy[first + j] = v;
        }
    }
    if (threadIdx.x == 0 && n <= first + SCAN_TILE) {        // the last tile
        const int total = before + tile_total;
        out[n] = total;
        if (a.mode == 0 || a.mode == 4) {
            hdr[CR_HDR_N_DST] = n_dst;
            hdr[CR_HDR_NNZ] = total;
            // a block sampled below a frontier that was cut short is as invalid as that frontier
            hdr[CR_HDR_STATUS] = a.prev_hdr ? a.prev_hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_STATUS] : 0;
            hdr[4] = hdr[5] = hdr[6] = hdr[7] = 0;
            if (a.head_ids) hdr[CR_HDR_N_SRC] = -1;
        } else if (a.mode == 1) {
            const int need = n_dst + total;
            if (need > a.cap_src) {        // only possible with capacities below the bound: cut the frontier, mark the block
                hdr[CR_HDR_N_SRC] = a.cap_src;
                atomicOr(&hdr[CR_HDR_STATUS], CR_ASYNC_FRONTIER_OVERFLOW);
                if (a.async_status) {
                    atomicOr(reinterpret_cast<unsigned long long *>(a.async_status), (unsigned long long)CR_ASYNC_FRONTIER_OVERFLOW);
                    atomicMax(reinterpret_cast<long long *>(a.async_status + 1), (long long)need);
                }
            } else {
                hdr[CR_HDR_N_SRC] = need;
            }
        }
    }
}

// For long inputs (the cells of a group-level row order: several hundred thousand) summing everything in front of
// every tile would read the input a hundred times over; two small kernels give the tiles their starting sums instead.
__global__ __launch_bounds__(SCAN_THREADS) void scan_tile_sums_kernel(const int32_t *in, int n, int32_t *tile_sum)
{
    __shared__ int lds[17];
    const int start = (int)blockIdx.x * SCAN_TILE + (int)threadIdx.x;
    int part = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        const int i = start + k * SCAN_THREADS;
        part += i < n ? in[i] : 0;
    }
    int total;
    block_exclusive_scan<SCAN_THREADS / WAVE>(part, lds, total);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// exclusive prefix sums of at most 1024 * 16 tile sums, in place, by one workgroup
__global__ __launch_bounds__(1024) void scan_tile_offsets_kernel(int32_t *tile_sum, int n_tiles)
{
    __shared__ int lds[17];
    int x[16], sum = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int i = (int)threadIdx.x * 16 + k;
        x[k] = i < n_tiles ? tile_sum[i] : 0;
        sum += x[k];
    }
    int total;
    int run = block_exclusive_scan_1024(sum, lds, total);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int i = (int)threadIdx.x * 16 + k;
        if (i < n_tiles) tile_sum[i] = run;
        run += x[k];
    }
}

// ---------------------------------------------------------------------------------------------
// Processing order of a block's destination rows (cr_block_set.row_order): rows grouped by the community of their
// node, a counting sort per batch over at most ORDER_BUCKETS buckets (communities are folded onto the buckets in
// order when there are more).  No global atomics (they resolve at the memory side on this part and cost ~200 ns
// each): a workgroup counts its ORDER_TILE rows per bucket in LDS and writes the counts bucket-major, one prefix sum
// per batch over (bucket, workgroup) gives every workgroup its first position in every bucket, and a second pass
// hands out positions from LDS cursors.  The order inside a (bucket, workgroup) cell follows the LDS atomics and is
// not reproducible, which is fine: the order only says which workgroup of the gather handles a row and when.
// ---------------------------------------------------------------------------------------------
constexpr int ORDER_BUCKETS = 4096;
constexpr int ORDER_TILE = 8192;          // rows per workgroup of 256 threads

struct OrderArgs {
    const int32_t *prev_hdr;
    int64_t n_roots_total;
    int32_t batch_size;
    const int32_t *dst_ids;
    int64_t dst_stride;
    const int32_t *comm;
    int32_t n_comm;
    int32_t n_buckets;        // min(n_comm, ORDER_BUCKETS)
    int32_t n_tiles;          // workgroups per batch (gridDim.x)
    int32_t *cells;           // [n_batches][n_buckets * n_tiles + 1]: counts, then (scanned, in `offsets`) first positions
    int32_t *offsets;
    int32_t *order;
    int64_t order_stride;
    int32_t grouped;          // 1: one order over all batches of the group, entries batch * cap_dst + row, count at the end
    int32_t cap_dst;
    uint16_t *bucket;         // [n_batches][bucket_stride]: a row's bucket, kept from the counting pass for the scatter pass
    int64_t bucket_stride;
    int32_t cap_rows;         // most rows a batch has
};

__device__ __forceinline__ int order_bucket(const OrderArgs &a, int node)
{
    const int cm = a.comm[node];
    const int c = a.n_comm <= ORDER_BUCKETS ? cm : (int)((int64_t)cm * ORDER_BUCKETS / a.n_comm);
    return min(max(c, 0), a.n_buckets - 1);
}

template <bool SCATTER>
__global__ __launch_bounds__(256) void order_pass_kernel(OrderArgs a)
{
    __shared__ int lds[ORDER_BUCKETS];
    const int g = blockIdx.y, tile = blockIdx.x;
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);
    // per batch: cells [bucket][tile] of this batch; grouped: cells [bucket][batch][tile] of the whole group
    const int col = a.grouped ? g * a.n_tiles + tile : tile;
    const int cols = a.grouped ? (int)gridDim.y * a.n_tiles : a.n_tiles;
    const int64_t cell0 = a.grouped ? 0 : (int64_t)g * ((int64_t)a.n_buckets * a.n_tiles + 1);
    for (int b = threadIdx.x; b < a.n_buckets; b += 256) lds[b] = SCATTER ? a.offsets[cell0 + (int64_t)b * cols + col] : 0;
    if (SCATTER && a.grouped && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        a.order[(int64_t)gridDim.y * a.cap_dst] = a.offsets[(int64_t)a.n_buckets * cols];      // number of entries
    __syncthreads();
    constexpr int PER = ORDER_TILE / 256;
    // the counting pass looks the rows' communities up (one scattered read per row) and leaves their buckets behind; the
    // scatter pass reads those in row order
    uint16_t *kept = a.bucket + (int64_t)g * a.bucket_stride;
    int bkt[PER];
    if (SCATTER) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int r = tile * ORDER_TILE + i * 256 + (int)threadIdx.x;
            bkt[i] = kept[min(r, max(n_dst - 1, 0))];
        }
    } else {
        int node[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int r = tile * ORDER_TILE + i * 256 + (int)threadIdx.x;
            node[i] = a.dst_ids[(int64_t)g * a.dst_stride + min(r, max(n_dst - 1, 0))];
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int r = tile * ORDER_TILE + i * 256 + (int)threadIdx.x;
            bkt[i] = order_bucket(a, node[i]);
            if (r < n_dst) kept[r] = (uint16_t)bkt[i];
        }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int r = tile * ORDER_TILE + i * 256 + (int)threadIdx.x;
        if (r < n_dst) {
            const int pos = atomicAdd(&lds[bkt[i]], 1);
            if (SCATTER) {
                if (a.grouped) a.order[pos] = g * a.cap_dst + r;
                else a.order[(int64_t)g * a.order_stride + pos] = r;
            }
        }
    }
    if (!SCATTER) {
        __syncthreads();
        for (int b = threadIdx.x; b < a.n_buckets; b += 256) a.cells[cell0 + (int64_t)b * cols + col] = lds[b];
    }
}

// The same for few rows (a group of at most ORDER_SMALL of them, or batches of at most as many): one workgroup counts, adds up
// and hands out positions, one launch instead of three (a group of one 64-root batch: 12 -> 4 us).
constexpr int ORDER_SMALL = 8192;
__global__ __launch_bounds__(1024) void order_small_kernel(OrderArgs a, int n_batches)
{
    __shared__ int count[ORDER_BUCKETS];
    __shared__ int lds[17];
    constexpr int PER = ORDER_SMALL / 1024, BPT = ORDER_BUCKETS / 1024;
    const int g0 = a.grouped ? 0 : (int)blockIdx.x, ng = a.grouped ? n_batches : 1, tid = threadIdx.x;
    for (int b = tid; b < ORDER_BUCKETS; b += 1024) count[b] = 0;
    __syncthreads();
    int bkt[PER];                            // row i of the workgroup: batch g0 + i / rows, row i % rows
    const int rows = a.cap_rows;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = k * 1024 + tid, g = g0 + i / rows, r = i % rows;
        bkt[k] = -1;
        if (i < ng * rows && r < group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size)) {
            bkt[k] = order_bucket(a, a.dst_ids[(int64_t)g * a.dst_stride + r]);
            atomicAdd(&count[bkt[k]], 1);
        }
    }
    __syncthreads();
    int x[BPT], sum = 0, total;
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        x[k] = count[tid * BPT + k];
        sum += x[k];
    }
    int run = block_exclusive_scan_1024(sum, lds, total);
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        count[tid * BPT + k] = run;
        run += x[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = k * 1024 + tid, g = g0 + i / rows, r = i % rows;
        if (bkt[k] < 0) continue;
        const int pos = atomicAdd(&count[bkt[k]], 1);
        if (a.grouped) a.order[pos] = g * a.cap_dst + r;
        else a.order[(int64_t)g * a.order_stride + pos] = r;
    }
    if (a.grouped && tid == 0) a.order[(int64_t)n_batches * a.cap_dst] = total;
}

// ---------------------------------------------------------------------------------------------
// frontier de-duplication: open-addressing table of (id << 32 | position), min position wins
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t hash_slot(uint32_t id, int bits) { return (id * 0x9E3779B1u) >> (32 - bits); }

__device__ __forceinline__ bool table_insert(unsigned long long *table, int bits, uint32_t id, uint32_t pos)
{
    const uint32_t mask = (1u << bits) - 1u;
    const unsigned long long mine = ((unsigned long long)id << 32) | pos;
    uint32_t h = hash_slot(id, bits);
    for (uint32_t probe = 0; probe <= mask; ++probe) {
        const unsigned long long old = atomicCAS(&table[h], EMPTY, mine);
        if (old == EMPTY) return true;
        if ((uint32_t)(old >> 32) == id) {
            atomicMin(&table[h], mine);
            return true;
        }
        h = (h + 1) & mask;
    }
    return false;
}

// returns the table slot of id (which must be present), or -1
__device__ __forceinline__ int table_find(const unsigned long long *table, int bits, uint32_t id, uint32_t &value)
{
    const uint32_t mask = (1u << bits) - 1u;
    uint32_t h = hash_slot(id, bits);
    for (uint32_t probe = 0; probe <= mask; ++probe) {
        const unsigned long long e = table[h];
        if ((uint32_t)(e >> 32) == id) { value = (uint32_t)e; return (int)h; }
        if (e == EMPTY) break;
        h = (h + 1) & mask;
    }
    value = 0;
    return -1;
}

// clears the first n (even) entries of every batch's table slice
__global__ __launch_bounds__(256) void fill_u64_kernel(unsigned long long *base, int64_t slice_stride, int64_t n, unsigned long long v)
{
    unsigned long long *p = base + (int64_t)blockIdx.y * slice_stride;
    int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 2;
    const int64_t stride = (int64_t)gridDim.x * 256 * 2;
    for (; i + 1 < n; i += stride) *reinterpret_cast<ulonglong2 *>(p + i) = make_ulonglong2(v, v);
    if (i < n) p[i] = v;
}

// Direct-address variant for graphs whose node count is within a small factor of the frontier
// capacity: one int32 per node holding the smallest position seen (INT_MAX = absent).  Insertion is a
// single no-return atomic, look-ups are single loads; touched entries are reset after the hop.
constexpr int32_t ABSENT = 0x7FFFFFFF;

struct DedupArgs {
    int32_t direct;           // 1: table is int32[n_nodes] per batch, 0: open-addressing table
    const int32_t *prev_hdr;
    int64_t n_roots_total;
    int32_t batch_size;
    int32_t fanout;
    int32_t gw;               // lanes per row: power of two >= fanout
    const int32_t *dst_ids;
    int64_t dst_stride;
    const int32_t *sel;
    int64_t sel_stride;
    unsigned long long *table;
    int64_t table_stride;
    int32_t table_bits;
    int32_t *hdr;
    int32_t *src_ids;
    int64_t src_stride;
    int32_t cap_src;          // entries the frontier array holds per batch
    int64_t *async_status;    // status words of the caller's context, or NULL
    int32_t *indptr;
    int64_t indptr_stride;
    int32_t *indices;
    int64_t indices_stride;
    int32_t *gather_ids;      // [G][cap_nnz] or NULL
    int32_t *newcnt;          // [G][cap_dst]
    int32_t *newoff;          // [G][cap_dst+1]
    unsigned long long *newmask;
    int64_t row_stride;       // stride of newcnt / newmask
    int64_t off_stride;
    int32_t *tcount;          // [G][cap_src] or NULL
    int32_t *tfill;           // [G][cap_src+1]
    int64_t t_stride;
    int32_t *t_indptr;
    int64_t t_indptr_stride;
    int32_t *t_indices;
    int32_t *t_tmp;           // [G][cap_nnz] destination rows in arrival order
    int32_t *t_pos;           // [G][cap_nnz] where each edge landed in t_tmp
    int64_t tt_stride;        // stride of t_tmp / t_pos
    int32_t *first;           // [G][cap_nnz] first appearance of every edge's neighbour (frontier in LDS; in t_pos' room)
    int64_t first_stride;
    int32_t *edge_rows;       // [G][cap_nnz] destination row of every edge, for the transpose in LDS, or NULL
    int64_t edge_rows_stride;
    // hops in several parts (frontier in LDS); all NULL otherwise
    int32_t *counters;        // [G][HOP_COUNTERS]: entries of every part's list, then of every source range's
    uint2 *lists;             // [G] x list_stride: [parts][LIST_CAP] (id, position)
    int32_t *t_lists;         // the same room, later: [t_parts][T_LIST] row << 14 | source in its range
    int64_t list_stride;      // in 8-byte words
    unsigned long long *seen_bits;    // [G][NUMBER_WORDS]: edges whose neighbour has appeared before
    int32_t *new_count;       // [G][HOP_CHUNKS_MAX]: edges whose neighbour has not, per stretch of words
    int32_t t_parts;          // source ranges of the transpose
};

// maps a thread to (row, j): gw lanes per row
#define CR_ROW_LANE()                                                                 \
    const int g = blockIdx.y;                                                         \
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);      \
    const int64_t gt = (int64_t)blockIdx.x * 256 + threadIdx.x;                       \
    const int row = (int)(gt / a.gw);                                                 \
    const int j = (int)(gt % a.gw);                                                   \
    const int32_t *indptr = a.indptr + (int64_t)g * a.indptr_stride;                  \
    const bool in_row = row < n_dst;                                                  \
    const int rstart = in_row ? indptr[row] : 0;                                      \
    const int k = in_row ? indptr[row + 1] - rstart : 0;                              \
    const bool active = in_row && j < k;                                              \
    const int64_t ell = (int64_t)row * a.fanout + j;                                  \
    unsigned long long *table = a.table + (int64_t)g * a.table_stride;                \
    int32_t *hdr = a.hdr + (int64_t)g * CR_HDR_WORDS;                                 \
    (void)hdr; (void)table; (void)ell; (void)rstart

__global__ __launch_bounds__(256) void insert_kernel(DedupArgs a)
{
    CR_ROW_LANE();
    bool ok = true;
    int32_t *dtab = reinterpret_cast<int32_t *>(table);
    if (in_row && j == 0) {
        const int32_t v = a.dst_ids[(int64_t)g * a.dst_stride + row];
        a.src_ids[(int64_t)g * a.src_stride + row] = v;
        if (a.direct) atomicMin(&dtab[v], row);
        else ok = table_insert(table, a.table_bits, (uint32_t)v, (uint32_t)row);
    }
    if (active) {
        const int32_t u = a.sel[(int64_t)g * a.sel_stride + ell];
        if (a.direct) atomicMin(&dtab[u], (int32_t)(n_dst + ell));
        else ok = table_insert(table, a.table_bits, (uint32_t)u, (uint32_t)(n_dst + ell)) && ok;
    }
    if (!ok) {
        atomicOr(&hdr[CR_HDR_STATUS], CR_ASYNC_TABLE_FULL);
        if (a.async_status) atomicOr(reinterpret_cast<unsigned long long *>(a.async_status), (unsigned long long)CR_ASYNC_TABLE_FULL);
    }
}

// which chosen neighbours are seen here for the first time (and are not destination nodes)
__global__ __launch_bounds__(256) void mark_new_kernel(DedupArgs a)
{
    CR_ROW_LANE();
    bool isnew = false;
    if (active) {
        const int32_t u = a.sel[(int64_t)g * a.sel_stride + ell];
        if (a.direct) {
            isnew = reinterpret_cast<const int32_t *>(table)[u] == (int32_t)(n_dst + ell);
        } else {
            uint32_t pos;
            const int h = table_find(table, a.table_bits, (uint32_t)u, pos);
            isnew = h >= 0 && pos == (uint32_t)(n_dst + ell);
        }
    }
    const uint64_t m = __ballot(isnew);
    if (in_row && j == 0) {
        const int sub = lane_id() / a.gw;
        const uint64_t rowmask = a.gw == 64 ? m : ((m >> (sub * a.gw)) & ((1ull << a.gw) - 1ull));
        a.newcnt[(int64_t)g * a.row_stride + row] = __popcll(rowmask);
        a.newmask[(int64_t)g * a.row_stride + row] = rowmask;
    }
}

// new nodes get consecutive frontier positions after the destination nodes; the table entry of a
// node now holds its position in the frontier
__global__ __launch_bounds__(256) void assign_kernel(DedupArgs a)
{
    CR_ROW_LANE();
    if (a.tcount) {   // clear the per-source counters of the transposed block
        const int n_src = hdr[CR_HDR_N_SRC];
        int32_t *tc = a.tcount + (int64_t)g * a.t_stride;
        for (int64_t i = gt; i < n_src; i += (int64_t)gridDim.x * 256) tc[i] = 0;
    }
    if (!active) return;
    const uint64_t rowmask = a.newmask[(int64_t)g * a.row_stride + row];
    if (!((rowmask >> j) & 1ull)) return;
    const int32_t u = a.sel[(int64_t)g * a.sel_stride + ell];
    const int local = n_dst + a.newoff[(int64_t)g * a.off_stride + row] + __popcll(rowmask & ((1ull << j) - 1ull));
    if (local < a.cap_src) a.src_ids[(int64_t)g * a.src_stride + local] = u;      // (a frontier cut short: the block is marked invalid)
    if (a.direct) {
        reinterpret_cast<int32_t *>(table)[u] = local;
    } else {
        uint32_t pos;
        const int h = table_find(table, a.table_bits, (uint32_t)u, pos);
        if (h >= 0) table[h] = ((unsigned long long)(uint32_t)u << 32) | (uint32_t)local;
    }
}

__global__ __launch_bounds__(256) void relabel_kernel(DedupArgs a)
{
    CR_ROW_LANE();
    if (!active) return;
    const int32_t u = a.sel[(int64_t)g * a.sel_stride + ell];
    uint32_t local;
    if (a.direct) local = (uint32_t)reinterpret_cast<const int32_t *>(table)[u];
    else table_find(table, a.table_bits, (uint32_t)u, local);
    if (local >= (uint32_t)a.cap_src) local = 0;       // only in a block that is marked invalid: keeps every later access in range
    a.indices[(int64_t)g * a.indices_stride + rstart + j] = (int32_t)local;
    if (a.gather_ids) a.gather_ids[(int64_t)g * a.indices_stride + rstart + j] = u;
    if (a.tcount) atomicAdd(&a.tcount[(int64_t)g * a.t_stride + local], 1);
    if (a.edge_rows) a.edge_rows[(int64_t)g * a.edge_rows_stride + rstart + j] = row;
}

// input-side block left in global ids: compact the chosen neighbours into CSR order, copy the
// destination nodes into the head of the frontier, mark the frontier size as not computed
__global__ __launch_bounds__(256) void compact_ids_kernel(DedupArgs a)
{
    CR_ROW_LANE();
    if (blockIdx.x == 0 && threadIdx.x == 0) hdr[CR_HDR_N_SRC] = -1;
    if (in_row && j == 0) a.src_ids[(int64_t)g * a.src_stride + row] = a.dst_ids[(int64_t)g * a.dst_stride + row];
    if (!active) return;
    a.gather_ids[(int64_t)g * a.indices_stride + rstart + j] = a.sel[(int64_t)g * a.sel_stride + ell];
}

// the same when the selection has already written the ids in place: only the destination nodes are left to copy, one
// thread per row
__global__ __launch_bounds__(256) void frontier_head_kernel(DedupArgs a)
{
    const int g = blockIdx.y;
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);
    const int row = (int)(blockIdx.x * 256 + threadIdx.x);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_N_SRC] = -1;
    if (row < n_dst) a.src_ids[(int64_t)g * a.src_stride + row] = a.dst_ids[(int64_t)g * a.dst_stride + row];
}

// direct-address table: put the entries this hop touched back to "absent"
__global__ __launch_bounds__(256) void reset_kernel(DedupArgs a)
{
    const int g = blockIdx.y;
    const int n_src = a.hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_N_SRC];
    int32_t *dtab = reinterpret_cast<int32_t *>(a.table + (int64_t)g * a.table_stride);
    const int32_t *src = a.src_ids + (int64_t)g * a.src_stride;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_src; i += (int64_t)gridDim.x * 256) dtab[src[i]] = ABSENT;
}

// transposed block: scatter the destination row of every edge into its source's segment in arrival
// order, then rank inside the segment so that the stored order is ascending (hence reproducible)
__global__ __launch_bounds__(256) void t_fill_kernel(DedupArgs a)
{
    CR_ROW_LANE();
    if (!active) return;
    const int64_t e = (int64_t)g * a.indices_stride + rstart + j;
    const int local = a.indices[e];
    const int p = atomicAdd(&a.tfill[(int64_t)g * a.t_stride + local], 1);
    a.t_tmp[(int64_t)g * a.tt_stride + p] = row;
    a.t_pos[(int64_t)g * a.tt_stride + rstart + j] = p;
}

__global__ __launch_bounds__(256) void t_rank_kernel(DedupArgs a)
{
    CR_ROW_LANE();
    if (!active) return;
    const int64_t e = (int64_t)g * a.indices_stride + rstart + j;
    const int local = a.indices[e];
    const int32_t *tp = a.t_indptr + (int64_t)g * a.t_indptr_stride;
    const int s0 = tp[local], s1 = tp[local + 1];
    const int32_t *tmp = a.t_tmp + (int64_t)g * a.tt_stride;
    const int mine = a.t_pos[(int64_t)g * a.tt_stride + rstart + j];
    int rank = 0;
    for (int q = s0; q < s1; ++q) {
        const int r = tmp[q];
        rank += (r < row || (r == row && q < mine)) ? 1 : 0;
    }
    a.t_indices[(int64_t)g * a.indices_stride + s0 + rank] = row;
}

// ---------------------------------------------------------------------------------------------
// Frontier of a hop in LDS.  The tables above live in memory, where an atomic of one XCD is resolved behind the caches
// all XCDs share; insert / mark / assign / relabel / reset, the scans between them and the clearing of a table were 335 us of
// a group of 32 products-like batches (second hop).  Here the ids of a hop (destination nodes and chosen neighbours) are dealt
// to parts of at most LIST_MEAN entries on average, by a hash (hop_part_kernel); a workgroup takes a part's list into LDS and
// finds every id's first appearance with an LDS table (hop_first_kernel).  hop_mark_kernel marks the first appearances, a bit per
// edge, and counts them; hop_number_kernel numbers them, relabels the edges, and deals these to ranges of sources;
// hop_transpose_kernel transposes the block, each range in its own workgroup.  Every id and edge is looked at once per
// kernel.  (Before, every part's workgroup went over all ids of the batch, every range's over all edges, and every stretch of the
// numbering over all edges in front of it, 12 to 20 instructions each time: 41 of 50 us of a part, 39 of 60 of a range of the
// reddit-like input hop.  8 batches of it: 92 us in five launches, 178 in three then; 32 products-like batches,
// second hop: 83, 91 then.)
// A hop that is one part (the hop at the roots) does all of this in one workgroup and launch, without leaving LDS.
// The chosen neighbours are stored as the block's edges are (row pointers are known before the selection); position n_dst + e
// is that of edge e.  Order, labels and transposes are those of the tables, bit for bit.
// ---------------------------------------------------------------------------------------------
constexpr int HOP_THREADS = 1024;
constexpr int LIST_CAP = 11264;                 // ids of one part (11 per thread)
constexpr int LIST_PER = LIST_CAP / HOP_THREADS;
constexpr int LIST_MEAN = 9216;                 // ids a part is sized for; the rest is for ids that repeat
constexpr int PART_TABLE = 16384;
constexpr int PARTS_MAX = 32;
constexpr int PARTS_MIN = 8;                    // (a group of 32 batches then fills the 256 compute units)
constexpr int PART_PER = 8;                     // ids that a thread of hop_part_kernel deals
constexpr int PART_CHUNK = PART_PER * HOP_THREADS;
constexpr int HOP_CHUNKS_MAX = 32;              // stretches that marking and numbering cut a batch's edges into
constexpr int NUMBER_WORDS = 5120;              // 64 edges each (a multiple of HOP_THREADS words)
constexpr int T_SOURCES = 11264;                // sources of one transposed range (at least LIST_CAP)
constexpr int T_LIST = 14336;                   // edges of one transposed range
constexpr int T_MEAN = 9216;
constexpr int T_PARTS_MAX = 40;
constexpr int HOP_COUNTERS = 128;               // words per batch: PARTS_MAX, then T_PARTS_MAX of them are used
static_assert(PARTS_MAX + T_PARTS_MAX <= HOP_COUNTERS, "a counter per list");
constexpr int T_RANK_WORK = 1 << 18;            // most comparisons that the rows of a range are ranked with (2^19 and 2^20 measure the
                                                // same; with 2^21 hops on skewed graphs take up to 2.8 times as long in all)
constexpr size_t DEDUP_LDS_BYTES = (size_t)(2 * LIST_CAP + PART_TABLE) * 4;
constexpr size_t NUMBER_LDS_BYTES = (size_t)NUMBER_WORDS * 12;
constexpr size_t T_LDS_BYTES = (size_t)(T_SOURCES + 1 + 2 * T_LIST + 32) * 4;
static_assert(PARTS_MAX * LIST_MEAN <= NUMBER_WORDS * 64, "the numbering pass holds a bit per edge");
static_assert(T_SOURCES <= (1 << 14) && T_SOURCES >= LIST_CAP, "a list entry holds the source in 14 bits; a hop of one part is one range");
static_assert(DEDUP_LDS_BYTES + 512 <= 160 * 1024 && T_LDS_BYTES + 512 <= 160 * 1024, "LDS of a compute unit");

// a bijection of the 32-bit integers whose every output bit depends on every input bit (the finaliser of MurmurHash3)
__device__ __forceinline__ uint32_t mix32(uint32_t h)
{
    h ^= h >> 16; h *= 0x85EBCA6Bu;
    h ^= h >> 13; h *= 0xC2B2AE35u;
    return h ^ (h >> 16);
}

// Which of `parts` (a power of two, at most 32) parts an id belongs to: its bits folded onto five (shifts and xors; 32-bit
// products run at a quarter of their rate).  Ids that all fold onto one value are not lost, they overflow the part's list.
__device__ __forceinline__ uint32_t id_part(uint32_t id, uint32_t parts)
{
    const uint32_t x = id ^ (id >> 15);
    return xor3(x, x >> 5, x >> 10) & (parts - 1u);
}

struct HopShared {
    int count, overflow, below, work;
    int scan[17];
};

// element i of an array that every lane has the same address of (fewer than 2^30 elements): base in scalar registers, one 32-bit offset
template <typename T>
__device__ __forceinline__ T &at32(T *p, int i)
{
    return *reinterpret_cast<T *>(reinterpret_cast<uintptr_t>(p) + (uint32_t)i * (uint32_t)sizeof(T));
}

__device__ __forceinline__ uint32_t hop_id(const int32_t *dst, const int32_t *sel, int n_dst, int i) { return (uint32_t)*(i < n_dst ? dst + i : sel + (i - n_dst)); }

// first[e] = smallest position (destination rows first, then edges) at which edge e's neighbour appears, for the edges whose
// neighbour belongs to this part.  ONE: the hop is one part; `first` is then in LDS (in the table's room).
template <bool ONE>
__device__ __forceinline__ void hop_first(const DedupArgs &a, int g, int n_dst, int nnz, uint32_t part, uint32_t parts, uint32_t *lds, HopShared &sh)
{
    uint32_t *lid = lds, *lpos = lds + LIST_CAP, *table = lds + 2 * LIST_CAP;
    const int tid = threadIdx.x;
    const int32_t *dst = a.dst_ids + (int64_t)g * a.dst_stride, *sel = a.sel + (int64_t)g * a.sel_stride;
    int32_t *first = ONE ? reinterpret_cast<int32_t *>(table) : a.first + (int64_t)g * a.first_stride;
    const int total = n_dst + nnz;
    auto id_at = [&](int i) { return hop_id(dst, sel, n_dst, i); };
    const int count = ONE ? total : a.counters[(int64_t)g * HOP_COUNTERS + part];
    if (ONE || count <= LIST_CAP) {
        const uint2 *list = ONE ? nullptr : a.lists + (int64_t)g * a.list_stride + (int64_t)part * LIST_CAP;
        for (int i = tid; i < PART_TABLE; i += HOP_THREADS) table[i] = ~0u;
        // (bounds are rounded up to whole rounds of the workgroup, so that a round's loads stand alone)
        uint32_t pos[LIST_PER], is_first = 0;
#pragma unroll
        for (int k = 0; k < LIST_PER; ++k) {
            const int i = tid + k * HOP_THREADS;
            pos[k] = 0;
            if (k * HOP_THREADS < count) {                     // (uniform)
                const int ic = min(i, count - 1);
                const uint2 x = ONE ? make_uint2(id_at(ic), (uint32_t)ic) : list[ic];
                pos[k] = x.y;
                lid[i] = x.x;
                lpos[i] = x.y;
            }
        }
        __syncthreads();
        // An id's entries agree on the one that got the table's slot first and leave the smallest position there.  A lane
        // goes through its entries on its own, so a wave takes as many rounds as its slowest lane has probes in all (~30),
        // not the longest probe of every entry in turn (~90).
        {
            int i = tid, k = 0;
            uint32_t id = lid[i], h = mix32(id), s = h & (PART_TABLE - 1);
            while (__ballot(i < count) != 0) {                 // (ends: the table has more slots than the list has entries)
                if (i < count) {
                    const uint32_t old = atomicCAS(&table[s], ~0u, (uint32_t)i);
                    const bool got = old == ~0u, same = lid[got ? (uint32_t)i : old] == id && !got;
                    if (got) is_first |= 1u << k;
                    if (same) lid[i] = old;                    // (nobody asks for the id of an entry the table does not name)
                    if (got || same) {
                        i += HOP_THREADS;
                        ++k;
                        id = lid[min(i, LIST_CAP - 1)];
                        h = mix32(id);
                        s = h & (PART_TABLE - 1);
                    } else {
                        s = (s + ((h >> 14) | 1u)) & (PART_TABLE - 1);
                    }
                }
            }
        }
        __syncthreads();                                       // (every own position has been read; the table is done with)
#pragma unroll
        for (int k = 0; k < LIST_PER; ++k)
            if (tid + k * HOP_THREADS < count && !((is_first >> k) & 1u)) atomicMin(&lpos[lid[tid + k * HOP_THREADS]], pos[k]);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < LIST_PER; ++k) {
            const int i = tid + k * HOP_THREADS;
            if (i < count && (int)pos[k] >= n_dst) first[(int)pos[k] - n_dst] = (int32_t)lpos[((is_first >> k) & 1u) ? (uint32_t)i : lid[i]];
        }
        return;
    }
    // More entries than the list holds (an id that very many rows share): a table of (id, position) filled straight from the
    // ids; more distinct ids than it holds: the part in 2, 4, .. slices, by bits of the hash that nothing else uses.
    uint32_t *keys = lds, *vals = lds + PART_TABLE;
    static_assert(2 * PART_TABLE <= 2 * LIST_CAP + PART_TABLE, "the fallback's table fits the list's room");
    for (int bits = 0; bits <= 18; ++bits) {          // (18: at most 2^14 ids are left per slice, each with a slot of its own)
        bool done = true;
        for (uint32_t slice = 0; slice < (1u << bits) && done; ++slice) {
            auto in_slice = [&](uint32_t id, uint32_t h) { return id_part(id, parts) == part && ((h >> 14) & ((1u << bits) - 1u)) == slice; };
            __syncthreads();
            for (int i = tid; i < PART_TABLE; i += HOP_THREADS) { keys[i] = ~0u; vals[i] = ~0u; }
            if (tid == 0) sh.overflow = 0;
            __syncthreads();
            for (int i = tid; i < total; i += HOP_THREADS) {
                const uint32_t id = id_at(i), h = mix32(id);
                if (!in_slice(id, h)) continue;
                uint32_t s = h & (PART_TABLE - 1), probes = 0;
                for (; probes < PART_TABLE; ++probes, s = (s + 1) & (PART_TABLE - 1)) {
                    const uint32_t old = atomicCAS(&keys[s], ~0u, id);
                    if (old == ~0u || old == id) break;
                }
                if (probes < PART_TABLE) atomicMin(&vals[s], (uint32_t)i);
                else sh.overflow = 1;
            }
            __syncthreads();
            done = sh.overflow == 0;             // (uniform: read between barriers)
            if (!done) break;
            for (int i = n_dst + tid; i < total; i += HOP_THREADS) {
                const uint32_t id = id_at(i), h = mix32(id);
                if (!in_slice(id, h)) continue;
                uint32_t s = h & (PART_TABLE - 1);
                while (keys[s] != id) s = (s + 1) & (PART_TABLE - 1);
                first[i - n_dst] = (int32_t)vals[s];
            }
        }
        if (done) return;
    }
}

// Words [w0, w1) of 64 edges each: a bit for the edges whose neighbour appears for the first time (SEEN: for the others); returns
// how many of the former this wave met.
template <bool SEEN>
__device__ __forceinline__ int mark_words(const int32_t *first, int n_dst, int nnz, int w0, int w1, unsigned long long *bits)
{
    constexpr int U = 8, NW = HOP_THREADS / WAVE;
    const int lane = lane_id(), wave = (int)threadIdx.x / WAVE;
    int met = 0;
    for (int w = w0 + wave; w < w1; w += U * NW) {
        int32_t f[U];
#pragma unroll
        for (int k = 0; k < U; ++k) f[k] = first[min((w + k * NW) * 64 + lane, nnz - 1)];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int e = (w + k * NW) * 64 + lane;
            const bool have = w + k * NW < w1 && e < nnz;
            const uint64_t m = __ballot(have && f[k] == n_dst + e), all = __ballot(have);
            if (lane == 0 && w + k * NW < w1) bits[w + k * NW] = SEEN ? all & ~m : m;
            met += (int)__popcll(m);
        }
    }
    return met;
}

// A workgroup takes U edges (row, source) of every thread to the lists of their ranges of sources; count is zero before and after.
template <int U>
__device__ __forceinline__ void deal_edges(const DedupArgs &a, int g, uint32_t range, const bool (&ok)[U], const int (&row)[U], const int (&source)[U],
                                           int *count, int *base)
{
    const int tid = threadIdx.x;
    int at[U], packed[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const uint32_t q = (uint32_t)source[k] / range;
        at[k] = 0;
        if (ok[k]) at[k] = atomicAdd(&count[q], 1);
        packed[k] = (int)(q << 14) | (int)((uint32_t)source[k] - q * range);
    }
    __syncthreads();
    if (tid < a.t_parts) {
        const int c = count[tid];
        base[tid] = c ? atomicAdd(&a.counters[(int64_t)g * HOP_COUNTERS + PARTS_MAX + tid], c) : 0;
        count[tid] = 0;
    }
    __syncthreads();
    int32_t *lists = a.t_lists + (int64_t)g * 2 * a.list_stride;
#pragma unroll
    for (int k = 0; k < U; ++k) {
        if (!ok[k]) continue;
        const int q = packed[k] >> 14, slot = base[q] + at[k];
        if (slot < T_LIST) at32(lists, q * T_LIST + slot) = (row[k] << 14) | (packed[k] & 16383);      // (rows < 2^17)
    }
}

// Numbers the first appearances and relabels the edges of one stretch of rows.  Returns the frontier's length.
// ONE: the hop is one part: `first` and the edges for the transpose (`list`, row << 14 | source by edge) are in LDS, at the
// places where hop_first leaves the one and hop_transpose looks for the others.  Otherwise the marks come from hop_mark_kernel
// and the edges go to the lists of their ranges of sources, if a transpose is wanted.
constexpr int ONE_FIRST = 2 * LIST_CAP, ONE_BITS = ONE_FIRST + LIST_CAP, ONE_LIST = T_SOURCES + 1;     // (places in LDS, in words)
static_assert(ONE_BITS % 2 == 0 && (size_t)(ONE_BITS + 3 * (LIST_CAP / 64)) * 4 <= T_LDS_BYTES, "marks of one part behind its first appearances");
static_assert(ONE_LIST + LIST_CAP - 1 <= ONE_FIRST, "the edges of one part (at least one id is a root) end in front of its first appearances");
template <bool ONE>
__device__ __forceinline__ int hop_number(const DedupArgs &a, int g, int n_dst, int nnz, int chunk, int chunks, uint32_t *lds, HopShared &sh)
{
    constexpr int WORDS = ONE ? LIST_CAP / 64 : NUMBER_WORDS, PER = (WORDS + HOP_THREADS - 1) / HOP_THREADS;
    constexpr int U = ONE ? 4 : 12;
    __shared__ int t_count[T_PARTS_MAX], t_base[T_PARTS_MAX];
    unsigned long long *bits = reinterpret_cast<unsigned long long *>(lds + (ONE ? ONE_BITS : 0));
    int *pre = reinterpret_cast<int *>(lds + (ONE ? ONE_BITS : 0) + 2 * WORDS);
    int32_t *list = reinterpret_cast<int32_t *>(lds + ONE_LIST);
    const int tid = threadIdx.x;
    const int32_t *dst = a.dst_ids + (int64_t)g * a.dst_stride, *sel = a.sel + (int64_t)g * a.sel_stride;
    const int32_t *first = ONE ? reinterpret_cast<const int32_t *>(lds + ONE_FIRST) : a.first + (int64_t)g * a.first_stride;
    int32_t *src = a.src_ids + (int64_t)g * a.src_stride, *indices = a.indices + (int64_t)g * a.indices_stride;
    const int32_t *indptr = a.indptr + (int64_t)g * a.indptr_stride;
    const int r0 = (int)((int64_t)n_dst * chunk / chunks), r1 = (int)((int64_t)n_dst * (chunk + 1) / chunks);
    const int words = (nnz + 63) / 64;
    // an edge's first appearance never lies behind it: the words up to the stretch's end are enough
    const int w1 = ONE || chunk == chunks - 1 ? words : (indptr[r1] + 63) / 64;
    if constexpr (ONE) {
        mark_words<false>(first, n_dst, nnz, 0, words, bits);
    } else {
        const unsigned long long *seen = a.seen_bits + (int64_t)g * NUMBER_WORDS;
        for (int w = tid; w < w1; w += HOP_THREADS) bits[w] = ~seen[w] & (nnz - w * 64 < 64 ? (1ull << (nnz - w * 64)) - 1ull : ~0ull);
        if (tid < T_PARTS_MAX) t_count[tid] = 0;
        if (tid < WAVE) {                                      // the number of first appearances of the whole hop
            int n = tid < chunks ? a.new_count[(int64_t)g * HOP_CHUNKS_MAX + tid] : 0;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off);
            if (tid == 0) sh.count = n;
        }
    }
    __syncthreads();
    int x[PER], sum = 0, total;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        x[k] = tid * PER + k < w1 ? (int)__popcll(bits[tid * PER + k]) : 0;
        sum += x[k];
    }
    int run = block_exclusive_scan_1024(sum, sh.scan, total);
    if (!ONE) total = sh.count;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (tid * PER + k < WORDS) pre[tid * PER + k] = run;
        run += x[k];
    }
    const int need = n_dst + total, n_src = min(need, a.cap_src);
    __syncthreads();
    for (int i = r0 + tid; i < r1; i += HOP_THREADS) src[i] = dst[i];
    const bool deal = !ONE && a.t_lists != nullptr;
    const uint32_t range = deal ? (uint32_t)((n_src + a.t_parts - 1) / a.t_parts) : 1u;
    // lanes by row: the edge's row is known, and it takes the place of the neighbour's id (which no other lane reads)
    const int gw_bits = a.fanout > 1 ? 32 - __builtin_clz((uint32_t)(a.fanout - 1)) : 0, gw = 1 << gw_bits, lanes = (r1 - r0) << gw_bits;
    for (int t0 = 0; t0 < lanes; t0 += U * HOP_THREADS) {
        int row[U], e[U], f[U], local[U];
        int32_t u[U];
        bool ok[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int t = t0 + k * HOP_THREADS + tid;
            row[k] = r0 + min(t >> gw_bits, r1 - r0 - 1);
            e[k] = at32(indptr, row[k]) + (t & (gw - 1));
            ok[k] = t < lanes && e[k] < at32(indptr, row[k] + 1);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if constexpr (ONE) f[k] = first[ok[k] ? e[k] : 0];
            else f[k] = at32(first, ok[k] ? e[k] : 0);
            u[k] = at32(sel, ok[k] ? e[k] : 0);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            local[k] = f[k];
            if (!ok[k]) continue;
            if (f[k] >= n_dst) {
                const int q = f[k] - n_dst;
                local[k] = n_dst + pre[q >> 6] + (int)__popcll(bits[q >> 6] & ((1ull << (q & 63)) - 1ull));
                if (q == e[k] && local[k] < a.cap_src) at32(src, local[k]) = u[k];      // (a frontier cut short: the block is marked invalid)
            }
            if (local[k] >= a.cap_src) local[k] = 0;                              // only in a block that is marked invalid
            at32(indices, e[k]) = local[k];
            if (a.gather_ids) at32(a.gather_ids + (int64_t)g * a.indices_stride, e[k]) = u[k];
            if (a.edge_rows) at32(a.edge_rows + (int64_t)g * a.edge_rows_stride, e[k]) = row[k];
            if constexpr (ONE) list[e[k]] = (row[k] << 14) | local[k];
        }
        if (deal) deal_edges<U>(a, g, range, ok, row, local, t_count, t_base);
    }
    if (chunk == chunks - 1 && tid == 0) {
        int32_t *hdr = a.hdr + (int64_t)g * CR_HDR_WORDS;
        hdr[CR_HDR_N_SRC] = n_src;
        if (need > a.cap_src) {                // only possible with capacities below the bound
            atomicOr(&hdr[CR_HDR_STATUS], CR_ASYNC_FRONTIER_OVERFLOW);
            if (a.async_status) {
                atomicOr(reinterpret_cast<unsigned long long *>(a.async_status), (unsigned long long)CR_ASYNC_FRONTIER_OVERFLOW);
                atomicMax(reinterpret_cast<long long *>(a.async_status + 1), (long long)need);
            }
        }
    }
    return n_src;
}

// Rows of a range of sources [lo, lo + n) that the lists of hop_transpose do not hold, or whose segments are so long that ranking
// their rows one against all takes longer than this.  Either is a matter of the graph: a few nodes that a large share of a hop's
// rows chooses are numbered early and lie in one range.  The edges are taken in order, those of the range collected in order, up
// to T_WINDOW of them; two stable passes of seven bits sort them by source, which leaves every source's rows ascending, and they
// go behind the rows of the windows before: start[s] is where the next row of source s goes.  Nothing here depends on how the
// edges spread over the sources.  (In place of ranks in memory for ranges that the lists do not hold, and merge networks for
// segments of more than 1024 rows.  One batch of 16384 rows, fanout 15, on a graph with a power law: 1946 -> 188 us, 690 with the
// counters in memory; 32 x 1024 rows, fanouts 15 10 5, half of the edges with 16 nodes: 4986 -> 86, 800; 2 x 2048 rows of 64
// there: 2926 -> 86, 200.)
constexpr int T_ROUND = 4 * HOP_THREADS;        // edges looked at between two barriers
constexpr int T_WINDOW = 2 * T_ROUND;           // a window is put in order once another round might not fit
static_assert(2 * T_WINDOW + T_SOURCES <= 2 * T_LIST, "the window and its copy and a word per source fit the room of the lists");
__device__ __forceinline__ void transpose_windows(const int32_t *indices, const int32_t *edge_rows, int nnz, int lo, int n, int *start, int32_t *room,
                                                  int *wave_sum /*[16]*/, HopShared &sh, int32_t *out)
{
    constexpr int WAVES = HOP_THREADS / WAVE, PER_WAVE = T_WINDOW / WAVES, DIGITS = 128;
    int32_t *list = room, *other = room + T_WINDOW;
    int *head = reinterpret_cast<int *>(room + 2 * T_WINDOW);      // [T_SOURCES]: first place of a source's rows in the sorted window
    int *digit = head;                                             // [DIGITS][WAVES], before that
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / WAVE;
    int held = 0;                                                  // (uniform, as everything that steers the loops)
    auto sort_pass = [&](const int32_t *from, int32_t *to, int shift) {
        for (int i = tid; i < DIGITS * WAVES; i += HOP_THREADS) digit[i] = 0;
        __syncthreads();
        const int first = wave * PER_WAVE + lane, last = min(held, (wave + 1) * PER_WAVE);
        for (int i = first; i < last; i += WAVE) atomicAdd(&digit[((from[i] >> shift) & (DIGITS - 1)) * WAVES + wave], 1);
        __syncthreads();
        static_assert(DIGITS * WAVES == 2 * HOP_THREADS, "two counters per thread");
        const int c0 = digit[2 * tid], c1 = digit[2 * tid + 1];
        int total;
        const int run = block_exclusive_scan_1024(c0 + c1, sh.scan, total);
        digit[2 * tid] = run;
        digit[2 * tid + 1] = run + c0;
        __syncthreads();
        for (int i = first; i - lane < last; i += WAVE) {          // (whole waves)
            const bool have = i < last;
            const int32_t x = have ? from[i] : 0;
            const int d = (x >> shift) & (DIGITS - 1);
            uint64_t peers = __ballot(have);                       // lanes with the same digit
#pragma unroll
            for (int b = 0; b < 7; ++b) {
                const uint64_t m = __ballot(have && ((d >> b) & 1));
                peers &= ((d >> b) & 1) ? m : ~m;
            }
            const int below = lanes_below(peers, 0);
            int at = 0;
            if (have) at = digit[d * WAVES + wave] + below;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (have && below == 0) digit[d * WAVES + wave] = at + __popcll(peers);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (have) to[at] = x;
        }
        __syncthreads();
    };
    for (int i0 = 0; i0 < nnz; i0 += T_ROUND) {
        // a wave takes consecutive edges, so that the list keeps their order
        const int e0 = i0 + wave * (T_ROUND / WAVES) + lane;
        int32_t x[4], row[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int e = min(e0 + k * WAVE, nnz - 1);
            x[k] = indices[e] - lo;
            row[k] = edge_rows[e];
        }
        bool take[4];
        int mine = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            take[k] = e0 + k * WAVE < nnz && (uint32_t)x[k] < (uint32_t)n;
            mine += __popcll(__ballot(take[k]));
        }
        if (lane == 0) wave_sum[wave] = mine;
        __syncthreads();
        int at = held, more = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const int c = wave_sum[w];
            at += w < wave ? c : 0;
            more += c;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t m = __ballot(take[k]);
            if (take[k]) list[lanes_below(m, at)] = (row[k] << 14) | x[k];      // (rows < 2^17)
            at += __popcll(m);
        }
        held += more;
        __syncthreads();
        if (held <= T_WINDOW - T_ROUND && i0 + T_ROUND < nnz) continue;
        sort_pass(list, other, 0);
        sort_pass(other, list, 7);
        for (int i = tid; i < held; i += HOP_THREADS) {
            const int s = list[i] & 16383;
            if (i == 0 || (list[i - 1] & 16383) != s) head[s] = i;
        }
        __syncthreads();
        for (int i = tid; i < held; i += HOP_THREADS) {
            const int32_t y = list[i];
            const int s = y & 16383;
            out[start[s] + i - head[s]] = y >> 14;
        }
        __syncthreads();
        for (int i = tid; i < held; i += HOP_THREADS) {
            const int s = list[i] & 16383;
            if (i == held - 1 || (list[i + 1] & 16383) != s) start[s] += i - head[s] + 1;
        }
        __syncthreads();
        held = 0;
    }
}

// Transposed block of one range of sources: row pointers and, per source, the destination rows that use it, ascending.  ONE: the
// whole block is one range and its edges are in the list already (hop_number).  Otherwise they come from the range's list in
// memory; a range may have more edges than that holds.
template <bool ONE>
__device__ __forceinline__ void hop_transpose(const DedupArgs &a, int g, int n_dst, int n_src, int nnz, int part, int parts, uint32_t *lds, HopShared &sh)
{
    int *start = reinterpret_cast<int *>(lds);                                  // [T_SOURCES + 1]
    int32_t *list = reinterpret_cast<int32_t *>(lds) + T_SOURCES + 1;           // [T_LIST] row << 14 | source, as they come
    int32_t *sorted = list + T_LIST;                                            // [T_LIST] ... source by source
    int *wave_sum = reinterpret_cast<int *>(sorted + T_LIST);                   // [32] of the windows
    const int tid = threadIdx.x;
    const int32_t *indices = a.indices + (int64_t)g * a.indices_stride;
    int32_t *t_indptr = a.t_indptr + (int64_t)g * a.t_indptr_stride, *t_indices = a.t_indices + (int64_t)g * a.indices_stride;
    const int range = (n_src + parts - 1) / parts;
    const int lo = min(n_src, part * range), hi = min(n_src, lo + range), n = hi - lo;
    if (part == parts - 1 && tid == 0) t_indptr[n_src] = nnz;
    if (n <= 0) return;                                                        // (uniform)
    const int32_t *edge_rows = a.edge_rows + (int64_t)g * a.edge_rows_stride;
    for (int i = tid; i <= n; i += HOP_THREADS) start[i] = 0;
    if (tid == 0) sh.work = 0;
    int count = nnz, base = 0;
    __syncthreads();
    if constexpr (!ONE) {
        const int32_t *sizes = a.counters + (int64_t)g * HOP_COUNTERS + PARTS_MAX;
        int below = tid < part ? sizes[tid] : 0;               // (at most T_PARTS_MAX ranges: the first wave's lanes)
        count = sizes[part];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) below += __shfl_xor(below, off);
        if (tid == 0) sh.below = below;
        __syncthreads();
        base = sh.below;
    }
    // starts of the segments from their lengths (a thread owns consecutive sources)
    auto scan_starts = [&]() {
        constexpr int PER = T_SOURCES / HOP_THREADS;
        int sum = 0, total;
        uint32_t squares = 0;
        const int s0 = tid * PER;
        int x[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            x[k] = s0 + k < n ? start[s0 + k] : 0;
            sum += x[k];
            squares += (uint32_t)x[k] * (uint32_t)x[k];
        }
        if (count <= T_LIST && squares > 1024u) atomicAdd(&sh.work, (int)squares);      // (the others: segments of 32 at most)
        int run = block_exclusive_scan_1024(sum, sh.scan, total);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (s0 + k < n) start[s0 + k] = run;
            run += x[k];
        }
        if (tid == 0) start[n] = total;
        __syncthreads();
        // (a thread's own stretch straight to memory would make every store touch 64 lines)
        for (int i = tid; i < n; i += HOP_THREADS) t_indptr[lo + i] = base + start[i];
        __syncthreads();
    };
    if (ONE || count <= T_LIST) {
        if constexpr (!ONE) {
            const int32_t *from = a.t_lists + (int64_t)g * 2 * a.list_stride + (int64_t)part * T_LIST;
#pragma unroll 8
            for (int i = tid; i < count; i += HOP_THREADS) list[i] = from[i];
        }
        __syncthreads();
        // (rolled loops: unrolled over the list, this function was 40 KB of code, most of which ran once per workgroup straight
        // from memory)
        for (int i = tid; i < count; i += HOP_THREADS) atomicAdd(&start[list[i] & 16383], 1);
        __syncthreads();
        scan_starts();
        if (sh.work <= T_RANK_WORK) {
            for (int i = tid; i < count; i += HOP_THREADS) {
                const int32_t x = list[i];
                sorted[atomicAdd(&start[x & 16383], 1)] = x;                   // start[s] becomes the segment's end
            }
            __syncthreads();
            for (int i = tid; i < count; i += HOP_THREADS) {
                const int32_t x = sorted[i];
                const int s = x & 16383, s0 = s > 0 ? start[s - 1] : 0, s1 = start[s];
                // (most segments hold one or two rows; the longer ones are read four at a time, or a wave waits out one LDS round
                // trip per row of its longest segment)
                int rank = 0;
                for (int q = s0; q < s1; q += 4) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int32_t y = sorted[min(q + u, s1 - 1)];
                        rank += (q + u < s1 && (y < x || (y == x && q + u < i))) ? 1 : 0;
                    }
                }
                t_indices[base + s0 + rank] = x >> 14;
            }
            return;
        }
    } else {
        // more edges than the lists hold
        constexpr int U = 8;
        for (int i0 = tid; i0 < nnz; i0 += U * HOP_THREADS) {
            int32_t x[U];
#pragma unroll
            for (int k = 0; k < U; ++k) x[k] = indices[min(i0 + k * HOP_THREADS, nnz - 1)];
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (i0 + k * HOP_THREADS < nnz && (uint32_t)(x[k] - lo) < (uint32_t)n) atomicAdd(&start[x[k] - lo], 1);
        }
        __syncthreads();
        scan_starts();
    }
    transpose_windows(indices, edge_rows, nnz, lo, n, start, list, wave_sum, sh, t_indices + base);
}

#define CR_HOP()                                                                      \
    extern __shared__ __attribute__((aligned(16))) uint32_t hop_lds[];                \
    __shared__ HopShared sh;                                                          \
    const int g = blockIdx.y;                                                         \
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);      \
    const int nnz = a.hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_NNZ]

// deals the ids of a hop (destination nodes, then chosen neighbours) to the lists of their parts, each with its position
__global__ __launch_bounds__(HOP_THREADS) void hop_part_kernel(DedupArgs a, uint32_t parts)
{
    __shared__ int count[PARTS_MAX], base[PARTS_MAX];
    const int g = blockIdx.y;
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);
    const int total = n_dst + a.hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_NNZ];
    const int tid = threadIdx.x, i0 = (int)blockIdx.x * PART_CHUNK + tid;
    if (i0 - tid >= total) return;
    const int32_t *dst = a.dst_ids + (int64_t)g * a.dst_stride, *sel = a.sel + (int64_t)g * a.sel_stride;
    if (tid < PARTS_MAX) count[tid] = 0;
    uint32_t id[PART_PER];
    int at[PART_PER];
#pragma unroll
    for (int k = 0; k < PART_PER; ++k) id[k] = hop_id(dst, sel, n_dst, min(i0 + k * HOP_THREADS, total - 1));
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PART_PER; ++k) {
        at[k] = 0;
        if (i0 + k * HOP_THREADS < total) at[k] = atomicAdd(&count[id_part(id[k], parts)], 1);
    }
    __syncthreads();
    if (tid < (int)parts) base[tid] = atomicAdd(&a.counters[(int64_t)g * HOP_COUNTERS + tid], count[tid]);
    __syncthreads();
    uint2 *lists = a.lists + (int64_t)g * a.list_stride;
#pragma unroll
    for (int k = 0; k < PART_PER; ++k) {
        const uint32_t p = id_part(id[k], parts);
        const int i = i0 + k * HOP_THREADS, slot = base[p] + at[k];
        if (i < total && slot < LIST_CAP) at32(lists, (int)p * LIST_CAP + slot) = make_uint2(id[k], (uint32_t)i);
    }
}

__global__ __launch_bounds__(HOP_THREADS) void hop_first_kernel(DedupArgs a)
{
    CR_HOP();
    hop_first<false>(a, g, n_dst, nnz, blockIdx.x, gridDim.x, hop_lds, sh);
}

__global__ __launch_bounds__(HOP_THREADS) void hop_mark_kernel(DedupArgs a)
{
    __shared__ int sum;
    const int g = blockIdx.y;
    const int n_dst = group_n_dst(a.prev_hdr, g, a.n_roots_total, a.batch_size);
    const int nnz = a.hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_NNZ];
    const int words = (nnz + 63) / 64, per = (words + (int)gridDim.x - 1) / (int)gridDim.x, w0 = min(words, (int)blockIdx.x * per);
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    const int met = mark_words<true>(a.first + (int64_t)g * a.first_stride, n_dst, nnz, w0, min(words, w0 + per), a.seen_bits + (int64_t)g * NUMBER_WORDS);
    if (lane_id() == 0 && met) atomicAdd(&sum, met);
    __syncthreads();
    if (threadIdx.x == 0) a.new_count[(int64_t)g * HOP_CHUNKS_MAX + blockIdx.x] = sum;
}

__global__ __launch_bounds__(HOP_THREADS) void hop_number_kernel(DedupArgs a)
{
    CR_HOP();
    hop_number<false>(a, g, n_dst, nnz, (int)blockIdx.x, (int)gridDim.x, hop_lds, sh);
}

// behind a frontier from the tables: the edges to the lists of their ranges of sources
constexpr int DEAL_PER = 8;
__global__ __launch_bounds__(HOP_THREADS) void hop_deal_kernel(DedupArgs a)
{
    __shared__ int count[T_PARTS_MAX], base[T_PARTS_MAX];
    const int g = blockIdx.y, tid = threadIdx.x;
    const int32_t *hdr = a.hdr + (int64_t)g * CR_HDR_WORDS;
    const int nnz = hdr[CR_HDR_NNZ], n_src = hdr[CR_HDR_N_SRC], e0 = (int)blockIdx.x * DEAL_PER * HOP_THREADS + tid;
    if (e0 - tid >= nnz) return;
    const int32_t *indices = a.indices + (int64_t)g * a.indices_stride, *edge_rows = a.edge_rows + (int64_t)g * a.edge_rows_stride;
    if (tid < T_PARTS_MAX) count[tid] = 0;
    int row[DEAL_PER], source[DEAL_PER];
    bool ok[DEAL_PER];
#pragma unroll
    for (int k = 0; k < DEAL_PER; ++k) {
        const int e = min(e0 + k * HOP_THREADS, nnz - 1);
        ok[k] = e0 + k * HOP_THREADS < nnz;
        source[k] = at32(indices, e);
        row[k] = at32(edge_rows, e);
    }
    __syncthreads();
    deal_edges<DEAL_PER>(a, g, (uint32_t)((n_src + a.t_parts - 1) / a.t_parts), ok, row, source, count, base);
}

__global__ __launch_bounds__(HOP_THREADS) void hop_transpose_kernel(DedupArgs a)
{
    CR_HOP();
    hop_transpose<false>(a, g, n_dst, a.hdr[(int64_t)g * CR_HDR_WORDS + CR_HDR_N_SRC], nnz, (int)blockIdx.x, (int)gridDim.x, hop_lds, sh);
}

// all of them for a hop that is one part
__global__ __launch_bounds__(HOP_THREADS) void hop_kernel(DedupArgs a)
{
    CR_HOP();
    hop_first<true>(a, g, n_dst, nnz, 0u, 1u, hop_lds, sh);
    __syncthreads();
    const int n_src = hop_number<true>(a, g, n_dst, nnz, 0, 1, hop_lds, sh);
    __syncthreads();
    if (a.t_indptr) hop_transpose<true>(a, g, n_dst, n_src, nnz, 0, 1, hop_lds, sh);
}

// one thread per 32 adjacency entries: find the row of the first one, then walk
__global__ __launch_bounds__(256) void edge_classes_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                           const int32_t *__restrict__ comm, int64_t n_nodes, int64_t n_entries,
                                                           uint32_t *__restrict__ out)
{
    const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t e0 = w * 32;
    if (e0 >= n_entries) return;
    int64_t lo = 0, hi = n_nodes;            // last row r with indptr[r] <= e0
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (indptr[mid] <= e0) lo = mid; else hi = mid;
    }
    int64_t r = lo, r_end = indptr[r + 1];
    int32_t cr = comm[r];
    uint32_t bits = 0;
    for (int b = 0; b < 32 && e0 + b < n_entries; ++b) {
        const int64_t e = e0 + b;
        while (e >= r_end) { ++r; r_end = indptr[r + 1]; cr = comm[r]; }
        if (comm[indices[e]] == cr) bits |= 1u << b;
    }
    out[w] = bits;
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
struct SamplePlan {
    int L;
    int32_t cap_dst[CR_MAX_LAYERS], cap_src[CR_MAX_LAYERS], cap_nnz[CR_MAX_LAYERS];
    int table_bits[CR_MAX_LAYERS];
    int64_t max_dst = 0, max_src_t = 0, max_nnz = 0, max_nnz_t = 0, max_table = 0;
    bool direct = false;      // direct-address de-duplication table (one int32 per node) instead of hashing
    int64_t table_stride = 0; // per batch, in 8-byte units
    // workspace slices
    int32_t *sel, *cnt, *newoff, *tcount, *tfill, *t_tmp, *t_pos, *order_hist, *order_cursor, *order_tiles;
    uint16_t *order_bucket;
    unsigned long long *newmask, *table;
    int32_t *hop_counters = nullptr, *hop_new_count = nullptr;      // hops in several parts (frontier in LDS)
    unsigned long long *hop_bits = nullptr;
    uint2 *hop_lists = nullptr;
    int64_t list_stride = 0;  // per batch, in entries
    size_t bytes;
};

// How a hop in several parts is cut up.  Small groups are cut finer, or most compute units sit idle.
static int hop_chunks_for(int n_batches) { return n_batches >= 32 ? PARTS_MIN : (n_batches <= 8 ? HOP_CHUNKS_MAX : 256 / n_batches); }
static int64_t hop_items_max(int n_batches) { return (n_batches < PARTS_MAX / PARTS_MIN ? PARTS_MIN * n_batches : PARTS_MAX) * (int64_t)LIST_MEAN; }
static int hop_parts_for(int64_t items, int n_batches)
{
    int parts = PARTS_MIN;
    while (parts * (int64_t)LIST_MEAN < items) parts *= 2;
    while (parts < PARTS_MAX && 2 * parts * (int64_t)n_batches <= 256) parts *= 2;
    return parts;
}
static int64_t hop_t_parts_for(int64_t cap_nnz, int64_t cap_src, int n_batches)
{
    int64_t parts = ceil_div(cap_nnz, T_MEAN);
    if (parts < ceil_div(cap_src, T_SOURCES)) parts = ceil_div(cap_src, T_SOURCES);
    return parts < hop_chunks_for(n_batches) ? hop_chunks_for(n_batches) : parts;
}

static bool hop_lds_ready()
{
    static PerDevice hop, first, transpose;
    constexpr size_t most = T_LDS_BYTES > DEDUP_LDS_BYTES ? T_LDS_BYTES : DEDUP_LDS_BYTES;
    return lds_opt_in(hop, reinterpret_cast<const void *>(&hop_kernel), most) &&
           lds_opt_in(first, reinterpret_cast<const void *>(&hop_first_kernel), DEDUP_LDS_BYTES) &&
           lds_opt_in(transpose, reinterpret_cast<const void *>(&hop_transpose_kernel), T_LDS_BYTES);
}

static cr_status make_plan(const cr_sample_cfg *cfg, int64_t n_nodes, int32_t batch_size, int32_t n_batches,
                           void *ws, SamplePlan &p)
{
    CR_REQUIRE(cfg != nullptr, CR_ERR_INVALID_ARG, "cfg is NULL");
    CR_REQUIRE(cfg->n_layers >= 1 && cfg->n_layers <= CR_MAX_LAYERS, CR_ERR_INVALID_ARG,
               "n_layers = %d outside 1..%d", cfg->n_layers, CR_MAX_LAYERS);
    CR_REQUIRE(n_nodes >= 1 && n_nodes <= 0x7FFFFFFF, CR_ERR_INVALID_ARG, "n_nodes must be in 1..2^31-1");
    CR_REQUIRE(batch_size >= 1, CR_ERR_INVALID_ARG, "batch_size must be positive");
    CR_REQUIRE(n_batches >= 1 && n_batches <= 65535, CR_ERR_INVALID_ARG, "n_batches must be in 1..65535");
    CR_REQUIRE(cfg->p_intra >= 0.5 && cfg->p_intra <= 1.0, CR_ERR_INVALID_ARG, "p_intra = %g outside [0.5, 1]", cfg->p_intra);
    CR_REQUIRE(cfg->epoch < (1u << 24), CR_ERR_INVALID_ARG, "epoch must be below 2^24");
    CR_REQUIRE(!((cfg->flags & CR_SAMPLE_TRANSPOSE_INPUT) && (cfg->flags & CR_SAMPLE_INPUT_GLOBAL_IDS)), CR_ERR_INVALID_ARG,
               "CR_SAMPLE_TRANSPOSE_INPUT and CR_SAMPLE_INPUT_GLOBAL_IDS exclude each other");
    p.L = cfg->n_layers;
    int64_t dst = batch_size;
    for (int l = p.L - 1; l >= 0; --l) {
        const int f = cfg->fanout[l];
        CR_REQUIRE(f >= 1 && f <= CR_MAX_FANOUT, CR_ERR_INVALID_ARG, "fanout[%d] = %d outside 1..%d", l, f, CR_MAX_FANOUT);
        const int64_t nnz = dst * f;
        int64_t src = dst * (1 + f);
        if (src > n_nodes) src = n_nodes;
        if (src < dst) src = dst;
        CR_REQUIRE(nnz <= 0x7FFFFFFF / 2, CR_ERR_UNSUPPORTED, "layer %d would hold %lld edges per batch", l, (long long)nnz);
        p.cap_dst[l] = (int32_t)dst;
        p.cap_src[l] = (int32_t)src;
        p.cap_nnz[l] = (int32_t)nnz;
        int bits = 4;
        while ((1ll << bits) < 2 * src) ++bits;
        CR_REQUIRE(bits <= 31, CR_ERR_UNSUPPORTED, "layer %d frontier too large for the de-duplication table", l);
        p.table_bits[l] = bits;
        p.max_dst = dst > p.max_dst ? dst : p.max_dst;
        p.max_nnz = nnz > p.max_nnz ? nnz : p.max_nnz;
        p.max_table = (1ll << bits) > p.max_table ? (1ll << bits) : p.max_table;
        if (l >= 1 || (cfg->flags & CR_SAMPLE_TRANSPOSE_INPUT)) {
            p.max_src_t = src > p.max_src_t ? src : p.max_src_t;
            p.max_nnz_t = nnz > p.max_nnz_t ? nnz : p.max_nnz_t;
        }
        dst = src;
    }
    const size_t G = (size_t)n_batches;
    Carver c(ws);
    p.sel = c.take<int32_t>(G * p.max_nnz);
    p.cnt = c.take<int32_t>(G * p.max_dst);
    p.newoff = c.take<int32_t>(G * (p.max_dst + 1));
    p.newmask = c.take<unsigned long long>(G * p.max_dst);
    p.direct = n_nodes <= 4 * p.max_table && !(cfg->flags & CR_SAMPLE_HASH_DEDUP);
    p.table_stride = p.direct ? round_up(ceil_div(n_nodes, 2), 2) : p.max_table;
    p.table = c.take<unsigned long long>(G * (size_t)p.table_stride);
    p.tcount = c.take<int32_t>(G * (p.max_src_t + 1));
    p.tfill = c.take<int32_t>(G * (p.max_src_t + 1));
    p.t_tmp = c.take<int32_t>(G * (p.max_nnz_t + 1));
    p.t_pos = c.take<int32_t>(G * (p.max_nnz_t + 1));
    if (cfg->flags & CR_SAMPLE_ROW_ORDER) {          // cells of the row-order counting sort, sized for 4096 buckets
        const size_t cells = (size_t)ORDER_BUCKETS * (size_t)ceil_div(p.max_dst, ORDER_TILE) + 1;
        p.order_hist = c.take<int32_t>(G * cells);
        p.order_cursor = c.take<int32_t>(G * cells);
        p.order_tiles = c.take<int32_t>(16384);
        p.order_bucket = c.take<uint16_t>(G * p.max_dst);
    } else {
        p.order_hist = p.order_cursor = p.order_tiles = nullptr;
        p.order_bucket = nullptr;
    }
    for (int l = 0; l < p.L; ++l) {                  // lists of the hops in several parts
        if (p.cap_nnz[l] > p.max_nnz_t) continue;    // (neither a frontier in LDS nor a transpose)
        const int64_t items = (int64_t)p.cap_dst[l] + p.cap_nnz[l], t_parts = hop_t_parts_for(p.cap_nnz[l], p.cap_src[l], n_batches);
        const int64_t lists = items > LIST_CAP && items <= hop_items_max(n_batches) ? (int64_t)hop_parts_for(items, n_batches) * LIST_CAP : 0;
        const int64_t t_lists = t_parts <= T_PARTS_MAX ? t_parts * T_LIST / 2 : 0;      // (behind the tables also where a hop is one part)
        if (p.list_stride < lists) p.list_stride = lists;
        if (p.list_stride < t_lists) p.list_stride = t_lists;
    }
    if (p.list_stride > 0) {
        p.hop_counters = c.take<int32_t>(G * HOP_COUNTERS);
        p.hop_new_count = c.take<int32_t>(G * HOP_CHUNKS_MAX);
        p.hop_bits = c.take<unsigned long long>(G * NUMBER_WORDS);
        p.hop_lists = c.take<uint2>(G * (size_t)p.list_stride);
    }
    p.bytes = c.bytes();
    return CR_OK;
}

}  // namespace cr

using namespace cr;

extern "C" cr_status cr_block_capacities(const cr_sample_cfg *cfg, int64_t n_nodes, int32_t batch_size,
                                         int32_t *cap_dst, int32_t *cap_src, int32_t *cap_nnz)
{
    SamplePlan p;
    cr_status st = make_plan(cfg, n_nodes, batch_size, 1, nullptr, p);
    if (st != CR_OK) return st;
    CR_REQUIRE(cap_dst && cap_src && cap_nnz, CR_ERR_INVALID_ARG, "output arrays must not be NULL");
    for (int l = 0; l < p.L; ++l) {
        cap_dst[l] = p.cap_dst[l];
        cap_src[l] = p.cap_src[l];
        cap_nnz[l] = p.cap_nnz[l];
    }
    return CR_OK;
}

extern "C" cr_status cr_sample_blocks_workspace_bytes(const cr_sample_cfg *cfg, int64_t n_nodes, int32_t batch_size,
                                                      int32_t n_batches, size_t *bytes)
{
    SamplePlan p;
    cr_status st = make_plan(cfg, n_nodes, batch_size, n_batches, nullptr, p);
    if (st != CR_OK) return st;
    CR_REQUIRE(bytes != nullptr, CR_ERR_INVALID_ARG, "bytes is NULL");
    *bytes = p.bytes;
    return CR_OK;
}

extern "C" cr_status cr_selftest_clock_approximation(float *result, void *stream)
{
    CR_REQUIRE(result != nullptr, CR_ERR_INVALID_ARG, "result must not be NULL");
    if (dry_run()) return CR_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(fill_u64_kernel, dim3(1), dim3(256), 0, s, reinterpret_cast<unsigned long long *>(result), (int64_t)0, (int64_t)2, 0ull);
    hipLaunchKernelGGL(clock_selftest_kernel, dim3(4096), dim3(256), 0, s, result);
    CR_LAUNCH_CHECK();
    return CR_OK;
}

extern "C" cr_status cr_sample_blocks_dedup_table(const cr_sample_cfg *cfg, int64_t n_nodes, int32_t batch_size, int32_t *kind)
{
    SamplePlan p;
    cr_status st = make_plan(cfg, n_nodes, batch_size, 1, nullptr, p);
    if (st != CR_OK) return st;
    CR_REQUIRE(kind != nullptr, CR_ERR_INVALID_ARG, "kind is NULL");
    *kind = p.direct ? CR_DEDUP_DIRECT : CR_DEDUP_HASH;
    return CR_OK;
}

extern "C" cr_status cr_graph_edge_classes(const cr_graph *graph, uint32_t *edge_intra, void *stream)
{
    CR_REQUIRE(graph != nullptr, CR_ERR_INVALID_ARG, "graph is NULL");
    CR_REQUIRE(graph->indptr && graph->indices && graph->comm, CR_ERR_INVALID_ARG, "graph has a NULL array");
    CR_REQUIRE(graph->n_nodes >= 1 && graph->n_entries >= 0, CR_ERR_INVALID_ARG, "graph sizes must be positive");
    CR_REQUIRE(edge_intra != nullptr, CR_ERR_INVALID_ARG, "edge_intra must not be NULL");
    if (dry_run() || graph->n_entries == 0) return CR_OK;
    const int64_t words = ceil_div(graph->n_entries, 32);
    hipLaunchKernelGGL(edge_classes_kernel, dim3((unsigned)ceil_div(words, 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       graph->indptr, graph->indices, graph->comm, graph->n_nodes, graph->n_entries, edge_intra);
    CR_LAUNCH_CHECK();
    return CR_OK;
}

extern "C" cr_status cr_sample_blocks(const cr_graph *graph, const cr_sample_cfg *cfg, const int32_t *roots,
                                      int64_t n_roots_total, int32_t batch_size, int32_t n_batches, void *ws,
                                      size_t ws_bytes, cr_block_set *layers, void *stream)
{
    CR_REQUIRE(graph != nullptr, CR_ERR_INVALID_ARG, "graph is NULL");
    CR_REQUIRE(graph->indptr && graph->indices && graph->comm, CR_ERR_INVALID_ARG, "graph has a NULL array");
    CR_REQUIRE(graph->n_comm >= 1, CR_ERR_INVALID_ARG, "n_comm must be positive");
    SamplePlan p;
    cr_status st = make_plan(cfg, graph->n_nodes, batch_size, n_batches, ws, p);
    if (st != CR_OK) return st;
    CR_REQUIRE(roots != nullptr && layers != nullptr, CR_ERR_INVALID_ARG, "roots / layers must not be NULL");
    CR_REQUIRE(n_roots_total > (int64_t)(n_batches - 1) * batch_size && n_roots_total <= (int64_t)n_batches * batch_size,
               CR_ERR_INVALID_ARG, "n_roots_total = %lld does not fill %d batches of %d (only the last may be short)",
               (long long)n_roots_total, n_batches, batch_size);
    CR_REQUIRE((uint64_t)cfg->first_batch + (uint64_t)n_batches <= 0xFFFFFFFFull, CR_ERR_INVALID_ARG, "batch index overflows 32 bits");
    CR_REQUIRE(ws != nullptr && aligned16(ws), CR_ERR_INVALID_ARG, "workspace must be a 16-byte aligned device pointer");
    CR_REQUIRE(ws_bytes >= p.bytes, CR_ERR_CAPACITY, "workspace of %zu bytes, %zu needed", ws_bytes, p.bytes);
    for (int l = 0; l < p.L; ++l) {
        const cr_block_set &b = layers[l];
        CR_REQUIRE(b.n_batches == n_batches && b.fanout == cfg->fanout[l], CR_ERR_INVALID_ARG,
                   "layers[%d]: n_batches / fanout do not match the request", l);
        if (!(cfg->flags & CR_SAMPLE_SMALL_FRONTIER)) {
            CR_REQUIRE(b.cap_dst >= p.cap_dst[l] && b.cap_src >= p.cap_src[l] && b.cap_nnz >= p.cap_nnz[l], CR_ERR_CAPACITY,
                       "layers[%d]: capacities (%d, %d, %d) below the bound (%d, %d, %d)", l, b.cap_dst, b.cap_src, b.cap_nnz,
                       p.cap_dst[l], p.cap_src[l], p.cap_nnz[l]);
        } else {
            // the rows of layer l are the frontier of layer l+1, which is cut at that layer's cap_src
            const int64_t rows = l == p.L - 1 ? (int64_t)batch_size
                                              : (layers[l + 1].cap_src < p.cap_dst[l] ? layers[l + 1].cap_src : p.cap_dst[l]);
            CR_REQUIRE(b.cap_dst >= rows && b.cap_src >= b.cap_dst && (int64_t)b.cap_nnz >= rows * cfg->fanout[l], CR_ERR_CAPACITY,
                       "layers[%d]: capacities (%d, %d, %d) cannot hold %lld rows of fanout %d and their own ids", l, b.cap_dst,
                       b.cap_src, b.cap_nnz, (long long)rows, cfg->fanout[l]);
        }
        CR_REQUIRE(b.hdr && b.src_ids && b.indptr && b.indices, CR_ERR_INVALID_ARG, "layers[%d] has a NULL array", l);
        CR_REQUIRE((b.t_indptr == nullptr) == (b.t_indices == nullptr), CR_ERR_INVALID_ARG,
                   "layers[%d]: t_indptr and t_indices must be given together", l);
        CR_REQUIRE(l >= 1 || b.t_indptr == nullptr || (cfg->flags & CR_SAMPLE_TRANSPOSE_INPUT), CR_ERR_UNSUPPORTED,
                   "layer 0 takes a transposed block only with CR_SAMPLE_TRANSPOSE_INPUT");
        CR_REQUIRE(l >= 1 || !(cfg->flags & CR_SAMPLE_INPUT_GLOBAL_IDS) || b.gather_ids != nullptr, CR_ERR_INVALID_ARG,
                   "CR_SAMPLE_INPUT_GLOBAL_IDS needs layers[0].gather_ids");
        CR_REQUIRE((b.row_order == nullptr && b.group_order == nullptr) || (cfg->flags & CR_SAMPLE_ROW_ORDER), CR_ERR_INVALID_ARG,
                   "layers[%d].row_order / group_order need CR_SAMPLE_ROW_ORDER (it sizes the workspace)", l);
        CR_REQUIRE(b.group_order == nullptr || (int64_t)n_batches * b.cap_dst < 0x7FFFFFFF, CR_ERR_UNSUPPORTED,
                   "layers[%d].group_order: n_batches * cap_dst does not fit 31 bits", l);
    }
    if (dry_run()) return CR_OK;

    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t q_in = (uint32_t)llround(cfg->p_intra * 65536.0);
    const uint32_t q_out = 65536u - q_in;
    const dim3 blk(256);
    bool table_clear = false;      // (direct-address table)
    for (int l = p.L - 1; l >= 0; --l) {
        const cr_block_set &b = layers[l];
        const int f = cfg->fanout[l];
        const bool root = l == p.L - 1;
        const int32_t *prev_hdr = root ? nullptr : layers[l + 1].hdr;
        const int32_t *dst_ids = root ? roots : layers[l + 1].src_ids;
        const int64_t dst_stride = root ? batch_size : layers[l + 1].cap_src;
        const int cap_dst = p.cap_dst[l];

        SelectArgs sa;
        sa.g_indptr = graph->indptr; sa.g_indices = graph->indices; sa.comm = graph->comm;
        sa.edge_intra = graph->edge_intra; sa.n_entries = graph->n_entries;
        sa.dst_ids = dst_ids; sa.dst_stride = dst_stride; sa.prev_hdr = prev_hdr;
        sa.n_roots_total = n_roots_total; sa.batch_size = batch_size; sa.fanout = f;
        sa.q_in = q_in; sa.q_out = q_out;
        sa.strict_p1 = (q_out == 0 && (cfg->flags & CR_SAMPLE_STRICT_INTRA)) ? 1u : 0u;
        sa.seed_lo = (uint32_t)cfg->seed; sa.seed_hi = (uint32_t)(cfg->seed >> 32);
        sa.ctr3 = (cfg->epoch << 8) | (DOMAIN_NEIGHBOUR << 4) | (uint32_t)l;
        sa.first_batch = cfg->first_batch;
        sa.sel = p.sel; sa.sel_stride = p.max_nnz; sa.cnt = p.cnt; sa.cnt_stride = p.max_dst;
        {   // fanout + four standard deviations and a little more: short about once in a few thousand long rows (those
            // take the general path), never near the buffer's end
            int target = f + (int)(4.0 * sqrt((double)f)) + 4;
            sa.cand_target = (uint32_t)(target > 96 ? 96 : target);
        }
        sa.exact_select = (cfg->flags & CR_SAMPLE_EXACT_RANKING) ? 1u : 0u;
        const dim3 sel_grid((unsigned)ceil_div(cap_dst, 4 * SEL_ROWS), n_batches);
        // Fewer rows per wave where 32 of them leave the chip short of waves: a wave's passes and long rows are taken one
        // after another, so a hop of a thousand roots, or of rows of hundreds of neighbours, lasts as long as its slowest
        // wave.  The packing of short rows into passes is looser then, which costs nothing on a chip that is not full.
        // Eight batches of the reddit-like graph at p = 0.9 (256 and 2816 waves of 32 rows): whole sampling 845 -> 649 us
        // (668 with at least 4 rows per wave); 32 products-like batches 1356 -> 1325; a group of one 64-root batch
        // 120 -> 113 us with its training step.  Half or twice the number of waves asked for measures the same.
        sa.rows_per_wave = QUAD_ROWS;
        while (sa.rows_per_wave > QUAD_MIN_ROWS && ceil_div(cap_dst, sa.rows_per_wave) * n_batches < QUAD_FILL_WAVES) sa.rows_per_wave /= 2;
        const dim3 quad_grid((unsigned)ceil_div(cap_dst, 4 * sa.rows_per_wave), n_batches);
        // Input-side block in global ids, every row keeps min(fanout, degree) neighbours: counts and row pointers first
        // (they need no selection), then the selection writes the chosen ids straight into the block.
        const bool global_ids = l == 0 && (cfg->flags & CR_SAMPLE_INPUT_GLOBAL_IDS), tr = !global_ids && b.t_indptr != nullptr;
        const bool direct_out = global_ids && !sa.strict_p1;
        // Frontier in LDS: hops of at most 32 parts of ids (294912) whose row pointers are known before the selection, that is
        // all but the strict setting (CR_SAMPLE_HASH_DEDUP asks for the table in so many words).  Against the tables in memory, all
        // kernels of the hop except its selection: 32 x 67 K ids (products-like, second hop) 335 -> 83 us, 32 x 6 K ids (its root
        // hop, one workgroup per batch and one launch instead of nine) 95 -> 23 us, 8 x 280 K ids (reddit-like input hop) 310 -> 92.
        // Eight parts per batch of the group and no more: the line was drawn when every part's workgroup went over all ids of its
        // batch, and the tables' kernels get shorter with fewer batches.  Whole calls beyond it, which take the tables, now against
        // this: one batch of 280 K ids (reddit-like) 162 us, 159 here; two 199, 176; one of 150 roots (products-like, transposed
        // input) 175, 150.
        const int64_t hop_items = (int64_t)cap_dst + p.cap_nnz[l];
        const int hop_chunks = hop_chunks_for(n_batches);
        const int64_t t_parts = hop_t_parts_for(p.cap_nnz[l], p.cap_src[l], n_batches);
        const bool lds_transpose = tr && t_parts <= T_PARTS_MAX && cap_dst < (1 << 17) && hop_lds_ready();
        const bool lds_hop = !global_ids && !sa.strict_p1 && !(cfg->flags & CR_SAMPLE_HASH_DEDUP) && hop_items <= hop_items_max(n_batches) &&
                             p.max_nnz_t >= p.cap_nnz[l] && (!tr || lds_transpose) && hop_lds_ready();
        const bool one_part = lds_hop && hop_items <= LIST_CAP;
        ScanArgs sc;
        sc.tile_before = nullptr;
        sc.prev_hdr = prev_hdr; sc.n_roots_total = n_roots_total; sc.batch_size = batch_size;
        sc.mode = 0; sc.in = p.cnt; sc.in_stride = p.max_dst; sc.out = b.indptr; sc.out_stride = b.cap_dst + 1;
        sc.out_copy = nullptr; sc.copy_stride = 0; sc.hdr = b.hdr;
        sc.cap_src = b.cap_src; sc.async_status = async_status();
        sc.g_indptr = graph->indptr; sc.dst_ids = dst_ids; sc.dst_stride = dst_stride; sc.fanout = f;
        sc.head_ids = nullptr; sc.head_stride = 0;
        sc.zero = (lds_hop || lds_transpose) && !one_part ? p.hop_counters : nullptr; sc.n_zero = HOP_COUNTERS;
        const dim3 scan_grid((unsigned)ceil_div(cap_dst, SCAN_TILE), n_batches);
        sa.out_indptr = nullptr; sa.out_indptr_stride = 0; sa.out_ids = nullptr; sa.out_stride = 0;
        sa.scan_here = (direct_out || lds_hop) && cap_dst <= SELECT_SCAN_ROWS && (q_in == q_out || graph->edge_intra) ? 1 : 0;
        if (direct_out || lds_hop) {
            if (cap_dst <= SCAN_TILE) {
                sc.mode = 4;
                if (direct_out) { sc.head_ids = b.src_ids; sc.head_stride = b.cap_src; }
            } else {
                hipLaunchKernelGGL(row_counts_kernel, dim3((unsigned)ceil_div(cap_dst, 256), n_batches), blk, 0, s, graph->indptr, dst_ids, dst_stride,
                                   prev_hdr, n_roots_total, batch_size, f, p.cnt, (int64_t)p.max_dst);
            }
            if (!sa.scan_here) hipLaunchKernelGGL(scan_kernel, scan_grid, dim3(SCAN_THREADS), 0, s, sc);
            sa.out_indptr = b.indptr; sa.out_indptr_stride = b.cap_dst + 1;
            sa.out_ids = direct_out ? b.gather_ids : p.sel; sa.out_stride = direct_out ? b.cap_nnz : p.max_nnz;
        }
        sa.scan = sc;
        if (q_in == q_out) hipLaunchKernelGGL(select_quad_kernel<0>, quad_grid, blk, 0, s, sa);
        else if (q_out == 0 && graph->edge_intra) hipLaunchKernelGGL(select_quad_kernel<1>, quad_grid, blk, 0, s, sa);
        else if (graph->edge_intra) hipLaunchKernelGGL(select_quad_kernel<2>, quad_grid, blk, 0, s, sa);
        else if (q_out == 0) hipLaunchKernelGGL(select_kernel<1>, sel_grid, blk, 0, s, sa);
        else hipLaunchKernelGGL(select_kernel<2>, sel_grid, blk, 0, s, sa);

        for (int grouped = 0; grouped < 2; ++grouped) {       // processing orders of this layer's destination rows
            int32_t *order = grouped ? b.group_order : b.row_order;
            if (!order) continue;
            OrderArgs oa;
            oa.prev_hdr = prev_hdr; oa.n_roots_total = n_roots_total; oa.batch_size = batch_size;
            oa.dst_ids = dst_ids; oa.dst_stride = dst_stride; oa.comm = graph->comm; oa.n_comm = graph->n_comm;
            oa.n_buckets = graph->n_comm < ORDER_BUCKETS ? graph->n_comm : ORDER_BUCKETS;
            oa.n_tiles = (int32_t)ceil_div(cap_dst, ORDER_TILE);
            oa.cells = p.order_hist; oa.offsets = p.order_cursor; oa.order = order; oa.order_stride = b.cap_dst;
            oa.grouped = grouped; oa.cap_dst = b.cap_dst;
            oa.bucket = p.order_bucket; oa.bucket_stride = p.max_dst;
            oa.cap_rows = cap_dst;
            if ((int64_t)cap_dst * (grouped ? n_batches : 1) <= ORDER_SMALL) {
                hipLaunchKernelGGL(order_small_kernel, dim3(grouped ? 1 : n_batches), dim3(1024), 0, s, oa, n_batches);
                continue;
            }
            const int n_cells = oa.n_buckets * oa.n_tiles * (grouped ? n_batches : 1);
            const dim3 og((unsigned)oa.n_tiles, n_batches);
            hipLaunchKernelGGL(order_pass_kernel<false>, og, blk, 0, s, oa);
            ScanArgs so;
            so.prev_hdr = prev_hdr; so.n_roots_total = n_roots_total; so.batch_size = batch_size;
            so.mode = 3; so.n_fixed = n_cells; so.in = p.order_hist; so.in_stride = n_cells + 1; so.out = p.order_cursor;
            so.out_stride = n_cells + 1; so.out_copy = nullptr; so.copy_stride = 0; so.hdr = b.hdr;
            so.tile_before = nullptr; so.cap_src = 0; so.async_status = nullptr; so.head_ids = nullptr; so.zero = nullptr; so.n_zero = 0;
            const int scan_tiles = (int)ceil_div(n_cells, SCAN_TILE);
            if (grouped && scan_tiles > 8 && scan_tiles <= 16384) {
                hipLaunchKernelGGL(scan_tile_sums_kernel, dim3((unsigned)scan_tiles), dim3(SCAN_THREADS), 0, s, p.order_hist, n_cells, p.order_tiles);
                hipLaunchKernelGGL(scan_tile_offsets_kernel, dim3(1), dim3(1024), 0, s, p.order_tiles, scan_tiles);
                so.tile_before = p.order_tiles;
            }
            hipLaunchKernelGGL(scan_kernel, dim3((unsigned)scan_tiles, grouped ? 1 : n_batches), dim3(SCAN_THREADS), 0, s, so);
            hipLaunchKernelGGL(order_pass_kernel<true>, og, blk, 0, s, oa);
        }

        if (!direct_out && !lds_hop) hipLaunchKernelGGL(scan_kernel, scan_grid, dim3(SCAN_THREADS), 0, s, sc);

        DedupArgs da;
        da.prev_hdr = prev_hdr; da.n_roots_total = n_roots_total; da.batch_size = batch_size; da.fanout = f;
        da.gw = f <= 16 ? 16 : (f <= 32 ? 32 : 64);
        da.dst_ids = dst_ids; da.dst_stride = dst_stride; da.sel = p.sel; da.sel_stride = p.max_nnz;
        da.direct = p.direct ? 1 : 0;
        da.table = p.table; da.table_stride = p.table_stride; da.table_bits = p.table_bits[l];
        da.hdr = b.hdr; da.src_ids = b.src_ids; da.src_stride = b.cap_src; da.cap_src = b.cap_src; da.async_status = async_status();
        da.indptr = b.indptr; da.indptr_stride = b.cap_dst + 1; da.indices = b.indices; da.indices_stride = b.cap_nnz; da.gather_ids = b.gather_ids;
        da.newcnt = p.cnt; da.newoff = p.newoff; da.newmask = p.newmask; da.row_stride = p.max_dst; da.off_stride = p.max_dst + 1;
        const dim3 grid((unsigned)ceil_div((int64_t)cap_dst * da.gw, 256), n_batches);
        da.first = p.t_pos; da.first_stride = p.max_nnz_t + 1;
        da.counters = nullptr; da.lists = nullptr; da.t_lists = nullptr; da.list_stride = 0; da.seen_bits = nullptr; da.new_count = nullptr; da.t_parts = 0;
        da.edge_rows = !lds_transpose ? nullptr : (lds_hop ? p.sel : p.t_pos); da.edge_rows_stride = lds_hop ? p.max_nnz : p.max_nnz_t + 1;
        if (global_ids) {
            da.tcount = nullptr; da.tfill = nullptr; da.t_stride = 0; da.t_indptr = nullptr; da.t_indptr_stride = 0;
            da.t_indices = nullptr; da.t_tmp = nullptr; da.t_pos = nullptr; da.tt_stride = 0;
            if (sc.head_ids) continue;                        // done with the row pointers
            if (direct_out) hipLaunchKernelGGL(frontier_head_kernel, dim3((unsigned)ceil_div(cap_dst, 256), n_batches), blk, 0, s, da);
            else hipLaunchKernelGGL(compact_ids_kernel, grid, blk, 0, s, da);
            continue;
        }

        da.tcount = tr && !lds_transpose ? p.tcount : nullptr; da.tfill = p.tfill; da.t_stride = p.max_src_t + 1;
        da.t_indptr = b.t_indptr; da.t_indptr_stride = b.cap_src + 1; da.t_indices = b.t_indices;
        da.t_tmp = p.t_tmp; da.t_pos = p.t_pos; da.tt_stride = p.max_nnz_t + 1;
        if (one_part) {
            hipLaunchKernelGGL(hop_kernel, dim3(1, n_batches), dim3(HOP_THREADS), T_LDS_BYTES > DEDUP_LDS_BYTES ? T_LDS_BYTES : DEDUP_LDS_BYTES, s, da);
            continue;
        }
        if (lds_hop) {
            const int parts = hop_parts_for(hop_items, n_batches);
            da.counters = p.hop_counters; da.lists = p.hop_lists; da.list_stride = p.list_stride; da.seen_bits = p.hop_bits; da.new_count = p.hop_new_count;
            da.t_lists = lds_transpose ? reinterpret_cast<int32_t *>(p.hop_lists) : nullptr; da.t_parts = (int32_t)t_parts;
            hipLaunchKernelGGL(hop_part_kernel, dim3((unsigned)ceil_div(hop_items, PART_CHUNK), n_batches), dim3(HOP_THREADS), 0, s, da, (uint32_t)parts);
            hipLaunchKernelGGL(hop_first_kernel, dim3((unsigned)parts, n_batches), dim3(HOP_THREADS), DEDUP_LDS_BYTES, s, da);
            hipLaunchKernelGGL(hop_mark_kernel, dim3((unsigned)hop_chunks, n_batches), dim3(HOP_THREADS), 0, s, da);
            hipLaunchKernelGGL(hop_number_kernel, dim3((unsigned)hop_chunks, n_batches), dim3(HOP_THREADS), NUMBER_LDS_BYTES, s, da);
        } else {
            if (!p.direct) {
                const int64_t table_size = 1ll << p.table_bits[l];
                hipLaunchKernelGGL(fill_u64_kernel, dim3((unsigned)(ceil_div(table_size, 512) < 4096 ? ceil_div(table_size, 512) : 4096), n_batches), blk, 0, s,
                                   p.table, p.table_stride, table_size, EMPTY);
            } else if (!table_clear) {   // once per call; every hop puts the entries it touched back
                table_clear = true;
                hipLaunchKernelGGL(fill_u64_kernel, dim3((unsigned)(ceil_div(p.table_stride, 512) < 4096 ? ceil_div(p.table_stride, 512) : 4096), n_batches), blk, 0, s,
                                   p.table, p.table_stride, p.table_stride, 0x7FFFFFFF7FFFFFFFull);
            }
            hipLaunchKernelGGL(insert_kernel, grid, blk, 0, s, da);
            hipLaunchKernelGGL(mark_new_kernel, grid, blk, 0, s, da);
            sc.mode = 1; sc.in = p.cnt; sc.in_stride = p.max_dst; sc.out = p.newoff; sc.out_stride = p.max_dst + 1;
            hipLaunchKernelGGL(scan_kernel, scan_grid, dim3(SCAN_THREADS), 0, s, sc);
            hipLaunchKernelGGL(assign_kernel, grid, blk, 0, s, da);
            hipLaunchKernelGGL(relabel_kernel, grid, blk, 0, s, da);
            if (p.direct)
                hipLaunchKernelGGL(reset_kernel, dim3((unsigned)ceil_div(p.cap_src[l], 1024), n_batches), blk, 0, s, da);
        }
        if (lds_transpose) {
            if (!lds_hop) {
                da.counters = p.hop_counters; da.list_stride = p.list_stride;
                da.t_lists = reinterpret_cast<int32_t *>(p.hop_lists); da.t_parts = (int32_t)t_parts;
                hipLaunchKernelGGL(hop_deal_kernel, dim3((unsigned)ceil_div(p.cap_nnz[l], DEAL_PER * HOP_THREADS), n_batches), dim3(HOP_THREADS), 0, s, da);
            }
            hipLaunchKernelGGL(hop_transpose_kernel, dim3((unsigned)t_parts, n_batches), dim3(HOP_THREADS), T_LDS_BYTES, s, da);
        } else if (tr) {
            sc.mode = 2; sc.in = p.tcount; sc.in_stride = p.max_src_t + 1; sc.out = b.t_indptr; sc.out_stride = b.cap_src + 1;
            sc.out_copy = p.tfill; sc.copy_stride = p.max_src_t + 1;
            hipLaunchKernelGGL(scan_kernel, dim3((unsigned)ceil_div(b.cap_src, SCAN_TILE), n_batches), dim3(SCAN_THREADS), 0, s, sc);
            hipLaunchKernelGGL(t_fill_kernel, grid, blk, 0, s, da);
            hipLaunchKernelGGL(t_rank_kernel, grid, blk, 0, s, da);
        }
    }
    CR_LAUNCH_CHECK();
    return CR_OK;
}
