// Step 2: sliding window over the last k step masks (Section 3.1 "The Sliding Window
// Technique", Fig. 4b) and Step 3: neuron-cache update (Section 3.3 items 1-2, Fig. 6).
//
// Window state ("last_k_active") is a ring of the last k step masks, one bit per neuron:
// the active set is their bitwise OR, so a 64-bit word settles 64 neurons at once.
// Everything is integer work: results are exact.
#pragma once

#include "lif_window_bits.h"

namespace lif {

// One workgroup does the window update and the deletion plan back to back.
//
// Window (Section 3.1): ring[j] holds the step masks of the last k steps; step t overwrites
// ring[t mod k].  The entry written a steps ago has age a; entries older than window_len left the window (or were
// never written) and are not read.  The bitmap of the cached set is double-buffered (set_par): a fused step writes the
// new one while others still read the old one.  Lane w owns the 64 neurons of word w:
//   prev = cached set (S_{t-1});  keep = OR of the ring entries of ages 1 .. k - 1;  S_t = keep | m
//   added = m & ~prev;  removed = prev & ~(keep | m)
// A workgroup-wide prefix sum over the popcounts puts the ids out in ascending order.
//
// Deletion plan (Section 3.3 item 1): a slot is dead iff its neuron was just removed (looked
// up in the removed words, kept in LDS).  With n' = n - c, the dead slots below n' ("holes",
// ascending) are filled by the live slots at or above n' ("fillers"): hole j takes the
// (H-1-j)-th filler - the lowest hole receives the last row, exactly what the sequential
// swap-with-last loop does.  Sources (>= n') and destinations (< n') are disjoint, so the
// moves can later run in any order.  Slots are walked in blocks of 64 (one per lane), block b
// by wave b mod 16; ballots rank the slots inside a block, a prefix over the per-block counts
// ranks the blocks.  Only the blocks below num_used are visited.
// Output of the plan: move_dst[q] for tail slot n' + q = destination slot, or -1 if dead.
//
// The loads that do not depend on the state (mask word, ring words, first block of pointers)
// are issued together with the state itself.
__global__ __launch_bounds__(kScanThreads) void k_window_plan(
    const uint8_t* __restrict__ step_mask, int ntok, int keep_tok, unsigned long long* __restrict__ ring,
    unsigned long long* __restrict__ cur_set, int ring_words, const int32_t* __restrict__ pointers, int F, int k,
    int capacity, int shrink, int32_t* __restrict__ added,
    int32_t* __restrict__ n_added, int32_t* __restrict__ removed, int32_t* __restrict__ n_removed,
    int32_t* __restrict__ move_dst, int32_t* __restrict__ hole_list, DevState* st) {
    constexpr int THREADS = kScanThreads;
    constexpr int NW = THREADS / kWave;
    __shared__ unsigned long long wave_tot[NW];
    __shared__ unsigned long long rem64[THREADS];
    __shared__ int hole_lds[kHoleLds];
    __shared__ int blk_h[THREADS], blk_f[THREADS];                // per 64-slot block: counts, then exclusive prefixes
    __shared__ int cnt_age[264];                                  // dynamic window: |union of the newest a masks| (a <= 256)
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int nwords = (F + 63) >> 6, nbytes = F >> 3;
    const bool have = tid < nwords;

    // ---- issue the state-independent loads ----
    unsigned long long m = have ? load_mask_word(step_mask, tid, nbytes) : 0ull;   // first (or only) mask of the step
    unsigned long long cur = have ? cur_set[tid] : 0ull;                             // what the cache holds now
    const unsigned long long cur1 = have ? cur_set[ring_words + tid] : 0ull;
    unsigned long long rv[kRingRegs];
#pragma unroll
    for (int j = 0; j < kRingRegs; ++j) rv[j] = (have && j < k) ? ring[(size_t)j * ring_words + tid] : 0ull;
    // slot owners of the first blocks of this wave (4096 slots over the workgroup), for the deletion plan below; the
    // array spans the capacity, entries past num_used are masked when used
    constexpr int kPtrPre = 64 / NW;
    int idpre[kPtrPre];
#pragma unroll
    for (int it = 0; it < kPtrPre; ++it) {
        const int s = (w + it * NW) * kWave + lane;
        idpre[it] = (s < capacity) ? pointers[s] : -1;
    }
    const int err = st->cur.error;
    const int t = st->cur.step;
    const int n = st->cur.num_used;
    const int wl_prev = st->cur.window_len;
    const int pos = st->cur.ring_pos;
    const int par = st->cur.set_par;
    if (par) cur = cur1;

    if (err) {
        if (tid == 0) {
            *n_added = 0;
            *n_removed = 0;
            st->cur.n_added = 0;
            st->cur.n_removed = 0;
        }
        return;
    }

    // ---- window ----
    const int slot = pos % k;                            // ring entry that this step's (first) mask replaces
    const unsigned long long prev = cur;
    unsigned long long keep = 0;
    const int oldest = min(wl_prev, k - 1);              // largest age that stays in the window
#pragma unroll
    for (int j = 0; j < kRingRegs; ++j)
        if (ring_age(j, slot, k) <= oldest) keep |= rv[j];
    if (have) {
        for (int j = kRingRegs; j < k; ++j) {                 // only for windows longer than kRingRegs steps
            const unsigned long long v = ring[(size_t)j * ring_words + tid];
            if (ring_age(j, slot, k) <= oldest) keep |= v;
        }
    }
    unsigned long long now = keep | m;                   // S_t with the full window
    int k_eff = k;
    const bool multi = ntok != 1 || keep_tok != 1;
    if (multi) {
        // Several tokens in one step (speculative verification, Section 4.3 "Speculative Decoding" and the
        // related-work note that the window is then updated with several tokens at once): all ntok masks
        // are needed for this step's FFN, but only the first keep_tok of them enter the window (one ring
        // entry per token, as if pushed one after the other); the others are transient.
        const size_t row_bytes = (size_t)nbytes;           // the host checks F % 64 == 0 for this path
        now = 0ull;
        if (have) {
            for (int i = 0; i < ntok; ++i) now |= load_mask_word(step_mask + (size_t)i * row_bytes, tid, nbytes);
            for (int j = 0; j < k; ++j) {
                const int age = ring_age(j, slot, k);        // the kept tokens overwrite the ages above k - keep_tok
                if (age <= min(wl_prev, k - keep_tok)) now |= ring[(size_t)j * ring_words + tid];
            }
        }
    }
    if (shrink && multi) {
        // Dynamic window for a pass of several tokens (Section 4.3 with the Appendix's dynamic window): T = all
        // masks of the pass is held in any case; the window after the pass - its masks by age a = 1 (newest)
        // .. k: the kept tokens, newest first, then the ring entries the pass does not overwrite - keeps the
        // newest k_eff masks, k_eff the largest count for which |T u U_a| fits the capacity (cnt_age[a], a = 0
        // .. k; the counts grow with a).  The kept tokens are subsets of T, so they always stay.
        auto age_mask = [&](int a) -> unsigned long long {        // mask of age a (1 <= a <= k), word of this lane
            if (a <= keep_tok) return load_mask_word(step_mask + (size_t)(keep_tok - a) * nbytes, tid, nbytes);
            const int m_old = a - keep_tok;                        // m_old-th most recent entry written before this pass
            if (m_old > wl_prev) return 0ull;
            return ring[(size_t)(((pos - m_old) % k + k) % k) * ring_words + tid];
        };
        for (int a = tid; a <= k; a += THREADS) cnt_age[a] = 0;
        __syncthreads();
        unsigned long long u = 0ull;
        if (have)
            for (int i = 0; i < ntok; ++i) u |= load_mask_word(step_mask + (size_t)i * nbytes, tid, nbytes);
        const unsigned long long pass_all = u;
        if (u) atomicAdd(&cnt_age[0], __popcll(u));
        for (int a = 1; a <= k; ++a) {
            if (have) u |= age_mask(a);
            if (u) atomicAdd(&cnt_age[a], __popcll(u));
        }
        __syncthreads();
        k_eff = -1;
        for (int a = 0; a <= k; ++a)
            if (cnt_age[a] <= capacity) k_eff = a;
        if (k_eff < 0) {                                     // uniform: the masks of the pass alone do not fit
            if (tid == 0) {
                st->cur.error = 3;                               // LIF_CAPACITY
                *n_added = 0;
                *n_removed = 0;
                st->cur.n_added = 0;
                st->cur.n_removed = 0;
            }
            return;
        }
        now = pass_all;
        if (have)
            for (int a = 1; a <= k_eff; ++a) now |= age_mask(a);
    }
    if (shrink && !multi) {
        // Dynamic window (Appendix, Persimmon / Phi-2: the window is reduced whenever the cache would
        // pass its memory limit): keep the newest k_eff <= k masks, k_eff the largest count whose
        // union fits the capacity.  U_a = union of the newest a masks (a = 1: this step's mask).
        for (int a = tid; a < k; a += THREADS) cnt_age[a] = 0;
        __syncthreads();
        unsigned long long ua[kRingRegs];                // ua[a - 1] = U_a, a = 1 .. min(k, kRingRegs)
        if (k <= kRingRegs && tid >= ((nwords + kWave - 1) & ~(kWave - 1))) {
            // this wave holds no mask word: nothing to count (all 16 waves share one compute unit, so the
            // idle ones would only slow the few that hold the masks)
#pragma unroll
            for (int a = 0; a < kRingRegs; ++a) ua[a] = 0ull;
        } else if (k <= kRingRegs) {
            // The ring entries in order of age (entry slot - a holds the mask pushed a steps ago) are picked out of the
            // register copy with selects on the wave-uniform index: some hundred instructions, but no second trip
            // to memory (measured: this phase 3.0 us with the reload).  Per-wave sums (two 16-bit counts per word) by
            // a prefix sum of DPP moves whose last lane holds the total, then one LDS atomic per wave and age.
            unsigned long long e[kRingRegs];
#pragma unroll
            for (int a = 1; a < kRingRegs; ++a) {
                const int idx = slot - a + (slot < a ? k : 0);
                unsigned long long v = 0ull;
#pragma unroll
                for (int j = 0; j < kRingRegs; ++j)
                    if (j == idx) v = rv[j];
                e[a] = (a <= oldest) ? v : 0ull;
            }
            unsigned long long u = m;
            ua[0] = u;
#pragma unroll
            for (int a = 1; a < kRingRegs; ++a) {
                u |= e[a];
                ua[a] = u;
            }
#pragma unroll
            for (int i = 0; i < kRingRegs / 2; ++i) {
                const int pk = __popcll(ua[2 * i]) | (__popcll(ua[2 * i + 1]) << 16);       // 64 lanes x 64 bits < 2^16
                const int v = __builtin_amdgcn_readlane(wave_inclusive_scan(pk, lane), kWave - 1);
                if (lane == 0 && v) {
                    if (2 * i < k) atomicAdd(&cnt_age[2 * i], v & 0xffff);
                    if (2 * i + 1 < k) atomicAdd(&cnt_age[2 * i + 1], (int)((unsigned)v >> 16));
                }
            }
        } else {
            unsigned long long u = m;
            for (int a = 1; a <= k; ++a) {
                if (a > 1 && a - 1 <= oldest && have) u |= ring[(size_t)((slot - (a - 1) + k) % k) * ring_words + tid];
                const int pc = __popcll(u);
                if (pc) atomicAdd(&cnt_age[a - 1], pc);
            }
        }
        __syncthreads();
        k_eff = 0;
        if (k <= kRingRegs) {
#pragma unroll
            for (int a = 1; a <= kRingRegs; ++a)
                if (a <= k && cnt_age[a - 1] <= capacity) k_eff = a;   // the counts grow with a
        } else {
            for (int a = 1; a <= k; ++a)
                if (cnt_age[a - 1] <= capacity) k_eff = a;
        }
        if (k_eff == 0) {                                    // uniform: this step's mask alone does not fit
            if (tid == 0) {
                st->cur.error = 3;                               // LIF_CAPACITY
                *n_added = 0;
                *n_removed = 0;
                st->cur.n_added = 0;
                st->cur.n_removed = 0;
            }
            return;
        }
        now = m;
        if (k <= kRingRegs) {
#pragma unroll
            for (int a = 1; a < kRingRegs; ++a)
                if (a < k_eff) now = ua[a];                  // U_a grows with a: the last one taken is U_{k_eff}
        } else if (have) {
            for (int a = 2; a <= k_eff && a - 1 <= oldest; ++a) now |= ring[(size_t)((slot - (a - 1) + k) % k) * ring_words + tid];
        }
    }
    unsigned long long abits = now & ~prev;
    unsigned long long rbits = prev & ~now;
    int off_a, off_r, tot_a, tot_r;
    block_exclusive_scan2<NW, false>(__popcll(abits), __popcll(rbits), wave_tot, &off_a, &off_r, &tot_a, &tot_r);

    const int n2 = n - tot_r;
    if (n2 < 0 || n2 + tot_a > capacity) {          // uniform: leave the window untouched
        if (tid == 0) {
            st->cur.error = 3;                           // LIF_CAPACITY
            *n_added = 0;
            *n_removed = 0;
            st->cur.n_added = 0;
            st->cur.n_removed = 0;
        }
        return;
    }
    rem64[tid] = rbits;
    lds_barrier();                                   // rem64 is read below

    // ---- deletion plan: classify the slots below n, block by block ----
    const int nblk = (n + kWave - 1) >> 6;           // <= 1024
    unsigned long long holebits = 0, fillbits = 0;   // bit it = flag of this lane in its it-th block
    for (int b = w, it = 0; b < nblk; b += NW, ++it) {
        const int s = b * kWave + lane;
        int id;
        if (it < kPtrPre) {                          // requested with the state
            id = idpre[0];
#pragma unroll
            for (int q = 1; q < kPtrPre; ++q)
                if (it == q) id = idpre[q];
            if (s >= n) id = -1;
        } else {
            id = (s < n) ? pointers[s] : -1;
        }
        bool hole = false, fill = false;
        if (s < n) {
            const bool dead = (id < 0 || id >= F) ? true : ((rem64[id >> 6] >> (id & 63)) & 1ull);
            hole = s < n2 && dead;
            fill = s >= n2 && !dead;
        }
        if (hole) holebits |= 1ull << it;
        if (fill) fillbits |= 1ull << it;
        const int ch = __popcll(__ballot(hole)), cf = __popcll(__ballot(fill));
        if (lane == 0) {
            blk_h[b] = ch;
            blk_f[b] = cf;
        }
    }
    lds_barrier();
    int H, Fc;
    // At most 64 blocks in use (4096 rows): every wave scans the block counts itself (one DPP prefix sum over
    // the lanes, both counts in one value) and picks the prefixes of its own blocks out of the lanes: no scan
    // across waves, no write-back, two barriers fewer.
    const bool few = nblk <= kWave;                  // uniform
    int ex_few = 0;
    if (few) {
        const int v = (lane < nblk) ? (blk_h[lane] | (blk_f[lane] << 16)) : 0;
        const int inc = wave_inclusive_scan(v, lane);
        ex_few = inc - v;
        const int tot = __builtin_amdgcn_readlane(inc, kWave - 1);
        H = tot & 0xffff;
        Fc = tot >> 16;
    } else {
        int pre_h, pre_f;
        const int vh = (tid < nblk) ? blk_h[tid] : 0, vf = (tid < nblk) ? blk_f[tid] : 0;
        block_exclusive_scan2<NW, false>(vh, vf, wave_tot, &pre_h, &pre_f, &H, &Fc);
        // the scan's barrier separates the reads of the counts above from these writes
        blk_h[tid] = pre_h;
        blk_f[tid] = pre_f;
        lds_barrier();
    }
    const bool in_lds = H <= kHoleLds;
    for (int b = w, it = 0; b < nblk; b += NW, ++it) {
        const bool hole = (holebits >> it) & 1ull;
        const unsigned long long bh = __ballot(hole);
        const int ph = few ? (__builtin_amdgcn_readlane(ex_few, b) & 0xffff) : blk_h[b];
        if (hole) {
            const int pos = ph + __popcll(bh & lt);
            if (in_lds) hole_lds[pos] = b * kWave + lane;
            else hole_list[pos] = b * kWave + lane;
        }
    }
    // the hole list (LDS, or global scratch when long) is read by other threads below
    if (in_lds) lds_barrier();
    else __syncthreads();
    for (int b = w, it = 0; b < nblk; b += NW, ++it) {
        const int s = b * kWave + lane;
        const bool fill = (fillbits >> it) & 1ull;
        const unsigned long long bf = __ballot(fill);
        const int pf = few ? (int)((unsigned)__builtin_amdgcn_readlane(ex_few, b) >> 16) : blk_f[b];
        if (s >= n2 && s < n) {
            int dst = -1;
            if (fill) {
                const int q = H - 1 - (pf + __popcll(bf & lt));
                if (q >= 0 && q < H) dst = in_lds ? hole_lds[q] : hole_list[q];
            }
            move_dst[s - n2] = dst;
        }
    }
    // ---- the new window and the id lists go out last: nothing in this kernel reads them back, and the plan above
    // does not wait for them ----
    if (have) {
        cur_set[par * ring_words + tid] = now;
        // (masks that the dynamic window dropped are older than window_len from now on)
        if (!multi) {
            ring[(size_t)slot * ring_words + tid] = m;
        } else {
            for (int i = max(0, keep_tok - k); i < keep_tok; ++i)
                ring[(size_t)((pos + i) % k) * ring_words + tid] =
                    load_mask_word(step_mask + (size_t)i * nbytes, tid, nbytes);
        }
    }
    while (abits) {
        added[off_a++] = tid * 64 + __ffsll((long long)abits) - 1;
        abits &= abits - 1;
    }
    while (rbits) {
        removed[off_r++] = tid * 64 + __ffsll((long long)rbits) - 1;
        rbits &= rbits - 1;
    }
    if (tid == 0) {
        *n_added = tot_a;
        *n_removed = tot_r;
        st->cur.n_added = tot_a;
        st->cur.n_removed = tot_r;
        st->cur.n_base = n2;
        st->cur.n_moved = H;
        st->cur.window_len = multi ? min(min(wl_prev + keep_tok, k), k_eff) : min(min(wl_prev + 1, k), k_eff);
        st->cur.ring_pos = (pos + (multi ? keep_tok : 1)) % k;
        st->cur.step = t + 1;
        atomicAdd(&st->c_steps, 1ull);
        atomicAdd(&st->c_added, (unsigned long long)tot_a);
        atomicAdd(&st->c_removed, (unsigned long long)tot_r);
        atomicAdd(&st->c_rows_moved, (unsigned long long)H);
    }
}

// Row moves of the deletion plan fused with the host-to-device append (Section 3.3 item 2; one contiguous bundle per neuron,
// Section 3.2).  Work item q covers tail slot s = n' + q:
//   (1) if slot s is a live tail row, copy it to its hole;  (2) if q < |added|, read the bundle of added[q] from pinned host
//   memory and write it to slot s.
// Every 16-byte piece of slot s is read (1) and overwritten (2) by the same thread in program order, holes lie below n' and
// appends at or above it, so no two work items touch the same bytes.
//
// Bound by the host link, which wants few requests in flight but never fewer than about 128 KiB.  A bundle is cut into equal
// chunks of at most kLoadChunk bytes; a unit is one chunk of one item, and every workgroup is a single wave that takes one
// unit after the other (the L1 of a compute unit returns loads in order: several waves on one would wait for each other).
// All numbers of a wave's units (ids, destinations, owners, biases: lane i those of its i-th unit) are read at once ahead
// of the first host read, and each host read is requested as soon as the stores of the unit before it have been issued.
// The units of a round are dealt one place further each round, so that the chunks read at a time fall on different parts of
// the rows.  With 32 workgroups of four waves, a bundle at a time
// each: bundles of 10 KiB, all four calls 75 -> 72 us; 2.4 KiB, 134 -> 106 us a step.
constexpr int kLoadPieces = 8;                           // pieces of 1 KiB per chunk at most
constexpr size_t kLoadChunk = kLoadPieces * 1024;
inline int load_chunks(size_t row_bytes) { return (int)((row_bytes + kLoadChunk - 1) / kLoadChunk); }

template <int NP>
__global__ __launch_bounds__(64) void k_load(char* __restrict__ matrix, int32_t* __restrict__ pointers,
                                             float* __restrict__ bias, const HostStore host,
                                             const float* __restrict__ b, const int32_t* __restrict__ added,
                                             const int32_t* __restrict__ move_dst, size_t row_bytes, int chunks,
                                             int chunk_bytes, int F, int capacity, DevState* st) {
    const int lane = threadIdx.x, nw = gridDim.x, lw = blockIdx.x;
    // unit i of this wave is number i * nw + (lw + i) mod nw; lane l reads the numbers of unit first + l
    auto unit_of = [&](int i) { return i * nw + (lw + i) % nw; };        // (below 65536 items of 6 chunks)
    int l_id = 0, l_dst = 0, l_owner = 0;
    float l_bias = 0.f, l_new = 0.f;
    auto request_lists = [&](int first) {                // (entries past the counts are read and not used)
        const int q = min(unit_of(first + lane) / chunks, min(F, capacity) - 1);
        l_id = added[q];
        l_dst = move_dst[q];
    };
    request_lists(0);
    if (st->cur.error) return;
    const int n2 = st->cur.n_base, c = st->cur.n_removed, a = st->cur.n_added;
    const int loads = a * chunks, total = max(c, a) * chunks;
    const unsigned lane_off = lane * 16u;
    f32x4 hv[NP], mv[NP];
    struct Unit {
        int s, dst, nid, off, len;
    };
    // (no branch around a load, which would make the compiler keep a second copy of its registers: a row that nothing is
    // moved from is read all the same.  Lanes past the end of the chunk read its last 16 bytes.)
    auto ask_host = [&](const Unit& r) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
            hv[p] = *reinterpret_cast<const f32x4*>(host_piece(host, max(r.nid, 0), r.off + min(p * 1024u + lane_off, r.len - 16u), row_bytes));
    };
    auto ask_row = [&](const Unit& r) {
        const char* row = matrix + (size_t)r.s * row_bytes + r.off;
#pragma unroll
        for (int p = 0; p < NP; ++p) mv[p] = *reinterpret_cast<const f32x4*>(row + min(p * 1024u + lane_off, r.len - 16u));
    };
    auto store = [&](const f32x4 (&v)[NP], const Unit& r, int slot) {
        char* row = matrix + (size_t)slot * row_bytes + r.off;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (p * 1024u + lane_off < (unsigned)r.len) *reinterpret_cast<f32x4*>(row + (p * 1024u + lane_off)) = v[p];
    };
    for (int first = 0; unit_of(first) < total; first += 64) {
        if (first > 0) request_lists(first);
        {
            const int s = min(n2 + unit_of(first + lane) / chunks, capacity - 1);
            l_owner = pointers[s];
            l_bias = bias[s];
            if ((unsigned)l_id >= (unsigned)F) l_id = -1;        // (not a neuron: its slot is left alone)
            l_new = b[max(l_id, 0)];
        }
        auto unit = [&](int i) {                         // i-th one from `first`
            const int u = unit_of(first + i), q = u / chunks, ch = u - q * chunks;
            Unit r;
            r.s = n2 + q;
            r.dst = __builtin_amdgcn_readlane(l_dst, i);
            if (q >= c) r.dst = -1;
            r.nid = __builtin_amdgcn_readlane(l_id, i);
            r.off = ch * chunk_bytes;
            r.len = min(chunk_bytes, (int)row_bytes - r.off);
            return r;
        };
        auto owner = [&](const Unit& r, int i, bool fresh) {
            if (r.off == 0 && lane == i) {
                if (r.dst >= 0) {
                    pointers[r.dst] = l_owner;
                    bias[r.dst] = l_bias;
                }
                if (fresh) {
                    pointers[r.s] = r.nid;
                    bias[r.s] = l_new;
                }
            }
        };
        int i = 0;
        if (unit_of(first) < loads) {
            Unit cu = unit(0);
            ask_host(cu);
            ask_row(cu);
            for (;;) {
                if (cu.dst >= 0) store(mv, cu, cu.dst);
                if (cu.nid >= 0) store(hv, cu, cu.s);
                owner(cu, i, cu.nid >= 0);
                ++i;
                if (i == 64 || unit_of(first + i) >= loads) break;
                cu = unit(i);
                ask_host(cu);
                ask_row(cu);
            }
        }
        for (; i < 64 && unit_of(first + i) < total; ++i) {      // more neurons removed than added: moves only
            const Unit r = unit(i);
            if (r.dst < 0) continue;
            ask_row(r);
            store(mv, r, r.dst);
            owner(r, i, false);
        }
    }
    if (lw == 0 && lane == 0) {
        st->cur.num_used = n2 + a;
        atomicAdd(&st->c_h2d_bytes, (unsigned long long)a * row_bytes);
    }
}

// Empty cache: no mask in the window, state and counters zero, no word handed over yet (the stamps start again).
// `words`: the hand-over words of the fused step, then the window ring and the two bitmaps of the cached set.
__global__ void k_reset(unsigned long long* __restrict__ words, int total_words, int32_t* __restrict__ stamp,
                        int capacity, DevState* st) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    for (int j = i; j < total_words; j += gridDim.x * blockDim.x) words[j] = 0ull;
    for (int j = i; j < capacity; j += gridDim.x * blockDim.x) stamp[j] = -1;   // no activation from a fused step
    if (i == 0) {
        DevState z = {};
        *st = z;
    }
}

}  // namespace lif
