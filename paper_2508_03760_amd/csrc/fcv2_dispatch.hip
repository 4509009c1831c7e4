// fcv2_dispatch.hip -- fcv2_dispatch_quant: stable counting sort of the routed copies, then quantize-and-scatter (Sections 3.1, 4.4).
#include <atomic>

#include "fcv2_host.h"

namespace fcv2 {

// ---- dispatch: stable counting sort of the routed copies by expert, then quantize-and-scatter ------------------------
// No order-dependent atomics, no waiting between blocks.  Small routings are one launch, the quantize-and-scatter kernel
// planning for itself (self_planned, plan_block); middle-sized ones two (ranked_plan, k_dispatch_rank); otherwise three:
//   1. k_dispatch_count_rank   per chunk of 256 routed slots: the chunk's histogram over the experts, and for every slot
//                              its stable rank among the chunk's slots of the same expert (one byte);
//   2. k_dispatch_scan_chunks  per expert: exclusive prefix of the histograms over the chunks (in place) and the total;
//   3. the quantize-and-scatter kernel: every block scans the E totals itself (expert starts), forms the destination row
//      of each of its routed copies as start[e] + copies in earlier chunks + rank inside the chunk, and publishes
//      row_src (block 0 also expert_offsets) -- all of it while its tokens' loads are in flight.
// Ids outside [0, E) (including -1) are dropped slots.

// Exclusive prefix sum of one value per thread over a block of up to 8 waves; *total gets the block sum.
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t* lds8, int32_t* total) {
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = (blockDim.x + 63) >> 6;
    int32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t up = __shfl_up(inc, d);
        if ((int)lane >= d) inc += up;
    }
    if (lane == 63) lds8[wave] = inc;
    __syncthreads();
    int32_t before = 0, all = 0;
    for (uint32_t w = 0; w < n_waves; ++w) {
        const int32_t t = lds8[w];
        if (w < wave) before += t;
        all += t;
    }
    *total = all;
    __syncthreads();
    return before + inc - v;
}

// Histogram of the chunk and stable in-chunk rank of every slot.  hist[chunk][e]; lrank[i] < 256.
// Every wave keeps, per expert, the 64-bit mask of its lanes that route to it (LDS integer OR: the result does not depend
// on the order of the lanes); a lane's rank inside the wave is the number of set bits below its own, the wave's count the
// number of set bits.  MASKS = false (more experts than the masks' LDS allows): the wave finds the lanes of each distinct
// expert with ballots instead, one round per distinct id.
template <bool MASKS>
__global__ __launch_bounds__(kChunk) void k_dispatch_count_rank(const int32_t* __restrict__ ids, uint32_t n_slots, uint32_t E,
                                                                int32_t* __restrict__ hist, uint8_t* __restrict__ lrank) {
    extern __shared__ uint32_t lds_cr[];  // MASKS: [kChunk/64][E][2] lane masks; else [kChunk/64][E] counts
    constexpr uint32_t kW = kChunk / 64;
    const uint32_t words = MASKS ? 2u : 1u;
    for (uint32_t t = threadIdx.x; t < kW * E * words; t += kChunk) lds_cr[t] = 0;
    __syncthreads();
    const uint32_t i = blockIdx.x * kChunk + threadIdx.x;
    const uint32_t wave = threadIdx.x / 64, lane = threadIdx.x & 63;
    int32_t e = -1;
    if (i < n_slots) {
        e = ids[i];
        if (e < 0 || (uint32_t)e >= E) e = -1;
    }
    uint32_t rank = 0;  // lanes below me in this wave with the same expert
    if (MASKS) {
        if (e >= 0) atomicOr(&lds_cr[(wave * E + (uint32_t)e) * 2 + (lane >> 5)], 1u << (lane & 31));
        __syncthreads();
        if (e >= 0) {
            uint32_t before = 0;
            for (uint32_t wv = 0; wv < wave; ++wv) before += __popc(lds_cr[(wv * E + e) * 2]) + __popc(lds_cr[(wv * E + e) * 2 + 1]);
            const uint32_t lo = lds_cr[(wave * E + e) * 2], hi = lds_cr[(wave * E + e) * 2 + 1];
            rank = lane < 32 ? __popc(lo & ((1u << lane) - 1u)) : __popc(lo) + __popc(hi & ((1u << (lane - 32)) - 1u));
            lrank[i] = (uint8_t)(before + rank);  // at most 255: a chunk has 256 slots
        }
        for (uint32_t t = threadIdx.x; t < E; t += kChunk) {
            int32_t c = 0;
#pragma unroll
            for (uint32_t wv = 0; wv < kW; ++wv) c += __popc(lds_cr[(wv * E + t) * 2]) + __popc(lds_cr[(wv * E + t) * 2 + 1]);
            hist[(uint64_t)blockIdx.x * E + t] = c;
        }
    } else {
        uint64_t todo = __ballot(e >= 0);
        while (todo) {  // one round per distinct expert id in the wave; every round clears at least one lane
            const int leader = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)todo) - 1);
            const int32_t el = __builtin_amdgcn_readlane(e, leader);  // a scalar read, not a trip through the LDS crossbar
            const uint64_t same = __ballot(e == el);
            if (e == el) {
                rank = __popcll(same & ((1ull << lane) - 1ull));
                if ((int)lane == leader) lds_cr[wave * E + el] = __popcll(same);
            }
            todo &= ~same;
        }
        __syncthreads();
        if (e >= 0) {
            uint32_t before = 0;
            for (uint32_t wv = 0; wv < wave; ++wv) before += lds_cr[wv * E + e];
            lrank[i] = (uint8_t)(before + rank);
        }
        for (uint32_t t = threadIdx.x; t < E; t += kChunk) {
            int32_t c = 0;
#pragma unroll
            for (uint32_t wv = 0; wv < kW; ++wv) c += (int32_t)lds_cr[wv * E + t];
            hist[(uint64_t)blockIdx.x * E + t] = c;
        }
    }
}

// One wave per expert: exclusive prefix over the chunks, in place; totals[e] = count of expert e.  A lane takes
// consecutive chunks; the scan across the lanes is a shuffle scan, so the kernel has no barrier.
__global__ __launch_bounds__(64) void k_dispatch_scan_chunks(int32_t* __restrict__ hist, uint32_t n_chunks, uint32_t E,
                                                             int32_t* __restrict__ totals) {
    const uint32_t e = blockIdx.x, lane = threadIdx.x;
    const uint32_t per = (n_chunks + 63) / 64;  // consecutive chunks per lane
    const uint32_t c0 = min(lane * per, n_chunks), c1 = min(c0 + per, n_chunks);
    int32_t s = 0;
    if (per <= 4) {  // up to 256 chunks (65,536 routed slots): four independent loads per lane
        int32_t v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) v[k] = hist[(uint64_t)min(c0 + k, n_chunks - 1u) * E + e];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            if (c0 + k >= c1) v[k] = 0;
            s += v[k];
        }
        int32_t inc = s;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t up = __shfl_up(inc, d);
            if ((int)lane >= d) inc += up;
        }
        if (lane == 63) totals[e] = inc;
        int32_t run = inc - s;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            if (c0 + k < c1) hist[(uint64_t)(c0 + k) * E + e] = run;
            run += v[k];
        }
    } else {
        for (uint32_t c = c0; c < c1; ++c) s += hist[(uint64_t)c * E + e];
        int32_t inc = s;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t up = __shfl_up(inc, d);
            if ((int)lane >= d) inc += up;
        }
        if (lane == 63) totals[e] = inc;
        int32_t run = inc - s;
        for (uint32_t c = c0; c < c1; ++c) {
            const int32_t v = hist[(uint64_t)c * E + e];
            hist[(uint64_t)c * E + e] = run;
            run += v;
        }
    }
}

// The plan of middle-sized routings in one launch: block e goes through all ids, which stay in registers (16 per thread),
// and writes rank[i], the number of earlier slots of expert e, for every slot i of that expert, and totals[e].  A wave
// counts with ballots; the counts of (step, wave) are scanned by one wave; matches, one in E, are ranked in a second pass over the
// registers.  ids are 16-byte aligned and fill at least one step.
constexpr uint32_t kRankThreads = 1024, kRankSteps = 4;
__global__ __launch_bounds__(kRankThreads) void k_dispatch_rank(const int32_t* __restrict__ ids, uint32_t n_slots, int32_t* __restrict__ totals,
                                                                int32_t* __restrict__ rank) {
    constexpr uint32_t W = kRankThreads / 64, KMAX = kRankSteps;
    __shared__ uint32_t before[KMAX * W];  // [step][wave]: the counts, then their exclusive sums
    const int32_t mine = (int32_t)blockIdx.x;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int4* ids4 = reinterpret_cast<const int4*>(ids);
    const uint32_t n4 = n_slots >> 2;
    int4 e[KMAX];
#pragma unroll
    for (uint32_t k = 0; k < KMAX; ++k) e[k] = ids4[min(k * kRankThreads + threadIdx.x, n4 - 1u)];
    uint64_t m[4];
    auto matches = [&](uint32_t k) {
        const bool in = k * kRankThreads + threadIdx.x < n4;
        m[0] = __ballot(in && e[k].x == mine);
        m[1] = __ballot(in && e[k].y == mine);
        m[2] = __ballot(in && e[k].z == mine);
        m[3] = __ballot(in && e[k].w == mine);
    };
#pragma unroll
    for (uint32_t k = 0; k < KMAX; ++k) {
        matches(k);
        if (lane == 0) before[k * W + wave] = __popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]);
    }
    __syncthreads();
    if (wave == 0) {
        constexpr uint32_t PER = KMAX * W / 64;
        uint32_t c[PER], sum = 0;
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            c[j] = before[lane * PER + j];
            sum += c[j];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t up = __shfl_up(inc, d);
            if ((int)lane >= d) inc += up;
        }
        uint32_t run = inc - sum;
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            before[lane * PER + j] = run;
            run += c[j];
        }
        if (lane == 63) {  // the last zero to three slots, and the total
            for (uint32_t i = 4 * n4; i < n_slots; ++i)
                if (ids[i] == mine) rank[i] = (int32_t)inc++;
            totals[mine] = (int32_t)inc;
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < KMAX; ++k) {
        matches(k);
        if ((m[0] | m[1] | m[2] | m[3]) == 0) continue;  // uniform in the wave
        uint32_t r = before[k * W + wave];
#pragma unroll
        for (int j = 0; j < 4; ++j) r += __builtin_amdgcn_mbcnt_hi((uint32_t)(m[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[j], 0u));
        int32_t* at = rank + 4 * (k * kRankThreads + threadIdx.x);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((m[j] >> lane) & 1u) at[j] = (int32_t)r++;
    }
}

// Expert starts (exclusive scan of the totals) into start[0..E), by the whole block, in two steps so that a caller can put
// other loads between them: the thread's share of the totals is read and summed first, the scan follows.  The second
// step returns the number of routed copies and ends with a barrier: start[] is complete for every thread.
struct StartsShare {
    uint32_t e0, e1;
    int32_t sum;
};
__device__ __forceinline__ StartsShare expert_starts_read(const int32_t* __restrict__ totals, uint32_t E) {
    const uint32_t per = (E + blockDim.x - 1) / blockDim.x;  // consecutive experts per thread
    StartsShare sh;
    sh.e0 = min(threadIdx.x * per, E);
    sh.e1 = min(sh.e0 + per, E);
    sh.sum = 0;
    for (uint32_t e = sh.e0; e < sh.e1; ++e) sh.sum += totals[e];
    return sh;
}
__device__ __forceinline__ int32_t expert_starts_scan(const StartsShare& sh, const int32_t* __restrict__ totals, int32_t* start, int32_t* lds8) {
    int32_t total;
    int32_t run = block_exclusive_scan(sh.sum, lds8, &total);
    for (uint32_t e = sh.e0; e < sh.e1; ++e) {
        start[e] = run;
        run += totals[e];
    }
    __syncthreads();
    return total;
}

// Destination row of routed slot i (or -1 for a dropped one) from the three planning results.
__device__ __forceinline__ int32_t dest_row_of(uint32_t i, const int32_t* __restrict__ ids, uint32_t E, const int32_t* __restrict__ hist,
                                               const uint8_t* __restrict__ lrank, const int32_t* start) {
    const int32_t e = ids[i];
    if (e < 0 || (uint32_t)e >= E) return -1;
    return start[e] + hist[(uint64_t)(i / kChunk) * E + e] + (int32_t)lrank[i];
}

// Only for row shapes the row-staged kernel cannot take: destination rows written out for the direct kernel.
__global__ __launch_bounds__(kChunk) void k_dispatch_dest(const int32_t* __restrict__ ids, uint32_t n_slots, uint32_t E,
                                                          const int32_t* __restrict__ hist, const int32_t* __restrict__ totals,
                                                          const uint8_t* __restrict__ lrank, int32_t* __restrict__ expert_offsets,
                                                          int32_t* __restrict__ dest, int32_t* __restrict__ row_src, uint32_t fresh) {
    extern __shared__ int32_t start[];  // [E]
    __shared__ int32_t lds8[8];
    const int32_t total = expert_starts_scan(expert_starts_read(totals, E), totals, start, lds8);
    if (blockIdx.x == 0) {
        for (uint32_t e = threadIdx.x; e < E; e += kChunk) expert_offsets[e] = start[e];
        if (threadIdx.x == 0) expert_offsets[E] = total;
    }
    const uint32_t i = blockIdx.x * kChunk + threadIdx.x;
    if (i < n_slots) {
        const int32_t r = dest_row_of(i, ids, E, hist, lrank, start);
        dest[i] = r;
        if (r >= 0) row_src[r] = (int32_t)i;
        if (fresh && i >= (uint32_t)total) row_src[i] = -1;
    }
}

// ---- quantize-and-scatter -------------------------------------------------------------------------------------------
// Every token is quantized once and its packed row stored K times.  `rec` holds the row's section offsets (align 16).
// Rows are multiples of 32 elements, so a lane (32 consecutive elements) never straddles rows.
//
// What the copies cost is decided by how the stores meet the 128-byte lines of the send buffer: rows are 16-byte aligned
// only, so a store instruction that writes "this wave's piece of a plane" starts and ends inside lines, and metadata
// written by one lane in four touches a few bytes of each line.  The main kernel therefore assembles whole records in
// LDS and copies each to its K destinations as one contiguous run whose store instructions cover 8 whole lines each,
// with the non-temporal hint (measured on the MI355X, 65,536 copies, this kernel alone: 2-bit rows of 2,352 bytes
// 83 -> 58 us, 8-bit rows of 7,728 bytes 174 -> 119 us).  The direct kernel below it serves the shapes whose records do not fit.

// Lane's share of a record, written at `o` (the record's first byte, LDS or global) through `ST`.
template <int BITS, int LPG, bool SR, class ST>
__device__ __forceinline__ void put_lane(const ST& st, const Rec& rec, uint32_t r, uint32_t lig, uint32_t meta_mode, const uint32_t (&c)[8],
                                         const GroupMeta& m) {
    using P = Planes<BITS>;
    constexpr int U = 4;
    uint32_t q4[U], q2[U], q1 = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        q4[u] = P::w4 ? pack_plane4<P::sh4, BITS>(c[2 * u], c[2 * u + 1]) : 0u;
        q2[u] = P::w2 ? pack_plane2<P::sh2, BITS>(c[2 * u], c[2 * u + 1]) : 0u;
        if (P::w1) q1 |= pack_plane1<P::sh1, BITS>(c[2 * u], c[2 * u + 1]) << (8 * u);
    }
    if (P::w8) {
        st.halves(rec.plane8 + 32u * r, make_uint4(c[0], c[1], c[2], c[3]), make_uint4(c[4], c[5], c[6], c[7]));
    }
    if (P::w4) st.plane(rec.plane4 + 16u * r, make_uint4(q4[0], q4[1], q4[2], q4[3]));
    if (P::w2) st.plane(rec.plane2 + 8u * r, make_uint2(q2[0] | (q2[1] << 16), q2[2] | (q2[3] << 16)));
    if (P::w1) st.plane(rec.plane1 + 4u * r, q1);
    if (lig == 0) {
        const uint32_t g = r / LPG;
        if (meta_mode == kMetaInt) {
            st.meta(rec.scale + g, (uint8_t)m.raw_s);
            st.meta(rec.zero + g, (uint8_t)m.raw_z);
        } else if (meta_mode == kMetaFp32) {
            st.meta(rec.scale + 4u * g, m.s);
            st.meta(rec.zero + 4u * g, m.lo);
        } else {
            st.meta(rec.scale + 2u * g, (uint16_t)(f2u(m.s) >> 16));
            st.meta(rec.zero + 2u * g, (uint16_t)(f2u(m.lo) >> 16));
        }
        if (SR) {
            st.meta(rec.spike_val + 4u * g, m.sv);
            if (rec.idx_bf16)
                st.meta(rec.spike_idx + 4u * g, idx_pair_to_bf16(m.si));
            else
                st.meta(rec.spike_idx + 2u * g, (uint16_t)m.si);
        }
    }
}

struct PutLds {  // into a record staged in LDS
    uint8_t* o;
    template <class V> __device__ __forceinline__ void plane(uint32_t off, V v) const { *reinterpret_cast<V*>(o + off) = v; }
    template <class V> __device__ __forceinline__ void meta(uint32_t off, V v) const { *reinterpret_cast<V*>(o + off) = v; }
    __device__ __forceinline__ void halves(uint32_t off, uint4 a, uint4 b) const {
        plane(off, a);
        plane(off + 16u, b);
    }
};
template <bool NT_META> struct PutGlobal {  // straight into the send buffer
    uint8_t* o;
    template <class V> __device__ __forceinline__ void plane(uint32_t off, V v) const { store_stream(o + off, v); }
    template <class V> __device__ __forceinline__ void meta(uint32_t off, V v) const {
        if (NT_META) store_stream(o + off, v);
        else *reinterpret_cast<V*>(o + off) = v;
    }
    // a lane's 32 bytes of the 8-bit plane as two stores 32 bytes apart per lane: half lines, so no hint
    __device__ __forceinline__ void halves(uint32_t off, uint4 a, uint4 b) const {
        *reinterpret_cast<uint4*>(o + off) = a;
        *reinterpret_cast<uint4*>(o + off + 16u) = b;
    }
};

constexpr int kRowsBlockMax = 512;  // threads of the row-staged kernel (8 waves)

// Row-staged kernel.  A block owns `rows_per_block` consecutive tokens (blockDim = their lanes rounded up to whole waves,
// chosen on the host: the count up to 64 that leaves the fewest idle lanes; 1 and 2 rows measure the same at H = 7168).
// Dynamic LDS: per wave the transpose scratch | the records | the destination rows | the tables.
constexpr uint32_t kPlanChunks = 0;  // k_dispatch_count_rank and k_dispatch_scan_chunks: hist, lrank, totals
constexpr uint32_t kPlanRanked = 1;  // k_dispatch_rank: rank, totals
constexpr uint32_t kPlanSelf = 2;    // no launch before this one (plan_block)
struct DispatchPlan {  // what the planning launches left in the workspace, and the two index outputs of the call
    const int32_t* ids;
    const int32_t* hist;
    const int32_t* totals;
    const uint8_t* lrank;
    const int32_t* rank;  // kPlanRanked only (otherwise anything that may be read at a slot's index)
    int32_t* expert_offsets;
    int32_t* row_src;
    uint32_t mode;  // who planned: kPlanChunks, kPlanRanked, kPlanSelf
    uint32_t E;
    uint32_t totals_last;  // last entry of totals that may be read
    uint32_t fresh_rows;  // T * K when send buffer and row_src hold no values yet (fcv2_fresh.h), else 0
};

// The whole plan of a small routing, made by every block for itself under its token loads instead of by two launches before
// the kernel.  Every block counts all routed slots in LDS, per expert the total in the low and the slots before the block's
// own in the high half of one word (integer additions: their order does not matter), wave 0 turns them into
// start[e] = first row of the expert + the slots of it in front of this block, start[E] = all routed copies.  Returns the
// rank of thread i < 64's slot among the block's slots of the same expert; block 0 writes expert_offsets.
__device__ __forceinline__ uint32_t plan_block(const DispatchPlan& plan, uint32_t n_slots, uint32_t first, uint32_t n_slots_here, int32_t my_e,
                                               uint32_t* counts, uint32_t* start) {
    constexpr uint32_t BATCH = 8;  // loads of four ids a thread has in flight: 8192 slots are one round of 256 threads
    // Neighbouring lanes often meet at a popular expert: up to 16 copies of the counters, a lane uses copy lane % copies.
    // Copies lie an odd number of words apart, so that the copies of one counter sit in different banks.
    const uint32_t stride = plan.E | 1u, room = min(blockDim.x >> 6, 2u) * (kWaveScratchBytes / 4);
    uint32_t copies = 1;
    if (n_slots > 4 * blockDim.x)
        while (copies < 16 && 2 * copies * stride <= room) copies *= 2;
    uint32_t* mine = counts + (threadIdx.x & (copies - 1)) * stride;
    for (uint32_t i = threadIdx.x; i < copies * stride; i += blockDim.x) counts[i] = 0u;
    __syncthreads();
    const int4* ids4 = reinterpret_cast<const int4*>(plan.ids);
    const uint32_t n4 = n_slots >> 2;
    auto count = [&](int32_t e, uint32_t i) {
        if ((uint32_t)e < plan.E) atomicAdd(&mine[e], i < first ? 0x10001u : 1u);
    };
    for (uint32_t i0 = threadIdx.x; i0 < n4; i0 += BATCH * blockDim.x) {
        int4 e[BATCH];
#pragma unroll
        for (uint32_t k = 0; k < BATCH; ++k) e[k] = ids4[min(i0 + k * blockDim.x, n4 - 1u)];
#pragma unroll
        for (uint32_t k = 0; k < BATCH; ++k) {
            const uint32_t i = i0 + k * blockDim.x;
            if (i >= n4) break;
            count(e[k].x, 4 * i);
            count(e[k].y, 4 * i + 1);
            count(e[k].z, 4 * i + 2);
            count(e[k].w, 4 * i + 3);
        }
    }
    const uint32_t rest = 4 * n4 + threadIdx.x;
    if (rest < n_slots) count(plan.ids[rest], rest);
    __syncthreads();
    if (copies > 1) {
        for (uint32_t e = threadIdx.x; e < plan.E; e += blockDim.x) {
            uint32_t both = 0;
            for (uint32_t c = 0; c < copies; c += 2) both += counts[c * stride + e] + counts[(c + 1) * stride + e];
            counts[e] = both;
        }
        __syncthreads();
    }
    uint32_t rank = 0;
    if (threadIdx.x < 64) {
        const uint32_t lane = threadIdx.x;
        const uint32_t per = (plan.E + 63) / 64, e0 = min(lane * per, plan.E), e1 = min(e0 + per, plan.E);  // at most 4 each
        uint32_t both[4], sum = 0;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) both[k] = counts[min(e0 + k, plan.E - 1u)];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            if (e0 + k >= e1) both[k] = 0;
            sum += both[k] & 0xFFFFu;
        }
        uint32_t inc = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t up = __shfl_up(inc, d);
            if ((int)lane >= d) inc += up;
        }
        uint32_t run = inc - sum;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            if (e0 + k < e1) {
                start[e0 + k] = run + (both[k] >> 16);
                if (blockIdx.x == 0) plan.expert_offsets[e0 + k] = (int32_t)run;
            }
            run += both[k] & 0xFFFFu;
        }
        if (lane == 63) {
            start[plan.E] = inc;
            if (blockIdx.x == 0) plan.expert_offsets[plan.E] = (int32_t)inc;
        }
        for (uint32_t j = 0; j < n_slots_here; ++j) {
            const int32_t ej = __builtin_amdgcn_readlane(my_e, (int)j);
            rank += (ej == my_e && j < lane) ? 1u : 0u;
        }
    }
    return rank;
}

// CHUNKS: planned by kPlanChunks; else by one of the other two, a branch on plan.mode.  With all three behind run-time branches the
// largest routings paid 0.5 us of 60.
template <int BITS, int LPG, bool SR, bool INT_META, bool CHUNKS>
__global__ __launch_bounds__(kRowsBlockMax) void k_dispatch_rows_t(const uint4* __restrict__ x, uint32_t T, uint32_t lanes_per_row,
                                                                  uint32_t K, DispatchPlan plan, uint8_t* __restrict__ send, Rec rec,
                                                                  uint32_t row_bytes, uint32_t meta_mode_arg, uint32_t rows_per_block) {
    // integer metadata is a compile-time variant, as in the quantize kernel: it would cost the float formats registers
    const uint32_t meta_mode = INT_META ? kMetaInt : (meta_mode_arg == kMetaFp32 ? kMetaFp32 : kMetaBf16);
    extern __shared__ uint4 smem[];
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t n_waves = blockDim.x >> 6;
    uint4* scratch = smem + wave * (64 * kRowU4);
    uint4* recs = smem + n_waves * (64 * kRowU4);
    const uint32_t row_pieces = row_bytes >> 4;
    int32_t* drow = reinterpret_cast<int32_t*>(recs + rows_per_block * row_pieces);
    int32_t* start = drow + rows_per_block * K;
    float* tabs = reinterpret_cast<float*>(start + plan.E + 8);
    const uint32_t row0 = blockIdx.x * rows_per_block;
    const uint32_t rows_here = min(rows_per_block, T - row0);
    const uint32_t block_lanes = rows_here * lanes_per_row;
    // Planning, arranged so that nothing in it is waited for alone.  Loads return in the order they were issued: the
    // expert id of "my" routed slot and wave 0's share of the expert totals go out first, the tokens after them.  Wave 0
    // turns the totals into the expert starts (a scan inside one wave: no barrier of its own) while the tokens are on
    // their way; after the block's barrier the two gathers that complete a destination row are issued, and they arrive
    // while the tokens are being quantized.
    const uint32_t n_slots_here = rows_here * K;
    const uint32_t my_slot = row0 * K + threadIdx.x;
    // Both small reads are unconditional (clamped addresses, every wave) and looked at only after the tokens' loads are
    // out: a branch around a load, or a glance at its value, would make the wave wait for it right here.
    int32_t my_e = plan.ids[min(my_slot, T * K - 1u)];
    const uint32_t per = (plan.E + 63) / 64;  // consecutive experts per lane of wave 0
    const uint32_t e0 = min(lane * per, plan.E), e1 = min(e0 + per, plan.E);
    int32_t tot[4];  // up to 256 experts: the lane's totals, four independent loads
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) tot[k] = plan.totals[min(e0 + k, CHUNKS ? plan.E - 1u : plan.totals_last)];
    const int32_t my_ranked = CHUNKS ? 0 : plan.rank[min(my_slot, T * K - 1u)];
    const bool self = !CHUNKS && plan.mode == kPlanSelf;
    const bool has_tile = wave * 64 < block_lanes;  // whole waves past the block's last row only help with the copies
    TileIn in = {};
    if (has_tile) in = tile_load(x, (row0 * lanes_per_row + wave * 64) * 4, lane, (block_lanes - wave * 64) * 4);
    if (threadIdx.x >= n_slots_here) my_e = -1;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
        if (per > 4 || e0 + k >= e1) tot[k] = 0;
    if (my_e < 0 || (uint32_t)my_e >= plan.E) my_e = -1;
    int32_t my_before = 0, my_rank = 0;
    if (self) {
        my_rank = (int32_t)plan_block(plan, T * K, row0 * K, n_slots_here, my_e, reinterpret_cast<uint32_t*>(smem),
                                      reinterpret_cast<uint32_t*>(start));
    } else if (wave == 0) {
        int32_t my_sum = tot[0] + tot[1] + tot[2] + tot[3];
        if (per > 4)  // more than 256 experts: read in a loop (each read waited for; such routings are rare)
            for (uint32_t e = e0; e < e1; ++e) my_sum += plan.totals[e];
        int32_t inc = my_sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t up = __shfl_up(inc, d);
            if ((int)lane >= d) inc += up;
        }
        int32_t run = inc - my_sum;
        if (per <= 4) {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                if (e0 + k < e1) {
                    start[e0 + k] = run;
                    if (blockIdx.x == 0) plan.expert_offsets[e0 + k] = run;
                }
                run += tot[k];
            }
        } else {
            for (uint32_t e = e0; e < e1; ++e) {
                start[e] = run;
                if (blockIdx.x == 0) plan.expert_offsets[e] = run;
                run += plan.totals[e];
            }
        }
        if (lane == 63) start[plan.E] = inc;
        if (blockIdx.x == 0 && lane == 63) plan.expert_offsets[plan.E] = inc;  // the last lane's inclusive sum: all routed copies
    }
    // the padding between a record's sections travels with the copies: it is written as zero
    for (uint32_t i = threadIdx.x; i < rows_here * row_pieces; i += blockDim.x) recs[i] = make_uint4(0, 0, 0, 0);
    if (INT_META) {
        for (uint32_t t = threadIdx.x; t < (uint32_t)kScaleTables; t += blockDim.x) tabs[t] = kScaleTablesInit.v[t];
    }
    __syncthreads();
    if (!CHUNKS) {
        if (!self) my_rank = my_ranked;
    } else if (my_e >= 0) {
        my_before = plan.hist[(uint64_t)(my_slot / kChunk) * plan.E + my_e];
        my_rank = (int32_t)plan.lrank[my_slot];
    }
    if (has_tile) {
        uint32_t w[16];
        tile_transpose(in, scratch, lane, w);
        const uint32_t l = wave * 64 + lane;
        uint32_t c[8];
        GroupMeta m;
        quantize_lane<BITS, kEplStream, LPG, SR>(w, lane & (LPG - 1), meta_mode, tabs, &scratch[lane * kRowU4], c, m);
        if (l < block_lanes) {
            const uint32_t rl = l / lanes_per_row;
            put_lane<BITS, LPG, SR>(PutLds{reinterpret_cast<uint8_t*>(recs + rl * row_pieces)}, rec, l - rl * lanes_per_row,
                                    lane & (LPG - 1), meta_mode, c, m);
        }
    }
    if (threadIdx.x < n_slots_here) {
        const int32_t r = my_e >= 0 ? start[my_e] + my_before + my_rank : -1;
        drow[threadIdx.x] = r;
        if (r >= 0) plan.row_src[r] = (int32_t)my_slot;
    }
    for (uint32_t i = threadIdx.x + blockDim.x; i < n_slots_here; i += blockDim.x) {  // more routed slots than threads: rare
        const uint32_t slot = row0 * K + i;
        int32_t r;
        if (!CHUNKS) {  // ranked: a block that plans for itself has no more slots than threads
            const int32_t e = plan.ids[slot];
            r = (uint32_t)e < plan.E ? start[e] + plan.rank[slot] : -1;
        } else {
            r = dest_row_of(slot, plan.ids, plan.E, plan.hist, plan.lrank, start);
        }
        drow[i] = r;
        if (r >= 0) plan.row_src[r] = (int32_t)slot;
    }
    __syncthreads();
    // Copies.  One unit = 64 consecutive 16-byte pieces of one copy, cut so that a unit starts on a line of the send
    // buffer (the first unit of a copy starts up to 7 pieces before the record and masks them off).
    const uint32_t n_seg = (row_pieces + 7 + 63) >> 6;
    const uint32_t units = rows_here * K * n_seg;
    for (uint32_t u = wave; u < units; u += n_waves) {
        const uint32_t rk = u / n_seg, j = u - rk * n_seg;
        const int32_t d = drow[rk];
        if (d < 0) continue;
        const uint32_t ro = __umul24((uint32_t)d, row_bytes);  // 32-bit offsets: checked on the host
        const uint32_t a0 = (uint32_t)(reinterpret_cast<uintptr_t>(send) >> 4) + (ro >> 4);  // the copy's first piece, counted in pieces
        const uint32_t shift = a0 & 7u;
        const int32_t p = (int32_t)(j * 64 + lane) - (int32_t)shift;
        if (p >= 0 && (uint32_t)p < row_pieces) {
            const uint4 v = recs[(rk / K) * row_pieces + (uint32_t)p];
            uint8_t* at = send + (ro + 16u * (uint32_t)p);
            // The line a copy starts in and the line it ends in are shared with the neighbouring rows, which other blocks
            // write: those pieces go out as ordinary stores, so that the halves of such a line meet in the cache.
            const uint32_t line = (a0 + (uint32_t)p) >> 3, end = a0 + row_pieces;
            const bool shared = (shift != 0 && line == (a0 >> 3)) || ((end & 7u) != 0 && line == (end >> 3));
            if (shared) *reinterpret_cast<uint4*>(at) = v;
            else store_stream(at, v);
        }
    }
    // Rows that no routed copy takes (dropped slots leave them at the end), one per wave at a time over the whole grid.
    for (uint32_t r = (uint32_t)start[plan.E] + blockIdx.x * n_waves + wave; r < plan.fresh_rows; r += gridDim.x * n_waves) {
        uint4* at = reinterpret_cast<uint4*>(send + __umul24(r, row_bytes));
        for (uint32_t p = lane; p < row_pieces; p += 64) at[p] = make_uint4(0, 0, 0, 0);
        if (lane == 0) plan.row_src[r] = -1;
    }
}

__global__ __launch_bounds__(kBlock) void k_dispatch_clear(uint4* __restrict__ send, uint32_t n16) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n16) store_stream(&send[i], make_uint4(0, 0, 0, 0));
}

// Direct kernel: one wave tile = 2048 consecutive elements of x, every lane stores its share of the K copies itself.
template <int BITS, int LPG, bool SR, bool INT_META>
__global__ __launch_bounds__(kBlock) void k_dispatch_quant_t(const uint4* __restrict__ x, uint32_t n_lanes, uint32_t lanes_per_row,
                                                             uint32_t K, const int32_t* __restrict__ dest, uint8_t* __restrict__ send,
                                                             Rec rec, uint32_t row_bytes, uint32_t meta_mode_arg) {
    const uint32_t meta_mode = INT_META ? kMetaInt : (meta_mode_arg == kMetaFp32 ? kMetaFp32 : kMetaBf16);
    constexpr int EPL = kEplStream;
    __shared__ uint4 lds[kWaves][64 * kRowU4];
    __shared__ float tabs[kScaleTables];
    if (INT_META) fill_scale_tables(tabs);
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t lig = lane & (LPG - 1);
    const uint32_t tile = blockIdx.x * kWaves + wave;
    if (tile * 64 >= n_lanes) return;
    const TileIn cur = tile_load(x, (uint64_t)tile * 256, lane, n_lanes * 4 - tile * 256);
    uint32_t w[16];
    tile_transpose(cur, lds[wave], lane, w);
    const uint32_t L = tile * 64 + lane;
    if (L >= n_lanes) return;
    const uint32_t t = L / lanes_per_row;
    const uint32_t r = L - t * lanes_per_row;  // lane inside the row
    uint32_t c[EPL / 4];
    GroupMeta m;
    quantize_lane<BITS, EPL, LPG, SR>(w, lig, meta_mode, tabs, &lds[wave][lane * kRowU4], c, m);
    for (uint32_t k0 = 0; k0 < K; k0 += 8) {
        int32_t rows[8];  // all destinations first: the loads overlap instead of queueing one behind the other
#pragma unroll
        for (int i = 0; i < 8; ++i) rows[i] = (k0 + i < K) ? dest[t * K + k0 + i] : -1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (rows[i] < 0) continue;
            // the hint pays for metadata only where every lane stores (groups of 32)
            put_lane<BITS, LPG, SR>(PutGlobal<LPG == 1>{send + __umul24((uint32_t)rows[i], row_bytes)}, rec, r, lig, meta_mode, c, m);
        }
    }
}

static_assert(64 * kRowU4 * 16 == kWaveScratchBytes && kRowsBlockMax == kRowsPlanThreadsMax, "the launch plan and the kernel disagree");

template <int BITS, int G, bool SR> struct LaunchDispatch {
    static int run(const void* x, uint32_t T, uint32_t H, uint32_t K, const DispatchPlan& plan, int32_t* dest, uint8_t* send,
                   const Rec& rec, uint32_t row_bytes, uint32_t meta_mode, hipStream_t st) {
        constexpr int EPL = kEplStream, LPG = G / EPL;
        const uint32_t lpr = H / EPL, n_lanes = T * lpr;
        const bool im = meta_mode == kMetaInt;
        const RowsPlan rp = rows_plan(lpr, K, row_bytes, im, plan.E);
        if (rp.rows) {
            const dim3 grid((T + rp.rows - 1) / rp.rows), block(rp.threads);
            auto rows = [&](auto kernel) {
                return launch(kernel, grid, block, rp.lds_bytes, st, (const uint4*)x, T, lpr, K, plan, send, rec, row_bytes, meta_mode, rp.rows);
            };
            if (plan.mode == kPlanChunks)
                return im ? rows(k_dispatch_rows_t<BITS, LPG, SR, true, true>) : rows(k_dispatch_rows_t<BITS, LPG, SR, false, true>);
            return im ? rows(k_dispatch_rows_t<BITS, LPG, SR, true, false>) : rows(k_dispatch_rows_t<BITS, LPG, SR, false, false>);
        }
        // Row shapes the staged kernel cannot take: destination rows written out by one more small launch, then the direct kernel.
        const uint32_t n_slots = T * K;
        if (launch(k_dispatch_dest, dim3((n_slots + kChunk - 1) / kChunk), dim3(kChunk), plan.E * 4, st, plan.ids, n_slots, plan.E, plan.hist,
                   plan.totals, plan.lrank, plan.expert_offsets, dest, plan.row_src, plan.fresh_rows) != FCV2_OK)
            return FCV2_ERR_LAUNCH;
        if (plan.fresh_rows) {  // the direct kernel leaves the padding inside rows alone: clear everything first
            const uint32_t n16 = (uint32_t)((uint64_t)n_slots * row_bytes / 16);
            if (launch(k_dispatch_clear, dim3((n16 + kBlock - 1) / kBlock), dim3(kBlock), 0, st, (uint4*)send, n16) != FCV2_OK) return FCV2_ERR_LAUNCH;
        }
        const dim3 grid(grid_lanes(n_lanes)), block(kBlock);
        if (im)
            return launch(k_dispatch_quant_t<BITS, LPG, SR, true>, grid, block, 0, st, (const uint4*)x, n_lanes, lpr, K, (const int32_t*)dest,
                          send, rec, row_bytes, meta_mode);
        return launch(k_dispatch_quant_t<BITS, LPG, SR, false>, grid, block, 0, st, (const uint4*)x, n_lanes, lpr, K, (const int32_t*)dest, send,
                      rec, row_bytes, meta_mode);
    }
};

// Whether every block of the row-staged kernel plans for itself (plan_block) instead of reading what two launches before it
// prepared.  A block then counts all routed slots, so the work grows with slots x blocks, while the two launches cost 2 to
// 4 us whatever the size.  Measured on the MI355X (4 bits, us per call, planned by launches -> by itself): 64 tokens x 8 on
// 256 experts 11.0 -> 7.4; 1021 x 6 on 64 (2 M) 12.2 -> 10.1; 1024 x 8 on 256 (8 M) 15.2 -> 13.3; 2048 x 2 on 8 (8 M)
// 12.9 -> 11.8; from 16 M the launches win: 2048 x 4 on 64 15.0 -> 15.5, 4096 x 2 of 1024 elements 11.0 -> 13.1.
// The block's own slots are ranked by one wave, the expert counts are four to a lane and the ids are read 16 bytes at a time.
static bool self_planned(const RowsPlan& rp, const int32_t* ids, uint32_t T, uint32_t K, uint32_t E) {
    if (rp.rows == 0 || rp.rows * K > 64u || E > 256u || (reinterpret_cast<uintptr_t>(ids) & 15u) != 0) return false;
    const uint64_t n_slots = (uint64_t)T * K, blocks = (T + rp.rows - 1) / rp.rows;
    return n_slots <= 8192u && n_slots * blocks <= (1u << 23);
}

// Whether one launch ranks all slots (k_dispatch_rank) where two would count and scan chunks.  A block per expert reads every id, so
// the work grows with slots x experts.  Measured on the MI355X (us per call, two launches -> one): 2048 tokens of 4096 elements x 4 on
// 64 experts 15.7 -> 13.9, 2048 x 7168 x 8 on 256 24.0 -> 22.8, 8192 x 1024 x 1 on 16 13.4 -> 12.4; with four times the registers
// for more slots 4096 x 1024 x 8 on 256 17.0 -> 19.8, 8192 x 7168 x 8 80.6 -> 86.7.
static bool ranked_plan(const RowsPlan& rp, const int32_t* ids, uint32_t n_slots, uint32_t E) {
    return rp.rows != 0 && (reinterpret_cast<uintptr_t>(ids) & 15u) == 0 && n_slots >= 4 && n_slots <= 4 * kRankThreads * kRankSteps && E <= 256u;
}

int launch_dispatch(const fcv2_fmt_t* fmt, const void* x, const int32_t* ids, uint32_t T, uint32_t H, uint32_t K, uint32_t E,
                    uint8_t* send, int32_t* expert_offsets, int32_t* row_src, void* ws, const Rec& rec, uint32_t row_bytes,
                    bool fresh, hipStream_t st) {
    const DispatchWs w = dispatch_ws(T, K, E);
    int32_t* hist = (int32_t*)((uint8_t*)ws + w.off_hist);
    int32_t* totals = (int32_t*)((uint8_t*)ws + w.off_totals);
    uint8_t* lrank = (uint8_t*)ws + w.off_lrank;
    int32_t* dest = (int32_t*)((uint8_t*)ws + w.off_dest);
    const RowsPlan rp = rows_plan(H / kEplStream, K, row_bytes, meta_mode_of(fmt) == kMetaInt, E);
    if (self_planned(rp, ids, T, K, E)) {
        const DispatchPlan plan = {ids, nullptr, ids, nullptr, ids, expert_offsets, row_src, kPlanSelf, E, 0u, fresh ? w.n_slots : 0u};
        return by_format<LaunchDispatch>(fmt, x, T, H, K, plan, dest, send, rec, row_bytes, meta_mode_of(fmt), st);
    }
    if (ranked_plan(rp, ids, w.n_slots, E)) {
        if (launch(k_dispatch_rank, dim3(E), dim3(kRankThreads), 0, st, ids, w.n_slots, totals, dest) != FCV2_OK) return FCV2_ERR_LAUNCH;
        const DispatchPlan plan = {ids, nullptr, totals, nullptr, dest, expert_offsets, row_src, kPlanRanked, E, E - 1u, fresh ? w.n_slots : 0u};
        return by_format<LaunchDispatch>(fmt, x, T, H, K, plan, dest, send, rec, row_bytes, meta_mode_of(fmt), st);
    }
    const size_t mask_bytes = (size_t)(kChunk / 64) * E * 8;  // lane masks per wave and expert: 8 KiB at 256 experts
    const int rc = mask_bytes <= 32 * 1024
                       ? launch(k_dispatch_count_rank<true>, dim3(w.n_chunks), dim3(kChunk), mask_bytes, st, ids, w.n_slots, E, hist, lrank)
                       : launch(k_dispatch_count_rank<false>, dim3(w.n_chunks), dim3(kChunk), mask_bytes / 2, st, ids, w.n_slots, E, hist, lrank);
    if (rc != FCV2_OK) return FCV2_ERR_LAUNCH;
    if (launch(k_dispatch_scan_chunks, dim3(E), dim3(64), 0, st, hist, w.n_chunks, E, totals) != FCV2_OK) return FCV2_ERR_LAUNCH;
    const DispatchPlan plan = {ids, hist, totals, lrank, ids, expert_offsets, row_src, kPlanChunks, E, E - 1u, fresh ? w.n_slots : 0u};
    return by_format<LaunchDispatch>(fmt, x, T, H, K, plan, dest, send, rec, row_bytes, meta_mode_of(fmt), st);
}

}  // namespace fcv2

// ---- the dispatch call for callers that cannot allocate ------------------------------------------------------------
// The planning kernels' scratch (per-chunk histograms, expert totals, one destination row per slot) lives in a
// file-scope device array instead of a caller-supplied workspace.  Every GPU the library runs on holds its own copy of
// the array, at its own address, until the process ends.  In host code the array's name is only a stand-in for the
// device symbol: the address that kernels and copies need is asked of the runtime once per device
// (hipGetSymbolAddress, with that device current) and kept; host code below uses that pointer, never the name.
static __device__ __align__(256) uint8_t scratch[FCV2_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];  // zero-initialised; filled on the first call on each device

// Address of `scratch` on the current device, or nullptr (the runtime refused, or a device ordinal beyond kMaxDevices).
void* scratch_of_current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (p) return p;
    // Two threads may both get here on a first call; both are told the same address, so the race is harmless.
    void* q = nullptr;
    if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) return nullptr;
    g_scratch_ptr[dev].store(q, std::memory_order_release);
    return q;
}
}  // namespace

extern "C" int fcv2_dispatch_quant_noalloc(const void* x, const int32_t* ids, uint32_t T, uint32_t H, uint32_t K, uint32_t E,
                                           const fcv2_fmt_t* fmt, void* send, int32_t* expert_offsets, int32_t* row_src, void* stream) {
    size_t need = 0;
    const int rc = fcv2_dispatch_workspace_bytes(T, K, E, &need);
    if (rc != FCV2_OK) return rc;
    if (need > (size_t)FCV2_STATIC_SCRATCH_BYTES) return FCV2_ERR_SCRATCH;  // the routing shape does not fit the static array
    void* ws = scratch_of_current_device();
    if (!ws) return FCV2_ERR_LAUNCH;
    // Nothing in the scratch has to start at zero: the counting kernel writes every histogram entry of every chunk, the
    // scan or the ranking kernel every total, k_dispatch_dest every destination row, before any of them is read.  The ranks
    // (of either kernel) are written for routed slots only; what the row kernel reads in a dropped slot's place it does not use.
    return fcv2::dispatch_checked(x, ids, T, H, K, E, fmt, send, expert_offsets, row_src, ws, FCV2_STATIC_SCRATCH_BYTES, false, stream);
}

