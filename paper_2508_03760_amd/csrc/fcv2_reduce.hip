// fcv2_reduce.hip -- fcv2_reduce_requant: the local step of the two-step AllReduce (Sections 3.1, 3.4), kernels and launch.
#include "fcv2_host.h"

// Elements per lane, waves per SIMD, peers in flight and the way spikes are restored, with what was measured on the
// MI355X (16 M-element payload, 8 peers, inputs not in the last-level cache, us per launch, runs on one machine):
//   at 2 / 3 / 4 / 5 / 6 / 7 / 8 bits, 16 elements per lane: overlay at 2 and 3 bits and park above (the choice below)
//   26.2 / 28.3 / 27.7 / 32.2 / 32.5 / 38.3 / 34.1; park everywhere 26.6 / 28.2 / 27.7 / 32.3 / 32.4 / 38.2 / 34.1;
//   (5 to 7 bits before their codes were joined in place; since then, groups of 128, on another machine 25.4 / 28.2 / 27.2 /
//   31.1 / 32.1 / 35.8 / 33.1, overlay everywhere 24.9 / 28.1 / 27.4 / 32.2 / 33.0 / 37.2 / 34.0);
//   32 elements per lane (112 registers, four waves per SIMD; five spill): within 1 us of 16 at every width, not better;
//   one peer in flight at eight waves 29.7 at 3 bits, two at seven waves 28.5, the next two peers requested under the
//   decoding of the current two 29.6 (against 28.8 in that run).
// The peer loop costs the same per element either way (the FMA, the add and the unpacking are per element); what 32
// elements per lane save in per-lane work they lose in occupancy.
#ifndef FCV2_REDUCE_EPL
#define FCV2_REDUCE_EPL(G) 16
#endif
#ifndef FCV2_REDUCE_WAVES32
#define FCV2_REDUCE_WAVES32 4
#endif
#ifndef FCV2_REDUCE_WAVES16
#define FCV2_REDUCE_WAVES16 6
#endif
#ifndef FCV2_REDUCE_CH
#define FCV2_REDUCE_CH 2
#endif
#ifndef FCV2_REDUCE_PATCH
#define FCV2_REDUCE_PATCH(BITS) ((BITS) <= 3 ? kPatchOverlay : kPatchPark)
#endif

namespace fcv2 {

// Local reduce step.  EPL = 16 elements per lane (groups of 32 are two lanes, larger ones four to sixteen).
//  - codes are unpacked into 16-bit halves and fed to v_fma_mix_f32 as fp16 denormals (q * 2^-24) against the
//    scale pre-multiplied by 2^24: the product is the same real number q * scale, the FMA rounds once, so the
//    result is bit-identical to fma(float(q), scale, lo) without a conversion instruction per element;
//  - the spikes of every peer are put back through a private row in LDS: a dynamic register index done by memory.
// Spike restoration (Section 3.3: after dequantization the two spikes of a group go back to their places).  A spike
// position is a dynamic index into the lane's registers, which only memory can do; each lane has a private row of 16
// dwords in LDS for it, and a lane's EPL elements are handled 16 at a time.  Two ways, chosen per bit width:
//   park:    a lane that owns a spike in these 16 elements writes its 16 decoded values to the row, overwrites the
//            spike slot and reads the row back.  No extra arithmetic, 8 sixteen-byte LDS operations.
//   overlay: the row is all zero between uses.  The wire format stores code 0 at a spike position, so what the decoder
//            puts there is t = fma(0, scale, zero), the same for the whole group and known without looking: the owner
//            writes (spike bits XOR t bits) into the slot, every lane reads its row back and XORs it onto its decoded
//            values on their way into the accumulators (t ^ spike ^ t = spike, everything else ^ 0 stays), the owner
//            puts the zero back.  Half the LDS traffic, one cheap XOR per element.  Records whose code at a spike
//            position is not 0 are malformed; with the overlay their spikes come back wrong.
// LDS is shared by the four SIMDs of a compute unit and the park's traffic alone fills most of it at the low widths,
// while the overlay's XORs land on the VALUs, which are the other thing this kernel runs out of.
constexpr int kPatchPark = 0, kPatchOverlay = 1;

// Which register of Q[8], and which half of it, holds element e of 16; by how much its code is shifted inside the half.
struct UnitPairMap {  // codes_pairs_b8 on two units of 8: unit u = Q[4u..4u+3], element k and k + 4, at bit 0
    static constexpr int k_of(int e) { return 4 * (e >> 3) + (e & 3); }
    static constexpr bool in_hi(int e) { return ((e >> 2) & 1) != 0; }
    static constexpr int pos(int) { return 0; }
};

template <int BITS> struct PairCodes {
    static constexpr bool kInPlace = BITS <= 7;  // the fields are only masked, never moved to bit 0 (codes_pairs16)
    using Map = typename std::conditional<kInPlace, PairMap<(kInPlace ? BITS : 2)>, UnitPairMap>::type;
};

// The codes of half h (16 elements) of a lane's planes as pair registers.
template <int BITS, int EPL> __device__ __forceinline__ void pair_codes(const RawPlanes<EPL>& r, int h, uint32_t (&Q)[8]) {
    using P = Planes<BITS>;
    if constexpr (PairCodes<BITS>::kInPlace) {
        const uint32_t p1 = P::w1 ? (EPL == 16 ? r.p1 : (h == 0 ? and_lit<0xFFFFu>(r.p1) : r.p1 >> 16)) : 0u;
        codes_pairs16<BITS>(P::w4 ? r.p4[(2 * h) % (EPL / 8)] : 0u, P::w4 ? r.p4[(2 * h + 1) % (EPL / 8)] : 0u,
                            P::w2 ? r.p2[h % ((EPL + 15) / 16)] : 0u, p1, Q);
    } else {
#pragma unroll
        for (int uu = 0; uu < 2; ++uu) {
            uint32_t Q4[4];
            codes_pairs_b8(r.p8[2 * (2 * h + uu)], r.p8[2 * (2 * h + uu) + 1], Q4);
#pragma unroll
            for (int k = 0; k < 4; ++k) Q[4 * uu + k] = Q4[k];
        }
    }
}

// (Measured and not used: taking the spread of the 3-bit format's extra bits from two 256-entry LDS tables instead of
// computing it -- 12 VALU cycles instead of 35 per peer and 16 elements -- made the kernel 7 % slower: two more LDS
// reads at scattered addresses per peer, in front of everything else the peer needs.)
template <int BITS, int EPL, bool SR, int PATCH>
__device__ __forceinline__ void add_peer_values(const RawPlanes<EPL>& r, const GroupMeta& m, uint32_t lig, uint4* row, float (&acc)[EPL]) {
    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
    using M = typename PairCodes<BITS>::Map;
    const float s = m.s, lo = m.lo;
    uint32_t relmin = 0xFFFFFFFFu, relmax = 0xFFFFFFFFu, t = 0u;
    if (SR) {
        relmin = (m.si & 0xFFu) - lig * (uint32_t)EPL;  // position inside this lane, or >= EPL when another lane owns the spike
        relmax = (m.si >> 8) - lig * (uint32_t)EPL;
        if (PATCH == kPatchOverlay) t = f2u(__fmaf_rn(0.0f, s, lo));  // what a zero code decodes to (-0 offsets, infinite scales included)
    }
    const uint32_t smin = m.sv << 16, smax = m.sv & 0xFFFF0000u;
    u32a* o = reinterpret_cast<u32a*>(row);
    float mult[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) mult[q] = s * __builtin_ldexpf(1.0f, 24 - q);  // only the positions in use survive
    // Decoding exists twice: for scales below 2^100 (always, unless the data spans more than that: 2^24 * scale could
    // overflow) codes go into the mixed-precision FMA as fp16 denormals; otherwise they are converted one by one.
    // codes16 prepares the 16 codes of half h in the form its kind of decoding takes, value decodes element e of them.
    struct Codes16 {
        uint32_t Q[8];
        float qf[16];
    };
    auto codes16 = [&](auto fast_tag, int h, Codes16& c) {
        if constexpr (decltype(fast_tag)::value) {
            pair_codes<BITS, EPL>(r, h, c.Q);
        } else {
#pragma unroll
            for (int uu = 0; uu < 2; ++uu) {
                float q8[8];
                unit_codes<BITS, EPL>(r, 2 * h + uu, q8);
#pragma unroll
                for (int j = 0; j < 8; ++j) c.qf[8 * uu + j] = q8[j];
            }
        }
    };
    auto value = [&](auto fast_tag, const Codes16& c, int e) -> float {
        if constexpr (!decltype(fast_tag)::value) {
            return __fmaf_rn(c.qf[e], s, lo);
        } else {
            const half2v hh = __builtin_bit_cast(half2v, c.Q[M::k_of(e)]);
            return __builtin_fmaf(M::in_hi(e) ? (float)hh.y : (float)hh.x, mult[M::pos(M::k_of(e))], lo);
        }
    };
    if constexpr (SR && PATCH == kPatchOverlay) {
        // everything of a peer inside one branch on the scale: the decoded values go straight into the accumulators, a
        // quarter at a time, so that they are never all live at once
        auto body = [&](auto fast_tag) {
#pragma unroll
            for (int h = 0; h < EPL / 16; ++h) {
                const uint32_t rmin = relmin - 16u * h, rmax = relmax - 16u * h;  // the same inside these 16 elements
                if (rmin < 16u) o[rmin] = smin ^ t;
                if (rmax < 16u) o[rmax] = smax ^ t;
                Codes16 c;
                codes16(fast_tag, h, c);
#pragma unroll
                for (int i = 0; i < 4; ++i) {  // a wave's LDS operations execute in issue order: these reads see the writes above
                    const uint4 x4 = row[i];
                    const uint32_t x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const int e = 4 * i + b;
                        acc[16 * h + e] = __fadd_rn(acc[16 * h + e], u2f(f2u(value(fast_tag, c, e)) ^ x[b]));
                    }
                }
                if (rmin < 16u) o[rmin] = 0u;  // ... and these zeros land after them
                if (rmax < 16u) o[rmax] = 0u;
            }
        };
        if (s < 0x1p+100f)
            body(std::true_type{});
        else
            body(std::false_type{});
    } else {
        // only the decoding sits inside the branch on the scale; parking and accumulating follow it once
#pragma unroll
        for (int h = 0; h < EPL / 16; ++h) {
            float v[16];
            if (s < 0x1p+100f) {
                Codes16 c;
                codes16(std::true_type{}, h, c);
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e] = value(std::true_type{}, c, e);
            } else {
                Codes16 c;
                codes16(std::false_type{}, h, c);
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e] = value(std::false_type{}, c, e);
            }
            if (SR) {
                const uint32_t rmin = relmin - 16u * h, rmax = relmax - 16u * h;
                if (rmin < 16u || rmax < 16u) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) row[i] = make_uint4(f2u(v[4 * i]), f2u(v[4 * i + 1]), f2u(v[4 * i + 2]), f2u(v[4 * i + 3]));
                    if (rmin < 16u) o[rmin] = smin;
                    if (rmax < 16u) o[rmax] = smax;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint4 a = row[i];
                        v[4 * i] = u2f(a.x);
                        v[4 * i + 1] = u2f(a.y);
                        v[4 * i + 2] = u2f(a.z);
                        v[4 * i + 3] = u2f(a.w);
                    }
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[16 * h + e] = __fadd_rn(acc[16 * h + e], v[e]);
        }
    }
}

// The sums of a wave's lanes, 64 bytes each, through the lanes' LDS rows into stores that cover whole lines: written from the lanes
// directly, a store instruction would touch a quarter of each of 32 lines.
// Measured on the MI355X (buffers not in the last-level cache, us per call, direct -> through LDS, with the non-temporal hint):
// 3.2 M elements of 5 peers at 8 bits 10.4 -> 6.7, 16 M of 8 at 3 bits 43.3 -> 35.3, 16 M of 4 at 8 bits 41.0 -> 31.5.
template <int EPL, int ROW> __device__ __forceinline__ void store_sums(float* sum_out, uint4* lds, uint32_t L, uint32_t n_lanes, const float (&acc)[EPL]) {
    const uint32_t lane = threadIdx.x & 63, first = threadIdx.x - lane, L0 = L - lane;
    const uint32_t here = min(64u, n_lanes - L0);  // lanes of the wave that have elements: the first ones
    uint8_t* dst = reinterpret_cast<uint8_t*>(sum_out) + (uint64_t)L0 * (EPL * 4);
#pragma unroll
    for (int h = 0; h < EPL / 16; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            lds[threadIdx.x * ROW + i] = make_uint4(f2u(acc[16 * h + 4 * i]), f2u(acc[16 * h + 4 * i + 1]), f2u(acc[16 * h + 4 * i + 2]),
                                                    f2u(acc[16 * h + 4 * i + 3]));
        wave_lds_sync();
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t piece = k * here + lane, r = piece >> 2, q = piece & 3u;
            store_stream(dst + (r * (EPL * 4) + 64 * h + 16 * q), lds[(first + r) * ROW + q]);
        }
        wave_lds_sync();
    }
}

template <int BITS, int EPL, int LPG, bool SR, int PATCH>
// Peers are taken two at a time (both peers' loads issued before either is decoded).  Every peer in flight costs
// about 15 registers; with two the kernel needs 65 to 74 and six or seven waves fit a SIMD, which measured faster
// than four peers in flight at four or five waves, and faster than one peer at eight.
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(EPL == 32 ? FCV2_REDUCE_WAVES32 : FCV2_REDUCE_WAVES16)))
void k_reduce_requant(PeerPtrs peers, int n_peers, uint32_t n_lanes, Rec rec_in,
                                                           uint8_t* __restrict__ out, Rec rec_out, float* __restrict__ sum_out,
                                                           uint32_t meta_mode_in, uint32_t meta_mode_out_arg) {
    const uint32_t meta_mode_out = meta_mode_out_arg & 3u;
    constexpr int CH = FCV2_REDUCE_CH;  // peers in flight
    constexpr int ROW = 16 / 4 + 1;  // uint4 per private row of 16 dwords, one of padding: conflict-free 16-byte accesses
    __shared__ uint4 lds[kBlock * ROW];  // 20 KiB: eight blocks fill the 160 KiB of a compute unit exactly
    extern __shared__ float tabs[];      // the scale tables of the integer metadata: dynamic, present only when a format uses them
    if (meta_mode_in == kMetaInt || meta_mode_out == kMetaInt) fill_scale_tables(tabs);
    const uint32_t L = xcd_tile_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if ((meta_mode_out_arg & kZeroPadding) && L < 64) zero_padding<BITS, SR>(out, rec_out, n_lanes * EPL, n_lanes / LPG, meta_mode_out, L);
    if (L >= n_lanes) return;
    const uint32_t lig = threadIdx.x & (LPG - 1);
    uint4* row = &lds[threadIdx.x * ROW];
    if (SR && PATCH == kPatchOverlay) {  // the lane's overlay row starts, and is left after every use, all zero
#pragma unroll
        for (int i = 0; i < 4; ++i) row[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    const MetaOffsets mo = meta_offsets<LPG, SR>(rec_in, L, meta_mode_in);
    // -0 is the identity of fp32 addition for every value including -0, so the chain below starts exactly at v_0
    float acc[EPL];
#pragma unroll
    for (int j = 0; j < EPL; ++j) acc[j] = -0.0f;
    // The peer loop exists twice, once per kind of metadata decoding, chosen by one uniform branch outside it.
    auto sum_peers = [&](auto int_meta) {
        constexpr bool INT_META = decltype(int_meta)::value;
        auto add_peer = [&](const RawPlanes<EPL>& r, uint32_t mraw, uint32_t mraw2) {
            const GroupMeta m = spread_meta<LPG, SR, INT_META>(mraw, mraw2, mo, tabs, rec_in.idx_bf16);
            add_peer_values<BITS, EPL, SR, PATCH>(r, m, lig, row, acc);
        };
        int p = 0;
        // CH peers at a time: all loads first, so their latencies overlap
        for (; p + CH <= n_peers; p += CH) {
            RawPlanes<EPL> r[CH];
            uint32_t mraw[CH], mraw2[CH];
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const BufferSrc src = buffer_src(peers.base[p + i], rec_in.total);
                r[i] = load_planes<BITS, EPL>(src, rec_in, L);
                mraw[i] = ld32(src, mo.at);
                mraw2[i] = (LPG < 4 && SR) ? ld32(src, mo.at2) : 0u;
            }
#pragma unroll
            for (int i = 0; i < CH; ++i) add_peer(r[i], mraw[i], mraw2[i]);
        }
        for (; p < n_peers; ++p) {
            const BufferSrc src = buffer_src(peers.base[p], rec_in.total);
            const RawPlanes<EPL> r = load_planes<BITS, EPL>(src, rec_in, L);
            const uint32_t mraw = ld32(src, mo.at);
            const uint32_t mraw2 = (LPG < 4 && SR) ? ld32(src, mo.at2) : 0u;
            add_peer(r, mraw, mraw2);
        }
    };
    if (meta_mode_in == kMetaInt)
        sum_peers(std::true_type{});
    else
        sum_peers(std::false_type{});
    if (sum_out) store_sums<EPL, ROW>(sum_out, lds, L, n_lanes, acc);
    uint32_t w[EPL / 2];
#pragma unroll
    for (int d = 0; d < EPL / 2; ++d) w[d] = pack_bf16(acc[2 * d], acc[2 * d + 1]);
    uint32_t c[EPL / 4];
    GroupMeta m;
    quantize_lane<BITS, EPL, LPG, SR>(w, lig, meta_mode_out, tabs, row, c, m);
    store_planes<BITS, EPL>(out, rec_out, L, c);
    if (lig == 0) store_meta<SR>(out, rec_out, L / LPG, m, meta_mode_out);
}

// Small payloads, 2 to 8 peers.  With 16 elements and all peers per lane a payload of half a million elements is less than one
// wave per SIMD, on half of the compute units, and what the call takes is one wave's chain through its peers: 0.3 us for each
// (unpacking, the overlay's trip through LDS, the wait for the next loads).  Here the peers of a tile of 1024 elements go to different waves of a block: wave w decodes peer w into LDS (the spikes simply
// overwrite their slots there), then two waves add the values up in peer order, 8 elements a lane, and quantize.
// Values of 4 consecutive elements are one 16-byte piece; a lane's four pieces are turned by its number, so that the writes of
// eight neighbouring lanes (64 bytes apart) fall into different bank groups.
constexpr uint32_t kSmallTile = 1024, kSmallPeers = 8;
__device__ __forceinline__ uint32_t small_piece(uint32_t lane, uint32_t q) { return lane * 4 + ((q + (lane >> 1)) & 3u); }

template <int BITS, int G, bool SR, bool INT_META>
__global__ __launch_bounds__(64 * kSmallPeers) void k_reduce_small(PeerPtrs peers, int n_peers, uint32_t n, Rec rec_in, uint8_t* __restrict__ out,
                                                                   Rec rec_out, float* __restrict__ sum_out, uint32_t meta_mode_in,
                                                                   uint32_t meta_mode_out_arg) {
    const uint32_t meta_mode_out = meta_mode_out_arg & 3u;
    extern __shared__ uint4 vals[];                     // [n_peers][kSmallTile / 4]
    __shared__ float tabs[INT_META ? kScaleTables : 1];
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t tile0 = blockIdx.x * kSmallTile;
    if (INT_META) {
        for (uint32_t t = threadIdx.x; t < (uint32_t)kScaleTables; t += blockDim.x) tabs[t] = kScaleTablesInit.v[t];
        __syncthreads();
    }
    const uint32_t L = tile0 / 16 + lane;
    if (L < n / 16) {
        constexpr int EPL = 16, LPG = G / EPL;
        using Codes = PairCodes<BITS>;
        using M = typename Codes::Map;
        typedef _Float16 half2v __attribute__((ext_vector_type(2)));
        const BufferSrc src = buffer_src(peers.base[wave], rec_in.total);
        const MetaOffsets mo = meta_offsets<LPG, SR>(rec_in, L, meta_mode_in);
        const RawPlanes<EPL> r = load_planes<BITS, EPL>(src, rec_in, L);
        const uint32_t mraw = ld32(src, mo.at), mraw2 = (LPG < 4 && SR) ? ld32(src, mo.at2) : 0u;
        const GroupMeta m = (INT_META && meta_mode_in == kMetaInt) ? spread_meta<LPG, SR, true>(mraw, mraw2, mo, tabs, rec_in.idx_bf16)
                                                                   : spread_meta<LPG, SR, false>(mraw, mraw2, mo, tabs, rec_in.idx_bf16);
        float v[16];
        if (m.s < 0x1p+100f) {  // codes as fp16 denormals, as in add_peer_values
            uint32_t Q[8];
            pair_codes<BITS, EPL>(r, 0, Q);
            float mult[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) mult[q] = m.s * __builtin_ldexpf(1.0f, 24 - q);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const half2v hh = __builtin_bit_cast(half2v, Q[M::k_of(e)]);
                v[e] = __builtin_fmaf(M::in_hi(e) ? (float)hh.y : (float)hh.x, mult[M::pos(M::k_of(e))], m.lo);
            }
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float q8[8];
                unit_codes<BITS, EPL>(r, u, q8);
#pragma unroll
                for (int j = 0; j < 8; ++j) v[8 * u + j] = __fmaf_rn(q8[j], m.s, m.lo);
            }
        }
        uint4* mine = vals + wave * (kSmallTile / 4);
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
            mine[small_piece(lane, q)] = make_uint4(f2u(v[4 * q]), f2u(v[4 * q + 1]), f2u(v[4 * q + 2]), f2u(v[4 * q + 3]));
        if (SR) {
            const uint32_t lig = lane & (LPG - 1);
            const uint32_t rmin = (m.si & 0xFFu) - lig * 16u, rmax = (m.si >> 8) - lig * 16u;  // >= 16: another lane's
            u32a* o = reinterpret_cast<u32a*>(mine);
            wave_lds_sync();
            if (rmin < 16u) o[small_piece(lane, rmin >> 2) * 4 + (rmin & 3u)] = m.sv << 16;
            wave_lds_sync();  // both spikes in one slot (a malformed record): the maximum stays, as in the general kernel
            if (rmax < 16u) o[small_piece(lane, rmax >> 2) * 4 + (rmax & 3u)] = m.sv & 0xFFFF0000u;
        }
    }
    if ((meta_mode_out_arg & kZeroPadding) && blockIdx.x == 0 && wave == (blockDim.x >> 6) - 1u)
        zero_padding<BITS, SR>(out, rec_out, n, n / G, meta_mode_out, lane);
    __syncthreads();
    constexpr int EPL = 8, LPG = G / EPL;
    const uint32_t L8 = tile0 / EPL + threadIdx.x;
    if (threadIdx.x >= kSmallTile / EPL || L8 >= n / EPL) return;
    float acc[EPL];
#pragma unroll
    for (int j = 0; j < EPL; ++j) acc[j] = -0.0f;
    const uint32_t row = threadIdx.x >> 1, q0 = 2 * (threadIdx.x & 1);
    const uint32_t at0 = small_piece(row, q0), at1 = small_piece(row, q0 + 1);
    auto add = [&](const uint4& a, const uint4& b) {
        const uint32_t x[EPL] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int j = 0; j < EPL; ++j) acc[j] = __fadd_rn(acc[j], u2f(x[j]));
    };
    uint4 a[kSmallPeers], b[kSmallPeers];  // all peers' values first (peers beyond the last repeat it and are not added)
#pragma unroll
    for (int p = 0; p < (int)kSmallPeers; ++p) {
        const uint4* from = vals + min(p, n_peers - 1) * (int)(kSmallTile / 4);
        a[p] = from[at0];
        b[p] = from[at1];
    }
#pragma unroll
    for (int p = 0; p < (int)kSmallPeers; ++p)
        if (p < n_peers) add(a[p], b[p]);
    if (sum_out) {
        float4* dst = reinterpret_cast<float4*>(sum_out) + (EPL / 4) * (uint64_t)L8;
        dst[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        dst[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    }
    uint32_t w[EPL / 2];
#pragma unroll
    for (int d = 0; d < EPL / 2; ++d) w[d] = pack_bf16(acc[2 * d], acc[2 * d + 1]);
    uint32_t c[EPL / 4];
    GroupMeta m;
    const uint32_t lig = threadIdx.x & (LPG - 1);
    // the lane's scratch: the pieces of its own elements of peer 0, which nothing else reads
    quantize_lane<BITS, EPL, LPG, SR>(w, lig, meta_mode_out, tabs, vals + at0, c, m);
    store_planes<BITS, EPL>(out, rec_out, L8, c);
    if (lig == 0) store_meta<SR>(out, rec_out, L8 / LPG, m, meta_mode_out);
}

// The same step when the peers' bit width differs from the output's: the input width is a run-time value
// (one uniform switch around the peer loop), the output width stays a template parameter.  A compatibility path next to
// the specialised kernel above: spikes always through the park, no choice of occupancy per width.
template <int BITS_OUT, int EPL, int LPG, bool SR>
__global__ __launch_bounds__(kBlock) void k_reduce_requant_mixed(PeerPtrs peers, int n_peers, uint32_t bits_in, uint32_t n_lanes,
                                                                 Rec rec_in, uint8_t* __restrict__ out, Rec rec_out,
                                                                 float* __restrict__ sum_out, uint32_t meta_mode_in,
                                                                 uint32_t meta_mode_out_arg) {
    const uint32_t meta_mode_out = meta_mode_out_arg & 3u;
    constexpr int ROW = 16 / 4 + 1;
    __shared__ uint4 lds[kBlock * ROW];
    __shared__ float tabs[kScaleTables];
    if (meta_mode_in == kMetaInt || meta_mode_out == kMetaInt) fill_scale_tables(tabs);
    const uint32_t L = xcd_tile_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if ((meta_mode_out_arg & kZeroPadding) && L < 64)
        zero_padding<BITS_OUT, SR>(out, rec_out, n_lanes * EPL, n_lanes / LPG, meta_mode_out, L);
    if (L >= n_lanes) return;
    const uint32_t lig = threadIdx.x & (LPG - 1);
    uint4* row = &lds[threadIdx.x * ROW];
    const MetaOffsets mo = meta_offsets<LPG, SR>(rec_in, L, meta_mode_in);
    float acc[EPL];
#pragma unroll
    for (int j = 0; j < EPL; ++j) acc[j] = -0.0f;
    // One uniform switch on the input width around the whole peer loop; inside it peers are taken two at a time, both
    // peers' loads issued before either is decoded (an odd last peer is requested twice and added once).
    auto sum_peers = [&](auto bits_tag) {
        constexpr int B = decltype(bits_tag)::value;
        auto add_peer = [&](const RawPlanes<EPL>& r, uint32_t mraw, uint32_t mraw2) {
            const GroupMeta m = (meta_mode_in == kMetaInt) ? spread_meta<LPG, SR, true>(mraw, mraw2, mo, tabs, rec_in.idx_bf16)
                                                           : spread_meta<LPG, SR, false>(mraw, mraw2, mo, tabs, rec_in.idx_bf16);
            add_peer_values<B, EPL, SR, kPatchPark>(r, m, lig, row, acc);
        };
        for (int p = 0; p < n_peers; p += 2) {
            const bool two = p + 1 < n_peers;
            RawPlanes<EPL> r[2];
            uint32_t mraw[2], mraw2[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const BufferSrc src = buffer_src(peers.base[(i == 1 && two) ? p + 1 : p], rec_in.total);
                r[i] = load_planes<B, EPL>(src, rec_in, L);
                mraw[i] = ld32(src, mo.at);
                mraw2[i] = (LPG < 4 && SR) ? ld32(src, mo.at2) : 0u;
            }
            add_peer(r[0], mraw[0], mraw2[0]);
            if (two) add_peer(r[1], mraw[1], mraw2[1]);
        }
    };
    switch (bits_in) {
        case 2: sum_peers(std::integral_constant<int, 2>{}); break;
        case 3: sum_peers(std::integral_constant<int, 3>{}); break;
        case 4: sum_peers(std::integral_constant<int, 4>{}); break;
        case 5: sum_peers(std::integral_constant<int, 5>{}); break;
        case 6: sum_peers(std::integral_constant<int, 6>{}); break;
        case 7: sum_peers(std::integral_constant<int, 7>{}); break;
        default: sum_peers(std::integral_constant<int, 8>{}); break;
    }
    if (sum_out) store_sums<EPL, ROW>(sum_out, lds, L, n_lanes, acc);
    uint32_t w[EPL / 2];
#pragma unroll
    for (int d = 0; d < EPL / 2; ++d) w[d] = pack_bf16(acc[2 * d], acc[2 * d + 1]);
    uint32_t c[EPL / 4];
    GroupMeta m;
    quantize_lane<BITS_OUT, EPL, LPG, SR>(w, lig, meta_mode_out, tabs, row, c, m);
    store_planes<BITS_OUT, EPL>(out, rec_out, L, c);
    if (lig == 0) store_meta<SR>(out, rec_out, L / LPG, m, meta_mode_out);
}

template <int BITS, int G, bool SR> struct LaunchReduce {
    static int run(const PeerPtrs& peers, int n_peers, uint64_t n, const Rec& rec_in, void* out, const Rec& rec_out,
                   float* sum_out, uint32_t mf_in, uint32_t mf_out, hipStream_t st) {
        const bool im = mf_in == kMetaInt || (mf_out & 3u) == kMetaInt;
        // Below a million elements the general kernel is less than one wave per SIMD and its time the chain of a wave through
        // its peers; above it, values passing through LDS cost more than they save.  Measured on the MI355X, us per call,
        // general -> small kernel: 3 bits of 64 x 7168 with 8 / 5 / 3 peers 6.2 -> 4.0, 5.2 -> 3.8, 4.4 -> 3.7; of 128 x 7168
        // 6.2 -> 5.6, 5.2 -> 4.3, 4.4 -> 3.9; of 192 x 7168 6.9 -> 7.2, 5.7 -> 5.7, 4.7 -> 4.6.  Without spikes the chain is
        // short: 8 bits of 64 x 7168 with 5 peers 3.6 -> 3.3, of 146 x 7168 3.7 -> 3.8.  One peer is no chain (3.3 -> 3.4).
        if (n <= (SR ? 1u << 20 : 1u << 19) && n_peers >= 2 && n_peers <= (int)kSmallPeers) {
            const dim3 grid((unsigned)((n + kSmallTile - 1) / kSmallTile)), block(64 * (unsigned)n_peers);
            const size_t lds = (size_t)n_peers * kSmallTile * 4;
            if (im)
                return launch(k_reduce_small<BITS, G, SR, true>, grid, block, lds, st, peers, n_peers, (uint32_t)n, rec_in, (uint8_t*)out,
                              rec_out, sum_out, mf_in, mf_out);
            return launch(k_reduce_small<BITS, G, SR, false>, grid, block, lds, st, peers, n_peers, (uint32_t)n, rec_in, (uint8_t*)out, rec_out,
                          sum_out, mf_in, mf_out);
        }
        constexpr int EPL = FCV2_REDUCE_EPL(G);
        constexpr int PATCH = FCV2_REDUCE_PATCH(BITS);
        const uint32_t n_lanes = (uint32_t)(n / EPL);
        const size_t tab_bytes = im ? sizeof(float) * kScaleTables : 0;
        return launch(k_reduce_requant<BITS, EPL, G / EPL, SR, PATCH>, dim3(grid_lanes_xcd(n_lanes)), dim3(kBlock), tab_bytes, st, peers,
                      n_peers, n_lanes, rec_in, (uint8_t*)out, rec_out, sum_out, mf_in, mf_out);
    }
};
template <int BITS, int G, bool SR> struct LaunchReduceMixed {  // BITS = output width
    static int run(const PeerPtrs& peers, int n_peers, uint32_t bits_in, uint64_t n, const Rec& rec_in, void* out,
                   const Rec& rec_out, float* sum_out, uint32_t mf_in, uint32_t mf_out, hipStream_t st) {
        constexpr int EPL = 16;
        const uint32_t n_lanes = (uint32_t)(n / EPL);
        return launch(k_reduce_requant_mixed<BITS, EPL, G / EPL, SR>, dim3(grid_lanes_xcd(n_lanes)), dim3(kBlock), 0, st, peers,
                      n_peers, bits_in, n_lanes, rec_in, (uint8_t*)out, rec_out, sum_out, mf_in, mf_out);
    }
};
int launch_reduce(const fcv2_fmt_t* fmt_in, const fcv2_fmt_t* fmt_out, const PeerPtrs& peers, int n_peers, uint64_t n,
                  const Rec& rec_in, void* out, const Rec& rec_out, float* sum_out, bool zero_pad, hipStream_t st) {
    const uint32_t mf_in = meta_mode_of(fmt_in), mf_out = meta_mode_of(fmt_out) | (zero_pad ? kZeroPadding : 0u);
    if (fmt_in->bits != fmt_out->bits)
        return by_format<LaunchReduceMixed>(fmt_out, peers, n_peers, fmt_in->bits, n, rec_in, out, rec_out, sum_out, mf_in, mf_out, st);
    return by_format<LaunchReduce>(fmt_in, peers, n_peers, n, rec_in, out, rec_out, sum_out, mf_in, mf_out, st);
}

}  // namespace fcv2
