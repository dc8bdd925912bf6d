// One-pass kernel for gfx950: a whole AllReduce plan as one launch that reads
// each buffer position once and writes it once, with every intermediate value
// in registers.
#pragma once

#include "kernels.hpp"
#include "resident.hpp"

namespace arp {

// ------------------------------------------------------------------------
// Every step is element-wise, so what a plan leaves at an element position is
// an expression over the n values the buffers hold there: folds of folds of
// buffer rows (leaves).  Where every buffer ends with the same value, as an
// AllReduce leaves them, the host (onepass.cpp) lists, per segment of
// positions with one expression, its leaves in the order they are computed
// in, a word each:
//   bits 15:0   the buffer;
//   kOnePush    the leaf starts a fold that is a later operand of another one:
//               the running sum is put aside (in LDS) and a new one starts;
//   kOneRound   after the leaf and its pops a step ends whose value is the
//               first operand of the next fold: the running sum is rounded to
//               the element type (bf16 only);
//   bits 31:24  pops: so many times the running sum is rounded (its step
//               ends) and added to the one last put aside.
// Every fold adds the same values in the same order as the plan's step and is
// rounded where the step ends, so the bits are the plan's (a step of two
// sources may have them swapped, which shows in nothing but which payload two
// NaNs leave; the compiler's operand order decides that in every launch form:
// of 3726 positions with NaNs co-located PS n = 6 over 4099 fp32 gives another
// than the first operand's in 2260 by its phase launches, in 2589 one-pass).  A sum
// starts from -0.0 (0 for int32), which adding a value to leaves its bits.
//
// A wavefront owns 64 lanes x U vectors of LB bytes at one place of a
// segment: it loads them of every leaf, B leaves at a time with all their
// loads in flight at once, folds, and stores the result to all n buffers.
// Nothing is kept in LDS but the sums put aside, so occupancy does not fall
// with n as it does where each buffer's tile has an LDS row.
//
// Segments may start and end at any element, and buffers may lie at any
// address that their element type may: vectors are loaded and stored with
// element alignment.  They lie on LB-byte boundaries where the buffers do
// (amask = VEC - 1) and are otherwise counted from the segment's start
// (amask = 0).  A vector that reaches over an end of the segment is loaded
// whole, from N - VEC where it would reach over the buffers' end (the host
// sees to N >= VEC), and only the segment's elements of it are stored: the
// others belong to another wavefront, and what is read of them is not used.
//
// The instances (one_config in onepass.cpp chooses; us per AllReduce on
// MI355X over three buffer sets in turn):
//  * LB 4, U 1, four waves a workgroup: few positions, so that they make
//    four times the wavefronts (Ring n = 64 over 65541 fp32 10.9 us, with
//    LB 16 18.1);
//  * LB 16, U 1, one wave a workgroup (tree (8, 8) over 1048581 fp32 97 us;
//    four waves 104, eight 115, sixteen 133: waves of a workgroup run in
//    step and end together), with as many leaves in a batch as n gives it
//    registers for no more (n = 3 over 2000003 fp32: B 4 9.0 us, B 16 11.3;
//    RHD n = 8 over 2^26: B 8 716, B 4 743);
//  * LB 16, U 4, 8 or 16 where that still makes 448 to 2048 wavefronts
//    (kOneWide): the whole launch is then resident at once, so that the chip
//    first reads and then writes, and each buffer is touched in 4, 8 or 16 KiB
//    pieces (Ring
//    n = 64 over 2^20 fp32: U 1 97 us, U 4 91; tree (8, 8) over 2^22: U 1
//    386, U 16 357; bf16, whose sums take twice the registers, U 1 192, U 8
//    187, U 16 209).  Larger ones run in many rounds anyhow and stream best
//    with U 1 (RHD n = 8 over 2^26: U 1 716, U 4 782, U 16 846), tile after
//    tile instead of an eighth of the vector on each XCD (eight times as many
//    streams), and with fewer wavefronts a compute unit than fit (one_lds).
constexpr uint32_t kOnePush = 1u << 16;
constexpr uint32_t kOneRound = 1u << 17;
constexpr int kOnePopShift = 24;
constexpr int kOneMaxDepth = 8;  // sums put aside at once
constexpr int kOneGroup = 8;     // leaves folded together where their words allow

struct OneSeg {
    int64_t lo, hi;   // element range
    int32_t off;      // first word of its leaves
    int32_t nleaf;    // number of leaves
};

// First element of tile t of a segment that starts at lo, tiles of te elements.
__host__ __device__ __forceinline__ int64_t one_tile(int64_t lo, int64_t t, int64_t te,
                                                     int32_t amask) {
    return (lo & ~int64_t(amask)) + t * te;
}
// A lane's vector in a tile at t0 that reaches over an end of its segment
// [lo, hi): it would start at element e; it is loaded from element `at` and
// elements [fa, fb) of it are stored (none when fa >= fb).
struct OneLane {
    int64_t at;
    int fa, fb;
};
__host__ __device__ __forceinline__ OneLane one_lane(int64_t t0, int64_t e, int64_t lo, int64_t hi,
                                                     int64_t N, int vec) {
    OneLane l;
    const bool in = e < hi;  // past the end: the tile's first vector, nothing stored
    const int64_t from = in ? e : t0;
    l.at = from < N - vec ? from : N - vec;
    l.fa = in ? int((e > lo ? e : lo) - l.at) : vec;
    l.fb = in ? int((e + vec < hi ? e + vec : hi) - l.at) : 0;
    return l;
}

// LB bytes of elements as a lane holds them (V), as they lie in memory (M:
// element alignment), and their sum.
typedef uint32_t u32_a2 __attribute__((aligned(2)));
template <int DT, int LB> struct OneVec;
template <int DT> struct OneVec<DT, 16> { using V = u32x4; using M = u32x4_a4; using Acc = VAcc<DT>; };
template <> struct OneVec<DT_BF16, 16> { using V = u32x4; using M = u32x4_a2; using Acc = VAcc<DT_BF16>; };
template <int DT> struct OneVec<DT, 4> { using V = uint32_t; using M = uint32_t; using Acc = WAcc<DT>; };
template <> struct OneVec<DT_BF16, 4> { using V = uint32_t; using M = u32_a2; using Acc = WAcc<DT_BF16>; };

// Element i of its vector's word x.
template <class T> __device__ __forceinline__ T one_elem(uint32_t x, int i);
template <> __device__ __forceinline__ float one_elem<float>(uint32_t x, int) { return __uint_as_float(x); }
template <> __device__ __forceinline__ uint32_t one_elem<uint32_t>(uint32_t x, int) { return x; }
template <> __device__ __forceinline__ uint16_t one_elem<uint16_t>(uint32_t x, int i) { return uint16_t(x >> (16 * (i & 1))); }

template <int DT, int LB, int U, int B, int W, int CM>
struct OnePass {
    using V = typename OneVec<DT, LB>::V;
    using M = typename OneVec<DT, LB>::M;
    using Acc = typename OneVec<DT, LB>::Acc;
    using T = typename Elem<DT>::T;
    static constexpr int VEC = LB / int(sizeof(T));
    static constexpr int AW = int(sizeof(Acc) / 4);  // words of a sum

    Acc acc[U];
    uint32_t* stk;    // this lane's part of the sums put aside
    int depth;
    uint32_t off[U];  // byte offset of the lane's vectors from the tile's base

    template <bool EDGE>
    __device__ __forceinline__ V load(uint64_t base, int u) const {
        const AR_GLOBAL char* p = (const AR_GLOBAL char*)base + off[EDGE ? u : 0];
        if (!EDGE) p += u * (64 * LB);
        if constexpr (CM & 1) return __builtin_nontemporal_load((const AR_GLOBAL M*)p);
        else return *(const AR_GLOBAL M*)p;
    }

    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t a[AW];
#pragma unroll
            for (int q = 0; q < AW; ++q) a[q] = DT == DT_I32 ? 0u : 0x80000000u;
            __builtin_memcpy(&acc[u], a, sizeof(Acc));
        }
    }
    __device__ __forceinline__ void push() {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t a[AW];
            __builtin_memcpy(a, &acc[u], sizeof(Acc));
#pragma unroll
            for (int q = 0; q < AW; ++q) stk[((depth * U + u) * AW + q) * (64 * W)] = a[q];
        }
        ++depth;
        zero();
    }
    __device__ __forceinline__ void pop_add() {
        --depth;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const V v = acc[u].out();
            uint32_t a[AW];
#pragma unroll
            for (int q = 0; q < AW; ++q) a[q] = stk[((depth * U + u) * AW + q) * (64 * W)];
            __builtin_memcpy(&acc[u], a, sizeof(Acc));
            acc[u].add(v);
        }
    }
    // what leaf j's word asks for after its row is added
    __device__ __forceinline__ void after(uint32_t w, int j) {
        const uint32_t o = uint32_t(__builtin_amdgcn_readlane(int(w), j));
        for (uint32_t k = o >> kOnePopShift; k; --k) pop_add();
        if (DT == DT_BF16 && (o & kOneRound))
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u].init(acc[u].out());
    }

    // Fold G leaves, j0 .. of the chunk (pushes, pops, rounds: bit j, leaf j's
    // word asks for it).  Two straight forms, a chain of two-source bf16 steps
    // and a run of one fold (a push before its first leaf, what follows its
    // first or last one), and the general one.
    template <int G>
    __device__ __forceinline__ void group(const V (&x)[G][U], uint32_t w, uint64_t pushes,
                                          uint64_t pops, uint64_t rounds, int j0) {
        constexpr uint64_t all = ~uint64_t(0) >> (64 - G);
        constexpr uint64_t ends = uint64_t(1) | uint64_t(1) << (G - 1);
        const uint64_t pu = (pushes >> j0) & all, po = (pops >> j0) & all;
        const uint64_t rd = DT == DT_BF16 ? (rounds >> j0) & all : 0;
        const uint64_t cl = po | rd;
        if (DT == DT_BF16 && (pu | po) == 0 && rd == all) {
#pragma unroll
            for (int j = 0; j < G; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    acc[u].add(x[j][u]);
                    acc[u].init(acc[u].out());
                }
        } else if ((pu & ~uint64_t(1)) == 0 && (cl & ~ends) == 0) {
            if (pu) push();
#pragma unroll
            for (int j = 0; j < G; ++j) {
#pragma unroll
                for (int u = 0; u < U; ++u) acc[u].add(x[j][u]);
                if (j == 0 && G > 1 && (cl & 1)) after(w, j0);
            }
            if (cl >> (G - 1)) after(w, j0 + G - 1);
        } else {
#pragma unroll
            for (int j = 0; j < G; ++j) {
                if ((pu >> j) & 1) push();
#pragma unroll
                for (int u = 0; u < U; ++u) acc[u].add(x[j][u]);
                if ((cl >> j) & 1) after(w, j0 + j);
            }
        }
    }

    // leaves j0 .. j0 + BB of a chunk whose words and pointers the lanes hold
    template <int BB, bool EDGE>
    __device__ __forceinline__ void batch(uint32_t w, uint32_t plo, uint32_t phi, uint64_t tbase,
                                          uint64_t pushes, uint64_t pops, uint64_t rounds, int j0) {
        constexpr int G = BB < kOneGroup ? BB : kOneGroup;
        V x[BB / G][G][U];
#pragma unroll
        for (int j = 0; j < BB; ++j) {
            const uint64_t base =
                ((uint64_t(uint32_t(__builtin_amdgcn_readlane(int(phi), j0 + j))) << 32) |
                 uint32_t(__builtin_amdgcn_readlane(int(plo), j0 + j))) + tbase;
#pragma unroll
            for (int u = 0; u < U; ++u) x[j / G][j % G][u] = load<EDGE>(base, u);
        }
#pragma unroll
        for (int g = 0; g < BB / G; ++g) group<G>(x[g], w, pushes, pops, rounds, j0 + g * G);
    }

    template <bool EDGE>
    __device__ __forceinline__ void fold(const uint64_t* __restrict__ ptab,
                                         const uint32_t* __restrict__ leaf, int nleaf,
                                         uint64_t tbase, int lane) {
        uint32_t w = lane < nleaf ? leaf[lane] : 0u;
        uint64_t p = ptab[w & 0xFFFFu];
        for (int c0 = 0; c0 < nleaf; c0 += 64) {
            const int m = min(64, nleaf - c0);
            const uint32_t plo = uint32_t(p), phi = uint32_t(p >> 32);
            const uint64_t pushes = __builtin_amdgcn_ballot_w64((w & kOnePush) != 0);
            const uint64_t pops = __builtin_amdgcn_ballot_w64(w >> kOnePopShift != 0);
            const uint64_t rounds = __builtin_amdgcn_ballot_w64((w & kOneRound) != 0);
            const uint32_t wn = c0 + 64 + lane < nleaf ? leaf[c0 + 64 + lane] : 0u;
            int j = 0;
            for (; j + B <= m; j += B) batch<B, EDGE>(w, plo, phi, tbase, pushes, pops, rounds, j);
            if constexpr (B > 16)
                if (j + 16 <= m) { batch<16, EDGE>(w, plo, phi, tbase, pushes, pops, rounds, j); j += 16; }
            if constexpr (B > 8)
                if (j + 8 <= m) { batch<8, EDGE>(w, plo, phi, tbase, pushes, pops, rounds, j); j += 8; }
            if constexpr (B > 4)
                if (j + 4 <= m) { batch<4, EDGE>(w, plo, phi, tbase, pushes, pops, rounds, j); j += 4; }
            if constexpr (B > 2)
                if (j + 2 <= m) { batch<2, EDGE>(w, plo, phi, tbase, pushes, pops, rounds, j); j += 2; }
            if constexpr (B > 1)
                if (j < m) batch<1, EDGE>(w, plo, phi, tbase, pushes, pops, rounds, j);
            if (c0 + 64 < nleaf) {
                w = wn;
                p = ptab[w & 0xFFFFu];
            }
        }
    }
};

// One launch: `nunits` tiles of 64 x U vectors, tile `t` of segment `s` from
// the table `tiles`, or arithmetic with tiles_per_seg of each (tiles past a
// segment's end do nothing).  ptab: the n buffer pointers.  CM: bit 0
// nontemporal loads, bit 1 nontemporal stores.  The grid is 8 * per_xcd:
// workgroups go to the eight XCDs in turn, and each runs a contiguous eighth
// of the tiles; per_xcd = 0: tile after tile, whatever the XCD.  (per_xcd is an
// argument: a kernel that reads gridDim takes the 256 bytes of implicit
// arguments, 1 us more a launch on the host.)
template <int DT, int LB, int U, int B, int W, int CM>
__global__ __launch_bounds__(64 * W) void onepass_kernel(
    const uint64_t* __restrict__ ptab, int32_t n, const uint32_t* __restrict__ prog,
    const OneSeg* __restrict__ segs, int32_t nseg, const int2* __restrict__ tiles, uint32_t nunits,
    uint32_t tiles_per_seg, uint32_t per_xcd, int64_t N, int32_t amask) {
    extern __shared__ uint32_t aside[];
    using K = OnePass<DT, LB, U, B, W, CM>;
    using V = typename K::V;
    using M = typename K::M;
    using T = typename K::T;
    constexpr int VEC = K::VEC;
    constexpr int64_t TE = int64_t(64) * U * VEC;  // elements of a tile
    const int lane = int(threadIdx.x) & 63;
    const uint32_t b = per_xcd ? (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3) : blockIdx.x;
    const uint32_t unit = b * W + uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    if (unit >= nunits) return;
    uint32_t s = 0, t = unit;
    if (tiles) {
        const int2 e = tiles[unit];
        s = uint32_t(__builtin_amdgcn_readfirstlane(e.x));
        t = uint32_t(__builtin_amdgcn_readfirstlane(e.y));
    } else if (nseg > 1) {
        s = unit / tiles_per_seg;
        t = unit - s * tiles_per_seg;
    }
    const OneSeg sg = segs[s];
    const int64_t t0 = one_tile(sg.lo, int64_t(t), TE, amask);
    if (t0 >= sg.hi) return;
    const bool edge = t0 < sg.lo || t0 + TE > sg.hi;
    // the lanes count from `back` elements before the tile: a vector moved
    // back from the buffers' end may start before it
    const int64_t back = t0 < VEC ? t0 : VEC;
    const uint64_t tbase = uint64_t(t0 - back) * sizeof(T);
    K k;
    k.stk = aside + threadIdx.x;
    k.depth = 0;
    k.zero();
    uint64_t dp = lane < n ? ptab[lane] : 0;
    if (!edge) {
        k.off[0] = uint32_t((back + lane * VEC) * int64_t(sizeof(T)));
        k.template fold<false>(ptab, prog + sg.off, sg.nleaf, tbase, lane);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const OneLane l = one_lane(t0, t0 + (u * 64 + lane) * VEC, sg.lo, sg.hi, N, VEC);
            k.off[u] = uint32_t((l.at - (t0 - back)) * int64_t(sizeof(T)));
        }
        k.template fold<true>(ptab, prog + sg.off, sg.nleaf, tbase, lane);
    }
    uint32_t full = 0;  // bit u: all of this lane's vector u is stored
    uint64_t part[U];   // lanes of which a part is
    if (edge) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const OneLane l = one_lane(t0, t0 + (u * 64 + lane) * VEC, sg.lo, sg.hi, N, VEC);
            const bool f = l.fa == 0 && l.fb == VEC;
            full |= uint32_t(f) << u;
            part[u] = __builtin_amdgcn_ballot_w64(!f && l.fa < l.fb);
        }
    }
    V out[U];
#pragma unroll
    for (int u = 0; u < U; ++u) out[u] = k.acc[u].out();
    for (int c0 = 0; c0 < n; c0 += 64) {
        const uint32_t plo = uint32_t(dp), phi = uint32_t(dp >> 32);
        const int m = min(64, n - c0);
        if (c0 + 64 < n) dp = c0 + 64 + lane < n ? ptab[c0 + 64 + lane] : 0;
        auto base = [&](int j) {
            return ((uint64_t(uint32_t(__builtin_amdgcn_readlane(int(phi), j))) << 32) |
                    uint32_t(__builtin_amdgcn_readlane(int(plo), j))) + tbase;
        };
        if (!edge) {
            for (int j = 0; j < m; ++j) {
                AR_GLOBAL char* p = (AR_GLOBAL char*)base(j) + k.off[0];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if constexpr (CM & 2) __builtin_nontemporal_store(out[u], (AR_GLOBAL M*)(p + u * (64 * LB)));
                    else *(AR_GLOBAL M*)(p + u * (64 * LB)) = out[u];
                }
            }
        } else {
            for (int j = 0; j < m; ++j) {
                AR_GLOBAL char* p = (AR_GLOBAL char*)base(j);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (full >> u & 1) *(AR_GLOBAL M*)(p + k.off[u]) = out[u];
            }
            // the vectors that reach over an end (two at most): each lane
            // stores their elements to the buffer whose pointer it holds
            if constexpr (VEC > 1) {
                const uint64_t mine = ((uint64_t(phi) << 32) | plo) + tbase;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    for (uint64_t pm = part[u]; pm; pm &= pm - 1) {
                        const int L = __builtin_ctzll(pm);
                        const OneLane l =
                            one_lane(t0, t0 + (u * 64 + L) * VEC, sg.lo, sg.hi, N, VEC);
                        AR_GLOBAL T* p = (AR_GLOBAL T*)(mine + uint64_t(l.at - (t0 - back)) * sizeof(T));
                        uint32_t word[LB / 4];
                        __builtin_memcpy(word, &out[u], LB);
#pragma unroll
                        for (int i = 0; i < VEC; ++i) {
                            const uint32_t x =
                                uint32_t(__builtin_amdgcn_readlane(int(word[i * int(sizeof(T)) / 4]), L));
                            const T v = one_elem<T>(x, i);
                            if (lane < m && i >= l.fa && i < l.fb) p[i] = v;
                        }
                    }
            }
        }
    }
}

// The same with a workgroup of W wavefronts per tile of 64 4-byte lanes, for
// few positions and many buffers, where a wavefront's time is its n loads and
// n stores one after the other: each wave loads LPW leaves of a chunk of
// W * LPW into LDS (the next chunk's loads go out before the current one is
// folded, two chunk buffers), one wave folds them from there, and each
// wave stores to its share of the buffers once every load has been used.
// LDS: two chunk buffers, the result, the sums put aside.
template <int DT, int W, int LPW>
__global__ __launch_bounds__(64 * W) void onepass_team_kernel(
    const uint64_t* __restrict__ ptab, int32_t n, const uint32_t* __restrict__ prog,
    const OneSeg* __restrict__ segs, int32_t nseg, const int2* __restrict__ tiles, uint32_t nunits,
    uint32_t tiles_per_seg, uint32_t per_xcd, int64_t N, int32_t amask) {
    extern __shared__ uint32_t lds[];
    using K = OnePass<DT, 4, 1, kOneGroup, 1, 0>;
    using V = typename K::V;
    using M = typename K::M;
    using T = typename K::T;
    constexpr int VEC = K::VEC;
    constexpr int64_t TE = int64_t(64) * VEC;
    constexpr int C = W * LPW;  // leaves of a chunk
    // workgroups on one compute unit (256 apart) fold on different SIMDs
    const int folder = int(blockIdx.x >> 8) % W;
    const int lane = int(threadIdx.x) & 63;
    const int wv = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const uint32_t unit = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (unit >= nunits) return;  // the same for the whole workgroup
    uint32_t s = 0, t = unit;
    if (tiles) {
        const int2 e = tiles[unit];
        s = uint32_t(__builtin_amdgcn_readfirstlane(e.x));
        t = uint32_t(__builtin_amdgcn_readfirstlane(e.y));
    } else if (nseg > 1) {
        s = unit / tiles_per_seg;
        t = unit - s * tiles_per_seg;
    }
    const OneSeg sg = segs[s];
    const int64_t t0 = one_tile(sg.lo, int64_t(t), TE, amask);
    if (t0 >= sg.hi) return;
    const int64_t back = t0 < VEC ? t0 : VEC;
    const uint64_t tbase = uint64_t(t0 - back) * sizeof(T);
    const OneLane l = one_lane(t0, t0 + lane * VEC, sg.lo, sg.hi, N, VEC);
    const uint32_t* const leaf = prog + sg.off;
    uint32_t* const res = lds + 2 * C * 64;
    K k;
    k.off[0] = uint32_t((l.at - (t0 - back)) * int64_t(sizeof(T)));
    k.stk = res + 64 + lane;
    k.depth = 0;
    k.zero();
    // this wave's leaves of the chunk at c0: their pointers, a lane each, then
    // their rows
    auto pointers = [&](int c0) -> uint64_t {
        const int i = c0 + wv * LPW + lane;
        return lane < LPW && i < sg.nleaf ? ptab[leaf[i] & 0xFFFFu] : 0;
    };
    V x[LPW];
    auto issue = [&](int c0, uint64_t p) {
        const int cnt = min(LPW, sg.nleaf - (c0 + wv * LPW));
        const uint32_t plo = uint32_t(p), phi = uint32_t(p >> 32);
        auto row = [&](int j) {
            return k.template load<false>(
                ((uint64_t(uint32_t(__builtin_amdgcn_readlane(int(phi), j))) << 32) |
                 uint32_t(__builtin_amdgcn_readlane(int(plo), j))) + tbase, 0);
        };
        if (cnt == LPW) {
#pragma unroll
            for (int j = 0; j < LPW; ++j) x[j] = row(j);
        } else {
#pragma unroll
            for (int j = 0; j < LPW; ++j) x[j] = j < cnt ? row(j) : V(0);
        }
    };
    issue(0, pointers(0));
    // the pointers of the buffers this wave stores to
    const int d0 = int(int64_t(n) * wv / W), d1 = int(int64_t(n) * (wv + 1) / W);
    uint64_t dp = d0 + lane < d1 ? ptab[d0 + lane] : 0;
    uint64_t pn = pointers(C);
    for (int c0 = 0; c0 < sg.nleaf; c0 += C) {
        uint32_t* const rows = lds + (c0 / C & 1) * C * 64;
#pragma unroll
        for (int j = 0; j < LPW; ++j) rows[(wv * LPW + j) * 64 + lane] = x[j];
        if (c0 + C < sg.nleaf) {
            issue(c0 + C, pn);
            pn = pointers(c0 + 2 * C);
        }
        __syncthreads();
        if (wv == folder) {
            for (int s0 = 0; s0 < C && c0 + s0 < sg.nleaf; s0 += 64) {
                const int m = min(min(64, C - s0), sg.nleaf - c0 - s0);
                const uint32_t w = lane < m ? leaf[c0 + s0 + lane] : 0u;
                const uint64_t pushes = __builtin_amdgcn_ballot_w64((w & kOnePush) != 0);
                const uint64_t pops = __builtin_amdgcn_ballot_w64(w >> kOnePopShift != 0);
                const uint64_t rounds = __builtin_amdgcn_ballot_w64((w & kOneRound) != 0);
                const uint32_t* const r = rows + s0 * 64 + lane;
                int j = 0;
                for (; j + kOneGroup <= m; j += kOneGroup) {
                    V y[kOneGroup][1];
#pragma unroll
                    for (int q = 0; q < kOneGroup; ++q) y[q][0] = r[(j + q) * 64];
                    k.template group<kOneGroup>(y, w, pushes, pops, rounds, j);
                }
                for (; j < m; ++j) {
                    V y[1][1] = {{r[j * 64]}};
                    k.template group<1>(y, w, pushes, pops, rounds, j);
                }
            }
        }
    }
    if (wv == folder) res[lane] = k.acc[0].out();
    __syncthreads();
    const V out = res[lane];
    const bool full = l.fa == 0 && l.fb == VEC;
    const uint64_t part = __builtin_amdgcn_ballot_w64(!full && l.fa < l.fb);
    for (int c0 = d0; c0 < d1; c0 += 64) {
        const uint32_t plo = uint32_t(dp), phi = uint32_t(dp >> 32);
        const int m = min(64, d1 - c0);
        if (c0 + 64 < d1) dp = c0 + 64 + lane < d1 ? ptab[c0 + 64 + lane] : 0;
        if (full)
            for (int j = 0; j < m; ++j) {
                const uint64_t base =
                    ((uint64_t(uint32_t(__builtin_amdgcn_readlane(int(phi), j))) << 32) |
                     uint32_t(__builtin_amdgcn_readlane(int(plo), j))) + tbase;
                *(AR_GLOBAL M*)((AR_GLOBAL char*)base + k.off[0]) = out;
            }
        if constexpr (VEC > 1) {
            const uint64_t mine = ((uint64_t(phi) << 32) | plo) + tbase;
            for (uint64_t pm = part; pm; pm &= pm - 1) {
                const int L = __builtin_ctzll(pm);
                const OneLane e = one_lane(t0, t0 + L * VEC, sg.lo, sg.hi, N, VEC);
                AR_GLOBAL T* p = (AR_GLOBAL T*)(mine + uint64_t(e.at - (t0 - back)) * sizeof(T));
                const uint32_t word = uint32_t(__builtin_amdgcn_readlane(int(out), L));
#pragma unroll
                for (int i = 0; i < VEC; ++i)
                    if (lane < m && i >= e.fa && i < e.fb) p[i] = one_elem<T>(word, i);
            }
        }
    }
}

}  // namespace arp
