// gfx950 kernels of the tiled D3Q19 lattice-Boltzmann method.
//
// Mapping (re-designed for CDNA4 from the paper's thread mapping, Section 3.1):
// one 4x4x4 tile = one wave64, lane n = x + 4y + 16z.  A tile's values form
// 19 blocks, one per direction ("data block", Section 3.2).
//
// Layout of a tile's blocks.  With FP64 and FP32 storage a tile with k fluid
// nodes owns one run of 19 * k values, block i at offset i * k, the node at
// slot = number of fluid nodes of the tile with a smaller node index; the run
// is padded to whole 128-byte lines, so solid nodes take no space and only
// lines holding fluid values are read or written.  With FP16 storage a block
// is 64 values, exactly one 128-byte line, and slot = node index.  This
// replaces the paper's per-direction node maps (Eq. 11-13), tuned for 32-byte
// Kepler sectors: at 128-byte lines what matters is how many lines a block
// touches.
//
// Streaming is a pull (gather) fused with collision (Sections 2.3 and 3.4,
// Alg. 2).
// For every direction the lanes split into at most four regions by which
// neighbour tile holds their source node; inside a region the source node is
// this lane's index plus a constant, so its slot is
//     slot = mbcnt(mask of that tile, shifted by the constant) + constant'
// (one v_mbcnt pair) and every tile number, shift and constant is computed
// once per wave on the scalar unit.  The scalar unit also combines the fluid
// masks into one 64-bit "source is fluid" mask per direction, used directly
// as the lane condition (inverse ballot) between the upstream value and the
// halfway bounce-back value at the node itself.
#include <hip/hip_runtime.h>

#include <climits>
#include <type_traits>
#include <utility>

#include "kernels.hpp"

namespace tlbm {

// ---------------------------------------------------------------------------
// storage codecs
//   F64 : f_i as double, arithmetic in double
//   F32 : d_i = f_i - w_i rho0 as float, arithmetic in float
//   F16S: h_i = fp16(s * d_i), s = 2^k, arithmetic in float
// The kernels work on the shifted value d_i = f_i - w_i rho_base (rho_base = 0
// for F64).  Opposite directions have equal weights, so a bounce-back copy
// needs no re-shift.
// ---------------------------------------------------------------------------
template <int ST> struct Codec;
template <> struct Codec<LBM_F64> {
    using S = double;
    using T = double;
    static constexpr bool RUNS = true;
    static constexpr bool SCALED = false;
    static __device__ __forceinline__ T dec(S v, float) { return v; }
    static __device__ __forceinline__ S enc(T v, float) { return v; }
};
template <> struct Codec<LBM_F32> {
    using S = float;
    using T = float;
    static constexpr bool RUNS = true;
    static constexpr bool SCALED = false;
    static __device__ __forceinline__ T dec(S v, float) { return v; }
    static __device__ __forceinline__ S enc(T v, float) { return v; }
};
template <> struct Codec<LBM_F16S> {
    using S = _Float16;
    using T = float;
    static constexpr bool RUNS = false;
    // The step works on the stored scale: D_i = s d_i with s = 2^k, so
    // decoding and encoding are bare conversions (38 fewer vector
    // multiplications per tile).  Scaling by a power of two is exact and
    // commutes with rounding, so this is the unscaled arithmetic up to the
    // compiler's choice of fused multiply-adds, which differs between the two
    // forms (stored values move by about one FP16 ulp).
    static constexpr bool SCALED = true;
    static __device__ __forceinline__ T dec(S v, float inv_scale) { return (float)v * inv_scale; }
    static __device__ __forceinline__ S enc(T v, float scale) { return (_Float16)(v * scale); }
    static __device__ __forceinline__ T dec_scaled(S v) { return (float)v; }
    static __device__ __forceinline__ S enc_scaled(T v) { return (_Float16)v; }
    // Stochastic rounding to FP16 with gfx950's conversion instruction: it
    // rounds away from zero with probability equal to the discarded fraction
    // of an FP16 ulp (normal and subnormal results alike), drawing on the high
    // bits of r; values exact in FP16 are unchanged.  The rounding error has
    // zero mean, so a per-step increment smaller than half an ulp is kept on
    // average instead of being lost.
    // The instruction writes one half of a 32-bit register and keeps the
    // other; `pair` carries that register from one call to the next.
    typedef _Float16 Pair __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ S enc_sr_scaled(T v, uint32_t r, Pair &pair) {
        pair = __builtin_amdgcn_cvt_sr_f16_f32(pair, v, r, false);
        return pair[0];
    }
};

// Counter-based random bits for the FP16 stochastic rounding: an integer hash
// (the "lowbias32" mixer of C. Wellons) of the node's coordinates and the
// launch counter, then a Weyl sequence over the 19 directions, whose high bits
// the conversion uses.
__device__ __forceinline__ uint32_t hash32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

// ---------------------------------------------------------------------------
// wave -> tile mapping
// ---------------------------------------------------------------------------
// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2;
// all of them share the Infinity Cache in front of HBM).  They are re-numbered
// so that each XCD works through chunks of 32 consecutive tiles (in the device
// tile order) and the 8 XCDs through 8 adjacent chunks at a time: most of a
// tile's neighbours are then in its own chunk, on the same L2, and the rest in
// chunks the other XCDs are working on at the same time, whose shared lines
// are still in the Infinity Cache.  Measured on a 256^3 sphere pack against
// one contiguous range per XCD: FP64 step 411.8 -> 387.9 us, FP32 234.2 ->
// 219.1 us, FP64 adjoint step 115.8 -> 111.7 us (LBMRT 122.1 -> 118.8 us at
// one tile per workgroup); chunks of 16 to 64 tiles are within 1% of that, of
// 8 or 256 tiles 2-3% slower.  The whole-block FP16 kernels are the
// exception: one contiguous range per XCD is 1.3% faster for them than any
// chunking.
// Blocks past the last whole round of 8 chunks keep their number.
__device__ __forceinline__ int remap_block(int b, int nb, int lc) {
    const int full = (nb >> (lc + 3)) << (lc + 3);
    if (b >= full) return b;
    const int xcd = b & 7, local = b >> 3;
    return ((((local >> lc) << 3) + xcd) << lc) + (local & ((1 << lc) - 1));
}

__device__ __forceinline__ int remap_block_contiguous(int b, int nb) {
    const int q = nb >> 3, r = nb & 7;
    const int xcd = b & 7, local = b >> 3;
    return xcd * q + (xcd < r ? xcd : r) + local;
}

// lw (log2 of the waves per workgroup, at most 3) and nb (workgroups) come
// in as kernel arguments: reading blockDim from the dispatch packet would cost
// every wave a memory round trip before its first instruction of real work.
constexpr int CHUNK_TILES_LOG2 = 5;
template <bool CONTIGUOUS = false>
__device__ __forceinline__ int wave_tile(int lw, int nb) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if constexpr (CONTIGUOUS) {
        return (remap_block_contiguous((int)blockIdx.x, nb) << lw) + wave;
    } else {
        const int lc = CHUNK_TILES_LOG2 - lw;  // workgroups per chunk = 32 >> lw
        return (remap_block((int)blockIdx.x, nb, lc) << lw) + wave;
    }
}

__device__ __forceinline__ bool lane_on(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

__device__ __forceinline__ uint64_t field_elems_dev(uint64_t mask) {
    const uint64_t k = (uint64_t)__builtin_popcountll(mask);
    return (3 * k + FIELD_PAD - 1) / FIELD_PAD * FIELD_PAD;
}

// number of set bits of m below this lane
__device__ __forceinline__ int mbcnt(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ---------------------------------------------------------------------------
// neighbourhood of a tile (wave-uniform: lives in SGPRs)
// ---------------------------------------------------------------------------
template <typename OffT>
struct Nbhd {
    uint64_t m[27];  // fluid masks (0 for a missing neighbour)
    OffT base[27];   // element offset of each neighbour's data
};

// A row as four 16-register scalar loads, waited for together: without the
// empty asm the compiler waits for the tile's own mask alone, branches on it
// and only then loads the rest of the row, a second round trip to memory
// before the first gather can be issued.
// (A scalar load asks for no more than 4-byte alignment, and neither the tables
// nor a kernel's arguments are sure to have more than 8.)
typedef uint32_t u32x16 __attribute__((ext_vector_type(16), aligned(4)));
struct RowRegs {
    u32x16 q[4];
    __device__ __forceinline__ explicit RowRegs(const NbRow *row, int t) {
        const u32x16 *p = reinterpret_cast<const u32x16 *>(row + t);
        q[0] = p[0];
        q[1] = p[1];
        q[2] = p[2];
        q[3] = p[3];
        asm volatile("" : "+s"(q[0]), "+s"(q[1]), "+s"(q[2]), "+s"(q[3]));
    }
    __device__ __forceinline__ uint32_t dword(int i) const { return q[i >> 4][i & 15]; }
    __device__ __forceinline__ uint64_t qword(int i) const { return dword(i) | (uint64_t)dword(i + 1) << 32; }
    __device__ __forceinline__ uint64_t mask(int s) const { return qword(2 * s); }
    __device__ __forceinline__ uint32_t base32(int s) const { return dword((int)offsetof(NbRow, base32) / 4 + s); }
    __device__ __forceinline__ uint64_t fbase() const { return qword((int)offsetof(NbRow, fbase) / 4); }
    __device__ __forceinline__ uint32_t xyz(int c) const { return dword((int)offsetof(NbRow, xyz) / 4 + c); }
};

// A tile's data starts on a line of 128 bytes, so with 64-bit offsets the row
// holds its line number (all of 512 GB) and the element offset is a shift
// away.  A table of 64-bit offsets beside the rows was a second read, waited
// for between the gathers (256^3 pack with 64-bit offsets, us a step: FP64
// 377 -> 361, FP32 222 -> 208, FP16 194 -> 165; FP64 LBMRT 410 -> 391, FP32
// 253 -> 228).  Dense boxes, where waves that start their gathers later get in
// each other's way less, lost by it (FP64 384^3 box 3198 -> 3257); they now keep
// fewer waves in flight instead: see stage_request.
template <typename S, typename OffT>
__device__ __forceinline__ void load_nbhd(Nbhd<OffT> &h, const RowRegs &r) {
    constexpr int LINE = __builtin_ctz(128 / sizeof(S));
#pragma unroll
    for (int k = 0; k < 27; ++k) {
        const int s = nb_slot(k);
        h.m[k] = s < 0 ? 0ull : r.mask(s);
        if constexpr (std::is_same<OffT, uint32_t>::value) h.base[k] = s < 0 ? 0u : r.base32(s);
        else h.base[k] = s < 0 ? 0ull : (uint64_t)r.base32(s) << LINE;
    }
}
constexpr int OWN = 13;  // the tile itself in its neighbourhood

// where this lane's own values live
template <bool RUNS, typename OffT>
struct Self {
    OffT base;    // element offset of the tile's data
    OffT stride;  // elements between directions: k (runs) or 64 (plain)
    int slot;     // this node's slot in each block
    int k;        // fluid nodes of the tile
    __device__ __forceinline__ Self(const TileRec &r, int lane) : Self(r.mask, (OffT)r.base, lane) {}
    __device__ __forceinline__ Self(const Nbhd<OffT> &h, int lane) : Self(h.m[OWN], h.base[OWN], lane) {}
    __device__ __forceinline__ Self(uint64_t mask, OffT first, int lane) {
        base = first;
        k = __builtin_popcountll(mask);
        if constexpr (RUNS) {
            stride = (OffT)k;
            slot = mbcnt(mask);
        } else {
            stride = (OffT)TILE;
            slot = lane;
        }
    }
    __device__ __forceinline__ OffT elem(int i) const { return base + (OffT)i * stride + (OffT)slot; }
};

// lanes whose source node (x+sx, y+sy, z+sz) leaves the tile exactly along the
// axes flagged bx, by, bz
constexpr uint64_t region_mask(int sx, int sy, int sz, int bx, int by, int bz) {
    uint64_t r = 0;
    for (int n = 0; n < 64; ++n) {
        const int x = n & 3, y = (n >> 2) & 3, z = n >> 4;
        const int cx = (x + sx < 0 || x + sx > 3), cy = (y + sy < 0 || y + sy > 3), cz = (z + sz < 0 || z + sz > 3);
        if (cx == bx && cy == by && cz == bz) r |= 1ull << n;
    }
    return r;
}

// Region (BX,BY,BZ) of the source offset (SX,SY,SZ): its lanes read the
// neighbour tile K at in-tile node lane + OFF.
template <int SX, int SY, int SZ, int BX, int BY, int BZ>
struct Region {
    static constexpr bool axes_ok = !((BX && !SX) || (BY && !SY) || (BZ && !SZ));
    static constexpr uint64_t LANES = axes_ok ? region_mask(SX, SY, SZ, BX, BY, BZ) : 0ull;
    static constexpr bool EXISTS = LANES != 0;
    static constexpr int K = 13 + BX * SX + 3 * BY * SY + 9 * BZ * SZ;
    static constexpr int OFF = SX + 4 * SY + 16 * SZ - 4 * BX * SX - 16 * BY * SY - 64 * BZ * SZ;
};

// bits of the neighbour mask that one region's lanes read, aligned to lanes
template <class R, class H>
__device__ __forceinline__ uint64_t region_source_bits(const H &h) {
    if constexpr (!R::EXISTS) {
        return 0ull;
    } else {
        const uint64_t mk = h.m[R::K];
        return R::OFF >= 0 ? (mk >> R::OFF) : (mk << (-R::OFF));
    }
}

template <int SX, int SY, int SZ, int BX, int BY, int BZ, class H>
__device__ __forceinline__ uint64_t region_fluid(const H &h) {
    using R = Region<SX, SY, SZ, BX, BY, BZ>;
    if constexpr (!R::EXISTS) return 0ull;
    else return region_source_bits<R>(h) & R::LANES;
}

// 64-bit mask: bit n set when lane n's source node exists and is fluid
template <int SX, int SY, int SZ, class H>
__device__ __forceinline__ uint64_t source_fluid(const H &h) {
    return region_fluid<SX, SY, SZ, 0, 0, 0>(h) | region_fluid<SX, SY, SZ, 1, 0, 0>(h) |
           region_fluid<SX, SY, SZ, 0, 1, 0>(h) | region_fluid<SX, SY, SZ, 1, 1, 0>(h) |
           region_fluid<SX, SY, SZ, 0, 0, 1>(h) | region_fluid<SX, SY, SZ, 1, 0, 1>(h) |
           region_fluid<SX, SY, SZ, 0, 1, 1>(h) | region_fluid<SX, SY, SZ, 1, 1, 1>(h);
}

// Element index (within the lattice) of direction I's value at this lane's
// source node, for the lanes of one region (tile K, in-tile node lane + OFF):
//   plain: base_K + I * 64 + lane + OFF
//   runs : base_K + I * k_K + mbcnt(m_K shifted by OFF) + c,
//          k_K = popcount(m_K), c = popcount(m_K below OFF) when OFF > 0
// Every term but the mbcnt is wave-uniform.
template <class R, int I, bool RUNS, typename OffT>
__device__ __forceinline__ OffT region_elem(const Nbhd<OffT> &h, int lane) {
    const uint64_t mk = h.m[R::K];
    if constexpr (RUNS) {
        constexpr int POS = R::OFF > 0 ? R::OFF : 0;
        const int c = POS ? __builtin_popcountll(mk & ((1ull << POS) - 1ull)) : 0;
        const OffT blk = (OffT)h.base[R::K] + (OffT)I * (OffT)__builtin_popcountll(mk) + (OffT)c;
        return (OffT)mbcnt(region_source_bits<R>(h)) + blk;
    } else {
        return (OffT)lane + ((OffT)h.base[R::K] + (OffT)(I * TILE + R::OFF));
    }
}

// computed for every lane and then selected (a lane select, not a branch)
template <int SX, int SY, int SZ, int BX, int BY, int BZ, int I, bool RUNS, typename OffT>
__device__ __forceinline__ OffT region_pick(const Nbhd<OffT> &h, int lane, OffT cur) {
    using R = Region<SX, SY, SZ, BX, BY, BZ>;
    if constexpr (!R::EXISTS) {
        return cur;
    } else {
        const OffT mine = region_elem<R, I, RUNS, OffT>(h, lane);
        return lane_on(R::LANES) ? mine : cur;
    }
}

template <typename OffT, typename S>
__device__ __forceinline__ S load_elem(const char *base, OffT elem) {
    return *reinterpret_cast<const S *>(base + elem * (OffT)sizeof(S));
}

// Gather of direction I for this lane: the value of direction I at the source
// node x - c_I (REV = false: pull streaming S) or x + c_I (REV = true: its
// transpose S^T), or, when that node is solid or missing, the value of the
// opposite direction at the node itself (halfway bounce-back).
// element of block I at this lane's source node (x + (SX, SY, SZ)), for
// every lane (valid where that node exists)
template <int SX, int SY, int SZ, int I, bool RUNS, typename OffT>
__device__ __forceinline__ OffT source_elem(const Nbhd<OffT> &h, int lane) {
    OffT e = region_elem<Region<SX, SY, SZ, 0, 0, 0>, I, RUNS, OffT>(h, lane);
    e = region_pick<SX, SY, SZ, 1, 0, 0, I, RUNS, OffT>(h, lane, e);
    e = region_pick<SX, SY, SZ, 0, 1, 0, I, RUNS, OffT>(h, lane, e);
    e = region_pick<SX, SY, SZ, 1, 1, 0, I, RUNS, OffT>(h, lane, e);
    e = region_pick<SX, SY, SZ, 0, 0, 1, I, RUNS, OffT>(h, lane, e);
    e = region_pick<SX, SY, SZ, 1, 0, 1, I, RUNS, OffT>(h, lane, e);
    e = region_pick<SX, SY, SZ, 0, 1, 1, I, RUNS, OffT>(h, lane, e);
    e = region_pick<SX, SY, SZ, 1, 1, 1, I, RUNS, OffT>(h, lane, e);
    return e;
}

// Plain layout with 32-bit offsets: the element of lane n is n + C_r for the
// region r holding n, C_r = base_K + I * 64 + OFF (wave-uniform).  A lane
// select per region costs a move of C_r into a vector register and the
// select (an instruction reads one scalar operand, and the lane mask is
// one); instead the element is n + C_00 plus, for each axis a the shift
// crosses, (M_a AND (C_a - C_00)), where M_a is all ones on the lanes that
// leave the tile along a, and for the two axes of an edge direction the
// inclusion-exclusion term (M_a AND M_b AND (C_ab - C_a - C_b + C_00)).
// Unsigned wrap-around keeps every partial sum exact modulo 2^32.
template <int SX, int SY, int SZ, int BX, int BY, int BZ, int I>
__device__ __forceinline__ uint32_t plain_region_const(const Nbhd<uint32_t> &h) {
    using R = Region<SX, SY, SZ, BX, BY, BZ>;
    static_assert(R::EXISTS, "every region of a face or edge shift holds lanes");
    return h.base[R::K] + (uint32_t)(I * TILE + R::OFF);
}

// all ones on the lanes whose node plus the unit shift (AX, AY, AZ) leaves
// the tile
template <int AX, int AY, int AZ>
__device__ __forceinline__ uint32_t axis_lanes() {
    constexpr uint64_t M = region_mask(AX, AY, AZ, AX != 0, AY != 0, AZ != 0);
    return lane_on(M) ? 0xffffffffu : 0u;
}

template <int SX, int SY, int SZ, int I>
__device__ __forceinline__ uint32_t plain_source_elem(const Nbhd<uint32_t> &h, int lane) {
    // the first and (for an edge direction) the second axis the shift moves along
    constexpr int A1X = SX, A1Y = SX ? 0 : SY, A1Z = (SX || SY) ? 0 : SZ;
    constexpr int A2X = 0, A2Y = SX ? SY : 0, A2Z = (SX || SY) ? SZ : 0;
    constexpr bool EDGE = (A2Y != 0) || (A2Z != 0);
    const uint32_t c00 = plain_region_const<SX, SY, SZ, 0, 0, 0, I>(h);
    const uint32_t c1 = plain_region_const<SX, SY, SZ, A1X != 0, A1Y != 0, A1Z != 0, I>(h);
    const uint32_t m1 = axis_lanes<A1X, A1Y, A1Z>();
    uint32_t e = (uint32_t)lane + c00 + (m1 & (c1 - c00));
    if constexpr (EDGE) {
        const uint32_t c2 = plain_region_const<SX, SY, SZ, 0, A2Y != 0, A2Z != 0, I>(h);
        const uint32_t c12 = plain_region_const<SX, SY, SZ, A1X != 0, (A1Y != 0) || (A2Y != 0), A2Z != 0, I>(h);
        const uint32_t m2 = axis_lanes<A2X, A2Y, A2Z>();
        e += (m2 & (c2 - c00)) + ((m1 & m2) & (c12 - c1 - c2 + c00));
    }
    return e;
}

template <int SX, int SY, int SZ, int I, bool RUNS, typename OffT>
__device__ __forceinline__ OffT gather_source_elem(const Nbhd<OffT> &h, int lane) {
    if constexpr (!RUNS && std::is_same<OffT, uint32_t>::value) return plain_source_elem<SX, SY, SZ, I>(h, lane);
    else return source_elem<SX, SY, SZ, I, RUNS, OffT>(h, lane);
}

template <int I, bool REV, bool RUNS, typename S, typename OffT>
__device__ __forceinline__ S gather_one(const Nbhd<OffT> &h, const char *base, const Self<RUNS, OffT> &me, int lane) {
    if constexpr (I == 0) {
        return load_elem<OffT, S>(base, me.elem(0));
    } else {
        constexpr int SX = REV ? CX[I] : -CX[I];
        constexpr int SY = REV ? CY[I] : -CY[I];
        constexpr int SZ = REV ? CZ[I] : -CZ[I];
        constexpr int OP = opposite(I);
        const uint64_t ok_mask = source_fluid<SX, SY, SZ>(h);
        const OffT e = gather_source_elem<SX, SY, SZ, I, RUNS, OffT>(h, lane);
        return load_elem<OffT, S>(base, lane_on(ok_mask) ? e : me.elem(OP));
    }
}

// The adjoint step needs S^T applied to one lattice (direction I from
// x + c_I) and S applied to another (direction opp(I) from x - c_opp(I),
// the same node): both come from one address computation, two loads.
template <int I, bool RUNS, typename S, typename OffT>
__device__ __forceinline__ void gather_pair(const Nbhd<OffT> &h, const char *rev_base, const char *fwd_base,
                                            const Self<RUNS, OffT> &me, int lane, S &rev_I, S &fwd_op) {
    constexpr int OP = opposite(I);
    if constexpr (I == 0) {
        rev_I = load_elem<OffT, S>(rev_base, me.elem(0));
        fwd_op = load_elem<OffT, S>(fwd_base, me.elem(0));
    } else {
        const bool ok = lane_on(source_fluid<CX[I], CY[I], CZ[I]>(h));
        const OffT e_rev = source_elem<CX[I], CY[I], CZ[I], I, RUNS, OffT>(h, lane);
        const OffT e_fwd = source_elem<CX[I], CY[I], CZ[I], OP, RUNS, OffT>(h, lane);
        rev_I = load_elem<OffT, S>(rev_base, ok ? e_rev : me.elem(OP));
        fwd_op = load_elem<OffT, S>(fwd_base, ok ? e_fwd : me.elem(I));
    }
}

template <bool RUNS, typename S, typename OffT, int... Is>
__device__ __forceinline__ void gather_pairs_impl(S (&rev)[Q], S (&fwd)[Q], const Nbhd<OffT> &h, const char *rev_base,
                                                  const char *fwd_base, const Self<RUNS, OffT> &me, int lane,
                                                  std::integer_sequence<int, Is...>) {
    ((gather_pair<Is, RUNS, S, OffT>(h, rev_base, fwd_base, me, lane, rev[Is], fwd[opposite(Is)]),
      __builtin_amdgcn_sched_barrier(0)),
     ...);
}

// rev = S^T applied to the lattice at rev_base, fwd = S applied to the one at
// fwd_base
template <bool RUNS, typename S, typename OffT>
__device__ __forceinline__ void gather_pairs(S (&rev)[Q], S (&fwd)[Q], const Nbhd<OffT> &h, const char *rev_base,
                                             const char *fwd_base, const Self<RUNS, OffT> &me, int lane) {
    gather_pairs_impl<RUNS, S, OffT>(rev, fwd, h, rev_base, fwd_base, me, lane, std::make_integer_sequence<int, Q>{});
}

template <bool REV, bool RUNS, typename S, typename OffT, int... Is>
__device__ __forceinline__ void gather_all_impl(S (&v)[Q], const Nbhd<OffT> &h, const char *base,
                                                const Self<RUNS, OffT> &me, int lane,
                                                std::integer_sequence<int, Is...>) {
    // one direction at a time: the scheduler may not hoist the next
    // direction's scalar address work above this one, which keeps the
    // wave-uniform values of a few directions live instead of all 18
    ((v[Is] = gather_one<Is, REV, RUNS, S, OffT>(h, base, me, lane), __builtin_amdgcn_sched_barrier(0)), ...);
}

template <bool REV, bool RUNS, typename S, typename OffT>
__device__ __forceinline__ void gather_all(S (&v)[Q], const Nbhd<OffT> &h, const char *base, const Self<RUNS, OffT> &me,
                                           int lane) {
    gather_all_impl<REV, RUNS, S, OffT>(v, h, base, me, lane, std::make_integer_sequence<int, Q>{});
}

// ---------------------------------------------------------------------------
// writing a tile's values
// ---------------------------------------------------------------------------
// Every 128-byte line a tile writes is written whole, and lines that hold no
// fluid value are neither read nor written.
//   runs : fluid lanes write their 19 values; then lanes 0..pad-1 write zeros
//          after the run's 19*k values up to the next line boundary
//   plain: every lane of a line holding a fluid node writes, solid ones a zero
template <typename S>
__device__ __forceinline__ void store_stream(S *p, S v) {
    __builtin_nontemporal_store(v, p);
}

// non-temporal store (nt, bit 1) of a run's value
constexpr int BUFFER_NT = 2;
__device__ __forceinline__ void store_run(__amdgpu_buffer_rsrc_t run, int at, int dir, double v) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), run, at, dir, BUFFER_NT);
}
__device__ __forceinline__ void store_run(__amdgpu_buffer_rsrc_t run, int at, int dir, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), run, at, dir, BUFFER_NT);
}

template <typename S, bool RUNS, typename OffT, bool STREAM, bool ZERO_SOLID = false, class Value>
__device__ __forceinline__ void store_tile(char *lattice, const Self<RUNS, OffT> &me, uint64_t own, bool fl, int lane,
                                           Value value) {
    S *out = reinterpret_cast<S *>(lattice);
    constexpr int L = 128 / (int)sizeof(S);
    if constexpr (RUNS) {
        if (fl) {
            if constexpr (STREAM) {
                // a buffer at the tile's run: the lane's byte offset is one
                // register for all directions and a direction's distance a
                // scalar one, where a pointer per direction is added up on the
                // vector unit after the collision (256^3 pack, FP32: 219.1 ->
                // 217.3 us a step, FP64 within 0.1%)
                const auto run = __builtin_amdgcn_make_buffer_rsrc(out + me.base, 0, (int)(Q * TILE * sizeof(S)), 0x00027000);
                const int at = me.slot * (int)sizeof(S), step = me.k * (int)sizeof(S);
#pragma unroll
                for (int i = 0; i < Q; ++i) store_run(run, at, i * step, value(i));
            } else {
#pragma unroll
                for (int i = 0; i < Q; ++i) out[(me.base + (OffT)i * me.stride) + me.slot] = value(i);
            }
        }
        const int used = Q * me.k;
        const int pad = (used + L - 1) / L * L - used;
        if (lane < pad) {
            S *p = out + me.base + (OffT)(used + lane);
            if constexpr (STREAM) store_stream(p, S(0));
            else *p = S(0);
        }
    } else {
        uint64_t cover = 0;
        if constexpr (L >= 64) {
            cover = own ? ~0ull : 0ull;
        } else {
            constexpr uint64_t G = (1ull << L) - 1;
#pragma unroll
            for (int g = 0; g < 64 / L; ++g)
                if ((own >> (g * L)) & G) cover |= G << (g * L);
        }
        // value(i) is evaluated on every covered lane (callers keep the
        // values of solid lanes defined, and zero when they pass ZERO_SOLID)
        if (lane_on(cover)) {
            // the tile's first block is wave-uniform, the lane's byte offset
            // 32 bits, and the blocks follow at fixed distances
            char *tile0 = lattice + (size_t)me.base * sizeof(S);
            const uint32_t lane_off = (uint32_t)lane * (uint32_t)sizeof(S);
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                S *p = reinterpret_cast<S *>(tile0 + (i * TILE * (int)sizeof(S) + lane_off));
                S v = value(i);
                if constexpr (!ZERO_SOLID) v = fl ? v : S(0);
                if constexpr (STREAM) store_stream(p, v);
                else *p = v;
            }
        }
    }
}

// The same through LDS: a wave puts its tile's blocks side by side and writes
// them 16 bytes per lane and store.  What a step is short of is the vector
// memory path of its compute unit, which takes a cycle per 16 lanes and line
// of an access and holds some 64 lines to come: a direction at a time a tile's
// stores took about 95 cycles of it, this way 30 to 76 (256^3 pack, us a step:
// FP64 388.5 -> 373.1, FP32 217.8 -> 202.5, FP16 159.0 -> 158.2; 128^3 dense
// box FP16 35.3 -> 34.7; FP64 adjoint step on a 128^3 pack 100.5 -> 98.5).  The LDS round
// trip is in every wave's way, though, and on a grid that is in flight all at
// once nothing hides it: see stage_stores.
// Same bytes as store_tile's.  For the plain layout value(i) is evaluated on
// every lane and has to be zero on solid ones.
template <typename S>
constexpr int STAGE_BYTES = Q * TILE * (int)sizeof(S);  // of a wave
extern __shared__ __align__(16) unsigned char stage_lds[];

template <typename S, bool RUNS, typename OffT, class Value>
__device__ __forceinline__ void store_tile_staged(char *lattice, const Self<RUNS, OffT> &me, bool fl, int lane,
                                                  Value value) {
    typedef uint32_t Chunk __attribute__((ext_vector_type(4)));
    constexpr int L = 128 / (int)sizeof(S), MOST = (STAGE_BYTES<S> / 16 + 63) / 64;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    unsigned char *stage = stage_lds + wave * STAGE_BYTES<S>;
    S *out = reinterpret_cast<S *>(stage);
    int end = Q * TILE;  // values written
    if constexpr (RUNS) {
        if (fl) {
#pragma unroll
            for (int i = 0; i < Q; ++i) out[i * me.k + me.slot] = value(i);
        }
        const int used = Q * me.k;
        end = (used + L - 1) / L * L;
        if (lane < end - used) out[used + lane] = S(0);
    } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) out[i * TILE + lane] = value(i);
    }
    // no other wave touches this one's part, and its own accesses are in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int chunks = end * (int)sizeof(S) / 16;
    Chunk *to = reinterpret_cast<Chunk *>(lattice + (size_t)me.base * sizeof(S));
    const Chunk *from = reinterpret_cast<const Chunk *>(stage);
#pragma unroll
    for (int c = 0; c < MOST; ++c) {
        if (c * 64 >= chunks) break;
        const int e = c * 64 + lane;
        if (e < chunks) __builtin_nontemporal_store(from[e], to + e);
    }
}

// ---------------------------------------------------------------------------
// collision: LBGK (Eq. 2, 7) with the quasi-compressible (Eq. 3, 5) or
// incompressible (Eq. 4, 6) equilibrium and Guo forcing, on shifted values
// d_i = f_i - w_i rho_base:
//   drho = sum d, rho = rho_base + drho, j = sum c d,
//   u = (j + F/2)/rho (model 0) or j + F/2 (model 1),
//   deq_i = w_i (drho + rho P_i) (model 0) or w_i (drho + P_i) (model 1),
//   P_i = 3 c.u + 4.5 (c.u)^2 - 1.5 u.u,
//   d*_i = d_i + omega (deq_i - d_i) + kg w_i (3 (c_i - u).F + 9 (c_i.u)(c_i.F))
// ---------------------------------------------------------------------------
// With SC the values are held on a scale s = 2^k (D = s d, sc = s, isc =
// 1/s): the sums are brought back to unit scale for rho and u, and the
// equilibrium and source terms are put on the scale; every product with a
// power of two is exact.
template <typename T, int MODEL, bool SC = false>
__device__ __forceinline__ void collide(T (&d)[Q], T rho_base, T omega, T kg, T Fx, T Fy, T Fz, T sc = T(1),
                                        T isc = T(1)) {
    T drho = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        drho += d[i];
        if (CX[i]) jx += CX[i] > 0 ? d[i] : -d[i];
        if (CY[i]) jy += CY[i] > 0 ? d[i] : -d[i];
        if (CZ[i]) jz += CZ[i] > 0 ? d[i] : -d[i];
    }
    const T drho_s = drho;  // on the stored scale: feeds the equilibrium's drho term
    if constexpr (SC) {
        drho *= isc;
        jx *= isc;
        jy *= isc;
        jz *= isc;
        kg *= sc;
    }
    const T rho = rho_base + drho;
    T ux = jx + T(0.5) * Fx, uy = jy + T(0.5) * Fy, uz = jz + T(0.5) * Fz;
    if constexpr (MODEL == LBM_QUASI_COMPRESSIBLE) {
        const T ir = T(1) / rho;
        ux *= ir;
        uy *= ir;
        uz *= ir;
    }
    const T usq = T(1.5) * (ux * ux + uy * uy + uz * uz);
    const T uF3 = T(3) * (ux * Fx + uy * Fy + uz * Fz);
    const T om1 = T(1) - omega;
    // omega deq_i = A_w + B_w P_i with A_w = omega w drho and B_w = omega w rho
    // (model 0) or omega w (model 1); the source is G_w (3 c_i.F - uF3 +
    // 9 (c_i.u)(c_i.F)) with G_w = kg w.  Per weight class:
    T bscale = MODEL == LBM_QUASI_COMPRESSIBLE ? rho : T(1);
    if constexpr (SC) bscale *= sc;
    const T od = omega * drho_s, ob = omega * bscale;
    {
        const T w = T(weight(0));
        d[0] = om1 * d[0] + (w * od - (w * ob) * usq) - (kg * w) * uF3;
    }
    // Opposite directions share c.u and c.F up to sign, so they are updated
    // together: P = q +- 3 c.u with q = 4.5 (c.u)^2 - 1.5 u.u, and the source
    // splits into a shared part and +- 3 G c.F.
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int j = opposite(i);
        if (j < i) continue;
        const T w = T(weight(i));
        const T A = w * od, B = w * ob, G = kg * w;
        const T cu = T(CX[i]) * ux + T(CY[i]) * uy + T(CZ[i]) * uz;
        const T cF = T(CX[i]) * Fx + T(CY[i]) * Fy + T(CZ[i]) * Fz;
        const T q = T(4.5) * cu * cu - usq;
        const T t = T(3) * cu;
        const T sh = G * (T(9) * cu * cF - uF3) + A;
        const T f = (T(3) * G) * cF;
        d[i] = om1 * d[i] + ((sh + f) + B * (q + t));
        d[j] = om1 * d[j] + ((sh - f) + B * (q - t));
    }
}

// ---------------------------------------------------------------------------
// out = R v for the multiple-relaxation-time operator
// R = M^T diag(s_k / |row k|^2) M (the rows of M are orthogonal).  Each row is
// even or odd under c -> -c, so it reads either the rest value and the 9 sums
// v_i + v_opp(i) or the 9 differences v_i - v_opp(i), and the outputs of a
// pair share one even and one odd sum: out_i = E + O, out_opp(i) = E - O.
// About half the operations of the plain product (both triangular halves of
// the integer matrix are folded by the compiler either way).
// ---------------------------------------------------------------------------
// Every index below is a template argument, so no loop is left for the
// compiler to unroll (a loop it kept would index the value arrays at run
// time and move them to scratch memory); sums start from -0, the identity of
// addition, so the first term needs no add.
template <int K, int P, typename T>
__device__ __forceinline__ void mrt_row_term(T &acc, const T (&vs)[NPAIR], const T (&va)[NPAIR]) {
    constexpr int c = MRT.c[K][pair_first(P)];
    if constexpr (c != 0) acc += T(c) * (mrt_row_odd(K) ? va[P] : vs[P]);
}
template <int K, typename T, int... Ps>
__device__ __forceinline__ T mrt_moment(T omega, T v0, const T (&vs)[NPAIR], const T (&va)[NPAIR],
                                        std::integer_sequence<int, Ps...>) {
    if constexpr (mrt_rate(K) == 0.0) {
        return T(0);
    } else {
        T acc = T(-0.0);
        if constexpr (!mrt_row_odd(K) && MRT.c[K][0] != 0) acc += T(MRT.c[K][0]) * v0;
        (mrt_row_term<K, Ps, T>(acc, vs, va), ...);
        const T rate = mrt_rate(K) < 0.0 ? omega : T(mrt_rate(K));
        return acc * (rate * T(1.0 / MRT.n[K]));
    }
}
// the even (ODD = false) or odd part of column I of M^T applied to mu
template <int I, bool ODD, int K, typename T>
__device__ __forceinline__ void mrt_col_term(T &acc, const T (&mu)[Q]) {
    constexpr int c = MRT.c[K][I];
    if constexpr (mrt_rate(K) != 0.0 && c != 0 && mrt_row_odd(K) == ODD) acc += T(c) * mu[K];
}
template <int I, bool ODD, typename T, int... Ks>
__device__ __forceinline__ T mrt_column(const T (&mu)[Q], std::integer_sequence<int, Ks...>) {
    T acc = T(-0.0);
    (mrt_col_term<I, ODD, Ks, T>(acc, mu), ...);
    return acc;
}
template <int P, typename T>
__device__ __forceinline__ void mrt_pair_out(const T (&mu)[Q], T (&out)[Q]) {
    constexpr int i = pair_first(P), j = opposite(pair_first(P));
    const T E = mrt_column<i, false, T>(mu, std::make_integer_sequence<int, Q>{});
    const T O = mrt_column<i, true, T>(mu, std::make_integer_sequence<int, Q>{});
    out[i] = E + O;
    out[j] = E - O;
}
template <typename T, int... Ps, int... Ks>
__device__ __forceinline__ void mrt_relax_impl(const T (&v)[Q], T omega, T (&out)[Q], std::integer_sequence<int, Ps...>,
                                               std::integer_sequence<int, Ks...>) {
    T vs[NPAIR], va[NPAIR];
    ((vs[Ps] = v[pair_first(Ps)] + v[opposite(pair_first(Ps))], va[Ps] = v[pair_first(Ps)] - v[opposite(pair_first(Ps))]),
     ...);
    T mu[Q];
    ((mu[Ks] = mrt_moment<Ks, T>(omega, v[0], vs, va, std::make_integer_sequence<int, NPAIR>{})), ...);
    out[0] = mrt_column<0, false, T>(mu, std::make_integer_sequence<int, Q>{});
    (mrt_pair_out<Ps, T>(mu, out), ...);
}
template <typename T>
__device__ __forceinline__ void mrt_relax(const T (&v)[Q], T omega, T (&out)[Q]) {
    mrt_relax_impl<T>(v, omega, out, std::make_integer_sequence<int, NPAIR>{}, std::make_integer_sequence<int, Q>{});
}

// ---------------------------------------------------------------------------
// multiple relaxation times (the paper's LBMRT), on shifted values: with
// r_i = d_i - deq_i and the Guo source G_i = w_i (3 (c_i - u).F + 9 (c_i.u)(c_i.F)),
//   m* = m - S (m - m_eq) + (I - S/2) M G,  f* = M^-1 m*
// is, in distribution space,
//   d*_i = d_i + G_i - [M^-1 S M (r + G/2)]_i,
// and M^-1 = M^T diag(1/|row|^2) since the rows are orthogonal.  The
// conserved moments (rate 0) drop out: their part of r + G/2 is zero.
// ---------------------------------------------------------------------------
template <typename T, int INC, bool SC = false>
__device__ __forceinline__ void collide_mrt(T (&d)[Q], T rho_base, T omega, T Fx, T Fy, T Fz, T sc = T(1),
                                            T isc = T(1)) {
    T drho = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        drho += d[i];
        if (CX[i]) jx += CX[i] > 0 ? d[i] : -d[i];
        if (CY[i]) jy += CY[i] > 0 ? d[i] : -d[i];
        if (CZ[i]) jz += CZ[i] > 0 ? d[i] : -d[i];
    }
    const T drho_s = drho;  // on the stored scale (see collide)
    if constexpr (SC) {
        drho *= isc;
        jx *= isc;
        jy *= isc;
        jz *= isc;
    }
    const T rho = rho_base + drho;
    T ux = jx + T(0.5) * Fx, uy = jy + T(0.5) * Fy, uz = jz + T(0.5) * Fz;
    if constexpr (!INC) {
        const T ir = T(1) / rho;
        ux *= ir;
        uy *= ir;
        uz *= ir;
    }
    const T usq = T(1.5) * (ux * ux + uy * uy + uz * uz);
    const T uF3 = T(3) * (ux * Fx + uy * Fy + uz * Fz);
    T bscale = INC ? T(1) : rho;
    T ws = T(1);  // the source's weight factor on the stored scale
    if constexpr (SC) {
        bscale *= sc;
        ws = sc;
    }
    T v[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const T w = T(weight(i));
        const T cu = T(CX[i]) * ux + T(CY[i]) * uy + T(CZ[i]) * uz;
        const T cF = T(CX[i]) * Fx + T(CY[i]) * Fy + T(CZ[i]) * Fz;
        const T deq = w * (drho_s + bscale * (T(3) * cu + T(4.5) * cu * cu - usq));
        T src = w * (T(3) * cF - uF3 + T(9) * cu * cF);
        if constexpr (SC) src *= ws;
        v[i] = d[i] - deq + T(0.5) * src;
        d[i] += src;  // d_i + G_i; the relaxation is subtracted below
    }
    T rv[Q];
    mrt_relax<T>(v, omega, rv);
#pragma unroll
    for (int i = 0; i < Q; ++i) d[i] -= rv[i];
}

// ---------------------------------------------------------------------------
// open boundaries (the paper's Zou-He velocity inlet and constant-pressure
// outlet) on faces normal to an axis.  Each boundary node carries a code
// 1..12: axis a = (code-1)/4, r = (code-1)%4: r = 0 velocity node whose
// unknown populations have c_a = +1, 1 pressure node c_a = -1, 2 velocity
// c_a = -1, 3 pressure c_a = +1.  After the gather, the unknown populations
// are rebuilt from their opposites:
//   f_i = f_opp(i) + 6 w_i (c_i . J) - sum_{t != a} c_it N_t,
//   N_t = 1/2 sum_{c_a = 0} c_t f - J_t / 3   (tangential-momentum correction),
// with J = rho u - F/2 (velocity node: rho from the known populations and
// u_a) or J_a from the prescribed density and J_t = -F_t/2 (pressure node).
// On shifted values the rebuild is unchanged (opposite directions have equal
// weights); only the density sums add rho_base times the weights of their
// sets (2/3 for c_a = 0, 1/6 for either normal set, for every axis).
// Per tile the boundary buffer holds a mask of its boundary nodes and their
// 64 codes: [n_tiles][9] uint64.
// ---------------------------------------------------------------------------
constexpr int axis_c(int a, int i) { return a == 0 ? CX[i] : (a == 1 ? CY[i] : CZ[i]); }

// The rebuild at the nodes of one axis.  The axis is a template argument: with
// a run-time axis the velocity components are read from a table in memory, one
// load waited for after another (19 in a row at the end of a boundary tile's
// gather: 20.4 us a step of a 101 x 61 x 47 channel, FP64, against 17.6 us).
template <typename T, int INC, int A>
__device__ __forceinline__ void open_boundary_axis(T (&d)[Q], const Phys &P, int r, T Fx, T Fy, T Fz) {
    const bool velocity = (r == 0 || r == 2);
    const int n = (r == 0 || r == 3) ? 1 : -1;  // c_a of the unknown populations
    const bool up = n == 1;
    const T rb = T(P.rho_base);
    T s_tan = 0, s_known = 0, tx = 0, ty = 0, tz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        if (axis_c(A, i) == 0) {
            s_tan += d[i];
            tx += T(CX[i]) * d[i];
            ty += T(CY[i]) * d[i];
            tz += T(CZ[i]) * d[i];
        } else if (axis_c(A, i) == -1) {
            s_known += up ? d[i] : d[opposite(i)];
        }
    }
    s_tan += rb * T(2.0 / 3.0);
    s_known += rb * T(1.0 / 6.0);
    const T Fa = A == 0 ? Fx : (A == 1 ? Fy : Fz);
    T Jx, Jy, Jz;
    if (velocity) {
        const T ux = T(P.bc_u[0]), uy = T(P.bc_u[1]), uz = T(P.bc_u[2]);
        const T ua = A == 0 ? ux : (A == 1 ? uy : uz);
        const T rho = INC ? T(1) : (s_tan + T(2) * s_known - T(0.5) * T(n) * Fa) / (T(1) - T(n) * ua);
        Jx = rho * ux - T(0.5) * Fx;
        Jy = rho * uy - T(0.5) * Fy;
        Jz = rho * uz - T(0.5) * Fz;
    } else {
        const T Ja = T(n) * (T(P.bc_rho) - s_tan - T(2) * s_known);
        Jx = A == 0 ? Ja : -T(0.5) * Fx;
        Jy = A == 1 ? Ja : -T(0.5) * Fy;
        Jz = A == 2 ? Ja : -T(0.5) * Fz;
    }
    const T Nx = A == 0 ? T(0) : T(0.5) * tx - Jx * T(1.0 / 3.0);
    const T Ny = A == 1 ? T(0) : T(0.5) * ty - Jy * T(1.0 / 3.0);
    const T Nz = A == 2 ? T(0) : T(0.5) * tz - Jz * T(1.0 / 3.0);
    // the unknowns (c_a = n) from their opposites (c_a = -n), which are known;
    // i and j run over the pairs with c_a(i) = 1
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        if (axis_c(A, i) != 1) continue;
        const int j = opposite(i);
        const T cJ = T(CX[i]) * Jx + T(CY[i]) * Jy + T(CZ[i]) * Jz;
        const T di = d[i], dj = d[j];
        const T vi = dj + T(6.0 * weight(i)) * cJ - T(CX[i]) * Nx - T(CY[i]) * Ny - T(CZ[i]) * Nz;
        const T vj = di + T(6.0 * weight(i)) * -cJ - T(CX[j]) * Nx - T(CY[j]) * Ny - T(CZ[j]) * Nz;
        d[i] = up ? vi : di;
        d[j] = up ? dj : vj;
    }
}

// `any`: the tile's boundary nodes, `codes`: the codes of its 64 nodes
template <typename T, int INC>
__device__ __forceinline__ void open_boundary(T (&d)[Q], const Phys &P, uint64_t any, const uint8_t *codes, int lane,
                                              T Fx, T Fy, T Fz) {
    if (!any) return;  // no boundary node in this tile
    if (!lane_on(any)) return;
    const int code = (int)codes[lane];
    const int a = (code - 1) >> 2, r = (code - 1) & 3;
    if (a == 0) open_boundary_axis<T, INC, 0>(d, P, r, Fx, Fy, Fz);
    else if (a == 1) open_boundary_axis<T, INC, 1>(d, P, r, Fx, Fy, Fz);
    else open_boundary_axis<T, INC, 2>(d, P, r, Fx, Fy, Fz);
}

// the collision of a model: LBGK (0, 1) or multiple relaxation times (2, 3)
template <typename T, int MODEL, bool SC = false>
__device__ __forceinline__ void collide_model(T (&d)[Q], T rho_base, T omega, T kg, T Fx, T Fy, T Fz, T sc = T(1),
                                              T isc = T(1)) {
    if constexpr (MODEL >= LBM_MRT_QUASI_COMPRESSIBLE)
        collide_mrt<T, (MODEL & 1), SC>(d, rho_base, omega, Fx, Fy, Fz, sc, isc);
    else
        collide<T, MODEL, SC>(d, rho_base, omega, kg, Fx, Fy, Fz, sc, isc);
}

struct KArgs {
    const char *src;
    char *dst;
    DevTables tb;
    int n_tiles;
    int lw;       // log2 of the waves (tiles) per workgroup
    int nblocks;  // workgroups in the grid
    Phys P;
};

// where a fluid node's entries of a per-node field live: component c at
// fbase[t] + c * k + slot, slot = the node's rank among the tile's fluid nodes
struct FieldSlot {
    uint64_t base;  // entry offset of the tile's field run (wave-uniform)
    int k;          // fluid nodes of the tile
    int slot;
    __device__ __forceinline__ FieldSlot(const DevTables &tb, int t, uint64_t mask) : FieldSlot(tb.fbase[t], mask) {}
    __device__ __forceinline__ FieldSlot(uint64_t first, uint64_t mask) {
        base = first;
        k = __builtin_popcountll(mask);
        slot = mbcnt(mask);
    }
    __device__ __forceinline__ uint64_t entry(int c) const { return base + (uint64_t)(c * k + slot); }
};

// a pointer read from memory is taken as one that may point to LDS unless its
// type says global
template <typename T>
using GlobalConst = const __attribute__((address_space(1))) T *;

// the per-node force field, one entry per fluid slot and component
template <typename T>
__device__ __forceinline__ void load_force(double F0, double F1, double F2, const void *field, uint64_t first,
                                           uint64_t mask, T &Fx, T &Fy, T &Fz) {
    Fx = T(F0);
    Fy = T(F1);
    Fz = T(F2);
    if (field) {
        const FieldSlot fs(first, mask);
        const GlobalConst<T> f = (GlobalConst<T>)reinterpret_cast<const T *>(field);
        Fx = f[fs.entry(0)];
        Fy = f[fs.entry(1)];
        Fz = f[fs.entry(2)];
    }
}

template <typename T>
__device__ __forceinline__ void load_force(const Phys &P, uint64_t first, uint64_t mask, T &Fx, T &Fy, T &Fz) {
    load_force<T>(P.F[0], P.F[1], P.F[2], P.field, first, mask, Fx, Fy, Fz);
}

// ---------------------------------------------------------------------------
// the fused step (Alg. 2): gather with bounce-back, collide, store
// ---------------------------------------------------------------------------
// The physics of a step, a kernel's last argument, OFF bytes into its
// arguments, read where this is called: after the gather's loads are issued and
// before the first of them is waited for.  Left to itself the compiler reads
// the arguments on entry, where they wait in scalar registers through the
// gather, which has none to spare, or where they are used, which puts a read
// of the argument buffer after the gather.
template <int OFF>
struct StepPhys {
    typedef const __attribute__((address_space(4))) char *ConstPtr;
    typedef uint32_t u32x4s __attribute__((ext_vector_type(4), aligned(4)));
    ConstPtr at;
    u32x16 v;  // Phys bytes 0..63
    u32x4s w;  // and 64..79
    __device__ __forceinline__ StepPhys() {
        at = (ConstPtr)__builtin_amdgcn_kernarg_segment_ptr() + OFF;
        asm volatile("" : "+s"(at));
        v = *(const __attribute__((address_space(4))) u32x16 *)at;
        w = *(const __attribute__((address_space(4))) u32x4s *)(at + 64);
        asm volatile("" : "+s"(v), "+s"(w));
    }
    __device__ __forceinline__ double f64(int byte) const {
        return __builtin_bit_cast(double, v[byte / 4] | (uint64_t)v[byte / 4 + 1] << 32);
    }
    __device__ __forceinline__ double omega() const { return f64(offsetof(Phys, omega)); }
    __device__ __forceinline__ double kg() const { return f64(offsetof(Phys, kg)); }
    __device__ __forceinline__ double rho_base() const { return f64(offsetof(Phys, rho_base)); }
    __device__ __forceinline__ double F(int c) const { return f64(offsetof(Phys, F) + 8 * c); }
    __device__ __forceinline__ const void *field() const {
        static_assert(offsetof(Phys, F) + 24 <= 64 && offsetof(Phys, field) == 64 && offsetof(Phys, scale) == 72 &&
                          offsetof(Phys, inv_scale) == 76,
                      "the fields a step reads");
        return (const void *)(w[0] | (uint64_t)w[1] << 32);
    }
    // by way of a scalar: a bit cast of a vector's element reads element 0
    __device__ __forceinline__ float f32(int i) const {
        const uint32_t bits = w[i];
        return __builtin_bit_cast(float, bits);
    }
    __device__ __forceinline__ float scale() const { return f32(2); }
    __device__ __forceinline__ float inv_scale() const { return f32(3); }
    __device__ __forceinline__ const Phys &all() const { return *(const Phys *)at; }
};
// where it lies: after row, src, dst, n_tiles, lw, nblocks, counter (and the
// boundary buffer), which is checked against the kernels' signatures below
constexpr int HOT_BYTES = 3 * 8 + 4 * 4;
constexpr int LW_MASK = 15, STOCHASTIC = 16;  // lw and a flag beside it in a step's shape argument
// the byte at which the last argument of a kernel lies
template <typename... A>
constexpr int last_argument(void (*)(A...)) {
    int at = 0, end = 0;
    ((at = (end + (int)alignof(A) - 1) / (int)alignof(A) * (int)alignof(A), end = at + (int)sizeof(A)), ...);
    return at;
}

template <int ST, int MODEL, typename OffT, bool OPEN, bool STAGED>
__device__ __forceinline__ void step_tile(const NbRow *row, const char *src, char *dst, int n_tiles,
                                          int shape, int nblocks, uint32_t counter, const uint64_t *bc) {
    using C = Codec<ST>;
    using S = typename C::S;
    using T = typename C::T;
    constexpr bool RN = C::RUNS;
    const int tw = wave_tile<!RN>(shape & LW_MASK, nblocks);
    if (tw >= n_tiles) return;
    // consecutive launches walk the tiles in opposite directions, so a step
    // starts on the tiles the previous one wrote last (FP16 166.7 -> 164.6 us
    // on a 256^3 sphere pack, FP64 389.2 -> 388.5 us, FP32 unchanged); the
    // order of the tiles within a step does not change any result
    const int t = (counter & 1u) ? n_tiles - 1 - tw : tw;
    const int lane = (int)(threadIdx.x & 63);
    uint64_t any = 0;  // the tile's boundary nodes
    if constexpr (OPEN) any = bc[9 * (size_t)t];
    const RowRegs r(row, t);
    Nbhd<OffT> h;
    load_nbhd<S>(h, r);
    const uint64_t fbase = r.fbase();
    // the tile's position keys the stochastic rounding
    uint32_t cx = 0, cy = 0, cz = 0;
    if constexpr (ST == LBM_F16S) {
        cx = r.xyz(0);
        cy = r.xyz(1);
        cz = r.xyz(2);
    }
    const uint64_t own = h.m[OWN];
    const bool fl = lane_on(own);
    const Self<RN, OffT> me(h, lane);
    T d[Q];
    if constexpr (!RN) {
        // solid lanes of the plain layout store zeros: encode 0 (exact in
        // every rounding) rather than branch around the encoding
#pragma unroll
        for (int i = 0; i < Q; ++i) d[i] = T(0);
    }
    if (fl) {  // solid nodes neither gather nor collide
        S raw[Q];
        gather_all<false, RN, S, OffT>(raw, h, src, me, lane);
        const StepPhys<HOT_BYTES + (OPEN ? 8 : 0)> P;
        const uint8_t *codes = OPEN ? reinterpret_cast<const uint8_t *>(bc + 9 * (size_t)t + 1) : nullptr;
        T Fx, Fy, Fz;
        load_force<T>(P.F(0), P.F(1), P.F(2), P.field(), fbase, own, Fx, Fy, Fz);
        if constexpr (C::SCALED) {
#pragma unroll
            for (int i = 0; i < Q; ++i) d[i] = C::dec_scaled(raw[i]);
            if constexpr (OPEN) {  // the rebuild works at unit scale (exact round trip)
#pragma unroll
                for (int i = 0; i < Q; ++i) d[i] *= P.inv_scale();
                open_boundary<T, (MODEL & 1)>(d, P.all(), any, codes, lane, Fx, Fy, Fz);
#pragma unroll
                for (int i = 0; i < Q; ++i) d[i] *= P.scale();
            }
            collide_model<T, MODEL, true>(d, T(P.rho_base()), T(P.omega()), T(P.kg()), Fx, Fy, Fz, T(P.scale()),
                                          T(P.inv_scale()));
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i) d[i] = C::dec(raw[i], 1.0f);
            if constexpr (OPEN) open_boundary<T, (MODEL & 1)>(d, P.all(), any, codes, lane, Fx, Fy, Fz);
            collide_model<T, MODEL>(d, T(P.rho_base()), T(P.omega()), T(P.kg()), Fx, Fy, Fz);
        }
    }
    const auto store = [&](auto value) {
        if constexpr (STAGED) store_tile_staged<S, RN, OffT>(dst, me, fl, lane, value);
        else store_tile<S, RN, OffT, true, !RN>(dst, me, own, fl, lane, value);
    };
    if constexpr (ST == LBM_F16S) {
        if (shape & STOCHASTIC) {
            // keyed on the node's position, not on where the tile is stored
            const uint32_t tile_seed = hash32(cx + hash32(cy + hash32(cz + hash32(counter))));
            const uint32_t seed = hash32(tile_seed + (uint32_t)lane);
            typename C::Pair pair = {};
            store([&](int i) { return C::enc_sr_scaled(d[i], seed + (uint32_t)i * 0x9E3779B9u, pair); });
            return;
        }
        store([&](int i) { return C::enc_scaled(d[i]); });
    } else {
        store([&](int i) { return C::enc(d[i], 1.0f); });
    }
}

// Open boundaries have kernels of their own: in one kernel their parameters
// and lane masks took scalar registers from every other step (12-16 spilled to
// vector lanes, 6 without them).  So have steps that do not stage their
// stores: a branch between the two ways at the end of one kernel cost 1-2%
// either way.
#define STEP_KERNEL(NAME, OPEN, STAGED, BC_PARAM, BC)                                                              \
    template <int ST, int MODEL, typename OffT>                                                                    \
    __global__ __launch_bounds__(512) void NAME(const NbRow *row, const char *src,                                 \
                                                char *dst, int n_tiles, int shape, int nblocks, uint32_t counter,  \
                                                BC_PARAM Phys P) {                                                 \
        step_tile<ST, MODEL, OffT, OPEN, STAGED>(row, src, dst, n_tiles, shape, nblocks, counter, BC);             \
    }
#define STEP_BC const uint64_t *bc,
STEP_KERNEL(k_step, false, true, , nullptr)
STEP_KERNEL(k_step_direct, false, false, , nullptr)
STEP_KERNEL(k_step_open, true, true, STEP_BC, bc)
STEP_KERNEL(k_step_open_direct, true, false, STEP_BC, bc)
static_assert(last_argument(k_step<LBM_F64, LBM_QUASI_COMPRESSIBLE, uint32_t>) == HOT_BYTES &&
                  last_argument(k_step_direct<LBM_F64, LBM_QUASI_COMPRESSIBLE, uint32_t>) == HOT_BYTES &&
                  last_argument(k_step_open<LBM_F64, LBM_QUASI_COMPRESSIBLE, uint32_t>) == HOT_BYTES + 8 &&
                  last_argument(k_step_open_direct<LBM_F64, LBM_QUASI_COMPRESSIBLE, uint32_t>) == HOT_BYTES + 8,
              "StepPhys reads the physics where the signature puts it");

// the paper's measurement kernels (Section 4.1): kind 1 "read/write only",
// kind 2 "propagation only"
template <typename S, bool RN, int KIND, typename OffT, bool STAGED>
__global__ __launch_bounds__(512) void k_calib(const NbRow *row, const char *src, char *dst, int n_tiles,
                                               int lw, int nblocks, const TileRec *rec) {
    const int t = wave_tile<!RN>(lw, nblocks);
    if (t >= n_tiles) return;
    const int lane = (int)(threadIdx.x & 63);
    Nbhd<OffT> h;
    if constexpr (KIND == 1) {  // no neighbours: the tile's record alone
        h.m[OWN] = rec[t].mask;
        h.base[OWN] = (OffT)rec[t].base;
    } else {
        load_nbhd<S>(h, RowRegs(row, t));
    }
    const uint64_t own = h.m[OWN];
    const bool fl = lane_on(own);
    const Self<RN, OffT> me(h, lane);
    S v[Q];
    if constexpr (!RN) {
        // whole-block stores write the solid lanes too: zeros, as the step does
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = S(0);
    }
    if (fl) {
        if constexpr (KIND == 1) {
#pragma unroll
            for (int i = 0; i < Q; ++i) v[i] = load_elem<OffT, S>(src, me.elem(i));
        } else {
            gather_all<false, RN, S, OffT>(v, h, src, me, lane);
        }
    }
    const auto value = [&](int i) { return v[i]; };  // as a step stores
    if constexpr (STAGED) store_tile_staged<S, RN, OffT>(dst, me, fl, lane, value);
    else store_tile<S, RN, OffT, true>(dst, me, own, fl, lane, value);
}

// The paper's intra-tile layout study (Section 3.3, Eqs. 11-13; Table 5):
// the propagation-only kernel on the plain layout, with the slot of node
// (x, y, z) in direction i's 64-slot block given per direction by
//   XYZ      x + 4y + 16z                                  (default)
//   YXZ      y + 4x + 16z        for E, W, ET, EB, NW, SW, WT, WB  (LS bit 0)
//   zigzagNE 2(x + 3y + [x = 3](3 - y)·4) + (z & 1) + 16(z & 2)
//                                for NE, SE                        (LS bit 1)
// LS = 4 is not the paper's: a face-major order for 128-byte lines, where the
// face a neighbour reads is one contiguous run of 16 nodes: x slowest
// (y + 4z + 16x) for E and W, y slowest (x + 4z + 16y) for N, S and the four
// xy edge directions, XYZ (z slowest already) for the rest.
// Only defined on tiles that are entirely fluid (the host checks), where the
// plain and the runs layouts occupy the same bytes.
__device__ __forceinline__ int layout_slot(int ls, int i, int x, int y, int z) {
    if (ls == 4) {
        if (i == 1 || i == 3) return y + 4 * z + 16 * x;
        if (i == 2 || i == 4 || (i >= 7 && i <= 10)) return x + 4 * z + 16 * y;
        return x + 4 * y + 16 * z;
    }
    const bool yxz = (ls & 1) && (i == 1 || i == 3 || i == 8 || i == 9 || i == 11 || i == 12 || i == 13 || i == 14);
    const bool zig = (ls & 2) && (i == 7 || i == 10);
    if (yxz) return y + 4 * x + 16 * z;
    if (zig) return 2 * (x + 3 * y + ((x + 1) & 4) * (3 - y)) + (z & 1) + 16 * (z & 2);
    return x + 4 * y + 16 * z;
}

template <int LS, int I, typename S, typename OffT>
__device__ __forceinline__ S gather_layout(const Nbhd<OffT> &h, const char *base, const Self<false, OffT> &me, int x,
                                           int y, int z, int lane) {
    if constexpr (I == 0) {
        return load_elem<OffT, S>(base, me.base + (OffT)layout_slot(LS, 0, x, y, z));
    } else {
        constexpr int SX = -CX[I], SY = -CY[I], SZ = -CZ[I], OP = opposite(I);
        const uint64_t ok = source_fluid<SX, SY, SZ>(h);
        const int xs = (x + SX) & 3, ys = (y + SY) & 3, zs = (z + SZ) & 3;
        // source_elem addresses slot xs + 4ys + 16zs of the source tile's block
        const OffT e = source_elem<SX, SY, SZ, I, false, OffT>(h, lane) - (OffT)(xs + 4 * ys + 16 * zs) +
                       (OffT)layout_slot(LS, I, xs, ys, zs);
        const OffT bb = me.base + (OffT)(OP * TILE + layout_slot(LS, OP, x, y, z));
        return load_elem<OffT, S>(base, lane_on(ok) ? e : bb);
    }
}

template <int LS, typename S, typename OffT, int... Is>
__device__ __forceinline__ void gather_layout_all(S (&v)[Q], const Nbhd<OffT> &h, const char *base,
                                                  const Self<false, OffT> &me, int x, int y, int z, int lane,
                                                  std::integer_sequence<int, Is...>) {
    ((v[Is] = gather_layout<LS, Is, S, OffT>(h, base, me, x, y, z, lane), __builtin_amdgcn_sched_barrier(0)), ...);
}

template <typename S, int LS, typename OffT>
__global__ __launch_bounds__(512) void k_calib_layout(const NbRow *row, const char *src, char *dst, int n_tiles,
                                               int lw, int nblocks) {
    const int t = wave_tile(lw, nblocks);
    if (t >= n_tiles) return;
    const int lane = (int)(threadIdx.x & 63);
    const int x = lane & 3, y = (lane >> 2) & 3, z = lane >> 4;
    Nbhd<OffT> h;
    load_nbhd<S>(h, RowRegs(row, t));
    const Self<false, OffT> me(h, lane);
    S v[Q];
    gather_layout_all<LS, S, OffT>(v, h, src, me, x, y, z, lane, std::make_integer_sequence<int, Q>{});
    S *out = reinterpret_cast<S *>(dst);
#pragma unroll
    for (int i = 0; i < Q; ++i) store_stream(out + (me.base + (OffT)(i * TILE + layout_slot(LS, i, x, y, z))), v[i]);
}

// ---------------------------------------------------------------------------
// initial state: feq(rho0, u0) at every fluid node of both lattices, 0 in the
// padding
// ---------------------------------------------------------------------------
template <int ST>
__global__ __launch_bounds__(512) void k_init(KArgs a, char *b, double ux, double uy, double uz) {
    using C = Codec<ST>;
    using S = typename C::S;
    const int t = wave_tile(a.lw, a.nblocks);
    if (t >= a.n_tiles) return;
    const int lane = (int)(threadIdx.x & 63);
    const TileRec rec = a.tb.rec[t];
    const bool fl = (rec.mask >> lane) & 1;
    const Self<C::RUNS, uint64_t> me(rec, lane);
    const double rho = a.P.rho0;
    const double usq = 1.5 * (ux * ux + uy * uy + uz * uz);
    auto feq = [&](int i) {
        const double cu = CX[i] * ux + CY[i] * uy + CZ[i] * uz;
        const double P = 3.0 * cu + 4.5 * cu * cu - usq;
        const double f = (a.P.model & 1) ? weight(i) * (rho + P) : weight(i) * rho * (1.0 + P);
        return C::enc((typename C::T)(f - weight(i) * a.P.rho_base), a.P.scale);
    };
    if constexpr (C::RUNS) {
        store_tile<S, true, uint64_t, false>(a.dst, me, rec.mask, fl, lane, feq);
        store_tile<S, true, uint64_t, false>(b, me, rec.mask, fl, lane, feq);
    } else {  // every slot of the 19 blocks, so solid slots start at 0 too
        S *pa = reinterpret_cast<S *>(a.dst), *pb = reinterpret_cast<S *>(b);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const S v = fl ? feq(i) : S(0);
            pa[me.elem(i)] = v;
            pb[me.elem(i)] = v;
        }
    }
}

__global__ void k_fill(double *p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.0;
}

__device__ __forceinline__ size_t dense_index(const int *xyz, int lane, int nx, int ny) {
    const int x = xyz[0] + (lane & 3), y = xyz[1] + ((lane >> 2) & 3), z = xyz[2] + (lane >> 4);
    return (size_t)x + (size_t)nx * ((size_t)y + (size_t)ny * (size_t)z);
}

// deterministic wave-wide sum / max (fixed butterfly)
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// ---------------------------------------------------------------------------
// a dense box, walked by rows of 16 nodes along x
// ---------------------------------------------------------------------------
// One workgroup of 4 waves takes a group of 4 tiles side by side along x, wave w
// their z-plane w: lane l is node (l & 15, l >> 4) of the 16 x 4 nodes of that plane,
// in tile l >> 2 & 3.  A store of a dense FP64 array is then 4 whole 128-byte
// lines (a wave on its own tile writes 16 pieces of 32 bytes), the nodes of
// tiles that were dropped are written too, so no pass over the array clears it
// first, and a read of a lattice block is the 16 consecutive slots of each of
// the 4 tiles' planes.
// In a box of one tile along x the group is 4 tiles along y, whose planes are 64
// consecutive nodes: lane l is node (l & 3, l >> 2), in tile l >> 4.
struct DenseBox {
    const int32_t *map;  // [tz][ty][tx] device tile number, -1 for a dropped tile
    int tx, ty, gx;      // tiles along the group's axis and (along x) the next one, groups along the axis
    int nx, ny, nz;
    bool along_y;
    // tile of the group, and y in it or (along y) in the group, of a lane of a plane
    __device__ __forceinline__ int tile_of(int lane) const { return lane >> (along_y ? 4 : 2) & 3; }
    __device__ __forceinline__ int y_of(int lane) const { return lane >> (along_y ? 2 : 4); }
    // the node of plane z of group (gx, row), and whether the box has it
    struct At {
        size_t at;
        bool in;
    };
    __device__ __forceinline__ At node(int gx, int row, int lane, int z) const {
        const int tz = row / ty, t = row - tz * ty;
        const int X = along_y ? lane & 3 : 16 * gx + (lane & 15), Y = (along_y ? 16 * gx : 4 * t) + y_of(lane);
        const int Z = 4 * tz + z;
        return At{(size_t)X + (size_t)nx * ((size_t)Y + (size_t)ny * (size_t)Z), X < nx && Y < ny && Z < nz};
    }
};

struct DenseNode {
    bool in, fl;    // inside the box; a fluid node of a kept tile
    int tile;       // device tile number, or -1
    int n;          // node in the tile
    int rank, k;    // the node's rank among the tile's k fluid nodes
    uint64_t base;  // element offset of the tile's data
    size_t at;      // index in a dense array
    template <bool RUNS>
    __device__ __forceinline__ uint64_t elem(int i) const {
        return base + (uint64_t)(RUNS ? i * k + rank : i * TILE + n);
    }
    __device__ __forceinline__ uint64_t field_entry(uint64_t first, int c) const {
        return first + (uint64_t)(c * k + rank);
    }
};

// The groups of 4 tiles blockIdx.x, blockIdx.x + gridDim.x, ...  A node's
// loads need its tile's record and that the tile's number: both are loaded
// ahead, the record one group and the number two, so a group waits for its
// lattice loads alone.
// Each XCD takes chunks of 16 groups, 256 nodes along x, so that it writes
// whole rows (256^3 pack, fields and sums: 378 us a call, 382 without the
// re-numbering, 387 with chunks of 64).
constexpr int DENSE_LC = 4;
constexpr int WALK_LW = 2;  // 4 waves in a workgroup
struct DenseWalk {
    const DevTables &tb;
    const DenseBox &b;
    const int groups;
    int g, tile1;
    int tile0;
    TileRec rec0;
    __device__ __forceinline__ DenseWalk(const DevTables &tb_, const DenseBox &b_, int groups_)
        : tb(tb_), b(b_), groups(groups_), g((int)blockIdx.x) {
        tile0 = lookup(g);
        tile1 = lookup(g + (int)gridDim.x);
        rec0 = record(tile0);
    }
    __device__ __forceinline__ bool more() const { return g < groups; }
    __device__ __forceinline__ int lookup(int i) const {
        if (i >= groups) return -1;
        const int gr = remap_block(i, groups, DENSE_LC);
        const int row = gr / b.gx, tx = 4 * (gr - row * b.gx) + b.tile_of((int)(threadIdx.x & 63));
        return tx < b.tx ? b.map[(size_t)row * b.tx + tx] : -1;
    }
    __device__ __forceinline__ TileRec record(int t) const { return t >= 0 ? tb.rec[t] : TileRec{0, 0}; }
    // the node of this thread in the present group; moves on to the next one
    __device__ __forceinline__ DenseNode next() {
        DenseNode d;
        const int lane = (int)(threadIdx.x & 63), z = (int)(threadIdx.x >> 6);
        const int gr = remap_block(g, groups, DENSE_LC);
        const int row = gr / b.gx, gx = gr - row * b.gx;
        const DenseBox::At at = b.node(gx, row, lane, z);
        d.in = at.in;
        d.at = at.at;
        d.n = (lane & 3) + 4 * (b.y_of(lane) & 3) + 16 * z;
        d.tile = tile0;
        d.base = rec0.base;
        d.fl = (rec0.mask >> d.n) & 1;
        d.k = __builtin_popcountll(rec0.mask);
        d.rank = __builtin_popcountll(rec0.mask & ((1ull << d.n) - 1ull));
        tile0 = tile1;
        rec0 = record(tile1);
        tile1 = lookup(g + 2 * (int)gridDim.x);
        g += (int)gridDim.x;
        return d;
    }
};

// The kept tiles alone, one for each wave, for an array that has been cleared:
// nodes that are not fluid count as outside.
struct TileWalk {
    const DevTables &tb;
    const DenseBox &b;
    const int n_tiles;
    int t;
    __device__ __forceinline__ TileWalk(const DevTables &tb_, const DenseBox &b_, int n_tiles_)
        : tb(tb_), b(b_), n_tiles(n_tiles_), t(wave_tile(WALK_LW, (int)gridDim.x)) {}
    __device__ __forceinline__ bool more() const { return t < n_tiles; }
    __device__ __forceinline__ DenseNode next() {
        const int lane = (int)(threadIdx.x & 63);
        const TileRec rec = tb.rec[t];
        DenseNode d;
        d.in = d.fl = (rec.mask >> lane) & 1;
        d.tile = t;
        d.n = lane;
        d.base = rec.base;
        d.k = __builtin_popcountll(rec.mask);
        d.rank = mbcnt(rec.mask);
        d.at = dense_index(tb.xyz + 4 * (size_t)t, lane, b.nx, b.ny);
        t = n_tiles;
        return d;
    }
};

// ---------------------------------------------------------------------------
// macroscopic fields of a stored post-collision lattice and their sums:
// rho = sum f*, u = (sum c f* - F/2)/rho
// ---------------------------------------------------------------------------
// A lane keeps the 8 sums of the nodes it visits and its workgroup reduces
// them once at the end: a butterfly per tile (96 cross-lane moves, through the
// LDS pipe) took longer than reading the tile.  Every workgroup leaves one row
// of partial sums; the work and the order of every addition follow from the
// tiles and the box alone, so the sums are bitwise reproducible.
// A lane adds up one node after another, where a butterfly per tile adds them
// in pairs: what each addition rounds off is kept beside the sum and added at
// the end, so the longer chain costs no accuracy.

// s + c += x, with c what the additions to s have rounded off so far (the
// two-term sum of D. E. Knuth, TAOCP vol. 2, 4.2.2)
__device__ __forceinline__ void add_kept(double &s, double &c, double x) {
    const double t = s + x, b = t - s;
    c += (s - (t - b)) + (x - b);
    s = t;
}
// a sum that has overflowed or met a NaN is what plain additions make of it
__device__ __forceinline__ double kept_total(double s, double c) { return isfinite(s) ? s + c : s; }

struct MacroSums {
    double v[NSUM], kept[NSUM];  // kept: of the five sums that round
    __device__ __forceinline__ MacroSums() {
#pragma unroll
        for (int c = 0; c < NSUM; ++c) v[c] = kept[c] = 0.0;
    }
    __device__ __forceinline__ void add(double rho, double ux, double uy, double uz) {
        const bool finite = isfinite(rho) && isfinite(ux) && isfinite(uy) && isfinite(uz);
        add_kept(v[0], kept[0], rho);
        add_kept(v[1], kept[1], rho * ux);
        add_kept(v[2], kept[2], rho * uy);
        add_kept(v[3], kept[3], rho * uz);
        v[4] += 1.0;
        if (finite) v[5] = fmax(v[5], sqrt(ux * ux + uy * uy + uz * uz));
        else v[6] += 1.0;
        add_kept(v[7], kept[7], ux);
    }
    // by all threads of a workgroup of MACRO_THREADS, into its row of partials
    __device__ __forceinline__ void store(double *partials);
};
constexpr int MACRO_THREADS = 256;
__device__ __forceinline__ void MacroSums::store(double *partials) {
    __shared__ double sh[MACRO_THREADS / 64][NSUM];
    const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
#pragma unroll
    for (int c = 0; c < NSUM; ++c) {
        const double r = c == 5 ? wave_max(v[c]) : wave_sum(kept_total(v[c], kept[c]));
        if (lane == 0) sh[wave][c] = r;
    }
    __syncthreads();
    if (threadIdx.x < NSUM) {
        const int c = (int)threadIdx.x;
        double r = sh[0][c];
        for (int w = 1; w < MACRO_THREADS / 64; ++w) r = c == 5 ? fmax(r, sh[w][c]) : r + sh[w][c];
        partials[(size_t)blockIdx.x * NSUM + c] = r;
    }
}

// rho and the velocity of one fluid node; load(i) is its stored value i
template <class Load>
__device__ __forceinline__ void macro_node(const Phys &P, double Fx, double Fy, double Fz, Load load, double &rho,
                                           double &ux, double &uy, double &uz) {
    double drho = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const double v = load(i);
        drho += v;
        jx += CX[i] * v;
        jy += CY[i] * v;
        jz += CZ[i] * v;
    }
    rho = P.rho_base + drho;
    ux = jx - 0.5 * Fx;
    uy = jy - 0.5 * Fy;
    uz = jz - 0.5 * Fz;
    if (!(P.model & 1)) {  // quasi-compressible velocity (either operator)
        ux = ux / rho;
        uy = uy / rho;
        uz = uz / rho;
    }
}

// rho and the velocity of this lane's node of a tile that holds it
template <int ST>
__device__ __forceinline__ void macro_of_tile(const KArgs &a, int t, const TileRec &rec, int lane, double &rho,
                                              double &ux, double &uy, double &uz) {
    using C = Codec<ST>;
    using S = typename C::S;
    using T = typename C::T;
    const Self<C::RUNS, uint64_t> me(rec, lane);
    S raw[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) raw[i] = load_elem<uint64_t, S>(a.src, me.elem(i));
    T Fx, Fy, Fz;
    load_force<T>(a.P, a.P.field ? a.tb.fbase[t] : 0, rec.mask, Fx, Fy, Fz);
    macro_node(a.P, (double)Fx, (double)Fy, (double)Fz,
               [&](int i) { return (double)C::dec(raw[i], a.P.inv_scale); }, rho, ux, uy, uz);
}

// tile after tile, for boxes of mostly dropped tiles: the sums, and the
// fluid nodes of the fields asked for
template <int ST>
__global__ __launch_bounds__(MACRO_THREADS) void k_sums(KArgs a, int nx, int ny, int nz, double *rho_out,
                                                        double *u_out, double *partials) {
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int waves = (int)gridDim.x * (MACRO_THREADS / 64);
    const size_t N = (size_t)nx * ny * nz;
    MacroSums sums;
    int t = (int)blockIdx.x * (MACRO_THREADS / 64) + wave;
    TileRec ahead = t < a.n_tiles ? a.tb.rec[t] : TileRec{0, 0};
    for (; t < a.n_tiles; t += waves) {
        const TileRec rec = ahead;
        ahead = t + waves < a.n_tiles ? a.tb.rec[t + waves] : TileRec{0, 0};
        if (!((rec.mask >> lane) & 1)) continue;
        double rho, ux, uy, uz;
        macro_of_tile<ST>(a, t, rec, lane, rho, ux, uy, uz);
        sums.add(rho, ux, uy, uz);
        if (rho_out || u_out) {
            const size_t at = dense_index(a.tb.xyz + 4 * (size_t)t, lane, nx, ny);
            if (rho_out) rho_out[at] = rho;
            if (u_out) {
                u_out[at] = ux;
                u_out[N + at] = uy;
                u_out[2 * N + at] = uz;
            }
        }
    }
    sums.store(partials);
}

// tables that are read through the scalar unit in a loop that stores: a vector
// load would be waited for with every store issued before it
template <typename T>
using Uniform = const __attribute__((address_space(4))) T *;

// A walk of the box, wave w on tile w of a group, lane n on its node n: the
// sums, and with FIELDS the fields asked for.  These pass
// through LDS into rows of 16 nodes along x, which makes a store of a wave 4
// whole lines; the loads are a tile's whole blocks, and the sums are the same
// additions in the same order whether the fields are written or not.  Bound by
// memory, with a group's latencies covered by 8 workgroups per CU (256^3 pack,
// FP64 / FP32 / FP16, us a call: fields 350 / 250 / 229, where lanes laid along
// the rows for the loads as well took 373 / 271 / 260; sums alone 219 / 134 /
// 128, of which the groups' dropped tiles take 10 / 13 / 29).
template <int ST, bool FIELDS>
__global__ __launch_bounds__(MACRO_THREADS) void k_fields(KArgs a, DenseBox b, int groups, double *rho_out,
                                                          double *u_out, double *partials) {
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const size_t N = (size_t)b.nx * b.ny * b.nz;
    __shared__ double rows[FIELDS ? 2 : 1][4][FIELDS ? MACRO_THREADS : 1];
    int buf = 0;
    MacroSums sums;
    const Uniform<int32_t> map = (Uniform<int32_t>)b.map;
    const Uniform<TileRec> recs = (Uniform<TileRec>)a.tb.rec;
    // the wave's tile of group i, or -1
    const auto lookup = [&](int i) {
        if (i >= groups) return -1;
        const int gr = remap_block(i, groups, DENSE_LC);
        const int row = gr / b.gx, tx = 4 * (gr - row * b.gx) + wave;
        return tx < b.tx ? map[(size_t)row * b.tx + tx] : -1;
    };
    const auto mask_of = [&](int t) { return t >= 0 ? recs[t].mask : 0ull; };
    const auto base_of = [&](int t) { return t >= 0 ? recs[t].base : 0ull; };
    // a tile's record is loaded one group ahead, its number two
    int g = (int)blockIdx.x;
    int t = lookup(g), t1 = lookup(g + (int)gridDim.x);
    uint64_t mask = mask_of(t), base = base_of(t);
    for (; g < groups; g += (int)gridDim.x) {
        const int t2 = lookup(g + 2 * (int)gridDim.x);
        const uint64_t mask1 = mask_of(t1), base1 = base_of(t1);
        double v[4] = {0.0, 0.0, 0.0, 0.0};  // rho, u
        if (lane_on(mask)) {
            macro_of_tile<ST>(a, t, TileRec{mask, base}, lane, v[0], v[1], v[2], v[3]);
            sums.add(v[0], v[1], v[2], v[3]);
        }
        if constexpr (FIELDS) {
            const int gr = remap_block(g, groups, DENSE_LC);
            const int row = gr / b.gx;
            // this node's place in its plane of the group
            const int y = lane >> 2 & 3;
            const int to = (lane >> 4) * 64 + (b.along_y ? 16 * wave + 4 * y : 16 * y + 4 * wave) + (lane & 3);
#pragma unroll
            for (int c = 0; c < 4; ++c) rows[buf][c][to] = v[c];
            __syncthreads();
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = rows[buf][c][threadIdx.x];
            buf ^= 1;  // the next barrier comes before this half is written again
            const DenseBox::At d = b.node(gr - row * b.gx, row, lane, wave);
            if (d.in) {
                if (rho_out) rho_out[d.at] = v[0];
                if (u_out) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) u_out[c * N + d.at] = v[1 + c];
                }
            }
        }
        t = t1;
        t1 = t2;
        mask = mask1;
        base = base1;
    }
    sums.store(partials);
}

// one workgroup reduces the rows of partial sums in a fixed order: thread t
// takes column t % 8 of every 64th row, then the 64 threads of a column meet
// in LDS
constexpr int RED_THREADS = 64 * NSUM;
__global__ __launch_bounds__(RED_THREADS) void k_reduce(const double *partials, int rows, double *out) {
    __shared__ double sh[RED_THREADS];
    const int tid = (int)threadIdx.x, c = tid % NSUM;
    double acc = 0.0, kept = 0.0, most = 0.0;  // the sum and the maximum, of which a column takes one
#pragma unroll 8
    for (int j = tid; j < rows * NSUM; j += RED_THREADS) {
        const double v = partials[j];
        add_kept(acc, kept, v);
        most = fmax(most, v);
    }
    sh[tid] = c == 5 ? most : kept_total(acc, kept);
    __syncthreads();
    for (int s = RED_THREADS / 2; s >= NSUM; s >>= 1) {
        if (tid < s) sh[tid] = (c == 5) ? fmax(sh[tid], sh[tid + s]) : sh[tid] + sh[tid + s];
        __syncthreads();
    }
    if (tid < NSUM) out[tid] = sh[tid];
}

// ---------------------------------------------------------------------------
// dense <-> tile conversions
// ---------------------------------------------------------------------------
template <class Walk, int ST>
__global__ __launch_bounds__(64 << WALK_LW) void k_get_state(KArgs a, DenseBox b, int groups, double *dense) {
    using C = Codec<ST>;
    using S = typename C::S;
    const size_t N = (size_t)b.nx * b.ny * b.nz;
    for (Walk w(a.tb, b, groups); w.more();) {
        const DenseNode d = w.next();
        S raw[Q];
        if (d.fl) {
#pragma unroll
            for (int i = 0; i < Q; ++i) raw[i] = load_elem<uint64_t, S>(a.src, d.template elem<C::RUNS>(i));
        }
        if (!d.in) continue;
#pragma unroll
        for (int i = 0; i < Q; ++i)
            dense[(size_t)i * N + d.at] =
                d.fl ? (double)C::dec(raw[i], a.P.inv_scale) + weight(i) * a.P.rho_base : 0.0;
    }
}

template <int ST>
__global__ __launch_bounds__(512) void k_set_state(KArgs a, const double *dense, int nx, int ny, int nz) {
    using C = Codec<ST>;
    using S = typename C::S;
    using T = typename C::T;
    const int t = wave_tile(a.lw, a.nblocks);
    if (t >= a.n_tiles) return;
    const int lane = (int)(threadIdx.x & 63);
    const TileRec rec = a.tb.rec[t];
    const bool fl = (rec.mask >> lane) & 1;
    const Self<C::RUNS, uint64_t> me(rec, lane);
    const size_t N = (size_t)nx * ny * nz;
    const size_t n = dense_index(a.tb.xyz + 4 * (size_t)t, lane, nx, ny);
    // every load before the first store (the compiler has to take it that a
    // store may change the dense array), and stores that do not displace what
    // the neighbouring tiles read of the same lines (128^3 pack, FP64: 92.8 ->
    // 84.8 us; 150 x 131 x 90 box, FP32: 91.7 -> 82.6)
    double v[Q];
    if (fl) {
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = dense[(size_t)i * N + n];
    }
    auto value = [&](int i) { return C::enc((T)(v[i] - weight(i) * a.P.rho_base), a.P.scale); };
    if constexpr (C::RUNS) {
        store_tile<S, true, uint64_t, true>(a.dst, me, rec.mask, fl, lane, value);
    } else {
        S *out = reinterpret_cast<S *>(a.dst);
#pragma unroll
        for (int i = 0; i < Q; ++i) out[me.elem(i)] = fl ? value(i) : S(0);
    }
}

// dense [3][nz][ny][nx] body acceleration -> force density F = rho0 g per
// fluid slot; the pad entries after a tile's 3k are set to 0
template <typename T>
__global__ __launch_bounds__(512) void k_force_to_tiles(KArgs a, const double *g, T *out, int nx, int ny, int nz) {
    const int t = wave_tile(a.lw, a.nblocks);
    if (t >= a.n_tiles) return;
    const int lane = (int)(threadIdx.x & 63);
    const uint64_t mask = a.tb.rec[t].mask;
    const FieldSlot fs(a.tb, t, mask);
    if ((mask >> lane) & 1) {
        const size_t N = (size_t)nx * ny * nz;
        const size_t n = dense_index(a.tb.xyz + 4 * (size_t)t, lane, nx, ny);
#pragma unroll
        for (int c = 0; c < 3; ++c) out[fs.entry(c)] = (T)(a.P.rho0 * g[(size_t)c * N + n]);
    }
    const int used = 3 * fs.k;
    if (lane < (int)field_elems_dev(mask) - used) out[fs.base + (uint64_t)(used + lane)] = T(0);
}

// per-fluid-slot field [3 components] -> dense FP64 [3][nz][ny][nx]
template <class Walk, typename T>
__global__ __launch_bounds__(64 << WALK_LW) void k_field_to_dense(KArgs a, DenseBox b, int groups, const T *in, double *dense) {
    const size_t N = (size_t)b.nx * b.ny * b.nz;
    for (Walk w(a.tb, b, groups); w.more();) {
        const DenseNode d = w.next();
        T v[3] = {T(0), T(0), T(0)};
        if (d.fl) {
            const uint64_t first = a.tb.fbase[d.tile];
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] = in[d.field_entry(first, c)];
        }
        if (!d.in) continue;
#pragma unroll
        for (int c = 0; c < 3; ++c) dense[(size_t)c * N + d.at] = (double)v[c];
    }
}

template <class Walk, typename T>
__global__ __launch_bounds__(64 << WALK_LW) void k_tiles_to_dense(KArgs a, DenseBox b, int groups, const T *in, int ncomp,
                                                                  double *dense) {
    const size_t N = (size_t)b.nx * b.ny * b.nz;
    for (Walk w(a.tb, b, groups); w.more();) {
        const DenseNode d = w.next();
        if (!d.in) continue;
        for (int c = 0; c < ncomp; ++c)
            dense[(size_t)c * N + d.at] = d.fl ? (double)in[((size_t)d.tile * ncomp + c) * TILE + d.n] : 0.0;
    }
}

// ---------------------------------------------------------------------------
// discrete adjoint (every model, runs layout; FP64 storage with FP64
// arithmetic or FP32 storage with FP32 arithmetic, gradient sums in FP64)
//
// For the quasi-compressible collision C(g, F) with rho = sum g,
// u = (sum c g + F/2)/rho (Eq. 3, 5):
//   (J^T lam)_j = (1 - 1/tau) lam_j + A + V.(c_j - u)/rho
//   A   = (1/tau) sum_i lam_i w_i (1 + 3 c.u + 4.5 (c.u)^2 - 1.5 u.u)
//   V   = sum_i lam_i [ (rho/tau) w_i (3 c_i + 9 (c_i.u) c_i - 3 u)
//                       + kg w_i (9 (c_i.F) c_i - 3 F) ]
//   (dC/dF)^T lam = V/(2 rho) + kg sum_i lam_i w_i (3 (c_i - u) + 9 (c_i.u) c_i)
// computed with the sums p = sum lam w (rho/tau (3 + 9 c.u) + 9 kg c.F) c,
// r = sum lam w (3 + 9 c.u) c and q = sum lam w.  J depends on g only through
// rho and j = sum c g, so the forward values may be the shifted ones
// d = g - w rho_base (rho = rho_base + sum d, j = sum c d).  The adjoint
// values themselves are never shifted.
// For the incompressible collision (Eq. 4, 6: feq linear in rho with the
// velocity terms not scaled by it, u = sum c g + F/2), du/dg_j = c_j and
// dfeq_i/drho = w_i, so
//   (J^T lam)_j = (1 - 1/tau) lam_j + q/tau + V.c_j,   (dC/dF)^T lam = V/2 + ...
// with V as above but 1/tau in place of rho/tau.
// ---------------------------------------------------------------------------
template <typename T, int INC = 0>
__device__ __forceinline__ void collide_jt(const T (&d)[Q], T rho_base, const T (&lam)[Q], T omega, T kg, T Fx, T Fy,
                                           T Fz, T (&eta)[Q], T &gx, T &gy, T &gz) {
    T drho = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        drho += d[i];
        if (CX[i]) jx += CX[i] > 0 ? d[i] : -d[i];
        if (CY[i]) jy += CY[i] > 0 ? d[i] : -d[i];
        if (CZ[i]) jz += CZ[i] > 0 ? d[i] : -d[i];
    }
    const T rho = rho_base + drho;
    T ir = T(1), ro = omega;
    if constexpr (!INC) {
        ir = T(1) / rho;
        ro = rho * omega;
    }
    const T ux = (jx + T(0.5) * Fx) * ir, uy = (jy + T(0.5) * Fy) * ir, uz = (jz + T(0.5) * Fz) * ir;
    const T usq = T(1.5) * (ux * ux + uy * uy + uz * uz);
    // rest direction
    T q = lam[0] * T(weight(0));
    T A = q * (T(1) - usq);
    T px = 0, py = 0, pz = 0, rx = 0, ry = 0, rz = 0;
    // Opposite directions i, j have c_j = -c_i and equal weights, so with
    // S = (lam_i + lam_j) w and D = (lam_i - lam_j) w their terms combine:
    //   A += S (1 + 4.5 (c.u)^2 - 1.5 u.u) + 3 (c.u) D,   q += S,
    //   p += c (3 rho/tau D + (9 rho/tau c.u + 9 kg c.F) S),
    //   r += c (3 D + 9 (c.u) S)
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int j = opposite(i);
        if (j < i) continue;
        const T w = T(weight(i));
        const T cu = T(CX[i]) * ux + T(CY[i]) * uy + T(CZ[i]) * uz;
        const T cF = T(CX[i]) * Fx + T(CY[i]) * Fy + T(CZ[i]) * Fz;
        const T S = (lam[i] + lam[j]) * w;
        const T D = (lam[i] - lam[j]) * w;
        A += S * (T(1) + T(4.5) * cu * cu - usq) + T(3) * cu * D;
        q += S;
        const T pi = T(3) * ro * D + (T(9) * ro * cu + T(9) * kg * cF) * S;
        const T ri = T(3) * D + T(9) * cu * S;
        if (CX[i]) { px += T(CX[i]) * pi; rx += T(CX[i]) * ri; }
        if (CY[i]) { py += T(CY[i]) * pi; ry += T(CY[i]) * ri; }
        if (CZ[i]) { pz += T(CZ[i]) * pi; rz += T(CZ[i]) * ri; }
    }
    A = INC ? q * omega : A * omega;
    const T Vx = px - q * (T(3) * ro * ux + T(3) * kg * Fx);
    const T Vy = py - q * (T(3) * ro * uy + T(3) * kg * Fy);
    const T Vz = pz - q * (T(3) * ro * uz + T(3) * kg * Fz);
    const T Vu = Vx * ux + Vy * uy + Vz * uz;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const T Vc = T(CX[j]) * Vx + T(CY[j]) * Vy + T(CZ[j]) * Vz;
        if constexpr (INC) eta[j] = (T(1) - omega) * lam[j] + A + Vc;
        else eta[j] = (T(1) - omega) * lam[j] + A + (Vc - Vu) * ir;
    }
    gx = T(0.5) * Vx * ir + kg * (rx - T(3) * q * ux);
    gy = T(0.5) * Vy * ir + kg * (ry - T(3) * q * uy);
    gz = T(0.5) * Vz * ir + kg * (rz - T(3) * q * uz);
}

// The same for the multiple-relaxation-time operator
//   f* = f - R (f - feq) + (I - R/2) G,   R = M^-1 S M,
// G_i = w_i (3 (c_i - u).F + 9 (c_i.u)(c_i.F)).  With M^-1 = M^T diag(1/|row|^2)
// R = M^T diag(s/|row|^2) M is symmetric, so mu = R^T lam is the forward
// relaxation applied to lam, and with nu = lam - mu/2
//   (J^T lam)_j = lam_j - mu_j + A + V.(c_j - u)/rho   (incompressible: V.c_j)
//   A = sum_i mu_i dfeq_i/drho,  V = sum_i [mu_i dfeq_i/du + nu_i w_i (9 (c_i.F) c_i - 3 F)]
//   (dC/dF)^T lam = V/(2 rho) (incompressible V/2) + sum_i nu_i w_i (3 (c_i - u) + 9 (c_i.u) c_i)
template <typename T, int INC>
__device__ __forceinline__ void collide_jt_mrt(const T (&d)[Q], T rho_base, const T (&lam)[Q], T omega, T Fx, T Fy,
                                               T Fz, T (&eta)[Q], T &gx, T &gy, T &gz) {
    T drho = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        drho += d[i];
        if (CX[i]) jx += CX[i] > 0 ? d[i] : -d[i];
        if (CY[i]) jy += CY[i] > 0 ? d[i] : -d[i];
        if (CZ[i]) jz += CZ[i] > 0 ? d[i] : -d[i];
    }
    const T rho = rho_base + drho;
    T ir = T(1);
    if constexpr (!INC) ir = T(1) / rho;
    const T ux = (jx + T(0.5) * Fx) * ir, uy = (jy + T(0.5) * Fy) * ir, uz = (jz + T(0.5) * Fz) * ir;
    const T usq = T(1.5) * (ux * ux + uy * uy + uz * uz);
    const T bs = INC ? T(1) : rho;
    T rl[Q];  // R^T lam = R lam (R is symmetric)
    mrt_relax<T>(lam, omega, rl);
    // P = sum (3a + 9a c.u + 9b c.F) c and Pd = sum (3b + 9b c.u) c with
    // a = mu w bs, b = nu w; Sa = sum a, Sb = sum b
    T A = 0, Sa = 0, Sb = 0, px = 0, py = 0, pz = 0, qx = 0, qy = 0, qz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const T mu = rl[i];
        const T nu = lam[i] - T(0.5) * mu;
        const T w = T(weight(i));
        const T cu = T(CX[i]) * ux + T(CY[i]) * uy + T(CZ[i]) * uz;
        const T cF = T(CX[i]) * Fx + T(CY[i]) * Fy + T(CZ[i]) * Fz;
        A += INC ? mu * w : mu * w * (T(1) + T(3) * cu + T(4.5) * cu * cu - usq);
        const T a = mu * w * bs, b = nu * w;
        Sa += a;
        Sb += b;
        const T pc = T(3) * a + T(9) * a * cu + T(9) * b * cF;
        const T qc = T(3) * b + T(9) * b * cu;
        if (CX[i]) { px += T(CX[i]) * pc; qx += T(CX[i]) * qc; }
        if (CY[i]) { py += T(CY[i]) * pc; qy += T(CY[i]) * qc; }
        if (CZ[i]) { pz += T(CZ[i]) * pc; qz += T(CZ[i]) * qc; }
        eta[i] = lam[i] - mu;
    }
    const T Vx = px - T(3) * (ux * Sa + Fx * Sb);
    const T Vy = py - T(3) * (uy * Sa + Fy * Sb);
    const T Vz = pz - T(3) * (uz * Sa + Fz * Sb);
    const T Vu = Vx * ux + Vy * uy + Vz * uz;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const T Vc = T(CX[j]) * Vx + T(CY[j]) * Vy + T(CZ[j]) * Vz;
        if constexpr (INC) eta[j] += A + Vc;
        else eta[j] += A + (Vc - Vu) * ir;
    }
    gx = T(0.5) * Vx * ir + (qx - T(3) * ux * Sb);
    gy = T(0.5) * Vy * ir + (qy - T(3) * uy * Sb);
    gz = T(0.5) * Vz * ir + (qz - T(3) * uz * Sb);
}

// the transposed Jacobian of a model's collision
template <typename T, int MODEL>
__device__ __forceinline__ void collide_jt_model(const T (&d)[Q], T rho_base, const T (&lam)[Q], T omega, T kg, T Fx,
                                                 T Fy, T Fz, T (&eta)[Q], T &gx, T &gy, T &gz) {
    if constexpr (MODEL >= LBM_MRT_QUASI_COMPRESSIBLE)
        collide_jt_mrt<T, (MODEL & 1)>(d, rho_base, lam, omega, Fx, Fy, Fz, eta, gx, gy, gz);
    else
        collide_jt<T, (MODEL & 1)>(d, rho_base, lam, omega, kg, Fx, Fy, Fz, eta, gx, gy, gz);
}

// The first arguments, ten registers, are what a wave needs before it can
// issue its gathers: the build has them preloaded.
struct AdjArgs {
    char *out;          // adjoint lattice written
    double *grad;       // dL/dg, FP64 per fluid slot (the force field's layout)
    Phys P;
};
//   s       forward lattice feeding the forward gather
//   eta_in  adjoint lattice feeding the reverse gather
#define ADJ_PARAMS                                                                                                 \
    const NbRow *row, const char *s, const char *eta_in, int n_tiles, int lw, int nblocks,                        \
        uint32_t counter, AdjArgs a

template <bool STAGED, typename T, typename OffT>
__device__ __forceinline__ void store_adjoint(char *lattice, const Self<true, OffT> &me, uint64_t own, bool fl, int lane,
                                              const T (&v)[Q]) {
    const auto value = [&](int i) { return v[i]; };
    if constexpr (STAGED) store_tile_staged<T, true, OffT>(lattice, me, fl, lane, value);
    else store_tile<T, true, OffT, true>(lattice, me, own, fl, lane, value);
}

// seed: from s_{T-1}: g_T = S s_{T-1}, s_T = C(g_T), lam_T = dL/ds_T,
// eta_T = J_T^T lam_T, grad = rho0 [(dC/dF)^T lam_T + dL/dF].  With
// u_x = (sum c_x s - F_x/2)/rho (quasi-compressible) lam_T depends on s_T; with
// u_x = sum c_x s - F_x/2 (incompressible) it is c_x / N_fluid.
template <int ST, int MODEL, typename OffT, bool STAGED>
__device__ __forceinline__ void adj_seed_tile(ADJ_PARAMS) {
    constexpr int INC = MODEL & 1;
    using T = typename Codec<ST>::S;
    const int t = wave_tile(lw, nblocks);
    if (t >= n_tiles) return;
    const int lane = (int)(threadIdx.x & 63);
    const RowRegs r(row, t);
    Nbhd<OffT> h;
    load_nbhd<T>(h, r);
    const uint64_t fbase = r.fbase();
    const uint64_t own = h.m[OWN];
    const bool fl = lane_on(own);
    const Self<true, OffT> me(h, lane);
    const T rb = T(a.P.rho_base), om = T(a.P.omega), kg = T(a.P.kg), inv_n = T(a.P.inv_nfluid);
    T eta[Q], gx = 0, gy = 0, gz = 0;
    if (fl) {
        T g[Q];
        gather_all<false, true, T, OffT>(g, h, s, me, lane);
        T Fx, Fy, Fz;
        load_force<T>(a.P, fbase, own, Fx, Fy, Fz);
        T lam[Q];
        T irT = T(1);
        if constexpr (INC) {
#pragma unroll
            for (int i = 0; i < Q; ++i) lam[i] = T(CX[i]) * inv_n;
        } else {
            T st[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) st[i] = g[i];
            collide_model<T, MODEL>(st, rb, om, kg, Fx, Fy, Fz);
            T drT = 0, jx = 0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                drT += st[i];
                jx += T(CX[i]) * st[i];
            }
            irT = T(1) / (rb + drT);
            const T uxT = (jx - T(0.5) * Fx) * irT;
#pragma unroll
            for (int i = 0; i < Q; ++i) lam[i] = (T(CX[i]) - uxT) * irT * inv_n;
        }
        collide_jt_model<T, MODEL>(g, rb, lam, om, kg, Fx, Fy, Fz, eta, gx, gy, gz);
        gx += T(-0.5) * irT * inv_n;
    }
    store_adjoint<STAGED, T, OffT>(a.out, me, own, fl, lane, eta);
    const FieldSlot fs(fbase, own);
    if (fl) {
        a.grad[fs.entry(0)] = a.P.rho0 * (double)gx;
        a.grad[fs.entry(1)] = a.P.rho0 * (double)gy;
        a.grad[fs.entry(2)] = a.P.rho0 * (double)gz;
    }
    const int used = 3 * fs.k;  // the seed also clears the run's pad entries
    if (lane < (int)field_elems_dev(own) - used) a.grad[fs.base + (uint64_t)(used + lane)] = 0.0;
}

// step: lam_{t-1} = S^T eta_t (reverse gather), g_{t-1} = S s_{t-2},
// eta_{t-1} = J^T lam_{t-1}, grad += rho0 (dC/dF)^T lam_{t-1}
// The adjoint lattice is written with non-temporal stores, as the forward
// step writes its lattice: the written lines then do not displace the lines
// of the two gathered lattices that neighbouring tiles read again from L2
// (FP64 LBGK step on the 128^3 pack 124.7 -> 118.5 us, LBMRT 137.1 -> 132.1).
// Waves per SIMD the adjoint step asks the register allocator for.  The
// FP32 quasi-compressible LBMRT step with 32-bit offsets needs 131 VGPRs
// unconstrained (3 waves); at 4 it fits 128 with no spill and runs 6%
// faster.  Every other instance keeps the allocator's choice: at 4 waves the
// 64-bit-offset one spills, and the FP64 ones spill and cost 33% (LBGK) to
// 3.4x (LBMRT).  That choice for the FP64 LBMRT steps, staged and direct: 156
// and 240 VGPRs (quasi-compressible), 146 and 170, so 3 waves and 2.
template <int ST, int MODEL, typename OffT>
constexpr int ADJ_WAVES = (ST == LBM_F32 && MODEL == LBM_MRT_QUASI_COMPRESSIBLE && sizeof(OffT) == 4) ? 4 : 1;

template <int ST, int MODEL, typename OffT, bool STAGED>
__device__ __forceinline__ void adj_step_tile(ADJ_PARAMS) {
    using T = typename Codec<ST>::S;
    const int tw = wave_tile(lw, nblocks);
    if (tw >= n_tiles) return;
    // consecutive adjoint launches walk the tiles in opposite directions, as
    // the forward steps do (FP64 LBGK 112.5 -> 109.5 us, LBMRT 120.0 -> 115.7
    // us on a 128^3 sphere pack; FP32 unchanged)
    const int t = (counter & 1u) ? n_tiles - 1 - tw : tw;
    const int lane = (int)(threadIdx.x & 63);
    const RowRegs r(row, t);
    Nbhd<OffT> h;
    load_nbhd<T>(h, r);
    const uint64_t fbase = r.fbase();
    const uint64_t own = h.m[OWN];
    const bool fl = lane_on(own);
    const Self<true, OffT> me(h, lane);
    T eta[Q];
    if (fl) {
        T lam[Q], g[Q];
        T Fx, Fy, Fz;
        T gx, gy, gz;
        if constexpr (ST == LBM_F64) {
            // the node's force and gradient entries do not depend on the
            // gather: their loads go first and are in flight with it (LBGK
            // 117.9 -> 117.1 us, incompressible 116.6 -> 114.8, LBMRT 130.0
            // -> 123.7 on a 128^3 sphere pack; FP32 gains nothing from it)
            const FieldSlot fs(fbase, own);
            const double g0 = a.grad[fs.entry(0)], g1 = a.grad[fs.entry(1)], g2 = a.grad[fs.entry(2)];
            load_force<T>(a.P, fbase, own, Fx, Fy, Fz);
            gather_pairs<true, T, OffT>(lam, g, h, eta_in, s, me, lane);
            collide_jt_model<T, MODEL>(g, T(a.P.rho_base), lam, T(a.P.omega), T(a.P.kg), Fx, Fy, Fz, eta, gx, gy,
                                       gz);
            a.grad[fs.entry(0)] = g0 + a.P.rho0 * (double)gx;
            a.grad[fs.entry(1)] = g1 + a.P.rho0 * (double)gy;
            a.grad[fs.entry(2)] = g2 + a.P.rho0 * (double)gz;
        } else {
            gather_pairs<true, T, OffT>(lam, g, h, eta_in, s, me, lane);
            load_force<T>(a.P, fbase, own, Fx, Fy, Fz);
            collide_jt_model<T, MODEL>(g, T(a.P.rho_base), lam, T(a.P.omega), T(a.P.kg), Fx, Fy, Fz, eta, gx, gy,
                                       gz);
            const FieldSlot fs(fbase, own);
            a.grad[fs.entry(0)] += a.P.rho0 * (double)gx;
            a.grad[fs.entry(1)] += a.P.rho0 * (double)gy;
            a.grad[fs.entry(2)] += a.P.rho0 * (double)gz;
        }
    }
    store_adjoint<STAGED, T, OffT>(a.out, me, own, fl, lane, eta);
}

// final: lam_0 = S^T eta_1
template <int ST, int MODEL, typename OffT, bool STAGED>
__device__ __forceinline__ void adj_final_tile(ADJ_PARAMS) {
    using T = typename Codec<ST>::S;
    const int t = wave_tile(lw, nblocks);
    if (t >= n_tiles) return;
    const int lane = (int)(threadIdx.x & 63);
    const RowRegs r(row, t);
    Nbhd<OffT> h;
    load_nbhd<T>(h, r);
    const uint64_t own = h.m[OWN];
    const bool fl = lane_on(own);
    const Self<true, OffT> me(h, lane);
    T lam[Q];
    if (fl) {
        gather_all<true, true, T, OffT>(lam, h, eta_in, me, lane);
    }
    store_adjoint<STAGED, T, OffT>(a.out, me, own, fl, lane, lam);
}

#define ADJ_NAMES row, s, eta_in, n_tiles, lw, nblocks, counter, a
#define ADJ_KERNEL(NAME, BODY, STAGED, ATTRIBUTES)                                 \
    template <int ST, int MODEL, typename OffT>                                    \
    __global__ __launch_bounds__(512) ATTRIBUTES void NAME(ADJ_PARAMS) {           \
        BODY<ST, MODEL, OffT, STAGED>(ADJ_NAMES);                                  \
    }
#define STEP_WAVES __attribute__((amdgpu_waves_per_eu(ADJ_WAVES<ST, MODEL, OffT>, 8)))
ADJ_KERNEL(k_adj_seed, adj_seed_tile, true, )
ADJ_KERNEL(k_adj_seed_direct, adj_seed_tile, false, )
ADJ_KERNEL(k_adj_step, adj_step_tile, true, STEP_WAVES)
ADJ_KERNEL(k_adj_step_direct, adj_step_tile, false, STEP_WAVES)
ADJ_KERNEL(k_adj_final, adj_final_tile, true, )
ADJ_KERNEL(k_adj_final_direct, adj_final_tile, false, )

// ---------------------------------------------------------------------------
// bandwidth probes: what the part sustains for plain streaming, the practical
// ceiling beside the nominal peak (the paper sets its GPU's measured copy
// bandwidth beside the peak, Section 4.1).  Kind 1 reads, kind 2 writes zeros,
// kind 3 copies; 16-byte non-temporal accesses, PROBE_UNROLL of them in
// flight per thread, grid-stride over the buffer.
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int PROBE_UNROLL = 4;

template <int KIND>
__global__ __launch_bounds__(1024) void k_probe(const u32x4 *src, u32x4 *dst, size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t acc = 0;
    for (; i + (PROBE_UNROLL - 1) * stride < n16; i += PROBE_UNROLL * stride) {
        u32x4 v[PROBE_UNROLL];
        if constexpr (KIND != 2) {
#pragma unroll
            for (int u = 0; u < PROBE_UNROLL; ++u) v[u] = __builtin_nontemporal_load(src + i + u * stride);
        }
#pragma unroll
        for (int u = 0; u < PROBE_UNROLL; ++u) {
            if constexpr (KIND == 1) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
            else if constexpr (KIND == 2) __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, dst + i + u * stride);
            else __builtin_nontemporal_store(v[u], dst + i + u * stride);
        }
    }
    for (; i < n16; i += stride) {
        if constexpr (KIND == 1) {
            const u32x4 v = __builtin_nontemporal_load(src + i);
            acc ^= v.x ^ v.y ^ v.z ^ v.w;
        } else if constexpr (KIND == 2) {
            __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, dst + i);
        } else {
            __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
        }
    }
    // the read probe stores only if its data hash to one fixed value, which
    // keeps every load without writing anything in practice
    if constexpr (KIND == 1) {
        if (acc == 0x9E3779B9u) reinterpret_cast<uint32_t *>(dst)[0] = acc;
    }
}

hipError_t launch_probe(hipStream_t s, int kind, const void *src, void *dst, size_t bytes, int blocks, int threads) {
    const u32x4 *in = reinterpret_cast<const u32x4 *>(src);
    u32x4 *out = reinterpret_cast<u32x4 *>(dst);
    const size_t n16 = bytes / 16;
    switch (kind) {
    case 1: hipLaunchKernelGGL(k_probe<1>, dim3(blocks), dim3(threads), 0, s, in, out, n16); break;
    case 2: hipLaunchKernelGGL(k_probe<2>, dim3(blocks), dim3(threads), 0, s, in, out, n16); break;
    default: hipLaunchKernelGGL(k_probe<3>, dim3(blocks), dim3(threads), 0, s, in, out, n16); break;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static KArgs make_args(const Launch &L, const Phys &P, const void *src, void *dst) {
    KArgs a;
    a.src = reinterpret_cast<const char *>(src);
    a.dst = reinterpret_cast<char *>(dst);
    a.tb = L.tb;
    a.n_tiles = L.n_tiles;
    a.lw = __builtin_ctz((unsigned)L.tpw);
    a.nblocks = L.grid;
    a.P = P;
    return a;
}

// The arguments that a wave needs before it can issue its gathers, the first
// of every kernel that gathers: the build has the command processor preload
// the first twelve argument registers (-amdgpu-kernarg-preload-count), so they
// are in scalar registers when a wave starts instead of a memory read away.
#define KHOT(a) (a).tb.row, (a).src, (a).dst, (a).n_tiles, (a).lw, (a).nblocks

// Whether a launch stages its stores: on grids of so many tiles that the waves
// that wait for the LDS are covered by others; within the 64 KB that a
// workgroup is sure to get; to lattices on a 16-byte boundary.  One line for
// all kernels, which costs none of them more than 2.5% (packs, us a step, direct
// -> staged):
//   tiles              512          3300         5124          6320          7324          10332         17233         169669
//   FP64 LBGK          5.7 -> 6.2   13.3 -> 13.5 16.0 -> 16.0  21.4 -> 21.4  24.2 -> 24.1  33.9 -> 33.8  50.2 -> 49.3  388 -> 374
//   FP64 LBMRT                                   17.0 -> 17.2  22.4 -> 22.4  25.4 -> 25.3  35.6 -> 35.5  51.7 -> 51.6  407 -> 406
//   FP32 LBGK                                    10.5 -> 10.3  13.4 -> 13.3  14.9 -> 14.6  19.9 -> 19.7  28.9 -> 28.1  220 -> 204
//   FP16 LBGK                                     9.3 -> 9.4   10.3 -> 10.4  10.9 -> 11.1  13.7 -> 14.1  19.9 -> 19.9  159 -> 158
//   FP64 LBGK adjoint                            23.8 -> 24.0  32.4 -> 32.4  36.8 -> 36.6  51.8 -> 51.7  78.3 -> 77.4  666 -> 653
//   FP32 LBGK adjoint                            15.8 -> 15.3  21.8 -> 21.1  24.5 -> 23.9  33.8 -> 32.8  50.2 -> 48.4  413 -> 393
constexpr int STAGE_MIN_TILES = 6144;
template <typename S>
static bool stage_stores(const Launch &L, const void *dst) {
    return L.n_tiles >= STAGE_MIN_TILES && L.tpw * STAGE_BYTES<S> <= 65536 && reinterpret_cast<uintptr_t>(dst) % 16 == 0;
}

// LDS bytes a staging workgroup asks for: its stage, and on grids whose tiles
// are nearly all full (`line` fluid nodes a tile on average) as much as leaves
// room for `waves` waves per CU alone.  Full tiles in flight on every wave that
// the registers allow take more than an XCD's 4 MB of L2 between them, and
// lines that a neighbour is about to read are lost (FP64, 16 waves: 5 MB).  us a
// step without -> with the limit: 256^3 box, FP64 LBGK 949 -> 908, LBMRT 979 -> 897,
// FP32 457 -> 451; 384^3, FP64 3302 -> 3034, FP32 1579 -> 1492; 251 x 243 x 197
// walled, FP64 642 -> 620, FP32 329 -> 326; adjoint step on it, FP64 LBGK 1063 -> 1049,
// FP32 609 -> 600.
// The lines: FP64 LBGK gains 2.5% at 61 and 0.4% at 46, LBMRT, whose waves take
// longer, gains 4-8% at 63 and 64, between -2 and +2% at 62, and loses 1-5% at 60 and
// 6% at 46; FP32 gains 0.6% at 62 and loses 2-5% at 32.  Tiles from where on, FP64
// LBGK adjoint step: 8000 +1%, 13824 -0.3%.
constexpr int FULL_TILES = 61, FULL_TILES_MRT64 = 63, FULL_MIN_TILES = 12288;
constexpr size_t LDS_OF_CU = 163840, LDS_GRANULE = 1280, LDS_OF_GROUP = 65536;
template <typename S>
static size_t stage_request(const Launch &L, int waves, int line) {
    const size_t stage = (size_t)L.tpw * STAGE_BYTES<S>;
    if (L.fill < line || L.n_tiles < FULL_MIN_TILES || waves < L.tpw) return stage;
    const size_t share = LDS_OF_CU / (waves / L.tpw) / LDS_GRANULE * LDS_GRANULE;
    const size_t ask = share < LDS_OF_GROUP ? share : LDS_OF_GROUP;
    return ask > stage ? ask : stage;
}
// waves per CU of a step (0: FP16 has no limit) and of an adjoint step on full tiles
template <int ST>
constexpr int STEP_WAVES_FULL = ST == LBM_F64 ? 12 : ST == LBM_F32 ? 20 : 0;
template <int ST>
constexpr int ADJ_WAVES_FULL = ST == LBM_F64 ? 8 : 20;

static dim3 block_of(const Launch &L) { return dim3(64 * L.tpw); }

template <int ST, int MODEL, typename OffT>
static hipError_t step_o(const Launch &L, KArgs a) {
    using S = typename Codec<ST>::S;
    if (a.P.f16_stochastic) a.lw |= STOCHASTIC;
    const bool staged = stage_stores<S>(L, a.dst);
    constexpr int line = ST == LBM_F64 && MODEL >= LBM_MRT_QUASI_COMPRESSIBLE ? FULL_TILES_MRT64 : FULL_TILES;
    const size_t lds = staged ? stage_request<S>(L, STEP_WAVES_FULL<ST>, line) : 0;
    if (a.P.bc) {
        const auto fn = staged ? k_step_open<ST, MODEL, OffT> : k_step_open_direct<ST, MODEL, OffT>;
        hipLaunchKernelGGL(fn, dim3(L.grid), block_of(L), lds, L.stream, KHOT(a), a.P.launch_counter, a.P.bc, a.P);
    } else {
        const auto fn = staged ? k_step<ST, MODEL, OffT> : k_step_direct<ST, MODEL, OffT>;
        hipLaunchKernelGGL(fn, dim3(L.grid), block_of(L), lds, L.stream, KHOT(a), a.P.launch_counter, a.P);
    }
    return hipGetLastError();
}

template <int ST, int MODEL>
static hipError_t step_t(const Launch &L, const KArgs &a) {
    return L.off32 ? step_o<ST, MODEL, uint32_t>(L, a) : step_o<ST, MODEL, uint64_t>(L, a);
}

template <int ST>
static hipError_t step_st(const Launch &L, const KArgs &a, int model) {
    switch (model) {
    case LBM_QUASI_COMPRESSIBLE: return step_t<ST, LBM_QUASI_COMPRESSIBLE>(L, a);
    case LBM_INCOMPRESSIBLE: return step_t<ST, LBM_INCOMPRESSIBLE>(L, a);
    case LBM_MRT_QUASI_COMPRESSIBLE: return step_t<ST, LBM_MRT_QUASI_COMPRESSIBLE>(L, a);
    case LBM_MRT_INCOMPRESSIBLE: return step_t<ST, LBM_MRT_INCOMPRESSIBLE>(L, a);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_step(const Launch &L, const Phys &P, const void *src, void *dst) {
    if (L.n_tiles == 0) return hipSuccess;
    const KArgs a = make_args(L, P, src, dst);
    switch (P.storage) {
    case LBM_F64: return step_st<LBM_F64>(L, a, P.model);
    case LBM_F32: return step_st<LBM_F32>(L, a, P.model);
    case LBM_F16S: return step_st<LBM_F16S>(L, a, P.model);
    }
    return hipErrorInvalidValue;
}

template <int ST, int KIND, typename OffT>
static hipError_t calib_o(const Launch &L, const KArgs &a) {
    using C = Codec<ST>;
    using S = typename C::S;
    const bool staged = stage_stores<S>(L, a.dst);
    const auto fn = staged ? k_calib<S, C::RUNS, KIND, OffT, true> : k_calib<S, C::RUNS, KIND, OffT, false>;
    const size_t lds = staged ? stage_request<S>(L, STEP_WAVES_FULL<ST>, FULL_TILES) : 0;  // as an LBGK step's
    hipLaunchKernelGGL(fn, dim3(L.grid), block_of(L), lds, L.stream, KHOT(a), a.tb.rec);
    return hipGetLastError();
}

template <int ST, int KIND>
static hipError_t calib_t(const Launch &L, const KArgs &a) {
    return L.off32 ? calib_o<ST, KIND, uint32_t>(L, a) : calib_o<ST, KIND, uint64_t>(L, a);
}

template <typename S, int LS>
static hipError_t calib_layout_t(const Launch &L, const KArgs &a) {
    if (L.off32)
        hipLaunchKernelGGL((k_calib_layout<S, LS, uint32_t>), dim3(L.grid), block_of(L), 0, L.stream, KHOT(a));
    else
        hipLaunchKernelGGL((k_calib_layout<S, LS, uint64_t>), dim3(L.grid), block_of(L), 0, L.stream, KHOT(a));
    return hipGetLastError();
}

template <typename S>
static hipError_t calib_layout_s(const Launch &L, const KArgs &a, int ls) {
    switch (ls) {
    case 0: return calib_layout_t<S, 0>(L, a);
    case 1: return calib_layout_t<S, 1>(L, a);
    case 2: return calib_layout_t<S, 2>(L, a);
    case 3: return calib_layout_t<S, 3>(L, a);
    default: return calib_layout_t<S, 4>(L, a);
    }
}

hipError_t launch_calib(const Launch &L, int kind, int storage, const void *src, void *dst) {
    if (L.n_tiles == 0) return hipSuccess;
    Phys P{};
    const KArgs a = make_args(L, P, src, dst);
    if (kind >= 3) {
        // kinds 3..6: layout sets XYZ, XYZ+zigzagNE, XYZ+YXZ, all three;
        // kind 7: face-major
        static constexpr int LS[5] = {0, 2, 1, 3, 4};
        const int ls = LS[kind - 3];
        if (storage == LBM_F64) return calib_layout_s<double>(L, a, ls);
        if (storage == LBM_F32) return calib_layout_s<float>(L, a, ls);
        return calib_layout_s<_Float16>(L, a, ls);
    }
    if (storage == LBM_F64) return kind == 1 ? calib_t<LBM_F64, 1>(L, a) : calib_t<LBM_F64, 2>(L, a);
    if (storage == LBM_F32) return kind == 1 ? calib_t<LBM_F32, 1>(L, a) : calib_t<LBM_F32, 2>(L, a);
    return kind == 1 ? calib_t<LBM_F16S, 1>(L, a) : calib_t<LBM_F16S, 2>(L, a);
}

hipError_t launch_init(const Launch &L, const Phys &P, void *a_buf, void *b_buf, double ux, double uy, double uz) {
    if (L.n_tiles == 0) return hipSuccess;
    const KArgs a = make_args(L, P, nullptr, a_buf);
    char *b = reinterpret_cast<char *>(b_buf);
    switch (P.storage) {
    case LBM_F64: hipLaunchKernelGGL(k_init<LBM_F64>, dim3(L.grid), block_of(L), 0, L.stream, a, b, ux, uy, uz); break;
    case LBM_F32: hipLaunchKernelGGL(k_init<LBM_F32>, dim3(L.grid), block_of(L), 0, L.stream, a, b, ux, uy, uz); break;
    default: hipLaunchKernelGGL(k_init<LBM_F16S>, dim3(L.grid), block_of(L), 0, L.stream, a, b, ux, uy, uz); break;
    }
    return hipGetLastError();
}

hipError_t launch_fill(hipStream_t s, double *p, size_t n) {
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

static DenseBox dense_box(const Launch &L, int nx, int ny, int nz) {
    DenseBox b;
    b.map = L.tb.map;
    b.tx = (nx + 3) / 4;
    b.ty = (ny + 3) / 4;
    b.along_y = b.tx == 1;
    if (b.along_y) {
        b.tx = b.ty;
        b.ty = 1;
    }
    b.gx = (b.tx + 3) / 4;
    b.nx = nx;
    b.ny = ny;
    b.nz = nz;
    return b;
}

// Workgroups of a pass that goes over the tiles or the box in strides: 2048 of
// 4 waves (8 waves per SIMD are as many; the passes have 5 to 8 resident), and
// 4 times that for the fields and sums of a large box (256^3 pack, FP64, us a call for the
// fields: 348 with 8192, 375 with 2048; 192^3 267 and 264; 128^3 68 and 57.5, every
// workgroup leaving a row to be added up).
constexpr int WALK_GROUPS = 2048;
constexpr int MACRO_GROUPS = 8192;

// The way over the box, and so the order of the additions, follows from the
// tiles and the box alone: a call with fields and one without return the same
// sums bit by bit.  A summing pass has at most one workgroup per tile, for
// which there are rows of partial sums.
template <int ST>
static hipError_t macro_t(const Launch &L, const KArgs &a, double *rho, double *u, int nx, int ny, int nz,
                          double *partials, int *rows) {
    if (L.walk) {
        const DenseBox b = dense_box(L, nx, ny, nz);
        const int groups = (int)dense_groups(nx, ny, nz);
        int grid = groups < 4 * MACRO_GROUPS ? WALK_GROUPS : MACRO_GROUPS;
        if (grid > groups) grid = groups;
        if (grid > L.n_tiles) grid = L.n_tiles;
        const auto fn = rho || u ? k_fields<ST, true> : k_fields<ST, false>;
        hipLaunchKernelGGL(fn, dim3(grid), dim3(MACRO_THREADS), 0, L.stream, a, b, groups, rho, u, partials);
        *rows = grid;
        return hipGetLastError();
    }
    const size_t N = (size_t)nx * ny * nz;
    hipError_t e = rho ? launch_fill(L.stream, rho, N) : hipSuccess;
    if (e == hipSuccess && u) e = launch_fill(L.stream, u, 3 * N);
    if (e != hipSuccess) return e;
    const int waves = MACRO_THREADS / 64, tiles = (L.n_tiles + waves - 1) / waves;
    const int grid = tiles < WALK_GROUPS ? tiles : WALK_GROUPS;
    hipLaunchKernelGGL(k_sums<ST>, dim3(grid), dim3(MACRO_THREADS), 0, L.stream, a, nx, ny, nz, rho, u, partials);
    *rows = grid;
    return hipGetLastError();
}

// rows: how many rows of partial sums launch_reduce is to add up (at most one
// per tile)
hipError_t launch_macro(const Launch &L, const Phys &P, const void *state, double *rho, double *u, int nx, int ny,
                        int nz, double *partials, int *rows) {
    *rows = 0;
    if (L.n_tiles == 0) return hipSuccess;
    const KArgs a = make_args(L, P, state, nullptr);
    switch (P.storage) {
    case LBM_F64: return macro_t<LBM_F64>(L, a, rho, u, nx, ny, nz, partials, rows);
    case LBM_F32: return macro_t<LBM_F32>(L, a, rho, u, nx, ny, nz, partials, rows);
    default: return macro_t<LBM_F16S>(L, a, rho, u, nx, ny, nz, partials, rows);
    }
}

hipError_t launch_reduce(hipStream_t s, const double *partials, int rows, double *out) {
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(RED_THREADS), 0, s, partials, rows, out);
    return hipGetLastError();
}

// runs a kernel over the box, or clears `out` and runs it over the kept tiles
// (without one the tables are absent)
template <class K, class... Args>
static hipError_t to_dense(const Launch &L, K by_box, K by_tile, const KArgs &a, int nx, int ny, int nz,
                           size_t out_elems, double *out, Args... args) {
    const DenseBox b = dense_box(L, nx, ny, nz);
    const int threads = 64 << WALK_LW;
    if (L.walk) {
        const int groups = (int)dense_groups(nx, ny, nz);
        hipLaunchKernelGGL(by_box, dim3(groups < WALK_GROUPS ? groups : WALK_GROUPS), dim3(threads), 0, L.stream, a, b,
                           groups, args...);
        return hipGetLastError();
    }
    const hipError_t e = launch_fill(L.stream, out, out_elems);
    if (e != hipSuccess || L.n_tiles == 0) return e;
    const int grid = (L.n_tiles + (1 << WALK_LW) - 1) >> WALK_LW;
    hipLaunchKernelGGL(by_tile, dim3(grid), dim3(threads), 0, L.stream, a, b, L.n_tiles, args...);
    return hipGetLastError();
}

template <int ST>
static hipError_t get_state_t(const Launch &L, const KArgs &a, double *dense, int nx, int ny, int nz) {
    return to_dense(L, k_get_state<DenseWalk, ST>, k_get_state<TileWalk, ST>, a, nx, ny, nz,
                    (size_t)Q * nx * ny * nz, dense, dense);
}

template <typename T>
static hipError_t field_t(const Launch &L, const KArgs &a, const void *field, double *dense, int nx, int ny, int nz) {
    return to_dense(L, k_field_to_dense<DenseWalk, T>, k_field_to_dense<TileWalk, T>, a, nx, ny, nz,
                    (size_t)3 * nx * ny * nz, dense, reinterpret_cast<const T *>(field), dense);
}

template <typename T>
static hipError_t tiles_t(const Launch &L, const KArgs &a, const void *buf, int ncomp, double *dense, int nx, int ny,
                          int nz) {
    return to_dense(L, k_tiles_to_dense<DenseWalk, T>, k_tiles_to_dense<TileWalk, T>, a, nx, ny, nz,
                    (size_t)ncomp * nx * ny * nz, dense, reinterpret_cast<const T *>(buf), ncomp, dense);
}

hipError_t launch_get_state(const Launch &L, const Phys &P, const void *state, double *dense, int nx, int ny, int nz) {
    const KArgs a = make_args(L, P, state, nullptr);
    switch (P.storage) {
    case LBM_F64: return get_state_t<LBM_F64>(L, a, dense, nx, ny, nz);
    case LBM_F32: return get_state_t<LBM_F32>(L, a, dense, nx, ny, nz);
    default: return get_state_t<LBM_F16S>(L, a, dense, nx, ny, nz);
    }
}

hipError_t launch_set_state(const Launch &L, const Phys &P, const double *dense, void *state, int nx, int ny, int nz) {
    if (L.n_tiles == 0) return hipSuccess;
    const KArgs a = make_args(L, P, nullptr, state);
    switch (P.storage) {
    case LBM_F64: hipLaunchKernelGGL(k_set_state<LBM_F64>, dim3(L.grid), block_of(L), 0, L.stream, a, dense, nx, ny, nz); break;
    case LBM_F32: hipLaunchKernelGGL(k_set_state<LBM_F32>, dim3(L.grid), block_of(L), 0, L.stream, a, dense, nx, ny, nz); break;
    default: hipLaunchKernelGGL(k_set_state<LBM_F16S>, dim3(L.grid), block_of(L), 0, L.stream, a, dense, nx, ny, nz); break;
    }
    return hipGetLastError();
}

hipError_t launch_force_to_tiles(const Launch &L, const Phys &P, const double *g, void *tile_buf, int nx, int ny, int nz) {
    if (L.n_tiles == 0) return hipSuccess;
    const KArgs a = make_args(L, P, nullptr, nullptr);
    if (P.storage == LBM_F64)
        hipLaunchKernelGGL(k_force_to_tiles<double>, dim3(L.grid), block_of(L), 0, L.stream, a, g,
                           reinterpret_cast<double *>(tile_buf), nx, ny, nz);
    else
        hipLaunchKernelGGL(k_force_to_tiles<float>, dim3(L.grid), block_of(L), 0, L.stream, a, g,
                           reinterpret_cast<float *>(tile_buf), nx, ny, nz);
    return hipGetLastError();
}

hipError_t launch_field_to_dense(const Launch &L, const void *field, int dtype, double *dense, int nx, int ny,
                                 int nz) {
    Phys P{};
    const KArgs a = make_args(L, P, nullptr, nullptr);
    return dtype == 0 ? field_t<double>(L, a, field, dense, nx, ny, nz) : field_t<float>(L, a, field, dense, nx, ny, nz);
}

hipError_t launch_tiles_to_dense(const Launch &L, const void *tile_buf, int ncomp, int dtype, double *dense, int nx,
                                 int ny, int nz) {
    Phys P{};
    const KArgs a = make_args(L, P, nullptr, nullptr);
    return dtype == 0 ? tiles_t<double>(L, a, tile_buf, ncomp, dense, nx, ny, nz)
                      : tiles_t<float>(L, a, tile_buf, ncomp, dense, nx, ny, nz);
}

// the adjoint kernels exist for FP64 and FP32 storage (runs layout) and every
// model; the final reverse gather has no model
template <int ST, int MODEL, typename OffT>
struct SeedK {
    static constexpr auto staged = k_adj_seed<ST, MODEL, OffT>, direct = k_adj_seed_direct<ST, MODEL, OffT>;
};
template <int ST, int MODEL, typename OffT>
struct StepK {
    static constexpr auto staged = k_adj_step<ST, MODEL, OffT>, direct = k_adj_step_direct<ST, MODEL, OffT>;
};
template <int ST, int MODEL, typename OffT>
struct FinalK {
    static constexpr auto staged = k_adj_final<ST, LBM_QUASI_COMPRESSIBLE, OffT>,
                          direct = k_adj_final_direct<ST, LBM_QUASI_COMPRESSIBLE, OffT>;
};
using AdjFn = void (*)(ADJ_PARAMS);

template <template <int, int, typename> class K, int ST, int MODEL>
static AdjFn adj_fn(const Launch &L, bool staged) {
    if (L.off32) return staged ? K<ST, MODEL, uint32_t>::staged : K<ST, MODEL, uint32_t>::direct;
    return staged ? K<ST, MODEL, uint64_t>::staged : K<ST, MODEL, uint64_t>::direct;
}

template <template <int, int, typename> class K, int ST>
static AdjFn adj_fn(const Launch &L, bool staged, int model) {
    switch (model) {
    case LBM_QUASI_COMPRESSIBLE: return adj_fn<K, ST, LBM_QUASI_COMPRESSIBLE>(L, staged);
    case LBM_INCOMPRESSIBLE: return adj_fn<K, ST, LBM_INCOMPRESSIBLE>(L, staged);
    case LBM_MRT_QUASI_COMPRESSIBLE: return adj_fn<K, ST, LBM_MRT_QUASI_COMPRESSIBLE>(L, staged);
    case LBM_MRT_INCOMPRESSIBLE: return adj_fn<K, ST, LBM_MRT_INCOMPRESSIBLE>(L, staged);
    }
    return nullptr;
}

// Mean fluid nodes of a tile from which on the FP64 LBMRT adjoint kernels store
// directly: staged they run 3 waves per SIMD, direct 2, and on full tiles the
// third costs more in lines lost from the L2 than it covers (us a step, staged
// and direct: 256^3 box 1570 and 1550, 251 x 243 x 197 walled 1087 and 1072, packs of 60
// nodes 1370 and 1347, 57 nodes 1239 and 1225, 53 nodes 1096 and 1090, 46 nodes
// 880 and 887, 40 nodes 665 and 693).
constexpr int MRT_DIRECT_FILL = 51;

template <template <int, int, typename> class K>
static hipError_t launch_adj(const Launch &L, const Phys &P, const void *s, const void *eta_in, void *out,
                             double *grad) {
    if (L.n_tiles == 0) return hipSuccess;
    const bool f32 = P.storage == LBM_F32;
    const bool full_mrt = !f32 && P.model >= LBM_MRT_QUASI_COMPRESSIBLE && L.fill >= MRT_DIRECT_FILL;
    const bool staged = f32 ? stage_stores<float>(L, out) : !full_mrt && stage_stores<double>(L, out);
    const AdjFn fn = f32 ? adj_fn<K, LBM_F32>(L, staged, P.model) : adj_fn<K, LBM_F64>(L, staged, P.model);
    if (!fn) return hipErrorInvalidValue;
    AdjArgs a;
    a.out = reinterpret_cast<char *>(out);
    a.grad = grad;
    a.P = P;
    const size_t lds = !staged ? 0
                       : f32   ? stage_request<float>(L, ADJ_WAVES_FULL<LBM_F32>, FULL_TILES)
                               : stage_request<double>(L, ADJ_WAVES_FULL<LBM_F64>, FULL_TILES);
    hipLaunchKernelGGL(fn, dim3(L.grid), block_of(L), lds, L.stream, L.tb.row,
                       reinterpret_cast<const char *>(s), reinterpret_cast<const char *>(eta_in), L.n_tiles,
                       __builtin_ctz((unsigned)L.tpw), L.grid, P.launch_counter, a);
    return hipGetLastError();
}

hipError_t launch_adjoint_seed(const Launch &L, const Phys &P, const void *s_prev, void *eta, double *grad) {
    return launch_adj<SeedK>(L, P, s_prev, nullptr, eta, grad);
}

hipError_t launch_adjoint_step(const Launch &L, const Phys &P, const void *s_prev2, const void *eta_in, void *eta_out,
                               double *grad) {
    return launch_adj<StepK>(L, P, s_prev2, eta_in, eta_out, grad);
}

hipError_t launch_adjoint_final(const Launch &L, const Phys &P, const void *eta_in, void *lambda_out) {
    return launch_adj<FinalK>(L, P, nullptr, eta_in, lambda_out, nullptr);
}

}  // namespace tlbm
