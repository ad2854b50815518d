// The walk step of the deterministic-walk claw search (Sec. 2 and Sec. 3) on gfx950.
//
// One walk is owned by a group of G = min(4^n, 64) lanes of one wavefront; lane gl holds the
// RPL = 4^n / G consecutive rows r = gl * RPL + j.  A step f(x, b) computes the matrix hash of
//   side 0: M = R(p_0) ... R(p_{h-1}),   side 1: M = S_c R(p_0)^T ... R(p_{h-1})^T
// (channel representations; p_j = base-xi digit j of x, plus one).  The hash needs only the row
// digests S_r = sum_q K[q] phi(M_rq) in Z/p, p = 2^61 - 1, phi(sqrt2) = 2^31, i.e. the vector
// phi(M) K.  By associativity that vector is computed without forming M:
//   side 0: S = R(p_0) (R(p_1) ( ... (R(p_{h-1}) K)))
//   side 1: S = phi(S_c) u,  u = R(p_0)^T ( ... (R(p_{h-1})^T K))
// Each factor touches the vector by the channel rep's column rule (one butterfly per
// anticommuting row; the 1/sqrt2 is a 61-bit rotation by 30); at n = 4 the first two factors
// applied to K come from a table of rotated keys built once per search seed (2 x 256^2 vectors of
// 256 values), so a step reads one row of it and applies the remaining h - 2.  The side-1 product
// with the fixed chunk matrix S_c = (A + B sqrt2)/sqrt2^e runs on int8 MFMA for n >= 3 (A and B in
// LDS as B-operand fragments, against signed base-256 digits of u and 2^31 u) and on int8 dot
// products (v_dot4_i32_i8) against 7-bit limbs of u for n <= 2.  At n = 4 a wavefront runs two
// walks, and when both next points are on side 1 one pass of the MFMAs serves both steps.  Then (nu + h of Sec. 2):
//   D_r = min(S_r, p - S_r)   (sign-normalised row: negating a row negates S_r)
//   H = mix64(sum_r g(D_r))   (mod 2^64: an additive multiset hash, so the order of the rows -- a
//                               left signed permutation -- drops out), with the element map
//   g(D) = ((D mod 2^32 + a) mod 2^32) ((D div 2^32 + b) mod 2^32),  a, b the halves of salt_h
//   (NH of Black, Halevi, Krawczyk, Krovetz and Rogaway, UMAC, CRYPTO 1999, on the digest's two
//   32-bit words: one 32 x 32 -> 64-bit product per row)
//   f(x, b) = (floor(H * xi^h / 2^64), H mod 2)                    (reduction back to a point)
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace tcw {

namespace {

template <int NQ>
struct Geo {
    static constexpr int R = 1 << (2 * NQ);
    static constexpr uint32_t XI = (uint32_t)R - 1;
    static constexpr int G = R < 64 ? R : 64;       // lanes per walk
    static constexpr int RPL = R / G;               // rows per lane (1 or 4)
    static constexpr int LRPL = RPL == 4 ? 2 : 0;
    static constexpr int WPW = 64 / G;              // walks per wavefront
    static constexpr int Q4 = R / 4;                // 4-column groups
    // most rotations per half with xi^h < 2^32
    static constexpr int HMAX = NQ == 1 ? 20 : (NQ == 2 ? 8 : (NQ == 3 ? 5 : 4));
};

typedef int v4i __attribute__((ext_vector_type(4)));

// n <= 2: S_c as int8 dwords [q/4][r] for v_dot4; per-walk limb buffer [q/4][limb].
template <int NQ, int WAVES>
struct Lds {
    uint32_t phiA[Geo<NQ>::Q4 * Geo<NQ>::R];
    uint32_t phiB[Geo<NQ>::Q4 * Geo<NQ>::R];
    uint64_t K[Geo<NQ>::R];
    uint32_t limbs[WAVES * Geo<NQ>::WPW][Geo<NQ>::Q4 * LIMB_STRIDE];
};

// n = 4: S_c as MFMA B-operand fragments.  With K stacked as [A | B] (512 columns), fragment
// (nt, kk) holds, for lane l, the 16 bytes S''[nt*16 + l%16][kk*64 + (l/16)*16 + 0..15] where
// S''[r][q] = A[r][q] for q < 256 and B[r][q - 256] otherwise; one ds_read_b128 per lane per MFMA.
// Per wavefront: digit rows [4][68] (signed base-256 digits of the rotated key vector, 4 columns per
// dword; the row stride of 68 dwords keeps the MFMA A-operand reads free of bank conflicts).
constexpr int N4_NT = 16, N4_KK = 8, N4_ROW = 68;
constexpr int N4_DIG = 8;  // signed base-256 digits of a residue below 2^62
template <int WAVES>
struct Lds<4, WAVES> {
    v4i frag[N4_NT * N4_KK * 64];
    uint64_t K[256];
    alignas(16) uint32_t limbs[WAVES][4 * N4_ROW];
};

// n = 3: S_c as MFMA B-operand fragments in the same layout with KK = 2 K steps and NT = 4 tiles;
// per walk (one per wavefront, lane l holds row l): digit rows [8][20] (64 bytes, one per column,
// plus padding).
constexpr int N3_NT = 4, N3_KK = 2, N3_ROW = 20;
template <int WAVES>
struct Lds<3, WAVES> {
    v4i frag[N3_NT * N3_KK * 64];
    uint64_t K[64];
    uint32_t limbs[WAVES][N4_DIG * N3_ROW];
    alignas(16) uint32_t zero_row[N3_ROW];
};

// A value every lane of the wavefront holds (the walk of a whole wavefront), made explicitly uniform.
__device__ inline uint64_t uniform64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline uint32_t uniform32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int NQ, int WAVES>
__device__ void load_lds(Lds<NQ, WAVES>& L, const SpaceDev& sp) {
    using Gm = Geo<NQ>;
    constexpr int NPHI = Gm::Q4 * Gm::R;
    if constexpr (NQ == 4) {
        const v4i* src = reinterpret_cast<const v4i*>(sp.phi);
        for (int i = threadIdx.x; i < N4_NT * N4_KK * 64; i += blockDim.x) L.frag[i] = src[i];
    } else if constexpr (NQ == 3) {
        const v4i* src = reinterpret_cast<const v4i*>(sp.phi);
        for (int i = threadIdx.x; i < N3_NT * N3_KK * 64; i += blockDim.x) L.frag[i] = src[i];
        for (int i = threadIdx.x; i < N3_ROW; i += blockDim.x) L.zero_row[i] = 0;
    } else {
        for (int i = threadIdx.x; i < NPHI; i += blockDim.x) {
            L.phiA[i] = sp.phi[i];
            L.phiB[i] = sp.phi[NPHI + i];
        }
    }
    for (int i = threadIdx.x; i < Gm::R; i += blockDim.x) L.K[i] = sp.keys[i];
}

// a 64-bit value moved by one DPP pattern (every source lane inside the wave: quad permutes, row
// rotations)
template <int CTRL>
__device__ inline uint64_t dpp64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, true);
    return ((uint64_t)hi << 32) | lo;
}

// x * 2^s mod p for a lane-dependent 0 <= s < 61 (x in [0, p])
__device__ inline uint64_t m61_rotv(uint64_t x, uint32_t s) {
    return ((x << s) | (x >> (61 - s))) & P61;
}

// sum_i acc_i 2^(7 i) mod p for nine signed limb sums |acc_i| < 2^24, exactly: the low five and
// the high four limbs are combined in 64-bit integers, then reduced.
__device__ inline uint64_t limbs_to_m61(const int32_t* acc) {
    uint64_t lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < 5; ++i) lo += (uint64_t)(int64_t)acc[i] << (7 * i);
#pragma unroll
    for (int i = 5; i < NLIMB; ++i) hi += (uint64_t)(int64_t)acc[i] << (7 * (i - 5));
    // |lo| < 2^53, |hi| < 2^46: adding 4p keeps the exact value positive and below 2^64
    const uint64_t l = m61_fold(lo + 4 * P61), hh = m61_fold(hi + 4 * P61);
    return m61_add(l, m61_rot(hh, 35));
}

// Cross-half exchanges without LDS (gfx950 v_permlane32_swap / v_permlane16_swap).  permlane32_swap
// exchanges lanes 32..63 of its first operand with lanes 0..31 of its second; permlane16_swap the
// odd 16-lane rows of the first with the even rows of the second.  So half_add32(x, y) leaves lanes
// 0..31 with x + x(lane + 32) and lanes 32..63 with y(lane - 32) + y; half_add16 likewise within
// each 32-lane half (rows 0, 2 get x + x(lane + 16), rows 1, 3 get y(lane - 16) + y).
// half_addNN(v, v) is v + v(lane ^ NN) in every lane.
// The halves are joined into a register pair before the add (an empty asm the compiler cannot see
// through), so the sum is one 64-bit add rather than a split low add, carry and high add.
__device__ inline uint64_t join64(uint32_t lo, uint32_t hi) {
    uint64_t v = ((uint64_t)hi << 32) | lo;
    asm("" : "+v"(v));
    return v;
}
__device__ inline uint64_t half_add32(uint64_t x, uint64_t y) {
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return join64(lo[0], hi[0]) + join64(lo[1], hi[1]);
}
__device__ inline uint64_t half_add16(uint64_t x, uint64_t y) {
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return join64(lo[0], hi[0]) + join64(lo[1], hi[1]);
}
// 32-bit version: x + x(lane + 32) in lanes 0..31, y(lane - 32) + y in lanes 32..63.
__device__ inline int32_t half_add32_i32(int32_t x, int32_t y) {
    const auto v = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    return (int32_t)(v[0] + v[1]);
}

// Two 16-lane rows' halves of one matrix row brought together: with x, y the same quantity of two tiles,
// even rows of lanes get (x, x(lane + 16)), odd rows (y(lane - 16), y): the first is from the lanes that
// hold the low digits, the second from those with the high ones.
struct LowHigh {
    int32_t low, high;
};
__device__ inline LowHigh swap_rows16(int32_t x, int32_t y) {
    const auto v = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    return {(int32_t)v[0], (int32_t)v[1]};
}

// A row digest from its eight signed digit sums, in the halves lo = acc_0 + 2^8 acc_1, hi = acc_2 + 2^8 acc_3 of
// the low and of the high four digits:
//   2^s (lo.low + 2^16 hi.low + 2^32 lo.high + 2^48 hi.high)  mod p, in [0, p],
// for |lo|, |hi| <= 257 * 512 * 128 * 127 < 2^31 - 2^23.  With A = lo.low + 2^16 hi.low and T = (A >> 32) + lo.high (within
// int32) this is
//   A mod 2^32 + 2^32 ((T mod 2^29) + 2^16 (hi.high mod 2^13)) + (T >> 29) + (hi.high >> 13)   (mod p),
// and the last two are kept positive by DIGEST_BIAS, taken off lo.low first.  So 0 <= x < 2^62 - 2^47, and x 2^s is
// ((x << s) mod 2^61) + (x >> (61 - s)) < 2^62 - 2^46, folded once.  Only 32-bit halves cross lanes and one
// modular word is formed per row; with a residue per half that crossed lanes as 64 bits, then folded and
// rotated, the recombination and the hash took 55 instead of 37 instructions a row.
constexpr int32_t DIGEST_BIAS = (1 << 18) + 4;
// x + v and x * 2^16 + v as one multiply-add each (full rate here); written as 64-bit sums they take
// moves to widen their operands.
__device__ inline uint64_t add_u32(uint64_t x, uint32_t v) {
    uint64_t r;
    asm("v_mad_u64_u32 %0, vcc, %1, 1, %2" : "=v"(r) : "v"(v), "v"(x) : "vcc");
    return r;
}
__device__ inline int64_t shl16_add(int32_t x, int32_t v) {
    int64_t r;
    asm("v_mad_i64_i32 %0, vcc, %1, %2, %3" : "=v"(r) : "v"(x), "s"(65536), "v"((int64_t)v) : "vcc");
    return r;
}
__device__ inline uint64_t digest_of(LowHigh lo, LowHigh hi, uint32_t s) {
    const int64_t A = shl16_add(hi.low, lo.low - DIGEST_BIAS);
    const int32_t T = (int32_t)(A >> 32) + lo.high;
    const uint32_t top = ((uint32_t)T & 0x1fffffffu) + (((uint32_t)hi.high & 0x1fffu) << 16);
    const uint64_t x = add_u32(((uint64_t)top << 32) | (uint32_t)A, (uint32_t)((T >> 29) + (hi.high >> 13) + DIGEST_BIAS));
    const uint64_t t = ((x << s) & P61) + (x >> (61 - s));
    return add_u32(t & P61, (uint32_t)(t >> 61));
}

// n <= 2: phi(S_c) u with v_dot4_i32_i8 on A, B (int8, LDS) and 7-bit limbs of u.
template <int NQ, int WAVES>
__device__ inline void side1_dot4(const Lds<NQ, WAVES>& L, uint32_t* limbs, const uint64_t* u, int gl, int rot_e,
                                  uint64_t* S) {
    using Gm = Geo<NQ>;
    constexpr int R = Gm::R, RPL = Gm::RPL, Q4 = Gm::Q4;
    // 7-bit limbs of u, four columns per dword, into this group's LDS slot
    if constexpr (RPL == 4) {
#pragma unroll
        for (int i = 0; i < NLIMB; ++i) {
            uint32_t dw = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) dw |= (uint32_t)((u[j] >> (7 * i)) & 127) << (8 * j);
            limbs[gl * LIMB_STRIDE + i] = dw;
        }
    } else {
        uint8_t* lb = reinterpret_cast<uint8_t*>(limbs);
#pragma unroll
        for (int i = 0; i < NLIMB; ++i)
            lb[((gl >> 2) * LIMB_STRIDE + i) * 4 + (gl & 3)] = (uint8_t)((u[0] >> (7 * i)) & 127);
    }
    wave_sync();
    int32_t accA[RPL][NLIMB], accB[RPL][NLIMB];
#pragma unroll
    for (int j = 0; j < RPL; ++j)
#pragma unroll
        for (int i = 0; i < NLIMB; ++i) accA[j][i] = accB[j][i] = 0;
#pragma unroll 2
    for (int q4 = 0; q4 < Q4; ++q4) {
        uint32_t U[NLIMB];
#pragma unroll
        for (int i = 0; i < NLIMB; ++i) U[i] = limbs[q4 * LIMB_STRIDE + i];
#pragma unroll
        for (int j = 0; j < RPL; ++j) {
            const int a = (int)L.phiA[q4 * R + gl * RPL + j];
            const int b = (int)L.phiB[q4 * R + gl * RPL + j];
#pragma unroll
            for (int i = 0; i < NLIMB; ++i) {
                accA[j][i] = __builtin_amdgcn_sdot4(a, (int)U[i], accA[j][i], false);
                accB[j][i] = __builtin_amdgcn_sdot4(b, (int)U[i], accB[j][i], false);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < RPL; ++j) {
        // phi(S_c) u = 2^(30 e) (A u + 2^31 B u)
        const uint64_t al = limbs_to_m61(accA[j]), be = limbs_to_m61(accB[j]);
        S[j] = m61_rot(m61_add(al, m61_rot(be, 31)), rot_e);
    }
    wave_sync();
}

// n = 4: phi(S_c) u on MFMA (v_mfma_i32_16x16x64_i8; N = 16 matrix rows per tile, 16 tiles; K = 512
// = [A | B] in 8 steps).  A-operand row m < 8 is digit m of u on the A half of K, row 8 + m digit m
// of 2^31 u on the B half, so sum_m 256^m (D[m][r] + D[8 + m][r]) = A u + 2^31 B u = 2^(-30 e) S_r
// (mod p).  Lane l holds rows 4g..4g+3 (g = l/16) of column l%16 of every tile; the four lane groups
// are combined by a reduce-scatter over lanes l^32, l^16, leaving each lane four finished rows.
// out[m] = bytes m of x[0..3] (byte j of out[m] = byte m of x[j]): two rounds of v_perm_b32.
__device__ inline void transpose_bytes4(const uint32_t* x, uint32_t* out) {
    const uint32_t t0 = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u);
    const uint32_t t1 = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u);
    const uint32_t t2 = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u);
    const uint32_t t3 = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
    out[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
}

// Digit rows of u (set 0) or of 2^31 u (set 1), four columns per lane: half 0 the low four, half 1 the high
// four, into the wavefront's 4-row buffer.  Signed base-256 digits: for v < 2^62, b = v + C0 with
// C0 = 0x8080808080808080 stays below 2^64 and v = sum_m (byte_m(b) - 128) 256^m, each digit in [-128, 127];
// as an int8 the digit is byte_m(b) xor 0x80.  u is lazily reduced (< 2^61 + 2^32), and so is its image
// 2^31 u = (u >> 30) + (u mod 2^30) 2^31 (mod p).
__device__ inline void digit_words(const uint64_t* u, int set, uint32_t* lo, uint32_t* hi) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint64_t v = set ? (u[j] >> 30) + ((u[j] & 0x3fffffffull) << 31) : u[j];
        const uint64_t b = v + 0x8080808080808080ull;
        lo[j] = (uint32_t)b;
        hi[j] = (uint32_t)(b >> 32);
    }
}
__device__ inline void digit_rows(uint32_t* limbs, const uint32_t* words, int lane) {
    // 4 x 4 byte transpose: digit row m gets byte m of the lane's four values (columns 4 lane + j)
    uint32_t dg[4];
    transpose_bytes4(words, dg);
#pragma unroll
    for (int m = 0; m < 4; ++m) limbs[m * N4_ROW + lane] = dg[m] ^ 0x80808080u;
    wave_sync();
}

template <int WAVES>
__device__ inline void side1_mfma(const Lds<4, WAVES>& L, uint32_t* limbs, const uint64_t* u, int lane, int rot_e,
                                  uint64_t* S) {
    const int g = lane >> 4, n16 = lane & 15;
    // A operand (16 rows x K = 512): rows 0..7 hold the digits of u on the A half of K (columns
    // q < 256) and are zero on the B half; rows 8..15 hold the digits of 2^31 u on the B half and
    // are zero on the A half.  Four rows at a time go through the LDS buffer.
    const uint32_t* arow = limbs + (n16 & 3) * N4_ROW;
    v4i afr[N4_KK];
#pragma unroll
    for (int kk = 0; kk < N4_KK; ++kk) afr[kk] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int set = 0; set < 2; ++set) {
        uint32_t words[2][4];
        digit_words(u, set, words[0], words[1]);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            digit_rows(limbs, words[half], lane);
            if ((n16 >> 2) == 2 * set + half) {
#pragma unroll
                for (int kq = 0; kq < 4; ++kq)
                    afr[set * 4 + kq] = *reinterpret_cast<const v4i*>(&arow[kq * 16 + g * 4]);
            }
            wave_sync();
        }
    }
    // N tiles in groups of NG: NG independent accumulation chains over the 8 K steps, then each
    // finished tile is combined at once, so only NG accumulators and 2 NG fragments (the current
    // and the next K step's) are live.
    // Accumulator row m = 4g + j of this lane is digit m % 8 of set g >> 1 (u, or 2^31 u), weight
    // 2^(8 (m % 8)).  Each row sums 256 products, |acc| <= 256 * 128 * 127 < 2^22.
    constexpr int NG = 2;
    // Fragments of tiles 8..15 lie beyond the 64 KiB reach of a DS immediate offset: they are read
    // through a second base address (kept opaque, so it is formed once instead of per read).
    uint32_t hi_base = 8 * N4_KK * 64;
    asm("" : "+v"(hi_base));
    const v4i* frag_hi = L.frag + hi_base;
    int32_t lo[N4_NT], hi[N4_NT];
    // tile groups in the order 0..1, 8..9, 4..5, 12..13, 2..3, ...: the tiles (i, 8 + i), then (i, i + 4) of
    // their sums, complete early, which keeps few halves live
    constexpr int order[8] = {0, 8, 4, 12, 2, 10, 6, 14};
#pragma unroll
    for (int gi = 0; gi < N4_NT / NG; ++gi) {
        const int n0 = order[gi];
        v4i acc[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) acc[i] = v4i{0, 0, 0, 0};
        // B fragments double-buffered: the next K step's NG fragments are read while this step's MFMAs
        // run, so each read has a whole step of MFMAs to cover its LDS latency
        auto frag = [&](int t, int kk) -> v4i {
            return t < 8 ? L.frag[(t * N4_KK + kk) * 64 + lane] : frag_hi[((t - 8) * N4_KK + kk) * 64 + lane];
        };
        v4i bf[2][NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) bf[0][i] = frag(n0 + i, 0);
#pragma unroll
        for (int kk = 0; kk < N4_KK; ++kk) {
            if (kk + 1 < N4_KK) {
#pragma unroll
                for (int i = 0; i < NG; ++i) bf[(kk + 1) & 1][i] = frag(n0 + i, kk + 1);
            }
            // the reads above are issued before this step's MFMAs (nothing moves across)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NG; ++i)
                acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(afr[kk], bf[kk & 1][i], acc[i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            lo[n0 + i] = acc[i][0] + acc[i][1] * 256;
            hi[n0 + i] = acc[i][2] + acc[i][3] * 256;
        }
        // reduce-scatter over the four lane groups.  Groups g and g ^ 2 carry the same digit weights,
        // so their halves add exactly first, in 32 bits (|lo + lo'| < 2^31): lanes g < 2 keep
        // tiles 0..7 plus their l^32 partner's, lanes g >= 2 keep tiles 8..15.  Then the low and the high
        // digits of tiles i and i + 4 meet.
        if (gi & 1) {
#pragma unroll
            for (int i = n0 - 8; i < n0 - 8 + NG; ++i) {
                lo[i] = half_add32_i32(lo[i], lo[8 + i]);
                hi[i] = half_add32_i32(hi[i], hi[8 + i]);
            }
        }
        if ((gi & 3) == 3) {
#pragma unroll
            for (int i = n0 - 12; i < n0 - 12 + NG; ++i)
                S[i] = digest_of(swap_rows16(lo[i], lo[4 + i]), swap_rows16(hi[i], hi[4 + i]), (uint32_t)rot_e);
        }
    }
}

// n = 4, two walks of one wavefront on side 1 together: walk w's digit rows become A-operand rows
// 8w .. 8w + 7, each over the whole K = [u | 2^31 u] (digit m of u on the A half, digit m of 2^31 u
// on the B half), so no A row is zero and one pass of the 128 MFMAs serves both walks.  Walk w's
// u goes through the wavefront's 4-row buffer half a digit set at a time; only the lanes that
// hold those rows take fragments from it.
__device__ inline void digits_pair(uint32_t* limbs, const uint64_t* u, int lane, int w, v4i* afr) {
    const int g = lane >> 4, n16 = lane & 15;
    int quarter = n16 >> 2;
    const uint32_t* arow = limbs + (n16 & 3) * N4_ROW;
#pragma unroll
    for (int set = 0; set < 2; ++set) {
        uint32_t words[2][4];
        digit_words(u, set, words[0], words[1]);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            digit_rows(limbs, words[half], lane);
            asm("" : "+v"(quarter));  // compared afresh: four lane masks kept for the whole launch would spill
            if (quarter == 2 * w + half) {
#pragma unroll
                for (int kq = 0; kq < 4; ++kq)
                    afr[set * 4 + kq] = *reinterpret_cast<const v4i*>(&arow[kq * 16 + g * 4]);
            }
            wave_sync();
        }
    }
}

// an element of the multiset hash: the map g of a digest c in [0, p] after the sign fold.  For c in
// [0, p]: p - c = c ^ p, and of c and p - c the smaller is the one with bit 60 clear, so
// min(c mod p, p - c mod p) = c ^ (bit 60 of c ? p : 0) (which also sends p to 0).
__device__ inline uint64_t digest_map(uint64_t c, uint32_t ka, uint32_t kb) {
    const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int32_t)(c >> 32), 28, 1);
    const uint32_t lo = (uint32_t)c ^ m, hi = (uint32_t)(c >> 32) ^ (m & 0x1fffffffu);
    return (uint64_t)(lo + ka) * (uint64_t)(hi + kb);
}

// The product of both walks on the shared A operand, and the hash elements of its rows summed per lane.
// Accumulator row m = 4g + j of lane l is digit 4 (g & 1) + j of walk g >> 1 summed over both digit sets:
// 512 products of at most 128 x 127, so lo = acc_0 + 2^8 acc_1 and hi = acc_2 + 2^8 acc_3 are within
// digest_of's bounds.  After the swap of a tile pair (i, 8 + i) a lane of even g has all digits of row
// 16 i + n16, one of odd g those of row 16 (8 + i) + n16, of walk g >> 1.
template <int WAVES>
__device__ inline uint64_t side1_mfma_pair(const Lds<4, WAVES>& L, const v4i* afr, int lane, uint32_t s, uint32_t ka,
                                           uint32_t kb) {
    constexpr int NG = 2;
    uint32_t hi_base = 8 * N4_KK * 64;
    asm("" : "+v"(hi_base));
    const v4i* frag_hi = L.frag + hi_base;
    int32_t lo[NG], hi[NG];
    uint64_t sum = 0;
#pragma unroll
    for (int gi = 0; gi < N4_NT / NG; ++gi) {
        const int n0 = (gi & 1) * 8 + (gi >> 1) * NG;
        v4i acc[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) acc[i] = v4i{0, 0, 0, 0};
        auto frag = [&](int t, int kk) -> v4i {
            return t < 8 ? L.frag[(t * N4_KK + kk) * 64 + lane] : frag_hi[((t - 8) * N4_KK + kk) * 64 + lane];
        };
        v4i bf[2][NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) bf[0][i] = frag(n0 + i, 0);
#pragma unroll
        for (int kk = 0; kk < N4_KK; ++kk) {
            if (kk + 1 < N4_KK) {
#pragma unroll
                for (int i = 0; i < NG; ++i) bf[(kk + 1) & 1][i] = frag(n0 + i, kk + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NG; ++i)
                acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(afr[kk], bf[kk & 1][i], acc[i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int32_t l = acc[i][0] + acc[i][1] * 256, h = acc[i][2] + acc[i][3] * 256;
            if (gi & 1) {
                sum += digest_map(digest_of(swap_rows16(lo[i], l), swap_rows16(hi[i], h), s), ka, kb);
            } else {
                lo[i] = l;
                hi[i] = h;
            }
        }
    }
    return sum;
}

// n = 3: phi(S_c) u on MFMA, the n = 4 scheme at R = 64 with one row per lane: A-operand rows 0..7
// are the signed base-256 digits of u on the A half of K = 128, rows 8..15 those of 2^31 u on the
// B half; 4 N tiles x 2 K steps.  Lane l holds accumulator rows 4g..4g+3 (g = l/16) of column l%16
// of each tile; groups g and g ^ 2 have equal digit weights, so their raw sums add first (l^32),
// then the low and the high digits of a row meet (l^16), leaving each lane one finished row.
template <int WAVES>
__device__ inline void side1_mfma3(const Lds<3, WAVES>& L, uint32_t* limbs, const uint64_t* u, int lane, int rot_e,
                                   uint64_t* S) {
    const int g = lane >> 4, n16 = lane & 15;
    const uint32_t* arow0 = n16 < N4_DIG ? limbs + n16 * N3_ROW : L.zero_row;
    const uint32_t* arow1 = n16 >= N4_DIG ? limbs + (n16 - N4_DIG) * N3_ROW : L.zero_row;
    uint8_t* lb = reinterpret_cast<uint8_t*>(limbs);
    v4i afr[N3_KK];
#pragma unroll
    for (int set = 0; set < 2; ++set) {
        // digits as for n = 4 (bytes of v + 0x8080808080808080, each minus 128); column = lane
        const uint64_t w = set ? (u[0] >> 30) + ((u[0] & 0x3fffffffull) << 31) : u[0];
        const uint64_t b = w + 0x8080808080808080ull;
#pragma unroll
        for (int m = 0; m < N4_DIG; ++m) lb[m * N3_ROW * 4 + lane] = (uint8_t)((b >> (8 * m)) ^ 0x80);
        wave_sync();
        const uint32_t* arow = set ? arow1 : arow0;
        afr[set] = *reinterpret_cast<const v4i*>(&arow[g * 4]);
        wave_sync();
    }
    int32_t lo[N3_NT], hi[N3_NT];
#pragma unroll
    for (int nt = 0; nt < N3_NT; ++nt) {
        v4i acc = v4i{0, 0, 0, 0};
#pragma unroll
        for (int kk = 0; kk < N3_KK; ++kk)
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(afr[kk], L.frag[(nt * N3_KK + kk) * 64 + lane], acc, 0, 0, 0);
        // |acc| <= 64 * 128 * 127 < 2^20
        lo[nt] = acc[0] + acc[1] * 256;
        hi[nt] = acc[2] + acc[3] * 256;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        lo[i] = half_add32_i32(lo[i], lo[2 + i]);
        hi[i] = half_add32_i32(hi[i], hi[2 + i]);
    }
    S[0] = digest_of(swap_rows16(lo[0], lo[1]), swap_rows16(hi[0], hi[1]), (uint32_t)rot_e);
}

// n = 3: for each (p, row r) bit 0 = P_p and P_r anticommute, bit 1 = their product's phase c is 3
// (the butterfly of R adds the partner), one byte each, computed at compile time.
struct Rot3Tab {
    uint8_t v[64 * 64];
};
constexpr Rot3Tab make_rot3_tab() {
    Rot3Tab t{};
    for (uint32_t p = 1; p < 64; ++p) {
        const uint32_t xp = p & 7, zp = p >> 3;
        for (uint32_t r = 0; r < 64; ++r) {
            const uint32_t xr = r & 7, zr = r >> 3;
            const uint32_t anti = (uint32_t)(__builtin_popcount(xp & zr) + __builtin_popcount(zp & xr)) & 1;
            const uint32_t c = (uint32_t)(__builtin_popcount(xp & zp) + __builtin_popcount(xr & zr) + 4 -
                                          __builtin_popcount((xp ^ xr) & (zp ^ zr)) + 2 * __builtin_popcount(zp & xr)) &
                               3;
            t.v[p * 64 + r] = (uint8_t)(anti | ((uint32_t)(c == 3) << 1));
        }
    }
    return t;
}
__device__ constexpr Rot3Tab ROT3_TAB = make_rot3_tab();

// n <= 3 (one row per lane, r = gl): the h rotations with the same lazy reduction as rotate4.
template <int NQ>
__device__ inline void rotate1(uint64_t& u, const uint32_t* dig, int h, int side, int gl, int gbase) {
    const uint32_t r = (uint32_t)gl;
    uint32_t tb[Geo<NQ>::HMAX];
    if constexpr (NQ == 3) {
        // every digit slot holds a valid code, so all loads stay in the table
#pragma unroll
        for (int t = 0; t < Geo<NQ>::HMAX; ++t) tb[t] = ROT3_TAB.v[dig[t] * 64 + r];
    }
#pragma unroll
    for (int t = Geo<NQ>::HMAX - 1; t >= 0; --t) {
        if (t >= h) continue;
        const uint32_t p = dig[t];
        const uint64_t part = shfl64(u, gbase + (gl ^ (int)p));
        // side 0 (R u): (u_r - s u_{r^p}) / sqrt2;  side 1 (R^T u): (u_r + s u_{r^p}) / sqrt2
        bool plus, anti;
        if constexpr (NQ == 3) {
            plus = (((tb[t] >> 1) ^ (uint32_t)side) & 1) != 0;
            anti = (tb[t] & 1) != 0;
        } else {
            plus = (side == 1) == (rotation_sign<NQ>(p, r) > 0);
            anti = anticommutes<NQ>(p, r) != 0;
        }
        const uint64_t q = plus ? part : (2 * P61 - part);
        const uint64_t sum = u + q;
        const uint64_t rot = (sum >> 31) + ((sum & 0x7fffffffull) << 30);
        u = anti ? rot : u;
    }
}

// n = 4: the h rotations applied to the key vector.  Lane l holds rows r_j = 4 l + j (j = 0..3).
// Rotation p touches row r when P_p and P_r anticommute (<p, r> = |x_p & z_r| + |z_p & x_r| odd);
// with P_p P_r = i^c P_{p^r}, c = |x_p & z_p| + |x_r & z_r| - |(x_p ^ x_r) & (z_p ^ z_r)| +
// 2 |z_p & x_r| (mod 4), the butterfly of R (side 0) adds the partner value u_{r^p} when c = 3
// and subtracts it when c = 1; R^T (side 1) the other way round.  Both bits depend only on (p, l, j)
// and sit in a compile-time table, one byte per (p, lane): bit j = anticommutes, bit 4 + j = c is 3.
struct Rot4Tab {
    uint8_t v[256 * 64];
};
constexpr Rot4Tab make_rot4_tab() {
    Rot4Tab t{};
    for (uint32_t p = 1; p < 256; ++p) {
        const uint32_t xp = p & 15, zp = p >> 4;
        for (uint32_t l = 0; l < 64; ++l) {
            uint32_t b = 0;
            for (uint32_t j = 0; j < 4; ++j) {
                const uint32_t r = 4 * l + j, xr = r & 15, zr = r >> 4;
                const uint32_t anti = (uint32_t)(__builtin_popcount(xp & zr) + __builtin_popcount(zp & xr)) & 1;
                const uint32_t c = (uint32_t)(__builtin_popcount(xp & zp) + __builtin_popcount(xr & zr) + 4 -
                                              __builtin_popcount((xp ^ xr) & (zp ^ zr)) +
                                              2 * __builtin_popcount(zp & xr)) & 3;
                b |= (anti << j) | ((uint32_t)(c == 3) << (4 + j));
            }
            t.v[p * 64 + l] = (uint8_t)b;
        }
    }
    return t;
}
__device__ constexpr Rot4Tab ROT4_TAB = make_rot4_tab();

// Values stay lazily reduced below 2^61 + 2^32: u + (2p - part) < 2^63, and for s = a 2^31 + b,
// s 2^30 = a 2^61 + b 2^30 = a + b 2^30 (mod p).
// part[j] = u[j ^ C] of lane src (C a compile-time register permutation).
template <int C>
__device__ inline void fetch4(const uint64_t* u, int src, uint64_t* part) {
#pragma unroll
    for (int j = 0; j < 4; ++j) part[j] = shfl64(u[j ^ C], src);
}

__device__ inline void rotate4(uint64_t* u, const uint32_t* dig, int h, int side, int gl, int gbase) {
    // the table bytes of the rotations to apply, first, so their latency overlaps the partner fetches
    uint32_t tb[Geo<4>::HMAX];
#pragma unroll
    for (int t = 0; t < Geo<4>::HMAX; ++t) tb[t] = t < h ? ROT4_TAB.v[dig[t] * 64 + gl] : 0u;
    const uint32_t side_b = side ? 0xf0u : 0u;
#pragma unroll
    for (int t = Geo<4>::HMAX - 1; t >= 0; --t) {
        if (t >= h) continue;
        const uint32_t p = dig[t];
        // partner rows r ^ p: lane l ^ (p >> 2), register j ^ (p & 3).  p is wave-uniform, so the
        // register order is a uniform branch and all eight partner fetches are issued together.
        const int src = gbase + (gl ^ (int)(p >> 2));
        uint64_t part[4];
        switch (p & 3) {
            case 0: fetch4<0>(u, src, part); break;
            case 1: fetch4<1>(u, src, part); break;
            case 2: fetch4<2>(u, src, part); break;
            default: fetch4<3>(u, src, part); break;
        }
        // bit j: anticommutes; bit 4 + j: the butterfly adds the partner (side 0: c = 3, side 1: c = 1)
        const uint32_t b = tb[t] ^ side_b;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t q = ((b >> (4 + j)) & 1) ? part[j] : (2 * P61 - part[j]);
            const uint64_t sum = u[j] + q;
            const uint64_t r = (sum >> 31) + ((sum & 0x7fffffffull) << 30);
            u[j] = ((b >> j) & 1) ? r : u[j];
        }
    }
}

// n = 4: the key vector with the first rotations already applied -- R(p_{h-2}) R(p_{h-1}) K or the
// transposes' from the two-rotation table, one rotation from the one-rotation table, or K itself --
// into u (lane gl's four rows); returns how many rotations are left to apply.
template <int WAVES>
__device__ inline int key_row4(const SpaceDev& sp, const Lds<4, WAVES>& L, const uint32_t* dig, int side, int gl,
                               uint64_t* u) {
    const int h = sp.h;
    if (sp.rkeys2 != nullptr && h >= 2) {
        const uint64_t* tp =
            sp.rkeys2 + ((((uint32_t)side * 256u + dig[h - 1]) * 256u + dig[h - 2]) * 256u + 4u * (uint32_t)gl);
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = tp[j];
        return h - 2;
    }
    if (sp.rkeys != nullptr && h >= 1) {
        const uint64_t* tp = sp.rkeys + ((uint32_t)side * 256u + dig[h - 1]) * 256u + 4u * (uint32_t)gl;
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = tp[j];
        return h - 1;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = L.K[gl * 4 + j];
    return h;
}

// One evaluation of f on `pt` by the walk group; every lane of the group returns the same values.
template <int NQ, int WAVES>
__device__ void walk_step(const SpaceDev& sp, const Lds<NQ, WAVES>& L, uint32_t* limbs, uint64_t pt, int gl,
                          int gbase, uint64_t& out_pt, uint64_t& out_h) {
    using Gm = Geo<NQ>;
    constexpr int R = Gm::R, RPL = Gm::RPL, Q4 = Gm::Q4, HMAX = Gm::HMAX;
    if constexpr (Gm::G == 64) pt = uniform64(pt);  // one walk per wavefront: decode on the scalar unit
    const uint32_t x = (uint32_t)pt;
    const int side = (int)((pt >> 32) & 1);
    const int h = sp.h;

    // mu: base-xi digits, least significant first; Pauli p_t = d_t + 1
    uint32_t dig[HMAX];
    {
        uint32_t xx = x;
#pragma unroll
        for (int t = 0; t < HMAX; ++t) {
            dig[t] = xx % Gm::XI + 1;
            xx /= Gm::XI;
        }
    }

    // key vector through the rotations, p_{h-1} first
    uint64_t u[RPL];
    if constexpr (NQ == 4) {
        // the first two rotations, R(p_{h-2}) R(p_{h-1}) K or the transposes', come precomputed for
        // every pair of Paulis (a 256 MiB table in HBM, 2 KiB per step in 32 contiguous bytes per
        // lane); with one rotation only, from a 1 MiB table; the others are applied here
        const int h_left = key_row4(sp, L, dig, side, gl, u);
        rotate4(u, dig, h_left, side, gl, gbase);
    } else {
        u[0] = L.K[gl];
        rotate1<NQ>(u[0], dig, h, side, gl, gbase);
    }

    uint64_t S[RPL];
    if (side) {
        if constexpr (NQ == 4) {
            side1_mfma<WAVES>(L, limbs, u, gl, sp.rot_e, S);
        } else if constexpr (NQ == 3) {
            side1_mfma3<WAVES>(L, limbs, u, gl, sp.rot_e, S);
        } else {
            side1_dot4<NQ, WAVES>(L, limbs, u, gl, sp.rot_e, S);
        }
    } else {
#pragma unroll
        for (int j = 0; j < RPL; ++j) S[j] = m61_fold(u[j]);  // n = 4 keeps u lazily reduced
    }

    // sign-normalised row digests and the multiset hash of the walk group's rows
    uint64_t acc = 0;
    const uint32_t ka = (uint32_t)sp.salt_h, kb = (uint32_t)(sp.salt_h >> 32);
#pragma unroll
    for (int j = 0; j < RPL; ++j) acc += digest_map(S[j], ka, kb);
    if constexpr (Gm::G == 64) {
        // within each 16-lane row by DPP (quad permutes, then row rotations by 4 and 8, which add the
        // other quads' sums), then across rows by the cross-half swaps: no LDS round trip
        acc += dpp64<0xB1>(acc);   // quad_perm [1,0,3,2]
        acc += dpp64<0x4E>(acc);   // quad_perm [2,3,0,1]
        acc += dpp64<0x124>(acc);  // row_ror:4
        acc += dpp64<0x128>(acc);  // row_ror:8
        acc = half_add16(acc, acc);
        acc = half_add32(acc, acc);
        // one walk per wavefront: the sum is the same in every lane; finish on the scalar unit
        acc = uniform64(acc);
    } else {
        // a walk group is a quad (n = 1) or a 16-lane row (n = 2): DPP within it, no LDS round trip
        static_assert(Gm::G == 4 || Gm::G == 16, "walk groups below 64 lanes are quads or rows");
        acc += dpp64<0xB1>(acc);  // quad_perm [1,0,3,2]
        acc += dpp64<0x4E>(acc);  // quad_perm [2,3,0,1]
        if constexpr (Gm::G == 16) {
            acc += dpp64<0x124>(acc);  // row_ror:4
            acc += dpp64<0x128>(acc);  // row_ror:8
        }
    }
    const uint64_t H = mix64(acc);
    out_h = H;
    out_pt = mulhi64(H, sp.n_half) | ((H & 1) << 32);
}

// n = 4: one evaluation of f for each of the wavefront's two walks, both points on side 1 (pa, pb
// uniform).  Each walk's key row, rotations and digits in turn, then the shared MFMA product, and each 32-lane half of the wavefront hashes its walk's
// 256 rows (eight per lane).  The values equal those of two walk_step calls.
template <int WAVES>
__device__ void walk_step_pair4(const SpaceDev& sp, const Lds<4, WAVES>& L, uint32_t* limbs, uint64_t pa,
                                uint64_t pb, int lane, uint64_t& out_a, uint64_t& h_a, uint64_t& out_b,
                                uint64_t& h_b) {
    constexpr int HMAX = Geo<4>::HMAX;
    // the points are the same in every lane: decode on the scalar unit (uniform branches below)
    pa = uniform64(pa);
    pb = uniform64(pb);
    v4i afr[N4_KK];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        uint32_t dig[HMAX];
        uint32_t xx = (uint32_t)(w ? pb : pa);
#pragma unroll
        for (int t = 0; t < HMAX; ++t) {
            dig[t] = xx % Geo<4>::XI + 1;
            xx /= Geo<4>::XI;
        }
        uint64_t u[4];
        const int h_left = key_row4(sp, L, dig, 1, lane, u);
        rotate4(u, dig, h_left, 1, lane, 0);
        digits_pair(limbs, u, lane, w, afr);
    }
    uint64_t acc = side1_mfma_pair<WAVES>(L, afr, lane, (uint32_t)sp.rot_e, (uint32_t)sp.salt_h,
                                          (uint32_t)(sp.salt_h >> 32));
    acc += dpp64<0xB1>(acc);   // quad_perm [1,0,3,2]
    acc += dpp64<0x4E>(acc);   // quad_perm [2,3,0,1]
    acc += dpp64<0x124>(acc);  // row_ror:4
    acc += dpp64<0x128>(acc);  // row_ror:8
    acc = half_add16(acc, acc);
    // lanes 0..31 now hold walk a's sum, lanes 32..63 walk b's
    auto lane64 = [&](int l) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)acc, l);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(acc >> 32), l);
        return ((uint64_t)hi << 32) | lo;
    };
    const uint64_t sa = lane64(0), sb = lane64(32);
    h_a = mix64(sa);
    h_b = mix64(sb);
    out_a = mulhi64(h_a, sp.n_half) | ((h_a & 1) << 32);
    out_b = mulhi64(h_b, sp.n_half) | ((h_b & 1) << 32);
}

__device__ inline bool is_dist(const SpaceDev& sp, uint64_t pt) {
    if (sp.delta == 0) return true;
    const uint64_t x = pt & 0xffffffffull, b = (pt >> 32) & 1;
    return (mix64(((x << 1) | b) ^ sp.salt_d) >> (64 - sp.delta)) == 0;
}

__device__ inline uint64_t start_point(const SpaceDev& sp, uint64_t w, uint32_t j) {
    const uint64_t g = sm64(sp.salt_s, (w << 32) | j);
    return mulhi64(g, sp.n_half) | ((g & 1) << 32);
}

// n = 4: one block per CU (S_c's fragments take 128 KiB of its LDS) of 16 wavefronts, four per SIMD.  Twelve
// were all that fitted while a wavefront had an 8-row digit buffer and the walks' states in vector
// registers (168 of them).  2^18 walks x 16 steps: 4.60 ms then; 4.38 with the digests of digest_of,
// 4.06 with 16 wavefronts, 3.52 with all of walk_block_pairs.
constexpr int WAVES_SMALL = 4;
template <int NQ>
struct WalkWaves {
    static constexpr int value = NQ == 4 ? 16 : WAVES_SMALL;
};

// ---- parity kernels ----
// A space that was made just before on the stream: its exponent read here, and nothing done where its
// flags refuse it (the host reads them afterwards).
__device__ inline bool space_ready(SpaceDev& sp) {
    if (sp.made == nullptr) return true;
    sp.rot_e = (int32_t)((30u * (uint32_t)sp.made[0]) % 61u);
    return sp.made[1] == 0;
}

template <int NQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_step(SpaceDev sp, const uint64_t* in, uint64_t* out,
                                                     uint64_t* hash, int64_t count) {
    using Gm = Geo<NQ>;
    __shared__ Lds<NQ, WAVES> L;
    if (!space_ready(sp)) return;
    load_lds(L, sp);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    uint32_t* limbs = L.limbs[wave * Gm::WPW + gi];
    const int64_t stride = (int64_t)gridDim.x * WAVES * Gm::WPW;
    for (int64_t base = ((int64_t)blockIdx.x * WAVES + wave) * Gm::WPW; base < count; base += stride) {
        const int64_t i = base + gi;
        if (i < count) {
            uint64_t o, hh;
            walk_step<NQ, WAVES>(sp, L, limbs, in[i], gl, gbase, o, hh);
            if (gl == 0) {
                out[i] = o;
                if (hash) hash[i] = hh;
            }
        }
    }
}

// A trail that comes back to a point it has passed has no distinguished point before it, so it never
// reaches one: it is abandoned there (as at the cap) instead of going round up to 20 / theta times.  Brent's
// cycle search (BIT 20, 1980): the point after 1, 2, 4, ... steps is kept and every later one compared with
// it.  A few such trails among 16384 at theta = 2^-8 held a launch for 5,120 steps in a row.
template <int NQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_trails(SpaceDev sp, const uint64_t* starts, int64_t count,
                                                       uint32_t cap, uint64_t* dp, uint32_t* len) {
    using Gm = Geo<NQ>;
    __shared__ Lds<NQ, WAVES> L;
    if (!space_ready(sp)) return;
    load_lds(L, sp);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    uint32_t* limbs = L.limbs[wave * Gm::WPW + gi];
    const int64_t stride = (int64_t)gridDim.x * WAVES * Gm::WPW;
    for (int64_t base = ((int64_t)blockIdx.x * WAVES + wave) * Gm::WPW; base < count; base += stride) {
        const int64_t i = base + gi;
        if (i < count) {
            uint64_t pt = starts[i], seen = pt;
            uint32_t d = 0, found = 0, mark = 1;
            for (uint32_t t = 1; t <= cap; ++t) {
                uint64_t nx, hh;
                walk_step<NQ, WAVES>(sp, L, limbs, pt, gl, gbase, nx, hh);
                pt = nx;
                if (is_dist(sp, pt)) {
                    d = t;
                    found = 1;
                    break;
                }
                if (pt == seen) break;
                if (t == mark) {
                    seen = pt;
                    mark *= 2;
                }
            }
            if (gl == 0) {
                dp[i] = found ? pt : 0;
                len[i] = found ? d : 0;
            }
        }
    }
}

// n = 4: a wavefront runs two trails at a time and takes the next one from *queue (zero before the launch) when
// one ends, so that two side-1 steps share a pass of the MFMAs as in the walk kernel and long trails leave no
// wavefront idle.  With no more trails than wavefronts each runs alone.  16384 trails at n = 4, k = 7,
// theta = 2^-8: 18 to 25 ms with one trail per wavefront to the cap, now 5.6 ms: about 3.3 ms at the walk
// kernel's rate and the last, longest trails.
struct TrailRun {
    int64_t i;  // < 0: none
    uint64_t pt, seen;
    uint32_t n, mark;
};
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_trails4(SpaceDev sp, const uint64_t* starts, int64_t count, uint32_t cap,
                                                        uint64_t* dp, uint32_t* len, unsigned int* queue) {
    __shared__ Lds<4, WAVES> L;
    if (!space_ready(sp)) return;
    load_lds(L, sp);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = (int)uniform32(threadIdx.x >> 6);
    uint32_t* limbs = L.limbs[wave];
    const bool two = count > (int64_t)gridDim.x * WAVES;
    auto take = [&](TrailRun& r) {
        uint32_t i = 0;
        if (lane == 0) i = atomicAdd(queue, 1u);
        i = uniform32(i);
        r.i = i < count ? (int64_t)i : -1;
        r.pt = r.seen = r.i >= 0 ? uniform64(starts[r.i]) : 0;
        r.n = 0;
        r.mark = 1;
    };
    auto advance = [&](TrailRun& r, uint64_t nx) {
        r.n++;
        const bool dist = is_dist(sp, nx);
        if (dist || nx == r.seen || r.n >= cap) {
            if (lane == 0) {
                dp[r.i] = dist ? nx : 0;
                len[r.i] = dist ? r.n : 0;
            }
            take(r);
            return;
        }
        if (r.n == r.mark) {
            r.seen = nx;
            r.mark *= 2;
        }
        r.pt = nx;
    };
    TrailRun a, b;
    take(a);
    b.i = -1;
    b.pt = b.seen = 0;
    b.n = b.mark = 0;
    if (two) take(b);
    while (a.i >= 0 || b.i >= 0) {
        const bool side_a = (a.pt >> 32) & 1, side_b = (b.pt >> 32) & 1;
        uint64_t na, ha, nb, hb;
        if (a.i >= 0 && b.i >= 0 && side_a && side_b) {
            walk_step_pair4<WAVES>(sp, L, limbs, a.pt, b.pt, lane, na, ha, nb, hb);
            advance(a, na);
            advance(b, nb);
        } else {
            const bool pick_b = a.i < 0 || (b.i >= 0 && side_a);
            walk_step<4, WAVES>(sp, L, limbs, pick_b ? b.pt : a.pt, lane, 0, na, ha);
            if (pick_b)
                advance(b, na);
            else
                advance(a, na);
        }
    }
}

// Canonical hash of explicit matrices: the side-1 product with u = K (no rotations).
template <int NQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_canon(SpaceDev sp, const uint32_t* phi_all, const int32_t* e,
                                                      int64_t count, uint64_t* out) {
    using Gm = Geo<NQ>;
    constexpr int NPHI = Gm::Q4 * Gm::R;
    __shared__ Lds<NQ, WAVES> L;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    uint32_t* limbs = L.limbs[wave * Gm::WPW + gi];
    for (int64_t m = blockIdx.x; m < count; m += gridDim.x) {
        SpaceDev s2 = sp;
        s2.phi = phi_all + (size_t)m * 2 * NPHI;
        s2.h = 0;
        s2.rot_e = (int32_t)(((30ll * e[m]) % 61 + 61) % 61);
        s2.n_half = 1;
        __syncthreads();
        load_lds(L, s2);
        __syncthreads();
        if (wave == 0 && gi == 0) {
            uint64_t o, hh;
            walk_step<NQ, WAVES>(s2, L, limbs, 1ull << 32, gl, gbase, o, hh);
            if (gl == 0) out[m] = hh;
        }
    }
}

// x y mod p for x, y < 2^61: x y = hi 2^64 + lo = 8 hi + lo (mod p), lo split at bit 61.
__device__ inline uint64_t m61_mul(uint64_t x, uint64_t y) {
    const uint64_t lo = x * y, hi = __umul64hi(x, y);
    return m61_fold((lo & P61) + (lo >> 61) + (hi << 3));
}

// Canonical hash of explicit matrices whose entries do not fit int8: the row digests
// S_r = sum_q phi(M_rq) K[q] by 64-bit modular products (one matrix per 64-lane block, rows over
// lanes), then the same sign fold, element map and sum as walk_step.  Exact for any int32 entries.
template <int NQ>
__global__ __launch_bounds__(64) void k_canon_wide(SpaceDev sp, const int32_t* a, const int32_t* b,
                                                   const int32_t* e, int64_t count, uint64_t* out) {
    constexpr int R = Geo<NQ>::R;
    const int lane = threadIdx.x;
    const uint32_t ka = (uint32_t)sp.salt_h, kb = (uint32_t)(sp.salt_h >> 32);
    for (int64_t m = blockIdx.x; m < count; m += gridDim.x) {
        // (a + b sqrt2) / sqrt2^e: phi(1/sqrt2) = 2^30, so the scale is a rotation by 30 e mod 61
        const int rot = (int)(((30ll * e[m]) % 61 + 61) % 61);
        uint64_t acc = 0;
        for (int r = lane; r < R; r += 64) {
            const int32_t* ar = a + ((size_t)m * R + r) * R;
            const int32_t* br = b + ((size_t)m * R + r) * R;
            uint64_t sum = 0;
            for (int q = 0; q < R; ++q) {
                const uint64_t v = m61_add(m61_from_i32(ar[q]), m61_rot(m61_from_i32(br[q]), 31));
                sum = m61_add(sum, m61_mul(v, sp.keys[q]));
            }
            const uint64_t c = m61_rot(sum, rot);
            const uint64_t d = c ^ (P61 & (0ull - ((c >> 60) & 1)));
            acc += (uint64_t)((uint32_t)d + ka) * (uint64_t)((uint32_t)(d >> 32) + kb);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc += shfl64(acc, lane ^ off);
        if (lane == 0) out[m] = mix64(acc);
    }
}

template <int NQ>
__global__ void k_pack_i32(const int32_t* a, const int32_t* b, int64_t count, uint32_t* phi, int* flag) {
    constexpr int R = Geo<NQ>::R, Q4 = Geo<NQ>::Q4;
    if constexpr (NQ >= 3) {
        // MFMA fragment layout (see Lds<4>, Lds<3>): 2 * Q4 * R dwords per matrix, KK = 2R / 64 K steps
        constexpr int KK = 2 * R / 64;
        const int64_t total4 = count * 2 * Q4 * R;
        for (int64_t idx = threadIdx.x + (int64_t)blockIdx.x * blockDim.x; idx < total4;
             idx += (int64_t)blockDim.x * gridDim.x) {
            const int64_t m = idx / (2 * Q4 * R);
            const int rem = (int)(idx % (2 * Q4 * R));
            const int fi = rem >> 2, w = rem & 3;
            const int l = fi & 63, fk = fi >> 6;
            const int nt = fk / KK, kk = fk % KK;
            const int r = nt * 16 + (l & 15);
            const int32_t* am = a + m * R * R;
            const int32_t* bm = b + m * R * R;
            uint32_t word = 0;
            for (int c = 0; c < 4; ++c) {
                const int qq = kk * 64 + (l >> 4) * 16 + 4 * w + c;
                const int32_t v = qq < R ? am[r * R + qq] : bm[r * R + qq - R];
                if (v > 127 || v < -127) atomicOr(flag, 2);
                word |= ((uint32_t)(uint8_t)(int8_t)v) << (8 * c);
            }
            phi[m * 2 * Q4 * R + rem] = word;
        }
        return;
    }
    const int64_t total = count * Q4 * R;
    for (int64_t idx = threadIdx.x + (int64_t)blockIdx.x * blockDim.x; idx < total;
         idx += (int64_t)blockDim.x * gridDim.x) {
        const int64_t m = idx / (Q4 * R);
        const int rem = (int)(idx % (Q4 * R));
        const int q4 = rem / R, r = rem % R;
        const int32_t* am = a + m * R * R;
        const int32_t* bm = b + m * R * R;
        uint32_t wa = 0, wb = 0;
        for (int c = 0; c < 4; ++c) {
            const int32_t va = am[r * R + 4 * q4 + c], vb = bm[r * R + 4 * q4 + c];
            if (va > 127 || va < -127 || vb > 127 || vb < -127) atomicOr(flag, 2);
            wa |= ((uint32_t)(uint8_t)(int8_t)va) << (8 * c);
            wb |= ((uint32_t)(uint8_t)(int8_t)vb) << (8 * c);
        }
        phi[m * 2 * Q4 * R + rem] = wa;
        phi[m * 2 * Q4 * R + Q4 * R + rem] = wb;
    }
}

__global__ void k_starts(SpaceDev sp, int64_t w0, uint32_t j, int64_t count, uint64_t* out) {
    for (int64_t i = threadIdx.x + (int64_t)blockIdx.x * blockDim.x; i < count; i += (int64_t)blockDim.x * gridDim.x)
        out[i] = start_point(sp, (uint64_t)(w0 + i), j);
}

// n = 4: out[side][p][q] = the first rotation of the walk step applied to K, by rotate4's butterfly
// (so the values are the ones the step would compute): side 0 R(p) K, side 1 R(p)^T K.  One block
// per (side, p), one thread per row q; p = 0 (no rotation) copies K.
__global__ void k_rot_keys(const uint64_t* keys, uint64_t* out) {
    const uint32_t q = threadIdx.x, p = blockIdx.x & 255u, side = blockIdx.x >> 8;
    uint64_t v = keys[q];
    if (p != 0) {
        const uint32_t b = ROT4_TAB.v[p * 64 + (q >> 2)], j = q & 3;
        if ((b >> j) & 1) {
            const uint64_t part = keys[q ^ p];
            const uint64_t w = (((b >> (4 + j)) ^ side) & 1) ? part : (2 * P61 - part);
            const uint64_t sum = v + w;
            v = (sum >> 31) + ((sum & 0x7fffffffull) << 30);
        }
    }
    out[(size_t)blockIdx.x * 256 + q] = v;
}

// n = 4: out[side][p][p'][q] = rotation p' (rotate4's butterfly) applied to rkeys[side][p]; one block
// per (side, p, p'), one thread per row q; p' = 0 copies.
__global__ void k_rot_keys2(const uint64_t* rkeys, uint64_t* out) {
    const uint32_t q = threadIdx.x, p2 = blockIdx.x & 255u, sp1 = blockIdx.x >> 8, side = sp1 >> 8;
    const uint64_t* in = rkeys + (size_t)sp1 * 256;
    uint64_t v = in[q];
    if (p2 != 0) {
        const uint32_t b = ROT4_TAB.v[p2 * 64 + (q >> 2)], j = q & 3;
        if ((b >> j) & 1) {
            const uint64_t part = in[q ^ p2];
            const uint64_t w = (((b >> (4 + j)) ^ side) & 1) ? part : (2 * P61 - part);
            const uint64_t sum = v + w;
            v = (sum >> 31) + ((sum & 0x7fffffffull) << 30);
        }
    }
    out[(size_t)blockIdx.x * 256 + q] = v;
}

// K[q] = (sm64(s_0, q) >> 3) mod p, s_0 = sm64(seed, 0)
__global__ void k_keys(int r, uint64_t seed, uint64_t* keys) {
    const int i = threadIdx.x + blockIdx.x * blockDim.x;
    if (i >= r) return;
    const uint64_t s0 = sm64(seed, 0);
    uint64_t k = sm64(s0, (uint64_t)i) >> 3;
    if (k >= P61) k -= P61;
    keys[i] = k;
}

// ---- the walk kernel: trails, distinguished-point table, backtracking (Sec. 3) ----

// Claim a slot for `dp` (linear probing).  Returns 1 = new (claimed), 2 = key present, 3 = full.
__device__ inline int table_claim_at(const WalkDev& wd, uint64_t dp, uint64_t s, uint64_t& slot) {
    const uint64_t mask = (1ull << wd.log2_table) - 1;
    s &= mask;
    for (int probe = 0; probe < 64; ++probe) {
        uint64_t expected = EMPTY_KEY;
        const bool won = __hip_atomic_compare_exchange_strong(&wd.table[2 * s], &expected, dp, __ATOMIC_RELAXED,
                                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (won) {
            slot = s;
            return 1;
        }
        if (expected == dp) {
            slot = s;
            return 2;
        }
        s = (s + 1) & mask;
    }
    return 3;
}

__device__ inline int table_claim(const WalkDev& wd, uint64_t dp, uint64_t& slot) {
    return table_claim_at(wd, dp, mix64(dp ^ 0x5bd1e9955bd1e995ull), slot);
}

__device__ inline uint64_t pack_value(uint64_t start, uint32_t len) {
    return (start & 0x1ffffffffull) | ((uint64_t)(len & 0x3fffffffu) << 33) | (1ull << 63);
}

// A walk group's event counts in LDS, in the order of the statistics, written by its leader lane.
struct WalkCounts {
    uint64_t steps = 0, dps = 0, ins = 0, ab = 0, rh = 0, same = 0, red = 0, claw = 0, full = 0, spin = 0,
             active = 0;
};
static_assert(sizeof(WalkCounts) == ST_COUNT * sizeof(uint64_t));

// The counts of the block's `groups` walk groups, added to the walks' statistics and cleared; between two
// barriers.  One addition a block and counter, none of a zero: additions to one address take about 9 ns
// each whoever makes them, and eleven for every walk group were up to 0.5 ms at the end of every launch
// (the three enumerations of an n = 3 search of depth 6: 413 us each, now 106; 2^18 walks x 16 steps at
// n = 4: 3.52 ms, now 3.32).
__device__ inline void flush_counts(const WalkDev& wd, uint64_t* counts, int groups) {
    const int f = (int)threadIdx.x;
    if (f >= ST_COUNT) return;
    uint64_t sum = 0;
    for (int g = 0; g < groups; ++g) {
        sum += counts[g * ST_COUNT + f];
        counts[g * ST_COUNT + f] = 0;
    }
    if (sum) atomicAdd(&wd.stats[f], (unsigned long long)sum);
}

// Events of one evaluation, as bits: advance_walk returns them and the walk group's leader adds
// them to the group's counts in LDS, so no count is held in registers through the step.
enum : uint32_t {
    EV_DP = 1, EV_INS = 2, EV_AB = 4, EV_RH = 8, EV_SAME = 16, EV_RED = 32, EV_CLAW = 64, EV_FULL = 128, EV_SPIN = 256
};

__device__ inline void count_events(WalkCounts& c, uint32_t ev) {
    if (ev & EV_DP) c.dps++;
    if (ev & EV_INS) c.ins++;
    if (ev & EV_AB) c.ab++;
    if (ev & EV_RH) c.rh++;
    if (ev & EV_SAME) c.same++;
    if (ev & EV_RED) c.red++;
    if (ev & EV_CLAW) c.claw++;
    if (ev & EV_FULL) c.full++;
    if (ev & EV_SPIN) c.spin++;
}

// A walk in hand: what every step uses, in registers, and what only backtracking uses, which a whole
// wavefront's walk keeps in LDS (in scalar registers the two walks of a wavefront spilled, and reading
// spilled values back took a tenth of the step's vector instructions).
struct Trail {
    uint64_t start, cur;
    uint32_t len, trail, mode;
};
struct Back {
    uint64_t pa, pb, na, ha;
    uint32_t rem;
};

template <bool WHOLE>
__device__ inline uint64_t same64(uint64_t v) {
    if constexpr (WHOLE) return uniform64(v);
    return v;
}

template <bool WHOLE>
__device__ inline void load_state(const WalkDev& wd, int64_t w, Trail& tr, Back& bk) {
    const WalkState st = wd.states[w];
    tr.start = same64<WHOLE>(st.start);
    tr.cur = same64<WHOLE>(st.cur);
    tr.len = (uint32_t)same64<WHOLE>(st.len);
    tr.trail = (uint32_t)same64<WHOLE>(st.trail);
    tr.mode = (uint32_t)same64<WHOLE>(st.mode);
    bk.pa = st.pa;
    bk.pb = st.pb;
    bk.na = st.na;
    bk.ha = st.ha;
    bk.rem = st.rem;
}

__device__ inline void store_state(const WalkDev& wd, int64_t w, const Trail& tr, const Back& bk) {
    WalkState st;
    st.start = tr.start;
    st.cur = tr.cur;
    st.pa = bk.pa;
    st.pb = bk.pb;
    st.na = bk.na;
    st.ha = bk.ha;
    st.len = tr.len;
    st.trail = tr.trail;
    st.mode = tr.mode;
    st.rem = bk.rem;
    wd.states[w] = st;
}

// The point a walk evaluates f on next: its current point while walking, else the backtracking point
// that ALIGN / LOCK advances.  Masks, since a choice of field would go through memory; a wavefront's own walk branches
// on its mode first, but where lanes of several walks share the wavefront a branch is two of them in a row.
template <bool WHOLE>
__device__ inline uint64_t step_arg(const Trail& tr, const Back& bk) {
    const bool walking = (tr.mode & 0xff) == MODE_WALK;
    if (WHOLE && walking) return tr.cur;
    const uint64_t second = 0ull - (uint64_t)((tr.mode >> 8) & 1);
    const uint64_t back = same64<WHOLE>((bk.pb & second) | (bk.pa & ~second));
    if constexpr (WHOLE) return back;
    const uint64_t walk = 0ull - (uint64_t)walking;
    return (tr.cur & walk) | (back & ~walk);
}

// Walk w's state after one evaluation f(arg) = (nxt, H): distinguished points into the table,
// backtracking of two trails that met (Sec. 3, Fig. 2), claws recorded, trails restarted.  WHOLE:
// the walk occupies the whole wavefront (its leader is lane 0).
template <bool WHOLE>
__device__ inline uint32_t advance_walk(const SpaceDev& sp, const WalkDev& wd, Trail& st, Back& bk, int64_t w,
                                        uint64_t arg, uint64_t nxt, uint64_t H, bool leader, int gbase) {
    uint32_t ev = 0;
    const uint32_t mode = st.mode & 0xff;
    const uint32_t which = (st.mode >> 8) & 1;
    bool restart = false;
    if (mode == MODE_WALK && wd.enumerate) {
        // exhaustive mode: every point once, the table keyed by its full matrix hash and holding,
        // in the two 32-bit halves of the value, the least x of each side that reached the key (a
        // 32-bit atomic minimum, so no ordering between writers is needed).  The pairs are read
        // out after the last point (k_enum_pairs): which pairs are reported does not depend on
        // the order in which walks arrive.
        ev |= EV_DP;
        const uint64_t key = H == EMPTY_KEY ? (H ^ 1) : H;
        int kind = 0;
        if (leader) {
            uint64_t slot = 0;
            kind = table_claim(wd, key, slot);
            if (kind != 3) {
                uint32_t* half = reinterpret_cast<uint32_t*>(&wd.table[2 * slot + 1]) + ((arg >> 32) & 1);
                atomicMin(half, (uint32_t)arg);
            }
        }
        if constexpr (WHOLE)
            kind = (int)uniform32((uint32_t)kind);
        else
            kind = (int)shfl32((uint32_t)kind, gbase);
        if (kind == 3)
            ev |= EV_FULL;
        else if (kind == 1)
            ev |= EV_INS;
        restart = true;
    } else if (mode == MODE_WALK) {
        st.len++;
        if (is_dist(sp, nxt)) {
            ev |= EV_DP;
            int kind = 0;
            uint64_t slot = 0, other = 0;
            if (leader) kind = table_claim(wd, nxt, slot);
            // The slot's writer publishes its value right after its claim.  The value word is
            // all a reader uses (start, length and a ready bit), so relaxed device-scope atomics
            // suffice; release and acquire would write back and invalidate the L2 of the
            // wavefront's XCD at every distinguished point.
            if (leader && kind == 1)
                __hip_atomic_store(&wd.table[2 * slot + 1], pack_value(st.start, st.len), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            if (leader && kind == 2) {
                int spin = 0;
                do {
                    other = __hip_atomic_load(&wd.table[2 * slot + 1], __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
                } while (other == 0 && ++spin < (1 << 20));
                if (other == 0) kind = 4;
            }
            if constexpr (WHOLE) {
                // the walk is the whole wavefront and its leader is lane 0: the answer stays scalar
                kind = (int)uniform32((uint32_t)kind);
                other = uniform64(other);
            } else {
                kind = (int)shfl32((uint32_t)kind, gbase);
                other = shfl64(other, gbase);
            }
            restart = true;
            if (kind == 1) {
                ev |= EV_INS;
            } else if (kind == 3) {
                ev |= EV_FULL;
            } else if (kind == 4) {
                ev |= EV_SPIN;
            } else if (kind == 2) {
                const uint64_t ostart = other & 0x1ffffffffull;
                const uint32_t olen = (uint32_t)((other >> 33) & 0x3fffffffu);
                if (ostart != st.start) {
                    // backtrack the two trails (Sec. 3, Fig. 2)
                    restart = false;
                    bk.pa = st.start;
                    bk.pb = ostart;
                    const uint32_t la = st.len, lb = olen;
                    if (la > lb) {
                        st.mode = MODE_ALIGN;
                        bk.rem = la - lb;
                        st.len = lb;
                    } else if (lb > la) {
                        st.mode = MODE_ALIGN | (1u << 8);
                        bk.rem = lb - la;
                        st.len = la;
                    } else {
                        st.mode = MODE_LOCK;
                        bk.rem = la;
                    }
                }
            }
        } else if (st.len >= wd.cap) {
            ev |= EV_AB;
            restart = true;
        } else {
            st.cur = nxt;
        }
    } else if (mode == MODE_ALIGN) {
        if constexpr (WHOLE) {
            const uint64_t second = 0ull - (uint64_t)which;
            bk.pa = (bk.pa & second) | (nxt & ~second);
            bk.pb = (nxt & second) | (bk.pb & ~second);
        } else {
            // the state is in registers; with the masks above n = 1 and 2 took 4 to 9 percent more a step (64 walks x 640
            // steps at n = 1, k = 8: 917 us, 995 with them and a branch in step_arg)
            if (which) bk.pb = nxt; else bk.pa = nxt;
        }
        const uint32_t rem = (uint32_t)same64<WHOLE>(bk.rem) - 1;
        bk.rem = rem;
        if (rem == 0) {
            if (same64<WHOLE>(bk.pa) == same64<WHOLE>(bk.pb)) {
                ev |= EV_RH;  // one trail started on the other
                restart = true;
            } else {
                st.mode = MODE_LOCK;
                bk.rem = st.len;
            }
        }
    } else {  // MODE_LOCK
        if (!which) {
            bk.na = nxt;
            bk.ha = H;
            st.mode = MODE_LOCK | (1u << 8);
        } else {
            const uint64_t na = same64<WHOLE>(bk.na);
            if (na == nxt) {
                // f(pa) = f(pb) with pa != pb: the merge
                const uint64_t sa = (same64<WHOLE>(bk.pa) >> 32) & 1, sb = (same64<WHOLE>(bk.pb) >> 32) & 1;
                if (sa == sb) {
                    ev |= EV_SAME;
                } else if (same64<WHOLE>(bk.ha) != H) {
                    ev |= EV_RED;
                } else {
                    ev |= EV_CLAW;
                    if (leader) {
                        const unsigned long long idx = atomicAdd(wd.claw_count, 1ull);
                        if (idx < wd.claw_cap) {
                            wd.claws[2 * idx] = bk.pa;
                            wd.claws[2 * idx + 1] = bk.pb;
                        }
                    }
                }
                restart = true;
            } else {
                const uint32_t rem = (uint32_t)same64<WHOLE>(bk.rem) - 1;
                bk.pa = na;
                bk.pb = nxt;
                bk.rem = rem;
                st.mode = MODE_LOCK;
                if (rem == 0) restart = true;  // cannot happen for two trails with one end
            }
        }
    }
    if (restart) {
        st.trail++;
        st.len = 0;
        st.mode = MODE_WALK;
        if (wd.enumerate) {
            const uint64_t idx = (uint64_t)w + (uint64_t)wd.walks * st.trail;
            if (idx >= wd.n_points) {
                st.mode = MODE_DONE;
            } else {
                st.start = (idx % sp.n_half) | ((idx / sp.n_half) << 32);
            }
        } else {
            st.start = start_point(sp, (uint64_t)w, st.trail);
        }
        st.cur = st.start;
    }
    return ev;
}

// `iters` evaluations of f for every walk of slice `block` of `nblocks` (walks (block * WAVES + wave)
// * WPW + group, then every nblocks * WAVES * WPW further).  cnt is the walk group's counts in LDS;
// only the group's leader lane writes it.
template <int NQ, int WAVES>
__device__ void walk_block_single(const SpaceDev& sp, const WalkDev& wd, int iters, Lds<NQ, WAVES>& L, int64_t block,
                                  int64_t nblocks, WalkCounts& cnt) {
    using Gm = Geo<NQ>;
    const int lane = threadIdx.x & 63, wave = (int)uniform32(threadIdx.x >> 6);
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    const bool leader = gl == 0;
    uint32_t* limbs = L.limbs[wave * Gm::WPW + gi];
    // the frequent events (every distinguished point, most of them inserts) are counted in registers
    // and added to cnt once; the rest go to cnt as they happen
    uint32_t steps = 0, active = 0, dps = 0, ins = 0;
    const int64_t stride = nblocks * WAVES * Gm::WPW;
    for (int64_t base = (block * WAVES + wave) * Gm::WPW; base < wd.walks; base += stride) {
        const int64_t w = Gm::G == 64 ? base : base + gi;
        if (w >= wd.walks) continue;
        Trail st;
        Back bk;
        load_state<Gm::G == 64>(wd, w, st, bk);
        if constexpr (Gm::G == 64) {
            bk.pa = uniform64(bk.pa);
            bk.pb = uniform64(bk.pb);
            bk.na = uniform64(bk.na);
            bk.ha = uniform64(bk.ha);
            bk.rem = uniform32(bk.rem);
        }
        for (int it = 0; it < iters; ++it) {
            if ((st.mode & 0xff) == MODE_DONE) break;
            const uint64_t arg = step_arg<Gm::G == 64>(st, bk);
            uint64_t nxt, H;
            walk_step<NQ, WAVES>(sp, L, limbs, arg, gl, gbase, nxt, H);
            steps++;
            const uint32_t ev = advance_walk<Gm::G == 64>(sp, wd, st, bk, w, arg, nxt, H, leader, gbase);
            dps += ev & EV_DP;
            ins += (ev >> 1) & 1;
            const uint32_t rare = ev & ~(uint32_t)(EV_DP | EV_INS);
            if (rare && leader) count_events(cnt, rare);
        }
        if ((st.mode & 0xff) != MODE_DONE) active++;
        if (leader) store_state(wd, w, st, bk);
    }
    if (leader) {
        cnt.steps += steps;
        cnt.active += active;
        cnt.dps += dps;
        cnt.ins += ins;
    }
}

// n = 4: each wavefront runs two walks, 2q and 2q + 1, and gives the pair 2 iters evaluations of f (a walk
// without a partner gets iters); cnt as in walk_block_single.  A walk whose next point is on side 0 steps
// alone; when both next points are on side 1 the two steps share one MFMA product (walk_step_pair4).  So
// the pair's steps add up to 2 iters while each walk's share varies with its sides: a launch's total is
// walks x iters.
// The block's pairs are runs of WAVES neighbours, q = block * WAVES + i for i < WAVES, then every nblocks * WAVES
// further.  SPREAD (one launch's blocks, side by side): runs while every block has a whole one; those left go to the
// blocks one at a time, so that a few walks spread over the CUs instead of filling the first ones' wavefronts (20,000
// walks x 64 steps at k = 7: 1.10 -> 0.96 ms; all pairs one at a time cost 2^20 walks 0.7 percent).  A queue's items
// follow each other on a CU, where a part of a run at the end of each would leave wavefronts idle every time (a
// batch of mixed n: 1.34e9 steps/s, 1.38e9 in runs).
// Its wavefronts take them in turn from *next (LDS, zero at the start).  With a fixed share each, the
// wavefronts that the SIMDs prefer finished early and few were left at the end: a wavefront lived 0.78 of
// the launch on average, now 0.98 (2^18 walks x 16 steps: 3.96 -> 3.62 ms).
template <int WAVES, bool SPREAD>
__device__ void walk_block_pairs(const SpaceDev& sp, const WalkDev& wd, int iters, Lds<4, WAVES>& L, int64_t block,
                                 int64_t nblocks, WalkCounts& cnt, uint32_t* next, Back* back) {
    // the wavefront's index made explicitly uniform, and with it the walks' numbers and states: they stay
    // in scalar registers (as lane values they took 60 vector registers)
    const int lane = threadIdx.x & 63, wave = (int)uniform32(threadIdx.x >> 6);
    const bool leader = lane == 0;
    uint32_t* limbs = L.limbs[wave];
    Back &ba = back[2 * wave], &bb = back[2 * wave + 1];  // every lane writes the same values
    uint32_t steps = 0, active = 0, dps = 0, ins = 0;  // frequent events in registers, as in walk_block_single
    const int64_t pairs = (wd.walks + 1) / 2;
    // of the block's, those in runs (at most 2^31 walks, and no more blocks than CUs: 32 bits hold both)
    const uint32_t whole = SPREAD ? (uint32_t)pairs / ((uint32_t)nblocks * WAVES) * WAVES : ~0u;
    for (;;) {
        uint32_t i = 0;
        if (leader) i = atomicAdd(next, 1u);
        i = uniform32(i);
        const int64_t q = i < whole ? ((int64_t)(i / WAVES) * nblocks + block) * WAVES + i % WAVES : i * nblocks + block;
        if (q >= pairs) break;
        const int64_t w0 = 2 * q, w1 = 2 * q + 1;
        const bool has_b = w1 < wd.walks;
        Trail sa, sb;
        load_state<true>(wd, w0, sa, ba);
        sb = sa;
        if (has_b) load_state<true>(wd, w1, sb, bb);
        const int total = has_b ? 2 * iters : iters;
        int left = total;
        while (left > 0) {
            const bool act_a = (sa.mode & 0xff) != MODE_DONE;
            const bool act_b = has_b && (sb.mode & 0xff) != MODE_DONE;
            if (!act_a && !act_b) break;
            const uint64_t arg_a = step_arg<true>(sa, ba), arg_b = has_b ? step_arg<true>(sb, bb) : arg_a;
            const bool s1a = (arg_a >> 32) & 1, s1b = (arg_b >> 32) & 1;
            uint64_t na = 0, ha = 0, nb = 0, hb = 0;
            bool do_a, do_b;
            if (act_a && act_b && s1a && s1b && left >= 2) {
                walk_step_pair4<WAVES>(sp, L, limbs, arg_a, arg_b, lane, na, ha, nb, hb);
                do_a = do_b = true;
                left -= 2;
            } else {
                // a side-0 step first; otherwise the one walk still stepping (or walk a, on the last step)
                const bool pick_b = !act_a || (act_b && s1a && !s1b);
                uint64_t nx, hh;
                walk_step<4, WAVES>(sp, L, limbs, pick_b ? arg_b : arg_a, lane, 0, nx, hh);
                na = nb = nx;
                ha = hb = hh;
                do_a = !pick_b;
                do_b = pick_b;
                left -= 1;
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (!(k ? do_b : do_a)) continue;
                Trail st = k ? sb : sa;
                const uint32_t ev =
                    advance_walk<true>(sp, wd, st, k ? bb : ba, k ? w1 : w0, k ? arg_b : arg_a, k ? nb : na, k ? hb : ha, leader, 0);
                dps += ev & EV_DP;
                ins += (ev >> 1) & 1;
                const uint32_t rare = ev & ~(uint32_t)(EV_DP | EV_INS);
                if (rare && leader) count_events(cnt, rare);
                if (k)
                    sb = st;
                else
                    sa = st;
            }
        }
        steps += (uint32_t)(total - left);
        if ((sa.mode & 0xff) != MODE_DONE) active++;
        if (has_b && (sb.mode & 0xff) != MODE_DONE) active++;
        if (leader) {
            store_state(wd, w0, sa, ba);
            if (has_b) store_state(wd, w1, sb, bb);
        }
    }
    if (leader) {
        cnt.steps += steps;
        cnt.active += active;
        cnt.dps += dps;
        cnt.ins += ins;
    }
}

// The walks of one slice: paired on side 1 at n = 4, one walk group at a time otherwise.
template <int NQ, int WAVES, bool SPREAD>
__device__ void walk_block(const SpaceDev& sp, const WalkDev& wd, int iters, Lds<NQ, WAVES>& L, int64_t block,
                           int64_t nblocks, WalkCounts& cnt, uint32_t* next, Back* back) {
    if constexpr (NQ == 4)
        walk_block_pairs<WAVES, SPREAD>(sp, wd, iters, L, block, nblocks, cnt, next, back);
    else
        walk_block_single<NQ, WAVES>(sp, wd, iters, L, block, nblocks, cnt);
}

template <int NQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_walk(SpaceDev sp, WalkDev wd, int iters) {
    __shared__ Lds<NQ, WAVES> L;
    constexpr int GROUPS = WAVES * Geo<NQ>::WPW;
    __shared__ uint64_t s_cnt[GROUPS * ST_COUNT];
    const int group = (int)(threadIdx.x >> 6) * Geo<NQ>::WPW + (int)(threadIdx.x & 63) / Geo<NQ>::G;
    WalkCounts& mine = reinterpret_cast<WalkCounts*>(s_cnt)[group];
    __shared__ uint32_t s_pair;
    __shared__ Back s_back[NQ == 4 ? 2 * WAVES : 1];
    for (int i = threadIdx.x; i < GROUPS * ST_COUNT; i += blockDim.x) s_cnt[i] = 0;
    if (threadIdx.x == 0) s_pair = 0;
    load_lds(L, sp);
    __syncthreads();
    walk_block<NQ, WAVES, true>(sp, wd, iters, L, blockIdx.x, gridDim.x, mine, &s_pair, s_back);
    __syncthreads();
    flush_counts(wd, s_cnt, GROUPS);
}

// Many members in one persistent launch per qubit count, fed from a device queue: each block takes
// the next item (a slice of one member's walks for that member's number of evaluations) until the
// queue is empty, and reloads the member's S_c and keys into LDS only when the member changes.
// head[0] is the queue position (zeroed by a kernel before the launch); count[0] items are queued.
// Every block leaves once the position passes the count, so the grid always drains.
template <int NQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_walk_queue(const SpaceDev* __restrict__ sps, const WalkDev* __restrict__ wds,
                                                           const WorkItem* __restrict__ items, const int32_t* count,
                                                           uint32_t* head) {
    __shared__ Lds<NQ, WAVES> L;
    __shared__ int32_t s_next;
    __shared__ uint32_t s_pair;
    __shared__ Back s_back[NQ == 4 ? 2 * WAVES : 1];
    // the loaded member's event counts so far, one slot per walk group, written by the group's leader
    // as events happen (in registers they would hold 22 more VGPRs through the step and spill)
    constexpr int GROUPS = WAVES * Geo<NQ>::WPW;
    __shared__ uint64_t s_cnt[GROUPS * ST_COUNT];
    const int32_t n_items = *count;
    const int group = (int)(threadIdx.x >> 6) * Geo<NQ>::WPW + (int)(threadIdx.x & 63) / Geo<NQ>::G;
    WalkCounts& mine = reinterpret_cast<WalkCounts*>(s_cnt)[group];
    for (int i = threadIdx.x; i < GROUPS * ST_COUNT; i += blockDim.x) s_cnt[i] = 0;  // read after the first barrier
    int32_t loaded = -1;
    for (;;) {
        if (threadIdx.x == 0) {
            s_next = (int32_t)atomicAdd(head, 1u);
            s_pair = 0;
        }
        __syncthreads();
        // the same value in every thread of the block; read from the first lane so that the item and
        // the member's descriptors are scalar loads
        const int32_t i = __builtin_amdgcn_readfirstlane(s_next);
        if (i >= n_items) break;
        const WorkItem it = items[i];
        // read through the pointer where used (scalar loads; the descriptors are never written during
        // the launch, which __restrict__ tells the compiler, so it may keep or reload them freely)
        const SpaceDev& sp = sps[it.slot];
        if (it.slot != loaded) {
            if (loaded >= 0) flush_counts(wds[loaded], s_cnt, GROUPS);
            load_lds(L, sp);
            loaded = it.slot;
        }
        __syncthreads();
        walk_block<NQ, WAVES, false>(sp, wds[it.slot], it.iters, L, it.unit, it.units, mine, &s_pair, s_back);
        __syncthreads();  // s_next and, for the next member, the LDS are rewritten after this
    }
    if (loaded >= 0) flush_counts(wds[loaded], s_cnt, GROUPS);  // the last item's closing barrier is past
}

__global__ void k_walk_init(SpaceDev sp, WalkDev wd) {
    for (int64_t w = threadIdx.x + (int64_t)blockIdx.x * blockDim.x; w < wd.walks;
         w += (int64_t)blockDim.x * gridDim.x) {
        WalkState st;
        st.trail = 0;
        st.len = 0;
        st.mode = MODE_WALK;
        st.rem = 0;
        st.pa = st.pb = st.na = st.ha = 0;
        if (wd.enumerate) {
            const uint64_t idx = (uint64_t)w;
            if (idx >= wd.n_points) {
                st.mode = MODE_DONE;
                st.start = 0;
            } else {
                st.start = (idx % sp.n_half) | ((idx / sp.n_half) << 32);
            }
        } else {
            st.start = start_point(sp, (uint64_t)w, 0);
        }
        st.cur = st.start;
        wd.states[w] = st;
    }
}

// Several batch members restarted in one launch: for member slots[blockIdx.x / RESTART_PER], its
// table cleared (EMPTY_KEY keys; values 0, or ENUM_TABLE_INIT in enumeration mode), its statistics
// and candidate count zeroed and its walk states set as k_walk_init sets them; RESTART_PER blocks
// share each member's work.
constexpr int RESTART_PER = 32;
__global__ __launch_bounds__(256) void k_member_restart(const SpaceDev* sps, const WalkDev* wds,
                                                        const int32_t* slots) {
    const int32_t slot = slots[blockIdx.x / RESTART_PER];
    const SpaceDev sp = sps[slot];
    const WalkDev wd = wds[slot];
    const uint64_t stride = (uint64_t)RESTART_PER * blockDim.x;
    const uint64_t first = (uint64_t)(blockIdx.x % RESTART_PER) * blockDim.x + threadIdx.x;
    const uint64_t value = wd.enumerate ? ENUM_TABLE_INIT : 0;
    const uint64_t nslots = 1ull << wd.log2_table;
    for (uint64_t i = first; i < nslots; i += stride) {
        wd.table[2 * i] = EMPTY_KEY;
        wd.table[2 * i + 1] = value;
    }
    for (uint64_t w = first; w < (uint64_t)wd.walks; w += stride) {
        WalkState st;
        st.trail = 0;
        st.len = 0;
        st.mode = MODE_WALK;
        st.rem = 0;
        st.pa = st.pb = st.na = st.ha = 0;
        if (wd.enumerate) {
            if (w >= wd.n_points) {
                st.mode = MODE_DONE;
                st.start = 0;
            } else {
                st.start = (w % sp.n_half) | ((w / sp.n_half) << 32);
            }
        } else {
            st.start = start_point(sp, w, 0);
        }
        st.cur = st.start;
        wd.states[w] = st;
    }
    if (first < ST_COUNT) wd.stats[first] = 0;
    if (first == 0) *wd.claw_count = 0;
}

__global__ void k_table_clear(uint64_t* table, uint64_t slots, uint64_t value) {
    for (uint64_t i = threadIdx.x + (uint64_t)blockIdx.x * blockDim.x; i < slots;
         i += (uint64_t)blockDim.x * gridDim.x) {
        table[2 * i] = EMPTY_KEY;
        table[2 * i + 1] = value;
    }
}

// After an exhaustive pass (enumeration mode): every key reached from both sides gives one
// candidate, the least x of side 0 against the least x of side 1.
__device__ inline void enum_pairs(const WalkDev& wd, uint64_t first, uint64_t stride) {
    const uint64_t slots = 1ull << wd.log2_table;
    unsigned long long found = 0;
    for (uint64_t i = first; i < slots; i += stride) {
        if (wd.table[2 * i] == EMPTY_KEY) continue;
        const uint64_t v = wd.table[2 * i + 1];
        const uint32_t x0 = (uint32_t)v, x1 = (uint32_t)(v >> 32);
        if (x0 == ENUM_NONE || x1 == ENUM_NONE) continue;
        ++found;
        const unsigned long long idx = atomicAdd(wd.claw_count, 1ull);
        if (idx < wd.claw_cap) {
            wd.claws[2 * idx] = (uint64_t)x0;
            wd.claws[2 * idx + 1] = (uint64_t)x1 | (1ull << 32);
        }
    }
    if (found) atomicAdd(&wd.stats[ST_CLAWS], found);
}
__global__ void k_enum_pairs(WalkDev wd) {
    enum_pairs(wd, threadIdx.x + (uint64_t)blockIdx.x * blockDim.x, (uint64_t)blockDim.x * gridDim.x);
}
// the same for batch member slots[blockIdx.x / per], per blocks each
__global__ __launch_bounds__(256) void k_member_pairs(const WalkDev* wds, const int32_t* slots, int per) {
    const WalkDev wd = wds[slots[blockIdx.x / (unsigned)per]];
    enum_pairs(wd, (uint64_t)(blockIdx.x % (unsigned)per) * blockDim.x + threadIdx.x, (uint64_t)per * blockDim.x);
}

// ---- meet-in-the-middle labels for the depth-order network ----
// Level table: key = matrix hash H (one salt for every h), value = 255 - (least h that reaches it).
__device__ inline int level_lookup(const uint64_t* table, int log2_table, uint64_t key) {
    const uint64_t mask = (1ull << log2_table) - 1;
    uint64_t s = mix64(key ^ 0x5bd1e9955bd1e995ull) & mask;
    for (int probe = 0; probe < 64; ++probe) {
        const uint64_t k = __hip_atomic_load(&table[2 * s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (k == key) {
            const uint64_t v = __hip_atomic_load(&table[2 * s + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return v ? 255 - (int)v : -1;
        }
        if (k == EMPTY_KEY) return -1;
        s = (s + 1) & mask;
    }
    return -1;
}

// Which products of rotations a level needs.  R(p_0) R(p_1) ... with two commuting neighbours equals the
// product with them swapped, so only p_t < p_{t+1} is kept; with two equal neighbours R(p)^2 is a
// Clifford, so the same left coset appears two levels lower on the identity's side, and on the
// target's side (where that Clifford moves to the far right and through the identity's half) its
// match does.  Sorting commuting neighbours ends, so each class keeps a member: at n = 3 about 47 of
// the 63 choices for each next rotation.
__device__ inline bool keep_pair(uint32_t p0, uint32_t p1, bool anti) { return anti || p0 < p1; }

// n <= 2: one walk group per product, as in the walk kernels.
template <int NQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_mitm_levels(SpaceDev sp, int h, uint64_t* table, int log2_table) {
    using Gm = Geo<NQ>;
    __shared__ Lds<NQ, WAVES> L;
    load_lds(L, sp);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    uint32_t* limbs = L.limbs[wave * Gm::WPW + gi];
    sp.h = h;
    const int64_t stride = (int64_t)gridDim.x * WAVES * Gm::WPW;
    for (int64_t base = ((int64_t)blockIdx.x * WAVES + wave) * Gm::WPW; base < (int64_t)sp.n_half; base += stride) {
        const int64_t x = base + gi;
        if (x >= (int64_t)sp.n_half) continue;
        uint64_t o, H;
        walk_step<NQ, WAVES>(sp, L, limbs, (uint64_t)x, gl, gbase, o, H);
        if (gl == 0) {
            const uint64_t key = H == EMPTY_KEY ? (H ^ 1) : H;
            uint64_t slot = 0;
            WalkDev wd{};
            wd.table = table;
            wd.log2_table = log2_table;
            if (table_claim(wd, key, slot) != 3) atomicMax(&table[2 * slot + 1], (uint64_t)(255 - h));
        }
    }
}

// Per target: least i + j over side-1 products of j <= h_max rotations from U whose hash is in the level
// table at level i; stops once j reaches the best total.  blockIdx.y shares a target's products between
// the blocks of one column; best_out starts at -1 (none), which as unsigned is above every total.
template <int NQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 4) void k_mitm_probe(SpaceDev sp0, const uint32_t* phi_all,
                                                           const int32_t* rot_e_all, int count, int h_max,
                                                           const uint64_t* table, int log2_table, int32_t* best_out) {
    using Gm = Geo<NQ>;
    constexpr int NPHI = Gm::Q4 * Gm::R;
    __shared__ Lds<NQ, WAVES> L;
    __shared__ uint32_t best;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    uint32_t* limbs = L.limbs[wave * Gm::WPW + gi];
    for (int t = blockIdx.x; t < count; t += gridDim.x) {
        SpaceDev sp = sp0;
        sp.phi = phi_all + (size_t)t * 2 * NPHI;
        sp.rot_e = rot_e_all[t];
        __syncthreads();
        load_lds(L, sp);
        if (threadIdx.x == 0) best = ~0u;
        __syncthreads();
        uint32_t nh = 1, so_far = ~0u;
        for (int j = 0; j <= h_max; ++j) {
            if ((uint32_t)j >= so_far) break;
            sp.h = j;
            sp.n_half = nh;
            for (int64_t base = ((int64_t)blockIdx.y * WAVES + wave) * Gm::WPW; base < (int64_t)nh;
                 base += (int64_t)gridDim.y * WAVES * Gm::WPW) {
                const int64_t x = base + gi;
                if (x >= (int64_t)nh) continue;
                uint64_t o, H;
                walk_step<NQ, WAVES>(sp, L, limbs, (uint64_t)x | (1ull << 32), gl, gbase, o, H);
                if (gl == 0) {
                    const int lvl = level_lookup(table, log2_table, H == EMPTY_KEY ? (H ^ 1) : H);
                    if (lvl >= 0) atomicMin(&best, (uint32_t)(j + lvl));
                }
            }
            nh *= Gm::XI;
            // read between two barriers: a level's wavefronts have all stopped changing it and the next level's
            // have not begun, so the block leaves the loop together
            __syncthreads();
            so_far = best;
            __syncthreads();
        }
        if (threadIdx.x == 0 && best != ~0u) atomicMin(reinterpret_cast<uint32_t*>(&best_out[t]), best);
    }
}

// ---- n = 3: both halves by families of products that share all but their last-applied rotation ----
// A wavefront takes one prefix (p_1, ..., p_{j-1}) and every p_0 that the pruning keeps: all 63 at j = 1, at most 62
// beyond.

// Row r = lane of the n = 3 butterflies: bit p of anti = P_p and P_r anticommute, bit p of plus = the
// butterfly of R (side 0) adds the partner; ROT3_TAB with the Paulis of a row side by side.
struct Rot3Masks {
    uint64_t anti[64], plus[64];
};
constexpr Rot3Masks make_rot3_masks() {
    Rot3Masks t{};
    constexpr Rot3Tab tab = make_rot3_tab();
    for (int r = 0; r < 64; ++r)
        for (int p = 1; p < 64; ++p) {
            t.anti[r] |= (uint64_t)(tab.v[p * 64 + r] & 1) << p;
            t.plus[r] |= (uint64_t)((tab.v[p * 64 + r] >> 1) & 1) << p;
        }
    return t;
}
__device__ constexpr Rot3Masks ROT3_MASKS = make_rot3_masks();

__device__ inline void rot3_masks(int lane, uint64_t& anti, uint64_t& plus) {
    anti = ROT3_MASKS.anti[lane];
    plus = ROT3_MASKS.plus[lane];
}

// one rotation of rotate1 at n = 3, p uniform
__device__ inline uint64_t rot3(uint64_t u, uint32_t p, uint64_t anti, uint64_t plus, int lane) {
    const uint64_t part = shfl64(u, lane ^ (int)p);
    const uint64_t q = ((plus >> p) & 1) ? part : (2 * P61 - part);
    const uint64_t sum = u + q;
    const uint64_t rot = (sum >> 31) + ((sum & 0x7fffffffull) << 30);
    return ((anti >> p) & 1) ? rot : u;
}

// p_1 .. p_{j-1} of prefix y (p[1] first), and the p_0 that may stand before them (bit p; bit 0 alone for
// the product of no rotation).  0: the prefix is pruned.
__device__ inline uint64_t prefix3(uint32_t y, int j, uint32_t* p) {
    constexpr int HMAX = Geo<3>::HMAX;
    if (j == 0) return 1;
#pragma unroll
    for (int t = 1; t < HMAX; ++t) {
        p[t] = y % Geo<3>::XI + 1;
        y /= Geo<3>::XI;
    }
    bool keep = true;
#pragma unroll
    for (int t = 1; t + 1 < HMAX; ++t)
        if (t + 1 < j) keep = keep && keep_pair(p[t], p[t + 1], anticommutes<3>(p[t], p[t + 1]) != 0);
    if (!keep) return 0;
    uint64_t m = ~1ull;
    if (j >= 2) {
        const uint32_t lane = threadIdx.x & 63;
        m = __ballot(lane != 0 && keep_pair(lane, p[1], anticommutes<3>(lane, p[1]) != 0));
    }
    return m;
}

// the next p_0 of a prefix's products, 0 after the last
__device__ inline uint32_t next_product(uint64_t& todo) {
    const uint32_t p0 = todo ? (uint32_t)__builtin_ctzll(todo) : 0u;
    todo &= todo - 1;
    return p0;
}

// The keys through the prefix's rotations (side 0: R, side 1: R^T), p_{j-1} first.
__device__ inline uint64_t prefix_keys3(uint64_t u, const uint32_t* p, int j, uint64_t anti, uint64_t plus, int lane) {
#pragma unroll
    for (int t = Geo<3>::HMAX - 1; t >= 1; --t)
        if (t < j) u = rot3(u, p[t], anti, plus, lane);
    return u;
}

// The level table's first look: the same row digests in the field of p31 = 2^31 - 1 elements (sqrt2 -> 2^16,
// a square root of 2 there; 1/sqrt2 -> 2^15), half the words of the hash's field.  Products whose first
// hash finds no entry with its tag are done; one that does is looked up by its full hash, so what counts as
// a match is decided by the full hash alone (equal cosets have equal first hashes, whatever their rows' order and
// signs).
constexpr uint32_t P31 = 0x7fffffffu;

// x mod p31 for x < 2^32 - 1, in [0, p31]
__device__ inline uint32_t fold31(uint32_t x) { return (x & P31) + (x >> 31); }

// a key of the hash's field as one of this field
__device__ inline uint32_t key31(uint64_t k) {
    return fold31(fold31((uint32_t)k & P31) + fold31((uint32_t)(k >> 31)));
}

// rot3 here: u and the partner in [0, p31], and so the result
__device__ inline uint32_t rot31(uint32_t u, uint32_t p, uint64_t anti, uint64_t plus, int lane) {
    const uint32_t part = shfl32(u, lane ^ (int)p);
    const uint32_t sum = u + (((plus >> p) & 1) ? part : P31 - part);
    const uint32_t rot = fold31(((sum & 0xffffu) << 15) + (sum >> 16));  // below 2^31 + 2^16 before the fold
    return ((anti >> p) & 1) ? rot : u;
}
__device__ inline uint32_t prefix_keys31(uint32_t u, const uint32_t* p, int j, uint64_t anti, uint64_t plus, int lane) {
#pragma unroll
    for (int t = Geo<3>::HMAX - 1; t >= 1; --t)
        if (t < j) u = rot31(u, p[t], anti, plus, lane);
    return u;
}

// an element of the first hash: of a digest c in [0, p31] and its negative the smaller (0 for p31)
__device__ inline uint64_t digest_map31(uint32_t c, uint32_t ka, uint32_t kb) {
    const uint32_t m = min(c, P31 - c);
    return (uint64_t)(m + ka) * (uint64_t)(m ^ kb);
}

// A table entry's value: the tag of its first hash over 255 - (least h that reaches it).
__device__ inline uint64_t level_value(uint64_t h31, int h) { return (h31 & ~255ull) | (uint64_t)(255 - h); }

// The level of the entry with this first hash, or -1; with a key also that full hash is asked for.
__device__ inline int level_lookup31(const uint64_t* table, int log2_table, uint64_t h31, bool full, uint64_t key) {
    const uint64_t mask = (1ull << log2_table) - 1;
    uint64_t s = (h31 >> 8) & mask;
    for (int probe = 0; probe < 64; ++probe) {
        const uint64_t k = __hip_atomic_load(&table[2 * s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t v = __hip_atomic_load(&table[2 * s + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (k == EMPTY_KEY) return -1;
        if (full ? k == key : ((v ^ h31) & ~255ull) == 0) return 255 - (int)(v & 255);
        s = (s + 1) & mask;
    }
    return -1;
}

// v summed over the lane's 16-lane row
__device__ inline uint64_t row_sum16(uint64_t v) {
    v += dpp64<0xB1>(v);
    v += dpp64<0x4E>(v);
    v += dpp64<0x124>(v);
    v += dpp64<0x128>(v);
    return v;
}

// Level h of the table: four products at a time, whose wave sums share their last stages (two
// cross-half exchanges leave one product per 16-lane row), each kept by one lane; then every lane
// finishes and stores its own product, so that the table's atomics, each a round trip to memory, run 64
// at a time.  Bound by the butterfly, the element map and the sums (about 45 VALU instructions a
// product) with the pruned products left out: the 16 million products of levels 0..4 take 0.78 ms (0.97 with FIRST, the
// first hash beside the full one),
// against 4.85 ms with a wavefront per product and one lane at the table.
constexpr int MITM_WAVES = 4;
template <bool FIRST>
__global__ __launch_bounds__(MITM_WAVES * 64, 4) void k_mitm_levels3(SpaceDev sp, int h, uint32_t prefixes, uint64_t* table,
                                                                  int log2_table) {
    const int lane = threadIdx.x & 63;
    const uint32_t ka = (uint32_t)sp.salt_h, kb = (uint32_t)(sp.salt_h >> 32);
    uint64_t anti, plus;
    rot3_masks(lane, anti, plus);
    const uint64_t key0 = sp.keys[lane];
    const uint32_t key0_31 = key31(key0);
    WalkDev wd{};
    wd.table = table;
    wd.log2_table = log2_table;
    for (uint32_t y = uniform32(blockIdx.x * MITM_WAVES + (threadIdx.x >> 6)); y < prefixes;
         y += gridDim.x * MITM_WAVES) {
        uint32_t p[Geo<3>::HMAX] = {};
        uint64_t todo = prefix3(y, h, p);
        const int products = (int)__popcll(todo);
        if (products == 0) continue;
        const uint64_t u = prefix_keys3(key0, p, h, anti, plus, lane);
        uint32_t u31 = 0;
        if constexpr (FIRST) u31 = prefix_keys31(key0_31, p, h, anti, plus, lane);
        uint64_t mine = 0, mine31 = 0;
        for (int quad = 0; todo != 0; ++quad) {
            uint64_t acc[4], acc31[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t p0 = next_product(todo);
                const uint64_t v = p0 ? rot3(u, p0, anti, plus, lane) : u;
                acc[i] = digest_map(m61_fold(v), ka, kb);
                if constexpr (FIRST) acc31[i] = digest_map31(p0 ? rot31(u31, p0, anti, plus, lane) : u31, ka, kb);
            }
            // rows 0..3 of 16 lanes: products 0, 1, 2, 3
            const uint64_t sum = row_sum16(half_add16(half_add32(acc[0], acc[2]), half_add32(acc[1], acc[3])));
            if ((lane & 15) == quad) mine = sum;
            if constexpr (FIRST) {
                const uint64_t sum31 =
                    row_sum16(half_add16(half_add32(acc31[0], acc31[2]), half_add32(acc31[1], acc31[3])));
                if ((lane & 15) == quad) mine31 = sum31;
            }
        }
        if (4 * (lane & 15) + (lane >> 4) < products) {
            const uint64_t H = mix64(mine), key = H == EMPTY_KEY ? (H ^ 1) : H, h31 = mix64(mine31);
            uint64_t slot = 0;
            if ((FIRST ? table_claim_at(wd, key, h31 >> 8, slot) : table_claim(wd, key, slot)) != 3)
                atomicMax(&table[2 * slot + 1], FIRST ? level_value(h31, h) : (uint64_t)(255 - h));
        }
    }
}

// The target-side keys u = R(p_0)^T ... R(p_{j-1})^T K as MFMA A-operand fragments: a prefix's products in the
// order of their p_0, two per 16-row operand (rows 0..7 the signed base-256 digits of the first, rows 8..15
// of the second), K = [u | 2^31 u] in two steps.  Lane l of a fragment holds row l % 16, columns
// 16 (l / 16) .. + 15.  The digits meet in PairRows, one for each wavefront.
constexpr int PAIR_PITCH = 64 + 16;  // bytes of a row of 64 digits: 16-byte aligned, spread over the banks
struct PairRows {
    v4i rows[2 * 16 * PAIR_PITCH / 16];
};
// the products p of the prefix's keys u (p = 0: u itself)
__device__ inline void pair_frags3(PairRows& L, uint64_t u, const uint32_t (&p)[2], uint64_t anti, uint64_t plus, int lane,
                                   v4i& a0, v4i& a1) {
    uint8_t* at = reinterpret_cast<uint8_t*>(L.rows) + lane;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const uint64_t v = p[w] ? rot3(u, p[w], anti, plus, lane) : u;
#pragma unroll
        for (int set = 0; set < 2; ++set) {
            const uint64_t x = set ? (v >> 30) + ((v & 0x3fffffffull) << 31) : v;
            const uint64_t b = (x + 0x8080808080808080ull) ^ 0x8080808080808080ull;
#pragma unroll
            for (int m = 0; m < N4_DIG; ++m) at[(set * 16 + w * 8 + m) * PAIR_PITCH] = (uint8_t)(b >> (8 * m));
        }
    }
    wave_sync();
    const v4i* from = L.rows + (lane & 15) * (PAIR_PITCH / 16) + (lane >> 4);
    a0 = from[0];
    a1 = from[16 * (PAIR_PITCH / 16)];
    wave_sync();
}

// The first hash's fragments: four products to an operand, the signed base-256 digits of their keys in
// (-2^30, 2^30) as rows 4w .. 4w + 3, K = [u | 2^16 u].
__device__ inline void quad_frags31(PairRows& L, uint32_t u, const uint32_t (&p)[4], uint64_t anti, uint64_t plus,
                                    int lane, v4i& a0, v4i& a1) {
    uint8_t* at = reinterpret_cast<uint8_t*>(L.rows) + lane;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t v = p[w] ? rot31(u, p[w], anti, plus, lane) : u;
#pragma unroll
        for (int set = 0; set < 2; ++set) {
            // 2^16 v = a 2^31 + b 2^16 with v = a 2^15 + b
            const uint32_t x = set ? fold31(((v & 0x7fffu) << 16) + (v >> 15)) : v;
            const uint32_t c = x > (P31 >> 1) ? x - P31 : x;
            const uint32_t b = (c + 0x80808080u) ^ 0x80808080u;
#pragma unroll
            for (int m = 0; m < 4; ++m) at[(set * 16 + w * 4 + m) * PAIR_PITCH] = (uint8_t)(b >> (8 * m));
        }
    }
    wave_sync();
    const v4i* from = L.rows + (lane & 15) * (PAIR_PITCH / 16) + (lane >> 4);
    a0 = from[0];
    a1 = from[16 * (PAIR_PITCH / 16)];
    wave_sync();
}

// Many targets share these fragments (2 KiB a quad, 16 quads a prefix: MITM_PREFIX_V4 vectors), made once.  Bound
// by the stores.
constexpr int MITM_PREFIX_V4 = 16 * 2 * 64;
__global__ __launch_bounds__(MITM_WAVES * 64, 4) void k_mitm_keys3(SpaceDev sp, int j, uint32_t y0, uint32_t prefixes,
                                                                v4i* frags) {
    __shared__ PairRows L[MITM_WAVES];
    const int lane = threadIdx.x & 63, wave = (int)uniform32(threadIdx.x >> 6);
    uint64_t anti, plus;
    rot3_masks(lane, anti, plus);
    plus = ~plus;  // R^T: the butterfly adds where R subtracts
    for (uint32_t i = blockIdx.x; i < prefixes; i += gridDim.x) {
        uint32_t p[Geo<3>::HMAX] = {};
        uint64_t todo = prefix3(uniform32(y0 + i), j, p);
        if (todo == 0) continue;
        const uint32_t u = prefix_keys31(key31(sp.keys[lane]), p, j, anti, plus, lane);
        v4i* out = frags + (size_t)i * MITM_PREFIX_V4 + lane;
        const int quads = ((int)__popcll(todo) + 3) / 4;  // what no product fills repeats the prefix
        for (int q = 0; q < quads; ++q) {
            const uint32_t four[4] = {next_product(todo), next_product(todo), next_product(todo), next_product(todo)};
            if ((q & (MITM_WAVES - 1)) != wave) continue;
            v4i a0, a1;
            quad_frags31(L[wave], u, four, anti, plus, lane, a0, a1);
            out[q * 128] = a0;
            out[q * 128 + 64] = a1;
        }
    }
}

// Four products' first hash sums from one pass of 8 MFMAs: accumulator row 4g + i of lane l (g = l / 16) is digit
// i of product g in matrix row 16 nt + l % 16, |acc| <= 128 * 128 * 127 < 2^21.  s31: the target's exponent as
// a power of two, (2^15)^e = 2^s31.
__device__ inline uint64_t quad_sum31(const v4i a0, const v4i a1, const v4i* bf, uint32_t two_s31, uint32_t ka, uint32_t kb) {
    constexpr int64_t BIAS = (int64_t)P31 << 17;  // a multiple of p31 above every |digest|
    uint64_t sum = 0;
#pragma unroll
    for (int nt = 0; nt < N3_NT; ++nt) {
        v4i acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, bf[2 * nt], v4i{0, 0, 0, 0}, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, bf[2 * nt + 1], acc, 0, 0, 0);
        const int32_t x = acc[0] + acc[1] * 256, y = acc[2] + acc[3] * 256;  // below 2^30 in magnitude
        const uint64_t v = (uint64_t)((int64_t)y * 65536 + ((int64_t)x + BIAS));  // below 2^49
        const uint32_t r = ((uint32_t)v & P31) + (uint32_t)(v >> 31);  // below 2^31 + 2^18
        const uint64_t w = (uint64_t)r * two_s31;                       // below 2^61 + 2^48
        const uint32_t c = fold31(((uint32_t)w & P31) + (uint32_t)(w >> 31));  // below 2^31 + 2^30 + 2^17 before
        sum += digest_map31(c, ka, kb);
    }
    return sum;
}

// Two products' hash sums from one pass of 8 MFMAs: accumulator row 4g + i of lane l (g = l / 16) is
// digit 4 (g & 1) + i of product g >> 1 in matrix row 16 nt + l % 16, |acc| <= 128 * 128 * 127.  The swap of
// 16-lane rows between the tiles nt and nt + 2 leaves every lane all eight digits of one row.
__device__ inline uint64_t pair_sum3(const v4i a0, const v4i a1, const v4i* bf, uint32_t s, uint32_t ka, uint32_t kb) {
    int32_t lo[N3_NT], hi[N3_NT];
#pragma unroll
    for (int nt = 0; nt < N3_NT; ++nt) {
        v4i acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, bf[2 * nt], v4i{0, 0, 0, 0}, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, bf[2 * nt + 1], acc, 0, 0, 0);
        lo[nt] = acc[0] + acc[1] * 256;
        hi[nt] = acc[2] + acc[3] * 256;
    }
    uint64_t sum = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        sum += digest_map(digest_of(swap_rows16(lo[i], lo[2 + i]), swap_rows16(hi[i], hi[2 + i]), s), ka, kb);
    return sum;
}

// Probes of `count` targets against the level table, products of j rotations of prefixes y0 ..
// y0 + prefixes - 1 (frags from k_mitm_keys3).  A wavefront keeps its target's packed U as eight B
// fragments in registers and shares the target's prefixes with the `slices` wavefronts of the same
// target; four products fill the four 16-lane rows, as in k_mitm_levels3, and 64 lanes look up
// at a time.  A target that an earlier level has answered is skipped, and one hit ends its level (each
// wavefront looks after every prefix): every coset of T-count <= h_id is tabled, so the first level with
// a hit is T - h_id (or 0) and its total T.  The wavefronts are ordered by slice, then target, so that
// a hit in one slice spares the target's later ones, and wavefronts that run together read the same
// prefixes.
// MAKE (few targets): by the full hash, the wavefront's own fragments.  Else by the first hash from stored
// fragments, and the full hash of what it finds: half the instructions and MFMAs a product (39 and four by
// the full hash alone, VALU-bound at 0.64 busy).  16384 circuits against the table of T-count <= 4: 2.1 ms, 3.1
// by the full hash alone (4.35 with its accumulators in AGPRs, a copied fragment set and each target's two
// wavefronts side by side: the second launch bound's 128 registers keep the accumulators in VGPRs).  One
// target's 142 thousand products of <= 3 rotations: 0.05 ms.
template <bool MAKE>
__global__ __launch_bounds__(MITM_WAVES * 64, 4) void k_mitm_probe3(SpaceDev sp, const v4i* __restrict__ phi_all,
                                                                 const int32_t* __restrict__ rot_e_all, int count,
                                                                 int j, uint32_t y0, uint32_t prefixes, int slices,
                                                                 const v4i* __restrict__ frags, const uint64_t* table,
                                                                 int log2_table, int32_t* best_out) {
    const int lane = threadIdx.x & 63;
    const int64_t unit = uniform32(blockIdx.x * MITM_WAVES + (threadIdx.x >> 6));
    const int t = (int)(unit % count), slice = (int)(unit / count);
    if (slice >= slices) return;
    uint32_t* best = reinterpret_cast<uint32_t*>(&best_out[t]);
    if (uniform32(__hip_atomic_load(best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != ~0u) return;
    const uint32_t ka = (uint32_t)sp.salt_h, kb = (uint32_t)(sp.salt_h >> 32);
    v4i bf[N3_NT * N3_KK];
#pragma unroll
    for (int i = 0; i < N3_NT * N3_KK; ++i) bf[i] = phi_all[((size_t)t * N3_NT * N3_KK + i) * 64 + lane];
    const uint32_t s = uniform32((uint32_t)rot_e_all[t]);
    // the exponent e from 30 e mod 61 (59 is 30's inverse there; e < 61 for int8 entries)
    const uint32_t two_s31 = 1u << (15u * (s * 59u % 61u) % 31u);
    __shared__ PairRows L[MITM_WAVES];
    PairRows& rows = L[threadIdx.x >> 6];
    uint64_t anti, plus;
    rot3_masks(lane, anti, plus);
    plus = ~plus;  // R^T
    const uint64_t key0 = sp.keys[lane];
    for (uint32_t y = (uint32_t)slice; y < prefixes; y += (uint32_t)slices) {
        uint32_t p[Geo<3>::HMAX] = {};
        const uint64_t all = prefix3(uniform32(y0 + y), j, p);
        const int products = (int)__popcll(all);
        if (products == 0) continue;
        const int quads = (products + 3) / 4;
        uint64_t mine = 0;
        if constexpr (MAKE) {
            uint64_t todo = all;
            const uint64_t u = prefix_keys3(key0, p, j, anti, plus, lane);
            for (int quad = 0; quad < quads; ++quad) {
                uint64_t pair[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint32_t two[2] = {next_product(todo), next_product(todo)};
                    v4i a0, a1;
                    pair_frags3(rows, u, two, anti, plus, lane, a0, a1);
                    pair[i] = pair_sum3(a0, a1, bf, s, ka, kb);
                }
                // 32-lane halves hold the two products of a pair; after the exchange row g of 16 lanes holds
                // product 0, 2, 1, 3 of the quad
                const uint64_t sum = row_sum16(half_add16(pair[0], pair[1]));
                if ((lane & 15) == quad) mine = sum;
            }
            const int g = lane >> 4, in_quad = ((g & 1) << 1) | (g >> 1);
            int lvl = -1;
            if (4 * (lane & 15) + in_quad < products) {
                const uint64_t H = mix64(mine);
                lvl = level_lookup(table, log2_table, H == EMPTY_KEY ? (H ^ 1) : H);
            }
            if (lvl >= 0) atomicMin(best, (uint32_t)(j + lvl));
            if (__ballot(lvl >= 0) != 0) return;
            if (uniform32(__hip_atomic_load(best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != ~0u) return;
            continue;
        }
        const auto work = [&](int quad, const v4i (&a)[2]) {
            const uint64_t sum = row_sum16(quad_sum31(a[0], a[1], bf, two_s31, ka, kb));
            if ((lane & 15) == quad) mine = sum;  // of product 4 quad + lane / 16
        };
        // the next quad's fragments are on their way while one is worked on: two register sets in turn, so
        // that none is copied to the other
        const v4i* f = frags + (size_t)y * MITM_PREFIX_V4 + lane;
        const auto fetch = [&](int quad, v4i (&to)[2]) {
            if (quad >= quads) return;
#pragma unroll
            for (int i = 0; i < 2; ++i) to[i] = f[quad * 128 + 64 * i];
        };
        v4i even[2], odd[2];
        fetch(0, even);
        for (int quad = 0; quad < quads; quad += 2) {
            fetch(quad + 1, odd);
            work(quad, even);
            if (quad + 1 >= quads) break;
            fetch(quad + 2, even);
            work(quad + 1, odd);
        }
        const int mine_at = 4 * (lane & 15) + (lane >> 4);
        const uint64_t h31 = mix64(mine);
        uint64_t found = __ballot(mine_at < products && level_lookup31(table, log2_table, h31, false, 0) >= 0);
        bool hit = false;
        while (found != 0) {
            // the whole wavefront takes the full hash of one such product
            const int l = (int)__builtin_ctzll(found);
            found &= found - 1;
            uint64_t rest = all;
            for (int i = 4 * (l & 15) + (l >> 4); i > 0; --i) rest &= rest - 1;
            const uint32_t p0 = next_product(rest), two[2] = {p0, p0};
            const uint64_t u = prefix_keys3(key0, p, j, anti, plus, lane);
            v4i a0, a1;
            pair_frags3(rows, u, two, anti, plus, lane, a0, a1);
            const uint64_t half = pair_sum3(a0, a1, bf, s, ka, kb);
            const uint64_t H = mix64(row_sum16(half_add16(half, half)));  // the same in every lane
            if (lane == l) {
                const int lvl = level_lookup31(table, log2_table, h31, true, H == EMPTY_KEY ? (H ^ 1) : H);
                if (lvl >= 0) {
                    atomicMin(best, (uint32_t)(j + lvl));
                    hit = true;
                }
            }
        }
        if (__ballot(hit) != 0) return;
        if (uniform32(__hip_atomic_load(best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != ~0u) return;
    }
}

template <typename F>
hipError_t dispatch_n(int n, F&& f) {
    switch (n) {
        case 1: return f.template operator()<1>();
        case 2: return f.template operator()<2>();
        case 3: return f.template operator()<3>();
        case 4: return f.template operator()<4>();
        default: return hipErrorInvalidValue;
    }
}

int cu_count(int device) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0)
        cus = 256;
    return cus;
}

}  // namespace

int walk_grid_blocks(int n, int device) {
    // one persistent block per CU for n = 4 (the int8 S_c fills most of the 160 KiB LDS); at n = 3 the
    // kernels' 66 and 69 VGPRs leave room for seven 4-wave blocks, of which six measured best: 2^16 walks
    // 2.35 steps a ns against 2.22 with five and 2.24 with seven, 2^20 walks 2.60 against 2.47 and 2.54; an
    // enumerated search's launches 102 and 119 us against 107 and 124 with five
    const int cus = cu_count(device);
    if (n == 3) return cus * 6;
    return n == 4 ? cus : cus * 4;
}

hipError_t keys_fill(int n, uint64_t seed, uint64_t* keys, hipStream_t s) {
    const int r = 1 << (2 * n);
    hipLaunchKernelGGL(k_keys, dim3((r + 255) / 256), dim3(256), 0, s, r, seed, keys);
    return hipGetLastError();
}

hipError_t rot_keys_fill(const uint64_t* keys, uint64_t* rkeys, hipStream_t s) {
    hipLaunchKernelGGL(k_rot_keys, dim3(512), dim3(256), 0, s, keys, rkeys);
    return hipGetLastError();
}

hipError_t rot_keys2_fill(const uint64_t* rkeys, uint64_t* rkeys2, hipStream_t s) {
    hipLaunchKernelGGL(k_rot_keys2, dim3(2 * 256 * 256), dim3(256), 0, s, rkeys, rkeys2);
    return hipGetLastError();
}

hipError_t launch_step(int n, const SpaceDev& sp, const uint64_t* in, uint64_t* out, uint64_t* hash, int64_t count,
                       hipStream_t s) {
    if (count <= 0) return hipSuccess;
    auto f = [&]<int NQ>() -> hipError_t {
        constexpr int W = WalkWaves<NQ>::value;
        const int64_t per_block = (int64_t)W * Geo<NQ>::WPW;
        int64_t blocks = (count + per_block - 1) / per_block;
        if (blocks > 4096) blocks = 4096;
        hipLaunchKernelGGL((k_step<NQ, W>), dim3((unsigned)blocks), dim3(W * 64), 0, s, sp, in, out, hash, count);
        return hipGetLastError();
    };
    return dispatch_n(n, f);
}

hipError_t launch_trails(int n, const SpaceDev& sp, const uint64_t* starts, int64_t count, uint32_t cap, uint64_t* dp,
                         uint32_t* len, unsigned int* queue, int device, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    auto f = [&]<int NQ>() -> hipError_t {
        constexpr int W = WalkWaves<NQ>::value;
        const int64_t per_block = (int64_t)W * Geo<NQ>::WPW;
        int64_t blocks = (count + per_block - 1) / per_block;
        if constexpr (NQ == 4) {
            // few trails: a block for each, so that they do not share a CU
            const int64_t cus = cu_count(device);
            blocks = count < cus ? count : cus;
            if (count < (1ll << 31)) {
                hipLaunchKernelGGL((k_trails4<W>), dim3((unsigned)blocks), dim3(W * 64), 0, s, sp, starts, count, cap,
                                   dp, len, queue);
                return hipGetLastError();
            }
        }
        if (blocks > 4096) blocks = 4096;
        hipLaunchKernelGGL((k_trails<NQ, W>), dim3((unsigned)blocks), dim3(W * 64), 0, s, sp, starts, count, cap,
                           dp, len);
        return hipGetLastError();
    };
    return dispatch_n(n, f);
}

hipError_t launch_starts(const SpaceDev& sp, int64_t w0, uint32_t j, int64_t count, uint64_t* out, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65535) blocks = 65535;
    hipLaunchKernelGGL(k_starts, dim3((unsigned)blocks), dim3(256), 0, s, sp, w0, j, count, out);
    return hipGetLastError();
}

hipError_t pack_phi_i32(int n, const int32_t* a, const int32_t* b, int64_t count, uint32_t* phi, int* flag,
                        hipStream_t s) {
    auto f = [&]<int NQ>() -> hipError_t {
        hipLaunchKernelGGL((k_pack_i32<NQ>), dim3(1024), dim3(256), 0, s, a, b, count, phi, flag);
        return hipGetLastError();
    };
    return dispatch_n(n, f);
}

hipError_t launch_canon_hash(int n, const SpaceDev& sp, const uint32_t* phi_all, const int32_t* e, int64_t count,
                             uint64_t* out, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    auto f = [&]<int NQ>() -> hipError_t {
        constexpr int W = WalkWaves<NQ>::value;
        const int64_t blocks = count < 1024 ? count : 1024;
        hipLaunchKernelGGL((k_canon<NQ, W>), dim3((unsigned)blocks), dim3(W * 64), 0, s, sp, phi_all, e, count,
                           out);
        return hipGetLastError();
    };
    return dispatch_n(n, f);
}

hipError_t launch_canon_wide(int n, const SpaceDev& sp, const int32_t* a, const int32_t* b, const int32_t* e,
                             int64_t count, uint64_t* out, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    auto f = [&]<int NQ>() -> hipError_t {
        const int64_t blocks = count < 4096 ? count : 4096;
        hipLaunchKernelGGL((k_canon_wide<NQ>), dim3((unsigned)blocks), dim3(64), 0, s, sp, a, b, e, count, out);
        return hipGetLastError();
    };
    return dispatch_n(n, f);
}

hipError_t launch_walk(int n, const SpaceDev& sp, const WalkDev& wd, int iters, int grid_blocks, hipStream_t s) {
    auto f = [&]<int NQ>() -> hipError_t {
        constexpr int W = WalkWaves<NQ>::value;
        const int64_t per_block = (int64_t)W * Geo<NQ>::WPW;
        // n = 4: a CU for each pair of walks while there are enough, so that they do not share one (64 walks x 64
        // steps, k = 5, theta = 2^-4: 209 us; with a block for every 16 walks, of which two had pairs, 340)
        int64_t blocks = NQ == 4 ? (wd.walks + 1) / 2 : (wd.walks + per_block - 1) / per_block;
        if (blocks > grid_blocks) blocks = grid_blocks;
        hipLaunchKernelGGL((k_walk<NQ, W>), dim3((unsigned)blocks), dim3(W * 64), 0, s, sp, wd, iters);
        return hipGetLastError();
    };
    return dispatch_n(n, f);
}

hipError_t launch_walk_queue(int n, const SpaceDev* sps, const WalkDev* wds, const WorkItem* items,
                             const int32_t* count, uint32_t* head, int blocks, hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    auto f = [&]<int NQ>() -> hipError_t {
        constexpr int W = WalkWaves<NQ>::value;
        hipLaunchKernelGGL((k_walk_queue<NQ, W>), dim3((unsigned)blocks), dim3(W * 64), 0, s, sps, wds, items, count,
                           head);
        return hipGetLastError();
    };
    return dispatch_n(n, f);
}

int walks_per_block(int n) {
    switch (n) {
        case 1: return WalkWaves<1>::value * Geo<1>::WPW;
        case 2: return WalkWaves<2>::value * Geo<2>::WPW;
        case 3: return WalkWaves<3>::value * Geo<3>::WPW;
        default: return WalkWaves<4>::value * Geo<4>::WPW;
    }
}

hipError_t launch_walk_init(const SpaceDev& sp, const WalkDev& wd, hipStream_t s) {
    int64_t blocks = (wd.walks + 255) / 256;
    if (blocks > 65535) blocks = 65535;
    hipLaunchKernelGGL(k_walk_init, dim3((unsigned)blocks), dim3(256), 0, s, sp, wd);
    return hipGetLastError();
}

hipError_t launch_member_restart(const SpaceDev* sps, const WalkDev* wds, const int32_t* slots, int count,
                                 hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_member_restart, dim3((unsigned)(count * RESTART_PER)), dim3(256), 0, s, sps, wds, slots);
    return hipGetLastError();
}

hipError_t launch_table_clear(uint64_t* table, int log2_table, uint64_t value, hipStream_t s) {
    const uint64_t slots = 1ull << log2_table;
    uint64_t blocks = (slots + 255) / 256;
    if (blocks > 65535) blocks = 65535;
    hipLaunchKernelGGL(k_table_clear, dim3((unsigned)blocks), dim3(256), 0, s, table, slots, value);
    return hipGetLastError();
}

// The scan is a chain of reads for each thread, so it wants a thread a slot, up to what fills the chip: the
// members of a launch share 4,096 blocks (as many as k_enum_pairs starts for one table), with at least 32 a
// member.  One member, 2^27 slots: 0.37 ms, with 32 blocks whatever the table's size 9.4; a depth's 63 chunks at
// n = 3 get 65 blocks each, its 255 at n = 4 32.
hipError_t launch_member_pairs(const WalkDev* wds, const int32_t* slots, int count, int log2_table, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const int64_t most = std::max<int64_t>(1, (int64_t)1 << std::max(0, log2_table - 8));
    const int per = (int)std::min<int64_t>(most, std::max(32, 4096 / count));
    hipLaunchKernelGGL(k_member_pairs, dim3((unsigned)count * per), dim3(256), 0, s, wds, slots, per);
    return hipGetLastError();
}

hipError_t launch_enum_pairs(const WalkDev& wd, hipStream_t s) {
    const uint64_t slots = 1ull << wd.log2_table;
    uint64_t blocks = (slots + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_enum_pairs, dim3((unsigned)blocks), dim3(256), 0, s, wd);
    return hipGetLastError();
}

}  // namespace tcw

namespace tcw {

// Up to MITM_MAKE targets are probed by the full hash alone and make their fragments themselves: the products of
// at most three rotations take 48 us for one target so, in one launch a level, and stored fragments of the
// full hash 79 to make and 45 to use.  More targets share stored fragments of the first hash, which the table
// then needs too: 0.97 ms instead of 0.78 for T-count <= 4, and 2.1 instead of 3.1 to probe 16384 circuits.
constexpr int MITM_MAKE = 4;
hipError_t mitm_levels(int n, const SpaceDev& sp, int h, int64_t count, uint64_t* table, int log2_table, hipStream_t s) {
    auto f = [&]<int NQ>() -> hipError_t {
        constexpr int W = WalkWaves<NQ>::value;
        if constexpr (NQ == 3) {
            const uint32_t prefixes = h == 0 ? 1 : sp.n_half / Geo<3>::XI;
            uint32_t blocks = (prefixes + MITM_WAVES - 1) / MITM_WAVES;
            if (blocks > 4096) blocks = 4096;
            if (count > MITM_MAKE)
                hipLaunchKernelGGL(k_mitm_levels3<true>, dim3(blocks), dim3(MITM_WAVES * 64), 0, s, sp, h, prefixes, table,
                                   log2_table);
            else
                hipLaunchKernelGGL(k_mitm_levels3<false>, dim3(blocks), dim3(MITM_WAVES * 64), 0, s, sp, h, prefixes, table,
                                   log2_table);
            return hipGetLastError();
        } else if constexpr (NQ <= 2) {
            int64_t blocks = ((int64_t)sp.n_half + W * Geo<NQ>::WPW - 1) / (W * Geo<NQ>::WPW);
            if (blocks > 4096) blocks = 4096;
            if (blocks < 1) blocks = 1;
            hipLaunchKernelGGL((k_mitm_levels<NQ, W>), dim3((unsigned)blocks), dim3(W * 64), 0, s, sp, h, table,
                               log2_table);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    };
    return dispatch_n(n, f);
}

// At n = 3 the fragments of at most MITM_CHUNK prefixes (64 KiB each) are held at a time.
constexpr uint32_t MITM_CHUNK = 1024;
static uint32_t mitm_prefixes(int j) {
    uint32_t v = 1;
    for (int i = 1; i < j; ++i) v *= Geo<3>::XI;
    return v;
}

size_t mitm_frag_bytes(int n, int h_max, int64_t count) {
    if (n != 3 || count <= MITM_MAKE) return 0;
    size_t all = 0;
    for (int j = 0; j <= h_max; ++j) all += mitm_prefixes(j);
    return std::min<size_t>(all, MITM_CHUNK) * MITM_PREFIX_V4 * sizeof(v4i);
}

// The wavefronts of k_mitm_probe3 that share a target: 32 rounds of the 4096 that the chip holds, one
// prefix each at least.  A label batch's targets end anywhere between their first product and the last
// (4096 at once, level 2: 16384 circuits take 3.89 ms with 8192 wavefronts, 3.49 with 16384, 3.22 with
// 32768, 3.09 with 131072); a single target has its prefixes one to a wavefront either way.
static int mitm_slices(int count, uint32_t prefixes) {
    const int64_t want = (131072 + count - 1) / count;
    return (int)std::max<int64_t>(1, std::min<int64_t>(want, prefixes));
}

static hipError_t mitm_keys(const SpaceDev& sp, int j, uint32_t y0, uint32_t prefixes, void* frags, hipStream_t s) {
    hipLaunchKernelGGL(k_mitm_keys3, dim3(prefixes), dim3(MITM_WAVES * 64), 0, s, sp, j, y0, prefixes, (v4i*)frags);
    return hipGetLastError();
}

static hipError_t mitm_probe3(const SpaceDev& sp, const uint32_t* phi_all, const int32_t* rot_e_all, int count, int j,
                              uint32_t y0, uint32_t prefixes, const void* frags, const uint64_t* table, int log2_table,
                              int32_t* best_out, hipStream_t s) {
    const int slices = mitm_slices(count, prefixes);
    const int64_t blocks = ((int64_t)count * slices + MITM_WAVES - 1) / MITM_WAVES;
    if (frags != nullptr)
        hipLaunchKernelGGL(k_mitm_probe3<false>, dim3((unsigned)blocks), dim3(MITM_WAVES * 64), 0, s, sp,
                           (const v4i*)phi_all, rot_e_all, count, j, y0, prefixes, slices, (const v4i*)frags, table,
                           log2_table, best_out);
    else
        hipLaunchKernelGGL(k_mitm_probe3<true>, dim3((unsigned)blocks), dim3(MITM_WAVES * 64), 0, s, sp,
                           (const v4i*)phi_all, rot_e_all, count, j, y0, prefixes, slices, (const v4i*)nullptr, table,
                           log2_table, best_out);
    return hipGetLastError();
}

hipError_t mitm_frags(int n, const SpaceDev& sp, int h_max, void* frags, hipStream_t s) {
    if (n != 3) return hipSuccess;
    uint32_t at = 0, all = 0;
    for (int j = 0; j <= h_max; ++j) all += mitm_prefixes(j);
    if (all > MITM_CHUNK) return hipSuccess;  // built chunk by chunk in mitm_probe
    for (int j = 0; j <= h_max; ++j) {
        const uint32_t m = mitm_prefixes(j);
        hipError_t e = mitm_keys(sp, j, 0, m, (v4i*)frags + (size_t)at * MITM_PREFIX_V4, s);
        if (e != hipSuccess) return e;
        at += m;
    }
    return hipSuccess;
}

hipError_t mitm_probe(int n, const SpaceDev& sp, const uint32_t* phi_all, const int32_t* rot_e_all, int count,
                      int h_max, void* frags, const uint64_t* table, int log2_table, int32_t* best_out, hipStream_t s) {
    hipError_t e = hipSuccess;
    if (n == 3) {
        uint32_t at = 0, all = 0;
        for (int j = 0; j <= h_max; ++j) all += mitm_prefixes(j);
        for (int j = 0; j <= h_max; ++j) {
            const uint32_t m = mitm_prefixes(j);
            if (frags == nullptr || all <= MITM_CHUNK) {
                const v4i* f = frags != nullptr ? (const v4i*)frags + (size_t)at * MITM_PREFIX_V4 : nullptr;
                e = mitm_probe3(sp, phi_all, rot_e_all, count, j, 0, m, f, table, log2_table, best_out, s);
                if (e != hipSuccess) return e;
                at += m;
                continue;
            }
            for (uint32_t y = 0; y < m; y += MITM_CHUNK) {
                const uint32_t c = std::min(MITM_CHUNK, m - y);
                e = mitm_keys(sp, j, y, c, frags, s);
                if (e == hipSuccess)
                    e = mitm_probe3(sp, phi_all, rot_e_all, count, j, y, c, frags, table, log2_table, best_out, s);
                if (e != hipSuccess) return e;
            }
        }
        return hipSuccess;
    }
    auto f = [&]<int NQ>() -> hipError_t {
        constexpr int W = WalkWaves<NQ>::value;
        if constexpr (NQ <= 2) {
            const int blocks = count < 4096 ? count : 4096;
            int64_t most = 1;  // products of the deepest level, a block's groups at a time
            for (int i = 0; i < h_max; ++i) most *= Geo<NQ>::XI;
            most = (most + W * Geo<NQ>::WPW - 1) / (W * Geo<NQ>::WPW);
            const int64_t slices = std::max<int64_t>(1, std::min<int64_t>(most, 1024 / blocks));
            hipLaunchKernelGGL((k_mitm_probe<NQ, W>), dim3(blocks, (unsigned)slices), dim3(W * 64), 0, s, sp, phi_all,
                               rot_e_all, count, h_max, table, log2_table, best_out);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    };
    return dispatch_n(n, f);
}

}  // namespace tcw
