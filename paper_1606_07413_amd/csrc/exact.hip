// Exact channel-representation arithmetic over Z[1/sqrt2] (Sec. 4.1) on the GPU.
//
// A matrix is M = (A + B sqrt2) / sqrt2^e with integer A, B (int64 for n <= 2, int32 for n >= 3)
// and minimal e.  Right multiplication by the channel rep of R(P_p) follows its sparse column
// rule: column q is e_q when <p, q> = 0, else (e_q + s(p, q) e_{p^q}) / sqrt2, so
//   (M R)[:, q] = (M[:, q] + s M[:, p^q]) / sqrt2        (anticommuting q)
//   (M R)[:, q] = (sqrt2 M[:, q]) / sqrt2, (a, b) -> (2b, a)   (commuting q)
// and R^T flips s.  These are set-up and verification paths (target preparation, chunk matrices S_c,
// claw checks), not the walk loop.
#include "common.h"
#include "internal.h"

namespace tcw {

namespace {

template <int NQ>
struct EGeo {
    static constexpr int R = 1 << (2 * NQ);
};

template <typename T>
__device__ inline T lim_of();
template <>
__device__ inline int32_t lim_of<int32_t>() { return (int32_t)1 << 29; }
template <>
__device__ inline int64_t lim_of<int64_t>() { return (int64_t)1 << 60; }

// (A, B, e) <- product with R(seq[0])^(T?) ... ; result left in (a, b).  Whole block cooperates.
template <int NQ, typename T>
__device__ void block_apply(T* a, T* b, T* ta, T* tb, int& e, const uint16_t* seq, const uint8_t* tr, int nseq,
                            int* flag) {
    constexpr int R = EGeo<NQ>::R;
    const T lim = lim_of<T>();
    T *ca = a, *cb = b, *na = ta, *nb = tb;
    for (int s = 0; s < nseq; ++s) {
        const uint32_t p = seq[s];
        const bool t = tr != nullptr && tr[s] != 0;
        for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) {
            const uint32_t q = idx & (R - 1);
            const int row = idx - (int)q;
            T va, vb;
            if (anticommutes<NQ>(p, q)) {
                int sg = rotation_sign<NQ>(p, q);
                if (t) sg = -sg;
                const int j = row + (int)(q ^ p);
                va = sg > 0 ? ca[idx] + ca[j] : ca[idx] - ca[j];
                vb = sg > 0 ? cb[idx] + cb[j] : cb[idx] - cb[j];
            } else {
                va = cb[idx] * 2;
                vb = ca[idx];
            }
            if (va > lim || va < -lim || vb > lim || vb < -lim) atomicOr(flag, 4);
            na[idx] = va;
            nb[idx] = vb;
        }
        __syncthreads();
        T* x = ca; ca = na; na = x;
        x = cb; cb = nb; nb = x;
        e += 1;
        // reduce: while every a is even, (a + b sqrt2)/sqrt2 = b + (a/2) sqrt2
        while (e > 0) {
            int odd = 0;
            for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) odd |= (int)(ca[idx] & 1);
            if (__syncthreads_or(odd)) break;
            for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) {
                const T va = ca[idx], vb = cb[idx];
                ca[idx] = vb;
                cb[idx] = va / 2;
            }
            e -= 1;
            __syncthreads();
        }
    }
    if (ca != a) {
        for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) {
            a[idx] = ca[idx];
            b[idx] = cb[idx];
        }
        __syncthreads();
    }
}

template <int NQ, typename T>
__device__ void block_reduce(T* a, T* b, int& e) {
    constexpr int R = EGeo<NQ>::R;
    while (e > 0) {
        int odd = 0;
        for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) odd |= (int)(a[idx] & 1);
        if (__syncthreads_or(odd)) break;
        for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) {
            const T va = a[idx], vb = b[idx];
            a[idx] = vb;
            b[idx] = va / 2;
        }
        e -= 1;
        __syncthreads();
    }
}

template <int NQ, typename T>
__global__ __launch_bounds__(1024) void k_identity(T* a, T* b, int32_t* e) {
    constexpr int R = EGeo<NQ>::R;
    for (int idx = threadIdx.x + blockIdx.x * blockDim.x; idx < R * R; idx += blockDim.x * gridDim.x) {
        const int r = idx / R, q = idx % R;
        a[idx] = (r == q) ? 1 : 0;
        b[idx] = 0;
    }
    if (threadIdx.x == 0 && blockIdx.x == 0) *e = 0;
}

template <int NQ, typename T>
__global__ __launch_bounds__(1024) void k_apply(T* a, T* b, T* ta, T* tb, int32_t* e_io, const T* sa, const T* sb,
                                                const int32_t* se, const uint16_t* seq, const uint8_t* tr, int nseq,
                                                int* flag) {
    constexpr int R = EGeo<NQ>::R;
    if (sa != a) {
        for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) {
            a[idx] = sa[idx];
            b[idx] = sb[idx];
        }
    }
    __syncthreads();
    int e = *se;
    __syncthreads();
    block_apply<NQ, T>(a, b, ta, tb, e, seq, tr, nseq, flag);
    if (threadIdx.x == 0) *e_io = e;
}

template <int NQ, typename T>
__global__ __launch_bounds__(1024) void k_from_i32(T* a, T* b, int32_t* e_io, const int32_t* ia, const int32_t* ib,
                                                   int32_t e0) {
    constexpr int R = EGeo<NQ>::R;
    for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) {
        a[idx] = (T)ia[idx];
        b[idx] = (T)ib[idx];
    }
    __syncthreads();
    int e = e0;
    block_reduce<NQ, T>(a, b, e);
    if (threadIdx.x == 0) *e_io = e;
}

template <int NQ, typename T>
__global__ void k_to_i32(const T* a, const T* b, int32_t* oa, int32_t* ob, int* flag) {
    constexpr int R = EGeo<NQ>::R;
    for (int idx = threadIdx.x + blockIdx.x * blockDim.x; idx < R * R; idx += blockDim.x * gridDim.x) {
        const T va = a[idx], vb = b[idx];
        if (va > (T)INT32_MAX || va < (T)INT32_MIN || vb > (T)INT32_MAX || vb < (T)INT32_MIN) atomicOr(flag, 4);
        oa[idx] = (int32_t)va;
        ob[idx] = (int32_t)vb;
    }
}

// X X^T = 2^e I with X = A + B sqrt2:  A A^T + 2 B B^T = 2^e I  and  A B^T + B A^T = 0.
template <int NQ, typename T>
__global__ void k_orthogonal(const T* a, const T* b, const int32_t* e_p, int* flag) {
    constexpr int R = EGeo<NQ>::R;
    const int idx = threadIdx.x + blockIdx.x * blockDim.x;
    if (idx >= R * R) return;
    const int i = idx / R, j = idx % R;
    const int e = *e_p;
    int64_t rat = 0, irr = 0;
    for (int k = 0; k < R; ++k) {
        const int64_t ai = a[i * R + k], bi = b[i * R + k], aj = a[j * R + k], bj = b[j * R + k];
        if (ai > (1 << 24) || ai < -(1 << 24) || bi > (1 << 24) || bi < -(1 << 24)) {
            atomicOr(flag, 4);
            return;
        }
        rat += ai * aj + 2 * bi * bj;
        irr += ai * bj + bi * aj;
    }
    const int64_t want = (i == j) ? ((e < 62) ? ((int64_t)1 << e) : -1) : 0;
    if (rat != want || irr != 0) atomicOr(flag, 1);
}

// ---- channel rep of an exact unitary (Sec. 4.1: U_hat_ij = 2^-n Tr(P_i U P_j U^dag)) ----
//
// U = V / sqrt2^e with V over Z[w], w = e^{i pi/4}, each entry four int64 coefficients of
// w^0..w^3 (w^4 = -1).  On the basis |c> (qubit 0 = most significant bit of c), the Pauli
// P_q = (x) sigma(x_j, z_j), sigma(x, z) = i^{xz} X^x Z^z, acts as
//   P_q |c> = i^{|x & z|} (-1)^{|z' & c|} |c ^ x'>,
// with x', z' the bit-reversed masks (qubit j on bit n-1-j).  Hence
//   Tr(P_i V P_j V^dag) = sum_{r,t} w^{k(r,t)} V[r ^ x_i'][t] conj(V[r][t ^ x_j'])
// with k = 2|x_i & z_i| + 4|z_i' & (r ^ x_i')| + 2|x_j & z_j| + 4|z_j' & (t ^ x_j')| (mod 8).
// The trace is real, t0 + t1 w + t2 w^2 + t3 w^3 with t2 = 0 and t3 = -t1, i.e. t0 + t1 sqrt2,
// and U_hat_ij = (t0 + t1 sqrt2) / sqrt2^(2(n + e)).

struct Zw {
    int64_t c[4];
};

__device__ inline Zw zw_load(const int64_t* p) { return Zw{{p[0], p[1], p[2], p[3]}}; }

__device__ inline Zw zw_mul_conj(const Zw& x, const Zw& y) {
    // x * conj(y), conj(y) = y0 - y3 w - y2 w^2 - y1 w^3
    const int64_t yc[4] = {y.c[0], -y.c[3], -y.c[2], -y.c[1]};
    Zw r{{0, 0, 0, 0}};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t v = x.c[i] * yc[j];
            if (i + j < 4) r.c[i + j] += v;
            else r.c[i + j - 4] -= v;
        }
    return r;
}

// acc += w^k x, k in 0..7
__device__ inline void zw_acc_rot(Zw& acc, const Zw& x, int k) {
    const int64_t sg = k >= 4 ? -1 : 1;
    const int kk = k & 3;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = i + kk;
        if (j < 4) acc.c[j] += sg * x.c[i];
        else acc.c[j - 4] -= sg * x.c[i];
    }
}

template <int NQ>
__device__ inline uint32_t bit_reverse_n(uint32_t v) {
    uint32_t r = 0;
#pragma unroll
    for (int j = 0; j < NQ; ++j) r |= ((v >> j) & 1u) << (NQ - 1 - j);
    return r;
}

// One thread per channel-rep entry (i, j).  flag |= 1 if an entry is not real, 4 if t0 or t1 leaves int32.
template <int NQ>
__global__ __launch_bounds__(256) void k_unitary_channel(const int64_t* v, int32_t* oa, int32_t* ob, int* flag) {
    constexpr int D = 1 << NQ;
    constexpr int R = D * D;
    __shared__ int64_t sv[D * D * 4];
    for (int x = threadIdx.x; x < D * D * 4; x += blockDim.x) sv[x] = v[x];
    __syncthreads();
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= R * R) return;
    const uint32_t i = (uint32_t)idx / R, j = (uint32_t)idx % R;
    const uint32_t xi = i & (D - 1), zi = i >> NQ, xj = j & (D - 1), zj = j >> NQ;
    const uint32_t xir = bit_reverse_n<NQ>(xi), zir = bit_reverse_n<NQ>(zi);
    const uint32_t xjr = bit_reverse_n<NQ>(xj), zjr = bit_reverse_n<NQ>(zj);
    const int k0 = 2 * __builtin_popcount(xi & zi) + 2 * __builtin_popcount(xj & zj);
    Zw acc{{0, 0, 0, 0}};
    for (uint32_t r = 0; r < (uint32_t)D; ++r) {
        const uint32_t s = r ^ xir;
        const int ks = k0 + 4 * __builtin_popcount(zir & s);
        for (uint32_t t = 0; t < (uint32_t)D; ++t) {
            const uint32_t u = t ^ xjr;
            const int k = (ks + 4 * __builtin_popcount(zjr & u)) & 7;
            const Zw prod = zw_mul_conj(zw_load(&sv[(s * D + t) * 4]), zw_load(&sv[(r * D + u) * 4]));
            zw_acc_rot(acc, prod, k);
        }
    }
    if (acc.c[2] != 0 || acc.c[3] != -acc.c[1]) atomicOr(flag, 1);
    if (acc.c[0] > INT32_MAX || acc.c[0] < INT32_MIN || acc.c[1] > INT32_MAX || acc.c[1] < INT32_MIN)
        atomicOr(flag, 4);
    oa[idx] = (int32_t)acc.c[0];
    ob[idx] = (int32_t)acc.c[1];
}

// V V^dag = 2^e I over Z[w], one thread per entry (r, c); flag |= 8 otherwise.
template <int NQ>
__global__ __launch_bounds__(256) void k_unitary_check(const int64_t* v, int32_t e, int* flag) {
    constexpr int D = 1 << NQ;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= D * D) return;
    const int r = idx / D, c = idx % D;
    Zw acc{{0, 0, 0, 0}};
    for (int t = 0; t < D; ++t) {
        const Zw prod = zw_mul_conj(zw_load(&v[(r * D + t) * 4]), zw_load(&v[(c * D + t) * 4]));
        zw_acc_rot(acc, prod, 0);
    }
    const int64_t want = r == c ? ((int64_t)1 << e) : 0;
    if (acc.c[0] != want || acc.c[1] != 0 || acc.c[2] != 0 || acc.c[3] != 0) atomicOr(flag, 8);
}

// Signed permutation test on a reduced matrix: e = 0, B = 0, each column one +-1.
template <int NQ, typename T>
__global__ __launch_bounds__(256) void k_signed_perm(const T* a, const T* b, const int32_t* e_p, int32_t* ok,
                                                     int32_t* perm, int8_t* sign) {
    constexpr int R = EGeo<NQ>::R;
    __shared__ int bad;
    if (threadIdx.x == 0) bad = (*e_p != 0);
    __syncthreads();
    for (int q = threadIdx.x; q < R; q += blockDim.x) {
        int cnt = 0, row = -1, sg = 0;
        for (int i = 0; i < R; ++i) {
            const T va = a[i * R + q], vb = b[i * R + q];
            if (vb != 0) cnt += 2;
            if (va != 0) {
                cnt += 1;
                row = i;
                sg = (va == 1) ? 1 : (va == -1 ? -1 : 0);
            }
        }
        if (cnt != 1 || sg == 0) atomicOr(&bad, 1);
        perm[q] = row;
        sign[q] = (int8_t)sg;
    }
    __syncthreads();
    if (threadIdx.x == 0) *ok = bad ? 0 : 1;
}

// int8 packing of S for the walk kernels: phi[q4 * R + r] = bytes A[r][4 q4 .. 4 q4 + 3] (then B).
// n >= 3 uses the MFMA fragment layout instead: with KK = 2R / 64 K steps and NT = R / 16 tiles,
// dword idx = ((nt * KK + kk) * 64 + l) * 4 + w holds the bytes S''[nt*16 + l%16][kk*64 + (l/16)*16 +
// 4w + c], c = 0..3, with S'' = [A | B] (R x 2R).
template <int NQ, typename T>
__global__ void k_pack_phi(const T* a, const T* b, uint32_t* phi, int* flag) {
    constexpr int R = EGeo<NQ>::R;
    constexpr int Q4 = R / 4;
    const int idx = threadIdx.x + blockIdx.x * blockDim.x;
    if constexpr (NQ >= 3) {
        constexpr int KK = 2 * R / 64;
        if (idx >= 2 * Q4 * R) return;
        const int fi = idx >> 2, w = idx & 3;
        const int l = fi & 63, fk = fi >> 6;
        const int nt = fk / KK, kk = fk % KK;
        const int r = nt * 16 + (l & 15);
        uint32_t word = 0;
        for (int c = 0; c < 4; ++c) {
            const int qq = kk * 64 + (l >> 4) * 16 + 4 * w + c;
            const T v = qq < R ? a[r * R + qq] : b[r * R + qq - R];
            if (v > 127 || v < -127) atomicOr(flag, 2);
            word |= ((uint32_t)(uint8_t)(int8_t)v) << (8 * c);
        }
        phi[idx] = word;
        return;
    }
    if (idx >= Q4 * R) return;
    const int q4 = idx / R, r = idx % R;
    uint32_t wa = 0, wb = 0;
    for (int c = 0; c < 4; ++c) {
        const T va = a[r * R + 4 * q4 + c], vb = b[r * R + 4 * q4 + c];
        if (va > 127 || va < -127 || vb > 127 || vb < -127) atomicOr(flag, 2);
        wa |= ((uint32_t)(uint8_t)(int8_t)va) << (8 * c);
        wb |= ((uint32_t)(uint8_t)(int8_t)vb) << (8 * c);
    }
    phi[idx] = wa;
    phi[Q4 * R + idx] = wb;
}

// ---- rows of a matrix under right-multiplied rotations ----
// Right multiplication acts on each row by itself (the column rule above), so a row lives in the
// registers of a group of G = min(R, 64) lanes: lane gl holds columns gl * CPL + j.
template <int NQ>
struct RowGeo {
    static constexpr int R = EGeo<NQ>::R;
    static constexpr int G = R < 64 ? R : 64;  // lanes per row
    static constexpr int CPL = R / G;          // columns per lane (1 or 4)
    static constexpr int RPW = 64 / G;         // rows per wavefront
};

__device__ inline int32_t shfl_t(int32_t v, int src) { return (int32_t)shfl32((uint32_t)v, src); }
__device__ inline int64_t shfl_t(int64_t v, int src) { return (int64_t)shfl64((uint64_t)v, src); }

template <int C, int CPL, typename T>
__device__ inline void fetch_cols(const T* v, int src, T* part) {
#pragma unroll
    for (int j = 0; j < CPL; ++j) part[j] = shfl_t(v[j ^ C], src);
}

// One rotation R(p) (R(p)^T if transposed) applied to NB rows held by the lane's group, unreduced: the
// exponent grows by one.  p is the same in every lane of the wavefront (1..4^n - 1).  SMALL: the values stay
// below 2^23 in magnitude, so a 24-bit multiply-add takes the partner with its sign, or not at all.
template <int NQ, int NB, typename T, bool SMALL = false>
__device__ inline void rotate_rows(T (*a)[RowGeo<NQ>::CPL], T (*b)[RowGeo<NQ>::CPL], uint32_t p, bool transposed, int gl,
                                   int gbase) {
    constexpr int CPL = RowGeo<NQ>::CPL;
    bool anti[CPL], plus[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
        const uint32_t q = (uint32_t)(gl * CPL + j);
        anti[j] = anticommutes<NQ>(p, q) != 0;
        plus[j] = (rotation_sign<NQ>(p, q) > 0) != transposed;
    }
    const int src = gbase + (gl ^ (int)(CPL == 4 ? p >> 2 : p));
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        T pa[CPL], pb[CPL];
        if constexpr (CPL == 4) {
            switch (p & 3) {  // uniform: the partner's register
                case 0: fetch_cols<0, CPL>(a[i], src, pa); fetch_cols<0, CPL>(b[i], src, pb); break;
                case 1: fetch_cols<1, CPL>(a[i], src, pa); fetch_cols<1, CPL>(b[i], src, pb); break;
                case 2: fetch_cols<2, CPL>(a[i], src, pa); fetch_cols<2, CPL>(b[i], src, pb); break;
                default: fetch_cols<3, CPL>(a[i], src, pa); fetch_cols<3, CPL>(b[i], src, pb); break;
            }
        } else {
            fetch_cols<0, CPL>(a[i], src, pa);
            fetch_cols<0, CPL>(b[i], src, pb);
        }
#pragma unroll
        for (int j = 0; j < CPL; ++j) {
            if constexpr (SMALL) {
                const int32_t s = anti[j] ? (plus[j] ? 1 : -1) : 0;
                const int32_t ra = anti[j] ? a[i][j] : 2 * b[i][j], rb = anti[j] ? b[i][j] : a[i][j];
                a[i][j] = __mul24(pa[j], s) + ra;
                b[i][j] = __mul24(pb[j], s) + rb;
                continue;
            }
            const T sa = plus[j] ? pa[j] : -pa[j], sb = plus[j] ? pb[j] : -pb[j];
            const T na = anti[j] ? a[i][j] + sa : 2 * b[i][j];
            b[i][j] = anti[j] ? b[i][j] + sb : a[i][j];
            a[i][j] = na;
        }
    }
}

// Claw check of (u0, u1): V = R(p_0)...R(p_{h-1}) from the side-0 point, W = S R(q_0)^T ... from
// the side-1 point, D = W V^T must be a signed permutation (Sec. 3, last merge case).
//   D = S R(q_0)^T ... R(q_{h-1})^T R(p_{h-1})^T ... R(p_0)^T
// is S under 2h rotations from the right, so no dense product is formed: one block per pair, its 16
// wavefronts each take rows of U through the rotations in registers (R(c)^T of the chunk first, at odd
// k), unreduced, at exponent E = e_U + k mod 2 + 2h.  S has int8 entries and orthonormal rows, so
// e_S <= log2(3 R 127^2), e_U <= e_S + 1 and every value, bounded by 2^(E/2), stays below 2^17 at n >= 3
// and 2^30 at n <= 2.  A row must hold one unit entry
// and the columns must differ; the first row that does not ends the pair.  Bound by the butterflies
// (2 h R^2 of them).  256 pairs at n = 4, k = 7, half of them claws: 81 us the whole call, 51 of them here
// (56 before the 24-bit multiply-adds); the dense product W V^T it replaces (R^3 64-bit products a pair,
// 16 blocks) took 244 ms.
constexpr int CLAW_WAVES = 16;
template <int NQ, typename T>
__global__ __launch_bounds__(CLAW_WAVES * 64) void k_claw(const T* __restrict__ sa, const T* __restrict__ sb,
                                                          const int32_t* se, uint32_t c, int k, const int32_t* made,
                                                          const uint64_t* u0, const uint64_t* u1, int64_t count,
                                                          int32_t* ok, int32_t* perm, int8_t* sign) {
    if (made[1] != 0) return;
    using Gm = RowGeo<NQ>;
    constexpr int R = Gm::R, CPL = Gm::CPL;
    constexpr uint32_t XI = R - 1;
    constexpr int NB = NQ >= 3 ? 4 : 1;  // row sets a wavefront holds at a time
    __shared__ uint16_t seq[64];
    __shared__ int cnt[R];
    __shared__ int rowof[R];
    __shared__ int sgn[R];
    __shared__ int bad;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    const int h = k / 2;
    const int first = c ? 1 : 0, steps = first + 2 * h;
    const int E = *se + steps;
    const T unit = (T)1 << (E / 2);
    for (int64_t pi = blockIdx.x; pi < count; pi += gridDim.x) {
        uint64_t p0 = u0[pi], p1 = u1[pi];
        if ((p0 >> 32) & 1) {
            const uint64_t x = p0; p0 = p1; p1 = x;
        }
        const bool sides_ok = (((p0 >> 32) & 1) == 0) && (((p1 >> 32) & 1) == 1);
        if (threadIdx.x == 0) {
            seq[0] = (uint16_t)c;
            uint32_t x = (uint32_t)p1;
            for (int t = 0; t < h; ++t) {
                seq[first + t] = (uint16_t)(x % XI + 1);
                x /= XI;
            }
            x = (uint32_t)p0;
            for (int t = 0; t < h; ++t) {
                seq[steps - 1 - t] = (uint16_t)(x % XI + 1);
                x /= XI;
            }
            bad = sides_ok ? 0 : 1;
        }
        for (int q = threadIdx.x; q < R; q += blockDim.x) cnt[q] = 0;
        __syncthreads();
        for (int r0 = wave * NB * Gm::RPW; r0 < R; r0 += CLAW_WAVES * NB * Gm::RPW) {
            // one answer for the whole wavefront: the rotations below exchange lanes
            if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(&bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)))
                break;
            T a[NB][CPL], b[NB][CPL];
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < CPL; ++j) {
                    // at n = 1 the wavefront has more lane groups than the matrix has rows
                    const int row = r0 + i * Gm::RPW + gi, at = row * R + gl * CPL + j;
                    a[i][j] = row < R ? sa[at] : 0;
                    b[i][j] = row < R ? sb[at] : 0;
                }
            for (int t = 0; t < steps; ++t)
                rotate_rows<NQ, NB, T, NQ >= 3>(a, b, (uint32_t)__builtin_amdgcn_readfirstlane(seq[t]), true, gl, gbase);
            bool row_ok = true;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                int nz = 0, col = 0, s = 0;
#pragma unroll
                for (int j = 0; j < CPL; ++j) {
                    const bool here = a[i][j] != 0 || b[i][j] != 0;
                    const uint64_t m = __ballot(here);
                    const uint64_t mine = Gm::G == 64 ? m : (m >> gbase) & ((1ull << (Gm::G & 63)) - 1);
                    nz += (int)__popcll(mine);
                    if (here) {
                        col = gl * CPL + j;
                        const T x = E % 2 == 0 ? a[i][j] : b[i][j], y = E % 2 == 0 ? b[i][j] : a[i][j];
                        s = y == 0 && (x == unit || x == -unit) ? (x > 0 ? 1 : -1) : 2;
                    }
                }
                if (r0 + i * Gm::RPW + gi >= R) continue;
                if (nz != 1 || s == 2) row_ok = false;
                if (nz == 1 && s != 0 && s != 2) {  // the lane that holds the row's entry
                    atomicAdd(&cnt[col], 1);
                    rowof[col] = r0 + i * Gm::RPW + gi;
                    sgn[col] = s;
                }
            }
            if (!row_ok) __hip_atomic_store(&bad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        for (int q = threadIdx.x; q < R; q += blockDim.x)
            if (cnt[q] != 1) __hip_atomic_store(&bad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        const int good = bad == 0 ? 1 : 0;
        for (int q = threadIdx.x; q < R; q += blockDim.x) {
            perm[pi * R + q] = good ? rowof[q] : -1;
            sign[pi * R + q] = (int8_t)(good ? sgn[q] : 0);
        }
        if (threadIdx.x == 0) ok[pi] = good;
        __syncthreads();
    }
}

// Canonical FP32 features of the exact matrix (a, b, e) held by the block (n <= 3): rows
// sign-normalised (first nonzero entry positive, decided exactly), sorted lexicographically as the
// integer sequences (a_0, b_0, a_1, b_1, ...), each entry (a + b sqrt2) 2^(-e/2) formed in double as
// t = a + b * SQRT2, t *= SQRT1_2 for odd e, t *= 2^(-floor(e/2)), rounded to float.
template <int NQ, typename T>
__device__ void block_features(const T* a, const T* b, int e, int32_t* rows /* R x 2R shared */,
                               int32_t* idx /* R shared */, float* out) {
    constexpr int R = EGeo<NQ>::R;
    for (int r = threadIdx.x; r < R; r += blockDim.x) {
        int sg = 0;
        for (int q = 0; q < R && sg == 0; ++q) {
            const int64_t va = a[r * R + q], vb = b[r * R + q];
            if (va == 0 && vb == 0) continue;
            if (va >= 0 && vb >= 0) sg = 1;
            else if (va <= 0 && vb <= 0) sg = -1;
            else if (va > 0) sg = (va * va > 2 * vb * vb) ? 1 : -1;
            else sg = (2 * vb * vb > va * va) ? 1 : -1;
        }
        if (sg == 0) sg = 1;
        for (int q = 0; q < R; ++q) {
            rows[r * 2 * R + 2 * q] = (int32_t)(sg * a[r * R + q]);
            rows[r * 2 * R + 2 * q + 1] = (int32_t)(sg * b[r * R + q]);
        }
        idx[r] = r;
    }
    __syncthreads();
    // bitonic sort of the row indices by lexicographic row order
    for (int k = 2; k <= R; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < R; i += blockDim.x) {
                const int l = i ^ j;
                if (l > i) {
                    const int ri = idx[i], rl = idx[l];
                    int cmp = 0;
                    for (int c = 0; c < 2 * R && cmp == 0; ++c) {
                        const int32_t x = rows[ri * 2 * R + c], y = rows[rl * 2 * R + c];
                        cmp = (x < y) ? -1 : (x > y ? 1 : 0);
                    }
                    const bool asc = (i & k) == 0;
                    if ((asc && cmp > 0) || (!asc && cmp < 0)) {
                        idx[i] = rl;
                        idx[l] = ri;
                    }
                }
            }
            __syncthreads();
        }
    }
    const double sqrt2 = 1.4142135623730951, sqrt1_2 = 0.7071067811865476;
    const double scale = ldexp(1.0, -(e / 2));
    for (int t = threadIdx.x; t < R * R; t += blockDim.x) {
        const int i = t / R, q = t % R;
        const int r = idx[i];
        double v = __dadd_rn((double)rows[r * 2 * R + 2 * q], __dmul_rn((double)rows[r * 2 * R + 2 * q + 1], sqrt2));
        if (e & 1) v = __dmul_rn(v, sqrt1_2);
        out[t] = (float)__dmul_rn(v, scale);
    }
    __syncthreads();
}

// ---- canonical features and packed targets from rows in registers (n <= 3) ----
// A matrix is held by WPT wavefronts, NB row sets each (RowGeo: one row per lane group).  At n = 3 a batch's
// targets take four each; a single target takes sixteen, one comparison of a row with four others each.
template <int NQ, int W = NQ == 3 ? 4 : 1>
struct FeatGeo {
    using Gm = RowGeo<NQ>;
    static constexpr int R = Gm::R;
    static constexpr int WPT = W;
    static constexpr int THREADS = WPT * 64;
    static constexpr int NB = NQ == 1 ? 1 : R / (Gm::RPW * WPT);
    static constexpr int WORDS = 2 * R / 8;          // 8-byte words of a row's sort key
    static constexpr int KEY = 2 * R / 8 + (NQ == 3 ? 1 : 0);  // row pitch in words (odd: lanes read a row each)
};

template <int NQ>
struct FeatLds {
    uint64_t key[FeatGeo<NQ>::R * FeatGeo<NQ>::KEY];
    int32_t rank[FeatGeo<NQ>::R];
};

// The canonical features of block_features, for entries within int8.  A row's key is its integer
// sequence (a_0, b_0, a_1, ...) as bytes v + 128, first entry in the highest byte, so rows compare as
// unsigned 8-byte words; a row's place is the number of rows below it.  Lane i compares row i with
// the rows j of its wavefront's share, a word at a time until every pair is decided.
template <int NQ, typename T, int W = FeatGeo<NQ>::WPT>
__device__ void rows_features(T (*a)[1], T (*b)[1], int e, FeatLds<NQ>& L, float* out) {
    using Fg = FeatGeo<NQ, W>;
    using Gm = RowGeo<NQ>;
    constexpr int R = Fg::R;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    for (int r = threadIdx.x; r < R; r += Fg::THREADS) L.rank[r] = 0;
#pragma unroll
    for (int i = 0; i < Fg::NB; ++i) {
        const int row = (wave * Fg::NB + i) * Gm::RPW + gi;
        const int32_t va = (int32_t)a[i][0], vb = (int32_t)b[i][0];
        // the sign of va + vb sqrt2, decided exactly
        const bool positive = (va >= 0 && vb >= 0) || (va > 0 && vb < 0 && va * va > 2 * vb * vb) ||
                              (va < 0 && vb > 0 && 2 * vb * vb > va * va);
        const uint64_t nz = __ballot(va != 0 || vb != 0), pos = __ballot(positive);
        const uint64_t mine = Gm::G == 64 ? nz : (nz >> gbase) & ((1ull << (Gm::G & 63)) - 1);
        const int first = mine ? gbase + (int)__builtin_ctzll(mine) : gbase;
        if (!((pos >> first) & 1)) {
            a[i][0] = -a[i][0];
            b[i][0] = -b[i][0];
        }
        if (row < R) {
            const uint32_t ka = (uint32_t)((int32_t)a[i][0] + 128), kb = (uint32_t)((int32_t)b[i][0] + 128);
            uint8_t* at = reinterpret_cast<uint8_t*>(&L.key[row * Fg::KEY + gl / 4]) + 6 - 2 * (gl & 3);
            *reinterpret_cast<uint16_t*>(at) = (uint16_t)((ka << 8) | (kb & 255));
        }
    }
    __syncthreads();
    if (lane < R) {
        uint64_t own[Fg::WORDS];
#pragma unroll
        for (int w = 0; w < Fg::WORDS; ++w) own[w] = L.key[lane * Fg::KEY + w];
        int below = 0;
        for (int j = wave * (R / Fg::WPT); j < (wave + 1) * (R / Fg::WPT); ++j) {
            bool open = lane != j, less = false;
#pragma unroll
            for (int w = 0; w < Fg::WORDS; ++w) {
                const uint64_t kj = L.key[j * Fg::KEY + w];
                less = (open && kj < own[w]) || less;
                open = open && kj == own[w];
                if (__ballot(open) == 0) break;
            }
            below += less;
        }
        atomicAdd(&L.rank[lane], below);
    }
    __syncthreads();
    const double sqrt2 = 1.4142135623730951, sqrt1_2 = 0.7071067811865476;
    const double scale = ldexp(1.0, -(e / 2));
#pragma unroll
    for (int i = 0; i < Fg::NB; ++i) {
        const int row = (wave * Fg::NB + i) * Gm::RPW + gi;
        if (row >= R) continue;
        double v = __dadd_rn((double)(int32_t)a[i][0], __dmul_rn((double)(int32_t)b[i][0], sqrt2));
        if (e & 1) v = __dmul_rn(v, sqrt1_2);
        out[L.rank[row] * R + gl] = (float)__dmul_rn(v, scale);
    }
    __syncthreads();
}

// One target's features.  Entries beyond int8 take block_features' general sort (32-bit entries, one
// row per thread): 72 us at n = 3 where the byte keys take 8 us (14 with four wavefronts).
template <int NQ>
using FeatOne = FeatGeo<NQ, NQ == 3 ? 16 : 1>;
template <int NQ, typename T>
__global__ __launch_bounds__(FeatOne<NQ>::THREADS) void k_features(const T* a, const T* b, const int32_t* e, float* out) {
    using Fg = FeatOne<NQ>;
    using Gm = RowGeo<NQ>;
    constexpr int R = Fg::R;
    __shared__ FeatLds<NQ> L;
    __shared__ int32_t rows[R * 2 * R];
    __shared__ int32_t idx[R];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G;
    T ra[Fg::NB][1], rb[Fg::NB][1];
    int wide = 0;
#pragma unroll
    for (int i = 0; i < Fg::NB; ++i) {
        const int row = (wave * Fg::NB + i) * Gm::RPW + gi;
        ra[i][0] = row < R ? a[row * R + gl] : 0;
        rb[i][0] = row < R ? b[row * R + gl] : 0;
        wide |= ra[i][0] > 127 || ra[i][0] < -127 || rb[i][0] > 127 || rb[i][0] < -127;
    }
    if (__syncthreads_or(wide))
        block_features<NQ, T>(a, b, *e, rows, idx, out);
    else
        rows_features<NQ, T, Fg::WPT>(ra, rb, *e, L, out);
}

// The signed permutation of columns that R(p)^2 is: an entry in column c of a row moves to column
// p ^ c with sign s(p, p ^ c) when P_p and P_c anticommute, and stays otherwise.
template <int NQ>
__device__ inline void clifford_step(uint32_t p, uint32_t& c, uint32_t& neg) {
    if (anticommutes<NQ>(p, c)) {
        c ^= p;
        neg ^= rotation_sign<NQ>(p, c) < 0 ? 1u : 0u;
    }
}

// Reduction steps that a matrix at exponent e allows, from the OR of its a and of its b entries (which
// has the least 2-adic valuation among them): the rule stands at or_entries.
template <typename T>
__device__ inline int reduction_steps(T or_a, T or_b, int e) {
    const int ma = or_a ? 2 * (int)__builtin_ctzll((unsigned long long)or_a) : 1 << 20;
    const int mb = or_b ? 2 * (int)__builtin_ctzll((unsigned long long)or_b) + 1 : 1 << 20;
    const int m = ma < mb ? ma : mb;
    return m < e ? m : e;
}
template <typename T>
__device__ inline void reduce_entry(T& a, T& b, int m) {
    const int j = m >> 1;
    const T va = a, vb = b;
    a = m & 1 ? vb >> j : va >> j;
    b = m & 1 ? va >> (j + 1) : vb >> j;
}

// Unreduced rotations stay exact up to this exponent: |a|, |b sqrt2| <= 2^(e/2) <= 2^28.
constexpr int E_FREE = 56;

// Network data: targets built exactly from their words (Clifford word then rotations), packed as
// int8 for the walk step (n <= 3 layout) and turned into canonical features.  One block per target,
// the rows in registers throughout: the Clifford word is a signed permutation of columns, so every
// lane follows one row's single entry through its share of the word; the rotations then act on the
// rows, reduced once at the end (and before every rotation beyond exponent E_FREE, where the entries'
// range is checked).  Bound by instructions (about 2,200 per wavefront): 16384 circuits of 48 Clifford
// factors and 1 to 10 rotations at n = 3 take 0.66 ms, against 33 ms with every factor as two rotations
// through global memory, a reduction after each.  The second launch bound keeps three wavefronts on a SIMD
// (0.86 ms with the two that 169 registers leave; four spill, 0.70 ms).
template <int NQ, typename T>
__global__ __launch_bounds__(FeatGeo<NQ>::THREADS, 3) void k_build_batch(const uint16_t* words, const int32_t* offsets,
                                                                      const int32_t* kof, int count, uint32_t* phi_out,
                                                                      int32_t* rot_e_out, float* feat_out, int* flag) {
    using Fg = FeatGeo<NQ>;
    using Gm = RowGeo<NQ>;
    constexpr int R = Fg::R, NB = Fg::NB, WPT = Fg::WPT, Q4 = R / 4;
    __shared__ FeatLds<NQ> L;
    __shared__ __attribute__((aligned(16))) int8_t bytes[2][R * R];  // A, then B
    __shared__ uint16_t part[WPT][R];  // each wavefront's share of the Clifford word: column | sign << 8
    __shared__ T ors[2][WPT];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    const T lim = lim_of<T>();
    for (int t = blockIdx.x; t < count; t += gridDim.x) {
        const int w0 = offsets[t], w1 = offsets[t + 1];
        int k = kof[t], m = w1 - w0 - k;
        if (2 * m + k > 256) {
            if (threadIdx.x == 0) atomicOr(flag, 8);
            k = m = 0;
        }
        {
            uint32_t c = (uint32_t)lane & (R - 1), neg = 0;
            for (int j = m * wave / WPT; j < m * (wave + 1) / WPT; ++j)
                clifford_step<NQ>((uint32_t)__builtin_amdgcn_readfirstlane(words[w0 + k + j]), c, neg);
            if (lane < R) part[wave][lane] = (uint16_t)(c | (neg << 8));
        }
        __syncthreads();
        uint32_t c = (uint32_t)lane & (R - 1), neg = 0;
#pragma unroll
        for (int w = 0; w < WPT; ++w) {
            const uint32_t v = part[w][c];
            c = v & 255u;
            neg ^= v >> 8;
        }
        T a[NB][1], b[NB][1];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int row = (wave * NB + i) * Gm::RPW + gi;
            const uint32_t v = shfl32(c | (neg << 8), row & (R - 1));
            a[i][0] = row < R && (int)(v & 255u) == gl ? (v >> 8 ? -1 : 1) : 0;
            b[i][0] = 0;
        }
        int e = 0;
        auto reduce = [&]() {
            T oa = 0, ob = 0;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                oa |= a[i][0];
                ob |= b[i][0];
            }
            for (int off = 32; off >= 1; off >>= 1) {
                oa |= shfl_t(oa, lane ^ off);
                ob |= shfl_t(ob, lane ^ off);
            }
            if constexpr (WPT > 1) {
                if (lane == 0) {
                    ors[0][wave] = oa;
                    ors[1][wave] = ob;
                }
                __syncthreads();
#pragma unroll
                for (int w = 0; w < WPT; ++w) {
                    oa |= ors[0][w];
                    ob |= ors[1][w];
                }
                __syncthreads();
            }
            const int steps = reduction_steps(oa, ob, e);
#pragma unroll
            for (int i = 0; i < NB; ++i) reduce_entry(a[i][0], b[i][0], steps);
            e -= steps;
        };
        for (int j = k - 1; j >= 0; --j) {
            if (e >= E_FREE) reduce();
            rotate_rows<NQ, NB, T>(a, b, (uint32_t)__builtin_amdgcn_readfirstlane(words[w0 + j]), false, gl, gbase);
            if (++e > E_FREE) {
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    if (a[i][0] > lim || a[i][0] < -lim || b[i][0] > lim || b[i][0] < -lim) atomicOr(flag, 4);
            }
        }
        reduce();
        bool wide = false;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int row = (wave * NB + i) * Gm::RPW + gi;
            wide |= a[i][0] > 127 || a[i][0] < -127 || b[i][0] > 127 || b[i][0] < -127;
            if (row < R) {
                bytes[0][row * R + gl] = (int8_t)a[i][0];
                bytes[1][row * R + gl] = (int8_t)b[i][0];
            }
        }
        if (wide) atomicOr(flag, 2);
        if (threadIdx.x == 0) rot_e_out[t] = (int32_t)((30ll * e) % 61);
        __syncthreads();
        if constexpr (NQ == 3) {
            // MFMA fragment layout (as k_pack_phi for n >= 3): 16 bytes of a row per lane
            typedef int v4 __attribute__((ext_vector_type(4)));
            v4* out = reinterpret_cast<v4*>(phi_out + (size_t)t * 2 * Q4 * R);
            for (int x = threadIdx.x; x < 2 * R * R / 16; x += Fg::THREADS) {
                const int l = x & 63, kk = (x >> 6) & 1, nt = x >> 7;
                out[x] = *reinterpret_cast<const v4*>(&bytes[kk][(nt * 16 + (l & 15)) * R + (l >> 4) * 16]);
            }
        } else {
            for (int x = threadIdx.x; x < 2 * Q4 * R; x += Fg::THREADS) {
                const int q4 = (x % (Q4 * R)) / R, r = x % R;
                phi_out[(size_t)t * 2 * Q4 * R + x] = *reinterpret_cast<const uint32_t*>(&bytes[x / (Q4 * R)][r * R + 4 * q4]);
            }
        }
        rows_features<NQ, T>(a, b, e, L, feat_out + (size_t)t * R * R);
    }
}

template <typename F>
hipError_t dispatch_exact(int n, F&& f) {
    switch (n) {
        case 1: return f.template operator()<1, int64_t>();
        case 2: return f.template operator()<2, int64_t>();
        case 3: return f.template operator()<3, int32_t>();
        case 4: return f.template operator()<4, int32_t>();
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t exact_alloc(ExactDev& m, int n) {
    m.n = n;
    m.r = 1 << (2 * n);
    m.elem = n <= 2 ? 8 : 4;
    const size_t bytes = (size_t)m.r * m.r * m.elem;
    hipError_t err = hipMalloc(&m.a, bytes);
    if (err == hipSuccess) err = hipMalloc(&m.b, bytes);
    if (err == hipSuccess) err = hipMalloc(&m.e, sizeof(int32_t));
    return err;
}

void exact_free(ExactDev& m) {
    if (m.a) (void)hipFree(m.a);
    if (m.b) (void)hipFree(m.b);
    if (m.e) (void)hipFree(m.e);
    m.a = m.b = nullptr;
    m.e = nullptr;
}

namespace {
struct ScratchPair {
    void* ta = nullptr;
    void* tb = nullptr;
};
hipError_t scratch_pair(const ExactDev& m, ScratchPair& sp) {
    const size_t bytes = (size_t)m.r * m.r * m.elem;
    hipError_t err = hipMalloc(&sp.ta, bytes);
    if (err == hipSuccess) err = hipMalloc(&sp.tb, bytes);
    return err;
}
void scratch_free(ScratchPair& sp) {
    if (sp.ta) (void)hipFree(sp.ta);
    if (sp.tb) (void)hipFree(sp.tb);
}
}  // namespace

hipError_t exact_apply_ws(ExactDev& dst, const ExactDev& src, const uint16_t* seq, const uint8_t* tr, int nseq,
                          void* ta, void* tb, int* flag, hipStream_t s) {
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        hipLaunchKernelGGL((k_apply<NQ, T>), dim3(1), dim3(1024), 0, s, (T*)dst.a, (T*)dst.b, (T*)ta, (T*)tb, dst.e,
                           (const T*)src.a, (const T*)src.b, src.e, seq, tr, nseq, flag);
        return hipGetLastError();
    };
    return dispatch_exact(dst.n, f);
}

hipError_t exact_apply(ExactDev& dst, const ExactDev& src, const uint16_t* seq, const uint8_t* tr, int nseq,
                       int* flag, hipStream_t s) {
    ScratchPair sp;
    hipError_t err = scratch_pair(dst, sp);
    if (err != hipSuccess) {
        scratch_free(sp);
        return err;
    }
    err = exact_apply_ws(dst, src, seq, tr, nseq, sp.ta, sp.tb, flag, s);
    if (err == hipSuccess) err = hipStreamSynchronize(s);
    scratch_free(sp);
    return err;
}

namespace {
// A matrix multiplied from the right on many blocks, in two passes with no work matrices: the first leaves
// the product unreduced and ors its a entries into ors[0] and its b entries into ors[1] (one atomic
// per block); the second takes all reduction steps in closed form.  A step (a, b) -> (b, a / 2) needs a
// even, so from (a, b) the steps alternate the conditions 2 | a, 2 | b, 4 | a, 4 | b, ... and entry (a, b)
// allows min(2 v2(a), 2 v2(b) + 1) of them (v2 = 2-adic valuation, unbounded for 0, that of an OR being
// the least of its terms'): reduction_steps.  After 2j steps an entry is (a, b) / 2^j, after 2j + 1 steps
// (b / 2^j, a / 2^(j + 1)): reduce_entry.
template <typename T, int WAVES>
__device__ inline void or_entries(T oa, T ob, unsigned long long* ors) {
    __shared__ T red[2][WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int off = 32; off >= 1; off >>= 1) {
        oa |= shfl_t(oa, lane ^ off);
        ob |= shfl_t(ob, lane ^ off);
    }
    if (lane == 0) {
        red[0][wave] = oa;
        red[1][wave] = ob;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        T v = 0;
        for (int w = 0; w < WAVES; ++w) v |= red[threadIdx.x][w];
        if (v) atomicOr(&ors[threadIdx.x], (unsigned long long)v);
    }
}

// (a, b) at exponent `grown`, reduced in place; *e_io = the exponent left.
template <int NQ, typename T>
__global__ __launch_bounds__(256) void k_reduce(T* a, T* b, int32_t* e_io, int grown, const unsigned long long* ors) {
    constexpr int R = EGeo<NQ>::R;
    const int m = reduction_steps((T)ors[0], (T)ors[1], grown);
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < R * R && m > 0) reduce_entry(a[idx], b[idx], m);
    if (idx == 0) *e_io = grown - m;
}

// A target from its words (m Clifford factors, then its rotations, as they are multiplied from the right):
// every wavefront takes rows of the product through the words in registers, as k_build_batch does, but
// one row set each, so that the rows of one target fill up to 64 blocks.  At most E_FREE rotations, so
// nothing leaves the exact range.  Bound by the chain of the Clifford word and by launches: at n = 4, 64
// factors and 7 rotations, building a target and reading it back takes 97 us, against 6.5 ms with every
// factor as two rotations on one block, a reduction after each (k_apply, which words with more rotations
// still take).
constexpr int WORDS_MAX = 1024;
struct Words {
    uint16_t w[WORDS_MAX];
};
constexpr int WORDS_WAVES = 4;
template <int NQ, typename T>
__global__ __launch_bounds__(WORDS_WAVES * 64) void k_words(Words words, int m, int k, T* a, T* b,
                                                            unsigned long long* ors) {
    using Gm = RowGeo<NQ>;
    constexpr int R = Gm::R, CPL = Gm::CPL;
    const int lane = threadIdx.x & 63;
    const int gi = lane / Gm::G, gl = lane % Gm::G, gbase = gi * Gm::G;
    const int row = (int)(blockIdx.x * WORDS_WAVES + (threadIdx.x >> 6)) * Gm::RPW + gi;
    uint32_t c = (uint32_t)row & (R - 1), neg = 0;
    for (int base = 0; base < m; base += 64) {
        const int n = m - base < 64 ? m - base : 64;
        const int mine = lane < n ? words.w[base + lane] : 0;
        for (int j = 0; j < n; ++j) clifford_step<NQ>((uint32_t)__builtin_amdgcn_readlane(mine, j), c, neg);
    }
    T ra[1][CPL], rb[1][CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
        ra[0][j] = row < R && (int)c == gl * CPL + j ? (neg ? -1 : 1) : 0;
        rb[0][j] = 0;
    }
    const int mine = lane < k ? words.w[m + lane] : 0;
    for (int j = 0; j < k; ++j)
        rotate_rows<NQ, 1, T>(ra, rb, (uint32_t)__builtin_amdgcn_readlane(mine, j), false, gl, gbase);
    T oa = 0, ob = 0;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
        if (row < R) {
            a[row * R + gl * CPL + j] = ra[0][j];
            b[row * R + gl * CPL + j] = rb[0][j];
        }
        oa |= ra[0][j];
        ob |= rb[0][j];
    }
    or_entries<T, WORDS_WAVES>(oa, ob, ors);
}

__global__ void k_clear_ors(unsigned long long* ors) {
    if (threadIdx.x < 2) ors[threadIdx.x] = 0;
}

// ---- search spaces (SpaceJob) ----
// Entry (row, q) of U R(c)^T, unreduced; c = 0: of U.
template <int NQ, typename T>
__device__ inline void chunk_entry(const T* a, const T* b, uint32_t c, int row, uint32_t q, T& va, T& vb) {
    constexpr int R = EGeo<NQ>::R;
    const int at = row * R + (int)q;
    va = a[at];
    vb = b[at];
    if (c == 0) return;
    if (anticommutes<NQ>(c, q)) {
        const int j = row * R + (int)(q ^ c);
        const bool plus = rotation_sign<NQ>(c, q) < 0;  // transposed
        va += plus ? a[j] : -a[j];
        vb += plus ? b[j] : -b[j];
    } else {
        const T x = va;
        va = 2 * vb;
        vb = x;
    }
}

// The int8 packing of S_c (the layouts of k_pack_phi) and the keys, by threads i, i + stride, ... of a job.
template <int NQ, typename T>
__device__ void space_pack(const SpaceJob& J, T or_a, T or_b, int i, int stride) {
    constexpr int R = EGeo<NQ>::R;
    constexpr int Q4 = R / 4;
    const T *a = (const T*)J.a, *b = (const T*)J.b;
    const int e1 = *J.e + (J.c ? 1 : 0);
    // a target is held reduced, so only a rotation's product has steps to take
    const int m = J.c ? reduction_steps(or_a, or_b, e1) : 0;
    int flags = 0;
    const T lim = lim_of<T>();
    auto entry = [&](int row, uint32_t q, bool second, T& v) {
        T va, vb;
        chunk_entry<NQ, T>(a, b, J.c, row, q, va, vb);
        if (J.c && (va > lim || va < -lim || vb > lim || vb < -lim)) flags |= 4;
        if (m > 0) reduce_entry(va, vb, m);
        v = second ? vb : va;
        if (v > 127 || v < -127) flags |= 2;
    };
    for (int idx = i; idx < 2 * Q4 * R; idx += stride) {
        uint32_t word = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            T v;
            if constexpr (NQ >= 3) {
                constexpr int KK = 2 * R / 64;
                const int fi = idx >> 2, l = fi & 63, fk = fi >> 6;
                const int qq = (fk % KK) * 64 + (l >> 4) * 16 + 4 * (idx & 3) + c;
                entry((fk / KK) * 16 + (l & 15), (uint32_t)(qq & (R - 1)), qq >= R, v);
            } else {
                const int x = idx % (Q4 * R);
                entry(x % R, (uint32_t)(4 * (x / R) + c), idx >= Q4 * R, v);
            }
            word |= ((uint32_t)(uint8_t)(int8_t)v) << (8 * c);
        }
        J.phi[idx] = word;
    }
    if (flags) atomicOr(&J.out[1], flags);
    const uint64_t s0 = sm64(J.seed, 0);
    for (int q = i; q < R; q += stride) {
        uint64_t k = sm64(s0, (uint64_t)q) >> 3;
        if (k >= P61) k -= P61;
        J.keys[q] = k;
    }
    if (i == 0) J.out[0] = e1 - m;
}

// n <= 3: one block per job
template <int NQ, typename T>
__global__ __launch_bounds__(1024) void k_space(SpaceJob one, const SpaceJob* many) {
    constexpr int R = EGeo<NQ>::R;
    const SpaceJob J = many ? many[blockIdx.x] : one;
    __shared__ unsigned long long ors[2];
    if (threadIdx.x < 2) ors[threadIdx.x] = 0;
    if (threadIdx.x == 0) J.out[1] = J.out[2] = 0;
    __syncthreads();
    if (J.c) {
        T oa = 0, ob = 0;
        for (int idx = threadIdx.x; idx < R * R; idx += blockDim.x) {
            T va, vb;
            chunk_entry<NQ, T>((const T*)J.a, (const T*)J.b, J.c, idx / R, (uint32_t)(idx & (R - 1)), va, vb);
            oa |= va;
            ob |= vb;
        }
        if (oa) atomicOr(&ors[0], (unsigned long long)oa);
        if (ob) atomicOr(&ors[1], (unsigned long long)ob);
    }
    __syncthreads();
    space_pack<NQ, T>(J, (T)ors[0], (T)ors[1], (int)threadIdx.x, (int)blockDim.x);
}

// n = 4: 32 blocks per job in each of two passes (blockIdx.y: the job)
constexpr int SPACE_BLOCKS = 32;
__global__ void k_space_clear(SpaceJob one, const SpaceJob* many, int count) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) {
        const SpaceJob J = many ? many[i] : one;
        J.ors[0] = J.ors[1] = 0;
        J.out[1] = J.out[2] = 0;
    }
}
__global__ __launch_bounds__(1024) void k_space_or4(SpaceJob one, const SpaceJob* many) {
    constexpr int R = 256;
    const SpaceJob J = many ? many[blockIdx.y] : one;
    if (J.c == 0) return;
    int32_t oa = 0, ob = 0;
    for (int idx = (int)(blockIdx.x * blockDim.x + threadIdx.x); idx < R * R; idx += SPACE_BLOCKS * (int)blockDim.x) {
        int32_t va, vb;
        chunk_entry<4, int32_t>((const int32_t*)J.a, (const int32_t*)J.b, J.c, idx / R, (uint32_t)(idx & (R - 1)), va, vb);
        oa |= va;
        ob |= vb;
    }
    or_entries<int32_t, 16>(oa, ob, J.ors);
}
__global__ __launch_bounds__(1024) void k_space_pack4(SpaceJob one, const SpaceJob* many) {
    const SpaceJob J = many ? many[blockIdx.y] : one;
    space_pack<4, int32_t>(J, (int32_t)J.ors[0], (int32_t)J.ors[1], (int)(blockIdx.x * blockDim.x + threadIdx.x),
                           SPACE_BLOCKS * (int)blockDim.x);
}

__global__ void k_seq_one(uint16_t* seq, uint8_t* tr, uint16_t p, uint8_t t) {
    if (threadIdx.x == 0) {
        seq[0] = p;
        tr[0] = t;
    }
}
__global__ void k_fill_i32(int* dst, int v, int count) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) dst[i] = v;
}
}  // namespace

hipError_t spaces_make(int n, const SpaceJob& one, const SpaceJob* many, int count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (n == 4) {
        // a grid's second dimension ends at 65,536 blocks: a batch of more members takes several launches
        constexpr int MOST = 32768;
        for (int at = 0; at < count; at += MOST) {
            const int jobs = count - at < MOST ? count - at : MOST;
            const SpaceJob* from = many ? many + at : nullptr;
            hipLaunchKernelGGL(k_space_clear, dim3(1), dim3(many ? 256 : 64), 0, s, one, from, jobs);
            if (many || one.c)
                hipLaunchKernelGGL(k_space_or4, dim3(SPACE_BLOCKS, jobs), dim3(1024), 0, s, one, from);
            hipLaunchKernelGGL(k_space_pack4, dim3(SPACE_BLOCKS, jobs), dim3(1024), 0, s, one, from);
        }
        return hipGetLastError();
    }
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        if constexpr (NQ <= 3) {
            hipLaunchKernelGGL((k_space<NQ, T>), dim3(count), dim3(NQ == 3 ? 1024 : 256), 0, s, one, many);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    };
    return dispatch_exact(n, f);
}

hipError_t exact_seq_one(uint16_t* seq, uint8_t* tr, uint16_t p, uint8_t transpose, hipStream_t s) {
    hipLaunchKernelGGL(k_seq_one, dim3(1), dim3(64), 0, s, seq, tr, p, transpose);
    return hipGetLastError();
}

hipError_t fill_i32(int* dst, int v, int count, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, dst, v, count);
    return hipGetLastError();
}

bool exact_words_fit(int m, int k) { return k <= E_FREE && m + k <= WORDS_MAX; }

hipError_t exact_words(ExactDev& dst, const uint16_t* clifford, int m, const uint16_t* rotations, int k, uint64_t* ors,
                       hipStream_t s) {
    if (!exact_words_fit(m, k)) return hipErrorInvalidValue;
    Words w;
    for (int j = 0; j < m; ++j) w.w[j] = clifford[j];
    for (int j = 0; j < k; ++j) w.w[m + j] = rotations[j];
    unsigned long long* o = reinterpret_cast<unsigned long long*>(ors);
    hipLaunchKernelGGL(k_clear_ors, dim3(1), dim3(64), 0, s, o);
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        constexpr int R = EGeo<NQ>::R, rows = RowGeo<NQ>::RPW * WORDS_WAVES;
        hipLaunchKernelGGL((k_words<NQ, T>), dim3((R + rows - 1) / rows), dim3(WORDS_WAVES * 64), 0, s, w, m, k,
                           (T*)dst.a, (T*)dst.b, o);
        hipLaunchKernelGGL((k_reduce<NQ, T>), dim3((R * R + 255) / 256), dim3(256), 0, s, (T*)dst.a, (T*)dst.b, dst.e,
                           k, o);
        return hipGetLastError();
    };
    return dispatch_exact(dst.n, f);
}

hipError_t exact_build(ExactDev& m, const uint16_t* seq, const uint8_t* tr, int nseq, int* flag, hipStream_t s) {
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        hipLaunchKernelGGL((k_identity<NQ, T>), dim3(64), dim3(1024), 0, s, (T*)m.a, (T*)m.b, m.e);
        return hipGetLastError();
    };
    hipError_t err = dispatch_exact(m.n, f);
    if (err != hipSuccess) return err;
    return exact_apply(m, m, seq, tr, nseq, flag, s);
}

hipError_t exact_from_i32(ExactDev& m, const int32_t* a, const int32_t* b, int32_t e, int* flag, hipStream_t s) {
    (void)flag;
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        hipLaunchKernelGGL((k_from_i32<NQ, T>), dim3(1), dim3(1024), 0, s, (T*)m.a, (T*)m.b, m.e, a, b, e);
        return hipGetLastError();
    };
    return dispatch_exact(m.n, f);
}

hipError_t exact_from_unitary(ExactDev& m, const int64_t* v, int32_t e, int32_t* a_tmp, int32_t* b_tmp, int* flag,
                              hipStream_t s) {
    const int n = m.n;
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        constexpr int D = 1 << NQ;
        constexpr int R = D * D;
        hipLaunchKernelGGL((k_unitary_check<NQ>), dim3((D * D + 255) / 256), dim3(256), 0, s, v, e, flag);
        hipLaunchKernelGGL((k_unitary_channel<NQ>), dim3((R * R + 255) / 256), dim3(256), 0, s, v, a_tmp, b_tmp,
                           flag);
        return hipGetLastError();
    };
    hipError_t err = dispatch_exact(n, f);
    if (err != hipSuccess) return err;
    return exact_from_i32(m, a_tmp, b_tmp, 2 * (n + e), flag, s);
}

hipError_t exact_to_i32(const ExactDev& m, int32_t* a, int32_t* b, int* flag, hipStream_t s) {
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        hipLaunchKernelGGL((k_to_i32<NQ, T>), dim3(64), dim3(1024), 0, s, (const T*)m.a, (const T*)m.b, a, b,
                           flag);
        return hipGetLastError();
    };
    return dispatch_exact(m.n, f);
}

hipError_t exact_check_orthogonal(const ExactDev& m, int* flag, hipStream_t s) {
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        constexpr int R = 1 << (2 * NQ);
        hipLaunchKernelGGL((k_orthogonal<NQ, T>), dim3((R * R + 255) / 256), dim3(256), 0, s, (const T*)m.a,
                           (const T*)m.b, m.e, flag);
        return hipGetLastError();
    };
    return dispatch_exact(m.n, f);
}

hipError_t exact_signed_perm(const ExactDev& m, int32_t* ok, int32_t* perm, int8_t* sign, hipStream_t s) {
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        hipLaunchKernelGGL((k_signed_perm<NQ, T>), dim3(1), dim3(256), 0, s, (const T*)m.a, (const T*)m.b, m.e,
                           ok, perm, sign);
        return hipGetLastError();
    };
    return dispatch_exact(m.n, f);
}

hipError_t exact_pack_phi(const ExactDev& m, uint32_t* phi, int* flag, hipStream_t s) {
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        constexpr int R = 1 << (2 * NQ);
        const int nthr = NQ >= 3 ? R / 2 * R : R / 4 * R;
        hipLaunchKernelGGL((k_pack_phi<NQ, T>), dim3((nthr + 255) / 256), dim3(256), 0, s, (const T*)m.a,
                           (const T*)m.b, phi, flag);
        return hipGetLastError();
    };
    return dispatch_exact(m.n, f);
}

hipError_t exact_claw_check(const ExactDev& U, uint32_t c, int k, const int32_t* made, const uint64_t* u0,
                            const uint64_t* u1, int64_t count, int32_t* ok, int32_t* perm, int8_t* sign, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        const int blocks = (int)(count < 4096 ? count : 4096);
        hipLaunchKernelGGL((k_claw<NQ, T>), dim3(blocks), dim3(CLAW_WAVES * 64), 0, s, (const T*)U.a, (const T*)U.b,
                           U.e, c, k, made, u0, u1, count, ok, perm, sign);
        return hipGetLastError();
    };
    return dispatch_exact(U.n, f);
}

}  // namespace tcw

namespace tcw {

hipError_t exact_features(const ExactDev& m, float* out, hipStream_t s) {
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        if constexpr (NQ <= 3) {
            hipLaunchKernelGGL((k_features<NQ, T>), dim3(1), dim3(FeatOne<NQ>::THREADS), 0, s, (const T*)m.a,
                               (const T*)m.b, m.e, out);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    };
    return dispatch_exact(m.n, f);
}

hipError_t build_batch(int n, const uint16_t* words, const int32_t* offsets, const int32_t* kof, int count,
                       uint32_t* phi_out, int32_t* rot_e_out, float* feat_out, int* flag, hipStream_t s) {
    auto f = [&]<int NQ, typename T>() -> hipError_t {
        if constexpr (NQ <= 3) {
            const int blocks = count < 8192 ? count : 8192;
            hipLaunchKernelGGL((k_build_batch<NQ, T>), dim3(blocks), dim3(FeatGeo<NQ>::THREADS), 0, s, words, offsets,
                               kof, count, phi_out, rot_e_out, feat_out, flag);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    };
    return dispatch_exact(n, f);
}

}  // namespace tcw
