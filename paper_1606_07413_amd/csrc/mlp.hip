// The depth-order network on gfx950: x -> [Linear -> GELU] x depth -> Linear -> softmax over T-counts,
// cross-entropy loss, Adam on FP32 master weights.  Every product is one BF16 x BF16 -> FP32 MFMA
// GEMM of the form C = A B^T with both operands stored K-contiguous (each row of A and of B holds
// consecutive k), so every operand fragment is one 16-byte load:
//   forward:  Z = H W + b              A = H (batch x in),      B = W^T (out x in)
//   dX:       G' = (G W^T) * gelu'(Z)  A = G (batch x out),     B = W (in x out)
//   dW:       dW = H^T G               A = H^T (in x batch),    B = G^T (out x batch)
// The epilogues write the transposed BF16 copies (H^T, G^T) the weight-gradient products read, so no
// product ever reads a strided operand.  Leading dimensions of BF16 buffers are multiples of 8.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "common.h"
#include "internal.h"

namespace tcw {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8), aligned(16)));

namespace {

enum Epi : int {
    EPI_STORE = 0,      // C = acc
    EPI_BIAS = 1,       // C = acc + bias
    EPI_BIAS_GELU = 2,  // C = Z = acc + bias (fp32), H = gelu(Z) (bf16), T = H^T (bf16, optional)
    EPI_GELU_GRAD = 3,  // C = G = acc * gelu'(Zin) (fp32), H = G (bf16), T = G^T (bf16, optional)
};

__device__ inline float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ inline float gelu_grad_f(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

constexpr int BN = 128, BK = 64, LDK = BK + 8;  // LDS rows of 64 k values padded to 144 bytes

// Eight consecutive k of an operand that is stored as BF16, or as FP32 and rounded on its way to LDS.
template <typename T>
struct Vec8;
template <>
struct Vec8<__bf16> {
    typedef bf16x8 type;
};
template <>
struct Vec8<float> {
    typedef f32x8 type;
};
__device__ inline bf16x8 rounded(const bf16x8& v) { return v; }
__device__ inline bf16x8 rounded(const f32x8& v) {
    bf16x8 w;
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = (__bf16)v[e];
    return w;
}

// 8 consecutive k of row r of a K-contiguous operand (leading dimension ld: a multiple of 8 for BF16, of 4 for
// FP32), zero outside rows < rows and k < kend.
template <typename T>
__device__ inline typename Vec8<T>::type load8(const T* __restrict__ p, int ld, int r, int k, int rows, int kend) {
    typedef typename Vec8<T>::type V;
    if (r < rows && k + 8 <= kend) return *reinterpret_cast<const V*>(p + (size_t)r * ld + k);
    V v;
    const T zero = (T)0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (r < rows && k + e < kend) ? p[(size_t)r * ld + k + e] : zero;
    return v;
}

// The epilogue of one output element v at (gm, gn), inside M x N; returns the BF16 value that also goes to
// the transposed copy.  C may be null where only H is wanted (inference needs no Z).
template <int EPI>
__device__ inline __bf16 epilogue(float v, int gm, int gn, float* __restrict__ C, int ldc,
                                  const float* __restrict__ bias, const float* __restrict__ Zin, int ldz,
                                  __bf16* __restrict__ Hout, int ldh) {
    const size_t o = (size_t)gm * ldc + gn;
    __bf16 tv = (__bf16)0.0f;
    if (EPI == EPI_STORE) {
        C[o] = v;
    } else if (EPI == EPI_BIAS) {
        C[o] = v + bias[gn];
    } else if (EPI == EPI_BIAS_GELU) {
        v += bias[gn];
        if (C != nullptr) C[o] = v;
        tv = (__bf16)gelu_f(v);
        Hout[(size_t)gm * ldh + gn] = tv;
    } else {
        v *= gelu_grad_f(Zin[(size_t)gm * ldz + gn]);
        C[o] = v;
        tv = (__bf16)v;
        Hout[(size_t)gm * ldh + gn] = tv;
    }
    return tv;
}

// The same for the columns gn and gn + 1 (gn, ldc, ldz and ldh even): one store of each kind.
template <int EPI>
__device__ inline void epilogue2(float2& v, int gm, int gn, float* __restrict__ C, int ldc,
                                 const float* __restrict__ bias, const float* __restrict__ Zin, int ldz,
                                 __bf16* __restrict__ Hout, int ldh) {
    float2* c = reinterpret_cast<float2*>(C + (size_t)gm * ldc + gn);
    if (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU) {
        v.x += bias[gn];
        v.y += bias[gn + 1];
    }
    if (EPI == EPI_GELU_GRAD) {
        const float2 z = *reinterpret_cast<const float2*>(Zin + (size_t)gm * ldz + gn);
        v.x *= gelu_grad_f(z.x);
        v.y *= gelu_grad_f(z.y);
    }
    if (EPI != EPI_BIAS_GELU || C != nullptr) *c = v;
    if (EPI == EPI_BIAS_GELU || EPI == EPI_GELU_GRAD) {
        bf16x2 h;
        h[0] = (__bf16)(EPI == EPI_BIAS_GELU ? gelu_f(v.x) : v.x);
        h[1] = (__bf16)(EPI == EPI_BIAS_GELU ? gelu_f(v.y) : v.y);
        *reinterpret_cast<bf16x2*>(Hout + (size_t)gm * ldh + gn) = h;
        v.x = (float)h[0];
        v.y = (float)h[1];
    }
}

// C[M x N] = A[M x K] B[N x K]^T.  (BM / WM) x (BN / WN) waves of 64 lanes, each computing a WM x WN
// tile of 32 x 32 MFMA tiles (v_mfma_f32_32x32x16_bf16); K in steps of BK = 64 staged through
// double-buffered LDS, the 16-byte global loads of the next PF = 2 steps held in registers (4 and 6 steps
// measured the same: the loop is bound by LDS and barriers, not by the loads).
// Eight wavefronts a block, with tiles that leave two each to every SIMD: one wavefront's GELU or LDS
// reads fill the other's waits (4096 x 512 x 512: 9.8 us with GELU and 13.9 with the gradient and both
// copies, with four wavefronts 12.7 and 18.8; 4096 x 512 x 4096 on 128 x 128 tiles 26.1 us, with four 29.0).
// K split: blockIdx.z = z takes k in [z kchunk, (z + 1) kchunk).  With a workspace `part` every block
// writes its FP32 partial tile to part[z] and k_splitk_epilogue adds the partials and applies the
// epilogue; without one (only when gridDim.z = 1) the block applies the epilogue itself, its tile passed
// through LDS so that rows, and rows of the transposed copy, leave in whole segments.
// TA = float: an FP32 A (the network's input in inference), rounded to BF16 between registers and LDS: 30.0 us for
// 4096 x 512 x 4096, against 26.7 and the 16.4 of a pass that writes the BF16 input.
template <typename TA, int BM, int BN_, int WM, int WN, int EPI>
__global__ __launch_bounds__((BM / WM) * (BN_ / WN) * 64) void k_gemm_nt(
    const TA* __restrict__ A, int lda, const __bf16* __restrict__ B, int ldb, int M, int N, int K,
    float* __restrict__ C, int ldc, const float* __restrict__ bias, const float* __restrict__ Zin, int ldz,
    __bf16* __restrict__ Hout, int ldh, __bf16* __restrict__ Tout, int ldt, int kchunk, float* __restrict__ part) {
    constexpr int WAVES_N = BN_ / WN, NT = (BM / WM) * WAVES_N * 64;
    constexpr int FM = WM / 32, FN = WN / 32;
    constexpr int RSTEP = NT / 8;                      // rows covered by one vector per thread
    constexpr int AV = BM / RSTEP, BV = BN_ / RSTEP;  // 16-byte vectors per thread per step
    static_assert(BM % RSTEP == 0 && BN_ % RSTEP == 0, "tile rows must be a multiple of threads / 8");
    constexpr int AS = BM * LDK, BS = BN_ * LDK, LDT = BN_ + 2;
    static_assert(BM * LDT * 4 <= 2 * (AS + BS) * 2, "the tile has to fit where the operands were");
    __shared__ __attribute__((aligned(16))) __bf16 smem[2 * (AS + BS)];
    __bf16* const As = smem;
    __bf16* const Bs = smem + 2 * AS;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    // Workgroups go to the 8 XCDs in turn (linear id mod 8), each XCD with its own L2.  With the grid's
    // row panels a multiple of 8, ids are remapped so that every tile of one row panel (one slice of A)
    // runs on the same XCD, which then fetches that slice once.
    int bx = blockIdx.x, by = blockIdx.y;
    if ((gridDim.y & 7) == 0) {
        const int id = blockIdx.x + gridDim.x * blockIdx.y, local = id >> 3;
        bx = local % gridDim.x;
        by = (local / gridDim.x) * 8 + (id & 7);
    }
    const int m0 = by * BM, n0 = bx * BN_;
    const int wm = (wave / WAVES_N) * WM, wn = (wave % WAVES_N) * WN;
    const int kb = blockIdx.z * kchunk, ke = min(K, kb + kchunk);
    const int kv = (t & 7) * 8, r0 = t >> 3;  // this thread's vectors: rows r0 + RSTEP i, k offset kv
    const bool inner_rows = m0 + BM <= M && n0 + BN_ <= N;  // uniform over the block
    constexpr int PF = 2;
    typename Vec8<TA>::type ra[PF][AV];
    bf16x8 rb[PF][BV];
    auto gload = [&](int st, int k0) {
        if (inner_rows && k0 + BK <= ke) {
            // the whole step lies inside both operands: plain 16-byte loads
#pragma unroll
            for (int i = 0; i < AV; ++i)
                ra[st][i] = *reinterpret_cast<const typename Vec8<TA>::type*>(A + (size_t)(m0 + r0 + RSTEP * i) * lda + k0 + kv);
#pragma unroll
            for (int i = 0; i < BV; ++i)
                rb[st][i] = *reinterpret_cast<const bf16x8*>(B + (size_t)(n0 + r0 + RSTEP * i) * ldb + k0 + kv);
        } else {
#pragma unroll
            for (int i = 0; i < AV; ++i) ra[st][i] = load8(A, lda, m0 + r0 + RSTEP * i, k0 + kv, M, ke);
#pragma unroll
            for (int i = 0; i < BV; ++i) rb[st][i] = load8(B, ldb, n0 + r0 + RSTEP * i, k0 + kv, N, ke);
        }
    };
    auto sstore = [&](int st, int buf) {
#pragma unroll
        for (int i = 0; i < AV; ++i)
            *reinterpret_cast<bf16x8*>(&As[buf * AS + (r0 + RSTEP * i) * LDK + kv]) = rounded(ra[st][i]);
#pragma unroll
        for (int i = 0; i < BV; ++i)
            *reinterpret_cast<bf16x8*>(&Bs[buf * BS + (r0 + RSTEP * i) * LDK + kv]) = rb[st][i];
    };
    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    // operand fragments: lane l holds row l % 32 of its 32-row tile, k = 8 (l / 32) .. + 7 of each 16
    const int fr = lane & 31, fk = 8 * (lane >> 5);
    const int steps = ke > kb ? (ke - kb + BK - 1) / BK : 0;
    static_assert(PF % 2 == 0, "a stage's LDS buffer is its parity");
#pragma unroll
    for (int st = 0; st < PF; ++st)
        if (st < steps) gload(st, kb + st * BK);
    for (int s0 = 0; s0 < steps; s0 += PF) {
#pragma unroll
        for (int st = 0; st < PF; ++st) {
            if (s0 + st >= steps) break;
            const int buf = st & 1;
            // the buffer's last readers passed the barrier of the step before this one
            sstore(st, buf);
            __syncthreads();
            if (s0 + st + PF < steps) gload(st, kb + (s0 + st + PF) * BK);
#pragma unroll
            for (int ks = 0; ks < BK; ks += 16) {
                bf16x8 a[FM], b[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    a[i] = *reinterpret_cast<const bf16x8*>(&As[buf * AS + (wm + 32 * i + fr) * LDK + ks + fk]);
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    b[j] = *reinterpret_cast<const bf16x8*>(&Bs[buf * BS + (wn + 32 * j + fr) * LDK + ks + fk]);
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        }
    }
    // D layout of a 32 x 32 tile: lane l holds column l % 32 and, in value r, row
    // 8 (r / 4) + 4 (l / 32) + r % 4
    if (part == nullptr) {
        // no workspace: the epilogue here (the host passes one whenever K is split)
        float* tile = reinterpret_cast<float*>(smem);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    tile[(wm + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * LDT + wn + 32 * j + fr] = acc[i][j][r];
        __syncthreads();
        // rows, two columns a lane
        const bool transposed = (EPI == EPI_BIAS_GELU || EPI == EPI_GELU_GRAD) && Tout != nullptr;
        const bool even = ((ldc | ldz | ldh) & 1) == 0 && (((uintptr_t)C | (uintptr_t)Zin) & 7) == 0;
        constexpr int LPR = BN_ / 2;
        const int col = 2 * (t % LPR), gn = n0 + col;
        for (int row = t / LPR; row < BM; row += NT / LPR) {
            const int gm = m0 + row;
            if (gm >= M) break;
            float2& at = *reinterpret_cast<float2*>(&tile[row * LDT + col]);
            float2 v = at;
            if (even && gn + 1 < N) {
                epilogue2<EPI>(v, gm, gn, C, ldc, bias, Zin, ldz, Hout, ldh);
            } else {
                if (gn < N) v.x = (float)epilogue<EPI>(v.x, gm, gn, C, ldc, bias, Zin, ldz, Hout, ldh);
                if (gn + 1 < N) v.y = (float)epilogue<EPI>(v.y, gm, gn + 1, C, ldc, bias, Zin, ldz, Hout, ldh);
            }
            if (transposed) at = v;
        }
        if (!transposed) return;
        __syncthreads();
        // rows of the transpose, four of its entries a lane (Tout's rows start 16-byte aligned)
        constexpr int LPC = BM / 4;
        const int row = 4 * (t % LPC);
        for (int c = t / LPC; c < BN_; c += NT / LPC) {
            if (n0 + c >= N) break;
            __bf16* tp = Tout + (size_t)(n0 + c) * ldt + m0 + row;
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (__bf16)tile[(row + e) * LDT + c];
            if (m0 + row + 4 <= M) {
                *reinterpret_cast<bf16x4*>(tp) = w;
            } else {
                for (int e = 0; e < 4 && m0 + row + e < M; ++e) tp[e] = w[e];
            }
        }
        return;
    }
    // split K: this block's partial tile
    float* mine = part + (size_t)blockIdx.z * M * N;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int gn = n0 + wn + 32 * j + fr;
            if (gn >= N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int gm = m0 + wm + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (gm < M) mine[(size_t)gm * N + gn] = acc[i][j][r];
            }
        }
}

// The split products' sum and epilogue: out(m, n) = sum over z = 0, 1, ... of part[z](m, n) (a fixed order,
// so the same sum on every run), then the epilogue.  32 x 32 tiles, 256 threads: coalesced reads and
// writes, the BF16 values staged in LDS for the transposed copy.
template <int EPI>
__global__ __launch_bounds__(256) void k_splitk_epilogue(const float* __restrict__ part, int splits, int M, int N,
                                                         float* __restrict__ C, int ldc, const float* __restrict__ bias,
                                                         const float* __restrict__ Zin, int ldz,
                                                         __bf16* __restrict__ Hout, int ldh, __bf16* __restrict__ Tout,
                                                         int ldt) {
    __shared__ __bf16 tile[32][33];
    const int n0 = blockIdx.x * 32, m0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const size_t mn = (size_t)M * N;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int rr = ty + 8 * i, gm = m0 + rr, gn = n0 + tx;
        __bf16 tv = (__bf16)0.0f;
        if (gm < M && gn < N) {
            const float* p = part + (size_t)gm * N + gn;
            // left to right over z, four partials loaded ahead of their adds
            float v = 0.f;
            int z = 0;
            for (; z + 4 <= splits; z += 4) {
                const float a0 = p[(size_t)z * mn], a1 = p[(size_t)(z + 1) * mn], a2 = p[(size_t)(z + 2) * mn],
                            a3 = p[(size_t)(z + 3) * mn];
                v += a0;
                v += a1;
                v += a2;
                v += a3;
            }
            for (; z < splits; ++z) v += p[(size_t)z * mn];
            tv = epilogue<EPI>(v, gm, gn, C, ldc, bias, Zin, ldz, Hout, ldh);
        }
        tile[rr][tx] = tv;
    }
    if ((EPI == EPI_BIAS_GELU || EPI == EPI_GELU_GRAD) && Tout != nullptr) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int cc = ty + 8 * i, gn = n0 + cc, gm = m0 + tx;
            if (gn < N && gm < M) Tout[(size_t)gn * ldt + gm] = tile[tx][cc];
        }
    }
}

// H = gelu(A W + b) for a few rows (M <= MR): a wavefront takes one column, its lanes eight k each, and
// every row's sum ends in the wavefront.  Bound by the latency of reading W^T once (4 MiB for 4096 x 512);
// the 64-row tiles of k_gemm_nt had four blocks to a row of tiles, K in splits and a second kernel to add
// them.  One row, 4096 -> 512 -> 512 -> 512: 13.5 us for the three products, on tiles 26 and the input's
// conversion.
template <typename TA, int MR>
__global__ __launch_bounds__(256) void k_rows(const TA* __restrict__ A, int lda, const __bf16* __restrict__ B, int ldb,
                                              int M, int N, int K, const float* __restrict__ bias,
                                              __bf16* __restrict__ Hout, int ldh) {
    constexpr int U = MR == 1 ? 4 : 1;  // steps of 512 k whose loads are sent together
    const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;
    float acc[MR];
#pragma unroll
    for (int m = 0; m < MR; ++m) acc[m] = 0.f;
    for (int k0 = 0; k0 < K; k0 += 512 * U) {
        bf16x8 b[U];
        typename Vec8<TA>::type a[U][MR];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 512 * u + 8 * lane;
            b[u] = load8(B, ldb, n, k, N, K);
#pragma unroll
            for (int m = 0; m < MR; ++m) a[u][m] = load8(A, lda, m, k, M, K);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                const bf16x8 w = rounded(a[u][m]);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[m] = fmaf((float)w[e], (float)b[u][e], acc[m]);
            }
    }
    float mine = 0.f;
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        float v = acc[m];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
        if (lane == m) mine = v;
    }
    if (lane < M) Hout[(size_t)lane * ldh + n] = (__bf16)gelu_f(mine + bias[n]);
}

// softmax over `classes` logits per row, loss sum, G = (p - onehot) / batch as fp32 (g, ld classes),
// bf16 (gb, ld ldgb) and transposed bf16 (gt: classes x batch, ld ldgt, optional)
__global__ void k_softmax_ce(const float* logits, const int32_t* labels, int batch, int classes, float* probs,
                             float* g, __bf16* gb, int ldgb, __bf16* gt, int ldgt, float* loss_sum) {
    const int i = threadIdx.x + blockIdx.x * blockDim.x;
    if (i >= batch) return;
    const float* z = logits + (size_t)i * classes;
    float m = z[0];
    for (int c = 1; c < classes; ++c) m = fmaxf(m, z[c]);
    float s = 0.f;
    for (int c = 0; c < classes; ++c) s += expf(z[c] - m);
    const int y = labels ? labels[i] : -1;
    for (int c = 0; c < classes; ++c) {
        const float p = expf(z[c] - m) / s;
        if (probs) probs[(size_t)i * classes + c] = p;
        if (g) {
            const float gv = (p - (c == y ? 1.f : 0.f)) / (float)batch;
            g[(size_t)i * classes + c] = gv;
            gb[(size_t)i * ldgb + c] = (__bf16)gv;
            if (gt) gt[(size_t)c * ldgt + i] = (__bf16)gv;
        }
    }
    if (loss_sum && y >= 0 && y < classes) atomicAdd(loss_sum, -(z[y] - m - logf(s)));
}

// The output layer of at most 32 classes in one kernel: logits = A B^T + bias (A: M x K, B: N x K), then
// k_softmax_ce's outputs.  A block takes 32 rows, its wavefront z the k of the product's split z in the
// order of k_gemm_nt, the splits' partial logits meet in LDS and are added in order: the same logits as
// from k_gemm_nt and k_splitk_epilogue, bit for bit.  With 11 classes the 64 x 128 tiles were nine tenths
// padding; 4096 x 512: 7.5 us, as three kernels 18 (23 with the gradient's outputs).
constexpr int HEAD_ROWS = 32, HEAD_MAX = 32, HEAD_LD = HEAD_MAX + 1, HEAD_SPLITS = 16;
__global__ __launch_bounds__(HEAD_SPLITS * 64) void k_head(const __bf16* __restrict__ A, int lda,
                                                           const __bf16* __restrict__ B, int ldb, int M, int N, int K,
                                                           int kchunk, const float* __restrict__ bias,
                                                           const int32_t* __restrict__ labels, float* __restrict__ probs,
                                                           float* __restrict__ g, __bf16* __restrict__ gb, int ldgb,
                                                           __bf16* __restrict__ gt, int ldgt, float* loss_sum) {
    __shared__ float red[HEAD_SPLITS][HEAD_ROWS * HEAD_LD];
    const int lane = threadIdx.x & 63, z = threadIdx.x >> 6, splits = blockDim.x >> 6;
    const int m0 = blockIdx.x * HEAD_ROWS;
    const int fr = lane & 31, fk = 8 * (lane >> 5);
    const int kb = z * kchunk, ke = min(K, kb + kchunk);
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    // rows past the last one repeat it: their sums are not looked at
    const __bf16* ap = A + (size_t)min(m0 + fr, M - 1) * lda + fk;
    const __bf16* bp = B + (size_t)min(fr, N - 1) * ldb + fk;
    int k = kb;
    // eight steps' loads together: taken step by step, each waited for its own
    for (; k + 128 <= ke; k += 128) {
        bf16x8 a[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            a[u] = *reinterpret_cast<const bf16x8*>(ap + k + 16 * u);
            b[u] = *reinterpret_cast<const bf16x8*>(bp + k + 16 * u);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u], b[u], acc, 0, 0, 0);
    }
    for (; k + 16 <= ke; k += 16)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(ap + k),
                                                      *reinterpret_cast<const bf16x8*>(bp + k), acc, 0, 0, 0);
    if (k < ke)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load8(A, lda, m0 + fr, k + fk, M, ke),
                                                      load8(B, ldb, fr, k + fk, N, ke), acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) red[z][(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * HEAD_LD + fr] = acc[r];
    __syncthreads();
    for (int i = threadIdx.x; i < HEAD_ROWS * HEAD_MAX; i += blockDim.x) {
        const int o = (i >> 5) * HEAD_LD + (i & 31);
        if ((i & 31) >= N) continue;
        float v = 0.f;
        for (int y = 0; y < splits; ++y) v += red[y][o];
        red[0][o] = v + bias[i & 31];
    }
    __syncthreads();
    const int i = m0 + (int)threadIdx.x;
    if (threadIdx.x >= HEAD_ROWS) return;
    float loss = 0.f;
    if (i < M) {
        float* l = &red[0][threadIdx.x * HEAD_LD];
        float m = l[0];
        for (int c = 1; c < N; ++c) m = fmaxf(m, l[c]);
        const int y = labels ? labels[i] : -1;
        const float zy = y >= 0 && y < N ? l[y] : 0.f;
        float s = 0.f;
        for (int c = 0; c < N; ++c) {
            const float e = expf(l[c] - m);
            l[c] = e;
            s += e;
        }
        for (int c = 0; c < N; ++c) {
            const float p = l[c] / s;
            if (probs) probs[(size_t)i * N + c] = p;
            if (g) {
                const float gv = (p - (c == y ? 1.f : 0.f)) / (float)M;
                g[(size_t)i * N + c] = gv;
                gb[(size_t)i * ldgb + c] = (__bf16)gv;
                if (gt) gt[(size_t)c * ldgt + i] = (__bf16)gv;
            }
        }
        if (y >= 0 && y < N) loss = -(zy - m - logf(s));
    }
    if (loss_sum == nullptr) return;
    // one addition a block (additions to one address take about 9 ns each)
#pragma unroll
    for (int d = HEAD_ROWS / 2; d >= 1; d >>= 1) loss += __shfl_down(loss, d, HEAD_ROWS);
    if (threadIdx.x == 0) atomicAdd(loss_sum, loss);
}

// Column sums of every layer's G (rows x out, row-major) in a fixed order: the bias gradients, in two
// launches for the whole network (two for each layer left 15 us between them at batch 4096).
// k_colsum_part: a block covers 64 columns x a slab of COLSUM_SLAB = 64 rows; its four groups of 64
// threads each load 16 consecutive rows of one column at once (coalesced across the columns), sum them
// in row order, and the four group sums are added in group order.  k_colsum_fin adds the slab sums the
// same way (four groups of consecutive slabs, then the groups in order).  A layer's columns are the strips
// strip0 .. of 64 and the columns 64 strip0 .. of part.
constexpr int COLSUM_SLAB = 64;

__device__ inline const MlpLayer& layer_of_strip(const MlpLayers& net, int strip) {
    int l = 0;
    while (l + 1 < net.count && strip >= net.l[l + 1].strip0) ++l;
    return net.l[l];
}

__global__ __launch_bounds__(256) void k_colsum_part(MlpLayers net, int rows, float* __restrict__ part) {
    __shared__ float red[4][64];
    const MlpLayer& y = layer_of_strip(net, (int)blockIdx.x);
    const float* __restrict__ g = y.g;
    const int cols = y.out, lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int col = ((int)blockIdx.x - y.strip0) * 64 + lane, r0 = blockIdx.y * COLSUM_SLAB + grp * 16;
    float a[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = (col < cols && r0 + i < rows) ? g[(size_t)(r0 + i) * cols + col] : 0.f;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += a[i];
    red[grp][lane] = sum;
    __syncthreads();
    if (grp == 0)
        part[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 64 + lane] =
            ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

__global__ __launch_bounds__(256) void k_colsum_fin(MlpLayers net, const float* __restrict__ part, int slabs) {
    __shared__ float red[4][64];
    const MlpLayer& y = layer_of_strip(net, (int)blockIdx.x);
    const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int col = ((int)blockIdx.x - y.strip0) * 64 + lane;
    const int per = (slabs + 3) / 4, z0 = grp * per, z1 = min(slabs, z0 + per);
    const size_t ld = (size_t)gridDim.x * 64;
    const float* mine = part + (size_t)blockIdx.x * 64 + lane;
    float sum = 0.f;
    int z = z0;
    for (; z + 8 <= z1; z += 8) {
        float a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = mine[(size_t)(z + i) * ld];
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += a[i];
    }
    for (; z < z1; ++z) sum += mine[(size_t)z * ld];
    red[grp][lane] = sum;
    __syncthreads();
    if (grp == 0 && col < y.out) y.db[col] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// x (rows x cols fp32, ld cols) -> y (bf16, ld ldy) and, if t != null, its transpose (cols x rows, ld
// ldt).  64 x 64 tiles through LDS, each thread 4 consecutive values per row: 16-byte loads, 8-byte
// stores in both directions (a row of 64 halves padded to 66 spreads a column read over the banks).
__global__ __launch_bounds__(256) void k_to_bf16_t(const float* __restrict__ x, int rows, int cols,
                                                   __bf16* __restrict__ y, int ldy, __bf16* __restrict__ t, int ldt) {
    __shared__ __bf16 tile[64][66];
    const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
    const int q = (threadIdx.x & 15) * 4, tr = threadIdx.x >> 4;  // 16 groups of 4 columns x 16 rows
    const bool vec = (cols & 3) == 0 && (ldy & 3) == 0;
    for (int rr = tr; rr < 64; rr += 16) {
        const int r = r0 + rr, c = c0 + q;
        bf16x4 v;
        if (r < rows && vec && c + 4 <= cols) {
            const float4 f = *reinterpret_cast<const float4*>(x + (size_t)r * cols + c);
            v[0] = (__bf16)f.x;
            v[1] = (__bf16)f.y;
            v[2] = (__bf16)f.z;
            v[3] = (__bf16)f.w;
            *reinterpret_cast<bf16x4*>(y + (size_t)r * ldy + c) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = (__bf16)0.0f;
                if (r < rows && c + e < cols) {
                    v[e] = (__bf16)x[(size_t)r * cols + c + e];
                    y[(size_t)r * ldy + c + e] = v[e];
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[rr][q + e] = v[e];
    }
    if (!t) return;
    __syncthreads();
    const bool tvec = (ldt & 3) == 0;
    for (int cc = tr; cc < 64; cc += 16) {
        const int c = c0 + cc, r = r0 + q;
        if (c >= cols) continue;
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = tile[q + e][cc];
        if (tvec && r + 4 <= rows) {
            *reinterpret_cast<bf16x4*>(t + (size_t)c * ldt + r) = w;
        } else {
            for (int e = 0; e < 4 && r + e < rows; ++e) t[(size_t)c * ldt + r + e] = w[e];
        }
    }
}

// W (rows x cols fp32, ld cols) -> Wb (bf16, ld ldb) and W^T (bf16, cols x rows, ld ldt)
__global__ __launch_bounds__(256) void k_weights_bf16(const float* __restrict__ w, int rows, int cols,
                                                      __bf16* __restrict__ wb, int ldb, __bf16* __restrict__ wt,
                                                      int ldt) {
    __shared__ __bf16 tile[32][33];
    const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int rr = ty; rr < 32; rr += 8) {
        const int r = r0 + rr, c = c0 + tx;
        __bf16 v = (__bf16)0.0f;
        if (r < rows && c < cols) {
            v = (__bf16)w[(size_t)r * cols + c];
            wb[(size_t)r * ldb + c] = v;
        }
        tile[rr][tx] = v;
    }
    __syncthreads();
    for (int cc = ty; cc < 32; cc += 8) {
        const int c = c0 + cc, r = r0 + tx;
        if (c < cols && r < rows) wt[(size_t)c * ldt + r] = tile[tx][cc];
    }
}

// Adam (Kingma & Ba 2015) on the FP32 master copy and the new weights' BF16 copies in both orientations, all
// layers in one launch: 32 x 32 tiles of each layer's (in + 1) x out parameters, the last row its bias.
// A weight gradient whose K was split comes as its partial products, summed here in the order of
// k_splitk_epilogue, so that it is not written and read again.  Bound by memory (seven words a parameter
// and a word a split).  The 2.6 million parameters of the 4096 -> 512 x 3 -> 11 network at batch 4096 (4, 8, 8
// and 16 splits): 34 us, with the sums and the copies in passes of their own for each layer 24 + 16 + 17.
__global__ __launch_bounds__(256) void k_adam(MlpLayers net, float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                              float b2, float eps, float c1, float c2) {
    __shared__ __bf16 tile[32][33];
    int l = 0;
    while (l + 1 < net.count && (int)blockIdx.x >= net.l[l + 1].tile0) ++l;
    const MlpLayer& y = net.l[l];
    const int across = (y.out + 31) / 32, at = (int)blockIdx.x - y.tile0;
    const int c0 = at % across * 32, r0 = at / across * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    __bf16* wb = (__bf16*)y.wb;
    __bf16* wt = (__bf16*)y.wt;
#pragma unroll
    for (int rr = ty; rr < 32; rr += 8) {
        const int r = r0 + rr, c = c0 + tx;
        if (r > y.in || c >= y.out) continue;
        const int64_t o = (int64_t)r * y.out + c, i = y.w + o;
        float gi = 0.f;
        if (y.splits > 1 && r < y.in) {
            const float* part = y.part + o;
            const int64_t wn = (int64_t)y.in * y.out;
            int z = 0;
            for (; z + 4 <= y.splits; z += 4) {
                const float a0 = part[z * wn], a1 = part[(z + 1) * wn], a2 = part[(z + 2) * wn], a3 = part[(z + 3) * wn];
                gi += a0;
                gi += a1;
                gi += a2;
                gi += a3;
            }
            for (; z < y.splits; ++z) gi += part[z * wn];
        } else {
            gi = g[i];
        }
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        p[i] = pi;
        if (r == y.in) continue;
        tile[rr][tx] = (__bf16)pi;
        wb[(size_t)r * y.ldb + c] = (__bf16)pi;
    }
    __syncthreads();
#pragma unroll
    for (int cc = ty; cc < 32; cc += 8) {
        const int c = c0 + cc, r = r0 + tx;
        if (c < y.out && r < y.in) wt[(size_t)c * y.ldt + r] = tile[tx][cc];
    }
}

// seeded initialisation: W uniform in [-1/sqrt(fan_in), 1/sqrt(fan_in)] from SplitMix64 outputs of
// the running index (u = (r >> 40) / 2^24), biases zero
__global__ void k_init(float* w, int64_t count, int64_t index0, int fan_in, uint64_t seed) {
    const double bound = 1.0 / sqrt((double)fan_in);
    for (int64_t i = threadIdx.x + (int64_t)blockIdx.x * blockDim.x; i < count; i += (int64_t)blockDim.x * gridDim.x) {
        const uint64_t r = sm64(seed, (uint64_t)(index0 + i));
        const double u = (double)(r >> 40) / 16777216.0;
        w[i] = (float)__dmul_rn(__dsub_rn(__dmul_rn(2.0, u), 1.0), bound);
    }
}

int cu_count() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            cus = v;
        else
            cus = 256;
    }
    return cus;
}

// Tiles of 128 x 128 (eight waves of 64 x 32) for the long products with many rows (M and K at least
// 2048), where the larger tile's operand reuse pays; else 64 x 128.  With fewer rows or a short K the
// 128 x 128 grid needs a deeper K split to fill the CUs, and its partials (written, then read back by
// the split sum) cost more than the smaller tile loses: on MI355X the 4096 x 512 x 512 products and the
// 512 x 512 x 4096 weight gradients take 4.7 us less, split sums included, on 64 x 128 tiles.
bool big_tiles(int M, int N, int K) { return M >= 2048 && N >= 128 && K >= 2048; }

int64_t tiles_of(int M, int N, int K) {
    const int bm = big_tiles(M, N, K) ? 128 : 64;
    return (int64_t)((M + bm - 1) / bm) * ((N + BN - 1) / BN);
}

// K is split until the grid holds about two workgroups per CU with 128 x 128 tiles (two fit in LDS and
// registers) or one with 64 x 128 tiles, with at least four K steps (256 k) per workgroup and at most
// 16 splits.
int splits_of(int M, int N, int K) {
    const int64_t tiles = tiles_of(M, N, K);
    const int64_t target = (big_tiles(M, N, K) ? 2 : 1) * (int64_t)cu_count();
    int splits = 1;
    while (splits < 16 && tiles * splits < target && K / (2 * splits) >= 4 * BK) splits *= 2;
    return splits;
}

// The most rows for which a product may take a wavefront per column instead of tiles (mlp_rows_fits).
constexpr int ROWS_MAX = 8;

template <int EPI, typename TA>
hipError_t gemm_nt_t(const TA* A, int lda, const __bf16* B, int ldb, int M, int N, int K, float* C, int ldc,
                     const float* bias, const float* Z, int ldz, __bf16* H, int ldh, __bf16* T, int ldt, float* part,
                     size_t part_floats, hipStream_t s, bool sum = true) {
    if (M <= 0 || N <= 0) return hipSuccess;
    int splits = splits_of(M, N, K);
    bool via_part = splits > 1;
    if (via_part && (part == nullptr || part_floats < (size_t)splits * M * N)) {
        splits = 1;  // no workspace: one workgroup per tile, epilogue in the GEMM
        via_part = false;
    }
    const int kchunk = ((K + splits - 1) / splits + BK - 1) / BK * BK;
    if (big_tiles(M, N, K)) {
        dim3 grid((N + BN - 1) / BN, (M + 127) / 128, splits);
        hipLaunchKernelGGL((k_gemm_nt<TA, 128, BN, 64, 32, EPI>), grid, dim3(512), 0, s, A, lda, B, ldb, M, N, K, C, ldc,
                           bias, Z, ldz, H, ldh, T, ldt, kchunk, via_part ? part : nullptr);
    } else {
        dim3 grid((N + BN - 1) / BN, (M + 63) / 64, splits);
        hipLaunchKernelGGL((k_gemm_nt<TA, 64, BN, 32, 32, EPI>), grid, dim3(512), 0, s, A, lda, B, ldb, M, N, K, C, ldc,
                           bias, Z, ldz, H, ldh, T, ldt, kchunk, via_part ? part : nullptr);
    }
    if (via_part && sum) {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        dim3 grid((N + 31) / 32, (M + 31) / 32);
        hipLaunchKernelGGL((k_splitk_epilogue<EPI>), grid, dim3(256), 0, s, part, splits, M, N, C, ldc, bias, Z, ldz,
                           H, ldh, T, ldt);
    }
    return hipGetLastError();
}

}  // namespace

size_t mlp_gemm_part_floats(int M, int N, int K) {
    // splits x M x N partials; M x N when unsplit, which serves the split products of smaller batches
    return (size_t)splits_of(M, N, K) * M * N;
}

static int colsum_slabs(int rows) { return (rows + COLSUM_SLAB - 1) / COLSUM_SLAB; }

size_t mlp_colsum_part_floats(int rows, const MlpLayers& net) { return (size_t)colsum_slabs(rows) * net.strips * 64; }

hipError_t mlp_gemm_nt(int epi, const void* A, int lda, const void* B, int ldb, int M, int N, int K, float* C, int ldc,
                       const float* bias, const float* Z, int ldz, void* H, int ldh, void* T, int ldt, float* part,
                       size_t part_floats, hipStream_t s) {
    const __bf16* a = (const __bf16*)A;
    const __bf16* b = (const __bf16*)B;
    __bf16* h = (__bf16*)H;
    __bf16* t = (__bf16*)T;
    switch (epi) {
        case EPI_STORE:
            return gemm_nt_t<EPI_STORE>(a, lda, b, ldb, M, N, K, C, ldc, bias, Z, ldz, h, ldh, t, ldt, part,
                                        part_floats, s);
        case EPI_BIAS:
            return gemm_nt_t<EPI_BIAS>(a, lda, b, ldb, M, N, K, C, ldc, bias, Z, ldz, h, ldh, t, ldt, part,
                                       part_floats, s);
        case EPI_BIAS_GELU:
            return gemm_nt_t<EPI_BIAS_GELU>(a, lda, b, ldb, M, N, K, C, ldc, bias, Z, ldz, h, ldh, t, ldt, part,
                                            part_floats, s);
        case EPI_GELU_GRAD:
            return gemm_nt_t<EPI_GELU_GRAD>(a, lda, b, ldb, M, N, K, C, ldc, bias, Z, ldz, h, ldh, t, ldt, part,
                                            part_floats, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t mlp_gemm_nt_f32(const float* A, int lda, const void* B, int ldb, int M, int N, int K, const float* bias,
                           void* H, int ldh, float* part, size_t part_floats, hipStream_t s) {
    if ((lda & 3) != 0 || ((uintptr_t)A & 15) != 0) return hipErrorInvalidValue;
    return gemm_nt_t<EPI_BIAS_GELU>(A, lda, (const __bf16*)B, ldb, M, N, K, nullptr, N, bias, nullptr, 0, (__bf16*)H,
                                    ldh, nullptr, 0, part, part_floats, s);
}

int mlp_gemm_splits(int M, int N, int K) { return splits_of(M, N, K); }

hipError_t mlp_gemm_parts(const void* A, int lda, const void* B, int ldb, int M, int N, int K, float* part,
                          size_t part_floats, hipStream_t s) {
    const int splits = splits_of(M, N, K);
    if (splits < 2 || part == nullptr || part_floats < (size_t)splits * M * N) return hipErrorInvalidValue;
    return gemm_nt_t<EPI_STORE>((const __bf16*)A, lda, (const __bf16*)B, ldb, M, N, K, nullptr, N, nullptr, nullptr, 0,
                                nullptr, 0, nullptr, 0, part, part_floats, s, false);
}

// A wavefront per column or tiles, for a few rows.  k_rows saves the second kernel that tiles need once their K is
// split (from 512 on), but every column reads all rows again and waits for a load every 512 k (2,048 k for one row,
// whose loads are sent four steps together).  So one row takes it unless K is short or the columns are many for
// their K; more rows only for a K in between, which ends earlier where A is FP32 and twice as long.  A product and
// the rest of a pass, wavefront per column against tiles in us: 1 x 512 x 4096 22.2, 26.6; 1 x 96 x 64 23.9, 21.9;
// 1 x 8192 x 256 34.7, 32.5; 8 x 2048 x 1024 (FP32) 25.9, 27.7; 2 x 512 x 4096 (FP32) 33.6, 27.0; 8 x 8192 x 1024
// (FP32) 42.8, 37.5.  A hidden layer alone: 8 x 512 x 512 3.7, 11.1; 2 x 2048 x 2048 9.8, 11.1; 2 x 2560 x 2560 12.6,
// 11.1; 8 x 256 x 256 5.5, 4.9.
bool mlp_rows_fits(int M, int N, int K, bool f32) {
    if (M > ROWS_MAX) return false;
    if (M == 1) return K >= 192 && N <= (int64_t)16 * K;
    return N <= 2048 && (f32 ? K >= 256 && K <= 1536 : K >= 384 && K <= 2048);
}

// Whether the first product of inference reads its FP32 input itself.  That saves the conversion pass, but each
// panel of 128 columns then reads four bytes where it would read two: worth it up to 16 panels, or 8 where a
// tile's rows of A no longer stay in an XCD's L2 (128 x 8192 x 4 bytes), and for any N while the pass is mostly its
// launch.  FP32 against converted in us: 4096 x 512 x 4096 56.5, 68.4; 4096 x 2048 x 4096 120, 125; 4096 x 4096 x 4096
// 232, 223; 4096 x 1024 x 16384 0.92 of it, 4096 x 4096 x 16384 834, 751; 64 x 4096 x 4096 43.6, 46.2; 256 x 8192 x 4096
// 81.0, 79.6.
bool mlp_f32_fits(int M, int N, int K) {
    return N <= 1024 || (N <= 2048 && K <= 8192) || (int64_t)M * K <= (1 << 21);
}

hipError_t mlp_rows(const void* A, bool f32, int lda, const void* B, int ldb, int M, int N, int K, const float* bias,
                    void* H, int ldh, hipStream_t s) {
    if (M < 1 || M > ROWS_MAX || (f32 && ((lda & 3) != 0 || ((uintptr_t)A & 15) != 0))) return hipErrorInvalidValue;
    const dim3 grid((N + 3) / 4);
    const __bf16* b = (const __bf16*)B;
    auto go = [&]<typename TA>(const TA* a) {
        if (M == 1)
            hipLaunchKernelGGL((k_rows<TA, 1>), grid, dim3(256), 0, s, a, lda, b, ldb, M, N, K, bias, (__bf16*)H, ldh);
        else
            hipLaunchKernelGGL((k_rows<TA, ROWS_MAX>), grid, dim3(256), 0, s, a, lda, b, ldb, M, N, K, bias, (__bf16*)H,
                               ldh);
    };
    if (f32)
        go((const float*)A);
    else
        go((const __bf16*)A);
    return hipGetLastError();
}

hipError_t mlp_softmax_ce(const float* logits, const int32_t* labels, int batch, int classes, float* probs, float* g,
                          void* gb, int ldgb, void* gt, int ldgt, float* loss_sum, hipStream_t s) {
    hipLaunchKernelGGL(k_softmax_ce, dim3((batch + 255) / 256), dim3(256), 0, s, logits, labels, batch, classes, probs,
                       g, (__bf16*)gb, ldgb, (__bf16*)gt, ldgt, loss_sum);
    return hipGetLastError();
}

hipError_t mlp_head(const void* A, int lda, const void* B, int ldb, int M, int N, int K, const float* bias,
                    const int32_t* labels, float* probs, float* g, void* gb, int ldgb, void* gt, int ldgt,
                    float* loss_sum, hipStream_t s) {
    if (M <= 0) return hipSuccess;
    if (N < 1 || N > HEAD_MAX) return hipErrorInvalidValue;
    const int splits = splits_of(M, N, K);
    const int kchunk = ((K + splits - 1) / splits + BK - 1) / BK * BK;
    hipLaunchKernelGGL(k_head, dim3((M + HEAD_ROWS - 1) / HEAD_ROWS), dim3(64 * splits), 0, s, (const __bf16*)A, lda,
                       (const __bf16*)B, ldb, M, N, K, kchunk, bias, labels, probs, g, (__bf16*)gb, ldgb, (__bf16*)gt,
                       ldgt, loss_sum);
    return hipGetLastError();
}

// A block of k_head reads its (up to 32) rows and B alone, on one CU, which three kernels on split tiles overtake
// where K is long, the blocks are few and what a block reads is much.  In us, k_head against the three: 4096 x 11 x
// 4096 44.1, 60.9; 32 x 11 x 4096 30.1, 33.2; 8 x 11 x 8192 32.4, 34.0; 32 x 11 x 8192 40.2, 38.0; 1 x 11 x 16384 40.0,
// 42.9; 8 x 11 x 16384 45.1, 43.5; 32 x 11 x 16384 61.2, 47.6; 4096 x 11 x 16384 137, 186; 32 x 32 x 65536 245, 109; at
// K = 6144 0.85 to 1.02 of them, from 512 rows on at K = 8192 0.91 to 1.04.
bool mlp_head_fits(int M, int N, int K) {
    if (N > HEAD_MAX) return false;
    if (K <= 6144 || M >= 2048 || (M >= 512 && K <= 8192)) return true;
    return (int64_t)K * (N + (M < HEAD_ROWS ? M : HEAD_ROWS)) <= 1 << 18;
}

hipError_t mlp_colsum(const MlpLayers& net, int rows, float* part, size_t part_floats, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    if (part == nullptr || part_floats < mlp_colsum_part_floats(rows, net)) return hipErrorInvalidValue;
    const int slabs = colsum_slabs(rows);
    hipLaunchKernelGGL(k_colsum_part, dim3(net.strips, (unsigned)slabs), dim3(256), 0, s, net, rows, part);
    hipLaunchKernelGGL(k_colsum_fin, dim3(net.strips), dim3(256), 0, s, net, part, slabs);
    return hipGetLastError();
}

hipError_t mlp_input_bf16(const float* x, int rows, int cols, void* y, int ldy, void* t, int ldt, hipStream_t s) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    dim3 grid((cols + 63) / 64, (rows + 63) / 64);
    hipLaunchKernelGGL(k_to_bf16_t, grid, dim3(256), 0, s, x, rows, cols, (__bf16*)y, ldy, (__bf16*)t, ldt);
    return hipGetLastError();
}

hipError_t mlp_weights_bf16(const float* w, int rows, int cols, void* wb, int ldb, void* wt, int ldt, hipStream_t s) {
    dim3 grid((cols + 31) / 32, (rows + 31) / 32);
    hipLaunchKernelGGL(k_weights_bf16, grid, dim3(256), 0, s, w, rows, cols, (__bf16*)wb, ldb, (__bf16*)wt, ldt);
    return hipGetLastError();
}

hipError_t mlp_adam(const MlpLayers& net, float* p, const float* g, float* m, float* v, float lr, float b1, float b2,
                    float eps, int step, hipStream_t s) {
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(net.tiles), dim3(256), 0, s, net, p, g, m, v, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t mlp_init(float* w, int64_t count, int64_t index0, int fan_in, uint64_t seed, hipStream_t s) {
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65535) blocks = 65535;
    hipLaunchKernelGGL(k_init, dim3((unsigned)blocks), dim3(256), 0, s, w, count, index0, fan_in, seed);
    return hipGetLastError();
}

}  // namespace tcw
