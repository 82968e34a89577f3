// Axis contractions of the angular transform (Sec. 4.1): one small dense matrix
// (the azimuthal DFT, or the per-m associated Legendre block) applied along one
// grid axis for every radial point; radius is the fastest axis of both layouts,
// so every load and store is coalesced along it.
//  * axis_mfma (complex64) and axis_mfma64 (complex128): the contraction as a
//    real product on the matrix cores, for matrices up to 64 x 64 in real form
//    (every Legendre block; the DFT while 2 N_phi <= 64).
//  * axis_mfma_big: the complex64 DFT for 64 < 2 N_phi <= 128, matrix in LDS.
//  * axis_apply: the vector kernel for the larger complex128 DFT.  A workgroup
//    takes one outer index and 64 consecutive radial points: their Q input
//    vectors and the Q x Q matrix are staged in LDS, and each of the four waves
//    accumulates every fourth output row for its 64 points, reading the matrix
//    as LDS broadcasts (one element per row and input, the same for the whole
//    wave).
//  * sht_both (complex64): both axis steps in one launch, where the N_theta x
//    N_phi values of 16 points fit in LDS.
// grid_phase and momentum_order are the diagonal factors and the reordering
// of the 3D split steps.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <vector>

#include "angular.h"

namespace dsbt {

namespace {

template <typename S> struct Cx;
template <> struct Cx<float> { typedef float2 t; };
template <> struct Cx<double> { typedef double2 t; };

constexpr int kRows = kShtMaxQ / 4;   // output rows per thread

// LDS bytes of one workgroup: 64 points x Q4 inputs and the Q x Q4 matrix, Q4 =
// Q rounded up to 4 (zero-padded), so that a wave reads four matrix columns as
// one 16-byte (real) or two (complex) broadcasts
__host__ __device__ constexpr int round4(int q) { return (q + 3) & ~3; }
template <typename S, bool CA>
constexpr size_t axis_lds_bytes(int Q) {
    return sizeof(typename Cx<S>::t) * 64 * (size_t)round4(Q) + sizeof(S) * (CA ? 2 : 1) * (size_t)Q * round4(Q);
}

template <typename S, bool CA>
__global__ void __launch_bounds__(256) axis_apply(const S* __restrict__ mat, int64_t mso, int tr, int cj,
                                                  const typename Cx<S>::t* __restrict__ src, int64_t so, int64_t sq,
                                                  typename Cx<S>::t* __restrict__ dst, int64_t dout, int64_t dq,
                                                  int Q, int Nr) {
    using V = typename Cx<S>::t;
    constexpr int AW = CA ? 2 : 1;   // scalars per matrix element
    const int Q4 = round4(Q);
    extern __shared__ __align__(16) unsigned char lds_raw[];
    V* X = reinterpret_cast<V*>(lds_raw);                       // X[q * 64 + point], q < Q4
    S* A = reinterpret_cast<S*>(lds_raw + sizeof(V) * 64 * Q4);  // A[(q' Q4 + q) AW], untransposed, q < Q4
    const int o = blockIdx.y;
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index (uniform)
    const bool live = i < Nr;
    // Staging: every lane issues its loads from addresses clamped into the rows,
    // points and matrix elements that exist, with no branch, and zeroes the rest
    // when it writes LDS; a load under a branch would be waited for inside it,
    // one round trip after another.
    {
        const int ic = min(i, Nr - 1);
        V xin[kShtMaxQ / 4];
#pragma unroll
        for (int u = 0; u < kShtMaxQ / 4; ++u) xin[u] = src[o * so + min(r + 4 * u, Q - 1) * sq + ic];
        constexpr int kMatPerThread = kShtMaxQ * kShtMaxQ / 256;
        const S* Ag = mat + o * mso;
        S av[kMatPerThread][AW];
#pragma unroll
        for (int u = 0; u < kMatPerThread; ++u) {
            const int e = min((int)threadIdx.x + 256 * u, Q * Q4 - 1);
            const int qo = e / Q4, q = min(e - qo * Q4, Q - 1);
            const int64_t g = tr ? (int64_t)q * Q + qo : (int64_t)qo * Q + q;
#pragma unroll
            for (int c = 0; c < AW; ++c) av[u][c] = Ag[AW * g + c];
        }
#pragma unroll
        for (int u = 0; u < kShtMaxQ / 4; ++u) {
            const int q = r + 4 * u;
            if (q < Q4) X[q * 64 + (threadIdx.x & 63)] = (live && q < Q) ? xin[u] : V{0, 0};
        }
#pragma unroll
        for (int u = 0; u < kMatPerThread; ++u) {
            const int e = threadIdx.x + 256 * u;
            if (e < Q * Q4) {
                const int qo = e / Q4, q = e - qo * Q4;
                if constexpr (CA) {
                    A[2 * e] = q < Q ? av[u][0] : S(0);
                    A[2 * e + 1] = q < Q ? (cj ? -av[u][1] : av[u][1]) : S(0);
                } else {
                    A[e] = q < Q ? av[u][0] : S(0);
                }
            }
        }
    }
    __syncthreads();
    V acc[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) acc[u] = V{0, 0};
    for (int q = 0; q < Q4; q += 4) {
        V x[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = X[(q + c) * 64 + (threadIdx.x & 63)];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int qo = r + 4 * u;
            if (qo < Q) {
                const S* a = A + ((size_t)qo * Q4 + q) * AW;
                if constexpr (CA) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const S ar = a[2 * c], ai = a[2 * c + 1];
                        acc[u].x += ar * x[c].x - ai * x[c].y;
                        acc[u].y += ar * x[c].y + ai * x[c].x;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        acc[u].x += a[c] * x[c].x;
                        acc[u].y += a[c] * x[c].y;
                    }
                }
            }
        }
    }
    if (!live) return;
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
        const int qo = r + 4 * u;
        if (qo < Q) dst[o * dout + qo * dq + i] = acc[u];
    }
}

// Axis step on the matrix cores, complex64 data, as one real FP32 product
// D = A X of (Q16 x Q16) x (Q16 x NCOL) per block of 64 radial points,
// Q16 = 16 NR:
//  * real matrix (the per-m Legendre blocks): it acts on real and imaginary
//    parts alike, so the 64 points are NCOL = 128 real columns (2 i + part)
//    and the contraction index is q;
//  * complex matrix (the azimuthal DFT): the contraction index is k = 2 q + part
//    and the output row 2 q' + part', with A = [[Re, -Im], [Im, Re]] per element,
//    so the 64 points are NCOL = 64 columns.
// Workgroup (x, o) takes the point blocks x, x + gridDim.x, ... of outer index
// o: its matrix is loaded once (into registers, or for the real form into LDS),
// and the inputs of the next block are loaded into registers while the current
// one is multiplied and stored, so that memory and matrix work overlap inside
// the workgroup.  The
// inputs are staged transposed in LDS (Xt[column][k], row pitch Q16 + 4 floats,
// so that the 16-byte reads of 16 lanes cover all 64 banks once); wave w takes
// NCOL / 4 columns and every row block.  v_mfma_f32_16x16x4_f32: lane l
// supplies A[l%16][l/16] and B[l/16][l%16], result register v of lane l is
// D[4 (l/16) + v][l%16].  The contraction index is split as
// k = 16 G + 4 (l/16) + s for instruction s of group G, so that each lane holds
// the four k of its four instructions as one 16-byte word, of the zero-padded
// matrix (row-major [Q16][Q16] at mat16 + o mso in global memory; As, pitch XS,
// for the real form) and of Xt.
// Results pass through LDS (over Xt, row pitch NCOL + 4 floats: conflict-free)
// and are written back coalesced.
typedef float f4v __attribute__((ext_vector_type(4)));

template <int NR, bool CPX>
__global__ void __launch_bounds__(256) axis_mfma(const float* __restrict__ mat16, int64_t mso,
                                                 const float2* __restrict__ src, int64_t so, int64_t sq,
                                                 float2* __restrict__ dst, int64_t dout, int64_t dq, int Q, int Nr) {
    constexpr int Q16 = 16 * NR, XS = Q16 + 4;
    constexpr int NCOL = CPX ? 64 : 128, NCB = NCOL / 64, YP = NCOL + 4;
    constexpr int NPF = CPX ? 2 : 4;   // input rows per staging item
    static_assert(Q16 * YP <= NCOL * XS, "result staging must fit in the input buffer");
    __shared__ __align__(16) float Xt[NCOL * XS];
    const int o = blockIdx.y;
    const int nblk = (Nr + 63) / 64;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float2* sp = src + o * so;
    float2* dp = dst + o * dout;
    // the matrix fragments: the complex form (at most 64 x 64, shared by every
    // outer index) in registers for the whole workgroup; the real per-m block
    // staged once in LDS (As[row][k], pitch XS), which leaves registers for a
    // third workgroup per compute unit
    f4v a[CPX ? NR : 1][NR];   // [G][rb]
    __shared__ __align__(16) float As[CPX ? 4 : Q16 * XS];
    if constexpr (CPX) {
        const float* Am = mat16 + o * mso + (lane & 15) * Q16 + 4 * (lane >> 4);
#pragma unroll
        for (int G = 0; G < NR; ++G)
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) a[G][rb] = *reinterpret_cast<const f4v*>(Am + 16 * rb * Q16 + 16 * G);
        // have them in registers here: a first use inside the block loop would
        // put a wait on every memory operation in flight into each iteration
#pragma unroll
        for (int G = 0; G < NR; ++G)
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) asm volatile("" ::"v"(a[G][rb]));
    } else {
        for (int e = threadIdx.x; e < Q16 * Q16 / 4; e += 256) {
            const int r = e / (Q16 / 4), k4 = e - r * (Q16 / 4);
            *reinterpret_cast<f4v*>(As + r * XS + 4 * k4) =
                *reinterpret_cast<const f4v*>(mat16 + o * mso + r * Q16 + 4 * k4);
        }
    }
    // staging item (g, il) = threadIdx.x + 256 u holds the contraction indices
    // 4 g .. 4 g + 3 of point il: input rows 2 g, 2 g + 1 (complex matrix) or
    // 4 g .. 4 g + 3 (real matrix)
    float2 pf[NR][NPF];
    // Every lane loads from an address clamped into the rows and points that
    // exist, with no branch, and the values outside are zeroed only when they
    // are staged: a load under a branch, or a value selected right after its
    // load, would be waited for at once, and the loads of the next block are
    // meant to stay in flight while the current one is multiplied.  Past the
    // last block every lane reads the same clamped element.
    auto fetch = [&](int bx) {
        const int ic = min(bx * 64 + (threadIdx.x & 63), Nr - 1);
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int g = (threadIdx.x + 256 * u) >> 6;
#pragma unroll
            for (int c = 0; c < NPF; ++c) pf[u][c] = sp[min(NPF * g + c, Q - 1) * sq + ic];
        }
    };
    int bx = blockIdx.x;
    fetch(bx);
    for (; bx < nblk; bx += gridDim.x) {
        const bool live = bx * 64 + (threadIdx.x & 63) < Nr;
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int e = threadIdx.x + 256 * u, il = e & 63, g = e >> 6;
            float2 v[NPF];
#pragma unroll
            for (int c = 0; c < NPF; ++c) v[c] = (live && NPF * g + c < Q) ? pf[u][c] : float2{0.f, 0.f};
            if constexpr (CPX) {
                *reinterpret_cast<f4v*>(Xt + il * XS + 4 * g) = f4v{v[0].x, v[0].y, v[1].x, v[1].y};
            } else {
                *reinterpret_cast<f4v*>(Xt + (2 * il) * XS + 4 * g) = f4v{v[0].x, v[1].x, v[2].x, v[3].x};
                *reinterpret_cast<f4v*>(Xt + (2 * il + 1) * XS + 4 * g) = f4v{v[0].y, v[1].y, v[2].y, v[3].y};
            }
        }
        __syncthreads();
        fetch(bx + gridDim.x);
        f4v acc[NR][NCB];
#pragma unroll
        for (int rb = 0; rb < NR; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) acc[rb][cb] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int G = 0; G < NR; ++G) {
            f4v ag[NR];
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) {
                if constexpr (CPX)
                    ag[rb] = a[G][rb];
                else
                    ag[rb] = *reinterpret_cast<const f4v*>(As + (16 * rb + (lane & 15)) * XS + 16 * G + 4 * (lane >> 4));
            }
            f4v b[NCB];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
                b[cb] = *reinterpret_cast<const f4v*>(Xt + (16 * (NCB * w + cb) + (lane & 15)) * XS + 16 * G +
                                                      4 * (lane >> 4));
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int rb = 0; rb < NR; ++rb)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
                        acc[rb][cb] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(ag[rb][s], b[cb][s], acc[rb][cb], 0, 0, 0);
        }
        __syncthreads();
        float* Ys = Xt;   // Ys[row][column], pitch YP
#pragma unroll
        for (int rb = 0; rb < NR; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    Ys[(16 * rb + 4 * (lane >> 4) + v) * YP + 16 * (NCB * w + cb) + (lane & 15)] = acc[rb][cb][v];
        __syncthreads();
        const int i0 = bx * 64;
        for (int e = threadIdx.x; e < Q * 64; e += 256) {
            const int t = e >> 6, il = e & 63;
            if (i0 + il >= Nr) continue;
            if constexpr (CPX)
                dp[t * dq + i0 + il] = float2{Ys[(2 * t) * YP + il], Ys[(2 * t + 1) * YP + il]};
            else
                dp[t * dq + i0 + il] = *reinterpret_cast<const float2*>(Ys + t * YP + 2 * il);
        }
        __syncthreads();
    }
}

// The complex64 azimuthal DFT for 64 < 2 N_phi <= 128 on the matrix cores: the
// real form of axis_mfma<NR, true> with NR = 5..8 row blocks, whose matrix does
// not fit in registers: it is staged once per workgroup in LDS (As[row][k],
// pitch Q16 + 4 like Xt, so the 16-byte fragment reads of 16 lanes cover all
// banks once), with the results in a third LDS buffer (Ys, pitch 68).  Dynamic
// LDS: (64 + Q16) (Q16 + 4) + 68 Q16 floats.
__host__ __device__ constexpr size_t axis_big_lds_bytes(int NR) {
    return sizeof(float) * ((size_t)(64 + 16 * NR) * (16 * NR + 4) + (size_t)68 * 16 * NR);
}

template <int NR>
__global__ void __launch_bounds__(256) axis_mfma_big(const float* __restrict__ mat16,
                                                     const float2* __restrict__ src, int64_t so, int64_t sq,
                                                     float2* __restrict__ dst, int64_t dout, int64_t dq, int Q,
                                                     int Nr) {
    constexpr int Q16 = 16 * NR, XS = Q16 + 4, YP = 68;
    extern __shared__ __align__(16) unsigned char lds_big[];
    float* Xt = reinterpret_cast<float*>(lds_big);   // Xt[point][k], 64 x XS
    float* As = Xt + 64 * XS;                         // As[row][k], Q16 x XS
    float* Ys = As + Q16 * XS;                        // Ys[row][point], Q16 x YP
    const int o = blockIdx.y;
    const int nblk = (Nr + 63) / 64;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float2* sp = src + o * so;
    float2* dp = dst + o * dout;
    for (int e = threadIdx.x; e < Q16 * Q16 / 4; e += 256) {
        const int r = e / (Q16 / 4), k4 = e - r * (Q16 / 4);
        *reinterpret_cast<f4v*>(As + r * XS + 4 * k4) = *reinterpret_cast<const f4v*>(mat16 + r * Q16 + 4 * k4);
    }
    // staging item (g, il) = threadIdx.x + 256 u: input rows 2 g, 2 g + 1 of point
    // il; loads from clamped addresses with no branch, zeroed when staged
    float2 pf[NR][2];
    auto fetch = [&](int bx) {
        const int ic = min(bx * 64 + (threadIdx.x & 63), Nr - 1);
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int g = (threadIdx.x + 256 * u) >> 6;
#pragma unroll
            for (int c = 0; c < 2; ++c) pf[u][c] = sp[min(2 * g + c, Q - 1) * sq + ic];
        }
    };
    int bx = blockIdx.x;
    fetch(bx);
    for (; bx < nblk; bx += gridDim.x) {
        const bool live = bx * 64 + (threadIdx.x & 63) < Nr;
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int e = threadIdx.x + 256 * u, il = e & 63, g = e >> 6;
            const float2 v0 = (live && 2 * g < Q) ? pf[u][0] : float2{0.f, 0.f};
            const float2 v1 = (live && 2 * g + 1 < Q) ? pf[u][1] : float2{0.f, 0.f};
            *reinterpret_cast<f4v*>(Xt + il * XS + 4 * g) = f4v{v0.x, v0.y, v1.x, v1.y};
        }
        __syncthreads();
        fetch(bx + gridDim.x);
        f4v acc[NR];
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) acc[rb] = f4v{0.f, 0.f, 0.f, 0.f};
        const int kl = 4 * (lane >> 4);
#pragma unroll
        for (int G = 0; G < NR; ++G) {
            const f4v b = *reinterpret_cast<const f4v*>(Xt + (16 * w + (lane & 15)) * XS + 16 * G + kl);
            f4v a[NR];
#pragma unroll
            for (int rb = 0; rb < NR; ++rb)
                a[rb] = *reinterpret_cast<const f4v*>(As + (16 * rb + (lane & 15)) * XS + 16 * G + kl);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int rb = 0; rb < NR; ++rb)
                    acc[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rb][s], b[s], acc[rb], 0, 0, 0);
        }
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < NR; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                Ys[(16 * rb + 4 * (lane >> 4) + v) * YP + 16 * w + (lane & 15)] = acc[rb][v];
        __syncthreads();
        const int i0 = bx * 64;
        for (int e = threadIdx.x; e < Q * 64; e += 256) {
            const int t = e >> 6, il = e & 63;
            if (i0 + il < Nr) dp[t * dq + i0 + il] = float2{Ys[(2 * t) * YP + il], Ys[(2 * t + 1) * YP + il]};
        }
        __syncthreads();
    }
}

// The axis steps for complex128 data on the FP64 matrix cores, in the forms of
// axis_mfma: the real per-m Legendre block on 32 radial points per block (64
// real columns 2 i + part), or the azimuthal DFT in its real form
// [[Re, -Im], [Im, Re]] (contraction index 2 q + part) on 64 points per block;
// either way 64 columns, wave w taking columns 16 w .. 16 w + 15.
// v_mfma_f64_16x16x4_f64 takes the operands of the FP32 form (lane l:
// A[l%16][l/16], B[l/16][l%16]) and returns row 4 v + l/16, column l%16 in
// result register v.  The contraction index is split as k = 16 G + 4 (l/16) + s,
// so that each lane holds the four k of its four instructions in 32 contiguous
// bytes of the matrix (registers, loaded once) and of the transposed LDS copy
// Xt[column][k] (pitch Q16 + 2).  Workgroups loop over point blocks of one
// outer index with the next block's loads issued, from clamped addresses with
// no branch, before the current one is multiplied.
typedef double d4v __attribute__((ext_vector_type(4)));

template <int NR, bool CPX>
__global__ void __launch_bounds__(256) axis_mfma64(const double* __restrict__ mat16, int64_t mso,
                                                   const double2* __restrict__ src, int64_t so, int64_t sq,
                                                   double2* __restrict__ dst, int64_t dout, int64_t dq, int Q,
                                                   int Nr) {
    constexpr int Q16 = 16 * NR, XS = Q16 + 2, NCOL = 64, YP = NCOL + 2, PB = CPX ? 64 : 32;
    constexpr int NIT = 2 * NR;   // staging items per thread: (input row, point)
    static_assert(Q16 * YP <= NCOL * XS, "result staging must fit in the input buffer");
    __shared__ __align__(16) double Xt[NCOL * XS];
    const int o = blockIdx.y;
    const int nblk = (Nr + PB - 1) / PB;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double2* sp = src + o * so;
    double2* dp = dst + o * dout;
    d4v a[NR][NR];   // [G][rb]: A[16 rb + l%16][16 G + 4 (l/16) + s]
    {
        const double* Am = mat16 + o * mso + (lane & 15) * Q16 + 4 * (lane >> 4);
#pragma unroll
        for (int G = 0; G < NR; ++G)
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) {
                const double2 lo = *reinterpret_cast<const double2*>(Am + 16 * rb * Q16 + 16 * G);
                const double2 hi = *reinterpret_cast<const double2*>(Am + 16 * rb * Q16 + 16 * G + 2);
                a[G][rb] = d4v{lo.x, lo.y, hi.x, hi.y};
            }
        // have them in registers here: a first use inside the block loop would
        // put a wait on every memory operation in flight into each iteration
#pragma unroll
        for (int G = 0; G < NR; ++G)
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) {
                // two 16-byte halves: a 32-byte operand here drops the kernel's host stub
                const d4v t = a[G][rb];
                asm volatile("" ::"v"(t.lo), "v"(t.hi));
            }
    }
    double2 pf[NIT];   // item e = threadIdx.x + 256 u: input row e / PB, point e % PB
    auto fetch = [&](int bx) {
#pragma unroll
        for (int u = 0; u < NIT; ++u) {
            const int e = threadIdx.x + 256 * u;
            pf[u] = sp[min(e / PB, Q - 1) * sq + min(bx * PB + e % PB, Nr - 1)];
        }
    };
    int bx = blockIdx.x;
    fetch(bx);
    for (; bx < nblk; bx += gridDim.x) {
        const int i0 = bx * PB;
#pragma unroll
        for (int u = 0; u < NIT; ++u) {
            const int e = threadIdx.x + 256 * u, q = e / PB, il = e % PB;
            const double2 v = (q < Q && i0 + il < Nr) ? pf[u] : double2{0.0, 0.0};
            if constexpr (CPX) {
                *reinterpret_cast<double2*>(Xt + il * XS + 2 * q) = v;
            } else {
                Xt[(2 * il) * XS + q] = v.x;
                Xt[(2 * il + 1) * XS + q] = v.y;
            }
        }
        __syncthreads();
        fetch(bx + gridDim.x);
        d4v acc[NR];
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) acc[rb] = d4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int G = 0; G < NR; ++G) {
            const double* xb = Xt + (16 * w + (lane & 15)) * XS + 16 * G + 4 * (lane >> 4);
            const double2 lo = *reinterpret_cast<const double2*>(xb);
            const double2 hi = *reinterpret_cast<const double2*>(xb + 2);
            const double b[4] = {lo.x, lo.y, hi.x, hi.y};
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int rb = 0; rb < NR; ++rb)
                    acc[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[G][rb][s], b[s], acc[rb], 0, 0, 0);
        }
        __syncthreads();
        double* Ys = Xt;   // Ys[row][column], pitch YP
#pragma unroll
        for (int rb = 0; rb < NR; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v) Ys[(16 * rb + 4 * v + (lane >> 4)) * YP + 16 * w + (lane & 15)] = acc[rb][v];
        __syncthreads();
        for (int e = threadIdx.x; e < Q * PB; e += 256) {
            const int t = e / PB, il = e % PB;
            if (i0 + il >= Nr) continue;
            if constexpr (CPX)
                dp[t * dq + i0 + il] = double2{Ys[(2 * t) * YP + il], Ys[(2 * t + 1) * YP + il]};
            else
                dp[t * dq + i0 + il] = double2{Ys[t * YP + 2 * il], Ys[t * YP + 2 * il + 1]};
        }
        __syncthreads();
    }
}

// Both axis steps of the complex64 transform in one launch: a workgroup takes 16
// radial points and keeps all of their N_theta x N_phi values in LDS between the
// steps, so the grid is read once and written once (64 x 17 x 4096: 71 MB per
// direction instead of 142), and both steps use their symmetries:
//  * DFT: with e_k = x_k + x_-k and o_k = x_k - x_-k the orders m and -m are
//    E_m -+ i O_m, E = C e, O = S o, with the real (M + 1) x (M + 1) matrices
//    C = cos(2 pi m k / N_phi) / sqrt(N_phi) and S = sin(...) / sqrt(N_phi); the
//    inverse has the same form with k and m exchanged and +- i;
//  * Legendre: nodes and weights are symmetric, P_t has the parity of t, so the
//    even t act on z_j + z_-j and the odd t on z_j - z_-j (N_theta/2 nodes).
// That leaves a quarter of the matrix instructions of the padded real forms of
// axis_mfma.  v_mfma_f32_16x16x4_f32: the 16 columns are the points, re and im
// separate products; instruction v of a 16-block takes the contraction indices
// 4 v + l/16, the tables hold the lane's four values contiguously.  Waves take DFT
// tasks by eta_j, and Legendre tasks by (m, parity of t) forward, by (m, block of
// eta_j) inverse; the first step reads memory, the second writes it.
// Element pairs are always added: the table entries of a self-paired element
// (k = 0, the middle node) carry the factor 1/2.  The sum of two finite values must
// not overflow where the result does not, so values are halved before it by powers of
// two that cancel: forward the loads by 1/4, the DFT tables carry 2 and the Legendre
// tables 2; inverse the Legendre tables carry 1/2 and the DFT tables 2.  Contraction indices past the end
// are clamped and meet zero table entries; result rows past the end are copies of
// the last row and are written onto it (LDS) or masked (memory).
// 64 x 17 x 4096 (256 workgroups): forward 19.3 us, inverse 22.7 (two launches:
// 48 each); the 71 MB alone take 14 at the rate of a large copy.  A workgroup by
// itself takes 9 to 10 us, of which 6.2 are matrix instructions, so the loads of a
// wave's next tasks are issued together and addresses are lane offset + wave offset
// of a buffer (with 64-bit lane addresses a workgroup took 15 us).
constexpr int kShtPts = 16, kShtWaves = 16;

typedef unsigned int u2v __attribute__((ext_vector_type(2)));
static __device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const float2* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(p), 0, bytes, 0x00020000);
}
// lane offset + wave offset: no address arithmetic in vector registers
static __device__ __forceinline__ float2 get(__amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t wave) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, lane, wave, 0));
}
static __device__ __forceinline__ void put(float2 v, __amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t wave) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2v, v), r, lane, wave, 0);
}

template <bool INV, int HB, int KS>
__global__ void __launch_bounds__(64 * kShtWaves) sht_both(const float* __restrict__ leg, const float* __restrict__ dft,
                                                           const float2* src, float2* dst, int nt, int nphi, int Nr) {
    extern __shared__ __align__(16) unsigned char lds_sht[];   // between the steps: float2 at ((j N_phi + q) 16 + point)
    const int lane = threadIdx.x & 63, c = lane & 15, q4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = blockIdx.x * kShtPts, M = (nphi - 1) / 2, H = (nt + 1) / 2;
    const bool live = i0 + c < Nr;
    const uint32_t rb = 8u * Nr, lrow = 8u * kShtPts;             // bytes of a row in memory, in LDS
    const uint32_t gin = 8u * min(i0 + c, Nr - 1), gout = 8u * (i0 + c), lc = 8u * c;
    constexpr int MB = (KS + 3) / 4, kAz = MB == 1 ? 2 : 1;       // kAz, kLg: tasks whose loads are issued together
    constexpr int kLg = 2;
    const __amdgpu_buffer_rsrc_t in = buffer(src, rb * nt * nphi), out = buffer(dst, rb * nt * nphi);

    // DFT task of node j: element pairs +-k -> +-m; up / un the lane's offsets of
    // +k / -k, rp / rn those of its results +m / -m
    f4v C[MB][MB], S[MB][MB];
    uint32_t up[MB][4], un[MB][4], rp[MB][4], rn[MB][4];
    auto dft_setup = [&]() {
        const f4v* Cs = reinterpret_cast<const f4v*>(dft) + lane;
#pragma unroll
        for (int a = 0; a < MB; ++a) {
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                C[a][b] = Cs[64 * (a * MB + b)];
                S[a][b] = Cs[64 * (MB * MB + a * MB + b)];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = min(16 * a + 4 * v + q4, M), m = min(16 * a + 4 * q4 + v, M);
                const int nk = k ? nphi - k : 0, nm = m ? nphi - m : 0;
                up[a][v] = INV ? (M + k) * lrow + lc : k * rb + gin;
                un[a][v] = INV ? (M - k) * lrow + lc : nk * rb + gin;
                rp[a][v] = INV ? nm * rb + gout : (M + m) * lrow + lc;    // E - i O
                rn[a][v] = INV ? m * rb + gout : (M - m) * lrow + lc;     // E + i O
            }
        }
    };
    auto dft_load = [&](int j, float2 (&x)[MB][4], float2 (&y)[MB][4]) {
        const unsigned char* lb = lds_sht + j * nphi * lrow;
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int v = 0; v < 4 && 4 * b + v < KS; ++v) {
                x[b][v] = INV ? *reinterpret_cast<const float2*>(lb + up[b][v]) : get(in, up[b][v], j * nphi * rb);
                y[b][v] = INV ? *reinterpret_cast<const float2*>(lb + un[b][v]) : get(in, un[b][v], j * nphi * rb);
            }
    };
    auto dft_task = [&](int j, const float2 (&x)[MB][4], const float2 (&y)[MB][4]) {
        f4v E[MB][2], O[MB][2];
#pragma unroll
        for (int a = 0; a < MB; ++a) E[a][0] = E[a][1] = O[a][0] = O[a][1] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int v = 0; v < 4 && 4 * b + v < KS; ++v) {
                const float h = INV ? 1.f : 0.25f;   // (the products by h are exact)
                const float2 p = float2{h * x[b][v].x, h * x[b][v].y}, n = y[b][v];
                const float er = fmaf(h, n.x, p.x), ei = fmaf(h, n.y, p.y);
                const float dr = fmaf(-h, n.x, p.x), di = fmaf(-h, n.y, p.y);
#pragma unroll
                for (int a = 0; a < MB; ++a) {
                    E[a][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(C[a][b][v], er, E[a][0], 0, 0, 0);
                    E[a][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(C[a][b][v], ei, E[a][1], 0, 0, 0);
                    O[a][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(S[a][b][v], dr, O[a][0], 0, 0, 0);
                    O[a][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(S[a][b][v], di, O[a][1], 0, 0, 0);
                }
            }
        unsigned char* lb = lds_sht + j * nphi * lrow;
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float re = E[a][0][v], im = E[a][1][v], orr = O[a][0][v], oi = O[a][1][v];
                const float2 lo = float2{re + oi, im - orr}, hi = float2{re - oi, im + orr};
                if constexpr (INV) {
                    if (live && 16 * a + 4 * q4 + v <= M) {
                        put(lo, out, rp[a][v], j * nphi * rb);
                        put(hi, out, rn[a][v], j * nphi * rb);
                    }
                } else {
                    *reinterpret_cast<float2*>(lb + rp[a][v]) = lo;
                    *reinterpret_cast<float2*>(lb + rn[a][v]) = hi;
                }
            }
    };
    const f4v* lt = reinterpret_cast<const f4v*>(leg) + lane;

    if constexpr (!INV) {
        dft_setup();
        for (int j0 = w; j0 < nt; j0 += kAz * kShtWaves) {
            float2 x[kAz][MB][4], y[kAz][MB][4];
#pragma unroll
            for (int u = 0; u < kAz; ++u) dft_load(min(j0 + u * kShtWaves, nt - 1), x[u], y[u]);
#pragma unroll
            for (int u = 0; u < kAz; ++u)
                if (j0 + u * kShtWaves < nt) dft_task(j0 + u * kShtWaves, x[u], y[u]);
        }
        uint32_t uj[HB][4], um[HB][4], ot[HB][4];
#pragma unroll
        for (int b = 0; b < HB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int j = min(16 * b + 4 * v + q4, H - 1);
                uj[b][v] = j * nphi * lrow + lc;
                um[b][v] = (nt - 1 - j) * nphi * lrow + lc;
                ot[b][v] = 2 * (16 * b + 4 * q4 + v) * rb + gout;
            }
        __syncthreads();
        for (int task = w; task < 2 * nphi; task += kShtWaves) {
            const int q = task >> 1, part = task & 1;
            const float sg = part ? -1.f : 1.f;
            const f4v* A = lt + 64 * (HB * HB) * task;
            f4v t[HB][HB];
#pragma unroll
            for (int i = 0; i < HB * HB; ++i) t[i / HB][i % HB] = A[64 * i];
            const unsigned char* lb = lds_sht + q * lrow;
            f4v acc[HB][2];
#pragma unroll
            for (int a = 0; a < HB; ++a) acc[a][0] = acc[a][1] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < HB; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float2 x = *reinterpret_cast<const float2*>(lb + uj[b][v]);
                    const float2 y = *reinterpret_cast<const float2*>(lb + um[b][v]);
                    const float zr = fmaf(y.x, sg, x.x), zi = fmaf(y.y, sg, x.y);
#pragma unroll
                    for (int a = 0; a < HB; ++a) {
                        acc[a][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[a][b][v], zr, acc[a][0], 0, 0, 0);
                        acc[a][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[a][b][v], zi, acc[a][1], 0, 0, 0);
                    }
                }
#pragma unroll
            for (int a = 0; a < HB; ++a)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (live && 2 * (16 * a + 4 * q4 + v) + part < nt)
                        put(float2{acc[a][0][v], acc[a][1][v]}, out, ot[a][v], (q * nt + part) * rb);
        }
    } else {
        uint32_t ut[2][HB][4];
#pragma unroll
        for (int i = 0; i < 8 * HB; ++i)
            ut[i / (4 * HB)][i / 4 % HB][i % 4] =
                min(2 * (16 * (i / 4 % HB) + 4 * (i % 4) + q4) + i / (4 * HB), nt - 1) * rb + gin;
        for (int t0 = w; t0 < HB * nphi; t0 += kLg * kShtWaves) {
            float2 x[kLg][2][HB][4];
#pragma unroll
            for (int u = 0; u < kLg; ++u) {
                const uint32_t base = min(t0 + u * kShtWaves, HB * nphi - 1) / HB * nt * rb;
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int b = 0; b < HB; ++b)
#pragma unroll
                        for (int v = 0; v < 4; ++v) x[u][e][b][v] = get(in, ut[e][b][v], base);
            }
#pragma unroll
            for (int u = 0; u < kLg; ++u) {
                const int task = t0 + u * kShtWaves, q = task / HB, a = task % HB;
                if (task >= HB * nphi) continue;
                const f4v* A = lt + 64 * (2 * HB) * task;
                f4v acc[2][2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    acc[e][0] = acc[e][1] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int b = 0; b < HB; ++b) {
                        const f4v t = A[64 * (e * HB + b)];
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            acc[e][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[v], x[u][e][b][v].x, acc[e][0], 0, 0, 0);
                            acc[e][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[v], x[u][e][b][v].y, acc[e][1], 0, 0, 0);
                        }
                    }
                }
                unsigned char* lb = lds_sht + q * lrow + lc;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int j = min(16 * a + 4 * q4 + v, H - 1);
                    *reinterpret_cast<float2*>(lb + __umul24(j, nphi * lrow)) =
                        float2{acc[0][0][v] + acc[1][0][v], acc[0][1][v] + acc[1][1][v]};
                    *reinterpret_cast<float2*>(lb + __umul24(nt - 1 - j, nphi * lrow)) =
                        float2{acc[0][0][v] - acc[1][0][v], acc[0][1][v] - acc[1][1][v]};
                }
            }
        }
        dft_setup();
        __syncthreads();
        for (int j = w; j < nt; j += kShtWaves) {
            float2 x[MB][4], y[MB][4];
            dft_load(j, x, y);
            dft_task(j, x, y);
        }
    }
}

// x[i] *= exp(-i (V0[i] + F V1[i]) dt/2), the angle formed and reduced mod 2 pi
// in FP64 (V0 or V1 may be null: zero)
template <typename S>
__global__ void __launch_bounds__(256) grid_phase(typename Cx<S>::t* __restrict__ x, const double* __restrict__ V0,
                                                  const double* __restrict__ V1, double F, double half_dt,
                                                  int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double a = ((V0 ? V0[i] : 0.0) + (V1 ? F * V1[i] : 0.0)) * half_dt;
    const double twopi = 6.283185307179586476925286766559;
    a -= twopi * rint(a / twopi);
    S sn, cs;
    if constexpr (sizeof(S) == sizeof(float)) {
        sincosf((float)a, &sn, &cs);
    } else {
        sincos(a, &sn, &cs);
    }
    const typename Cx<S>::t z = x[i];
    x[i] = {z.x * cs + z.y * sn, z.y * cs - z.x * sn};
}

// Channel (q, t), l = |q - M| + t, of Nr slots: forward, out[u] = i^-l in[j(u)]
// with j(u) = (u + 1) mod Nr for odd l (the n = 0 slot moves to the top of the
// unified grid n = 1..Nr) and j(u) = u for even l; inverse, out[j] = i^l in[u(j)].
template <typename S>
__global__ void __launch_bounds__(256) momentum_order(const typename Cx<S>::t* __restrict__ src,
                                                      typename Cx<S>::t* __restrict__ dst, int nt, int M, int Nr,
                                                      int inverse) {
    const int c = blockIdx.y;
    const int x = blockIdx.x * 256 + threadIdx.x;
    if (x >= Nr) return;
    const int q = c / nt, t = c - q * nt;
    const int l = (q > M ? q - M : M - q) + t;
    int from = x;
    if (l & 1) from = inverse ? (x + Nr - 1) % Nr : (x + 1) % Nr;
    const typename Cx<S>::t z = src[(int64_t)c * Nr + from];
    // multiply by i^e, e = -l (forward) or l (inverse), e mod 4
    const int e = ((inverse ? l : -l) % 4 + 4) % 4;
    typename Cx<S>::t w;
    if (e == 0) w = z;
    else if (e == 1) w = {-z.y, z.x};
    else if (e == 2) w = {-z.x, -z.y};
    else w = {z.y, -z.x};
    dst[(int64_t)c * Nr + x] = w;
}

}  // namespace

template <typename S>
hipError_t launch_momentum_order(const void* src, void* dst, int nt, int nphi, int Nr, bool inverse, hipStream_t s) {
    hipLaunchKernelGGL(momentum_order<S>, dim3((unsigned)((Nr + 255) / 256), (unsigned)(nt * nphi)), dim3(256), 0, s,
                       (const typename Cx<S>::t*)src, (typename Cx<S>::t*)dst, nt, (nphi - 1) / 2, Nr,
                       inverse ? 1 : 0);
    return hipGetLastError();
}
template hipError_t launch_momentum_order<float>(const void*, void*, int, int, int, bool, hipStream_t);
template hipError_t launch_momentum_order<double>(const void*, void*, int, int, int, bool, hipStream_t);

template <typename S>
hipError_t launch_grid_phase(void* x, const double* V0, const double* V1, double F, double dt, int64_t n,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(grid_phase<S>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       (typename Cx<S>::t*)x, V0, V1, F, 0.5 * dt, n);
    return hipGetLastError();
}
template hipError_t launch_grid_phase<float>(void*, const double*, const double*, double, double, int64_t,
                                             hipStream_t);
template hipError_t launch_grid_phase<double>(void*, const double*, const double*, double, double, int64_t,
                                              hipStream_t);

template <typename S, bool CA>
hipError_t launch_axis_apply(const S* mat, int64_t mso, bool tr, bool cj, const void* src, int64_t so, int64_t sq,
                             void* dst, int64_t dout, int64_t dq, int Q, int nouter, int Nr, hipStream_t s) {
    using V = typename Cx<S>::t;
    if (Q < 1 || Q > kShtMaxQ || nouter < 1 || Nr < 1) return hipErrorInvalidValue;
    const size_t lds = axis_lds_bytes<S, CA>(Q);
    hipLaunchKernelGGL((axis_apply<S, CA>), dim3((Nr + 63) / 64, nouter), dim3(256), lds, s, mat, mso, tr ? 1 : 0,
                       cj ? 1 : 0, (const V*)src, so, sq, (V*)dst, dout, dq, Q, Nr);
    return hipGetLastError();
}

// Workgroups of axis_mfma<nr, CPX> resident on the device at once, queried on
// the first call (set_lds_limits_axis makes that call before any launch, so
// that no query falls inside a stream capture); -1 if the query fails.
template <bool CPX>
static int axis_mfma_fit(int nr) {
    static std::atomic<int> fit[4] = {{0}, {0}, {0}, {0}};
    if (nr < 1 || nr > 4) return -1;
    int f = fit[nr - 1].load(std::memory_order_relaxed);
    if (f > 0) return f;
    const void* k = nr == 1   ? (const void*)axis_mfma<1, CPX>
                    : nr == 2 ? (const void*)axis_mfma<2, CPX>
                    : nr == 3 ? (const void*)axis_mfma<3, CPX>
                              : (const void*)axis_mfma<4, CPX>;
    int dev = 0, ncu = 0, occ = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, 256, 0) != hipSuccess)
        return -1;
    f = std::max(1, occ) * std::max(1, ncu);
    fit[nr - 1].store(f, std::memory_order_relaxed);
    return f;
}

// Workgroups of axis_mfma_big<nr> (nr = 5..8) resident on the device at once,
// with its dynamic LDS (queried once, first from set_lds_limits_axis); -1 if
// the query fails.
static int axis_big_fit(int nr) {
    static std::atomic<int> fit[4] = {{0}, {0}, {0}, {0}};
    if (nr < 5 || nr > 8) return -1;
    int f = fit[nr - 5].load(std::memory_order_relaxed);
    if (f > 0) return f;
    const void* k = nr == 5   ? (const void*)axis_mfma_big<5>
                    : nr == 6 ? (const void*)axis_mfma_big<6>
                    : nr == 7 ? (const void*)axis_mfma_big<7>
                              : (const void*)axis_mfma_big<8>;
    int dev = 0, ncu = 0, occ = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, 256, axis_big_lds_bytes(nr)) != hipSuccess)
        return -1;
    f = std::max(1, occ) * std::max(1, ncu);
    fit[nr - 5].store(f, std::memory_order_relaxed);
    return f;
}

template <bool CPX>
static hipError_t launch_axis_mfma_t(const float* mat16, int64_t mso, const void* src, int64_t so, int64_t sq,
                                     void* dst, int64_t dout, int64_t dq, int Q, int nouter, int Nr, hipStream_t s) {
    const int nr = ((CPX ? 2 * Q : Q) + 15) / 16;
    if (Q < 1 || nr > (CPX ? 8 : 4) || nouter < 1 || Nr < 1) return hipErrorInvalidValue;
    if (CPX && nr > 4 && mso != 0) return hipErrorInvalidValue;   // the large form takes one shared matrix
    const int fit0 = nr > 4 ? axis_big_fit(nr) : axis_mfma_fit<CPX>(nr);
    if (fit0 < 0) return hipErrorInvalidValue;
    const int nblk = (Nr + 63) / 64;
    // as many workgroups as fit on the device at once (at least one per outer
    // index), each taking an equal share of the point blocks of its outer index
    const int fit = std::max(1, std::min(nblk, fit0 / nouter));
    const int per = (nblk + fit - 1) / fit;
    const dim3 grid((unsigned)((nblk + per - 1) / per), (unsigned)nouter);
    const float2* x = static_cast<const float2*>(src);
    float2* y = static_cast<float2*>(dst);
    if (nr > 4) {
        const size_t lds = axis_big_lds_bytes(nr);
        switch (nr) {
            case 5: hipLaunchKernelGGL(axis_mfma_big<5>, grid, dim3(256), lds, s, mat16, x, so, sq, y, dout, dq, Q, Nr); break;
            case 6: hipLaunchKernelGGL(axis_mfma_big<6>, grid, dim3(256), lds, s, mat16, x, so, sq, y, dout, dq, Q, Nr); break;
            case 7: hipLaunchKernelGGL(axis_mfma_big<7>, grid, dim3(256), lds, s, mat16, x, so, sq, y, dout, dq, Q, Nr); break;
            default: hipLaunchKernelGGL(axis_mfma_big<8>, grid, dim3(256), lds, s, mat16, x, so, sq, y, dout, dq, Q, Nr); break;
        }
        return hipGetLastError();
    }
    switch (nr) {
        case 1: hipLaunchKernelGGL((axis_mfma<1, CPX>), grid, dim3(256), 0, s, mat16, mso, x, so, sq, y, dout, dq, Q, Nr); break;
        case 2: hipLaunchKernelGGL((axis_mfma<2, CPX>), grid, dim3(256), 0, s, mat16, mso, x, so, sq, y, dout, dq, Q, Nr); break;
        case 3: hipLaunchKernelGGL((axis_mfma<3, CPX>), grid, dim3(256), 0, s, mat16, mso, x, so, sq, y, dout, dq, Q, Nr); break;
        default: hipLaunchKernelGGL((axis_mfma<4, CPX>), grid, dim3(256), 0, s, mat16, mso, x, so, sq, y, dout, dq, Q, Nr); break;
    }
    return hipGetLastError();
}

// Workgroups of axis_mfma64<nr, CPX> resident on the device at once (queried
// once, first from set_lds_limits_axis); -1 if the query fails.
template <bool CPX>
static int axis_mfma64_fit(int nr) {
    static std::atomic<int> fit[4] = {{0}, {0}, {0}, {0}};
    if (nr < 1 || nr > 4) return -1;
    int f = fit[nr - 1].load(std::memory_order_relaxed);
    if (f > 0) return f;
    const void* k = nr == 1   ? (const void*)axis_mfma64<1, CPX>
                    : nr == 2 ? (const void*)axis_mfma64<2, CPX>
                    : nr == 3 ? (const void*)axis_mfma64<3, CPX>
                              : (const void*)axis_mfma64<4, CPX>;
    int dev = 0, ncu = 0, occ = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, 256, 0) != hipSuccess)
        return -1;
    f = std::max(1, occ) * std::max(1, ncu);
    fit[nr - 1].store(f, std::memory_order_relaxed);
    return f;
}

template <bool CPX>
static hipError_t launch_axis_mfma64_t(const double* mat16, int64_t mso, const void* src, int64_t so, int64_t sq,
                                       void* dst, int64_t dout, int64_t dq, int Q, int nouter, int Nr,
                                       hipStream_t s) {
    const int nr = ((CPX ? 2 * Q : Q) + 15) / 16;
    if (Q < 1 || nr > 4 || nouter < 1 || Nr < 1) return hipErrorInvalidValue;
    const int fit0 = axis_mfma64_fit<CPX>(nr);
    if (fit0 < 0) return hipErrorInvalidValue;
    const int pb = CPX ? 64 : 32;
    const int nblk = (Nr + pb - 1) / pb;
    const int fit = std::max(1, std::min(nblk, fit0 / nouter));
    const int per = (nblk + fit - 1) / fit;
    const dim3 grid((unsigned)((nblk + per - 1) / per), (unsigned)nouter);
    const double2* x = static_cast<const double2*>(src);
    double2* y = static_cast<double2*>(dst);
    switch (nr) {
        case 1: hipLaunchKernelGGL((axis_mfma64<1, CPX>), grid, dim3(256), 0, s, mat16, mso, x, so, sq, y, dout, dq, Q, Nr); break;
        case 2: hipLaunchKernelGGL((axis_mfma64<2, CPX>), grid, dim3(256), 0, s, mat16, mso, x, so, sq, y, dout, dq, Q, Nr); break;
        case 3: hipLaunchKernelGGL((axis_mfma64<3, CPX>), grid, dim3(256), 0, s, mat16, mso, x, so, sq, y, dout, dq, Q, Nr); break;
        default: hipLaunchKernelGGL((axis_mfma64<4, CPX>), grid, dim3(256), 0, s, mat16, mso, x, so, sq, y, dout, dq, Q, Nr); break;
    }
    return hipGetLastError();
}

hipError_t launch_axis_mfma64(bool complex_matrix, const double* mat16, int64_t mso, const void* src, int64_t so,
                              int64_t sq, void* dst, int64_t dout, int64_t dq, int Q, int nouter, int Nr,
                              hipStream_t s) {
    return complex_matrix ? launch_axis_mfma64_t<true>(mat16, mso, src, so, sq, dst, dout, dq, Q, nouter, Nr, s)
                          : launch_axis_mfma64_t<false>(mat16, mso, src, so, sq, dst, dout, dq, Q, nouter, Nr, s);
}

hipError_t launch_axis_mfma(bool complex_matrix, const float* mat16, int64_t mso, const void* src, int64_t so,
                            int64_t sq, void* dst, int64_t dout, int64_t dq, int Q, int nouter, int Nr,
                            hipStream_t s) {
    return complex_matrix ? launch_axis_mfma_t<true>(mat16, mso, src, so, sq, dst, dout, dq, Q, nouter, Nr, s)
                          : launch_axis_mfma_t<false>(mat16, mso, src, so, sq, dst, dout, dq, Q, nouter, Nr, s);
}

// LDS bytes of sht_both
static size_t sht_both_lds(int nt, int nphi) { return sizeof(float2) * kShtPts * (size_t)nt * nphi; }

bool sht_both_fits(int nt, int nphi, int Nr) {
    return sht_both_lds(nt, nphi) <= 160 * 1024 && nt <= 64 && nphi <= 63 && Nr >= 1 &&
           8.0 * nt * nphi * Nr < 4294967296.0;   // 32-bit lane offsets
}

// One direction's tables: forward blocks [q][parity of t][row block][block],
// rows t/2, columns j; inverse blocks [q][row block][parity][block], rows j,
// columns t/2; per block the lane's four values A[l%16][4 v + l/16].
static void sht_blocks(const std::vector<double>& P, int nt, int nphi, bool inverse, std::vector<double>& out) {
    const int H = (nt + 1) / 2, HB = (H + 15) / 16;
    out.assign((size_t)nphi * 2 * HB * HB * 256, 0.0);
    for (int q = 0; q < nphi; ++q)
        for (int e = 0; e < 2; ++e)
            for (int a = 0; a < HB; ++a)
                for (int b = 0; b < HB; ++b) {
                    const int blk = inverse ? (a * 2 + e) * HB + b : (e * HB + a) * HB + b;
                    double* o = out.data() + ((size_t)q * 2 * HB * HB + blk) * 256;
                    for (int l = 0; l < 64; ++l)
                        for (int v = 0; v < 4; ++v) {
                            const int row = 16 * a + l % 16, col = 16 * b + 4 * v + l / 16;
                            const int t = 2 * (inverse ? col : row) + e, j = inverse ? std::min(row, H - 1) : col;
                            const bool middle = 2 * j == nt - 1;
                            if (t >= nt || j >= H || (e && middle)) continue;
                            const double* p = P.data() + ((size_t)q * nt + t) * nt;
                            // equal up to rounding and the sign (-1)^t; times 2 (forward) or 1/2
                            o[4 * l + v] = (inverse ? 0.25 : 1.0) * (p[j] + (e ? -p[nt - 1 - j] : p[nt - 1 - j]));
                            if (middle && !inverse) o[4 * l + v] *= 0.5;   // its sum is z + z
                        }
                }
}

void sht_both_tables(const std::vector<double>& P, int nt, int nphi, std::vector<double>& leg,
                     std::vector<double>& dft) {
    std::vector<double> inv;
    sht_blocks(P, nt, nphi, false, leg);
    sht_blocks(P, nt, nphi, true, inv);
    leg.insert(leg.end(), inv.begin(), inv.end());
    const int M = (nphi - 1) / 2, MB = M / 16 + 1;
    const double pi = 3.14159265358979323846, sc = 2.0 / std::sqrt((double)nphi);
    dft.assign((size_t)2 * MB * MB * 256, 0.0);
    for (int a = 0; a < MB; ++a)
        for (int b = 0; b < MB; ++b)
            for (int l = 0; l < 64; ++l)
                for (int v = 0; v < 4; ++v) {
                    const int m = std::min(16 * a + l % 16, M), k = 16 * b + 4 * v + l / 16;
                    if (k > M) continue;
                    const double ang = 2.0 * pi * (m * k % nphi) / nphi;   // m k mod N_phi, exact
                    dft[((size_t)a * MB + b) * 256 + 4 * l + v] = std::cos(ang) * sc * (k ? 1.0 : 0.5);
                    dft[((size_t)MB * MB + a * MB + b) * 256 + 4 * l + v] = std::sin(ang) * sc;
                }
}

// the kernel for H = ceil(N_theta / 2) node pairs and M + 1 element pairs
typedef void (*ShtKernel)(const float*, const float*, const float2*, float2*, int, int, int);
template <bool INV, int HB>
static ShtKernel sht_both_kernel(int pairs) {
    if (pairs <= 8) return sht_both<INV, HB, 2>;
    if (pairs <= 12) return sht_both<INV, HB, 3>;
    if (pairs <= 16) return sht_both<INV, HB, 4>;
    return pairs <= 24 ? sht_both<INV, HB, 6> : sht_both<INV, HB, 8>;
}
static ShtKernel sht_both_kernel(bool inverse, int hb, int pairs) {
    if (inverse) return hb == 1 ? sht_both_kernel<true, 1>(pairs) : sht_both_kernel<true, 2>(pairs);
    return hb == 1 ? sht_both_kernel<false, 1>(pairs) : sht_both_kernel<false, 2>(pairs);
}

hipError_t launch_sht_both(const float* leg, const float* dft, const void* src, void* dst, int nt, int nphi, int Nr,
                           bool inverse, hipStream_t s) {
    if (nt < 1 || nphi < 1 || nphi % 2 == 0 || !sht_both_fits(nt, nphi, Nr)) return hipErrorInvalidValue;
    const int hb = ((nt + 1) / 2 + 15) / 16;
    const float* lg = leg + (inverse ? (size_t)nphi * 2 * hb * hb * 256 : 0);
    const dim3 grid((unsigned)((Nr + kShtPts - 1) / kShtPts)), block(64 * kShtWaves);
    const size_t lds = sht_both_lds(nt, nphi);
    const float2* x = static_cast<const float2*>(src);
    float2* y = static_cast<float2*>(dst);
    hipLaunchKernelGGL(sht_both_kernel(inverse, hb, (nphi + 1) / 2), grid, block, lds, s, lg, dft, x, y, nt, nphi, Nr);
    return hipGetLastError();
}

hipError_t set_lds_limits_axis() {
    for (int i = 0; i < 20; ++i) {
        const int pairs[5] = {8, 12, 16, 24, 32};
        const void* k = reinterpret_cast<const void*>(sht_both_kernel(i >= 10, 1 + i / 5 % 2, pairs[i % 5]));
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    {
        const void* big[4] = {(const void*)axis_mfma_big<5>, (const void*)axis_mfma_big<6>,
                              (const void*)axis_mfma_big<7>, (const void*)axis_mfma_big<8>};
        for (int i = 0; i < 4; ++i) {
            const hipError_t e = hipFuncSetAttribute(big[i], hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)axis_big_lds_bytes(5 + i));
            if (e != hipSuccess) return e;
            if (axis_big_fit(5 + i) < 0) return hipErrorInvalidDeviceFunction;
        }
    }
    for (int nr = 1; nr <= 4; ++nr)
        if (axis_mfma_fit<true>(nr) < 0 || axis_mfma_fit<false>(nr) < 0 ||
            axis_mfma64_fit<true>(nr) < 0 || axis_mfma64_fit<false>(nr) < 0)
            return hipErrorInvalidDeviceFunction;
    hipError_t e = hipFuncSetAttribute((const void*)axis_apply<float, true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)axis_lds_bytes<float, true>(kShtMaxQ));
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)axis_apply<float, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)axis_lds_bytes<float, false>(kShtMaxQ));
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)axis_apply<double, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)axis_lds_bytes<double, true>(kShtMaxQ));
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)axis_apply<double, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)axis_lds_bytes<double, false>(kShtMaxQ));
    return e;
}

template hipError_t launch_axis_apply<float, true>(const float*, int64_t, bool, bool, const void*, int64_t, int64_t,
                                                   void*, int64_t, int64_t, int, int, int, hipStream_t);
template hipError_t launch_axis_apply<float, false>(const float*, int64_t, bool, bool, const void*, int64_t, int64_t,
                                                    void*, int64_t, int64_t, int, int, int, hipStream_t);
template hipError_t launch_axis_apply<double, true>(const double*, int64_t, bool, bool, const void*, int64_t, int64_t,
                                                    void*, int64_t, int64_t, int, int, int, hipStream_t);
template hipError_t launch_axis_apply<double, false>(const double*, int64_t, bool, bool, const void*, int64_t,
                                                     int64_t, void*, int64_t, int64_t, int, int, int, hipStream_t);

}  // namespace dsbt
