// Moment stage for tiles of B = 64 on the CDNA4 matrix cores: one workgroup of
// eight waves per item, an item being 8 NCB complex channels of one (l, N) in
// NCB = 1 or 2 column blocks of 16 matrix columns (8 channels times (re, im)).
// T: arithmetic and tables (float or double), D: data in memory.
//
// Per tile J the tiled moment form (Sec. 2.4-2.5) maps [x_J; mu_J] to
// [o_J; mu_J+1] with A' = M_J (forward) or M_J^T (inverse, tiles in reverse).
// Rows and columns come in blocks of 16: four of tile slots, KB = ceil(k/16) of
// moments.  The only serial dependence is mu_J+1 = Q x_J + D mu_J, so the waves
// take roles, one tile ("step") apart, with one LDS barrier per step:
//   two loading waves   half a tile each, brought into the operand form and put
//                       into LDS (the kinetic factors of a split step are
//                       applied here, inverse only); for KB > 2 also one row
//                       block of Q x each
//   one wave            q = Q x, row blocks 0 and 1
//   the chain wave      mu_J+1 = q + D mu_J, mu kept in registers
//   four result waves   one row block of o = W x + E mu each, stored to memory
//
// Lane layouts (lane l, quarter q = l/16, column l%16).  Every block of 16 rows
// of a vector is held as four values per lane: of the tile's slots rows 4 q .. 4 q
// + 3 (contiguous in memory), of the moments rows q, 4 + q, 8 + q, 12 + q.  One is
// the result layout of v_mfma_f32_16x16x4_f32 (row 4 q + v in register v), the other
// that of v_mfma_f64_16x16x4_f64 (row 4 v + q); the table's rows are permuted for
// the one that an instruction does not have; and as
// the contraction index may be permuted alike in both operands (instruction v
// takes register v of every lane), they are the operand layouts too: results need no
// rearrangement on the serial path.  (Moments: instruction v then takes the
// consecutive rows 4 v .. 4 v + 3, so that in the triangular D nothing but zeros is
// added after the diagonal term, or, in the inverse with the instructions from the
// last, little; each later term would round at the moment's size, in every tile.)  The tables hold for each tile its non-zero
// 16 x 16 blocks (the in-tile band and D are triangular), 4 values per lane, in
// the order of the roles: 19, 29, 40 or 52 blocks for KB = 1 .. 4.
//
// Why tiles of 64 and eight waves: the chain takes half the steps of tiles of
// 32 with no more blocks per slot, and two waves on each SIMD hide each other's
// LDS and memory latency; the matrix instructions (32 cycles, FP64 64; nothing
// else issues on the SIMD meanwhile, measured) are what a step costs.
//
// Prefetch: the blocks of tile t + SETS are loaded into the registers that tile
// t's matrix instructions have just read.  Every global read of a tile is at
// least two steps before its write, so the stage runs in place.
#include "mstage_chain.h"

#include <type_traits>

namespace dsbt {

namespace {

template <typename T> struct Vec;
template <> struct Vec<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    typedef float v2 __attribute__((ext_vector_type(2)));
    static __device__ v4 mfma(float a, float b, v4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};
template <> struct Vec<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    typedef double v2 __attribute__((ext_vector_type(2)));
    static __device__ v4 mfma(double a, double b, v4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
};

constexpr int kXRing = 4;   // tile data: written in step t, last read in step t + 2 (a power of two of slots)
constexpr int kRing = 2;    // q and moments: written in one step, read in the next

// The blocks of one tile.  Row block rb of the tile slots takes blocks
// [x_lo, x_hi) of the data (lower band forward, upper inverse) and all KB of the
// moments; row block rb of the moments all 4 of the data and [d_lo, d_hi) of the
// moments.  b_*: first block of a row block in the table: results, then Q, then D.
__host__ __device__ constexpr int x_lo(bool inv, int rb) { return inv ? rb : 0; }
__host__ __device__ constexpr int x_hi(bool inv, int rb) { return inv ? 4 : rb + 1; }
__host__ __device__ constexpr int d_lo(bool inv, int rb) { return inv ? rb : 0; }
__host__ __device__ constexpr int d_hi(bool inv, int kb, int rb) { return inv ? kb : rb + 1; }
// Column block (0..3 data, 4.. moments) of the i-th block of result row block rb, in
// the order of its products: data farthest from the diagonal first, then the moments,
// the diagonal block last.  The diagonal terms are the largest; added first, every
// later sum rounds at their size; and the sums over the data and over the moments are
// kept apart until the end.  The order costs nothing.  FP32 errors against 64 bits,
// diagonal first (inverse) or before the moments (forward), one sum / now (with the
// order of D's terms above): random data of N = 2048, l <= 62, forward 1.42e-7 / 1.31e-7,
// inverse 1.68e-7 / 1.36e-7 (tiles of 32: 1.41e-7, 1.57e-7); l = 64 to 127 1.85e-7 /
// 1.52e-7 and 2.09e-7 / 1.58e-7; Gaussian sums of N = 8192, l = 96 to 127, 2.82e-7 /
// 2.54e-7 and 3.44e-7 / 2.63e-7.
__host__ __device__ constexpr int out_col(bool inv, int kb, int rb, int i) {
    const int n = x_hi(inv, rb) - x_lo(inv, rb) - 1;
    return i < n ? (inv ? 3 - i : i) : i < n + kb ? 4 + i - n : rb;
}
__host__ __device__ constexpr int b_out(bool inv, int kb, int rb) {
    int b = 0;
    for (int r = 0; r < rb; ++r) b += x_hi(inv, r) - x_lo(inv, r) + kb;
    return b;
}
__host__ __device__ constexpr int b_q(bool inv, int kb, int rb) { return b_out(inv, kb, 4) + 4 * rb; }
__host__ __device__ constexpr int b_d(bool inv, int kb, int rb) {
    int b = b_q(inv, kb, kb);
    for (int r = 0; r < rb; ++r) b += d_hi(inv, kb, r) - d_lo(inv, r);
    return b;
}
// column block of the i-th block of moment row block rb: the diagonal block last
__host__ __device__ constexpr int d_col(bool inv, int kb, int i) { return inv ? kb - 1 - i : i; }
__host__ __device__ constexpr int b_all(bool inv, int kb) { return b_d(inv, kb, kb); }
__host__ __device__ constexpr int moment_blocks(int k) { return k > 16 ? (k + 15) / 16 : 1; }

// Two consecutive complex values of the data precision (complex64 data are 8-byte aligned).
template <typename D> struct Quad;
template <> struct Quad<float> { typedef float t __attribute__((ext_vector_type(4), aligned(8))); };
template <> struct Quad<double> { typedef double t __attribute__((ext_vector_type(4), aligned(16))); };

// the value of lane l ^ 1 (DPP quad permutation 1, 0, 3, 2)
__device__ __forceinline__ float swap_pair(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ double swap_pair(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0xB1, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0xB1, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

template <typename T, typename D, bool INV, bool KPH, int KB, int NCB>
struct Pipe64 {
    using V4 = typename Vec<T>::v4;
    using V2 = typename Vec<T>::v2;
    using D4 = typename Quad<D>::t;
    static constexpr bool F64 = sizeof(T) == sizeof(double);
    static constexpr int BLK = 64 * sizeof(V4);            // bytes of a block
    static constexpr int TILE = BLK * b_all(INV, KB);      // table bytes of a tile
    static constexpr int XSLOT = NCB * 4 * BLK, MSLOT = NCB * KB * BLK;
    // register sets of the table blocks (tiles in flight) and of the tile data
    // Step of the chain and result waves minus their tile.  FP32: 3, one more than
    // the data need, so that a wave reads its LDS operands of the next tile in the
    // step before; an FP64 step is twice as long and short of steps, not of time.
    static constexpr int kSkew = F64 ? 2 : 3;
    static constexpr int SETS = F64 ? (KB <= 2 ? 2 : 1) : (NCB == 2 && KB > 2 ? 2 : 4);
    static constexpr int SX = F64 || NCB == 2 ? 2 : 4;

    const D DSBT_GLOBAL* src;
    D DSBT_GLOBAL* dst;
    const unsigned char DSBT_GLOBAL* tab;
    const V2 DSBT_GLOBAL* kphase;
    const V2 DSBT_GLOBAL* kphase_lo;   // FP32: lo parts of the kinetic factors (kernels.h)
    unsigned char* xring;
    unsigned char* qring;
    unsigned char* mring;
    int NT, k, p, lane, q, odd;
    bool conj;
    int64_t e0[NCB];   // scalar index of slot 0 of this lane's channel, 8 cb + (l%16)/2

    __device__ Pipe64(const MItem& it, const void* s_, void* d_, const PhaseArgs& ph, unsigned char* lds)
        : src(as_global(static_cast<const D*>(s_))), dst(as_global_rw(static_cast<D*>(d_))) {
        NT = it.NT;
        k = it.k;
        p = it.p;
        lane = threadIdx.x & 63;
        q = lane >> 4;
        odd = lane & 1;
        conj = ph.conj != 0;
        tab = as_global(static_cast<const unsigned char*>(INV ? it.mf_i : it.mf_f));
        kphase = as_global(static_cast<const V2*>(it.kphase));
        kphase_lo = as_global(static_cast<const V2*>(it.kphase_lo));
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) e0[cb] = 2 * it.off[8 * cb + ((lane & 15) >> 1)];
        xring = lds;
        mring = xring + kXRing * XSLOT;
        qring = mring + kRing * MSLOT;
    }

    __device__ int tile(int t) const {
        const int c = t < NT ? t : NT - 1;
        return INV ? NT - 1 - c : c;
    }
    // A block, in a table or in LDS: FP32 16 bytes per lane; FP64 two halves of
    // 16 bytes per lane (each access of a wave is contiguous)
    template <typename P>
    static __device__ V4 ld_blk(P* s, int lane) {
        if constexpr (F64) {
            const V2 a = reinterpret_cast<const V2 DSBT_GLOBAL*>(s)[lane],
                     b = reinterpret_cast<const V2 DSBT_GLOBAL*>(s)[64 + lane];
            return V4{a[0], a[1], b[0], b[1]};
        } else {
            return reinterpret_cast<const V4 DSBT_GLOBAL*>(s)[lane];
        }
    }
    __device__ V4 ld_lds(const unsigned char* s) const {
        if constexpr (F64) {
            const V2 a = reinterpret_cast<const V2*>(s)[lane], b = reinterpret_cast<const V2*>(s)[64 + lane];
            return V4{a[0], a[1], b[0], b[1]};
        } else {
            return reinterpret_cast<const V4*>(s)[lane];
        }
    }
    __device__ void st_lds(unsigned char* s, V4 v) const {
        if constexpr (F64) {
            reinterpret_cast<V2*>(s)[lane] = V2{v[0], v[1]};
            reinterpret_cast<V2*>(s)[64 + lane] = V2{v[2], v[3]};
        } else {
            reinterpret_cast<V4*>(s)[lane] = v;
        }
    }
    // blocks B .. B + N - 1 of tile t
    template <int N>
    __device__ void ld_tab(V4* a, int t, int B) const {
        const unsigned char DSBT_GLOBAL* s = tab + (size_t)tile(t) * TILE + (size_t)B * BLK;
#pragma unroll
        for (int n = 0; n < N; ++n) a[n] = ld_blk(s + n * BLK, lane);
    }
    // One use of the N blocks a of tile t (block B of the table on): product i
    // with a[i], and block i of tile t + SETS into its registers once product
    // i + 1 is issued (issued sooner, the load would wait for the operand reads
    // of the product; later, it comes closer to its own use)
    template <int N, typename F>
    __device__ void use_blocks(V4* a, int t, int B, F&& product) const {
        const unsigned char DSBT_GLOBAL* s = tab + (size_t)tile(t + SETS) * TILE + (size_t)B * BLK;
#pragma unroll
        for (int i = 0; i <= N; ++i) {
            if (i < N) product(i);
            __builtin_amdgcn_sched_barrier(0);
            if (i > 0) a[i - 1] = ld_blk(s + (i - 1) * BLK, lane);
        }
    }
    // the blocks of tiles 0 .. SETS - 1 into their sets, in the order of the
    // steps: a wait on one set must not cover the loads of a later one
    template <int N>
    __device__ void ld_first(V4 (*a)[N], int B) const {
#pragma unroll
        for (int S = 0; S < SETS; ++S) {
            __builtin_amdgcn_sched_barrier(0);
            ld_tab<N>(a[S], S, B);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ unsigned char* x_at(int t, int cb, int b) const { return xring + (t % kXRing) * XSLOT + (cb * 4 + b) * BLK; }
    __device__ unsigned char* m_at(int t, int cb, int b) const { return mring + (t % kRing) * MSLOT + (cb * KB + b) * BLK; }
    __device__ unsigned char* q_at(int t, int cb, int b) const { return qring + (t % kRing) * MSLOT + (cb * KB + b) * BLK; }

    // c[cb] += a x[cb]: one 16 x 16 block, four instructions; two accumulators
    // per column block when only one is in flight.  REV: the instructions from the last
    template <bool REV = false>
    static __device__ void mma(V4 (*c)[2], V4 a, const V4* x) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                const int v = REV ? 3 - u : u;
                c[cb][v & 1] = Vec<T>::mfma(a[v], x[cb][v], c[cb][v & 1]);
            }
    }
    static __device__ V4 zero4() { return V4{0, 0, 0, 0}; }

    // f(set number, tile) for tiles 0 .. NT - 1, the set cycling through U
    // register sets.  The loop has no exit but its end: a break would reach the
    // loop's head in the flow graph, and its wait would then cover the loads of
    // every set.
    template <int U, int S, typename F>
    __device__ static void round(F&& f, int t) {
        if constexpr (S < U) {
            __builtin_amdgcn_sched_barrier(0);   // keep the steps in order
            f(std::integral_constant<int, S>{}, t + S);
            lds_barrier();
            round<U, S + 1>(f, t);
        }
    }
    template <int U, int S, typename F>
    __device__ void rest(F&& f, int t) const {
        if constexpr (S < U - 1) {
            if (t + S < NT) {
                f(std::integral_constant<int, S>{}, t + S);
                lds_barrier();
                rest<U, S + 1>(f, t);
            }
        }
    }
    template <int U, typename F>
    __device__ void steps(F&& f) const {
        int t = 0;
        for (; t + U <= NT; t += U) round<U, 0>(f, t);
        rest<U, 0>(f, t);
    }

    // ---- q = Q x: row blocks RB0 .. RB0 + NQ - 1 of tile s - 1 in step s ----
    template <int NQ>
    struct Qw {
        V4 a[SETS][NQ > 0 ? 4 * NQ : 1];
    };
    template <int S, int RB0, int NQ>
    __device__ void q_step(Qw<NQ>& r, int t) const {
        V4 x[4][NCB], c[NQ][NCB][2];
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) x[b][cb] = ld_lds(x_at(t, cb, b));
#pragma unroll
        for (int h = 0; h < NQ; ++h)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) c[h][cb][0] = c[h][cb][1] = zero4();
        use_blocks<4 * NQ>(r.a[S], t, b_q(INV, KB, RB0), [&](int i) { mma(c[i >> 2], r.a[S][i], x[i & 3]); });
#pragma unroll
        for (int h = 0; h < NQ; ++h)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) st_lds(q_at(t, cb, RB0 + h), c[h][cb][0] + c[h][cb][1]);
    }

    // ---- loading waves: half L of tile s in step s ----
    struct Kph {
        V4 w[2], wl[2];   // kinetic factors of the lane's four slots (wl: FP32 lo parts)
    };
    struct Load {
        D4 x[SX][NCB][2];
        Kph k[SX];
    };
    template <int L, int S>
    __device__ void x_load(Load& r, int t) const {
        // the lane's four slots of half L: in block 2 L (even lanes) or 2 L + 1 (odd)
        const int n0 = 64 * tile(t) + 32 * L + 16 * odd + 4 * q;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const D4 DSBT_GLOBAL* s = reinterpret_cast<const D4 DSBT_GLOBAL*>(src + e0[cb] + 2 * (int64_t)n0);
            r.x[S][cb][0] = s[0];
            r.x[S][cb][1] = s[1];
        }
        if constexpr (KPH) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                r.k[S].w[i] = *reinterpret_cast<const V4 DSBT_GLOBAL*>(kphase + n0 + 2 * i);
                if constexpr (!F64) r.k[S].wl[i] = *reinterpret_cast<const V4 DSBT_GLOBAL*>(kphase_lo + n0 + 2 * i);
            }
        }
    }
    // (v0 + i v1, v2 + i v3) times the kinetic factors w (+ l)
    __device__ V4 times_kphase(V4 v, V4 w, V4 l) const {
        const T s1 = conj ? -w[1] : w[1], s2 = conj ? -w[3] : w[3];
        if constexpr (!F64) {
            const T l1 = conj ? -l[1] : l[1], l2 = conj ? -l[3] : l[3];
            const float2 a = mul_unit(make_float2(v[0], v[1]), make_float2(w[0], s1), make_float2(l[0], l1));
            const float2 b = mul_unit(make_float2(v[2], v[3]), make_float2(w[2], s2), make_float2(l[2], l2));
            return V4{a.x, a.y, b.x, b.y};
        } else {
            return V4{v[0] * w[0] - v[1] * s1, v[0] * s1 + v[1] * w[0], v[2] * w[2] - v[3] * s2, v[2] * s2 + v[3] * w[2]};
        }
    }
    template <int L, int S>
    __device__ void x_stage(const Load& r, int t) const {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const D4* x = r.x[S][cb];
            // the lane pair (re, im) of a channel trades halves: the even lane
            // ends with the re of blocks 2 L and 2 L + 1, the odd one with the im
            V4 b[2];
            if constexpr (KPH) {
                V4 z[2];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    z[i] = times_kphase(__builtin_convertvector(x[i], V4), r.k[S].w[i], r.k[S].wl[i]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const T re = z[j >> 1][2 * (j & 1)], im = z[j >> 1][2 * (j & 1) + 1];
                    const T sre = swap_pair(re), sim = swap_pair(im);
                    b[0][j] = odd ? sim : re;
                    b[1][j] = odd ? im : sre;
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const D re = x[j >> 1][2 * (j & 1)], im = x[j >> 1][2 * (j & 1) + 1];
                    const D sre = swap_pair(re), sim = swap_pair(im);
                    b[0][j] = (T)(odd ? sim : re);
                    b[1][j] = (T)(odd ? im : sre);
                }
            }
            st_lds(x_at(t, cb, 2 * L), b[0]);
            st_lds(x_at(t, cb, 2 * L + 1), b[1]);
        }
    }
    template <int L, int S = 0>
    __device__ void x_first(Load& r) const {
        if constexpr (S < SX) {
            __builtin_amdgcn_sched_barrier(0);
            x_load<L, S>(r, S);
            x_first<L, S + 1>(r);
        }
    }
    template <int L>
    __device__ void run_load() const {
        Load r;
        x_first<L>(r);
        if constexpr (KB <= 2 + L) {
            steps<SX>([&](auto S, int t) {
                x_stage<L, S>(r, t);
                x_load<L, S>(r, t + SX);
            });
            for (int i = 0; i < kSkew; ++i) lds_barrier();
        } else {
            // also the q row block 2 + L: in the step that stages tile t + 1, of tile t
            Qw<1> w;
            ld_first(w.a, b_q(INV, KB, 2 + L));
            x_stage<L, 0>(r, 0);
            x_load<L, 0>(r, SX);
            lds_barrier();
            constexpr int U = SX > SETS ? SX : SETS;
            steps<U>([&](auto S, int t) {
                x_stage<L, (S + 1) % SX>(r, t + 1);   // (past the last tile: into a slot that no wave reads)
                x_load<L, (S + 1) % SX>(r, t + 1 + SX);
                q_step<S % SETS, 2 + L, 1>(w, t);
            });
            for (int i = 1; i < kSkew; ++i) lds_barrier();
        }
    }

    template <int RB0, int NQ>
    __device__ void run_q() const {
        Qw<NQ> r;
        ld_first(r.a, b_q(INV, KB, RB0));
        lds_barrier();
        steps<SETS>([&](auto S, int t) { q_step<S, RB0, NQ>(r, t); });
        for (int i = 1; i < kSkew; ++i) lds_barrier();
    }

    // ---- chain wave: mu_t+1 = q_t + D mu_t, tile s - kSkew in step s ----
    static constexpr int ND = KB * (KB + 1) / 2;
    struct Chain {
        V4 a[SETS][ND];
        V4 mu[KB][NCB];
        V4 q[KB][NCB];
    };
    __device__ void mu_out(const Chain& r, int t) const {
#pragma unroll
        for (int h = 0; h < KB; ++h)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) st_lds(m_at(t, cb, h), r.mu[h][cb]);
    }
    __device__ void chain_q(Chain& r, int t) const {
#pragma unroll
        for (int h = 0; h < KB; ++h)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) r.q[h][cb] = ld_lds(q_at(t, cb, h));
    }
    template <int S>
    __device__ void chain_step(Chain& r, int t) const {
        if constexpr (kSkew == 2) chain_q(r, t);
        V4 c[KB][NCB][2];
#pragma unroll
        for (int h = 0; h < KB; ++h)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                c[h][cb][0] = r.q[h][cb];
                c[h][cb][1] = zero4();
            }
        use_blocks<ND>(r.a[S], t, b_d(INV, KB, 0), [&](int i) {
#pragma unroll
            for (int h = 0; h < KB; ++h) {   // block i of D: row block h, column block b
                const int n = i - (b_d(INV, KB, h) - b_d(INV, KB, 0));
                if (n >= 0 && i < b_d(INV, KB, h + 1) - b_d(INV, KB, 0))
                    mma<INV>(c[h], r.a[S][i], r.mu[d_col(INV, KB, n)]);
            }
        });
        if constexpr (kSkew == 3) chain_q(r, t + 1);   // (past the last tile: an old value, not used)
#pragma unroll
        for (int h = 0; h < KB; ++h)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) r.mu[h][cb] = c[h][cb][0] + c[h][cb][1];
        mu_out(r, t + 1);
    }
    __device__ void run_chain() const {
        __builtin_amdgcn_s_setprio(2);   // the serial role goes first on its SIMD
        Chain r;
        ld_first(r.a, b_d(INV, KB, 0));
        // mu_0: zero forward; inverse (-1)^p times the completion slots 0..k-1
        // of tile 0 (with their kinetic factors)
        const T sgn = p ? -1 : 1;
#pragma unroll
        for (int h = 0; h < KB; ++h)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    T x = 0;
                    if constexpr (INV) {
                        const int row = 16 * h + 4 * v + q;
                        const int n = row < k ? row : 0;
                        T re = (T)src[e0[cb] + 2 * n], im = (T)src[e0[cb] + 2 * n + 1];
                        if constexpr (KPH) {
                            const V2 w = kphase[n];
                            V2 l = {0, 0};
                            if constexpr (!F64) l = kphase_lo[n];
                            const V4 z = times_kphase(V4{re, im, 0, 0}, V4{w[0], w[1], 0, 0}, V4{l[0], l[1], 0, 0});
                            re = z[0];
                            im = z[1];
                        }
                        x = row < k ? sgn * (odd ? im : re) : T(0);
                    }
                    r.mu[h][cb][v] = x;
                }
        mu_out(r, 0);
        for (int i = 0; i < 2; ++i) lds_barrier();
        if constexpr (kSkew == 3) {
            chain_q(r, 0);
            lds_barrier();
        }
        steps<SETS>([&](auto S, int t) { chain_step<S>(r, t); });
        if constexpr (!INV) {
            // completion rows (-1)^p mu_NT into slots 0..k-1 of tile 0, after the
            // result waves' stores of tile 0
            __syncthreads();
#pragma unroll
            for (int h = 0; h < KB; ++h)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 16 * h + 4 * v + q;
                        if (row < k) dst[e0[cb] + 2 * row + odd] = (D)(sgn * r.mu[h][cb][v]);
                    }
        }
    }

    // ---- result waves: row block RB of o_t, tile s - kSkew in step s ----
    template <int RB>
    struct Out {
        static constexpr int NXB = x_hi(INV, RB) - x_lo(INV, RB), N = NXB + KB;
        V4 a[SETS][N];
        V4 x[NXB][NCB];   // the data blocks of the next tile, read one step ahead
    };
    template <int RB>
    __device__ void out_x(Out<RB>& r, int t) const {
#pragma unroll
        for (int b = 0; b < Out<RB>::NXB; ++b)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) r.x[b][cb] = ld_lds(x_at(t, cb, x_lo(INV, RB) + b));
    }
    template <int RB, int S>
    __device__ void out_step(Out<RB>& r, int t) const {
        if constexpr (kSkew == 2) out_x(r, t);
        V4 m[KB][NCB], c[NCB][2], e[NCB][2];
#pragma unroll
        for (int h = 0; h < KB; ++h)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) m[h][cb] = ld_lds(m_at(t, cb, h));
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) c[cb][0] = c[cb][1] = e[cb][0] = e[cb][1] = zero4();
        use_blocks<Out<RB>::N>(r.a[S], t, b_out(INV, KB, RB), [&](int i) {
            const int col = out_col(INV, KB, RB, i);
            if (col < 4) mma(c, r.a[S][i], r.x[col < 4 ? col - x_lo(INV, RB) : 0]);
            else mma(e, r.a[S][i], m[col < 4 ? 0 : col - 4]);
        });
        if constexpr (kSkew == 3) out_x(r, t + 1);   // staged two steps ago (past the last tile: an old slot, not used)
        // a lane holds rows 4 q + v of the re (even) or im (odd) part: the pair
        // trades values so that the even lane stores slots 4 q, 4 q + 1 and the
        // odd one 4 q + 2, 4 q + 3 as (re, im, re, im).  Forward: slots 0..k-1 of
        // tile 0 are rewritten with the completion rows at the end.
        const int n0 = 64 * tile(t) + 16 * RB + 4 * q + 2 * odd;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const V4 o = (c[cb][0] + c[cb][1]) + (e[cb][0] + e[cb][1]);
            const D w[4] = {(D)o[0], (D)o[1], (D)o[2], (D)o[3]};
            const D s0 = swap_pair(w[0]), s1 = swap_pair(w[1]), s2 = swap_pair(w[2]), s3 = swap_pair(w[3]);
            *reinterpret_cast<D4 DSBT_GLOBAL*>(dst + e0[cb] + 2 * (int64_t)n0) =
                D4{odd ? s2 : w[0], odd ? w[2] : s0, odd ? s3 : w[1], odd ? w[3] : s1};
        }
    }
    template <int RB>
    __device__ void run_out() const {
        Out<RB> r;
        ld_first(r.a, b_out(INV, KB, RB));
        for (int i = 0; i < 2; ++i) lds_barrier();
        if constexpr (kSkew == 3) {
            out_x(r, 0);
            lds_barrier();
        }
        steps<SETS>([&](auto S, int t) { out_step<RB, S>(r, t); });
    }

    __device__ void run() const {
        // Waves w and w + 4 share a SIMD, and no instruction of one issues during
        // a matrix instruction of the other: the roles are paired so that the
        // four SIMDs carry about the same number of blocks.  H(i): the result
        // row block with the i-th most blocks.  Blocks per tile and SIMD, for
        // KB = 1: 5, 1 + 4, 3 + 2, 4; 2: 6, 3 + 5, 4 + 3, 8; 3: 7 + 4, 6 + 5,
        // 6 + 4, 8; 4: 8 + 4, 10 + 5, 7 + 6, 8 + 4.
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        constexpr int H0 = INV ? 0 : 3, H1 = INV ? 1 : 2, H2 = INV ? 2 : 1, H3 = INV ? 3 : 0;
        constexpr int PC = KB <= 2 ? H1 : KB == 3 ? H2 : H3;   // beside the chain
        constexpr int PA = KB <= 2 ? H2 : H1, PB = KB <= 3 ? H3 : H2;
        switch (wave) {
            case 0: run_out<H0>(); break;
            case 1: run_chain(); break;
            case 2: run_out<PA>(); break;
            case 3: run_q<0, (KB > 1 ? 2 : 1)>(); break;
            case 4: run_load<0>(); break;
            case 5: run_out<PC>(); break;
            case 6: run_out<PB>(); break;
            default: run_load<1>(); break;
        }
        if constexpr (!INV) {
            if (wave != 1) __syncthreads();   // pairs with the one before the completion rows
        }
    }
};

template <typename T, typename D, bool INV, bool KPH, int KBMAX, int NCB>
__device__ __forceinline__ void pipe_item(const MItem& it, const void* src, void* dst, const PhaseArgs& ph,
                                          unsigned char* lds) {
    const int kb = moment_blocks(it.k);
    if constexpr (KBMAX > 2) {
        if (kb == 3) {
            Pipe64<T, D, INV, KPH, 3, NCB>(it, src, dst, ph, lds).run();
            return;
        }
        if (kb == 4) {
            Pipe64<T, D, INV, KPH, 4, NCB>(it, src, dst, ph, lds).run();
            return;
        }
    }
    if (kb == 2) Pipe64<T, D, INV, KPH, 2, NCB>(it, src, dst, ph, lds).run();
    else Pipe64<T, D, INV, KPH, 1, NCB>(it, src, dst, ph, lds).run();
}

template <typename T, typename D, bool INV, bool KPH, int KBMAX>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) mstage_pipe(const MItem* __restrict__ items, const void* src, void* dst,
                                                   PhaseArgs ph) {
    extern __shared__ __align__(16) unsigned char lds_pipe[];
    const MItem& it = items[blockIdx.x];
    if (it.nch == 0) return;   // idle slot of the per-XCD schedule
    if constexpr (sizeof(T) == sizeof(float)) {
        if (it.NCB == 2) {
            pipe_item<T, D, INV, KPH, KBMAX, 2>(it, src, dst, ph, lds_pipe);
            return;
        }
    }
    pipe_item<T, D, INV, KPH, KBMAX, 1>(it, src, dst, ph, lds_pipe);   // FP64 items have one column block
}

// Items of both tile sizes in one launch (FP32 plans with l on both sides of 64):
// workgroup b takes entries 2 b and 2 b + 1 of the list, either an item of tiles of
// 64 (entry 2 b, all eight waves) or two items of tiles of 32, four waves each, or
// one and an empty entry.  Waves w and w + 4 share a SIMD, so the roles of the
// second item are one place further along: each SIMD holds role r of one item and
// r - 1 of the other (mstage_chain.h).  The two items meet at the same barriers; an
// item with fewer tiles, or an empty entry, ends early, and the barrier then waits
// for the waves that are left.  As two launches in turn each waits for its longest
// chain: uneven batch of 512 channels (l <= 127, N to 8192), forward and inverse, 525
// us as two launches, 390 in one; 3D step 64 x 17 x 4096 (l <= 71) 404 and 302.
template <bool INV, bool KPH>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) mstage_mixed(const MItem* __restrict__ items, const void* src, void* dst,
                                                    PhaseArgs ph) {
    extern __shared__ __align__(16) unsigned char lds_pipe[];
    const MItem* pair = items + 2 * blockIdx.x;
    if (pair[0].B == 64) {
        if (pair[0].NCB == 2) pipe_item<float, float, INV, KPH, 4, 2>(pair[0], src, dst, ph, lds_pipe);
        else pipe_item<float, float, INV, KPH, 4, 1>(pair[0], src, dst, ph, lds_pipe);
        return;
    }
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int role = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) + 3 * half) & 3;
    const MItem& it = pair[half];
    if (it.nch == 0) return;
    float* lds = reinterpret_cast<float*>(lds_pipe) + (half ? chain::chain_lds_values(pair[0].NCB) : 0);
    if (it.NCB == 2) chain::run_item<float, float, INV, KPH, 2>(it, src, dst, ph, lds, role);
    else chain::run_item<float, float, INV, KPH, 1>(it, src, dst, ph, lds, role);
}

// One 16 x 16 block per workgroup (tile blockIdx.x, block blockIdx.y) of the
// table of one direction from the FP64 blocks M_J[r][q] (row-major, R = 64 + k).
// The weight w_0 of odd l is folded into slot 0 of tile 0.
template <typename T>
__global__ void __launch_bounds__(64) pack_blocks(const double* __restrict__ blocks, int k, int p, int inverse,
                                                  T* __restrict__ out) {
    const int J = blockIdx.x, u = blockIdx.y, lane = threadIdx.x;
    const bool inv = inverse != 0;
    const int kb = moment_blocks(k), R = 64 + k;
    int row0 = 0, col0 = 0, rb = 0;   // first row and column of the block (64..: the moments)
    if (u < b_q(inv, kb, 0)) {
        while (u >= b_out(inv, kb, rb + 1)) ++rb;
        row0 = 16 * rb;
        col0 = 16 * out_col(inv, kb, rb, u - b_out(inv, kb, rb));
    } else if (u < b_d(inv, kb, 0)) {
        const int i = u - b_q(inv, kb, 0);
        row0 = 64 + 16 * (i / 4);
        col0 = 16 * (i % 4);
    } else {
        while (u >= b_d(inv, kb, rb + 1)) ++rb;
        row0 = 64 + 16 * rb;
        col0 = 64 + 16 * d_col(inv, kb, u - b_d(inv, kb, rb));
    }
    const int i = lane & 15, q = lane >> 4;
    // result row i of the instruction is at lane quarter i / 4, register i % 4 (FP64 the
    // other way round): permuted where that is not the lane layout of the rows
    const bool swap = (row0 >= 64) != (sizeof(T) == sizeof(double));
    const int row = row0 + (swap ? 4 * (i & 3) + (i >> 2) : i);
    const double* M = blocks + (size_t)J * R * R;
    T* o = out + ((size_t)J * gridDim.y + u) * 256;
    for (int v = 0; v < 4; ++v) {
        const int col = col0 + (col0 >= 64 ? 4 * v + q : 4 * q + v);
        double a = 0.0;
        if (row < R && col < R) {
            a = inv ? M[(size_t)col * R + row] : M[(size_t)row * R + col];
            if (J == 0 && p == 0 && (inv ? row : col) == 0) a *= 0.70710678118654752440;
        }
        o[sizeof(T) == sizeof(double) ? 128 * (v >> 1) + 2 * lane + (v & 1) : 4 * lane + v] = (T)a;
    }
}

}  // namespace

template <typename T>
size_t pipe_table_bytes(int k, int NT) {
    return (size_t)NT * b_all(false, moment_blocks(k)) * 256 * sizeof(T);
}

template <typename T>
hipError_t launch_pack_pipe(const double* d_blocks, int k, int p, int NT, bool inverse, void* out, hipStream_t s) {
    if (k < 0 || k > 64 || NT < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(pack_blocks<T>, dim3(NT, b_all(inverse, moment_blocks(k))), dim3(64), 0, s, d_blocks, k, p,
                       inverse ? 1 : 0, static_cast<T*>(out));
    return hipGetLastError();
}

template <typename T>
size_t pipe_lds_bytes(int k, int ncb) {
    return (size_t)ncb * (4 * kXRing + 2 * kRing * moment_blocks(k)) * 256 * sizeof(T);
}

template <typename T>
hipError_t set_lds_limits_pipe() {
    hipError_t e = hipSuccess;
    const int bytes = (int)pipe_lds_bytes<T>(64, sizeof(T) == sizeof(float) ? 2 : 1);
    auto set = [&](const void* f) {
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    };
    set((const void*)mstage_pipe<T, float, true, false, 2>);
    set((const void*)mstage_pipe<T, float, true, true, 2>);
    set((const void*)mstage_pipe<T, float, false, false, 2>);
    set((const void*)mstage_pipe<T, float, true, false, 4>);
    set((const void*)mstage_pipe<T, float, true, true, 4>);
    set((const void*)mstage_pipe<T, float, false, false, 4>);
    if constexpr (sizeof(T) == sizeof(double)) {
        set((const void*)mstage_pipe<T, double, true, false, 2>);
        set((const void*)mstage_pipe<T, double, true, true, 2>);
        set((const void*)mstage_pipe<T, double, false, false, 2>);
        set((const void*)mstage_pipe<T, double, true, false, 4>);
        set((const void*)mstage_pipe<T, double, true, true, 4>);
        set((const void*)mstage_pipe<T, double, false, false, 4>);
    }
    return e;
}

hipError_t launch_mstage_mixed(const MItem* d_items, int nblocks, size_t lds, const void* src, void* dst, bool inverse,
                               PhaseArgs ph, hipStream_t s) {
    if (nblocks <= 0) return hipSuccess;
    if (!inverse && ph.use) return hipErrorInvalidValue;   // phases are applied to the inverse's input only
    const dim3 grid(nblocks), block(512);
    if (inverse && ph.use)
        hipLaunchKernelGGL((mstage_mixed<true, true>), grid, block, lds, s, d_items, src, dst, ph);
    else if (inverse)
        hipLaunchKernelGGL((mstage_mixed<true, false>), grid, block, lds, s, d_items, src, dst, ph);
    else
        hipLaunchKernelGGL((mstage_mixed<false, false>), grid, block, lds, s, d_items, src, dst, ph);
    return hipGetLastError();
}

hipError_t set_lds_limits_mixed() {
    const int bytes = (int)(2 * chain_lds_bytes<float>(2));   // two items of two column blocks: the most of any entry pair
    for (const void* f : {(const void*)mstage_mixed<true, false>, (const void*)mstage_mixed<true, true>,
                          (const void*)mstage_mixed<false, false>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T, typename D, int KBMAX>
static void launch_kb(const MItem* d_items, int nitems, size_t lds, const void* src, void* dst, bool inverse,
                      PhaseArgs ph, hipStream_t s) {
    const dim3 grid(nitems), block(512);
    if (inverse && ph.use)
        hipLaunchKernelGGL((mstage_pipe<T, D, true, true, KBMAX>), grid, block, lds, s, d_items, src, dst, ph);
    else if (inverse)
        hipLaunchKernelGGL((mstage_pipe<T, D, true, false, KBMAX>), grid, block, lds, s, d_items, src, dst, ph);
    else
        hipLaunchKernelGGL((mstage_pipe<T, D, false, false, KBMAX>), grid, block, lds, s, d_items, src, dst, ph);
}

template <typename T, typename D>
hipError_t launch_mstage_pipe(const MItem* d_items, int nitems, int maxk, size_t lds, const void* src, void* dst,
                              bool inverse, PhaseArgs ph, hipStream_t s) {
    if (nitems <= 0) return hipSuccess;
    if (maxk < 0 || maxk > 64) return hipErrorInvalidValue;
    if (!inverse && ph.use) return hipErrorInvalidValue;   // phases are applied to the inverse's input only
    if (maxk <= 32) launch_kb<T, D, 2>(d_items, nitems, lds, src, dst, inverse, ph, s);
    else launch_kb<T, D, 4>(d_items, nitems, lds, src, dst, inverse, ph, s);
    return hipGetLastError();
}

template size_t pipe_table_bytes<float>(int, int);
template size_t pipe_table_bytes<double>(int, int);
template hipError_t launch_pack_pipe<float>(const double*, int, int, int, bool, void*, hipStream_t);
template hipError_t launch_pack_pipe<double>(const double*, int, int, int, bool, void*, hipStream_t);
template size_t pipe_lds_bytes<float>(int, int);
template size_t pipe_lds_bytes<double>(int, int);
template hipError_t set_lds_limits_pipe<float>();
template hipError_t set_lds_limits_pipe<double>();
template hipError_t launch_mstage_pipe<float, float>(const MItem*, int, int, size_t, const void*, void*, bool, PhaseArgs,
                                                     hipStream_t);
template hipError_t launch_mstage_pipe<double, float>(const MItem*, int, int, size_t, const void*, void*, bool, PhaseArgs,
                                                      hipStream_t);
template hipError_t launch_mstage_pipe<double, double>(const MItem*, int, int, size_t, const void*, void*, bool, PhaseArgs,
                                                       hipStream_t);

}  // namespace dsbt
