// kernels.hip — gfx950 kernels of the KKT hot path.
//
//   assembly   K = W + Sigma + rho J^T J (Sec. 3.3, eq. K1) or the stabilized
//              [[W + Sigma, J^T], [J, -1/rho I]] (Sec. 3.2, eq. K2r) on the
//              fixed pattern in FP64, a block per chunk of rows, which also
//              takes the rows' norms.
//   factor     supernodal multifrontal LDL^T with the static-pivot rule of
//              Sec. 3.1 (|d| < thr -> d = sign * thr, sign of the pivot's
//              block before reordering); fronts processed level by level:
//                * small fronts: one or four waves per front, its tiles in
//                  MFMA accumulators (children's contribution blocks gathered
//                  into them), its pivot columns in LDS;
//                * large fronts: the front lives in the factor buffer; one
//                  launch assembles it column by column, then per pivot panel
//                  a diagonal-block factor and its inverse by four waves, a
//                  panel solve, and a trailing update on MFMA
//                  (v_mfma_f64_16x16x4 / f32) beside the next diagonal block.
//   solve      level-scheduled multifrontal forward sweep (children's
//              update vectors pulled by the parent: no atomics), D^-1, and
//              backward sweep, for one right-hand side or, on MFMA, sixteen.
//   refinement residual b - K x with per-system backward errors.
// All reductions are deterministic; integer atomics only count inertia.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "kernels.hpp"

namespace ncl {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ double to_d(double x) { return x; }
__device__ __forceinline__ double to_d(float x) { return (double)x; }

// Static-pivot thresholds of one system (Sec. 3.1): p for pivots of the
// primal block, n for pivots of the dual block (equal unless the thresholds
// are block-scaled).
struct PivThr {
    double p, n;
    __device__ PivThr(const double* sys_thr, int sys) : p(sys_thr[2 * sys]), n(sys_thr[2 * sys + 1]) {}
};

// Adds a workgroup's pivot counts to one of the system's partial counters
// (many fronts finish at once; one shared counter would serialize them).
__device__ __forceinline__ void add_inertia(unsigned long long* part, int sys, const unsigned int* cnt, int slot) {
    unsigned long long* in4 = part + 4 * ((int64_t)sys * kInertiaSlots + (slot & (kInertiaSlots - 1)));
    for (int k = 0; k < 4; ++k)
        if (cnt[k]) atomicAdd(&in4[k], (unsigned long long)cnt[k]);
}

// 16x16x4 MFMA wrappers.  Operands: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16].  Result item r of lane l is D[row(l / 16, r)][l % 16];
// the row order differs between the f64 and f32 instructions (checked on
// gfx950 with a one-hot probe).
//
// The compiler inserts the wait states of dependent MFMAs itself (none between
// the links of a chain on one accumulator, 19 before an f64 result is read).
// Chains once carried 16 more each, against a difference from run to run that
// was the panel solve's (see panel_body).
template <typename T> struct Mfma;
template <> struct Mfma<double> {
    typedef f64x4 acc_t;
    static __device__ __forceinline__ acc_t run(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lk, int r) { return 4 * r + lk; }
};
template <> struct Mfma<float> {
    typedef f32x4 acc_t;
    static __device__ __forceinline__ acc_t run(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lk, int r) { return 4 * lk + r; }
};

// 1/d from the hardware reciprocal refined by two Newton steps (within ~1 ulp
// of the rounded quotient); shorter dependent latency than a full division.
__device__ __forceinline__ double fast_rcp(double d) {
    double r = __builtin_amdgcn_rcp(d);
    double e = __builtin_fma(-d, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-d, r, 1.0);
    return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float fast_rcp(float d) {
    float r = __builtin_amdgcn_rcpf(d);
    const float e = __builtin_fmaf(-d, r, 1.0f);
    return __builtin_fmaf(r, e, r);
}

// Value of `v` held by lane `src` (a compile-time / wave-uniform lane index).
__device__ __forceinline__ double bcast(double v, int src) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), src);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ float bcast(float v, int src) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
}

// Compiler-level fence: keeps LDS accesses of one wave in program order.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_wave_barrier();
    __asm__ volatile("" ::: "memory");
}

// Value of lane 16 * (lane / 16) + U of each 16-lane row (DPP row_newbcast).
template <int U>
__device__ __forceinline__ double rowbcast(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const long long r = __builtin_amdgcn_update_dpp(b, b, 0x150 + U, 0xf, 0xf, true);
    return __builtin_bit_cast(double, r);
}
template <int U>
__device__ __forceinline__ float rowbcast(float v) {
    const int b = __builtin_bit_cast(int, v);
    const int r = __builtin_amdgcn_update_dpp(b, b, 0x150 + U, 0xf, 0xf, true);
    return __builtin_bit_cast(float, r);
}
template <typename T>
__device__ __forceinline__ T rowbcast_n(T v, int u) {   // u: a compile-time constant after unrolling
    switch (u) {
        case 0: return rowbcast<0>(v);   case 1: return rowbcast<1>(v);   case 2: return rowbcast<2>(v);
        case 3: return rowbcast<3>(v);   case 4: return rowbcast<4>(v);   case 5: return rowbcast<5>(v);
        case 6: return rowbcast<6>(v);   case 7: return rowbcast<7>(v);   case 8: return rowbcast<8>(v);
        case 9: return rowbcast<9>(v);   case 10: return rowbcast<10>(v); case 11: return rowbcast<11>(v);
        case 12: return rowbcast<12>(v); case 13: return rowbcast<13>(v); case 14: return rowbcast<14>(v);
        default: return rowbcast<15>(v);
    }
}

// The pivots of one 16-column sub-panel: right-looking LDL^T of the 16 x 16
// diagonal block with one more row per lane below it, by the static-pivot rule of
// Sec. 3.1: a pivot |d| < t (strict), t the threshold of its block, becomes +t for a
// primal pivot and -t for a dual one (bit t of dual).  rp: row lane % 16 of the
// diagonal block, the same in each 16-lane row of the wave, so that the pivots'
// reciprocals and the multipliers of the other columns come from lane t and u of the
// lane's own row by DPP (one instruction, against two readlanes through scalar
// registers); x: the lane's own row below.  On return both hold L, dk the pivot of
// row lane % 16 and pk whether it was replaced.  The next pivot's column is updated
// first, so that its reciprocal runs under the other columns' updates.
// The chain is bound by the issue of ~45 instructions per pivot (290 cycles, against
// ~65 of dependent latency), so each lane applies the rule to its own row's pivot
// with its own threshold: one comparison and a select before the broadcast.  (One
// test after all 16 pivots, against the larger threshold, and a sub-panel that failed
// it done again pivot by pivot in LDS: a stabilized OPF factorization of order 8k
// took 927 us with the absolute rule, 1618 with the block rule and 1568 with the
// global one, so 909, 913 and 909.  The rule on the broadcast pivot, with the
// thresholds in scalar registers: 2.5 to 5 per cent longer factorizations.)
// Pivots t >= bw are skipped.
template <typename T>
__device__ __forceinline__ void pivots16(T (&rp)[16], T (&x)[16], T& dk, bool& pk, int bw, PivThr thr,
                                         unsigned int dual, int li) {
    const bool n = dual >> li & 1u;
    const double tl = n ? thr.n : thr.p;
    const T rl = (T)(n ? -tl : tl), il = T(1) / rl;
    auto reciprocal = [&](T d) {
        const T r = fast_rcp(d);
        return fabs(to_d(d)) < tl ? il : r;
    };
    T inv = rowbcast_n(reciprocal(rp[0]), 0);
    dk = T(1);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        if (t >= bw) continue;   // uniform
        const T l = rp[t] * inv;
        const T lx = x[t] * inv;
        if (t + 1 < 16) {
            const T c = rowbcast_n(rp[t], t + 1);
            rp[t + 1] -= l * c;
            x[t + 1] -= lx * c;
            inv = rowbcast_n(reciprocal(rp[t + 1]), t + 1);
        }
#pragma unroll
        for (int u = t + 2; u < 16; ++u) {
            const T c = rowbcast_n(rp[t], u);
            rp[u] -= l * c;
            x[u] -= lx * c;
        }
        dk = li == t ? rp[t] : dk;
        rp[t] = l;
        x[t] = lx;
        // x is updated here, not where the caller comes to use it: that would hold
        // all 120 broadcasts in registers until then
        if ((t & 3) == 3)
#pragma unroll
            for (int u = 0; u < 16; ++u) asm volatile("" : "+v"(x[u]));
    }
#pragma unroll
    for (int t = 0; t < 16; ++t) asm volatile("" : "+v"(x[t]));   // (bw < 16)
    pk = fabs(to_d(dk)) < tl;
    dk = pk ? rl : dk;
}

// Counts of a sub-panel's first bw pivots (lane % 16 < bw): positive, negative,
// zero, replaced; and whether one is not finite.
template <typename T>
__device__ __forceinline__ void count_pivots(T dk, bool pk, int bw, int lane, unsigned int* cnt, bool& bad) {
    const bool in = lane < bw;
    const unsigned int a = __popcll(__ballot(in && to_d(dk) > 0.0)), b = __popcll(__ballot(in && to_d(dk) < 0.0)),
                       c = __popcll(__ballot(in && to_d(dk) == 0.0)), e = __popcll(__ballot(in && pk));
    bad |= __ballot(in && !isfinite(to_d(dk))) != 0ULL;
    cnt[0] += a; cnt[1] += b; cnt[2] += c; cnt[3] += e;
}

// ---- one diagonal block of a large front ---------------------------------
// LDL^T of a kPanel x kPanel diagonal block and Z = L^-1, by the workgroup.
// The block's ten lower 16 x 16 tiles stay in MFMA accumulators (three a wave)
// and only the next 16-column sub-panel goes through LDS, where wave 0 factors
// it; meanwhile waves 1..3 apply the previous sub-panel to the tiles beyond
// and build the block row of Z that it completes.  The block was a chain of
// LDS round trips: with every tile in LDS and Z formed afterwards it took
// 10 us + 4.4 us a block (order 20k), of which the pivots themselves are 3.8.
// Tiles are held transposed (lane % 16 = row), so that a column's entries are
// contiguous over lanes in LDS and in the front.
constexpr int kDiagLd = 80;   // leading dimension of the LDS block: 16 mod 32 doubles, so that the
                              // four 16-row column pieces an operand load takes lie in different banks

// The tiles of a wave: slot t of wave v is block row ti, block column tj.
// Wave 0 has (0,0) only, wave 1 (1,0), (1,1), (3,3), waves 2 and 3 their block
// row's first three.
__device__ __forceinline__ int diag_ti(int wave, int t) { return wave == 1 && t == 2 ? 3 : wave; }
__device__ __forceinline__ int diag_tj(int wave, int t) { return wave == 1 && t == 2 ? 3 : t; }
__device__ __forceinline__ bool diag_has(int wave, int t) { return wave > 0 || t == 0; }

// Z[u][t] of the LDS block: strictly lower entries are stored transposed in
// the strictly upper triangle.
template <typename T>
__device__ __forceinline__ T zget(const T* B, int u, int t) {
    return u > t ? B[t + u * kDiagLd] : (u == t ? T(1) : T(0));
}

// acc (a tile at block (ti, tj), transposed) -= L_ti D L_tj^T of sub-panel q,
// L in LDS with leading dimension ld.  The 16 products are summed from zero: added
// one by one to the tile, each was rounded to its last place (unrefined residuals of
// an OPF of order 2000 up to 1.35 times as large, the same time).
template <typename T>
__device__ __forceinline__ void diag_apply(typename Mfma<T>::acc_t& acc, const T* B, int ld, const T* dv, int q, int ti,
                                           int tj, int lr, int lk) {
    T a[4], b[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const int t = 16 * q + 4 * st + lk;
        a[st] = B[(16 * tj + lr) + t * ld] * -dv[t];
        b[st] = B[(16 * ti + lr) + t * ld];
    }
    typename Mfma<T>::acc_t sum = {0, 0, 0, 0};
#pragma unroll
    for (int st = 0; st < 4; ++st) sum = Mfma<T>::run(a[st], b[st], sum);
    acc += sum;
}

// Z_qq = L_qq^-1 of a 16 x 16 unit lower block by one wave: lane % 16 = row j
// of Z, the same in each 16-lane row; step t takes L[j][t] times row t away
// (DPP broadcast).  Waves that need Z_qq at the same time each do this and write the
// same values.
template <typename T>
__device__ __forceinline__ void diag_inv16(T* B, int ld, int q, int lane) {
    const int o = 16 * q, j = lane & 15;
    T z[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) z[u] = (u == j) ? T(1) : T(0);
#pragma unroll
    for (int t = 0; t < 15; ++t) {
        const T x = B[(o + j) + (o + t) * ld];
        const T l = j > t ? x : T(0);
#pragma unroll
        for (int u = 0; u <= t; ++u) z[u] = __builtin_fma(-l, rowbcast_n(z[u], t), z[u]);
    }
    wave_fence();
    if (lane < 16) {
#pragma unroll
        for (int u = 0; u < 15; ++u)
            if (j > u) B[(o + u) + (o + j) * ld] = z[u];
    }
    wave_fence();
}

// Column j of Z's block row i, first half: S = sum_{k = j}^{i - 1} L_ik Z_kj.
template <typename T>
__device__ __forceinline__ void diag_zsum(typename Mfma<T>::acc_t& S, const T* B, int i, int j, int lr, int lk) {
    S = typename Mfma<T>::acc_t{0, 0, 0, 0};
    for (int k = j; k < i; ++k) {
        T la[4], zb[4];
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            const int kk = 16 * k + Mfma<T>::row(lk, st);
            la[st] = B[(16 * i + lr) + kk * kDiagLd];
            zb[st] = zget(B, kk, 16 * j + lr);
        }
#pragma unroll
        for (int st = 0; st < 4; ++st) S = Mfma<T>::run(la[st], zb[st], S);
    }
}

// ... second half: Z_ij = -Z_ii S.
template <typename T>
__device__ __forceinline__ void diag_zrow(const typename Mfma<T>::acc_t& S, T* B, int i, int j, int lr, int lk) {
    typename Mfma<T>::acc_t R = {0, 0, 0, 0};
    T zi[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) zi[st] = zget(B, 16 * i + lr, 16 * i + Mfma<T>::row(lk, st));
#pragma unroll
    for (int st = 0; st < 4; ++st) R = Mfma<T>::run(zi[st], S[st], R);
#pragma unroll
    for (int r = 0; r < 4; ++r) B[(16 * j + lr) + (16 * i + Mfma<T>::row(lk, r)) * kDiagLd] = -R[r];
    wave_fence();
}

// Factors the block whose tiles are in acc (first w pivots; entries beyond are
// taken as the identity), leaving L strictly below the diagonal of B, Z
// transposed above it (rows past the last sub-panel unwritten) and the pivots
// in dv.  Bit c of negmask: pivot c takes the negative sign; wave 0 adds the
// counts of the w pivots to its cnt[4].  Called by all 256 threads; B is
// free on entry; ends with a barrier.
template <typename T>
__device__ __forceinline__ void diag_factor(typename Mfma<T>::acc_t (&acc)[3], T* B, T* dv,
                                            unsigned long long negmask, int w, PivThr thr,
                                            unsigned int* cnt, bool& bad_out, int tid) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lr = lane & 15, lk = lane >> 4;
    const int nq = (w + 15) >> 4;
    bool bad_any = false;
    typename Mfma<T>::acc_t S = {0, 0, 0, 0};
    // side work of waves 1..3 once sub-panel i is factored: the diagonal block
    // of Z, and block (i, wave - 1) from the sum formed before
    auto zstep = [&](int i) {
        if (wave <= i + 1) diag_inv16<T>(B, kDiagLd, i, lane);
        if (wave <= i) diag_zrow<T>(S, B, i, wave - 1, lr, lk);
    };
#pragma unroll 1
    for (int q = 0; q < nq; ++q) {
        const int kb = 16 * q;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            if (!diag_has(wave, t) || diag_tj(wave, t) != q) continue;   // uniform
            const int row = 16 * diag_ti(wave, t) + lr;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int col = kb + Mfma<T>::row(lk, r);
                B[row + col * kDiagLd] = row < w && col < w ? acc[t][r] : (row == col ? T(1) : T(0));
            }
        }
        __syncthreads();
        if (wave == 0) {
            const int row = kb + 16 + lane;
            const int rowc = min(row, kPanel - 1);
            T rp[16], x[16], dk;
            bool pk;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                rp[t] = B[(kb + lr) + (kb + t) * kDiagLd];
                x[t] = B[rowc + (kb + t) * kDiagLd];
            }
            pivots16(rp, x, dk, pk, 16, thr, (unsigned int)(negmask >> kb) & 0xffffu, lr);
            // the diagonal block's upper triangle takes scratch values: it
            // is written as Z before it is read
            if (row < kPanel)
#pragma unroll
                for (int t = 0; t < 16; ++t) B[row + (kb + t) * kDiagLd] = x[t];
            if (lane < 16) {
#pragma unroll
                for (int t = 0; t < 16; ++t) B[(kb + lane) + (kb + t) * kDiagLd] = rp[t];
                dv[kb + lane] = dk;
            }
            count_pivots(dk, pk, min(16, w - kb), lane, cnt, bad_any);
        } else if (q > 0) {
#pragma unroll
            for (int t = 0; t < 3; ++t)
                if (diag_tj(wave, t) > q) diag_apply<T>(acc[t], B, kDiagLd, dv, q - 1, diag_ti(wave, t), diag_tj(wave, t), lr, lk);
            zstep(q - 1);
            if (wave <= q) diag_zsum<T>(S, B, q, wave - 1, lr, lk);
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 3; ++t)
            if (diag_has(wave, t) && diag_tj(wave, t) == q + 1)
                diag_apply<T>(acc[t], B, kDiagLd, dv, q, diag_ti(wave, t), q + 1, lr, lk);
    }
    if (wave > 0) zstep(nq - 1);
    __syncthreads();
    bad_out = bad_any;
}

// Workgroups are dealt to the 8 XCDs round-robin (workgroup b runs on XCD
// b mod 8), each XCD with its own L2.  Task index for workgroup b of n such
// that every XCD takes one contiguous range of tasks: neighbouring tiles of a
// front share their panel operands, which then stay in one L2.
__device__ __forceinline__ int xcd_task(int b, int n) {
    const int x = b & 7, q = n >> 3, r = n & 7;
    return x * q + min(x, r) + (b >> 3);
}

inline unsigned int blocks_for(int64_t n, int bs) { return (unsigned int)((n + bs - 1) / bs); }

// ---------------------------------------------------------------------------
// assembly
// ---------------------------------------------------------------------------
// Block per chunk of rows (one system): K's entries in those rows, then max
// |K_ij|, max row sum of |K| and max |K_ij| over the primal block (i, j <
// n_primal), with eight lanes a row, from what the block has just written (still
// in its L2).  A lane has two entries with two products each in flight: bound by
// the trips to memory of lists and of the values they name, in no order (order
// 500k: 13 M entries, 21 M products, 300 us; with one entry and one product in
// flight 400 us, with four entries 430).  The norms in two launches of their own,
// with each entry's row, two source indices and 64-bit list bounds read: 322 us.
constexpr int kAsmAhead = 2, kProdAhead = 2;
__global__ __launch_bounds__(256) void k_assemble(DevPlan d, const RowChunk* __restrict__ chunks,
                                                  const double* __restrict__ W, const double* __restrict__ Sigma,
                                                  const double* __restrict__ J, const double* __restrict__ sys_rho,
                                                  const double* __restrict__ omega, double* K,
                                                  double* __restrict__ partial) {
    const int c = blockIdx.x;
    const RowChunk ch = chunks[c];
    const int tid = threadIdx.x;
    const double rho = sys_rho[ch.sys];
    const int* __restrict__ pa = d.prod_a + ch.prod0;
    const int* __restrict__ pb = d.prod_b + ch.prod0;
    for (int64_t eb = ch.ent0 + tid; eb < ch.ent1; eb += 256 * kAsmAhead) {
        int src[kAsmAhead];
        uint8_t fl[kAsmAhead];
        unsigned int q[kAsmAhead], n[kAsmAhead], most = 0;
#pragma unroll
        for (int u = 0; u < kAsmAhead; ++u) {
            const int64_t e = min(eb + 256 * u, ch.ent1 - 1);
            src[u] = d.src[e];
            fl[u] = d.src_flag[e];
            q[u] = d.prod_ptr[e];
            n[u] = (e + 1 < ch.ent1 ? d.prod_ptr[e + 1] : ch.nprod) - q[u];
        }
        double v[kAsmAhead], acc[kAsmAhead];
#pragma unroll
        for (int u = 0; u < kAsmAhead; ++u) {
            v[u] = src[u] >= 0 ? W[src[u]] : src[u] < -1 ? J[-2 - src[u]] : 0.0;
            acc[u] = 0.0;
            most = max(most, n[u]);
        }
        for (unsigned int k = 0; k < most; k += kProdAhead) {
            int a[kAsmAhead][kProdAhead], b[kAsmAhead][kProdAhead];
#pragma unroll
            for (int u = 0; u < kAsmAhead; ++u)
#pragma unroll
                for (int t = 0; t < kProdAhead; ++t) {
                    const bool in = k + t < n[u];
                    a[u][t] = in ? pa[q[u] + k + t] : -1;
                    b[u][t] = in ? pb[q[u] + k + t] : -1;
                }
            double ja[kAsmAhead][kProdAhead], jb[kAsmAhead][kProdAhead];
#pragma unroll
            for (int u = 0; u < kAsmAhead; ++u)
#pragma unroll
                for (int t = 0; t < kProdAhead; ++t) {
                    ja[u][t] = jb[u][t] = 0.0;
                    if (a[u][t] >= 0) {
                        ja[u][t] = J[a[u][t]];
                        jb[u][t] = J[b[u][t]];
                        if (omega) ja[u][t] *= omega[d.jrow_of[a[u][t]]];
                    }
                }
            // explicit fma: with every Omega_rr = 1 the K1s products (each row r
            // of J weighted by Omega_rr) round exactly like K1's
#pragma unroll
            for (int u = 0; u < kAsmAhead; ++u)
#pragma unroll
                for (int t = 0; t < kProdAhead; ++t)
                    if (k + t < n[u]) acc[u] = fma(ja[u][t], jb[u][t], acc[u]);
        }
#pragma unroll
        for (int u = 0; u < kAsmAhead; ++u) {
            const int64_t e = eb + 256 * u;
            if (e >= ch.ent1) break;
            if (fl[u] & 1) v[u] += Sigma[d.Kj[e]];   // a diagonal entry: its column is its row
            if (n[u] > 0) v[u] += rho * acc[u];
            if (fl[u] & 2) v[u] += -1.0 / rho;
            K[e] = v[u];
        }
    }
    __syncthreads();
    const int sub = tid & 7, grp = tid >> 3;   // 32 row groups of 8 lanes
    const bool all_primal = d.n_primal >= d.N;
    double mx = 0.0, rsmax = 0.0, pmx = 0.0;
    bool bad = false;
    for (int r = grp; r < ch.rows; r += 32) {
        const int row = ch.row0 + r;
        const bool prow = row < d.n_primal;
        double rs = 0.0;
        for (int64_t e = d.Kp[row] + sub; e < d.Kp[row + 1]; e += 8) {
            const double v = K[e];
            bad |= !isfinite(v);
            const double a = fabs(v);
            mx = fmax(mx, a);
            if (prow && (all_primal || d.Kj[e] < d.n_primal)) pmx = fmax(pmx, a);
            rs += a;
        }
        for (int o = 4; o > 0; o >>= 1) rs += __shfl_xor(rs, o, 8);
        rsmax = fmax(rsmax, rs);
    }
    if (bad) { mx = INFINITY; rsmax = INFINITY; pmx = INFINITY; }
    __shared__ double sm[3][256];
    sm[0][tid] = mx;
    sm[1][tid] = rsmax;
    sm[2][tid] = pmx;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) {
            sm[0][tid] = fmax(sm[0][tid], sm[0][tid + o]);
            sm[1][tid] = fmax(sm[1][tid], sm[1][tid + o]);
            sm[2][tid] = fmax(sm[2][tid], sm[2][tid + o]);
        }
        __syncthreads();
    }
    if (tid < 3) partial[3 * (int64_t)c + tid] = sm[tid][0];
}

// Block per (system, column group): reduction over the system's chunks of
// `width` values, in a fixed order (deterministic): a sum for the columns k
// with bit (k mod period) of sum_mask set, a max otherwise.
__global__ __launch_bounds__(256) void k_reduce_partials(const int* __restrict__ sys_chunk_ptr, int width, int period,
                                                         unsigned int sum_mask, const double* __restrict__ partial,
                                                         double* out) {
    const int s = blockIdx.x;
    const int k = blockIdx.y;
    const int tid = threadIdx.x;
    const bool sum = (sum_mask >> (k % period)) & 1u;
    double acc = 0.0;
    for (int c = sys_chunk_ptr[s] + tid; c < sys_chunk_ptr[s + 1]; c += 256) {
        const double v = partial[(int64_t)c * width + k];
        acc = sum ? acc + v : fmax(acc, v);
    }
    __shared__ double sm[256];
    sm[tid] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) sm[tid] = sum ? sm[tid] + sm[tid + o] : fmax(sm[tid], sm[tid + o]);
        __syncthreads();
    }
    if (tid == 0) out[(int64_t)s * width + k] = sm[0];
}

// Block per system: the norms (max |K_ij|, ||K||_inf, max over the primal block)
// from its chunks', then kinf and the two static-pivot thresholds of Sec. 3.1.
// mode 0, global rule: both eps * max |K_ij|.  mode 1, block rule (stabilized
// form): primal pivots eps * max |K_xx|, dual pivots eps / rho, the norm of
// the -1/rho I block of Sec. 3.2, eq. K2r.  mode 2: eps itself for both (the
// pivot epsilon of Sec. 4.3 as an absolute bound).  Non-finite norms set
// kNonfiniteInput.
__global__ __launch_bounds__(256) void k_thresholds(const int* __restrict__ sys_chunk_ptr,
                                                    const double* __restrict__ partial, double eps, int mode,
                                                    const double* __restrict__ sys_rho, double* kinf, double* thr,
                                                    int* nonfinite) {
    const int s = blockIdx.x, tid = threadIdx.x;
    double v[3] = {0.0, 0.0, 0.0};
    for (int c = sys_chunk_ptr[s] + tid; c < sys_chunk_ptr[s + 1]; c += 256)
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = fmax(v[k], partial[3 * (int64_t)c + k]);
    __shared__ double sm[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        for (int o = 32; o > 0; o >>= 1) v[k] = fmax(v[k], __shfl_xor(v[k], o));
        if ((tid & 63) == 0) sm[k][tid >> 6] = v[k];
    }
    __syncthreads();
    if (tid > 0) return;
    double n[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) n[k] = fmax(fmax(sm[k][0], sm[k][1]), fmax(sm[k][2], sm[k][3]));
    const double a = n[0], b = n[1], pm = n[2];
    kinf[s] = b;
    thr[2 * s] = mode == 2 ? eps : (mode == 1 ? pm : a) * eps;
    thr[2 * s + 1] = mode == 2 ? eps : (mode == 1 ? eps / sys_rho[s] : eps * a);
    if (!isfinite(a) || !isfinite(b)) atomicOr(nonfinite, kNonfiniteInput);
}

// ---------------------------------------------------------------------------
// small fronts (order up to kSmallMax)
// ---------------------------------------------------------------------------
// One front by NW waves: one for orders up to 64, four for those up to 128.
// The front's lower 16 x 16 tiles are MFMA accumulators (held transposed, lane
// % 16 = row): the children's contribution blocks are gathered straight into
// them through byte maps (front row -> child row), and what is left in them
// after the last pivot is the front's own contribution block.  Only the pivot
// columns live in LDS (a strip of 16-column sub-panels, leading dimension
// front_ld): K's entries are scattered there, a sub-panel's tiles are added
// when its turn comes, wave 0 eliminates it (wave 1 takes the rows more than
// 64 below its diagonal block), and the other waves apply the previous one
// meanwhile.
// The whole front in LDS, as before, took 128 KB at order 128 (one workgroup a
// CU) and pulled the children one after the other through LDS with two
// barriers each: 36..45 us for a lone front of order 65..128, 20 us for
// one of 33..64 (order 20k).  Bound by latency: about six dependent trips to
// memory, then the pivots (1.2 us per 16).
constexpr int kKidBatch = 4;   // children whose maps are in LDS at a time

// Leading dimension of the strip: 16 mod 32 elements, see kDiagLd.
__host__ __device__ constexpr int front_ld(int nt) { return 16 * (nt | 1); }

// Tile idx of the lower triangle of NT x NT tiles, column by column.
template <int NT>
__device__ __forceinline__ int tile_col(int idx) {
    int c = 0;
#pragma unroll
    for (int j = 1; j < NT; ++j) c += idx >= j * NT - j * (j - 1) / 2;
    return c;
}
template <int NT>
__device__ __forceinline__ int tile_row(int idx) {
    const int c = tile_col<NT>(idx);
    return c + idx - (c * NT - c * (c - 1) / 2);
}

template <int NW>
__device__ __forceinline__ void front_sync() {
    if (NW > 1) __syncthreads();
    else wave_fence();
}

// Waves a SIMD: without a bound the one-wave forms took 281 and 177 registers, one
// and two waves; the launches of orders 33..64 at order 500k 312 us, so 250.
template <typename T, int NT, int NW>
__global__ __launch_bounds__(64 * NW, NW > 1 || NT > 2 ? 2 : 3) void k_front(FrontPlan d, const FrontTask* __restrict__ tasks,
                                                               const double* __restrict__ K, T* __restrict__ F,
                                                               T* __restrict__ D) {
    constexpr int kThreads = 64 * NW, kTiles = NT * (NT + 1) / 2, kSlots = (kTiles + NW - 1) / NW, kRows = 16 * NT;
    constexpr int kE = NW > 1 ? 2 : NT;   // K entries a thread holds from the start
    constexpr int kSigns = NT > 4 ? 2 : 1;
    typedef typename Mfma<T>::acc_t acc_t;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* S = reinterpret_cast<T*>(smem_raw);
    __shared__ T dv[kRows];
    __shared__ __align__(4) uint8_t mrow[kKidBatch][kRows], mcol[kKidBatch][kRows];
    const FrontTask* tk = tasks + blockIdx.x;
    const int first = tk->first, p = tk->p, f = tk->f, nkid = tk->nkid, kid0 = tk->kid0, kn = tk->kn;
    const int nt = (f + 15) >> 4, nq = (p + 15) >> 4, ld = front_ld(nt), rows = 16 * nt;
    const int tid = threadIdx.x, lane = tid & 63, wave = NW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const int lr = lane & 15, lk = lane >> 4;
    const int64_t* __restrict__ kc = d.kent_csr + tk->k0;
    const int* __restrict__ krc = d.kent_rc + tk->k0;
    // K entries: places and values, in flight over the fill of the strip
    int rc[kE];
    T kv[kE];
#pragma unroll
    for (int u = 0; u < kE; ++u) {
        const int e = tid + kThreads * u;
        const int ec = min(e, kn - 1);
        rc[u] = krc[ec];
        kv[u] = (T)K[kc[ec]];
    }
    const PivThr thr(d.sys_thr, tk->sys);
    // the pivots' signs, 64 a word (the last pivot's repeated)
    int8_t sg[kSigns];
#pragma unroll
    for (int u = 0; u < kSigns; ++u) sg[u] = d.piv_sign[first + min(64 * u + lane, p - 1)];
    // the maps of children kid .. kid + kKidBatch - 1; columns in the order in
    // which a lane's accumulator items take them
    auto load_maps = [&](int kid) {
        constexpr int kN = kKidBatch * kRows;
#pragma unroll
        for (int i0 = 0; i0 < kN; i0 += kThreads) {
            const int i = i0 + tid, k = i / kRows, m = i % kRows;
            uint8_t v = 255;
            if (i < kN && kid + k < nkid && m < f) v = d.kid_map[d.kids[kid0 + kid + k].map_off + m];
            if (i < kN) {
                mrow[k][m] = v;
                const int r = m & 15;
                mcol[k][(m & ~15) + (sizeof(T) == 8 ? 4 * (r & 3) + (r >> 2) : r)] = v;
            }
        }
    };
    load_maps(0);
    for (int i = tid; i < ld * 16 * nq; i += kThreads) S[i] = T(0);
    front_sync<NW>();
#pragma unroll
    for (int u = 0; u < kE; ++u)
        if (tid + kThreads * u < kn) S[(rc[u] & 255) + (rc[u] >> 8) * ld] = kv[u];
    for (int e = tid + kThreads * kE; e < kn; e += kThreads) S[(krc[e] & 255) + (krc[e] >> 8) * ld] = (T)K[kc[e]];
    // K's entries come from any thread, and the owner of a tile adds to them below
    front_sync<NW>();
    acc_t acc[kSlots];
#pragma unroll
    for (int t = 0; t < kSlots; ++t) acc[t] = acc_t{0, 0, 0, 0};
    for (int kb = 0; kb < nkid; kb += kKidBatch) {
        if (kb > 0) {
            front_sync<NW>();
            load_maps(kb);
            front_sync<NW>();
        }
        const int kn2 = min(kKidBatch, nkid - kb);
        for (int k = 0; k < kn2; ++k) {
            const KidMap km = d.kids[kid0 + kb + k];
            const T* __restrict__ CB = F + km.CB_off;
            T v[kSlots][4];
            unsigned long long ok = 0;
#pragma unroll
            for (int t = 0; t < kSlots; ++t) {
                const int idx = min(NW * t + wave, kTiles - 1);   // (a slot past the last tile is not used)
                const int a = (int8_t)mrow[k][16 * tile_row<NT>(idx) + lr];   // -1: none
                const unsigned int b4 = *reinterpret_cast<const unsigned int*>(&mcol[k][16 * tile_col<NT>(idx) + 4 * lk]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int b = (int)(b4 >> (8 * r) & 255u);                // 255: none
                    const bool in = a >= b;
                    const unsigned int off = in ? (unsigned int)a + __umul24((unsigned int)b, (unsigned int)km.ld) : 0u;
                    v[t][r] = CB[off];
                    ok |= (unsigned long long)in << (4 * t + r);
                }
            }
#pragma unroll
            for (int t = 0; t < kSlots; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[t][r] += (ok >> (4 * t + r) & 1ULL) ? v[t][r] : T(0);
        }
    }
    unsigned long long negs[kSigns];
#pragma unroll
    for (int u = 0; u < kSigns; ++u) negs[u] = __ballot(sg[u] < 0);
    unsigned int cnt[4] = {0, 0, 0, 0};
    bool bad = false;
#pragma unroll 1
    for (int q = 0; q < nq; ++q) {
        const int kb = 16 * q, bw = min(16, p - kb);
        const unsigned int neg = (unsigned int)(negs[kb < 64 ? 0 : kSigns - 1] >> (kb & 63)) & 0xffffu;
#pragma unroll
        for (int t = 0; t < kSlots; ++t) {
            const int idx = NW * t + wave, ti = tile_row<NT>(idx);
            if (tile_col<NT>(idx) != q || ti >= nt) continue;   // uniform
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = Mfma<T>::row(lk, r);
                if (c < bw) S[(16 * ti + lr) + (kb + c) * ld] += acc[t][r];
            }
        }
        front_sync<NW>();
        const bool two = NT > 4 && kb + 80 < rows;   // rows beyond the 64 that wave 0 takes
        const int row = kb + 16 + 64 * wave + lane, rowc = min(row, rows - 1);
        const bool act = wave == 0 || (wave == 1 && two);
        T rp[16], x[16], dk = T(0);
        bool pk;
        if (act) {
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                rp[t] = S[(kb + lr) + (kb + t) * ld];
                x[t] = S[rowc + (kb + t) * ld];
            }
        }
        if (NW > 1 && two) __syncthreads();   // wave 1 has read the diagonal block that wave 0 overwrites
        if (act) {
            pivots16(rp, x, dk, pk, bw, thr, neg, lr);
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                if (t >= bw) continue;   // uniform: columns past the last pivot stay zero
                if (row < rows) S[row + (kb + t) * ld] = x[t];
                if (wave == 0 && lane < 16) S[(kb + lane) + (kb + t) * ld] = rp[t];
            }
            if (wave == 0) {
                if (lane < 16) dv[kb + lane] = lane < bw ? dk : T(0);
                count_pivots(dk, pk, bw, lane, cnt, bad);
            }
        }
        if (q > 0) {
#pragma unroll
            for (int t = 0; t < kSlots; ++t) {
                const int idx = NW * t + wave, ti = tile_row<NT>(idx), tj = tile_col<NT>(idx);
                if (tj > q && ti < nt) diag_apply<T>(acc[t], S, ld, dv, q - 1, ti, tj, lr, lk);
            }
        }
        front_sync<NW>();
        if (q + 1 < nq) {
#pragma unroll
            for (int t = 0; t < kSlots; ++t) {
                const int idx = NW * t + wave, ti = tile_row<NT>(idx);
                if (tile_col<NT>(idx) == q + 1 && ti < nt) diag_apply<T>(acc[t], S, ld, dv, q, ti, q + 1, lr, lk);
            }
        }
    }
    // the last sub-panel, also on its own block column where that holds columns
    // past the last pivot
    if (f > p) {
        const int tj0 = p >> 4;
        const int64_t ldc = tk->CB_ld;
        T* __restrict__ CB = F + tk->CB_off;
#pragma unroll
        for (int t = 0; t < kSlots; ++t) {
            const int idx = NW * t + wave, ti = tile_row<NT>(idx), tj = tile_col<NT>(idx);
            if (tj < tj0 || ti >= nt) continue;   // uniform
            diag_apply<T>(acc[t], S, ld, dv, nq - 1, ti, tj, lr, lk);
            const int i = 16 * ti + lr;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = 16 * tj + Mfma<T>::row(lk, r);
                if (j >= p && i >= j && i < f) CB[(i - p) + (j - p) * ldc] = acc[t][r];
            }
        }
    }
    if (tid == 0) {
        add_inertia(d.inertia_part, tk->sys, cnt, tk->s);
        if (bad) atomicOr(d.nonfinite, kNonfiniteFactor);
    }
    for (int k = tid; k < p; k += kThreads) D[first + k] = dv[k];
    front_sync<NW>();
    // column j of L from the top of its diagonal block (what is above the diagonal
    // is not used)
    T* __restrict__ L = F + tk->L_off;
    for (int j = wave; j < p; j += NW)
        for (int i = (j & ~15) + lane; i < f; i += 64) L[i + (int64_t)j * f] = S[i + j * ld];
}

// ---------------------------------------------------------------------------
// large fronts (front stored in the factor buffer, ld = f)
// ---------------------------------------------------------------------------
// Orders one wave's accesses to its column: LDS accesses of a wave execute in
// order; global stores must have completed before other lanes read them back.
template <bool kLds>
__device__ __forceinline__ void asm_fence() {
    if (!kLds) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wave_fence();
}

// Reads back an element of the column being built.  In global memory (front
// too large for the LDS slice) the read bypasses the CU's L1, which may hold a
// copy of the line from before the wave's own stores.
template <bool kLds, typename T>
__device__ __forceinline__ T col_read(const T* p) {
    if (kLds) return *p;
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One wave per (large front, column j), four columns per workgroup: assemble
// column j (rows >= j) from K and the children's contribution blocks.  The
// task's column base, K-entry range and contribution segments (one per child
// whose CB maps a column onto j) come precomputed, so the wave starts with
// one round of independent loads.  kLds: the column is built in the wave's
// LDS slice (dynamic, 4 x >= f elements) and written once; otherwise in place.
// A wave's LDS accesses execute in order, so no workgroup barrier is needed;
// children are added one after the other (two may map onto the same row).
template <typename T, bool kLds>
__device__ __forceinline__ void asm_column(const DevPlan& d, int64_t t, const double* __restrict__ K,
                                           T* __restrict__ F, T* slice, int lane) {
    const int64_t colbase = d.asm_col[t];
    const int f = d.asm_fj[2 * t], j = d.asm_fj[2 * t + 1];
    const int64_t e0 = d.asm_kr[2 * t], e1 = d.asm_kr[2 * t + 1];
    const int64_t g0 = d.asm_seg_ptr[t], g1 = d.asm_seg_ptr[t + 1];
    T* __restrict__ Acol = F + colbase;                      // Acol[i] = A[i, j]
    T* __restrict__ cv = kLds ? slice : Acol;
    const int64_t jf = (int64_t)j * f;
    for (int i = j + lane; i < f; i += 64) cv[i] = T(0);
    asm_fence<kLds>();
    for (int64_t e = e0 + lane; e < e1; e += 64) cv[d.kent_pos[e] - jf] = (T)K[d.kent_csr[e]];
    asm_fence<kLds>();
    for (int64_t g = g0; g < g1; ++g) {
        const T* __restrict__ CB = F + d.asm_seg_cb[g];
        const int* __restrict__ r = d.rel + d.asm_seg_rel[g];
        const int b = d.asm_seg_bc[2 * g], cc = d.asm_seg_bc[2 * g + 1];
        for (int a0 = b + lane; a0 < cc; a0 += 64 * 4) {
            T v[4];
            int ri[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int a = min(a0 + 64 * u, cc - 1);
                v[u] = CB[a];
                ri[u] = r[a];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (a0 + 64 * u < cc) cv[ri[u]] = col_read<kLds>(cv + ri[u]) + v[u];
        }
        asm_fence<kLds>();
    }
    if (kLds)
        for (int i = j + lane; i < f; i += 64) Acol[i] = cv[i];
}

template <typename T, bool kLds>
__global__ __launch_bounds__(256) void k_large_asm(DevPlan d, int64_t task0, int count, int fcap,
                                                   const double* __restrict__ K, T* __restrict__ F) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t q = 4 * (int64_t)blockIdx.x + wave;
    if (q >= count) return;
    asm_column<T, kLds>(d, task0 + q, K, F, reinterpret_cast<T*>(smem_raw) + (int64_t)wave * fcap, lane);
}

// Writes the factored diagonal block of a panel (in LDS: L strictly below the
// diagonal, Z = L^-1 transposed strictly above it, dv = pivots) to its
// consumers: D, the front's L
// (strictly lower part of the block), and Zg = Z (column-major, kPanel x
// kPanel, unit diagonal, identity beyond w) for the panel solves and the
// sweeps, with Z^T in its strictly upper triangle.
template <typename T>
__device__ __forceinline__ void publish_diag(T* A, int f, int k0, int w, const T* B, const T* dv, T* D, int first,
                                             T* Zg, int tid) {
    if (tid < w) D[first + k0 + tid] = dv[tid];
#pragma unroll
    for (int it = 0; it < kPanel * kPanel / 256; ++it) {
        const int idx = tid + 256 * it;
        const int u = idx & (kPanel - 1), t = idx / kPanel;   // row u, column t
        if (u < w && t < u) A[(k0 + u) + (int64_t)(k0 + t) * f] = B[u + t * kDiagLd];
        const int lo = max(u, t), hi = min(u, t);
        Zg[idx] = u == t ? T(1) : (lo < w ? B[hi + lo * kDiagLd] : T(0));
    }
}

// C - L_I D_k L_J^T for the 64x64 tile at rows i0, columns j0 of front A
// (ld f), with panel k = columns [k0, k0 + w): four waves, each a 32x32
// quadrant as 2x2 blocks of 16x16 (v_mfma 16x16x4).  The accumulators start
// from C (prefetched with the operands, clamped addresses) and one operand
// is negated, so the result is the updated tile.  Blocks are held transposed
// (lane % 16 = row): C is read and written 16 rows of a column at a time.
// acc[bi][bj][r] holds entry (i0 + wr + 16 bi + lr, j0 + wc + 16 bj + row(lk, r)).
template <typename T>
__device__ __forceinline__ void tile_update(const T* __restrict__ A, int f, int k0, int w, int i0, int j0,
                                            const T* __restrict__ Dk, typename Mfma<T>::acc_t (&acc)[2][2], int tid) {
    const int wave = tid >> 6, lane = tid & 63;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi) {
        const int gi = min(i0 + wr + 16 * bi + lr, f - 1);
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gj = min(j0 + wc + 16 * bj + Mfma<T>::row(lk, r), f - 1);
                acc[bi][bj][r] = A[gi + (int64_t)gj * f];
            }
    }
    constexpr int KS = kPanel / 4;
    T av[KS][2], bv[KS][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int t = 4 * ks + lk;
        const bool tv = t < w;
        const int tc = tv ? t : 0;
        const int64_t cofs = (int64_t)(k0 + tc) * f;
        const T dtr = Dk[tc];
        const T ndt = tv ? -dtr : T(0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ri = i0 + wr + 16 * h + lr, rj = j0 + wc + 16 * h + lr;
            const T a = A[min(ri, f - 1) + cofs], b = A[min(rj, f - 1) + cofs];
            av[ks][h] = (tv && ri < f) ? a : T(0);
            bv[ks][h] = (rj < f) ? b * ndt : T(0);
        }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj) acc[bi][bj] = Mfma<T>::run(bv[ks][bj], av[ks][bi], acc[bi][bj]);
}

// One workgroup per (large front, panel k0): bring the panel's diagonal block
// up to date (for k0 > 0 it applies the previous panel's update to the block
// itself, which the update launch of that panel leaves out, so the two run
// side by side), factor it with the static-pivot rule of Sec. 3.1, count its
// inertia, invert its unit lower triangle and publish L, D and Z = L_kk^-1.
// When the panel is narrower than 64, the block's rows past the last pivot
// belong to the panel rows below it / the contribution block and are written
// back to the front.
template <typename T>
__device__ __forceinline__ void diag_body(const DevPlan& d, const LargeTask* tk, T* F, T* D, T* Zbuf, int tid) {
    const int first = tk->first, p = tk->p, f = tk->f, k0 = tk->k0;
    const int w = min(kPanel, p - k0);
    T* __restrict__ A = F + tk->L_off;
    __shared__ T B[kPanel * kDiagLd];
    __shared__ T dv[kPanel];
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lr = lane & 15, lk = lane >> 4;
    __builtin_amdgcn_s_setprio(3);   // the launch waits for this chain, not for the tiles beside it
    const int8_t sg = lane < w ? d.piv_sign[first + k0 + lane] : 1;
    const PivThr thr(d.sys_thr, tk->sys);
    typename Mfma<T>::acc_t acc[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        if (!diag_has(wave, t)) continue;   // uniform
        const int gi = min(k0 + 16 * diag_ti(wave, t) + lr, f - 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int gj = min(k0 + 16 * diag_tj(wave, t) + Mfma<T>::row(lk, r), f - 1);
            acc[t][r] = A[gi + (int64_t)gj * f];
        }
    }
    if (k0 > 0) {
        // The block's own update by the previous panel (columns kp = k0 - 64
        // .. k0, all 64 wide): its 64 rows of L staged in B.
        const int kp = k0 - kPanel;
        const int nr = min(kPanel, f - k0);
        {
            constexpr int kIt = kPanel * kPanel / 256;   // all loads first, then the LDS stores
            T lv[kIt];
            const T* __restrict__ src = A + min(k0 + lane, f - 1);
#pragma unroll
            for (int it = 0; it < kIt; ++it) lv[it] = src[(int64_t)(kp + 4 * it + wave) * f];
            const T dl = wave == 0 ? D[first + kp + lane] : T(0);
#pragma unroll
            for (int it = 0; it < kIt; ++it) B[lane + (4 * it + wave) * kDiagLd] = lane < nr ? lv[it] : T(0);
            if (wave == 0) dv[lane] = dl;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < 3; ++t)
                if (diag_has(wave, t))
                    diag_apply<T>(acc[t], B, kDiagLd, dv, q, diag_ti(wave, t), diag_tj(wave, t), lr, lk);
        if (w < kPanel) {
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                if (!diag_has(wave, t)) continue;
                const int li = 16 * diag_ti(wave, t) + lr;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int lj = 16 * diag_tj(wave, t) + Mfma<T>::row(lk, r);
                    if (li >= w && li >= lj && li < nr) A[(k0 + li) + (int64_t)(k0 + lj) * f] = acc[t][r];
                }
            }
        }
        __syncthreads();   // the staged rows have been read
    }
    unsigned int cnt[4] = {0, 0, 0, 0};
    bool bad = false;
    diag_factor<T>(acc, B, dv, __ballot(sg < 0), w, thr, cnt, bad, tid);
    if (tid == 0) {
        add_inertia(d.inertia_part, tk->sys, cnt, tk->s + k0);
        if (bad) atomicOr(d.nonfinite, kNonfiniteFactor);
    }
    publish_diag<T>(A, f, k0, w, B, dv, D, first, Zbuf + tk->M_off + (int64_t)(k0 / kPanel) * (kPanel * kPanel), tid);
}

// The first panels' diagonal blocks of a level (later ones run in
// k_large_dstep beside the previous panel's trailing update).
template <typename T>
__global__ __launch_bounds__(256, 2) void k_large_diag(DevPlan d, const LargeTask* __restrict__ tasks, T* __restrict__ F,
                                                    T* __restrict__ D, T* __restrict__ Zbuf) {
    diag_body<T>(d, tasks + blockIdx.x, F, D, Zbuf, threadIdx.x);
}

// One workgroup per (front, panel, 32-row block) below the panel's diagonal
// block: L[i, k0:k1] = A[i, k0:k1] Z^T D^-1 with Z = L_kk^-1 (published by the
// diagonal-block factorization), on MFMA.  The result is also stored
// transposed in the front's upper triangle (never used by the factorization)
// so that the backward solve reads L^T rows contiguously.  Wave w takes rows r0 + 16 (w & 1)
// and the output column blocks J = w >> 1 and 3 - (w >> 1); Z is lower
// triangular, so block J contracts over k < 16 (J + 1) only.
template <typename T>
__device__ __forceinline__ void panel_body(const LargeTask* tk, T* F, const T* D, const T* Zbuf, int tid) {
    const int first = tk->first, p = tk->p, f = tk->f, k0 = tk->k0, r0 = tk->a;
    const int w = min(kPanel, p - k0);
    T* __restrict__ A = F + tk->L_off;
    const T* __restrict__ Zt = Zbuf + tk->M_off + (int64_t)(k0 / kPanel) * (kPanel * kPanel);
    const int wave = tid >> 6, lane = tid & 63;
    const int lr = lane & 15, lk = lane >> 4;
    const int rb = r0 + 16 * (wave & 1);
    const int row = rb + lr;
    const bool rv = row < f;
    T a[4][4];
#pragma unroll
    for (int K = 0; K < 4; ++K)
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            const int kk = 16 * K + Mfma<T>::row(lk, st);
            a[K][st] = (rv && kk < w) ? A[row + (int64_t)(k0 + kk) * f] : T(0);
        }
    typedef typename Mfma<T>::acc_t acc_t;
    // Z operands of both output blocks (blocks K <= J only: Z is lower
    // triangular), loaded before the MFMA chains
    T zo[2][4][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int J = h ? 3 - (wave >> 1) : (wave >> 1);
#pragma unroll
        for (int K = 0; K < 4; ++K) {
            if (K > J) continue;   // uniform
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const T z = Zt[(16 * K + Mfma<T>::row(lk, st)) * kPanel + 16 * J + lr];
                zo[h][K][st] = K < J || Mfma<T>::row(lk, st) <= lr ? z : T(0);   // Z^T lies above the diagonal
            }
        }
    }
    // The results overwrite A[rows, panel] in place, and the two waves that
    // share a row block each read all of its panel columns but write only
    // their own output blocks: every wave's loads must have returned before
    // any wave stores.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int J = h ? 3 - (wave >> 1) : (wave >> 1);
        acc_t acc = {0, 0, 0, 0};
#pragma unroll
        for (int K = 0; K < 4; ++K) {
            if (K > J) continue;   // uniform
#pragma unroll
            for (int st = 0; st < 4; ++st) acc = Mfma<T>::run(a[K][st], zo[h][K][st], acc);
        }
        const int col = 16 * J + lr;
        if (col < w) {
            const T dinv = T(1) / D[first + k0 + col];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gi = rb + Mfma<T>::row(lk, r);
                if (gi < f) {
                    const T x = acc[r] * dinv;
                    A[gi + (int64_t)(k0 + col) * f] = x;
                    A[(k0 + col) + (int64_t)gi * f] = x;   // L^T in the unused upper triangle
                }
            }
        }
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_large_panel(const LargeTask* __restrict__ tasks, T* __restrict__ F,
                                                     const T* __restrict__ D, const T* __restrict__ Zbuf) {
    panel_body<T>(tasks + blockIdx.x, F, D, Zbuf, threadIdx.x);
}

// Trailing update of one 64x64 lower tile: C -= L_I D_k L_J^T on MFMA, with
// the operands read straight from the front (no LDS).  The next panel's
// diagonal tile is not in the task list: its diagonal-block workgroup updates it.
template <typename T>
__device__ __forceinline__ void update_body(const LargeTask* tk, T* F, const T* D, int tid) {
    const int first = tk->first, p = tk->p, f = tk->f, k0 = tk->k0, i0 = tk->a, j0 = tk->b;
    const int w = min(kPanel, p - k0);
    T* __restrict__ A = F + tk->L_off;
    typename Mfma<T>::acc_t acc[2][2];
    tile_update<T>(A, f, k0, w, i0, j0, D + first + k0, acc, tid);
    const int wave = tid >> 6, lane = tid & 63;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gi = i0 + wr + bi * 16 + lr, gj = j0 + wc + bj * 16 + Mfma<T>::row(lk, r);
                if (gi < f && gj < f && gi >= gj) A[gi + (int64_t)gj * f] = acc[bi][bj][r];
            }
}

// Panel k's trailing update and panel k+1's diagonal blocks in one launch
// (they touch disjoint tiles): the first nd workgroups factor the diagonal
// blocks (their own update read from the front, like a tile), workgroups from nd8 = nd rounded up to a
// multiple of 8 take the update tiles with the XCD-contiguous mapping.
template <typename T>
__global__ __launch_bounds__(256, 2) void k_large_dstep(DevPlan d, const LargeTask* __restrict__ dtasks, int nd,
                                                     const LargeTask* __restrict__ utasks, int nu, T* __restrict__ F,
                                                     T* __restrict__ D, T* __restrict__ Zbuf) {
    const int nd8 = (nd + 7) & ~7;
    const int b = blockIdx.x;
    if (b < nd) diag_body<T>(d, dtasks + b, F, D, Zbuf, threadIdx.x);
    else if (b >= nd8) update_body<T>(utasks + xcd_task(b - nd8, nu), F, D, threadIdx.x);
}

// ---------------------------------------------------------------------------
// solves
// ---------------------------------------------------------------------------
// Vectors in pivot order: one value a row for one right-hand side, kNrhsMax
// (unused columns zero) for several, so that a row's columns are
// contiguous and a 16-row, 16-column piece is one MFMA operand.
//   Y   the right-hand side, updated in place for rows not yet solved
//   Y2  the pivots' y after the forward sweep
//   X   the pivots' x after the backward sweep
//   U   the fronts' update vectors (rows below the pivots)
// B: column q of row i at B[i si + q sq].
template <typename T, int LD>
__global__ void k_permute_in(DevPlan d, const double* __restrict__ B, int64_t si, int64_t sq, int nrhs,
                             T* __restrict__ Y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t k = i / LD;
    const int q = (int)(i % LD);
    if (k >= d.N) return;
    Y[i] = q < nrhs ? (T)B[d.perm[k] * si + q * sq] : T(0);
}

template <typename T, int LD>
__global__ void k_permute_out(DevPlan d, const T* __restrict__ X, int nrhs, double* __restrict__ Xo, int64_t ldx) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t k = i / LD;
    const int q = (int)(i % LD);
    if (k >= d.N || q >= nrhs) return;
    Xo[d.perm[k] + q * ldx] = to_d(X[i]);
}

// One launch per step of a level holds the tasks of its large fronts (one
// workgroup each) and, in the level's first step, its small fronts (one wave
// each, or a workgroup each in a backward step of few).  A large front's panels are taken two at a time, columns
// [c0, c0 + w1) and [c0 + w1, c0 + w1 + w2) (w1 = 64 when w2 > 0), through
//   G1, G2  the inverses Z = L_kk^-1 of their diagonal blocks (unit lower,
//           with Z^T in the strictly upper triangle) and
//   L21     the second panel's rows of the first:
//   forward:  y1 = Z1 b1, y2 = Z2 (b2 - L21 y1), rows below -= L1 y1 + L2 y2
//   backward: v = y / d - L^T x (rows below), x2 = Z2^T v2, x1 = Z1^T (v1 - L21^T x2)
// (Through the inverse of the pair's whole triangle, with P = -Z2 L21 Z1 formed after
// the factorization, every result was one product with what the launch starts from:
// a solve of one column at order 500k 1332 us, so 1385, a factorization 5685, so 5652.
// But its rounding was 1.1 times as large for one column and 1.3 to 1.45 times for
// several, FP32 fronts of order 320 and 576.)
// The rows below are split into tasks of 64.
//   forward:  every task forms the pair's y itself; task 0 stores it.
//   backward: a pair with one task is finished by it.  The tasks of any other
//     leave their sums in pw (slot0 + task), and the next launch on the stream
//     finishes it: the front's previous pair's tasks 0 and 1, whose rows begin
//     with the two panels, or, for a front's first pair, two records of their
//     own after the level's last step.  No task waits for another of its launch.
// Children's update vectors come through a table: row i of the front takes
// U[gat[k f + i]], k = 0 .. gk - 1 in the children's order (-1: none), and then,
// where rows have more (deep), those of its list, see Plan::gather.
// The sweeps are bound by the latency of their chain of launches; panel by
// panel, with the one-wave fronts forked to a second stream, a forward step
// took 10 us, a backward one 6 and the fork and join 9 (order 20k).

// Values of a pair's pivots and of the task's rows before the step.
template <typename T>
__device__ __forceinline__ T gather1(const T* __restrict__ U, const int* __restrict__ gat, int f, int gk, bool deep,
                                    int i, T v) {
    for (int k0 = 0; k0 < gk; k0 += 4) {
        int o[4];
        T u[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = k0 + k < gk ? gat[(int64_t)(k0 + k) * f + i] : -1;
#pragma unroll
        for (int k = 0; k < 4; ++k) u[k] = U[max(o[k], 0)];
#pragma unroll
        for (int k = 0; k < 4; ++k) v += o[k] >= 0 ? u[k] : T(0);
    }
    if (deep) {   // uniform
        const int* __restrict__ start = gat + (int64_t)gk * f;
        const int* __restrict__ list = start + f + 1;
        const int q1 = start[i + 1];
        for (int q = start[i]; q < q1; q += 8) {
            T u[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) u[k] = U[list[min(q + k, q1 - 1)]];
#pragma unroll
            for (int k = 0; k < 8; ++k) v += q + k < q1 ? u[k] : T(0);
        }
    }
    return v;
}

// ---- one right-hand side ----------------------------------------------------
// The waves' shares of a 64-vector: wave q4's entry `lane` at part[64 q4 + lane].
template <typename T>
__device__ __forceinline__ T share_sum(const T* part, int lane) {
    return (part[lane] + part[64 + lane]) + (part[128 + lane] + part[192 + lane]);
}
// A wave's copy of a vector whose entry `lane` is x, for its reads of 16 entries
// (xw: 64 values of its own; its LDS accesses are in order).
template <typename T>
__device__ __forceinline__ const T* wave_copy(T* xw, T x, int lane) {
    wave_fence();
    xw[lane] = x;
    wave_fence();
    return xw;
}
template <typename T>
__device__ __forceinline__ T dot16(const T (&a)[16], const T* x) {
    T s = T(0);
#pragma unroll
    for (int j = 0; j < 16; ++j) s += a[j] * x[j];
    return s;
}

// A wave holds 16 columns of every operand; each product's four shares meet in LDS
// and every wave sums them for itself, so a product costs one barrier.
template <typename T>
__device__ __forceinline__ void fwd_panels1(const PanelTask* tk, const T* __restrict__ F, const T* __restrict__ Zbuf,
                                            const int* __restrict__ gatab, T* __restrict__ Y, T* __restrict__ Y2,
                                            T* __restrict__ U) {
    __shared__ T v[128], rw[64], part[2][256], xw[4][64];
    const int first = tk->first, p = tk->p, f = tk->f, c0 = tk->c0, w1 = tk->w1, w2 = tk->w2;
    const int r0 = tk->r0, nr = tk->r1 - r0;
    const int tid = threadIdx.x, lane = tid & 63, q4 = tid >> 6;
    const T* __restrict__ L = F + tk->L_off;
    const T* __restrict__ G1 = Zbuf + tk->M_off + (int64_t)(c0 / kPanel) * (kPanel * kPanel);
    const T* __restrict__ G2 = G1 + kPanel * kPanel;
    T* __restrict__ Us = U + tk->U_off;
    // right-hand side: the pair's pivots, then the task's rows
    if (tid < 192) {
        const int gi = tid < 128 ? c0 + tid : r0 + tid - 128;
        const bool in = tid < 128 ? tid < w1 + w2 : tid - 128 < nr;
        T b = T(0);
        if (in) {
            if (gi < p) b = Y[first + gi];
            else if (c0 > 0) b = Us[gi - p];
            if (tk->gk > 0) b = gather1(U, gatab + tk->gat, f, tk->gk, tk->deep != 0, gi, b);
        }
        (tid < 128 ? v[tid] : rw[tid - 128]) = b;
    }
    T z1[16], z2[16], lb[16], l1[16], l2[16];
    const bool rv = lane < nr;
    const T* __restrict__ Lr = L + r0 + (rv ? lane : 0);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int k = 16 * q4 + j;
        z1[j] = G1[k * kPanel + lane];
        l1[j] = (rv && k < w1) ? Lr[(int64_t)(c0 + k) * f] : T(0);
    }
    if (w2 > 0) {
        const T* __restrict__ L21 = L + c0 + kPanel + min(lane, w2 - 1);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int k = 16 * q4 + j;
            lb[j] = L21[(int64_t)(c0 + k) * f];
            z2[j] = G2[k * kPanel + lane];
            l2[j] = (rv && k < w2) ? Lr[(int64_t)(c0 + kPanel + k) * f] : T(0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) z1[j] = 16 * q4 + j <= lane ? z1[j] : T(0);   // Z^T lies above
    part[0][tid] = dot16(z1, v + 16 * q4);
    __syncthreads();
    const T y1 = share_sum(part[0], lane);   // (zero beyond w1)
    if (tid < w1 && tk->index == 0) Y2[first + c0 + tid] = y1;
    const T* x = wave_copy(xw[q4], y1, lane) + 16 * q4;
    T a = dot16(l1, x);
    if (w2 > 0) {
        part[1][tid] = dot16(lb, x);
        __syncthreads();
        const T b2 = lane < w2 ? v[64 + lane] - share_sum(part[1], lane) : T(0);
        x = wave_copy(xw[q4], b2, lane) + 16 * q4;
#pragma unroll
        for (int j = 0; j < 16; ++j) z2[j] = 16 * q4 + j <= lane ? z2[j] : T(0);
        part[0][tid] = dot16(z2, x);
        __syncthreads();
        const T y2 = share_sum(part[0], lane);
        if (tid < w2 && tk->index == 0) Y2[first + c0 + kPanel + tid] = y2;
        x = wave_copy(xw[q4], y2, lane) + 16 * q4;
        a += dot16(l2, x);
    }
    if (nr == 0) return;   // the whole workgroup
    part[1][tid] = a;
    __syncthreads();
    if (tid < nr) {
        const T val = rw[tid] - share_sum(part[1], tid);
        const int gi = r0 + tid;
        if (gi < p) Y[first + gi] = val;
        else Us[gi - p] = val;
    }
}

// A small front by one wave: lane = row and (kHi: order above 64) row + 64; column by column, the
// pivot's y (readlane) times its column of L.
template <typename T, bool kHi>
__device__ __forceinline__ void fwd_front1(const SmallTask* tk, const T* __restrict__ F, const int* __restrict__ gatab,
                                           const T* __restrict__ Y, T* __restrict__ Y2, T* __restrict__ U, int lane) {
    const int first = tk->first, p = tk->p, f = tk->f, gk = tk->gk;
    const T* __restrict__ L = F + tk->L_off;
    T* __restrict__ Us = U + tk->U_off;
    const int* __restrict__ gat = gatab + tk->gat;
    const int i0 = min(lane, f - 1), i1 = min(lane + 64, f - 1);
    constexpr int kC = 16;
    T l0[kC], l1[kC];
    auto load = [&](int kb) {
#pragma unroll
        for (int t = 0; t < kC; ++t) {
            const T* __restrict__ c = L + (int64_t)min(kb + t, p - 1) * f;
            l0[t] = c[i0];
            if (kHi) l1[t] = c[i1];
        }
    };
    load(0);
    T v0 = lane < p ? Y[first + lane] : T(0);
    T v1 = kHi && lane + 64 < p ? Y[first + lane + 64] : T(0);
    if (gk > 0) {
        v0 = gather1(U, gat, f, gk, tk->deep != 0, i0, v0);
        if (kHi) v1 = gather1(U, gat, f, gk, tk->deep != 0, i1, v1);
    }
    for (int kb = 0; kb < p; kb += kC) {
        if (kb > 0) load(kb);
        // rows below the sub-panel sum its products from zero
        const bool own0 = lane < kb + kC, own1 = lane + 64 < kb + kC;
        T w0 = own0 ? v0 : T(0), w1 = own1 ? v1 : T(0);
#pragma unroll
        for (int t = 0; t < kC; ++t) {
            const int k = kb + t;
            if (k >= p) continue;   // uniform
            const T yk = !kHi || k < 64 ? bcast(w0, k) : bcast(w1, k - 64);
            w0 -= (lane > k ? l0[t] : T(0)) * yk;
            if (kHi) w1 -= (lane + 64 > k ? l1[t] : T(0)) * yk;
        }
        v0 = own0 ? w0 : v0 + w0;
        if (kHi) v1 = own1 ? w1 : v1 + w1;
    }
    if (lane < p) Y2[first + lane] = v0;
    else if (lane < f) Us[lane - p] = v0;
    if (kHi) {
        if (lane + 64 < p) Y2[first + lane + 64] = v1;
        else if (lane + 64 < f) Us[lane + 64 - p] = v1;
    }
}

// np panel tasks, one workgroup each, then ns small fronts, four a workgroup.
template <typename T, bool kPanels>
__global__ __launch_bounds__(256, kPanels ? 2 : 4) void k_fwd1(const PanelTask* __restrict__ pt, int np,
                                                 const SmallTask* __restrict__ st, int ns, const int* __restrict__ gat,
                                                 const T* __restrict__ F, const T* __restrict__ Zbuf,
                                                 T* __restrict__ Y, T* __restrict__ Y2, T* __restrict__ U) {
    const int b = blockIdx.x;
    if (kPanels && b < np) {
        fwd_panels1<T>(pt + b, F, Zbuf, gat, Y, Y2, U);
    } else {
        const int t = 4 * (b - np) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        if (t >= ns) return;
        if (st[t].f > 64) fwd_front1<T, true>(st + t, F, gat, Y, Y2, U, threadIdx.x & 63);
        else fwd_front1<T, false>(st + t, F, gat, Y, Y2, U, threadIdx.x & 63);
    }
}

// A pair's x from v = y / d - sums (v: 128 in LDS, zero beyond its columns): x2 =
// Z2^T v2, then, with `one`, x1 = Z1^T (v1 - L21^T x2).  Wave q4 takes rows 16 q4 ..
// of each product; entry `lane` of x1 and x2 in every wave.
template <typename T>
struct PairOps {
    T z1[16], z2[16], lb[16];
    // A: the front; (c0, w2): the pair's first column and its second panel's width
    __device__ __forceinline__ void load(const T* __restrict__ G1, const T* __restrict__ A, int f, int c0, int w2,
                                         bool one, int lane, int q4) {
        const T* __restrict__ G2 = G1 + kPanel * kPanel;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int u = 16 * q4 + j;
            z1[j] = one && u >= lane ? G1[u * kPanel + lane] : T(0);   // Z^T is upper
            z2[j] = w2 > 0 && u >= lane ? G2[u * kPanel + lane] : T(0);
            lb[j] = one && u < w2 ? A[c0 + lane + (int64_t)(c0 + kPanel + u) * f] : T(0);   // L^T lies above
        }
    }
    // part: 2 x 256, xw: the wave's 64
    __device__ __forceinline__ void apply(const T* v, bool two, bool one, T (*part)[256], T* xw, int lane, int q4,
                                          T& x1, T& x2) const {
        const int tid = 64 * q4 + lane;
        T v1 = v[lane];
        x2 = T(0);
        if (two) {
            part[0][tid] = dot16(z2, v + 64 + 16 * q4);
            __syncthreads();
            x2 = share_sum(part[0], lane);
            if (!one) return;
            part[1][tid] = dot16(lb, wave_copy(xw, x2, lane) + 16 * q4);
            __syncthreads();
            v1 -= share_sum(part[1], lane);
        }
        part[0][tid] = dot16(z1, wave_copy(xw, v1, lane) + 16 * q4);
        __syncthreads();
        x1 = share_sum(part[0], lane);
    }
};

template <typename T>
__device__ __forceinline__ void bwd_panels1(const PanelTask* tk, const int* __restrict__ rows, const T* __restrict__ F,
                                            const T* __restrict__ Zbuf, const T* __restrict__ D,
                                            const T* __restrict__ Y2, T* __restrict__ X, T* __restrict__ pw,
                                            const T* __restrict__ pr) {
    __shared__ T v[128], xs[64], part[2][256], xw[4][64];
    const int first = tk->first, p = tk->p, f = tk->f, c0 = tk->c0, w = tk->w1 + tk->w2;
    const int r0 = tk->r0, nr = tk->r1 - r0;
    const int tid = threadIdx.x, lane = tid & 63, q4 = tid >> 6;
    const bool own = tk->index >= 0;                 // else a finish-only record
    const bool fin = tk->fntask > 0, self = own && tk->ntask == 1;
    const int xc0 = fin ? tk->fc0 : c0, xw1 = fin ? tk->fw1 : tk->w1, xw2 = fin ? tk->fw2 : tk->w2;
    const int which = fin ? tk->which : 0;           // the panel it finishes
    const T* __restrict__ A = F + tk->L_off;
    // L^T operands (a large front keeps L^T above its diagonal): one panel: 64
    // columns in four groups of 16 rows, two: 128 in two of 32
    const bool two = tk->w2 > 0;
    const int cols = two ? 128 : 64, col = tid & (cols - 1), rg = tid / cols, nrg = two ? 2 : 4, rpg = 64 / nrg;
    T lv[32];
    {
        const bool cv = own && col < w;
        const T* __restrict__ src = A + c0 + (cv ? col : 0) + (int64_t)(r0 + rpg * rg) * f;
        const int n = cv ? nr - rpg * rg : 0;
#pragma unroll
        for (int m = 0; m < 16; ++m) lv[m] = m < n ? src[(int64_t)m * f] : T(0);
        if (two)
#pragma unroll
            for (int m = 16; m < 32; ++m) lv[m] = m < n ? src[(int64_t)m * f] : T(0);
    }
    PairOps<T> ops;
    if (fin || self)
        ops.load(Zbuf + tk->M_off + (int64_t)(xc0 / kPanel) * (kPanel * kPanel), A, f, xc0, xw2, which == 0, lane, q4);
    T yd = T(0);   // y / d of the pair to finish
    if (tid < xw1 + xw2 && (fin || self)) yd = Y2[first + xc0 + tid] * (T(1) / D[first + xc0 + tid]);
    if (own && tid < 64) {
        const int gi = r0 + tid;
        xs[tid] = tid >= nr ? T(0) : X[gi < p ? first + gi : rows[tk->rows_off + gi]];
    }
    if (fin) {
        // the sums of the pair's tasks: column tid & 127, tasks of one parity
        const int c = tid & 127, g1 = tid >> 7;
        T a = T(0);
        const T* __restrict__ src = pr + (int64_t)tk->fslot0 * 128 + c;
        for (int g0 = g1; g0 < tk->fntask; g0 += 16) {
            T u[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) u[k] = g0 + 2 * k < tk->fntask ? src[(int64_t)(g0 + 2 * k) * 128] : T(0);
#pragma unroll
            for (int k = 0; k < 8; ++k) a += u[k];
        }
        part[0][tid] = a;
        __syncthreads();
        if (tid < 128) v[tid] = tid < xw1 + xw2 ? yd - (part[0][tid] + part[0][tid + 128]) : T(0);
        __syncthreads();
        T x1, x2;
        ops.apply(v, xw2 > 0, which == 0, part, xw[q4], lane, q4, x1, x2);
        if (tid < (which ? xw2 : xw1)) {
            const T x = which ? x2 : x1;
            const int gi = xc0 + 64 * which + tid;
            X[first + gi] = x;
            if (own) xs[gi - r0] = x;
        }
    }
    if (!own) return;   // the whole workgroup
    __syncthreads();
    {
        const T* xr = xs + rpg * rg;
        T a = T(0), b = T(0);
#pragma unroll
        for (int m = 0; m < 16; ++m) a += lv[m] * xr[m];
        if (two)
#pragma unroll
            for (int m = 16; m < 32; ++m) b += lv[m] * xr[m];
        part[1][tid] = a + b;
    }
    __syncthreads();
    if (tid < 128) {
        const T* pp = part[1] + tid;
        const T s = tid >= cols ? T(0) : two ? pp[0] + pp[128] : (pp[0] + pp[64]) + (pp[128] + pp[192]);
        if (self) v[tid] = tid < w ? yd - s : T(0);
        else if (tid < cols) pw[(int64_t)(tk->slot0 + tk->index) * 128 + tid] = s;
    }
    if (!self) return;
    __syncthreads();
    T x1, x2;
    ops.apply(v, two, true, part, xw[q4], lane, q4, x1, x2);
    if (tid < tk->w1) X[first + c0 + tid] = x1;
    if (tid < tk->w2) X[first + c0 + kPanel + tid] = x2;
}

// A small front by one wave, its 16-column sub-panels from the last: lane =
// (column, row group g of four); the groups' sums meet by lane exchange, then
// the sub-panel's transposed triangle is substituted within each 16-lane row.
// A sub-panel's operands are loaded before the one after it is finished, the
// first ones before x is gathered.  Each load takes pieces of 16 columns, 16 lines
// of the cache, so rows and columns past the front are skipped, not clamped: with
// 31 loads a sub-panel whatever its size the lowest levels of order 500k took 42 us a
// launch, so 22.
template <typename T>
__device__ __forceinline__ void bwd_front1(const SmallTask* tk, const int* __restrict__ rows, const T* __restrict__ F,
                                           const T* __restrict__ D, const T* __restrict__ Y2, T* __restrict__ X,
                                           T* xs, int lane) {
    const int first = tk->first, p = tk->p, f = tk->f;
    const T* __restrict__ L = F + tk->L_off;
    const int t = lane & 15, g = lane >> 4;
    T l[16], z[16], yd;   // rows base + 4 m + g below the sub-panel; its own triangle; y / d
    auto load = [&](int kb) {
        const int bw = min(16, p - kb), c = kb + min(t, bw - 1), base = kb + bw;
        const T* __restrict__ Lc = L + (int64_t)c * f;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            l[m] = T(0);
            if (base + 4 * m < f) l[m] = Lc[min(base + 4 * m + g, f - 1)];   // uniform
        }
#pragma unroll
        for (int u = 1; u < 16; ++u) {
            z[u] = T(0);
            if (u < bw) z[u] = Lc[kb + u];   // uniform; masked where it is used
        }
        yd = Y2[first + c] * (T(1) / D[first + c]);
    };
    int kb = (p - 1) & ~15;
    load(kb);
    for (int i = p + lane; i < f; i += 64) xs[i] = X[rows[tk->rows_off + i]];
    wave_fence();
    for (; kb >= 0; kb -= 16) {
        const int bw = min(16, p - kb), base = kb + bw;
        T acc = T(0);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int i = base + 4 * m + g;
            if (base + 4 * m < f) acc += i < f ? l[m] * xs[min(i, kSmallMax - 1)] : T(0);   // uniform
        }
        if (base + 64 < f) {   // uniform: orders above 64
            const T* __restrict__ Lc = L + (int64_t)(kb + min(t, bw - 1)) * f;
            T h[16];
#pragma unroll
            for (int m = 0; m < 16; ++m) h[m] = Lc[min(base + 64 + 4 * m + g, f - 1)];
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                const int i = base + 64 + 4 * m + g;
                acc += i < f ? h[m] * xs[min(i, kSmallMax - 1)] : T(0);
            }
        }
        acc += __shfl_xor(acc, 16);
        acc += __shfl_xor(acc, 32);
        T x = yd - acc;
#pragma unroll
        for (int u = 15; u > 0; --u) x -= (u > t ? z[u] : T(0)) * rowbcast_n(x, u);
        if (kb > 0) load(kb - 16);
        if (lane < bw) {
            xs[kb + lane] = x;
            X[first + kb + lane] = x;
        }
        wave_fence();
    }
}

// The same by the four waves of a workgroup, where fronts are few: sub-panels w
// and w + 4 belong to wave w, which loads all it needs of them at once; the rows
// below the pivots are summed before the first is solved, and each solved
// sub-panel's x is added to the sums above it by their waves.  One wave's loads,
// a sub-panel at a time, were the chain: 8 to 14 us a launch of lone fronts of
// order 65..128 (order 625), so 3.0 to 5.7.
template <typename T>
__device__ __forceinline__ void bwd_front1_wg(const SmallTask* tk, const int* __restrict__ rows,
                                              const T* __restrict__ F, const T* __restrict__ D,
                                              const T* __restrict__ Y2, T* __restrict__ X, T* xs, int tid) {
    constexpr int kBlocks = kSmallMax / 16;
    static_assert(kBlocks == 8, "two sub-panels a wave");
    const int first = tk->first, p = tk->p, f = tk->f, nq = (p + 15) >> 4, nb = (f + 15) >> 4;
    const T* __restrict__ L = F + tk->L_off;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, t = lane & 15, g = lane >> 4;
    T l[2][kBlocks][4], z[2][16], yd[2], acc[2];   // l: rows 16 b + 4 m + g of column t
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int q = wave + 4 * s, kb = 16 * q, bw = min(16, p - kb);
        acc[s] = yd[s] = T(0);
        if (q >= nq) continue;   // uniform
        const int c = kb + min(t, bw - 1);
        const T* __restrict__ Lc = L + (int64_t)c * f;
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            if (b < q || b >= nb) continue;   // uniform
#pragma unroll
            for (int m = 0; m < 4; ++m) l[s][b][m] = Lc[min(16 * b + 4 * m + g, f - 1)];
        }
#pragma unroll
        for (int u = 1; u < 16; ++u) z[s][u] = Lc[kb + min(u, bw - 1)];
        yd[s] = Y2[first + c];
        acc[s] = D[first + c];
    }
    if (tid >= p && tid < f) xs[tid] = X[rows[tk->rows_off + tid]];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int q = wave + 4 * s, bw = min(16, p - 16 * q);
        if (q >= nq) continue;
        yd[s] *= T(1) / acc[s];
        acc[s] = T(0);
#pragma unroll
        for (int u = 1; u < 16; ++u) z[s][u] = u > t && u < bw ? z[s][u] : T(0);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int q = wave + 4 * s;
        if (q >= nq) continue;
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            if (b < nq - 1 || b >= nb) continue;   // uniform
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int i = 16 * b + 4 * m + g;
                acc[s] += i >= p && i < f ? l[s][b][m] * xs[i] : T(0);
            }
        }
    }
#pragma unroll
    for (int q = kBlocks - 1; q >= 0; --q) {
        if (q >= nq) continue;   // uniform over the workgroup
        const int kb = 16 * q, bw = min(16, p - kb);
        if (wave == (q & 3)) {
            T a = acc[q >> 2];
            a += __shfl_xor(a, 16);
            a += __shfl_xor(a, 32);
            T x = yd[q >> 2] - a;
#pragma unroll
            for (int u = 15; u > 0; --u) x -= z[q >> 2][u] * rowbcast_n(x, u);
            if (lane < bw) {
                xs[kb + lane] = x;
                X[first + kb + lane] = x;
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (wave + 4 * s >= q) continue;   // uniform
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int i = kb + 4 * m + g;
                acc[s] += i < p ? l[s][q][m] * xs[i] : T(0);
            }
        }
    }
}

template <typename T, bool kPanels, bool kWg>
__global__ __launch_bounds__(256, kPanels || kWg ? 2 : 4) void k_bwd1(const PanelTask* __restrict__ pt, int np,
                                                 const SmallTask* __restrict__ st, int ns, const int* __restrict__ rows,
                                                 const T* __restrict__ F, const T* __restrict__ Zbuf,
                                                 const T* __restrict__ D, const T* __restrict__ Y2, T* __restrict__ X,
                                                 T* __restrict__ pw, const T* __restrict__ pr) {
    const int b = blockIdx.x;
    if (kPanels && b < np) {
        bwd_panels1<T>(pt + b, rows, F, Zbuf, D, Y2, X, pw, pr);
        return;
    }
    __shared__ T xs[kWg ? 1 : 4][kSmallMax];
    if (kWg) {
        bwd_front1_wg<T>(st + (b - np), rows, F, D, Y2, X, xs[0], threadIdx.x);
    } else {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), t = 4 * (b - np) + wave;
        if (t < ns) bwd_front1<T>(st + t, rows, F, D, Y2, X, xs[wave], threadIdx.x & 63);
    }
}

// ---- several right-hand sides (up to kNrhsMax, on MFMA) ----------------------
// A 16-row piece of a vector is one accumulator: item r of a lane is row
// row(lk, r), column lr.  Such a piece is also the second operand of a product
// whose contraction takes rows row(lk, st) in step st.
template <typename T>
__device__ __forceinline__ typename Mfma<T>::acc_t rows16(const T* V, int lr, int lk) {   // V: row-major, 16 a row
    typename Mfma<T>::acc_t a;
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = V[Mfma<T>::row(lk, r) * kNrhsMax + lr];
    return a;
}

// 16 rows of a product with a 64 x 16 piece V: op[kk][st] the lane's operands for
// rows 16 kk + row(lk, st) of V.  Four chains from zero, one per 16 rows, as the sums
// of one column are taken.
template <typename T>
__device__ __forceinline__ typename Mfma<T>::acc_t product16(const T (&op)[4][4], const T* V, int lr, int lk) {
    typename Mfma<T>::acc_t c[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const typename Mfma<T>::acc_t b = rows16<T>(V + 16 * kk * kNrhsMax, lr, lk);
        c[kk] = typename Mfma<T>::acc_t{0, 0, 0, 0};
#pragma unroll
        for (int st = 0; st < 4; ++st) c[kk] = Mfma<T>::run(op[kk][st], b[st], c[kk]);
    }
    return (c[0] + c[1]) + (c[2] + c[3]);
}

// Adds the children's update vectors to rows i0 .. i0 + 15 (those < iend) of a
// front; row(r): the row of item r, from i0.
template <typename T, typename Row>
__device__ __forceinline__ void gather16(typename Mfma<T>::acc_t& a, const T* __restrict__ U,
                                         const int* __restrict__ gat, int f, int gk, bool deep, int i0, int iend,
                                         int lr, Row row) {
    for (int k = 0; k < gk; ++k) {
        int o[4];
        T u[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = i0 + row(r);
            o[r] = i < iend ? gat[(int64_t)k * f + i] : -1;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) u[r] = U[(int64_t)max(o[r], 0) * kNrhsMax + lr];
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] += o[r] >= 0 ? u[r] : T(0);
    }
    if (deep) {   // uniform
        const int* __restrict__ start = gat + (int64_t)gk * f;
        const int* __restrict__ list = start + f + 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = i0 + row(r);
            if (i >= iend) continue;
            const int q1 = start[i + 1];
            for (int q = start[i]; q < q1; q += 8) {
                T u[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] = U[(int64_t)list[min(q + k, q1 - 1)] * kNrhsMax + lr];
#pragma unroll
                for (int k = 0; k < 8; ++k) a[r] += q + k < q1 ? u[k] : T(0);
            }
        }
    }
}

template <typename T>
__device__ __forceinline__ void fwd_panels16(const PanelTask* tk, const T* __restrict__ F, const T* __restrict__ Zbuf,
                                             const int* __restrict__ gatab, T* __restrict__ Y, T* __restrict__ Y2,
                                             T* __restrict__ U) {
    typedef typename Mfma<T>::acc_t acc_t;
    __shared__ T b[128 * kNrhsMax], y[128 * kNrhsMax];
    const int first = tk->first, p = tk->p, f = tk->f, c0 = tk->c0, w1 = tk->w1, w2 = tk->w2, w = w1 + w2;
    const int r0 = tk->r0, r1 = tk->r1, gk = tk->gk;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const T* __restrict__ L = F + tk->L_off;
    const T* __restrict__ G1 = Zbuf + tk->M_off + (int64_t)(c0 / kPanel) * (kPanel * kPanel);
    T* __restrict__ Us = U + tk->U_off * kNrhsMax;
    const int* __restrict__ gat = gatab + tk->gat;
    const int i0 = r0 + 16 * wave;   // the wave's 16 rows
    const bool act = i0 < r1;        // uniform
    // the pair's right-hand side: rows 16 wave and 64 + 16 wave
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int l0 = 64 * h + 16 * wave;
        acc_t a = {0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = l0 + Mfma<T>::row(lk, r);
            if (i < w) a[r] = Y[(int64_t)(first + c0 + i) * kNrhsMax + lr];
        }
        if (gk > 0) gather16<T>(a, U, gat, f, gk, tk->deep != 0, c0 + l0, c0 + w, lr, [&](int r) { return Mfma<T>::row(lk, r); });
#pragma unroll
        for (int r = 0; r < 4; ++r) b[(l0 + Mfma<T>::row(lk, r)) * kNrhsMax + lr] = a[r];
    }
    acc_t a = {0, 0, 0, 0};
    if (act) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = i0 + Mfma<T>::row(lk, r);
            if (i < r1) {
                if (i < p) a[r] = Y[(int64_t)(first + i) * kNrhsMax + lr];
                else if (c0 > 0) a[r] = Us[(int64_t)(i - p) * kNrhsMax + lr];
            }
        }
        if (gk > 0) gather16<T>(a, U, gat, f, gk, tk->deep != 0, i0, r1, lr, [&](int r) { return Mfma<T>::row(lk, r); });
    }
    // every operand before the first product: Z1, Z2 and L21 for the wave's 16 rows
    // of y, L for its rows (zero blocks past the diagonal are multiplied too:
    // a loop up to it would wait for its loads block by block)
    const bool two = w2 > 0;   // uniform
    T z1[4][4], z2[4][4], lb[4][4], l1[4][4], l2[4][4];
    const T* __restrict__ Lr = L + min(i0 + lr, f - 1);
    const T* __restrict__ L21 = L + min(c0 + kPanel + 16 * wave + lr, f - 1);
    const bool rv = i0 + lr < r1;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            const int k = 16 * kk + Mfma<T>::row(lk, st);
            z1[kk][st] = k <= 16 * wave + lr ? G1[k * kPanel + 16 * wave + lr] : T(0);
            l1[kk][st] = rv && k < w1 ? Lr[(int64_t)(c0 + k) * f] : T(0);
        }
    if (two)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const int k = 16 * kk + Mfma<T>::row(lk, st);
                z2[kk][st] = k <= 16 * wave + lr ? G1[(kPanel + k) * kPanel + 16 * wave + lr] : T(0);
                lb[kk][st] = 16 * wave + lr < w2 ? L21[(int64_t)(c0 + k) * f] : T(0);
                l2[kk][st] = rv && k < w2 ? Lr[(int64_t)(c0 + kPanel + k) * f] : T(0);
            }
    __syncthreads();
    // the wave's 16 rows of panel h's y
    auto store_y = [&](const acc_t& s, int h) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 64 * h + 16 * wave + Mfma<T>::row(lk, r);
            y[i * kNrhsMax + lr] = s[r];
            if (tk->index == 0 && i < w) Y2[(int64_t)(first + c0 + i) * kNrhsMax + lr] = s[r];
        }
    };
    store_y(product16<T>(z1, b, lr, lk), 0);
    __syncthreads();
    if (two) {
        const acc_t s = product16<T>(lb, y, lr, lk);
#pragma unroll
        for (int r = 0; r < 4; ++r) b[(64 + 16 * wave + Mfma<T>::row(lk, r)) * kNrhsMax + lr] -= s[r];
        __syncthreads();
        store_y(product16<T>(z2, b + 64 * kNrhsMax, lr, lk), 1);
        __syncthreads();
    }
    if (!act) return;
    a -= product16<T>(l1, y, lr, lk);
    if (two) a -= product16<T>(l2, y + 64 * kNrhsMax, lr, lk);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + Mfma<T>::row(lk, r);
        if (i >= r1) continue;
        if (i < p) Y[(int64_t)(first + i) * kNrhsMax + lr] = a[r];
        else Us[(int64_t)(i - p) * kNrhsMax + lr] = a[r];
    }
}

// Small fronts hold their pieces in one order for both types: item r of a lane is
// row 4 r + lk.  The f32 products give it when the lane's row of the first operand
// is the (4, 4)-transposed one (an involution), and step st contracts rows 4 st + lk.
template <typename T>
__device__ __forceinline__ int op_row(int lr) { return sizeof(T) == 8 ? lr : 4 * (lr & 3) + (lr >> 2); }

// The four 16-lane rows of v, each spread over the wave (lane % 16 kept): gfx950's
// row swaps, a few cycles each against an LDS permute's hundred.
__device__ __forceinline__ void spread_rows(unsigned int v, unsigned int (&o)[4]) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);          // rows 0 0 2 2 and 1 1 3 3
    const auto b = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);    // 0 and 2
    const auto c = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);    // 1 and 3
    o[0] = b[0]; o[1] = c[0]; o[2] = b[1]; o[3] = c[1];
}
__device__ __forceinline__ void spread_rows(float v, float (&o)[4]) {
    unsigned int u[4];
    spread_rows(__builtin_bit_cast(unsigned int, v), u);
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = __builtin_bit_cast(float, u[k]);
}
__device__ __forceinline__ void spread_rows(double v, double (&o)[4]) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    unsigned int lo[4], hi[4];
    spread_rows((unsigned int)b, lo);
    spread_rows((unsigned int)(b >> 32), hi);
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = __builtin_bit_cast(double, (unsigned long long)hi[k] << 32 | lo[k]);
}

// Substitution with a 16 x 16 unit triangle for 16 columns: a (item r: row 4 r + lk)
// becomes L^-1 a, or, kBack, L^-T a.  Four rows at a time, by every lane for its
// column, then one product takes them to the other rows.  d: step st's first
// operand, forward d[st] = L[op_row][4 st + lk], backward d[st] = L[4 st + lk][op_row],
// zero on and above the diagonal.  With the triangle's explicit inverse (four products
// a triangle; a solve of 16 columns at order 500k 3710 us, so 3775) the residuals of an
// OPF of order 625 to 2000 were 1.22 to 1.59 times those of one column at a time, so
// 1.07 to 1.13.
template <typename T, bool kBack>
__device__ __forceinline__ void substitute16(typename Mfma<T>::acc_t& a, const T (&d)[4], int lr, int lk) {
    const int m = op_row<T>(lr);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = kBack ? 3 - q : q;
        T l[4][4], v[4];   // l: the 4 x 4 triangle, from the lane that holds each entry
#pragma unroll
        for (int i = 1; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < i; ++j)
                l[i][j] = kBack ? bcast(d[r], 16 * i + op_row<T>(4 * r + j)) : bcast(d[r], 16 * j + op_row<T>(4 * r + i));
        spread_rows(a[r], v);
        if (!kBack) {
            v[1] -= l[1][0] * v[0];
            v[2] -= l[2][0] * v[0];
            v[3] -= l[3][0] * v[0];
            v[2] -= l[2][1] * v[1];
            v[3] -= l[3][1] * v[1];
            v[3] -= l[3][2] * v[2];
        } else {
            v[2] -= l[3][2] * v[3];
            v[1] -= l[3][1] * v[3];
            v[0] -= l[3][0] * v[3];
            v[1] -= l[2][1] * v[2];
            v[0] -= l[2][0] * v[2];
            v[0] -= l[1][0] * v[1];
        }
        a[r] = lk == 0 ? v[0] : lk == 1 ? v[1] : lk == 2 ? v[2] : v[3];
        if (q < 3) a = Mfma<T>::run((kBack ? m < 4 * r : m > 4 * r + 3) ? -d[r] : T(0), a[r], a);
    }
}

// A small front of order up to 16 NT by one wave, all of it in registers.  Each
// sub-panel's products are summed from zero before they are added to a piece: added
// one after the other to a large value they are rounded to its last place each time.
template <typename T, int NT>
__device__ __forceinline__ void fwd_front16(const SmallTask* tk, const T* __restrict__ F, const int* __restrict__ gatab,
                                            const T* __restrict__ Y, T* __restrict__ Y2, T* __restrict__ U, int lane) {
    typedef typename Mfma<T>::acc_t acc_t;
    const int first = tk->first, p = tk->p, f = tk->f, gk = tk->gk;
    const int lr = lane & 15, lk = lane >> 4, m = op_row<T>(lr);
    const T* __restrict__ L = F + tk->L_off;
    T* __restrict__ Us = U + tk->U_off * kNrhsMax;
    acc_t a[NT];
#pragma unroll
    for (int ti = 0; ti < NT; ++ti) {
        a[ti] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * ti + 4 * r + lk;
            if (i < p) a[ti][r] = Y[(int64_t)(first + i) * kNrhsMax + lr];
        }
        if (gk > 0) gather16<T>(a[ti], U, gatab + tk->gat, f, gk, tk->deep != 0, 16 * ti, f, lr, [&](int r) { return 4 * r + lk; });
    }
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        const int kb = 16 * q, bw = min(16, p - kb);
        if (bw <= 0) break;   // uniform
        T l[4];
#pragma unroll
        for (int ti = q; ti < NT; ++ti) {
            const int i = 16 * ti + m;
            const T* __restrict__ Li = L + min(i, f - 1);
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const int k = 4 * st + lk;
                const T x = Li[(int64_t)(kb + min(k, bw - 1)) * f];
                l[st] = k < bw && i < f && (ti > q || m > k) ? x : T(0);
            }
            if (ti == q) {
                substitute16<T, false>(a[q], l, lr, lk);
                continue;
            }
            acc_t s = {0, 0, 0, 0};
#pragma unroll
            for (int st = 0; st < 4; ++st) s = Mfma<T>::run(l[st], a[q][st], s);
            a[ti] -= s;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * r + lk;
            if (i < bw) Y2[(int64_t)(first + kb + i) * kNrhsMax + lr] = a[q][r];
        }
    }
#pragma unroll
    for (int ti = 0; ti < NT; ++ti) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * ti + 4 * r + lk;
            if (i >= p && i < f) Us[(int64_t)(i - p) * kNrhsMax + lr] = a[ti][r];
        }
    }
}

template <typename T, bool kPanels>
__global__ __launch_bounds__(256, kPanels ? 2 : 3) void k_fwd16(const PanelTask* __restrict__ pt, int np,
                                                  const SmallTask* __restrict__ st, int ns,
                                                  const int* __restrict__ gat, const T* __restrict__ F,
                                                  const T* __restrict__ Zbuf, T* __restrict__ Y, T* __restrict__ Y2,
                                                  T* __restrict__ U) {
    const int b = blockIdx.x;
    if (kPanels && b < np) {
        fwd_panels16<T>(pt + b, F, Zbuf, gat, Y, Y2, U);
    } else {
        const int t = 4 * (b - np) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        if (t >= ns) return;
        const int lane = threadIdx.x & 63;
        if (st[t].f <= 32) fwd_front16<T, 2>(st + t, F, gat, Y, Y2, U, lane);
        else if (st[t].f <= 64) fwd_front16<T, 4>(st + t, F, gat, Y, Y2, U, lane);
        else fwd_front16<T, 8>(st + t, F, gat, Y, Y2, U, lane);
    }
}

// A pair's x from v (128 x 16 in LDS, zero beyond its columns): x2 = Z2^T v2, then,
// with `one`, x1 = Z1^T (v1 - L21^T x2); wave w's 16 rows of each.  x2 takes v2's
// place, v1 - L21^T x2 that of v1.
template <typename T>
struct PairOps16 {
    typedef typename Mfma<T>::acc_t acc_t;
    T z1[4][4], z2[4][4], lb[4][4];
    __device__ __forceinline__ void load(const T* __restrict__ G1, const T* __restrict__ A, int f, int c0, int w2,
                                         bool one, int wave, int lr, int lk) {
        const T* __restrict__ G2 = G1 + kPanel * kPanel;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const int u = 16 * kk + Mfma<T>::row(lk, st), t = 16 * wave + lr;
                z1[kk][st] = one && u >= t ? G1[u * kPanel + t] : T(0);   // (Z^T)[t][u] above the diagonal
                z2[kk][st] = w2 > 0 && u >= t ? G2[u * kPanel + t] : T(0);
                lb[kk][st] = one && u < w2 ? A[c0 + t + (int64_t)(c0 + kPanel + u) * f] : T(0);
            }
    }
    __device__ __forceinline__ void apply(T* v, bool two, bool one, int wave, int lr, int lk, acc_t& x1,
                                          acc_t& x2) const {
        if (two) {
            x2 = product16<T>(z2, v + 64 * kNrhsMax, lr, lk);
            if (!one) return;
            __syncthreads();   // v2 has been read
            put(v + 64 * kNrhsMax, x2, wave, lr, lk);
            __syncthreads();
            const acc_t s = product16<T>(lb, v + 64 * kNrhsMax, lr, lk);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[(16 * wave + Mfma<T>::row(lk, r)) * kNrhsMax + lr] -= s[r];
            __syncthreads();
        }
        x1 = product16<T>(z1, v, lr, lk);
    }
    static __device__ __forceinline__ void put(T* v, const acc_t& x, int wave, int lr, int lk) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[(16 * wave + Mfma<T>::row(lk, r)) * kNrhsMax + lr] = x[r];
    }
};

template <typename T>
__device__ __forceinline__ void bwd_panels16(const PanelTask* tk, const int* __restrict__ rows, const T* __restrict__ F,
                                             const T* __restrict__ Zbuf, const T* __restrict__ D,
                                             const T* __restrict__ Y2, T* __restrict__ X, T* __restrict__ pw,
                                             const T* __restrict__ pr) {
    typedef typename Mfma<T>::acc_t acc_t;
    __shared__ T v[128 * kNrhsMax], xs[64 * kNrhsMax];
    const int first = tk->first, p = tk->p, f = tk->f, c0 = tk->c0, w = tk->w1 + tk->w2;
    const int r0 = tk->r0, nr = tk->r1 - r0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const bool own = tk->index >= 0, fin = tk->fntask > 0, self = own && tk->ntask == 1;
    const int xc0 = fin ? tk->fc0 : c0, xw1 = fin ? tk->fw1 : tk->w1, xw2 = fin ? tk->fw2 : tk->w2;
    const T* __restrict__ A = F + tk->L_off;
    const int which = fin ? tk->which : 0;   // the panel it finishes
    const bool two = tk->w2 > 0;             // uniform
    PairOps16<T> ops;
    if (fin || self)
        ops.load(Zbuf + tk->M_off + (int64_t)(xc0 / kPanel) * (kPanel * kPanel), A, f, xc0, xw2, which == 0, wave, lr,
                 lk);
    // L^T operands: wave w takes columns 16 w and 64 + 16 w
    T l1[4][4], l2[4][4];
    if (own) {
        const int cl = 16 * wave + lr;
        const T* __restrict__ src = A + c0;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const int i = 16 * kk + Mfma<T>::row(lk, st);
                const T* __restrict__ row = src + (int64_t)min(r0 + i, f - 1) * f;
                l1[kk][st] = i < nr && cl < w ? row[cl] : T(0);
                if (two) l2[kk][st] = i < nr && 64 + cl < w ? row[64 + cl] : T(0);
            }
    }
    if (own) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int i = (tid >> 4) + 16 * it, gi = r0 + i;
            xs[i * kNrhsMax + (tid & 15)] =
                i < nr ? X[(int64_t)(gi < p ? first + gi : rows[tk->rows_off + gi]) * kNrhsMax + (tid & 15)] : T(0);
        }
    }
    if (fin) {
        // v = y / d - sum over the pair's tasks, eight entries a thread
        T a[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = T(0);
        const T* __restrict__ src = pr + (int64_t)tk->fslot0 * (128 * kNrhsMax) + tid;
        for (int g0 = 0; g0 < tk->fntask; g0 += 4) {
            T u[4][8];
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    u[g][k] = g0 + g < tk->fntask ? src[(int64_t)(g0 + g) * (128 * kNrhsMax) + 256 * k] : T(0);
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int k = 0; k < 8; ++k) a[k] += u[g][k];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int e = tid + 256 * k, i = e >> 4;
            v[e] = i < xw1 + xw2
                       ? Y2[(int64_t)(first + xc0) * kNrhsMax + e] * (T(1) / D[first + xc0 + i]) - a[k] : T(0);
        }
        __syncthreads();
        acc_t x1, x2;
        ops.apply(v, xw2 > 0, which == 0, wave, lr, lk, x1, x2);
        const acc_t s = which ? x2 : x1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * wave + Mfma<T>::row(lk, r);
            if (i >= (which ? xw2 : xw1)) continue;
            X[(int64_t)(first + xc0 + 64 * which + i) * kNrhsMax + lr] = s[r];
            if (own) xs[(xc0 + 64 * which + i - r0) * kNrhsMax + lr] = s[r];
        }
    }
    if (!own) return;   // the whole workgroup
    __syncthreads();
    // the sums
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h == 1 && !two) break;   // uniform
        const acc_t s = product16<T>(h ? l2 : l1, xs, lr, lk);
        if (!self) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                pw[((int64_t)(tk->slot0 + tk->index) * 128 + 64 * h + 16 * wave + Mfma<T>::row(lk, r)) * kNrhsMax + lr] =
                    s[r];
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 64 * h + 16 * wave + Mfma<T>::row(lk, r);
                v[i * kNrhsMax + lr] = i < w ? Y2[(int64_t)(first + c0 + i) * kNrhsMax + lr] * (T(1) / D[first + c0 + i]) - s[r]
                                             : T(0);
            }
        }
    }
    if (!self) return;
    __syncthreads();
    acc_t x1, x2;
    ops.apply(v, two, true, wave, lr, lk, x1, x2);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 16 * wave + Mfma<T>::row(lk, r);
        if (i < tk->w1) X[(int64_t)(first + c0 + i) * kNrhsMax + lr] = x1[r];
        if (i < tk->w2) X[(int64_t)(first + c0 + kPanel + i) * kNrhsMax + lr] = x2[r];
    }
}

// Sums of 16 rows from zero, as in fwd_front16: with all rows in one chain the residuals
// were up to 1.04 times as large, and a solve of 16 columns at order 500k took 3256 us,
// so 3323 (two waves a SIMD instead of three).
template <typename T, int NT>
__device__ __forceinline__ void bwd_front16(const SmallTask* tk, const int* __restrict__ rows, const T* __restrict__ F,
                                            const T* __restrict__ D, const T* __restrict__ Y2, T* __restrict__ X,
                                            int lane) {
    typedef typename Mfma<T>::acc_t acc_t;
    const int first = tk->first, p = tk->p, f = tk->f;
    const int lr = lane & 15, lk = lane >> 4, m = op_row<T>(lr);
    const T* __restrict__ L = F + tk->L_off;
    acc_t x[NT];
#pragma unroll
    for (int ti = 0; ti < NT; ++ti) {
        x[ti] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * ti + 4 * r + lk;
            if (i >= p && i < f) x[ti][r] = X[(int64_t)rows[tk->rows_off + i] * kNrhsMax + lr];
        }
    }
#pragma unroll
    for (int q = NT - 1; q >= 0; --q) {
        const int kb = 16 * q, bw = min(16, p - kb);
        if (bw <= 0) continue;   // uniform
        acc_t s = {0, 0, 0, 0};
        const T* __restrict__ Lc = L + (int64_t)(kb + min(m, bw - 1)) * f;
        T d[4];   // the sub-panel's own triangle
#pragma unroll
        for (int ti = q; ti < NT; ++ti) {
            T l[4];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const int i = 16 * ti + 4 * st + lk;
                const T e = Lc[min(i, f - 1)];
                l[st] = m < bw && i < f && i >= kb + bw ? e : T(0);
                if (ti == q) d[st] = 4 * st + lk < bw && 4 * st + lk > m ? e : T(0);
            }
            acc_t u = {0, 0, 0, 0};
#pragma unroll
            for (int st = 0; st < 4; ++st) u = Mfma<T>::run(l[st], x[ti][st], u);
            s += u;
        }
        acc_t v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * r + lk, ic = kb + min(i, bw - 1);
            v[r] = i < bw ? Y2[(int64_t)(first + ic) * kNrhsMax + lr] * (T(1) / D[first + ic]) - s[r] : T(0);
        }
        substitute16<T, true>(v, d, lr, lk);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * r + lk;
            if (i < bw) {
                X[(int64_t)(first + kb + i) * kNrhsMax + lr] = v[r];
                x[q][r] = v[r];
            }
        }
    }
}

template <typename T, bool kPanels>
__global__ __launch_bounds__(256, 2) void k_bwd16(const PanelTask* __restrict__ pt, int np,
                                                  const SmallTask* __restrict__ st, int ns,
                                                  const int* __restrict__ rows, const T* __restrict__ F,
                                                  const T* __restrict__ Zbuf, const T* __restrict__ D,
                                                  const T* __restrict__ Y2, T* __restrict__ X, T* __restrict__ pw,
                                                  const T* __restrict__ pr) {
    const int b = blockIdx.x;
    if (kPanels && b < np) {
        bwd_panels16<T>(pt + b, rows, F, Zbuf, D, Y2, X, pw, pr);
    } else {
        const int t = 4 * (b - np) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        if (t >= ns) return;
        const int lane = threadIdx.x & 63;
        if (st[t].f <= 32) bwd_front16<T, 2>(st + t, rows, F, D, Y2, X, lane);
        else if (st[t].f <= 64) bwd_front16<T, 4>(st + t, rows, F, D, Y2, X, lane);
        else bwd_front16<T, 8>(st + t, rows, F, D, Y2, X, lane);
    }
}

// ---------------------------------------------------------------------------
// refinement
// ---------------------------------------------------------------------------
// s = a + b rounded, err = its exact rounding error (a + b = s + err, Knuth's
// two-sum; no reassociation: the build does not allow it).
__device__ __forceinline__ double two_sum(double a, double b, double& err) {
    const double s = a + b;
    const double bb = s - a;
    err = (a - (s - bb)) + (b - bb);
    return s;
}

// One row of R = B - K X and its part of the chunk's figures.  Each row sum is
// compensated (products split with fma, sums with two-sum: the Dot2 scheme of
// Ogita, Rump and Oishi, 2005), so r_i is accurate to about one rounding of
// itself rather than of |K||x|_i: the residual's own rounding stays near one
// unit of |b - Kx|, and refinement is not held at the rounding floor of a
// plain FP64 row sum.
struct RowSum {
    double acc = 0.0, cmp = 0.0, aacc = 0.0;
    __device__ __forceinline__ void add(double k, double x) {
        const double pr = k * x;
        const double pe = fma(k, x, -pr);
        double t;
        acc = two_sum(acc, pr, t);
        cmp += t + pe;
        aacc += fabs(k) * fabs(x);
    }
    // r_i; v: max |r_i|, max |x_i|, max |b_i|, sum r_i^2, sum b_i^2 and max_i
    // |r_i| / (|K| |x| + |b|)_i (the componentwise backward error; 0/0 counts
    // as 0, r/0 as infinite)
    __device__ __forceinline__ double finish(double b, double x, double (&v)[kResWidth]) const {
        double t;
        const double hi = two_sum(b, -acc, t);
        const double rr = hi + (t - cmp);
        const bool nan = rr != rr;
        const double den = aacc + fabs(b);
        const double cw = nan ? INFINITY : (den > 0.0 ? fabs(rr) / den : (rr != 0.0 ? INFINITY : 0.0));
        v[0] = nan ? INFINITY : fmax(v[0], fabs(rr));   // NaN residual -> infinite
        v[1] = fmax(v[1], fabs(x));
        v[2] = fmax(v[2], fabs(b));
        v[3] += nan ? INFINITY : rr * rr;
        v[4] += b * b;
        v[5] = fmax(v[5], cw);
        return rr;
    }
};

__device__ __forceinline__ double res_join(int k, double a, double b) { return k == 3 || k == 4 ? a + b : fmax(a, b); }

// One right-hand side: block per chunk of rows (one system); eight lanes share a row.
// The chunk's figures go to partial[stride c ..].
__global__ __launch_bounds__(256) void k_residual(DevPlan d, const double* __restrict__ K,
                                                  const double* __restrict__ B, const double* __restrict__ x,
                                                  double* __restrict__ R, const RowChunk* __restrict__ chunks, double* partial,
                                                  int stride) {
    const int c = blockIdx.x, row0 = chunks[c].row0, rows = chunks[c].rows;
    const int tid = threadIdx.x, sub = tid & 7, grp = tid >> 3;
    __shared__ double sm[kResWidth][256];
    double v[kResWidth] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int r = grp; r < rows; r += 32) {
        const int row = row0 + r;
        RowSum s;
        for (int64_t e = d.Kp[row] + sub; e < d.Kp[row + 1]; e += 8) s.add(K[e], x[d.Kj[e]]);
        for (int o = 4; o > 0; o >>= 1) {
            double t;
            s.acc = two_sum(s.acc, __shfl_xor(s.acc, o, 8), t);
            s.cmp += __shfl_xor(s.cmp, o, 8) + t;
            s.aacc += __shfl_xor(s.aacc, o, 8);
        }
        if (sub == 0) R[row] = s.finish(B[row], x[row], v);
    }
#pragma unroll
    for (int k = 0; k < kResWidth; ++k) sm[k][tid] = v[k];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) {
#pragma unroll
            for (int k = 0; k < kResWidth; ++k) sm[k][tid] = res_join(k, sm[k][tid], sm[k][tid + o]);
        }
        __syncthreads();
    }
    if (tid < kResWidth) partial[(int64_t)c * stride + tid] = sm[tid][0];
}

// Several right-hand sides: 16 lanes share a row, one column each, so K is read
// once for all of them and x (row-major, kNrhsMax a row) 16 columns at a time;
// R is row-major too.  Column by column, K was read again for each: 537 us for
// 16 columns at order 100k.
__global__ __launch_bounds__(256) void k_residual16(DevPlan d, const double* __restrict__ K,
                                                    const double* __restrict__ B, int64_t ldb,
                                                    const double* __restrict__ Xr, double* __restrict__ R, int nrhs,
                                                    const RowChunk* __restrict__ chunks, double* partial) {
    static_assert(kNrhsMax == 16, "one lane per column");
    const int c = blockIdx.x, row0 = chunks[c].row0, rows = chunks[c].rows;
    const int tid = threadIdx.x, q = tid & 15, grp = tid >> 4;
    __shared__ double sm[kResWidth][256];
    double v[kResWidth] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int r = grp; r < rows; r += 16) {
        const int row = row0 + r;
        RowSum s;
        const int64_t e1 = d.Kp[row + 1];
        for (int64_t e0 = d.Kp[row]; e0 < e1; e0 += 8) {
            double k[8], x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t e = min(e0 + u, e1 - 1);
                k[u] = K[e];
                x[u] = Xr[(int64_t)d.Kj[e] * kNrhsMax + q];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (e0 + u < e1) s.add(k[u], x[u]);
        }
        if (q < nrhs)
            R[(int64_t)row * kNrhsMax + q] = s.finish(B[row + q * ldb], Xr[(int64_t)row * kNrhsMax + q], v);
    }
#pragma unroll
    for (int k = 0; k < kResWidth; ++k) sm[k][tid] = v[k];
    __syncthreads();
    for (int o = 128; o >= 16; o >>= 1) {
        if (tid < o) {
#pragma unroll
            for (int k = 0; k < kResWidth; ++k) sm[k][tid] = res_join(k, sm[k][tid], sm[k][tid + o]);
        }
        __syncthreads();
    }
    if (tid < nrhs)
#pragma unroll
        for (int k = 0; k < kResWidth; ++k) partial[((int64_t)c * nrhs + tid) * kResWidth + k] = sm[k][tid];
}

// Xr[row][q] = X[row + q ldx], zero for q >= nrhs: 64 rows a block, through LDS.
__global__ __launch_bounds__(256) void k_to_rows(int64_t N, const double* __restrict__ X, int64_t ldx, int nrhs,
                                                 double* __restrict__ Xr) {
    __shared__ double t[kNrhsMax][65];
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    for (int i = threadIdx.x; i < 64 * kNrhsMax; i += 256) {
        const int r = i & 63, q = i >> 6;
        t[q][r] = q < nrhs && r0 + r < N ? X[r0 + r + q * ldx] : 0.0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * kNrhsMax; i += 256) {
        const int q = i & (kNrhsMax - 1), r = i / kNrhsMax;
        if (r0 + r < N) Xr[(r0 + r) * kNrhsMax + q] = t[q][r];
    }
}

__global__ void k_axpy_cols(double* X, int64_t ldx, const double* DX, int64_t N, int nrhs) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    for (int q = 0; q < nrhs; ++q) X[i + q * ldx] += DX[i + q * N];
}

__global__ void k_copy_cols(double* dst, int64_t ldd, const double* src, int64_t lds, int64_t N, int nrhs) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    for (int q = 0; q < nrhs; ++q) dst[i + q * ldd] = src[i + q * lds];
}

// Before a factorization: rho from the host's buffer (read over the bus, once;
// nullptr: unchanged), status bits and inertia counters cleared.
__global__ void k_begin(int S, const double* __restrict__ rho_host, double* __restrict__ rho, int* nonfinite,
                        unsigned long long* __restrict__ part) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 4 * (int64_t)S * kInertiaSlots) part[i] = 0ULL;
    if (rho_host && i < S) rho[i] = rho_host[i];
    if (i == 0) *nonfinite = 0;
}

// After it, a block per system: the counters' sums, ||K||_inf and the status
// bits straight into the host's buffer (4 S, S and one value).  Copied there, they
// were three transfers behind the last kernel, and ||K||_inf a fourth after a
// first wait: 50 us between a factorization and its solve at order 625.
__global__ __launch_bounds__(4 * kInertiaSlots) void k_end(DevPlan d, const double* __restrict__ kinf,
                                                           unsigned long long* host) {
    const int s = blockIdx.x, tid = threadIdx.x;
    __shared__ unsigned long long sm[4 * kInertiaSlots];
    sm[tid] = d.inertia_part[4 * (int64_t)s * kInertiaSlots + tid];
    __syncthreads();
    for (int o = 2 * kInertiaSlots; o >= 4; o >>= 1) {
        if (tid < o) sm[tid] += sm[tid + o];
        __syncthreads();
    }
    if (tid < 4) host[4 * (int64_t)s + tid] = sm[tid];
    if (tid == 4) host[4 * (int64_t)d.S + s] = (unsigned long long)__double_as_longlong(kinf[s]);
    if (tid == 5 && s == 0) host[5 * (int64_t)d.S] = (unsigned long long)(unsigned int)*d.nonfinite;
}

// ---------------------------------------------------------------------------
// slack elimination (K1s) and the recovery of the rest of the Newton step
// ---------------------------------------------------------------------------
// Every row r of J carries Sigma_s[r] >= 0 (its slack's barrier term) or
// +inf (an equality row: Omega = 1, no slack); rho_r = rho-hat of the row's
// system.  Sec. 3.3, Proposition "Condensed KKT system" and its proof.

// Omega_rr = Sigma_s / (rho + Sigma_s); a negative or NaN Sigma_s sets
// kNonfiniteInput.
__global__ void k_k1s_omega(int64_t nrows, const double* __restrict__ Sigma_s, const int* __restrict__ Jrow_sys,
                            const double* __restrict__ sys_rho, double* __restrict__ omega, int* nonfinite) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    const double S = Sigma_s[r];
    if (!(S >= 0.0)) {
        atomicOr(nonfinite, kNonfiniteInput);
        omega[r] = 0.0;
        return;
    }
    omega[r] = isinf(S) ? 1.0 : S / (sys_rho[Jrow_sys[r]] + S);
}

// b = r_t + rho J_I^T (Sigma_s + rho I)^-1 r_s: one thread per variable i,
// over the rows of column i of J in increasing order (J^T in CSC: Jt_ptr,
// Jt_row, Jt_k = index of the entry in J's values).
__global__ void k_k1s_rhs(int64_t n, const int64_t* __restrict__ Jt_ptr, const int* __restrict__ Jt_row,
                          const int* __restrict__ Jt_k, const double* __restrict__ J, const double* __restrict__ r_t,
                          const double* __restrict__ r_s, const double* __restrict__ Sigma_s,
                          const int* __restrict__ Jrow_sys, const double* __restrict__ sys_rho,
                          const int* __restrict__ row_sys, double* __restrict__ b) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double acc = 0.0;
    for (int64_t q = Jt_ptr[i]; q < Jt_ptr[i + 1]; ++q) {
        const int r = Jt_row[q];
        const double S = Sigma_s[r];
        if (isinf(S)) continue;
        acc += J[Jt_k[q]] * (r_s[r] / (S + sys_rho[Jrow_sys[r]]));
    }
    b[i] = r_t[i] + sys_rho[row_sys[i]] * acc;
}

// Delta s_r = (rho (J dt)_r + r_s,r) / (Sigma_s,r + rho) on inequality rows, 0
// on equality rows.
__global__ void k_k1s_ds(int64_t nrows, const int64_t* __restrict__ Jp, const int* __restrict__ Jj,
                         const double* __restrict__ J, const double* __restrict__ dt, const double* __restrict__ r_s,
                         const double* __restrict__ Sigma_s, const int* __restrict__ Jrow_sys,
                         const double* __restrict__ sys_rho, double* __restrict__ ds) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    const double S = Sigma_s[r];
    if (isinf(S)) {
        ds[r] = 0.0;
        return;
    }
    double a = 0.0;
    for (int64_t k = Jp[r]; k < Jp[r + 1]; ++k) a += J[k] * dt[Jj[k]];
    const double rho = sys_rho[Jrow_sys[r]];
    ds[r] = (rho * a + r_s[r]) / (S + rho);
}

// Delta y = -rho (J dx + c) + y_k - y (Sec. 3.3, eq. K1-elimination).
__global__ void k_recover_dy(int64_t nrows, const int64_t* __restrict__ Jp, const int* __restrict__ Jj,
                             const double* __restrict__ J, const double* __restrict__ dx, const double* __restrict__ c,
                             const double* __restrict__ y_k, const double* __restrict__ y,
                             const int* __restrict__ Jrow_sys, const double* __restrict__ sys_rho,
                             double* __restrict__ dy) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    double a = 0.0;
    for (int64_t k = Jp[r]; k < Jp[r + 1]; ++k) a += J[k] * dx[Jj[k]];
    dy[r] = -sys_rho[Jrow_sys[r]] * (a + c[r]) + y_k[r] - y[r];
}

// Delta r = (Delta y - y_k + y) / rho - r (Sec. 3.2, eq. K2-elimination,
// theta = 1 / rho-hat).
__global__ void k_recover_dr(int64_t nrows, const double* __restrict__ dy, const double* __restrict__ y_k,
                             const double* __restrict__ y, const double* __restrict__ r,
                             const int* __restrict__ Jrow_sys, const double* __restrict__ sys_rho,
                             double* __restrict__ dr) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nrows) return;
    dr[q] = (1.0 / sys_rho[Jrow_sys[q]]) * (dy[q] - y_k[q] + y[q]) - r[q];
}

// Delta z_l = -(Z_l dx - mu) / (x - l) - z_l, Delta z_u = (Z_u dx + mu) / (u - x)
// - z_u (Sec. 3.1, the blocks eliminated from eq. K3); an infinite bound
// makes the quotient 0.
__global__ void k_recover_dz(int64_t n, const double* __restrict__ x, const double* __restrict__ l,
                             const double* __restrict__ u, const double* __restrict__ z_l,
                             const double* __restrict__ z_u, const double* __restrict__ dx, double mu,
                             double* __restrict__ dz_l, double* __restrict__ dz_u) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    dz_l[i] = -(z_l[i] * dx[i] - mu) / (x[i] - l[i]) - z_l[i];
    dz_u[i] = (z_u[i] * dx[i] + mu) / (u[i] - x[i]) - z_u[i];
}

// out = in + delta (the primal regularization of eq. K2 applied to Sigma).
__global__ void k_add_scalar(int64_t n, const double* __restrict__ in, double delta, double* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = in[i] + delta;
}

// Sigma = Z_l / (x - l) + Z_u / (u - x) (Sec. 3.1, below eq. K2unreg).
__global__ void k_barrier_sigma(int64_t n, const double* __restrict__ x, const double* __restrict__ l,
                                const double* __restrict__ u, const double* __restrict__ z_l,
                                const double* __restrict__ z_u, double* __restrict__ sigma) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    sigma[i] = z_l[i] / (x[i] - l[i]) + z_u[i] / (u[i] - x[i]);
}

// ---------------------------------------------------------------------------
// adjoint (condensed form)
// ---------------------------------------------------------------------------
__global__ void k_jmul(int64_t nrows, const int64_t* __restrict__ Jp, const int* __restrict__ Jj,
                       const double* __restrict__ Jv, const double* __restrict__ X, const double* __restrict__ Lam,
                       int64_t ld, int nrhs, double* JX, double* JL) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    for (int q = 0; q < nrhs; ++q) {
        double a = 0.0, b = 0.0;
        for (int64_t k = Jp[r]; k < Jp[r + 1]; ++k) {
            a += Jv[k] * X[Jj[k] + q * ld];
            b += Jv[k] * Lam[Jj[k] + q * ld];
        }
        JX[r + q * nrows] = a;
        JL[r + q * nrows] = b;
    }
}

__global__ void k_grad_W(int64_t nnzW, const int* __restrict__ Wr, const int* __restrict__ Wc,
                         const double* __restrict__ X, const double* __restrict__ Lam, int64_t ld, int nrhs,
                         double* gW) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnzW) return;
    const int i = Wr[e], j = Wc[e];
    double g = 0.0;
    for (int q = 0; q < nrhs; ++q) {
        g -= Lam[i + q * ld] * X[j + q * ld];
        if (i != j) g -= Lam[j + q * ld] * X[i + q * ld];
    }
    gW[e] = g;
}

__global__ void k_grad_S(int64_t N, const double* __restrict__ X, const double* __restrict__ Lam, int64_t ld,
                         int nrhs, double* gS) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    double g = 0.0;
    for (int q = 0; q < nrhs; ++q) g -= Lam[i + q * ld] * X[i + q * ld];
    gS[i] = g;
}

__global__ void k_grad_J(int64_t nrows, const int64_t* __restrict__ Jp, const int* __restrict__ Jj,
                         const int* __restrict__ Jrow_sys, const double* __restrict__ sys_rho,
                         const double* __restrict__ X, const double* __restrict__ Lam, int64_t ld, int nrhs,
                         const double* __restrict__ JX, const double* __restrict__ JL, double* gJ) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    const double rho = sys_rho[Jrow_sys[r]];
    for (int64_t k = Jp[r]; k < Jp[r + 1]; ++k) {
        const int i = Jj[k];
        double g = 0.0;
        for (int q = 0; q < nrhs; ++q)
            g += Lam[i + q * ld] * JX[r + q * nrows] + X[i + q * ld] * JL[r + q * nrows];
        gJ[k] = -rho * g;
    }
}

// One block per system: gRho[s] = -sum over the system's J rows and columns of JL * JX.
__global__ __launch_bounds__(256) void k_grad_rho(const int64_t* __restrict__ sys_jrow, int64_t nrows, int nrhs,
                                                  const double* __restrict__ JX, const double* __restrict__ JL,
                                                  double* gRho) {
    const int s = blockIdx.x, tid = threadIdx.x;
    double acc = 0.0;
    for (int q = 0; q < nrhs; ++q)
        for (int64_t r = sys_jrow[s] + tid; r < sys_jrow[s + 1]; r += 256) acc += JL[r + q * nrows] * JX[r + q * nrows];
    __shared__ double sm[256];
    sm[tid] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) sm[tid] += sm[tid + o];
        __syncthreads();
    }
    if (tid == 0) gRho[s] = -sm[0];
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {
thread_local LaunchTimer* tl_timer = nullptr;

template <typename X> struct same_t { using type = X; };

// Every launch goes through here: plain hipLaunchKernelGGL, or the extended
// launch with the installed timer's events.
template <typename... KArgs>
void launch(void (*k)(KArgs...), dim3 grid, dim3 block, uint32_t lds, hipStream_t st,
            typename same_t<KArgs>::type... args) {
    hipEvent_t e0, e1;
    if (tl_timer && tl_timer->take(&e0, &e1))
        hipExtLaunchKernelGGL(k, grid, block, lds, st, e0, e1, 0, args...);
    else
        hipLaunchKernelGGL(k, grid, block, lds, st, args...);
}
}  // namespace

LaunchTimer* set_launch_timer(LaunchTimer* t) {
    LaunchTimer* old = tl_timer;
    tl_timer = t;
    return old;
}

void launch_assemble(const DevPlan& d, const RowChunk* chunks, int nchunks, const double* W, const double* Sigma,
                     const double* J, const double* sys_rho, const double* omega, double* K, double* partial,
                     hipStream_t st) {
    launch(k_assemble, dim3(nchunks), dim3(256), 0, st, d, chunks, W, Sigma, J, sys_rho, omega, K, partial);
}

void launch_k1s_omega(int64_t nrows, const double* Sigma_s, const int* Jrow_sys, const double* sys_rho, double* omega,
                      int* nonfinite, hipStream_t st) {
    if (nrows <= 0) return;
    launch(k_k1s_omega, dim3(blocks_for(nrows, 256)), dim3(256), 0, st, nrows, Sigma_s, Jrow_sys, sys_rho, omega,
           nonfinite);
}

void launch_k1s_rhs(int64_t n, const int64_t* Jt_ptr, const int* Jt_row, const int* Jt_k, const double* J,
                    const double* r_t, const double* r_s, const double* Sigma_s, const int* Jrow_sys,
                    const double* sys_rho, const int* row_sys, double* b, hipStream_t st) {
    if (n <= 0) return;
    launch(k_k1s_rhs, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, Jt_ptr, Jt_row, Jt_k, J, r_t, r_s, Sigma_s,
           Jrow_sys, sys_rho, row_sys, b);
}

void launch_k1s_ds(int64_t nrows, const int64_t* Jp, const int* Jj, const double* J, const double* dt,
                   const double* r_s, const double* Sigma_s, const int* Jrow_sys, const double* sys_rho, double* ds,
                   hipStream_t st) {
    if (nrows <= 0) return;
    launch(k_k1s_ds, dim3(blocks_for(nrows, 256)), dim3(256), 0, st, nrows, Jp, Jj, J, dt, r_s, Sigma_s, Jrow_sys,
           sys_rho, ds);
}

void launch_recover_dy(int64_t nrows, const int64_t* Jp, const int* Jj, const double* J, const double* dx,
                       const double* c, const double* y_k, const double* y, const int* Jrow_sys, const double* sys_rho,
                       double* dy, hipStream_t st) {
    if (nrows <= 0) return;
    launch(k_recover_dy, dim3(blocks_for(nrows, 256)), dim3(256), 0, st, nrows, Jp, Jj, J, dx, c, y_k, y, Jrow_sys,
           sys_rho, dy);
}

void launch_recover_dr(int64_t nrows, const double* dy, const double* y_k, const double* y, const double* r,
                       const int* Jrow_sys, const double* sys_rho, double* dr, hipStream_t st) {
    if (nrows <= 0) return;
    launch(k_recover_dr, dim3(blocks_for(nrows, 256)), dim3(256), 0, st, nrows, dy, y_k, y, r, Jrow_sys, sys_rho, dr);
}

void launch_recover_dz(int64_t n, const double* x, const double* l, const double* u, const double* z_l,
                       const double* z_u, const double* dx, double mu, double* dz_l, double* dz_u, hipStream_t st) {
    if (n <= 0) return;
    launch(k_recover_dz, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, x, l, u, z_l, z_u, dx, mu, dz_l, dz_u);
}

void launch_add_scalar(int64_t n, const double* in, double delta, double* out, hipStream_t st) {
    if (n <= 0) return;
    launch(k_add_scalar, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, in, delta, out);
}

void launch_barrier_sigma(int64_t n, const double* x, const double* l, const double* u, const double* z_l,
                          const double* z_u, double* sigma, hipStream_t st) {
    if (n <= 0) return;
    launch(k_barrier_sigma, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, x, l, u, z_l, z_u, sigma);
}

void launch_reduce(const int* sys_chunk_ptr, int S, int width, int period, unsigned int sum_mask,
                   const double* partial, double* out, hipStream_t st) {
    launch(k_reduce_partials, dim3(S, width), dim3(256), 0, st, sys_chunk_ptr, width, period, sum_mask, partial,
           out);
}

void launch_thresholds(const int* sys_chunk_ptr, int S, const double* partial, double eps, int mode,
                       const double* sys_rho, double* kinf, double* thr, int* nonfinite, hipStream_t st) {
    launch(k_thresholds, dim3(S), dim3(256), 0, st, sys_chunk_ptr, partial, eps, mode, sys_rho, kinf, thr, nonfinite);
}

template <typename T>
void launch_fronts(const FrontPlan& d, const FrontTask* tasks, int count, int fmax, int strip, const double* K, T* F,
                   T* D, hipStream_t st) {
    if (count <= 0) return;
    const uint32_t lds = (uint32_t)(strip * sizeof(T));
    if (fmax <= 32) launch(k_front<T, 2, 1>, dim3(count), dim3(64), lds, st, d, tasks, K, F, D);
    else if (fmax <= 64) launch(k_front<T, 4, 1>, dim3(count), dim3(64), lds, st, d, tasks, K, F, D);
    else if (fmax <= 96) launch(k_front<T, 6, 4>, dim3(count), dim3(256), lds, st, d, tasks, K, F, D);
    else launch(k_front<T, 8, 4>, dim3(count), dim3(256), lds, st, d, tasks, K, F, D);
}

template <typename T>
void launch_large_asm(const DevPlan& d, int64_t first, int count, int fmax, const double* K, T* F, hipStream_t st) {
    if (count <= 0) return;
    const size_t lds = 4 * (size_t)fmax * sizeof(T);
    const dim3 grid((count + 3) / 4);
    if (lds <= kAsmLdsMax)
        launch(k_large_asm<T, true>, grid, dim3(256), lds, st, d, first, count, fmax, K, F);
    else
        launch(k_large_asm<T, false>, grid, dim3(256), 0, st, d, first, count, fmax, K, F);
}

template <typename T>
void launch_large_diag(const DevPlan& d, const LargeTask* tasks, int count, T* F, T* D, T* M, hipStream_t st) {
    if (count <= 0) return;
    launch(k_large_diag<T>, dim3(count), dim3(256), 0, st, d, tasks, F, D, M);
}

template <typename T>
void launch_large_panel(const LargeTask* tasks, int count, T* F, const T* D, const T* M, hipStream_t st) {
    if (count <= 0) return;
    launch(k_large_panel<T>, dim3(count), dim3(256), 0, st, tasks, F, D, M);
}

template <typename T>
void launch_large_dstep(const DevPlan& d, const LargeTask* dtasks, int nd, const LargeTask* utasks, int nu, T* F,
                        T* D, T* M, hipStream_t st) {
    if (nd <= 0 && nu <= 0) return;
    const int nd8 = (nd + 7) & ~7;
    launch(k_large_dstep<T>, dim3(nd8 + nu), dim3(256), 0, st, d, dtasks, nd, utasks, nu, F, D, M);
}

template <typename T>
void launch_permute_in(const DevPlan& d, const double* B, int64_t si, int64_t sq, int nrhs, T* Y, hipStream_t st) {
    if (nrhs == 1)
        launch(k_permute_in<T, 1>, dim3(blocks_for(d.N, 256)), dim3(256), 0, st, d, B, si, sq, nrhs, Y);
    else
        launch(k_permute_in<T, kNrhsMax>, dim3(blocks_for(d.N * kNrhsMax, 256)), dim3(256), 0, st, d, B, si, sq, nrhs,
               Y);
}

template <typename T>
void launch_permute_out(const DevPlan& d, const T* X, int nrhs, double* Xo, int64_t ldx, hipStream_t st) {
    if (nrhs == 1)
        launch(k_permute_out<T, 1>, dim3(blocks_for(d.N, 256)), dim3(256), 0, st, d, X, nrhs, Xo, ldx);
    else
        launch(k_permute_out<T, kNrhsMax>, dim3(blocks_for(d.N * kNrhsMax, 256)), dim3(256), 0, st, d, X, nrhs, Xo,
               ldx);
}

// A step with panel tasks and more small fronts than this takes two launches: the
// small fronts' own kernel keeps twice as many waves in flight, and they are then
// bound by that rather than by the launch.
constexpr int kSplitSmall = 1024;
// Up to this many small fronts in a backward step get a workgroup each (two fit a
// CU at once): launches of 5 to 304 fronts at order 20k 8 to 12 us by waves, 3.8 to 9.2.
constexpr int kWgSmall = 512;

template <typename T>
void launch_fwd(bool many, const PanelTask* pt, int np, const SmallTask* sm, int ns, const int* gat, const T* F,
                const T* Z, T* Y, T* Y2, T* U, hipStream_t st) {
    if (np > 0 && ns > kSplitSmall) {
        launch_fwd<T>(many, pt, 0, sm, ns, gat, F, Z, Y, Y2, U, st);
        ns = 0;
    }
    const int grid = np + (ns + 3) / 4;
    if (grid <= 0) return;
    auto k = np > 0 ? (many ? k_fwd16<T, true> : k_fwd1<T, true>) : (many ? k_fwd16<T, false> : k_fwd1<T, false>);
    launch(k, dim3(grid), dim3(256), 0, st, pt, np, sm, ns, gat, F, Z, Y, Y2, U);
}

template <typename T>
void launch_bwd(bool many, const PanelTask* pt, int np, const SmallTask* sm, int ns, const int* rows, const T* F,
                const T* Z, const T* D, const T* Y2, T* X, T* pw, const T* pr, hipStream_t st) {
    if (np > 0 && ns > kSplitSmall) {
        launch_bwd<T>(many, pt, 0, sm, ns, rows, F, Z, D, Y2, X, pw, pr, st);
        ns = 0;
    }
    const bool wg = !many && ns <= kWgSmall;
    const int grid = np + (wg ? ns : (ns + 3) / 4);
    if (grid <= 0) return;
    auto k = np > 0 ? (many ? k_bwd16<T, true> : wg ? k_bwd1<T, true, true> : k_bwd1<T, true, false>)
                    : (many ? k_bwd16<T, false> : wg ? k_bwd1<T, false, true> : k_bwd1<T, false, false>);
    launch(k, dim3(grid), dim3(256), 0, st, pt, np, sm, ns, rows, F, Z, D, Y2, X, pw, pr);
}

void launch_residual(const DevPlan& d, const double* K, const double* B, int64_t ldb, const double* X, int64_t ldx,
                     double* Xr, double* R, int nrhs, const RowChunk* chunks, int nchunks, double* partial,
                     hipStream_t st) {
    if (nrhs < kManyColumns) {
        for (int q = 0; q < nrhs; ++q)
            launch(k_residual, dim3(nchunks), dim3(256), 0, st, d, K, B + q * ldb, X + q * ldx, R + q * d.N, chunks,
                   partial + q * kResWidth, nrhs * kResWidth);
        return;
    }
    launch(k_to_rows, dim3(blocks_for(d.N, 64)), dim3(256), 0, st, d.N, X, ldx, nrhs, Xr);
    launch(k_residual16, dim3(nchunks), dim3(256), 0, st, d, K, B, ldb, Xr, R, nrhs, chunks, partial);
}

void launch_axpy_cols(double* X, int64_t ldx, const double* DX, int64_t N, int nrhs, hipStream_t st) {
    launch(k_axpy_cols, dim3(blocks_for(N, 256)), dim3(256), 0, st, X, ldx, DX, N, nrhs);
}

void launch_copy_cols(double* dst, int64_t ldd, const double* src, int64_t lds, int64_t N, int nrhs, hipStream_t st) {
    launch(k_copy_cols, dim3(blocks_for(N, 256)), dim3(256), 0, st, dst, ldd, src, lds, N, nrhs);
}

void launch_begin(int S, const double* rho_host, double* rho, int* nonfinite, unsigned long long* part,
                  hipStream_t st) {
    launch(k_begin, dim3(blocks_for(4 * (int64_t)S * kInertiaSlots, 256)), dim3(256), 0, st, S, rho_host, rho, nonfinite,
           part);
}

void launch_end(const DevPlan& d, const double* kinf, unsigned long long* host, hipStream_t st) {
    launch(k_end, dim3(d.S), dim3(4 * kInertiaSlots), 0, st, d, kinf, host);
}

void launch_adjoint(const DevPlan& d, int64_t nnzW, const int* W_row, const int* W_col, int64_t nJrows,
                    const int64_t* Jp, const int* Jj, const int* Jrow_sys, const double* Jval, const double* sys_rho,
                    const double* X, const double* Lam, int64_t ld, int nrhs, double* gW, double* gSigma,
                    double* gJ, double* gRho, double* JX, double* JL, const int64_t* sys_jrow, hipStream_t st) {
    if (nJrows > 0)
        launch(k_jmul, dim3(blocks_for(nJrows, 256)), dim3(256), 0, st, nJrows, Jp, Jj, Jval, X, Lam, ld,
                           nrhs, JX, JL);
    if (gW && nnzW > 0)
        launch(k_grad_W, dim3(blocks_for(nnzW, 256)), dim3(256), 0, st, nnzW, W_row, W_col, X, Lam, ld,
                           nrhs, gW);
    if (gSigma)
        launch(k_grad_S, dim3(blocks_for(d.N, 256)), dim3(256), 0, st, d.N, X, Lam, ld, nrhs, gSigma);
    if (gJ && nJrows > 0)
        launch(k_grad_J, dim3(blocks_for(nJrows, 256)), dim3(256), 0, st, nJrows, Jp, Jj, Jrow_sys,
                           sys_rho, X, Lam, ld, nrhs, JX, JL, gJ);
    if (gRho)
        launch(k_grad_rho, dim3(d.S), dim3(256), 0, st, sys_jrow, nJrows, nrhs, JX, JL, gRho);
}

// Allow the LDS-resident kernels to request more than 64 KiB of dynamic LDS
// (gfx950 has 160 KiB per workgroup).
hipError_t configure_kernels(int max_dynamic_lds) {
    hipError_t e = hipSuccess, r;
    const void* fns[] = {(const void*)k_front<double, 6, 4>, (const void*)k_front<double, 8, 4>,
                         (const void*)k_front<float, 6, 4>, (const void*)k_front<float, 8, 4>,
                         (const void*)k_large_asm<double, true>, (const void*)k_large_asm<float, true>};
    for (const void* f : fns) {
        hipFuncAttributes at{};
        r = hipFuncGetAttributes(&at, f);
        if (r != hipSuccess) { e = r; continue; }
        const int dyn = max_dynamic_lds - (int)at.sharedSizeBytes;
        r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
        if (r != hipSuccess) e = r;
    }
    return e;
}

#define NCL_INSTANTIATE(T)                                                                                         \
    template void launch_fronts<T>(const FrontPlan&, const FrontTask*, int, int, int, const double*, T*, T*,       \
                                   hipStream_t);                                                                   \
    template void launch_large_asm<T>(const DevPlan&, int64_t, int, int, const double*, T*, hipStream_t);          \
    template void launch_large_diag<T>(const DevPlan&, const LargeTask*, int, T*, T*, T*, hipStream_t);          \
    template void launch_large_panel<T>(const LargeTask*, int, T*, const T*, const T*, hipStream_t);               \
    template void launch_large_dstep<T>(const DevPlan&, const LargeTask*, int, const LargeTask*, int, T*, T*, T*,  \
                                        hipStream_t);                                                              \
    template void launch_permute_in<T>(const DevPlan&, const double*, int64_t, int64_t, int, T*, hipStream_t);     \
    template void launch_permute_out<T>(const DevPlan&, const T*, int, double*, int64_t, hipStream_t);             \
    template void launch_fwd<T>(bool, const PanelTask*, int, const SmallTask*, int, const int*, const T*,          \
                                const T*, T*, T*, T*, hipStream_t);                                                \
    template void launch_bwd<T>(bool, const PanelTask*, int, const SmallTask*, int, const int*, const T*,          \
                                const T*, const T*, const T*, T*, T*, const T*, hipStream_t);

NCL_INSTANTIATE(double)
NCL_INSTANTIATE(float)

}  // namespace ncl
