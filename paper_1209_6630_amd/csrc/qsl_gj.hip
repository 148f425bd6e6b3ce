// FP64 log|det|, sign and inverse of the Slater matrices (inversion step,
// section "Overall performance of QMC=Chem"; Slater matrix D_ij = phi_i(r_j)).
//
// One workgroup inverts one n x n matrix (n <= 224) held entirely in
// registers, by Gauss-Jordan elimination with partial pivoting on the rows of
// D: at step k the pivot is the largest |D[i][k]| over rows not yet used
// (smallest i on exact ties; for n > 128, among values within 2^-12 relative
// of the largest, which leaves the elimination as stable).  Pivot rows are
// not moved; the pivot sequence p_k is recorded and the result is un-permuted
// on the way out: D^-1[k][p_j] = M[p_k][j].
// The pivots are the diagonal of U in P D = L U, so log|det| = sum log|pivot|
// and sign = sign(permutation) prod sign(pivot).  2 n^3 flops per matrix.
//
// The rank-1 step of column k, with multipliers f_i = -D[i][k] / pv (0 in the
// pivot row, which stays unscaled until the end): M[i][c] += f_i M[p_k][c],
// and column k takes pv + 1 for its pivot-row entry, which turns it into
// -D[i][k] / pv.  Steps are taken 16 columns (a panel) at a time without
// changing a single rounding: one wave eliminates the panel, whose columns it
// holds in its own registers (only lane exchanges inside a step), and
// publishes the multipliers F of its steps; for every other column the
// pivot-row entries w_k at step k come from those at the panel's start by
// forward substitution (w_k += F_m[p_k] w_m, m < k ascending), and then
// v += F w.  v_mfma_f64_16x16x4f64 adds its four products to the accumulator
// one after the other in order, each with one rounding, as a chain of FMAs
// does, so the updates on it give the rank-1 steps' values bit for bit.  A
// panel's own column c is a column whose entries w_k with k <= c are 0.
//
// Layout: wave u of NU owns the D columns of tiles u and u + NU, 16 each, as
// MFMA results (register row (lane / 16) + 4 r of a tile is D column e, lane
// % 16 is D row i, so C_1[e][i], F and the panel are read and written in runs
// of 16 values); the last wave is the panel wave.  Look-ahead: the wave
// owning the next panel's columns updates that tile first and hands it over
// in LDS, and the panel wave eliminates it while the others finish; one
// barrier per panel publishes F.
//
// Bound: the panel wave's chain of search, reciprocal and update (about 800
// cycles a step at n = 79, 1200 at n = 217), then the rank-16 updates at the
// FP64 matrix rate (the same as the vector rate here).  A matrix of up to 16
// takes its own n steps only, not the identity's: 65536 of n = 1 in 126 us (321
// with all 16 steps, 131 by rank-1 steps), 60000 of n = 5 in 208 (298, 284),
// 8192 of n = 8 in 42 (50, 78).  Measured, against the
// eight waves that published one or two rank-1 steps at a time through LDS
// before: one matrix of n = 79 in 53 us (162), 2048 of them in 205 us (775),
// 777 of n = 132 in 479 us (741), 2048 of n = 217 in 2.30 ms (2.61).
#include <algorithm>

#include "qsl_internal.h"

namespace qsl {

typedef __attribute__((ext_vector_type(4))) double f64x4;
typedef __attribute__((ext_vector_type(2))) double f64x2;

// Shapes: n <= 16 NT.
template <int NT>
struct GJT {
    static constexpr int CT = 2;                    // D column tiles per updating wave
    static constexpr int NU = (NT + CT - 1) / CT;   // updating waves
    static constexpr int THREADS = (NU + 1) * 64;   // and the panel wave
    // waves per SIMD asked of the compiler; its registers allow 4 up to NT = 3,
    // 2 at 4, 3 at 5, 7 and 8 (5 to 13 spilled), 1 at 6, 2 from 9 on (76 and 119
    // spilled at 13 and 14: 260 and 288 bytes a lane)
    static constexpr int WPE = NT <= 4 ? 4 : NT <= 9 ? 3 : 2;
    static constexpr int NP = 16 * NT;
    static constexpr int RPL = (NP + 63) / 64;      // panel rows per lane
    static constexpr bool EXACT = NT <= GJ_V_APPROX;  // pivot by the full |a| (else to 2^-12)
    // row strides in doubles: 8 mod 16, so that four rows of 16 consecutive
    // values cover every LDS bank evenly (and 8 spare entries)
    static constexpr int LS = NP + 8;
    static constexpr int PS = 16 * CT + 8;
    // doubles: the panel handed over, F of two panels, pivot rows per wave
    static constexpr int MAIN = 3 * 16 * LS + NU * 16 * PS;
    // output staging (over all that): QC rows of D^-1
    static constexpr int SS = NP + 2;
    static constexpr int QC = MAIN / SS < NP ? MAIN / SS : NP;
};

// Flag accesses in LDS.  The LDS executes the DS instructions of one wave in
// program order, so a flag written after a wave's data accesses is seen only
// once they are done, and data read after a flag was seen is the data
// published before it; only the compiler has to keep the order (the
// signal fences), no wait is needed.
__device__ __forceinline__ int flag_load(int* f) {
    const int v = __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ void flag_store(int* f, int v) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __hip_atomic_store(f, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Waits until *f >= v; false when the bound on the wait was reached.
__device__ __forceinline__ bool flag_wait(int* f, int v) {
    for (int it = 0; it < (1 << 22); ++it)
        if (flag_load(f) >= v) return true;
    return false;
}

template <int NT>
struct GJShared {
    double main[GJT<NT>::MAIN];
    double pvs[GJT<NT>::NP];   // pivot of step k
    double row[16];            // the panel wave's pivot row
    int perm[GJT<NT>::NP];     // row of step k
    uint32_t ord[16][4];       // byte i / 16 of row i % 16: 1 + the step that took row i (0: none)
    int xready;                // last panel handed over to the panel wave
    int xfree;                 // last panel whose columns were taken from there
    int bad;                   // 1: zero pivot, 2: non-finite pivot (or a wait that gave up)
    int bad_panel;             // the pivot's panel (np: none so far)
    // (the panel first: its addresses are constants within an LDS
    // instruction's offset)
    __device__ double* X() { return main; }
    __device__ double* F(int p) { return main + (1 + (p & 1)) * 16 * GJT<NT>::LS; }
    __device__ uint8_t& ord_of(int i) { return ((uint8_t*)ord)[(i & 15) * 16 + (i >> 4)]; }
};

// One stage of the wave maximum of a 32-bit key: quad swaps, half-row and
// row mirrors inside rows of 16 lanes, then the row results passed on to the
// next row and the upper half; lane 63 ends with the maximum.
template <int STAGE>
__device__ __forceinline__ uint32_t umax_stage(uint32_t x) {
    constexpr int ctrl[6] = {0xB1, 0x4E, 0x141, 0x140, 0x142, 0x143};
    return max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl[STAGE], STAGE == 4 ? 0xa : STAGE == 5 ? 0xc : 0xf,
                                                        0xf, false));
}

// What one inversion reads of its Job.
struct GJArgs {
    const void* C;
    double* Dinv;
    double* logdet;
    int8_t* sign;
    uint32_t* status;
    int64_t c1_stride;  // values between walkers' C_1
    int n, spin, mode;
};
__host__ __device__ __forceinline__ GJArgs gj_args(const Job& j) {
    return GJArgs{j.C, j.Dinv, j.logdet, j.sign, j.status, c1_stride(j), j.n, j.spin, j.mode};
}

// Search keys of an entry x of row i.  EXACT: the high word of |x| above a
// set bit (rows alike in it are told apart by their low words afterwards);
// else exponent and 20 significand bits above 255 - i, which gives the row
// back and the smallest of rows alike.
template <bool EXACT>
__device__ __forceinline__ uint32_t gj_key(double x, int i) {
    const uint32_t hi = (uint32_t)((uint64_t)__double_as_longlong(x) >> 32);
    return EXACT ? hi << 1 | 1u : (hi & 0x7fffff00u) | (uint32_t)(255 - i);
}
// Whether the largest key is no normal finite number's.
template <bool EXACT>
__device__ __forceinline__ bool gj_odd(uint32_t key) {
    return EXACT ? key - 0x00200000u >= 0xffc00000u : key - 0x00100000u >= 0x7fe00000u;
}
template <bool EXACT>
__device__ __forceinline__ double gj_recip(double pv) {
    if constexpr (EXACT) return 1.0 / pv;
    // hardware reciprocal and two Newton steps
    double inv = __builtin_amdgcn_rcp(pv);
    inv = fma(inv, fma(-pv, inv, 1.0), inv);
    return fma(inv, fma(-pv, inv, 1.0), inv);
}

// A panel one of whose largest keys was no ordinary number's: its steps on
// the panel in LDS, with NaN left out of the search.  Returns 0, or 1 where no
// row or a zero is left, 2 where the pivot is infinite.  The identity's steps
// past n are taken as they are known to be: the infinite reciprocal of a
// subnormal pivot has left NaN in its rows by then (0 times infinity).
template <int NT>
__device__ __forceinline__ int gjt_panel_careful(GJShared<NT>& S, int p, int n, int lane) {
    using P = GJT<NT>;
    constexpr int LS = P::LS;
    const int n16 = (n + 15) & ~15;
    double *X = S.X(), *F = S.F(p);
#pragma unroll 1
    for (int k = 0; k < min(16, n - 16 * p); ++k) {
        uint64_t best = 0;  // |x| and 255 - i, or the key, to be largest
        int at = 0;
#pragma unroll 1
        for (int row = lane; row < n16; row += 64) {
            const double x = X[k * LS + row];
            if (S.ord_of(row) != 0 || x != x) continue;
            const uint64_t b = P::EXACT ? ((uint64_t)__double_as_longlong(x) << 1 | 1u) : gj_key<false>(x, row);
            if (b > best) { best = b; at = row; }
        }
#pragma unroll 1
        for (int o = 1; o < 64; o <<= 1) {
            const uint64_t ob = (uint64_t)__shfl_xor((unsigned long long)best, o);
            const int oa = __shfl_xor(at, o);
            if (ob > best || (ob == best && oa < at)) { best = ob; at = oa; }
        }
        if (best == 0) return 1;
        const double pv = X[k * LS + at];
        if (pv == 0.0) return 1;
        if (!isfinite(pv)) return 2;
        const double inv = gj_recip<P::EXACT>(pv);
        if (lane == 0) {
            S.pvs[16 * p + k] = pv;
            S.perm[16 * p + k] = at;
            S.ord_of(at) = (uint8_t)(16 * p + k + 1);
        }
#pragma unroll 1
        for (int row = lane; row < P::NP; row += 64) {
            const double x = X[k * LS + row];
            const double f = row == at ? 0.0 : -(x * inv);
            F[k * LS + row] = f;
#pragma unroll 1
            for (int c = k + 1; c < 16; ++c)
                if (row != at) X[c * LS + row] = fma(f, X[c * LS + at], X[c * LS + row]);
            X[k * LS + row] = fma(f, pv + 1.0, x);
        }
    }
    if (16 * p + lane >= n && lane < 16) {
        S.pvs[16 * p + lane] = 1.0;
        S.perm[16 * p + lane] = 16 * p + lane;
        S.ord_of(16 * p + lane) = (uint8_t)(16 * p + lane + 1);
    }
#pragma unroll 1
    for (int q = max(n - 16 * p, 0) * LS + lane; q < 16 * LS; q += 64) F[q] = 0.0;
    return 0;
}

// The panel wave.  Lane l holds rows l + 64 r of the panel's 16 columns.  One
// wave issues an instruction in about five cycles, a branch costs 25 and an
// LDS write 16 per eight bytes of a lane, so a step costs what it issues:
// each lane takes the reciprocal of its own candidate during the maximum, the
// next column is updated and searched first (its pivot-row entry comes by
// lane exchange), the pivot row reaches the columns after it through LDS, and
// the stages of the maximum stand between their updates.  A largest key
// that is no ordinary number's is only noted; the panel is then done again.
template <int NT>
__device__ __forceinline__ bool gjt_panels(const GJArgs& j, GJShared<NT>& S, int w, int lane) {
    using P = GJT<NT>;
    constexpr int RPL = P::RPL, LS = P::LS;
    constexpr bool EXACT = P::EXACT;
    const int n = j.n, np = (n + 15) >> 4;
    uint64_t open[RPL];  // rows not yet used
    int mine[RPL];       // this lane's rows (those past NP: the spare entries)
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        const int row = lane + 64 * r;
        open[r] = __ballot(row < (NT == 1 ? n : 16 * np));
        mine[r] = row < P::NP ? row : P::NP + (lane & 7);
    }
    int inversions = 0;  // of the pivot permutation, by lanes
    if constexpr (NT == 1) {  // the identity's steps past n, which are not taken
        for (int k = n; k < 16; ++k) S.F(0)[k * LS + mine[0]] = 0.0;
        if (lane >= n && lane < 16) {
            S.pvs[lane] = 1.0;
            S.perm[lane] = lane;
        }
    }
    __builtin_amdgcn_s_setprio(3);
#pragma unroll 1
    for (int p = 0; p < np; ++p) {
        uint64_t before[RPL];  // the open rows as the panel begins
#pragma unroll
        for (int r = 0; r < RPL; ++r) before[r] = open[r];
        int code = flag_wait(&S.xready, p) ? 0 : 2;
        double *Xb = S.X(), *Fb = S.F(p);
        double X[RPL][16];
#pragma unroll
        for (int r = 0; r < RPL; ++r)
#pragma unroll
            for (int c = 0; c < 16; ++c) X[r][c] = Xb[c * LS + mine[r]];
        uint32_t kr[RPL], key = 0;   // the searched column's keys, their largest
        double cand = 0, linv = 0;   // this lane's best candidate, its reciprocal
        auto keys = [&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const uint32_t q = gj_key<EXACT>(X[r][k], lane + 64 * r);
                kr[r] = __builtin_amdgcn_inverse_ballot_w64(open[r]) ? q : 0u;
                const bool up = r == 0 || kr[r] > key;
                cand = up ? X[r][k] : cand;
                key = up ? kr[r] : key;
            }
        };
        bool odd = false;
        keys(std::integral_constant<int, 0>{});
        linv = gj_recip<EXACT>(cand);
        static_for<0, 6>([&](auto sc) __attribute__((always_inline)) { key = umax_stage<decltype(sc)::value>(key); });
        static_for<0, 16>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            if (NT == 1 && k >= n) return;  // (a whole panel of a tiny matrix is mostly identity)
            const uint32_t sk = (uint32_t)__builtin_amdgcn_readlane((int)key, 63);
            odd |= gj_odd<EXACT>(sk);
            uint64_t m[RPL];  // the pivot's lane
            int rs = 0, ls;
            double inv, pv;
            if constexpr (EXACT) {
                int cnt = 0;
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    m[r] = __ballot(kr[r] == sk);
                    cnt += __popcll(m[r]);
                }
                if (__builtin_expect(cnt != 1, 0)) {
                    // alike in the high word: the largest low word, then the
                    // smallest row
                    uint32_t lo = 0;
#pragma unroll
                    for (int r = 0; r < RPL; ++r)
                        if (kr[r] == sk) lo = max(lo, (uint32_t)__double_as_longlong(X[r][k]));
                    static_for<0, 6>([&](auto sc) __attribute__((always_inline)) { lo = umax_stage<decltype(sc)::value>(lo); });
                    lo = (uint32_t)__builtin_amdgcn_readlane((int)lo, 63);
                    bool found = false;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) {
                        const uint64_t b = __ballot(kr[r] == sk && (uint32_t)__double_as_longlong(X[r][k]) == lo);
                        m[r] = found ? 0 : b & (0 - b);
                        found |= b != 0;
                    }
                    double y = X[0][k];
#pragma unroll
                    for (int r = 1; r < RPL; ++r) y = m[r] ? X[r][k] : y;
                    cand = y;
                    linv = 1.0 / y;
                }
#pragma unroll
                for (int r = 1; r < RPL; ++r) rs = m[r] ? r : rs;
                uint64_t mm = m[0];
#pragma unroll
                for (int r = 1; r < RPL; ++r) mm |= m[r];
                ls = __builtin_ctzll(mm | 1ull << 63);
            } else {
                const int si = (int)(~sk & 0xffu);
                rs = si >> 6;
                ls = si & 63;
#pragma unroll
                for (int r = 0; r < RPL; ++r) m[r] = rs == r ? 1ull << ls : 0;
            }
            inv = readlane_f64(linv, ls);
            pv = readlane_f64(cand, ls);
            double x1 = 0.0;  // the pivot row's entry of the next column
            if constexpr (k + 1 < 16) {
                double y[RPL];
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    y[r] = X[r][k + 1];
                    asm("" : "+v"(y[r]));  // (values, not addresses, are selected)
                }
#pragma unroll
                for (int r = 1; r < RPL; ++r) y[0] = rs == r ? y[r] : y[0];
                x1 = readlane_f64(y[0], ls);
            }
            // the pivot row of the columns after the next one, by way of LDS
            constexpr int c0 = (k + 2) & ~1;
            auto put = [&](auto rc) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                if (__builtin_amdgcn_inverse_ballot_w64(m[r])) {
#pragma unroll
                    for (int c = c0; c < 16; c += 2) *(f64x2*)&S.row[c] = f64x2{X[r][c], X[r][c + 1]};
                    S.pvs[16 * p + k] = pv;
                    S.perm[16 * p + k] = lane + 64 * r;
                }
                if constexpr (RPL > 1) asm volatile("; pivot row %0" ::"n"(r));
            };
            using R0 = std::integral_constant<int, 0>;
            using R1 = std::integral_constant<int, (RPL > 1 ? 1 : 0)>;
            using R2 = std::integral_constant<int, (RPL > 2 ? 2 : 0)>;
            using R3 = std::integral_constant<int, (RPL > 3 ? 3 : 0)>;
            if constexpr (RPL == 1) put(R0{});
            else if constexpr (RPL == 2) {
                if (rs == 0) put(R0{});
                else put(R1{});
            } else {
                if (rs < 2) {
                    if (rs == 0) put(R0{});
                    else put(R1{});
                } else {
                    if (RPL == 3 || rs == 2) put(R2{});
                    else put(R3{});
                }
            }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            double rv[16], f[RPL];
#pragma unroll
            for (int c = k + 2; c < 16; ++c) rv[c] = S.row[c];
            const double pv1 = pv + 1.0;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const double fr = -(X[r][k] * inv);
                f[r] = __builtin_amdgcn_inverse_ballot_w64(m[r]) ? 0.0 : fr;
                open[r] &= ~m[r];
                X[r][k] = fma(f[r], pv1, X[r][k]);
                if constexpr (k + 1 < 16) X[r][k + 1] = fma(f[r], x1, X[r][k + 1]);
            }
            auto col = [&](auto cc) __attribute__((always_inline)) {
                constexpr int c = decltype(cc)::value;
                if constexpr (c < 16) {
#pragma unroll
                    for (int r = 0; r < RPL; ++r) X[r][c] = fma(f[r], rv[c], X[r][c]);
                }
            };
            auto put_f = [&](int r) __attribute__((always_inline)) {
                Fb[k * LS + mine[r]] = f[r];
            };
            if constexpr (k + 1 < 16) {
                keys(std::integral_constant<int, k + 1>{});
                linv = gj_recip<EXACT>(cand);
                static_for<0, 6>([&](auto sc) __attribute__((always_inline)) {
                    constexpr int st = decltype(sc)::value;
                    key = umax_stage<st>(key);
                    if constexpr (st < RPL) put_f(st);
                    if constexpr (st >= 2) {  // (the pivot row is back from LDS)
                        col(std::integral_constant<int, k + 2 * st - 2>{});
                        col(std::integral_constant<int, k + 2 * st - 1>{});
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                static_for<k + 10, (k + 10 < 16 ? 16 : k + 10)>(col);
            } else {
#pragma unroll
                for (int r = 0; r < RPL; ++r) put_f(r);
            }
        });
        if (__builtin_expect(odd || code, 0)) {
            if (!code) code = gjt_panel_careful<NT>(S, p, n, lane);
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int row = lane + 64 * r;
                open[r] = __ballot(row < 16 * np && S.ord_of(row & 255) == 0);
            }
            if (code && lane == 0) {
                S.bad = code;
                S.bad_panel = p;
            }
        } else {
            // the panel's columns, for the wave that owns them
#pragma unroll
            for (int r = 0; r < RPL; ++r)
#pragma unroll
                for (int c = 0; c < 16; ++c) Xb[c * LS + mine[r]] = X[r][c];
            if (lane < 16) S.ord_of(S.perm[16 * p + lane]) = (uint8_t)(16 * p + lane + 1);
        }
        __syncthreads();
        if (code) return false;
        // the inversions that this panel's rows add to the permutation, lane
        // k < 16 those of step k (the smaller rows still open when it was
        // taken)
        {
            const int row = S.perm[16 * p + (lane & 15)];
            int below = 0;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int d = row - 64 * r;
                below += __popcll(before[r] & (d >= 64 ? ~0ull : d > 0 ? (1ull << d) - 1 : 0ull));
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) below -= k < lane && __builtin_amdgcn_readlane(row, k) < row;
            inversions += lane < (NT == 1 ? n : 16) ? below : 0;
        }
    }
    __builtin_amdgcn_s_setprio(0);
    // log|det| = sum log|pivot|, by rows: those of a lane, then the lanes (up
    // to 128 rows), or lanes 0 .. 63 of each 64 rows, then those in order
    double ld = 0.0, part = 0.0;
    int neg = inversions;
#pragma unroll 1
    for (int r = 0; r < RPL; ++r) {
        const int row = lane + 64 * r;
        double lg = 0.0;
        if (row < n) {
            const double v = S.pvs[(int)S.ord_of(row) - 1];
            lg = log(fabs(v));
            neg += v < 0.0;
        }
        part += lg;
        if (EXACT && r + 1 < RPL) continue;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) part += __shfl_xor(part, o);
        ld += part;
        part = 0.0;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) neg += __shfl_xor(neg, o);
    if (lane == 0) {
        if (j.logdet) j.logdet[2 * (size_t)w + j.spin] = ld;
        if (j.sign) j.sign[2 * (size_t)w + j.spin] = (neg & 1) ? -1 : 1;
        if (j.status && !isfinite(ld)) atomicOr(j.status + w, QSL_STATUS_NONFINITE);
    }
    return true;
}

// Register tiles of an updating wave from C_1[e][i], the identity past n (so
// that the last panel has 16 columns; its inverse and determinant add
// nothing).  A whole column tile's loads are in flight at once.  A row is
// read past its end (into the next row, or the gradient block after C_1)
// rather than clamped, except where the matrix is too small for that (NT <= 2
// also serves n < 8; a larger NT has n >= 8, and 4 n n + n >= GJ_READ_PAST).
template <int NT, typename Tin>
__device__ __forceinline__ void gjt_load(const Tin* __restrict__ C1, int n, int u, int lane,
                                         f64x4 (&acc)[NT][GJT<NT>::CT]) {
    using P = GJT<NT>;
    const int li = lane & 15, lg = lane >> 4;
#pragma unroll
    for (int ct = 0; ct < P::CT; ++ct) {
        Tin v[4][NT];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = 16 * (u + P::NU * ct) + lg + 4 * r;
            const Tin* row = C1 + min(e, n - 1) * n;
#pragma unroll
            for (int t = 0; t < NT; ++t) v[r][t] = gmem(row)[NT <= 2 ? min(16 * t + li, n - 1) : 16 * t + li];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = 16 * (u + P::NU * ct) + lg + 4 * r;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t][ct][r] = e < n && 16 * t + li < n ? (double)v[r][t] : (e == 16 * t + li ? 1.0 : 0.0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Staged rows q0 .. of D^-1 to memory, between the workgroup's barriers.
template <int NT>
__device__ __forceinline__ void gjt_copy_out(const GJArgs& j, GJShared<NT>& S, int w, int q0, int wave, int lane) {
    using P = GJT<NT>;
    const int n = j.n, rows = min(P::QC, n - q0);
    double* Dw = j.Dinv + (size_t)w * n * n + (size_t)q0 * n;
    __syncthreads();
    for (int rr = wave; rr < rows; rr += P::NU + 1)
        for (int cc = lane; cc < n; cc += 64) gmem(Dw)[rr * n + cc] = S.main[rr * P::SS + cc];
    __syncthreads();
}

// An updating wave: its tiles through every panel, then D^-1 into the
// staging rows.  Leaves after a bad pivot.
template <int NT>
__device__ __forceinline__ void gjt_update(const GJArgs& j, GJShared<NT>& S, int w, int u, int lane) {
    using P = GJT<NT>;
    constexpr int CT = P::CT, NU = P::NU, LS = P::LS, PS = P::PS;
    static_assert(CT == 2, "two column tiles per wave");
    const int li = lane & 15, lg = lane >> 4;
    const int n = j.n, np = (n + 15) >> 4;
    f64x4 acc[NT][CT];
    if (j.mode == QSL_FP64) gjt_load<NT>((const double*)j.C + (size_t)w * j.c1_stride, n, u, lane, acc);
    else gjt_load<NT>((const float*)j.C + (size_t)w * j.c1_stride, n, u, lane, acc);
    // pivot-row entries of this wave's columns, [k][16 ct + 4 (e % 4) + e / 4]
    double* pr = S.main + 3 * 16 * LS + u * 16 * PS;
    double* Xw = S.X() + lg * LS + li;
    // column tile ct to the panel wave
    auto stage_tile = [&](auto ctc, int p) __attribute__((always_inline)) {
        constexpr int ct = decltype(ctc)::value;
#pragma unroll
        for (int ti = 0; ti < NT; ++ti)
#pragma unroll
            for (int r = 0; r < 4; ++r) Xw[4 * r * LS + 16 * ti] = acc[ti][ct][r];
        if (lane == 0) flag_store(&S.xready, p);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    if (u == 0) stage_tile(I0{}, 0);
#pragma unroll 1
    for (int p = 0; p < np; ++p) {
        __syncthreads();  // F of panel p is published; every update of panel p - 1 is done
        // (the panel wave may already be past panel p + 1: a pivot that fails
        // there ends this loop for all waves at the next barrier alike)
        if (S.bad_panel <= p) return;
        const double* Fp = S.F(p);
        const double* L = Fp + lg * LS + li;
        // the panel's columns come back as their own steps left them
        if (p % NU == u) {
            static_for<0, CT>([&](auto ctc) __attribute__((always_inline)) {
                constexpr int ct = decltype(ctc)::value;
                if (p == u + NU * ct) {
#pragma unroll
                    for (int ti = 0; ti < NT; ++ti)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[ti][ct][r] = Xw[4 * r * LS + 16 * ti];
                }
            });
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            if (lane == 0) flag_store(&S.xfree, p);
        }
        if (NT == 1 && n == 1) break;  // no further step
        // the pivot rows' entries of this wave's columns
        {
            const uint4 o4 = *(const uint4*)S.ord[li];
            const uint32_t ov[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
            for (int ti = 0; ti < NT; ++ti) {
                const uint32_t k = ((ov[ti >> 2] >> (8 * (ti & 3))) & 0xffu) - (uint32_t)(16 * p + 1);
                if (k < 16u) {
                    f64x4* pk = (f64x4*)(pr + k * PS + 4 * lg);
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) pk[4 * ct] = acc[ti][ct];
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        // w from them: lane (lg, li) of register b holds step 4 b + lg of
        // column li, which is also how the products read it as an operand;
        // one product per step m, its multipliers F_m[p_k] masked to the rows
        // k > m (entries of an own column up to its own step start and stay 0)
        const int prow = S.perm[16 * p + li];
        double* pw = pr + lg * PS + 4 * (li & 3) + (li >> 2);
        auto solve = [&](int ct) __attribute__((always_inline)) {
            const bool own = p == u + NU * ct;
            f64x4 wv;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const double x = pw[4 * b * PS + 16 * ct];
                wv[b] = own && 4 * b + lg <= li ? 0.0 : x;
            }
            static_for<0, 4>([&](auto bc) __attribute__((always_inline)) {
                constexpr int b = decltype(bc)::value;
                const double nb = Fp[(4 * b + lg) * LS + prow];
                static_for<0, (b == 3 ? 3 : 4)>([&](auto kc) __attribute__((always_inline)) {
                    constexpr int kk = decltype(kc)::value;
                    const double a = lg == kk && li > 4 * b + kk ? nb : 0.0;
                    wv = __builtin_amdgcn_mfma_f64_16x16x4f64(a, wv[b], wv, 0, 0, 0);
                });
            });
#pragma unroll
            for (int b = 0; b < 4; ++b) pw[4 * b * PS + 16 * ct] = wv[b];
        };
        const bool next = p + 1 < np && (p + 1) % NU == u, second = p + 1 >= NU;
        // the next panel's columns in a pass of their own first, handed over
        // before the rest (the wave four further on runs on the same SIMD
        // and lets them pass)
        if (next) __builtin_amdgcn_s_setprio(2);
        if (NU > 4 && p + 1 < np && (p + 1) % NU == (u ^ 4)) flag_wait(&S.xready, p + 1);
#pragma unroll 1
        for (int pass = next ? 0 : 1; pass < 2; ++pass) {
            const bool do0 = pass == 0 ? !second : u != p + 1;
            const bool do1 = pass == 0 ? second : u + NU < NT && u + NU != p + 1;
#pragma unroll 1
            for (int ct = 0; ct < CT; ++ct)
                if (ct == 0 ? do0 : do1) solve(ct);
            __builtin_amdgcn_wave_barrier();
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll 1
            for (int kk = 0; kk < 4; ++kk) {
                const double* Lk = L + 4 * kk * LS;
                if (do0) {
                    const double a = pw[4 * kk * PS];
#pragma unroll
                    for (int ti = 0; ti < NT; ++ti)
                        acc[ti][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Lk[16 * ti], acc[ti][0], 0, 0, 0);
                }
                if (do1) {
                    const double a = pw[4 * kk * PS + 16];
#pragma unroll
                    for (int ti = 0; ti < NT; ++ti)
                        acc[ti][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Lk[16 * ti], acc[ti][1], 0, 0, 0);
                }
            }
            if (pass == 0) {
                // (gave up: goes on to the same barriers, and all ends as NaN)
                if (!flag_wait(&S.xfree, p) && lane == 0) S.bad = 2;
                if (second) stage_tile(I1{}, p + 1);
                else stage_tile(I0{}, p + 1);
                __builtin_amdgcn_s_setprio(0);
            }
        }
    }
    __syncthreads();  // the panels are no longer read
    const uint4 o4 = *(const uint4*)S.ord[li];
    const uint32_t ov[4] = {o4.x, o4.y, o4.z, o4.w};
    auto step_of = [&](int ti) __attribute__((always_inline)) { return (int)((ov[ti >> 2] >> (8 * (ti & 3))) & 0xffu) - 1; };
    // D^-1[k][p_j] = M[p_k][j] / pivot(k), staged QC rows at a time.  The
    // pivot entries were left at pv during the elimination (the pivot row is
    // never scaled); their value in the scaled representation is 1, and later
    // updates of them only added terms: M[p_k][k] += 1 - pv_k
    int pd[CT][4];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = 16 * (u + NU * ct) + lg + 4 * r;
            pd[ct][r] = e < n ? S.perm[e] : P::NP;  // (past n: a spare column)
        }
#pragma unroll 1
    for (int q0 = 0; q0 < n; q0 += P::QC) {
#pragma unroll
        for (int ti = 0; ti < NT; ++ti) {
            const int k = step_of(ti);
            if ((uint32_t)(k - q0) < (uint32_t)P::QC) {
                const double pv = S.pvs[k], rs = 1.0 / pv;
                double* to = S.main + (k - q0) * P::SS;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const double d = 16 * (u + NU * ct) + lg + 4 * r == k ? 1.0 - pv : 0.0;
                        const double x = acc[ti][ct][r] + d;
                        to[pd[ct][r]] = x * rs;
                    }
            }
        }
        gjt_copy_out<NT>(j, S, w, q0, u, lane);
    }
}

template <int NT>
__device__ __forceinline__ void gjt_body(const GJArgs& j, int w) {
    using P = GJT<NT>;
    __shared__ __align__(32) GJShared<NT> S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 64) ((uint32_t*)S.ord)[tid] = 0u;
    if (tid == 0) { S.xready = S.xfree = -1; S.bad = 0; S.bad_panel = (j.n + 15) >> 4; }
    __syncthreads();
    if (wave == P::NU) {
        if (gjt_panels<NT>(j, S, w, lane)) {
            __syncthreads();
            for (int q0 = 0; q0 < j.n; q0 += P::QC) gjt_copy_out<NT>(j, S, w, q0, wave, lane);
        }
    } else {
        gjt_update<NT>(j, S, w, wave, lane);
    }
    if (S.bad) {
        // undefined inverse: NaN, sign = 0, log|det| = -inf (a zero pivot) or NaN
        const size_t nn = (size_t)j.n * j.n;
        double* Dw = j.Dinv + (size_t)w * nn;
        for (size_t q = tid; q < nn; q += P::THREADS) Dw[q] = __longlong_as_double(0x7ff8000000000000ll);
        if (tid == 64 * P::NU) {  // (the panel wave, which may have written a log|det|)
            if (j.logdet) j.logdet[2 * (size_t)w + j.spin] = S.bad == 1 ? -INFINITY : __longlong_as_double(0x7ff8000000000000ll);
            if (j.sign) j.sign[2 * (size_t)w + j.spin] = 0;
            if (j.status) atomicOr(j.status + w, S.bad == 1 ? QSL_STATUS_SINGULAR : QSL_STATUS_NONFINITE);
        }
    }
}

// One workgroup per matrix: of the Job described by value, or (jobs) of a
// batched launch.
template <int NT>
__global__ __launch_bounds__(GJT<NT>::THREADS, GJT<NT>::WPE) void gjt_kernel(GJArgs a, const Job* jobs, const int* prefix, int njobs) {
    int w = blockIdx.x;
    if (jobs) {
        const int ji = __builtin_amdgcn_readfirstlane(find_job(prefix, njobs, w));
        w -= prefix[ji];
        a = gj_args(jobs[ji]);
    }
    gjt_body<NT>(a, w);
}

__global__ void empty_spin_kernel(int64_t W, int spin, double* logdet, int8_t* sign) {
    int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w < W) {
        if (logdet) logdet[2 * w + spin] = 0.0;
        if (sign) sign[2 * w + spin] = 1;
    }
}

// Variants by matrix size: 0 .. 13 register-resident, n <= 16 (v + 1);
// GJ_V_BLOCKED: blocked, n <= 1024.
int gj_variant(int n) { return gj_blocked(n) ? GJ_V_BLOCKED : (std::max(n, 1) - 1) / 16; }
int gj_job_variant(const Job& j) {
    const int v = gj_variant(j.n);
    return v == GJ_V_BLOCKED ? v : std::min(GJ_V_BLOCKED - 1, v + std::max(0, j.gj_bias));
}

void gj_share_variant(int (&v)[2], const int (&n)[2]) {
    const auto kind = [](int x) { return x == GJ_V_BLOCKED ? 2 : x >= GJ_V_APPROX ? 1 : 0; };
    if (v[0] >= 0 && v[1] >= 0 && kind(v[0]) == kind(v[1]) && std::min(n[0], n[1]) >= 8) v[0] = v[1] = std::max(v[0], v[1]);
}

static hipError_t gj_dispatch(const GJArgs& a, int v, const Job* jobs, const int* prefix, int njobs, int grid,
                              hipStream_t st) {
    switch (v) {
#define QSL_GJ(NT)                                                                                        \
    case NT - 1: gjt_kernel<NT><<<(unsigned)grid, GJT<NT>::THREADS, 0, st>>>(a, jobs, prefix, njobs); break;
        QSL_GJ(1) QSL_GJ(2) QSL_GJ(3) QSL_GJ(4) QSL_GJ(5) QSL_GJ(6) QSL_GJ(7)
        QSL_GJ(8) QSL_GJ(9) QSL_GJ(10) QSL_GJ(11) QSL_GJ(12) QSL_GJ(13) QSL_GJ(14)
#undef QSL_GJ
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gj(const Job& j0, hipStream_t st) {
    if (j0.W <= 0) return hipSuccess;
    Job j = j0;
    j.gx = (int)j.W; j.gy = 1; j.gz = 1;
    if (j.n == 0) {
        empty_spin_kernel<<<(unsigned)((j.W + 255) / 256), 256, 0, st>>>(j.W, j.spin, j.logdet, j.sign);
        return hipGetLastError();
    }
    if (j.n > GJ_NMAX) return hipErrorInvalidValue;
    const int v = gj_job_variant(j);
    if (v == GJ_V_BLOCKED) return launch_gjb(j, st);
    return gj_dispatch(gj_args(j), v, nullptr, nullptr, 0, (int)j.W, st);
}

// One batched launch of GJ variant v over Jobs whose n all fit it (the
// plan launches each variant present in its batch once; the blocked
// variant is a sequence of launches over panels, see qsl_gjb.hip).
hipError_t launch_gj_batched(int v, const Job* jobs, const int* prefix, int njobs, int grid, hipStream_t st) {
    if (v < 0 || v >= GJ_V_BLOCKED) return hipErrorInvalidValue;
    if (grid <= 0) return hipSuccess;
    return gj_dispatch(GJArgs{}, v, jobs, prefix, njobs, grid, st);
}

}  // namespace qsl
