// Several determinants: Psi_det = sum_K c_K Det_K_up Det_K_dn (the Psi_T
// equation of section "The quantum Monte Carlo method"), each determinant
// built from n_s orbitals (columns) of one orbital set of n_orb >= n_s MOs
// per spin.  The products C_n = A B_n run once for the whole orbital set
// (equation (abc)); each determinant gathers its columns of C, is inverted
// in FP64 (log|det|, sign, D^-1) and gives its drift and Laplacian ratio;
// the determinants are then combined per walker:
//   log|Psi_det| = m + log|S|,  S = sum_K s_K |c_K| e^(L_K - m),
//   L_K = log|Det_K_up| + log|Det_K_dn|,  m = max_K (L_K + log|c_K|) - log|c_K| shift,
//   drift_e = sum_K w_K drift_K(e),  lap_e = sum_K w_K lap_K(e),
//   w_K = c_K Det_K_up Det_K_dn / Psi_det,
// since grad_e and lap_e act on the one determinant of electron e's spin.
#include <math.h>

#include <algorithm>

#include "qsl_internal.h"

namespace qsl {

// The values C_1 of one determinant's columns out of the orbital set, which
// the inversion reads: c1[K][w][e][i] = C_orb[w][0][e][occ_K[i]], for the
// determinants K0 .. K0 + gridDim.y - 1 and both spins (blockIdx.z).
struct MDGather {
    int64_t W;
    int n[2], nmo[2], off[2];  // electrons, orbitals, the spin's first entry of an occupation
    int N;
    const int* occ;            // [n_det][N], from determinant K0
    const void* corb[2];
    void* c1[2];
};
template <typename T>
__global__ void gather_det_kernel(MDGather g) {
    const int s = blockIdx.z, n = g.n[s];
    const int64_t total = g.W * n * n;
    const int* __restrict__ occ = g.occ + (size_t)blockIdx.y * g.N + g.off[s];
    const T* __restrict__ corb = (const T*)g.corb[s];
    T* __restrict__ c1 = (T*)g.c1[s] + blockIdx.y * total;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total; q += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(q % n);
        const int64_t row = q / n;  // (w, e)
        c1[q] = corb[(row / n * 5 * n + row % n) * g.nmo[s] + occ[i]];
    }
}

// The Jobs of a group of determinants: two lists for the inversion and two for
// the drift and Laplacian (the first holds both spins, or each holds one), in
// determinant order.  job[s] are determinant 0 of the group's; the others' pointers lie
// `step` apart.
struct MDLists {
    char* list[4];           // Jobs, then the block prefix
    int spins[4], total[4];  // per list: spins in it, blocks per determinant
    int slot[4][2], first[4][2], blocks[4][2];  // place (-1: not in the list), first block, blocks of each spin
    int group;              // determinants
    int64_t W, N;
    int64_t c1_bytes[2], dinv[2];
    const void* corb[2];
};
__global__ void md_lists_kernel(Job a, Job b, MDLists m) {
    const int K = blockIdx.x, l = threadIdx.x >> 7, s = (threadIdx.x >> 6) & 1;
    if ((threadIdx.x & 63) != 0 || m.slot[l][s] < 0) return;
    Job j = s ? b : a;
    j.C = (char*)j.C + K * m.c1_bytes[s];
    j.Dinv += K * m.dinv[s];
    j.logdet += K * m.W * 2;
    j.sign += K * m.W * 2;
    j.drift += K * m.W * m.N * 3;
    j.lap += K * m.W * m.N;
    j.status += K * m.W;
    if (j.occ) j.occ += K * m.N;
    if (l >= 2) j.C = const_cast<void*>(m.corb[s]);
    j.gx = m.blocks[l][s];
    j.gy = j.gz = 1;
    const int at = K * m.spins[l] + m.slot[l][s];
    int* prefix = (int*)(m.list[l] + (size_t)m.group * m.spins[l] * sizeof(Job));
    ((Job*)m.list[l])[at] = j;
    prefix[at] = K * m.total[l] + m.first[l][s];
    if (at + 1 == m.group * m.spins[l]) prefix[at + 1] = m.group * m.total[l];
}

struct MDComb {
    int64_t W;
    int N, n_up, n_det;
    const double* coef;       // [n_det]
    const double* logdet;     // [n_det][W][2]
    const int8_t* sign;       // [n_det][W][2]
    const double* drift;      // [n_det][W][N][3]
    const double* lap;        // [n_det][W][N]
    const uint32_t* dstatus;  // [n_det][W]
    const uint32_t* st0;      // [W] near ties of the products
    double* out_logpsi;       // [W]
    int8_t* out_sign;         // [W]
    double* out_drift;        // [W][N][3]
    double* out_lap;          // [W][N]
    uint32_t* out_status;     // [W]
};

// One thread per (walker, electron): the determinants' weights from their
// log|det| (max-shifted), then the weighted drift and Laplacian ratio.
__global__ void combine_kernel(MDComb c) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= c.W * c.N) return;
    const int64_t w = q / c.N;
    const int e = (int)(q % c.N);
    double m = -INFINITY;
    for (int K = 0; K < c.n_det; ++K) {
        const int8_t s = c.sign[(K * c.W + w) * 2] * c.sign[(K * c.W + w) * 2 + 1];
        if (s == 0 || c.coef[K] == 0.0) continue;
        const double L = c.logdet[(K * c.W + w) * 2] + c.logdet[(K * c.W + w) * 2 + 1] + log(fabs(c.coef[K]));
        m = fmax(m, L);
    }
    double S = 0.0;
    for (int K = 0; K < c.n_det; ++K) {
        const int8_t s = c.sign[(K * c.W + w) * 2] * c.sign[(K * c.W + w) * 2 + 1];
        if (s == 0 || c.coef[K] == 0.0) continue;
        const double L = c.logdet[(K * c.W + w) * 2] + c.logdet[(K * c.W + w) * 2 + 1] + log(fabs(c.coef[K]));
        S += (c.coef[K] > 0 ? s : -s) * exp(L - m);
    }
    double g0 = 0.0, g1 = 0.0, g2 = 0.0, l = 0.0;
    if (S != 0.0) {
        for (int K = 0; K < c.n_det; ++K) {
            const int8_t s = c.sign[(K * c.W + w) * 2] * c.sign[(K * c.W + w) * 2 + 1];
            if (s == 0 || c.coef[K] == 0.0) continue;
            const double L = c.logdet[(K * c.W + w) * 2] + c.logdet[(K * c.W + w) * 2 + 1] + log(fabs(c.coef[K]));
            const double wk = (c.coef[K] > 0 ? s : -s) * exp(L - m) / S;
            const size_t r = ((size_t)K * c.W + w) * c.N + e;
            g0 += wk * c.drift[3 * r];
            g1 += wk * c.drift[3 * r + 1];
            g2 += wk * c.drift[3 * r + 2];
            l += wk * c.lap[r];
        }
    } else {
        g0 = g1 = g2 = l = NAN;
    }
    const size_t o = (size_t)w * c.N + e;
    if (c.out_drift) {
        c.out_drift[3 * o] = g0;
        c.out_drift[3 * o + 1] = g1;
        c.out_drift[3 * o + 2] = g2;
    }
    if (c.out_lap) c.out_lap[o] = l;
    if (e == 0) {
        if (c.out_logpsi) c.out_logpsi[w] = S != 0.0 ? m + log(fabs(S)) : -INFINITY;
        if (c.out_sign) c.out_sign[w] = S > 0 ? 1 : (S < 0 ? -1 : 0);
        if (c.out_status) {
            uint32_t st = c.st0[w] | (S == 0.0 ? QSL_STATUS_SINGULAR : 0u);
            for (int K = 0; K < c.n_det; ++K) st |= c.dstatus[K * c.W + w] & (QSL_STATUS_NEAR_TIE | QSL_STATUS_NONFINITE);
            c.out_status[w] = st;
        }
    }
}

// Determinants of a group: inverted in one launch.  At 158 electrons and 256
// walkers one determinant's 512 matrices leave the chip to one chain of steps
// each (54 us a launch); groups fill it.  Bounded by 512 MB of C_1 and
// inverses, by MD_GROUP_MATRICES per launch, beyond which the chip is full
// anyway, and one at a time where the blocked inversion needs a workspace per
// matrix.
constexpr size_t MD_GROUP_BYTES = (size_t)512 << 20;
constexpr int64_t MD_GROUP_MATRICES = 65536;
constexpr int MD_GROUP_MAX = 4096;  // (their Jobs: 19 MB)

struct MDLayout {
    WsLayout base;
    int group;  // determinants per group
    size_t corb[2], c1[2], dinv[2], list[4], logdet, sign, drift, lap, dstatus, st0, occ, coef, total;
};

// (group_max: at most so many determinants per group)
static MDLayout md_layout(const DevSys& d, const DevMO mo[2], int64_t W, int mode, int n_det, int group_max = MD_GROUP_MAX) {
    MDLayout L{};
    L.base = ws_layout(d, W, mode, /*sort=*/false);  // the forward's part
    size_t off = L.base.fwd_total;
    const size_t cb = mode == QSL_FP64 ? 8 : 4;
    const int N = d.n_up + d.n_dn;
    size_t one = 0;  // bytes of a determinant
    for (int s = 0; s < 2; ++s) one += (size_t)W * n_spin(d, s) * n_spin(d, s) * (cb + 8);
    int g = (int)std::min<size_t>({(size_t)std::min(n_det, group_max), MD_GROUP_BYTES / std::max<size_t>(one, 1),
                                   (size_t)(MD_GROUP_MATRICES / std::max<int64_t>(2 * W, 1))});
    if (g < 1 || gj_blocked(d.n_up) || gj_blocked(d.n_dn)) g = 1;
    L.group = (n_det + (n_det + g - 1) / g - 1) / ((n_det + g - 1) / g);  // groups of like sizes
    for (int s = 0; s < 2; ++s) {
        const size_t n = (size_t)n_spin(d, s);
        L.corb[s] = off;
        off = round_up(off + (size_t)W * 5 * n * mo[s].n * cb, 256);
        L.c1[s] = off;
        off = round_up(off + (L.group * (size_t)W * n * n + GJ_READ_PAST) * cb, 256);
        L.dinv[s] = off;
        off = round_up(off + L.group * (size_t)W * n * n * 8, 256);
    }
    for (int l = 0; l < 4; ++l) {
        L.list[l] = off;
        off = round_up(off + 2 * L.group * sizeof(Job) + (2 * L.group + 1) * sizeof(int), 256);
    }
    L.logdet = off;
    off = round_up(off + (size_t)n_det * W * 2 * 8, 256);
    L.sign = off;
    off = round_up(off + (size_t)n_det * W * 2, 256);
    L.drift = off;
    off = round_up(off + (size_t)n_det * W * N * 3 * 8, 256);
    L.lap = off;
    off = round_up(off + (size_t)n_det * W * N * 8, 256);
    L.dstatus = off;
    off = round_up(off + (size_t)n_det * W * 4, 256);
    L.st0 = off;
    off = round_up(off + (size_t)W * 4, 256);
    L.occ = off;
    off = round_up(off + (size_t)n_det * N * 4, 256);
    L.coef = off;
    off = round_up(off + (size_t)n_det * 8, 256);
    L.total = off;
    return L;
}

static int grid_of(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 65536)); }

}  // namespace qsl

using namespace qsl;

extern "C" {

qsl_status qsl_multidet_workspace_size(const qsl_system* sys, int64_t W, int32_t mode, int32_t n_det, size_t* bytes) {
    if (!sys || !bytes || W < 0 || n_det < 1) return bad(QSL_ERR_INVALID_ARG, "NULL argument, W < 0 or n_det < 1");
    if (mode < QSL_FP64 || mode > QSL_BF16X3) return bad(QSL_ERR_INVALID_ARG, "bad mode");
    *bytes = md_layout(sys->d, sys->mo, W, mode, n_det).total;
    return QSL_OK;
}

qsl_status qsl_multidet_forward(qsl_system* sys, const qsl_multidet_args* a, void* stream) {
    if (!sys || !a) return bad(QSL_ERR_INVALID_ARG, "NULL argument");
    if (a->W < 0 || a->n_det < 1) return bad(QSL_ERR_INVALID_ARG, "W < 0 or n_det < 1");
    if (a->mode < QSL_FP64 || a->mode > QSL_BF16X3) return bad(QSL_ERR_INVALID_ARG, "bad mode");
    if (!a->occ || !a->coef) return bad(QSL_ERR_INVALID_ARG, "NULL occupations or coefficients");
    const DevSys& d = sys->d;
    const int N = d.n_up + d.n_dn;
    for (int s = 0; s < 2; ++s) {
        const int n = n_spin(d, s);
        if (!n) continue;
        if (!sys->mo[s].set) return bad(QSL_ERR_INVALID_ARG, "orbitals of a spin were never set");
        if (n > GJ_NMAX) return bad(QSL_ERR_UNSUPPORTED, "more electrons of one spin than the inversion supports");
    }
    for (int K = 0; K < a->n_det; ++K) {
        if (!std::isfinite(a->coef[K])) return bad(QSL_ERR_INVALID_ARG, "non-finite determinant coefficient");
        for (int e = 0; e < N; ++e) {
            const int s = e < d.n_up ? 0 : 1;
            const int o = a->occ[(size_t)K * N + e];
            if (o < 0 || o >= sys->mo[s].n) return bad(QSL_ERR_INVALID_ARG, "orbital index out of range");
        }
    }
    if (a->W == 0) return QSL_OK;
    if (!a->R) return bad(QSL_ERR_INVALID_ARG, "NULL R");
    // A workspace sized for more walkers or determinants always serves fewer:
    // its groups may have been smaller, then these are too (one determinant at
    // a time needs less for less of either).
    MDLayout L = md_layout(d, sys->mo, a->W, a->mode, a->n_det);
    for (int g = L.group - 1; a->ws_bytes < L.total && g >= 1; --g) L = md_layout(d, sys->mo, a->W, a->mode, a->n_det, g);
    if (!a->ws || a->ws_bytes < L.total) return bad(QSL_ERR_WORKSPACE, "workspace missing or too small");
    hipStream_t st = (hipStream_t)stream;
    char* ws = (char*)a->ws;
    const int64_t W = a->W;
    const int nd = a->n_det;
    hipError_t e;
    // occupations and coefficients to the device (the host arrays may be
    // reused once the call returns)
    if ((e = hipMemcpyAsync(ws + L.occ, a->occ, (size_t)nd * N * 4, hipMemcpyHostToDevice, st)) != hipSuccess ||
        (e = hipMemcpyAsync(ws + L.coef, a->coef, (size_t)nd * 8, hipMemcpyHostToDevice, st)) != hipSuccess)
        return hip_fail(e, "multidet: upload of occupations");
    uint32_t* st0 = (uint32_t*)(ws + L.st0);
    if ((e = fill_u32(st0, 0u, W, st)) != hipSuccess) return hip_fail(e, "multidet: status clear");
    double* dlog = (double*)(ws + L.logdet);
    int8_t* dsgn = (int8_t*)(ws + L.sign);
    double* ddr = (double*)(ws + L.drift);
    double* dlap = (double*)(ws + L.lap);
    uint32_t* dstat = (uint32_t*)(ws + L.dstatus);
    const int* occ = (const int*)(ws + L.occ);
    if ((e = fill_u32(dstat, 0u, (int64_t)nd * W, st)) != hipSuccess) return hip_fail(e, "multidet: status clear");
    // the products of the whole orbital set, once
    enum { SCREEN, CONTRACT };
    CallLists P(ws + L.base.call_off);
    const int nmo_max = std::max(d.n_up ? sys->mo[0].n : 0, d.n_dn ? sys->mo[1].n : 0);
    for (int s = 0; s < 2; ++s) {
        Job j{};
        j.s = d;
        j.mo = sys->mo[s];
        j.spin = s;
        j.n = n_spin(d, s);
        j.mode = a->mode;
        j.gw = 1;
        j.W = W;
        j.R = a->R;
        j.nwin = (int*)(ws + L.base.nwin_off[s]);
        j.win = (int*)(ws + L.base.win_off[s]);
        j.f32_tile = a->mode == QSL_FP64 ? contract_f64_tile(nmo_max) : F32_TILE_DEFAULT;
        j.status = st0;
        j.C = ws + L.corb[s];
        P.job[s] = j;
        if (!j.n) continue;
        P.add(SCREEN, s, screen_blocks(j, 0));
        contract_grid(j);
        P.add(CONTRACT, s, j.gx, j.gy, j.gz);
    }
    if ((e = P.store(st)) != hipSuccess) return hip_fail(e, "job lists");
    if (P.any(SCREEN)) {
        ProfScope ps("screen", st);
        e = P.run(SCREEN, [&](const Job* js, const int* pre, int nj, int nb) { return launch_screen_batched(js, pre, nj, nb, 0, st); });
        if (e != hipSuccess) return hip_fail(e, "screen kernel");
    }
    if (P.any(CONTRACT)) {
        ProfScope ps(contract_label(a->mode), st);
        const int tile = P.job[d.n_up ? 0 : 1].f32_tile;
        e = P.run(CONTRACT, [&](const Job* js, const int* pre, int nj, int nb) {
            return launch_contract_batched(a->mode, tile, nullptr, js, pre, nj, nb, st);
        });
        if (e != hipSuccess) return hip_fail(e, "contraction kernel");
    }
    // the determinants, a group at a time
    MDLists m{};
    MDGather g{};
    g.W = m.W = W;
    g.N = (int)(m.N = N);
    int variant[2] = {-1, -1};
    Job jd[2];
    for (int s = 0; s < 2; ++s) {
        const int n = n_spin(d, s);
        Job& j = jd[s] = P.job[s];
        j.mo.n = n;  // a square Slater matrix from here on
        j.c1_stride = (int64_t)n * n;
        j.c_ld = sys->mo[s].n;
        j.C = ws + L.c1[s];
        j.Dinv = (double*)(ws + L.dinv[s]);
        if (gj_blocked(n)) j.gjws = (double*)(ws + L.base.gj_off[s]);
        if (n) variant[s] = gj_job_variant(j);
        g.n[s] = n;
        g.nmo[s] = sys->mo[s].n;
        g.off[s] = s ? d.n_up : 0;
        g.corb[s] = m.corb[s] = ws + L.corb[s];
        g.c1[s] = ws + L.c1[s];
        m.c1_bytes[s] = W * n * n * (a->mode == QSL_FP64 ? 8 : 4);
        m.dinv[s] = W * n * n;
    }
    gj_share_variant(variant, {d.n_up, d.n_dn});
    // both spins in a launch unless they have more threads together than one can
    const bool apart = (W * N / 4 + 2 * W) * L.group >= (1ll << 32) / 512;
    for (int l = 0; l < 4; ++l) {
        m.list[l] = ws + L.list[l];
        for (int s = 0; s < 2; ++s) {
            const bool in = variant[s] >= 0 && (l & 1) == (apart ? s : l < 2 ? gj_list(variant, s) : 0);
            m.slot[l][s] = in ? m.spins[l]++ : -1;
            if (!in) continue;
            m.first[l][s] = m.total[l];
            m.blocks[l][s] = l >= 2 ? epilogue_blocks(jd[s]) : (int)W;
            m.total[l] += m.blocks[l][s];
        }
    }
    for (int K0 = 0; K0 < nd; K0 += L.group) {
        m.group = std::min(L.group, nd - K0);
        for (int s = 0; s < 2; ++s) {
            Job& j = jd[s];
            j.logdet = dlog + (size_t)K0 * W * 2;
            j.sign = dsgn + (size_t)K0 * W * 2;
            j.drift = ddr + (size_t)K0 * W * N * 3;
            j.lap = dlap + (size_t)K0 * W * N;
            j.status = dstat + (size_t)K0 * W;
            j.occ = occ + (size_t)K0 * N + g.off[s];
            if (j.n) continue;
            for (int K = K0; K < K0 + m.group; ++K) {  // a spin without electrons
                Job z = j;
                z.logdet = dlog + (size_t)K * W * 2;
                z.sign = dsgn + (size_t)K * W * 2;
                if ((e = launch_gj(z, st)) != hipSuccess) return hip_fail(e, "empty spin kernel");
            }
        }
        md_lists_kernel<<<m.group, 512, 0, st>>>(jd[0], jd[1], m);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "multidet: job lists");
        {
            ProfScope ps("gather_det", st);
            g.occ = occ + (size_t)K0 * N;
            const int64_t most = std::max(m.dinv[0], m.dinv[1]);
            const dim3 grid(std::min(grid_of(most), 4096), m.group, 2);
            if (a->mode == QSL_FP64) gather_det_kernel<double><<<grid, 256, 0, st>>>(g);
            else gather_det_kernel<float><<<grid, 256, 0, st>>>(g);
            if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "multidet: gather kernel");
        }
        const auto prefix = [&](int l) { return (const int*)(m.list[l] + (size_t)m.group * m.spins[l] * sizeof(Job)); };
        for (int l = 0; l < 2; ++l) {
            const int nj = m.group * m.spins[l], blocks = m.group * m.total[l];
            if (!nj) continue;
            ProfScope ps("gauss_jordan", st);
            const int v = variant[m.slot[l][0] >= 0 ? 0 : 1];
            e = v == GJ_V_BLOCKED ? launch_gjb_batched(a->mode, (const Job*)m.list[l], prefix(l), nj, blocks,
                                                       std::max(d.n_up, d.n_dn), st)
                                  : launch_gj_batched(v, (const Job*)m.list[l], prefix(l), nj, blocks, st);
            if (e != hipSuccess) return hip_fail(e, "inversion kernel");
        }
        for (int l = 2; l < 4; ++l) {
            const int nj = m.group * m.spins[l], blocks = m.group * m.total[l];
            if (!nj) continue;
            ProfScope ps("drift_lap", st);
            if ((e = launch_epilogue_batched(a->mode, (const Job*)m.list[l], prefix(l), nj, blocks, st)) != hipSuccess)
                return hip_fail(e, "epilogue kernel");
        }
    }
    MDComb c{};
    c.W = W;
    c.N = N;
    c.n_up = d.n_up;
    c.n_det = nd;
    c.coef = (const double*)(ws + L.coef);
    c.logdet = dlog;
    c.sign = dsgn;
    c.drift = ddr;
    c.lap = dlap;
    c.dstatus = dstat;
    c.st0 = st0;
    c.out_logpsi = a->logpsi;
    c.out_sign = a->sign;
    c.out_drift = a->drift;
    c.out_lap = a->lap;
    c.out_status = a->status;
    {
        ProfScope ps("combine_dets", st);
        combine_kernel<<<grid_of(W * N), 256, 0, st>>>(c);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "multidet: combine kernel");
    }
    if (a->det_logdet &&
        (e = hipMemcpyAsync(a->det_logdet, dlog, (size_t)nd * W * 2 * 8, hipMemcpyDeviceToDevice, st)) != hipSuccess)
        return hip_fail(e, "multidet: copy of determinant logs");
    if (a->det_sign && (e = hipMemcpyAsync(a->det_sign, dsgn, (size_t)nd * W * 2, hipMemcpyDeviceToDevice, st)) != hipSuccess)
        return hip_fail(e, "multidet: copy of determinant signs");
    return QSL_OK;
}

}  // extern "C"
