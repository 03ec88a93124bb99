// HIP kernels (gfx950) for the e-ph collision integral and its consumers.
//
// Data layout in HBM (built once by layout.cpp, uploaded by api.hip):
//   pnu [E]  u32   partner << 3 | mode, sorted by (destination, partner, mode)
//   g2  [E]  T     |g|^2 of the entry's channel (each channel stored twice)
//   st  [S]  {T eps; u32 kq}   state energy and k in q-grid units (10 bits/axis)
//   hw  [Nq][n_modes] T, nph [Nq][n_modes] T (caller's occupations)
//   chunk_beg [n_chunks+1] i64, chunk_dest [n_chunks] i32: workgroup work items,
//   each a contiguous run of one destination's entries.
//
// One workgroup reduces one chunk: its threads stride the chunk's entries
// (coalesced pnu/g2 streams), gather the partner's state record, occupation
// and phonon data (cache resident), evaluate the two Gaussians and fold the
// entry into two running sums, then combine lanes with a fixed
// shuffle tree and waves through LDS in fixed order.  Floating-point sums
// never use atomics; the single-copy pass and the phonon-side rate add
// 64-bit fixed-point integers with integer atomics, which are associative,
// so every result is bitwise reproducible.
//
// Entry algebra (Eq. 2 with the golden-rule occupation factors).  With
// da = exp(-(e_d - e_p + hw)^2 / 2 s^2), de = exp(-(e_d - e_p - hw)^2 / 2 s^2)
// (evaluated as powers of two),
// t = N (da + de):
//   a = g2 (t + de)  (weight of the out-scattering product f_d (1 - f_p))
//   b = g2 (t + da)  (weight of the in-scattering product  f_p (1 - f_d))
// and I_d = K [ (1 - f_d) sum b f_p  -  f_d sum a (1 - f_p) ] with
// K = 2 pi / (hbar N_q) / (s sqrt(2 pi)).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace ephbte {

// kq:  k in q-grid units, 10 bits per axis (a0 << 20 | a1 << 10 | a2)
// kqp: the same k in shifted coordinates c (0 .. span - 1 per axis) as the
//      linear index (c0 b1 + c1) b2 + c2 on the (b0, b1, b2) = 2 span - 1 box
//      of QBox, so that kqp_p - kqp_d + offset is the box row of q = k_p - k_d
//      (each axis difference + span - 1 lies in [0, b), so no borrow crosses axes)
template <typename T> struct StateRec;
template <> struct alignas(16) StateRec<double> {
    double eps;
    uint32_t kq;
    uint32_t kqp;
};
template <> struct alignas(16) StateRec<float> {
    float eps;
    uint32_t kq;
    uint32_t kqp;
    uint32_t pad;
};

// Base-2 exponential of the (pre-scaled, never positive) Gaussian exponent;
// the log2(e) factor is folded into the exponent scale on the host.
// FP32: the hardware exponential.  FP64: y = n + r with n = rint(y), which
// is exact, so |r| <= 1/2; 2^r = exp(r ln2) by its Taylor series to degree
// 12 (truncation below 2e-16 relative for |r ln2| <= 0.347, Horner form);
// 2^n by ldexp.  y is clamped at -1100, where the result is already 0.
__device__ __forceinline__ double gauss_exp2(double y) {
    y = fmax(y, -1100.0);
    const double n = __builtin_rint(y);
    const double r = y - n;
    // coefficients (ln 2)^k / k!, k = 12 .. 0
    double p = 2.5678435993488196e-11;
    p = fma(p, r, 4.44553827187081e-10);
    p = fma(p, r, 7.054911620801121e-09);
    p = fma(p, r, 1.0178086009239696e-07);
    p = fma(p, r, 1.3215486790144305e-06);
    p = fma(p, r, 1.5252733804059838e-05);
    p = fma(p, r, 0.00015403530393381606);
    p = fma(p, r, 0.0013333558146428441);
    p = fma(p, r, 0.009618129107628477);
    p = fma(p, r, 0.055504108664821576);
    p = fma(p, r, 0.2402265069591007);
    p = fma(p, r, 0.6931471805599453);
    p = fma(p, r, 1.0);
    return ldexp(p, static_cast<int>(n));
}
// Table-driven base-2 exponential (Tang, ACM TOMS 15(2), 1989) for the
// streaming kernels.  Takes y256 = 256 y.  With n = rint(y256) and
// r = y256 - n (exact, |r| <= 1/2): 2^y = 2^(n >> 8) 2^((n & 255)/256) 2^(r/256).
// The middle factor comes from a 256-entry table of 2^(j/256) held in LDS;
// the last is exp(r ln2/256) by its Taylor series to degree 4
// (|r ln2/256| <= 1.36e-3, truncation below 4e-17 relative); coefficients
// (ln2/256)^k / k!.  y256 is clamped where the result is already 0, which
// keeps the integer conversion in range.
__device__ __forceinline__ double gauss_exp2_tab(double y256, const double *tab) {
    y256 = fmax(y256, -300000.0);
    const double n = __builtin_rint(y256);
    const double r = y256 - n;
    double p = 2.239395190875157e-12;
    p = fma(p, r, 3.3083026805413713e-09);
    p = fma(p, r, 3.6655655969101062e-06);
    p = fma(p, r, 0.0027076061740622863);
    p = fma(p, r, 1.0);
    const int i = static_cast<int>(n);
    return ldexp(tab[i & 255] * p, i >> 8);
}

__device__ __forceinline__ double gauss_exp(double a) { return gauss_exp2(a); }
__device__ __forceinline__ float gauss_exp(float a) { return __builtin_amdgcn_exp2f(a); }

template <typename T> struct alignas(4 * sizeof(T)) Vec4 {
    T x, y, z, w;
};

// linear q index of k_p - k_d (both given in q-grid units, 10 bits per axis)
__device__ __forceinline__ int q_linear(uint32_t kd, uint32_t kp, int n0, int n1, int n2) {
    int a0 = static_cast<int>(kp >> 20) - static_cast<int>(kd >> 20);
    int a1 = static_cast<int>((kp >> 10) & 1023u) - static_cast<int>((kd >> 10) & 1023u);
    int a2 = static_cast<int>(kp & 1023u) - static_cast<int>(kd & 1023u);
    a0 += (a0 < 0) ? n0 : 0;
    a1 += (a1 < 0) ? n1 : 0;
    a2 += (a2 < 0) ? n2 : 0;
    return (a0 * n1 + a1) * n2 + a2;
}

// chunk served by this workgroup; with xcd_m > 0 the 8 XCDs (which receive
// workgroups round-robin) each get a contiguous range of chunks, so every
// L2 sees neighbouring destinations
__device__ __forceinline__ int64_t chunk_of_block(int64_t n_chunks, int64_t xcd_m) {
    int64_t b = blockIdx.x;
    if (xcd_m > 0) return (b & 7) * xcd_m + (b >> 3);
    return b;
}

// Tile served by this workgroup.  Workgroups are dispatched to the 8 XCDs
// round-robin (block b runs on XCD b % 8); with xcd set, each XCD gets a
// contiguous range of tiles, so the workgroups sharing one L2 work on
// neighbouring destinations, whose partner and {hw, N} gathers overlap.
// The grid then has 8 ceil(n / 8) blocks; the extra ones get -1.
__device__ __forceinline__ int64_t tile_of_block(int64_t n, int xcd) {
    const int64_t b = blockIdx.x;
    if (!xcd) return b;
    const int64_t t = (b & 7) * ((n + 7) / 8) + (b >> 3);
    return t < n ? t : -1;
}

template <typename T> struct Tables {
    const uint32_t *__restrict__ pnu;
    const T *__restrict__ g2;
    const StateRec<T> *__restrict__ st;
    const T *__restrict__ hw;
    const T *__restrict__ nph;
    const int64_t *__restrict__ chunk_beg;
    const int32_t *__restrict__ chunk_dest;
    const int32_t *__restrict__ dest_chunk;
    const int32_t *__restrict__ ent_chan;
    int64_t n_chunks;
    int64_t xcd_m;
    int S, nm, nq0, nq1, nq2;
    T mc;   // Gaussian exponent scale, base 2: -log2(e) / (2 s^2)
    T K;    // 2 pi / (hbar N_q) / (s sqrt(2 pi))
};

// Per-destination epilogue applied to the value v = I_d (forward) or
// v = dL/df_d (reverse), for vector b.
template <typename T> struct Epi {
    int mode;              // see apply_epi
    int neg;               // mode 0: store -v (Bose plans)
    T *out;                // mode 0: output [B][ld_out]
    int64_t ld_out;
    const T *f0;           // RK4: step start f (caller layout, ld_f0)
    int64_t ld_f0;
    T *u_out;              // RK4: next stage input [B][S]
    T *acc;                // RK4: k1 + 2k2 + 2k3 accumulator [B][S]
    T *f_out;              // RK4 stage 4: f at the end of the step (ld_f0)
    T dt;
    // adjoint stages: lam_out = cg * gbar + cv * v
    const T *gbar;
    T *gbar_out;
    T cg, cv;
    // field term of Eq. 1 (RK and adjoint modes, when nbr is set): v gains
    // dsign * D[x], D[x]_d = -sum_a rate[a] (x[up_a] - x[down_a]) / 2, with x the
    // stage input (forward: the stage's f, dsign = 1; adjoint: the stage's
    // lambda, dsign = -1, since D^T = -D for a symmetric neighbour relation)
    const int32_t *nbr;    // [S][3][2], -1: not in the list (x = 0 there)
    const T *x;
    int64_t ld_x;
    T rate[3];
    T dsign;
};

template <typename T>
__device__ __forceinline__ T drift_term(const Epi<T> &E, int b, int d) {
    const int32_t *nb = E.nbr + 6 * static_cast<int64_t>(d);
    const T *xb = E.x + static_cast<int64_t>(b) * E.ld_x;
    T s = T(0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int up = nb[2 * a], dn = nb[2 * a + 1];
        const T xu = up >= 0 ? xb[up] : T(0);
        const T xd = dn >= 0 ? xb[dn] : T(0);
        s += E.rate[a] * (xu - xd);
    }
    return E.dsign * (T(-0.5) * s);
}

enum EpiMode {
    EPI_STORE = 0,
    EPI_RK1 = 1,     // acc = v;       u = f0 + dt/2 v
    EPI_RK2 = 2,     // acc += 2v;     u = f0 + dt/2 v
    EPI_RK3 = 3,     // acc += 2v;     u = f0 + dt v
    EPI_RK4 = 4,     // f_out = f0 + dt/6 (acc + v)
    EPI_ADJ_FIRST = 5,   // acc = v;   u = cg gbar + cv v
    EPI_ADJ_MID = 6,     // acc += v;  u = cg gbar + cv v
    EPI_ADJ_LAST = 7,    // gbar_out = gbar + acc + v
};

template <typename T>
__device__ __forceinline__ void apply_epi(const Epi<T> &E, int b, int d, int S, T v) {
    const int64_t iw = static_cast<int64_t>(b) * S + d;
    if (E.mode > EPI_STORE && E.nbr) v += drift_term(E, b, d);
    switch (E.mode) {
    case EPI_STORE: E.out[static_cast<int64_t>(b) * E.ld_out + d] = E.neg ? -v : v; break;
    case EPI_RK1: {
        T f = E.f0[static_cast<int64_t>(b) * E.ld_f0 + d];
        E.acc[iw] = v;
        E.u_out[iw] = f + (E.dt * T(0.5)) * v;
    } break;
    case EPI_RK2: {
        T f = E.f0[static_cast<int64_t>(b) * E.ld_f0 + d];
        E.acc[iw] += T(2) * v;
        E.u_out[iw] = f + (E.dt * T(0.5)) * v;
    } break;
    case EPI_RK3: {
        T f = E.f0[static_cast<int64_t>(b) * E.ld_f0 + d];
        E.acc[iw] += T(2) * v;
        E.u_out[iw] = f + E.dt * v;
    } break;
    case EPI_RK4: {
        int64_t i = static_cast<int64_t>(b) * E.ld_f0 + d;
        T f = E.f0[i];
        E.f_out[i] = f + (E.dt / T(6)) * (E.acc[iw] + v);
    } break;
    case EPI_ADJ_FIRST:
        E.acc[iw] = v;
        E.u_out[iw] = E.cg * E.gbar[iw] + E.cv * v;
        break;
    case EPI_ADJ_MID:
        E.acc[iw] += v;
        E.u_out[iw] = E.cg * E.gbar[iw] + E.cv * v;
        break;
    case EPI_ADJ_LAST: E.gbar_out[iw] = E.gbar[iw] + E.acc[iw] + v; break;
    default: break;
    }
}

// ---- block reduction of NV values, fixed order --------------------------
template <typename T> __device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Reduces v[0..NV) over the block; thread 0 receives the totals.
template <typename T, int NV>
__device__ __forceinline__ void block_sum(T (&v)[NV]) {
    __shared__ T red[NV][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nw = (blockDim.x + 63) >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) red[k][wave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            T s = red[k][0];
            for (int w = 1; w < nw; ++w) s += red[k][w];
            v[k] = s;
        }
    }
}

// ---- per-entry coefficient evaluation -----------------------------------
template <typename T> struct EntryCoef {
    T ah, bh;   // t + de, t + da  (without |g|^2)
};

template <typename T>
__device__ __forceinline__ EntryCoef<T> entry_coef(const Tables<T> &P, T eps_d, uint32_t kq_d,
                                                   uint32_t pn, const StateRec<T> &sp) {
    const int nu = static_cast<int>(pn & 7u);
    const int q = q_linear(kq_d, sp.kq, P.nq0, P.nq1, P.nq2);
    const int64_t qi = static_cast<int64_t>(q) * P.nm + nu;
    const T w = P.hw[qi];
    const T N = P.nph[qi];
    const T de = eps_d - sp.eps;
    const T xa = de + w, xe = de - w;
    const T da = gauss_exp(xa * xa * P.mc);
    const T dem = gauss_exp(xe * xe * P.mc);
    const T t = N * (da + dem);
    EntryCoef<T> c;
    c.ah = t + dem;
    c.bh = t + da;
    return c;
}

// ---- forward, LDS-tiled --------------------------------------------------
// One workgroup per tile (a run of chunks whose destinations' partners fit an
// LDS window).  The tile's partner states {eps, f} and packed k are staged in
// LDS once; wave w then reduces chunks w, w + n_waves, ... of the tile, each
// with a fixed shuffle tree.  A destination with a single chunk is finished
// by that wave; others leave two partial sums for k_tiled_finish.  All loop
// bounds are wave-uniform scalars (chunk index, entry range), so every wave
// runs its loops in lock step with no divergent exits.
struct TileRec {
    int64_t c0, c1;
    int32_t p_lo, p_hi, lds, pad;
};

template <typename T> struct alignas(2 * sizeof(T)) Pair2 {
    T a, b;
};

// Maxima left by the workgroups of a preparing kernel (k_prep); the kernels that
// set a fixed-point scale from them take the largest themselves (scale_load), one
// launch fewer than a kernel that reduces them.  At most 64 values; n = 0: none.
struct MaxList {
    const double *v;
    int n;
};

template <typename T> struct TiledArgs {
    const uint32_t *__restrict__ pnu;
    const T *__restrict__ g2;
    const StateRec<T> *__restrict__ st;
    const Pair2<T> *__restrict__ hwN;   // {hw, N} of (q, mode) at hwN[q tq + mode tm]
    int64_t tq, tm;                     // (n_modes, 1): the modes of one q adjacent;
                                        // (1, table rows): one block per mode
    const int64_t *__restrict__ chunk_beg;
    const int32_t *__restrict__ chunk_dest;
    const int32_t *__restrict__ dest_chunk;
    const TileRec *__restrict__ tiles;
    int64_t n_chunks;
    int S, nm, nq0, nq1, nq2, lds_states;
    int padq;          // 1: hwN is the box table of QBox, indexed by kqp differences
    int qoff;          // box row of the q = 0 difference
    T mc, K;
    const double *__restrict__ e2tab;   // 2^(j/256), j = 0 .. 255 (FP64 kernels)
    double mc256;                       // 256 mc, the table exponential's scale
    int64_t n_tiles;
    int xcd;                            // tile ranges per XCD (tile_of_block)
    // single-copy pass only
    const int64_t *__restrict__ chunk_end;           // chunk c is [chunk_beg[c], chunk_end[c])
    unsigned long long *__restrict__ jacc;           // [S] partner-side sums, fixed point
    MaxList nmax;                                    // max |N| of the packed table
    const unsigned long long *__restrict__ gmax_bits;  // max over states of sum |g|^2 (double bits)
    // pair records (k_fwd_pairs): pnu holds partners, g2 is [n_modes][pld]
    int64_t pld;
    int all_q;                                       // every tile is q-ordered: no row partials
    // occupations outside [0, 1] (the Bose plans' negated n): max |f| of the
    // call's input, or n = 0 when f lies in [0, 1]
    MaxList fmax;
};

// ---- fixed point for the partner side of the single-copy pass -------------
// Contributions to I_p (p > d) arrive from many rows; they are rounded to
// integers on a common scale 2^s and summed with integer atomics, which are
// associative, so the sums do not depend on the order of arrival.  With
// |N| <= N_max, f in [0, 1] and the Gaussians <= 1, one entry's share is at
// most |g|^2 (2 N_max + 1), a state's column at most (2 N_max + 1) G_max with
// G_max the largest sum of |g|^2 over one state's channels; s puts that bound
// below 2^61.  With |f| <= m instead, the occupation products of a term,
// at most 1 in [0, 1], are at most (1 + 2m)^2, a factor on the bound.
// Values a scale is made of, one of each list per lane (lists hold at most 64):
// loaded at the top of a kernel, so that they arrive while it stages its window.
struct ScaleIn {
    double n, f, l, g;
    bool occ, one;   // one: every list holds one value
};
__device__ __forceinline__ double list_value(MaxList l) {
    const int i = l.n == 1 ? 0 : static_cast<int>(threadIdx.x & 63);
    return i < l.n ? l.v[i] : 0.0;
}
__device__ __forceinline__ ScaleIn scale_load(MaxList nmax, const unsigned long long *gmax_bits, MaxList fmax_l,
                                              MaxList lmax) {
    ScaleIn s;
    s.n = list_value(nmax);
    s.f = list_value(fmax_l);
    s.l = list_value(lmax);
    s.g = __longlong_as_double(static_cast<long long>(*gmax_bits));
    s.occ = fmax_l.n > 0;
    s.one = nmax.n <= 1 && fmax_l.n <= 1 && lmax.n <= 1;
    return s;
}
// the largest over the wave (all lanes take part)
__device__ __forceinline__ double wave_max(double m, bool one) {
    if (one) return m;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    return m;
}
__device__ __forceinline__ double occ_factor(const ScaleIn &s) {
    if (!s.occ) return 1.0;
    const double m = wave_max(s.f, s.one);
    return (1.0 + 2.0 * m) * (1.0 + 2.0 * m);
}
__device__ __forceinline__ double scale_of_bound(double bound) {
    if (!(bound > 0.0) || !(bound < 1e300)) return 1.0;
    int e;
    (void)frexp(bound, &e);   // bound < 2^e
    return ldexp(1.0, 61 - e);
}
__device__ __forceinline__ double sym_scale(const ScaleIn &s) {
    return scale_of_bound((2.0 * wave_max(s.n, s.one) + 1.0) * s.g * occ_factor(s));
}

// y integral-valued with |y| < 2^62, as a two's-complement 64-bit integer
template <typename T> __device__ __forceinline__ unsigned long long to_fixed(T y) {
    const T hi = floor(y * T(2.3283064365386963e-10));   // y / 2^32, rounded down
    const T lo = fma(hi, T(-4294967296.0), y);           // y - hi 2^32, exact, in [0, 2^32)
    const uint32_t l = static_cast<uint32_t>(lo);
    const uint32_t h = static_cast<uint32_t>(static_cast<int32_t>(hi));
    return (static_cast<unsigned long long>(h) << 32) | l;
}

// max of v over the workgroup (blockDim.x <= 1024), stored by thread 0 to *dst
__device__ __forceinline__ void block_max_to(double v, double *dst) {
    __shared__ double s_m[16];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = s_m[0];
        for (int w = 1; w < static_cast<int>(blockDim.x >> 6); ++w) m = fmax(m, s_m[w]);
        *dst = m;
    }
}

// The maxima that the workgroups of a part of k_prep left, more than a list holds,
// folded into one (workgroup = part; n = 0: none)
struct FoldPart {
    const double *v;
    int n;             // at most 1024
    double *out;
};
__global__ __launch_bounds__(1024) void k_fold_max(FoldPart a, FoldPart b, FoldPart c) {
    const FoldPart p = blockIdx.x == 0 ? a : blockIdx.x == 1 ? b : c;
    if (p.n == 0) return;
    block_max_to(static_cast<int>(threadIdx.x) < p.n ? p.v[threadIdx.x] : 0.0, p.out);
}

// each list's largest value, to its own place in out (one wave)
__global__ __launch_bounds__(64) void k_reduce_lists(MaxList a, MaxList b, MaxList c, double *out) {
    const double x = wave_max(list_value(a), false), y = wave_max(list_value(b), false),
                 z = wave_max(list_value(c), false);
    if (threadIdx.x == 0) {
        out[0] = x;
        out[1] = y;
        out[2] = z;
    }
}

__global__ void k_zero_u64(unsigned long long *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// entries of the exponential table that the FP64 streaming kernels keep in LDS
constexpr int kExpTab = 256;

// The padded q table.  States carry k in shifted coordinates c (per axis, 0
// .. span - 1 after a per-axis origin); a pair's difference c_p - c_d lies in
// [-(span - 1), span - 1], so the row x = c_p - c_d + (span - 1) of a
// (2 span - 1)-point axis names it without a modulo, and the three axes give
// the row of one box, qp = (x0 b1 + x1) b2 + x2.  The q it stands for is
// (x - (span - 1)) mod Nq per axis.  The box holds every difference between
// two states, so every row is filled; its size follows the extent of the
// states in k, not the q grid.
struct QBox {
    int n[3];   // q grid
    int b[3];   // box axis lengths, 2 span - 1
    int h[3];   // span - 1
};

// (box rows and q points are below 2^31: 32-bit arithmetic)
__device__ __forceinline__ int box_q(int qp, const QBox &B) {
    int x[3];
    x[2] = qp % B.b[2];
    qp /= B.b[2];
    x[1] = qp % B.b[1];
    x[0] = qp / B.b[1];
    int q = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int v = x[a] - B.h[a];
        v += v < 0 ? B.n[a] : 0;
        q = q * B.n[a] + v;
    }
    return q;
}

// What a call prepares before its main kernel, in one launch.
//  - The {hw, N} table: with the box, of the rows `used` (the rows some entry
//    references), every mode: row qp, mode nu at qp nm + nu (mode_major = 0) or
//    nu rows + qp (mode_major = 1), fewer than 2^31 entries (the plan sizes it
//    under 256 MB); rows not listed keep their zeros.  Without the box, all of it.
//  - Up to two vectors: max |x|, and -x where a Bose plan asks for it.
// Each part has its own workgroups, and each workgroup leaves the max of its part.
template <typename T> struct PackPart {
    const T *hw, *nph;
    Pair2<T> *out;
    QBox box;
    int padq, nm, rows, mode_major;
    const int32_t *used;
    int64_t n;         // entries
    double *bmax;
    int blocks;        // 0: no table
};
template <typename T> struct VecPart {
    const T *x;
    T *neg;            // null: no copy
    int64_t n;
    double *bmax;
    int blocks;        // 0: no vector
};
template <typename T>
__global__ __launch_bounds__(1024) void k_prep(PackPart<T> P, VecPart<T> V0, VecPart<T> V1) {
    double m = 0.0;
    double *dst;
    int b = blockIdx.x;
    if (b < P.blocks) {
        dst = P.bmax + b;
        for (int64_t i = static_cast<int64_t>(b) * blockDim.x + threadIdx.x; i < P.n;
             i += static_cast<int64_t>(P.blocks) * blockDim.x) {
            int64_t src = i, o = i;
            if (P.padq) {
                const int i32 = static_cast<int>(i);
                const int nu = i32 % P.nm, qp = P.used[i32 / P.nm];
                src = static_cast<int64_t>(box_q(qp, P.box)) * P.nm + nu;
                o = P.mode_major ? nu * P.rows + qp : qp * P.nm + nu;
            }
            Pair2<T> v;
            v.a = P.hw[src];
            v.b = P.nph[src];
            P.out[o] = v;
            m = fmax(m, fabs(static_cast<double>(v.b)));
        }
    } else {
        b -= P.blocks;
        const bool second = b >= V0.blocks;
        if (second) b -= V0.blocks;
        const T *__restrict__ x = second ? V1.x : V0.x;
        T *__restrict__ neg = second ? V1.neg : V0.neg;
        const int64_t n = second ? V1.n : V0.n;
        const int64_t stride = static_cast<int64_t>(second ? V1.blocks : V0.blocks) * blockDim.x;
        dst = (second ? V1.bmax : V0.bmax) + b;
        for (int64_t i = static_cast<int64_t>(b) * blockDim.x + threadIdx.x; i < n; i += stride) {
            const T v = x[i];
            if (neg) neg[i] = -v;
            m = fmax(m, fabs(static_cast<double>(v)));
        }
    }
    block_max_to(m, dst);
}

// exp of the Gaussian exponent x2 * (-1/(2 s^2)) for the streaming kernels
template <typename T>
__device__ __forceinline__ T stream_gauss(const TiledArgs<T> &A, T x2, const double *tab) {
    if constexpr (sizeof(T) == 8) return gauss_exp2_tab(x2 * A.mc256, tab);
    else return __builtin_amdgcn_exp2f(x2 * A.mc);
}

// Chunk reduction with a three-stage pipeline (stream loads two batches
// ahead, partner/table gathers one batch ahead of the evaluation).  The entry
// arrays are padded past their end, so stream loads are unconditional.  Only
// a chunk's last batch can hold lanes past its end (they read the padding or
// the next chunk); that batch is gathered with a mask that makes those lanes
// contribute zero, the others without one (the choice is uniform per wave).
// Offsets are 32-bit and relative to the chunk start.
template <typename T, bool LDS, bool PADQ, int U>
__device__ __forceinline__ void fwd_chunk2(const TiledArgs<T> &A, const T *__restrict__ fb,
                                           const Pair2<T> *s_ef, const uint32_t *s_kq, int p_lo,
                                           const double *s_tab, int64_t c, int b,
                                           T *__restrict__ part, const Epi<T> &E) {
    const int lane = threadIdx.x & 63;
    const int d = A.chunk_dest[c];
    const int64_t beg = A.chunk_beg[c];
    const int len = static_cast<int>(A.chunk_beg[c + 1] - beg);
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ gb = A.g2 + beg;
    const StateRec<T> sd = A.st[d];
    const uint32_t kd = PADQ ? sd.kqp : sd.kq;
    T acc_a = T(0), acc_b = T(0);
    uint32_t pn1[U];
    T gs1[U];
    T g0[U], de0[U], fp0[U];
    Pair2<T> wn0[U];
    auto load_stream = [&](int r0, uint32_t (&pn)[U], T (&gs)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pn[u] = pb[r0 + u * 64 + lane];
            gs[u] = gb[r0 + u * 64 + lane];
        }
    };
    auto gather = [&](auto masked, const uint32_t (&pn)[U], const T (&gs)[U], int r0,
                      T (&go)[U], T (&deo)[U], T (&fpo)[U], Pair2<T> (&wno)[U]) {
        constexpr bool M = decltype(masked)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool v = !M || r0 + u * 64 + lane < len;
            const int p = static_cast<int>(pn[u] >> 3);
            T ep, fp;
            uint32_t kp;
            if (LDS) {
                // a masked lane reads slot 0 (inside the allocation) and then
                // replaces what it read: partner = destination, so its table
                // index is the q = 0 entry and its operands are finite,
                // whatever the slot holds
                const int pl = v ? p - p_lo : 0;
                const Pair2<T> ef = s_ef[pl];
                ep = v ? ef.a : sd.eps;
                fp = v ? ef.b : T(0);
                kp = v ? s_kq[pl] : kd;
            } else {
                const StateRec<T> sp = A.st[p];
                ep = sp.eps;
                kp = PADQ ? sp.kqp : sp.kq;
                fp = fb[p];
            }
            const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff
                               : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
            const Pair2<T> w = A.hwN[static_cast<int64_t>(q) * A.tq + static_cast<int64_t>(pn[u] & 7u) * A.tm];
            if constexpr (M) {
                // a table entry without channels may hold a non-finite N, so both
                // fields are replaced (using both keeps the {hw, N} pair one
                // 16-byte load)
                wno[u].a = v ? w.a : T(0);
                wno[u].b = v ? w.b : T(0);
                go[u] = v ? gs[u] : T(0);
            } else {
                wno[u] = w;
                go[u] = gs[u];
            }
            deo[u] = sd.eps - ep;
            fpo[u] = fp;
        }
    };
    using Masked = std::integral_constant<bool, true>;
    using Full = std::integral_constant<bool, false>;
    {
        uint32_t pn0[U];
        T gs0[U];
        load_stream(0, pn0, gs0);
        load_stream(64 * U, pn1, gs1);
        if (64 * U <= len) gather(Full{}, pn0, gs0, 0, g0, de0, fp0, wn0);
        else gather(Masked{}, pn0, gs0, 0, g0, de0, fp0, wn0);
    }
    for (int r = 0; r < len; r += 64 * U) {
        T g1[U], de1[U], fp1[U];
        Pair2<T> wn1[U];
        if (r + 128 * U <= len) gather(Full{}, pn1, gs1, r + 64 * U, g1, de1, fp1, wn1);
        else gather(Masked{}, pn1, gs1, r + 64 * U, g1, de1, fp1, wn1);
        load_stream(r + 128 * U, pn1, gs1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T xa = de0[u] + wn0[u].a, xe = de0[u] - wn0[u].a;
            const T da = stream_gauss(A, xa * xa, s_tab);
            const T dem = stream_gauss(A, xe * xe, s_tab);
            const T t = wn0[u].b * (da + dem);
            acc_a += g0[u] * (t + dem) * (T(1) - fp0[u]);
            acc_b += g0[u] * (t + da) * fp0[u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            g0[u] = g1[u];
            de0[u] = de1[u];
            fp0[u] = fp1[u];
            wn0[u] = wn1[u];
        }
    }
    acc_a = wave_sum(acc_a);
    acc_b = wave_sum(acc_b);
    if (lane == 0) {
        if (A.dest_chunk[d + 1] - A.dest_chunk[d] == 1) {
            const T fd = fb[d];
            apply_epi(E, b, d, A.S, A.K * ((T(1) - fd) * acc_b - fd * acc_a));
        } else {
            T *pp = part + (static_cast<int64_t>(b) * A.n_chunks + c) * 2;
            pp[0] = acc_a;
            pp[1] = acc_b;
        }
    }
}

template <typename T, int U, int MAXT, bool PADQ>
__global__ __launch_bounds__(MAXT) void k_fwd_tiled(TiledArgs<T> A, const T *__restrict__ f,
                                                    int64_t ldf, T *__restrict__ part, Epi<T> E) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    const int b = blockIdx.y;
    const T *fb = f + static_cast<int64_t>(b) * ldf;
    Pair2<T> *s_ef = reinterpret_cast<Pair2<T> *>(smem);
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_ef + A.lds_states);
    double *s_tab = reinterpret_cast<double *>(s_kq + A.lds_states);
    if (t.lds) {
        const int n = t.p_hi - t.p_lo + 1;
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const StateRec<T> sr = A.st[t.p_lo + i];
            Pair2<T> ef;
            ef.a = sr.eps;
            ef.b = fb[t.p_lo + i];
            s_ef[i] = ef;
            s_kq[i] = PADQ ? sr.kqp : sr.kq;
        }
    }
    if constexpr (sizeof(T) == 8)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    for (int64_t c = t.c0 + wave; c < t.c1; c += nw) {
        if (t.lds)
            fwd_chunk2<T, true, PADQ, U>(A, fb, s_ef, s_kq, t.p_lo, s_tab, c, b, part, E);
        else
            fwd_chunk2<T, false, PADQ, U>(A, fb, s_ef, s_kq, t.p_lo, s_tab, c, b, part, E);
    }
}

// ---- forward, single copy ---------------------------------------------------
// Each channel is evaluated once, from the row of its smaller state d (the
// entries p > d of that row, the upper part of the destination-sorted layout).
// With Y = (1 - f_d) b f_p - f_d a (1 - f_p) (a, b as in the duplicated pass),
// I_d receives K Y and I_p receives -K Y: the row side is reduced in registers
// as in fwd_chunk2, the partner side is added to a fixed-point accumulator per
// partner (LDS for an LDS tile, then flushed to the global one).

// max over states of the sum of |g|^2 over the state's entries, one wave per state
template <typename T>
__global__ void k_row_gmax(const T *__restrict__ g2, const int64_t *__restrict__ chunk_beg,
                           const int32_t *__restrict__ dest_chunk, int S,
                           unsigned long long *gmax_bits) {
    const int d = static_cast<int>((blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    double sum = 0.0;
    if (d < S) {
        const int64_t b = chunk_beg[dest_chunk[d]], e = chunk_beg[dest_chunk[d + 1]];
        for (int64_t x = b + lane; x < e; x += 64) sum += fabs(static_cast<double>(g2[x]));
    }
    sum = wave_sum(sum);
    if (lane == 0 && d < S)
        atomicMax(gmax_bits, static_cast<unsigned long long>(__double_as_longlong(sum)));
}

template <typename T, bool LDS, bool PADQ, int U>
__device__ __forceinline__ void sym_chunk(const TiledArgs<T> &A, const T *__restrict__ fb,
                                          const Pair2<T> *s_ef, const uint32_t *s_kq, int p_lo,
                                          const double *s_tab, unsigned long long *s_j, T scale,
                                          int64_t c, T *__restrict__ part) {
    const int lane = threadIdx.x & 63;
    const int d = A.chunk_dest[c];
    const int64_t beg = A.chunk_beg[c];
    const int len = static_cast<int>(A.chunk_end[c] - beg);
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ gb = A.g2 + beg;
    const StateRec<T> sd = A.st[d];
    const uint32_t kd = PADQ ? sd.kqp : sd.kq;
    const T fd = fb[d];
    const T cfd = T(1) - fd;
    T acc_a = T(0), acc_b = T(0);
    uint32_t pn1[U];
    T gs1[U];
    T g0[U], de0[U], fp0[U];
    int pl0[U];
    Pair2<T> wn0[U];
    auto load_stream = [&](int r0, uint32_t (&pn)[U], T (&gs)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pn[u] = pb[r0 + u * 64 + lane];
            gs[u] = gb[r0 + u * 64 + lane];
        }
    };
    auto gather = [&](auto masked, const uint32_t (&pn)[U], const T (&gs)[U], int r0, T (&go)[U],
                      T (&deo)[U], T (&fpo)[U], Pair2<T> (&wno)[U], int (&plo)[U]) {
        constexpr bool M = decltype(masked)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool v = !M || r0 + u * 64 + lane < len;
            const int p = static_cast<int>(pn[u] >> 3);
            T ep, fp;
            uint32_t kp;
            if (LDS) {
                // a masked lane: partner = destination (finite operands, the
                // q = 0 table entry); it adds zero to slot 0 of the window
                const int pl = v ? p - p_lo : 0;
                const Pair2<T> ef = s_ef[pl];
                ep = v ? ef.a : sd.eps;
                fp = v ? ef.b : T(0);
                kp = v ? s_kq[pl] : kd;
                plo[u] = pl;
            } else {
                const StateRec<T> sp = A.st[p];
                ep = sp.eps;
                kp = PADQ ? sp.kqp : sp.kq;
                fp = fb[p];
                plo[u] = p;
            }
            const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff
                               : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
            const Pair2<T> w = A.hwN[static_cast<int64_t>(q) * A.tq + static_cast<int64_t>(pn[u] & 7u) * A.tm];
            if constexpr (M) {
                // a table entry without channels may hold a non-finite N; the
                // masked lanes then add zero to partner slot 0 (or state p)
                wno[u].a = v ? w.a : T(0);
                wno[u].b = v ? w.b : T(0);
                go[u] = v ? gs[u] : T(0);
            } else {
                wno[u] = w;
                go[u] = gs[u];
            }
            deo[u] = sd.eps - ep;
            fpo[u] = fp;
        }
    };
    using Masked = std::integral_constant<bool, true>;
    using Full = std::integral_constant<bool, false>;
    {
        uint32_t pn0[U];
        T gs0[U];
        load_stream(0, pn0, gs0);
        load_stream(64 * U, pn1, gs1);
        if (64 * U <= len) gather(Full{}, pn0, gs0, 0, g0, de0, fp0, wn0, pl0);
        else gather(Masked{}, pn0, gs0, 0, g0, de0, fp0, wn0, pl0);
    }
    for (int r = 0; r < len; r += 64 * U) {
        T g1[U], de1[U], fp1[U];
        int pl1[U];
        Pair2<T> wn1[U];
        if (r + 128 * U <= len) gather(Full{}, pn1, gs1, r + 64 * U, g1, de1, fp1, wn1, pl1);
        else gather(Masked{}, pn1, gs1, r + 64 * U, g1, de1, fp1, wn1, pl1);
        load_stream(r + 128 * U, pn1, gs1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T xa = de0[u] + wn0[u].a, xe = de0[u] - wn0[u].a;
            const T da = stream_gauss(A, xa * xa, s_tab);
            const T dem = stream_gauss(A, xe * xe, s_tab);
            const T t = wn0[u].b * (da + dem);
            const T ta = g0[u] * (t + dem) * (T(1) - fp0[u]);
            const T tb = g0[u] * (t + da) * fp0[u];
            acc_a += ta;
            acc_b += tb;
            // partner side: -Y = f_d ta - (1 - f_d) tb, on the fixed-point scale
            const unsigned long long v = to_fixed(__builtin_rint(fma(fd, ta, -cfd * tb) * scale));
            if (LDS) atomicAdd(s_j + pl0[u], v);
            else atomicAdd(A.jacc + pl0[u], v);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            g0[u] = g1[u];
            de0[u] = de1[u];
            fp0[u] = fp1[u];
            wn0[u] = wn1[u];
            pl0[u] = pl1[u];
        }
    }
    acc_a = wave_sum(acc_a);
    acc_b = wave_sum(acc_b);
    if (lane == 0) {
        part[2 * c] = acc_a;
        part[2 * c + 1] = acc_b;
    }
}

template <typename T, int U, bool PADQ>
__global__ __launch_bounds__(1024) void k_fwd_sym(TiledArgs<T> A, const T *__restrict__ f,
                                                  T *__restrict__ part) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    const ScaleIn si = scale_load(A.nmax, A.gmax_bits, A.fmax, MaxList{nullptr, 0});
    // LDS: partner-side sums (8 B), {eps, f}, packed k, exponential table
    unsigned long long *s_j = reinterpret_cast<unsigned long long *>(smem);
    Pair2<T> *s_ef = reinterpret_cast<Pair2<T> *>(s_j + A.lds_states);
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_ef + A.lds_states);
    double *s_tab = reinterpret_cast<double *>(s_kq + A.lds_states);
    const int n = t.lds ? t.p_hi - t.p_lo + 1 : 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const StateRec<T> sr = A.st[t.p_lo + i];
        Pair2<T> ef;
        ef.a = sr.eps;
        ef.b = f[t.p_lo + i];
        s_ef[i] = ef;
        s_kq[i] = PADQ ? sr.kqp : sr.kq;
        s_j[i] = 0ull;
    }
    if constexpr (sizeof(T) == 8)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    const T scale = static_cast<T>(sym_scale(si));
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    for (int64_t c = t.c0 + wave; c < t.c1; c += nw) {
        if (t.lds)
            sym_chunk<T, true, PADQ, U>(A, f, s_ef, s_kq, t.p_lo, s_tab, s_j, scale, c, part);
        else
            sym_chunk<T, false, PADQ, U>(A, f, s_ef, s_kq, t.p_lo, s_tab, s_j, scale, c, part);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const unsigned long long v = s_j[i];
        if (v) atomicAdd(A.jacc + t.p_lo + i, v);
    }
}

// ---- forward, single copy over pair records ----------------------------------
// The same pass over pair records: a lane takes one pair (d, p), p > d, with
// all its modes.  The partner's {eps, f} and k are gathered once per pair, the
// {hw, N} of the modes of q = k_p - k_d are adjacent in the table, and the
// partner side of the pair (summed over its modes in a fixed order) is one
// fixed-point atomic.  A slot without a channel has |g|^2 = 0; its N is
// replaced by 0 so that a non-finite table entry of that mode (N at an
// acoustic q = 0) cannot turn the zero into a NaN.

// v where keep holds, else +0, by masking the bits: unlike a select of a
// loaded value, this cannot be turned into a load under a branch (which would
// make the wave wait for every load in flight, the next batch's stream too)
__device__ __forceinline__ double keep_or_zero(double v, bool keep) {
    const unsigned long long m = keep ? ~0ull : 0ull;
    return __longlong_as_double(static_cast<long long>(static_cast<unsigned long long>(__double_as_longlong(v)) & m));
}
__device__ __forceinline__ float keep_or_zero(float v, bool keep) {
    const int m = keep ? -1 : 0;
    return __int_as_float(__float_as_int(v) & m);
}

// FP64 Gaussian of the pair pass: the table exponential (TAB) or the
// degree-12 polynomial one (no LDS reads); FP32: the hardware exponential
template <typename T, bool TAB>
__device__ __forceinline__ T pair_gauss(const TiledArgs<T> &A, T x2, const double *tab) {
    if constexpr (sizeof(T) == 8 && TAB) return gauss_exp2_tab(x2 * A.mc256, tab);
    else if constexpr (sizeof(T) == 8) return gauss_exp2(x2 * A.mc);
    else return __builtin_amdgcn_exp2f(x2 * A.mc);
}

// The pair's sums over its modes of a = |g|^2 (t + G(x - hw)) and
// b = |g|^2 (t + G(x + hw)), t = N (G(x + hw) + G(x - hw)), x = de; the
// occupation factors are the pair's.  Slots past nm, and every slot of a
// masked lane (v false), count as empty.
template <typename T, int NM, bool TAB>
__device__ __forceinline__ void pair_mode_sums(const TiledArgs<T> &A, T de, const Pair2<T> (&w)[NM],
                                               const T (&g)[NM], bool v, const double *s_tab, T &sa, T &sb) {
    const int nm = A.nm;
    sa = T(0);
    sb = T(0);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        const T gm = v && m < nm ? g[m] : T(0);
        const T N = keep_or_zero(w[m].b, gm != T(0));
        const T xa = de + w[m].a, xe = de - w[m].a;
        const T da = pair_gauss<T, TAB>(A, xa * xa, s_tab);
        const T dem = pair_gauss<T, TAB>(A, xe * xe, s_tab);
        const T t = N * (da + dem);
        sa = fma(gm, t + dem, sa);
        sb = fma(gm, t + da, sb);
    }
}

template <typename T, bool LDS, bool PADQ, int NM, bool TAB>
__device__ __forceinline__ void pair_chunk(const TiledArgs<T> &A, const T *__restrict__ fb,
                                           const Pair2<T> *s_ef, const uint32_t *s_kq, int p_lo,
                                           const double *s_tab, unsigned long long *s_j, T scale,
                                           int64_t c, T *__restrict__ part) {
    const int lane = threadIdx.x & 63;
    const int nm = A.nm;   // <= NM
    const int d = A.chunk_dest[c];
    const int64_t beg = A.chunk_beg[c];
    const int len = static_cast<int>(A.chunk_end[c] - beg);
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ gb = A.g2 + beg;
    const StateRec<T> sd = A.st[d];
    const uint32_t kd = PADQ ? sd.kqp : sd.kq;
    const T fd = fb[d];
    const T cfd = T(1) - fd;
    T acc_a = T(0), acc_b = T(0);
    // the stream (partner and |g|^2 slots) runs one batch ahead of the
    // gathers and the evaluation.  The arrays are padded past their end, so
    // no stream load needs a bound.
    // Mode slots past nm (NM rounds nm up) re-read the last mode and count
    // as empty, so the mode loops carry no branch.  The stream values are
    // kept as loaded and masked where they are used: a mask applied at the
    // end of the batch would make the wave wait there for the loads it has
    // just issued.
    // Two register sets alternate (the loop is unrolled twice), so the
    // values loaded for the next batch need no copy at the end of a batch,
    // which would wait for them.
    uint32_t pn0 = pb[lane], pn1 = 0;
    T g0[NM], g1[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) g0[m] = gb[min(m, nm - 1) * A.pld + lane];
    auto batch = [&](int r, const uint32_t pn, const T (&g)[NM], uint32_t &pn_next, T (&g_next)[NM]) {
        const bool v = r + lane < len;
        const int p = static_cast<int>(pn);
        T ep, fp;
        uint32_t kp;
        int pl;
        // A masked lane takes a valid partner (the window's first state, or
        // the destination) and |g|^2 = 0, so its operands are finite and it
        // adds nothing.  The partner's values are loaded unconditionally: a
        // choice between a loaded value and another one is compiled into a
        // branch around the load, which waits for every load in flight.
        if (LDS) {
            pl = v ? p - p_lo : 0;
            const Pair2<T> ef = s_ef[pl];
            ep = ef.a;
            fp = ef.b;
            kp = s_kq[pl];
        } else {
            pl = v ? p : d;
            const StateRec<T> sp = A.st[pl];
            ep = sp.eps;
            kp = PADQ ? sp.kqp : sp.kq;
            fp = fb[pl];
        }
        const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
        const Pair2<T> *__restrict__ wq = A.hwN + static_cast<int64_t>(q) * A.tq;
        Pair2<T> w[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) w[m] = wq[min(m, nm - 1) * A.tm];
        // the next batch's stream loads are issued after this batch's table
        // gathers: loads complete in issue order for the wait counter, so
        // waiting for the gathers does not wait for the stream.  The
        // scheduling barriers keep that order and keep the compiler from
        // sinking any of these loads towards their first use, which would
        // serialise the gathers.
        __builtin_amdgcn_sched_barrier(0);
        pn_next = pb[r + 64 + lane];
#pragma unroll
        for (int m = 0; m < NM; ++m) g_next[m] = gb[min(m, nm - 1) * A.pld + r + 64 + lane];
        __builtin_amdgcn_sched_barrier(0);
        const T ofp = T(1) - fp;
        T sa, sb;
        pair_mode_sums<T, NM, TAB>(A, sd.eps - ep, w, g, v, s_tab, sa, sb);
        const T ta = sa * ofp, tb = sb * fp;
        acc_a += ta;
        acc_b += tb;
        // partner side: -Y = f_d ta - (1 - f_d) tb
        const T y = fma(fd, ta, -cfd * tb);
        if (v) {
            const unsigned long long fx = to_fixed(__builtin_rint(y * scale));
            if (LDS) atomicAdd(s_j + pl, fx);
            else atomicAdd(A.jacc + pl, fx);
        }
    };
    for (int r = 0; r < len; r += 128) {
        batch(r, pn0, g0, pn1, g1);
        if (r + 64 >= len) break;
        batch(r + 64, pn1, g1, pn0, g0);
    }
    acc_a = wave_sum(acc_a);
    acc_b = wave_sum(acc_b);
    if (lane == 0) {
        part[2 * c] = acc_a;
        part[2 * c + 1] = acc_b;
    }
}

// The same pass over a q-ordered tile.  Its records are sorted by the table
// row of q = k_p - k_d (then destination, partner), so the lanes of a batch
// read a few rows of the {hw, N} table instead of one each.  A record's word
// holds the window offsets of its partner (high 16 bits) and destination (low
// 16 bits); the window stages both.  The destination's side of the pair, -y,
// goes to the same fixed-point accumulator as the partner's, +y, so the
// tile has no row partials.  The waves take the tile's batches in turn, so that
// together they sweep its runs: the table rows, the |g|^2 lines and, in the
// passes that write per pair, the output lines in flight belong to one run.
// With 100^3 (198 M channels) against one sorted range per tile and a part of it
// per wave: forward 466 -> 430 us, reverse with channel gradients 1227 -> 1124,
// pair matrix 940 -> 756.  Runs of 384 / 768 / 1536 / 4096 / 16384 records:
// reverse 1124 / 1134 / 1135 / 1146 / 1155 us, pair matrix 756 / 776 / 801 / 832 /
// 879 (727 over 100 calls traced later, 389 FP32); the forward pass, which writes nothing per pair, 420 .. 445 without a trend.
template <typename T, bool PADQ, int NM, bool TAB>
__device__ __forceinline__ void pair_chunk_q(const TiledArgs<T> &A, const Pair2<T> *s_ef, const uint32_t *s_kq,
                                             const double *s_tab, unsigned long long *s_j, T scale, int64_t beg,
                                             int len, int wave, int nw) {
    const int lane = threadIdx.x & 63;
    const int nm = A.nm;
    const int first = wave * 64, step = nw * 64;
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ gb = A.g2 + beg;
    // stream one batch ahead, two register sets (see pair_chunk)
    uint32_t pn0 = pb[first + lane], pn1 = 0;
    T g0[NM], g1[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) g0[m] = gb[min(m, nm - 1) * A.pld + first + lane];
    auto batch = [&](int r, const uint32_t pn, const T (&g)[NM], uint32_t &pn_next, T (&g_next)[NM]) {
        const bool v = r + lane < len;
        // a masked lane takes window slot 0 as both states (q = 0) and adds nothing
        const int wd = v ? static_cast<int>(pn & 0xffffu) : 0;
        const int wp = v ? static_cast<int>(pn >> 16) : 0;
        const Pair2<T> efd = s_ef[wd], efp = s_ef[wp];
        const uint32_t kd = s_kq[wd], kp = s_kq[wp];
        const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
        const Pair2<T> *__restrict__ wq = A.hwN + static_cast<int64_t>(q) * A.tq;
        Pair2<T> w[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) w[m] = wq[min(m, nm - 1) * A.tm];
        __builtin_amdgcn_sched_barrier(0);
        pn_next = pb[r + step + lane];
#pragma unroll
        for (int m = 0; m < NM; ++m) g_next[m] = gb[min(m, nm - 1) * A.pld + r + step + lane];
        __builtin_amdgcn_sched_barrier(0);
        T sa, sb;
        pair_mode_sums<T, NM, TAB>(A, efd.a - efp.a, w, g, v, s_tab, sa, sb);
        const T fd = efd.b, fp = efp.b;
        const T ta = sa * (T(1) - fp), tb = sb * fp;
        const T y = fma(fd, ta, -(T(1) - fd) * tb);
        if (v) {
            const unsigned long long fx = to_fixed(__builtin_rint(y * scale));
            atomicAdd(s_j + wp, fx);
            atomicAdd(s_j + wd, 0ull - fx);
        }
    };
    for (int r = first; r < len; r += 2 * step) {
        batch(r, pn0, g0, pn1, g1);
        if (r + step >= len) break;
        batch(r + step, pn1, g1, pn0, g0);
    }
}

template <typename T, bool PADQ, int NM, bool TAB>
__global__ __launch_bounds__(1024) void k_fwd_pairs(TiledArgs<T> A, const T *__restrict__ f,
                                                    T *__restrict__ part) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    const ScaleIn si = scale_load(A.nmax, A.gmax_bits, A.fmax, MaxList{nullptr, 0});
    unsigned long long *s_j = reinterpret_cast<unsigned long long *>(smem);
    Pair2<T> *s_ef = reinterpret_cast<Pair2<T> *>(s_j + A.lds_states);
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_ef + A.lds_states);
    double *s_tab = reinterpret_cast<double *>(s_kq + A.lds_states);
    const int n = t.lds ? t.p_hi - t.p_lo + 1 : 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const StateRec<T> sr = A.st[t.p_lo + i];
        Pair2<T> ef;
        ef.a = sr.eps;
        ef.b = f[t.p_lo + i];
        s_ef[i] = ef;
        s_kq[i] = PADQ ? sr.kqp : sr.kq;
        s_j[i] = 0ull;
    }
    if constexpr (sizeof(T) == 8 && TAB)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    const T scale = static_cast<T>(sym_scale(si));
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    if (t.lds == 2) {
        const int64_t beg = A.chunk_beg[t.c0];
        pair_chunk_q<T, PADQ, NM, TAB>(A, s_ef, s_kq, s_tab, s_j, scale, beg,
                                       static_cast<int>(A.chunk_end[t.c1 - 1] - beg), wave, nw);
        if (!A.all_q)
            for (int64_t c = 2 * t.c0 + threadIdx.x; c < 2 * t.c1; c += blockDim.x) part[c] = T(0);
    }
    for (int64_t c = t.c0 + wave; t.lds != 2 && c < t.c1; c += nw) {
        if (t.lds)
            pair_chunk<T, true, PADQ, NM, TAB>(A, f, s_ef, s_kq, t.p_lo, s_tab, s_j, scale, c, part);
        else
            pair_chunk<T, false, PADQ, NM, TAB>(A, f, s_ef, s_kq, t.p_lo, s_tab, s_j, scale, c, part);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const unsigned long long v = s_j[i];
        if (v) atomicAdd(A.jacc + t.p_lo + i, v);
    }
}

// ---- reverse, single copy over pair records ----------------------------------
// Each channel (d, p, nu), d < p, of a pair record enters L = sum lam I through
// (lam_d - lam_p) X with X = K |g|^2 [(1 - f_d) bh f_p - f_d ah (1 - f_p)]
// (ah = t + G(x - hw), bh = t + G(x + hw), t = N (G(x + hw) + G(x - hw)),
// x = e_d - e_p).  Hence, with dl = lam_d - lam_p:
//   dL/df_d  += -K dl |g|^2 (ah (1 - f_p) + bh f_p)          (row side, registers)
//   dL/df_p  +=  K dl |g|^2 (bh (1 - f_d) + ah f_d)          (partner side, fixed point)
//   dL/d|g|^2 =  K dl ((1 - f_d) bh f_p - f_d ah (1 - f_p))   (one writer per channel;
//                chan0 holds the record's first channel when its slots are the
//                consecutive channels of the caller's list, else -1)
// The partner side of a pair is summed over its modes and added with one
// integer atomic, on the scale of vjp_scale.  Each channel is read once.
__device__ __forceinline__ double vjp_scale(const ScaleIn &s) {
    // |dl| <= 2 max |lam|: a state's column is at most 2 max|lam| (2 N_max + 1) G_max
    // (times occ_factor when f leaves [0, 1])
    return scale_of_bound(2.0 * wave_max(s.l, s.one) * (2.0 * wave_max(s.n, s.one) + 1.0) * s.g * occ_factor(s));
}

// threads per workgroup of the pair reverse pass: 16 waves, as the forward
// (a lane holds at most 128 registers; the pass needs about 100 with the
// modes summed per pair)
constexpr int kVjpPairThreads = 1024;

// The pair's sums over its modes of |g|^2 ah and |g|^2 bh, and per mode
// dL/d|g|^2 = kb bh - ka ah (gv); empty slots as in pair_mode_sums.
template <typename T, int NM, bool TAB>
__device__ __forceinline__ void vjp_mode_sums(const TiledArgs<T> &A, T x, T kb, T ka, const Pair2<T> (&w)[NM],
                                              const T (&g)[NM], bool v, const double *s_tab, T &sa, T &sb,
                                              double (&gv)[NM]) {
    const int nm = A.nm;
    sa = T(0);
    sb = T(0);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        const Pair2<T> wm = w[m];
        const T gm = v && m < nm ? g[m] : T(0);
        const T N = keep_or_zero(wm.b, gm != T(0));
        const T xa = x + wm.a, xe = x - wm.a;
        const T da = pair_gauss<T, TAB>(A, xa * xa, s_tab);
        const T dem = pair_gauss<T, TAB>(A, xe * xe, s_tab);
        const T t = N * (da + dem);
        const T ah = t + dem, bh = t + da;
        sa = fma(gm, ah, sa);
        sb = fma(gm, bh, sb);
        gv[m] = static_cast<double>(fma(kb, bh, -ka * ah));
    }
}

// Writes (gg2_mode 1) or adds (2) the record's dL/d|g|^2 to its channels:
// c0 >= 0 when they are the consecutive channels c0, c0 + 1, ..; else each
// slot's channel is cb[m pld] (-1: no channel)
template <int NM>
__device__ __forceinline__ void write_gg2(double *__restrict__ gg2, int gg2_mode, int32_t c0,
                                          const int32_t *__restrict__ cb, int64_t pld, int nm,
                                          const double (&gv)[NM]) {
    // The overwriting stores do not share instructions with the accumulating
    // ones: a store of either a loaded value or another would wait for every
    // load in flight, the next batch's stream too.
    if (c0 >= 0 && NM == nm && (NM & 1) == 0 && (c0 & 1) == 0) {
        // 16-byte aligned: the lane writes them as whole pairs
        double2 *dst = reinterpret_cast<double2 *>(gg2 + c0);
        if (gg2_mode == 2) {
#pragma unroll
            for (int k = 0; k < NM / 2; ++k) {
                double2 o = dst[k];
                o.x += gv[2 * k];
                o.y += gv[2 * k + 1];
                dst[k] = o;
            }
        } else {
#pragma unroll
            for (int k = 0; k < NM / 2; ++k) dst[k] = make_double2(gv[2 * k], gv[2 * k + 1]);
        }
    } else if (c0 >= 0 && gg2_mode != 2) {
#pragma unroll
        for (int m = 0; m < NM; ++m)
            if (m < nm) gg2[c0 + m] = gv[m];
    } else {
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            if (m >= nm) break;
            const int32_t ch = c0 >= 0 ? c0 + m : cb[m * pld];
            if (ch >= 0) gg2[ch] = gg2_mode == 2 ? gg2[ch] + gv[m] : gv[m];
        }
    }
}

// Lanes of a wave hand values over through LDS: the writes above are seen by the
// reads below.
__device__ __forceinline__ void wave_lds_sync() {
#ifdef __HIP__
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#else
    (void)__shfl(0, 0, 64);
#endif
}

// The same for the 64 records of a wave at once (every lane calls it; v: the
// lane has a record).  Each record's channels are 8 nm consecutive bytes in a
// place of its own, so a lane that writes its record takes a cache line a lane
// and an instruction; where all records have consecutive channels the wave's
// values go through LDS (s_st, 64 NM doubles of the wave) and are written in
// channel order instead, 64 / nm records an instruction.  Measured with gradients
// (nm 6, 198 M channels) 1174 -> 1156 us, (nm 3, 13.5 M channels) 92 -> 82 us; the
// same values written to consecutive memory would take 879 us: what is left is
// the runs of 48 bytes being scattered, a request each to L2.
template <int NM>
__device__ __forceinline__ void wave_write_gg2(double *__restrict__ gg2, int gg2_mode, bool v, int32_t c0,
                                               const int32_t *__restrict__ cb, int64_t pld, int nm,
                                               const double (&gv)[NM], double *s_st) {
    if (s_st == nullptr || NM != nm || __ballot(v && c0 < 0) != 0) {
        if (v) write_gg2<NM>(gg2, gg2_mode, c0, cb, pld, nm, gv);
        return;
    }
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int m = 0; m < NM; ++m) s_st[lane * NM + m] = gv[m];
    wave_lds_sync();
    const int32_t cv = v ? c0 : -1;
    if (gg2_mode == 2) {
#pragma unroll
        for (int j = 0; j < NM; ++j) {
            const int u = j * 64 + lane, rec = u / NM;
            const int32_t ch = __shfl(cv, rec, 64);
            if (ch >= 0) gg2[ch + (u - rec * NM)] += s_st[u];
        }
    } else {
#pragma unroll
        for (int j = 0; j < NM; ++j) {
            const int u = j * 64 + lane, rec = u / NM;
            const int32_t ch = __shfl(cv, rec, 64);
            if (ch >= 0) gg2[ch + (u - rec * NM)] = s_st[u];
        }
    }
    wave_lds_sync();   // the next batch overwrites s_st
}

template <typename T, bool LDS, bool PADQ, int NM, bool TAB>
__device__ __forceinline__ void vjp_pair_chunk(const TiledArgs<T> &A, const T *__restrict__ fb,
                                               const T *__restrict__ lb, const Pair2<T> *s_ef,
                                               const uint32_t *s_kq, const T *s_l, int p_lo,
                                               const double *s_tab, unsigned long long *s_j, T scale,
                                               int64_t c, T *__restrict__ part, bool want_f,
                                               const int32_t *__restrict__ chan,
                                               const int32_t *__restrict__ chan0, double *__restrict__ gg2,
                                               int gg2_mode) {
    const int lane = threadIdx.x & 63;
    const int nm = A.nm;
    const int d = A.chunk_dest[c];
    const int64_t beg = A.chunk_beg[c];
    const int len = static_cast<int>(A.chunk_end[c] - beg);
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ gb = A.g2 + beg;
    const int32_t *__restrict__ cb = chan + beg;
    const int32_t *__restrict__ cb0 = chan0 + beg;
    const StateRec<T> sd = A.st[d];
    const uint32_t kd = PADQ ? sd.kqp : sd.kq;
    const T fd = fb[d];
    const T cfd = T(1) - fd;
    const T ld = lb[d];
    T acc = T(0);
    uint32_t pn = pb[lane];
    for (int r = 0; r < len; r += 64) {
        const bool v = r + lane < len;
        const uint32_t pn_next = pb[r + 64 + lane];
        // mode slots past nm re-read the last mode and count as empty; the
        // values are masked where they are used (see pair_chunk)
        T g[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) g[m] = gb[min(m, nm - 1) * A.pld + r + lane];
        const int32_t c0 = gg2_mode ? cb0[r + lane] : -1;
        const int p = static_cast<int>(pn);
        T ep, fp, lp;
        uint32_t kp;
        int pl;
        // a masked lane takes a valid partner and |g|^2 = 0 (see pair_chunk)
        if (LDS) {
            pl = v ? p - p_lo : 0;
            const Pair2<T> ef = s_ef[pl];
            ep = ef.a;
            fp = ef.b;
            lp = s_l[pl];
            kp = s_kq[pl];
        } else {
            pl = v ? p : d;
            const StateRec<T> sp = A.st[pl];
            ep = sp.eps;
            kp = PADQ ? sp.kqp : sp.kq;
            fp = fb[pl];
            lp = lb[pl];
        }
        const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
        const Pair2<T> *__restrict__ wq = A.hwN + static_cast<int64_t>(q) * A.tq;
        Pair2<T> w[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) w[m] = wq[min(m, nm - 1) * A.tm];
        // all table gathers are in flight before the first is waited for
        __builtin_amdgcn_sched_barrier(0);
        const T x = sd.eps - ep;
        const T ofp = T(1) - fp;
        const T dl = ld - lp;
        // per mode dL/d|g|^2 = kb bh - ka ah; the pair's sums of |g|^2 ah and
        // |g|^2 bh serve both occupation sides
        const T kb = A.K * dl * cfd * fp, ka = A.K * dl * fd * ofp;
        T sa, sb;
        double gv[NM];
        vjp_mode_sums<T, NM, TAB>(A, x, kb, ka, w, g, v, s_tab, sa, sb, gv);
        acc += dl * fma(sa, ofp, sb * fp);
        const T y = dl * fma(sb, cfd, sa * fd);
        // consecutive records of a row write consecutive memory when their
        // channels are consecutive in the caller's order
        if (gg2_mode && v) write_gg2<NM>(gg2, gg2_mode, c0, cb + r + lane, A.pld, nm, gv);
        if (want_f && v) {
            const unsigned long long fx = to_fixed(__builtin_rint(y * scale));
            if (LDS) atomicAdd(s_j + pl, fx);
            else atomicAdd(A.jacc + pl, fx);
        }
        pn = pn_next;
    }
    if (!want_f) return;
    acc = wave_sum(acc);
    if (lane == 0) part[c] = acc;
}

// The reverse pass over a q-ordered tile (see pair_chunk_q): both sides of a
// pair go to the fixed-point accumulator, -K dl (ah (1 - f_p) + bh f_p) |g|^2
// summed over modes to the destination and the partner's side as in
// vjp_pair_chunk.
template <typename T, bool PADQ, int NM, bool TAB>
__device__ __forceinline__ void vjp_pair_chunk_q(const TiledArgs<T> &A, const Pair2<T> *s_ef,
                                                 const uint32_t *s_kq, const T *s_l, const double *s_tab,
                                                 unsigned long long *s_j, T scale, int64_t beg, int len,
                                                 int wave, int nw, bool want_f, const int32_t *__restrict__ chan,
                                                 const int32_t *__restrict__ chan0, double *__restrict__ gg2,
                                                 int gg2_mode, double *s_st) {
    const int lane = threadIdx.x & 63;
    const int nm = A.nm;
    const int first = wave * 64, step = nw * 64;
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ gb = A.g2 + beg;
    const int32_t *__restrict__ cb = chan + beg;
    const int32_t *__restrict__ cb0 = chan0 + beg;
    // stream one batch ahead, two register sets (see pair_chunk)
    uint32_t pn0 = pb[first + lane], pn1 = 0;
    int32_t h0 = gg2_mode ? cb0[first + lane] : -1, h1 = -1;
    T g0[NM], g1[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) g0[m] = gb[min(m, nm - 1) * A.pld + first + lane];
    auto batch = [&](int r, const uint32_t pn, const T (&g)[NM], const int32_t c0, uint32_t &pn_next,
                     T (&g_next)[NM], int32_t &c0_next) {
        const bool v = r + lane < len;
        // a masked lane takes window slot 0 as both states and adds nothing
        const int wd = v ? static_cast<int>(pn & 0xffffu) : 0;
        const int wp = v ? static_cast<int>(pn >> 16) : 0;
        const Pair2<T> efd = s_ef[wd], efp = s_ef[wp];
        const T ld = s_l[wd], lp = s_l[wp];
        const uint32_t kd = s_kq[wd], kp = s_kq[wp];
        const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
        const Pair2<T> *__restrict__ wq = A.hwN + static_cast<int64_t>(q) * A.tq;
        Pair2<T> w[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) w[m] = wq[min(m, nm - 1) * A.tm];
        __builtin_amdgcn_sched_barrier(0);
        pn_next = pb[r + step + lane];
#pragma unroll
        for (int m = 0; m < NM; ++m) g_next[m] = gb[min(m, nm - 1) * A.pld + r + step + lane];
        c0_next = gg2_mode ? cb0[r + step + lane] : -1;
        __builtin_amdgcn_sched_barrier(0);
        const T fd = efd.b, cfd = T(1) - fd, fp = efp.b, ofp = T(1) - fp;
        const T dl = ld - lp;
        const T kb = A.K * dl * cfd * fp, ka = A.K * dl * fd * ofp;
        T sa, sb;
        double gv[NM];
        vjp_mode_sums<T, NM, TAB>(A, efd.a - efp.a, kb, ka, w, g, v, s_tab, sa, sb, gv);
        if (gg2_mode) wave_write_gg2<NM>(gg2, gg2_mode, v, c0, cb + r + lane, A.pld, nm, gv, s_st);
        if (want_f && v) {
            const T rd = dl * fma(sa, ofp, sb * fp);
            const T y = dl * fma(sb, cfd, sa * fd);
            atomicAdd(s_j + wp, to_fixed(__builtin_rint(y * scale)));
            atomicAdd(s_j + wd, to_fixed(__builtin_rint(-rd * scale)));
        }
    };
    for (int r = first; r < len; r += 2 * step) {
        batch(r, pn0, g0, h0, pn1, g1, h1);
        if (r + step >= len) break;
        batch(r + step, pn1, g1, h1, pn0, g0, h0);
    }
}

template <typename T, bool PADQ, int NM, bool TAB>
__global__ __launch_bounds__(kVjpPairThreads) void k_vjp_pairs(TiledArgs<T> A, const T *__restrict__ f,
                                                    const T *__restrict__ lam, T *__restrict__ part, int want_f,
                                                    MaxList lmax,
                                                    const int32_t *__restrict__ chan,
                                                    const int32_t *__restrict__ chan0, double *__restrict__ gg2,
                                                    int gg2_mode, int staged) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    const ScaleIn si = scale_load(A.nmax, A.gmax_bits, A.fmax, lmax);
    unsigned long long *s_j = reinterpret_cast<unsigned long long *>(smem);
    Pair2<T> *s_ef = reinterpret_cast<Pair2<T> *>(s_j + A.lds_states);
    T *s_l = reinterpret_cast<T *>(s_ef + A.lds_states);
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_l + A.lds_states);
    double *s_tab = reinterpret_cast<double *>(s_kq + A.lds_states);
    const int n = t.lds ? t.p_hi - t.p_lo + 1 : 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const StateRec<T> sr = A.st[t.p_lo + i];
        Pair2<T> ef;
        ef.a = sr.eps;
        ef.b = f[t.p_lo + i];
        s_ef[i] = ef;
        s_l[i] = lam[t.p_lo + i];
        s_kq[i] = PADQ ? sr.kqp : sr.kq;
        s_j[i] = 0ull;
    }
    if constexpr (sizeof(T) == 8 && TAB)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    const T scale = static_cast<T>(vjp_scale(si));
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    double *s_st = staged ? s_tab + (sizeof(T) == 8 ? kExpTab : 0) + wave * 64 * NM : nullptr;
    if (t.lds == 2) {
        const int64_t beg = A.chunk_beg[t.c0];
        vjp_pair_chunk_q<T, PADQ, NM, TAB>(A, s_ef, s_kq, s_l, s_tab, s_j, scale, beg,
                                           static_cast<int>(A.chunk_end[t.c1 - 1] - beg), wave, nw, want_f != 0, chan,
                                           chan0, gg2, gg2_mode, s_st);
        if (want_f && !A.all_q)
            for (int64_t c = t.c0 + threadIdx.x; c < t.c1; c += blockDim.x) part[c] = T(0);
    }
    for (int64_t c = t.c0 + wave; t.lds != 2 && c < t.c1; c += nw) {
        if (t.lds)
            vjp_pair_chunk<T, true, PADQ, NM, TAB>(A, f, lam, s_ef, s_kq, s_l, t.p_lo, s_tab, s_j, scale, c, part,
                                                   want_f != 0, chan, chan0, gg2, gg2_mode);
        else
            vjp_pair_chunk<T, false, PADQ, NM, TAB>(A, f, lam, s_ef, s_kq, s_l, t.p_lo, s_tab, s_j, scale, c,
                                                    part, want_f != 0, chan, chan0, gg2, gg2_mode);
    }
    if (!want_f) return;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const unsigned long long v = s_j[i];
        if (v) atomicAdd(A.jacc + t.p_lo + i, v);
    }
}

// dL/df_d = K [-(row partials, chunk order) + partner side], then the
// epilogue; the partner-side accumulator of d is cleared for the next call.
template <typename T>
__global__ void k_vjp_pairs_finish(TiledArgs<T> A, const T *__restrict__ part,
                                   MaxList lmax, Epi<T> E) {
    const double inv = 1.0 / vjp_scale(scale_load(A.nmax, A.gmax_bits, A.fmax, lmax));
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= A.S) return;
    T a = T(0);
    if (!A.all_q)
        for (int c = A.dest_chunk[d]; c < A.dest_chunk[d + 1]; ++c) a += part[c];
    const long long j = static_cast<long long>(A.jacc[d]);
    A.jacc[d] = 0ull;
    const T jside = static_cast<T>(static_cast<double>(j) * inv);
    apply_epi(E, 0, d, A.S, A.K * (jside - a));
}

// I_d = K [(1 - f_d) sum b - f_d sum a] from the row side (chunk partials in
// chunk order) plus the partner side, then the epilogue; the partner-side
// accumulator of d is cleared for the next call.
template <typename T>
__global__ void k_sym_finish(TiledArgs<T> A, const T *__restrict__ f, const T *__restrict__ part,
                             Epi<T> E) {
    const double inv = 1.0 / sym_scale(scale_load(A.nmax, A.gmax_bits, A.fmax, MaxList{nullptr, 0}));
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= A.S) return;
    T a = T(0), b = T(0);
    if (!A.all_q)
        for (int c = A.dest_chunk[d]; c < A.dest_chunk[d + 1]; ++c) {
            a += part[2 * c];
            b += part[2 * c + 1];
        }
    const long long j = static_cast<long long>(A.jacc[d]);
    A.jacc[d] = 0ull;
    const T fd = f[d];
    const T jside = static_cast<T>(static_cast<double>(j) * inv);
    apply_epi(E, 0, d, A.S, A.K * ((T(1) - fd) * b - fd * a + jside));
}

// destinations with several chunks: sum their partials in chunk order
template <typename T>
__global__ void k_tiled_finish(TiledArgs<T> A, const T *__restrict__ f, int64_t ldf,
                               const T *__restrict__ part, Epi<T> E) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= A.S) return;
    const int c0 = A.dest_chunk[d], c1 = A.dest_chunk[d + 1];
    if (c1 - c0 == 1) return;
    const int b = blockIdx.y;
    const T *pb = part + static_cast<int64_t>(b) * A.n_chunks * 2;
    T a = T(0), bb = T(0);
    for (int c = c0; c < c1; ++c) {
        a += pb[2 * c];
        bb += pb[2 * c + 1];
    }
    const T fd = f[static_cast<int64_t>(b) * ldf + d];
    apply_epi(E, b, d, A.S, A.K * ((T(1) - fd) * bb - fd * a));
}

// ---- reverse, LDS-tiled ---------------------------------------------------
// Same tiles, chunks and stream pipeline as the forward pass.  Per entry:
//   dL/df_d  += -K (lam_d - lam_p) (a (1 - f_p) + b f_p)
//   dL/dg2_c  =  K (lam_d - lam_p) (bh f_p (1 - f_d) - ah f_d (1 - f_p))   (p > d only)
// The partner's {eps, f} and k come from LDS, lam_p from global memory.
template <typename T, bool LDS, bool PADQ, int U>
__device__ __forceinline__ void vjp_chunk2(const TiledArgs<T> &A, const T *__restrict__ fb,
                                           const T *__restrict__ lb, const Pair2<T> *s_ef,
                                           const uint32_t *s_kq, int p_lo, const double *s_tab,
                                           int64_t c, T *__restrict__ part, const Epi<T> &E,
                                           const int32_t *__restrict__ ent_chan,
                                           double *__restrict__ gg2, int gg2_mode) {
    const int lane = threadIdx.x & 63;
    const int d = A.chunk_dest[c];
    const int64_t beg = A.chunk_beg[c];
    const int len = static_cast<int>(A.chunk_beg[c + 1] - beg);
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ gb = A.g2 + beg;
    const int32_t *__restrict__ cb = ent_chan + beg;
    const StateRec<T> sd = A.st[d];
    const uint32_t kd = PADQ ? sd.kqp : sd.kq;
    const T fd = fb[d];
    const T ld = lb[d];
    T acc = T(0);
    // one batch of gathered operands: coupling, energy difference, partner
    // occupation, lam_d - lam_p, {hw, N}, and the dL/d|g|^2 slot this entry
    // writes (-1: none) with its previous value when accumulating
    struct Gath {
        T g[U], de[U], fp[U], dl[U];
        Pair2<T> wn[U];
        int32_t ch[U];
        double old[U];
    };
    uint32_t pn1[U];
    T gs1[U];
    Gath G0;
    auto load_stream = [&](int r0, uint32_t (&pn)[U], T (&gs)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pn[u] = pb[r0 + u * 64 + lane];
            gs[u] = gb[r0 + u * 64 + lane];
        }
    };
    auto gather = [&](auto masked, const uint32_t (&pn)[U], const T (&gs)[U], int r0, Gath &o) {
        constexpr bool M = decltype(masked)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int rel = r0 + u * 64 + lane;
            const bool v = !M || rel < len;
            const int p = static_cast<int>(pn[u] >> 3);
            T ep, fp;
            uint32_t kp;
            if (LDS) {
                // a masked lane reads slot 0 (inside the allocation) and then
                // replaces what it read: partner = destination, so its table
                // index is the q = 0 entry and its operands are finite,
                // whatever the slot holds
                const int pl = v ? p - p_lo : 0;
                const Pair2<T> ef = s_ef[pl];
                ep = v ? ef.a : sd.eps;
                fp = v ? ef.b : T(0);
                kp = v ? s_kq[pl] : kd;
            } else {
                const StateRec<T> sp = A.st[p];
                ep = sp.eps;
                kp = PADQ ? sp.kqp : sp.kq;
                fp = fb[p];
            }
            const T lp = lb[p];
            const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff
                               : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
            const Pair2<T> w = A.hwN[static_cast<int64_t>(q) * A.tq + static_cast<int64_t>(pn[u] & 7u) * A.tm];
            if constexpr (M) {
                // a table entry without channels may hold a non-finite N
                o.wn[u].a = v ? w.a : T(0);
                o.wn[u].b = v ? w.b : T(0);
                o.g[u] = v ? gs[u] : T(0);
            } else {
                o.wn[u] = w;
                o.g[u] = gs[u];
            }
            o.de[u] = sd.eps - ep;
            o.fp[u] = fp;
            o.dl[u] = ld - lp;
            const bool wr = gg2_mode && v && p > d;
            o.ch[u] = wr ? cb[rel] : -1;
            o.old[u] = (wr && gg2_mode == 2) ? gg2[o.ch[u]] : 0.0;
        }
    };
    using Masked = std::integral_constant<bool, true>;
    using Full = std::integral_constant<bool, false>;
    {
        uint32_t pn0[U];
        T gs0[U];
        load_stream(0, pn0, gs0);
        load_stream(64 * U, pn1, gs1);
        if (64 * U <= len) gather(Full{}, pn0, gs0, 0, G0);
        else gather(Masked{}, pn0, gs0, 0, G0);
    }
    for (int r = 0; r < len; r += 64 * U) {
        Gath G1;
        if (r + 128 * U <= len) gather(Full{}, pn1, gs1, r + 64 * U, G1);
        else gather(Masked{}, pn1, gs1, r + 64 * U, G1);
        load_stream(r + 128 * U, pn1, gs1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T xa = G0.de[u] + G0.wn[u].a, xe = G0.de[u] - G0.wn[u].a;
            const T da = stream_gauss(A, xa * xa, s_tab);
            const T dem = stream_gauss(A, xe * xe, s_tab);
            const T t = G0.wn[u].b * (da + dem);
            const T ah = t + dem, bh = t + da;
            const T fp = G0.fp[u], dl = G0.dl[u];
            acc += dl * G0.g[u] * (ah * (T(1) - fp) + bh * fp);
            if (G0.ch[u] >= 0)
                gg2[G0.ch[u]] = G0.old[u] + static_cast<double>(
                                                A.K * dl * (bh * fp * (T(1) - fd) - ah * fd * (T(1) - fp)));
        }
        G0 = G1;
    }
    if (E.mode < 0) return;
    acc = wave_sum(acc);
    if (lane == 0) {
        if (A.dest_chunk[d + 1] - A.dest_chunk[d] == 1)
            apply_epi(E, 0, d, A.S, -A.K * acc);
        else
            part[c] = acc;
    }
}

template <typename T, int U, bool PADQ>
__global__ __launch_bounds__(512) void k_vjp_tiled(TiledArgs<T> A, const T *__restrict__ f,
                                                   const T *__restrict__ lam, T *__restrict__ part,
                                                   Epi<T> E, const int32_t *__restrict__ ent_chan,
                                                   double *__restrict__ gg2, int gg2_mode) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    Pair2<T> *s_ef = reinterpret_cast<Pair2<T> *>(smem);
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_ef + A.lds_states);
    double *s_tab = reinterpret_cast<double *>(s_kq + A.lds_states);
    if (t.lds) {
        const int n = t.p_hi - t.p_lo + 1;
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const StateRec<T> sr = A.st[t.p_lo + i];
            Pair2<T> ef;
            ef.a = sr.eps;
            ef.b = f[t.p_lo + i];
            s_ef[i] = ef;
            s_kq[i] = PADQ ? sr.kqp : sr.kq;
        }
    }
    if constexpr (sizeof(T) == 8)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    for (int64_t c = t.c0 + wave; c < t.c1; c += nw) {
        if (t.lds)
            vjp_chunk2<T, true, PADQ, U>(A, f, lam, s_ef, s_kq, t.p_lo, s_tab, c, part, E,
                                         ent_chan, gg2, gg2_mode);
        else
            vjp_chunk2<T, false, PADQ, U>(A, f, lam, s_ef, s_kq, t.p_lo, s_tab, c, part, E,
                                          ent_chan, gg2, gg2_mode);
    }
}

template <typename T>
__global__ void k_vjp_tiled_finish(TiledArgs<T> A, const T *__restrict__ part, Epi<T> E) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= A.S) return;
    const int c0 = A.dest_chunk[d], c1 = A.dest_chunk[d + 1];
    if (c1 - c0 == 1) return;
    T a = T(0);
    for (int c = c0; c < c1; ++c) a += part[c];
    apply_epi(E, 0, d, A.S, -A.K * a);
}

// ---- transport iteration, LDS-tiled -------------------------------------
// x_new_d = tau_d (rhs_d + sum_entries W_e x_p) for the three field
// directions.  The partner window of x is staged in LDS (3 values per state)
// when the plan's LDS budget allows it, else x_p is gathered from global memory.
template <typename T, bool LDS>
__device__ __forceinline__ void tr_chunk(const TiledArgs<T> &A, const T *__restrict__ W,
                                         const Vec4<T> *__restrict__ x, const T *s_x, int p_lo,
                                         int64_t c, const Vec4<T> *__restrict__ rhs,
                                         const T *__restrict__ tau, Vec4<T> *__restrict__ part,
                                         Vec4<T> *__restrict__ x_new) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 63;
    const int d = A.chunk_dest[c];
    const int64_t beg = A.chunk_beg[c];
    const int len = static_cast<int>(A.chunk_beg[c + 1] - beg);
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ wb = W + beg;
    T a0 = T(0), a1 = T(0), a2 = T(0);
    auto load = [&](int r0, uint32_t (&pn)[U], T (&w)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pn[u] = pb[r0 + u * 64 + lane];
            w[u] = wb[r0 + u * 64 + lane];
        }
    };
    auto body = [&](auto masked, int r, const uint32_t (&pn)[U], const T (&w)[U]) {
        constexpr bool M = decltype(masked)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool v = !M || r + u * 64 + lane < len;
            const int p = static_cast<int>(pn[u] >> 3);
            T x0, x1, x2;
            if (LDS) {
                // a masked lane reads slot 0 and discards it (its weight is 0,
                // and 0 times a stale non-finite value would not be)
                const int pl = v ? p - p_lo : 0;
                x0 = v ? s_x[3 * pl] : T(0);
                x1 = v ? s_x[3 * pl + 1] : T(0);
                x2 = v ? s_x[3 * pl + 2] : T(0);
            } else {
                const Vec4<T> xp = x[p];
                x0 = xp.x;
                x1 = xp.y;
                x2 = xp.z;
            }
            const T ww = M ? (v ? w[u] : T(0)) : w[u];
            a0 += ww * x0;
            a1 += ww * x1;
            a2 += ww * x2;
        }
    };
    // the next batch's stream loads are in flight while this batch is
    // reduced; the arrays are padded, so they need no bound
    uint32_t pn0[U];
    T w0[U];
    load(0, pn0, w0);
    for (int r = 0; r < len; r += 64 * U) {
        uint32_t pn1[U];
        T w1[U];
        load(r + 64 * U, pn1, w1);
        if (r + 64 * U <= len) body(std::integral_constant<bool, false>{}, r, pn0, w0);
        else body(std::integral_constant<bool, true>{}, r, pn0, w0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pn0[u] = pn1[u];
            w0[u] = w1[u];
        }
    }
    a0 = wave_sum(a0);
    a1 = wave_sum(a1);
    a2 = wave_sum(a2);
    if (lane == 0) {
        if (A.dest_chunk[d + 1] - A.dest_chunk[d] == 1) {
            const Vec4<T> rr = rhs[d];
            const T t = tau[d];
            Vec4<T> o;
            o.x = t * (rr.x + a0);
            o.y = t * (rr.y + a1);
            o.z = t * (rr.z + a2);
            o.w = T(0);
            x_new[d] = o;
        } else {
            Vec4<T> o;
            o.x = a0;
            o.y = a1;
            o.z = a2;
            o.w = T(0);
            part[c] = o;
        }
    }
}

// W must be padded past its end like the entry arrays.
template <typename T>
__global__ __launch_bounds__(512) void k_tr_tiled(TiledArgs<T> A, int use_lds, const T *__restrict__ W,
                                                  const Vec4<T> *__restrict__ x,
                                                  const Vec4<T> *__restrict__ rhs,
                                                  const T *__restrict__ tau, Vec4<T> *__restrict__ part,
                                                  Vec4<T> *__restrict__ x_new) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    T *s_x = reinterpret_cast<T *>(smem);
    const bool lds = use_lds && t.lds;
    if (lds) {
        const int n = t.p_hi - t.p_lo + 1;
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const Vec4<T> v = x[t.p_lo + i];
            s_x[3 * i] = v.x;
            s_x[3 * i + 1] = v.y;
            s_x[3 * i + 2] = v.z;
        }
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    for (int64_t c = t.c0 + wave; c < t.c1; c += nw) {
        if (lds)
            tr_chunk<T, true>(A, W, x, s_x, t.p_lo, c, rhs, tau, part, x_new);
        else
            tr_chunk<T, false>(A, W, x, s_x, t.p_lo, c, rhs, tau, part, x_new);
    }
}

template <typename T>
__global__ void k_tr_tiled_finish(TiledArgs<T> A, const Vec4<T> *__restrict__ part,
                                  const Vec4<T> *__restrict__ rhs, const T *__restrict__ tau,
                                  Vec4<T> *__restrict__ x_new) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= A.S) return;
    const int c0 = A.dest_chunk[d], c1 = A.dest_chunk[d + 1];
    if (c1 - c0 == 1) return;
    T a0 = T(0), a1 = T(0), a2 = T(0);
    for (int c = c0; c < c1; ++c) {
        a0 += part[c].x;
        a1 += part[c].y;
        a2 += part[c].z;
    }
    const Vec4<T> rr = rhs[d];
    const T t = tau[d];
    Vec4<T> o;
    o.x = t * (rr.x + a0);
    o.y = t * (rr.y + a1);
    o.z = t * (rr.z + a2);
    o.w = T(0);
    x_new[d] = o;
}

// ---- a bath per vector, over pair records -------------------------------------
// The passes over q-ordered pair records for B vectors with a phonon table each.
// A pair's Gaussians do not depend on the bath: with c = |g|^2 (G(x + hw) +
// G(x - hw)) per mode and A0 = sum |g|^2 G(x - hw), B0 = sum |g|^2 G(x + hw),
//   a_b = A0 + sum_m c_m N_b(q, m),   b_b = B0 + sum_m c_m N_b(q, m),
// so a workgroup evaluates them once for VB vectors (as many as its LDS holds: f
// and a fixed-point sum per window state and vector) and each vector adds a short
// sum of N, which the lanes of a batch read from the few rows they share
// (tabN: [group of VB][table row][mode][VB]).  Both sides of a pair are
// fixed-point sums on the vector's own scale.  From 8 vectors on (where the pass over
// entries sums in floating point) a second word keeps 2^-48 of the first one's unit:
// one word's unit is 2^-61 of a bound over all states, which left an element 5e-13 of
// itself in the median and 3e-10 at the 99th percentile (50^3, 20 baths), against
// 4e-15 and 3e-13 by entries and with two words.  A term that is not finite marks the
// two states it belongs to, and a vector whose numbers leave no scale marks all:
// their sums are formed again by k_pv_finish over their own entries, so that such a
// value reaches its partners, and them only.  Bound by LDS atomics (two a pair and
// vector, the second words mostly skipped in FP32) and FP64 issue: 50^3, 6 modes, 20
// baths, whole calls: forward 1002 us by entries, 96 with one word, 110 now (kernel 96
// of it), reverse 2764 and 185.

// tabN of vector blockIdx.y, the {hw, N} table (by vector 0), and the largest finite
// |N|, |f|, |1 - f| and |lam| of the vector (64 values a list), and a Bose plan's
// -f and -lam.
template <typename T> struct PvPrep {
    PackPart<T> p;      // nph: B tables
    T *tab_n;
    int vb;
    int64_t rows;       // table rows (box rows or Nq)
    const T *f, *lam;   // [B][ld], lam may be null
    int64_t ldf, ldl;
    T *neg_f, *neg_l;   // [B][S] or null
    int S;
    double *nmax, *fmax, *cmax, *lmax;   // [B][64]
};
__device__ __forceinline__ double max_finite(double m, double v) {
    v = fabs(v);
    return v <= 1.7976931348623157e308 ? fmax(m, v) : m;
}
template <typename T> __global__ __launch_bounds__(1024) void k_prep_pv(PvPrep<T> P) {
    const int b = blockIdx.y, nb = gridDim.x;
    const PackPart<T> &t = P.p;
    const int64_t tab = static_cast<int64_t>(t.box.n[0]) * t.box.n[1] * t.box.n[2] * t.nm;
    const T *__restrict__ nph = t.nph + b * tab;
    T *__restrict__ out = P.tab_n + (b / P.vb) * P.rows * t.nm * P.vb + b % P.vb;
    double m = 0.0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < t.n;
         i += static_cast<int64_t>(nb) * blockDim.x) {
        const int64_t r = i / t.nm;
        const int nu = static_cast<int>(i - r * t.nm);
        int64_t row = r, src = i;
        if (t.padq) {
            row = t.used[r];
            src = static_cast<int64_t>(box_q(static_cast<int>(row), t.box)) * t.nm + nu;
        }
        const T v = nph[src];
        out[(row * t.nm + nu) * P.vb] = v;
        if (b == 0) {
            Pair2<T> w;
            w.a = t.hw[src];
            w.b = v;
            t.out[t.padq && t.mode_major ? nu * static_cast<int64_t>(t.rows) + row : row * t.nm + nu] = w;
        }
        m = max_finite(m, static_cast<double>(v));
    }
    block_max_to(m, P.nmax + b * 64 + blockIdx.x);
    auto vec = [&](const T *__restrict__ x, T *__restrict__ neg, double *dst, double *dst_c) {
        double mv = 0.0, mc = 0.0;
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < P.S; i += nb * blockDim.x) {
            const T v = x[i];
            if (neg) neg[static_cast<int64_t>(b) * P.S + i] = -v;
            const double u = neg ? -static_cast<double>(v) : static_cast<double>(v);
            mv = max_finite(mv, u);
            mc = max_finite(mc, 1.0 - u);
        }
        __syncthreads();
        block_max_to(mv, dst + b * 64 + blockIdx.x);
        if (!dst_c) return;
        __syncthreads();
        block_max_to(mc, dst_c + b * 64 + blockIdx.x);
    };
    vec(P.f + b * P.ldf, P.neg_f, P.fmax, P.cmax);
    if (P.lam) vec(P.lam + b * P.ldl, P.neg_l, P.lmax, nullptr);
}

template <typename T> struct PvArgs {
    const T *__restrict__ f, *__restrict__ lam;
    int64_t ldf, ldl;
    const T *__restrict__ tab_n;
    int64_t gstride;        // values of tabN per group
    int B, vb, n_list;
    const double *__restrict__ nmax, *__restrict__ fmax, *__restrict__ cmax, *__restrict__ lmax;
    unsigned long long *__restrict__ jacc;   // [B][S]
    uint32_t *__restrict__ bad;              // [B][S] nonzero: the sum is formed again
    unsigned long long *__restrict__ jlo;    // [B][S] second words, or null: one word
};
// The scale of vector b (all lanes of a wave): as sym_scale and vjp_scale, with the
// occupations as they are.  f in [0, 1]: a forward term's products are at most
// max f max (1 - f), a reverse term's at most 1; else 2 max|f| max|1 - f| and
// 2 max(max|f|, max|1 - f|).  0 where the bound leaves no power of two.
template <typename T>
__device__ __forceinline__ double pv_scale(const TiledArgs<T> &A, const PvArgs<T> &V, int b) {
    const MaxList none{nullptr, 0};
    const ScaleIn s = scale_load(MaxList{V.nmax + b * 64, V.n_list}, A.gmax_bits, MaxList{V.fmax + b * 64, V.n_list},
                                 V.lam ? MaxList{V.lmax + b * 64, V.n_list} : none);
    const double mf = wave_max(s.f, s.one), mc = wave_max(list_value(MaxList{V.cmax + b * 64, V.n_list}), s.one);
    const double n = wave_max(s.n, s.one), l = wave_max(s.l, s.one), m = fmax(mf, mc);
    const double occ = V.lam ? 2.0 * l * (m > 1.0 ? 2.0 * m : 1.0) : (m > 1.0 ? 2.0 * mf * mc : mf * mc);
    const double bound = (2.0 * n + 1.0) * s.g * occ;
    if (bound == 0.0) return 1.0;   // every term is 0
    return bound > 1e-200 && bound < 1e200 ? scale_of_bound(bound) : 0.0;
}
// A term z in units of the scale, added to a window state's sum (one or two words);
// false where it is not finite.  A window holds fewer than 2^13 terms of a state, so
// the sum of second words, at most 2^47 each, stays below 2^60.
__device__ __forceinline__ bool pv_add(double z, unsigned long long *j, unsigned long long *lo) {
    if (!(fabs(z) < 4.6e18)) return false;   // 2^62
    const double h = __builtin_rint(z);
    atomicAdd(j, to_fixed(h));
    if (lo) {
        const double l = __builtin_rint((z - h) * 281474976710656.0);   // 2^48
        if (l != 0.0) atomicAdd(lo, to_fixed(l));
    }
    return true;
}

template <typename T, bool PADQ, int NM, bool TAB>
__global__ __launch_bounds__(1024) void k_fwd_pairs_pv(TiledArgs<T> A, PvArgs<T> V) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double s_scale[16];
    const TileRec t = A.tiles[blockIdx.x];
    const int W = A.lds_states, VB = V.vb, b0 = blockIdx.y * VB;
    const int nv = min(VB, V.B - b0);
    double *s_tab = reinterpret_cast<double *>(smem);
    unsigned long long *s_j = reinterpret_cast<unsigned long long *>(s_tab + (sizeof(T) == 8 ? kExpTab : 0));
    unsigned long long *s_lo = V.jlo ? s_j + VB * W : nullptr;
    T *s_f = reinterpret_cast<T *>(s_j + (V.jlo ? 2 : 1) * VB * W);
    T *s_e = s_f + VB * W;
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_e + W);
    const int n = t.p_hi - t.p_lo + 1;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const StateRec<T> sr = A.st[t.p_lo + i];
        s_e[i] = sr.eps;
        s_kq[i] = PADQ ? sr.kqp : sr.kq;
        for (int v = 0; v < nv; ++v) {
            if (s_lo) s_lo[v * W + i] = 0ull;
            s_f[v * W + i] = V.f[static_cast<int64_t>(b0 + v) * V.ldf + t.p_lo + i];
            s_j[v * W + i] = 0ull;
        }
    }
    if constexpr (sizeof(T) == 8 && TAB)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    for (int v = wave; v < nv; v += nw) {
        const double sc = pv_scale(A, V, b0 + v);
        if ((threadIdx.x & 63) == 0) s_scale[v] = sc;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int nm = A.nm;
    const T *__restrict__ tn = V.tab_n + blockIdx.y * V.gstride;
    {
        const int64_t beg = A.chunk_beg[t.c0];
        const int len = static_cast<int>(A.chunk_end[t.c1 - 1] - beg);
        const int first = wave * 64, step = nw * 64;
        const uint32_t *__restrict__ pb = A.pnu + beg;
        const T *__restrict__ gb = A.g2 + beg;
        uint32_t pn = pb[first + lane];
        T g[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) g[m] = gb[min(m, nm - 1) * A.pld + first + lane];
        for (int r = first; r < len; r += step) {
            const bool on = r + lane < len;
            // a masked lane takes window slot 0 as both states and adds nothing
            const int wd = on ? static_cast<int>(pn & 0xffffu) : 0;
            const int wp = on ? static_cast<int>(pn >> 16) : 0;
            const uint32_t kd = s_kq[wd], kp = s_kq[wp];
            const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
            const T x = s_e[wd] - s_e[wp];
            T cm[NM], a0 = T(0), bb = T(0);
            bool has[NM];
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const T w = A.hwN[static_cast<int64_t>(q) * A.tq + min(m, nm - 1) * A.tm].a;
                const T gm = on && m < nm ? g[m] : T(0);
                const T xa = x + w, xe = x - w;
                const T da = pair_gauss<T, TAB>(A, xa * xa, s_tab);
                const T dem = pair_gauss<T, TAB>(A, xe * xe, s_tab);
                cm[m] = gm * (da + dem);
                a0 = fma(gm, dem, a0);
                bb = fma(gm, da, bb);
                has[m] = gm != T(0);
            }
            pn = pb[r + step + lane];
#pragma unroll
            for (int m = 0; m < NM; ++m) g[m] = gb[min(m, nm - 1) * A.pld + r + step + lane];
            const T *__restrict__ nq = tn + static_cast<int64_t>(q) * nm * VB;
            for (int v = 0; v < nv; ++v) {
                T ns = T(0);
#pragma unroll
                for (int m = 0; m < NM; ++m) ns = fma(cm[m], keep_or_zero(nq[min(m, nm - 1) * VB + v], has[m]), ns);
                const T fd = s_f[v * W + wd], fp = s_f[v * W + wp];
                const T ta = (a0 + ns) * (T(1) - fp), tb = (bb + ns) * fp;
                const T y = fma(fd, ta, -(T(1) - fd) * tb);
                if (on) {
                    const double z = static_cast<double>(y) * s_scale[v];
                    const int xp = v * W + wp, xd = v * W + wd;
                    if (pv_add(z, s_j + xp, s_lo ? s_lo + xp : nullptr)) {
                        (void)pv_add(-z, s_j + xd, s_lo ? s_lo + xd : nullptr);
                    } else {
                        uint32_t *bad = V.bad + static_cast<int64_t>(b0 + v) * A.S + t.p_lo;
                        bad[wp] = 1u;
                        bad[wd] = 1u;
                    }
                }
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        for (int v = 0; v < nv; ++v) {
            const int64_t o = static_cast<int64_t>(b0 + v) * A.S + t.p_lo + i;
            const unsigned long long u = s_j[v * W + i];
            if (u) atomicAdd(V.jacc + o, u);
            if (s_lo && s_lo[v * W + i]) atomicAdd(V.jlo + o, s_lo[v * W + i]);
        }
}

// The sums of state d and vector b over d's own entries (the destination layout D):
// - (1 / K) I_d, or with V.lam the reverse pass's sum; used where the fixed point has none.
template <typename T>
__device__ T pv_own_sum(const TiledArgs<T> &D, const PvArgs<T> &V, int b, int d) {
    const T *__restrict__ tn = V.tab_n + (b / V.vb) * V.gstride + b % V.vb;
    const T *__restrict__ f = V.f + b * V.ldf, *__restrict__ lam = V.lam ? V.lam + b * V.ldl : nullptr;
    const StateRec<T> sd = D.st[d];
    const T fd = f[d], ld = lam ? lam[d] : T(0);
    T sa = T(0), sb = T(0), sl = T(0);
    for (int64_t e = D.chunk_beg[D.dest_chunk[d]]; e < D.chunk_beg[D.dest_chunk[d + 1]]; ++e) {
        const uint32_t w = D.pnu[e];
        const int p = static_cast<int>(w >> 3), nu = static_cast<int>(w & 7u);
        const StateRec<T> sp = D.st[p];
        const int64_t q = D.padq ? static_cast<int>(sp.kqp - sd.kqp) + D.qoff : q_linear(sd.kq, sp.kq, D.nq0, D.nq1, D.nq2);
        const T hw = D.hwN[q * D.tq + nu * D.tm].a, N = tn[(q * D.nm + nu) * V.vb], g = D.g2[e];
        const T x = sd.eps - sp.eps, xa = x + hw, xe = x - hw;
        const T da = pair_gauss<T, false>(D, xa * xa, nullptr), dem = pair_gauss<T, false>(D, xe * xe, nullptr);
        const T t = N * (da + dem), a = g * (t + dem), bw = g * (t + da), fp = f[p];
        if (lam) {
            sl += (ld - lam[p]) * (a * (T(1) - fp) + bw * fp);
        } else {
            sa += a * (T(1) - fp);
            sb += bw * fp;
        }
    }
    return lam ? -sl : (T(1) - fd) * sb - fd * sa;
}

// out_b,d = K (fixed-point sum) / scale, then the epilogue; the sums are cleared
// for the next call (grid.y = vector)
template <typename T> __global__ void k_pv_finish(TiledArgs<T> A, TiledArgs<T> D, PvArgs<T> V, Epi<T> E) {
    const int b = blockIdx.y;
    const double sc = pv_scale(A, V, b), inv = sc != 0.0 ? 1.0 / sc : 0.0;
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= A.S) return;
    const int64_t o = static_cast<int64_t>(b) * A.S + d;
    double j = static_cast<double>(static_cast<long long>(V.jacc[o]));
    V.jacc[o] = 0ull;
    if (V.jlo) {
        // (a window's second words may sum to several units of the first)
        j += static_cast<double>(static_cast<long long>(V.jlo[o])) * 3.552713678800501e-15;   // 2^-48
        V.jlo[o] = 0ull;
    }
    T v = static_cast<T>(j * inv);
    if (V.bad[o] != 0u || sc == 0.0) v = pv_own_sum<T>(D, V, b, d);
    V.bad[o] = 0u;
    apply_epi(E, b, d, A.S, A.K * v);
}

// The reverse pass (FP64 plans).  Per pair and vector, with dl = lam_d - lam_p,
// P1 = dl f_d (1 - f_p), P2 = dl f_p (1 - f_d):
//   dL/df_d += -dl (a_b (1 - f_p) + b_b f_p),  dL/df_p += dl (b_b (1 - f_d) + a_b f_d)
// (times K), and a channel's gradient is, summed over the vectors of the group in
// order in the lane that holds the pair,
//   K [ G(x + hw) sum P2 - G(x - hw) sum P1 + (G(x + hw) + G(x - hw)) sum N_b (P2 - P1) ].
// A later group adds to it (gg2_mode 2).
template <bool PADQ, int NM, bool TAB>
__global__ __launch_bounds__(1024) void k_vjp_pairs_pv(TiledArgs<double> A, PvArgs<double> V, int group, int want_f,
                                                       const int32_t *__restrict__ chan,
                                                       const int32_t *__restrict__ chan0, double *__restrict__ gg2,
                                                       int gg2_mode) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double s_scale[16];
    const TileRec t = A.tiles[blockIdx.x];
    const int W = A.lds_states, VB = V.vb, b0 = group * VB;
    const int nv = min(VB, V.B - b0);
    double *s_tab = reinterpret_cast<double *>(smem);
    // {f, lam} first: 16-byte values, and W and VB may both be odd
    Pair2<double> *s_fl = reinterpret_cast<Pair2<double> *>(s_tab + kExpTab);
    unsigned long long *s_j = reinterpret_cast<unsigned long long *>(s_fl + VB * W);
    unsigned long long *s_lo = V.jlo ? s_j + VB * W : nullptr;
    double *s_e = reinterpret_cast<double *>(s_j + (V.jlo ? 2 : 1) * VB * W);
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_e + W);
    const int n = t.p_hi - t.p_lo + 1;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const StateRec<double> sr = A.st[t.p_lo + i];
        s_e[i] = sr.eps;
        s_kq[i] = PADQ ? sr.kqp : sr.kq;
        for (int v = 0; v < nv; ++v) {
            if (s_lo) s_lo[v * W + i] = 0ull;
            Pair2<double> fl;
            fl.a = V.f[static_cast<int64_t>(b0 + v) * V.ldf + t.p_lo + i];
            fl.b = V.lam[static_cast<int64_t>(b0 + v) * V.ldl + t.p_lo + i];
            s_fl[v * W + i] = fl;
            s_j[v * W + i] = 0ull;
        }
    }
    if constexpr (TAB)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    for (int v = wave; v < nv; v += nw) {
        const double sc = pv_scale(A, V, b0 + v);
        if ((threadIdx.x & 63) == 0) s_scale[v] = sc;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int nm = A.nm;
    const double *__restrict__ tn = V.tab_n + group * V.gstride;
    {
        const int64_t beg = A.chunk_beg[t.c0];
        const int len = static_cast<int>(A.chunk_end[t.c1 - 1] - beg);
        const int first = wave * 64, step = nw * 64;
        const uint32_t *__restrict__ pb = A.pnu + beg;
        const double *__restrict__ gb = A.g2 + beg;
        const int32_t *__restrict__ cb = chan + beg;
        const int32_t *__restrict__ cb0 = chan0 + beg;
        for (int r = first; r < len; r += step) {
            const bool on = r + lane < len;
            const uint32_t pn = pb[r + lane];
            const int32_t c0 = gg2_mode ? cb0[r + lane] : -1;
            const int wd = on ? static_cast<int>(pn & 0xffffu) : 0;
            const int wp = on ? static_cast<int>(pn >> 16) : 0;
            const uint32_t kd = s_kq[wd], kp = s_kq[wp];
            const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
            const double x = s_e[wd] - s_e[wp];
            double da[NM], dem[NM], g[NM], rn[NM], a0 = 0.0, bb = 0.0;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const double w = A.hwN[static_cast<int64_t>(q) * A.tq + min(m, nm - 1) * A.tm].a;
                const double gs = gb[min(m, nm - 1) * A.pld + r + lane];
                g[m] = on && m < nm ? gs : 0.0;
                const double xa = x + w, xe = x - w;
                da[m] = pair_gauss<double, TAB>(A, xa * xa, s_tab);
                dem[m] = pair_gauss<double, TAB>(A, xe * xe, s_tab);
                a0 = fma(g[m], dem[m], a0);
                bb = fma(g[m], da[m], bb);
                rn[m] = 0.0;
            }
            const double *__restrict__ nq = tn + static_cast<int64_t>(q) * nm * VB;
            double p1 = 0.0, p2 = 0.0;
            for (int v = 0; v < nv; ++v) {
                const Pair2<double> fd = s_fl[v * W + wd], fp = s_fl[v * W + wp];
                const double dl = fd.b - fp.b;
                const double q1 = dl * fd.a * (1.0 - fp.a), q2 = dl * fp.a * (1.0 - fd.a), dq = q2 - q1;
                double ns = 0.0;
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    const double N = nq[min(m, nm - 1) * VB + v];
                    // a slot without a channel may hold a non-finite N; its
                    // gradient is not written
                    ns = fma(g[m] * (da[m] + dem[m]), keep_or_zero(N, g[m] != 0.0), ns);
                    rn[m] = fma(N, dq, rn[m]);
                }
                p1 += q1;
                p2 += q2;
                if (want_f && on) {
                    const double sc = s_scale[v];
                    const double a = a0 + ns, b = bb + ns;
                    const double rd = dl * fma(a, 1.0 - fp.a, b * fp.a);
                    const double y = dl * fma(b, 1.0 - fd.a, a * fd.a);
                    const int xp = v * W + wp, xd = v * W + wd;
                    uint32_t *bad = V.bad + static_cast<int64_t>(b0 + v) * A.S + t.p_lo;
                    if (!pv_add(y * sc, s_j + xp, s_lo ? s_lo + xp : nullptr)) bad[wp] = 1u;
                    if (!pv_add(-rd * sc, s_j + xd, s_lo ? s_lo + xd : nullptr)) bad[wd] = 1u;
                }
            }
            if (gg2_mode && on) {
                double gv[NM];
#pragma unroll
                for (int m = 0; m < NM; ++m)
                    gv[m] = A.K * (da[m] * p2 - dem[m] * p1 + (da[m] + dem[m]) * rn[m]);
                write_gg2<NM>(gg2, gg2_mode, c0, cb + r + lane, A.pld, nm, gv);
            }
        }
    }
    if (!want_f) return;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        for (int v = 0; v < nv; ++v) {
            const int64_t o = static_cast<int64_t>(b0 + v) * A.S + t.p_lo + i;
            const unsigned long long u = s_j[v * W + i];
            if (u) atomicAdd(V.jacc + o, u);
            if (s_lo && s_lo[v * W + i]) atomicAdd(V.jlo + o, s_lo[v * W + i]);
        }
}

// ---- the pair matrix ---------------------------------------------------------
// Where a call applies one bath's collision integral more than once (RK4 steps,
// the transport iteration, several occupation vectors), the coefficients are
// evaluated once, summed over the modes of each pair, into a matrix over states:
//   M[d][p] = sum over modes of |g|^2 (t + G(x + hw)),  x = e_d - e_p,
// the in-scattering weight b of destination d from partner p.  With tables even
// in q the out-scattering weight a of d to p is M[p][d], so one matrix serves
//   I_d = K [ (1 - f_d) sum_p M[d][p] f_p  -  f_d sum_p M[p][d] (1 - f_p) ]
// and, per field direction, W x of the linearised equation,
//   (W x)_d = K [ (1 - f_d) sum_p M[d][p] x_p + f_d sum_p M[p][d] x_p ].
// It is stored in 64 x 64 blocks (build_matrix_layout), each as 4 x 4 sub-blocks
// of 16 x 16 values, row-major: a wave reads a sub-block as one contiguous run
// for either use (rows for M, columns for its transpose).  Entries without a
// pair are zero from the allocation; every pair's two entries are rewritten by
// k_pair_matrix.  Sums over partners are held in FP64 in both precisions.
struct MxCol {
    int32_t i, j, id_t, pad;   // block row, block column and the block (j, i)
};
template <typename T> struct MxArgs {
    T *__restrict__ m;                     // [blocks][64 x 64]
    const int32_t *__restrict__ pos;       // [S] position of a state
    const int32_t *__restrict__ state;     // [nb 64] state at a position, -1 past the last
    const int32_t *__restrict__ blk;       // [nb][nb] block of (I, J), -1: none
    const int32_t *__restrict__ row;       // [nb + 1]
    const MxCol *__restrict__ col;         // [blocks]
    int nb, S;
};
constexpr int kMxBlock = 64 * 64;

// offset of row r, column c inside a block
__device__ __forceinline__ int mx_inner(int r, int c) {
    return ((((r >> 4) << 2) | (c >> 4)) << 8) | ((r & 15) << 4) | (c & 15);
}

// Fills the matrix from the pair records, in the forward pass's tiles and
// pipeline (see pair_chunk); no occupations enter.  The two 8-byte stores of a
// pair go to different rows for each lane of a q-ordered batch, so the pass is
// bound by the store requests as well as by the exponentials.
template <typename T, bool PADQ, int NM, bool TAB, bool QORD>
__device__ __forceinline__ void mx_chunk(const TiledArgs<T> &A, const MxArgs<T> &X, const T *s_e,
                                         const uint32_t *s_kq, const int32_t *s_pos, const double *s_tab, int64_t c,
                                         int64_t beg, int len, int first, int step) {
    const int lane = threadIdx.x & 63;
    const int nm = A.nm;
    const int dc = QORD ? 0 : A.chunk_dest[c];
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const T *__restrict__ gb = A.g2 + beg;
    uint32_t pn0 = pb[first + lane], pn1 = 0;
    T g0[NM], g1[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) g0[m] = gb[min(m, nm - 1) * A.pld + first + lane];
    auto batch = [&](int r, const uint32_t pn, const T (&g)[NM], uint32_t &pn_next, T (&g_next)[NM]) {
        const bool v = r + lane < len;
        T ed, ep;
        uint32_t kd, kp;
        int xd, xp;
        if (QORD) {
            // a masked lane takes window slot 0 as both states
            const int wd = v ? static_cast<int>(pn & 0xffffu) : 0;
            const int wp = v ? static_cast<int>(pn >> 16) : 0;
            ed = s_e[wd];
            ep = s_e[wp];
            kd = s_kq[wd];
            kp = s_kq[wp];
            xd = s_pos[wd];
            xp = s_pos[wp];
        } else {
            const int p = v ? static_cast<int>(pn) : dc;
            const StateRec<T> sd = A.st[dc], sp = A.st[p];
            ed = sd.eps;
            ep = sp.eps;
            kd = PADQ ? sd.kqp : sd.kq;
            kp = PADQ ? sp.kqp : sp.kq;
            xd = X.pos[dc];
            xp = X.pos[p];
        }
        const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
        const Pair2<T> *__restrict__ wq = A.hwN + static_cast<int64_t>(q) * A.tq;
        Pair2<T> w[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) w[m] = wq[min(m, nm - 1) * A.tm];
        const int bd = xd >> 6, bp = xp >> 6;
        const int id = X.blk[bd * X.nb + bp], it = X.blk[bp * X.nb + bd];
        __builtin_amdgcn_sched_barrier(0);
        pn_next = pb[r + step + lane];
#pragma unroll
        for (int m = 0; m < NM; ++m) g_next[m] = gb[min(m, nm - 1) * A.pld + r + step + lane];
        __builtin_amdgcn_sched_barrier(0);
        T sa, sb;
        pair_mode_sums<T, NM, TAB>(A, ed - ep, w, g, v, s_tab, sa, sb);
        if (v) {
            X.m[static_cast<int64_t>(id) * kMxBlock + mx_inner(xd & 63, xp & 63)] = sb;
            X.m[static_cast<int64_t>(it) * kMxBlock + mx_inner(xp & 63, xd & 63)] = sa;
        }
    };
    for (int r = first; r < len; r += 2 * step) {
        batch(r, pn0, g0, pn1, g1);
        if (r + step >= len) break;
        batch(r + step, pn1, g1, pn0, g0);
    }
}

template <typename T, bool PADQ, int NM, bool TAB>
__global__ __launch_bounds__(1024) void k_pair_matrix(TiledArgs<T> A, MxArgs<T> X) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    // LDS: exponential table (FP64), energies, packed k and positions of the window
    double *s_tab = reinterpret_cast<double *>(smem);
    T *s_e = reinterpret_cast<T *>(s_tab + (sizeof(T) == 8 ? kExpTab : 0));
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_e + A.lds_states);
    int32_t *s_pos = reinterpret_cast<int32_t *>(s_kq + A.lds_states);
    const int n = t.lds == 2 ? t.p_hi - t.p_lo + 1 : 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const StateRec<T> sr = A.st[t.p_lo + i];
        s_e[i] = sr.eps;
        s_kq[i] = PADQ ? sr.kqp : sr.kq;
        s_pos[i] = X.pos[t.p_lo + i];
    }
    if constexpr (sizeof(T) == 8 && TAB)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    if (t.lds == 2) {
        const int64_t beg = A.chunk_beg[t.c0];
        mx_chunk<T, PADQ, NM, TAB, true>(A, X, s_e, s_kq, s_pos, s_tab, t.c0, beg,
                                         static_cast<int>(A.chunk_end[t.c1 - 1] - beg), wave * 64, nw * 64);
        return;
    }
    for (int64_t c = t.c0 + wave; c < t.c1; c += nw)
        mx_chunk<T, PADQ, NM, TAB, false>(A, X, s_e, s_kq, s_pos, s_tab, c, A.chunk_beg[c],
                                          static_cast<int>(A.chunk_end[c] - A.chunk_beg[c]), 0, 64);
}

// Runs of the stored blocks, one a wave: the first r waves take q + 1 blocks, the
// others q (q W + r blocks over W waves).
struct MxRuns {
    int W, q, r;
};
__device__ __forceinline__ int mx_wave_of(const MxRuns &N, int x) {
    const int head = N.r * (N.q + 1);
    return x < head ? x / (N.q + 1) : N.r + (x - head) / N.q;
}

// The matrix and its transpose applied to NC columns, each value read once: every
// wave takes an equal run of the stored blocks, whatever rows they belong to.  Lane (i, g) = (lane / 4, lane %
// 4) holds row i and columns 4 g .. 4 g + 3 of a sub-block.  Rows: sum_p M[d][p]
// u1_p in registers while the block row stays I, then to part1[w + I][64][NC]
// (along a run of blocks w + I never repeats).  Columns: the block's share of the
// transposed product, sum over its rows of M[d][p] u2_d, to part2[block][64][NC].
// The k_mx_* finish kernels add the shares.  Bound by the matrix bytes: four
// sub-blocks are in flight while four are multiplied.  rev != 0 walks the blocks
// backwards: calls that alternate find the end of the last walk in the 256 MB
// memory-side cache.
template <typename T, int NC>
__global__ __launch_bounds__(256, NC == 1 ? 3 : 2) void k_mx_vec(const T *__restrict__ mat,
                                                                 const MxCol *__restrict__ col, MxRuns N,
                                                                 const double *__restrict__ u1,
                                                                 const double *__restrict__ u2,
                                                                 double *__restrict__ part1,
                                                                 double *__restrict__ part2, int rev) {
    const int lane = threadIdx.x & 63;
    const int i = lane >> 2, g = lane & 3;
    int w = static_cast<int>(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    if (rev) w = N.W - 1 - w;
    const int xb = w * N.q + min(w, N.r);
    const int nx = N.q + (w < N.r ? 1 : 0);
    if (nx == 0) return;
    auto at = [&](int k) { return rev ? xb + nx - 1 - min(k, nx - 1) : xb + min(k, nx - 1); };
    const bool h5 = (lane & 32) != 0, h4 = (lane & 16) != 0, h3 = (lane & 8) != 0, h2 = (lane & 4) != 0;
    double v2[4][NC], acc[4][NC], half[4][NC], a0[4][NC], a1[4][NC];
    T w0[4][4], w1[4][4];
    // sub-blocks (0 .. 3, C) of block x and the columns they meet
    auto load = [&](int x, int C, T (&wt)[4][4], double (&a)[4][NC]) {
        const T *__restrict__ m = mat + static_cast<int64_t>(x) * kMxBlock + C * 256 + lane * 4;
#pragma unroll
        for (int R = 0; R < 4; ++R) {
            const Vec4<T> q = *reinterpret_cast<const Vec4<T> *>(m + R * 1024);
            wt[R][0] = q.x;
            wt[R][1] = q.y;
            wt[R][2] = q.z;
            wt[R][3] = q.w;
        }
        const double *__restrict__ ub = u1 + (static_cast<int64_t>(col[x].j) * 64 + C * 16 + 4 * g) * NC;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int k = 0; k < NC; ++k) a[t][k] = ub[t * NC + k];
    };
    auto step = [&](int C, const T (&wt)[4][4], const double (&a)[4][NC]) {
        double cs[4][NC];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int k = 0; k < NC; ++k) cs[t][k] = 0.0;
#pragma unroll
        for (int R = 0; R < 4; ++R)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double m = static_cast<double>(wt[R][t]);
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    acc[R][k] = fma(m, a[t][k], acc[R][k]);
                    cs[t][k] = fma(m, v2[R][k], cs[t][k]);
                }
            }
        // half of the sum over the 16 rows i: lane bits 5 and 4 each halve the
        // four columns
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const double c0 = cs[0][k], c1 = cs[1][k], c2 = cs[2][k], c3 = cs[3][k];
            const double p0 = (h5 ? c2 : c0) + __shfl_xor(h5 ? c0 : c2, 32, 64);
            const double p1 = (h5 ? c3 : c1) + __shfl_xor(h5 ? c1 : c3, 32, 64);
            half[C][k] = (h4 ? p1 : p0) + __shfl_xor(h4 ? p0 : p1, 16, 64);
        }
    };
    // the other half: bits 3 and 2 each halve the four sub-blocks, so that every
    // lane holds one column of the block (no branch around the store: the
    // compiler would sink the row sums past it and hold every operand until then)
    auto end_block = [&](int x) {
        double *__restrict__ pc =
            part2 + (static_cast<int64_t>(x) * 64 + (h3 ? 32 : 0) + (h2 ? 16 : 0) + 4 * g + (h5 ? 2 : 0) + (h4 ? 1 : 0)) * NC;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const double c0 = half[0][k], c1 = half[1][k], c2 = half[2][k], c3 = half[3][k];
            const double p0 = (h3 ? c2 : c0) + __shfl_xor(h3 ? c0 : c2, 8, 64);
            const double p1 = (h3 ? c3 : c1) + __shfl_xor(h3 ? c1 : c3, 8, 64);
            pc[k] = (h2 ? p1 : p0) + __shfl_xor(h2 ? p0 : p1, 4, 64);
        }
    };
    auto begin_row = [&](int I) {
#pragma unroll
        for (int R = 0; R < 4; ++R)
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                v2[R][k] = u2[(static_cast<int64_t>(I) * 64 + R * 16 + i) * NC + k];
                acc[R][k] = 0.0;
            }
    };
    auto end_row = [&](int I) {
        double *__restrict__ po = part1 + static_cast<int64_t>(w + I) * 64 * NC;
#pragma unroll
        for (int R = 0; R < 4; ++R)
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                double s = acc[R][k];
                s += __shfl_xor(s, 1, 64);
                s += __shfl_xor(s, 2, 64);
                if (g == 0) po[(R * 16 + i) * NC + k] = s;
            }
    };
    int x = at(0), I = col[x].i;
    load(x, 0, w0, a0);
    begin_row(I);
    for (int k = 0; k < nx; ++k) {
        const int xn = at(k + 1);
        load(x, 1, w1, a1);
        __builtin_amdgcn_sched_barrier(0);
        step(0, w0, a0);
        load(x, 2, w0, a0);
        __builtin_amdgcn_sched_barrier(0);
        step(1, w1, a1);
        load(x, 3, w1, a1);
        __builtin_amdgcn_sched_barrier(0);
        step(2, w0, a0);
        load(xn, 0, w0, a0);
        __builtin_amdgcn_sched_barrier(0);
        step(3, w1, a1);
        end_block(x);
        const int In = col[xn].i;
        if (In != I) {
            end_row(I);
            begin_row(In);
            I = In;
        }
        x = xn;
    }
    end_row(I);
}

constexpr int kMxParts = 16;   // waves of the finish kernels
// Sums of a block row's partials (1024 threads, thread = position r and one of
// 16 parts of the shares, so that few loads follow each other; the parts are
// added in order): o1 over the waves that held the row, o2 over the blocks of
// its block column.  Threads below 64 hold the totals of position I 64 + r.
template <typename T, int NC>
__device__ __forceinline__ void mx_vec_sums(const MxArgs<T> &X, const double *__restrict__ part1, MxRuns N,
                                            const double *__restrict__ part2, int I, double (&o1)[NC],
                                            double (&o2)[NC]) {
    __shared__ double s_q[kMxParts][2 * NC][64];
    const int r = threadIdx.x & 63, seg = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NC; ++k) o1[k] = o2[k] = 0.0;
    for (int x = X.row[I] + seg; x < X.row[I + 1]; x += kMxParts) {
        const double *__restrict__ p = part2 + (static_cast<int64_t>(X.col[x].id_t) * 64 + r) * NC;
#pragma unroll
        for (int k = 0; k < NC; ++k) o2[k] += p[k];
    }
    if (X.row[I] < X.row[I + 1]) {
        // the waves that held a block of this row (see k_mx_vec)
        const int we = mx_wave_of(N, X.row[I + 1] - 1);
        for (int w = mx_wave_of(N, X.row[I]) + seg; w <= we; w += kMxParts) {
            const double *__restrict__ p = part1 + (static_cast<int64_t>(w + I) * 64 + r) * NC;
#pragma unroll
            for (int k = 0; k < NC; ++k) o1[k] += p[k];
        }
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        s_q[seg][k][r] = o1[k];
        s_q[seg][NC + k][r] = o2[k];
    }
    __syncthreads();
    if (seg == 0) {
#pragma unroll
        for (int k = 0; k < NC; ++k)
#pragma unroll
            for (int q = 1; q < kMxParts; ++q) {
                o1[k] += s_q[q][k][r];
                o2[k] += s_q[q][NC + k][r];
            }
    }
}

// A non-finite value of some state reaches every row of its blocks through the
// blocks' zero entries.  Where a sum of d came out non-finite it is taken again
// over d's own partners (the entry rows of the destination layout).
template <typename T>
__device__ void mx_own_sums(const TiledArgs<T> &A, const MxArgs<T> &X, int d, const double *__restrict__ u1,
                            const double *__restrict__ u2, int nc, int k, double &o1, double &o2) {
    const int xd = X.pos[d];
    int last = -1;
    o1 = o2 = 0.0;
    for (int64_t e = A.chunk_beg[A.dest_chunk[d]]; e < A.chunk_beg[A.dest_chunk[d + 1]]; ++e) {
        const int p = static_cast<int>(A.pnu[e] >> 3);
        if (p == last) continue;
        last = p;
        const int xp = X.pos[p];
        const int64_t id = X.blk[(xd >> 6) * X.nb + (xp >> 6)], it = X.blk[(xp >> 6) * X.nb + (xd >> 6)];
        o1 += static_cast<double>(X.m[id * kMxBlock + mx_inner(xd & 63, xp & 63)]) *
              u1[static_cast<int64_t>(xp) * nc + k];
        o2 += static_cast<double>(X.m[it * kMxBlock + mx_inner(xp & 63, xd & 63)]) *
              u2[static_cast<int64_t>(xp) * nc + k];
    }
}

__device__ __forceinline__ bool mx_finite(double a, double b) { return fabs(a) + fabs(b) < 1.7e308; }

// u1 = f and u2 = 1 - f by position (0 past the last state)
template <typename T>
__global__ void k_mx_load(MxArgs<T> X, const T *__restrict__ f, double *__restrict__ u1, double *__restrict__ u2) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= X.nb * 64) return;
    const int d = X.state[x];
    u1[x] = d >= 0 ? static_cast<double>(f[d]) : 0.0;
    u2[x] = d >= 0 ? static_cast<double>(T(1) - f[d]) : 0.0;
}

// I_d = K [(1 - f_d) o1 - f_d o2] of the loaded vector, then the epilogue of the
// RK4 stage; the next stage's input replaces u1 and u2.  One workgroup per block
// row.  A: the destination layout (k_mx_own_sums).
template <typename T>
__global__ __launch_bounds__(64 * kMxParts) void k_mx_rk_finish(TiledArgs<T> A, MxArgs<T> X, const double *__restrict__ part1,
                                                      MxRuns N, const double *__restrict__ part2, double K,
                                                      const double *__restrict__ u1, const double *__restrict__ u2,
                                                      double *__restrict__ n1, double *__restrict__ n2, Epi<T> E) {
    double o1[1], o2[1];
    mx_vec_sums<T, 1>(X, part1, N, part2, blockIdx.x, o1, o2);
    if (threadIdx.x >= 64) return;
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int d = X.state[x];
    if (d < 0) {   // a position without a state: its column is zero in every stage
        n1[x] = n2[x] = 0.0;
        return;
    }
    if (!mx_finite(o1[0], o2[0])) mx_own_sums<T>(A, X, d, u1, u2, 1, 0, o1[0], o2[0]);
    apply_epi(E, 0, d, X.S, static_cast<T>(K * (u2[x] * o1[0] - u1[x] * o2[0])));
    const T y = E.mode == EPI_RK4 ? E.f_out[d] : E.u_out[d];
    n1[x] = static_cast<double>(y);
    n2[x] = static_cast<double>(T(1) - y);
}

// 1 / tau_d = K (o1 + o2) with u1 = f0, u2 = 1 - f0
__global__ __launch_bounds__(64 * kMxParts) void k_mx_tau_finish(TiledArgs<double> A, MxArgs<double> X,
                                                                 const double *__restrict__ part1, MxRuns N,
                                                                 const double *__restrict__ part2, double K,
                                                                 const double *__restrict__ u1,
                                                                 const double *__restrict__ u2,
                                                                 double *__restrict__ tau_inv) {
    double o1[1], o2[1];
    mx_vec_sums<double, 1>(X, part1, N, part2, blockIdx.x, o1, o2);
    if (threadIdx.x >= 64) return;
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int d = X.state[x];
    if (d < 0) return;
    if (!mx_finite(o1[0], o2[0])) mx_own_sums<double>(A, X, d, u1, u2, 1, 0, o1[0], o2[0]);
    tau_inv[d] = K * (o1[0] + o2[0]);
}

// Block row and share of this workgroup: workgroups go round-robin to the 8 XCDs;
// each XCD takes a contiguous range of rows, share after share of a row, so that
// the columns its rows read (those of one component, or a few) stay in its L2.
// False for the workgroups that pad the grid to 8 ranges.
__device__ __forceinline__ bool mx_row_of_block(int nb, int nsplit, int &I, int &sp) {
    const int per = (nb + 7) >> 3;
    const int w = static_cast<int>(blockIdx.x) >> 3;
    I = (static_cast<int>(blockIdx.x) & 7) * per + w / nsplit;
    sp = w % nsplit;
    return w / nsplit < per && I < nb;
}

// D += A B on one 16 x 16 tile, A 16 x 4 and B 4 x 16 over the wave: lane
// (j, g) = (lane % 16, lane / 16) gives A[j][g] and B[g][j] and holds
// D[4 v + g][j] in d[v].
#ifdef __HIP__
typedef double mx_d4 __attribute__((vector_size(32)));
__device__ __forceinline__ void mx_mfma(double a, double b, double (&d)[4]) {
    mx_d4 c = {d[0], d[1], d[2], d[3]};
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    d[0] = c[0];
    d[1] = c[1];
    d[2] = c[2];
    d[3] = c[3];
}
#else   // a build without the matrix instruction: the same product by lane exchange
inline void mx_mfma(double a, double b, double (&d)[4]) {
    const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
    for (int k = 0; k < 4; ++k) {
        const double bk = __shfl(b, 16 * k + j, 64);
        for (int v = 0; v < 4; ++v) d[v] = fma(__shfl(a, 16 * k + 4 * v + g, 64), bk, d[v]);
    }
}
#endif

// The matrix and its transpose applied to 16 NCT columns on the FP64 matrix
// cores: workgroup = block row I and a share of its blocks; waves 0 - 3 take M u1
// and waves 4 - 7 the transposed product with u2, 16 rows each.  Per block the 64
// rows of u1 and u2 ([position][ld], columns from c0) are staged in LDS (rows
// padded by 4 values: the four k groups of a wave's read fall on different
// banks); a wave reads its rows of block (I, J) or its columns of block (J, I) as
// whole sub-block runs, once, a block ahead, so the matrix passes through
// registers only.  The k index of the instruction's step t stands for partner
// 4 g + t of a sub-block.  The sums of a share go to part1 and part2
// ([split][position][ld]).  Bound by the matrix cores at 64 columns (17 GF on the
// 100^3 system, 72 TF measured for a large product) and by the matrix bytes
// below 32.
template <typename T, int NCT>
__global__ __launch_bounds__(512, 4) void k_mx_gemm(MxArgs<T> X, const double *__restrict__ u1,
                                                    const double *__restrict__ u2, int ld, int c0, int nsplit,
                                                    double *__restrict__ part1, double *__restrict__ part2) {
    constexpr int NC = 16 * NCT, LD = NC + 4;
    extern __shared__ __align__(16) unsigned char smem[];
    double *s1 = reinterpret_cast<double *>(smem), *s2 = s1 + 64 * LD;
    int I, sp;
    if (!mx_row_of_block(X.nb, nsplit, I, sp)) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int R = wave & 3;
    const bool tr = wave >= 4;
    const int j = lane & 15, g = lane >> 4;
    const int r0 = X.row[I], n = X.row[I + 1] - r0;
    const int xb = r0 + static_cast<int>(static_cast<int64_t>(n) * sp / nsplit);
    const int xe = r0 + static_cast<int>(static_cast<int64_t>(n) * (sp + 1) / nsplit);
    double acc[NCT][4];
#pragma unroll
    for (int c = 0; c < NCT; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[c][v] = 0.0;
    auto sweep = [&](auto trc) {
        constexpr bool TR = decltype(trc)::value;
        const double *__restrict__ su = (TR ? s2 : s1) + 4 * g * LD + j;
        T w[4][4];
        auto load = [&](int x, int C) {
            if constexpr (TR) {
                const T *__restrict__ m = X.m + static_cast<int64_t>(X.col[x].id_t) * kMxBlock + R * 256 + g * 64 + j;
#pragma unroll
                for (int t = 0; t < 4; ++t) w[C][t] = m[C * 1024 + t * 16];
            } else {
                const T *__restrict__ m = X.m + static_cast<int64_t>(x) * kMxBlock + R * 1024 + j * 16 + 4 * g;
                const Vec4<T> v = *reinterpret_cast<const Vec4<T> *>(m + C * 256);
                w[C][0] = v.x;
                w[C][1] = v.y;
                w[C][2] = v.z;
                w[C][3] = v.w;
            }
        };
        // the next block's rows of u1 and u2 are in registers while this block is
        // multiplied: a barrier waits for every load in flight, so a load issued
        // between two barriers would be waited for there
        double n1[2 * NCT], n2[2 * NCT];
        auto stage = [&](int x) {
            const int64_t u0 = static_cast<int64_t>(X.col[x].j) * 64 * ld + c0;
#pragma unroll
            for (int e = 0; e < NCT; ++e) {
                const int idx = e * 512 + static_cast<int>(threadIdx.x);
                const int r = idx / (NC / 2), k = idx - r * (NC / 2);
                const int64_t o = u0 + static_cast<int64_t>(r) * ld + 2 * k;
                n1[2 * e] = u1[o];
                n1[2 * e + 1] = u1[o + 1];
                n2[2 * e] = u2[o];
                n2[2 * e + 1] = u2[o + 1];
            }
        };
        if (xb >= xe) return;
        stage(xb);
#pragma unroll
        for (int C = 0; C < 4; ++C) load(xb, C);
        for (int x = xb; x < xe; ++x) {
            const int xn = min(x + 1, xe - 1);
            __syncthreads();
#pragma unroll
            for (int e = 0; e < NCT; ++e) {
                const int idx = e * 512 + static_cast<int>(threadIdx.x);
                const int r = idx / (NC / 2), k = idx - r * (NC / 2);
                s1[r * LD + 2 * k] = n1[2 * e];
                s1[r * LD + 2 * k + 1] = n1[2 * e + 1];
                s2[r * LD + 2 * k] = n2[2 * e];
                s2[r * LD + 2 * k + 1] = n2[2 * e + 1];
            }
            __syncthreads();
            stage(xn);
#pragma unroll
            for (int C = 0; C < 4; ++C) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const double wt = static_cast<double>(w[C][t]);
#pragma unroll
                    for (int c = 0; c < NCT; ++c) mx_mfma(wt, su[(C * 16 + t) * LD + 16 * c], acc[c]);
                }
                load(xn, C);
            }
        }
    };
    if (tr) sweep(std::integral_constant<bool, true>{});
    else sweep(std::integral_constant<bool, false>{});
    double *__restrict__ po = (tr ? part2 : part1) +
                              ((static_cast<int64_t>(sp) * X.nb + I) * 64 + R * 16) * ld + c0 + j;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < NCT; ++c) po[static_cast<int64_t>(4 * v + g) * ld + 16 * c] = acc[c][v];
}

// u1 = f and u2 = 1 - f of nb vectors by position, NC columns (0 past the last
// vector and state): workgroup = 64 positions x 16 columns, turned in LDS
template <typename T>
__global__ __launch_bounds__(256) void k_mx_load_batch(MxArgs<T> X, const T *__restrict__ f, int64_t ldf, int nvec,
                                                       int NC, double *__restrict__ u1, double *__restrict__ u2) {
    __shared__ T s_f[16][65];
    const int x0 = blockIdx.x * 64, c0 = blockIdx.y * 16;
    const int r = threadIdx.x & 63;
    const int d = X.state[x0 + r];
    for (int c = threadIdx.x >> 6; c < 16; c += 4)
        s_f[c][r] = d >= 0 && c0 + c < nvec ? f[static_cast<int64_t>(c0 + c) * ldf + d] : T(0);
    __syncthreads();
    const int c = threadIdx.x & 15;
    for (int q = threadIdx.x >> 4; q < 64; q += 16) {
        const bool in = X.state[x0 + q] >= 0 && c0 + c < nvec;
        const T v = s_f[c][q];
        const int64_t o = static_cast<int64_t>(x0 + q) * NC + c0 + c;
        u1[o] = static_cast<double>(v);
        u2[o] = in ? static_cast<double>(T(1) - v) : 0.0;
    }
}

// I = K [(1 - f) o1 - f o2] per state and vector b0 + column, then the epilogue;
// workgroup = 64 positions x 16 columns
template <typename T>
__global__ __launch_bounds__(1024) void k_mx_batch_finish(TiledArgs<T> A, MxArgs<T> X,
                                                         const double *__restrict__ part1,
                                                         const double *__restrict__ part2, int nsplit, int NC, int b0,
                                                         int nvec, double K, const double *__restrict__ u1,
                                                         const double *__restrict__ u2, const T *__restrict__ f,
                                                         int64_t ldf, Epi<T> E) {
    __shared__ double s_o[2][16][65];
    const int x0 = blockIdx.x * 64, c0 = blockIdx.y * 16;
    const int64_t np = static_cast<int64_t>(X.nb) * 64 * NC;
    {
        const int c = threadIdx.x & 15, q = threadIdx.x >> 4;
        const int64_t o = static_cast<int64_t>(x0 + q) * NC + c0 + c;
        double o1 = 0.0, o2 = 0.0;
        for (int sp = 0; sp < nsplit; ++sp) {
            o1 += part1[sp * np + o];
            o2 += part2[sp * np + o];
        }
        s_o[0][c][q] = o1;
        s_o[1][c][q] = o2;
    }
    __syncthreads();
    const int q = threadIdx.x & 63, c = threadIdx.x >> 6;
    const int d = X.state[x0 + q];
    if (d < 0 || c0 + c >= nvec) return;
    double o1 = s_o[0][c][q], o2 = s_o[1][c][q];
    if (!mx_finite(o1, o2)) mx_own_sums<T>(A, X, d, u1, u2, NC, c0 + c, o1, o2);
    const int b = b0 + c0 + c;
    const T fd = f[static_cast<int64_t>(b) * ldf + d];
    apply_epi(E, b, d, X.S, static_cast<T>(K * (static_cast<double>(T(1) - fd) * o1 - static_cast<double>(fd) * o2)));
}

// ---- reverse, several vectors, over the pair matrix ----------------------------
// With o1 = M x and o2 = M^T x per column,
//   dL/df_d = K [ o1(lam f) + o2(lam (1 - f)) - lam_d (o1(f) + o2(1 - f)) ]
// is one product of the matrix with 2 V columns (u1 = [f, lam f], u2 = [1 - f,
// lam (1 - f)], V the vectors rounded up to 16), and the gradient of a channel
// (d, p) sums over the vectors before its Gaussians enter,
//   dL/d|g|^2 = K [ bh G[d][p] + ah G[p][d] ],
//   G[d][p] = sum_b (lam_d - lam_p) (1 - f_d) f_p,
// formed from lam_d - lam_p itself in the plan's type (k_mx_outer): the difference of two products, which the matrix cores could take, loses the digits
// that lam_d and lam_p share (FP64, 64 vectors, lam a smooth function of the energy:
// error of dL/d|g|^2 1.1e-15 of its norm, 2.4e-16 from the differences).

// Only differences of lam enter, but dL/df takes them as differences of sums, which
// lose the digits that a vector's lam share.  Where a vector has such an offset (the
// middle three of five of its values lie closer to each other than to 0) it is taken
// off first: a constant lam gives 0 exactly (energy or particle number as a loss), an
// offset costs no digits, and a few values far from the others do not matter.
__device__ __forceinline__ void order2(double &a, double &b) {
    const double lo = fmin(a, b), hi = fmax(a, b);
    a = lo;
    b = hi;
}
template <typename T>
__device__ __forceinline__ double lam_offset(const T *__restrict__ lam, int S) {
    double v[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) v[k] = static_cast<double>(lam[static_cast<int64_t>(S - 1) * k / 4]);
#pragma unroll
    for (int k = 4; k >= 1; --k)
#pragma unroll
        for (int m = 0; m < k; ++m) order2(v[m], v[m + 1]);
    return v[3] - v[1] < fabs(v[2]) && fabs(v[2]) < 1.7e308 ? v[2] : 0.0;
}

// u1 and u2 of nvec vectors by position, 2 V columns; with fl also f and lam
// themselves (for k_mx_outer: f, lam [position][V], f, lam [block][V][64])
template <typename T>
__global__ __launch_bounds__(256) void k_mx_load_vjp(MxArgs<T> X, const T *__restrict__ f, int64_t ldf,
                                                     const T *__restrict__ lam, int64_t ldl, int nvec, int V,
                                                     double *__restrict__ u1, double *__restrict__ u2,
                                                     T *__restrict__ fl) {
    __shared__ T s_f[16][65], s_l[16][65];
    const int x0 = blockIdx.x * 64, c0 = blockIdx.y * 16;
    {
        const int r = threadIdx.x & 63;
        const int d = X.state[x0 + r];
        for (int c = threadIdx.x >> 6; c < 16; c += 4) {
            const bool in = d >= 0 && c0 + c < nvec;
            s_f[c][r] = in ? f[static_cast<int64_t>(c0 + c) * ldf + d] : T(0);
            s_l[c][r] = in ? lam[static_cast<int64_t>(c0 + c) * ldl + d] : T(0);
        }
    }
    __syncthreads();
    const int c = threadIdx.x & 15;
    const double off = c0 + c < nvec ? lam_offset(lam + static_cast<int64_t>(c0 + c) * ldl, X.S) : 0.0;
    for (int q = threadIdx.x >> 4; q < 64; q += 16) {
        const bool in = X.state[x0 + q] >= 0 && c0 + c < nvec;
        const double v = static_cast<double>(s_f[c][q]), l = in ? static_cast<double>(s_l[c][q]) - off : 0.0;
        const double w = in ? 1.0 - v : 0.0;
        const int64_t o = static_cast<int64_t>(x0 + q) * 2 * V + c0 + c;
        u1[o] = v;
        u1[o + V] = l * v;
        u2[o] = w;
        u2[o + V] = l * w;
        if (fl) {
            const int64_t y = static_cast<int64_t>(x0 + q) * V + c0 + c;
            fl[y] = s_f[c][q];
            fl[static_cast<int64_t>(X.nb) * 64 * V + y] = s_l[c][q];
        }
    }
    if (!fl) return;
    T *__restrict__ ft = fl + 2 * static_cast<int64_t>(X.nb) * 64 * V;
    const int r = threadIdx.x & 63;
    for (int k = threadIdx.x >> 6; k < 16; k += 4) {
        const int64_t y = (static_cast<int64_t>(blockIdx.x) * V + c0 + k) * 64 + r;
        ft[y] = s_f[k][r];
        ft[static_cast<int64_t>(X.nb) * 64 * V + y] = s_l[k][r];
    }
}

// dL/df per state and vector; workgroup = 64 positions x 16 vectors
template <typename T>
__global__ __launch_bounds__(1024) void k_mx_vjp_finish(TiledArgs<T> A, MxArgs<T> X, const double *__restrict__ part1,
                                                        const double *__restrict__ part2, int nsplit, int V, int nvec,
                                                        double K, const double *__restrict__ u1,
                                                        const double *__restrict__ u2, const T *__restrict__ lam,
                                                        int64_t ldl, T *__restrict__ gf, int64_t ldgf) {
    __shared__ double s_o[4][16][65];
    const int x0 = blockIdx.x * 64, c0 = blockIdx.y * 16;
    const int64_t np = static_cast<int64_t>(X.nb) * 64 * 2 * V;
    {
        const int c = threadIdx.x & 15, q = threadIdx.x >> 4;
        const int64_t o = static_cast<int64_t>(x0 + q) * 2 * V + c0 + c;
        double a[4] = {0.0, 0.0, 0.0, 0.0};
        for (int sp = 0; sp < nsplit; ++sp) {
            a[0] += part1[sp * np + o];
            a[1] += part2[sp * np + o];
            a[2] += part1[sp * np + o + V];
            a[3] += part2[sp * np + o + V];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) s_o[k][c][q] = a[k];
    }
    __syncthreads();
    const int q = threadIdx.x & 63, c = threadIdx.x >> 6;
    const int d = X.state[x0 + q];
    if (d < 0 || c0 + c >= nvec) return;
    double a[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = s_o[k][c][q];
    if (!mx_finite(a[0], a[1]) || !mx_finite(a[2], a[3])) {
        mx_own_sums<T>(A, X, d, u1, u2, 2 * V, c0 + c, a[0], a[1]);
        mx_own_sums<T>(A, X, d, u1, u2, 2 * V, V + c0 + c, a[2], a[3]);
    }
    const T *__restrict__ lv = lam + static_cast<int64_t>(c0 + c) * ldl;
    const double l = static_cast<double>(lv[d]) - lam_offset(lv, X.S);
    gf[static_cast<int64_t>(c0 + c) * ldgf + d] = static_cast<T>(K * (a[2] + a[3] - l * (a[0] + a[1])));
}

// G over the stored blocks ([blocks][64 x 64], the matrix's layout) in the plan's
// type, as H[d][p] = -G[p][d] = sum_b (lam_d - lam_p) f_d (1 - f_p), added to what gm
// holds when add != 0.  With the operations of k_vjp_batched<float>: the vectors' terms
// (1 - f_p) (f_d (lam_d - lam_p)) are summed as a balanced tree over 64 vectors in order,
// whose first level is a fused multiply-add (FP64: trees over 16, then in order).  (The
// other term of a pair, f_p (1 - f_d) (lam_d - lam_p), is minus the first with d and p
// exchanged, digit for digit.)  Not on the matrix cores: as sum_b f_d lam_d (1 - f_p)
// - ... the difference would lose the digits that lam_d and lam_p share (2-norm error of
// dL/d|g|^2 for slowly varying lam, 64 vectors: 1.1e-15 against 2.4e-16 here).  Lane =
// column p, wave = 16 rows d whose values are scalar operands; 16 vectors of a column
// are in registers at a time, and the loop over such groups stays a loop: unrolled, the
// loads of all groups are issued first, and one wave a SIMD is left (62^3, 64 vectors,
// FP64, whole reverse pass: 712 us, 327 now).  About three and a half operations per
// pair and vector on the vector units, which bound it, against a 64-lane sum per pair
// over entries (1149 us).
template <typename T, int VT>
__global__ __launch_bounds__(256) void k_mx_outer(MxArgs<T> X, const T *__restrict__ fl, T *__restrict__ gm, int add,
                                                  int nsplit) {
    constexpr int V = 16 * VT;
    auto fma1 = [](T a, T b, T c) {
        if constexpr (sizeof(T) == 4) return __builtin_fmaf(a, b, c);
        else return __builtin_fma(a, b, c);
    };
    int I, sp;
    if (!mx_row_of_block(X.nb, nsplit, I, sp)) return;
    const int lane = threadIdx.x & 63;
    const int R = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int r0 = X.row[I], n = X.row[I + 1] - r0;
    const int xb = r0 + static_cast<int>(static_cast<int64_t>(n) * sp / nsplit);
    const int xe = r0 + static_cast<int>(static_cast<int64_t>(n) * (sp + 1) / nsplit);
    const int64_t np = static_cast<int64_t>(X.nb) * 64 * V;
    const T *__restrict__ ll = fl + np, *__restrict__ ft = fl + 2 * np, *__restrict__ lt = fl + 3 * np;
    const int64_t row0 = (static_cast<int64_t>(I) * 64 + R * 16) * V;
    for (int x = xb; x < xe; ++x) {
        const int64_t col = static_cast<int64_t>(X.col[x].j) * 64 * V + lane;
        T res[16], odd[16];
#pragma unroll 1
        for (int q = 0; q < VT; ++q) {
            T wc[16], lc[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                wc[k] = T(1) - ft[col + (16 * q + k) * 64];
                lc[k] = lt[col + (16 * q + k) * 64];
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const T *__restrict__ fr = fl + row0 + r * V + 16 * q, *__restrict__ lr = ll + row0 + r * V + 16 * q;
                T a[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const T m0 = fr[2 * k] * (lr[2 * k] - lc[2 * k]);
                    const T m1 = fr[2 * k + 1] * (lr[2 * k + 1] - lc[2 * k + 1]);
                    a[k] = fma1(wc[2 * k + 1], m1, wc[2 * k] * m0);
                }
                const T t = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
                if (sizeof(T) == 8 || q < 2) res[r] = q == 0 ? t : res[r] + t;
                else odd[r] = q == 2 ? t : odd[r] + t;
            }
        }
        T *__restrict__ po = gm + static_cast<int64_t>(x) * kMxBlock + (R * 4 + (lane >> 4)) * 256 + (lane & 15);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const T t = VT > 2 && sizeof(T) == 4 ? res[r] + odd[r] : res[r];
            po[r * 16] = add ? po[r * 16] + t : t;
        }
    }
}

// dL/d|g|^2 of every channel from G, over the pair records in the forward pass's
// tiles: the record word, its first channel and two values of G per pair, no
// |g|^2 stream.  Each channel is written once (gg2_mode as in k_vjp_pairs).
template <typename T, bool PADQ, int NM, bool TAB, bool QORD>
__device__ __forceinline__ void mx_gg2_chunk(const TiledArgs<T> &A, const MxArgs<T> &X, const T *__restrict__ gm,
                                             const T *s_e, const uint32_t *s_kq, const int32_t *s_pos,
                                             const double *s_tab, int64_t c, int64_t beg,
                                             int len, int first, int step,
                                             const int32_t *__restrict__ chan, const int32_t *__restrict__ chan0,
                                             double *__restrict__ gg2, int gg2_mode) {
    const int lane = threadIdx.x & 63;
    const int nm = A.nm;
    const int dc = QORD ? 0 : A.chunk_dest[c];
    const uint32_t *__restrict__ pb = A.pnu + beg;
    const int32_t *__restrict__ cb = chan + beg;
    const int32_t *__restrict__ cb0 = chan0 + beg;
    uint32_t pn = pb[first + lane];
    int32_t h = cb0[first + lane];
    for (int r = first; r < len; r += step) {
        const bool v = r + lane < len;
        T ed, ep;
        uint32_t kd, kp;
        int xd, xp;
        if (QORD) {
            const int wd = v ? static_cast<int>(pn & 0xffffu) : 0;
            const int wp = v ? static_cast<int>(pn >> 16) : 0;
            ed = s_e[wd];
            ep = s_e[wp];
            kd = s_kq[wd];
            kp = s_kq[wp];
            xd = s_pos[wd];
            xp = s_pos[wp];
        } else {
            const int p = v ? static_cast<int>(pn) : dc;
            const StateRec<T> sd = A.st[dc], sp = A.st[p];
            ed = sd.eps;
            ep = sp.eps;
            kd = PADQ ? sd.kqp : sd.kq;
            kp = PADQ ? sp.kqp : sp.kq;
            xd = X.pos[dc];
            xp = X.pos[p];
        }
        const int bd = xd >> 6, bp = xp >> 6;
        // a masked lane may name a block that is not stored
        const int64_t id = max(X.blk[bd * X.nb + bp], 0), it = max(X.blk[bp * X.nb + bd], 0);
        const T g1 = gm[id * kMxBlock + mx_inner(xd & 63, xp & 63)];
        const T g2 = gm[it * kMxBlock + mx_inner(xp & 63, xd & 63)];
        const int q = PADQ ? static_cast<int>(kp - kd) + A.qoff : q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
        const Pair2<T> *__restrict__ wq = A.hwN + static_cast<int64_t>(q) * A.tq;
        Pair2<T> w[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) w[m] = wq[min(m, nm - 1) * A.tm];
        const int32_t c0 = h;
        __builtin_amdgcn_sched_barrier(0);
        pn = pb[r + step + lane];
        h = cb0[r + step + lane];
        __builtin_amdgcn_sched_barrier(0);
        const T x = ed - ep;
        double gv[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const T xa = x + w[m].a, xe = x - w[m].a;
            const T da = pair_gauss<T, TAB>(A, xa * xa, s_tab);
            const T dem = pair_gauss<T, TAB>(A, xe * xe, s_tab);
            if constexpr (sizeof(T) == 4) {
                // as k_vjp_batched<float> rounds it
                const float sm = da + dem;
                const float bh = __builtin_fmaf(w[m].b, sm, da), ah = __builtin_fmaf(w[m].b, sm, dem);
                gv[m] = static_cast<double>(A.K * __builtin_fmaf(bh, -g2, -(g1 * ah)));
            } else {
                const T t = w[m].b * (da + dem);
                gv[m] = -A.K * (g2 * (t + da) + g1 * (t + dem));
            }
        }
        if (v) write_gg2<NM>(gg2, gg2_mode, c0, cb + r + lane, A.pld, nm, gv);
    }
}

template <typename T, bool PADQ, int NM, bool TAB>
__global__ __launch_bounds__(1024) void k_mx_gg2(TiledArgs<T> A, MxArgs<T> X, const T *__restrict__ gm,
                                                 const int32_t *__restrict__ chan, const int32_t *__restrict__ chan0,
                                                 double *__restrict__ gg2, int gg2_mode) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    // LDS as in k_pair_matrix
    double *s_tab = reinterpret_cast<double *>(smem);
    T *s_e = reinterpret_cast<T *>(s_tab + (sizeof(T) == 8 ? kExpTab : 0));
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_e + A.lds_states);
    int32_t *s_pos = reinterpret_cast<int32_t *>(s_kq + A.lds_states);
    const int n = t.lds == 2 ? t.p_hi - t.p_lo + 1 : 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const StateRec<T> sr = A.st[t.p_lo + i];
        s_e[i] = sr.eps;
        s_kq[i] = PADQ ? sr.kqp : sr.kq;
        s_pos[i] = X.pos[t.p_lo + i];
    }
    if constexpr (sizeof(T) == 8 && TAB)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    if (t.lds == 2) {
        const int64_t beg = A.chunk_beg[t.c0];
        mx_gg2_chunk<T, PADQ, NM, TAB, true>(A, X, gm, s_e, s_kq, s_pos, s_tab, t.c0, beg,
                                             static_cast<int>(A.chunk_end[t.c1 - 1] - beg), wave * 64, nw * 64, chan,
                                             chan0, gg2, gg2_mode);
        return;
    }
    for (int64_t c = t.c0 + wave; c < t.c1; c += nw)
        mx_gg2_chunk<T, PADQ, NM, TAB, false>(A, X, gm, s_e, s_kq, s_pos, s_tab, c, A.chunk_beg[c],
                                              static_cast<int>(A.chunk_end[c] - A.chunk_beg[c]), 0, 64, chan, chan0,
                                              gg2, gg2_mode);
}

// x by position, three components each
__global__ void k_mx_load3(MxArgs<double> X, const Vec4<double> *__restrict__ x, double *__restrict__ u) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= X.nb * 64) return;
    const int d = X.state[i];
    Vec4<double> v;
    v.x = v.y = v.z = 0.0;
    if (d >= 0) v = x[d];
    u[3 * i] = v.x;
    u[3 * i + 1] = v.y;
    u[3 * i + 2] = v.z;
}

// x_new_d = tau_d (rhs_d + K [(1 - f0_d) o1 + f0_d o2]); u holds x by position
// and the next iterate goes to un.
__global__ __launch_bounds__(64 * kMxParts) void k_mx_tr_finish(TiledArgs<double> A, MxArgs<double> X,
                                                                const double *__restrict__ part1, MxRuns N,
                                                                const double *__restrict__ part2, double K,
                                                                const double *__restrict__ f0,
                                                                const Vec4<double> *__restrict__ rhs,
                                                                const double *__restrict__ tau,
                                                                const double *__restrict__ u, double *__restrict__ un,
                                                                Vec4<double> *__restrict__ x_new) {
    double o1[3], o2[3];
    mx_vec_sums<double, 3>(X, part1, N, part2, blockIdx.x, o1, o2);
    if (threadIdx.x >= 64) return;
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int d = X.state[x];
    if (d < 0) {   // a position without a state: its column is zero in every iteration
        un[3 * x] = un[3 * x + 1] = un[3 * x + 2] = 0.0;
        return;
    }
    const double f = f0[d], t = tau[d];
    const Vec4<double> r = rhs[d];
    const double rr[3] = {r.x, r.y, r.z};
    double y[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (!mx_finite(o1[k], o2[k])) mx_own_sums<double>(A, X, d, u, u, 3, k, o1[k], o2[k]);
        y[k] = t * (rr[k] + K * ((1.0 - f) * o1[k] + f * o2[k]));
        un[3 * x + k] = y[k];
    }
    Vec4<double> o;
    o.x = y[0];
    o.y = y[1];
    o.z = y[2];
    o.w = 0.0;
    x_new[d] = o;
}

// ---- forward, batched (B vectors in one pass) -----------------------------
// Workgroup = batch tile: up to DPW destinations per wave, consecutive
// destinations sharing a partner window.  The window is walked in sub-tiles
// of PT partners; for each, f[p][0:64] (64 vectors, transposed, padded) and
// the partners' {eps, k} are staged in LDS.  For each of its destinations a
// wave then computes the coefficients of the entries whose partner lies in
// the sub-tile (lane = entry), merges entries with the same partner by a
// segmented shuffle reduction, and applies every merged coefficient pair to
// the 64 vectors (lane = vector):
//   acc_a[b] += a_p (1 - f_{p,b}),  acc_b[b] += b_p f_{p,b}.
// Each entry's coefficients are evaluated once per pass, not once per vector.
struct BTileRec {
    int32_t d0, d1;        // destinations [d0, d1)
    int32_t p_lo, n_sub;   // window start and number of sub-tiles
    int64_t off_base;      // sub_off index of destination d0
};

template <typename T> struct BArgs {
    const uint32_t *__restrict__ pnu;
    const T *__restrict__ g2;
    const StateRec<T> *__restrict__ st;
    const Pair2<T> *__restrict__ hwN;
    int64_t tq, tm;                          // as in TiledArgs
    const BTileRec *__restrict__ btiles;
    const int64_t *__restrict__ sub_off;   // per destination: n_sub + 1 entry offsets
    int S, nm, nq0, nq1, nq2, pt;
    int padq, qoff;                          // as in TiledArgs
    T mc, K;
    int64_t n_btiles;
    int xcd;                                 // as in TiledArgs
};

// Sub-tile entry offsets of the batch tiles: one workgroup per tile, one
// thread per (destination, slot); slot k is the first entry of the
// destination whose partner is >= p_lo + k pt (a lower bound on the sorted
// partner << 3 | mode keys; the row end if there is none).  A destination's
// entries are [chunk_beg[dest_chunk[x]], chunk_beg[dest_chunk[x + 1]]).
__global__ void k_sub_offsets(const BTileRec *__restrict__ tiles, const uint32_t *__restrict__ pnu,
                              const int64_t *__restrict__ chunk_beg,
                              const int32_t *__restrict__ dest_chunk, int S, int pt,
                              int64_t *__restrict__ sub_off) {
    const BTileRec t = tiles[blockIdx.x];
    const int per = t.n_sub + 1;
    const int n = (t.d1 - t.d0) * per;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int x = t.d0 + i / per;
        const int k = i % per;
        int64_t lo = chunk_beg[dest_chunk[x]], hi = chunk_beg[dest_chunk[x + 1]];
        const int64_t p = static_cast<int64_t>(t.p_lo) + static_cast<int64_t>(k) * pt;
        const uint32_t key = p >= S ? UINT32_MAX : static_cast<uint32_t>(p) << 3;
        while (lo < hi) {
            const int64_t mid = lo + (hi - lo) / 2;
            if (pnu[mid] < key) lo = mid + 1;
            else hi = mid;
        }
        sub_off[t.off_base + i] = lo;
    }
}

// Entries of one (destination, partner) pair: one per mode, at most 8 modes,
// no duplicates (both checked at plan build).
constexpr int kMaxRun = 8;

template <typename T> __device__ __forceinline__ T lane_bcast(T v, int src);
template <> __device__ __forceinline__ double lane_bcast(double v, int src) {
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(bits & 0xffffffffLL), src);
    const int hi = __builtin_amdgcn_readlane(static_cast<int>(bits >> 32), src);
    return __longlong_as_double((static_cast<long long>(hi) << 32) |
                                (static_cast<long long>(lo) & 0xffffffffLL));
}
template <> __device__ __forceinline__ float lane_bcast(float v, int src) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}

// Fourth word of a raw buffer resource on gfx9-family parts (32-bit data
// format; no swizzle, no index stride)
constexpr int kBufferDword3 = 0x00020000;

template <typename T> __device__ __forceinline__ T buffer_load_value(__amdgpu_buffer_rsrc_t r, int voff, int soff);
template <> __device__ __forceinline__ double buffer_load_value(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <> __device__ __forceinline__ float buffer_load_value(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// RUN = 0: one phonon table for all vectors.  RUN > 0: a bath per vector
// (RUN bounds the entries of one pair, the mode count rounded up): N comes
// from nvec, [row][mode][64] for the launch's 64 vectors (nvec_ld values; row
// = the q index of the shared table), and an entry's coefficients split into
// the part without
// N, summed over the pair's modes as before, and |g|^2 (G(x + hw) +
// G(x - hw)), applied per vector with that vector's N.
template <typename T, int DPW, int RUN>
__global__ __launch_bounds__(512) void k_fwd_batched(BArgs<T> A, const T *__restrict__ f,
                                                     int64_t ldf, int B, Epi<T> E,
                                                     const T *__restrict__ nvec, int64_t nvec_ld) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int PT = A.pt;
    T *s_F = reinterpret_cast<T *>(smem);                                   // [PT][65]
    StateRec<T> *s_ek = reinterpret_cast<StateRec<T> *>(s_F + PT * 65);    // [PT]
    const int64_t ti = tile_of_block(A.n_btiles, A.xcd);
    if (ti < 0) return;
    const BTileRec t = A.btiles[ti];
    const int b0 = blockIdx.y * 64;
    const int nb = min(64, B - b0);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    const int nd = t.d1 - t.d0;
    T acc_a[DPW], acc_b[DPW];
#pragma unroll
    for (int j = 0; j < DPW; ++j) {
        acc_a[j] = T(0);
        acc_b[j] = T(0);
    }
    for (int k = 0; k < t.n_sub; ++k) {
        const int pa = t.p_lo + k * PT;
        const int pc = min(PT, A.S - pa);
        __syncthreads();
        for (int i = threadIdx.x; i < pc * nb; i += blockDim.x) {
            const int bb = i / pc, pl = i - bb * pc;
            s_F[pl * 65 + bb] = f[static_cast<int64_t>(b0 + bb) * ldf + pa + pl];
        }
        for (int i = threadIdx.x; i < pc; i += blockDim.x) s_ek[i] = A.st[pa + i];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < DPW; ++j) {
            const int dl = wave + j * nw;
            if (dl < nd) {
                const int d = t.d0 + dl;
                const int64_t *so = A.sub_off + t.off_base + static_cast<int64_t>(dl) * (t.n_sub + 1);
                const int64_t e_lo = so[k], e_hi = so[k + 1];
                const StateRec<T> sd = A.st[d];
                // the sub-tile's terms are summed on their own, then added to
                // the running sums (two levels: each sum has at most PT terms
                // plus one per sub-tile, instead of one per partner)
                T sa = T(0), sb = T(0);
                for (int64_t e0 = e_lo; e0 < e_hi; e0 += 64) {
                    const int64_t e = e0 + lane;
                    const bool valid = e < e_hi;
                    int pl = -1 - lane;     // distinct for invalid lanes: never merged
                    T ca = T(0), cb = T(0), c1 = T(0);
                    int ti = 0;
                    if (valid) {
                        const uint32_t pn = A.pnu[e];
                        const T g = A.g2[e];
                        pl = static_cast<int>(pn >> 3) - pa;
                        const StateRec<T> sp = s_ek[pl];
                        const int q = A.padq ? static_cast<int>(sp.kqp - sd.kqp) + A.qoff
                                             : q_linear(sd.kq, sp.kq, A.nq0, A.nq1, A.nq2);
                        const Pair2<T> wn = A.hwN[static_cast<int64_t>(q) * A.tq + static_cast<int64_t>(pn & 7u) * A.tm];
                        const T de = sd.eps - sp.eps;
                        const T xa = de + wn.a, xe = de - wn.a;
                        const T da = gauss_exp(xa * xa * A.mc);
                        const T dem = gauss_exp(xe * xe * A.mc);
                        if constexpr (RUN > 0) {
                            ca = g * dem;
                            cb = g * da;
                            c1 = g * (da + dem);
                            ti = q * A.nm + static_cast<int>(pn & 7u);
                        } else {
                            const T tt = wn.b * (da + dem);
                            ca = g * (tt + dem);
                            cb = g * (tt + da);
                        }
                    }
                    // sum each run of equal partners into its first lane (a run is
                    // one pair over its modes, at most kMaxRun lanes)
#pragma unroll
                    for (int off = 1; off < kMaxRun; off <<= 1) {
                        const T oa = __shfl_down(ca, off, 64);
                        const T ob = __shfl_down(cb, off, 64);
                        const int op = __shfl_down(pl, off, 64);
                        if (lane + off < 64 && op == pl) {
                            ca += oa;
                            cb += ob;
                        }
                    }
                    const int prev = __shfl_up(pl, 1, 64);
                    const bool head = valid && (lane == 0 || prev != pl);
                    unsigned long long m = __ballot(head);
                    if constexpr (RUN > 0) {
                        // the run of a head ends at the next head or at the
                        // last valid lane; each of its entries adds
                        // c1 N_b(q, mode) for this lane's vector b
                        const int nvalid = static_cast<int>(min<int64_t>(64, e_hi - e0));
                        // buffer loads: the row offset is a scalar operand and
                        // the lane offset a fixed register, so a load needs no
                        // address registers (whose reuse would make the wave
                        // wait for loads in flight); reads past the table
                        // return 0
                        const __amdgpu_buffer_rsrc_t nvr = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<T *>(nvec), 0, static_cast<int>(nvec_ld * sizeof(T)), kBufferDword3);
                        const int lane_off = lane * static_cast<int>(sizeof(T));
                        // entries past a run re-read its last one, weighted 0
                        auto load_run = [&](int src, int end, T (&buf)[RUN]) {
#pragma unroll
                            for (int r = 0; r < RUN; ++r) {
                                const int j = min(src + r, end - 1);
                                const int row = __builtin_amdgcn_readlane(ti, j) * 64 * static_cast<int>(sizeof(T));
                                buf[r] = buffer_load_value<T>(nvr, lane_off, row);
                            }
                        };
                        auto apply_run = [&](int src, int end, const T (&buf)[RUN]) {
                            T nsum = T(0);
#pragma unroll
                            for (int r = 0; r < RUN; ++r) {
                                const int j = min(src + r, end - 1);
                                const T w = src + r < end ? lane_bcast(c1, j) : T(0);
                                nsum += w * buf[r];
                            }
                            const T a = lane_bcast(ca, src) + nsum;
                            const T bq = lane_bcast(cb, src) + nsum;
                            const int pls = __builtin_amdgcn_readlane(pl, src);
                            const T fpb = s_F[pls * 65 + lane];
                            sa += a * (T(1) - fpb);
                            sb += bq * fpb;
                        };
                        // two runs in flight: the next run's N loads are
                        // issued before this run's are waited for (two
                        // register sets, so nothing is copied between them).
                        // Past the last run the loads repeat the current
                        // one, so every step issues the same number of loads
                        // and the wait for a run never covers the next.
                        if (m) {
                            T b0[RUN], b1[RUN];
                            int s0 = __builtin_ctzll(m), s1, t1;
                            m &= m - 1;
                            int t0 = m ? __builtin_ctzll(m) : nvalid;
                            load_run(s0, t0, b0);
                            while (true) {
                                const bool h1 = m != 0;
                                s1 = h1 ? __builtin_ctzll(m) : s0;
                                m &= m - 1;
                                t1 = h1 ? (m ? __builtin_ctzll(m) : nvalid) : t0;
                                load_run(s1, t1, b1);
                                apply_run(s0, t0, b0);
                                if (!h1) break;
                                const bool h0 = m != 0;
                                s0 = h0 ? __builtin_ctzll(m) : s1;
                                m &= m - 1;
                                t0 = h0 ? (m ? __builtin_ctzll(m) : nvalid) : t1;
                                load_run(s0, t0, b0);
                                apply_run(s1, t1, b1);
                                if (!h0) break;
                            }
                        }
                    } else {
                        while (m) {
                            const int src = __builtin_ctzll(m);
                            m &= m - 1;
                            const T a = lane_bcast(ca, src);
                            const T bq = lane_bcast(cb, src);
                            const int pls = __builtin_amdgcn_readlane(pl, src);
                            const T fpb = s_F[pls * 65 + lane];
                            sa += a * (T(1) - fpb);
                            sb += bq * fpb;
                        }
                    }
                }
                acc_a[j] += sa;
                acc_b[j] += sb;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < DPW; ++j) {
        const int dl = wave + j * nw;
        if (dl < nd && lane < nb) {
            const int d = t.d0 + dl;
            const int b = b0 + lane;
            const T fd = f[static_cast<int64_t>(b) * ldf + d];
            apply_epi(E, b, d, A.S, A.K * ((T(1) - fd) * acc_b[j] - fd * acc_a[j]));
        }
    }
}

// Moves v from the lane the DPP control selects (rows of 16 lanes; ROWS masks
// the rows that receive, the others and lanes without a source get 0).
template <int CTRL, int ROWS> __device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_mov(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

// Sum over the 64 lanes of a wave, returned to every lane, without LDS:
// shifts by 1, 2, 4 and 8 lanes inside each row of 16 leave the row's sum in
// its lane 15; broadcasting lane 15 into the next row (rows 1 and 3) and then
// lane 31 into rows 2 and 3 leaves the total in lane 63.  Fixed order.
template <typename T> __device__ __forceinline__ T wave_total(T v) {
    v += dpp_mov<0x111, 0xf>(v);   // row_shr:1
    v += dpp_mov<0x112, 0xf>(v);   // row_shr:2
    v += dpp_mov<0x114, 0xf>(v);   // row_shr:4
    v += dpp_mov<0x118, 0xf>(v);   // row_shr:8
    v += dpp_mov<0x142, 0xa>(v);   // row_bcast:15
    v += dpp_mov<0x143, 0xc>(v);   // row_bcast:31
    return lane_bcast(v, 63);
}

// Reverse mode of Eq. 2 for up to 64 vectors sharing one phonon table
// (vectors b0 .. b0 + nb - 1; lane = vector).  Tiles and sub-tiles as in
// k_fwd_batched; the LDS tile holds {f_p, lam_p} per (partner, vector).
//   dL/df_d = -K sum_e (lam_d - lam_p) u_e,  u_e = a_e (1 - f_p) + b_e f_p,
// summed per lane as lam_d sum u - sum lam_p u.  The |g|^2 gradient of a
// channel, written by its entry with p > d, is
//   K [bh sum_b (lam_d - lam_p) f_p (1 - f_d) - ah sum_b (lam_d - lam_p) f_d (1 - f_p)],
// where the two sums over the vectors depend only on the pair (d, p): they are
// reduced across the wave once per run of equal partners and serve every mode
// of the run.  gg2_mode: 0 none, 1 overwrite, 2 add.  Every slot is written by
// one lane of one launch: deterministic.
// RUN > 0: a bath per vector, N from nvec as in k_fwd_batched (the 64
// vectors of this launch).  With c = G(x + hw) + G(x - hw) the coefficients
// split into the N-free parts and c N_b; a channel's |g|^2 gradient is
//   K [G(x + hw) p2 - G(x - hw) p1 + c sum_b N_b (P2_b - P1_b)],
// P1_b = (lam_d - lam_p) f_d (1 - f_p), P2_b = (lam_d - lam_p) f_p (1 - f_d),
// p1 and p2 their sums over the vectors: one more sum over the wave per
// channel.
template <typename T, int DPW, int RUN>
__global__ __launch_bounds__(512) void k_vjp_batched(BArgs<T> A, const T *__restrict__ f, int64_t ldf,
                                                     const T *__restrict__ lam, int64_t ldl, int b0,
                                                     int nb, T *__restrict__ gf, int64_t ldgf,
                                                     const int32_t *__restrict__ ent_chan,
                                                     double *__restrict__ gg2, int gg2_mode,
                                                     const T *__restrict__ nvec, int64_t nvec_ld) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int PT = A.pt;
    Pair2<T> *s_FL = reinterpret_cast<Pair2<T> *>(smem);                   // [PT][65]
    StateRec<T> *s_ek = reinterpret_cast<StateRec<T> *>(s_FL + PT * 65);  // [PT]
    const int64_t ti = tile_of_block(A.n_btiles, A.xcd);
    if (ti < 0) return;
    const BTileRec t = A.btiles[ti];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    const int nd = t.d1 - t.d0;
    const bool lv = lane < nb;
    T fd[DPW], ld[DPW], acc_u[DPW], acc_l[DPW];
#pragma unroll
    for (int j = 0; j < DPW; ++j) {
        const int dl = wave + j * nw;
        const bool ok = dl < nd && lv;
        const int64_t row = static_cast<int64_t>(b0 + lane);
        fd[j] = ok ? f[row * ldf + t.d0 + dl] : T(0);
        ld[j] = ok ? lam[row * ldl + t.d0 + dl] : T(0);
        acc_u[j] = T(0);
        acc_l[j] = T(0);
    }
    for (int k = 0; k < t.n_sub; ++k) {
        const int pa = t.p_lo + k * PT;
        const int pc = min(PT, A.S - pa);
        __syncthreads();
        // vectors past nb hold f = lam = 0: their terms vanish in every sum
        for (int i = threadIdx.x; i < pc * 64; i += blockDim.x) {
            const int bb = i / pc, pl = i - bb * pc;
            Pair2<T> v;
            v.a = T(0);
            v.b = T(0);
            if (bb < nb) {
                const int64_t row = static_cast<int64_t>(b0 + bb);
                v.a = f[row * ldf + pa + pl];
                v.b = lam[row * ldl + pa + pl];
            }
            s_FL[pl * 65 + bb] = v;
        }
        for (int i = threadIdx.x; i < pc; i += blockDim.x) s_ek[i] = A.st[pa + i];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < DPW; ++j) {
            const int dl = wave + j * nw;
            if (dl < nd) {
                const int d = t.d0 + dl;
                const int64_t *so = A.sub_off + t.off_base + static_cast<int64_t>(dl) * (t.n_sub + 1);
                const int64_t e_lo = so[k], e_hi = so[k + 1];
                const StateRec<T> sd = A.st[d];
                // the pairs of this sub-tile with p > d carry the |g|^2 gradients
                const bool g_any = gg2_mode != 0 && pa + pc - 1 > d;
                T su = T(0), sl = T(0);   // this sub-tile's sums (two-level, as in the forward)
                for (int64_t e0 = e_lo; e0 < e_hi; e0 += 64) {
                    const int64_t e = e0 + lane;
                    const bool valid = e < e_hi;
                    int pl = -1 - lane;     // distinct for invalid lanes: never merged
                    T ca = T(0), cb = T(0), ah = T(0), bh = T(0), c1 = T(0);
                    int32_t ch = -1;
                    int ti = 0;
                    if (valid) {
                        const uint32_t pn = A.pnu[e];
                        const T g = A.g2[e];
                        pl = static_cast<int>(pn >> 3) - pa;
                        const StateRec<T> sp = s_ek[pl];
                        const int q = A.padq ? static_cast<int>(sp.kqp - sd.kqp) + A.qoff
                                             : q_linear(sd.kq, sp.kq, A.nq0, A.nq1, A.nq2);
                        const Pair2<T> wn = A.hwN[static_cast<int64_t>(q) * A.tq + static_cast<int64_t>(pn & 7u) * A.tm];
                        const T de = sd.eps - sp.eps;
                        const T xa = de + wn.a, xe = de - wn.a;
                        const T da = gauss_exp(xa * xa * A.mc);
                        const T dem = gauss_exp(xe * xe * A.mc);
                        if constexpr (RUN > 0) {
                            // ah, bh keep the N-free parts; c1 the N coefficient
                            ah = dem;
                            bh = da;
                            ca = g * dem;
                            cb = g * da;
                            c1 = g * (da + dem);
                            ti = q * A.nm + static_cast<int>(pn & 7u);
                        } else {
                            const T tt = wn.b * (da + dem);
                            ah = tt + dem;
                            bh = tt + da;
                            ca = g * ah;
                            cb = g * bh;
                        }
                        if (g_any && pa + pl > d) ch = ent_chan[e];
                    }
                    // sum each run of equal partners into its first lane (a run is
                    // one pair over its modes, at most kMaxRun lanes)
#pragma unroll
                    for (int off = 1; off < kMaxRun; off <<= 1) {
                        const T oa = __shfl_down(ca, off, 64);
                        const T ob = __shfl_down(cb, off, 64);
                        const int op = __shfl_down(pl, off, 64);
                        if (lane + off < 64 && op == pl) {
                            ca += oa;
                            cb += ob;
                        }
                    }
                    const int prev = __shfl_up(pl, 1, 64);
                    const bool head = valid && (lane == 0 || prev != pl);
                    unsigned long long m = __ballot(head);
                    if constexpr (RUN > 0) {
                        // a run of entries (one pair over its modes) ends at
                        // the next head or the last valid lane; its N per
                        // vector through a buffer resource (reads past the
                        // table return 0)
                        const int nvalid = static_cast<int>(min<int64_t>(64, e_hi - e0));
                        const __amdgpu_buffer_rsrc_t nvr = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<T *>(nvec), 0, static_cast<int>(nvec_ld * sizeof(T)), kBufferDword3);
                        const int lane_off = lane * static_cast<int>(sizeof(T));
                        while (m) {
                            const int src = __builtin_ctzll(m);
                            m &= m - 1;
                            const int end = m ? __builtin_ctzll(m) : nvalid;
                            T nv[RUN];
#pragma unroll
                            for (int r = 0; r < RUN; ++r) {
                                const int jj = min(src + r, end - 1);
                                const int row = __builtin_amdgcn_readlane(ti, jj) * 64 * static_cast<int>(sizeof(T));
                                nv[r] = buffer_load_value<T>(nvr, lane_off, row);
                            }
                            T nsum = T(0);
#pragma unroll
                            for (int r = 0; r < RUN; ++r) {
                                const int jj = min(src + r, end - 1);
                                const T w = src + r < end ? lane_bcast(c1, jj) : T(0);
                                nsum += w * nv[r];
                            }
                            const T a = lane_bcast(ca, src) + nsum;
                            const T bq = lane_bcast(cb, src) + nsum;
                            const int pls = __builtin_amdgcn_readlane(pl, src);
                            const Pair2<T> fl = s_FL[pls * 65 + lane];
                            const T u = a + (bq - a) * fl.a;
                            su += u;
                            sl += fl.b * u;
                            if (g_any && pa + pls > d) {
                                const T dlm = ld[j] - fl.b;
                                const T q1 = dlm * fd[j] * (T(1) - fl.a);
                                const T q2 = dlm * fl.a * (T(1) - fd[j]);
                                const T p1 = wave_total(q1);
                                const T p2 = wave_total(q2);
#pragma unroll
                                for (int r = 0; r < RUN; ++r) {
                                    if (src + r >= end) break;
                                    const T rn = wave_total(nv[r] * (q2 - q1));
                                    if (lane == src + r && ch >= 0) {
                                        const double v = static_cast<double>(A.K * (bh * p2 - ah * p1 + (ah + bh) * rn));
                                        gg2[ch] = gg2_mode == 2 ? gg2[ch] + v : v;
                                    }
                                }
                            }
                        }
                    } else {
                        while (m) {
                            const int src = __builtin_ctzll(m);
                            m &= m - 1;
                            const T a = lane_bcast(ca, src);
                            const T bq = lane_bcast(cb, src);
                            const int pls = __builtin_amdgcn_readlane(pl, src);
                            const Pair2<T> fl = s_FL[pls * 65 + lane];
                            const T u = a + (bq - a) * fl.a;
                            su += u;
                            sl += fl.b * u;
                            if (g_any && pa + pls > d) {
                                const T dlm = ld[j] - fl.b;
                                const T p1 = wave_total(dlm * fd[j] * (T(1) - fl.a));
                                const T p2 = wave_total(dlm * fl.a * (T(1) - fd[j]));
                                if (pl == pls && ch >= 0) {
                                    const double v = static_cast<double>(A.K * (bh * p2 - ah * p1));
                                    gg2[ch] = gg2_mode == 2 ? gg2[ch] + v : v;
                                }
                            }
                        }
                    }
                }
                acc_u[j] += su;
                acc_l[j] += sl;
            }
        }
    }
    if (!gf) return;
#pragma unroll
    for (int j = 0; j < DPW; ++j) {
        const int dl = wave + j * nw;
        if (dl < nd && lv)
            gf[static_cast<int64_t>(b0 + lane) * ldgf + t.d0 + dl] = -A.K * (ld[j] * acc_u[j] - acc_l[j]);
    }
}

// ---- phonon side of the same processes (coupled e-ph dynamics) ----------
// A channel (i, j, nu) carries the processes that exchange phonon (nu, q),
// q = k_j - k_i (i -> j absorbing it, j -> i emitting it, delta
// G(e_i - e_j + hw)), and those that exchange (nu, -q) (delta
// G(e_i - e_j - hw)).  The channels are grouped by the unordered pair
// {qc, -qc} into pair records (a, b) with k_b - k_a = qc and one |g|^2 slot
// per mode (zero where the pair has no channel of that mode), bucketed by qc
// and cut into chunks of at most kPhChunk records.  One wave reduces one
// chunk: with P1 = f_b (1 - f_a), P2 = f_a (1 - f_b), a record adds
//   |g|^2 G(e_a - e_b + hw(qc)) (P1 + N(qc) (P1 - P2))    to bin (qc, nu),
//   |g|^2 G(e_a - e_b - hw(-qc)) (P2 - N(-qc) (P1 - P2))  to bin (-qc, nu),
// (net emission: (N+1) x gain - N x loss), in registers, in record order;
// the two sums per mode go to the chunk's partials, and k_phonon_bins_finish
// adds the partials of each bin in chunk order.  No atomics.
constexpr int kPhChunk = 512;

template <typename T> struct PhArgs {
    const uint32_t *__restrict__ pa;
    const uint32_t *__restrict__ pb;
    const T *__restrict__ g2;          // [n_modes][ld]
    int64_t ld;
    const StateRec<T> *__restrict__ st;
    const T *__restrict__ hw;          // [Nq][n_modes]
    const int64_t *__restrict__ chunk_beg;    // [n_chunks + 1] record ranges
    const int32_t *__restrict__ chunk_bucket; // [n_chunks]
    const int32_t *__restrict__ bucket_chunk; // [n_buckets + 1]
    const int32_t *__restrict__ bucket_q;     // [n_buckets] qc
    const int32_t *__restrict__ bucket_qm;    // [n_buckets] -qc
    const uint32_t *__restrict__ bucket_modes;
    const int32_t *__restrict__ q_bucket;     // [Nq] 2 bucket + side, -1: none
    int64_t n_chunks;
    int64_t nq;
    int nm;
    T mc;                    // Gaussian exponent scale, base 2
    double mc256;            // 256 mc (FP64 table exponential)
    const double *__restrict__ e2tab;
    double Kp;               // 2 pi / (hbar N_k) / (sigma sqrt(2 pi))
    uint32_t elastic;        // bit nu: mode nu is elastic (no phonon side)
    const int32_t *__restrict__ chan;   // [n_modes][ld] caller channel of each slot, -1: none
};

// a b + c rounded once, in the type of its arguments
__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename T>
__device__ __forceinline__ T ph_gauss(const PhArgs<T> &A, T x, const double *tab) {
    if constexpr (sizeof(T) == 8) return gauss_exp2_tab(x * x * A.mc256, tab);
    else return __builtin_amdgcn_exp2f(x * x * A.mc);
}

// The mode loop is unrolled to NM >= nm slots (1, 2, 3, 4, 6 or 8).  The
// record stream (a, b and the |g|^2 slots) runs one batch ahead of the state
// gathers and the evaluation, with two register sets, as in the pair pass;
// a lane past the chunk's end re-reads the chunk's last record and adds
// nothing.
template <typename T, int NM>
__global__ __launch_bounds__(256) void k_phonon_bins(PhArgs<T> A, const T *__restrict__ f,
                                                     const T *__restrict__ nph, T *__restrict__ part) {
    __shared__ double s_tab[kExpTab];
    if constexpr (sizeof(T) == 8)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t c = static_cast<int64_t>(blockIdx.x) * (blockDim.x >> 6) +
                      __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    if (c >= A.n_chunks) return;
    const int nm = A.nm;
    const int bk = A.chunk_bucket[c];
    const int64_t qc = A.bucket_q[bk], qm = A.bucket_qm[bk];
    const uint32_t modes = A.bucket_modes[bk] & ~A.elastic;
    T w1[NM], n1[NM], w2[NM], n2[NM], acc1[NM], acc2[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        const bool on = m < nm && ((modes >> m) & 1u);
        const int mm = min(m, nm - 1);
        w1[m] = on ? A.hw[qc * nm + mm] : T(0);
        n1[m] = on ? nph[qc * nm + mm] : T(0);
        w2[m] = on ? A.hw[qm * nm + mm] : T(0);
        n2[m] = on ? nph[qm * nm + mm] : T(0);
        acc1[m] = T(0);
        acc2[m] = T(0);
    }
    const int64_t beg = A.chunk_beg[c];
    const int n = static_cast<int>(A.chunk_beg[c + 1] - beg);
    auto rec = [&](int r) { return beg + min(r + lane, n - 1); };
    uint32_t a0 = A.pa[rec(0)], b0 = A.pb[rec(0)], a1 = 0, b1 = 0;
    T g0[NM], g1[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) g0[m] = A.g2[min(m, nm - 1) * A.ld + rec(0)];
    auto batch = [&](int r, const uint32_t a, const uint32_t b, const T (&g)[NM], uint32_t &an, uint32_t &bn,
                     T (&gn)[NM]) {
        const bool v = r + lane < n;
        const T fa = f[a], fb = f[b];
        const T d = A.st[a].eps - A.st[b].eps;
        __builtin_amdgcn_sched_barrier(0);
        const int64_t x = rec(r + 64);
        an = A.pa[x];
        bn = A.pb[x];
#pragma unroll
        for (int m = 0; m < NM; ++m) gn[m] = A.g2[min(m, nm - 1) * A.ld + x];
        __builtin_amdgcn_sched_barrier(0);
        const T p1 = fb * (T(1) - fa), p2 = fa * (T(1) - fb);
        const T dp = p1 - p2;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            // modes outside the bucket (and elastic ones) add nothing
            const T gm = keep_or_zero(g[m], v && m < nm && ((modes >> m) & 1u));
            const T ga = ph_gauss(A, d + w1[m], s_tab);
            const T ge = ph_gauss(A, d - w2[m], s_tab);
            acc1[m] = fma(gm * ga, fma(n1[m], dp, p1), acc1[m]);
            acc2[m] = fma(gm * ge, fma(-n2[m], dp, p2), acc2[m]);
        }
    };
    for (int r = 0; r < n; r += 128) {
        batch(r, a0, b0, g0, a1, b1, g1);
        if (r + 64 >= n) break;
        batch(r + 64, a1, b1, g1, a0, b0, g0);
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        acc1[m] = wave_sum(acc1[m]);
        acc2[m] = wave_sum(acc2[m]);
    }
    if (lane == 0) {
        T *pc = part + c * 2 * nm;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            if (m >= nm) break;
            pc[m] = acc1[m];
            pc[nm + m] = acc2[m];
        }
    }
}

// Reverse mode over the same records at a stage (u, N) of the coupled step,
// given lam = dL/dI and mu = dL/d(dN/dt) per bin.  Per record and mode, with
// x = e_a - e_b, G1 = G(x + hw(qc)), E1 = G(x - hw(qc)), G2 = G(x + hw(-qc)),
// E2 = G(x - hw(-qc)) (two exponentials when hw(-qc) = hw(qc)):
//   bin (qc, nu):  |g|^2 (f_b - f_a) [Ke lam_a (G1 + E1) + Kp mu(qc) G1]
//   bin (-qc, nu): |g|^2 (f_a - f_b) [Ke lam_b (G2 + E2) + Kp mu(-qc) E2]
// (dL/dN: the collision integral is affine in N, the phonon-side rate too);
// and, for phonon modes, dL/d|g|^2 of the record's channel gains
//   Kp [mu(qc) G1 (P1 + N(qc) (P1 - P2)) + mu(-qc) E2 (P2 - N(-qc) (P1 - P2))]
// (its only writer: every channel has one slot).  Elastic modes have no
// phonon side: only their lam terms.  lam or mu may be null (taken as 0).
// The mode loop is unrolled to NM >= nm slots and the record stream (a, b,
// |g|^2 slots and, with gg2, the slots' channels) runs one batch ahead, as in
// k_phonon_bins.  With gg2, the old values of a batch's channels are loaded
// before the next batch's stream is issued, so that waiting for them does
// not wait for the stream; each channel has one slot, so nothing else writes
// it in between.  Where the channels of every record of a batch are consecutive
// they are read and written in channel order, the values passing through LDS
// (see wave_write_gg2).  Bound by that and by the few waves in flight (207 VGPRs
// in FP64 at six modes, two waves a SIMD; three waves by launch bounds spill:
// 237 us).  1.9 M records, six modes, FP64: 148 us, 198 with a lane per record
// and the mode constants in registers (276, one wave).  A lane past the chunk's end, or a slot without a channel,
// loads a valid address and stores nothing.
// Which products are fused into an addition is written out: dL/d|g|^2 is an FP64
// output in FP32 plans too, and the choice, left to the compiler, moved it by FP32
// roundings (4e-9 of its norm over a coupled adjoint) when the constants went to
// LDS.  It is the one that the build with the constants in registers made: in a
// bin's term the sum of the Gaussians is the fused factor in the even batches of
// more than one mode slot, the channel's mu elsewhere.
template <typename T, int NM>
__global__ __launch_bounds__(256) void k_phonon_bins_adj(PhArgs<T> A, const T *__restrict__ f,
                                                         const T *__restrict__ nph, const T *__restrict__ lam,
                                                         const T *__restrict__ mu, T *__restrict__ part,
                                                         double *__restrict__ gg2, double Ke) {
    __shared__ double s_tab[kExpTab];
    __shared__ double s_g[4][64 * NM];
    __shared__ T s_k[4][6 * NM];
    if constexpr (sizeof(T) == 8)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t c = static_cast<int64_t>(blockIdx.x) * (blockDim.x >> 6) +
                      __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    if (c >= A.n_chunks) return;
    double *s_w = s_g[threadIdx.x >> 6];
    const int nm = A.nm;
    const int bk = A.chunk_bucket[c];
    const int64_t qc = A.bucket_q[bk], qm = A.bucket_qm[bk];
    const uint32_t modes = A.bucket_modes[bk];
    const uint32_t phon = mu ? modes & ~A.elastic : 0u;
    const bool want_g = gg2 != nullptr && phon != 0u;
    const T ke = static_cast<T>(Ke), kp = static_cast<T>(A.Kp);
    // per mode hw(qc), hw(-qc), mu and N of both: the wave's, kept in LDS (in
    // registers they cost 72 VGPRs in FP64 at six modes, and with them all but one
    // wave of a SIMD)
    T *s_c = s_k[threadIdx.x >> 6];
    bool other = false;   // hw(-qc) != hw(qc) for a mode of the bucket
    if (lane < NM) {
        const int mm = min(lane, nm - 1);
        const bool on = lane < nm && ((modes >> lane) & 1u);
        const bool ph = lane < nm && ((phon >> lane) & 1u);
        const T wa = on ? A.hw[qc * nm + mm] : T(0), wb = on ? A.hw[qm * nm + mm] : T(0);
        s_c[6 * lane] = wa;
        s_c[6 * lane + 1] = wb;
        s_c[6 * lane + 2] = ph ? mu[qc * nm + mm] : T(0);
        s_c[6 * lane + 3] = ph ? mu[qm * nm + mm] : T(0);
        s_c[6 * lane + 4] = ph ? nph[qc * nm + mm] : T(0);
        s_c[6 * lane + 5] = ph ? nph[qm * nm + mm] : T(0);
        other = wb != wa;
    }
    const bool same = __ballot(other) == 0;
    wave_lds_sync();
    T acc1[NM], acc2[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) acc1[m] = acc2[m] = T(0);
    const int64_t beg = A.chunk_beg[c];
    const int n = static_cast<int>(A.chunk_beg[c + 1] - beg);
    auto rec = [&](int r) { return beg + min(r + lane, n - 1); };
    uint32_t a0 = A.pa[rec(0)], b0 = A.pb[rec(0)], a1 = 0, b1 = 0;
    T g0[NM], g1[NM];
    int32_t h0[NM], h1[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        g0[m] = A.g2[min(m, nm - 1) * A.ld + rec(0)];
        h0[m] = want_g ? A.chan[min(m, nm - 1) * A.ld + rec(0)] : -1;
    }
    auto batch = [&](auto oddc, int r, const uint32_t a, const uint32_t b, const T (&g)[NM], const int32_t (&h)[NM],
                     uint32_t &an, uint32_t &bn, T (&gn)[NM], int32_t (&hn)[NM]) {
        // a b + c d (which product is fused: see above)
        auto term = [](T a, T b, T c, T d) {
            return NM == 1 || decltype(oddc)::value ? fused(c, d, a * b) : fused(a, b, c * d);
        };
        const bool v = r + lane < n;
        const T fa = f[a], fb = f[b];
        const T la = lam ? lam[a] : T(0), lb = lam ? lam[b] : T(0);
        const T x = A.st[a].eps - A.st[b].eps;
        double old[NM];
        bool seq = false;
        const int32_t cv = v ? h[0] : -1;
        if (want_g) {
            bool own = nm == NM && h[0] >= 0;
#pragma unroll
            for (int m = 1; m < NM; ++m) own = own && h[m] == h[0] + m;
            seq = NM > 1 && __ballot(v && !own) == 0;
            if (seq) {
#pragma unroll
                for (int j = 0; j < NM; ++j) {
                    const int u = j * 64 + lane, rec = u / NM;
                    const int32_t ch = __shfl(cv, rec, 64);
                    old[j] = gg2[ch >= 0 ? ch + (u - rec * NM) : 0];
                }
            } else {
#pragma unroll
                for (int m = 0; m < NM; ++m) old[m] = gg2[h[m] >= 0 ? h[m] : 0];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        const int64_t xi = rec(r + 64);
        an = A.pa[xi];
        bn = A.pb[xi];
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            gn[m] = A.g2[min(m, nm - 1) * A.ld + xi];
            hn[m] = want_g ? A.chan[min(m, nm - 1) * A.ld + xi] : -1;
        }
        __builtin_amdgcn_sched_barrier(0);
        const T ofa = T(1) - fa, p1 = fb * ofa, p2 = fa * (T(1) - fb);
        const T dp = fused(fb, ofa, -p2);   // = f_b - f_a
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const bool on = v && m < nm && ((modes >> m) & 1u);
            const T gm = keep_or_zero(g[m], on);
            const T *k = s_c + 6 * m;
            const T w1 = k[0], w2 = k[1], m1 = k[2], m2 = k[3];
            const T gq1 = ph_gauss(A, x + w1, s_tab);
            const T e1 = ph_gauss(A, x - w1, s_tab);
            T gq2 = gq1, e2 = e1;
            if (!same) {
                gq2 = ph_gauss(A, x + w2, s_tab);
                e2 = ph_gauss(A, x - w2, s_tab);
            }
            const T gd = gm * dp;
            acc1[m] = fused(gd, term(ke * la, gq1 + e1, kp * m1, gq1), acc1[m]);
            acc2[m] = fused(-gd, term(ke * lb, gq2 + e2, kp * m2, e2), acc2[m]);
            if (want_g) {
                const T c2 = m2 * e2 * fused(-k[5], dp, p2);
                const double dg = static_cast<double>(kp * fused(m1 * gq1, fused(k[4], dp, p1), c2));
                if (seq) s_w[lane * NM + m] = dg;
                else if (on && ((phon >> m) & 1u) && h[m] >= 0) gg2[h[m]] = old[m] + dg;
            }
        }
        if (seq) {
            wave_lds_sync();
#pragma unroll
            for (int j = 0; j < NM; ++j) {
                const int u = j * 64 + lane, rec = u / NM, m = u - rec * NM;
                const int32_t ch = __shfl(cv, rec, 64);
                if (ch >= 0 && ((phon >> m) & 1u)) gg2[ch + m] = old[j] + s_w[u];
            }
            wave_lds_sync();
        }
    };
    for (int r = 0; r < n; r += 128) {
        batch(std::false_type{}, r, a0, b0, g0, h0, a1, b1, g1, h1);
        if (r + 64 >= n) break;
        batch(std::true_type{}, r + 64, a1, b1, g1, h1, a0, b0, g0, h0);
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        acc1[m] = wave_sum(acc1[m]);
        acc2[m] = wave_sum(acc2[m]);
    }
    if (lane == 0) {
        T *pc = part + c * 2 * nm;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            if (m >= nm) break;
            pc[m] = acc1[m];
            pc[nm + m] = acc2[m];
        }
    }
}

// Per-vector baths of the batched pass, 64 vectors: entry (row nm + nu) 64 + j
// holds N of vector j (0 past the last of the B vectors) at table row `row`
// and mode nu, for the box rows in `used` (pad != 0; other rows keep their
// zeros) or every q (pad = 0, n_rows = Nq).  nph holds B tables of [Nq][nm].
template <typename T>
__global__ void k_pack_nvec(const T *__restrict__ nph, T *__restrict__ out, int pad, QBox Bx, int nm,
                            const int32_t *__restrict__ used, int n_rows, int B) {
    const int64_t tab = static_cast<int64_t>(Bx.n[0]) * Bx.n[1] * Bx.n[2] * nm;
    const int64_t n = static_cast<int64_t>(n_rows) * nm * 64;
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int j = static_cast<int>(i & 63);
        const int64_t r = i >> 6;
        const int nu = static_cast<int>(r % nm);
        const int u = static_cast<int>(r / nm);
        const int row = pad ? used[u] : u;
        const int64_t q = pad ? box_q(row, Bx) : row;
        out[(static_cast<int64_t>(row) * nm + nu) * 64 + j] = j < B ? nph[static_cast<int64_t>(j) * tab + q * nm + nu] : T(0);
    }
}

// {hw, N, mu} per (q, mode) for the reverse of the phonon-side rate: the
// box of k_pack_hwN_pad with the modes of one row adjacent (pad != 0), or the
// plain table.
template <typename T>
__global__ void k_pack_hwNmu(const T *__restrict__ hw, const T *__restrict__ nph, const T *__restrict__ mu,
                             Vec4<T> *__restrict__ out, int pad, QBox B, int nm, const int32_t *__restrict__ used,
                             int64_t n) {
    // pad != 0: n = (rows in used) nm, other box rows keep their zeros
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        int64_t src = i, dst = i;
        if (pad) {
            const int row = used[i / nm];
            src = static_cast<int64_t>(box_q(row, B)) * nm + i % nm;
            dst = static_cast<int64_t>(row) * nm + i % nm;
        }
        Vec4<T> v;
        v.x = hw[src];
        v.y = nph[src];
        v.z = mu[src];
        v.w = T(0);
        out[dst] = v;
    }
}

// Electron side of the reverse of the phonon-side rate: for every entry
// (d, p, nu) with q = k_p - k_d (x = e_d - e_p),
//   dL/df_d += Kp |g|^2 [mu(-q) G(x - hw(-q)) (N(-q) + 1 - f_p) - mu(q) G(x + hw(q)) (N(q) + f_p)]
// (the entry's channel feeds bin q through G(x + hw(q)) and bin -q through
// G(x - hw(-q)); the same form holds from either end of the channel).  One
// workgroup per chunk of the destination layout; a destination with one
// chunk adds its sum to out, others leave a partial for k_vjp_phonon_f_finish.
// The entry stream (partner word, |g|^2) runs one batch ahead of the state
// and table gathers, with two register sets, as in the pair pass; the
// entry arrays are padded past their end, so the prefetch needs no bound, and
// a thread past the row's end (or on an elastic mode) adds nothing.
template <typename T>
__global__ __launch_bounds__(256) void k_vjp_phonon_f(TiledArgs<T> A, const Vec4<T> *__restrict__ tab,
                                                      const T *__restrict__ f, uint32_t elastic,
                                                      double Kp, T *__restrict__ out, T *__restrict__ part) {
    __shared__ double s_tab[kExpTab];
    if constexpr (sizeof(T) == 8)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    __syncthreads();
    const int64_t c = blockIdx.x;
    if (c >= A.n_chunks) return;
    const int d = A.chunk_dest[c];
    const int64_t beg = A.chunk_beg[c], end = A.chunk_beg[c + 1];
    const StateRec<T> sd = A.st[d];
    const int64_t stride = blockDim.x;
    T acc[1] = {T(0)};
    int64_t e = beg + threadIdx.x;
    uint32_t pn0 = A.pnu[e], pn1 = 0;
    T g0 = A.g2[e], g1 = T(0);
    auto step = [&](int64_t x, const uint32_t pn, const T g, uint32_t &pn_next, T &g_next) {
        const int mode = static_cast<int>(pn & 7u);
        const int p = static_cast<int>(pn >> 3);
        const StateRec<T> sp = A.st[p];
        const T fp = f[p];
        int64_t iq, im;
        if (A.padq) {
            iq = static_cast<int64_t>(static_cast<int>(sp.kqp - sd.kqp) + A.qoff);
            im = 2 * static_cast<int64_t>(A.qoff) - iq;
        } else {
            iq = q_linear(sd.kq, sp.kq, A.nq0, A.nq1, A.nq2);
            im = q_linear(sp.kq, sd.kq, A.nq0, A.nq1, A.nq2);
        }
        const Vec4<T> t1 = tab[iq * A.nm + mode], t2 = tab[im * A.nm + mode];
        __builtin_amdgcn_sched_barrier(0);
        pn_next = A.pnu[x + stride];
        g_next = A.g2[x + stride];
        __builtin_amdgcn_sched_barrier(0);
        const T gm = keep_or_zero(g, x < end && !((elastic >> mode) & 1u));
        const T xe = sd.eps - sp.eps;
        const T ga = stream_gauss(A, (xe + t1.x) * (xe + t1.x), s_tab);
        const T ge = stream_gauss(A, (xe - t2.x) * (xe - t2.x), s_tab);
        acc[0] += gm * (t2.z * ge * (t2.y + T(1) - fp) - t1.z * ga * (t1.y + fp));
    };
    for (; e < end; e += 2 * stride) {
        step(e, pn0, g0, pn1, g1);
        if (e + stride >= end) break;
        step(e + stride, pn1, g1, pn0, g0);
    }
    block_sum<T, 1>(acc);
    if (threadIdx.x == 0) {
        const T v = static_cast<T>(Kp) * acc[0];
        if (A.dest_chunk[d + 1] - A.dest_chunk[d] == 1) out[d] += v;
        else part[c] = v;
    }
}

template <typename T>
__global__ void k_vjp_phonon_f_finish(TiledArgs<T> A, const T *__restrict__ part, T *__restrict__ out) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= A.S) return;
    const int c0 = A.dest_chunk[d], c1 = A.dest_chunk[d + 1];
    if (c1 - c0 == 1) return;
    T a = T(0);
    for (int c = c0; c < c1; ++c) a += part[c];
    out[d] += a;
}

// The same over pair records when every tile of the pair pass is q-ordered.
// A lane takes one pair (d, p) with all its modes; seen from p, q and -q swap
// roles and x = e_d - e_p changes sign, so the channel's two Gaussians
// ga = G(x + hw(q)) and ge = G(x - hw(-q)) serve both states:
//   dL/df_d += Kp |g|^2 [mu(-q) ge (N(-q) + 1 - f_p) - mu(q) ga (N(q) + f_p)]
//   dL/df_p += Kp |g|^2 [mu(q) ga (N(q) + 1 - f_d) - mu(-q) ge (N(-q) + f_d)]
// Each channel is read once and the lanes of a batch share the table rows of
// their q.  Both sides are fixed-point LDS sums on the scale of vjp_scale
// (max |mu| in place of max |lambda|), flushed to the global accumulator;
// k_vjp_phonon_pairs_finish adds them to out.  A slot without a channel (or
// of an elastic mode) is masked after its product, since its N may be
// infinite (acoustic modes at q = 0).  Fused products are written out, as in
// k_phonon_bins_adj, whose input lam these sums lead to.
template <typename T, bool PADQ, int NM>
__global__ __launch_bounds__(1024) void k_vjp_phonon_pairs(TiledArgs<T> A, const Vec4<T> *__restrict__ tab,
                                                          const T *__restrict__ f, uint32_t elastic,
                                                          MaxList mmax) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t ti = tile_of_block(A.n_tiles, A.xcd);
    if (ti < 0) return;
    const TileRec t = A.tiles[ti];
    const ScaleIn si = scale_load(A.nmax, A.gmax_bits, A.fmax, mmax);
    unsigned long long *s_j = reinterpret_cast<unsigned long long *>(smem);
    Pair2<T> *s_ef = reinterpret_cast<Pair2<T> *>(s_j + A.lds_states);
    uint32_t *s_kq = reinterpret_cast<uint32_t *>(s_ef + A.lds_states);
    double *s_tab = reinterpret_cast<double *>(s_kq + A.lds_states);
    const int n = t.p_hi - t.p_lo + 1;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const StateRec<T> sr = A.st[t.p_lo + i];
        Pair2<T> ef;
        ef.a = sr.eps;
        ef.b = f[t.p_lo + i];
        s_ef[i] = ef;
        s_kq[i] = PADQ ? sr.kqp : sr.kq;
        s_j[i] = 0ull;
    }
    if constexpr (sizeof(T) == 8)
        for (int i = threadIdx.x; i < kExpTab; i += blockDim.x) s_tab[i] = A.e2tab[i];
    const T scale = static_cast<T>(vjp_scale(si));
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int nw = static_cast<int>(blockDim.x >> 6);
    const int nm = A.nm;
    {
        const int64_t beg = A.chunk_beg[t.c0];
        const int len = static_cast<int>(A.chunk_end[t.c1 - 1] - beg);
        const int first = wave * 64, step = nw * 64;
        const uint32_t *__restrict__ pb = A.pnu + beg;
        const T *__restrict__ gb = A.g2 + beg;
        for (int r = first; r < len; r += step) {
            const bool v = r + lane < len;
            const uint32_t pn = pb[r + lane];
            // a masked lane takes window slot 0 as both states and adds nothing
            const int wd = v ? static_cast<int>(pn & 0xffffu) : 0;
            const int wp = v ? static_cast<int>(pn >> 16) : 0;
            const Pair2<T> efd = s_ef[wd], efp = s_ef[wp];
            const uint32_t kd = s_kq[wd], kp = s_kq[wp];
            int64_t iq, im;
            if (PADQ) {
                iq = static_cast<int64_t>(static_cast<int>(kp - kd) + A.qoff);
                im = 2 * static_cast<int64_t>(A.qoff) - iq;
            } else {
                iq = q_linear(kd, kp, A.nq0, A.nq1, A.nq2);
                im = q_linear(kp, kd, A.nq0, A.nq1, A.nq2);
            }
            const T x = efd.a - efp.a, fd = efd.b, fp = efp.b;
            T sd = T(0), sp = T(0);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int mm = min(m, nm - 1);
                const Vec4<T> t1 = tab[iq * nm + mm], t2 = tab[im * nm + mm];
                const T g = gb[mm * A.pld + r + lane];
                const bool on = v && m < nm && !((elastic >> m) & 1u) && g != T(0);
                const T ga = stream_gauss(A, (x + t1.x) * (x + t1.x), s_tab);
                const T ge = stream_gauss(A, (x - t2.x) * (x - t2.x), s_tab);
                const T a1 = t1.z * ga, a2 = t2.z * ge;
                sd += keep_or_zero(g * fused(a2, t2.y + T(1) - fp, -(a1 * (t1.y + fp))), on);
                sp += keep_or_zero(g * fused(a1, t1.y + T(1) - fd, -(a2 * (t2.y + fd))), on);
            }
            if (v) {
                atomicAdd(s_j + wd, to_fixed(__builtin_rint(sd * scale)));
                atomicAdd(s_j + wp, to_fixed(__builtin_rint(sp * scale)));
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const unsigned long long u = s_j[i];
        if (u) atomicAdd(A.jacc + t.p_lo + i, u);
    }
}

// out[d] += Kp (the fixed-point sum of d) / scale; the accumulator of d is
// cleared for the next call
template <typename T>
__global__ void k_vjp_phonon_pairs_finish(TiledArgs<T> A, MaxList mmax,
                                          double Kp, T *__restrict__ out) {
    const double inv = 1.0 / vjp_scale(scale_load(A.nmax, A.gmax_bits, A.fmax, mmax));
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= A.S) return;
    const long long j = static_cast<long long>(A.jacc[d]);
    A.jacc[d] = 0ull;
    out[d] += static_cast<T>(Kp * static_cast<double>(j) * inv);
}

// out = x (mode 0) or out = (x(q) + x(-q)) / 2 per (q, mode) (mode 1): the
// even part in q, which is its own transpose
template <typename T>
__global__ void k_even_q(const T *__restrict__ x, T *__restrict__ out, int n0, int n1, int n2, int nm) {
    const int64_t n = static_cast<int64_t>(n0) * n1 * n2 * nm;
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t q = i / nm;
        const int nu = static_cast<int>(i - q * nm);
        const int a2 = static_cast<int>(q % n2), a1 = static_cast<int>((q / n2) % n1),
                  a0 = static_cast<int>(q / (static_cast<int64_t>(n1) * n2));
        const int64_t qm = (static_cast<int64_t>((n0 - a0) % n0) * n1 + (n1 - a1) % n1) * n2 + (n2 - a2) % n2;
        out[i] = T(0.5) * (x[i] + x[qm * nm + nu]);
    }
}

// out = a x + b y (y may be null: out = a x)
template <typename T>
__global__ void k_axpby(int64_t n, T a, const T *__restrict__ x, T b, const T *__restrict__ y, T *__restrict__ out) {
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        out[i] = y ? a * x[i] + b * y[i] : a * x[i];
}

// dst[b][d] = -src[b][d] for B rows of S values (row strides lds, ldd; dst may
// be src)
template <typename T>
__global__ void k_neg_rows(const T *src, int64_t lds, T *dst, int64_t ldd, int B, int S) {
    const int64_t n = static_cast<int64_t>(B) * S;
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t b = i / S, d = i - b * S;
        dst[b * ldd + d] = -src[b * lds + d];
    }
}

// |g|^2 slots of the pair records from the caller's list (update_g2)
template <typename T>
__global__ void k_ph_gather_g2(const int32_t *__restrict__ chan, const double *__restrict__ g2,
                               T *__restrict__ out, int64_t n) {
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int32_t c = chan[i];
        out[i] = c >= 0 ? static_cast<T>(g2[c]) : T(0);
    }
}

// dN(q, nu) = Kp (sum over the chunks of q's bucket of q's side, in chunk
// order; both sides when q = -q), 0 for bins without channels.
template <typename T>
__global__ void k_phonon_bins_finish(PhArgs<T> A, const T *__restrict__ part, T *__restrict__ out) {
    const int64_t n = A.nq * A.nm;
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t q = i / A.nm;
        const int m = static_cast<int>(i - q * A.nm);
        const int qb = A.q_bucket[q];
        T sum = T(0);
        if (qb >= 0) {
            const int bk = qb >> 1, side = qb & 1;
            const int c0 = A.bucket_chunk[bk], c1 = A.bucket_chunk[bk + 1];
            for (int c = c0; c < c1; ++c) sum += part[(static_cast<int64_t>(c) * 2 + side) * A.nm + m];
            if (A.bucket_q[bk] == A.bucket_qm[bk])
                for (int c = c0; c < c1; ++c) sum += part[(static_cast<int64_t>(c) * 2 + 1) * A.nm + m];
        }
        out[i] = static_cast<T>(A.Kp * static_cast<double>(sum));
    }
}

// Pair records in a new order: slot m of position i takes slot m of position
// idx[i] (|g|^2 and channel), and so does the first-channel array; positions
// np .. ld - 1 get the padding values (|g|^2 0, channel -1).  idx[i] < np.
template <typename T>
__global__ __launch_bounds__(256) void k_permute_pairs(const uint32_t *__restrict__ idx, int64_t np, int64_t ld,
                                                       int nm, const T *__restrict__ g_in, T *__restrict__ g_out,
                                                       const int32_t *__restrict__ c_in, int32_t *__restrict__ c_out,
                                                       const int32_t *__restrict__ c0_in,
                                                       int32_t *__restrict__ c0_out) {
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < ld;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const bool in = i < np;
        const int64_t j = in ? static_cast<int64_t>(idx[i]) : 0;
        for (int m = 0; m < nm; ++m) {
            g_out[m * ld + i] = in ? g_in[m * ld + j] : T(0);
            c_out[m * ld + i] = in ? c_in[m * ld + j] : -1;
        }
        c0_out[i] = in ? c0_in[j] : -1;
    }
}

// ---- transport ----------------------------------------------------------
// Linearisation at f0: per entry W_dp = K g2 [da (N + 1 - f0_d) + de (N + f0_d)]
// is stored; 1/tau_d = K sum g2 [da (N + f0_p) + de (N + 1 - f0_p)].
template <typename T, bool FUSED>
__global__ __launch_bounds__(512) void k_transport_setup(Tables<T> P, const T *__restrict__ f0,
                                                         T *__restrict__ W, T *__restrict__ part,
                                                         T *__restrict__ tau_inv) {
    const int64_t c = chunk_of_block(P.n_chunks, P.xcd_m);
    if (c >= P.n_chunks) return;
    const int d = P.chunk_dest[c];
    const int64_t beg = P.chunk_beg[c], end = P.chunk_beg[c + 1];
    const StateRec<T> sd = P.st[d];
    const T fd = f0[d];
    T acc[1] = {T(0)};
    for (int64_t e = beg + threadIdx.x; e < end; e += blockDim.x) {
        const uint32_t pn = P.pnu[e];
        const T g = P.g2[e];
        const int p = static_cast<int>(pn >> 3);
        const StateRec<T> sp = P.st[p];
        const T fp = f0[p];
        EntryCoef<T> k = entry_coef(P, sd.eps, sd.kq, pn, sp);
        // ah = N(da+de) + de, bh = N(da+de) + da
        // W  = g [ (N(da+de) + da) - f0_d (da - de) ]  = g [bh - f0_d (da - de)]
        // out= g [ (N(da+de) + de) + f0_p (da - de) ]  = g [ah + f0_p (da - de)]
        const T dd = k.bh - k.ah;   // da - de
        W[e] = P.K * g * (k.bh - fd * dd);
        acc[0] += g * (k.ah + fp * dd);
    }
    block_sum<T, 1>(acc);
    if (threadIdx.x == 0) {
        if (FUSED) tau_inv[d] = P.K * acc[0];
        else part[c] = acc[0];
    }
}

template <typename T>
__global__ void k_transport_setup_finish(Tables<T> P, const T *__restrict__ part,
                                         T *__restrict__ tau_inv) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= P.S) return;
    T a = T(0);
    for (int c = P.dest_chunk[d]; c < P.dest_chunk[d + 1]; ++c) a += part[c];
    tau_inv[d] = P.K * a;
}

}  // namespace ephbte
