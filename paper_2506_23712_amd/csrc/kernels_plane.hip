// kernels_plane.hip -- the plane pass of a Runge-Kutta stage: y inverse, x pass
// and y forward of a z plane held in one workgroup's LDS.
#include "step_common.hpp"

namespace ens {

// ================================================================== plane pass
// y inverse, x pass and y forward of one z plane by one workgroup, for the N
// whose six y-physical fields of a plane fit its LDS (plane_ok): the plane's
// spectral fields are read once and its nonlinear term written once, and a
// stage has one launch for three passes and the band step.  The three passes
// move 5 zl + 6 yl, 9 yl and 3 yl + 3 zl values per member (zl = 2/3 yl) and,
// at these N, are launches of 5 to 10 us whatever they move; here 8 zl values.
// FP32: 1725 vector instructions per wave (the arithmetic of 8.1 transforms a
// thread) keep the VALU active in 50 % of the launch's cycles and the LDS in 25 %
// (12 members of 64^3).  FP64: VALU 28 %, LDS 30 % (28 % of that bank conflicts),
// the waves waiting in half of their cycles: one workgroup of 8 waves on a compute
// unit, whose phases are apart by barriers, and 585 workgroups (nine 64^3
// members) are 2.3 rounds of 256.  For few members the latency of the phases is
// the time.  Per RK step, before and now: one 32^3 FP64 member with its state read
// back 143 -> 66 us, five 64^3 FP32 members 196 -> 114 us, nine 64^3 FP64 members
// (profiled launches, y inverse, x pass, y forward and band step) 228 -> 161 us, 47
// of 64^3 FP32 528 -> 321 us.
//
// The plane lives in LDS as rows (f, kx) of N y positions.  Phase 1, one row per
// group of M = N/8 or N/4 lanes: the row's spectral line (the vorticity's formed on
// load), inverse transform inside the row.  Phase 2, one y per group: the 3
// pairs of fields inverse transformed along x, n = u x omega, forward, the
// exchanges in the group's own column of the plane (the fields it has read).
// Phase 3, one row per group: forward along y, staged in mode order and stored
// as one contiguous run per field.  A group's lanes are in one wave, so that
// only the changes of phase need a workgroup barrier.  LDS places: position p
// of a row is XOR-ed with p / 8 in its low three bits, and the FP32 rows are 8
// values (half the banks) out of step, so that lanes at stride 8 and at stride
// 1 along a row, and lanes along a column, spread over all banks.
// The workgroup after the last plane performs the member's band step, which
// needs only the velocity, and which only the z forward waits for.
template <typename P, int N> struct PlaneCfg {
    static constexpr int K = N / 3, KX = K + 1, E = N == 16 || (N == 32 && sizeof(P) == 4) ? 4 : 8, M = N / E;
    static constexpr int ROWS = 6 * KX, NP = (2 * K + 1) * KX;
    static constexpr int PITCH = sizeof(P) == 4 ? N + 8 : N;
    // N = 64: 64 groups of 8 lanes take the 132, 64 and 66 lines of the phases
    // in 2, 1 and 1 rounds and a rest that one wave takes (8 waves, so that FP32
    // has two workgroups on a compute unit at 128 registers and FP64 256 registers);
    // N = 32: 72 groups of 8 in FP32 (4 values per thread: 109 -> 104 us a step
    // for 50 members; FP64 has no gain) or 80 of 4 (66, 32, 33 lines), N = 16: 48
    // of 4 (36, 16, 18)
    static constexpr int NT = N == 64 ? 512 : N == 32 ? (E == 4 ? 576 : 320) : 192, G = NT / M;
    static constexpr int MINW = N == 64 ? (sizeof(P) == 4 ? 4 : 2) : 1;   // waves per SIMD
    static constexpr int RPW = 64 / M;                         // columns of a wave in phase 2
    // FP64: each thread's twiddles in registers (a table in LDS is read at
    // strides that share banks, and its registers are free: the LDS admits one
    // workgroup per compute unit); FP32: in LDS (registers are what bound its
    // workgroups per compute unit)
    static constexpr bool REGTW = sizeof(P) == 8;
    static constexpr int NB = NT >= 256 ? 256 : 128;           // threads of the band step
    __device__ static __forceinline__ int sw(int p) { return p ^ ((p >> 3) & 7); }
    struct Row {                                               // exchange inside row l
        __device__ static __forceinline__ int slot(int p, int l) { return l * PITCH + sw(p); }
    };
    struct Col {                                               // exchange inside column l
        __device__ static __forceinline__ int slot(int p, int l) { return (p ^ ((p >> 3) & 1)) * PITCH + sw(l); }
    };
    static_assert(N % RPW == 0 && N / RPW <= NT / 64 && 2 * K + 1 <= PITCH && N <= 3 * KX, "plane shape");
};

template <typename P, int N>
__global__ void __launch_bounds__((PlaneCfg<P, N>::NT), (PlaneCfg<P, N>::MINW)) k_plane(const MemberDev *__restrict__ mems, const Cx<P> *__restrict__ twg, int stage) {
    using C = PlaneCfg<P, N>;
    using Row = typename C::Row;
    using Col = typename C::Col;
    constexpr int E = C::E, M = C::M, K = C::K, KX = C::KX, NT = C::NT, ZP = Cfg<P, N, 8>::ZP;
    constexpr unsigned ZM = truncated_slots(N, E, K);
    __shared__ __attribute__((aligned(16))) LdsT<P> pl[C::ROWS * C::PITCH];
    __shared__ Cx<P> twl[C::REGTW ? 1 : twiddle_span(N, E)];
    TwRegs<P, N, E> twr;
    const auto &tw = [&]() -> const auto & {
        if constexpr (C::REGTW) return twr;
        else return twl;
    }();
    unsigned tile, mem_i;
    xcd_tile(tile, mem_i);
    const MemberDev &md = mems[mem_i];
    if (tile == N) {                                           // uniform over the workgroup
        band_energy<P, C::NB>(md, stage, reinterpret_cast<double *>(pl));
        return;
    }
    const int z = (int)tile, tid = (int)threadIdx.x;
    const P dk = (P)md.dk;
    if constexpr (C::REGTW) twr.load(twg, tid % M);
    else for (int i = tid; i < twiddle_span(N, E); i += NT) twl[i] = twg[i];
    // ---- phase 1: y inverse of row r = (f, kx), f = u_x, u_y, u_z, omega_x, omega_y, omega_z
    {
        const int t = tid % M;
        constexpr int RD = (C::ROWS + C::G - 1) / C::G;
        auto load = [&](Cx<P> *v, int rd) {
            const int r = tid / M + rd * C::G;
            if (r >= C::ROWS) return;
            const int f = r / KX, kx = r % KX;
            // omega_x = i k_y u_z - W_y, omega_y = W_x - i k_x u_z, omega_z = i k_x u_y - i k_y u_x
            const int fa = f < 3 ? f : (f == 3 ? 2 : (f == 4 ? 3 : 1)), fb = f == 3 ? 4 : (f == 4 ? 2 : 0);
            const Fld<P> A(md.bufA, ((long long)fa * N + z) * ZP), B(md.bufA, ((long long)fb * N + z) * ZP);
            const P kxv = dk * (P)kx;
#pragma unroll
            for (int m = 0; m < E; m++) {
                const int my = mode_of(t + M * m, N);
                v[m] = czero<P>();
                if (my < -K || my > K) continue;
                const uint32_t at = (uint32_t)((my >= 0 ? my : my + 2 * K + 1) * KX + kx);
                const P kyv = dk * (P)my;
                Cx<P> x = A.ld(at);
                if (f >= 3) {
                    const Cx<P> b = B.ld(at);
                    if (f == 3) x = mul_i(cscale(x, kyv)) - b;
                    else if (f == 4) x = x - mul_i(cscale(b, kxv));
                    else x = mul_i(cscale(x, kxv)) - mul_i(cscale(b, kyv));
                }
                v[m] = x;
            }
        };
        auto transform = [&](Cx<P> *v, int rd) {
            const int r = tid / M + rd * C::G;
            if (r >= C::ROWS) return;
            line_fft<P, N, E, 1, +1, 2, Row, ZM>(v, pl, r, t, tw);
            wave_fence();
#pragma unroll
            for (int s = 0; s < E; s++) lds_put<P>(pl, Row::slot(Plan<N, E>::out_pos(t, s), r), v[s]);
        };
        // FP32: the loads of two rounds first; FP64: of one (registers)
        constexpr int PR = sizeof(P) == 4 && RD > 1 ? 2 : 1;
        Cx<P> v[PR][E];
#pragma unroll
        for (int rd = 0; rd < PR; rd++) load(v[rd], rd);
        if constexpr (!C::REGTW) __syncthreads();              // twiddles
#pragma unroll
        for (int rd = 0; rd < RD; rd++) {
            if (rd >= PR) load(v[rd % PR], rd);
            transform(v[rd % PR], rd);
        }
    }
    __syncthreads();
    // ---- phase 2: x inverse of the field pairs, u x omega, x forward of column y
    {
        const int lane = tid & 63, wave = tid >> 6;
        const int y = wave * C::RPW + lane % C::RPW, t = lane / C::RPW;
        if constexpr (C::REGTW) twr.load(twg, t);
        if (y < N) {                                           // whole waves
            // packed two-for-one spectrum of fields 2 pr, 2 pr + 1: C = A + i B, Hermitian fill
            auto gather = [&](Cx<P> *v, int pr) {
#pragma unroll
                for (int m = 0; m < E; m++) {
                    const int n = t + M * m;
                    const bool lo = n <= K, hi = n >= N - K;
                    const int kx = lo ? n : N - n;
                    Cx<P> A = czero<P>(), B = czero<P>();
                    if (lo || hi) {
                        A = lds_get<P>(pl, Row::slot(y, 2 * pr * KX + kx));
                        B = lds_get<P>(pl, Row::slot(y, (2 * pr + 1) * KX + kx));
                    }
                    if (n == 0) v[m] = {A.re, B.re};
                    else if (lo) v[m] = {A.re - B.im, A.im + B.re};
                    else v[m] = {A.re + B.im, B.re - A.im};
                }
            };
            // the exchanges use rows 0 .. N - 1 of the column, i.e. fields 0 to
            // 2, so the first two pairs are read before the first transform
            P ph[6][E];
            Cx<P> v[E], w[E];
            gather(v, 0);
            gather(w, 1);
            wave_fence();
            line_fft<P, N, E, 1, +1, 2, Col, ZM>(v, pl, y, t, tw);
#pragma unroll
            for (int s = 0; s < E; s++) { ph[0][s] = v[s].re; ph[1][s] = v[s].im; }
            gather(v, 2);
            wave_fence();
            line_fft<P, N, E, 1, +1, 2, Col, ZM>(w, pl, y, t, tw);
#pragma unroll
            for (int s = 0; s < E; s++) { ph[2][s] = w[s].re; ph[3][s] = w[s].im; }
            line_fft<P, N, E, 1, +1, 2, Col, ZM>(v, pl, y, t, tw);
#pragma unroll
            for (int s = 0; s < E; s++) { ph[4][s] = v[s].re; ph[5][s] = v[s].im; }
            // ph: 0 u_x, 1 u_y, 2 u_z, 3 omega_x, 4 omega_y, 5 omega_z
            if (stage == 0) {
                P mx = P(0);
#pragma unroll
                for (int s = 0; s < E; s++) {
                    const P a = fabs(ph[0][s]) + fabs(ph[1][s]) + fabs(ph[2][s]);
                    mx = a > mx ? a : mx;
                }
                double dm = (double)mx;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    const double o = __shfl_xor(dm, off, 64);
                    dm = o > dm ? o : dm;
                }
                if (lane == 0) atomicMax(&md.st->umax_bits, (unsigned long long)__double_as_longlong(dm));
            }
            Cx<P> d1[E], d2[E];
#pragma unroll
            for (int s = 0; s < E; s++) {
                d1[s] = {ph[1][s] * ph[5][s] - ph[2][s] * ph[4][s], ph[2][s] * ph[3][s] - ph[0][s] * ph[5][s]};
                d2[s] = {ph[0][s] * ph[4][s] - ph[1][s] * ph[3][s], P(0)};
            }
            line_fft_T<P, N, E, 1, -1, 2, Col>(d1, pl, y, t, tw);      // d1[m] = D1[t + M m]
            line_fft_T<P, N, E, 1, -1, 2, Col>(d2, pl, y, t, tw);
            wave_fence();
#pragma unroll
            for (int m = 0; m < E; m++)          // the split reads only the partner positions 0 and >= N - K
                if (m == 0 || M * m + M - 1 >= N - K) lds_put<P>(pl, Col::slot(t + M * m, y), d1[m]);
            wave_fence();
            // split D1 into the x-spectra of n_x and n_y
            Cx<P> ox[E], oy[E];
#pragma unroll
            for (int m = 0; m < E; m++) {
                const int k = t + M * m;
                if (M * m <= K && k <= K) {
                    const Cx<P> a = d1[m];
                    const Cx<P> b = lds_get<P>(pl, Col::slot((N - k) % N, y));
                    const P h = P(0.5);
                    ox[m] = {h * (a.re + b.re), h * (a.im - b.im)};
                    oy[m] = {h * (a.im + b.im), h * (b.re - a.re)};
                }
            }
            wave_fence();
#pragma unroll
            for (int m = 0; m < E; m++) {
                const int k = t + M * m;
                if (M * m <= K && k <= K) {
                    lds_put<P>(pl, Row::slot(y, k), ox[m]);
                    lds_put<P>(pl, Row::slot(y, KX + k), oy[m]);
                    lds_put<P>(pl, Row::slot(y, 2 * KX + k), d2[m]);
                }
            }
        }
    }
    __syncthreads();
    // ---- phase 3: y forward of row r = (f, kx), f = n_x, n_y, n_z, staged as [f][m_y][kx]
    LdsT<P> *stg = pl + 3 * KX * C::PITCH;
    {
        const int t = tid % M;
        if constexpr (C::REGTW) twr.load(twg, t);
        for (int r = tid / M; r < 3 * KX; r += C::G) {
            Cx<P> v[E];
#pragma unroll
            for (int m = 0; m < E; m++) v[m] = lds_get<P>(pl, Row::slot(t + M * m, r));
            wave_fence();
            line_fft<P, N, E, 1, -1, 2, Row>(v, pl, r, t, tw);
            const int f = r / KX, kx = r % KX;
#pragma unroll
            for (int s = 0; s < E; s++) {
                const int my = mode_of(Plan<N, E>::out_pos(t, s), N);
                if (my >= -K && my <= K) lds_put<P>(stg, f * C::NP + (my >= 0 ? my : my + 2 * K + 1) * KX + kx, v[s]);
            }
        }
    }
    __syncthreads();
    for (int e = tid; e < 3 * C::NP; e += NT) {
        const int f = e / C::NP;
        Fld<P>(md.bufB, ((long long)f * N + z) * ZP).st((uint32_t)(e - f * C::NP), lds_get<P>(stg, e));
    }
}

template <typename P, int N>
static hipError_t plane_n(const MemberDev *mem, int count, int stage, bool band, const void *tw, hipStream_t s) {
    k_plane<P, N><<<dim3(N + (band ? 1 : 0), count), PlaneCfg<P, N>::NT, 0, s>>>(mem, reinterpret_cast<const Cx<P> *>(tw), stage);
    return hipGetLastError();
}

template <typename P>
static hipError_t plane_p(int n, const MemberDev *mem, int count, int stage, bool band, const void *tw, hipStream_t s) {
    switch (n) {
    case 16: return plane_n<P, 16>(mem, count, stage, band, tw, s);
    case 32: return plane_n<P, 32>(mem, count, stage, band, tw, s);
    case 64: return plane_n<P, 64>(mem, count, stage, band, tw, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_plane(int n, int prec, const MemberDev *mem, int count, int stage, bool band, const void *tw, hipStream_t s) {
    return prec == ENS_FP32 ? plane_p<float>(n, mem, count, stage, band, tw, s)
                            : plane_p<double>(n, mem, count, stage, band, tw, s);
}

}  // namespace ens
