// step_common.hpp -- what the kernels of a Runge-Kutta stage share: pass
// configurations, truncated loads, the band step and FP64 block sums.
#pragma once

#include "ens_internal.h"
#include "fft.hpp"
#include "gmem.hpp"

namespace ens {

__device__ __forceinline__ int mode_of(int n, int N) { return n <= N / 2 ? n : n - N; }

// FP64 sum over the first NT threads (a power of two) of a workgroup with a
// fixed combination order (deterministic); every thread calls it.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double *red) {
    if ((int)threadIdx.x < NT) red[threadIdx.x] = v;
    __syncthreads();
#pragma unroll
    for (int s = NT / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    double r = red[0];
    __syncthreads();
    return r;
}

// Whether a z plane's six y-physical fields fit one workgroup's LDS in both
// precisions (135 KB for N = 64 in FP64): the plane pass exists for these N.
constexpr bool plane_ok(int N) { return N <= 64; }

// The x-pass variant whose kernel `variant` runs at grid size n: itself, or the
// one that stands for it where it has no kernel of its own.  Lines of n < 64 are
// too short to stream.  Streamed with 16 values per thread (one LDS
// exchange per 256-point transform) in FP32 only: FP64 would need more than 256
// registers.
constexpr int xpass_kernel(int n, bool fp32, int variant) {
    if (variant == 5 && plane_ok(n)) return 5;
    if (variant >= 4) return n >= 64 ? 6 : 0;                   // wave-private, pairs staged through two buffers
    if (variant == 3) return fp32 && n >= 128 && n <= 512 ? 3 : xpass_kernel(n, fp32, 2);
    if (variant == 2) return n >= 64 ? 2 : 0;
    return variant;
}

// ------------------------------------------------------------ pass configs
// E = complex values per thread (a line of N uses N/E threads).  Variants of
// E are compiled for the pencil passes and the x pass; the host picks one per
// (pass, N, precision) from its tuning table.
template <typename P, int N, int E_, int TM = 1> struct Cfg {
    static constexpr int K = N / 3, KX = K + 1;                 // x-modes kept
    static constexpr int NZLS = (2 * K + 1) * KX;               // z-lines: modes of a z plane
    static constexpr int ZP = state_pitch(K, (int)sizeof(Cx<P>));  // plane pitch (whole 128-byte lines)
    static constexpr int S = (2 * K + 1) * ZP;                  // state elements per component
    static constexpr int NYL = N * KX;                          // y-lines
    // y-pencil buffers are blocked by z: ZB consecutive z rows (BL = ZB (K+1)
    // lines, the fewest that fill whole 128-byte lines) are stored together,
    // position by position, so that a pass's position stride is BL values
    // (5.5 KB at N = 256) instead of the whole y-line count
    static constexpr int TLB = 128 / (int)sizeof(Cx<P>);
    static constexpr int ZB = TLB / gcd_int(KX, TLB), BL = ZB * KX;
    // element of line L at position p of a y-pencil buffer with NP positions
    __device__ static constexpr uint32_t yel(int L, int p, int NP) {
        return (uint32_t)(L / BL) * (uint32_t)(NP * BL) + (uint32_t)p * BL + (uint32_t)(L % BL);
    }
    static constexpr int E = E_ > N ? N : E_;
    static constexpr int M = N / E;
    // Lines per workgroup of the y/z pencil passes: at least 256 threads (128 for
    // N <= 64, whose members have few lines) and
    // at least one 128-byte line per position (16 FP32 / 8 FP64 consecutive
    // lines, a multiple of which is where every tile starts), so that every
    // store covers whole lines; at most 1024 threads (512
    // with 16 values per thread, so that a wave may use 256 VGPRs); gfx950
    // gives a workgroup up to 160 KiB of LDS.
    static constexpr int TL = 128 / (int)sizeof(Cx<P>);
    static constexpr int MAXT = E >= 16 ? 512 : 1024;             // 16 values/thread: keep 256 VGPRs available
    // TM > 1 (autotuner variants 2, 3 of the y/z passes): TM times as many
    // lines, i.e. TM whole lines per position, where the thread budget above
    // allows it (not for 16 FP64 values per thread, which would spill)
    static constexpr int T1 = N <= 64 ? (128 / M > TL ? 128 / M : TL) : N <= 256 ? (256 / M > TL ? 256 / M : TL) : (TL * M <= MAXT ? TL : MAXT / M);
    static constexpr int T = (T1 * TM * M <= MAXT && !(sizeof(P) == 8 && E >= 16)) ? T1 * TM : T1;
    static constexpr int NT = T * M;
    // z/y inverse passes: waves per SIMD the register budget is cut for
    static constexpr int PMINW = (sizeof(P) == 4 && E == 16 && NT == 256) ? 3 : 1;
    static constexpr int TX = 256 / M;                          // x pass: 256 threads
    // y-pencils of the z forward's input stored plane by plane ([3][N (z)][ZP],
    // as the z inverse's output) instead of in blocks of z: where the plane pass
    // writes them (it owns a plane, so a plane's values are contiguous)
    static constexpr bool PLN = plane_ok(N);
    // z forward + update: one 128-byte line per position from N = 128, the
    // smallest workgroup that stores whole lines: its phases (loads, transforms,
    // update, transforms) are apart by barriers, and several small workgroups on
    // a compute unit overlap them where one of 512 threads per compute unit
    // (FP64) had nothing beside it.  us a step against 512 threads: eight 128^3
    // FP64 members 521 -> 468, one 256^3 FP64 member 525 -> 484, six 128^3 FP32
    // members 196 -> 191; N = 512 with 8 values (16: 212 registers FP32, one wave
    // per SIMD in FP64): 2370 -> 2238 FP32, 4730 -> 4350 FP64.  At least 128
    // threads for N <= 64, whose members have few lines (15 workgroups of 512
    // threads for a 64^3 member, 2 for a 32^3 one, on 256 compute units).
    // Values per thread: 8; 4 for N <= 64, where a wave's own instructions are
    // the time (us a step, one 32^3 FP64 member 37 -> 29, nine 64^3 FP64 members
    // 88 -> 76, 47 of 64^3 FP32 equal; against 512 threads with 8 values: 56 / 29,
    // 74 / 76, 199 / 190), and in FP64 at N = 128 (eight members 468
    // -> 454; FP32 191 -> 199; FP64 at N = 256 484 -> 567); 16 at N = 1024.
    static constexpr int EZ = N <= 64 || (sizeof(P) == 8 && N == 128) ? 4 : N <= 512 ? 8 : 16, MZ = N / EZ;
    static constexpr int TZ = N <= 64 ? (128 / MZ > TL ? 128 / MZ : TL) : N <= 512 ? TL : 512 / MZ;
    static constexpr int NTZ = TZ * MZ;
    // z forward + update, waves per SIMD the register budget is cut for
    static constexpr int ZMINB = N <= 64 || N == 1024 ? 1 : sizeof(P) == 4 ? 4 : 2;
};

// -------------------------------------------------------------------- band
// One workgroup per member: the band's part of the m_x = 0 plane made
// Hermitian, then E_f over the forcing band (FP64, fixed order).  NB of the
// workgroup's threads work (a power of two); all of them call it.
template <typename P, int NB>
__device__ __forceinline__ void band_energy(const MemberDev &md, int stage, double *red) {
    const bool on = (int)threadIdx.x < NB;
    const int K = md.K;
    const long long zp = md.zp;
    const long long S = (long long)(2 * K + 1) * zp;
    int B = (int)floor(sqrt(md.kf_hi2));
    if (B > K) B = K;
    const int W = 2 * B + 1;
    const long long ncand = (long long)(B + 1) * W * W;
    // The velocity is real, so the m_x = 0 plane of its half spectrum is
    // Hermitian: u(0, -m_y, -m_z) = conj u(0, m_y, m_z).  A part breaking
    // that is invisible to the nonlinear term, and the linear forcing would
    // amplify it in the band; the band's part of the plane is made Hermitian
    // here (one thread per pair) before E_f is summed.
    for (int c = on ? (int)threadIdx.x : W * W; c < W * W; c += NB) {
        const int my = c % W - B, mz = c / W - B;
        const int m2 = my * my + mz * mz;
        if (!(mz > 0 || (mz == 0 && my > 0)) || (double)m2 < md.kf_lo2 || (double)m2 > md.kf_hi2) continue;
        const int iy = my >= 0 ? my : my + 2 * K + 1, iz = mz;
        const int jy = my > 0 ? 2 * K + 1 - my : -my, jz = mz > 0 ? 2 * K + 1 - mz : 0;
        const uint32_t i1 = (uint32_t)((long long)iz * zp + (long long)iy * (K + 1));
        const uint32_t i2 = (uint32_t)((long long)jz * zp + (long long)jy * (K + 1));
#pragma unroll
        for (int comp = 0; comp < 3; comp++) {
            const Fld<P> F(md.uh, comp * S);
            const Cx<P> a = F.ld(i1), b = F.ld(i2);
            const Cx<P> h = {P(0.5) * (a.re + b.re), P(0.5) * (a.im - b.im)};
            F.st(i1, h);
            F.st(i2, {h.re, -h.im});
        }
    }
    __syncthreads();
    double acc = 0.0;
    for (long long c = on ? (long long)threadIdx.x : ncand; c < ncand; c += NB) {
        const int mx = (int)(c % (B + 1));
        const int my = (int)((c / (B + 1)) % W) - B;
        const int mz = (int)(c / ((long long)(B + 1) * W)) - B;
        const int m2 = mx * mx + my * my + mz * mz;
        if (m2 == 0 || (double)m2 < md.kf_lo2 || (double)m2 > md.kf_hi2) continue;
        const int iy = my >= 0 ? my : my + 2 * K + 1, iz = mz >= 0 ? mz : mz + 2 * K + 1;
        const long long idx = (long long)iz * zp + (long long)iy * (K + 1) + mx;
        const double w = mx > 0 ? 1.0 : 0.5;
#pragma unroll
        for (int comp = 0; comp < 3; comp++) {
            Cx<P> v = Fld<P>(md.uh, comp * S).ld((uint32_t)idx);
            acc += w * ((double)v.re * (double)v.re + (double)v.im * (double)v.im);
        }
    }
    const double ef = block_sum<NB>(acc, red);
    if (threadIdx.x == 0) {
        // A band holding no more than kForceEmptyFrac of the energy the field
        // had at the start of the step (diag.E) is empty: the linear forcing,
        // eps/(2 E_f) u, would otherwise amplify rounding-level band modes to
        // inject eps.  Ef = 0 tells the update to add no forcing.
        const bool forced = ef > kForceEmptyFrac * md.st->diag.E;
        md.st->Ef = forced ? ef : 0.0;
        if (stage == 0) {
            md.st->diag.E_f = ef;
            md.st->diag.inj = forced ? md.eps_m : 0.0;
            if (!forced && md.eps_m != 0.0) md.st->diag.flags |= 2;
        }
    }
}

}  // namespace ens
