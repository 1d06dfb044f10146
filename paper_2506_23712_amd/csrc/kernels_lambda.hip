// kernels_lambda.hip -- a lambda density from samples of its characteristic
// function exp(K(i omega; Z)): the cumulant generating function at imaginary
// argument, inverted by a discrete Fourier transform.
#include "ens_lambda.h"

namespace ens {

// One wave per output sample j, its lanes striding over the terms k, summed
// lane by lane in increasing k and then over the lanes in a fixed butterfly
// (deterministic).  The term k is psi_k w^(k j mod M), psi_k = phi_k
// e^(-i omega_k lam0), w = e^(-2 pi i / M).  The sum is bound by FP64 arithmetic:
// psi is formed once per workgroup of kWaves samples (a sincos per term, shared
// through LDS) and w^m is the product of two LDS table entries, w^(256 h) and
// w^l with m = 256 h + l (k j is reduced mod M in integers, so both angles are
// exact multiples of 2 pi / M), where a sincos per (j, k) pair by one thread per
// sample took 1472 us at M = 4096 (16 workgroups) against 21 us.  Two workgroups
// on a compute unit (64 registers): with one, M = 16384 takes 281 us instead of 250.
constexpr int kWaves = 16, kChunk = 1024, kLo = 256;

__global__ void __launch_bounds__(64 * kWaves, 8) k_cf_invert(const double2 *__restrict__ phi, int M, double lam0, double h,
                                                           double *__restrict__ pdf) {
    __shared__ double2 psi[kChunk];
    __shared__ double2 lo[kLo], hi[kMaxCfTable / kLo];
    __shared__ int apart;
    const double two_pi = 6.283185307179586476925286766559;
    const int tid = threadIdx.x, lane = tid & 63, j = blockIdx.x * kWaves + (tid >> 6);
    for (int i = tid; i < kLo + (M + kLo - 1) / kLo; i += 64 * kWaves) {
        const int m = i < kLo ? i : (i - kLo) * kLo;
        double sn, cs;
        sincos(-two_pi * (double)m / (double)M, &sn, &cs);
        (i < kLo ? lo[i] : hi[i - kLo]) = double2{cs, sn};
    }
    // k j mod M of the wave's terms: k = lane + 64 i
    const int jj = j < M ? j : 0;
    int m = (int)(((long long)lane * jj) % M);
    const int step = (int)((64ll * jj) % M);
    double acc = 0.0;
    if (tid == 0) apart = 0;
    for (int k0 = 0; k0 < M; k0 += kChunk) {
        __syncthreads();
        const int kt = k0 + tid;
        if (kt < M) {
            const int f = kt < M / 2 ? kt : kt - M;                // frequency index
            const double omega = two_pi * (double)f / ((double)M * h);
            double sn, cs;
            sincos(-(omega * lam0), &sn, &cs);
            const double2 p = phi[kt];
            const double2 q = double2{p.x * cs - p.y * sn, p.x * sn + p.y * cs};
            psi[tid] = q;
            if (!isfinite(q.x) || !isfinite(q.y)) apart = 1;
        }
        __syncthreads();
        const int n = M - k0 < kChunk ? M - k0 : kChunk;
        for (int k = lane; k < n; k += 64) {
            const double2 p = psi[k], a = hi[m / kLo], b = lo[m % kLo];
            acc = fma(p.x, a.x * b.x - a.y * b.y, acc);
            acc = fma(-p.y, a.x * b.y + a.y * b.x, acc);
            m += step;
            m -= m >= M ? M : 0;
        }
    }
    // An infinity or NaN among the phi_k (or an overflow of psi_k) turns both
    // parts of psi_k, and with them every sample, into NaN: the sum is then
    // taken again, each term as phi_k times its whole phase factor.
    if (apart) {                                               // uniform over the workgroup
        acc = 0.0;
        for (int k = lane; k < M; k += 64) {
            const int f = k < M / 2 ? k : k - M;
            const double omega = two_pi * (double)f / ((double)M * h);
            double sn, cs;
            sincos(-(omega * lam0) - two_pi * (double)(((long long)k * jj) % M) / (double)M, &sn, &cs);
            const double2 p = phi[k];
            acc += p.x * cs - p.y * sn;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0 && j < M) pdf[j] = acc / ((double)M * h);
}

hipError_t launch_cf_invert(const double *phi, int M, double lam0, double h, double *pdf, hipStream_t s) {
    if (M < 2 || M > kMaxCfTable || !(h > 0) || !phi || !pdf) return hipErrorInvalidValue;
    k_cf_invert<<<(M + kWaves - 1) / kWaves, 64 * kWaves, 0, s>>>(reinterpret_cast<const double2 *>(phi), M, lam0, h, pdf);
    return hipGetLastError();
}

}  // namespace ens
