// Weight gradient and update of fully-connected layers with few weights and
// few samples (Algorithm 1, g(l) = a(l-1) (x) e(l), w <- w - g; Section 3.3):
// classifier heads and the layers of small networks.
//
//   g32[k][c] = sum over samples i of dy[i][k] * x[i][c]
//
// Such a layer is bound by latency: one memory round trip per launch and the
// launches themselves.  A workgroup owns a 32 x 32 tile of g32 and its eight
// waves take interleaved slices of 32 samples, every load of a slice in
// flight at once, straight into MFMA operand registers; the partial tiles
// meet in LDS.  The contraction is so short that it is cheaper to run it
// twice than to pass g32 through memory and two more kernels: the first
// launch only folds the tile maxima into the tensor maximum, the second forms
// the tile again, rounds it with the now known shift and updates the weights
// (784 -> 128, 32 samples: 12.8 us in three launches before, 7.6 us in two).
// A caller that asks for g32 gets it from the first launch.
//
// Each lane's 16 operand bytes are one column over 16 samples, so they are
// gathered byte by byte (any channel count, any alignment): a wave's 64 byte
// loads cover two runs of 32 consecutive bytes.
#include "niti_internal.h"

namespace niti {

namespace {

constexpr int SW = 8;            // waves per workgroup (sample slices)
constexpr int ST = SW * 64;
constexpr int RP = 36;           // LDS row pitch of a partial tile (ints; 16-byte aligned)
constexpr int kMaxPix = 1024;    // eligibility: at most this many samples

// 16 samples from p of column col (both in range after clamping), zero for
// samples at or past n or when col_ok is false.
__device__ __forceinline__ v4i gather16(const int8_t* base, int pitch, int col, bool col_ok, int p, int n) {
    uint32_t b[16];
#pragma unroll
    for (int i = 0; i < 16; i++) b[i] = (uint8_t)base[(int64_t)min(p + i, n - 1) * pitch + col];
    v4i r;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        uint32_t w = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) w |= (p + 4 * q + i < n ? b[4 * q + i] : 0u) << (8 * i);
        r[q] = col_ok ? (int)w : 0;
    }
    return r;
}

// FINISH < 0: fold the tile maximum in (and store g32 when P.part is given);
// otherwise round in mode FINISH with the call's shift and update w.
template <int FINISH>
__global__ __launch_bounds__(ST) void wgrad_small_kernel(WgradProblem P, int8_t* w, niti_stats* st, int mu,
                                                         uint32_t static_flags, int tiles_c) {
    __shared__ __attribute__((aligned(16))) int32_t red[SW * 32 * RP];
    __shared__ uint32_t wmax[SW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = (int)(blockIdx.x % (uint32_t)tiles_c) * 32, k0 = (int)(blockIdx.x / (uint32_t)tiles_c) * 32;
    int slot = 0;
    RoundK rk{};
    if (FINISH >= 0) {
        rk = make_round(block_bp(shared_call_state(st).mx, mu), FINISH);
        sr_key_recorded(rk, st);
    } else {
        slot = call_slot(st);
        begin_call(st, slot, -1);
    }
    const int r32 = lane & 31, half = (lane >> 5) * 16;
    const bool cok = c0 + r32 < P.C, kok = k0 + r32 < P.K;
    const int cc = min(c0 + r32, P.C - 1), kk = min(k0 + r32, P.K - 1);
    v16i acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0;
    for (int p0 = wave * 32; p0 < P.npix; p0 += SW * 32) {
        const v4i a = gather16(P.x, P.C, cc, cok, p0 + half, P.npix);
        const v4i b = gather16(P.dy, P.K, kk, kok, p0 + half, P.npix);
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc, 0, 0, 0);
    }
    // acc element 4*jj + i: column c0 + 8*jj + 4*(lane/32) + i, channel k0 + lane%32.
    int32_t* mine = red + (wave * 32 + r32) * RP + 4 * (lane >> 5);
#pragma unroll
    for (int jj = 0; jj < 4; jj++) *(v4i*)(mine + 8 * jj) = v4i{acc[4 * jj], acc[4 * jj + 1], acc[4 * jj + 2], acc[4 * jj + 3]};
    __syncthreads();
    uint32_t tmax = 0;
    if (threadIdx.x < 256) {
        const int row = threadIdx.x >> 3, c4 = (threadIdx.x & 7) * 4;
        const int k = k0 + row, c = c0 + c4;
        v4i s = *(const v4i*)(red + row * RP + c4);
#pragma unroll
        for (int v = 1; v < SW; v++) s += *(const v4i*)(red + (v * 32 + row) * RP + c4);
        if (k < P.K && c < P.C) {   // C % 4 == 0: the four columns are all valid
            const int64_t at = (int64_t)k * P.C + c;
            if (FINISH >= 0) {
                const int32_t g[4] = {s[0], s[1], s[2], s[3]};
                uint32_t* dst = (uint32_t*)(w + at);
                *dst = update_word<FINISH>(*dst, g, rk, (uint64_t)at);
            } else {
                if (P.part) *(int4*)(P.part + at) = make_int4(s[0], s[1], s[2], s[3]);
                tmax = max(max(mag32(s[0]), mag32(s[1])), max(mag32(s[2]), mag32(s[3])));
            }
        }
    }
    if (FINISH >= 0) {
        if (is_finisher()) finish_call(st, mu, ExpArgs{nullptr, nullptr, nullptr}, static_flags, 0);
    } else {
        const uint64_t snap = max_snapshot(st, slot);
        block_publish_max32(st, slot, tmax, wmax, snap);   // magnitudes <= 2^31
    }
}

}  // namespace

// Plain products (1 x 1 filter, no padding, no stride): x and dy are matrices
// with one row per sample.  The byte gathers issue 32 loads per MFMA, twice, so
// the launches saved pay for one tile per CU and no more where the LDS-staged
// DMA kernel can run (channels in whole 16s).  Whole calls in us, gathered /
// DMA kernel: 464 x 544 weights and 21 samples (255 tiles) 8.9 / 9.4; 1168 x
// 368, 53 samples (444 tiles) 15.0 / 9.5; 1264 x 512, 1003 samples (640) 26.7 /
// 17.5; 4352 x 224, 17 samples (952) 23.5 / 9.8.  The general kernel, which
// takes the other channel counts, gathers too and walks its samples in steps:
// 480 tiles and 105 samples 11.4 / 20.2, 594 tiles and 28 samples 16.3 / 15.3,
// 1000 tiles and 10 samples 25.0 / 16.2, 896 tiles and 167 samples 15.7 / 27.3.
bool wgrad_small_eligible(const WgradProblem& p) {
    if (p.win || p.R != 1 || p.S != 1 || p.sh != 1 || p.sw != 1 || p.ph != 0 || p.pw != 0) return false;
    if (p.H != p.P || p.W != p.Q || p.npix < 1 || p.npix > kMaxPix || p.C % 4 != 0) return false;
    const int64_t tiles = (int64_t)((p.C + 31) / 32) * ((p.K + 31) / 32);
    if (wgrad_dma_eligible(p)) return tiles <= 256;
    return tiles <= (p.npix >= 128 ? 1024 : 512);
}

hipError_t wgrad_small_run(WgradProblem& p, int8_t* w, int32_t* g32, int mu, int mode, niti_stats* st,
                           uint32_t static_flags, hipStream_t stream) {
    p.part = g32;
    const int tc = (p.C + 31) / 32, tk = (p.K + 31) / 32;
    int t = timing_on() ? timing_begin(NITI_TIMING_KERNEL, stream, kernel_label("wgrad_small_kernel<%d>", -1)) : -1;
    const dim3 grid(tc * tk), block(ST);
    hipLaunchKernelGGL(wgrad_small_kernel<-1>, grid, block, 0, stream, p, w, st, mu, static_flags, tc);
    timing_end(t, stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    t = timing_on() ? timing_begin(NITI_TIMING_KERNEL, stream, kernel_label("wgrad_small_kernel<%d>", mode)) : -1;
    if (mode == NITI_ROUND_SR)
        hipLaunchKernelGGL(wgrad_small_kernel<NITI_ROUND_SR>, grid, block, 0, stream, p, w, st, mu, static_flags, tc);
    else if (mode == NITI_ROUND_RTN)
        hipLaunchKernelGGL(wgrad_small_kernel<NITI_ROUND_RTN>, grid, block, 0, stream, p, w, st, mu, static_flags, tc);
    else
        hipLaunchKernelGGL(wgrad_small_kernel<NITI_ROUND_PSR>, grid, block, 0, stream, p, w, st, mu, static_flags, tc);
    timing_end(t, stream);
    return hipGetLastError();
}

}  // namespace niti
