// Matrix products with few outputs and a long reduction (Algorithm 1's
// forward and back-propagation contractions of a classifier head: a batch of
// a few hundred samples against a few hundred to a few thousand classes).
//
//   out[m][n] = round( sum_k  wgt[n][k] * act[m][k] ),  k < L
//
// With so few outputs a tiled kernel runs on a handful of CUs and each of
// them walks the reduction step by step, paying a memory round trip per
// step.  Here a workgroup owns one output tile of 32 channels and 32 or 64
// rows and its eight waves take interleaved 64-byte slices of the reduction:
// every wave issues all of its operand loads at once (straight into MFMA
// operand registers, no LDS staging), runs its MFMAs, and the eight partial
// tiles are added in LDS.  The 16 x 16 x 64 MFMA makes a load instruction read
// 64 consecutive bytes of 16 rows; the 32 x 32 x 32 one read 32 of 32 rows, and
// rows are far apart, so that each instruction touched twice as many cache
// lines for the same data.  The epilogue (optional ReLU, tensor maximum, shift-and-round,
// backward ReLU mask) and the exponent handling (rounding with a guessed
// shift, then a fix-up launch that recomputes on a miss) are those of the
// other implicit-GEMM kernels.
#include "niti_internal.h"

namespace niti {

namespace {

constexpr int SW = 8;                 // waves per workgroup (reduction slices)
constexpr int ST = SW * 64;           // threads per workgroup
constexpr int RP = 36;                // LDS row pitch of a partial tile (ints; 16-byte aligned)
constexpr int MAX_M = 1024;           // eligibility: at most this many output rows

// An operand's 16-byte piece is loaded from offset off, moved into the tensor
// where it would pass the end, without a branch, so that all pieces of a batch
// are in flight at once.  bytes >= 16.
__device__ __forceinline__ v4i piece_load(const int8_t* base, uint32_t off, uint32_t bytes) {
    return __builtin_bit_cast(v4i, load16_any(base + min(off, bytes - 16)));
}
// A piece of the last step: zeros past L and, where the load was moved, the
// bytes gathered singly.  Rows whose length is a multiple of 16 (WHOLE) need
// only the zeroing, earlier steps none of it.
template <bool WHOLE>
__device__ __forceinline__ v4i piece_cut(v4i v, const int8_t* base, uint32_t off, uint32_t bytes, int k, int L) {
    if (k >= L) return v4i{0, 0, 0, 0};
    if (!WHOLE && k + 16 > L) {
        if (off + 16 <= bytes) return __builtin_bit_cast(v4i, keep_bytes(__builtin_bit_cast(uint4, v), 0, L - k));
        const int n = min(16, L - k);
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        for (int i = 0; i < n; i++) w[i >> 2] |= (uint32_t)(uint8_t)base[off + i] << (8 * (i & 3));
        return v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
    }
    return v;
}

// One tile of 16 FM rows x 32 channels: reduce, add the slices, then (four
// consecutive channels of one row per thread) fold the maximum and store.
template <bool WHOLE, int FM>
__device__ __forceinline__ void small_tile(const IgemmProblem& P, int tile, int32_t* red, const RoundK& rk,
                                           int relu, bool do_store, bool do_max, uint32_t& tmax) {
    constexpr int FN = 2, ROWS = 16 * FM;
    // 64-byte reduction steps per wave and load batch, steps past the end
    // skipped.  Eight instead of five for 32 rows: 256 x 10 x 8192 16.5 -> 18.0
    // us, 176 x 48 x 4864 the same 14.5 (16.2 with four).
    constexpr int KB = FM == 2 ? 5 : 4;
    const int tiles_n = (P.Nout + 31) >> 5;
    const int tm = tile / tiles_n, tn = tile - tm * tiles_n;
    const int m0 = tm * ROWS, n0 = tn * 32;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, kh = (lane >> 4) * 16;
    const int L = P.L;
    // Operand rows of this lane.  Rows past the edge read the first one: what
    // they give is neither stored nor part of the maximum.
    uint32_t wrow[FN], arow[FM];
#pragma unroll
    for (int f = 0; f < FN; f++) {
        const int n = n0 + 16 * f + r16;
        wrow[f] = (uint32_t)(n < P.Nout ? n : 0) * (uint32_t)L;
    }
#pragma unroll
    for (int f = 0; f < FM; f++) {
        const int m = m0 + 16 * f + r16;
        arow[f] = (uint32_t)(m < P.M ? m : 0) * (uint32_t)L;
    }
    const uint32_t wbytes = (uint32_t)P.wgt_bytes, abytes = (uint32_t)P.act_bytes;

    v4i acc[FN][FM];
#pragma unroll
    for (int a = 0; a < FN; a++)
#pragma unroll
        for (int b = 0; b < FM; b++) acc[a][b] = v4i{0, 0, 0, 0};
    const int nks = (L + 63) >> 6;
    for (int ks0 = wave; ks0 < nks; ks0 += SW * KB) {
        v4i w[KB][FN], x[KB][FM];
#pragma unroll
        for (int j = 0; j < KB; j++) {
            if (ks0 + j * SW >= nks) break;   // uniform
            const uint32_t k = (uint32_t)((ks0 + j * SW) * 64 + kh);
#pragma unroll
            for (int f = 0; f < FN; f++) w[j][f] = piece_load(P.wgt, wrow[f] + k, wbytes);
#pragma unroll
            for (int f = 0; f < FM; f++) x[j][f] = piece_load(P.act, arow[f] + k, abytes);
        }
#pragma unroll
        for (int j = 0; j < KB; j++) {
            if (ks0 + j * SW >= nks) break;
            if (ks0 + j * SW == nks - 1) {   // uniform
                const int k = (ks0 + j * SW) * 64 + kh;
#pragma unroll
                for (int f = 0; f < FN; f++) w[j][f] = piece_cut<WHOLE>(w[j][f], P.wgt, wrow[f] + k, wbytes, k, L);
#pragma unroll
                for (int f = 0; f < FM; f++) x[j][f] = piece_cut<WHOLE>(x[j][f], P.act, arow[f] + k, abytes, k, L);
            }
#pragma unroll
            for (int a = 0; a < FN; a++)
#pragma unroll
                for (int b = 0; b < FM; b++)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[j][a], x[j][b], acc[a][b], 0, 0, 0);
        }
    }

    // acc[a][b] element i: channel n0 + 16 a + 4*(lane/16) + i, row m0 + 16 b + lane%16.
#pragma unroll
    for (int a = 0; a < FN; a++)
#pragma unroll
        for (int b = 0; b < FM; b++)
            *(v4i*)(red + (wave * ROWS + 16 * b + r16) * RP + 16 * a + 4 * (lane >> 4)) = acc[a][b];
    __syncthreads();
    if (threadIdx.x < ROWS * 8) {
        const int row = threadIdx.x >> 3, c4 = (threadIdx.x & 7) * 4;
        const int m = m0 + row, n = n0 + c4;
        v4i s = *(const v4i*)(red + row * RP + c4);
#pragma unroll
        for (int w = 1; w < SW; w++) s += *(const v4i*)(red + (w * ROWS + row) * RP + c4);
        if (m < P.M && n < P.Nout) {
            const int nv = min(4, P.Nout - n);
            int32_t v[4] = {s[0], s[1], s[2], s[3]};
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (relu && v[i] < 0) v[i] = 0;
            if (do_max) {
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (i < nv) tmax = max(tmax, mag32(v[i]));
            }
            if (do_store) {
                const int64_t off = (int64_t)m * P.ldo + n;
                uint32_t packed = 0;
#pragma unroll
                for (int i = 0; i < 4; i++) packed |= (uint32_t)(uint8_t)round_i32(v[i], rk) << (8 * i);
                if (P.mask) {
                    const int8_t* ms = P.mask + off;
                    for (int i = 0; i < nv; i++)
                        if (ms[i] <= 0) packed &= ~(0xFFu << (8 * i));
                }
                int8_t* dst = P.out + off;
                if (nv == 4 && (((uintptr_t)dst) & 3) == 0) {
                    *(uint32_t*)dst = packed;
                } else {
                    for (int i = 0; i < nv; i++) dst[i] = (int8_t)(packed >> (8 * i));
                }
            }
        }
    }
    __syncthreads();   // red is reused by the next tile
}

// Main launch: every tile once, the maximum folded in, the output rounded
// with a guessed shift (none stored without one).
template <bool WHOLE, int FM>
__global__ __launch_bounds__(ST) void igemm_small_main(IgemmProblem P, IgemmCtl ctl) {
    __shared__ __attribute__((aligned(16))) int32_t red[SW * 16 * FM * RP];
    __shared__ uint32_t wmax[ST / 64];
    niti_stats* st = ctl.stats;
    const int slot = call_slot(st);
    const uint64_t snap = max_snapshot(st, slot);
    const int hint = st->bp_hint;
    begin_call(st, slot, hint);
    const RoundK rk = make_round(hint < 0 ? 0 : hint, ctl.mode);
    uint32_t tmax = 0;
    small_tile<WHOLE, FM>(P, blockIdx.x, red, rk, ctl.relu, hint >= 0, true, tmax);
    block_publish_max32(st, slot, tmax, wmax, snap);  // magnitudes <= 2^31
}

// Fix-up launch: with the final maximum, recompute every tile when the
// guessed shift was wrong; workgroup 0 then finalizes the statistics.
template <bool WHOLE, int FM>
__global__ __launch_bounds__(ST) void igemm_small_fixup(IgemmProblem P, IgemmCtl ctl, int ntiles) {
    __shared__ __attribute__((aligned(16))) int32_t red[SW * 16 * FM * RP];
    niti_stats* st = ctl.stats;
    const CallState cs = shared_call_state(st);
    const int hint = cs.hint;
    const int bp = block_bp(cs.mx, ctl.target);
    if (bp != hint) {
        const RoundK rk = make_round(bp, ctl.mode);
        uint32_t dummy = 0;
        for (int t = blockIdx.x; t < ntiles; t += gridDim.x) small_tile<WHOLE, FM>(P, t, red, rk, ctl.relu, true, false, dummy);
    }
    if (is_finisher()) finish_call(st, ctl.target, ctl.ex, ctl.static_flags, 1);
}

}  // namespace

// A single plain matrix product: 1 x 1 taps over an unpadded, unstrided
// input whose rows are the L-byte reduction vectors, written densely
// (row stride = Nout), with at most MAX_M rows and few 128 x 128 tiles.
bool igemm_small_eligible(const IgemmBatch& b) {
    if (b.nprob != 1) return false;
    const IgemmProblem& p = b.p[0];
    if (p.M < 1 || p.M > MAX_M || p.Nout < 1 || p.L < 0) return false;
    if (p.R != 1 || p.S != 1 || p.C != p.L || p.win) return false;
    if (p.H != p.OHc || p.W != p.OWc || p.st != 1 || p.off_h != 0 || p.off_w != 0) return false;
    if (p.OH != p.OHc || p.OW != p.OWc || p.os != 1 || p.oa != 0 || p.ob != 0) return false;
    if (p.ldo != p.Nout || p.zsib) return false;
    if (p.L > 0 && (p.act_bytes < 16 || p.wgt_bytes < 16)) return false;   // pieces are loaded whole
    const int64_t tiles128 = (int64_t)((p.M + 127) / 128) * ((p.Nout + 127) / 128);
    return tiles128 < 64;
}

namespace {
template <bool WHOLE, int FM>
hipError_t launch_small(const IgemmProblem& p, const IgemmCtl& ctl, hipStream_t stream) {
    const int ntiles = ((p.M + 16 * FM - 1) / (16 * FM)) * ((p.Nout + 31) / 32);
    const int tk = timing_on() ? timing_begin(NITI_TIMING_KERNEL, stream, kernel_label("igemm_small_main<%d,%d>", (int)WHOLE, FM))
                               : -1;
    hipLaunchKernelGGL((igemm_small_main<WHOLE, FM>), dim3(ntiles), dim3(ST), 0, stream, p, ctl);
    timing_end(tk, stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int fix_grid = ntiles < kFixupGrid ? ntiles : kFixupGrid;
    hipLaunchKernelGGL((igemm_small_fixup<WHOLE, FM>), dim3(fix_grid), dim3(ST), 0, stream, p, ctl, ntiles);
    return hipGetLastError();
}
}  // namespace

// 64 rows per tile read the weights half as often; taken where tiles of 32
// rows are more than one per CU, so that a second round of them would follow,
// and those of 64 are not, or the reduction is one batch of their loads (2048
// bytes; half of that where pieces are unaligned): tiles of 64 rows that are a
// round and a little more, each of several memory round trips, lose to
// those of 32, of which two share a CU.
// Products in us, tiles of 32 / 64 rows: 64 x 4096 x 4096 (256 tiles of 32)
// 15.3 / 17.5, 63 x 2645 x 4192 (166) 12.3 / 13.8; 67 x 2765 x 200 (261) 10.7 /
// 8.4, 353 x 1084 x 2588 (408) 20.2 / 13.1, 44 x 6541 x 1844 (410) 19.6 / 12.5.
// 89 x 4688 x 2880 (441 of 32, 294 of 64) 14.8 / 19.3, 1003 x 655 x 3280 (672,
// 336) 21.2 / 27.5, 195 x 3328 x 2058 (728, 416) 27.8 / 36.7.
// Training passes at batch 128, 32 rows / 64 rows: 4096 -> 4096 84.6 / 76.2;
// 9216 -> 4096 138.5 / 130.4; 4096 -> 1000 87.0 / 78.4.
hipError_t igemm_small_run(IgemmBatch& b, IgemmCtl ctl, hipStream_t stream) {
    const IgemmProblem& p = b.p[0];
    const int64_t cols = (p.Nout + 31) / 32, low = (p.M + 31) / 32 * cols, high = (p.M + 63) / 64 * cols;
    const bool whole = p.L % 16 == 0;
    const bool tall = p.M > 32 && low > 256 && (high <= 256 || p.L <= (whole ? 2048 : 1024));
    if (whole) return tall ? launch_small<true, 4>(p, ctl, stream) : launch_small<true, 2>(p, ctl, stream);
    return tall ? launch_small<false, 4>(p, ctl, stream) : launch_small<false, 2>(p, ctl, stream);
}

}  // namespace niti
