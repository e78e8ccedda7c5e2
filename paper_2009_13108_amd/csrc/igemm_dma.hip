// Implicit-GEMM int8 MFMA kernel with a multi-stage LDS ring filled by
// direct-to-LDS buffer loads (gfx950 buffer_load_dwordx4 ... lds).  Same
// problem form, epilogue and exponent speculation as igemm.hip, which keeps
// the general path (odd channel counts such as a 4-channel image layer).
//
// Load modes; all but kConv16 keep the per-step address work uniform:
//   kGemm   plain matrix rows (H = W = 1, one tap): a lane's offset is fixed
//           and the K step adds a uniform amount;
//   kConv   convolutions whose channels are whole K steps: every step lies in
//           one filter tap (r, s) and channel block c0, all uniform, so a lane
//           only checks that its pixel's tap is inside the image;
//   kWin    convolutions with few channels (S*C <= 64) over a zero-padded
//           copy of the input: a filter row is one contiguous window of
//           L = 16, 32 or 64 bytes (S pixels, zero weights past them), a K
//           step covers KS/L filter rows, and every window is in bounds, so
//           a lane's offset is fixed and the step adds a uniform amount;
//   kConv16 convolutions with C % 16 == 0 that the others do not take (96
//           channels, or more than 32 taps): each 16-byte piece lies in one
//           filter tap, but the four pieces of a step may lie in different
//           ones, so a lane carries its piece's (row, pixel, channel) and
//           moves it by a step with two carries; ~18 vector
//           instructions per step.  Before, such layers ran on the general
//           kernel: 5x5, 96 -> 256 channels at 27x27, batch 128: 156 -> 85 us.
//
// K steps are KS = 64 or 128 bytes per row.  Rows are hundreds of bytes apart,
// and half of a 128-byte cache line costs the CU's load path as much as all
// of it: a load-only probe of 16 KB steps took 0.19..0.25 us per CU in
// 64-byte row segments (which is what a K step of the 128 x 128 tile took, not
// its MFMAs) and 0.13 us in 128-byte ones.
//
// Loads.  Each wave instruction moves 64 lanes x 16 bytes into one 1 KiB LDS
// block (lane l lands at block + 16 l); a block holds 1024 / KS operand rows
// of one K step.  A lane whose piece is outside the image, past the tensor
// or past K uses an offset beyond the buffer's size, which the hardware
// answers with zeros.  Within a row the 16-byte chunks are stored
// XOR-swizzled (position = chunk ^ f(row)) so that the 32x32x32 MFMA fragment
// reads (16 bytes per lane, one chunk of 32 rows) hit distinct banks.
//
// Pipeline.  NS stages; stage k+NS-1 is issued while stage k is computed.
// Loads past the last K step are issued anyway (as zeros), so the wait
// count before each step is a constant.
#include "niti_internal.h"

namespace niti {

namespace {

constexpr uint32_t kOOB = 0x80000000u;
constexpr int kGemm = 0;
constexpr int kConv = 1;
constexpr int kWin = 2;
constexpr int kConv16 = 3;

typedef __attribute__((address_space(3))) void lds_void;

template <int KS>
__device__ __forceinline__ int swz(int row) {
    return KS == 64 ? ((row >> 1) ^ (row >> 2)) & 3 : (row >> 1) & 7;
}

template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// vmcnt <= N and lgkmcnt == 0 (this wave's LDS reads done).
template <int N>
__device__ __forceinline__ void wait_vm_lgkm0() {
    static_assert(N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
}

template <int BM, int BN, int NS, int WGM, int WGN, int KS>
struct Cfg {
    static constexpr int RPB = 1024 / KS;                   // rows per 1 KiB block
    static constexpr int LPR = KS / 16;                     // lanes per row
    static constexpr int NH = KS / 32;                      // MFMA depths per step
    static constexpr int NWAVES = WGM * WGN;
    static constexpr int NT = 64 * NWAVES;
    static constexpr int WTM = BM / WGM, WTN = BN / WGN;   // wave tile: pixels x channels
    static constexpr int FM = WTM / 32, FN = WTN / 32;
    static constexpr int BLOCKS = (BM + BN) / RPB;          // 1 KiB blocks per stage
    static constexpr int ABLK = BN / RPB;                   // blocks holding weight rows
    // Weight blocks per wave: ABLK / NWAVES each, or (fewer blocks than
    // waves) one each for waves 0 .. ABLK-1.  A wave takes every NWAVES-th
    // block of an operand: the swizzle of 8-row blocks alternates with the
    // block's parity, which a wave's blocks then share.
    static constexpr bool W_EVEN = ABLK % NWAVES == 0;
    static constexpr int IPW_W = W_EVEN ? ABLK / NWAVES : 1;
    static constexpr int IPW_A = (BLOCKS - ABLK) / NWAVES;  // activation blocks per wave
    static_assert((BLOCKS - ABLK) % NWAVES == 0 && (W_EVEN || ABLK < NWAVES), "load split over waves");
    static_assert(NWAVES % 2 == 0 && ABLK % 2 == 0, "one swizzle parity per wave");
    static constexpr int STAGE_BYTES = (BM + BN) * KS;
    static constexpr int LDS_BYTES = NS * STAGE_BYTES;
    static constexpr int WGM_ = WGM, BN_ = BN;
    static_assert(BM * (BN + 16) <= LDS_BYTES, "output tile fits in the ring");
};

// Round one accumulator (Algorithm 3 in the closed form of niti_device.h,
// or nearest) with the tile's uniform shift; RELU: v is already
// non-negative.  Magnitudes are at most 2^31, so the 32-bit maximum is
// exact.  Returns the int8 in the low byte.
template <bool RELU, bool RTN>
__device__ __forceinline__ uint32_t round_acc(int32_t v, const RoundK& k, uint32_t& tmax) {
    const uint32_t x = RELU ? (uint32_t)v : (v < 0 ? 0u - (uint32_t)v : (uint32_t)v);
    tmax = x > tmax ? x : tmax;
    uint32_t q;
    if (RTN) {
        q = x >> k.bp;
        q = min(q + (k.bp ? __builtin_amdgcn_ubfe(x, k.bp - 1, 1) : 0u), 127u);
    } else {
        q = round_psr_mag_fast(x, k);
    }
    if (RELU) return q;
    const uint32_t sgn = (uint32_t)(v >> 31);
    return ((q ^ sgn) - sgn) & 0xFFu;
}

// Tile maximum and rounded bytes of the register accumulators; the bytes go
// to an LDS tile [BM][BN + 16] (row = tile pixel).
template <typename T, bool RELU, bool RTN>
__device__ __forceinline__ void epilogue_regs(v16i (&acc)[T::FN][T::FM], int8_t* lds, const RoundK& rk,
                                              int do_store, int do_max, uint64_t& tmax) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % T::WGM_, wn = wave / T::WGM_;
    constexpr int PITCH = T::BN_ + 16;
    uint32_t mx = 0;
#pragma unroll
    for (int b = 0; b < T::FM; b++) {
        const int row = wm * T::WTM + b * 32 + (lane & 31);
#pragma unroll
        for (int a = 0; a < T::FN; a++)
#pragma unroll
            for (int jj = 0; jj < 4; jj++) {
                uint32_t packed = 0;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    int32_t v = acc[a][b][4 * jj + i];
                    if (RELU) v = v < 0 ? 0 : v;
                    packed |= round_acc<RELU, RTN>(v, rk, mx) << (8 * i);
                }
                if (do_store) {
                    const int col = wn * T::WTN + a * 32 + 8 * jj + 4 * (lane >> 5);
                    *(uint32_t*)(lds + row * PITCH + col) = packed;
                }
            }
    }
    if (do_max) tmax = (uint64_t)mx > tmax ? (uint64_t)mx : tmax;
}

// Out-of-tile accumulators are zero (their operand rows were zero-filled),
// so including them in the maximum is harmless.  The LDS tile is written to
// the output in 16-byte row pieces, with the backward ReLU mask applied.  Whole
// pieces are stored as such at any address (output rows whose channels are no
// multiple of 16 are unaligned): byte by byte the stores alone bounded such
// products (18508 x 1539 x 128 60.9 us, 31119 x 1165 x 128 81.7; 44.9 whole).
template <typename T, int BM, int BN>
__device__ __forceinline__ void store_tile(const IgemmProblem& P, int tm, int tn, const int8_t* lds) {
    constexpr int PITCH = BN + 16;
    constexpr int PPR = BN / 16;  // pieces per row
    const bool dense = P.os == 1 && P.OHc == P.OH && P.OWc == P.OW;
    for (int idx = threadIdx.x; idx < BM * PPR; idx += T::NT) {
        const int row = idx / PPR, pc = idx - row * PPR;
        const int m = tm * BM + row;
        const int n0 = tn * BN + pc * 16;
        if (m >= P.M || n0 >= P.Nout) continue;
        int64_t ooff;
        const int nv = min(16, P.Nout - n0);
        if (dense) {
            ooff = (int64_t)m * P.ldo + n0;   // the output grid is the pixel grid
        } else {
            const uint32_t img = fdiv((uint32_t)m, P.div_ohw);
            const uint32_t rem = (uint32_t)m - img * (uint32_t)(P.OHc * P.OWc);
            const uint32_t i0 = fdiv(rem, P.div_ow);
            const uint32_t j0 = rem - i0 * (uint32_t)P.OWc;
            const int oh = (int)i0 * P.os + P.oa;
            const int ow = (int)j0 * P.os + P.ob;
            ooff = (((int64_t)img * P.OH + oh) * P.OW + ow) * P.ldo + n0;
            if (P.zsib) store_zero_siblings(P, ooff, zero_siblings(P, oh, ow), nv);
        }
        uint4 v = *(const uint4*)(lds + row * PITCH + pc * 16);
        int8_t* dst = P.out + ooff;
        const bool full = nv == 16;
        if (P.mask) {
            const int8_t* ms = P.mask + ooff;
            uint32_t mw[4] = {0u, 0u, 0u, 0u};
            if (full) {
                const uint4 mv = load16_any(ms);
                mw[0] = mv.x; mw[1] = mv.y; mw[2] = mv.z; mw[3] = mv.w;
            } else {
                for (int e = 0; e < nv; e++) mw[e >> 2] |= (uint32_t)(uint8_t)ms[e] << (8 * (e & 3));
            }
            uint32_t vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int q = 0; q < 4; q++) vw[q] &= positive_bytes(mw[q]);
            v = make_uint4(vw[0], vw[1], vw[2], vw[3]);
        }
        if (full) {
            store16_any(dst, v);
        } else {
            const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
            for (int e = 0; e < nv; e++) dst[e] = (int8_t)(vw[e >> 2] >> (8 * (e & 3)));
        }
    }
}

template <int BM, int BN, int NS, int WGM, int WGN, int KS, int MODE>
__device__ __forceinline__ void dma_tile(const IgemmProblem& P, int tm, int tn, int8_t* lds, const RoundK& rk,
                                         int relu, int do_store, int do_max, uint64_t& tmax, niti_stats* snap_st,
                                         int snap_slot, uint64_t& snap) {
    using T = Cfg<BM, BN, NS, WGM, WGN, KS>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WGM, wn = wave / WGM;

    const u32x4 act_rs = raw_rsrc(P.act, (uint32_t)P.act_bytes);
    const u32x4 wgt_rs = raw_rsrc(P.wgt, (uint32_t)P.wgt_bytes);

    // Per-lane row state for each load instruction: a wave issues IPW_W
    // weight blocks and IPW_A activation blocks per stage; wb / ab is the
    // lane's byte offset at K step 0 (kOOB for a row past the operand).
    const int lrow = lane / T::LPR;   // row within a block
    const uint32_t kpo = (uint32_t)(((lane % T::LPR) ^ swz<KS>((wave & 1) * T::RPB + lrow)) << 4);  // byte offset of this lane's chunk
    uint32_t wb[T::IPW_W], ab[T::IPW_A];
    // kConv: taps (bit r*S+s) outside the image; kWin: filter row of the
    // piece; kConv16: filter rows (low half) and columns (high half) inside
    uint32_t aux[T::IPW_A];
    const bool wload = T::W_EVEN || wave < T::ABLK;   // this wave loads weight blocks (uniform)
#pragma unroll
    for (int i = 0; i < T::IPW_W; i++) {
        const int n = tn * BN + (wave + i * T::NWAVES) * T::RPB + lrow;
        wb[i] = (wload && n < P.Nout) ? (uint32_t)n * (uint32_t)P.Ktot + kpo : kOOB;
    }
#pragma unroll
    for (int i = 0; i < T::IPW_A; i++) {
        const int m = tm * BM + (wave + i * T::NWAVES) * T::RPB + lrow;
        aux[i] = 0;
        if (MODE == kGemm) {
            ab[i] = m < P.M ? (uint32_t)m * (uint32_t)P.C + kpo : kOOB;
        } else {
            const uint32_t mm = m < P.M ? (uint32_t)m : 0u;
            const uint32_t img = fdiv(mm, P.div_ohw);
            const uint32_t rem = mm - img * (uint32_t)(P.OHc * P.OWc);
            const uint32_t oh = fdiv(rem, P.div_ow);
            const uint32_t ow = rem - oh * (uint32_t)P.OWc;
            if (MODE == kWin) {
                const int rr = (int)kpo / P.L;              // filter row of this piece within a step
                const int j0 = (int)kpo - rr * P.L;
                aux[i] = (uint32_t)rr;
                ab[i] = m < P.M ? (uint32_t)(((img * (uint32_t)P.H + oh * (uint32_t)P.st + (uint32_t)rr) *
                                                  (uint32_t)P.W + ow * (uint32_t)P.st) * (uint32_t)P.C) + (uint32_t)j0
                                : kOOB;
            } else {
                const int h0 = (int)oh * P.st + P.off_h;
                const int w0 = (int)ow * P.st + P.off_w;
                ab[i] = (uint32_t)((int64_t)img * P.H * P.W * P.C + ((int64_t)h0 * P.W + w0) * P.C) + kpo;
                // taps (r, s) whose input pixel lies outside the image (all of
                // them for a row past M)
                uint32_t rows = 0, cols = 0, valid = 0;
                for (int r = 0; r < P.R; r++) rows |= (uint32_t)((unsigned)(h0 + r) < (unsigned)P.H) << r;
                for (int c = 0; c < P.S; c++) cols |= (uint32_t)((unsigned)(w0 + c) < (unsigned)P.W) << c;
                if (MODE == kConv16) {
                    ab[i] -= kpo;   // the piece's offset is carried apart
                    aux[i] = m < P.M ? rows | (cols << 16) : 0u;
                } else {
                    for (int r = 0; r < P.R; r++)
                        if ((rows >> r) & 1u) valid |= cols << (r * P.S);
                    aux[i] = m < P.M ? ~valid : ~0u;
                }
            }
        }
    }

    const int nk = (P.Ktot + KS - 1) / KS;
    // Scalar instructions issue at about one per cycle per CU, shared by all
    // waves, so the load side keeps its per-step uniform work small: the
    // lanes' current offsets cvw / cva change only at events (a filter tap
    // change, the last K step, the end of K), counted down by ev; between
    // events a step adds to the two uniform offsets kb (weights, and kGemm
    // activations) and sa (kConv: channel offset within the tap; kWin:
    // window row offset).  The uniform part of an offset rides in the
    // instruction's SGPR offset; every lane offset that is not kOOB stays
    // inside its buffer together with it, and lanes whose piece is past K,
    // past R or outside the image get kOOB (zeros).
    const uint32_t lds0 = lds_address(lds);
    uint32_t wdst[T::IPW_W], adst[T::IPW_A];   // this wave's blocks in stage 0
#pragma unroll
    for (int i = 0; i < T::IPW_W; i++) wdst[i] = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(wave + i * T::NWAVES) * 1024u);
#pragma unroll
    for (int i = 0; i < T::IPW_A; i++)
        adst[i] = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(T::ABLK + wave + i * T::NWAVES) * 1024u);
    const int cbs = __builtin_amdgcn_readfirstlane(MODE == kConv ? P.C / KS : 1);   // steps per tap
    const int ntap = __builtin_amdgcn_readfirstlane(P.R * P.S);
    const uint32_t da = __builtin_amdgcn_readfirstlane(
        MODE == kWin ? (uint32_t)(KS / P.L) * (uint32_t)(P.W * P.C) : (uint32_t)KS);
    const uint32_t klim = __builtin_amdgcn_readfirstlane(
        MODE == kWin ? (uint32_t)(P.R - (nk - 1) * (KS / P.L)) : 0u);   // kWin: filter rows of the last step
    const uint32_t kend = __builtin_amdgcn_readfirstlane((uint32_t)(P.Ktot - (nk - 1) * KS));   // its K bytes
    // kConv16: this lane's piece as filter row, pixel in it, channel, and its
    // offset from the pixel's first tap; a step of 64 bytes in those units.
    int pr = 0, ps = 0, pc = 0;
    uint32_t poff = 0;
    int step_r = 0, step_s = 0, step_c = 0;
    uint32_t step_off = 0, row_wrap = 0;
    if constexpr (MODE == kConv16) {
        pr = div64((int)kpo, P.L);
        ps = div64((int)kpo - pr * P.L, P.C);
        pc = (int)kpo - pr * P.L - ps * P.C;
        poff = (uint32_t)((pr * P.W + ps) * P.C + pc);
        step_r = div64(KS, P.L);
        step_s = div64(KS - step_r * P.L, P.C);
        step_c = KS - step_r * P.L - step_s * P.C;
        step_off = (uint32_t)((step_r * P.W + step_s) * P.C + step_c);
        row_wrap = (uint32_t)((P.W - P.S) * P.C);
    }
    uint32_t kb = 0, sa = 0, tapbase = 0;
    int ev = 0, tap = 0, ts = 0, ph = 0;
    uint32_t cvw[T::IPW_W], cva[T::IPW_A];
#pragma unroll
    for (int i = 0; i < T::IPW_W; i++) cvw[i] = wb[i];
    auto set_tap = [&]() {
#pragma unroll
        for (int i = 0; i < T::IPW_A; i++) cva[i] = (__builtin_amdgcn_ubfe(aux[i], (uint32_t)tap, 1) << 31) | (ab[i] + tapbase);
    };
    // last K step (kGemm: pieces past K; kWin: rows past R masked)
    auto last_step = [&]() {
        ph = 1;
        ev = 1;
#pragma unroll
        for (int i = 0; i < T::IPW_W; i++) cvw[i] = kpo >= kend ? kOOB : wb[i];
#pragma unroll
        for (int i = 0; i < T::IPW_A; i++) cva[i] = (MODE == kGemm ? kpo >= kend : aux[i] >= klim) ? kOOB : ab[i];
    };
#pragma unroll
    for (int i = 0; i < T::IPW_A; i++) cva[i] = ab[i];
    if (nk <= 0) {
        ph = 2;
        ev = 1 << 30;
    } else if (MODE == kConv) {
        set_tap();
        ev = cbs;
    } else {
        ev = nk - 1;
        if (ev == 0) last_step();
    }
    // Events are handled at the start of the issue that follows them.
    auto advance = [&]() {
        if (MODE == kConv && tap + 1 < ntap) {
            ++tap;
            if (++ts == P.S) {
                ts = 0;
                tapbase += (uint32_t)((P.W - P.S + 1) * P.C);
            } else {
                tapbase += (uint32_t)P.C;
            }
            set_tap();
            sa = 0;
            ev = cbs;
            return;
        }
        if (MODE != kConv && ph == 0) {
            last_step();
            return;
        }
        // Past the end of K the loads go on as zeros: they keep the wait
        // counts constant, and the stages they fill are never multiplied.
#pragma unroll
        for (int i = 0; i < T::IPW_W; i++) cvw[i] = kOOB;
#pragma unroll
        for (int i = 0; i < T::IPW_A; i++) cva[i] = kOOB;
        tap = 1 << 30;
        ph = 2;
        ev = 1 << 30;
    };
    // issue(j): load K step j (ring slot j % NS)
    auto issue = [&](int j) {
        const uint32_t slot = (uint32_t)(j % NS) * (uint32_t)T::STAGE_BYTES;
        if constexpr (MODE == kConv16) {
            // Pieces past the last filter row have no row bit and load zeros.
            const bool kin = kpo + kb < (uint32_t)P.Ktot;
            if (wload) {
#pragma unroll
                for (int i = 0; i < T::IPW_W; i++) lds_dma16_at(wgt_rs, wdst[i], slot, kin ? wb[i] : kOOB, kb);
            }
#pragma unroll
            for (int i = 0; i < T::IPW_A; i++) {
                const uint32_t in = (aux[i] >> pr) & (aux[i] >> (16 + ps)) & 1u;
                lds_dma16_at(act_rs, adst[i], slot, in && kin ? ab[i] + poff : kOOB, 0);
            }
            kb += KS;
            pc += step_c;
            ps += step_s;
            pr += step_r;
            poff += step_off;
            if (pc >= P.C) {
                pc -= P.C;
                ++ps;
            }
            if (ps >= P.S) {
                ps -= P.S;
                ++pr;
                poff += row_wrap;
            }
            return;
        }
        if (ev == 0) advance();
        if (wload) {
#pragma unroll
            for (int i = 0; i < T::IPW_W; i++) lds_dma16_at(wgt_rs, wdst[i], slot, cvw[i], kb);
        }
#pragma unroll
        for (int i = 0; i < T::IPW_A; i++) lds_dma16_at(act_rs, adst[i], slot, cva[i], MODE == kGemm ? kb : sa);
        kb += KS;
        sa += da;
        ev = __builtin_amdgcn_readfirstlane(ev - 1);
    };

    v16i acc[T::FN][T::FM];
#pragma unroll
    for (int a = 0; a < T::FN; a++)
#pragma unroll
        for (int b = 0; b < T::FM; b++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[a][b][e] = 0;

    int a_off[T::FN], b_off[T::FM], a_sw[T::FN], b_sw[T::FM];
#pragma unroll
    for (int a = 0; a < T::FN; a++) {
        const int row = wn * T::WTN + a * 32 + (lane & 31);
        a_off[a] = row * KS;
        a_sw[a] = swz<KS>(row & 15);
    }
#pragma unroll
    for (int b = 0; b < T::FM; b++) {
        const int row = wm * T::WTM + b * 32 + (lane & 31);
        b_off[b] = BN * KS + row * KS;
        b_sw[b] = swz<KS>(row & 15);
    }

#pragma unroll
    for (int s = 0; s < NS - 1; s++) issue(s);

    // Register double buffer over the 32-byte depths of a K step: a depth's
    // fragments are read while the previous one's MFMAs run, and the next
    // stage's first right after the barrier, before this stage's last MFMAs.
    // Before each barrier a wave waits for its own fragment reads (lgkmcnt 0),
    // so once all waves pass it no read of the stage that the next load
    // overwrites is still in flight.
    v4i fa[2][T::FN], fb[2][T::FM];
    auto read_depth = [&](const int8_t* st, int ks) {
        const int kp = (lane >> 5) + 2 * ks;
#pragma unroll
        for (int a = 0; a < T::FN; a++) fa[ks & 1][a] = *(const v4i*)(st + a_off[a] + ((kp ^ a_sw[a]) << 4));
#pragma unroll
        for (int b = 0; b < T::FM; b++) fb[ks & 1][b] = *(const v4i*)(st + b_off[b] + ((kp ^ b_sw[b]) << 4));
    };
    auto mma_depth = [&](int ks) {
#pragma unroll
        for (int a = 0; a < T::FN; a++)
#pragma unroll
            for (int b = 0; b < T::FM; b++)
                acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks & 1][a], fb[ks & 1][b], acc[a][b], 0, 0, 0);
    };
    // Loads per stage of this wave (uniform): the stage-exact wait counts.
    constexpr int LW = T::IPW_A + T::IPW_W, LA = T::IPW_A;
    if (wload)
        wait_vm<(NS - 2) * LW>();
    else
        wait_vm<(NS - 2) * LA>();
    __builtin_amdgcn_s_barrier();
    read_depth(lds, 0);
    for (int kt = 0; kt < nk; kt++) {
        const int8_t* st = lds + (kt % NS) * T::STAGE_BYTES;
        issue(kt + NS - 1);   // into the slot of stage kt - 1, which every wave has finished reading
#pragma unroll
        for (int ks = 0; ks + 1 < T::NH; ks++) {
            read_depth(st, ks + 1);
            mma_depth(ks);
        }
        // (after the last step this reads a stage loaded past the end of K,
        // which no MFMA uses: it keeps the loop free of branches)
        if (wload)
            wait_vm_lgkm0<(NS - 2) * LW>();
        else
            wait_vm_lgkm0<(NS - 2) * LA>();
        __builtin_amdgcn_s_barrier();
        read_depth(lds + ((kt + 1) % NS) * T::STAGE_BYTES, 0);
        mma_depth(T::NH - 1);
    }
    // Drain the loads issued past the end before the ring is reused.
    wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    // Snapshot of the tensor maximum for the skip test of the publishing
    // thread: read now, used after the epilogue, so its latency is hidden
    // and it includes the workgroups that finished meanwhile.
    if (snap_st && threadIdx.x == 0) snap = load_acc(snap_st, snap_slot);

    // Epilogue.  acc[a][b] element 4*jj + i is channel
    // wn*WTN + a*32 + 8*jj + 4*(lane/32) + i of tile pixel wm*WTM + b*32 + lane%32.
    // Rounded bytes go to the (drained) LDS ring as a [BM][BN] tile, then
    // leave in 16-byte row pieces.
    const int mode_sel = (relu ? 1 : 0) | (rk.rtn ? 2 : 0);
    switch (mode_sel) {
        case 0: epilogue_regs<T, false, false>(acc, lds, rk, do_store, do_max, tmax); break;
        case 1: epilogue_regs<T, true, false>(acc, lds, rk, do_store, do_max, tmax); break;
        case 2: epilogue_regs<T, false, true>(acc, lds, rk, do_store, do_max, tmax); break;
        default: epilogue_regs<T, true, true>(acc, lds, rk, do_store, do_max, tmax); break;
    }
    if (!do_store) return;
    __syncthreads();
    store_tile<T, BM, BN>(P, tm, tn, lds);
    __syncthreads();
}

__device__ __forceinline__ void locate(const IgemmBatch& b, int t, int& prob, int& tm, int& tn) {
    int p = 0;
#pragma unroll
    for (int i = 1; i < kMaxProblems; i++)
        if (i < b.nprob && t >= b.p[i].tile_base) p = i;
    const int local = t - b.p[p].tile_base;
    prob = p;
    tm = local / b.p[p].tiles_n;
    tn = local - tm * b.p[p].tiles_n;
}

template <int BM, int BN, int NS, int WGM, int WGN, int KS, int MODE>
__global__ __launch_bounds__(64 * WGM * WGN, 1) void igemm_dma_main(IgemmBatch batch, IgemmCtl ctl) {
    extern __shared__ __attribute__((aligned(1024))) int8_t dyn_lds[];
    niti_stats* st = ctl.stats;
    const int slot = call_slot(st);
    uint64_t snap = 0;
    const int hint = st->bp_hint;
    begin_call(st, slot, hint);
    int prob, tm, tn;
    locate(batch, blockIdx.x, prob, tm, tn);
    const RoundK rk = make_round(hint < 0 ? 0 : hint, ctl.mode);
    uint64_t tmax = 0;
    dma_tile<BM, BN, NS, WGM, WGN, KS, MODE>(batch.p[prob], tm, tn, dyn_lds, rk, ctl.relu, hint >= 0, 1, tmax, st, slot,
                                         snap);
    // Accumulator magnitudes are at most 2^31: 32-bit reductions are exact.
    // The ring is drained and the tile stored: its first bytes serve the
    // reduction (no static LDS, so two 80 KiB workgroups fit one CU).
    block_publish_max32(st, slot, (uint32_t)tmax, (uint32_t*)dyn_lds, snap);
}

template <int BM, int BN, int NS, int WGM, int WGN, int KS, int MODE>
__global__ __launch_bounds__(64 * WGM * WGN, 1) void igemm_dma_fixup(IgemmBatch batch, IgemmCtl ctl) {
    extern __shared__ __attribute__((aligned(1024))) int8_t dyn_lds[];
    niti_stats* st = ctl.stats;
    const CallState cs = shared_call_state(st, dyn_lds);
    const int hint = cs.hint;
    const int bp = block_bp(cs.mx, ctl.target);
    if (bp != hint) {
        const RoundK rk = make_round(bp, ctl.mode);
        for (int t = blockIdx.x; t < batch.total_tiles; t += gridDim.x) {
            int prob, tm, tn;
            locate(batch, t, prob, tm, tn);
            uint64_t dummy = 0, nosnap = 0;
            dma_tile<BM, BN, NS, WGM, WGN, KS, MODE>(batch.p[prob], tm, tn, dyn_lds, rk, ctl.relu, 1, 0, dummy, nullptr, 0,
                                                 nosnap);
        }
    }
    if (is_finisher()) finish_call(st, ctl.target, ctl.ex, ctl.static_flags, 1);
}

template <int BM, int BN, int NS, int WGM, int WGN, int KS, int MODE>
hipError_t launch_dma(IgemmBatch& b, IgemmCtl ctl, hipStream_t stream) {
    using T = Cfg<BM, BN, NS, WGM, WGN, KS>;
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute((const void*)igemm_dma_main<BM, BN, NS, WGM, WGN, KS, MODE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess) return e;
        e = hipFuncSetAttribute((const void*)igemm_dma_fixup<BM, BN, NS, WGM, WGN, KS, MODE>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_done = true;
    }
    int base = 0;
    for (int i = 0; i < b.nprob; i++) {
        IgemmProblem& p = b.p[i];
        p.tiles_m = (p.M + BM - 1) / BM;
        p.tiles_n = (p.Nout + BN - 1) / BN;
        p.tile_base = base;
        base += p.tiles_m * p.tiles_n;
    }
    b.total_tiles = base;
    const int tk = timing_on() ? timing_begin(NITI_TIMING_KERNEL, stream,
                                              kernel_label("igemm_dma_main<%d,%d,%d,%d,%d,%d,%d>", BM, BN, NS, WGM,
                                                           WGN, KS, MODE))
                               : -1;
    hipLaunchKernelGGL((igemm_dma_main<BM, BN, NS, WGM, WGN, KS, MODE>), dim3(base), dim3(T::NT), T::LDS_BYTES, stream,
                       b, ctl);
    timing_end(tk, stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int fix_grid = base < kFixupGrid ? base : kFixupGrid;
    hipLaunchKernelGGL((igemm_dma_fixup<BM, BN, NS, WGM, WGN, KS, MODE>), dim3(fix_grid), dim3(T::NT), T::LDS_BYTES,
                       stream, b, ctl);
    return hipGetLastError();
}

int problem_mode(const IgemmProblem& p) {
    if (p.win) return kWin;
    if (p.H == 1 && p.W == 1 && p.R == 1 && p.off_h == 0 && p.off_w == 0 && p.L == p.C) return kGemm;
    return p.C % 64 == 0 && p.R * p.S <= 32 ? kConv : kConv16;
}

// The classes of a strided back-propagation share a launch and so a mode: a
// class with too many taps for kConv takes the others along.
int batch_mode(const IgemmBatch& b) {
    int mode = problem_mode(b.p[0]);
    for (int i = 1; i < b.nprob; i++) {
        const int m = problem_mode(b.p[i]);
        if (m == mode) continue;
        if ((m == kConv && mode == kConv16) || (m == kConv16 && mode == kConv))
            mode = kConv16;
        else
            return -1;
    }
    return mode;
}

// Carried pieces set up more per lane than the general kernel, whose 64 x 64
// tiles also leave less of a narrow output empty.  With up to 16 output channels,
// or a number that is no multiple of 16 (a row's last piece goes by bytes), short
// reductions on few tiles are faster there, and with fewer than 16 channels
// (no whole piece) not only the shortest.  Calls in us, general / ring: 507 x 36
// x 112 13.4 / 15.1, 4096 x 20 x 288 14.3 / 15.2, 6272 x 10 x 288 9.6 / 11.1, 3724 x
// 10 x 432 10.6 / 11.7; but 2704 x 68 x 432 16.1 / 15.5, 588 x 36 x 720 12.8 /
// 11.4, 64 x 10 x 720 11.1 / 10.4, 83106 x 36 x 16 (652 tiles) 17.6 / 16.8, and
// 1183 x 32 x 288 (whole pieces) 9.5 / 8.9.
bool carried_too_short(const IgemmBatch& b) {
    int64_t tiles128 = 0;
    for (int i = 0; i < b.nprob; i++) {
        const IgemmProblem& p = b.p[i];
        if (p.Ktot > (p.Nout < 16 ? 576 : 288) || (p.Nout > 16 && p.Nout % 16 == 0)) return false;
        tiles128 += (int64_t)((p.M + 127) / 128) * ((p.Nout + 127) / 128);
    }
    return tiles128 < 128;
}

// K steps of 128 bytes per row, or of 64 in a ring of twice the stages.  Called
// where a step is uniform (matrix rows, or channels in whole 128s; windows and
// carried pieces stay at 64: 5x5, 96 channels, training pass 272 us at 64, 287
// at 128) and tiles are wider than 64 columns (256 x 64 tiles gain nothing from
// the longer rows and lose the ring's depth: 50176 x 64 x 3456 27.9 / 31.1).
// They pay where whole cache lines are loaded many times over: 14x14, 256
// channels, batch 128 (training pass) 104.0 / 97.7; 8192^3 421 / 404.  They lose
//  - up to one 128 x 128 tile per CU (2048^3 18.8 / 19.5);
//  - where a reduction ends with 64 bytes or fewer in its last step, which is
//    then half empty, unless it is long;
//  - in 256 x 256 tiles where rows are odd multiples of 64 bytes: every other
//    row's pieces then straddle two lines, which 64-byte ones never do;
//  - in short reductions, the sooner the more rounds of tiles there are;
//  - where less than half the CUs have two workgroups, or the last round leaves
//    most of them one: the ring is then all that hides a load.  Above all in
//    convolutions, whose rows are gathered tap by tap (3x3 on 525 tiles, 22320 x
//    320 x 2304 33.0 / 44.9; on 360, 23004 x 256 x 1152 18.0 / 21.2; but on 392,
//    28x28, 128 -> 256, stride 2, batch 128, training pass 85.6 / 83.8).
// Products in us at 64 / 128: 2009 x 3664 x 8592 132.4 / 96.4, 1163 x 15776 x 8192
// (256 x 256 tiles) 213.3 / 184.0; but 12760 x 3952 x 448 52.0 / 58.7 and 8660 x
// 12508 x 304 (256) 101.8 / 109.1 (half a step), 15524 x 944 x 11328 (256) 153.7 /
// 168.4 and 1815 x 4811 x 1728 (570 tiles) 33.5 / 38.4 (odd multiples of 64).
// The limits are from 7000 random products timed both ways: of those with 128
// wherever there is more than one tile per CU 18% were more than 3% slower than
// the better form, with these limits 5%; 1x1 layers of 128 to 512 channels on
// 256 x 256 tiles are 2 to 6% faster.
constexpr int kHalfStep = 64;
bool wide_steps(int K, int64_t tiles128, bool big, bool conv) {
    const int tail = K % 128;   // bytes in the last step (0: a whole one)
    const bool half_empty = tail != 0 && tail <= kHalfStep;
    const bool half_round = (tiles128 - 1) % 512 < 256;   // the last round leaves most CUs one workgroup
    if (tiles128 <= 256) return false;
    if (conv) {
        if (big) return K >= 2048;
        if (K > 1024 && (half_round || (tiles128 < 384 && K < 2048))) return false;
    }
    if (big) return tail != kHalfStep && K >= (half_empty ? 2048 : 640);
    if (tiles128 > 1536) return K >= (half_empty ? 1536 : 768);
    if (tail == kHalfStep && half_round && K >= 1024 && K < 4096) return false;
    return K >= 384;
}

// 256 x 256 tiles, one per CU, or 128 x 128 with eight 32 x 64 waves: two
// workgroups per CU and four waves per SIMD, which hide each other's LDS and
// barrier waits (256 x 128 tiles, one wave per SIMD, were slower: 3000 x 3000 x
// 256 35.5 us against 25.6, 28x28 192 -> 160 training pass 157 against 126).
// Which are faster goes by rounds, 256 tiles or 512: by how far each overfills
// its last one and pads the edges.  A round of 128 covers half the area of one
// of 256 and takes about 1.9 K + 4000 where half the latter takes K + 4000 (1.7
// fits as well on average, but is more often far off for 128).
// Products in us, tiles of 128 / 256 (rounds): 2321 x 5958 x 12352 231.7 / 154.8
// (2, 1), 2819 x 10544 x 1136 73.9 / 53.6 (4, 2); but 3108 x 5008 x 9600 144.3 /
// 206.4 (2, 2), 7235 x 6880 x 384 49.4 / 66.3 (7, 4).  Over 8400 random products
// and convolutions the choice takes 1.4% longer than the better one; 256
// wherever it does not pad the channels further than 128 took 6.3%.
bool tiles_of_256(const IgemmBatch& b, int64_t K, int64_t tiles128) {
    int64_t tiles256 = 0;
    for (int i = 0; i < b.nprob; i++)
        tiles256 += (int64_t)((b.p[i].M + 255) / 256) * ((b.p[i].Nout + 255) / 256);
    const int64_t r256 = (tiles256 + 255) / 256, r128 = (tiles128 + 511) / 512;
    return 20 * r256 * (K + 4000) <= r128 * (19 * K + 40000);
}

template <int MODE>
hipError_t run_mode(IgemmBatch& b, IgemmCtl ctl, hipStream_t stream) {
    int64_t work = 0;
    int maxN = 0, maxK = 0;
    int64_t tiles128 = 0;
    bool whole128 = true;   // kConv: every step of 128 bytes lies in one tap
    for (int i = 0; i < b.nprob; i++) {
        work += (int64_t)b.p[i].M * b.p[i].Nout;
        maxN = b.p[i].Nout > maxN ? b.p[i].Nout : maxN;
        maxK = b.p[i].Ktot > maxK ? b.p[i].Ktot : maxK;
        whole128 = whole128 && b.p[i].C % 128 == 0;
        tiles128 += (int64_t)((b.p[i].M + 127) / 128) * ((b.p[i].Nout + 127) / 128);
    }
    const bool big = maxN > 128 && work >= (int64_t)200 * 256 * 256 && tiles_of_256(b, maxK, tiles128);
    const bool step128 = (MODE == kGemm || (MODE == kConv && whole128)) && maxN > 64 && wide_steps(maxK, tiles128, big, MODE == kConv);
    if constexpr (MODE == kGemm || MODE == kConv) {
        if (step128) {
            if (maxN <= 128) return launch_dma<128, 128, 2, 4, 2, 128, MODE>(b, ctl, stream);
            if (big) return launch_dma<256, 256, 2, 2, 4, 128, MODE>(b, ctl, stream);
            return launch_dma<128, 128, 2, 4, 2, 128, MODE>(b, ctl, stream);
        }
    }
    if (maxN <= 64) return launch_dma<256, 64, 4, 8, 1, 64, MODE>(b, ctl, stream);
    if (maxN <= 128) return launch_dma<128, 128, 4, 4, 2, 64, MODE>(b, ctl, stream);
    if (big) return launch_dma<256, 256, 3, 2, 4, 64, MODE>(b, ctl, stream);
    return launch_dma<128, 128, 4, 4, 2, 64, MODE>(b, ctl, stream);
}

}  // namespace

// True when every problem has whole 16-byte pieces handled by one of the
// load modes and both operands are addressable with 32-bit buffer offsets.
bool igemm_dma_eligible(const IgemmBatch& b) {
    const int mode = batch_mode(b);
    if (mode < 0 || (mode == kConv16 && carried_too_short(b))) return false;
    for (int i = 0; i < b.nprob; i++) {
        const IgemmProblem& p = b.p[i];
        if (p.act_bytes <= 0 || p.act_bytes >= ((int64_t)1 << 31) || p.wgt_bytes <= 0 ||
            p.wgt_bytes >= ((int64_t)1 << 31))
            return false;
        if (mode == kGemm) {
            if (p.C % 16 != 0 || p.Ktot != p.C) return false;
        } else if (mode == kWin) {
            if ((p.L != 16 && p.L != 32 && p.L != 64) || p.Ktot != (p.R * p.L + 63) / 64 * 64 ||
                p.off_h != 0 || p.off_w != 0)
                return false;
        } else {
            if (p.C % 16 != 0 || p.L != p.S * p.C || p.Lpad != p.L || p.Ktot != p.R * p.L) return false;
            // row and column masks of 16 bits; the row of a piece past the
            // last one stays within them for the few steps loaded too far
            if (mode == kConv16 && (p.R > 16 || p.S > 16)) return false;
        }
    }
    return true;
}

hipError_t igemm_dma_run(IgemmBatch& b, IgemmCtl ctl, hipStream_t stream) {
    switch (batch_mode(b)) {
        case kGemm: return run_mode<kGemm>(b, ctl, stream);
        case kWin: return run_mode<kWin>(b, ctl, stream);
        case kConv16: return run_mode<kConv16>(b, ctl, stream);
        default: return run_mode<kConv>(b, ctl, stream);
    }
}

}  // namespace niti
