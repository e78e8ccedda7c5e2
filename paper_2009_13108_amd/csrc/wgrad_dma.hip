// Weight-gradient contraction g32 = a(l-1) (x) e(l) (Algorithm 1; Section
// 3.3) with a DMA-fed LDS ring and LDS transpose reads, for layers whose
// channel counts are multiples of 16 (the general path is wgrad.hip).
//
//   g32[k][col] = sum over pixels pix of dy[pix][k] * X[pix][col],
//   col = (r*S + s)*C + c,  X[pix][col] = x[n][oh*sh - ph + r][ow*sw - pw + s][c]
//
// Both operands are stored in LDS pixel-major, exactly as they arrive from
// NHWC memory (a row per pixel: 128 columns or 64/128 channels, 16-byte
// chunks XOR-swizzled by pixel).  The MFMA wants each lane's 16 bytes along
// the reduction (pixels); ds_read_b64_tr_b8 delivers that directly: within a
// group of 16 lanes that each address 8 bytes of a pixel row, lane i < 8
// receives byte i of the even lanes' rows and lane 8 + i byte i of the odd
// lanes' rows.  With lanes 2q and 2q+1 addressing the two 8-byte halves of
// pixel row q, every lane gets one column over 8 pixels; two such reads give
// the 16 pixel bytes of a 32x32x32 fragment lane.
//
// Each workgroup reduces one pixel range for one output tile and stores the
// partial tile to its own slice; a bandwidth pass sums the slices.
//
// One pixel range (a fully-connected layer's batch): the contraction is run
// twice instead, once for the tensor maximum and once to round and update the
// weights in its epilogue, and g32 never goes through memory
// (wgrad_twice_run).
//
// Window mode (few channels, S*C <= 64): x is a zero-padded copy of the
// input, and a filter row (r) is one window of Lw bytes (S pixels and zero
// columns past them), so column col = r*Lw + j of X is x_pad at pixel row
// oh*sh + r, byte (ow*sw)*C + j: always in bounds.  Only columns with j <
// S*C are stored, compacted to r*S*C + j.
#include "niti_internal.h"

namespace niti {

namespace {

constexpr int PIX = 64;                 // pixels per stage
constexpr uint32_t kOOB = 0x80000000u;
constexpr int64_t kOver = 5 * PIX;      // pixels past the last one that the ring may form offsets of, and one stage

typedef __attribute__((address_space(3))) v2i lds_v2i;

template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// Swizzle of a pixel row's 16-byte chunks: conflict-free transpose reads
// over 8 consecutive pixels for 128-byte rows and 64-byte rows.
template <int RB>
__device__ __forceinline__ int swz(int pix) {
    return RB == 128 ? (pix & 7) : ((pix >> 1) & 3);
}

template <int TBK, int TBC, int NS>
struct WCfg {
    static constexpr int XBLK = TBC * PIX / 1024;      // 1 KiB blocks of the X tile per stage
    static constexpr int DBLK = TBK * PIX / 1024;      // blocks of the dy tile
    static constexpr int BLOCKS = XBLK + DBLK;
    static constexpr int XPW = XBLK / 4, DPW = DBLK / 4;   // blocks a wave loads per stage
    static constexpr int IPW = XPW + DPW;
    static constexpr int XBYTES = TBC * PIX;
    static constexpr int STAGE = (TBC + TBK) * PIX;
    static constexpr int LDS = NS * STAGE;
    static constexpr int WTK = TBK / 2, WTC = TBC / 2;  // 2 x 2 waves
    static constexpr int FK = WTK / 32, FC = WTC / 32;
    static_assert(XBLK % 4 == 0 && DBLK % 4 == 0, "blocks per wave");
};

// One 32 x 32-pixel fragment from a pixel-major region with RB-byte rows:
// lane gets 16 pixel bytes (pixels p0 + 16*(lane/32) ...) of column cbase + lane%32.
template <int RB>
__device__ __forceinline__ v4i tr_fragment(const int8_t* region, int p0, int cbase, int lane) {
    const int g = lane >> 4, j = lane & 15;
    const int col0 = cbase + 16 * (g & 1);            // 16-column group of this lane group
    const int chunk = col0 >> 4;
    const int prow = p0 + 16 * (g >> 1) + (j >> 1);   // pixel row this lane addresses
    const int half = (j & 1) * 8;
    const int8_t* a0 = region + prow * RB + ((chunk ^ swz<RB>(prow)) << 4) + half;
    const int8_t* a1 = region + (prow + 8) * RB + ((chunk ^ swz<RB>(prow + 8)) << 4) + half;
    const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)a0);
    const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)a1);
    v4i r;
    r[0] = lo[0];
    r[1] = lo[1];
    r[2] = hi[0];
    r[3] = hi[1];
    return r;
}

// What becomes of a tile (template argument EP): stored as a partial sum;
// folded into the call's maximum; or, for EP >= 0, rounded in mode EP with the
// call's shift and subtracted from w.
constexpr int kStore = -2;
constexpr int kMaxOnly = -1;
struct WgradFinish {
    int8_t* w;
    niti_stats* st;
    int mu;
    uint32_t static_flags;
};

// log2 of a window's bytes (16, 32 or 64).
__device__ __forceinline__ int window_log(const WgradProblem& P) { return P.Lw == 16 ? 4 : (P.Lw == 32 ? 5 : 6); }

template <int TBK, int TBC, int NS, int EP>
__device__ __forceinline__ void wgrad_tile(const WgradProblem& P, int8_t* lds, int split, int c0, int k0,
                                           const WgradFinish& fin, const RoundK& rk, uint32_t& tmax) {
    using T = WCfg<TBK, TBC, NS>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave & 1, wc = wave >> 1;
    const int pbeg = split * P.chunk;
    const int pend = min(P.npix, pbeg + P.chunk);
    const int nsteps = pend > pbeg ? (pend - pbeg + PIX - 1) / PIX : 0;

    // Loads go out as inline assembly (lds_dma16): with the load builtin the
    // compiler waits for the whole ring before every transpose read.
    const u32x4 xrs = raw_rsrc(P.x, (uint32_t)P.x_bytes);
    const u32x4 drs = raw_rsrc(P.dy, (uint32_t)P.dy_bytes);
    const uint32_t lds0 = lds_address(lds);

    // Loads of a wave and stage: XPW blocks of the X tile (8 pixels x 128
    // bytes) and DPW of the dy tile.  A lane keeps the buffer offset of its
    // 16 bytes and moves it by PIX pixels per stage with adds and two wraps
    // (row, image) instead of decoding the pixel again: the address work
    // was ~200 vector instructions per stage against 8 MFMAs, half of the
    // waves did all of it for X, and it bounded the kernel.  Pixels at or past
    // npix need no test: their dy offsets lie past the buffer's end and load
    // zeros (a split's range ends on a stage, or at npix).
    uint32_t xoff[T::XPW], doff[T::DPW];
    int ih[T::XPW], iw[T::XPW], lim_h[T::XPW], lim_w[T::XPW];   // input position of the tap, and its wraps
    const bool lin = !P.win && P.R == 1 && P.S == 1 && P.sh == 1 && P.sw == 1 && P.ph == 0 && P.pw == 0;
    const int pq = P.P * P.Q;
    const int dn = (int)fdiv(PIX, P.div_pq), drem = PIX - dn * pq;
    const int doh = (int)fdiv((uint32_t)drem, P.div_q), dow = drem - doh * P.Q;
    const uint32_t off_step = lin ? (uint32_t)(PIX * P.C) : (uint32_t)(((dn * P.H + doh * P.sh) * P.W + dow * P.sw) * P.C);
    const uint32_t wrap_w = (uint32_t)((P.sh * P.W - P.Q * P.sw) * P.C);
    const uint32_t wrap_h = (uint32_t)((P.H - P.P * P.sh) * P.W * P.C);
    const int step_w = dow * P.sw, step_h = doh * P.sh, span_w = P.Q * P.sw, span_h = P.P * P.sh;
#pragma unroll
    for (int i = 0; i < T::XPW; i++) {
        const int p = (wave * T::XPW + i) * 8 + (lane >> 3);
        const int col = c0 + 16 * ((lane & 7) ^ swz<TBC>(p));
        const bool cok = col < (P.win ? P.ncol_w : P.ncol);
        const int cc = cok ? col : 0;
        int tdh = 0, tdw = 0;
        uint32_t toff;
        if (P.win) {
            const int r = cc >> window_log(P);
            toff = (uint32_t)(r * P.W * P.C + (cc - r * P.Lw));
        } else {
            const int r = (int)fdiv((uint32_t)cc, P.div_l);
            const int jj = cc - r * P.L;
            const int s = (int)fdiv((uint32_t)jj, P.div_c);
            tdh = r - P.ph;
            tdw = s - P.pw;
            toff = (uint32_t)(jj - s * P.C);
        }
        const int pix = pbeg + p;
        const int n = (int)fdiv((uint32_t)pix, P.div_pq);
        const int rem = pix - n * pq;
        const int oh = (int)fdiv((uint32_t)rem, P.div_q);
        const int ow = rem - oh * P.Q;
        ih[i] = oh * P.sh + tdh;
        iw[i] = ow * P.sw + tdw;
        xoff[i] = (uint32_t)(((n * P.H + ih[i]) * P.W + iw[i]) * P.C) + toff;
        lim_h[i] = span_h + tdh;
        lim_w[i] = span_w + tdw;
        if (!cok) {   // a column past the edge: never inside
            if (P.win || lin)
                xoff[i] = kOOB;
            else
                ih[i] = -(1 << 30), lim_h[i] = 1 << 30;
        }
    }
    constexpr int PPB = 1024 / TBK, CPR = TBK / 16;   // dy: pixels per block, chunks per row
#pragma unroll
    for (int i = 0; i < T::DPW; i++) {
        const int p = (wave * T::DPW + i) * PPB + lane / CPR;
        const int k = k0 + 16 * ((lane % CPR) ^ swz<TBK>(p));
        doff[i] = k < P.K ? (uint32_t)(pbeg + p) * (uint32_t)P.K + (uint32_t)k : kOOB;
    }

    int next = 0;
    const uint32_t xdst = lds0 + (uint32_t)(wave * T::XPW) * 1024u;
    const uint32_t ddst = lds0 + (uint32_t)(T::XBLK + wave * T::DPW) * 1024u;
    // kOOB offsets of channels and columns past the edge move too and may come
    // round to the buffer: what they load is in bounds and ends in sums that
    // are not stored.  Where all sums enter the maximum they must not
    // (wgrad_twice_eligible).
    auto issue = [&]() {
        const uint32_t slot = (uint32_t)((next % NS) * T::STAGE);
#pragma unroll
        for (int i = 0; i < T::XPW; i++) {
            const bool in = P.win || lin || ((unsigned)ih[i] < (unsigned)P.H && (unsigned)iw[i] < (unsigned)P.W);
            lds_dma16_at(xrs, xdst, slot + i * 1024, in ? xoff[i] : kOOB, 0);
            xoff[i] += off_step;
            if (!lin) {
                iw[i] += step_w;
                ih[i] += step_h;
                const bool ww = iw[i] >= lim_w[i];
                iw[i] -= ww ? span_w : 0;
                ih[i] += ww ? P.sh : 0;
                xoff[i] += ww ? wrap_w : 0u;
                const bool wh = ih[i] >= lim_h[i];
                ih[i] -= wh ? span_h : 0;
                xoff[i] += wh ? wrap_h : 0u;
            }
        }
#pragma unroll
        for (int i = 0; i < T::DPW; i++) {
            lds_dma16_at(drs, ddst, slot + i * 1024, doff[i], 0);
            doff[i] += (uint32_t)(PIX * P.K);
        }
        next++;
    };

    v16i acc[T::FC][T::FK];
#pragma unroll
    for (int a = 0; a < T::FC; a++)
#pragma unroll
        for (int b = 0; b < T::FK; b++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[a][b][e] = 0;

#pragma unroll
    for (int s = 0; s < NS - 1; s++) issue();
    // The weights this lane updates (16 consecutive columns per fragment, see
    // the epilogue), on their way during the contraction.
    uint4 wold[EP >= 0 ? T::FC : 1][T::FK];
    auto weight_at = [&](int a, int b, int& k, int& col) {
        k = k0 + wk * T::WTK + b * 32 + (lane & 31);
        col = c0 + wc * T::WTC + a * 32 + 16 * (lane >> 5);
        return k < P.K && col < P.ncol;   // ncol % 16 == 0
    };
    if constexpr (EP >= 0) {
#pragma unroll
        for (int a = 0; a < T::FC; a++)
#pragma unroll
            for (int b = 0; b < T::FK; b++) {
                int k, col;
                wold[a][b] = weight_at(a, b, k, col) ? *(const uint4*)(fin.w + (int64_t)k * P.ncol + col)
                                                     : make_uint4(0, 0, 0, 0);
            }
    }
    for (int it = 0; it < nsteps; it++) {
        wait_vm<(NS - 2) * T::IPW>();
        __builtin_amdgcn_s_barrier();
        issue();
        const int8_t* st = lds + (it % NS) * T::STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            v4i fa[T::FC], fb[T::FK];
#pragma unroll
            for (int a = 0; a < T::FC; a++) fa[a] = tr_fragment<TBC>(st, 32 * ks, wc * T::WTC + a * 32, lane);
#pragma unroll
            for (int b = 0; b < T::FK; b++)
                fb[b] = tr_fragment<TBK>(st + T::XBYTES, 32 * ks, wk * T::WTK + b * 32, lane);
#pragma unroll
            for (int a = 0; a < T::FC; a++)
#pragma unroll
                for (int b = 0; b < T::FK; b++)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
    }
    wait_vm<0>();

    if constexpr (EP == kMaxOnly) {
        // columns and channels past the edge accumulated zeros
#pragma unroll
        for (int a = 0; a < T::FC; a++)
#pragma unroll
            for (int b = 0; b < T::FK; b++)
#pragma unroll
                for (int e = 0; e < 16; e++) tmax = max(tmax, mag32(acc[a][b][e]));
        return;
    }
    if constexpr (EP >= 0) {
#pragma unroll
        for (int b = 0; b < T::FK; b++) {
            const int k = k0 + wk * T::WTK + b * 32 + (lane & 31);
#pragma unroll
            for (int a = 0; a < T::FC; a++) {
                // The lane holds old weights of sixteen consecutive columns
                // (lanes 0..31 columns 0..15 of the fragment, lanes 32..63
                // 16..31); two half-wave swaps (lanes 32..63 of the first
                // operand with lanes 0..31 of the second) give it the words
                // its accumulators belong to (word jj: columns 8 jj +
                // 4 (lane / 32) ..), and the same swaps undo that.
                const uint4 o = wold[a][b];
                const auto o02 = __builtin_amdgcn_permlane32_swap(o.x, o.y, false, false);
                const auto o13 = __builtin_amdgcn_permlane32_swap(o.z, o.w, false, false);
                const uint32_t ow[4] = {o02[0], o13[0], o02[1], o13[1]};
                uint32_t nw[4];
#pragma unroll
                for (int jj = 0; jj < 4; jj++) {
                    const int32_t g[4] = {acc[a][b][4 * jj], acc[a][b][4 * jj + 1], acc[a][b][4 * jj + 2],
                                          acc[a][b][4 * jj + 3]};
                    const int cl = c0 + wc * T::WTC + a * 32 + 8 * jj + 4 * (lane >> 5);
                    nw[jj] = update_word<EP>(ow[jj], g, rk, (uint64_t)k * P.ncol + cl);
                }
                const auto n02 = __builtin_amdgcn_permlane32_swap(nw[0], nw[2], false, false);
                const auto n13 = __builtin_amdgcn_permlane32_swap(nw[1], nw[3], false, false);
                int kw, col;
                if (weight_at(a, b, kw, col))
                    *(uint4*)(fin.w + (int64_t)kw * P.ncol + col) = make_uint4(n02[0], n02[1], n13[0], n13[1]);
            }
        }
        return;
    }
    // acc[a][b] element 4*jj + i: column c0 + wc*WTC + a*32 + 8*jj + 4*(lane/32) + i,
    // channel k0 + wk*WTK + b*32 + lane%32: four consecutive columns per store.
    // Rows and column groups are multiples of four (channels are, and L in
    // window mode) and the partial sums 16-byte aligned, so every store is
    // whole.  A test for it made the compiler move the stores out of line, and
    // sixteen jumps to code not yet in the instruction cache cost ~1.3 us per
    // launch (192 -> 208 channels, 2 pixels: 6.6 against 5.3 us).
    int32_t* out = P.part + (int64_t)split * P.K * P.ncol;
    const int lw_log = window_log(P);
#pragma unroll
    for (int b = 0; b < T::FK; b++) {
        const int k = k0 + wk * T::WTK + b * 32 + (lane & 31);
        if (k >= P.K) continue;
        int32_t* grow = out + (int64_t)k * P.ncol;
#pragma unroll
        for (int a = 0; a < T::FC; a++)
#pragma unroll
            for (int jj = 0; jj < 4; jj++) {
                int cidx = c0 + wc * T::WTC + a * 32 + 8 * jj + 4 * (lane >> 5);
                if (P.win) {
                    // window column r*Lw + j -> stored column r*L + j, j < L (groups of 4 stay whole)
                    if (cidx >= P.ncol_w) continue;
                    const int r = cidx >> lw_log, j = cidx - (r << lw_log);
                    if (j >= P.L) continue;
                    cidx = r * P.L + j;
                }
                if (cidx >= P.ncol) continue;
                *(int4*)(grow + cidx) = make_int4(acc[a][b][4 * jj], acc[a][b][4 * jj + 1], acc[a][b][4 * jj + 2],
                                                  acc[a][b][4 * jj + 3]);
            }
    }
}

// Workgroup order.  Workgroups go to the eight XCDs (each with its own L2)
// in turn by linear index, so workgroup L runs on XCD L % 8.  The work items
// (split, tile), tile fastest, are cut into eight equal consecutive runs, one
// per XCD: the output tiles of one pixel range, which read the same input
// pixels (shifted per tap) and the same errors, then mostly share an XCD and
// meet in its L2, and every XCD gets the same amount of work.  A grid smaller
// than the item count strides over its XCD's run.
template <int TBK, int TBC, int NS, int EP>
__global__ __launch_bounds__(256, 1) void wgrad_dma_kernel(WgradProblem P, int tiles_c, int tiles_k, int splits,
                                                           WgradFinish fin) {
    extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
    const int ntiles = tiles_c * tiles_k;
    const int per_xcd = (ntiles * splits + 7) / 8;
    int slot = 0;
    RoundK rk{};
    if constexpr (EP == kMaxOnly) {
        slot = call_slot(fin.st);
        begin_call(fin.st, slot, -1);
    }
    if constexpr (EP >= 0) {
        rk = make_round(block_bp(shared_call_state(fin.st, lds).mx, fin.mu), EP);
        sr_key_recorded(rk, fin.st);
    }
    uint32_t tmax = 0;
    if constexpr (EP == kStore) {   // one item per workgroup
        const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
        if ((blockIdx.x >> 3) >= per_xcd || item >= ntiles * splits) return;
        const int split = item / ntiles;
        const int tile = item - split * ntiles;
        wgrad_tile<TBK, TBC, NS, EP>(P, lds, split, (tile % tiles_c) * TBC, (tile / tiles_c) * TBK, fin, rk, tmax);
        return;
    }
    for (int s = blockIdx.x >> 3; s < per_xcd; s += gridDim.x >> 3) {
        const int item = (blockIdx.x & 7) * per_xcd + s;
        if (item >= ntiles * splits) break;
        const int split = item / ntiles;
        const int tile = item - split * ntiles;
        wgrad_tile<TBK, TBC, NS, EP>(P, lds, split, (tile % tiles_c) * TBC, (tile / tiles_c) * TBK, fin, rk, tmax);
        __syncthreads();   // the ring is free for the next tile
    }
    if constexpr (EP == kMaxOnly) {
        const uint64_t snap = max_snapshot(fin.st, slot);
        block_publish_max32(fin.st, slot, tmax, (uint32_t*)lds, snap);   // magnitudes <= 2^31
    }
    if constexpr (EP >= 0) {
        if (is_finisher()) finish_call(fin.st, fin.mu, ExpArgs{nullptr, nullptr, nullptr}, fin.static_flags, 0);
    }
}

template <int TBK, int TBC, int NS, int EP>
hipError_t launch(const WgradProblem& p, const WgradPlan& plan, hipStream_t stream, WgradFinish fin = WgradFinish{}) {
    using T = WCfg<TBK, TBC, NS>;
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute((const void*)wgrad_dma_kernel<TBK, TBC, NS, EP>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
        if (e != hipSuccess) return e;
        attr_done = true;
    }
    const int tc = ((p.win ? p.ncol_w : p.ncol) + TBC - 1) / TBC;
    const int tk = (p.K + TBK - 1) / TBK;
    int64_t grid = (int64_t)8 * (((int64_t)tc * tk * plan.splits + 7) / 8);
    // Each workgroup of a call's maximum or update launch goes to the one
    // statistics line, where requests queue at several nanoseconds each: two
    // per CU and no more.
    if (EP != kStore && grid > 512) grid = 512;
    const int t = timing_on() ? timing_begin(NITI_TIMING_KERNEL, stream,
                                             kernel_label("wgrad_dma_kernel<%d,%d,%d,%d>", TBK, TBC, NS, EP))
                              : -1;
    hipLaunchKernelGGL((wgrad_dma_kernel<TBK, TBC, NS, EP>), dim3((unsigned)grid), dim3(256), T::LDS, stream, p, tc, tk,
                       plan.splits, fin);
    timing_end(t, stream);
    return hipGetLastError();
}

}  // namespace

bool wgrad_dma_eligible(const WgradProblem& p) {
    const bool cols = p.win ? (p.Lw % 16 == 0 && p.L % 4 == 0 && p.ph == 0 && p.pw == 0) : p.C % 16 == 0;
    // The ring runs up to four stages past the last pixel.  The error offsets it
    // forms there must lie past the buffer, also mod 2^32: their zeros cancel
    // whatever the input offsets of such pixels meet in their own buffer.
    return cols && p.K % 16 == 0 && p.x_bytes > 0 && p.x_bytes < ((int64_t)1 << 31) && p.dy_bytes > 0 &&
           p.dy_bytes < ((int64_t)1 << 31) && p.dy_bytes + kOver * p.K < ((int64_t)1 << 32);
}

hipError_t wgrad_dma_run(WgradProblem& p, const WgradPlan& plan, hipStream_t stream) {
    p.chunk = plan.chunk;
    if (plan.tbk == 64) return launch<64, 128, 4, kStore>(p, plan, stream);
    return launch<128, 128, 4, kStore>(p, plan, stream);
}

// Running the contraction again costs its 2 npix operations per weight and its
// latency once more, on as many CUs as it has tiles, and saves the int32
// gradient's round trips: 12 bytes per weight (written, read for the maximum,
// read for the update) by kernels that always fill the chip.  So it pays from a
// number of weights on that grows with the samples.  Stochastic rounding's 64-bit
// draws are the dearer part of the epilogue on few CUs, and with 32 channels or
// fewer most of a tile's epilogue is for rows that do not exist.  The limits
// are the best of a grid over 285 (94 for stochastic rounding) random layers:
// at most 9% (14%) off the better form.  Whole calls in us, stored / twice:
// 4096 -> 4096, 128 samples 61.0 / 31.4; 1808 -> 720, 53 samples 18.3 / 10.6;
// 304 -> 48, 464 samples 9.6 / 11.6; 80 -> 448, 294 samples, stochastic 10.3 /
// 14.9; 8256 -> 16, 5x5, 98 pixels, stochastic 27.7 / 33.5; 5616 -> 16, 3x3, 240
// pixels 14.8 / 16.0.
bool wgrad_twice_eligible(const WgradProblem& p, const WgradPlan& plan, int mode) {
    if (plan.splits != 1 || p.win || p.npix > 512 || p.K <= 32 || !wgrad_dma_eligible(p)) return false;
    const int64_t edge = p.K > p.C ? p.K : p.C;   // offsets past the edge stay past the buffers
    if ((p.npix + kOver) * edge >= ((int64_t)1 << 31)) return false;
    const int64_t weights = (int64_t)p.K * p.ncol;
    return mode == NITI_ROUND_SR ? weights >= (1 << 17) + (int64_t)2048 * p.npix
                                 : weights >= (1 << 15) + (int64_t)512 * p.npix;
}

hipError_t wgrad_twice_run(WgradProblem& p, const WgradPlan& plan, int8_t* w, int mu, int mode, niti_stats* st,
                           uint32_t static_flags, hipStream_t stream) {
    p.chunk = plan.chunk;
    // Three stages: a batch of 128 samples is two, so the whole reduction is in
    // flight at once and a fourth would only load zeros.
    const WgradFinish fin{w, st, mu, static_flags};
#define NITI_TWICE(EP) (plan.tbk == 64 ? launch<64, 128, 3, EP>(p, plan, stream, fin) : launch<128, 128, 3, EP>(p, plan, stream, fin))
    hipError_t e = NITI_TWICE(kMaxOnly);
    if (e != hipSuccess) return e;
    if (mode == NITI_ROUND_SR) return NITI_TWICE(NITI_ROUND_SR);
    if (mode == NITI_ROUND_RTN) return NITI_TWICE(NITI_ROUND_RTN);
    return NITI_TWICE(NITI_ROUND_PSR);
#undef NITI_TWICE
}

}  // namespace niti
