// Implicit-GEMM convolution with fp32 operands split into three bf16 parts
// (v_mfma_f32_32x32x16_bf16).
//
// gfx950's bf16 matrix instructions do 16 times the multiply-adds of its fp32
// ones per cycle.  An fp32 value of 2^-109 and more is the sum of three bf16
// values,
//   h = bf16(x), m = bf16(x - h), l = bf16(x - h - m),
// exactly (24 significand bits in three parts of 8, each rounded to nearest,
// so each remainder has a sign of its own), and a product x*w is
//   xh*wh + (xh*wm + xm*wh) + (xm*wm + xh*wl + xl*wh) + terms below 2^-24 |x*w|.
// So six bf16 products replace one fp32 product: 2.7 times the fp32 matrix
// rate.  The products of bf16 values are exact in fp32, and the leading
// product has an accumulator of its own (the five small ones, 2^-8 and less of
// it, share another): the rounding of the accumulation is then that of one
// addition per 16 terms where the fp32 instructions round once per term.
// Measured against 64 bits, 2-norm, against the fp32 kernels that ran the layer
// before: 0.3 times their error on 3x3 64->64 at 224^2 (1.4e-7, 4.5e-7) and
// 128->128 at 112^2, 0.4 on 64->96 at 301x403 and 75->150 at 61x45, 0.55 on 1x1
// 256->128 at 56^2; one chain of 12800 terms 7.2e-7 against 2.1e-6.  (With one
// accumulator for all six products 0.85 times and a bias of a third of that.)
//
// Two limits of the split, and what is done about them.  A value whose bf16
// rounding overflows, an infinity or a NaN gives NaN parts, so every output
// it touches is not finite; such outputs are computed again with fp32 matrix
// instructions before they are stored (at the kernel's end), which gives what
// the fp32 kernels give.  And bf16 ends at 2^-133: a value below 2^-109 in
// magnitude keeps an absolute error of at most 2^-134, which ilpm.h states.
// (Both operands scaled by 2^24 at their splitting, two multiplications a pair
// and the outputs scaled back, would keep all bits of every value; it made the
// measured layers 2-7% slower.)
//
// GEMM view: rows = output channels, columns = output pixels, contraction =
// input channels x taps: a store instruction then writes 32 consecutive pixels
// of two output channels, whole 64-byte pieces whatever the tile's alignment.
// (The other way round a lane holds four consecutive pixels of one channel;
// stored one by one where they are not aligned they cost 30 us on 64->64 at
// 224^2.)  With the 2x2 max-pool in the kernel the roles are swapped and the
// tile's pixels (slots) numbered window by window, so that a window is four of
// a lane's own registers.  Both ways give the same sums bit for bit.
//
// A stage is CC input channels, in two LDS buffers.  While a stage computes,
// the next one's weights fly into LDS by DMA as they are (fp32), and its halo
// pixels into registers; those are split once per workgroup and written to
// LDS in the middle of the stage.  One barrier ends the stage.
//   pixels   [8-channel group][halo pixel][part][8 channels]  (bf16)
//   weights  OIHW: [8-channel group][output channel] runs of 8*K*K floats (see
//            SplitCfg); prepacked: [unit][half][output channel][4 channels],
//            unit = (tap, 8-channel group)
// A step is two units, one per half of the matrix instruction's lanes, so with
// 16-channel stages a step is a tap and no product is spent on padding (the
// 16x16x32 instruction takes four units a step: 18 of them in 5 steps).  For
// each step a wave reads its weights (8 per lane) two steps ahead, splits them
// during the step before and runs all its pixel blocks with them.  Splitting
// the weights at their use costs 44 VALU instructions per step, placed one by
// one beside its 6*NB matrix instructions of 32 cycles (NB = 1 to 4 pixel
// blocks; a burst of them before the matrix instructions costs more), and as
// many times over as waves share an output channel: a quarter to a third of a
// 3x3 stage; splitting them once on the way into LDS measured
// slower: a serial phase per stage of 1.5 us (prepacked) to 3.3 us (OIHW,
// through a transposition in LDS) against 1.9 us of matrix work, which two
// workgroups per compute unit, in step with each other, did not hide.
// The tile is TH x TW output pixels, chosen per shape when the plan is made,
// at most PX of them; stride and tile only enter through two small tables in
// LDS (slot -> halo pixel, slot -> output).
//
// gfx950 serves a ds_read_b128 16 lanes at a time over 64 banks: lanes 0-3,
// 12-15, 20-23 and 24-27 together, then the other 16 of the first 32.  At 48
// bytes between lanes each 16 are on different banks (measured: 185 bytes per
// cycle and compute unit; 120 where two lanes of a group share a bank).
#pragma once

#include "conv_igemm.h"

namespace ilpm {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int cmin(int a, int b) { return a < b ? a : b; }

template <int KS_, int S_, int CC_, int MA_, int NB_, int WC_, int WP_, int WK_, int XPIX_, int WPE_ = 2>
struct SplitCfg {
    static constexpr int KS = KS_, S = S_, CC = CC_;
    static constexpr int MA = MA_;  // 32-channel blocks per wave
    static constexpr int NB = NB_;  // 32-pixel blocks per wave
    static constexpr int WC = WC_, WP = WP_, WK = WK_;  // waves over channels, pixels, steps
    static constexpr int XPIX = XPIX_;  // most halo pixels of a tile
    static constexpr int WPE = WPE_;    // wavefronts per SIMD the registers are budgeted for
    static constexpr int NW = WC * WP * WK, NT = 64 * NW;
    static constexpr int COT = 32 * MA * WC, PX = 32 * NB * WP;
    static constexpr int KK = KS * KS, C8 = CC / 8;
    // Halo pixels between output pixels (1x1 filters load only the pixels they
    // use, every SplitTile::step-th, and so take any stride).
    static constexpr int OS = KS == 1 ? 1 : S;
    static constexpr int U = KK * C8;            // units per stage
    static constexpr int NSTEP = (U + 1) / 2;    // steps per stage
    static constexpr int PXB = 48;                              // bytes per halo pixel and 8-channel group
    static constexpr int XPL = (XPIX * PXB + 255) / 256 * 256;  // bytes per 8-channel group
    static constexpr int XB = C8 * XPL + 256;  // and room for what lanes without a pixel write
    static constexpr int ROW = CC * KK;          // floats per OIHW row of a stage
    // OIHW weights in LDS: a run of RUN floats per (output channel, 8-channel
    // group) -- for 1x1 filters the whole row -- in 16-byte pieces.  32 lanes
    // (output channels) read one float each of their runs: with an odd number
    // of pieces per run the lanes of 8 output channels are 4 banks apart, and a
    // run starts run_shift floats into its first piece, which puts the other 24
    // on the banks between.
    static constexpr int RUN = KK > 1 ? 8 * KK : ROW, NRUN = ROW / RUN;
    static constexpr int RQ = KK > 1 ? (RUN + 3 + 3) / 4 : ROW / 4 + 1;  // pieces per run
    static_assert(RQ % 2 == 1, "runs of an odd number of pieces");
    __device__ static constexpr int run_shift(int co) { return KK > 1 ? co >> 3 & 3 : 0; }
    static constexpr int RUNB = RQ * 16;         // bytes per run
    static constexpr int WQ = COT * NRUN * RQ;   // pieces of a stage (prepacked: COT * ROW / 4, fewer)
    static constexpr int WJ = (WQ + 64 * NW - 1) / (64 * NW);  // DMA instructions of a stage per wave
    static constexpr int WB = WJ * NW * 1024;
    static constexpr int XI = (XPIX * C8 + NT - 1) / NT;   // pixel items (8 channels) per thread
    // The end: a wave's sums are ITEMS items (block b, quad q: four registers)
    // per channel block, item e = 4*b + q; with WK > 1 wave wk = e mod WK adds
    // up the item's partial sums, EG groups of WK items at a time through the
    // pixel buffers.
    static constexpr int ITEMS = 4 * NB;
    static_assert(ITEMS % WK == 0, "every wave finishes as many items");
    static constexpr int GROUPS = ITEMS / WK;
    static constexpr int EG = cmin(GROUPS, 2 * XB / (NW * cmax(WK - 1, 1) * MA * 1024));
    static_assert(EG >= 1, "room for one group of partial sums");
    static constexpr int LDS_BYTES = 2 * (XB + WB) + PX * 8;
    static_assert(CC % 8 == 0 && (C8 == 1 || C8 % 2 == 0), "units of a step share a tap or are two taps");
    static_assert(ROW % 4 == 0, "rows of whole 16-byte pieces");
    static_assert(LDS_BYTES <= 160 * 1024 && NT <= 1024 && PX <= NT, "LDS and workgroup size");
};

typedef unsigned uint4v __attribute__((ext_vector_type(4)));

// Two fp32 values rounded to bf16, the first in the low half.
__device__ __forceinline__ unsigned bf16_pair(float a, float b)
{
    typedef float float2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const float2v f = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}

// Two fp32 values -> their bf16 parts, packed (11 instructions).
__device__ __forceinline__ void split_two(float a, float b, unsigned &h, unsigned &m, unsigned &l)
{
    h = bf16_pair(a, b);
    const float ra = a - __builtin_bit_cast(float, h << 16);
    const float rb = b - __builtin_bit_cast(float, h & 0xffff0000u);
    m = bf16_pair(ra, rb);
    l = bf16_pair(ra - __builtin_bit_cast(float, m << 16), rb - __builtin_bit_cast(float, m & 0xffff0000u));
}

// split_two as single steps, to be placed between matrix instructions: step k
// (0..10) of pair p = 4*m + i, the values v[m][2*i], v[m][2*i+1].
struct SplitOps {
    unsigned h, m, l;
    float ta, tb, ra, rb;
    template <int MA>
    __device__ __forceinline__ void op(int k, int p, unsigned __attribute__((ext_vector_type(4))) (&f)[MA][3],
                                       const float (&v)[MA][8])
    {
        const int b = p / 4, i = p % 4;
        switch (k) {
        case 0: h = bf16_pair(v[b][2 * i], v[b][2 * i + 1]); break;
        case 1: ta = __builtin_bit_cast(float, h << 16); break;
        case 2: tb = __builtin_bit_cast(float, h & 0xffff0000u); break;
        case 3: ra = v[b][2 * i] - ta; break;
        case 4: rb = v[b][2 * i + 1] - tb; break;
        case 5: m = bf16_pair(ra, rb); break;
        case 6: ta = __builtin_bit_cast(float, m << 16); break;
        case 7: tb = __builtin_bit_cast(float, m & 0xffff0000u); break;
        case 8: ra -= ta; break;
        case 9: rb -= tb; break;
        default:
            l = bf16_pair(ra, rb);
            // (Opaque, or the compiler moves all of it to where it is used.)
            asm volatile("" : "+v"(h), "+v"(m), "+v"(l));
            f[b][0][i] = h;
            f[b][1][i] = m;
            f[b][2][i] = l;
        }
    }
};

// Eight fp32 values -> their three bf16 parts.
struct Parts {
    uint4v h, m, l;
};
__device__ __forceinline__ Parts split_parts(const float (&v)[8])
{
    Parts p;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned h, m, l;
        split_two(v[2 * i], v[2 * i + 1], h, m, l);
        p.h[i] = h;
        p.m[i] = m;
        p.l[i] = l;
    }
    return p;
}

// This wave's loads but the K latest, and its LDS accesses, are complete; then
// every wave's.
template <int K>
__device__ __forceinline__ void stage_ready_keep_lds()
{
    static_assert(K >= 0 && K < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0x0070 | (K & 15) | ((K >> 4) << 14));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ bool not_finite(float v) { return !(__builtin_fabsf(v) < __builtin_inff()); }

// Tile pixel of a slot: row by row, or (pooled) window by window, a window's
// four pixels in the order (0,0), (0,1), (1,0), (1,1).  tile.tw_d divides by
// TW, pooled by TW / 2.
template <bool POOL>
__device__ __forceinline__ void slot_pixel(int slot, const SplitTile &t, int &r, int &c)
{
    if constexpr (POOL) {
        const int q = slot >> 2;
        const int wr = (int)fast_div((unsigned)q, t.tw_d);
        const int wc = q - wr * (int)t.tw_d.d;
        r = 2 * wr + ((slot >> 1) & 1);
        c = 2 * wc + (slot & 1);
    } else {
        r = (int)fast_div((unsigned)slot, t.tw_d);
        c = slot - r * (int)t.tw_d.d;
    }
}

template <class C, bool PK, bool POOL>
__global__ __launch_bounds__(C::NT, C::WPE) void conv_split(const float *__restrict__ x, const float *__restrict__ w,
                                                            const float *__restrict__ bias, float *__restrict__ out,
                                                            float *__restrict__ part, IgArgs a, SplitTile t)
{
    // The two weight buffers as objects of their own, so that the compiler can
    // tell a read of one from the DMA filling the other.
    __shared__ __attribute__((aligned(256))) char xs[2 * C::XB];
    char *const x0 = xs, *const x1 = xs + C::XB;
    __shared__ __attribute__((aligned(256))) char w0[C::WB];
    __shared__ __attribute__((aligned(256))) char w1[C::WB];
    __shared__ __attribute__((aligned(16))) int s_in[C::PX];   // slot -> byte offset of its halo pixel
    __shared__ __attribute__((aligned(16))) int s_out[C::PX];  // slot -> output element (pooled: of its window)

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __builtin_assume(wave >= 0 && wave < C::NW);
    const int wc = wave % C::WC;
    const int wp = (wave / C::WC) % C::WP;
    const int wk = wave / (C::WC * C::WP);
    const int g = lane >> 5;
    const int l32 = lane & 31;

    // Workgroup -> (split, tile), contiguous runs of tiles per XCD (as in
    // conv_igemm).
    const int nwg = (int)gridDim.x;
    const int xcd = (int)blockIdx.x % 8, slot8 = (int)blockIdx.x / 8;
    const int per = nwg / 8, extra = nwg % 8;
    const int lin = xcd * per + min(xcd, extra) + slot8;
    const int split = (int)fast_div((unsigned)lin, a.ntiles);
    const int tile = lin - split * (int)a.ntiles.d;
    int sp, co_t;
    if (a.sp_fast) {
        co_t = (int)fast_div((unsigned)tile, a.sp_tiles);
        sp = tile - co_t * (int)a.sp_tiles.d;
    } else {
        sp = (int)fast_div((unsigned)tile, a.co_tiles);
        co_t = tile - sp * (int)a.co_tiles.d;
    }
    const int th_i = (int)fast_div((unsigned)sp, a.tiles_w);
    const int tw_i = sp - th_i * (int)a.tiles_w.d;
    const int co0 = co_t * C::COT;
    const int oh0 = th_i * t.th, ow0 = tw_i * t.tw;
    const int c_begin = split * a.chunks_per_split;
    const int c_end = min(c_begin + a.chunks_per_split, a.nchunks);

    // Pixel items of this thread: halo pixel p, 8-channel group c8.  Offsets
    // outside the image start at 2^31, past every descriptor's range whatever
    // channel offset is added.
    const int stride = C::KS == 1 ? t.step : C::S;
    const int hc = (int)t.hc_d.d, npix = (int)t.npix_d.d;
    const unsigned plane4 = (unsigned)a.h * (unsigned)a.w * 4u;
    unsigned xoff[C::XI];
    int xlds[C::XI];
#pragma unroll
    for (int j = 0; j < C::XI; ++j) {
        const int idx = j * C::NT + tid;
        const int c8 = (int)fast_div((unsigned)idx, t.npix_d);
        const int p = idx - c8 * npix;
        const int hr = (int)fast_div((unsigned)p, t.hc_d);
        const int ih = oh0 * stride - a.pad + hr * t.step, iw = ow0 * stride - a.pad + (p - hr * hc) * t.step;
        const bool ok = c8 < C::C8 && ih >= 0 && ih < a.h && iw >= 0 && iw < a.w;
        xoff[j] = ok ? (unsigned)(ih * a.w + iw) * 4u + (unsigned)(8 * c8) * plane4 : 0x80000000u;
        xlds[j] = c8 < C::C8 ? p * C::PXB + c8 * C::XPL : C::C8 * C::XPL;
    }
    float xr[C::XI][8];
    // The input from a chunk on; for chunks past this split's last one an
    // empty range (the loads are issued all the same, read zeros and touch no
    // memory: with the same loads in flight on every path the compiler's waits
    // for them are exact.  Where the last stage is compiled on its own, its
    // pixel loads, whose values nothing reads, go; its weight DMA, of an empty
    // range too, may then still be in flight after it, so nothing may use the
    // weight buffers again).
    auto chunk_rsrc = [&](int chunk) {
        const int ci0 = chunk * C::CC;
        return make_rsrc(x + (size_t)ci0 * (plane4 / 4u), chunk < c_end ? (unsigned)(a.c_in - ci0) * plane4 : 0u);
    };
    auto load_item = [&](int j, const __amdgpu_buffer_rsrc_t &rx) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            xr[j][e] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rx, (int)(xoff[j] + (unsigned)e * plane4), 0, 0));
    };
    auto load_x = [&](int chunk) {
        const __amdgpu_buffer_rsrc_t rx = chunk_rsrc(chunk);
#pragma unroll
        for (int j = 0; j < C::XI; ++j) load_item(j, rx);
    };
    auto put_item = [&](char *buf, int j, const uint4v &h, const uint4v &m, const uint4v &l) {
        uint4v *d = reinterpret_cast<uint4v *>(buf + xlds[j]);
        d[0] = h;
        d[1] = m;
        d[2] = l;
    };

    // Weights: 16-byte piece idx of a stage lands at byte 16*idx of the
    // buffer.  OIHW: piece q of run (co, c8), idx = (c8*COT + co)*RQ + q.  A
    // run's first and last pieces also hold floats next to it, and in the last
    // stage a run may reach past C_in.  Floats past the tensor read 0 (the
    // range check is per 4 bytes).
    const unsigned wrow = (unsigned)a.c_in * C::KK;  // floats per OIHW row
    const float *const w_packed = w + (size_t)co_t * a.nchunks * (C::COT * C::ROW);
    unsigned woff[PK ? 1 : C::WJ];
    if constexpr (PK) woff[0] = (unsigned)(wave * 64 + lane) * 16u;
#pragma unroll
    for (int j = 0; j < C::WJ; ++j) {
        const int idx = (j * C::NW + wave) * 64 + lane;
        if constexpr (!PK) {
            const int run = idx / C::RQ, q = idx - run * C::RQ;
            const int c8 = run / C::COT, co = run - c8 * C::COT;
            woff[j] = run < C::COT * C::NRUN
                          ? ((unsigned)(co0 + co) * wrow + (unsigned)(c8 * C::RUN + 4 * q - C::run_shift(co))) * 4u
                          : 0x80000000u;
        }
    }
    // Instructions j0 .. j1-1 (of WJ) of this wave.
    auto dma_w = [&](char *buf, int chunk, int j0, int j1) {
        const unsigned bytes = PK ? C::COT * C::ROW * 4u : (unsigned)a.c_out * wrow * 4u;
        const __amdgpu_buffer_rsrc_t rw =
            make_rsrc(PK ? w_packed + (size_t)chunk * (C::COT * C::ROW) : w, chunk < c_end ? bytes : 0u);
        const unsigned first = PK ? 0u : (unsigned)chunk * (C::ROW * 4u);
#pragma unroll
        for (int j = j0; j < j1; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr_t)(buf + (j * C::NW + wave) * 1024), 16,
                                                     (int)(PK ? woff[0] + (unsigned)(j * C::NW * 1024) : woff[j] + first),
                                                     0, 0, 0);
    };

    load_x(c_begin);
    dma_w(w0, c_begin, 0, C::WJ);

    // Slot tables.
    const int ho2 = POOL ? a.h_out / 2 : a.h_out, wo2 = POOL ? a.w_out / 2 : a.w_out;
    if (tid < C::PX) {
        int r, c;
        slot_pixel<POOL>(tid, t, r, c);
        const bool in = tid < t.th * t.tw;
        s_in[tid] = in ? (r * C::OS * hc + c * C::OS) * C::PXB : 0;
        int o = -1;
        if constexpr (POOL) {
            const int pr = (oh0 + r) >> 1, pc = (ow0 + c) >> 1;
            if (in && pr < ho2 && pc < wo2) o = pr * wo2 + pc;
        } else {
            if (in && oh0 + r < a.h_out && ow0 + c < a.w_out) o = (oh0 + r) * a.w_out + ow0 + c;
        }
        s_out[tid] = o;
    }

    floatx16 hi[C::NB][C::MA], lo[C::NB][C::MA];
#pragma unroll
    for (int b = 0; b < C::NB; ++b)
#pragma unroll
        for (int m = 0; m < C::MA; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) hi[b][m][r] = lo[b][m][r] = 0.f;

    int xb[C::NB];  // this lane's halo pixel of each block, plus its 8-channel group

    // Unit of this lane in step s, as (tap, 8-channel group); past the last
    // unit the last one (its weights are masked).
    auto unit_of = [&](int s, int &tap, int &c8) {
        if constexpr (C::C8 == 1) {
            tap = 2 * s + g;
            if (C::U % 2 != 0) tap = tap < C::KK ? tap : C::KK - 1;
            c8 = 0;
        } else {
            tap = s / (C::C8 / 2);
            c8 = s % (C::C8 / 2) * 2 + g;
        }
    };
    // Where its pixels lie: at xb[b] + px_off(s) (xb holds group c8 = g).
    auto px_off = [&](int s) -> int {
        int tap, c8;
        unit_of(s, tap, c8);
        const int group = C::C8 == 1 ? 0 : (c8 - g) * C::XPL;
        if constexpr (C::KS == 1) return group;
        const int kh = (tap * (65536 / C::KS + 1)) >> 16;
        return (kh * hc + (tap - kh * C::KS)) * C::PXB + group;
    };
    // Its weights as they are: 8 channels of its unit's tap, for each of the
    // lane's output channels.
    const int co_w = wc * 32 * C::MA + l32;
    auto read_w = [&](float (&v)[C::MA][8], const char *buf, int s) {
        int tap, c8;
        unit_of(s, tap, c8);
        if constexpr (!PK && C::KK > 1) {
            const float *p =
                reinterpret_cast<const float *>(buf + (c8 * C::COT + co_w) * C::RUNB) + C::run_shift(l32) + tap;
#pragma unroll
            for (int m = 0; m < C::MA; ++m)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[m][e] = p[m * (32 * C::RUNB / 4) + e * C::KK];
        } else {
            // Two pieces of 4 channels.
            const char *p = PK ? buf + (tap * C::C8 + c8) * (C::COT * 32) + co_w * 16 : buf + co_w * C::RUNB + c8 * 32;
            constexpr int next_m = PK ? 32 * 16 : 32 * C::RUNB, next_q = PK ? C::COT * 16 : 16;
#pragma unroll
            for (int m = 0; m < C::MA; ++m)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const floatx4 f = *reinterpret_cast<const floatx4 *>(p + m * next_m + q * next_q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[m][4 * q + e] = f[e];
                }
        }
    };
    // Pair p (of 4*MA) of a step's weights split: pairs m*4 + i, floats 2i, 2i+1.
    auto split_pair = [&](uint4v (&f)[C::MA][3], const float (&v)[C::MA][8], int p) {
        const int m = p / 4, i = p % 4;
        unsigned h, mid, l;
        split_two(v[m][2 * i], v[m][2 * i + 1], h, mid, l);
        f[m][0][i] = h;
        f[m][1][i] = mid;
        f[m][2][i] = l;
    };
    // Units past a stage's last one: zero weights.
    auto mask_w = [&](uint4v (&f)[C::MA][3], int s) {
        if (C::U % 2 != 0 && s == C::NSTEP - 1) {
            const unsigned keep = 2 * s + g < C::U ? ~0u : 0u;
#pragma unroll
            for (int m = 0; m < C::MA; ++m)
#pragma unroll
                for (int q = 0; q < 3; ++q) f[m][q] &= uint4v{keep, keep, keep, keep};
        }
    };
    auto read_x = [&](bf16x8 (&f)[3], const char *buf, int addr) {
#pragma unroll
        for (int q = 0; q < 3; ++q) f[q] = *reinterpret_cast<const bf16x8 *>(buf + addr + q * 16);
    };
    auto mul = [](bf16x8 fx, bf16x8 fw, floatx16 c) {
        return POOL ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx, fw, c, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw, fx, c, 0, 0, 0);
    };
    // One step: 6*MA*NB matrix instructions, and beside each its share of
    // splitting NX of the next stage's pixel items (J0, J0 + 1, ...; written to
    // xn) and then the next step's weights (wv -> nw), in exactly this order.
    // A block's small products come first, and the pixels' parts one after the
    // other, each replaced by the next block's after its last use, three
    // instructions or more before that one's first.  `between` is called after
    // each block for the loads it issues.
    auto step = [&](auto nx_c, auto j0_c, const char *xc, char *xn, int off, int noff, bf16x8 (&fx)[3],
                    const uint4v (&fw)[C::MA][3], uint4v (&nw)[C::MA][3], const float (&wv)[C::MA][8],
                    auto between) {
        constexpr int NX = decltype(nx_c)::value, J0 = decltype(j0_c)::value;
        constexpr int ix[6] = {2, 1, 1, 0, 0, 0}, iw[6] = {0, 1, 0, 2, 1, 0};
        constexpr int xops = 44 * NX, ops = xops + 44 * C::MA, slots = C::NB * 6 * C::MA;
        SplitOps so;
        uint4v xp[1][3];
#pragma unroll
        for (int b = 0; b < C::NB; ++b) {
            const char *next = xc + (b + 1 < C::NB ? xb[b + 1] + off : xb[0] + noff);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
#pragma unroll
                for (int m = 0; m < C::MA; ++m) {
                    floatx16 &c = k == 5 ? hi[b][m] : lo[b][m];
                    c = mul(fx[ix[k]], __builtin_bit_cast(bf16x8, fw[m][iw[k]]), c);
                    const int slot = (b * 6 + k) * C::MA + m;
#pragma unroll
                    for (int o = slot * ops / slots; o < (slot + 1) * ops / slots; ++o) {
                        if (o < xops) {
                            const float(&v)[1][8] = reinterpret_cast<const float(&)[1][8]>(xr[J0 + o / 44]);
                            so.op(o % 11, o / 11 % 4, xp, v);
                            if (o % 44 == 43) put_item(xn, J0 + o / 44, xp[0][0], xp[0][1], xp[0][2]);
                        } else {
                            so.op((o - xops) % 11, (o - xops) / 11, nw, wv);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (k == 5 || ix[k + 1] != ix[k]) {
                    fx[ix[k]] = *reinterpret_cast<const bf16x8 *>(next + ix[k] * 16);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            between(b);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // The first stage's pixels; every wave's DMA has landed at the barrier.
#pragma unroll
    for (int j = 0; j < C::XI; ++j) {
        const Parts p = split_parts(xr[j]);
        put_item(x0, j, p.h, p.m, p.l);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    load_x(c_begin + 1);
#pragma unroll
    for (int b = 0; b < C::NB; ++b)
        xb[b] = s_in[(wp * C::NB + b) * 32 + l32] + (C::C8 == 1 ? 0 : g * C::XPL);

    // The last stage's rows of OIHW weights may reach past C_in, into the next
    // row.  Its floats would meet pixels that read 0, which leaves the sums
    // alone unless one is not finite; zero them.
    auto clear_tail = [&](char *buf, int chunk) {
        const int valid = (a.c_in - chunk * C::CC) * C::KK;  // floats of a row that belong to it
        if (!PK && valid < C::ROW) {
            for (int i = tid; i < C::COT * C::ROW; i += C::NT) {
                const int co = i / C::ROW, k = i - co * C::ROW;
                const int c8 = k / C::RUN;
                if (k >= valid)
                    *(reinterpret_cast<float *>(buf + (c8 * C::COT + co) * C::RUNB) + C::run_shift(co) + k -
                      c8 * C::RUN) = 0.f;
            }
            lds_barrier();
        }
    };

    // One stage from (xc, wcur).  Meanwhile the next one's weights go to wn
    // and its pixels, loaded during the stage before, to xn, and the pixels of
    // the one after it are loaded, all of it spread over the stage's first
    // steps (issued together at its start the loads held the waves up, their
    // matrix pipe idle).  Steps go round robin over the WK waves, stage after
    // stage: `phase` is this wave's first one.  Every wave has at least MINS.
    constexpr int MINS = C::NSTEP / C::WK;
    static_assert(MINS >= 1, "every wave has a step in every stage");
    constexpr int NXS = (C::XI + MINS - 1) / MINS;  // pixel items per step
    int phase = wk;
    auto stage = [&](const char *xc, char *wcur, char *xn, char *wn, int chunk) {
        clear_tail(wcur, chunk);
        int s = phase;
        float wv[C::MA][8];
        uint4v fw[C::MA][3];
        bf16x8 fx[3];
        int off = px_off(s);
        read_w(wv, wcur, s);
        read_x(fx, xc, xb[0] + off);
#pragma unroll
        for (int p = 0; p < 4 * C::MA; ++p) split_pair(fw, wv, p);
        mask_w(fw, s);
        auto following = [&] { return s + C::WK < C::NSTEP ? s + C::WK : s; };
        read_w(wv, wcur, following());
        auto advance = [&](const uint4v (&nw)[C::MA][3], int noff) {
            s += C::WK;
            off = noff;
#pragma unroll
            for (int m = 0; m < C::MA; ++m)
#pragma unroll
                for (int q = 0; q < 3; ++q) fw[m][q] = nw[m][q];
            mask_w(fw, s);
            read_w(wv, wcur, following());
        };
        for_each_index(std::make_integer_sequence<int, MINS>{}, [&](auto ic) {
            constexpr int I = decltype(ic)::value;
            constexpr int J0 = cmin(I * NXS, C::XI), J1 = cmin(J0 + NXS, C::XI);
            uint4v nw[C::MA][3];
            const int noff = px_off(following());
            step(std::integral_constant<int, J1 - J0>{}, std::integral_constant<int, J0>{}, xc, xn, off, noff, fx, fw,
                 nw, wv, [&](int b) {
                     if (I == 0) {
                         dma_w(wn, chunk + 1, b * C::WJ / C::NB, (b + 1) * C::WJ / C::NB);
                         // stage_ready_keep_lds counts on the pixel loads following:
                         // no memory instruction passes here.
                         __builtin_amdgcn_sched_barrier(0x48f);
                     }
                     if (b == C::NB - 1 && J1 > J0) {
                         const __amdgpu_buffer_rsrc_t rx = chunk_rsrc(chunk + 2);
#pragma unroll
                         for (int j = J0; j < J1; ++j) load_item(j, rx);
                     }
                 });
            advance(nw, noff);
        });
        if (C::NSTEP % C::WK != 0 && s < C::NSTEP) {
            uint4v nw[C::MA][3];
            step(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, xc, xn, off, off, fx, fw, nw, wv,
                 [](int) {});
            s += C::WK;
        }
        phase = s - C::NSTEP;
        // This wave's DMA has landed; the pixel loads issued after it may
        // still fly.
        stage_ready_keep_lds<C::XI * 8>();
    };
    int chunk = c_begin;
    for (; chunk + 1 < c_end; chunk += 2) {
        stage(x0, w0, x1, w1, chunk);
        stage(x1, w1, x0, w0, chunk + 1);
    }
    if (chunk < c_end) stage(x0, w0, x1, w1, chunk);

    // The sums: item e = 4*b + q of channel block m is registers 4q..4q+3 of
    // block (b, m).  (Every wave has read the last stage: its barrier.)
    floatx4 sum[C::ITEMS][C::MA];
#pragma unroll
    for (int e = 0; e < C::ITEMS; ++e)
#pragma unroll
        for (int m = 0; m < C::MA; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float h = hi[e / 4][m][e % 4 * 4 + r], l = lo[e / 4][m][e % 4 * 4 + r];
                sum[e][m][r] = h + l;
            }
    floatx4 *const red = reinterpret_cast<floatx4 *>(xs);
    if constexpr (C::WK > 1) {
        // Where wave k puts its part of item e: k owns one item of each group
        // and writes the other WK - 1.
        auto red_at = [&](int k, int e, int m) -> floatx4 & {
            const int rank = (e % C::WK - k + C::WK) % C::WK - 1;
            return red[((((k * C::WP + wp) * C::WC + wc) * C::EG + e / C::WK % C::EG) * (C::WK - 1) + rank) *
                           (C::MA * 64) + m * 64 + lane];
        };
#pragma unroll
        for (int g0 = 0; g0 < C::GROUPS; g0 += C::EG) {
#pragma unroll
            for (int e = g0 * C::WK; e < cmin(C::GROUPS, g0 + C::EG) * C::WK; ++e)
                if (e % C::WK != wk)
#pragma unroll
                    for (int m = 0; m < C::MA; ++m) red_at(wk, e, m) = sum[e][m];
            lds_barrier();
#pragma unroll
            for (int e = g0 * C::WK; e < cmin(C::GROUPS, g0 + C::EG) * C::WK; ++e)
                if (e % C::WK == wk)
#pragma unroll
                    for (int m = 0; m < C::MA; ++m) {
                        floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};  // in wave order
#pragma unroll
                        for (int k = 0; k < C::WK; ++k) v += k == e % C::WK ? sum[e][m] : red_at(k, e, m);
                        sum[e][m] = v;
                    }
            lds_barrier();
        }
    }

    // Element r of item (e, m): output channel co0 + el_co, slot el_slot.
    auto el_co = [&](int e, int m, int r) { return (wc * C::MA + m) * 32 + (POOL ? l32 : 8 * (e % 4) + 4 * g + r); };
    auto el_slot = [&](int e, int r) { return (wp * C::NB + e / 4) * 32 + (POOL ? 8 * (e % 4) + 4 * g + r : l32); };
    const bool with_bias = bias != nullptr && split == 0;
    float sum0 = 0.f;  // stays 0 while every value is finite
    if (with_bias) {
        const __amdgpu_buffer_rsrc_t rb = make_rsrc(bias, (unsigned)a.c_out * 4u);
#pragma unroll
        for (int m = 0; m < C::MA; ++m) {
            float bv[POOL ? 1 : 16];  // of the lane's 16 rows (channels past C_out read 0)
#pragma unroll
            for (int r = 0; r < (POOL ? 1 : 16); ++r)
                bv[r] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(rb, (co0 + el_co(r / 4, m, r % 4)) * 4, 0, 0));
#pragma unroll
            for (int e = 0; e < C::ITEMS; ++e)
                if (e % C::WK == wk)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sum[e][m][r] += bv[POOL ? 0 : e % 4 * 4 + r];
        }
    }
#pragma unroll
    for (int e = 0; e < C::ITEMS; ++e)
        if (e % C::WK == wk)
#pragma unroll
            for (int m = 0; m < C::MA; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) sum0 = __builtin_fmaf(sum[e][m][r], 0.f, sum0);

    // A value that is not finite: an infinity, a NaN or a value near the top
    // of the range among its operands, or a true overflow.  Compute its 32x32
    // block again with fp32 matrix instructions from memory, a lane's half
    // taking every other input channel, and keep what is finite.  (All of a
    // wave's blocks together, the loads of a batch of products flying while the
    // batch before multiplies.  64->64 at 224^2: finite 27 us a call, one NaN
    // pixel 65, NaN everywhere 104; 256->256 at 56^2 31, 317 and 359.  By single
    // lanes over C_in*K*K these were 1579 and 3479, 1868 and 3392 us.)
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(sum0 != 0.f || sum0 != sum0) != 0, 0)) {
        constexpr int CB = C::KS == 1 ? 4 : 1, KH = C::KS == 5 ? 1 : C::KS, BATCH = CB * KH * C::KS;
        const __amdgpu_buffer_rsrc_t rx = make_rsrc(x, (unsigned)a.c_in * plane4);
        const __amdgpu_buffer_rsrc_t rw = PK ? make_rsrc(w_packed, (unsigned)a.nchunks * (C::COT * C::ROW * 4u))
                                             : make_rsrc(w, (unsigned)a.c_out * wrow * 4u);
        const int ci_end = min(c_end * C::CC, a.c_in);
        int ih0[C::NB], iw0[C::NB];
#pragma unroll
        for (int b = 0; b < C::NB; ++b) {
            int pr, pc;
            slot_pixel<POOL>((wp * C::NB + b) * 32 + l32, t, pr, pc);
            ih0[b] = (oh0 + pr) * stride - a.pad;
            iw0[b] = (ow0 + pc) * stride - a.pad;
        }
#pragma unroll
        for (int m = 0; m < C::MA; ++m) {
            bool redo[C::NB];
            floatx16 acc[C::NB];
#pragma unroll
            for (int b = 0; b < C::NB; ++b) {
                bool bad = false;
#pragma unroll
                for (int e = 4 * b; e < 4 * b + 4; ++e)
                    if (e % C::WK == wk)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            bad |= not_finite(sum[e][m][r]) && s_out[el_slot(e, r)] >= 0 &&
                                   co0 + el_co(e, m, r) < a.c_out;
                redo[b] = __builtin_amdgcn_ballot_w64(bad) != 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int co = co0 + el_co(r / 4, m, r % 4);
                    acc[b][r] = with_bias && co < a.c_out ? bias[co] : 0.f;
                }
            }
            const int co_l = (wc * C::MA + m) * 32 + l32;
            // Batch (ci0, kh0): channels ci0 + 2*cb + g, rows kh0 .. of the filter.
            float xv[C::NB][BATCH], wv[BATCH], xn[C::NB][BATCH], wn[BATCH];
            auto load = [&](int ci0, int kh0) {
#pragma unroll
                for (int j = 0; j < BATCH; ++j) {
                    const int ci = ci0 + j / (KH * C::KS) * 2 + g;
                    const int kh = kh0 + j / C::KS % KH, kw = j % C::KS, tap = kh * C::KS + kw;
                    const int cl = ci % C::CC;
                    unsigned wo = 0x80000000u;
                    if (PK) {
                        if (ci < ci_end)
                            wo = (unsigned)(ci / C::CC * (C::COT * C::ROW) +
                                            (((tap * C::C8 + cl / 8) * 2 + cl % 8 / 4) * C::COT + co_l) * 4 + cl % 4) *
                                 4u;
                    } else {
                        if (ci < ci_end && co0 + co_l < a.c_out)
                            wo = ((unsigned)(co0 + co_l) * wrow + (unsigned)(ci * C::KK + tap)) * 4u;
                    }
                    wn[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw, (int)wo, 0, 0));
#pragma unroll
                    for (int b = 0; b < C::NB; ++b)
                        if (redo[b]) {
                            const int ih = ih0[b] + kh, iw = iw0[b] + kw;
                            const bool in = ci < ci_end && ih >= 0 && ih < a.h && iw >= 0 && iw < a.w;
                            const unsigned xo =
                                in ? (unsigned)ci * plane4 + (unsigned)(ih * a.w + iw) * 4u : 0x80000000u;
                            xn[b][j] =
                                __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, (int)xo, 0, 0));
                        }
                }
            };
            int ci0 = c_begin * C::CC, kh0 = 0;
            load(ci0, kh0);
#pragma unroll 1
            while (ci0 < ci_end) {
#pragma unroll
                for (int j = 0; j < BATCH; ++j) {
                    wv[j] = wn[j];
#pragma unroll
                    for (int b = 0; b < C::NB; ++b) xv[b][j] = xn[b][j];
                }
                kh0 += KH;
                if (kh0 >= C::KS) {
                    kh0 = 0;
                    ci0 += 2 * CB;
                }
                load(ci0, kh0);  // (past the last channel: zeros)
#pragma unroll
                for (int b = 0; b < C::NB; ++b)
                    if (redo[b])
#pragma unroll
                        for (int j = 0; j < BATCH; ++j)
                            acc[b] = POOL ? __builtin_amdgcn_mfma_f32_32x32x2f32(xv[b][j], wv[j], acc[b], 0, 0, 0)
                                          : __builtin_amdgcn_mfma_f32_32x32x2f32(wv[j], xv[b][j], acc[b], 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < C::ITEMS; ++e)
                if (e % C::WK == wk && redo[e / 4])
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (not_finite(sum[e][m][r])) sum[e][m][r] = acc[e / 4][e % 4 * 4 + r];
        }
    }

    // Stores.  Lanes outside the output get an offset past the descriptor's
    // range (< 2^30 bytes, checked when the plan is made).
    const unsigned oplane4 = (unsigned)ho2 * (unsigned)wo2 * 4u;
    const __amdgpu_buffer_rsrc_t ro =
        a.to_part ? make_rsrc(part + (size_t)split * a.c_out * (oplane4 / 4u), (unsigned)a.c_out * oplane4)
                  : make_rsrc(out, (unsigned)a.c_out * oplane4);
    const bool relu = a.relu && !a.to_part;
    const bool whole = co0 + C::COT <= a.c_out;  // every channel of the tile exists
#pragma unroll
    for (int e = 0; e < C::ITEMS; ++e) {
        if (e % C::WK != wk) continue;
        const int so = s_out[el_slot(e, 0)];
        const unsigned base = (unsigned)(co0 + el_co(0, 0, 0)) * oplane4 + 4u * (unsigned)so;
        const int off = (int)(so >= 0 ? base : 0x40000000u);
        // A value `row` channels past the lane's first one.
        auto store = [&](float v, int row) {
            if (relu && v < 0.f) v = 0.f;
            const unsigned bits = __builtin_bit_cast(unsigned, v);
            if (whole) {
                __builtin_amdgcn_raw_buffer_store_b32(bits, ro, off, (int)(row * oplane4), kPolicyDeviceScope);
            } else {
                const bool ok = so >= 0 && co0 + el_co(0, 0, 0) + row < a.c_out;
                __builtin_amdgcn_raw_buffer_store_b32(bits, ro, (int)(ok ? base + row * oplane4 : 0x40000000u), 0,
                                                      kPolicyDeviceScope);
            }
        };
#pragma unroll
        for (int m = 0; m < C::MA; ++m) {
            const floatx4 v = sum[e][m];
            if constexpr (POOL) {
                float mx = v[0], q = v[1];
                mx = q > mx ? q : mx;
                q = v[2];
                mx = q > mx ? q : mx;
                q = v[3];
                mx = q > mx ? q : mx;
                store(mx, 32 * m);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float q = v[r];
                    store(q, 32 * m + e % 4 * 8 + r);
                }
            }
        }
    }
}

template <class C>
void launch_split(dim3 grid, hipStream_t st, const float *x, const float *w, const float *b, float *o, float *ws,
                  const IgArgs &a, const SplitTile &t, bool packed)
{
    if (a.pool_tile) {
        if (packed) hipLaunchKernelGGL((conv_split<C, true, true>), grid, dim3(C::NT), 0, st, x, w, b, o, ws, a, t);
        else hipLaunchKernelGGL((conv_split<C, false, true>), grid, dim3(C::NT), 0, st, x, w, b, o, ws, a, t);
    } else {
        if (packed) hipLaunchKernelGGL((conv_split<C, true, false>), grid, dim3(C::NT), 0, st, x, w, b, o, ws, a, t);
        else hipLaunchKernelGGL((conv_split<C, false, false>), grid, dim3(C::NT), 0, st, x, w, b, o, ws, a, t);
    }
}

// th, tw: the tile that variant_info names; a plan's own tile has at most
// C::PX pixels and is chosen for its shape.
template <class C>
constexpr Variant make_split_variant(const char *name, int th, int tw, bool even, const Variant::Times &us)
{
    Variant v = {name, C::KS, C::S, th, tw, C::WC, C::WP, C::WK, C::MA, C::CC,
                 C::NT, C::COT, C::LDS_BYTES, 0, false, 2, false, even, false, nullptr};
    v.launch3 = &launch_split<C>;
    v.px = C::PX;
    v.xpix = C::XPIX;
    v.even = even;
    v.per_cu = C::LDS_BYTES <= 80 * 1024 && C::NT <= 256 ? 2 : 1;
    v.us = us;
    return v;
}

}  // namespace
}  // namespace ilpm
