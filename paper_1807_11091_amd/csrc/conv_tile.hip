// gfx950 direct CONV (implicit GEMM) over a group's compacted matrix: every tap
// of one run of 8k input channels, read straight from the NHWC input.
//
// k_conv_tile: persistent workgroups of four MFMA wavefronts (consumers) and
// four fetching wavefronts (producers).  Operands travel in
// slices of 64 columns through a ring of S LDS buffers: a producer's
// buffer_load ... lds writes 16 bytes per lane (8 rows of 128 bytes per
// instruction) straight into LDS, S slices ahead and across tile boundaries,
// so the first slices of the next tile arrive while the output of the current
// one is written.  Padding pixels, filters past M and columns past K are
// offsets beyond the buffer's range, which land in LDS as +0.
//
// Why it is built this way (conv [154 of 256, 256, 3, 3] on 14x14, batch 64,
// 36 slices, one tile per CU; all sides measured):
//  - DMA instructions stall the wavefront that issues them (the address unit
//    takes 16 clocks for each): issued by the MFMA wavefronts between their
//    MFMAs the slice takes 0.34 us, by wavefronts of their own 0.18 us
//    (17.2 -> 12.5 us per call; two producers instead of four: 16.3 us).
//  - The DMA statements are inline asm: after the compiler's own LDS-DMA
//    builtin every LDS read waits for all loads in flight (vmcnt(0)), which
//    leaves no slice in flight (ring of 3 at 128x128: 26 us).  The asm has no
//    outputs; the waits are wait_vm() on the producers' side and the barrier.
//  - Fragments of slice s + 1 are read from LDS while slice s is multiplied.
//    The 16-byte chunks of a row are XOR-swizzled by (row >> 1) & 7, applied
//    to the source address (the DMA writes lanes consecutively): 16 rows of
//    one chunk column hit 16 distinct 16-byte banks.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "conv_ig.h"
#include "conv_tile.h"
#include "sa_conv_device.h"
#include "sa_host.h"

namespace sa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kTileLds = 160 * 1024;

__device__ inline i32x4 dma_rsrc(const void *base, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    return i32x4{(int)(uint32_t)a, (int)((uint32_t)(a >> 32) & 0xffffu), (int)bytes, kRsrcWord3};
}
// 16 bytes per lane straight from memory to LDS: lane i's land at lds + 16 * i
// (M0 holds the LDS address).  M0 is declared, so that the compiler lets no use
// of its own rest on a value from before the statement; its warning says that a
// reserved register is not saved around the asm, which nothing here needs.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void dma16(i32x4 r, uint32_t voff, uint32_t soff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff),
                 "s"(r), "s"(soff)
                 : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ inline void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// waits until at most `left` (0 .. MAX) slices of L loads each are outstanding
template <int L, int MAX>
__device__ inline void wait_slices(int left) {
    if constexpr (MAX == 0) {
        wait_vm<0>();
    } else {
        if (left >= MAX) wait_vm<L * MAX>();
        else wait_slices<L, MAX - 1>(left);
    }
}
// a wavefront-uniform value kept in a scalar register: the asm statements of
// the slice loop clobber memory, so the compiler would re-read kernel
// arguments from memory in every slice otherwise
__device__ inline int sgpr(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline FastDiv sgpr(const FastDiv &f) {
    return FastDiv{(uint32_t)sgpr((int)f.mul), (uint32_t)sgpr((int)f.shift), (uint32_t)sgpr((int)f.d)};
}
// this wavefront's LDS reads and writes done, then the workgroup's barrier
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// BM pixels x BN filters per tile, WN x WM consumer wavefronts, S slices in the
// ring, MI x MI MFMA tiles (16x16x32 or 32x32x16)
template <int BM, int BN, int WN, int WM, int S, int MI>
struct TileCfg {
    static constexpr int NW = WN * WM, PW = 4, NT = 64 * (NW + PW);
    static constexpr int WTM = BN / WM, WTN = BM / WN;  // wavefront tile (m, px)
    static constexpr int TM = WTM / MI, TN = WTN / MI;
    static constexpr int KS = MI == 16 ? 2 : 4;  // MFMA steps of a slice
    // DMA loads per producer and slice; a load past the tile's BN filters
    // reads nothing (every producer issues the same number)
    static constexpr int AL = (BN / 8 + PW - 1) / PW, BL = BM / 8 / PW;
    static constexpr int a_bytes = AL * PW * 1024;
    static constexpr int stage = a_bytes + BM * kBK * 2;
    static constexpr int c_bytes = 2 * BM * (BN + 8);
    static constexpr int lds = S * stage + c_bytes;
    static_assert(BN % 16 == 0 && BM % (8 * PW) == 0, "whole loads per producer");
    static_assert(WTM % MI == 0 && WTN % MI == 0, "tile shape");
    static_assert(S >= 2 && (S - 1) * (AL + BL) <= 63, "vmcnt range");
    static_assert(lds <= kTileLds, "LDS");
};

// One tile of a workgroup's range: its group, origin and slices.
struct Tile {
    int gi, m0, n0, s0, ns, chunk;  // ns >= 1 (a group without columns runs one slice of zeros)
};

template <int BM, int BN, bool ONE, bool SPLIT>
__device__ inline Tile tile_at(const ConvArgs &a, int t) {
    Tile T;
    T.chunk = 0;
    if constexpr (SPLIT) {
        T.chunk = t / a.base_blocks;
        t -= T.chunk * a.base_blocks;
    }
    T.gi = 0;
    if constexpr (!ONE)
        while (T.gi + 1 < a.ngroups && t >= a.g[T.gi + 1].begin) ++T.gi;
    const ConvGroup &G = a.g[T.gi];
    const int lb = ONE ? t : t - G.begin;
    const int nt = (int)fdiv((uint32_t)lb, G.divMt);
    T.m0 = (lb - nt * G.mtiles) * BN;
    T.n0 = nt * BM;
    T.s0 = 0;
    T.ns = G.ldk / kBK;
    if constexpr (SPLIT) {
        T.s0 = T.ns * T.chunk / a.ksplit;
        T.ns = G.ldk / kBK * (T.chunk + 1) / a.ksplit - T.s0;
    }
    T.ns = max(1, T.ns);
    return T;
}

// UNI: every slice lies in one tap (run a multiple of 64) and there are at most
// 31 taps, so a row's in-image taps are one bit mask; otherwise each lane
// divides its column by the run and checks the pixel against the image.
// ONE: a single conv group.  SPLIT: binary32 partial sums of a chunk of slices.
template <int BM, int BN, int WN, int WM, int S, int MI, bool UNI, bool ONE, bool SPLIT>
__global__ __launch_bounds__(64 * (WN * WM + 4)) void k_conv_tile(ConvArgs a) {
    using Cfg = TileCfg<BM, BN, WN, WM, S, MI>;
    using Acc = typename std::conditional<MI == 16, f32x4, f32x16>::type;
    constexpr int WTM = Cfg::WTM, WTN = Cfg::WTN, TM = Cfg::TM, TN = Cfg::TN, NW = Cfg::NW, PW = Cfg::PW;
    constexpr int AL = Cfg::AL, BL = Cfg::BL, L = AL + BL;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // [S] slices, then the output tile

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = sgpr(tid >> 6);
    // contiguous range of tiles of this workgroup (every XCD walks one range)
    const int wg = xcd_remap(blockIdx.x, a.nblocks);
    const int per = a.tiles / a.nblocks, extra = a.tiles - per * a.nblocks;
    const int t0 = wg * per + min(wg, extra), t1 = t0 + per + (wg < extra ? 1 : 0);

    if (wave >= NW) {
        // ---- producers
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
        const int pw = wave - NW;
        const int D = sgpr(a.D), W = sgpr(a.W), H = sgpr(a.H), C = sgpr(a.C), NPQ = sgpr(a.NPQ), flat = sgpr(a.flat);
        const int stride = sgpr(a.stride), pad = sgpr(a.pad), PQ = sgpr(a.P * a.Q), Q = sgpr(a.Q);
        const FastDiv divD = sgpr(a.divD), divPQ = sgpr(a.divPQ), divQ = sgpr(a.divQ);
        // load i of this wavefront fills rows 8 * (i * PW + pw) .. + 7 of a tile
        const int rl = lane >> 3;
        const int kc = (lane & 7) ^ (4 * (pw & 1) + (lane >> 4));  // source chunk (8 columns)
        uint32_t aoff[AL], xoff[BL], vmask[BL], vx[BL];
        int xh0[BL], xw0[BL];
        // The stream of slices of all the workgroup's tiles: slice n goes to
        // ring slot n mod S once slice n - S has been read.  Barrier g tells
        // that slice g has landed and that slice g - 1 has been read; after the
        // last slice of a tile one more barrier goes with its staged output.
        int n = 0, g = 0, ct = t0;                                    // issued, next barrier, consumers' tile
        int cleft = sgpr(tile_at<BM, BN, ONE, SPLIT>(a, t0).ns);      // its slices left
        uint32_t base = lds0 + pw * 1024;
        const uint32_t base_end = base + S * Cfg::stage;
        auto passed = [&]() {
            ++g;
            if (--cleft == 0) {
                if constexpr (!SPLIT) lds_barrier();
                if (++ct < t1) cleft = sgpr(tile_at<BM, BN, ONE, SPLIT>(a, ct).ns);
            }
        };
        // Between a barrier and the loads that it releases, and between those
        // and the next barrier, stands as little as possible: with the
        // addresses of each slice worked out here (60 scalar instructions) a
        // slice took 0.34 us instead of 0.18.
        auto room = [&]() {
            if (n >= S) {
                if (n == S) {
                    wait_vm<L *(S - 1)>();
                    lds_barrier();
                    passed();
                }
                wait_vm<L *(S - 2)>();
                lds_barrier();
                passed();
            }
            ++n;
        };
        auto next_slot = [&]() {
            base += Cfg::stage;
            base = base == base_end ? base - S * Cfg::stage : base;
        };
        for (int ft = t0; ft < t1; ++ft) {
            const Tile T = tile_at<BM, BN, ONE, SPLIT>(a, ft);
            const ConvGroup &G = a.g[T.gi];
            const int ldk = sgpr(G.ldk), Cx = sgpr(G.Cx), K = sgpr(G.K), run = ldk > 0 ? sgpr(G.run) : kBK;
            const int run_base = sgpr(G.run_base);
            const FastDiv divRun = sgpr(G.divRun);
            const i32x4 wrs = dma_rsrc(G.Wc, (uint32_t)G.M * (uint32_t)ldk * 2u);
            // UNI: offsets count from `shift` bytes before the input, so that
            // the pixel of tap (0, 0) has one also where it lies in the padding
            const uint32_t shift = UNI ? (uint32_t)(pad * (W + 1)) * (uint32_t)Cx * 2u : 0u;
            const i32x4 xrs = dma_rsrc(reinterpret_cast<const uint8_t *>(G.X) - shift, G.x_bytes + shift);
#pragma unroll
            for (int i = 0; i < AL; ++i) {
                const int r = 8 * (i * PW + pw) + rl;
                const bool in = ldk > 0 && (BN % (8 * PW) == 0 || r < BN);
                aoff[i] = in ? ((uint32_t)(T.m0 + r) * (uint32_t)ldk + kc * 8) * 2u : kInvalidOffset;
            }
            // the input pixel of tap (0, 0) of each row's output pixel, and
            // (UNI) the taps that fall inside the image
#pragma unroll
            for (int i = 0; i < BL; ++i) {
                const int pxr = T.n0 + 8 * (i * PW + pw) + rl;
                if (UNI && flat) {  // 1x1, stride 1, no padding: output pixel = input pixel
                    xoff[i] = ((uint32_t)pxr * (uint32_t)Cx + run_base + kc * 8) * 2u;
                    vmask[i] = ldk > 0 && pxr < NPQ ? 1u : 0u;
                    continue;
                }
                const int px = min(pxr, NPQ - 1);
                const int nn = (int)fdiv((uint32_t)px, divPQ);
                const int rem = px - nn * PQ;
                const int p = (int)fdiv((uint32_t)rem, divQ);
                const int h0 = p * stride - pad, w0 = (rem - p * Q) * stride - pad;
                xoff[i] = ((uint32_t)((nn * H + h0) * W + w0) * (uint32_t)Cx + run_base + (UNI ? kc * 8 : 0)) * 2u + shift;
                if constexpr (UNI) {
                    // taps d with 0 <= w0 + d < W, repeated for the rows c with 0 <= h0 + c < H
                    const uint32_t lo = (uint32_t)min(D, max(0, -w0)), hi = (uint32_t)max(0, min(D, W - w0));
                    const uint32_t cols = ((1u << hi) - 1u) & ~((1u << lo) - 1u);
                    uint32_t vm = 0;
                    for (int c = 0; c < C; ++c) vm |= (unsigned)(h0 + c) < (unsigned)H ? cols << (c * D) : 0u;
                    vmask[i] = ldk > 0 && pxr < NPQ ? vm : 0u;
                } else {
                    xh0[i] = ldk > 0 && pxr < NPQ ? h0 : -(1 << 28);
                    xw0[i] = w0;
                }
            }
            int s = sgpr(T.s0);
            const int send = s + sgpr(T.ns);
            if constexpr (UNI) {
                int tap = 0, tch = 0, tc = 0, td = 0;
                if (SPLIT) {
                    tap = (int)fdiv((uint32_t)(s * kBK), divRun);
                    tch = s * kBK - tap * run;
                    tc = (int)fdiv((uint32_t)tap, divD);
                    td = tap - tc * D;
                }
                while (s < send) {
                    // the slices of one tap
#pragma unroll
                    for (int i = 0; i < BL; ++i) vx[i] = (vmask[i] >> tap) & 1u ? xoff[i] : kInvalidOffset;
                    uint32_t sa = (uint32_t)s * (kBK * 2), sx = ((uint32_t)(tc * W + td) * Cx + tch) * 2u;
                    const int e = min(send, s + (run - tch) / kBK);
                    for (; s < e; ++s) {
                        room();
#pragma unroll
                        for (int i = 0; i < AL; ++i) dma16(wrs, aoff[i], sa, base + i * PW * 1024);
#pragma unroll
                        for (int i = 0; i < BL; ++i) dma16(xrs, vx[i], sx, base + Cfg::a_bytes + i * PW * 1024);
                        sa += kBK * 2;
                        sx += kBK * 2;
                        next_slot();
                    }
                    tch = 0;
                    ++tap;
                    ++td;
                    tc += td == D ? 1 : 0;
                    td = td == D ? 0 : td;
                }
            } else {
                for (; s < send; ++s) {
                    const int k = s * kBK + kc * 8;
                    const int t = (int)fdiv((uint32_t)k, divRun);
                    const int ch = k - t * run;
                    const int c = (int)fdiv((uint32_t)t, divD);
                    const int d = t - c * D;
                    const uint32_t delta = ((uint32_t)(c * W + d) * Cx + ch) * 2u;
                    const bool kin = k < K;
#pragma unroll
                    for (int i = 0; i < BL; ++i) {
                        const bool in = kin && (unsigned)(xh0[i] + c) < (unsigned)H && (unsigned)(xw0[i] + d) < (unsigned)W;
                        vx[i] = in ? xoff[i] + delta : kInvalidOffset;
                    }
                    room();
#pragma unroll
                    for (int i = 0; i < AL; ++i) dma16(wrs, aoff[i], (uint32_t)s * (kBK * 2), base + i * PW * 1024);
#pragma unroll
                    for (int i = 0; i < BL; ++i) dma16(xrs, vx[i], 0u, base + Cfg::a_bytes + i * PW * 1024);
                    next_slot();
                }
            }
        }
        while (g < n) {  // the slices still in flight
            wait_slices<L, S - 1>(n - 1 - g);
            lds_barrier();
            passed();
        }
        return;  // every load has landed
    }

    // ---- consumers
    const int wn = wave % WN, wm = wave / WN;
    constexpr int KS = Cfg::KS, KC = kBK / KS;
    // fragment of MI rows: row lane % MI, columns q * KC + 8 * (lane / MI), swizzled chunk
    const int frow = lane & (MI - 1);
    uint32_t foff[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) foff[q] = frow * 128 + (((q * (KC / 8) + lane / MI) ^ ((frow >> 1) & 7)) << 4);
    struct Frags {
        bf16x8 a[TM], b[TN];
    };
    const uint32_t fa = wm * WTM * 128, fb = Cfg::a_bytes + wn * WTN * 128;
    uint16_t *sC = reinterpret_cast<uint16_t *>(smem + S * Cfg::stage);  // [BM][BN + 8]
    int slot = 0;
    Acc acc[TM][TN];
    // One MFMA step is multiplied from cur while the next step's fragments
    // (step q of the current ring slot) are read into next.
    auto step = [&](const Frags &cur, Frags &next, int q, bool read) {
        const uint8_t *st = smem + slot * Cfg::stage;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (read) {
                if (i == 0) {
#pragma unroll
                    for (int j = 0; j < TN; ++j) next.b[j] = *reinterpret_cast<const bf16x8 *>(st + fb + foff[q] + j * MI * 128);
                }
                next.a[i] = *reinterpret_cast<const bf16x8 *>(st + fa + foff[q] + i * MI * 128);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (MI == 16)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.a[i], cur.b[j], acc[i][j], 0, 0, 0);
                else
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[i], cur.b[j], acc[i][j], 0, 0, 0);
            }
        }
        // the reads go out ahead of the MFMAs that hide them
        if (read) {
            __builtin_amdgcn_sched_group_barrier(0x100, TN + TM, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = t0; t < t1; ++t) {
        const Tile T = tile_at<BM, BN, ONE, SPLIT>(a, t);
        const int ns = sgpr(T.ns);
        Frags f[2];
        lds_barrier();
#pragma unroll
        for (int j = 0; j < TN; ++j) f[0].b[j] = *reinterpret_cast<const bf16x8 *>(smem + slot * Cfg::stage + fb + foff[0] + j * MI * 128);
#pragma unroll
        for (int i = 0; i < TM; ++i) f[0].a[i] = *reinterpret_cast<const bf16x8 *>(smem + slot * Cfg::stage + fa + foff[0] + i * MI * 128);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = Acc{};
        for (int s = 1; s < ns; ++s) {
#pragma unroll
            for (int q = 0; q + 1 < KS; ++q) step(f[q & 1], f[(q + 1) & 1], q + 1, true);
            slot = slot + 1 == S ? 0 : slot + 1;
            lds_barrier();  // the next slice has landed (and this one has been read)
            step(f[(KS - 1) & 1], f[KS & 1], 0, true);
        }
#pragma unroll
        for (int q = 0; q + 1 < KS; ++q) step(f[q & 1], f[(q + 1) & 1], q + 1, true);
        slot = slot + 1 == S ? 0 : slot + 1;
        step(f[(KS - 1) & 1], f[KS & 1], 0, false);

        // accumulator r of a lane: filter (r / 4) * 8 + (lane / 32) * 4 + r % 4 (MI = 32) or
        // (lane / 16) * 4 + r (MI = 16), pixel lane % MI
        const ConvGroup &G = a.g[T.gi];
        if constexpr (SPLIT) {  // k_splitk_sum adds the chunks
            float *part = a.part + (int64_t)T.chunk * a.part_stride;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r4 = 0; r4 < MI * MI / 256; ++r4) {
                        const int m = T.m0 + wm * WTM + i * MI + r4 * 8 + (lane / MI) * 4;
                        const int px = T.n0 + wn * WTN + j * MI + (lane & (MI - 1));
                        if (px >= a.NPQ) continue;
                        float *dst = part + (int64_t)px * a.Cy + G.o_off + m;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (m + e < G.M) dst[e] = acc[i][j][r4 * 4 + e];
                    }
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r4 = 0; r4 < MI * MI / 256; ++r4) {
                        const int ml = wm * WTM + i * MI + r4 * 8 + (lane / MI) * 4;
                        const int pl = wn * WTN + j * MI + (lane & (MI - 1));
                        bf16x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = (__bf16)acc[i][j][r4 * 4 + e];  // round to nearest even
                        *reinterpret_cast<bf16x4 *>(&sC[pl * (BN + 8) + ml]) = o;
                    }
            lds_barrier();
            // the next tile's output is staged only after a slice barrier that
            // follows these reads
            if (a.Cy % 8 != 0 && a.ldy == a.Cy && G.mtiles == 1 && G.M == a.Cy && ((uintptr_t)a.Y & 15) == 0) {
                // whole, unaligned rows
                store_tile_rows<BN + 8>(a.Y, sC, T.n0, min(BM, a.NPQ - T.n0), a.Cy, a.divCy, tid, 64 * NW);
                continue;
            }
            // the last channels of a row may run on into the row's padding (staged
            // rows past the group's filters hold +0)
            const int lim = G.o_off + G.M == a.Cy ? a.ldy - G.o_off : G.M;
            constexpr int CPR = BN / 8;  // 16-byte chunks per output row
            for (int c = tid; c < BM * CPR; c += 64 * NW) {
                const int pl = c / CPR, mc = c - pl * CPR;
                const int px = T.n0 + pl, m = T.m0 + mc * 8;
                if (px >= a.NPQ || m >= G.M) continue;
                uint16_t *dst = a.Y + (int64_t)px * a.ldy + G.o_off + m;
                store_out8(dst, &sC[pl * (BN + 8) + mc * 8], min(8, lim - m));
            }
        }
    }
}

// ---------------------------------------------------------------- host side
// Workgroups of `kern` (nt threads, lds bytes) that the GPU holds at once;
// raises the kernel's LDS limit on the first call per device.
int resident_workgroups(const void *kern, int nt, int lds, int *wgs) {
    static std::mutex mu;
    static std::map<std::pair<const void *, int>, int> known;
    int dev = 0;
    if (int rc = check_hip(hipGetDevice(&dev), "conv: current device")) return rc;
    std::lock_guard<std::mutex> lock(mu);
    auto it = known.find({kern, dev});
    if (it != known.end()) {
        *wgs = it->second;
        return SA_OK;
    }
    if (int rc = check_hip(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, kTileLds),
                           "conv: set LDS size"))
        return rc;
    int per_cu = 0, cus = 0;
    if (int rc = check_hip(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, nt, lds), "conv: occupancy"))
        return rc;
    if (int rc = check_hip(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "conv: CU count"))
        return rc;
    *wgs = std::max(1, per_cu) * std::max(1, cus);
    known[{kern, dev}] = *wgs;
    return SA_OK;
}

// Every slice of 64 columns lies in one tap (runs are multiples of 64), at most
// 31 taps (one bit each), and the input with its padded border below 2 GiB.
// The loads' scalar offset (last tap and channel) stays within that range too:
// the unit compares a lane's offset with the range less the scalar offset, which
// must not fall below zero (a single image smaller than the kernel, where the
// last taps are padding for every pixel).
bool uniform_taps(const ConvArgs &a) {
    bool uni = a.C * a.D <= 31;
    for (int i = 0; i < a.ngroups; ++i) {
        const ConvGroup &G = a.g[i];
        const int64_t range = (int64_t)G.x_bytes + (int64_t)a.pad * (a.W + 1) * G.Cx * 2;
        const int64_t last = (((int64_t)(a.C - 1) * a.W + a.D - 1) * G.Cx + G.run) * 2;
        uni = uni && G.run % kBK == 0 && G.run > 0 && range < (int64_t(1) << 31) && last <= range;
    }
    return uni;
}

template <int BM, int BN, int WN, int WM, int S, int MI, bool SPLIT>
int launch(ConvArgs a, hipStream_t stream) {
    using Cfg = TileCfg<BM, BN, WN, WM, S, MI>;
    // tiles of group i: [begin, begin + mtiles * ntiles), m-tiles fastest;
    // with split K, ksplit copies of that range, one per chunk of slices
    const int ntiles = (a.NPQ + BM - 1) / BM;
    int begin = 0;
    for (int i = 0; i < a.ngroups; ++i) {
        a.g[i].mtiles = (a.g[i].M + BN - 1) / BN;
        a.g[i].begin = begin;
        a.g[i].divMt = make_fastdiv((uint32_t)a.g[i].mtiles);
        begin += a.g[i].mtiles * ntiles;
    }
    const bool uni = uniform_taps(a);
    a.flat = a.C * a.D == 1 && a.stride == 1 && a.pad == 0;
    a.base_blocks = begin;
    a.tiles = begin * (SPLIT ? a.ksplit : 1);
    using Kern = void (*)(ConvArgs);
    Kern kern;
    if constexpr (SPLIT)
        kern = uni ? k_conv_tile<BM, BN, WN, WM, S, MI, true, false, true>
                   : k_conv_tile<BM, BN, WN, WM, S, MI, false, false, true>;
    else if (a.ngroups == 1)
        kern = uni ? k_conv_tile<BM, BN, WN, WM, S, MI, true, true, false>
                   : k_conv_tile<BM, BN, WN, WM, S, MI, false, true, false>;
    else
        kern = uni ? k_conv_tile<BM, BN, WN, WM, S, MI, true, false, false>
                   : k_conv_tile<BM, BN, WN, WM, S, MI, false, false, false>;
    int wgs = 0;
    if (int rc = resident_workgroups(reinterpret_cast<const void *>(kern), Cfg::NT, Cfg::lds, &wgs)) return rc;
    a.nblocks = std::min(a.tiles, wgs);
    hipLaunchKernelGGL(kern, dim3(a.nblocks), dim3(Cfg::NT), Cfg::lds, stream, a);
    return check_hip(hipGetLastError(), "k_conv_tile");
}

// ---------------------------------------------------------------- time model
// A launch of `tiles` tiles of `ns` slices on `cus` CUs, R workgroups of the
// shape per CU, takes
//   launch + max(rounds * (ns * slice + round), load * (ns * share + tile), bytes / rate)
// microseconds: rounds = tiles per resident workgroup, each a serial chain of
// slices (`alone` instead of `slice` while every workgroup has a CU of its
// own); load = tiles per CU, which share the CU's matrix cores, LDS and fetch
// path; rate in TB/s.  The constants are least-squares fits of the logarithm
// to 244 measured layers (ResNet-50's at batch 64 pruned and dense, and 192
// with random sizes: 450 to 300,000 pixels, 4 to 2048 filters, 1 to 160
// slices), once for layers whose slices lie in one tap and once for the rest.
// Choosing by it costs 3% over the best shape of each layer; over those layers
// the choice takes 0.83 (one tap) and 0.88 (the rest) of k_conv's time.
struct Model {
    int16_t BM, BN, R;
    float launch, round, slice, share, tile, rate, alone;
};
constexpr Model kModel[2][9] = {
    {   // slices in one tap
        {64, 64, 2, 2.91f, 0.88f, 0.27f, 0.16f, 0.43f, 5.84f, 0.24f},
        {128, 48, 2, 2.65f, 2.25f, 0.25f, 0.24f, 1.18f, 6.96f, 0.30f},
        {128, 80, 2, 2.23f, 2.73f, 0.48f, 0.27f, 1.57f, 6.40f, 0.37f},
        {64, 160, 1, 3.92f, 1.07f, 0.30f, 0.11f, 0.47f, 7.59f, 0.27f},
        {64, 160, 2, 3.41f, 1.35f, 0.55f, 0.19f, 0.69f, 9.00f, 0.34f},
        {128, 128, 1, 4.63f, 1.49f, 0.38f, 0.09f, 0.29f, 6.67f, 0.32f},
        {64, 128, 2, 3.34f, 0.86f, 0.47f, 0.26f, 0.54f, 6.52f, 0.34f},
        {128, 128, 2, 3.30f, 2.08f, 0.91f, 0.46f, 1.07f, 7.78f, 0.55f},
        {128, 64, 2, 3.34f, 1.28f, 0.29f, 0.30f, 1.03f, 5.78f, 0.37f},
    },
    {   // any run of 8k channels
        {64, 64, 2, 2.99f, 1.08f, 0.27f, 0.18f, 0.84f, 5.41f, 0.17f},
        {128, 48, 2, 3.40f, 0.84f, 0.17f, 0.28f, 1.29f, 6.22f, 0.29f},
        {128, 80, 2, 3.91f, 1.00f, 0.72f, 0.26f, 1.73f, 6.58f, 0.27f},
        {64, 160, 1, 2.78f, 2.28f, 0.30f, 0.23f, 1.49f, 9.00f, 0.23f},
        {64, 160, 2, 3.58f, 1.61f, 0.61f, 0.24f, 1.59f, 7.47f, 0.24f},
        {128, 128, 1, 4.02f, 2.62f, 0.40f, 0.23f, 0.98f, 8.19f, 0.24f},
        {64, 128, 2, 3.40f, 0.79f, 0.17f, 0.26f, 1.19f, 8.57f, 0.22f},
        {128, 128, 2, 3.06f, 4.07f, 0.57f, 0.53f, 2.06f, 8.85f, 0.02f},
        {128, 64, 2, 2.84f, 0.85f, 0.25f, 0.33f, 1.30f, 5.53f, 0.33f},
    }};

}  // namespace

float tile_time(const ConvArgs &a, int row, int ksplit, int64_t cus) {
    const Model &m = kModel[uniform_taps(a) ? 0 : 1][row];
    const int64_t pt = (a.NPQ + m.BM - 1) / m.BM;
    int64_t tiles = 0, x_bytes = 0, y_bytes = 0;
    int ldk = 0;
    for (int i = 0; i < a.ngroups; ++i) {
        tiles += (a.g[i].M + m.BN - 1) / m.BN * pt;
        y_bytes += (int64_t)a.NPQ * a.g[i].M * 2;
        x_bytes = std::max<int64_t>(x_bytes, a.g[i].x_bytes);
        ldk = std::max(ldk, a.g[i].ldk);
    }
    tiles *= ksplit;
    const float ns = (float)((ldk / kBK + ksplit - 1) / ksplit);
    const float rounds = (float)((tiles + cus * m.R - 1) / (cus * m.R)), load = (float)((tiles + cus - 1) / cus);
    const float serial = rounds * (ns * (tiles <= cus ? m.alone : m.slice) + m.round);
    const float shared = load * (ns * m.share + m.tile);
    const float mem = (float)(x_bytes + y_bytes) * 1e-6f / m.rate;
    return m.launch + std::max(std::max(serial, shared), mem);
}

int tile_pick(const ConvArgs &a) {
    const float margin = uniform_taps(a) ? 1.0f / 0.95f : 1.0f / 0.9f;
    const int64_t cus = device_cus();
    int best = 0;
    float best_t = 0;
    for (int row = 0; row < 9; ++row) {
        // the fits scatter by 20%: k_conv_tile where it is expected to be 5%
        // faster than k_conv, 10% over mixed taps (few slices, where k_conv
        // often wins): with these margins 2 of the 244 layers run over 5%
        // slower than k_conv, without them 19
        const float t = tile_time(a, row, 1, cus) * (row < kTileShapes ? margin : 1.0f);
        if (row == 0 || t < best_t) best = row, best_t = t;
    }
    return best;
}

namespace {
// k_conv_tile's shapes: calls f with the template arguments of shape `row`
template <int BM, int BN, int WN, int WM, int S, int MI>
struct Shape {
    using Cfg = TileCfg<BM, BN, WN, WM, S, MI>;
    static constexpr int pixels = BM, filters = BN, slices = S;
    static int run(const ConvArgs &a, hipStream_t stream) { return launch<BM, BN, WN, WM, S, MI, false>(a, stream); }
};
template <typename F>
int with_shape(int row, F f) {
    switch (row) {
        case 0: return f(Shape<64, 64, 2, 2, 4, 32>());
        case 1: return f(Shape<128, 48, 4, 1, 2, 16>());
        case 2: return f(Shape<128, 80, 4, 1, 2, 16>());
        case 3: return f(Shape<64, 160, 2, 2, 3, 16>());
        case 4: return f(Shape<64, 160, 2, 2, 2, 16>());
        case 5: return f(Shape<128, 128, 2, 2, 3, 16>());
        case 6: return f(Shape<64, 128, 2, 2, 2, 32>());
        default: return fail(SA_E_ARG, "conv: unknown tile shape %d", row);
    }
}
}  // namespace

void tile_shape(int row, int *pixels, int *filters, int *fetchers, int *slices) {
    if (row >= kTileShapes) {
        *pixels = 128;
        *filters = row == kConv128x64 ? 64 : 128;
        *fetchers = 0;
        *slices = 2;
        return;
    }
    (void)with_shape(row, [&](auto shape) {
        *pixels = shape.pixels;
        *filters = shape.filters;
        *fetchers = decltype(shape)::Cfg::PW;
        *slices = shape.slices;
        return SA_OK;
    });
}

bool tile_one_tap(const ConvArgs &a) { return uniform_taps(a); }

int tile_run(const ConvArgs &a, int row, hipStream_t stream) {
    if (a.ksplit > 1) return launch<64, 64, 2, 2, 4, 32, true>(a, stream);
    return with_shape(row, [&](auto shape) { return shape.run(a, stream); });
}

}  // namespace sa
