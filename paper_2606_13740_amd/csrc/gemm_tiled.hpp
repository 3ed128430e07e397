// Tiled GEMM for many token rows (prompt processing, wide windows): Y = X W^T, where the
// streaming kernel's waves each fetch their own operand fragments and the matrix cores
// stay ~30% busy.
//
// Workgroup = 8 waves = 2 row halves x 4 token quarters; it owns RT row tiles x TT token
// tiles and a K range (split-K over grid.y, for partial sums).  K advances in steps of 32
// columns.  The operands are copied once per workgroup into LDS rings with direct
// global->LDS loads: a step's activation chunks (hi and lo plane per token tile), and the
// weights in their packed form, one chunk per row tile (32 columns bf16: one step; 64
// columns int8 / Q4_0: two steps, so half of a chunk's tiles, or its codes and then its
// scales, are copied per step).  Every wave multiplies its RT / 2 row tiles by its TT / 4
// token tiles from there.  The packed formats are the streaming kernel's (chunks are
// already in MFMA fragment order).  int8 is widened to bf16 and Q4_0 unpacked after the LDS
// read, by each wave that uses the chunk: one widening serves TT / 2 MFMAs of 16 cycles, so
// it hides behind the matrix cores at 16 token tiles and costs ~15% at 8.
//
// What bounds it: the matrix cores (two products per weight, hi and lo).  At 16 x 16 tiles a
// step is 64 MFMAs per wave against 16 KiB of LDS reads; read at the head of the step, as
// the scheduler arranges them, those take as long as half the MFMAs and nothing runs
// meanwhile.  So a step's barrier stands in the middle of its products, the next step's
// fragments are read under the second half, and each row tile's weights under the products
// of the one before: gate/up at 4096 rows 1128 -> 1047 us (1.57 PFLOP/s of MFMAs), one
// 16 x 16 step on an otherwise idle chip 1.26 -> 1.09 us of the 0.85 us its MFMAs take.
// Against the streaming layouts at 473 rows Q4_0: gate/up 321 -> 212 us, QKV 169 -> 122,
// O + down 227 -> 160; int8 at 4096 rows: gate/up 1643 -> 1285 us, O + down 981 -> 808;
// bf16 at 200 rows: gate/up 140 -> 103 us, QKV 99 -> 73, O + down 110 -> 79.
// Results go through the same epilogues, in four passes of TT / 4 token tiles.
#pragma once

#include "gemm.hpp"

namespace dllm {

template <int WT, int RT_, int TT_>
struct TiledShape {
    static_assert(WT == WT_BF16 || WT == WT_I8 || WT == WT_Q4, "tiled GEMM: bf16, int8 or Q4_0 weights");
    static_assert(RT_ % 2 == 0 && RT_ <= 16 && TT_ % 4 == 0 && TT_ <= 16, "at most 16 x 16 tiles");
    static constexpr int XPER = WTraits<WT>::XPER;   // steps (activation chunks) per weight chunk
    static constexpr int RT = RT_;                   // row tiles per workgroup
    static constexpr int TT = TT_;                   // token tiles per workgroup
    static constexpr int WR = RT / 2;                // row tiles per wave
    static constexpr int WM = TT / 4;                // token tiles per wave
    static constexpr int SX = 3;                     // activation ring slots
    static constexpr int SW = XPER == 1 ? 4 : 3;     // weight ring slots
    static constexpr int WCB = wchunk_bytes<WT>();   // bytes of a packed weight chunk
    static constexpr int WB = RT * WCB + (WT == WT_Q4 ? 1024 : 0);   // weight slot (+ Q4_0 scales)
    static constexpr int XB = TT * 2048;             // activation slot: hi + lo of every token tile
    static constexpr int XL = TT / 4;                // 1 KiB global->LDS loads per wave and step
    static constexpr int WL = XPER == 1 ? (RT + 7) / 8 : 1;
    static constexpr int LOADS = XL + WL;
    static constexpr int LDY = 16 * RT + 4;          // epilogue tile: [16 WM tokens][LDY]
    static constexpr int RING = SW * WB + SX * XB;
    static constexpr int YB = 16 * WM * LDY * 4;     // epilogue tile, then row scales and biases
    static constexpr int EPI = YB + 2 * 16 * RT * 4;
    static constexpr int SMEM = RING > EPI ? RING : EPI;
};

// m_tiles: token tiles of X; rows past them are never read (loads clamp to the last
// tile) and never written.
template <int WT, int RT_, int TT_, class Epi>
__global__ void __launch_bounds__(512) gemm_tiled_kernel(GemmArgs g, Epi epi, int m_tiles) {
    using T = TiledShape<WT, RT_, TT_>;
    constexpr int XPER = T::XPER;
    __shared__ __attribute__((aligned(1024))) char sm[T::SMEM];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave & 1, wq = wave >> 1;
    const int nt0 = blockIdx.x * T::RT, mt0 = blockIdx.z * T::TT;
    const int KC = g.KCw;
    const unsigned KS = gridDim.y;
    const int c0 = (int)((blockIdx.y * (unsigned)KC) / KS), c1 = (int)(((blockIdx.y + 1) * (unsigned)KC) / KS);
    const int steps = (c1 - c0) * XPER;
    char* const wring = sm;
    char* const xring = sm + T::SW * T::WB;

    // Buffer loads: the workgroup's operands sit behind 32-bit offsets from its first tile.
    // (With the global_load_lds form the compiler waited for every outstanding LDS read at
    // each use of one.)
    const char* const xsrc = (const char*)g.X + (size_t)mt0 * g.KCx * 2048;
    const char* const wsrc = (const char*)g.W + (size_t)nt0 * KC * T::WCB;
    [[maybe_unused]] const char* const qsrc = (const char*)g.qs + (size_t)nt0 * KC * 64;
    const int xlast = m_tiles - 1 - mt0, wlast = g.n_tiles - 1 - nt0;
    // activation chunks of step j: 1 KiB slot q = wave + 8i is token tile q / 2, plane q % 2
    auto stage_x = [&](int j, int slot) {
        const int kc = c0 * XPER + min(j, steps - 1);
        char* base = xring + slot * T::XB;
#pragma unroll
        for (int i = 0; i < T::XL; ++i) {
            const int q = wave + 8 * i;
            buffer_to_lds16(xsrc, lane * 16, (min(q >> 1, xlast) * g.KCx + kc) * 2048 + (q & 1) * 1024, base + q * 1024);
        }
    };
    // weight piece p.  bf16: the chunks of step p, row tiles wave, wave + 8.  int8: half
    // p % 2 of the row tiles of chunk p / 2.  Q4_0: the codes (p even, two tiles per load)
    // or the scales (p odd) of chunk p / 2.  A wave without a tile of its own repeats
    // another's copy (same bytes, same place), so that every wave has the same number of
    // loads in flight.
    auto stage_w = [&](int p, int slot) {
        char* base = wring + slot * T::WB;
        const int c = c0 + min(p / XPER, c1 - c0 - 1);
        if constexpr (XPER == 1) {
#pragma unroll
            for (int j = 0; j < T::WL; ++j) {
                const int q = wave + 8 * j;
                const int i = q < T::RT ? q : wave % T::RT;
                buffer_to_lds16(wsrc, lane * 16, (min(i, wlast) * KC + c) * 1024, base + i * 1024);
            }
        } else if constexpr (WT == WT_I8) {
            const int i = (p & 1) * (T::RT / 2) + wave % (T::RT / 2);
            buffer_to_lds16(wsrc, lane * 16, (min(i, wlast) * KC + c) * 1024, base + i * 1024);
        } else if ((p & 1) == 0) {
            const int q = wave % (T::RT / 2), i = 2 * q + (lane >> 5);
            buffer_to_lds16(wsrc, min(i, wlast) * KC * 512 + (lane & 31) * 16, c * 512, base + q * 1024);
        } else {
            const int i = min(lane >> 2, T::RT - 1);
            buffer_to_lds16(qsrc, min(i, wlast) * KC * 64 + (lane & 3) * 16, c * 64, base + T::RT * 512);
        }
    };

    f32x4_t acc[T::WR][T::WM];
#pragma unroll
    for (int f = 0; f < T::WR; ++f)
#pragma unroll
        for (int t = 0; t < T::WM; ++t) acc[f][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    if (steps > 0) {
        // Group s of loads: the activations of step s + 3 and the weights of step s + 3
        // (64-column chunks: piece s + 4, so that a chunk's second half is in the group its
        // first step needs); past the end, the last chunk again into a slot nobody reads.
        // Groups -3 .. -1 go out here, group s in the middle of step s, so each wave always
        // has exactly LOADS loads issued after the ones it waits for.
        auto wslot = [](int p) { return (p / XPER) % T::SW; };
        stage_w(0, 0);
        if constexpr (XPER == 2) stage_w(1, 0);
        stage_x(0, 0);
#pragma unroll
        for (int j = 1; j < 3; ++j) {
            stage_w(j + XPER - 1, wslot(j + XPER - 1));
            stage_x(j, j);
        }
        u32x4_t x[2][2 * T::WM];                   // activation fragments of a step (hi, lo) and of the next
        [[maybe_unused]] u32x2_t held[T::WR];      // second step's half of a 64-column chunk
        [[maybe_unused]] uint32_t hsc[T::WR];      // Q4_0: the chunk's two scales of this lane's row
        u32x4_t raw[2];
        const char* const xbase = xring + T::WM * wq * 2048 + lane * 16;
        auto read_x = [&](u32x4_t* d, int t, int slot) {
            d[2 * t] = *(const u32x4_t*)(xbase + slot * T::XB + t * 2048);
            d[2 * t + 1] = *(const u32x4_t*)(xbase + slot * T::XB + t * 2048 + 1024);
        };
        // weights of row tile f (XPER 2: only at a chunk's first step h = 0)
        auto read_w = [&](int f, int h, int slot) {
            const char* p = wring + slot * T::WB + (T::WR * wr + f) * T::WCB;
            if constexpr (WT == WT_BF16) {
                raw[f & 1] = *(const u32x4_t*)(p + lane * 16);
            } else if constexpr (WT == WT_I8) {
                if (h == 0) raw[f & 1] = *(const u32x4_t*)(p + lane * 16);
            } else if (h == 0) {
                held[f] = *(const u32x2_t*)(p + lane * 8);
                hsc[f] = *(const uint32_t*)(wring + slot * T::WB + T::RT * 512 + (T::WR * wr + f) * 64 +
                                            (lane & 15) * 4);
            }
        };
        // the products of row tile f with the wave's token tiles
        [[maybe_unused]] f32x4_t zp[T::WM];
        auto products = [&](int f, int h, const u32x4_t* xs, const u32x4_t& cur) {
            u32x4_t w;
            if constexpr (WT == WT_Q4) {
                w = q4_unpack(held[f][h]);
            } else if constexpr (WT == WT_I8) {
                if (h == 0) {
                    w = i8x8_to_bf16x8(cur[0], cur[1]);
                    held[f] = u32x2_t{cur[2], cur[3]};
                } else {
                    w = i8x8_to_bf16x8(held[f][0], held[f][1]);
                }
            } else {
                w = cur;
            }
            if constexpr (WT == WT_Q4) {
                const float sc = f16_bits_to_f32(h == 0 ? (hsc[f] & 0xFFFFu) : (hsc[f] >> 16));
#pragma unroll
                for (int t = 0; t < T::WM; ++t) {
                    f32x4_t v = mfma_bf16(xs[2 * t], w, zp[t]);
                    v = mfma_bf16(xs[2 * t + 1], w, v);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[f][t][e] = fmaf(sc, v[e], acc[f][t][e]);
                }
            } else {
#pragma unroll
                for (int t = 0; t < T::WM; ++t) {
                    acc[f][t] = mfma_bf16(w, xs[2 * t], acc[f][t]);
                    acc[f][t] = mfma_bf16(w, xs[2 * t + 1], acc[f][t]);
                }
            }
        };
        // every scalar load is done (lgkmcnt(0), other counters untouched): the compiler
        // does not see the waits in the asm below, and with a scalar load possibly
        // outstanding it would wait for all LDS reads at each use instead of counting them
        __builtin_amdgcn_s_waitcnt(0xC07F);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * T::LOADS) : "memory");
        int xs = 0, ws = 0;                        // ring slots of this step's activations and weights
        int wn = wslot(XPER == 1 ? 3 : 4);         // weight slot filled next
        auto next = [](int v, int n) { return v == n - 1 ? 0 : v + 1; };
        read_w(0, 0, 0);
#pragma unroll
        for (int t = 0; t < T::WM; ++t) read_x(x[0], t, 0);
        constexpr int F1 = T::WR / 2;              // row tiles before the step's barrier
        constexpr int XPF = (T::WM + T::WR - F1 - 1) / (T::WR - F1);   // token tiles read per row tile after it
        for (int i = 0; i < steps; i += 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (XPER == 1 && u == 1 && i + 1 >= steps) break;
                const int h = XPER == 1 ? 0 : u;
                const int xnext = next(xs, T::SX), wnext = (XPER == 1 || u == 1) ? next(ws, T::SW) : ws;
                if constexpr (WT == WT_Q4) {
                    // as in the streaming kernel: weights are the B operand, codes stand for
                    // 128 + q, a block's products start from -136 * sum_k x
                    const u32x4_t ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};   // bf16 1.0
#pragma unroll
                    for (int t = 0; t < T::WM; ++t) {
                        f32x4_t z = mfma_bf16(x[u][2 * t], ones, f32x4_t{0.f, 0.f, 0.f, 0.f});
                        z = mfma_bf16(x[u][2 * t + 1], ones, z);
#pragma unroll
                        for (int e = 0; e < 4; ++e) zp[t][e] = -136.0f * z[e];
                    }
                }
#pragma unroll
                for (int f = 0; f < T::WR; ++f) {
                    if (f == F1) {
                        // This wave's copies for step s + 1 have landed (group s - 1 may still be
                        // in flight); after the barrier every wave's have, and nobody reads the
                        // slots that group s refills: the activations of step s (already in
                        // registers everywhere) and the weights of step s - 1.  The next
                        // step's fragments are then read under the second half's products.
                        // (__syncthreads would also wait for group s - 1: the fence before its
                        // barrier waits for all outstanding vector memory operations.)
                        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(T::LOADS) : "memory");
                        stage_w(i + u + (XPER == 1 ? 3 : 4), wn);
                        stage_x(i + u + 3, xs);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    const u32x4_t cur = raw[f & 1];    // (an odd WR reads the next step's first tile into it)
                    if (f + 1 < T::WR) read_w(f + 1, h, ws);
                    else read_w(0, XPER == 1 ? 0 : h ^ 1, wnext);
                    if (f >= F1) {
#pragma unroll
                        for (int j = 0; j < XPF; ++j)
                            if ((f - F1) * XPF + j < T::WM) read_x(x[u ^ 1], (f - F1) * XPF + j, xnext);
                    }
                    products(f, h, x[u], cur);
                    __builtin_amdgcn_sched_barrier(0);
                }
                xs = xnext;
                ws = wnext;
                if (XPER == 1 || u == 1) wn = next(wn, T::SW);   // piece s + 5 starts the next chunk after an odd s
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();

    // epilogue: four passes of WM token tiles over the ring buffers
    float* Y = (float*)sm;
    float* ws_sm = (float*)(sm + T::YB);
    float* b_sm = ws_sm + 16 * T::RT;
    const int nrows = 16 * max(0, min(T::RT, g.n_tiles - nt0));
    const int r = lane & 15, gq = lane >> 4;
    const bool rowsc = g.wscale != nullptr || g.bias != nullptr;
    if (rowsc) {
        for (int n = threadIdx.x; n < nrows; n += blockDim.x) {
            ws_sm[n] = g.wscale != nullptr ? g.wscale[nt0 * 16 + n] : 1.f;
            b_sm[n] = g.bias != nullptr ? g.bias[nt0 * 16 + n] : 0.f;
        }
    }
    for (int p = 0; p < 4; ++p) {
        const int mtp = mt0 + T::WM * p;
        if (mtp >= m_tiles || nrows == 0) break;
        const int mcols = 16 * min(T::WM, m_tiles - mtp);
        if (wq == p) {
#pragma unroll
            for (int f = 0; f < T::WR; ++f)
#pragma unroll
                for (int t = 0; t < T::WM; ++t) {
                    const int n0 = 16 * (T::WR * wr + f), m0 = 16 * t;
                    if constexpr (WT == WT_Q4) {      // transposed: element i is token 4gq + i of row r
#pragma unroll
                        for (int i = 0; i < 4; ++i) Y[(m0 + 4 * gq + i) * T::LDY + n0 + r] = acc[f][t][i];
                    } else {
                        *(f32x4_t*)(Y + (m0 + r) * T::LDY + n0 + 4 * gq) = acc[f][t];
                    }
                }
        }
        __syncthreads();
        const YTokens<T::LDY> yv{Y};
        if (rowsc) {
            YScale sc;
            if (g.wscale != nullptr) sc.ws = ws_sm;
            if (g.bias != nullptr) sc.b = b_sm;
            epi(yv, nt0 * 16, nrows, mtp * 16, mcols, blockIdx.x, nullptr, sc);
        } else {
            epi(yv, nt0 * 16, nrows, mtp * 16, mcols, blockIdx.x, nullptr, NoScale{});
        }
        __syncthreads();
    }
}

// Split-K finish of the tiled kernel for the QKV projection of short prompts (whose
// tiles alone leave the chip half idle): each workgroup sums the KS partial slices
// P[s][m][n] of a 128-row x 32-token block in slice order into an LDS tile, adds the bias
// once, and runs the projection's epilogue on it, as the tiled kernel does with its own
// sums.  Bound by the latency of its loads: small blocks, so that every CU has several,
// and four loads per thread and slice in flight (200 rows, 2 slices: 18.6 us with one
// load at a time over 256 x 64 blocks).
constexpr int SPLIT_EPI_RT = 8, SPLIT_EPI_WM = 2;   // row tiles x token tiles per workgroup
template <class Epi>
__global__ void __launch_bounds__(256) split_epilogue_kernel(const float* P, int ks, int rows, int ldn, int n_tiles,
                                                             int m_tiles, const float* bias, Epi epi) {
    constexpr int RT = SPLIT_EPI_RT, WM = SPLIT_EPI_WM, LDY = 16 * RT + 4;
    __shared__ __attribute__((aligned(16))) float Y[16 * WM * LDY];
    const int nt0 = blockIdx.x * RT, mt0 = blockIdx.y * WM;
    const int nrows = 16 * min(RT, n_tiles - nt0), mcols = 16 * min(WM, m_tiles - mt0);
    const int n0 = nt0 * 16, m0 = mt0 * 16;
    const size_t slice = (size_t)rows * ldn;
    // four consecutive outputs of one token per item (16-byte loads along P's rows), U items
    // per thread in flight
    constexpr int U = 4;
    const int nq = nrows >> 2, nitems = nq * mcols;
    for (int base = threadIdx.x; base < nitems; base += U * blockDim.x) {
        const float* p[U];
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = min(base + u * (int)blockDim.x, nitems - 1);   // past the end: the last item again
            p[u] = P + (size_t)(m0 + idx / nq) * ldn + n0 + 4 * (idx % nq);
            v[u] = *(const float4*)p[u];
        }
#pragma unroll 3
        for (int k = 1; k < ks; ++k)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float4 w = *(const float4*)(p[u] + k * slice);
                v[u].x += w.x; v[u].y += w.y; v[u].z += w.z; v[u].w += w.w;
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = base + u * (int)blockDim.x;
            if (idx >= nitems) break;
            const int nl = 4 * (idx % nq), ml = idx / nq;
            if (bias != nullptr) {
                const float4 bv = *(const float4*)(bias + n0 + nl);
                v[u].x += bv.x; v[u].y += bv.y; v[u].z += bv.z; v[u].w += bv.w;
            }
            *(float4*)(Y + ml * LDY + nl) = v[u];
        }
    }
    __syncthreads();
    epi(YTokens<LDY>{Y}, n0, nrows, m0, mcols, blockIdx.x, nullptr, NoScale{});
}

}  // namespace dllm
