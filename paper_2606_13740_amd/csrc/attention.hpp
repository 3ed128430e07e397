// Window-vs-prefix attention (bidirectional inside the window, no causal mask).
//
// For a head h and a block of query rows, softmax(q k^T / sqrt(Dh)) v over keys
// [0, T) (or [0, lim[row]) for rows with their own limit), flash-style: the key
// range is cut into 32-key blocks; each wave streams its share of blocks with
// an online softmax; splits of the key range are merged by attn_combine.
//
// MFMA path, computed transposed so that no operand needs a shuffle:
//   S^T (16 keys x 16 queries) = K_tile (A: 16 keys x 32 dims) * Q^T (B)
//   O^T (16 dims x 16 queries) += V^T_tile (A: 16 dims x 32 keys) * P^T (B)
// K rows are loaded in the order key = 8*(r/4) + 4t + r%4 for tile t, so that
// lane group g ends up holding the probabilities of keys 8g .. 8g+7 of the
// block in B-operand order, and V^T (stored [dim][pos]) gives those 8 keys as
// one 16-byte load.
#pragma once

#include "common.hpp"

namespace dllm {

struct AttnArgs {
    const void* q;        // [rows][H][Dh]
    size_t q_plane;       // elements from the hi to the lo plane of q (fp16 path)
    const void* K;        // layer base [Hkv][Cs][Dh]
    const void* Vt;       // layer base [Hkv][Dh][Cs]
    int Cs;               // cache row stride (multiple of 32)
    int H;                // query heads
    int G;                // query heads per K/V head (grouped-query attention; 1 = multi-head)
    int T;                // keys [0, T) for rows without their own limit
    const int* lim;       // per-row key limit (rows < M) or nullptr
    int M;                // real rows
    int rows;             // rows of q and of the outputs (M padded to whole tiles)
    int nsplit, bps;      // key-range splits, 32-key blocks per split
    float scale;          // 1 / sqrt(Dh)
    void* o;              // output fragments (K = d), used when nsplit == 1
    int KCx;
    float* opart;         // [nsplit][rows_ld][H][Dh]  unnormalised partial outputs
    float* mlpart;        // [nsplit][rows_ld][H][2]   (running max in log2 units, sum)
    int rows_ld;
};

// fp16 MFMA path (v_mfma_f32_16x16x32_f16).  The cache holds K and V^T as one fp16
// plane each; Q arrives as an fp16 hi + lo pair and the probabilities P are split the
// same way in registers, so every product takes two MFMAs (K * Q_hi + K * Q_lo,
// V^T * P_hi + V^T * P_lo) and the scores and outputs keep the cache's precision.
//
// Workgroup = (key split, head, group of QG x QT query tiles of 16 rows), QG waves of QT
// tiles.  Each 32-key block of the split is staged in LDS once with direct global->LDS
// loads in a ring of NB buffers, so that later blocks stream in while one is used, and the
// waves read their MFMA fragments from there.  LDS rows are XOR-swizzled in 16-byte
// columns so that the 16 rows one fragment read touches fall in distinct banks:
//   K  [32 keys][Dh/8 cols]: col' = col ^ (((key & 3) | (4 * ((key >> 3) & 3))) mod Dh/8)
//   V^T [Dh dims][4 cols]:   col' = col ^ ((dim >> 2) & 3)
// With one split the normalised output goes to the O projection's fragments; otherwise
// (m, l, o) per split goes to attn_combine.
//
// What bounds it: short ranges, the launch and the chain of one block (LDS reads, scores,
// softmax, products; ~1 us); long ones, that chain on few waves, or at many query tiles
// the VALU work of the softmax beside the MFMAs.  Reading all of a block's fragments ahead
// of their products instead of at each took (with the merge, 32 heads) 64 rows over 4160
// keys from 25.7 to 22.4 us (8 splits, 3 buffers; 15 splits of 2 before), 32 rows over
// 544 keys from 9.7 to 9.0, 512 over 512 from 20.4 to 17.2, 256 over 1700 from 47.9 (no
// splits) to 28.2 (2 splits), and two tiles per wave 4096 over 4096 from 462 to 440 us.
__device__ __forceinline__ int swz_k(int key) { return (key & 3) | (((key >> 3) & 3) << 2); }

// At most two waves per SIMD's worth of registers (256): with the 512 a workgroup of
// 2-4 waves may take, the compiler chose the AGPR form of the MFMAs and copied every
// output tile VGPR -> AGPR around each product.
// log2-domain slack of the lazily rescaled softmax maximum: probabilities <= 2^8
constexpr float ATTN_SLACK = 8.f;

template <int DH, int QG, int QT, int NB>
__global__ void __launch_bounds__(QG * 64) __attribute__((amdgpu_waves_per_eu(2)))
attn_f16_kernel(AttnArgs a) {
    constexpr int NC = DH / 32;               // 32-dim chunks
    constexpr int ND = DH / 16;               // 16-dim output tiles
    constexpr int KCOLS = DH / 8;             // 16-byte columns per key row
    constexpr int KPLANE = 32 * DH * 2;       // bytes of a block's K (fp16)
    constexpr int VPLANE = DH * 64;           // bytes of a block's V^T (fp16)
    constexpr int BUF = KPLANE + VPLANE;
    constexpr int KI = KPLANE / 1024, VI = VPLANE / 1024;   // 1 KiB wave loads per block
    static_assert(KI * 1024 == KPLANE && VI * 1024 == VPLANE, "planes must be whole wave loads");
    static_assert(NB == 2 || NB == 3, "2 or 3 staging buffers");
    constexpr int LPW = KI / QG + VI / QG;    // loads each wave issues per staged block, at least
    __shared__ __attribute__((aligned(1024))) char lds[NB * BUF];

    const int lane = threadIdx.x & 63, qw = QG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    // 1-D grid over (head h, query group z, split) items, in that order.  The dispatcher
    // deals consecutive workgroups to the 8 XCDs in turn; XCD x takes the x-th of 8 shares
    // (the first nitems mod 8 hold one item more), so the query groups and splits of a
    // head (which read the same K/V, the splits adjacent 64-byte halves of the same
    // V^T lines) and the heads of a K/V group share one L2.  (Three Dream-7B layers, 28 heads
    // in 9 splits, 32 rows over 4032 keys: 404 us with the 252 items, which do not divide by
    // 8, in the dispatcher's order, 401 so; over 8032 keys 431 and 427.)
    const int nitems = (int)gridDim.x;
    const int nqg = nitems / (a.nsplit * a.H);
    const int xcd = blockIdx.x & 7;
    const int item = xcd * (nitems >> 3) + min(xcd, nitems & 7) + (int)(blockIdx.x >> 3);
    const int split = item % a.nsplit, z = (item / a.nsplit) % nqg, h = item / (a.nsplit * nqg);
    const int row = z * 16 * QG * QT + 16 * QT * qw + r;     // this lane's first query row (+ 16 per tile)
    const int ld = a.H * DH;
    const float sl2 = a.scale * 1.4426950408889634f;

    const uint16_t* qp = (const uint16_t*)a.q;
    const int hk = h / a.G;                                  // K/V head of this query head
    const uint16_t* Kp = (const uint16_t*)a.K + (size_t)hk * a.Cs * DH;
    const uint16_t* Vp = (const uint16_t*)a.Vt + (size_t)hk * DH * a.Cs;

    const int nblk = (a.T + 31) >> 5;
    const int kb0 = split * a.bps, kb1 = min(nblk, kb0 + a.bps);

    // Stage block kb into buffer `buf`: wave load i of a plane is its bytes [1024 i, 1024 i +
    // 1024), taken by wave i % QG.  Buffer loads from the head's planes (with the
    // global_load_lds form the compiler waited for every outstanding LDS read at each use
    // of one); no branch per load (one cost a 16-row window 2 us per launch).
    auto stage = [&](int kb, int buf) {
        const int k0 = kb * 32;
        char* base = lds + buf * BUF;
#pragma unroll
        for (int j = 0; j < (KI + QG - 1) / QG; ++j) {       // K: 32 x KCOLS slots
            const int i = qw + j * QG;
            if (KI % QG != 0 && i >= KI) break;
            const int key = (i * 64 + lane) / KCOLS, pc = lane % KCOLS;
            const int col = pc ^ (swz_k(key) & (KCOLS - 1));
            buffer_to_lds16(Kp, (key * DH + col * 8) * 2, k0 * DH * 2, base + i * 1024);
        }
#pragma unroll
        for (int j = 0; j < (VI + QG - 1) / QG; ++j) {       // V^T: DH x 4 slots
            const int i = qw + j * QG;
            if (VI % QG != 0 && i >= VI) break;
            const int dim = (i * 64 + lane) >> 2, pc = lane & 3;
            const int col = pc ^ ((dim >> 2) & 3);
            buffer_to_lds16(Vp, (dim * a.Cs + col * 8) * 2, k0 * 2, base + KPLANE + i * 1024);
        }
    };

    // zero the V^T values of keys >= T in the slots this wave staged into buffer `buf`
    // (cache rows past T may hold anything, and 0 * NaN would reach O); K needs no
    // such care, its scores past T are masked
    auto zero_tail = [&](int kb, int buf) {
        const int k0 = kb * 32;
        char* base = lds + buf * BUF + KPLANE;
#pragma unroll
        for (int j = 0; j < (VI + QG - 1) / QG; ++j) {
            const int i = qw + j * QG;
            if (VI % QG != 0 && i >= VI) break;
            const int dim = (i * 64 + lane) >> 2, pc = lane & 3;
            const int key = k0 + 8 * (pc ^ ((dim >> 2) & 3));      // the slot's first key
            if (key + 8 <= a.T) continue;
            u32x4_t* slot = (u32x4_t*)(base + i * 1024 + lane * 16);
            u32x4_t v = *slot;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] &= (key + 2 * e >= a.T ? 0u : 0x0000FFFFu) | (key + 2 * e + 1 >= a.T ? 0u : 0xFFFF0000u);
            *slot = v;
        }
    };

    u32x4_t qf[QT][NC][2];
    int lim[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        // Rows past the last real one repeat it: q holds what earlier calls left there, and
        // the rescale below is decided over all 16 rows of a tile, so a stale row would
        // reach the last bits of the real ones.
        const int rq = min(row + 16 * q, a.M - 1);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint16_t* src = qp + (size_t)rq * ld + h * DH + 32 * c + 8 * g;
            qf[q][c][0] = ldg16(src);
            qf[q][c][1] = ldg16(src + a.q_plane);
        }
        lim[q] = a.lim != nullptr ? a.lim[rq] : a.T;
    }

    // Ring of NB buffers: the first NB - 1 blocks are staged here (after the Q loads, so
    // the ring's waits below count only block loads issued after the block they wait
    // for), and round t stages block t + NB - 1 into the buffer round t - 1 used.  Every
    // split has a block.
    const int rounds = kb1 - kb0;
#pragma unroll
    for (int j = 0; j < NB - 1; ++j)
        if (j == 0 || j < rounds) stage(kb0 + j, j);

    // smallest key limit of the wave's rows (lanes 0-15 hold each tile's): blocks below it
    // need no per-key mask.  Read lane by lane into a scalar, so that the per-block
    // test is a scalar branch.
    int lim_w = a.T;
#pragma unroll
    for (int q = 0; q < QT; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) lim_w = min(lim_w, __builtin_amdgcn_readlane(lim[q], i));

    float mrun[QT], lrun[QT];
    f32x4_t oacc[QT][ND];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        mrun[q] = -INFINITY;
        lrun[q] = 0.f;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) oacc[q][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    const int krow0 = 8 * (r >> 2) + (r & 3);   // + 4t: the key this lane reads for tile t

    // no scalar load outstanding past here (lgkmcnt(0), other counters untouched): the
    // compiler does not see the waits in the loop's asm and would otherwise wait for all
    // LDS reads at each use
    __builtin_amdgcn_s_waitcnt(0xC07F);
    for (int t = 0; t < rounds; ++t) {
        const int kb = kb0 + t;
        const int cur = t % NB;
        // This wave's loads of block t have landed once at most LPW of the block staged after
        // it are outstanding (loads complete in issue order, and the loop issues no other
        // vector-memory operations); the barrier then makes every wave's loads visible and
        // frees the buffer round t - 1 read.  No workgroup fence: with loads into LDS in
        // flight it would wait for all of them.
        if (kb * 32 + 32 > a.T) {               // the block holding T: the last
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            zero_tail(kb, cur);                 // before the barrier, so no other wave reads first
        }
        if (NB > 2 && t + 1 < rounds) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LPW) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (t + NB - 1 < rounds) stage(kb + NB - 1, (t + NB - 1) % NB);
        const char* Kb = lds + cur * BUF;
        const char* Vb = Kb + KPLANE;
        const int k0 = kb * 32;

        // All of the block's K fragments are read before the first product and its V^T
        // fragments between the scores and the softmax, which covers their latency (read
        // at each use, every pair of products waited for its own LDS round trip).  The
        // QT tiles share both: at one tile per wave the LDS reads take as long as the
        // MFMAs.
        u32x4_t kf[NC][2], vf[ND];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int key = krow0 + 4 * t;
                const int off = key * (DH * 2) + (((4 * c + g) ^ (swz_k(key) & (KCOLS - 1))) << 4);
                kf[c][t] = *(const u32x4_t*)(Kb + off);
            }
        __builtin_amdgcn_sched_barrier(0);
        f32x4_t s[QT][2];
#pragma unroll
        for (int q = 0; q < QT; ++q) s[q][0] = s[q][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int q = 0; q < QT; ++q)
#pragma unroll
                    for (int t = 0; t < 2; ++t) s[q][t] = mfma_f16(kf[c][t], qf[q][c][p], s[q][t]);
        auto read_v = [&](int dt) {
            const int dim = 16 * dt + r;
            vf[dt] = *(const u32x4_t*)(Vb + dim * 64 + ((g ^ ((dim >> 2) & 3)) << 4));
        };
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) read_v(dt);
        __builtin_amdgcn_sched_barrier(0);

        u32x4_t ph[QT], pl[QT];
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            // unscaled scores of keys k0 + 8g + j (j = 0..7); keys past a row's limit -> -inf
            float sv[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sv[i] = s[q][0][i];
                sv[4 + i] = s[q][1][i];
            }
            if (k0 + 32 > lim_w) {                  // some row of the wave stops inside the block
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int key0 = k0 + 8 * g + i;
                    if (key0 >= lim[q]) sv[i] = -INFINITY;
                    if (key0 + 4 >= lim[q]) sv[4 + i] = -INFINITY;
                }
            }
            // the row's block maximum over its four lane groups (lanes l, l ^ 16, l ^ 32,
            // l ^ 48): each swap hands a lane its partner's value, and max is symmetric
            float bm = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])),
                             fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
            {
                const auto w32 =
                    __builtin_amdgcn_permlane32_swap(__float_as_uint(bm), __float_as_uint(bm), false, false);
                bm = fmaxf(__uint_as_float(w32[0]), __uint_as_float(w32[1]));
                const auto w16 =
                    __builtin_amdgcn_permlane16_swap(__float_as_uint(bm), __float_as_uint(bm), false, false);
                bm = fmaxf(__uint_as_float(w16[0]), __uint_as_float(w16[1]));
            }
            const float bms = bm * sl2;             // log2-domain block maximum (sl2 > 0)
            // Lazy rescaling: the reference maximum mrun moves only when some row of the
            // wave exceeds it by more than ATTN_SLACK (and on a row's first unmasked key),
            // so the probabilities stay <= 2^ATTN_SLACK and most blocks skip the rescale.
            // O, l and m are exact for any reference value; the split merge uses the same m.
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(bms > mrun[q] + ATTN_SLACK) != 0, 0)) {
                const float mnew = fmaxf(mrun[q], bms);
                const float alpha = (mnew == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(mrun[q] - mnew);
                lrun[q] *= alpha;
#pragma unroll
                for (int dt = 0; dt < ND; ++dt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) oacc[q][dt][i] *= alpha;
                mrun[q] = mnew;
            }
            // a row with no unmasked key yet keeps m = -inf; its masked scores give p = 0
            const float mref = (mrun[q] == -INFINITY) ? 0.f : mrun[q];
            float ps;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // v_exp_f32 directly: the arguments are <= ATTN_SLACK (or -inf); results below
                // 2^-126 (flushed to zero) are the only ones that differ from exp2f
                const float p0 = __builtin_amdgcn_exp2f(fmaf(sv[2 * e], sl2, -mref));
                const float p1 = __builtin_amdgcn_exp2f(fmaf(sv[2 * e + 1], sl2, -mref));
                ps = e ? ps + (p0 + p1) : p0 + p1;
                // hi = fp16 toward zero, lo = the remainder toward zero
                const auto hi = __builtin_amdgcn_cvt_pkrtz(p0, p1);
                const auto lo = __builtin_amdgcn_cvt_pkrtz(p0 - (float)hi[0], p1 - (float)hi[1]);
                ph[q][e] = __builtin_bit_cast(uint32_t, hi);
                pl[q][e] = __builtin_bit_cast(uint32_t, lo);
            }
            lrun[q] += ps;
        }
        // (V^T of keys past T was zeroed when the block holding T was staged)
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
#pragma unroll
            for (int q = 0; q < QT; ++q) {
                oacc[q][dt] = mfma_f16(vf[dt], ph[q], oacc[q][dt]);
                oacc[q][dt] = mfma_f16(vf[dt], pl[q], oacc[q][dt]);
            }
    }

    float l[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        l[q] = lrun[q] + __shfl_xor(lrun[q], 16);
        l[q] += __shfl_xor(l[q], 32);
    }
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        const int rq = row + 16 * q;
        if (rq >= a.rows) continue;
        if (a.nsplit == 1) {
            const float inv = 1.f / l[q];
#pragma unroll
            for (int dt = 0; dt < ND; ++dt)
                xfrag_store4<false>(a.o, rq, h * DH + 16 * dt + 4 * g, a.KCx,
                                    make_float4(oacc[q][dt][0] * inv, oacc[q][dt][1] * inv, oacc[q][dt][2] * inv,
                                                oacc[q][dt][3] * inv));
        } else {
            float* op = a.opart + (((size_t)split * a.rows_ld + rq) * a.H + h) * DH;
#pragma unroll
            for (int dt = 0; dt < ND; ++dt)
                *(float4*)(op + 16 * dt + 4 * g) =
                    make_float4(oacc[q][dt][0], oacc[q][dt][1], oacc[q][dt][2], oacc[q][dt][3]);
            if (g == 0) {
                float* ml = a.mlpart + (((size_t)split * a.rows_ld + rq) * a.H + h) * 2;
                ml[0] = mrun[q];
                ml[1] = l[q];
            }
        }
    }
}

// Merge key-range splits: O = sum_s o_s 2^(m_s - M) / sum_s l_s 2^(m_s - M).
// 32 lanes per (row, head), four consecutive dims per lane (head dims <= 128);
// ATTN_MERGE_PAIRS (row, head) pairs per workgroup: 4, so that a 32-row window over
// 32 heads gives every CU one workgroup (LLaDA-8B, 32 rows: attention + merge 13.8 ->
// 12.1 us per layer against 8 pairs and 128 workgroups; 2 pairs and 512 workgroups:
// no gain).
constexpr int ATTN_MERGE_PAIRS = 4;
template <bool XF32>
__global__ void __launch_bounds__(32 * ATTN_MERGE_PAIRS) attn_combine_kernel(AttnArgs a, int rows, int DH) {
    constexpr int MAXS = 16;                                   // = the runtime's split cap
    const int pair = blockIdx.x * ATTN_MERGE_PAIRS + (threadIdx.x >> 5);
    const int l = threadIdx.x & 31;
    if (pair >= rows * a.H) return;
    const int h = pair % a.H, row = pair / a.H;
    const size_t stride_s = (size_t)a.rows_ld * a.H;          // (row, head) records per split
    const size_t rec = (size_t)row * a.H + h;
    const int d0 = 4 * l;
    const bool has_d = d0 < DH;
    // every split's (m, l) and output loads go out before any is used: one memory
    // round trip
    float2 ml[MAXS];
    float4 v[MAXS];
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
        ml[s] = (s < a.nsplit) ? *(const float2*)(a.mlpart + (s * stride_s + rec) * 2)
                               : make_float2(-INFINITY, 0.f);
        v[s] = (s < a.nsplit && has_d) ? *(const float4*)(a.opart + (s * stride_s + rec) * DH + d0)
                                       : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < MAXS; ++s) mx = fmaxf(mx, ml[s].x);
    float w[MAXS], L = 0.f;
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
        w[s] = (ml[s].x == -INFINITY) ? 0.f : exp2f(ml[s].x - mx);
        L += ml[s].y * w[s];
    }
    const float inv = 1.f / L;
    if (!has_d) return;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int s = 0; s < MAXS; ++s) {
        o.x += v[s].x * w[s]; o.y += v[s].y * w[s]; o.z += v[s].z * w[s]; o.w += v[s].w * w[s];
    }
    xfrag_store4<XF32>(a.o, row, h * DH + d0, a.KCx, make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv));
}

// fp32 path (small models): one workgroup of 4 waves per (row, head); wave w takes 64-key
// chunks w, w + 4, ...  A chunk's scores have one key per lane, its output one dim (DH 128:
// two) per lane with the probabilities broadcast from LDS; the waves' states are merged in
// wave order.  Latency-bound: with a key per lane in both halves, the butterfly that merged
// 64 lanes' O vectors was most of the time (32 rows, 4 heads of 64, 96 keys: 57 -> 5.7 us).
constexpr int ATTN_F32_WAVES = 4;
template <int DH>
__global__ void __launch_bounds__(64 * ATTN_F32_WAVES) attn_f32_kernel(AttnArgs a) {
    constexpr int NW = ATTN_F32_WAVES, ND = (DH + 63) / 64;
    __shared__ __attribute__((aligned(16))) float q_s[DH];
    __shared__ __attribute__((aligned(16))) float p_s[NW][64];
    __shared__ float o_s[NW][DH], m_s[NW], l_s[NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = blockIdx.x, h = blockIdx.y;
    const int hk = h / a.G;                                  // K/V head of this query head
    const float* Kp = (const float*)a.K + (size_t)hk * a.Cs * DH;
    const float* Vp = (const float*)a.Vt + (size_t)hk * DH * a.Cs;
    const int lim = (a.lim != nullptr && row < a.M) ? a.lim[row] : a.T;
    if (threadIdx.x < DH) q_s[threadIdx.x] = ((const float*)a.q)[(size_t)row * a.H * DH + h * DH + threadIdx.x];
    __syncthreads();

    float m = -INFINITY, l = 0.f;                            // the same in every lane
    float o[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) o[d] = 0.f;
    for (int k0 = 64 * wave; k0 < lim; k0 += 64 * NW) {
        const int n = min(64, lim - k0);                     // keys past the limit are never read
        float s = -INFINITY;
        if (lane < n) {
            const float4* kr = (const float4*)(Kp + (size_t)(k0 + lane) * DH);
            s = 0.f;
#pragma unroll
            for (int j = 0; j < DH / 4; ++j) {
                const float4 kv = kr[j], qv = *(const float4*)(q_s + 4 * j);
                s = fmaf(qv.x, kv.x, s);
                s = fmaf(qv.y, kv.y, s);
                s = fmaf(qv.z, kv.z, s);
                s = fmaf(qv.w, kv.w, s);
            }
            s *= a.scale;
        }
        const float mn = fmaxf(m, warp_max(s));
        const float alpha = expf(m - mn);
        const float p = lane < n ? expf(s - mn) : 0.f;
        l = l * alpha + warp_sum(p);
        m = mn;
        p_s[wave][lane] = p;                                 // read back by the same wave only
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            const int dim = lane + 64 * d;
            if (dim >= DH) break;
            const float* vr = Vp + (size_t)dim * a.Cs + k0;
            float acc = o[d] * alpha;
            int j = 0;
#pragma unroll 8
            for (; j + 4 <= n; j += 4) {
                const float4 vv = *(const float4*)(vr + j), pv = *(const float4*)(p_s[wave] + j);
                acc = fmaf(pv.x, vv.x, acc);
                acc = fmaf(pv.y, vv.y, acc);
                acc = fmaf(pv.z, vv.z, acc);
                acc = fmaf(pv.w, vv.w, acc);
            }
            for (; j < n; ++j) acc = fmaf(p_s[wave][j], vr[j], acc);
            o[d] = acc;
        }
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int d = 0; d < ND; ++d)
        if (lane + 64 * d < DH) o_s[wave][lane + 64 * d] = o[d];
    if (lane == 0) {
        m_s[wave] = m;
        l_s[wave] = l;
    }
    __syncthreads();
    if (threadIdx.x < DH) {
        float mx = m_s[0];                                   // wave 0 always has a key
#pragma unroll
        for (int w = 1; w < NW; ++w) mx = fmaxf(mx, m_s[w]);
        float L = 0.f, ov = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float e = expf(m_s[w] - mx);               // 0 for a wave without keys
            L += l_s[w] * e;
            ov += o_s[w][threadIdx.x] * e;
        }
        xfrag_store<true>(a.o, row, h * DH + threadIdx.x, a.KCx, ov / L);
    }
}

}  // namespace dllm
