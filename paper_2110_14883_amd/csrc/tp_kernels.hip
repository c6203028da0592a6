// gfx950 (MI355X, CDNA4) kernels for one rank's share of a tensor-parallel linear layer
// (paper Section 2.2, tensor parallelism: the local block products of the 1D / 2D-SUMMA / 2.5D /
// 3D schemes, C = sum_k A_k B_k over the steps, then bias + erf-GeLU; and the two backward
// products).  bf16 operands, fp32 accumulation in MFMA 32x32x16 tiles.
//
// The eight-wave GEMM of this file serves operands that the 32-bit offsets of the other GEMM kernels cannot reach (and
// 256 x 256 tiles on request); the rest of the file holds the split-K fix-up and the elementwise kernels.  One kernel template
// serves the three memory forms (NN forward, NT dX, TN dW):
//   * persistent workgroups (one per CU) of 8 wave64 walk over the BM x BN tiles of C; a tile's
//     accumulators stay in registers across ALL steps and all K tiles -- no partial C leaves the
//     chip unless the host asked for a cross-workgroup split of K;
//   * ping-pong: waves 0-3 ("P", one per SIMD) stage operand A, waves 4-7 ("Q") stage operand B.
//     Inside one K tile P multiplies first and refills LDS afterwards, Q refills first and
//     multiplies afterwards, so every SIMD always has one wave with MFMAs ready while the other
//     one waits on global loads or writes LDS.  One workgroup barrier per K tile;
//   * K tiles of 64 are double-buffered in LDS (2 x 64 KB); the tile after next travels through
//     registers, fetched with 128-bit buffer loads whose out-of-range chunks read as zero (that
//     is how ragged M / K tails are masked);
//   * operands whose contraction index is not contiguous in memory are transposed in registers
//     (8 x 8 blocks, byte permutes) on the way into LDS, so the MFMA side always reads 8
//     consecutive k with one ds_read_b128; LDS rows are 128 B with the 16-byte chunk index
//     XOR-swizzled so that fragment reads and both kinds of writes are free of bank conflicts;
//   * the MFMA is issued with the operands swapped (C^T = B^T A^T) so that each lane ends up with
//     4 consecutive columns of one row of C: bias / GeLU / GeLU' run in registers, and each 32-row
//     slab then passes through a wave-private LDS patch so that the stores are whole 128-byte row
//     segments.  (This kernel's pipeline drains at every C tile: the next tile's first fetch is
//     issued after the epilogue.  The four-wave kernel of tp_gemm4.hip, which takes the 256 x 256
//     tiles, keeps its K tiles flowing across C tiles.)
//   * tile ids are spread so that each XCD (own L2) works on a compact patch of tiles.
#include "tp_device.h"

namespace tpl {

template <int V> using KS = std::integral_constant<int, V>;

struct TileCoord { int m0, n0, z, rot, g; };

// ---------------------------------------------------------------------------------------------
// one wave group's part of the GEMM (IS_P: waves 0-3, stage A;  else waves 4-7, stage B)
// ---------------------------------------------------------------------------------------------
template <int BM, int BN, bool A_KC, bool B_KC, int EPI, bool F32_OUT, bool IS_P>
__device__ __forceinline__ void gemm_role(const GemmArgs& p, char* lds, const int t, const int w) {
    constexpr int TM = BM / 64;      // 32-row MFMA tiles per wave along M (2 waves along M)
    constexpr int TN = BN / 128;     // 32-col MFMA tiles per wave along N (4 waves along N)
    constexpr int A_BYTES = BM * BK * 2;
    constexpr int STAGE_BYTES = (BM + BN) * BK * 2;
    constexpr int PART = IS_P ? 0 : A_BYTES;          // where this group's operand sits inside a stage
    using Stage = typename std::conditional<IS_P,
        typename std::conditional<A_KC, HalfKC<BM>, HalfXC<BM>>::type,
        typename std::conditional<B_KC, HalfKC<BN>, HalfXC<BN>>::type>::type;

    const int l = t & 63, tg = t & 255;
    const int wm = w & 1, wn = ((w >> 1) & 1) | ((w >> 2) << 1);   // P waves: wn in {0,1}; Q waves: wn in {2,3}
    const int ra = wm * (BM / 2) + (l & 31);       // fragment rows inside the wave's slab
    const int rb = wn * (BN / 4) + (l & 31);
    const int ch = l >> 5;                         // k chunk = 2 ks + lane/32
    char* const eps = lds + 2 * STAGE_BYTES + w * EPI_BYTES_PER_WAVE;   // wave-private epilogue patch

    const int KT = (p.K + BK - 1) / BK;
    const int T = p.n_steps * KT;
    const int Z = p.split_k;
    const int total = p.tiles_m * p.tiles_n * Z;

    Stage st;
    // Inside a step the K tiles are taken in a rotated order that differs from C tile to C tile, so
    // that the CUs of one XCD are not all asking the same memory channel for the same K offset.
    // Operand stream of this wave group.  The K tiles of a C tile are fetched strictly in order (units
    // z, z+Z, z+2Z, ... of the n_steps x KT sequence), so the step a fetch belongs to is tracked
    // incrementally: the operand block's pointer and leading dimension are re-read from the argument
    // block only when the step changes, and nothing is divided inside the K loop.
    int f_step = 0, f_kt = 0;                     // step (operand slot) and K tile inside it, before the rotation
    const uint16_t* f_ptr = nullptr;
    int f_ld = 0;
    auto open_step = [&](int s) __attribute__((always_inline)) {
        f_step = s;
        if constexpr (IS_P) { f_ptr = static_cast<const uint16_t*>(p.a[s]); f_ld = p.lda[s]; }
        else                { f_ptr = static_cast<const uint16_t*>(p.b[s]); f_ld = p.ldb[s]; }
    };
    auto seek = [&](const TileCoord& c, int unit) __attribute__((always_inline)) {
        const int s = unit / KT;
        f_kt = unit - s * KT;
        open_step(s + c.g);                       // a grouped launch has one step per group: operand slot = group
    };
    auto fetch_next = [&](const TileCoord& c) __attribute__((always_inline)) {
        int kt = f_kt + c.rot;
        if (kt >= KT) kt -= KT;
        const int k0 = kt * BK;
        // (the leading dimension is made opaque here: seen as loop-invariant, the per-lane row offsets
        // of all eight loads would be kept in registers across the K loop, which does not have them)
        asm volatile("" : "+s"(f_ld));
        if constexpr (IS_P) {
            if constexpr (A_KC) st.load(f_ptr, f_ld, p.M, c.m0, p.K, k0, tg);
            else                st.load(f_ptr, f_ld, p.K, k0, p.M, c.m0, tg);
        } else {
            if constexpr (B_KC) st.load(f_ptr, f_ld, p.N, c.n0, p.K, k0, tg);
            else                st.load(f_ptr, f_ld, p.K, k0, p.N, c.n0, tg);
        }
        f_kt += Z;
        while (f_kt >= KT && f_step + 1 < TP_MAX_STEPS) {      // (past the last step only after the tile's last fetch)
            f_kt -= KT;
            open_step(f_step + 1);
        }
    };
    auto locate = [&](int v) __attribute__((always_inline)) {
        int tm, tn, z;
        tile_of_id(p, v, tm, tn, z);
        const int rot = p.rotate ? ((tm * 3 + tn * 5) & 7) % KT : 0;
        int g = 0;
        if (p.n_groups > 1) {
            if (p.group_along_n) { g = tn / p.group_tiles; tn -= g * p.group_tiles; }
            else                 { g = tm / p.group_tiles; tm -= g * p.group_tiles; }
        }
        return TileCoord{tm * BM, tn * BN, z, rot, g};
    };

    f32x16_t acc[TM][TN];
    // One K tile = 4 MFMA k-steps.  The fragment reads of step ks+1 are issued while the MFMAs of
    // step ks run: the B fragments are double-buffered, an A fragment's registers are re-read as
    // soon as its two MFMAs have issued.  The sched_group_barrier calls pin that interleaving
    // (2 MFMA, 1 LDS read, ...), so a wave that multiplies alone still keeps the MFMA pipe busy.
    auto compute = [&](int cur) __attribute__((always_inline)) {
        const char* la = lds + cur * STAGE_BYTES;
        const char* lb = la + A_BYTES;
        bf16x8_t fa[TM], fb[2][TN];
#pragma unroll
        for (int j = 0; j < TN; ++j)
            fb[0][j] = *reinterpret_cast<const bf16x8_t*>(lb + lds_off(rb + 32 * j, ch));
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[i] = *reinterpret_cast<const bf16x8_t*>(la + lds_off(ra + 32 * i, ch));
        __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const bool more = ks + 1 < BK / 16;
            if (more) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    fb[(ks + 1) & 1][j] = *reinterpret_cast<const bf16x8_t*>(lb + lds_off(rb + 32 * j, 2 * (ks + 1) + ch));
                __builtin_amdgcn_sched_group_barrier(0x100, TN, 0);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks & 1][j], fa[i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, TN, 0);
                if (more) {
                    fa[i] = *reinterpret_cast<const bf16x8_t*>(la + lds_off(ra + 32 * i, 2 * (ks + 1) + ch));
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
            }
        }
        __builtin_amdgcn_s_setprio(0);
    };

    int v = blockIdx.x;
    if (v >= total) return;
    TileCoord cur_tile = locate(v);
    seek(cur_tile, cur_tile.z);
    fetch_next(cur_tile);

    while (true) {
        const int z = cur_tile.z;
        const int my_tiles = (T - z + Z - 1) / Z;       // K tiles z, z+Z, ...: every step is visited
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

        // K tile 0 -> LDS stage 0, K tile 1 -> registers
        st.store(lds + PART, tg);
        if (my_tiles > 1) fetch_next(cur_tile);
        __syncthreads();

        for (int i = 0; i < my_tiles; ++i) {
            const int cur = i & 1;
            char* refill = lds + (cur ^ 1) * STAGE_BYTES + PART;    // last read one iteration ago, by everybody
            if constexpr (IS_P) {
                compute(cur);
                if (i + 1 < my_tiles) st.store(refill, tg);
                if (i + 2 < my_tiles) fetch_next(cur_tile);
            } else {
                if (i + 1 < my_tiles) st.store(refill, tg);
                if (i + 2 < my_tiles) fetch_next(cur_tile);
                compute(cur);
            }
            __syncthreads();
        }


        // ---------------------------------------------------------------- epilogue
        // acc[i][j][e]: row m = 32 i + lane%32, columns n = 32 j + 8 (e/4) + 4 (lane/32) + e%4.
        // Bias / GeLU / GeLU' are applied in registers; every 32-row slab then passes through a
        // wave-private 4 KB LDS patch so that the global stores are whole 128-byte row segments.
        {
            const int m_sub = cur_tile.m0 + wm * (BM / 2);          // first row of this wave's slab
            const int n_sub = cur_tile.n0 + wn * (BN / 4);          // first column
            // (lane-derived values of the epilogue are formed here, from an opaque copy of the lane id, so
            // that none of them is computed ahead of the K loop and carried across it in a register)
            int le = l;
            asm volatile("" : "+v"(le));
            const int r = le & 31;                                  // row of this lane inside a 32-row slab
            const int ch = le >> 5;                                 // which half of each 8-column group this lane holds
            const int l = le;
            const bool partial = Z > 1;          // split K: raw fp32 partials, the fix-up kernel runs the epilogue
            constexpr bool use_bias = EPI == EPI_BIAS || EPI == EPI_BIAS_GELU;
            constexpr bool use_gelu = EPI == EPI_BIAS_GELU;
            constexpr bool use_dg = EPI == EPI_MUL_DGELU;
            const bool use_pre = !use_dg && p.pre != nullptr;

            // value functors: 4 consecutive columns (j, g) of row r of slab i
            auto raw4 = [&](int i, int j, int g, float (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * g + e];
            };
            auto preact4 = [&](int i, int j, int g, float (&v)[4]) __attribute__((always_inline)) {
                raw4(i, j, g, v);
                if constexpr (use_bias) {
                    const int n = n_sub + 32 * j + 8 * g + 4 * ch;
                    u32x2_t b = {0u, 0u};
                    if (n < p.N) b = *reinterpret_cast<const u32x2_t*>(static_cast<const uint16_t*>(p.bias) + n);
                    v[0] += bf16_lo(b[0]); v[1] += bf16_hi(b[0]); v[2] += bf16_lo(b[1]); v[3] += bf16_hi(b[1]);
                }
            };
            auto final4 = [&](int i, int j, int g, float (&v)[4]) __attribute__((always_inline)) {
                preact4(i, j, g, v);
                if constexpr (use_gelu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = gelu_f(v[e]);
                }
                if constexpr (use_dg) {
                    const int m = m_sub + 32 * i + r, n = n_sub + 32 * j + 8 * g + 4 * ch;
                    if (m < p.M && n < p.N) {
                        const u32x2_t a = *reinterpret_cast<const u32x2_t*>(static_cast<const uint16_t*>(p.dg) + (int64_t)m * p.lddg + n);
                        v[0] = dgelu_times(v[0], bf16_lo(a[0])); v[1] = dgelu_times(v[1], bf16_hi(a[0]));
                        v[2] = dgelu_times(v[2], bf16_lo(a[1])); v[3] = dgelu_times(v[3], bf16_hi(a[1]));
                    }
                }
            };
            // bf16 slab: rows of 32*TN bf16 (RB bytes); lane writes 8 bytes, reads back 16
            constexpr int RB = 32 * TN * 2, CPR = RB / 16, RPI = 64 / CPR;      // chunks per row, rows per instruction
            auto sw16 = [](int row) { return (row / (256 / RB)) & (CPR - 1); };
            auto slab_bf16 = [&](int i, auto value4, uint16_t* base, int64_t ld) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float x[4];
                        value4(i, j, g, x);
                        const u32x2_t v = {pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
                        *reinterpret_cast<u32x2_t*>(eps + r * RB + (((4 * j + g) ^ sw16(r)) << 4) + 8 * ch) = v;
                    }
#pragma unroll
                for (int it = 0; it < 32 / RPI; ++it) {
                    const int rr = it * RPI + l / CPR, c = l % CPR;
                    const u32x4_t v = *reinterpret_cast<const u32x4_t*>(eps + rr * RB + ((c ^ sw16(rr)) << 4));
                    const int m = m_sub + 32 * i + rr, n = n_sub + 8 * c;
                    if (m < p.M && n < p.N) *reinterpret_cast<u32x4_t*>(base + (int64_t)m * ld + n) = v;
                }
            };
            // fp32 slab, one 32-column block at a time: rows of 128 bytes; lane writes 16 bytes, reads back 16
            auto slab_f32 = [&](int i, auto value4, float* base, int64_t ld) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float x[4];
                        value4(i, j, g, x);
                        const f32x4_t v = {x[0], x[1], x[2], x[3]};
                        *reinterpret_cast<f32x4_t*>(eps + r * 128 + (((2 * g + ch) ^ ((r >> 1) & 7)) << 4)) = v;
                    }
#pragma unroll
                    for (int it = 0; it < 4; ++it) {
                        const int rr = it * 8 + (l >> 3), c = l & 7;
                        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(eps + rr * 128 + ((c ^ ((rr >> 1) & 7)) << 4));
                        const int m = m_sub + 32 * i + rr, n = n_sub + 32 * j + 4 * c;
                        if (m < p.M && n < p.N) *reinterpret_cast<f32x4_t*>(base + (int64_t)m * ld + n) = v;
                    }
                }
            };

            if (partial) {
                float* const wsz = p.ws + ((int64_t)z * p.n_groups + cur_tile.g) * p.M * p.N;
#pragma unroll
                for (int i = 0; i < TM; ++i) slab_f32(i, raw4, wsz, (int64_t)p.N);
            } else {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    if constexpr (!use_dg) {
                        if (use_pre) slab_bf16(i, preact4, static_cast<uint16_t*>(p.pre), p.ldp);
                    }
                    if constexpr (F32_OUT) slab_f32(i, final4, static_cast<float*>(p.outs[cur_tile.g]), p.ldos[cur_tile.g]);
                    else                   slab_bf16(i, final4, static_cast<uint16_t*>(p.outs[cur_tile.g]), p.ldos[cur_tile.g]);
                }
            }
        }
        v += gridDim.x;
        if (v >= total) break;
        cur_tile = locate(v);
        seek(cur_tile, cur_tile.z);
        fetch_next(cur_tile);
    }
}

template <int BM, int BN, bool A_KC, bool B_KC, int EPI, bool F32_OUT>
__global__ __launch_bounds__(NTHREADS) void tp_gemm_kernel(const GemmArgs p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int t = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);     // wave index, known uniform
    if (w < 4) gemm_role<BM, BN, A_KC, B_KC, EPI, F32_OUT, true>(p, lds, t, w);
    else       gemm_role<BM, BN, A_KC, B_KC, EPI, F32_OUT, false>(p, lds, t, w);
}

// ---------------------------------------------------------------------------------------------
// split-K fix-up: sum the fp32 partials in a fixed order, then the same epilogue.  Z: number of planes, all of a
// thread's loads in flight together.  Bound by memory (the planes), by latency where they are small.
// ---------------------------------------------------------------------------------------------
template <int Z>
__global__ __launch_bounds__(256) void tp_reduce_kernel(const ReduceArgs p, const uint32_t total, const Divisor d) {
    const uint32_t idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const int m = (int)quotient(d, idx), n = (int)(idx - m * d.d) * 4;
    Epilogue e{p.out, p.ldo, p.out_f32, p.pre, p.ldp, p.bias, p.gelu, p.dg, p.lddg};
    const float* const src = p.ws + (int64_t)m * p.N + n;
    f32x4_t q[Z];
#pragma unroll
    for (int z = 0; z < Z; ++z) q[z] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(src + z * p.plane));
    f32x4_t s = q[0];
#pragma unroll
    for (int z = 1; z < Z; ++z) { s[0] += q[z][0]; s[1] += q[z][1]; s[2] += q[z][2]; s[3] += q[z][3]; }
    float v[4] = {s[0], s[1], s[2], s[3]};
    epilogue4(e, v, m, n);
}

// ---------------------------------------------------------------------------------------------
// da = bf16(dy * GeLU'(pre)).  8 elements per 128-bit access.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ u32x4_t dgelu8(const u32x4_t g, const u32x4_t a) {
    u32x4_t o;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        o[i] = pack_bf16(dgelu_times(bf16_lo(g[i]), bf16_lo(a[i])), dgelu_times(bf16_hi(g[i]), bf16_hi(a[i])));
    return o;
}
// One 128-bit access per thread and a grid that covers the block: neighbouring workgroups then touch neighbouring memory, which
// measured 15 % faster than a persistent grid-stride loop with several loads in flight; the streaming (nontemporal) hint on loads and
// stores is worth another 9 %: 4096 x 24576 in 92 us, 6.6 TB/s (98 us with a 64-bit division a thread), against 5.9 for a plain bf16 add.
__global__ __launch_bounds__(256) void tp_dgelu_kernel(const uint16_t* dy, int64_t ld_dy, const uint16_t* pre, int64_t ld_pre, uint16_t* da,
                                                       int64_t ld_da, const uint32_t total, const Divisor d) {
    const uint32_t idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const int64_t r = quotient(d, idx);
    const uint32_t c = (idx - (uint32_t)r * d.d) * 8;
    const u32x4_t g = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(dy + r * ld_dy + c));
    const u32x4_t a = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(pre + r * ld_pre + c));
    __builtin_nontemporal_store(dgelu8(g, a), reinterpret_cast<u32x4_t*>(da + r * ld_da + c));
}

// y = [GeLU](c + bias) over an fp32 block (what follows the summation of forward partials), optional bf16 copy of
// c + bias; 4 elements per thread (8 are 8 % slower), same launch shape and hints as tp_dgelu_kernel.  What is written is
// compiled in: between branches the second store waits for the first.
template <bool GELU, bool PRE, bool F32>
__global__ __launch_bounds__(256) void tp_bias_act_kernel(const float* c, int64_t ldc, const uint16_t* bias, void* y, int64_t ldy, uint16_t* pre,
                                                          int64_t ldp, const uint32_t total, const Divisor d) {
    const uint32_t idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const int64_t r = quotient(d, idx);
    const uint32_t n = (idx - (uint32_t)r * d.d) * 4;
    f32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(c + r * ldc + n));
    if (bias) {
        const u32x2_t b = *reinterpret_cast<const u32x2_t*>(bias + n);
        v[0] += bf16_lo(b[0]); v[1] += bf16_hi(b[0]); v[2] += bf16_lo(b[1]); v[3] += bf16_hi(b[1]);
    }
    if constexpr (PRE) {
        const u32x2_t s = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        __builtin_nontemporal_store(s, reinterpret_cast<u32x2_t*>(pre + r * ldp + n));
    }
    if constexpr (GELU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = gelu_f(v[i]);
    }
    if constexpr (F32) {
        __builtin_nontemporal_store(v, reinterpret_cast<f32x4_t*>(static_cast<float*>(y) + r * ldy + n));
    } else {
        const u32x2_t o = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        __builtin_nontemporal_store(o, reinterpret_cast<u32x2_t*>(static_cast<uint16_t*>(y) + r * ldy + n));
    }
}

// Column sums of a bf16 [rows][cols] block into fp32.  Workgroup (bx, by) sums rows
// [by * rows_per_split, ...) of columns COLS bx .. COLS (bx + 1) - 1 into out[by][cols]; with one split that is the
// result, with several tp_colsum_finish_kernel adds the splits.  Every order of summation is fixed by the rows, the columns
// and the number of splits, whatever COLS is: the result is reproducible.
// FROM_DY: the block does not exist yet; it is formed on the way, da = dy * GeLU'(pre), and written.  The own dA
// block and its bias gradient then take one pass over memory (6 bytes per element) instead of 8 and one launch less;
// the sums are those of the finished block, bit for bit.  Bound by memory, and by latency where a workgroup walks many
// rows or there are few workgroups: launch_dgelu_colsum has both sides.
constexpr int COLSUM_LANES = 32;                              // rows side by side
template <bool FROM_DY, int COLS>
__global__ __launch_bounds__(COLS * 4) void tp_colsum_kernel(const uint16_t* dy, int64_t ld_dy, const uint16_t* pre, int64_t ld_pre,
                                                             uint16_t* da, int64_t ld, int64_t rows, int cols, float* out,
                                                             int64_t rows_per_split) {
    __shared__ float part[COLSUM_LANES][COLS + 1];
    constexpr int CL = COLS / 8;                                  // chunk lanes x 32 row lanes
    const int cl = threadIdx.x % CL, rl = threadIdx.x / CL;
    const int c = blockIdx.x * COLS + cl * 8;
    const int64_t r_begin = (int64_t)blockIdx.y * rows_per_split;
    const int64_t r_end = r_begin + rows_per_split < rows ? r_begin + rows_per_split : rows;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    // rows r0 + rl + 32 u, u < n, in flight together; FULL: all of them exist, else those past the end are loaded from the
    // last row and dropped
    auto some_rows = [&](auto n_, auto full_, int64_t r0) __attribute__((always_inline)) {
        constexpr int n = decltype(n_)::value;
        constexpr bool FULL = decltype(full_)::value;
        u32x4_t v[n], a[n];
#pragma unroll
        for (int u = 0; u < n; ++u) {
            int64_t row = r0 + rl + COLSUM_LANES * u;
            if (!FULL && row >= r_end) row = r_end - 1;
            const u32x4_t* const src = reinterpret_cast<const u32x4_t*>(FROM_DY ? dy + row * ld_dy + c : da + row * ld + c);
            if constexpr (FROM_DY || n > 1) v[u] = __builtin_nontemporal_load(src);
            else                            v[u] = *src;
            if constexpr (FROM_DY) a[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(pre + row * ld_pre + c));
        }
#pragma unroll
        for (int u = 0; u < n; ++u) {
            const int64_t row = r0 + rl + COLSUM_LANES * u;
            if (!FULL && row >= r_end) break;
            if constexpr (FROM_DY) {
                v[u] = dgelu8(v[u], a[u]);
                __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4_t*>(da + row * ld + c));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) { s[2 * i] += bf16_lo(v[u][i]); s[2 * i + 1] += bf16_hi(v[u][i]); }
        }
    };
    if (c < cols) {
        int64_t r = r_begin;
        if constexpr (FROM_DY) {                                  // the remainder in one batch: each trip is two loads, GeLU' and a store
            for (; r + 4 * COLSUM_LANES <= r_end; r += 4 * COLSUM_LANES) some_rows(std::integral_constant<int, 4>{}, std::true_type{}, r);
            const int64_t left = (r_end - r + COLSUM_LANES - 1) / COLSUM_LANES;
            if (left > 3)       some_rows(std::integral_constant<int, 4>{}, std::false_type{}, r);
            else if (left == 3) some_rows(std::integral_constant<int, 3>{}, std::false_type{}, r);
            else if (left == 2) some_rows(std::integral_constant<int, 2>{}, std::false_type{}, r);
            else if (left == 1) some_rows(std::integral_constant<int, 1>{}, std::false_type{}, r);
        } else {
            for (; r + rl + 3 * COLSUM_LANES < r_end; r += 4 * COLSUM_LANES) some_rows(std::integral_constant<int, 4>{}, std::true_type{}, r);
            for (; r + rl < r_end; r += COLSUM_LANES) some_rows(std::integral_constant<int, 1>{}, std::true_type{}, r);
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) part[rl][cl * 8 + i] = s[i];
    __syncthreads();
    if (threadIdx.x < COLS) {
        float tot = 0.0f;
#pragma unroll
        for (int r = 0; r < COLSUM_LANES; ++r) tot += part[r][threadIdx.x];
        const int cc = blockIdx.x * COLS + threadIdx.x;
        if (cc < cols) out[(int64_t)blockIdx.y * cols + cc] = tot;
    }
}
// Bound by latency: 8 threads share a column's (at most 64) splits, each adding every eighth in ascending order, and
// their sums meet in LDS.  (One thread a column, in a chain of loads, took 5 - 9 us.)
__global__ __launch_bounds__(256) void tp_colsum_finish_kernel(const float* part, int splits, int cols, float* out) {
    __shared__ float sums[8][32];
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5, c = blockIdx.x * 32 + x;
    float tot = 0.0f;
    if (c < cols) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = y + 8 * i;
            if (r < splits) tot += part[(int64_t)r * cols + c];
        }
    }
    sums[y][x] = tot;
    __syncthreads();
    if (y == 0 && c < cols) {
#pragma unroll
        for (int i = 1; i < 8; ++i) tot += sums[i][x];
        out[c] = tot;
    }
}

// ---------------------------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------------------------
void tile_shape(int tile_id, int* bm, int* bn) {
    switch (tile_id) {
        case TILE_128x256: *bm = 128; *bn = 256; break;
        case TILE_256x128: *bm = 256; *bn = 128; break;
        case TILE_128x128: *bm = 128; *bn = 128; break;
        default:           *bm = 256; *bn = 256; break;
    }
}

template <int BM, int BN, bool A_KC, bool B_KC, int EPI, bool F32_OUT>
static hipError_t launch_one(const GemmArgs& a, hipStream_t stream) {
    constexpr int lds_bytes = 2 * (BM + BN) * BK * 2 + 8 * EPI_BYTES_PER_WAVE;
    // the LDS limit is a per-device attribute of the kernel: set it once on every device that launches
    // it (same value every time, so a repeated or concurrent set is harmless)
    static std::atomic<uint64_t> attr_done{0};
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_done.load(std::memory_order_relaxed) & bit)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tp_gemm_kernel<BM, BN, A_KC, B_KC, EPI, F32_OUT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        attr_done.fetch_or(bit, std::memory_order_relaxed);
    }
    // persistent: never more workgroups than the chip holds at once (one per CU with this much LDS)
    const int total = a.tiles_m * a.tiles_n * a.split_k;
    const unsigned grid = (unsigned)(total < a.max_workgroups ? total : a.max_workgroups);
    return launch_kernel(tp_gemm_kernel<BM, BN, A_KC, B_KC, EPI, F32_OUT>, dim3(grid), dim3(NTHREADS), lds_bytes, stream, a);
}

template <int BM, int BN>
static hipError_t launch_tile(int form, const GemmArgs& a, hipStream_t s) {
    // the epilogue is compiled in, per memory form: forward (NN) adds bias / GeLU, dX (NT) may
    // multiply by GeLU', dW (TN) stores plain fp32.  A launch that splits K writes raw partials.
    const int epi = a.split_k > 1 ? EPI_NONE : (a.dg ? EPI_MUL_DGELU : (a.gelu ? EPI_BIAS_GELU : (a.bias ? EPI_BIAS : EPI_NONE)));
    const bool f32 = a.split_k > 1 || a.out_f32;
    switch (form) {
        case FORM_NN:
            if (epi == EPI_BIAS_GELU) return f32 ? launch_one<BM, BN, true, false, EPI_BIAS_GELU, true>(a, s) : launch_one<BM, BN, true, false, EPI_BIAS_GELU, false>(a, s);
            if (epi == EPI_BIAS)      return f32 ? launch_one<BM, BN, true, false, EPI_BIAS, true>(a, s) : launch_one<BM, BN, true, false, EPI_BIAS, false>(a, s);
            if (epi == EPI_NONE)      return f32 ? launch_one<BM, BN, true, false, EPI_NONE, true>(a, s) : launch_one<BM, BN, true, false, EPI_NONE, false>(a, s);
            return hipErrorInvalidValue;
        case FORM_NT:
            if (epi == EPI_MUL_DGELU) return f32 ? launch_one<BM, BN, true, true, EPI_MUL_DGELU, true>(a, s) : launch_one<BM, BN, true, true, EPI_MUL_DGELU, false>(a, s);
            if (epi == EPI_NONE)      return f32 ? launch_one<BM, BN, true, true, EPI_NONE, true>(a, s) : launch_one<BM, BN, true, true, EPI_NONE, false>(a, s);
            return hipErrorInvalidValue;
        case FORM_TN:
            if (epi == EPI_NONE && f32) return launch_one<BM, BN, false, false, EPI_NONE, true>(a, s);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

// Whether stores of an output, one of `total` bytes in this launch, carry the streaming hint (why: store_c_block).  A streamed piece of a 64-byte
// sector goes to memory as it is, and a row off those boundaries has one at both ends of every tile's segment: over a product's time more than
// memory takes.  Nothing else of an output that size stays in the 32 MB of the L2s either; a small one is better off leaving early all the same.
// Rows off the boundaries, with the hint / without, us: 24777 x 5640 fp32, K = 216 300 / 182; 17425 x 3432 fp32, K = 200 132 / 78; two of
// 11015 x 3000 fp32, K = 64 146 / 82; 6144 x 5256 bf16 twice, K = 768 86 / 72.  Means over 413 drawn products from memory / cached, by outputs:
// below 16 MB 1.02 / 0.99 x, 16 to 35 MB 0.98 / 0.91, 35 to 90 0.91 / 0.87, beyond 0.81 / 0.76.
static bool streams(const void* p, int64_t ld, int es, int64_t total) {
    return total <= (16 << 20) || (((uint64_t)(uintptr_t)p | (uint64_t)(ld * es)) & 63) == 0;
}

// A plain launch is one group whose output is `out`; false: a grouped one that does not hold together.
static bool normalise(GemmArgs& a) {
    if (a.tiles_m < 1 || a.tiles_n < 1 || a.group_m < 1) return false;
    a.by_tiles = divisor((uint32_t)(a.tiles_m * a.tiles_n));
    a.by_group = divisor((uint32_t)(a.group_m * a.tiles_n));
    a.by_height = divisor((uint32_t)a.group_m);
    a.by_last = divisor((uint32_t)(a.tiles_m % a.group_m ? a.tiles_m % a.group_m : a.group_m));
    if (a.n_groups <= 1) {
        a.n_groups = 1; a.group_along_n = 1; a.group_tiles = a.tiles_n;
        a.outs[0] = a.out; a.ldos[0] = a.ldo;
    } else if (a.n_steps != 1 || a.n_groups > TP_MAX_STEPS || a.group_tiles < 1 || a.bias || a.dg || a.pre ||
               (a.group_along_n ? a.tiles_n : a.tiles_m) != a.n_groups * a.group_tiles) {
        return false;
    }
    const int es = a.out_f32 ? 4 : 2;
    const int64_t total = (int64_t)a.M * a.N * (es * a.n_groups + (a.pre ? 2 : 0));
    a.stream = !a.pre || streams(a.pre, a.ldp, 2, total);
    for (int g = 0; g < a.n_groups; ++g) a.stream &= streams(a.outs[g], a.ldos[g], es, total);
    return true;
}

hipError_t launch_gemm_pair(int tile_x, const GemmArgs& x, int tile_w, const GemmArgs& w, hipStream_t s) {
    GemmArgs nx = x, nw = w;
    if (!normalise(nx) || !normalise(nw)) return hipErrorInvalidValue;
    return launch_small_pair(tile_x, nx, tile_w, nw, s);
}

hipError_t launch_gemm(int form, int tile_id, const GemmArgs& args, hipStream_t s) {
    GemmArgs a = args;
    if (!normalise(a)) return hipErrorInvalidValue;
    switch (tile_id) {
        case TILE_256x256: return launch_tile<256, 256>(form, a, s);
        case TILE_128x256: return launch_tile<128, 256>(form, a, s);
        case TILE_256x128: return launch_tile<256, 128>(form, a, s);
        case TILE_128x128: return launch_tile<128, 128>(form, a, s);
        case TILE_256x256_W4: return launch_gemm4(form, a, s);
        case TILE_128x256_MS: case TILE_256x128_MS: case TILE_128x128_MS: return launch_gemm_ms(form, tile_id, a, s);
        case TILE_32x32_SMALL: case TILE_16x32_SMALL: case TILE_32x16_SMALL: case TILE_16x16_SMALL: case TILE_16x64_SMALL: case TILE_32x64_SMALL: return launch_small(form, tile_id, a, s);
        default: return hipErrorInvalidValue;
    }
}

// f(first row, rows, threads, Divisor): launches over the rows of a block, at most 2^31 - 1 threads each
template <class F>
static hipError_t over_rows(int64_t rows, int64_t per_row, F&& f) {
    if (rows <= 0 || per_row <= 0) return hipSuccess;
    if (per_row >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    const Divisor d = divisor((uint32_t)per_row);
    const int64_t most = (((int64_t)1 << 31) - 1) / per_row;
    for (int64_t r = 0; r < rows; r += most) {
        const int64_t n = rows - r < most ? rows - r : most;
        if (hipError_t e = f(r, n, (uint32_t)(n * per_row), d); e != hipSuccess) return e;
    }
    return hipSuccess;
}
static dim3 covering(uint32_t threads) { return dim3((threads + 255u) / 256u); }

template <int Z>
static hipError_t reduce_planes(const ReduceArgs& a, hipStream_t s) {
    return over_rows(a.M, a.N >> 2, [&](int64_t r, int64_t n, uint32_t total, Divisor d) {
        ReduceArgs p = a;
        p.M = (int32_t)n;
        p.ws += r * a.N;
        p.out = static_cast<char*>(a.out) + r * a.ldo * (a.out_f32 ? 4 : 2);
        if (a.pre) p.pre = static_cast<char*>(a.pre) + r * a.ldp * 2;
        if (a.dg) p.dg = static_cast<const char*>(a.dg) + r * a.lddg * 2;
        return launch_kernel(tp_reduce_kernel<Z>, covering(total), dim3(256), 0, s, p, total, d);
    });
}
hipError_t launch_reduce(const ReduceArgs& a, hipStream_t s) {
    switch (a.split_k) {
        case 2: return reduce_planes<2>(a, s);
        case 3: return reduce_planes<3>(a, s);
        case 4: return reduce_planes<4>(a, s);
        case 5: return reduce_planes<5>(a, s);
        case 6: return reduce_planes<6>(a, s);
        case 7: return reduce_planes<7>(a, s);
        case 8: return reduce_planes<8>(a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_dgelu(const void* dy, int64_t ld_dy, const void* pre, int64_t ld_pre, void* da, int64_t ld_da,
                        int64_t rows, int64_t cols, hipStream_t s) {
    return over_rows(rows, cols >> 3, [&](int64_t r, int64_t, uint32_t total, Divisor d) {
        return launch_kernel(tp_dgelu_kernel, covering(total), dim3(256), 0, s, static_cast<const uint16_t*>(dy) + r * ld_dy, ld_dy,
                             static_cast<const uint16_t*>(pre) + r * ld_pre, ld_pre, static_cast<uint16_t*>(da) + r * ld_da, ld_da, total, d);
    });
}

template <bool GELU, bool PRE, bool F32>
static hipError_t bias_act(const float* c, int64_t ldc, const void* bias, void* y, int64_t ldy, void* pre, int64_t ldp, int64_t rows,
                           int64_t cols, hipStream_t s) {
    return over_rows(rows, cols >> 2, [&](int64_t r, int64_t, uint32_t total, Divisor d) {
        return launch_kernel(tp_bias_act_kernel<GELU, PRE, F32>, covering(total), dim3(256), 0, s, c + r * ldc, ldc, static_cast<const uint16_t*>(bias),
                             static_cast<void*>(static_cast<char*>(y) + r * ldy * (F32 ? 4 : 2)), ldy,
                             PRE ? static_cast<uint16_t*>(pre) + r * ldp : nullptr, ldp, total, d);
    });
}
hipError_t launch_bias_act(const float* c, int64_t ldc, const void* bias, int gelu, void* y, int64_t ldy, int y_f32,
                           void* pre, int64_t ldp, int64_t rows, int64_t cols, hipStream_t s) {
    auto pick = [&](auto g, auto p) {
        return y_f32 ? bias_act<decltype(g)::value, decltype(p)::value, true>(c, ldc, bias, y, ldy, pre, ldp, rows, cols, s)
                     : bias_act<decltype(g)::value, decltype(p)::value, false>(c, ldc, bias, y, ldy, pre, ldp, rows, cols, s);
    };
    using Y = std::true_type;
    using N = std::false_type;
    return gelu ? (pre ? pick(Y{}, Y{}) : pick(Y{}, N{})) : (pre ? pick(N{}, Y{}) : pick(N{}, N{}));
}

// Row splits that the workspace of a column sum is sized for: columns counted in strips of 64, workgroups enough to fill the
// chip four times over, at least 256 rows each.  (Callers size workspaces by this; how many splits run, and how wide
// the strips are, is decided below within it.)
int colsum_splits(int64_t rows, int64_t cols) {
    const int64_t col_blocks = (cols + 63) / 64;
    if (col_blocks >= 256) return 1;                    // one workgroup per 64 columns already fills the chip
    int64_t r = col_blocks > 0 ? (1024 + col_blocks - 1) / col_blocks : 1;
    const int64_t by_rows = (rows + 255) / 256;
    if (r > by_rows) r = by_rows;
    if (r > 64) r = 64;
    return r < 1 ? 1 : (int)r;
}
size_t colsum_ws_bytes(int64_t rows, int64_t cols) {
    const int r = colsum_splits(rows, cols);
    return r > 1 ? (size_t)r * (size_t)cols * 4 : 0;
}
// How the sum runs.  Times in us, replayed graphs.
struct ColsumPlan { int splits; bool wide; int64_t per; };
ColsumPlan colsum_plan(int64_t rows, int64_t cols, bool has_ws, bool from_dy) {
    ColsumPlan p;
    // up to 512 rows one slab: a second one costs the finish launch (300 x 1024: 3.1 against 4.8, 300 x 8192 3.3 / 5.0)
    p.splits = has_ws && rows > 512 ? colsum_splits(rows, cols) : 1;
    p.per = p.splits == 1 ? rows : ((rows + p.splits - 1) / p.splits + 31) / 32 * 32;
    // Strips of 128 columns (256-byte pieces of a row) where they make workgroups enough, else 64 (twice the workgroups).
    // One slab: 128 once the narrow ones no longer fit one to a CU: 4096 x 16384 31.4 against 29.2 (64), 4096 x 20480 34.6 / 44.0,
    // 2048 x 2560 14.4 / 13.0.  Several: 4096 x 1024 (128 workgroups) 6.5 / 5.3, 1024 x 6184 (196) 7.0 / 7.5, 4096 x 8192 15.5 / 16.7.
    // Few rows keep 64 (600 x 6184, three slabs, 7.4 / 6.0; 150 x 24576 3.8 / 3.3) unless dA is formed too (600 x 20480 19.4 / 24.4,
    // 600 x 12288, three slabs, 14.2 / 15.4).
    const int64_t strips = (cols + 127) / 128;
    p.wide = strips * p.splits > 128 && (rows >= 1024 || (from_dy && (p.splits == 1 || strips * p.splits > 256)));
    return p;
}
template <bool FROM_DY, int COLS>
static hipError_t colsum_passes(const ColsumPlan& p, const uint16_t* dy, int64_t ld_dy, const uint16_t* pre, int64_t ld_pre, uint16_t* da,
                                int64_t ld, int64_t rows, int64_t cols, float* out, float* ws, hipStream_t s) {
    const unsigned strips = (unsigned)((cols + COLS - 1) / COLS);
    if (hipError_t e = launch_kernel(tp_colsum_kernel<FROM_DY, COLS>, dim3(strips, (unsigned)p.splits), dim3(COLS * 4), 0, s, dy, ld_dy,
                                     pre, ld_pre, da, ld, rows, (int)cols, p.splits == 1 ? out : ws, p.per); e != hipSuccess || p.splits == 1)
        return e;
    return launch_kernel(tp_colsum_finish_kernel, dim3((unsigned)((cols + 31) / 32)), dim3(256), 0, s,
                         static_cast<const float*>(ws), p.splits, (int)cols, out);
}
// ws: colsum_ws_bytes(rows, cols) bytes, or null for the single-slab form
hipError_t launch_colsum(const void* da, int64_t ld, int64_t rows, int64_t cols, float* out, float* ws, hipStream_t s) {
    const ColsumPlan p = colsum_plan(rows, cols, ws != nullptr, false);
    uint16_t* const block = static_cast<uint16_t*>(const_cast<void*>(da));
    return p.wide ? colsum_passes<false, 128>(p, nullptr, 0, nullptr, 0, block, ld, rows, cols, out, ws, s)
                  : colsum_passes<false, 64>(p, nullptr, 0, nullptr, 0, block, ld, rows, cols, out, ws, s);
}
// da = dy * GeLU'(pre) and its column sums, in one pass or in two (the elementwise kernel's own grid, then the sums; times
// in us, one pass / two).
//   One pass where no workgroup walks more than 384 rows (300 x 1024 6.9 / 7.3, 2048 x 1024 8.8 / 9.6, 8192 x 1024 15.1 / 17.5;
//   one slab of 424 x 1792 9.9 / 8.7) or where at least 192 strips of 64 columns are at work (4096 x 12288, one slab, 70.5 / 77.4;
//   32896 x 2560 121.6 / 120.9; below: 4096 x 8192, one slab, 64.9 / 59.0; 100000 x 8, 64 slabs, 71 / 18; 2048 x 2560, one slab, 33 / 20).
//   Two passes where the last strip has 8 columns: half a 32-byte sector a row, 5 us by itself (300 x 136 11.5 / 6.8, 300 x 144
//   6.6 / 7.0, 5760 x 8 15.2 / 7.1), or the only one less than 32 (300 x 16 6.3 / 5.5, 61 x 8 4.6 / 3.9); not for a few rows
//   (88 x 2632 4.9 / 6.3, 14 x 8 3.3 / 3.8).
//   Rows that start off cache lines leave each workgroup partial lines to write: two passes too, once the block is so large
//   (7M elements) that traffic counts: 8192 x 656 14.0 / 15.0, 837 x 9752 22.2 / 20, 8192 x 6184 112 / 80, 32896 x 656 49 / 42;
//   with one slab of wide strips from 32M on (941 x 29552 43 / 47, 4096 x 16400 116 / 108, 6717 x 27448 344 / 287).
hipError_t launch_dgelu_colsum(const void* dy, int64_t ld_dy, const void* pre, int64_t ld_pre, void* da, int64_t ld, int64_t rows,
                               int64_t cols, float* out, float* ws, hipStream_t s) {
    const ColsumPlan p = colsum_plan(rows, cols, ws != nullptr, true);
    const bool off_lines = ((ld_dy | ld_pre | ld) & 63) || ((reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(pre) |
                                                             reinterpret_cast<uintptr_t>(da)) & 127);
    const bool ragged = cols < 32 ? rows > 32 : cols % 64 == 8 && rows > 96;
    const bool partial_lines = off_lines && rows * cols > ((int64_t)(p.wide && p.splits == 1 ? 32 : 7) << 20);
    if (!ragged && !partial_lines && (p.per <= 384 || (cols + 63) / 64 * p.splits >= 192)) {
        const uint16_t *g = static_cast<const uint16_t*>(dy), *a = static_cast<const uint16_t*>(pre);
        uint16_t* const block = static_cast<uint16_t*>(da);
        return p.wide ? colsum_passes<true, 128>(p, g, ld_dy, a, ld_pre, block, ld, rows, cols, out, ws, s)
                      : colsum_passes<true, 64>(p, g, ld_dy, a, ld_pre, block, ld, rows, cols, out, ws, s);
    }
    if (hipError_t e = launch_dgelu(dy, ld_dy, pre, ld_pre, da, ld, rows, cols, s); e != hipSuccess) return e;
    return launch_colsum(da, ld, rows, cols, out, ws, s);
}

}  // namespace tpl
