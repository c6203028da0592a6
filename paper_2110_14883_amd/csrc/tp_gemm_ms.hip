// gfx950 (MI355X, CDNA4): the GEMM of libtplinear for products with too few 256 x 256 tiles to fill the chip
// (paper Section 2.2, tensor parallelism: the local block products of the 1D / 2D / 2.5D / 3D schemes and the
// two backward products): macro-tiles of 128 x 128, 128 x 256 and 256 x 128, one C tile per workgroup.
//
//   * four wave64 per workgroup, one per SIMD, 2 x 2 over the C tile; K tiles of 64;
//   * bound: a K tile of 128 x 128 is 512 cycles of MFMA, less than the time a load from memory takes, so what
//     counts is how many K tiles are on their way at once.  All of the CU's LDS is a ring of stages (5 of 32 KB,
//     or 3 of 48 KB), filled by direct-to-LDS loads: while tile u is multiplied, tiles u + 1 .. u + NS - 1 are in
//     flight, and one barrier per K tile hands stages over.  The epilogue's patch reuses the ring;
//   * an operand whose contraction index is not contiguous is transposed on the way out of LDS, by
//     ds_read_b64_tr_b16 (layouts as in the 256 x 256 kernel);
//   * fragments of MFMA step ks + 1 are read under the MFMAs of step ks; the barrier stands before the last step,
//     whose MFMAs cover the first fragment reads of the next tile.
//
// Against the eight-wave kernel with the same tiles and splits (two stages, operands through registers), same run:
//   8192 x 1024 x 1024, 2 steps: forward 53.4 -> 42.0 us (128 x 256), dX 41.5 -> 35.4, dW 73.9 -> 42.4 (128 x 128, split 4);
//   1111 x 2056 x 520, 3 steps: forward 30.7 -> 21.6 us, dX 29.1 -> 25.0 (split 4), dW 31.8 -> 21.9 (split 2);
//   2048 x 8192 x 2048, 4 steps, 128 x 128 tiles: forward 459 -> 299 us, dW 444 -> 273 (256 x 256: 237 and 206).
#include "tp_stream.h"

namespace tpl {

namespace {
constexpr int MS_THREADS = 256;
template <int BM, int BN> struct MsShape {
    static constexpr int A_BYTES = BM * BK * 2, STAGE = (BM + BN) * BK * 2;
    static constexpr int NS = 163840 / STAGE;                 // 5 stages of 32 KB or 3 of 48 KB
    static constexpr int LDS_BYTES = NS * STAGE;
};
}  // namespace

// STREAM: stores carry the streaming hint
template <int BM, int BN, bool A_KC, bool B_KC, int EPI, bool F32_OUT, bool STREAM>
__global__ __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(1, 1)))
void tp_gemm_ms_kernel(const GemmArgs p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    using Sh = MsShape<BM, BN>;
    preload(p);
    constexpr int NS = Sh::NS, STAGE = Sh::STAGE, A_BYTES = Sh::A_BYTES;
    constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 32, TN = WN / 32;      // a wave's share of the C tile
    constexpr int LA = BM / 32, LB = BN / 32;                                // loads per wave and K tile
    const int t = threadIdx.x;
    const int l = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = w & 1, wn = w >> 1;

    const int KT = (p.K + BK - 1) / BK;
    const int Z = p.split_k;
    int tm, tn, z, g = 0;
    tile_of_id(p, (int)blockIdx.x, tm, tn, z);
    if (p.n_groups > 1) {
        if (p.group_along_n) { g = tn / p.group_tiles; tn -= g * p.group_tiles; }
        else                 { g = tm / p.group_tiles; tm -= g * p.group_tiles; }
    }
    const int rot = uni(p.rotate ? ((tm * 3 + tn * 5) & 7) % KT : 0);
    const int m0 = uni(tm * BM), n0 = uni(tn * BN);
    z = uni(z); g = uni(g);

    // ------------------------------------------------------------------ fragment addresses, per lane (bytes)
    // A stage holds operand A, then operand B.  Contraction-contiguous: rows of 128 B, chunk c of row r at
    // c ^ ((r >> 1) & 7) ^ ((r >> 4) & 3); otherwise 64 rows of k with 2 BM (2 BN) bytes, chunk c of row k at
    // c ^ 4 (k % 4).  Block i of 32 rows / columns, step ks: see read_frag.
    const int lr = l & 31, ch = l >> 5;
    constexpr int NRA = A_KC ? 4 : TM, NRB = B_KC ? 4 : TN;
    uint32_t ra[NRA], rb[NRB];
    {
        const int L = ch ^ ((lr >> 1) & 7) ^ (lr >> 4);
        const int r = (l & 15) >> 2, low = 2 * ((l >> 4) & 1) + ((l >> 1) & 1);
#pragma unroll
        for (int vi = 0; vi < NRA; ++vi)
            ra[vi] = A_KC ? (uint32_t)((wm * WM + lr) * 128 + ((L ^ (2 * vi)) << 4))
                          : (uint32_t)((ch * 8 + r) * (2 * BM) + (((wm * (WM / 8) + 4 * vi + low) ^ (4 * r)) << 4) + (l & 1) * 8);
#pragma unroll
        for (int vi = 0; vi < NRB; ++vi)
            rb[vi] = A_BYTES + (B_KC ? (uint32_t)((wn * WN + lr) * 128 + ((L ^ (2 * vi)) << 4))
                                     : (uint32_t)((ch * 8 + r) * (2 * BN) + (((wn * (WN / 8) + 4 * vi + low) ^ (4 * r)) << 4) + (l & 1) * 8));
    }

    // ------------------------------------------------------------------ fetch cursor and loads
    // K tiles z, z + Z, ... of the n_steps x KT sequence.  Per step an operand has one buffer descriptor that
    // starts at the tile's first row (or column) and ends with the operand block; past the last K tile the
    // descriptors are empty and the loads write zeros that nobody multiplies.
    // Load n of wave w fills bytes 4096 n + 1024 w .. + 1023 of the operand's part of the stage:
    //   contraction-contiguous: rows 32 n + 8 w + l / 8, position l % 8 (the chunk differs between even and odd
    //     n by chunk ^ 2);  otherwise: k row (4096 n + 1024 w) / pitch + 16 l / pitch, position l % (pitch / 16).
    const int total_k = Z == 1 ? p.n_steps * KT : (p.n_steps * KT - z + Z - 1) / Z;     // K tiles of this workgroup (split_k <= their number: >= 1)
    int f_left = uni(total_k), f_step, f_kt;
    f_kt = uni(z); f_step = uni(g);
    while (f_kt >= KT) { f_kt -= KT; ++f_step; }               // (z < 8)
    u32x4_t rw_a, rw_b;
    uint32_t dl_a[2], dl_b[2], dv_a[2], dv_b[2];
    int a_step, b_step, a_kmul, b_kmul;
    const int d_rl = w * 8 + (l >> 3);
    const int d_c0 = (l & 7) ^ ((d_rl >> 1) & 7) ^ (d_rl >> 4);
    const uint32_t s_wbase = (uint32_t)(w * 1024);
    auto open_operand = [&](auto is_a) __attribute__((always_inline)) {
        constexpr bool IS_A = decltype(is_a)::value;
        constexpr bool KC = IS_A ? A_KC : B_KC;
        constexpr int R = IS_A ? BM : BN, CH = R / 8, ROWS = 2048 / R;        // chunks of a k row; k rows of one load (all waves)
        const int s = f_step < TP_MAX_STEPS ? f_step : TP_MAX_STEPS - 1;
        const uint16_t* ptr = uni_ptr(IS_A ? p.a[s] : p.b[s]);
        const int ld = uni(IS_A ? p.lda[s] : p.ldb[s]);
        const int X = IS_A ? p.M : p.N, x0 = IS_A ? m0 : n0;
        const int xs = (X - x0) < R ? (X - x0) : R;
        const int64_t nrec = f_left > 0 ? (KC ? (int64_t)(xs - 1) * ld + p.K : (int64_t)(p.K - 1) * ld + xs) * 2 : 0;
        const uint64_t base = reinterpret_cast<uint64_t>(KC ? ptr + (int64_t)x0 * ld : ptr + x0);
        const u32x4_t rw = {(uint32_t)uni((int)(uint32_t)base), (uint32_t)uni((int)((uint32_t)(base >> 32) & 0xffffu)),
                            (uint32_t)uni((int)(uint32_t)nrec), 0x00020000u};
        const int step = uni(KC ? 64 * ld : 2 * ROWS * ld), kmul = uni(KC ? 2 : 2 * ld);
        if constexpr (IS_A) { rw_a = rw; a_step = step; a_kmul = kmul; }
        else                { rw_b = rw; b_step = step; b_kmul = kmul; }
        const int x_k = w * (ROWS / 4) + l / CH, x_x = ((l % CH) ^ ((x_k & 3) << 2)) * 8;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t off = KC ? (uint32_t)((d_rl * ld + (d_c0 ^ (2 * h)) * 8) * 2)
                                    : (x_x < xs ? (uint32_t)((x_k * ld + x_x) * 2) : OOB_OFFSET);
            if constexpr (IS_A) dl_a[h] = off; else dl_b[h] = off;
        }
    };
    auto prep_tile = [&]() __attribute__((always_inline)) {
        int kt = f_kt + rot;
        if (kt >= KT) kt -= KT;
        const int k0 = kt * BK;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool kok = (k0 + (d_c0 ^ (2 * h)) * 8) < p.K;
            dv_a[h] = !A_KC || kok ? dl_a[h] + (uint32_t)(k0 * a_kmul) : OOB_OFFSET;
            dv_b[h] = !B_KC || kok ? dl_b[h] + (uint32_t)(k0 * b_kmul) : OOB_OFFSET;
        }
    };
    auto advance = [&]() __attribute__((always_inline)) {
        if (f_left > 0) {
            --f_left;
            f_kt += Z;
            if (f_left == 0 || f_kt >= KT) {
                if (f_left > 0) do { f_kt -= KT; ++f_step; } while (f_kt >= KT);
                else f_kt = 0;
                open_operand(std::true_type{});
                open_operand(std::false_type{});
            }
        }
        prep_tile();
    };
    auto load1 = [&](auto is_a, auto n_, uint32_t stage_off) __attribute__((always_inline)) {
        constexpr bool IS_A = decltype(is_a)::value;
        constexpr int n = decltype(n_)::value;
        if constexpr (IS_A) dtl_load16(rw_a, dv_a[n & 1] + (uint32_t)(n * a_step), s_wbase + stage_off + n * 4096);
        else                dtl_load16(rw_b, dv_b[n & 1] + (uint32_t)(n * b_step), s_wbase + stage_off + A_BYTES + n * 4096);
    };

    // ------------------------------------------------------------------ fragments and accumulators
    bf16x8_t fa[2][TM], fb[2][TN];
    f32x16_t acc[TM][TN];
    constexpr int RA = A_KC ? 1 : 2, RB = B_KC ? 1 : 2, NR = TM * RA + TN * RB;
    auto read_frag = [&](auto is_a, auto ks_, auto i_, auto h_) __attribute__((always_inline)) {
        constexpr bool IS_A = decltype(is_a)::value;
        constexpr int ks = decltype(ks_)::value & 3, i = decltype(i_)::value, h = decltype(h_)::value;
        constexpr int PITCH = IS_A ? 2 * BM : 2 * BN;
        auto& set = [&]() -> auto& { if constexpr (IS_A) return fa[ks & 1]; else return fb[ks & 1]; }();
        bf16x8_t& f = set[i];
        uint32_t addr;
        if constexpr (IS_A ? A_KC : B_KC) {
            if constexpr (IS_A) addr = ra[ks ^ (i & 1)]; else addr = rb[ks ^ (i & 1)];
            f = lds_load_frag(addr + i * 4096);
        } else {
            if constexpr (IS_A) addr = ra[i]; else addr = rb[i];
            const bf16x4_t v = lds_load_tr(addr + (ks * 16 + h * 4) * PITCH);
            if constexpr (h == 0) f = __builtin_shufflevector(v, v, 0, 1, 2, 3, 0, 1, 2, 3);
            else                  f = __builtin_shufflevector(f, __builtin_shufflevector(v, v, 0, 1, 2, 3, 0, 1, 2, 3), 0, 1, 2, 3, 8, 9, 10, 11);
        }
    };
    // reads of a step in the order its MFMAs need them: B0, A0, the other B, the other A
    auto read_n = [&](auto n_, auto ks_) __attribute__((always_inline)) {
        constexpr int n = decltype(n_)::value;
        constexpr int e1 = RB, e2 = RB + RA, e3 = RA + TN * RB;
        using AT = std::true_type;
        using BT = std::false_type;
        if constexpr (n < e1)      read_frag(BT{}, ks_, std::integral_constant<int, 0>{}, std::integral_constant<int, n>{});
        else if constexpr (n < e2) read_frag(AT{}, ks_, std::integral_constant<int, 0>{}, std::integral_constant<int, n - e1>{});
        else if constexpr (n < e3) read_frag(BT{}, ks_, std::integral_constant<int, 1 + (n - e2) / RB>{}, std::integral_constant<int, (n - e2) % RB>{});
        else                       read_frag(AT{}, ks_, std::integral_constant<int, 1 + (n - e3) / RA>{}, std::integral_constant<int, (n - e3) % RA>{});
    };
    // (not __syncthreads(): its fence could wait for the loads in flight)
    auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // (the bias is on its way while the K loop runs and is added once, before the epilogue)
    constexpr bool USE_BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_GELU;
    BiasBlock<TN> bias;
    if constexpr (USE_BIAS) load_bias(bias, p, n0 + wn * WN);

    // ------------------------------------------------------------------ prologue: tiles 0 .. NS - 2, and A of tile NS - 1
    open_operand(std::true_type{});
    open_operand(std::false_type{});
    prep_tile();
    static_for<NS - 1>([&](auto s_) __attribute__((always_inline)) {
        static_for<LA>([&](auto n_) __attribute__((always_inline)) { load1(std::true_type{}, n_, decltype(s_)::value * STAGE); });
        static_for<LB>([&](auto n_) __attribute__((always_inline)) { load1(std::false_type{}, n_, decltype(s_)::value * STAGE); });
        advance();
    });
    static_for<LA>([&](auto n_) __attribute__((always_inline)) { load1(std::true_type{}, n_, (NS - 1) * STAGE); });
    wait_vm<(NS - 2) * (LA + LB) + LA>();
    barrier();
    static_for<NR>([&](auto n_) __attribute__((always_inline)) { read_n(n_, std::integral_constant<int, 0>{}); });

    // ------------------------------------------------------------------ one K tile: 4 steps of TM x TN MFMAs
    // Operand B of tile u + NS - 1 is fetched during steps 0 and 1 (its stage, that of tile u - 1, was given up at
    // the barrier of body u - 1) and, after the barrier before step 3, operand A of tile u + NS into the stage of
    // tile u, whose last fragments everybody has by then.  That barrier also says that tile u + 1 has landed.
    constexpr int Q = TM * TN;
    uint32_t so = 0, so_b = (NS - 1) * STAGE;                 // stage of tile u; stage of tile u + NS - 1
    for (int u = 0; u < total_k; ++u) {
        const uint32_t so_n = so + STAGE == NS * STAGE ? 0u : so + STAGE;
        static_for<4 * Q>([&](auto s_) __attribute__((always_inline)) {
            constexpr int s = decltype(s_)::value;
            constexpr int ks = s / Q, q = s % Q, i = q / TN, j = q % TN;
            if constexpr (s == 3 * Q) {
                wait_vm<(NS - 2) * (LA + LB)>();
                barrier();
                const uint32_t d = so_n - so;
#pragma unroll
                for (int vi = 0; vi < NRA; ++vi) ra[vi] += d;
#pragma unroll
                for (int vi = 0; vi < NRB; ++vi) rb[vi] += d;
            }
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks & 1][j], fa[ks & 1][i], acc[i][j], 0, 0, 0);
            static_for<((q + 1) * NR) / Q - (q * NR) / Q>([&](auto n_) __attribute__((always_inline)) {
                read_n(std::integral_constant<int, (q * NR) / Q + decltype(n_)::value>{}, std::integral_constant<int, ks + 1>{});
            });
            if constexpr (s < 2 * Q)
                static_for<((s + 1) * LB) / (2 * Q) - (s * LB) / (2 * Q)>([&](auto n_) __attribute__((always_inline)) {
                    load1(std::false_type{}, std::integral_constant<int, (s * LB) / (2 * Q) + decltype(n_)::value>{}, so_b);
                });
            if constexpr (s == 2 * Q) advance();
            if constexpr (ks == 3)
                static_for<((q + 1) * LA) / Q - (q * LA) / Q>([&](auto n_) __attribute__((always_inline)) {
                    load1(std::true_type{}, std::integral_constant<int, (q * LA) / Q + decltype(n_)::value>{}, so);
                });
            __builtin_amdgcn_sched_barrier(0);
        });
        so_b = so;
        so = so_n;
    }
    // every load has landed and every fragment is in registers before the patch reuses the ring
    wait_vm<0>();
    barrier();
    if constexpr (USE_BIAS) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float b = bias_of(bias, j, e);
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[i][j][e] += b;
            }
    }
    store_c_block<TM, TN, EPI, F32_OUT, false, false, STREAM>(p, acc, m0 + wm * WM, n0 + wn * WN, z, g, bias, lds + w * 8192, p.pre != nullptr, [] {});
}

// ---------------------------------------------------------------------------------------------
// host launcher
// ---------------------------------------------------------------------------------------------
template <int BM, int BN, bool A_KC, bool B_KC, int EPI, bool F32_OUT, bool STREAM>
static hipError_t launch_ms_as(const GemmArgs& a, hipStream_t stream) {
    static std::atomic<uint64_t> attr_done{0};
    constexpr int lds_bytes = MsShape<BM, BN>::LDS_BYTES;
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_done.load(std::memory_order_relaxed) & bit)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tp_gemm_ms_kernel<BM, BN, A_KC, B_KC, EPI, F32_OUT, STREAM>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        attr_done.fetch_or(bit, std::memory_order_relaxed);
    }
    const unsigned grid = (unsigned)(a.tiles_m * a.tiles_n * a.split_k);
    return launch_kernel(tp_gemm_ms_kernel<BM, BN, A_KC, B_KC, EPI, F32_OUT, STREAM>, dim3(grid), dim3(MS_THREADS), lds_bytes, stream, a);
}

template <int BM, int BN, bool A_KC, bool B_KC, int EPI, bool F32_OUT>
static hipError_t launch_ms_one(const GemmArgs& a, hipStream_t s) {
    return a.stream ? launch_ms_as<BM, BN, A_KC, B_KC, EPI, F32_OUT, true>(a, s) : launch_ms_as<BM, BN, A_KC, B_KC, EPI, F32_OUT, false>(a, s);
}

template <int BM, int BN>
static hipError_t launch_ms_tile(int form, const GemmArgs& a, hipStream_t s) {
    const int epi = a.split_k > 1 ? EPI_NONE : (a.dg ? EPI_MUL_DGELU : (a.gelu ? EPI_BIAS_GELU : (a.bias ? EPI_BIAS : EPI_NONE)));
    const bool f32 = a.split_k > 1 || a.out_f32;
    switch (form) {
        case FORM_NN:
            if (epi == EPI_BIAS_GELU) return f32 ? launch_ms_one<BM, BN, true, false, EPI_BIAS_GELU, true>(a, s) : launch_ms_one<BM, BN, true, false, EPI_BIAS_GELU, false>(a, s);
            if (epi == EPI_BIAS)      return f32 ? launch_ms_one<BM, BN, true, false, EPI_BIAS, true>(a, s) : launch_ms_one<BM, BN, true, false, EPI_BIAS, false>(a, s);
            if (epi == EPI_NONE)      return f32 ? launch_ms_one<BM, BN, true, false, EPI_NONE, true>(a, s) : launch_ms_one<BM, BN, true, false, EPI_NONE, false>(a, s);
            return hipErrorInvalidValue;
        case FORM_NT:
            if (epi == EPI_MUL_DGELU) return f32 ? launch_ms_one<BM, BN, true, true, EPI_MUL_DGELU, true>(a, s) : launch_ms_one<BM, BN, true, true, EPI_MUL_DGELU, false>(a, s);
            if (epi == EPI_NONE)      return f32 ? launch_ms_one<BM, BN, true, true, EPI_NONE, true>(a, s) : launch_ms_one<BM, BN, true, true, EPI_NONE, false>(a, s);
            return hipErrorInvalidValue;
        case FORM_TN:
            if (epi == EPI_NONE && f32) return launch_ms_one<BM, BN, false, false, EPI_NONE, true>(a, s);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm_ms(int form, int tile_id, const GemmArgs& a, hipStream_t s) {
    switch (tile_id) {
        case TILE_128x256_MS: return launch_ms_tile<128, 256>(form, a, s);
        case TILE_256x128_MS: return launch_ms_tile<256, 128>(form, a, s);
        case TILE_128x128_MS: return launch_ms_tile<128, 128>(form, a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tpl
