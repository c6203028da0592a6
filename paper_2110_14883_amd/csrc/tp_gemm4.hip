// gfx950 (MI355X, CDNA4): the 256 x 256 macro-tile GEMM of libtplinear as ONE software pipeline per
// workgroup (paper Section 2.2, tensor parallelism: the local block products C = sum_k A_k B_k of
// the 1D / 2D / 2.5D / 3D schemes and the two backward products).
//
//   * four wave64 per workgroup, one per SIMD, each owning a 128 x 128 block of the C tile: 16 MFMA
//     32x32x16 accumulators = 256 registers in the accumulator half of the register file, and only
//     32 LDS fragment reads per 64 MFMAs (the eight-wave kernel reads 48);
//   * the K tiles of ALL the C tiles a persistent workgroup owns form one stream: while K tile u is being
//     multiplied, tiles u+1 and u+2 travel into the other LDS stages (three of operand A, two of B: all of the
//     CU's LDS), across C-tile boundaries too, so the epilogue of a C tile runs with the next one's first K tiles in LDS or on
//     their way; its patch is the one stage that is free just then;
//   * both operands of every memory form go from memory straight into LDS.  An operand whose contraction
//     index is not contiguous is transposed on the way OUT, by ds_read_b64_tr_b16.  (It used to be
//     transposed in registers on the way in, 8 loads, 32 byte permutes and 8 LDS writes per wave and K
//     tile; on 16384 x 4096 x 4096 that form took 1.53 us (NN) and 1.62 us (TN) per K tile and round
//     against 1.42 us of NT; all three forms now take the time of NT: 418 -> 405 us NN, 449 -> 430 us TN,
//     on a box where NT itself was 4 % slower.)
//   * every load and fragment read has a fixed slot between two MFMAs of the 64-MFMA K tile (scheduling
//     fences pin the order); the one workgroup barrier per K tile sits after MFMA 48, and the last 16
//     MFMAs cover the first fragment reads of the next K tile, so no LDS latency is exposed at the tile
//     boundary;
//   * tile order and epilogue (bias / GeLU / GeLU' in registers, then through a wave-private LDS patch so
//     that stores are whole 128-byte row segments) are those of the eight-wave kernel.
#include "tp_stream.h"

namespace tpl {

namespace {

constexpr int W4_THREADS = 256;
constexpr int W4_BM = 256, W4_BN = 256;
constexpr int W4_STAGE = W4_BM * BK * 2;                     // 32 KB: one stage of one operand
constexpr int W4_A_BASE = 2 * W4_STAGE;                      // LDS: two stages of operand B | three of operand A
constexpr int W4_LDS_BYTES = 5 * W4_STAGE;                   // all 160 KB
constexpr int W4_EPI_BYTES_PER_WAVE = 8192;                  // 32 rows x 256 bytes, in the stage that is free between two C tiles

}  // namespace

// PRE: the pre-activation is stored too; STREAM: stores carry the streaming hint.  (Compiled in: with both ways through the epilogue in one
// kernel, the one without the pre-activation took 143 us for 16384 x 1024, K = 4096 with GeLU, alone 134.5; and a branch around the
// stores cost the one with it 2 %, 32896 x 2560, K = 2 x 640 230.5 -> 235.4.)
template <bool A_KC, bool B_KC, int EPI, bool F32_OUT, bool PRE, bool STREAM>
__global__ __launch_bounds__(W4_THREADS) __attribute__((amdgpu_waves_per_eu(1, 1)))
void tp_gemm4_kernel(const GemmArgs p) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr int TM = 4, TN = 4;                  // 32 x 32 MFMA tiles per wave along M and N
    preload(p);
    const int t = threadIdx.x;
    const int l = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = w & 1, wn = w >> 1;

    const int KT = (p.K + BK - 1) / BK;
    const int T = p.n_steps * KT;
    const int Z = p.split_k;
    const int total = p.tiles_m * p.tiles_n * Z;
    const int grid = (int)gridDim.x;

    // ------------------------------------------------------------------ LDS addresses (bytes), per lane
    // LDS map: two stages of operand B, three of A, 32 KB each.  A K tile's addresses are those of the last one plus the
    // distance to the next stage: four registers an operand.
    // Fragment of 32 rows (columns of C) x 16 k for MFMA step ks, block i.
    // Contraction-contiguous operand (rows of 128 B, chunks swizzled as in lds_off()): lane reads row
    // lr + 32 i of the wave's 128-row slab, chunk 2 ks + lane/32, with one ds_read_b128.  The chunk
    // position is L ^ 2 (ks ^ (i & 1)) with L a lane constant: four address registers cover every (ks, i);
    // 32 i rows = an immediate offset of 4096 i bytes.
    // Otherwise (64 rows of k, 512 B each, 32 chunks of 8 x): ds_read_b64_tr_b16 transposes on the way
    // out.  16 lanes take 4 rows of k x 16 x (lane i: row r = i / 4, its 4 x at 4 (i % 4)) and receive 4
    // consecutive k of one x each; two of them make a fragment.  With rows at a pitch of 512 B the four
    // rows would share 16 banks (measured: 8 cycles per wave instruction, 64 B/clk); with chunk c of row k
    // kept at position c ^ 4 (k % 4) a half-wave covers all 64 banks (3.06 cycles, 167 B/clk; a linear
    // b64 read takes the same, ds_read_b128 4.0).  The XOR turns block i into i ^ r: four address
    // registers again, ks and the second half of the k in the immediate.
    const int lr = l & 31, ch = l >> 5;
    uint32_t ra_addr[4], rb_addr[4];
    {
        const int L = ch ^ ((lr >> 1) & 7) ^ (lr >> 4);
        const int r = (l & 15) >> 2, low = 2 * ((l >> 4) & 1) + ((l >> 1) & 1);
#pragma unroll
        for (int vi = 0; vi < 4; ++vi) {
            ra_addr[vi] = W4_A_BASE + (A_KC ? (uint32_t)((wm * 128 + lr) * 128 + ((L ^ (2 * vi)) << 4))
                                                         : (uint32_t)((ch * 8 + r) * 512 + (wm * 16 + 4 * (vi ^ r) + low) * 16 + (l & 1) * 8));
            rb_addr[vi] = (B_KC ? (uint32_t)((wn * 128 + lr) * 128 + ((L ^ (2 * vi)) << 4))
                                               : (uint32_t)((ch * 8 + r) * 512 + (wn * 16 + 4 * (vi ^ r) + low) * 16 + (l & 1) * 8));
            // (opaque, so that the constant part of every address goes into the instruction's offset field)
            asm volatile("" : "+v"(ra_addr[vi]), "+v"(rb_addr[vi]));
        }
    }
    // ------------------------------------------------------------------ cursors over the K-tile stream
    // left: K tiles of the cursor's C tile still to come (the current one included); 0 = past the end of the stream
    struct Cursor { int v, m0, n0, z, rot, g, step, kt, left; };
    auto start = [&](Cursor& c, int v) __attribute__((always_inline)) {
        c.v = v;
        c.left = 0;
        if (v >= total) return;
        int tm, tn, z;
        tile_of_id(p, v, tm, tn, z);
        c.rot = uni(p.rotate ? ((tm * 3 + tn * 5) & 7) % KT : 0);
        int g = 0;
        if (p.n_groups > 1) {
            if (p.group_along_n) { g = tn / p.group_tiles; tn -= g * p.group_tiles; }
            else                 { g = tm / p.group_tiles; tm -= g * p.group_tiles; }
        }
        c.m0 = uni(tm * W4_BM); c.n0 = uni(tn * W4_BN); c.z = uni(z); c.g = uni(g);
        c.kt = uni(z);
        c.step = uni(g);                          // a grouped launch has one step per group: operand slot = group
        while (c.kt >= KT) { c.kt -= KT; ++c.step; }      // (z < 8)
        c.left = uni(Z == 1 ? T : (T - z + Z - 1) / Z);        // K tiles z, z + Z, ... of the n_steps x KT sequence
    };
    Cursor f, c;                                  // fetch cursor (two K tiles ahead) and compute cursor

    // ------------------------------------------------------------------ loads
    // Per (C tile, step) an operand has one buffer descriptor that starts at the tile's first row (or
    // column) and ends with the operand block, so rows past a ragged edge read as zero; per K tile only
    // the lane offsets move.  (The host sends a product here only if those offsets fit 31 bits.)
    // Load n of wave w fills bytes 4096 n + 1024 w .. + 1023 of the operand's stage.
    //   contraction-contiguous: rows 32 n + 8 w .. + 7; lane l holds position l % 8 of row 8 w + l / 8,
    //     i.e. the chunk the swizzle puts there, which differs between even and odd n by chunk ^ 2;
    //   otherwise: k rows 8 n + 2 w and + 1; lane l holds position l % 32 of row 2 w + l / 32.
    // dl: lane offsets at k = 0 (of even and odd n);  dv: the same for the fetch cursor's K tile.
    u32x4_t rw_a, rw_b;
    uint32_t dl_a[2], dl_b[2], dv_a[2], dv_b[2];
    int a_step, b_step, a_kmul, b_kmul;            // bytes between a lane's loads; bytes per unit of k
    const int d_rl = w * 8 + (l >> 3);
    const int d_c0 = (l & 7) ^ ((d_rl >> 1) & 7) ^ (d_rl >> 4);
    const int x_k = 2 * w + ch, x_x = ((l & 31) ^ ((x_k & 3) << 2)) * 8;
    const uint32_t s_wbase = (uint32_t)(w * 1024);
    auto open_operand = [&](auto is_a) __attribute__((always_inline)) {
        constexpr bool IS_A = decltype(is_a)::value;
        constexpr bool KC = IS_A ? A_KC : B_KC;
        const bool ok = f.left != 0;
        const int s = f.step < TP_MAX_STEPS ? f.step : TP_MAX_STEPS - 1;
        const uint16_t* ptr = uni_ptr(IS_A ? p.a[s] : p.b[s]);
        const int ld = uni(IS_A ? p.lda[s] : p.ldb[s]);
        const int X = IS_A ? p.M : p.N, x0 = IS_A ? f.m0 : f.n0;
        const int xs = (X - x0) < 256 ? (X - x0) : 256;       // rows (columns) of this tile that exist
        const int64_t nrec = ok ? (KC ? (int64_t)(xs - 1) * ld + p.K : (int64_t)(p.K - 1) * ld + xs) * 2 : 0;
        const uint64_t base = reinterpret_cast<uint64_t>(KC ? ptr + (int64_t)x0 * ld : ptr + x0);
        const u32x4_t rw = {(uint32_t)uni((int)(uint32_t)base), (uint32_t)uni((int)((uint32_t)(base >> 32) & 0xffffu)),
                            (uint32_t)uni((int)(uint32_t)nrec), 0x00020000u};
        const int step = uni(KC ? 64 * ld : 16 * ld), kmul = uni(KC ? 2 : 2 * ld);
        if constexpr (IS_A) { rw_a = rw; a_step = step; a_kmul = kmul; }
        else                { rw_b = rw; b_step = step; b_kmul = kmul; }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t off = KC ? (uint32_t)((d_rl * ld + (d_c0 ^ (2 * h)) * 8) * 2)
                                    : (x_x < xs ? (uint32_t)((x_k * ld + x_x) * 2) : OOB_OFFSET);
            if constexpr (IS_A) dl_a[h] = off; else dl_b[h] = off;
        }
    };
    // lane offsets of the fetch cursor's K tile, in three parts.  (k beyond K: a contraction-contiguous chunk is masked
    // here; a row of the other kind lies past the end of its descriptor.)
    int t_k0 = 0;
    auto prep_k0 = [&]() __attribute__((always_inline)) {
        int kt = f.kt + f.rot;
        if (kt >= KT) kt -= KT;
        t_k0 = kt * BK;
    };
    auto prep_operand = [&](auto is_a) __attribute__((always_inline)) {
        constexpr bool IS_A = decltype(is_a)::value;
        constexpr bool KC = IS_A ? A_KC : B_KC;
        const uint32_t at = (uint32_t)(t_k0 * (IS_A ? a_kmul : b_kmul));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool kok = !KC || (t_k0 + (d_c0 ^ (2 * h)) * 8) < p.K;
            if constexpr (IS_A) dv_a[h] = kok ? dl_a[h] + at : OOB_OFFSET;
            else                dv_b[h] = kok ? dl_b[h] + at : OOB_OFFSET;
        }
    };
    auto prep_tile = [&]() __attribute__((always_inline)) {
        prep_k0();
        prep_operand(std::true_type{});
        prep_operand(std::false_type{});
    };
    // Move the fetch cursor to the next K tile of the stream.  The common case (same C tile, same step)
    // is a few scalar instructions issued between two MFMAs; a change of step or of C tile needs other
    // blocks and other descriptors (advance_slow()).
    int f_live = 0, f_reopen = 0;
    auto advance_count = [&]() __attribute__((always_inline)) {
        f_live = f.left != 0 ? 1 : 0;             // past the end nothing moves: every further tile reads as zero
        f.left -= f_live;
    };
    auto advance_k = [&]() __attribute__((always_inline)) { f.kt += f_live ? Z : 0; };
    auto advance_check = [&]() __attribute__((always_inline)) { f_reopen = f_live != 0 && (f.left == 0 || f.kt >= KT); };
    auto advance_slow = [&]() __attribute__((always_inline)) {
        if (f.left != 0) {                        // next step of this C tile
            do { f.kt -= KT; ++f.step; } while (f.kt >= KT);
        } else {
            start(f, f.v + grid);                 // next C tile (or the end)
        }
        open_operand(std::true_type{});
        open_operand(std::false_type{});
    };
    // n-th direct-to-LDS load of an operand, into the stage that starts at byte `stage` of the LDS (plus this wave's share)
    auto dtl1 = [&](auto is_a, auto n_, uint32_t stage) __attribute__((always_inline)) {
        constexpr bool IS_A = decltype(is_a)::value;
        constexpr int n = decltype(n_)::value;
        if constexpr (IS_A) dtl_load16_at<n * 4096>(rw_a, dv_a[n & 1] + (uint32_t)(n * a_step), stage);
        else                dtl_load16_at<n * 4096>(rw_b, dv_b[n & 1] + (uint32_t)(n * b_step), stage);
    };

    // ------------------------------------------------------------------ fragments and accumulators
    bf16x8_t fa[2][TM], fb[2][TN];
    f32x16_t acc[TM][TN];
    // read n (0 .. NR - 1) of MFMA step ks, in the order the step's MFMAs need the fragments:
    // B0, A0, B1, B2, B3, A1, A2, A3 (a transposed fragment takes two reads)
    constexpr int RA = A_KC ? 1 : 2, RB = B_KC ? 1 : 2, NR = 4 * (RA + RB);
    auto read_frag = [&](auto is_a, auto ks_, auto i_, auto h_) __attribute__((always_inline)) {
        constexpr bool IS_A = decltype(is_a)::value;
        constexpr int ks = decltype(ks_)::value & 3, i = decltype(i_)::value, h = decltype(h_)::value;
        bf16x8_t& f = IS_A ? fa[ks & 1][i] : fb[ks & 1][i];
        if constexpr (IS_A ? A_KC : B_KC) {
            f = lds_load_frag((IS_A ? ra_addr : rb_addr)[ks ^ (i & 1)] + i * 4096);
        } else {
            const bf16x4_t v = lds_load_tr((IS_A ? ra_addr : rb_addr)[i] + (ks * 8192 + h * 2048));
            if constexpr (h == 0) f = __builtin_shufflevector(v, v, 0, 1, 2, 3, 0, 1, 2, 3);
            else                  f = __builtin_shufflevector(f, __builtin_shufflevector(v, v, 0, 1, 2, 3, 0, 1, 2, 3), 0, 1, 2, 3, 8, 9, 10, 11);
        }
    };
    auto read_n = [&](auto n_, auto ks_) __attribute__((always_inline)) {
        constexpr int n = decltype(n_)::value;
        constexpr int e1 = RB, e2 = RB + RA, e3 = RA + 4 * RB;         // ends of B0, A0, B1 .. B3
        using AT = std::true_type;
        using BT = std::false_type;
        if constexpr (n < e1)      read_frag(BT{}, ks_, std::integral_constant<int, 0>{}, std::integral_constant<int, n>{});
        else if constexpr (n < e2) read_frag(AT{}, ks_, std::integral_constant<int, 0>{}, std::integral_constant<int, n - e1>{});
        else if constexpr (n < e3) read_frag(BT{}, ks_, std::integral_constant<int, 1 + (n - e2) / RB>{}, std::integral_constant<int, (n - e2) % RB>{});
        else                       read_frag(AT{}, ks_, std::integral_constant<int, 1 + (n - e3) / RA>{}, std::integral_constant<int, (n - e3) % RA>{});
    };
    // The bias is added to the finished sums, in the epilogue: a sum that starts from it is rounded at its size with every 16 k (bias 8 to
    // 15.5, products of 1e-5, K = 4096: off by 3.3e-5, now by 4.8e-7, the one rounding).  A lane keeps one word of it through the K loop.  The word of the next C tile
    // is asked for before the epilogue of this one and named behind its last stores, so that the wait for it lies there, with those
    // stores still under way: at its use the loads of the next K tiles, which the compiler does not see, would be waited for too.
    constexpr bool USE_BIAS = EPI == EPI_BIAS || EPI == EPI_BIAS_GELU;
    uint32_t own_bias = 0, next_bias = 0;
    auto take_bias = [&]() __attribute__((always_inline)) {
        if constexpr (USE_BIAS) {
            asm volatile("" : "+v"(next_bias));
            own_bias = next_bias;
        }
    };
    auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    };

    // ------------------------------------------------------------------ one K tile: 64 MFMA slots
    // Multiplies K tile u and keeps the loads going.  Slot s = 16 ks + 4 i + j issues MFMA (ks, i, j), then at most one
    // fragment read and at most one load.
    //   reads: those of MFMA step ks + 1 during step ks (every other slot when there are 8, every slot but
    //     every fourth when 12, every slot when 16); those of step 0 of the NEXT K tile during step 3,
    //     from the next stages, after the barrier before slot 48;
    //   loads: those of K tile u + 2.  A has three stages: its loads come from slot 9 on, every fourth slot, into the stage of
    //     tile u - 1, free since the last barrier; they have 75 - 103 slots to land.  B has two: its loads come after the barrier, every other
    //     slot, into the stage that tile u has just been read from, and have 49 - 63.  (All four waves run the same schedule, so a slot
    //     with a load asks the CU's one address path for 4 KB, two slots at 64 B/clk; four where rows are off cache lines.)
    //   With two stages of each and the epilogue's patches beside them one operand had 17 - 47 slots, less than a load from beyond the
    //   L2 takes.  From memory, in us, before and now: dX 2048 x 2048, K = 4 x 8192 255 -> 224; 4096 x 6144, K = 24576 1026 -> 946;
    //   32896 x 640 243 -> 225; dW 640 x 2560, K = 2 x 32896 222 -> 208; rows off cache lines: 6144 x 768, K = 4 x 5256 227 -> 199,
    //   dW 3680 x 5128, K = 3 x 5904 715 -> 635, dX 19633 x 3424, K = 4880 626 -> 585; aligned products that were short of nothing
    //   (forward 16384 x 4096, K = 4096; dW 6144 x 24576, K = 4096) within 1 %.  Which operand is the deep one, and loads every second to fifth
    //   slot, make less than 1 %.
    using OpA = std::true_type;
    using OpB = std::false_type;
    // at_a, at_b: stages of tile u (from slot 44 / 46 on: u + 1), in bytes from the operand's first one; fill_a, fill_b: this
    // wave's share of those to refill; to_next_a: from the stage of tile u to that of u + 1
    uint32_t at_a = 0, at_b = 0, fill_a = s_wbase + W4_A_BASE + 2 * W4_STAGE, fill_b = 0, to_next_a = 0;
    auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto k_tile = [&]() __attribute__((always_inline)) {
        static_for<64>([&](auto s_) __attribute__((always_inline)) {
            constexpr int s = decltype(s_)::value;
            constexpr int ks = s >> 4, q = s & 15, i = (s >> 2) & 3, j = s & 3;
            if constexpr (s == 48) {
                // this wave's loads of tile u + 1 have landed (A's of tile u + 2 may be under way); after the
                // barrier everybody's have, and nobody reads tile u any more (the step-3 fragments were requested
                // during step 2 and have arrived: the barrier waits for them)
                wait_vm<8>();
                barrier();
#pragma unroll
                for (int vi = 0; vi < 4; ++vi) {
                    ra_addr[vi] += to_next_a;
                    rb_addr[vi] ^= W4_STAGE;
                }
            }
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ks & 1][j], fa[ks & 1][i], acc[i][j], 0, 0, 0);
            using KN = std::integral_constant<int, ks + 1>;
            if constexpr (NR == 8)       { if constexpr (q % 2 == 0) read_n(std::integral_constant<int, q / 2>{}, KN{}); }
            else if constexpr (NR == 12) { if constexpr (q % 4 != 3) read_n(std::integral_constant<int, q - q / 4>{}, KN{}); }
            else                         read_n(std::integral_constant<int, q>{}, KN{});
            // (about seven instructions pass under an MFMA: the cursor's are spread)
            if constexpr (s == 0) advance_count();
            if constexpr (s == 1) advance_k();
            if constexpr (s == 2) advance_check();
            if constexpr (s == 3) { if (f_reopen) advance_slow(); }
            if constexpr (s == 4) prep_k0();
            if constexpr (s == 6) prep_operand(OpA{});
            if constexpr (s == 8) prep_operand(OpB{});
            if constexpr (s >= 9 && s < 41 && s % 4 == 1) dtl1(OpA{}, std::integral_constant<int, (s - 9) / 4>{}, fill_a);
            if constexpr (s == 42) to_next_a = at_a == 2 * W4_STAGE ? 0u - 2 * W4_STAGE : (uint32_t)W4_STAGE;
            if constexpr (s == 44) { fill_a = s_wbase + W4_A_BASE + at_a; at_a += to_next_a; }
            if constexpr (s == 46) { fill_b = s_wbase + at_b; at_b ^= W4_STAGE; }
            if constexpr ((s & 1) == 1 && s > 48) dtl1(OpB{}, std::integral_constant<int, (s - 49) / 2>{}, fill_b);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // ------------------------------------------------------------------ the stream
    start(f, (int)blockIdx.x);
    if (f.left == 0) return;
    c = f;
    open_operand(std::true_type{});
    open_operand(std::false_type{});
    prep_tile();
    if constexpr (USE_BIAS) next_bias = bias_word(p, c.n0 + wn * 128);
    // K tiles 0 and 1
    auto load_both = [&](uint32_t a, uint32_t b) __attribute__((always_inline)) {
        static_for<8>([&](auto n_) __attribute__((always_inline)) { dtl1(OpA{}, n_, s_wbase + W4_A_BASE + a); });
        static_for<8>([&](auto n_) __attribute__((always_inline)) { dtl1(OpB{}, n_, s_wbase + b); });
    };
    load_both(0, 0);
    advance_count();
    advance_k();
    advance_check();
    if (f_reopen) advance_slow();
    prep_tile();
    load_both(W4_STAGE, W4_STAGE);
    wait_vm<16>();
    take_bias();
    barrier();
    static_for<NR>([&](auto n_) __attribute__((always_inline)) { read_n(n_, std::integral_constant<int, 0>{}); });

    while (true) {
        zero_acc();
        for (int n = c.left; n > 0; --n) k_tile();
        const Cursor done = c;
        start(c, c.v + grid);
        if constexpr (USE_BIAS) { if (c.left != 0) next_bias = bias_word(p, c.n0 + wn * 128); }
        // A's stage of the last K tile is free until the next body's loads: the wave's patch
        char* const eps = lds + (fill_a - s_wbase) + w * W4_EPI_BYTES_PER_WAVE;
        BiasBlock<TN> bias;
        if constexpr (USE_BIAS) spread_bias(bias, own_bias, eps);
        store_c_block<TM, TN, EPI, F32_OUT, true, USE_BIAS, STREAM>(p, acc, done.m0 + wm * 128, done.n0 + wn * 128, done.z, done.g, bias, eps,
                                                            std::bool_constant<PRE>{}, take_bias);
        if (c.left == 0) break;
        barrier();                                    // every wave is done with its patch
    }
}

// ---------------------------------------------------------------------------------------------
// host launcher
// ---------------------------------------------------------------------------------------------
template <bool A_KC, bool B_KC, int EPI, bool F32_OUT, bool PRE, bool STREAM>
static hipError_t launch4_as(const GemmArgs& a, hipStream_t stream) {
    static std::atomic<uint64_t> attr_done{0};
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_done.load(std::memory_order_relaxed) & bit)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tp_gemm4_kernel<A_KC, B_KC, EPI, F32_OUT, PRE, STREAM>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, W4_LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_done.fetch_or(bit, std::memory_order_relaxed);
    }
    const int total = a.tiles_m * a.tiles_n * a.split_k;
    const unsigned grid = (unsigned)(total < a.max_workgroups ? total : a.max_workgroups);
    return launch_kernel(tp_gemm4_kernel<A_KC, B_KC, EPI, F32_OUT, PRE, STREAM>, dim3(grid), dim3(W4_THREADS), W4_LDS_BYTES, stream, a);
}

template <bool A_KC, bool B_KC, int EPI, bool F32_OUT, bool PRE = false>
static hipError_t launch4_one(const GemmArgs& a, hipStream_t s) {
    // (planes never carry the hint: either kernel stores them)
    return a.stream ? launch4_as<A_KC, B_KC, EPI, F32_OUT, PRE, true>(a, s) : launch4_as<A_KC, B_KC, EPI, F32_OUT, PRE, false>(a, s);
}

// (the pre-activation of a split product is the fix-up's to store)
template <int EPI>
static hipError_t launch4_nn(const GemmArgs& a, bool f32, hipStream_t s) {
    if (a.pre && a.split_k == 1)
        return f32 ? launch4_one<true, false, EPI, true, true>(a, s) : launch4_one<true, false, EPI, false, true>(a, s);
    return f32 ? launch4_one<true, false, EPI, true>(a, s) : launch4_one<true, false, EPI, false>(a, s);
}

hipError_t launch_gemm4(int form, const GemmArgs& a, hipStream_t s) {
    const int epi = a.split_k > 1 ? EPI_NONE : (a.dg ? EPI_MUL_DGELU : (a.gelu ? EPI_BIAS_GELU : (a.bias ? EPI_BIAS : EPI_NONE)));
    const bool f32 = a.split_k > 1 || a.out_f32;
    switch (form) {
        case FORM_NN:
            if (epi == EPI_BIAS_GELU) return launch4_nn<EPI_BIAS_GELU>(a, f32, s);
            if (epi == EPI_BIAS)      return launch4_nn<EPI_BIAS>(a, f32, s);
            if (epi == EPI_NONE)      return launch4_nn<EPI_NONE>(a, f32, s);
            return hipErrorInvalidValue;
        case FORM_NT:
            if (epi == EPI_MUL_DGELU) return f32 ? launch4_one<true, true, EPI_MUL_DGELU, true>(a, s) : launch4_one<true, true, EPI_MUL_DGELU, false>(a, s);
            if (epi == EPI_NONE)      return f32 ? launch4_one<true, true, EPI_NONE, true>(a, s) : launch4_one<true, true, EPI_NONE, false>(a, s);
            return hipErrorInvalidValue;
        case FORM_TN:
            if (epi == EPI_NONE && f32) return launch4_one<false, false, EPI_NONE, true>(a, s);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tpl
