// gfx950 (MI355X, CDNA4): the GEMM of libtplinear for small products and for few rows (paper Section 2.2, tensor
// parallelism: the local block products C = sum_k A_k B_k and the two backward products).
//
//   * bound: latency (small products) or the stream of the weights (a handful of token rows), never MFMA.  So the
//     macro-tile is small, 16 or 32 rows by 16, 32 or 64 columns, which gives every CU one, and K is split over the
//     eight waves of the WORKGROUP: the partial sums meet in LDS, in a fixed order, and the epilogue follows in the
//     same launch -- no partial planes, no second kernel.  Tiles of 64 columns (forward of at most 32 rows: whole cache lines of weight
//     rows) may split K over workgroups too, with planes and a fix-up: 33.5 MB of weights from memory 19.9 -> 13.6 us;
//   * waves take the chunks of 64 k in turn (wave w of part z of Z: 8 z + w, 8 (z + Z) + w, ...), across the steps of the sum, and work alone until
//     the end: each has its own ring of LDS slots, filled by direct-to-LDS loads (16 bytes a lane: 8 lines or 16
//     half lines an instruction) one to three chunks ahead (slots - 1; a tile of 32 x 64 has one slot and none ahead), with no barrier in the K loop.  An operand that is not
//     contraction-contiguous is transposed on the way out, by ds_read_b64_tr_b16.
//     (Fragments loaded straight into registers, 16 bytes of a row or 4 bytes of 8 rows a lane, kept the address path
//     busy four times as long: 16 x 4096 x 4096 dX 13.9 us against 8.0, 512 x 1024 x 1024 dX 12.5 against 7.5, forward
//     10.7 against 8.8.)
#include "tp_stream.h"

namespace tpl {

namespace {
constexpr int SM_WAVES = 8, SM_THREADS = 64 * SM_WAVES;
template <int MT, int NT> struct SmShape {
    static constexpr int BM = 16 * MT, BN = 16 * NT, A_BYTES = BM * 128, B_BYTES = BN * 128, SLOT = A_BYTES + B_BYTES;   // one chunk of 64 k of both operands
    static constexpr int NS = 163840 / (SM_WAVES * SLOT) > 4 ? 4 : 163840 / (SM_WAVES * SLOT), LDS_BYTES = SM_WAVES * NS * SLOT;
    static_assert(SM_WAVES * BM * BN * 4 <= LDS_BYTES && LDS_BYTES <= 163840);
};
}

// One workgroup's tile `id` of a product.  MT, NT: 16-row and 16-column blocks of the tile (MT 2 if A is not
// contraction-contiguous, NT 2 or 4 if B is not, else 1 or 2 each)
template <int MT, int NT, bool A_KC, bool B_KC>
__device__ __forceinline__ void small_tile(const GemmArgs& p, const Epilogue& e, const int id) {
    static_assert((MT == 2 || (MT == 1 && A_KC)) && (B_KC ? NT <= 2 : NT >= 2));
    using Sh = SmShape<MT, NT>;
    preload(p);
    asm volatile("" :: "s"(e.out), "s"(e.dg));
    constexpr int BM = Sh::BM, BN = Sh::BN, NS = Sh::NS, A_BYTES = Sh::A_BYTES;
    constexpr int LA = A_BYTES / 1024, LB = Sh::B_BYTES / 1024, LPC = LA + LB;    // loads of a chunk
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int t = threadIdx.x, l = t & 63, c = l & 15, kg = l >> 4;
    const int w = uni(t >> 6);
    int tm, tn, z, g = 0;
    tile_of_id(p, id, tm, tn, z);
    if (p.n_groups > 1) {
        if (p.group_along_n) { g = tn / p.group_tiles; tn -= g * p.group_tiles; }
        else                 { g = tm / p.group_tiles; tm -= g * p.group_tiles; }
    }
    g = uni(g);
    const int m0 = uni(tm * BM), n0 = uni(tn * BN);
    const int KC = (p.K + 63) / 64, T = p.n_steps * KC;           // chunks of 64 k: of a step, in all
    const uint32_t mine = (uint32_t)(w * NS * Sh::SLOT);

    // Descriptors start at the tile's first row (column).  A contraction-contiguous one ends with the tile's last row that
    // exists: its size stays below OOB_OFFSET for every leading dimension, however many rows the matrix has.  The other kind
    // ends with the block (the host refuses spans of 2 GiB).  So rows past a ragged edge, and rows of k past the last one,
    // read as zero; the rest is masked per lane.
    //   contraction-contiguous: rows of 128 bytes, chunk q of row r at q ^ ((r >> 1) & 7); load n: rows 8 n + l / 8;
    //   otherwise: 64 rows of k, placed so that the groups of 4 rows x 16 columns of a half-wave's transposing read (8 rows
    //     apart) lie in different banks: of 64 bytes (32 columns), chunk q of row k at q ^ 2 ((k >> 3) & 1), load n: rows 16 n + l / 4; of
    //     128 bytes (64 columns), chunk q of row k at q ^ 2 ((k & 3) ^ ((k >> 3) & 1)), load n: rows 8 n + l / 8.
    auto load_kc = [&](auto n_loads, const void* ptr, int ld, int rows, int row0, int k0, bool live, uint32_t dst) __attribute__((always_inline)) {
        const uint64_t base = reinterpret_cast<uint64_t>(static_cast<const uint16_t*>(ptr) + (int64_t)row0 * ld);
        constexpr int R = 8 * decltype(n_loads)::value;
        const int have = rows - row0 < R ? rows - row0 : R;
        const int64_t nrec = live ? ((int64_t)(have - 1) * ld + p.K) * 2 : 0;
        const u32x4_t rw = {(uint32_t)uni((int)(uint32_t)base), (uint32_t)uni((int)((uint32_t)(base >> 32) & 0xffffu)),
                            (uint32_t)uni((int)(uint32_t)nrec), 0x00020000u};
        static_for<decltype(n_loads)::value>([&](auto n_) __attribute__((always_inline)) {
            constexpr int n = decltype(n_)::value;
            const int r = 8 * n + (l >> 3), k = k0 + (((l & 7) ^ ((r >> 1) & 7)) << 3);
            dtl_load16(rw, k < p.K ? (uint32_t)((r * ld + k) * 2) : OOB_OFFSET, dst + n * 1024);
        });
    };
    auto load_xc = [&](auto blocks, const void* ptr, int ld, int X, int x0, int k0, bool live, uint32_t dst) __attribute__((always_inline)) {
        const uint64_t base = reinterpret_cast<uint64_t>(static_cast<const uint16_t*>(ptr) + x0);
        const int64_t nrec = live ? ((int64_t)(p.K - 1) * ld + (X - x0)) * 2 : 0;
        const u32x4_t rw = {(uint32_t)uni((int)(uint32_t)base), (uint32_t)uni((int)((uint32_t)(base >> 32) & 0xffffu)),
                            (uint32_t)uni((int)(uint32_t)nrec), 0x00020000u};
        if constexpr (decltype(blocks)::value == 4) {
            static_for<8>([&](auto n_) __attribute__((always_inline)) {
                constexpr int n = decltype(n_)::value;
                const int x = ((l & 7) ^ (2 * (((l >> 3) & 3) ^ (n & 1)))) * 8;
                dtl_load16(rw, x0 + x < X ? (uint32_t)(((k0 + 8 * n + (l >> 3)) * ld + x) * 2) : OOB_OFFSET, dst + n * 1024);
            });
        } else {
            const int x = ((l & 3) ^ (2 * (l >> 5))) * 8;
            const uint32_t off = x0 + x < X ? (uint32_t)(((k0 + (l >> 2)) * ld + x) * 2) : OOB_OFFSET;
            static_for<4>([&](auto n_) __attribute__((always_inline)) {
                constexpr int n = decltype(n_)::value;
                dtl_load16(rw, off + (uint32_t)(32 * n * ld), dst + n * 1024);
            });
        }
    };
    const int first = z * SM_WAVES + w, stride = SM_WAVES * p.split_k;   // this wave's chunks of the sum
    int step = 0, kc = first;                                      // the next chunk to fetch, as (step, chunk of the step)
    while (kc >= KC && step < p.n_steps) { kc -= KC; ++step; }
    auto fetch = [&](auto slot) __attribute__((always_inline)) {   // (past the end: empty descriptors, zeros nobody uses)
        const bool live = step < p.n_steps;
        const int s = uni((live ? step : p.n_steps - 1) + g), k0 = uni(kc * 64);
        const uint32_t dst = mine + decltype(slot)::value * Sh::SLOT;
        if constexpr (A_KC) load_kc(std::integral_constant<int, LA>{}, p.a[s], uni(p.lda[s]), p.M, m0, k0, live, dst);
        else                load_xc(std::integral_constant<int, MT>{}, p.a[s], uni(p.lda[s]), p.M, m0, k0, live, dst);
        if constexpr (B_KC) load_kc(std::integral_constant<int, LB>{}, p.b[s], uni(p.ldb[s]), p.N, n0, k0, live, dst + A_BYTES);
        else                load_xc(std::integral_constant<int, NT>{}, p.b[s], uni(p.ldb[s]), p.N, n0, k0, live, dst + A_BYTES);
        kc += stride;
        while (kc >= KC && step < p.n_steps) { kc -= KC; ++step; }
        if (step >= p.n_steps) kc = 0;
    };
    // fragment (16 rows or columns, block i) x (32 k, half h)
    auto frag = [&](auto kc_form, auto blocks, uint32_t at, int i, int h) __attribute__((always_inline)) {
        if constexpr (decltype(kc_form)::value) {
            const int r = 16 * i + c;
            return lds_load_frag(at + r * 128 + (((4 * h + kg) ^ ((r >> 1) & 7)) << 4));
        } else {
            const int k = 32 * h + 8 * kg + (c >> 2);              // and k + 4
            const uint32_t a = decltype(blocks)::value == 4 ? at + k * 128 + ((2 * (i ^ (c >> 2) ^ (kg & 1))) << 4) + 8 * (l & 3)
                                                            : at + k * 64 + ((2 * i ^ 2 * (kg & 1)) << 4) + 8 * (l & 3);
            const bf16x4_t lo = lds_load_tr(a), hi = lds_load_tr(a + (decltype(blocks)::value == 4 ? 512 : 256));
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };
    f32x4_t acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    auto one_chunk = [&](auto slot_) __attribute__((always_inline)) {
        constexpr int slot = decltype(slot_)::value;
        // the slot to refill was read one chunk ago: its fragments have arrived
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        fetch(std::integral_constant<int, (slot + NS - 1) % NS>{});
        wait_vm<(NS - 1) * LPC>();                                 // this wave's own loads: no barrier
        asm volatile("" ::: "memory");
        const uint32_t at = mine + slot * Sh::SLOT;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8_t fb[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) fb[j] = frag(std::integral_constant<bool, B_KC>{}, std::integral_constant<int, NT>{}, at + A_BYTES, j, h);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const bf16x8_t fa = frag(std::integral_constant<bool, A_KC>{}, std::integral_constant<int, MT>{}, at, i, h);
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa, acc[i][j], 0, 0, 0);
            }
        }
    };
    static_for<NS - 1>([&](auto s_) __attribute__((always_inline)) { fetch(s_); });
    for (int u = first; u < T; u += stride * NS)                     // (a chunk past the end of the last round is zeros)
        static_for<NS>([&](auto s_) __attribute__((always_inline)) { one_chunk(s_); });

    // The operands are swapped (C^T = B^T A^T): acc[i][j][q] is row 16 i + c, column 16 j + 4 kg + q of the tile.
    // LDS: per wave BM rows of 4 BN bytes, 16-byte chunk n of row r at n ^ (r & (BN / 4 - 1)).
    constexpr int CH = BN / 4;
    wait_vm<0>();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int r = 16 * i + c;
#pragma unroll
        for (int j = 0; j < NT; ++j)
            *reinterpret_cast<f32x4_t*>(lds + w * (BM * BN * 4) + r * (BN * 4) + (((4 * j + kg) ^ (r & (CH - 1))) << 4)) = acc[i][j];
    }
    __syncthreads();
    if (t < BM * CH) {
        const int r = t / CH, n = t % CH, row = m0 + r, col = n0 + 4 * n;
        const char* const at = lds + r * (BN * 4) + ((n ^ (r & (CH - 1))) << 4);
        f32x4_t sum = *reinterpret_cast<const f32x4_t*>(at);
#pragma unroll
        for (int i = 1; i < SM_WAVES; ++i) {
            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(at + i * (BM * BN * 4));
            sum = f32x4_t{sum[0] + v[0], sum[1] + v[1], sum[2] + v[2], sum[3] + v[3]};
        }
        if (row < p.M && col < p.N) {
            if (p.split_k > 1) {                                   // the fix-up kernel adds the planes and runs the epilogue
                *reinterpret_cast<f32x4_t*>(p.ws + ((int64_t)(z * p.n_groups + g) * p.M + row) * p.N + col) = sum;
                return;
            }
            float x[4] = {sum[0], sum[1], sum[2], sum[3]};
            Epilogue eg = e;
            eg.out = p.outs[g]; eg.ldo = p.ldos[g];
            epilogue4(eg, x, row, col);
        }
    }
}

template <int MT, int NT, bool A_KC, bool B_KC>
__global__ __launch_bounds__(SM_THREADS)
void tp_small_kernel(const GemmArgs p, const Epilogue e) {
    small_tile<MT, NT, A_KC, B_KC>(p, e, (int)blockIdx.x);
}

// dX (NT) and dW (TN) of one backward call in one launch: the two do not depend on each other, neither fills the chip for long, and
// a launch of its own costs each about as much as its work (300 x 136, K = 2 x 328 and 136 x 328, K = 2 x 300: 5.2 + 5.2 us).
template <int MT, int NT>
__global__ __launch_bounds__(SM_THREADS)
void tp_small_pair_kernel(const GemmArgs px, const Epilogue ex, const GemmArgs pw, const Epilogue ew, const int n_first) {
    if ((int)blockIdx.x < n_first) small_tile<MT, NT, true, true>(px, ex, (int)blockIdx.x);
    else                           small_tile<2, 2, false, false>(pw, ew, (int)blockIdx.x - n_first);
}

// the kernel with its LDS limit raised, once per device
template <class... P>
static hipError_t launch_with_lds(void (*kernel)(P...), std::atomic<uint64_t>& attr_done, unsigned grid, int lds_bytes, hipStream_t s, P... args) {
    int dev = 0;
    if (hipError_t err = hipGetDevice(&dev); err != hipSuccess) return err;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_done.load(std::memory_order_relaxed) & bit)) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (err != hipSuccess) return err;
        attr_done.fetch_or(bit, std::memory_order_relaxed);
    }
    return launch_kernel(kernel, dim3(grid), dim3(SM_THREADS), lds_bytes, s, args...);
}
static Epilogue epilogue_of(const GemmArgs& a) { return Epilogue{a.out, a.ldo, a.out_f32, a.pre, a.ldp, a.bias, a.gelu, a.dg, a.lddg}; }

template <int MT, int NT, bool A_KC, bool B_KC>
static hipError_t launch_small_one(const GemmArgs& a, hipStream_t s) {
    static std::atomic<uint64_t> attr_done{0};
    return launch_with_lds(tp_small_kernel<MT, NT, A_KC, B_KC>, attr_done, (unsigned)(a.tiles_m * a.tiles_n * a.split_k), SmShape<MT, NT>::LDS_BYTES, s, GemmArgs(a),
                           epilogue_of(a));
}
template <int MT, int NT>
static hipError_t launch_pair_one(const GemmArgs& x, const GemmArgs& w, hipStream_t s) {
    static std::atomic<uint64_t> attr_done{0};
    constexpr int lds_bytes = SmShape<MT, NT>::LDS_BYTES > SmShape<2, 2>::LDS_BYTES ? SmShape<MT, NT>::LDS_BYTES : SmShape<2, 2>::LDS_BYTES;
    const int n_first = x.tiles_m * x.tiles_n;
    return launch_with_lds(tp_small_pair_kernel<MT, NT>, attr_done, (unsigned)(n_first + w.tiles_m * w.tiles_n), lds_bytes, s, GemmArgs(x), epilogue_of(x),
                           GemmArgs(w), epilogue_of(w), int(n_first));
}
hipError_t launch_small_pair(int tile_x, const GemmArgs& x, int tile_w, const GemmArgs& w, hipStream_t s) {
    if (x.split_k != 1 || w.split_k != 1 || tile_w != TILE_32x32_SMALL) return hipErrorInvalidValue;
    switch (tile_x) {
        case TILE_32x32_SMALL: return launch_pair_one<2, 2>(x, w, s);
        case TILE_16x32_SMALL: return launch_pair_one<1, 2>(x, w, s);
        case TILE_32x16_SMALL: return launch_pair_one<2, 1>(x, w, s);
        case TILE_16x16_SMALL: return launch_pair_one<1, 1>(x, w, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_small(int form, int tile_id, const GemmArgs& a, hipStream_t s) {
    switch (form) {
        case FORM_NN:
            switch (tile_id) {
                case TILE_32x32_SMALL: return launch_small_one<2, 2, true, false>(a, s);
                case TILE_16x32_SMALL: return launch_small_one<1, 2, true, false>(a, s);
                case TILE_16x64_SMALL: return launch_small_one<1, 4, true, false>(a, s);
                case TILE_32x64_SMALL: return launch_small_one<2, 4, true, false>(a, s);
                default: return hipErrorInvalidValue;
            }
        case FORM_NT:
            switch (tile_id) {
                case TILE_32x32_SMALL: return launch_small_one<2, 2, true, true>(a, s);
                case TILE_16x32_SMALL: return launch_small_one<1, 2, true, true>(a, s);
                case TILE_32x16_SMALL: return launch_small_one<2, 1, true, true>(a, s);
                case TILE_16x16_SMALL: return launch_small_one<1, 1, true, true>(a, s);
                default: return hipErrorInvalidValue;
            }
        case FORM_TN: return tile_id == TILE_32x32_SMALL ? launch_small_one<2, 2, false, false>(a, s) : hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tpl
