// gfx950 (MI355X, CDNA4): the GEMM of libtplinear for small products and for few rows (paper Section 2.2, tensor
// parallelism: the local block products C = sum_k A_k B_k and the two backward products).
//
//   * bound: latency (small products) or the stream of the weights (a handful of token rows), never MFMA.  So the
//     macro-tile is small, 32 x 32 (16 x 32 for at most 16 rows), which gives every CU one, and K is split over the
//     16 waves of the WORKGROUP: the partial sums meet in LDS, in a fixed order, and the epilogue follows in the
//     same launch -- no partial planes, no second kernel;
//   * no LDS staging and no barrier in the K loop: a wave loads its own fragments, 2 chunks of 64 k (whole 128-byte
//     lines of a contraction-contiguous operand) ahead of their
//     MFMAs (16 x 16 x 32).  A contraction-contiguous operand comes as 16 bytes per lane, which is a fragment; of
//     the other kind a lane takes 2 columns x 8 rows of k (dwords, a row of 16 lanes is 64 contiguous bytes) and
//     byte permutes make two fragments of them, whose column c is column 2 c + i of the tile;
//   * waves take the chunks in turn (wave w: w, w + 16, ...), across the steps of the sum.
#include "tp_stream.h"

namespace tpl {

namespace {
constexpr int SM_WAVES = 16, SM_THREADS = 64 * SM_WAVES, SM_BN = 32, SM_UNROLL = 2;
}

// MT: 16-row blocks of the tile (1 or 2; 2 if A is not contraction-contiguous)
template <int MT, bool A_KC, bool B_KC>
__global__ __launch_bounds__(SM_THREADS)
void tp_small_kernel(const GemmArgs p, const Epilogue e) {
    static_assert(MT == 2 || (MT == 1 && A_KC));
    constexpr int BM = 16 * MT;
    __shared__ __attribute__((aligned(16))) char red[SM_WAVES * BM * SM_BN * 4];
    const int t = threadIdx.x, l = t & 63, c = l & 15, kg = l >> 4;
    const int w = uni(t >> 6);
    int tm, tn, z, g = 0;
    tile_of_id(p, (int)blockIdx.x, tm, tn, z);
    if (p.n_groups > 1) {
        if (p.group_along_n) { g = tn / p.group_tiles; tn -= g * p.group_tiles; }
        else                 { g = tm / p.group_tiles; tm -= g * p.group_tiles; }
    }
    g = uni(g);
    const int m0 = uni(tm * BM), n0 = uni(tn * SM_BN);
    const int KC = (p.K + 63) / 64, T = p.n_steps * KC;           // chunks of 64 k: of a step, in all

    // Operand fragments of 32 k.  Descriptors start at the tile's first row (column) and end with the block:
    // rows past a ragged edge, and rows of k past the last one, read as zero; the rest is masked per lane.
    auto load_kc = [&](u32x4_t (&r)[2], int nb, const void* ptr, int ld, int rows, int row0, int k0) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(uni_ptr(static_cast<const uint16_t*>(ptr) + (int64_t)row0 * ld),
                                                    ((int64_t)(rows - row0 - 1) * ld + p.K) * 2);
        const int k = k0 + 8 * kg;
        const uint32_t off = k < p.K ? (uint32_t)((c * ld + k) * 2) : OOB_OFFSET;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (i < nb) r[i] = buf_load16(rs, off + (uint32_t)(16 * i * ld * 2));
    };
    auto load_xc = [&](uint32_t (&r)[8], const void* ptr, int ld, int X, int x0, int k0) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(uni_ptr(static_cast<const uint16_t*>(ptr) + x0),
                                                    ((int64_t)(p.K - 1) * ld + (X - x0)) * 2);
        const uint32_t off = x0 + 2 * c < X ? (uint32_t)(((k0 + 8 * kg) * ld + 2 * c) * 2) : OOB_OFFSET;
#pragma unroll
        for (int j = 0; j < 8; ++j) r[j] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(off + (uint32_t)(j * ld * 2)), 0, 0);
    };
    auto frag_xc = [&](const uint32_t (&r)[8], int i) __attribute__((always_inline)) {
        const uint32_t sel = i ? 0x07060302u : 0x05040100u;
        const u32x4_t v = {__builtin_amdgcn_perm(r[1], r[0], sel), __builtin_amdgcn_perm(r[3], r[2], sel),
                           __builtin_amdgcn_perm(r[5], r[4], sel), __builtin_amdgcn_perm(r[7], r[6], sel)};
        return __builtin_bit_cast(bf16x8_t, v);
    };

    f32x4_t acc[MT][2];
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i][0] = acc[i][1] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    int step = 0, kc = w;                                          // chunk w, as (step, chunk of the step)
    while (kc >= KC && step < p.n_steps) { kc -= KC; ++step; }
    for (int u = w; u < T; u += SM_WAVES * SM_UNROLL) {
        u32x4_t a_kc[2 * SM_UNROLL][2], b_kc[2 * SM_UNROLL][2];
        uint32_t a_xc[2 * SM_UNROLL][8], b_xc[2 * SM_UNROLL][8];
#pragma unroll
        for (int n = 0; n < 2 * SM_UNROLL; ++n) {
            // (a chunk past the end lies at K or beyond: every lane is masked, or past the descriptor's end)
            const int s = uni((step < p.n_steps ? step : p.n_steps - 1) + g);
            const int k0 = uni((step < p.n_steps ? kc : KC) * 64 + 32 * (n & 1));
            const int lda = uni(p.lda[s]), ldb = uni(p.ldb[s]);
            if constexpr (A_KC) load_kc(a_kc[n], MT, p.a[s], lda, p.M, m0, k0); else load_xc(a_xc[n], p.a[s], lda, p.M, m0, k0);
            if constexpr (B_KC) load_kc(b_kc[n], 2, p.b[s], ldb, p.N, n0, k0);  else load_xc(b_xc[n], p.b[s], ldb, p.N, n0, k0);
            if (n & 1) {
                kc += SM_WAVES;
                while (kc >= KC && step < p.n_steps) { kc -= KC; ++step; }
            }
        }
#pragma unroll
        for (int n = 0; n < 2 * SM_UNROLL; ++n) {
            bf16x8_t fb[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if constexpr (B_KC) fb[j] = __builtin_bit_cast(bf16x8_t, b_kc[n][j]); else fb[j] = frag_xc(b_xc[n], j);
            }
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                bf16x8_t fa;
                if constexpr (A_KC) fa = __builtin_bit_cast(bf16x8_t, a_kc[n][i]); else fa = frag_xc(a_xc[n], i);
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa, acc[i][j], 0, 0, 0);
            }
        }
    }

    // The operands are swapped (C^T = B^T A^T): a lane holds column block c's row of C.  acc[i][j][q]:
    // row 16 i + c (A contraction-contiguous) or 2 c + i, column 16 j + 4 kg + q or 8 kg + 2 q + j.
    // LDS: per wave BM rows of 128 bytes, 16-byte chunk n of row r at n ^ (r & 7).
    char* const mine = red + w * (BM * SM_BN * 4);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int r = A_KC ? 16 * i + c : 2 * c + i;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int n = B_KC ? 4 * h + kg : 2 * kg + h;
            f32x4_t v;
            if constexpr (B_KC) v = acc[i][h];
            else                v = f32x4_t{acc[i][0][2 * h], acc[i][1][2 * h], acc[i][0][2 * h + 1], acc[i][1][2 * h + 1]};
            *reinterpret_cast<f32x4_t*>(mine + r * 128 + ((n ^ (r & 7)) << 4)) = v;
        }
    }
    __syncthreads();
    if (t < BM * 8) {
        const int r = t >> 3, n = t & 7, row = m0 + r, col = n0 + 4 * n;
        const char* const at = red + r * 128 + ((n ^ (r & 7)) << 4);
        f32x4_t sum = *reinterpret_cast<const f32x4_t*>(at);
#pragma unroll
        for (int i = 1; i < SM_WAVES; ++i) {
            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(at + i * (BM * SM_BN * 4));
            sum = f32x4_t{sum[0] + v[0], sum[1] + v[1], sum[2] + v[2], sum[3] + v[3]};
        }
        if (row < p.M && col < p.N) {
            float x[4] = {sum[0], sum[1], sum[2], sum[3]};
            Epilogue eg = e;
            eg.out = p.outs[g]; eg.ldo = p.ldos[g];
            epilogue4(eg, x, row, col);
        }
    }
}

template <int MT, bool A_KC, bool B_KC>
static hipError_t launch_small_one(const GemmArgs& a, hipStream_t s) {
    const Epilogue e{a.out, a.ldo, a.out_f32, a.pre, a.ldp, a.bias, a.gelu, a.dg, a.lddg};
    return launch_kernel(tp_small_kernel<MT, A_KC, B_KC>, dim3((unsigned)(a.tiles_m * a.tiles_n)), dim3(SM_THREADS), 0, s, a, e);
}

hipError_t launch_small(int form, int tile_id, const GemmArgs& a, hipStream_t s) {
    if (a.split_k != 1) return hipErrorInvalidValue;
    const bool m16 = tile_id == TILE_16x32_SMALL;
    switch (form) {
        case FORM_NN: return m16 ? launch_small_one<1, true, false>(a, s) : launch_small_one<2, true, false>(a, s);
        case FORM_NT: return m16 ? launch_small_one<1, true, true>(a, s) : launch_small_one<2, true, true>(a, s);
        case FORM_TN: return m16 ? hipErrorInvalidValue : launch_small_one<2, false, false>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tpl
