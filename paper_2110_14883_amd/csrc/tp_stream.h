// Device-side helpers of the GEMM kernels that load straight from memory into LDS (tp_gemm4.hip, tp_gemm_ms.hip):
// compile-time loops, LDS access by address, direct-to-LDS loads, and the epilogue of one wave's block of C.
#pragma once
#include <utility>

#include "tp_device.h"

namespace tpl {

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// a value every lane agrees on, pinned to a scalar register (keeps the cursor arithmetic on the scalar unit)
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ const uint16_t* uni_ptr(const void* q) {
    const uint64_t v = reinterpret_cast<uint64_t>(q);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return reinterpret_cast<const uint16_t*>(((uint64_t)hi << 32) | lo);
}

// LDS access by 32-bit byte address.  The kernel has no static LDS, so its dynamic LDS starts at
// address 0 and an address is the offset into it.
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
typedef __attribute__((ext_vector_type(4))) short i16x4_t;
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;
__device__ __forceinline__ bf16x8_t lds_load_frag(uint32_t addr) { return *reinterpret_cast<const lds_bf16x8_t*>(addr); }
__device__ __forceinline__ bf16x4_t lds_load_tr(uint32_t addr) {
    return __builtin_bit_cast(bf16x4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_i16x4_t*>(addr)));
}

// One direct-to-LDS load: each lane's 16 bytes go from global memory straight into LDS, lane l at
// byte lds_base + 16 l (lds_base: wave-uniform, travels in M0), without touching the vector registers.
// Out-of-range lanes write zeros.  The compiler does not see this load: whoever reads the data waits
// for it with wait_vm() and a barrier.
__device__ __forceinline__ void dtl_load16(u32x4_t rsrc_words, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds_base), "v"(voff), "s"(rsrc_words) : "memory");
}
// the same at a constant distance from a wave-uniform base
template <int OFF> __device__ __forceinline__ void dtl_load16_at(u32x4_t rsrc_words, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds_base), "v"(voff), "s"(rsrc_words), "i"(OFF) : "memory", "scc");
}
template <int N> __device__ __forceinline__ void wait_vm() {      // at most N vector-memory operations outstanding
    static_assert(N >= 0 && N < 64);
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// The bias of a wave's 32 TN columns from n_sub, as the accumulators need it: word pair (j, g) is columns 32 j + 8 g + 4 (lane/32) .. + 3.
// Columns past N read as zero.
template <int TN> struct BiasBlock { u32x2_t v[TN][4]; };
template <int TN>
__device__ __forceinline__ void load_bias(BiasBlock<TN>& b, const GemmArgs& p, const int n_sub) {
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(uni_ptr(p.bias), (int64_t)p.N * 2);
    const int at = n_sub + 4 * ((threadIdx.x & 63) >> 5);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const u32x2_t w = __builtin_amdgcn_raw_buffer_load_b64(rs, (at + 32 * j + 8 * g) * 2, 0, 0);
            b.v[j][g] = w;
        }
}
// its value for accumulator element e of column block j
template <int TN>
__device__ __forceinline__ float bias_of(const BiasBlock<TN>& b, int j, int e) {
    const uint32_t w = b.v[j][e >> 2][(e >> 1) & 1];
    return e & 1 ? bf16_hi(w) : bf16_lo(w);
}

// The same through the wave's LDS patch, from one word a lane: columns 2 lane and 2 lane + 1 of the 128 (bias_word()).
__device__ __forceinline__ uint32_t bias_word(const GemmArgs& p, const int n_sub) {
    return __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(uni_ptr(p.bias), (int64_t)p.N * 2), (n_sub + 2 * (int)(threadIdx.x & 63)) * 2, 0, 0);
}
__device__ __forceinline__ void spread_bias(BiasBlock<4>& b, const uint32_t word, char* const eps) {
    const int l = threadIdx.x & 63;
    *reinterpret_cast<uint32_t*>(eps + 4 * l) = word;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) b.v[j][g] = *reinterpret_cast<const u32x2_t*>(eps + (32 * j + 8 * g + 4 * (l >> 5)) * 2);
}

// Epilogue of one wave's block of C: 32 TM rows x 32 TN columns from (m_sub, n_sub).  ADD_BIAS: `bias` goes on top of the finished
// sum (else it is there already, or there is none): one rounding, as in every other kernel here.
// acc[i][j][e]: row m = 32 i + lane%32, columns n = 32 j + 8 (e/4) + 4 (lane/32) + e%4.
// No branch depends on a lane: every global access goes through a buffer descriptor that starts at
// the first row of the block and ends with the last row of the matrix, so rows below a ragged edge are
// dropped by the range check, and a lane whose columns lie beyond N carries an out-of-range offset.
// One slab = 32 rows x 32 TN columns passes through the wave's LDS patch `eps` (2 TN KB, at least 4) so that
// stores are whole row segments.  ACC_HALF: the accumulators live in the accumulator half of the register file.
// Outputs leave with the streaming hint, K-split planes without: an output is not read again by this launch, and as ordinary lines
// of the L2 it drives out the operand panels that the XCD's other workgroups are about to read (6144 x 24576 fp32, K = 4096: 991 ->
// 905 us; 32896 x 2560 bf16 twice, K = 2 x 640: 287 -> 272; 8192 x 1024 bf16, K = 2 x 1024: 43 -> 40).  Whether they do is the host's to say
// (GemmArgs::stream).  The planes are read by the fix-up at once, from wherever they still are: with the hint 520 x 2056 in three planes takes 23.2 us against 21.8.
constexpr int ST_PLAIN = 0, ST_STREAM = 2;        // cache policy bits of a buffer store
// STREAM: the outputs' stores carry the hint.  keep: whether the pre-activation is stored too, a bool or (one way through, no branch) an
// integral_constant.  last(): called behind the last stores.
template <int TM, int TN, int EPI, bool F32_OUT, bool ACC_HALF, bool ADD_BIAS, bool STREAM, class Keep, class Last>
__device__ __forceinline__ void store_c_block(const GemmArgs& p, f32x16_t (&acc)[TM][TN], const int m_sub, const int n_sub,
                                              const int z, const int g_out, const BiasBlock<TN>& bias, char* const eps, Keep keep, Last last) {
    const int l = threadIdx.x & 63, r = l & 31, ch = l >> 5;
    const bool partial = !ADD_BIAS && !std::is_same_v<Keep, std::true_type> && p.split_k > 1;    // split K: raw fp32 partials, the fix-up kernel runs the epilogue
    constexpr bool use_gelu = EPI == EPI_BIAS_GELU;
    constexpr bool use_dg = EPI == EPI_MUL_DGELU;
    const bool use_pre = !use_dg && keep;
    constexpr bool one_pass = !F32_OUT && std::is_same_v<Keep, std::true_type>;
    const int rows_left = p.M - m_sub;
    // rows m_sub .. M - 1 of a matrix with leading dimension ld (elements of es bytes), N columns
    auto block_rsrc = [&](const void* base, int64_t ld, int es) __attribute__((always_inline)) {
        const int64_t nrec = rows_left > 0 ? ((int64_t)(rows_left - 1) * ld + p.N) * es : 0;
        return make_rsrc(uni_ptr(static_cast<const char*>(base) + (int64_t)m_sub * ld * es), nrec);
    };
    __amdgpu_buffer_rsrc_t rs_dg;
    uint32_t dg_lane = 0;
    if constexpr (use_dg) {
        rs_dg = block_rsrc(p.dg, p.lddg, 2);
        dg_lane = (uint32_t)((r * (int)p.lddg + n_sub + 4 * ch) * 2);   // columns past N: the next row's values or zeros, never stored
    }
    // ACC_HALF: the accumulators stay where the MFMAs keep them (the accumulator half of the register file) and
    // are fetched four at a time, where they are used: left to itself the compiler copies all 256 out
    // at once, which cannot fit beside the staging registers.
    auto raw4 = [&](int i, int j, int g, float (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (ACC_HALF) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[e]) : "a"(acc[i][j][4 * g + e]));
            else                    v[e] = acc[i][j][4 * g + e];
        }
    };
    auto preact4 = [&](int i, int j, int g, float (&v)[4]) __attribute__((always_inline)) {
        raw4(i, j, g, v);
        if constexpr (ADD_BIAS) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t w = bias.v[j][g][h];
                // (with fp32 outputs unpacked where it is used: the unpacked block is another 64 registers)
                if constexpr (F32_OUT) asm volatile("" : "+v"(w));
                v[2 * h] += bf16_lo(w);
                v[2 * h + 1] += bf16_hi(w);
            }
        }
    };
    u32x2_t dg_v[TN][4];                         // (asked for one slab ahead the pass is 2 % slower)
    auto load_dg = [&](int i) __attribute__((always_inline)) {
        if constexpr (use_dg) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    dg_v[j][g] = __builtin_amdgcn_raw_buffer_load_b64(rs_dg, dg_lane + (uint32_t)(((32 * i) * (int)p.lddg + 32 * j + 8 * g) * 2), 0, 0);
        }
    };
    auto final4 = [&](int i, int j, int g, float (&v)[4]) __attribute__((always_inline)) {
        preact4(i, j, g, v);
        if constexpr (use_gelu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_f(v[e]);
        }
        if constexpr (use_dg) {
            const u32x2_t a = dg_v[j][g];
            v[0] = dgelu_times(v[0], bf16_lo(a[0])); v[1] = dgelu_times(v[1], bf16_hi(a[0]));
            v[2] = dgelu_times(v[2], bf16_lo(a[1])); v[3] = dgelu_times(v[3], bf16_hi(a[1]));
        }
    };
    // bf16 slab of 32 rows x 32 TN columns: rows of 64 TN bytes in the patch; a lane writes 8 bytes and
    // reads back 16 (chunk index XOR row keeps both conflict-free), stores are whole row segments:
    // lane l stores columns 8 (l % CPR) .. + 7 of rows l / CPR + RPI it
    constexpr int CPR = 4 * TN, RPI = 64 / CPR;        // 16-byte chunks of a row; rows a wave instruction covers
    static_assert(TN == 2 || TN == 4);
    auto swz = [](int row) __attribute__((always_inline)) { return TN == 4 ? row & 15 : (row >> 1) & 7; };
    auto lane_bf16 = [&](int ld) __attribute__((always_inline)) {
        return (n_sub + 8 * (l % CPR)) < p.N ? (uint32_t)(((l / CPR) * ld + n_sub + 8 * (l % CPR)) * 2) : OOB_OFFSET;
    };
    auto put_bf16 = [&](int j, int g, const u32x2_t v) __attribute__((always_inline)) {
        *reinterpret_cast<u32x2_t*>(eps + r * (16 * CPR) + (((4 * j + g) ^ swz(r)) << 4) + 8 * ch) = v;
    };
    constexpr int out_policy = STREAM ? ST_STREAM : ST_PLAIN;
    auto store_bf16 = [&](int i, __amdgpu_buffer_rsrc_t rs, int ld, uint32_t lane) __attribute__((always_inline)) {
        const int cc = l % CPR;
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int rr = it * RPI + l / CPR;
            const u32x4_t v = *reinterpret_cast<const u32x4_t*>(eps + rr * (16 * CPR) + ((cc ^ swz(rr)) << 4));
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)(lane + (uint32_t)((32 * i + RPI * it) * ld * 2)), 0, out_policy);
        }
    };
    auto slab_bf16 = [&](int i, auto value4, __amdgpu_buffer_rsrc_t rs, int ld) __attribute__((always_inline)) {
        const uint32_t lane = lane_bf16(ld);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float x[4];
                value4(i, j, g, x);
                put_bf16(j, g, u32x2_t{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])});
            }
        store_bf16(i, rs, ld, lane);
    };
    // The pre-activation and the bf16 output: the accumulators are read and the bias added once.  (The output's stores follow its own
    // arithmetic: right behind those of the pre-activation they take 5 % longer where rows are off cache lines.)
    auto slab_pre_out = [&](int i, __amdgpu_buffer_rsrc_t rs_p, int ldp, __amdgpu_buffer_rsrc_t rs_o, int ldo) __attribute__((always_inline)) {
        float x[TN][4][4];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                preact4(i, j, g, x[j][g]);
                put_bf16(j, g, u32x2_t{pack_bf16(x[j][g][0], x[j][g][1]), pack_bf16(x[j][g][2], x[j][g][3])});
            }
        store_bf16(i, rs_p, ldp, lane_bf16(ldp));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if constexpr (use_gelu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[j][g][e] = gelu_f(x[j][g][e]);
                }
                put_bf16(j, g, u32x2_t{pack_bf16(x[j][g][0], x[j][g][1]), pack_bf16(x[j][g][2], x[j][g][3])});
            }
        store_bf16(i, rs_o, ldo, lane_bf16(ldo));
    };
    // fp32 slab, one 32-column block at a time: rows of 128 bytes; lane l stores columns
    // 4 (l % 8) .. + 3 of rows l / 8 + 8 it
    auto slab_f32 = [&](int i, auto value4, auto policy, __amdgpu_buffer_rsrc_t rs, int ld) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n_sub + 32 * j + 4 * (l & 7);
            const uint32_t lane = n < p.N ? (uint32_t)(((l >> 3) * ld + n) * 4) : OOB_OFFSET;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float x[4];
                value4(i, j, g, x);
                const f32x4_t v = {x[0], x[1], x[2], x[3]};
                *reinterpret_cast<f32x4_t*>(eps + r * 128 + (((2 * g + ch) ^ ((r >> 1) & 7)) << 4)) = v;
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int rr = it * 8 + (l >> 3), cc = l & 7;
                const u32x4_t v = *reinterpret_cast<const u32x4_t*>(eps + rr * 128 + ((cc ^ ((rr >> 1) & 7)) << 4));
                __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)(lane + (uint32_t)((32 * i + 8 * it) * ld * 4)), 0, decltype(policy)::value);
            }
        }
    };
    // (with ACC_HALF the last MFMA's result is read by hand-placed instructions: give it the 19 cycles it needs)
    if constexpr (ACC_HALF) asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
    if (partial) {
        const __amdgpu_buffer_rsrc_t rs_ws = block_rsrc(p.ws + ((int64_t)z * p.n_groups + g_out) * p.M * p.N, (int64_t)p.N, 4);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            slab_f32(i, raw4, std::integral_constant<int, ST_PLAIN>{}, rs_ws, p.N);
            __builtin_amdgcn_sched_barrier(0);
        }
        last();
    } else {
        const int ldo = (int)p.ldos[g_out];
        const __amdgpu_buffer_rsrc_t rs_out = block_rsrc(p.outs[g_out], ldo, F32_OUT ? 4 : 2);
        __amdgpu_buffer_rsrc_t rs_pre;
        if constexpr (!use_dg) rs_pre = block_rsrc(p.pre, p.ldp, 2);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            load_dg(i);
            if constexpr (one_pass) {
                slab_pre_out(i, rs_pre, (int)p.ldp, rs_out, ldo);
            } else {
                if constexpr (!use_dg) {
                    if (use_pre) slab_bf16(i, preact4, rs_pre, (int)p.ldp);
                }
                if constexpr (F32_OUT) slab_f32(i, final4, std::integral_constant<int, out_policy>{}, rs_out, ldo);
                else                   slab_bf16(i, final4, rs_out, ldo);
            }
            if (i == TM - 1) last();
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

}  // namespace tpl
