// Batched CSB-MVM for gfx950 from the quad section of the image: Y = A X in steps of FOUR kernel rows.
//
// v_mfma_f32_4x4x1_16b_f32 is sixteen 4 x 4 outer products side by side, as fast per multiply-add as the 16 x 16
// forms (measured, clocks per SIMD: 9.8 for 256 multiply-adds; 34 for the 1024 of the 16 x 16 x 4 form).  With the right-hand
// sides of one input row spread over its sixteen blocks (lane = right-hand side) and its A operand taken from ONE
// block (CBSZ broadcasts, ABID names the block), an instruction multiplies four kernel rows by one input row of 64
// right-hand sides: a 7 x 7 kernel costs 14 of them per 64 right-hand sides, where 16-row instructions, rows
// scattered over a 32-row tile, spend as long as 56.  One register of A serves many instructions, and a result
// register IS an output row (lane = right-hand side): it is added to the wavefront's accumulator of that row, a
// register picked by the row's place in the tile (VGPR indexing), so results pass through LDS once, at
// the end, when the wavefronts' tiles are summed in wavefront order.
// What it all hangs on is in a pass's record (QuadRec), which comes in over the scalar path: no record is staged, nothing is
// looked up per lane.  An input row that is not finite reaches the rows that use it and no others.
//
// What bounds it: the pipe that MFMA and vector instructions share (with every load hitting the caches it is no faster;
// without the products 8192 x 8192 x 128 takes 16 us instead of 35): products of 4 x 4 granularity, 1.45 times those of the
// matrix, the row sums (a vector instruction per row and 64 right-hand sides), about 30 others per pass.  Scalar instructions
// run beside it.  8192 x 8192 at 12x in 32 x 32 blocks, us, records and 16-row instructions from the tile sections / here: 128
// right-hand sides 63.0 / 34.8 (41 TFLOP/s of products the matrix has), 64 36.9 / 25.0, 16 24.7 / 21.7, 512 242 / 116;
// 4096 x 4096 in 16-row blocks x 128 29.2 / 15.8, in 64-row blocks 17.0 / 11.0; two LSTM layers of 1024 at batch 64 13.7 / 11.2
// per step.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "csb_spmm.hpp"

namespace csb {

typedef float floatx32 __attribute__((ext_vector_type(32)));

// ---- the accumulators: registers with fixed numbers, so that one of them can be picked by an index ----------
// NT tiles of 32 rows from v60 on; behind each a spare one (index 32) for the rows a quad lacks.
template <int NT>
struct QuadAcc {
    floatx32 v[NT];
};

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"      // (M0 is named as clobbered: nothing here keeps a value in it)
// Rows s of the accumulators += d, s four places of a byte each.  The wait in front covers an MFMA that wrote d; the index
// is the low byte of the scalar.
__device__ __forceinline__ void add_rows(QuadAcc<1> &acc, const floatx4 (&d)[1], const uint32_t s) {
    asm volatile("s_nop 7\n\ts_set_gpr_idx_on %[s0], 0x9\n\tv_add_f32 v60, v60, %[d0]\n\ts_set_gpr_idx_idx %[s1]\n\tv_add_f32 v60, v60, %[d1]\n\t"
                 "s_set_gpr_idx_idx %[s2]\n\tv_add_f32 v60, v60, %[d2]\n\ts_set_gpr_idx_idx %[s3]\n\tv_add_f32 v60, v60, %[d3]\n\ts_set_gpr_idx_off"
                 : "+{v[60:91]}"(acc.v[0])
                 : [d0] "v"(d[0][0]), [d1] "v"(d[0][1]), [d2] "v"(d[0][2]), [d3] "v"(d[0][3]), [s0] "s"(s), [s1] "s"(s >> 8), [s2] "s"(s >> 16),
                   [s3] "s"(s >> 24)
                 : "v92", "m0");
}
#define CSB_ROW2(I) "v_add_f32 v60, v60, %[d" #I "]\n\tv_add_f32 v94, v94, %[e" #I "]\n\t"
__device__ __forceinline__ void add_rows(QuadAcc<2> &acc, const floatx4 (&d)[2], const uint32_t s) {
    asm volatile("s_nop 7\n\ts_set_gpr_idx_on %[s0], 0x9\n\t" CSB_ROW2(0) "s_set_gpr_idx_idx %[s1]\n\t" CSB_ROW2(1) "s_set_gpr_idx_idx %[s2]\n\t" CSB_ROW2(2)
                 "s_set_gpr_idx_idx %[s3]\n\t" CSB_ROW2(3) "s_set_gpr_idx_off"
                 : "+{v[60:91]}"(acc.v[0]), "+{v[94:125]}"(acc.v[1])
                 : [d0] "v"(d[0][0]), [d1] "v"(d[0][1]), [d2] "v"(d[0][2]), [d3] "v"(d[0][3]), [e0] "v"(d[1][0]), [e1] "v"(d[1][1]),
                   [e2] "v"(d[1][2]), [e3] "v"(d[1][3]), [s0] "s"(s), [s1] "s"(s >> 8), [s2] "s"(s >> 16), [s3] "s"(s >> 24)
                 : "v92", "v126", "m0");
}
#undef CSB_ROW2
#pragma clang diagnostic pop

// NT times 64 / G right-hand sides, in G groups of 64 / G lanes that take every G-th column of a pass (each
// group holds partial sums; they meet with the wavefronts' at the end).  G = 1 or 2: four groups of 16 right-hand sides
// are never faster than two of 32 with half the lanes idle (8192 x 8192 x 16: 21.7 and 21.2 us; 8192 x 2048 x 16
// in 64 x 64 blocks 7.2 and 6.6): a pass's instructions are the same.
template <int NT, int G>
struct QuadForm {
    static_assert(G == 1 || G == 2, "one or two groups");
    static constexpr uint32_t lanes = 64 / G;            // lanes of a group
    static constexpr uint32_t columns = lanes * NT;      // right-hand sides per workgroup
    static constexpr int steps = kQuadCols / G;          // input loads, and instructions per four rows, of a pass
    static constexpr int cbsz = G == 1 ? 4 : 3;
};

// The two halves of a pass's record, in scalar registers: the kernels read them through the constant address space.
typedef uint32_t uint32x8 __attribute__((ext_vector_type(8)));
#define CSB_CONST_AS __attribute__((address_space(4)))

__device__ __forceinline__ uint32_t first_record(const QuadMat &m, const uint32_t list) {
    return m.list_stride ? list * m.list_stride : ((const uint32_t CSB_CONST_AS *)(uintptr_t)m.table)[list];
}
__device__ __forceinline__ uint32_t list_length(const QuadMat &m, const uint32_t list, const uint32x8 &first) {
    if (m.list_stride) return first[6];
    const uint32_t CSB_CONST_AS *t = (const uint32_t CSB_CONST_AS *)(uintptr_t)m.table + list;
    return t[1] - t[0];
}

template <int NT, int G>
struct QuadOps {
    uint32_t a[4];                                       // register j: rows of the quads j and 4 + j by 8 columns
    uint32_t x[kQuadCols / G][NT];                       // a lane's right-hand sides of G columns
};

template <int S, int S1, int Q, int NT, int G>
__device__ __forceinline__ void quad_steps(const QuadOps<NT, G> &o, floatx4 (&D)[NT]) {
    if constexpr (S < S1) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
            D[t] = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(o.a[Q & 3]), __uint_as_float(o.x[S][t]), D[t], QuadForm<NT, G>::cbsz, 2 * S + (Q >> 2), 0);
        quad_steps<S + 1, S1, Q>(o, D);
    }
}

// One list of a tile's passes, added into `acc`.  bt0: first right-hand side
// of the workgroup.
template <int NT, int G, bool TWO>
__device__ __forceinline__ void quad_passes(const QuadMat &m, const XSrc &X, const uint32_t list, const uint32_t bt0,
                                            const uint32_t batch, QuadAcc<NT> &acc) {
    using F = QuadForm<NT, G>;
    const uint32_t lane = threadIdx.x & 63u, group = lane / F::lanes;
    // the lane's place in an A register: row of its quad, which of the two quads, column of the pass
    const uint32_t blk = (lane >> 2) % (16u / G);
    const uint32_t arow = lane & 3u, ahalf = (blk & 1u) * 16u, acol = G * (blk >> 1) + group;
    const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)m.vals, 0, (int)m.vals_bytes, 0x00020000);
    // The range of a source ends with the batch of its last column: a lane past the batch reads its neighbours (nothing is
    // made of them) or a zero, a column that a pass does not have is a zero and no traffic.
    const uint32_t xlane = (lane % F::lanes) * 4u;
    const uint32_t sj0 = uni_(X.sj0), sj1 = uni_(X.sj1), n0 = TWO ? uni_(X.n0) : m.cols;
    const uint64_t p0 = (uint64_t)(uintptr_t)(X.p0 + bt0), p1 = (uint64_t)(uintptr_t)(X.p1 + bt0);
    const uint32_t end0 = ((n0 - 1u) * sj0 + batch - bt0) * 4u, end1 = TWO ? ((m.cols - n0 - 1u) * sj1 + batch - bt0) * 4u : 0u;
    const uint8_t CSB_CONST_AS *rec = (const uint8_t CSB_CONST_AS *)(uintptr_t)m.recs + (size_t)first_record(m, list) * sizeof(QuadRec);
    auto read_loads = [&](int i) { return *(const uint32x8 CSB_CONST_AS *)(rec + i * (int)sizeof(QuadRec)); };
    auto read_slots = [&](int i) { return *(const uint32x8 CSB_CONST_AS *)(rec + i * (int)sizeof(QuadRec) + 32); };

    auto issue = [&](const uint32x8 &r, QuadOps<NT, G> &o) {         // 1 + NT * steps loads
        const uint32_t stride = r[1] & 0xffffu;
        const bool second = TWO && ((r[1] >> 24) & kQuadSecond) != 0u;
        uint32_t row = (second ? sj1 : sj0) * 4u;        // bytes from one column's right-hand sides to the next's
        asm("" : "+v"(row));                             // (in a vector register: then a column's offset is one instruction)
        const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)(second ? p1 : p0), 0, (int)(second ? end1 : end0), 0x00020000);
#pragma unroll
        for (int s = 0; s < F::steps; ++s) {
            uint32_t col;
            if constexpr (G == 1) {
                col = (s & 1) ? r[2 + s / 2] >> 16 : r[2 + s / 2] & 0xffffu;
            } else {
                col = group ? r[2 + s] >> 16 : r[2 + s] & 0xffffu;
            }
            const uint32_t off = mul24_(col, row) + xlane;
#pragma unroll
            for (int t = 0; t < NT; ++t) o.x[s][t] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)(off + 256u * t), 0, 0);
        }
        // (of quads a pass does not have: what lies there, and no use is made of it)
        typedef uint32_t vec4 __attribute__((ext_vector_type(4)));
        const vec4 a = __builtin_bit_cast(vec4, __builtin_amdgcn_raw_buffer_load_b128(vrsrc, (int)(mul24_(acol, stride) + mul24_(arow, stride >> 2) + ahalf + r[0]), 0, 0));
#pragma unroll
        for (int j = 0; j < 4; ++j) o.a[j] = a[j];
    };
    auto multiply = [&](const uint32_t w, const uint32x8 &slots, const QuadOps<NT, G> &o) {
        // the loads of the next pass may be in flight, this one's are here (one wait; left to itself the compiler
        // puts one in front of every product)
        constexpr int kYounger = 1 + NT * F::steps;
        __builtin_amdgcn_s_waitcnt((kYounger & 15) | (kYounger >> 4) << 14 | 0x0f70);
        const uint32_t quads = (w >> 16) & 0xffu;
        auto product = [&](auto qc, floatx4 (&D)[NT]) {
            constexpr int Q = decltype(qc)::value;
#pragma unroll
            for (int t = 0; t < NT; ++t) D[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
            quad_steps<0, F::steps / 2, Q>(o, D);
            if ((w >> 24) & kQuadWide) quad_steps<F::steps / 2, F::steps, Q>(o, D);
        };
        auto pair = [&](auto qc) {
            constexpr int Q = decltype(qc)::value;
            floatx4 D0[NT], D1[NT];
            product(qc, D0);
            if constexpr (NT > 1) add_rows(acc, D0, slots[Q]);            // (registers for one quad's results)
            if (Q + 1u < quads) product(std::integral_constant<int, Q + 1>{}, D1);   // (uniform)
            if constexpr (NT == 1) add_rows(acc, D0, slots[Q]);
            if (Q + 1u < quads) add_rows(acc, D1, slots[Q + 1]);
        };
        pair(std::integral_constant<int, 0>{});
        if (quads <= 2u) return;
        pair(std::integral_constant<int, 2>{});
        if (quads <= 4u) return;
        pair(std::integral_constant<int, 4>{});
        if (quads <= 6u) return;
        pair(std::integral_constant<int, 6>{});
    };
    // A pass's loads fly while the one before multiplies.  Scalar loads come back in any order, so that waiting for one is
    // waiting for all: they are asked for behind the only wait of a turn and used in the next one.
    QuadOps<NT, G> oa, ob;
    uint32x8 r = read_loads(0), sa = read_slots(0), sb;
    uint32_t left = list_length(m, list, r), wa = r[1], wb;
    if (left == 0u) return;
    issue(r, oa);
    r = read_loads(1);
    while (true) {
        issue(r, ob);
        wb = r[1];
        r = read_loads(2); sb = read_slots(1);
        multiply(wa, sa, oa);
        if (--left == 0u) break;
        issue(r, oa);
        wa = r[1];
        r = read_loads(3); sa = read_slots(2);
        multiply(wb, sb, ob);
        if (--left == 0u) break;
        rec += 2 * sizeof(QuadRec);
    }
}

// ---- 16-bit values times 16-bit right-hand sides (v_mfma_f32_4x4x4_16b) -----------------------------------------
// (Products run in panels, further down; these steps compute the tiles that an input which is not finite reaches.)
// An instruction takes four columns.  With NT = 2 a lane holds two neighbouring right-hand sides of an input row in one
// register; tile t holds the right-hand sides 2 n + t, its operand the halves t of four rows.
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
struct QuadOps16 {
    uint32_t a[4];                                       // registers 2 j and 2 j + 1: rows of the quads 4 j ... by 4 columns each
    uint32_t x[kQuadCols];                               // NT right-hand sides of a column
};

// One product: quad Q by the four columns S.
template <int S, int Q, int NT, bool HALF>
__device__ __forceinline__ void quad16_step(const QuadOps16 &o, const uint32_t (&b)[NT][2], floatx4 (&D)[NT]) {
    constexpr int cbsz = 4, abid = 4 * S + (Q & 3);
    const uint2 a = make_uint2(o.a[2 * (Q >> 2)], o.a[2 * (Q >> 2) + 1]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const uint2 x = make_uint2(b[t][0], b[t][1]);
        if constexpr (HALF) D[t] = __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(f16x4, a), __builtin_bit_cast(f16x4, x), D[t], cbsz, abid, 0);
        else D[t] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(bf16x4, a), __builtin_bit_cast(bf16x4, x), D[t], cbsz, abid, 0);
    }
}

// (X: the rows of 16-bit right-hand sides; its stride counts elements)
template <int NT, bool HALF>
__device__ __forceinline__ void quad16_passes(const QuadMat &m, const XSrc &X, const uint32_t list, const uint32_t bt0,
                                              const uint32_t batch, QuadAcc<NT> &acc) {
    constexpr int steps = 2;                             // of four columns
    const uint32_t lane = threadIdx.x & 63u;
    // the lane's place in an A register: row of a quad, which of four quads, which four columns (lanes 32 ... 63: as 0 ... 31)
    const uint32_t arow = ((lane >> 2 & 3u) * 4u + (lane & 3u)) * 16u + (lane >> 4 & 1u) * 8u;
    const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)m.vals, 0, (int)m.vals_bytes, 0x00020000);
    const uint32_t xlane = lane * 2u * NT;
    uint32_t row = uni_(X.sj0) * 2u;
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const uint16_t *)X.p0 + bt0), 0,
                                                                           (int)(((m.cols - 1u) * uni_(X.sj0) + batch - bt0) * 2u), 0x00020000);
    asm("" : "+v"(row));                                 // (in a vector register: then a column's offset is one instruction)
    uint32_t lo = 0x05040100u, hi = 0x07060302u;         // v_perm selectors: the low, the high halves of two registers
    asm("" : "+v"(lo), "+v"(hi));
    const uint8_t CSB_CONST_AS *rec = (const uint8_t CSB_CONST_AS *)(uintptr_t)m.recs + (size_t)first_record(m, list) * sizeof(QuadRec);
    auto read_loads = [&](int i) { return *(const uint32x8 CSB_CONST_AS *)(rec + i * (int)sizeof(QuadRec)); };
    auto read_slots = [&](int i) { return *(const uint32x8 CSB_CONST_AS *)(rec + i * (int)sizeof(QuadRec) + 32); };
    constexpr int kLoads = 2 + 4 * steps;                // of a pass

    auto issue = [&](const uint32x8 &r, QuadOps16 &o) {
        // (of rows that a pass does not have: what lies there, and no use is made of it; the second four columns are multiplied where
        // it has none, too: a branch around that is slower, 8192 x 8192 x 512 70.9 us instead of 66.7)
        const uint32_t at = arow + r[0] * 16u;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint2 a = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vrsrc, (int)(at + 256u * j), 0, 0));
            o.a[2 * j] = a.x; o.a[2 * j + 1] = a.y;
        }
        auto cols = [&](int i) { return (i & 1) ? r[2 + i / 2] >> 16 : r[2 + i / 2] & 0xffffu; };
#pragma unroll
        for (int i = 0; i < 4 * steps; ++i) {
            if constexpr (NT == 2) o.x[i] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)(mul24_(cols(i), row) + xlane), 0, 0);
            else o.x[i] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(xrsrc, (int)(mul24_(cols(i), row) + xlane), 0, 0);
        }
    };
    auto multiply = [&](const uint32_t w, const uint32x8 &slots, const QuadOps16 &o) {
        __builtin_amdgcn_s_waitcnt((kLoads & 15) | (kLoads >> 4) << 14 | 0x0f70);      // (see quad_passes)
        const uint32_t quads = (w >> 16) & 0xffu;
        uint32_t b[steps][NT][2];                        // [four columns][tile][words of two columns]
#pragma unroll
        for (int s = 0; s < steps; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                b[s][0][h] = __builtin_amdgcn_perm(o.x[4 * s + 2 * h + 1], o.x[4 * s + 2 * h], lo);
                if constexpr (NT == 2) b[s][1][h] = __builtin_amdgcn_perm(o.x[4 * s + 2 * h + 1], o.x[4 * s + 2 * h], hi);
            }
        auto quad = [&](auto qc) {
            constexpr int Q = decltype(qc)::value;
            floatx4 D[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) D[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
            quad16_step<0, Q, NT, HALF>(o, b[0], D);
            quad16_step<1, Q, NT, HALF>(o, b[1], D);
            add_rows(acc, D, slots[Q]);
        };
        quad(std::integral_constant<int, 0>{});
        if (quads <= 1u) return;
        quad(std::integral_constant<int, 1>{});
        if (quads <= 2u) return;
        quad(std::integral_constant<int, 2>{});
        if (quads <= 3u) return;
        quad(std::integral_constant<int, 3>{});
        if (quads <= 4u) return;
        quad(std::integral_constant<int, 4>{});
        if (quads <= 5u) return;
        quad(std::integral_constant<int, 5>{});
        if (quads <= 6u) return;
        quad(std::integral_constant<int, 6>{});
        if (quads <= 7u) return;
        quad(std::integral_constant<int, 7>{});
    };
    QuadOps16 oa, ob;
    uint32x8 r = read_loads(0), sa = read_slots(0), sb;
    uint32_t left = list_length(m, list, r), wa = r[1], wb;
    if (left == 0u) return;
    issue(r, oa);
    r = read_loads(1);
    while (true) {                                       // (as in quad_passes)
        issue(r, ob);
        wb = r[1];
        r = read_loads(2); sb = read_slots(1);
        multiply(wa, sa, oa);
        if (--left == 0u) break;
        issue(r, oa);
        wa = r[1];
        r = read_loads(3); sa = read_slots(2);
        multiply(wb, sb, ob);
        if (--left == 0u) break;
        rec += 2 * sizeof(QuadRec);
    }
}

// VF: format of the values and the right-hand sides.
template <int NT, int G, bool TWO, int NW, int VF = CSB_VAL_F32>
__device__ __forceinline__ void spmm_quad_body(const QuadMat &m, const XSrc &X, float *__restrict__ Y, const int64_t ldy, const uint32_t batch,
                                               const uint32_t tile, const uint32_t block_y) {
    extern __shared__ float4 smem4[];
    using F = QuadForm<NT, G>;
    constexpr uint32_t NTHR = NW * 64;
    const uint32_t wave = uni_(threadIdx.x >> 6);
    const uint32_t bt0 = block_y * F::columns;
    QuadAcc<NT> acc;
#pragma unroll
    for (int t = 0; t < NT; ++t) acc.v[t] = 0.0f;
    for (uint32_t k = 0; k < (uint32_t)(kQuadLists / NW); ++k) {
        const uint32_t list = tile * kQuadLists + wave * (kQuadLists / NW) + k;
        if constexpr (VF == CSB_VAL_F32) quad_passes<NT, G, TWO>(m, X, list, bt0, batch, acc);
        else quad16_passes<NT, VF == CSB_VAL_F16>(m, X, list, bt0, batch, acc);
    }

    // The wavefronts' tiles, RM rows at a time.  (The lane is asked for again: kept over the passes it is a register too many.)
    uint32_t lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    const uint32_t tid = wave * 64u + lane;
    constexpr int RM = NT == 2 ? 16 : 32;
    const uint32_t row0 = tile * m.tile_rows, tile_rows = min(m.tile_rows, m.rows - row0);
    float *red = (float *)smem4;                         // [waves][RM][NT][64]
#pragma unroll
    for (int r0 = 0; r0 < kQuadRows; r0 += RM) {
        if ((uint32_t)r0 >= tile_rows) break;            // (uniform)
        if (r0) __syncthreads();                         // the rows before are done with
#pragma unroll
        for (int i = 0; i < RM; ++i) {
            if (i == 16 && tile_rows <= 16u) break;      // (uniform)
#pragma unroll
            for (int t = 0; t < NT; ++t) red[((wave * RM + i) * NT + t) * 64u + lane] = acc.v[t][r0 + i];
        }
        __syncthreads();
        const uint32_t rows = min(tile_rows - r0, (uint32_t)RM);
        for (uint32_t e = tid; e < rows * F::columns; e += NTHR) {
            const uint32_t i = e / F::columns, n = e % F::columns;
            const uint32_t at = VF == CSB_VAL_F32 || NT == 1 ? n : n / 2u + 64u * (n & 1u);      // tile t: right-hand sides 64 t + lane, or 2 lane + t
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int g = 0; g < G; ++g) s += red[(w * RM + i) * (64u * NT) + g * F::lanes + at];
            if (bt0 + n < batch) Y[(size_t)(row0 + r0 + i) * ldy + bt0 + n] = s;
        }
    }
}

template <int NT, int G, bool TWO, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4))) void spmm_quad_kernel(const QuadMat m, const XSrc X, float *__restrict__ Y,
                                                                                              const int64_t ldy, const uint32_t batch) {
    spmm_quad_body<NT, G, TWO, NW>(m, X, Y, ldy, batch, blockIdx.x, blockIdx.y);
}
// Several independent products in one launch (blockIdx.z picks the product).
template <int NT, int G, bool TWO, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4))) void spmm_quad_multi_kernel(const QuadJobs J, const uint32_t batch) {
    const uint32_t j = blockIdx.z;
    if (blockIdx.x >= J.m[j].n_tiles) return;            // the grid is as wide as the widest product
    spmm_quad_body<NT, G, TWO, NW>(J.m[j], J.X[j], J.Y[j], J.ldy[j], batch, blockIdx.x, blockIdx.y);
}

// ---- 16-bit operands in panels -------------------------------------------------------------------------------------
// v_mfma_f32_16x16x32 multiplies 16 rows by 32 columns of 16 right-hand sides four times as fast per multiply-add as the 4 x 4
// forms, so that rows may stay where they are in the tile and be zero where a pass lacks them: four passes (a list for
// every 16 lanes) are a panel of 32 columns, nothing is added row by row, and a wavefront's sums are the accumulators of
// its instructions.  A lane is row i of 16 and takes the eight values of its row from a pass, found by counting the rows in front
// of it in the record's mask (a row that the pass lacks reads past the end: zeros), and of each of the pass's eight columns 8
// neighbouring right-hand sides, or twice 2; v_perm puts columns side by side.  The record comes in as a word per lane and is handed
// round by DPP.
// What bounds it: the loads' way through the L1: with the products left out a launch is as long, from 16 rows of X that always hit it is no
// shorter (measured).  A load of 4 bytes per lane takes it about 4 clocks, of 8 bytes 12, of 16 bytes 13: lanes take 16 where there are
// 128 right-hand sides, else 4 twice; with 8 bytes 8192 x 8192 at 12x, bfloat16, took 66 us instead of 44 at 512 right-hand sides, 12.8
// instead of 10.6 at 64.  Four-row steps / panels, us, launches replayed back to back: x 512 72.7 / 44.9 (a call among others 63.8 / 42), x 128
// 21.9 / 14.4, x 64 17.5 / 10.5, x 8 17.5 / 9.9; 4096 x 4096 in 16-row blocks x 256 22.6 / 15.5; 1024 x 665 at 8x x 32 4.4 / 3.8.  Error
// against 64 bits, of the norm, four-row steps / panels: x 512 0.749e-7 / 0.693e-7, x 128 0.845e-7 / 0.692e-7, binary16 x 512 0.979e-7 /
// 0.876e-7; 4096 x 4096 in 16-row blocks at 12x x 256 0.661e-7 / 0.598e-7.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Value of lane N of the own 16 lanes.
template <int N>
__device__ __forceinline__ uint32_t row_lane(const uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + N, 0xf, 0xf, false); }

// H: tile of 16 H rows; NC: right-hand sides of a lane (4, as two and two, or 8), 16 NC of a workgroup; S: wavefronts that share a list.
template <int H, int NC>
struct PanelOps {
    uint32_t x[kQuadCols][NC / 2];                       // right-hand sides of each column of the lane's pass, two to a word
    uint4 a[H];                                          // its columns of a row
};

// The passes `part`, part + S, ... of four lists of a tile, one list for every 16 lanes; col0: the lane's first right-hand side.
template <int H, int NC, int S, int VF>
__device__ __forceinline__ void panel_passes(const QuadMat &m, const uint16_t *X, const uint32_t ldx, const uint32_t batch, const uint32_t tile,
                                             const uint32_t col0, const uint32_t wave, floatx4 (&acc)[H][NC]) {
    const uint32_t lane = threadIdx.x & 63u, i = lane & 15u, part = wave >> 2;
    const uint32_t list0 = tile * kQuadLists, list = list0 + (wave & 3u) * 4u + (lane >> 4);
    const uint32_t first0 = m.list_stride ? list0 * m.list_stride : m.table[list0], first = m.list_stride ? list * m.list_stride : m.table[list];
    const uint32_t len = m.list_stride ? ((const QuadRec *)m.recs)[first].list_len : m.table[list + 1] - first;
    const uint32_t longest = max(max(__builtin_amdgcn_readlane(len, 0), __builtin_amdgcn_readlane(len, 16)),
                                 max(__builtin_amdgcn_readlane(len, 32), __builtin_amdgcn_readlane(len, 48)));
    // (from the tile's first record on: those of a matrix may lie further apart than an offset reaches, those of a tile do not)
    const __amdgpu_buffer_rsrc_t rrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const QuadRec *)m.recs + first0), 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)m.vals, 0, (int)m.vals_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)(((m.cols - 1u) * ldx + batch) * 2u), 0x00020000);
    // a record's eight words come in by eight lanes
    const uint32_t word = i & 7u, rec0 = (first - first0) * (uint32_t)sizeof(QuadRec) + word * 4u;
    const uint32_t none = word >= 2u && word < 6u ? 0xffffffffu : 0u;     // a record of no columns and no rows
    uint32_t row = ldx * 2u, xlane = col0 * 2u;          // (bytes from one column's right-hand sides to the next's: 16 bits)
    asm("" : "+v"(row), "+v"(xlane));
    uint32_t lo = 0x05040100u, hi = 0x07060302u;         // v_perm selectors: the low, the high halves of two registers
    asm("" : "+s"(lo), "+s"(hi));
    auto records = [&](const uint32_t j) {
        return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rrsrc, (int)(j < len ? rec0 + j * (uint32_t)sizeof(QuadRec) : 0x80000000u), 0, 0);
    };
    auto issue = [&](const uint32_t w, PanelOps<H, NC> &o) {
        const uint32_t val = row_lane<0>(w), rows = row_lane<7>(w);
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const uint32_t place = 16u * h + i, q = __popc(rows & ((1u << place) - 1u)) + val;       // the row's place among the pass's
            const uint32_t lacks = ~rows << (31u - place) & 0x80000000u;                            // (past the end of the values: zeros)
            o.a[h] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(vrsrc, (int)(q << 4 | lacks), 0, 0));
        }
        const uint32_t cols[4] = {row_lane<2>(w), row_lane<3>(w), row_lane<4>(w), row_lane<5>(w)};
#pragma unroll
        for (int e = 0; e < kQuadCols; ++e) {
            uint32_t at;                                 // column times row + the lane's place
            if (e & 1) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(at) : "v"(cols[e / 2]), "v"(row), "v"(xlane));
            else asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(at) : "v"(cols[e / 2]), "v"(row), "v"(xlane));
            if constexpr (NC == 8) {
                const uint4 v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (int)at, 0, 0));
                o.x[e][0] = v.x; o.x[e][1] = v.y; o.x[e][2] = v.z; o.x[e][3] = v.w;
            } else {
                o.x[e][0] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)at, 0, 0);
                o.x[e][1] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)(at + 64u), 0, 0);
            }
        }
    };
    auto multiply = [&](const PanelOps<H, NC> &o) {
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            auto pair = [&](int e) { return __builtin_amdgcn_perm(o.x[e + 1][n / 2], o.x[e][n / 2], n & 1 ? hi : lo); };
            const uint4 b = make_uint4(pair(0), pair(2), pair(4), pair(6));
#pragma unroll
            for (int h = 0; h < H; ++h) {
                if constexpr (VF == CSB_VAL_F16) acc[h][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, o.a[h]), __builtin_bit_cast(f16x8, b), acc[h][n], 0, 0, 0);
                else acc[h][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, o.a[h]), __builtin_bit_cast(bf16x8, b), acc[h][n], 0, 0, 0);
            }
        }
    };
    if (part >= longest) return;
    auto valid = [&](const uint32_t at, const uint32_t w) { return at < len ? w : none; };
    // A pass's loads fly while the one before multiplies; its record was asked for in front of those.  (One way out of the loop:
    // with another in its middle the compiler keeps the sums twice and moves loads behind it.)
    // (In front of the products, where there are registers for both; with 32 rows, 128 right-hand sides and eight wavefronts, 16 on a CU
    // are worth more: x 512 52 -> 44 us, x 256 26 -> 24, x 128 13.8 -> 13.9.)
    constexpr bool kEarly = H * NC < 16 || S == 1;
    PanelOps<H, NC> oa, ob;
    uint32_t j = part, w = valid(j, records(j)), w1 = records(j + S);
    issue(w, oa);
    while (j + S < longest) {
        w = records(j + 2 * S);
        __builtin_amdgcn_sched_barrier(0);
        issue(valid(j + S, w1), ob);
        if constexpr (kEarly) __builtin_amdgcn_sched_barrier(0);
        multiply(oa);
        w1 = records(j + 3 * S);
        __builtin_amdgcn_sched_barrier(0);
        issue(valid(j + 2 * S, w), oa);
        if constexpr (kEarly) __builtin_amdgcn_sched_barrier(0);
        multiply(ob);
        j += 2 * S;
    }
    if (j < longest) multiply(oa);
}

template <int H, int NC, int S, int VF>
__global__ __launch_bounds__(256 * S) __attribute__((amdgpu_waves_per_eu(H * NC == 16 && S == 1 ? 3 : 4))) void spmm_panel16_kernel(
    const QuadMat m, const uint16_t *__restrict__ X, const uint32_t ldx, float *__restrict__ Y, const int64_t ldy, const uint32_t batch) {
    extern __shared__ float4 smem4[];
    constexpr int NW = 4 * S;
    constexpr uint32_t N = 16 * NC;
    const uint32_t groups = (batch + N - 1u) / N, tile = blockIdx.x / groups, group = blockIdx.x - tile * groups, bt0 = group * N;
    const uint32_t wave = uni_(threadIdx.x >> 6);
    // a lane's right-hand sides: two and the two 32 further on, or eight; the last four of a batch come with the four before them
    auto first_of = [&](const uint32_t ln) { return bt0 + (NC == 4 ? 2u : 8u) * (ln & 15u); };
    auto from = [&](const uint32_t own) { return NC == 8 && own + 4u == batch ? own - 4u : own; };
    floatx4 acc[H][NC];
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
        for (int n = 0; n < NC; ++n) acc[h][n] = 0.0f;
    panel_passes<H, NC, S, VF>(m, X, ldx, batch, tile, from(first_of(threadIdx.x)), wave, acc);
    uint32_t lane;                                       // (asked for again: kept over the passes it is a register too many)
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    const uint32_t own = first_of(lane), col0 = from(own);
    // the wavefronts' sums, 16 rows at a time: [wave][row of four][four right-hand sides][lane]
    const uint32_t row0 = tile * m.tile_rows;
    bool odd = false;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        if (h) __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < NC / 4; ++c)
                smem4[((wave * 4u + r) * (NC / 4) + c) * 64u + lane] = make_float4(acc[h][4 * c][r], acc[h][4 * c + 1][r], acc[h][4 * c + 2][r], acc[h][4 * c + 3][r]);
        __syncthreads();
        for (uint32_t k = wave; k < (uint32_t)NC; k += NW) {
            // (four and four in a row, then those: nearer to 64 bits than all in a row)
            auto four = [&](const int w0) {
                float4 v = smem4[((uint32_t)w0 * NC + k) * 64u + lane];
#pragma unroll
                for (int w = w0 + 1; w < w0 + 4; ++w) {
                    const float4 p = smem4[((uint32_t)w * NC + k) * 64u + lane];
                    v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
                }
                return v;
            };
            float4 s = four(0);
            if constexpr (NW == 8) {
                asm volatile("" : "+v"(s.x), "+v"(s.y), "+v"(s.z), "+v"(s.w));      // (not the registers for all eight)
                const float4 v = four(4);
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            }
            const uint32_t row = row0 + 16u * h + 4u * (lane >> 4) + k / (NC / 4);
            auto store = [&](const uint32_t n, const float v0, const float v1) {      // (batches are even, and so is n)
                if (row >= m.rows || n < own || n >= batch) return;
                odd = odd || !(fabsf(v0) < INFINITY && fabsf(v1) < INFINITY);
                float *y = Y + (size_t)row * ldy + n;
                y[0] = v0; y[1] = v1;
            };
            if constexpr (NC == 4) {
                store(col0, s.x, s.y);
                store(col0 + 32u, s.z, s.w);
            } else if (const uint32_t n = col0 + 4u * (k % (NC / 4)); row < m.rows && n >= own && n < batch) {
                odd = odd || !(fabsf(s.x) < INFINITY && fabsf(s.y) < INFINITY && fabsf(s.z) < INFINITY && fabsf(s.w) < INFINITY);
                float *y = Y + (size_t)row * ldy + n;
                y[0] = s.x; y[1] = s.y; y[2] = s.z; y[3] = s.w;
            }
        }
    }
    // Rows that a pass does not have were multiplied by zeros, which an infinite or undefined input makes NaN of: such a
    // tile is computed again in steps of the rows there are, of 128 right-hand sides only the 64 that need it.  8192 x 8192 at 12x, us, all finite /
    // an infinite input that 682 rows use / nothing but NaN: x 512 48 / 82 / 109 (110 and 158 with all by 64 and 64), x 128 14.5 / 36 / 41 (53 and 62),
    // x 64 10.7 / 28 / 30.  (Four-row steps alone: 71, 21.7, 17.9 whatever the inputs.)
    if (!__syncthreads_or(odd)) return;
    const XSrc src{(const float *)X, m.cols, ldx, (const float *)X, ldx};
    if constexpr (NC == 4) {
        spmm_quad_body<1, 1, false, NW, VF>(m, src, Y, ldy, batch, tile, group);
    } else {
        const bool odd0 = __syncthreads_or(odd && (lane & 8u) == 0u), odd1 = __syncthreads_or(odd && (lane & 8u) != 0u);
        if (odd0 && odd1) spmm_quad_body<2, 1, false, NW, VF>(m, src, Y, ldy, batch, tile, group);
        else spmm_quad_body<1, 1, false, NW, VF>(m, src, Y, ldy, batch, tile, group * 2u + (odd1 ? 1u : 0u));
    }
}

// ---- launches ------------------------------------------------------------------------------------------------
QuadMat quad_mat(const csb_matrix *m, bool low) {
    const QuadPlan &qp = low && m->plan.quad_low.valid ? m->plan.quad_low : m->plan.quad;
    uint8_t *b = (uint8_t *)m->d_buf;
    return QuadMat{(const uint32_t *)(b + qp.off_table), b + qp.off_recs, b + qp.off_vals, (uint32_t)qp.vals_bytes, qp.n_tiles, qp.tile_rows, qp.rows,
                   (uint32_t)m->plan.hdr.cols, qp.list_stride};
}

// ---- the launch's shape, by an estimate of its time --------------------------------------------------------------
// What counts is the number of turns the workgroups take over the 256 CUs and how long a turn is: of 16 wavefronts a CU holds
// one workgroup; of 8, two, which overlap one's merge with the other's products but leave the last turn half empty (`one`: a
// turn of up to 256 of those, `two`: of up to 512).  A turn takes the merge of the wavefronts' tiles and what the passes of a
// list take.  Lists are as long as the matrix makes them, so that no line between the forms lies at one size: the constants
// (us per pass, step and row of a list) are fitted to 400 matrices of 256 x 128 to
// 40000 x 8192 in blocks of 4 to 128, pruned 1 to 25 times by three laws, at 2 to 512 right-hand sides in every form of
// both sections: half of the estimates are within 3 % and nine of ten within 10; on matrices that were not fitted the form
// taken is 0.5 % off the best one on average and 3.5 at the 95th percentile.  (With one length of a turn for all
// matrices, that of 8192 x 8192 at 12x, and never the tile-based sections: 2.9 and 19.)
// us on 8192 x 8192 at 12x, 256 tiles, 512 right-hand sides: 128 columns by 16 wavefronts 128, by 8 115.  32-row / 16-row tiles: 2048 x
// 2048 x 64 in 32-row blocks 7.4 / 6.0, 4096 x 2048 x 128 in 64-row blocks 6.3 / 6.8.
struct QuadTurn { double merge, pass, step, row; };
struct QuadCost {
    int columns, nw;
    double base, out;                                    // out: per million output words
    QuadTurn one, two;
};
static const QuadCost kQuadCost[] = {
    {32, 16, 2.23, 2.91, {1.34, 0.333, 0.00412, 0.026}, {}},
    {64, 16, 2.24, 2.11, {1.16, 0.351, 0.00845, 0.0321}, {}},
    {128, 16, 2.1, 1.3, {2.76, 0.44, 0.014, 0.0428}, {}},
    {128, 8, 2.73, 0.95, {1.63, 0.512, 0.0186, 0.0363}, {1.57, 0.84, 0.0287, 0.0691}},
};
static double quad_us(const QuadCost &f, const QuadWork &w, double tiles, double mean_rows, double out_words, int32_t batch) {
    const double wgs = tiles * ((batch + f.columns - 1) / f.columns), slots = f.nw == 8 ? 512 : 256;
    const double full = (double)(uint64_t)(wgs / slots), rest = wgs - full * slots;
    double one = full + (rest > 0 ? 1 : 0), two = 0;
    if (f.nw == 8) { two = full + (rest > 256 ? 1 : 0); one = rest > 0 && rest <= 256 ? 1 : 0; }
    const double lists = tiles * kQuadLists, longest = 1 + (w.uneven - 1) / std::max(one + two, 1.0);      // (one turn is as long as its longest list)
    auto turn = [&](const QuadTurn &t) {
        return t.merge * mean_rows / kQuadRows + longest * (t.pass * w.passes + t.step * w.steps + t.row * w.rows) / lists;
    };
    return f.base + f.out * out_words * 1e-6 + one * turn(f.one) + two * turn(f.two);
}

QuadShape quad_shape(const csb_matrix *const *mats, int n, int32_t batch) {
    QuadShape best{};
    best.us = 1e300;
    bool any_low = false;
    for (int i = 0; i < n; ++i) any_low = any_low || mats[i]->plan.quad_low.valid;
    for (int low = 0; low < (any_low ? 2 : 1); ++low) {
        QuadWork sum{};
        double tiles = 0, rows = 0, out_rows = 0;
        unsigned most_tiles = 0;
        for (int i = 0; i < n; ++i) {
            const Plan &pl = mats[i]->plan;
            const QuadPlan &qp = low && pl.quad_low.valid ? pl.quad_low : pl.quad;
            sum.passes += qp.work.passes; sum.rows += qp.work.rows; sum.steps += qp.work.steps;
            sum.uneven = std::max(sum.uneven, qp.work.uneven);
            tiles += qp.n_tiles; rows += (double)qp.n_tiles * qp.tile_rows; out_rows += qp.rows;
            most_tiles = std::max(most_tiles, (unsigned)qp.n_tiles);
        }
        for (const QuadCost &f : kQuadCost) {
            const double us = quad_us(f, sum, tiles, rows / tiles, out_rows * batch, batch);
            if (us < best.us)
                best = QuadShape{f.columns, f.nw, low != 0, (size_t)f.nw * kQuadRows * 64 * sizeof(float), most_tiles,
                                 (unsigned)((batch + f.columns - 1) / f.columns), us};
        }
    }
    return best;
}

bool quad_source(const SpmmCall &c, XSrc *X, bool *two) {
    const QuadPlan &qp = c.mat->plan.quad;
    const uint64_t cols = c.mat->plan.hdr.cols;
    if (!qp.valid || qp.val_fmt != CSB_VAL_F32 || c.mat->batch_form == kFormTiles) return false;
    // a pass takes its columns from one source: two sources need a plan that was cut where they meet; one source
    // under such a plan is two that follow each other
    const bool two_given = c.n0 < (uint32_t)cols;
    *two = qp.split_col > 0 && qp.split_col < cols;
    if (two_given && (!*two || qp.split_col != c.n0)) return false;
    *X = two_given || !*two ? XSrc{c.p0, c.n0, (uint32_t)c.sj0, c.p1, (uint32_t)c.sj1}
                            : XSrc{c.p0, qp.split_col, (uint32_t)c.sj0, c.p0 + (size_t)qp.split_col * c.sj0, (uint32_t)c.sj0};
    // 32-bit byte offsets, that of kQuadNoCol among them
    return X->sj0 <= kQuadMaxStride && X->sj1 <= kQuadMaxStride;
}

bool quad16_source(const csb_matrix *mat, int64_t ldx) {
    const QuadPlan &qp = mat->plan.quad;
    return qp.valid && qp.val_fmt != CSB_VAL_F32 && qp.split_col == 0 && ldx <= kQuadMaxStride && mat->batch_form != kFormTiles;
}

const void *quad_kernel(const QuadShape &sh, bool two, bool multi) {
#define CSB_Q(NT, G, TWO, NW) (multi ? (const void *)spmm_quad_multi_kernel<NT, G, TWO, NW> : (const void *)spmm_quad_kernel<NT, G, TWO, NW>)
#define CSB_QV(NT, G, NW) return two ? CSB_Q(NT, G, true, NW) : CSB_Q(NT, G, false, NW);
    if (sh.columns == 128) {
        if (sh.nw == 8) { CSB_QV(2, 1, 8) }
        CSB_QV(2, 1, 16)
    }
    if (sh.columns == 64) { CSB_QV(1, 1, 16) }
    CSB_QV(1, 2, 16)
#undef CSB_QV
#undef CSB_Q
}

// The shape of a launch of panels, by an estimate of its time: a CU works off its workgroups at a rate that depends on little but
// the panels (`panel`: us for the passes that four wavefronts take at once), however many of them it holds.  Fitted to 1573
// launches in every form (260 to 20000 rows, 128 to 8192 columns, blocks of 4 to 64, pruned 1 to 25 times by three laws, 4 to 512
// right-hand sides): half of the estimates are within 4 %.  Over 2086 others the form taken is 0.9 % off the best one on average and 5 at
// the 95th percentile; it is furthest off beyond 256 tiles and between 64 and 128 right-hand sides, where 64 columns take twice the workgroups
// (8342 x 7541 unpruned x 72 64.5 us, 128 columns 48.3; 10856 x 6632 unpruned x 84 63.2 and 46.4).  Against the older forms, four-row steps and
// tile-based sections as the estimate chose between them, panels took 0.73 of the time on average over 4215 such launches, and the worst
// 1.07 of it (9880 x 3359 unpruned x 100: 50.9 / 54.6 us); a dozen others, of at most 330 columns, lost up to 0.1 us of 3.3 to 4.1.
// Four wavefronts where a list has at most 16 passes; longer sums in one accumulator are further off 64 bits than the halves of two: error against 64 bits, of
// the norm, 8192 x 8192 in 16-row blocks at 8x, by 4 and by 8 wavefronts 0.96e-7 and 0.78e-7 (four-row steps 0.83e-7).
struct PanelCost { int rows, columns, share; double base, out, merge, panel; };      // out: per million output words (four forms of 16 rows, four of 32)
static const PanelCost kPanelCost[] = {
    {16, 64, 1, 3.26, 0.748, 0, 0.239},     {16, 64, 2, 3.13, 2.34, 0, 0.195},     {16, 128, 1, 3.69, 1.40, 0.069, 0.289},
    {16, 128, 2, 3.50, 1.91, 0.006, 0.283}, {32, 64, 1, 3.66, 1.20, 0, 0.249},     {32, 64, 2, 3.40, 1.79, 0.301, 0.227},
    {32, 128, 1, 4.34, 1.16, 0.343, 0.330}, {32, 128, 2, 3.98, 1.39, 0.572, 0.348},
};
PanelShape panel_shape(const csb_matrix *m, int32_t batch) {
    PanelShape best{};
    double best_us = 1e300;
    // (a small call's kernel is done in 3 us: what is the same for several forms is worked out once)
    for (int low = 0; low < (m->plan.quad_low.valid ? 2 : 1); ++low) {
        const QuadPlan &qp = low ? m->plan.quad_low : m->plan.quad;
        const double passes = qp.work.passes / ((double)qp.n_tiles * kQuadLists), out = (double)qp.rows * batch * 1e-6;
        const uint64_t wgs64 = (uint64_t)qp.n_tiles * (((uint32_t)batch + 63u) >> 6), wgs128 = (uint64_t)qp.n_tiles * (((uint32_t)batch + 127u) >> 7);
        const double turns64 = (double)((wgs64 + 255) >> 8), turns128 = (double)((wgs128 + 255) >> 8);
        const PanelCost *forms = kPanelCost + (qp.tile_rows == 16 ? 0 : 4);
        for (const PanelCost *f = forms; f < forms + 4; ++f) {
            if ((f->columns == 128 && batch < 8) || (f->share == 1 && passes > 16)) continue;     // (128: a lane has eight right-hand sides)
            const double us = f->base + f->out * out + (f->columns == 128 ? turns128 : turns64) * (f->merge + (passes + 0.5 * f->share) * f->panel);
            if (us < best_us) {
                best_us = us;
                best = PanelShape{f->rows, f->columns, f->share, low != 0, (size_t)4 * f->share * kQuadRows * 64 * sizeof(float),
                                  (unsigned)(f->columns == 128 ? wgs128 : wgs64), batch};
            }
        }
    }
    // a grid's row has fewer than 2^32 threads (65536 tiles by 512 threads by 128 workgroups a tile are as many)
    const uint64_t tiles = (best.low ? m->plan.quad_low : m->plan.quad).n_tiles, groups = std::max<uint64_t>(0xffffffffull / (256u * best.share) / tiles, 1);
    if (groups * best.columns < (uint64_t)batch) { best.batch = (int32_t)(groups * best.columns); best.workgroups = (unsigned)(groups * tiles); }
    return best;
}

const void *panel16_kernel(const PanelShape &ps, bool half) {
#define CSB_P16(H, NC, S) (half ? (const void *)spmm_panel16_kernel<H, NC, S, CSB_VAL_F16> : (const void *)spmm_panel16_kernel<H, NC, S, CSB_VAL_BF16>)
#define CSB_P16S(H, NC) (ps.share == 2 ? CSB_P16(H, NC, 2) : CSB_P16(H, NC, 1))
    if (ps.rows == 16) return ps.columns == 128 ? CSB_P16S(1, 8) : CSB_P16S(1, 4);
    return ps.columns == 128 ? CSB_P16S(2, 8) : CSB_P16S(2, 4);
#undef CSB_P16S
#undef CSB_P16
}

}  // namespace csb
