// Batched CSB-MVM for gfx950: Y = A X with fp32 MFMA.
//
// With B right-hand sides a kernel matrix K_b (r x c) meets a gathered c x B slab of X: a
// real dense product, so it goes to the matrix cores (v_mfma_f32_16x16x4_f32).  One
// workgroup owns one output row tile and one batch tile.  The tile's records
// (virtual blocks, lane descriptors, input-offset lists) are staged in LDS one segment at a
// time; the wavefronts take the segment's virtual blocks round-robin, each as 16-row
// slices: per 4 columns one A operand (16 x 4 of the kernel) feeds one MFMA per 16 batch
// columns.
// The 16 x 16 results are added at the block's row indices into a per-wavefront
// accumulator tile in LDS (the role of NeuronAccumBuffer, Sec. 4.3.1); the wavefronts'
// tiles are summed in wavefront order, so the result does not depend on timing.  The
// paper's engine is batch 1 only; this is the batched extension the matrix cores make
// worthwhile.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "csb_internal.hpp"
#include "csb_kernels.hpp"
#include "csb_spmm.hpp"
#include "csbrnn_debug.h"

namespace csb {

// NT neighbouring right-hand sides (a load of NT words, aligned to one word).
template <int NT> struct RhsVec;
template <> struct RhsVec<1> { typedef float type __attribute__((ext_vector_type(1))); };
template <> struct RhsVec<2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct RhsVec<4> { typedef float type __attribute__((ext_vector_type(4))); };

// One pass: up to 4 KS columns (KS MFMA k-steps) of one 16-row slice of one virtual block.
struct Pass {
    uint32_t k;           // virtual block, counted inside the segment
    uint32_t m0, kc;      // first row of the slice, first column of the pass
    uint32_t r, c, lane0; // the block's rows, columns, first lane
    uint32_t val_off;     // the group's values
    uint32_t desc;        // LDS byte offset of the group's lane descriptors
    uint32_t list;        // LDS byte offset of the block's input-offset list
    bool valid;
};

template <int NT, int KS>
struct Operands {                            // of up to KS k-steps of 4 columns each
    uint32_t av[KS];                         // kernel values as stored
    typename RhsVec<NT>::type bv[KS];        // NT right-hand sides of the lane's column
};

// What bounds it: instructions and load issue, not the matrix cores.  The products of a pruned gate matrix are
// tiny (13 x 13 kernels out of 64 x 64 blocks, 7 x 7 out of 32 x 32), so a pass is written to cost little: a lane
// reads its NT neighbouring right-hand sides with one load (tile t of the MFMA holds the right-hand sides
// NT n + t; the loads are aligned to a word, and lanes past the batch are moved back to its last NT right-hand
// sides, so any batch and stride will do), rows and columns a block lacks repeat its last ones instead of being
// branched around, operands are masked in a block's last, partial k-step only, and rows a slice lacks go
// to a spare row of the accumulator instead of being predicated.  K-steps a block lacks are not loaded, though:
// their loads cost as much as those of the ones it has, and 16 wavefronts per workgroup hide what
// conservative waits at the branches cost.  The 8 of the 64-column form on tall tiles (NT = 4) do not: there a pass
// always issues the same loads and the waits are counted (8192 x 8192 in 64 x 64 blocks at batch 256: 111 -> 102 us).
// The room of a pass is 32 columns (16 at NT = 4, whose operands take the registers, and where blocks are no
// wider): with 16, fuller blocks need another pass.  Nothing is loaded past a wavefront's last pass.
// Measured on 8192 x 2048 at batch 16 / 3000 x 3000 in 64 x 64 blocks at batch 64 / two LSTM layers of 1024 at
// batch 64, us: 8.8 / 15.1 / 14.5; four k-steps always loaded, two passes ahead, 16 columns: 10.8 / 17.1 / 15.6;
// branches per k-step, value format and slice, masked operands throughout: 8.9 / 15.6 / 17.7.
template <int NT, bool TWO, int NW, int KS>
__device__ __forceinline__ void spmm_body(const DevMat &m, const XSrc &X, float *__restrict__ Y, const int64_t ldy,
                                          const uint32_t batch, const uint32_t block_x, const uint32_t block_y) {
    extern __shared__ float4 smem4[];
    typedef typename RhsVec<NT>::type vec;
    typedef vec vec_u __attribute__((aligned(4)));
    constexpr uint32_t NB = 16 * NT;               // batch columns per workgroup
    constexpr uint32_t PC = 4 * KS;                // columns per pass
    constexpr bool kCounted = NT == 4 && NW == 8;  // every pass issues the same loads
    constexpr uint32_t NTHR = NW * 64;             // NW wavefronts
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uni_(tid >> 6);
    const uint32_t bt0 = block_y * NB;
    const uint32_t br = m.br;
    if (block_x >= m.n_nz_tiles) {                 // a row tile without work: zeros
        const uint32_t tile = m.zero_tiles[block_x - m.n_nz_tiles];
        for (uint32_t e = tid; e < br * NB; e += NTHR) {
            const uint32_t row = tile * br + e / NB, n = bt0 + e % NB;
            if (row < m.rows_out && n < batch) Y[(size_t)row * ldy + n] = 0.0f;
        }
        return;
    }
    uint8_t *meta = (uint8_t *)smem4;                              // one record segment
    float *acc = (float *)(meta + m.seg_meta);                     // [waves][br + 1][NB], the last row a spare one
    const uint32_t acc_wave = (br + 1u) * NB;
    float *myacc = acc + (size_t)wave * acc_wave;
    for (uint32_t e = lane; e < acc_wave / 4u; e += 64) ((float4 *)myacc)[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const uint32_t rank = block_x, tile = m.nz_tiles[rank];
    const uint32_t vf = uni_(m.val_fmt);                           // storage format of the value stream
    const uint32_t mrow = lane & 15u, kq = lane >> 4;              // A: row, column-in-4; B: right-hand sides, column-in-4
    const uint32_t nstart = min(bt0 + NT * mrow, batch - NT);      // this lane's first right-hand side (batch >= NT)
    const uint32_t split4 = 4u * X.n0, sj0 = uni_(X.sj0), sj1 = uni_(X.sj1);   // (see uni_)
    const uint8_t *const x0 = (const uint8_t *)(X.p0 + nstart);
    const uint8_t *const x1 = (const uint8_t *)(X.p1 + nstart) - (size_t)split4 * sj1;

    const uint32_t sg0 = first_segment(m, rank), sg1 = first_segment(m, rank + 1u);
    for (uint32_t sg = sg0; sg < sg1; ++sg) {
        // ---- stage the segment's records ------------------------------------------------
        const SegRec *sp = m.segs + sg;
        const uint32_t vb0 = sp->vb0, nvbs = sp->nvbs, idx0 = sp->idx0, idx_bytes = sp->idx_bytes;
        const uint32_t ioff = nvbs * (uint32_t)sizeof(VbRec);
        __syncthreads();                                           // the previous segment is done with
        {
            const float4 *vs = (const float4 *)(m.vbs + vb0);
            float4 *vd = (float4 *)meta;
            for (uint32_t i = tid; i < nvbs; i += NTHR) vd[i] = vs[i];
            const float4 *is = (const float4 *)(m.idx + idx0);
            float4 *id = (float4 *)(meta + ioff);
            for (uint32_t i = tid; i < idx_bytes >> 4; i += NTHR) id[i] = is[i];
        }
        __syncthreads();
        if (wave >= nvbs) continue;                                // (uniform per wavefront; the barriers above are passed by all)

        // ---- passes of this wavefront's virtual blocks ----------------------------------
        auto open_vb = [&](uint32_t k, Pass &p) {
            const uint4 v = *(const uint4 *)(meta + k * (uint32_t)sizeof(VbRec));
            const uint32_t v0 = uni_(v.x);
            p.k = k;
            p.r = v0 & 0xffu; p.lane0 = (v0 >> 8) & 0xffu; p.c = v0 >> 16;
            p.val_off = uni_(v.y);
            p.desc = ioff + (uni_(v.z) - idx0);
            p.list = ioff + (uni_(v.w) - idx0);
        };
        // The pass after p; past the wavefront's last one only `valid` means anything.
        auto next_pass = [&](const Pass &p) -> Pass {
            const bool cols = p.kc + PC < p.c, rows = p.m0 + 16u < p.r, more = p.k + NW < nvbs;
            Pass q;
            open_vb(cols || rows || !more ? p.k : p.k + NW, q);
            q.valid = cols || rows || more;
            q.kc = cols ? p.kc + PC : 0u;
            q.m0 = cols ? p.m0 : rows ? p.m0 + 16u : 0u;
            return q;
        };
        // The loads of the k-steps the block has; those of the first two (kCounted: of all) are issued in any
        // case.  Rows and columns the block lacks repeat its last ones.
        auto load_pass = [&](const Pass &p) -> Operands<NT, KS> {
            Operands<NT, KS> o;                                        // (k-steps the block lacks stay undefined and unused)
            const uint32_t *gv = (const uint32_t *)m.vals + (vf == CSB_VAL_F32 ? p.val_off : p.val_off >> 1);
            const uint32_t arow = p.lane0 + min(p.m0 + mrow, p.r - 1u);
            const uint32_t half = vf == CSB_VAL_F32 ? 0u : 1u;     // 16-bit: a word per lane and PAIR of columns
            uint32_t jc[KS], cb[KS];
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                jc[s] = min(p.kc + 4u * s + kq, p.c - 1u);
                cb[s] = *(const uint16_t *)(meta + p.list + 2u * jc[s]);                   // 4 * column
            }
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (s >= (kCounted ? KS : 2) && p.kc + 4u * s >= p.c) break;         // (uniform)
                o.av[s] = gv[(jc[s] >> half) * (uint32_t)kWave + arow];
                const bool first = !TWO || cb[s] < split4;
                const uint8_t *src = (first ? x0 : x1) + (size_t)mul24_(cb[s], first ? sj0 : sj1);
                o.bv[s] = *(const vec_u *)src;
            }
            return o;
        };
        floatx4 D[NT];
        auto mult_pass = [&](const Pass &p, const Operands<NT, KS> &o) {
            if (p.kc == 0) {                                       // (uniform) a new slice
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) D[nt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
            }
            const uint32_t left = p.c - p.kc;                      // columns from here on
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (4u * s >= left) break;                         // (uniform) k-steps the block does not have
                uint32_t w = o.av[s];
                vec b = o.bv[s];
                if (vf != CSB_VAL_F32) {                           // (uniform) this lane's column of the pair: kc is even, so its parity is kq's
                    const uint32_t bits = (kq & 1u) ? w >> 16 : w & 0xffffu;
                    w = vf == CSB_VAL_BF16 ? bits << 16 : __float_as_uint((float)__builtin_bit_cast(_Float16, (uint16_t)bits));
                }
                if (4u * s + 4u > left) {                          // (uniform) the last, partial one
                    const bool ok = 4u * s + kq < left;
                    w = ok ? w : 0u;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) b[nt] = ok ? b[nt] : 0.0f;
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    D[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w), b[nt], D[nt], 0, 0, 0);
            }
            if (left > PC) return;                                 // the slice has more columns
            // lane holds rows 4 kq + i, right-hand sides NT mrow + t of each result; the rows of a slice
            // are distinct, so no two lanes meet in the accumulator (but in its spare row, which nobody
            // reads): all reads, then all writes
            uint32_t at[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t mr = p.m0 + 4u * kq + i;
                const uint32_t slot = meta[p.desc + 4u * (p.lane0 + min(mr, p.r - 1u))];
                at[i] = (mr < p.r ? slot : br) * NB + NT * mrow;
            }
            vec old[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) old[i] = *(const vec *)(myacc + at[i]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) old[i][nt] += D[nt][i];
                *(vec *)(myacc + at[i]) = old[i];
            }
        };
        Pass pa, pb;
        open_vb(wave, pa);
        pa.m0 = pa.kc = 0;
        Operands<NT, KS> oa = load_pass(pa), ob;
        if constexpr (kCounted) {
            while (true) {                                         // (loads outside of branches: the waits are counted)
                pb = next_pass(pa);
                if (!pb.valid) { mult_pass(pa, oa); break; }
                ob = load_pass(pb);
                mult_pass(pa, oa);
                pa = next_pass(pb);
                if (!pa.valid) { mult_pass(pb, ob); break; }
                oa = load_pass(pa);
                mult_pass(pb, ob);
            }
        } else {
            while (true) {                                         // the next pass's loads fly while one multiplies
                pb = next_pass(pa);
                if (pb.valid) ob = load_pass(pb);
                mult_pass(pa, oa);
                if (!pb.valid) break;
                pa = next_pass(pb);
                if (pa.valid) oa = load_pass(pa);
                mult_pass(pb, ob);
                if (!pa.valid) break;
            }
        }
    }
    __syncthreads();
    for (uint32_t e = tid; e < br * 16u; e += NTHR) {              // a row and a lane's NT right-hand sides
        vec s = *(const vec *)(acc + (size_t)e * NT);
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *(const vec *)(acc + (size_t)w * acc_wave + (size_t)e * NT);
        const uint32_t row = tile * br + (e >> 4), n_lane = bt0 + NT * (e & 15u);
        if (row >= m.rows_out) continue;
#pragma unroll
        for (int t = 0; t < NT; ++t) {                             // (a group moved back repeats right-hand sides of the one before)
            const uint32_t n = min(n_lane, batch - NT) + t;
            if (n >= n_lane) Y[(size_t)row * ldy + n] = s[t];
        }
    }
}

template <int NT, bool TWO, int NW, int KS>
__global__ __launch_bounds__(NW * 64) void spmm_kernel(const DevMat m, const XSrc X, float *__restrict__ Y,
                                                             const int64_t ldy, const uint32_t batch) {
    spmm_body<NT, TWO, NW, KS>(m, X, Y, ldy, batch, blockIdx.x, blockIdx.y);
}

// ---------------------------------------------------------------------------------------
// bfloat16 operands (v_mfma_f32_16x16x16_bf16): the kernel values are stored as bfloat16
// (csb_set_value_format) and the right-hand sides arrive as bfloat16, [cols][ldx] with the
// batch contiguous; products are exact in binary32 and are accumulated in binary32.  One
// MFMA takes 16 columns of a block (four times the f32 instruction's) and the gather of X --
// what bounds the f32 kernel -- moves half the bytes.  Same tiling as the wide f32 form: a
// lane loads four neighbouring right-hand sides of an input row at once (8 bytes), tile t
// holds the right-hand sides 4 n + t.
// The same kernel serves binary16 (HALF: v_mfma_f32_16x16x16_f16, values and right-hand sides
// as binary16, whose products are exact in binary32 as well).
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
template <bool HALF>
__device__ __forceinline__ floatx4 mfma_16bit(const uint2 a, const uint2 b, const floatx4 c) {
    if constexpr (HALF) return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, a), __builtin_bit_cast(f16x4, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, a), __builtin_bit_cast(bf16x4, b), c, 0, 0, 0);
}

template <int KS>
struct OperandsBf {
    uint2 a[KS];          // four consecutive columns of this lane's row
    uint2 b[KS][4];       // per tile: the same four columns of its right-hand side
};

template <int NW, bool HALF>
__global__ __launch_bounds__(NW * 64) void spmm_bf16_kernel(const DevMat m, const uint16_t *__restrict__ Xb, const uint32_t ldx,
                                                           float *__restrict__ Y, const int64_t ldy, const uint32_t batch) {
    extern __shared__ float4 smem4[];
    constexpr int NT = 4, NB = 64, KS = 2;         // 64 batch columns per workgroup, 32 block columns per pass
    constexpr uint32_t NTHR = NW * 64;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uni_(tid >> 6);
    const uint32_t bt0 = blockIdx.y * NB;
    const uint32_t br = m.br;
    if (blockIdx.x >= m.n_nz_tiles) {              // a row tile without work: zeros
        const uint32_t tile = m.zero_tiles[blockIdx.x - m.n_nz_tiles];
        for (uint32_t e = tid; e < br * NB; e += NTHR) {
            const uint32_t row = tile * br + e / NB, n = bt0 + e % NB;
            if (row < m.rows_out && n < batch) Y[(size_t)row * ldy + n] = 0.0f;
        }
        return;
    }
    uint8_t *meta = (uint8_t *)smem4;
    float *acc = (float *)(meta + m.seg_meta);     // [waves][br][NB]
    float *myacc = acc + (size_t)wave * br * NB;
    for (uint32_t e = lane; e < br * NB; e += 64) myacc[e] = 0.0f;
    const uint32_t rank = blockIdx.x, tile = m.nz_tiles[rank];
    const uint32_t mrow = lane & 15u, kq = lane >> 4;
    const uint32_t ncol = bt0 + 4u * mrow;         // first of this lane's four right-hand sides (batch % 4 == 0)
    const uint32_t noff = (ncol < batch ? ncol : 0u) * 2u;   // bytes; one past the batch reads 0..3, never stored

    const uint32_t sg0 = first_segment(m, rank), sg1 = first_segment(m, rank + 1u);
    for (uint32_t sg = sg0; sg < sg1; ++sg) {
        const SegRec *sp = m.segs + sg;
        const uint32_t vb0 = sp->vb0, nvbs = sp->nvbs, idx0 = sp->idx0, idx_bytes = sp->idx_bytes;
        const uint32_t ioff = nvbs * (uint32_t)sizeof(VbRec);
        __syncthreads();
        {
            const float4 *vs = (const float4 *)(m.vbs + vb0);
            float4 *vd = (float4 *)meta;
            for (uint32_t i = tid; i < nvbs; i += NTHR) vd[i] = vs[i];
            const float4 *is = (const float4 *)(m.idx + idx0);
            float4 *id = (float4 *)(meta + ioff);
            for (uint32_t i = tid; i < idx_bytes >> 4; i += NTHR) id[i] = is[i];
        }
        __syncthreads();

        auto open_vb = [&](uint32_t k) -> Pass {
            Pass p{};
            p.k = k;
            p.valid = k < nvbs;
            if (!p.valid) return p;
            const uint4 v = *(const uint4 *)(meta + k * (uint32_t)sizeof(VbRec));
            const uint32_t v0 = uni_(v.x);
            p.r = v0 & 0xffu; p.lane0 = (v0 >> 8) & 0xffu; p.c = v0 >> 16;
            p.val_off = uni_(v.y);
            p.desc = ioff + (uni_(v.z) - idx0);
            p.list = ioff + (uni_(v.w) - idx0);
            p.m0 = 0; p.kc = 0;
            return p;
        };
        auto next_pass = [&](const Pass &p) -> Pass {
            Pass q = p;
            q.kc += 16 * KS;
            if (q.kc < q.c) return q;
            q.kc = 0; q.m0 += 16;
            if (q.m0 < q.r) return q;
            return open_vb(p.k + NW);
        };
        auto load_pass = [&](const Pass &p, OperandsBf<KS> &o) {
            // one word per lane and pair of columns, the even column in the low half; a block
            // with an odd number of columns has a zero in its last word's high half
            const uint32_t *gv16 = (const uint32_t *)m.vals + (p.val_off >> 1);
            const uint16_t *colp = (const uint16_t *)(meta + p.list);
            const bool row_ok = p.m0 + mrow < p.r;
            const uint32_t arow = p.lane0 + p.m0 + (row_ok ? mrow : 0u);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (p.kc + 16u * s >= p.c) break;                  // uniform: columns the block does not have
                const uint32_t j0 = p.kc + 16u * s + 4u * kq;      // this lane's four columns
                const bool ok0 = j0 < p.c, ok1 = j0 + 2u < p.c;
                const uint32_t w0 = gv16[((ok0 ? j0 : 0u) >> 1) * (uint32_t)kWave + arow];
                const uint32_t w1 = gv16[((ok1 ? j0 + 2u : 0u) >> 1) * (uint32_t)kWave + arow];
                o.a[s] = make_uint2(ok0 && row_ok ? w0 : 0u, ok1 && row_ok ? w1 : 0u);
                // (a lane without a column reads the block's first one, times a zero)
                uint2 x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t jj = j0 + (uint32_t)i;
                    const uint32_t cb = colp[jj < p.c ? jj : 0u];  // 4 * column
                    x[i] = *(const uint2 *)((const uint8_t *)Xb + (mul24_(cb, ldx) >> 1) + noff);
                }
                // x[i] = right-hand sides 0..3 at column i; tile t wants columns 0..3 at right-hand side t
                o.b[s][0] = make_uint2((x[0].x & 0xffffu) | (x[1].x << 16), (x[2].x & 0xffffu) | (x[3].x << 16));
                o.b[s][1] = make_uint2((x[0].x >> 16) | (x[1].x & 0xffff0000u), (x[2].x >> 16) | (x[3].x & 0xffff0000u));
                o.b[s][2] = make_uint2((x[0].y & 0xffffu) | (x[1].y << 16), (x[2].y & 0xffffu) | (x[3].y << 16));
                o.b[s][3] = make_uint2((x[0].y >> 16) | (x[1].y & 0xffff0000u), (x[2].y >> 16) | (x[3].y & 0xffff0000u));
            }
        };
        floatx4 D[NT];
        const floatx4 zero4 = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) D[nt] = zero4;
        auto mult_pass = [&](const Pass &p, const OperandsBf<KS> &o) {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (p.kc + 16u * s >= p.c) break;                  // uniform
                if (s == 0 && p.kc == 0) {                         // uniform: a slice starts from a zero operand
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) D[nt] = mfma_16bit<HALF>(o.a[s], o.b[s][nt], zero4);
                } else {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) D[nt] = mfma_16bit<HALF>(o.a[s], o.b[s][nt], D[nt]);
                }
            }
            if (p.kc + 16 * KS < p.c) return;                      // the slice has more columns
            // lane holds rows 4*(lane/16)+i, right-hand side group lane%16 of each result tile
            uint32_t at[4];
            bool on[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t mr = p.m0 + 4u * kq + i;
                on[i] = mr < p.r;
                const uint32_t slot = meta[p.desc + 4u * (p.lane0 + (on[i] ? mr : 0u))];
                at[i] = slot * NB + 4u * mrow;
            }
            float4 old4[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) old4[i] = *(const float4 *)(myacc + at[i]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (on[i])
                    *(float4 *)(myacc + at[i]) = make_float4(old4[i].x + D[0][i], old4[i].y + D[1][i],
                                                             old4[i].z + D[2][i], old4[i].w + D[3][i]);
        };
        auto nxt = [&](const Pass &p) -> Pass { return p.valid ? next_pass(p) : p; };
        OperandsBf<KS> oa, ob, oc;                                  // three passes in flight
        Pass pa = open_vb(wave), pb = nxt(pa), pc{};
        if (pa.valid) load_pass(pa, oa);
        if (pb.valid) load_pass(pb, ob);
        while (true) {
            pc = nxt(pb); if (pc.valid) load_pass(pc, oc);
            if (!pa.valid) break;
            mult_pass(pa, oa);
            pa = nxt(pc); if (pa.valid) load_pass(pa, oa);
            if (!pb.valid) break;
            mult_pass(pb, ob);
            pb = nxt(pa); if (pb.valid) load_pass(pb, ob);
            if (!pc.valid) break;
            mult_pass(pc, oc);
        }
    }
    __syncthreads();
    for (uint32_t e = tid; e < br * NB; e += NTHR) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += acc[(size_t)w * br * NB + e];
        const uint32_t row = tile * br + e / NB, n = bt0 + e % NB;
        if (row < m.rows_out && n < batch) Y[(size_t)row * ldy + n] = s;
    }
}

// ---------------------------------------------------------------------------------------
// The wide form for row tiles of 16 or 32 rows, with the results kept in registers (VF: storage
// format of the kernel values; 16-bit values come as one word per row and pair of columns and
// are unpacked to binary32 on their way into the MFMA).  What bounds the kernel-row form above on long tiles is
// instructions, not the gather: on the 8192 x 8192 matrix with 128 right-hand sides, in its first version, vector
// instructions other than MFMA kept every SIMD busy for 38 % of the launch (among them the accumulate of every
// 16-row slice's 16 x 64 results into the wavefront's LDS tile: four 16-byte reads and four writes per lane), the matrix
// pipe a quarter, and pointing every gather at ONE row of X made it only 7 % faster.  Here the kernel operand of an MFMA is not the block's kernel matrix but its
// rows ALREADY SCATTERED to their places in the row tile: for each 16-row part of the tile, lane
// (row, k) holds the block's value at that tile row, or zero if the block does not keep the
// row.  The 16 x 64 results of a part then add up in the SAME registers over all blocks the
// wavefront works on, and go to LDS once, at the end.  The price is matrix-pipe work for parts
// a block has few rows in (parts it has none in are skipped).  Which kernel row sits at a tile
// row comes from a 64-byte map per wavefront in LDS that the block's lanes fill from their row
// slots.  A pass ALWAYS issues 4 NH kernel-value loads and 4 NQ 16-byte input loads (k-steps and
// parts a block does not have repeat a valid address and are not multiplied), so the loads of
// the NEXT pass are in flight while this pass multiplies and the compiler's counted waits hold.
// A row the block does not keep is a zero times the inputs of its columns: an input that is not finite makes NaN of
// the rows of the tile (the header says so; checking the results for it and computing such rows again, entry
// by entry, cost 0.1 to 0.7 us per launch on finite inputs: 8192 x 8192 x 512 bfloat16 119.2 -> 122.2 us).
// Same records, same value layout, same merge of the wavefronts' tiles as the general kernel.
//
// NQ: how many times 64 right-hand sides a workgroup takes.  What a pass costs besides its
// products -- opening the block, the map, the column list, the kernel values -- is the same for 64
// and for 128 right-hand sides, and so are a workgroup's records, its barriers and its place in
// the launch, so the wide form (NQ = 2; 8 wavefronts, whose registers hold the 32 x 128 results)
// does half of all that.  The wavefronts' tiles are merged 64 columns at a time, so the LDS does
// not grow.
// Measured on the 8192 x 8192 matrix at 12x (32 x 32 blocks), 64 -> 128 right-hand sides per
// workgroup: float32, batch 128, 71.2 -> 63.4 us (22.7 TFLOP/s; there the chip is filled by
// one turn of 256 workgroups instead of two of 512); bfloat16, batch 512, 169.7 -> 121.1 us.
template <int NH, int NQ>
struct RegOps {
    float av[NH][4];
    float4 bv[4][NQ];
    uint32_t parts;              // bit h: the block has rows in part h (uniform)
};
// ... with 16-bit right-hand sides (X16): a pass is ONE 16-column MFMA step per part and tile; a
// lane's four columns of its tile row are two words of the value stream, its four right-hand
// sides of a column eight bytes of X.
template <int NH, int NQ>
struct RegOps16 {
    uint32_t aw[NH][2];
    uint2 xv[4][NQ];
    uint32_t parts;
};
struct RegPass {
    uint32_t k, kc;              // virtual block (inside the segment), first column of the pass
    uint32_t r, c, lane0;        // the block's rows, columns, first lane
    uint32_t val_off, desc, list;
    bool valid;
};

template <bool TWO, int NW, int NH, int VF, int NQ, bool X16 = false>
__device__ __forceinline__ void spmm_reg_body(const DevMat &m, const XSrc &X, float *__restrict__ Y, const int64_t ldy,
                                              const uint32_t batch, const uint32_t block_x, const uint32_t block_y) {
    extern __shared__ float4 smem4[];
    constexpr uint32_t NB = 64, NTHR = NW * 64;                    // right-hand sides per merge
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uni_(tid >> 6);
    const uint32_t bt0 = block_y * (NB * NQ);
    const uint32_t br = m.br;                                      // == 16 NH
    if (block_x >= m.n_nz_tiles) {                 // a row tile without work: zeros
        const uint32_t tile = m.zero_tiles[block_x - m.n_nz_tiles];
        for (uint32_t e = tid; e < br * NB * NQ; e += NTHR) {
            const uint32_t row = tile * br + e / (NB * NQ), n = bt0 + e % (NB * NQ);
            if (row < m.rows_out && n < batch) Y[(size_t)row * ldy + n] = 0.0f;
        }
        return;
    }
    uint8_t *meta = (uint8_t *)smem4;                              // one record segment
    float *acc = (float *)(meta + m.seg_meta);                     // [waves][br][NB]
    float *myacc = acc + (size_t)wave * br * NB;
    uint8_t *inv = (uint8_t *)(acc + (size_t)NW * br * NB) + wave * 64u;   // tile row -> kernel row of the current block, 0xff: none
    const uint32_t rank = block_x, tile = m.nz_tiles[rank];
    const uint32_t mrow = lane & 15u, kq = lane >> 4;              // A: tile row in its part, column-in-4; B: right-hand sides 4 mrow .. + 3, row-in-4
    uint32_t nbyte[NQ];                            // this lane's right-hand sides: bt0 + 64 q + 4 mrow .. + 3
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const uint32_t ncol = bt0 + 64u * q + 4u * mrow;
        nbyte[q] = (ncol < batch ? ncol : 0u) * (X16 ? 2u : 4u);   // (batch is a multiple of 4: the four are in or out together)
    }
    const uint32_t split4 = 4u * X.n0, sj0 = uni_(X.sj0), sj1 = uni_(X.sj1);   // (see uni_)
    // (the lane's own pointers: choosing one of them is a choice between registers)
    const uint8_t *const x0 = (const uint8_t *)X.p0 + nbyte[0], *const x1 = (const uint8_t *)X.p1 + nbyte[0];
    floatx4 D[NH][NQ][4];
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) D[h][q][nt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    const uint32_t sg0 = first_segment(m, rank), sg1 = first_segment(m, rank + 1u);
    for (uint32_t sg = sg0; sg < sg1; ++sg) {
        // ---- stage the segment's records ------------------------------------------------
        const SegRec *sp = m.segs + sg;
        const uint32_t vb0 = sp->vb0, nvbs = sp->nvbs, idx0 = sp->idx0, idx_bytes = sp->idx_bytes;
        const uint32_t ioff = nvbs * (uint32_t)sizeof(VbRec);
        __syncthreads();                                           // the previous segment is done with
        {
            const float4 *vs = (const float4 *)(m.vbs + vb0);
            float4 *vd = (float4 *)meta;
            for (uint32_t i = tid; i < nvbs; i += NTHR) vd[i] = vs[i];
            const float4 *is = (const float4 *)(m.idx + idx0);
            float4 *id = (float4 *)(meta + ioff);
            for (uint32_t i = tid; i < idx_bytes >> 4; i += NTHR) id[i] = is[i];
        }
        __syncthreads();
        if (wave >= nvbs) continue;                                // (uniform per wavefront; the barriers above are passed by all)

        // Kernel values come through a buffer descriptor over the value stream: a load whose offset lies
        // past the stream returns zero, which is what a lane without a row or a column gets (its offset
        // is pushed there), so no operand is ever masked after the load.
        const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)m.vals, 0, (int)m.vals_bytes, 0x00020000);
        uint32_t irow4[NH];                                        // byte offset of this lane's kernel row in the current block's values, per part (bit 31: none)
        uint32_t parts = 0;
        // A block's data in LDS is four dependent reads deep (record, row slots, map, input offsets), as long as
        // its products.  With 128 right-hand sides of one source, records are read two blocks ahead and row
        // slots one, and a block opens with one wait: the map's (8192 x 8192 x 128 float32 63.4 -> 62.7 us, x 512
        // bfloat16 121.1 -> 118.6).  What that holds costs 10 to 20 registers, which the others have not got: two
        // sources with 32 rows and 16-bit values went to scratch, and the 16-bit form of 16 rows and 64
        // right-hand sides no longer had two workgroups on a CU (8192 x 2048 x 64 18.6 us, 16.0 without).
        constexpr bool kAhead = !TWO && NQ == 2;
        auto read_rec = [&](uint32_t k) { return *(const uint4 *)(meta + min(k, nvbs - 1u) * (uint32_t)sizeof(VbRec)); };
        auto decode = [&](const uint4 v, uint32_t k) -> RegPass {
            RegPass p;
            const uint32_t v0 = uni_(v.x);
            p.k = k; p.valid = k < nvbs; p.kc = 0;
            p.r = v0 & 0xffu; p.lane0 = (v0 >> 8) & 0xffu; p.c = v0 >> 16;
            p.val_off = uni_(v.y);
            p.desc = ioff + (uni_(v.z) - idx0);
            p.list = ioff + (uni_(v.w) - idx0);
            return p;
        };
        auto read_slot = [&](const RegPass &p) -> uint32_t { return meta[p.desc + 4u * (p.lane0 + (lane < p.r ? lane : 0u))]; };
        // 4 * column of this lane's columns of pass p
        auto read_cols = [&](const RegPass &p, uint32_t (&c)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                c[i] = *(const uint16_t *)(meta + p.list + 2u * min(p.kc + (X16 ? 4u * kq + i : 4u * i + kq), p.c - 1u));
        };
        uint32_t cb_ahead[4];                                      // (kAhead: of the pass opened last)
        // The map of block p: cleared, then every kernel row of the block enters itself at its tile row (the
        // wavefront's LDS operations execute in order).
        auto map_rows = [&](const RegPass &p, const uint32_t slot) {
            if (lane < 16u) ((uint32_t *)inv)[lane] = 0xffffffffu;
            if (lane < p.r) inv[slot] = (uint8_t)lane;
            parts = 0;
            // (16-bit formats: one 32-bit word per kernel row and PAIR of columns, the even column in the low half)
            const uint32_t base4 = ((VF == CSB_VAL_F32 ? p.val_off : p.val_off >> 1) + p.lane0) * 4u;
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const uint32_t ir = inv[16u * h + mrow];
                irow4[h] = ir != 0xffu ? base4 + ir * 4u : 0x80000000u;
                parts |= __ballot(ir != 0xffu) != 0ull ? 1u << h : 0u;
            }
        };
        RegPass ahead;                                             // the next block ...
        uint32_t ahead_slot;                                       // ... its rows' places
        uint4 after;                                               // the record of the one after it
        if constexpr (kAhead) {
            ahead = decode(read_rec(wave), wave);
            ahead_slot = read_slot(ahead);
            after = read_rec(wave + NW);
        }
        auto open = [&](uint32_t k) -> RegPass {                   // block k of the segment; blocks are opened in order
            RegPass p;
            uint32_t slot;
            if constexpr (kAhead) {
                p = ahead;
                slot = ahead_slot;
                read_cols(p, cb_ahead);
                ahead = decode(after, k + NW);
                ahead_slot = read_slot(ahead);
                after = read_rec(k + 2u * NW);
            } else {
                p = decode(read_rec(k), k);
                slot = read_slot(p);
            }
            map_rows(p, slot);
            return p;
        };
        // The pass after p.  Only LDS is read on the way, so the count of the global loads in flight is the same
        // on every path and the compiler's counted waits stay exact.  Past the wavefront's last pass some
        // block of the segment is opened again: its loads are dropped.  (Without the read-ahead a block
        // is opened again for its further passes, too: a branch around that takes registers.)
        auto advance = [&](const RegPass &p) -> RegPass {
            const bool same = p.kc + 16u < p.c;                    // (uniform)
            RegPass q = p;
            if constexpr (kAhead) {
                if (!same) return open(p.k + NW);
                q.kc = p.kc + 16u;
                read_cols(q, cb_ahead);
            } else {
                q = open(same ? p.k : p.k + NW);
                q.kc = same ? p.kc + 16u : 0u;
            }
            return q;
        };
        // 4 NH + 4 NQ loads, always.  (Uses irow4 / parts of the block opened last: p's.)
        auto issue = [&](const RegPass &p, RegOps<NH, NQ> &o) {
            uint32_t ja[4];
            o.parts = parts;
            uint32_t cb[4];
            if constexpr (kAhead) { for (int i = 0; i < 4; ++i) cb[i] = cb_ahead[i]; } else read_cols(p, cb);
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                const uint32_t jj = p.kc + 4u * s4 + kq;
                ja[s4] = jj < p.c ? jj : 0x7fffffu;                             // a column the block lacks: past the stream
            }
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
#pragma unroll
                for (int h = 0; h < NH; ++h)
                    if constexpr (VF == CSB_VAL_F32) {
                        o.av[h][s4] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vrsrc, (int)(ja[s4] * 256u + irow4[h]), 0, 0));
                    } else {                                        // (unpacked in multiply: the load's result is not waited for here)
                        o.av[h][s4] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vrsrc, (int)((ja[s4] >> 1) * 256u + irow4[h]), 0, 0));
                    }
                if constexpr (TWO) {
                    const bool first = cb[s4] < split4;
                    const uint8_t *src = first ? x0 + mul24_(cb[s4], sj0) : x1 + mul24_(cb[s4] - split4, sj1);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) o.bv[s4][q] = *(const float4 *)(src + (int)(nbyte[q] - nbyte[0]));
                } else {
                    const uint32_t joff = mul24_(cb[s4], sj0);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) o.bv[s4][q] = *(const float4 *)((const uint8_t *)X.p0 + (size_t)(joff + nbyte[q]));
                }
            }
        };
        auto multiply = [&](const RegPass &p, const RegOps<NH, NQ> &o) {
            const uint32_t nk = min(4u, (p.c - p.kc + 3u) >> 2);      // k-steps the block has in this pass (uniform)
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                if (!((o.parts >> h) & 1u)) continue;              // (uniform) no row of the block in this part
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4) {
                    if ((uint32_t)s4 >= nk) break;
                    float a = o.av[h][s4];
                    if constexpr (VF != CSB_VAL_F32) {              // this lane's column of the pair: kc is even, so its parity is kq's
                        const uint32_t w = __float_as_uint(a);
                        if constexpr (VF == CSB_VAL_BF16) a = __uint_as_float((kq & 1u) ? w & 0xffff0000u : w << 16);
                        else a = (float)__builtin_bit_cast(_Float16, (uint16_t)((kq & 1u) ? w >> 16 : w & 0xffffu));
                    }
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        D[h][q][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, o.bv[s4][q].x, D[h][q][0], 0, 0, 0);
                        D[h][q][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, o.bv[s4][q].y, D[h][q][1], 0, 0, 0);
                        D[h][q][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, o.bv[s4][q].z, D[h][q][2], 0, 0, 0);
                        D[h][q][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, o.bv[s4][q].w, D[h][q][3], 0, 0, 0);
                    }
                }
            }
        };
        // The same two steps with 16-bit right-hand sides (X.p0: their rows, X.sj0: elements per row):
        // 2 NH + 4 NQ loads, always, and one 16-column MFMA per part and tile.
        auto issue16 = [&](const RegPass &p, RegOps16<NH, NQ> &o) {
            o.parts = parts;
            uint32_t cb[4];
            if constexpr (kAhead) { for (int i = 0; i < 4; ++i) cb[i] = cb_ahead[i]; } else read_cols(p, cb);
            const uint32_t j0 = p.kc + 4u * kq;                                  // this lane's four columns
            const uint32_t w0 = j0 < p.c ? (j0 >> 1) * 256u : 0x3fffff00u;       // words of the pairs (j0, j0 + 1), (j0 + 2, j0 + 3);
            const uint32_t w1 = j0 + 2u < p.c ? (j0 >> 1) * 256u + 256u : 0x3fffff00u;   // a pair the block lacks: past the stream
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                o.aw[h][0] = __builtin_amdgcn_raw_buffer_load_b32(vrsrc, (int)(w0 + irow4[h]), 0, 0);
                o.aw[h][1] = __builtin_amdgcn_raw_buffer_load_b32(vrsrc, (int)(w1 + irow4[h]), 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)      // (a column the block lacks reads its last one, times a zero)
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    o.xv[i][q] = *(const uint2 *)((const uint8_t *)X.p0 + (size_t)((mul24_(cb[i], sj0) >> 1) + nbyte[q]));
        };
        auto multiply16 = [&](const RegOps16<NH, NQ> &o) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                // xv[i] = right-hand sides 0..3 at column i; tile t wants columns 0..3 at right-hand side t
                const uint2 x0 = o.xv[0][q], x1 = o.xv[1][q], x2 = o.xv[2][q], x3 = o.xv[3][q];
                const uint2 b0 = make_uint2((x0.x & 0xffffu) | (x1.x << 16), (x2.x & 0xffffu) | (x3.x << 16));
                const uint2 b1 = make_uint2((x0.x >> 16) | (x1.x & 0xffff0000u), (x2.x >> 16) | (x3.x & 0xffff0000u));
                const uint2 b2 = make_uint2((x0.y & 0xffffu) | (x1.y << 16), (x2.y & 0xffffu) | (x3.y << 16));
                const uint2 b3 = make_uint2((x0.y >> 16) | (x1.y & 0xffff0000u), (x2.y >> 16) | (x3.y & 0xffff0000u));
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    if (!((o.parts >> h) & 1u)) continue;          // (uniform) no row of the block in this part
                    const uint2 a = make_uint2(o.aw[h][0], o.aw[h][1]);
                    D[h][q][0] = mfma_16bit<VF == CSB_VAL_F16>(a, b0, D[h][q][0]);
                    D[h][q][1] = mfma_16bit<VF == CSB_VAL_F16>(a, b1, D[h][q][1]);
                    D[h][q][2] = mfma_16bit<VF == CSB_VAL_F16>(a, b2, D[h][q][2]);
                    D[h][q][3] = mfma_16bit<VF == CSB_VAL_F16>(a, b3, D[h][q][3]);
                }
            }
        };
        if constexpr (X16) {
            RegOps16<NH, NQ> oa, ob;
            RegPass pa = open(wave), pb;
            issue16(pa, oa);
            while (true) {
                pb = advance(pa);
                issue16(pb, ob);
                multiply16(oa);
                if (!pb.valid) break;
                pa = advance(pb);
                issue16(pa, oa);
                multiply16(ob);
                if (!pa.valid) break;
            }
            continue;                                              // (the next segment)
        }
        RegOps<NH, NQ> oa, ob;
        RegPass pa = open(wave), pb;
        issue(pa, oa);
        while (true) {
            pb = advance(pa);
            issue(pb, ob);
            multiply(pa, oa);
            if (!pb.valid) break;
            pa = advance(pb);
            issue(pa, oa);
            multiply(pb, ob);
            if (!pa.valid) break;
        }
    }
    // the wavefront's tile, 64 columns at a time: lane holds rows 16 h + 4 kq + i, right-hand sides 4 mrow + t (tile t)
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        if (q > 0) __syncthreads();                                // the columns before are summed
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(float4 *)(myacc + (16u * h + 4u * kq + i) * NB + 4u * mrow) = make_float4(D[h][q][0][i], D[h][q][1][i], D[h][q][2][i], D[h][q][3][i]);
        __syncthreads();
        for (uint32_t e = tid; e < br * NB; e += NTHR) {
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += acc[(size_t)w * br * NB + e];
            const uint32_t row = tile * br + e / NB, n = bt0 + 64u * q + e % NB;
            if (row < m.rows_out && n < batch) Y[(size_t)row * ldy + n] = s;
        }
    }
}

template <bool TWO, int NW, int NH, int VF, int NQ>
__global__ __launch_bounds__(NW * 64) void spmm_reg_kernel(const DevMat m, const XSrc X, float *__restrict__ Y,
                                                           const int64_t ldy, const uint32_t batch) {
    spmm_reg_body<TWO, NW, NH, VF, NQ>(m, X, Y, ldy, batch, blockIdx.x, blockIdx.y);
}

// 16-bit kernel values times 16-bit right-hand sides (X.p0: the rows of X, X.sj0: elements per row).
template <int NW, int NH, int VF, int NQ>
__global__ __launch_bounds__(NW * 64) void spmm_reg16_kernel(const DevMat m, const XSrc X, float *__restrict__ Y,
                                                             const int64_t ldy, const uint32_t batch) {
    static_assert(VF == CSB_VAL_F16 || VF == CSB_VAL_BF16, "16-bit formats only");
    spmm_reg_body<false, NW, NH, VF, NQ, true>(m, X, Y, ldy, batch, blockIdx.x, blockIdx.y);
}

template <int NT, bool TWO, int NW, int KS>
__global__ __launch_bounds__(NW * 64) void spmm_multi_kernel(const SpmmJobs J, const uint32_t batch) {
    const uint32_t j = blockIdx.z;
    if (blockIdx.x >= J.m[j].n_nz_tiles + J.m[j].n_zero_tiles) return;      // the grid is as wide as the widest product
    spmm_body<NT, TWO, NW, KS>(J.m[j], J.X[j], J.Y[j], J.ldy[j], batch, blockIdx.x, blockIdx.y);
}

template <bool TWO, int NW, int NH, int VF, int NQ>
__global__ __launch_bounds__(NW * 64) void spmm_reg_multi_kernel(const SpmmJobs J, const uint32_t batch) {
    const uint32_t j = blockIdx.z;
    if (blockIdx.x >= J.m[j].n_nz_tiles + J.m[j].n_zero_tiles) return;      // the grid is as wide as the widest product
    spmm_reg_body<TWO, NW, NH, VF, NQ>(J.m[j], J.X[j], J.Y[j], J.ldy[j], batch, blockIdx.x, blockIdx.y);
}

// Launch shape of one product: batch columns per workgroup (16 nt), wavefronts per workgroup.
struct SpmmShape {
    int nt, nw;
    int ks;                 // k-steps a pass of the general form has room for: 8 (32 columns), or 4 at NT = 4 and where
                            // blocks are no wider than 16: half the registers, more workgroups on a CU (6727 x 4661 in
                            // 16 x 16 blocks at batch 6: 34.0 -> 27.0 us)
    bool two;
    int reg_parts;          // 64 columns, row tiles of 16 or 32 rows: the kernel that keeps the results in
                            // registers, with this many 16-row parts (else 0; 64-row tiles' four parts do not fit the registers
                            // of a 16-wavefront workgroup; for one of 8 there is no such kernel)
    int nq;                 // ... and this many times 64 right-hand sides per workgroup
    int vf;                 // storage format of the kernel values
    size_t lds;
    unsigned tiles, batch_tiles;
};

// ---- estimate of a launch's time from the tile-based sections -----------------------------------------------------
// The section of four-row steps takes a pass for every 8 columns of a block and a row sum for every row; here a 16-row product
// takes a block's rows, many or few, and sums them as it goes: faster where blocks are nearly full, and for few right-hand sides of
// many row tiles.  Constants as in csb_spmm_quad.hip (us per block record and 8 of its columns, `full` where it keeps
// them all and they are neighbours, `uneven` what the longest share of 16 has more than
// their mean; general forms: per 16 rows of a block), from the same measurements.  A launch takes these sections where they save 5 % by the estimates; blocks
// of more than 32 rows were never faster here.  us here / in four-row steps: 4096 x 4096 in 32-row blocks x 128 unpruned
// 45.0 / 63.7, at 2x 38.6 / 43.8, 4x 30.6 / 28.0; 2048 x 2048 in 16-row blocks x 16 at 2x 12.1 / 14.2, 4x 11.0 / 9.9; 4100 x 2048
// in 24-row blocks x 4 at 4x 10.7 / 15.7, x 32 18.8 / 15.7.
struct TileTurn { double base, block, cols, full, uneven; };
struct TileCost {
    int form, rows, nw, room;   // general form: 0, 16 nt columns, wavefronts, k-steps; in registers: 1, 16-row parts, wavefronts, 64 nq columns
    double base, out;
    TileTurn one, two;
};
static const TileCost kTileCost[] = {
    {0, 1, 16, 4, 3.97, 0.697, {0, 0.589, 0.337, 0.293, 0}, {}},
    {0, 1, 16, 8, 3.04, 5.08, {0.885, 0.512, 0.404, 0.397, 1.22}, {}},
    {0, 1, 8, 4, 4.49, 0, {0, 0.371, 0.0379, 0, 0}, {0, 0.475, 0.475, 0.395, 0}},
    {0, 1, 8, 8, 3.13, 0.0977, {0, 0.288, 0.134, 0.177, 0}, {0.739, 0.329, 0.565, 0.553, 1.52}},
    {0, 2, 16, 4, 3.08, 2.84, {0.889, 0.763, 0.51, 0.468, 0}, {}},
    {0, 2, 16, 8, 3.17, 2.34, {1.32, 0.596, 0.565, 0.569, 1.41}, {}},
    {0, 2, 8, 4, 3.87, 5.45, {0, 0.362, 0.188, 0.216, 0}, {0, 0.618, 0.438, 0.376, 0}},
    {0, 2, 8, 8, 3.4, 4.13, {0.326, 0.423, 0.312, 0.299, 0.651}, {0.296, 0.548, 0.595, 0.62, 1.7}},
    {0, 4, 16, 4, 2.64, 2.28, {1.74, 0.73, 0.939, 0.874, 1.32}, {}},
    {1, 1, 16, 1, 2.33, 3.14, {1.85, 0.716, 0.403, 0.367, 0}, {}},
    {1, 1, 8, 2, 2.06, 1.33, {3.02, 0.528, 0.46, 0.412, 0.0323}, {5.43, 1.03, 0.926, 0.813, 0}},
    {1, 2, 16, 1, 2.84, 2.32, {2.61, 0.517, 1.23, 1.02, 0.0987}, {}},
    {1, 2, 8, 2, 2.8, 1, {3.78, 0.413, 1.09, 0.984, 0.868}, {7.47, 0.809, 2.23, 1.9, 1.19}},
};
// Of n products that share a launch of the shape (form, rows, nw, room).
static double tile_us(int form, int rows, int nw, int room, const csb_matrix *const *mats, int n, int32_t batch, unsigned batch_tiles) {
    const TileCost *f = nullptr;
    for (const TileCost &c : kTileCost) if (c.form == form && c.rows == rows && c.nw == nw && c.room == room) f = &c;
    double tiles = 0, blocks = 0, vbs = 0, cols = 0, full_cols = 0, squares = 0, out_words = 0;
    for (int i = 0; i < n; ++i) {
        const Plan &pl = mats[i]->plan;
        if (pl.hdr.br > 32) f = nullptr;
        tiles += (double)pl.hdr.n_nz_tiles + pl.hdr.n_zero_tiles;
        vbs += pl.hdr.n_vbs;
        blocks += form == 0 && pl.hdr.br > 16 ? pl.vb_slices : pl.hdr.n_vbs;      // (the general forms take 16 rows at a time)
        cols += pl.vb_cols - pl.vb_full;
        full_cols += pl.vb_full;
        squares += pl.vb_squares;
        out_words += (double)pl.hdr.rows_out * batch;
    }
    if (!f || vbs == 0) return 1e300;
    const double wgs = tiles * batch_tiles, slots = nw == 8 ? 512 : 256;
    const double full = (double)(uint64_t)(wgs / slots), rest = wgs - full * slots;
    double one = full + (rest > 0 ? 1 : 0), two = 0;
    if (nw == 8) { two = full + (rest > 256 ? 1 : 0); one = rest > 0 && rest <= 256 ? 1 : 0; }
    const double per_wave = blocks / tiles / nw;
    const double mean = (cols + full_cols) / vbs, spread = std::sqrt(std::max(squares / vbs - mean * mean, 0.0) * per_wave) / 8;
    auto turn = [&](const TileTurn &t) {
        return t.base + per_wave * (t.block + (t.cols * cols + t.full * full_cols) / (8 * vbs)) + t.uneven * spread;
    };
    return f->base + f->out * out_words * 1e-6 + one * turn(f->one) + two * turn(f->two);
}
// (Two sources: a choice per lane and load.  The steps of two GRU layers of 512 at 3x and batch 256 took 30.9 us with 128 columns
// in registers, 22.7 in four-row steps, where products of one source are as fast; those of a Li-GRU layer of 1024 at 3x and
// batch 128, 64 columns, 18.0 and 15.7, at 2x and batch 16, 16 columns, 13.0 and 14.8.)
static double tile_us(const SpmmShape &sh, const csb_matrix *const *mats, int n, int32_t batch) {
    const double two = !sh.two || sh.nt == 1 ? 1.0 : sh.nq > 1 ? 1.5 : 1.2;
    return two * (sh.reg_parts ? tile_us(1, sh.reg_parts, sh.nw, sh.nq, mats, n, batch, sh.batch_tiles)
                               : tile_us(0, sh.nt, sh.nw, sh.ks, mats, n, batch, sh.batch_tiles));
}
static bool prefers_quads(double quads_us, double tiles_us) { return 0.95 * quads_us <= tiles_us; }

// How many times 64 right-hand sides a workgroup of the register-accumulating kernels takes, for `tiles` row tiles
// of `rows` rows in the launch and right-hand sides of 32 or 16 bits.  128 halve what is done per block, and
// where every one of the 256 CUs has a workgroup of them, what counts is the number of turns the workgroups take
// over the CUs (a CU holds one of either kind, or two, which then share its units): the last turn may be
// nearly empty, and so may the last 64 right-hand sides, whose products are computed all the same.  A turn
// at 128 takes 1.6 to 1.75 times as long as at 64 (32-row tiles, float32), 1.3 to 1.45 (16-bit right-hand sides), 1.55
// to 1.65 (16-row tiles).  us at 64 / 128: 8192 x 8192 float32 x 128 72 / 63, x 132 106 / 123, x 256 140 / 124, x 260 174 /
// 183; bfloat16 x 132 65 / 61; 8224 x 4096 float32 x 128 55.6 / 61.7, x 452 165 / 157; 4096 x 2048 x 260 34.8 / 37.5; 4300 x
// 2048 in 16-row tiles x 132 42 / 47, x 196 54 / 48.
static int reg_columns(size_t tiles, uint32_t rows, int32_t batch, bool bits16) {
    const size_t wgs64 = tiles * (size_t)((batch + 63) / 64), wgs128 = tiles * (size_t)((batch + 127) / 128);
    if (batch <= 64 || wgs128 < 256) return 1;
    const size_t turn128 = rows <= 16 ? 16 : bits16 ? 14 : 17;                // ten times a turn's length against 64
    return (wgs128 + 255) / 256 * turn128 < (wgs64 + 255) / 256 * 10 ? 2 : 1;
}

// Row tiles with many blocks (of the n products that share a launch, on average): 12 and more for each of 8 wavefronts.
static bool long_tiles(const SpmmCall *calls, int n) {
    uint64_t blocks = 0, tiles = 0;
    for (int i = 0; i < n; ++i) { blocks += calls[i].mat->plan.hdr.n_vbs; tiles += calls[i].mat->plan.hdr.n_nz_tiles; }
    return blocks >= 96 * tiles;
}

static int spmm_ready(const csb_matrix *mat) {
    if (mat->plan.valid && mat->uploaded && mat->d_buf) return CSB_OK;
    set_error("csb_spmm: matrix not planned and uploaded");
    return CSB_ESTATE;
}

// Checks one product's operands and chooses its launch shape; `launch_wgs_factor` products of
// this size share the launch, which counts when the launch is sized against the GPU's 256 CUs.
static int spmm_shape(const SpmmCall &c, int32_t batch, size_t launch_wgs_factor, bool long_tiles, SpmmShape *out, XSrc *X) {
    const csb_matrix *mat = c.mat;
    const DevHeader &h = mat->plan.hdr;
    // 32-bit element offsets, 24-bit multiplies
    const int64_t smax_j = std::max(c.sj0, c.sj1);
    if (c.sj0 < 0 || c.sj1 < 0 || smax_j >= (1 << 24) || (int64_t)h.cols >= (1 << 24) ||
        (int64_t)h.cols * smax_j + (int64_t)batch >= (1ll << 30)) {
        set_error("csb_spmm: strides or sizes beyond the kernel's 32-bit element offsets");
        return CSB_EUNSUPPORTED;
    }
    *X = XSrc{c.p0, c.n0, (uint32_t)c.sj0, c.p1, (uint32_t)c.sj1};
    const bool two = c.n0 < (uint32_t)h.cols;
    // batch columns per workgroup: the widest form whose launch still gives every CU (256) a workgroup;
    // 16 wavefronts share a tile's blocks when their accumulator tiles fit LDS and the launch alone would
    // not give every CU two workgroups (64 columns: always when they fit), else 8.  64 columns by 8 wavefronts
    // (tiles of more than 36 rows) read a tile's blocks half as often as 32 do, and their merge is twice as long: they
    // pay where a wavefront has many blocks.  us at 32 / 64 columns, 64 x 64 blocks, 5 blocks per wavefront:
    // 8192 x 300 x 97 in blocks of 48 11.7 / 14.3, 8192 x 2048 x 129 39.0 / 48.1, two GRU layers of 2048 at batch 64
    // 38.6 / 41.4; 16 per wavefront: 8192 x 8192 x 128 75 / 52; 12: 8192 x 4000 x 128 in blocks of 40 55.1 / 54.3.
    const size_t tiles = (size_t)h.n_nz_tiles + h.n_zero_tiles;
    auto wgs = [&](int n) { return tiles * (size_t)((batch + 16 * n - 1) / (16 * n)); };
    auto acc_lds = [&](int n, int waves) { return (size_t)h.seg_meta + (size_t)waves * (h.br + 1) * 16 * n * sizeof(float); };
    int nt = 1;
    if (h.br <= 128 && batch > 16 && wgs(2) * launch_wgs_factor >= 256) nt = 2;
    if (batch >= 48 && wgs(4) * launch_wgs_factor >= 256 && acc_lds(4, long_tiles || h.br <= 32 ? 8 : 16) <= (size_t)kLdsBudget) nt = 4;
    const bool fits16 = acc_lds(nt, 16) <= (size_t)kLdsBudget;
    const int nw = fits16 && (nt == 4 || wgs(nt) * launch_wgs_factor < 2 * 256) ? 16 : 8;
    const int ks = nt == 4 || h.bc <= 16 ? 4 : 8;
    // The register-accumulating kernels: row tiles of 16 or 32 rows, 16-byte aligned rows of the input, batch in
    // fours (their 32-bit byte offsets into the value stream must stay below the out-of-range marker).
    const bool aligned = ((uintptr_t)c.p0 % 16 == 0) && c.sj0 % 4 == 0 && (!two || (((uintptr_t)c.p1 % 16 == 0) && c.sj1 % 4 == 0));
    const size_t reg_wave = (size_t)h.br * 64 * sizeof(float) + 64;
    const int nq = reg_columns(tiles * launch_wgs_factor, h.br, batch, false), nwr = nq > 1 ? 8 : nw;
    const int reg_parts = (nt == 4 && aligned && batch % 4 == 0 && (h.br == 16 || h.br == 32) && h.n_vals * 4 < 0x7fffff00ull &&
                           (size_t)h.seg_meta + (size_t)nwr * reg_wave <= (size_t)160 * 1024) ? (int)h.br / 16 : 0;
    if (reg_parts)
        *out = SpmmShape{nt, nwr, ks, two, reg_parts, nq, (int)h.val_fmt, (size_t)h.seg_meta + (size_t)nwr * reg_wave, (unsigned)tiles,
                         (unsigned)((batch + 64 * nq - 1) / (64 * nq))};
    else
        *out = SpmmShape{nt, nw, ks, two, 0, 1, (int)h.val_fmt, acc_lds(nt, nw), (unsigned)tiles, (unsigned)((batch + 16 * nt - 1) / (16 * nt))};
    return CSB_OK;
}

// The kernel instantiation for a launch shape (one product per launch, or several).
template <bool MULTI>
static const void *spmm_kernel_for(const SpmmShape &sh) {
#define CSB_SPMM_K(NT, TWO, NW, KS) (MULTI ? (const void *)spmm_multi_kernel<NT, TWO, NW, KS> : (const void *)spmm_kernel<NT, TWO, NW, KS>)
    if (sh.reg_parts) {
#define CSB_SPMM_RV(TWO, NW, NH, VF, NQ) (MULTI ? (const void *)spmm_reg_multi_kernel<TWO, NW, NH, VF, NQ> : (const void *)spmm_reg_kernel<TWO, NW, NH, VF, NQ>)
#define CSB_SPMM_R(TWO, NW, NH, NQ) (sh.vf == CSB_VAL_F16 ? CSB_SPMM_RV(TWO, NW, NH, CSB_VAL_F16, NQ) : sh.vf == CSB_VAL_BF16 ? CSB_SPMM_RV(TWO, NW, NH, CSB_VAL_BF16, NQ) : CSB_SPMM_RV(TWO, NW, NH, CSB_VAL_F32, NQ))
#define CSB_SPMM_RN(NH) \
        if (sh.nq == 2) return sh.two ? CSB_SPMM_R(true, 8, NH, 2) : CSB_SPMM_R(false, 8, NH, 2); \
        if (sh.nw == 16) return sh.two ? CSB_SPMM_R(true, 16, NH, 1) : CSB_SPMM_R(false, 16, NH, 1); \
        return sh.two ? CSB_SPMM_R(true, 8, NH, 1) : CSB_SPMM_R(false, 8, NH, 1);
        if (sh.reg_parts == 1) { CSB_SPMM_RN(1) }
        CSB_SPMM_RN(2)
#undef CSB_SPMM_RN
#undef CSB_SPMM_R
#undef CSB_SPMM_RV
    }
#define CSB_SPMM_KN(NT, KS) \
    if (sh.nw == 16) return sh.two ? CSB_SPMM_K(NT, true, 16, KS) : CSB_SPMM_K(NT, false, 16, KS); \
    return sh.two ? CSB_SPMM_K(NT, true, 8, KS) : CSB_SPMM_K(NT, false, 8, KS);
    if (sh.nt == 4) { CSB_SPMM_KN(4, 4) }
    if (sh.nt == 2 && sh.ks == 4) { CSB_SPMM_KN(2, 4) }
    if (sh.nt == 2) { CSB_SPMM_KN(2, 8) }
    if (sh.ks == 4) { CSB_SPMM_KN(1, 4) }
    CSB_SPMM_KN(1, 8)
#undef CSB_SPMM_KN
#undef CSB_SPMM_K
}

int spmm_strided(const csb_matrix *mat, const float *p0, uint32_t n0, int64_t sj0, const float *p1,
                 int64_t sj1, float *d_Y, int64_t ldy, int32_t batch, void *stream) {
    const SpmmCall c{mat, p0, n0, sj0, p1, sj1, d_Y, ldy};
    SpmmShape sh;
    XSrc X;
    int rc = spmm_ready(mat);
    if (rc == CSB_OK) rc = spmm_shape(c, batch, 1, long_tiles(&c, 1), &sh, &X);
    if (rc != CSB_OK) return rc;
    uint32_t b = (uint32_t)batch;
    int64_t ld = ldy;
    XSrc QX;
    bool two;
    hipError_t e;
    const bool quads = quad_source(c, &QX, &two);
    const QuadShape qs = quads ? quad_shape(&mat, 1, batch) : QuadShape{};
    if (quads && (mat->batch_form == kFormQuads || prefers_quads(qs.us, tile_us(sh, &mat, 1, batch)))) {
        QuadMat qm = quad_mat(mat, qs.low);
        void *args[] = {&qm, &QX, &d_Y, &ld, &b};
        const void *kern = quad_kernel(qs, two, false);
        e = ensure_dynamic_lds(kern, qs.lds);
        if (e == hipSuccess)
            e = hipLaunchKernel(kern, dim3(qs.tiles, qs.batch_tiles), dim3(qs.nw * 64), args, qs.lds, (hipStream_t)stream);
    } else {
        DevMat dm = dev_mat(mat);
        void *args[] = {&dm, &X, &d_Y, &ld, &b};
        const void *kern = spmm_kernel_for<false>(sh);
        e = ensure_dynamic_lds(kern, sh.lds);
        if (e == hipSuccess)
            e = hipLaunchKernel(kern, dim3(sh.tiles, sh.batch_tiles), dim3(sh.nw * 64), args, sh.lds, (hipStream_t)stream);
    }
    if (e != hipSuccess) { set_error(std::string("csb_spmm: ") + hipGetErrorString(e)); return CSB_EDEVICE; }
    return CSB_OK;
}

// Up to kMaxJobsPerLaunch independent products in ONE launch when they agree on the launch shape
// (same-shaped layers do); otherwise one launch each.
int spmm_strided_multi(const SpmmCall *calls, int n, int32_t batch, void *stream) {
    if (n <= 0) return CSB_OK;
    SpmmShape sh[kMaxJobsPerLaunch];
    SpmmJobs J{};
    bool same = n <= kMaxJobsPerLaunch && n > 1;
    if (same) {
        size_t lds = 0;
        unsigned tiles = 0;
        const bool many = long_tiles(calls, n);
        for (int i = 0; i < n; ++i) {
            int rc = spmm_ready(calls[i].mat);
            if (rc == CSB_OK) rc = spmm_shape(calls[i], batch, (size_t)n, many, &sh[i], &J.X[i]);
            if (rc != CSB_OK) return rc;
            same = same && sh[i].nt == sh[0].nt && sh[i].nw == sh[0].nw && sh[i].two == sh[0].two && sh[i].reg_parts == sh[0].reg_parts && sh[i].nq == sh[0].nq && sh[i].vf == sh[0].vf;
            lds = std::max(lds, sh[i].lds);
            sh[0].ks = std::max(sh[0].ks, sh[i].ks);               // (the wider pass takes any block)
            tiles = std::max(tiles, sh[i].tiles);
            J.m[i] = dev_mat(calls[i].mat);
            J.Y[i] = calls[i].Y;
            J.ldy[i] = calls[i].ldy;
        }
        // (tiles of both heights share a launch of the section's: a workgroup asks its product for its rows)
        QuadJobs QJ{};
        const csb_matrix *mats[kMaxJobsPerLaunch];
        bool quads = true, two = false, forced = false;
        for (int i = 0; i < n; ++i) {
            bool t = false;
            mats[i] = calls[i].mat;
            quads = quads && quad_source(calls[i], &QJ.X[i], &t) && (i == 0 || t == two);
            two = t;
            forced = forced || mats[i]->batch_form == kFormQuads;
        }
        const QuadShape qs = quads ? quad_shape(mats, n, batch) : QuadShape{};
        if (quads && !forced) {
            double us = 0;
            if (same) us = tile_us(sh[0], mats, n, batch);
            else for (int i = 0; i < n; ++i) us += tile_us(sh[i], &mats[i], 1, batch);
            quads = prefers_quads(qs.us, us);
        }
        if (quads) {
            for (int i = 0; i < n; ++i) {
                QJ.m[i] = quad_mat(mats[i], qs.low);
                QJ.Y[i] = calls[i].Y;
                QJ.ldy[i] = calls[i].ldy;
            }
            uint32_t b = (uint32_t)batch;
            void *args[] = {&QJ, &b};
            const void *kern = quad_kernel(qs, two, true);
            hipError_t e = ensure_dynamic_lds(kern, qs.lds);
            if (e == hipSuccess)
                e = hipLaunchKernel(kern, dim3(qs.tiles, qs.batch_tiles, (unsigned)n), dim3(qs.nw * 64), args, qs.lds, (hipStream_t)stream);
            if (e != hipSuccess) { set_error(std::string("csb_spmm: ") + hipGetErrorString(e)); return CSB_EDEVICE; }
            return CSB_OK;
        }
        if (same) {
            uint32_t b = (uint32_t)batch;
            void *args[] = {&J, &b};
            const void *kern = spmm_kernel_for<true>(sh[0]);
            hipError_t e = ensure_dynamic_lds(kern, lds);
            if (e == hipSuccess)
                e = hipLaunchKernel(kern, dim3(tiles, sh[0].batch_tiles, (unsigned)n), dim3(sh[0].nw * 64), args, lds, (hipStream_t)stream);
            if (e != hipSuccess) { set_error(std::string("csb_spmm: ") + hipGetErrorString(e)); return CSB_EDEVICE; }
            return CSB_OK;
        }
    }
    for (int i = 0; i < n; ++i) {
        const SpmmCall &c = calls[i];
        int rc = spmm_strided(c.mat, c.p0, c.n0, c.sj0, c.p1, c.sj1, c.Y, c.ldy, batch, stream);
        if (rc != CSB_OK) return rc;
    }
    return CSB_OK;
}

}  // namespace csb

namespace csb {
// Launch shape of a product of 16-bit values and 16-bit right-hand sides from the tile-based sections.
struct Spmm16Shape {
    bool reg;                // row tiles of 16 or 32 rows: the kernel that keeps its results in registers
    int nw, nq, nwr;         // wavefronts of the general form; 64-column groups and wavefronts of the other
    size_t lds;
    unsigned tiles, batch_tiles;
};
static bool spmm16_fits(const DevHeader &h) { return (size_t)h.seg_meta + 8 * (size_t)h.br * 64 * sizeof(float) <= (size_t)kLdsBudget; }
static Spmm16Shape spmm16_shape(const csb_matrix *m, int32_t batch) {
    const DevHeader &h = m->plan.hdr;
    Spmm16Shape s{};
    const size_t acc_per_wave = (size_t)h.br * 64 * sizeof(float);
    s.nw = (size_t)h.seg_meta + 16 * acc_per_wave <= (size_t)kLdsBudget ? 16 : 8;
    s.tiles = (unsigned)(h.n_nz_tiles + h.n_zero_tiles);
    s.nq = reg_columns(s.tiles, h.br, batch, true);
    s.nwr = s.nq > 1 ? 8 : s.nw;
    const size_t lds_reg = (size_t)h.seg_meta + (size_t)s.nwr * acc_per_wave + (size_t)s.nwr * 64;
    s.reg = (h.br == 16 || h.br == 32) && h.n_vals * 4 < 0x7fffff00ull && lds_reg <= (size_t)160 * 1024;
    s.lds = s.reg ? lds_reg : (size_t)h.seg_meta + (size_t)s.nw * acc_per_wave;
    s.batch_tiles = (unsigned)(s.reg ? (batch + 64 * s.nq - 1) / (64 * s.nq) : (batch + 63) / 64);
    return s;
}

// csb_spmm_bfloat / csb_spmm_half: both operands in the 16-bit format `fmt`
static int spmm_16bit(const char *who, int fmt, const csb_matrix *m, const uint16_t *d_X, int64_t ldx, float *d_Y, int64_t ldy,
                      int32_t batch, void *stream) {
    const std::string w(who);
    if (!m || !d_X || !d_Y) { set_error(w + ": NULL pointer"); return CSB_EINVAL; }
    if (batch <= 0 || ldx < batch || ldy < batch) { set_error(w + ": batch <= 0 or a leading dimension below batch"); return CSB_EINVAL; }
    if (!m->plan.valid || !m->uploaded || !m->d_buf) { set_error(w + ": matrix not planned and uploaded"); return CSB_ESTATE; }
    if (m->plan.split.active()) { set_error(w + ": matrix is planned for a GRU step"); return CSB_ESTATE; }
    const DevHeader &h = m->plan.hdr;
    if ((int)h.val_fmt != fmt) { set_error(w + ": the matrix does not store its values in this format (csb_set_value_format)"); return CSB_ESTATE; }
    // four right-hand sides per 8-byte load; 32-bit byte offsets and a 24-bit multiply
    if (batch % 4 != 0 || ldx % 4 != 0 || (uintptr_t)d_X % 8 != 0) {
        set_error(w + ": batch and ldx must be multiples of 4 and X 8-byte aligned");
        return CSB_EUNSUPPORTED;
    }
    if (ldx >= (1 << 24) || (int64_t)h.cols * ldx + batch >= (1ll << 30)) {
        set_error(w + ": sizes beyond the kernel's 32-bit offsets");
        return CSB_EUNSUPPORTED;
    }
    if (!spmm16_fits(h)) {
        set_error(w + ": the block rows are too tall for the accumulator tiles");
        return CSB_EUNSUPPORTED;
    }
    if (quad16_source(m, ldx)) {
        int32_t n = 0;
        for (int32_t n0 = 0; n0 < batch; n0 += n) {
            const PanelShape ps = panel_shape(m, batch - n0);
            n = ps.batch;
            QuadMat qm = quad_mat(m, ps.low);
            const uint16_t *x = d_X + n0;
            float *y = d_Y + n0;
            uint32_t b = (uint32_t)n, ld = (uint32_t)ldx;
            int64_t ldy_ = ldy;
            void *args[] = {&qm, &x, &ld, &y, &ldy_, &b};
            const void *kern = panel16_kernel(ps, fmt == CSB_VAL_F16);
            hipError_t e = ensure_dynamic_lds(kern, ps.lds);
            if (e == hipSuccess) e = hipLaunchKernel(kern, dim3(ps.workgroups), dim3(256 * ps.share), args, ps.lds, (hipStream_t)stream);
            if (e != hipSuccess) { set_error(w + ": " + hipGetErrorString(e)); return CSB_EDEVICE; }
        }
        return CSB_OK;
    }
    const Spmm16Shape sh = spmm16_shape(m, batch);
    DevMat dm = dev_mat(m);
    uint32_t b = (uint32_t)batch, ld = (uint32_t)ldx;
    int64_t ldy_ = ldy;
    const bool half = fmt == CSB_VAL_F16;
    if (sh.reg) {
        XSrc X{(const float *)d_X, (uint32_t)h.cols, ld, (const float *)d_X, ld};
        void *rargs[] = {&dm, &X, &d_Y, &ldy_, &b};
        const void *kern;
#define CSB_R16(NW, NH, NQ) (half ? (const void *)spmm_reg16_kernel<NW, NH, CSB_VAL_F16, NQ> : (const void *)spmm_reg16_kernel<NW, NH, CSB_VAL_BF16, NQ>)
        if (sh.nq == 2) kern = h.br == 16 ? CSB_R16(8, 1, 2) : CSB_R16(8, 2, 2);
        else if (sh.nw == 16) kern = h.br == 16 ? CSB_R16(16, 1, 1) : CSB_R16(16, 2, 1);
        else kern = h.br == 16 ? CSB_R16(8, 1, 1) : CSB_R16(8, 2, 1);
#undef CSB_R16
        hipError_t e = ensure_dynamic_lds(kern, sh.lds);
        if (e == hipSuccess)
            e = hipLaunchKernel(kern, dim3(sh.tiles, sh.batch_tiles), dim3(sh.nwr * 64), rargs, sh.lds,
                                (hipStream_t)stream);
        if (e != hipSuccess) { set_error(w + ": " + hipGetErrorString(e)); return CSB_EDEVICE; }
        return CSB_OK;
    }
    void *args[] = {&dm, &d_X, &ld, &d_Y, &ldy_, &b};
    const void *kern = sh.nw == 16 ? (half ? (const void *)spmm_bf16_kernel<16, true> : (const void *)spmm_bf16_kernel<16, false>)
                                : (half ? (const void *)spmm_bf16_kernel<8, true> : (const void *)spmm_bf16_kernel<8, false>);
    hipError_t e = ensure_dynamic_lds(kern, sh.lds);
    if (e == hipSuccess)
        e = hipLaunchKernel(kern, dim3(sh.tiles, sh.batch_tiles), dim3(sh.nw * 64), args, sh.lds,
                            (hipStream_t)stream);
    if (e != hipSuccess) { set_error(w + ": " + hipGetErrorString(e)); return CSB_EDEVICE; }
    return CSB_OK;
}
}  // namespace csb

extern "C" int csb_spmm_bfloat(const csb_matrix *m, const uint16_t *d_Xb, int64_t ldx, float *d_Y, int64_t ldy,
                               int32_t batch, void *stream) {
    return csb::spmm_16bit("csb_spmm_bfloat", CSB_VAL_BF16, m, d_Xb, ldx, d_Y, ldy, batch, stream);
}

extern "C" int csb_spmm_half(const csb_matrix *m, const uint16_t *d_Xh, int64_t ldx, float *d_Y, int64_t ldy,
                             int32_t batch, void *stream) {
    return csb::spmm_16bit("csb_spmm_half", CSB_VAL_F16, m, d_Xh, ldx, d_Y, ldy, batch, stream);
}

extern "C" int csb_spmm(const csb_matrix *m, const float *d_X, int64_t ldx, float *d_Y, int64_t ldy,
                        int32_t batch, void *d_ws, void *stream) {
    (void)d_ws;
    if (!m || !d_X || !d_Y) { csb::set_error("csb_spmm: NULL pointer"); return CSB_EINVAL; }
    if (batch <= 0 || ldx < batch || ldy < batch) { csb::set_error("csb_spmm: batch <= 0 or a leading dimension below batch"); return CSB_EINVAL; }
    if (m->plan.valid && m->plan.split.active()) { csb::set_error("csb_spmm: matrix is planned for a GRU step"); return CSB_ESTATE; }
    return csb::spmm_strided(m, d_X, (uint32_t)m->cols, ldx, d_X, ldx, d_Y, ldy, batch, stream);
}

extern "C" int csb_debug_spmm_force(csb_matrix *m, int32_t form) {
    if (!m || form < csb::kFormAuto || form > csb::kFormQuads) { csb::set_error("csb_debug_spmm_force: NULL pointer or unknown form"); return CSB_EINVAL; }
    m->batch_form = form;
    return CSB_OK;
}

extern "C" int csb_debug_spmm_form(const csb_matrix *m, int32_t batch, int32_t bits16, int32_t *form) {
    using namespace csb;
    if (!m || !form || batch <= 0) { set_error("csb_debug_spmm_form: NULL pointer or batch <= 0"); return CSB_EINVAL; }
    if (!m->plan.valid) { set_error("csb_debug_spmm_form: matrix not planned"); return CSB_ESTATE; }
    if (bits16) return csb_debug_spmm_panel(m, batch, form);
    const uint32_t cols = (uint32_t)m->plan.hdr.cols;
    SpmmCall c{m, nullptr, cols, batch, nullptr, batch, nullptr, batch};
    XSrc X;
    bool two, quads = quad_source(c, &X, &two);
    if (quads && m->batch_form != kFormQuads) {
        SpmmShape sh;
        const int rc = spmm_shape(c, batch, 1, long_tiles(&c, 1), &sh, &X);
        if (rc != CSB_OK) return rc;
        quads = prefers_quads(quad_shape(&m, 1, batch).us, tile_us(sh, &m, 1, batch));
    }
    form[0] = form[1] = form[2] = 0;
    if (quads) {
        const QuadShape qs = quad_shape(&m, 1, batch);
        form[0] = (int32_t)(qs.low ? m->plan.quad_low : m->plan.quad).tile_rows; form[1] = qs.columns; form[2] = qs.nw;
    }
    return CSB_OK;
}

extern "C" int csb_debug_spmm_panel(const csb_matrix *m, int32_t batch, int32_t *form) {
    using namespace csb;
    if (!m || !form || batch <= 0) { set_error("csb_debug_spmm_panel: NULL pointer or batch <= 0"); return CSB_EINVAL; }
    if (!m->plan.valid) { set_error("csb_debug_spmm_panel: matrix not planned"); return CSB_ESTATE; }
    form[0] = form[1] = form[2] = 0;
    if (!quad16_source(m, batch)) return CSB_OK;
    const PanelShape ps = panel_shape(m, batch);
    form[0] = ps.rows; form[1] = ps.columns; form[2] = 4 * ps.share;
    return CSB_OK;
}

extern "C" int csb_debug_spmm_columns(int64_t row_tiles, int32_t rows_per_tile, int32_t batch, int32_t bits16) {
    return 64 * csb::reg_columns((size_t)row_tiles, (uint32_t)rows_per_tile, batch, bits16 != 0);
}
