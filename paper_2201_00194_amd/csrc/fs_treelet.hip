// Traversal over byte ranks and treelets (format: fs_treelet.h), S1 + S2 of fs_score_families.
//
// One kernel does both halves of the work on a workgroup's 64-row tiles:
//   1. coding: every column's fp32 values -> ranks among the model's own thresholds, one byte
//      each, into LDS;
//   2. the walk: every lane owns a row and walks four to twelve trees side by side, two levels per
//      step, through treelets that stream through LDS in chunks; the leaf values are added in tree
//      order, so the row score has the bits of a plain sequential sum.
//
// Why this form.  The walk over fp32 tiles and 8-byte nodes (fs_traverse_lds.hip) is bound by LDS
// instructions, two per level, and its tiles leave room for two per compute unit, so that the
// leaf values of a chunk have to be parked and summed behind a barrier.  With one byte per value
// four tiles take the room of one; in long launches two wavefronts share a tile, each with half of a
// chunk's trees, and add their values from registers in turn.  A treelet entry covers two levels in
// the eight bytes of one node: three LDS and about eight vector instructions per two levels instead
// of four and eight, conflict-free feature reads, and a chunk holds four times the trees.
#include "fs_internal.h"
#include "fs_lds.h"
#include "fs_treelet.h"

namespace fs {

static __device__ __forceinline__ uint32_t lds_u8(uint32_t a) { return *FS_LDS_PTR(const uint8_t, a); }
static __device__ __forceinline__ void lds_store_u(uint32_t a, uint32_t v) { *FS_LDS_PTR(uint32_t, a) = v; }

// 1 KB from memory straight to LDS, lane l's 16 bytes at dst + 16*l.  As an instruction of its own
// and not the builtin: the compiler would take every later LDS read for a possible reader and put a
// wait in front of it.  Nothing is waited for: dma_wait() before the barrier that publishes the data.
// (The compiler's own waits stay right: they count loads in order, and more in flight than it
// knows of only makes it wait longer.)
static __device__ __forceinline__ void dma_1k(const uint8_t *src, uint32_t dst, int lane)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const uint8_t *p = src + 16 * lane;
    // (m0, the LDS address of such loads, has no other user in these kernels)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(uniform((int)dst)), "v"(p) : "memory");
#else
    (void)src; (void)dst; (void)lane;
#endif
}

static __device__ __forceinline__ uint32_t round_kb(uint32_t bytes) { return (bytes + 1023u) & ~1023u; }

// Instructions stay on their side of this point.
static __device__ __forceinline__ void keep_order()
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// All loads are there.  (The builtin, so that the compiler knows it too: behind a wait of inline assembly it put waits of
// its own in front of a batch's searches, which were waits for the values of the next batch as well.)
static __device__ __forceinline__ void dma_wait()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0)
    asm volatile("" ::: "memory");
#endif
}

template <int N> struct Int { static constexpr int value = N; };

// ---- coding ------------------------------------------------------------------------------------
// The last step of four searches, r[k] += (key[k] > x[k]).
static __device__ __forceinline__ void count_above(const float *key, const float *x, uint32_t *r)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_gt_f32_e64 %[m0], %[k0], %[x0]\n\t"
        "v_cmp_gt_f32_e64 %[m1], %[k1], %[x1]\n\t"
        "v_cmp_gt_f32_e64 %[m2], %[k2], %[x2]\n\t"
        "v_cmp_gt_f32_e64 %[m3], %[k3], %[x3]\n\t"
        "v_addc_co_u32_e64 %[r0], vcc, %[r0], 0, %[m0]\n\t"
        "v_addc_co_u32_e64 %[r1], vcc, %[r1], 0, %[m1]\n\t"
        "v_addc_co_u32_e64 %[r2], vcc, %[r2], 0, %[m2]\n\t"
        "v_addc_co_u32_e64 %[r3], vcc, %[r3], 0, %[m3]"
        : [r0] "+&v"(r[0]), [r1] "+&v"(r[1]), [r2] "+&v"(r[2]), [r3] "+&v"(r[3]), [m0] "=&s"(m0), [m1] "=&s"(m1),
          [m2] "=&s"(m2), [m3] "=&s"(m3)
        : [k0] "v"(key[0]), [k1] "v"(key[1]), [k2] "v"(key[2]), [k3] "v"(key[3]), [x0] "v"(x[0]), [x1] "v"(x[1]),
          [x2] "v"(x[2]), [x3] "v"(x[3])
        : "vcc");
#else
    (void)key; (void)x; (void)r;
#endif
}

// The same of the four tiles of a column: the ranks as the bytes of a word, written there by the additions themselves.
static __device__ __forceinline__ uint32_t count_above_bytes(const float *key, const float *x, const uint32_t *r, uint32_t zero)
{
    uint32_t word = 0;
#if defined(__HIP_DEVICE_COMPILE__)
    uint64_t m1, m2, m3;
    asm("v_cmp_gt_f32_e32 vcc, %[k0], %[x0]\n\t"
        "v_cmp_gt_f32_e64 %[m1], %[k1], %[x1]\n\t"
        "v_cmp_gt_f32_e64 %[m2], %[k2], %[x2]\n\t"
        "v_cmp_gt_f32_e64 %[m3], %[k3], %[x3]\n\t"
        "v_addc_co_u32_sdwa %[w], vcc, %[r0], %[z], vcc dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD\n\t"
        "s_mov_b64 vcc, %[m1]\n\t"
        "s_nop 0\n\t"
        "v_addc_co_u32_sdwa %[w], vcc, %[r1], %[z], vcc dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "s_mov_b64 vcc, %[m2]\n\t"
        "s_nop 0\n\t"
        "v_addc_co_u32_sdwa %[w], vcc, %[r2], %[z], vcc dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "s_mov_b64 vcc, %[m3]\n\t"
        "s_nop 0\n\t"
        "v_addc_co_u32_sdwa %[w], vcc, %[r3], %[z], vcc dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD\n\t"
        "s_nop 1"
        : [w] "=&v"(word), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3)
        : [k0] "v"(key[0]), [k1] "v"(key[1]), [k2] "v"(key[2]), [k3] "v"(key[3]), [x0] "v"(x[0]), [x1] "v"(x[1]),
          [x2] "v"(x[2]), [x3] "v"(x[3]), [r0] "v"(r[0]), [r1] "v"(r[1]), [r2] "v"(r[2]), [r3] "v"(r[3]), [z] "v"(zero)
        : "vcc");
#else
    (void)key; (void)x; (void)r; (void)zero;
#endif
    return word;
}

// A lane's offset as it is at this point: what the compiler widens to 64 bits ahead of a loop costs every load behind a
// scalar base an addition.
static __device__ __forceinline__ uint32_t here(uint32_t v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(v));
#endif
    return v;
}

// x * scale + offset, clamped to [0, 1], NaN to 0.
static __device__ __forceinline__ float fma_clamped(float x, float scale, float offset)
{
    float u = 0.0f;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("v_fma_f32 %0, %1, %2, %3 clamp" : "=v"(u) : "v"(x), "s"(scale), "v"(offset));
#endif
    return u;
}

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// One wavefront codes columns in batches of NC columns x T tiles (batch wave, wave + n_waves, ...),
// NC * T searches side by side: bucket of the value (fs_treelet.h), thresholds below the bucket, then a
// bisection of the bucket's few.  `slot` is LDS of this wavefront only: the tables of the batch in
// work and, where `halves` is 2, of the next one, `half_bytes` each.  The next batch's values (and tables)
// are on their way while a batch is searched.
//
// Vector issue is what a search costs the walks of the other workgroup, so it takes nine instructions where it took
// sixteen, and of the cheap ones (and, add, multiply-add with vector operands: 3 clocks, all others 4.5 to 5) where it can:
// LDS addresses are multiply-adds of denormal floats, which carry integers as they are; the clamp is a modifier; NaN needs no
// test; ranks are added up in their bytes; loads have a scalar base.
template <int T, int NC>
__device__ __forceinline__ void code_columns(const FamDesc &d, const TreeletSegment &m, int tile_first,
                                             int n_tiles, int wave, int n_waves, int lane, uint32_t slot,
                                             uint32_t half_bytes, int halves)
{
    constexpr int kChains = T * NC;
    static_assert(kChains % 4 == 0, "searches go in fours");
    const int C = m.n_cols, F = d.n_features;
    const uint32_t stride = (uint32_t)m.table_stride, buckets = (uint32_t)m.buckets;
    auto cols = FS_CONST(TreeletCol, m.cols);
    const int n_batches = (C + NC - 1) / NC;
    const bool rowmajor = d.layout == FS_ROWMAJOR;
    // Tiles of both layouts start 64 * F values apart.  What is left of an address is a scalar offset of the feature and
    // these of the lane's rows (row-major: the last tile's missing rows repeat the last row).
    auto X = FS_GLOBAL(const uint8_t, d.features) + (int64_t)tile_first * F * 256;
    const uint32_t feature_bytes = rowmajor ? 4u : 256u;
    uint32_t row_at[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
        row_at[t] = rowmajor ? (uint32_t)min(64 * t + lane, d.n_rows - 1 - 64 * tile_first) * 4u * (uint32_t)F
                             : (uint32_t)min(t, n_tiles - 1 - tile_first) * 256u * (uint32_t)F + 4u * (uint32_t)lane;
    auto col_of = [&](int b, int j) { return min(b * NC + j, C - 1); };   // past the last: it again
    // What a batch's searches need, asked for at once and before the wait for its values.  (Sixteen columns' do not all fit the
    // scalar registers: the forms of one and two tiles a workgroup spill 109 and 43 of them to vector registers.)
    struct Batch { float scale[NC], offset[NC]; int steps[NC]; };
    auto read_batch = [&](int b) {
        Batch q;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = col_of(b, j);
            q.scale[j] = cols[c].scale;
            q.offset[j] = cols[c].offset;
            q.steps[j] = cols[c].steps;
        }
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
        for (int j = 0; j < NC; ++j)
            asm volatile("" : "+s"(q.scale[j]), "+s"(q.offset[j]), "+s"(q.steps[j]));
#endif
        return q;
    };
    auto fetch_values = [&](int b, float (&x)[kChains]) {
        if (rowmajor) {
            // four neighbouring features of a row are one load
            bool quads = NC % 4 == 0;
#pragma unroll
            for (int j = 0; j + 1 < NC; ++j)
                quads = quads && ((j & 3) == 3 ||
                                  cols[col_of(b, j + 1)].feature == cols[col_of(b, j)].feature + 1);
            if (quads) {
#pragma unroll
                for (int j = 0; j + 3 < NC; j += 4) {
                    auto at = X + (uint32_t)cols[col_of(b, j)].feature * 4u;
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        const f32x4u v = *(__attribute__((address_space(1))) const f32x4u *)(at + here(row_at[t]));
                        x[j * T + t] = v.x;
                        x[(j + 1) * T + t] = v.y;
                        x[(j + 2) * T + t] = v.z;
                        x[(j + 3) * T + t] = v.w;
                    }
                }
                return;
            }
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            auto at = X + (uint32_t)cols[col_of(b, j)].feature * feature_bytes;
#pragma unroll
            for (int t = 0; t < T; ++t)
                x[j * T + t] = *(__attribute__((address_space(1))) const float *)(at + here(row_at[t]));
        }
    };
    auto fetch_tables = [&](int b, uint32_t to) {    // whole KB; the tables are padded behind the last one
        const uint32_t bytes = (uint32_t)NC * stride;
        for (uint32_t at = 0; at < bytes; at += 1024u)
            dma_1k(m.tables + (size_t)b * bytes + at, to + at, lane);
    };
    float last_bucket = __uint_as_float(buckets - 1u), four = 4.0f;
    uint32_t zero = 0u;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+v"(last_bucket), "+v"(four), "+v"(zero));             // vector registers: the fast forms
#endif
    auto search = [&](int b, const Batch &q, const float (&x)[kChains], uint32_t tab) {
        uint32_t r[kChains];
        float keys[NC], key[kChains];                // LDS addresses of the thresholds, as floats
        int steps = 0;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int c = col_of(b, j);
            const uint32_t lut = tab + (uint32_t)(c - b * NC) * stride;
            steps = max(steps, q.steps[j]);
            float lut_f = __uint_as_float(lut), offset = q.offset[j];
            keys[j] = __uint_as_float(lut + buckets);
#if defined(__HIP_DEVICE_COMPILE__)
            asm("" : "+v"(lut_f), "+v"(keys[j]), "+v"(offset));
#endif
#pragma unroll
            for (int t = 0; t < T; ++t)
                r[j * T + t] = lds_u8(__float_as_uint(__builtin_fmaf(fma_clamped(x[j * T + t], q.scale[j], offset), last_bucket, lut_f)));
        }
        // threshold r + 2^s - 1 of the column; those past the last are NaN and never counted
        auto probe = [&](int s) {
#pragma unroll
            for (int j = 0; j < NC; ++j)
#pragma unroll
                for (int t = 0; t < T; ++t)
                    key[j * T + t] = lds_f(__float_as_uint(__builtin_fmaf(__uint_as_float(r[j * T + t]), four, keys[j])) + (4u << s) - 4u);
        };
        auto step = [&](int s) {
#pragma unroll
            for (int k = 0; k < kChains; ++k)
                r[k] += key[k] > x[k] ? 1u << s : 0u;
        };
        for (int s = steps - 1; s > 1; --s) {
            probe(s);
            step(s);
        }
        if (steps > 1) {
            probe(1);
            step(1);
        }
        if (T == 4 && steps > 0) {
            probe(0);
#pragma unroll
            for (int j = 0; j < NC; ++j)
                lds_store_u((uint32_t)col_of(b, j) * 256u + 4u * (uint32_t)lane,
                            count_above_bytes(key + 4 * j, x + 4 * j, r + 4 * j, zero));
            return;
        }
        if (steps > 0) {
            probe(0);
#pragma unroll
            for (int k = 0; k < kChains; k += 4)
                count_above(key + k, x + k, r + k);
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            uint32_t word = r[j * T];
#pragma unroll
            for (int t = 1; t < T; ++t)
                word |= r[j * T + t] << (8 * t);
            lds_store_u((uint32_t)col_of(b, j) * 256u + 4u * (uint32_t)lane, word);
        }
    };
    float xa[kChains], xb[kChains];                  // taken in turn
    const uint32_t slot1 = halves == 2 ? slot + half_bytes : slot;
    if (wave < n_batches) {
        fetch_tables(wave, slot);
        fetch_values(wave, xa);
    }
    for (int b = wave; b < n_batches; b += 2 * n_waves) {
        const int b1 = b + n_waves, b2 = b1 + n_waves;
        const Batch q = read_batch(b);
        dma_wait();
        if (b1 < n_batches) {
            if (halves == 2)
                fetch_tables(b1, slot1);
            fetch_values(b1, xb);
        }
        search(b, q, xa, slot);
        if (b1 >= n_batches)
            break;
        if (halves != 2)
            fetch_tables(b1, slot1);
        const Batch q1 = read_batch(b1);
        dma_wait();
        if (b2 < n_batches) {
            if (halves == 2)
                fetch_tables(b2, slot);
            fetch_values(b2, xa);
        }
        search(b1, q1, xb, slot1);
        if (halves != 2 && b2 < n_batches)
            fetch_tables(b2, slot);
    }
}

// ---- the walk ----------------------------------------------------------------------------------
// The vector instructions are what binds the walk (the LDS instructions come second), so the two
// decisions of a step are written out: eight instructions per walk and step, where the compiler's own
// code takes twelve (it has no add with carry-in for 2*i + c, and shifts and masks what the sub-dword
// operands pick for free).  Four walks per block keep two instructions between a compare and the
// readers of its mask, which this hardware wants.
//
// First decision of four walks: x[k] >= rank of w0[k]?  c[k] = the chosen child's half of w1[k],
// i[k] = 2 * block + decision, at[k] = LDS address of the child's column for this row.
static __device__ __forceinline__ void decide_first(const uint32_t *x, const uint32_t *w0, const uint32_t *w1,
                                                    uint32_t row, uint32_t *c, uint32_t *i, uint32_t *at)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint64_t m1, m2, m3;
    asm("v_cmp_ge_u32_sdwa vcc, %[x0], %[a0] src0_sel:DWORD src1_sel:BYTE_0\n\t"
        "v_cmp_ge_u32_sdwa %[m1], %[x1], %[a1] src0_sel:DWORD src1_sel:BYTE_0\n\t"
        "v_cmp_ge_u32_sdwa %[m2], %[x2], %[a2] src0_sel:DWORD src1_sel:BYTE_0\n\t"
        "v_cmp_ge_u32_sdwa %[m3], %[x3], %[a3] src0_sel:DWORD src1_sel:BYTE_0\n\t"
        "v_cndmask_b32_sdwa %[c0], %[b0], %[b0], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n\t"
        "v_addc_co_u32_sdwa %[i0], vcc, %[a0], %[a0], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_1\n\t"
        "s_mov_b64 vcc, %[m1]\n\t"
        "v_and_or_b32 %[n0], %[c0], %[mask], %[row]\n\t"
        "v_cndmask_b32_sdwa %[c1], %[b1], %[b1], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n\t"
        "v_addc_co_u32_sdwa %[i1], vcc, %[a1], %[a1], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_1\n\t"
        "s_mov_b64 vcc, %[m2]\n\t"
        "v_and_or_b32 %[n1], %[c1], %[mask], %[row]\n\t"
        "v_cndmask_b32_sdwa %[c2], %[b2], %[b2], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n\t"
        "v_addc_co_u32_sdwa %[i2], vcc, %[a2], %[a2], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_1\n\t"
        "s_mov_b64 vcc, %[m3]\n\t"
        "v_and_or_b32 %[n2], %[c2], %[mask], %[row]\n\t"
        "v_cndmask_b32_sdwa %[c3], %[b3], %[b3], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n\t"
        "v_addc_co_u32_sdwa %[i3], vcc, %[a3], %[a3], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_1\n\t"
        "v_and_or_b32 %[n3], %[c3], %[mask], %[row]"
        : [c0] "=&v"(c[0]), [c1] "=&v"(c[1]), [c2] "=&v"(c[2]), [c3] "=&v"(c[3]), [i0] "=&v"(i[0]),
          [i1] "=&v"(i[1]), [i2] "=&v"(i[2]), [i3] "=&v"(i[3]), [n0] "=&v"(at[0]), [n1] "=&v"(at[1]),
          [n2] "=&v"(at[2]), [n3] "=&v"(at[3]), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3)
        : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [a0] "v"(w0[0]), [a1] "v"(w0[1]),
          [a2] "v"(w0[2]), [a3] "v"(w0[3]), [b0] "v"(w1[0]), [b1] "v"(w1[1]), [b2] "v"(w1[2]), [b3] "v"(w1[3]),
          [mask] "s"(0xFF00u), [row] "v"(row)
        : "vcc");
#else
    (void)x; (void)w0; (void)w1; (void)row; (void)c; (void)i; (void)at;
#endif
}

// Second decision of four walks: i[k] = 2 * i[k] + (x[k] >= rank of c[k]).
static __device__ __forceinline__ void decide_second(const uint32_t *x, const uint32_t *c, uint32_t *i)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint64_t m0, m1, m2, m3;
    asm("v_cmp_ge_u32_sdwa %[m0], %[x0], %[c0] src0_sel:DWORD src1_sel:BYTE_0\n\t"
        "v_cmp_ge_u32_sdwa %[m1], %[x1], %[c1] src0_sel:DWORD src1_sel:BYTE_0\n\t"
        "v_cmp_ge_u32_sdwa %[m2], %[x2], %[c2] src0_sel:DWORD src1_sel:BYTE_0\n\t"
        "v_cmp_ge_u32_sdwa %[m3], %[x3], %[c3] src0_sel:DWORD src1_sel:BYTE_0\n\t"
        "v_addc_co_u32_e64 %[i0], vcc, %[i0], %[i0], %[m0]\n\t"
        "v_addc_co_u32_e64 %[i1], vcc, %[i1], %[i1], %[m1]\n\t"
        "v_addc_co_u32_e64 %[i2], vcc, %[i2], %[i2], %[m2]\n\t"
        "v_addc_co_u32_e64 %[i3], vcc, %[i3], %[i3], %[m3]"
        : [i0] "+&v"(i[0]), [i1] "+&v"(i[1]), [i2] "+&v"(i[2]), [i3] "+&v"(i[3]), [m0] "=&s"(m0), [m1] "=&s"(m1),
          [m2] "=&s"(m2), [m3] "=&s"(m3)
        : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [c0] "v"(c[0]), [c1] "v"(c[1]),
          [c2] "v"(c[2]), [c3] "v"(c[3])
        : "vcc");
#else
    (void)x; (void)c; (void)i;
#endif
}

// K trees (a multiple of four) of the chunk at `buf`, roots j.., for this lane's row (`row` =
// 4*lane + tile).  Leaves the values in v and their value indices in i.
template <int K>
__device__ __forceinline__ void treelet_walk(uint32_t buf, uint32_t val, int j, int steps, uint32_t row,
                                             uint32_t (&i)[K], float (&v)[K])
{
    uint32_t w0[K], w1[K];
    const uint32_t root = buf + 8u * (uint32_t)j;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const u32x2 nd = lds_u2(root + 8u * (uint32_t)k);
        w0[k] = nd.x;
        w1[k] = nd.y;
    }
    // Block by block (of four walks), so that a block's reads are in flight while the others decide.
    // 8 * i + buf as a float multiply-add: denormal numbers carry the integers as they are, and this is
    // one of the instructions that run at twice the rate of an integer shift-and-add.
    float buf_f = __uint_as_float(buf), val_f = __uint_as_float(val), eight = 8.0f, four = 4.0f;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+v"(buf_f), "+v"(val_f), "+v"(eight), "+v"(four));     // vector registers: the fast form
#endif
    uint32_t x[K], c[K], at[K];
    auto columns = [&](int k) {
#pragma unroll
        for (int u = k; u < k + 4; ++u)
            x[u] = lds_u8((w0[u] & 0xFF00u) | row);
        keep_order();
    };
    auto first = [&](int k) {
        decide_first(x + k, w0 + k, w1 + k, row, c + k, i + k, at + k);
#pragma unroll
        for (int u = k; u < k + 4; ++u)
            x[u] = lds_u8(at[u]);
        keep_order();
    };
    for (int s = steps; s > 1; --s) {
#pragma unroll
        for (int k = 0; k < K; k += 4)
            columns(k);
#pragma unroll
        for (int k = 0; k < K; k += 4)
            first(k);
#pragma unroll
        for (int k = 0; k < K; k += 4) {
            decide_second(x + k, c + k, i + k);
#pragma unroll
            for (int u = k; u < k + 4; ++u) {
                const u32x2 nd = lds_u2(__float_as_uint(__builtin_fmaf(__uint_as_float(i[u]), eight, buf_f)));
                w0[u] = nd.x;
                w1[u] = nd.y;
            }
            keep_order();
        }
    }
#pragma unroll
    for (int k = 0; k < K; k += 4)
        columns(k);
#pragma unroll
    for (int k = 0; k < K; k += 4)
        first(k);
#pragma unroll
    for (int k = 0; k < K; k += 4) {
        decide_second(x + k, c + k, i + k);
#pragma unroll
        for (int u = k; u < k + 4; ++u)
            v[u] = lds_f(__float_as_uint(__builtin_fmaf(__uint_as_float(i[u]), four, val_f)));
        keep_order();
    }
}

template <int K>
__device__ __forceinline__ void dump_leaves(uint16_t *leaf_row, const TreeletModel &m, const TreeletChunk &h,
                                            int j, const uint32_t (&i)[K])
{
    if (!leaf_row)
        return;
    auto ids = FS_GLOBAL(const uint16_t, m.ids + h.id_off);
    auto out = FS_GLOBAL(uint16_t, leaf_row + h.first_tree);
#pragma unroll
    for (int k = 0; k < K; ++k)
        if ((uint32_t)(j + k) < h.n_real)
            out[j + k] = ids[i[k]];
}

static __device__ __forceinline__ TreeletChunk load_chunk(const TreeletChunk *p_)
{
    auto p = FS_CONST(TreeletChunk, p_);
    TreeletChunk h;
    h.byte_off = p->byte_off;
    h.bytes = p->bytes;
    h.n_trees = p->n_trees;
    h.first_tree = p->first_tree;
    h.n_real = p->n_real;
    h.val_off = p->val_off;
    h.steps = p->steps;
    h.id_off = p->id_off;
    return h;
}

static __device__ __forceinline__ TreeletModel load_model(const TreeletModel *p_)
{
    auto p = FS_CONST(TreeletModel, p_);
    TreeletModel m;
    m.image = p->image;
    m.chunks = p->chunks;
    m.segments = p->segments;
    m.ids = p->ids;
    m.n_segments = p->n_segments;
    m.most_cols = p->most_cols;
    m.buf_bytes = p->buf_bytes;
    m.max_trees = p->max_trees;
    return m;
}

static __device__ __forceinline__ TreeletSegment load_segment(const TreeletSegment *p_)
{
    auto p = FS_CONST(TreeletSegment, p_);
    TreeletSegment g;
    g.cols = p->cols;
    g.tables = p->tables;
    g.n_cols = p->n_cols;
    g.buckets = p->buckets;
    g.table_stride = p->table_stride;
    g.first_chunk = p->first_chunk;
    g.n_chunks = p->n_chunks;
    return g;
}

static __device__ __forceinline__ int treelet_family(const FamDesc *descs, int n_families, int launch)
{
    int lo = 0, hi = n_families - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (descs[mid].tl_block0[launch] <= (int)blockIdx.x)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

static __device__ __forceinline__ void fetch_chunk(const TreeletModel &m, const TreeletChunk &h, uint32_t dst,
                                                   int wave, int n_waves, int lane)
{
    for (uint32_t at = 1024u * (uint32_t)wave; at < h.bytes; at += 1024u * (uint32_t)n_waves)
        dma_1k(m.image + h.byte_off + at, dst + at, lane);
}

// Long launches: four tiles and eight wavefronts; two workgroups share a compute unit, so that one
// walks while the other codes or waits at a barrier.  Two wavefronts share a tile: the first walks
// the front half of a chunk's trees, the second the back half (in rounds of kTreeletRound, side by
// side).  The row's running sum goes to and fro between them through LDS: the first adds its values
// before the barrier that ends the walks, the second behind it, while the next chunk travels from memory to
// LDS; a second barrier publishes both.  (The latency of that is the other workgroup's time: the LDS is what
// is short, and a chunk that waits in registers and is stored from there takes more of it: eight families of 300
// perfect trees of depth 8 1024 us instead of 1000, 64 of deep irregular trees 2211 instead of 2161.)  (One wavefront per tile needs no
// hand-over, but eight wavefronts per compute unit leave the vector units half idle: 3.15 ms on thirty
// families of power-law size, 200 irregular trees of depth 8, against 2.30 ms then; the float-threshold kernel took
// 3.62 ms there.)  Vector issue and the LDS bound this kernel alike: there it issues 1.02e9 vector instructions, which
// at four clocks are 78 % of the SIMDs' clocks, and a compute unit an LDS instruction every 4.2 clocks, where
// conflict-free ones take 2.4.  (Leaf values read from memory instead of the LDS: 2.36 ms, 2.26 so.)
// LDS: [columns][chunk][running sums of the tiles, by hand-over]; the coder's tables are where the
// chunks will be.
constexpr int kPairTiles = 4;
constexpr int kPairWaves = 2 * kPairTiles;

template <bool DUMP>
__global__ void __launch_bounds__(64 * kPairWaves, 4)
treelet_pair_kernel(const FamDesc *__restrict__ descs, int n_families, int launch)
{
    const FamDesc &d = descs[treelet_family(descs, n_families, launch)];
    const TreeletModel m = load_model(d.tl);
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int my_tile = wave % kPairTiles;
    const bool back = wave >= kPairTiles;
    const int n_tiles = row_tiles(d.n_rows);
    const int tile_first = (blockIdx.x - d.tl_block0[launch]) * kPairTiles;
    const uint32_t buf = (uint32_t)m.most_cols * 256u;
    const uint32_t sum_at = (uint32_t)kTreeletLds - kTreeletSumBytes + 256u * (uint32_t)my_tile + 4u * (uint32_t)lane;
    constexpr uint32_t kBack = 256u * (uint32_t)kPairTiles;      // sums of the back half's wavefronts
    const uint32_t r = (uint32_t)(tile_first + my_tile) * 64u + (uint32_t)lane;   // (past 2^31 in missing tiles)
    const uint32_t row = 4u * (uint32_t)lane + (uint32_t)my_tile;
    float acc = d.bias;
    uint16_t *leaf_row = nullptr;
    if (DUMP) {
        if (d.leaf_idx && r < (uint32_t)d.n_rows)
            leaf_row = d.leaf_idx + (int64_t)r * d.n_trees;
    }

    for (int si = 0; si < m.n_segments; ++si) {
        const TreeletSegment g = load_segment(m.segments + si);
        // double-buffered tables of as many columns as fit where the chunks will be
        const uint32_t room = (uint32_t)kTreeletLds - kTreeletSumBytes - buf;
        const uint32_t half4 = round_kb(4u * (uint32_t)g.table_stride), half2 = round_kb(2u * (uint32_t)g.table_stride),
                       half1 = round_kb((uint32_t)g.table_stride);
        constexpr uint32_t kHalves = 2u * (uint32_t)kPairWaves;
        if (kHalves * half4 <= room)
            code_columns<kPairTiles, 4>(d, g, tile_first, n_tiles, wave, kPairWaves, lane, buf + 2u * half4 * (uint32_t)wave, half4, 2);
        else if (kHalves * half2 <= room)
            code_columns<kPairTiles, 2>(d, g, tile_first, n_tiles, wave, kPairWaves, lane, buf + 2u * half2 * (uint32_t)wave, half2, 2);
        else {                                       // the packer sees to it that one buffer fits
            const uint32_t halves = kHalves * half1 <= room ? 2u : 1u;
            code_columns<kPairTiles, 1>(d, g, tile_first, n_tiles, wave, kPairWaves, lane, buf + halves * half1 * (uint32_t)wave, half1, (int)halves);
        }
        if (si == 0)
            lds_store_f(sum_at + kBack, acc);        // (both wavefronts of a tile, the same value)
        __syncthreads();                             // columns coded, tables free
        const TreeletChunk *chunks = m.chunks + g.first_chunk;
        TreeletChunk h = load_chunk(chunks), hn = load_chunk(chunks + min(1, g.n_chunks - 1));
        fetch_chunk(m, h, buf, wave, kPairWaves, lane);
        dma_wait();
        __syncthreads();

        for (int c = 0; c < g.n_chunks; ++c) {
            const bool more = c + 1 < g.n_chunks;
            const uint32_t val = buf + h.val_off;
            const int units = (int)h.n_trees / kTreeletUnit, front = (units + 1) / 2;
            int j0 = back ? front * kTreeletUnit : 0;
            int left = back ? units - front : front;             // in units
            float v[kTreeletRound], v1[kTreeletRound];           // this round's values, and those of the round before
#pragma unroll
            for (int k = 0; k < kTreeletRound; ++k)
                v[k] = v1[k] = -0.0f;                            // adding -0 changes nothing
            if (!back)
                acc = lds_f(sum_at + kBack);
            for (;;) {
                auto walk = [&](auto walks) {
                    constexpr int K = decltype(walks)::value;
                    uint32_t i[K];
                    float vk[K];
                    treelet_walk<K>(buf, val, j0, (int)h.steps, row, i, vk);
#pragma unroll
                    for (int k = 0; k < kTreeletRound; ++k)
                        v[k] = k < K ? vk[k] : -0.0f;
                    if (DUMP)
                        dump_leaves<K>(leaf_row, m, h, j0, i);
                };
                switch (left) {
                case 0: break;
                case 1: walk(Int<4>()); break;
                case 2: walk(Int<8>()); break;
                default: walk(Int<kTreeletRound>());
                }
                left -= kTreeletRound / kTreeletUnit;
                j0 += kTreeletRound;
                if (left <= 0)
                    break;
                if (!back) {
#pragma unroll
                    for (int k = 0; k < kTreeletRound; ++k)
                        acc = acc + v[k];
                } else {
#pragma unroll
                    for (int k = 0; k < kTreeletRound; ++k)
                        v1[k] = v[k];
                }
            }
            // The header after next, here where its latency passes behind the hand-over: a scalar load
            // on its way during a walk would turn every wait of the walk into a wait for everything.
            const TreeletChunk hnn = load_chunk(chunks + min(c + 2, g.n_chunks - 1));
            if (!back) {
#pragma unroll
                for (int k = 0; k < kTreeletRound; ++k)
                    acc = acc + v[k];
                lds_store_f(sum_at, acc);
            }
            __syncthreads();
            if (more)                                // every walk of this chunk is done
                fetch_chunk(m, hn, buf, wave, kPairWaves, lane);
            if (back) {
                acc = lds_f(sum_at);
#pragma unroll
                for (int k = 0; k < kTreeletRound; ++k)
                    acc = acc + v1[k];
#pragma unroll
                for (int k = 0; k < kTreeletRound; ++k)
                    acc = acc + v[k];
                lds_store_f(sum_at + kBack, acc);
            }
            if (more) {
                dma_wait();
                __syncthreads();
            }
            h = hn;
            hn = hnn;
        }
    }
    if (back && r < (uint32_t)d.n_rows)
        FS_GLOBAL(float, d.row_score)[r] = acc;
}

// Short launches: T tiles and S wavefronts per tile, which split the trees of a chunk in units of four,
// park the leaf values, and leave the sum to one wavefront per tile.  What bounds a launch of a
// few workgroups is latency, so where LDS takes two chunks and their value rows the next chunk travels
// while one is walked, and one chunk's values are summed while the next is walked (one barrier a
// chunk); the first chunk travels during the coding.
// LDS: [columns][chunk buffers][value rows: [tree][tile][lane], per buffer]; the coder's tables lie
// over what follows the first buffer.
template <int T, int S, bool DUMP>
__global__ void __launch_bounds__(64 * T * S)
treelet_spread_kernel(const FamDesc *__restrict__ far, int n_families, int launch, NearFams)
{
    const FamDesc *descs = where_descs(far, offsetof(FamArgs2, near));
    constexpr int kWaves = T * S;
    const FamDesc &d = descs[treelet_family(descs, n_families, launch)];
    const TreeletModel m = load_model(d.tl);
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int my_tile = wave % T, my_slot = wave / T;
    const int n_tiles = row_tiles(d.n_rows);
    const int tile_first = (blockIdx.x - d.tl_block0[launch]) * T;
    const uint32_t area = (uint32_t)m.most_cols * 256u, chunk_bytes = (uint32_t)m.buf_bytes;
    constexpr uint32_t kValStride = 256u * (uint32_t)T;
    const uint32_t row_bytes = (uint32_t)m.max_trees * kValStride;
    const uint32_t room = (uint32_t)kTreeletLdsWhole - area;     // one buffer and its rows fit by packing
    const bool two = 2u * (chunk_bytes + row_bytes) <= room;
    const uint32_t val_rows = area + (two ? 2u : 1u) * chunk_bytes;
    const uint32_t r = (uint32_t)(tile_first + my_tile) * 64u + (uint32_t)lane;   // (past 2^31 in missing tiles)
    const uint32_t row = 4u * (uint32_t)lane + (uint32_t)my_tile;
    float acc = d.bias;
    uint16_t *leaf_row = nullptr;
    if (DUMP) {
        if (d.leaf_idx && r < (uint32_t)d.n_rows)
            leaf_row = d.leaf_idx + (int64_t)r * d.n_trees;
    }
    for (int si = 0; si < m.n_segments; ++si) {
        const TreeletSegment g = load_segment(m.segments + si);
        const TreeletChunk *chunks = m.chunks + g.first_chunk;
        TreeletChunk h = load_chunk(chunks);
        {
            // tables of eight (four on two tiles, two on four) columns' searches if they fit beside the first
            // chunk, else of fewer over its place
            constexpr int kWide = 16 / T, kNarrow = 4 / T;
            const uint32_t wide = round_kb((uint32_t)(kWide * g.table_stride)), narrow = round_kb((uint32_t)(kNarrow * g.table_stride));
            if (kWaves * wide + chunk_bytes <= room) {
                fetch_chunk(m, h, area, wave, kWaves, lane);
                code_columns<T, kWide>(d, g, tile_first, n_tiles, wave, kWaves, lane,
                                       area + chunk_bytes + wide * (uint32_t)wave, wide, 1);
            } else {
                const int halves = 2u * kWaves * narrow <= room ? 2 : 1;
                code_columns<T, kNarrow>(d, g, tile_first, n_tiles, wave, kWaves, lane,
                                         area + (uint32_t)halves * narrow * (uint32_t)wave, narrow, halves);
                __syncthreads();
                fetch_chunk(m, h, area, wave, kWaves, lane);
            }
        }
        dma_wait();
        __syncthreads();
        for (int c = 0; c < g.n_chunks; ++c) {
            const uint32_t odd = two ? (uint32_t)(c & 1) : 0u;
            const bool more = c + 1 < g.n_chunks;
            const TreeletChunk hn = load_chunk(chunks + min(c + 1, g.n_chunks - 1));
            if (two && more)                         // its buffer's last readers passed a barrier since
                fetch_chunk(m, hn, area + (odd ^ 1u) * chunk_bytes, wave, kWaves, lane);
            const uint32_t buf = area + odd * chunk_bytes, val = buf + h.val_off;
            const uint32_t my_val = val_rows + odd * row_bytes + 256u * (uint32_t)my_tile + 4u * (uint32_t)lane;
            const int units = (int)h.n_trees / kTreeletUnit;
            int u = my_slot * units / S;
            const int end = (my_slot + 1) * units / S;
            while (u < end) {
                const int j = u * kTreeletUnit;
                const uint32_t at = my_val + (uint32_t)j * kValStride;
                auto walk = [&](auto walks) {
                    constexpr int K = decltype(walks)::value;
                    uint32_t i[K];
                    float v[K];
                    treelet_walk<K>(buf, val, j, (int)h.steps, row, i, v);
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        lds_store_f(at + (uint32_t)k * kValStride, v[k]);
                    if (DUMP)
                        dump_leaves<K>(leaf_row, m, h, j, i);
                    u += K / kTreeletUnit;
                };
                if (u + 2 <= end)
                    walk(Int<8>());
                else
                    walk(Int<4>());
            }
            dma_wait();
            __syncthreads();                         // values parked, next chunk there (two buffers)
            if (!two && more)                        // every walk of this chunk is done
                fetch_chunk(m, hn, area, wave, kWaves, lane);
            if (my_slot == 0)
                ordered_add_n(acc, my_val, kValStride, units * kTreeletUnit);
            if (!two) {
                dma_wait();
                __syncthreads();
            }
            h = hn;
        }
        if (two && si + 1 < m.n_segments)
            __syncthreads();                         // the next segment's tables overwrite the last values
    }
    if (my_slot == 0 && r < (uint32_t)d.n_rows)
        FS_GLOBAL(float, d.row_score)[r] = acc;
}

// `near`: the descriptors by value, for kernels that take them so.
template <class Kernel, class... Near>
static int launch_form(Kernel kernel, int form, int threads, int lds, const Descs<FamDesc> &descs,
                       int launch, int total_blocks, hipStream_t stream, Near... near)
{
    static bool configured[16][kTreeletForms * 2] = {};
    int dev = 0;
    FS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 16 || !configured[dev][form]) {
        // the kernels address LDS from 0: no static LDS
        hipFuncAttributes attr;
        FS_HIP(hipFuncGetAttributes(&attr, (const void *)kernel));
        if (attr.sharedSizeBytes != 0)
            return fail(FS_EDEVICE, "a treelet kernel was built with %zu bytes of static LDS",
                        (size_t)attr.sharedSizeBytes);
        FS_HIP(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        if (dev >= 0 && dev < 16)
            configured[dev][form] = true;
    }
    hipLaunchKernelGGL(kernel, dim3(total_blocks), dim3(threads), lds, stream, descs.far, descs.n, launch, near...);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_hip(e, "treelet kernel launch");
    return FS_OK;
}

int launch_treelet(const Descs<FamDesc> &descs, int launch, int form, int total_blocks, bool dump,
                   hipStream_t stream)
{
    const NearFams near = near_descs<NearFams>(descs);
    const int id = 2 * form + (dump ? 1 : 0);
    switch (id) {
    case 2 * kTreeletPair:
        return launch_form(treelet_pair_kernel<false>, id, 64 * kPairWaves, kTreeletLds, descs, launch, total_blocks, stream);
    case 2 * kTreeletPair + 1:
        return launch_form(treelet_pair_kernel<true>, id, 64 * kPairWaves, kTreeletLds, descs, launch, total_blocks, stream);
    case 2 * kTreeletSpread4:
        return launch_form(treelet_spread_kernel<4, 3, false>, id, 768, kTreeletLdsWhole, descs, launch, total_blocks, stream, near);
    case 2 * kTreeletSpread4 + 1:
        return launch_form(treelet_spread_kernel<4, 3, true>, id, 768, kTreeletLdsWhole, descs, launch, total_blocks, stream, near);
    case 2 * kTreeletSpread2:
        return launch_form(treelet_spread_kernel<2, 6, false>, id, 768, kTreeletLdsWhole, descs, launch, total_blocks, stream, near);
    case 2 * kTreeletSpread2 + 1:
        return launch_form(treelet_spread_kernel<2, 6, true>, id, 768, kTreeletLdsWhole, descs, launch, total_blocks, stream, near);
    case 2 * kTreeletSpread1:
        return launch_form(treelet_spread_kernel<1, 12, false>, id, 768, kTreeletLdsWhole, descs, launch, total_blocks, stream, near);
    case 2 * kTreeletSpread1 + 1:
        return launch_form(treelet_spread_kernel<1, 12, true>, id, 768, kTreeletLdsWhole, descs, launch, total_blocks, stream, near);
    default:
        return fail(FS_EUNSUPPORTED, "unknown treelet form %d", form);
    }
}

}  // namespace fs
