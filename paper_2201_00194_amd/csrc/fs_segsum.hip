// Per-program segmented sum of row scores (CSR offsets), order preserving.
//
// A candidate program's score is the sum of the model's outputs over its statement rows;
// the additions are sequential fp32 in ascending row order starting from +0, so the
// result is reproducible bit for bit.  One lane owns one program.  A wavefront takes the contiguous rows of its 64
// programs to LDS, a window at a time with coalesced loads that are all in flight at once, and every lane adds its own from
// there, in order.  (Rows read from memory by each lane for itself, four at a time, were a chain of up to 16 latencies of
// lines that 64 lanes share with nobody: 200 000 programs of 1 to 64 rows 32.5 us, sixteen at
// a time 26.3, so 16.9; 80 000 of 16 rows 7.7 and 5.3.)
// Two kinds of wavefronts read their rows without LDS, see below: those of long programs, where few lanes have rows in a
// window, and those of programs of one or two rows, where it is a detour.
#include "fs_internal.h"
#include "fs_lds.h"
#include "fs_runs.h"

namespace fs {

// Rows in LDS of a wavefront; a word of padding every 16 keeps programs of 16, 32 ... rows off each other's banks.  Calls of
// at most four rows a program on average have windows of 256: 34 KB of LDS a workgroup leave a compute unit 16
// wavefronts.  The call with one tree, 1.2 M programs of a row 53.0 us with windows of 2048, 47.7 with 256; 400 000 of
// three 45.0 and 43.3; from six rows on no difference.
constexpr int kSegWindow = 2048, kSegShortWindow = 256;
constexpr int kSegShortRows = 4;
// Every window takes as long as its longest program, so programs are long where windows times their rows are more than
// this: 15 000 programs of 80 rows (three windows, 240) 51.3 us from LDS and 51.5 by lanes, 9375 of 128 (512) 59.5
// and 56.1, 4687 of 256 186 and 70, 40 of 1000 519 and 43; 100 000 of 1 to 128 rows (384) 201 and 197.
constexpr int kSegLong = 288, kSegShortLong = 64;
// 1.2 M programs of a row 46.1 us by lanes instead of 47.7, 600 000 of two 44.6 and 45.0, 300 000 of four 43.9 and 44.0.
constexpr int kSegDirect = 2;
constexpr int kSegLoads = 16;            // loads in flight per lane
constexpr int kSegAdds = 8;              // LDS reads in flight per lane
template <int N> struct SegInt { static constexpr int value = N; };
__device__ __forceinline__ int seg_word(int i) { return i + (i >> 4); }

// What this wavefront has done in LDS is done.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int WINDOW>
__global__ void __launch_bounds__(kSegProgsPerBlock)
segsum_kernel(const FamDesc *__restrict__ far, int n_families, NearFams)
{
    const FamDesc *descs = where_descs(far, offsetof(FamArgs1, near));
    int lo = 0, hi = n_families - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (descs[mid].seg_block0 <= (int)blockIdx.x)
            lo = mid;
        else
            hi = mid - 1;
    }
    const FamDesc &d = descs[lo];
    const int n_programs = d.n_programs;
    const int32_t *__restrict__ off = d.prog_off;
    const float *__restrict__ rs = d.row_score;
    const int lane = threadIdx.x & 63;
    const int p_wave = (blockIdx.x - d.seg_block0) * kSegProgsPerBlock + (threadIdx.x & ~63);
    if (p_wave >= n_programs)
        return;                                     // whole wavefront leaves together
    const int p = p_wave + lane;
    const int p_last = p_wave + min(64, n_programs - p_wave);
    const int n_rows = d.n_rows;
    // Lanes past the family's last program own no rows but load for the others.
    int begin = 0, end = 0;
    if (p < n_programs) {
        begin = min(max(off[p], 0), n_rows);
        end = min(max(off[p + 1], begin), n_rows);
    }
    const int w_begin = min(max(off[p_wave], 0), n_rows);
    const int w_end = min(max(off[p_last], w_begin), n_rows);

    __shared__ float s_rows[kSegProgsPerBlock / 64][WINDOW + WINDOW / 16];
    float *const mine = s_rows[threadIdx.x >> 6];
    auto rows = FS_GLOBAL(const float, rs);
    float acc = 0.0f;
    const int windows = (int)(((uint32_t)(w_end - w_begin) + WINDOW - 1) / WINDOW);
    auto own_rows = [&](auto loads) {                            // every lane reads its own
        constexpr int L = decltype(loads)::value;
        in_runs<L>(begin, end, [&](int r, int left) {
            float v[L];
#pragma unroll
            for (int u = 0; u < L; ++u)
                v[u] = rows[r + min(u, left - 1)];
#pragma unroll
            for (int u = 0; u < L; ++u)
                acc = u < left ? acc + v[u] : acc;
        });
    };
    if (windows > 1 && __any((int64_t)(end - begin) * windows > (WINDOW == kSegWindow ? kSegLong : kSegShortLong))) {
        own_rows(SegInt<kSegLoads>());
    } else if (WINDOW == kSegShortWindow && !__any(end - begin > kSegDirect)) {
        own_rows(SegInt<kSegDirect>());
    } else {
        in_runs<WINDOW>(w_begin, w_end, [&](int base, int left) {
            constexpr int L = WINDOW / 64 < kSegLoads ? WINDOW / 64 : kSegLoads;
            const int n = min(WINDOW, left);
            for (int at = lane; at < n; at += 64 * L) {
                float v[L];
#pragma unroll
                for (int u = 0; u < L; ++u)
                    v[u] = rows[base + min(at + 64 * u, n - 1)];
#pragma unroll
                for (int u = 0; u < L; ++u)
                    mine[seg_word(at + 64 * u)] = v[u];    // (at + 64 * u < WINDOW)
            }
            wave_sync();
            const int from = max(begin - base, 0), to = min(end - base, n);
            for (int i = from; i < to; i += kSegAdds) {
                float v[kSegAdds];
#pragma unroll
                for (int u = 0; u < kSegAdds; ++u)
                    v[u] = mine[seg_word(min(i + u, to - 1))];
#pragma unroll
                for (int u = 0; u < kSegAdds; ++u)
                    acc = i + u < to ? acc + v[u] : acc;
            }
            wave_sync();                                   // read before the next window is written
        });
    }
    if (p < n_programs)
        d.prog_score[p] = acc;
}

template <int WINDOW>
static int launch_window(const Descs<FamDesc> &descs, int total_blocks, hipStream_t stream)
{
    hipLaunchKernelGGL(segsum_kernel<WINDOW>, dim3(total_blocks), dim3(kSegProgsPerBlock), 0, stream,
                       descs.far, descs.n, near_descs<NearFams>(descs));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_hip(e, "segsum_kernel launch");
    return FS_OK;
}

int launch_segsum(const Descs<FamDesc> &descs, int64_t rows, int64_t programs, int total_blocks, hipStream_t stream)
{
    return rows <= kSegShortRows * programs ? launch_window<kSegShortWindow>(descs, total_blocks, stream)
                                        : launch_window<kSegWindow>(descs, total_blocks, stream);
}

}  // namespace fs
