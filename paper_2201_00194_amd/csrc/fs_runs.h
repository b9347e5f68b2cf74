// Rows in runs of a fixed length.
#ifndef FS_RUNS_H
#define FS_RUNS_H

#if defined(__HIPCC__)
#define FS_BOTH __host__ __device__ __forceinline__
#else
#define FS_BOTH inline
#endif

namespace fs {

// run(first row, rows left) for [from, to), STEP rows at a time.  It counts what is left: a row number goes up to 2^31 - 1,
// so the one after the last run need not fit.
template <int STEP, class Run>
FS_BOTH void in_runs(int from, int to, Run run)
{
    for (int left = to - from; left > 0; left -= STEP)
        run(to - left, left);
}

}  // namespace fs
#endif
