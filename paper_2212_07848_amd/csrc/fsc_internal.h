// fsc_internal.h -- declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>
#include <stdint.h>

#include <vector>

#include "fsc_device.h"

namespace fsc {

// Host-side range around a library call, shown by profilers that collect
// markers (rocprofv3 --marker-trace); without one attached it costs a call.
struct TraceRange {
    explicit TraceRange(const char *name) { roctxRangePushA(name); }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange &) = delete;
    TraceRange &operator=(const TraceRange &) = delete;
};

// Tile shape of the fused step kernel: a TX x TY cross-section (TY = 1 in 2D)
// marching along the slowest axis.
struct TileShape {
    int tx, ty, pf;     // cross-section tile and register prefetch depth (planes)
    int steps = 1;      // time steps per launch: 1, or 2 (two-step kernel, 2D FP32)
};

// Launch of one step over every replica of an ensemble.
struct StepLaunch {
    const RepDesc *reps;       // device
    const int *tile_begin;     // device, [nrep]
    int nrep;
    int total_tiles;
    int parity;                // source buffer index
    const uint64_t *step_base; // device
    uint32_t step_off;
    int D, stencil, precision; // selects the instantiation
    bool noise;
    bool wide;                 // a replica's buffers reach 4 GiB (single-step kernel only)
    TileShape tile;
};

// One launch of the tile's kernel: one step, or two when L.tile.steps == 2
// (then the state goes from buf[parity] at step_base + step_off to
// buf[parity ^ 1] at two steps later).  hipErrorInvalidValue when no
// instantiation matches.
hipError_t launch_step(const StepLaunch &L, hipStream_t s);
// Several steps per launch on small 2D lattices (fsc_block_kernel.h).  Tiles of
// one replica: tiles_x x ceil(ny / ty) tiles of tx x ty nodes (tx == nx with one
// tile across: whole periodic rows).
struct BlockTile {
    int begin, tiles_x, tx, ty;
};
constexpr int BLOCK_ROWS = 4;  // rows of a step per wave, at most
struct BlockLaunch {
    const RepDesc *reps;       // device
    const BlockTile *tiles;    // device, [nrep]
    int nrep, blocks;
    int parity, T;             // source buffer, steps
    const uint64_t *step_base; // device
    uint32_t step_off;
    int stencil, precision;
    bool noise;
    int ws;                    // columns of the region: 64 or 128
    size_t lds;
};
// The state goes from buf[parity] at step_base + step_off to buf[parity ^ 1] T
// steps later.
hipError_t launch_block(const BlockLaunch &L, hipStream_t s);
// Waves of a block and LDS bytes of one row of its region.
inline int block_waves(int precision, int ws) { return ws == 128 && precision == 0 ? 16 : 8; }
inline size_t block_row_bytes(int precision, int ws) { return size_t(10) * ws * (precision == 0 ? 4 : 8); }

// Tile shapes compiled for a lattice/stencil; the first is the default.
int tile_shapes(int D, int stencil, int precision, TileShape *out, int max);

// Adds k to the device step counter (one thread).
hipError_t launch_step_advance(uint64_t *step_base, uint64_t k, hipStream_t s);

// ---------------------------------------------------------------------------
// Measurement kernels (fsc_measure.hip).
// ---------------------------------------------------------------------------
struct Geometry {
    int D, nx, ny, nz;
    int64_t N;
};

// Density n(x) in double of the x-rows row0 .. row0 + rows - 1 (row = y + ny z).
hipError_t launch_density(const Geometry &g, int precision, const void *buf, double rho0, int64_t row0,
                          int64_t rows, double *out, hipStream_t s);
// Its deviation n(x) - rho0 from an FP32 lattice, as floats, all rows.
hipError_t launch_deviation(const Geometry &g, const float *buf, float *out, hipStream_t s);
// Streamed populations shift[i] + df_i in double, elements e0 .. e0 + n - 1 of
// [i][z][y][x].
hipError_t launch_streamed(const Geometry &g, int precision, const void *buf, const double *shift, int64_t e0,
                           int64_t n, double *out, hipStream_t s);
// A result in pinned host memory and the word there that announces it: the
// kernel stores `seq` to *flag, visible to the host, after the result.
struct Mail {
    double *out;
    uint32_t *flag;
    uint32_t seq;
};
// FP64 state reductions into mail.out[8] (see fsc_stats); `partials` holds
// stats_partials_len() doubles, *done is 0 between calls.
size_t stats_partials_len();
hipError_t launch_stats(const Geometry &g, int precision, const void *buf, double rho0,
                        double *partials, int *done, const Mail &mail, hipStream_t s);
// n doubles of device memory into mail.out.
hipError_t launch_mail(const double *src, int n, const Mail &mail, hipStream_t s);

// Pinned host memory that kernels mail results to, one result at a time.
class Mailbox {
  public:
    Mailbox() = default;
    Mailbox(const Mailbox &) = delete;
    Mailbox &operator=(const Mailbox &) = delete;
    ~Mailbox() {
        if (flag_) (void)hipHostFree(flag_);
    }
    double *data() const { return data_; }
    // allocates at the first call (always the same size)
    hipError_t make(size_t bytes) {
        if (flag_) return hipSuccess;
        void *p = nullptr;
        const hipError_t e = hipHostMalloc(&p, HEAD + bytes, hipHostMallocDefault);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
        flag_ = static_cast<uint32_t *>(p);
        *flag_ = 0;
        data_ = reinterpret_cast<double *>(static_cast<char *>(p) + HEAD);
        return hipSuccess;
    }
    Mail next() { return Mail{data_, flag_, ++seq_}; }
    // Waits for the last mail of next(): polls for about a millisecond, then waits
    // for the stream (long runs, and whatever keeps the kernel from running).
    hipError_t wait(hipStream_t s) const {
        for (int k = 0; k < POLLS; ++k) {
            if (__atomic_load_n(flag_, __ATOMIC_ACQUIRE) == seq_) return hipSuccess;
            __builtin_ia32_pause();
        }
        const hipError_t e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        return __atomic_load_n(flag_, __ATOMIC_ACQUIRE) == seq_ ? hipSuccess : hipErrorUnknown;
    }

  private:
    static constexpr size_t HEAD = 64;  // the flag's line
    static constexpr int POLLS = 20000;
    uint32_t *flag_ = nullptr, seq_ = 0;
    double *data_ = nullptr;
};

// What a thread's synchronous calls without a handle (field S(k), linear S(k)) keep
// between them: the pinned result and up to KEEP bytes of device work area on the
// device it last ran on (beyond 256 KB hipMalloc and hipFree take 20 us, as much
// as the transforms of 16 fields of 128^2).  Every call ends with its device work
// done, so the next one may use another stream.  Given back when the thread ends.
class ThreadWork {
  public:
    static constexpr size_t MAIL = size_t(16) << 10, KEEP = size_t(8) << 20;
    ~ThreadWork() { drop(); }
    Mailbox *mailbox() { return box_.make(MAIL) == hipSuccess ? &box_ : nullptr; }
    int take(size_t bytes, void **out);  // an FSC_ code
    void done(void *p) {
        if (p != kept_) (void)hipFree(p);
    }

  private:
    void drop() {
        if (kept_) (void)hipFree(kept_);
        kept_ = nullptr;
        bytes_ = 0;
        dev_ = -1;
    }
    Mailbox box_;
    void *kept_ = nullptr;
    size_t bytes_ = 0;
    int dev_ = -1;
};
ThreadWork &thread_work();

// Transform of one axis: lines of n values over m points, m = 2^logm (n itself,
// or at least 2n - 1 for the chirp form), or m = n and logm = -1 (direct sum).
// wide: a chirp transform of FP32 data, with its lines in LDS and its table in
// doubles (see sk_axis).
struct SkAxis {
    int n, m, logm, wide;
};
SkAxis sk_axis(int n, int precision);
// bytes of a complex value of an axis' lines in LDS and of its table
inline size_t sk_value_bytes(int precision, const SkAxis &x) { return precision == 0 && !x.wide ? 8 : 16; }
// complex values of an axis' table: the m-th roots of unity, and for the chirp
// form the chirp and its spectrum
size_t sk_table_len(const SkAxis &x);
// Fills a table; the same launch clears `zero_words` 32-bit words at `zero`.
// Synchronises the stream for the chirp form.
hipError_t sk_table(int precision, const SkAxis &x, void *tab, void *zero, int64_t zero_words, hipStream_t s);
// LDS of `lines` lines of m complex values of csz bytes (see sk_stride)
__host__ __device__ inline size_t sk_line_bytes(size_t csz, int lines, int m) {
    return (csz * size_t(lines) * size_t(m + (m >> 3) + 1) + 15) & ~size_t(15);
}

// Where the |X(k)|^2 / N of one spectrum go: FP64 axis and radial accumulators.
struct BinTargets {
    double *axis_sum, *axis_sq;  // [D][n_axis], or null
    double *rad_sum, *rad_sq;    // [n_rad] (rad_sq may be null)
    int n_axis, n_rad;
    // time series (null when disabled): per-sample sum P and sum |k| P, and
    // rows [cap][2 + n_rad] = (step, L, per-shell sums of P) at row *series_n
    double *mom;
    double *series;
    const int *series_n;
    int series_cap;
};
// One replica's part of a batched S(k) sample: a device table filled by the
// host.  The sampled density is dn(x) = sum_i f_i(x) - rho0 of the streamed
// state, gathered from the stored post-collision buffer buf[parity].
struct MeasRep {
    const void *buf[2];   // population buffers
    void *cbuf, *ctmp;    // half spectra, (nx/2 + 1) ny nz complex values (ctmp: 3D only)
    const void *tab[3];   // transform tables per axis (see sk_table)
    SkAxis ax[3];         // set by measure_plan, as are
    int lc[3];            // lines per block of the row, mid and last launches
    Geometry g;
    BinTargets t;         // accumulators; t.mom == nullptr: no time series
    double invN;
    int *series_n;        // the time series' row counter (t.series_n, writable)
    double *modes;        // mode recorder rows [cap][D][nm][2], or null
    int *modes_n;
    int modes_nm, modes_cap;
    int *done;            // blocks of the last launch that have finished (0 between samples)
};
// kinds of work in one sample
constexpr int MK_ROWS = 0, MK_MID = 1, MK_LAST = 2, MK_COUNT = 3;
struct MeasPlan {
    int nrep = 0, D = 2;
    size_t esz = 4;          // bytes of one real (set by the caller)
    std::vector<int> pre;    // [MK_COUNT][nrep + 1]: first block of each replica per kind
    size_t shm[MK_COUNT] = {};
    int threads[MK_COUNT] = {};
    bool wide[MK_COUNT] = {};  // some replica's axis is wide
};
// Fills the block prefixes, block sizes and LDS sizes of P, and the transforms
// of the host copy of the replica table; -1 if a side exceeds 8192 or a grid
// exceeds 2^31 blocks.
int measure_plan(MeasRep *reps, int nrep, MeasPlan &P);
// One S(k) sample of every replica in P (bins, mode records, series rows), in
// two (2D) or three launches.  Adds `advance` to the step counter step_base[0]
// first (the steps enqueued before the sample, once none of their launches is
// still to read it); the sampled state is step_base[0] + step_off after that.
hipError_t launch_measure(const MeasPlan &P, const MeasRep *dev_reps, const int *dev_pre, int precision,
                          int parity, uint64_t *step_base, uint64_t advance, uint32_t step_off, hipStream_t s);

// S(k) of `batch` device fields [n][n]: adds every field's shell sums of |X|^2 /
// n^2 and its sum P and sum |k| P to acc + f field_acc_len(n_rad).  spec:
// batch (n/2 + 1) n complex floats; tab: the table of sk_axis(n, 0).
__host__ __device__ inline size_t field_acc_len(int n_rad) { return size_t(n_rad) + 2; }
hipError_t launch_field_sk(const float *fields, int batch, int n, int n_rad, void *spec, const void *tab,
                           double *acc, hipStream_t s);

// Block means of the density over f x f blocks (2D) into out[(ny/f) x (nx/f)].
hipError_t launch_coarsen(const Geometry &g, int precision, const void *buf, double rho0, int f,
                          float *out, hipStream_t s);
// Plain copy of `bytes` (multiple of 16) bytes.
hipError_t launch_copy(const void *src, void *dst, int64_t bytes, hipStream_t s);

// Device Philox / normals checks.
hipError_t launch_philox(const uint32_t *ctr, const uint32_t *key, uint32_t *out, int64_t n,
                         hipStream_t s);
hipError_t launch_normals(int D, int precision, uint64_t seed, uint32_t replica,
                          const int64_t *node, const int64_t *step, int64_t n, double *out,
                          hipStream_t s);

}  // namespace fsc
