// lf_internal.h -- structures shared by the host side (lf_api.cpp) and the
// kernels (lf_kernels.hip) of the GPU library.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lfk {

constexpr int NL = 12;
constexpr int MAX_WINDOW = 64;    // n_hits_window upper bound (6-bit window-relative indices)
constexpr int MAX_TRIPLETS = 32;  // n_triplets upper bound

// Sums and solves of a candidate's fits that depend only on which layers have
// a hit, for hits on the layer planes: the serial sums over the present layers
// in ascending order of 1, s, h, s^2, s h, h^2 (x fit) and 1, s, s^2 over the
// stereo layers (y fit), the x fit's cofactors and determinant, the y fit's
// determinant, C(n_hits), and the binary64 reciprocals (recip, see div_by) of det and D
// (of 1 where they are 0), n - 3 and n_uv - 2.
struct alignas(16) FitRow {
    float S0, S1, S2, S11;
    float S12, S22, m00, m01;
    float m02, det, YS0, YS1;
    float YS11, D, C, unused;
    double r_det, r_D, r_nx, r_ny;
};

constexpr uint32_t FIT_ROWS = 1u << NL;   // one for each mask

// Geometry and parameters: one block of device memory per context.
struct KParams {
    float z[NL], dxdy[NL];
    float z_in, z_mag, z_ref, z_T, kick, kappa, dRatio;
    int32_t polarity;
    float T_triplet, T_x, T_uv_scale, T_uv_floor, T_ty, T_y, T_Q;
    float xtol_const, xtol_pscale, xasym, uv_halfwidth, K_first, K_last;
    float magtol_const, magtol_pscale, magtol_txscale, magtol_min, magtol_max, p_charge_cut;
    float C_nhits[4];
    int32_t n_hits_window, n_triplets;
    // No-UT tuning (VELO-only input): straight-line extrapolation, assumed
    // minimum momentum, two windows per layer
    int32_t velo_only;
    float noUT_c[8], noUT_p_min, noUT_pt_min, noUT_overlap;
    // Momentum form: 0 linear kick; 1 sqrt-normalised pt-kick with the
    // integrated field F(tx, ty, dSlope) = sum_i c_i dSlope^i, c_i from F_coef
    int32_t field_form;
    float F_coef[5][10];
    // Triplet seeding in binary16 (VELO-UT input only)
    int32_t seed_fp16;
    // What hits on the layer planes make constant (two tracks per wavefront,
    // lf_pair.h): u = z - z_ref and g(u) of each layer, and the fits'
    // h = s^2 (1 + dRatio u), s = u / 1024; per seed set (layers l0, l1, l2) the triplet
    // model's u0, g0, u1 - u0, u2 - u1, G01, G12 - G01, then z_l0, z_l1,
    // z_l2 - z_l0, 1 / (z_mag - z_l0) (bracket only), K and z_mag - z_l0;
    // fit_tab[mask] for each 12-bit mask of layers with a hit.  pair_ok: the
    // planes allow that path (lever arms and set lengths above 1 mm).
    alignas(16) float lay_u[NL];
    float lay_g[NL], lay_h[NL];
    float set_tab[2][12];
    // binary64 reciprocals (recip, see div_by): per seed set of z_l2 - z_l0,
    // u1 - u0, u2 - u1 and G12 - G01; of dxdy of each layer, T_x, T_y and kick
    double r_set[2][4], r_dxdy[NL], r_Tx, r_Ty, r_kick;
    int32_t pair_ok;
    const FitRow *fit_tab;   // [FIT_ROWS] device memory
};

// Where a sorted search in one hit bucket starts: the bucket's x range cut into
// IDX_CELLS equal cells, start[c] = first hit (bucket-relative) of cell >= c.
// cell(x) is non-decreasing in x under rounding, so the hits of smaller cells
// than cell(key) are below the key and those of larger cells are not: the
// lower bound of the key lies in [start[c], start[c + 1]], c = cell(key).
constexpr int IDX_CELLS = 64;
struct alignas(16) BucketIndex {
    float lo, scale;
    // ranges over the bucket: z, max dxdy - min dxdy, max |dxdy|, max |x|
    float zmin, zmax, dspread, dabs, xabs;
    uint16_t start[IDX_CELLS + 1], flags;
};
static_assert(sizeof(BucketIndex) == 160, "written as 40 words");
__host__ __device__ inline int index_cell(float x, float lo, float scale) {
    return (int)fminf(fmaxf((x - lo) * scale, 0.0f), (float)(IDX_CELLS - 1));
}
constexpr uint32_t IDX_MAX_BUCKET = 65535;   // hits of a bucket the index can hold

// Flags of an event: of its buckets six by six in BucketIndex::flags of the
// first of the six, or, in a batch without indexes, of all in DevBatch::uni.
enum { EV_MIXED = 1,       // in some bucket the hits differ in z or dxdy (bit for bit)
       EV_OFF_PLANES = 2,  // some hit is off the geometry's layer planes (z, and dxdy on stereo layers)
       EV_NO_INDEX = 4 };  // a bucket is too long for the index
constexpr int EV_PARTS = 4, EV_PART = 24 / EV_PARTS;

// Device view of one resident batch (SoA, all in HBM).
struct DevBatch {
    const uint32_t *hit_off;   // [24*E+1]
    const float *hx, *hz, *hd; // [H]
    const uint32_t *trk_off;   // [E+1]
    const uint32_t *trk_ev;    // [T] event of each track
    const float *tx_, *ty_, *ttx, *tty, *tqop;  // [T]
    const uint8_t *uni;        // [E] EV_* flags (without bidx)
    const BucketIndex *bidx;   // [24*E], or nullptr: searches start from the whole bucket
    uint8_t *found, *nhits;    // [T]
    int32_t *hit_idx;          // [12*T]
    float *a, *b, *c, *y0, *ty, *qop, *Q;  // [T]
    uint32_t *counter;         // [QUEUE_WORDS] persistent-mode queue heads and exit counts, zero between launches
    unsigned long long *stats; // [32] work counters (counting launch only)
    uint32_t n_events, n_tracks;
    // batched mode over slots of a resident pool: result slot t (< n_map)
    // follows input track trk_map[t] (nullptr: slot t is track t)
    const uint32_t *trk_map;
    uint32_t n_map;
};

// Work queues of the persistent mode: QUEUE_SUB per XCD (8 XCDs), heads
// QUEUE_STRIDE words (256 bytes) apart, each followed by the count of its
// exited waves, then the count of queues whose waves have all exited.
constexpr uint32_t QUEUE_SUB = 16;
constexpr uint32_t QUEUE_N = 8 * QUEUE_SUB;
constexpr uint32_t QUEUE_STRIDE = 64;
constexpr uint32_t QUEUE_WORDS = QUEUE_STRIDE * (QUEUE_N + 1);

struct ExecCfg {
    int waves_per_block;
    int items_per_grab;
    // persistent grid; its default is what is resident of the kernel that pair_ok
    // names.  A batch without search indexes runs the one-track kernel on the same
    // grid: 20,000 short events 1,692 us against 1,568 on a grid of its own, 200
    // nominal events 143 against 155, 300 short ones 69 against 82.
    int blocks_per_cu;
    int n_cu;
    // batched and persistent mode: the geometry's planes allow the two-track
    // kernel (which a batch without search indexes does not run all the same)
    bool pair_ok;
    int n_triplets;   // of the context's parameters
};

// One event of a serving batch: its blob in pinned host memory (device
// address) -- [bucket offsets, event-local: u32 x 25][x H][z H][dxdy H]
// [track x, y, tx, ty, q/p: 5 x T] -- and where it goes in the batch.
struct GatherDesc {
    uint64_t src;
    uint32_t hit_base, trk_base, n_hits, n_tracks;
};

// Writable view of a batch's input arrays (the serving gather fills them).
struct BatchIn {
    uint32_t *hit_off;
    float *hx, *hz, *hd;
    uint32_t *trk_off, *trk_ev;
    float *tx, *ty, *ttx, *tty, *tqop;
};

// Assembles a batch of E events on the device from their host blobs
// (zero-copy reads over the host link): offsets rebased, hits and track
// states copied, trk_ev filled.  desc is in device memory.
hipError_t launch_gather(const GatherDesc *desc, uint32_t n_events, const BatchIn &out, hipStream_t s);

// Result slots of a batch of pool events evs[0..n_events) (slots [toff[e],
// toff[e+1]) for event e, n_slots = toff[n_events], read on the device):
// map[i] = the pool track slot i follows.  All arrays in device memory.
hipError_t launch_track_map(const uint32_t *evs, const uint32_t *toff, uint32_t n_events, uint32_t n_slots,
                            const uint32_t *pool_trk_off, uint32_t *map, hipStream_t s);
// The hot path.  P points to a KParams in device memory.  mode: 0 plain
// (per-event launches), 1 batched (one launch, two tracks per wavefront), 2 persistent
// (resident wavefronts pulling from per-XCD work queues).
// trk_off_host is read by mode 0 only.
// n_sides: 1 for VELO-UT input, 2 for VELO-only input (two windows per
// layer), 3 for VELO-UT input with the binary16 seeding build.
hipError_t launch_find(const DevBatch &b, const KParams *P, int n_hits_window, int n_sides, int mode,
                       const ExecCfg &cfg, const uint32_t *trk_off_host, hipStream_t s);
// What the hot path needs to know of each event beside its hits (four blocks per
// event, or one without indexes; the batch's hits and offsets must be in place):
// the bucket indexes b.bidx with the event's flags or, where b.bidx is nullptr, the
// flags uni[E], and trk_ev.
hipError_t launch_event_index(const DevBatch &b, const KParams *P, uint8_t *uni, hipStream_t s);
// Fills the parts of k that follow from its geometry (lay_*, set_*, pair_ok).
void plane_constants(KParams &k);
// Fills the FIT_ROWS rows of the fit table of P (both in device memory).
hipError_t launch_fit_table(const KParams *P, FitRow *rows, hipStream_t s);
// Counting launch: one wavefront per track, adds the work counters of every
// track into b.stats (which must be zeroed first).
hipError_t launch_count(const DevBatch &b, const KParams *P, int n_hits_window, int n_sides, hipStream_t s);
// Fills the result slots with a poison pattern (kernel, no memset).
hipError_t launch_poison(const DevBatch &b, hipStream_t s);
// Resident blocks per compute unit of the persistent kernel (0 on error).
int persistent_blocks_per_cu(int n_hits_window, int n_sides, const ExecCfg &cfg);

// Fixed scratch of the non-allocating entry point: one array in the code
// object's device memory per GPU, holding the persistent mode's queue words,
// the per-event flags, the event of each track and the bucket indexes of
// batches of up to FIXED_IDX_EVENTS events (larger ones go without).
constexpr uint32_t FIXED_MAX_EVENTS = 1u << 20;
constexpr uint32_t FIXED_MAX_TRACKS = 1u << 22;
constexpr size_t FIXED_QUEUE_OFF = 0;                       // QUEUE_WORDS x u32
constexpr size_t FIXED_UNI_OFF = 4 * (size_t)QUEUE_WORDS;   // FIXED_MAX_EVENTS x u8
constexpr size_t FIXED_TRK_EV_OFF = FIXED_UNI_OFF + FIXED_MAX_EVENTS;   // FIXED_MAX_TRACKS x u32
constexpr uint32_t FIXED_IDX_EVENTS = 8192;
constexpr size_t FIXED_IDX_OFF = FIXED_TRK_EV_OFF + 4 * (size_t)FIXED_MAX_TRACKS;   // 24 x FIXED_IDX_EVENTS x BucketIndex
constexpr size_t FIXED_BYTES = FIXED_IDX_OFF + 24 * (size_t)FIXED_IDX_EVENTS * sizeof(BucketIndex);
static_assert(FIXED_IDX_OFF % 16 == 0, "the indexes are 16-byte aligned");
// Device address of the current device's copy of the fixed scratch, looked
// up once per device (the first call on a device must run with it current).
hipError_t fixed_scratch(void **out);
// Writes zeros to n words with a kernel (no memset node under capture).
hipError_t launch_zero_words(uint32_t *p, uint32_t n, hipStream_t s);

}  // namespace lfk
