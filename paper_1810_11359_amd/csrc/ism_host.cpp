// C ABI of libism.so (declared in include/ism.h): argument checks, FP64 host
// planning, workspace layout and kernel launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <memory>
#include <thread>
#include <vector>

#include "ism.h"
#include "ism_debug.h"
#include "ism_internal.h"
#include "ism_tuning.h"

namespace ism {
int launch_tables(const RoomArgs &ra, const float *src, const float *rcv, const float *orient, AxisEntry *tab,
                  AxisOrigin *origin, int *valid, int n_rir, float W, bool half, float *wc, hipStream_t st);
int launch_accumulate(int wt, bool gen, int kind, bool lut, bool polar, const RoomArgs &ra, const PlanArgs &pa,
                      uint32_t n_items, const AxisEntry *tab, const AxisOrigin *origin, const int *valid, float *out,
                      float *part, float *marg, const float *wc, hipStream_t st);
int launch_reduce(const RoomArgs &ra, const PlanArgs &pa, int n_rir, const float *part, const float *marg,
                  float *out, hipStream_t st);
bool supported_window(int wt, bool gen);
int launch_dump(bool half, const RoomArgs &ra, const PlanArgs &pa, uint32_t n_items, const AxisEntry *tab,
                const AxisOrigin *origin, const int *valid, DumpArgs dump, hipStream_t st);
int launch_batch(const JobDev *jobs, int n_jobs, bool any_gen, const BatchRir *rirs, uint32_t n_rir,
                 const BatchItem *items, const BatchClass *cls, int n_classes, bool half, bool lut, bool polar,
                 const BatchReduce *red, uint32_t n_red, uint32_t n_red_split, bool long_runs, int max_tile,
                 AxisEntry *tab,
                 AxisOrigin *origin, int *valid, float *part, float *marg, uint32_t *queue, hipStream_t st,
                 hipEvent_t ev_start, hipEvent_t ev_stop);
int launch_diffuse(const float *ism, int k_diff, float *out, int n_samples, int n_rir, double fs, double t_diff,
                   double t60, uint64_t seed, hipStream_t st);
int launch_filter(const float *x, int n_x, const float *rir, int n_pos, int n_mic, int n_rir, float *y,
                  hipStream_t st);
bool fft_plan(int n_x, int n_pos, int n_mic, int n_rir, int max_pieces, FftPlan &f);
bool seg_plan(int n_x, int n_pos, int n_mic, int n_rir, FftPlan &f);
int launch_filter_fft(const float *x, int n_x, const float *rir, int n_pos, int n_mic, int n_rir, float *y,
                      const FftPlan &f, bool contain, void *ws, hipStream_t st);
}  // namespace ism

using namespace ism;

namespace {

constexpr double kPi = 3.14159265358979323846;

// A failed HIP runtime call: names it on stderr and maps it to ISM_E_DEVICE.
int device_error(const char *where, hipError_t e) {
  fprintf(stderr, "libism: %s: %s\n", where, hipGetErrorString(e));
  return ISM_E_DEVICE;
}

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

int lattice_lo(int N) { return -(N / 2); }       // ceil(-N/2)
int lattice_hi(int N) { return (N + 1) / 2; }    // ceil(N/2), exclusive

void split(double v, float &hi, float &lo) {
  hi = (float)v;
  lo = (float)(v - (double)hi);
}

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

// Window length W = t_w * fs in samples when it is an even integer (within
// 1e-9 relative); 0 otherwise.
int even_window(const ism_room &r) {
  const double W = r.t_w * r.fs;
  const double k = std::nearbyint(W);
  if (std::fabs(W - k) > 1e-9 * W) return 0;
  const long iw = (long)k;
  if (iw < 2 || (iw & 1)) return 0;
  return (int)iw;
}

// Kernel class of a window of W = t_w fs samples (Eq. (6)): exact mode for an
// even integer W in {32, 64, 96, 128} (cap WT = W), else general mode with
// the cap WT = the next multiple of 32 (at least 32, at most MAX_WINDOW).
int window_class(const ism_room &r, int &wt, bool &gen, double &W) {
  W = r.t_w * r.fs;
  const int ev = even_window(r);
  if (ev == 32 || ev == 64 || ev == 96 || ev == 128) {
    wt = ev;
    gen = false;
    W = ev;
    return ISM_OK;
  }
  if (W > MAX_WINDOW * (1.0 + 1e-9)) return ISM_E_TOO_LARGE;
  W = std::min(W, (double)MAX_WINDOW);
  wt = std::max(32, 32 * (int)std::ceil(W / 32.0 - 1e-9));
  gen = true;
  return ISM_OK;
}

struct Plan {
  RoomArgs ra;
  PlanArgs pa;
  double tile_taps[MAX_TILES];  // estimated taps of each tile's image shell
  double total_taps;            // over all RIRs
  int wt;     // window cap WT (kernel layout)
  bool gen;   // general-mode window (per-call tap constants)
  double win; // W = t_w fs
  bool half;
  bool lut;  // table taps (Eq. (9)); FP32 arithmetic otherwise
  int kind;  // of its work items
  int n_rir;
  uint32_t n_items;
  bool any_split;
  size_t off_valid, off_origin, off_tab, off_part, off_marg, off_wc, off_pos, ws_bytes;
};

// Work-item size in estimated taps. FP16: a launch should hold about balance_items
// items (some eight per resident wave) so that the largest-first order keeps
// every CU busy to the end; small calls keep items of min_item_taps. Both come
// from the tuning table (ism_tuning.h) for the window unless the call's schedule
// (ism_schedule) replaces them.
constexpr double kMinItemTaps = 1.2e5;
constexpr double kBalanceItems = 49152.0;
// FP32 items (four waves, a convolution per item) cost images rather than taps.
// A call is cut into about kMomItems items, one per resident workgroup (a
// 32-receiver room took 187, 151 and 152 us with 512, 1024 and 2048), but an item's
// fixed part is worth some thousand images: items hold at least kMomFullImages
// (a 11200-sample RIR took 34.5 and 40 us with items of 3800 and 1900 images, 6
// directional RIRs at 44.1 kHz 61, 69 and 78 us with 4000, 2000 and 1000) unless
// that leaves fewer than kMomFewItems, then at least kMomMinImages (a single
// 4800-sample RIR took 30, 24.5, 25 and 40 us with items of 160, 780, 1600 and 7800
// images). At most kMomMaxImages (or a kMomMaxItems-th of the call), so that long
// calls end evenly.
constexpr double kMomMinImages = 800.0;
constexpr double kMomFewItems = 192.0;
constexpr double kMomFullImages = 4000.0;
constexpr double kMomItems = 1024.0;
constexpr double kMomMaxImages = 65536.0;
constexpr double kMomMaxItems = 8192.0;
// mom: items cut by images; otherwise by taps, the FP16 items (half) or the cut that sizes
// the workspace of the others.
double item_target(double total_taps, int wt, bool half, bool mom, int64_t n_samples, const ism_schedule *sc) {
  if (mom) {
    const double few = std::min(kMomFullImages * wt, total_taps / kMomFewItems);
    double min_taps = std::max(kMomMinImages * wt, few), balance = kMomItems,
           max_taps = std::max(kMomMaxImages * wt, total_taps / kMomMaxItems);
    if (sc && sc->balance_items > 0.0) {
      balance = std::max(1.0, sc->balance_items);
      min_taps = kMomMinImages * wt;
      max_taps = total_taps;
    }
    if (sc && sc->min_item_taps > 0.0) min_taps = std::max(1e3, sc->min_item_taps);
    return std::max(min_taps, std::min(max_taps, total_taps / balance));
  }
  double min_taps = kMinItemTaps, balance = kBalanceItems;
  for (const ItemTuning &t : kItemTuning)
    if (t.wt == wt && t.half == (half ? 1 : 0) && n_samples <= t.ns_max) {
      min_taps = t.min_item_taps;
      balance = t.balance_items;
      break;
    }
  if (sc && sc->min_item_taps > 0.0) min_taps = std::max(1e3, sc->min_item_taps);
  if (sc && sc->balance_items > 0.0) balance = std::max(1.0, sc->balance_items);
  return std::max(min_taps, total_taps / balance);
}

// Largest work item of an FP16 batch job, or of the cut that sizes the workspace of the
// others (by window class; classes without a row take kBatchItemTaps).
constexpr double kBatchItemTaps = 2.5e5;
double batch_item_taps(int wt, bool half) {
  for (const BatchTuning &t : kBatchTuning)
    if (t.wt == wt && t.half == (half ? 1 : 0)) return t.item_taps;
  return kBatchItemTaps;
}

// Workgroups of the accumulate kernel resident on the device at once (256 CUs x
// 4 SIMDs x the waves per SIMD the kernel is built for, over its waves per
// item), and the default rounds of them over which a single call tapers its tail.
double resident_items(int kind, bool lut) {
  return 256.0 * 4.0 * waves_per_simd(kind, lut) * 64.0 / item_threads(kind);
}
constexpr double kTailRounds = 1.0;

// Small calls: a call whose work does not give every resident wave an item
// of the tuned size is spread over them instead, total / resident waves per
// item but at least kSmallItemTaps, which is also the taper's lowest item (a
// single 4800-sample RIR, 1e7 taps, measured 27 us per accumulate launch with
// 1e4-tap items against 35 us with the earlier floor of an eighth of 1.2e5
// and 103 us with 1.2e5-tap items).
constexpr double kSmallItemTaps = 1e4;
double small_call_floor(double total_taps, double resident) { return std::max(kSmallItemTaps, total_taps / resident); }

bool valid_schedule(const ism_schedule *sc) {
  if (!sc) return true;
  const double v[5] = {sc->item_taps, sc->min_item_taps, sc->balance_items, sc->tail_rounds, sc->batch_waves};
  for (double x : v)
    if (!std::isfinite(x)) return false;
  return sc->item_taps >= 0.0 && sc->min_item_taps >= 0.0 && sc->balance_items >= 0.0 && sc->batch_waves >= 0.0 &&
         sc->batch_waves <= 16.0;
}

// Cuts the tiles of a call into items of about target taps (tapered over the
// last tail_rounds rounds of the resident items, down to floor_taps): the items
// per tile into chunks (may be null), their total over all RIRs and the part of
// it in split tiles. False when the total exceeds a launch.
bool cut_tiles(const Plan &p, const double *tile_taps, int n_tiles, double target, double floor_taps,
               double tail_rounds, double resident, uint8_t *chunks, uint64_t &n_items, uint64_t &n_split) {
  n_items = n_split = 0;
  double rem = p.total_taps;
  for (int t = n_tiles - 1; t >= 0; --t) {  // dispatch order: last tile first
    const double taps = tile_taps[t];
    double tt = target;
    if (tail_rounds > 0.0) tt = std::max(floor_taps, std::min(target, rem / (tail_rounds * resident)));
    const int ch = std::max(1, std::min((int)std::ceil(taps / tt), MAX_CHUNKS));
    if (chunks) chunks[t] = (uint8_t)ch;
    if (ch > 1) n_split += (uint64_t)p.n_rir * ch;
    rem -= taps * p.n_rir;
    n_items += (uint64_t)p.n_rir * ch;
    if (n_items > 0x7fffffffULL) return false;
  }
  return true;
}

// Bytes of the partial tiles (where some tile is split) and margins of a call's items.
size_t item_arrays(uint64_t items, bool split, int tile, int wt) {
  return align_up(split ? sizeof(float) * (size_t)items * tile : 0) + align_up(sizeof(float) * (size_t)items * wt);
}

// Estimated taps of the tiles of T samples of one RIR: the owned shell volume over
// the image density 1 / (Lx Ly Lz) (one image per mirrored room copy), times the
// window cap. Returns their number; taps has MAX_TILES entries.
int shell_taps(const ism_room &r, const Plan &p, int T, double *taps) {
  const double q = r.fs / r.c;
  const double cell = r.room[0] * r.room[1] * r.room[2] * q * q * q;
  const double lattice = (double)r.n_img[0] * r.n_img[1] * r.n_img[2];
  const int n = (p.ra.k_end + T - 1) / T;
  for (int t = 0; t < n && t < MAX_TILES; ++t) {
    const double x0 = (double)t * T, x1 = std::min((double)(t + 1) * T, (double)p.ra.k_end);
    taps[t] = std::min(4.0 / 3.0 * kPi * (x1 * x1 * x1 - x0 * x0 * x0) / cell, lattice) * (double)p.wt;
  }
  return n;
}

// Whether an FP32 call takes tiles of LONG_TILE samples. A long tile halves the
// columns walked per image, whose number grows with the shortest side (a column's
// images lie half of its period apart), and a tile's fixed part; its lists are
// shorter, which costs every image about 15 lane instructions. In lane
// instructions per image, columns take 0.045 per sample of the shortest side and
// the fixed part 9e4 over the images of a TILE-sample tile.
// TILE against LONG_TILE, us per pass: 32 receivers in 4 x 5 x 3 m (11) 150 and 165,
// 4 receivers in 3 x 4 x 2.5 m (7) 70 and 81; 64 microphones at 48 kHz in
// 6 x 9 x 3.5 m (27) 2359 and 2219, 1024 diffuse RIRs of 2400 samples (50) 223 and
// 193.
// alone: a single call, whose few items are held up by their own length: fewer than
// kLongTileItems long tiles are not taken (8 RIRs of 7900 samples at 44.1 kHz, 128
// long tiles: 25.8 us with TILE, 27.8 with LONG_TILE; 30 RIRs at 32 kHz, 690: 49.8
// and 47.5).
constexpr double kLongTileGain = 19.0;
constexpr int64_t kLongTileItems = 512;
bool long_tiles(const ism_room &r, const Plan &p, bool alone) {
  if (alone && (int64_t)p.n_rir * ((p.ra.k_end + LONG_TILE - 1) / LONG_TILE) < kLongTileItems) return false;
  const double q = r.fs / r.c, k = (double)p.ra.k_end;
  const double side = std::min(r.room[0], std::min(r.room[1], r.room[2])) * q;
  const double images = std::min(4.0 / 3.0 * kPi * k * k * k / (r.room[0] * r.room[1] * r.room[2] * q * q * q),
                                 (double)r.n_img[0] * r.n_img[1] * r.n_img[2]);
  return 0.045 * side + 9.0e4 * k / (TILE * std::max(images, 1.0)) > kLongTileGain;
}

// Whether an FP32 or table-tap call takes one-wave items, image by image. An item of
// moments costs its lists and its product whatever it holds, and 1024 run at once; one
// wave pays 64 lanes x (W / 64) taps per image, but 6144 run at once. n: tiles over all RIRs
// of the launch. One wave is taken where even the fullest tile, the last whole one, holds
// few images, or, where the launch fills the chip with them, where tiles hold few on
// average: up to 250 images (table taps, whose moment items hold 17 planes, 800), and fewer
// in launches of fewer tiles, which the fullest item holds up. Moments against one wave, us
// per call at W = 64 and 30, 150 and 400 images per tile: 512 RIRs of 9600 samples (20 000
// tiles) 158 and 49, 168 and 109, 187 and 201; 64 RIRs of 2400 (630) 19 and 16, 19 and 21,
// 21 and 25; 8 RIRs of 2400 (80) 15 and 15, 15 and 20, 16 and 21. Table taps, the same: 335
// and 49, 346 and 114, 371 and 201; 24 and 17, 24 and 23, 26 and 28; 15 and 16, 16 and 22,
// 18 and 26. The limits are about the least of W = 32 .. 244.
constexpr double kFewFullest = 40.0;
constexpr double kFewTiles = 16.0, kFewMean = 250.0;
constexpr double kFewLutFirst = 500.0, kFewLutTiles = 4.0, kFewLutMean = 800.0;
struct TileImages {
  double mean, fullest;
};
TileImages tile_images(const ism_room &r, const Plan &p) {
  const double q = r.fs / r.c, k = (double)p.ra.k_end, k0 = std::max(k - TILE, 0.0);
  const double cell = r.room[0] * r.room[1] * r.room[2] * q * q * q;
  const double lattice = (double)r.n_img[0] * r.n_img[1] * r.n_img[2];
  return {std::min(4.0 / 3.0 * kPi * k * k * k / cell, lattice) / std::ceil(k / TILE),
          std::min(4.0 / 3.0 * kPi * (k * k * k - k0 * k0 * k0) / cell, lattice)};
}
bool few_images(TileImages t, bool lut, int64_t n) {
  if (t.fullest <= kFewFullest) return true;
  return t.mean <= (lut ? std::min(((double)n - kFewLutFirst) / kFewLutTiles, kFewLutMean)
                        : std::min((double)n / kFewTiles, kFewMean));
}
int64_t rir_tiles(const Plan &p) { return (int64_t)p.n_rir * ((p.ra.k_end + TILE - 1) / TILE); }
// The same for a batch of several jobs, whose items all cost some 10 ns to fetch: t is the
// average over its tiles and the fullest tile of all. FP32 batches that fill the chip keep to
// moments, and the limits are lower, since the long jobs of a mixed batch hold it up. Moments
// against one wave, us, 64 jobs of one length x 16 RIRs, at 20, 80, 160 and 300 images: 3072
// tiles 56 and 50, 58 and 52, 59 and 83, 59 and 109; 10 240 tiles 104 and 138, 106 and 171,
// 110 and 177, 115 and 193; table taps 81 and 52, 81 and 53, 83 and 85, 84 and 113; 203 and
// 139, 204 and 174, 206 and 184, 212 and 200. Lengths and rooms at random (8 jobs x 4: 96
// tiles) at 40 and 80: 18.9 and 20.0, 19.5 and 24.2; table taps 19.5 and 22.5, 19.7 and 26.9.
constexpr double kFewBatchMean = 40.0, kFewBatchFull = 4096.0;
constexpr double kFewLutBatchFirst = 75.0, kFewLutBatchTiles = 64.0, kFewLutBatchMean = 300.0;
bool few_images_batch(TileImages t, bool lut, int64_t n) {
  if (!lut && (double)n > kFewBatchFull) return false;
  if (t.fullest <= kFewFullest) return true;
  const double most = lut ? std::min(kFewLutBatchFirst + (double)n / kFewLutBatchTiles, kFewLutBatchMean) : kFewBatchMean;
  return t.mean <= std::min((double)n / kFewTiles, most);
}

// sched: the call's schedule (null = the tuned default).
// taper: cut the items dispatched last (single calls; a batch's tail is the
// largest-first order over all its jobs' items instead).
// kind: of FP32 and table-tap items (-1: the call's own).
int make_plan(const ism_room *r, int n_src, int n_rcv, int precision, Plan &p, const ism_schedule *sched = nullptr,
              bool taper = true, int kind = -1) {
  int st = ism_check_room(r);
  if (st != ISM_OK) return st;
  if (!valid_schedule(sched)) return ISM_E_INVALID_ARG;
  if (n_src < 1 || n_rcv < 1) return ISM_E_INVALID_ARG;
  if ((int64_t)n_src * n_rcv > ISM_MAX_PAIRS) return ISM_E_TOO_LARGE;
  if (precision != ISM_FP32 && precision != ISM_FP16 && precision != ISM_FP32_LUT)
    return precision == ISM_BF16 ? ISM_E_UNSUPPORTED : ISM_E_INVALID_ARG;
  p.half = precision == ISM_FP16;
  p.lut = precision == ISM_FP32_LUT;
  st = window_class(*r, p.wt, p.gen, p.win);
  if (st != ISM_OK) return st;
  // table taps are built for the exact windows only
  if (!supported_window(p.wt, p.gen) || (p.gen && p.lut)) return ISM_E_UNSUPPORTED;
  const int64_t nS = ism_n_samples(r->t_max, r->fs);
  const double W = (double)p.wt;
  const double q = r->fs / r->c;

  RoomArgs &ra = p.ra;
  std::memset(&ra, 0, sizeof(ra));
  // table axes: room axes by decreasing length (stable), shortest innermost
  int perm[3] = {0, 1, 2};
  std::stable_sort(perm, perm + 3, [&](int a, int b) { return r->room[a] > r->room[b]; });
  int off = 0;
  for (int k = 0; k < 3; ++k) {
    const int a = perm[k];
    ra.perm[k] = a;
    split(r->room[a], ra.L_hi[k], ra.L_lo[k]);
    ra.lo[k] = lattice_lo(r->n_img[a]);
    ra.N[k] = r->n_img[a];
    ra.off[k] = off;
    off += r->n_img[a];
    ra.inv_period[k] = (float)(1.0 / (2.0 * r->room[a] * q));
    split(r->beta[2 * a], ra.beta[2 * k], ra.beta_lo[2 * k]);
    split(r->beta[2 * a + 1], ra.beta[2 * k + 1], ra.beta_lo[2 * k + 1]);
  }
  ra.n_tab = off;
  split(q, ra.q_hi, ra.q_lo);
  ra.kappa = (float)(r->fs / (4.0 * kPi * r->c));
  ra.half_w = (float)(W / 2.0);
  ra.win_hw = (float)(p.win / 2.0);
  ra.inv_win = (float)(1.0 / p.win);
  ra.n_samples = (int)nS;
  ra.k_end = (int)nS + p.wt / 2 - 1;
  ra.n_src = n_src;
  ra.n_rcv = n_rcv;

  // Work split: tile t owns the images with k0 in [t T, min((t+1) T, k_end)).
  p.n_rir = n_src * n_rcv;
  PlanArgs &pa = p.pa;
  std::memset(&pa, 0, sizeof(pa));
  const bool tapered = taper && !(sched && (sched->item_taps > 0.0 || sched->tail_rounds == 0.0));
  p.kind = p.half                                                    ? ITEM_FP16
           : kind >= 0                                               ? kind
           : few_images(tile_images(*r, p), p.lut, rir_tiles(p))     ? ITEM_FEW
                                                                     : ITEM_MOMENTS;
  ra.tile = p.kind == ITEM_MOMENTS && !p.lut && long_tiles(*r, p, tapered) ? LONG_TILE : TILE;
  pa.n_rir = p.n_rir;
  pa.n_tiles = shell_taps(*r, p, ra.tile, p.tile_taps);
  if ((ra.k_end + TILE - 1) / TILE > MAX_TILES) return ISM_E_TOO_LARGE;
  p.total_taps = 0.0;
  for (int t = 0; t < pa.n_tiles; ++t) p.total_taps += p.tile_taps[t] * p.n_rir;
  // an explicit item size is used as given
  const bool fixed = sched && sched->item_taps > 0.0;
  const bool mom = p.kind == ITEM_MOMENTS;  // items of images, otherwise of taps
  double target = fixed ? std::max(1e3, sched->item_taps) : item_target(p.total_taps, p.wt, p.half, mom, nS, sched);
  const double resident = resident_items(p.kind, p.lut);
  if (!fixed && !mom && p.total_taps < resident * target)
    target = std::min(target, small_call_floor(p.total_taps, resident));
  // Tail taper: tiles are dispatched last first, and the items of a tile
  // dispatched when the work left (this tile included) is below tail_rounds
  // rounds of the resident waves are cut to that work over tail_rounds x the
  // resident waves, down to target / 8 but not below kSmallItemTaps, so the
  // last waves of a launch finish close together instead of one full-size
  // item after another. FP32 items end with a convolution, so theirs are only
  // halved (16 RIRs of 11200 samples: 145 us per call, without any taper 178).
  auto rounds = [&](double deflt) {
    return (fixed || !taper) ? 0.0 : (sched && sched->tail_rounds >= 0.0 ? sched->tail_rounds : deflt);
  };
  auto taps_floor = [](double tgt) { return std::min(tgt, std::max(kSmallItemTaps, tgt / 8.0)); };
  // FP32 calls take fewer, larger items than the other taps, but ask for the
  // workspace of items cut by taps: a call's workspace, and with it what fits a
  // fixed one, does not depend on how its items are cut, and a schedule that
  // asks for more items than that is cut by taps as well
  uint64_t n_items = 0, n_split = 0;
  size_t ws_arrays = 0;  // bytes of the partial tiles and margins the workspace is sized for
  auto arrays = [&](uint64_t items, uint64_t split, int T) { return item_arrays(items, split > 0, T, p.wt); };
  if (!p.half && !fixed && taper) {
    double tt = item_target(p.total_taps, p.wt, false, false, nS, sched);
    const double res = resident_items(ITEM_FP16, false);
    if (p.total_taps < res * tt) tt = std::min(tt, small_call_floor(p.total_taps, res));
    double taps[MAX_TILES];
    const int n = shell_taps(*r, p, TILE, taps);
    if (!cut_tiles(p, taps, n, tt, taps_floor(tt), rounds(kTailRounds), res, nullptr, n_items, n_split))
      return ISM_E_TOO_LARGE;
    ws_arrays = arrays(n_items, n_split, TILE);
  }
  for (;;) {
    if (!cut_tiles(p, p.tile_taps, pa.n_tiles, target, mom ? target / 2.0 : taps_floor(target), rounds(kTailRounds),
                   resident, pa.chunks, n_items, n_split))
      return ISM_E_TOO_LARGE;
    if (ws_arrays == 0 || arrays(n_items, n_split, ra.tile) <= ws_arrays || n_split == 0) break;
    target *= 2.0;
  }
  ws_arrays = std::max(ws_arrays, arrays(n_items, n_split, ra.tile));
  p.any_split = n_split > 0;
  uint64_t acc = 0;
  for (int pos = 0; pos < pa.n_tiles; ++pos) {
    if (pos % PLAN_BLK == 0) pa.first_blk[pos / PLAN_BLK] = (uint32_t)acc;
    acc += (uint64_t)p.n_rir * pa.chunks[pa.n_tiles - 1 - pos];
  }
  pa.first_blk[(pa.n_tiles + PLAN_BLK - 1) / PLAN_BLK] = (uint32_t)acc;
  p.n_items = (uint32_t)acc;

  p.off_valid = 0;
  p.off_origin = align_up(sizeof(int) * (size_t)p.n_rir);
  p.off_tab = align_up(p.off_origin + sizeof(AxisOrigin) * (size_t)p.n_rir);
  p.off_part = align_up(p.off_tab + sizeof(AxisEntry) * (size_t)p.n_rir * ra.n_tab);
  p.off_marg = align_up(p.off_part + (p.any_split ? sizeof(float) * (size_t)p.n_items * ra.tile : 0));
  // general-mode window constants
  p.off_wc = align_up(p.off_marg + sizeof(float) * (size_t)p.n_items * p.wt);
  // host-position calls copy src then rcv here
  p.off_pos = align_up(p.off_wc + (p.gen ? sizeof(float) * WC_STRIDE * (size_t)p.wt : 0));
  size_t o = p.off_part + ws_arrays;
  o = align_up(o + (p.gen ? sizeof(float) * WC_STRIDE * (size_t)p.wt : 0));
  p.ws_bytes = align_up(o + sizeof(float) * 3 * ((size_t)n_src + (size_t)n_rcv));
  return ISM_OK;
}

}  // namespace

extern "C" {

const char *ism_status_string(int status) {
  switch (status) {
    case ISM_OK: return "ok";
    case ISM_E_INVALID_ARG: return "invalid argument";
    case ISM_E_INFEASIBLE_T60: return "T60 infeasible by Sabine's formula (absorption > 1)";
    case ISM_E_OUT_OF_ROOM: return "position not strictly inside the room";
    case ISM_E_WORKSPACE: return "workspace missing or too small";
    case ISM_E_DEVICE: return "HIP device error";
    case ISM_E_TOO_LARGE: return "problem exceeds a library limit";
    case ISM_E_UNSUPPORTED: return "request not supported by the library";
    default: return "unknown status";
  }
}

int ism_abi_version(void) { return ISM_ABI_VERSION; }

int ism_beta_from_t60(const double room[3], double t60, double beta_out[6]) {
  if (!room || !beta_out) return ISM_E_INVALID_ARG;
  if (!finite_pos(room[0]) || !finite_pos(room[1]) || !finite_pos(room[2]) || !finite_pos(t60)) return ISM_E_INVALID_ARG;
  const double V = room[0] * room[1] * room[2];
  const double S = 2.0 * (room[0] * room[1] + room[0] * room[2] + room[1] * room[2]);
  const double alpha = 0.161 * V / (S * t60);  // Eq. (7) with one alpha for all walls
  if (alpha > 1.0) return ISM_E_INFEASIBLE_T60;
  const double b = std::sqrt(1.0 - alpha);  // alpha = 1 - beta^2
  for (int i = 0; i < 6; ++i) beta_out[i] = b;
  return ISM_OK;
}

int ism_n_img_for_time(const double room[3], double c, double t, int n_out[3]) {
  if (!room || !n_out) return ISM_E_INVALID_ARG;
  if (!finite_pos(c) || !finite_pos(t)) return ISM_E_INVALID_ARG;
  for (int a = 0; a < 3; ++a) {
    if (!finite_pos(room[a])) return ISM_E_INVALID_ARG;
    const double k = std::ceil(c * t / (2.0 * room[a]));
    if (k > (ISM_MAX_N_IMG - 2) / 4) return ISM_E_TOO_LARGE;
    n_out[a] = 4 * (int)k + 2;
  }
  return ISM_OK;
}

int ism_time_for_attenuation(double t60, double att_db, double *t_out) {
  if (!t_out || !finite_pos(t60) || !std::isfinite(att_db) || att_db < 0.0) return ISM_E_INVALID_ARG;
  *t_out = t60 * att_db / 60.0;
  return ISM_OK;
}

int64_t ism_n_samples(double t_max, double fs) {
  if (!finite_pos(t_max) || !finite_pos(fs)) return -1;
  const double v = t_max * fs;
  if (v > 9.0e15) return -1;
  const double r = std::nearbyint(v);
  if (std::fabs(v - r) <= 1e-9 * v) return (int64_t)r;
  return (int64_t)std::ceil(v);
}

int ism_check_room(const ism_room *r) {
  if (!r) return ISM_E_INVALID_ARG;
  for (int a = 0; a < 3; ++a) {
    if (!finite_pos(r->room[a])) return ISM_E_INVALID_ARG;
    if (r->n_img[a] < 1) return ISM_E_INVALID_ARG;
    if (r->n_img[a] > ISM_MAX_N_IMG) return ISM_E_TOO_LARGE;
  }
  for (int i = 0; i < 6; ++i)
    if (!std::isfinite(r->beta[i]) || std::fabs(r->beta[i]) > 1.0) return ISM_E_INVALID_ARG;
  if (!finite_pos(r->c) || !finite_pos(r->fs) || !finite_pos(r->t_max) || !finite_pos(r->t_w)) return ISM_E_INVALID_ARG;
  const int64_t nS = ism_n_samples(r->t_max, r->fs);
  if (nS < 1) return ISM_E_INVALID_ARG;
  if (nS > ISM_MAX_SAMPLES) return ISM_E_TOO_LARGE;
  return ISM_OK;
}

int ism_check_positions(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv) {
  int st = ism_check_room(room);
  if (st != ISM_OK) return st;
  if (!src || !rcv || n_src < 1 || n_rcv < 1) return ISM_E_INVALID_ARG;
  auto inside = [&](const float *p) {
    for (int a = 0; a < 3; ++a)
      if (!(std::isfinite(p[a]) && p[a] > 0.0f && (double)p[a] < room->room[a])) return false;
    return true;
  };
  for (int i = 0; i < n_src; ++i)
    if (!inside(src + 3 * i)) return ISM_E_OUT_OF_ROOM;
  for (int i = 0; i < n_rcv; ++i)
    if (!inside(rcv + 3 * i)) return ISM_E_OUT_OF_ROOM;
  for (int i = 0; i < n_src; ++i)
    for (int j = 0; j < n_rcv; ++j)
      if (src[3 * i] == rcv[3 * j] && src[3 * i + 1] == rcv[3 * j + 1] && src[3 * i + 2] == rcv[3 * j + 2])
        return ISM_E_INVALID_ARG;
  return ISM_OK;
}

int ism_count_taps(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv,
                   int64_t *taps_out) {
  if (!taps_out) return ISM_E_INVALID_ARG;
  int st = ism_check_room(room);
  if (st != ISM_OK) return st;
  if (!src || !rcv || n_src < 1 || n_rcv < 1) return ISM_E_INVALID_ARG;
  const double W = room->t_w * room->fs, hw = W / 2.0;
  const double q = room->fs / room->c;
  const int64_t nS = ism_n_samples(room->t_max, room->fs);
  const int n_pairs = n_src * n_rcv;
  std::atomic<int> next{0};
  std::atomic<int64_t> total{0};
  auto worker = [&]() {
    for (;;) {
      const int pidx = next.fetch_add(1);
      if (pidx >= n_pairs) return;
      const float *s = src + 3 * (pidx / n_rcv);
      const float *r = rcv + 3 * (pidx % n_rcv);
      // per-axis squared displacements (samples^2) of every lattice index
      std::vector<double> d2[3];
      for (int a = 0; a < 3; ++a) {
        for (int n = lattice_lo(room->n_img[a]); n < lattice_hi(room->n_img[a]); ++n) {
          const double coord = (n % 2 == 0) ? n * room->room[a] + s[a] : (n + 1) * room->room[a] - s[a];
          const double dd = (coord - r[a]) * q;
          d2[a].push_back(dd * dd);
        }
      }
      int64_t cnt = 0;
      for (double dx : d2[0])
        for (double dy : d2[1])
          for (double dz : d2[2]) {
            const double x = std::sqrt(dx + dy + dz);
            int64_t first = (int64_t)std::floor(x - hw) + 1;
            int64_t last = (int64_t)std::ceil(x + hw) - 1;
            if (first < 0) first = 0;
            if (last > nS - 1) last = nS - 1;
            if (last >= first) cnt += last - first + 1;
          }
      total.fetch_add(cnt);
    }
  };
  const unsigned hc = std::max(1u, std::min(std::thread::hardware_concurrency(), (unsigned)n_pairs));
  std::vector<std::thread> th;
  for (unsigned i = 1; i < hc; ++i) th.emplace_back(worker);
  worker();
  for (auto &t : th) t.join();
  *taps_out = total.load();
  return ISM_OK;
}

int ism_workspace_size_ex(const ism_room *room, int n_src, int n_rcv, int precision, const ism_schedule *sched,
                          size_t *bytes) {
  if (!bytes) return ISM_E_INVALID_ARG;
  Plan p;
  const int st = make_plan(room, n_src, n_rcv, precision, p, sched);
  if (st != ISM_OK) return st;
  *bytes = p.ws_bytes;
  return ISM_OK;
}

int ism_workspace_size(const ism_room *room, int n_src, int n_rcv, int precision, size_t *bytes) {
  return ism_workspace_size_ex(room, n_src, n_rcv, precision, nullptr, bytes);
}

int ism_simulate(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv, int precision,
                 float *out, void *ws, size_t ws_bytes, void *stream) {
  return ism_simulate_ex(room, src, n_src, rcv, n_rcv, precision, nullptr, out, ws, ws_bytes, stream, nullptr,
                         nullptr);
}

// Launches the ISM kernels of a plan: tables, taps, completion of the tiles.
// ws holds at least p.ws_bytes; out is device [n_rir][nS].
// orient: device [n_rcv][3] receiver orientations for a polar call (p.ra.dir_a,
// dir_b set), else null.
static int run_plan(const Plan &p, const float *src, const float *rcv, float *out, void *ws, void *stream,
                    void *ev_start, void *ev_stop, const float *orient = nullptr) {
  hipStream_t s = (hipStream_t)stream;
  char *w = (char *)ws;
  int *valid = (int *)(w + p.off_valid);
  AxisOrigin *origin = (AxisOrigin *)(w + p.off_origin);
  AxisEntry *tab = (AxisEntry *)(w + p.off_tab);
  float *part = p.any_split ? (float *)(w + p.off_part) : nullptr;
  float *marg = (float *)(w + p.off_marg);
  float *wc = p.gen ? (float *)(w + p.off_wc) : nullptr;
  if (launch_tables(p.ra, src, rcv, orient, tab, origin, valid, p.n_rir, (float)p.win, p.half, wc, s) != 0)
    return ISM_E_DEVICE;
  if (ev_start && hipEventRecord((hipEvent_t)ev_start, s) != hipSuccess) return ISM_E_DEVICE;
  if (launch_accumulate(p.wt, p.gen, p.kind, p.lut, orient != nullptr, p.ra, p.pa, p.n_items, tab, origin, valid, out,
                        part, marg, wc, s) != 0)
    return ISM_E_DEVICE;
  if (ev_stop && hipEventRecord((hipEvent_t)ev_stop, s) != hipSuccess) return ISM_E_DEVICE;
  // split tiles and the margins between neighbouring tiles
  if ((p.any_split || p.pa.n_tiles > 1) && launch_reduce(p.ra, p.pa, p.n_rir, part, marg, out, s) != 0)
    return ISM_E_DEVICE;
  return ISM_OK;
}

int ism_simulate_ex(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv, int precision,
                    const ism_schedule *sched, float *out, void *ws, size_t ws_bytes, void *stream, void *ev_start,
                    void *ev_stop) {
  Plan p;
  const int st = make_plan(room, n_src, n_rcv, precision, p, sched);
  if (st != ISM_OK) return st;
  if (!src || !rcv || !out) return ISM_E_INVALID_ARG;
  if (!ws || ws_bytes < p.ws_bytes) return ISM_E_WORKSPACE;
  return run_plan(p, src, rcv, out, ws, stream, ev_start, ev_stop);
}

int ism_simulate_timed(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv,
                       int precision, float *out, void *ws, size_t ws_bytes, void *stream, void *ev_start,
                       void *ev_stop) {
  return ism_simulate_ex(room, src, n_src, rcv, n_rcv, precision, nullptr, out, ws, ws_bytes, stream, ev_start,
                         ev_stop);
}

int ism_simulate_host(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv,
                      int precision, float *out, void *ws, size_t ws_bytes, void *stream) {
  Plan p;
  int st = make_plan(room, n_src, n_rcv, precision, p);
  if (st != ISM_OK) return st;
  if (!src || !rcv || !out) return ISM_E_INVALID_ARG;
  st = ism_check_positions(room, src, n_src, rcv, n_rcv);
  if (st != ISM_OK) return st;
  if (!ws || ws_bytes < p.ws_bytes) return ISM_E_WORKSPACE;
  // positions into the workspace: pageable host memory, so the call returns
  // once the host arrays have been read
  hipStream_t s = (hipStream_t)stream;
  float *pos = (float *)((char *)ws + p.off_pos);
  if (hipMemcpyAsync(pos, src, sizeof(float) * 3 * (size_t)n_src, hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemcpyAsync(pos + 3 * (size_t)n_src, rcv, sizeof(float) * 3 * (size_t)n_rcv, hipMemcpyHostToDevice, s) !=
          hipSuccess)
    return ISM_E_DEVICE;
  return run_plan(p, pos, pos + 3 * (size_t)n_src, out, ws, stream, nullptr, nullptr);
}

int ism_debug_enumerate(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv,
                        const ism_schedule *sched, void *records, uint32_t cap, uint32_t *count, void *ws,
                        size_t ws_bytes, void *stream) {
  return ism_debug_enumerate_ex(room, src, n_src, rcv, n_rcv, ISM_FP32, sched, records, cap, count, ws, ws_bytes,
                                stream);
}

int ism_debug_enumerate_ex(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv,
                           int precision, const ism_schedule *sched, void *records, uint32_t cap, uint32_t *count,
                           void *ws, size_t ws_bytes, void *stream) {
  Plan p;
  const int st = make_plan(room, n_src, n_rcv, precision, p, sched);
  if (st != ISM_OK) return st;
  if (!src || !rcv || !count || (cap > 0 && !records)) return ISM_E_INVALID_ARG;
  if (!ws || ws_bytes < p.ws_bytes) return ISM_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  char *w = (char *)ws;
  int *valid = (int *)(w + p.off_valid);
  AxisOrigin *origin = (AxisOrigin *)(w + p.off_origin);
  AxisEntry *tab = (AxisEntry *)(w + p.off_tab);
  if (launch_tables(p.ra, src, rcv, nullptr, tab, origin, valid, p.n_rir, 0.0f, false, nullptr, s) != 0) {
    fprintf(stderr, "ism_debug_enumerate: tables launch failed\n");
    return ISM_E_DEVICE;
  }
  DumpArgs d{(DumpRec *)records, count, cap};
  if (launch_dump(p.half, p.ra, p.pa, p.n_items, tab, origin, valid, d, s) != 0) return ISM_E_DEVICE;
  return ISM_OK;
}

int ism_simulate_polar(const ism_room *room, const float *src, int n_src, const float *rcv, int n_rcv,
                       const float *orient, double pattern, int precision, float *out, void *ws, size_t ws_bytes,
                       void *stream) {
  Plan p;
  const int st = make_plan(room, n_src, n_rcv, precision, p);
  if (st != ISM_OK) return st;
  if (!src || !rcv || !out || !orient) return ISM_E_INVALID_ARG;
  if (!(pattern >= 0.0 && pattern <= 1.0)) return ISM_E_INVALID_ARG;
  if (!ws || ws_bytes < p.ws_bytes) return ISM_E_WORKSPACE;
  p.ra.dir_a = (float)pattern;
  p.ra.dir_b = (float)(1.0 - pattern);
  return run_plan(p, src, rcv, out, ws, stream, nullptr, nullptr, orient);
}

// ---- Diffuse tail (Sec. 2.2, Eq. (8); Sec. 3.3) ------------------------------
// The ISM part is planned as a call with t_max = t_diff; its RIRs go to the
// workspace after the plan's own arrays, and the diffuse kernel writes the
// full RIRs (ISM part copied, tail drawn) to out.
static int diffuse_plan(const ism_room *r, double t_diff, double t60, int n_src, int n_rcv, int precision, Plan &p,
                        int64_t &n_full, size_t &off_ism, size_t &ws_bytes) {
  if (!r) return ISM_E_INVALID_ARG;
  if (!(t_diff > 0.0) || !(t60 > 0.0) || !std::isfinite(t_diff) || !std::isfinite(t60)) return ISM_E_INVALID_ARG;
  const int rs = ism_check_room(r);
  if (rs != ISM_OK) return rs;
  if (!(t_diff <= r->t_max)) return ISM_E_INVALID_ARG;
  ism_room ri = *r;
  ri.t_max = t_diff;
  const int st = make_plan(&ri, n_src, n_rcv, precision, p);
  if (st != ISM_OK) return st;
  n_full = ism_n_samples(r->t_max, r->fs);
  if (p.ra.n_samples > n_full) return ISM_E_INVALID_ARG;
  off_ism = align_up(p.ws_bytes);
  ws_bytes = off_ism + sizeof(float) * (size_t)p.n_rir * (size_t)p.ra.n_samples;
  return ISM_OK;
}

int ism_diffuse_workspace_size(const ism_room *room, double t_diff, double t60, int n_src, int n_rcv, int precision,
                               size_t *bytes) {
  if (!bytes) return ISM_E_INVALID_ARG;
  Plan p;
  int64_t n_full;
  size_t off_ism, ws;
  const int st = diffuse_plan(room, t_diff, t60, n_src, n_rcv, precision, p, n_full, off_ism, ws);
  if (st != ISM_OK) return st;
  *bytes = ws;
  return ISM_OK;
}

int ism_simulate_diffuse(const ism_room *room, double t_diff, double t60, uint64_t seed, const float *src, int n_src,
                         const float *rcv, int n_rcv, int precision, float *out, void *ws, size_t ws_bytes,
                         void *stream) {
  return ism_simulate_diffuse_timed(room, t_diff, t60, seed, src, n_src, rcv, n_rcv, precision, out, ws, ws_bytes,
                                    stream, nullptr, nullptr);
}

// Diffuse RIRs; orient != null makes the receivers directional (pattern a).
static int simulate_diffuse(const ism_room *room, double t_diff, double t60, uint64_t seed, const float *src,
                            int n_src, const float *rcv, int n_rcv, const float *orient, double pattern,
                            int precision, float *out, void *ws, size_t ws_bytes, void *stream, void *ev_start,
                            void *ev_stop) {
  Plan p;
  int64_t n_full;
  size_t off_ism, need;
  const int st = diffuse_plan(room, t_diff, t60, n_src, n_rcv, precision, p, n_full, off_ism, need);
  if (st != ISM_OK) return st;
  if (!src || !rcv || !out) return ISM_E_INVALID_ARG;
  if (orient && !(pattern >= 0.0 && pattern <= 1.0)) return ISM_E_INVALID_ARG;
  if (!ws || ws_bytes < need) return ISM_E_WORKSPACE;
  if (orient) {
    p.ra.dir_a = (float)pattern;
    p.ra.dir_b = (float)(1.0 - pattern);
  }
  float *ism = (float *)((char *)ws + off_ism);
  const int rs = run_plan(p, src, rcv, ism, ws, stream, ev_start, ev_stop, orient);
  if (rs != ISM_OK) return rs;
  if (launch_diffuse(ism, p.ra.n_samples, out, (int)n_full, p.n_rir, room->fs, t_diff, t60, seed,
                     (hipStream_t)stream) != 0)
    return ISM_E_DEVICE;
  return ISM_OK;
}

int ism_simulate_diffuse_timed(const ism_room *room, double t_diff, double t60, uint64_t seed, const float *src,
                               int n_src, const float *rcv, int n_rcv, int precision, float *out, void *ws,
                               size_t ws_bytes, void *stream, void *ev_start, void *ev_stop) {
  return simulate_diffuse(room, t_diff, t60, seed, src, n_src, rcv, n_rcv, nullptr, 1.0, precision, out, ws,
                          ws_bytes, stream, ev_start, ev_stop);
}

int ism_simulate_diffuse_polar(const ism_room *room, double t_diff, double t60, uint64_t seed, const float *src,
                               int n_src, const float *rcv, int n_rcv, const float *orient, double pattern,
                               int precision, float *out, void *ws, size_t ws_bytes, void *stream) {
  if (!orient) return ISM_E_INVALID_ARG;
  return simulate_diffuse(room, t_diff, t60, seed, src, n_src, rcv, n_rcv, orient, pattern, precision, out, ws,
                          ws_bytes, stream, nullptr, nullptr);
}

// ---- batches ------------------------------------------------------------------

namespace {

constexpr int kMaxClasses = kMaxBatchLaunches;

struct BatchState {  // stored in ism_batch::opaque
  uint64_t ws;
  uint64_t off_jobs, off_rirs, off_items, off_red, off_pos, off_valid, off_origin, off_tab, off_part, off_marg,
      off_queue, off_wc;
  uint32_t n_rir, n_red, n_classes, mode;  // mode: 0 FP32, 1 FP16, 2 table taps
  uint32_t polar, n_jobs, any_gen, long_runs;  // polar: directional kernels; any_gen: general-mode windows;
                                               // long_runs: a tile of RED_SLICE_MIN items or more
  uint32_t n_red_split, pad;                    // reduce entries of split tiles (they come first)
  uint32_t class_count[kMaxClasses];
  uint16_t class_code[kMaxClasses];             // cap / 32, general << 4, long tiles << 5, few images << 6, waves per SIMD << 8
};
static_assert(sizeof(BatchState) <= sizeof(ism_batch), "ism_batch too small");

struct BatchPlan {
  std::vector<JobDev> jobs;
  std::vector<BatchRir> rirs;
  std::vector<BatchItem> items;
  std::vector<BatchReduce> red;
  std::vector<size_t> pos_off;  // per job: offset (floats) of its src, rcv, orient in the position area
  BatchState st;
  size_t ws_bytes;
};

// Largest-first order without a comparison sort: items go into buckets of
// their estimated cost, eight per octave, filled from the most expensive down
// (stable: jobs, tiles, RIRs and chunks keep their order inside a bucket).
constexpr int kCostBuckets = 512;
int cost_bucket(double cost) {
  const int b = (int)std::floor(8.0 * std::log2(cost + 1.0));
  return std::max(0, std::min(kCostBuckets - 1, b));
}

// Plans a batch. With fill == false only the counts and the workspace layout
// are computed (ism_batch_workspace_size); with fill == true the job, RIR,
// item and reduce tables are built as well (ism_batch_prepare).
int plan_batch(const ism_job *jobs, int n_jobs, int precision, const ism_schedule *sched, BatchPlan &bp,
               bool fill) {
  if (!jobs || n_jobs < 1) return ISM_E_INVALID_ARG;
  std::memset(&bp.st, 0, sizeof(bp.st));
  // Each job is planned as a single call without the tail taper (tapering
  // every job would only fragment small jobs; the batch's own tail is the
  // largest-first order over all its items), with an item size taken from
  // the whole batch (pass 0).
  std::vector<Plan> plans(n_jobs);
  bool polar = false;
  for (int j = 0; j < n_jobs; ++j) {
    if (!jobs[j].src || !jobs[j].rcv || !jobs[j].out) return ISM_E_INVALID_ARG;
    if (jobs[j].orient) {
      if (!(jobs[j].pattern >= 0.0 && jobs[j].pattern <= 1.0)) return ISM_E_INVALID_ARG;
      polar = true;
    }
  }
  // with any directional job the batch runs the directional kernels; the
  // others take the pattern a = 1, b = 0, whose factor is exactly 1
  // pass 0: every job's estimated work. The batch fills the device with all
  // of it, so its items are sized from the batch's total as a single call
  // sizes them from its own (max(min_item_taps, total / balance_items) of
  // the job's class), FP16 items capped at the tuned batch item size: many small
  // items cost margin and partial writes, a few large ones leave an uneven tail;
  // an FP16 batch with less work than that per resident wave gets items of its
  // work over the resident waves (at least kSmallItemTaps).
  double batch_taps = 0.0;
  int64_t batch_tiles = 0;
  for (int j = 0; j < n_jobs; ++j) {
    Plan &p = plans[j];
    const int stt = make_plan(&jobs[j].room, jobs[j].n_src, jobs[j].n_rcv, precision, p, sched, false);
    if (stt != ISM_OK) return stt;
    batch_taps += p.total_taps;
    batch_tiles += rir_tiles(p);
  }
  // one kind of items for the whole batch: two are two launches, each with a tail of its own
  TileImages images{0.0, 0.0};
  for (int j = 0; j < n_jobs; ++j) {
    const TileImages t = tile_images(jobs[j].room, plans[j]);
    images.mean += t.mean * (double)rir_tiles(plans[j]) / (double)batch_tiles;
    images.fullest = std::max(images.fullest, t.fullest);
  }
  int kind = plans[0].kind;  // of one job: that of its single call
  if (n_jobs > 1 && precision != ISM_FP16)
    kind = few_images_batch(images, precision == ISM_FP32_LUT, batch_tiles) ? ITEM_FEW : ITEM_MOMENTS;
  // pass 1: plans, window classes and counts
  int n_classes = 0;
  int class_wt[kMaxClasses] = {}, class_gen[kMaxClasses] = {}, class_tile[kMaxClasses] = {}, class_kind[kMaxClasses] = {},
      n_windows = 0;
  std::vector<int> job_cls(n_jobs);
  uint64_t tab_entries = 0, n_rir = 0, n_items = 0, slots = 0, n_red = 0, marg_units = 0, wc_floats = 0,
           max_chunks = 0, ws_items = 0, ws_slots = 0, ws_marg = 0, ws_red = 0;  // ws: counts the workspace is sized for
  std::vector<uint64_t> bucket_count((size_t)kMaxClasses * kCostBuckets, 0);
  for (int j = 0; j < n_jobs; ++j) {
    Plan &p = plans[j];
    if (!(sched && sched->item_taps > 0.0)) {
      ism_schedule js{};
      if (sched) js = *sched;
      p.kind = kind;
      const bool mom = p.kind == ITEM_MOMENTS;
      double t = item_target(batch_taps, p.wt, p.half, mom, p.ra.n_samples, sched);
      if (!mom) t = std::min(t, batch_item_taps(p.wt, p.half));
      // a batch too small to give every resident wave an item of that size is
      // spread over them instead (the small-call rule of single calls)
      const double resident = resident_items(p.kind, p.lut);
      js.item_taps = !mom && batch_taps < resident * t ? std::min(t, small_call_floor(batch_taps, resident)) : t;
      size_t ws_arrays = 0;
      if (!p.half) {  // the workspace is that of items cut by taps, as for single calls
        const double res = resident_items(ITEM_FP16, false);
        double tt = std::min(batch_item_taps(p.wt, false),
                             item_target(batch_taps, p.wt, false, false, p.ra.n_samples, sched));
        if (batch_taps < res * tt) tt = std::min(tt, small_call_floor(batch_taps, res));
        uint64_t n = 0, ns = 0;
        double taps[MAX_TILES];
        const int nt = shell_taps(jobs[j].room, p, TILE, taps);
        if (!cut_tiles(p, taps, nt, tt, tt, 0.0, res, nullptr, n, ns)) return ISM_E_TOO_LARGE;
        ws_arrays = item_arrays(n, ns > 0, TILE, p.wt);
        ws_items += n;
        ws_slots += ns;
        ws_marg += n * (uint64_t)(p.wt / MARG_UNIT);
        ws_red += (uint64_t)nt * p.n_rir;
      }
      for (;;) {  // items that outgrow it are doubled, as in a single call
        const int stt = make_plan(&jobs[j].room, jobs[j].n_src, jobs[j].n_rcv, precision, p, &js, false, p.kind);
        if (stt != ISM_OK) return stt;
        if (p.half || !p.any_split || item_arrays(p.n_items, true, p.ra.tile, p.wt) <= ws_arrays) break;
        js.item_taps *= 2.0;
      }
    }
    int cls = -1;
    bool window_known = false;
    for (int k = 0; k < n_classes; ++k)
      if (class_wt[k] == p.wt && class_gen[k] == (p.gen ? 1 : 0)) {
        window_known = true;
        if (class_tile[k] == p.ra.tile && class_kind[k] == p.kind) cls = k;
      }
    if (cls < 0) {
      if (!window_known && n_windows++ == kMaxBatchClasses) return ISM_E_UNSUPPORTED;
      cls = n_classes++;
      class_wt[cls] = p.wt;
      class_gen[cls] = p.gen ? 1 : 0;
      class_tile[cls] = p.ra.tile;
      class_kind[cls] = p.kind;
    }
    job_cls[j] = cls;
    if (p.gen) wc_floats += (uint64_t)WC_STRIDE * p.wt;
    for (int t = 0; t < p.pa.n_tiles; ++t) {
      const uint64_t C = p.pa.chunks[t];
      max_chunks = std::max(max_chunks, C);
      n_items += C * p.n_rir;
      marg_units += C * p.n_rir * (uint64_t)(p.wt / MARG_UNIT);
      if (C > 1) slots += C * p.n_rir * (uint64_t)(p.ra.tile / TILE);
      bucket_count[(size_t)cls * kCostBuckets + cost_bucket(p.tile_taps[t] / C)] += C * p.n_rir;
    }
    n_red += (uint64_t)p.pa.n_tiles * p.n_rir;
    tab_entries += (uint64_t)p.n_rir * p.ra.n_tab;
    n_rir += (uint64_t)p.n_rir;
  }
  if (n_rir > 0x7fffffffULL || n_items > 0x7fffffffULL || slots > 0xffffffffULL || n_red > 0x7fffffffULL ||
      marg_units > 0xffffffffULL)
    return ISM_E_TOO_LARGE;
  // item positions: classes in order, each class from its most expensive bucket down
  std::vector<uint64_t> bucket_next((size_t)kMaxClasses * kCostBuckets, 0);
  uint64_t acc = 0;
  for (int k = 0; k < n_classes; ++k) {
    const uint64_t first = acc;
    for (int b = kCostBuckets - 1; b >= 0; --b) {
      bucket_next[(size_t)k * kCostBuckets + b] = acc;
      acc += bucket_count[(size_t)k * kCostBuckets + b];
    }
    bp.st.class_count[k] = (uint32_t)(acc - first);
    // persistent grid: the tuned waves per SIMD (or the schedule's)
    int waves = waves_per_simd(class_kind[k], precision == ISM_FP32_LUT);
    if (precision == ISM_FP16)
      for (const BatchTuning &t : kBatchTuning)
        if (t.wt == class_wt[k] && t.half == 1) waves = t.waves;
    if (sched && sched->batch_waves > 0.0) waves = std::max(1, (int)std::lround(sched->batch_waves));
    bp.st.class_code[k] =
        (uint16_t)(class_wt[k] / 32 | class_gen[k] << 4 | (class_tile[k] == LONG_TILE ? 1 : 0) << 5 |
                   (class_kind[k] == ITEM_FEW ? 1 : 0) << 6 | waves << 8);
  }
  bp.st.n_jobs = (uint32_t)n_jobs;
  bp.st.any_gen = wc_floats > 0 ? 1u : 0u;
  bp.st.long_runs = max_chunks >= (uint64_t)RED_SLICE_MIN ? 1u : 0u;
  bp.st.n_classes = (uint32_t)n_classes;
  bp.st.mode = precision == ISM_FP16 ? 1u : precision == ISM_FP32_LUT ? 2u : 0u;
  bp.st.polar = polar ? 1u : 0u;
  bp.st.n_rir = (uint32_t)n_rir;
  bp.st.n_red = (uint32_t)n_red;
  if (ws_items > 0x7fffffffULL || ws_slots > 0xffffffffULL || ws_marg > 0xffffffffULL || ws_red > 0x7fffffffULL)
    return ISM_E_TOO_LARGE;
  // positions of every job (ism_simulate_batch copies host positions here)
  bp.pos_off.resize(n_jobs);
  size_t pos_floats = 0;
  for (int j = 0; j < n_jobs; ++j) {
    bp.pos_off[j] = pos_floats;
    pos_floats += 3 * ((size_t)jobs[j].n_src + (size_t)jobs[j].n_rcv * (jobs[j].orient ? 2 : 1));
  }
  auto layout = [&](uint64_t items, uint64_t part_slots, uint64_t marg, uint64_t red, BatchState &st) {
    size_t o = 0;
    st.off_jobs = o;
    o = align_up(o + sizeof(JobDev) * (size_t)n_jobs);
    st.off_rirs = o;
    o = align_up(o + sizeof(BatchRir) * (size_t)n_rir);
    st.off_items = o;
    o = align_up(o + sizeof(BatchItem) * (size_t)items);
    st.off_red = o;
    o = align_up(o + sizeof(BatchReduce) * (size_t)red);
    st.off_pos = o;
    o = align_up(o + sizeof(float) * pos_floats);
    st.off_valid = o;
    o = align_up(o + sizeof(int) * n_rir);
    st.off_origin = o;
    o = align_up(o + sizeof(AxisOrigin) * n_rir);
    st.off_tab = o;
    o = align_up(o + sizeof(AxisEntry) * tab_entries);
    st.off_part = o;
    o = align_up(o + sizeof(float) * (size_t)part_slots * TILE);
    st.off_marg = o;
    o = align_up(o + sizeof(float) * MARG_UNIT * (size_t)marg);
    // work-queue counters of the persistent launches, one per window class
    st.off_queue = o;
    o = align_up(o + sizeof(uint32_t) * kMaxClasses);
    // general-mode window constants, one block per such job
    st.off_wc = o;
    return align_up(o + sizeof(float) * (size_t)wc_floats);
  };
  BatchState unused = {};
  bp.ws_bytes = layout(n_items, slots, marg_units, n_red, bp.st);
  bp.ws_bytes = std::max(bp.ws_bytes, layout(ws_items, ws_slots, ws_marg, ws_red, unused));
  if (!fill) return ISM_OK;

  // pass 2: tables. Margin records are numbered in (job, tile, RIR, chunk)
  // order, so the records of one (tile, RIR) are contiguous.
  bp.jobs.resize(n_jobs);
  bp.rirs.resize(n_rir);
  bp.items.resize(n_items);
  bp.red.resize(n_red);
  uint64_t rir_base = 0, tab_base = 0, mslot = 0, red_i = 0, wc_base = 0;
  uint32_t slot = 0;
  for (int j = 0; j < n_jobs; ++j) {
    const Plan &p = plans[j];
    const ism_job &jb = jobs[j];
    JobDev &d = bp.jobs[j];
    std::memset(&d, 0, sizeof(d));
    d.ra = p.ra;
    d.ra.dir_a = jb.orient ? (float)jb.pattern : 1.0f;
    d.ra.dir_b = jb.orient ? (float)(1.0 - jb.pattern) : 0.0f;
    d.src = jb.src;
    d.rcv = jb.rcv;
    d.out = jb.out;
    d.orient = jb.orient;
    d.tab_base = tab_base;
    d.rir_base = (uint32_t)rir_base;
    if (p.gen) {  // device address filled in by prepare_batch (ws base unknown here)
      d.wc = (float *)(uintptr_t)(wc_base + 1);
      wc_base += (uint64_t)WC_STRIDE * p.wt;
    }
    for (int r = 0; r < p.n_rir; ++r) bp.rirs[rir_base + r] = BatchRir{(uint32_t)j, (uint32_t)r};
    const int nt = p.pa.n_tiles;
    const uint32_t su = (uint32_t)(p.ra.tile / TILE);  // partial tile, in units of TILE floats
    // margin records (units of MARG_UNIT floats, wu units each): the first
    // record of (tile t, RIR r) is mfirst_t + r * chunks[t] * wu
    const uint64_t wu = (uint64_t)(p.wt / MARG_UNIT);
    std::vector<uint64_t> mfirst(nt);
    for (int t = 0; t < nt; ++t) {
      mfirst[t] = mslot;
      mslot += (uint64_t)p.pa.chunks[t] * p.n_rir * wu;
    }
    for (int t = 0; t < nt; ++t) {
      const int C = p.pa.chunks[t];
      uint64_t &pos = bucket_next[(size_t)job_cls[j] * kCostBuckets + cost_bucket(p.tile_taps[t] / C)];
      for (int r = 0; r < p.n_rir; ++r) {
        BatchReduce &rd = bp.red[red_i++];
        std::memset(&rd, 0, sizeof(rd));
        rd.job = (uint32_t)j;
        rd.rir = (uint32_t)r;
        rd.tile = (uint16_t)t;
        rd.chunks = (uint16_t)C;
        rd.first = C > 1 ? slot : 0xffffffffu;
        if (t > 0) {
          rd.mprev = (uint32_t)(mfirst[t - 1] + (uint64_t)r * p.pa.chunks[t - 1] * wu);
          rd.nprev = p.pa.chunks[t - 1];
        }
        if (t + 1 < nt) {
          rd.mnext = (uint32_t)(mfirst[t + 1] + (uint64_t)r * p.pa.chunks[t + 1] * wu);
          rd.nnext = p.pa.chunks[t + 1];
        }
        for (int c = 0; c < C; ++c)
          bp.items[pos++] = BatchItem{(uint32_t)j, (uint32_t)r, (uint16_t)t, (uint8_t)c, (uint8_t)C,
                                      C > 1 ? slot + (uint32_t)c * su : 0xffffffffu,
                                      (uint32_t)(mfirst[t] + ((uint64_t)r * C + c) * wu)};
        if (C > 1) slot += (uint32_t)C * su;
      }
    }
    tab_base += (uint64_t)p.n_rir * p.ra.n_tab;
    rir_base += (uint64_t)p.n_rir;
  }
  if (mslot > 0xffffffffULL) return ISM_E_TOO_LARGE;
  // split tiles first (their whole tile is summed), then the tiles whose own
  // samples are already final (only their margin samples change)
  const auto mid = std::stable_partition(bp.red.begin(), bp.red.end(),
                                         [](const BatchReduce &r) { return r.chunks > 1; });
  bp.st.n_red_split = (uint32_t)(mid - bp.red.begin());
  return ISM_OK;
}

}  // namespace

int ism_batch_workspace_size_ex(const ism_job *jobs, int n_jobs, int precision, const ism_schedule *sched,
                                size_t *bytes) {
  if (!bytes) return ISM_E_INVALID_ARG;
  BatchPlan bp;
  const int st = plan_batch(jobs, n_jobs, precision, sched, bp, false);
  if (st != ISM_OK) return st;
  *bytes = bp.ws_bytes;
  return ISM_OK;
}

int ism_batch_workspace_size(const ism_job *jobs, int n_jobs, int precision, size_t *bytes) {
  return ism_batch_workspace_size_ex(jobs, n_jobs, precision, nullptr, bytes);
}

namespace {
// Plans a batch and uploads its tables (and, with host_pos, the jobs' host
// positions) into ws with one host-to-device copy on stream.
int prepare_batch(const ism_job *jobs, int n_jobs, int precision, const ism_schedule *sched, void *ws,
                  size_t ws_bytes, void *stream, bool host_pos, ism_batch *batch) {
  if (!batch) return ISM_E_INVALID_ARG;
  BatchPlan bp;
  int st = plan_batch(jobs, n_jobs, precision, sched, bp, true);
  if (st != ISM_OK) return st;
  if (host_pos) {
    for (int j = 0; j < n_jobs; ++j) {
      st = ism_check_positions(&jobs[j].room, jobs[j].src, jobs[j].n_src, jobs[j].rcv, jobs[j].n_rcv);
      if (st != ISM_OK) return st;
      if (jobs[j].orient)
        for (int i = 0; i < jobs[j].n_rcv; ++i) {
          const float *o = jobs[j].orient + 3 * i;
          if (!(std::isfinite(o[0]) && std::isfinite(o[1]) && std::isfinite(o[2])) ||
              (o[0] == 0.0f && o[1] == 0.0f && o[2] == 0.0f))
            return ISM_E_INVALID_ARG;
        }
    }
  }
  if (!ws || ws_bytes < bp.ws_bytes) return ISM_E_WORKSPACE;
  // one contiguous host image of the metadata, copied with a single transfer
  // (alignment gaps between the tables are left uninitialised)
  std::unique_ptr<char[]> host_buf(new char[bp.st.off_valid]);
  char *const host = host_buf.get();
  if (host_pos) {
    // the jobs' device view points into the position area of ws
    float *dpos = (float *)((char *)ws + bp.st.off_pos);
    float *hpos = (float *)(host + bp.st.off_pos);
    for (int j = 0; j < n_jobs; ++j) {
      const ism_job &jb = jobs[j];
      JobDev &d = bp.jobs[j];
      size_t o = bp.pos_off[j];
      std::memcpy(hpos + o, jb.src, sizeof(float) * 3 * (size_t)jb.n_src);
      d.src = dpos + o;
      o += 3 * (size_t)jb.n_src;
      std::memcpy(hpos + o, jb.rcv, sizeof(float) * 3 * (size_t)jb.n_rcv);
      d.rcv = dpos + o;
      o += 3 * (size_t)jb.n_rcv;
      if (jb.orient) {
        std::memcpy(hpos + o, jb.orient, sizeof(float) * 3 * (size_t)jb.n_rcv);
        d.orient = dpos + o;
      }
    }
  }
  for (JobDev &d : bp.jobs)  // general-mode window constants: offsets into ws
    if (d.wc) d.wc = (float *)((char *)ws + bp.st.off_wc) + ((uintptr_t)d.wc - 1);
  std::memcpy(host + bp.st.off_jobs, bp.jobs.data(), sizeof(JobDev) * bp.jobs.size());
  std::memcpy(host + bp.st.off_rirs, bp.rirs.data(), sizeof(BatchRir) * bp.rirs.size());
  std::memcpy(host + bp.st.off_items, bp.items.data(), sizeof(BatchItem) * bp.items.size());
  if (!bp.red.empty()) std::memcpy(host + bp.st.off_red, bp.red.data(), sizeof(BatchReduce) * bp.red.size());
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = hipMemcpyAsync(ws, host, bp.st.off_valid, hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return device_error("batch tables upload", e);
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return device_error("batch tables upload (synchronize)", e);
  bp.st.ws = (uint64_t)(uintptr_t)ws;
  std::memset(batch, 0, sizeof(*batch));
  std::memcpy(batch, &bp.st, sizeof(bp.st));
  return ISM_OK;
}
}  // namespace

int ism_batch_prepare_ex(const ism_job *jobs, int n_jobs, int precision, const ism_schedule *sched, void *ws,
                         size_t ws_bytes, void *stream, ism_batch *batch) {
  return prepare_batch(jobs, n_jobs, precision, sched, ws, ws_bytes, stream, false, batch);
}

int ism_batch_prepare(const ism_job *jobs, int n_jobs, int precision, void *ws, size_t ws_bytes, void *stream,
                      ism_batch *batch) {
  return prepare_batch(jobs, n_jobs, precision, nullptr, ws, ws_bytes, stream, false, batch);
}

int ism_simulate_batch(const ism_job *jobs, int n_jobs, int precision, void *ws, size_t ws_bytes, void *stream) {
  ism_batch b;
  const int st = prepare_batch(jobs, n_jobs, precision, nullptr, ws, ws_bytes, stream, true, &b);
  if (st != ISM_OK) return st;
  return ism_batch_run(&b, stream);
}

int ism_batch_run(const ism_batch *batch, void *stream) { return ism_batch_run_timed(batch, stream, nullptr, nullptr); }

int ism_batch_run_timed(const ism_batch *batch, void *stream, void *ev_start, void *ev_stop) {
  if (!batch) return ISM_E_INVALID_ARG;
  BatchState b;
  std::memcpy(&b, batch, sizeof(b));
  if (!b.ws || b.n_rir == 0 || b.n_classes == 0 || b.n_classes > (uint32_t)kMaxClasses || b.n_red_split > b.n_red)
    return ISM_E_INVALID_ARG;
  char *w = (char *)(uintptr_t)b.ws;
  BatchClass cls[kMaxClasses];
  uint32_t first = 0;
  int max_tile = TILE;
  for (uint32_t k = 0; k < b.n_classes; ++k) {
    const uint32_t code = b.class_code[k], waves = code >> 8;
    cls[k].first = first;
    cls[k].count = b.class_count[k];
    cls[k].kind = b.mode == 1 ? ITEM_FP16 : (code >> 6 & 1u) ? ITEM_FEW : ITEM_MOMENTS;
    cls[k].grid = std::min(b.class_count[k], 1024u * waves * 64u / (uint32_t)item_threads(cls[k].kind));
    cls[k].wt = (int)(code & 15u) * 32;
    cls[k].gen = (int)(code >> 4 & 1u);
    cls[k].tile = (code >> 5 & 1u) ? LONG_TILE : TILE;
    max_tile = std::max(max_tile, cls[k].tile);
    first += b.class_count[k];
  }
  const int rc = launch_batch((const JobDev *)(w + b.off_jobs), (int)b.n_jobs, b.any_gen != 0,
                              (const BatchRir *)(w + b.off_rirs), b.n_rir, (const BatchItem *)(w + b.off_items), cls,
                              (int)b.n_classes, b.mode == 1, b.mode == 2, b.polar != 0,
                              (const BatchReduce *)(w + b.off_red), b.n_red, b.n_red_split, b.long_runs != 0, max_tile,
                              (AxisEntry *)(w + b.off_tab), (AxisOrigin *)(w + b.off_origin),
                              (int *)(w + b.off_valid), (float *)(w + b.off_part), (float *)(w + b.off_marg),
                              (uint32_t *)(w + b.off_queue), (hipStream_t)stream,
                              (hipEvent_t)ev_start, (hipEvent_t)ev_stop);
  return rc == 0 ? ISM_OK : ISM_E_DEVICE;
}

}  // extern "C"

// ---- Moving-source filtering (Sec. 3.4) --------------------------------------
namespace {
constexpr int kFftMaxPieces = 16;  // segments one FFT input block may touch
constexpr int kAutoMaxPieces = 4;
// Segment blocks take the place of the direct sum from 2048 taps on: there their error
// is no larger than the sum's (2 microphones, segments of 64: 2.1e-7 of the norm and
// 2.2e-7; below, up to 1.2 times it), and they are faster at every segment length (2
// microphones, 16000 samples, 2048 taps, segments of 4, 64 and 200: 79, 24 and 22 us
// against 7500, 455 and 41).
constexpr int kSegMinRir = 2048;
constexpr size_t kSegSpare = 16u << 20;  // beside the RIRs' size, for the partition groups of small calls

int filter_args(const float *x, int n_x, const float *rir, int n_pos, int n_mic, int n_rir, const float *y) {
  if (!x || !rir || !y) return ISM_E_INVALID_ARG;
  if (n_x < 1 || n_pos < 1 || n_mic < 1 || n_rir < 1 || n_pos > n_x) return ISM_E_INVALID_ARG;
  if (n_mic > 65535 || (int64_t)n_x + n_rir - 1 > (int64_t)0x7fffffff) return ISM_E_TOO_LARGE;
  return ISM_OK;
}

// The plans a call may take, in order of preference: segment blocks, fixed blocks, the
// direct sum. Fixed blocks: method FFT, or auto with RIRs of 1024 taps and more when an
// input block touches at most kAutoMaxPieces segments; the direct sum: the other calls.
// The first whose workspace is there is taken.
struct FilterPlans {
  bool seg, fixed;
  FftPlan s, f;
};

int filter_plans(int n_x, int n_pos, int n_mic, int n_rir, int method, FilterPlans &p) {
  if (method != ISM_FILTER_AUTO && method != ISM_FILTER_DIRECT && method != ISM_FILTER_FFT) return ISM_E_INVALID_ARG;
  p.seg = p.fixed = false;
  if (method == ISM_FILTER_DIRECT) return ISM_OK;
  const bool ok = fft_plan(n_x, n_pos, n_mic, n_rir, method == ISM_FILTER_FFT ? kFftMaxPieces : kAutoMaxPieces, p.f);
  if (method == ISM_FILTER_FFT && !ok) return ISM_E_UNSUPPORTED;
  p.fixed = ok && (method == ISM_FILTER_FFT || n_rir >= 1024);
  if (!p.fixed && n_rir < kSegMinRir) return ISM_OK;
  p.seg = seg_plan(n_x, n_pos, n_mic, n_rir, p.s);
  // a call that needed no workspace is not given one larger than its RIRs
  if (!p.fixed && p.seg) p.seg = p.s.bytes <= sizeof(float) * (size_t)n_pos * n_mic * n_rir + kSegSpare;
  return ISM_OK;
}

}  // namespace

int ism_filter_workspace_size(int n_x, int n_pos, int n_mic, int n_rir, int method, size_t *bytes) {
  if (!bytes) return ISM_E_INVALID_ARG;
  if (n_x < 1 || n_pos < 1 || n_mic < 1 || n_rir < 1 || n_pos > n_x) return ISM_E_INVALID_ARG;
  if (n_mic > 65535 || (int64_t)n_x + n_rir - 1 > (int64_t)0x7fffffff) return ISM_E_TOO_LARGE;
  FilterPlans p;
  const int st = filter_plans(n_x, n_pos, n_mic, n_rir, method, p);
  if (st != ISM_OK) return st;
  *bytes = p.seg ? p.s.bytes : p.fixed ? p.f.bytes : 0;
  return ISM_OK;
}

int ism_filter_trajectory_ex(const float *x, int n_x, const float *rir, int n_pos, int n_mic, int n_rir, int method,
                             float *y, void *ws, size_t ws_bytes, void *stream) {
  int st = filter_args(x, n_x, rir, n_pos, n_mic, n_rir, y);
  if (st != ISM_OK) return st;
  FilterPlans p;
  st = filter_plans(n_x, n_pos, n_mic, n_rir, method, p);
  if (st != ISM_OK) return st;
  const bool seg = p.seg && ws && ws_bytes >= p.s.bytes;
  if (!seg && !p.fixed) return ism_filter_trajectory(x, n_x, rir, n_pos, n_mic, n_rir, y, stream);
  const FftPlan &f = seg ? p.s : p.f;
  if (!ws || ws_bytes < f.bytes) return ISM_E_WORKSPACE;
  // (segment blocks in place of the direct sum keep what is not finite where it belongs)
  if (launch_filter_fft(x, n_x, rir, n_pos, n_mic, n_rir, y, f, seg && !p.fixed, ws, (hipStream_t)stream) != 0)
    return ISM_E_DEVICE;
  return ISM_OK;
}

int ism_filter_trajectory(const float *x, int n_x, const float *rir, int n_pos, int n_mic, int n_rir, float *y,
                          void *stream) {
  if (!x || !rir || !y) return ISM_E_INVALID_ARG;
  if (n_x < 1 || n_pos < 1 || n_mic < 1 || n_rir < 1 || n_pos > n_x) return ISM_E_INVALID_ARG;
  if (n_mic > 65535 || (int64_t)n_x + n_rir - 1 > (int64_t)0x7fffffff) return ISM_E_TOO_LARGE;
  const int rc = launch_filter(x, n_x, rir, n_pos, n_mic, n_rir, y, (hipStream_t)stream);
  if (rc == -2) return ISM_E_TOO_LARGE;
  if (rc != 0) return ISM_E_DEVICE;
  return ISM_OK;
}
