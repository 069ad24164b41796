// Host side of the C ABI: argument validation, the nano-batch plan (integer bookkeeping), workspace
// layout and the launch sequence of the forward and backward passes.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <list>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "../../include/tlora.h"
#include "tlora_internal.h"
#include "tlora_kernels.h"

// Device memory of tlora_fwd_noalloc: the forward's workspace for callers that cannot allocate.  Every GPU the
// library runs on holds its own copy of this array at its own address until the process ends.  In host code the
// name is only a handle for hipGetSymbolAddress: the address that kernels and fills get is the per-device pointer
// looked up below, never the name.
// (its first part holds what decides whether a problem fits; the fp32 sums of split launches lie behind)
static __device__ __align__(256) unsigned char scratch[TLORA_NOALLOC_SCRATCH_BYTES + TLORA_NOALLOC_SUM_BYTES];

namespace tlora {
namespace {

constexpr int kMaxDevices = 64;
// What the HIP runtime said when a call last failed (for tlora_last_hip_error): the code and the line of this file.
int g_hip_err = 0, g_hip_line = 0;
inline int hip_failed(hipError_t e, int line) {
  g_hip_err = (int)e;  g_hip_line = line;
  return TLORA_EHIP;
}
// TLORA_OK, or TLORA_EHIP if the runtime reports an error from the launches queued so far
inline int launches_ok(int line) {
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? TLORA_OK : hip_failed(e, line);
}
#define TLORA_HIP(expr) do { const hipError_t e_ = (expr); if (e_ != hipSuccess) return hip_failed(e_, __LINE__); } while (0)

constexpr size_t kNoAllocMaxTableBytes = 64 * 3584;   // plan tables of tlora_fwd_noalloc: at most 64 argument chunks
uint8_t* g_scratch_ptr[kMaxDevices] = {};   // per device: address of `scratch` on that device (0 = not looked up yet)

// Address of the static scratch array on the current device (looked up once per device, with that device current).
int scratch_of_current_device(uint8_t** out) {
  int dev = -1;
  TLORA_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return TLORA_EINVAL;
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    TLORA_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return TLORA_EHIP;
    g_scratch_ptr[dev] = static_cast<uint8_t*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return TLORA_OK;
}

struct Options {
  int shrink_rows = 0;          // 0 = chosen per problem (32 | 64 | 128), else forced
  int shrink_stages = 4;
  int grad_tokens = 256;
  int dx_transposed_w = 1;
  int plan_cache = 1;           // reuse plans of problems seen before (keyed by their contents)
  int indexed_direct = 1;       // token-indexed bf16 calls fetch rows through the index inside the kernels' loads
  int table_copy_kernel = 1;    // plan tables reach the workspace through a kernel that reads the pinned staging buffer
};
Options g_opt;
std::recursive_mutex g_mu;   // the nano-batch entry points call tlora_fwd / tlora_bwd under it

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- the plan ---------------------------------------------------------------------------------------
struct Plan {
  int J = 0, T = 0, d_in = 0, d_out = 0, dtype = 0;
  int max_rpad = 0;
  int shrink_rows = 128;                                // token rows per unit of the streaming shrink kernel
  std::vector<JobDev> jobs;
  std::vector<TileDev> tile_jobs;
  std::vector<ShrinkUnit> shrink_units;                 // generic kernel: 64 rows x 64 rank columns
  std::vector<ShrinkUnit> stream_units;                 // streaming kernel: shrink_rows x 128 rank columns
  std::vector<GradUnit> gradB_units, gradA_units;      // dB: columns over d_out;  dA: columns over d_in;

  bool grads_merged = false;                            // dB and dA share a launch
  int64_t grad_partial = 0;                             // floats of partial tiles in use at a time (merged: those of dB first)
  std::vector<GradGroup> gradB_groups, gradA_groups;
  int64_t s_elems = 0;                                  // elements of the packed S (= dS) buffer
  int64_t atp_elems = 0;
  int r_total = 0;                                      // sum of rpad_j
  int64_t sx_elems = 0;                                 // elements of the per-tile K-extension operands
  int shrink_splits_x = 1, shrink_splits_dy = 1;        // contraction splits of the shrinks over d_in (S) and d_out (dS)
  GemmSplit gemm_split_fwd, gemm_split_bwd;             // tiles of the two GEMMs that are cut along the contraction
  GemmSplit pair_split_fwd, pair_split_bwd;             // and of two such GEMMs in one launch
  int small_x = 0, small_dy = 0;                        // splits of a small batch's two-launch form (0: not taken), X and dY side
  bool frags_wait = false;                              // dY's fragments lie behind the sums that making S again writes
  size_t partial_bytes = 0;                             // what off_partial holds: dA / dB tiles, or sums of split launches
  // workspace byte offsets
  size_t off_tables = 0, off_S = 0, off_dS = 0, off_Shi = 0, off_Slo = 0, off_dShi = 0, off_dSlo = 0, off_Sx = 0, off_dSx = 0, off_atp = 0, off_wt = 0, off_wt_state = 0, off_ap = 0,
         off_bp = 0,
         off_partial = 0, total = 0;
  size_t tables_bytes = 0;
  // offsets of each table inside the table blob
  size_t tb_jobs = 0, tb_tiles = 0, tb_shrink = 0, tb_stream = 0, tb_gBu = 0, tb_gBg = 0, tb_gAu = 0, tb_gAg = 0, tb_f32 = 0;
  size_t off_clock = 0;                                 // kClockBytes outside the uploaded tables: GEMM clock probe
  size_t f32_reserved = 0;
};

constexpr size_t kClockBytes = 64;
constexpr int64_t kMaxUnits = (int64_t)1 << 22;   // most GEMM tiles / work units of one kind in a launch

int validate(const tlora_problem_t* p) {
  if (!p) return TLORA_ENULL;
  if (p->dtype != TLORA_F32 && p->dtype != TLORA_BF16) return TLORA_EDTYPE;
  if (p->num_jobs < 1 || p->d_in < 8 || p->d_out < 8 || (p->d_in % 8) || (p->d_out % 8)) return TLORA_EINVAL;
  if (p->num_jobs > TLORA_MAX_JOBS || p->d_in > TLORA_MAX_FEATURES || p->d_out > TLORA_MAX_FEATURES) return TLORA_EINVAL;
  if (!p->ranks || !p->offsets || !p->scales) return TLORA_ENULL;
  if (p->offsets[0] != 0) return TLORA_EINVAL;
  for (int j = 0; j < p->num_jobs; ++j) {
    if (p->offsets[j + 1] < p->offsets[j]) return TLORA_EINVAL;
    if (p->ranks[j] < 0 || p->ranks[j] > TLORA_MAX_RANK) return TLORA_EINVAL;
  }
  if (p->offsets[p->num_jobs] > TLORA_MAX_TOKENS) return TLORA_EINVAL;
  {   // one workgroup per GEMM tile: the grid (and the 32-bit tile index arithmetic) must hold them all
    const int64_t tiles_m = (p->offsets[p->num_jobs] + kGemmBM - 1) / kGemmBM;
    const int64_t tiles_n = (std::max(p->d_in, p->d_out) + kGemmBN - 1) / kGemmBN;
    if (tiles_m * tiles_n > kMaxUnits) return TLORA_EINVAL;
  }
  return TLORA_OK;
}

// Work units of the dA / dB token reductions (rank-aware nano-batches of one job's tokens).  A job's rank rows are cut into blocks
// of 128, of which a unit multiplies only the live 32-row sub-blocks, and its tokens into chunks.  A job of one chunk stores its
// gradient itself; the chunks of others leave partial tiles of live_rows * 256 * 4 bytes that are written and read once more.
// Units are issued longest first.
constexpr int64_t kGradUnitsWanted = 1024;
// Upper bounds over every batch in which no job has more tokens than in this one (see Reserve).
struct GradBounds {
  int64_t units = 0, floats = 0;
};
constexpr int kGradBlockRanks = kGradMaxBlocks * kGradRanks;
int grad_live_blocks(const JobDev& jb, int pb) {
  return std::min(kGradMaxBlocks, (jb.rpad - pb * kGradBlockRanks + kGradRanks - 1) / kGradRanks);
}
// Output tiles of dA / dB (256 columns x 128 ranks) over D columns.
int64_t grad_tiles(const Plan& pl, int D) {
  int64_t n = 0;
  for (const JobDev& jb : pl.jobs) n += jb.rank > 0 ? (jb.rpad + kGradBlockRanks - 1) / kGradBlockRanks : 0;
  return n * ((D + kGradCols - 1) / kGradCols);
}
int grad_chunk(int tokens) {
  tokens = std::max(g_opt.grad_tokens, (tokens + kGradStep - 1) / kGradStep * kGradStep);
  return std::min(tokens, kGradMaxTokens);           // the kernel stages at most that many row indices per unit
}
// Bounds for D columns; false: more units than a launch may have (refused before the tables are built).
bool grad_bounds(const Plan& pl, int D, GradBounds& bounds) {
  const int ncb = (D + kGradCols - 1) / kGradCols;
  auto chunk_of = [&](int live, double shrink) { return grad_chunk((int)(32 * kGradRanks * live * shrink)); };
  auto count = [&](double shrink) {
    GradBounds n;
    for (const JobDev& jb : pl.jobs) {
      if (jb.rank == 0 || jb.row1 == jb.row0) continue;
      for (int pb = 0; pb * kGradBlockRanks < jb.rpad; ++pb) {
        const int mb = grad_live_blocks(jb, pb), chunk = chunk_of(mb, shrink);
        const int64_t u = (int64_t)((jb.row1 - jb.row0 + chunk - 1) / chunk) * ncb;
        n.units += u;
        n.floats += u * mb * kGradRanks * kGradCols;
      }
    }
    return n;
  };
  double shrink = 1.0;
  while (shrink > 1.0 / 64 && count(shrink).units < kGradUnitsWanted) shrink *= 0.5;
  if (count(shrink).units > kMaxUnits) return false;
  // Grows with every job's tokens: what chunks of 1024 tokens per live block give, or, of each tile height at most what the
  // shortest chunks give, the tallest tiles first, 2046 units.  The chunks below are chosen within it (those of 4096 tokens always
  // are); the output tiles of idle jobs, which are zeros, come on top.
  const GradBounds whole = count(1.0);
  int64_t by_height[kGradMaxBlocks + 1] = {}, left = 2 * (kGradUnitsWanted - 1);
  for (const JobDev& jb : pl.jobs)
    for (int pb = 0; jb.rank > 0 && pb * kGradBlockRanks < jb.rpad; ++pb) {
      const int mb = grad_live_blocks(jb, pb), chunk = chunk_of(mb, 0.0);
      by_height[mb] += (int64_t)((jb.row1 - jb.row0 + chunk - 1) / chunk) * ncb;
    }
  for (int mb = kGradMaxBlocks; mb > 0; --mb) {
    const int64_t u = std::min(by_height[mb], left);
    bounds.units += u;  bounds.floats += u * mb * kGradRanks * kGradCols;  left -= u;
  }
  bounds.units = std::max(whole.units, bounds.units);
  bounds.floats = std::max(whole.floats, bounds.floats);
  return true;
}
// Chunks whose units take at most `limit` us: a step of 32 tokens takes 0.13 us and 0.155 for every live block.
double grad_step_us(int mb) { return 0.13 + 0.155 * mb; }
struct GradCost {
  double longest = 0.0, sum = 0.0, bytes = 0.0;
  int64_t units = 0, floats = 0;
};
int grad_chunk_of(int mb, double limit) { return grad_chunk((int)std::min<double>(kGradMaxTokens, kGradStep * limit / grad_step_us(mb))); }
GradCost grad_cost(const Plan& pl, int D, double limit) {
  GradCost g;
  const int ncb = (D + kGradCols - 1) / kGradCols;
  for (const JobDev& jb : pl.jobs) {
    const int T = jb.row1 - jb.row0;
    for (int pb = 0; jb.rank > 0 && pb * kGradBlockRanks < jb.rpad; ++pb) {
      const int mb = grad_live_blocks(jb, pb), chunk = grad_chunk_of(mb, limit), n = std::max(1, (T + chunk - 1) / chunk);
      const double step = grad_step_us(mb), fixed = 3.0 + mb;
      g.longest = std::max(g.longest, fixed + step * ((std::min(T, chunk) + kGradStep - 1) / kGradStep));
      g.sum += ncb * (n * fixed + step * ((T + kGradStep - 1) / kGradStep));
      g.bytes += (double)ncb * T * kGradCols * 2;
      if (T > 0) g.units += (int64_t)n * ncb;
      if (n > 1) g.floats += (int64_t)n * ncb * mb * kGradRanks * kGradCols;
    }
  }
  return g;
}
// The limit for one launch over the given widths: the cheapest of a few, by the longest unit, the units' sum over 256 CUs, the bytes
// of the activations at 5 TB/s, and for the partial tiles a launch of 5 us and their bytes, written and read, at 4 TB/s.  Negative:
// none whose partial tiles, room floats of them, have a place (for one width there always is one, see grad_bounds).
double grad_limit(const Plan& pl, const int* widths, const GradBounds* bounds, int n, int64_t room) {
  double best = -1.0, best_us = 0.0;
  for (double limit : {1e9, 96.0, 64.0, 48.0, 32.0, 24.0, 16.0, 12.0, 8.0, 6.0}) {
    double longest = 0.0, sum = 0.0, bytes = 0.0, extra = 0.0;
    int64_t floats = 0;
    bool fits = true;
    for (int i = 0; i < n; ++i) {
      const GradCost g = grad_cost(pl, widths[i], limit);
      fits = fits && g.units <= bounds[i].units;
      floats += g.floats;
      longest = std::max(longest, g.longest);  sum += g.sum;  bytes += g.bytes;
      if (g.floats > 0) extra += 5.0 + (double)g.floats * 8 / 4.0e6;
    }
    const double us = std::max({longest, sum / 256, bytes / 5.0e6}) + 0.5 * longest * (sum > 256 * longest) + extra;
    if (fits && floats <= room && (best < 0.0 || us < best_us)) { best = limit;  best_us = us; }
  }
  return best;
}
// idle_units: the output tiles of jobs without tokens are units, which store zeros; else groups of no partial tiles, which do too.
void build_grad_units(const Plan& pl, int D, double limit, bool idle_units, std::vector<GradUnit>& units,
                      std::vector<GradGroup>& groups, int64_t& partial_floats /* in: first free float, out: past the last */) {
  const int ncb = (D + kGradCols - 1) / kGradCols;
  for (int j = 0; j < pl.J; ++j) {
    const JobDev& jb = pl.jobs[j];
    if (jb.rank == 0) continue;
    const int Tj = jb.row1 - jb.row0;
    for (int pb = 0; pb * kGradBlockRanks < jb.rpad; ++pb) {
      const int mb = grad_live_blocks(jb, pb), chunk = grad_chunk_of(mb, limit);
      const int nchunks = std::max(1, (Tj + chunk - 1) / chunk);
      for (int cb = 0; cb < ncb; ++cb) {
        if (nchunks == 1 && (Tj > 0 || idle_units)) {
          units.push_back(GradUnit{j, jb.row0, jb.row1, cb, pb, mb, -1});
          continue;
        }
        GradGroup g{};
        g.job = j;  g.cb = cb;  g.pb = pb;  g.mb = mb;  g.nunits = Tj > 0 ? nchunks : 0;  g.part_off = partial_floats;
        if (Tj == 0) {
          groups.push_back(g);
          continue;
        }
        for (int c = 0; c < nchunks; ++c) {
          const int t0 = jb.row0 + c * chunk;
          units.push_back(GradUnit{j, t0, std::min(jb.row1, t0 + chunk), cb, pb, mb, partial_floats});
          partial_floats += (int64_t)mb * kGradRanks * kGradCols;
        }
        groups.push_back(g);
      }
    }
  }
  // longest first: the tail of the launch is made of the short units
  std::stable_sort(units.begin(), units.end(), [](const GradUnit& a, const GradUnit& b) {
    return (a.t1 - a.t0) * grad_step_us(a.mb) > (b.t1 - b.t0) * grad_step_us(b.mb);
  });
}

// Splits of a streaming shrink over K of a plan whose units have 32 rows: enough that units x splits fill the 512
// workgroup slots (80 KB of LDS each, two per CU), while a split keeps at least 4 K-steps of 64 (three are in flight
// before the first is multiplied).  Fewer if the fp32 sums (4 bytes per packed S element and split) would not fit.
constexpr int kGemmMaxSplits = 16;
constexpr int kShrinkSlots = 512, kShrinkMinSteps = 4, kShrinkMaxSplits = 32;
int shrink_splits(const Plan& pl, int K, size_t max_bytes) {
  if (pl.shrink_rows != 32 || g_opt.shrink_rows != 0 || K % 64 || pl.stream_units.empty()) return 1;
  int64_t s = std::min<int64_t>(kShrinkSlots / (int64_t)pl.stream_units.size(), K / 64 / kShrinkMinSteps);
  s = std::min<int64_t>({s, kShrinkMaxSplits, (int64_t)(max_bytes / (4 * (size_t)pl.s_elems))});
  return s < 2 ? 1 : (int)s;
}

// Microseconds of `units` workgroups of the GEMM, `steps` 32-wide K-steps each, 256 at a time: ~6.5 outside the K-loop, and
// per step 0.43 for one workgroup and 0.64 when all CUs run (16 tiles over K = 1024, 4096, 12288: 26, 69, 183 with the
// launch's ~5; 240 tiles: 33, 92, 253).
double gemm_us(int64_t units, int steps) {
  double us = 0.0;
  for (; units > 0; units -= 256) us += 6.5 + steps * (0.432 + 0.205 * (double)std::min<int64_t>(units, 256) / 256.0);
  return us;
}
// Which tiles of the GEMM over [T, K] x [K, N] to cut along K, and into how many shares.  256 tiles run at once, so those
// beyond the last multiple of 256 cost a whole contraction however few they are.  Cut, they cost their shares, and for the
// fp32 sums a launch (4 us) and a microsecond per 4.7 MB written, read and added (32 tiles over K = 4096: 69 us, in 5 shares
// 38; 64 over 12288: 189, in 4 shares 95).  After many rounds the workgroups are out of step and a tail hides among them,
// while the kernel that can cut is slower per tile (23 scalars in vector registers); over short contractions cuts then lose
// (2048 -> 2048, 30 rounds and 80 tiles: 1539 us, cut 1594; 4096 -> 4096, 24 and 128: 2270, 2299), over long ones they never do
// (17408 -> 5120, 30 and 80: 12461, 12083).  So rounds beyond the sixth are charged 5 us each, less with the length, nothing
// from 6144 on, and the cheapest number of shares is taken if that saves 2 us and 3 % of the uncut tail.  Over 581 sizes
// (K = 1024 ... 17408, 0 to 30 rounds, 12 to 240 tiles beyond them) that is 0.22 % from the best choice on average and slower
// than no cut at three, by at most 1.5 %; without the charge at thirteen, by up to 3.5 %; a charge of 2 us for every round loses
// nothing but leaves 0.49 %.
GemmSplit gemm_split(const Plan& pl, int K, int N, size_t max_bytes, int products = 1) {
  GemmSplit best;
  if (K % kGemmBK || pl.T == 0) return best;
  int kext = 0;
  for (const TileDev& td : pl.tile_jobs) kext = std::max(kext, td.kext);
  const int steps = (K + kext) / kGemmBK;
  const int64_t nb = products * (int64_t)pl.tile_jobs.size() * ((N + kGemmBN - 1) / kGemmBN);
  const int64_t n_tail = nb % 256;
  if (n_tail == 0) return best;
  const size_t tile_bytes = sizeof(float) * kGemmBN * (size_t)std::min(pl.T, kGemmBM);
  const double uncut = gemm_us(n_tail, steps);
  const double rounds = (double)std::max<int64_t>(0, nb / 256 - 6) * std::max(0.0, 5.0 * (1.0 - steps / 192.0));
  double best_gain = std::max(2.0, 0.03 * uncut);
  for (int s = 2; s <= kGemmMaxSplits && steps / s >= 4; ++s) {
    const int share = gemm_share(steps, s);
    if ((steps + share - 1) / share != s) continue;           // even shares of this size are fewer: tried under their number
    const size_t bytes = tile_bytes * (size_t)n_tail * s;
    if (bytes > max_bytes) break;
    const double gain = uncut - rounds - gemm_us(n_tail * s, share) - 4.0 - (double)bytes / 4.7e6;
    if (gain > best_gain) { best_gain = gain;  best.splits = s;  best.n_direct = (int32_t)(nb - n_tail); }
  }
  return best;
}
// Whether dX = dY.W^T of a batch runs against W as it lies instead of against a transposed copy.  Whole rounds of tiles are
// 2 to 9 % faster against the copy (its tiles are 64 rows of 512 contiguous bytes, those of W 256 rows of 128), but the copy
// reads and writes W once: forward and backward of 512 tokens, 4096 -> 12288, 215 us with the copy, 176 without; 17408 -> 5120,
// 256 tokens, 262 and 175.  They meet between 6000 tokens (gains of 0.9 to 3 % over nine pairs of feature sizes) and 8192 (0.8 %
// gained at 4096 -> 4096, 2.7 % lost at 17408 -> 5120).  A weight below 2^19 elements keeps the copy, a launch of 3 us: of
// 1024 x 1024 on, the smallest measured, leaving it out gains 2 to 4 us.  Same bits either way.
inline bool dx_direct(int64_t tokens, int64_t d_in, int64_t d_out) { return tokens <= 6144 && d_in * d_out >= (1 << 19); }
size_t gemm_split_bytes(const Plan& pl, const GemmSplit& g, int N, int products = 1) {
  if (g.splits < 2) return 0;
  const int64_t nb = products * (int64_t)pl.tile_jobs.size() * ((N + kGemmBN - 1) / kGemmBN);
  return sizeof(float) * kGemmBN * (size_t)std::min(pl.T, kGemmBM) * (size_t)(nb - g.n_direct) * g.splits;
}

// Bytes of the sums of a small batch and of its activations as fragments.
size_t small_part_bytes(const Plan& pl, int N, int splits) {
  return sizeof(float) * (size_t)pl.T * (size_t)small_ld(N, pl.r_total) * (size_t)splits;
}
size_t small_frag_bytes(const Plan& pl, int K) {
  const int rb = small_blocks(pl.T);
  return small_frags(rb) ? align_up((size_t)rb * 32 * (size_t)K, 256) : 0;
}
// Where the fragments of X (side 0) and dY (side 1) lie in the room of the sums: behind those of the two-launch form of either
// direction, and those of dY, which a backward writes with its first launch, also behind the sums of a general S = X.A if that
// backward may make S again first (frags_wait; where the room does not hold both, they are written after S).
size_t small_frag_at(const Plan& pl, int side) {
  const size_t shrink = pl.small_x || pl.shrink_splits_x < 2 ? 0 : sizeof(float) * (size_t)pl.s_elems * (size_t)pl.shrink_splits_x;
  const size_t sums = std::max({pl.small_x ? small_part_bytes(pl, pl.d_out, pl.small_x) : 0,
                                pl.small_dy ? small_part_bytes(pl, pl.d_in, pl.small_dy) : 0, pl.frags_wait ? shrink : 0});
  return align_up(sums, 256) + (side ? small_frag_bytes(pl, pl.d_in) : 0);
}
FragPack small_frag_pack(const Plan& pl, int side, const void* act, const int32_t* in_index, void* sums) {
  FragPack f;
  f.act = static_cast<const uint16_t*>(act);  f.in_index = in_index;
  f.T = pl.T;  f.K = side ? pl.d_out : pl.d_in;  f.rb = small_blocks(pl.T);
  if (small_frags(f.rb)) f.out = reinterpret_cast<uint16_t*>(static_cast<uint8_t*>(sums) + small_frag_at(pl, side));
  return f;
}
// Splits of the two-launch form of a small batch over [T, K] x [K, N] (0: the general kernels); kn: against a weight as the
// forward reads it.  A direction takes about 20 us, 0.115 us per MB of W and rank rows, and `piece` us per workgroup of the busiest
// CU and piece of 128 k-values of a wave, with 4 waves to a workgroup and 64 columns and a split each; the general kernels (cut
// shrink, sums, cut product, sums) about 29, or 32 in the backward, 0.26 us per MB and 2 us per 64 tokens.  Fitted to 608 launches of
// 16 to 128 tokens (K and N 1024 to 17408, 64 and 512 rank rows, 1 to 8 splits; 4 to 6 % off each, W from memory); the rule is
// 2 % off the best choice on average.  Measured, general / this, forward and backward without gradients: 4096 -> 4096, 64 tokens, 45 /
// 34 and 47 / 32 us; 4096 -> 12288, 16 tokens, 52 / 43 and 61 / 42; 1024 -> 1024, 128 tokens, 33 / 24; 17408 -> 5120, 128 tokens,
// 80 / 81 (general).  Each wave should have a piece (K >= 512), and idle jobs' rank rows, which are contracted too, must not be the bulk.
int small_splits(const Plan& pl, int K, int N, bool kn, size_t max_bytes) {
  if (pl.T < 1 || pl.T > kSmallRows || pl.d_in % 64 || pl.d_out % 64 || K < 512 || g_opt.shrink_rows != 0) return 0;
  int active = 0;
  for (const JobDev& jb : pl.jobs) active += jb.row1 > jb.row0 ? jb.rpad : 0;
  if (pl.r_total > 2 * active) return 0;
  const int steps = K / 64, tiles = N / 64 + (pl.r_total + 63) / 64, rb = small_blocks(pl.T);
  const size_t bytes = small_part_bytes(pl, N, 1), frags = 2 * small_frag_bytes(pl, std::max(pl.d_in, pl.d_out));
  const double piece = kn ? (rb == 1 ? 1.84 : rb == 2 ? 2.33 : rb == 4 ? 2.6 : 4.0) : (rb == 1 ? 1.04 : rb == 2 ? 1.47 : rb == 4 ? 1.8 : 2.97);
  int best = 0;
  double best_us = 0.95 * ((kn ? 9.0 : 11.0) + 0.144e-6 * 2 * (double)K * N + pl.T / 32.0);
  for (int s = 1; s <= kGemmMaxSplits && s <= steps && align_up(bytes * s, 256) + frags <= max_bytes; ++s) {
    const int pieces = ((steps + s - 1) / s + 7) / 8;
    const double us = piece * ((tiles * s + 255) / 256) * pieces + 0.15e-6 * (double)bytes * s;
    if (us < best_us) { best = s;  best_us = us; }
  }
  return best;
}

// Whether the forward of the full plan packs A_j side by side as well: for a dX product of the same batch against W as it lies.
bool packs_a_all(const Plan& pl) { return dx_direct(pl.T, pl.d_in, pl.d_out) && !pl.small_dy; }

// Room for the sums of cut launches in the full plan: two rounds of 256 whole tiles (128 MiB: 144 tiles over K = 15072 in
// three shares take 23 us off a dX of 400 tiles), or less for few tokens, whose workspace has to stay far from another dense
// matrix: 12 bytes per token and feature for the GEMMs (12 T (d_in + d_out) < 2 d_in d_out up to T = d / 12; it holds 61 tokens
// over 4096 -> 4096 at 6 shares, 22.8 us, where 14 would take about 17), and what the most shares of all shrink units take.
// It grows with the tokens of each job.
size_t sums_room(const Plan& pl) {
  const size_t gemm = 12 * (size_t)pl.T * (size_t)(pl.d_in + pl.d_out);
  const size_t shrink = sizeof(float) * (size_t)pl.s_elems * kShrinkMaxSplits;
  return std::min<size_t>(std::max(gemm, shrink), 2 * (size_t)TLORA_NOALLOC_SUM_BYTES);
}
// Room for the partial tiles of dA / dB and those sums, which use it in turn: what either gradient may leave alone.  One launch for
// both needs less than both bounds together nearly always (a job of one unit leaves none): while the room was their sum, workspaces
// grew by up to 70 % (one job of rank 512, 6812 tokens, 5120 -> 5120: 381 to 649 MB).
size_t grads_room(const Plan& pl, const GradBounds& gB, const GradBounds& gA) {
  return std::max(sums_room(pl), sizeof(float) * (size_t)std::max(gB.floats, gA.floats));
}
// Bytes of the forward-only plan's workspace (the self-check holds the layout to this sum).
size_t forward_bytes(const Plan& pl) {
  auto a = [](size_t bytes) { return align_up(bytes, 256); };
  return a(sizeof(JobDev) * pl.jobs.size()) + a(sizeof(TileDev) * pl.tile_jobs.size()) +
         a(sizeof(ShrinkUnit) * pl.shrink_units.size()) + a(sizeof(ShrinkUnit) * pl.stream_units.size()) + a(kClockBytes) +
         2 * a(2 * (size_t)pl.s_elems) + a(2 * (size_t)pl.sx_elems + 256) + a(2 * ((size_t)pl.atp_elems + 32 * (size_t)pl.d_in)) +
         (a(2 * (size_t)pl.d_in * (size_t)(pl.r_total + 32)) + a(2 * (size_t)pl.d_out * (size_t)(pl.r_total + 32)));
}
// The forward's part of that room, the same in both plans, so that both cut alike and a row of Y has the same bits through
// tlora_fwd and tlora_fwd_noalloc: what lies behind the static scratch where the scratch holds the problem.
size_t forward_sums_room(const Plan& pl) {
  return std::min<size_t>(sums_room(pl), forward_bytes(pl) <= TLORA_NOALLOC_SCRATCH_BYTES ? TLORA_NOALLOC_SUM_BYTES : SIZE_MAX);
}

// What the full plan reserves where a smaller batch can need more than a larger one (fewer, longer units; jobs that happen
// to share row tiles): upper bounds over every batch of the same jobs in which none has more tokens.  So a workspace that
// serves a batch serves every smaller one, as callers that keep one (and W^T inside it) for all their batches expect.
struct Reserve {
  size_t tables = 0;                                    // bytes of the table blob
  int64_t sx_elems = 0;
  size_t partial = 0;                                   // bytes of dA / dB partial tiles or sums of cut launches
};
Reserve reserve_of(const Plan& pl, const GradBounds& gB, const GradBounds& gA) {
  Reserve r;
  // a job's rows touch at most (T_j + 254) / 256 + 1 row tiles; one without tokens lies inside one at most
  for (const JobDev& jb : pl.jobs) r.sx_elems += (int64_t)jb.rpad * (jb.row1 == jb.row0 ? 1 : (jb.row1 - jb.row0 + 254) / kGemmBM + 1);
  r.sx_elems = kGemmBM * (r.sx_elems + (int64_t)pl.tile_jobs.size() * kGemmBK);
  const int rows = g_opt.shrink_rows != 0 ? pl.shrink_rows : pl.d_in % 64 == 0 && pl.d_out % 64 == 0 ? 32 : 64;
  int64_t stream = 0;
  for (const JobDev& jb : pl.jobs) stream += (int64_t)((jb.row1 - jb.row0 + rows - 1) / rows) * ((jb.rpad + 127) / 128);
  auto table = [&](size_t bytes) { r.tables += align_up(bytes, 256); };
  table(sizeof(JobDev) * pl.jobs.size());
  table(sizeof(TileDev) * pl.tile_jobs.size());
  table(sizeof(ShrinkUnit) * pl.shrink_units.size());
  table(sizeof(ShrinkUnit) * (size_t)stream);
  // (an output tile is units and a group, or one unit or a group if its job is idle)
  static_assert(sizeof(GradUnit) == sizeof(GradGroup), "they share a table's room");
  for (int d = 0; d < 2; ++d)
    table(sizeof(GradUnit) * (size_t)((d ? gA.units : gB.units) + grad_tiles(pl, d ? pl.d_in : pl.d_out)));
  r.partial = grads_room(pl, gB, gA);
  return r;
}

// fwd_only: tables and workspace of the forward alone (no transposed W, no dS, no dA / dB units or partial tiles)
int build_plan(const tlora_problem_t* p, Plan& pl, bool fwd_only = false) {
  const int rc = validate(p);
  if (rc != TLORA_OK) return rc;
  pl.J = p->num_jobs;  pl.T = (int)p->offsets[p->num_jobs];  pl.d_in = p->d_in;  pl.d_out = p->d_out;
  pl.dtype = p->dtype;
  pl.jobs.resize(pl.J);
  int64_t soff = 0, atp = 0;
  int64_t roff = 0;
  for (int j = 0; j < pl.J; ++j) {
    JobDev& jb = pl.jobs[j];
    memset(&jb, 0, sizeof(jb));
    jb.row0 = (int32_t)p->offsets[j];  jb.row1 = (int32_t)p->offsets[j + 1];
    jb.rank = p->ranks[j];
    jb.rpad = (jb.rank + kRankGranule - 1) / kRankGranule * kRankGranule;
    jb.scale = p->scales[j];
    jb.soff = soff;  jb.atp_off = atp;  jb.roff = (int32_t)roff;
    // rows of the packed intermediates are padded (with zeros) to the dA / dB kernel's token step
    soff += (int64_t)((jb.row1 - jb.row0 + kGradStep - 1) / kGradStep * kGradStep) * jb.rpad;
    atp += (int64_t)jb.rpad * pl.d_in;
    roff += jb.rpad;
    pl.max_rpad = std::max(pl.max_rpad, jb.rpad);
  }
  if (roff > (int64_t)1 << 22) return TLORA_EINVAL;   // rows of the stacked adapter operands: 256 of them span 32-bit byte offsets
  pl.s_elems = soff;  pl.atp_elems = atp;  pl.r_total = (int)roff;

  // row tiles of the backbone GEMM (nano-batches of the concatenated batch, Sec. 3.3)
  const int tiles_m = (pl.T + kGemmBM - 1) / kGemmBM;
  pl.tile_jobs.resize(tiles_m);
  {
    int j = 0;
    for (int tm = 0; tm < tiles_m; ++tm) {
      const int r0 = tm * kGemmBM, r1 = std::min(pl.T, r0 + kGemmBM);
      while (pl.jobs[j].row1 <= r0) ++j;             // first job with a row at or after r0
      int last = j;
      for (int k = j; k < pl.J && pl.jobs[k].row0 < r1; ++k)
        if (pl.jobs[k].row1 > pl.jobs[k].row0) last = k;
      TileDev& td = pl.tile_jobs[tm];
      td.first = j;  td.last = last;
      // adapter K-extension of the tile: padded ranks of jobs first..last, rounded up to the K-step
      td.roff_first = pl.jobs[j].roff;
      const int span = pl.jobs[last].roff + pl.jobs[last].rpad - td.roff_first;
      td.kext = (span + kGemmBK - 1) / kGemmBK * kGemmBK;
      td.aoff = pl.sx_elems;
      pl.sx_elems += (int64_t)kGemmBM * td.kext;
    }
  }
  GradBounds gB, gA;
  if (pl.dtype == TLORA_BF16) {
    // Rows per unit of the streaming shrink: 128 when that still gives enough workgroups for the 256 CUs, else 64, else
    // 32 (a small batch would otherwise stream its activations through a few dozen CUs).  The 32-row kernel exists for
    // K-steps of 64 only, and the units serve both the forward (K = d_in) and the backward (K = d_out) shrink.
    {
      auto count = [&](int rows) {
        int64_t n = 0;
        for (const JobDev& jb : pl.jobs)
          if (jb.rpad > 0) n += (int64_t)((jb.row1 - jb.row0 + rows - 1) / rows) * ((jb.rpad + 127) / 128);
        return n;
      };
      int64_t generic = 0;                           // units of the generic kernel: 64 rows x 64 rank columns
      for (const JobDev& jb : pl.jobs)
        generic += (int64_t)((jb.row1 - jb.row0 + 63) / 64) * ((jb.rpad + kShrinkCols - 1) / kShrinkCols);
      if (generic > kMaxUnits || count(32) > kMaxUnits) return TLORA_EINVAL;
      const bool can32 = pl.d_in % 64 == 0 && pl.d_out % 64 == 0;
      if (g_opt.shrink_rows != 0) pl.shrink_rows = (g_opt.shrink_rows == 32 && !can32) ? 64 : g_opt.shrink_rows;
      else pl.shrink_rows = count(128) >= 192 ? 128 : (count(64) >= 192 || !can32) ? 64 : 32;
    }
    for (int j = 0; j < pl.J; ++j) {
      const JobDev& jb = pl.jobs[j];
      if (jb.rpad == 0) continue;
      const int npb = (jb.rpad + kShrinkCols - 1) / kShrinkCols;
      for (int t0 = jb.row0; t0 < jb.row1; t0 += 64)
        for (int pb = 0; pb < npb; ++pb) {
          ShrinkUnit u;
          u.job = j;  u.t0 = t0;  u.nrows = std::min(64, jb.row1 - t0);  u.pb = pb;
          pl.shrink_units.push_back(u);
        }
      const int npb2 = (jb.rpad + 127) / 128;
      for (int t0 = jb.row0; t0 < jb.row1; t0 += pl.shrink_rows)
        for (int pb = 0; pb < npb2; ++pb) {
          ShrinkUnit u;
          u.job = j;  u.t0 = t0;  u.nrows = std::min(pl.shrink_rows, jb.row1 - t0);  u.pb = pb;
          pl.stream_units.push_back(u);
        }
    }
    if (!fwd_only) {
      if (!grad_bounds(pl, pl.d_out, gB) || !grad_bounds(pl, pl.d_in, gA)) return TLORA_EINVAL;
      // One launch for both from 32 output tiles on, with fewer either way is a few workgroups; and if the partial tiles of both have
      // room at a time.  Where they have not, either has rounds of units of its own and two launches take as long (backward of 20000
      // and 24000 tokens at ranks 512 and 1024, 4096 -> 12288: one 6.80 ms, two 6.84; 25000 at rank 1024, 5120 -> 17408: 7.00, 6.98).
      // A launch has at most kMaxUnits units (2^31 threads): with more, which takes tens of thousands of jobs, the idle ones go with
      // the reduction and each side has a launch of its own.
      const int64_t tiles = grad_tiles(pl, pl.d_out) + grad_tiles(pl, pl.d_in);
      const bool one_launch_holds = gB.units + gA.units + tiles <= kMaxUnits;
      pl.grads_merged = tiles >= 32 && one_launch_holds;
      const int widths[2] = {pl.d_out, pl.d_in};
      const GradBounds bounds[2] = {gB, gA};
      const int64_t room = (int64_t)(grads_room(pl, gB, gA) / sizeof(float));
      double limit[2] = {-1.0, -1.0};
      if (pl.grads_merged) limit[0] = limit[1] = grad_limit(pl, widths, bounds, 2, room);
      pl.grads_merged = limit[0] >= 0.0;
      int64_t used[2] = {};
      for (int d = 0; d < 2; ++d) {
        if (!pl.grads_merged) limit[d] = grad_limit(pl, widths + d, bounds + d, 1, room);
        else if (d) used[1] = used[0];
        build_grad_units(pl, widths[d], limit[d], one_launch_holds, d ? pl.gradA_units : pl.gradB_units,
                         d ? pl.gradA_groups : pl.gradB_groups, used[d]);
      }
      pl.grad_partial = std::max(used[0], used[1]);
    }
  }

  // table blob
  size_t o = 0;
  auto place = [&](size_t bytes) { const size_t at = o;  o = align_up(o + bytes, 256);  return at; };
  pl.tb_jobs = place(sizeof(JobDev) * pl.jobs.size());
  pl.tb_tiles = place(sizeof(TileDev) * pl.tile_jobs.size());
  pl.tb_shrink = place(sizeof(ShrinkUnit) * pl.shrink_units.size());
  pl.tb_stream = place(sizeof(ShrinkUnit) * pl.stream_units.size());
  for (int d = 0; d < 2; ++d) {                         // the groups right behind the units
    const size_t units = sizeof(GradUnit) * (d ? pl.gradA_units : pl.gradB_units).size();
    const size_t groups = sizeof(GradGroup) * (d ? pl.gradA_groups : pl.gradB_groups).size();
    size_t& at = d ? pl.tb_gAu : pl.tb_gBu;
    at = place(units + groups);
    (d ? pl.tb_gAg : pl.tb_gBg) = at + units;
  }
  if (pl.dtype == TLORA_F32) {
    // the fp32 path needs at most 3 J + 1 products per launch, two launches per pass
    const size_t max_units = 2 * (size_t)(3 * pl.J + 1);
    size_t max_tiles = 0;
    auto tiles_of = [](int64_t m, int64_t n) { return (size_t)(((m + 63) / 64) * ((n + 63) / 64)); };
    max_tiles += 2 * tiles_of(pl.T, std::max(pl.d_in, pl.d_out));
    for (int j = 0; j < pl.J; ++j) {
      const JobDev& jb = pl.jobs[j];
      const int Tj = jb.row1 - jb.row0;
      max_tiles += 2 * tiles_of(Tj, jb.rank) + tiles_of(Tj, std::max(pl.d_in, pl.d_out)) +
                   tiles_of(pl.d_in, jb.rank) + tiles_of(jb.rank, pl.d_out);
    }
    pl.f32_reserved = align_up(sizeof(F32Unit) * max_units, 256) + align_up(sizeof(F32Tile) * max_tiles, 256) + 4 * 256;
    pl.tb_f32 = place(pl.f32_reserved);
  }
  pl.tables_bytes = o;

  // workspace layout
  const bool full = pl.dtype == TLORA_BF16 && !fwd_only;
  const Reserve res = full ? reserve_of(pl, gB, gA) : Reserve();
  size_t w = 0;
  auto wplace = [&](size_t bytes) { const size_t at = w;  w = align_up(w + bytes, 256);  return at; };
  // the transposed W first, then its state: their place depends on nothing but d_in x d_out, so a copy made by one call is found
  // by later calls on other token batches (nano-batches) that share the workspace
  if (full) {
    pl.off_wt = wplace(2 * (size_t)pl.d_in * (size_t)pl.d_out);
    pl.off_clock = wplace(kClockBytes + sizeof(WtState));
    pl.off_wt_state = pl.off_clock + kClockBytes;       // (in the rest of the clock's 256 bytes)
  }
  // so do the packed adapters, whose places depend on the feature sizes and ranks
  if (pl.dtype == TLORA_BF16) {
    pl.off_atp = wplace(2 * ((size_t)pl.atp_elems + 32 * (size_t)pl.d_in));
    pl.off_bp = wplace(2 * (size_t)pl.d_out * (size_t)(pl.r_total + 32));
    pl.off_ap = wplace(2 * (size_t)pl.d_in * (size_t)(pl.r_total + 32));
  }
  pl.off_tables = wplace(full ? res.tables : pl.tables_bytes);
  if (!full) pl.off_clock = wplace(kClockBytes);
  if (pl.dtype == TLORA_F32) {
    pl.off_S = wplace(sizeof(float) * (size_t)pl.s_elems);
    if (!fwd_only) pl.off_dS = wplace(sizeof(float) * (size_t)pl.s_elems);
  }
  if (pl.dtype == TLORA_BF16) {
    pl.off_Shi = wplace(2 * (size_t)pl.s_elems);
    pl.off_Slo = wplace(2 * (size_t)pl.s_elems);
    if (!fwd_only) {
      pl.off_dShi = wplace(2 * (size_t)pl.s_elems);
      pl.off_dSlo = wplace(2 * (size_t)pl.s_elems);
    }
    // + 256: a 64-wide K-step over a last 32-wide slice reads (and ignores) 64 bytes past each operand row
    pl.off_Sx = wplace(2 * (size_t)(full ? res.sx_elems : pl.sx_elems) + 256);
    if (!fwd_only) pl.off_dSx = wplace(2 * (size_t)res.sx_elems + 256);
    // Sums of cut launches: in the full plan in the block of the dA / dB partial tiles (the launches follow one another); in
    // the forward-only plan behind the static scratch, so that a cut never makes a problem too large for it.  While they
    // had what the scratch itself left (2 to 14 MiB), 128 tiles over K = 12288 (1900 tokens, 4096 features) ran uncut:
    // 269 us against 176 for two halves and their sum.
    const size_t room = forward_sums_room(pl);
    pl.shrink_splits_x = shrink_splits(pl, pl.d_in, room);
    pl.gemm_split_fwd = gemm_split(pl, pl.d_in, pl.d_out, room);
    pl.small_x = small_splits(pl, pl.d_in, pl.d_out, true, room);
    if (fwd_only) {
      pl.partial_bytes = room;                           // (more than there is only in a plan that does not fit)
      pl.off_partial = TLORA_NOALLOC_SCRATCH_BYTES;      // (beyond pl.total)
    } else {
      pl.shrink_splits_dy = shrink_splits(pl, pl.d_out, sums_room(pl));
      pl.gemm_split_bwd = gemm_split(pl, pl.d_out, pl.d_in, sums_room(pl));
      pl.pair_split_fwd = gemm_split(pl, pl.d_in, pl.d_out, sums_room(pl), 2);
      pl.pair_split_bwd = gemm_split(pl, pl.d_out, pl.d_in, sums_room(pl), 2);
      pl.small_dy = small_splits(pl, pl.d_out, pl.d_in, false, sums_room(pl));
      pl.partial_bytes = res.partial;
      pl.frags_wait = true;
      pl.frags_wait = small_frag_at(pl, 1) + small_frag_bytes(pl, pl.d_out) <= pl.partial_bytes;
      pl.off_partial = wplace(pl.partial_bytes);
    }
  }
  pl.total = std::max<size_t>(w, 256);
  return TLORA_OK;
}

// ---- pinned staging for the table upload ----------------------------------------------------------------
// A small ring of pinned host buffers; a slot is reused only after the copy that read it has finished.
struct Slot {
  void* host = nullptr;
  void* dev_view = nullptr;   // the same buffer as the device addresses it (null: not mapped, copy commands are used)
  size_t cap = 0;
  hipEvent_t ev = nullptr;
  bool busy = false;
};
constexpr int kSlots = 16;
Slot g_slots[kSlots];
int g_next_slot = 0;

int upload_tables(const std::vector<uint8_t>& blob, void* dst, hipStream_t st, const WtCall& wt = WtCall(),
                  const FragPack& frags = FragPack()) {
  Slot& s = g_slots[g_next_slot];
  g_next_slot = (g_next_slot + 1) % kSlots;
  if (s.busy) {
    TLORA_HIP(hipEventSynchronize(s.ev));
    s.busy = false;
  }
  if (s.cap < blob.size()) {
    if (s.host) (void)hipHostFree(s.host);
    s.host = nullptr;  s.dev_view = nullptr;  s.cap = 0;
    const size_t cap = align_up(blob.size() * 2, 4096);
    TLORA_HIP(hipHostMalloc(&s.host, cap, hipHostMallocDefault));
    s.cap = cap;
    if (hipHostGetDevicePointer(&s.dev_view, s.host, 0) != hipSuccess) {
      s.dev_view = nullptr;
      (void)hipGetLastError();
    }
  }
  if (!s.ev) TLORA_HIP(hipEventCreateWithFlags(&s.ev, hipEventDisableTiming));
  memcpy(s.host, blob.data(), blob.size());
  if (g_opt.table_copy_kernel && s.dev_view && blob.size() % 16 == 0 && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
    launch_table_copy(s.dev_view, dst, blob.size(), wt, frags, st);
    TLORA_HIP(hipGetLastError());
  } else {
    TLORA_HIP(hipMemcpyAsync(dst, s.host, blob.size(), hipMemcpyHostToDevice, st));
    launch_table_copy(nullptr, nullptr, 0, wt, frags, st);
    TLORA_HIP(hipGetLastError());
  }
  TLORA_HIP(hipEventRecord(s.ev, st));
  s.busy = true;
  return TLORA_OK;
}

// ---- optional per-kernel event timing ---------------------------------------------------------------------
struct Pending {
  int cls;
  hipEvent_t a, b;
};
bool g_prof_on = false;
bool g_prof_gemm_only = false;   // mode 2: only the two segmented-GEMM classes are bracketed
std::vector<Pending> g_pending;
std::vector<hipEvent_t> g_event_pool;
double g_prof_ms[TLORA_K_COUNT] = {};
unsigned long long* g_clock_slot[2] = {nullptr, nullptr};   // device slots of the last profiled fwd / dX GEMM
int64_t g_prof_n[TLORA_K_COUNT] = {};

hipEvent_t prof_event() {
  if (!g_event_pool.empty()) {
    hipEvent_t e = g_event_pool.back();
    g_event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Brackets one launch with events when profiling is on.
struct Timed {
  hipStream_t st;
  Pending p{};
  bool on;
  Timed(int cls, hipStream_t s, bool enable = true)
      : st(s), on(g_prof_on && enable && (!g_prof_gemm_only || cls == TLORA_K_GEMM_FWD || cls == TLORA_K_GEMM_BWD)) {
    if (!on) return;
    p.cls = cls;  p.a = prof_event();  p.b = prof_event();
    if (!p.a || !p.b) { on = false; return; }
    (void)hipEventRecord(p.a, st);
  }
  ~Timed() {
    if (!on) return;
    (void)hipEventRecord(p.b, st);
    g_pending.push_back(p);
  }
};

int prof_drain() {
  for (const Pending& p : g_pending) {
    TLORA_HIP(hipEventSynchronize(p.b));
    float ms = 0.f;
    TLORA_HIP(hipEventElapsedTime(&ms, p.a, p.b));
    g_prof_ms[p.cls] += ms;
    g_prof_n[p.cls] += 1;
    g_event_pool.push_back(p.a);
    g_event_pool.push_back(p.b);
  }
  g_pending.clear();
  return TLORA_OK;
}

// Two projections of a block over the same rows and sizes (gate and up, k and v).  Together they fill the rounds of 256 tiles that
// either would leave partly empty or cut: forward and backward of an MLP block, apart / in pairs, 271 / 228 us at 300 tokens and
// 1024 -> 2816, 1267 / 1188 at 1900 and 4096 -> 12288, 6450 / 6400 at 12000 (9 rounds each).  Over many rounds there is nothing
// left to fill, while two weights share the caches: 12590 / 12610 at 24000 (17 rounds), 63430 / 63800 for a decoder layer of 83968
// (61).  So pairs are for products of up to 12 rounds.
constexpr int64_t kPairTiles = 12 * 256;
// A backbone product that is ready to run.
struct GemmCall {
  int kernel = 0;                                       // what it is timed as
  bool w_is_kn = false, timed = true;
  const TileDev* tiles = nullptr;
  GemmOperands op;                                      // (out null: nothing to run)
  int r_total = 0, T = 0, K = 0, N = 0;
  const int32_t *out_index = nullptr, *in_index = nullptr;
  unsigned long long* clk = nullptr;
  GemmSplit split, pair_split;
  float* sums = nullptr;
  bool pairs() const {
    const int64_t tiles = (int64_t)((T + kGemmBM - 1) / kGemmBM) * ((N + kGemmBN - 1) / kGemmBN);
    return K % kGemmBK == 0 && !out_index && !in_index && tiles <= kPairTiles;
  }
};
// second: another one over the same jobs, in the same launch; their sums have one place.
// A profiled one is counted, the pair as a whole, into the clock slot of the first.
void launch_gemm(const GemmCall& g, const GemmCall* second, hipStream_t st) {
  if (g.clk) {
    launch_zero_fill(g.clk, 16, st);
    g_clock_slot[g.kernel == TLORA_K_GEMM_FWD ? 0 : 1] = g.clk;
  }
  Timed t(g.kernel, st, g.timed);
  launch_seg_gemm(g.w_is_kn, g.tiles, g.op.act, g.op.W, g.op.Sx, g.op.packed, g.r_total, g.op.out, g.out_index, g.in_index, g.T,
                  g.K, g.N, g.clk, second ? g.pair_split : g.split, g.sums, second ? second->op : GemmOperands(), st);
}
void launch_gemm_pair(const GemmCall& a, const GemmCall& b, hipStream_t st) {
  if (a.op.out && b.op.out && a.w_is_kn == b.w_is_kn && a.K == b.K && a.N == b.N && a.T == b.T && a.r_total == b.r_total &&
      a.sums == b.sums) {
    launch_gemm(a, &b, st);
    return;
  }
  if (a.op.out) launch_gemm(a, nullptr, st);
  if (b.op.out) launch_gemm(b, nullptr, st);
}

// S_j = X_j.A_j (or dS_j = dY_j.B_j^T): streaming kernel when the contraction length allows, else generic
void run_shrink(const Plan& pl, const uint8_t* tb, const JobDev* jobs, const TileDev* tiles, const uint16_t* act, int K,
                const uint16_t* packed, bool packed_is_atp, uint16_t* hi, uint16_t* lo, uint16_t* Sx,
                const int32_t* row_index, float* part, hipStream_t st) {
  const int splits = packed_is_atp ? pl.shrink_splits_x : pl.shrink_splits_dy;
  if (splits > 1) {
    launch_shrink_split(jobs, tiles, reinterpret_cast<const ShrinkUnit*>(tb + pl.tb_stream), (int)pl.stream_units.size(),
                        splits, pl.T, act, K, packed, packed_is_atp, hi, lo, Sx, row_index, part, pl.s_elems, st);
    return;
  }
  launch_zero_fill(Sx, 2 * (size_t)pl.sx_elems, st);
  if (K % 32 == 0)
    launch_shrink_stream(jobs, tiles, reinterpret_cast<const ShrinkUnit*>(tb + pl.tb_stream),
                         (int)pl.stream_units.size(), pl.shrink_rows, g_opt.shrink_stages, act, K, packed, packed_is_atp,
                         hi, lo, Sx, row_index, st);
  else
    launch_shrink(jobs, tiles, reinterpret_cast<const ShrinkUnit*>(tb + pl.tb_shrink), (int)pl.shrink_units.size(), 64,
                  act, K, packed, packed_is_atp, hi, lo, Sx, row_index, st);
}

int check_arch() {
  static int cached = 1;   // 1 = unknown
  if (cached != 1) return cached;
  int dev = 0;
  TLORA_HIP(hipGetDevice(&dev));
  hipDeviceProp_t prop;
  TLORA_HIP(hipGetDeviceProperties(&prop, dev));
  cached = strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? TLORA_OK : TLORA_EARCH;
  return cached;
}

inline bool misaligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) != 0; }

template <class T>
void put(std::vector<uint8_t>& blob, size_t at, const std::vector<T>& v) {
  if (!v.empty()) memcpy(blob.data() + at, v.data(), sizeof(T) * v.size());
}

std::vector<uint8_t> make_blob(const Plan& pl) {
  std::vector<uint8_t> blob(pl.tables_bytes, 0);
  put(blob, pl.tb_jobs, pl.jobs);
  put(blob, pl.tb_tiles, pl.tile_jobs);
  put(blob, pl.tb_shrink, pl.shrink_units);
  put(blob, pl.tb_stream, pl.stream_units);
  put(blob, pl.tb_gBu, pl.gradB_units);
  put(blob, pl.tb_gBg, pl.gradB_groups);
  put(blob, pl.tb_gAu, pl.gradA_units);
  put(blob, pl.tb_gAg, pl.gradA_groups);
  return blob;
}

// ---- plan cache ---------------------------------------------------------------------------------------------
// A plan depends only on (dtype, d_in, d_out, ranks, offsets), the forward-only flag and the tiling options; the
// per-call values (scales, adapter and gradient pointers) live in the job table alone, which every call patches into
// its copy of the cached table blob.  Training loops call with the same few problems step after step, so building
// the plan (vectors, unit sorting) and assembling the blob are paid once per distinct problem.  Entries are kept in
// most-recently-used order; everything here runs under g_mu.
struct PlanEntry {
  std::vector<int64_t> key;
  Plan pl;
  std::vector<uint8_t> blob;     // tables with a job table whose per-call fields are zero
};
constexpr size_t kPlanCacheEntries = 128;
std::list<PlanEntry> g_plans;
PlanEntry g_plan_uncached;       // the plan of the current call when the cache is switched off

void plan_key(const tlora_problem_t* p, bool fwd_only, std::vector<int64_t>& key) {
  key.clear();
  key.reserve(10 + 2 * (size_t)p->num_jobs);
  key.push_back(p->dtype);  key.push_back(p->num_jobs);  key.push_back(p->d_in);  key.push_back(p->d_out);
  key.push_back(fwd_only ? 1 : 0);
  key.push_back(g_opt.shrink_rows);  key.push_back(g_opt.grad_tokens);
  for (int j = 0; j < p->num_jobs; ++j) key.push_back(p->ranks[j]);
  for (int j = 0; j <= p->num_jobs; ++j) key.push_back(p->offsets[j]);
}

// The plan of a problem: from the cache, or built and inserted.
int get_plan(const tlora_problem_t* p, bool fwd_only, const PlanEntry** out) {
  const int rc = validate(p);
  if (rc != TLORA_OK) return rc;
  if (!g_opt.plan_cache) {
    g_plan_uncached = PlanEntry();
    const int rb = build_plan(p, g_plan_uncached.pl, fwd_only);
    if (rb != TLORA_OK) return rb;
    g_plan_uncached.blob = make_blob(g_plan_uncached.pl);
    *out = &g_plan_uncached;
    return TLORA_OK;
  }
  static std::vector<int64_t> key;
  plan_key(p, fwd_only, key);
  for (auto it = g_plans.begin(); it != g_plans.end(); ++it)
    if (it->key == key) {
      if (it != g_plans.begin()) g_plans.splice(g_plans.begin(), g_plans, it);
      *out = &g_plans.front();
      return TLORA_OK;
    }
  PlanEntry e;
  const int rb = build_plan(p, e.pl, fwd_only);
  if (rb != TLORA_OK) return rb;
  e.key = key;
  e.blob = make_blob(e.pl);
  g_plans.push_front(std::move(e));
  if (g_plans.size() > kPlanCacheEntries) g_plans.pop_back();
  *out = &g_plans.front();
  return TLORA_OK;
}

// fp32 path: append the tiles of one product
void f32_add(std::vector<F32Unit>& units, std::vector<F32Tile>& tiles, const F32Unit& u) {
  if (u.M <= 0 || u.N <= 0) return;
  const int id = (int)units.size();
  units.push_back(u);
  for (int tm = 0; tm < (u.M + 63) / 64; ++tm)
    for (int tn = 0; tn < (u.N + 63) / 64; ++tn) tiles.push_back(F32Tile{id, tm, tn, 0});
}
F32Unit f32_unit(const float* A, int64_t a_rs, int64_t a_cs, const float* B, int64_t b_rs, int64_t b_cs, float* C,
                 int64_t c_rs, int M, int N, int K, float alpha, bool accumulate) {
  F32Unit u{};
  u.A = A;  u.B = B;  u.C = C;  u.M = M;  u.N = N;  u.K = K;  u.accumulate = accumulate ? 1 : 0;
  u.a_rs = a_rs;  u.a_cs = a_cs;  u.b_rs = b_rs;  u.b_cs = b_cs;  u.c_rs = c_rs;  u.alpha = alpha;
  return u;
}

// Write the two launches' unit/tile tables into the blob's fp32 area and return their device addresses.
struct F32Launch {
  size_t units_at[2], tiles_at[2];
  int ntiles[2];
  size_t end;               // the blob is used up to here
};
int f32_place(const Plan& pl, std::vector<uint8_t>& blob, std::vector<F32Unit> units[2], std::vector<F32Tile> tiles[2],
              F32Launch& L) {
  size_t o = pl.tb_f32;
  for (int i = 0; i < 2; ++i) {
    // tile indices are per launch: rebase nothing, each launch has its own unit array
    L.units_at[i] = o;
    o = align_up(o + sizeof(F32Unit) * units[i].size(), 256);
    L.tiles_at[i] = o;
    o = align_up(o + sizeof(F32Tile) * tiles[i].size(), 256);
    L.ntiles[i] = (int)tiles[i].size();
  }
  if (o > pl.tb_f32 + pl.f32_reserved) return TLORA_EWORKSPACE;
  L.end = o;
  for (int i = 0; i < 2; ++i) {
    put(blob, L.units_at[i], units[i]);
    put(blob, L.tiles_at[i], tiles[i]);
  }
  return TLORA_OK;
}

// static_scratch: the "workspace" is the library's static scratch array and only the forward will run.
// shared_sums: the workspace ends where the sums begin (a block's projections have one place for them).
// Gives the (cached) plan and this call's job table: the plan's with the caller's scales and adapter pointers.
int common_checks(const tlora_problem_t* p, const PlanEntry** entry, std::vector<JobDev>& hjobs, void* ws, size_t ws_bytes,
                  bool static_scratch = false, bool shared_sums = false) {
  int rc = get_plan(p, static_scratch, entry);
  if (rc != TLORA_OK) return rc;
  const Plan& pl = (*entry)->pl;
  if ((pl.T > 0 && !p->X) || !p->W || !p->A || !p->B) return TLORA_ENULL;
  for (int j = 0; j < pl.J; ++j)
    if (pl.jobs[j].rank > 0 && (!p->A[j] || !p->B[j])) return TLORA_ENULL;
  if (misaligned16(p->X) || misaligned16(p->W)) return TLORA_EALIGN;
  if (static_scratch && ws_bytes < pl.total) return TLORA_ESCRATCH;
  const size_t need = shared_sums ? pl.off_partial : pl.total;
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) || ws_bytes < need) return TLORA_EWORKSPACE;
  hjobs = pl.jobs;
  for (int j = 0; j < pl.J; ++j) {
    hjobs[j].scale = p->scales[j];
    hjobs[j].A = p->A[j];
    hjobs[j].B = p->B[j];
  }
  return TLORA_OK;
}

}  // namespace
}  // namespace tlora

using namespace tlora;

extern "C" {

size_t tlora_workspace_bytes(const tlora_problem_t* p) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  const PlanEntry* e = nullptr;
  if (get_plan(p, false, &e) != TLORA_OK) return 0;
  return e->pl.total;
}

}  // extern "C"

namespace tlora {
namespace {
// The forward's launch sequence.  no_alloc: the workspace is the static device scratch (`workspace` = its address on
// the current device, `ws_bytes` = its size); the plan and the workspace layout are the forward's alone, the tables
// reach the device as kernel arguments (no staging buffer, no copy node), and nothing is timed: no HIP object is
// created and no memory of any kind is allocated on this path.
// Token-indexed calls (bf16): out_index = the batch row of every token row of the job-sorted order -- the GEMM scatters
// its output rows there; in_index = the same list when X is the batch in its own order, fetched through the list
// inside the kernels' loads (null: X already lies in job-sorted order).
// packed: this workspace already holds the packed copies of the same adapters (a nano-batch after the first).
// shared_sums: where the sums of cut launches go instead of the workspace's own last part.
// later: where given, a product that a pair may take is written down there instead of launched.
int fwd_impl(const tlora_problem_t* p, void* Y, void* workspace, size_t ws_bytes, void* hip_stream, bool no_alloc,
             const int32_t* out_index = nullptr, const int32_t* in_index = nullptr, bool packed = false,
             uint8_t* shared_sums = nullptr, GemmCall* later = nullptr) {
  const PlanEntry* entry = nullptr;
  std::vector<JobDev> hjobs;
  int rc = common_checks(p, &entry, hjobs, workspace, ws_bytes, no_alloc, shared_sums != nullptr);
  if (rc != TLORA_OK) return rc;
  const Plan& pl = entry->pl;
  if (pl.T > 0 && !Y) return TLORA_ENULL;
  if (misaligned16(Y)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK) return rc;
  if (pl.T == 0) return TLORA_OK;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  uint8_t* tb = ws + pl.off_tables;
  std::vector<uint8_t> blob = entry->blob;          // the cached tables, with this call's job table
  put(blob, pl.tb_jobs, hjobs);
  const JobDev* jobs = reinterpret_cast<const JobDev*>(tb + pl.tb_jobs);
  const bool timed = g_prof_on && !no_alloc;
  auto upload = [&](size_t used) {
    if (!no_alloc) return upload_tables(blob, tb, st);
    if (used > kNoAllocMaxTableBytes) return (int)TLORA_ESCRATCH;
    launch_table_write(blob.data(), used, tb, st);
    return (int)TLORA_OK;
  };

  if (pl.dtype == TLORA_F32) {
    float* S = reinterpret_cast<float*>(ws + pl.off_S);
    const float* X = static_cast<const float*>(p->X);
    const float* W = static_cast<const float*>(p->W);
    float* Yf = static_cast<float*>(Y);
    std::vector<F32Unit> units[2];
    std::vector<F32Tile> tiles[2];
    f32_add(units[0], tiles[0], f32_unit(X, pl.d_in, 1, W, pl.d_out, 1, Yf, pl.d_out, pl.T, pl.d_out, pl.d_in, 1.f, false));
    for (int j = 0; j < pl.J; ++j) {
      const JobDev& jb = hjobs[j];
      const int Tj = jb.row1 - jb.row0;
      if (jb.rank == 0 || Tj == 0) continue;
      const float* Xj = X + (int64_t)jb.row0 * pl.d_in;
      float* Sj = S + jb.soff;
      f32_add(units[0], tiles[0], f32_unit(Xj, pl.d_in, 1, static_cast<const float*>(jb.A), jb.rank, 1, Sj, jb.rpad,
                                           Tj, jb.rank, pl.d_in, 1.f, false));
      f32_add(units[1], tiles[1], f32_unit(Sj, jb.rpad, 1, static_cast<const float*>(jb.B), pl.d_out, 1,
                                           Yf + (int64_t)jb.row0 * pl.d_out, pl.d_out, Tj, pl.d_out, jb.rank, jb.scale,
                                           true));
    }
    F32Launch L;
    rc = f32_place(pl, blob, units, tiles, L);
    if (rc != TLORA_OK) return rc;
    rc = upload(L.end);
    if (rc != TLORA_OK) return rc;
    for (int i = 0; i < 2; ++i) {
      Timed t(TLORA_K_F32, st, timed);
      launch_f32_units(reinterpret_cast<const F32Unit*>(tb + L.units_at[i]),
                       reinterpret_cast<const F32Tile*>(tb + L.tiles_at[i]), L.ntiles[i], st);
    }
    return launches_ok(__LINE__);
  }

  // The forward's tables lie in front of the backward's.  They go with the packing's launch where they fit and it has work.
  const bool with_pack = !packed && pl.max_rpad > 0 && pl.tb_gBu <= kPackArgBytes && pl.tb_jobs == 0;
  if (no_alloc && pl.tables_bytes > kNoAllocMaxTableBytes) return TLORA_ESCRATCH;
  if (!with_pack) {
    rc = upload(pl.tables_bytes);
    if (rc != TLORA_OK) return rc;
  }
  uint16_t* Sx = reinterpret_cast<uint16_t*>(ws + pl.off_Sx);
  uint16_t* atp = reinterpret_cast<uint16_t*>(ws + pl.off_atp);
  uint16_t* bp = reinterpret_cast<uint16_t*>(ws + pl.off_bp);
  float* sums = reinterpret_cast<float*>(shared_sums ? shared_sums : ws + pl.off_partial);
  const TileDev* tiles = reinterpret_cast<const TileDev*>(tb + pl.tb_tiles);
  const FragPack frags = pl.small_x ? small_frag_pack(pl, 0, p->X, in_index, sums) : FragPack();
  if (packed) {
    launch_frag_pack(frags, st);
  } else {
    Timed t(TLORA_K_PACK, st, timed);
    // (a backward that reuses this packing may need A_j side by side)
    uint16_t* const ap = !no_alloc && packs_a_all(pl) ? reinterpret_cast<uint16_t*>(ws + pl.off_ap) : nullptr;
    launch_pack_adapters(reinterpret_cast<JobDev*>(tb), pl.J, pl.d_in, pl.d_out, pl.max_rpad, pl.r_total, atp, ap, bp, frags,
                         with_pack ? blob.data() : nullptr, pl.tb_gBu, st);
  }
  if (pl.small_x) {
    Timed tg(TLORA_K_GEMM_FWD, st, timed);
    if (timed) g_clock_slot[0] = nullptr;             // (it takes no sample)
    launch_small(true, jobs, tiles, frags.out ? frags.out : static_cast<const uint16_t*>(p->X), static_cast<const uint16_t*>(p->W), atp, bp, pl.r_total,
                 static_cast<uint16_t*>(Y), out_index, in_index, pl.T, pl.d_in, pl.d_out, pl.small_x, sums,
                 no_alloc ? nullptr : reinterpret_cast<uint16_t*>(ws + pl.off_Shi), reinterpret_cast<uint16_t*>(ws + pl.off_Slo), st);
    return launches_ok(__LINE__);
  }
  {
    Timed t(TLORA_K_SHRINK, st, timed);
    run_shrink(pl, tb, jobs, tiles, static_cast<const uint16_t*>(p->X), pl.d_in, atp, true,
               reinterpret_cast<uint16_t*>(ws + pl.off_Shi), reinterpret_cast<uint16_t*>(ws + pl.off_Slo), Sx, in_index,
               sums, st);
  }
  GemmCall g;
  g.kernel = TLORA_K_GEMM_FWD;  g.w_is_kn = true;  g.timed = timed;
  g.tiles = tiles;
  g.op = {static_cast<const uint16_t*>(p->X), static_cast<const uint16_t*>(p->W), Sx, bp, static_cast<uint16_t*>(Y)};
  g.r_total = pl.r_total;  g.T = pl.T;  g.K = pl.d_in;  g.N = pl.d_out;
  g.out_index = out_index;  g.in_index = in_index;
  g.clk = timed ? reinterpret_cast<unsigned long long*>(ws + pl.off_clock) : nullptr;
  g.split = pl.gemm_split_fwd;  g.pair_split = pl.pair_split_fwd;  g.sums = sums;
  if (later && g.pairs()) *later = g;
  else launch_gemm(g, nullptr, st);
  return launches_ok(__LINE__);
}
}  // namespace
}  // namespace tlora

extern "C" {

int tlora_fwd(const tlora_problem_t* p, void* Y, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  return fwd_impl(p, Y, workspace, ws_bytes, hip_stream, false);
}

int tlora_fwd_noalloc(const tlora_problem_t* p, void* Y, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  uint8_t* ws = nullptr;
  const int rc = scratch_of_current_device(&ws);
  if (rc != TLORA_OK) return rc;
  return fwd_impl(p, Y, ws, TLORA_NOALLOC_SCRATCH_BYTES, hip_stream, true);
}

}  // extern "C"

namespace tlora {
namespace {
// What the nano-batches of one call have left in its workspace for those after them, copy by copy: a nano-batch in the two-launch
// form makes neither a_all nor W^T, and a later one of the other form may read either.
struct Copies {
  bool adapters = false;                                // A_j^T and B_j, packed
  bool a_all = false;                                   // A_j side by side
  bool wt = false;                                      // W^T
};
// The backward's launch sequence (out_index / in_index as in fwd_impl: dX rows are scattered; X and dY are fetched
// through the list; shared_sums as there, also for the partial tiles of dA / dB; later as there, the product then follows the
// gradients).
// copies: of the nano-batches before this one, brought up to date (null: no nano-batch).
// batch_tokens: of the whole batch, if the call is one of its nano-batches.  It decides whether dX has use for a copy of W^T.
int bwd_impl(const tlora_problem_t* p, const void* dY, void* dX, void* const* dA, void* const* dB, int flags,
             void* workspace, size_t ws_bytes, void* hip_stream, const int32_t* out_index, const int32_t* in_index,
             uint8_t* shared_sums = nullptr, GemmCall* later = nullptr, Copies* copies = nullptr, int64_t batch_tokens = 0) {
  const PlanEntry* entry = nullptr;
  std::vector<JobDev> hjobs;
  int rc = common_checks(p, &entry, hjobs, workspace, ws_bytes, false, shared_sums != nullptr);
  if (rc != TLORA_OK) return rc;
  const Plan& pl = entry->pl;
  if (pl.T > 0 && !dY) return TLORA_ENULL;
  if ((dA == nullptr) != (dB == nullptr)) return TLORA_ENULL;
  if (misaligned16(dY) || (dX && misaligned16(dX))) return TLORA_EALIGN;
  const bool want_grads = dA != nullptr;
  if (want_grads)
    for (int j = 0; j < pl.J; ++j) {
      if (pl.jobs[j].rank > 0 && (!dA[j] || !dB[j])) return TLORA_ENULL;
      hjobs[j].dA = dA[j];
      hjobs[j].dB = dB[j];
    }
  if (flags & ~(TLORA_BWD_REUSE_S | TLORA_BWD_REUSE_WT | TLORA_BWD_ACCUMULATE)) return TLORA_EINVAL;
  const bool accumulate = (flags & TLORA_BWD_ACCUMULATE) != 0;
  rc = check_arch();
  if (rc != TLORA_OK) return rc;
  const bool reuse_S = (flags & TLORA_BWD_REUSE_S) != 0;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  uint8_t* tb = ws + pl.off_tables;
  std::vector<uint8_t> blob = entry->blob;          // the cached tables, with this call's job table
  put(blob, pl.tb_jobs, hjobs);
  const JobDev* jobs = reinterpret_cast<const JobDev*>(tb + pl.tb_jobs);

  if (pl.dtype == TLORA_F32) {
    float* S = reinterpret_cast<float*>(ws + pl.off_S);
    float* dS = reinterpret_cast<float*>(ws + pl.off_dS);
    const float* X = static_cast<const float*>(p->X);
    const float* W = static_cast<const float*>(p->W);
    const float* dYf = static_cast<const float*>(dY);
    float* dXf = static_cast<float*>(dX);
    std::vector<F32Unit> units[2];
    std::vector<F32Tile> tiles[2];
    if (dXf)   // dX = dY . W^T : B(k = o, n = i) = W[i, o]
      f32_add(units[0], tiles[0], f32_unit(dYf, pl.d_out, 1, W, 1, pl.d_out, dXf, pl.d_in, pl.T, pl.d_in, pl.d_out, 1.f, false));
    for (int j = 0; j < pl.J; ++j) {
      const JobDev& jb = hjobs[j];
      const int Tj = jb.row1 - jb.row0;
      if (jb.rank == 0) continue;
      const float* Aj = static_cast<const float*>(jb.A);
      const float* Bj = static_cast<const float*>(jb.B);
      const float* Xj = X + (int64_t)jb.row0 * pl.d_in;
      const float* dYj = dYf + (int64_t)jb.row0 * pl.d_out;
      float* Sj = S + jb.soff;
      float* dSj = dS + jb.soff;
      // dS_j = dY_j . B_j^T : B(k = o, n = p) = B_j[p, o]
      f32_add(units[0], tiles[0], f32_unit(dYj, pl.d_out, 1, Bj, 1, pl.d_out, dSj, jb.rpad, Tj, jb.rank, pl.d_out, 1.f, false));
      if (!reuse_S && want_grads)
        f32_add(units[0], tiles[0], f32_unit(Xj, pl.d_in, 1, Aj, jb.rank, 1, Sj, jb.rpad, Tj, jb.rank, pl.d_in, 1.f, false));
      if (dXf)   // dX_j += s_j dS_j . A_j^T : B(k = p, n = i) = A_j[i, p]
        f32_add(units[1], tiles[1], f32_unit(dSj, jb.rpad, 1, Aj, 1, jb.rank, dXf + (int64_t)jb.row0 * pl.d_in, pl.d_in,
                                             Tj, pl.d_in, jb.rank, jb.scale, true));
      if (want_grads) {
        // dA_j = s_j X_j^T . dS_j : A(m = i, k = t) = X_j[t, i]
        f32_add(units[1], tiles[1], f32_unit(Xj, 1, pl.d_in, dSj, jb.rpad, 1, static_cast<float*>(jb.dA), jb.rank,
                                             pl.d_in, jb.rank, Tj, jb.scale, accumulate));
        // dB_j = s_j S_j^T . dY_j : A(m = p, k = t) = S_j[t, p]
        f32_add(units[1], tiles[1], f32_unit(Sj, 1, jb.rpad, dYj, pl.d_out, 1, static_cast<float*>(jb.dB), pl.d_out,
                                             jb.rank, pl.d_out, Tj, jb.scale, accumulate));
      }
    }
    F32Launch L;
    rc = f32_place(pl, blob, units, tiles, L);
    if (rc != TLORA_OK) return rc;
    rc = upload_tables(blob, tb, st);
    if (rc != TLORA_OK) return rc;
    for (int i = 0; i < 2; ++i) {
      Timed t(TLORA_K_F32, st);
      launch_f32_units(reinterpret_cast<const F32Unit*>(tb + L.units_at[i]),
                       reinterpret_cast<const F32Tile*>(tb + L.tiles_at[i]), L.ntiles[i], st);
    }
    return launches_ok(__LINE__);
  }

  const bool direct = dx_direct(std::max<int64_t>(batch_tokens, pl.T), pl.d_in, pl.d_out);
  // (the nano-batches of a large batch share its copy)
  const bool small = pl.small_dy && (batch_tokens <= pl.T || direct);
  const bool promised = (flags & TLORA_BWD_REUSE_WT) != 0, wt_there = copies && copies->wt;
  const bool wt = g_opt.dx_transposed_w != 0 && !small && (promised || !direct);
  const bool wt_made = wt && !promised && !wt_there;    // by a launch of its own, below
  uint16_t* Wt = reinterpret_cast<uint16_t*>(ws + pl.off_wt);
  WtCall wc;
  if (dX && pl.T > 0) {
    if (wt_there) wc.action = kWtKeep;
    else if (promised) wc.action = wt ? kWtEnsure : kWtKeep;
    else wc.action = wt ? kWtMade : kWtNone;
    wc.state = reinterpret_cast<WtState*>(ws + pl.off_wt_state);
    wc.W = static_cast<const uint16_t*>(p->W);
    wc.Wt = Wt;
    wc.rows = pl.d_in;  wc.cols = pl.d_out;
  }
  float* partial = reinterpret_cast<float*>(shared_sums ? shared_sums : ws + pl.off_partial);
  const bool redo_S = want_grads && !reuse_S;
  const FragPack frags = small && pl.T > 0 ? small_frag_pack(pl, 1, dY, in_index, partial) : FragPack();
  const bool frags_late = redo_S && !pl.frags_wait;
  rc = upload_tables(blob, tb, st, wc, frags_late ? FragPack() : frags);
  if (rc != TLORA_OK) return rc;
  uint16_t* Sx = reinterpret_cast<uint16_t*>(ws + pl.off_Sx);
  uint16_t* dSx = reinterpret_cast<uint16_t*>(ws + pl.off_dSx);
  uint16_t* Shi = reinterpret_cast<uint16_t*>(ws + pl.off_Shi);
  uint16_t* Slo = reinterpret_cast<uint16_t*>(ws + pl.off_Slo);
  uint16_t* dShi = reinterpret_cast<uint16_t*>(ws + pl.off_dShi);
  uint16_t* dSlo = reinterpret_cast<uint16_t*>(ws + pl.off_dSlo);
  uint16_t* atp = reinterpret_cast<uint16_t*>(ws + pl.off_atp);
  uint16_t* ap = reinterpret_cast<uint16_t*>(ws + pl.off_ap);
  uint16_t* bp = reinterpret_cast<uint16_t*>(ws + pl.off_bp);
  const TileDev* tiles = reinterpret_cast<const TileDev*>(tb + pl.tb_tiles);
  const uint16_t* Xb = static_cast<const uint16_t*>(p->X);
  const uint16_t* dYb = static_cast<const uint16_t*>(dY);

  {
    Timed t(TLORA_K_PACK, st);
    // with TLORA_BWD_REUSE_S the forward's packed copies of the (unchanged) adapters are still in the workspace, and a_all,
    // which only a dX product against W as it lies reads, if the forward's batch is one for it
    const bool need_a_all = dX && !wt && !small;
    const Copies have = reuse_S ? Copies{true, packs_a_all(pl)} : copies ? *copies : Copies();
    if (!have.adapters || (need_a_all && !have.a_all))
      launch_pack_adapters(reinterpret_cast<JobDev*>(tb), pl.J, pl.d_in, pl.d_out, pl.max_rpad, pl.r_total, atp,
                           need_a_all ? ap : nullptr, bp, FragPack(), nullptr, 0, st);
    if (copies) *copies = {true, have.a_all || need_a_all, wt_there || (dX && pl.T > 0 && wt)};
  }
  if (pl.T > 0) {
    if (redo_S) {
      Timed t(TLORA_K_SHRINK, st);
      if (pl.small_x) {
        const FragPack xf = small_frag_pack(pl, 0, Xb, in_index, partial);
        launch_frag_pack(xf, st);
        launch_small(true, jobs, tiles, xf.out ? xf.out : Xb, nullptr, atp, bp, pl.r_total, nullptr, nullptr, in_index, pl.T, pl.d_in, pl.d_out,
                     pl.small_x, partial, Shi, Slo, st);
      } else {
        run_shrink(pl, tb, jobs, tiles, Xb, pl.d_in, atp, true, Shi, Slo, Sx, in_index, partial, st);
      }
    }
    if (small) {
      Timed t(dX ? TLORA_K_GEMM_BWD : TLORA_K_SHRINK, st);
      if (g_prof_on && dX) g_clock_slot[1] = nullptr;
      if (frags_late) launch_frag_pack(frags, st);
      launch_small(false, jobs, tiles, frags.out ? frags.out : dYb, static_cast<const uint16_t*>(p->W), bp, atp, pl.r_total, static_cast<uint16_t*>(dX),
                   out_index, in_index, pl.T, pl.d_out, pl.d_in, pl.small_dy, partial, dShi, dSlo, st);
    } else {
      Timed t(TLORA_K_SHRINK, st);
      run_shrink(pl, tb, jobs, tiles, dYb, pl.d_out, bp, false, dShi, dSlo, dSx, in_index, partial, st);
    }
    if (dX && !small) {
      // dX = dY . W^T contracts over W's contiguous dimension.  Against a transposed copy of W the weight tiles
      // are 64 rows of 512 contiguous bytes instead of 256 rows of 128, which the load stream handles markedly
      // better (the copy costs one read and one write of W; W is frozen, so REUSE_WT skips it).
      if (wt_made) {
        Timed t(TLORA_K_WT, st);
        launch_transpose_bf16(static_cast<const uint16_t*>(p->W), Wt, pl.d_in, pl.d_out, st);
      }
      GemmCall g;
      g.kernel = TLORA_K_GEMM_BWD;  g.w_is_kn = wt;
      g.tiles = tiles;
      g.op = {dYb, wt ? Wt : static_cast<const uint16_t*>(p->W), dSx, wt ? atp : ap, static_cast<uint16_t*>(dX)};
      g.r_total = pl.r_total;  g.T = pl.T;  g.K = pl.d_out;  g.N = pl.d_in;
      g.out_index = out_index;  g.in_index = in_index;
      g.clk = g_prof_on ? reinterpret_cast<unsigned long long*>(ws + pl.off_clock) + 2 : nullptr;
      g.split = pl.gemm_split_bwd;  g.pair_split = pl.pair_split_bwd;  g.sums = partial;
      if (later && g.pairs()) *later = g;
      else launch_gemm(g, nullptr, st);
    }
  }
  if (want_grads) {
    const GradSide b = {reinterpret_cast<const GradUnit*>(tb + pl.tb_gBu), Shi, Slo, dYb, pl.d_out, (int)pl.gradB_units.size()};
    const GradSide a = {reinterpret_cast<const GradUnit*>(tb + pl.tb_gAu), dShi, dSlo, Xb, pl.d_in, (int)pl.gradA_units.size()};
    const GradSide none;
    auto gradients = [&](const GradSide& dB_side, const GradSide& dA_side) {
      Timed t(TLORA_K_RANK_GRAD, st);
      launch_rank_grad(jobs, dB_side, dA_side, partial, accumulate, in_index, st);
    };
    auto reduce = [&](size_t groups, size_t count, int D, bool out_is_dA) {
      Timed t(TLORA_K_GRAD_REDUCE, st);
      launch_grad_reduce(jobs, reinterpret_cast<const GradGroup*>(tb + groups), (int)count, partial, D, out_is_dA, accumulate, st);
    };
    gradients(b, pl.grads_merged ? a : none);
    reduce(pl.tb_gBg, pl.gradB_groups.size(), pl.d_out, false);
    if (!pl.grads_merged) gradients(none, a);           // (its partial tiles take the place of those of dB)
    reduce(pl.tb_gAg, pl.gradA_groups.size(), pl.d_in, true);
  }
  return launches_ok(__LINE__);
}

}  // namespace
}  // namespace tlora

extern "C" {

int tlora_bwd(const tlora_problem_t* p, const void* dY, void* dX, void* const* dA, void* const* dB, int flags,
              void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  return bwd_impl(p, dY, dX, dA, dB, flags, workspace, ws_bytes, hip_stream, nullptr, nullptr);
}

// ---- adaptive nano-batching (Sec. 3.3) --------------------------------------------------------------------
int tlora_aimd_init(tlora_aimd_t* c, int32_t n0, int32_t alpha, double beta, double tau_rel, int32_t n_max) {
  if (!c) return TLORA_ENULL;
  if (n0 < 1 || alpha < 1 || !(beta > 0.0 && beta < 1.0) || !(tau_rel >= 0.0) || n_max < 0) return TLORA_EINVAL;
  c->n = n_max > 0 ? std::min(n0, n_max) : n0;
  c->alpha = alpha;  c->n_max = n_max;  c->have_prev = 0;
  c->beta = beta;  c->tau_rel = tau_rel;  c->t_prev = 0.0;
  return TLORA_OK;
}

int tlora_aimd_update(tlora_aimd_t* c, double t_step, int32_t* n_next) {
  if (!c) return TLORA_ENULL;
  if (!(t_step >= 0.0) || c->n < 1) return TLORA_EINVAL;
  int64_t n = c->n;
  if (c->have_prev) {
    const double tau = c->tau_rel * c->t_prev;
    if (t_step <= c->t_prev - tau) n = n + c->alpha;                              // additive increase
    else n = std::max<int64_t>(1, (int64_t)std::floor(c->beta * (double)c->n));   // multiplicative decrease
  }
  if (c->n_max > 0) n = std::min<int64_t>(n, c->n_max);
  n = std::min<int64_t>(n, INT32_MAX);
  c->n = (int32_t)n;  c->t_prev = t_step;  c->have_prev = 1;
  if (n_next) *n_next = c->n;
  return TLORA_OK;
}

namespace {
// token boundary n of N nano-batches: whole samples of `granule` tokens, floor(n U / N) of the U samples
int64_t nano_bound(int64_t T, int64_t n, int64_t N, int64_t granule) {
  const int64_t units = (T + granule - 1) / granule;
  return std::min<int64_t>(T, granule * (int64_t)(((__int128)n * units) / N));
}
// sub-problem of one nano-batch: same jobs, the rows of each segment that fall into [b0, b1)
struct NanoSub {
  tlora_problem_t p;
  std::vector<int64_t> off;
  int64_t b0 = 0, b1 = 0;
};
int make_sub(const tlora_problem_t* p, int32_t n_nano, int64_t granule, int32_t n, NanoSub& s) {
  const int rc = validate(p);
  if (rc != TLORA_OK) return rc;
  if (n_nano < 1 || granule < 1 || n < 0 || n >= n_nano) return TLORA_EINVAL;
  const int64_t T = p->offsets[p->num_jobs];
  s.b0 = nano_bound(T, n, n_nano, granule);
  s.b1 = nano_bound(T, n + 1, n_nano, granule);
  s.off.resize(p->num_jobs + 1);
  for (int j = 0; j <= p->num_jobs; ++j) s.off[j] = std::min(std::max(p->offsets[j], s.b0), s.b1) - s.b0;
  s.p = *p;
  s.p.offsets = s.off.data();
  const size_t elt = p->dtype == TLORA_F32 ? 4 : 2;
  s.p.X = p->X ? static_cast<const uint8_t*>(p->X) + (size_t)s.b0 * p->d_in * elt : nullptr;
  return TLORA_OK;
}
}  // namespace

int tlora_nano_split(const tlora_problem_t* p, int32_t n_nano, int64_t granule, int32_t n, int64_t* row0,
                     int64_t* row1, int64_t* sub_offsets) {
  NanoSub s;
  const int rc = make_sub(p, n_nano, granule, n, s);
  if (rc != TLORA_OK) return rc;
  if (row0) *row0 = s.b0;
  if (row1) *row1 = s.b1;
  if (sub_offsets) std::copy(s.off.begin(), s.off.end(), sub_offsets);
  return TLORA_OK;
}

size_t tlora_nano_workspace_bytes(const tlora_problem_t* p, int32_t n_nano, int64_t granule) {
  size_t need = 0;
  for (int32_t n = 0; n < n_nano; ++n) {
    NanoSub s;
    if (make_sub(p, n_nano, granule, n, s) != TLORA_OK) return 0;
    const size_t b = tlora_workspace_bytes(&s.p);
    if (b == 0) return 0;
    need = std::max(need, b);
  }
  return need;
}

int tlora_fwd_nano(const tlora_problem_t* p, int32_t n_nano, int64_t granule, void* Y, void* workspace, size_t ws_bytes,
                   void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (!p) return TLORA_ENULL;
  const size_t need = tlora_nano_workspace_bytes(p, n_nano, granule);
  if (need == 0) return validate(p) != TLORA_OK ? validate(p) : TLORA_EINVAL;
  if (!workspace || ws_bytes < need) return TLORA_EWORKSPACE;
  const size_t elt = p->dtype == TLORA_F32 ? 4 : 2;
  bool packed = false;                            // the adapters are packed once: their copies lie where no batch size moves them
  for (int32_t n = 0; n < n_nano; ++n) {          // one after the other, on the caller's stream
    NanoSub s;
    int rc = make_sub(p, n_nano, granule, n, s);
    if (rc != TLORA_OK) return rc;
    if (s.b1 == s.b0) continue;
    rc = fwd_impl(&s.p, Y ? static_cast<uint8_t*>(Y) + (size_t)s.b0 * p->d_out * elt : nullptr, workspace, ws_bytes,
                  hip_stream, false, nullptr, nullptr, packed);
    if (rc != TLORA_OK) return rc;
    packed = true;
  }
  return TLORA_OK;
}

int tlora_bwd_nano(const tlora_problem_t* p, int32_t n_nano, int64_t granule, const void* dY, void* dX, void* const* dA,
                   void* const* dB, int flags, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (!p) return TLORA_ENULL;
  if (flags & ~(TLORA_BWD_REUSE_WT | TLORA_BWD_ACCUMULATE)) return TLORA_EINVAL;   // S of a nano-batch is not kept
  const size_t need = tlora_nano_workspace_bytes(p, n_nano, granule);
  if (need == 0) return validate(p) != TLORA_OK ? validate(p) : TLORA_EINVAL;
  if (!workspace || ws_bytes < need) return TLORA_EWORKSPACE;
  const size_t elt = p->dtype == TLORA_F32 ? 4 : 2;
  const int64_t T = p->offsets[p->num_jobs];
  bool first = true;
  Copies copies;
  for (int32_t n = 0; n < n_nano; ++n) {
    NanoSub s;
    int rc = make_sub(p, n_nano, granule, n, s);
    if (rc != TLORA_OK) return rc;
    if (s.b1 == s.b0 && !(first && n == n_nano - 1)) continue;      // (an all-empty batch still zeroes dA / dB once)
    // the adapter gradients are sums over the job's tokens: the first nano-batch overwrites, the others add
    const int f = first ? flags : flags | TLORA_BWD_ACCUMULATE;
    rc = bwd_impl(&s.p, dY ? static_cast<const uint8_t*>(dY) + (size_t)s.b0 * p->d_out * elt : nullptr,
                  dX ? static_cast<uint8_t*>(dX) + (size_t)s.b0 * p->d_in * elt : nullptr, dA, dB, f, workspace, ws_bytes,
                  hip_stream, nullptr, nullptr, nullptr, nullptr, &copies, T);
    if (rc != TLORA_OK) return rc;
    first = false;
  }
  return TLORA_OK;
}

// ---- per-job optimizer step ---------------------------------------------------------------------------------
size_t tlora_adamw_workspace_bytes(int32_t count) {
  if (count < 0) return 0;
  return std::max<size_t>(256, align_up(sizeof(AdamwDev) * (size_t)count, 256));
}

int tlora_adamw_step(const tlora_adamw_tensor_t* tensors, int32_t count, int32_t dtype, void* workspace, size_t ws_bytes,
                     void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (count < 0) return TLORA_EINVAL;
  if (dtype != TLORA_F32 && dtype != TLORA_BF16) return TLORA_EDTYPE;
  if (count > 0 && !tensors) return TLORA_ENULL;
  if (count > 65535) return TLORA_EINVAL;
  std::vector<uint8_t> blob(sizeof(AdamwDev) * (size_t)count);
  AdamwDev* d = reinterpret_cast<AdamwDev*>(blob.data());
  int64_t max_n = 0;
  for (int i = 0; i < count; ++i) {
    const tlora_adamw_tensor_t& t = tensors[i];
    if (t.n < 0 || t.step < 1 || !(t.beta1 >= 0.f && t.beta1 < 1.f) || !(t.beta2 >= 0.f && t.beta2 < 1.f) ||
        !(t.eps >= 0.f) || !(t.lr >= 0.f) || !(t.weight_decay >= 0.f))
      return TLORA_EINVAL;
    if (t.n > 0 && (!t.param || !t.grad || !t.m || !t.v)) return TLORA_ENULL;
    if (t.n > 0 && dtype == TLORA_BF16 && !t.master) return TLORA_ENULL;   // a bf16 tensor cannot carry the update
    d[i].param = t.param;  d[i].master = t.master;  d[i].grad = t.grad;  d[i].m = t.m;  d[i].v = t.v;  d[i].n = t.n;
    d[i].lr = t.lr;  d[i].beta1 = t.beta1;  d[i].beta2 = t.beta2;  d[i].eps = t.eps;  d[i].weight_decay = t.weight_decay;
    d[i].c1 = (float)(1.0 / (1.0 - std::pow((double)t.beta1, (double)t.step)));
    d[i].c2 = (float)(1.0 / (1.0 - std::pow((double)t.beta2, (double)t.step)));
    d[i].param_is_bf16 = dtype == TLORA_BF16;
    max_n = std::max(max_n, t.n);
  }
  if (count == 0 || max_n == 0) return TLORA_OK;
  if (!workspace || ws_bytes < tlora_adamw_workspace_bytes(count) || (reinterpret_cast<uintptr_t>(workspace) & 255))
    return TLORA_EWORKSPACE;
  int rc = check_arch();
  if (rc != TLORA_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  rc = upload_tables(blob, workspace, st);
  if (rc != TLORA_OK) return rc;
  {
    Timed t(TLORA_K_OPT, st);
    launch_adamw(static_cast<const AdamwDev*>(workspace), count, max_n, st);
  }
  return launches_ok(__LINE__);
}

// ---- MLP block: RMSNorm -> gate / up (fused multi-LoRA) -> silu(G) * U -> down (fused multi-LoRA) -> + X -------
namespace {
// One projection of a block.  The projections run one after the other on one stream, so the block has one place for their
// sums and partial tiles (the last part of a workspace); everything else of a workspace is the projection's own.
struct LayerBytes {
  size_t own = 0, sums = 0;
};
bool layer_bytes(const tlora_problem_t* p, LayerBytes& b) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  const PlanEntry* e = nullptr;
  if (get_plan(p, false, &e) != TLORA_OK) return false;
  const bool bf16 = e->pl.dtype == TLORA_BF16;
  b.own = bf16 ? e->pl.off_partial : e->pl.total;
  b.sums = bf16 ? e->pl.partial_bytes : 0;
  return true;
}
int layer_fwd(const tlora_problem_t* p, void* Y, uint8_t* ws, size_t own, uint8_t* sums, void* hip_stream,
              GemmCall* later = nullptr) {
  return fwd_impl(p, Y, ws, own, hip_stream, false, nullptr, nullptr, false, p->dtype == TLORA_BF16 ? sums : nullptr, later);
}
int layer_bwd(const tlora_problem_t* p, const void* dY, void* dX, void* const* dA, void* const* dB, int flags, uint8_t* ws,
              size_t own, uint8_t* sums, void* hip_stream, GemmCall* later = nullptr) {
  return bwd_impl(p, dY, dX, dA, dB, flags, ws, own, hip_stream, nullptr, nullptr,
                  p->dtype == TLORA_BF16 ? sums : nullptr, later);
}

struct MlpLayout {
  tlora_problem_t gate, up, down;      // the three fused layers (X pointers filled in below)
  size_t elt = 2;
  int64_t T = 0;
  size_t off_xn = 0, off_rstd = 0, off_g = 0, off_u = 0, off_z = 0, off_d = 0, off_dz = 0, off_dg = 0, off_du = 0,
         off_dxa = 0, off_dxb = 0, off_ws_gate = 0, off_ws_up = 0, off_ws_down = 0, off_sums = 0;
  size_t ws_gate = 0, ws_up = 0, ws_down = 0, total = 0;
};
int mlp_layout(const tlora_mlp_t* p, MlpLayout& L) {
  if (!p) return TLORA_ENULL;
  if (p->dtype != TLORA_F32 && p->dtype != TLORA_BF16) return TLORA_EDTYPE;
  if (!(p->eps >= 0.f)) return TLORA_EINVAL;
  auto layer = [&](int d_in, int d_out, const void* W, const void* const* A, const void* const* B) {
    tlora_problem_t q;
    memset(&q, 0, sizeof(q));
    q.dtype = p->dtype;  q.num_jobs = p->num_jobs;  q.d_in = d_in;  q.d_out = d_out;
    q.ranks = p->ranks;  q.offsets = p->offsets;  q.scales = p->scales;
    q.X = nullptr;  q.W = W;  q.A = A;  q.B = B;
    return q;
  };
  L.gate = layer(p->d_model, p->d_ff, p->W_gate, p->A_gate, p->B_gate);
  L.up = layer(p->d_model, p->d_ff, p->W_up, p->A_up, p->B_up);
  L.down = layer(p->d_ff, p->d_model, p->W_down, p->A_down, p->B_down);
  L.gate.X = L.up.X = L.down.X = p->X;          // placeholder so that validation sees a non-null activation
  int rc = validate(&L.gate);
  if (rc == TLORA_OK) rc = validate(&L.up);
  if (rc == TLORA_OK) rc = validate(&L.down);
  if (rc != TLORA_OK) return rc;
  L.T = p->offsets[p->num_jobs];
  if (L.T > 0 && !p->gamma) return TLORA_ENULL;
  L.elt = p->dtype == TLORA_F32 ? 4 : 2;
  size_t w = 0;
  auto place = [&](size_t bytes) { const size_t at = w;  w = align_up(w + bytes, 256);  return at; };
  const size_t td = (size_t)L.T * p->d_model * L.elt, tf = (size_t)L.T * p->d_ff * L.elt;
  L.off_xn = place(td);  L.off_rstd = place(sizeof(float) * (size_t)L.T);
  L.off_g = place(tf);  L.off_u = place(tf);  L.off_z = place(tf);  L.off_d = place(td);
  L.off_dz = place(tf);  L.off_dg = place(tf);  L.off_du = place(tf);  L.off_dxa = place(td);  L.off_dxb = place(td);
  LayerBytes gate, up, down;
  if (!layer_bytes(&L.gate, gate) || !layer_bytes(&L.up, up) || !layer_bytes(&L.down, down)) return TLORA_EINVAL;
  L.ws_gate = gate.own;  L.ws_up = up.own;  L.ws_down = down.own;
  L.off_ws_gate = place(L.ws_gate);  L.off_ws_up = place(L.ws_up);  L.off_ws_down = place(L.ws_down);
  L.off_sums = place(std::max({gate.sums, up.sums, down.sums}));
  L.total = w;
  return TLORA_OK;
}
}  // namespace

size_t tlora_mlp_workspace_bytes(const tlora_mlp_t* p) {
  MlpLayout L;
  return mlp_layout(p, L) == TLORA_OK ? L.total : 0;
}

int tlora_mlp_fwd(const tlora_mlp_t* p, void* Out, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  MlpLayout L;
  int rc = mlp_layout(p, L);
  if (rc != TLORA_OK) return rc;
  if (!workspace || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TLORA_EWORKSPACE;
  if (L.T > 0 && (!p->X || !Out)) return TLORA_ENULL;
  if (misaligned16(p->X) || misaligned16(Out) || misaligned16(p->gamma)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK) return rc;
  if (L.T == 0) return TLORA_OK;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  const bool bf = p->dtype == TLORA_BF16;
  {
    Timed t(TLORA_K_GLUE, st);
    launch_rmsnorm_fwd(bf, p->X, p->gamma, p->eps, (int)L.T, p->d_model, ws + L.off_xn,
                       reinterpret_cast<float*>(ws + L.off_rstd), st);
  }
  L.gate.X = L.up.X = ws + L.off_xn;
  GemmCall gate, up;
  rc = layer_fwd(&L.gate, ws + L.off_g, ws + L.off_ws_gate, L.ws_gate, ws + L.off_sums, hip_stream, &gate);
  if (rc != TLORA_OK) return rc;
  rc = layer_fwd(&L.up, ws + L.off_u, ws + L.off_ws_up, L.ws_up, ws + L.off_sums, hip_stream, &up);
  if (rc != TLORA_OK) return rc;
  launch_gemm_pair(gate, up, st);
  {
    Timed t(TLORA_K_GLUE, st);
    launch_swiglu_fwd(bf, ws + L.off_g, ws + L.off_u, ws + L.off_z, L.T * p->d_ff, st);
  }
  L.down.X = ws + L.off_z;
  rc = layer_fwd(&L.down, ws + L.off_d, ws + L.off_ws_down, L.ws_down, ws + L.off_sums, hip_stream);
  if (rc != TLORA_OK) return rc;
  {
    Timed t(TLORA_K_GLUE, st);
    launch_residual_add(bf, p->X, ws + L.off_d, Out, L.T * p->d_model, st);
  }
  return launches_ok(__LINE__);
}

int tlora_mlp_bwd(const tlora_mlp_t* p, const void* dOut, void* dX, void* const* dA_gate, void* const* dB_gate,
                  void* const* dA_up, void* const* dB_up, void* const* dA_down, void* const* dB_down, int flags,
                  void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  MlpLayout L;
  int rc = mlp_layout(p, L);
  if (rc != TLORA_OK) return rc;
  if (flags & ~(TLORA_BWD_ACCUMULATE | TLORA_BWD_REUSE_WT)) return TLORA_EINVAL;
  if (!workspace || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TLORA_EWORKSPACE;
  if (L.T > 0 && (!p->X || !dOut || !dX)) return TLORA_ENULL;
  if (!dA_gate || !dB_gate || !dA_up || !dB_up || !dA_down || !dB_down) return TLORA_ENULL;
  if (misaligned16(p->X) || misaligned16(dOut) || misaligned16(dX) || misaligned16(p->gamma)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  const bool bf = p->dtype == TLORA_BF16;
  // every layer's workspace still holds its S_j from tlora_mlp_fwd
  const int lf = flags | TLORA_BWD_REUSE_S;
  L.gate.X = L.up.X = ws + L.off_xn;
  L.down.X = ws + L.off_z;
  rc = layer_bwd(&L.down, dOut, ws + L.off_dz, dA_down, dB_down, lf, ws + L.off_ws_down, L.ws_down, ws + L.off_sums, hip_stream);
  if (rc != TLORA_OK) return rc;
  if (L.T > 0) {
    Timed t(TLORA_K_GLUE, st);
    launch_swiglu_bwd(bf, ws + L.off_g, ws + L.off_u, ws + L.off_dz, ws + L.off_dg, ws + L.off_du, L.T * p->d_ff, st);
  }
  GemmCall gate, up;
  rc = layer_bwd(&L.gate, ws + L.off_dg, ws + L.off_dxa, dA_gate, dB_gate, lf, ws + L.off_ws_gate, L.ws_gate, ws + L.off_sums, hip_stream, &gate);
  if (rc != TLORA_OK) return rc;
  rc = layer_bwd(&L.up, ws + L.off_du, ws + L.off_dxb, dA_up, dB_up, lf, ws + L.off_ws_up, L.ws_up, ws + L.off_sums, hip_stream, &up);
  if (rc != TLORA_OK) return rc;
  launch_gemm_pair(gate, up, st);
  if (L.T > 0) {
    Timed t(TLORA_K_GLUE, st);
    launch_rmsnorm_bwd(bf, p->X, p->gamma, reinterpret_cast<const float*>(ws + L.off_rstd), ws + L.off_dxa,
                       ws + L.off_dxb, nullptr, dOut, (int)L.T, p->d_model, dX, st);
  }
  return launches_ok(__LINE__);
}

// ---- attention half: rotary embedding, causal grouped-query attention, and the block around them ----------
namespace {
struct AttnPlan {
  int64_t T = 0;
  std::vector<AttnTile> tiles;
  std::vector<int32_t> pos;
  int64_t max_len = 0;
  size_t off_tiles = 0, off_pos = 0, off_D = 0, off_rope = 0, blob_bytes = 0, total = 0;
};
// tables: [tiles | positions] (uploaded), then D fp32 [T, n_heads] and the rotary (cos, sin) table [longest sequence, 64]
int attn_plan(int32_t num_seqs, const int64_t* seq_offsets, int32_t n_heads, bool want_tables, AttnPlan& A) {
  if (num_seqs < 0 || n_heads < 1) return TLORA_EINVAL;
  if (!seq_offsets) return TLORA_ENULL;
  if (seq_offsets[0] != 0) return TLORA_EINVAL;
  size_t n_tiles = 0;
  for (int32_t s = 0; s < num_seqs; ++s) {
    const int64_t len = seq_offsets[s + 1] - seq_offsets[s];
    if (len < 0 || seq_offsets[s + 1] > (int64_t)INT32_MAX) return TLORA_EINVAL;
    n_tiles += (size_t)((len + 127) / 128);
    A.max_len = std::max(A.max_len, len);
  }
  A.T = seq_offsets[num_seqs];
  if ((int64_t)A.T * n_heads > (int64_t)INT32_MAX) return TLORA_EINVAL;
  if (want_tables) {
    A.tiles.reserve(n_tiles);
    A.pos.resize((size_t)A.T);
    // longest sequences' last tiles first: a tile's work grows with t0, so the heavy ones start early
    for (int32_t s = 0; s < num_seqs; ++s) {
      const int64_t a = seq_offsets[s], len = seq_offsets[s + 1] - a;
      for (int64_t t0 = 0; t0 < len; t0 += 128) A.tiles.push_back(AttnTile{(int32_t)a, (int32_t)len, (int32_t)t0, 0});
      for (int64_t i = 0; i < len; ++i) A.pos[(size_t)(a + i)] = (int32_t)i;
    }
    std::stable_sort(A.tiles.begin(), A.tiles.end(), [](const AttnTile& x, const AttnTile& y) { return x.t0 > y.t0; });
  }
  size_t w = 0;
  auto place = [&](size_t bytes) { const size_t at = w;  w = align_up(w + bytes, 256);  return at; };
  A.off_tiles = place(n_tiles * sizeof(AttnTile));
  A.off_pos = place((size_t)A.T * sizeof(int32_t));
  A.blob_bytes = w;
  A.off_D = place((size_t)A.T * n_heads * sizeof(float));
  A.off_rope = place((size_t)A.max_len * 64 * 2 * sizeof(float));
  A.total = std::max<size_t>(w, 256);
  return TLORA_OK;
}
int attn_upload(const AttnPlan& A, void* ws, hipStream_t st) {
  std::vector<uint8_t> blob(A.blob_bytes, 0);
  if (!A.tiles.empty()) memcpy(blob.data() + A.off_tiles, A.tiles.data(), A.tiles.size() * sizeof(AttnTile));
  if (!A.pos.empty()) memcpy(blob.data() + A.off_pos, A.pos.data(), A.pos.size() * sizeof(int32_t));
  if (blob.empty()) return TLORA_OK;
  return upload_tables(blob, ws, st);
}
int attn_heads_ok(int32_t n_heads, int32_t n_kv, int32_t head_dim) {
  if (head_dim != kAttnHeadDim) return TLORA_EINVAL;
  if (n_heads < 1 || n_kv < 1 || n_heads % n_kv != 0 || n_heads > 4096) return TLORA_EINVAL;   // 32-bit byte offsets inside a tile
  return TLORA_OK;
}
inline bool bad_ws(const void* ws, size_t have, size_t need) {
  return !ws || have < need || (reinterpret_cast<uintptr_t>(ws) & 255);
}
}  // namespace

size_t tlora_attention_workspace_bytes(int32_t num_seqs, const int64_t* seq_offsets, int32_t n_heads) {
  AttnPlan A;
  return attn_plan(num_seqs, seq_offsets, n_heads, false, A) == TLORA_OK ? A.total : 0;
}

int tlora_rope(void* X, int32_t num_seqs, const int64_t* seq_offsets, int32_t heads, int32_t head_dim, float rope_base,
               int32_t inverse, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (head_dim != kAttnHeadDim || !(rope_base > 1.f) || heads > 4096) return TLORA_EINVAL;
  AttnPlan A;
  int rc = attn_plan(num_seqs, seq_offsets, heads, true, A);
  if (rc != TLORA_OK) return rc;
  if (bad_ws(workspace, ws_bytes, A.total)) return TLORA_EWORKSPACE;
  if (A.T > 0 && !X) return TLORA_ENULL;
  if (misaligned16(X)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK || A.T == 0) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  rc = attn_upload(A, ws, st);
  if (rc != TLORA_OK) return rc;
  {
    Timed t(TLORA_K_ROPE, st);
    launch_rope_table(reinterpret_cast<float*>(ws + A.off_rope), (int)A.max_len, rope_base, st);
    launch_rope(static_cast<uint16_t*>(X), reinterpret_cast<const int32_t*>(ws + A.off_pos),
                reinterpret_cast<const float*>(ws + A.off_rope), A.T, heads, inverse != 0, st);
  }
  return launches_ok(__LINE__);
}

int tlora_attention_fwd(const void* Q, const void* K, const void* V, void* O, float* lse, int32_t num_seqs,
                        const int64_t* seq_offsets, int32_t n_heads, int32_t n_kv_heads, int32_t head_dim, void* workspace,
                        size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  int rc = attn_heads_ok(n_heads, n_kv_heads, head_dim);
  if (rc != TLORA_OK) return rc;
  AttnPlan A;
  rc = attn_plan(num_seqs, seq_offsets, n_heads, true, A);
  if (rc != TLORA_OK) return rc;
  if (bad_ws(workspace, ws_bytes, A.total)) return TLORA_EWORKSPACE;
  if (A.T > 0 && (!Q || !K || !V || !O || !lse)) return TLORA_ENULL;
  if (misaligned16(Q) || misaligned16(K) || misaligned16(V) || misaligned16(O)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK || A.T == 0) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  rc = attn_upload(A, ws, st);
  if (rc != TLORA_OK) return rc;
  {
    Timed t(TLORA_K_ATTN_FWD, st);
    launch_attn_fwd(reinterpret_cast<const AttnTile*>(ws + A.off_tiles), (int)A.tiles.size(), static_cast<const uint16_t*>(Q),
                    static_cast<const uint16_t*>(K), static_cast<const uint16_t*>(V), static_cast<uint16_t*>(O), lse,
                    n_heads, n_kv_heads, st);
  }
  return launches_ok(__LINE__);
}

int tlora_attention_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO, const float* lse,
                        void* dQ, void* dK, void* dV, int32_t num_seqs, const int64_t* seq_offsets, int32_t n_heads,
                        int32_t n_kv_heads, int32_t head_dim, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  int rc = attn_heads_ok(n_heads, n_kv_heads, head_dim);
  if (rc != TLORA_OK) return rc;
  AttnPlan A;
  rc = attn_plan(num_seqs, seq_offsets, n_heads, true, A);
  if (rc != TLORA_OK) return rc;
  if (bad_ws(workspace, ws_bytes, A.total)) return TLORA_EWORKSPACE;
  if (A.T > 0 && (!Q || !K || !V || !O || !dO || !lse || !dQ || !dK || !dV)) return TLORA_ENULL;
  if (misaligned16(Q) || misaligned16(K) || misaligned16(V) || misaligned16(O) || misaligned16(dO) || misaligned16(dQ) ||
      misaligned16(dK) || misaligned16(dV))
    return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK || A.T == 0) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  rc = attn_upload(A, ws, st);
  if (rc != TLORA_OK) return rc;
  {
    Timed t(TLORA_K_ATTN_BWD, st);
    launch_attn_bwd(reinterpret_cast<const AttnTile*>(ws + A.off_tiles), (int)A.tiles.size(), static_cast<const uint16_t*>(Q),
                    static_cast<const uint16_t*>(K), static_cast<const uint16_t*>(V), static_cast<const uint16_t*>(O),
                    static_cast<const uint16_t*>(dO), lse, reinterpret_cast<float*>(ws + A.off_D),
                    static_cast<uint16_t*>(dQ), static_cast<uint16_t*>(dK), static_cast<uint16_t*>(dV), n_heads,
                    n_kv_heads, st);
  }
  return launches_ok(__LINE__);
}

namespace {
struct AttnLayout {
  tlora_problem_t q, k, v, o;
  AttnPlan A;
  int64_t T = 0;
  size_t off_attn = 0, off_xn = 0, off_rstd = 0, off_q = 0, off_k = 0, off_v = 0, off_o = 0, off_lse = 0, off_d = 0,
         off_do = 0, off_dq = 0, off_dk = 0, off_dv = 0, off_dxa = 0, off_dxb = 0, off_dxc = 0, off_ws[4] = {0, 0, 0, 0}, off_sums = 0;
  size_t ws_l[4] = {0, 0, 0, 0}, total = 0;
};
int attn_layout(const tlora_attn_t* p, bool want_tables, AttnLayout& L) {
  if (!p) return TLORA_ENULL;
  if (p->dtype != TLORA_BF16) return TLORA_EDTYPE;
  if (!(p->eps >= 0.f) || !(p->rope_base > 1.f)) return TLORA_EINVAL;
  int rc = attn_heads_ok(p->n_heads, p->n_kv_heads, p->head_dim);
  if (rc != TLORA_OK) return rc;
  if (p->num_jobs < 0 || !p->offsets) return p->offsets ? TLORA_EINVAL : TLORA_ENULL;
  const int dq = p->n_heads * p->head_dim, dkv = p->n_kv_heads * p->head_dim;
  auto layer = [&](int d_in, int d_out, const void* W, const void* const* A, const void* const* B) {
    tlora_problem_t q;
    memset(&q, 0, sizeof(q));
    q.dtype = p->dtype;  q.num_jobs = p->num_jobs;  q.d_in = d_in;  q.d_out = d_out;
    q.ranks = p->ranks;  q.offsets = p->offsets;  q.scales = p->scales;
    q.X = p->X;  q.W = W;  q.A = A;  q.B = B;      // X: placeholder so that validation sees a non-null activation
    return q;
  };
  L.q = layer(p->d_model, dq, p->W_q, p->A_q, p->B_q);
  L.k = layer(p->d_model, dkv, p->W_k, p->A_k, p->B_k);
  L.v = layer(p->d_model, dkv, p->W_v, p->A_v, p->B_v);
  L.o = layer(dq, p->d_model, p->W_o, p->A_o, p->B_o);
  tlora_problem_t* ls[4] = {&L.q, &L.k, &L.v, &L.o};
  for (tlora_problem_t* l : ls) {
    rc = validate(l);
    if (rc != TLORA_OK) return rc;
  }
  L.T = p->offsets[p->num_jobs];
  rc = attn_plan(p->num_seqs, p->seq_offsets, p->n_heads, want_tables, L.A);
  if (rc != TLORA_OK) return rc;
  if (L.A.T != L.T) return TLORA_EINVAL;
  if (L.T > 0 && !p->gamma) return TLORA_ENULL;
  size_t w = 0;
  auto place = [&](size_t bytes) { const size_t at = w;  w = align_up(w + bytes, 256);  return at; };
  const size_t td = (size_t)L.T * p->d_model * 2, tq = (size_t)L.T * dq * 2, tk = (size_t)L.T * dkv * 2;
  L.off_attn = place(L.A.total);
  L.off_xn = place(td);  L.off_rstd = place(sizeof(float) * (size_t)L.T);
  L.off_q = place(tq);  L.off_k = place(tk);  L.off_v = place(tk);  L.off_o = place(tq);
  L.off_lse = place(sizeof(float) * (size_t)L.T * p->n_heads);
  L.off_d = place(td);
  L.off_do = place(tq);  L.off_dq = place(tq);  L.off_dk = place(tk);  L.off_dv = place(tk);
  L.off_dxa = place(td);  L.off_dxb = place(td);  L.off_dxc = place(td);
  size_t sums = 0;
  for (int i = 0; i < 4; ++i) {
    LayerBytes b;
    if (!layer_bytes(ls[i], b)) return TLORA_EINVAL;
    L.ws_l[i] = b.own;
    L.off_ws[i] = place(b.own);
    sums = std::max(sums, b.sums);
  }
  L.off_sums = place(sums);
  L.total = w;
  return TLORA_OK;
}
}  // namespace

size_t tlora_attn_workspace_bytes(const tlora_attn_t* p) {
  AttnLayout L;
  return attn_layout(p, false, L) == TLORA_OK ? L.total : 0;
}

int tlora_attn_fwd(const tlora_attn_t* p, void* Out, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  AttnLayout L;
  int rc = attn_layout(p, true, L);
  if (rc != TLORA_OK) return rc;
  if (bad_ws(workspace, ws_bytes, L.total)) return TLORA_EWORKSPACE;
  if (L.T > 0 && (!p->X || !Out)) return TLORA_ENULL;
  if (misaligned16(p->X) || misaligned16(Out) || misaligned16(p->gamma)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK || L.T == 0) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  uint8_t* aw = ws + L.off_attn;
  rc = attn_upload(L.A, aw, st);
  if (rc != TLORA_OK) return rc;
  {
    Timed t(TLORA_K_GLUE, st);
    launch_rmsnorm_fwd(true, p->X, p->gamma, p->eps, (int)L.T, p->d_model, ws + L.off_xn,
                       reinterpret_cast<float*>(ws + L.off_rstd), st);
  }
  L.q.X = L.k.X = L.v.X = ws + L.off_xn;
  rc = layer_fwd(&L.q, ws + L.off_q, ws + L.off_ws[0], L.ws_l[0], ws + L.off_sums, hip_stream);
  GemmCall k, v;
  if (rc == TLORA_OK) rc = layer_fwd(&L.k, ws + L.off_k, ws + L.off_ws[1], L.ws_l[1], ws + L.off_sums, hip_stream, &k);
  if (rc == TLORA_OK) rc = layer_fwd(&L.v, ws + L.off_v, ws + L.off_ws[2], L.ws_l[2], ws + L.off_sums, hip_stream, &v);
  if (rc != TLORA_OK) return rc;
  launch_gemm_pair(k, v, st);
  const int32_t* pos = reinterpret_cast<const int32_t*>(aw + L.A.off_pos);
  {
    Timed t(TLORA_K_ROPE, st);
    float* tab = reinterpret_cast<float*>(aw + L.A.off_rope);
    launch_rope_table(tab, (int)L.A.max_len, p->rope_base, st);
    launch_rope(reinterpret_cast<uint16_t*>(ws + L.off_q), pos, tab, L.T, p->n_heads, false, st);
    launch_rope(reinterpret_cast<uint16_t*>(ws + L.off_k), pos, tab, L.T, p->n_kv_heads, false, st);
  }
  {
    Timed t(TLORA_K_ATTN_FWD, st);
    launch_attn_fwd(reinterpret_cast<const AttnTile*>(aw + L.A.off_tiles), (int)L.A.tiles.size(),
                    reinterpret_cast<const uint16_t*>(ws + L.off_q), reinterpret_cast<const uint16_t*>(ws + L.off_k),
                    reinterpret_cast<const uint16_t*>(ws + L.off_v), reinterpret_cast<uint16_t*>(ws + L.off_o),
                    reinterpret_cast<float*>(ws + L.off_lse), p->n_heads, p->n_kv_heads, st);
  }
  L.o.X = ws + L.off_o;
  rc = layer_fwd(&L.o, ws + L.off_d, ws + L.off_ws[3], L.ws_l[3], ws + L.off_sums, hip_stream);
  if (rc != TLORA_OK) return rc;
  {
    Timed t(TLORA_K_GLUE, st);
    launch_residual_add(true, p->X, ws + L.off_d, Out, L.T * p->d_model, st);
  }
  return launches_ok(__LINE__);
}

int tlora_attn_bwd(const tlora_attn_t* p, const void* dOut, void* dX, void* const* const* dA, void* const* const* dB,
                   int flags, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  AttnLayout L;
  int rc = attn_layout(p, true, L);
  if (rc != TLORA_OK) return rc;
  if (flags & ~(TLORA_BWD_ACCUMULATE | TLORA_BWD_REUSE_WT)) return TLORA_EINVAL;
  if (bad_ws(workspace, ws_bytes, L.total)) return TLORA_EWORKSPACE;
  if (L.T > 0 && (!p->X || !dOut || !dX)) return TLORA_ENULL;
  if (!dA || !dB) return TLORA_ENULL;
  for (int i = 0; i < 4; ++i)
    if (!dA[i] || !dB[i]) return TLORA_ENULL;
  if (misaligned16(p->X) || misaligned16(dOut) || misaligned16(dX) || misaligned16(p->gamma)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  uint8_t* aw = ws + L.off_attn;
  const int lf = flags | TLORA_BWD_REUSE_S;            // every projection's workspace still holds its S_j
  L.q.X = L.k.X = L.v.X = ws + L.off_xn;
  L.o.X = ws + L.off_o;
  rc = layer_bwd(&L.o, dOut, ws + L.off_do, dA[3], dB[3], lf, ws + L.off_ws[3], L.ws_l[3], ws + L.off_sums, hip_stream);
  if (rc != TLORA_OK) return rc;
  if (L.T > 0) {
    const int32_t* pos = reinterpret_cast<const int32_t*>(aw + L.A.off_pos);   // tables uploaded by tlora_attn_fwd
    {
      Timed t(TLORA_K_ATTN_BWD, st);
      launch_attn_bwd(reinterpret_cast<const AttnTile*>(aw + L.A.off_tiles), (int)L.A.tiles.size(),
                      reinterpret_cast<const uint16_t*>(ws + L.off_q), reinterpret_cast<const uint16_t*>(ws + L.off_k),
                      reinterpret_cast<const uint16_t*>(ws + L.off_v), reinterpret_cast<const uint16_t*>(ws + L.off_o),
                      reinterpret_cast<const uint16_t*>(ws + L.off_do), reinterpret_cast<const float*>(ws + L.off_lse),
                      reinterpret_cast<float*>(aw + L.A.off_D), reinterpret_cast<uint16_t*>(ws + L.off_dq),
                      reinterpret_cast<uint16_t*>(ws + L.off_dk), reinterpret_cast<uint16_t*>(ws + L.off_dv),
                      p->n_heads, p->n_kv_heads, st);
    }
    {
      Timed t(TLORA_K_ROPE, st);
      const float* tab = reinterpret_cast<const float*>(aw + L.A.off_rope);     // written by tlora_attn_fwd
      launch_rope(reinterpret_cast<uint16_t*>(ws + L.off_dq), pos, tab, L.T, p->n_heads, true, st);
      launch_rope(reinterpret_cast<uint16_t*>(ws + L.off_dk), pos, tab, L.T, p->n_kv_heads, true, st);
    }
  }
  rc = layer_bwd(&L.q, ws + L.off_dq, ws + L.off_dxa, dA[0], dB[0], lf, ws + L.off_ws[0], L.ws_l[0], ws + L.off_sums, hip_stream);
  GemmCall k, v;
  if (rc == TLORA_OK) rc = layer_bwd(&L.k, ws + L.off_dk, ws + L.off_dxb, dA[1], dB[1], lf, ws + L.off_ws[1], L.ws_l[1], ws + L.off_sums, hip_stream, &k);
  if (rc == TLORA_OK) rc = layer_bwd(&L.v, ws + L.off_dv, ws + L.off_dxc, dA[2], dB[2], lf, ws + L.off_ws[2], L.ws_l[2], ws + L.off_sums, hip_stream, &v);
  if (rc != TLORA_OK) return rc;
  launch_gemm_pair(k, v, st);
  if (L.T > 0) {
    Timed t(TLORA_K_GLUE, st);
    launch_rmsnorm_bwd(true, p->X, p->gamma, reinterpret_cast<const float*>(ws + L.off_rstd), ws + L.off_dxa,
                       ws + L.off_dxb, ws + L.off_dxc, dOut, (int)L.T, p->d_model, dX, st);
  }
  return launches_ok(__LINE__);
}

// ---- one decoder layer: attention block, then MLP block -----------------------------------------------------
namespace {
struct LayerLayout {
  tlora_attn_t attn;
  tlora_mlp_t mlp;
  int64_t T = 0;
  size_t off_h = 0, off_dh = 0, off_attn = 0, off_mlp = 0, ws_attn = 0, ws_mlp = 0, total = 0;
};
int layer_layout(const tlora_layer_t* p, LayerLayout& L) {
  if (!p) return TLORA_ENULL;
  L.attn = p->attn;
  L.mlp = p->mlp;
  const tlora_attn_t& a = L.attn;
  const tlora_mlp_t& m = L.mlp;
  if (a.dtype != TLORA_BF16 || m.dtype != TLORA_BF16) return TLORA_EDTYPE;
  if (a.num_jobs != m.num_jobs || a.d_model != m.d_model || a.num_jobs < 0) return TLORA_EINVAL;
  if (!a.offsets || !m.offsets) return TLORA_ENULL;
  if (a.num_jobs > 0 && (!a.ranks || !m.ranks || !a.scales || !m.scales)) return TLORA_ENULL;
  for (int j = 0; j < a.num_jobs; ++j)
    if (a.ranks[j] != m.ranks[j] || a.scales[j] != m.scales[j] || a.offsets[j] != m.offsets[j]) return TLORA_EINVAL;
  if (a.offsets[a.num_jobs] != m.offsets[a.num_jobs]) return TLORA_EINVAL;
  L.mlp.X = a.X;                         // placeholder for validation; the real input is H
  L.ws_attn = tlora_attn_workspace_bytes(&L.attn);
  L.ws_mlp = tlora_mlp_workspace_bytes(&L.mlp);
  if (!L.ws_attn || !L.ws_mlp) return TLORA_EINVAL;
  L.T = a.offsets[a.num_jobs];
  size_t w = 0;
  auto place = [&](size_t bytes) { const size_t at = w;  w = align_up(w + bytes, 256);  return at; };
  const size_t td = (size_t)L.T * a.d_model * 2;
  L.off_h = place(td);  L.off_dh = place(td);
  L.off_attn = place(L.ws_attn);  L.off_mlp = place(L.ws_mlp);
  L.total = std::max<size_t>(w, 256);
  return TLORA_OK;
}
}  // namespace

size_t tlora_layer_workspace_bytes(const tlora_layer_t* p) {
  LayerLayout L;
  return layer_layout(p, L) == TLORA_OK ? L.total : 0;
}

int tlora_layer_fwd(const tlora_layer_t* p, void* Out, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  LayerLayout L;
  int rc = layer_layout(p, L);
  if (rc != TLORA_OK) return rc;
  if (bad_ws(workspace, ws_bytes, L.total)) return TLORA_EWORKSPACE;
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  rc = tlora_attn_fwd(&L.attn, ws + L.off_h, ws + L.off_attn, L.ws_attn, hip_stream);
  if (rc != TLORA_OK) return rc;
  L.mlp.X = ws + L.off_h;
  return tlora_mlp_fwd(&L.mlp, Out, ws + L.off_mlp, L.ws_mlp, hip_stream);
}

int tlora_layer_bwd(const tlora_layer_t* p, const void* dOut, void* dX, void* const* const* dA, void* const* const* dB,
                    int flags, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  LayerLayout L;
  int rc = layer_layout(p, L);
  if (rc != TLORA_OK) return rc;
  if (bad_ws(workspace, ws_bytes, L.total)) return TLORA_EWORKSPACE;
  if (!dA || !dB) return TLORA_ENULL;
  for (int i = 0; i < 7; ++i)
    if (!dA[i] || !dB[i]) return TLORA_ENULL;
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  L.mlp.X = ws + L.off_h;
  rc = tlora_mlp_bwd(&L.mlp, dOut, ws + L.off_dh, dA[4], dB[4], dA[5], dB[5], dA[6], dB[6], flags, ws + L.off_mlp, L.ws_mlp,
                     hip_stream);
  if (rc != TLORA_OK) return rc;
  return tlora_attn_bwd(&L.attn, ws + L.off_dh, dX, dA, dB, flags, ws + L.off_attn, L.ws_attn, hip_stream);
}

// ---- general token -> adapter assignment (Sec. 3.3: tokens of an adapter are gathered, results scattered back) ----
namespace {
struct IndexedLayout {
  size_t inner = 0, off_x = 0, off_y = 0, off_dx = 0, off_idx = 0, total = 0, elt = 2;
  int64_t T = 0;
};
// The kernels that fetch rows through the index list keep 32-bit byte offsets from the tensor's base.
inline bool direct_index_ok(int64_t T, int64_t width) {
  return g_opt.indexed_direct != 0 && T * width * 2 < ((int64_t)1 << 32);
}
int indexed_layout(const tlora_problem_t* p, IndexedLayout& L) {
  const int rc = validate(p);
  if (rc != TLORA_OK) return rc;
  L.inner = tlora_workspace_bytes(p);
  if (L.inner == 0) return TLORA_EINVAL;
  L.T = p->offsets[p->num_jobs];
  L.elt = p->dtype == TLORA_F32 ? 4 : 2;
  L.off_x = align_up(L.inner, 256);
  L.off_y = align_up(L.off_x + (size_t)L.T * p->d_in * L.elt, 256);
  L.off_dx = align_up(L.off_y + (size_t)L.T * p->d_out * L.elt, 256);
  // the fp32 configuration has no scattering epilogue: its sorted dX is staged and scattered by a copy pass
  L.off_idx = align_up(L.off_dx + (p->dtype == TLORA_F32 ? (size_t)L.T * p->d_in * L.elt : 0), 256);
  // the row list as the kernels use it: the caller's, with every entry forced into [0, T)
  L.total = align_up(L.off_idx + (size_t)L.T * sizeof(int32_t), 256);
  return TLORA_OK;
}
// Everything tlora_fwd / tlora_bwd would reject, checked before the first launch of an indexed call.
int indexed_checks(const tlora_problem_t* q, void* workspace, size_t inner, bool backward, void* const* dA,
                   void* const* dB, int flags) {
  const PlanEntry* e = nullptr;
  std::vector<JobDev> hj;
  const int rc = common_checks(q, &e, hj, workspace, inner);
  if (rc != TLORA_OK || !backward) return rc;
  if ((dA == nullptr) != (dB == nullptr)) return TLORA_ENULL;
  if (dA)
    for (int j = 0; j < q->num_jobs; ++j)
      if (q->ranks[j] > 0 && (!dA[j] || !dB[j])) return TLORA_ENULL;
  if (flags & ~(TLORA_BWD_REUSE_S | TLORA_BWD_REUSE_WT | TLORA_BWD_ACCUMULATE)) return TLORA_EINVAL;
  return TLORA_OK;
}
}  // namespace

size_t tlora_indexed_workspace_bytes(const tlora_problem_t* p) {
  IndexedLayout L;
  return indexed_layout(p, L) == TLORA_OK ? L.total : 0;
}

int tlora_fwd_indexed(const tlora_problem_t* p, const int32_t* row_index, void* Y, void* workspace, size_t ws_bytes,
                      void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  IndexedLayout L;
  int rc = indexed_layout(p, L);
  if (rc != TLORA_OK) return rc;
  if (!workspace || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TLORA_EWORKSPACE;
  if (L.T > 0 && (!row_index || !Y || !p->X)) return TLORA_ENULL;
  if (misaligned16(Y) || misaligned16(p->X)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK) return rc;
  if (L.T == 0) return TLORA_OK;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  int32_t* const index = reinterpret_cast<int32_t*>(ws + L.off_idx);
  // bf16: the kernels fetch the activation rows through the list inside their loads and the GEMM scatters its output
  // rows, so the batch is read and written exactly as often as in a contiguous call (the in-kernel row offsets are 32
  // bits: larger activations take the gathered copy below)
  const bool direct = p->dtype == TLORA_BF16 && direct_index_ok(L.T, p->d_in);
  tlora_problem_t q = *p;
  if (!direct) q.X = ws + L.off_x;
  rc = indexed_checks(&q, workspace, L.inner, false, nullptr, nullptr, 0);
  if (rc != TLORA_OK) return rc;
  {
    Timed t(TLORA_K_PERMUTE, st);
    launch_clamp_index(row_index, index, L.T, st);
  }
  if (direct) return fwd_impl(p, Y, workspace, L.inner, hip_stream, false, index, index);
  {
    Timed t(TLORA_K_PERMUTE, st);
    launch_permute_rows(p->X, ws + L.off_x, index, L.T, (int64_t)p->d_in * L.elt, false, st);
  }
  if (p->dtype == TLORA_BF16) return fwd_impl(&q, Y, workspace, L.inner, hip_stream, false, index);
  rc = tlora_fwd(&q, ws + L.off_y, workspace, L.inner, hip_stream);
  if (rc != TLORA_OK) return rc;
  Timed t(TLORA_K_PERMUTE, st);
  launch_permute_rows(ws + L.off_y, Y, index, L.T, (int64_t)p->d_out * L.elt, true, st);
  return launches_ok(__LINE__);
}

int tlora_bwd_indexed(const tlora_problem_t* p, const int32_t* row_index, const void* dY, void* dX, void* const* dA,
                      void* const* dB, int flags, void* workspace, size_t ws_bytes, void* hip_stream) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  IndexedLayout L;
  int rc = indexed_layout(p, L);
  if (rc != TLORA_OK) return rc;
  if (!workspace || ws_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255)) return TLORA_EWORKSPACE;
  if (L.T > 0 && (!row_index || !dY || !p->X)) return TLORA_ENULL;
  if (misaligned16(dY) || misaligned16(dX) || misaligned16(p->X)) return TLORA_EALIGN;
  rc = check_arch();
  if (rc != TLORA_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  int32_t* const index = reinterpret_cast<int32_t*>(ws + L.off_idx);
  const bool direct = p->dtype == TLORA_BF16 && direct_index_ok(L.T, std::max(p->d_in, p->d_out));
  tlora_problem_t q = *p;
  if (!direct) q.X = ws + L.off_x;
  rc = indexed_checks(&q, workspace, L.inner, true, dA, dB, flags);
  if (rc != TLORA_OK) return rc;
  if (L.T > 0) {   // made again: the region may have been reused since the forward
    Timed t(TLORA_K_PERMUTE, st);
    launch_clamp_index(row_index, index, L.T, st);
  }
  if (direct) return bwd_impl(p, dY, dX, dA, dB, flags, workspace, L.inner, hip_stream, index, index);
  if (L.T > 0) {
    Timed t(TLORA_K_PERMUTE, st);
    // the sorted activations are gathered again: the region may have been reused since the forward
    launch_permute_rows(p->X, ws + L.off_x, index, L.T, (int64_t)p->d_in * L.elt, false, st);
    launch_permute_rows(dY, ws + L.off_y, index, L.T, (int64_t)p->d_out * L.elt, false, st);
  }
  if (p->dtype == TLORA_BF16 || !dX)
    return bwd_impl(&q, ws + L.off_y, dX, dA, dB, flags, workspace, L.inner, hip_stream, index, nullptr);
  rc = tlora_bwd(&q, ws + L.off_y, ws + L.off_dx, dA, dB, flags, workspace, L.inner, hip_stream);
  if (rc != TLORA_OK) return rc;
  Timed t(TLORA_K_PERMUTE, st);
  launch_permute_rows(ws + L.off_dx, dX, index, L.T, (int64_t)p->d_in * L.elt, true, st);
  return launches_ok(__LINE__);
}

int tlora_plan_dump(const tlora_problem_t* p, int32_t* rpad, int64_t* soff, int32_t* tile_rows, int64_t* tile_row0,
                    int32_t* tile_nrows, int32_t* tile_job_first, int32_t* tile_job_last, int64_t* n_tiles) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  const PlanEntry* e = nullptr;
  const int rc = get_plan(p, false, &e);
  if (rc != TLORA_OK) return rc;
  const Plan& pl = e->pl;
  for (int j = 0; j < pl.J; ++j) {
    if (rpad) rpad[j] = pl.jobs[j].rpad;
    if (soff) soff[j] = pl.jobs[j].soff;
  }
  if (soff) soff[pl.J] = pl.s_elems;
  if (tile_rows) *tile_rows = kGemmBM;
  const int64_t nt = (int64_t)pl.tile_jobs.size();
  if (n_tiles) {
    const int64_t cap = *n_tiles;
    *n_tiles = nt;
    if (cap < nt && (tile_row0 || tile_nrows || tile_job_first || tile_job_last)) return TLORA_EINVAL;
  } else if (tile_row0 || tile_nrows || tile_job_first || tile_job_last) {
    return TLORA_ENULL;
  }
  for (int64_t t = 0; t < nt; ++t) {
    if (tile_row0) tile_row0[t] = t * kGemmBM;
    if (tile_nrows) tile_nrows[t] = (int32_t)std::min<int64_t>(kGemmBM, pl.T - t * kGemmBM);
    if (tile_job_first) tile_job_first[t] = pl.tile_jobs[t].first;
    if (tile_job_last) tile_job_last[t] = pl.tile_jobs[t].last;
  }
  return TLORA_OK;
}

// Host-side consistency check of a freshly built plan: every table entry and every workspace region that a kernel
// will index lies where the kernels assume.  Numbered checks; returns the number of the first one that fails.
static int check_plan(const Plan& pl, bool fwd_only) {
  const bool bf16 = pl.dtype == TLORA_BF16;
  // 1x: jobs
  int64_t soff = 0, atp = 0, roff = 0;
  int row = 0;
  for (int j = 0; j < pl.J; ++j) {
    const JobDev& jb = pl.jobs[j];
    if (jb.row0 != row || jb.row1 < jb.row0) return 10;
    row = jb.row1;
    if (jb.rpad < jb.rank || jb.rpad % kRankGranule || jb.rpad - jb.rank >= kRankGranule) return 11;
    if (jb.soff != soff || jb.atp_off != atp || jb.roff != roff) return 12;
    soff += (int64_t)((jb.row1 - jb.row0 + kGradStep - 1) / kGradStep * kGradStep) * jb.rpad;
    atp += (int64_t)jb.rpad * pl.d_in;
    roff += jb.rpad;
  }
  if (row != pl.T || soff != pl.s_elems || atp != pl.atp_elems || roff != pl.r_total) return 13;
  // 2x: row tiles of the GEMM
  if ((int64_t)pl.tile_jobs.size() != ((int64_t)pl.T + kGemmBM - 1) / kGemmBM) return 20;
  int64_t aoff = 0;
  for (size_t tm = 0; tm < pl.tile_jobs.size(); ++tm) {
    const TileDev& td = pl.tile_jobs[tm];
    const int r0 = (int)tm * kGemmBM, r1 = std::min(pl.T, r0 + kGemmBM);
    if (td.first < 0 || td.last < td.first || td.last >= pl.J) return 21;
    for (int j = 0; j < pl.J; ++j) {          // every job with a row inside the tile lies in first..last
      const JobDev& jb = pl.jobs[j];
      const bool inside = std::max(jb.row0, r0) < std::min(jb.row1, r1);
      if (inside && (j < td.first || j > td.last)) return 22;
    }
    if (td.kext < 0 || td.kext % kGemmBK || td.roff_first != pl.jobs[td.first].roff) return 23;
    if (pl.jobs[td.last].roff + pl.jobs[td.last].rpad > td.roff_first + td.kext) return 24;
    if (td.roff_first + td.kext > pl.r_total + 32) return 25;       // the packed adapters carry 32 spare rank rows
    if (td.aoff != aoff) return 26;
    aoff += (int64_t)kGemmBM * td.kext;
  }
  if (aoff != pl.sx_elems) return 27;
  if (bf16) {
    // 3x: shrink work units tile [row0, row1) x [0, rpad) of every job exactly once
    auto check_shrink = [&](const std::vector<ShrinkUnit>& units, int rows, int cols) -> int {
      std::vector<int64_t> covered(pl.J, 0);
      for (const ShrinkUnit& u : units) {
        if (u.job < 0 || u.job >= pl.J) return 30;
        const JobDev& jb = pl.jobs[u.job];
        if (u.nrows < 1 || u.nrows > rows || u.t0 < jb.row0 || u.t0 + u.nrows > jb.row1) return 31;
        if ((u.t0 - jb.row0) % rows) return 32;
        if (u.pb < 0 || u.pb * cols >= jb.rpad) return 33;
        covered[u.job] += (int64_t)u.nrows * std::min(cols, jb.rpad - u.pb * cols);
      }
      for (int j = 0; j < pl.J; ++j)
        if (covered[j] != (int64_t)(pl.jobs[j].row1 - pl.jobs[j].row0) * pl.jobs[j].rpad) return 34;
      return 0;
    };
    if (pl.shrink_rows != 32 && pl.shrink_rows != 64 && pl.shrink_rows != 128) return 35;
    if (pl.shrink_rows == 32 && (pl.d_in % 64 || pl.d_out % 64)) return 36;
    if (int rc = check_shrink(pl.shrink_units, 64, kShrinkCols)) return rc;
    if (int rc = check_shrink(pl.stream_units, pl.shrink_rows, 128)) return rc + 100;
    // 4x: dA / dB work units and their partial tiles
    std::vector<std::pair<int64_t, int64_t>> spans;                  // of partial tiles in use at a time
    auto check_grad = [&](const std::vector<GradUnit>& units, const std::vector<GradGroup>& groups, int D) -> int {
      std::map<std::tuple<int, int, int>, std::vector<const GradUnit*>> by_tile;
      for (const GradUnit& u : units) {
        if (u.job < 0 || u.job >= pl.J) return 40;
        const JobDev& jb = pl.jobs[u.job];
        if (u.t0 < jb.row0 || u.t1 < u.t0 || u.t1 > jb.row1 || u.t1 - u.t0 > kGradMaxTokens) return 41;
        if ((u.t0 - jb.row0) % kGradStep) return 42;                 // the packed S rows are padded to the token step
        if (u.cb < 0 || u.cb * kGradCols >= D || u.pb < 0 || u.pb * kGradBlockRanks >= jb.rpad || jb.rank == 0) return 43;
        if (u.mb != grad_live_blocks(jb, u.pb) || u.mb < 1) return 44;
        const int64_t n = (int64_t)u.mb * kGradRanks * kGradCols;
        by_tile[{u.job, u.cb, u.pb}].push_back(&u);
        if (u.part_off < 0) {                                        // the whole job, also an idle one
          if (u.t0 != jb.row0 || u.t1 != jb.row1) return 54;
          continue;
        }
        if (u.t1 == u.t0) return 41;
        if (u.part_off + n > pl.grad_partial) return 45;
        spans.push_back({u.part_off, n});
      }
      // every output tile (job with a rank, column block, rank block) has a unit of its own, or one group whose partial tiles are
      // the units of the same (job, cb, pb), consecutive in memory and covering the job's tokens (none, if it has no tokens)
      if ((int64_t)units.size() > kMaxUnits) return 56;
      size_t alone = 0;
      for (const GradGroup& g : groups)
        if (g.nunits == 0) by_tile[{g.job, g.cb, g.pb}];
      for (const auto& t : by_tile) alone += t.second.size() == 1 && t.second[0]->part_off < 0;
      if ((int64_t)by_tile.size() != grad_tiles(pl, D) || alone + groups.size() != by_tile.size()) return 47;
      for (const GradGroup& g : groups) {
        if (g.job < 0 || g.job >= pl.J) return 48;
        const JobDev& jb = pl.jobs[g.job];
        auto& us = by_tile[{g.job, g.cb, g.pb}];
        if ((int)us.size() != g.nunits || (g.nunits < 2 && (g.nunits != 0 || jb.row1 != jb.row0))) return 49;
        std::sort(us.begin(), us.end(), [](const GradUnit* a, const GradUnit* b) { return a->t0 < b->t0; });
        int t = jb.row0;
        for (int k = 0; k < g.nunits; ++k) {
          if (us[k]->t0 != t || us[k]->mb != g.mb) return 50;
          if (us[k]->part_off != g.part_off + (int64_t)k * g.mb * kGradRanks * kGradCols) return 51;
          t = us[k]->t1;
        }
        if (t != jb.row1) return 52;
      }
      return 0;
    };
    if (!fwd_only) {
      auto disjoint = [&] {
        std::sort(spans.begin(), spans.end());
        for (size_t i = 1; i < spans.size(); ++i)
          if (spans[i - 1].first + spans[i - 1].second > spans[i].first) return false;
        return true;
      };
      if (int rc = check_grad(pl.gradB_units, pl.gradB_groups, pl.d_out)) return rc;
      if (!disjoint()) return 46;
      if (!pl.grads_merged) spans.clear();
      if (int rc = check_grad(pl.gradA_units, pl.gradA_groups, pl.d_in)) return rc + 100;
      if (!disjoint()) return 146;
      if (pl.grads_merged && (int64_t)(pl.gradB_units.size() + pl.gradA_units.size()) > kMaxUnits) return 56;
    } else if (!pl.gradA_units.empty() || !pl.gradB_units.empty()) {
      return 55;
    }
  }
  // 6x: tables inside the blob, regions inside the workspace, nothing overlapping
  {
    std::vector<std::pair<size_t, size_t>> t = {
        {pl.tb_jobs, sizeof(JobDev) * pl.jobs.size()},          {pl.tb_tiles, sizeof(TileDev) * pl.tile_jobs.size()},
        {pl.tb_shrink, sizeof(ShrinkUnit) * pl.shrink_units.size()}, {pl.tb_stream, sizeof(ShrinkUnit) * pl.stream_units.size()},
        {pl.tb_gBu, sizeof(GradUnit) * pl.gradB_units.size()},  {pl.tb_gBg, sizeof(GradGroup) * pl.gradB_groups.size()},
        {pl.tb_gAu, sizeof(GradUnit) * pl.gradA_units.size()},  {pl.tb_gAg, sizeof(GradGroup) * pl.gradA_groups.size()}};
    if (pl.dtype == TLORA_F32) t.push_back({pl.tb_f32, pl.f32_reserved});
    size_t end = 0;
    for (auto& r : t) {
      if (r.first % (r.first == pl.tb_gBg || r.first == pl.tb_gAg ? sizeof(GradGroup) : 256) || r.first < end) return 60;
      end = r.first + r.second;
    }
    if (end > pl.tables_bytes) return 61;
  }
  {
    std::vector<std::pair<size_t, size_t>> w;
    const size_t se = (size_t)pl.s_elems, sx = 2 * (size_t)pl.sx_elems + 256;
    if (bf16 && !fwd_only) {
      w.push_back({pl.off_wt, 2 * (size_t)pl.d_in * (size_t)pl.d_out});
      if (pl.off_wt_state != pl.off_clock + kClockBytes) return 77;
      w.push_back({pl.off_clock, kClockBytes + sizeof(WtState)});
    }
    if (bf16) {
      w.push_back({pl.off_atp, 2 * ((size_t)pl.atp_elems + 32 * (size_t)pl.d_in)});
      w.push_back({pl.off_bp, 2 * (size_t)pl.d_out * (size_t)(pl.r_total + 32)});
      w.push_back({pl.off_ap, 2 * (size_t)pl.d_in * (size_t)(pl.r_total + 32)});
    }
    w.push_back({pl.off_tables, pl.tables_bytes});
    if (!bf16 || fwd_only) w.push_back({pl.off_clock, kClockBytes});
    if (!bf16) {
      w.push_back({pl.off_S, 4 * se});
      if (!fwd_only) w.push_back({pl.off_dS, 4 * se});
    } else {
      w.push_back({pl.off_Shi, 2 * se});
      w.push_back({pl.off_Slo, 2 * se});
      if (!fwd_only) { w.push_back({pl.off_dShi, 2 * se});  w.push_back({pl.off_dSlo, 2 * se}); }
      w.push_back({pl.off_Sx, sx});
      if (!fwd_only) w.push_back({pl.off_dSx, sx});
      if (4 * (size_t)pl.grad_partial > pl.partial_bytes) return 64;
      for (int k : {pl.shrink_splits_x, pl.shrink_splits_dy})
        if (k < 1 || (k > 1 && 4 * se * (size_t)k > pl.partial_bytes)) return 65;
      for (int d = 0; d < 2; ++d) {
        const GemmSplit& g = d ? pl.gemm_split_bwd : pl.gemm_split_fwd;
        if (g.splits < 1 || g.splits > kGemmMaxSplits || g.n_direct < 0 || g.n_direct % 256) return 67;
        if (g.splits > 1) {                              // all shares have work in the longest tile
          int kext = 0;
          for (const TileDev& td : pl.tile_jobs) kext = std::max(kext, td.kext);
          const int steps = ((d ? pl.d_out : pl.d_in) + kext) / kGemmBK;
          if (gemm_share(steps, g.splits) * (g.splits - 1) >= steps) return 69;
        }
        if (gemm_split_bytes(pl, g, d ? pl.d_in : pl.d_out) > pl.partial_bytes) return 68;
        if (!fwd_only && gemm_split_bytes(pl, d ? pl.pair_split_bwd : pl.pair_split_fwd, d ? pl.d_in : pl.d_out, 2) > pl.partial_bytes)
          return 68;
      }
      for (int d = 0; d < 2; ++d) {
        const int k = d ? pl.small_dy : pl.small_x, K = d ? pl.d_out : pl.d_in, N = d ? pl.d_in : pl.d_out;
        if (k == 0) continue;
        if (pl.T < 1 || pl.T > kSmallRows || pl.tile_jobs.size() != 1 || K % 64 || N % 64 || k < 1 || k > K / 64) return 71;
        if (small_part_bytes(pl, N, k) > pl.partial_bytes) return 72;
        if (!small_frags(small_blocks(pl.T))) continue;
        const size_t at = small_frag_at(pl, d);
        if (at % 256 || at + small_frag_bytes(pl, K) > pl.partial_bytes) return 73;
        if (at < small_part_bytes(pl, N, k)) return 74;
        // dY's beside what making S again writes
        if (d && pl.small_x &&
            at < std::max(small_part_bytes(pl, pl.d_out, pl.small_x), small_frag_at(pl, 0) + small_frag_bytes(pl, pl.d_in))) return 75;
        if (d && !pl.small_x && pl.frags_wait && pl.shrink_splits_x > 1 && at < 4 * se * (size_t)pl.shrink_splits_x) return 76;
      }
      if (!fwd_only) w.push_back({pl.off_partial, pl.partial_bytes});
      else if (pl.total != forward_bytes(pl)) return 70;
      else if (pl.off_partial < TLORA_NOALLOC_SCRATCH_BYTES ||
               (pl.total <= TLORA_NOALLOC_SCRATCH_BYTES && pl.partial_bytes > TLORA_NOALLOC_SUM_BYTES)) return 66;
    }
    size_t end = 0;
    for (auto& r : w) {
      if (r.first % 256 || r.first < end) return 62;
      end = r.first + r.second;
    }
    if (end > pl.total) return 63;
  }
  return 0;
}

int tlora_plan_check(const tlora_problem_t* p, int32_t fwd_only, int32_t* failed_check) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (failed_check) *failed_check = 0;
  Plan pl;
  const int rc = build_plan(p, pl, fwd_only != 0);
  if (rc != TLORA_OK) return rc;
  const int bad = check_plan(pl, fwd_only != 0);
  if (failed_check) *failed_check = bad;
  return bad ? TLORA_EINVAL : TLORA_OK;
}

int tlora_plan_cuts(const tlora_problem_t* p, int32_t fwd_only, int32_t* cuts) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (!cuts) return TLORA_ENULL;
  Plan pl;
  const int rc = build_plan(p, pl, fwd_only != 0);
  if (rc != TLORA_OK) return rc;
  cuts[0] = pl.shrink_splits_x;
  cuts[1] = pl.shrink_splits_dy;
  for (int d = 0; d < 2; ++d) {
    const GemmSplit& g = d ? pl.gemm_split_bwd : pl.gemm_split_fwd;
    const int N = d ? pl.d_in : pl.d_out;
    cuts[2 + 2 * d] = g.splits > 1 ? g.n_direct : (int32_t)(pl.tile_jobs.size() * ((N + kGemmBN - 1) / kGemmBN));
    cuts[3 + 2 * d] = g.splits;
    const int small = d ? pl.small_dy : pl.small_x;
    if (small) {                                         // shares of a split: its workgroups' waves
      const int steps = (d ? pl.d_out : pl.d_in) / 64 / small;
      cuts[d] = cuts[3 + 2 * d] = small * std::min(4, std::max(1, (steps + 1) / 2));
      cuts[2 + 2 * d] = 0;
    }
  }
  return TLORA_OK;
}

int tlora_profile(int enable) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  const int rc = prof_drain();
  if (enable < 0 || enable > 2) return TLORA_EINVAL;
  g_prof_on = enable != 0;
  g_prof_gemm_only = enable == 2;
  if (g_prof_on) g_clock_slot[0] = g_clock_slot[1] = nullptr;
  if (g_prof_on)
    for (int i = 0; i < TLORA_K_COUNT; ++i) {
      g_prof_ms[i] = 0.0;
      g_prof_n[i] = 0;
    }
  return rc;
}

int tlora_profile_read(int kernel_class, double* total_ms, int64_t* launches) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (kernel_class < 0 || kernel_class >= TLORA_K_COUNT) return TLORA_EINVAL;
  const int rc = prof_drain();
  if (rc != TLORA_OK) return rc;
  if (total_ms) *total_ms = g_prof_ms[kernel_class];
  if (launches) *launches = g_prof_n[kernel_class];
  return TLORA_OK;
}

int tlora_profile_clock(double* ghz_fwd, double* ghz_bwd) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  double* out[2] = {ghz_fwd, ghz_bwd};
  for (int i = 0; i < 2; ++i) {
    if (!out[i]) continue;
    *out[i] = 0.0;
    if (!g_clock_slot[i]) continue;
    unsigned long long h[2] = {0, 0};
    TLORA_HIP(hipMemcpy(h, g_clock_slot[i], sizeof(h), hipMemcpyDeviceToHost));
    if (h[1] > 0) *out[i] = (double)h[0] / ((double)h[1] * 10.0);     // cycles per 10 ns tick -> GHz
  }
  return TLORA_OK;
}

int tlora_set_option(const char* name, int64_t value) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (!name) return TLORA_ENULL;
  const std::string n(name);
  if (n == "shrink_rows") {
    if (value != 0 && value != 32 && value != 64 && value != 128) return TLORA_EINVAL;
    g_opt.shrink_rows = (int)value;
    return TLORA_OK;
  }
  if (n == "shrink_stages") {
    if (value != 4 && value != 8) return TLORA_EINVAL;
    g_opt.shrink_stages = (int)value;
    return TLORA_OK;
  }
  if (n == "dx_transposed_w") {
    if (value != 0 && value != 1) return TLORA_EINVAL;
    g_opt.dx_transposed_w = (int)value;
    return TLORA_OK;
  }
  if (n == "indexed_direct") {
    if (value != 0 && value != 1) return TLORA_EINVAL;
    g_opt.indexed_direct = (int)value;
    return TLORA_OK;
  }
  if (n == "table_copy_kernel") {
    if (value != 0 && value != 1) return TLORA_EINVAL;
    g_opt.table_copy_kernel = (int)value;
    return TLORA_OK;
  }
  if (n == "plan_cache") {
    if (value != 0 && value != 1) return TLORA_EINVAL;
    g_opt.plan_cache = (int)value;
    g_plans.clear();
    return TLORA_OK;
  }
  if (n == "grad_tokens") {
    if (value < 64 || value % 64 || value > kGradMaxTokens) return TLORA_EINVAL;
    g_opt.grad_tokens = (int)value;
    return TLORA_OK;
  }
  return TLORA_EINVAL;
}

const char* tlora_last_hip_error(void) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  static char text[160];
  if (g_hip_err == 0) return "none";
  snprintf(text, sizeof(text), "%s (%d) at line %d of tlora_api.hip", hipGetErrorName((hipError_t)g_hip_err), g_hip_err,
           g_hip_line);
  return text;
}

const char* tlora_strerror(int status) {
  switch (status) {
    case TLORA_OK: return "ok";
    case TLORA_EINVAL: return "invalid problem size, offsets, rank or option";
    case TLORA_ENULL: return "a required pointer is null";
    case TLORA_EDTYPE: return "unsupported dtype";
    case TLORA_EWORKSPACE: return "workspace missing, misaligned or too small";
    case TLORA_EARCH: return "the current device is not gfx950";
    case TLORA_EHIP: return "a HIP runtime call failed";
    case TLORA_EALIGN: return "X, W, Y, dY or dX is not 16-byte aligned";
    case TLORA_ESCRATCH: return "problem too large for the static scratch of tlora_fwd_noalloc";
    default: return "unknown status";
  }
}

const char* tlora_version(void) { return "tlora-gfx950 0.1"; }

}  // extern "C"
