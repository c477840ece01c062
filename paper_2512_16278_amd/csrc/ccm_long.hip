// Sums of Eq. 1 (Sec. 3.2) for sub-intervals longer than the int32 bound
// (Table 1 runs sub-intervals up to 10 s = 203,450 samples of 49.152 us).
//
// Each sub-interval's time range is cut into P chunks of c samples, the last
// one shorter. One launch of the sums engine forms the exact int32 sums of every
// (sub-interval, chunk) pair, as if each chunk were a sub-interval of its own
// (ksplit = P), and a widening pass adds the P int32 records of each cell into
// its int64 record
//     rec[cell][b]          = sum_t x_b(t)
//     rec[cell][n + pair]   = sum_t x_a(t) x_b(t)
// exact for any L <= RFI_MAX_COUNT_LONG (|sums| < 255^2 2^18 < 2^34).
//
// P is at least ceil(L / RFI_MAX_COUNT) (each chunk within the int32 bound);
// beyond that it fills the chip's workgroup slots (a single 10 s sub-interval of
// 4096 channels is only 64 tiles) in whole rounds: see split_for.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace rfi {
namespace {

constexpr int kWidenThreads = 256;
constexpr int kMaxSplit = 64;
constexpr int64_t kTargetTileChannels = (int64_t)2048 * 64;

inline size_t up256(size_t x) { return (x + 255) / 256 * 256; }

// Largest split (sizes the scratch, for any L <= RFI_MAX_COUNT_LONG): about 2048
// workgroups of 64 channels, at most kMaxSplit beyond what exactness needs.
int max_split(int nsub, int nchan) {
  const int need = (RFI_MAX_COUNT_LONG + RFI_MAX_COUNT - 1) / RFI_MAX_COUNT;
  int64_t want = (kTargetTileChannels + (int64_t)nsub * nchan - 1) / ((int64_t)nsub * nchan);
  if (want > kMaxSplit) want = kMaxSplit;
  return need > (int)want ? need : (int)want;
}

// Chunks per sub-interval: the least cost, in quarters of a 32-sample step of a
// slot, of rounds x (steps per chunk + a workgroup's prologue and epilogue) and of
// the records, written by the sums and read by the widening pass (8 bytes a row
// against the 256 slots x 32 samples x nbeam bytes of a step's channels). A packed
// tile's step, of twice the channels or beside a second workgroup, takes 1.5 or 2
// of a whole-block one's (36 beams, rounds of 250 steps: 989 against 643 us). The
// streaming bound is reached by full rounds, not by many workgroups: 19 beams x
// 4096 channels, 3 sub-intervals of 40690 samples (192 tiles): 11 chunks (2112
// workgroups, 8.25 rounds) and a launch for the remainder 1971 us with a widening
// pass of 42 us, 4 chunks (3 rounds) 1826 and 17 us. Where several workgroups share
// a CU (up to 7 beams) one round, which all start and end together, is up to a tenth
// slower than its steps say, so four rounds or more are taken at up to a fifth of
// additional cost: 1 sub-interval of 100000 samples x 4096 channels in 8 and 32
// chunks: 2 beams 327 and 288 us, 4 beams 358 and 339, 6 beams 529 and 470.
int split_for(int L, int nsub, int nchan, int nbeam, const CcmTune* t, bool lined) {
  const int need = (L + RFI_MAX_COUNT - 1) / RFI_MAX_COUNT;
  const int most = max_split(nsub, nchan) < L / 256 ? max_split(nsub, nchan) : L / 256;
  const int rows = 1 + (nbeam + 1) / 2;       // record rows per beam
  int best = need, many = 0;                  // many: of four rounds or more
  int64_t best_cost = INT64_MAX, many_cost = INT64_MAX;
  bool one_round = false;
  for (int p = need; p <= most || p == need; ++p) {
    const int c = (L + p - 1) / p;
    CcmClass cc;                              // of this launch
    if (ccm_class(nbeam, &cc, t, (int64_t)nsub * p * nchan, c, lined) != hipSuccess) return need;
    const int64_t tiles = (int64_t)nsub * p * ((nchan + cc.cw - 1) / cc.cw);
    const int step = cc.engine != 2 ? 4 : nbeam < 32 ? 8 : 6;
    const int64_t rounds = (tiles + cc.slots - 1) / cc.slots;
    const int64_t cost = rounds * ((c + 31) / 32 + 8) * step + tiles * rows / 256;
    const bool shared_cu = cc.engine == 1 && cc.slots > 256;
    if (cost < best_cost) {
      best_cost = cost;
      best = p;
      one_round = shared_cu && rounds == 1;
    }
    if (shared_cu && tiles >= 4 * cc.slots && cost < many_cost) {
      many_cost = cost;
      many = p;
    }
  }
  return one_round && many && many_cost <= best_cost + best_cost / 5 ? many : best;
}

// rec64[cell][row] = sum over the P chunk records of that cell; count[k] = L.
// With accumulate the sums and counts are added to what the records and counts
// hold.
__global__ __launch_bounds__(kWidenThreads) void widen_kernel(const int32_t* __restrict__ rec32,
                                                              int64_t* __restrict__ rec64,
                                                              int nsub, int nchan, int nrow,
                                                              int P,
                                                              int32_t* __restrict__ count,
                                                              int L, int accumulate) {
  const int64_t per_sub = (int64_t)nchan * nrow;         // values of one sub-interval
  const int64_t n = (int64_t)nsub * per_sub;
  const int64_t i = (int64_t)blockIdx.x * kWidenThreads + threadIdx.x;
  if (count && blockIdx.x == 0)
    for (int k = threadIdx.x; k < nsub; k += kWidenThreads)
      count[k] = accumulate ? count[k] + L : L;
  if (i >= n) return;
  const int64_t k = i / per_sub, w = i % per_sub;
  const int32_t* src = rec32 + k * P * per_sub + w;
  int64_t acc = 0;
  for (int j = 0; j < P; ++j) acc += src[(int64_t)j * per_sub];
  rec64[i] = accumulate ? rec64[i] + acc : acc;
}

}  // namespace

size_t ccm_long_tmp_bytes(int nbeam, int nchan, int nsub) {
  const size_t per_sub = (size_t)nchan * (nbeam + npair_of(nbeam));
  const size_t P = (size_t)max_split(nsub, nchan);
  return up256((size_t)nsub * (P + 1) * per_sub * 4) + up256((size_t)nsub * (P + 1) * 4);
}

hipError_t launch_ccm_long(const BeamPtrs& bp, int nbeam, int nchan, int64_t row_stride,
                           int64_t t0, int L, int nsub, int64_t* rec, int32_t* count, void* tmp,
                           hipStream_t s, const CcmTune* t, int accumulate) {
  if (nsub == 0) return hipSuccess;
  const int nrow = nbeam + npair_of(nbeam);
  const int P = split_for(L, nsub, nchan, nbeam, t, ccm_lined_up(bp.p, nbeam, row_stride));
  // whole 32-sample steps per chunk where the last one still has samples
  int c = (L + P - 1) / P;
  const int c32 = (c + 31) / 32 * 32;
  if (c32 <= RFI_MAX_COUNT && (int64_t)(P - 1) * c32 < L) c = c32;
  const size_t per_sub = (size_t)nchan * nrow;
  const int Pmax = max_split(nsub, nchan);
  int32_t* rec32 = (int32_t*)tmp;
  int32_t* cnt32 = (int32_t*)((char*)tmp + up256((size_t)nsub * (Pmax + 1) * per_sub * 4));
  // every chunk of every sub-interval: launch sub-interval k P + j is chunk j
  // of sub-interval k, records [k P + j][channel][row]
  hipError_t e = launch_ccm_mfma(bp, nbeam, nchan, row_stride, t0, c, nsub * P, rec32, nullptr,
                                 cnt32, 0, 0, s, t, 1, (int64_t)L, P, L - (P - 1) * c);
  if (e != hipSuccess) return e;
  const int64_t nval = (int64_t)nsub * (int64_t)per_sub;
  const unsigned grid = (unsigned)((nval + kWidenThreads - 1) / kWidenThreads);
  hipLaunchKernelGGL(widen_kernel, dim3(grid), dim3(kWidenThreads), 0, s, rec32, rec, nsub, nchan,
                     nrow, P, count, L, accumulate);
  return hipGetLastError();
}

}  // namespace rfi
