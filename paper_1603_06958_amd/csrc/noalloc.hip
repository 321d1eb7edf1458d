// famsa_lcs_family_noalloc: the LCS of every pair of one family, from device
// inputs into a device output, with no allocation of any kind.
//
// The plan path (famsa_lcs_plan / famsa_lcs_tiles) allocates its device
// batch, work lists, queue counters and step buffers, and plans the work on
// the host.  Here every one of those lives in `scratch`, one file-scope
// device array of fixed size per GPU, and the planning runs on the device:
//   na_prep_kernel   -- the first workgroup plans: lengths and offsets
//                       checked, rows sorted by length (counting sort), the
//                       family mode work lists of the plan path (64-row
//                       groups, column items); the others stage sequences,
//                       four at a time, once they have found every length and
//                       offset of the family valid: codes checked, the column
//                       stream (code c stored as c * 1024) and the match masks
//                       PM[c][w] written into the sequence's slot;
//   lcs_small_kernel -- families of few items: every class in one launch; or
//   lcs_fast_kernel  -- the plan path's own kernels, classes 2, 1, 0, and
//   na_finish_kernel -- the status; every output set to -1 on invalid input
//                       (the last launch does this, whichever it is).
// Results are the plan path's bit for bit (same kernels, same recurrence).
// A call of 48 sequences takes 38 us (90 us when the sort was bitonic, staging
// waited for the plan, and every class had a launch of a full grid), one of
// 8,192 sequences of 300 residues 6.0 ms (7.2 ms; the LCS kernel is 5.9).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "noalloc_input.h"
#include "runtime.h"

namespace famsa {
namespace {

constexpr uint32_t kNaMaxSeq = FAMSA_LCS_NOALLOC_MAX_SEQ;
constexpr uint32_t kNaMaxGroups = kNaMaxSeq / kLanes;
constexpr uint32_t kNaMaxItems = 8192;
constexpr uint32_t kNaMaxLen20 = FAMSA_LCS_NOALLOC_MAX_LEN;      // 28 dwords: the fast classes for sigma <= 20
constexpr uint32_t kNaMaxLen32 = FAMSA_LCS_NOALLOC_MAX_LEN_S32;  // 16 dwords: class 2 holds 4 quads of 32 planes
constexpr uint32_t kNaSymSlot = 2 * kNaMaxLen20 + 16;  // bytes: uint16 per residue and the spare chunk
constexpr uint32_t kNaMaskSlot = 20 * 28;               // dwords: >= 20 x 28 and >= 32 x 16
constexpr int kNaMaxDevices = 64;
constexpr uint32_t kNaThreads = 1024;
constexpr uint32_t kNaTeam = 256;  // threads that stage a sequence
constexpr uint32_t kNaStageBlocks = 512;  // at most so many workgroups stage: each reads all offsets first (64 KB at most)

constexpr size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr size_t kOffCtl = 0;    // StepCtl
constexpr size_t kOffCheck = 64;   // InputCheck
constexpr size_t kOffRange = 128;  // StepRange of the one step
constexpr size_t kOffGroups = 256;
constexpr size_t kOffLanes = align256(kOffGroups + sizeof(GroupDesc) * kNaMaxGroups);
constexpr size_t kOffItems = align256(kOffLanes + sizeof(LaneDesc) * kNaMaxSeq);
constexpr size_t kOffColmap = align256(kOffItems + sizeof(ItemDesc) * kNaMaxItems);
constexpr size_t kOffRowbase = align256(kOffColmap + sizeof(uint32_t) * kNaMaxSeq);
constexpr size_t kOffLen = align256(kOffRowbase + sizeof(uint64_t) * kNaMaxSeq);
constexpr size_t kOffSymOff = align256(kOffLen + sizeof(uint32_t) * kNaMaxSeq);
constexpr size_t kOffMaskOff = align256(kOffSymOff + sizeof(uint64_t) * kNaMaxSeq);
constexpr size_t kOffSym = align256(kOffMaskOff + sizeof(uint64_t) * kNaMaxSeq);
constexpr size_t kOffMasks = align256(kOffSym + (size_t)kNaSymSlot * kNaMaxSeq);
constexpr size_t kNaBytes = align256(kOffMasks + sizeof(uint32_t) * kNaMaskSlot * kNaMaxSeq);
static_assert(kNaBytes == FAMSA_LCS_NOALLOC_SCRATCH_BYTES, "header states the scratch size");
static_assert(kNaSymSlot % 16 == 0, "column streams are read in 16-byte chunks");
static_assert(sizeof(StepCtl) <= 64 && sizeof(InputCheck) <= 64 && sizeof(StepRange) <= 128, "control block layout");

// Each GPU holds its own copy.  Host code never passes this name to a kernel:
// it takes the device address from hipGetSymbolAddress.
static __device__ __align__(256) uint8_t scratch[kNaBytes];

struct NaView {  // device addresses inside one GPU's scratch
  uint8_t* base;
  StepCtl* ctl() const { return reinterpret_cast<StepCtl*>(base + kOffCtl); }
  StepRange* range() const { return reinterpret_cast<StepRange*>(base + kOffRange); }
};

__host__ __device__ inline InputCheck* na_check(uint8_t* base) { return reinterpret_cast<InputCheck*>(base + kOffCheck); }

struct NaResident {  // workgroups of each class that the GPU holds
  uint32_t c0, c1, c2;
};

// The plan, by one workgroup.  Rows sorted longest first by a counting sort
// (rows of one length in any order: their values do not depend on it); groups
// of 64 consecutive sorted rows; column position q is sequence colmap[q], and
// a pair lands in the upper-triangle row of its smaller index.
// SMALL: every class goes in one launch.
template <bool SMALL>
__device__ void na_plan(const uint64_t* __restrict__ seq_off, uint32_t k, uint32_t maxlen, NaResident resident,
                        uint8_t* __restrict__ base) {
  __shared__ uint32_t s_at[1024];  // rows longer than L, then the next place of a row of length L (at 1023 - L)
  __shared__ uint32_t s_wave[16];
  __shared__ uint16_t s_row[kNaMaxSeq], s_len[kNaMaxSeq];
  __shared__ uint32_t s_first[kNaMaxGroups + 1], s_cols[kNaMaxGroups];
  __shared__ uint32_t s_err, s_cnt[3];
  __shared__ uint64_t s_span[2];  // the family's first and last offset
  uint32_t* len = reinterpret_cast<uint32_t*>(base + kOffLen);
  uint64_t* sym_off = reinterpret_cast<uint64_t*>(base + kOffSymOff);
  uint64_t* mask_off = reinterpret_cast<uint64_t*>(base + kOffMaskOff);
  uint32_t* colmap = reinterpret_cast<uint32_t*>(base + kOffColmap);
  uint64_t* rowbase = reinterpret_cast<uint64_t*>(base + kOffRowbase);
  LaneDesc* lanes = reinterpret_cast<LaneDesc*>(base + kOffLanes);
  GroupDesc* groups = reinterpret_cast<GroupDesc*>(base + kOffGroups);
  ItemDesc* items = reinterpret_cast<ItemDesc*>(base + kOffItems);
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  if (tid < 3) s_cnt[tid] = 0;
  if (tid == 3) s_err = 0;
  s_at[tid] = 0;
  __syncthreads();
  for (uint32_t i = tid; i < k; i += kNaThreads) {
    const uint64_t a = seq_off[i], b = seq_off[i + 1];
    uint32_t L = 0;
    if (b < a || b - a > maxlen) atomicOr(&s_err, 1u);
    else L = (uint32_t)(b - a);
    len[i] = L;
    sym_off[i] = (uint64_t)i * kNaSymSlot;
    mask_off[i] = (uint64_t)i * kNaMaskSlot;
    s_len[i] = (uint16_t)L;
    if (i == 0) s_span[0] = a;
    if (i == k - 1) s_span[1] = b;
    atomicAdd(&s_at[1023u - L], 1u);  // L <= 896
  }
  __syncthreads();
  {  // exclusive prefix over the lengths, longest first
    const uint32_t n = s_at[tid];
    uint32_t sum = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(sum, d, 64);
      if (lane >= (uint32_t)d) sum += y;
    }
    if (lane == 63) s_wave[wave] = sum;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < wave; ++w) before += s_wave[w];
    s_at[tid] = before + sum - n;
  }
  __syncthreads();
  for (uint32_t i = tid; i < k; i += kNaThreads) s_row[atomicAdd(&s_at[1023u - s_len[i]], 1u)] = (uint16_t)i;
  __syncthreads();
  for (uint32_t q = tid; q < k; q += kNaThreads) {
    const uint32_t a = s_row[q];
    const uint64_t ro = (uint64_t)a * k - (uint64_t)a * (a + 1) / 2;  // offset of pair (a, a + 1)
    colmap[q] = a;
    rowbase[q] = ro;
    LaneDesc d;
    d.out_off = ro;
    d.seq = a;
    d.pos = q;
    d.orig = a;
    d.pad = 0;
    lanes[q] = d;
  }
  const uint32_t G = na_groups(k);
  if (wave < 2) {  // a lane a group; items numbered by a prefix sum
    const uint32_t g = tid;
    uint32_t ni = 0, W = 1, cols = 1;
    int cls = 0;
    if (g < G) {
      W = max(1u, (s_len[s_row[kLanes * g]] + 31u) >> 5);  // dwords of the group's longest row
      const uint32_t Q = (W + 3u) >> 2;
      cls = Q <= (uint32_t)kClassQMax[0] ? 0 : (Q <= (uint32_t)kClassQMax[1] ? 1 : 2);
      const uint32_t held = cls == 0 ? resident.c0 : (cls == 1 ? resident.c1 : resident.c2);
      cols = na_cols(k, g, SMALL ? na_runs_small() : na_runs(k, s_span[1] - s_span[0], held));
      ni = na_items(k, g, cols);
      s_cols[g] = cols;
    }
    uint32_t sum = ni;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(sum, d, 64);
      if (lane >= (uint32_t)d) sum += y;
    }
    if (lane == 63) s_wave[wave] = sum;
    s_first[g] = sum - ni;  // within its wave
    if (g < G) {
      const uint32_t P = kLanes * g;
      GroupDesc gd;
      gd.lane_first = P;
      gd.nrows = min((uint32_t)kLanes, k - P);
      gd.W = W;
      gd.fam_base = 0;
      gd.colmap_base = 0;
      gd.rowbase_base = 0;
      gd.nmap = k;
      gd.shift = 0;
      gd.lpr = 0;
      gd.pad[0] = gd.pad[1] = gd.pad[2] = 0;
      groups[g] = gd;
      atomicAdd(&s_cnt[cls], ni);  // classes do not increase with g: rows are sorted longest first
    }
  }
  __syncthreads();
  for (uint32_t g = wave; g < G; g += kNaThreads / 64) {
    const uint32_t f = s_first[g] + (g >= 64 ? s_wave[0] : 0u), C = s_cols[g], ni = na_items(k, g, C);
    for (uint32_t t = lane; t < ni; t += 64) {
      ItemDesc it;
      it.group = g;
      it.c0 = kLanes * g + 1 + t * C;
      it.c1 = min(k, it.c0 + C);
      it.pad = 0;
      items[f + t] = it;
    }
  }
  if (tid == 0) {
    const uint32_t n2 = s_cnt[2], n1 = s_cnt[1], n = n2 + n1 + s_cnt[0];
    const uint32_t ends[5] = {s_err ? 0u : n, s_err ? 0u : n2 + n1, s_err ? 0u : n2, 0u, 0u};  // items: class 2, 1, 0
    StepRange* r = reinterpret_cast<StepRange*>(base + kOffRange);
    for (int c = 0; c < 5; ++c) {
      r->begin[c] = c < 2 ? ends[c + 1] : 0u;
      r->end[c] = ends[c];
    }
    r->plain_pairs = 0;
    StepCtl* ctl = reinterpret_cast<StepCtl*>(base + kOffCtl);
    ctl->step = 0;
    ctl->next_step = 0;
    ctl->stride = 0;
    ctl->pad = 0;
    for (int c = 0; c < 4; ++c) ctl->cursor[c] = 0;
    na_check(base)->lengths = s_err;
    na_check(base)->begun = na_check(base)->ended + 1;
  }
}

// A sequence's column stream and match masks (bit p of PM[c][w] set iff
// residue 32 w + p equals c; zero past the end), by `kNaTeam` threads: a wave
// takes 64 residues, and one ballot a code is two mask words.  A thread a word
// compared its 32 residues with every code: 40 us for 8,192 sequences of 300.
// A code outside the alphabet is marked and staged as code 0, so that the LCS
// kernels stay within their tables whatever the input.  [a, b): the sequence in
// `codes`; the caller has found every offset of the family valid.
__device__ void na_stage(const uint8_t* __restrict__ codes, uint64_t a, uint64_t b, uint32_t s, uint32_t sigma,
                         uint8_t* __restrict__ base) {
  const uint32_t L = (uint32_t)(b - a), W = (L + 31u) >> 5, lane = threadIdx.x & 63u;
  const uint32_t w0 = (threadIdx.x & (kNaTeam - 1u)) >> 6;
  const uint8_t* src = codes + a;
  uint16_t* sym = reinterpret_cast<uint16_t*>(base + kOffSym + (size_t)s * kNaSymSlot);
  uint32_t* m = reinterpret_cast<uint32_t*>(base + kOffMasks) + (size_t)s * kNaMaskSlot;
  for (uint32_t p0 = 64 * w0; p0 < L; p0 += 64 * (kNaTeam / 64)) {
    const uint32_t p = p0 + lane;
    uint32_t c = p < L ? (uint32_t)src[p] : 0xFFu;
    if (p < L && c >= sigma) {
      atomicOr(&na_check(base)->bad[na_check(base)->ended & 1u], 1u);
      c = 0;
    }
    if (p < L) sym[p] = (uint16_t)(c * 1024u);
    uint64_t mine = 0;  // lane c: the residues that equal code c
    for (uint32_t x = 0; x < sigma; ++x) {
      const uint64_t eq = __ballot(c == x);
      mine = lane == x ? eq : mine;
    }
    const uint32_t w = p0 >> 5;
    if (lane < sigma) {
      m[(size_t)lane * W + w] = (uint32_t)mine;
      if (w + 1 < W) m[(size_t)lane * W + w + 1] = (uint32_t)(mine >> 32);
    }
  }
}

template <bool SMALL>
__global__ __launch_bounds__(kNaThreads) void na_prep_kernel(const uint8_t* __restrict__ codes,
                                                             const uint64_t* __restrict__ seq_off, uint32_t k,
                                                             uint32_t sigma, uint32_t maxlen, NaResident resident,
                                                             uint8_t* __restrict__ base) {
  if (blockIdx.x == 0) {
    na_plan<SMALL>(seq_off, k, maxlen, resident, base);
    return;
  }
  constexpr uint32_t per = kNaThreads / kNaTeam;
  uint32_t s = (blockIdx.x - 1) * per + threadIdx.x / kNaTeam;
  uint64_t a = seq_off[min(s, k)], b = seq_off[min(s + 1, k)];  // the first sequence's, with the check's loads
  // no residue is read before the whole family's offsets are known to be valid: a sequence after an invalid one
  // may lie outside the caller's codes
  if (!__syncthreads_and(na_share_valid(seq_off, k, maxlen, threadIdx.x, kNaThreads))) return;
  while (s < k) {
    na_stage(codes, a, b, s, sigma, base);
    s += (gridDim.x - 1) * per;
    if (s < k) {
      a = seq_off[s];
      b = seq_off[s + 1];
    }
  }
}

__global__ __launch_bounds__(256) void na_finish_kernel(uint8_t* __restrict__ base, int32_t* __restrict__ out,
                                                        uint64_t npairs, int32_t* __restrict__ status) {
  const uint32_t fail = na_check(base)->failed();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (status) *status = fail ? FAMSA_LCS_EINVAL : FAMSA_LCS_OK;
    na_check(base)->end();
  }
  if (!fail) return;
  const uint64_t n = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < npairs; p += n) out[p] = -1;
}

// Per device: the scratch address and the fast kernels' launch shapes.
struct NaDevice {
  uint8_t* ptr = nullptr;
  int cus = 0;
  uint32_t blocks[2][3] = {};  // [sigma <= 20, sigma <= 32][class]: workgroups per launch
  uint32_t waves[2][3] = {};
  bool ready = false;
};
std::mutex g_na_mu;
NaDevice g_na[kNaMaxDevices];

uint32_t na_qcap(int sig32, int cls) { return (sig32 && cls == 2) ? 4u : (uint32_t)kClassQMax[cls]; }

// Once per device, with that device current.
int na_setup(int device, NaDevice** out) {
  std::lock_guard<std::mutex> lock(g_na_mu);
  NaDevice& d = g_na[device];
  if (!d.ready) {
    void* p = nullptr;
    FAMSA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    int cus = 0, lds = 0;
    FAMSA_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device));
    FAMSA_HIP(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device));
    if (lds > 0) g_max_lds = std::min<size_t>(kMaxLds, (size_t)lds);
    const LaunchParams lp;
    for (int s = 0; s < 2; ++s) {
      const uint32_t sigma = s ? 32u : 20u;
      for (int c = 0; c < 3; ++c) {
        uint32_t waves = lp.waves[c];
        int n = 0;
        int e = fast_prepare(c, sigma, na_qcap(s, c), waves, &n);
        while (e == 0 && n == 0 && waves > 1) {
          waves /= 2;
          e = fast_prepare(c, sigma, na_qcap(s, c), waves, &n);
        }
        if (e || n == 0)
          return set_error(FAMSA_LCS_EDEVICE, "fast kernel %d setup for sigma %u failed", c, sigma);
        d.blocks[s][c] = (uint32_t)n * (uint32_t)cus;
        d.waves[s][c] = waves;
      }
      const int e = small_prepare(sigma, na_qcap(s, 2));
      if (e) return set_error(FAMSA_LCS_EDEVICE, "small-step kernel setup for sigma %u failed", sigma);
    }
    d.ptr = static_cast<uint8_t*>(p);
    d.cus = cus;
    d.ready = true;
  }
  *out = &d;
  return 0;
}

int na_run(const uint8_t* codes, const uint64_t* seq_off, uint32_t nseq, uint32_t sigma, int32_t* out,
           int32_t* status, int device, hipStream_t st) {
  NaDevice* d = nullptr;
  int rc = na_setup(device, &d);
  if (rc) return rc;
  uint8_t* base = d->ptr;
  const int s32 = sig_cap(sigma) == 32 ? 1 : 0;
  const uint32_t maxlen = s32 ? kNaMaxLen32 : kNaMaxLen20;
  const uint64_t npairs = (uint64_t)nseq * (nseq ? nseq - 1 : 0) / 2;
  uint32_t n = na_all_items(nseq, na_runs_small());
  const bool small = n <= 2u * (uint32_t)d->cus;  // as the plan path's small steps; the widest group is not known here
  if (!small) n = na_all_items(nseq, na_runs_most());
  if (n > kNaMaxItems) return set_error(FAMSA_LCS_EINVAL, "%u work items", n);  // never: 7,816 at most
  const uint32_t per = kNaThreads / kNaTeam, stage = std::min((nseq + per - 1) / per, kNaStageBlocks);
  const NaResident resident{d->blocks[s32][0], d->blocks[s32][1], d->blocks[s32][2]};
  auto prep = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(1 + stage), dim3(kNaThreads), 0, st, codes, seq_off, nseq, sigma, maxlen, resident,
                       base);
  };
  if (small) prep(na_prep_kernel<true>);
  else prep(na_prep_kernel<false>);
  FAMSA_HIP(hipGetLastError());
  // A launch after this one that fails: the call is still ended on the device, so that what it found of its input
  // is not taken for the next call's.
  auto failed = [&](const char* kernel, int e) {
    hipLaunchKernelGGL(na_finish_kernel, dim3(1), dim3(256), 0, st, base, out, (uint64_t)0, (int32_t*)nullptr);
    (void)hipGetLastError();
    return set_error(FAMSA_LCS_EDEVICE, "%s launch failed: %s", kernel, hipGetErrorString((hipError_t)e));
  };
  if (npairs) {
    DeviceBatch b{};
    b.sym = base + kOffSym;
    b.sym_off = reinterpret_cast<const uint64_t*>(base + kOffSymOff);
    b.len = reinterpret_cast<const uint32_t*>(base + kOffLen);
    b.mask_off = reinterpret_cast<const uint64_t*>(base + kOffMaskOff);
    b.masks = reinterpret_cast<const uint32_t*>(base + kOffMasks);
    b.values = FAMSA_LCS_VALUES_LCS;
    DeviceWork w{};
    w.groups = reinterpret_cast<const GroupDesc*>(base + kOffGroups);
    w.lanes = reinterpret_cast<const LaneDesc*>(base + kOffLanes);
    w.items = reinterpret_cast<const ItemDesc*>(base + kOffItems);
    w.colmap = reinterpret_cast<const uint32_t*>(base + kOffColmap);
    w.rowbase = reinterpret_cast<const uint64_t*>(base + kOffRowbase);
    w.ranges = reinterpret_cast<const StepRange*>(base + kOffRange);
    StepCtl* ctl = reinterpret_cast<StepCtl*>(base + kOffCtl);
    if (small) {
      const int e = launch_small(b, w, ctl, out, sigma, na_qcap(s32, 2), std::min(n, (uint32_t)d->cus),
                                 std::min(16u, na_cols(nseq, 0, na_runs_small())), na_check(base), status, npairs, st);
      return e ? failed("lcs_small", e) : 0;
    }
    for (int c = 2; c >= 0; --c) {  // heaviest class first; a class with no items returns at once
      const int e = launch_fast(c, b, w, ctl, out, sigma, na_qcap(s32, c), std::min(n, d->blocks[s32][c]),
                                d->waves[s32][c], st);
      if (e) return failed("lcs_fast", e);
    }
  }
  hipLaunchKernelGGL(na_finish_kernel, dim3(npairs ? 256 : 1), dim3(256), 0, st, base, out, npairs, status);
  FAMSA_HIP(hipGetLastError());
  return 0;
}

}  // namespace
}  // namespace famsa

extern "C" int famsa_lcs_family_noalloc(const uint8_t* codes, const uint64_t* seq_off, uint32_t nseq,
                                        uint32_t alphabet_size, int32_t* out, int32_t* status, int device,
                                        void* stream) {
  using namespace famsa;
  if (alphabet_size < 1 || alphabet_size > FAMSA_LCS_MAX_ALPHABET)
    return set_error(FAMSA_LCS_EINVAL, "alphabet_size %u not in [1, %u]", alphabet_size, FAMSA_LCS_MAX_ALPHABET);
  if (nseq > kNaMaxSeq)
    return set_error(FAMSA_LCS_EINVAL, "nseq %u exceeds the static scratch limit of %u sequences", nseq, kNaMaxSeq);
  if (!seq_off) return set_error(FAMSA_LCS_EINVAL, "seq_off is NULL");
  if (nseq && !codes) return set_error(FAMSA_LCS_EINVAL, "codes is NULL");
  if (nseq >= 2 && !out) return set_error(FAMSA_LCS_EINVAL, "out is NULL");
  if (device < 0 || device >= kNaMaxDevices) return set_error(FAMSA_LCS_EINVAL, "device %d out of range", device);
  int ndev = 0;
  FAMSA_HIP(hipGetDeviceCount(&ndev));
  if (device >= ndev) return set_error(FAMSA_LCS_EINVAL, "device %d of %d", device, ndev);
  int cur = 0;
  FAMSA_HIP(hipGetDevice(&cur));
  FAMSA_HIP(hipSetDevice(device));
  const int rc = na_run(codes, seq_off, nseq, alphabet_size, out, status, device, (hipStream_t)stream);
  FAMSA_HIP(hipSetDevice(cur));
  return rc;
}
