// Device-side BITCOS packer: the same blob bytes as bitcos_pack, computed on
// the GPU from a ternary matrix already in device memory (Sec. II-A: presence
// bitmap + sign vector compacted to the non-zeros, in row-major order).
//
//   plan:  one wave per row counts its non-zeros (and flags values outside
//          {-1, 0, 1}); one workgroup turns the counts into exclusive row
//          offsets and sums up the header.
//   pack:  a first kernel writes what is not streams (unit offsets, validated
//          scales, padding) and clears the sign dwords in which rows meet;
//          then one wave per row walks the row's 32-weight words 64 at a
//          time, writes each presence word, compacts the word's sign bits
//          (negative weights among the present ones, in order) and joins them
//          in LDS at the row offset plus a wavefront prefix of the words'
//          popcounts, from where they are stored a dword at a time; only a
//          row's first and last dwords, which its neighbours share, are ORed
//          in memory.
// Where everything goes follows from the non-zero count, so the call that
// plans and packs at once (bitcos_pack_device_noalloc) reads the count back
// only at the end: the pack kernels take it from the workspace and write
// nothing if the plan failed or the blob would not fit.
//
// Workspace layout (caller device memory, bitcos_plan_device_workspace bytes):
//   u32[0] value flag of the plan (weight outside {-1,0,1}), u32[1] value flag
//   of the pack (bad scale, or W changed between plan and pack), u64 at byte
//   8: nnz, u32[4 ..] row offsets, n + 1 entries.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../../include/bitcos.h"
#include "device_common.h"
#include "launch_common.h"
#include "plan.h"

namespace {

using namespace bitcos_dev;

constexpr int kRowsPerBlock = 4;  // one wave per row
constexpr int kScanThreads = 1024;

struct WsHeader {
  uint32_t plan_flag;
  uint32_t pack_flag;
  uint64_t nnz;
};
static_assert(sizeof(WsHeader) == 16, "workspace header is 16 bytes");

__device__ __forceinline__ uint32_t* ws_rows(void* ws) {
  return reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(ws) + sizeof(WsHeader));
}

// Presence and negative bytes of 8 weights (two dwords of int8).  A weight is
// present where its bit 0 is set and negative where its bit 7 is; `bad`
// collects where the byte is not the one those two bits name.
__device__ __forceinline__ void classify8(uint32_t v0, uint32_t v1, uint32_t& pres, uint32_t& neg, uint32_t& bad) {
  const uint32_t p0 = v0 & 0x01010101u, p1 = v1 & 0x01010101u;
  const uint32_t n0 = (v0 >> 7) & 0x01010101u, n1 = (v1 >> 7) & 0x01010101u;
  bad |= (v0 ^ (((n0 << 8) - n0) | p0)) | (v1 ^ (((n1 << 8) - n1) | p1));
  pres = __builtin_amdgcn_udot4(p1, 0x80402010u, __builtin_amdgcn_udot4(p0, 0x08040201u, 0u, false), false);
  neg = __builtin_amdgcn_udot4(n1, 0x80402010u, __builtin_amdgcn_udot4(n0, 0x08040201u, 0u, false), false);
}

// Presence / negative words of the 32 weights starting at weight 32 * word of
// row `row` (zero past the end of the row or matrix).
__device__ __forceinline__ void word_masks(rsrc_t rw, int row, int k, int word, uint32_t& pres,
                                           uint32_t& neg, uint32_t& bad) {
  const bool in = word < k / 32;
  const uint32_t off = in ? (static_cast<uint32_t>(row) * static_cast<uint32_t>(k) + 32u * word) : kOOB;
  uint32_t p[4], n[4];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const uint4 q = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rw, off + 16u * c, 0, 0));
    classify8(q.x, q.y, p[2 * c], n[2 * c], bad);
    classify8(q.z, q.w, p[2 * c + 1], n[2 * c + 1], bad);
  }
  pres = p[0] | p[1] << 8 | p[2] << 16 | p[3] << 24;
  neg = n[0] | n[1] << 8 | n[2] << 16 | n[3] << 24;
}

// A row's count; its top bit says that the row holds a bad value (k < 2^31).
constexpr uint32_t kBadRow = 0x80000000u;

__global__ void __launch_bounds__(kRowsPerBlock * kWave) count_rows_kernel(const int8_t* w, int n, int k, void* ws) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
  if (row >= n) return;  // whole wave
  const rsrc_t rw = make_rsrc(w, static_cast<uint32_t>(n) * static_cast<uint32_t>(k));
  uint32_t cnt = 0, bad = 0;
  for (int w0 = 0; w0 < k / 32; w0 += kWave) {
    uint32_t pres, neg;
    word_masks(rw, row, k, w0 + lane, pres, neg, bad);
    cnt += __builtin_popcount(pres);
  }
  const int tot = seg_sum<64>(static_cast<int>(cnt));
  const bool any_bad = __any(bad != 0u);
  if (lane == 63) ws_rows(ws)[row] = static_cast<uint32_t>(tot) | (any_bad ? kBadRow : 0u);
}

// Exclusive scan of the n row counts in place (row offsets), the total into
// row n and the whole header.  One workgroup; four rows per thread and pass
// (n k < 2^31: 32 bits hold every sum).
__global__ void __launch_bounds__(kScanThreads) scan_rows_kernel(int n, void* ws) {
  constexpr int kWaves = kScanThreads / kWave;
  __shared__ uint32_t part[kWaves];
  __shared__ uint32_t any_bad;
  uint32_t* rows = ws_rows(ws);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  if (t == 0) any_bad = 0;
  uint32_t run = 0, bad = 0;
  for (int base = 0; base < n; base += 4 * kScanThreads) {
    const int i0 = base + 4 * t;
    uint32_t c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      c[i] = i0 + i < n ? rows[i0 + i] : 0u;
      bad |= c[i] & kBadRow;
      c[i] &= ~kBadRow;
    }
    const uint32_t s = c[0] + c[1] + c[2] + c[3];
    const uint32_t incl = static_cast<uint32_t>(wave_incl_scan(static_cast<int>(s)));
    __syncthreads();  // the previous pass has read `part`
    if (lane == 63) part[wv] = incl;
    __syncthreads();
    uint32_t before = run;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
      before += i < wv ? part[i] : 0u;
      run += part[i];
    }
    uint32_t at = before + incl - s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i0 + i < n) rows[i0 + i] = at;
      at += c[i];
    }
  }
  if (bad) atomicOr(&any_bad, 1u);
  __syncthreads();
  if (t == 0) {
    WsHeader* h = static_cast<WsHeader*>(ws);
    h->plan_flag = any_bad;
    h->pack_flag = 0;
    h->nnz = run;
    rows[n] = run;
  }
}

// The sign bits `neg` of the present weights `pres` of one word, compacted in
// order: the parallel-suffix compress of Warren, "Hacker's Delight" (7-4),
// five rounds that each move the bits whose distance has that power of two.
__device__ __forceinline__ uint32_t compact_signs(uint32_t pres, uint32_t neg) {
  uint32_t x = neg & pres, m = pres;
  uint32_t mk = ~m << 1;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    uint32_t mp = mk ^ (mk << 1);
    mp ^= mp << 2;
    mp ^= mp << 4;
    mp ^= mp << 8;
    mp ^= mp << 16;
    const uint32_t mv = mp & m;
    m = (m ^ mv) | (mv >> (1 << i));
    const uint32_t t = x & mv;
    x = (x ^ t) | (t >> (1 << i));
    mk &= ~mp;
  }
  return x;
}

// What the pack kernels write to.  The sections after the signs start where
// the non-zero count puts them: `nnz`, or with from_ws the plan's in the
// workspace, and then only if the plan found no bad value and the blob fits.
struct PackTarget {
  uint8_t* dst;
  uint64_t cap;
  uint64_t off_signs;
  uint64_t nnz;
  int64_t ns;
  int n, k, unit_rows, units;
  bool from_ws;
};
struct Sections {
  uint64_t nnz, signs_end, off_offsets, off_scales, total;  // signs_end: of the stream, without its padding
  bool ok;
};
__host__ __device__ __forceinline__ uint64_t align256(uint64_t v) { return (v + 255u) & ~uint64_t(255); }
constexpr uint64_t kSignPad = 16;  // zero bytes after the sign stream
__device__ __forceinline__ Sections sections(const PackTarget& p, const void* ws) {
  Sections s;
  const WsHeader* h = static_cast<const WsHeader*>(ws);
  s.nnz = p.from_ws ? h->nnz : p.nnz;
  s.signs_end = p.off_signs + (s.nnz + 31) / 32 * 4;
  s.off_offsets = align256(s.signs_end + kSignPad);
  s.off_scales = align256(s.off_offsets + 4u * (static_cast<uint64_t>(p.units) + 1));
  s.total = align256(s.off_scales + 2u * static_cast<uint64_t>(p.ns));
  s.ok = !p.from_ws || (h->plan_flag == 0 && s.total <= p.cap);
  return s;
}

// Unit offsets, scales, zero padding, and zeros in the sign dwords that no row
// has to itself: those that hold a row's first bit (which rows may share), and
// those past the last planned row where the layout has room for more signs (a
// layout of more non-zeros than the workspace's plan).
constexpr int kSideThreads = 256;
__global__ void __launch_bounds__(kSideThreads) pack_side_kernel(const uint16_t* scales, PackTarget p, void* ws) {
  const Sections s = sections(p, ws);
  if (!s.ok) return;
  const uint32_t* rows = ws_rows(ws);
  uint32_t* signs = reinterpret_cast<uint32_t*>(p.dst + p.off_signs);
  uint32_t* offsets = reinterpret_cast<uint32_t*>(p.dst + s.off_offsets);
  uint16_t* out = reinterpret_cast<uint16_t*>(p.dst + s.off_scales);
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kSideThreads;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * kSideThreads + threadIdx.x;
  for (int64_t i = t; i <= p.n; i += stride) {
    const uint32_t at = rows[i];
    if (at <= s.nnz) signs[at >> 5] = 0;
  }
  const uint64_t sign_dwords = (s.nnz + 31) / 32;
  for (uint64_t d = (static_cast<uint64_t>(rows[p.n]) + 31) / 32 + t; d < sign_dwords; d += stride) signs[d] = 0;
  for (int64_t u = t; u <= p.units; u += stride)
    offsets[u] = rows[u * p.unit_rows < p.n ? u * p.unit_rows : p.n];
  bool bad = false;
  for (int64_t i = t; i < p.ns; i += stride) {
    const uint16_t h = scales[i];
    out[i] = h;
    bad |= (h & 0x8000u) || (h & 0x7C00u) == 0x7C00u;
  }
  if (bad) atomicOr(&static_cast<WsHeader*>(ws)->pack_flag, 1u);
  if (blockIdx.x == 0) {
    const auto clear = [&](uint64_t from, uint64_t to) {  // 2-byte steps: scales may end at an odd one
      for (uint64_t i = from + 2u * threadIdx.x; i < to; i += 2u * kSideThreads)
        *reinterpret_cast<uint16_t*>(p.dst + i) = 0;
    };
    clear(static_cast<uint64_t>(p.n) * static_cast<uint64_t>(p.k) / 8, p.off_signs);
    clear(s.signs_end, s.off_offsets);
    clear(s.off_offsets + 4u * (static_cast<uint64_t>(p.units) + 1), s.off_scales);
    clear(s.off_scales + 2u * static_cast<uint64_t>(p.ns), s.total);
  }
}

// Presence words and signs of one row per wave.  A pass's sign bits (at most
// 64 x 32, starting anywhere in a dword) are ORed together in LDS; dwords the
// row has to itself are stored, the others ORed (two atomics per row; ORing
// every word's bits into memory took 22 us of a 5120 x 5120 pack, this 10.5:
// 26 MB read and 6 MB written at 3.1 TB/s).
__global__ void __launch_bounds__(kRowsPerBlock * kWave) pack_rows_kernel(const int8_t* w, PackTarget p, void* ws) {
  __shared__ uint32_t bits[kRowsPerBlock][kWave + 1];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int row = blockIdx.x * kRowsPerBlock + wv;
  const Sections s = sections(p, ws);
  if (row >= p.n || !s.ok) return;  // whole wave
  uint32_t* bitmap = reinterpret_cast<uint32_t*>(p.dst);
  uint32_t* signs = reinterpret_cast<uint32_t*>(p.dst + p.off_signs);
  const uint32_t* rows = ws_rows(ws);
  const uint32_t start = rows[row], end = rows[row + 1];
  const rsrc_t rw = make_rsrc(w, static_cast<uint32_t>(p.n) * static_cast<uint32_t>(p.k));
  const int upr = p.k / 32;
  // The planned row range bounds every write (W changed since the plan:
  // flagged, nothing written outside the row's range).
  const bool planned = start <= end && end <= s.nnz;
  uint32_t carry = start, bad = planned ? 0u : 1u;
  uint32_t left = 0;  // the row's bits in the dword that `carry` points into
  for (int w0 = 0; w0 < upr; w0 += kWave) {
    const int word = w0 + lane;
    uint32_t pres, neg;
    word_masks(rw, row, p.k, word, pres, neg, bad);
    const uint32_t pc = static_cast<uint32_t>(__builtin_popcount(pres));
    const uint32_t incl = static_cast<uint32_t>(wave_incl_scan(static_cast<int>(pc)));
    const uint32_t pos = carry + incl - pc;
    const uint32_t base = carry >> 5;  // the pass's first dword
    carry += static_cast<uint32_t>(lane63(static_cast<int>(incl)));
    if (word < upr) bitmap[static_cast<size_t>(row) * upr + word] = pres;
    bits[wv][lane] = lane == 0 ? left : 0u;
    if (lane == 0) bits[wv][kWave] = 0;
    __builtin_amdgcn_wave_barrier();
    if (pc > 0 && planned && pos + pc <= end) {
      const uint32_t cs = compact_signs(pres, neg);
      const uint32_t d = (pos >> 5) - base, sh = pos & 31u;  // d <= 63
      atomicOr(&bits[wv][d], cs << sh);
      if (sh + pc > 32u) atomicOr(&bits[wv][d + 1], cs >> (32u - sh));
    } else if (pc > 0) {
      bad = 1;
    }
    __builtin_amdgcn_wave_barrier();
    // The dwords this pass completes; the one it ends in waits for the next.
    const uint32_t done = (carry >> 5) - base;  // <= 64
    left = bits[wv][done];
    const uint32_t at = base + static_cast<uint32_t>(lane);
    if (planned && static_cast<uint32_t>(lane) < done && (at << 5) < end) {
      const uint32_t v = bits[wv][lane];
      if ((at << 5) >= start && (at << 5) + 32u <= end)
        signs[at] = v;
      else if (v)
        atomicOr(&signs[at], v);
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (lane == 0 && planned && left && ((carry >> 5) << 5) < end) atomicOr(&signs[carry >> 5], left);
  if (lane == 63 && carry != end) bad = 1;
  if (bad) atomicOr(&static_cast<WsHeader*>(ws)->pack_flag, 1u);
}

int check_shape(int32_t n, int32_t k, int32_t group, int32_t unit_rows) {
  if (n < 1 || k < 1 || unit_rows < 0) return BITCOS_E_ARG;
  if (group != 0 && group != 128) return BITCOS_E_ARG;
  if (k % (group == 128 ? 128 : 32)) return BITCOS_E_ARG;
  if (static_cast<int64_t>(n) * k >= (int64_t(1) << 31)) return BITCOS_E_UNSUPPORTED;  // buffer ranges
  return BITCOS_OK;
}

int sync_status(hipStream_t st) {
  if (hipGetLastError() != hipSuccess) return BITCOS_E_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return BITCOS_E_HIP;
  return BITCOS_OK;
}

// Enqueues the plan: row offsets and header into the workspace.
void launch_plan(const int8_t* w, int n, int k, void* ws, hipStream_t s) {
  const unsigned blocks = static_cast<unsigned>((n + kRowsPerBlock - 1) / kRowsPerBlock);
  hipLaunchKernelGGL(count_rows_kernel, dim3(blocks), dim3(kRowsPerBlock * kWave), 0, s, w, n, k, ws);
  hipLaunchKernelGGL(scan_rows_kernel, dim3(1), dim3(kScanThreads), 0, s, n, ws);
}

// Enqueues the pack of a planned matrix into dst; L: its layout, or with
// from_ws the layout of any count (the kernels take the plan's).
void launch_pack(const int8_t* w, const uint16_t* scales, const bitcos_layout& L, void* dst, size_t cap, bool from_ws,
                 void* ws, hipStream_t s) {
  PackTarget p;
  p.dst = static_cast<uint8_t*>(dst);
  p.cap = cap;
  p.off_signs = L.sec_off[BITCOS_SEC_SIGNS];
  p.nnz = L.nnz;
  p.ns = L.group == 128 ? static_cast<int64_t>(L.n) * (L.k / 128) : 1;
  p.n = L.n;
  p.k = L.k;
  p.unit_rows = L.unit_rows;
  p.units = static_cast<int>((static_cast<int64_t>(L.n) + L.unit_rows - 1) / L.unit_rows);
  p.from_ws = from_ws;
  const int64_t most = p.ns > p.n + 1 ? p.ns : p.n + 1;
  const int64_t side = (most + kSideThreads - 1) / kSideThreads;
  hipLaunchKernelGGL(pack_side_kernel, dim3(static_cast<unsigned>(side < 1024 ? side : 1024)), dim3(kSideThreads), 0,
                     s, scales, p, ws);
  hipLaunchKernelGGL(pack_rows_kernel, dim3(static_cast<unsigned>((p.n + kRowsPerBlock - 1) / kRowsPerBlock)),
                     dim3(kRowsPerBlock * kWave), 0, s, w, p, ws);
}

// Reads the workspace header back and waits for the stream.
int read_header(WsHeader* h, const void* ws, hipStream_t s) {
  if (hipMemcpyAsync(h, ws, sizeof(*h), hipMemcpyDeviceToHost, s) != hipSuccess) return BITCOS_E_HIP;
  return sync_status(s);
}

// Workspace of bitcos_pack_device_noalloc for matrices of up to
// BITCOS_NOALLOC_MAX_ROWS rows: the header and n + 1 row offsets of the
// plan.  One copy per GPU the library runs on, held until the process ends.
constexpr size_t kNoallocBytes =
    (sizeof(WsHeader) + 4u * (static_cast<size_t>(BITCOS_NOALLOC_MAX_ROWS) + 1) + 15u) / 16u * 16u;
__device__ __align__(256) uint8_t scratch[kNoallocBytes];

constexpr int kMaxDevices = 64;

// Device address of this GPU's `scratch`, looked up once per device with
// that device current.  The host-side name of a __device__ array is not its
// device address; only this pointer may reach kernels and copies.
int noalloc_workspace(void** out) {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BITCOS_E_HIP;
  std::lock_guard<std::mutex> g(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return BITCOS_E_HIP;
    addr[dev] = p;
  }
  *out = addr[dev];
  return BITCOS_OK;
}

}  // namespace

extern "C" {

size_t bitcos_plan_device_workspace(int32_t n) {
  if (n < 1) return 0;
  return (sizeof(WsHeader) + 4u * (static_cast<size_t>(n) + 1) + 15u) / 16u * 16u;
}

int bitcos_plan_device(const int8_t* w_dev, int32_t n, int32_t k, int32_t group, int32_t unit_rows,
                       void* ws_dev, size_t ws_bytes, bitcos_layout* out, void* stream) {
  if (!w_dev || !ws_dev || !out) return BITCOS_E_ARG;
  int st = check_shape(n, k, group, unit_rows);
  if (st) return st;
  if (ws_bytes < bitcos_plan_device_workspace(n)) return BITCOS_E_SPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  launch_plan(w_dev, n, k, ws_dev, s);
  WsHeader h;
  st = read_header(&h, ws_dev, s);
  if (st) return st;
  if (h.plan_flag) return BITCOS_E_VALUE;
  return bitcos::bitcos_layout_for(n, k, group, unit_rows, h.nnz, out);
}

int bitcos_pack_device(const int8_t* w_dev, const uint16_t* scales_dev, const bitcos_layout* L,
                       void* ws_dev, size_t ws_bytes, void* dst_dev, size_t cap, void* stream) {
  if (!w_dev || !scales_dev || !L || !ws_dev || !dst_dev) return BITCOS_E_ARG;
  if (L->version != BITCOS_LAYOUT_VERSION || L->format != BITCOS_FMT_BITCOS || L->unit_rows < 1)
    return BITCOS_E_ARG;
  int st = check_shape(L->n, L->k, L->group, L->unit_rows);
  if (st) return st;
  if (ws_bytes < bitcos_plan_device_workspace(L->n)) return BITCOS_E_SPACE;
  if (cap < L->total_bytes) return BITCOS_E_SPACE;
  bitcos_layout chk;  // the layout must be the one the plan gives for its nnz
  st = bitcos::bitcos_layout_for(L->n, L->k, L->group, L->unit_rows, L->nnz, &chk);
  if (st || chk.total_bytes != L->total_bytes || chk.sec_off[BITCOS_SEC_SCALES] != L->sec_off[BITCOS_SEC_SCALES])
    return BITCOS_E_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (hipMemsetAsync(&static_cast<WsHeader*>(ws_dev)->pack_flag, 0, sizeof(uint32_t), s) != hipSuccess)
    return BITCOS_E_HIP;
  launch_pack(w_dev, scales_dev, chk, dst_dev, cap, false, ws_dev, s);
  WsHeader h;
  st = read_header(&h, ws_dev, s);
  if (st) return st;
  return h.pack_flag ? BITCOS_E_VALUE : BITCOS_OK;
}

int bitcos_pack_device_noalloc(const int8_t* w_dev, const uint16_t* scales_dev, int32_t n, int32_t k,
                               int32_t group, int32_t unit_rows, bitcos_layout* out, void* dst_dev, size_t cap,
                               void* stream) {
  if (!w_dev || !scales_dev || !out || !dst_dev) return BITCOS_E_ARG;
  int st = check_shape(n, k, group, unit_rows);
  if (st) return st;
  if (n > BITCOS_NOALLOC_MAX_ROWS) return BITCOS_E_SPACE;  // more rows than the fixed workspace holds
  void* ws = nullptr;
  st = noalloc_workspace(&ws);
  if (st) return st;
  // The sections' places for any count but the sign stream's length: the
  // kernels work out the rest from the count in the workspace.
  bitcos_layout base;
  st = bitcos::bitcos_layout_for(n, k, group, unit_rows, 0, &base);
  if (st) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  launch_plan(w_dev, n, k, ws, s);
  launch_pack(w_dev, scales_dev, base, dst_dev, cap, true, ws, s);
  WsHeader h;
  st = read_header(&h, ws, s);
  if (st) return st;
  if (h.plan_flag) return BITCOS_E_VALUE;
  st = bitcos::bitcos_layout_for(n, k, group, unit_rows, h.nnz, out);
  if (st) return st;
  if (cap < out->total_bytes) return BITCOS_E_SPACE;  // *out tells the caller the size
  return h.pack_flag ? BITCOS_E_VALUE : BITCOS_OK;
}

}  // extern "C"
