// gfx950 kernels of the NetFlow v5 decode step and its C-ABI launcher.
//
// The paper's border routers export NetFlow V5 datagrams over UDP (48-byte
// records, at most 30 per datagram) and a receiver thread stores the records
// in a host buffer (§III.B.1, FlowData Receiver Thread; §IV.A.3).  Here the
// datagrams, as received back to back, are decoded on the GPU into the
// structure-of-arrays window that the classify path reads:
//   1. v5_count_kernel: checks every datagram's header and span, and scans
//      the record counts (0 = rejected) within blocks of 1,024 datagrams;
//   2. v5_decode_kernel: one workgroup per 32 datagrams.  It sums the block
//      totals before its own (a one-workgroup v5_scan_kernel does that first
//      for more than 2,048 blocks), reads its records as contiguous 16-byte
//      pieces into LDS, and writes each output field with full-wave
//      coalesced stores, lane i decoding record i of the tile.
// Up to 2,048 datagrams need no first kernel: every decode workgroup counts
// them all itself (12.3 us a call against 14.0 us with the count kernel at
// 1,900 datagrams, 12.5 against 14.6 at 360, with a host side of the call, most
// of both, that was 4 us longer than now: 8.5 at 351).
// The decode is bound by memory, 48 B read and 33 B written per record: 149
// to 157 us (two cards) for 10 M records, 5.2 to 5.5 TB/s, what a large copy
// reaches here.  One half-wave per datagram with each lane reading its own
// record (four 8-byte loads, 48 bytes apart) took 197 us: every load touched a
// line per lane, and the streaming loads fetched lines again.  The count kernel
// (12 us, one scattered line per datagram) replaces a count and three scan
// kernels (32 us).
// Field layout (public NetFlow version 5 export format, big-endian): header
// of 24 bytes starting with version u16 and count u16; records of 48 bytes:
// srcaddr, dstaddr, nexthop u32; input, output u16; dPkts, dOctets, First,
// Last u32; srcport, dstport u16; pad1, tcp_flags, prot, tos u8; src_as,
// dst_as u16; src_mask, dst_mask u8; pad2 u16.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "registry.h"

namespace gnm {
namespace {

typedef unsigned long long u64;

constexpr uint32_t kV5Header = 24;
constexpr uint32_t kV5Record = 48;
constexpr uint32_t kV5MaxRecords = 30;
constexpr uint32_t kThreads = 256;         // count and decode workgroups
constexpr uint32_t kCountPer = 4;          // consecutive datagrams per lane of the count kernel
constexpr uint32_t kBlock = kThreads * kCountPer;  // datagrams scanned together
constexpr uint32_t kTile = 32;             // datagrams per decode workgroup (divides kBlock)
constexpr uint32_t kTileRecords = kTile * 30;
constexpr uint32_t kPieces = 3;            // 16-byte pieces of a record
constexpr uint32_t kPieceLoads = 6;        // pieces in flight per lane
constexpr uint32_t kSmallPer = 8;          // single-launch form: datagrams per lane
constexpr uint64_t kSmall = (uint64_t)kThreads * kSmallPer;
// Block totals a decode workgroup sums itself, which saves the scan kernel's
// launch (10,000 datagrams of 30 records 13.3 us a call, 15.9 with it) until it
// reads too many: 1 M datagrams (977 blocks) 484 and 490 us, 2 M 982 and 986,
// 4.2 M (4,096 blocks) 2,270 and 2,095.  (Between 100 and 350 blocks the two are
// within 1.5 us, the scan kernel ahead.)
constexpr uint32_t kInlineBlocks = 2048;
constexpr uint32_t kScanThreads = 1024;
constexpr uint32_t kCountBits = 5;         // a scanned count: records before it in its block << 5 | records
static_assert(kV5MaxRecords < (1u << kCountBits) && kBlock % kTile == 0 && kSmall % kTile == 0, "packed counts");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(4)));  // 16-byte loads need no 16-byte alignment

struct V5Out {
  uint32_t *src, *dst;
  uint16_t *sport, *dport;  // may be NULL
  uint8_t *proto;           // may be NULL
  uint64_t *bytes;
  uint32_t *packets, *first, *last;
  uint64_t capacity;
};

__device__ __forceinline__ uint32_t be32(uint32_t x) { return __builtin_bswap32(x); }

// Records of the datagram with span [s, e): 0 (rejected) unless the span lies
// in the buffer, starts at a multiple of 4, and holds the header, version 5,
// count 1..30 and count records.  Split so that a lane's header loads are in
// flight together: the header word is only read where the span allows it.
__device__ __forceinline__ bool v5_span_ok(uint64_t s, uint64_t e, uint64_t buf_bytes) {
  return e >= s && e <= buf_bytes && e - s >= kV5Header && (s & 3u) == 0u;
}
__device__ __forceinline__ uint32_t v5_count(uint32_t head, uint64_t s, uint64_t e) {
  const uint32_t h = be32(head), version = h >> 16, count = h & 0xFFFFu;
  return version == 5u && count >= 1u && count <= kV5MaxRecords && e - s >= kV5Header + (uint64_t)kV5Record * count
             ? count
             : 0u;
}

// Record counts of the PER consecutive datagrams from d0 (0 beyond n).
template <uint32_t PER>
__device__ __forceinline__ void v5_counts(const uint8_t *buf, uint64_t buf_bytes, const uint64_t *off, uint64_t n,
                                          uint64_t d0, uint32_t (&c)[PER], uint64_t (&start)[PER]) {
  uint64_t o[PER + 1];
  uint32_t head[PER];
#pragma unroll
  for (uint32_t j = 0; j <= PER; ++j) o[j] = d0 < n ? off[d0 + j < n ? d0 + j : n] : 0u;
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j)
    head[j] = d0 + j < n && v5_span_ok(o[j], o[j + 1], buf_bytes) ? *(const uint32_t *)(buf + o[j]) : 0u;
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    c[j] = v5_count(head[j], o[j], o[j + 1]);  // header 0 is version 0: no records
    start[j] = o[j];
  }
}

__device__ __forceinline__ u64 wave_sum(u64 x) {
#pragma unroll
  for (uint32_t o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Exclusive scan of one value per lane over a workgroup of W waves; `total`
// receives the sum.  `wsum` holds W words.
template <uint32_t W>
__device__ __forceinline__ u64 block_exclusive(u64 x, u64 &total, u64 *wsum) {
  const uint32_t lane = threadIdx.x % 64u, wave = threadIdx.x / 64u;
  u64 incl = x;
#pragma unroll
  for (uint32_t o = 1; o < 64; o <<= 1) {
    const u64 y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  __syncthreads();  // earlier readers of wsum are done
  if (lane == 63u) wsum[wave] = incl;
  __syncthreads();
  u64 before = 0, t = 0;
#pragma unroll
  for (uint32_t v = 0; v < W; ++v) {
    if (v < wave) before += wsum[v];
    t += wsum[v];
  }
  total = t;
  return before + incl - x;
}

// Block b: the counts of its datagrams with the records before each in the
// block, and the block's totals (records, and rejected datagrams << 32).
__global__ __launch_bounds__(kThreads) void v5_count_kernel(const uint8_t *__restrict__ buf, uint64_t buf_bytes,
                                                            const uint64_t *__restrict__ off, uint64_t n,
                                                            uint32_t *__restrict__ cnt, u64 *__restrict__ sums) {
  __shared__ u64 wsum[kThreads / 64];
  const uint64_t d0 = (uint64_t)blockIdx.x * kBlock + kCountPer * threadIdx.x;
  uint32_t c[kCountPer];
  uint64_t start[kCountPer];
  v5_counts<kCountPer>(buf, buf_bytes, off, n, d0, c, start);
  u64 mine = 0;
#pragma unroll
  for (uint32_t j = 0; j < kCountPer; ++j)
    if (d0 + j < n) mine += (u64)c[j] + (c[j] == 0u ? 1ull << 32 : 0ull);
  u64 total;
  uint32_t run = (uint32_t)block_exclusive<kThreads / 64>(mine, total, wsum);
#pragma unroll
  for (uint32_t j = 0; j < kCountPer; ++j) {
    if (d0 + j < n) cnt[d0 + j] = (run << kCountBits) | c[j];
    run += c[j];
  }
  if (threadIdx.x == 0u) sums[blockIdx.x] = total;
}

// One workgroup: base[b] = records before block b, for more blocks than a
// decode workgroup sums itself; the totals go out.
__global__ __launch_bounds__(kScanThreads) void v5_scan_kernel(const u64 *__restrict__ sums, uint64_t G,
                                                               u64 *__restrict__ base, u64 *__restrict__ n_records,
                                                               u64 *__restrict__ n_rejected) {
  __shared__ u64 wsum[kScanThreads / 64];
  u64 running = 0, rejected = 0;
  for (uint64_t b0 = 0; b0 < G; b0 += kScanThreads) {
    const uint64_t b = b0 + threadIdx.x;
    const u64 v = b < G ? sums[b] : 0ull;
    u64 total, bad;
    const u64 before = block_exclusive<kScanThreads / 64>(v & 0xFFFFFFFFull, total, wsum);
    block_exclusive<kScanThreads / 64>(v >> 32, bad, wsum);
    if (b < G) base[b] = running + before;
    running += total;
    rejected += bad;
  }
  if (threadIdx.x == 0u) {
    *n_records = running;
    *n_rejected = rejected;
  }
}

struct DecodeArgs {
  const uint8_t *buf;
  uint64_t buf_bytes;
  const uint64_t *off;
  uint64_t n;
  const uint32_t *cnt;  // scanned counts
  const u64 *sums;      // block totals
  const u64 *base;      // records before each block (NULL: summed here from the totals)
  u64 *n_records, *n_rejected;  // written by workgroup 0 (not with `base`)
  V5Out out;
};

// Workgroup x decodes datagrams 32x .. 32x + 31: up to 960 records, 45 KB of
// LDS, so that three workgroups share a CU and a tile's loads are in flight
// while others store.  SMALL: every workgroup counts all (at most kSmall)
// datagrams itself.  Records past the capacity are dropped; the reported
// total still counts them.
template <bool SMALL>
__global__ __launch_bounds__(kThreads) void v5_decode_kernel(const DecodeArgs q) {
  __shared__ u32x4 s_rec[kTileRecords * kPieces];
  __shared__ uint8_t s_dg[kTileRecords];  // each record's datagram
  __shared__ uint64_t s_start[kTile];
  __shared__ uint32_t s_cnt[kTile], s_first[kTile];  // records; records before it in the tile
  __shared__ u64 wsum[kThreads / 64], s_base;
  const uint32_t tid = threadIdx.x;
  const uint64_t t0 = (uint64_t)blockIdx.x * kTile;
  if (SMALL) {
    const uint64_t d0 = (uint64_t)kSmallPer * tid;
    uint32_t c[kSmallPer];
    uint64_t start[kSmallPer];
    v5_counts<kSmallPer>(q.buf, q.buf_bytes, q.off, q.n, d0, c, start);
    u64 mine = 0;
#pragma unroll
    for (uint32_t j = 0; j < kSmallPer; ++j)
      if (d0 + j < q.n) mine += (u64)c[j] + (c[j] == 0u ? 1ull << 32 : 0ull);
    u64 total;
    uint32_t run = (uint32_t)block_exclusive<kThreads / 64>(mine, total, wsum);
    // the tile's 32 datagrams belong to 4 whole lanes
    if (d0 >= t0 && d0 < t0 + kTile) {
      if (d0 == t0) s_base = run;
#pragma unroll
      for (uint32_t j = 0; j < kSmallPer; ++j) {
        s_cnt[d0 - t0 + j] = c[j];
        s_first[d0 - t0 + j] = run;  // less the tile's first, below
        s_start[d0 - t0 + j] = start[j];
        run += c[j];
      }
    }
    __syncthreads();
    if (tid < kTile) s_first[tid] -= (uint32_t)s_base;
    if (blockIdx.x == 0 && tid == 0) {
      *q.n_records = total & 0xFFFFFFFFull;
      *q.n_rejected = total >> 32;
    }
  } else {
    if (tid < kTile) {
      const bool in = t0 + tid < q.n;
      const uint32_t v = in ? q.cnt[t0 + tid] : 0u, first = __shfl(v >> kCountBits, 0, 64);
      s_cnt[tid] = v & ((1u << kCountBits) - 1u);
      s_first[tid] = in ? (v >> kCountBits) - first : 0u;
      s_start[tid] = in ? q.off[t0 + tid] : 0ull;
      if (tid == 0) s_base = first;
    }
  }
  __syncthreads();
  // 8 lanes per datagram mark its records
  {
    const uint32_t d = tid / 8u, c = s_cnt[d], first = s_first[d];
    for (uint32_t k = tid % 8u; k < c; k += 8u) s_dg[first + k] = (uint8_t)d;
  }
  const uint32_t last = q.n - t0 < kTile ? (uint32_t)(q.n - t0) : kTile;  // datagrams of the tile (0: n == 0)
  const uint32_t records = last ? s_first[last - 1u] + s_cnt[last - 1u] : 0u;
  __syncthreads();
  const uint32_t pieces = kPieces * records;
  for (uint32_t p0 = 0; p0 < pieces; p0 += kPieceLoads * kThreads) {
    u32x4 v[kPieceLoads];
#pragma unroll
    for (uint32_t j = 0; j < kPieceLoads; ++j) {
      const uint32_t p = p0 + j * kThreads + tid, r = p / kPieces;
      if (p < pieces) {
        const uint32_t d = s_dg[r];
        v[j] = *(const u32x4_any *)(q.buf + s_start[d] + kV5Header + 16u * (p - kPieces * s_first[d]));
      }
    }
#pragma unroll
    for (uint32_t j = 0; j < kPieceLoads; ++j) {
      const uint32_t p = p0 + j * kThreads + tid;
      if (p < pieces) s_rec[p] = v[j];
    }
  }
  // records before the tile's block (the loads above are in flight meanwhile)
  u64 before = 0;
  if (!SMALL) {
    const uint64_t b = t0 / kBlock;
    if (q.base) {
      before = q.base[b];
    } else {
      u64 sum = 0, all = 0;
      const uint64_t G = (q.n + kBlock - 1u) / kBlock, upto = blockIdx.x == 0 ? G : b;
      for (uint64_t i = tid; i < upto; i += kThreads) {
        const u64 v = q.sums[i];
        sum += i < b ? v & 0xFFFFFFFFull : 0ull;
        all += v;  // workgroup 0: at most 2,048 blocks, so both halves fit
      }
      sum = wave_sum(sum);
      if (tid % 64u == 0u) wsum[tid / 64u] = sum;
      __syncthreads();
#pragma unroll
      for (uint32_t v = 0; v < kThreads / 64u; ++v) before += wsum[v];
      if (blockIdx.x == 0) {
        all = wave_sum(all);
        __syncthreads();
        if (tid % 64u == 0u) wsum[tid / 64u] = all;
        __syncthreads();
        if (tid == 0) {
          u64 t = 0;
          for (uint32_t v = 0; v < kThreads / 64u; ++v) t += wsum[v];
          *q.n_records = t & 0xFFFFFFFFull;
          *q.n_rejected = t >> 32;
        }
      }
    }
  }
  __syncthreads();
  const u64 out0 = before + s_base;
  const V5Out &o = q.out;
  for (uint32_t r = tid; r < records; r += kThreads) {
    const u32x4 a = s_rec[kPieces * r], e = s_rec[kPieces * r + 1u], f = s_rec[kPieces * r + 2u];
    const uint64_t i = out0 + r;
    if (i >= o.capacity) continue;
    o.src[i] = be32(a.x);
    o.dst[i] = be32(a.y);
    o.packets[i] = be32(e.x);
    o.bytes[i] = be32(e.y);
    o.first[i] = be32(e.z);
    o.last[i] = be32(e.w);
    const uint32_t ports = be32(f.x);
    if (o.sport) o.sport[i] = (uint16_t)(ports >> 16);
    if (o.dport) o.dport[i] = (uint16_t)(ports & 0xFFFFu);
    if (o.proto) o.proto[i] = (uint8_t)(f.y >> 16);  // bytes pad1, tcp_flags, prot, tos: prot is the third
  }
}

int fail(hipError_t e, const char *where) {
  set_last_error(std::string(where) + ": " + hipGetErrorString(e));
  return GNM_E_HIP;
}

uint64_t align256(uint64_t x) { return (x + 255u) & ~255ull; }

}  // namespace
}  // namespace gnm

using namespace gnm;

extern "C" uint64_t gnm_netflow_v5_workspace_bytes(uint64_t n_datagrams) {
  // scanned counts; block totals and bases (in room that also fits workspaces sized for 8-byte bases)
  return align256(n_datagrams * 4u) + align256(n_datagrams * 8u) + 2u * 1024u * 8u;
}

extern "C" int gnm_netflow_v5_decode(const uint8_t *datagrams, uint64_t buf_bytes, const uint64_t *offsets,
                                     uint64_t n_datagrams, void *workspace, uint64_t workspace_bytes,
                                     const gnm_records_out *out, uint64_t *n_records, uint64_t *n_rejected,
                                     hipStream_t stream) {
  if (!offsets || !out || !n_records || !n_rejected || !workspace) {
    set_last_error("NULL argument");
    return GNM_E_INVAL;
  }
  if (n_datagrams > 0 && !datagrams) { set_last_error("NULL datagram buffer"); return GNM_E_INVAL; }
  if ((uintptr_t)datagrams & 3u) { set_last_error("datagram buffer not 4-byte aligned"); return GNM_E_INVAL; }
  if (((uintptr_t)offsets | (uintptr_t)n_records | (uintptr_t)n_rejected) & 7u) {
    set_last_error("offsets or counters not 8-byte aligned");
    return GNM_E_INVAL;
  }
  if (n_datagrams > (1ull << 31)) { set_last_error("more than 2^31 datagrams"); return GNM_E_INVAL; }
  if (!out->src_ip || !out->dst_ip || !out->bytes || !out->packets || !out->first_ms || !out->last_ms) {
    set_last_error("NULL output field");
    return GNM_E_INVAL;
  }
  if (workspace_bytes < gnm_netflow_v5_workspace_bytes(n_datagrams) || ((uintptr_t)workspace & 255u)) {
    set_last_error("workspace too small or not 256-byte aligned");
    return GNM_E_INVAL;
  }
  const uint64_t n = n_datagrams;
  const uint64_t G = (n + kBlock - 1) / kBlock;
  DecodeArgs q{};
  q.buf = datagrams;
  q.buf_bytes = buf_bytes;
  q.off = offsets;
  q.n = n;
  q.n_records = (u64 *)n_records;
  q.n_rejected = (u64 *)n_rejected;
  q.out = V5Out{out->src_ip, out->dst_ip, out->src_port, out->dst_port, out->proto, out->bytes,
                out->packets, out->first_ms, out->last_ms, out->capacity};
  const uint64_t tiles = n ? (n + kTile - 1) / kTile : 1;
  hipError_t e;
  if (n <= kSmall) {
    hipLaunchKernelGGL(v5_decode_kernel<true>, dim3((uint32_t)tiles), dim3(kThreads), 0, stream, q);
    if ((e = hipGetLastError()) != hipSuccess) return fail(e, "decode launch");
    return GNM_OK;
  }
  uint32_t *cnt = (uint32_t *)workspace;
  u64 *sums = (u64 *)((uint8_t *)workspace + align256(n * 4u));
  q.cnt = cnt;
  q.sums = sums;
  hipLaunchKernelGGL(v5_count_kernel, dim3((uint32_t)G), dim3(kThreads), 0, stream, datagrams, buf_bytes, offsets, n,
                     cnt, sums);
  if ((e = hipGetLastError()) != hipSuccess) return fail(e, "count launch");
  if (G > kInlineBlocks) {
    q.base = sums + G;
    hipLaunchKernelGGL(v5_scan_kernel, dim3(1), dim3(kScanThreads), 0, stream, (const u64 *)sums, G, sums + G,
                       q.n_records, q.n_rejected);
    if ((e = hipGetLastError()) != hipSuccess) return fail(e, "scan launch");
  }
  hipLaunchKernelGGL(v5_decode_kernel<false>, dim3((uint32_t)tiles), dim3(kThreads), 0, stream, q);
  if ((e = hipGetLastError()) != hipSuccess) return fail(e, "decode launch");
  return GNM_OK;
}
