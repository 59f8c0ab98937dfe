// HIP kernels of libflowpool for gfx950 (CDNA4).
//
// k_pack  : the consumer's translate-gather-pack of one microbatch
//           (paper Sec. 3.1 / Sec. 3.2): per row, its run (a stretch of one
//           sample's text rows or image rows, listed by the host in row
//           order); for image rows the GVA page walk through the page table;
//           then 16-byte vector copies of every row from its page or
//           embedding-table row into the packed output; cu_seqlens as a
//           wave-wide prefix sum of the sample lengths, and position ids.
// k_write : the producer's write of one sample's image rows into its pages,
//           through the same page table (Sec. 3.2, producer side), the upload
//           of its metadata and publication of its descriptor.
// k_migrate: the copy of a migration's pages between the tiers and the upload
//           of the samples' new page lists (Sec. 3.2).
// k_cost  : per-sample cost K*l + l^2 for the planner (Sec. 3.4).
//
// Nothing here is a dense contraction, so there is no MFMA: the pack is a
// bandwidth-bound gather whose cost is HBM bytes.

#include "fp_internal.h"

#include <algorithm>
#include <cstring>

namespace fp {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// Global-address-space views: loads through them compile to global_load
// (vector memory counter only) instead of flat loads, which also count
// against the LDS counter and force the compiler to wait for each one.
typedef __attribute__((address_space(1))) const u32x4 g_u32x4_c;
typedef __attribute__((address_space(1))) u32x4 g_u32x4;

__device__ __forceinline__ u32x4 load16(const uint8_t* p) {
  return __builtin_nontemporal_load((g_u32x4_c*)p);
}

// Embedding-table rows are read at random ids, a few KiB each, and may be
// read again by later packs: plain loads let the memory-side cache keep
// them (see kTablePlainLoads), while rows read in page order are about 2 %
// faster non-temporal. The policy is an instruction bit, so the pack picks
// it per chunk.
__device__ __forceinline__ u32x4 load16_table(const uint8_t* p) {
  return *(g_u32x4_c*)p;
}

// Stores carry the nt and sc1 cache-policy bits of the gfx950 global store:
// on the pack this measured about 1.5 % faster than nt alone. The
// compiler has no builtin for that bit combination, hence the asm; it has
// no outputs, so the compiler still waits for the loaded data it stores.
// The compiler does not see inside the asm, so the asm carries the wait that
// gfx940-class parts need between a store of more than 8 bytes and a VALU
// write to its data registers (two wait states): without it the compiler
// may reuse those registers right after the store and corrupt its data.
__device__ __forceinline__ void store16(uint8_t* p, u32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}

// Reads through constant-address-space views of uniform addresses compile to
// scalar loads (scalar cache), which do not queue behind the vector memory
// traffic of the copies; the per-lane path reads through global views.
// Loads for the two ways rows are resolved: kScalar (one row per wave,
// wave-uniform addresses) or per lane.
template <bool kScalar, typename T>
__device__ __forceinline__ T ld(const void* p) {
  if constexpr (kScalar) {
    return *(const __attribute__((address_space(4))) T*)p;
  } else {
    return *(const __attribute__((address_space(1))) T*)p;
  }
}

// The pack's leading kernel arguments: everything a wave needs to address its
// row's bucket run and bucket-index entry. They are separate scalar arguments, ahead of PackArgs,
// so that the hardware preloads them into scalar registers at wave launch
// (kernarg preloading); the first loads of the row lookup then leave at once,
// alongside the kernel-argument loads of the rest.
struct PackHead {
  int32_t g0, g1, t1, t2;   // chunk geometry (as in PackPlan)
  uint64_t div_mul;         // e / (row_bytes / 16) == (e * div_mul) >> div_shift
  int32_t div_shift;
  int32_t bucket_shift;
  const uint8_t* tb;        // run table: staged copy, or null = the one in PackArgs
  int32_t off_brun;         // byte offsets of the bucket runs and the bucket index in the run table
  int32_t off_bucket;
  int32_t total;            // vectors of the microbatch
};

// A run index: bucket size and where its bucket runs and bucket entries sit
// in the run table.
struct RunIndex {
  int32_t shift, off_brun, off_bucket;
};

// e / (row_bytes / 16) as a multiply and a shift (host-computed constants).
__device__ __forceinline__ int div_vpr(const PackHead& h, int e) {
  return (int)(((uint64_t)(uint32_t)e * h.div_mul) >> h.div_shift);
}

// One run, as a single 16-byte load.
template <bool kScalar>
__device__ __forceinline__ PackRun ld_run(const PackRun* rp) {
  const u32x4 d = ld<kScalar, u32x4>(rp);
  return PackRun{(int32_t)d.x, (int32_t)d.y, (int32_t)d.z, (int32_t)d.w};
}

// The first two loads of a row's lookup, independent of each other: its
// bucket's run (the run holding the bucket's first row) and the word of the
// bucket index that holds that run's number.
struct BucketHit {
  PackRun r;
  uint32_t w;
};

template <bool kScalar>
__device__ __forceinline__ BucketHit bucket_of(const RunIndex& x, const uint8_t* tb, int row) {
  const int b = row >> x.shift;
  return BucketHit{ld_run<kScalar>(reinterpret_cast<const PackRun*>(tb + x.off_brun) + b),
                   ld<kScalar, uint32_t>(tb + x.off_bucket + 4 * (b >> 1))};
}

// Run holding row `row`: its bucket's run, or a later one, stepped to from
// that run's number when the bucket's run ends at or before the row.
template <bool kScalar>
__device__ __forceinline__ PackRun run_of(const RunIndex& x, int32_t off_runs, const uint8_t* tb, int row,
                                          const BucketHit& hit, int* s_out = nullptr) {
  PackRun r = hit.r;
  if (r.end <= row || s_out) {
    const int b = row >> x.shift;
    int s = (int)((b & 1) ? (hit.w >> 16) : (hit.w & 0xffffu));
    const PackRun* runs = reinterpret_cast<const PackRun*>(tb + off_runs);
    while (r.end <= row) r = ld_run<kScalar>(runs + ++s);
    if (s_out) *s_out = s;
  }
  return r;
}

// Row of physical memory holding visual row `vidx` of an image run: visual
// index -> page GVA -> page-table entry (the GVA's page number) -> row in the
// physical page. `word` >= 0: the sample's page GVAs start at 64-bit word
// `word` of the arena (the page list). `word` < 0: the sample's pages have
// consecutive GVAs, page lp's GVA is page 0's plus lp pages, and -word - 1 is
// page 0's page number, so the page number needs no load. Returns the
// page-table entry's flags in *flags.
template <bool kScalar, class Args>
__device__ __forceinline__ uint64_t walk(const Args& a, int32_t word, uint32_t vidx, uint64_t* flags) {
  const int lp = (int)(((uint64_t)vidx * a.pt_mul) >> a.pt_shift);
  const int in_page = (int)vidx - lp * a.page_tokens;
  uint64_t vpn;
  if (word < 0) {
    vpn = (uint64_t)(-(int64_t)word - 1) + (uint64_t)lp;
  } else {
    const uint64_t gva = ld<kScalar, uint64_t>(a.meta + 8 * ((int64_t)word + lp));
    vpn = __umul64hi(gva - a.gva_start, a.pb_mul) >> a.pb_shift;
  }
  const uint64_t pte = ld<kScalar, uint64_t>(a.pte + vpn);
  *flags = pte;
  return (pte & PTE_ADDR_MASK) + (uint64_t)in_page * (uint64_t)a.row_bytes;
}

template <class Args>
__device__ __forceinline__ uint64_t text_row(const Args& a, int32_t id) {
  return reinterpret_cast<uint64_t>(a.table) + (uint64_t)(uint32_t)id * (uint64_t)a.row_bytes;
}

// Source address of packed row `row` of run r, or 0 when the tier mask
// leaves the row out. A text row's id selects an embedding-table row; an
// image row walks the page table.
template <bool kScalar, class Args>
__device__ __forceinline__ uint64_t row_source(const Args& a, const PackRun& run, int row) {
  if (run.head < 0) {
    if (!(a.tier_mask & 1)) return 0;
    return text_row(a, ld<kScalar, int32_t>(a.meta + 4 * ((int64_t)run.word + row)));
  }
  uint64_t flags = 0;
  const uint64_t src = walk<kScalar>(a, run.word, (uint32_t)(row + run.vdelta), &flags);
  if (!(a.tier_mask & ((flags & PTE_HOST) ? 2 : 1))) return 0;
  return src;
}

// Moves a thread's first N vectors of a chunk: vector u comes from from[u] and
// goes to vector v0 + u * kPackBlock + tid of the output. kWhole: every
// vector is live, so there is no predication and the compiler keeps all
// loads in flight and waits for them one at a time before each store;
// otherwise only live vectors are loaded and stored. kTable: the chunk holds
// embedding-table rows and takes plain loads, else non-temporal ones. The
// two load forms differ only in a cache-policy bit, which the compiler drops
// when it merges otherwise identical code of two branches into one; the
// table form is therefore fenced by asm statements (they emit no
// instructions) that nothing can be merged across.
template <int N, bool kTable, bool kWhole>
__device__ __forceinline__ void copy_vectors(const uint64_t* from, const bool* live, uint8_t* out, int v0,
                                             int tid) {
  if constexpr (kTable) asm volatile(";; table-row chunk");
  u32x4 v[N];
#pragma unroll
  for (int u = 0; u < N; ++u)
    if (kWhole || live[u]) {
      const uint8_t* p = reinterpret_cast<const uint8_t*>(from[u]);
      v[u] = kTable ? load16_table(p) : load16(p);
    }
#pragma unroll
  for (int u = 0; u < N; ++u)
    if (kWhole || live[u]) store16(out + (size_t)(v0 + u * kPackBlock + tid) * 16, v[u]);
  if constexpr (kTable) asm volatile(";; table-row chunk end");
}

// One workgroup packs one chunk of 256 * VPT 16-byte vectors of the output
// (rows are contiguous in the output, so a chunk is a contiguous byte range
// that may start and end inside rows; the last chunks are smaller): it
// resolves the source of every row the chunk touches, then moves up to VPT
// vectors per thread with all loads in flight before the stores. VPT is 3
// (12 KiB chunks), or 2 for rows of kSmallChunkRowBytes or more.
//
// Up to kWaveRows rows per wave (the usual case: a chunk touches two or three
// rows at realistic hidden sizes), each row is resolved by one wave with
// scalar loads, so the only vector memory loads are the copies. Chunks of
// many short rows resolve one row per lane.
template <int VPT, class Args>
__global__ __launch_bounds__(kPackBlock) void k_pack(int32_t g0, int32_t g1, int32_t t1, int32_t t2,
                                                      uint64_t div_mul, int32_t div_shift, int32_t bucket_shift,
                                                      const uint8_t* staged, int32_t off_brun, int32_t off_bucket,
                                                      int32_t total, Args a) {
  constexpr int kChunk = kPackBlock * VPT;       // vectors of a full chunk
  extern __shared__ __align__(16) uint64_t s_src[];
  __shared__ int32_t s_flags[kPackBlock / 64];
  const PackHead h{g0, g1, t1, t2, div_mul, div_shift, bucket_shift, staged, off_brun, off_bucket, total};
  const RunIndex cx{h.bucket_shift, h.off_brun, h.off_bucket};
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const uint8_t* tb = h.tb ? h.tb : a.run_table;
  int my_skip = 0;                                  // a row of this chunk is not copied
  int my_table = 0;                                 // a row of this chunk is an embedding-table row

  const int bx = (int)blockIdx.x;
  int v0, v1;
  if (bx < h.g0) {
    v0 = bx * kChunk;
    v1 = v0 + kChunk;
  } else if (bx < h.g1) {
    v0 = h.t1 + (bx - h.g0) * kTail1Vecs;
    v1 = min(v0 + kTail1Vecs, h.t2);
  } else {
    v0 = h.t2 + (bx - h.g1) * kTail2Vecs;
    v1 = min(v0 + kTail2Vecs, h.total);
  }
  const int r0 = div_vpr(h, v0);
  const int rows = v1 > v0 ? div_vpr(h, v1 - 1) - r0 + 1 : 0;
  // The bucket run and index entry of the wave's first row (a row of the
  // chunk; row 0 of an empty pack, whose table always has them), then the other kernel
  // arguments the row resolution uses in one batch of scalar loads, in flight
  // together with it (the compiler would otherwise split the batch and load
  // it first).
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const BucketHit w0 = bucket_of<true>(cx, tb, r0 + min(wave, max(rows - 1, 0)));
  asm volatile("" : : "s"(w0.w), "s"(w0.r.end), "s"(w0.r.head), "s"(w0.r.vdelta), "s"(w0.r.word),
               "s"(a.off_runs), "s"(a.meta), "s"(a.table), "s"(a.pte), "s"(a.gva_start), "s"(a.pt_mul), "s"(a.pt_shift), "s"(a.pb_mul), "s"(a.pb_shift), "s"(a.page_tokens),
               "s"(a.tier_mask), "s"(a.row_bytes));
  const bool write_meta = (a.tier_mask & 1) != 0;
  const int vpr = a.row_bytes >> 4;

  if (rows <= kWaveRows * (kPackBlock / 64)) {
    // Wave w resolves rows w, w + 4, ... of the chunk, so the dependent load
    // chains of different rows overlap.
    for (int t = wave; t < rows; t += kPackBlock / 64) {
      const int row = r0 + t;
      const BucketHit w = t == wave ? w0 : bucket_of<true>(cx, tb, row);
      const PackRun run = run_of<true>(cx, a.off_runs, tb, row, w);
      const uint64_t src = row_source<true>(a, run, row);
      if (lane == 0) {
        s_src[t] = src;
        if (!src) my_skip = 1;
        else if (run.head < 0) my_table = 1;
      }
    }
  } else {
    for (int t = tid; t < rows; t += kPackBlock) {
      const int row = r0 + t;
      const PackRun run = run_of<false>(cx, a.off_runs, tb, row, bucket_of<false>(cx, tb, row));
      const uint64_t src = row_source<false>(a, run, row);
      s_src[t] = src;
      if (!src) my_skip = 1;
      else if (run.head < 0) my_table = 1;
    }
  }
  // Flags per wave, written before and read after the only barrier.
  const int wave_flags = (__any(my_skip) ? 1 : 0) | (__any(my_table) ? 2 : 0);
  if (lane == 0) s_flags[tid >> 6] = wave_flags;
  __syncthreads();
  int flags = 0;
#pragma unroll
  for (int w = 0; w < kPackBlock / 64; ++w) flags |= s_flags[w];
  flags = __builtin_amdgcn_readfirstlane(flags);   // the same in every lane
  const bool skip = (flags & 1) != 0;
  // Plain loads for the whole chunk (for tables small enough to cache).
  const bool table = (flags & 2) != 0 && (a.tier_mask & kTablePlainLoads) != 0;

  // Vector e of the chunk belongs to row e / vpr (multiply-shift division).
  // A vector is live if it lies in the chunk and its row is copied; only
  // live vectors get an address, dead ones are never loaded or stored.
  uint64_t from[VPT];
  bool live[VPT];
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int e = v0 + u * kPackBlock + tid;
    from[u] = 0;
    live[u] = false;
    if (e < v1) {
      const int row = div_vpr(h, e);
      const uint64_t base = s_src[row - r0];
      live[u] = base != 0;
      from[u] = live[u] ? base + (uint64_t)(e - row * vpr) * 16 : 0;
    }
  }
  // Full chunks and the two tail sizes (whole multiples of the block) with
  // every row copied move their vectors unpredicated; the last chunk and
  // chunks with rows the tier mask leaves out are predicated per vector.
  static_assert(kTail1Vecs % kPackBlock == 0 && kTail2Vecs % kPackBlock == 0 && kTail2Vecs < kTail1Vecs &&
                    kTail1Vecs <= kChunk, "tail chunks are whole multiples of the block");
  constexpr int kT1 = kTail1Vecs / kPackBlock, kT2 = kTail2Vecs / kPackBlock;
  const int n_vec = v1 - v0;
  if (!skip && n_vec == kChunk) {
    if (table) copy_vectors<VPT, true, true>(from, live, a.out, v0, tid);
    else copy_vectors<VPT, false, true>(from, live, a.out, v0, tid);
  } else if (!skip && n_vec == kTail1Vecs) {
    if (table) copy_vectors<kT1, true, true>(from, live, a.out, v0, tid);
    else copy_vectors<kT1, false, true>(from, live, a.out, v0, tid);
  } else if (!skip && n_vec == kTail2Vecs) {
    if (table) copy_vectors<kT2, true, true>(from, live, a.out, v0, tid);
    else copy_vectors<kT2, false, true>(from, live, a.out, v0, tid);
  } else {
    if (table) copy_vectors<VPT, true, false>(from, live, a.out, v0, tid);
    else copy_vectors<VPT, false, false>(from, live, a.out, v0, tid);
  }

  // cu_seqlens and position ids, by the last wave after its copies.
  // Workgroup 0 writes cu_seqlens: an exclusive prefix sum of the sample
  // lengths, 64 samples per step of a wave-wide scan. Workgroup b writes the
  // position ids of rows [64 p, 64 p + 64) for blocks p = b, b + grid, ...,
  // so every cache line of them is written whole by one store instruction:
  // a row's id is the row minus the first row of its sample, taken from the
  // runs that start inside the block.
  if (write_meta && tid >= kPackBlock - 64) {
    if (blockIdx.x == 0 && a.cu) {
      if (lane == 0) a.cu[0] = 0;
      int carry = 0;
      for (int base = 0; base < a.n; base += 64) {
        const int i = base + lane;
        int v = i < a.n ? ld<false, int32_t>(tb + 4 * i) : 0;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const int t = __shfl_up(v, d, 64);
          if (lane >= d) v += t;
        }
        if (i < a.n) a.cu[i + 1] = carry + v;
        carry += __shfl(v, 63, 64);
      }
    }
    if (a.pos) {
      const PackRun* runs = reinterpret_cast<const PackRun*>(tb + a.off_runs);
      for (int blk = blockIdx.x; blk * 64 < a.n_tokens; blk += gridDim.x) {
        const int first = blk * 64, row = first + lane;
        const int last = min(first + 63, a.n_tokens - 1);
        int s;
        PackRun r = run_of<true>(cx, a.off_runs, tb, first, bucket_of<true>(cx, tb, first), &s);
        int start = r.head & 0x7fffffff;
        while (r.end <= last) {
          const int next = r.end;
          r = ld_run<true>(runs + ++s);
          if (row >= next) start = r.head & 0x7fffffff;
        }
        if (row < a.n_tokens) a.pos[row] = row - start;
      }
    }
  }
}

// The vectors [*v0, *v1) of workgroup bx's chunk (geometry as in PackPlan).
template <int VPT>
__device__ __forceinline__ void chunk_range(int bx, int32_t g0, int32_t g1, int32_t t1, int32_t t2, int32_t total,
                                            int* v0, int* v1) {
  constexpr int kChunk = kPackBlock * VPT;
  if (bx < g0) {
    *v0 = bx * kChunk;
    *v1 = *v0 + kChunk;
  } else if (bx < g1) {
    *v0 = t1 + (bx - g0) * kTail1Vecs;
    *v1 = min(*v0 + kTail1Vecs, t2);
  } else {
    *v0 = t2 + (bx - g1) * kTail2Vecs;
    *v1 = min(*v0 + kTail2Vecs, total);
  }
}

// Rows [r0, r0 + rows) of a write: their destinations, into LDS.
template <class Args>
__device__ __forceinline__ void write_rows(const Args& a, int r0, int rows, uint64_t* s_dst, int tid) {
  auto dest = [&](auto scalar, int row) {
    constexpr bool kScalar = decltype(scalar)::value;
    const int lp = (int)(((uint64_t)(uint32_t)row * a.pt_mul) >> a.pt_shift);
    const int in_page = row - lp * a.page_tokens;
    uint64_t vpn;
    if constexpr (Args::kPages > 1) {
      vpn = ld<kScalar, uint32_t>(&a.page[lp]);
    } else if (!a.staged_pages) {
      vpn = (uint64_t)a.page[0] + (uint64_t)lp;
    } else {
      vpn = __umul64hi(ld<kScalar, uint64_t>(a.stage + 8 * (size_t)lp) - a.gva_start, a.pb_mul) >> a.pb_shift;
    }
    return (ld<kScalar, uint64_t>(a.pte + vpn) & PTE_ADDR_MASK) + (uint64_t)in_page * (uint64_t)a.row_bytes;
  };
  if (rows <= kWaveRows * (kPackBlock / 64)) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int t = wave; t < rows; t += kPackBlock / 64) {
      const uint64_t d = dest(std::true_type{}, r0 + t);
      if ((tid & 63) == 0) s_dst[t] = d;
    }
  } else {
    for (int t = tid; t < rows; t += kPackBlock) s_dst[t] = dest(std::false_type{}, r0 + t);
  }
}

// Moves the vectors [v0, v1) of a write, N per thread: loads, then the rows'
// destinations while the loads are in flight, then stores. kWhole: the chunk
// is N full blocks; otherwise a thread past its end loads the last vector
// again and stores nothing (a predicated load would be waited for at once).
template <int N, bool kWhole, class Args>
__device__ __forceinline__ void write_chunk(const Args& a, const uint8_t* vis, uint64_t div_mul, int div_shift,
                                            int v0, int v1, uint64_t* s_dst, int tid) {
  u32x4 v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = v0 + u * kPackBlock + tid;
    v[u] = load16(vis + (size_t)(uint32_t)(kWhole ? e : min(e, v1 - 1)) * 16);
  }
  auto div_row = [&](int e) { return (int)(((uint64_t)(uint32_t)e * div_mul) >> div_shift); };
  const int r0 = div_row(v0);
  write_rows(a, r0, div_row(v1 - 1) - r0 + 1, s_dst, tid);
  __syncthreads();
  const int vpr = a.row_bytes >> 4;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int e = v0 + u * kPackBlock + tid;
    if (kWhole || e < v1) {
      const int row = div_row(e);
      store16(reinterpret_cast<uint8_t*>(s_dst[row - r0]) + (size_t)(e - row * vpr) * 16, v[u]);
    }
  }
}

// Producer write (Sec. 3.2): the first n_meta workgroups copy the sample's
// metadata block from pinned host memory into the arena and publish the
// descriptor; the others move the sample's contiguous visual rows into its
// pages, one chunk each, with the pack's chunk geometry. A thread's rows do
// not depend on where they go, so their loads are issued first and the
// destinations (visual row -> page number -> page-table entry -> row in the
// physical page) are resolved while they are in flight, one row per wave with
// scalar loads or, for chunks of many short rows, one row per lane.
//
// Small writes are bound by their launches: the metadata as a copy of its own
// ahead of the kernel and an event after each cost 8 us of host time and 6 us
// of GPU time per write. A sample of 31 MB read and written takes 6.7 us in
// this kernel (4.7 TB/s; 7.8 us with chunks of one size and the loads after
// the walk), one of 64 rows of 512 bytes 2.3 us (3.4 us, and a 2.2 us copy).
template <int VPT, class Args>
__global__ __launch_bounds__(kPackBlock) void k_write(int32_t g0, int32_t g1, int32_t t1, int32_t t2,
                                                       uint64_t div_mul, const uint8_t* vis, int32_t div_shift,
                                                       int32_t total, int32_t n_meta, Args a) {
  extern __shared__ __align__(16) uint64_t s_dst[];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < n_meta) {
#pragma unroll
    for (int u = 0; u < kMetaVecs / kPackBlock; ++u) {
      const int e = (int)blockIdx.x * kMetaVecs + u * kPackBlock + tid;
      if (e < a.meta_vecs) reinterpret_cast<u32x4*>(a.meta)[e] = load16(a.stage + (size_t)e * 16);
    }
    if (blockIdx.x == 0 && tid == 0) a.desc_table[a.slot] = a.desc;
    return;
  }
  int v0, v1;
  chunk_range<VPT>((int)blockIdx.x - n_meta, g0, g1, t1, t2, total, &v0, &v1);
  const int n_vec = v1 - v0;
  if (n_vec == kPackBlock * VPT) write_chunk<VPT, true>(a, vis, div_mul, div_shift, v0, v1, s_dst, tid);
  else if (n_vec == kTail1Vecs) write_chunk<kTail1Vecs / kPackBlock, true>(a, vis, div_mul, div_shift, v0, v1, s_dst, tid);
  else if (n_vec == kTail2Vecs) write_chunk<kTail2Vecs / kPackBlock, true>(a, vis, div_mul, div_shift, v0, v1, s_dst, tid);
  else write_chunk<VPT, false>(a, vis, div_mul, div_shift, v0, v1, s_dst, tid);
}

// One step of a migration, by one wave: n vectors of a piece (at most
// kMigrateVecs). kWhole as in write_chunk. Stores to HBM are the compiler's own:
// it does not see those of an asm block, so that its wait for a load issued
// before them waits for them as well.
template <bool kWhole, bool kToHost>
__device__ __forceinline__ void migrate_step(const uint8_t* src, uint8_t* dst, uint32_t n, uint32_t lane) {
  constexpr int N = kMigrateVecs / 64;
  u32x4 v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const uint32_t e = u * 64 + lane;
    v[u] = load16(src + (size_t)(kWhole ? e : min(e, n - 1)) * 16);
  }
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const uint32_t e = u * 64 + lane;
    if (kWhole || e < n) {
      if constexpr (kToHost) store16(dst + (size_t)e * 16, v[u]);
      else __builtin_nontemporal_store(v[u], (g_u32x4*)(dst + (size_t)e * 16));
    }
  }
  if constexpr (kWhole) asm volatile(";; whole step");   // keeps the two forms' last stores, and their waits, apart
}

// A piece of the work list, by wave-uniform loads.
__device__ __forceinline__ MigratePiece ld_piece(const uint8_t* p) {
  return MigratePiece{ld<true, uint64_t>(p + offsetof(MigratePiece, src)),
                      ld<true, uint64_t>(p + offsetof(MigratePiece, dst)),
                      ld<true, uint32_t>(p + offsetof(MigratePiece, vecs)), 0, 0};
}

// Tier migration (Sec. 3.2): workgroups [0, n_lists) each put one sample's new
// page list into the arena and its place into the descriptor; a few others walk
// the pieces in steps of kMigrateVecs vectors, reading or writing the host
// tier's memory directly. A workgroup is one wave.
//
// The link to the host bounds it, and all it needs of the chip is enough bytes
// in flight to cover the link's latency: 57 GB/s is the rate of one large copy.
// To keep them in flight whatever the pages' size, adjacent small pages are cut
// into whole steps and a piece's place in the work list, itself across the link,
// is read a step ahead: 33.6 MB of adjacent 8 KiB pages take 773 us to HBM and
// 753 to the host tier, of 512 KiB pages 623 and 614; with one page a step, its
// place read in front of it, 1372 and 864, 645 and 611 (as one DMA copy per
// adjacent run 770 and 788, 730 and 739).
//
// What packs beside it lose decides the shape. A CU returns its loads in order,
// so a read across the link holds up the packs' loads there: single waves spread
// over more CUs cost the packs less than as many in groups of four, and waves
// that do not wait for their stores are fewer. (To the host tier they do wait, as
// a side effect of store16; stores without its sc1 bit gather in the L2 and then hold up
// all traffic: packs 60 us.) 194 MB of scattered 512 KiB pages beside packs of 235
// MB (38.0 us alone), the packs / the migration / the migration alone:
//   to HBM    16 waves 40.7 us, 6.4 ms, 4.3   21 waves 41.2, 5.0, 3.51   26 waves 42.0, 4.2, 3.49
//             10 groups of 4, waiting for their stores 41.4, 7.3, 3.57   as DMA copies 39.9, 7.8, 7.3
//   to host   36 waves 39.6, 5.6, 3.50   40 waves 39.9, 5.1, 3.47   48 waves 40.6, 4.5, 3.46
//             16 groups of 4 40.1, 4.8, 3.45   as DMA copies 39.7, 7.8, 7.3
// To HBM the packs lose as much to a migration as to its DMA copies (their delay
// times its duration), to the host tier three quarters of that.
template <bool kToHost>
__global__ __launch_bounds__(kMigrateBlock) void k_migrate(MigrateArgs a) {
  const uint32_t lane = threadIdx.x;
  if ((int)blockIdx.x < a.n_lists) {
    const uint8_t* l = a.stage + sizeof(MigrateList) * (size_t)blockIdx.x;
    const int64_t words_at = ld<true, int64_t>(l + offsetof(MigrateList, words_at));
    const int64_t meta_off = ld<true, int64_t>(l + offsetof(MigrateList, meta_off));
    const int32_t n_words = ld<true, int32_t>(l + offsetof(MigrateList, n_words));
    const int32_t slot = ld<true, int32_t>(l + offsetof(MigrateList, slot));
    // Two words a vector: both ends have room for the one past an odd number.
    const uint32_t vecs = ((uint32_t)n_words + 1) / 2;
    const uint8_t* from = a.stage + words_at;
    uint8_t* to = a.meta + meta_off;
    for (uint32_t v = 0; v < vecs; v += kMigrateVecs)
      migrate_step<false, false>(from + (size_t)v * 16, to + (size_t)v * 16, min(vecs - v, kMigrateVecs), lane);
    if (lane == 0) a.desc_table[slot].page_off = meta_off;
    return;
  }
  const uint8_t* pieces = a.stage + a.pieces_at;
  const uint32_t first = blockIdx.x - (uint32_t)a.n_lists;
  const uint32_t stride = gridDim.x - (uint32_t)a.n_lists;
  const uint32_t piece_stride = stride / a.steps_per_piece, step_stride = stride % a.steps_per_piece;
  uint32_t piece = first / a.steps_per_piece, step = first % a.steps_per_piece;
  if (piece >= a.n_pieces) return;
  MigratePiece cur = ld_piece(pieces + sizeof(MigratePiece) * (size_t)piece);
  // Waited for here: the first step's wait would otherwise be placed behind the
  // next piece's load and wait for that one too, in every step.
  asm volatile("" : : "s"(cur.src), "s"(cur.dst), "s"(cur.vecs));
  for (;;) {
    uint32_t next = piece + piece_stride, next_step = step + step_stride;
    if (next_step >= a.steps_per_piece) {
      next_step -= a.steps_per_piece;
      ++next;
    }
    // The next piece's place, in flight while this step's vectors are.
    MigratePiece then = cur;
    if (next < a.n_pieces) then = ld_piece(pieces + sizeof(MigratePiece) * (size_t)next);
    const uint32_t done = step * kMigrateVecs;
    if (cur.vecs > done) {
      const uint32_t n = cur.vecs - done;
      const uint8_t* from = reinterpret_cast<const uint8_t*>(cur.src) + (uint64_t)done * 16;
      uint8_t* to = reinterpret_cast<uint8_t*>(cur.dst) + (uint64_t)done * 16;
      if (n >= kMigrateVecs) migrate_step<true, kToHost>(from, to, kMigrateVecs, lane);
      else migrate_step<false, kToHost>(from, to, n, lane);
    }
    if (next >= a.n_pieces) return;
    piece = next;
    step = next_step;
    cur = then;
  }
}

// One thread per sample. Bound by latency: the host waits for the launch, a
// dependent pair of loads and the stores to pinned memory, 5 to 6 us in all
// beside the 3.6 us of the launch; the kernel itself takes 2.2 us over 411 samples.
__global__ __launch_bounds__(kBlock) void k_cost(CostArgs a) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < a.n) {
    const int64_t l = a.desc[a.slots ? a.slots[i] : a.slot[i]].len;
    a.out[i] = a.k * l + l * l;
  }
}

template <class T>
struct As {
  using type = T;
};

// Launches a kernel of `block` threads a workgroup; `done`, if not null,
// completes with it. The status is the launch's own: the thread's
// last error (hipGetLastError) may be an earlier call's, of this library or of
// the caller, and the kernel is queued all the same.
// An event recorded after a kernel costs the stream about 3 us; a launch's own
// stop event next to nothing.
template <class... P>
static hipError_t launch(void (*kernel)(P...), int grid, int block, size_t lds, hipStream_t stream, hipEvent_t done,
                         const typename As<P>::type&... arg) {
  void* args[] = {const_cast<void*>(static_cast<const void*>(&arg))...};
  const void* f = reinterpret_cast<const void*>(kernel);
  if (done) return hipExtLaunchKernel(f, dim3(grid), dim3(block), args, lds, stream, nullptr, done, 0);
  return hipLaunchKernel(f, dim3(grid), dim3(block), args, lds, stream);
}

size_t pack_lds_bytes(const PackPlan& pl) { return sizeof(uint64_t) * (size_t)std::max(pl.max_chunk_rows, 1); }

// Chunk geometry over `vecs` vectors: full chunks of kPackBlock * vpt
// vectors, then a wave of resident workgroups (CUs x kPackPerCU) of
// kTail1Vecs, then half a wave of kTail2Vecs.
static void chunk_geometry(int64_t vecs, int n_cu, PackPlan* pl) {
  const int64_t chunk = (int64_t)kPackBlock * pl->vpt;
  const int64_t wave = (int64_t)std::max(n_cu, 1) * kPackPerCU;
  const int64_t t2 = std::max<int64_t>(vecs - (wave / 2) * kTail2Vecs, 0);
  const int64_t t1 = (std::max<int64_t>(t2 - wave * kTail1Vecs, 0) / chunk) * chunk;
  pl->g0 = (int32_t)(t1 / chunk);
  pl->g1 = (int32_t)(pl->g0 + (t2 - t1 + kTail1Vecs - 1) / kTail1Vecs);
  pl->t1 = (int32_t)t1;
  pl->t2 = (int32_t)t2;
}

static int vectors_per_thread(int64_t row_bytes) { return row_bytes >= kSmallChunkRowBytes ? 2 : kVecsPerThread; }

void pack_chunks(PackPlan* pl, int n_cu) {
  pl->vpt = vectors_per_thread(pl->a.row_bytes);
  chunk_geometry((int64_t)pl->a.n_tokens * (pl->a.row_bytes >> 4), n_cu, pl);
}

template <int VPT, class Args>
static hipError_t launch_pack_as(const PackPlan& pl, const Args& a, int grid, int32_t total, hipStream_t stream,
                                 hipEvent_t done) {
  return launch(&k_pack<VPT, Args>, grid, kPackBlock, pack_lds_bytes(pl), stream, done, pl.g0, pl.g1, pl.t1, pl.t2,
                pl.div_mul, pl.div_shift, a.bucket_shift, pl.staged, a.off_brun, a.off_bucket, total, a);
}

hipError_t launch_pack(const PackPlan& pl, hipStream_t stream, hipEvent_t done) {
  const int64_t vecs = (int64_t)pl.a.n_tokens * (pl.a.row_bytes >> 4);
  const int64_t grid64 = pl.g1 + (vecs - pl.t2 + kTail2Vecs - 1) / kTail2Vecs;
  const int grid = grid64 > 0 ? (int)grid64 : 1;
  const int32_t total = (int32_t)vecs;               // the host keeps this below 2^31
  if (pl.small) {
    PackArgsSmall s;
    std::memcpy(static_cast<void*>(&s), &pl.a, sizeof(s));
    return pl.vpt == 2 ? launch_pack_as<2>(pl, s, grid, total, stream, done)
                       : launch_pack_as<kVecsPerThread>(pl, s, grid, total, stream, done);
  }
  return pl.vpt == 2 ? launch_pack_as<2>(pl, pl.a, grid, total, stream, done)
                     : launch_pack_as<kVecsPerThread>(pl, pl.a, grid, total, stream, done);
}

// ---------------------------------------------------------------------------
// Measurement aids, not steps of the method: a plain copy, and a plain gather
// of rows from given addresses into consecutive output rows, with the pack's
// chunk geometry (chunks of 256 threads x VPT vectors, the same shrinking
// tail stages) and its load and store cache policy. They move the bytes a
// pack moves and do nothing else, so the pack can be timed against them in
// the same run.

// The pack's copy of one chunk's vectors (see k_pack): full chunks and the
// two tail sizes unpredicated, the last chunk predicated per vector.
template <int VPT, bool kTable>
__device__ __forceinline__ void copy_chunk(const uint64_t* from, const bool* live, uint8_t* dst, int v0, int v1) {
  constexpr int kT1 = kTail1Vecs / kPackBlock, kT2 = kTail2Vecs / kPackBlock;
  const int tid = (int)threadIdx.x;
  if (v1 - v0 == kPackBlock * VPT) copy_vectors<VPT, kTable, true>(from, live, dst, v0, tid);
  else if (v1 - v0 == kTail1Vecs) copy_vectors<kT1, kTable, true>(from, live, dst, v0, tid);
  else if (v1 - v0 == kTail2Vecs) copy_vectors<kT2, kTable, true>(from, live, dst, v0, tid);
  else copy_vectors<VPT, kTable, false>(from, live, dst, v0, tid);
}

template <int VPT>
__global__ __launch_bounds__(kPackBlock) void k_copy(int32_t g0, int32_t g1, int32_t t1, int32_t t2, int32_t total,
                                                      const uint8_t* src, uint8_t* dst) {
  int v0, v1;
  chunk_range<VPT>((int)blockIdx.x, g0, g1, t1, t2, total, &v0, &v1);
  uint64_t from[VPT];
  bool live[VPT];
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int e = v0 + u * kPackBlock + (int)threadIdx.x;
    live[u] = e < v1;
    from[u] = live[u] ? reinterpret_cast<uint64_t>(src) + (uint64_t)e * 16 : 0;
  }
  copy_chunk<VPT, false>(from, live, dst, v0, v1);
}

// Output row r is the row_bytes bytes at address rows_src[r] & ~15; bit 0 of
// an entry marks an embedding-table row, and a chunk holding one takes the
// pack's plain loads.
template <int VPT>
__global__ __launch_bounds__(kPackBlock) void k_gather(int32_t g0, int32_t g1, int32_t t1, int32_t t2, int32_t total,
                                                        uint64_t div_mul, int32_t div_shift, int32_t row_bytes,
                                                        const uint64_t* rows_src, uint8_t* dst) {
  extern __shared__ __align__(16) uint64_t s_src[];
  __shared__ int32_t s_table;
  int v0, v1;
  chunk_range<VPT>((int)blockIdx.x, g0, g1, t1, t2, total, &v0, &v1);
  auto div_row = [&](int e) { return (int)(((uint64_t)(uint32_t)e * div_mul) >> div_shift); };
  const int vpr = row_bytes >> 4;
  const int r0 = div_row(v0);
  const int rows = v1 > v0 ? div_row(v1 - 1) - r0 + 1 : 0;
  if (threadIdx.x == 0) s_table = 0;
  __syncthreads();
  for (int t = threadIdx.x; t < rows; t += kPackBlock) {
    const uint64_t x = rows_src[r0 + t];
    s_src[t] = x & ~(uint64_t)15;
    if (x & 1) s_table = 1;
  }
  __syncthreads();
  uint64_t from[VPT];
  bool live[VPT];
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int e = v0 + u * kPackBlock + (int)threadIdx.x;
    live[u] = e < v1;
    from[u] = 0;
    if (live[u]) {
      const int row = div_row(e);
      from[u] = s_src[row - r0] + (uint64_t)(e - row * vpr) * 16;
    }
  }
  if (__builtin_amdgcn_readfirstlane(s_table)) copy_chunk<VPT, true>(from, live, dst, v0, v1);
  else copy_chunk<VPT, false>(from, live, dst, v0, v1);
}

// The pack's chunk geometry for `vecs` vectors of rows of row_bytes bytes.
static void plain_geometry(int64_t vecs, int64_t row_bytes, int n_cu, PackPlan* pl) {
  pl->vpt = vectors_per_thread(row_bytes);
  chunk_geometry(vecs, n_cu, pl);
}

hipError_t launch_copy(const void* src, void* dst, int64_t vecs, int64_t row_bytes, int n_cu, hipStream_t stream) {
  if (vecs <= 0) return hipSuccess;
  PackPlan pl{};
  plain_geometry(vecs, row_bytes, n_cu, &pl);
  const int grid = (int)(pl.g1 + (vecs - pl.t2 + kTail2Vecs - 1) / kTail2Vecs);
  return launch(pl.vpt == 2 ? &k_copy<2> : &k_copy<kVecsPerThread>, grid, kPackBlock, 0, stream, nullptr, pl.g0, pl.g1,
                pl.t1, pl.t2, (int32_t)vecs, (const uint8_t*)src, (uint8_t*)dst);
}

hipError_t launch_gather(const uint64_t* rows_src, int32_t n_rows, int64_t row_bytes, void* dst, int n_cu,
                         hipStream_t stream) {
  if (n_rows <= 0) return hipSuccess;
  const int64_t vecs = (int64_t)n_rows * (row_bytes >> 4);
  PackPlan pl{};
  plain_geometry(vecs, row_bytes, n_cu, &pl);
  const Divisors dv = make_divisors(row_bytes, 1, 16);
  const int grid = (int)(pl.g1 + (vecs - pl.t2 + kTail2Vecs - 1) / kTail2Vecs);
  const size_t lds = sizeof(uint64_t) * (size_t)std::min<int64_t>(n_rows, kChunkVecs / (row_bytes >> 4) + 2);
  return launch(pl.vpt == 2 ? &k_gather<2> : &k_gather<kVecsPerThread>, grid, kPackBlock, lds, stream, nullptr, pl.g0,
                pl.g1, pl.t1, pl.t2, (int32_t)vecs, dv.div_mul, dv.div_shift, (int32_t)row_bytes, rows_src,
                (uint8_t*)dst);
}

template <int VPT, class Args>
static hipError_t launch_write_as(const WritePlan& w, const Args& a, const PackPlan& geo, int32_t total,
                                  int32_t n_meta, hipStream_t stream, hipEvent_t done) {
  const int grid = n_meta + (total > 0 ? geo.g1 + (total - geo.t2 + kTail2Vecs - 1) / kTail2Vecs : 0);
  const size_t lds = sizeof(uint64_t) * (size_t)std::max(w.max_chunk_rows, 1);
  return launch(&k_write<VPT, Args>, grid, kPackBlock, lds, stream, done, geo.g0, geo.g1, geo.t1, geo.t2, w.div_mul,
                w.vis, w.div_shift, total, n_meta, a);
}

hipError_t launch_write(const WritePlan& w, int n_cu, hipStream_t stream, hipEvent_t done) {
  const WriteArgs& a = w.a;
  const int32_t total = w.vis ? a.desc.n_vis * (a.row_bytes >> 4) : 0;   // the host keeps this below 2^31
  const int32_t n_meta = std::max((a.meta_vecs + kMetaVecs - 1) / kMetaVecs, 1);
  PackPlan geo{};
  plain_geometry(total, a.row_bytes, n_cu, &geo);
  if (w.inline_pages)
    return geo.vpt == 2 ? launch_write_as<2>(w, a, geo, total, n_meta, stream, done)
                        : launch_write_as<kVecsPerThread>(w, a, geo, total, n_meta, stream, done);
  WriteArgsSmall s;
  std::memcpy(static_cast<void*>(&s), &a, sizeof(s));
  return geo.vpt == 2 ? launch_write_as<2>(w, s, geo, total, n_meta, stream, done)
                      : launch_write_as<kVecsPerThread>(w, s, geo, total, n_meta, stream, done);
}

hipError_t launch_migrate(const MigrateArgs& a, hipStream_t stream, hipEvent_t done) {
  const int64_t steps = (int64_t)a.n_pieces * a.steps_per_piece;
  const int grid = a.n_lists + (int)std::min<int64_t>(steps, kMigrateGrid[a.tier]);
  return launch(a.tier ? &k_migrate<true> : &k_migrate<false>, grid, kMigrateBlock, 0, stream, done, a);
}

Divisors make_divisors(int64_t row_bytes, int64_t page_tokens, uint64_t page_bytes) {
  Divisors d{};
  // e / q for e < 2^31: with s = 31 + ceil(log2 q), m = ceil(2^s / q), e / q == (e * m) >> s.
  auto small = [](int64_t q, uint64_t* mul, int32_t* shift) {
    int c = 0;
    while ((1ll << c) < q) ++c;
    *shift = 31 + c;
    *mul = (uint64_t)(((1ull << *shift) + (uint64_t)q - 1) / (uint64_t)q);
  };
  small(row_bytes / 16, &d.div_mul, &d.div_shift);
  small(page_tokens, &d.pt_mul, &d.pt_shift);
  // GVA offset d < 2^52 by page_bytes: with c = ceil(log2 pb), N = max(52, 64 - c)
  // and s = N + c, m = ceil(2^s / pb) fits in 64 bits and d / pb == (d * m) >> s,
  // taken as the high 64 bits of the 128-bit product shifted by s - 64.
  int c = 0;
  while ((1ull << c) < page_bytes) ++c;
  const int sh = std::max(52, 64 - c) + c;
  d.pb_mul = (uint64_t)((((unsigned __int128)1 << sh) + page_bytes - 1) / page_bytes);
  d.pb_shift = sh - 64;
  return d;
}

hipError_t launch_cost(const SampleDesc* desc, const int32_t* slots, const int32_t* slots_dev, int32_t n, int64_t k,
                       int64_t* out_cost, hipStream_t stream, hipEvent_t done) {
  CostArgs a;
  a.desc = desc;
  a.slots = n > kCostSlots ? slots_dev : nullptr;
  a.out = out_cost;
  a.k = k;
  a.n = n;
  std::memcpy(a.slot, slots, sizeof(int32_t) * (size_t)std::min<int32_t>(n, kCostSlots));
  return launch(&k_cost, (n + kBlock - 1) / kBlock, kBlock, 0, stream, done, a);
}

}  // namespace fp
