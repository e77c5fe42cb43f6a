// HIP kernels of the voxmesh library for gfx950 (wave64).
//
// Per-block work (fusion, import, classification, vertices, the TSDF
// backward) gives each 8^3 block one wave, and the block's halo is staged in
// the wave's own LDS, so waves of a workgroup never wait for each other.
// Fusion and import give lane q the column of eight voxels at (x, y) =
// (q & 7, q >> 3); classification, vertices and the backward give it the row
// along x at (y, z) = (q & 7, q >> 3), whose eight cube types, edge bits and
// masks are one word each, and handle the row's eight cubes at once.  Work
// lists live on the device and every kernel loops over its list on a grid
// sized to the device, so the host never waits for a count.  Lists are
// appended to with at most one atomic per workgroup (per wave for the short
// list of extra vertex blocks); pool allocations take one atomic per block
// on the block's pool segment.
#include "voxmesh.h"
#include "vm_internal.h"

namespace vm {

// ============================================================================
// bookkeeping
// ============================================================================
// Segment s as closing it would leave it (nothing is written back).
__device__ inline Seg closed_segment(const VolDev& v, uint32_t s) {
  Seg g = v.vseg[s];
  finalise_seg(g, seg_size(s, v.vseg_cap, v.max_vertices));
  return g;
}

// Segment statistics summed over all segments (running counts, modulo 2^32).
struct SegSums {
  uint32_t nw, upd, freed, mov, chg, ref, fnew, fold;
};

// One full wave closes every vertex pool segment (lane q takes segments q,
// q + 64, ...: slots freed by earlier passes become available) and sums the
// segment statistics; every lane receives the sums.
__device__ inline SegSums close_segments(const VolDev& v) {
  static_assert(kSegs % 64 == 0, "whole waves of segments");
  constexpr int kPer = kSegs / 64;
  SegSums r{0, 0, 0, 0, 0, 0, 0, 0};
  // every lane's segments are read before any is written back
  Seg g[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int s = __lane_id() + 64 * j;
    g[j] = v.vseg[s];
    const Seg& cs = v.cseg[s];
    r.chg += cs.st_chg, r.ref += cs.st_ref, r.fnew += cs.st_fnew, r.fold += cs.st_fold;
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int s = __lane_id() + 64 * j;
    finalise_seg(g[j], seg_size(s, v.vseg_cap, v.max_vertices));
    r.nw += g[j].st_new, r.upd += g[j].st_upd, r.freed += g[j].st_freed, r.mov += g[j].st_mov;
    Seg& vs = v.vseg[s];
    vs.hwm = g[j].hwm, vs.head = g[j].head, vs.count = g[j].count;
    vs.ticket = 0, vs.push = 0, vs.st_new = g[j].st_new, vs.st_freed = g[j].st_freed;
  }
  r.nw = wave_sum(r.nw), r.upd = wave_sum(r.upd), r.freed = wave_sum(r.freed);
  r.mov = wave_sum(r.mov), r.chg = wave_sum(r.chg), r.ref = wave_sum(r.ref);
  r.fnew = wave_sum(r.fnew), r.fold = wave_sum(r.fold);
  return r;
}

// Start of an extraction (refine = false) or of a refinement's vertex pass,
// done by one full wave while nothing else touches the segments: the segments
// are closed, and lane 0 records the statistics the call reports per call and
// clears the list lengths of the next call.  A refinement's classification
// has run by then: it counts apart (st_pass), and its counts join the running
// ones here, so that the call needs no launch of its own to begin with (5 us
// of a refinement pass).
__device__ inline void begin_call(const VolDev& v, bool refine) {
  uint32_t pass[kSegs / 64];
  if (refine)
#pragma unroll
    for (int j = 0; j < kSegs / 64; ++j) pass[j] = v.cseg[__lane_id() + 64 * j].st_pass;
  const SegSums m = close_segments(v);
  if (refine)
#pragma unroll
    for (int j = 0; j < kSegs / 64; ++j) {
      Seg& cs = v.cseg[__lane_id() + 64 * j];
      cs.st_chg += pass[j], cs.st_ref += pass[j], cs.st_pass = 0;
    }
  if (__lane_id() != 0) return;
  Counters* c = v.cnt;
  if (!refine) c->n_dirty[v.xsel ^ 1u] = 0;
  c->n_vblocks[v.vsel ^ 1u] = 0;
  c->base_new = m.nw;
  c->base_upd = m.upd;
  c->base_freed = m.freed;
  c->base_chg = m.chg;
  c->base_ref = m.ref;
}

// One wave: the segments closed for a call that reads them.
__global__ __launch_bounds__(64) void k_close(VolDev v) { close_segments(v); }

// The counters and the segments' sums, written to the host's record by one
// workgroup, a lane per segment.  One launch and a wait of the host take 15
// us where copies of the counters and both segment tables took 45.
__global__ __launch_bounds__(256) void k_report(VolDev v, Report* __restrict__ out) {
  static_assert(kSegs == 256, "a lane per segment");
  constexpr int kSums = 13;
  __shared__ unsigned long long part[4][kSums];
  const Seg g = closed_segment(v, threadIdx.x);
  const Seg c = v.cseg[threadIdx.x];
  unsigned long long x[kSums] = {g.st_new,  g.st_upd,  g.st_mov, g.st_freed, c.st_chg,
                                 c.st_ref,  c.st_fnew, c.st_fold, c.st_cnew, c.st_cold,
                                 g.hwm,     g.count,   g.hwm - min(g.hwm, g.count)};
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
      const unsigned long long y = shfl64(x[k], __lane_id() ^ off);
      x[k] = k < kSums - 1 ? x[k] + y : max(x[k], y);
    }
  if (__lane_id() == 0)
    for (int k = 0; k < kSums; ++k) part[threadIdx.x >> 6][k] = x[k];
  __syncthreads();
  if (threadIdx.x < kSums) {
    unsigned long long y = 0;
    for (int w = 0; w < 4; ++w)
      y = threadIdx.x < kSums - 1 ? y + part[w][threadIdx.x] : max(y, part[w][threadIdx.x]);
    (&out->st_new)[threadIdx.x] = y;
  }
  static_assert(offsetof(Report, seg_live) == offsetof(Report, st_new) + 8 * (kSums - 1), "sums");
  if (threadIdx.x < VM_TOTAL_COUNT) out->acc[threadIdx.x] = v.cnt->acc[threadIdx.x];
  if (threadIdx.x != 0) return;
  const Counters& n = *v.cnt;
  out->error = n.error, out->n_blocks = n.n_blocks;
  for (int k = 0; k < 2; ++k) {
    out->n_frame[k] = n.n_frame[k], out->n_pending[k] = n.n_pending[k];
    out->n_dirty[k] = n.n_dirty[k], out->n_vblocks[k] = n.n_vblocks[k];
  }
  out->base_new = n.base_new, out->base_upd = n.base_upd, out->base_freed = n.base_freed;
  out->base_chg = n.base_chg, out->base_ref = n.base_ref;
  out->dl_nv = n.dl_nv, out->dl_nt = n.dl_nt;
}

// Sixteen bytes per store over [p, p + n16 * 16), shared by `step` lanes.
__device__ inline void fill16(void* p, uint64_t n16, uint32_t x, uint64_t i, uint64_t step) {
  uint4* q = reinterpret_cast<uint4*>(p);
  for (; i < n16; i += step) q[i] = make_uint4(x, x, x, x);
}

// Empty the volume: the hash slots to "empty", the slot and block stamps to
// 0, the counters and segments to 0.  The first workgroup folds the segment
// statistics into the running totals before it clears them (create: the
// workspace holds nothing yet, and the totals start at 0 as well); the
// others fill.  Bound by the launch: a volume of 2^17 hash slots and 2^15
// blocks has 2.5 MB to clear, 0.5 us at this card's copy rate, where one fill
// kernel per region and the fold took ten launches of 1.3 to 4.4 us each.
__global__ __launch_bounds__(256) void k_reset(VolDev v, int create) {
  if (blockIdx.x > 0) {
    const uint64_t i = (uint64_t)(blockIdx.x - 1) * blockDim.x + threadIdx.x;
    const uint64_t step = (uint64_t)(gridDim.x - 1) * blockDim.x;
    const uint64_t H = (uint64_t)v.hash_mask + 1;
    uint4* slots = reinterpret_cast<uint4*>(v.slots);
    for (uint64_t k = i; k < H; k += step) slots[k] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u);
    // the four block stamps lie one after the other (256-byte regions)
    const uint64_t stamps = (uint64_t)((char*)v.st_frame - (char*)v.st_pending) +
                            (((uint64_t)v.max_blocks * 4 + 15) & ~15ull);
    fill16(v.st_pending, stamps / 16, 0u, i, step);
    return;
  }
  if (!create && threadIdx.x < 64) {
    const SegSums m = close_segments(v);
    if (threadIdx.x == 0) {
      unsigned long long* acc = v.cnt->acc;
      acc[VM_TOTAL_NEW_TRIANGLES] += m.fnew;
      acc[VM_TOTAL_DROPPED_TRIANGLES] += m.fold;
      acc[VM_TOTAL_NEW_VERTICES] += m.nw;
      acc[VM_TOTAL_UPDATED_VERTICES] += m.upd;
      acc[VM_TOTAL_MOVED_VERTICES] += m.mov;
      acc[VM_TOTAL_FREED_VERTICES] += m.freed;
      acc[VM_TOTAL_CHANGED_CUBES] += m.chg;
      acc[VM_TOTAL_REFINED_CUBES] += m.ref;
    }
  }
  __syncthreads();  // the statistics are read
  // (a segment's dl_top says which download rows there may be: it stays)
  for (uint32_t i = threadIdx.x; i < sizeof(Seg) * kSegs / 4; i += blockDim.x)
    if (create || i % (sizeof(Seg) / 4) != offsetof(Seg, dl_top) / 4)
      reinterpret_cast<uint32_t*>(v.vseg)[i] = 0u;
  fill16(v.cseg, sizeof(Seg) * kSegs / 16, 0u, threadIdx.x, blockDim.x);
  const uint32_t words = (create ? sizeof(Counters) : offsetof(Counters, acc)) / 4;
  for (uint32_t i = threadIdx.x; i < words; i += blockDim.x)
    reinterpret_cast<uint32_t*>(v.cnt)[i] = 0u;
}

// ============================================================================
// block collection (Eq. 1)
// ============================================================================

// P pixels per lane, one wave per tile of 8 x 8 P pixels, a workgroup per
// 32 x 16 P.  Each valid pixel spans the integer box of blocks between
// its ray points at camera depth D - mu and D + mu.  Neighbouring pixels
// span nearly the same blocks, so the wave forms the union of its pixels'
// boxes as a bit mask over a 4 x 4 x 4 window of blocks placed at one
// pixel's box (an OR over the wave) and lists the blocks in LDS; pixels
// whose boxes leave the window (a depth edge inside the tile) go on with a
// window placed at one of theirs, until none is left.  Its lanes then take
// the listed blocks one each.  A box of more than three blocks on some axis
// (a truncation of more than about eight voxels) fits no window: the wave
// agrees on its blocks by a slower ballot loop.
// The lanes holding distinct blocks insert them into the hash and claim the
// slot for this frame (exchange of the slot's frame stamp): the one claim
// that wins lists the block.  The workgroup gathers its claims in LDS and
// appends them with one atomic per list: the frame list, the pending list
// (blocks touched since the last extraction) and, for blocks new to the
// hash, pool indices, given here with their neighbour tables cleared.  The
// three appends are one packed 64-bit atomic (one per workgroup).
// Bound by latency, a chain of about seven dependent accesses, and in large
// images by that atomic, on one address from every workgroup (of 640 x 480
// pixels at 8 mm 2.4 of 11.8 us): two pixels per lane halve the workgroups.
// With P = 1 and 2: 11.8 and 9.9 us at 640 x 480 (600 workgroups of P = 1),
// 9.3 and 9.5 at 400 x 300 (247), 8.4 and 11.4 at 240 x 180 (96); 13.6 and
// 11.6 at 4 mm.  P = 4 takes 11.5 and 15.8 us at 640 x 480.
constexpr int kClaimCap = 512;   // claims per workgroup gathered in LDS
constexpr int kWaveKeys = 128;   // keys a wave gathers before claiming them

// List a claimed block: frame list entry, pending list entry (once per
// extraction epoch) and, for a block new to the hash, its pool index (slot
// value and key record updated, neighbour table cleared).  fpos, ppos and
// bidx are the positions the caller reserved.
__device__ inline void list_claim(const VolDev& v, uint32_t s, unsigned long long seen,
                                  bool pend, uint32_t fpos, uint32_t ppos, uint32_t bidx,
                                  uint32_t frame, uint32_t epoch) {
  uint32_t idx = (uint32_t)(seen & kIdxMask), entry = idx;
  if (idx == kPending) {
    if (bidx < v.max_blocks) {
      idx = bidx;
      const uint64_t key = seen >> kIdxBits;
      v.slots[s] = HashSlot{(key << kIdxBits) | idx, frame, epoch};  // new: listed as well
      v.block_key[idx] = key;
      int32_t* nb = v.nbr + (size_t)idx * 27;
      for (int d = 0; d < 27; ++d) nb[d] = d == kSelf ? (int32_t)idx : -1;
      entry = idx | kNewFlag;
    } else {
      atomicOr(&v.cnt->error, kErrBlocks);
      idx = kNone;
      entry = kNone;
    }
  }
  if (fpos < v.max_blocks) {
    v.frame_list[fpos] = entry;
    v.frame_key[fpos] = seen >> kIdxBits;
  } else {
    atomicOr(&v.cnt->error, kErrBlocks);
  }
  if (pend) {
    if (idx != kNone) v.st_pending[idx] = epoch;
    if (idx == (uint32_t)(seen & kIdxMask)) v.slots[s].listed = epoch;
    if (ppos < v.max_blocks) v.pending[ppos] = idx;
    else atomicOr(&v.cnt->error, kErrBlocks);
  }
}

template <int P>
__global__ __launch_bounds__(512) void k_collect(VolDev v, FrameParams fp,
                                                const float* __restrict__ depth, uint32_t epoch) {
  __shared__ unsigned long long sseen[kClaimCap];  // slot contents seen by the claim
  __shared__ uint32_t sslot[kClaimCap];            // slot | pending << 31
  __shared__ unsigned long long skeys_all[8][kWaveKeys];  // keys each wave is to claim
  __shared__ uint32_t nclaim;
  __shared__ uint32_t swave[8];
  __shared__ uint32_t sbase[3];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = __lane_id();
  const int tiles_x = (fp.W + kTileW - 1) / kTileW;
  const int px = (int)(blockIdx.x % tiles_x) * kTileW + (wave & 3) * 8 + (q & 7);
  const int py0 = (int)(blockIdx.x / tiles_x) * (kTileH * P) + (wave >> 2) * 8 * P + (q >> 3);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    // the other parity's list and appends are the next frame's
    v.cnt->n_frame[(fp.frame + 1) & 1] = 0;
    v.cnt->collect_acc[(fp.frame + 1) & 1] = 0;
    v.cnt->acc[VM_TOTAL_FRAMES] += 1;
  }
  // the lists this frame appends to: the frame list starts empty, the
  // pending list and the pool continue from where they stand (nothing else
  // changes them during this kernel)
  unsigned long long* acc = &v.cnt->collect_acc[fp.frame & 1];
  const uint32_t pend_base = v.cnt->n_pending[epoch & 1], blk_base = v.cnt->n_blocks;
  // cleared here, first used after the barrier below
  if (threadIdx.x == 0) nclaim = 0;
  float D[P];
#pragma unroll
  for (int k = 0; k < P; ++k) {
    const int py = py0 + 8 * k;
    D[k] = px < fp.W && py < fp.H ? depth[py * fp.W + px] : 0.f;
  }
  int lo[P][3], ext[P][3], nbox[P];
#pragma unroll
  for (int k = 0; k < P; ++k) {
    const int py = py0 + 8 * k;
    nbox[k] = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) lo[k][i] = 0, ext[k][i] = 1;
    if (px < fp.W && py < fp.H && depth_ok(D[k], fp.dmin, fp.dmax)) {
      const float xn = ((float)px - fp.cx) / fp.fx;
      const float yn = ((float)py - fp.cy) / fp.fy;
      int b[2][3];
      bool ok = true;
#pragma unroll
      for (int end = 0; end < 2; ++end) {
        const float z = end == 0 ? D[k] - v.mu_m : D[k] + v.mu_m;
        const float p0 = xn * z, p1 = yn * z;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          float X = fp.Rcw[3 * i] * p0;
          X = X + fp.Rcw[3 * i + 1] * p1;
          X = X + fp.Rcw[3 * i + 2] * z;
          X = X + fp.tcw[i];
          const float fb = floorf(X * v.inv_block);
          ok = ok && (fb >= -8192.f && fb <= 8191.f);
          b[end][i] = ok ? (int)fb : 0;
        }
      }
      if (ok) {
        nbox[k] = 1;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          lo[k][i] = min(b[0][i], b[1][i]);
          ext[k][i] = abs(b[1][i] - b[0][i]) + 1;
          nbox[k] *= ext[k][i];
        }
      }
    }
  }
  // Claim one key per lane (has: the lane holds one): insert it, take the
  // slot's frame stamp, and gather the winners in the workgroup's list with
  // whether each must join the pending list.
  auto claim = [&](bool has, uint64_t key) {
    HashSlot seen{};
    int64_t s = -1;
    if (has) {
      s = hash_insert_seen(v, key, &seen);
      if (s < 0) atomicOr(&v.cnt->error, kErrHash);
    }
    const bool won = s >= 0 && take_stamp(v, s, seen, fp.frame);
    const bool pend = won && must_list(seen, epoch);
    const uint64_t bw = __ballot(won);
    if (bw == 0ull) return;
    uint32_t c0 = 0;
    if (q == 0) c0 = atomicAdd(&nclaim, (uint32_t)__popcll(bw));
    const uint32_t c = uniform(c0) + mask_rank(bw);
    if (!won) return;
    if (c < (uint32_t)kClaimCap) {
      sslot[c] = (uint32_t)s | (pend ? 0x80000000u : 0u);
      sseen[c] = seen.entry;
    } else {
      // more claims than the workgroup gathers: list this one alone
      const bool isnew = (uint32_t)(seen.entry & kIdxMask) == kPending;
      const uint64_t p = atomicAdd(acc, (unsigned long long)collect_pack(1u, pend, isnew));
      list_claim(v, (uint32_t)s, seen.entry, pend, collect_frame(p), pend_base + collect_pend(p),
                 blk_base + collect_new(p), fp.frame, epoch);
    }
  };
  unsigned long long* skeys = skeys_all[wave];
  uint32_t nkeys = 0;
  auto claim_keys = [&]() {
    wave_sync();
    for (uint32_t i0 = 0; i0 < nkeys; i0 += 64) {
      const uint32_t i = i0 + (uint32_t)q;
      claim(i < nkeys, i < nkeys ? skeys[i] : 0ull);
    }
    nkeys = 0;
    wave_sync();
  };
  // window by window, the union of the boxes that fit it (duplicates between
  // windows are left to the claim)
  bool wide[P];
  uint64_t left[P];
#pragma unroll
  for (int k = 0; k < P; ++k) {
    wide[k] = nbox[k] > 0 && max(ext[k][0], max(ext[k][1], ext[k][2])) > 3;
    left[k] = __ballot(nbox[k] > 0 && !wide[k]);
  }
  __syncthreads();  // the claim count is cleared
#pragma unroll
  for (int k0 = 0; k0 < P; ++k0) {
    while (left[k0]) {
      const int lead = __builtin_ctzll(left[k0]);
      const int w0 = __builtin_amdgcn_readlane(lo[k0][0], lead) - 1,
                w1 = __builtin_amdgcn_readlane(lo[k0][1], lead) - 1,
                w2 = __builtin_amdgcn_readlane(lo[k0][2], lead) - 1;
      uint64_t m = 0;
#pragma unroll
      for (int k = k0; k < P; ++k) {
        const int ox = lo[k][0] - w0, oy = lo[k][1] - w1, oz = lo[k][2] - w2;
        const bool fits = ((left[k] >> q) & 1ull) && ox >= 0 && oy >= 0 && oz >= 0 &&
                          ox + ext[k][0] <= 4 && oy + ext[k][1] <= 4 && oz + ext[k][2] <= 4;
        if (fits) {
          // the box's rows along x as runs of bits
          const uint64_t row = ((1ull << ext[k][0]) - 1ull) << ox;
          for (int z = 0; z < ext[k][2]; ++z)
            for (int y = 0; y < ext[k][1]; ++y) m |= row << (4 * (oy + y) + 16 * (oz + z));
        }
        left[k] &= ~__ballot(fits);
      }
      const uint64_t u = wave_or64(m);
      if (nkeys + (uint32_t)__popcll(u) > (uint32_t)kWaveKeys) claim_keys();
      // lane c, for a cell c in the union, lists it at its rank
      if ((u >> q) & 1ull)
        skeys[nkeys + mask_rank(u)] = pack_key(w0 + (q & 3), w1 + ((q >> 2) & 3), w2 + (q >> 4));
      nkeys += (uint32_t)__popcll(u);
    }
  }
  // boxes that fit no window: the wave agrees on their distinct keys per box
  // position (duplicates between positions are left to the claim)
#pragma unroll
  for (int k = 0; k < P; ++k) {
    if (__ballot(wide[k]) == 0ull) continue;
    const int nslow = wide[k] ? nbox[k] : 0;
    int cx = 0, cy = 0, cz = 0;
    const uint64_t below = lanes_below();
    for (int j = 0; __ballot(j < nslow); ++j) {
      bool has = j < nslow;
      uint64_t key = 0;
      if (has) {
        key = pack_key(lo[k][0] + cx, lo[k][1] + cy, lo[k][2] + cz);
        if (++cx == ext[k][0]) {
          cx = 0;
          if (++cy == ext[k][1]) cy = 0, ++cz;
        }
      }
      bool mine = false;  // this lane holds the first copy of its key
      uint64_t todo = __ballot(has);
      while (todo) {
        // the leader is wave-uniform: its key is read lane to scalar
        const int leader = __builtin_ctzll(todo);
        const uint32_t klo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, leader);
        const uint32_t khi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(key >> 32), leader);
        const uint64_t lk = ((uint64_t)khi << 32) | klo;
        const bool same = has && key == lk;
        todo &= ~__ballot(same);
        if (q == leader) mine = true;
        if (same) has = false;
      }
      const uint64_t bm = __ballot(mine);
      const uint32_t nm = (uint32_t)__popcll(bm);
      if (nkeys + nm > (uint32_t)kWaveKeys) claim_keys();
      if (mine) skeys[nkeys + (uint32_t)__popcll(bm & below)] = key;
      nkeys += nm;
    }
  }
  claim_keys();
  __syncthreads();
  // one claim per thread: the three lists' positions from one workgroup
  // scan of packed counts (fields of 10 bits, at most 512 each)
  const uint32_t nc = min(nclaim, (uint32_t)kClaimCap);
  const uint32_t c = threadIdx.x;
  const bool hit = c < nc;
  unsigned long long seen = 0;
  uint32_t slot = 0;
  bool isnew = false, pend = false;
  if (hit) {
    seen = sseen[c];
    slot = sslot[c];
    pend = (slot >> 31) != 0u;
    slot &= 0x7FFFFFFFu;
    isnew = (uint32_t)(seen & kIdxMask) == kPending;
  }
  const uint64_t bh = __ballot(hit), bn = __ballot(isnew), bp = __ballot(pend);
  if (q == 0)
    swave[wave] = (uint32_t)__popcll(bh) | (uint32_t)__popcll(bn) << 10 |
                  (uint32_t)__popcll(bp) << 20;
  __syncthreads();
  uint32_t before = 0, all = 0;
  const int nwave = (int)(blockDim.x >> 6);
  for (int w = 0; w < nwave; ++w) {
    const uint32_t cw = swave[w];
    if (w < wave) before += cw;
    all += cw;
  }
  if (threadIdx.x == 0 && (all & 1023u)) {
    const uint64_t p = atomicAdd(
        acc, (unsigned long long)collect_pack(all & 1023u, all >> 20, (all >> 10) & 1023u));
    sbase[0] = collect_frame(p);
    sbase[1] = blk_base + collect_new(p);
    sbase[2] = pend_base + collect_pend(p);
  }
  __syncthreads();
  if (hit)
    list_claim(v, slot, seen, pend, sbase[0] + (before & 1023u) + mask_rank(bh),
               sbase[2] + (before >> 20) + mask_rank(bp),
               sbase[1] + ((before >> 10) & 1023u) + mask_rank(bn), fp.frame, epoch);
}

// Import, rows to blocks, in two launches: a key goes into the hash and the
// row that takes its slot's frame stamp first speaks for it (the rows of a
// call name distinct keys; of several naming one, one is taken).  Such a row
// lists its block in the frame list, numbers it when it is new and adds it to
// the pending list once per extraction epoch, all in row order: the insert
// knows and records what each row will append and counts per part of
// kImportRows rows, and every part of the second launch sums the parts before
// it by itself.  (Winners found and counted by a launch of their own, and a
// one-workgroup scan over the parts, cost 14 us of 65 for 230,000 rows, and
// two launches of the smallest import.  Each part sums all before it: 57,000
// rows are numbered in 9 us where the three launches took 19, 1 million in 65
// against 140, 2 million, the largest pool, in 128 against 272.)
constexpr uint32_t kRowHit = 1u << 31, kRowNew = 1u << 30, kRowPend = 1u << 29;  // beside the slot

__global__ __launch_bounds__(kImportRows) void k_import_insert(
    VolDev v, const int32_t* __restrict__ slots, const int32_t* __restrict__ coords, uint32_t n,
    uint32_t frame, uint32_t epoch) {
  __shared__ uint32_t swave[16];
  const uint32_t i = blockIdx.x * kImportRows + threadIdx.x;
  if (i == 0) {
    // this import's list starts empty, and so does the next frame's: an
    // integration appends to its own parity's list (and packed appends)
    // without clearing them; the lists the import appends to start from here
    v.cnt->n_frame[frame & 1] = 0;
    v.cnt->n_frame[(frame + 1) & 1] = 0;
    v.cnt->collect_acc[0] = 0;
    v.cnt->collect_acc[1] = 0;
    v.cnt->acc[VM_TOTAL_FRAMES] += 1;
    v.cnt->import_base = v.cnt->n_blocks;
    v.cnt->import_pend = v.cnt->n_pending[epoch & 1];
  }
  bool ok = i < n;
  int x = 0, y = 0, z = 0;
  if (ok) {
    x = coords[3 * (size_t)i], y = coords[3 * (size_t)i + 1], z = coords[3 * (size_t)i + 2];
    if (slots) {
      const int k = slots[i];
      ok = k >= 0 && (uint32_t)k < v.batch && x >= 0 && x <= kSlotSpan - 2;
      x += kSlotSpan * k - kKeyBias;
    }
    ok = ok && key_in_range(x, y, z);
    if (!ok) atomicOr(&v.cnt->error, kErrRange);
  }
  uint32_t row = 0;
  if (ok) {
    HashSlot seen;
    const int64_t s = hash_insert_seen(v, pack_key(x, y, z), &seen);
    if (s < 0) {
      atomicOr(&v.cnt->error, kErrHash);
    } else if (take_stamp(v, s, seen, frame)) {
      row = kRowHit | (uint32_t)s |
            ((uint32_t)(seen.entry & kIdxMask) == kPending ? kRowNew : 0u) |
            (must_list(seen, epoch) ? kRowPend : 0u);
    }
  }
  if (i < n) v.row_slot[i] = row;
  uint32_t t_hit, t_new, t_pend;
  wg_scan_bits<1>((row & kRowHit) != 0u, swave, &t_hit);
  wg_scan_bits<1>((row & kRowNew) != 0u, swave, &t_new);
  wg_scan_bits<1>((row & kRowPend) != 0u, swave, &t_pend);
  if (threadIdx.x == 0) {
    v.scan[3 * blockIdx.x] = t_hit;
    v.scan[3 * blockIdx.x + 1] = t_new;
    v.scan[3 * blockIdx.x + 2] = t_pend;
  }
}

__global__ __launch_bounds__(kImportRows) void k_import_assign(VolDev v, uint32_t n, uint32_t frame,
                                                                uint32_t epoch) {
  __shared__ uint32_t swave[16];
  __shared__ uint32_t sbefore[3][kImportRows / 64];
  const uint32_t i = blockIdx.x * kImportRows + threadIdx.x;
  const uint32_t row = i < n ? v.row_slot[i] : 0u, slot = row & ~(kRowHit | kRowNew | kRowPend);
  const bool hit = (row & kRowHit) != 0u, fresh = (row & kRowNew) != 0u, pend = (row & kRowPend) != 0u;
  const unsigned long long entry0 = hit ? v.slots[slot].entry : 0ull;
  // the appends of the parts before this one
  uint32_t before[3] = {0u, 0u, 0u};
  for (uint32_t p = threadIdx.x; p < blockIdx.x; p += kImportRows)
#pragma unroll
    for (int k = 0; k < 3; ++k) before[k] += v.scan[3 * p + k];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    before[k] = wave_sum(before[k]);
    if (__lane_id() == 0) sbefore[k][threadIdx.x >> 6] = before[k];
  }
  uint32_t t_hit, t_new, t_pend;
  const uint32_t r_hit = wg_scan_bits<1>(hit, swave, &t_hit);
  const uint32_t r_new = wg_scan_bits<1>(fresh, swave, &t_new);
  const uint32_t r_pend = wg_scan_bits<1>(pend, swave, &t_pend);
  uint32_t base[3] = {0u, v.cnt->import_base, v.cnt->import_pend};
#pragma unroll
  for (int k = 0; k < 3; ++k)
    for (int w = 0; w < kImportRows / 64; ++w) base[k] += sbefore[k][w];
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    v.cnt->n_frame[frame & 1] = base[0] + t_hit;
    v.cnt->n_blocks = base[1] + t_new;
    v.cnt->n_pending[epoch & 1] = base[2] + t_pend;
  }
  if (!hit) return;
  const uint32_t pos = base[0] + r_hit, t = base[1] + r_new, p = base[2] + r_pend;
  uint32_t idx = (uint32_t)(entry0 & kIdxMask), entry = idx;
  if (fresh) {
    if (t < v.max_blocks) {
      idx = t;
      const uint64_t key = entry0 >> kIdxBits;
      v.slots[slot] = HashSlot{(key << kIdxBits) | idx, 0u, epoch};  // new: listed as well
      v.block_key[idx] = key;
      int32_t* nb = v.nbr + (size_t)idx * 27;
      for (int d = 0; d < 27; ++d) nb[d] = d == kSelf ? (int32_t)idx : -1;
      entry = idx | kNewFlag;
    } else {
      atomicOr(&v.cnt->error, kErrBlocks);
      idx = kNone;
      entry = kNone;
    }
  }
  // the row is placed, and its claim is dropped: a graph that holds this import
  // and no reset runs it again under the same frame number
  if (!fresh || idx == kNone) v.slots[slot].stamp = 0u;
  if (pos < v.max_blocks) {
    v.frame_list[pos] = entry;
    v.frame_src[pos] = i;
  } else {
    atomicOr(&v.cnt->error, kErrBlocks);
  }
  if (pend) {
    if (idx != kNone) v.st_pending[idx] = epoch;
    if (!fresh) v.slots[slot].listed = epoch;
    if (p < v.max_blocks) v.pending[p] = idx;
    else atomicOr(&v.cnt->error, kErrBlocks);
  }
}

// A new block's neighbour in direction l (lanes 0..26; -1: none), to be
// linked in both directions.  With forward_only, only the 13 neighbours after
// it (l > kSelf) are looked up: enough when every block present is new in the
// same call, as each pair is then linked by its first block.
__device__ inline int32_t find_neighbour(const VolDev& v, uint64_t key, int l,
                                         bool forward_only = false) {
  if (l >= 27 || l == kSelf || (forward_only && l < kSelf)) return -1;
  int x, y, z;
  unpack_key(key, x, y, z);
  const int nx = x + l % 3 - 1, ny = y + (l / 3) % 3 - 1, nz = z + l / 9 - 1;
  return key_in_range(nx, ny, nz) ? hash_find(v, pack_key(nx, ny, nz)) : -1;
}
__device__ inline void link_block(const VolDev& v, uint32_t idx, int l, int32_t nb) {
  if (nb < 0) return;
  v.nbr[(size_t)idx * 27 + l] = nb;
  v.nbr[(size_t)nb * 27 + (26 - l)] = (int32_t)idx;
}

// A new block's row q of cubes: no type (before the last extraction by the
// block's blank flag), and none of the row's edges holds a vertex (an edge's
// slot is meaningful only under its set bit, so the slots are not written).
__device__ inline void init_row(const VolDev& v, uint32_t idx, int q) {
  const size_t o = (size_t)idx * 64 + q;
  v.tcur[o] = 0;
  v.emask[o] = 0;
  if (q == 0) v.btri[idx] = 0, v.blank[idx] = 1;
}

// ============================================================================
// fusion (Eq. 2) and import
// ============================================================================
// One wave per collected block, eight voxels per lane (one column of the
// block), so that many blocks are in flight per CU.  The list entry and
// block key of the wave's next block are requested one block ahead, so a
// block waits only for its TSDF, weights and depth samples; with the
// strided mapping a wave's first item does not depend on the list length,
// and its entry and key are requested together with it (an entry past the
// length is ignored).
template <int W>
__global__ __launch_bounds__(64 * W) void k_fuse(VolDev v, FrameParams fp,
                                                 const float* __restrict__ depth, uint32_t epoch) {
  // the collection's appends: its frame list length, and (one thread) the
  // lengths the later kernels read
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool strided = (v.order & 3u) == 0u;
  const uint32_t i0 = blockIdx.x * W + (uint32_t)wave;
  uint32_t e0 = kNone;
  uint64_t k0 = 0;
  if (strided && i0 < v.max_blocks) e0 = v.frame_list[i0], k0 = v.frame_key[i0];
  const uint64_t app = v.cnt->collect_acc[fp.frame & 1];
  const uint32_t n = min(collect_frame(app), v.max_blocks);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    v.cnt->acc[VM_TOTAL_FRAME_BLOCKS] += n;
    v.cnt->n_frame[fp.frame & 1] = collect_frame(app);
    v.cnt->n_pending[epoch & 1] += collect_pend(app);
    v.cnt->n_blocks += collect_new(app);
  }
  ItemLoop it = item_loop(v, n, W, wave);
  auto entry = [&](uint32_t i) -> uint32_t { return i < it.end ? v.frame_list[i] : kNone; };
  auto key_at = [&](uint32_t i) -> uint64_t { return i < it.end ? v.frame_key[i] : 0ull; };
  // this block's entry and key
  uint32_t e1 = strided ? (it.i < it.end ? e0 : kNone) : entry(it.i);
  uint64_t k1 = strided ? k0 : key_at(it.i);
  for (; it.i < it.end; it.i += it.step) {
    const uint32_t e = uniform(e1);
    const uint64_t key = ((uint64_t)uniform((uint32_t)(k1 >> 32)) << 32) | uniform((uint32_t)k1);
    e1 = entry(it.i + it.step);
    k1 = key_at(it.i + it.step);
    if (e == kNone) continue;
    const int q = fresh_lane(), lx = q & 7, ly = q >> 3;
    const uint32_t idx = e & ~kNewFlag;
    const bool isnew = (e & kNewFlag) != 0;
    int bx, by, bz;
    unpack_key(key, bx, by, bz);
    float d[8], w[8];
    if (isnew) {
      init_row(v, idx, q);
#pragma unroll
      for (int lz = 0; lz < 8; ++lz) d[lz] = 0.f, w[lz] = 0.f;
      link_block(v, idx, q, find_neighbour(v, key, q));
    } else {
#pragma unroll
      for (int lz = 0; lz < 8; ++lz) {
        d[lz] = v.d[(size_t)idx * kVox + q + 64 * lz];
        w[lz] = v.w[(size_t)idx * kVox + q + 64 * lz];
      }
    }
    // every voxel's depth sample is requested before any is used (a voxel
    // that projects nowhere reads pixel 0 and ignores it)
    FuseProj pr[8];
    float D[8];
#pragma unroll
    for (int lz = 0; lz < 8; ++lz) {
      pr[lz] = fuse_project(v, fp, 8 * bx + lx, 8 * by + ly, 8 * bz + lz);
      D[lz] = depth[pr[lz].pix >= 0 ? pr[lz].pix : 0];
    }
    // lane lz < 8 keeps the observed, negative-TSDF and near-zero (|TSDF| <
    // eps, the refinement's test) masks of layer lz
    uint64_t mine = 0, mneg = 0, mnear = 0;
#pragma unroll
    for (int lz = 0; lz < 8; ++lz) {
      const FuseSample fs = fuse_finish(v, fp, pr[lz], D[lz]);
      const size_t o = (size_t)idx * kVox + q + 64 * lz;
      float dn = d[lz];
      if (fs.upd) {
        float num = d[lz] * w[lz];
        num = num + fs.dt;
        const float den = w[lz] + 1.0f;
        dn = num / den;
        v.d[o] = dn;
        v.w[o] = den;
      } else if (isnew) {
        v.d[o] = d[lz];
        v.w[o] = w[lz];
      }
      const uint64_t m = __ballot(fs.upd || w[lz] > 0.f), mn = __ballot(dn < 0.f);
      const uint64_t mz = __ballot(fabsf(dn) < v.eps);
      if (q == lz) mine = m, mneg = mn, mnear = mz;
    }
    if (q < 8) {
      v.wmask[(size_t)idx * 8 + q] = mine;
      v.smask[(size_t)idx * 8 + q] = mneg;
      v.nmask[(size_t)idx * 8 + q] = mnear;
    }
    if (q == 0) v.st_frame[idx] = fp.frame;
  }
}

// One wave per imported block, eight voxels per lane: the caller's rows are
// requested first, then the new block's neighbours are looked up while they
// arrive, the next block's list entry with them.  With bound arrays (the
// caller's rows are the volume's TSDF and weights) a block must land on its
// own row, and nothing is copied: the rows are read only for the
// observed-voxel, negative-TSDF and near-zero masks.
// Bound by bandwidth as long as every load is issued before the first store,
// as a load after stores waits for them, and each mask leaves in one store:
// 230,000 blocks of bound rows, which are read but not copied (6.5 KB of
// counted traffic a block), take 310 us at 4.8 TB/s, the rate of a large copy.
// With the block initialised before the lookups and one lane storing 24 mask
// words, and types of 512 bytes written per block, they took 400.  Loads past
// the caches (nontemporal) measured no gain over the step: the vertex pass
// finds fewer of these rows again.
template <int W>
__global__ __launch_bounds__(64 * W) void k_import_copy(VolDev v, const float* __restrict__ tsdf,
                                                        const float* __restrict__ weight,
                                                        uint32_t frame, int32_t* __restrict__ rows) {
  const uint32_t n = min(v.cnt->n_frame[frame & 1], v.max_blocks);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (blockIdx.x == 0 && threadIdx.x == 0) v.cnt->acc[VM_TOTAL_FRAME_BLOCKS] += n;
  // into an empty pool every neighbour is new too: link forward only
  const bool forward_only = v.cnt->import_base == 0;
  ItemLoop it = item_loop(v, n, W, wave);
  auto entry = [&](uint32_t i) -> uint32_t { return i < it.end ? v.frame_list[i] : kNone; };
  auto source = [&](uint32_t i) -> uint32_t { return i < it.end ? v.frame_src[i] : 0u; };
  uint32_t e1 = entry(it.i), r1 = source(it.i);
  for (; it.i < it.end; it.i += it.step) {
    const uint32_t e = uniform(e1), row = uniform(r1);
    e1 = entry(it.i + it.step);
    r1 = source(it.i + it.step);
    if (e == kNone) continue;
    const int q = fresh_lane();
    const uint32_t idx = e & ~kNewFlag;
    const bool isnew = (e & kNewFlag) != 0;
    if (v.bound && idx != row) {
      // refused; a new block is numbered and listed all the same, so it starts
      // as one that nothing was observed in
      if (isnew) {
        init_row(v, idx, q);
        if (q < 8) {
          const size_t o = (size_t)idx * 8 + q;
          v.wmask[o] = 0, v.smask[o] = 0, v.nmask[o] = 0;
        }
      }
      if (q == 0) atomicOr(&v.cnt->error, kErrRange);
      continue;
    }
    const uint64_t key = isnew ? v.block_key[idx] : 0ull;
    float d[8], w[8];
#pragma unroll
    for (int lz = 0; lz < 8; ++lz) {
      d[lz] = tsdf[(size_t)row * kVox + q + 64 * lz];
      w[lz] = weight[(size_t)row * kVox + q + 64 * lz];
    }
    const int32_t nb = isnew ? find_neighbour(v, key, q, forward_only) : -1;
    // lane lz < 8 keeps the masks of layer lz
    uint64_t mine = 0, mneg = 0, mnear = 0;
#pragma unroll
    for (int lz = 0; lz < 8; ++lz) {
      const uint64_t m = __ballot(w[lz] > 0.f), mn = __ballot(d[lz] < 0.f);
      const uint64_t mz = __ballot(fabsf(d[lz]) < v.eps);
      if (q == lz) mine = m, mneg = mn, mnear = mz;
    }
    if (isnew) {
      link_block(v, idx, q, nb);
      init_row(v, idx, q);
    }
    if (!v.bound) {
#pragma unroll
      for (int lz = 0; lz < 8; ++lz) {
        v.d[(size_t)idx * kVox + q + 64 * lz] = d[lz];
        v.w[(size_t)idx * kVox + q + 64 * lz] = w[lz];
      }
    }
    if (q < 8) {
      v.wmask[(size_t)idx * 8 + q] = mine;
      v.smask[(size_t)idx * 8 + q] = mneg;
      v.nmask[(size_t)idx * 8 + q] = mnear;
    }
    if (q == 0) {
      v.st_frame[idx] = frame;
      if (rows) rows[row] = (int32_t)idx;
    }
  }
}

// ============================================================================
// extraction: dirty set, classification (+ refinement), vertices, triangles
// ============================================================================

// Dirty = pending blocks and their allocated neighbours at offsets {-1,0}^3.
// Candidates (8 per pending block) are claimed through a per-block pass
// stamp and compacted tile by tile, one atomic per tile.
// The last workgroup's first wave also starts the extraction (segments,
// statistics, next list lengths): nothing else in this kernel touches them,
// and the last workgroup has the fewest candidates (usually none), so the
// chain of dependent accesses this takes runs beside the claims.
__global__ __launch_bounds__(256) void k_dirty(VolDev v, uint32_t pass, uint32_t epoch) {
  __shared__ uint32_t swave[16];
  __shared__ uint32_t sbase;
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x < 64) begin_call(v, false);
  const uint32_t np = min(v.cnt->n_pending[epoch & 1], v.max_blocks);
  if (blockIdx.x == 0 && threadIdx.x == 0) v.cnt->n_pending[(epoch + 1) & 1] = 0;
  const uint32_t total = np * 8u;
  for (uint32_t t0 = blockIdx.x * kTile; t0 < total; t0 += gridDim.x * kTile) {
    int32_t got[kTilePer];
    uint32_t cnt = 0;
#pragma unroll
    for (int k = 0; k < kTilePer; ++k) {
      const uint32_t t = t0 + threadIdx.x * kTilePer + k;
      got[k] = -1;
      if (t >= total) continue;
      const uint32_t idx = v.pending[t >> 3], o = t & 7u;
      if (idx == kNone) continue;
      const int32_t nb =
          v.nbr[(size_t)idx * 27 + nbr_dir(-(int)(o & 1), -(int)((o >> 1) & 1), -(int)(o >> 2))];
      if (nb >= 0 && atomicMax(&v.st_dirty[nb], pass) < pass) {
        got[k] = nb;
        ++cnt;
      }
    }
    uint32_t tot;
    uint32_t r = wg_scan_bits<kTileBits>(cnt, swave, &tot);  // cnt <= kTilePer
    if (tot == 0) continue;
    if (threadIdx.x == 0) sbase = atomicAdd(&v.cnt->n_dirty[v.xsel], tot);
    __syncthreads();
    r += sbase;
#pragma unroll
    for (int k = 0; k < kTilePer; ++k)
      if (got[k] >= 0) v.dirty[r++] = (uint32_t)got[k];
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_dirty_all(VolDev v, uint32_t pass) {
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x < 64) begin_call(v, false);
  const uint32_t n = min(v.cnt->n_blocks, v.max_blocks);
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    v.dirty[i] = i;
    v.st_dirty[i] = pass;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    v.cnt->n_dirty[v.xsel] = n;
    v.cnt->n_pending[0] = 0;
    v.cnt->n_pending[1] = 0;
  }
}

// refine_candidates of every type, formed by the compiler.
struct RefineTable {
  uint64_t cand[256];
};
constexpr RefineTable refine_table() {
  RefineTable r{};
  for (uint32_t t = 0; t < 256; ++t) r.cand[t] = refine_candidates(t);
  return r;
}
__device__ const RefineTable kRefineTable = refine_table();

// One wave per dirty block, four blocks per workgroup, no workgroup
// barriers: per-block work is a chain of dependent memory round trips, and
// many independent waves hide it better than one wide workgroup.  Lane q
// owns the row of eight cubes at y = q & 7, z = q >> 3.  What the cubes need
// of their corners, the block's and its +x/+y/+z halo layer (9^3), is one
// bit each, read from per-block masks that fusion and import keep (byte q of
// a block's 64 is its row q): the sign, whether the corner is observed and,
// for refinement, whether |TSDF| < eps; the TSDF itself is never read.  The
// corners' rows of nine bits go through the wave's LDS, and the eight types
// of a lane's row follow from four of them as bit planes, with no work per
// cube.  The statistics of changed cubes work on bytes (an 8 x 8 bit
// transpose), only where a row has such cubes; refinement lists the cubes it
// may change (near a corner with |TSDF| < eps and neither regular nor empty,
// found on the planes) and evaluates them one per lane.
// What bounds it is instruction issue (a wave64 vector instruction takes four
// cycles) and the chain list, neighbours, masks: with a lane per column and
// its eight types formed one by one (eight byte loads and stores each of the
// types too) a 4 mm frame's 23,000 blocks took 31.5 us with refinement; with
// rows as planes and refinement evaluated column by column in every row 26.5;
// with the cubes listed 25.7, and with the table of candidates formed by the
// compiler instead of each workgroup 23.3.
// Mode, fixed at compile time so that each keeps only its own code:
// kExtract: new cube types from the signs (Sec. V-B), previous type saved;
// kExtractRefined: the same, each new type refined by Eqs. (3)-(5) against
// the type it replaces before it is written (Sec. V-F applies the regular
// type before marching cubes); kRefine: Eqs. (3)-(5) applied to the current
// types (Sec. V-F).
// Writing a cube's new type replaces its triangles (Sec. V-D): the type
// names them and the edges they use, and a cube whose type is unchanged
// keeps them.  The blocks whose vertices must be recomputed: on extraction
// every dirty block (its edges' end points may have moved) and the
// neighbours, not dirty themselves, that own edges of changed cubes on its
// +x/+y/+z faces, appended to a short list; on refinement the owners of the
// edges of changed cubes (this block and neighbours), claimed once per pass
// and written as candidates at fixed positions 8i..8i+7 for compaction.
template <int W, int refine>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(8))) void k_classify(VolDev v, uint32_t pass) {
  __shared__ uint32_t srow_all[W][81];  // corner rows: signs | observed << 9 | near << 18
  // per cube type: its triangles and, for refinement, its regular-type candidates
  __shared__ uint8_t sntri[256];
  __shared__ uint32_t scand_lo[refine ? 256 : 1], scand_hi[refine ? 256 : 1];
  // refinement's cubes (row << 3 | x), the rows' types they compare with (and
  // their own for kRefine), and what changes
  __shared__ uint16_t slist_all[refine ? W : 1][refine ? kVox : 1];
  __shared__ uint2 sprev_all[refine ? W : 1][64], scur_all[refine == 1 ? W : 1][64];
  __shared__ uint2 sflip_all[refine ? W : 1][64];
  // with the strided mapping the wave's first block is requested at once,
  // before the list length (an entry past the length is ignored)
  const bool strided = (v.order & 3u) == 0u;
  const uint32_t i0 = blockIdx.x * W + (threadIdx.x >> 6);
  const uint32_t d0 = strided && i0 < v.max_blocks ? v.dirty[i0] : kNone;
  for (int j = threadIdx.x; j < 256; j += blockDim.x) {
    sntri[j] = v.tri_table[j * 16];
    if (refine) {
      const uint64_t c = kRefineTable.cand[j];
      scand_lo[j] = (uint32_t)c;
      scand_hi[j] = (uint32_t)(c >> 32);
    }
  }
  __syncthreads();
  auto refined = [&](uint32_t t, uint32_t prev, uint32_t near8) -> uint32_t {
    const uint64_t cand = (uint64_t)scand_hi[t] << 32 | scand_lo[t];
    return refine_type(t, prev, (scand_hi[prev] >> 31) != 0u, near8, cand);
  };
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* srow = srow_all[wave];
  uint16_t* slist = slist_all[refine ? wave : 0];
  uint2 *sprev = sprev_all[refine ? wave : 0], *scur = scur_all[refine == 1 ? wave : 0];
  uint2* sflip = sflip_all[refine ? wave : 0];
  const uint8_t* smask = reinterpret_cast<const uint8_t*>(v.smask);
  const uint8_t* wmask = reinterpret_cast<const uint8_t*>(v.wmask);
  const uint8_t* nmask = reinterpret_cast<const uint8_t*>(v.nmask);
  // row r of the corners of block b0 (bits 0..7) and of its +x neighbour b1
  // (bit 8), a missing block's being neither negative nor observed
  auto corner_row = [&](int32_t b0, int32_t b1, uint32_t r) -> uint32_t {
    uint32_t c = 0;
    if (b0 >= 0) {
      const size_t o = (size_t)b0 * 64 + r;
      c = (uint32_t)smask[o] | (uint32_t)wmask[o] << 9 | (refine ? (uint32_t)nmask[o] << 18 : 0u);
    }
    if (b1 >= 0) {
      const size_t o = (size_t)b1 * 64 + r;
      c |= (smask[o] & 1u) << 8 | (wmask[o] & 1u) << 17 | (refine ? (nmask[o] & 1u) << 26 : 0u);
    }
    return c;
  };
  const uint32_t n = min(v.cnt->n_dirty[v.xsel], v.max_blocks);
  if (blockIdx.x == 0 && threadIdx.x == 0) v.cnt->acc[VM_TOTAL_DIRTY_BLOCKS] += n;
  for (ItemLoop it = item_loop(v, n, W, wave); it.i < it.end; it.i += it.step) {
    // lane addressing is formed again per block (fewer registers)
    const int q = fresh_lane(), y = q & 7, z = q >> 3;
    const uint32_t i = it.i;
    const uint32_t idx = uniform(strided && i == i0 ? d0 : v.dirty[i]);
    const int32_t mynb = q < 8 ? v.nbr[(size_t)idx * 27 + nbr_dir(q & 1, (q >> 1) & 1, q >> 2)] : -1;
    // the row's own types and corners, independent of the neighbours (the
    // previous applied types only for refinement)
    uint2* cur = reinterpret_cast<uint2*>(v.tcur + (size_t)idx * 64);
    uint2* before = reinterpret_cast<uint2*>(v.tprev + (size_t)idx * 64);
    const uint2 old = cur[q];
    uint2 prev = make_uint2(0u, 0u);
    if (refine == 1) {
      const uint2 kept = before[q];
      if (v.blank[idx] == 0u) prev = kept;
    }
    // row (y, z), y and z in 0..8, lies at y + 9 z: the lane's own, and for
    // lanes 0..16 one of the +y face (y = 8), the +z face (z = 8) or the edge
    // between them
    uint32_t r00 = corner_row((int32_t)idx, -1, (uint32_t)q);
    r00 |= corner_row(-1, __builtin_amdgcn_readlane(mynb, 1), (uint32_t)q);
    {
      const int dir = q < 8 ? 2 : (q < 16 ? 4 : 6);
      const int32_t h0 = __shfl(mynb, dir), h1 = __shfl(mynb, dir | 1);
      if (q < 17)
        srow[q < 8 ? 8 + 9 * q : 64 + q] =
            corner_row(h0, h1, q < 8 ? 8u * (uint32_t)q : (q < 16 ? (uint32_t)q - 8u : 0u));
    }
    srow[y + 9 * z] = r00;
    wave_sync();
    const uint32_t r10 = srow[y + 1 + 9 * z], r01 = srow[y + 9 * z + 9], r11 = srow[y + 10 + 9 * z];
    // cubes with all eight corners observed, and the row's types
    const uint32_t seen = r00 & r10 & r01 & r11;
    const uint32_t valid = (seen >> 9) & (seen >> 10) & 0xFFu;
    auto planes = [&](uint32_t ra, uint32_t rb, uint32_t m) -> uint32_t {
      return (ra & m) | ((ra >> 1) & m) << 8 | ((rb >> 1) & m) << 16 | (rb & m) << 24;
    };
    uint32_t lo = planes(r00, r10, valid), hi = planes(r01, r11, valid);
    uint32_t nrefined = 0;
    if (refine == 1) lo = old.x, hi = old.y;
    if (refine) {
      // a block lists 512 cubes at most
      const uint32_t rn = (r00 | r10 | r01 | r11) >> 18;
      const uint32_t act = valid & (rn | rn >> 1) & refinable_cubes(lo, hi);
      uint32_t cnt, at = wave_prefix_bits<4>((uint32_t)__popc(act), &cnt);
      if (cnt) {
        for (uint32_t m = act; m; m &= m - 1u)
          slist[at++] = (uint16_t)((uint32_t)q << 3 | (uint32_t)__builtin_ctz(m));
        sprev[q] = refine == 1 ? prev : old;
        if (refine == 1) scur[q] = old;
        sflip[q] = make_uint2(0u, 0u);
        wave_sync();
        uint32_t changed = 0;
        for (uint32_t i0 = 0; i0 < cnt; i0 += 64) {
          const bool on = i0 + q < cnt;
          const uint32_t item = slist[on ? i0 + q : 0u], row = item >> 3, x = item & 7u;
          const uint32_t* c = srow + (row & 7u) + 9u * (row >> 3);
          const uint32_t c00 = c[0], c10 = c[1], c01 = c[9], c11 = c[10];
          const uint2 pw = sprev[row];
          const uint2 tw = refine == 1 ? scur[row] : make_uint2(0u, 0u);
          const uint32_t t = refine == 1 ? planes_type(tw.x, tw.y, x) : corner_bits(c00, c10, c01, c11, x);
          const uint32_t r = refined(t, planes_type(pw.x, pw.y, x), corner_bits(c00, c10, c01, c11, x + 18u));
          const bool flips = on && r != t;
          const uint64_t bf = __ballot(flips);
          if (bf == 0ull) continue;
          changed += (uint32_t)__popcll(bf);
          if (flips) {
            const uint32_t f = t ^ r;
            atomicXor(&sflip[row].x, planes_flip(f, x));
            atomicXor(&sflip[row].y, planes_flip(f >> 4, x));
          }
        }
        if (changed) {
          wave_sync();
          const uint2 f = sflip[q];
          lo ^= f.x, hi ^= f.y;
          if (refine == 2) nrefined = changed;
        }
      }
    }
    if (refine != 1) {
      // the types to keep for a refinement: a block that had none says so in
      // one word instead of 512 bytes (of a batch's 230,000 new blocks that
      // is every one: 148 -> 131 us here and 362 -> 344 in the import)
      const bool none = __ballot((old.x | old.y) != 0u) == 0ull;
      if (!none) before[q] = old;
      if (q == 0) v.blank[idx] = none;
    }
    uint32_t chg = (lo ^ old.x) | (hi ^ old.y);
    chg |= chg >> 16;
    chg = (chg | chg >> 8) & 0xFFu;
    if (chg) cur[q] = make_uint2(lo, hi);
    // an unchanged cube keeps its triangles: only changed ones count
    const uint32_t tri_old = surface_cubes(old.x, old.y), tri_new = surface_cubes(lo, hi);
    const uint32_t tc = chg & (tri_old | tri_new);
    const uint64_t rows = __ballot(tc != 0u);
    uint32_t wflags = refine == 1 ? 0u : 1u, nchanged = 0;
    uint32_t cnew = 0, cold = 0, fnew = 0, fold = 0;
    if (rows) {
      // owners of the changed cubes' edges: this block and, on its +x/+y/+z
      // faces, the neighbours (never the +x+y+z corner one)
      const uint64_t rx = __ballot((tc & 0x80u) != 0u);
      constexpr uint64_t kY = 0x8080808080808080ull, kZ = 0xFF00000000000000ull;
      wflags = 1u | (rx ? 2u : 0u) | (rows & kY ? 4u : 0u) | (rx & kY ? 8u : 0u) |
               (rows & kZ ? 16u : 0u) | (rx & kZ ? 32u : 0u) | (rows & kY & kZ ? 64u : 0u);
      uint32_t ol = old.x, oh = old.y, nl = lo, nh = hi;
      transpose8(ol, oh);
      transpose8(nl, nh);
      for (uint32_t m = tc; m; m &= m - 1u) {
        const int x = __builtin_ctz(m), sh = 8 * (x & 3);
        fold += sntri[((x & 4 ? oh : ol) >> sh) & 255u];
        fnew += sntri[((x & 4 ? nh : nl) >> sh) & 255u];
      }
      // per lane at most 8 cubes of at most 5 triangles
      nchanged = wave_sum_bits<4>((uint32_t)__popc(tc));
      cnew = wave_sum_bits<4>((uint32_t)__popc(tc & tri_new));
      cold = wave_sum_bits<4>((uint32_t)__popc(tc & tri_old));
      fnew = wave_sum_bits<6>(fnew);
      fold = wave_sum_bits<6>(fold);
    }
    if (refine != 1) {
      // extraction: the vertex pass walks every dirty block, this one
      // included; a +x/+y/+z neighbour that owns edges of changed cubes and
      // is not dirty itself joins as an extra block, claimed once per pass
      // and appended with one atomic per wave
      bool extra = false;
      if (q >= 1 && q < 8 && ((wflags >> q) & 1u) && mynb >= 0)
        extra = v.st_dirty[mynb] != pass && v.st_vtx[mynb] != pass &&
                atomicMax(&v.st_vtx[mynb], pass) < pass;
      const uint64_t be = __ballot(extra);
      if (be) {
        uint32_t b0 = 0;
        if (q == 0) b0 = atomicAdd(&v.cnt->n_vblocks[v.vsel], (uint32_t)__popcll(be));
        const uint32_t pos = uniform(b0) + mask_rank(be);
        if (extra) {
          if (pos < v.max_blocks) v.vblocks[pos] = (uint32_t)mynb;
          else atomicOr(&v.cnt->error, kErrBlocks);
        }
      }
    } else if (q < 8) {
      uint32_t out = kNone;
      if ((wflags >> q) & 1u) {
        const int32_t nb = q == 0 ? (int32_t)idx : mynb;
        if (nb >= 0 && v.st_vtx[nb] != pass && atomicMax(&v.st_vtx[nb], pass) < pass)
          out = (uint32_t)nb;
      }
      v.vcand[(size_t)i * 8 + q] = out;
    }
    if (q == 0 && (nchanged | nrefined)) {
      Seg& cs = v.cseg[idx % v.nseg];
      auto add2 = [](uint32_t* w, uint32_t a, uint32_t b) {
        atomicAdd(reinterpret_cast<unsigned long long*>(w),
                  (unsigned long long)a | (unsigned long long)b << 32);
      };
      if (refine == 1) atomicAdd(&cs.st_pass, nchanged);
      else add2(&cs.st_chg, nchanged, nrefined);
      if (cnew | cold) add2(&cs.st_cnew, cnew, cold);
      if (fnew | fold) {
        add2(&cs.st_fnew, fnew, fold);
        atomicAdd(&v.btri[idx], fnew - fold);
      }
    }
    wave_sync();
  }
}

// Compact the vertex-block candidates a refinement wrote (8 per dirty
// block, already claimed), one atomic per tile.
// The candidate list is 8 entries per dirty block and mostly empty, and
// can be long (every block of a large import), so each lane takes 8 entries
// (coalesced: entry k of a lane sits k * 256 past the first) and a tile of
// 2048 entries costs one atomic on the list length.
// As in k_dirty, the last workgroup's first wave starts the call for the
// vertex pass that follows.
constexpr int kVbPer = 8;
__global__ __launch_bounds__(256) void k_vblock_compact(VolDev v) {
  __shared__ uint32_t swave[16];
  __shared__ uint32_t sbase;
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x < 64) begin_call(v, true);
  const uint32_t n = min(v.cnt->n_dirty[v.xsel], v.max_blocks);
  const uint32_t total = n * 8u;
  constexpr uint32_t kT = 256 * kVbPer;
  for (uint32_t t0 = blockIdx.x * kT; t0 < total; t0 += gridDim.x * kT) {
    uint32_t got[kVbPer], cnt = 0;
#pragma unroll
    for (int k = 0; k < kVbPer; ++k) {
      const uint32_t t = t0 + k * 256 + threadIdx.x;
      got[k] = t < total ? v.vcand[t] : kNone;
      cnt += got[k] != kNone;
    }
    uint32_t tot;
    uint32_t r = wg_scan_bits<count_bits(kVbPer)>(cnt, swave, &tot);
    if (tot == 0) continue;
    if (threadIdx.x == 0) sbase = atomicAdd(&v.cnt->n_vblocks[v.vsel], tot);
    __syncthreads();
    r += sbase;
#pragma unroll
    for (int k = 0; k < kVbPer; ++k)
      if (got[k] != kNone) v.vblocks[r++] = got[k];
    __syncthreads();
  }
}

// Which of the eight blocks whose cubes touch a block's edges have triangles:
// bit k stands for the neighbour at -(k & 1), -(k >> 1 & 1), -(k >> 2).  The
// cubes of the others are of types 0 and 255, which use no edge.  mynb: the
// block's neighbour table, lanes 0..26.
__device__ inline uint32_t surface_around(const VolDev& v, int32_t mynb) {
  const int q = __lane_id();
  const int32_t nb = __shfl(mynb, kSelf - (q & 1) - 3 * ((q >> 1) & 1) - 9 * ((q >> 2) & 1));
  return (uint32_t)__ballot(q < 8 && nb >= 0 && v.btri[nb] != 0u);
}

// One wave per listed block.  Each voxel owns the edges from it along +x,
// +y, +z.  The reference count of an edge is the number of triangles, over
// the four cubes around it, that use it; a positive count needs a vertex
// (created here on first use, Sec. V-C), whose parameter t is rewritten
// from the end point TSDF values when either end point may have changed
// since the last extraction.  Counts are formed, never stored, and the pass
// needs only whether they are positive: a cube uses an edge exactly when its
// type differs at the edge's ends, so a lane forms, for its row of eight
// cubes at once (bit planes), which edges around it they use (row_edges),
// and a voxel row's edges are an OR over four rows of cubes, exchanged
// through LDS with the -x/-y/-z halo.  Which edges hold a vertex is one
// 24-bit word per lane (bit 8a + x), read at the start and written back when
// it changes.  New
// vertices take slots from the block's pool segment, one atomic per block,
// and the recycled slots it takes are fetched in one batch.  The edges with
// work (a vertex to create, to free, or to move) are listed in LDS row by
// row, each lane's place from a prefix sum of the lanes' counts, so that
// neighbouring edges' parameters and slots share a cache line; the
// write pass runs over that list, 64 edges per step, in chunks of kWorkCap
// edges.  Each chunk first requests everything it reads, the freed
// vertices' slots and the end point TSDF values of the others, and only
// then stores: on this hardware a load issued after stores waits for them
// too.  A block with no vertex and no cube with triangles around its edges
// (one in free space) stops there.
// Bound by instruction issue: summing the counts from a table of edge uses
// per cube type, a column of cubes per lane, it took 14.2 us for an 8 mm
// frame's 5,700 blocks and 39 us for a 4 mm frame's 23,000; with rows as
// planes 12.7 and 33.7, and with list entries of one operation each, a write
// pass without branches per edge and sums only where something changes 11.7
// and 31.0.
constexpr int kRingBatch = 256;  // recycled slots fetched per block at once
constexpr int kWorkCap = 512;    // listed edges per chunk of the write pass

template <int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(6))) void k_vertices(VolDev v, uint32_t moved, int walk_dirty) {
  __shared__ uint32_t st_all[W][kRingBatch];  // edges used per row of cubes at -1..7, then slots
  __shared__ uint32_t swork_all[W][kWorkCap]; // row q << 5 | edge's bit 8a + x
  __shared__ int32_t snb_all[W][27];
  static_assert(kRingBatch >= 2 * 81, "the rows' edges fit the slot batch");
  // the blocks: after an extraction the dirty list and then the extra
  // blocks classification appended; after a refinement the compacted list
  const uint32_t nd = walk_dirty ? min(v.cnt->n_dirty[v.xsel], v.max_blocks) : 0u;
  const uint32_t n = nd + min(v.cnt->n_vblocks[v.vsel], v.max_blocks);
  if (blockIdx.x == 0 && threadIdx.x == 0) v.cnt->acc[VM_TOTAL_VERTEX_BLOCKS] += n;
  // many blocks per wave: the pass is bound by what it reads, and the types
  // of a block without triangles are not asked for (where it has none around
  // and no vertex, the block is done); with one block per wave asking first
  // only lengthens the chain of a list whose blocks mostly have triangles.
  // Without / with asking first, us: the 23,000 blocks of a 4 mm frame 34.5 /
  // 35.6; blocks of 160 vertices 45,000 253 / 259, 66,000 394 / 395, 230,000
  // 1,473 / 1,473; of 39 vertices 23,000 36 / 35, 66,000 133 / 125, 230,000
  // 483 / 459; mostly free space 23,000 20 / 18, 66,000 52 / 44, 230,000 171 /
  // 134.  From this line on (65,536 with the default mapping) asking is behind
  // nowhere.
  const bool long_list = n > 4u * gridDim.x * W;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* snext = st_all[wave];  // row (y, z) of cubes, y and z in -1..7, at (y + 1) + 9 (z + 1)
  uint32_t* sdiag = st_all[wave] + 81;
  uint32_t* sring = st_all[wave];
  uint32_t* swork = swork_all[wave];
  int32_t* snb = snb_all[wave];
  for (ItemLoop it = item_loop(v, n, W, wave); it.i < it.end; it.i += it.step) {
    // lane addressing is formed again per block rather than held in
    // registers across the loop
    const int q = fresh_lane(), y = q & 7, z = q >> 3;
    const uint32_t idx = uniform(it.i < nd ? v.dirty[it.i] : v.vblocks[it.i - nd]);
    const uint32_t sg = uniform(idx % v.nseg);
    // the block's edge arrays, addressed by block-local edge a * 512 + l;
    // pool arrays by 32-bit byte offsets from their bases (every index here
    // is below 2^30 entries of 4 bytes)
    const size_t eb = (size_t)idx * (3 * kVox);
    int32_t* evtx_b = v.evtx + eb;
    float* et_b = v.et + eb;
    auto pool32 = [](uint32_t* base, uint32_t s) -> uint32_t& {
      return *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base) + s * 4u);
    };
    // requested at once: the neighbour table, which edges hold a vertex,
    // the row's cube types and the block's pool segment (fixed during this
    // kernel)
    const int32_t mynb = q < 27 ? v.nbr[(size_t)idx * 27 + q] : -1;
    const uint32_t has = v.emask[(size_t)idx * 64 + q];
    uint32_t with = 0xFFu;  // the blocks around whose types are asked for
    if (long_list) {
      with = surface_around(v, mynb);
      if (with == 0u && __ballot(has != 0u) == 0ull) continue;
    }
    auto types_at = [&](int32_t blk, uint32_t r, uint32_t ask) -> uint2 {
      return blk >= 0 && ask ? reinterpret_cast<const uint2*>(v.tcur)[(size_t)blk * 64 + r]
                      : make_uint2(0u, 0u);
    };
    const uint2 own = types_at((int32_t)idx, (uint32_t)q, with & 1u);
    const Seg& g = v.vseg[sg];
    const uint32_t head = g.head, count = g.count, hwm = g.hwm;
    if (q < 27) snb[q] = mynb;
    // the -x neighbour's row; for lanes 0..16 a row of the -y face (lanes
    // 0..7), of the -z face (8..15) or of the edge between them, with its -x
    // neighbour's
    const uint2 ownx = types_at(__builtin_amdgcn_readlane(mynb, nbr_dir(-1, 0, 0)), (uint32_t)q, with & 2u);
    uint2 halo = make_uint2(0u, 0u), halox = halo;
    {
      const int dir = q < 8 ? nbr_dir(0, -1, 0) : (q < 16 ? nbr_dir(0, 0, -1) : nbr_dir(0, -1, -1));
      const uint32_t r = q < 8 ? 7u + 8u * (uint32_t)q : (q < 16 ? 48u + (uint32_t)q : 63u);
      const int32_t h = __shfl(mynb, dir), hx = __shfl(mynb, dir - 1);
      const uint32_t at = with >> (q < 8 ? 2 : (q < 16 ? 4 : 6));
      if (q < 17) halo = types_at(h, r, at & 1u), halox = types_at(hx, r, at & 2u);
    }
    uint32_t mv = 0xFFFFFFu;  // edges whose end points may have moved (bit 8a + x)
    if (moved != kMovedAll) {
      // after an extraction of pending blocks: which of this block and its
      // +x/+y/+z neighbours were pending
      const bool pend = q < 27 && mynb >= 0 && v.st_pending[mynb] == moved;
      const uint64_t pm = __ballot(pend);
      if (!((pm >> kSelf) & 1u)) {
        mv = (((pm >> nbr_dir(1, 0, 0)) & 1u) ? 0x80u : 0u) |
             (y == 7 && ((pm >> nbr_dir(0, 1, 0)) & 1u) ? 0xFF00u : 0u) |
             (z == 7 && ((pm >> nbr_dir(0, 0, 1)) & 1u) ? 0xFF0000u : 0u);
      }
    }
    // edges with a positive count, bit 8a + x
    uint32_t R, next, diag;
    if (q < 17) {
      (void)row_edges(halo.x, halo.y, halox.x, halox.y, &next, &diag);
      const int at = q < 8 ? 9 * (q + 1) : (q < 16 ? q - 7 : 0);
      snext[at] = next;
      sdiag[at] = diag;
    }
    R = row_edges(own.x, own.y, ownx.x, ownx.y, &next, &diag);
    snext[(y + 1) + 9 * (z + 1)] = next;
    sdiag[(y + 1) + 9 * (z + 1)] = diag;
    wave_sync();
    {
      const uint32_t back_y = snext[y + 9 * (z + 1)], back_z = snext[(y + 1) + 9 * z] >> 16;
      R |= (back_y & 0xFFu) | (back_y & 0xFF00u) << 8 | back_z | sdiag[y + 9 * z];
    }
    // no cube around the block's edges has triangles and no edge holds a
    // vertex: every count stays zero and there is nothing to write (about a
    // third of the blocks of a frame of the room sequence lie in free space)
    if (__ballot((has | R) != 0u) == 0ull) {
      wave_sync();
      continue;
    }
    const uint32_t need = R & ~has, freed = has & ~R, kept = R & has;
    const uint32_t work = need | freed | (kept & mv);
    // one atomic per block takes its allocations and its places for frees; a
    // vertex whose count dropped to zero goes back to the segment's ring
    // at once (Sec. V-E), where it can be taken again once the ring is
    // closed, never by this pass
    // per lane at most 24 of each (three edges of eight voxels)
    uint32_t total = 0, tfree = 0;
    if (__ballot((need | freed) != 0u)) {
      total = wave_sum_bits<5>((uint32_t)__popc(need));
      tfree = wave_sum_bits<5>((uint32_t)__popc(freed));
    }
    uint32_t nwork;
    const uint32_t wpos = wave_prefix_bits<5>((uint32_t)__popc(work), &nwork);
    uint32_t base = 0, fbase = 0;
    if (q == 0) {
      if (total | tfree) {
        const unsigned long long b =
            atomicAdd(reinterpret_cast<unsigned long long*>(&v.vseg[sg].ticket),
                      (unsigned long long)total | (unsigned long long)tfree << 32);
        base = (uint32_t)b, fbase = (uint32_t)(b >> 32);
      }
    }
    base = uniform(base);
    fbase = uniform(fbase);
    const uint32_t gbase = sg * v.vseg_cap, gsize = seg_size(sg, v.vseg_cap, v.max_vertices);
    const uint32_t rtail = ring_pos(head, count, gsize);  // where pushes start
    // the slots of the first kRingBatch allocations, fetched together (the
    // rows' edges are no longer needed: the batch reuses their LDS)
    wave_sync();
    const uint32_t batch = min(total, (uint32_t)kRingBatch);
    for (uint32_t k = q; k < batch; k += 64)
      sring[k] = seg_slot(head, count, hwm, base + k, v.vring, gbase, gsize);
    // slot of allocation k of this block (k counted from 0)
    auto new_slot = [&](uint32_t k) -> uint32_t {
      return k < batch ? sring[k] : seg_slot(head, count, hwm, base + k, v.vring, gbase, gsize);
    };
    // the edge's vertex is no longer used: back to the ring (k-th free of
    // this block).  Only slots that were handed out come back (an edge whose
    // allocation failed holds no vertex), so the ring never runs over.
    auto free_vertex = [&](uint32_t s, uint32_t k) {
      pool32(v.vring, gbase + ring_pos(rtail, fbase + k, gsize)) = s;
      pool32(v.vowner, s) = kNone;
    };
    uint32_t nfail = 0, knew = 0, kfree = 0;  // tickets beyond a full segment; placed so far
    uint32_t lost = 0;  // the row's edges whose allocation failed (bit 8a + x)
    // the blocks with the longest write pass finish last and so set the
    // kernel's end: their waves take issue priority over the others on the
    // SIMD until their writes are done
    if (nwork > 128u) __builtin_amdgcn_s_setprio(2);
    for (uint32_t c0 = 0; c0 < nwork; c0 += kWorkCap) {
      // the lane's items of this chunk, at its place in the list
      wave_sync();
      if (nwork <= (uint32_t)kWorkCap) {
        uint32_t* p = swork + wpos;
        for (uint32_t rem = work; rem; rem &= rem - 1u)
          *p++ = (uint32_t)q << 5 | (uint32_t)__builtin_ctz(rem);
      } else {
        uint32_t p = wpos - c0;
        for (uint32_t rem = work; rem; rem &= rem - 1u, ++p)
          if (p < (uint32_t)kWorkCap) swork[p] = (uint32_t)q << 5 | (uint32_t)__builtin_ctz(rem);
      }
      wave_sync();
      const uint32_t m = min(nwork - c0, (uint32_t)kWorkCap);
      // the chunk's loads: per item of the lane the TSDF at its edge's two end
      // points (the far one in the +axis neighbour when the owner sits on the
      // block's +axis face) and, where the step frees any, the vertex's slot
      constexpr int kSteps = kWorkCap / 64;
      uint32_t edge[kSteps];  // a * 512 + l | count > 0 << 11 | has vertex << 12
      uint32_t fslot[kSteps];
      float da[kSteps], db[kSteps];
#pragma unroll
      for (int k = 0; k < kSteps; ++k) {
        edge[k] = 0u;
        fslot[k] = 0u;
        da[k] = db[k] = 0.f;
        if (64u * (uint32_t)k < m) {
          const uint32_t item = swork[min(64u * (uint32_t)k + q, m - 1u)];
          const uint32_t row = item >> 5, bit = item & 31u, a = bit >> 3;
          const uint32_t used = (uint32_t)__shfl((int)R, (int)row) >> bit & 1u;
          const uint32_t held = (uint32_t)__shfl((int)has, (int)row) >> bit & 1u;
          const uint32_t l = row << 3 | (bit & 7u);
          edge[k] = a << 9 | l | used << 11 | held << 12;
          const bool face = ((l >> (3u * a)) & 7u) == 7u;
          const uint32_t stp = 1u << (3u * a);
          const int32_t fb = snb[kSelf + (face ? (0x931u >> (4u * a)) & 15u : 0u)];
          const uint32_t fl = l + stp - (face ? 8u * stp : 0u);
          da[k] = v.d[(size_t)idx * kVox + l];
          const float far = v.d[(size_t)(uint32_t)(fb >= 0 ? fb : (int32_t)idx) * kVox + fl];
          db[k] = fb >= 0 ? far : 0.f;
          if (__ballot(used == 0u)) fslot[k] = used ? 0u : (uint32_t)evtx_b[edge[k] & 2047u];
        }
      }
#pragma unroll
      for (int k = 0; k < kSteps; ++k) {
        const uint32_t i0 = 64u * (uint32_t)k;
        if (i0 >= m) break;
        const bool act = i0 + q < m;
        const uint32_t e = edge[k] & 2047u;
        const bool cnt = (edge[k] >> 11) & 1u, hv = (edge[k] >> 12) & 1u;
        const bool is_new = act && cnt && !hv, is_free = act && !cnt;
        bool place = act && cnt;
        if (total | tfree) {
          const uint64_t bn = __ballot(is_new), bf = __ballot(is_free);
          if (is_new) {
            const uint32_t ns = new_slot(mask_rank(bn, knew));
            if (ns == kNone) {
              // segment full: the edge stays without a vertex, its triangles
              // reference none (slot -1), and the next pass that visits the
              // block asks for one again
              atomicOr(&v.cnt->error, kErrVertices);
              evtx_b[e] = -1;
              place = false;
            } else {
              evtx_b[e] = (int32_t)ns;
              pool32(v.vowner, ns) = (uint32_t)eb + e;
              pool32(v.vbirth, ns) = v.frame;
            }
          }
          if (is_free) free_vertex(fslot[k], mask_rank(bf, kfree));
          knew += (uint32_t)__popcll(bn);
          kfree += (uint32_t)__popcll(bf);
          const uint64_t bl = __ballot(is_new && !place);
          nfail += (uint32_t)__popcll(bl);
          for (uint64_t rem = bl; rem; rem &= rem - 1ull) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)e, __builtin_ctzll(rem));
            if ((uint32_t)q == ((x >> 3) & 63u)) lost |= 1u << ((x >> 9) * 8u + (x & 7u));
          }
        }
        if (place) et_b[e] = edge_param(da[k], db[k]);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    const uint32_t now = R & ~lost;
    if (now != has) v.emask[(size_t)idx * 64 + q] = now;
    const uint32_t nupd = wave_sum_bits<5>((uint32_t)__popc(kept));
    const uint32_t nmov =
        __ballot((kept & ~mv) != 0u) ? wave_sum_bits<5>((uint32_t)__popc(kept & mv)) : nupd;
    if (q == 0) {
      if (nupd | nmov)
        atomicAdd(reinterpret_cast<unsigned long long*>(&v.vseg[sg].st_upd),
                  (unsigned long long)nupd | (unsigned long long)nmov << 32);
      // (tickets beyond a full segment are no new vertices)
      if (nfail) atomicSub(&v.vseg[sg].st_new, nfail);
    }
    wave_sync();
  }
}

// Owner of each cube edge: offset from the cube's anchor voxel and axis,
// packed as ox | oy << 1 | oz << 2 | axis << 3.
// e0 (000,x) e1 (100,y) e2 (010,x) e3 (000,y) e4 (001,x) e5 (101,y)
// e6 (011,x) e7 (001,y) e8 (000,z) e9 (100,z) e10 (110,z) e11 (010,z)
__device__ inline void edge_owner(int e, int& ox, int& oy, int& oz, int& axis) {
  static constexpr uint8_t kOwn[12] = {0, 9, 2, 8, 4, 13, 6, 12, 16, 17, 19, 18};
  const uint32_t p = kOwn[e];
  ox = (int)(p & 1u);
  oy = (int)((p >> 1) & 1u);
  oz = (int)((p >> 2) & 1u);
  axis = (int)(p >> 3);
}

// ============================================================================
// ablation: the paper's two ways of sharing vertices between cubes
// ============================================================================
// Sec. V-C gives two GPU schemes that initialise each vertex once while the
// cubes around its edge run in parallel, and Sec. VI-A times them against
// each other.  These kernels reproduce both, for measurement beside edge
// ownership, on the cubes of the last extraction's dirty blocks, one lane
// per cube: for every edge its type uses, a vertex is allocated (one atomic
// on a global counter, as from a heap) if the edge has none, and the edge
// parameter t is written.  The state is the caller's: slot[e] (-1: none) and
// t[e], e = (block * 3 + axis) * 512 + voxel, kept across calls.

// Index of the owner edge of cube-edge e of cube l in block idx, -1 when the
// owner block is not allocated; t receives its parameter.
__device__ inline int64_t cube_edge_slot_index(const VolDev& v, uint32_t idx, int l, int e,
                                               float& t) {
  int ox, oy, oz, axis;
  edge_owner(e, ox, oy, oz, axis);
  const int x = (l & 7) + ox, y = ((l >> 3) & 7) + oy, z = (l >> 6) + oz;
  const int32_t nb = v.nbr[(size_t)idx * 27 + nbr_dir(x >> 3, y >> 3, z >> 3)];
  const int fx = x + (axis == 0), fy = y + (axis == 1), fz = z + (axis == 2);
  const int32_t fb = v.nbr[(size_t)idx * 27 + nbr_dir(fx >> 3, fy >> 3, fz >> 3)];
  if (nb < 0 || fb < 0) return -1;
  const int ol = (x & 7) + 8 * (y & 7) + 64 * (z & 7);
  t = edge_param(v.d[(size_t)nb * kVox + ol],
                 v.d[(size_t)fb * kVox + (fx & 7) + 8 * (fy & 7) + 64 * (fz & 7)]);
  return ((int64_t)nb * 3 + axis) * kVox + ol;
}

// Lock-based: the first lane to take an edge (compare-and-swap from -1)
// allocates its vertex; every lane using the edge writes the same t.
__global__ __launch_bounds__(256) void k_share_lock(VolDev v, int32_t* __restrict__ slot,
                                                    float* __restrict__ tv,
                                                    uint32_t* __restrict__ counter) {
  const uint32_t n = min(v.cnt->n_dirty[v.xsel], v.max_blocks) * kVox;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t idx = v.dirty[i / kVox];
    const int l = (int)(i % kVox);
    const uint32_t type = cube_type(v.tcur, idx, l);
    if (v.tri_table[type * 16] == 0) continue;
    for (int e = 0; e < 12; ++e) {
      if (!v.edge_uses[type * 12 + e]) continue;
      float t;
      const int64_t eo = cube_edge_slot_index(v, idx, l, e, t);
      if (eo < 0) continue;
      if (atomicCAS(&slot[eo], -1, -2) == -1) slot[eo] = (int32_t)atomicAdd(counter, 1u);
      tv[eo] = t;
    }
  }
}

// Lock-free: the cubes of each 2x2x2 cell form four groups of two at
// opposite corners (parities 000/111, 100/011, 010/101, 001/110); no two
// cubes of a group share an edge, so within one launch a lane allocates
// without any claim.  The four groups are four launches.
__global__ __launch_bounds__(256) void k_share_free(VolDev v, int group,
                                                    int32_t* __restrict__ slot,
                                                    float* __restrict__ tv,
                                                    uint32_t* __restrict__ counter) {
  const uint32_t n = min(v.cnt->n_dirty[v.xsel], v.max_blocks) * 128u;
  const int first = group == 0 ? 0 : (1 << (group - 1));  // parity x | y << 1 | z << 2
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t idx = v.dirty[i / 128u];
    const int k = (int)(i % 128u), cell = k & 63;
    const int p = (k >> 6) ? first ^ 7 : first;
    const int x = 2 * (cell & 3) + (p & 1), y = 2 * ((cell >> 2) & 3) + ((p >> 1) & 1),
              z = 2 * (cell >> 4) + (p >> 2);
    const int l = x + 8 * y + 64 * z;
    const uint32_t type = cube_type(v.tcur, idx, l);
    if (v.tri_table[type * 16] == 0) continue;
    for (int e = 0; e < 12; ++e) {
      if (!v.edge_uses[type * 12 + e]) continue;
      float t;
      const int64_t eo = cube_edge_slot_index(v, idx, l, e, t);
      if (eo < 0) continue;
      if (slot[eo] < 0) slot[eo] = (int32_t)atomicAdd(counter, 1u);
      tv[eo] = t;
    }
  }
}

// ============================================================================
// download: counts, then vertices and triangles in pool order
// ============================================================================
__device__ inline bool slot_in_use(const Seg* seg, uint32_t cap, uint32_t i) {
  const uint32_t s = i / cap;
  return i - s * cap < seg[s].hwm;
}

// Pool entry i holds a live vertex (its segment closed).
__device__ inline bool vertex_live(const VolDev& v, uint32_t i) {
  return i < v.max_vertices && slot_in_use(v.vseg, v.vseg_cap, i) && v.vowner[i] != kNone;
}

// Position in metres of the vertex at parameter t on edge rem (axis * 512 +
// voxel) of the block with key bkey, in the frame of its volume (the slot's
// own frame in a batch): owner voxel g, plus t along the edge's axis.
// Returns the slot.
__device__ inline int edge_position(const VolDev& v, uint64_t bkey, uint32_t rem, float t,
                                    float p[3]) {
  const int axis = (int)(rem / kVox), local = (int)(rem % kVox);
  int bx, by, bz, slot;
  unpack_key(bkey, bx, by, bz);
  block_frame(v, bx, slot);
  const int g[3] = {8 * bx + (local & 7), 8 * by + ((local >> 3) & 7), 8 * bz + (local >> 6)};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float c = (float)g[a];
    if (a == axis) c = c + t;
    p[a] = c * v.s;
  }
  return slot;
}

// A download of large capacities counts first, so that each writer finds its
// place by itself (dl_counts says when; smaller ones leave it to the vertex
// writer, which saves a launch): the live vertices of each chunk of kDlSlots slots of a segment (one wave
// each; chunks past the segment's high-water mark hold none and are
// skipped), and, per chunk of kDlBlocks blocks (one workgroup each), every
// block's first triangle within the chunk and the chunk's total, from the
// counts classification keeps.  Reads 4 bytes per used slot and per block, so
// it ends within a few microseconds of its launch (counting the blocks' types
// here took 17 to 24 us for 30,000 to 44,000 blocks).
__global__ __launch_bounds__(1024) void k_dl_count(VolDev v, uint32_t tri_groups) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = __lane_id();
  if (blockIdx.x >= tri_groups) {
    const uint32_t cps = dl_chunks(v.vseg_cap), items = v.nseg * cps;
    const uint32_t step = (gridDim.x - tri_groups) * 16u;
    for (uint32_t it = (blockIdx.x - tri_groups) * 16u + (uint32_t)wave; it < items; it += step) {
      // segment by segment: the chunks in use are the first of each, and
      // consecutive workgroups, on other XCDs, then share them
      const uint32_t chunk = it / v.nseg, sg = it - chunk * v.nseg, lo = chunk * kDlSlots;
      const uint32_t hwm = closed_segment(v, sg).hwm;
      if (lo >= hwm) continue;
      const uint32_t* owner = v.vowner + (size_t)sg * v.vseg_cap + lo;
      uint32_t o[kDlSlots / 64], live = 0;
#pragma unroll
      for (int r = 0; r < kDlSlots / 64; ++r)
        o[r] = lo + 64u * r + q < hwm ? owner[64 * r + q] : kNone;
#pragma unroll
      for (int r = 0; r < kDlSlots / 64; ++r) live += (uint32_t)__popcll(__ballot(o[r] != kNone));
      if (q == 0) v.scan[sg * cps + chunk] = live;
    }
    return;
  }
  static_assert(kDlBlocks == 1024, "a lane per block");
  __shared__ uint32_t swave[16];
  const uint32_t n = min(v.cnt->n_blocks, v.max_blocks);
  for (uint32_t c = blockIdx.x; c * kDlBlocks < n; c += tri_groups) {
    const uint32_t b = c * kDlBlocks + threadIdx.x;
    uint32_t total;
    const uint32_t pre = wg_scan(b < n ? v.btri[b] : 0u, swave, &total);
    if (b < n) v.vcand[b] = pre;
    if (threadIdx.x == 0) v.vcand[v.max_blocks + c] = total;
  }
}

// Live vertices in pool order, one workgroup per chunk of kDlSlots slots:
// its place is the live vertices of the segments before (each segment's
// counters say how many it holds) and of the segment's chunks before (their
// counts, or counted here).  Each used slot's row (or -1) is recorded; slots up to the
// highest one that any download has given a row are visited, so that those
// above never keep one from before a reset.  The workgroups past `groups`
// see to the triangles' places: with counts one turns the chunks' totals into
// their first triangles, without them each takes a chunk of kDlBlocks blocks
// and sums the blocks before it (4 bytes each, from the caches).
__global__ __launch_bounds__(256) void k_dl_vertices(VolDev v, float* __restrict__ verts,
                                                     uint64_t* __restrict__ keys, uint32_t vcap,
                                                     uint32_t groups, int counted) {
  static_assert(kSegs == 256, "a lane per segment");
  __shared__ uint32_t sbase[kSegs], shwm[kSegs], stop[kSegs];
  __shared__ uint32_t swave[16];
  __shared__ uint32_t slive[4], sbefore[4];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = __lane_id();
  {
    uint32_t live = 0, hwm = 0, top = 0;
    if (threadIdx.x < v.nseg) {
      const Seg g = closed_segment(v, threadIdx.x);
      hwm = g.hwm;
      top = max(hwm, g.dl_top);
      live = hwm - min(hwm, g.count);
    }
    uint32_t total;
    if (blockIdx.x >= groups && !counted) {
      static_assert(kDlBlocks == 1024, "four blocks per lane");
      const uint32_t n = min(v.cnt->n_blocks, v.max_blocks);
      const uint32_t c = blockIdx.x - groups, b0 = c * kDlBlocks;
      if (b0 >= n) {
        if (n == 0 && c == 0 && threadIdx.x == 0) v.cnt->dl_nt = 0;
        return;
      }
      const uint4* tri = reinterpret_cast<const uint4*>(v.btri);
      uint32_t sum = 0;
#pragma unroll 8
      for (uint32_t k = threadIdx.x; k < b0 / 4; k += 256) {
        const uint4 x = tri[k];
        sum += x.x + x.y + x.z + x.w;
      }
      uint32_t base;
      wg_scan(sum, swave, &base);
      const uint32_t b = b0 + 4 * threadIdx.x;
      uint32_t x[4], own = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        x[k] = b + k < n ? v.btri[b + k] : 0u;
        own += x[k];
      }
      uint32_t at = base + wg_scan(own, swave, &total);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (b + k < n) v.vcand[b + k] = at;
        at += x[k];
      }
      if (b0 + kDlBlocks >= n && threadIdx.x == 0) v.cnt->dl_nt = base + total;
      return;
    }
    if (blockIdx.x >= groups) {
      const uint32_t n = (min(v.cnt->n_blocks, v.max_blocks) + kDlBlocks - 1) / kDlBlocks;
      uint32_t* chunk = v.vcand + v.max_blocks;
      uint32_t carry = 0;
      for (uint32_t c0 = 0; c0 < n; c0 += 256) {
        const uint32_t c = c0 + threadIdx.x;
        const uint32_t pre = wg_scan(c < n ? chunk[c] : 0u, swave, &total);
        if (c < n) chunk[c] = carry + pre;
        carry += total;
      }
      if (threadIdx.x == 0) v.cnt->dl_nt = carry;
      return;
    }
    sbase[threadIdx.x] = wg_scan(live, swave, &total);
    shwm[threadIdx.x] = hwm;
    stop[threadIdx.x] = top;
    if (blockIdx.x == 0 && threadIdx.x == 0) v.cnt->dl_nv = total;
    __syncthreads();
  }
  const uint32_t cps = dl_chunks(v.vseg_cap), items = v.nseg * cps;
  constexpr int kRows = kDlSlots / 256;
  for (uint32_t it = blockIdx.x; it < items; it += groups) {
    const uint32_t chunk = it / v.nseg, sg = it - chunk * v.nseg, lo = chunk * kDlSlots;
    const uint32_t hwm = shwm[sg], top = stop[sg];
    if (lo >= top) continue;
    const uint32_t gbase = sg * v.vseg_cap, l0 = lo + (uint32_t)wave * (64 * kRows) + q;
    uint32_t own[kRows], wlive = 0, before = 0;
    uint64_t m[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
      own[r] = l0 + 64u * r < hwm ? v.vowner[gbase + l0 + 64u * r] : kNone;
    if (lo < hwm && counted) {
      for (uint32_t k = threadIdx.x; k < chunk; k += 256) before += v.scan[sg * cps + k];
    } else if (lo < hwm) {
#pragma unroll 8
      for (uint32_t k = threadIdx.x; k < lo; k += 256) before += v.vowner[gbase + k] != kNone;
    }
    before = wave_sum(before);
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      m[r] = __ballot(own[r] != kNone);
      wlive += (uint32_t)__popcll(m[r]);
    }
    if (q == 0) slive[wave] = wlive, sbefore[wave] = before;
    __syncthreads();
    uint32_t j = sbase[sg];
    for (int w = 0; w < 4; ++w) j += sbefore[w] + (w < wave ? slive[w] : 0u);
    __syncthreads();
    // the rows' owners: block keys and edge parameters, requested together
    uint64_t bkey[kRows];
    float t[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const bool on = own[r] != kNone;
      bkey[r] = on ? v.block_key[own[r] / (3 * kVox)] : 0ull;
      t[r] = on ? v.et[own[r]] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const uint32_t slot = l0 + 64u * r, row = j + mask_rank(m[r]);
      const bool on = own[r] != kNone;
      if (slot < top) v.vdl[gbase + slot] = on ? (int32_t)row : -1;
      if (on && row < vcap) {
        float p[3];
        edge_position(v, bkey[r], own[r] % (3 * kVox), t[r], p);
#pragma unroll
        for (int a = 0; a < 3; ++a) verts[3 * (size_t)row + a] = p[a];
        if (keys)
          keys[row] = edge_key(bkey[r], (int)(own[r] % kVox), (int)(own[r] % (3 * kVox) / kVox));
      }
      j += (uint32_t)__popcll(m[r]);
    }
  }
}

// Every vertex pool entry's position (0 and slot -1 for entries without a
// live vertex): no compaction, so no host round trip.
__global__ __launch_bounds__(256) void k_positions(VolDev v, float* __restrict__ pos,
                                                   int32_t* __restrict__ slot_of) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < v.max_vertices;
       i += gridDim.x * blockDim.x) {
    float p[3] = {0.f, 0.f, 0.f};
    int slot = -1;
    if (vertex_live(v, i)) {
      const uint32_t owner = v.vowner[i];
      slot = edge_position(v, v.block_key[owner / (3 * kVox)], owner % (3 * kVox), v.et[owner], p);
    }
    pos[3 * (size_t)i] = p[0];
    pos[3 * (size_t)i + 1] = p[1];
    pos[3 * (size_t)i + 2] = p[2];
    if (slot_of) slot_of[i] = slot;
  }
}

// Triangles of every cube, in pool order: the cube's type lists its
// triangles as cube edges, each edge is resolved to the vertex its owner
// voxel holds (the owner block through the cube's neighbour table), and the
// vertex to its row in this download.  One wave per block: lane q puts each
// of its row's cubes into LDS at its first triangle's place, then a lane
// takes a triangle, whose cube is the last one placed at or before it,
// resolves its three corners together and stores its 12 bytes next to its
// neighbours'.  Bound by the chain block, list, edge, vertex, so each
// wave requests its next block's record while it works on one and resolves up
// to 128 triangles, two per lane, at once; tables in LDS give a triangle's
// three owner offsets in one word, and the owner's place follows from
// byte-wise sums.
// 3.48 million triangles of an 8 mm room take 43 us; a lane per corner over
// a list of triangles built cube by cube took 89 us.
// The last workgroup closes the segments, the first one tells the host.
constexpr int kTriList = 512;  // triangles listed at once per wave
__global__ __launch_bounds__(256) void k_dl_triangles(VolDev v, int32_t* __restrict__ tris,
                                                      uint32_t tcap, int counted,
                                                      Report* __restrict__ out) {
  __shared__ uint16_t stri[256 * 5];           // per type and triangle: its three edges, 4 bits each
  __shared__ uint8_t sntri[256];
  __shared__ uint32_t sowner[12];              // per edge: owner offset x, y, z and axis, in bytes
  // at its first listed triangle: cube | type << 9 | triangle << 17 | 1 << 31
  __shared__ uint32_t slist_all[4][kTriList];
  __shared__ int32_t snb_all[4][8];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  {
    // a type's 16 bytes in one load (a load per edge, triangle by triangle,
    // kept every workgroup waiting up to five times before its first block)
    const uint4 row = reinterpret_cast<const uint4*>(v.tri_table)[threadIdx.x];
    const uint32_t tab[4] = {row.x, row.y, row.z, row.w};
    auto at = [&](int i) -> uint32_t { return (tab[i >> 2] >> (8 * (i & 3))) & 255u; };
    sntri[threadIdx.x] = (uint8_t)at(0);
#pragma unroll
    for (int t = 0; t < 5; ++t)
      stri[threadIdx.x * 5 + t] =
          (uint16_t)(at(1 + 3 * t) | at(2 + 3 * t) << 4 | at(3 + 3 * t) << 8);
    if (threadIdx.x < 12) {
      int ox, oy, oz, axis;
      edge_owner((int)threadIdx.x, ox, oy, oz, axis);
      sowner[threadIdx.x] = (uint32_t)(ox | oy << 8 | oz << 16 | axis << 24);
    }
  }
  if (blockIdx.x == gridDim.x - 1 && wave == 0) {
    close_segments(v);
    for (uint32_t s = __lane_id(); s < v.nseg; s += 64) v.vseg[s].dl_top = v.vseg[s].hwm;
  }
  uint32_t* slist = slist_all[wave];
  int32_t* snb = snb_all[wave];
  const uint32_t n = min(v.cnt->n_blocks, v.max_blocks);
  const uint32_t* chunk = v.vcand + v.max_blocks;
  if (blockIdx.x == 0 && threadIdx.x == 0 && out) {
    out->dl_nv = v.cnt->dl_nv, out->dl_nt = v.cnt->dl_nt;
    out->error = v.cnt->error;
  }
  __syncthreads();  // the tables are ready
  const uint32_t step = gridDim.x * 4u;
  const int q = __lane_id();
  // a block's triangles, its first one's place, its types and its neighbours
  uint32_t all1 = 0, first1 = 0;
  uint2 tt1 = make_uint2(0u, 0u);
  int32_t nb1 = -1;
  auto request = [&](uint32_t idx) {
    if (idx >= n) return;
    all1 = v.btri[idx];
    first1 = v.vcand[idx] + (counted ? chunk[idx / kDlBlocks] : 0u);
    tt1 = reinterpret_cast<const uint2*>(v.tcur)[(size_t)idx * 64 + q];
    nb1 = q < 8 ? v.nbr[(size_t)idx * 27 + nbr_dir(q & 1, (q >> 1) & 1, q >> 2)] : -1;
  };
  uint32_t idx = blockIdx.x * 4u + (uint32_t)wave;
  request(idx);
  for (; idx < n; idx += step) {
    const uint32_t all = uniform(all1), first = uniform(first1);
    uint2 tt = tt1;
    const int32_t nb = nb1;
    request(idx + step);
    if (all == 0) continue;
    {
      transpose8(tt.x, tt.y);
      uint32_t nt[8], cnt = 0, sum;
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        nt[x] = sntri[((x < 4 ? tt.x : tt.y) >> (8 * (x & 3))) & 255u];
        cnt += nt[x];
      }
      const uint32_t before = wave_prefix_bits<6>(cnt, &sum);
      if (q < 8) snb[q] = nb;
      for (uint32_t c0 = 0; c0 < all; c0 += kTriList) {
        const uint32_t count = min(all - c0, (uint32_t)kTriList);
        wave_sync();
        for (uint32_t i = (uint32_t)q; i < count; i += 64) slist[i] = 0u;
        wave_sync();
        // a cube listed before c0 with triangles from c0 on stands at c0
        int32_t p = (int32_t)(before - c0);
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const uint32_t type = ((x < 4 ? tt.x : tt.y) >> (8 * (x & 3))) & 255u;
          const int32_t at = max(p, 0), end = p + (int32_t)nt[x];
          if (at < min(end, (int32_t)kTriList))
            slist[at] = 0x80000000u | (8u * (uint32_t)q + x) | type << 9 | (uint32_t)(at - p) << 17;
          p = end;
        }
        wave_sync();
        // the cube the last window ended in, and its place
        uint32_t last_e = 0, last_at = 0;
        for (uint32_t i0 = 0; i0 < count; i0 += 128) {
          int32_t s[6], row[6];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t w0 = i0 + 64u * h, i = w0 + (uint32_t)q;
            uint32_t e = i < count ? slist[i] : 0u;
            const uint64_t starts = __ballot(e != 0u);
            const uint64_t upto = starts & (~0ull >> (63 - q));
            const int src = upto ? 63 - __builtin_clzll(upto) : 0;
            const uint32_t es = __shfl(e, src);
            if (starts) {
              const int l = 63 - __builtin_clzll(starts);
              const uint32_t el = (uint32_t)__builtin_amdgcn_readlane((int)e, l);
              e = upto ? es : last_e;
              const uint32_t at = upto ? w0 + (uint32_t)src : last_at;
              e += (i - at) << 17;
              last_e = el, last_at = w0 + (uint32_t)l;
            } else {
              e = last_e + ((i - last_at) << 17);
            }
            const uint32_t l = e & 511u;
            const uint32_t edges = i < count ? stri[((e >> 9) & 255u) * 5u + ((e >> 17) & 7u)] : 0u;
            const uint32_t cube = (l & 7u) | (l & 0x38u) << 5 | (l & 0x1C0u) << 10;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const uint32_t o = sowner[(edges >> (4 * k)) & 15u];
              // the owner voxel, byte by byte; a carry to 8 is the neighbour's 0
              const uint32_t w = cube + (o & 0x010101u), c = w & 0x080808u;
              const int32_t ob = snb[(c >> 3 | c >> 10 | c >> 17) & 7u];
              const uint32_t ol = (w & 7u) | ((w >> 5) & 0x38u) | ((w >> 10) & 0x1C0u);
              s[3 * h + k] = -1;
              if (i < count && ob >= 0) s[3 * h + k] = v.evtx[((size_t)ob * 3 + (o >> 24)) * kVox + ol];
            }
          }
#pragma unroll
          for (int k = 0; k < 6; ++k) row[k] = s[k] >= 0 ? v.vdl[s[k]] : -1;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t i = i0 + 64u * h + (uint32_t)q;
            if (i < count && first + c0 + i < tcap) {
              int32_t* o = tris + 3 * (size_t)(first + c0 + i);
#pragma unroll
              for (int k = 0; k < 3; ++k) o[k] = row[3 * h + k];
            }
          }
        }
      }
      wave_sync();
    }
  }
}

// The live vertices that the last download gave a row, for the kernels that
// follow its rows: one workgroup per 256 slots of a segment, chunks past the
// segment's high-water mark skipped.  f(pool entry, row).
template <typename F>
__device__ inline void for_downloaded(const VolDev& v, F f) {
  const uint32_t nv = v.cnt->dl_nv;
  const uint32_t cps = (v.vseg_cap + 255u) / 256u;
  for (uint32_t it = blockIdx.x; it < v.nseg * cps; it += gridDim.x) {
    const uint32_t chunk = it / v.nseg, sg = it - chunk * v.nseg, lo = chunk * 256u;
    const uint32_t hwm = v.vseg[sg].hwm;
    if (lo >= hwm) continue;
    const uint32_t s = sg * v.vseg_cap + lo + threadIdx.x;
    if (lo + threadIdx.x >= hwm || v.vowner[s] == kNone) continue;
    const int32_t row = v.vdl[s];
    if (row >= 0 && (uint32_t)row < nv) f(s, (uint32_t)row);
  }
}

// Unit normals of the vertices of the last download, in its row order (the
// paper keeps a normal in every vertex, Sec. IV): the TSDF gradient at the
// edge's two end points, interpolated at t and normalised, (0, 0, 0) when it
// vanishes; it points to increasing TSDF.  The gradient at a voxel is, per
// axis, the central difference over its two neighbours, one-sided when only
// one is observed, 0 when neither is.  One lane per pool slot.
// Bound by gathers: an edge's two ends need twelve voxels between them, whose
// blocks (the own one but for neighbours across a face), TSDF values and
// observed bits are each requested together.  Fetching every voxel's block,
// TSDF and weight gradient by gradient, 42 gathers a vertex in chains, over
// the pool's whole capacity, took 113 us for 1.74 million vertices; this takes
// 53.
__global__ __launch_bounds__(256) void k_dl_normals(VolDev v, float* __restrict__ normals) {
  const uint8_t* wmask = reinterpret_cast<const uint8_t*>(v.wmask);
  for_downloaded(v, [&](uint32_t s, uint32_t row) {
    const uint32_t eo = v.vowner[s];
    const float t = v.et[eo];
    const uint32_t idx = eo / (3 * kVox), a = (eo / kVox) % 3, l = eo % kVox;
    const int x = (int)(l & 7u), y = (int)((l >> 3) & 7u), z = (int)(l >> 6);
    // voxels along the edge (one before it, its ends, one after it), then per
    // other axis one step back and forth from each end
    constexpr int kN = 12;
    int32_t blk[kN];
    uint32_t vox[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      // offset along the edge's axis and along axis a + 1 or a + 2
      const int along = k < 4 ? k - 1 : ((k - 4) >> 1) & 1;
      const int side = k < 4 ? 0 : (k & 1 ? 1 : -1);
      const uint32_t b = k < 8 ? (a == 2 ? 0u : a + 1u) : (a == 0 ? 2u : a - 1u);
      const int px = x + (a == 0 ? along : 0) + (b == 0 ? side : 0);
      const int py = y + (a == 1 ? along : 0) + (b == 1 ? side : 0);
      const int pz = z + (a == 2 ? along : 0) + (b == 2 ? side : 0);
      const int dir = (px >> 3) + 3 * (py >> 3) + 9 * (pz >> 3);
      blk[k] = dir == 0 ? (int32_t)idx : v.nbr[(size_t)idx * 27 + kSelf + dir];
      vox[k] = (uint32_t)((px & 7) | (py & 7) << 3 | (pz & 7) << 6);
    }
    float d[kN];
    uint32_t w[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      d[k] = blk[k] >= 0 ? v.d[(size_t)blk[k] * kVox + vox[k]] : 0.f;
      w[k] = blk[k] >= 0 ? (uint32_t)wmask[(size_t)blk[k] * 64 + (vox[k] >> 3)] : 0u;
    }
    // one axis' difference from the voxels back and forth of centre c
    auto diff = [&](int c, int back, int forth) -> float {
      const bool hp = (w[forth] >> (vox[forth] & 7u)) & 1u, hm = (w[back] >> (vox[back] & 7u)) & 1u;
      return hp && hm ? (d[forth] - d[back]) * 0.5f
                      : (hp ? d[forth] - d[c] : (hm ? d[c] - d[back] : 0.f));
    };
    const float ga = (1.f - t) * diff(1, 0, 2) + t * diff(2, 1, 3);
    const float gb = (1.f - t) * diff(1, 4, 5) + t * diff(2, 6, 7);
    const float gc = (1.f - t) * diff(1, 8, 9) + t * diff(2, 10, 11);
    float n[3];
    n[0] = a == 0 ? ga : (a == 2 ? gb : gc);
    n[1] = a == 1 ? ga : (a == 0 ? gb : gc);
    n[2] = a == 2 ? ga : (a == 1 ? gb : gc);
    const float len = sqrtf(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
#pragma unroll
    for (int j = 0; j < 3; ++j) normals[3 * (size_t)row + j] = len > 0.f ? n[j] / len : 0.f;
  });
}

// Birth frames of the vertices of the last download, in its row order: the
// frame (integration or import count) of the pass in which the vertex's
// count last became positive.
__global__ __launch_bounds__(256) void k_dl_births(VolDev v, uint32_t* __restrict__ births) {
  for_downloaded(v, [&](uint32_t s, uint32_t row) { births[row] = v.vbirth[s]; });
}

// ============================================================================
// backward passes
// ============================================================================

// dL/d(TSDF) of every voxel of the listed blocks, one wave per block, lane q
// the row of eight voxels at y = q & 7, z = q >> 3.  A voxel's gradient sums,
// in a fixed order, the contributions of the at most six edges incident to
// it: per axis its own edge (the voxel is the first end point), then the edge
// owned by the voxel one step back (the voxel is the second); each
// contribution is the vertex gradient along the axis times s times dt/dd.
// Only edges that carry a vertex contribute, about one in a hundred: the
// block's edge masks (one word per lane) and the three back faces' words say
// which, those edges are listed row by row, and each one's slot, end point
// TSDF values and upstream gradient are fetched once, for both its ends.  A
// voxel then finds its edges' places in the list from the same masks.  A
// block with more edges than the list holds (dense sign fields) is worked
// through layer by layer; one layer always fits.
constexpr int kGradCap = 320;  // listed edges at once; one layer has at most 272

template <int W>
__global__ __launch_bounds__(64 * W) void k_bwd_tsdf(VolDev v, const float* __restrict__ dL_dv,
                                                     int by_slot, const int32_t* __restrict__ rows,
                                                     uint32_t n_rows, float* __restrict__ out) {
  // edge a * 512 + l | 2048 when voxel l is the edge's second end point
  __shared__ uint16_t slist_all[W][kGradCap];
  // contributions to the owner voxel and to the second end point; then the
  // block's sums on their way out
  __shared__ __align__(16) float sc_all[W][2 * kGradCap];
  __shared__ int32_t snb_all[W][27];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint16_t* slist = slist_all[wave];
  float* sown = sc_all[wave];
  float* sfar = sc_all[wave] + kGradCap;
  static_assert(2 * kGradCap >= kVox, "a block's sums fit");
  int32_t* snb = snb_all[wave];
  const uint32_t nb_all = min(v.cnt->n_blocks, v.max_blocks);
  const uint32_t n = rows ? n_rows : nb_all;
  const uint32_t nv = v.cnt->dl_nv;
  // the caller's array may be aligned to its floats alone
  const bool wide = ((uintptr_t)out & 15u) == 0u;
  for (ItemLoop it = item_loop(v, n, W, wave); it.i < it.end; it.i += it.step) {
    const int q = fresh_lane(), y = q & 7, z = q >> 3;
    const int32_t idx = rows ? (int32_t)uniform((uint32_t)rows[it.i]) : (int32_t)it.i;
    float* o = out + (size_t)it.i * kVox;
    // a block without a gradient: zeros, whole lines per store
    auto store_zero = [&]() {
      if (wide) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
          reinterpret_cast<float4*>(o)[q + 64 * k] = make_float4(0.f, 0.f, 0.f, 0.f);
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) o[q + 64 * k] = 0.f;
      }
    };
    if (idx < 0 || (uint32_t)idx >= nb_all) {
      store_zero();
      continue;
    }
    // the block's edge masks and its neighbours'; an edge ending at a voxel
    // from behind is owned by the voxel one step back: bit x - 1, the lane at
    // y - 1 or z - 1 or, on the block's back faces, the -x neighbour's bit 7,
    // the -y neighbour's row y = 7, the -z neighbour's row z = 7
    const int32_t mynb = q < 27 ? v.nbr[(size_t)idx * 27 + q] : -1;
    const uint32_t hm = v.emask[(size_t)idx * 64 + q];
    if (q < 27) snb[q] = mynb;
    const int32_t bnx = __builtin_amdgcn_readlane(mynb, nbr_dir(-1, 0, 0)),
                  bny = __builtin_amdgcn_readlane(mynb, nbr_dir(0, -1, 0)),
                  bnz = __builtin_amdgcn_readlane(mynb, nbr_dir(0, 0, -1));
    const uint32_t fx = bnx >= 0 ? v.emask[(size_t)bnx * 64 + q] : 0u;
    const uint32_t fy = bny >= 0 ? v.emask[(size_t)bny * 64 + (q | 7)] : 0u;
    const uint32_t fz = bnz >= 0 ? v.emask[(size_t)bnz * 64 + (q | 56)] : 0u;
    // edges ending at the row's voxels that no row of this block owns
    const uint32_t back_xy = ((fx >> 7) & 1u) | (y == 0 ? fy & 0xFF00u : 0u);
    const uint32_t back_z = fz & 0xFF0000u;
    uint32_t all;
    (void)wave_prefix_bits<6>((uint32_t)(__popc(hm) + __popc(back_xy | (z == 0 ? back_z : 0u))),
                              &all);
    if (all == 0) {
      store_zero();
      continue;
    }
    const uint32_t hup = __shfl(hm, (q - 8) & 63);
    const int dz = all <= (uint32_t)kGradCap ? 8 : 1;
    for (int z0 = 0; z0 < 8; z0 += dz) {
      // the edges of the rows of layers [z0, z0 + dz): their own, then those
      // ending there from rows outside
      const bool in = z >= z0 && z < z0 + dz;
      const uint32_t own = in ? hm : 0u;
      const uint32_t back =
          in ? back_xy | (z == z0 ? (z0 == 0 ? back_z : hup & 0xFF0000u) : 0u) : 0u;
      uint32_t cnt;
      const uint32_t pre = wave_prefix_bits<6>((uint32_t)(__popc(own) + __popc(back)), &cnt);
      const uint32_t pre2 = pre + (uint32_t)__popc(own);
      wave_sync();
      {
        uint32_t p = pre;
        for (uint32_t m = own; m; m &= m - 1u) {
          const uint32_t k = (uint32_t)__builtin_ctz(m);
          slist[p++] = (uint16_t)((k & 0x18u) << 6 | (uint32_t)q << 3 | (k & 7u));
        }
        for (uint32_t m = back; m; m &= m - 1u) {
          const uint32_t k = (uint32_t)__builtin_ctz(m);
          slist[p++] = (uint16_t)(2048u | (k & 0x18u) << 6 | (uint32_t)q << 3 | (k & 7u));
        }
      }
      wave_sync();
      for (uint32_t i = (uint32_t)q; i < cnt; i += 64) {
        const uint32_t e = slist[i], l = e & 511u, a = (e >> 9) & 3u;
        const uint32_t c = a == 0 ? (l & 7u) : (a == 1 ? ((l >> 3) & 7u) : (l >> 6));
        const uint32_t stp = a == 0 ? 1u : (a == 1 ? 8u : 64u);
        const int dir = a == 0 ? 1 : (a == 1 ? 3 : 9);
        // owner voxel (block ob, local ol) and far end point (fb, fl)
        int32_t ob = idx, fb = idx;
        uint32_t ol = l, fl = l;
        if (e < 2048u) {
          if (c < 7u) fl = l + stp;
          else fb = snb[kSelf + dir], fl = l - 7u * stp;
        } else {
          if (c > 0u) ol = l - stp;
          else ob = snb[kSelf - dir], ol = l + 7u * stp;
        }
        float cown = 0.f, cfar = 0.f;
        if (ob >= 0 && fb >= 0) {
          const int32_t s = v.evtx[((size_t)ob * 3 + a) * kVox + ol];
          const float da = v.d[(size_t)ob * kVox + ol], db = v.d[(size_t)fb * kVox + fl];
          int32_t r = -1;
          if (s >= 0) {
            if (by_slot) {
              r = s;
            } else {
              r = v.vdl[s];
              if (!(r >= 0 && (uint32_t)r < nv)) r = -1;
            }
          }
          if (r >= 0 && da != db) {
            const float g = dL_dv[3 * (size_t)r + a] * v.s;
            const float den = (da - db) * (da - db);
            cown = g * (-db / den);
            cfar = g * (da / den);
          }
        }
        sown[i] = cown;
        sfar[i] = cfar;
      }
      wave_sync();
      const uint32_t oy = __shfl(own, (q - 1) & 63), py = __shfl(pre, (q - 1) & 63);
      const uint32_t oz = __shfl(own, (q - 8) & 63), pz = __shfl(pre, (q - 8) & 63);
      const uint32_t my = y > 0 ? oy : back, ay = y > 0 ? py : pre2;
      const uint32_t mz = z > z0 ? oz : back, az = z > z0 ? pz : pre2;
      float sum[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        float acc = 0.f;
        // bit k of m: the edge at its rank among m's bits from `at` on (an
        // edge that does not contribute is listed with 0)
        auto add = [&](const float* c, uint32_t m, uint32_t at, int k) {
          if ((m >> k) & 1u) acc = acc + c[at + (uint32_t)__popc(m & ((1u << k) - 1u))];
        };
        add(sown, own, pre, x);
        if (x > 0) add(sfar, own, pre, x - 1);
        else add(sfar, back, pre2, 0);
        add(sown, own, pre, 8 + x);
        add(sfar, my, ay, 8 + x);
        add(sown, own, pre, 16 + x);
        add(sfar, mz, az, 16 + x);
        sum[x] = acc;
      }
      // rows to whole lines through LDS (a row per lane would leave every
      // store half a line apart from its neighbour's)
      wave_sync();
      float4* so = reinterpret_cast<float4*>(sc_all[wave]);
      so[2 * q] = make_float4(sum[0], sum[1], sum[2], sum[3]);
      so[2 * q + 1] = make_float4(sum[4], sum[5], sum[6], sum[7]);
      wave_sync();
      // layer z is the 64 floats from 64 z on
      if (wide) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int e = q + 64 * k;
          if ((e >> 4) >= z0 && (e >> 4) < z0 + dz) reinterpret_cast<float4*>(o)[e] = so[e];
        }
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (k >= z0 && k < z0 + dz) o[q + 64 * k] = sc_all[wave][q + 64 * k];
      }
    }
    wave_sync();
  }
}

// Gradient of the squared distance of every vertex pool entry to its slot's
// target sphere (the batched workload's loss): 2 (|p - c| - r) (p - c) / |p - c|,
// |p - c| as two hypot calls and at least 1e-30.  rows spheres; entry i has
// sphere slot[i] modulo rows, so -1 (no vertex) takes the last one.  One pass
// over the entries, 28 bytes each: 4.9 million take 29 us where the same
// operations as eleven elementwise launches took 156 us.
__global__ __launch_bounds__(256) void k_sphere_loss(const float* pos, const int32_t* slot,
                                                     const float* __restrict__ centers,
                                                     const float* __restrict__ radii, int32_t rows,
                                                     uint64_t n, float* out) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    int32_t k = slot[i] % rows;
    if (k < 0) k += rows;
    float d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) d[a] = pos[3 * i + a] - centers[3 * (size_t)k + a];
    float dist = hypotf(hypotf(d[0], d[1]), d[2]);
    dist = dist < 1e-30f ? 1e-30f : dist;
    const float scale = (dist - radii[k]) / dist * 2.f;
#pragma unroll
    for (int a = 0; a < 3; ++a) out[3 * i + a] = d[a] * scale;
  }
}

// Backward of the last fusion (Eq. 2) with its branches fixed.
__global__ __launch_bounds__(512) void k_bwd_fusion(VolDev v, FrameParams fp,
                                                    const float* __restrict__ depth,
                                                    const float* __restrict__ g1,
                                                    float* __restrict__ g0,
                                                    float* __restrict__ gD) {
  const uint32_t n = min(v.cnt->n_blocks, v.max_blocks);
  const int l = threadIdx.x, lx = l & 7, ly = (l >> 3) & 7, lz = l >> 6;
  for (ItemLoop it = item_loop(v, n, 1, 0); it.i < it.end; it.i += it.step) {
    const uint32_t idx = it.i;
    const size_t o = (size_t)idx * kVox + l;
    const float g = g1[o];
    float out = g;
    if (v.st_frame[idx] == fp.frame) {
      int bx, by, bz;
      unpack_key(v.block_key[idx], bx, by, bz);
      const FuseSample fs = fuse_sample(v, fp, depth, 8 * bx + lx, 8 * by + ly, 8 * bz + lz);
      if (fs.upd) {
        const float W1 = v.w[o];
        const float W0 = W1 - 1.0f;
        out = g * (W0 / W1);
        if (!fs.clamped && g != 0.f) unsafeAtomicAdd(&gD[fs.pixel], g * (v.inv_s / W1));
      }
    }
    g0[o] = out;
  }
}

__global__ void k_zero_f32(float* p, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = 0.f;
}

// ============================================================================
// inspection
// ============================================================================
// Reference count of edge (axis a, voxel l) of block blk, formed from the
// applied types of the four cubes around it (in this block or its -x/-y/-z
// neighbours; a missing block's cubes have no type).
__device__ inline int32_t edge_count(const VolDev& v, uint32_t blk, int a, int l) {
  // per axis, the four cubes as offsets from the voxel and the cube edge
  // that is this edge in each: x (0,0,0) e0, (0,-1,0) e2, (0,0,-1) e4,
  // (0,-1,-1) e6; y (0,0,0) e3, (-1,0,0) e1, (0,0,-1) e7, (-1,0,-1) e5;
  // z (0,0,0) e8, (-1,0,0) e9, (-1,-1,0) e10, (0,-1,0) e11
  const int8_t off[3][4][4] = {{{0, 0, 0, 0}, {0, -1, 0, 2}, {0, 0, -1, 4}, {0, -1, -1, 6}},
                               {{0, 0, 0, 3}, {-1, 0, 0, 1}, {0, 0, -1, 7}, {-1, 0, -1, 5}},
                               {{0, 0, 0, 8}, {-1, 0, 0, 9}, {-1, -1, 0, 10}, {0, -1, 0, 11}}};
  const int x = l & 7, y = (l >> 3) & 7, z = l >> 6;
  int32_t c = 0;
  for (int j = 0; j < 4; ++j) {
    const int cx = x + off[a][j][0], cy = y + off[a][j][1], cz = z + off[a][j][2];
    const int32_t b = v.nbr[(size_t)blk * 27 + nbr_dir(cx < 0 ? -1 : 0, cy < 0 ? -1 : 0, cz < 0 ? -1 : 0)];
    if (b < 0) continue;
    const uint32_t t = cube_type(v.tcur, (size_t)b, (cx & 7) + 8 * (cy & 7) + 64 * (cz & 7));
    c += v.edge_uses[t * 12 + off[a][j][3]];
  }
  return c;
}

// Cube types one byte each, as the caller takes them; blank (or null): the
// flags of blocks whose types are all 0 and not written.
__global__ void k_export_types(const uint64_t* __restrict__ types,
                               const uint32_t* __restrict__ blank, uint8_t* __restrict__ out,
                               uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    out[i] = blank && blank[i / kVox] ? 0 : (uint8_t)planes_type(types[i >> 3], (int)(i & 7));
}

__global__ void k_export_vertices(VolDev v, uint64_t* keys, float* t, int32_t* ref, uint32_t n) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t owner = slot_in_use(v.vseg, v.vseg_cap, i) ? v.vowner[i] : kNone;
    uint64_t k = ~0ull;
    int32_t r = -1;
    if (owner != kNone) {
      const uint32_t blk = owner / (3 * kVox), rem = owner % (3 * kVox);
      k = edge_key(v.block_key[blk], (int)(rem % kVox), (int)(rem / kVox));
      r = edge_count(v, blk, (int)(rem / kVox), (int)(rem % kVox));
    }
    keys[i] = k;
    ref[i] = r;
    t[i] = owner != kNone ? v.et[owner] : 0.f;
  }
}

__global__ void k_lookup(VolDev v, const int32_t* __restrict__ coords, int32_t* __restrict__ idx,
                         uint32_t n) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int x = coords[3 * i], y = coords[3 * i + 1], z = coords[3 * i + 2];
    idx[i] = key_in_range(x, y, z) ? hash_find(v, pack_key(x, y, z)) : -1;
  }
}

#define VM_CLASSIFY_MODES(W)                                      \
  template __global__ void k_classify<W, kExtract>(VolDev, uint32_t); \
  template __global__ void k_classify<W, kRefine>(VolDev, uint32_t);  \
  template __global__ void k_classify<W, kExtractRefined>(VolDev, uint32_t);
VM_CLASSIFY_MODES(2)
VM_CLASSIFY_MODES(4)
VM_CLASSIFY_MODES(8)
template __global__ void k_collect<1>(VolDev, FrameParams, const float*, uint32_t);
template __global__ void k_collect<2>(VolDev, FrameParams, const float*, uint32_t);
template __global__ void k_vertices<2>(VolDev, uint32_t, int);
template __global__ void k_vertices<4>(VolDev, uint32_t, int);
template __global__ void k_vertices<8>(VolDev, uint32_t, int);
template __global__ void k_fuse<2>(VolDev, FrameParams, const float*, uint32_t);
template __global__ void k_fuse<4>(VolDev, FrameParams, const float*, uint32_t);
template __global__ void k_fuse<8>(VolDev, FrameParams, const float*, uint32_t);
template __global__ void k_import_copy<2>(VolDev, const float*, const float*, uint32_t, int32_t*);
template __global__ void k_import_copy<4>(VolDev, const float*, const float*, uint32_t, int32_t*);
template __global__ void k_import_copy<8>(VolDev, const float*, const float*, uint32_t, int32_t*);
template __global__ void k_bwd_tsdf<2>(VolDev, const float*, int, const int32_t*, uint32_t, float*);
template __global__ void k_bwd_tsdf<4>(VolDev, const float*, int, const int32_t*, uint32_t, float*);
template __global__ void k_bwd_tsdf<8>(VolDev, const float*, int, const int32_t*, uint32_t, float*);

}  // namespace vm
