// kb_api.hip -- host side of the C ABI declared in include/kbuild.h.
//
// Validates arguments, carves the caller's workspace and enqueues the kernel
// sequence on the caller's stream.  Allocates nothing and keeps no state.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <cmath>

#include "kb_adjoint.hpp"
#include "kb_batch.hpp"
#include "kb_launch.hpp"
#include "kbuild.h"

namespace kb {
KB_INSTANCES(extern, Prec::F64)
KB_INSTANCES(extern, Prec::F32)
KB_INSTANCES(extern, Prec::F32FB)
}  // namespace kb

namespace {

using namespace kb;

// compute units of the current device, cached per device ordinal
int device_cus(int* out) {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return KB_EHIP;
  if (dev >= 0 && dev < 64) {
    const int c = cache[dev].load(std::memory_order_relaxed);
    if (c > 0) {
      *out = c;
      return KB_OK;
    }
  }
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return KB_EHIP;
  if (dev >= 0 && dev < 64) cache[dev].store(n, std::memory_order_relaxed);
  *out = n;
  return KB_OK;
}

int ilog2_ceil(int64_t x) {
  int k = 0;
  while (((int64_t)1 << k) < x) ++k;
  return k;
}

// dof > 1: element matrices with dof components per node are assembled as elements of
// nen * dof "nodes" (global DOF dof * E_a + i); nen and nn below are those of that view
// csr_cap > 0: each pass also reads back up to csr_cap entries of running sums as two
// pairs each (value and residual), and writes residuals (grouped builds)
int make_plan(const kb_mesh* m, int prec, const kb_tuning* tu, Plan* p, int dof = 1, int64_t csr_cap = 0) {
  if (!m) return KB_EINVAL;
  if (m->elem != KB_HEX8 && m->elem != KB_TET4) return KB_EINVAL;
  if (prec != KB_FP64 && prec != KB_FP32 && prec != KB_FP32_FB64) return KB_EINVAL;
  if (m->n_elem < 0 || m->n_node < 0 || (m->op != KB_OP_STIFFNESS && m->op != KB_OP_MASS)) return KB_EINVAL;
  if (dof < 1 || dof > 3) return KB_EINVAL;
  p->op = m->op;
  p->dof = dof;
  p->nen = m->elem * dof;
  p->te = p->nen * (p->nen + 1) / 2;
  p->prec = prec;
  p->nel = m->n_elem;
  if (m->n_node >= (int64_t)INT32_MAX / dof) return KB_ERANGE;
  p->nn = m->n_node * dof;
  if (p->nn >= (int64_t)INT32_MAX) return KB_ERANGE;
  if (csr_cap < 0) return KB_EINVAL;
  if (p->nel > (int64_t)INT32_MAX / p->te || csr_cap > ((int64_t)INT32_MAX - p->nel * p->te) / 2) return KB_ERANGE;
  p->csr_cap = csr_cap;
  p->T = p->nel * p->te + 2 * csr_cap;  // pairs of one pass
  p->vbytes = prec == KB_FP64 ? 8 : 4;
  int bucket_bits = 0, sub_bits = 0;
  if (tu) {
    if (tu->block) {
      if (tu->block < 64 || tu->block > 1024 || (tu->block & 63)) return KB_EINVAL;
      p->block = tu->block;
    }
    if (tu->fb_tau != 0.0f) {
      if (!(tu->fb_tau > 1.0f)) return KB_EINVAL;
      p->tau = tu->fb_tau;
    }
    if (tu->sub_bits < 0 || tu->sub_bits > 8 || tu->bucket_bits < 0 || tu->bucket_bits > 16) return KB_EINVAL;
    if (tu->bucket_bits && tu->sub_bits && tu->sub_bits > tu->bucket_bits) return KB_EINVAL;
    bucket_bits = tu->bucket_bits;
    sub_bits = tu->sub_bits;
    if (tu->seg_pairs != 0 && tu->seg_pairs != kSeg && tu->seg_pairs != kSegLong) return KB_EINVAL;
    if (tu->table_slots != 0 && (tu->table_slots < kHTMin || tu->table_slots > kHTMax ||
                                 (tu->table_slots & (tu->table_slots - 1))))
      return KB_EINVAL;
  }
  // sub-buckets: about a third of the pass-3 hash table of distinct entries on average;
  // distinct entries per row estimated from the pairs per row and the typical number
  // of elements sharing an entry (about 7 for tetrahedra, 2.5 for bricks)
  p->colbits = 1;
  while (((int64_t)1 << p->colbits) < p->nn) ++p->colbits;
  // (running sums read back bring up to csr_cap distinct entries of their own)
  const double avg = p->nn > 0 ? (double)(p->nel * p->te) / (double)p->nn : 1.0;
  const double u_row = std::max(1.0, avg / (m->elem == KB_TET4 ? 7.4 : 2.5) +
                                         (p->nn > 0 ? (double)csr_cap / (double)p->nn : 0.0));
  const int s2_max = std::min(8, 31 - p->colbits);
  if (sub_bits) {
    if (sub_bits > s2_max) return KB_EINVAL;
    p->s2 = sub_bits;
  } else {
    int s2 = 0;
    while (s2 < s2_max && ((double)(1 << (s2 + 1))) * u_row <= kSubEntries) ++s2;
    p->s2 = s2;
  }
  // hash slots: about four per expected distinct entry (short probe chains)
  p->ht = kHTMin;
  while (p->ht < kHTMax && p->ht < 4.0 * (double)(1 << p->s2) * u_row) p->ht *= 2;
  if (bucket_bits) {
    p->s1 = bucket_bits < p->s2 ? p->s2 : bucket_bits;
  } else {
    const int64_t nsub_min = div_up(p->nn > 0 ? p->nn : 1, (int64_t)1 << p->s2);
    int d = ilog2_ceil(div_up(nsub_min, kTargetBuckets));
    if (d > 10) d = 10;
    // rows are stored within their bucket in 16 bits: at most 2^16 rows per bucket
    p->s1 = std::min(16, p->s2 + d);
  }
  if (p->s1 - p->s2 > 10) return KB_EINVAL;
  // pass-1 staging per tile (bytes): the smallest tile the plan may take, and the scan words
  const size_t wide_tile = std::min<size_t>(256, std::max<size_t>(1, kWideStage / ((size_t)p->te * (8 + p->vbytes))));
  const size_t stage_min = p->nen <= 8 ? (size_t)(p->nen == 4 ? (prec == KB_FP64 ? 384 : 512) : 128) * p->te *
                                                 (8 + p->vbytes) + 4 * (2 * 512 / 64 + 2)
                                       : wide_tile * p->te * (8 + p->vbytes) + 4 * (kWideThreads / 64 + 2) +
                                             wide_tile * ((size_t)p->nen * 12 + 4) + 2 * (size_t)p->te;
  if (!bucket_bits && !sub_bits) {
    // very many rows: pass 1 keeps two LDS counters per bucket beside its staged pairs;
    // widen the buckets (beyond 1024 sub-buckets per bucket, the sub-buckets too) until
    // they fit beside the smallest tile
    // (the sub-bucket key packs the row within its sub-bucket beside the column in 31
    // bits, so the sub-buckets widen only up to s2_max: about 1.3e8 rows at most)
    while (p->s1 < 16 && stage_min + 8 * (size_t)div_up(p->nn, (int64_t)1 << p->s1) > 163840) {
      if (p->s1 + 1 - p->s2 > 10) {
        if (p->s2 + 1 > s2_max) break;
        ++p->s2;
        while (p->ht < kHTMax && p->ht < 4.0 * (double)(1 << p->s2) * u_row) p->ht *= 2;
      }
      ++p->s1;
    }
  }
  if (tu && tu->table_slots) p->ht = tu->table_slots;
  p->p2 = 1 << (p->s1 - p->s2);
  p->nb = (int)div_up(p->nn, (int64_t)1 << p->s1);
  p->nsub = (int64_t)p->nb * p->p2;
  // the direct way's sub-buckets fill the table further, so an entry's average number of
  // elements has to be known better: elements that share no node give a row (nen + 1) / 2
  // entries, each of one element; with more elements a row (1-cell beams, 1-cell sheets, boxes)
  // its entries grow as the power of its pairs that meets the boxes' figure above (a sheet's and
  // a beam's within 8%: 9.5 and 6.5 entries a row of bricks, 6 and 4.5 of tetrahedra)
  const double u_alone = 0.5 * (p->nen + 1);
  const double u_wide = std::max(u_row, u_alone * pow(std::max(1.0, avg / u_alone), m->elem == KB_TET4 ? 0.37 : 0.546) +
                                            (p->nn > 0 ? (double)csr_cap / (double)p->nn : 0.0));
  p->s2d = p->s2;
  if (!sub_bits && p->nsub >= kWideSubs)
    while (p->s2d < s2_max && (double)(2 << p->s2d) * u_wide <= kDirectLoad * p->ht) ++p->s2d;
  auto set_direct = [&](int s2d) {
    p->s2d = s2d;
    p->nsub_d = s2d == p->s2 ? p->nsub : div_up(p->nn, (int64_t)1 << s2d);
  };
  set_direct(p->s2d);
  // pass-1 tiles: pairs staged in LDS as (8-byte key, value).  Up to 8 rows: one
  // element per lane, `block` may pick the half-size tile (two workgroups per CU);
  // more rows (several DOFs per node): as many elements as keep the staged pairs near
  // 110 KB, on kWideThreads threads
  auto lds_of = [&](int tile, int mode) {
    const size_t slots = 4 * PairOut<double>::slot_words(mode, p->nb, p->nsub_d);
    if (p->nen <= 8)  // (scan words for up to two lanes per element)
      return (size_t)tile * p->te * (8 + p->vbytes) + slots + 4 * (2 * (size_t)tile / 64 + 2);
    return (size_t)tile * p->te * (8 + p->vbytes) + slots + 4 * (kWideThreads / 64 + 2) +
           (size_t)tile * p->nen * 12 + 4 * (size_t)tile + 2 * (size_t)p->te;
  };
  bool tile_set = false;
  if (p->nen <= 8) {
    const int big = p->nen == 4 ? (prec == KB_FP64 ? 768 : 1024) : 256;
    const int small = big / 2 % 64 == 0 ? big / 2 : 64 * ((big / 2 + 63) / 64);
    // FP64 with 8 rows: the 256 tile's staged pairs take 147 KB; with more than about
    // 2000 buckets their counters no longer fit beside it, and a 192 tile takes over
    // (measured on the 27M bricks, FP64: 256 lanes, one wave on each SIMD, pass 1
    // 12.2 -> 9.5 ms against 192)
    const int mid = (p->nen == 8 && prec == KB_FP64) ? 192 : 0;
    p->tile = big;
    // bricks: the half tile (two workgroups per CU, one's gathers under the other's
    // writes) when the tile x bucket histogram it doubles stays small next to the pairs
    // (measured: randomly numbered 1M bricks 10% faster pass 1; the 256-brick batch, whose
    // histogram is 1/6 of its pairs, 4% slower overall)
    if (m->elem == KB_HEX8 && p->dof == 1 && p->nb > 0 &&
        (double)p->T >= kHalfTileRatio * (double)p->nb * (double)div_up(p->nel, small))
      p->tile = small;
    tile_set = tu && (tu->block == big || tu->block == small || (mid && tu->block == mid));
    if (tile_set) p->tile = tu->block;
    if (mid && p->tile == big && lds_of(big, kTwoLevel) > 163840) p->tile = mid;
    if (lds_of(p->tile, kTwoLevel) > 163840) p->tile = small;  // many buckets: the counters need the room
  } else {
    p->tile = (int)wide_tile;
  }
  // where pass 1 sends its pairs (kb_assemble.hpp): widths set by hand mean the two levels
  p->mode = kTwoLevel;
  if (p->nel > 0 && p->nb > 0 && !(tu && (tu->bucket_bits || tu->seg_pairs))) {
    const int s2d = p->s2d;
    set_direct(p->s2);  // few sub-buckets: their number, not their size, keeps the device busy
    if (csr_cap == 0 && p->nsub_d <= kSlotsArray) {
      int tile = p->tile;
      if (p->nen <= 8 && !tile_set && div_up(p->nel, tile) < kDirectTiles) tile = kSmallTile;
      if (div_up(p->nel, tile) * p->nsub_d <= kDirectRuns && lds_of(tile, kDirect) <= 163840) {
        p->mode = kDirect;
        p->tile = tile;
      }
    }
    if (p->mode == kTwoLevel) {
      set_direct(s2d);
      if (lds_of(p->tile, kAsk) <= 163840) p->mode = kAsk;
    }
  }
  p->lds1 = lds_of(p->tile, p->mode);
  p->ntiles = div_up(p->nel, p->tile);
  p->ntiles_csr = div_up(csr_cap, kCsrTile);
  p->nhist = p->mode == kDirect ? 0 : (int64_t)p->nb * (p->ntiles + p->ntiles_csr);
  p->lds_csr = 2 * (size_t)kCsrTile * (8 + p->vbytes) + 4 * PairOut<double>::slot_words(p->mode, p->nb, p->nsub_d) +
               4 * (kCsrThreads / 64 + 2);
  if (csr_cap > 0 && p->lds_csr > 163840) return KB_EINVAL;
  if (tu && tu->seg_pairs)
    p->seg = tu->seg_pairs;
  else
    p->seg = (m->elem == KB_TET4 && (int64_t)kSeg < (int64_t)kMinRun * p->p2) ? kSegLong : kSeg;
  p->nseg_max = div_up(p->T, p->seg) + p->nb;
  p->lds2 = (size_t)p->seg * (p->vbytes + 4 + 2) + 2 * 4 * (size_t)p->p2 + 4 * (kSegThreads / 64 + 1);
  if (p->lds1 > 163840 || p->lds2 > 163840) return KB_EINVAL;
  size_t off = 0;
  auto take = [&](size_t bytes) {  // every region at least one aligned block
    size_t o = off;
    off = align_up(off + (bytes > 0 ? bytes : 1));
    return o;
  };
  const size_t T = (size_t)p->T;
  p->o_coords4 = take(p->dof > 1 ? 0 : 32 * (size_t)p->nn);  // assembly with several DOFs: no geometry
  p->o_hist = take(4 * (size_t)p->nhist);
  p->o_csum = take(4 * (size_t)div_up(p->ntiles + p->ntiles_csr, kColChunk) * (size_t)p->nb);
  p->o_tot = take(4 * (size_t)p->nb);
  p->o_part = take(4 * (size_t)(div_up(p->nsub, kScanChunk) + 1));
  p->o_bstart = take(4 * ((size_t)p->nb + 1));
  p->o_segbase = take(4 * ((size_t)p->nb + 1));
  p->o_hist2 = take(4 * (size_t)(p->nseg_max * p->p2));  // (direct: the nsub sub-bucket counters)
  p->o_seg2b = take(4 * (size_t)p->nseg_max);
  p->o_head = take(4 * kHeadWords);      // largest value exponent, heavy sub-buckets, ... (k_begin)
  p->o_ovl = take(4 * (size_t)p->nsub);  // heavy sub-buckets (k_heavy)
  p->o_hvy = take(4 * ((size_t)kHeavyPar * kHvyWords + kBigWords));  // their split tables and big leaves
  p->o_dconn = take(p->dof > 1 ? 4 * (size_t)p->nen * (size_t)p->nel : 0);  // expanded connectivity
  p->o_tres = take(csr_cap > 0 ? p->vbytes * T : 0);  // residuals of the reduced entries
  p->o_row1 = take(2 * T);
  p->o_col1 = take(4 * T);
  p->o_val1 = take(p->vbytes * T);
  p->o_key2 = take(4 * T);
  p->o_val2 = take(p->vbytes * T);
  p->o_sbb = take(4 * ((size_t)p->nsub + 1));
  p->o_rowoff = take(4 * (size_t)p->nn);
  p->o_usub = take(4 * ((size_t)p->nsub + 1));
  p->o_ubase = take(4 * ((size_t)p->nsub + 1));
  p->total = off;
  return KB_OK;
}

template <int NEN>
int dispatch_build(const Plan& p, const kb_mesh* m, const void* klow, unsigned char* ws, int32_t* row_ptr,
                   int32_t* col_idx, void* vals, int64_t cap, int64_t* nnz_dev, uint32_t* status, Events& ev,
                   hipStream_t s, const Carry* cr = nullptr, const BatchRows* br = nullptr) {
  switch (p.prec) {
    case KB_FP64:
      return build_impl<NEN, Prec::F64>(p, m, klow, ws, row_ptr, col_idx, vals, cap, nnz_dev, status, ev, s, cr, br);
    case KB_FP32:
      return build_impl<NEN, Prec::F32>(p, m, klow, ws, row_ptr, col_idx, vals, cap, nnz_dev, status, ev, s, cr, br);
    default:
      return build_impl<NEN, Prec::F32FB>(p, m, klow, ws, row_ptr, col_idx, vals, cap, nnz_dev, status, ev, s, cr, br);
  }
}

// Grouped build workspace: one pass's (the largest group plus the running sums read
// back), then the second set of running sums (CSR, residuals, rows, count) and the
// residuals and rows of the caller's set.  Passes alternate between the two sets so
// that the last one writes the caller's arrays.
struct GroupPlan {
  Plan p;
  int64_t group = 0, n_groups = 0;
  size_t o_rpB = 0, o_colB = 0, o_valB = 0, o_resB = 0, o_rowsB = 0, o_nnzB = 0, o_resA = 0, o_rowsA = 0, total = 0;
};

int make_group_plan(const kb_mesh* m, int prec, const kb_tuning* tu, int64_t group_elems, int64_t cap,
                    GroupPlan* gp) {
  if (!m || group_elems < 1 || cap < 0 || m->n_elem < 0) return KB_EINVAL;
  if (m->op != KB_OP_STIFFNESS && m->op != KB_OP_MASS) return KB_EINVAL;
  if (cap >= (int64_t)INT32_MAX) return KB_ERANGE;
  gp->group = std::min<int64_t>(group_elems, std::max<int64_t>(m->n_elem, 1));
  gp->n_groups = std::max<int64_t>(1, div_up(m->n_elem, gp->group));
  kb_mesh g = *m;
  g.n_elem = std::min<int64_t>(gp->group, m->n_elem);
  KB_TRY(make_plan(&g, prec, tu, &gp->p, 1, gp->n_groups > 1 ? cap : 0));
  size_t off = gp->p.total;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + (bytes > 0 ? bytes : 1));
    return o;
  };
  const size_t c = gp->n_groups > 1 ? (size_t)cap : 0, vb = gp->p.vbytes;
  gp->o_rpB = take(gp->n_groups > 1 ? 4 * ((size_t)gp->p.nn + 1) : 0);
  gp->o_colB = take(4 * c);
  gp->o_valB = take(vb * c);
  gp->o_resB = take(vb * c);
  gp->o_rowsB = take(4 * c);
  gp->o_nnzB = take(8);
  gp->o_resA = take(vb * c);
  gp->o_rowsA = take(4 * c);
  gp->total = off;
  return KB_OK;
}

template <int NEN>
int dispatch_integrate(const Plan& p, const kb_mesh* m, void* vals, uint32_t* status, Events& ev, hipStream_t s) {
  switch (p.prec) {
    case KB_FP64:
      return integrate_impl<NEN, Prec::F64>(p, m, vals, status, ev, s);
    case KB_FP32:
      return integrate_impl<NEN, Prec::F32>(p, m, vals, status, ev, s);
    default:
      return integrate_impl<NEN, Prec::F32FB>(p, m, vals, status, ev, s);
  }
}

// the batch as one mesh (its connectivity replaced by the shifted copy at launch)
int batch_as_mesh(const kb_batch* b, kb_mesh* m) {
  if (!b || b->n_mesh < 0) return KB_EINVAL;
  *m = kb_mesh{b->elem, KB_OP_STIFFNESS, b->n_elem, b->n_node, b->conn, b->coords, b->coef};
  return KB_OK;
}

// batch workspace: the pipeline's, then the shifted connectivity and one flag word
struct BatchPlan {
  Plan p;
  size_t o_gconn = 0, o_flags = 0, total = 0;
};

int make_batch_plan(const kb_batch* b, int prec, const kb_tuning* tu, BatchPlan* bp) {
  kb_mesh m;
  KB_TRY(batch_as_mesh(b, &m));
  KB_TRY(make_plan(&m, prec, tu, &bp->p));
  size_t off = bp->p.total;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + (bytes > 0 ? bytes : 1));
    return o;
  };
  bp->o_gconn = take(4 * (size_t)bp->p.nen * (size_t)bp->p.nel);
  // (not used, once the union's row pointers: the plan is at least this much above a mesh's)
  take(4 * ((size_t)bp->p.nn + 1));
  bp->o_flags = take(4);
  bp->total = off;
  return KB_OK;
}

int check_mesh_ptrs(const kb_mesh* m, bool need_geometry) {
  if ((m->n_elem > 0 && !m->conn)) return KB_EINVAL;
  if (need_geometry && m->n_elem > 0 && (!m->coords || !m->coef)) return KB_EINVAL;
  return KB_OK;
}

}  // namespace

// adjoint workspace: corner records and places, the large buckets' node accumulators,
// bucket counts and starts, head words, the list of large buckets
namespace {
struct AdjointPlan {
  int bits = kAdjMinBits;  // nodes per bucket: 2^bits
  int64_t nb = 0, extra = 0;  // buckets; workgroups beyond one a bucket at most
  size_t o_rec = 0, o_rel = 0, o_acc = 0, o_cnt = 0, o_start = 0, o_head = 0, o_big = 0, total = 0;
};

int make_adjoint_plan(const kb_mesh* m, AdjointPlan* p) {
  if (!m) return KB_EINVAL;
  if (m->elem != KB_HEX8 && m->elem != KB_TET4) return KB_EINVAL;
  if (m->n_elem < 0 || m->n_node < 0 || m->op != KB_OP_STIFFNESS) return KB_EINVAL;
  if (m->n_node >= (int64_t)INT32_MAX || m->n_elem > (int64_t)INT32_MAX / m->elem) return KB_ERANGE;
  while (p->bits < kAdjMaxBits && div_up(m->n_node, (int64_t)1 << p->bits) > kAdjBuckets) ++p->bits;
  p->nb = div_up(m->n_node, (int64_t)1 << p->bits);
  const size_t nc = (size_t)m->elem * (size_t)m->n_elem;
  p->extra = (int64_t)(nc / kAdjChunk);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + (bytes > 0 ? bytes : 1));
    return o;
  };
  p->o_rec = take(sizeof(AdjointRecord) * nc);
  p->o_rel = take(4 * nc);
  p->o_acc = take(8 * kAdjAcc * ((size_t)std::min(p->extra, p->nb) << p->bits));
  p->o_cnt = take(4 * (size_t)p->nb);
  p->o_start = take(4 * ((size_t)p->nb + 1));
  p->o_head = take(16);
  p->o_big = take(12 * (size_t)p->extra);
  p->total = off;
  return KB_OK;
}

template <int NEN>
int launch_adjoint(const AdjointPlan& p, const kb_mesh* m, const int32_t* row_ptr, const int32_t* col_idx,
                   const double* w, int64_t nnz, unsigned char* ws, double* grad_coef, double* grad_coords,
                   uint32_t* status, hipStream_t s) {
  auto* rec = (AdjointRecord*)(ws + p.o_rec);
  auto* rel = (uint32_t*)(ws + p.o_rel);
  auto* acc = (unsigned long long*)(ws + p.o_acc);
  auto* cnt = (uint32_t*)(ws + p.o_cnt);
  auto* start = (uint32_t*)(ws + p.o_start);
  auto* head = (uint32_t*)(ws + p.o_head);
  auto* big = (uint32_t*)(ws + p.o_big);
  const int64_t nel = m->n_elem, nn = m->n_node;
  const int nb = (int)p.nb;
  k_adjoint_begin<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>(div_up(p.nb, 256), 1024)), 256, 0, s>>>(
      status, head, cnt, p.nb);
  KB_LAUNCH_CHECK();
  // (also without elements or nodes: the bucket starts, the flags)
  const size_t slots = 4 * (size_t)(nb <= kAdjArray ? std::max(nb, 1) : 2 * kSlotsHash);
  k_adjoint_count<NEN><<<(unsigned)std::max<int64_t>(1, div_up(nel, 256 * kAdjPer)), 256, slots, s>>>(
      m->conn, nel, nn, p.bits, nb, cnt, start, rel, head, big);
  KB_LAUNCH_CHECK();
  if (nel > 0) {
    k_adjoint_elems<NEN><<<grid_for(nel, kAdjElemThreads), kAdjElemThreads, 0, s>>>(
        m->conn, m->coords, m->coef, nel, nn, row_ptr, col_idx, nnz, w, grad_coef, p.bits, start, rel, rec, acc, head,
        big, status);
    KB_LAUNCH_CHECK();
  }
  if (nn > 0) {
    const size_t lds = (size_t)48 << p.bits;
    if (!set_lds(k_adjoint_reduce, lds)) return KB_EHIP;
    k_adjoint_reduce<<<(unsigned)(p.nb + p.extra), kAdjThreads, lds, s>>>(rec, start, nn, p.bits, nb, head, big, acc,
                                                                          grad_coords);
    KB_LAUNCH_CHECK();
  }
  return KB_OK;
}
}  // namespace

// Fixed scratch of kb_build_lower_csr_noalloc: one copy per device, resident until the
// process ends.  Host code never uses the array's name as an address: the device address
// is looked up once per device (hipGetSymbolAddress) and kept in scratch_ptr.
static __device__ __align__(256) unsigned char scratch[KB_SCRATCH_BYTES];

static constexpr int kMaxDevices = 64;

// device address of this device's scratch array, looked up on the first call per device
static int scratch_address(void** out) {
  static std::atomic<void*> scratch_ptr[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KB_EHIP;
  void* ptr = scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return KB_EHIP;
    scratch_ptr[dev].store(ptr, std::memory_order_release);
  }
  *out = ptr;
  return KB_OK;
}

extern "C" {

int kb_version(void) { return KB_VERSION; }

const char* kb_status_string(int code) {
  switch (code) {
    case KB_OK: return "ok";
    case KB_EINVAL: return "invalid argument";
    case KB_ERANGE: return "size exceeds int32 indexing";
    case KB_ENOSPC: return "workspace too small";
    case KB_EHIP: return "HIP launch failure";
    case (int)KB_F_INDEX: return "node id out of range";
    case (int)KB_F_REPEAT: return "node repeated within an element";
    case (int)KB_F_INVERTED: return "non-positive Jacobian determinant";
    case (int)KB_F_NONFINITE: return "non-finite input or value";
    case (int)KB_F_CAPACITY: return "nnz exceeds capacity";
    default: return "unknown status";
  }
}

int kb_plan(const kb_mesh* mesh, int prec, const kb_tuning* tuning, size_t* ws_bytes, int64_t* n_triplets) {
  Plan p;
  KB_TRY(make_plan(mesh, prec, tuning, &p));
  if (ws_bytes) *ws_bytes = p.total;
  if (n_triplets) *n_triplets = p.T;
  return KB_OK;
}

static_assert(kTwoLevel == KB_WAY_BUCKETS && kDirect == KB_WAY_DIRECT && kAsk == KB_WAY_SAMPLED, "as in the header");

int kb_plan_way(const kb_mesh* mesh, int prec, const kb_tuning* tuning, int32_t* way, int32_t* tile, size_t* way_at) {
  Plan p;
  KB_TRY(make_plan(mesh, prec, tuning, &p));
  if (way) *way = p.mode;
  if (tile) *tile = p.tile;
  if (way_at) *way_at = p.o_head + 4 * kHeadWay;
  return KB_OK;
}

// use_scratch: the library's fixed scratch array is the workspace (ws, ws_bytes ignored);
// every host check comes before the device is touched
static int build_common(const kb_mesh* mesh, int prec, const kb_tuning* tuning, const void* klow, void* ws,
                        size_t ws_bytes, int32_t* row_ptr, int32_t* col_idx, void* vals, int64_t cap, int64_t* nnz_dev,
                        uint32_t* status_dev, void* stream, bool use_scratch = false) {
  Plan p;
  KB_TRY(make_plan(mesh, prec, tuning, &p));
  KB_TRY(check_mesh_ptrs(mesh, klow == nullptr));
  if (!row_ptr || !nnz_dev || !status_dev || cap < 0) return KB_EINVAL;
  if (cap > 0 && (!col_idx || !vals)) return KB_EINVAL;
  if (use_scratch) {
    if (p.total > (size_t)KB_SCRATCH_BYTES) return KB_ENOSPC;
    KB_TRY(scratch_address(&ws));
    ws_bytes = (size_t)KB_SCRATCH_BYTES;
  }
  if (ws_bytes < p.total) return KB_ENOSPC;
  if (p.total > 0 && !ws) return KB_EINVAL;
  KB_TRY(device_cus(&p.cus));
  Events ev{tuning ? tuning->stage_events : nullptr, (hipStream_t)stream};
  auto* w = (unsigned char*)ws;
  auto s = (hipStream_t)stream;
  if (p.nen == 8) return dispatch_build<8>(p, mesh, klow, w, row_ptr, col_idx, vals, cap, nnz_dev, status_dev, ev, s);
  return dispatch_build<4>(p, mesh, klow, w, row_ptr, col_idx, vals, cap, nnz_dev, status_dev, ev, s);
}

int kb_build_lower_csr(const kb_mesh* mesh, int prec, const kb_tuning* tuning, void* ws, size_t ws_bytes,
                       int32_t* row_ptr, int32_t* col_idx, void* vals, int64_t cap, int64_t* nnz_dev,
                       uint32_t* status_dev, void* stream) {
  return build_common(mesh, prec, tuning, nullptr, ws, ws_bytes, row_ptr, col_idx, vals, cap, nnz_dev, status_dev,
                      stream);
}

int kb_build_lower_csr_noalloc(const kb_mesh* mesh, int prec, const kb_tuning* tuning, int32_t* row_ptr,
                               int32_t* col_idx, void* vals, int64_t cap, int64_t* nnz_dev, uint32_t* status_dev,
                               void* stream) {
  return build_common(mesh, prec, tuning, nullptr, nullptr, 0, row_ptr, col_idx, vals, cap, nnz_dev, status_dev,
                      stream, true);
}

int kb_assemble_lower_csr(const kb_mesh* mesh, int prec, const kb_tuning* tuning, const void* klow, void* ws,
                          size_t ws_bytes, int32_t* row_ptr, int32_t* col_idx, void* vals, int64_t cap,
                          int64_t* nnz_dev, uint32_t* status_dev, void* stream) {
  if (!mesh) return KB_EINVAL;
  if (mesh->n_elem > 0 && !klow) return KB_EINVAL;
  // klow selects the assembly-only path; a non-null marker is needed even when empty
  static const double kEmpty = 0.0;
  return build_common(mesh, prec, tuning, klow ? klow : (const void*)&kEmpty, ws, ws_bytes, row_ptr, col_idx, vals,
                      cap, nnz_dev, status_dev, stream);
}

int kb_plan_dof(const kb_mesh* mesh, int dof, int prec, const kb_tuning* tuning, size_t* ws_bytes,
                int64_t* n_triplets) {
  Plan p;
  KB_TRY(make_plan(mesh, prec, tuning, &p, dof));
  if (ws_bytes) *ws_bytes = p.total;
  if (n_triplets) *n_triplets = p.T;
  return KB_OK;
}

int kb_assemble_lower_csr_dof(const kb_mesh* mesh, int dof, int prec, const kb_tuning* tuning, const void* klow,
                              void* ws, size_t ws_bytes, int32_t* row_ptr, int32_t* col_idx, void* vals, int64_t cap,
                              int64_t* nnz_dev, uint32_t* status_dev, void* stream) {
  if (dof == 1)
    return kb_assemble_lower_csr(mesh, prec, tuning, klow, ws, ws_bytes, row_ptr, col_idx, vals, cap, nnz_dev,
                                 status_dev, stream);
  Plan p;
  KB_TRY(make_plan(mesh, prec, tuning, &p, dof));
  KB_TRY(check_mesh_ptrs(mesh, false));
  if (p.nel > 0 && !klow) return KB_EINVAL;
  if (!row_ptr || !nnz_dev || !status_dev || cap < 0) return KB_EINVAL;
  if (cap > 0 && (!col_idx || !vals)) return KB_EINVAL;
  if (ws_bytes < p.total) return KB_ENOSPC;
  if (!ws) return KB_EINVAL;
  KB_TRY(device_cus(&p.cus));
  auto* w = (unsigned char*)ws;
  auto s = (hipStream_t)stream;
  // the DOF view: elements of nen * dof rows over dof * n_node global DOFs
  kb_mesh vm = *mesh;
  vm.elem = p.nen;
  vm.n_node = p.nn;
  vm.conn = (const int32_t*)(w + p.o_dconn);
  if (p.nel > 0) {
    const int64_t n = p.nel * mesh->elem;
    k_dof_conn<<<(unsigned)std::min<int64_t>(div_up(n, 256), 65536), 256, 0, s>>>(mesh->conn, n, dof,
                                                                                   (int32_t*)(w + p.o_dconn));
    KB_LAUNCH_CHECK();
  }
  static const double kEmpty = 0.0;
  const void* kl = klow ? klow : (const void*)&kEmpty;  // selects the assembly-only path
  Events ev{tuning ? tuning->stage_events : nullptr, s};
  switch (p.nen) {
    case 8:  // tetrahedra, 2 DOFs
      return dispatch_build<8>(p, &vm, kl, w, row_ptr, col_idx, vals, cap, nnz_dev, status_dev, ev, s);
    case 12:
      return dispatch_build<12>(p, &vm, kl, w, row_ptr, col_idx, vals, cap, nnz_dev, status_dev, ev, s);
    case 16:
      return dispatch_build<16>(p, &vm, kl, w, row_ptr, col_idx, vals, cap, nnz_dev, status_dev, ev, s);
    case 24:
      return dispatch_build<24>(p, &vm, kl, w, row_ptr, col_idx, vals, cap, nnz_dev, status_dev, ev, s);
    default:
      return KB_EINVAL;
  }
}

int kb_plan_grouped(const kb_mesh* mesh, int prec, const kb_tuning* tuning, int64_t group_elems, int64_t cap,
                    size_t* ws_bytes) {
  GroupPlan gp;
  KB_TRY(make_group_plan(mesh, prec, tuning, group_elems, cap, &gp));
  if (ws_bytes) *ws_bytes = gp.total;
  return KB_OK;
}

// One pass g of a grouped build: group g's elements (conn_g, coef_g: its n_elem rows)
// integrated and assembled together with the running sums of the passes before it.
// The two sets of running sums alternate (A = the caller's arrays, B = workspace) so
// that the last pass writes the caller's arrays.
static int grouped_pass(const GroupPlan& gp, const kb_mesh* mesh, int64_t g, const int32_t* conn_g,
                        const double* coef_g, unsigned char* w, int32_t* row_ptr, int32_t* col_idx, void* vals,
                        int64_t cap, int64_t* nnz_dev, uint32_t* status_dev, const kb_tuning* tuning, hipStream_t s) {
  Events none{nullptr, s};
  Events ev{tuning ? tuning->stage_events : nullptr, s};
  struct Set {
    int32_t* rp;
    int32_t* col;
    void* val;
    void* res;
    int32_t* rows;
    int64_t* nnz;
  };
  const Set A{row_ptr, col_idx, vals, w + gp.o_resA, (int32_t*)(w + gp.o_rowsA), nnz_dev};
  const Set B{(int32_t*)(w + gp.o_rpB), (int32_t*)(w + gp.o_colB), w + gp.o_valB, w + gp.o_resB,
              (int32_t*)(w + gp.o_rowsB), (int64_t*)(w + gp.o_nnzB)};
  kb_mesh mg = *mesh;  // this group's elements as a mesh; all nodes
  const int64_t e0 = g * gp.group;
  mg.n_elem = std::max<int64_t>(0, std::min<int64_t>(gp.group, mesh->n_elem - e0));
  mg.conn = conn_g;
  mg.coef = coef_g;
  Plan p = gp.p;
  p.nel = mg.n_elem;
  p.ntiles = div_up(p.nel, p.tile);
  const Set& out = ((gp.n_groups - 1 - g) % 2 == 0) ? A : B;
  const Set& in = (&out == &A) ? B : A;
  Carry cr;
  cr.first = g == 0;
  if (g > 0) {
    cr.rows = in.rows;
    cr.cols = in.col;
    cr.vals = in.val;
    cr.res = in.res;
    cr.nnz = in.nnz;
  }
  cr.res_out = out.res;
  cr.rows_out = out.rows;
  const Carry* crp = gp.n_groups > 1 ? &cr : nullptr;
  Events& e = g == gp.n_groups - 1 ? ev : none;
  if (p.nen == 8)
    return dispatch_build<8>(p, &mg, nullptr, w, out.rp, out.col, out.val, cap, out.nnz, status_dev, e, s, crp);
  return dispatch_build<4>(p, &mg, nullptr, w, out.rp, out.col, out.val, cap, out.nnz, status_dev, e, s, crp);
}

static int check_grouped_args(const GroupPlan& gp, int32_t* row_ptr, int32_t* col_idx, void* vals, int64_t cap,
                              int64_t* nnz_dev, uint32_t* status_dev, void* ws, size_t ws_bytes) {
  if (!row_ptr || !nnz_dev || !status_dev) return KB_EINVAL;
  if (cap > 0 && (!col_idx || !vals)) return KB_EINVAL;
  if (ws_bytes < gp.total) return KB_ENOSPC;
  if (!ws) return KB_EINVAL;
  return KB_OK;
}

int kb_build_lower_csr_grouped(const kb_mesh* mesh, int prec, const kb_tuning* tuning, int64_t group_elems, void* ws,
                               size_t ws_bytes, int32_t* row_ptr, int32_t* col_idx, void* vals, int64_t cap,
                               int64_t* nnz_dev, uint32_t* status_dev, void* stream) {
  GroupPlan gp;
  KB_TRY(make_group_plan(mesh, prec, tuning, group_elems, cap, &gp));
  KB_TRY(check_mesh_ptrs(mesh, true));
  KB_TRY(check_grouped_args(gp, row_ptr, col_idx, vals, cap, nnz_dev, status_dev, ws, ws_bytes));
  KB_TRY(device_cus(&gp.p.cus));
  for (int64_t g = 0; g < gp.n_groups; ++g) {
    const int64_t e0 = g * gp.group;
    const int32_t* cg = mesh->n_elem > 0 ? mesh->conn + e0 * mesh->elem : nullptr;
    const double* fg = mesh->n_elem > 0 ? mesh->coef + e0 : nullptr;
    KB_TRY(grouped_pass(gp, mesh, g, cg, fg, (unsigned char*)ws, row_ptr, col_idx, vals, cap, nnz_dev, status_dev,
                        tuning, (hipStream_t)stream));
  }
  return KB_OK;
}

int kb_build_lower_csr_group_pass(const kb_mesh* mesh, int prec, const kb_tuning* tuning, int64_t group_elems,
                                  int64_t group, const int32_t* group_conn, const double* group_coef, void* ws,
                                  size_t ws_bytes, int32_t* row_ptr, int32_t* col_idx, void* vals, int64_t cap,
                                  int64_t* nnz_dev, uint32_t* status_dev, void* stream) {
  GroupPlan gp;
  KB_TRY(make_group_plan(mesh, prec, tuning, group_elems, cap, &gp));
  if (group < 0 || group >= gp.n_groups) return KB_EINVAL;
  const int64_t ng = std::max<int64_t>(0, std::min<int64_t>(gp.group, mesh->n_elem - group * gp.group));
  if (ng > 0 && (!group_conn || !group_coef || !mesh->coords)) return KB_EINVAL;
  KB_TRY(check_grouped_args(gp, row_ptr, col_idx, vals, cap, nnz_dev, status_dev, ws, ws_bytes));
  KB_TRY(device_cus(&gp.p.cus));
  return grouped_pass(gp, mesh, group, group_conn, group_coef, (unsigned char*)ws, row_ptr, col_idx, vals, cap,
                      nnz_dev, status_dev, tuning, (hipStream_t)stream);
}

int kb_plan_batched(const kb_batch* batch, int prec, const kb_tuning* tuning, size_t* ws_bytes,
                    int64_t* n_triplets) {
  BatchPlan bp;
  KB_TRY(make_batch_plan(batch, prec, tuning, &bp));
  if (ws_bytes) *ws_bytes = bp.total;
  if (n_triplets) *n_triplets = bp.p.T;
  return KB_OK;
}

int kb_build_lower_csr_batched(const kb_batch* batch, int prec, const kb_tuning* tuning, void* ws, size_t ws_bytes,
                               int32_t* row_ptr, int32_t* col_idx, void* vals, int64_t cap, int64_t* nnz_off,
                               uint32_t* status_dev, void* stream) {
  BatchPlan bp;
  KB_TRY(make_batch_plan(batch, prec, tuning, &bp));
  Plan& p = bp.p;
  kb_mesh m;
  KB_TRY(batch_as_mesh(batch, &m));
  KB_TRY(check_mesh_ptrs(&m, true));
  if (!batch->elem_off || !batch->node_off || !row_ptr || !nnz_off || !status_dev || cap < 0) return KB_EINVAL;
  if (cap > 0 && (!col_idx || !vals)) return KB_EINVAL;
  if (ws_bytes < bp.total) return KB_ENOSPC;
  if (!ws) return KB_EINVAL;
  KB_TRY(device_cus(&p.cus));
  auto* w = (unsigned char*)ws;
  auto s = (hipStream_t)stream;
  auto* gconn = (int32_t*)(w + bp.o_gconn);
  auto* flags = (uint32_t*)(w + bp.o_flags);
  const int64_t nm = batch->n_mesh;
  k_fill_i32<<<1, 64, 0, s>>>((int32_t*)flags, 1, 0);
  KB_LAUNCH_CHECK();
  k_batch_check<<<grid_for(nm + 1, 256), 256, 0, s>>>(batch->elem_off, batch->node_off, nm, p.nel, p.nn, flags);
  KB_LAUNCH_CHECK();
  if (p.nel > 0 && nm > 0) {
    const unsigned g = (unsigned)std::min<int64_t>(div_up(p.nel, 256), 65536);
    if (p.nen == 8)
      k_batch_conn<8><<<g, 256, 0, s>>>(batch->conn, batch->elem_off, batch->node_off, nm, p.nel, flags, gconn);
    else
      k_batch_conn<4><<<g, 256, 0, s>>>(batch->conn, batch->elem_off, batch->node_off, nm, p.nel, flags, gconn);
    KB_LAUNCH_CHECK();
    m.conn = gconn;
  }
  // the batch's matrix, written mesh by mesh; nnz_off[n_mesh] receives the total
  Events ev{tuning ? tuning->stage_events : nullptr, s};
  const BatchRows br{batch->node_off, nm, flags};
  if (p.nen == 8)
    KB_TRY(dispatch_build<8>(p, &m, nullptr, w, row_ptr, col_idx, vals, cap, nnz_off + nm, status_dev, ev, s, nullptr,
                             &br));
  else
    KB_TRY(dispatch_build<4>(p, &m, nullptr, w, row_ptr, col_idx, vals, cap, nnz_off + nm, status_dev, ev, s, nullptr,
                             &br));
  k_batch_meshes<<<grid_for(std::max<int64_t>(nm, 1), 256), 256, 0, s>>>(
      (const uint32_t*)(w + p.o_ubase), (const uint32_t*)(w + p.o_rowoff), sub_buckets(p, w), p.nn, batch->node_off,
      nm, flags, row_ptr, nnz_off, status_dev);
  KB_LAUNCH_CHECK();
  return KB_OK;
}

int kb_plan_adjoint(const kb_mesh* mesh, size_t* ws_bytes) {
  AdjointPlan p;
  KB_TRY(make_adjoint_plan(mesh, &p));
  if (ws_bytes) *ws_bytes = p.total;
  return KB_OK;
}

int kb_adjoint_lower(const kb_mesh* mesh, const int32_t* row_ptr, const int32_t* col_idx, const double* w,
                     int64_t nnz, void* ws, size_t ws_bytes, double* grad_coef, double* grad_coords,
                     uint32_t* status_dev, void* stream) {
  AdjointPlan p;
  KB_TRY(make_adjoint_plan(mesh, &p));
  KB_TRY(check_mesh_ptrs(mesh, true));
  if (!status_dev || !ws) return KB_EINVAL;
  if (ws_bytes < p.total) return KB_ENOSPC;
  if (nnz < 0 || nnz >= (int64_t)INT32_MAX) return nnz < 0 ? KB_EINVAL : KB_ERANGE;
  if (mesh->n_elem > 0 && (!row_ptr || !grad_coef || (nnz > 0 && (!col_idx || !w)))) return KB_EINVAL;
  if (mesh->n_node > 0 && !grad_coords) return KB_EINVAL;
  auto* launch = mesh->elem == 8 ? launch_adjoint<8> : launch_adjoint<4>;
  return launch(p, mesh, row_ptr, col_idx, w, nnz, (unsigned char*)ws, grad_coef, grad_coords, status_dev,
                (hipStream_t)stream);
}

int kb_integrate_lower(const kb_mesh* mesh, int prec, const kb_tuning* tuning, void* vals, uint32_t* status_dev,
                       void* stream) {
  Plan p;
  KB_TRY(make_plan(mesh, prec, tuning, &p));
  KB_TRY(check_mesh_ptrs(mesh, true));
  if (!status_dev || (p.nel > 0 && !vals)) return KB_EINVAL;
  Events ev{tuning ? tuning->stage_events : nullptr, (hipStream_t)stream};
  auto s = (hipStream_t)stream;
  if (p.nen == 8) return dispatch_integrate<8>(p, mesh, vals, status_dev, ev, s);
  return dispatch_integrate<4>(p, mesh, vals, status_dev, ev, s);
}

}  // extern "C"
