// Emission: the clipped pieces' cell terms and element records (rpd_common.h) turned into the sums of the cells, faces,
// edges and RPVs, and into the element pieces that the components are found over.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rpd_device.h"
#include "rpd_launch.h"

namespace rpd {

// Workgroups go to the chip's eight dies in turn, each die with an L2 cache of its own: die x takes the x-th eighth of
// the items, so that neighbouring items (pieces of neighbouring tets, which look at the same lines) share a cache.
// f(k) for the items of this thread, in [0, n), by unit consecutive items.
constexpr int DIES = 8;
template <typename F>
__device__ __forceinline__ void for_items(int n, int unit, int first, int step, F f) {  // first, step: among the die's threads
  const int per = ((n + DIES - 1) / DIES + unit - 1) / unit * unit;
  const int k0 = (int)(blockIdx.x % DIES) * per, k1 = min(n, k0 + per);
  for (int k = k0 + first; k < k1; k += step) f(k);
}

// One element piece (element, tet) is emitted exactly once per shape: adding sets its gluing bits and count,
// removing (the same piece recomputed from the state before an incremental update, sign -1) takes both back.
// The two happen in one launch, in either order. Each records the piece's gluing bits in its own half of the
// piece's tag pair; a scan after the launch flags the element for a new union-find only where the two differ (a
// piece put back with the same gluing bits leaves the element's forest as it was).
template <bool HASH>
__device__ inline void node_emit(const ShapeArgs& a, int sign, unsigned long long key, int glue) {
  if (!HASH) return;
  int ns = node_insert(a.N, key, a.status);
  if (ns < 0) return;
  atomicAdd(&a.N.rec[ns].st, sign * (NODE_UNIT + glue));  // removal re-emits the same bits, so this is exact
  if (a.touch_cell) a.removed[2 * (size_t)ns + (sign > 0)] = (unsigned short)(0x100 | glue);
}

// a per-piece element term for sampled comparisons (RPD_KEEP_PIECES only)
__device__ inline void keep_term(const ShapeArgs& a, int kind, int t, int i, int j, int k, int l, int glue,
                                 long long num) {
  if (!(a.flags & RPD_KEEP_PIECES)) return;
  const unsigned long long idx = atomicAdd(&a.counters[C_TERMS], 1ull);
  if (idx < (unsigned long long)a.term_cap) {
    TermRec r;
    r.kind = kind;
    r.t = t;
    r.i = i;
    r.j = j;
    r.k = k;
    r.l = l;
    r.glue = glue;
    r.pad = 0;
    r.num = num;
    a.terms[idx] = r;
  } else {
    atomicOr(a.status, ST_TABLE_FULL);
  }
}

__device__ inline long long fixed56(double v) { return llrint(v * 72057594037927936.0); }  // 2^-56 units

// Cell volumes and first moments are exact sums of 128-bit integers in units of 2^-80 (resolution 8e-25, range
// 2^47), so that a nonempty piece far smaller than a grid cell still counts, every sum is independent of the order
// of the additions, and a removal pass takes its contributions back exactly. An accumulator is a (low, high) pair
// of 64-bit words; an addition adds the low word atomically and carries into the high word only when needed.
struct Fix128 {
  unsigned long long lo;
  long long hi;
};
__device__ inline Fix128 fixed80(double v) {
  const double D = rint(ldexp(v, 80));  // exact scaling, then the nearest integer
  const double h = floor(ldexp(D, -64));
  const double l = D - ldexp(h, 64);    // in [0, 2^64): the low bits of D, exact
  return Fix128{(unsigned long long)l, (long long)h};
}
__device__ inline Fix128 signed128(Fix128 x, int sign) {
  if (sign > 0) return x;
  return Fix128{0ull - x.lo, -x.hi - (x.lo != 0ull ? 1 : 0)};
}
__device__ inline void acc128(unsigned long long* p, Fix128 v) {
  const unsigned long long old = atomicAdd(p, v.lo);
  const long long h = v.hi + (old + v.lo < old ? 1 : 0);  // carry out of the low word
  if (h) atomicAdd(p + 1, (unsigned long long)h);
}

// Sums of a workgroup's cell terms, one slot per site (open addressing): consecutive piece slots belong to
// neighbouring tets, so a few dozen sites own EMIT_PIECES of them and the global accumulators see one addition per
// site and workgroup.
constexpr int EMIT_NT = 256;
constexpr int EMIT_PIECES = 1024;  // piece slots per workgroup and step
constexpr int CELL_SLOTS = 256;
struct CellSums {
  int site[CELL_SLOTS];  // -1: free
  int np[CELL_SLOTS];
  long long chi[CELL_SLOTS];
  unsigned long long lo[4 * CELL_SLOTS];
  int hi[4 * CELL_SLOTS];  // a workgroup's sum stays below 2^84: 32 bits suffice
};

__device__ inline int cell_slot(CellSums& S, int site) {
  unsigned s = ((unsigned)site * 2654435761u) >> 24;
  for (int probe = 0; probe < 16; ++probe) {
    const int old = atomicCAS(&S.site[s], -1, site);
    if (old == -1 || old == site) return (int)s;
    s = (s + 1) & (CELL_SLOTS - 1);
  }
  return -1;
}

template <bool HASH>
__device__ __forceinline__ void emit_cells(const ShapeArgs& a) {
  static_assert(CELL_SLOTS == 256 && EMIT_NT == CELL_SLOTS, "one slot per thread; the hash takes the top 8 bits");
  __shared__ CellSums S;
  const int tid = threadIdx.x;
  const int np_all = (int)min(a.counters[C_PIECE_SLOTS], (unsigned long long)a.pcap);
  long long pairs = 0;  // nonempty pieces added less those taken back
  const int per = ((np_all + DIES - 1) / DIES + EMIT_PIECES - 1) / EMIT_PIECES * EMIT_PIECES;
  const int end = min(np_all, (int)(blockIdx.x % DIES + 1) * per);
  for (int base = (int)(blockIdx.x % DIES) * per + (int)(blockIdx.x / DIES) * EMIT_PIECES; base < end;
       base += (int)(gridDim.x / DIES) * EMIT_PIECES) {
    S.site[tid] = -1;
    S.np[tid] = 0;
    S.chi[tid] = 0;
    for (int d = 0; d < 4; ++d) {
      S.lo[4 * tid + d] = 0;
      S.hi[4 * tid + d] = 0;
    }
    __syncthreads();
    for (int q = 0; q < EMIT_PIECES / EMIT_NT; ++q) {
      const int p = base + q * EMIT_NT + tid;
      if (p >= end) break;
      const unsigned word = a.pref[p].word;
      if (!(word & 1u)) continue;
      const PieceOut o = a.pout[p];
      const PieceDesc d = a.pdesc[p];
      const ShapeDesc& sd = a.shapes[d.shape];
      const int i = a.psite[p], sign = sd.sign, glue = pw_glue(word);
      const int t = (int)(sd.tet_off + d.t);
      const double v[4] = {o.vol, o.mx, o.my, o.mz};
      const int s = cell_slot(S, i);
      if (s >= 0) {
        atomicAdd(&S.np[s], sign);
        atomicAdd((unsigned long long*)&S.chi[s], (unsigned long long)(sign * o.chi));
        for (int k = 0; k < 4; ++k) {
          const Fix128 g = signed128(fixed80(v[k]), sign);
          const unsigned long long old = atomicAdd(&S.lo[4 * s + k], g.lo);
          const long long h = g.hi + (old + g.lo < old ? 1 : 0);
          if (h) atomicAdd(&S.hi[4 * s + k], (int)h);
        }
      } else {
        atomicAdd(&a.cell_np[i], sign);
        atomicAdd((unsigned long long*)&a.cell_chi[i], (unsigned long long)(sign * o.chi));
        for (int k = 0; k < 4; ++k)
          acc128((unsigned long long*)&a.cell_geo[8 * (size_t)i + 2 * k], signed128(fixed80(v[k]), sign));
      }
      if (!HASH) a.pparent[p] = p;
      node_emit<HASH>(a, sign, node_key(1, i, t), glue);
      pairs += sign;
      keep_term(a, 1, t, i, -1, -1, -1, glue, o.chi);
      if (a.flags & RPD_KEEP_PIECES) {
        const unsigned long long idx = atomicAdd(&a.counters[C_PIECES], 1ull);
        if (idx < (unsigned long long)a.piece_cap) {
          PieceRec pr;
          pr.t = t;
          pr.i = i;
          pr.vol = (float)o.vol;
          pr.mx = (float)o.mx;
          pr.my = (float)o.my;
          pr.mz = (float)o.mz;
          pr.chi = o.chi;
          a.pieces[idx] = pr;
        } else {
          atomicOr(a.status, ST_TABLE_FULL);
        }
      }
    }
    __syncthreads();
    const int i = S.site[tid];
    if (i >= 0) {
      if (S.np[tid]) atomicAdd(&a.cell_np[i], S.np[tid]);
      if (S.chi[tid]) atomicAdd((unsigned long long*)&a.cell_chi[i], (unsigned long long)S.chi[tid]);
      for (int d = 0; d < 4; ++d)
        acc128((unsigned long long*)&a.cell_geo[8 * (size_t)i + 2 * d],
               Fix128{S.lo[4 * tid + d], (long long)S.hi[4 * tid + d]});
    }
    __syncthreads();
  }
  for (int off = 32; off > 0; off >>= 1) pairs += __shfl_xor(pairs, off);
  if ((tid & 63) || !pairs) return;
  stat_add(a, C_PAIRS, (unsigned long long)pairs);  // in two's complement
  if (!HASH) stat_add(a, C_NODES, (unsigned long long)pairs);
}

// one element record
template <bool HASH>
__device__ __forceinline__ void emit_record(const ShapeArgs& a, int r, unsigned long long& nodes,
                                            unsigned long long& rpvs) {
  const ElemRec R = a.recs[r];
  const int kind = R.z >> REC_SHIFT;
  if (kind == REC_NONE) return;
  const int low = R.z & ((1 << REC_SHIFT) - 1);
  const int i = a.psite[R.p];
  const PieceDesc d = a.pdesc[R.p];
  const ShapeDesc& sd = a.shapes[d.shape];
  const int sign = sd.sign;
  const int t = (int)(sd.tet_off + d.t);  // batch-global tet id (node keys, piece records)
  if (kind == REC_FACE) {
    const int fs = ht_insert(a.F, ((unsigned long long)i << 32) | (unsigned)R.j, a.status);
    if (fs >= 0) {
      atomicAdd((unsigned long long*)&a.face_chi[fs], (unsigned long long)(sign * R.num));
      atomicAdd(&a.face_np[fs], sign);
      node_emit<HASH>(a, sign, node_key(2, fs, t), low);
      if (!HASH) {
        a.recs[r].num = fs;
        a.rparent[r] = r;
      }
    }
    ++nodes;
    keep_term(a, 2, t, i, R.j, -1, -1, low, R.num);
    return;
  }
  const int es = ht_insert(a.E, ((unsigned long long)i << 42) | ((unsigned long long)R.j << 21) | (unsigned)R.k, a.status);
  if (kind == REC_EDGE) {
    if (es >= 0) {
      atomicAdd((unsigned long long*)&a.edge_chi[es], (unsigned long long)(sign * R.num));
      atomicAdd(&a.edge_np[es], sign);
      atomicAdd((unsigned long long*)&a.edge_len[es], (unsigned long long)(sign * fixed56(R.len)));
      node_emit<HASH>(a, sign, node_key(3, es, t), low);
      if (!HASH) {
        a.recs[r].num = es;
        a.rparent[r] = r;
      }
    }
    ++nodes;
    keep_term(a, 3, t, i, R.j, R.k, -1, low, R.num);
    return;
  }
  if (es >= 0) {
    const int qs = ht_insert(a.Q, ((unsigned long long)es << 21) | (unsigned)low, a.status);
    if (qs >= 0) atomicAdd(&a.rpv_cnt[qs], sign);
  }
  ++rpvs;
  keep_term(a, 4, t, i, R.j, R.k, low, 0, 1);
}

// The records of a pass: f(r) for every one, the chunks' ranges in blockIdx.y 1 and the pool in blockIdx.y 2 of a launch
// of EMIT_NT threads per workgroup.
template <typename F>
__device__ __forceinline__ void for_records(const ShapeArgs& a, F f) {
  const int tid = threadIdx.x;
  if (blockIdx.y == 1) {
    const int per = EMIT_NT / 64;
    for_items((int)a.counters[C_CHUNKS], 1, (int)(blockIdx.x / DIES) * per + (tid >> 6), (int)(gridDim.x / DIES) * per,
              [&](int c) {
                const int n = a.chunk_recs[c];
                for (int q = tid & 63; q < n; q += 64) f(c * REC_CHUNK + q);
              });
  } else {
    const int n = (int)min(a.counters[C_REC_POOL], (unsigned long long)a.pool_cap);
    const int r0 = chunk_cap(a.pcap) * REC_CHUNK;
    for (int q = blockIdx.x * EMIT_NT + tid; q < n; q += gridDim.x * EMIT_NT) f(r0 + q);
  }
}
// f(p) for every piece slot
template <typename F>
__device__ __forceinline__ void for_pieces(const ShapeArgs& a, F f) {
  for_items((int)min(a.counters[C_PIECE_SLOTS], (unsigned long long)a.pcap), EMIT_NT,
            (int)(blockIdx.x / DIES) * EMIT_NT + threadIdx.x, (int)(gridDim.x / DIES) * EMIT_NT, f);
}

// One launch for everything (blockIdx.y: cells, the chunks' records, the pool's records). Bound by the random accesses
// of the table inserts, all of which are in flight at once over a grid that fills the chip. HASH (sessions): every
// element piece goes into the table N as well.
template <bool HASH>
__global__ __launch_bounds__(EMIT_NT) void k_emit(ShapeArgs a) {
  if (*a.status) return;  // the call fails or is redone: slots may be unfilled, and tets without any
  if (blockIdx.y == 0) {
    emit_cells<HASH>(a);
    return;
  }
  unsigned long long nodes = 0, rpvs = 0;
  for_records(a, [&](int r) { emit_record<HASH>(a, r, nodes, rpvs); });
  for (int off = 32; off > 0; off >>= 1) {
    rpvs += __shfl_xor(rpvs, off);
    nodes += __shfl_xor(nodes, off);
  }
  if ((threadIdx.x & 63) == 0) {
    if (rpvs) stat_add(a, C_RPV, rpvs);
    if (!HASH && nodes) stat_add(a, C_NODES, nodes);
  }
}

// The counts are known on the device only: a grid of the workgroups that fit the chip, grid-stride.
static int pass_grid(const ShapeArgs& a) { return DIES * std::max(1, std::min(a.pcap / (4 * CHUNK), 2048) / DIES); }

hipError_t launch_emit(const ShapeArgs& a, hipStream_t s) {
  if (a.tet_slots) hipLaunchKernelGGL(k_emit<false>, dim3(pass_grid(a), 3), dim3(EMIT_NT), 0, s, a);
  else hipLaunchKernelGGL(k_emit<true>, dim3(pass_grid(a), 3), dim3(EMIT_NT), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// components of a build's elements (Sec. 4.1.1): union-find over the pieces and records themselves
// ---------------------------------------------------------------------------------------------------------------
__device__ inline int uf_find(int* parent, int x) {
  while (true) {
    const int p = parent[x];
    if (p == x) return x;
    const int gp = parent[p];
    if (gp != p) parent[x] = gp;
    x = p;
  }
}
// hook the larger root under the smaller with CAS; path halving
__device__ inline void uf_union(int* parent, int a, int b) {
  while (true) {
    a = uf_find(parent, a);
    b = uf_find(parent, b);
    if (a == b) return;
    if (a < b) {
      const int t = a;
      a = b;
      b = t;
    }
    if (atomicCAS(&parent[a], a, b) == a) return;
  }
}

// For the gluing bits g of an element piece of site i in tet t: f(q, m) for the nonempty piece q of the same site in
// every face-adjacent tet of higher number across a face in g, m its gluing bit for that face. A bit whose neighbour
// has no such piece breaks an invariant. (Each glued pair is met once, from its lower tet; that the other side agrees
// is checked there, and that no bit is left over by counting.)
template <typename F>
__device__ __forceinline__ void for_glued(const ShapeArgs& a, const PieceDesc& d, int i, int g, F f) {
  const ShapeDesc& sd = a.shapes[d.shape];
  const int4 nb = reinterpret_cast<const int4*>(sd.tn)[d.t];
  // the boundary never carries a bit; the other side matches lower ids
  g &= (nb.x > d.t ? 1 : 0) | (nb.y > d.t ? 2 : 0) | (nb.z > d.t ? 4 : 0) | (nb.w > d.t ? 8 : 0);
  for (; g; g &= g - 1) {
    const int face = __builtin_ctz(g);
    const int t2 = face == 0 ? nb.x : face == 1 ? nb.y : face == 2 ? nb.z : nb.w;
    const int4 nb2 = reinterpret_cast<const int4*>(sd.tn)[t2];
    const int2 run = a.tet_slots[sd.tet_off + t2];
    const int f2 = nb2.x == d.t ? 0 : nb2.y == d.t ? 1 : nb2.z == d.t ? 2 : 3;
    int q = -1;
    if (run.x < 0 || run.y < 0 || run.y > a.pcap - run.x) {  // not a run of piece slots
      atomicOr(a.status, ST_INTERNAL);
      continue;
    }
    for (int c = 0; c < run.y; ++c)
      if (a.psite[run.x + c] == i) {
        q = run.x + c;
        break;
      }
    const PieceRef ref = q >= 0 ? a.pref[q] : PieceRef{0, 0u};
    if (!(ref.word & 1u)) atomicOr(a.status, ST_INTERNAL);
    else f(q, ref, 1 << f2);
  }
}

// Every gluing bit matched and united. A tet's pieces sit in consecutive slots, in the spatial order of the tets, so
// a lookup reads a few neighbouring lines, where one in a hash table of all element pieces reads a random one.
__global__ __launch_bounds__(EMIT_NT) void k_glue_pieces(ShapeArgs a) {
  if (*a.status) return;
  unsigned long long bits = 0, pairs = 0;
  if (blockIdx.y == 0) {
    for_pieces(a, [&](int p) {
      const unsigned w = a.pref[p].word;
      const int g = (w & 1u) ? pw_glue(w) & 15 : 0;
      if (!g) return;
      bits += __popc(g);
      for_glued(a, a.pdesc[p], a.psite[p], g, [&](int q, const PieceRef& ref, int bit) {
        if (!(pw_glue(ref.word) & bit)) {
          atomicOr(a.status, ST_INTERNAL);
          return;
        }
        ++pairs;
        uf_union(a.pparent, p, q);
      });
    });
  } else {
    for_records(a, [&](int r) {
      const ElemRec R = a.recs[r];
      const int kind = R.z >> REC_SHIFT, g = R.z & 15;
      if ((kind != REC_FACE && kind != REC_EDGE) || !g) return;
      bits += __popc(g);
      for_glued(a, a.pdesc[R.p], a.psite[R.p], g, [&](int, const PieceRef& ref, int bit) {
        const int nf = pw_faces(ref.word);
        const int q0 = ref.rec + (kind == REC_FACE ? 0 : nf), n = kind == REC_FACE ? nf : pw_edges(ref.word);
        for (int q = q0; q < q0 + n; ++q) {
          if (a.recs[q].j != R.j || a.recs[q].k != R.k) continue;
          if (!(a.recs[q].z & bit)) break;
          ++pairs;
          uf_union(a.rparent, r, q);
          return;
        }
        atomicOr(a.status, ST_INTERNAL);
      });
    });
  }
  for (int off = 32; off > 0; off >>= 1) {
    bits += __shfl_xor(bits, off);
    pairs += __shfl_xor(pairs, off);
  }
  if ((threadIdx.x & 63) == 0) {
    if (bits) stat_add(a, C_GLUE_BITS, bits);
    if (pairs) stat_add(a, C_GLUE_PAIRS, pairs);
  }
}

// one root per component
__global__ __launch_bounds__(EMIT_NT) void k_count_piece_roots(ShapeArgs a, int* cell_b0, int* face_b0, int* edge_b0) {
  if (*a.status) return;
  if (blockIdx.y == 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && stat_sum(a, C_GLUE_BITS) != 2 * stat_sum(a, C_GLUE_PAIRS))
      atomicOr(a.status, ST_INTERNAL);  // a gluing bit without its counterpart
    for_pieces(a, [&](int p) {
      if ((a.pref[p].word & 1u) && a.pparent[p] == p) atomicAdd(&cell_b0[a.psite[p]], 1);
    });
    return;
  }
  for_records(a, [&](int r) {
    const int kind = a.recs[r].z >> REC_SHIFT;
    if ((kind == REC_FACE || kind == REC_EDGE) && a.rparent[r] == r)
      atomicAdd(&(kind == REC_FACE ? face_b0 : edge_b0)[(int)a.recs[r].num], 1);
  });
}

hipError_t launch_glue_pieces(const ShapeArgs& a, int* cell_b0, int* face_b0, int* edge_b0, hipStream_t s) {
  hipLaunchKernelGGL(k_glue_pieces, dim3(pass_grid(a), 3), dim3(EMIT_NT), 0, s, a);
  hipLaunchKernelGGL(k_count_piece_roots, dim3(pass_grid(a), 3), dim3(EMIT_NT), 0, s, a, cell_b0, face_b0, edge_b0);
  return hipGetLastError();
}

}  // namespace rpd
