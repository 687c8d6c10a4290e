// Tet-Cell clipping (paper Sec. 5.2) with on-the-fly fractional Euler characteristic (Sec. 4.1.2) and the gluing
// information for connected components (Sec. 4.1.1), in two kernels.
//
// Candidate kernel: one wavefront owns up to TB spatially consecutive tets. It selects the sites that can own any
// point of the group's bounding box, then per tet the candidate sites that can own a point of the tet, sorted by power
// distance at the tet centroid, and hands every tet a run of piece slots, one per candidate.
//
// Piece kernel: 64 consecutive piece slots per wavefront, one lane per piece: the tet is clipped by the bisectors of
// all other candidates with the polytope in LDS, and the piece's cell terms and element records (faces, edges, RPVs:
// chi numerators, gluing bits, lengths) are written out. No hash table and no shared accumulator is touched here: the
// emission kernel turns the records into sums.
//
// Tets with too many candidates and pieces whose predicates stay undecided in FP64 go to the large-capacity kernel,
// which computes them with FP64 constructions and exact predicates.
#include <hip/hip_runtime.h>

#include <climits>

#include <algorithm>
#include <type_traits>

#include "rpd_device.h"
#include "rpd_launch.h"

namespace rpd {

// ---------------------------------------------------------------------------------------------------------------
// the terms of one nonempty piece
// ---------------------------------------------------------------------------------------------------------------
template <typename Topo>
__device__ inline int pos_of(typename Topo::W w, int p) {
  if (Topo::plane(w, 0) == p) return 0;
  if (Topo::plane(w, 1) == p) return 1;
  if (Topo::plane(w, 2) == p) return 2;
  return -1;
}

template <typename Topo>
__device__ inline long long wv_of(typename Topo::W w, const unsigned* nu, long long L) {
  return w_vertex(Topo::plane(w, 0), Topo::plane(w, 1), Topo::plane(w, 2), nu, L);
}

// What the first pass over a piece's vertices leaves for emit_out.
template <typename CL>
struct EmitAcc {
  typedef typename CL::Real T;
  typedef typename CL::MaskT Mask;
  MaskCounts w;             // vertices less edges (emit_out: plus faces) by their face mask
  T gx, gy, gz;             // vertex sums
  int nv;
  unsigned planes;          // planes present (Topo32: at most 32 of them)
  unsigned fplanes;         // those of element faces
  int nface, nedge, nrpv;   // element records of the piece (elements whose smallest site is the piece's)
  Mask edge[3], rpv;        // vertices k with such an edge at position f (k below its other end), or such an RPV
  __device__ int records() const { return nface + nedge + nrpv; }
};

// vertex pass: vertex and edge weights, the first vertex of every face (kept in the clipper's table), the records
template <typename CL>
__device__ __forceinline__ void emit_scan(CL& c, EmitAcc<CL>& e) {
  typedef typename CL::TopoT Topo;
  typedef typename Topo::W W;
  const int i = c.env.site_i;  // batch-global site id
  e.w.lo = e.w.hi = 0;
  e.gx = e.gy = e.gz = 0;
  e.nv = e.nface = e.nedge = e.nrpv = 0;
  e.planes = e.fplanes = 0;
  e.edge[0] = e.edge[1] = e.edge[2] = e.rpv = 0;
  for (auto m = c.live; m; m &= m - 1) {
    const int k = ctz_mask(m);
    const W w = c.st.topo(k);
    const auto v = c.st.get(k);
    e.gx += v.x;
    e.gy += v.y;
    e.gz += v.z;
    ++e.nv;
    const int p0 = Topo::plane(w, 0), p1 = Topo::plane(w, 1), p2 = Topo::plane(w, 2);
    e.w.add(face_bit(p0) | face_bit(p1) | face_bit(p2), 1);
    bool above[3];  // the plane is a bisector against a higher site
    for (int f = 0; f < 3; ++f) {
      const int p = Topo::plane(w, f);
      above[f] = p >= 4 && c.env.cand_id(p - 4) > i;
      if (c.tab.get(p) == 0) {
        c.tab.set(p, k + 1);
        if (CL::FEW_PLANES) e.planes |= 1u << (p & 31);
        if (above[f]) {
          ++e.nface;
          if (CL::FEW_PLANES) e.fplanes |= 1u << (p & 31);
        }
      }
    }
    for (int f = 0; f < 3; ++f) {
      if (k < Topo::nb(w, f)) {
        const int f1 = f == 2 ? 0 : f + 1, f2 = f == 0 ? 2 : f - 1;
        e.w.add(face_bit(Topo::plane(w, f1)) | face_bit(Topo::plane(w, f2)), -1);
        if (above[f1] && above[f2]) {
          ++e.nedge;
          e.edge[f] |= CL::bit(k);
        }
      }
    }
    if (above[0] && above[1] && above[2]) {
      ++e.nrpv;
      e.rpv |= CL::bit(k);
    }
  }
}

// The piece's cell terms and its element records, written to slot p_slot and to records [base, base + e.records()).
// Every loop takes one item of the lane's own list per trip (an edge, an RPV, a face vertex), so that lanes whose
// pieces have different shapes stay together; a loop over plane numbers and one over the face's edges inside it kept
// one lane in five busy.
template <typename CL>
__device__ __forceinline__ void emit_out(CL& c, const ShapeDesc& sd, int tl, EmitAcc<CL>& e, int p_slot, int base,
                                         const ShapeArgs& a) {
  typedef typename CL::Real T;
  typedef typename CL::TopoT Topo;
  typedef typename Topo::W W;
  const int i = c.env.site_i;
  const unsigned* nu = sd.nu + 14 * (size_t)tl;
  const long long L = sd.L;
  const int4 tn4 = reinterpret_cast<const int4*>(sd.tn)[tl];  // face neighbours (-1: boundary), one load
  const unsigned interior = (tn4.x >= 0 ? 1u : 0u) | (tn4.y >= 0 ? 2u : 0u) | (tn4.z >= 0 ? 4u : 0u) |
                            (tn4.w >= 0 ? 8u : 0u);  // bit f: face f is shared with another tet
  auto put = [&](int r, int j, int k, int z, long long num, double len) {
    ElemRec R;
    R.j = j;
    R.k = k;
    R.z = z;
    R.p = p_slot;
    R.num = num;
    R.len = len;
    a.recs[r] = R;
  };
  auto inner = [&](int p) { return p < 4 ? (int)(interior & (1u << p)) : 0; };  // the gluing bit of an interior face
  int re = base + e.nface;
  while (e.edge[0] | e.edge[1] | e.edge[2]) {  // RPE pieces
    const int k = ctz_mask(e.edge[0] | e.edge[1] | e.edge[2]);
    const auto b = CL::bit(k);
    const int f = (e.edge[0] & b) ? 0 : (e.edge[1] & b) ? 1 : 2;
    if (f == 0) e.edge[0] &= ~b;
    else if (f == 1) e.edge[1] &= ~b;
    else e.edge[2] &= ~b;
    const W wk = c.st.topo(k);
    const int n = Topo::nb(wk, f);
    const W wn = c.st.topo(n);
    const auto C = c.st.get(k), N = c.st.get(n);
    const int pa = Topo::plane(wk, f == 2 ? 0 : f + 1), pb = Topo::plane(wk, f == 0 ? 2 : f - 1);
    const int ea = pos_of<Topo>(wn, pa), eb = pos_of<Topo>(wn, pb);
    if (ea < 0 || eb < 0) atomicOr(a.status, ST_INTERNAL);
    const int sa = c.env.cand_id(pa - 4), sb = c.env.cand_id(pb - 4);
    const T lx = N.x - C.x, ly = N.y - C.y, lz = N.z - C.z;
    const long long ev = wv_of<Topo>(wk, nu, L) + wv_of<Topo>(wn, nu, L) - L;
    // the third planes at the two ends
    const int g = inner(Topo::plane(wk, f)) | inner(Topo::plane(wn, (3 - ea - eb) & 3));
    put(re++, min(sa, sb), max(sa, sb), (REC_EDGE << REC_SHIFT) | g, ev, (double)sqrt(lx * lx + ly * ly + lz * lz));
  }
  int rq = base + e.nface + e.nedge;
  for (auto m = e.rpv; m; m &= m - 1) {  // an RPV is recorded once, from its smallest site
    const W w = c.st.topo(ctz_mask(m));
    const int s0 = c.env.cand_id(Topo::plane(w, 0) - 4), s1 = c.env.cand_id(Topo::plane(w, 1) - 4),
              s2 = c.env.cand_id(Topo::plane(w, 2) - 4);
    const int lo = min(s0, min(s1, s2)), hi = max(s0, max(s1, s2)), mid = s0 + s1 + s2 - lo - hi;
    put(rq++, lo, mid, (REC_RPV << REC_SHIFT) | hi, 1, 0.0);
  }
  const T inv_nv = T(1) / T(e.nv);
  const T ax = e.gx * inv_nv, ay = e.gy * inv_nv, az = e.gz * inv_nv;

  // ---- the cycles of the element faces (their terms), one vertex per trip. Apart from the fans: one walk for both ran
  // every face's trips, and a trip at both ends of each, through the code of both, and was half of the piece kernel
  // (128^3 genus-3 solid: 1.44 -> 1.27 ms apart; 64^3 torus, bound by the longest chunks: 258 -> 253 us)
  int rf = base;
  {
    unsigned todo = e.fplanes;
    auto next_face = [&](int p) {  // the next plane with an element face, or -1
      if (CL::FEW_PLANES) {
        if (!todo) return -1;
        const int q = ctz_mask(todo);
        todo &= todo - 1;
        return q;
      }
      for (p = max(p + 1, 4); p < c.np; ++p)
        if (c.tab.get(p) && c.env.plane_site(p) > i) return p;
      return -1;
    };
    int p = next_face(-1);
    bool start = true;
    int r = 0, nxt = 0, acur = 0, steps = 0, fglue = 0;
    long long fchi = 0, fe = 0, fv = 0;  // fe, fv: read in one trip, added in the next (not waited for)
    while (p >= 0) {
      if (start) r = nxt = c.tab.get(p) - 1;
      const W wn = c.st.topo(nxt);
      const int epn = pos_of<Topo>(wn, p);
      const int ea = start ? 0 : pos_of<Topo>(wn, acur);
      fchi += fv - fe;
      fe = fv = 0;
      if (ea < 0 || epn < 0 || steps > CL::SLOTS) {  // a broken polytope: the call fails
        atomicOr(a.status, ST_INTERNAL);
        start = true;
        steps = 0;
        if (rf < base + e.nface) put(rf++, 0, 0, REC_NONE << REC_SHIFT, 0, 0.0);
        p = next_face(p);
        continue;
      }
      if (start) {
        fchi = L;
        fglue = 0;
        steps = 0;
        fv = wv_of<Topo>(wn, nu, L);
        acur = Topo::plane(wn, epn == 2 ? 0 : epn + 1);
        nxt = Topo::nb(wn, epn == 0 ? 2 : epn - 1);
        start = false;
        continue;
      }
      fe = w_edge(p, acur, nu, L);  // the edge to nxt lies on planes {p, acur}
      fglue |= inner(acur);
      if (nxt == r) {
        if (rf < base + e.nface) put(rf++, c.env.plane_site(p), -1, (REC_FACE << REC_SHIFT) | fglue, fchi - fe, 0.0);
        fe = 0;
        start = true;
        p = next_face(p);
      } else {
        fv = wv_of<Topo>(wn, nu, L);
        ++steps;
        nxt = Topo::nb(wn, ea);  // leave the vertex along {p, its third plane}: the neighbour opposite acur
        acur = Topo::plane(wn, (3 - ea - epn) & 3);
      }
    }
  }
  // ---- every face's fan, by ascending plane: one triangle (R, C, N) per trip
  int cell_glue = 0;
  T vol = 0, mx = 0, my = 0, mz = 0;
  {
    auto next_face = [&](int p) {  // the next plane with a face, or -1
      if (CL::FEW_PLANES) {
        if (!e.planes) return -1;
        const int q = ctz_mask(e.planes);
        e.planes &= e.planes - 1;
        return q;
      }
      for (++p; p < c.np; ++p)
        if (c.tab.get(p)) return p;
      return -1;
    };
    int p = next_face(-1);
    bool start = true;
    int r = 0, nxt = 0, acur = 0, steps = 0;
    T Rx = 0, Ry = 0, Rz = 0, Cx = 0, Cy = 0, Cz = 0;
    while (p >= 0) {
      if (start) {  // R, its neighbour C and what follows it
        r = c.tab.get(p) - 1;
        c.tab.set(p, 0);
        const W wr = c.st.topo(r);
        const int epr = pos_of<Topo>(wr, p) & 3;
        const int n1 = Topo::nb(wr, epr == 0 ? 2 : epr - 1);
        acur = Topo::plane(wr, epr == 2 ? 0 : epr + 1);
        const auto R = c.st.get(r), C = c.st.get(n1);
        const W wc = c.st.topo(n1);
        Rx = R.x;
        Ry = R.y;
        Rz = R.z;
        Cx = C.x;
        Cy = C.y;
        Cz = C.z;
        e.w.add(face_bit(p), 1);
        if (p < 4) cell_glue |= inner(p) ? 1 << p : 16 << p;  // glue across an interior face; boundary contact
        const int ep = pos_of<Topo>(wc, p), ea = pos_of<Topo>(wc, acur);
        if (ep < 0 || ea < 0) {  // a broken polytope: the call fails
          atomicOr(a.status, ST_INTERNAL);
          p = next_face(p);
          continue;
        }
        nxt = Topo::nb(wc, ea);
        acur = Topo::plane(wc, (3 - ea - ep) & 3);
        steps = 0;
        start = nxt == r;
      }
      if (!start) {
        const W wn = c.st.topo(nxt);
        const auto N = c.st.get(nxt);
        const int ep = pos_of<Topo>(wn, p), ea = pos_of<Topo>(wn, acur);
        {  // with the apex: a tet of the piece
          T ux = Cx - Rx, uy = Cy - Ry, uz = Cz - Rz;
          T vx = N.x - Rx, vy = N.y - Ry, vz = N.z - Rz;
          T wx = ax - Rx, wy = ay - Ry, wz = az - Rz;
          T det = ux * (vy * wz - vz * wy) - uy * (vx * wz - vz * wx) + uz * (vx * wy - vy * wx);
          T tv = fabs(det) * T(1.0 / 6.0);
          vol += tv;
          mx += tv * (Rx + Cx + N.x + ax);
          my += tv * (Ry + Cy + N.y + ay);
          mz += tv * (Rz + Cz + N.z + az);
        }
        Cx = N.x;
        Cy = N.y;
        Cz = N.z;
        if (ep < 0 || ea < 0 || ++steps > CL::SLOTS) {
          atomicOr(a.status, ST_INTERNAL);
          start = true;
        } else {
          nxt = Topo::nb(wn, ea);
          acur = Topo::plane(wn, (3 - ea - ep) & 3);
          start = nxt == r;
        }
      }
      if (start) p = next_face(p);
    }
  }
  // records counted but not written (a broken polytope): nothing may read stale ones
  for (; rf < base + e.nface; ++rf) put(rf, 0, 0, REC_NONE << REC_SHIFT, 0, 0.0);
  // moments were accumulated with 4x the centroid sum; shift to absolute coordinates
  const float4 o = c.env.o;
  PieceOut out;
  out.vol = (double)vol;
  out.mx = (double)mx * 0.25 + out.vol * o.x;
  out.my = (double)my * 0.25 + out.vol * o.y;
  out.mz = (double)mz * 0.25 + out.vol * o.z;
  out.chi = e.w.sum(nu, L) - L;
  a.pout[p_slot] = out;
  PieceRef ref;
  ref.rec = base;
  ref.word = piece_word(e.nface, e.nedge, e.nrpv, cell_glue);
  a.pref[p_slot] = ref;
}

// Room for n records in the pool, from the calling lane: the first, or -1 when the pool is full.
__device__ inline int pool_records(const ShapeArgs& a, int n) {
  if (n == 0) return 0;
  const unsigned long long q = atomicAdd(&a.counters[C_REC_POOL], (unsigned long long)n);
  if (q + n > (unsigned long long)a.pool_cap) {
    atomicOr(a.status, ST_POOL_FULL);
    return -1;
  }
  return chunk_cap(a.pcap) * REC_CHUNK + (int)q;
}

// A piece clipped outside its chunk's pass: terms to its slot, records to the pool.
template <typename CL>
__device__ __forceinline__ void emit_alone(CL& c, const ShapeDesc& sd, int tl, int p_slot, const ShapeArgs& a) {
  EmitAcc<CL> e;
  emit_scan(c, e);
  const int base = pool_records(a, e.records());
  if (base >= 0) emit_out(c, sd, tl, e, p_slot, base, a);
}

// Hands piece slot p (or, with p = -1, every candidate of the tet) to the large-capacity kernel. first: the tet's
// first piece slot, or -1 when its candidates are still to be found.
__device__ inline void defer_item(const ShapeArgs& a, int shape, int t, int p, int first) {
  const unsigned long long idx = atomicAdd(&a.counters[C_DEFER_ITEMS], 1ull);
  if (idx < (unsigned long long)a.deferred_cap) a.deferred[idx] = make_int4(shape, t, p, first);
  else atomicOr(a.status, ST_PASS_FULL);
}

// ---------------------------------------------------------------------------------------------------------------
// clipping of one (tet, candidate) piece against the other candidates in order; returns CLIP_* for the piece
// ---------------------------------------------------------------------------------------------------------------
template <typename CL>
__device__ __forceinline__ int clip_piece(CL& cl, int m) {
  typedef typename CL::Real T;
  const TetEnv& env = cl.env;
  const float4 o = env.o;
  const double y1x = (double)env.tv[1].x - o.x, y1y = (double)env.tv[1].y - o.y, y1z = (double)env.tv[1].z - o.z;
  const double y2x = (double)env.tv[2].x - o.x, y2y = (double)env.tv[2].y - o.y, y2z = (double)env.tv[2].z - o.z;
  const double y3x = (double)env.tv[3].x - o.x, y3y = (double)env.tv[3].y - o.y, y3z = (double)env.tv[3].z - o.z;
  // CUT: the bisector against candidate c cuts the tet; SKIP: the tet lies in its kept half-space; else it lies outside
  enum { SKIP, CUT, OUTSIDE };
  auto classify = [&](int c, Plane<double>& P) {
    const float4 sj = env.cand_site(c);
    P = bisector64(env.si, sj, o);
    if (P.nx == 0.0 && P.ny == 0.0 && P.nz == 0.0) {  // concentric spheres: the larger one owns everything
      if (P.d > 0) return SKIP;
      // equal spheres: under the weight perturbation eps_i - eps_j the lower site id owns everything
      return P.d == 0 && env.site_i < env.cand_id(c) ? SKIP : OUTSIDE;
    }
    // the bisector's values at the tet vertices are exact in FP64
    const double h0 = P.d;
    const double h1 = fma(P.nx, y1x, fma(P.ny, y1y, fma(P.nz, y1z, P.d)));
    const double h2 = fma(P.nx, y2x, fma(P.ny, y2y, fma(P.nz, y2z, P.d)));
    const double h3 = fma(P.nx, y3x, fma(P.ny, y3y, fma(P.nz, y3z, P.d)));
    if (h0 > 0 && h1 > 0 && h2 > 0 && h3 > 0) return SKIP;
    if (h0 < 0 && h1 < 0 && h2 < 0 && h3 < 0) return OUTSIDE;
    return CUT;
  };
  cl.init_tet();
  Plane<double> P;
  if (CL::FEW_PLANES) {  // at most 28 candidates: find the cutting ones first, then every lane clips by its next one
    unsigned cut = 0;
    for (int c = 0; c < m; ++c) {
      if (c == env.ci) continue;
      const int k = classify(c, P);
      if (k == OUTSIDE) return CLIP_EMPTY;
      if (k == CUT) cut |= 1u << c;
    }
    for (; cut; cut &= cut - 1) {
      const int c = ctz_mask(cut);
      const int r = cl.clip(4 + c, round_plane<T>(bisector64(env.si, env.cand_site(c), o)));
      if (r != CLIP_OK) return r;
    }
    return CLIP_OK;
  }
  for (int c = 0; c < m; ++c) {
    if (c == env.ci) continue;
    const int k = classify(c, P);
    if (k == OUTSIDE) return CLIP_EMPTY;
    if (k == SKIP) continue;
    const int r = cl.clip(4 + c, round_plane<T>(P));
    if (r != CLIP_OK) return r;
  }
  return CLIP_OK;
}

// ---------------------------------------------------------------------------------------------------------------
// candidate kernel
// ---------------------------------------------------------------------------------------------------------------
__device__ inline double wave_min(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
  return v;
}
__device__ inline float wave_minf(float v) {
  for (int off = 32; off > 0; off >>= 1) v = fminf(v, __shfl_xor(v, off));
  return v;
}
__device__ inline float wave_maxf(float v) {
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// Per group of neighbouring blocks (a block, or an octree cell of two or four times a block's side), the shape's sites
// that its blocks have to look at: a few hundred instead of all of the shape's (up to 20,000 on the 128^3 genus-3
// solid, where the scans of all sites were most of the candidate kernel). Site j is listed when
//   min over the box of d_j  <=  min over sites s of (max over the box of d_s)  +  the squared diagonal of a block.
// Every test that a block's candidate search makes compares g = d - |x - o|^2 (o and x in the block's box) of a site
// against a bound at most min_s max d_s, and |x - o| is at most the block's diagonal: a site left out here fails them
// all, so the search finds what it would among all sites.
__global__ __launch_bounds__(256) void k_group_sites(ShapeArgs a) {
  if (*a.status & ST_INVALID) return;
  __shared__ double s_red[4];
  __shared__ int s_list[GROUP_CAP];
  __shared__ int s_n, s_at;
  int lo = 0, hi = a.nshapes - 1;  // the shape of this group
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.shapes[mid].grp_off <= (int)blockIdx.x) lo = mid;
    else hi = mid - 1;
  }
  const ShapeDesc& sd = a.shapes[lo];
  const int g = blockIdx.x, lane = threadIdx.x & 63;
  const float* bx = sd.grpbox + 7 * (size_t)(g - sd.grp_off);
  const float x0 = bx[0], y0 = bx[1], z0 = bx[2], x1 = bx[3], y1 = bx[4], z1 = bx[5];
  const float4* ssite = a.site + sd.site_off;
  if (threadIdx.x == 0) s_n = 0;
  double u = INFINITY;
  for (int j = threadIdx.x; j < sd.ns; j += 256) {
    const float4 s = ssite[j];
    const double dx = fmax((double)s.x - x0, (double)x1 - s.x), dy = fmax((double)s.y - y0, (double)y1 - s.y),
                 dz = fmax((double)s.z - z0, (double)z1 - s.z);
    u = fmin(u, dx * dx + dy * dy + dz * dz - (double)s.w * s.w);
  }
  u = wave_min(u);
  if (lane == 0) s_red[threadIdx.x >> 6] = u;
  __syncthreads();
  u = fmin(fmin(s_red[0], s_red[1]), fmin(s_red[2], s_red[3])) + (double)bx[6];
  for (int base = 0; base < sd.ns; base += 256) {
    const int j = base + threadIdx.x;
    bool take = false;
    if (j < sd.ns) {
      const float4 s = ssite[j];
      const double dx = fmax(0.0, fmax((double)x0 - s.x, (double)s.x - x1)),
                   dy = fmax(0.0, fmax((double)y0 - s.y, (double)s.y - y1)),
                   dz = fmax(0.0, fmax((double)z0 - s.z, (double)s.z - z1));
      take = dx * dx + dy * dy + dz * dz - (double)s.w * s.w <= u;
    }
    const unsigned long long m = __ballot(take);
    if (!m) continue;
    int at = 0;
    if (lane == 0) at = atomicAdd(&s_n, __popcll(m));
    at = __shfl(at, 0) + __popcll(m & ((1ull << lane) - 1ull));
    if (take && at < GROUP_CAP) s_list[at] = j;
  }
  __syncthreads();
  if (threadIdx.x == 0) {  // a list that does not fit: the blocks look at all sites
    s_at = -1;
    if (s_n <= GROUP_CAP) {
      const unsigned long long q = atomicAdd(&a.counters[C_GROUP_SITES], (unsigned long long)s_n);
      if (q + s_n <= (unsigned long long)a.grp_cap) s_at = (int)q;
    }
    a.grp_run[g] = make_int2(s_at, s_n);
  }
  __syncthreads();
  if (s_at < 0) return;
  for (int q = threadIdx.x; q < s_n; q += 256) {
    a.grp_site[s_at + q] = ssite[s_list[q]];
    a.grp_id[s_at + q] = s_list[q];
  }
}

// g_j at the four tet vertices (tet-local frame, exact in FP64)
__device__ __forceinline__ void g4(const float4* tv, const float4& s, double* g) {
  const float4 o = tv[0];
  double ax = (double)s.x - o.x, ay = (double)s.y - o.y, az = (double)s.z - o.z;
  double D = ax * ax + ay * ay + az * az - (double)s.w * s.w;
  g[0] = D;
  for (int v = 1; v < 4; ++v)
    g[v] = D - 2.0 * (((double)tv[v].x - o.x) * ax + ((double)tv[v].y - o.y) * ay + ((double)tv[v].z - o.z) * az);
}

// A candidate that another one beats at all four tet vertices owns nothing on the tet, and its bisector constrains no
// piece (g is affine, so it is beaten everywhere on the tet; the values are exact in FP64).
//
// The budget decides by what these rounds leave where a tet with a longer list goes: the list is sorted by the power
// distance at the centroid, and three candidates at a time in list order drop those after them that one of them beats,
// while candidates remain past them. beaten: bit c where any other candidate beats the list's c-th (moved along with
// it). Returns the new count; order is kept.
__device__ __forceinline__ int refine_candidates(const float4* tv, const float4* sites, unsigned char* cand, int m,
                                                 unsigned long long& beaten) {
  for (int d = 0; d + 3 < m; d += 3) {
    double g0[4], g1[4], g2[4];
    g4(tv, sites[cand[d]], g0);
    g4(tv, sites[cand[d + 1]], g1);
    g4(tv, sites[cand[d + 2]], g2);
    int w = d + 3;
    unsigned long long b = beaten & ((1ull << w) - 1ull);
    for (int c = d + 3; c < m; ++c) {
      double g[4];
      g4(tv, sites[cand[c]], g);
      const bool dom = (g[0] > g0[0] && g[1] > g0[1] && g[2] > g0[2] && g[3] > g0[3]) ||
                       (g[0] > g1[0] && g[1] > g1[1] && g[2] > g1[2] && g[3] > g1[3]) ||
                       (g[0] > g2[0] && g[1] > g2[1] && g[2] > g2[2] && g[3] > g2[3]);
      if (!dom) {
        b |= ((beaten >> c) & 1ull) << w;
        cand[w++] = cand[c];
      }
    }
    m = w;
    beaten = b;
  }
  return m;
}

// A list within the budget is cut down to the candidates that no other one beats. Whatever was dropped before was beaten
// by one of these, so the tet's list is the same however the search came to it: an incremental update takes pieces back
// with the list that they were added with, though the sites around have changed.
__device__ __forceinline__ int drop_beaten(unsigned char* cand, int m, unsigned long long beaten) {
  if (!beaten) return m;
  int w = 0;
  for (int c = 0; c < m; ++c)
    if (!((beaten >> c) & 1ull)) cand[w++] = cand[c];
  return w;
}

// Which tets the candidate kernel takes next. It starts with ITEM_TETS of the item's, sharing the sites of their block's
// box; where those overflow the shared list, with chunks of SUB tets and the sites of their boxes, and where a chunk's
// overflow it, with DIRECT tets at a time that look among the source sites themselves.
struct TetRun {
  int sub, n;      // tets [sub, sub + n) of the item
  int direct_end;  // tets up to here are taken DIRECT at a time
  int all;
  bool split;
  static constexpr int DIRECT = 4;
  __device__ bool direct() const { return direct_end > sub; }
  __device__ void chunks() {
    split = true;
    n = min(SUB, all - sub);
  }
  __device__ void directly() {
    direct_end = sub + n;
    n = min(DIRECT, n);
  }
  __device__ bool next() {
    sub += n;
    if (!split) {
      n = min(ITEM_TETS, all - sub);
      return sub < all;
    }
    if (direct_end > sub) {
      n = min(DIRECT, direct_end - sub);
      return true;
    }
    direct_end = 0;
    n = min(SUB, all - sub);
    return sub < all;
  }
};

// One wavefront per work item (a part of a block, or all of it). A tet goes to the large-capacity kernel only for
// reasons that depend on its own candidates (more than fit its list, or the clip budget), never on its neighbours' or
// on sites that own nothing in it: an incremental update, which recomputes a tet's pieces to take them back, must take
// the path that added them.
__global__ __launch_bounds__(64, 3) void k_candidates(ShapeArgs a) {
  static_assert(SLMAX <= 256 && TetRun::DIRECT * KRAW <= SLMAX, "candidate bytes index the site list");
  constexpr int IT = ITEM_TETS;
  __shared__ float4 s_site[SLMAX];
  __shared__ int s_sid[SLMAX];
  __shared__ unsigned char s_raw[IT][KRAW];   // candidates (list positions) as found
  __shared__ unsigned char s_cand[IT][KRAW];  // ... and sorted
  __shared__ float s_key[IT][KRAW];           // sort keys
  __shared__ int s_m[IT];                     // candidates of each tet
  __shared__ unsigned long long s_beaten[IT]; // those of them (bits of sorted positions) that another one beats
  __shared__ short s_off[IT + 1];
  __shared__ short s_order[IT];
  __shared__ int s_nsl;

  const int tid = threadIdx.x, lane = tid;
  // (a shape of NaNs has no site that reaches anything: its lists would be empty)
  const bool invalid = (*a.status & ST_INVALID) != 0;
  const int nlisted = a.nitems_dev ? *a.nitems_dev : a.nitems;
  const int nitems = invalid ? 0 : nlisted;
  unsigned long long n_cand = 0;
  // A build's grid covers the items (every block of every shape, in a.parts parts), one item per workgroup. The passes
  // of an incremental round read a list of items whose length is known on the device only and launch a grid sized to
  // the resident workgroups, each taking items in grid-stride order.
  for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
  int shape, blk, tb0, ntb_all;
  unsigned long long item_mask = ~0ull;  // the tets of the item to clip, relative to its first tet
  if (a.items) {
    const int2 wi = a.items[item];
    shape = __builtin_amdgcn_readfirstlane(wi.x & 0xffff);
    const unsigned tet_mask16 = (unsigned)wi.x >> 16;  // the tets a new sphere can reach, or 0: all
    if (tet_mask16) item_mask = (unsigned long long)tet_mask16;
    blk = wi.y & ((1 << ITEM_PART_SHIFT) - 1);
    const int part = wi.y >> ITEM_PART_SHIFT;  // (only parts that exist are listed)
    const int* bk = a.shapes[shape].blk;
    tb0 = bk[blk] + (part - 1) * SPLIT_TETS;
    ntb_all = min(SPLIT_TETS, bk[blk + 1] - tb0);
  } else {
    const int it = a.item_mul == 1 ? item : (int)((unsigned long long)item * a.item_mul % (unsigned)nitems);
    int lo = 0, hi = a.nshapes - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.shapes[mid].item_off <= it) lo = mid;
      else hi = mid - 1;
    }
    shape = lo;
    const int local = it - a.shapes[shape].item_off, parts = a.shapes[shape].parts, pt = TB / parts;
    blk = local / parts;
    const int* bk = a.shapes[shape].blk;
    tb0 = bk[blk] + (local % parts) * pt;
    ntb_all = min(pt, bk[blk + 1] - tb0);
    if (ntb_all <= 0) continue;
  }
  const ShapeDesc sd = a.shapes[shape];
  // the sites to look among: the block's group's, or all
  const float4* src = a.site + sd.site_off;
  const int* src_id = nullptr;
  int nsrc = sd.ns;
  if (a.grp_run) {
    const int2 r = a.grp_run[sd.grp_off + (sd.grp ? sd.grp[blk] : blk)];
    if (r.x >= 0) {
      src = a.grp_site + r.x;
      src_id = a.grp_id + r.x;
      nsrc = r.y;
    }
  }
  auto source = [&](int q, int& id) {
    id = sd.site_off + (src_id ? src_id[q] : q);
    return src[q];
  };
  const bool all_slow = (a.flags & RPD_FORCE_SLOW_PATH) != 0;
  TetRun run{0, min(IT, ntb_all), 0, ntb_all, false};
  do {
  const int t0 = tb0 + run.sub;
  const int ntb = run.n;
  const unsigned long long cmask = item_mask >> run.sub;  // bit lt: tet t0 + lt is clipped
  if (run.split && !(cmask & ((1ull << ntb) - 1ull))) continue;  // a chunk without such tets
  __syncthreads();  // the shared arrays of the chunk before are free
  if (tid < IT) {
    s_m[tid] = 0;
    s_beaten[tid] = 0;
  }
  if (tid == 0) s_nsl = 0;
  __syncthreads();
  bool tight = false;
  if (!run.direct()) {
    // ---- 1. the sites that can own a point of a box around the tets: min over the box of g_j <= min over j of max over
    //         the box (g_j(x) = d_j(x) - |x - o|^2 with o the box's low corner is affine; values exact in FP64). The box
    //         is the block's, or the chunk's own.
    float lo[3], hi[3];
    if (!run.split) {
      const float* bx = sd.blkbox + 7 * (size_t)blk;
      for (int k = 0; k < 3; ++k) {
        lo[k] = bx[k];
        hi[k] = bx[3 + k];
      }
    } else {
      for (int k = 0; k < 3; ++k) {
        lo[k] = INFINITY;
        hi[k] = -INFINITY;
      }
      if (tid < ntb && ((cmask >> tid) & 1ull)) {
        const float4* tp = sd.tp + 4 * (size_t)(t0 + tid);
        for (int v = 0; v < 4; ++v) {
          const float4 p = tp[v];
          lo[0] = fminf(lo[0], p.x);
          lo[1] = fminf(lo[1], p.y);
          lo[2] = fminf(lo[2], p.z);
          hi[0] = fmaxf(hi[0], p.x);
          hi[1] = fmaxf(hi[1], p.y);
          hi[2] = fmaxf(hi[2], p.z);
        }
      }
      for (int k = 0; k < 3; ++k) {
        lo[k] = wave_minf(lo[k]);
        hi[k] = wave_maxf(hi[k]);
      }
    }
    const double bx = lo[0], by = lo[1], bz = lo[2];
    const double ex = (double)hi[0] - bx, ey = (double)hi[1] - by, ez = (double)hi[2] - bz;
    auto range = [&](const float4& s, double& gmin, double& gmax) {
      const double ax = (double)s.x - bx, ay = (double)s.y - by, az = (double)s.z - bz;
      const double D = ax * ax + ay * ay + az * az - (double)s.w * s.w;
      const double wx = -2.0 * ex * ax, wy = -2.0 * ey * ay, wz = -2.0 * ez * az;
      gmin = D + fmin(0.0, wx) + fmin(0.0, wy) + fmin(0.0, wz);
      gmax = D + fmax(0.0, wx) + fmax(0.0, wy) + fmax(0.0, wz);
    };
    double u = INFINITY;
    for (int q = tid; q < nsrc; q += 64) {
      double gmin, gmax;
      range(src[q], gmin, gmax);
      u = fmin(u, gmax);
    }
    u = wave_min(u);
    int n = 0;
    for (int q0 = 0; q0 < nsrc; q0 += 64) {
      const int q = q0 + tid;
      bool take = false;
      int id = 0;
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
      if (q < nsrc) {
        double gmin, gmax;
        s = source(q, id);
        range(s, gmin, gmax);
        take = gmin <= u;
      }
      const unsigned long long mk = __ballot(take);
      const int at = n + __popcll(mk & ((1ull << lane) - 1ull));
      if (take && at < SLMAX) {
        s_site[at] = s;
        s_sid[at] = id;
      }
      n += __popcll(mk);
    }
    if (n > SLMAX && !all_slow) {
      if (!run.split && tid == 0) stat_add(a, C_SPLIT, 1ull);
      if (!run.split) run.chunks();
      else run.directly();
      run.sub -= run.n;  // next() comes back to the same tets
      continue;
    }
    n = min(n, SLMAX);
    __syncthreads();
    // At most as many sites as a tet may keep candidates: no tet can be over the budget. The list is then cut down to
    // the sites that no owner of a box corner or of the centre beats on the whole box (exact in FP64): such a site owns
    // nothing here and its bisectors constrain no piece. (25 sites go down to 7 on the torus.)
    tight = n <= a.kmax && !all_slow;
    if (tight) {
      const float4 s = s_site[min(lane, n - 1)];
      const int id = s_sid[min(lane, n - 1)];
      const double cx = 0.5 * ex + bx, cy = 0.5 * ey + by, cz = 0.5 * ez + bz;
      const double ax = s.x - cx, ay = s.y - cy, az = s.z - cz;
      const double Dc = ax * ax + ay * ay + az * az - (double)s.w * s.w;
      bool keep = lane < n;
      for (int c = 0; c < 9; ++c) {
        // d at corner c (c = 8: the centre) up to a term common to all sites
        const double d = c == 8 ? Dc : Dc - ((c & 1) ? ex : -ex) * ax - ((c & 2) ? ey : -ey) * ay - ((c & 4) ? ez : -ez) * az;
        const double dmin = wave_min(lane < n ? d : INFINITY);
        const int w = __builtin_ctzll(__ballot(lane < n && d == dmin));
        const double Dw = __shfl(Dc, w);
        const double fx = fabs((double)s.x - __shfl(s.x, w)), fy = fabs((double)s.y - __shfl(s.y, w)),
                     fz = fabs((double)s.z - __shfl(s.z, w));
        keep = keep && !(Dc - Dw > ex * fx + ey * fy + ez * fz);
      }
      const unsigned long long mk = __ballot(keep);
      __syncthreads();
      if (keep) {
        const int at = __popcll(mk & ((1ull << lane) - 1ull));
        s_site[at] = s;
        s_sid[at] = id;
      }
      n = __popcll(mk);
    }
    if (tid == 0) s_nsl = n;
    __syncthreads();
  }

  // ---- 2. candidates of every tet: sites whose minimum over the tet is <= min_j max over the tet
  int tpt = 2;  // lanes per tet
  while (tpt < 64 && 2 * tpt * ntb <= 64) tpt *= 2;
  const int lt = tid / tpt, h = tid % tpt;
  auto tet_candidates = [&](int n, auto get, auto place, auto dominators) {  // get(q, id): site q; place(q, s, id): its
    constexpr bool DOM = decltype(dominators)::value;                        // list position
    const float4* tv = sd.tp + 4 * (size_t)(t0 + lt);
    const float4 o = tv[0];
    double y[3][3];
    for (int v = 1; v < 4; ++v) {
      y[v - 1][0] = (double)tv[v].x - o.x;
      y[v - 1][1] = (double)tv[v].y - o.y;
      y[v - 1][2] = (double)tv[v].z - o.z;
    }
    const double ycx = (y[0][0] + y[1][0] + y[2][0]) * 0.25, ycy = (y[0][1] + y[1][1] + y[2][1]) * 0.25,
                 ycz = (y[0][2] + y[1][2] + y[2][2]) * 0.25;
    double ax_, ay_, az_;
    auto values = [&](const float4& s, double* g) {
      ax_ = (double)s.x - o.x;
      ay_ = (double)s.y - o.y;
      az_ = (double)s.z - o.z;
      g[0] = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
      for (int v = 0; v < 3; ++v) g[v + 1] = g[0] - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
    };
    double U;
    // five dominators, each a site with its list position and id (the lowest id on ties, so that the choice does
    // not depend on the list's order): [0] attains U = min over sites of the maximum of g over the tet, [1 + v]
    // the minimum of g at vertex v (that vertex's owner). A site that one of them beats at all four vertices owns no
    // point of the tet and its bisector constrains no piece (the dominator is a candidate, and its own bisector already
    // does), so it is not a candidate; the same test among all candidates follows once they are sorted.
    double gb[DOM ? 5 : 1][4];
    if constexpr (DOM) {
      double dv[5];
      int dq[5], did[5];
      for (int k = 0; k < 5; ++k) {
        dv[k] = INFINITY;
        dq[k] = 0;
        did[k] = 0x7fffffff;
      }
      for (int q = h; q < n; q += tpt) {
        int id;
        const float4 s = get(q, id);
        double gq[4];
        values(s, gq);
        const double gmx = fmax(fmax(gq[0], gq[1]), fmax(gq[2], gq[3]));
        for (int k = 0; k < 5; ++k) {
          const double x = k == 0 ? gmx : gq[k - 1];
          if (x < dv[k] || (x == dv[k] && id < did[k])) {
            dv[k] = x;
            dq[k] = q;
            did[k] = id;
          }
        }
      }
      for (int off = 1; off < tpt; off <<= 1)
        for (int k = 0; k < 5; ++k) {
          const double x2 = __shfl_xor(dv[k], off);
          const int q2 = __shfl_xor(dq[k], off), id2 = __shfl_xor(did[k], off);
          if (x2 < dv[k] || (x2 == dv[k] && id2 < did[k])) {
            dv[k] = x2;
            dq[k] = q2;
            did[k] = id2;
          }
        }
      U = dv[0];
      for (int k = 0; k < 5; ++k) {
        int id;
        values(get(dq[k], id), gb[k]);
      }
    } else {
      U = INFINITY;
      for (int q = h; q < n; q += tpt) {
        int id;
        double gq[4];
        values(get(q, id), gq);
        U = fmin(U, fmax(fmax(gq[0], gq[1]), fmax(gq[2], gq[3])));
      }
      for (int off = 1; off < tpt; off <<= 1) U = fmin(U, __shfl_xor(U, off));
    }
    if (a.tet_U && sd.sign > 0 && h == 0) a.tet_U[sd.tet_off + t0 + lt] = U;
    for (int q = h; q < n; q += tpt) {
      int id;
      const float4 s = get(q, id);
      double g[4];
      values(s, g);
      const double gmn = fmin(fmin(g[0], g[1]), fmin(g[2], g[3]));
      bool dom = false;
      if constexpr (DOM)
        for (int k = 0; k < 5; ++k)
          dom = dom || (g[0] > gb[k][0] && g[1] > gb[k][1] && g[2] > gb[k][2] && g[3] > gb[k][3]);
      if (gmn <= U && !dom) {
        const int pos = atomicAdd(&s_m[lt], 1);
        if (pos < KRAW) {
          s_raw[lt][pos] = (unsigned char)place(q, s, id);
          s_key[lt][pos] = (float)(g[0] - 2.0 * (ycx * ax_ + ycy * ay_ + ycz * az_));
        }
      }
    }
  };
  const bool active = lt < ntb && ((cmask >> lt) & 1ull) && !all_slow;
  auto from_list = [&](int q, int& id) {
    id = s_sid[q];
    return s_site[q];
  };
  auto in_list = [](int q, const float4&, int) { return q; };
  if (run.direct()) {
    if (active)
      tet_candidates(nsrc, source,
                     [&](int, const float4& s, int id) {
                       const int at = atomicAdd(&s_nsl, 1);  // at most DIRECT x KRAW of them
                       s_site[at] = s;
                       s_sid[at] = id;
                       return at;
                     },
                     std::true_type{});
  } else if (tight) {
    if (active) tet_candidates(s_nsl, from_list, in_list, std::false_type{});
  } else if (active) {
    tet_candidates(s_nsl, from_list, in_list, std::true_type{});
  }
  __syncthreads();
  // ---- 3. each tet's candidates sorted by (power distance at the centroid, site id), one lane per candidate ranking
  //         it among its tet's and finding whether another one beats it (such a one is no further away)
  const bool mine = tid < ntb && ((cmask >> tid) & 1ull);
  int m = mine ? s_m[tid] : 0;
  if (mine && all_slow) m = KRAW + 1;
  {
    const int mr = m <= KRAW ? m : 0;
    int incl = mr;
    for (int off = 1; off < IT; off <<= 1) {
      const int v = __shfl_up(incl, off);
      if (lane >= off) incl += v;
    }
    if (tid < IT) s_off[tid] = (short)(incl - mr);
    if (tid == IT - 1) s_off[IT] = (short)incl;
  }
  __syncthreads();
  for (int e = tid; e < s_off[IT]; e += 64) {
    int lo_ = 0, hi_ = IT - 1;  // the last tet with s_off <= e
    while (lo_ < hi_) {
      const int mid = (lo_ + hi_ + 1) >> 1;
      if (s_off[mid] <= e) lo_ = mid;
      else hi_ = mid - 1;
    }
    const int c = e - s_off[lo_], n = s_m[lo_];
    const float kx = s_key[lo_][c];
    const unsigned char cx = s_raw[lo_][c];
    const int ix = s_sid[cx];
    const float4* tv = sd.tp + 4 * (size_t)(t0 + lo_);
    double gc[4];
    g4(tv, s_site[cx], gc);
    int rank = 0;
    bool beaten = false;
    for (int x = 0; x < n; ++x) {
      const float k = s_key[lo_][x];
      const int rx = s_raw[lo_][x];
      rank += (k < kx || (k == kx && s_sid[rx] < ix)) ? 1 : 0;
      if (k <= kx && !beaten) {
        double g[4];
        g4(tv, s_site[rx], g);
        beaten = g[0] < gc[0] && g[1] < gc[1] && g[2] < gc[2] && g[3] < gc[3];
      }
    }
    s_cand[lo_][rank] = cx;
    if (beaten) atomicOr(&s_beaten[lo_], 1ull << rank);
  }
  __syncthreads();
  if (mine) {
    // a tet over the budget goes to the large-capacity kernel, with its sorted, refined candidates when they fit the
    // list (else that kernel finds them among all sites); either way the choice depends on its own candidates only
    const float4* tv = sd.tp + 4 * (size_t)(t0 + tid);
    unsigned long long beaten = s_beaten[tid];
    if (m > a.kmax && m <= KRAW) m = refine_candidates(tv, s_site, s_cand[tid], m, beaten);
    if (m <= a.kmax) m = drop_beaten(s_cand[tid], m, beaten);
    if (m > a.kmax) stat_add(a, all_slow ? C_DEFER_BLOCK : C_DEFER_KMAX, 1ull);
    if (m > KRAW) {
      m = 0;
      defer_item(a, shape, t0 + tid, -1, -1);
    }
    s_m[tid] = m;
  }
  // ---- 4. piece slots, tet by tet with the tets ordered by candidate count, largest first: every piece of a tet
  //         loops over the same planes, so a wavefront's lanes then have similar trip counts
  {
    int rank = 0, off = 0;
    for (int u = 0; u < IT; ++u) {
      const int mu = __shfl(m, u);
      if (mu > m || (mu == m && u < tid)) {
        ++rank;
        off += mu;
      }
    }
    __syncthreads();
    if (tid < IT) {
      s_order[rank] = (short)tid;
      s_off[rank] = (short)off;
      if (rank == IT - 1) s_off[IT] = (short)(off + m);
    }
  }
  __syncthreads();
  const int npairs = s_off[IT];
  // one cursor per lane: lane 0 the piece slots, lane 1 + c the class's pieces (a contiguous range of the item's, since
  // its tets are ordered by candidate count)
  int c0 = 0, c1 = npairs;
  if (lane >= 1 && lane <= NCLASS) {
    const int lim1 = min(class_first(lane), a.kmax + 1), lim0 = min(class_first(lane - 1), a.kmax + 1);
    c0 = c1 = 0;
    for (int q = 0; q < IT; ++q) {
      const int mq = s_m[s_order[q]];
      if (mq >= lim1) c0 = s_off[q + 1];
      if (mq >= lim0) c1 = s_off[q + 1];
    }
  }
  long long at = 0;
  if (lane <= NCLASS && c1 > c0)
    at = (long long)atomicAdd(&a.counters[lane == 0 ? C_PIECE_SLOTS : C_CLASS + lane - 1], (unsigned long long)(c1 - c0));
  const long long base_l = __shfl(at, 0);
  if (base_l + npairs > (long long)a.pcap) {
    if (lane == 0) atomicOr(a.status, ST_PASS_FULL);
  } else {
    const int base = (int)base_l;
    for (int p0 = 0; p0 < npairs; p0 += 64) {
      const int p = p0 + tid;
      int lo_ = 0, hi_ = IT - 1;  // last position j with s_off[j] <= p
      while (lo_ < hi_) {
        const int mid = (lo_ + hi_ + 1) >> 1;
        if (s_off[mid] <= p) lo_ = mid;
        else hi_ = mid - 1;
      }
      const int tl = s_order[lo_], first = s_off[lo_], mt = p < npairs ? s_m[tl] : 0;
      int cl = 0;  // the piece's class
      for (int c = 1; c < NCLASS; ++c) cl += mt >= class_first(c) ? 1 : 0;
      const long long cl_at = __shfl(at, cl + 1);
      const int cl_c0 = __shfl(c0, cl + 1);
      if (p < npairs) {
        a.psite[base + p] = s_sid[s_cand[tl][p - first]];
        PieceDesc d;
        d.t = t0 + tl;
        d.shape = shape;
        d.first = base + first;
        d.m = mt;
        a.pdesc[base + p] = d;
        if (p == first && a.tet_slots) a.tet_slots[sd.tet_off + t0 + tl] = make_int2(base + first, mt);
        if (mt > a.kmax) {
          if (p == first) defer_item(a, shape, t0 + tl, -1, base + first);
        } else {
          // (items that found no slots have advanced the class cursors too, maybe before this one)
          const long long o = cl_at + (p - cl_c0);
          if (o < (long long)a.pcap) a.order[(size_t)cl * a.pcap + o] = base + p;
          else atomicOr(a.status, ST_PASS_FULL);
          ++n_cand;
        }
      }
    }
  }
  } while (run.next());
  }
  for (int off = 32; off > 0; off >>= 1) n_cand += __shfl_xor(n_cand, off);
  if (lane == 0 && n_cand) stat_add(a, C_CAND, n_cand);
}

// ---------------------------------------------------------------------------------------------------------------
// piece kernel
// ---------------------------------------------------------------------------------------------------------------
// Vertex slots per piece: 16 (19.7 KB of LDS a wavefront in FP32) or 12 (15.6 KB: more wavefronts fit a compute unit).
// A piece that outgrows them is redone after its chunk with a 64-slot polytope; the arithmetic is the same.
//
// A piece's terms are plain stores, no value of which the kernel waits for: with the sums and the element pieces
// entered into hash tables here, a chunk spent most of its time on the round trips of those dependent atomics.
constexpr int WIN = CHUNK + 2 * KMAX;  // candidates of the tets that a chunk touches

template <typename T, int SLOTS>
__global__ __launch_bounds__(64) void k_clip_pieces(ShapeArgs a) {
  typedef typename StoreOf<T, Topo32, SLOTS>::type PolyStore;
  __shared__ __attribute__((aligned(16))) unsigned char s_poly[PolyStore::coord_bytes(64)];
  __shared__ unsigned s_topo[SLOTS * 64];
  __shared__ float4 s_csite[WIN];
  __shared__ int s_csid[WIN];
  __shared__ int s_over[CHUNK];  // this chunk's pieces that ran out of vertex slots
  __shared__ int s_nover;
  if (*a.status & ST_PASS_FULL) return;  // some slots were never filled; the pass is redone with larger buffers
  const int lane = threadIdx.x;
  // the chunks of the classes, the most candidates first (their chunks take longest)
  int nc[NCLASS], nchunks = 0;
  for (int c = 0; c < NCLASS; ++c) {
    nc[c] = (int)a.counters[C_CLASS + c];
    nchunks += (nc[c] + CHUNK - 1) / CHUNK;
  }
  if (lane == 0) {
    s_nover = 0;
    if (blockIdx.x == 0) a.counters[C_CHUNKS] = (unsigned long long)nchunks;
  }
  unsigned long long n64 = 0;
  for (int chunk = blockIdx.x; chunk < nchunks; chunk += gridDim.x) {
    int cls = NCLASS - 1, k0 = chunk;
    while (k0 >= (nc[cls] + CHUNK - 1) / CHUNK) {
      k0 -= (nc[cls] + CHUNK - 1) / CHUNK;
      --cls;
    }
    k0 *= CHUNK;
    const int last = min(CHUNK, nc[cls] - k0) - 1;
    const int p = a.order[(size_t)cls * a.pcap + k0 + min(lane, last)];
    const PieceDesc d = a.pdesc[p];
    const bool run = lane <= last;
    // the candidates of the chunk's tets, tet by tet (a tet's pieces are consecutive entries): the lanes' own sites,
    // what the first lane's tet has before it and what the last one's has after it
    const int ci = p - d.first;
    const int before = __shfl(ci, 0), after = __shfl(d.m - 1 - ci, last), p_first = __shfl(d.first, 0), p_last = __shfl(p, last);
    __syncthreads();
    for (int q = lane; q < before + last + 1 + after; q += 64) {
      const int e = q - before;  // relative to the chunk
      const int s = e < 0 ? p_first + q : e > last ? p_last + (e - last) : -1;
      if (s >= 0) {
        const int id = a.psite[s];
        s_csid[q] = id;
        s_csite[q] = a.site[id];
      }
    }
    if (run) {
      const int id = a.psite[p];
      s_csid[before + lane] = id;
      s_csite[before + lane] = a.site[id];
    }
    __syncthreads();
    const ShapeDesc& sd = a.shapes[d.shape];
    const int co = before + lane - ci;  // where the tet's candidates start
    auto bind = [&](TetEnv& env, int t, int c0, int ci) {
      env.tv = sd.tp + 4 * (size_t)t;
      env.o = env.tv[0];
      env.face64 = sd.tf + 4 * (size_t)t;
      env.sid = s_csid + c0;
      env.csite = s_csite + c0;
      env.site = nullptr;
      env.ncs = INT_MAX;
      env.ci = ci;
      env.si = env.csite[ci];
      env.site_i = env.sid[ci];
    };
    typedef Clipper<T, Topo32, unsigned, SLOTS, false, RegTab> CL;
    CL cl;
    EmitAcc<CL> e;
    e.nface = e.nedge = e.nrpv = 0;
    int r = CLIP_EMPTY;
    if (run) {
      cl.st.bind(s_poly, s_topo, lane, 64);
      cl.tab.clear(0);
      cl.a = nullptr;  // only the exact predicates use it (not compiled into this kernel)
      cl.flags = a.flags;
      cl.np = 4 + d.m;
      cl.n64 = 0;
      cl.nex = 0;
      bind(cl.env, d.t, co, p - d.first);
      r = clip_piece(cl, d.m);
      n64 += cl.n64;
      if (r == CLIP_OK) {
        emit_scan(cl, e);
      } else {
        a.pref[p].word = 0;
        if (r == CLIP_DEFER) {
          stat_add(a, C_DEFER_CLIP, 1ull);
          defer_item(a, d.shape, d.t, p, d.first);
        } else if (r == CLIP_FULL) {
          s_over[atomicAdd(&s_nover, 1)] = lane;
        }
      }
    }
    // records: the lanes' runs one after the other, in the chunk's own range when they fit
    const int n = e.records();
    int incl = n;
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    const int total = __shfl(incl, 63);
    int base = chunk * REC_CHUNK;
    if (total > REC_CHUNK) {
      int q = 0;
      if (lane == 0) q = pool_records(a, total);
      base = __builtin_amdgcn_readfirstlane(q);
    }
    if (lane == 0) a.chunk_recs[chunk] = total > REC_CHUNK ? 0 : total;
    if (run && r == CLIP_OK && base >= 0) emit_out(cl, sd, d.t, e, p, base + incl - n, a);
    // Pieces that ran out of vertex slots are redone here, one per lane, with a BIG_VCAP-slot polytope. The chunk's
    // small polytopes are dead by now, so the first records live in their LDS; more go to a global-memory pool (same
    // arithmetic, same bits). Which path computes a piece must depend on the piece alone (an incremental update must
    // take back exactly the bits it added), so a full pool is a table overflow (the call is redone with larger
    // buffers), never a deferral.
    __syncthreads();
    const int nover = s_nover;
    if (nover) {
      if (lane < nover) {
        const int src = s_over[lane];  // the lane that had the piece
        const int pb = a.order[(size_t)cls * a.pcap + k0 + src];
        const PieceDesc db = a.pdesc[pb];
        const int cb0 = before + src - (pb - db.first);
        const ShapeDesc& sb = a.shapes[db.shape];
        const int m = db.m;
        constexpr size_t CB = sizeof(typename Coord4<T>::type) * BIG_VCAP;
        constexpr size_t REC = (CB + 8 * BIG_VCAP + 64 + 15) / 16 * 16;
        constexpr int NLDS = (int)(sizeof(s_poly) / REC);
        static_assert(CB + 8 * BIG_VCAP + 32 <= BIG_BYTES, "large-capacity polytope record");
        atomicAdd(&a.counters[C_BIG], 1ull);
        const unsigned long long slot = lane < NLDS ? 0ull : atomicAdd(&a.counters[C_BIG_POOL], 1ull);
        if (lane >= NLDS && slot >= (unsigned long long)a.big_cap) {
          atomicOr(a.status, ST_PASS_FULL);
        } else {
          unsigned char* b = lane < NLDS ? s_poly + (size_t)lane * REC : a.big + slot * BIG_BYTES;
          Clipper<T, Topo64, unsigned long long, BIG_VCAP, false, MemTab> cb;
          cb.st.c = reinterpret_cast<typename Coord4<T>::type*>(b);
          cb.st.w = reinterpret_cast<unsigned long long*>(b + CB);
          cb.st.stride = 1;
          cb.tab.base = b + CB + 8 * BIG_VCAP;
          cb.tab.stride = 1;
          cb.tab.clear(4 + m);
          cb.a = nullptr;
          cb.flags = a.flags;
          cb.np = 4 + m;
          cb.n64 = 0;
          cb.nex = 0;
          {
            cb.env.tv = sb.tp + 4 * (size_t)db.t;
            cb.env.o = cb.env.tv[0];
            cb.env.face64 = sb.tf + 4 * (size_t)db.t;
            cb.env.sid = s_csid + cb0;
            cb.env.csite = s_csite + cb0;
            cb.env.site = nullptr;
            cb.env.ncs = INT_MAX;
            cb.env.ci = pb - db.first;
            cb.env.si = cb.env.csite[cb.env.ci];
            cb.env.site_i = cb.env.sid[cb.env.ci];
          }
          const int rb = clip_piece(cb, m);
          n64 += cb.n64;
          if (rb == CLIP_OK) {
            emit_alone(cb, sb, db.t, pb, a);
          } else if (rb != CLIP_EMPTY) {  // a predicate undecided in FP64, or over BIG_VCAP vertices
            stat_add(a, C_DEFER_CLIP, 1ull);
            defer_item(a, db.shape, db.t, pb, db.first);
          }
        }
      }
      __syncthreads();
      if (lane == 0) s_nover = 0;
    }
  }
  for (int off = 32; off > 0; off >>= 1) n64 += __shfl_xor(n64, off);
  if (lane == 0 && n64) stat_add(a, C_FP64, n64);
}

// ---------------------------------------------------------------------------------------------------------------
// large-capacity kernel: one wavefront per deferred item, FP64 constructions, exact predicates, global scratch
// ---------------------------------------------------------------------------------------------------------------
struct SlowScratch {  // per wave, in global memory: the candidate lists, their vertex values, the global-memory polytopes
  static constexpr size_t cand_bytes = SLOW_KMAX * sizeof(int);
  static constexpr size_t key_bytes = SLOW_KMAX * sizeof(double);
  static constexpr size_t g_bytes = SLOW_KMAX * 4 * sizeof(double);   // g_j at the four tet vertices
  static constexpr size_t wave_bytes = 2 * (cand_bytes + key_bytes) + g_bytes;  // unsorted and sorted lists
  static constexpr size_t xyz_bytes = 64 * SLOW_VMAX * sizeof(Coord4<double>::type);  // [slot][lane]
  static constexpr size_t topo_bytes = 64 * SLOW_VMAX * sizeof(unsigned long long);    // [slot][lane]
  static constexpr size_t tab_bytes = 64 * (size_t)SLOW_PMAX;                          // [plane][lane]
  static constexpr size_t bytes = wave_bytes + xyz_bytes + topo_bytes + tab_bytes;
};
constexpr int SLOW_LDS_ITEMS = 512;  // the first deferred items go to the LDS variant (one item per wave)

// The LDS variant (few items: latency) keeps the candidate lists and 32 lanes' polytopes (32 vertices) in LDS; an item
// with more than 256 candidates, or a piece with more vertices, is handed to the global variant through the overflow
// list, and so are the candidates past an item's first 32: one wave that took them round after round was the launch's
// tail (1.23 -> 0.77 ms on a batch of 48 shapes). The global variant (many items: throughput) keeps the lists and all 64
// lanes' polytopes (64 vertices) in its scratch and takes the items past the LDS variant's share, then the overflow
// list.
template <bool LDS>
struct SlowCfg;
template <>
struct SlowCfg<true> {
  static constexpr int CL = 32, VCAP = 32, KCAP = 256;
  typedef unsigned Mask;
};
template <>
struct SlowCfg<false> {
  static constexpr int CL = 64, VCAP = SLOW_VMAX, KCAP = SLOW_KMAX;
  typedef unsigned long long Mask;
};

__device__ inline void push_overflow(const ShapeArgs& a, int4 item) {
  const unsigned long long idx = atomicAdd(&a.counters[C_DEFER2], 1ull);
  if (idx < (unsigned long long)a.deferred2_cap) a.deferred2[idx] = item;
  else atomicOr(a.status, ST_PASS_FULL);
}

// One wavefront per deferred item: the lanes split the scan over all of the shape's sites (candidates are
// compacted in ascending site order by ballots), drop dominated candidates and rank-sort the rest, then clip the
// pieces with FP64 polytopes (lanes interleaved slot by slot).
template <bool LDS>
__global__ __launch_bounds__(64, LDS ? 1 : 2) void k_clip_slow(ShapeArgs a, unsigned char* scratch, int item_begin, int item_end) {
  typedef SlowCfg<LDS> C;
  constexpr int CL = C::CL, KC = C::KCAP;
  __shared__ Coord4<double>::type s_xyz[LDS ? C::VCAP * CL : 1];
  __shared__ unsigned long long s_topo[LDS ? C::VCAP * CL : 1];
  __shared__ unsigned char s_tab[LDS ? (4 + KC) * CL : 1];
  __shared__ int s_cand[LDS ? 2 * KC : 1];
  __shared__ double s_key[LDS ? 6 * KC : 1];
  // on-chip copies for the clipping loop, whose plane rebuilds would otherwise wait on memory: the item's tet and
  // the sites of its first SC candidates (sorted positions)
  constexpr int SC = 256;
  __shared__ float4 s_tv4[4];
  __shared__ double4 s_tf4[4];
  __shared__ float4 s_csite[SC];
  constexpr int NDOM = 6;
  __shared__ double s_dom[NDOM][4];
  if (*a.status & ST_PASS_FULL) return;
  const int n_main = (int)min(min(a.counters[C_DEFER_ITEMS], (unsigned long long)a.deferred_cap),
                              (unsigned long long)item_end);
  const int n_over = LDS ? 0 : (int)min(a.counters[C_DEFER2], (unsigned long long)a.deferred2_cap);
  const int n_items = max(n_main - item_begin, 0) + n_over;
  const int lane = threadIdx.x;
  unsigned char* wbase = scratch + (size_t)blockIdx.x * SlowScratch::bytes;
  int* cand = LDS ? s_cand : (int*)wbase;
  int* scand = LDS ? s_cand + KC : (int*)(wbase + SlowScratch::cand_bytes + SlowScratch::key_bytes);
  double* key = LDS ? s_key : (double*)(wbase + SlowScratch::cand_bytes);
  double* skey = LDS ? s_key + KC : (double*)(wbase + 2 * SlowScratch::cand_bytes + SlowScratch::key_bytes);
  double* gv = LDS ? s_key + 2 * KC : (double*)(wbase + 2 * (SlowScratch::cand_bytes + SlowScratch::key_bytes));
  const int cl_lane = lane < CL ? lane : 0;
  Coord4<double>::type* xyz =
      LDS ? s_xyz + cl_lane : (Coord4<double>::type*)(wbase + SlowScratch::wave_bytes) + cl_lane;
  unsigned long long* topo =
      LDS ? s_topo + cl_lane
          : (unsigned long long*)(wbase + SlowScratch::wave_bytes + SlowScratch::xyz_bytes) + cl_lane;
  unsigned char* tab =
      LDS ? s_tab + cl_lane : wbase + SlowScratch::wave_bytes + SlowScratch::xyz_bytes + SlowScratch::topo_bytes + cl_lane;
  unsigned long long n64 = 0, nex = 0;
  for (int vi = blockIdx.x; vi < n_items; vi += gridDim.x) {
    const int main_count = max(n_main - item_begin, 0);
    const int4 di = vi < main_count ? a.deferred[item_begin + vi] : a.deferred2[vi - main_count];
    const ShapeDesc sd = a.shapes[__builtin_amdgcn_readfirstlane(di.x)];
    const int t = di.y;
    const int want = di.z;  // piece slot, or -1: every candidate of the tet, or -1 - k: those from the k-th on
    int first = di.w;       // the tet's first piece slot, or -1: its candidates are found here
    const float4* ssite = a.site + sd.site_off;
    float4 tv[4];
    for (int v = 0; v < 4; ++v) tv[v] = sd.tp[4 * (size_t)t + v];
    if (lane < 4) {
      s_tv4[lane] = sd.tp[4 * (size_t)t + lane];
      s_tf4[lane] = sd.tf[4 * (size_t)t + lane];
    }
    const float4 o = tv[0];
    double y[3][3];
    for (int v = 1; v < 4; ++v) {
      y[v - 1][0] = (double)tv[v].x - o.x;
      y[v - 1][1] = (double)tv[v].y - o.y;
      y[v - 1][2] = (double)tv[v].z - o.z;
    }
    const double ycx = (y[0][0] + y[1][0] + y[2][0]) * 0.25, ycy = (y[0][1] + y[1][1] + y[2][1]) * 0.25,
                 ycz = (y[0][2] + y[1][2] + y[2][2]) * 0.25;
    // a tet's sorted candidates come with its piece slots when they fit the candidate kernel's list (a function of
    // the tet's candidates only); otherwise they are found here among all sites
    int m = 0;
    if (first >= 0) {
      m = a.pdesc[first].m;
      if (LDS && m > KC) {  // (a tet whose candidates this kernel's global variant found)
        if (lane == 0) push_overflow(a, di);
        continue;
      }
      for (int x = lane; x < m; x += 64) {
        const int sx = a.psite[first + x];
        scand[x] = sx;
        if (x < SC) s_csite[x] = a.site[sx];
      }
      __syncthreads();
    } else {
      // candidates among ALL sites of the shape (same exact test as the fast kernel)
      // the sites least at each vertex, at the centre and in their largest vertex value: what one of these beats at all
      // four vertices is left out of the list at once
      double lv[NDOM];
      int ls[NDOM];
      for (int q = 0; q < NDOM; ++q) {
        lv[q] = INFINITY;
        ls[q] = 0;
      }
      for (int j = lane; j < sd.ns; j += 64) {
        float4 s = ssite[j];
        double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
        double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
        double g[NDOM];
        g[0] = D;
        g[4] = D;
        for (int v = 0; v < 3; ++v) {
          g[1 + v] = D - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
          g[4] = fmax(g[4], g[1 + v]);
        }
        g[5] = D - 2.0 * (ycx * ax_ + ycy * ay_ + ycz * az_);
        for (int q = 0; q < NDOM; ++q)
          if (g[q] < lv[q]) {
            lv[q] = g[q];
            ls[q] = j;
          }
      }
      for (int q = 0; q < NDOM; ++q)
        for (int off = 32; off > 0; off >>= 1) {
          const double v = __shfl_xor(lv[q], off);
          const int j = __shfl_xor(ls[q], off);
          if (v < lv[q] || (v == lv[q] && j < ls[q])) {
            lv[q] = v;
            ls[q] = j;
          }
        }
      const double U = lv[4];
      if (a.tet_U && sd.sign > 0 && lane == 0) a.tet_U[sd.tet_off + t] = U;
      __syncthreads();  // the last item's dominators have been read
      if (lane < NDOM) {
        int j = 0;
        for (int q = 0; q < NDOM; ++q) j = lane == q ? ls[q] : j;
        const float4 s = ssite[j];
        const double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
        const double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
        s_dom[lane][0] = D;
        for (int v = 0; v < 3; ++v) s_dom[lane][1 + v] = D - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
      }
      __syncthreads();
      int raw = 0;  // candidates before that
      for (int base = 0; base < sd.ns; base += 64) {
        const int j = base + lane;
        bool take = false;
        double kk = 0.0;
        if (j < sd.ns) {
          float4 s = ssite[j];
          double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
          double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
          double gmn = D, g[4];
          g[0] = D;
          for (int v = 0; v < 3; ++v) {
            g[1 + v] = D - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
            gmn = fmin(gmn, g[1 + v]);
          }
          take = gmn <= U;
          raw += take ? 1 : 0;
          for (int q = 0; q < NDOM && take; ++q)
            take = !(s_dom[q][0] < g[0] && s_dom[q][1] < g[1] && s_dom[q][2] < g[2] && s_dom[q][3] < g[3]);
          kk = D - 2.0 * (ycx * ax_ + ycy * ay_ + ycz * az_);
        }
        unsigned long long mask = __ballot(take);
        int pos = m + __popcll(mask & ((1ull << lane) - 1ull));
        if (take && pos < KC) {
          cand[pos] = sd.site_off + j;
          key[pos] = kk;
        }
        m += __popcll(mask);
      }
      for (int off = 32; off > 0; off >>= 1) raw += __shfl_xor(raw, off);
      if (raw > SLOW_KMAX) {
        if (lane == 0) atomicOr(a.status, ST_SLOW_CAPACITY);
        continue;
      }
      if (m > KC) {  // (the LDS variant only)
        if (lane == 0) push_overflow(a, di);
        continue;
      }
      __syncthreads();
      // drop every candidate that another one beats at all four tet vertices (g is affine, so then everywhere on the
      // tet: it owns nothing and its bisector constrains no piece); the values are exact in FP64
      for (int x = lane; x < m; x += 64) {
        const float4 s = a.site[cand[x]];
        const double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
        const double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
        gv[4 * x] = D;
        for (int v = 0; v < 3; ++v) gv[4 * x + 1 + v] = D - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
      }
      __syncthreads();
      int kept = 0;
      for (int base = 0; base < m; base += 64) {
        const int x = base + lane;
        bool keep = false;
        double kx = 0.0;
        int cx = 0;
        if (x < m) {
          const double g0 = gv[4 * x], g1 = gv[4 * x + 1], g2 = gv[4 * x + 2], g3 = gv[4 * x + 3];
          keep = true;
          for (int q = 0; q < m && keep; ++q)
            keep = !(gv[4 * q] < g0 && gv[4 * q + 1] < g1 && gv[4 * q + 2] < g2 && gv[4 * q + 3] < g3);
          kx = key[x];
          cx = cand[x];
        }
        const unsigned long long mask = __ballot(keep);
        __syncthreads();  // every lane has read cand/key of this chunk before they are overwritten in place
        if (keep) {
          const int pos = kept + __popcll(mask & ((1ull << lane) - 1ull));
          cand[pos] = cx;
          key[pos] = kx;
        }
        kept += __popcll(mask);
      }
      m = kept;
      __syncthreads();
      // rank sort by (key, position): positions ascend with the site id, so ties keep the site order
      for (int x = lane; x < m; x += 64) {
        const double kx = key[x];
        int rank = 0;
        for (int q = 0; q < m; ++q) {
          const double kq = key[q];
          rank += (kq < kx || (kq == kx && q < x)) ? 1 : 0;
        }
        scand[rank] = cand[x];
        skey[rank] = kx;
        if (rank < SC) s_csite[rank] = a.site[cand[x]];
      }
      // piece slots for the tet's candidates
      __syncthreads();
      int q = -1;
      if (lane == 0) {
        const unsigned long long at = atomicAdd(&a.counters[C_PIECE_SLOTS], (unsigned long long)m);
        if (at + m <= (unsigned long long)a.pcap) q = (int)at;
        else atomicOr(a.status, ST_PASS_FULL);
      }
      first = __builtin_amdgcn_readfirstlane(q);
      if (first < 0) continue;
      if (lane == 0 && a.tet_slots) a.tet_slots[sd.tet_off + t] = make_int2(first, m);
      for (int x = lane; x < m; x += 64) {
        PieceDesc d;
        d.t = t;
        d.shape = di.x;
        d.first = first;
        d.m = m;
        a.pdesc[first + x] = d;
        a.psite[first + x] = scand[x];
        a.pref[first + x].word = 0;
      }
    }
    if (lane < CL)
      for (int k = 0; k < 4 + m; ++k) tab[CL * k] = 0;  // the plane ids of this item start unpaired
    __syncthreads();
    // one round of the LDS variant; the others run beside each other in the global one
    if (LDS && want < 0 && m > CL && lane == 0) push_overflow(a, make_int4(di.x, t, -1 - CL, first));
    const int c_end = LDS && want < 0 ? min(m, CL) : m;
    for (int ci = lane + (want < 0 ? -1 - want : 0); ci < c_end && lane < CL; ci += CL) {
      if (want >= 0 && first + ci != want) continue;
      Clipper<double, Topo64, typename C::Mask, C::VCAP, true, MemTab> cl;
      cl.st.c = xyz;
      cl.st.w = topo;
      cl.st.stride = CL;
      cl.tab = MemTab{tab, CL};
      cl.a = &a;
      cl.flags = a.flags & ~RPD_FORCE_FP64;
      cl.np = 4 + m;
      cl.n64 = 0;
      cl.nex = 0;
      cl.env.tv = s_tv4;
      cl.env.o = s_tv4[0];
      cl.env.face64 = s_tf4;
      cl.env.sid = scand;
      cl.env.csite = s_csite;
      cl.env.site = a.site;
      cl.env.ncs = min(m, SC);
      cl.env.ci = ci;
      cl.env.si = a.site[scand[ci]];
      cl.env.site_i = scand[ci];
      a.pref[first + ci].word = 0;
      int r = clip_piece(cl, m);
      n64 += cl.n64;
      nex += cl.nex;
      if (r == CLIP_FULL) {  // out of vertex slots: the global variant redoes the piece with the same candidates
        if (LDS) push_overflow(a, make_int4(di.x, t, first + ci, first));
        else atomicOr(a.status, ST_SLOW_CAPACITY);
        continue;
      }
      if (r == CLIP_OK) {
        emit_alone(cl, sd, t, first + ci, a);
      }
    }
    __syncthreads();  // the candidate list is rewritten by the next item
  }
  for (int off = 32; off > 0; off >>= 1) {
    n64 += __shfl_xor(n64, off);
    nex += __shfl_xor(nex, off);
  }
  if (lane == 0) {
    if (n64) stat_add(a, C_FP64, n64);
    if (nex) stat_add(a, C_EXACT, nex);
  }
}

// ---------------------------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------------------------
// The piece count is known on the device only: a grid of several times the wavefronts that fit the chip takes the
// chunks in grid-stride order (workgroups past the last chunk exit at once).
template <typename T, int SLOTS>
static hipError_t launch_pieces(const ShapeArgs& a, hipStream_t s) {
  const int grid = std::max(1, std::min(chunk_cap(a.pcap), 8192));
  hipLaunchKernelGGL((k_clip_pieces<T, SLOTS>), dim3(grid), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_candidates(const ShapeArgs& a, hipStream_t s) {
  if (a.nitems == 0) return hipSuccess;
  if (a.ngrp > 0) hipLaunchKernelGGL(k_group_sites, dim3(a.ngrp), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_candidates, dim3(a.nitems), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_clip_pieces(const ShapeArgs& a, int precision, int slots, hipStream_t s) {
  if (a.nitems == 0) return hipSuccess;
  if (precision == RPD_FP64) return launch_pieces<double, 16>(a, s);
  if (slots == 12) return launch_pieces<float, 12>(a, s);
  return launch_pieces<float, 16>(a, s);
}

size_t slow_scratch_bytes(int waves) { return (size_t)waves * SlowScratch::bytes; }

// the first SLOW_LDS_ITEMS items by the LDS variant, the rest by the global one (whose waves exit at once when there
// is no rest); the item count is read on the device
hipError_t launch_clip_slow(const ShapeArgs& a, unsigned char* scratch, int waves, hipStream_t s) {
  const int lds_waves = waves < SLOW_LDS_ITEMS ? waves : SLOW_LDS_ITEMS;
  hipLaunchKernelGGL(k_clip_slow<true>, dim3(lds_waves), dim3(64), 0, s, a, scratch, 0, SLOW_LDS_ITEMS);
  hipLaunchKernelGGL(k_clip_slow<false>, dim3(waves), dim3(64), 0, s, a, scratch, SLOW_LDS_ITEMS, INT_MAX);
  return hipGetLastError();
}

}  // namespace rpd
