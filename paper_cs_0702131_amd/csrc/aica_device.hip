// HIP (gfx950) kernels and the C ABI of the AICA Lennard-Jones library.
//
// Per step (aica_bin, then aica_forces / aica_forces_adjoint):
//   locate (and count) -> scan -> scatter -> in-cell sort      : CSR cell occupancy (Sec. 2.2)
//   gather                                                     : cell-sorted SoA, group-local coordinates
//   pair kernel                                                : real-real and periodic referred pairs
//                                                                (Sec. 2.3.1, 2.3.2): the full lists (aica_neigh.inc:
//                                                                every pair from both sides, forces in caller
//                                                                order) or the half lists (aica_pair.inc: Newton
//                                                                reactions, Sec. 2.2, kept as records)
//   finalize (half lists), reduce                              : per-molecule sums in caller order, U, W
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <type_traits>
#include <string>
#include <vector>

#include "aica_internal.h"
#include "aica_kernels.h"

namespace aica {
const char *last_error_cstr();
}

using namespace aica;

#define HIPCHK(x)                                                                                       \
  do {                                                                                                  \
    hipError_t _e = (x);                                                                                \
    if (_e != hipSuccess) return fail(AICA_E_HIP, std::string("HIP error: ") + hipGetErrorString(_e) + \
                                                      " at " + __FILE__ + ":" + std::to_string(__LINE__)); \
  } while (0)

namespace {

struct DBuf {
  void *p = nullptr;
  size_t bytes = 0;
  ~DBuf() {
    if (p) (void)hipFree(p);
  }
  int ensure(size_t nbytes) {
    if (nbytes <= bytes && p) return AICA_OK;
    if (p) {
      (void)hipFree(p);
      p = nullptr;
      bytes = 0;
    }
    size_t nb = std::max<size_t>(nbytes, 256);
    if (hipMalloc(&p, nb) != hipSuccess) {
      p = nullptr;
      return fail(AICA_E_NOMEM, "device allocation of " + std::to_string(nb) + " bytes failed");
    }
    bytes = nb;
    return AICA_OK;
  }
  template <class T>
  T *as() const {
    return (T *)p;
  }
  void swap(DBuf &o) {
    std::swap(p, o.p);
    std::swap(bytes, o.bytes);
  }
};

template <class T>
int upload(DBuf &b, const std::vector<T> &v) {
  int rc = b.ensure(sizeof(T) * std::max<size_t>(v.size(), 1));
  if (rc) return rc;
  if (!v.empty()) HIPCHK(hipMemcpy(b.p, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice));
  return AICA_OK;
}

struct Timer {
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pending;
  double ms = 0;
  int64_t launches = 0;
};

}  // namespace

struct aica_dil {
  Geometry geo;
  std::vector<int32_t> order, rank;
  std::vector<uint8_t> split_depth;  // k-d tree of the sorted order (groups are its subtrees)
  std::vector<CellPair> pairs;
  double rcut = 0, guard = 0, build_seconds = 0, group_seconds = 0;
  int32_t predicate = AICA_DIL_CLOSEST;
  int device = 0;
  bool geometry_on_device = false;
  // device geometry for point location (mesh cell ids)
  DBuf d_rec_off, d_rec, d_bb;  // point-location cell records and padded boxes, sorted cell order
  DBuf d_rec32;                 // FP32 records for the previous-cell test (cells of at most kR32 float4)
  DBuf d_pl32;                  // plane records of the boundary triangles (kPl float4 per cell, with d_rec32)
  DBuf d_nbr_off, d_nbr;        // cells across each cell's interior faces (sorted ids)
  bool has_rec32 = false;
  DBuf d_gb_off, d_gb_cell;
  double glo[3] = {0, 0, 0}, gh = 1;
  int64_t gnb[3] = {1, 1, 1};
  // interaction groups (depend on the number density; built on the first aica_bin)
  bool groups_ready = false, neigh_ready = false;
  Groups grp;
  DBuf d_orig, d_g_cell0, d_e_off, d_e_B, d_e_vec32, d_e_vec64, d_nl_off, d_nl_e, d_nl_d, d_nl_r, d_rcnt;
  // full neighbour lists of the force kernel (its own groups; same lifetime)
  Neigh nb;
  DBuf d_nb_cell0, d_nb_run_off, d_nb_runs, d_nb_vec32, d_nb_vec64, d_nb_orig, d_nb_eoff, d_nb_ioff, d_nb_imask;
  DBuf d_of_cell, d_half;       // the half lists' group of each sorted cell; HalfFrames
  // a pair vector formed in the frames of the full lists differs per axis from that of the half lists by at most
  // (half an ulp of the compute type) * frame_reach (FP32, FP64) + frame_err
  double frame_reach[2] = {0, 0}, frame_err = 0;
  DBuf d_box;                   // [groups][6] box of each group's molecules in its frame (compute type)
  // rotating referral: the groups of the full lists without a turned entry, then those with one
  DBuf d_nb_glist;
  int64_t nb_plain_groups = 0;
  DBuf d_rot64;                 // [27][9] rotation of every image code (only with rotational referral)
  // per step
  bool bin_valid = false;
  int64_t wsteps_groups = 0;  // groups whose wave-step counts d_gnp holds (a forward call on the current binning)
  int64_t n = 0;
  unsigned long long *host_status = nullptr;    // pinned: the counts of a binning
  const void *bin_pos = nullptr;
  int32_t bin_dtype = 0;
  int64_t jtotal = 0;
  DBuf d_cell_of, d_count, d_cell_start, d_rank, d_perm, d_slot_base, d_cell_sorted;
  DBuf d_scan_tmp, d_status, d_slow;
  DBuf d_ref;                   // [n] float4 per caller molecule id: centre and radius of a ball that lies
                                // inside the molecule's cell of the last binning (radius 0: none)
  DBuf d_perm_prev;     // the previous binning's permutation during aica_bin
  int64_t perm_n = -1;  // molecule count of the binning held in d_perm and d_cell_sorted (-1: none)
  int64_t located[3] = {0, 0, 0};  // last binning: molecules located by their ball, by the FP32 record, slowly
  // force / adjoint workspace
  DBuf d_pos, d_own, d_jpart, d_gpart, d_gnp, d_gG, d_gpar;
  DBuf d_pairs, d_pcount;
  DBuf d_red;  // stage-1 rows of the group reductions
  bool profiling = false;
  uint32_t epoch = 0;          // tag of the reaction records written by the current call
  size_t jpart_tagged = 0;     // bytes of d_jpart known to hold no valid tag
  std::map<std::string, Timer> timers;
  ~aica_dil() {
    if (host_status) (void)hipHostFree(host_status);
  }
};

// =====================================================================================================
// kernels: binning

namespace {

__device__ __forceinline__ double orient3(const double *a, const double *b, const double *c, const double *d) {
  const double u0 = b[0] - a[0], u1 = b[1] - a[1], u2 = b[2] - a[2];
  const double v0 = c[0] - a[0], v1 = c[1] - a[1], v2 = c[2] - a[2];
  const double w0 = d[0] - a[0], w1 = d[1] - a[1], w2 = d[2] - a[2];
  return u0 * (v1 * w2 - v2 * w1) + u1 * (v2 * w0 - v0 * w2) + u2 * (v0 * w1 - v1 * w0);
}

// Cell records for point location, one per sorted cell, contiguous:
//   [nf, cc(3), fc_0(3) .. fc_{nf-1}(3), len_0 .. len_{nf-1}, loop_0(3 len_0) .. loop_{nf-1}(3 len_{nf-1})]
// with cc the cell's vertex mean, fc the face centroids and each face's vertex loop oriented outward
// from the cell (counts stored as doubles, exact).
//
// Is p inside the cell: some tetrahedron (cc, fc, v_k, v_k+1) contains p, with a relative tolerance tau
// of that tetrahedron's volume (tau = 1e-12 for membership; the tests of the previous cell and its neighbours ask
// for tau = -1e-9, i.e. strictly inside).  The four barycentric tests of tetrahedron k are: the outer face,
// orient(p, fc, v_k, v_k+1) >= -tol; the edge plane through cc, orient(cc, p, v_k, v_k+1) >= -tol; and
// the two spoke planes (cc, fc, v_k), (cc, fc, v_k+1).  A group of 32 lanes deals the tetrahedra out (the same value
// in the group's lanes).
__device__ __forceinline__ bool point_in_rec(const double *p, const double *R, double tau) {
  const int lane = (int)(threadIdx.x & 31), g0 = (int)(threadIdx.x & 32);
  const int nf = (int)R[0];
  const double cc[3] = {R[1], R[2], R[3]};
  const double *FC = R + 4, *LEN = FC + 3 * nf, *V = LEN + nf;
  bool in = false;
  int off = 0;  // tetrahedra of the faces before kb
  for (int kb = 0; kb < nf; kb += 32) {
    const int m = min(nf - kb, 32);
    const int len = lane < m ? (int)LEN[kb + lane] : 0;  // lane k: face kb + k
    for (int t0 = 0, end = 1; t0 < end; t0 += 32) {
      const int t = t0 + lane;  // the lane's tetrahedron, of face f, whose fl tetrahedra start at v0
      int f = 0, v0 = 0, fl = 0;
      end = 0;
      for (int k = 0; k < m; ++k) {
        const int lk = __shfl(len, g0 + k, 64);
        if (t >= end) {
          f = k;
          v0 = end;
          fl = lk;
        }
        end += lk;
      }
      if (t < end) {
        const double *fc = FC + 3 * (int64_t)(kb + f), *vp = V + 3 * (int64_t)(off + t);
        const double *vn = V + 3 * (int64_t)(off + (t + 1 == v0 + fl ? v0 : t + 1));
        const double tol = -tau * fabs(orient3(cc, fc, vp, vn));
        in = in || (orient3(cc, fc, vp, p) >= tol && -orient3(cc, fc, vn, p) >= tol && orient3(p, fc, vp, vn) >= tol &&
                    orient3(cc, p, vp, vn) >= tol);
      }
      if (t0 + 32 >= end) off += end;
    }
  }
  return ((__builtin_amdgcn_ballot_w64(in) >> (threadIdx.x & 32)) & 0xFFFFFFFFull) != 0;
}

// FP32 copies of the cell records for the previous-cell test, fixed stride kR32 float4 per sorted cell:
//   [0] (nf, a.x, a.y, a.z) with a the FP32-rounded vertex mean; [1] (cc - a, 0);
//   [2 .. 2 + nf) (fc_k - a, len_k); then the face loops, one vertex (v - a, 0) per float4, except that the
//   first vertex of face k's loop carries in .w the sorted id of the cell across face k (int bits; -1 on
//   a boundary face).
// A point is accepted when some tetrahedron contains it with every orientation above 1e-4 of that
// tetrahedron's own (FP32) orientation.  The FP32 rounding of the records and of the orientations is
// below 1e-5 of that scale, so an accepted point is strictly inside in exact arithmetic too (the FP64
// test with tau = -1e-9 accepts it); anything else goes to the FP64 test.
constexpr int kR32 = 32;

__device__ __forceinline__ float orient3f(const float *a, const float *b, const float *c, const float *d) {
  const float u0 = b[0] - a[0], u1 = b[1] - a[1], u2 = b[2] - a[2];
  const float v0 = c[0] - a[0], v1 = c[1] - a[1], v2 = c[2] - a[2];
  const float w0 = d[0] - a[0], w1 = d[1] - a[1], w2 = d[2] - a[2];
  return u0 * (v1 * w2 - v2 * w1) + u1 * (v2 * w0 - v0 * w2) + u2 * (v0 * w1 - v1 * w0);
}

// Plane records: per sorted cell kPl float4 (n, d), one per boundary triangle of the cell's face fans: the
// inward unit normal n and d = n.(f - a) for a point f of the triangle, in the frame a of the cell's FP32
// record, so that n.(p - a) - d is the signed distance of p from the triangle's plane (positive inside).
// Unused entries are (0, 0, 0, -3e38); a cell with more triangles than kPl has (0, 0, 0, 3e38) in entry 0,
// so that its test never accepts.
constexpr int kPl = 24;

// The FP32 tests of one molecule by a group of 32 lanes, a boundary triangle (and its tetrahedron) per lane: the lanes
// read a record in a few wide loads and no lane walks the faces in turn.  With the fixed stride of the records a cell
// has at most 7 faces and 26 triangles (over kPl of them, its plane test never accepts).
struct RecLane {
  float f[3], vp[3], vn[3];  // this lane's triangle: face centroid and two consecutive vertices, relative to a
  float pr[3], cc[3];
  bool on;                   // the lane has a triangle
  int32_t across;            // the cell across the face whose centroid direction best matches p - cc (-1: boundary)
};
__device__ __forceinline__ RecLane load_rec32(const double *p, const float4 *R) {
  const int c = (int)(threadIdx.x & 31), g0 = (int)(threadIdx.x & 32);
  const float4 h = R[0], h2 = R[1];
  const int nf = (int)h.x;
  RecLane r;
  r.pr[0] = (float)(p[0] - (double)h.y);
  r.pr[1] = (float)(p[1] - (double)h.z);
  r.pr[2] = (float)(p[2] - (double)h.w);
  r.cc[0] = h2.x;
  r.cc[1] = h2.y;
  r.cc[2] = h2.z;
  const float4 fk = c < nf ? R[2 + c] : make_float4(0.f, 0.f, 0.f, 0.f);  // lane k: face k
  // the lane's triangle: face `face` starts at vertex v0 of the list and has len of them
  int face = 0, v0 = 0, len = 0, off = 0;
  float bs = -3.0e38f;
  int boff = 0;
  const float e0 = fk.x - r.cc[0], e1 = fk.y - r.cc[1], e2 = fk.z - r.cc[2];
  const float sc = c < nf ? ((r.pr[0] - r.cc[0]) * e0 + (r.pr[1] - r.cc[1]) * e1 + (r.pr[2] - r.cc[2]) * e2) /
                                (e0 * e0 + e1 * e1 + e2 * e2)
                          : -3.0e38f;
  for (int k = 0; k < nf; ++k) {
    const int lk = (int)__shfl(fk.w, g0 + k, 64);
    const float sk = __shfl(sc, g0 + k, 64);
    if (c >= off) {
      face = k;
      v0 = off;
      len = lk;
    }
    if (sk > bs) {
      bs = sk;
      boff = off;
    }
    off += lk;
  }
  r.on = c < off;
  r.f[0] = __shfl(fk.x, g0 + face, 64);
  r.f[1] = __shfl(fk.y, g0 + face, 64);
  r.f[2] = __shfl(fk.z, g0 + face, 64);
  const float4 *V = R + 2 + nf;
  const int j = r.on ? c : 0, jn = r.on ? (c + 1 == v0 + len ? v0 : c + 1) : 0;
  const float4 a = V[j], b = V[jn];
  r.vp[0] = a.x;
  r.vp[1] = a.y;
  r.vp[2] = a.z;
  r.vn[0] = b.x;
  r.vn[1] = b.y;
  r.vn[2] = b.z;
  r.across = __float_as_int(__shfl(a.w, g0 + boff, 64));
  return r;
}
// Some tetrahedron surely contains the point (the margin at kR32); the same value in all 32 lanes.
__device__ __forceinline__ bool rec_lanes_inside(const RecLane &r) {
  const float tol = 1e-4f * fabsf(orient3f(r.cc, r.f, r.vp, r.vn));
  const bool in = r.on && orient3f(r.cc, r.f, r.vp, r.pr) > tol && -orient3f(r.cc, r.f, r.vn, r.pr) > tol &&
                  orient3f(r.pr, r.f, r.vp, r.vn) > tol && orient3f(r.cc, r.pr, r.vp, r.vn) > tol;
  return ((__builtin_amdgcn_ballot_w64(in) >> (threadIdx.x & 32)) & 0xFFFFFFFFull) != 0;
}
// Radius of a ball about p that lies inside the cell of FP32 record R, for a p that the record shows
// strictly inside (a triangle per lane): the cell's boundary is made of the face-fan triangles, and the distance from p to a
// triangle is at least the distance to its plane, so the smallest plane distance bounds the distance to
// the boundary from below.  FP32 rounding is covered by a margin of 1e-4 of the cell's size.  Returns the
// ball as (centre rounded to FP32, radius reduced by that rounding); radius 0 when nothing is left.
__device__ __forceinline__ float4 rec_lanes_ball(const RecLane &r, const double *p, const float4 *R) {
  const float a0 = r.vp[0] - r.f[0], a1 = r.vp[1] - r.f[1], a2 = r.vp[2] - r.f[2];
  const float b0 = r.vn[0] - r.f[0], b1 = r.vn[1] - r.f[1], b2 = r.vn[2] - r.f[2];
  const float n0 = a1 * b2 - a2 * b1, n1 = a2 * b0 - a0 * b2, n2 = a0 * b1 - a1 * b0;
  const float nn = sqrtf(n0 * n0 + n1 * n1 + n2 * n2);
  const float dd = fabsf(n0 * (r.pr[0] - r.f[0]) + n1 * (r.pr[1] - r.f[1]) + n2 * (r.pr[2] - r.f[2]));
  float dmin = r.on ? (nn > 0.f ? dd / nn : 0.f) : 3.0e38f;
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) dmin = fminf(dmin, __shfl_xor(dmin, o, 64));
  const float size = R[1].w;  // the largest distance from the vertex mean to a face centroid
  const float pc[3] = {(float)p[0], (float)p[1], (float)p[2]};
  const double s0 = p[0] - (double)pc[0], s1 = p[1] - (double)pc[1], s2 = p[2] - (double)pc[2];
  const double rad = (double)dmin * (1.0 - 1e-6) - 1e-4 * (double)size - sqrt(s0 * s0 + s1 * s1 + s2 * s2);
  return make_float4(pc[0], pc[1], pc[2], rad > 0 ? (float)rad : 0.f);
}
// A point on the inner side of every boundary triangle's plane is strictly inside the cell: from a point
// outside the cell (or on its boundary), a segment to an interior point enters the cell through some
// boundary triangle, so that point lies on the outer side of (or on) the triangle's plane.  Accepts p when
// the smallest signed distance exceeds 1e-4 of the cell's size (the FP32 rounding of the planes, of p - a
// and of the sums is below 1e-6 of it), and gives the ball about p (centre rounded to FP32) that stays
// inside: radius = that distance less the margin and the centre's rounding.  A point inside but not this
// far from every plane (near the boundary, or beside a reflex crease of a non-convex cell) is left to the
// fan test.
// A group of LANES lanes (a power of two) deals the planes out.
template <int LANES>
__device__ __forceinline__ bool plane_ball(const double *p, const float4 *R, const float4 *PL, float4 &ball) {
  const int c = (int)(threadIdx.x & (LANES - 1));
  const float4 h = R[0];
  const float size = R[1].w;
  const float pr0 = (float)(p[0] - (double)h.y), pr1 = (float)(p[1] - (double)h.z), pr2 = (float)(p[2] - (double)h.w);
  float smin = 3.0e38f;
#pragma unroll
  for (int k = 0; k < (kPl + LANES - 1) / LANES; ++k) {
    const int i = k * LANES + c;
    const float4 q = PL[i < kPl ? i : 0];
    smin = fminf(smin, fmaf(q.x, pr0, fmaf(q.y, pr1, fmaf(q.z, pr2, -q.w))));
  }
#pragma unroll
  for (int o = 1; o < LANES; o <<= 1) smin = fminf(smin, __shfl_xor(smin, o, 64));
  if (!(smin > 1e-4f * size)) return false;
  const float pc[3] = {(float)p[0], (float)p[1], (float)p[2]};
  const double s0 = p[0] - (double)pc[0], s1 = p[1] - (double)pc[1], s2 = p[2] - (double)pc[2];
  const double r = (double)smin * (1.0 - 1e-6) - 1e-4 * (double)size - sqrt(s0 * s0 + s1 * s1 + s2 * s2);
  ball = make_float4(pc[0], pc[1], pc[2], r > 0 ? (float)r : 0.f);
  return true;
}

// Locate each molecule: cell_of[i] = sorted index of the cell that contains x_i, in two kernels so that
// the rare slow cases do not hold up whole waves.
// k_locate_fast visits molecules in the order trav (the previous binning's sorted order, so that neighbouring threads
// read neighbouring cell records), MPB per block, in three phases over lists in LDS: a molecule still inside the ball
// kept from its last record test is in its previous cell (hint), one lane each; the others take the plane test of that
// cell, eight lanes each; what it does not accept takes the FP32 fan of that cell, then both tests of the cell across
// the face most likely crossed, 32 lanes each (a molecule that a record shows strictly inside a cell is in no other);
// every other molecule goes to a list.  What bounds the record tests is the latency of their loads: with one lane per
// molecule (24 planes and up to 24 tetrahedra in turn) this kernel took 39 us on 864 molecules and 0.68 ms on 6.7
// million, in this form 10 us and 0.37 ms (0.54 with an atomic per molecule that stays in its ball).  k_locate_slow takes the list, a group of lanes per molecule: the FP64
// previous-cell test and the cells across the previous cell's faces (a molecule that left its cell has crossed one of
// them: the paper's membership tracking), each accepted only when the point is strictly inside; then
// every cell whose padded box holds the point, in ascending mesh cell id (the lowest containing cell wins
// a tie on a shared face, edge or vertex).  Without FP32 records (a cell too large for the fixed stride)
// or without a previous binning every molecule takes the slow path.
// Both kernels index their state by t, the molecule's slot in the previous binning's sorted order
// (trav[t] = its caller index, hint[t] = its previous cell; without a previous binning t is the
// caller index and there is no hint), so that only the positions are read out of order.
constexpr int kRouteSlots = 64;
// Molecules per block.  256 fill the block's lanes in every phase; up to two such blocks per CU (131,072 molecules) 32
// give each CU more of the record tests' loads in flight.  A binning (device time) with 32 / 256: 13,440 molecules 51 /
// 58 us, 100,000 77 / 80, 60,001 in cells of a hundred 97 / 88, 219,488 92 / 86, 371,896 117 / 99.
constexpr int kMpb = 256, kMpbFew = 32;
constexpr int64_t kFewMolecules = 131072;

template <typename PT, int MPB>
__global__ __launch_bounds__(256) void k_locate_fast(
    const PT *__restrict__ pos, int64_t n, const int32_t *__restrict__ trav, const int32_t *__restrict__ hint,
    const float4 *__restrict__ rec32, const float4 *__restrict__ pl32, float4 *__restrict__ ref,
    int32_t *__restrict__ cell_t, int32_t *__restrict__ rank_t, int32_t *__restrict__ count,
    unsigned long long *__restrict__ nslow, int32_t *__restrict__ slow, unsigned long long *__restrict__ routes) {
  // molecules (relative to the block's first) for the plane test, for the fan, and for the slow kernel
  __shared__ int32_t plane_l[MPB], fan_l[MPB], slow_l[MPB];
  __shared__ int32_t np, nf, ns, nrec;
  __shared__ unsigned long long start;
  const int tid = (int)threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * MPB;
  if (tid == 0) np = nf = ns = nrec = 0;
  __syncthreads();
  auto take = [&](int64_t t, int64_t i, int32_t c, const float4 &ball) {
    ref[i] = ball;
    cell_t[t] = c;
    rank_t[t] = atomicAdd(&count[c], 1);
  };
  // ---- the ball test
#pragma unroll
  for (int k = 0; k < (MPB + 255) / 256; ++k) {
    const int off = k * 256 + tid;
    const int64_t t = base + off;
    int32_t h0 = -1;
    bool stay = false;
    if ((MPB >= 256 || off < MPB) && t < n) {
      const int64_t i = trav ? trav[t] : t;
      const double p[3] = {(double)pos[3 * i], (double)pos[3 * i + 1], (double)pos[3 * i + 2]};
      if (hint) h0 = hint[t];
      bool rec = false;
      if (h0 >= 0 && isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2])) {
        // still inside the ball found inside this cell when it was last tested: no record needed
        const float4 b = ref[i];
        const double e0 = p[0] - (double)b.x, e1 = p[1] - (double)b.y, e2 = p[2] - (double)b.z;
        stay = b.w > 0.f && e0 * e0 + e1 * e1 + e2 * e2 < (double)b.w * (double)b.w;
        rec = !stay && rec32;
      }
      if (stay) cell_t[t] = h0;
      else if (rec) plane_l[atomicAdd(&np, 1)] = off;
      else slow_l[atomicAdd(&ns, 1)] = off;
    }
    // the molecules that stay are counted a run of neighbouring lanes with one previous cell at a time
    const int lane = tid & 63;
    const int32_t hp = __shfl_up(h0, 1, 64);
    const unsigned long long upto = ~0ull >> (63 - lane), heads = __builtin_amdgcn_ballot_w64(lane == 0 || hp != h0);
    const int first = 63 - __builtin_clzll(heads & upto);
    const unsigned long long after = heads & ~upto;
    const unsigned long long run = (after ? (1ull << __builtin_ctzll(after)) - 1 : ~0ull) & (~0ull << first) &
                                   __builtin_amdgcn_ballot_w64(stay);
    const int lead = run ? (int)__builtin_ctzll(run) : lane;
    int32_t place = 0;
    if (stay && lane == lead) place = atomicAdd(&count[h0], (int32_t)__builtin_popcountll(run));
    place = __shfl(place, lead, 64);
    if (stay) rank_t[t] = place + (int32_t)__builtin_popcountll(run & (upto >> 1));
  }
  __syncthreads();
  // ---- the plane test of the previous cell, eight lanes per molecule (the group's lanes stay together)
  for (int k = tid >> 3; k < np; k += 32) {
    const int off = plane_l[k];
    const int64_t t = base + off;
    const int64_t i = trav[t];
    const double p[3] = {(double)pos[3 * i], (double)pos[3 * i + 1], (double)pos[3 * i + 2]};
    const int32_t h0 = hint[t];
    float4 ball;
    const bool in = plane_ball<8>(p, rec32 + (int64_t)kR32 * h0, pl32 + (int64_t)kPl * h0, ball);
    if ((tid & 7) == 0) {
      if (in) {
        take(t, i, h0, ball);
        atomicAdd(&nrec, 1);
      } else {
        fan_l[atomicAdd(&nf, 1)] = off;
      }
    }
  }
  __syncthreads();
  // ---- the fan of the previous cell, then the cell across the face most likely crossed, 32 lanes per molecule
  for (int k = tid >> 5; k < nf; k += 8) {
    const int off = fan_l[k];
    const int64_t t = base + off;
    const int64_t i = trav[t];
    const double p[3] = {(double)pos[3 * i], (double)pos[3 * i + 1], (double)pos[3 * i + 2]};
    const int32_t h0 = hint[t];
    const float4 *R = rec32 + (int64_t)kR32 * h0;
    int32_t found = -1;
    float4 ball;
    const RecLane r = load_rec32(p, R);
    if (rec_lanes_inside(r)) {
      found = h0;
      ball = rec_lanes_ball(r, p, R);
    } else if (r.across >= 0) {
      const float4 *Ra = rec32 + (int64_t)kR32 * r.across;
      if (plane_ball<32>(p, Ra, pl32 + (int64_t)kPl * r.across, ball)) {
        found = r.across;
      } else {
        const RecLane ra = load_rec32(p, Ra);
        if (rec_lanes_inside(ra)) {
          found = r.across;
          ball = rec_lanes_ball(ra, p, Ra);
        }
      }
    }
    if ((tid & 31) == 0) {
      if (found >= 0) {
        take(t, i, found, ball);
        atomicAdd(&nrec, 1);
      } else {
        slow_l[atomicAdd(&ns, 1)] = off;
      }
    }
  }
  __syncthreads();
  // ---- the block's share of the slow list (one atomic), and of the route counters (spread over kRouteSlots addresses
  // so that the blocks do not queue on one)
  if (ns > 0) {
    if (tid == 0) start = atomicAdd(nslow, (unsigned long long)ns);
    __syncthreads();
    for (int b = tid; b < ns; b += 256) slow[start + b] = (int32_t)(base + slow_l[b]);
  }
  if (tid == 0 && nrec > 0) atomicAdd(routes + blockIdx.x % kRouteSlots, (unsigned long long)nrec);
}

// The slow path for one molecule at p with previous cell h0 (-1: none), by a group of 32 lanes.  The previous cell
// and the cells across its faces, each accepted only when p is strictly inside (so at most one accepts), then the
// cells of the background bin whose padded box holds p, in ascending mesh cell id, the first containing one.  The
// lanes test 32 boxes at a time and then the tetrahedra of one cell, three loads deep: what bounds the kernel is the
// chain of loads of its longest molecule.  Cells by lane, one tetrahedron after another, it took 45 to 65 us for the
// few hundred molecules of a step of 13,440 to 100,000, and a first binning of 371,896 1.1 ms (now 0.65), of 6.7
// million 15.8 ms (10.1).
__device__ int32_t slow_find(const double *p, int32_t h0, const int64_t *__restrict__ rec_off,
                             const double *__restrict__ rec, const int64_t *__restrict__ nbr_off,
                             const int32_t *__restrict__ nbr, const double *__restrict__ bb,
                             const int64_t *__restrict__ gb_off, const int32_t *__restrict__ gb_cell, double glo0,
                             double glo1, double glo2, double gh, int64_t nb0, int64_t nb1, int64_t nb2) {
  const int lane = (int)(threadIdx.x & 31), g0 = (int)(threadIdx.x & 32);
  // the first of cand[b .. e) (in order) whose box holds p and whose tetrahedra do, with tolerance tau
  auto first_of = [&](const int32_t *cand, int64_t b, int64_t e, double tau) -> int32_t {
    for (int64_t k = b; k < e; k += 32) {
      int32_t c = -1;
      bool box = false;
      if (k + lane < e) {
        c = cand[k + lane];
        const double *B = bb + 6 * (int64_t)c;
        box = !(p[0] < B[0] || p[1] < B[1] || p[2] < B[2] || p[0] > B[3] || p[1] > B[4] || p[2] > B[5]);
      }
      unsigned hits = (unsigned)(__builtin_amdgcn_ballot_w64(box) >> g0);
      while (hits) {
        const int32_t d = __shfl(c, g0 + __builtin_ctz(hits), 64);
        if (point_in_rec(p, rec + rec_off[d], tau)) return d;
        hits &= hits - 1;
      }
    }
    return -1;
  };
  if (h0 >= 0) {
    if (point_in_rec(p, rec + rec_off[h0], -1e-9)) return h0;
    const int32_t c = first_of(nbr, nbr_off[h0], nbr_off[h0 + 1], -1e-9);
    if (c >= 0) return c;
  }
  const double f0 = floor((p[0] - glo0) / gh), f1 = floor((p[1] - glo1) / gh), f2 = floor((p[2] - glo2) / gh);
  if (!(f0 >= 0 && f1 >= 0 && f2 >= 0 && f0 < (double)nb0 && f1 < (double)nb1 && f2 < (double)nb2)) return -1;
  const int64_t bin = (int64_t)f0 + nb0 * ((int64_t)f1 + nb1 * (int64_t)f2);
  return first_of(gb_cell, gb_off[bin], gb_off[bin + 1], 1e-12);
}

// The slow kernel, two molecules per wave (at the first binning every molecule comes here).  A fixed grid strides over
// the list, whose length is only known on the device; a short list is spread over the waves first.
template <typename PT>
__global__ __launch_bounds__(256) void k_locate_slow(
    const PT *__restrict__ pos, const unsigned long long *__restrict__ nslow, const int32_t *__restrict__ slow,
    const int32_t *__restrict__ trav, const int32_t *__restrict__ hint, const float4 *__restrict__ rec32,
    const float4 *__restrict__ pl32, const int64_t *__restrict__ rec_off, const double *__restrict__ rec,
    const int64_t *__restrict__ nbr_off,
    const int32_t *__restrict__ nbr, const double *__restrict__ bb, const int64_t *__restrict__ gb_off,
    const int32_t *__restrict__ gb_cell, double glo0, double glo1, double glo2, double gh, int64_t nb0, int64_t nb1,
    int64_t nb2, float4 *__restrict__ ref, int32_t *__restrict__ cell_t, int32_t *__restrict__ rank_t,
    int32_t *__restrict__ count, unsigned long long *__restrict__ status) {
  const int64_t ns = (int64_t)*nslow;
  const int64_t nw = (int64_t)gridDim.x * 4, wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  for (int64_t u = wave + (threadIdx.x & 32 ? nw : 0); u < ns; u += 2 * nw) {  // uniform in each half wave
    const int64_t t = slow[u];
    const int64_t i = trav ? trav[t] : t;
    const double p[3] = {(double)pos[3 * i], (double)pos[3 * i + 1], (double)pos[3 * i + 2]};
    int32_t found = -1;
    if (isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]))
      found = slow_find(p, hint ? hint[t] : -1, rec_off, rec, nbr_off, nbr, bb, gb_off, gb_cell, glo0, glo1, glo2, gh, nb0,
                        nb1, nb2);
    // the ball about p inside the cell found, when the plane test shows p that far inside; else no ball
    // until the next record test in this cell
    float4 ball = make_float4(0.f, 0.f, 0.f, 0.f);
    if (found >= 0 && pl32) {
      float4 b;
      if (plane_ball<32>(p, rec32 + (int64_t)kR32 * found, pl32 + (int64_t)kPl * found, b)) ball = b;
    }
    if ((threadIdx.x & 31) == 0) {
      cell_t[t] = found;
      ref[i] = ball;
      if (found < 0)
        atomicAdd(status, 1ull);
      else
        rank_t[t] = atomicAdd(&count[found], 1);
    }
  }
}


// ---- exclusive scans over the cells: occupancy -> cell_start, and occupancy x reaction slots per molecule -> slot_base
// (HALF: the steps whose FP32 forces take the half lists; otherwise only its total).  out[n] = total.

constexpr int kScanThreads = 1024, kScanItems = 4, kScanTile = kScanThreads * kScanItems;

template <typename OutT>
__device__ OutT block_exclusive_scan(OutT v, OutT *sh, OutT &total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  OutT x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    OutT y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[w] = x;
  __syncthreads();
  if (w == 0) {
    OutT s = lane < (kScanThreads / 64) ? sh[lane] : 0;
    OutT t = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      OutT y = __shfl_up(t, o, 64);
      if (lane >= o) t += y;
    }
    if (lane < kScanThreads / 64) sh[lane] = t - s;
    if (lane == kScanThreads / 64 - 1) sh[kScanThreads / 64] = t;
  }
  __syncthreads();
  total = sh[kScanThreads / 64];
  OutT r = x - v + sh[w];
  __syncthreads();
  return r;
}

// What bounds a small system's binning is its launches (2.5 to 5 us each): both scans are one pass over the cells and,
// up to kScanDirect cells, one launch.
// One tile of kScanTile cells: its offsets and totals.
template <bool HALF>
__device__ __forceinline__ void scan_tile(const int32_t *count, const int32_t *rcnt, int64_t n, int64_t tile,
                                          int32_t *cell_start, int64_t *slot_base, int32_t &ctot, int64_t &stot) {
  __shared__ int32_t shc[kScanThreads / 64 + 1];
  __shared__ int64_t shs[kScanThreads / 64 + 1];
  const int64_t base = tile * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int32_t v[kScanItems], c = 0;
  int64_t x[kScanItems], sl = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? count[base + k] : 0;
    x[k] = base + k < n ? (int64_t)v[k] * rcnt[base + k] : 0;
    c += v[k];
    sl += x[k];
  }
  int32_t ec = block_exclusive_scan<int32_t>(c, shc, ctot);
  int64_t es = block_exclusive_scan<int64_t>(sl, shs, stot);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) {
      cell_start[base + k] = ec;
      if (HALF) slot_base[base + k] = es;
    }
    ec += v[k];
    es += x[k];
  }
}
// Few cells: one block, a run of consecutive cells per thread, read twice (its total, then its offsets).  The loads of a
// run are all in flight at once: tile after tile, 13,824 cells took 20 us.
template <bool HALF>
__global__ __launch_bounds__(kScanThreads) void k_scan_cells(const int32_t *__restrict__ count,
                                                              const int32_t *__restrict__ rcnt, int64_t n,
                                                              int32_t *__restrict__ cell_start,
                                                              int64_t *__restrict__ slot_base,
                                                              unsigned long long *__restrict__ slots) {
  __shared__ int32_t shc[kScanThreads / 64 + 1];
  __shared__ int64_t shs[kScanThreads / 64 + 1];
  const int64_t per = ((n + kScanThreads - 1) / kScanThreads + 3) & ~(int64_t)3;  // whole int4
  const int64_t b = min(n, per * threadIdx.x), e = min(n, b + per);
  int32_t c = 0, ct;
  int64_t s = 0, st;
  auto each = [&](auto &&f) {
    int64_t k = b;
#pragma unroll 4
    for (; k + 4 <= e; k += 4) {
      const int4 v = *reinterpret_cast<const int4 *>(count + k), r = *reinterpret_cast<const int4 *>(rcnt + k);
      f(k, v.x, r.x);
      f(k + 1, v.y, r.y);
      f(k + 2, v.z, r.z);
      f(k + 3, v.w, r.w);
    }
    for (; k < e; ++k) f(k, count[k], rcnt[k]);
  };
  each([&](int64_t, int32_t v, int32_t r) {
    c += v;
    s += (int64_t)v * r;
  });
  c = block_exclusive_scan<int32_t>(c, shc, ct);
  s = block_exclusive_scan<int64_t>(s, shs, st);
  each([&](int64_t k, int32_t v, int32_t r) {
    cell_start[k] = c;
    if (HALF) slot_base[k] = s;
    c += v;
    s += (int64_t)v * r;
  });
  if (threadIdx.x == 0) {
    cell_start[n] = ct;
    if (HALF) slot_base[n] = st;
    *slots = (unsigned long long)st;
  }
}
// Many tiles: every tile on its own, the tile totals, then the totals before each tile added.
template <bool HALF>
__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const int32_t *count, const int32_t *rcnt, int64_t n,
                                                              int32_t *cell_start, int64_t *slot_base, int64_t *tile_sum) {
  int32_t ct;
  int64_t st;
  scan_tile<HALF>(count, rcnt, n, blockIdx.x, cell_start, slot_base, ct, st);
  if (threadIdx.x == 0) {
    tile_sum[2 * (int64_t)blockIdx.x] = ct;
    tile_sum[2 * (int64_t)blockIdx.x + 1] = st;
  }
}
template <bool HALF>
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(int64_t *tile_sum, int64_t ntiles, int64_t n, int32_t *cell_start,
                                                             int64_t *slot_base, unsigned long long *slots) {
  __shared__ int64_t sh[kScanThreads / 64 + 1];
  int64_t carry[2] = {0, 0};
  for (int64_t b = 0; b < ntiles; b += kScanThreads) {
    const int64_t i = b + threadIdx.x;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int64_t v = i < ntiles ? tile_sum[2 * i + k] : 0;
      int64_t total;
      const int64_t ex = block_exclusive_scan<int64_t>(v, sh, total);
      if (i < ntiles) tile_sum[2 * i + k] = ex + carry[k];
      carry[k] += total;
    }
  }
  if (threadIdx.x == 0) {
    cell_start[n] = (int32_t)carry[0];
    if (HALF) slot_base[n] = carry[1];
    *slots = (unsigned long long)carry[1];
  }
}
template <bool HALF>
__global__ void k_scan_add(int64_t n, const int64_t *tile_sum, int32_t *cell_start, int64_t *slot_base) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  cell_start[i] += (int32_t)tile_sum[2 * (i / kScanTile)];
  if (HALF) slot_base[i] += tile_sum[2 * (i / kScanTile) + 1];
}

// rank_t[t]: the place the locate kernels' count took for the molecule inside its cell (any order; the cells are
// sorted by molecule id next).  raw: the molecules by cell; cell_of: their cells.
__global__ void k_scatter(const int32_t *cell_t, const int32_t *trav, int64_t n, const int32_t *cell_start,
                          const int32_t *rank_t, int32_t *raw, int32_t *cell_of) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int32_t c = cell_t[t];
  if (c < 0) return;  // unlocated (an error)
  const int32_t m = cell_start[c] + rank_t[t];
  raw[m] = trav ? trav[t] : (int32_t)t;
  cell_of[m] = c;
}

// Ascending molecule id inside every cell (the locate kernels' counters leave an arbitrary order): every molecule
// counts the smaller ids of its cell.  One thread per molecule: an insertion sort with a thread per cell took
// 1.67 ms on 60,001 molecules in cells of a hundred.
__global__ void k_sort_cells(const int32_t *__restrict__ cell_start, const int32_t *__restrict__ cell_of,
                             const int32_t *__restrict__ raw, int64_t nc, int64_t n, int32_t *__restrict__ perm) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n || m >= cell_start[nc]) return;  // fewer slots than n when some molecule is unlocated
  const int32_t c = cell_of[m], b = cell_start[c], e = cell_start[c + 1], v = raw[m];
  int32_t r = b;
  for (int32_t k = b; k < e; ++k) r += raw[k] < v;
  perm[r] = v;
}

// A binning as the pair kernels read it where they decide a pair close to the cut-off.
struct BinRef {
  const void *pos;         // [n][3] as passed by the caller, double if pos64, else float
  const int32_t *perm;     // caller id of each sorted molecule
  const int32_t *cell_of;  // its sorted cell
  int32_t pos64;
};
// Group frames of the half lists, in which such a pair is decided, written with the lists; bin by every binning.  In
// device memory: as arguments of the pair kernels, the pointers would take scalar registers from their loops.
struct HalfFrames {
  const int32_t *of_cell;   // group of each sorted cell
  const double *orig;       // [groups][3]
  const int64_t *e_off;     // [groups+1] entries, sorted by (j-group, image code)
  const int32_t *e_B;
  const float4 *e_vec32;    // offset and image code of each entry
  const double4 *e_vec64;
  BinRef bin;
};

// At the start of a binning: the cells' occupancies and the status words cleared, the frames' reference to the binning.
__global__ void k_clear_bin(int32_t *count, int64_t nc, unsigned long long *status, int nstatus, HalfFrames *half,
                            BinRef bin) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nc) count[i] = 0;
  if (i < nstatus) status[i] = 0;
  if (i == 0) half->bin = bin;
}

template <typename T>
__global__ void k_fill(T *p, int64_t n, T v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// =====================================================================================================
// kernels: forces

template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
  using type = float4;
};
template <>
struct Vec4<double> {
  using type = double4;
};

// Gather by groups, one wave each: positions in cell-sorted order relative to the group's origin (species id in .w as
// integer bits), and the box of the group's molecules (empty: lo > hi).
template <typename T, typename PT>
__global__ __launch_bounds__(256) void k_gather_groups(const PT *__restrict__ pos, const int32_t *__restrict__ species,
                                                       const int32_t *__restrict__ perm,
                                                       const int32_t *__restrict__ cell_start,
                                                       const int32_t *__restrict__ cell0, const double *__restrict__ orig,
                                                       int64_t ng, int nsp, typename Vec4<T>::type *__restrict__ out,
                                                       T *__restrict__ box, const T *__restrict__ G,
                                                       typename Vec4<T>::type *__restrict__ gout) {
  const int lane = threadIdx.x & 63;
  const int64_t a = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (a >= ng) return;
  const int32_t m0 = cell_start[cell0[a]], m1 = cell_start[cell0[a + 1]];
  const double o[3] = {orig[3 * a], orig[3 * a + 1], orig[3 * a + 2]};
  T lo[3] = {(T)1e30, (T)1e30, (T)1e30}, hi[3] = {(T)-1e30, (T)-1e30, (T)-1e30};
  for (int32_t m = m0 + lane; m < m1; m += 64) {
    const int64_t id = perm[m];
    T x[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      x[k] = (T)((double)pos[3 * id + k] - o[k]);
      lo[k] = min(lo[k], x[k]);
      hi[k] = max(hi[k], x[k]);
    }
    const int32_t t = species ? min(max(species[id], 0), nsp - 1) : 0;  // out-of-range ids are clamped
    typename Vec4<T>::type v;
    v.x = x[0];
    v.y = x[1];
    v.z = x[2];
    if constexpr (sizeof(T) == 4)
      v.w = __builtin_bit_cast(float, t);
    else
      v.w = __builtin_bit_cast(double, (int64_t)t);
    out[m] = v;
    if (G) {  // the adjoint's upstream gradient
      v.x = G[3 * id];
      v.y = G[3 * id + 1];
      v.z = G[3 * id + 2];
      v.w = (T)0;
      gout[m] = v;
    }
  }
  if (!box) return;
#pragma unroll
  for (int s = 1; s < 64; s <<= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lo[k] = min(lo[k], __shfl_xor(lo[k], s, 64));
      hi[k] = max(hi[k], __shfl_xor(hi[k], s, 64));
    }
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      box[6 * a + k] = lo[k];
      box[6 * a + 3 + k] = hi[k];
    }
}

struct LJTab {
  float sig2[64], e24[64], e4[64];
  double sig2d[64], e24d[64], e4d[64];
  float rc2, band;
  float rc2lo, rc2hi;  // rc^2 -+ band: an FP32 s below rc2lo is surely inside, at or above rc2hi surely outside
  double rc2d;
  // rc^2 -+ the most that a full list's square of a pair can differ by from the half lists' (rounding of positions in, and
  // of offsets between, the group frames of either, and of the square): in between, the half lists' decision is taken
  float near_lo, near_hi;
  double near_lod, near_hid;
  // radius^2 within which the full lists' box test and search keep every pair: rc^2, or near_hi less what those allow anyway
  double reach2, reach2d;
  int nsp;
};
template <typename T>
__device__ __forceinline__ double reach2(const LJTab &t) {
  if constexpr (sizeof(T) == 4) return t.reach2; else return t.reach2d;
}
template <typename T>
__device__ __forceinline__ T near_lo(const LJTab &t) {
  if constexpr (sizeof(T) == 4) return t.near_lo; else return t.near_lod;
}
template <typename T>
__device__ __forceinline__ T near_hi(const LJTab &t) {
  if constexpr (sizeof(T) == 4) return t.near_hi; else return t.near_hid;
}

template <typename T>
__device__ __forceinline__ int type_of(T w) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(int, w);
  else
    return (int)__builtin_bit_cast(int64_t, w);
}

template <typename T>
__device__ __forceinline__ T tab_sig2(const LJTab &t, int k) {
  if constexpr (sizeof(T) == 4) return t.sig2[k]; else return t.sig2d[k];
}
template <typename T>
__device__ __forceinline__ T tab_e24(const LJTab &t, int k) {
  if constexpr (sizeof(T) == 4) return t.e24[k]; else return t.e24d[k];
}
template <typename T>
__device__ __forceinline__ T tab_e4(const LJTab &t, int k) {
  if constexpr (sizeof(T) == 4) return t.e4[k]; else return t.e4d[k];
}

// Per-lane Lennard-Jones parameters of the lane's i-species against j-species 0 and 1 (MIX <= 1),
// or the full table (MIX == 2: looked up per pair).
template <typename T, int MIX>
struct LaneLJ {
  T s0, s1, g0, g1, u0, u1;
  int ti;
  // One or two species: the parameters are selected from kernel-argument values (no per-lane
  // memory access, which would otherwise be waited for inside the pair loops).
  __device__ __forceinline__ void init(const LJTab &t, int ti_) {
    ti = ti_;
    if (MIX == 0) {
      s0 = tab_sig2<T>(t, 0);
      g0 = tab_e24<T>(t, 0);
      u0 = tab_e4<T>(t, 0);
    } else if (MIX == 1) {
      const bool b = ti != 0;
      s0 = b ? tab_sig2<T>(t, 8) : tab_sig2<T>(t, 0);
      g0 = b ? tab_e24<T>(t, 8) : tab_e24<T>(t, 0);
      u0 = b ? tab_e4<T>(t, 8) : tab_e4<T>(t, 0);
      s1 = b ? tab_sig2<T>(t, 9) : tab_sig2<T>(t, 1);
      g1 = b ? tab_e24<T>(t, 9) : tab_e24<T>(t, 1);
      u1 = b ? tab_e4<T>(t, 9) : tab_e4<T>(t, 1);
    } else {
      s0 = tab_sig2<T>(t, ti * 8);
      g0 = tab_e24<T>(t, ti * 8);
      u0 = tab_e4<T>(t, ti * 8);
    }
  }
  __device__ __forceinline__ void get(const LJTab &t, int tj, T &sig2, T &e24, T &e4) const {
    if (MIX == 0) {
      sig2 = s0;
      e24 = g0;
      e4 = u0;
    } else if (MIX == 1) {
      const bool b = tj != 0;
      sig2 = b ? s1 : s0;
      e24 = b ? g1 : g0;
      e4 = b ? u1 : u0;
    } else {
      const int k = ti * 8 + tj;
      sig2 = tab_sig2<T>(t, k);
      e24 = tab_e24<T>(t, k);
      e4 = tab_e4<T>(t, k);
    }
  }
};

__device__ __forceinline__ float fast_rcp(float s) { return __builtin_amdgcn_rcpf(s); }
// FP64: the hardware reciprocal refined by two Newton steps (about 1 ulp, against the ten instructions of
// a correctly rounded division; the FP64 path's bar is 1e-12 of the result)
__device__ __forceinline__ double fast_rcp(double s) {
  double r = __builtin_amdgcn_rcp(s);
  r = fma(r, fma(-s, r, 1.0), r);
  return fma(r, fma(-s, r, 1.0), r);
}

template <typename T>
__device__ __forceinline__ T far_i() { return (T)1e15; }
template <typename T>
__device__ __forceinline__ T far_j() { return (T)-1e15; }

}  // namespace

#include "aica_pair.inc"
#include "aica_neigh.inc"

namespace {

// Deterministic reductions of per-group partials (rows of doubles, or of unsigned integers read as doubles: integer
// sums stay exact below 2^53), always in a fixed order.  Up to kRedDirect rows one block sums them at once; more
// rows go through stage-1 rows, one per block over a fixed range, which the last block's kernel sums in block order.
// Each launch costs about 5 us here whatever it does, so the rows of several arrays share one.
constexpr int kRedBlocks = 512, kRedThreads = 256;
constexpr int64_t kRedDirect = 4096;

// Column sums of rows r0 .. r1 - 1 by the whole block, in out[K] of every thread.
template <int K, typename F>
__device__ void block_sum_rows(int64_t r0, int64_t r1, double *out, F row) {
  __shared__ double sh[kRedThreads / 64][K];
  double acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = 0;
  for (int64_t r = r0 + threadIdx.x; r < r1; r += kRedThreads) {
    double v[K];
    row(r, v);
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] += v[k];
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1)
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] += __shfl_xor(acc[k], o, 64);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < K; ++k) sh[threadIdx.x >> 6][k] = acc[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    out[k] = sh[0][k];
    for (int w = 1; w < kRedThreads / 64; ++w) out[k] += sh[w][k];
  }
}

// U, W and the pair count: rows (U, W) of gpart and the first column of gnp.
__device__ __forceinline__ void uw_row(const double *gpart, const unsigned long long *gnp, int64_t r, double *v) {
  v[0] = gpart[2 * r];
  v[1] = gpart[2 * r + 1];
  v[2] = (double)gnp[2 * r];
}
__global__ __launch_bounds__(kRedThreads) void k_reduce_uw_rows(const double *gpart, const unsigned long long *gnp,
                                                                 int64_t ng, int64_t chunk, double *part) {
  double v[3];
  block_sum_rows<3>(blockIdx.x * chunk, std::min<int64_t>(ng, (blockIdx.x + 1) * chunk), v,
                    [&](int64_t r, double *x) { uw_row(gpart, gnp, r, x); });
  if (threadIdx.x < 3) part[3 * (int64_t)blockIdx.x + threadIdx.x] = v[threadIdx.x];
}
// sides: how often each pair was counted.
__global__ __launch_bounds__(kRedThreads) void k_reduce_uw(const double *gpart, const unsigned long long *gnp, int64_t ng,
                                                            const double *part, int nb, double *uw, int64_t *npairs,
                                                            int sides) {
  double v[3];
  if (nb > 0)
    block_sum_rows<3>(0, nb, v, [&](int64_t r, double *x) {
#pragma unroll
      for (int k = 0; k < 3; ++k) x[k] = part[3 * r + k];
    });
  else
    block_sum_rows<3>(0, ng, v, [&](int64_t r, double *x) { uw_row(gpart, gnp, r, x); });
  if (threadIdx.x == 0) {
    if (uw) {
      uw[0] = v[0];
      uw[1] = v[1];
    }
    if (npairs) npairs[0] = (int64_t)v[2] / sides;
  }
}

// Stage-1 blocks (0: the rows are few enough for one block) and the rows of each.
inline int red_blocks(int64_t ng, int64_t &chunk) {
  chunk = ng;
  if (ng <= kRedDirect) return 0;
  const int nb = (int)std::min<int64_t>(kRedBlocks, (ng + kRedThreads - 1) / kRedThreads);
  chunk = (ng + nb - 1) / nb;
  return nb;
}

inline unsigned grid1d(int64_t n, int b) { return (unsigned)std::max<int64_t>(1, (n + b - 1) / b); }

// cell_start, slot_base (half) and the number of reaction slots from the cells' occupancies.
// One block up to 16,384 cells: a binning with 4,225 cells took 48 us with one launch and 55 with three, with 13,824
// cells 57 either way, with 67,240 143 and 77.
constexpr int64_t kScanDirect = 4 * kScanTile;
int scan_cells(aica_dil *h, int64_t nc, bool half, unsigned long long *slots, hipStream_t st) {
  const int64_t ntiles = std::max<int64_t>(1, (nc + kScanTile - 1) / kScanTile);
  const int32_t *count = h->d_count.as<int32_t>(), *rcnt = h->d_rcnt.as<int32_t>();
  int32_t *cs = h->d_cell_start.as<int32_t>();
  int64_t *sb = h->d_slot_base.as<int64_t>();
  if (nc <= kScanDirect) {
    hipLaunchKernelGGL(half ? k_scan_cells<true> : k_scan_cells<false>, dim3(1), dim3(kScanThreads), 0, st, count, rcnt, nc,
                       cs, sb, slots);
  } else {
    int rc = h->d_scan_tmp.ensure(sizeof(int64_t) * 2 * ntiles);
    if (rc) return rc;
    int64_t *ts = h->d_scan_tmp.as<int64_t>();
    hipLaunchKernelGGL(half ? k_scan_tiles<true> : k_scan_tiles<false>, dim3((unsigned)ntiles), dim3(kScanThreads), 0, st,
                       count, rcnt, nc, cs, sb, ts);
    hipLaunchKernelGGL(half ? k_scan_sums<true> : k_scan_sums<false>, dim3(1), dim3(kScanThreads), 0, st, ts, ntiles, nc, cs,
                       sb, slots);
    hipLaunchKernelGGL(half ? k_scan_add<true> : k_scan_add<false>, dim3(grid1d(nc, 256)), dim3(256), 0, st, nc,
                       (const int64_t *)ts, cs, sb);
  }
  HIPCHK(hipGetLastError());
  return AICA_OK;
}

struct ProfScope {
  aica_dil *h;
  const char *name;
  hipStream_t st;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  ProfScope(aica_dil *h_, const char *n, hipStream_t s) : h(h_), name(n), st(s) {
    if (h->profiling) {
      (void)hipEventCreate(&e0);
      (void)hipEventCreate(&e1);
      (void)hipEventRecord(e0, st);
    }
  }
  ~ProfScope() {
    if (h->profiling && e0) {
      (void)hipEventRecord(e1, st);
      h->timers[name].pending.push_back({e0, e1});
      h->timers[name].launches++;
    }
  }
};

}  // namespace

// =====================================================================================================
// setup helpers

static int upload_geometry(aica_dil *h) {
  const Geometry &g = h->geo;
  int rc;
  // cell records for point location, in sorted cell order (layout described at point_in_rec)
  {
    std::vector<int64_t> roff(g.nc + 1, 0);
    for (int64_t s = 0; s < g.nc; ++s) {
      const int64_t c = h->order[s];
      int64_t sz = 4;
      for (int64_t k = g.cf_off[c]; k < g.cf_off[c + 1]; ++k) {
        const int32_t f = g.cf[k];
        sz += 4 + 3 * (g.foff[f + 1] - g.foff[f]);
      }
      roff[s + 1] = roff[s] + sz;
    }
    std::vector<double> rec(roff[g.nc]);
    parallel_for(g.nc, [&](int64_t s0, int64_t s1, int) {
      for (int64_t s = s0; s < s1; ++s) {
        const int64_t c = h->order[s];
        const int64_t nf = g.cf_off[c + 1] - g.cf_off[c];
        double *R = rec.data() + roff[s];
        R[0] = (double)nf;
        for (int q = 0; q < 3; ++q) R[1 + q] = g.ccen[3 * c + q];
        double *FC = R + 4, *LEN = FC + 3 * nf, *V = LEN + nf;
        for (int64_t k = 0; k < nf; ++k) {
          const int32_t f = g.cf[g.cf_off[c] + k];
          const int64_t b0 = g.foff[f], len = g.foff[f + 1] - b0;
          const bool rev = g.cf_sgn[g.cf_off[c] + k] < 0;  // the neighbour side walks the loop backwards
          for (int q = 0; q < 3; ++q) FC[3 * k + q] = g.fcen[3 * (int64_t)f + q];
          LEN[k] = (double)len;
          for (int64_t j = 0; j < len; ++j) {
            const int64_t jj = rev ? (len - j) % len : j;
            for (int q = 0; q < 3; ++q) V[3 * j + q] = g.pts[3 * (int64_t)g.fpts[b0 + jj] + q];
          }
          V += 3 * len;
        }
      }
    });
    if ((rc = upload(h->d_rec_off, roff))) return rc;
    if ((rc = upload(h->d_rec, rec))) return rc;
    // FP32 records (layout at kR32), when every cell fits the fixed stride
    bool fits = true;
    for (int64_t s = 0; s < g.nc && fits; ++s) {
      const double *R = rec.data() + roff[s];
      const int64_t nf = (int64_t)R[0];
      int64_t nv = 0;
      for (int64_t k = 0; k < nf; ++k) nv += (int64_t)R[4 + 3 * nf + k];
      fits = 2 + nf + nv <= kR32;
    }
    h->has_rec32 = fits;
    if (fits) {
      std::vector<float4> r32((size_t)g.nc * kR32), pl32((size_t)g.nc * kPl);
      parallel_for(g.nc, [&](int64_t s0, int64_t s1, int) {
        for (int64_t s = s0; s < s1; ++s) {
          const double *R = rec.data() + roff[s];
          const int64_t nf = (int64_t)R[0];
          float4 *O = r32.data() + (size_t)s * kR32;
          const double a[3] = {(double)(float)R[1], (double)(float)R[2], (double)(float)R[3]};
          const double *FC = R + 4, *LEN = FC + 3 * nf, *V = LEN + nf;
          // the cell's size: the largest distance from the vertex mean to a face centroid
          double size = 0;
          for (int64_t k = 0; k < nf; ++k) {
            const double e0 = FC[3 * k] - R[1], e1 = FC[3 * k + 1] - R[2], e2 = FC[3 * k + 2] - R[3];
            size = std::max(size, std::sqrt(e0 * e0 + e1 * e1 + e2 * e2));
          }
          O[0] = make_float4((float)nf, (float)a[0], (float)a[1], (float)a[2]);
          O[1] = make_float4((float)(R[1] - a[0]), (float)(R[2] - a[1]), (float)(R[3] - a[2]), (float)size);
          // plane records (layout at plane_ball): the face loops run with the right-hand normal out of the cell
          float4 *PL = pl32.data() + (size_t)s * kPl;
          for (int k = 0; k < kPl; ++k) PL[k] = make_float4(0.f, 0.f, 0.f, -3.0e38f);
          {
            int ntri = 0;
            const double *Vk = V;
            for (int64_t k = 0; k < nf; ++k) {
              const int64_t len = (int64_t)LEN[k];
              const double *f = FC + 3 * k;
              for (int64_t j = 0; j < len; ++j) {
                const double *v0 = Vk + 3 * j, *v1 = Vk + 3 * ((j + 1) % len);
                const double u[3] = {v0[0] - f[0], v0[1] - f[1], v0[2] - f[2]};
                const double w[3] = {v1[0] - f[0], v1[1] - f[1], v1[2] - f[2]};
                double nrm[3] = {-(u[1] * w[2] - u[2] * w[1]), -(u[2] * w[0] - u[0] * w[2]), -(u[0] * w[1] - u[1] * w[0])};
                const double nn = std::sqrt(nrm[0] * nrm[0] + nrm[1] * nrm[1] + nrm[2] * nrm[2]);
                if (ntri < kPl && nn > 0) {
                  for (int q = 0; q < 3; ++q) nrm[q] /= nn;
                  const double dd = nrm[0] * (f[0] - a[0]) + nrm[1] * (f[1] - a[1]) + nrm[2] * (f[2] - a[2]);
                  PL[ntri] = make_float4((float)nrm[0], (float)nrm[1], (float)nrm[2], (float)dd);
                }
                if (!(nn > 0)) ntri = kPl;  // a degenerate triangle: no plane test for this cell
                ++ntri;
              }
              Vk += 3 * len;
            }
            if (ntri > kPl) PL[0] = make_float4(0.f, 0.f, 0.f, 3.0e38f);
          }
          int64_t nv = 0;
          for (int64_t k = 0; k < nf; ++k) {
            O[2 + k] = make_float4((float)(FC[3 * k] - a[0]), (float)(FC[3 * k + 1] - a[1]), (float)(FC[3 * k + 2] - a[2]),
                                   (float)LEN[k]);
            nv += (int64_t)LEN[k];
          }
          for (int64_t j = 0; j < nv; ++j)
            O[2 + nf + j] = make_float4((float)(V[3 * j] - a[0]), (float)(V[3 * j + 1] - a[1]), (float)(V[3 * j + 2] - a[2]), 0.f);
          // the cell across each face, on the first vertex of the face's loop
          const int64_t c = h->order[s];
          int64_t v0 = 0;
          for (int64_t k = 0; k < nf; ++k) {
            const int32_t f = g.cf[g.cf_off[c] + k];
            const int64_t other = g.own[f] == c ? g.nei[f] : g.own[f];
            const int32_t across = g.nei[f] >= 0 && other >= 0 ? (int32_t)h->rank[other] : -1;
            O[2 + nf + v0].w = __builtin_bit_cast(float, across);
            v0 += (int64_t)LEN[k];
          }
        }
      });
      if ((rc = upload(h->d_rec32, r32))) return rc;
      if ((rc = upload(h->d_pl32, pl32))) return rc;
    }
  }
  // cells across each cell's interior faces, sorted ids in sorted cell order
  {
    std::vector<int64_t> noff(g.nc + 1, 0);
    const int64_t nf = g.nf;
    for (int64_t f = 0; f < nf; ++f)
      if (g.nei[f] >= 0) {
        noff[h->rank[g.own[f]] + 1]++;
        noff[h->rank[g.nei[f]] + 1]++;
      }
    for (int64_t s = 0; s < g.nc; ++s) noff[s + 1] += noff[s];
    std::vector<int32_t> nb(noff[g.nc]);
    std::vector<int64_t> fill(noff.begin(), noff.end() - 1);
    for (int64_t f = 0; f < nf; ++f)
      if (g.nei[f] >= 0) {
        const int32_t a = h->rank[g.own[f]], b = h->rank[g.nei[f]];
        nb[fill[a]++] = b;
        nb[fill[b]++] = a;
      }
    if ((rc = upload(h->d_nbr_off, noff))) return rc;
    if ((rc = upload(h->d_nbr, nb))) return rc;
  }
  // padded bounding boxes (sorted cell order) and the point-location grid (sorted cell indices listed in
  // every bin their box touches, in ascending mesh cell id so the lowest containing cell is found first)
  std::vector<double> bb(6 * g.nc);
  for (int64_t c = 0; c < g.nc; ++c)
    for (int q = 0; q < 3; ++q) {
      const double ext = g.hi[3 * c + q] - g.lo[3 * c + q];
      bb[6 * c + q] = g.lo[3 * c + q] - 1e-9 * ext;
      bb[6 * c + 3 + q] = g.hi[3 * c + q] + 1e-9 * ext;
    }
  {
    std::vector<double> bbs(6 * g.nc);
    for (int64_t s = 0; s < g.nc; ++s)
      for (int q = 0; q < 6; ++q) bbs[6 * s + q] = bb[6 * (int64_t)h->order[s] + q];
    if ((rc = upload(h->d_bb, bbs))) return rc;
  }
  double gh = std::cbrt(g.total_volume / (double)g.nc);
  for (int q = 0; q < 3; ++q) gh = std::max(gh, (g.dom_hi[q] - g.dom_lo[q]) / 2048.0);
  int64_t nb[3];
  for (int q = 0; q < 3; ++q) {
    h->glo[q] = g.dom_lo[q] - 1e-9 * (g.dom_hi[q] - g.dom_lo[q]) - 1e-300;
    nb[q] = std::max<int64_t>(1, (int64_t)std::ceil((g.dom_hi[q] + 1e-9 * (g.dom_hi[q] - g.dom_lo[q]) - h->glo[q]) / gh));
    h->gnb[q] = nb[q];
  }
  h->gh = gh;
  const int64_t nbins = nb[0] * nb[1] * nb[2];
  std::vector<int64_t> off(nbins + 1, 0);
  auto range = [&](int64_t c, int q, int64_t &b0, int64_t &b1) {
    b0 = (int64_t)std::floor((bb[6 * c + q] - h->glo[q]) / gh);
    b1 = (int64_t)std::floor((bb[6 * c + 3 + q] - h->glo[q]) / gh);
    b0 = std::min(std::max<int64_t>(b0, 0), nb[q] - 1);
    b1 = std::min(std::max<int64_t>(b1, 0), nb[q] - 1);
  };
  for (int64_t c = 0; c < g.nc; ++c) {
    int64_t lo[3], hi[3];
    for (int q = 0; q < 3; ++q) range(c, q, lo[q], hi[q]);
    for (int64_t z = lo[2]; z <= hi[2]; ++z)
      for (int64_t y = lo[1]; y <= hi[1]; ++y)
        for (int64_t x = lo[0]; x <= hi[0]; ++x) off[x + nb[0] * (y + nb[1] * z) + 1]++;
  }
  for (int64_t b = 0; b < nbins; ++b) off[b + 1] += off[b];
  std::vector<int32_t> cells(off[nbins]);
  std::vector<int64_t> fill(off.begin(), off.end() - 1);
  for (int64_t c = 0; c < g.nc; ++c) {
    int64_t lo[3], hi[3];
    for (int q = 0; q < 3; ++q) range(c, q, lo[q], hi[q]);
    for (int64_t z = lo[2]; z <= hi[2]; ++z)
      for (int64_t y = lo[1]; y <= hi[1]; ++y)
        for (int64_t x = lo[0]; x <= hi[0]; ++x) cells[fill[x + nb[0] * (y + nb[1] * z)]++] = h->rank[c];
  }
  if ((rc = upload(h->d_gb_off, off))) return rc;
  if ((rc = upload(h->d_gb_cell, cells))) return rc;
  return AICA_OK;
}

// The half lists' groups and lists for a number density.
static int make_groups(aica_dil *h, double density, double target) {
  h->groups_ready = false;
  int rc = build_groups(h->geo, h->order, h->split_depth, h->pairs, density, target, h->grp);
  if (rc) return rc;
  const Groups &G = h->grp;
  const int64_t E = G.e_off[G.ng];
  std::vector<float4> v32(E);
  std::vector<double4> v64(E);
  // Entry offsets: a j of group B at xm relative to orig_B is referred into A's frame at R xm + o with
  // o = T(orig_B) - orig_A (R = I and o = orig_B + t - orig_A for a translation).  The fourth component
  // holds the image code, plus kRotFlag when the image has a rotation (whose R the kernels look up).
  const std::array<Xf, 27> image = image_table(h->geo);
  parallel_for(G.ng, [&](int64_t b, int64_t en, int) {
    for (int64_t A = b; A < en; ++A)
      for (int64_t e = G.e_off[A]; e < G.e_off[A + 1]; ++e) {
        const int64_t B = G.e_B[e];
        const int img = 9 * (G.e_img[3 * e] + 1) + 3 * (G.e_img[3 * e + 1] + 1) + (G.e_img[3 * e + 2] + 1);
        const Xf &T = image[img];
        double o[3];
        if (T.rot) {
          double tb[3];
          T.apply(&G.orig[3 * B], tb);
          for (int q = 0; q < 3; ++q) o[q] = tb[q] - G.orig[3 * A + q];
        } else {
          for (int q = 0; q < 3; ++q) o[q] = G.orig[3 * B + q] + T.y[q] - G.orig[3 * A + q];
        }
        const int code = img + (T.rot ? kRotFlag : 0);
        v32[e] = make_float4((float)o[0], (float)o[1], (float)o[2], __builtin_bit_cast(float, code));
        v64[e] = make_double4(o[0], o[1], o[2], __builtin_bit_cast(double, (int64_t)code));
      }
  });
  if (h->geo.has_rot) {  // R of every image code (the identity for translations)
    std::vector<double> r64(27 * 9);
    for (int code = 0; code < 27; ++code)
      for (int i = 0; i < 9; ++i) r64[9 * code + i] = image[code].R[i];
    if ((rc = upload(h->d_rot64, r64))) return rc;
  }
  if ((rc = upload(h->d_g_cell0, G.cell0))) return rc;
  if ((rc = upload(h->d_e_off, G.e_off))) return rc;
  if ((rc = upload(h->d_e_B, G.e_B))) return rc;
  if ((rc = upload(h->d_e_vec32, v32))) return rc;
  if ((rc = upload(h->d_e_vec64, v64))) return rc;
  if ((rc = upload(h->d_nl_off, G.nl_off))) return rc;
  if ((rc = upload(h->d_nl_e, G.nl_e))) return rc;
  if ((rc = upload(h->d_nl_d, G.nl_d))) return rc;
  if ((rc = upload(h->d_nl_r, G.nl_r))) return rc;
  {
    std::vector<int32_t> rcnt(h->geo.nc);
    for (int64_t d = 0; d < h->geo.nc; ++d) rcnt[d] = (int32_t)(G.rc_off[d + 1] - G.rc_off[d] + 1);
    if ((rc = upload(h->d_rcnt, rcnt))) return rc;
  }
  if ((rc = upload(h->d_orig, G.orig))) return rc;
  if ((rc = upload(h->d_of_cell, G.of_cell))) return rc;
  const HalfFrames hf{h->d_of_cell.as<int32_t>(), h->d_orig.as<double>(), h->d_e_off.as<int64_t>(), h->d_e_B.as<int32_t>(),
                      h->d_e_vec32.as<float4>(), h->d_e_vec64.as<double4>(), {}};
  if ((rc = upload(h->d_half, std::vector<HalfFrames>{hf}))) return rc;
  h->groups_ready = true;
  return AICA_OK;
}

// The full lists' groups and lists (with the vertex predicate, those with masks).
static int make_neigh(aica_dil *h, double density, double target) {
  h->neigh_ready = false;
  int rc = h->predicate == AICA_DIL_VERTEX
               ? build_neigh_masked(h->geo, h->order, h->split_depth, h->grp, density, target, h->nb)
               : build_neigh(h->geo, h->order, h->split_depth, h->pairs, density, target, h->nb);
  if (rc) return rc;
  const Neigh &N = h->nb;
  const int64_t NE = N.e_off[N.ng];
  std::vector<float4> v32(NE);
  std::vector<double4> v64(NE);
  const std::array<Xf, 27> image = image_table(h->geo);
  parallel_for(N.ng, [&](int64_t b, int64_t e, int) {
    for (int64_t a = b; a < e; ++a)
      for (int64_t k = N.e_off[a]; k < N.e_off[a + 1]; ++k) {
        const int64_t B = N.e_B[k];
        const int c = N.e_code[k];
        const Xf &T = image[c];
        double o[3], tb[3] = {0, 0, 0};
        if (T.rot) T.apply(&N.orig[3 * B], tb);
        for (int q = 0; q < 3; ++q)
          o[q] = T.rot ? tb[q] - N.orig[3 * a + q] : N.orig[3 * B + q] + T.y[q] - N.orig[3 * a + q];
        const int code = c + (T.rot ? kRotFlag : 0);
        v32[k] = make_float4((float)o[0], (float)o[1], (float)o[2], __builtin_bit_cast(float, code));
        v64[k] = make_double4(o[0], o[1], o[2], __builtin_bit_cast(double, (int64_t)code));
      }
  });
  if (h->geo.has_rot) {
    std::vector<int32_t> list, turned;
    for (int64_t a = 0; a < N.ng; ++a) {
      bool rot = false;
      for (int64_t e = N.e_off[a]; e < N.e_off[a + 1] && !rot; ++e) rot = image[N.e_code[e]].rot;
      (rot ? turned : list).push_back((int32_t)a);
    }
    h->nb_plain_groups = (int64_t)list.size();
    list.insert(list.end(), turned.begin(), turned.end());
    if ((rc = upload(h->d_nb_glist, list))) return rc;
  }
  if ((rc = upload(h->d_nb_cell0, N.cell0))) return rc;
  if ((rc = upload(h->d_nb_run_off, N.run_off))) return rc;
  if ((rc = upload(h->d_nb_runs, N.runs))) return rc;
  if ((rc = upload(h->d_nb_eoff, N.e_off))) return rc;
  if ((rc = upload(h->d_nb_ioff, N.i_off))) return rc;
  if ((rc = upload(h->d_nb_imask, N.i_mask))) return rc;
  if ((rc = upload(h->d_nb_vec32, v32))) return rc;
  if ((rc = upload(h->d_nb_vec64, v64))) return rc;
  if ((rc = upload(h->d_nb_orig, N.orig))) return rc;
  if (getenv("AICA_VERBOSE"))
    fprintf(stderr, "neighbour lists: %lld groups, %lld entries, %lld runs, reach %.3f\n", (long long)N.ng, (long long)NE,
            (long long)N.runs.size(), N.reach);
  if (getenv("AICA_VERBOSE")) {
    double vol = 0, cells = 0;
    for (const CellRun &r : N.runs)
      for (int32_t s = r.d0; s < r.d1; ++s) {
        vol += h->geo.vol[h->order[s]];
        cells += 1;
      }
    fprintf(stderr, "neighbour lists: per group %.1f runs, %.1f cells, %.1f molecules expected\n", (double)N.runs.size() / N.ng,
            cells / N.ng, vol * density / N.ng);
  }
  h->neigh_ready = true;
  return AICA_OK;
}

// Both sets of lists, for n molecules (any call may need either: the full lists decide pairs near rc^2 in the frames of the
// half lists).  Full lists: groups of up to 128 expected molecules, or 64 while that leaves fewer
// of them than CUs (a pass of FP64 forces and adjoint, us, 64 against 128: 7,000 molecules 168 and 180, 13,000 166 and
// 188, 28,000 191 and 190, 31,999 of five species 180 and 185; 40,000 232 and 203; with 32 no size is faster).  They are kept while n leaves the cuts as they are: a program whose molecule
// count changes from step to step would rebuild them at every binning (107 ms of host work at 371,896 molecules, 1.3 s at
// 6.7 million).
static int ensure_groups(aica_dil *h, int64_t n, hipStream_t st) {
  const double density = (double)n / h->geo.total_volume;
  double target = 64.0;  // largest expected occupancy of a group (k-d subtree; measured best on the channel)
  if (const char *e = getenv("AICA_GROUP_TARGET")) target = std::max(1.0, atof(e));
  double nb_target = n < 256 * 128 ? 64.0 : 128.0;
  if (const char *e = getenv("AICA_NB_TARGET")) nb_target = std::max(1.0, atof(e));
  const bool keep = h->groups_ready && h->grp.cut.holds(density, target);
  // the lists with masks depend on the half lists as well
  const bool nb_keep =
      h->neigh_ready && h->nb.cut.holds(density, nb_target) && (keep || h->predicate != AICA_DIL_VERTEX);
  if (keep && nb_keep) return AICA_OK;
  // the lists are overwritten in place: work of the last steps that still reads them has to end first (the copies are not
  // ordered with a non-blocking stream)
  HIPCHK(hipStreamSynchronize(st));
  auto t0 = std::chrono::steady_clock::now();
  int rc;
  if (!keep && (rc = make_groups(h, density, target))) return rc;
  if (!nb_keep && (rc = make_neigh(h, density, nb_target))) return rc;
  // Half-ulp roundings per axis of a pair vector: a translated one's at most three of the frame's reach (the two
  // positions in their groups' frames, the offset, the sum), a rotated one's six in FP64 (in FP32 three: it is formed in
  // FP64); and in FP64, at the size of the coordinates themselves, those of the offsets (T orig_B - orig_A), and how far
  // a transform and its inverse miss.
  const bool rot = h->geo.has_rot;
  h->frame_reach[0] = 3.0 * (h->nb.reach + h->grp.reach);
  h->frame_reach[1] = (rot ? 6.0 : 3.0) * (h->nb.reach + h->grp.reach);
  h->frame_err = std::ldexp(1.0, -53) * (rot ? 20.0 : 2.5) * coordinate_size(h->geo) + transform_skew(h->geo);
  h->group_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  return AICA_OK;
}

// =====================================================================================================
// C ABI (every entry point is declared extern "C" in aica.h)

const char *aica_last_error(void) { return last_error_cstr(); }

int aica_build_dil(const aica_mesh *mesh, double rcut, double guard, aica_dil **out) {
  return aica_build_dil_ex(mesh, rcut, guard, AICA_DIL_CLOSEST, out);
}

int aica_build_dil_ex(const aica_mesh *mesh, double rcut, double guard, int32_t predicate, aica_dil **out) {
  if (!out) return fail(AICA_E_INVAL, "out is NULL");
  *out = nullptr;
  if (predicate != AICA_DIL_CLOSEST && predicate != AICA_DIL_VERTEX)
    return fail(AICA_E_INVAL, "predicate must be AICA_DIL_CLOSEST or AICA_DIL_VERTEX");
  if (!(rcut > 0) || !std::isfinite(rcut) || !(guard >= 0) || !std::isfinite(guard))
    return fail(AICA_E_INVAL, "rcut must be > 0 and guard >= 0");
  auto t0 = std::chrono::steady_clock::now();
  aica_dil *h = new (std::nothrow) aica_dil();
  if (!h) return fail(AICA_E_NOMEM, "handle allocation failed");
  int rc = build_geometry(mesh, h->geo);
  if (rc) {
    delete h;
    return rc;
  }
  h->rcut = rcut;
  h->guard = guard;
  h->predicate = predicate;
  const bool verbose = getenv("AICA_VERBOSE") != nullptr;
  auto t1 = std::chrono::steady_clock::now();
  spatial_order(h->geo, h->order, h->rank, h->split_depth);
  auto t2 = std::chrono::steady_clock::now();
  rc = build_cell_pairs(h->geo, h->order, h->rank, rcut + guard, predicate, h->pairs);
  if (verbose)
    fprintf(stderr, "aica_build_dil: geometry %.2fs order %.2fs pairs %.2fs (%zu)\n",
            std::chrono::duration<double>(t1 - t0).count(), std::chrono::duration<double>(t2 - t1).count(),
            std::chrono::duration<double>(std::chrono::steady_clock::now() - t2).count(), h->pairs.size());
  if (rc) {
    delete h;
    return rc;
  }
  h->build_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  *out = h;
  return AICA_OK;
}

void aica_dil_free(aica_dil *h) {
  if (!h) return;
  for (auto &kv : h->timers)
    for (auto &ev : kv.second.pending) {
      (void)hipEventDestroy(ev.first);
      (void)hipEventDestroy(ev.second);
    }
  delete h;
}

// Which lists a force call runs on.  The full lists (k_force: every pair from both sides, no reaction records) take
// FP64, and FP32 from 200,000 molecules on without rotation: 6.7 million molecules take 1.50 ms in place of 2.50 ms (pair
// kernel) and 0.34 ms (finalize).  The line is not where the two take the same time.  FP32 bin and forces of a liquid of
// density 0.8, us, half and full lists: 13,440 molecules 81 and 90, 30,000 103 and 90, 60,000 109 and 102, 100,000 143 and
// 112, 150,000 173 and 127, 200,000 198 and 135, 400,000 267 and 186.  Nor is it one of accuracy: from 1,000 to 400,000
// molecules the rms errors against FP64 are the same on either to the second digit (U 2e-8 to 2e-7, W 1.1e-7 to 1.6e-7,
// F 4.0e-7 to 4.3e-7 of the rms force).  Below it and across rotations the half lists are kept so that U and W stay what
// they were to the last digits: the lists add FP32 terms in another order, which moves them by about 1e-9.
// With the vertex predicate both precisions keep them: it does not list every pair in range, and the half lists decide
// which are left out.
static bool full_lists(const aica_dil *h, int64_t n, int tsize) {
  return h->predicate != AICA_DIL_VERTEX && (tsize == 8 || (n >= 200000 && !h->geo.has_rot));
}

int aica_bin(aica_dil *h, const void *pos_dev, int32_t pos_dtype, int64_t n, void *hip_stream) {
  if (!h) return fail(AICA_E_INVAL, "handle is NULL");
  h->bin_valid = false;
  h->wsteps_groups = 0;
  if (n < 0 || (n > 0 && !pos_dev)) return fail(AICA_E_INVAL, "bad positions");
  if (n >= (1LL << 28) - 1) return fail(AICA_E_INVAL, "too many molecules (the pair kernels take fewer than 2^28 - 1)");
  if (pos_dtype != AICA_FP32 && pos_dtype != AICA_FP64) return fail(AICA_E_INVAL, "pos_dtype must be AICA_FP32 or AICA_FP64");
  hipStream_t st = (hipStream_t)hip_stream;
  int rc;
  if (!h->geometry_on_device) {
    // the device copy of the geometry is made on first use, so that setup and the interaction
    // lists can be built and inspected without a GPU
    if (hipGetDevice(&h->device) != hipSuccess) return fail(AICA_E_HIP, "no HIP device");
    if ((rc = upload_geometry(h))) return rc;
    h->geometry_on_device = true;
  }
  rc = ensure_groups(h, n, st);
  if (rc) return rc;
  const int64_t nc = h->geo.nc;
  if (!h->host_status && hipHostMalloc((void **)&h->host_status, 8 * (8 + kRouteSlots)) != hipSuccess) {
    h->host_status = nullptr;
    return fail(AICA_E_NOMEM, "pinned host allocation failed");
  }
  if ((rc = h->d_cell_of.ensure(4 * std::max<int64_t>(n, 1)))) return rc;
  if ((rc = h->d_count.ensure(4 * nc))) return rc;
  if ((rc = h->d_cell_start.ensure(4 * (nc + 1)))) return rc;
  if ((rc = h->d_rank.ensure(4 * std::max<int64_t>(n, 1)))) return rc;
  if ((rc = h->d_perm.ensure(4 * std::max<int64_t>(n, 1)))) return rc;
  if ((rc = h->d_slot_base.ensure(8 * (nc + 1)))) return rc;
  if ((rc = h->d_cell_sorted.ensure(4 * std::max<int64_t>(n, 1)))) return rc;
  if ((rc = h->d_status.ensure(8 * (8 + kRouteSlots)))) return rc;
  if ((rc = h->d_slow.ensure(4 * std::max<int64_t>(n, 1)))) return rc;
  if ((rc = h->d_ref.ensure(16 * std::max<int64_t>(n, 1)))) return rc;

  ProfScope ps(h, "bin", st);
  unsigned long long *status = h->d_status.as<unsigned long long>();
  unsigned long long *routes = status + 8;
  // the previous binning of the same n (if any) gives the traversal order and the hints: its
  // permutation moves to d_perm_prev, and d_cell_sorted still holds its cells until rebuilt below
  const bool prev = h->perm_n == n && n > 0;
  h->perm_n = -1;
  if (prev) h->d_perm.swap(h->d_perm_prev);
  if ((rc = h->d_perm.ensure(4 * std::max<int64_t>(n, 1)))) return rc;
  // status: [0] unlocated, [1] reaction slots, [2] slow-kernel molecules, [8 ..) counters of the molecules the
  // records located
  hipLaunchKernelGGL(k_clear_bin, dim3(grid1d(std::max<int64_t>(nc, 8 + kRouteSlots), 256)), dim3(256), 0, st,
                     h->d_count.as<int32_t>(), nc, status, 8 + kRouteSlots, h->d_half.as<HalfFrames>(),
                     BinRef{pos_dev, h->d_perm.as<int32_t>(), h->d_cell_sorted.as<int32_t>(), pos_dtype == AICA_FP64});
  const int32_t *trav = prev ? h->d_perm_prev.as<int32_t>() : nullptr;
  const int32_t *hint = prev ? h->d_cell_sorted.as<int32_t>() : nullptr;
  if (n > 0) {
    const float4 *r32 = h->has_rec32 ? h->d_rec32.as<float4>() : nullptr;
    const float4 *pl = h->has_rec32 ? h->d_pl32.as<float4>() : nullptr;
    int32_t *slow = h->d_slow.as<int32_t>();
    unsigned long long *nslow = status + 2;
    const int mpb = n <= kFewMolecules ? kMpbFew : kMpb;
#define AICA_LOCATE(PT)                                                                                            \
  hipLaunchKernelGGL(n <= kFewMolecules ? (k_locate_fast<PT, kMpbFew>) : (k_locate_fast<PT, kMpb>), dim3(grid1d(n, mpb)), \
                     dim3(256), 0, st, (const PT *)pos_dev, \
                     n, trav, hint, r32, pl, h->d_ref.as<float4>(), h->d_cell_of.as<int32_t>(), h->d_rank.as<int32_t>(), \
                     h->d_count.as<int32_t>(), nslow, slow, routes);                                               \
  hipLaunchKernelGGL((k_locate_slow<PT>), dim3(std::min<int64_t>(grid1d(n, 8), 2048)), dim3(256), 0, st,            \
                     (const PT *)pos_dev, nslow, slow, trav, hint, r32, pl, h->d_rec_off.as<int64_t>(),          \
                     h->d_rec.as<double>(), h->d_nbr_off.as<int64_t>(),                                            \
                     h->d_nbr.as<int32_t>(), h->d_bb.as<double>(), h->d_gb_off.as<int64_t>(),                       \
                     h->d_gb_cell.as<int32_t>(), h->glo[0], h->glo[1], h->glo[2], h->gh, h->gnb[0], h->gnb[1],      \
                     h->gnb[2], h->d_ref.as<float4>(), h->d_cell_of.as<int32_t>(), h->d_rank.as<int32_t>(),       \
                     h->d_count.as<int32_t>(), status)
    if (pos_dtype == AICA_FP64) {
      AICA_LOCATE(double);
    } else {
      AICA_LOCATE(float);
    }
#undef AICA_LOCATE
    HIPCHK(hipGetLastError());
  }
  // the unlocated count is read with the other counts below (one synchronisation per binning); an
  // unlocated molecule is left out of the occupancy and of the permutation
  if ((rc = scan_cells(h, nc, !full_lists(h, n, 4), status + 1, st))) return rc;
  if (n > 0) {
    // the slow list is done with: its space takes the unsorted molecules
    hipLaunchKernelGGL(k_scatter, dim3(grid1d(n, 256)), dim3(256), 0, st, h->d_cell_of.as<int32_t>(), trav, n,
                       h->d_cell_start.as<int32_t>(), h->d_rank.as<int32_t>(), h->d_slow.as<int32_t>(),
                       h->d_cell_sorted.as<int32_t>());
    hipLaunchKernelGGL(k_sort_cells, dim3(grid1d(n, 256)), dim3(256), 0, st, h->d_cell_start.as<int32_t>(),
                       h->d_cell_sorted.as<int32_t>(), h->d_slow.as<int32_t>(), nc, n, h->d_perm.as<int32_t>());
  }
  HIPCHK(hipGetLastError());
  // the counts come back through pinned memory of the handle, in one copy
  unsigned long long *stat = h->host_status;
  HIPCHK(hipMemcpyAsync(stat, status, 8 * (8 + kRouteSlots), hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  const int64_t jt = (int64_t)stat[1];
  const unsigned long long unl = stat[0];
  if (unl > 0) return fail(AICA_E_UNLOCATED, std::to_string(unl) + " molecule(s) lie in no mesh cell");
  h->located[1] = 0;
  for (int k = 0; k < kRouteSlots; ++k) h->located[1] += (int64_t)stat[8 + k];
  h->located[2] = (int64_t)stat[2];
  h->located[0] = n - h->located[1] - h->located[2];
  if (jt >= (1LL << 31)) return fail(AICA_E_NOMEM, "reaction slots exceed 2^31; split the system");
  h->perm_n = n;  // d_perm holds this binning's permutation
  h->jtotal = jt;
  h->n = n;
  h->bin_pos = pos_dev;
  h->bin_dtype = pos_dtype;
  h->bin_valid = true;
  return AICA_OK;
}

static int build_tab(const aica_dil *h, const aica_params *p, LJTab &t) {
  if (!p) return fail(AICA_E_INVAL, "params is NULL");
  if (!(p->rcut > 0) || p->rcut > h->rcut * (1 + 1e-15))
    return fail(AICA_E_INVAL, "params.rcut must be > 0 and not exceed the DIL's rcut");
  if (p->n_species < 1 || p->n_species > 8 || !p->eps || !p->sigma)
    return fail(AICA_E_INVAL, "n_species must be 1..8 with eps and sigma given");
  if (p->precision != AICA_FP32 && p->precision != AICA_FP64) return fail(AICA_E_INVAL, "bad precision");
  memset(&t, 0, sizeof t);
  for (int a = 0; a < p->n_species; ++a)
    if (!(p->eps[a] > 0) || !(p->sigma[a] > 0)) return fail(AICA_E_INVAL, "eps and sigma must be positive");
  for (int a = 0; a < p->n_species; ++a)
    for (int b = 0; b < p->n_species; ++b) {
      const double e = a == b ? p->eps[a] : std::sqrt(p->eps[a] * p->eps[b]);
      const double s = a == b ? p->sigma[a] : 0.5 * (p->sigma[a] + p->sigma[b]);
      const int k = a * 8 + b;
      t.sig2d[k] = s * s;
      t.e24d[k] = 24.0 * e;
      t.e4d[k] = 4.0 * e;
      t.sig2[k] = (float)(s * s);
      t.e24[k] = (float)(24.0 * e);
      t.e4[k] = (float)(4.0 * e);
    }
  t.rc2d = p->rcut * p->rcut;
  t.rc2 = (float)t.rc2d;
  t.band = (float)(t.rc2d * std::ldexp(1.0, -20));
  t.rc2lo = (float)(t.rc2d - (double)t.band);
  t.rc2hi = (float)(t.rc2d + (double)t.band);
  // the square of a pair at about rc whose vector is off by at most err per axis, and the roundings of the square
  auto near = [&](double half_ulp, double reach) {
    const double err = half_ulp * reach + h->frame_err;
    return 3.5 * p->rcut * err + 3.0 * err * err + 16.0 * t.rc2d * half_ulp;
  };
  const double n32 = near(std::ldexp(1.0, -24), h->frame_reach[0]), n64 = near(std::ldexp(1.0, -53), h->frame_reach[1]);
  t.near_lo = (float)(t.rc2d - n32);
  t.near_hi = (float)(t.rc2d + n32);
  t.near_lod = t.rc2d - n64;
  t.near_hid = t.rc2d + n64;
  t.reach2 = std::max(t.rc2d, (t.rc2d + n32) * (1.0 - 5e-5));
  t.reach2d = std::max(t.rc2d, (t.rc2d + n64) * (1.0 - 5e-5));
  t.nsp = p->n_species;
  return AICA_OK;
}

// Device buffers of one force call: the handle's grow-only workspace, or regions of the fixed scratch array
// (aica_forces_noalloc).  pos: [n] gathered positions; box: the groups' boxes (full lists); own: [2n] (hi, lo) own
// records and jpart: [J] reaction records tagged with epoch (half lists); gpart, gnp: per-group partials; red: stage-1
// reduction rows.
struct ForceWs {
  void *pos = nullptr, *box = nullptr, *own = nullptr, *jpart = nullptr, *gpart = nullptr, *gnp = nullptr, *red = nullptr;
  uint32_t epoch = 0;
};


// Reaction buffer: (re)allocate, fill with a pattern no epoch can equal, and advance the epoch.
static int prepare_jpart(aica_dil *h, size_t bytes, hipStream_t st) {
  const void *old = h->d_jpart.p;
  // a growing buffer gets 1/8 headroom: the slot count follows the occupancy of every step, and each
  // reallocation costs a fill of the whole buffer
  int rc = h->d_jpart.ensure(bytes > h->d_jpart.bytes ? bytes + bytes / 8 : bytes);
  if (rc) return rc;
  if (h->d_jpart.p != old || h->jpart_tagged < h->d_jpart.bytes || h->epoch >= kMaxEpoch) {
    const int64_t words = (int64_t)(h->d_jpart.bytes / 4);
    hipLaunchKernelGGL((k_fill<uint32_t>), dim3(grid1d(words, 256)), dim3(256), 0, st, h->d_jpart.as<uint32_t>(),
                       words, 0xFFFFFFFFu);
    HIPCHK(hipGetLastError());
    h->jpart_tagged = h->d_jpart.bytes;
    h->epoch = 0;
  }
  h->epoch += 1;
  return AICA_OK;
}

// A block of four waves per group up to this many groups, a wave per group beyond: a small system has fewer groups than
// the chip has SIMDs (1024), so a group's own length is what the call takes.  Pair kernel, FP32, one wave against a
// block per group: 16 groups 63 and 26 us, 256 groups 77 and 31, 629 groups 69 and 37, 616 groups of two passes 264
// and 71, 130,000 molecules 121 and 85, 160,000 98 and 104, 7963 groups 257 and 268.  (With every wave listing and
// pruning the whole j-side the blocks took 40, 44, 43 and 228 us; eight waves gain 4 us on 16 and 256 groups and lose
// 15 on 629.)
constexpr int64_t kSplitGroups = 3072;

// The half-list pair kernel: forces (MODE 0), pair export and per-molecule counts (MODE 1).
template <typename T, int MODE>
static int launch_pair(aica_dil *h, const ForceWs &ws, const LJTab &tab, bool comp, hipStream_t st, int64_t cap,
                       unsigned long long *pcount, int32_t *mol_count = nullptr) {
  using V4 = typename Vec4<T>::type;
  const int64_t ng = h->grp.ng;
  constexpr int NW = pair_waves(sizeof(T));
  constexpr bool SPLITS = MODE == 0 && sizeof(T) == 4;
  const bool split = SPLITS && ng <= kSplitGroups;  // few groups: a whole block per group
  const int64_t nblocks = split ? ng : (ng + NW - 1) / NW;
  const int64_t padded = ((nblocks + 7) / 8) * 8;
  const V4 *pos = (const V4 *)ws.pos;
  const V4 *ev = sizeof(T) == 4 ? (const V4 *)h->d_e_vec32.p : (const V4 *)h->d_e_vec64.p;
  T *jpart = MODE == 1 ? nullptr : (T *)ws.jpart;
  T *own = MODE == 1 ? nullptr : (T *)ws.own;
  double *gpart = MODE == 0 ? (double *)ws.gpart : nullptr;
  unsigned long long *gnp = MODE == 0 ? (unsigned long long *)ws.gnp : nullptr;
  int32_t *pairs_out = (MODE == 1 && cap >= 0) ? h->d_pairs.as<int32_t>() : nullptr;  // cap < 0: counts only
  // rotating referral: FP64 rotations and offsets for both precisions (the referred position is rounded once)
  const double *rot = h->geo.has_rot ? h->d_rot64.as<double>() : nullptr;
  const double4 *evd = h->geo.has_rot ? h->d_e_vec64.as<double4>() : nullptr;
  const int nsp = tab.nsp;
#define AICA_LAUNCH_S(MIX, COMP, ROT, SPLIT)                                                                       \
  hipLaunchKernelGGL((k_pair<T, MIX, MODE, COMP, ROT, SPLIT>), dim3((unsigned)padded), dim3(64 * NW), 0, st, pos,         \
                     h->d_g_cell0.as<int32_t>(), h->d_cell_start.as<int32_t>(), ev,                                        \
                     h->d_slot_base.as<int64_t>(), h->d_nl_off.as<int64_t>(), h->d_nl_e.as<int32_t>(),            \
                     h->d_nl_d.as<int32_t>(), h->d_nl_r.as<int32_t>(), jpart, own, gpart, gnp, ng, padded, tab,     \
                     rot, evd, h->d_perm.as<int32_t>(), cap, pairs_out, pcount, mol_count, ws.epoch)
#define AICA_LAUNCH_R(MIX, COMP, ROT)                    \
  do {                                                   \
    if constexpr (SPLITS) {                              \
      if (split) AICA_LAUNCH_S(MIX, COMP, ROT, true);    \
      else AICA_LAUNCH_S(MIX, COMP, ROT, false);         \
    } else {                                             \
      AICA_LAUNCH_S(MIX, COMP, ROT, false);              \
    }                                                    \
  } while (0)
#define AICA_LAUNCH(COMP, ROT)                 \
  do {                                         \
    if (nsp == 1) AICA_LAUNCH_R(0, COMP, ROT); \
    else if (nsp == 2) AICA_LAUNCH_R(1, COMP, ROT); \
    else AICA_LAUNCH_R(2, COMP, ROT);          \
  } while (0)
  if constexpr (MODE == 1) {  // the pairs are the same whatever the species (compensation is of no account)
    if (rot) AICA_LAUNCH_R(0, true, true);
    else AICA_LAUNCH_R(0, true, false);
  } else if (rot) {  // rotating referral: compensated sums always (the variants with a rotation are built once)
    AICA_LAUNCH(true, true);
  } else if constexpr (sizeof(T) == 4) {  // compensated sums exist in FP32 only
    if (comp) AICA_LAUNCH(true, false);
    else AICA_LAUNCH(false, false);
  } else {
    AICA_LAUNCH(false, false);
  }
#undef AICA_LAUNCH
#undef AICA_LAUNCH_R
#undef AICA_LAUNCH_S
  HIPCHK(hipGetLastError());
  return AICA_OK;
}

// The full lists, over all groups (part -1) or, with rotating referral, over those without (0) or with a turned entry (1):
// the kernels with rotations hold fewer blocks per CU and form the pair vector in more steps, and only the groups along
// the coupled sides need them (371,896-molecule wedge, FP32 adjoint: 284 us for all groups with rotations, 151 + 89 in
// two launches).
template <typename T>
static NbLists nb_lists(const aica_dil *h, int part) {
  NbLists nl;
  nl.cell0 = h->d_nb_cell0.as<int32_t>();
  nl.run_off = h->d_nb_run_off.as<int64_t>();
  nl.runs = h->d_nb_runs.as<int4>();
  nl.e_off = h->d_nb_eoff.as<int64_t>();
  nl.e_vec = sizeof(T) == 4 ? h->d_nb_vec32.p : h->d_nb_vec64.p;
  nl.e_vec64 = h->d_nb_vec64.as<double4>();
  nl.rot = h->geo.has_rot ? h->d_rot64.as<double>() : nullptr;
  nl.list = nullptr;
  nl.ng = h->nb.ng;
  nl.half = h->d_half.as<HalfFrames>();
  nl.i_off = h->d_nb_ioff.as<int64_t>();
  nl.i_mask = h->d_nb_imask.as<uint32_t>();
  if (h->geo.has_rot && part >= 0) {
    nl.list = h->d_nb_glist.as<int32_t>() + (part ? h->nb_plain_groups : 0);
    nl.ng = part ? h->nb.ng - h->nb_plain_groups : h->nb_plain_groups;
  }
  return nl;
}

// The force kernel: one block per group of the full neighbour lists.
template <typename T>
static int launch_force(aica_dil *h, const ForceWs &ws, const LJTab &tab, bool comp, void *out, hipStream_t st) {
  using V4 = typename Vec4<T>::type;
  const int nsp = tab.nsp;
  constexpr bool C = sizeof(T) == 4;  // compensated sums exist in FP32 only
#define AICA_FORCE(MIX, COMP, ROT)                                                                                  \
  hipLaunchKernelGGL((k_force<T, MIX, COMP, ROT>), dim3((unsigned)padded), dim3(kNbThreads), 0, st, nl,             \
                     (const V4 *)ws.pos, (const T *)ws.box, h->d_cell_start.as<int32_t>(), h->d_perm.as<int32_t>(),  \
                     padded, tab, (T *)out, (double *)ws.gpart, (unsigned long long *)ws.gnp)
  for (int part = 0; part < (h->geo.has_rot ? 2 : 1); ++part) {
    const NbLists nl = nb_lists<T>(h, part);
    const int64_t padded = ((nl.ng + 7) / 8) * 8;
    if (nl.ng == 0) continue;
    if (part == 1) {  // rotating referral: FP64 only (full_lists)
      if constexpr (sizeof(T) == 8) {
        if (nsp == 1) AICA_FORCE(0, false, true);
        else if (nsp == 2) AICA_FORCE(1, false, true);
        else AICA_FORCE(2, false, true);
      }
    } else if (C && comp) {
      if (nsp == 1) AICA_FORCE(0, C, false);
      else if (nsp == 2) AICA_FORCE(1, C, false);
      else AICA_FORCE(2, C, false);
    } else {
      if (nsp == 1) AICA_FORCE(0, false, false);
      else if (nsp == 2) AICA_FORCE(1, false, false);
      else AICA_FORCE(2, false, false);
    }
  }
#undef AICA_FORCE
  HIPCHK(hipGetLastError());
  return AICA_OK;
}

// The adjoint kernel (one, two, or three to eight species), on the groups of the full lists.
template <typename T>
static int launch_adj(aica_dil *h, const LJTab &tab, const AdjTab &at, void *out, hipStream_t st) {
  using V4 = typename Vec4<T>::type;
#define AICA_LAUNCH_ADJ(MIX, ROT, MASK)                                                                              \
  hipLaunchKernelGGL((k_force_adj<T, MIX, ROT, MASK>), dim3((unsigned)padded), dim3(kNbThreads), 0, st, nl,          \
                     h->d_pos.as<V4>(), h->d_gG.as<V4>(), h->d_box.as<T>(), h->d_cell_start.as<int32_t>(),           \
                     h->d_perm.as<int32_t>(), padded, tab, at, (T *)out, h->d_gpar.as<double>())
  const bool vertex = h->predicate == AICA_DIL_VERTEX;  // lists with masks, in one launch
  for (int part = vertex ? -1 : 0; part < (vertex ? 0 : h->geo.has_rot ? 2 : 1); ++part) {
    const NbLists nl = nb_lists<T>(h, part);
    const int64_t padded = ((nl.ng + 7) / 8) * 8;
    if (nl.ng == 0) continue;
    if (part < 0 && h->geo.has_rot) {
      if (tab.nsp == 1) AICA_LAUNCH_ADJ(0, true, true);
      else if (tab.nsp == 2) AICA_LAUNCH_ADJ(1, true, true);
      else AICA_LAUNCH_ADJ(2, true, true);
    } else if (part < 0) {
      if (tab.nsp == 1) AICA_LAUNCH_ADJ(0, false, true);
      else if (tab.nsp == 2) AICA_LAUNCH_ADJ(1, false, true);
      else AICA_LAUNCH_ADJ(2, false, true);
    } else if (part == 1) {
      if (tab.nsp == 1) AICA_LAUNCH_ADJ(0, true, false);
      else if (tab.nsp == 2) AICA_LAUNCH_ADJ(1, true, false);
      else AICA_LAUNCH_ADJ(2, true, false);
    } else {
      if (tab.nsp == 1) AICA_LAUNCH_ADJ(0, false, false);
      else if (tab.nsp == 2) AICA_LAUNCH_ADJ(1, false, false);
      else AICA_LAUNCH_ADJ(2, false, false);
    }
  }
#undef AICA_LAUNCH_ADJ
  HIPCHK(hipGetLastError());
  return AICA_OK;
}

template <typename T, bool COMP>
static void launch_finalize(aica_dil *h, const ForceWs &ws, void *out, hipStream_t st) {
  const int64_t n = h->n;
  hipLaunchKernelGGL((k_finalize<T, COMP>), dim3(grid1d(n, 256)), dim3(256), 0, st, (const T *)ws.own,
                     (const T *)ws.jpart, h->jtotal, n, h->d_cell_sorted.as<int32_t>(), h->d_cell_start.as<int32_t>(),
                     h->d_slot_base.as<int64_t>(), h->d_rcnt.as<int32_t>(), h->d_perm.as<int32_t>(), (T *)out,
                     ws.epoch);
}

// Gather the binned positions by groups (one wave each) into pos: the half lists' groups, or the full lists' with their
// boxes into box (and G into gsort).
template <typename T>
static int gather(aica_dil *h, bool full, const void *pos_dev, const int32_t *species, int nsp, hipStream_t st, void *pos,
                  void *box, const void *G = nullptr, void *gsort = nullptr) {
  using V4 = typename Vec4<T>::type;
  const int64_t ng = full ? h->nb.ng : h->grp.ng;
  const int32_t *cell0 = full ? h->d_nb_cell0.as<int32_t>() : h->d_g_cell0.as<int32_t>();
  const double *orig = full ? h->d_nb_orig.as<double>() : h->d_orig.as<double>();
#define AICA_GATHER(PT)                                                                                               \
  hipLaunchKernelGGL((k_gather_groups<T, PT>), dim3(grid1d(ng, 4)), dim3(256), 0, st, (const PT *)pos_dev, species,   \
                     h->d_perm.as<int32_t>(), h->d_cell_start.as<int32_t>(), cell0, orig, ng, nsp, (V4 *)pos,         \
                     (T *)box, (const T *)G, (V4 *)gsort)
  if (h->bin_dtype == AICA_FP64) AICA_GATHER(double);
  else AICA_GATHER(float);
#undef AICA_GATHER
  HIPCHK(hipGetLastError());
  return AICA_OK;
}

// Positions for pair export and counts, in the handle's buffer (these make no records and need no slot_base).
template <typename T>
static int gather_half(aica_dil *h, const void *pos_dev, hipStream_t st) {
  int rc = h->d_pos.ensure(sizeof(typename Vec4<T>::type) * std::max<int64_t>(h->n, 1));
  if (rc) return rc;
  return gather<T>(h, false, pos_dev, nullptr, 1, st, h->d_pos.p, nullptr);
}

// The handle's grow-only workspace for a force call (allocating on first use or growth).
template <typename T>
static int handle_ws(aica_dil *h, ForceWs &ws, hipStream_t st) {
  using V4 = typename Vec4<T>::type;
  const bool full = full_lists(h, h->n, sizeof(T));
  const int64_t n = h->n, ng = full ? h->nb.ng : h->grp.ng;
  int rc;
  if ((rc = h->d_pos.ensure(sizeof(V4) * std::max<int64_t>(n, 1)))) return rc;
  if (full) {
    if ((rc = h->d_box.ensure(sizeof(T) * 6 * std::max<int64_t>(ng, 1)))) return rc;
  } else {
    if ((rc = prepare_jpart(h, sizeof(T) * 4 * std::max<int64_t>(h->jtotal, 1), st))) return rc;
    if ((rc = h->d_own.ensure(sizeof(T) * 8 * std::max<int64_t>(n, 1)))) return rc;
  }
  if ((rc = h->d_gpart.ensure(sizeof(double) * 2 * std::max<int64_t>(ng, 1)))) return rc;
  if ((rc = h->d_gnp.ensure(16 * std::max<int64_t>(ng, 1)))) return rc;
  if ((rc = h->d_red.ensure(sizeof(double) * 8 * kRedBlocks))) return rc;
  ws.pos = h->d_pos.p;
  ws.box = h->d_box.p;
  ws.own = h->d_own.p;
  ws.jpart = h->d_jpart.p;
  ws.gpart = h->d_gpart.p;
  ws.gnp = h->d_gnp.p;
  ws.red = h->d_red.p;
  ws.epoch = h->epoch;
  return AICA_OK;
}

static int check_step(aica_dil *h, const void *pos_dev) {
  if (!h) return fail(AICA_E_INVAL, "handle is NULL");
  if (!h->bin_valid) return fail(AICA_E_INVAL, "aica_bin must succeed before this call");
  if (pos_dev != h->bin_pos) return fail(AICA_E_INVAL, "positions differ from the array passed to aica_bin");
  return AICA_OK;
}

// Gather, pair kernel, finalize and reductions of a force call on the workspace ws.
template <typename T>
static int forces_impl(aica_dil *h, const ForceWs &ws, const void *pos_dev, const int32_t *species, const LJTab &tab,
                       bool comp, void *forces_dev, double *uw_dev, int64_t *npairs_dev, hipStream_t st,
                       bool prof = true) {
  const bool full = full_lists(h, h->n, sizeof(T));
  const int64_t n = h->n, ng = full ? h->nb.ng : h->grp.ng;
  int rc;
  const bool was = h->profiling;
  h->profiling = was && prof;  // the timing events are created only where the call may allocate
  struct Restore {
    aica_dil *h;
    bool v;
    ~Restore() { h->profiling = v; }
  } restore{h, was};
  if ((rc = gather<T>(h, full, pos_dev, species, tab.nsp, st, ws.pos, full ? ws.box : nullptr))) return rc;
  {
    ProfScope ps(h, "pair_fwd", st);
    if (full) {
      if ((rc = launch_force<T>(h, ws, tab, comp, forces_dev, st))) return rc;
    } else {
      if ((rc = launch_pair<T, 0>(h, ws, tab, comp, st, 0, nullptr))) return rc;
    }
    h->wsteps_groups = ws.gnp == h->d_gnp.p ? ng : 0;  // the lane-pair diagnostic reads the handle's partials
  }
  {
    ProfScope ps(h, "finalize", st);
    if (!full && n > 0 && forces_dev) {
      constexpr bool C = sizeof(T) == 4;  // compensated sums exist in FP32 only
      if (comp)
        launch_finalize<T, C>(h, ws, forces_dev, st);
      else
        launch_finalize<T, false>(h, ws, forces_dev, st);
    }
    if (uw_dev || npairs_dev) {
      int64_t chunk;
      const int nb = red_blocks(ng, chunk);
      const double *gp = (const double *)ws.gpart;
      const unsigned long long *gn = (const unsigned long long *)ws.gnp;
      if (nb > 0)
        hipLaunchKernelGGL(k_reduce_uw_rows, dim3(nb), dim3(kRedThreads), 0, st, gp, gn, ng, chunk, (double *)ws.red);
      // with the full lists each pair is counted from both sides
      hipLaunchKernelGGL(k_reduce_uw, dim3(1), dim3(kRedThreads), 0, st, gp, gn, ng, (const double *)ws.red, nb, uw_dev,
                         npairs_dev, full ? 2 : 1);
    }
    HIPCHK(hipGetLastError());
  }
  return AICA_OK;
}

template <typename T>
static int forces_alloc(aica_dil *h, const void *pos_dev, const int32_t *species, const LJTab &tab, bool comp,
                        void *forces_dev, double *uw_dev, int64_t *npairs_dev, hipStream_t st) {
  ForceWs ws;
  int rc = handle_ws<T>(h, ws, st);
  if (rc) return rc;
  return forces_impl<T>(h, ws, pos_dev, species, tab, comp, forces_dev, uw_dev, npairs_dev, st);
}

int aica_forces(aica_dil *h, const void *pos_dev, const int32_t *species_dev, const aica_params *params,
                void *forces_dev, double *uw_dev, int64_t *npairs_dev, void *hip_stream) {
  int rc = check_step(h, pos_dev);
  if (rc) return rc;
  LJTab tab;
  if ((rc = build_tab(h, params, tab))) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  if (params->precision == AICA_FP32)
    return forces_alloc<float>(h, pos_dev, species_dev, tab, params->compensated != 0, forces_dev, uw_dev, npairs_dev, st);
  return forces_alloc<double>(h, pos_dev, species_dev, tab, false, forces_dev, uw_dev, npairs_dev, st);
}

// ---- aica_forces without allocation: every buffer of the call lies in this fixed array (one copy per GPU,
// held until the process ends).  Host code never passes the array's name to a kernel: it resolves the
// array's device address once per device (hipGetSymbolAddress) and uses that.
constexpr size_t kScratchBytes = (size_t)128 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mu;

static int scratch_address(int dev, void **out) {
  if (dev < 0 || dev >= kMaxDevices) return fail(AICA_E_INVAL, "device index out of range for the scratch array");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(AICA_E_HIP, "hipGetSymbolAddress returned no address for the scratch array");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return AICA_OK;
}

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

template <typename T>
static int forces_noalloc(aica_dil *h, const void *pos_dev, const int32_t *species, const LJTab &tab, bool comp,
                          void *forces_dev, double *uw_dev, int64_t *npairs_dev, hipStream_t st) {
  using V4 = typename Vec4<T>::type;
  const bool full = full_lists(h, h->n, sizeof(T));
  const int64_t n = h->n, ng = full ? h->nb.ng : h->grp.ng, J = h->jtotal;
  const size_t b_pos = align256(sizeof(V4) * std::max<int64_t>(n, 1));
  const size_t b_own = align256(sizeof(T) * 8 * std::max<int64_t>(n, 1));
  const size_t b_jpart = align256(sizeof(T) * 4 * std::max<int64_t>(J, 1));
  const size_t b_gpart = align256(sizeof(double) * 2 * std::max<int64_t>(h->grp.ng, 1));
  const size_t b_gnp = align256(16 * std::max<int64_t>(h->grp.ng, 1));
  const size_t b_red = align256(sizeof(double) * 8 * kRedBlocks);
  // What the half lists take decides for both whether a step fits, so that it does not depend on which lists run.  The
  // full lists take less: boxes in place of the records.
  const size_t b_box = align256(sizeof(T) * 6 * std::max<int64_t>(ng, 1));
  const size_t b_full = b_pos + b_box + 2 * align256(16 * std::max<int64_t>(ng, 1)) + b_red;
  const size_t need = std::max(b_pos + b_own + b_jpart + b_gpart + b_gnp + b_red, full ? b_full : 0);
  if (need > kScratchBytes)
    return fail(AICA_E_INVAL, "aica_forces_noalloc needs " + std::to_string(need) + " bytes of scratch for " +
                                  std::to_string(n) + " molecules; the fixed scratch holds " +
                                  std::to_string(kScratchBytes) + " (use aica_forces)");
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  char *base = nullptr;
  int rc = scratch_address(dev, (void **)&base);
  if (rc) return rc;
  ForceWs ws;
  ws.pos = base;
  if (full) {
    ws.box = base + b_pos;
    ws.gpart = base + b_pos + b_box;
    ws.gnp = (char *)ws.gpart + align256(16 * std::max<int64_t>(ng, 1));
    ws.red = (char *)ws.gnp + align256(16 * std::max<int64_t>(ng, 1));
  } else {
    ws.own = base + b_pos;
    ws.jpart = base + b_pos + b_own;
    ws.gpart = base + b_pos + b_own + b_jpart;
    ws.gnp = base + b_pos + b_own + b_jpart + b_gpart;
    ws.red = base + b_pos + b_own + b_jpart + b_gpart + b_gnp;
  }
  if (!full) {
    // the array keeps the last call's records: every record's tag is cleared (a fill kernel, no memset node)
    ws.epoch = 1;
    const int64_t words = (int64_t)(sizeof(T) * 4 * std::max<int64_t>(J, 1) / 4);
    hipLaunchKernelGGL((k_fill<uint32_t>), dim3(grid1d(words, 256)), dim3(256), 0, st, (uint32_t *)ws.jpart, words,
                       0xFFFFFFFFu);
    HIPCHK(hipGetLastError());
  }
  return forces_impl<T>(h, ws, pos_dev, species, tab, comp, forces_dev, uw_dev, npairs_dev, st, false);
}

int aica_forces_noalloc(aica_dil *h, const void *pos_dev, const int32_t *species_dev, const aica_params *params,
                        void *forces_dev, double *uw_dev, int64_t *npairs_dev, void *hip_stream) {
  int rc = check_step(h, pos_dev);
  if (rc) return rc;
  LJTab tab;
  if ((rc = build_tab(h, params, tab))) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  if (params->precision == AICA_FP32)
    return forces_noalloc<float>(h, pos_dev, species_dev, tab, params->compensated != 0, forces_dev, uw_dev, npairs_dev, st);
  return forces_noalloc<double>(h, pos_dev, species_dev, tab, false, forces_dev, uw_dev, npairs_dev, st);
}

int aica_pairs_export(aica_dil *h, const void *pos_dev, const aica_params *params, int64_t cap, int64_t *n_out,
                      int32_t *a, int32_t *b, int8_t *img, void *hip_stream) {
  int rc = check_step(h, pos_dev);
  if (rc) return rc;
  if (!n_out || cap < 0 || (cap > 0 && (!a || !b || !img))) return fail(AICA_E_INVAL, "bad output arrays");
  LJTab tab;
  if ((rc = build_tab(h, params, tab))) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  if ((rc = h->d_pairs.ensure(12 * std::max<int64_t>(cap, 1)))) return rc;
  if ((rc = h->d_pcount.ensure(64))) return rc;
  unsigned long long *pc = h->d_pcount.as<unsigned long long>();
  hipLaunchKernelGGL((k_fill<unsigned long long>), dim3(1), dim3(64), 0, st, pc, (int64_t)1, 0ull);
  if (params->precision == AICA_FP32) {
    if ((rc = gather_half<float>(h, pos_dev, st))) return rc;
    ForceWs ws;
    ws.pos = h->d_pos.p;
    if ((rc = launch_pair<float, 1>(h, ws, tab, false, st, cap, pc))) return rc;
  } else {
    if ((rc = gather_half<double>(h, pos_dev, st))) return rc;
    ForceWs ws;
    ws.pos = h->d_pos.p;
    if ((rc = launch_pair<double, 1>(h, ws, tab, false, st, cap, pc))) return rc;
  }
  unsigned long long cnt = 0;
  HIPCHK(hipMemcpyAsync(&cnt, pc, 8, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  *n_out = (int64_t)cnt;
  const int64_t k = std::min<int64_t>((int64_t)cnt, cap);
  if (k > 0) {
    std::vector<int32_t> buf(3 * k);
    HIPCHK(hipMemcpy(buf.data(), h->d_pairs.p, 12 * k, hipMemcpyDeviceToHost));
    for (int64_t i = 0; i < k; ++i) {
      int32_t x = buf[3 * i], y = buf[3 * i + 1], code = buf[3 * i + 2];
      int n0 = code / 9 - 1, n1 = (code / 3) % 3 - 1, n2 = code % 3 - 1;
      // d = x_i - x_j - t with t = image of the entry; report (min id, max id, image of that order)
      if (x > y) {
        std::swap(x, y);
        n0 = -n0;
        n1 = -n1;
        n2 = -n2;
      }
      a[i] = x;
      b[i] = y;
      img[3 * i] = (int8_t)n0;
      img[3 * i + 1] = (int8_t)n1;
      img[3 * i + 2] = (int8_t)n2;
    }
  }
  return AICA_OK;
}

int aica_forces_adjoint(aica_dil *h, const void *pos_dev, const int32_t *species_dev, const aica_params *params,
                        const void *grad_forces_dev, double grad_energy, void *grad_pos_dev, double *grad_eps_dev,
                        double *grad_sigma_dev, void *hip_stream);

int aica_pair_counts(aica_dil *h, const void *pos_dev, const aica_params *params, int32_t *counts_dev,
                     void *hip_stream) {
  int rc = check_step(h, pos_dev);
  if (rc) return rc;
  if (h->n > 0 && !counts_dev) return fail(AICA_E_INVAL, "counts_dev is NULL");
  LJTab tab;
  if ((rc = build_tab(h, params, tab))) return rc;
  hipStream_t st = (hipStream_t)hip_stream;
  if (h->n == 0) return AICA_OK;
  hipLaunchKernelGGL((k_fill<int32_t>), dim3(grid1d(h->n, 256)), dim3(256), 0, st, counts_dev, h->n, 0);
  if (params->precision == AICA_FP32) {
    if ((rc = gather_half<float>(h, pos_dev, st))) return rc;
    ForceWs ws;
    ws.pos = h->d_pos.p;
    if ((rc = launch_pair<float, 1>(h, ws, tab, false, st, -1, nullptr, counts_dev))) return rc;
  } else {
    if ((rc = gather_half<double>(h, pos_dev, st))) return rc;
    ForceWs ws;
    ws.pos = h->d_pos.p;
    if ((rc = launch_pair<double, 1>(h, ws, tab, false, st, -1, nullptr, counts_dev))) return rc;
  }
  HIPCHK(hipGetLastError());
  return AICA_OK;
}

int aica_dil_export(const aica_dil *h, int64_t *n, int32_t *c, int32_t *d, int8_t *img) {
  if (!h || !n) return fail(AICA_E_INVAL, "NULL argument");
  *n = (int64_t)h->pairs.size();
  if (!c) return AICA_OK;
  if (!d || !img) return fail(AICA_E_INVAL, "NULL output array");
  for (size_t i = 0; i < h->pairs.size(); ++i) {
    const CellPair &p = h->pairs[i];
    int32_t x = h->order[p.sc], y = h->order[p.sd];
    int n0 = p.img[0], n1 = p.img[1], n2 = p.img[2];
    if (x > y) {
      std::swap(x, y);
      n0 = -n0;
      n1 = -n1;
      n2 = -n2;
    }
    c[i] = x;
    d[i] = y;
    img[3 * i] = (int8_t)n0;
    img[3 * i + 1] = (int8_t)n1;
    img[3 * i + 2] = (int8_t)n2;
  }
  return AICA_OK;
}

int aica_bin_export(const aica_dil *h, int32_t *cell_of, int32_t *order, int64_t *cell_count) {
  if (!h) return fail(AICA_E_INVAL, "handle is NULL");
  if (!h->bin_valid) return fail(AICA_E_INVAL, "aica_bin must succeed first");
  const int64_t n = h->n, nc = h->geo.nc;
  if (cell_of && n > 0) {
    std::vector<int32_t> cs(n), pm(n);
    HIPCHK(hipMemcpy(cs.data(), h->d_cell_sorted.p, 4 * n, hipMemcpyDeviceToHost));
    HIPCHK(hipMemcpy(pm.data(), h->d_perm.p, 4 * n, hipMemcpyDeviceToHost));
    for (int64_t s = 0; s < n; ++s) cell_of[pm[s]] = h->order[cs[s]];
  }
  if (order && n > 0) HIPCHK(hipMemcpy(order, h->d_perm.p, 4 * n, hipMemcpyDeviceToHost));
  if (cell_count) {
    std::vector<int32_t> cs(nc + 1);
    HIPCHK(hipMemcpy(cs.data(), h->d_cell_start.p, 4 * (nc + 1), hipMemcpyDeviceToHost));
    for (int64_t s = 0; s < nc; ++s) cell_count[h->order[s]] = cs[s + 1] - cs[s];
  }
  return AICA_OK;
}

int aica_dil_info(const aica_dil *h, aica_info *info) {
  if (!h || !info) return fail(AICA_E_INVAL, "NULL argument");
  memset(info, 0, sizeof *info);
  info->n_cells = h->geo.nc;
  info->n_dil = (int64_t)h->pairs.size();
  info->n_groups = h->groups_ready ? h->grp.ng : 0;
  info->n_group_pairs = h->groups_ready ? h->grp.e_off[h->grp.ng] : 0;
  info->n_molecules = h->n;
  info->n_jslots = h->jtotal;
  info->mesh_volume = h->geo.total_volume;
  info->build_seconds = h->build_seconds;
  info->group_seconds = h->group_seconds;
  info->lane_steps = -1;
  info->located_ball = h->located[0];
  info->located_record = h->located[1];
  info->located_search = h->located[2];
  return AICA_OK;
}

int aica_work_stats(const aica_dil *h, int64_t *dil_candidates, int64_t *lane_pairs) {
  if (!h) return fail(AICA_E_INVAL, "handle is NULL");
  if (!h->bin_valid) return fail(AICA_E_INVAL, "aica_bin must succeed first");
  const int64_t nc = h->geo.nc, ng = h->wsteps_groups;
  std::vector<int32_t> cs(nc + 1);
  HIPCHK(hipMemcpy(cs.data(), h->d_cell_start.p, 4 * (nc + 1), hipMemcpyDeviceToHost));
  if (dil_candidates) {
    int64_t cand = 0;
    for (int64_t s = 0; s < nc; ++s) {
      const int64_t n = cs[s + 1] - cs[s];
      cand += n * (n - 1) / 2;
    }
    for (const CellPair &p : h->pairs) cand += (int64_t)(cs[p.sc + 1] - cs[p.sc]) * (cs[p.sd + 1] - cs[p.sd]);
    *dil_candidates = cand;
  }
  if (lane_pairs) {
    // wave-steps counted by the last forward pair kernel, 64 lane-pair evaluations each
    if (ng == 0) return fail(AICA_E_INVAL, "aica_forces must run after aica_bin first");
    std::vector<unsigned long long> gn(2 * ng);
    HIPCHK(hipMemcpy(gn.data(), h->d_gnp.p, 16 * ng, hipMemcpyDeviceToHost));
    int64_t lp = 0;
    for (int64_t a = 0; a < ng; ++a) lp += 64 * (int64_t)gn[2 * a + 1];
    *lane_pairs = lp;
  }
  return AICA_OK;
}

int aica_profile(aica_dil *h, int32_t enable) {
  if (!h) return fail(AICA_E_INVAL, "handle is NULL");
  h->profiling = enable != 0;
  return AICA_OK;
}

int aica_profile_read(aica_dil *h, const char *kernel, double *ms_total, int64_t *launches, int32_t reset) {
  if (!h || !kernel) return fail(AICA_E_INVAL, "NULL argument");
  Timer &t = h->timers[kernel];
  for (auto &ev : t.pending) {
    HIPCHK(hipEventSynchronize(ev.second));
    float ms = 0;
    HIPCHK(hipEventElapsedTime(&ms, ev.first, ev.second));
    t.ms += ms;
    (void)hipEventDestroy(ev.first);
    (void)hipEventDestroy(ev.second);
  }
  t.pending.clear();
  if (ms_total) *ms_total = t.ms;
  if (launches) *launches = t.launches;
  if (reset) {
    t.ms = 0;
    t.launches = 0;
  }
  return AICA_OK;
}


#include "aica_adjoint.inc"
