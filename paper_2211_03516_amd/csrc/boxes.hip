// Lab-box tiling of the forward projection (Sec. 2.4 of Webber et al.) and
// of the dose deposit (Sec. 2.5).
//
// The vial turns about +z, so every ray sample has a fixed position in the
// lab frame; only its volume-frame position depends on the angle.  At setup
// the resin samples of every ray are cut into segments, one per lab-frame
// box of B^3 voxels that they cross, and each segment is stored as a compact
// record: its first sample's lab position relative to the box, its
// direction, its sample count and the attenuated weight of its first sample.
// Both operators then run one workgroup per (box, angle): the box, rotated
// into the volume frame, covers a small footprint of the padded grid (at
// most ~(B sqrt 2 + 3)^2 (B + 2) cells), which the workgroup stages in LDS
// (forward: the volume; deposit: a fixed-point accumulator) while it marches
// all segments of the box -- about 40 samples per voxel at the full-optics
// workload.  The per-sample work (position, trilinear weights of Sec. 2.2,
// Beer-Lambert attenuation) is the same as in the ray-driven kernels; only
// the place where the eight corner values are read or added changes, from
// global memory to LDS.

#include <algorithm>
#include <atomic>
#include <cmath>
#include <new>
#include <thread>
#include <type_traits>

#include "launch_cut.h"
#include "vam_internal.h"

namespace vam {

constexpr int kBox = 12;  // default lab box edge (fastest measured for both operators)

// Compile-time footprints for the supported box edges: row pitch WXY, WZ
// slices (the largest footprint of a rotated box: extent B(|cos| + |sin|) <=
// B sqrt 2 cells in x and y plus the rounding margin and the +1 corner, B + 2
// in z).
template <int B>
struct Fixed;
template <>
struct Fixed<8> {
  static constexpr int WXY = 14, WZ = 10;
};
template <>
struct Fixed<12> {
  static constexpr int WXY = 19, WZ = 14;
};
template <>
struct Fixed<16> {
  static constexpr int WXY = 25, WZ = 18;
};

bool supported_box_edge(int B) { return B == 8 || B == 12 || B == 16; }

static void footprint_bound(int B, int px, int py, int pz, int& wxy, int& wz) {
  wxy = std::min((int)std::floor(B * std::sqrt(2.0) + 3.02), std::max(px, py));
  wz = std::min(B + 2, pz);
}

__device__ inline int box_of(const BoxGrid& G, double x, double y, double z) {
  int bx = (int)floor((x - G.x0) / G.B);
  int by = (int)floor((y - G.y0) / G.B);
  int bz = (int)floor((z - G.z0) / G.B);
  bx = min(max(bx, 0), G.nbx - 1);
  by = min(max(by, 0), G.nby - 1);
  bz = min(max(bz, 0), G.nbz - 1);
  return (bz * G.nby + by) * G.nbx + bx;
}

// Coordinates of a linear box number in one word (24 bits for x and y, whose
// count follows the vial, 16 for z): the box kernels unpack them with shifts
// instead of two divisions in every wave.
static inline int64_t pack_box(const BoxGrid& G, int box) {
  return (int64_t)(box % G.nbx) | (int64_t)(box / G.nbx % G.nby) << 24 | (int64_t)(box / (G.nbx * G.nby)) << 48;
}
__device__ inline int box_x(int64_t id) { return (int)(id & 0xffffff); }
__device__ inline int box_y(int64_t id) { return (int)(id >> 24 & 0xffffff); }
__device__ inline int box_z(int64_t id) { return (int)(id >> 48); }

// Walk the z-clipped samples of a ray in the lab frame (FP64, sample k at
// e + (k + 1/2) step d) and call emit(box, first k, count, rank) once per
// maximal run of samples in one box (SPLIT: in one box and one z cell); rank
// numbers the runs of a ray from 0 in marching order.
__device__ inline int z_cell(const BoxGrid& G, double z) { return min(max((int)floor(z - G.z0), 0), G.nbz * G.B - 1); }

template <bool SPLIT, class F>
__device__ inline void walk_segments(const BoxGrid& G, const RayRec& R, const double* o, double step,
                                     F emit) {
  if (R.n <= 0) return;
  int cur = -1, cell = 0, start = 0, rank = 0;
  for (int k = R.k0; k < R.k0 + R.n; ++k) {
    const double s = (k + 0.5) * step;
    const int b = box_of(G, o[0] + s * o[3], o[1] + s * o[4], o[2] + s * o[5]);
    const int c = SPLIT ? z_cell(G, o[2] + s * o[5]) : 0;
    if (b != cur || c != cell) {
      if (cur >= 0) emit(cur, start, k - start, rank++);
      cur = b;
      cell = c;
      start = k;
    }
  }
  if (cur >= 0) emit(cur, start, R.k0 + R.n - start, rank);
}

template <bool SPLIT>
__global__ void k_seg_count(BoxGrid G, const RayRec* rays, const double* ray64, int64_t n_rays, double step,
                            int* box_count, int* ray_nseg) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rays) return;
  int n = 0;
  walk_segments<SPLIT>(G, rays[r], ray64 + r * kRay64Fields, step, [&](int b, int, int, int) {
    atomicAdd(box_count + b, 1);
    ++n;
  });
  if (ray_nseg) ray_nseg[r] = n;
}

template <bool SPLIT>
__global__ void k_seg_fill(BoxGrid G, const RayRec* rays, const double* ray64, int64_t n_rays, double step,
                           const int* box_off, int* cursor, int4* segs) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rays) return;
  walk_segments<SPLIT>(G, rays[r], ray64 + r * kRay64Fields, step, [&](int b, int k, int n, int rank) {
    const int slot = box_off[b] + atomicAdd(cursor + b, 1);
    segs[slot] = make_int4((int)r, k, n, rank);
  });
}

// Compact records of the (sorted) segments {ray, first k, count, rank} of
// every box, one workgroup per box.  The lab position of the segment's
// middle sample m = (count - 1) / 2 (rounded down) is formed in FP64 and
// stored relative to the box (x, y from its centre, z from its bottom face),
// so FP32 keeps it to ~1e-6 voxel, and the kernels step from it by at most
// half the segment (the rounding of the direction grows with the distance
// stepped); the weight is (T1 T2 / n_pupil) step exp(-alpha s) at the
// segment's first sample, rounded once.
//   pw = (x_m - xc, y_m - yc, z_m - zb, weight), dn = (d_x, d_y, d_z, count;
//   deposit: plus 2^24 times the z cell of its samples in the box),
//   idx = pixel (deposit) or partial-sum slot rank * n_rays + ray (forward:
//   lanes marching neighbouring rays write neighbouring slots).
constexpr int kCountBits = 24;  // a segment has fewer than 2^24 samples
__device__ inline int seg_count(const float4& dn) { return __float_as_int(dn.w) & ((1 << kCountBits) - 1); }
__device__ inline int seg_z_cell(const float4& dn) { return __float_as_int(dn.w) >> kCountBits; }

__global__ void k_seg_pack(BoxGrid G, const int64_t* box_id, const int* box_begin, const int4* segs,
                           const double* ray64, int n_rays, double step, double alpha, int npix,
                           int forward, float4* pw, float4* dn, int* idx) {
  const int b = blockIdx.x;
  const int64_t box = box_id[b];
  const int bx = box_x(box), by = box_y(box), bz = box_z(box);
  const double xc = G.x0 + (bx + 0.5) * G.B, yc = G.y0 + (by + 0.5) * G.B, zb = G.z0 + (double)bz * G.B;
  for (int i = box_begin[b] + threadIdx.x; i < box_begin[b + 1]; i += blockDim.x) {
    const int4 sg = segs[i];
    const double* o = ray64 + (int64_t)sg.x * kRay64Fields;
    const double s = (sg.y + 0.5) * step;
    const double sm = (sg.y + (sg.z - 1) / 2 + 0.5) * step;
    pw[i] = make_float4((float)(o[0] + sm * o[3] - xc), (float)(o[1] + sm * o[4] - yc),
                        (float)(o[2] + sm * o[5] - zb), (float)(o[8] * step * exp(-alpha * s)));
    const int iz = forward ? 0 : min(max(z_cell(G, o[2] + s * o[5]) - bz * G.B, 0), G.B - 1);
    dn[i] = make_float4((float)o[3], (float)o[4], (float)o[5], __int_as_float(sg.z | iz << kCountBits));
    idx[i] = forward ? sg.w * n_rays + sg.x : sg.x % npix;
  }
}

// ------------------------------------------------- fixed-point bound ------

// Samples per lab-frame unit cell (x, y from -R, padded z), from the same
// FP64 positions the segment records are made of.
__global__ void k_lab_count(const RayRec* rays, const double* ray64, int64_t n_rays, double step, double x0,
                            double z0, int ncx, int ncz, unsigned* count) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rays) return;
  const RayRec R = rays[r];
  const double* o = ray64 + r * kRay64Fields;
  for (int k = R.k0; k < R.k0 + R.n; ++k) {
    const double s = (k + 0.5) * step;
    const int ix = min(max((int)floor(o[0] + s * o[3] - x0), 0), ncx - 1);
    const int iy = min(max((int)floor(o[1] + s * o[4] - x0), 0), ncx - 1);
    const int iz = min(max((int)floor(o[2] + s * o[5] - z0), 0), ncz - 1);
    atomicAdd(count + ((int64_t)iz * ncx + iy) * ncx + ix, 1u);
  }
}

// Per-box bound of the fixed-point deposit: the most samples OF THE BOX in
// any 4 x 4 x 3 block of lab-frame unit cells.  The box's samples are the
// samples inside its B^3 cells, so that is the largest window sum of the
// cell counts clipped to the box; a voxel's turned support (a 2 x 2 x 2
// cube: at most 2 sqrt 2 wide in x and y) always fits in such a block, so
// at any angle the box adds at most that many samples into one LDS cell.
// One workgroup per box.
__global__ void k_box_supp(BoxGrid G, const int64_t* box_id, const unsigned* count, int ncx, int ncz, int* supp) {
  __shared__ unsigned s_max;
  if (threadIdx.x == 0) s_max = 0u;
  __syncthreads();
  const int64_t box = box_id[blockIdx.x];
  const int bx = box_x(box), by = box_y(box), bz = box_z(box);
  const int x0 = bx * G.B, y0 = by * G.B, z0 = bz * G.B;
  const int x1 = min(x0 + G.B, ncx), y1 = min(y0 + G.B, ncx), z1 = min(z0 + G.B, ncz);
  // window anchors (lowest cell) from 3 (x, y) or 2 (z) cells before the box
  const int nwx = G.B + 3, nwz = G.B + 2;
  unsigned best = 0;
  for (int w = threadIdx.x; w < nwx * nwx * nwz; w += blockDim.x) {
    const int wx = x0 - 3 + w % nwx, wy = y0 - 3 + (w / nwx) % nwx, wz = z0 - 2 + w / (nwx * nwx);
    unsigned sum = 0;
    for (int z = max(wz, z0); z < min(wz + 3, z1); ++z)
      for (int y = max(wy, y0); y < min(wy + 4, y1); ++y)
        for (int x = max(wx, x0); x < min(wx + 4, x1); ++x) sum += count[((int64_t)z * ncx + y) * ncx + x];
    best = max(best, sum);
  }
  atomicMax(&s_max, best);
  __syncthreads();
  if (threadIdx.x == 0) supp[blockIdx.x] = (int)min(max(s_max, 1u), 0x3fffffffu);
}

// Per-box n_supp of the fixed-point deposit (synchronises the stream).
static vam_status support_bound(vam_geometry* h, const BoxGrid& G, hipStream_t s) {
  const double R = h->desc.r_inner + 1.0;
  const int ncx = (int)std::ceil(2.0 * R), ncz = h->pz;
  const int64_t ncell = (int64_t)ncx * ncx * ncz;
  unsigned* count = nullptr;
  VAM_HIP_TRY(dev_alloc((void**)&count, ncell * sizeof(unsigned)), "allocating lab cell counts");
  hipError_t e = hipMemsetAsync(count, 0, ncell * sizeof(unsigned), s);
  if (e == hipSuccess) {
    const double z0 = -(0.5 * (h->desc.nz - 1) + kPad);
    hipLaunchKernelGGL(k_lab_count, dim3((unsigned)((h->n_rays + 255) / 256)), dim3(256), 0, s, h->rays, h->ray64,
                       h->n_rays, h->desc.step, -R, z0, ncx, ncz, count);
    if (h->n_boxes > 0)
      hipLaunchKernelGGL(k_box_supp, dim3((unsigned)h->n_boxes), dim3(256), 0, s, G, h->box_id, count, ncx, ncz,
                         h->box_supp);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(count);
  if (e != hipSuccess) return hip_check(e, "bounding samples per voxel support");
  // a 4 x 4 x 3 block of cells meets at most 2 boxes along each axis (the
  // box edge is at least 8), so all boxes together put at most 8 x the
  // largest box_supp samples into one voxel's support
  std::vector<int> hb(std::max(h->n_boxes, 1), 0);
  if (h->n_boxes > 0) {
    e = hipMemcpy(hb.data(), h->box_supp, h->n_boxes * sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_check(e, "reading the support bounds");
  }
  h->supp_bound = 8 * (int64_t)*std::max_element(hb.begin(), hb.end());
  return VAM_OK;
}

// ------------------------------------------------------ decomposition ------

static void free_table(SegTable& t) {
  void* ptrs[] = {t.pw, t.dn, t.idx, t.box_begin};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  t = SegTable{};
}

void free_boxes(vam_geometry* h) {
  free_table(h->seg_dep);
  free_table(h->seg_fwd);
  if (h->vol_turn) (void)hipFree(h->vol_turn);
  h->vol_turn = nullptr;
  h->vol_turn_captured = 0;
  void* ptrs[] = {h->box_id, h->box_supp, h->ray_nseg, h->seg_part};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  h->box_id = nullptr;
  h->box_supp = nullptr;
  h->ray_nseg = nullptr;
  h->seg_part = nullptr;
  h->seg_part_angles = 0;
  h->n_boxes = 0;
  h->n_segments = 0;
  h->max_seg_per_ray = 0;
  h->boxes_ready = 0;
}

static vam_status alloc_table(SegTable& t, int64_t n) {
  t.n = n;
  const int64_t m = std::max<int64_t>(n, 1);
  VAM_HIP_TRY(dev_alloc((void**)&t.pw, m * sizeof(float4)), "allocating segment records");
  VAM_HIP_TRY(dev_alloc((void**)&t.dn, m * sizeof(float4)), "allocating segment records");
  VAM_HIP_TRY(dev_alloc((void**)&t.idx, m * sizeof(int)), "allocating segment records");
  return VAM_OK;
}

// Order of the segments inside a box, which decides which lanes march
// together (host sort keys; measured orders, see vam_set_variant op 4):
//  0: by ray -- neighbouring lanes handle neighbouring pixels;
//  1: by decreasing length -- lanes of a wave march similar lengths;
//  2: by pixel parity class (u mod 2, v mod 2), then ray -- the lanes of
//     a wave handle pixels two apart, whose trilinear stencils are disjoint;
//  3, 4: the same with classes (u mod m, v mod m), m = 3, 4;
//  5: by a hash of the ray index (lanes at unrelated positions);
//  6: by pixel, then pupil sample -- the rays of one pixel, which meet at
//     the focus plane, go to neighbouring lanes;
//  7, 8: order 3, then each run of 1024 (7) or 2048 (8) consecutive
//     segments by decreasing length in steps of two samples (a stable sort:
//     equal steps keep their class order), so that the 64 lanes of a wave
//     march similar lengths and the waves of a workgroup get equal shares;
//  9: by pupil sample, then pixel column u, then row v -- neighbouring
//     lanes march rays one pixel apart in z, which does not turn;
//  10: by class (u mod 3, v mod 2), then ray (lanes three pixels apart
//     along a row, rows two apart);
//  11, 12, 13: order 10, then the whole box (11) or each run of 512 (12) or
//     2048 (13) consecutive segments by decreasing length (the plane-by-plane
//     deposit at 256^3: runs of 512 / 2048 segments 118 / 107 ms, the whole box
//     105);
//  14, 15, 16: by ray, then each run of 256 (14) or 1024 (15) segments, or
//     the whole box (16), by decreasing length in steps of two samples
//     (ties keep the ray order).
//
// Segments of one ray in one box (the deposit's, cut at z cells) follow in
// marching order, so that the order never depends on the fill kernel's
// scheduling.  Boxes are sorted by up to 16 threads, with each key formed
// once (256^3, two tables: 4.0 s a geometry on one thread, now 0.47).  False if host memory ran
// out.
static bool sort_segments(std::vector<int4>& hs, const std::vector<int>& begin, int order, int nu, int nv, int np) {
  auto key = [&](const int4& s, int ord) -> int64_t {
    const int r = s.x;
    const int u = r % nu, v = (r / nu) % nv;
    if (ord == 1) return ((int64_t)(0x7fffffff - s.z) << 32) | (uint32_t)r;
    if (ord >= 2 && ord <= 4) return ((int64_t)((v % ord) * ord + (u % ord)) << 32) | (uint32_t)r;
    if (ord == 6) return (int64_t)(r % (nu * nv)) * np + r / (nu * nv);
    if (ord == 9) return ((int64_t)(r / (nu * nv)) * nu + u) * nv + v;
    if (ord == 10) return ((int64_t)((v % 2) * 3 + (u % 3)) << 32) | (uint32_t)r;
    if (ord == 5) {
      uint64_t x = (uint64_t)r + 0x9e3779b97f4a7c15ull;  // SplitMix64 finaliser
      x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
      x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
      return (int64_t)((x ^ (x >> 31)) >> 1);
    }
    return r;
  };
  const int korder = (order == 7 || order == 8) ? 3 : (order >= 11 && order <= 13) ? 10 : order >= 14 ? 0 : order;
  const int run = (order == 7 || order == 15) ? 1024 : (order == 8 || order == 13) ? 2048
                : order == 12 ? 512 : order == 14 ? 256 : (order == 11 || order == 16) ? 0x7fffffff : 0;
  struct Item {
    int64_t key;
    int4 seg;
  };
  auto by_key = [](const Item& x, const Item& y) { return x.key != y.key ? x.key < y.key : x.seg.y < y.seg.y; };
  auto by_length = [&](const Item& x, const Item& y) {
    const int lx = x.seg.z >> 1, ly = y.seg.z >> 1;
    return lx != ly ? lx > ly : by_key(x, y);
  };
  const size_t n_boxes = begin.size() - 1;
  std::atomic<size_t> next{0};
  std::atomic<bool> ok{true};
  auto work = [&]() {
    try {
      std::vector<Item> items;
      for (size_t i = next++; ok && i < n_boxes; i = next++) {
        items.resize(begin[i + 1] - begin[i]);
        for (size_t k = 0; k < items.size(); ++k) items[k] = {key(hs[begin[i] + k], korder), hs[begin[i] + k]};
        if (run == 0x7fffffff) {
          std::sort(items.begin(), items.end(), by_length);
        } else {
          std::sort(items.begin(), items.end(), by_key);
          for (size_t g = 0; run && g < items.size(); g += run)
            std::sort(items.begin() + g, items.begin() + std::min(g + run, items.size()), by_length);
        }
        for (size_t k = 0; k < items.size(); ++k) hs[begin[i] + k] = items[k].seg;
      }
    } catch (const std::bad_alloc&) {
      ok = false;
    }
  };
  // a thread that cannot be started leaves its boxes to the others
  std::vector<std::thread> threads;
  const unsigned n_threads = std::min({16u, std::thread::hardware_concurrency(), (unsigned)(n_boxes / 8 + 1)});
  try {
    for (unsigned t = 1; t < n_threads; ++t) threads.emplace_back(work);
  } catch (const std::exception&) {
  }
  work();
  for (std::thread& t : threads) t.join();
  return ok;
}

// One table of segments, in the order `order` inside each box, packed into
// compact records: the forward's or the deposit's runs of samples in a box, or
// (SPLIT, deposit) runs that also end where the z cell changes (z does not turn,
// so a segment then has one z cell at every angle).  ids: the boxes that hold
// segments (the same for all); host: the sorted segments, for the caller.
// Synchronises the stream.  Host memory that runs out is thrown.
template <bool SPLIT>
static vam_status build_table(vam_geometry* h, const BoxGrid& G, bool deposit, SegTable& t, std::vector<int64_t>& ids,
                              std::vector<int4>& host, hipStream_t s) {
  const vam_geometry_desc& D = h->desc;
  const int nb_all = G.nbx * G.nby * G.nbz;
  int* ray_nseg = deposit ? nullptr : h->ray_nseg;
  // staging: box counts, offsets and cursors, then the unsorted segments
  struct Staging {
    int* count = nullptr;
    int4* segs = nullptr;
    void release() {
      if (count) (void)hipFree(count);
      if (segs) (void)hipFree(segs);
      count = nullptr;
      segs = nullptr;
    }
    ~Staging() { release(); }
  } staging;
  int*& count = staging.count;
  int4*& segs = staging.segs;
  auto release = [&]() { staging.release(); };
  hipError_t e = dev_alloc((void**)&count, 2 * (int64_t)nb_all * sizeof(int));
  if (e != hipSuccess) return hip_check(e, "allocating box counts");
  int* off = count + nb_all;
  e = hipMemsetAsync(count, 0, nb_all * sizeof(int), s);
  const int threads = 256;
  const unsigned blocks = (unsigned)((h->n_rays + threads - 1) / threads);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_seg_count<SPLIT>, dim3(blocks), dim3(threads), 0, s, G, h->rays, h->ray64, h->n_rays, D.step,
                       count, ray_nseg);
    e = hipGetLastError();
  }
  std::vector<int> hc(nb_all), ns(deposit ? 0 : h->n_rays);
  if (e == hipSuccess) e = hipMemcpyAsync(hc.data(), count, nb_all * sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess && !deposit)
    e = hipMemcpyAsync(ns.data(), ray_nseg, h->n_rays * sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    release();
    return hip_check(e, "counting box segments");
  }
  std::vector<int> hoff(nb_all), begin;
  ids.clear();
  int64_t total = 0;
  for (int b = 0; b < nb_all; ++b) {
    hoff[b] = (int)std::min<int64_t>(total, 0x7fffffff);
    if (hc[b] > 0) {
      ids.push_back(pack_box(G, b));
      begin.push_back((int)std::min<int64_t>(total, 0x7fffffff));
    }
    total += hc[b];
  }
  begin.push_back((int)std::min<int64_t>(total, 0x7fffffff));
  if (total >= 0x7fffffffLL) {
    release();
    return fail(VAM_ERR_UNSUPPORTED, "more than 2^31 ray segments");
  }
  if (!deposit) {
    // forward partial-sum slots rank * n_rays + ray must be 32-bit offsets
    h->max_seg_per_ray = ns.empty() ? 0 : *std::max_element(ns.begin(), ns.end());
    if ((int64_t)h->max_seg_per_ray * h->n_rays >= 0x7fffffffLL) {
      release();
      return fail(VAM_ERR_UNSUPPORTED, "more than 2^31 forward partial-sum slots per angle");
    }
  }
  e = dev_alloc((void**)&segs, std::max<int64_t>(total, 1) * sizeof(int4));
  if (e == hipSuccess) e = dev_alloc((void**)&t.box_begin, begin.size() * sizeof(int));
  if (e == hipSuccess) e = hipMemcpyAsync(off, hoff.data(), nb_all * sizeof(int), hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(t.box_begin, begin.data(), begin.size() * sizeof(int), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipMemsetAsync(count, 0, nb_all * sizeof(int), s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_seg_fill<SPLIT>, dim3(blocks), dim3(threads), 0, s, G, h->rays, h->ray64, h->n_rays, D.step,
                       off, count, segs);
    e = hipGetLastError();
  }
  host.resize(std::max<int64_t>(total, 1));
  if (e == hipSuccess) e = hipMemcpyAsync(host.data(), segs, total * sizeof(int4), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    release();
    return hip_check(e, "filling box segments");
  }
  h->n_boxes = (int)ids.size();
  if (!h->box_id) {
    e = dev_alloc((void**)&h->box_id, std::max<size_t>(ids.size(), 1) * sizeof(int64_t));
    if (e == hipSuccess && !ids.empty())
      e = hipMemcpyAsync(h->box_id, ids.data(), ids.size() * sizeof(int64_t), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) {
      release();
      return hip_check(e, "listing the boxes");
    }
  }
  vam_status st = alloc_table(t, total);
  if (st != VAM_OK) {
    release();
    return st;
  }
  // (the sort also makes the order independent of the scheduling of the fill
  // kernel)
  if (!sort_segments(host, begin, deposit ? h->seg_order : h->seg_order_fwd, D.n_u, D.n_v, D.n_pupil)) {
    release();
    return fail(VAM_ERR_OUT_OF_MEMORY, "sorting the box segments: out of host memory");
  }
  e = hipMemcpyAsync(segs, host.data(), total * sizeof(int4), hipMemcpyHostToDevice, s);
  if (e == hipSuccess && h->n_boxes > 0) {
    hipLaunchKernelGGL(k_seg_pack, dim3((unsigned)h->n_boxes), dim3(256), 0, s, G, h->box_id, t.box_begin, segs,
                       h->ray64, (int)h->n_rays, D.step, D.alpha, D.n_u * D.n_v, deposit ? 0 : 1, t.pw, t.dn, t.idx);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  release();
  if (e != hipSuccess) return hip_check(e, "packing box segments");
  host.resize(total);
  return VAM_OK;
}

// Build the decomposition into the handle (everything it allocates is
// recorded in the handle as soon as it exists, so free_boxes releases it
// on any failure).  Synchronises the stream.
static vam_status build_boxes_into(vam_geometry* h, hipStream_t s) {
  const vam_geometry_desc& D = h->desc;
  BoxGrid G;
  G.B = h->box_edge > 0 ? h->box_edge : kBox;
  const double R = D.r_inner + 1.0;
  G.x0 = -R;
  G.y0 = -R;
  G.z0 = -(0.5 * (D.nz - 1) + kPad);  // lab z of padded grid coordinate 0
  G.nbx = (int)std::ceil(2.0 * R / G.B);
  G.nby = G.nbx;
  G.nbz = (int)std::ceil((double)h->pz / G.B);
  h->boxes = G;
  VAM_HIP_TRY(dev_alloc((void**)&h->ray_nseg, h->n_rays * sizeof(int)), "allocating segment counts");
  std::vector<int64_t> ids;
  std::vector<int4> hs;
  vam_status st = build_table<false>(h, G, false, h->seg_fwd, ids, hs, s);
  if (st != VAM_OK) return st;
  h->n_segments = (int64_t)hs.size();
  {
    // the most samples of one pixel over all its rays (bounds the
    // fixed-point forward's sums)
    const int npix = D.n_u * D.n_v;
    std::vector<int64_t> per(npix, 0);
    for (const int4& sg : hs) per[sg.x % npix] += sg.z;
    h->pix_samples_max = per.empty() ? 0 : *std::max_element(per.begin(), per.end());
  }
  // The deposit's segments cut at z cells are about twice as many where rays
  // climb.  Where they are too many, or memory is short of them, the deposit takes
  // whole runs, one angle at a time (see k_back_box).
  auto deposit_table = [&](auto build) {
    try {
      return build();
    } catch (const std::bad_alloc&) {
      return fail(VAM_ERR_OUT_OF_MEMORY, "building the deposit's segments: out of host memory");
    }
  };
  h->deposit_whole = 0;
  st = deposit_table([&] { return build_table<true>(h, G, true, h->seg_dep, ids, hs, s); });
  if (st == VAM_ERR_UNSUPPORTED || st == VAM_ERR_OUT_OF_MEMORY) {
    (void)hipGetLastError();  // handled here
    clear_error();
    free_table(h->seg_dep);
    std::vector<int4>().swap(hs);
    h->deposit_whole = 1;
    st = deposit_table([&] { return build_table<false>(h, G, true, h->seg_dep, ids, hs, s); });
  }
  if (st != VAM_OK) return st;
  VAM_HIP_TRY(dev_alloc((void**)&h->box_supp, std::max(h->n_boxes, 1) * sizeof(int)), "allocating support bounds");
  st = support_bound(h, G, s);
  if (st != VAM_OK) return st;
  int wxy, wz;
  footprint_bound(G.B, h->px, h->py, h->pz, wxy, wz);
  h->box_cells = wxy * wxy * wz;
  return VAM_OK;
}

vam_status build_boxes(vam_geometry* h, hipStream_t s) {
  free_boxes(h);
  vam_status st;
  try {
    st = build_boxes_into(h, s);
  } catch (const std::bad_alloc&) {
    st = fail(VAM_ERR_OUT_OF_MEMORY, "building the box decomposition: out of host memory");
  }
  if (st != VAM_OK) {
    free_boxes(h);  // nothing half-built stays behind; boxes_ready stays 0
    return st;
  }
  h->boxes_ready = 1;
  return VAM_OK;
}

// ---------------------------------------------------------- launch data ----

struct BoxParams {
  BoxGrid G;
  int nboxes, na;      // work items of the launch: boxes x angles
  int xcd;             // work order (see work_item)
  SegTable seg;
  const int* box_begin;
  const int64_t* box_id;
  const int* box_supp; // fixed-point deposit: per-box n_supp
  int wxy_max, wz_max;
  int npix;            // n_u * n_v
  unsigned per_npix;   // 2^32 / npix, rounded down (at most 2^32 - 1)
  int px, py, pz;
  double w_coef;       // step / n_pupil: no sample weight exceeds it times |P|
  // one-angle forward: angle a is member a / turn_stride of representative
  // a % turn_stride; member0's turned volume comes first, the others follow
  int turn_stride, member0;
};

static BoxParams box_params(const vam_geometry* h, const SegTable& t, int na, int xcd) {
  BoxParams Bp;
  Bp.G = h->boxes;
  Bp.nboxes = h->n_boxes;
  Bp.na = na;
  Bp.xcd = xcd;
  Bp.seg = t;
  Bp.box_begin = t.box_begin;
  Bp.box_id = h->box_id;
  Bp.box_supp = h->box_supp;
  footprint_bound(h->boxes.B, h->px, h->py, h->pz, Bp.wxy_max, Bp.wz_max);
  Bp.npix = h->desc.n_u * h->desc.n_v;
  Bp.per_npix = (unsigned)std::min<uint64_t>((uint64_t(1) << 32) / (unsigned)Bp.npix, 0xffffffffu);
  Bp.px = h->px;
  Bp.py = h->py;
  Bp.pz = h->pz;
  Bp.w_coef = h->desc.step / h->desc.n_pupil;
  Bp.turn_stride = h->desc.n_angles;
  Bp.member0 = 0;
  return Bp;
}

// Pixel of a segment's slot (rank * n_rays + pupil * npix + pixel): slot modulo
// npix, by the reciprocal (the quotient is exact or one too small).
__device__ inline unsigned pixel_of(const BoxParams& Bp, unsigned slot) {
  const unsigned r = slot - __umulhi(slot, Bp.per_npix) * (unsigned)Bp.npix;
  return min(r, r - (unsigned)Bp.npix);
}

// Work order of the (box, angle) workgroups.
//   xcd = 0: boxes fastest, every XCD on the same angles;
//   xcd = 1: each XCD takes a contiguous range of (box, all angles) items, so
//            a box's segment records are reused from that XCD's L2 across
//            all angles;
//   xcd = A >= 2: the same, with the angles in blocks of at most A: a box's records
//            are reused across A angles while at most A workgroups of one box
//            flush into the same dose cells at a time.
__device__ inline bool work_item(int nboxes, int na, int xcd, int& b, int& a) {
  // a launch has fewer than 2^32 lanes (for_launches), so 32 bits hold every number here
  const unsigned L = blockIdx.x, nb = nboxes;
  if (!xcd) {
    if (L >= nb * (unsigned)na) return false;
    a = (int)(L / nb);
    b = (int)(L - a * nb);
    return true;
  }
  // nblk blocks of A or, the first `more` of them, A + 1 angles: every XCD gets
  // as many items as the next (blocks of exactly A left the last one short, and
  // its XCDs idle: 256^3, 90 representatives in
  // blocks of 16 69.4 against 64.3 ms)
  const unsigned nblk = xcd == 1 ? 1u : (unsigned)(na + xcd - 1) / (unsigned)xcd;
  const unsigned A = (unsigned)na / nblk, more = (unsigned)na - A * nblk;
  const unsigned W = nb * (unsigned)na, per = (W + kXcds - 1) / kXcds;
  const unsigned i = L / kXcds, w = (L % kXcds) * per + i;
  if (i >= per || w >= W) return false;
  const unsigned head = more * (A + 1) * nb;  // items of the longer blocks
  const bool longer = w < head;
  const unsigned len = longer ? A + 1 : A, first = longer ? 0u : head;
  const unsigned blk = (w - first) / (nb * len), rem = (w - first) - blk * (nb * len);
  b = (int)(rem / len);
  a = (int)((longer ? 0u : more * (A + 1)) + blk * len + (rem - b * len));
  return true;
}

static inline dim3 work_grid(int nboxes, int na, int xcd) {
  const int64_t W = (int64_t)nboxes * na;
  return dim3((unsigned)(xcd ? (W + kXcds - 1) / kXcds * kXcds : W));
}

// Calls launch(grid, part, a0) for the launches that the boxes and angles of Bp
// take (launch_cut): part has a launch's boxes and angles, the first of which
// is Bp's angle a0.
template <class F>
static void for_launches(const BoxParams& Bp, int threads, F launch) {
  if (Bp.nboxes < 1 || Bp.na < 1) return;
  const LaunchCut cut = launch_cut(Bp.nboxes, Bp.na, threads);
  for (int a0 = 0; a0 < Bp.na; a0 += cut.angles)
    for (int64_t b0 = 0; b0 < Bp.nboxes; b0 += cut.boxes) {
      BoxParams part = Bp;
      part.na = std::min(cut.angles, Bp.na - a0);
      part.nboxes = (int)std::min<int64_t>(cut.boxes, Bp.nboxes - b0);
      part.box_begin += b0;
      part.box_id += b0;
      part.box_supp += b0;
      launch(work_grid(part.nboxes, part.na, part.xcd), part, a0);
    }
}

// Rotated-box footprint [X0, X0 + WX) x [Y0, Y0 + WY) x [Z0, Z0 + WZ) in
// padded grid cells, and the box's centre in footprint coordinates.
struct Foot {
  int X0, Y0, Z0, WX, WY, WZ;
  float cx, cy, zoff;  // box centre (x, y) and bottom face (z) in footprint cells
};

__device__ inline Foot footprint(const BoxParams& Bp, int64_t box, double c, double s, double cx, double cy) {
  const BoxGrid& G = Bp.G;
  const int bz = box_z(box);
  const double xc = G.x0 + (box_x(box) + 0.5) * G.B, yc = G.y0 + (box_y(box) + 0.5) * G.B;
  const double gx = c * xc + s * yc + cx, gy = -s * xc + c * yc + cy;  // the turned centre
  const double half = 0.5 * G.B * (fabs(c) + fabs(s));
  // [lo, hi) clamped inside the padded grid, at least 2 and at most wmax
  // cells wide; a box outside the grid maps onto the padding at its edge
  auto range = [](double gmin, double gmax, int n, int wmax, int& lo, int& w) {
    lo = min(max((int)floor(gmin - 0.01), 0), n - 2);
    int hi = min(min((int)floor(gmax + 0.01) + 2, n), lo + wmax);
    w = max(hi, lo + 2) - lo;
  };
  Foot f;
  range(gx - half, gx + half, Bp.px, Bp.wxy_max, f.X0, f.WX);
  range(gy - half, gy + half, Bp.py, Bp.wxy_max, f.Y0, f.WY);
  // z does not turn and the boxes sit on whole cells: the box's samples have
  // z in [bz B, (bz + 1) B) up to the FP32 rounding of their positions, so
  // the footprint starts at bz B and ends one cell above the last corner
  f.Z0 = min(max(bz * G.B, 0), Bp.pz - 2);
  const int zhi = min(min((bz + 1) * G.B + 2, Bp.pz), f.Z0 + Bp.wz_max);
  f.WZ = max(zhi, f.Z0 + 2) - f.Z0;
  f.cx = (float)(gx - f.X0);
  f.cy = (float)(gy - f.Y0);
  f.zoff = (float)(bz * G.B - f.Z0);
  return f;
}

// Number of the footprint's first cell in the padded grid.
__device__ inline int64_t tile_base(const BoxParams& Bp, const Foot& f) {
  return ((int64_t)f.Z0 * Bp.py + f.Y0) * Bp.px + f.X0;
}

// A footprint's cells among NT lanes: a lane has one column (x, y) and every
// kSlices-th slice of it, so the divisions and the comparisons in x and y are
// made once, the slices' addresses are scalar and their LDS offsets constant.
// (With the cells dealt out one after the other their numbers cost 50 clocks of
// vector work for 64 cells, an eighth of a forward with 1300 segments a box.)
template <int COL, int NT>
constexpr int kSlices = NT >= COL ? NT / COL : 1;

// Loads the footprint's cells of a padded volume; put(i, v) takes cell i of the
// LDS tile (slice pitch SZ), zero outside the footprint.  All loads of a column
// are in flight before the first is waited for.
template <int SY, int SZ, int WZ, int NT, class T, class F>
__device__ inline void load_tile(const T* tile, int px, int py, const Foot& f, F put) {
  constexpr int COL = SY * SY, G = kSlices<COL, NT>, PER = (WZ + G - 1) / G;
  for (int i = threadIdx.x; i < G * COL; i += NT) {
    const int zg = G == 1 ? 0 : i / COL, c = i - zg * COL, y = c / SY, x = c - y * SY;
    const bool in = x < f.WX && y < f.WY;
    const unsigned from = (unsigned)((zg * py + y) * px + x);
    T v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      v[k] = T{};
      if (in && zg + k * G < f.WZ) v[k] = (tile + (int64_t)k * G * py * px)[from];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (WZ % G == 0 || zg + k * G < WZ) put(zg * SZ + c + k * G * SZ, v[k]);
  }
}

// Middle sample and step of a segment in footprint cells at angle (c, s);
// sample k of the segment (k = 0 .. count - 1) is at p + (k - m) d.
struct SegPos {
  float px, py, pz;   // middle sample m = (count - 1) / 2, rounded down
  float dx, dy, dz;   // step between samples
  float k0, k1;       // first and last sample relative to m: -m and count - 1 - m
};

__device__ inline SegPos seg_pos(const float4& pw, const float4& dn, int cnt, const Foot& f, float c, float s,
                                 float sc, float ss, float step) {
  SegPos g;
  g.px = fmaf(c, pw.x, fmaf(s, pw.y, f.cx));
  g.py = fmaf(c, pw.y, fmaf(-s, pw.x, f.cy));
  g.pz = pw.z + f.zoff;
  g.dx = fmaf(sc, dn.x, ss * dn.y);
  g.dy = fmaf(sc, dn.y, -ss * dn.x);
  g.dz = step * dn.z;
  const int m = (cnt - 1) >> 1;
  g.k0 = (float)(-m);
  g.k1 = (float)(cnt - 1 - m);
  return g;
}

// Lower bound of the unclamped fast path: a sample computed as
// fma(k, d, p) lies within one rounding (< 2^-20 cell here) of the segment
// between its endpoints, so endpoints at >= 2^-12 keep every sample's floor
// >= 0.
constexpr float kLo = 1.0f / 4096.0f;

// True when every sample of the segment lies inside [kLo, h] on all axes, so
// the sample loop needs no clamps (the samples lie on the line between its
// two ends).
__device__ inline bool seg_inside(const SegPos& g, float hx, float hy, float hz) {
  const float x0 = fmaf(g.k0, g.dx, g.px), y0 = fmaf(g.k0, g.dy, g.py), z0 = fmaf(g.k0, g.dz, g.pz);
  const float x1 = fmaf(g.k1, g.dx, g.px), y1 = fmaf(g.k1, g.dy, g.py), z1 = fmaf(g.k1, g.dz, g.pz);
  return fminf(x0, x1) >= kLo && fmaxf(x0, x1) <= hx && fminf(y0, y1) >= kLo && fmaxf(y0, y1) <= hy &&
         fminf(z0, z1) >= kLo && fmaxf(z0, z1) <= hz;
}

// Coordinate of a sample, clamped into [0, h] where the segment may leave
// the footprint (rounding at its faces, or a box beyond the padded grid,
// whose samples then read or write only padding).
template <bool CLAMP>
__device__ inline float coord(float k, float d, float p, float h) {
  const float x = fmaf(k, d, p);
  return CLAMP ? __builtin_amdgcn_fmed3f(x, 0.0f, h) : x;
}

// ------------------------------------------------------------- forward ---
//
// The workgroup of a (box, angle) stages the rotated box footprint of the
// padded volume in LDS (one coalesced read per cell), then every segment of
// the box gathers its samples from LDS.  The segment's partial sum (Horner
// over its samples from the far end, S <- S r + val with r = exp(-alpha
// step) applied as r_hi + r_lo, times the weight of its first sample) is
// added to its pixel as a 64-bit integer (the default), or written to
// part[angle][rank][ray] for a second kernel that adds, per pixel, the
// partials of its rays in a fixed order (pupil index, then rank).  Either
// way the result does not depend on scheduling.

// Storage of the staged volume footprint: FP32 values, or (for BF16 and FP16
// volumes) one 32-bit word per cell holding the 16-bit values of voxel x
// (low half) and voxel x + 1 (high half), so that a sample reads its 8
// corners as 4 words instead of 8.  Widening a BF16 or FP16 value to FP32 is
// exact, so both layouts give the same sums.
// (Named: kernel signatures are spelled with it, and host and device number
// unnamed types differently.)
enum VolFormat { kVolF32 = 0, kVolBF16Pairs = 1, kVolF16Pairs = 2 };

// The x-lerp of the corner pair at word o: v_x + fx (v_{x+1} - v_x), FP32.
// FP16 halves feed the mixed-precision FMA directly (v_fma_mix_f32 widens
// either half of its operands), so the pair costs the same two VALU ops as
// two FP32 values; BF16 halves are widened by a shift and a mask.
template <int FMT>
__device__ inline float lerp_x(const uint32_t* sv, unsigned o, float fx) {
  if constexpr (FMT == kVolF32) {
    const float lo = __uint_as_float(sv[o]), hi = __uint_as_float(sv[o + 1]);
    return fmaf(fx, hi - lo, lo);
  } else if constexpr (FMT == kVolBF16Pairs) {
    const uint32_t w = sv[o];
    const float lo = __uint_as_float(w << 16), hi = __uint_as_float(w & 0xffff0000u);
    return fmaf(fx, hi - lo, lo);
  } else {
    const uint32_t w = sv[o];
    // d = hi - lo straight from the two halves (exact to one FP32 rounding,
    // as a subtraction of the widened values); the compiler folds the
    // product by one and would widen both halves separately first.
    float d;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(w));
    const float lo = (float)__builtin_bit_cast(_Float16, (unsigned short)(w & 0xffffu));
    return fmaf(fx, d, lo);
  }
}

// Horner sum over the samples kfirst, kfirst + STRIDE, ..., klast of a
// segment, from the far end: S <- S r + val with r = r_hi + r_lo the
// attenuation over STRIDE samples.
template <int SY, int SZ, bool CLAMP, int FMT, int STRIDE>
__device__ inline float march_forward(const uint32_t* sv, const SegPos& g, float kfirst, float klast, float hx,
                                      float hy, float hz, float r_hi, float r_lo) {
  float S = 0.0f;
  for (float kf = klast; kf >= kfirst; kf -= (float)STRIDE) {
    const float x = coord<CLAMP>(kf, g.dx, g.px, hx);
    const float y = coord<CLAMP>(kf, g.dy, g.py, hy);
    const float z = coord<CLAMP>(kf, g.dz, g.pz, hz);
    const float fx = __builtin_amdgcn_fractf(x), fy = __builtin_amdgcn_fractf(y), fz = __builtin_amdgcn_fractf(z);
    const unsigned o = __umul24((unsigned)z, SZ) + __umul24((unsigned)y, SY) + (unsigned)x;
    const float c00 = lerp_x<FMT>(sv, o, fx);
    const float c01 = lerp_x<FMT>(sv, o + SY, fx);
    const float c10 = lerp_x<FMT>(sv, o + SZ, fx);
    const float c11 = lerp_x<FMT>(sv, o + SZ + SY, fx);
    const float c0 = fmaf(fy, c01 - c00, c00);
    const float c1 = fmaf(fy, c11 - c10, c10);
    const float val = fmaf(fz, c1 - c0, c0);
    S = fmaf(S, r_hi, fmaf(S, r_lo, val));
  }
  return S;
}

// The same sum, one lane per segment, keeping the LDS words of the current
// cell in registers: a sample in the same cell as the one before reads no
// LDS (the reads are issued only for lanes whose cell changed).
template <int SY, int SZ, bool CLAMP, int FMT>
__device__ inline float march_forward_cached(const uint32_t* sv, const SegPos& g, float hx, float hy, float hz,
                                             float r_hi, float r_lo) {
  constexpr bool F32 = FMT == kVolF32;
  float S = 0.0f;
  unsigned cur = 0xffffffffu;
  uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (float kf = g.k1; kf >= g.k0; kf -= 1.0f) {
    const float x = coord<CLAMP>(kf, g.dx, g.px, hx);
    const float y = coord<CLAMP>(kf, g.dy, g.py, hy);
    const float z = coord<CLAMP>(kf, g.dz, g.pz, hz);
    const float fx = __builtin_amdgcn_fractf(x), fy = __builtin_amdgcn_fractf(y), fz = __builtin_amdgcn_fractf(z);
    const unsigned o = __umul24((unsigned)z, SZ) + __umul24((unsigned)y, SY) + (unsigned)x;
    if (o != cur) {
      cur = o;
      w[0] = sv[o];
      w[2] = sv[o + SY];
      w[4] = sv[o + SZ];
      w[6] = sv[o + SZ + SY];
      if constexpr (F32) {
        w[1] = sv[o + 1];
        w[3] = sv[o + SY + 1];
        w[5] = sv[o + SZ + 1];
        w[7] = sv[o + SZ + SY + 1];
      }
    }
    float c[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (F32) {
        const float lo = __uint_as_float(w[2 * j]), hi = __uint_as_float(w[2 * j + 1]);
        c[j] = fmaf(fx, hi - lo, lo);
      } else if constexpr (FMT == kVolBF16Pairs) {
        const float lo = __uint_as_float(w[2 * j] << 16), hi = __uint_as_float(w[2 * j] & 0xffff0000u);
        c[j] = fmaf(fx, hi - lo, lo);
      } else {
        float d;
        asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(w[2 * j]));
        const float lo = (float)__builtin_bit_cast(_Float16, (unsigned short)(w[2 * j] & 0xffffu));
        c[j] = fmaf(fx, d, lo);
      }
    }
    const float c0 = fmaf(fy, c[1] - c[0], c[0]);
    const float c1 = fmaf(fy, c[3] - c[2], c[2]);
    const float val = fmaf(fz, c1 - c0, c0);
    S = fmaf(S, r_hi, fmaf(S, r_lo, val));
  }
  return S;
}

// Number of the cell at whole coordinates: in FP32 (exact below 2^24) with one
// conversion, which costs twice an addition, where integers took three and two
// multiplications of that cost.
template <int SY, int SZ>
__device__ inline unsigned cell_number(float x, float y, float z) {
  return (unsigned)fmaf(z, (float)SZ, fmaf(y, (float)SY, x));
}

// The same sum from FP32 cells that hold a voxel and its x neighbour (float2).
template <int SY, int SZ, bool CLAMP>
__device__ inline float march_forward_cells(const float2* sv, const SegPos& g, float hx, float hy, float hz,
                                            float r_hi, float r_lo) {
  float S = 0.0f;
  unsigned cur = 0xffffffffu;
  float2 w[4] = {};
  for (float kf = g.k1; kf >= g.k0; kf -= 1.0f) {
    const float x = coord<CLAMP>(kf, g.dx, g.px, hx);
    const float y = coord<CLAMP>(kf, g.dy, g.py, hy);
    const float z = coord<CLAMP>(kf, g.dz, g.pz, hz);
    const float fx = __builtin_amdgcn_fractf(x), fy = __builtin_amdgcn_fractf(y), fz = __builtin_amdgcn_fractf(z);
    const unsigned o = cell_number<SY, SZ>(x - fx, y - fy, z - fz);
    if (o != cur) {
      cur = o;
      w[0] = sv[o];
      w[1] = sv[o + SY];
      w[2] = sv[o + SZ];
      w[3] = sv[o + SZ + SY];
    }
    float c[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = fmaf(fx, w[j].y - w[j].x, w[j].x);
    const float c0 = fmaf(fy, c[1] - c[0], c[0]);
    const float c1 = fmaf(fy, c[3] - c[2], c[2]);
    const float val = fmaf(fz, c1 - c0, c0);
    S = fmaf(S, r_hi, fmaf(S, r_lo, val));
  }
  return S;
}

// March modes of the fixed-point box forward (k_forward_box's MODE).
constexpr int kMarchOne = 1, kMarchPair = 2, kMarchCached = 3, kMarchCells = 4;

// Fixed-point forward (the default).  A pixel's value is a sum of segment
// partials pw.w S, each at most (step / n_pupil) n V in magnitude (sample
// weights <= step / n_pupil, attenuation <= 1, trilinear values <= V, the
// volume's largest |value|, n the segment's samples), so the pixel's exact
// sum and every partial sum of it are at most bound = (step / n_pupil)
// pix_samples_max V.  With the power of two scale 2^(61 - e), bound < 2^e,
// every FP32 partial times the scale is exact in FP64 and below 2^61; it is
// rounded to an integer (<= 1/2 off, i.e. <= 2^(e - 62) <= bound 2^-61) and added to the
// pixel's 64-bit integer, which stays below 2^62: integer adds commute, so
// the result does not depend on the order of the atomics.

// vol: the padded working volume, FP32 values or 16-bit pairs (FMT).
// FX = false: partial sums to part[angle][rank][ray] (slots per angle);
// FX = true: fixed-point adds into pfx[angle][pixel].
// MODE: how lanes march a segment.  kMarchOne: one lane, all samples.
// kMarchPair: two neighbouring lanes share a segment, one taking its even
// and the other its odd samples (Horner with r^2 each; the pair's sum is
// S_even + r S_odd); their samples are half a voxel apart, so they often
// read the same LDS words, which the LDS serves as one broadcast.
// kMarchCached: one lane, the current cell's LDS words kept in registers.
// kMarchCells (the default at the default box edge): the same with FP32 cells of a voxel and its x
// neighbour, so a sample's corners are four 8-byte reads (7.7 clocks for 64
// unrelated lanes, as much as one of 4 bytes) and 16-bit values are widened once
// a cell.  Bound by vector issue and LDS reads, each about 70 % of the time.
template <int MODE>
constexpr int kForwardThreads = MODE == kMarchCells ? 512 : 256;
template <int B, int FMT, bool FX, int MODE>
__global__ __launch_bounds__(kForwardThreads<MODE>) void k_forward_box(MarchParams P, BoxParams Bp, const uint32_t* __restrict__ vol,
                                                     float* __restrict__ part, int64_t slots,
                                                     unsigned long long* __restrict__ pfx,
                                                     const unsigned* __restrict__ vmax, double fx_coef) {
  constexpr int SY = Fixed<B>::WXY, SZ = SY * SY, NC = SZ * Fixed<B>::WZ;
  using Cell = std::conditional_t<MODE == kMarchCells, float2, uint32_t>;
  __shared__ Cell sv[NC];
  int b, a;
  if (!work_item(Bp.nboxes, Bp.na, Bp.xcd, b, a)) return;
  const int member = (P.a0 + a) / Bp.turn_stride;
  const double2 cs = P.cs[P.a0 + a - member * Bp.turn_stride];
  vol += (int64_t)(member - Bp.member0) * Bp.px * Bp.py * Bp.pz;
  const Foot f = footprint(Bp, Bp.box_id[b], cs.x, cs.y, P.cx, P.cy);
  load_tile<SY, SZ, Fixed<B>::WZ, kForwardThreads<MODE>>(
      vol + tile_base(Bp, f), Bp.px, Bp.py, f, [&](int i, uint32_t v) {
        if constexpr (MODE != kMarchCells) {
          sv[i] = v;
        } else if constexpr (FMT == kVolF32) {
          // (the last cell of a row gets a neighbour that no sample reads)
          sv[i].x = __uint_as_float(v);
          if (i > 0) sv[i - 1].y = __uint_as_float(v);
        } else if constexpr (FMT == kVolBF16Pairs) {
          sv[i] = make_float2(__uint_as_float(v << 16), __uint_as_float(v & 0xffff0000u));
        } else {
          sv[i] = make_float2((float)__builtin_bit_cast(_Float16, (uint16_t)v),
                              (float)__builtin_bit_cast(_Float16, (uint16_t)(v >> 16)));
        }
      });
  __syncthreads();
  const float hx = (float)f.WX - 1.001f, hy = (float)f.WY - 1.001f, hz = (float)f.WZ - 1.001f;
  const float c = (float)cs.x, s = (float)cs.y, sc = P.step * c, ss = P.step * s;
  const int s_end = Bp.box_begin[b + 1];
  float* out = part + (int64_t)a * slots;
  double scale = 1.0;
  bool finite = true;
  if constexpr (FX) {
    const unsigned vm = *vmax;
    finite = vm < 0x7f800000u;
    scale = fx_scale(vm, fx_coef);
  }
  unsigned long long* row = pfx + (int64_t)a * Bp.npix;
  const int part_of = MODE == kMarchPair ? (int)(threadIdx.x & 1u) : 0;
  constexpr int LPS = MODE == kMarchPair ? 2 : 1;  // lanes per segment
  for (int si = Bp.box_begin[b] + (int)threadIdx.x / LPS; si < s_end; si += (int)blockDim.x / LPS) {
    const float4 pw = Bp.seg.pw[si], dn = Bp.seg.dn[si];
    const SegPos g = seg_pos(pw, dn, __float_as_int(dn.w), f, c, s, sc, ss, P.step);
    float S;
    if constexpr (MODE == kMarchCells) {
      S = seg_inside(g, hx, hy, hz) ? march_forward_cells<SY, SZ, false>(sv, g, hx, hy, hz, P.r_hi, P.r_lo)
                                    : march_forward_cells<SY, SZ, true>(sv, g, hx, hy, hz, P.r_hi, P.r_lo);
    } else if constexpr (MODE == kMarchCached) {
      S = seg_inside(g, hx, hy, hz) ? march_forward_cached<SY, SZ, false, FMT>(sv, g, hx, hy, hz, P.r_hi, P.r_lo)
                                    : march_forward_cached<SY, SZ, true, FMT>(sv, g, hx, hy, hz, P.r_hi, P.r_lo);
    } else if constexpr (MODE == kMarchOne) {
      S = seg_inside(g, hx, hy, hz)
              ? march_forward<SY, SZ, false, FMT, 1>(sv, g, g.k0, g.k1, hx, hy, hz, P.r_hi, P.r_lo)
              : march_forward<SY, SZ, true, FMT, 1>(sv, g, g.k0, g.k1, hx, hy, hz, P.r_hi, P.r_lo);
    } else {
      // this lane's samples: k0 + part_of, then every second one (none if
      // the segment is shorter); both lanes of a pair take the same branch
      const float kfirst = g.k0 + (float)part_of;
      const float klast = kfirst + 2.0f * floorf((g.k1 - kfirst) * 0.5f);
      S = seg_inside(g, hx, hy, hz)
              ? march_forward<SY, SZ, false, FMT, 2>(sv, g, kfirst, klast, hx, hy, hz, P.r2_hi, P.r2_lo)
              : march_forward<SY, SZ, true, FMT, 2>(sv, g, kfirst, klast, hx, hy, hz, P.r2_hi, P.r2_lo);
      const float odd = __shfl_xor(S, 1);
      S = fmaf(odd, P.r_hi, fmaf(odd, P.r_lo, S));
    }
    const float v = pw.w * S;
    if constexpr (FX) {
      if (part_of == 0 && finite && v != 0.0f)
        atomicAdd(row + pixel_of(Bp, (unsigned)Bp.seg.idx[si]),
                  (unsigned long long)__double2ll_rn((double)v * scale));
    } else {
      out[Bp.seg.idx[si]] = v;
    }
  }
}

// ------------------------------------- forward, several angles at once ---
//
// Angles that are whole quarter turns apart (find_turns) share every sample's
// position, cell and offsets; only the values under the cell differ.  One
// workgroup takes a box at all NQ = 2 or 4 of them: the LDS holds, per cell of
// the representative's footprint, the NQ volumes turned into its frame
// (interleaved, staged from a copy that k_pad_turned makes), a corner is one
// LDS read of NQ values, and the position work and the segment records are
// paid once.  The arithmetic per angle is march_forward's, so the projections
// are the same bits as one angle at a time.
//
// The cells hold FP32 whatever the caller's type (widening is exact): 16-bit
// cells halve the LDS bytes but their widening costs more VALU issue than the
// bytes do (256^3, 360 angles: 71.1 ms with FP32 cells, 91.2 with FP16 cells
// read by mixed-precision FMAs; BF16 at 512^3 338 against 300 ms).
//
// Bounds: a wave's step takes about 80 VALU instructions for its 4 x 64 samples (71 %
// of the issue slots at 256^3) and up to eight 16-byte reads.  A read of 64
// unrelated cells takes 7.6 clocks for 4 bytes a lane, 7.7 for 8 and 12.8 for
// 16 (measured: 20 words a clock against 8.4), so wide cells move 2.4 times the
// words.  256^3, 360 angles: 64 ms against 123 one angle at a time (512^3, BF16
// 273 against 532).

template <int NQ>
struct CellVec;
template <>
struct CellVec<2> {
  using T = float2;
};
template <>
struct CellVec<4> {
  using T = float4;
};

// march_forward_cached for NQ members: S[q] is member q's Horner sum.
template <int SY, int SZ, bool CLAMP, int NQ, class Cell>
__device__ inline void march_forward_turned(const Cell* sv, const SegPos& g, float hx, float hy,
                                            float hz, float r_hi, float r_lo, float (&S)[NQ]) {
  constexpr int off[8] = {0, 1, SY, SY + 1, SZ, SZ + 1, SZ + SY, SZ + SY + 1};
  float w[8][NQ] = {};
  unsigned cur = 0xffffffffu;
#pragma unroll
  for (int q = 0; q < NQ; ++q) S[q] = 0.0f;
  for (float kf = g.k1; kf >= g.k0; kf -= 1.0f) {
    const float x = coord<CLAMP>(kf, g.dx, g.px, hx);
    const float y = coord<CLAMP>(kf, g.dy, g.py, hy);
    const float z = coord<CLAMP>(kf, g.dz, g.pz, hz);
    const float fx = __builtin_amdgcn_fractf(x), fy = __builtin_amdgcn_fractf(y), fz = __builtin_amdgcn_fractf(z);
    const unsigned o = cell_number<SY, SZ>(x - fx, y - fy, z - fz);
    if (o != cur) {
      cur = o;
#pragma unroll
      for (int j = 0; j < 8; j += sizeof(Cell) / (4 * NQ)) {
        const Cell v = sv[o + off[j]];
        __builtin_memcpy(w[j], &v, sizeof(v));
      }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float c00 = fmaf(fx, w[1][q] - w[0][q], w[0][q]);
      const float c01 = fmaf(fx, w[3][q] - w[2][q], w[2][q]);
      const float c10 = fmaf(fx, w[5][q] - w[4][q], w[4][q]);
      const float c11 = fmaf(fx, w[7][q] - w[6][q], w[6][q]);
      const float c0 = fmaf(fy, c01 - c00, c00);
      const float c1 = fmaf(fy, c11 - c10, c10);
      const float val = fmaf(fz, c1 - c0, c0);
      S[q] = fmaf(S[q], r_hi, fmaf(S[q], r_lo, val));
    }
  }
}

// Value of the lane whose number differs in bit BIT (0 or 1) of the quad.
template <int BIT>
__device__ inline unsigned long long quad_xor(unsigned long long v) {
  constexpr int perm = BIT == 0 ? 0xB1 : 0x4E;  // lanes 1 0 3 2, or 2 3 0 1
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)v, perm, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), perm, 0xf, 0xf, true);
  return (unsigned long long)(uint32_t)lo | (unsigned long long)(uint32_t)hi << 32;
}

// v[j] of lane i <-> v[i] of lane j within groups of NQ = 2 or 4 lanes (all
// lanes of the wave must be active).
template <int NQ>
__device__ inline void transpose_lanes(unsigned long long (&v)[NQ]) {
  const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
#pragma unroll
  for (int p = 0; p < NQ; p += 2) {
    const unsigned long long got = quad_xor<0>(b0 ? v[p] : v[p + 1]);
    v[p] = b0 ? got : v[p];
    v[p + 1] = b0 ? v[p + 1] : got;
  }
  if constexpr (NQ == 4) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const unsigned long long got = quad_xor<1>(b1 ? v[p] : v[p + 2]);
      v[p] = b1 ? got : v[p];
      v[p + 2] = b1 ? v[p + 2] : got;
    }
  }
}

// Lane j's value within groups of NQ lanes.
template <int NQ>
__device__ inline unsigned lane_of(unsigned v, int j) {
  if constexpr (NQ == 2)
    return j ? __builtin_amdgcn_mov_dpp(v, 0xF5, 0xf, 0xf, true) : __builtin_amdgcn_mov_dpp(v, 0xA0, 0xf, 0xf, true);
  return j == 0   ? __builtin_amdgcn_mov_dpp(v, 0x00, 0xf, 0xf, true)
         : j == 1 ? __builtin_amdgcn_mov_dpp(v, 0x55, 0xf, 0xf, true)
         : j == 2 ? __builtin_amdgcn_mov_dpp(v, 0xAA, 0xf, 0xf, true)
                  : __builtin_amdgcn_mov_dpp(v, 0xFF, 0xf, 0xf, true);
}

// P.a0 + a is the representative's angle; the sums of work item a go to
// pfx[a][pixel][member].  A pixel's members lie side by side, and NQ lanes
// exchange their segments' sums first, so that the NQ lanes add to one
// pixel's members at a time: one request of 8 NQ bytes instead of NQ of 8.
// Cell: the members' values, or for two members theirs and their x neighbours'.
template <int NQ, int NT, class Cell>
__global__ __launch_bounds__(NT) void k_forward_turned(
    MarchParams P, BoxParams Bp, const typename CellVec<NQ>::T* __restrict__ vol,
    unsigned long long* __restrict__ pfx, const unsigned* __restrict__ vmax, double fx_coef) {
  // slice pitch two cells longer than a slice: 69.7 against 71.0 ms at 256^3
  constexpr int SY = Fixed<kBox>::WXY, SZ = SY * SY + 2;
  using Vec = typename CellVec<NQ>::T;
  __shared__ Cell sv[SZ * Fixed<kBox>::WZ];
  int b, a;
  if (!work_item(Bp.nboxes, Bp.na, Bp.xcd, b, a)) return;
  const unsigned vm = *vmax;
  if (vm >= 0x7f800000u) return;  // a non-finite value: k_fx_store writes NaN
  const double2 cs = P.cs[P.a0 + a];
  const Foot f = footprint(Bp, Bp.box_id[b], cs.x, cs.y, P.cx, P.cy);
  load_tile<SY, SZ, Fixed<kBox>::WZ, NT>(vol + tile_base(Bp, f), Bp.px, Bp.py, f, [&](int i, const Vec& v) {
    // (the last cell of a row gets a neighbour that no sample reads)
    __builtin_memcpy(__builtin_assume_aligned(&sv[i], sizeof(Vec)), &v, sizeof(Vec));
    if constexpr (sizeof(Cell) > sizeof(Vec))
      if (i > 0) __builtin_memcpy(__builtin_assume_aligned((char*)&sv[i - 1] + sizeof(Vec), sizeof(Vec)), &v, sizeof(Vec));
  });
  __syncthreads();
  const float hx = (float)f.WX - 1.001f, hy = (float)f.WY - 1.001f, hz = (float)f.WZ - 1.001f;
  const float c = (float)cs.x, s = (float)cs.y, sc = P.step * c, ss = P.step * s;
  const int s_end = Bp.box_begin[b + 1];
  const double scale = fx_scale(vm, fx_coef);
  unsigned long long* row = pfx + (int64_t)a * Bp.npix * NQ + (threadIdx.x & (NQ - 1));
  // whole waves go round together: lanes without a segment add nothing
  for (int s0 = Bp.box_begin[b] + (int)(threadIdx.x & ~63u); s0 < s_end; s0 += NT) {
    const int si = s0 + (int)(threadIdx.x & 63u);
    unsigned long long sum[NQ] = {};
    unsigned pixel = 0u;
    if (si < s_end) {
      const float4 pw = Bp.seg.pw[si], dn = Bp.seg.dn[si];
      const unsigned slot = (unsigned)Bp.seg.idx[si];  // loaded before the march, used after it
      const SegPos g = seg_pos(pw, dn, __float_as_int(dn.w), f, c, s, sc, ss, P.step);
      float S[NQ];
      if (seg_inside(g, hx, hy, hz))
        march_forward_turned<SY, SZ, false, NQ>(sv, g, hx, hy, hz, P.r_hi, P.r_lo, S);
      else
        march_forward_turned<SY, SZ, true, NQ>(sv, g, hx, hy, hz, P.r_hi, P.r_lo, S);
      pixel = pixel_of(Bp, slot);
#pragma unroll
      for (int q = 0; q < NQ; ++q) sum[q] = (unsigned long long)__double2ll_rn((double)(pw.w * S[q]) * scale);
    }
    transpose_lanes<NQ>(sum);
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const unsigned at = lane_of<NQ>(pixel, j);
      if (sum[j] != 0) atomicAdd(row + (int64_t)at * NQ, sum[j]);
    }
  }
}

// Clears the fixed-point projections of a call and the volume maximum.
__global__ void k_fx_clear(unsigned long long* __restrict__ p, int64_t n, unsigned* __restrict__ vmax) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
  if (i == 0) *vmax = 0u;
}

// Largest |value| of the padded working volume as FP32 bits (non-negative
// floats order as their bit patterns; a NaN or infinity compares above every
// finite value).
template <int FMT>
__device__ inline unsigned abs_bits(uint32_t w) {
  if constexpr (FMT == kVolF32) {
    return w & 0x7fffffffu;
  } else if constexpr (FMT == kVolBF16Pairs) {
    return max((w << 16) & 0x7fffffffu, w & 0x7fff0000u);
  } else {
    const float lo = (float)__builtin_bit_cast(_Float16, (unsigned short)(w & 0xffffu));
    const float hi = (float)__builtin_bit_cast(_Float16, (unsigned short)(w >> 16));
    return max(__float_as_uint(lo) & 0x7fffffffu, __float_as_uint(hi) & 0x7fffffffu);
  }
}

// Blocks of the two largest-value kernels: two workgroups of 1024 lanes a CU
// cover the memory latency, and more blocks only add atomics on one address.
constexpr unsigned kMaxBlocks = 512;
static inline dim3 max_grid(int64_t n) {
  return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 4095) / 4096, kMaxBlocks)));
}

template <typename PT>
__device__ inline void store_proj(PT* p, int64_t i, float x);
template <>
__device__ inline void store_proj<float>(float* p, int64_t i, float x) {
  p[i] = x;
}
template <>
__device__ inline void store_proj<uint16_t>(uint16_t* p, int64_t i, float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) {
    p[i] = (uint16_t)((u >> 16) | 0x40u);  // quiet NaN
  } else {
    u += 0x7fffu + ((u >> 16) & 1u);       // round to nearest even
    p[i] = (uint16_t)(u >> 16);
  }
}
template <>
__device__ inline void store_proj<__half>(__half* p, int64_t i, float x) {
  p[i] = __float2half_rn(x);
}

// Fixed-point projections -> stored projections: the integer over the scale,
// rounded to FP32 (then to BF16 / FP16 on store); all NaN if the volume held
// a NaN or an infinity.
template <typename PT>
__global__ void k_fx_store(const unsigned long long* __restrict__ pfx, PT* __restrict__ proj, int64_t n,
                           const unsigned* __restrict__ vmax, double fx_coef) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const unsigned vm = *vmax;
  const bool finite = vm < 0x7f800000u;
  const float x = finite ? (float)((double)(long long)pfx[i] / fx_scale(vm, fx_coef)) : __uint_as_float(0x7fc00000u);
  store_proj(proj, i, x);
}

// The same for groups of NQ members: n (work item, pixel) pairs, the members of
// a pixel side by side in pfx and member_stride values apart in proj.
template <typename PT, int NQ>
__global__ void k_fx_store_turned(const unsigned long long* __restrict__ pfx, PT* __restrict__ proj, int64_t n,
                                  int64_t member_stride, const unsigned* __restrict__ vmax, double fx_coef) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const unsigned vm = *vmax;
  const bool finite = vm < 0x7f800000u;
  const double scale = fx_scale(vm, fx_coef);
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    store_proj(proj, i + q * member_stride,
               finite ? (float)((double)(long long)pfx[i * NQ + q] / scale) : __uint_as_float(0x7fc00000u));
}

template <typename PT>
__global__ void k_reduce_segments(const float* __restrict__ part, const int* __restrict__ nseg,
                                  PT* __restrict__ proj, int npix, int np, int64_t n_rays, int64_t slots,
                                  int na) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)na * npix) return;
  const int a = (int)(i / npix);
  const int pix = (int)(i - (int64_t)a * npix);
  const float* base = part + (int64_t)a * slots;
  float acc = 0.0f;
  for (int j = 0; j < np; ++j) {
    const int64_t r = (int64_t)j * npix + pix;
    const int ns = nseg[r];
    const float* b = base + r;
    // four running sums in a fixed interleave keep four loads in flight;
    // the order is the same on every call
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
    int q = 0;
    for (; q + 4 <= ns; q += 4) {
      s0 += b[(int64_t)q * n_rays];
      s1 += b[(int64_t)(q + 1) * n_rays];
      s2 += b[(int64_t)(q + 2) * n_rays];
      s3 += b[(int64_t)(q + 3) * n_rays];
    }
    for (; q < ns; ++q) s0 += b[(int64_t)q * n_rays];
    acc += (s0 + s1) + (s2 + s3);
  }
  store_proj(proj, i, acc);
}

// Forward launch arguments beyond the march and box parameters.
struct FwdOut {
  float* part;              // partial sums (fx = false)
  int64_t slots;
  unsigned long long* pfx;  // fixed-point projections (fx = true)
  const unsigned* vmax;
  double fx_coef;
  int mode;                 // march mode (fx = true): kMarchOne, kMarchPair, kMarchCached or kMarchCells
};

template <int B, int FMT, bool FX, int MODE>
static void launch_forward_box_m(hipStream_t s, const MarchParams& P, const BoxParams& Bp, const uint32_t* vol,
                                 const FwdOut& o) {
  constexpr int NT = kForwardThreads<MODE>;
  for_launches(Bp, NT, [&](dim3 grid, const BoxParams& part, int64_t a0) {
    MarchParams Pa = P;
    Pa.a0 += (int)a0;
    hipLaunchKernelGGL((k_forward_box<B, FMT, FX, MODE>), grid, dim3(NT), 0, s, Pa, part, vol,
                       FX ? o.part : o.part + a0 * o.slots, o.slots, FX ? o.pfx + a0 * Bp.npix : o.pfx, o.vmax,
                       o.fx_coef);
  });
}

template <int B, int FMT, bool FX>
static void launch_forward_box_f(hipStream_t s, const MarchParams& P, const BoxParams& Bp, const uint32_t* vol,
                                 const FwdOut& o) {
  if constexpr (FX) {
    if constexpr (B == kBox)
      if (o.mode == kMarchCells) return launch_forward_box_m<B, FMT, FX, kMarchCells>(s, P, Bp, vol, o);
    if (o.mode == kMarchCached) return launch_forward_box_m<B, FMT, FX, kMarchCached>(s, P, Bp, vol, o);
    if (o.mode == kMarchPair) return launch_forward_box_m<B, FMT, FX, kMarchPair>(s, P, Bp, vol, o);
  }
  launch_forward_box_m<B, FMT, FX, kMarchOne>(s, P, Bp, vol, o);
}

template <int B, bool FX>
static void launch_forward_box(hipStream_t s, const MarchParams& P, const BoxParams& Bp, int fmt,
                               const uint32_t* vol, const FwdOut& o) {
  switch (fmt) {
    case kVolBF16Pairs: launch_forward_box_f<B, kVolBF16Pairs, FX>(s, P, Bp, vol, o); break;
    case kVolF16Pairs: launch_forward_box_f<B, kVolF16Pairs, FX>(s, P, Bp, vol, o); break;
    default: launch_forward_box_f<B, kVolF32, FX>(s, P, Bp, vol, o); break;
  }
}

template <bool FX>
static void launch_forward_box_edge(int edge, hipStream_t s, const MarchParams& P, const BoxParams& Bp, int fmt,
                                    const uint32_t* vol, const FwdOut& o) {
  switch (edge) {
    case 8: launch_forward_box<8, FX>(s, P, Bp, fmt, vol, o); break;
    case 12: launch_forward_box<12, FX>(s, P, Bp, fmt, vol, o); break;
    default: launch_forward_box<16, FX>(s, P, Bp, fmt, vol, o); break;
  }
}

// Caller volume -> padded working volume of the box forward, NQ copies
// interleaved, copy j turned by turns.q[j] quarter turns into the frame of its
// group's representative angle (zero in the padding).  A cell holds NQ FP32
// words; alone (NQ = 1) a 16-bit value is stored as a pair word with its x
// neighbour.  Also raises *vmax to the largest |value|
// (FP32 bits) unless vmax is NULL.
//
// One workgroup per 32 x 32 tile of a slice (and every gridDim.z-th slice):
// copies turned by an odd number of quarter turns read the volume along the
// tile's y, so every read and write is along a row; the tile turns in LDS.
struct Turns {
  int q[4];
};

// A caller's value (VFMT) as stored in a cell (FMT: the same, or FP32 words).
template <int VFMT, int FMT, typename VT>
__device__ inline uint32_t cell_bits(VT v) {
  if constexpr (VFMT == kVolF32) return __float_as_uint(v);
  else if constexpr (VFMT == FMT) return v;
  else if constexpr (VFMT == kVolBF16Pairs) return (uint32_t)v << 16;
  else return __float_as_uint((float)__builtin_bit_cast(_Float16, v));
}

template <int VFMT, int FMT, int NQ>
__global__ __launch_bounds__(256) void k_pad_turned(
    const std::conditional_t<VFMT == kVolF32, float, uint16_t>* __restrict__ vol, uint32_t* __restrict__ out,
    int nx, int ny, int nz, int px, int py, int pz, Turns turns, unsigned* __restrict__ vmax) {
  constexpr int T = 32, TX = FMT != kVolF32 && NQ == 1 ? T + 1 : T;  // pairs: one more column
  __shared__ uint32_t tile[NQ][T][T + 3];
  const int X0 = blockIdx.x * T, Y0 = blockIdx.y * T;
  unsigned m = 0u;
  for (int z = blockIdx.z; z < pz; z += gridDim.z) {
    const int iz = z - kPad;
    for (int j = 0; j < NQ; ++j) {
      const int turn = turns.q[j];
      for (int i = threadIdx.x; i < T * TX; i += 256) {
        const int lx = turn & 1 ? i / T : i % TX, ly = turn & 1 ? i % T : i / TX;
        const int X = X0 + lx, Y = Y0 + ly;
        const int x = turn == 0 ? X : turn == 1 ? Y : turn == 2 ? px - 1 - X : px - 1 - Y;
        const int y = turn == 0 ? Y : turn == 1 ? py - 1 - X : turn == 2 ? py - 1 - Y : X;
        const int ix = x - kPad, iy = y - kPad;
        uint32_t v = 0u;
        if (X < px && Y < py && ix >= 0 && ix < nx && iy >= 0 && iy < ny && iz >= 0 && iz < nz)
          v = cell_bits<VFMT, FMT>(vol[((int64_t)iz * ny + iy) * nx + ix]);
        tile[j][ly][lx] = v;
        if (j == 0) m = max(m, abs_bits<FMT>(v));
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < T * T; i += 256) {
      const int lx = i % T, ly = i / T, X = X0 + lx, Y = Y0 + ly;
      if (X >= px || Y >= py) continue;
      const int64_t o = ((int64_t)z * py + Y) * px + X;
      if constexpr (NQ == 1) {
        out[o] = FMT == kVolF32 ? tile[0][ly][lx] : tile[0][ly][lx] | (tile[0][ly][lx + (TX > T)] << 16);
      } else {
        uint32_t v[NQ];
#pragma unroll
        for (int j = 0; j < NQ; ++j) v[j] = tile[j][ly][lx];
        __builtin_memcpy(__builtin_assume_aligned(out + o * NQ, sizeof(v)), v, sizeof(v));
      }
    }
    __syncthreads();
  }
  if (vmax) {
    m = block_max(m);
    if (threadIdx.x == 0) raise_max(vmax, m);
  }
}

template <int VFMT, int FMT, int NQ>
static void pad_turned(const vam_geometry* h, const void* vol, void* out, const Turns& t, unsigned* vmax,
                       hipStream_t s) {
  using VT = std::conditional_t<VFMT == kVolF32, float, uint16_t>;
  const vam_geometry_desc& D = h->desc;
  const int tx = (h->px + 31) / 32, ty = (h->py + 31) / 32;
  const dim3 grid(tx, ty, std::min(h->pz, std::max(1, 2048 / (tx * ty))));
  hipLaunchKernelGGL((k_pad_turned<VFMT, FMT, NQ>), grid, dim3(256), 0, s, (const VT*)vol, (uint32_t*)out,
                     D.nx, D.ny, D.nz, h->px, h->py, h->pz, t, vmax);
}

// fmt: the caller's format.
template <int NQ>
static void pad_turned(const vam_geometry* h, const void* vol, int fmt, void* out, const Turns& t, unsigned* vmax,
                       hipStream_t s) {
  switch (fmt) {
    case kVolBF16Pairs: pad_turned<kVolBF16Pairs, NQ == 1 ? kVolBF16Pairs : kVolF32, NQ>(h, vol, out, t, vmax, s); break;
    case kVolF16Pairs: pad_turned<kVolF16Pairs, NQ == 1 ? kVolF16Pairs : kVolF32, NQ>(h, vol, out, t, vmax, s); break;
    default: pad_turned<kVolF32, kVolF32, NQ>(h, vol, out, t, vmax, s);
  }
}

// How many members of each representative a call's angles [a0, a0 + na) are
// taken together: 4 or 2 where the call is whole quarters of a turn (two of
// them side by side, or two members half a turn apart), else 1.  Either way
// every angle is computed in its representative's frame, so how a turn is cut
// into calls does not change a bit.  (Three quarters, or a call that cuts
// through a quarter, go one angle at a time in one launch: a pair launch and a
// launch for the rest were 3 % slower at 179 of 180 angles of 128^3, each with
// its own tail.)
static int members_together(const vam_geometry* h, int a0, int na) {
  const int M = h->turn_members, Q = h->turn_stride;
  if (M == 1 || a0 % Q != 0) return 1;
  return na == 4 * Q ? 4 : na == 2 * Q ? 2 : 1;
}

// Work order of the forward of na angles (or representatives) where none was
// chosen: blocks of at most 16, and at least four blocks, so that the XCDs'
// parts of a block's boxes are alike (45 of them in blocks of 16 / 12: 128^3 2.35
// / 2.23 ms, one at a time in FP16 1.11 / 1.01, 256^3 telecentric 18.9 / 18.3; 90
// in blocks of 16 / 12, 256^3: 64.3 / 67.0).  Edges 8 and 16: blocks of 16 (30 of
// 90 angles of 128^3 at edge 8 in blocks of 8 / 15: 2.34 / 2.13 ms).
static int forward_order(const vam_geometry* h, int na) {
  return h->xcd_forward >= 0 ? h->xcd_forward : h->boxes.B != kBox ? 16 : std::max(2, std::min(16, (na + 3) / 4));
}

// Segments a box from which the forward's cells take 16 bytes, so that two
// workgroups fit a CU's LDS instead of four: four members together (fewer: two
// and two), and pairs with their x neighbours (four 16-byte reads a sample
// instead of eight of 8).  With fewer segments two workgroups keep too few
// waves busy.  180 angles, members by fours / by twos: 64^3 and 128^3 with one
// pupil point (150 segments) 0.252 / 0.226 and 1.50 / 1.28 ms, two points (300)
// 1.62 / 1.63, four (600) 1.97 / 2.74.  90 angles by twos, 16-byte / 8-byte
// cells: 128^3 one point 1.11 / 0.65 ms, two 1.16 / 0.82, four 1.32 / 1.33, eight
// (1300, thin lens) 1.50 / 2.13; 64^3 eight 0.31 / 0.37; 256^3 telecentric eight
// 19.1 / 20.2.
constexpr int kQuadSegments = 250, kWideSegments = 800;
static bool segments_a_box(const vam_geometry* h, int least) {
  return h->seg_fwd.n >= least * (int64_t)h->n_boxes;
}

// The members' padded FP32 volumes side by side (vol_turn), allocated by the first
// call that needs them; false without that memory.  They are more than a call
// has to have, so they take at most half of what is free, are given back when
// the handle needs the memory for what it has to have (dev_alloc_for), and no
// call allocates them while its stream is captured.
static bool turned_volumes(vam_geometry* h, hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusActive;
  if (hipStreamIsCapturing(s, &status) != hipSuccess) (void)hipGetLastError();
  const bool capturing = status != hipStreamCaptureStatusNone;
  if (h->vol_turn) {
    if (capturing) h->vol_turn_captured = 1;
    return true;
  }
  size_t free_bytes = 0, total = 0;
  const size_t bytes = (size_t)h->pad_voxels * h->turn_members * sizeof(float);
  if (capturing || hipMemGetInfo(&free_bytes, &total) != hipSuccess || bytes > free_bytes / 2 ||
      dev_alloc(&h->vol_turn, bytes) != hipSuccess) {
    (void)hipGetLastError();  // handled here
    h->vol_turn = nullptr;
    return false;
  }
  return true;
}

// Default forward: every segment adds its partial to its pixel in 64-bit
// fixed point (scale from the volume's largest |value|), then one pass
// rounds the integers to the stored projections.  Variant 2 (below) writes
// FP32 partial sums instead and adds them per pixel in a fixed order.
// Workgroup sizes: 16-byte cells take 81 KB of LDS, so two workgroups fit a CU
// (four members, 256^3: 512 lanes 74.4 ms, 768 71.0, 1024 70.0; 128^3: 3.21,
// 3.19, 3.27); 8-byte cells 41 KB, four fit (256^3 telecentric, 90 angles: 512
// lanes 20.0 ms, 768 22.5, 1024 23.2).
template <int NQ>
static void launch_forward_turned(const vam_geometry* h, const MarchParams& P, const BoxParams& Bp, const float* vol,
                                  unsigned long long* pfx, double coef, hipStream_t s) {
  using Vec = typename CellVec<NQ>::T;
  auto launch = [&](auto kernel, int threads) {
    for_launches(Bp, threads, [&](dim3 grid, const BoxParams& part, int64_t a0) {
      MarchParams Pa = P;
      Pa.a0 += (int)a0;
      hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, Pa, part, (const Vec*)vol, pfx + a0 * Bp.npix * NQ,
                         h->vol_absmax, coef);
    });
  };
  if constexpr (NQ == 2)
    if (!segments_a_box(h, kWideSegments)) return launch(k_forward_turned<2, 512, Vec>, 512);
  launch(k_forward_turned<NQ, 768, float4>, 768);
}

// The members m0 .. m0 + n - 1 of every representative, NQ at a time.
template <int NQ, typename PT>
static vam_status forward_members(vam_geometry* h, const void* volume, PT* proj, int m0, int n, int fmt, double coef,
                                  hipStream_t s) {
  const int Q = h->turn_stride, T = h->turn_quarters;
  const int64_t npix = (int64_t)h->desc.n_u * h->desc.n_v, groups = Q * npix;
  const MarchParams P = march_params(h, 0);
  const BoxParams Bp = box_params(h, h->seg_fwd, Q, forward_order(h, Q));
  unsigned long long* pfx = (unsigned long long*)h->proj_fx;
  float* vol = (float*)h->vol_turn;
  for (int j = 0; j < n; j += NQ) {
    const int m = m0 + j;
    pad_turned<NQ>(h, volume, fmt, vol + j * h->pad_voxels, Turns{{m * T, (m + 1) * T, (m + 2) * T, (m + 3) * T}},
                   j == 0 ? h->vol_absmax : nullptr, s);
  }
  VAM_HIP_TRY(hipEventRecord(h->ev[0], s), "recording an event");
  for (int j = 0; j < n && h->n_boxes > 0; j += NQ)
    launch_forward_turned<NQ>(h, P, Bp, vol + j * h->pad_voxels, pfx + j * groups, coef, s);
  for (int j = 0; j < n; j += NQ)
    hipLaunchKernelGGL((k_fx_store_turned<PT, NQ>), dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s,
                       pfx + j * groups, proj + j * groups, groups, groups, h->vol_absmax, coef);
  return VAM_OK;
}

template <typename PT>
static vam_status forward_box_fx(vam_geometry* h, const void* volume, PT* proj, int a0, int na, int fmt,
                                 hipStream_t s) {
  const vam_geometry_desc& D = h->desc;
  const int64_t npix = (int64_t)D.n_u * D.n_v;
  if (!h->proj_fx) {
    VAM_HIP_TRY(dev_alloc((void**)&h->proj_fx, (int64_t)D.n_angles * npix * sizeof(int64_t)),
                "allocating the fixed-point projections");
  }
  if (!h->vol_absmax) VAM_HIP_TRY(dev_alloc((void**)&h->vol_absmax, sizeof(unsigned)), "allocating a maximum");
  const int Q = h->turn_stride, T = h->turn_quarters, m0 = a0 / Q, m1 = (a0 + na - 1) / Q;
  // members taken together (a chosen march mode or box edge takes one angle at
  // a time) and calls over several members need their volumes side by side;
  // without that memory the angles go one at a time, member after member, with
  // the same bits
  int nq = h->forward_lanes == 0 && h->boxes.B == kBox ? members_together(h, a0, na) : 1;
  const bool turned = m0 != m1 && turned_volumes(h, s);
  if (!turned) nq = 1;
  unsigned long long* pfx = (unsigned long long*)h->proj_fx;
  const int64_t n = (int64_t)na * npix;
  hipLaunchKernelGGL(k_fx_clear, dim3((unsigned)std::max<int64_t>((n + 255) / 256, 1)), dim3(256), 0, s, pfx, n,
                     h->vol_absmax);
  const double coef = D.step / D.n_pupil * (double)h->pix_samples_max;
  if (nq > 1) {
    const vam_status st = nq == 4 && segments_a_box(h, kQuadSegments)
                              ? forward_members<4>(h, volume, proj, m0, nq, fmt, coef, s)
                              : forward_members<2>(h, volume, proj, m0, nq, fmt, coef, s);
    if (st != VAM_OK) return st;
  } else {
    // one turned copy of the volume per member in the call, beside each other
    // (in vol_turn) and one launch, or without that memory one after the other
    const bool together = m0 == m1 || turned;
    void* vol = m0 == m1 ? (void*)h->vol_pad : h->vol_turn;
    for (int m = m0; m <= m1; ++m) {
      pad_turned<1>(h, volume, fmt, together ? (uint32_t*)vol + (m - m0) * h->pad_voxels : (uint32_t*)h->vol_pad,
                    Turns{{m * T, 0, 0, 0}}, m == m0 ? h->vol_absmax : nullptr, s);
      if (together && m < m1) continue;
      if (together || m == m0) VAM_HIP_TRY(hipEventRecord(h->ev[0], s), "recording an event");
      if (h->n_boxes == 0) continue;
      const int first = together ? a0 : std::max(a0, m * Q), last = together ? a0 + na : std::min(a0 + na, (m + 1) * Q);
      BoxParams Bp = box_params(h, h->seg_fwd, last - first, forward_order(h, last - first));
      Bp.turn_stride = Q;
      Bp.member0 = together ? m0 : m;
      // (128^3, 60 of 180 angles, FP32: one lane 1.75 ms, its words in
      // registers 1.47, FP32 cells 1.45; 64^3, 180 angles 0.51 and 0.48; FP16,
      // 45 angles of 128^3: 1.16, 1.16, 1.14.  At edge 16 the wide cells leave one
      // workgroup a CU: 90 angles of 128^3, FP32 / FP16 words in registers or one
      // lane 5.8 / 4.6 ms, FP32 cells 7.6 / 7.3; edge 8 about alike.)
      const int mode = h->forward_lanes          ? h->forward_lanes
                       : h->boxes.B == kBox      ? kMarchCells
                       : fmt == kVolF16Pairs     ? kMarchOne
                                                 : kMarchCached;
      const FwdOut o{nullptr, 0, pfx + (first - a0) * npix, h->vol_absmax, coef, mode};
      launch_forward_box_edge<true>(h->boxes.B, s, march_params(h, first), Bp, fmt,
                                    together ? (const uint32_t*)vol : (const uint32_t*)h->vol_pad, o);
    }
    hipLaunchKernelGGL(k_fx_store<PT>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, pfx, proj, n,
                       h->vol_absmax, coef);
  }
  VAM_HIP_TRY(hipGetLastError(), "launching the fixed-point forward projector");
  VAM_HIP_TRY(hipEventRecord(h->ev[1], s), "recording an event");
  return VAM_OK;
}

template <typename PT>
static vam_status forward_box_t(vam_geometry* h, const void* volume, PT* proj, int a0, int na, int fmt, hipStream_t s) {
  if (h->forward_variant != 2) return forward_box_fx(h, volume, proj, a0, na, fmt, s);
  const vam_geometry_desc& D = h->desc;
  pad_turned<1>(h, volume, fmt, h->vol_pad, Turns{}, nullptr, s);
  VAM_HIP_TRY(hipGetLastError(), "launching the volume copy");
  const MarchParams P0 = march_params(h, a0);
  VAM_HIP_TRY(hipEventRecord(h->ev[0], s), "recording an event");
  const int64_t slots = (int64_t)std::max(h->max_seg_per_ray, 1) * h->n_rays;
  if (!h->seg_part) {
    // partial sums for a chunk of angles, at most 8 GiB (fewer launch tails
    // and reductions than small chunks); if the device cannot hold that
    // much, halve the chunk until the allocation succeeds
    int64_t angles = std::max<int64_t>(1, std::min<int64_t>(D.n_angles, (int64_t(1) << 31) / slots));
    for (;;) {
      const hipError_t e = dev_alloc_for(h, (void**)&h->seg_part, slots * angles * sizeof(float));
      if (e == hipSuccess) break;
      h->seg_part = nullptr;
      if (e != hipErrorOutOfMemory || angles == 1) return hip_check(e, "allocating segment partial sums");
      (void)hipGetLastError();  // the failed allocation's error is handled here
      angles = (angles + 1) / 2;
    }
    h->seg_part_angles = (int)angles;
  }
  const int npix = D.n_u * D.n_v;
  for (int c0 = 0; c0 < na; c0 += h->seg_part_angles) {
    const int nc = std::min(h->seg_part_angles, na - c0);
    MarchParams P = P0;
    P.a0 = P0.a0 + c0;
    if (h->n_boxes > 0) {
      const BoxParams Bp = box_params(h, h->seg_fwd, nc, forward_order(h, nc));
      const FwdOut o{h->seg_part, slots, nullptr, nullptr, 0.0, kMarchOne};
      launch_forward_box_edge<false>(h->boxes.B, s, P, Bp, fmt, (const uint32_t*)h->vol_pad, o);
    }
    const int64_t n = (int64_t)nc * npix;
    hipLaunchKernelGGL(k_reduce_segments<PT>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, h->seg_part,
                       h->ray_nseg, proj + (int64_t)c0 * npix, npix, D.n_pupil, h->n_rays, slots, nc);
    VAM_HIP_TRY(hipGetLastError(), "launching the box-tiled forward projector");
  }
  VAM_HIP_TRY(hipEventRecord(h->ev[1], s), "recording an event");
  return VAM_OK;
}

vam_status launch_box_forward(vam_geometry* h, const void* vol, vam_dtype vol_t, void* proj, vam_dtype proj_t, int a0,
                              int na, hipStream_t s) {
  if (!h->boxes_ready)
    return fail(VAM_ERR_INVALID_ARG, "the box decomposition is not available (a rebuild failed); "
                                     "set the box edge again or create a new geometry");
  const int fmt = vol_t == VAM_BF16 ? kVolBF16Pairs : vol_t == VAM_F16 ? kVolF16Pairs : kVolF32;
  switch (proj_t) {
    case VAM_F32: return forward_box_t(h, vol, (float*)proj, a0, na, fmt, s);
    case VAM_BF16: return forward_box_t(h, vol, (uint16_t*)proj, a0, na, fmt, s);
    case VAM_F16: return forward_box_t(h, vol, (__half*)proj, a0, na, fmt, s);
  }
  return fail(VAM_ERR_INVALID_ARG, "unknown projection dtype");
}

// ------------------------------------------------------------- deposit ---
//
// The deposit adds 8 corner weights per sample into the (box, angle)
// workgroup's LDS footprint in 32-bit fixed point (gfx950 adds 32-bit
// integers in LDS ~45x faster than FP32 and ~2x faster than FP64), then adds
// each touched cell once to its voxel's 64-bit integer (a power-of-two scale
// from the call's largest |projection value|; integer adds commute, so the
// dose is deterministic).  Overflow in LDS is ruled
// out per workgroup: a cell's exact sum is at most bound = n x (step /
// n_pupil) x M, where n is the box's n_supp (the most samples of the box in
// any 4 x 4 x 3 block of lab-frame unit cells, which holds the turned
// support of any voxel), no sample weight exceeds step / n_pupil times |P|,
// and M is the largest |projection value| among the box's segments at this
// angle.  With S = (2^31 - n - 2^12)(1 - 2^-12) / bound, each of the at most
// n adds into a cell rounds a value that is within 2^-12 of exact (the FP32
// run sums of at most a few thousand same-sign terms) to the nearest
// integer, so every partial sum stays below 2^31 in magnitude; the rounding
// error of an add is at most 1/(2S) ~ bound 2^-32.  A non-finite
// projection value makes the whole dose NaN (the workgroups add nothing and
// the dose copy writes NaN).
//
// Run aggregation keeps the 8 corner sums of consecutive samples in one cell
// in registers and adds them to LDS when the cell changes; the sums restart
// through a factor keep in {0, 1} (w <- keep w + q, one FMA) rather than a
// branch, so the loop carries them without register copies.

template <typename PT>
__device__ inline float load_p(const PT* p, int64_t i);
template <>
__device__ inline float load_p<float>(const float* p, int64_t i) {
  return p[i];
}
template <>
__device__ inline float load_p<uint16_t>(const uint16_t* p, int64_t i) {
  return __uint_as_float((uint32_t)p[i] << 16);
}
template <>
__device__ inline float load_p<__half>(const __half* p, int64_t i) {
  return __half2float(p[i]);
}

// v clamped to [0, 1] (free as an instruction modifier).
__device__ inline float unit(float v) { return __builtin_amdgcn_fmed3f(v, 0.0f, 1.0f); }

// Round to the nearest integer, halves upwards (one v_cvt_rpi_i32_f32).
__device__ inline int round_to_int(float v) {
  int r;
  asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(v));
  return r;
}

template <int SY, int SZ>
__device__ inline void flush8(int* acc, unsigned cur, const float* w) {
  int* p = (int*)((char*)acc + cur);
  atomicAdd(p, round_to_int(w[0]));
  atomicAdd(p + 1, round_to_int(w[1]));
  atomicAdd(p + SY, round_to_int(w[2]));
  atomicAdd(p + SY + 1, round_to_int(w[3]));
  atomicAdd(p + SZ, round_to_int(w[4]));
  atomicAdd(p + SZ + 1, round_to_int(w[5]));
  atomicAdd(p + SZ + SY, round_to_int(w[6]));
  atomicAdd(p + SZ + SY + 1, round_to_int(w[7]));
}

// zc: the segment's z cell in the footprint, one for all its samples (WHOLE: each
// sample has its own, and zc is 0).
template <int SY, int SZ, bool CLAMP, bool WHOLE>
__device__ inline void march_deposit(int* acc, const SegPos& g, int zc, float e, float hx, float hy, float hz,
                                     float r_hi, float r_lo) {
  // at whole coordinates (see cell_number)
  auto cell_bytes = [](float x, float y, float z) {
    const float yx = fmaf(y, (float)(SY * 4), x * 4.0f);
    return (unsigned)(WHOLE ? fmaf(z, (float)(SZ * 4), yx) : yx);
  };
  acc += zc * SZ;
  const float pz = g.pz - (float)zc;
  float w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  // byte offset of the cell whose corners w holds, starting at the first
  // sample's (w is zero until its first add)
  unsigned cur = cell_bytes(floorf(coord<CLAMP>(g.k0, g.dx, g.px, hx)), floorf(coord<CLAMP>(g.k0, g.dy, g.py, hy)),
                            WHOLE ? floorf(coord<CLAMP>(g.k0, g.dz, pz, hz)) : 0.0f);
  // exact: a segment has fewer than 2^24 samples
  for (float kf = g.k0; kf <= g.k1; kf += 1.0f) {
    const float x = coord<CLAMP>(kf, g.dx, g.px, hx);
    const float y = coord<CLAMP>(kf, g.dy, g.py, hy);
    const float z = coord<CLAMP && WHOLE>(kf, g.dz, pz, hz);
    const float fx = __builtin_amdgcn_fractf(x), fy = __builtin_amdgcn_fractf(y);
    const float fz = WHOLE ? __builtin_amdgcn_fractf(z) : unit(z);
    const float z1 = e * fz, z0 = e - z1;
    const float y01 = z0 * fy, y00 = z0 - y01;
    const float y11 = z1 * fy, y10 = z1 - y11;
    const unsigned ob = cell_bytes(x - fx, y - fy, z - fz);
    const bool fl = ob != cur;
    if (fl) flush8<SY, SZ>(acc, cur, w);
    const float keep = fl ? 0.0f : 1.0f;
    cur = ob;
    // w[2j] += yz (1 - fx), w[2j+1] += yz fx, accumulated into w itself
    const float yz[4] = {y00, y01, y10, y11};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      w[2 * j] = fmaf(-yz[j], fx, fmaf(keep, w[2 * j], yz[j]));
      w[2 * j + 1] = fmaf(yz[j], fx, keep * w[2 * j + 1]);
    }
    e = fmaf(e, r_hi, e * r_lo);
  }
  flush8<SY, SZ>(acc, cur, w);  // a segment has at least one sample
}

// acc: the padded dose as 64-bit integers at the scale fx_scale(*pmax,
// dep_coef), pmax the largest |projection value| of the call (FP32 bits;
// a NaN or infinity among them leaves acc untouched: the dose copy then
// writes NaN everywhere).
// WHOLE: segments are not cut at z cells (see build_boxes_into), so samples form
// theirs (256^3, 360 angles of a thin lens: 179 ms; k_back_planes, which needs
// them cut, 104).
template <int B, typename PT, int NT, bool WHOLE>
__global__ __launch_bounds__(NT) void k_back_box(MarchParams P, BoxParams Bp, const PT* __restrict__ proj,
                                                 unsigned long long* __restrict__ acc64,
                                                 const unsigned* __restrict__ pmax, double dep_coef) {
  // slice pitch one word longer than a slice: 3 % faster than SY * SY at
  // edge 12 (the pitch decides which LDS banks the lanes' adds share)
  constexpr int SY = Fixed<B>::WXY, SZ = SY * SY + 1, NC = SZ * Fixed<B>::WZ;
  __shared__ int acc[NC];
  __shared__ unsigned s_pvmax;
  int b, a;
  if (!work_item(Bp.nboxes, Bp.na, Bp.xcd, b, a)) return;
  const unsigned pm = *pmax;
  if (pm >= 0x7f800000u) return;  // a non-finite projection value: the dose is NaN
  const double G = fx_scale(pm, dep_coef);
  const double2 cs = P.cs[P.a0 + a];
  const Foot f = footprint(Bp, Bp.box_id[b], cs.x, cs.y, P.cx, P.cy);
  for (int i = threadIdx.x; i < NC; i += blockDim.x) acc[i] = 0;
  if (threadIdx.x == 0) s_pvmax = 0u;
  __syncthreads();
  const float hx = (float)f.WX - 1.001f, hy = (float)f.WY - 1.001f, hz = (float)f.WZ - 1.001f;
  const int64_t pbase = (int64_t)a * Bp.npix;
  const int s_end = Bp.box_begin[b + 1];
  // the box's largest |projection value| at this angle sets the scale
  float m = 0.0f;
  for (int si = Bp.box_begin[b] + threadIdx.x; si < s_end; si += blockDim.x)
    m = fmaxf(m, fabsf(load_p(proj, pbase + Bp.seg.idx[si])));
  atomicMax(&s_pvmax, __float_as_uint(m));  // non-negative floats order as their bits
  __syncthreads();
  const int nb = Bp.box_supp[b];
  const double bound = (double)nb * Bp.w_coef * (double)__uint_as_float(s_pvmax);
  // capped below FP32's largest value (a smaller S only rounds coarser)
  const float S = bound > 0.0 ? (float)fmin((2147483648.0 - nb - 4096.0) * (1.0 - 1.0 / 4096.0) / bound, 3.0e38)
                              : 1.0f;
  // a cell's integer at the dose scale: raw / S x G, rounded (G a power of two)
  const double toG = G / (double)S;
  const float c = (float)cs.x, s = (float)cs.y, sc = P.step * c, ss = P.step * s;
  for (int si = Bp.box_begin[b] + threadIdx.x; si < s_end; si += blockDim.x) {
    const float pv = load_p(proj, pbase + Bp.seg.idx[si]);
    if (pv == 0.0f) continue;
    const float4 pw = Bp.seg.pw[si], dn = Bp.seg.dn[si];
    const SegPos g = seg_pos(pw, dn, seg_count(dn), f, c, s, sc, ss, P.step);
    const float e = pw.w * pv * S;  // sample weights in the fixed-point units
    const int zc = WHOLE ? 0 : min(max(seg_z_cell(dn) + (int)f.zoff, 0), f.WZ - 2);
    if (seg_inside(g, hx, hy, hz))
      march_deposit<SY, SZ, false, WHOLE>(acc, g, zc, e, hx, hy, hz, P.r_hi, P.r_lo);
    else
      march_deposit<SY, SZ, true, WHOLE>(acc, g, zc, e, hx, hy, hz, P.r_hi, P.r_lo);
  }
  __syncthreads();
  unsigned long long* tile = acc64 + tile_base(Bp, f);
  constexpr int COL = SY * SY, Z = kSlices<COL, NT>;
  for (int i = threadIdx.x; i < Z * COL; i += NT) {
    const int zg = Z == 1 ? 0 : i / COL, col = i - zg * COL, y = col / SY, x = col - y * SY;
    if (x >= f.WX || y >= f.WY) continue;
    for (int z = zg; z < f.WZ; z += Z) {
      const int raw = acc[z * SZ + col];
      if (raw != 0)
        atomicAdd(tile + (int64_t)z * Bp.py * Bp.px + (unsigned)(y * Bp.px + x),
                  (unsigned long long)__double2ll_rn((double)raw * toG));
    }
  }
}

// ------------------------------------------------ deposit, plane by plane --
//
// The deposit of four angles that are whole quarter turns apart (find_turns).
//
// What bounds a deposit that adds a run's 8 corners whenever a lane's cell
// changes (k_back_box): the LDS adds.  A wave's ds_add_u32 takes 4.3 clocks
// however few of its lanes are active, 7.8 with 64 unrelated ones; at 256^3
// each step of a wave issues 8 of them with 37 active lanes, 41 clocks of the
// 43 that a step takes.  So here the lanes add together and less often:
//
//  * A lane walks its segment along the axis (x or y) that it advances along
//    fastest, plane by plane.  All samples between planes j and j + 1 go
//    into registers: sums for the columns of plane j (started by the samples
//    before it) and of plane j + 1.  Then the whole wave adds plane j to LDS
//    and moves on.  A corner that several cells share is added once, and a
//    step covers 1 / |advance| >= 2 samples at the usual half-voxel spacing.
//  * The other axis and the direction are mirrored so that both coordinates
//    grow.  Between two planes the cross coordinate grows by less than one
//    cell, so a plane receives at most four columns, from the cell of its
//    first sample on.  Columns are kept as sums of clamp(u - i) over the
//    samples (u from the base column): the tent weights are their
//    differences, exactly zero in columns that no sample reached, which are
//    not added (so no add leaves the footprint).
//  * z does not turn: the deposit's segments end where their z cell changes,
//    so a segment has two z corners throughout.
//  * The four angles share all of it: the sums are free of the projection
//    value, and the members' sums of a corner leave as two 64-bit adds
//    (ds_add_u64: 12.8 clocks for 64 lanes, 6.4 a member), each the exact
//    integer hi 2^32 + lo of two members' 32-bit sums, whose bound is
//    k_back_box's: a corner gets at most one add per sample of its support.
//
// 256^3, 360 angles, 16 pupil points: 105 ms against 193 corner by corner with
// every pixel lit, 87 against 127 on projections dark outside a part's shadow
// (more sizes at launch_back_box_t).  With few segments a box the adds into the
// voxels bind, the same for both.  In the kernel's first form, which took 111 ms,
// the time without its LDS adds and their conversions was 82 ms, without the
// adds into the voxels 105: the adds and the vector work both bind, and neither
// hides the other fully.
// Two members, or one, per workgroup were slower in that form (128^3: 90 angles
// in pairs 3.01 ms against 3.30 corner by corner, but 23.4 against 21.0 at 256^3
// telecentric on dark-edged projections, and one angle 2.30 against 1.79): per
// member the vector work grows past what the adds save, so those go corner by
// corner.

// Largest value of the wave.
__device__ inline float wave_max(float m) {
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  return m;
}

constexpr int kTurns = 4;  // members of a work item

// Adds a corner's sums t f[q] of the members, rounded, at element `at`.
template <int PLANE>
__device__ inline void add_members(unsigned long long* acc, int at, float t, const float (&f)[kTurns]) {
#pragma unroll
  for (int p = 0; p < kTurns; p += 2) {
    const int lo = round_to_int(t * f[p]), hi = round_to_int(t * f[p + 1]) + (lo >> 31);
    atomicAdd(acc + p / 2 * PLANE + at, (unsigned long long)(uint32_t)lo | (unsigned long long)(uint32_t)hi << 32);
  }
}

// One segment.  m, c: main and cross coordinate of its middle sample, dm >= dc
// >= 0 their steps; element(m, c) = base + m sm + c sc is the footprint's
// corner in the lower z slice of the segment's cell.
template <int SZ, int PLANE, bool CLAMP>
__device__ inline void march_planes(unsigned long long* acc, float k0, float k1, float pm, float dm, float hm, float pc, float dc,
                                    float hc, float pz, float dz, int base, int sm, int sc, float e,
                                    const float (&f)[kTurns], float r_hi, float r_lo) {
  float A[2][4] = {}, B[2][3] = {};  // [z][column sums] of the planes jf and jf + 1
  float kf = k0;
  float m = coord<CLAMP>(kf, dm, pm, hm);
  float jf = floorf(m);
  float bB = floorf(coord<CLAMP>(kf, dc, pc, hc)), bA = bB;
  bool last = false;
  for (;;) {
    const float end = jf + 1.0f;
    while (kf <= k1 && !(m >= end)) {
      const float c = coord<CLAMP>(kf, dc, pc, hc);
      const float fz = unit(fmaf(kf, dz, pz)), fm = unit(m - jf);
      const float a1 = unit(c - bA), a2 = unit(c - (bA + 1.0f)), a3 = unit(c - (bA + 2.0f));
      const float b1 = unit(c - bB), b2 = unit(c - (bB + 1.0f));
      const float e1 = e * fz, ez[2] = {e - e1, e1};
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        const float wb = ez[z] * fm, wa = ez[z] - wb;
        A[z][0] += wa;
        A[z][1] = fmaf(wa, a1, A[z][1]);
        A[z][2] = fmaf(wa, a2, A[z][2]);
        A[z][3] = fmaf(wa, a3, A[z][3]);
        B[z][0] += wb;
        B[z][1] = fmaf(wb, b1, B[z][1]);
        B[z][2] = fmaf(wb, b2, B[z][2]);
      }
      e = fmaf(e, r_hi, e * r_lo);
      kf += 1.0f;
      m = coord<CLAMP>(kf, dm, pm, hm);
    }
    int at = base + (int)jf * sm + (int)bA * sc;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float t0 = i < 3 ? A[0][i] - A[0][i + 1] : A[0][3], t1 = i < 3 ? A[1][i] - A[1][i + 1] : A[1][3];
      if (fabsf(t0) + fabsf(t1) != 0.0f) {
        add_members<PLANE>(acc, at, t0, f);
        add_members<PLANE>(acc, at + SZ, t1, f);
      }
      at += sc;
    }
    if (last) break;
    last = !(kf <= k1);
#pragma unroll
    for (int z = 0; z < 2; ++z) {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        A[z][i] = B[z][i];
        B[z][i] = 0.0f;
      }
      A[z][3] = 0.0f;
    }
    jf = end;
    bA = bB;
    bB = floorf(coord<CLAMP>(kf, dc, pc, hc));
  }
}

// Work item (b, a): the box at the members of representative angle P.a0 + a: rows a,
// a + member_rows, ... of proj, member q turned by q quarter turns.  acc64, pmax, dep_coef: as for k_back_box.
template <typename PT, int NT>
__global__ __launch_bounds__(NT) void k_back_planes(MarchParams P, BoxParams Bp, const PT* __restrict__ proj,
                                                    int64_t member_rows,
                                                    unsigned long long* __restrict__ acc64,
                                                    const unsigned* __restrict__ pmax, double dep_coef) {
  constexpr int SY = Fixed<kBox>::WXY, SZ = SY * SY + 1, PLANE = SZ * Fixed<kBox>::WZ;
  constexpr int NQ = kTurns, NC = PLANE * (NQ / 2);
  __shared__ unsigned long long acc[NC];
  __shared__ unsigned s_pvmax[NQ];
  int b, a;
  if (!work_item(Bp.nboxes, Bp.na, Bp.xcd, b, a)) return;
  const unsigned pm_bits = *pmax;
  if (pm_bits >= 0x7f800000u) return;  // a non-finite projection value: the dose is NaN
  const double G = fx_scale(pm_bits, dep_coef);
  const double2 cs = P.cs[P.a0 + a];
  const Foot f = footprint(Bp, Bp.box_id[b], cs.x, cs.y, P.cx, P.cy);
  for (int i = threadIdx.x; i < NC; i += NT) acc[i] = 0;
  if (threadIdx.x < NQ) s_pvmax[threadIdx.x] = 0u;
  __syncthreads();
  const PT* rows[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) rows[q] = proj + (a + q * member_rows) * Bp.npix;
  const int s_begin = Bp.box_begin[b], s_end = Bp.box_begin[b + 1];
  // the box's largest |projection value| of each member sets its scale
  {
    float mx[NQ] = {};
    for (int si = s_begin + (int)threadIdx.x; si < s_end; si += NT) {
      const int pix = Bp.seg.idx[si];
#pragma unroll
      for (int q = 0; q < NQ; ++q) mx[q] = fmaxf(mx[q], fabsf(load_p(rows[q], pix)));
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float w = wave_max(mx[q]);
      if ((threadIdx.x & 63) == 0) atomicMax(&s_pvmax[q], __float_as_uint(w));  // non-negative floats order as their bits
    }
  }
  __syncthreads();
  const int nb = Bp.box_supp[b];
  float S[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const double bound = (double)nb * Bp.w_coef * (double)__uint_as_float(s_pvmax[q]);
    // capped below FP32's largest value (a smaller S only rounds coarser)
    S[q] = bound > 0.0 ? (float)fmin((2147483648.0 - nb - 4096.0) * (1.0 - 1.0 / 4096.0) / bound, 3.0e38) : 1.0f;
  }
  const float hx = (float)f.WX - 1.001f, hy = (float)f.WY - 1.001f, hz = (float)f.WZ - 1.001f;
  const float c = (float)cs.x, s = (float)cs.y, sc = P.step * c, ss = P.step * s;
  // (the next round's pixel is loaded a round ahead: its projection values
  // wait for it)
  int next = s_begin + (int)threadIdx.x < s_end ? Bp.seg.idx[s_begin + (int)threadIdx.x] : 0;
  for (int si = s_begin + (int)threadIdx.x; si < s_end; si += NT) {
    const int pix = next;
    if (si + NT < s_end) next = Bp.seg.idx[si + NT];
    float v[NQ];
    bool lit = false;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float pv = load_p(rows[q], pix);
      lit |= pv != 0.0f;
      v[q] = pv * S[q];  // sample weights in the fixed-point units
    }
    if (!lit) continue;
    const float4 pw = Bp.seg.pw[si], dn = Bp.seg.dn[si];
    const SegPos g = seg_pos(pw, dn, seg_count(dn), f, c, s, sc, ss, P.step);
    // main axis, and both axes mirrored to grow along the segment
    const bool x_main = fabsf(g.dx) > fabsf(g.dy);
    float m = x_main ? g.px : g.py, dm = x_main ? g.dx : g.dy, u = x_main ? g.py : g.px, du = x_main ? g.dy : g.dx;
    const int wm = x_main ? f.WX : f.WY, wu = x_main ? f.WY : f.WX;
    int sm = x_main ? 1 : SY, su = x_main ? SY : 1;
    const int iz = min(max(seg_z_cell(dn) + (int)f.zoff, 0), f.WZ - 2);
    int base = iz * SZ;
    if (dm < 0.0f) {
      m = (float)(wm - 1) - m;
      dm = -dm;
      base += (wm - 1) * sm;
      sm = -sm;
    }
    if (du < 0.0f) {
      u = (float)(wu - 1) - u;
      du = -du;
      base += (wu - 1) * su;
      su = -su;
    }
    const float z = g.pz - (float)iz;
    if (seg_inside(g, hx, hy, hz))
      march_planes<SZ, PLANE, false>(acc, g.k0, g.k1, m, dm, 0.0f, u, du, 0.0f, z, g.dz, base, sm, su, pw.w, v,
                                         P.r_hi, P.r_lo);
    else
      march_planes<SZ, PLANE, true>(acc, g.k0, g.k1, m, dm, (float)wm - 1.001f, u, du, (float)wu - 1.001f, z, g.dz,
                                        base, sm, su, pw.w, v, P.r_hi, P.r_lo);
  }
  __syncthreads();
  // each touched cell to its voxel, members turned back; an odd number of
  // quarter turns is read along y, which is the volume's x then
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const double toG = G / (double)S[q];
    // volume voxel of footprint cell (x, y, z): tile[z pz + y py + x px]
    const int64_t X = f.X0, Y = f.Y0;
    int64_t first;
    int px, py;
    if (q == 0) { first = Y * Bp.px + X; px = 1; py = Bp.px; }
    else if (q == 1) { first = (Bp.py - 1 - X) * Bp.px + Y; px = -Bp.px; py = 1; }
    else if (q == 2) { first = (Bp.py - 1 - Y) * Bp.px + (Bp.px - 1 - X); px = -1; py = -Bp.px; }
    else { first = X * Bp.px + (Bp.px - 1 - Y); px = Bp.px; py = -1; }
    unsigned long long* tile = acc64 + (int64_t)f.Z0 * Bp.py * Bp.px + first;
    constexpr int COL = SY * SY, Z = kSlices<COL, NT>;
    for (int i = threadIdx.x; i < Z * COL; i += NT) {
      const int zg = Z == 1 ? 0 : i / COL, rem = i - zg * COL, hi = rem / SY, lo = rem - hi * SY;
      const int x = q & 1 ? hi : lo, y = q & 1 ? lo : hi;
      if (x >= f.WX || y >= f.WY) continue;
      for (int z = zg; z < f.WZ; z += Z) {
        const unsigned long long w = acc[q / 2 * PLANE + z * SZ + y * SY + x];
        int raw = (int)(uint32_t)w;
        if (q & 1) raw = (int)(((long long)w - (long long)raw) >> 32);
        if (raw != 0)
          atomicAdd(tile + (int64_t)z * Bp.py * Bp.px + (y * py + x * px),
                    (unsigned long long)__double2ll_rn((double)raw * toG));
      }
    }
  }
}

// Largest |value| of the na x npix projections of a call, as FP32 bits
// (a NaN or infinity compares above every finite value).  16-byte loads
// between the caller's first and last 16-byte boundary, single values outside
// (67 us with one atomic per wave at 90 x 64^2, now 5 us; 115 -> 25 us at
// 360 x 256^2).
template <typename PT>
__device__ inline unsigned word_max(uint32_t w) {
  if constexpr (std::is_same<PT, float>::value) return abs_bits<kVolF32>(w);
  else if constexpr (std::is_same<PT, __half>::value) return abs_bits<kVolF16Pairs>(w);
  else return abs_bits<kVolBF16Pairs>(w);
}

template <typename PT>
__global__ __launch_bounds__(1024) void k_proj_absmax(const PT* __restrict__ proj, int64_t n, unsigned* __restrict__ pmax) {
  constexpr int PER = 16 / sizeof(PT);
  unsigned m = 0u;
  const int64_t step = (int64_t)gridDim.x * blockDim.x, t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t head = min<int64_t>(n, (int64_t)((16u - ((uintptr_t)proj & 15u)) & 15u) / (int)sizeof(PT));
  const int64_t body = (n - head) / PER, tail = n - head - body * PER;
  const uint4* p4 = (const uint4*)(proj + head);
  for (int64_t i = t; i < body; i += step) {
    const uint4 w = p4[i];
    m = max(max(m, max(word_max<PT>(w.x), word_max<PT>(w.y))), max(word_max<PT>(w.z), word_max<PT>(w.w)));
  }
  if (t < head) m = max(m, __float_as_uint(load_p(proj, t)) & 0x7fffffffu);
  if (t < tail) m = max(m, __float_as_uint(load_p(proj, n - 1 - t)) & 0x7fffffffu);
  m = block_max(m);
  if (threadIdx.x == 0) raise_max(pmax, m);
}

// Bound on a voxel's dose per unit of the largest |projection value|: per
// angle at most supp_bound samples meet its support, each of weight at most
// step / n_pupil.
double deposit_coef(const vam_geometry* h, int na) {
  return (double)na * (double)std::max<int64_t>(h->supp_bound, 1) * h->desc.step / h->desc.n_pupil;
}

// Work order of the deposit where none was chosen: angles (or representatives)
// in blocks of 4.  Corner by corner, blocks of 4 / 8: 180 angles of 128^3,
// telecentric with one pupil point 4.09 / 4.27 ms, on projections dark outside a
// part's shadow 2.58 / 2.69, 90 angles of 256^3 with eight points on such 19.7 /
// 20.0, 45 of 180 angles of 128^3 through a lens 1.89 / 1.89; plane by plane, 180
// angles of 128^3 4.12 / 4.18, 360 of 256^3 105.3 / 105.0.
static int deposit_order(const vam_geometry* h) { return h->xcd_deposit >= 0 ? h->xcd_deposit : 4; }

template <int B, typename PT>
static void launch_back_box(vam_geometry* h, const MarchParams& P, const PT* proj, int na, double* acc,
                            hipStream_t s) {
  const BoxParams Bp = box_params(h, h->seg_dep, na, deposit_order(h));
  unsigned long long* a64 = (unsigned long long*)acc;
  const unsigned* pm = (const unsigned*)(acc + h->pad_voxels);
  const double coef = deposit_coef(h, na);
  auto launch = [&](auto kernel, int threads) {
    for_launches(Bp, threads, [&](dim3 grid, const BoxParams& part, int64_t a0) {
      MarchParams Pa = P;
      Pa.a0 += (int)a0;
      hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, Pa, part, proj + a0 * Bp.npix, a64, pm, coef);
    });
  };
  if (h->deposit_whole)
    launch(k_back_box<B, PT, 256, true>, 256);
  else if (h->deposit_threads == 512)
    launch(k_back_box<B, PT, 512, false>, 512);
  else
    launch(k_back_box<B, PT, 256, false>, 256);
}

template <typename PT>
static void launch_back_box_t(vam_geometry* h, const MarchParams& P, const PT* proj, int na, double* acc,
                              hipStream_t s) {
  // the largest |projection value| first (its slot was cleared with acc)
  const int64_t n = (int64_t)na * h->desc.n_u * h->desc.n_v;
  hipLaunchKernelGGL(k_proj_absmax<PT>, max_grid(n), dim3(1024), 0, s, proj, n, (unsigned*)(acc + h->pad_voxels));
  // plane by plane for whole turns of quarter-turn angles where no plane
  // between two samples is skipped and the boxes hold enough segments to fill
  // its workgroups (and at the default edge and workgroup size); else corner
  // by corner.  128^3, 180 angles, planes / corners, telecentric: 1 pupil point
  // (150 segments a box) 4.16 / 4.13 ms, 2 points 4.65 / 4.75, 4 points (650) 4.84 /
  // 5.02, 8 points 5.17 / 6.91; on projections dark outside a part's shadow 2.82 /
  // 2.56, 3.19 / 3.05, 3.57 / 3.43, 4.36 / 5.08.  Thin lens, dark: 1.77 / 1.69, 1.95 /
  // 1.91, 2.21 / 2.59, 3.37 / 4.45.  64^3, 180 angles, 1 point 0.60 / 0.58, dark 0.47 / 0.37.
  if (h->boxes.B == kBox && h->desc.step <= 0.99 && h->deposit_threads == 256 && !h->deposit_whole &&
      h->seg_dep.n >= 500 * (int64_t)h->n_boxes && members_together(h, P.a0, na) == 4) {
    // two workgroups fit a CU's LDS: 24 waves at 77 registers (256^3: 512 lanes
    // 141 ms, 768 120; 1024 need 64 registers to fit twice, 170 in one)
    constexpr int NT = 768;
    const BoxParams Bp = box_params(h, h->seg_dep, h->turn_stride, deposit_order(h));
    for_launches(Bp, NT, [&](dim3 grid, const BoxParams& part, int64_t a0) {
      MarchParams Pa = P;
      Pa.a0 += (int)a0;
      hipLaunchKernelGGL((k_back_planes<PT, NT>), grid, dim3(NT), 0, s, Pa, part, proj + a0 * Bp.npix,
                         (int64_t)h->turn_stride, (unsigned long long*)acc, (const unsigned*)(acc + h->pad_voxels),
                         deposit_coef(h, na));
    });
    return;
  }
  switch (h->boxes.B) {
    case 8: launch_back_box<8, PT>(h, P, proj, na, acc, s); break;
    case 12: launch_back_box<12, PT>(h, P, proj, na, acc, s); break;
    default: launch_back_box<16, PT>(h, P, proj, na, acc, s); break;
  }
}

vam_status launch_box_deposit(vam_geometry* h, const MarchParams& P, const void* proj, vam_dtype proj_t, int na,
                              double* acc, hipStream_t s) {
  if (!h->boxes_ready)
    return fail(VAM_ERR_INVALID_ARG, "the box decomposition is not available (a rebuild failed); "
                                     "set the box edge again or create a new geometry");
  if (h->n_boxes == 0) return VAM_OK;
  switch (proj_t) {
    case VAM_F32: launch_back_box_t(h, P, (const float*)proj, na, acc, s); break;
    case VAM_BF16: launch_back_box_t(h, P, (const uint16_t*)proj, na, acc, s); break;
    case VAM_F16: launch_back_box_t(h, P, (const __half*)proj, na, acc, s); break;
  }
  return VAM_OK;
}

}  // namespace vam
