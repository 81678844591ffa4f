// Device-side candidate generation, per-frame argmax and the warm-start chain of
// Algorithm 1 (Sec. 3.2): see chain.hpp for how the kernels surround a launch of the
// search kernels.
#include <math.h>

#include "chain.hpp"

namespace prnu {

namespace {

// Grid nodes in FP64, generated exactly as centre + (k - (n - 1) / 2) * step with every
// product and sum rounded on its own (no fused multiply-add), the form the host-side
// grid helpers use, so that the device and the host name the same candidates.
#pragma clang fp contract(off)
__device__ double grid_node_d(int k, int n, double lo, double hi) {
  const double centre = (lo + hi) / 2.0;
  const double step = n > 1 ? (hi - lo) / (double)(n - 1) : 0.0;
  const double half = (double)(n - 1) / 2.0;
  return centre + ((double)k - half) * step;
}

__device__ double local_node_d(int k, int n, double centre, double step) {
  const double half = (double)(n - 1) / 2.0;
  return centre + ((double)k - half) * step;
}

// Inverse-warp coefficients of a candidate (Eq. 4, similarity form):
// a = cos(theta) / s, b = sin(theta) / s in FP64, rounded once to float.
__device__ CandParam param_of(const CandSite& c, int slot, int fslot) {
  const double th = c.t * (3.14159265358979323846 / 180.0);
  double sn, cs;
  sincos(th, &sn, &cs);
  CandParam p;
  p.a = (float)(cs / c.s);
  p.b = (float)(sn / c.s);
  p.frame = slot;
  p.fp = fslot;
  return p;
}
#pragma clang fp contract(on)

__device__ CandSite gen_site(const GridGen& g, int i) {
  if (g.kind == kGenList) return g.list[i];
  const int si = i / g.nr, ri = i % g.nr;
  if (g.kind == kGenFull) return CandSite{grid_node_d(si, g.ns, g.lo0, g.hi0), grid_node_d(ri, g.nr, g.lo1, g.hi1)};
  const ChainState c = *g.centre;
  return CandSite{local_node_d(si, g.ns, c.cs, g.lo0), local_node_d(ri, g.nr, c.ct, g.lo1)};
}

// Candidate i of an item into the launch's list.
__device__ __forceinline__ void gen_candidate(const ItemDesc& it, int i, CandParam* cand, CandSite* site) {
  const CandSite c = gen_site(it.gen, i);
  cand[it.off + i] = param_of(c, it.slot, it.fslot);
  site[it.off + i] = c;
}

// The launch's candidate list; n_dev (if any), the length of its fallback list, starts
// from zero.
__global__ __launch_bounds__(256) void k_gen(const ItemDesc* items, CandParam* cand, CandSite* site, int* n_dev) {
  if (n_dev && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *n_dev = 0;
  const ItemDesc& it = items[blockIdx.x];
  const int i = (int)blockIdx.y * 256 + (int)threadIdx.x;
  if (i < it.n) gen_candidate(it, i, cand, site);
}

// x beats the current best (bv, bi): finite comparison in FP64, the lower index on
// equal scores, NaN never.
__device__ __forceinline__ bool beats(double v, int i, double bv, int bi) {
  if (v != v) return false;
  return bi < 0 || v > bv || (v == bv && i < bi);
}

// Best of records [0, n) (index -1 if every score is NaN), valid in thread 0.
template <int T>
__device__ void segment_best(const CandRecord* rec, int n, double& bv, int& bi) {
  __shared__ double sv[T / 64];
  __shared__ int si[T / 64];
  bv = 0.0;
  bi = -1;
  for (int i = (int)threadIdx.x; i < n; i += T) {
    const double v = rec[i].pce;
    if (beats(v, i, bv, bi)) {
      bv = v;
      bi = i;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ov = __shfl_xor(bv, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (oi >= 0 && beats(ov, oi, bv, bi)) {
      bv = ov;
      bi = oi;
    }
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) {
    sv[w] = bv;
    si[w] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < T / 64; ++k)
      if (si[k] >= 0 && beats(sv[k], si[k], bv, bi)) {
        bv = sv[k];
        bi = si[k];
      }
  }
}

// Fold segment best (record r at list position idx, or none when idx < 0) into the
// running best; candidates of earlier segments win ties.
__device__ void fold(FrameBest& fb, const CandRecord* rec, const CandSite* site, int bi, int base, int n) {
  if (bi >= 0) {
    const double v = rec[bi].pce;
    if (fb.index < 0 || v > fb.rec.pce) {
      fb.rec = rec[bi];
      fb.s = site[bi].s;
      fb.t = site[bi].t;
      fb.index = base + bi;
    }
  }
  fb.n_eval = base + n;
}

// The frame's result record and the centre of the video's next local grid.
__device__ void commit(const ItemDesc& it, const FrameBest& fb) {
  prnu_frame_result r;
  r.pce = 0.0;
  r.rho = 0.0;
  r.scale = 0.0;
  r.rot_deg = 0.0;
  r.dx = r.dy = 0;
  r.cand_index = 0;
  r.fell_back = fb.fell_back;
  r.n_evaluated = fb.n_eval;
  r.iterations = it.mode == kModeRefine ? it.iter : 0;
  r.used_init = 0;
  if (fb.index < 0) {
    r.status = PRNU_E_NONFINITE;
    r.pce = __builtin_nan("");
  } else {
    r.pce = fb.rec.pce;
    r.rho = fb.rec.rho;
    r.scale = fb.s;
    r.rot_deg = fb.t;
    r.dx = fb.rec.dx;
    r.dy = fb.rec.dy;
    r.cand_index = fb.index;
    r.status = isfinite(fb.rec.pce) ? PRNU_OK : PRNU_E_NONFINITE;
    if (it.state) {
      it.state->cs = fb.s;
      it.state->ct = fb.t;
      it.state->have = 1;
    }
  }
  if (it.result) *it.result = r;
}

// One block per item over its segment of the launch's list: the item's best, and for a
// warm item whose local best falls short the fallback grid, which takes the next fb_n
// places of the fallback list (in any order of the items: a candidate's score does not
// depend on its place) and is written there by the block.
template <int T>
__global__ __launch_bounds__(T) void k_argmax(const ItemDesc* items, ItemOut* outs, const CandRecord* rec,
                                              const CandSite* site, int* n_dev, CandParam* fb_cand,
                                              CandSite* fb_site) {
  const ItemDesc& it = items[blockIdx.x];
  ItemOut& out = outs[blockIdx.x];
  __shared__ int fb_at;  // the fallback grid's first place, or -1
  double bv;
  int bi;
  const CandRecord* r = rec + it.off;
  const CandSite* c = site + it.off;
  segment_best<T>(r, it.n, bv, bi);
  if (threadIdx.x == 0) {
    FrameBest fb;
    if (it.mode == kModeRefine && it.merge) {
      fb = *it.best;
    } else {
      fb.index = -1;
      fb.n_eval = 0;
      fb.fell_back = 0;
      fb.pad = 0;
      fb.s = fb.t = 0.0;
      fb.rec = CandRecord{};
    }
    fold(fb, r, c, bi, fb.n_eval, it.n);
    int need = 0;
    if (it.mode == kModeWarm) {
      if (!it.state->have) {
        // no earlier frame of the video has a finite result: this frame is searched like
        // a first frame, on the full grid alone (the local segment does not count)
        fb.index = -1;
        fb.n_eval = 0;
        fb.fell_back = 0;
        need = 1;
      } else {
        // the local best falls short (or nothing finite was scored): the full grid follows
        need = (bi < 0 || !(r[bi].pce >= it.fallback_pce)) ? 1 : 0;
        fb.fell_back = need;
      }
    }
    fb_at = need ? atomicAdd(n_dev, it.fb_n) : -1;
    out.need = need;
    out.fb_off = need ? fb_at : 0;
    out.seg_index = bi;
    out.seg_s = bi >= 0 ? c[bi].s : 0.0;
    out.seg_t = bi >= 0 ? c[bi].t : 0.0;
    out.seg_pce = bi >= 0 ? r[bi].pce : 0.0;
    *it.best = fb;
    if (!need) commit(it, fb);
  }
  if (it.mode != kModeWarm) return;  // uniform per block
  __syncthreads();
  if (fb_at < 0) return;
  for (int i = (int)threadIdx.x; i < it.fb_n; i += T) {
    const CandSite x = gen_site(it.full, i);
    fb_cand[fb_at + i] = param_of(x, it.slot, it.fslot);
    fb_site[fb_at + i] = x;
  }
}

// One block per warm item after its fallback grid, if it needed one, was searched: the
// grid's best folded into the frame's.  With next (one item only), the block then
// generates the video's next item, whose centre the frame's result has set, in the same
// launch.
template <int T>
__global__ __launch_bounds__(T) void k_merge(const ItemDesc* items, const ItemOut* outs, const CandRecord* fb_rec,
                                             const CandSite* fb_site, const ItemDesc* next, CandParam* cand,
                                             CandSite* site, int* n_dev) {
  const ItemDesc& it = items[blockIdx.x];
  const ItemOut& out = outs[blockIdx.x];
  if (it.mode == kModeWarm && out.need) {  // uniform per block
    double bv;
    int bi;
    const CandRecord* r = fb_rec + out.fb_off;
    const CandSite* c = fb_site + out.fb_off;
    segment_best<T>(r, it.fb_n, bv, bi);
    if (threadIdx.x == 0) {
      FrameBest fb = *it.best;
      fold(fb, r, c, bi, fb.n_eval, it.fb_n);
      *it.best = fb;
      commit(it, fb);
    }
  }
  if (!next) return;
  __syncthreads();  // the state the next item's grid is centred on
  if (threadIdx.x == 0) *n_dev = 0;
  const ItemDesc nx = *next;
  for (int i = (int)threadIdx.x; i < nx.n; i += T) gen_candidate(nx, i, cand, site);
}

__global__ void k_chain_init(ChainState* st, int has_init, double cs, double ct) {
  st->cs = cs;
  st->ct = ct;
  st->have = has_init;
  st->pad = 0;
}

__global__ void k_put(Blob blob, unsigned char* dst) {
  for (int i = (int)threadIdx.x; i < blob.n; i += (int)blockDim.x) dst[i] = blob.b[i];
}

__global__ void k_scatter(const CandRecord* rec, int n, double* pce, double* rho, int32_t* dx, int32_t* dy) {
  const int i = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (i >= n) return;
  const CandRecord r = rec[i];
  if (pce) pce[i] = r.pce;
  if (rho) rho[i] = r.rho;
  if (dx) dx[i] = r.dx;
  if (dy) dy[i] = r.dy;
}

}  // namespace

hipError_t launch_gen(const ItemDesc* items, int n, int max_n, CandParam* cand, CandSite* site, int* n_dev,
                      hipStream_t s) {
  if (n <= 0 || max_n <= 0) return hipSuccess;
  k_gen<<<dim3((unsigned)n, (unsigned)((max_n + 255) / 256)), 256, 0, s>>>(items, cand, site, n_dev);
  return hipGetLastError();
}

hipError_t launch_argmax(const ItemDesc* items, int n, ItemOut* outs, const CandRecord* rec, const CandSite* site,
                         int* n_dev, CandParam* fb_cand, CandSite* fb_site, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_argmax<256><<<dim3((unsigned)n), 256, 0, s>>>(items, outs, rec, site, n_dev, fb_cand, fb_site);
  return hipGetLastError();
}

hipError_t launch_merge(const ItemDesc* items, int n, const ItemOut* outs, const CandRecord* fb_rec,
                        const CandSite* fb_site, const ItemDesc* next, CandParam* cand, CandSite* site, int* n_dev,
                        hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (next && n != 1) return hipErrorInvalidValue;
  k_merge<256><<<dim3((unsigned)n), 256, 0, s>>>(items, outs, fb_rec, fb_site, next, cand, site, n_dev);
  return hipGetLastError();
}

hipError_t launch_chain_init(ChainState* st, int has_init, double cs, double ct, hipStream_t s) {
  k_chain_init<<<1, 1, 0, s>>>(st, has_init, cs, ct);
  return hipGetLastError();
}

hipError_t launch_put(const Blob& blob, void* dst, hipStream_t s) {
  if (blob.n <= 0) return hipSuccess;
  k_put<<<1, 256, 0, s>>>(blob, reinterpret_cast<unsigned char*>(dst));
  return hipGetLastError();
}

hipError_t launch_scatter(const CandRecord* rec, int n, double* pce, double* rho, int32_t* dx, int32_t* dy,
                          hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_scatter<<<dim3((unsigned)((n + 255) / 256)), 256, 0, s>>>(rec, n, pce, rho, dx, dy);
  return hipGetLastError();
}

}  // namespace prnu
