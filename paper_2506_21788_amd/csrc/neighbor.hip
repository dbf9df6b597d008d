// Radius graph on the GPU: cell-list candidate search, exact float32 cutoff test, destination-sorted
// CSR with rows ordered by (source, shift), and the source-sorted transpose plan.
//
// Design for gfx950: atoms are sorted by bin (bins live in fractional coordinates of the graph's cell, at least
// one cutoff wide wherever the cell allows it; cells thinner than the cutoff are covered by integer image shifts
// instead) into an array of (x, y, z, atom) quadruples, so a bin's atoms are one contiguous run of 16-byte records.
// A workgroup takes up to 16 destination atoms of ONE bin: it stages the shifted positions of every candidate of
// the (2R+1)^3 bins around it in LDS once (coalesced loads, no pointer chasing) and each wavefront then tests
// whole groups of 64 candidates per destination atom out of LDS; hits are compacted with a ballot into a per-
// wavefront LDS row, ranked there against each other (rows are short) and written out in (source, shift) order.
// The same kernel counts (first call) and fills (second call). Rows with more hits than the LDS row holds are
// walked again and ranked from memory. Only integer atomics are used (bin histogram / cursors); the
// output does not depend on their order.
//
// The cutoff test is the one fixed in include/hgnn.h: each float operation is an explicitly rounded
// intrinsic so that the compiler cannot contract them into fused multiply-adds.
#include "common.h"
#include "prof.h"

namespace hgnn {

// ---------------------------------------------------------------------------------------------
// error text (thread local), shared by all translation units
// ---------------------------------------------------------------------------------------------
static thread_local char g_err[512] = "";

int32_t set_error(int32_t code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

// ---------------------------------------------------------------------------------------------
// exclusive scan (three small kernels; block sums kept in int64 so that overflow is detectable)
// ---------------------------------------------------------------------------------------------
constexpr int SCAN_T = 256;
constexpr int SCAN_PER = 4;
constexpr int SCAN_BLK = SCAN_T * SCAN_PER;

__device__ inline int block_exclusive_scan_256(int v, int* total, int* sh) {
  // sh: 256 ints. Hillis-Steele inclusive scan, then shift.
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int o = 1; o < SCAN_T; o <<= 1) {
    int add = (t >= o) ? sh[t - o] : 0;
    __syncthreads();
    sh[t] += add;
    __syncthreads();
  }
  int incl = sh[t];
  *total = sh[SCAN_T - 1];
  __syncthreads();
  return incl - v;
}

__global__ void k_scan_local(const int32_t* __restrict__ in, int32_t* __restrict__ out, int64_t n,
                             long long* __restrict__ blocksum) {
  __shared__ int sh[SCAN_T];
  const int64_t base = (int64_t)blockIdx.x * SCAN_BLK + (int64_t)threadIdx.x * SCAN_PER;
  int v[SCAN_PER];
  int s = 0;
#pragma unroll
  for (int k = 0; k < SCAN_PER; ++k) {
    v[k] = (base + k < n) ? in[base + k] : 0;
    s += v[k];
  }
  int tot;
  int ex = block_exclusive_scan_256(s, &tot, sh);
#pragma unroll
  for (int k = 0; k < SCAN_PER; ++k) {
    if (base + k < n) out[base + k] = ex;
    ex += v[k];
  }
  if (threadIdx.x == 0) blocksum[blockIdx.x] = tot;
}

__global__ void k_scan_blocksums(long long* __restrict__ blocksum, int64_t nb) {
  // single thread block; serial carry over chunks of 256 block sums (nb is small)
  __shared__ long long sh[SCAN_T];
  __shared__ long long carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t c0 = 0; c0 < nb; c0 += SCAN_T) {
    const int64_t idx = c0 + threadIdx.x;
    long long v = idx < nb ? blocksum[idx] : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < SCAN_T; o <<= 1) {
      long long add = (threadIdx.x >= o) ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += add;
      __syncthreads();
    }
    long long incl = sh[threadIdx.x];
    long long c = carry;
    if (idx < nb) blocksum[idx] = c + incl - v;
    __syncthreads();
    if (threadIdx.x == SCAN_T - 1) carry = c + incl;
    __syncthreads();
  }
  if (threadIdx.x == 0) blocksum[nb] = carry;  // grand total
}

__global__ void k_scan_add(int32_t* __restrict__ out, int64_t n, const long long* __restrict__ blocksum,
                           int64_t nb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (int32_t)(out[i] + blocksum[i / SCAN_BLK]);
  if (i == n) out[n] = (int32_t)blocksum[nb];
}

size_t scan_scratch_ints(int64_t n) {
  int64_t nb = (n + SCAN_BLK - 1) / SCAN_BLK;
  return (size_t)(2 * (nb + 2));  // int64 entries counted in int32 units
}

int32_t exclusive_scan_i32(hipStream_t st, const int32_t* in, int32_t* out, int64_t n, int32_t* scratch) {
  long long* bs = reinterpret_cast<long long*>(scratch);
  int64_t nb = (n + SCAN_BLK - 1) / SCAN_BLK;
  if (nb > 0) {
    k_scan_local<<<dim3((unsigned)nb), dim3(SCAN_T), 0, st>>>(in, out, n, bs);
    HGNN_LAUNCH_CHECK("k_scan_local");
  }
  k_scan_blocksums<<<dim3(1), dim3(SCAN_T), 0, st>>>(bs, nb);
  HGNN_LAUNCH_CHECK("k_scan_blocksums");
  int64_t tot = n + 1;
  k_scan_add<<<dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st>>>(out, n, bs, nb);
  HGNN_LAUNCH_CHECK("k_scan_add");
  return HGNN_OK;
}

// Degrees -> row_ptr (blockIdx.y = 0) and source counts -> colT_ptr (1) in one launch without any hand-over between
// workgroups: each adds up everything in front of its own 4,096 values before it scans them. That is n^2 / 8192 reads
// from the L2 (3 MB at n = 80,000), which up to SCAN_PAIR_MAX cost less than the two further launches of the block-sum
// form (7,105 atoms: 2 x 8.9 us by one walking workgroup -> 5 us; 80,000: 6 launches of 4.5 us -> 7 us). The last
// workgroup of the degrees, which has the total, also leaves the result of the counting call for the host.
constexpr int64_t SCAN_PAIR_MAX = 131072;
constexpr int SP_BLK = 4096;
__global__ void __launch_bounds__(1024)
k_scan_pair(const int32_t* __restrict__ in0, int32_t* __restrict__ out0, const int32_t* __restrict__ in1,
            int32_t* __restrict__ out1, int n, const int32_t* __restrict__ status, HostMail* mail) {
  __shared__ long long sh_front[16];
  __shared__ int sh_own[16];
  const int32_t* in = blockIdx.y ? in1 : in0;
  int32_t* out = blockIdx.y ? out1 : out0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int base = blockIdx.x * SP_BLK;
  long long front = 0;
  for (int i = tid * 4; i < base; i += SP_BLK) {     // base is a multiple of SP_BLK: whole 16-byte groups
    const int4 v = *reinterpret_cast<const int4*>(in + i);
    front += ((long long)v.x + v.y) + ((long long)v.z + v.w);
  }
  const int i0 = base + tid * 4;
  int v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = i0 + k < n ? in[i0 + k] : 0;
  const int own = (v[0] + v[1]) + (v[2] + v[3]);
  int incl = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
    front += __shfl_xor(front, o);
  }
  if (lane == 63) {
    sh_own[wave] = incl;
    sh_front[wave] = front;
  }
  __syncthreads();
  long long before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    before += sh_front[w] + (w < wave ? sh_own[w] : 0);
    all += sh_front[w] + sh_own[w];
  }
  int ex = (int)before + incl - own;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (i0 + k < n) out[i0 + k] = ex;
    ex += v[k];
  }
  if (blockIdx.x == gridDim.x - 1 && tid == 0) {
    out[n] = (int)all;
    if (blockIdx.y == 0) post_mail(mail, all, status[0]);
  }
}
// larger batches: the total behind the block sums of the last scan, posted by a launch of its own
__global__ void k_post_total(const long long* __restrict__ total, const int32_t* __restrict__ status, HostMail* mail) {
  post_mail(mail, *total, status[0]);
}

// ---------------------------------------------------------------------------------------------
// per-graph metadata
// ---------------------------------------------------------------------------------------------
constexpr int SR_HOME = 16;   // most destination atoms of a work item of the search
struct GMeta {
  float cell[9];   // rows a, b, c (zeros when not periodic)
  float inv[9];    // fractional = (pos - org) * inv   (row vector times matrix)
  float org[3];
  int nb[3];       // bins per lattice direction
  int R[3];        // search reach in bins
  int bin_off;     // first global bin of this graph (see first_bin())
  int periodic;
  int lo, hi;      // atom range
  int home;        // destination atoms of a work item of the search
};

enum : int {
  ST_BAD_OFFSETS = 1,
  ST_BAD_CELL = 2,
  ST_OUT_OF_CELL = 4,
};
// periodic atoms must lie inside their cell: fractional coordinates within this distance of [0, 1]
constexpr float FRAC_TOL = 1e-5f;

constexpr float BIN_MARGIN = 1.001f;  // bins are at least 1.001 * rc wide: absorbs float32 binning error
constexpr int NB_MAX = 256;

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__device__ inline float wave_min(float x) {
  for (int o = 32; o > 0; o >>= 1) x = fminf(x, __shfl_xor(x, o));
  return x;
}
__device__ inline float wave_max(float x) {
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}

// Bins and image reach of one graph from its extent (not periodic: bounding box mn .. mx) or its cell. Called by a whole
// wavefront with the same arguments; lane k < 3 works out lattice direction k (the double-precision divisions and
// square roots of the three directions are the longest chain of the binning). Returns the number of bins.
__device__ inline int graph_meta(int lo, int hi, bool periodic, const float* __restrict__ cell_g, const float* mn,
                                 const float* mx, float rc, GMeta* __restrict__ m, int32_t* __restrict__ status) {
  const int lane = threadIdx.x & 63;
  const int k = lane < 3 ? lane : 0;
  const double rcm = (double)rc * (double)BIN_MARGIN;
  double hgt;
  if (lane == 0) {
    m->lo = lo;
    m->hi = hi;
  }
  if (lane < 9) m->cell[lane] = periodic ? cell_g[lane] : 0.f;
  if (periodic) {
    double C[9];
    for (int q = 0; q < 9; ++q) C[q] = (double)cell_g[q];
    // cross product of the other two lattice vectors
    const double u0 = C[(3 * k + 3) % 9], u1 = C[(3 * k + 4) % 9], u2 = C[(3 * k + 5) % 9];
    const double w0 = C[(3 * k + 6) % 9], w1 = C[(3 * k + 7) % 9], w2 = C[(3 * k + 8) % 9];
    const double c0 = u1 * w2 - u2 * w1, c1 = u2 * w0 - u0 * w2, c2 = u0 * w1 - u1 * w0;
    const double det = __shfl(C[0] * c0 + C[1] * c1 + C[2] * c2, 0);   // lane 0: first vector . (second x third)
    if (!(fabs(det) >= 1e-6)) {
      if (lane == 0) {
        atomicOr(status, ST_BAD_CELL);
        m->periodic = 0;
        for (int q = 0; q < 3; ++q) { m->nb[q] = 1; m->R[q] = 0; m->org[q] = 0.f; }
        for (int q = 0; q < 9; ++q) m->inv[q] = 0.f;
      }
      return 1;
    }
    // inverse: column k of C^-1 is this cross product / det  (f_k = (pos . cr[k]) / det)
    hgt = fabs(det) / sqrt(c0 * c0 + c1 * c1 + c2 * c2);
    if (lane < 3) {
      m->inv[k] = (float)(c0 / det);
      m->inv[3 + k] = (float)(c1 / det);
      m->inv[6 + k] = (float)(c2 / det);
      m->org[k] = 0.f;
    }
  } else {
    const float a = hi == lo ? 0.f : (k == 0 ? mn[0] : (k == 1 ? mn[1] : mn[2]));
    const float b = hi == lo ? 0.f : (k == 0 ? mx[0] : (k == 1 ? mx[1] : mx[2]));
    const double ext = (double)b - (double)a;
    const double pad = 1e-3 * (1.0 + ext);
    hgt = ext + 2.0 * pad;
    if (lane < 3) {
      m->inv[k] = k == 0 ? (float)(1.0 / hgt) : 0.f;
      m->inv[3 + k] = k == 1 ? (float)(1.0 / hgt) : 0.f;
      m->inv[6 + k] = k == 2 ? (float)(1.0 / hgt) : 0.f;
      m->org[k] = (float)((double)a - pad);
    }
  }
  const double q = floor(hgt / rcm);
  const int mine = q < 1.0 ? 1 : (q > (double)NB_MAX ? NB_MAX : (int)q);
  int nb[3] = {__shfl(mine, 0), __shfl(mine, 1), __shfl(mine, 2)};
  // keep the number of bins proportional to the number of atoms (bounded workspace)
  const long long nat = hi - lo;
  const long long cap = 4 * nat > 1 ? 4 * nat : 1;
  while ((long long)nb[0] * nb[1] * nb[2] > cap) {
    const int t = (nb[0] >= nb[1] && nb[0] >= nb[2]) ? 0 : (nb[1] >= nb[2] ? 1 : 2);
    nb[t] -= 1;
  }
  if (lane < 3) {
    const int n = k == 0 ? nb[0] : (k == 1 ? nb[1] : nb[2]);
    int R = (int)ceil(rcm / (hgt / n));
    if (R < 1) R = 1;
    if (!periodic && R > n - 1) R = n - 1;  // nothing outside the bounding box
    if (R > 127) {
      atomicOr(status, ST_BAD_CELL);
      R = 0;
    }
    m->nb[k] = n;
    m->R[k] = R;
    if (k == 0) m->periodic = periodic ? 1 : 0;
  }
  return nb[0] * nb[1] * nb[2];
}

__device__ inline bool bad_range(int g, int G, int N, int lo, int hi) {
  return lo > hi || lo < 0 || hi > N || (g == 0 && lo != 0) || (g == G - 1 && hi != N);
}
// Bins of graph g start at this place of the bin arrays: a graph has at most max(4 atoms, 1) bins, and one more entry
// ends its last bin, so no scan over the graphs is needed to place them.
__device__ inline int first_bin(int lo, int g) { return 4 * lo + 2 * g; }
__device__ inline void no_bins(GMeta* m, int lo, int g) {
  *m = GMeta{};
  m->nb[0] = m->nb[1] = m->nb[2] = 1;
  m->bin_off = first_bin(lo, g);
}

// one wavefront (block of 64) per graph
__global__ void k_graph_meta(int N, int G, const float* __restrict__ pos, const int32_t* __restrict__ graph_off,
                             const float* __restrict__ cell, const uint8_t* __restrict__ pbc, float rc,
                             GMeta* __restrict__ meta, int32_t* __restrict__ status) {
  const int g = blockIdx.x;
  const int lane = threadIdx.x;
  const int lo = graph_off[g], hi = graph_off[g + 1];
  if (bad_range(g, G, N, lo, hi)) {
    if (lane == 0) {
      atomicOr(status, ST_BAD_OFFSETS);
      no_bins(&meta[g], 0, g);
    }
    return;
  }
  const bool periodic = (pbc != nullptr) && (cell != nullptr) && (pbc[g] != 0);
  float mn[3] = {3.0e38f, 3.0e38f, 3.0e38f}, mx[3] = {-3.0e38f, -3.0e38f, -3.0e38f};
  if (!periodic) {
    for (int i = lo + lane; i < hi; i += 64) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        float x = pos[3 * (size_t)i + c];
        mn[c] = fminf(mn[c], x);
        mx[c] = fmaxf(mx[c], x);
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      mn[c] = wave_min(mn[c]);
      mx[c] = wave_max(mx[c]);
    }
  }
  graph_meta(lo, hi, periodic, cell + 9 * (size_t)g, mn, mx, rc, &meta[g], status);
  if (lane == 0) {
    meta[g].bin_off = first_bin(lo, g);
    meta[g].home = SR_HOME;
  }
}

__device__ inline int find_graph(const int32_t* __restrict__ graph_off, int G, int i) {
  // largest g with graph_off[g] <= i  (empty graphs share an offset; the last of them wins, and its
  // successor is the one that really holds atom i) -> search for the first g with graph_off[g+1] > i
  int lo = 0, hi = G - 1;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (graph_off[mid + 1] > i) hi = mid; else lo = mid + 1;
  }
  return lo;
}

// bin of an atom inside its graph; outside: a fractional coordinate outside the cell (also NaN)
__device__ inline int atom_bin_of(const GMeta& m, float x, float y, float z, bool& outside) {
  const float d[3] = {x - m.org[0], y - m.org[1], z - m.org[2]};
  int b[3];
  outside = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float f = d[0] * m.inv[k] + d[1] * m.inv[3 + k] + d[2] * m.inv[6 + k];
    outside = outside || !(f >= -FRAC_TOL && f <= 1.0f + FRAC_TOL);
    int q = (int)floorf(f * (float)m.nb[k]);
    b[k] = q < 0 ? 0 : (q >= m.nb[k] ? m.nb[k] - 1 : q);
  }
  return (b[0] * m.nb[1] + b[1]) * m.nb[2] + b[2];
}

// Small batches of small graphs (see bin_by_graph()): everything between the input and the search in one launch, one
// workgroup per graph. A graph's atoms are contiguous in the batch, so its bins' runs are too: histogram, scan and
// placement stay inside the workgroup, in LDS (seven launches of 2-14 us before: the atomics of a molecule's atoms on
// its one or two bins in memory alone were 13 + 13 us at 7,105 atoms). Larger batches keep the grid-wide kernels below,
// where one large graph is spread over many workgroups, and so do batches of large graphs: the host knows the mean only.
// Whole graph, grid-wide -> by graph: one cell of 4,000 atoms 129 -> 109 us, four of them 193 -> 184, one of 5,000 102 -> 104, of
// 7,000 118 -> 123, of 16,000 168 -> 201, two of 7,000 178 -> 185; 470 molecules 96 -> 82.
constexpr int BIN_GRAPHS_MAX = 16384, BIN_GRAPH_MEAN = 4500;
static bool bin_by_graph(int N, int G) {
  return N <= BIN_GRAPHS_MAX && G <= BIN_GRAPHS_MAX && N <= (int64_t)BIN_GRAPH_MEAN * G;
}
constexpr int BG_BINS = 4096;    // bins of a graph counted in LDS; more: in the workspace
// Destination atoms per work item in a batch of N atoms whose graphs are binned one by one. Staging the candidates is paid once per
// item, so large batches take 16; with fewer items than the chip holds workgroups (three per compute unit) the longest item is
// what the launch takes, and items of cells with many images are long: thousands of candidate records, streamed through the LDS
// again for every four destination atoms. Graphs of few candidates (HOME_FEW) keep 16, and so do large graphs (HOME_LARGE atoms),
// whose bins are a cutoff wide and whose items are many. Whole graph, 16 -> 8 -> 4 per item: 64 crystals (4,096 atoms) 219 -> 140 -> 122
// us, 543 mixed atoms 138 -> 94 -> 75, 5,530 mixed 147 -> 100 -> 84, 7,734 mixed 147 -> 101 -> 97, 9,680 mixed 128 -> 100 -> 113, 10,660 of
// crystals 150 -> 129 -> 132; the other way for 7,105 of molecules 69 -> 73 -> 80, 15,138 of molecules 92 -> 100 -> 115, three cells of 2,000
// 103 -> 122 -> 143, 38,889 mixed 256 -> 256 -> 308.
static int search_home(int N) { return N <= 6144 ? 4 : N <= 12288 ? 8 : SR_HOME; }
constexpr float HOME_FEW = 512.f;
constexpr int HOME_LARGE = 1024;
struct BinArgs {
  int N, G;
  const float* pos;
  const int32_t* graph_off;
  const float* cell;
  const uint8_t* pbc;
  float rc;
  GMeta* meta;
  int32_t *atom_graph, *bin_cnt, *bin_start;
  float4* spos;
  int32_t *status, *nlist;
  int2* list;
  int home;   // search_home()
  int4* zeroed;   // one graph: the counters to clear here (see BIN_CLEARS)
  int nzeroed4;
};
// A batch of one graph is binned by one workgroup, which can clear the counters and check the offsets before it begins: a launch less
// in a structure's graph (one molecule, energies and forces, 123 -> 119 us, one crystal of 60 atoms 187 -> 183, conservative forces of
// 187 atoms 469 -> 466), while the clearing is a few stores per thread.
constexpr int BIN_CLEARS = 4096;   // 16-byte groups
__global__ void __launch_bounds__(256) k_bin_graphs(BinArgs p) {
  __shared__ GMeta m;
  __shared__ int hist[BG_BINS];
  __shared__ float red[4][6];
  __shared__ int wsum[4][2];
  __shared__ int s_at;
  const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lo = p.graph_off[g], hi = p.graph_off[g + 1];
  // With a bad offset anywhere (found by the launch before) no graph is binned: graphs that overlap would share bins, and
  // count on top of one another's record places.
  bool bad;
  if (p.zeroed) {
    bad = bad_range(0, 1, p.N, lo, hi);
    for (int i = tid; i < p.nzeroed4; i += 256) p.zeroed[i] = make_int4(i == 0 && bad ? ST_BAD_OFFSETS : 0, 0, 0, 0);
    __threadfence();   // before anyone's atomics on them
    __syncthreads();
  } else {
    bad = (*p.status & ST_BAD_OFFSETS) != 0;
  }
  if (bad) return;   // uniform
  const bool periodic = (p.pbc != nullptr) && (p.cell != nullptr) && (p.pbc[g] != 0);
  float mn[3] = {3.0e38f, 3.0e38f, 3.0e38f}, mx[3] = {-3.0e38f, -3.0e38f, -3.0e38f};
  if (!periodic) {
    for (int i = lo + tid; i < hi; i += 256) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float x = p.pos[3 * (size_t)i + c];
        mn[c] = fminf(mn[c], x);
        mx[c] = fmaxf(mx[c], x);
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      mn[c] = wave_min(mn[c]);
      mx[c] = wave_max(mx[c]);
      if (lane == 0) { red[wave][c] = mn[c]; red[wave][3 + c] = mx[c]; }
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w)
      for (int c = 0; c < 3; ++c) { mn[c] = fminf(mn[c], red[w][c]); mx[c] = fmaxf(mx[c], red[w][3 + c]); }
  }
  const int off = first_bin(lo, g);
  if (wave == 0) {
    graph_meta(lo, hi, periodic, p.cell + 9 * (size_t)g, mn, mx, p.rc, &m, p.status);
    if (lane == 0) m.bin_off = off;
  }
  __syncthreads();   // (graph_meta() leaves a lattice direction to a lane each)
  const int nbins = m.nb[0] * m.nb[1] * m.nb[2];
  const float block = (float)(2 * m.R[0] + 1) * (float)(2 * m.R[1] + 1) * (float)(2 * m.R[2] + 1);   // bins around one
  const bool few = (float)(hi - lo) * block <= HOME_FEW * (float)nbins;
  const int home = few || hi - lo > HOME_LARGE ? SR_HOME : p.home;
  if (tid == 0) {
    p.meta[g] = m;
    p.meta[g].home = home;
  }
  const bool in_lds = nbins <= BG_BINS;
  int* cnt = p.bin_cnt + off;                        // cleared by the launch before
  if (in_lds)
    for (int b = tid; b < nbins; b += 256) hist[b] = 0;
  __syncthreads();
  for (int i = lo + tid; i < hi; i += 256) {
    bool outside;
    const int b = atom_bin_of(m, p.pos[3 * (size_t)i], p.pos[3 * (size_t)i + 1], p.pos[3 * (size_t)i + 2], outside);
    if (outside && periodic) atomicOr(p.status, ST_OUT_OF_CELL);
    p.atom_graph[i] = g;
    if (in_lds) atomicAdd(&hist[b], 1); else atomicAdd(&cnt[b], 1);
  }
  if (!in_lds) __threadfence();
  __syncthreads();
  // bins -> first record of every bin, and the work list (1,024 bins at a time)
  int carry = lo;
  for (int b0 = 0; b0 < nbins; b0 += 1024) {
    int c[4], own = 0, items = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int b = b0 + tid * 4 + u;
      c[u] = b < nbins ? (in_lds ? hist[b] : __hip_atomic_load(&cnt[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : 0;
      own += c[u];
      items += (c[u] + home - 1) / home;
    }
    int ia = own, ii = items;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int ua = __shfl_up(ia, o), ui = __shfl_up(ii, o);
      if (lane >= o) { ia += ua; ii += ui; }
    }
    if (lane == 63) { wsum[wave][0] = ia; wsum[wave][1] = ii; }
    __syncthreads();
    int ta = 0, ti = 0, ba = 0, bi = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (w < wave) { ba += wsum[w][0]; bi += wsum[w][1]; }
      ta += wsum[w][0];
      ti += wsum[w][1];
    }
    if (tid == 0) s_at = atomicAdd(p.nlist, ti);
    __syncthreads();
    int at = s_at + bi + ii - items, ex = carry + ba + ia - own;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int b = b0 + tid * 4 + u;
      if (b < nbins) {
        p.bin_start[off + b] = ex;
        if (in_lds) hist[b] = ex; else cnt[b] = ex;   // from here on: the bin's next free record
        for (int k = 0; k < c[u]; k += home, ++at) p.list[at] = make_int2(off + b, k);
      }
      ex += c[u];
    }
    carry += ta;
    __syncthreads();
  }
  if (tid == 0) p.bin_start[off + nbins] = hi;
  if (!in_lds) __threadfence();
  __syncthreads();
  for (int i = lo + tid; i < hi; i += 256) {
    const float x = p.pos[3 * (size_t)i], y = p.pos[3 * (size_t)i + 1], z = p.pos[3 * (size_t)i + 2];
    bool outside;
    const int b = atom_bin_of(m, x, y, z, outside);
    const int k = in_lds ? atomicAdd(&hist[b], 1) : atomicAdd(&cnt[b], 1);
    p.spos[k] = make_float4(x, y, z, __int_as_float(i));
  }
}

__global__ void k_bin_atoms_count(int N, int G, const float* __restrict__ pos, const int32_t* __restrict__ graph_off,
                                  const GMeta* __restrict__ meta, int32_t* __restrict__ atom_graph,
                                  int32_t* __restrict__ atom_bin, int32_t* __restrict__ bin_cnt,
                                  int32_t* __restrict__ status) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  int g = find_graph(graph_off, G, i);
  const GMeta& m = meta[g];
  bool outside;
  const int bin = m.bin_off + atom_bin_of(m, pos[3 * (size_t)i], pos[3 * (size_t)i + 1], pos[3 * (size_t)i + 2], outside);
  if (outside && m.periodic) atomicOr(status, ST_OUT_OF_CELL);
  atom_graph[i] = g;
  atom_bin[i] = bin;
  atomicAdd(&bin_cnt[bin], 1);
}

// atoms in bin order: (x, y, z, index) as one 16-byte record (the bin's count runs down to its next free record); and,
// in the workgroups behind those of the atoms, the work list of the search: one entry per SR_HOME destination atoms of
// a non-empty bin (order does not matter)
__global__ void k_bin_place(int N, unsigned natom_blocks, const float* __restrict__ pos, const int32_t* __restrict__ atom_bin,
                            const int32_t* __restrict__ bin_start, int32_t* __restrict__ bin_cnt,
                            float4* __restrict__ spos, int64_t maxbins,
                            int32_t* __restrict__ nlist, int2* __restrict__ list) {
  if (blockIdx.x >= natom_blocks) {
    const int64_t b = (int64_t)(blockIdx.x - natom_blocks) * blockDim.x + threadIdx.x;
    if (b >= maxbins) return;
    const int c = bin_start[b + 1] - bin_start[b];
    if (c <= 0) return;
    int at = atomicAdd(nlist, (c + SR_HOME - 1) / SR_HOME);
    for (int k = 0; k < c; k += SR_HOME) list[at++] = make_int2((int)b, k);
    return;
  }
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int bin = atom_bin[i];
  const int k = bin_start[bin] + atomicAdd(&bin_cnt[bin], -1) - 1;
  spos[k] = make_float4(pos[3 * (size_t)i], pos[3 * (size_t)i + 1], pos[3 * (size_t)i + 2], __int_as_float(i));
}

// ---------------------------------------------------------------------------------------------
// search: one workgroup per (bin, up to SR_HOME destination atoms), candidates staged in LDS
// ---------------------------------------------------------------------------------------------
__device__ inline int floordiv(int a, int b) { return (a >= 0) ? a / b : -((-a + b - 1) / b); }

constexpr int SR_CHUNK = 1024;   // candidates staged at once
constexpr int SR_EXT = 256;      // bins of the (2R+1)^3 block enumerated at once (one per thread)
constexpr int SR_CAP = 256;      // hits of one row that the LDS row holds; longer rows are walked and ranked from memory, see long_row()
constexpr int SR_ZERO_CODE = (128 << 16) | (128 << 8) | 128;
constexpr int SR_GRID = 2048;    // workgroups of the search (they walk the work list with this stride)

struct SearchLds {
  __align__(16) unsigned long long row[4][SR_CAP + 4];   // per wavefront: (atom << 24 | code) of the hits of one row
  float cx[SR_CHUNK], cy[SR_CHUNK], cz[SR_CHUNK];   // shifted candidate positions  pos_j + t
  int cj[SR_CHUNK], cc[SR_CHUNK];                   // candidate atom and shift code
  int ch[SR_CHUNK];                                 // hits of each staged candidate in this work item (then, in the
                                                    // filling pass: the candidate's first place in its source group)
  unsigned short rowk[4][SR_CAP];                   // per wavefront: candidate slot of each hit of the row at hand
  unsigned short rinfo[SR_HOME][SR_CAP];            // per destination atom and edge: slot | place among the item's hits << 10
  int rstart[SR_HOME], rcnt[SR_HOME];               // first edge and edge count of the item's rows (0: row not dealt here)
  int ext_start[SR_EXT];                            // first record of each enumerated bin
  int ext_pref[SR_EXT + 1];                         // exclusive prefix of their atom counts
  int ext_code[SR_EXT];
  float ext_t[3][SR_EXT];                           // shift vector t = (s0*a + s1*b) + s2*c
  int scan[4];
};

struct SearchArgs {
  int N;
  const float* pos;
  const GMeta* meta;
  const int32_t* atom_graph;
  const int32_t* bin_start;
  const float4* spos;
  const int32_t* nlist;
  const int2* list;
  const int32_t* status;
  float rc;
  // count
  int32_t* deg;
  int32_t* colT_cnt;
  // fill
  const int32_t* row_ptr;
  int32_t* dst;
  int32_t* col;
  int8_t* shift;
  float* d2;
  float* rvec;
  const int32_t* colT_ptr;   // fill: first place of each source's group
  int32_t* colT_cur;         // fill: places of each group handed out so far
  int32_t* unsorted;         // fill: the groups' edges in the order they were dealt
  int32_t *key_j, *key_c;    // fill: the hits of long rows, one int per edge each
};

// t = (s0*a + s1*b) + s2*c, every operation rounded on its own
__device__ __forceinline__ void shift_vector(const float* cell, int s0, int s1, int s2, float& tx, float& ty, float& tz) {
  const float f0 = (float)s0, f1 = (float)s1, f2 = (float)s2;
  tx = __fadd_rn(__fadd_rn(__fmul_rn(f0, cell[0]), __fmul_rn(f1, cell[3])), __fmul_rn(f2, cell[6]));
  ty = __fadd_rn(__fadd_rn(__fmul_rn(f0, cell[1]), __fmul_rn(f1, cell[4])), __fmul_rn(f2, cell[7]));
  tz = __fadd_rn(__fadd_rn(__fmul_rn(f0, cell[2]), __fmul_rn(f1, cell[5])), __fmul_rn(f2, cell[8]));
}

// Rows longer than the LDS row, by the wavefront that met them: it walks the bins from memory, stores the hits unordered (key_j,
// key_c: room for one int per edge each) and ranks them from memory. (Rows listed for a launch of their own before: 2-5 us and a
// launch in every call for rows that only cells with hundreds of neighbours have.)
__device__ inline void long_row(const SearchArgs& p, const GMeta& m, int i, int b0, int b1, int b2, float pix, float piy, float piz, float rc2) {
  const int lane = threadIdx.x & 63;
  const int nb0 = m.nb[0], nb1 = m.nb[1], nb2 = m.nb[2];
  const bool per = m.periodic != 0;
  int count = 0;
  const int start = p.row_ptr[i], end = p.row_ptr[i + 1];
  for (int B0 = b0 - m.R[0]; B0 <= b0 + m.R[0]; ++B0) {
    int s0 = 0, c0 = B0;
    if (per) { s0 = floordiv(B0, nb0); c0 = B0 - s0 * nb0; } else if (B0 < 0 || B0 >= nb0) continue;
    for (int B1 = b1 - m.R[1]; B1 <= b1 + m.R[1]; ++B1) {
      int s1 = 0, c1 = B1;
      if (per) { s1 = floordiv(B1, nb1); c1 = B1 - s1 * nb1; } else if (B1 < 0 || B1 >= nb1) continue;
      for (int B2 = b2 - m.R[2]; B2 <= b2 + m.R[2]; ++B2) {
        int s2 = 0, c2 = B2;
        if (per) { s2 = floordiv(B2, nb2); c2 = B2 - s2 * nb2; } else if (B2 < 0 || B2 >= nb2) continue;
        const int bin = m.bin_off + (c0 * nb1 + c1) * nb2 + c2;
        float tx, ty, tz;
        shift_vector(m.cell, s0, s1, s2, tx, ty, tz);
        const bool zero_shift = (s0 | s1 | s2) == 0;
        const int code = ((s0 + 128) << 16) | ((s1 + 128) << 8) | (s2 + 128);
        const int kb = p.bin_start[bin], ke = p.bin_start[bin + 1];
        for (int k0 = kb; k0 < ke; k0 += 64) {
          const int k = k0 + lane;
          bool hit = false;
          int j = 0;
          if (k < ke) {
            const float4 a = p.spos[k];
            j = __float_as_int(a.w);
            const float rx = __fsub_rn(pix, __fadd_rn(a.x, tx)), ry = __fsub_rn(piy, __fadd_rn(a.y, ty)), rz = __fsub_rn(piz, __fadd_rn(a.z, tz));
            const float dd = __fadd_rn(__fadd_rn(__fmul_rn(rx, rx), __fmul_rn(ry, ry)), __fmul_rn(rz, rz));
            hit = (dd < rc2) && !(zero_shift && j == i);
          }
          const unsigned long long mask = __ballot(hit);
          const int at = start + count + __popcll(mask & ((1ull << lane) - 1ull));
          if (hit && at < end) {
            p.key_j[at] = j;
            p.key_c[at] = code;
          }
          count += __popcll(mask);
        }
      }
    }
  }
  // the row's hits are in memory: every lane of this wavefront reads them all below
  __threadfence();
  __builtin_amdgcn_wave_barrier();
  for (int t = start + lane; t < end; t += 64) {
    const int mj = p.key_j[t], mc = p.key_c[t];
    int rank = 0;
    for (int u = start; u < end; ++u) {
      const int uj = p.key_j[u], uc = p.key_c[u];
      rank += (uj < mj) || (uj == mj && uc < mc);
    }
    const int e = start + rank;
    const int s0 = ((mc >> 16) & 255) - 128, s1 = ((mc >> 8) & 255) - 128, s2 = (mc & 255) - 128;
    float tx, ty, tz;
    shift_vector(m.cell, s0, s1, s2, tx, ty, tz);
    const float qx = __fadd_rn(p.pos[3 * (size_t)mj], tx);
    const float qy = __fadd_rn(p.pos[3 * (size_t)mj + 1], ty);
    const float qz = __fadd_rn(p.pos[3 * (size_t)mj + 2], tz);
    const float rx = __fsub_rn(pix, qx), ry = __fsub_rn(piy, qy), rz = __fsub_rn(piz, qz);
    const float dd = __fadd_rn(__fadd_rn(__fmul_rn(rx, rx), __fmul_rn(ry, ry)), __fmul_rn(rz, rz));
    p.unsorted[p.colT_ptr[mj] + atomicAdd(&p.colT_cur[mj], 1)] = e;   // the edge's place in its source group
    p.dst[e] = i;
    p.col[e] = mj;
    p.shift[3 * (size_t)e] = (int8_t)s0;
    p.shift[3 * (size_t)e + 1] = (int8_t)s1;
    p.shift[3 * (size_t)e + 2] = (int8_t)s2;
    p.d2[e] = dd;
    p.rvec[3 * (size_t)e] = rx;
    p.rvec[3 * (size_t)e + 1] = ry;
    p.rvec[3 * (size_t)e + 2] = rz;
  }
}

template <bool FILL>
__global__ void __launch_bounds__(256) k_search(SearchArgs p) {
  __shared__ SearchLds L;
  if (p.status[0] != 0) return;          // bad input: the host reports it, nothing is searched
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nlist = *p.nlist;
  const float rc2 = __fmul_rn(p.rc, p.rc);
  unsigned long long* row = L.row[wave];
  for (int item = blockIdx.x; item < nlist; item += gridDim.x) {
    const int2 it = p.list[item];
    const int hb = it.x, h0 = it.y;
    const int hb_start = p.bin_start[hb];
    const int hb_cnt = p.bin_start[hb + 1] - hb_start;
    const int i_first = __float_as_int(p.spos[hb_start].w);
    const GMeta& m = p.meta[p.atom_graph[i_first]];
    const int nhome = hb_cnt - h0 < m.home ? hb_cnt - h0 : m.home;
    const int nb0 = m.nb[0], nb1 = m.nb[1], nb2 = m.nb[2];
    const int R0 = m.R[0], R1 = m.R[1], R2 = m.R[2];
    const int lb = hb - m.bin_off;
    const int b2 = lb % nb2, b1 = (lb / nb2) % nb1, b0 = lb / (nb1 * nb2);
    const int n1 = 2 * R1 + 1, n2 = 2 * R2 + 1;
    const int next = (2 * R0 + 1) * n1 * n2;
    const bool per = m.periodic != 0;
    float cell[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) cell[k] = m.cell[k];

    // bins eg .. eg+SR_EXT-1 of the block around the home bin: record range, shift, prefix of the atom counts.
    // Returns the number of candidates they hold. All threads call it (it synchronises).
    auto enumerate = [&](int eg) -> int {
      const int q = eg + tid;
      int count = 0, start = 0, code = SR_ZERO_CODE;
      float tx = 0.f, ty = 0.f, tz = 0.f;
      if (q < next) {
        const int d0 = q / (n1 * n2), d1 = (q / n2) % n1, d2 = q % n2;
        const int B0 = b0 + d0 - R0, B1 = b1 + d1 - R1, B2 = b2 + d2 - R2;
        int s0 = 0, s1 = 0, s2 = 0, c0 = B0, c1 = B1, c2 = B2;
        bool ok = true;
        if (per) {
          s0 = floordiv(B0, nb0); c0 = B0 - s0 * nb0;
          s1 = floordiv(B1, nb1); c1 = B1 - s1 * nb1;
          s2 = floordiv(B2, nb2); c2 = B2 - s2 * nb2;
        } else {
          ok = B0 >= 0 && B0 < nb0 && B1 >= 0 && B1 < nb1 && B2 >= 0 && B2 < nb2;
        }
        if (ok) {
          const int bin = m.bin_off + (c0 * nb1 + c1) * nb2 + c2;
          start = p.bin_start[bin];
          count = p.bin_start[bin + 1] - start;
          code = ((s0 + 128) << 16) | ((s1 + 128) << 8) | (s2 + 128);
          shift_vector(cell, s0, s1, s2, tx, ty, tz);
        }
      }
      // exclusive scan over the 256 threads: inside each wavefront by lane shifts, then the four wavefront totals
      int incl = count;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
      }
      if (lane == 63) L.scan[wave] = incl;
      __syncthreads();
      const int w0 = L.scan[0], w1 = L.scan[1], w2 = L.scan[2], w3 = L.scan[3];
      const int total = w0 + w1 + w2 + w3;
      const int ex = incl - count + (wave > 0 ? w0 : 0) + (wave > 1 ? w1 : 0) + (wave > 2 ? w2 : 0);
      L.ext_start[tid] = start;
      L.ext_pref[tid] = ex;
      L.ext_code[tid] = code;
      L.ext_t[0][tid] = tx; L.ext_t[1][tid] = ty; L.ext_t[2][tid] = tz;
      if (tid == 0) L.ext_pref[SR_EXT] = total;
      __syncthreads();
      return total;
    };
    // candidates c0 .. c0+n-1 of the enumerated bins -> LDS (all threads; the caller synchronises)
    auto stage = [&](int c0, int n) {
      if (next <= 32 && c0 == 0 && n == L.ext_pref[SR_EXT]) {
        // few bins and all their atoms at once: eight threads per bin copy its run, no search for the owner
        const int eb = tid >> 3;
        const int lo = L.ext_pref[eb], cnt = L.ext_pref[eb + 1] - lo, src = L.ext_start[eb];
        const float tx = L.ext_t[0][eb], ty = L.ext_t[1][eb], tz = L.ext_t[2][eb];
        const int code = L.ext_code[eb];
        for (int a = tid & 7; a < cnt; a += 8) {
          const float4 r = p.spos[src + a];
          L.cx[lo + a] = __fadd_rn(r.x, tx);
          L.cy[lo + a] = __fadd_rn(r.y, ty);
          L.cz[lo + a] = __fadd_rn(r.z, tz);
          L.cj[lo + a] = __float_as_int(r.w);
          L.cc[lo + a] = code;
        }
        return;
      }
      for (int k = tid; k < n; k += 256) {
        const int q = c0 + k;
        int lo = 0, hi = SR_EXT;               // last bin with ext_pref <= q (bins without atoms share a prefix)
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (L.ext_pref[mid] <= q) lo = mid; else hi = mid;
        }
        const float4 a = p.spos[L.ext_start[lo] + (q - L.ext_pref[lo])];
        L.cx[k] = __fadd_rn(a.x, L.ext_t[0][lo]);
        L.cy[k] = __fadd_rn(a.y, L.ext_t[1][lo]);
        L.cz[k] = __fadd_rn(a.z, L.ext_t[2][lo]);
        L.cj[k] = __float_as_int(a.w);
        L.cc[k] = L.ext_code[lo];
      }
    };
    // this wavefront's destination atom against the n staged candidates; cnt = hits so far
    // lds_hist (counting pass): a hit adds to the candidate's LDS counter (flushed by the caller) instead of to the
    // source histogram in memory
    auto scan = [&](int i, float pix, float piy, float piz, int n, int& cnt, bool lds_hist) {
      for (int k0 = 0; k0 < n; k0 += 256) {
        // four groups of 64 candidates: their LDS reads are in flight together
        int jj[4], cd[4];
        float qx[4], qy[4], qz[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = k0 + 64 * u + lane;
          const int kk = k < n ? k : 0;
          jj[u] = L.cj[kk]; cd[u] = L.cc[kk];
          qx[u] = L.cx[kk]; qy[u] = L.cy[kk]; qz[u] = L.cz[kk];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (k0 + 64 * u >= n) break;                       // uniform
          const int k = k0 + 64 * u + lane;
          const float rx = __fsub_rn(pix, qx[u]), ry = __fsub_rn(piy, qy[u]), rz = __fsub_rn(piz, qz[u]);
          const float dd = __fadd_rn(__fadd_rn(__fmul_rn(rx, rx), __fmul_rn(ry, ry)), __fmul_rn(rz, rz));
          const bool hit = k < n && (dd < rc2) && !(cd[u] == SR_ZERO_CODE && jj[u] == i);
          const unsigned long long mask = __ballot(hit);
          if (hit) {
            if (FILL) {
              const int at = cnt + __popcll(mask & ((1ull << lane) - 1ull));
              if (at < SR_CAP) {
                row[at] = ((unsigned long long)(unsigned)jj[u] << 24) | (unsigned)cd[u];
                L.rowk[wave][at] = (unsigned short)k;
              }
            } else if (lds_hist) {
              atomicAdd(&L.ch[k], 1);
            } else {
              atomicAdd(&p.colT_cnt[jj[u]], 1);
            }
          }
          cnt += __popcll(mask);
        }
      }
    };
    // the row is complete: count, or order it and write the edges
    // h >= 0: the row's edges are dealt to their sources at the end of the work item (slot and place kept in LDS);
    // h < 0 (candidates streamed in chunks): every edge takes its place with an addition of its own
    auto finish = [&](int i, float pix, float piy, float piz, int cnt, int h) {
      if (!FILL) {
        if (lane == 0) p.deg[i] = cnt;
        return;
      }
      if (cnt > SR_CAP) {
        if (h >= 0 && lane == 0) L.rcnt[h] = 0;
        long_row(p, m, i, b0, b1, b2, pix, piy, piz, rc2);
        return;
      }
      if (lane < 3) row[cnt + lane] = ~0ull;   // pad to a multiple of four for the 16-byte reads below
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      const int start = p.row_ptr[i];
      if (h >= 0 && lane == 0) {
        L.rstart[h] = start;
        L.rcnt[h] = cnt;
      }
      for (int t = lane; t < cnt; t += 64) {
        const unsigned long long key = row[t];
        int rank = 0;
        for (int u = 0; u < cnt; u += 4) {
          const ulonglong2 ka = *reinterpret_cast<const ulonglong2*>(&row[u]);
          const ulonglong2 kb = *reinterpret_cast<const ulonglong2*>(&row[u + 2]);
          rank += (ka.x < key) + (ka.y < key) + (kb.x < key) + (kb.y < key);
        }
        const int e = start + rank;
        const int mj = (int)(key >> 24), mc = (int)(key & 0xffffffu);
        const int s0 = ((mc >> 16) & 255) - 128, s1 = ((mc >> 8) & 255) - 128, s2 = (mc & 255) - 128;
        float tx, ty, tz;
        shift_vector(cell, s0, s1, s2, tx, ty, tz);
        const float qx = __fadd_rn(p.pos[3 * (size_t)mj], tx);
        const float qy = __fadd_rn(p.pos[3 * (size_t)mj + 1], ty);
        const float qz = __fadd_rn(p.pos[3 * (size_t)mj + 2], tz);
        const float rx = __fsub_rn(pix, qx), ry = __fsub_rn(piy, qy), rz = __fsub_rn(piz, qz);
        const float dd = __fadd_rn(__fadd_rn(__fmul_rn(rx, rx), __fmul_rn(ry, ry)), __fmul_rn(rz, rz));
        if (h >= 0) {
          const int k = L.rowk[wave][t];
          const int place = atomicAdd(&L.ch[k], 1);   // < SR_HOME: a destination atom hits a slot once
          L.rinfo[h][rank] = (unsigned short)(k | (place << 10));
        } else {
          p.unsorted[p.colT_ptr[mj] + atomicAdd(&p.colT_cur[mj], 1)] = e;
        }
        p.dst[e] = i;
        p.col[e] = mj;
        p.shift[3 * (size_t)e] = (int8_t)s0;
        p.shift[3 * (size_t)e + 1] = (int8_t)s1;
        p.shift[3 * (size_t)e + 2] = (int8_t)s2;
        p.d2[e] = dd;
        p.rvec[3 * (size_t)e] = rx;
        p.rvec[3 * (size_t)e + 1] = ry;
        p.rvec[3 * (size_t)e + 2] = rz;
      }
      __builtin_amdgcn_wave_barrier();   // the row buffer is reused by the next destination atom
    };

    const int nrounds = (nhome + 3) >> 2;          // four destination atoms (one per wavefront) per round
    const int total0 = enumerate(0);
    if (next <= SR_EXT && total0 <= SR_CHUNK) {
      // the usual case: every candidate fits in LDS at once; staged once, then the wavefronts run on their own
      stage(0, total0);
      for (int k = tid; k < total0; k += 256) L.ch[k] = 0;
      __syncthreads();
      for (int r = 0; r < nrounds; ++r) {
        const int h = 4 * r + wave;
        if (h >= nhome) break;
        const float4 a = p.spos[hb_start + h0 + h];
        const int i = __float_as_int(a.w);
        int cnt = 0;
        scan(i, a.x, a.y, a.z, total0, cnt, true);
        finish(i, a.x, a.y, a.z, cnt, h);
      }
      if (!FILL) {
        // the source histogram: one addition per candidate that was hit (a candidate is hit by up to 16 destination
        // atoms of the work item), not one per hit
        __syncthreads();
        for (int k = tid; k < total0; k += 256) {
          const int c = L.ch[k];
          if (c) atomicAdd(&p.colT_cnt[L.cj[k]], c);
        }
      } else {
        // transpose plan: every candidate that was hit takes its places in its source group with one addition, then
        // the item's edges go to their places (any order inside a group: the groups are put in edge order afterwards)
        __syncthreads();
        for (int k = tid; k < total0; k += 256) {
          const int c = L.ch[k];
          if (c) L.ch[k] = atomicAdd(&p.colT_cur[L.cj[k]], c);
        }
        __syncthreads();
        for (int h = wave; h < nhome; h += 4) {
          const int cnt = L.rcnt[h], start = L.rstart[h];
          for (int t = lane; t < cnt; t += 64) {
            const int info = L.rinfo[h][t];
            const int k = info & 1023;
            p.unsorted[p.colT_ptr[L.cj[k]] + L.ch[k] + (info >> 10)] = start + t;
          }
        }
      }
    } else {
      // many periodic images or a crowded bin: the candidates are streamed through LDS in chunks, once per round
      for (int r = 0; r < nrounds; ++r) {
        const int h = 4 * r + wave;
        const bool on = h < nhome;
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        if (on) a = p.spos[hb_start + h0 + h];
        const int i = __float_as_int(a.w);
        int cnt = 0;
        for (int eg = 0; eg < next; eg += SR_EXT) {
          const int total = (eg == 0 && r == 0) ? total0 : enumerate(eg);
          for (int c0 = 0; c0 < total; c0 += SR_CHUNK) {
            const int n = total - c0 < SR_CHUNK ? total - c0 : SR_CHUNK;
            __syncthreads();               // the previous chunk has been read by every wavefront
            stage(c0, n);
            __syncthreads();
            if (on) scan(i, a.x, a.y, a.z, n, cnt, false);
          }
          __syncthreads();                 // before the bin table is overwritten
        }
        if (on) finish(i, a.x, a.y, a.z, cnt, -1);
      }
    }
    __syncthreads();                       // before the next work item reuses the tables
  }
}

// ---------------------------------------------------------------------------------------------
// transpose plan: the histogram of sources is taken by the counting search; the filling search deals the edges to
// their source's group (any order, see k_search); here each group is put into ascending edge order, in place
// ---------------------------------------------------------------------------------------------
constexpr int TS_CAP = 512;   // group members ranked out of LDS; longer groups are ranked from memory
// (also writes the two offset arrays that leave with the edges: see write_offsets())
__device__ __forceinline__ void write_offsets(int64_t i, int N, int G, const int32_t* graph_off, const int32_t* row_ptr,
                                              const int32_t* colT_ptr, int32_t* egp, int32_t* colT_out) {
  if (i <= N) colT_out[i] = colT_ptr[i];            // the source groups' offsets
  if (i <= G) egp[i] = row_ptr[graph_off[i]];       // first edge of every graph
}
__global__ void __launch_bounds__(256)
k_offsets(int N, int G, const int32_t* __restrict__ graph_off, const int32_t* __restrict__ row_ptr,
          const int32_t* __restrict__ colT_ptr, int32_t* __restrict__ egp, int32_t* __restrict__ colT_out) {
  write_offsets((int64_t)blockIdx.x * 256 + threadIdx.x, N, G, graph_off, row_ptr, colT_ptr, egp, colT_out);
}
__global__ void __launch_bounds__(256)
k_rank_sources(unsigned nrank, int N, int G, const int32_t* __restrict__ graph_off, const int32_t* __restrict__ row_ptr,
               const int32_t* __restrict__ colT_ptr, int32_t* __restrict__ egp, int32_t* __restrict__ colT_out,
               int32_t* __restrict__ permT, int32_t* __restrict__ copy, int32_t* __restrict__ colT_cur) {
  if (blockIdx.x >= nrank) {   // the workgroups behind those of the source groups
    write_offsets((int64_t)(blockIdx.x - nrank) * 256 + threadIdx.x, N, G, graph_off, row_ptr, colT_ptr, egp, colT_out);
    return;
  }
  // permT holds the groups as they were dealt; copy: room for one int per edge (long groups are ranked out of it)
  const int32_t* unsorted = permT;
  __shared__ __align__(16) int grp[4][TS_CAP + 4];
  const int j = (int)(((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (j >= N) return;
  if (lane == 0) colT_cur[j] = 0;   // the filling call leaves its counters at zero: it may be repeated after one count
  const int start = colT_ptr[j], end = colT_ptr[j + 1];
  const int n = end - start;
  if (n <= 0) return;
  if (n <= TS_CAP) {
    int* g = grp[(threadIdx.x >> 6) & 3];
    for (int t = lane; t < n; t += 64) g[t] = unsorted[start + t];
    if (lane < 4) g[n + lane] = 0x7fffffff;      // pad to a multiple of four for the 16-byte reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    for (int t = lane; t < n; t += 64) {
      const int me = g[t];
      int rank = 0;
      for (int u = 0; u < n; u += 4) {
        const int4 q = *reinterpret_cast<const int4*>(&g[u]);
        rank += (q.x < me) + (q.y < me) + (q.z < me) + (q.w < me);
      }
      permT[start + rank] = me;
    }
    return;
  }
  for (int t = start + lane; t < end; t += 64) copy[t] = unsorted[t];
  __threadfence();
  __builtin_amdgcn_wave_barrier();
  for (int t = start + lane; t < end; t += 64) {
    const int me = copy[t];
    int rank = 0;
    for (int u = start; u < end; ++u) rank += copy[u] < me;
    permT[start + rank] = me;
  }
}

// ---------------------------------------------------------------------------------------------
// workspace layout
// ---------------------------------------------------------------------------------------------
struct NeighWs {
  GMeta* meta;          // [G]
  int32_t* atom_graph;  // [N]
  int32_t* atom_bin;    // [N]
  int32_t* zeroed;      // status | deg | colT_cnt | colT_cur | bin_cnt, cleared by one launch
  int64_t nzeroed;
  int32_t* status;      // 0 input errors, 1 work-list length
  int32_t* deg;         // [N]
  int32_t* colT_cnt;    // [N]
  int32_t* colT_cur;    // [N]
  int32_t* bin_cnt;     // [maxbins]
  int32_t* bin_start;   // [maxbins+1]
  float4* spos;         // [N] (x, y, z, atom) in bin order
  int2* list;           // [N] work list of the search
  int32_t* colT_ptr;    // [N+1] kept from the counting call for the filling call
  int32_t* scan;        // scratch
  size_t bytes;
  int64_t maxbins;
};

static NeighWs carve_neigh(void* ws, int N, int G) {
  NeighWs w;
  Carver c(ws);
  w.maxbins = 4ll * N + 2ll * G + 2;      // first_bin() of the last graph + its bins + 1
  w.meta = c.take<GMeta>((size_t)G + 1);
  w.atom_graph = c.take<int32_t>((size_t)N + 1);
  w.atom_bin = c.take<int32_t>((size_t)N + 1);
  const int64_t n4 = (int64_t)(align_up((size_t)N + 1, 64));   // sub-arrays start at multiples of 256 bytes
  w.nzeroed = 64 + 3 * n4 + (int64_t)align_up((size_t)w.maxbins, 64);
  w.zeroed = c.take<int32_t>((size_t)w.nzeroed);
  w.status = w.zeroed;
  w.deg = w.zeroed + 64;
  w.colT_cnt = w.deg + n4;
  w.colT_cur = w.colT_cnt + n4;
  w.bin_cnt = w.colT_cur + n4;
  w.bin_start = c.take<int32_t>((size_t)w.maxbins + 1);
  w.spos = c.take<float4>((size_t)N + 1);
  w.list = c.take<int2>((size_t)N + 1);
  w.colT_ptr = c.take<int32_t>((size_t)N + 2);
  w.scan = c.take<int32_t>(scan_scratch_ints(w.maxbins + 8) + 8);
  w.bytes = c.used();
  return w;
}
// Clears the counters; the first workgroup checks every graph's offsets meanwhile, and starts status[0] (the first of the
// cleared words) with what it finds. n > 0.
__global__ void __launch_bounds__(256)
k_clear_and_check(int4* p, int64_t n, int N, int G, const int32_t* __restrict__ graph_off) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int bad = 0;
  if (blockIdx.x == 0) {
#pragma unroll 4
    for (int g = threadIdx.x; g < G; g += 256) bad |= bad_range(g, G, N, graph_off[g], graph_off[g + 1]) ? 1 : 0;
    bad = __syncthreads_or(bad);
  }
  if (i < n) p[i] = make_int4(i == 0 && bad ? ST_BAD_OFFSETS : 0, 0, 0, 0);
}

static inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

static SearchArgs search_args(const NeighWs& w, int N, const float* pos, float rc) {
  SearchArgs a = {};
  a.N = N; a.pos = pos; a.meta = w.meta; a.atom_graph = w.atom_graph; a.bin_start = w.bin_start; a.spos = w.spos;
  a.nlist = w.status + 1; a.list = w.list; a.status = w.status; a.rc = rc;
  return a;
}

}  // namespace hgnn

using namespace hgnn;

extern "C" const char* hgnn_last_error_string(void) { return g_err; }
extern "C" int32_t hgnn_version(void) { return 2; }

extern "C" int32_t hgnn_radius_graph_workspace_bytes(int32_t N, int32_t G, size_t* bytes_host) {
  HGNN_REQUIRE(bytes_host != nullptr, HGNN_ERR_NULLPTR, "bytes_host is null");
  HGNN_REQUIRE(N >= 0 && G >= 0, HGNN_ERR_BAD_SHAPE, "negative N or G");
  *bytes_host = carve_neigh(nullptr, N, G).bytes;
  return HGNN_OK;
}

extern "C" int32_t hgnn_radius_graph_count(void* stream, int32_t N, int32_t G, const float* pos,
                                           const int32_t* graph_off, const float* cell, const uint8_t* pbc,
                                           float rc, void* ws, size_t ws_bytes, int32_t* row_ptr,
                                           int64_t* E_host) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  HGNN_REQUIRE(N >= 0 && G >= 0, HGNN_ERR_BAD_SHAPE, "negative N or G");
  HGNN_REQUIRE(E_host && row_ptr && graph_off && ws, HGNN_ERR_NULLPTR, "radius_graph_count: null pointer");
  HGNN_REQUIRE(pos || N == 0, HGNN_ERR_NULLPTR, "pos is null");
  HGNN_REQUIRE(rc > 0.f && rc < 1e18f, HGNN_ERR_BAD_SHAPE, "cutoff must be positive");
  HGNN_REQUIRE(G > 0 || N == 0, HGNN_ERR_BAD_OFFSETS, "atoms without a graph");
  NeighWs w = carve_neigh(ws, N, G);
  HGNN_REQUIRE(ws_bytes >= w.bytes, HGNN_ERR_WORKSPACE_TOO_SMALL, "radius graph workspace: need %zu bytes, got %zu",
               w.bytes, ws_bytes);
  *E_host = 0;
  if (N == 0 || G == 0) {
    k_fill_i32<<<1, 64, 0, st>>>(row_ptr, 1, 0);
    k_fill_i32<<<1, 64, 0, st>>>(w.colT_ptr, 1, 0);
    HGNN_LAUNCH_CHECK("k_fill_i32");
    HGNN_HIP(hipStreamSynchronize(st));
    return HGNN_OK;
  }
  MailSlot mail;
  HGNN_TRY(mail.take(st));
  // Everything below is enqueued in one go: a bad offset or cell is recorded in status[0], leaves every later
  // kernel with in-range (if meaningless) indices or without work, keeps the search from running, and is reported after
  // the one wait at the end.
  {
    ProfScope ps(PT_NEIGH_SETUP, st);
    const bool by_graph = bin_by_graph(N, G), clears = by_graph && G == 1 && w.nzeroed / 4 <= BIN_CLEARS;
    int4* zeroed = reinterpret_cast<int4*>(w.zeroed);
    if (!clears) {
      k_clear_and_check<<<nblk(w.nzeroed / 4, 256), 256, 0, st>>>(zeroed, w.nzeroed / 4, N, G, graph_off);
      HGNN_LAUNCH_CHECK("k_clear_and_check");
    }
    if (by_graph) {
      const BinArgs a = {N, G, pos, graph_off, cell, pbc, rc, w.meta, w.atom_graph, w.bin_cnt, w.bin_start, w.spos, w.status, w.status + 1, w.list, search_home(N),
                         clears ? zeroed : nullptr, (int)(w.nzeroed / 4)};
      k_bin_graphs<<<G, 256, 0, st>>>(a);
      HGNN_LAUNCH_CHECK("k_bin_graphs");
    } else {
      k_graph_meta<<<G, 64, 0, st>>>(N, G, pos, graph_off, cell, pbc, rc, w.meta, w.status);
      HGNN_LAUNCH_CHECK("k_graph_meta");
      k_bin_atoms_count<<<nblk(N, 256), 256, 0, st>>>(N, G, pos, graph_off, w.meta, w.atom_graph, w.atom_bin, w.bin_cnt,
                                                      w.status);
      HGNN_LAUNCH_CHECK("k_bin_atoms_count");
      HGNN_TRY(exclusive_scan_i32(st, w.bin_cnt, w.bin_start, w.maxbins, w.scan));
      const unsigned na = nblk(N, 256);
      k_bin_place<<<na + nblk(w.maxbins, 256), 256, 0, st>>>(N, na, pos, w.atom_bin, w.bin_start, w.bin_cnt,
                                                             w.spos, w.maxbins, w.status + 1, w.list);
      HGNN_LAUNCH_CHECK("k_bin_place");
    }
  }
  {
    ProfScope ps(PT_NEIGH_COUNT, st);
    SearchArgs a = search_args(w, N, pos, rc);
    a.deg = w.deg; a.colT_cnt = w.colT_cnt;
    k_search<false><<<SR_GRID < N ? SR_GRID : N, 256, 0, st>>>(a);
    HGNN_LAUNCH_CHECK("k_search<count>");
  }
  {
    ProfScope ps(PT_NEIGH_SETUP, st);
    if (N <= SCAN_PAIR_MAX) {
      k_scan_pair<<<dim3(nblk(N, SP_BLK), 2), 1024, 0, st>>>(w.deg, row_ptr, w.colT_cnt, w.colT_ptr, N, w.status, mail.dev());
      HGNN_LAUNCH_CHECK("k_scan_pair");
    } else {
      HGNN_TRY(exclusive_scan_i32(st, w.colT_cnt, w.colT_ptr, N, w.scan));
      HGNN_TRY(exclusive_scan_i32(st, w.deg, row_ptr, N, w.scan));
      const int64_t nbs = ((int64_t)N + SCAN_BLK - 1) / SCAN_BLK;   // the grand total sits behind the block sums
      k_post_total<<<1, 1, 0, st>>>(reinterpret_cast<long long*>(w.scan) + nbs, w.status, mail.dev());
      HGNN_LAUNCH_CHECK("k_post_total");
    }
  }
  HGNN_HIP(mail.wait());
  const long long total = mail.value();
  const int status_h = mail.status();
  HGNN_REQUIRE(!(status_h & ST_BAD_OFFSETS), HGNN_ERR_BAD_OFFSETS,
               "graph_off must start at 0, be non-decreasing and end at N");
  HGNN_REQUIRE(!(status_h & ST_BAD_CELL), HGNN_ERR_BAD_CELL,
               "a periodic graph has a singular cell or needs more than 127 images per direction");
  HGNN_REQUIRE(!(status_h & ST_OUT_OF_CELL), HGNN_ERR_BAD_CELL,
               "an atom of a periodic graph lies outside its cell (fractional coordinates must be in [0, 1])");
  HGNN_REQUIRE(total < (1ll << 31), HGNN_ERR_OVERFLOW, "edge count %lld does not fit int32", total);
  *E_host = total;
  return HGNN_OK;
}

extern "C" int32_t hgnn_radius_graph_fill(void* stream, int32_t N, int32_t G, const float* pos,
                                          const int32_t* graph_off, const float* cell, const uint8_t* pbc, float rc,
                                          void* ws, size_t ws_bytes, void* tmp, size_t tmp_bytes,
                                          const int32_t* row_ptr, int64_t E, int32_t* dst, int32_t* col,
                                          int8_t* shift, float* d2, float* rvec, int32_t* edge_graph_ptr,
                                          int32_t* colT_ptr, int32_t* permT) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  (void)cell; (void)pbc;
  HGNN_REQUIRE(N >= 0 && G >= 0 && E >= 0, HGNN_ERR_BAD_SHAPE, "negative size");
  HGNN_REQUIRE(E < (1ll << 31), HGNN_ERR_OVERFLOW, "edge count does not fit int32");
  HGNN_REQUIRE(ws && row_ptr && graph_off && edge_graph_ptr && colT_ptr, HGNN_ERR_NULLPTR, "radius_graph_fill: null pointer");
  HGNN_REQUIRE(E == 0 || (tmp && dst && col && shift && d2 && rvec && permT && pos), HGNN_ERR_NULLPTR,
               "radius_graph_fill: null edge array");
  HGNN_REQUIRE(rc > 0.f, HGNN_ERR_BAD_SHAPE, "cutoff must be positive");
  NeighWs w = carve_neigh(ws, N, G);
  HGNN_REQUIRE(ws_bytes >= w.bytes, HGNN_ERR_WORKSPACE_TOO_SMALL, "radius graph workspace too small");
  HGNN_REQUIRE(tmp_bytes >= (size_t)E * 8, HGNN_ERR_WORKSPACE_TOO_SMALL, "radius graph tmp: need %zu bytes", (size_t)E * 8);
  if (N == 0) {
    k_fill_i32<<<nblk(G + 1, 256), 256, 0, st>>>(edge_graph_ptr, G + 1, 0);
    k_fill_i32<<<1, 64, 0, st>>>(colT_ptr, 1, 0);
    HGNN_LAUNCH_CHECK("k_fill_i32");
    return HGNN_OK;
  }
  int32_t* key_j = static_cast<int32_t*>(tmp);
  int32_t* key_c = key_j + E;
  if (E > 0) {
    {
      ProfScope ps(PT_NEIGH_FILL, st);
      SearchArgs a = search_args(w, N, pos, rc);
      a.row_ptr = row_ptr; a.dst = dst; a.col = col; a.shift = shift; a.d2 = d2; a.rvec = rvec;
      a.colT_ptr = w.colT_ptr; a.colT_cur = w.colT_cur; a.unsorted = permT;   // the groups are ordered in place below
      a.key_j = key_j; a.key_c = key_c;
      k_search<true><<<SR_GRID < N ? SR_GRID : N, 256, 0, st>>>(a);
      HGNN_LAUNCH_CHECK("k_search<fill>");
    }
  }
  const unsigned noff = nblk((int64_t)(N > G ? N : G) + 1, 256);
  if (E > 0) {
    ProfScope pst(PT_NEIGH_TRANSPOSE, st);
    // (the keys of the long rows are dead by now; the counters of the filling pass go back to zero)
    const unsigned nrank = nblk((int64_t)N * 64, 256);
    k_rank_sources<<<nrank + noff, 256, 0, st>>>(nrank, N, G, graph_off, row_ptr, w.colT_ptr, edge_graph_ptr, colT_ptr, permT,
                                                 key_j, w.colT_cur);
    HGNN_LAUNCH_CHECK("k_rank_sources");
  } else {
    ProfScope ps(PT_NEIGH_EMIT, st);
    k_offsets<<<noff, 256, 0, st>>>(N, G, graph_off, row_ptr, w.colT_ptr, edge_graph_ptr, colT_ptr);
    HGNN_LAUNCH_CHECK("k_offsets");
  }
  return HGNN_OK;
}
