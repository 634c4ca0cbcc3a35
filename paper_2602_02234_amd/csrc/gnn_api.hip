// C ABI of the GNN-variant model (declared in include/dp.h): model file, device
// weights, per-step buffers and the launch order of one energy/force/virial step.
// The neighbour search, force gather and float64 reductions are the library's shared
// kernels; the message-passing layers are in gnn.hip.
#include <cmath>
#include <cstring>
#include <fstream>
#include <map>
#include <string>
#include <vector>

#include "../../include/dp.h"
#include "gnn.h"
#include "node_fit.h"

using namespace dp;

struct dp_gnn {
  int device = 0;
  int prec = 0;
  double rc = 0, rcs = 0, rca = 0;
  int sel = 0, asel = 0, ntypes = 0;
  void *wbuf = nullptr;
  NodeFit fit{};
  gnn::Weights w{};
  Workspace ws;
  gnn::Buffers b;
  double *fpark = nullptr;  // forces when only the virial is asked for
  int64_t fpark_cap = 0;
  int64_t *tot_host = nullptr;  // pinned: angles, edges, angle-list edges
  int64_t angles_for = 0;       // atoms up to which steps use the angle buffers as they are
  int64_t last_angles = 0, last_edges = 0, last_aedges = 0;
  // per-phase device time (dp_gnn_profile_enable): lists, forward layers, backward
  // layers, forces and reductions
  bool prof = false;
  hipEvent_t ev[5] = {};
  double prof_ms[4] = {};
  int64_t prof_calls[4] = {};
  double lists_ms = 0.0;
};

namespace {

#define G_TRY(expr)                                                                        \
  do {                                                                                     \
    hipError_t e_ = (expr);                                                                \
    if (e_ != hipSuccess) {                                                                \
      set_error(std::string(#expr) + ": " + hipGetErrorString(e_));                        \
      return e_ == hipErrorOutOfMemory ? DP_ERR_OOM : DP_ERR_HIP;                          \
    }                                                                                      \
  } while (0)

using gnn::ADIM;
using gnn::EDIM;
using gnn::FWID;
using gnn::NDIM;
using gnn::NLAYER;

// (name, element count) of every array of the file, in file order.
std::vector<std::pair<std::string, size_t>> gnn_arrays(int ntypes) {
  std::vector<std::pair<std::string, size_t>> v = {
      {"TN", (size_t)ntypes * NDIM}, {"We0", EDIM}, {"be0", EDIM}, {"Wa0", ADIM}, {"ba0", ADIM}};
  for (int l = 0; l < NLAYER; ++l) {
    const std::string s = std::to_string(l);
    v.push_back({"Waa" + s, (size_t)(ADIM + 64) * ADIM});
    v.push_back({"baa" + s, ADIM});
    v.push_back({"Wea" + s, (size_t)(ADIM + 32) * EDIM});
    v.push_back({"bea" + s, EDIM});
    v.push_back({"Wee" + s, (size_t)(2 * NDIM + EDIM) * EDIM});
    v.push_back({"bee" + s, EDIM});
    v.push_back({"Wnn" + s, (size_t)(NDIM + EDIM) * NDIM});
    v.push_back({"bnn" + s, NDIM});
  }
  v.push_back({"G1", (size_t)NDIM * FWID});
  v.push_back({"d1", FWID});
  v.push_back({"G2", (size_t)FWID * FWID});
  v.push_back({"d2", FWID});
  v.push_back({"G3", FWID});
  v.push_back({"d3", 1});
  return v;
}

int load_weights(dp_gnn *m, const char *path) {
  std::ifstream f(path, std::ios::binary);
  if (!f) {
    set_error(std::string("cannot open GNN model file ") + path);
    return DP_ERR_MODEL_FILE;
  }
  const std::vector<char> raw = read_all(f);
  if (raw.size() < 128 || std::memcmp(raw.data(), "DPGNNv01", 8) != 0) {
    set_error("GNN model file: bad magic or short header");
    return DP_ERR_MODEL_FILE;
  }
  int32_t iv[16];
  double dv[4];
  std::memcpy(iv, raw.data() + 8, 64);
  std::memcpy(dv, raw.data() + 72, 32);
  if (iv[0] != 1 || iv[1] != NTYPES || iv[2] != NDIM || iv[3] != EDIM || iv[4] != ADIM || iv[5] != NLAYER ||
      iv[6] != FWID || iv[7] != SEL || iv[8] < 2 || iv[8] > gnn::ASEL) {
    set_error("GNN model file: version or dimensions differ from the compiled kernels");
    return DP_ERR_MODEL_FILE;
  }
  m->ntypes = iv[1];
  m->sel = iv[7];
  m->asel = iv[8];
  m->rc = dv[0];
  m->rcs = dv[1];
  m->rca = dv[2];
  if (!(m->rc > m->rcs && m->rcs > 0 && m->rca > m->rcs && m->rca <= m->rc)) {
    set_error("GNN model file: need 0 < rcs < rca <= rc");
    return DP_ERR_MODEL_FILE;
  }
  // device image: every array as float32 (256-byte aligned), plus G3 in float64
  std::vector<unsigned char> img;
  img.reserve(2 * raw.size());  // the arrays and their fragment-ordered copies in float32
  std::vector<size_t> offs;
  size_t off = 128;
  double d3 = 0.0;
  std::map<std::string, std::vector<double>> src;
  for (auto &a : gnn_arrays(m->ntypes)) {
    if (off + 8 * a.second > raw.size()) {
      set_error("GNN model file: truncated at " + a.first);
      return DP_ERR_MODEL_FILE;
    }
    std::vector<double> v(a.second);
    std::memcpy(v.data(), raw.data() + off, 8 * a.second);
    off += 8 * a.second;
    for (double x : v)
      if (!std::isfinite(x)) {
        set_error("GNN model file: non-finite value in " + a.first);
        return DP_ERR_MODEL_FILE;
      }
    if (a.first == "d3") d3 = v[0];
    const size_t o = (img.size() + 255) & ~size_t(255);
    img.resize(o + 4 * v.size());
    for (size_t k = 0; k < v.size(); ++k) {
      const float x = (float)v[k];
      std::memcpy(img.data() + o + 4 * k, &x, 4);
    }
    offs.push_back(o);
    src[a.first] = std::move(v);
  }
  if (off != raw.size()) {
    set_error("GNN model file: size does not match its header");
    return DP_ERR_MODEL_FILE;
  }
  const size_t og = (img.size() + 255) & ~size_t(255);
  img.resize(og + 8 * FWID);
  std::memcpy(img.data() + og, src["G3"].data(), 8 * FWID);
  // transposed copies and MFMA fragments (their order: gnn.hip, X and W)
  auto put = [&](const void *p, size_t bytes) {
    const size_t o = (img.size() + 255) & ~size_t(255);
    img.resize(o + bytes);
    std::memcpy(img.data() + o, p, bytes);
    offs.push_back(o);
  };
  auto transposed = [&](const std::vector<double> &v, int rows, int cols) {  // of the first `rows` rows
    std::vector<float> t((size_t)rows * cols);
    for (int r = 0; r < rows; ++r)
      for (int c = 0; c < cols; ++c) t[(size_t)c * rows + r] = (float)v[(size_t)r * cols + c];
    put(t.data(), 4 * t.size());
  };
  auto frag32 = [&](int outs, int K, auto W) {
    const std::vector<float> v = node_fragments(outs, K, W);
    put(v.data(), 4 * v.size());
  };
  auto frag16 = [&](int outs, int K, auto W) {
    std::vector<uint16_t> v((size_t)outs * K);
    for (int t = 0; t < outs / 16; ++t)
      for (int k = 0; k < K / 32; ++k)
        for (int ln = 0; ln < 64; ++ln)
          for (int s = 0; s < 8; ++s) {  // round to nearest even (the weights are finite)
            const float x = (float)W(16 * t + ln % 16, 32 * k + 16 * (s / 4) + 4 * (ln / 16) + s % 4);
            uint32_t u;
            std::memcpy(&u, &x, 4);
            v[((size_t)(t * (K / 32) + k) * 64 + ln) * 8 + s] = (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
          }
    put(v.data(), 2 * v.size());
  };
  auto frag = [&](int outs, int K, auto W) {
    if (m->prec == DP_BF16) frag16(outs, K, W);
    else frag32(outs, K, W);
  };
  transposed(src["G1"], NDIM, FWID);
  transposed(src["G2"], FWID, FWID);
  const std::vector<double> &g1 = src["G1"], &g2 = src["G2"];
  frag32(FWID, NDIM, [&](int o, int k) { return g1[k * FWID + o]; });
  frag32(FWID, FWID, [&](int o, int k) { return g2[k * FWID + o]; });
  frag32(FWID, FWID, [&](int o, int k) { return g2[o * FWID + k]; });
  frag32(NDIM, FWID, [&](int o, int k) { return g1[o * FWID + k]; });
  for (int l = 0; l < NLAYER; ++l) {
    const std::string s = std::to_string(l);
    const std::vector<double> &aa = src["Waa" + s], &ea = src["Wea" + s], &ee = src["Wee" + s];
    transposed(src["Wnn" + s], 2 * NDIM, NDIM);
    transposed(ee, NDIM, EDIM);
    frag(ADIM, ADIM, [&](int o, int k) { return aa[k * ADIM + o]; });
    frag(EDIM, ADIM, [&](int o, int k) { return ea[k * EDIM + o]; });
    frag(ADIM, EDIM, [&](int o, int k) { return ea[o * EDIM + k]; });
    frag(ADIM, ADIM, [&](int o, int k) { return aa[o * ADIM + k]; });
    frag(EDIM, 2 * EDIM, [&](int o, int k) { return ee[(NDIM + k) * EDIM + o]; });
    frag(EDIM, EDIM, [&](int o, int k) { return ee[(NDIM + o) * EDIM + k]; });
    frag(EDIM, EDIM, [&](int o, int k) { return ee[(2 * NDIM + o) * EDIM + k]; });
    frag32(128, ADIM, [&](int o, int k) {
      return o < 32 ? aa[(ADIM + k) * ADIM + o] : (o < 64 ? aa[(2 * ADIM + k) * ADIM + o - 32] : ea[(ADIM + k) * EDIM + o - 64]);
    });
    frag32(ADIM, 128, [&](int o, int k) {
      return k < 32 ? aa[(ADIM + o) * ADIM + k] : (k < 64 ? aa[(2 * ADIM + o) * ADIM + k - 32] : ea[(ADIM + o) * EDIM + k - 64]);
    });
  }
  G_TRY(hipMalloc(&m->wbuf, img.size()));
  G_TRY(hipMemcpy(m->wbuf, img.data(), img.size(), hipMemcpyHostToDevice));
  const unsigned char *base = (const unsigned char *)m->wbuf;
  size_t k = 0;
  auto nxt = [&]() { return (const float *)(base + offs[k++]); };
  gnn::Weights &w = m->w;
  w.TN = nxt(); w.We0 = nxt(); w.be0 = nxt(); w.Wa0 = nxt(); w.ba0 = nxt();
  for (int l = 0; l < NLAYER; ++l) {
    (void)nxt();  // Waa, and Wea below
    w.baa[l] = nxt();
    (void)nxt();
    w.bea[l] = nxt();
    w.Wee[l] = nxt(); w.bee[l] = nxt(); w.Wnn[l] = nxt(); w.bnn[l] = nxt();
  }
  w.G1 = nxt(); w.d1 = nxt(); w.G2 = nxt(); w.d2 = nxt(); w.G3 = nxt();
  (void)nxt();  // d3 goes by value
  w.G3d = (const double *)(base + og);
  w.G1T = nxt(); w.G2T = nxt();
  NodeFit &nf = m->fit;
  nf.d1 = w.d1; nf.d2 = w.d2; nf.G3 = w.G3; nf.G3d = w.G3d;
  nf.G1 = nxt(); nf.G2 = nxt(); nf.G2T = nxt(); nf.G1T = nxt();
  for (int l = 0; l < NLAYER; ++l) {
    auto fr = [&](gnn::Frag &f) {
      const void *p = base + offs[k++];
      if (m->prec == DP_BF16) f.b16 = (const bf16_t *)p;
      else f.f32 = (const float *)p;
    };
    w.WnnT[l] = nxt(); w.WeeT[l] = nxt();
    fr(w.A[l]); fr(w.Mg[l]); fr(w.Xt[l]); fr(w.Yt[l]); fr(w.E[l]); fr(w.N[l]); fr(w.D[l]);
    w.PQ[l] = nxt(); w.PS[l] = nxt();
  }
  w.d3 = m->fit.d3 = d3;
  return DP_OK;
}

void free_buffers(gnn::Buffers &b) {
  void *ps[] = {b.aoff, b.nf, b.ef, b.af, b.da, b.de, b.dnj, b.dnl, b.gs, b.slot};
  for (void *p : ps)
    if (p) (void)hipFree(p);
  b = gnn::Buffers{};
}

int ensure_atoms(gnn::Buffers &b, int64_t n) {
  if (n <= b.cap) return DP_OK;
  const int64_t cap = std::max<int64_t>(n, b.cap + b.cap / 4);
  void *ps[] = {b.aoff, b.nf, b.ef, b.de, b.dnj, b.dnl, b.gs, b.slot};
  for (void *p : ps)
    if (p) (void)hipFree(p);
  b.aoff = nullptr; b.nf = b.ef = b.de = b.dnj = b.dnl = b.gs = nullptr;
  b.slot = nullptr;
  b.cap = 0;
  const size_t c = (size_t)cap, e = c * SEL * EDIM;
  G_TRY(hipMalloc(&b.aoff, (c + 1) * sizeof(int64_t)));
  G_TRY(hipMalloc(&b.nf, 2 * c * NDIM * sizeof(float)));
  G_TRY(hipMalloc(&b.ef, 3 * e * sizeof(float)));
  G_TRY(hipMalloc(&b.de, e * sizeof(float)));
  G_TRY(hipMalloc(&b.dnj, 2 * e * sizeof(float)));
  G_TRY(hipMalloc(&b.dnl, c * NDIM * sizeof(float)));
  G_TRY(hipMalloc(&b.gs, c * SEL * 2 * sizeof(float)));
  G_TRY(hipMalloc(&b.slot, c * SEL * sizeof(int)));
  b.cap = cap;
  return DP_OK;
}

int ensure_angles(gnn::Buffers &b, int64_t na) {
  if (na <= b.acap) return DP_OK;
  const int64_t cap = std::max<int64_t>(na, b.acap + b.acap / 4);
  if (b.af) (void)hipFree(b.af);
  if (b.da) (void)hipFree(b.da);
  b.af = b.da = nullptr;
  b.acap = 0;
  G_TRY(hipMalloc(&b.af, 2 * (size_t)cap * ADIM * sizeof(float)));
  G_TRY(hipMalloc(&b.da, (size_t)cap * ADIM * sizeof(float)));
  b.acap = cap;
  return DP_OK;
}

int gnn_status(const Workspace &ws) {
  const int s = step_status(ws);
  if (s == DP_WARN_SEL_OVERFLOW) {
    set_error("an atom has more than sel neighbours within rc; the message-passing model needs complete lists");
    return DP_ERR_TOO_LARGE;
  }
  return s;
}

// One step.  The angle buffers are sized by the number of angles, which the device counts:
// the host waits for it where the buffers are new for this many atoms (or phases are
// timed); otherwise the whole step is enqueued with the buffers there are, and if they turn
// out too small (FLAG_ANGLES, DP_RETRY) the caller enlarges them and repeats it.  The wait cost 45 us of
// a 192-atom step of 560.
int gnn_step(dp_gnn *m, int64_t natoms, const double *X, const int32_t *types, const double *box, double *energy,
             double *forces, double *virial, double *atom_energy, hipStream_t st) {
  Workspace &ws = m->ws;
  const int n = (int)natoms;
  Grid g;
  int s = make_grid(m->rc, m->rc, box, g);
  if (s != DP_OK) return s;
  s = ensure_ws(ws, m->prec, n, 1, false, true);
  if (s != DP_OK) return s;
  s = ensure_atoms(m->b, n);
  if (s != DP_OK) return s;
  const bool open = box == nullptr;
  const int ncells = open ? MAX_CELLS : g.ncells;
  const OneSystem one{g, open ? 0 : 1, {0, n, 0, n}};
  if (m->prof) G_TRY(hipEventRecord(m->ev[0], st));
  launch_prologue(ws, 1, n, ncells + 1, true, st, &one);
  launch_cells(ws, X, types, n, m->ntypes, open, ncells, m->rc, st);
  launch_nlist(ws, X, n, 0, n, n, m->rc, false, st);
  gnn::Geo geo{(float)m->rc, (float)m->rcs, (float)m->rca, 1.f / (float)m->sel, 1.f / (float)m->asel, m->asel};
  const bool wait = m->prof || n > m->angles_for;
  gnn::Buffers b = m->b;
  if (wait) b.acap = INT64_MAX;  // made to fit below
  gnn::launch_angle_offsets(b, ws, X, n, geo, m->tot_host, st);
  G_TRY(hipGetLastError());
  if (m->prof) G_TRY(hipEventRecord(m->ev[1], st));
  if (wait) {
    G_TRY(hipMemcpyAsync(ws.flags_host, ws.flags, 4 * sizeof(unsigned), hipMemcpyDeviceToHost, st));
    G_TRY(hipStreamSynchronize(st));
    if (m->prof) {
      float ms = 0.f;
      m->lists_ms = hipEventElapsedTime(&ms, m->ev[0], m->ev[1]) == hipSuccess ? ms : 0.0;
    }
    s = gnn_status(ws);
    if (s != DP_OK) return s;
    s = ensure_angles(m->b, std::max<int64_t>(m->tot_host[0], 1));
    if (s != DP_OK) return s;
    m->angles_for = std::max<int64_t>(m->angles_for, n);
  }
  const bool bwd = forces || virial;
  if (m->prof) G_TRY(hipEventRecord(m->ev[2], st));
  for (int l = 0; l < NLAYER; ++l) {
    if (m->prec == DP_BF16)
      gnn::launch_layer_fwd<bf16_t>(m->w, m->b, ws, X, types, n, l, geo, ws.Ei, st);
    else
      gnn::launch_layer_fwd<float>(m->w, m->b, ws, X, types, n, l, geo, ws.Ei, st);
  }
  if (gnn::separate_fit(n)) launch_node_fit(m->fit, m->b.dnl, n, ws.Ei, ws.flags, st);
  if (m->prof) G_TRY(hipEventRecord(m->ev[3], st));
  if (bwd) {
    launch_rev_slots(ws, n, m->b.slot, st);
    for (int l = NLAYER - 1; l >= 0; --l) {
      if (m->prec == DP_BF16)
        gnn::launch_layer_bwd<bf16_t>(m->w, m->b, ws, X, types, n, l, geo, st);
      else
        gnn::launch_layer_bwd<float>(m->w, m->b, ws, X, types, n, l, geo, st);
    }
  }
  if (m->prof) G_TRY(hipEventRecord(m->ev[4], st));
  if (bwd) {
    double *F = forces;
    if (!F) {
      if (m->fpark_cap < n) {
        if (m->fpark) (void)hipFree(m->fpark);
        m->fpark = nullptr;
        m->fpark_cap = 0;
        G_TRY(hipMalloc(&m->fpark, (size_t)n * 3 * sizeof(double)));
        m->fpark_cap = n;
      }
      F = m->fpark;
    }
    launch_forces(ws, X, n, nullptr, F, false, false, st);
  }
  launch_reduce(ws, ws.sys_off, 1, energy, atom_energy, virial, 1, st);
  G_TRY(hipGetLastError());
  if (m->prof) G_TRY(hipEventRecord(m->ev[0], st));  // end of the last phase (ev[0] is free again)
  G_TRY(hipStreamSynchronize(st));
  s = gnn_status(ws);
  if (s == DP_OK && (ws.flags_host[0] & FLAG_ANGLES)) {
    s = ensure_angles(m->b, m->tot_host[0]);
    return s == DP_OK ? DP_RETRY : s;
  }
  if (s >= 0) {
    m->last_angles = m->tot_host[0];
    m->last_edges = m->tot_host[1];
    m->last_aedges = m->tot_host[2];
  }
  if (s >= 0 && m->prof) {
    // phases: lists ev1 - (start), fwd ev3 - ev2, bwd ev4 - ev3, forces/reductions end - ev4
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, m->ev[2], m->ev[3]) == hipSuccess) { m->prof_ms[1] += ms; m->prof_calls[1] += 1; }
    if (bwd && hipEventElapsedTime(&ms, m->ev[3], m->ev[4]) == hipSuccess) {
      m->prof_ms[2] += ms;
      m->prof_calls[2] += 1;
    }
    if (hipEventElapsedTime(&ms, m->ev[4], m->ev[0]) == hipSuccess) { m->prof_ms[3] += ms; m->prof_calls[3] += 1; }
    m->prof_ms[0] += m->lists_ms;
    m->prof_calls[0] += 1;
  }
  return s;
}

}  // namespace

extern "C" {

int dp_gnn_load(const char *path, int precision, int device, dp_gnn **out) {
  set_error("");
  if (!path || !out || (precision != DP_FP32 && precision != DP_BF16)) {
    set_error("dp_gnn_load: bad argument");
    return DP_ERR_ARG;
  }
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) {
    set_error("dp_gnn_load: no such device");
    return DP_ERR_ARG;
  }
  G_TRY(hipSetDevice(device));
  dp_gnn *m = new dp_gnn();
  m->device = device;
  m->prec = precision;
  int s = load_weights(m, path);
  if (s == DP_OK && hipHostMalloc(&m->tot_host, 3 * sizeof(int64_t), hipHostMallocDefault) != hipSuccess) {
    set_error("dp_gnn_load: pinned allocation failed");
    s = DP_ERR_OOM;
  }
  if (s != DP_OK) {
    dp_gnn_free(m);
    return s;
  }
  *out = m;
  return DP_OK;
}

void dp_gnn_free(dp_gnn *m) {
  if (!m) return;
  (void)hipSetDevice(m->device);
  (void)hipDeviceSynchronize();
  free_buffers(m->b);
  free_ws(m->ws);
  if (m->fpark) (void)hipFree(m->fpark);
  if (m->wbuf) (void)hipFree(m->wbuf);
  if (m->tot_host) (void)hipHostFree(m->tot_host);
  for (auto &e : m->ev)
    if (e) (void)hipEventDestroy(e);
  delete m;
}

int dp_gnn_info(const dp_gnn *m, double *rc, double *rca, int *sel, int *asel) {
  if (!m) {
    set_error("dp_gnn_info: bad argument");
    return DP_ERR_ARG;
  }
  if (rc) *rc = m->rc;
  if (rca) *rca = m->rca;
  if (sel) *sel = m->sel;
  if (asel) *asel = m->asel;
  return DP_OK;
}

int dp_gnn_compute_device(dp_gnn *m, int64_t natoms, const double *d_coords, const int32_t *d_types,
                          const double *box_host, double *d_energy, double *d_forces, double *d_virial,
                          double *d_atom_energy, void *hip_stream) {
  set_error("");
  if (!m || natoms < 1 || !d_coords || !d_types || !d_energy) {
    set_error("dp_gnn_compute_device: bad argument");
    return DP_ERR_ARG;
  }
  if (natoms > (1 << 24)) {
    set_error("natoms above the library limit");
    return DP_ERR_TOO_LARGE;
  }
  G_TRY(hipSetDevice(m->device));
  int s = gnn_step(m, natoms, d_coords, d_types, box_host, d_energy, d_forces, d_virial, d_atom_energy,
                  (hipStream_t)hip_stream);
  if (s == DP_RETRY)
    s = gnn_step(m, natoms, d_coords, d_types, box_host, d_energy, d_forces, d_virial, d_atom_energy,
                  (hipStream_t)hip_stream);
  return s;
}

int dp_gnn_graph_size(const dp_gnn *m, int64_t *edges, int64_t *angle_edges, int64_t *angles) {
  if (!m) {
    set_error("dp_gnn_graph_size: bad argument");
    return DP_ERR_ARG;
  }
  if (edges) *edges = m->last_edges;
  if (angle_edges) *angle_edges = m->last_aedges;
  if (angles) *angles = m->last_angles;
  return DP_OK;
}

int dp_gnn_profile_enable(dp_gnn *m, int enable) {
  if (!m) {
    set_error("dp_gnn_profile_enable: bad argument");
    return DP_ERR_ARG;
  }
  G_TRY(hipSetDevice(m->device));
  if (enable && !m->ev[0])
    for (auto &e : m->ev) G_TRY(hipEventCreate(&e));
  m->prof = enable != 0;
  for (int k = 0; k < 4; ++k) {
    m->prof_ms[k] = 0.0;
    m->prof_calls[k] = 0;
  }
  return DP_OK;
}

int dp_gnn_profile_read(const dp_gnn *m, double *ms, int64_t *calls, int max) {
  if (!m || !ms || !calls || max < 0) {
    set_error("dp_gnn_profile_read: bad argument");
    return DP_ERR_ARG;
  }
  const int k = max < 4 ? max : 4;
  for (int q = 0; q < k; ++q) {
    ms[q] = m->prof_ms[q];
    calls[q] = m->prof_calls[q];
  }
  return k;
}

}  // extern "C"
