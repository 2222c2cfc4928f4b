// C ABI of the warm-start network (warmstart.h): parameters, Adam state,
// workspace and the launch sequence of the forward and backward passes.
#include "warmstart.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "nn_kernels.hpp"

namespace {

thread_local std::string g_create_error;

constexpr int kMostLayers = 14;   // embedding, residual layers, head

struct LayerSpec {
  int cout, cin, K, stride, dil, pad;
  int64_t w_off, b_off;
  int64_t weights() const { return int64_t(cout) * cin * K; }
};

const char* check_config(const ws_config& c) {
  if (c.window < 4 || c.window > 4096) return "window must be in [4, 4096]";
  if (c.patch < 1 || c.window % c.patch != 0) return "patch must divide window";
  if ((c.window / c.patch) % 4 != 0) return "window / patch must be a multiple of 4";
  if (c.width < 1 || c.width > 4096) return "width must be in [1, 4096]";
  static_assert(kMostLayers == 12 + 2, "the largest number of layers");
  if (c.hidden < 0 || c.hidden > 12) return "hidden must be in [0, 12]";
  if (c.nx < 1 || c.nx > 64) return "nx must be in [1, 64]";
  if (c.ny < 1 || c.ny > 32) return "ny must be in [1, 32]";
  if (c.max_batch < 1 || int64_t(c.max_batch) * c.window > (int64_t(1) << 30))
    return "max_batch must be >= 1 with max_batch * window <= 2^30";
  return nullptr;
}

std::vector<LayerSpec> layer_specs(const ws_config& c) {
  std::vector<LayerSpec> L;
  L.push_back({c.width, 2 * c.ny, c.patch, c.patch, 1, 0, 0, 0});
  for (int l = 1; l <= c.hidden; ++l) {
    const int d = 1 << (l - 1);
    L.push_back({c.width, c.width, 3, 1, d, d, 0, 0});
  }
  L.push_back({c.patch * c.nx, c.width, 1, 1, 0, 0, 0, 0});
  int64_t off = 0;
  for (auto& s : L) {
    s.w_off = off;
    s.b_off = off + s.weights();
    off = s.b_off + s.cout;
  }
  return L;
}

int64_t total_params(const std::vector<LayerSpec>& L) { return L.back().b_off + L.back().cout; }

std::string hip_msg(hipError_t e, const char* what) { return std::string(what) + ": " + hipGetErrorString(e); }

}  // namespace

struct ws_net {
  ws_config cfg{};
  hipStream_t stream = nullptr;
  std::string err;
  std::vector<LayerSpec> layers;
  int64_t n_params = 0;
  int64_t step = 0;
  int Lpos = 0;   // positions per window after the embedding
  std::vector<void*> allocs;
  float *theta = nullptr, *grad = nullptr, *adam_m = nullptr, *adam_v = nullptr;
  float *mu = nullptr, *sigma = nullptr;
  float *xb = nullptr, *tb = nullptr, *out = nullptr, *dout = nullptr;
  std::vector<float*> H, A;   // H[0..hidden], A[1..hidden] (A[0] unused: h0 is its own relu output)
  float *dh[2] = {nullptr, nullptr}, *dz[2] = {nullptr, nullptr};
  float *part = nullptr, *loss_part = nullptr, *loss = nullptr;
  int* bad_index = nullptr;   // set by the batch gather when an index is out of range
  short* wt16 = nullptr;      // BF16 weights packed for k_net_mfma: embedding, residual layers, head
  bool net_fused = false;     // the inference form runs k_net_mfma (C = 128 or 256, 128 % Lpos == 0)
  // FP32 weights packed for k_conv_direct: of each layer for the forward pass,
  // then of each layer after the embedding for the backward one
  float* wt32 = nullptr;
  std::vector<float*> wt_fwd, wt_bwd;   // null: the layer does not run it
  int64_t part_floats = 0;
  int* win_track = nullptr;
  int* win_start = nullptr;
  int* first = nullptr;
  int64_t* meas_off = nullptr;
  int64_t n_windows = 0;
  int n_tracks = 0;
  std::vector<void*> plan_allocs;

  ws_status fail(ws_status s, std::string msg) {
    err = std::move(msg);
    return s;
  }

  hipError_t alloc(void** p, size_t bytes, std::vector<void*>& list) {
    const hipError_t e = hipMalloc(p, std::max<size_t>(bytes, 16));
    if (e == hipSuccess) list.push_back(*p);
    return e;
  }

  ~ws_net() {
    for (void* p : plan_allocs) (void)hipFree(p);
    for (void* p : allocs) (void)hipFree(p);
  }

  wsn::WindowTable table() const { return {win_track, win_start, meas_off, first}; }

  ws_status setup(const ws_config& c, hipStream_t s) {
    cfg = c;
    stream = s;
    layers = layer_specs(c);
    n_params = total_params(layers);
    Lpos = c.window / c.patch;
    const int64_t nb = c.max_batch;
    const size_t pos = size_t(nb) * Lpos;
    hipError_t e = hipSuccess;
    auto A_ = [&](float** p, size_t floats) {
      if (e == hipSuccess) e = alloc(reinterpret_cast<void**>(p), floats * sizeof(float), allocs);
    };
    A_(&theta, n_params);
    A_(&grad, n_params);
    A_(&adam_m, n_params);
    A_(&adam_v, n_params);
    A_(&mu, c.nx);
    A_(&sigma, c.nx);
    A_(&xb, size_t(2 * c.ny) * nb * c.window);
    A_(&tb, size_t(c.patch) * c.nx * pos);
    A_(&out, size_t(c.patch) * c.nx * pos);
    A_(&dout, size_t(c.patch) * c.nx * pos);
    H.assign(c.hidden + 1, nullptr);
    A.assign(c.hidden + 1, nullptr);
    for (int l = 0; l <= c.hidden; ++l) A_(&H[l], size_t(c.width) * pos);
    for (int l = 1; l <= c.hidden; ++l) A_(&A[l], size_t(c.width) * pos);
    for (int i = 0; i < 2; ++i) {
      A_(&dh[i], size_t(c.width) * pos);
      A_(&dz[i], size_t(c.width) * pos);
    }
    // bounds, not the chunks of max_batch: smaller batches may have more (wgrad_chunks.hpp)
    for (const auto& L : layers) {
      const int Kr = L.cin * L.K;
      const int chunks =
          direct(L) ? wsn::direct_bound(L.cout, wgrad_channels(L), int(pos)) : wsn::wgrad_bound(L.cout, Kr, int(pos));
      part_floats = std::max<int64_t>(part_floats, int64_t(chunks) * L.cout * (Kr + 1));
    }
    A_(&part, part_floats);
    A_(&loss_part, 1024);
    A_(&loss, 1);
    if (e == hipSuccess) e = alloc(reinterpret_cast<void**>(&bad_index), sizeof(int), allocs);
    net_fused = (c.width == 128 || c.width == 256) && wsn::kNetP % Lpos == 0;
    if (net_fused && e == hipSuccess) {
      int64_t words = 0;
      for (const auto& L : layers) words += wsn::net_words(L.cout, L.cin * L.K);
      e = alloc(reinterpret_cast<void**>(&wt16), sizeof(short) * size_t(words), allocs);
    }
    int64_t words = 0;
    std::vector<int64_t> at;
    for (int tr = 0; tr < 2; ++tr)
      for (const auto& L : layers) {
        const bool used = direct(L) && !(tr && &L == &layers.front());
        at.push_back(used ? words : -1);
        if (used) words += direct_words(L, tr);
      }
    A_(&wt32, size_t(words));
    for (size_t i = 0; i < at.size(); ++i)
      (i < layers.size() ? wt_fwd : wt_bwd).push_back(at[i] < 0 ? nullptr : wt32 + at[i]);
    if (e != hipSuccess)
      return fail(e == hipErrorOutOfMemory ? WS_ENOMEM : WS_EDEVICE, hip_msg(e, "device allocation"));
    std::vector<float> ones(c.nx, 1.f);
    e = hipMemsetAsync(theta, 0, sizeof(float) * n_params, stream);
    if (e == hipSuccess) e = hipMemsetAsync(adam_m, 0, sizeof(float) * n_params, stream);
    if (e == hipSuccess) e = hipMemsetAsync(adam_v, 0, sizeof(float) * n_params, stream);
    if (e == hipSuccess) e = hipMemsetAsync(mu, 0, sizeof(float) * c.nx, stream);
    if (e == hipSuccess) e = hipMemsetAsync(bad_index, 0, sizeof(int), stream);
    if (e == hipSuccess) e = hipMemcpyAsync(sigma, ones.data(), sizeof(float) * c.nx, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) {
      pack();
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return fail(WS_EDEVICE, hip_msg(e, "initialisation"));
    return WS_OK;
  }

  // the generic forms: FP32 (residual, backward), and BF16 products (forward)
  template <int EPI>
  void conv(const wsn::ConvArgs& a) {
    const dim3 grid(unsigned((a.N + wsn::kTile - 1) / wsn::kTile), unsigned((a.M + wsn::kTile - 1) / wsn::kTile));
    hipLaunchKernelGGL(wsn::k_conv<EPI>, grid, dim3(wsn::kThreads), 0, stream, a);
  }
  template <int EPI>
  void conv_mfma(const wsn::ConvArgs& a) {
    const dim3 grid(unsigned((a.N + wsn::kTile - 1) / wsn::kTile), unsigned((a.M + wsn::kTile - 1) / wsn::kTile));
    hipLaunchKernelGGL(wsn::k_conv_mfma<EPI>, grid, dim3(wsn::kThreads), 0, stream, a);
  }

  wsn::Gather gather_of(const LayerSpec& L, const float* src, int n, bool transpose_taps) const {
    const int W = cfg.window;
    if (&L == &layers.front()) return {src, n * W, L.K, Lpos, W, L.stride, L.dil, L.pad};
    if (transpose_taps) return {src, n * Lpos, L.K, Lpos, Lpos, 1, -L.dil, -L.pad};
    return {src, n * Lpos, L.K, Lpos, Lpos, 1, L.dil, L.pad};
  }

  // Whether a layer runs the direct matrix-core forms: its taps stay in the
  // window, so a tile of 64 positions has to hold whole windows; one tap needs
  // nothing of the sort.
  bool direct(const LayerSpec& L) const { return L.K == 1 || &L == &layers.front() || wsn::kDirP % Lpos == 0; }

  // rows, channels and taps of a layer's convolution; the embedding takes each
  // patch's steps as channels
  wsn::PackDirect pack_of(const LayerSpec& L, bool transposed) const {
    const bool embed = &L == &layers.front();
    return {theta + L.w_off, transposed ? L.cin : L.cout, transposed ? L.cout : (embed ? L.cin * L.K : L.cin),
            embed ? 1 : L.K, transposed ? 1 : 0, nullptr};
  }
  int64_t direct_words(const LayerSpec& L, bool transposed) const {
    const wsn::PackDirect p = pack_of(L, transposed);
    return wsn::direct_words(p.M, p.Cin, p.KT);
  }

  // The packed copies of the weights (wt32, wt16).  Queued by every call that
  // changes the parameters, right behind the change: whatever is queued later,
  // a replay of a captured call among it, finds the copies of the parameters it
  // runs with, and no call has to know which parameters were packed last.
  void pack() {
    static_assert(2 * kMostLayers <= wsn::kPackDirect && kMostLayers <= wsn::kPackNet, "tables of k_pack");
    wsn::PackArgs a{};
    for (int tr = 0; tr < 2; ++tr)
      for (size_t l = 0; l < layers.size(); ++l) {
        float* out = (tr ? wt_bwd : wt_fwd)[l];
        if (!out) continue;
        a.direct[a.n_direct] = pack_of(layers[l], tr != 0);
        a.direct[a.n_direct++].out = out;
      }
    if (net_fused) {
      short* out = wt16;
      for (size_t l = 0; l < layers.size(); ++l) {
        const LayerSpec& L = layers[l];
        a.net[a.n_net++] = {theta + L.w_off, L.cout, L.cin, L.K, l > 0 ? 1 : 0, out};
        out += wsn::net_words(L.cout, L.cin * L.K);
      }
    }
    hipLaunchKernelGGL(wsn::k_pack, dim3(64, unsigned(a.n_direct + a.n_net)), dim3(256), 0, stream, a);
  }

  // src as the layer's channels see it
  wsn::DirectArgs direct_args(const LayerSpec& L, const float* src, int n, bool transposed) const {
    const bool embed = &L == &layers.front();
    const wsn::PackDirect p = pack_of(L, transposed);
    wsn::DirectArgs a{};
    a.N = n * Lpos;
    a.M = p.M;
    a.Cin = p.Cin;
    a.Lpos = Lpos;
    a.W = (transposed ? wt_bwd : wt_fwd)[&L - layers.data()];
    a.bias = theta + L.b_off;
    a.src = src;
    a.ld = embed ? n * cfg.window : a.N;
    a.patch = embed ? L.K : 1;
    a.dil = transposed ? -L.dil : L.dil;
    return a;
  }

  template <int KT, int EPI>
  void conv_direct_k(const wsn::DirectArgs& a) {
    const unsigned gy = unsigned((a.M + 127) / 128);
    if (KT == 1 || 32 % a.Lpos == 0)
      hipLaunchKernelGGL((wsn::k_conv_direct<KT, EPI, 1>), dim3(unsigned((a.N + 31) / 32), gy), dim3(256), 0, stream, a);
    else
      hipLaunchKernelGGL((wsn::k_conv_direct<KT, EPI, 2>), dim3(unsigned((a.N + 63) / 64), gy), dim3(512), 0, stream, a);
  }
  template <int EPI>
  void conv_direct(const LayerSpec& L, const wsn::DirectArgs& a) {
    if (L.K == 3 && &L != &layers.front()) conv_direct_k<3, EPI>(a);
    else conv_direct_k<1, EPI>(a);
  }

  // xb [2 ny][n W] -> out [P nx][n L]; keeps every activation for the backward pass
  void forward(int n) {
    const int Hn = cfg.hidden;
    wsn::DirectArgs e = direct_args(layers[0], xb, n, false);
    e.out = H[0];
    conv_direct<wsn::kEpiRelu>(layers[0], e);
    for (int l = 1; l <= Hn; ++l) {
      const LayerSpec& L = layers[l];
      if (direct(L)) {
        wsn::DirectArgs d = direct_args(L, H[l - 1], n, false);
        d.out = A[l];
        d.out2 = H[l];
        d.in2 = H[l - 1];
        conv_direct<wsn::kEpiResidual>(L, d);
      } else {
        conv<wsn::kEpiResidual>({L.cout, L.cin * L.K, n * Lpos, theta + L.w_off, 0, theta + L.b_off,
                                 gather_of(L, H[l - 1], n, false), A[l], H[l], H[l - 1], nullptr});
      }
    }
    wsn::DirectArgs h = direct_args(layers[Hn + 1], H[Hn], n, false);
    h.out = out;
    conv_direct<wsn::kEpiLinear>(layers[Hn + 1], h);
  }

  // The inference form of the products layer by layer (BF16 operands on the
  // matrix cores, FP32 accumulation), where k_net_mfma does not apply
  void forward_mfma(int n) {
    const int Hn = cfg.hidden;
    embed_mfma(n);
    for (int l = 1; l <= Hn; ++l) {
      wsn::ConvArgs a = args_mfma(layers[l], H[l - 1], n);
      a.out = A[l];
      a.out2 = H[l];
      a.in2 = H[l - 1];
      conv_mfma<wsn::kEpiResidual>(a);
    }
    head_mfma(n);
  }
  wsn::ConvArgs args_mfma(const LayerSpec& L, const float* src, int n) const {
    return {L.cout, L.cin * L.K, n * Lpos, theta + L.w_off, 0, theta + L.b_off, gather_of(L, src, n, false),
            nullptr, nullptr, nullptr, nullptr};
  }
  void embed_mfma(int n) {
    wsn::ConvArgs a = args_mfma(layers[0], xb, n);
    a.out = H[0];
    conv_mfma<wsn::kEpiRelu>(a);
  }
  void head_mfma(int n) {
    wsn::ConvArgs a = args_mfma(layers.back(), H[cfg.hidden], n);
    a.out = out;
    conv_mfma<wsn::kEpiLinear>(a);
  }

  // network inputs of planned windows w0 .. w0 + n - 1 into xb
  void features(const double* d_y, int64_t w0, int n) {
    const int64_t cnt = int64_t(n) * cfg.window;
    hipLaunchKernelGGL(wsn::k_features, dim3(unsigned((cnt + 255) / 256)), dim3(256), 0, stream, table(), d_y, cfg.ny,
                       cfg.window, w0, n, 1, xb);
  }
  // states of those windows from their outputs
  void scatter(double* d_mean, int64_t w0, int n) {
    const int64_t cnt = int64_t(n) * cfg.window;
    hipLaunchKernelGGL(wsn::k_scatter, dim3(unsigned((cnt + 255) / 256)), dim3(256), 0, stream, table(),
                       static_cast<const float*>(out), w0, n, cfg.window, cfg.patch, cfg.nx,
                       static_cast<const float*>(mu), static_cast<const float*>(sigma), d_mean);
  }

  template <int C>
  void net_mfma(const wsn::NetArgs& a, dim3 grid, bool wide_in, bool wide_out) {
    if (wide_in && wide_out)
      hipLaunchKernelGGL((wsn::k_net_mfma<C, false, false>), grid, dim3(256), 0, stream, a);
    else if (wide_in)
      hipLaunchKernelGGL((wsn::k_net_mfma<C, false, true>), grid, dim3(256), 0, stream, a);
    else if (wide_out)
      hipLaunchKernelGGL((wsn::k_net_mfma<C, true, false>), grid, dim3(256), 0, stream, a);
    else
      hipLaunchKernelGGL((wsn::k_net_mfma<C, true, true>), grid, dim3(256), 0, stream, a);
  }

  // Trajectory of every planned window through k_net_mfma.  A block of it works
  // through all columns of the embedding and all rows of the head of its 128
  // positions.  Where blocks are few and columns or rows many, these two are
  // launches of their own, which spread over rows and columns too, with their
  // operands in the workspace.
  // Embedding: in the kernel with one block of `width` columns, or, when the
  // blocks fill the chip, with more of them (2 sensors, patches of 64, 512 blocks:
  // 233 us, 323 with a launch of its own; 16 sensors, patches of 16: 4 blocks 158
  // and 120, 128 blocks 178 and 168); never when a sensor's sines and cosines would
  // fall into different blocks (2 sensors, 4096 steps in 4 patches, 4 blocks: 23.3
  // ms a call when every column block formed all of them, 0.58 now).
  // Head: 0.19 us a row in the kernel whatever the blocks, 15 us and 1.8 ns a row
  // and block outside (320 rows: 4 blocks 120 and 79 us a call, 128 blocks 138 and
  // 166), equal where rows (104 - blocks) = 8300.
  void trajectory_fused(const double* d_y, double* d_mean) {
    const LayerSpec &LE = layers.front(), &LH = layers.back();
    wsn::NetArgs a{};
    a.tab = table();
    a.y = d_y;
    a.mean = d_mean;
    a.ny = cfg.ny;
    a.W = cfg.window;
    a.P = cfg.patch;
    a.nx = cfg.nx;
    a.Lpos = Lpos;
    a.hidden = cfg.hidden;
    a.we = wt16;
    a.wr = a.we + wsn::net_words(LE.cout, LE.cin * LE.K);
    a.wh = a.wr + cfg.hidden * wsn::net_words(cfg.width, 3 * cfg.width);
    a.be = theta + LE.b_off;
    a.bh = theta + LH.b_off;
    a.br = theta + layers[1].b_off;     // without residual layers not read
    a.br_stride = layers[1].weights() + layers[1].cout;
    a.mu = mu;
    a.sigma = sigma;
    const int64_t blocks = (n_windows * Lpos + wsn::kNetP - 1) / wsn::kNetP;
    const bool wide_in = LE.cin * LE.K > cfg.width && (blocks < 256 || cfg.width % (2 * cfg.patch) != 0);
    const bool wide_out = LH.cout * (104 - blocks) > 8300;
    // windows per launch: the workspace, else the grid size
    const int64_t most = wide_in || wide_out ? cfg.max_batch : int64_t(1) << 20;
    for (int64_t w0 = 0; w0 < n_windows; w0 += most) {
      a.w0 = w0;
      a.n = std::min(most, n_windows - w0);
      if (wide_in) {
        features(d_y, w0, int(a.n));
        embed_mfma(int(a.n));
        a.h0 = H[0];
      }
      if (wide_out) a.h1 = H[cfg.hidden];
      const dim3 grid(unsigned((a.n * Lpos + wsn::kNetP - 1) / wsn::kNetP));
      if (cfg.width == 128) net_mfma<128>(a, grid, wide_in, wide_out);
      else net_mfma<256>(a, grid, wide_in, wide_out);
      if (wide_out) {
        head_mfma(int(a.n));
        scatter(d_mean, w0, int(a.n));
      }
    }
  }

  // source channels of a layer's direct weight gradient
  int wgrad_channels(const LayerSpec& L) const { return &L == &layers.front() ? L.cin * L.K : L.cin; }

  template <int KT>
  void wgrad_direct_k(const wsn::DirectWgradArgs& a, int chunks) {
    hipLaunchKernelGGL(wsn::k_wgrad_direct<KT>,
                       dim3(unsigned((a.Cin + 31) / 32), unsigned((a.M + 127) / 128), unsigned(chunks)), dim3(256), 0,
                       stream, a);
  }

  // gradient of layer L: D [cout][N] its output's, src its input
  void wgrad(const LayerSpec& L, const float* D, const float* src, int n) {
    const int N = n * Lpos;
    const int Kr = L.cin * L.K;
    if (direct(L)) {
      const bool embed = &L == &layers.front();
      wsn::DirectWgradArgs a{};
      a.M = L.cout;
      a.Cin = wgrad_channels(L);
      const wsn::Chunks c = wsn::direct_chunks(a.M, a.Cin, N);
      a.chunk = c.chunk;
      a.N = N;
      a.Lpos = Lpos;
      a.D = D;
      a.src = src;
      a.ld = embed ? n * cfg.window : N;
      a.patch = embed ? L.K : 1;
      a.dil = L.dil;
      a.part = part;
      if (L.K == 3 && !embed) wgrad_direct_k<3>(a, c.count);
      else wgrad_direct_k<1>(a, c.count);
      wgrad_sum(L, c.count);
      return;
    }
    const wsn::Gather g = gather_of(L, src, n, false);
    const wsn::Chunks c = wsn::wgrad_chunks(L.cout, Kr, N);
    const wsn::WgradArgs a{L.cout, Kr, N, c.chunk, D, g, part};
    const dim3 grid(unsigned((Kr + 1 + wsn::kTile - 1) / wsn::kTile), unsigned((L.cout + wsn::kTile - 1) / wsn::kTile),
                    unsigned(c.count));
    hipLaunchKernelGGL(wsn::k_wgrad, grid, dim3(wsn::kThreads), 0, stream, a);
    wgrad_sum(L, c.count);
  }

  void wgrad_sum(const LayerSpec& L, int chunks) {
    const int Kr = L.cin * L.K, cnt = L.cout * (Kr + 1);
    hipLaunchKernelGGL(wsn::k_wgrad_reduce, dim3(unsigned((cnt + 63) / 64)), dim3(256), 0, stream,
                       static_cast<const float*>(part), chunks, L.cout, Kr, grad, L.w_off, L.b_off);
  }

  // loss of out against tb, gradient of every parameter into grad
  void loss_and_backward(int n) {
    const int N = n * Lpos;
    const int Hn = cfg.hidden;
    const int64_t count = int64_t(cfg.patch) * cfg.nx * N;
    const int blocks = int(std::min<int64_t>(1024, (count + 255) / 256));
    hipLaunchKernelGGL(wsn::k_mse, dim3(blocks), dim3(256), 0, stream, static_cast<const float*>(out),
                       static_cast<const float*>(tb), dout, count, float(2.0 / double(count)), loss_part);
    hipLaunchKernelGGL(wsn::k_sum, dim3(1), dim3(256), 0, stream, static_cast<const float*>(loss_part), blocks,
                       float(1.0 / double(count)), loss);
    const LayerSpec& LH = layers[Hn + 1];
    wgrad(LH, dout, H[Hn], n);
    {
      wsn::DirectArgs d = direct_args(LH, dout, n, true);
      d.out = dh[0];
      d.out2 = dz[0];
      d.mask = Hn >= 1 ? A[Hn] : H[0];
      conv_direct<wsn::kEpiBackward>(LH, d);
    }
    int cur = 0;
    for (int l = Hn; l >= 1; --l) {
      const LayerSpec& L = layers[l];
      wgrad(L, dz[cur], H[l - 1], n);
      float* below = l > 1 ? dh[1 - cur] : nullptr;
      const float* mask = l - 1 >= 1 ? A[l - 1] : H[0];
      if (direct(L)) {
        wsn::DirectArgs d = direct_args(L, dz[cur], n, true);
        d.out = below;
        d.out2 = dz[1 - cur];
        d.in2 = dh[cur];
        d.mask = mask;
        conv_direct<wsn::kEpiBackward>(L, d);
        cur ^= 1;
        continue;
      }
      wsn::ConvArgs a{L.cin, L.cout * L.K, N, theta + L.w_off, 1, nullptr, gather_of(L, dz[cur], n, true),
                      below, dz[1 - cur], dh[cur], mask};
      conv<wsn::kEpiBackward>(a);
      cur ^= 1;
    }
    const LayerSpec& L0 = layers[0];
    wgrad(L0, dz[cur], xb, n);
  }

  void gather_batch(const float* x, const float* lab, int64_t n_data, const int32_t* idx, int n) {
    const int64_t cnt = int64_t(n) * cfg.window;
    hipLaunchKernelGGL(wsn::k_gather_batch, dim3(unsigned((cnt + 255) / 256)), dim3(256), 0, stream, x, lab, n_data,
                       idx, n, 2 * cfg.ny, cfg.window, cfg.patch, cfg.nx, static_cast<const float*>(mu),
                       static_cast<const float*>(sigma), xb, lab ? tb : nullptr, bad_index);
  }

  // Waits for the stream; reports (and clears) an out-of-range batch index
  // seen since the last check.
  ws_status sync_and_check(const char* what) {
    int bad = 0;
    hipError_t e = hipMemcpyAsync(&bad, bad_index, sizeof(int), hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return fail(WS_EDEVICE, hip_msg(e, what));
    if (bad) {
      e = hipMemsetAsync(bad_index, 0, sizeof(int), stream);
      if (e == hipSuccess) e = hipStreamSynchronize(stream);
      return fail(WS_EINVAL, "a batch index was outside [0, n_data): its window was read as zeros");
    }
    return WS_OK;
  }
};

namespace {

ws_status launch_status(ws_t h, const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return h->fail(WS_EDEVICE, hip_msg(e, what));
  return WS_OK;
}

const char* check_batch(ws_t h, const void* x, int64_t n_data, const int32_t* idx, int32_t n, bool limited) {
  if (!x || !idx) return "null device pointer";
  if (n_data < 1) return "n_data must be >= 1";
  if (n < 1) return "batch size must be >= 1";
  if (limited && n > h->cfg.max_batch) return "batch size exceeds max_batch";
  return nullptr;
}

}  // namespace

extern "C" {

void ws_config_defaults(ws_config* c) {
  if (!c) return;
  c->window = 64;
  c->patch = 4;
  c->width = 128;
  c->hidden = 4;
  c->nx = 5;
  c->ny = 2;
  c->max_batch = 1024;
}

int64_t ws_param_count(const ws_config* c) {
  if (!c || check_config(*c)) return 0;
  return total_params(layer_specs(*c));
}

ws_status ws_create(const ws_config* cfg, void* hip_stream, ws_t* out) {
  if (!out) {
    g_create_error = "out is NULL";
    return WS_EINVAL;
  }
  *out = nullptr;
  if (!cfg) {
    g_create_error = "cfg is NULL";
    return WS_EINVAL;
  }
  if (const char* m = check_config(*cfg)) {
    g_create_error = m;
    return WS_EINVAL;
  }
  ws_net* h = new (std::nothrow) ws_net();
  if (!h) {
    g_create_error = "host allocation failed";
    return WS_ENOMEM;
  }
  const ws_status s = h->setup(*cfg, static_cast<hipStream_t>(hip_stream));
  if (s != WS_OK) {
    g_create_error = h->err;
    delete h;
    return s;
  }
  *out = h;
  return WS_OK;
}

ws_status ws_set_params(ws_t h, const float* params, int64_t n) {
  if (!h) return WS_ESTATE;
  if (!params || n != h->n_params) return h->fail(WS_EINVAL, "params must hold ws_param_count() floats");
  for (int64_t i = 0; i < n; ++i)
    if (!std::isfinite(params[i])) return h->fail(WS_EINVAL, "params must be finite");
  hipError_t e = hipMemcpyAsync(h->theta, params, sizeof(float) * n, hipMemcpyHostToDevice, h->stream);
  if (e == hipSuccess) {
    h->pack();
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemsetAsync(h->adam_m, 0, sizeof(float) * n, h->stream);
  if (e == hipSuccess) e = hipMemsetAsync(h->adam_v, 0, sizeof(float) * n, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return h->fail(WS_EDEVICE, hip_msg(e, "parameter upload"));
  h->step = 0;
  return WS_OK;
}

ws_status ws_get_params(ws_t h, float* params, int64_t n) {
  if (!h) return WS_ESTATE;
  if (!params || n != h->n_params) return h->fail(WS_EINVAL, "params must hold ws_param_count() floats");
  hipError_t e = hipMemcpyAsync(params, h->theta, sizeof(float) * n, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return h->fail(WS_EDEVICE, hip_msg(e, "parameter download"));
  return WS_OK;
}

ws_status ws_set_normalization(ws_t h, const float* mu, const float* sigma) {
  if (!h) return WS_ESTATE;
  if (!mu || !sigma) return h->fail(WS_EINVAL, "mu and sigma are required");
  for (int i = 0; i < h->cfg.nx; ++i)
    if (!std::isfinite(mu[i]) || !std::isfinite(sigma[i]) || !(sigma[i] > 0.f))
      return h->fail(WS_EINVAL, "mu must be finite and sigma finite and positive");
  hipError_t e = hipMemcpyAsync(h->mu, mu, sizeof(float) * h->cfg.nx, hipMemcpyHostToDevice, h->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(h->sigma, sigma, sizeof(float) * h->cfg.nx, hipMemcpyHostToDevice, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return h->fail(WS_EDEVICE, hip_msg(e, "normalisation upload"));
  return WS_OK;
}

ws_status ws_set_tracks(ws_t h, const int64_t* offsets, int32_t n_tracks, int64_t* n_windows) {
  if (!h) return WS_ESTATE;
  if (!offsets || n_tracks < 1) return h->fail(WS_EINVAL, "offsets and n_tracks >= 1 are required");
  if (offsets[0] != 0) return h->fail(WS_EINVAL, "offsets[0] must be 0");
  const int W = h->cfg.window;
  std::vector<int> track, start, first(size_t(n_tracks) + 1, 0);
  for (int i = 0; i < n_tracks; ++i) {
    const int64_t T = offsets[i + 1] - offsets[i];
    if (T < 1) return h->fail(WS_EINVAL, "every track needs T >= 1 measurements");
    if (T > (int64_t(1) << 30)) return h->fail(WS_EINVAL, "track too long");
    const int64_t nw = (T + W - 1) / W;
    if (int64_t(track.size()) + nw > (int64_t(1) << 31) - 1) return h->fail(WS_EINVAL, "too many windows");
    for (int64_t w = 0; w < nw; ++w) {
      track.push_back(i);
      start.push_back(int(w < nw - 1 ? 1 + W * w : std::max<int64_t>(1, T - W + 1)));
    }
    first[i + 1] = int(track.size());
  }
  for (void* p : h->plan_allocs) (void)hipFree(p);
  h->plan_allocs.clear();
  h->n_windows = 0;
  h->n_tracks = 0;
  const size_t nw = track.size();
  hipError_t e = h->alloc(reinterpret_cast<void**>(&h->win_track), sizeof(int) * nw, h->plan_allocs);
  if (e == hipSuccess) e = h->alloc(reinterpret_cast<void**>(&h->win_start), sizeof(int) * nw, h->plan_allocs);
  if (e == hipSuccess) e = h->alloc(reinterpret_cast<void**>(&h->first), sizeof(int) * first.size(), h->plan_allocs);
  if (e == hipSuccess)
    e = h->alloc(reinterpret_cast<void**>(&h->meas_off), sizeof(int64_t) * (size_t(n_tracks) + 1), h->plan_allocs);
  if (e == hipSuccess) e = hipMemcpyAsync(h->win_track, track.data(), sizeof(int) * nw, hipMemcpyHostToDevice, h->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(h->win_start, start.data(), sizeof(int) * nw, hipMemcpyHostToDevice, h->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(h->first, first.data(), sizeof(int) * first.size(), hipMemcpyHostToDevice, h->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(h->meas_off, offsets, sizeof(int64_t) * (size_t(n_tracks) + 1), hipMemcpyHostToDevice,
                       h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return h->fail(e == hipErrorOutOfMemory ? WS_ENOMEM : WS_EDEVICE, hip_msg(e, "window plan"));
  h->n_windows = int64_t(nw);
  h->n_tracks = n_tracks;
  if (n_windows) *n_windows = int64_t(nw);
  return WS_OK;
}

ws_status ws_windows(ws_t h, const double* d_y, float* d_x) {
  if (!h) return WS_ESTATE;
  if (!h->n_windows) return h->fail(WS_ESTATE, "no tracks planned (ws_set_tracks)");
  if (!d_y || !d_x) return h->fail(WS_EINVAL, "null device pointer");
  if (h->n_windows > (int64_t(1) << 31) - 1) return h->fail(WS_EINVAL, "too many windows");
  const int64_t cnt = h->n_windows * h->cfg.window;
  hipLaunchKernelGGL(wsn::k_features, dim3(unsigned((cnt + 255) / 256)), dim3(256), 0, h->stream, h->table(), d_y,
                     h->cfg.ny, h->cfg.window, int64_t(0), int(h->n_windows), 0, d_x);
  return launch_status(h, "feature kernel");
}

ws_status ws_labels(ws_t h, const double* d_mean, float* d_lab) {
  if (!h) return WS_ESTATE;
  if (!h->n_windows) return h->fail(WS_ESTATE, "no tracks planned (ws_set_tracks)");
  if (!d_mean || !d_lab) return h->fail(WS_EINVAL, "null device pointer");
  const int64_t cnt = h->n_windows * h->cfg.window;
  hipLaunchKernelGGL(wsn::k_labels, dim3(unsigned((cnt + 255) / 256)), dim3(256), 0, h->stream, h->table(), d_mean,
                     h->cfg.nx, h->cfg.window, h->n_windows, d_lab);
  return launch_status(h, "label kernel");
}

ws_status ws_train_step(ws_t h, const float* d_x, const float* d_lab, int64_t n_data, const int32_t* d_idx,
                        int32_t n, const ws_adam* opt, float* loss_out) {
  if (!h) return WS_ESTATE;
  if (const char* m = check_batch(h, d_x, n_data, d_idx, n, true)) return h->fail(WS_EINVAL, m);
  if (!d_lab || !opt) return h->fail(WS_EINVAL, "labels and optimiser settings are required");
  if (!(opt->lr > 0.f) || !(opt->beta1 >= 0.f && opt->beta1 < 1.f) || !(opt->beta2 >= 0.f && opt->beta2 < 1.f) ||
      !(opt->eps > 0.f))
    return h->fail(WS_EINVAL, "Adam needs lr > 0, 0 <= beta < 1, eps > 0");
  h->gather_batch(d_x, d_lab, n_data, d_idx, n);
  h->forward(n);
  h->loss_and_backward(n);
  h->step += 1;
  const float c1 = float(1.0 - std::pow(double(opt->beta1), double(h->step)));
  const float c2 = float(1.0 - std::pow(double(opt->beta2), double(h->step)));
  hipLaunchKernelGGL(wsn::k_adam, dim3(unsigned((h->n_params + 255) / 256)), dim3(256), 0, h->stream, h->theta,
                     static_cast<const float*>(h->grad), h->adam_m, h->adam_v, h->n_params, opt->lr, opt->beta1,
                     opt->beta2, opt->eps, c1, c2);
  h->pack();
  ws_status s = launch_status(h, "training step");
  if (s != WS_OK || !loss_out) return s;
  const hipError_t e = hipMemcpyAsync(loss_out, h->loss, sizeof(float), hipMemcpyDeviceToHost, h->stream);
  if (e != hipSuccess) return h->fail(WS_EDEVICE, hip_msg(e, "loss download"));
  return h->sync_and_check("loss download");
}

ws_status ws_gradient(ws_t h, const float* d_x, const float* d_lab, int64_t n_data, const int32_t* d_idx,
                      int32_t n, float* grad, float* loss_out) {
  if (!h) return WS_ESTATE;
  if (const char* m = check_batch(h, d_x, n_data, d_idx, n, true)) return h->fail(WS_EINVAL, m);
  if (!d_lab) return h->fail(WS_EINVAL, "labels are required");
  h->gather_batch(d_x, d_lab, n_data, d_idx, n);
  h->forward(n);
  h->loss_and_backward(n);
  ws_status s = launch_status(h, "gradient");
  if (s != WS_OK) return s;
  hipError_t e = hipSuccess;
  if (grad) e = hipMemcpyAsync(grad, h->grad, sizeof(float) * h->n_params, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess && loss_out) e = hipMemcpyAsync(loss_out, h->loss, sizeof(float), hipMemcpyDeviceToHost, h->stream);
  if (e != hipSuccess) return h->fail(WS_EDEVICE, hip_msg(e, "gradient download"));
  return h->sync_and_check("gradient download");
}

ws_status ws_predict(ws_t h, const float* d_x, int64_t n_data, const int32_t* d_idx, int32_t n, float* d_states) {
  if (!h) return WS_ESTATE;
  if (const char* m = check_batch(h, d_x, n_data, d_idx, n, false)) return h->fail(WS_EINVAL, m);
  if (!d_states) return h->fail(WS_EINVAL, "null device pointer");
  const int W = h->cfg.window;
  for (int32_t b0 = 0; b0 < n; b0 += h->cfg.max_batch) {
    const int nb = std::min(h->cfg.max_batch, n - b0);
    h->gather_batch(d_x, nullptr, n_data, d_idx + b0, nb);
    h->forward(nb);
    const int64_t cnt = int64_t(nb) * W;
    hipLaunchKernelGGL(wsn::k_states, dim3(unsigned((cnt + 255) / 256)), dim3(256), 0, h->stream,
                       static_cast<const float*>(h->out), nb, W, h->cfg.patch, h->cfg.nx,
                       static_cast<const float*>(h->mu), static_cast<const float*>(h->sigma),
                       d_states + size_t(b0) * W * h->cfg.nx);
  }
  const ws_status s = launch_status(h, "prediction");
  if (s != WS_OK) return s;
  return h->sync_and_check("prediction");
}

static ws_status trajectory(ws_t h, const double* d_y, double* d_mean, bool mfma) {
  if (!h) return WS_ESTATE;
  if (!h->n_windows) return h->fail(WS_ESTATE, "no tracks planned (ws_set_tracks)");
  if (!d_y || !d_mean) return h->fail(WS_EINVAL, "null device pointer");
  if (mfma && h->net_fused) {
    h->trajectory_fused(d_y, d_mean);
    return launch_status(h, "trajectory");
  }
  for (int64_t w0 = 0; w0 < h->n_windows; w0 += h->cfg.max_batch) {
    const int nb = int(std::min<int64_t>(h->cfg.max_batch, h->n_windows - w0));
    h->features(d_y, w0, nb);
    if (mfma) h->forward_mfma(nb);
    else h->forward(nb);
    h->scatter(d_mean, w0, nb);
  }
  return launch_status(h, "trajectory");
}

ws_status ws_trajectory(ws_t h, const double* d_y, double* d_mean) { return trajectory(h, d_y, d_mean, false); }

ws_status ws_trajectory_mfma(ws_t h, const double* d_y, double* d_mean) { return trajectory(h, d_y, d_mean, true); }

const char* ws_last_error(ws_t h) { return h ? h->err.c_str() : g_create_error.c_str(); }

void ws_destroy(ws_t h) {
  if (!h) return;
  (void)hipStreamSynchronize(h->stream);
  delete h;
}

}  // extern "C"
