// Host side of the warm-start network: layer plan, workspace layout and the
// launch sequences of inference, loss gradient and Adam.  Included inside the
// library's internal namespace of rism3d.hip (uses fail / HIP_TRY / TIMED).
//
// Architecture (levels L, channels C_l = base * 2^l, 3x3x3 convolutions with
// zero padding, leaky activations, 2x2x2 average pooling, nearest upsampling):
//   encoder l:  a_l = act(conv(in_l)), e_l = act(conv(a_l)), in_0 = input,
//               in_{l+1} = pool(e_l);
//   decoder l = L-2 .. 0:  da_l = act(conv([up(d_{l+1}), e_l])), d_l = act(conv(da_l)),
//               d_{L-1} = e_{L-1};
//   output = conv(d_0).
// Parameters (FP32, flat): per convolution in the order enc0a, enc0b, ...,
// enc{L-1}b, dec{L-2}a, dec{L-2}b, ..., dec0a, dec0b, out: W[C_out][27][C_in]
// (tap k = (dz * 3 + dy) * 3 + dx for offsets (dz-1, dy-1, dx-1)) then b[C_out].

struct NetLayer {
  int cin, cout;          // real channel counts
  int cin_pad, cout_pad;  // packed: cin to a multiple of 8, cout to a multiple of 16
  int level;
  size_t w_off, b_off;    // offsets in the parameter vector (floats)
  size_t wp, wf;          // workspace offsets of the packed and flipped BF16 weights
};

constexpr int kNetMaxLevels = 6;

struct NetPlan {
  rism3d_unet_config cfg;
  int nz[kNetMaxLevels], ny[kNetMaxLevels], nx[kNetMaxLevels];
  size_t nvox[kNetMaxLevels];
  std::vector<NetLayer> layers;
  size_t n_params = 0;
  size_t x0 = 0, a[kNetMaxLevels] = {}, e[kNetMaxLevels] = {}, p[kNetMaxLevels] = {},
         da[kNetMaxLevels] = {}, db[kNetMaxLevels] = {};
  size_t out = 0, ge[kNetMaxLevels] = {}, gdx = 0, dyp[2] = {}, partials = 0, loss = 0, slabs = 0;
  size_t total_infer = 0, total_train = 0;
  int c(int l) const { return cfg.base << l; }
};

constexpr int kMsePartials = 1024;

// The weight-gradient launch of a layer: output tiles a workgroup holds (two share
// a staged input tile; four would leave one workgroup a compute unit), voxel
// tiles, and the workgroups (= slabs) they are dealt to, for about 512 workgroups
// (two a compute unit) in all.
struct WgradShape {
  int ot, ypairs, tiles, per, slabs;
};
WgradShape wgrad_shape(int cin_pad, int cout_pad, int nx, int ny, int nz) {
  WgradShape w;
  const int cot = cout_pad / 16, cit = (cin_pad + 15) / 16;
  w.ot = cot >= 2 ? 2 : 1;
  w.ypairs = cit * ((cot + w.ot - 1) / w.ot);
  w.tiles = ((nx + net::kWgX - 1) / net::kWgX) * ((ny + net::kWgY - 1) / net::kWgY) *
            ((nz + net::kWgZ - 1) / net::kWgZ);
  const int want = std::max(1, 512 / w.ypairs);
  w.per = std::max(1, (w.tiles + want - 1) / want);
  w.slabs = (w.tiles + w.per - 1) / w.per;
  return w;
}

rism3d_status net_plan(const rism3d_unet_config* cfg, int nx, int ny, int nz, NetPlan* P) {
  if (!cfg) return fail(RISM3D_E_ARG, "null network configuration");
  const int L = cfg->levels;
  if (L < 1 || L > kNetMaxLevels) return fail(RISM3D_E_ARG, "levels must be in 1..%d", kNetMaxLevels);
  if (cfg->base < 16 || cfg->base % 16 || (cfg->base << (L - 1)) > 128)
    return fail(RISM3D_E_ARG, "base channels must be a multiple of 16 with base * 2^(levels-1) <= 128");
  if (cfg->in_channels < 1 || cfg->in_channels > 64 || cfg->out_channels < 1 ||
      cfg->out_channels > 64)
    return fail(RISM3D_E_ARG, "in/out channels must be in 1..64");
  if (!(cfg->slope >= 0.0f && cfg->slope < 1.0f)) return fail(RISM3D_E_ARG, "slope must be in [0, 1)");
  const int m = 1 << (L - 1);
  if (nx < m || ny < m || nz < m || nx % m || ny % m || nz % m)
    return fail(RISM3D_E_ARG, "grid %dx%dx%d: every axis must be a positive multiple of %d", nx, ny,
                nz, m);
  if ((size_t)nx * ny * nz > ((size_t)1 << 30))
    return fail(RISM3D_E_ARG, "grid too large for the network");
  P->cfg = *cfg;
  for (int l = 0; l < L; ++l) {
    P->nx[l] = nx >> l;
    P->ny[l] = ny >> l;
    P->nz[l] = nz >> l;
    P->nvox[l] = (size_t)P->nx[l] * P->ny[l] * P->nz[l];
  }
  P->layers.clear();
  auto add = [&](int cin, int cout, int level) {
    NetLayer ly;
    ly.cin = cin;
    ly.cout = cout;
    ly.cin_pad = (cin + 7) & ~7;
    ly.cout_pad = (cout + 15) & ~15;
    ly.level = level;
    ly.w_off = P->n_params;
    P->n_params += (size_t)cout * 27 * cin;
    ly.b_off = P->n_params;
    P->n_params += cout;
    P->layers.push_back(ly);
  };
  P->n_params = 0;
  for (int l = 0; l < L; ++l) {
    add(l == 0 ? cfg->in_channels : P->c(l - 1), P->c(l), l);
    add(P->c(l), P->c(l), l);
  }
  for (int l = L - 2; l >= 0; --l) {
    add(P->c(l + 1) + P->c(l), P->c(l), l);
    add(P->c(l), P->c(l), l);
  }
  add(P->c(0), cfg->out_channels, 0);
  // (192 x 128 channel pairs at most: base 16, 4 levels)
  for (const NetLayer& ly : P->layers)
    if ((ly.cout_pad / 16) * ((ly.cin_pad + 15) / 16) > 64)
      return fail(RISM3D_E_ARG, "layer %d x %d channels exceeds the weight-gradient tile budget",
                  ly.cin, ly.cout);

  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return o;
  };
  for (NetLayer& ly : P->layers) {
    ly.wp = take(net::conv_packed(ly.cout_pad, ly.cin_pad) * 2);
    ly.wf = take(net::conv_packed((ly.cin + 15) & ~15, ly.cout_pad) * 2);
  }
  P->x0 = take(P->nvox[0] * P->layers[0].cin_pad * 2);
  for (int l = 0; l < L; ++l) {
    if (l > 0) P->p[l] = take(P->nvox[l] * P->c(l - 1) * 2);
    P->a[l] = take(P->nvox[l] * P->c(l) * 2);
    P->e[l] = take(P->nvox[l] * P->c(l) * 2);
  }
  for (int l = L - 2; l >= 0; --l) {
    P->da[l] = take(P->nvox[l] * P->c(l) * 2);
    P->db[l] = take(P->nvox[l] * P->c(l) * 2);
  }
  P->total_infer = off;
  P->out = take(P->nvox[0] * cfg->out_channels * 4);
  // training: the BF16 gradient of the layer at hand and of the next, the FP32
  // gradients that cross a level (up or down), and the skip branches'
  size_t max_dx = 4, max_cout_pad = 0;
  for (const NetLayer& ly : P->layers)
    max_cout_pad = std::max(max_cout_pad, P->nvox[ly.level] * (size_t)ly.cout_pad);
  for (int l = 0; l + 1 < L; ++l) {
    P->ge[l] = take(P->nvox[l] * P->c(l) * 4);
    max_dx = std::max(max_dx, std::max(P->nvox[l] * P->c(l + 1), P->nvox[l + 1] * P->c(l)));
  }
  P->gdx = take(max_dx * 4);
  for (size_t& d : P->dyp) d = take(max_cout_pad * 2);
  P->partials = take(kMsePartials * sizeof(double));
  P->loss = take(sizeof(double));
  size_t slab_floats = 0;   // the slabs of the largest layer's gradient
  for (const NetLayer& ly : P->layers) {
    const WgradShape w = wgrad_shape(ly.cin_pad, ly.cout_pad, P->nx[ly.level], P->ny[ly.level],
                                     P->nz[ly.level]);
    slab_floats = std::max(slab_floats,
                           (size_t)w.slabs * ((size_t)ly.cout * 27 * ly.cin + ly.cout));
  }
  P->slabs = take(slab_floats * sizeof(float));
  P->total_train = off;
  return RISM3D_OK;
}

template <typename T>
T* wsp(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

unsigned net_blocks(size_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

void net_pack(const NetPlan& P, const float* params, void* ws, bool flipped, hipStream_t s) {
  net::PackTable t;
  memset(&t, 0, sizeof(t));
  size_t most = 0;
  for (size_t j = 0; j < P.layers.size(); ++j) {
    const NetLayer& ly = P.layers[j];
    const int cin16 = (ly.cin + 15) & ~15;
    t.l[j] = {params + ly.w_off, wsp<uint16_t>(ws, ly.wp),
              flipped ? wsp<uint16_t>(ws, ly.wf) : nullptr, ly.cout, ly.cin, ly.cout_pad, ly.cin_pad,
              cin16};
    most = std::max(most, net::conv_packed(ly.cout_pad, ly.cin_pad) +
                              (flipped ? net::conv_packed(cin16, ly.cout_pad) : 0));
  }
  // (one launch instead of a layer's each, which the 4 us of a launch bounded)
  hipLaunchKernelGGL(net::k_pack_weights, dim3(net_blocks(most / 8, 256), (unsigned)P.layers.size()),
                     dim3(256), 0, s, t);
}

// One convolution (channel counts are multiples of 8): the halo-tiled
// kernel, staging conv_chunk() channel groups (at most 67.5 KB of LDS) at a time.
// Tiles of 16 x 8 x 4 voxels, or 16 x 2 x 4 where those would give fewer than 512
// workgroups (the coarse levels); two output tiles a workgroup where that leaves
// 512 workgroups (64^3, 96 -> 32 channels: 85 us with one, 45 with two; three, for
// 16 -> 48 at 128^3, take 234 us against 145 with one, their accumulators spill).
template <int EPI, int CGC, int TY, int MT>
void net_conv_mt(const net::ConvArgs& a, unsigned tiles, hipStream_t s) {
  hipLaunchKernelGGL((net::k_conv3<EPI, CGC, TY, MT>), dim3(tiles, (unsigned)a.cout_pad / 16 / MT),
                     dim3(net::kConvThreads), 0, s, a);
}

template <int EPI, int CGC, int TY>
void net_conv_tiles(const net::ConvArgs& a, unsigned tiles, hipStream_t s) {
  const unsigned cot = (unsigned)a.cout_pad / 16;
  if constexpr (EPI != net::EPI_F32_SITE)
    if (cot % 2 == 0 && tiles * (cot / 2) >= 512) return net_conv_mt<EPI, CGC, TY, 2>(a, tiles, s);
  net_conv_mt<EPI, CGC, TY, 1>(a, tiles, s);
}

template <int EPI, int CGC>
void net_conv_chunks(const net::ConvArgs& a, hipStream_t s) {
  auto tiles = [&](int ty) {
    return (unsigned)((a.nx + net::kTileX - 1) / net::kTileX) * (unsigned)((a.ny + ty - 1) / ty) *
           (unsigned)((a.nz + net::kTileZ - 1) / net::kTileZ);
  };
  if (tiles(8) * (unsigned)(a.cout_pad / 16) >= 512) net_conv_tiles<EPI, CGC, 8>(a, tiles(8), s);
  else net_conv_tiles<EPI, CGC, 2>(a, tiles(2), s);
}

template <int EPI>
void net_conv(const net::ConvArgs& a, hipStream_t s) {
  switch (net::conv_chunk((a.in.ca + a.in.cb) / 8)) {
    case 4: net_conv_chunks<EPI, 4>(a, s); break;
    case 3: net_conv_chunks<EPI, 3>(a, s); break;
    case 2: net_conv_chunks<EPI, 2>(a, s); break;
    default: net_conv_chunks<EPI, 1>(a, s); break;
  }
}

net::ConvArgs conv_args(const NetPlan& P, const NetLayer& ly, void* ws, net::ConvIn in,
                        const float* params) {
  net::ConvArgs a;
  a.in = in;
  a.w = wsp<uint16_t>(ws, ly.wp);
  a.bias = params + ly.b_off;
  a.yb = nullptr;
  a.yf = a.yf2 = nullptr;
  a.act = nullptr;
  a.split = 0;
  a.cout = ly.cout;
  a.cout_pad = ly.cout_pad;
  a.nz = P.nz[ly.level];
  a.ny = P.ny[ly.level];
  a.nx = P.nx[ly.level];
  a.slope = P.cfg.slope;
  return a;
}

// Inputs of every convolution in parameter order (needed again by the
// weight gradients).
std::vector<net::ConvIn> net_inputs(const NetPlan& P, void* ws) {
  const int L = P.cfg.levels;
  std::vector<net::ConvIn> in;
  for (int l = 0; l < L; ++l) {
    if (l == 0) in.push_back({wsp<uint16_t>(ws, P.x0), nullptr, P.layers[0].cin_pad, 0, 0});
    else in.push_back({wsp<uint16_t>(ws, P.p[l]), nullptr, P.c(l - 1), 0, 0});
    in.push_back({wsp<uint16_t>(ws, P.a[l]), nullptr, P.c(l), 0, 0});
  }
  for (int l = L - 2; l >= 0; --l) {
    const size_t dprev = (l == L - 2) ? P.e[L - 1] : P.db[l + 1];
    in.push_back({wsp<uint16_t>(ws, dprev), wsp<uint16_t>(ws, P.e[l]), P.c(l + 1), P.c(l), 1});
    in.push_back({wsp<uint16_t>(ws, P.da[l]), nullptr, P.c(l), 0, 0});
  }
  in.push_back({wsp<uint16_t>(ws, L >= 2 ? P.db[0] : P.e[0]), nullptr, P.c(0), 0, 0});
  return in;
}

// Output tensor (BF16 activation) of every hidden convolution.
std::vector<size_t> net_outputs(const NetPlan& P) {
  const int L = P.cfg.levels;
  std::vector<size_t> out;
  for (int l = 0; l < L; ++l) {
    out.push_back(P.a[l]);
    out.push_back(P.e[l]);
  }
  for (int l = L - 2; l >= 0; --l) {
    out.push_back(P.da[l]);
    out.push_back(P.db[l]);
  }
  return out;
}

// Forward pass: input FP32 site-major [in_channels][N0] -> out FP32
// site-major [out_channels][N0].  Weights must be packed (net_pack).
void net_forward(const NetPlan& P, const float* params, const float* input, float* out, void* ws,
                 hipStream_t s) {
  const int L = P.cfg.levels;
  const NetLayer& l0 = P.layers[0];
  hipLaunchKernelGGL(net::k_to_channels_last, dim3(net_blocks(P.nvox[0], 256)),
                     dim3(256), 0, s, input, P.cfg.in_channels, l0.cin_pad, P.nvox[0],
                     wsp<uint16_t>(ws, P.x0));
  const std::vector<net::ConvIn> in = net_inputs(P, ws);
  const std::vector<size_t> outs = net_outputs(P);
  for (size_t j = 0; j + 1 < P.layers.size(); ++j) {
    const NetLayer& ly = P.layers[j];
    if (j >= 2 && j < (size_t)2 * L && j % 2 == 0) {   // encoder level l = j / 2 >= 1: pool e_{l-1}
      const int l = (int)j / 2;
      hipLaunchKernelGGL(net::k_pool2, dim3(net_blocks(P.nvox[l] * (P.c(l - 1) / 8), 256)),
                         dim3(256), 0, s, wsp<uint16_t>(ws, P.e[l - 1]), wsp<uint16_t>(ws, P.p[l]),
                         P.nz[l - 1], P.ny[l - 1], P.nx[l - 1], P.c(l - 1));
    }
    net::ConvArgs a = conv_args(P, ly, ws, in[j], params);
    a.yb = wsp<uint16_t>(ws, outs[j]);
    net_conv<net::EPI_BF16_LEAKY>(a, s);
  }
  const NetLayer& lo = P.layers.back();
  net::ConvArgs a = conv_args(P, lo, ws, in.back(), params);
  a.yf = out;
  net_conv<net::EPI_F32_SITE>(a, s);
}

// dX of one convolution: the transposed convolution of dy_pre with the flipped
// weights.
net::ConvArgs conv_dx_args(const NetPlan& P, const NetLayer& ly, void* ws, const uint16_t* dyp) {
  net::ConvArgs a;
  a.in = {dyp, nullptr, ly.cout_pad, 0, 0};
  a.w = wsp<uint16_t>(ws, ly.wf);
  a.bias = nullptr;
  a.yb = nullptr;
  a.yf = a.yf2 = nullptr;
  a.act = nullptr;
  a.split = 0;
  a.cout = ly.cin;
  a.cout_pad = (ly.cin + 15) & ~15;
  a.nz = P.nz[ly.level];
  a.ny = P.ny[ly.level];
  a.nx = P.nx[ly.level];
  a.slope = P.cfg.slope;
  return a;
}

// ... times the derivative of the activation act that the layer read: dy_pre of
// the layer before, BF16.
void net_conv_dx_leaky(const NetPlan& P, const NetLayer& ly, void* ws, const uint16_t* dyp,
                       size_t act, uint16_t* out, hipStream_t s) {
  net::ConvArgs a = conv_dx_args(P, ly, ws, dyp);
  a.act = wsp<uint16_t>(ws, act);
  a.yb = out;
  net_conv<net::EPI_BF16_DLEAKY>(a, s);
}

// ... in FP32 channels last: the first `split` channels to dx, the others to skip.
void net_conv_dx_split(const NetPlan& P, const NetLayer& ly, void* ws, const uint16_t* dyp, int split,
                       float* dx, float* skip, hipStream_t s) {
  net::ConvArgs a = conv_dx_args(P, ly, ws, dyp);
  a.yf = dx;
  a.yf2 = skip;
  a.split = split;
  net_conv<net::EPI_F32_SPLIT>(a, s);
}

// Weight and bias gradients of one layer, written to grad + w_off (b follows W).
void net_conv_dw(const NetPlan& P, const NetLayer& ly, const net::ConvIn& in, void* ws,
                 const uint16_t* dyp, float* grad, hipStream_t s) {
  const WgradShape sh = wgrad_shape(ly.cin_pad, ly.cout_pad, P.nx[ly.level], P.ny[ly.level],
                                    P.nz[ly.level]);
  float* slabs = wsp<float>(ws, P.slabs);
  net::WgradArgs w;
  w.in = in;
  w.dy = dyp;
  w.dw = slabs;
  w.cin_real = ly.cin;
  w.cout = ly.cout;
  w.cout_pad = ly.cout_pad;
  w.nz = P.nz[ly.level];
  w.ny = P.ny[ly.level];
  w.nx = P.nx[ly.level];
  w.tiles = sh.tiles;
  w.per = sh.per;
  const dim3 grid((unsigned)sh.slabs, (unsigned)sh.ypairs), block(net::kConvThreads);
  hipLaunchKernelGGL(sh.ot == 2 ? &net::k_conv3_wgrad<2> : &net::k_conv3_wgrad<1>, grid, block, 0,
                     s, w);
  const size_t n = (size_t)ly.cout * 27 * ly.cin + ly.cout;
  // sixteen threads an element where there are slabs for them: 15.5 us a layer of
  // the 128^3 step with one, 6.0 with up to sixteen
  const unsigned rows = sh.slabs >= 64 ? 16 : sh.slabs >= 16 ? 4 : 1;
  hipLaunchKernelGGL(net::k_sum_slabs, dim3(net_blocks(n, 64)), dim3(64, rows), 0, s, slabs,
                     sh.slabs, n, grad + ly.w_off);
}

// Loss (mean squared error against target, FP32 site-major) and its
// gradient with respect to every parameter (grad, FP32, overwritten).
void net_gradient(const NetPlan& P, const float* params, const float* input, const float* target,
                  float* grad, void* ws, hipStream_t s) {
  const int L = P.cfg.levels;
  float* out = wsp<float>(ws, P.out);
  net_forward(P, params, input, out, ws, s);
  const NetLayer& lo = P.layers.back();
  hipLaunchKernelGGL(net::k_mse, dim3(kMsePartials), dim3(256), 0, s, out, target, lo.cout,
                     lo.cout_pad, P.nvox[0], wsp<uint16_t>(ws, P.dyp[0]), wsp<double>(ws, P.partials));
  hipLaunchKernelGGL(net::k_sum_partials, dim3(1), dim3(256), 0, s, wsp<double>(ws, P.partials),
                     kMsePartials, 1.0 / ((double)lo.cout * (double)P.nvox[0]),
                     wsp<double>(ws, P.loss));
  const std::vector<net::ConvIn> in = net_inputs(P, ws);
  const std::vector<size_t> outs = net_outputs(P);
  // dy is the BF16 gradient before the activation of the layer at hand; every
  // step leaves the next one's in the other buffer
  uint16_t* dy = wsp<uint16_t>(ws, P.dyp[0]);
  uint16_t* next = wsp<uint16_t>(ws, P.dyp[1]);
  float* gdx = wsp<float>(ws, P.gdx);
  const float slope = P.cfg.slope;
  // layer j: its weight gradient, then dy of layer `before` whose output it read
  auto through = [&](size_t j, size_t before) {
    net_conv_dw(P, P.layers[j], in[j], ws, dy, grad, s);
    net_conv_dx_leaky(P, P.layers[j], ws, dy, outs[before], next, s);
    std::swap(dy, next);
  };
  const size_t jo = P.layers.size() - 1;
  through(jo, jo - 1);
  for (int l = 0; l <= L - 2; ++l) {
    const size_t jb = jo - 1 - 2 * (size_t)l, ja = jb - 1;
    through(jb, ja);
    const int ca = P.c(l + 1);
    net_conv_dw(P, P.layers[ja], in[ja], ws, dy, grad, s);
    net_conv_dx_split(P, P.layers[ja], ws, dy, ca, gdx, wsp<float>(ws, P.ge[l]), s);
    // the upsampled tensor is the output of the layer before (d_{l+1} or e_{L-1})
    hipLaunchKernelGGL(net::k_up2_bwd_leaky, dim3(net_blocks(P.nvox[l + 1] * (ca / 4), 256)),
                       dim3(256), 0, s, gdx, wsp<uint16_t>(ws, outs[ja - 1]), next, P.nz[l], P.ny[l],
                       P.nx[l], ca, slope);
    std::swap(dy, next);
  }
  for (int l = L - 1; l >= 0; --l) {
    const size_t jb = 2 * (size_t)l + 1, ja = jb - 1;
    through(jb, ja);
    net_conv_dw(P, P.layers[ja], in[ja], ws, dy, grad, s);
    if (l > 0) {
      const int C = P.c(l - 1);
      net_conv_dx_split(P, P.layers[ja], ws, dy, C, gdx, nullptr, s);
      hipLaunchKernelGGL(net::k_pool2_bwd_leaky, dim3(net_blocks(P.nvox[l - 1] * (C / 4), 256)),
                         dim3(256), 0, s, gdx, wsp<float>(ws, P.ge[l - 1]),
                         wsp<uint16_t>(ws, outs[jb - 2]), next, P.nz[l - 1], P.ny[l - 1],
                         P.nx[l - 1], C, slope);
      std::swap(dy, next);
    }
  }
}
