// Host runtime of the packed-MLP library: argument checking, hyperparameter
// sampling, the packed layout planner, initial parameters, workspace binding,
// launch sequencing of the training step / evaluation / greedy selection, and
// the C ABI declared in include/tabpack.h.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/tabpack.h"
#include "pack_internal.h"
#include "philox.h"

using namespace tabpack;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIP_TRY(expr)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) return fail(PACK_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

constexpr uint32_t kTagHparam = 1, kTagInit = 2;
// Evaluation and prediction take their rows in chunks of eval_rows() of the
// levels 0 .. eval_levels - 1 (each a quarter of the one before).
constexpr int kEvalLevels = PACK_EVAL_LEVELS;
constexpr int kGroups = 4;  // at most this many member groups run their GEMM chains concurrently

int64_t round_up(int64_t x, int64_t q) { return (x + q - 1) / q * q; }
int64_t mini_tiles(int M, int N) { return (int64_t)((M + kMiniTile - 1) / kMiniTile) * ((N + kMiniTile - 1) / kMiniTile); }
int64_t small_tiles(int M, int N) { return (int64_t)((M + kSmallTile - 1) / kSmallTile) * ((N + kSmallTile - 1) / kSmallTile); }

struct Key {
  uint32_t k0, k1;
};
Key stream_key(uint64_t seed, uint32_t tag) {
  return Key{(uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32) ^ (tag << 28)};
}

// Double in [0, 1) with 53 random bits from two 32-bit words.
double u53(uint32_t a, uint32_t b) {
  return ((double)(a >> 5) * 67108864.0 + (double)(b >> 6)) * (1.0 / 9007199254740992.0);
}

double log_uniform(double lo, double hi, double u) {
  if (lo == hi) return lo;
  return std::exp(std::log(lo) + u * (std::log(hi) - std::log(lo)));
}

struct Member {
  int width, dp;
  int depth;  // hidden Linear-ReLU-Dropout blocks, 1 .. L
  double dropout, lr, wd, scale;
  double muon_lr = 0.0;  // Muon learning rate of the hidden weights (Muon packs)
  int d_emb = 0;         // periodic embedding size per feature (0: the features feed W_1 directly)
  double sigma = 0.0;    // standard deviation of the embedding frequencies' initial values
  int p_in = 0;          // columns of W_1 and of the first layer's input (padded d_in * d_emb, or Pin)
  int64_t eoff[4] = {};  // embedding parameters w, b, alpha, beta (offsets in theta)
  int64_t h0_off = 0;    // the member's first-layer input block (elements of the H_0 / E buffer)
  int64_t etab_off = 0;  // the member's embedding column table (entries of the table buffer)
  uint32_t t;
  std::vector<int64_t> toff;  // packed offsets of W_1, b_1, ..., W_depth, b_depth, W_out, b_out
  int64_t act_off;
};

struct Launch {
  int desc0, ndesc;
  int tile0, ntiles;
  double flops;  // algorithmic flops of the launch (true member shapes)
  double bytes;  // algorithmic HBM bytes: operands read once, outputs written once
  TileSet ts = TILES_SMALL;  // tile set of its tiles (set by add_tiles / add_tiles_sym)
};

// One timed launch: events recorded on the launch stream around it.
struct TimedLaunch {
  int group;
  hipEvent_t start, stop;
};

struct ProfGroup {
  std::string name;
  int kind;
  int launches = 0;
  double total_ms = 0.0, flops = 0.0, bytes = 0.0;
};

}  // namespace

// Device buffers carved out of the caller's workspace.
struct Bufs {
  float *theta = nullptr, *grad = nullptr, *m = nullptr, *v = nullptr;
  uint16_t* shadow = nullptr;
  char* H0 = nullptr;  // first-layer inputs: gathered batches [Bp, Pin], or embedded batches E [Bp, p_in], per member
  float4* etab = nullptr;  // embeddings: the members' column tables (MemberDev::e_tab), rebuilt every step
  float* dE = nullptr; // embeddings: at each member's E offset / 16, the dE GEMM's sums [Bp / 64][4][p_in] (fp32)
  char* H = nullptr;   // L activation buffers H_1..H_L
  char* dz = nullptr;  // ndz() buffers for dZ_1..dZ_L
  float* colpart = nullptr;  // bias-gradient partials of the dX epilogues, (L - 1) x A / kPartRows floats
  uint32_t* mask = nullptr;  // ReLU/dropout keep bits of H_1..H_L, L * A / 32 words
  uint32_t* keepw = nullptr; // dropout keep words, 2 copies of L * A / 32 words
  char* zeros = nullptr;     // 256 zero bytes: GEMM loads of out-of-range elements read them
  float *dY = nullptr, *rowloss = nullptr;
  MemberDev* d_mem = nullptr;
  int64_t* d_bias_off = nullptr;  // [L][K] offsets of b_l
  GemmDesc* d_descs = nullptr;
  Tile* d_tiles = nullptr;
  size_t tile_cap = 0;  // entries of d_tiles
  ColTile* d_coltiles = nullptr;
  HeadTile* d_headtiles = nullptr;
  int32_t* d_members = nullptr;
  int32_t* d_active = nullptr;  // active member ids, increasing
  // Muon scratch: two X buffers, A, B' (GEMM precision), tile partial norms,
  // inverse norms and the matrix / tile tables
  char* mX[2] = {nullptr, nullptr};
  char* mA = nullptr;
  char* mB = nullptr;
  double* mpart = nullptr;
  float* minv = nullptr;
  MuonMat* d_mmats = nullptr;
  MuonTile* d_mtiles = nullptr;
  int32_t* d_mtile0 = nullptr;
  float* headpart = nullptr;  // head backward partials, (Bp / RB) * (d_out + 1) * A / Bp floats
  uint32_t* status = nullptr; // asynchronous error flags (pack_status)
};

struct pack_handle {
  pack_config cfg;
  Prec prec;
  Task task;
  int q, Bp, Pin;
  // pack_bind_data: the first layer's forward and weight-gradient GEMMs read
  // the batch rows straight from a bf16 copy of X (xb, data_N rows of Pin)
  // through the batch indices; no H_0 is gathered
  bool stream_rows = false;
  const float* data_X = nullptr;
  int64_t data_N = 0;
  void* xb = nullptr;
  std::vector<Member> mem;
  int64_t P = 0;     // packed parameter count (multiple of kChunk)
  int64_t A = 0;     // elements of one activation buffer (all members)
  std::vector<float> theta_host;  // host copy of the parameters, packed layout
  // Members in the pack's launches (Section 3.6: a base model that stops
  // improving is removed from the pack); inactive members keep their state.
  std::vector<uint8_t> active;
  std::vector<int32_t> active_ids;   // increasing
  bool muon = false;                 // hidden weights on Muon (pack_config.optimizer)
  bool emb = false;                  // periodic feature embeddings (pack_config.emb_lo > 0)
  Launch de[kGroups]{};
  int ns_steps = 5;
  int n_mmats = 0, n_mtiles = 0;     // Muon matrices and tiles of the active members
  // per member group g: matrices [mmat0[g], mmat0[g+1]), tiles [mtileg[g], mtileg[g+1])
  int mmat0[kGroups + 1]{}, mtileg[kGroups + 1]{};
  Launch nsA[2][kGroups]{}, nsB[kGroups]{}, nsX[2][kGroups]{};

  bool bound = false;
  Bufs b;
  // per layer (index l-1); the forward launches exist once per keep-word
  // buffer: the dropout keep words alternate between two copies by step
  // parity, so the next step's are produced while this step's backward runs
  std::vector<Launch> fwd[2][kGroups], dx[kGroups], dw[kGroups];  // [keep-word parity][group] / [group]
  // evaluation and prediction: one launch a layer over all active members, per
  // chunk level; chunks of level i hold Bp << eval_shift >> 2 i rows
  std::vector<Launch> ev[kEvalLevels];
  int eval_shift = 0, eval_levels = 1;
  int64_t eval_cap = 0;  // rows of a chunk that the GEMM loaders reach (kOperandBytes)
  // the last forward pass: rows of its activation blocks (Bp, or an evaluation
  // chunk's), and how many of them it computed
  int last_rows = 0, last_valid = 0;
  // The members are split into ngroups groups of about equal GEMM work; each
  // group's GEMM chain runs on its own stream (group 0 on the caller's), which
  // measured faster than one launch over all members.
  int ngroups = 1;
  // Small packs (small_pack, but not muon_split) run the whole step on the
  // caller's stream, with one weight-gradient launch for all layers: such a step
  // is bound by its launches and events, not by what runs side by side.
  bool one_stream = false;
  Launch dw_all{};                   // one_stream and small: the weight gradients of all layers (embedded packs: 2..L)
  // a small pack with all its members active: the training head in one kernel,
  // and a gradient buffer for every layer (decided once, whoever is active)
  bool small = false;
  // dZ_l buffers: one a layer, so that all weight gradients can follow the dX
  // chain, or two in turn
  int ndz() const { return small ? cfg.L : 2; }
  std::vector<int> group[kGroups];
  int sumtile0[kGroups + 1] = {};    // gradient-sum work items of group g: [sumtile0[g], sumtile0[g + 1])
  int headtile0[kGroups + 1] = {};   // head-backward tiles of group g
  int member0[kGroups + 1] = {};     // group g's members: d_members[member0[g] .. member0[g+1])
  hipStream_t gstream[kGroups] = {};  // streams of groups 1.. (entry 0 unused)
  hipEvent_t ev_split = nullptr, ev_merge[kGroups] = {};
  hipEvent_t ev_gather[kGroups] = {};  // group g's gather done (group g + 1 gathers after it)
  hipEvent_t ev_bias[kGroups] = {};    // group g's last backward producer done (its gradient sums follow)
  int ncoltiles = 0;
  int nheadtiles = 0;
  int head_rb = 0;  // rows per head-backward block
  uint64_t t = 0;
  // tile sets of the forward, data- and weight-gradient GEMMs: -1 chooses per
  // launch (launch_tiles), else a fixed TileSet
  int tiles_fwd = -1, tiles_dx = -1, tiles_dw = -1;
  int ns_tiles = -1;  // tile set of the Newton-Schulz GEMMs: -1 chooses per launch, else a fixed TileSet
  TileSet emb_tiles = TILES_SMALL;  // tile set of the embedded first layer's forward (training and evaluation)
  bool muon_fused = true;  // the Muon update in the last Newton-Schulz GEMM's epilogue
  // side stream for ALU-bound work that overlaps memory-bound kernels of the
  // caller's stream, joined back through events (created by pack_bind)
  hipStream_t side = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  hipEvent_t ev_keep[2] = {nullptr, nullptr};  // keep words of the step with that parity are ready
  uint64_t keep_ready = 0;                     // step whose keep words are (being) produced ahead

  // optional per-kernel timing
  bool prof = false;
  std::vector<TimedLaunch> timed;
  std::vector<hipEvent_t> event_pool;
  size_t pool_used = 0;
  std::vector<ProfGroup> groups;

  size_t elt() const { return prec == Prec::BF16 ? 2 : 4; }
  int eval_rows(int level) const { return (int)(((int64_t)Bp << eval_shift) >> (2 * level)); }
  int64_t H0e = 0;  // elements of the H_0 / E buffer (every member's first-layer input block)
  int64_t Etab = 0; // entries of the embedding column tables (p_in per embedded member)
};

namespace {

int validate(const pack_config* c) {
  if (!c) return fail(PACK_EINVAL, "cfg is NULL");
  if (c->K < 1 || c->K > 65535) return fail(PACK_EINVAL, "K=%d out of [1, 65535]", c->K);
  if (c->d_in < 1 || c->d_in > (1 << 20)) return fail(PACK_EINVAL, "d_in=%d out of range", c->d_in);
  if (c->L < 1 || c->L > 8) return fail(PACK_EINVAL, "L=%d out of [1, 8]", c->L);
  if (!(c->depth_lo == 0 && c->depth_hi == 0) && !(1 <= c->depth_lo && c->depth_lo <= c->depth_hi && c->depth_hi <= c->L))
    return fail(PACK_EINVAL, "depth range [%d, %d] must lie in [1, L=%d] (0, 0: every member has L blocks)",
                c->depth_lo, c->depth_hi, c->L);
  if (c->B < 1 || c->B > 65536) return fail(PACK_EINVAL, "B=%d out of [1, 65536]", c->B);
  if (c->task < 0 || c->task > 2) return fail(PACK_EINVAL, "unknown task %d", c->task);
  if (c->precision != PACK_PREC_BF16 && c->precision != PACK_PREC_FP32)
    return fail(PACK_EINVAL, "unknown precision %d", c->precision);
  if (c->task == PACK_TASK_MULTI_CE) {
    if (c->d_out < 2 || c->d_out > kMaxOut) return fail(PACK_EINVAL, "CE needs 2 <= d_out <= %d", kMaxOut);
  } else if (c->d_out != 1) {
    return fail(PACK_EINVAL, "MSE/BCE tasks need d_out == 1");
  }
  const int q = c->quantum ? c->quantum : 32;
  if (q < 8 || q > 512 || q % 8) return fail(PACK_EINVAL, "quantum %d must be a multiple of 8 in [8, 512]", q);
  if (c->keep_grads != 0 && c->keep_grads != 1) return fail(PACK_EINVAL, "keep_grads must be 0 or 1");
  if (!(c->beta1 >= 0 && c->beta1 < 1 && c->beta2 >= 0 && c->beta2 < 1 && c->eps > 0))
    return fail(PACK_EINVAL, "AdamW constants out of range");
  if (c->emb_lo != 0) {
    if (c->emb_lo < 8 || c->emb_hi < c->emb_lo || c->emb_hi > 32 || c->emb_step < 1 ||
        (c->emb_hi - c->emb_lo) % c->emb_step)
      return fail(PACK_EINVAL, "embedding size range [%d, %d] step %d invalid (8 <= lo <= hi <= 32)", c->emb_lo,
                  c->emb_hi, c->emb_step);
    if (!c->members && !(c->sigma_lo > 0 && c->sigma_hi >= c->sigma_lo))
      return fail(PACK_EINVAL, "embedding sigma range must be positive and ordered");
    if (c->B > kMapRows)
      return fail(PACK_EINVAL, "B=%d: periodic embeddings take batches of at most %d rows", c->B, kMapRows);
  }
  if (c->optimizer != PACK_OPT_ADAMW && c->optimizer != PACK_OPT_MUON)
    return fail(PACK_EINVAL, "unknown optimizer %d", c->optimizer);
  if (c->optimizer == PACK_OPT_MUON) {
    if (c->ns_steps < 0 || c->ns_steps > 16) return fail(PACK_EINVAL, "ns_steps=%d out of [1, 16]", c->ns_steps);
    if (!(c->muon_momentum >= 0 && c->muon_momentum < 1)) return fail(PACK_EINVAL, "Muon momentum out of [0, 1)");
    if (!c->members && !(c->muon_lr_lo > 0 && c->muon_lr_hi >= c->muon_lr_lo))
      return fail(PACK_EINVAL, "Muon learning-rate range must be positive and ordered");
  }
  if (!c->members) {
    if (c->width_lo < 1 || c->width_hi < c->width_lo || c->width_hi > 16384)
      return fail(PACK_EINVAL, "width range [%d, %d] invalid", c->width_lo, c->width_hi);
    if (!(c->dropout_lo >= 0 && c->dropout_hi >= c->dropout_lo && c->dropout_hi < 1))
      return fail(PACK_EINVAL, "dropout range invalid");
    if (!(c->lr_lo > 0 && c->lr_hi >= c->lr_lo) || !(c->wd_lo > 0 && c->wd_hi >= c->wd_lo))
      return fail(PACK_EINVAL, "lr/wd ranges must be positive and ordered");
  }
  return PACK_OK;
}

void sample_members(pack_handle* h) {
  const pack_config& c = h->cfg;
  const Key key = stream_key(c.seed, kTagHparam);
  for (int k = 0; k < c.K; ++k) {
    const Words4 a = philox4x32_10((uint32_t)k, 0, 0, 0, key.k0, key.k1);
    const Words4 b = philox4x32_10((uint32_t)k, 1, 0, 0, key.k0, key.k1);
    Member& m = h->mem[k];
    m.width = c.width_lo + (int)std::floor(u53(a.w0, a.w1) * (double)(c.width_hi - c.width_lo + 1));
    m.dropout = c.dropout_lo + u53(a.w2, a.w3) * (c.dropout_hi - c.dropout_lo);
    m.lr = log_uniform(c.lr_lo, c.lr_hi, u53(b.w0, b.w1));
    m.wd = log_uniform(c.wd_lo, c.wd_hi, u53(b.w2, b.w3));
    m.depth = c.L;
    if (c.depth_lo > 0) {  // depth ~ UniformInt[depth_lo, depth_hi] from block (k, 2, 0, 0)
      const Words4 d = philox4x32_10((uint32_t)k, 2, 0, 0, key.k0, key.k1);
      m.depth = c.depth_lo + (int)std::floor(u53(d.w0, d.w1) * (double)(c.depth_hi - c.depth_lo + 1));
    }
    if (c.optimizer == PACK_OPT_MUON) {  // Muon learning rate from block (k, 3, 0, 0)
      const Words4 d = philox4x32_10((uint32_t)k, 3, 0, 0, key.k0, key.k1);
      m.muon_lr = log_uniform(c.muon_lr_lo, c.muon_lr_hi, u53(d.w0, d.w1));
    }
    if (c.emb_lo > 0) {  // embedding size and sigma from block (k, 4, 0, 0)
      const Words4 d = philox4x32_10((uint32_t)k, 4, 0, 0, key.k0, key.k1);
      m.d_emb = c.emb_lo + c.emb_step * (int)std::floor(u53(d.w0, d.w1) * (double)((c.emb_hi - c.emb_lo) / c.emb_step + 1));
      m.sigma = log_uniform(c.sigma_lo, c.sigma_hi, u53(d.w2, d.w3));
    }
  }
}

// Packed layout: per member, tensors W_1 [dp, Pin], b_1 [dp], W_l [dp, dp],
// b_l [dp], W_out [d_out, dp], b_out [d_out]; every tensor starts on a
// kChunk-element boundary.  Padding rows/columns hold exact zeros forever: their
// inputs or output gradients are zero, so their gradients and AdamW moments
// stay zero.
int emb_dp(int d_emb) { return (d_emb + 7) & ~7; }

void plan_layout(pack_handle* h) {
  const pack_config& c = h->cfg;
  int64_t off = 0, aoff = 0;
  int64_t h0 = 0, tab = 0;
  for (int k = 0; k < c.K; ++k) {
    Member& m = h->mem[k];
    m.dp = (int)round_up(m.width, h->q);
    // embedded: feature i owns columns i dp .. i dp + dp - 1 of W_1 (dp = d_emb
    // rounded up to 8, the last dp - d_emb zero padding), so that every
    // 16-byte chunk of a row the GEMMs produce belongs to one feature
    m.p_in = m.d_emb ? c.d_in * emb_dp(m.d_emb) : h->Pin;
    m.h0_off = h0;
    h0 += (int64_t)h->Bp * m.p_in;
    m.etab_off = tab;
    if (m.d_emb) tab += m.p_in;
    if (m.d_emb) {  // embedding parameters first: w, b [d_in, d_emb-1], alpha, beta [d_in, d_emb] (AdamW)
      const int64_t n[4] = {(int64_t)c.d_in * (m.d_emb - 1), (int64_t)c.d_in * (m.d_emb - 1),
                            (int64_t)c.d_in * m.d_emb, (int64_t)c.d_in * m.d_emb};
      for (int t = 0; t < 4; ++t) {
        m.eoff[t] = off;
        off += round_up(n[t], kChunk);
      }
    }
    m.toff.assign(2 * m.depth + 2, 0);
    for (int l = 0; l <= m.depth; ++l) {
      const int64_t rows = l < m.depth ? m.dp : c.d_out;
      const int64_t cols = l == 0 ? m.p_in : m.dp;
      for (int part = 0; part < 2; ++part) {
        const int64_t n = part == 0 ? rows * cols : rows;
        m.toff[2 * l + part] = off;
        off += round_up(n, kChunk);
      }
    }
    m.act_off = aoff;
    aoff += (int64_t)h->Bp * m.dp;
  }
  h->P = off;
  h->A = aoff;
  h->H0e = h0;
  h->Etab = tab;
}

// Packed column of dense column cc (feature-major i d_emb + j) of W_1.
int64_t w1_col(const Member& m, int64_t cc) {
  return m.d_emb ? (cc / m.d_emb) * emb_dp(m.d_emb) + cc % m.d_emb : cc;
}

// torch.nn.Linear default initialisation, U(-1/sqrt(fan_in), 1/sqrt(fan_in)),
// drawn from the init stream: element e of tensor t of member k uses word
// (e & 3) of block (e >> 2, e >> 34, t, k); u = (word >> 8) * 2^-24.
void init_params(pack_handle* h) {
  const pack_config& c = h->cfg;
  h->theta_host.assign((size_t)h->P, 0.0f);
  const Key key = stream_key(c.seed, kTagInit);
  for (int k = 0; k < c.K; ++k) {
    const Member& m = h->mem[k];
    if (m.d_emb) {
      // embedding frequencies w ~ N(0, sigma) by Box-Muller: element e takes block
      // (e >> 1, 0, 100, k); u1 = ((word0 >> 8) + 1) 2^-24, u2 = (word1 >> 8) 2^-24;
      // cos for even e, sin for odd e.  b, alpha, beta start at zero.
      const int64_t n = (int64_t)c.d_in * (m.d_emb - 1);
      float* dst = h->theta_host.data() + m.eoff[0];
      for (int64_t e = 0; e < n; ++e) {
        const Words4 w = philox4x32_10((uint32_t)(e >> 1), 0, 100, (uint32_t)k, key.k0, key.k1);
        const double u1 = (double)((w.w0 >> 8) + 1) * (1.0 / 16777216.0);
        const double u2 = (double)(w.w1 >> 8) * (1.0 / 16777216.0);
        const double r = std::sqrt(-2.0 * std::log(u1));
        const double z = r * ((e & 1) == 0 ? std::cos(2.0 * M_PI * u2) : std::sin(2.0 * M_PI * u2));
        dst[e] = (float)(m.sigma * z);
      }
    }
    for (int l = 0; l <= m.depth; ++l) {
      const int rows = l < m.depth ? m.width : c.d_out;
      const int fan_in = l == 0 ? (m.d_emb ? c.d_in * m.d_emb : c.d_in) : m.width;
      const int64_t ld = l == 0 ? m.p_in : m.dp;
      const double bound = 1.0 / std::sqrt((double)fan_in);
      for (int part = 0; part < 2; ++part) {
        const uint32_t tid = (uint32_t)(2 * l + part);
        const int64_t n = part == 0 ? (int64_t)rows * fan_in : rows;
        float* dst = h->theta_host.data() + m.toff[2 * l + part];
        Words4 w{};
        for (int64_t e = 0; e < n; ++e) {
          if ((e & 3) == 0 || e == 0)
            w = philox4x32_10((uint32_t)(e >> 2), (uint32_t)(e >> 34), tid, (uint32_t)k, key.k0, key.k1);
          const uint32_t word = (e & 3) == 0 ? w.w0 : (e & 3) == 1 ? w.w1 : (e & 3) == 2 ? w.w2 : w.w3;
          const double u = (double)(word >> 8) * (1.0 / 16777216.0);
          const float val = (float)((2.0 * u - 1.0) * bound);
          if (part == 0)
            dst[(e / fan_in) * ld + (l == 0 ? w1_col(m, e % fan_in) : e % fan_in)] = val;
          else
            dst[e] = val;
        }
      }
    }
  }
}

// Dense <-> packed copies of one member's tensors.
int64_t dense_count(const pack_handle* h, int k) {
  const Member& m = h->mem[k];
  const pack_config& c = h->cfg;
  const int64_t fi = m.d_emb ? (int64_t)c.d_in * m.d_emb : c.d_in;
  const int64_t emb = m.d_emb ? 2 * (int64_t)c.d_in * (2 * m.d_emb - 1) : 0;
  return emb + (int64_t)m.width * fi + m.width + (int64_t)(m.depth - 1) * ((int64_t)m.width * m.width + m.width) +
         (int64_t)c.d_out * m.width + c.d_out;
}

template <typename F>
void for_each_dense(const pack_handle* h, int k, F f) {  // f(dense_index, packed_index)
  const Member& m = h->mem[k];
  const pack_config& c = h->cfg;
  int64_t di = 0;
  if (m.d_emb) {  // embedding parameters first: w, b [d_in, d_emb-1], alpha, beta [d_in, d_emb]
    const int64_t n[4] = {(int64_t)c.d_in * (m.d_emb - 1), (int64_t)c.d_in * (m.d_emb - 1),
                          (int64_t)c.d_in * m.d_emb, (int64_t)c.d_in * m.d_emb};
    for (int t = 0; t < 4; ++t)
      for (int64_t e = 0; e < n[t]; ++e) f(di++, m.eoff[t] + e);
  }
  for (int l = 0; l <= m.depth; ++l) {
    const int rows = l < m.depth ? m.width : c.d_out;
    const int cols = l == 0 ? (m.d_emb ? c.d_in * m.d_emb : c.d_in) : m.width;
    const int64_t ld = l == 0 ? m.p_in : m.dp;
    for (int r = 0; r < rows; ++r)
      for (int cc = 0; cc < cols; ++cc) f(di++, m.toff[2 * l] + (int64_t)r * ld + (l == 0 ? w1_col(m, cc) : cc));
    for (int r = 0; r < rows; ++r) f(di++, m.toff[2 * l + 1] + r);
  }
}

int64_t member_span_begin(const pack_handle* h, int k) {
  return h->mem[k].d_emb ? h->mem[k].eoff[0] : h->mem[k].toff[0];
}
int64_t member_span_end(const pack_handle* h, int k) {
  return k + 1 < h->cfg.K ? member_span_begin(h, k + 1) : h->P;
}

// Device-table sizes.
struct Plan {
  TileSet tile_set = TILES_SMALL;
  bool unsorted = false;  // only the tables' sizes are wanted: sort_launch leaves the tiles as they are
  std::vector<GemmDesc> descs;
  std::vector<Tile> tiles;
  std::vector<int64_t> cost;  // planner's cost of each tile (depth x valid area), as added (before sort_launch)
  std::vector<ColTile> coltiles;
  std::vector<HeadTile> headtiles;
  std::vector<Launch> fwd[2][kGroups], dx[kGroups], dw[kGroups];
  Launch dw_all{};
  std::vector<Launch> ev[kEvalLevels];  // evaluation, per chunk level and layer
  int sumtile0[kGroups + 1] = {};  // see build_plan
  int headtile0[kGroups + 1] = {};
  std::vector<int32_t> members;  // member ids in group order
  int member0[kGroups + 1] = {};
  // Muon: the hidden weights, their 64 x 64 tiles (matrix k owns tiles
  // mtile0[k] .. mtile0[k+1]) and the Newton-Schulz products: A = X X^T and
  // X' = a X + B' X for each parity of the X buffers, B' = b A + c A A
  std::vector<MuonMat> mmats;
  std::vector<MuonTile> mtiles;
  std::vector<int32_t> mtile0;
  int mmat0[kGroups + 1]{}, mtileg[kGroups + 1]{};  // per member group: first matrix, first tile
  Launch nsA[2][kGroups]{}, nsB[kGroups]{}, nsX[2][kGroups]{};
  // embeddings: dE = dZ_1 W_1 per group (the first layer's data gradient,
  // reduced in the epilogue into the embedding-gradient sums)
  Launch de[kGroups]{};
};

// Tiles of one member's M x N output.  Big set: 256 x 256 tiles, except that
// a remainder of at most 128 rows or columns is covered by a strip of small
// 128 x 128 tiles (a larger remainder takes one more, partly filled, big
// tile).  Tall set: 256 x 128 tiles, rows as in the big set, the last column
// tile partly filled.  Small set: 128 x 128 tiles only.  Mini set: 64 x 64
// tiles only.
void add_tiles(Plan& p, Launch& ln, int d, int M, int N, int kdepth) {
  const size_t first = p.tiles.size();
  ln.ts = p.tile_set;
  auto big_end = [&](int E) {
    const int r = E % kBigTile;
    return r == 0 ? E : (r > kSmallTile ? E - r + kBigTile : E - r);
  };
  if (p.tile_set == TILES_WIDE || p.tile_set == TILES_HUGE) {
    // 128 x 256 (huge: 256 x 256) tiles; a last strip of at most 128 columns on 256 x 128 tiles
    const int r = N % kBigTile, Nw = r > 0 && r <= kSmallTile ? N - r : N;
    const bool huge = p.tile_set == TILES_HUGE;
    const int tm = huge ? kBigTile : kSmallTile;
    for (int m0 = 0; m0 < M; m0 += tm)
      for (int n0 = 0; n0 < Nw; n0 += kBigTile) {
        p.tiles.push_back(Tile{d, m0, n0, huge ? kShapeHuge : kShapeWide});
        p.cost.push_back((int64_t)kdepth * std::min(tm, M - m0) * std::min(kBigTile, N - n0));
      }
    if (Nw < N)
      for (int m0 = 0; m0 < M; m0 += kBigTile) {
        p.tiles.push_back(Tile{d, m0, Nw, kShapeTall8});
        p.cost.push_back((int64_t)kdepth * std::min(kBigTile, M - m0) * (N - Nw));
      }
    ln.ntiles = (int)p.tiles.size() - ln.tile0;
    return;
  }
  const bool big = p.tile_set == TILES_BIG, tall = p.tile_set == TILES_TALL;
  const bool mini = p.tile_set == TILES_MINI;
  const int edge = mini ? kMiniTile : kSmallTile;  // the square tiles (all of them, or the edge strips)
  const int Mb = big || tall ? big_end(M) : 0;
  const int Nb = big ? big_end(N) : (tall ? (int)round_up(N, kSmallTile) : 0);
  const int tn = big ? kBigTile : kSmallTile;  // columns of the large tile
  const int large = big ? kShapeBig : kShapeTall;
  auto push = [&](int m0, int n0, int shape) {
    const int tm = shape == kShapeBig || shape == kShapeTall ? kBigTile : edge;
    const int tw = shape == kShapeBig ? kBigTile : edge;
    if (mini) shape = kShapeMini;
    const int mb = std::min(tm, M - m0), nb = std::min(tw, N - n0);
    p.tiles.push_back(Tile{d, m0, n0, shape});
    p.cost.push_back((int64_t)kdepth * std::max(mb, 0) * std::max(nb, 0));
  };
  for (int m0 = 0; m0 < Mb; m0 += kBigTile)
    for (int n0 = 0; n0 < Nb; n0 += tn) push(m0, n0, large);
  for (int m0 = 0; m0 < Mb; m0 += kSmallTile)
    for (int n0 = Nb; n0 < N; n0 += kSmallTile) push(m0, n0, kShapeSmall);
  for (int m0 = Mb; m0 < M; m0 += edge)
    for (int n0 = 0; n0 < N; n0 += edge) push(m0, n0, kShapeSmall);
  // Wider than tall (the embedded first layer's dE = dZ_1 W_1 and dW_1 =
  // dZ_1^T E, thousands of columns): tiles in column-strip order, so the row
  // tiles sharing a strip of the wide operand run together and read it once
  // while the narrow operand stays in L2 (row order re-reads every strip once
  // per row tile).
  if (N > M) {
    std::vector<std::pair<Tile, int64_t>> v;
    for (size_t i = first; i < p.tiles.size(); ++i) v.push_back({p.tiles[i], p.cost[i]});
    std::stable_sort(v.begin(), v.end(), [](const std::pair<Tile, int64_t>& x, const std::pair<Tile, int64_t>& y) {
      return x.first.n0 != y.first.n0 ? x.first.n0 < y.first.n0 : x.first.m0 < y.first.m0;
    });
    for (size_t i = 0; i < v.size(); ++i) {
      p.tiles[first + i] = v[i].first;
      p.cost[first + i] = v[i].second;
    }
  }
  ln.ntiles = (int)p.tiles.size() - ln.tile0;
}

// Launch order of one grouped GEMM.  Workgroup i runs on XCD i % 8, and each
// XCD has its own L2, so all tiles of a member go to one XCD (members are
// packed into the 8 XCD bins longest-first by total cost), and within a bin
// tiles run longest-first so the launch ends on short tiles.
void sort_launch(Plan& p, const Launch& ln) {
  if (p.unsorted || ln.ntiles == 0) return;
  const Tile* tiles = p.tiles.data() + ln.tile0;
  const int64_t* cost = p.cost.data() + ln.tile0;
  int lo = tiles[0].desc, hi = lo;
  for (int i = 1; i < ln.ntiles; ++i) {
    lo = std::min(lo, tiles[i].desc);
    hi = std::max(hi, tiles[i].desc);
  }
  std::vector<int> bin_of(hi - lo + 1, -1);              // the descriptor's entry of member_cost, then its XCD
  std::vector<std::pair<int64_t, int>> member_cost;  // (cost, desc - lo)
  for (int i = 0; i < ln.ntiles; ++i) {
    int& e = bin_of[tiles[i].desc - lo];
    if (e < 0) {
      e = (int)member_cost.size();
      member_cost.push_back({0, tiles[i].desc - lo});
    }
    member_cost[e].first += cost[i];
  }
  std::stable_sort(member_cost.begin(), member_cost.end(),
                   [](const std::pair<int64_t, int>& a, const std::pair<int64_t, int>& b) { return a.first > b.first; });
  std::vector<int64_t> load(kXcds, 0);
  for (const auto& mc : member_cost) {
    const int b = (int)(std::min_element(load.begin(), load.end()) - load.begin());
    load[b] += mc.first;
    bin_of[mc.second] = b;
  }
  std::vector<std::pair<int64_t, int>> bins[kXcds];  // (cost, tile)
  for (int i = 0; i < ln.ntiles; ++i) bins[bin_of[tiles[i].desc - lo]].push_back({cost[i], i});
  auto longer = [](const std::pair<int64_t, int>& a, const std::pair<int64_t, int>& b) { return a.first > b.first; };
  for (auto& b : bins)
    if (!std::is_sorted(b.begin(), b.end(), longer)) std::stable_sort(b.begin(), b.end(), longer);
  std::vector<Tile> out(ln.ntiles);
  size_t next[kXcds] = {};
  for (int i = 0; i < ln.ntiles; ++i) {
    int b = i % kXcds;
    if (next[b] == bins[b].size()) {  // this XCD's bin is empty: take from the fullest remaining
      size_t best = 0;
      for (int c = 0; c < kXcds; ++c)
        if (bins[c].size() - next[c] > best) best = bins[c].size() - next[c], b = c;
    }
    out[i] = tiles[bins[b][next[b]++].second];
  }
  std::copy(out.begin(), out.end(), p.tiles.begin() + ln.tile0);
}

// Whether the given members make a small pack: their activations are at most
// kOneStreamTiles 128 x 128 tiles a layer (two for each CU).  Its step is one
// chain of 3 + 2 L launches (2 + 2 L with bound data, 6 + 2 L with embeddings;
// Muon's products besides) instead of up to 30 launches and as many event
// operations in three streams, which took the host about 150 us.  Measured, two
// groups / one stream: 4 fp32 members of widths 64..256 at batch 256 (16 tiles)
// 200 / 52 us; 16 bf16 members of 128..512 at batch 512 (~180) 200 / 107 us; 41 of
// 159..502 at batch 372 (490) 361 / 286 us; 32 of 256..1024 at batch 1024 (~1,300)
// 639 / 641 us, where side by side the groups' weight-update traffic and matrix
// products overlap.  The size of the first layer does not move the line: 4
// members of width 256 on 16,000 features 261 / 199 us, 64 of 512 on 4,000 (8,192
// weight-gradient tiles) 838 / 795; embedded 8 of 512 on 100 features 206 / 163, 16
// of 512 on 400 at batch 512 656 / 643.  (Muon: muon_split.)
constexpr int64_t kOneStreamTiles = 512;
bool small_pack(const pack_handle* h, const std::vector<int>& ids) {
  int64_t n = 0;
  for (int k : ids) n += small_tiles(h->Bp, h->mem[k].dp);
  return n <= kOneStreamTiles;
}

// Shape of the Newton-Schulz iterate of member m's hidden weight l (1-based):
// padded [R x Cp] storage; X is [S x L], U or U^T (tall: true rows > true columns).
struct MuonShape {
  int R, Cp, S, L, r, c;
  bool tall;
};
MuonShape muon_shape(const pack_handle* h, const Member& m, int l) {
  MuonShape q;
  q.R = m.dp;
  q.Cp = l == 1 ? m.p_in : m.dp;
  q.r = m.width;
  q.c = l == 1 ? (m.d_emb ? h->cfg.d_in * m.d_emb : h->cfg.d_in) : m.width;
  q.tall = q.r > q.c;
  q.S = q.tall ? q.Cp : q.R;
  q.L = q.tall ? q.R : q.Cp;
  return q;
}

// The Newton-Schulz products of the given members in 128 x 128 tiles: the
// symmetric ones (on and above the diagonal) or X' (S x L); *work: tiles times depth.
int64_t ns_small_tiles(const pack_handle* h, const std::vector<int>& ids, bool sym, int64_t* work = nullptr) {
  int64_t n = 0;
  for (int k : ids)
    for (int l = 1; l <= h->mem[k].depth; ++l) {
      const MuonShape q = muon_shape(h, h->mem[k], l);
      const int64_t r = (q.S + kSmallTile - 1) / kSmallTile;
      const int64_t t = sym ? r * (r + 1) / 2 : small_tiles(q.S, q.L);
      n += t;
      if (work) *work += t * (sym ? q.L : q.S);
    }
  return n;
}

// Whether a small pack's Newton-Schulz products are better split over two
// streams than one launch each: X' numbers kMuonSplitX small tiles or more, the
// symmetric ones kMuonSplitSym (fewer: a wide first layer, whose products are
// shallow), and in bf16 X' not so many that the split costs the caches more than
// it overlaps (from kMuonSplitMax on one launch measured up to 30% faster, or the
// same within 4%, but for 3 members of width 4096).  fp32 products run at 1/16 of
// the bf16 rate: they split earlier (into mini tiles) and have no such end.
// Measured at batch 256, one stream / two groups (us; X' and symmetric tiles): bf16
// 8 members of width 1024 (576, 296) 504 / 528; 32 of 512 (640, 352) 422 / 399; 3 of
// 2048 (816, 411) 957 / 1,023; 4 of 2048 (1,088, 548) 1,358 / 1,165; 64 of 512 (1,280,
// 704) 757 / 651; 90 of 128 on 1,500 features (1,080, 90) 393 / 403; 60 of 128 on 3,000
// (1,500, 120) 537 / 569; 40 embedded of 256 (1,200, 160) 554 / 525; 2 of 3072 (1,200,
// 602) 1,937 / 1,663; 2 of 4096 (2,112, 1,058) 3,839 / 3,535; 10 of 2048 (2,720) 2,769 /
// 2,887; 5 of 3072 (3,000) 4,139 / 4,505; 16 of 2048 (4,352) 4,361 / 4,308; 2 of 4096, L 4
// (6,208) 10,961 / 14,297; fp32 3 of 1024 (216, 111) 970 / 1,053; 16 embedded of 256 (320,
// 64) 759 / 818; 4 of 1024 (288, 148) 1,486 / 1,182; 64 of 256 (384, 256) 630 / 514; 2 of
// 2048 (544, 274) 5,185 / 3,897; 16 of 2048 (4,352, 2,192) 24,649 / 24,030.
constexpr int64_t kMuonSplitX = 1024, kMuonSplitXF32 = 256, kMuonSplitSym = 144, kMuonSplitMax = 2560;
bool muon_split(const pack_handle* h, const std::vector<int>& ids) {
  if (!h->muon || ids.size() < 2 || ns_small_tiles(h, ids, true) < kMuonSplitSym) return false;
  const int64_t n = ns_small_tiles(h, ids, false);
  if (h->prec == Prec::FP32) return n >= kMuonSplitXF32;
  return n >= kMuonSplitX && n < kMuonSplitMax;
}

// Members into ngroups groups of about equal GEMM work (longest first, each
// to the lightest group).  Default: 2 groups, 3 with Muon, whose per-group
// Newton-Schulz chains overlap better in three (regression_large: 1.398
// against 1.409 ms per step, Muon 5.33 against 5.39 ms; one group 1.53 ms;
// 4 groups exceed the four hardware queues); small packs one, or two where
// muon_split says so (three: 64 members of width 512 720 us, two 651).
// TABPACK_STREAMS (1 .. 4) overrides it.
void split_members(pack_handle* h) {
  const bool small = small_pack(h, h->active_ids);
  h->one_stream = small && !muon_split(h, h->active_ids);
  int ng = h->one_stream ? 1 : h->muon && !small ? 3 : 2;
  if (const char* e = getenv("TABPACK_STREAMS")) ng = std::max(1, std::min(kGroups, atoi(e)));
  h->ngroups = std::max(1, std::min(ng, (int)h->active_ids.size()));
  h->one_stream = h->one_stream && h->ngroups == 1;
  for (auto& v : h->group) v.clear();
  std::vector<std::pair<double, int>> cost;
  for (int k : h->active_ids) {
    const double w = h->mem[k].dp;
    cost.push_back({w * (h->mem[k].p_in + (h->mem[k].depth - 1) * w), k});
  }
  std::stable_sort(cost.begin(), cost.end(), [](const auto& x, const auto& y) { return x.first > y.first; });
  std::vector<double> load(h->ngroups, 0.0);
  for (const auto& ck : cost) {
    const int g = (int)(std::min_element(load.begin(), load.end()) - load.begin());
    load[g] += ck.first;
    h->group[g].push_back(ck.second);
  }
  for (auto& v : h->group) std::sort(v.begin(), v.end());
}

// The largest first-layer width p_in among the given members.
int max_pin(const pack_handle* h, const std::vector<int>& ids) {
  int m = 0;
  for (int k : ids) m = std::max(m, h->mem[k].p_in);
  return m;
}

// Rows per head-backward block: up to 256, dividing Bp.
int head_rows(const pack_handle* h) { return h->small ? kHeadRows : h->Bp % 256 == 0 ? 256 : h->Bp; }

// Elements of one X buffer and of the A (or B') buffer for the given members.
template <typename It>
void muon_sizes(const pack_handle* h, It begin, It end, int64_t& xe, int64_t& ae) {
  xe = ae = 0;
  for (It it = begin; it != end; ++it) {
    const Member& m = h->mem[*it];
    for (int l = 1; l <= m.depth; ++l) {
      const MuonShape q = muon_shape(h, m, l);
      xe += round_up((int64_t)q.S * q.L, kChunk);
      ae += round_up((int64_t)q.S * q.S, kChunk);
    }
  }
}

// Tiles on and above the diagonal of a symmetric S x S result (the others are
// written as mirror images by the tiles above the diagonal).  Rows go in
// blocks as in add_tiles; within its row block a diagonal block takes small
// tiles on and above its own diagonal, and the columns right of it take the
// tile set's large tiles (a remainder of at most 128 columns small ones).
void add_tiles_sym(Plan& p, Launch& ln, int d, int S, int kdepth) {
  ln.ts = p.tile_set;
  auto push = [&](int m0, int n0, int shape) {
    const int tm = shape == kShapeSmall ? kSmallTile : kBigTile;
    const int tw = shape == kShapeBig ? kBigTile : kSmallTile;
    const int mb = std::min(tm, S - m0), nb = std::min(tw, S - n0);
    p.tiles.push_back(Tile{d, m0, n0, shape});
    // a tile above the diagonal also stores its mirror image
    p.cost.push_back((int64_t)kdepth * mb * nb * (m0 < n0 ? 2 : 1));
  };
  if (p.tile_set == TILES_SMALL) {
    for (int m0 = 0; m0 < S; m0 += kSmallTile)
      for (int n0 = m0; n0 < S; n0 += kSmallTile) push(m0, n0, kShapeSmall);
  } else if (p.tile_set == TILES_MINI) {
    for (int m0 = 0; m0 < S; m0 += kMiniTile)
      for (int n0 = m0; n0 < S; n0 += kMiniTile) {
        p.tiles.push_back(Tile{d, m0, n0, kShapeMini});
        p.cost.push_back((int64_t)kdepth * std::min(kMiniTile, S - m0) * std::min(kMiniTile, S - n0) *
                         (m0 < n0 ? 2 : 1));
      }
  } else {
    const bool big = p.tile_set == TILES_BIG;
    const int large = big ? kShapeBig : kShapeTall, tn = big ? kBigTile : kSmallTile;
    const int r = S % kBigTile;
    const int Mb = r == 0 ? S : (r > kSmallTile ? S - r + kBigTile : S - r);
    for (int m0 = 0; m0 < Mb; m0 += kBigTile) {
      const int e = std::min(m0 + kBigTile, S);  // end of the diagonal block
      for (int i0 = m0; i0 < e; i0 += kSmallTile)
        for (int n0 = i0; n0 < e; n0 += kSmallTile) push(i0, n0, kShapeSmall);
      const int rc = (S - e) % tn;
      const int Nb = big ? (rc == 0 || rc > kSmallTile ? S : S - rc) : S;
      for (int n0 = e; n0 < Nb; n0 += tn) push(m0, n0, large);
      for (int i0 = m0; i0 < e; i0 += kSmallTile)
        for (int n0 = Nb; n0 < S; n0 += kSmallTile) push(i0, n0, kShapeSmall);
    }
    for (int m0 = Mb; m0 < S; m0 += kSmallTile)
      for (int n0 = m0; n0 < S; n0 += kSmallTile) push(m0, n0, kShapeSmall);
  }
  ln.ntiles = (int)p.tiles.size() - ln.tile0;
}

// Tile set of one forward / data-gradient / weight-gradient launch by its
// 128 x 128 tiles: fixed by `forced` (>= 0), mini or huge tiles by the rules below,
// else 256 x 128 tiles when there are at least kTallMinTiles small ones (two full rounds of tall
// tiles at two workgroups per CU), small tiles otherwise.  Measured (ms per
// step, all small / all tall / chosen): 64 members of widths 64..2048 at batch
// 2048 (launches of 700..2800 small tiles) 6.29 / 5.76; 64 of widths
// 256..1024 at batch 1024 (500..840) 1.45 / 1.53 (tall dW alone 1.53);
// 32 of 256..1024 (~440) 0.63 / 0.67.
// Weight-gradient launches also need a depth (padded batch) of at least
// kTallMinDepthDw: their small tiles stream the fused optimizer over the whole
// staged gradient tile, which the tall tiles do not, and at a 1024-row batch
// that epilogue outweighs the tall tiles' faster main loop (the embedded first
// layer's dW: 7.05 ms small, 7.99 ms tall), at 2048 rows it does not
// (widths 64..2048: 6.29 -> 6.09 ms per step with tall dW tiles alone).
constexpr int kTallMinTiles = 1024, kTallMinDepthDw = 2048;
// Mini tiles below kMiniMaxTiles small ones (one for each CU): such a launch
// leaves CUs idle, and four times the workgroups share its depth chains (fp32
// ones above all, whose MFMAs run at 1/16 of the bf16 rate).  Measured, small /
// mini: a prediction of 37 rows by 16 members of widths 128..512 (48 small
// tiles a layer) 56 / 46 us; an fp32 step of 9 members of widths 33..301 at
// batch 300 (at most 45) 464 / 265 us.  In bf16 with several groups, whose launches
// run side by side, all groups' launches of the layer together must also have fewer
// than kMiniSide mini tiles (narrow members fill them better than small ones), in
// packs of one block, whose groups reach them at the same time, than kMiniSideL1
// (two a CU).  (Not the weight gradients of deeper packs at batches of at most kMiniSideRows rows:
// they are short, and mini tiles were never slower.)
// Measured, small / mini weight gradients of two groups (small tiles of both, us a
// step): 10 members of widths 53..211 at batch 4806 (28, 22, 22) 361 / 261; 17 of 114..456
// at batch 1411 (48, 154, 154) 259 / 220; 29 of 106..423 at batch 1080 (73, 207, 207, 207)
// 314 / 275; 66 of width 185 at batch 7287 (264, 594 mini ones) 1,239 / 1,118; 26 of 378
// (234, 936) 736 / 728; 9 of 338..1350 at batch 1831 (330, 391, 391) 441 / 495; 17 of
// 274..1096 at batch 4960 (102, 341, 268) 839 / 908; one block: 20 of 36..142 at batch 7750
// (24) 237 / 214, 108 of 83..329 (235, about 780) 178 / 185, 22 of 159..634 (308) 481 /
// 538; short batches: 56 of 104..415 at batch 916 (420, 384, 384, 384) 455 / 438, 122 of 161 at batch 333 (488)
// 270 / 256.
constexpr int kMiniMaxTiles = 256, kMiniSide = 896, kMiniSideL1 = 512, kMiniSideRows = 1024;
// Huge tiles for forward (and evaluation) launches from kHugeFwd.tiles small ones
// on and data-gradient launches from kHugeDx.tiles on.  Measured, small / tall /
// huge forward launches: 1,000 rows by 16 of 32 members of widths 256..1024 (700
// small tiles a launch) 146 / 141 / 137 us, by all 32 (1,400) 205 / 220 / 198;
// a step of 32 such members (700) 644 / 634 / 632 us, of 24 (525) 504 / 512 /
// 511; tall / huge: evaluation of 64 members (5,400) 22.3 / 21.4 ms.  Data
// gradients, steps with tall / huge ones: widths 64..2048 at batch 2048 (4,350)
// 6.26 / 6.13 ms, 256..1024 at batch 1024 (1,350) 1.265 / 1.284 ms.
// Evaluation chunks of fewer rows than one huge tile keep the smaller tiles
// (huge / tall, us): 37 rows by 64 members of width 2048 (chunks of 64 rows, 1,024
// tiles) 189 / 176, 100 rows (of 128) 242 / 222, by 200 of width 512 165 / 149.
// Shallow launches leave them nothing to cover the tile's start and end with
// (one workgroup a CU): below a mean depth of kHuge*.depth they cost time.  small
// or tall / huge forward launches of two groups (us a step; depth a layer): 108
// members of width 329, one layer (104) 178 / 198; 27 of 192 at batch 6467 (16, 148) 391 /
// 423; 26 of 378 (200, 384, 384, 384) 736 / 769; 17 of 373 (320, 284, 284) 587 / 620; 30 of
// 505 (616, 512, 512) 1,033 / 1,003; 15 of 1154 (128, 853, 853) 655 / 639; 11 of 1909 (424,
// 1,388, ..) 2,465 / 2,369; huge data gradients 77 of 362 (264) 1,772 / 1,841; 116 of 625
// (640) 1,624 / 1,669; 18 of 1222 (1,248) 2,283 / 2,080.  Against small tiles (fewer than
// kTallMinTiles) of two members or more an XCD, which even them out, half that depth will
// do: 32 members of widths 256..1024 on 256 features 563 / 557, 64 of 128..512 on 300 427 /
// 421; against tall ones 64 of 256..1024 on 256 1,170 / 1,180.  Evaluation, whose one
// launch a layer runs alone, gains from them down to a depth of about 192 (us, tall below
// a depth of 64 / 192 / 512): 100 members of widths 100..200 on 20,000 rows 1,533 / 1,455 /
// 1,456; 40 of 300..700 on 128 features 1,431 / 1,382 / 1,383; 16 of 150..300 341 / 340 / 355;
// 8 of 256..512 on 200 333 / 332 / 354; 30 of 100..400 on 2,000 rows 137 / 137 / 148; but 128 of
// 100..384 on 300 2,763 / 2,762 / 2,501.
struct HugeMin {
  int tiles = 0, depth = 0;  // least small tiles and tile-weighted mean depth of a launch (tiles 0: never)
};
constexpr HugeMin kHugeFwd{640, 512}, kHugeDx{2048, 768}, kHugeEval{640, 192};
// The output tiles of a launch, or of the launches of all member groups.
struct LaunchSize {
  int64_t small = 0, mini = 0, work = 0, members = 0;  // work: small tiles times depth
  void add(int M, int N, int depth) {
    small += small_tiles(M, N);
    mini += mini_tiles(M, N);
    work += small_tiles(M, N) * depth;
    ++members;
  }
};
// own: the launch; side: it and those of the other groups, which run beside it.
TileSet launch_tiles(const pack_handle* h, int forced, const LaunchSize& own, const LaunchSize& side, HugeMin huge = {},
                     int min_depth = 0) {
  if (forced >= 0) return (TileSet)forced;
  const bool one_block = h->cfg.L == 1;
  const bool beside = h->prec == Prec::BF16 && h->ngroups > 1;
  if (own.small < kMiniMaxTiles && (!beside || side.mini < (one_block ? kMiniSideL1 : kMiniSide))) return TILES_MINI;
  if (h->prec != Prec::BF16 || h->Bp < min_depth) return TILES_SMALL;
  const bool tall = own.small >= kTallMinTiles;
  const int depth = tall || own.members < 2 * kXcds ? huge.depth : huge.depth / 2;
  if (huge.tiles > 0 && own.small >= huge.tiles && own.work >= own.small * depth) return TILES_HUGE;
  return tall ? TILES_TALL : TILES_SMALL;
}

// Rows of an evaluation chunk: the training batch's padded rows times a power
// of two, up to kEvalTiles 128 x 128 activation tiles a layer and kEvalRows
// rows (the activation buffers grow with it), and quarters of that down to 64
// rows for short inputs and last chunks.  A chunk of Bp rows leaves the CUs
// idle at the ends of a layer's launch, and a call waits for launches in
// proportion to its chunks.  Measured, chunks of Bp rows with a launch per
// member group / these chunks: 64 members of widths 256..1024 on 70,000 rows
// 26.1 / 21.6 ms, 32 of them on 20,000 rows 4.56 / 3.38 ms, 16 members of
// 128..512 on 37 rows 39.9 / 28.6 us (chunks of 512 rows, of 128).
// Wide inputs bound the growth too: the gathered rows H_0 are one GEMM operand,
// which must stay below kOperandBytes (a smaller bound costs requests that then
// fall into a chunk four times their rows, planned for other tiles: 256 MiB took
// 1,100 rows of 16,000 fp32 features from 629 to 1,260 us).  Where even a chunk of
// Bp rows holds a larger operand, a chunk takes the rows below the limit
// (eval_cap).
constexpr int64_t kEvalTiles = 8192, kEvalRows = 8192;
void plan_eval(pack_handle* h) {
  int64_t n = 0, row = h->emb ? 0 : h->Pin;
  for (const Member& m : h->mem) {
    n += small_tiles(h->Bp, m.dp);
    row = std::max(row, (int64_t)m.dp);
  }
  const int64_t in_row = h->emb ? 0 : h->Pin * (int64_t)h->elt();
  h->eval_cap = kOperandBytes / (row * (int64_t)h->elt());
  h->eval_shift = 0;
  auto fits = [&](int shift) {
    const int64_t rows = (int64_t)h->Bp << shift;
    return n << shift <= kEvalTiles && rows <= kEvalRows && rows * in_row <= kOperandBytes;
  };
  while (fits(h->eval_shift + 1)) ++h->eval_shift;
  h->eval_levels = 1;
  while (h->eval_levels < kEvalLevels && h->eval_rows(h->eval_levels) >= 64 && h->eval_rows(h->eval_levels) % 32 == 0)
    ++h->eval_levels;
}

// Tile set of the Newton-Schulz products of a step, the symmetric ones (A, B') or
// X': mini tiles where a launch has fewer than kMiniMaxTiles small ones -- with
// several groups in bf16, whose launches run side by side and fill the CUs
// together, only where all of them have fewer than kSideTiles or their work
// (tiles times depth) is below kSideSym / kSideX.  Measured, products of all groups small / sym mini / both mini
// (us a step, three groups; sym tiles and thousands of work, X' work): 16 members of
// width 512 at batch 2048 (176, 92; 135) 494 / 412 / 406; 32 of 512 (352, 180; 270) 548 /
// 512 / 538; 6 of 1024 (222, 227; 396) 780 / 706 / 728; 8 of 1024 (296, 303; 528) 720 / 707
// / 751; 64 of 512 (704, 360; 541) 707 / 737 / 794; 12 of 1024 (444, 454; 793) 835 / 881 /
// 970; 4 of 2048 (548, 1,122; 2,102) 1,347 / 1,715 / 1,919; in two groups 16 of 512 on 2,000
// features (320, 402) 705 / 644.  fp32 products, at 1/16 of the rate, gain from them at any
// depth: 3 of 2048 (sym 137, X' 272 tiles a group) 7,805 / 7,559 / 7,705, 4 of 1024 (148, 288
// in all) 3,080 / 2,451 / 2,148.
constexpr int64_t kSideTiles = 400, kSideSym = 256 << 10, kSideX = 176 << 10;
TileSet ns_tiles(const pack_handle* h, const std::vector<int> (&group)[kGroups], bool sym, bool sizing) {
  if (h->ns_tiles >= 0) return (TileSet)h->ns_tiles;
  if (sizing) return TILES_SMALL;
  int64_t most = 0, all = 0, work = 0;
  int groups = 0;
  for (const std::vector<int>& g : group) {
    groups += !g.empty();
    const int64_t n = ns_small_tiles(h, g, sym, &work);
    most = std::max(most, n);
    all += n;
  }
  if (most >= kMiniMaxTiles) return TILES_SMALL;
  const bool full = groups > 1 && h->prec == Prec::BF16 && all >= kSideTiles;
  return full && work >= (sym ? kSideSym : kSideX) ? TILES_SMALL : TILES_MINI;
}

void plan_muon(const pack_handle* h, const Bufs& bf, const std::vector<int> (&group)[kGroups], Plan& p,
               bool sizing) {
  const size_t es = h->elt();
  const TileSet saved = p.tile_set;
  const TileSet sym_set = ns_tiles(h, group, true, sizing), x_set = ns_tiles(h, group, false, sizing);
  int64_t xo = 0, ao = 0;
  struct Item {
    MuonShape q;
    int64_t xoff, aoff;
    int mi;  // its MuonMat in p.mmats
  };
  auto xp = [&](int par, int64_t off) { return (void*)(bf.mX[par] + (size_t)off * es); };
  auto ap = [&](const char* base, int64_t off) { return (void*)(base + (size_t)off * es); };
  p.mtile0.push_back(0);
  for (int hf = 0; hf < kGroups; ++hf) {
    p.mmat0[hf] = (int)p.mmats.size();
    p.mtileg[hf] = (int)p.mtiles.size();
    std::vector<Item> items;
    for (int k : group[hf]) {
      const Member& m = h->mem[k];
      for (int l = 1; l <= m.depth; ++l) {
        const MuonShape q = muon_shape(h, m, l);
        MuonMat mm{};
        mm.woff = m.toff[2 * (l - 1)];
        mm.xoff = xo;
        mm.aoff = ao;
        mm.R = q.R;
        mm.Cp = q.Cp;
        mm.tall = q.tall ? 1 : 0;
        mm.member = k;
        mm.decay = (float)(1.0 - m.muon_lr * m.wd);
        mm.step = (float)(m.muon_lr * std::sqrt(std::max(1.0, (double)q.r / q.c)));
        const int mi = (int)p.mmats.size();
        p.mmats.push_back(mm);
        for (int r0 = 0; r0 < q.R; r0 += 64)
          for (int c0 = 0; c0 < q.Cp; c0 += 64) p.mtiles.push_back(MuonTile{mi, r0, c0, 0});
        p.mtile0.push_back((int32_t)p.mtiles.size());
        items.push_back(Item{q, xo, ao, mi});
        xo += round_up((int64_t)q.S * q.L, kChunk);
        ao += round_up((int64_t)q.S * q.S, kChunk);
      }
    }
    p.tile_set = sym_set;
    // A = X X^T, one launch per parity of the X buffer it reads
    for (int par = 0; par < 2; ++par) {
      Launch& ln = p.nsA[par][hf];
      ln = Launch{(int)p.descs.size(), 0, (int)p.tiles.size(), 0, 0.0, 0.0};
      for (const Item& it : items) {
        GemmDesc d{};
        d.A = d.B = xp(par, it.xoff);
        d.lda = d.ldb = it.q.L;
        d.C = ap(bf.mA, it.aoff);
        d.ldc = it.q.S;
        d.M = d.N = it.q.S;
        d.Kd = it.q.L;
        add_tiles_sym(p, ln, (int)p.descs.size(), it.q.S, d.Kd);
        p.descs.push_back(d);
        ++ln.ndesc;
        const double s = std::min(it.q.r, it.q.c), l = std::max(it.q.r, it.q.c);
        ln.flops += s * (s + 1) * l;  // a symmetric result: the upper triangle
        ln.bytes += es * (s * l + s * s);
      }
      sort_launch(p, ln);
    }
    // B' = b A + c A A: A is stored exactly symmetric (mirrored tiles), so A A =
    // A A^T reads both operands depth-contiguous, and B' is symmetric too
    {
      Launch& ln = p.nsB[hf];
      ln = Launch{(int)p.descs.size(), 0, (int)p.tiles.size(), 0, 0.0, 0.0};
      for (const Item& it : items) {
        GemmDesc d{};
        d.A = d.B = ap(bf.mA, it.aoff);
        d.lda = d.ldb = it.q.S;
        d.C = ap(bf.mB, it.aoff);
        d.ldc = it.q.S;
        d.Y = ap(bf.mA, it.aoff);
        d.ldy = it.q.S;
        d.M = d.N = d.Kd = it.q.S;
        add_tiles_sym(p, ln, (int)p.descs.size(), it.q.S, d.Kd);
        p.descs.push_back(d);
        ++ln.ndesc;
        const double s = std::min(it.q.r, it.q.c);
        ln.flops += s * (s + 1) * s;  // a symmetric result: the upper triangle
        ln.bytes += es * 3.0 * s * s;
      }
      sort_launch(p, ln);
    }
    p.tile_set = x_set;
    // X' = a X + B' X, reading X from buffer par and writing buffer 1 - par
    for (int par = 0; par < 2; ++par) {
      Launch& ln = p.nsX[par][hf];
      ln = Launch{(int)p.descs.size(), 0, (int)p.tiles.size(), 0, 0.0, 0.0};
      for (const Item& it : items) {
        GemmDesc d{};
        d.A = ap(bf.mB, it.aoff);
        d.lda = it.q.S;
        d.B = xp(par, it.xoff);
        d.ldb = it.q.L;
        d.C = xp(par ^ 1, it.xoff);
        d.ldc = it.q.L;
        d.Y = xp(par, it.xoff);
        d.ldy = it.q.L;
        d.M = it.q.S;
        d.N = it.q.L;
        d.Kd = it.q.S;
        // the weight the last iteration updates in its epilogue
        const MuonMat& mm = p.mmats[it.mi];
        d.poff = mm.woff;
        d.ns_tall = mm.tall;
        d.ns_decay = mm.decay;
        d.ns_step = mm.step;
        add_tiles(p, ln, (int)p.descs.size(), d.M, d.N, d.Kd);
        p.descs.push_back(d);
        ++ln.ndesc;
        const double s = std::min(it.q.r, it.q.c), l = std::max(it.q.r, it.q.c);
        ln.flops += 2.0 * s * s * l;
        ln.bytes += es * (s * s + 2.0 * s * l);
      }
      sort_launch(p, ln);
    }
  }
  p.mmat0[kGroups] = (int)p.mmats.size();
  p.mtileg[kGroups] = (int)p.mtiles.size();
  p.tile_set = saved;
}

// Launch tables over the members of `group` (the active members split into
// streams; carve() sizes the workspace with every member in one group).
Plan build_plan(const pack_handle* h, const Bufs& bf, const std::vector<int> (&group)[kGroups],
                bool sizing = false) {
  Plan p;
  p.unsorted = sizing;
  // sizing: small tiles for the main GEMMs (the largest tile count of any choice)
  auto choose = [&](int forced, const LaunchSize& own, const LaunchSize& side, HugeMin huge, int min_depth = 0) {
    return sizing ? TILES_SMALL : launch_tiles(h, forced, own, side, huge, min_depth);
  };
  // choose() for group hf's launch over the members that have layer l, whose products are shape(member, M, N, depth)
  auto choose_layer = [&](int forced, int hf, int l, auto shape, HugeMin huge, int min_depth = 0,
                          bool alone = false) {
    LaunchSize own, side;
    for (int g = 0; g < kGroups; ++g)
      for (int k : group[g]) {
        if (h->mem[k].depth < l) continue;
        int M = 0, N = 0, depth = 0;
        shape(h->mem[k], M, N, depth);
        side.add(M, N, depth);
        if (g == hf) own.add(M, N, depth);
      }
    return choose(forced, own, alone ? LaunchSize{} : side, huge, min_depth);
  };
  const pack_config& c = h->cfg;
  const size_t es = h->elt();
  const void* wsrc = h->prec == Prec::BF16 ? (const void*)bf.shadow : (const void*)bf.theta;
  auto Hl = [&](int l) -> void* { return bf.H + (size_t)(l - 1) * h->A * es; };
  auto dzb = [&](int l) -> void* { return bf.dz + (size_t)((l - 1) % h->ndz()) * h->A * es; };
  auto wptr = [&](int k, int l) -> const void* {  // weight of hidden layer l (1-based) for GEMM reads
    return (const char*)wsrc + (size_t)h->mem[k].toff[2 * (l - 1)] * es;
  };
  auto act = [&](void* base, int k) -> void* { return (char*)base + (size_t)h->mem[k].act_off * es; };
  auto maskp = [&](int l, int k) -> uint32_t* {  // keep bits of H_l (1-based) of member k
    return bf.mask + (size_t)(l - 1) * (h->A / 32) + h->mem[k].act_off / 32;
  };
  auto h0 = [&](int k) -> void* { return bf.H0 + (size_t)h->mem[k].h0_off * es; };
  auto keepw = [&](int par, int l, int k) -> const uint32_t* {
    return bf.keepw + (size_t)par * c.L * (h->A / 32) + (maskp(l, k) - bf.mask);
  };
  for (int par = 0; par < 2; ++par)
  for (int hf = 0; hf < kGroups; ++hf)
  for (int l = 1; l <= c.L; ++l) {
    // forward: Z_l = H_{l-1} W_l^T + b_l, rows = batch (Bp), cols = dp; members
    // with fewer than l hidden blocks are not in the launch
    Launch f{(int)p.descs.size(), 0, (int)p.tiles.size(), 0, 0.0};
    // the embedded first layer (E produced in the GEMM): its own tile set
    auto fwd_shape = [&](const Member& m, int& M, int& N, int& d) { M = h->Bp, N = m.dp, d = l == 1 ? m.p_in : m.dp; };
    p.tile_set = l == 1 && h->emb ? (sizing ? TILES_SMALL : h->emb_tiles)
                                  : choose_layer(h->tiles_fwd, hf, l, fwd_shape, kHugeFwd);
    for (int k : group[hf]) {
      const Member& m = h->mem[k];
      if (m.depth < l) continue;
      ++f.ndesc;
      GemmDesc d{};
      d.A = l == 1 ? (m.d_emb ? nullptr : h0(k)) : act(Hl(l - 1), k);  // the embedded E is produced in the GEMM
      d.lda = l == 1 ? m.p_in : m.dp;
      d.B = wptr(k, l);
      d.ldb = l == 1 ? m.p_in : m.dp;
      d.C = act(Hl(l), k);
      d.ldc = m.dp;
      d.bias = bf.theta + m.toff[2 * (l - 1) + 1];
      d.M = h->Bp;
      d.N = m.dp;
      d.Kd = l == 1 ? m.p_in : m.dp;
      d.width = m.width;
      d.member = k;
      d.drop_t = m.t;
      d.drop_s = (float)m.scale;
      d.mask = maskp(l, k);
      d.keepw = keepw(par, l, k);
      if (l == 1 && h->stream_rows && m.d_emb == 0 && !sizing) {  // rows straight from the data copy
        d.A = h->xb;
        d.lda = h->Pin;
        d.xrows_n = c.B;
        d.xsrc_rows = h->data_N;
      }
      add_tiles(p, f, (int)p.descs.size(), h->Bp, m.dp, d.Kd);
      p.descs.push_back(d);
      {
        const double fi = l == 1 ? (m.d_emb ? (double)c.d_in * m.d_emb : c.d_in) : m.width, w = m.width;
        f.flops += 2.0 * c.B * w * fi;
        // H_{l-1} and W_l read, H_l written (2-byte elements in bf16), keep words read, mask words written;
        // the embedded first layer reads the batch's data rows and the column table instead of E
        f.bytes += (double)h->elt() * (fi * w + c.B * w) + c.B * w / 4.0 +
                   (l == 1 && m.d_emb ? 4.0 * c.B * c.d_in + 16.0 * fi : (double)h->elt() * c.B * fi);
      }
    }
    sort_launch(p, f);
    p.fwd[par][hf].push_back(f);
  }
  // evaluation: all members in one launch a layer (no second stream runs beside
  // it), over chunks of R rows whose activation blocks are R / Bp times the
  // training ones; the first layer reads the chunk's rows from H_0 block 0
  for (int lv = 0; lv < h->eval_levels; ++lv) {
    const int R = h->eval_rows(lv);
    auto ract = [&](int l, int k) -> void* {
      return bf.H + ((size_t)(l - 1) * (h->A / h->Bp) + (size_t)(h->mem[k].act_off / h->Bp)) * R * es;
    };
    for (int l = 1; l <= c.L; ++l) {
      Launch f{(int)p.descs.size(), 0, (int)p.tiles.size(), 0, 0.0, 0.0};
      LaunchSize z;
      for (int hf = 0; hf < kGroups; ++hf)
        for (int k : group[hf])
          if (h->mem[k].depth >= l) z.add(R, h->mem[k].dp, l == 1 ? h->mem[k].p_in : h->mem[k].dp);
      p.tile_set = l == 1 && h->emb ? (sizing ? TILES_SMALL : h->emb_tiles)
                                    : choose(h->tiles_fwd, z, LaunchSize{}, R >= kBigTile ? kHugeEval : HugeMin{});
      for (int hf = 0; hf < kGroups; ++hf)
        for (int k : group[hf]) {
          const Member& m = h->mem[k];
          if (m.depth < l) continue;
          GemmDesc d{};
          d.A = l > 1 ? ract(l - 1, k) : m.d_emb ? nullptr : (void*)bf.H0;
          d.lda = d.ldb = l == 1 ? m.p_in : m.dp;
          d.B = wptr(k, l);
          d.C = ract(l, k);
          d.ldc = m.dp;
          d.bias = bf.theta + m.toff[2 * (l - 1) + 1];
          d.M = R;
          d.N = m.dp;
          d.Kd = l == 1 ? m.p_in : m.dp;
          d.width = m.width;
          d.member = k;
          add_tiles(p, f, (int)p.descs.size(), R, m.dp, d.Kd);
          p.descs.push_back(d);
          ++f.ndesc;
        }
      sort_launch(p, f);
      p.ev[lv].push_back(f);
    }
  }
  for (int hf = 0; hf < kGroups; ++hf)
  for (int l = 1; l <= c.L; ++l) {
    // weight gradient: dW_l^T[out, in] = sum_rows dZ_l[row, out] H_{l-1}[row, in]
    Launch w{(int)p.descs.size(), 0, (int)p.tiles.size(), 0, 0.0};
    auto dw_shape = [&](const Member& m, int& M, int& N, int& d) { M = m.dp, N = l == 1 ? m.p_in : m.dp, d = h->Bp; };
    const bool alone = c.L > 1 && h->Bp <= kMiniSideRows;  // (short: the other groups' launches do not count)
    p.tile_set = l == 1 && h->emb ? TILES_SMALL
                                  : choose_layer(h->tiles_dw, hf, l, dw_shape, {}, kTallMinDepthDw, alone);
    for (int k : group[hf]) {
      const Member& m = h->mem[k];
      if (m.depth < l) continue;
      ++w.ndesc;
      GemmDesc d{};
      d.A = act(dzb(l), k);
      d.lda = m.dp;
      d.B = l == 1 ? (m.d_emb ? nullptr : h0(k)) : act(Hl(l - 1), k);
      d.ldb = l == 1 ? m.p_in : m.dp;
      d.C = bf.grad + m.toff[2 * (l - 1)];
      d.ldc = l == 1 ? m.p_in : m.dp;
      d.M = m.dp;
      d.N = l == 1 ? m.p_in : m.dp;
      d.Kd = h->Bp;
      d.member = k;
      d.poff = m.toff[2 * (l - 1)];
      d.lr = (float)m.lr;
      d.wd = (float)m.wd;
      // the rows that exist (the member's true width): the optimizer leaves the zero padding rows
      // alone (1.365 -> 1.359 ms per step; skipping the padding columns as well, which leaves
      // holes in the rows' streaming stores, measured 1.362 ms, and 12.5 against 12.2 ms on the
      // embedded step)
      d.opt_rows = m.width;
      if (l == 1 && h->stream_rows && m.d_emb == 0 && !sizing) {  // rows straight from the data copy
        d.B = h->xb;
        d.ldb = h->Pin;
        d.xrows_n = c.B;
        d.xsrc_rows = h->data_N;
      }
      if (l == 1 && m.d_emb) {  // E produced in the GEMM from the batch rows' data rows
        d.xrows_n = c.B;
      }
      add_tiles(p, w, (int)p.descs.size(), d.M, d.N, d.Kd);
      p.descs.push_back(d);
      {
        const double fi = l == 1 ? (m.d_emb ? (double)c.d_in * m.d_emb : c.d_in) : m.width, wd = m.width;
        w.flops += 2.0 * c.B * wd * fi;
        // dZ_l and H_{l-1} read (the embedded first layer: the data rows and the column table);
        // per weight: the fused AdamW's theta, m, v read and written (24 B) and the bf16 shadow
        // written (2 B), plus the fp32 gradient when it is kept
        w.bytes += (double)h->elt() * c.B * wd +
                   (l == 1 && m.d_emb ? 4.0 * c.B * c.d_in + 16.0 * fi : (double)h->elt() * c.B * fi) +
                   wd * fi * (24.0 + (h->prec == Prec::BF16 ? 2.0 : 0.0) + (c.keep_grads ? 4.0 : 0.0));
      }
    }
    sort_launch(p, w);
    p.dw[hf].push_back(w);
    // data gradient (l >= 2): dZ_{l-1} = (dZ_l W_l) * [H_{l-1} > 0] * s_k
    Launch x{(int)p.descs.size(), 0, (int)p.tiles.size(), 0, 0.0};
    if (l >= 2) {
      auto dx_shape = [&](const Member& m, int& M, int& N, int& d) { M = h->Bp, N = d = m.dp; };
      p.tile_set = choose_layer(h->tiles_dx, hf, l, dx_shape, kHugeDx);
      for (int k : group[hf]) {
        const Member& m = h->mem[k];
        if (m.depth < l) continue;
        ++x.ndesc;
        GemmDesc d{};
        d.A = act(dzb(l), k);
        d.lda = m.dp;
        d.B = wptr(k, l);
        d.ldb = m.dp;
        d.C = act(dzb(l - 1), k);
        d.mask = maskp(l - 1, k);
        d.colpart = bf.colpart + (size_t)(l - 2) * (h->A / kPartRows) + h->mem[k].act_off / kPartRows;
        d.ldc = m.dp;
        d.M = h->Bp;
        d.N = m.dp;
        d.Kd = m.dp;
        d.member = k;
        d.drop_s = (float)m.scale;
        add_tiles(p, x, (int)p.descs.size(), h->Bp, m.dp, d.Kd);
        p.descs.push_back(d);
        x.flops += 2.0 * c.B * m.width * m.width;
        // dZ_l and W_l read, dZ_{l-1} written, mask words read, bias partials written
        x.bytes += (double)h->elt() * (2.0 * c.B * m.width + (double)m.width * m.width) + c.B * m.width / 8.0 +
                   4.0 * (h->Bp / kPartRows) * m.width;
      }
      sort_launch(p, x);
    }
    p.dx[hf].push_back(x);
  }
  if (h->small && (h->one_stream || sizing)) {
    // one launch for the weight gradients of all layers, from the same
    // descriptors: a second copy of their tiles in the table
    Launch& w = p.dw_all;
    w = Launch{0, 0, (int)p.tiles.size(), 0, 0.0, 0.0};
    LaunchSize z;
    for (int l = h->emb ? 2 : 1; l <= c.L; ++l)
      for (int i = 0; i < p.dw[0][l - 1].ndesc; ++i) {
        const GemmDesc& d = p.descs[p.dw[0][l - 1].desc0 + i];
        z.add(d.M, d.N, d.Kd);
      }
    p.tile_set = choose(h->tiles_dw, z, LaunchSize{}, {}, kTallMinDepthDw);
    for (int l = h->emb ? 2 : 1; l <= c.L; ++l) {
      const Launch& ln = p.dw[0][l - 1];
      for (int i = 0; i < ln.ndesc; ++i) {
        const GemmDesc& d = p.descs[ln.desc0 + i];
        add_tiles(p, w, ln.desc0 + i, d.M, d.N, d.Kd);
      }
      w.flops += ln.flops;
      w.bytes += ln.bytes;
    }
    w.ts = p.tile_set;
    sort_launch(p, w);
  }
  // gradient-sum work items of group g (one launch after the group's last
  // backward launch): coltiles[sumtile0[g] .. sumtile0[g + 1]) -- the bias
  // columns of every dX launch (layer l >= 2: b_{l-1} of the members with at
  // least l hidden blocks), then every member's head columns (per output), then
  // its head biases and loss
  for (int hf = 0; hf < kGroups; ++hf) {
    p.sumtile0[hf] = (int)p.coltiles.size();
    for (int l = 2; l <= c.L; ++l)
      for (int k : group[hf])
        if (h->mem[k].depth >= l)
          for (int c0 = 0; c0 < h->mem[k].dp; c0 += 64) p.coltiles.push_back(ColTile{k, c0, l - 2, 0});
    for (int k : group[hf])
      for (int o = 0; o <= c.d_out; ++o)
        for (int c0 = 0; c0 < h->mem[k].dp; c0 += 64) p.coltiles.push_back(ColTile{k, c0, kSumHead, o});
    for (int k : group[hf])
      for (int o = 0; o <= c.d_out; ++o) p.coltiles.push_back(ColTile{k, 0, kSumLoss, o});
  }
  p.sumtile0[kGroups] = (int)p.coltiles.size();
  const TileSet saved_ts = p.tile_set;
  p.tile_set = TILES_SMALL;  // the embedding's data-gradient GEMM runs small tiles only
  for (int hf = 0; hf < kGroups; ++hf) {
    Launch& ln = p.de[hf];
    ln = Launch{(int)p.descs.size(), 0, (int)p.tiles.size(), 0, 0.0, 0.0};
    for (int k : group[hf]) {
      const Member& m = h->mem[k];
      if (!m.d_emb) continue;
      GemmDesc d{};
      d.A = act(dzb(1), k);
      d.lda = m.dp;
      d.B = wptr(k, 1);  // W_1 [dp, p_in] read as rows-contiguous: element (n, k) at W_1[k * p_in + n]
      d.ldb = m.p_in;
      d.C = bf.dE + m.h0_off / 16;
      d.ldc = m.p_in;
      d.M = h->Bp;
      d.N = m.p_in;
      d.Kd = m.dp;
      d.member = k;
      add_tiles(p, ln, (int)p.descs.size(), d.M, d.N, d.Kd);
      p.descs.push_back(d);
      ++ln.ndesc;
      const double e = (double)c.d_in * m.d_emb;
      ln.flops += 2.0 * c.B * m.width * e;
      // dZ_1 and W_1 read, x of the rows' features, four fp32 sums per column and 64-row block
      ln.bytes += (double)h->elt() * (c.B * m.width + m.width * e) + 4.0 * c.B * c.d_in + 16.0 * (h->Bp / 64) * e;
    }
    sort_launch(p, ln);
  }
  p.tile_set = saved_ts;
  const int hcols = head_bwd_cols(c.d_out), hrb = head_rows(h);
  for (int hf = 0; hf < kGroups; ++hf) {
    p.headtile0[hf] = (int)p.headtiles.size();
    p.member0[hf] = (int)p.members.size();
    for (int r0 = 0; r0 < h->Bp; r0 += hrb)
      for (int k : group[hf])
        for (int c0 = 0; c0 < h->mem[k].dp; c0 += hcols) p.headtiles.push_back(HeadTile{k, c0, r0});
    for (int k : group[hf]) p.members.push_back(k);
  }
  p.headtile0[kGroups] = (int)p.headtiles.size();
  p.member0[kGroups] = (int)p.members.size();
  if (h->muon) plan_muon(h, bf, group, p, sizing);
  return p;
}

struct Carve {
  char* base;
  size_t off = 0;
  template <typename T>
  T* take(size_t count) {
    off = (size_t)round_up((int64_t)off, 256);
    T* p = reinterpret_cast<T*>(reinterpret_cast<uintptr_t>(base) + off);
    off += count * sizeof(T);
    return p;
  }
};

// Lays out the workspace.  With base == nullptr it only measures: the
// pointers are then offsets from address 0 and are never dereferenced.
size_t carve(const pack_handle* h, char* base, Bufs& bf) {
  const pack_config& c = h->cfg;
  Carve cv{base};
  bf.theta = cv.take<float>(h->P);
  bf.grad = cv.take<float>(h->P);
  bf.m = cv.take<float>(h->P);
  bf.v = cv.take<float>(h->P);
  bf.shadow = h->prec == Prec::BF16 ? cv.take<uint16_t>(h->P) : nullptr;
  // embedded packs never store E (the first layer's GEMMs produce it)
  const int64_t emax = h->eval_rows(0);  // rows of the largest evaluation chunk
  bf.H0 = h->emb ? nullptr : cv.take<char>((size_t)std::max(h->H0e, emax * h->Pin) * h->elt());
  // each member's sums at its E offset / 16 (Bp is a multiple of 256, so the
  // offsets divide; a member's [Bp / 64][4][p_in] sums fill Bp p_in / 16)
  bf.dE = h->emb ? cv.take<float>((size_t)h->H0e / 16) : nullptr;
  bf.etab = h->emb ? cv.take<float4>((size_t)h->Etab) : nullptr;
  bf.H = cv.take<char>((size_t)c.L * (h->A / h->Bp) * emax * h->elt());
  bf.dz = cv.take<char>((size_t)h->ndz() * h->A * h->elt());
  bf.colpart = cv.take<float>((size_t)std::max(1, c.L - 1) * (h->A / kPartRows));
  bf.mask = cv.take<uint32_t>((size_t)c.L * (h->A / 32));
  bf.keepw = cv.take<uint32_t>((size_t)2 * c.L * (h->A / 32));
  bf.zeros = cv.take<char>(256);
  bf.dY = cv.take<float>((size_t)c.K * emax * c.d_out);
  bf.rowloss = cv.take<float>((size_t)c.K * h->Bp);
  bf.d_mem = cv.take<MemberDev>(c.K);
  bf.d_bias_off = cv.take<int64_t>((size_t)c.L * c.K);
  std::vector<int> all[kGroups];
  for (int k = 0; k < c.K; ++k) all[0].push_back(k);
  if (h->muon) {
    int64_t xe = 0, ae = 0;
    muon_sizes(h, all[0].begin(), all[0].end(), xe, ae);
    bf.mX[0] = cv.take<char>((size_t)xe * h->elt());
    bf.mX[1] = cv.take<char>((size_t)xe * h->elt());
    bf.mA = cv.take<char>((size_t)ae * h->elt());
    bf.mB = cv.take<char>((size_t)ae * h->elt());
  }
  // The tables are sized by a plan with every member in one launch per layer
  // (and, for small packs, the weight gradients of all layers once more in
  // one) and small tiles for the main GEMMs.  Tall, wide, huge and big tile
  // sets take at most as many, and a split of the members the same.  Mini
  // tiles, four times as many at most, are chosen only for launches of fewer
  // than kMiniMaxTiles small ones (up to 4 L + 5 launches a group -- forward
  // twice, data and weight gradients, dE, five Newton-Schulz products --, the
  // weight gradients in one, L an evaluation level), or forced.
  Plan plan = build_plan(h, bf, all, true);
  const bool mini_forced = h->tiles_fwd == TILES_MINI || h->tiles_dx == TILES_MINI || h->tiles_dw == TILES_MINI ||
                           h->ns_tiles == TILES_MINI;
  const size_t launches = kGroups * (4 * (size_t)c.L + 5) + 1 + kEvalLevels * (size_t)c.L;
  bf.tile_cap = mini_forced ? 4 * plan.tiles.size() : plan.tiles.size() + (size_t)4 * kMiniMaxTiles * launches;
  if (h->muon) {
    bf.mpart = cv.take<double>(plan.mtiles.size());
    bf.minv = cv.take<float>(plan.mmats.size());
    bf.d_mmats = cv.take<MuonMat>(plan.mmats.size());
    bf.d_mtiles = cv.take<MuonTile>(plan.mtiles.size());
    bf.d_mtile0 = cv.take<int32_t>(plan.mtile0.size());
  }
  bf.d_descs = cv.take<GemmDesc>(plan.descs.size());
  bf.d_tiles = cv.take<Tile>(bf.tile_cap);
  bf.d_coltiles = cv.take<ColTile>(plan.coltiles.size());
  bf.d_headtiles = cv.take<HeadTile>(plan.headtiles.size());
  bf.d_members = cv.take<int32_t>(plan.members.size());
  bf.d_active = cv.take<int32_t>(c.K);
  bf.headpart = cv.take<float>((size_t)(h->Bp / head_rows(h)) * (c.d_out + 1) * (h->A / h->Bp));
  bf.status = cv.take<uint32_t>(64);
  return (size_t)round_up((int64_t)cv.off, 256);
}

int check_member(const pack_handle* h, int32_t k) {
  if (!h) return fail(PACK_EINVAL, "handle is NULL");
  if (k < 0 || k >= h->cfg.K) return fail(PACK_EINVAL, "member %d out of [0, %d)", k, h->cfg.K);
  return PACK_OK;
}

uint32_t as_u32(uint64_t x) { return (uint32_t)(x & 0xFFFFFFFFu); }

GemmArgs base_args(const pack_handle* h) {
  GemmArgs a{};
  a.descs = h->b.d_descs;
  a.tiles = h->b.d_tiles;
  a.zeros = h->b.zeros;
  a.tile_set = TILES_SMALL;
  const Key kd = stream_key(h->cfg.seed, kTagDropout);
  a.key0 = kd.k0;
  a.key1 = kd.k1;
  return a;
}

GemmArgs for_launch(GemmArgs a, const Launch& ln) {
  a.tiles += ln.tile0;
  a.ntiles = ln.ntiles;
  a.tile_set = ln.ts;
  return a;
}

// The first-layer arguments of a GEMM that produces the embedded input E
// (OP_EMB): the data X (N rows), and the batch indices (training forward) or
// the first data row (idx == nullptr: evaluation).
void set_emb(const pack_handle* h, GemmArgs& a, const float* X, int64_t N, const int32_t* idx, int64_t row_base) {
  a.emb_x = X;
  a.emb_x_rows = N;
  a.emb_idx = idx;
  a.emb_row_base = row_base;
  a.emb_mem = h->b.d_mem;
  a.emb_d_in = h->cfg.d_in;
  a.emb_tab = h->b.etab;
}

hipEvent_t pool_event(pack_handle* h) {
  if (h->pool_used == h->event_pool.size()) {
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    h->event_pool.push_back(e);
  }
  return h->event_pool[h->pool_used++];
}

int group_id(pack_handle* h, const std::string& name, int kind) {
  for (size_t i = 0; i < h->groups.size(); ++i)
    if (h->groups[i].name == name) return (int)i;
  h->groups.push_back(ProfGroup{name, kind});
  return (int)h->groups.size() - 1;
}

// Runs `fn` (which enqueues one kernel on `stream`) and, when profiling,
// brackets it with events and attributes `work` to the named kernel.
template <typename F>
hipError_t timed(pack_handle* h, const char* name, int kind, double flops, double bytes, hipStream_t stream, F fn) {
  if (!h->prof) return fn();
  hipEvent_t a = pool_event(h), b = pool_event(h);
  if (!a || !b) return hipErrorOutOfMemory;
  hipError_t e = hipEventRecord(a, stream);
  if (e != hipSuccess) return e;
  e = fn();
  if (e != hipSuccess) return e;
  e = hipEventRecord(b, stream);
  const int g = group_id(h, name, kind);
  h->groups[g].flops += flops;  // summed here, averaged per launch when read
  h->groups[g].bytes += bytes;
  h->timed.push_back(TimedLaunch{g, a, b});
  return e;
}

// The column tables of the listed members' embeddings from their current
// parameters (d_members: the same member ids in device memory).
hipError_t emb_tables(pack_handle* h, const int32_t* d_members, const std::vector<int>& ids, hipStream_t s) {
  double nb = 0;
  for (int k : ids) nb += 32.0 * h->mem[k].p_in;  // four parameters read, one 16-byte entry written per column
  return timed(h, "embed_table", 1, 0.0, nb, s, [&] {
    return launch_embed_table(h->prec, h->cfg.d_in, h->b.d_mem, d_members, (int)ids.size(), max_pin(h, ids),
                              h->b.theta, h->b.etab, s);
  });
}

void set_active_ids(pack_handle* h) {
  h->active_ids.clear();
  for (int k = 0; k < h->cfg.K; ++k)
    if (h->active[k]) h->active_ids.push_back(k);
}

// Builds the launch tables of the active members, uploads them into the bound
// workspace, and records the launches.  Synchronizes `stream`: the host tables are freed on
// return.  The caller's earlier work on `stream` is ordered before the copies.
int upload_plan(pack_handle* h, hipStream_t stream) {
  const pack_config& c = h->cfg;
  Plan plan = build_plan(h, h->b, h->group);
  if (plan.tiles.size() > h->b.tile_cap)
    return fail(PACK_EINVAL, "internal: the plan holds %zu GEMM tiles, the device table %zu", plan.tiles.size(),
                h->b.tile_cap);
  auto up = [&](void* dst, const void* src, size_t bytes) {
    return bytes ? hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, stream) : hipSuccess;
  };
  HIP_TRY(up(h->b.d_active, h->active_ids.data(), h->active_ids.size() * 4));
  HIP_TRY(up(h->b.d_descs, plan.descs.data(), plan.descs.size() * sizeof(GemmDesc)));
  HIP_TRY(up(h->b.d_tiles, plan.tiles.data(), plan.tiles.size() * sizeof(Tile)));
  HIP_TRY(up(h->b.d_coltiles, plan.coltiles.data(), plan.coltiles.size() * sizeof(ColTile)));
  HIP_TRY(up(h->b.d_headtiles, plan.headtiles.data(), plan.headtiles.size() * sizeof(HeadTile)));
  HIP_TRY(up(h->b.d_members, plan.members.data(), plan.members.size() * sizeof(int32_t)));
  if (h->muon) {
    HIP_TRY(up(h->b.d_mmats, plan.mmats.data(), plan.mmats.size() * sizeof(MuonMat)));
    HIP_TRY(up(h->b.d_mtiles, plan.mtiles.data(), plan.mtiles.size() * sizeof(MuonTile)));
    HIP_TRY(up(h->b.d_mtile0, plan.mtile0.data(), plan.mtile0.size() * sizeof(int32_t)));
  }
  HIP_TRY(hipStreamSynchronize(stream));
  h->n_mmats = (int)plan.mmats.size();
  h->n_mtiles = (int)plan.mtiles.size();
  for (int g = 0; g <= kGroups; ++g) {
    h->mmat0[g] = plan.mmat0[g];
    h->mtileg[g] = plan.mtileg[g];
  }
  for (int g = 0; g < kGroups; ++g) {
    for (int par = 0; par < 2; ++par) {
      h->nsA[par][g] = plan.nsA[par][g];
      h->nsX[par][g] = plan.nsX[par][g];
    }
    h->nsB[g] = plan.nsB[g];
  }
  for (int hf = 0; hf < kGroups; ++hf) h->de[hf] = plan.de[hf];
  for (int hf = 0; hf < kGroups; ++hf) {
    h->fwd[0][hf] = plan.fwd[0][hf];
    h->fwd[1][hf] = plan.fwd[1][hf];
    h->dx[hf] = plan.dx[hf];
    h->dw[hf] = plan.dw[hf];
  }
  for (int lv = 0; lv < kEvalLevels; ++lv) h->ev[lv] = plan.ev[lv];
  h->dw_all = plan.dw_all;
  for (int g = 0; g <= kGroups; ++g) h->sumtile0[g] = plan.sumtile0[g];
  for (int i = 0; i <= kGroups; ++i) {
    h->headtile0[i] = plan.headtile0[i];
    h->member0[i] = plan.member0[i];
  }
  h->ncoltiles = (int)plan.coltiles.size();
  h->nheadtiles = (int)plan.headtiles.size();
  h->head_rb = head_rows(h);
  (void)c;
  return PACK_OK;
}

const char* gemm_name(Prec p, OpKind a, OpKind b, EpiKind e);

// Muon step of the hidden weights of member group g's active members (their
// gradients are in grad): momentum and tile norms, inverse norms, X0, ns_steps
// Newton-Schulz iterations of three grouped GEMMs, update.  On the group's
// stream after its backward pass, so one group's step overlaps the others'
// backward passes and Muon steps.
hipError_t muon_step(pack_handle* h, const GemmArgs& base, int g, hipStream_t stream) {
  const int mat0 = h->mmat0[g], nmats = h->mmat0[g + 1] - mat0;
  const int tile0 = h->mtileg[g], ntiles = h->mtileg[g + 1] - tile0;
  if (nmats == 0) return hipSuccess;
  const pack_config& c = h->cfg;
  const float mu = (float)c.muon_momentum;
  const int nest = c.muon_nesterov ? 1 : 0;
  const MuonTile* tiles = h->b.d_mtiles + tile0;
  const double wbytes = (double)ntiles * 64 * 64;  // upper bound of the weights' elements
  hipError_t e = timed(h, "muon_prep", 1, 0.0, wbytes * 12.0, stream, [&] {
    return launch_muon_prep(h->b.d_mmats, tiles, ntiles, h->b.grad, h->b.m, mu, nest, h->b.mpart + tile0, stream);
  });
  if (e != hipSuccess) return e;
  e = timed(h, "muon_norm", 1, 0.0, 8.0 * ntiles, stream, [&] {
    return launch_muon_norm(h->b.d_mtile0 + mat0, nmats, h->b.mpart, h->b.minv + mat0, stream);
  });
  if (e != hipSuccess) return e;
  e = timed(h, "muon_convert", 1, 0.0, wbytes * (8.0 + h->elt()), stream, [&] {
    return launch_muon_convert(h->prec, h->b.d_mmats, tiles, ntiles, h->b.grad, h->b.m, mu, nest, h->b.minv,
                               h->b.mX[0], stream);
  });
  if (e != hipSuccess) return e;
  static const float kA = 3.4445f, kB = -4.7750f, kC = 2.0315f;
  auto ns_args = [&](const GemmArgs& b0, const Launch& ln, OpKind bk, float alpha, float beta, bool sym) {
    GemmArgs ga = for_launch(b0, ln);
    ga.ns_alpha = alpha;
    ga.ns_beta = beta;
    ga.ns_sym = sym ? 1 : 0;
    return timed(h, gemm_name(h->prec, OP_KMAJ, bk, EPI_NS), 0, ln.flops, ln.bytes, stream,
                 [&] { return launch_gemm(h->prec, OP_KMAJ, bk, EPI_NS, ga, stream); });
  };
  auto ns = [&](const Launch& ln, OpKind bk, float alpha, float beta, bool sym) {
    return ns_args(base, ln, bk, alpha, beta, sym);
  };
  // the last iteration's X launch applies the update in its epilogue
  // (TABPACK_MUON_FUSED_UPDATE=0: a separate update kernel reads the stored X)
  const bool fused = h->muon_fused;
  for (int it = 0; it < h->ns_steps; ++it) {
    const int par = it & 1;
    if ((e = ns(h->nsA[par][g], OP_KMAJ, 0.0f, 1.0f, true)) != hipSuccess) return e;
    if ((e = ns(h->nsB[g], OP_KMAJ, kB, kC, true)) != hipSuccess) return e;
    if (fused && it + 1 == h->ns_steps) {
      GemmArgs fa = base;
      fa.ns_theta = h->b.theta;
      fa.ns_shadow = h->b.shadow;
      if ((e = ns_args(fa, h->nsX[par][g], OP_RMAJ, kA, 1.0f, false)) != hipSuccess) return e;
      return hipSuccess;
    }
    if ((e = ns(h->nsX[par][g], OP_RMAJ, kA, 1.0f, false)) != hipSuccess) return e;
  }
  return timed(h, "muon_update", 1, 0.0, wbytes * (8.0 + h->elt() + (h->prec == Prec::BF16 ? 2.0 : 0.0)), stream,
               [&] {
                 return launch_muon_update(h->prec, h->b.d_mmats, tiles, ntiles, h->b.theta, h->b.shadow,
                                           h->b.mX[h->ns_steps & 1], stream);
               });
}

const char* gemm_name(Prec p, OpKind a, OpKind b, EpiKind e) {
  static const char* ops[] = {"kmaj", "rmaj", "emb"};
  static const char* epis[] = {"fwd", "fwd_eval", "dx", "dw", "ns", "de"};
  static thread_local char buf[64];
  snprintf(buf, sizeof buf, "gemm_%s_%s_%s_%s", p == Prec::BF16 ? "bf16" : "f32", ops[a], ops[b], epis[e]);
  return buf;
}

// A handle of the pack with its members, layout and launch rules, without the
// parameters' initial values.
int make_pack(const pack_config* cfg, pack_handle** out) {
  int rc = validate(cfg);
  if (rc) return rc;
  pack_handle* h = new (std::nothrow) pack_handle();
  if (!h) return fail(PACK_EINVAL, "out of host memory");
  h->cfg = *cfg;
  h->cfg.members = nullptr;
  h->prec = cfg->precision == PACK_PREC_BF16 ? Prec::BF16 : Prec::FP32;
  h->task = (Task)cfg->task;
  h->q = cfg->quantum ? cfg->quantum : 32;
  // The tile sets of the main GEMMs are chosen per launch (launch_tiles);
  // TABPACK_GEMM_TILES=big|tall|small|mini|huge fixes them all (huge: forward and
  // data gradient, the weight gradient small; fp32: small or mini),
  // TABPACK_TILES_FWD / _DX / _DW one kind.
  auto tile_env = [&](const char* name, bool main = true, bool huge = false) {
    const char* e = getenv(name);
    if (!e && main) e = getenv("TABPACK_GEMM_TILES");
    if (!e) return -1;
    const std::string v(e);
    if (v == "mini") return (int)TILES_MINI;
    if (h->prec == Prec::FP32) return (int)TILES_SMALL;
    if (v == "huge" && huge) return (int)TILES_HUGE;
    return (int)(v == "big" ? TILES_BIG : (v == "tall" ? TILES_TALL : TILES_SMALL));
  };
  h->tiles_fwd = tile_env("TABPACK_TILES_FWD", true, true);
  h->tiles_dx = tile_env("TABPACK_TILES_DX", true, true);
  h->tiles_dw = tile_env("TABPACK_TILES_DW");
  // Newton-Schulz GEMMs: small tiles measured 3.79 ms per Muon step on the
  // 64-member regression workload, tall 4.03, big 5.53; TABPACK_NS_TILES overrides
  h->ns_tiles = tile_env("TABPACK_NS_TILES", false);
  // the embedded first layer's forward: wide tiles in bf16 (each produced E
  // element feeds 256 output columns); TABPACK_EMB_TILES=small overrides
  h->emb_tiles = h->prec == Prec::BF16 ? TILES_WIDE : TILES_SMALL;
  if (const char* e = getenv("TABPACK_EMB_TILES"))
    if (std::string(e) == "small") h->emb_tiles = TILES_SMALL;
  if (const char* e = getenv("TABPACK_MUON_FUSED_UPDATE")) h->muon_fused = std::string(e) != "0";
  h->muon = cfg->optimizer == PACK_OPT_MUON;
  h->emb = cfg->emb_lo > 0;
  h->ns_steps = cfg->ns_steps ? cfg->ns_steps : 5;
  h->Bp = (int)round_up(cfg->B, kRowAlign);
  h->Pin = (int)round_up(cfg->d_in, 8);
  h->mem.resize(cfg->K);
  if (cfg->members) {
    for (int k = 0; k < cfg->K; ++k) {
      const pack_member_hp& e = cfg->members[k];
      if (e.width < 1 || e.width > 16384 || !(e.dropout >= 0 && e.dropout < 1) || !(e.lr > 0) ||
          !(e.wd >= 0) || e.depth < 0 || e.depth > cfg->L ||
          (cfg->optimizer == PACK_OPT_MUON && !(e.muon_lr > 0)) ||
          (cfg->emb_lo > 0 && (e.d_emb < 8 || e.d_emb > 32 || !(e.sigma > 0)))) {
        delete h;
        return fail(PACK_EINVAL, "explicit hyperparameters of member %d out of range", k);
      }
      h->mem[k].width = e.width;
      h->mem[k].dropout = e.dropout;
      h->mem[k].lr = e.lr;
      h->mem[k].wd = e.wd;
      h->mem[k].depth = e.depth ? e.depth : cfg->L;
      h->mem[k].muon_lr = cfg->optimizer == PACK_OPT_MUON ? e.muon_lr : 0.0;
      h->mem[k].d_emb = cfg->emb_lo > 0 ? e.d_emb : 0;
      h->mem[k].sigma = cfg->emb_lo > 0 ? e.sigma : 0.0;
    }
  } else {
    sample_members(h);
  }
  for (Member& m : h->mem) {
    m.t = (uint32_t)std::min(std::floor(m.dropout * 65536.0), 65535.0);  // threshold of a 16-bit draw
    m.scale = 1.0 / (1.0 - m.dropout);
  }
  plan_layout(h);
  // Operands the GEMM loaders cannot reach whole would lose their last rows.
  for (int k = 0; k < cfg->K; ++k) {
    const Member& m = h->mem[k];
    const int64_t e = (int64_t)h->elt(), cols = m.depth > 1 ? std::max(m.p_in, m.dp) : m.p_in;
    const int64_t weight = m.width * cols * e, act = (int64_t)cfg->B * m.dp * e;
    if (weight > kOperandBytes || act > kOperandBytes) {
      const int64_t width = m.width;
      delete h;
      return fail(PACK_EINVAL, "member %d (width %lld): %s of %lld bytes; a GEMM operand is limited to 2 GiB", k,
                  (long long)width, weight > kOperandBytes ? "a weight matrix" : "activations",
                  (long long)std::max(weight, act));
    }
  }
  plan_eval(h);
  h->active.assign(cfg->K, 1);
  set_active_ids(h);
  h->small = small_pack(h, h->active_ids);
  split_members(h);
  *out = h;
  return PACK_OK;
}

}  // namespace

extern "C" {

const char* pack_last_error(void) { return g_err.c_str(); }

int pack_init(const pack_config* cfg, pack_handle** out) {
  if (!out) return fail(PACK_EINVAL, "out is NULL");
  *out = nullptr;
  pack_handle* h = nullptr;
  const int rc = make_pack(cfg, &h);
  if (rc) return rc;
  init_params(h);
  *out = h;
  g_err.clear();
  return PACK_OK;
}

int pack_debug_plan(const pack_config* cfg, const uint8_t* active, pack_plan_info* out) {
  if (!out) return fail(PACK_EINVAL, "out is NULL");
  pack_handle* h = nullptr;
  const int rc = make_pack(cfg, &h);
  if (rc) return rc;
  carve(h, nullptr, h->b);  // addresses from 0, never read
  if (active) {
    for (int k = 0; k < cfg->K; ++k) h->active[k] = active[k] ? 1 : 0;
    set_active_ids(h);
    split_members(h);
  }
  const Plan plan = build_plan(h, h->b, h->group);
  *out = pack_plan_info{};
  out->tiles = (int64_t)plan.tiles.size();
  out->tile_capacity = (int64_t)h->b.tile_cap;
  out->groups = h->ngroups;
  out->one_stream = h->one_stream ? 1 : 0;
  if (h->muon) {
    out->ns_sym = plan.nsB[0].ts;
    out->ns_x = plan.nsX[0][0].ts;
  }
  out->tiles_fwd = plan.fwd[0][0].back().ts;
  out->tiles_dx = plan.dx[0].back().ts;
  out->tiles_dw = plan.dw[0].back().ts;
  out->eval_levels = h->eval_levels;
  for (int lv = 0; lv < h->eval_levels; ++lv) {
    out->eval_rows[lv] = h->eval_rows(lv);
    for (const Launch& ln : plan.ev[lv]) {
      if (lv == 0)
        for (int i = 0; i < ln.ndesc; ++i) {
          const GemmDesc& d = plan.descs[ln.desc0 + i];
          const int64_t rows = std::min((int64_t)d.M, h->eval_cap);
          if (d.A) out->eval_operand = std::max(out->eval_operand, rows * d.lda * (int64_t)h->elt());
        }
      if (!plan.ev[lv].empty()) out->eval_tiles[lv] = plan.ev[lv].back().ts;
    }
  }
  pack_destroy(h);
  return PACK_OK;
}

int pack_destroy(pack_handle* h) {
  if (h) {
    for (hipEvent_t e : h->event_pool) (void)hipEventDestroy(e);
    if (h->ev_fork) (void)hipEventDestroy(h->ev_fork);
    if (h->ev_join) (void)hipEventDestroy(h->ev_join);
    for (hipEvent_t e : h->ev_keep)
      if (e) (void)hipEventDestroy(e);
    if (h->side) (void)hipStreamDestroy(h->side);
    if (h->ev_split) (void)hipEventDestroy(h->ev_split);
    for (int g = 1; g < kGroups; ++g) {
      if (h->ev_merge[g]) (void)hipEventDestroy(h->ev_merge[g]);
      if (h->gstream[g]) (void)hipStreamDestroy(h->gstream[g]);
    }
    for (hipEvent_t e : h->ev_gather)
      if (e) (void)hipEventDestroy(e);
    for (hipEvent_t e : h->ev_bias)
      if (e) (void)hipEventDestroy(e);
  }
  delete h;
  return PACK_OK;
}

int pack_get_hparams(const pack_handle* h, pack_member_hp* out) {
  if (!h || !out) return fail(PACK_EINVAL, "NULL argument");
  for (int k = 0; k < h->cfg.K; ++k) {
    const Member& m = h->mem[k];
    out[k] = pack_member_hp{m.width, m.dp, m.t, m.depth, m.dropout, m.lr, m.wd, m.scale, m.muon_lr, m.d_emb, 0,
                            m.sigma};
  }
  return PACK_OK;
}

int pack_workspace_size(const pack_handle* h, size_t* bytes) {
  if (!h || !bytes) return fail(PACK_EINVAL, "NULL argument");
  Bufs tmp;
  *bytes = carve(h, nullptr, tmp);
  return PACK_OK;
}

int pack_bind(pack_handle* h, void* workspace, size_t bytes, hipStream_t stream) {
  if (!h || !workspace) return fail(PACK_EINVAL, "NULL argument");
  if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(PACK_EINVAL, "workspace must be 256-byte aligned");
  size_t need = 0;
  pack_workspace_size(h, &need);
  if (bytes < need) return fail(PACK_EINVAL, "workspace has %zu bytes, %zu needed", bytes, need);
  carve(h, static_cast<char*>(workspace), h->b);
  if (!h->side) {
    HIP_TRY(hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking));
    HIP_TRY(hipEventCreateWithFlags(&h->ev_fork, hipEventDisableTiming));
    HIP_TRY(hipEventCreateWithFlags(&h->ev_join, hipEventDisableTiming));
    for (hipEvent_t& e : h->ev_keep) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    HIP_TRY(hipEventCreateWithFlags(&h->ev_split, hipEventDisableTiming));
    for (int g = 1; g < kGroups; ++g) {
      HIP_TRY(hipStreamCreateWithFlags(&h->gstream[g], hipStreamNonBlocking));
      HIP_TRY(hipEventCreateWithFlags(&h->ev_merge[g], hipEventDisableTiming));
    }
    for (hipEvent_t& e : h->ev_gather) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    for (hipEvent_t& e : h->ev_bias) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  }
  h->keep_ready = 0;
  h->last_rows = h->Bp;
  h->last_valid = h->cfg.B;
  HIP_TRY(hipMemsetAsync(workspace, 0, need, stream));
  HIP_TRY(hipMemcpyAsync(h->b.theta, h->theta_host.data(), h->P * sizeof(float), hipMemcpyHostToDevice, stream));
  std::vector<MemberDev> md(h->cfg.K);
  std::vector<int64_t> boff((size_t)h->cfg.L * h->cfg.K);
  for (int k = 0; k < h->cfg.K; ++k) {
    const Member& m = h->mem[k];
    md[k] = MemberDev{m.width, m.dp, m.t, (float)m.scale, (float)m.lr, (float)m.wd, m.act_off,
                      m.toff[2 * m.depth], m.toff[2 * m.depth + 1], m.toff[2 * m.depth - 1],
                      (int64_t)(m.depth - 1) * h->A + m.act_off, (int64_t)((m.depth - 1) % h->ndz()) * h->A + m.act_off,
                      m.depth, m.d_emb, m.eoff[0], m.eoff[1], m.eoff[2], m.eoff[3], m.h0_off, m.etab_off, m.p_in, 0};
    for (int l = 1; l <= m.depth; ++l) boff[(size_t)(l - 1) * h->cfg.K + k] = m.toff[2 * (l - 1) + 1];
  }
  HIP_TRY(hipMemcpyAsync(h->b.d_mem, md.data(), md.size() * sizeof(MemberDev), hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(h->b.d_bias_off, boff.data(), boff.size() * 8, hipMemcpyHostToDevice, stream));
  if (h->prec == Prec::BF16) HIP_TRY(launch_to_shadow(h->b.theta, h->b.shadow, h->P, stream));
  const int rc = upload_plan(h, stream);  // synchronizes the stream
  if (rc) return rc;
  h->t = 0;
  h->bound = true;
  return PACK_OK;
}

int pack_set_active(pack_handle* h, const uint8_t* active, hipStream_t stream) {
  if (!h || !active) return fail(PACK_EINVAL, "NULL argument");
  for (int k = 0; k < h->cfg.K; ++k)
    if (active[k] > 1) return fail(PACK_EINVAL, "active[%d] = %d is not 0 or 1", k, (int)active[k]);
  h->active.assign(active, active + h->cfg.K);
  set_active_ids(h);
  split_members(h);
  if (!h->bound) return PACK_OK;
  // a member that comes back needs keep words for the next step, which were
  // produced (during the last step) for the previous set only
  h->keep_ready = 0;
  return upload_plan(h, stream);
}

int pack_train_step(pack_handle* h, const float* X, const void* y, int64_t N, const int32_t* idx,
                    uint64_t step, float* loss_out, hipStream_t stream) {
  if (!h) return fail(PACK_EINVAL, "handle is NULL");
  if (!h->bound) return fail(PACK_ESTATE, "pack_bind() has not been called");
  if (!X || !y || !idx || !loss_out) return fail(PACK_EINVAL, "NULL device pointer");
  if (N < 1) return fail(PACK_EINVAL, "N=%lld must be positive", (long long)N);
  if (step != h->t + 1) return fail(PACK_ESTATE, "step %llu given, %llu expected", (unsigned long long)step,
                                    (unsigned long long)(h->t + 1));
  if (h->active_ids.empty()) return fail(PACK_ESTATE, "no member is active");
  if (h->stream_rows && (X != h->data_X || N != h->data_N))
    return fail(PACK_EINVAL, "X / N differ from the data bound with pack_bind_data (bind it again, or unbind "
                             "it with X = NULL)");
  const pack_config& c = h->cfg;
  if (!h->stream_rows && !h->emb && (int64_t)c.B * h->Pin * (int64_t)h->elt() > kOperandBytes)
    return fail(PACK_EINVAL, "a gathered batch of %d rows of %d features passes the GEMMs' operand limit of 2 GiB", c.B,
                c.d_in);
  h->last_rows = h->Bp;
  h->last_valid = c.B;
  const int nact = (int)h->active_ids.size();
  GemmArgs a = base_args(h);
  a.rows_valid = c.B;
  a.step = as_u32(step);
  a.idx = idx;
  int max_dp = 0;
  double act_bytes = 0, nkeep = 0;
  for (int k : h->active_ids) {
    const Member& m = h->mem[k];
    max_dp = std::max(max_dp, m.dp);
    act_bytes += (double)c.B * h->elt() * m.width;
    nkeep += (double)m.depth * h->Bp * m.dp / 8;
  }
  const double bc1 = 1.0 - std::pow(c.beta1, (double)step);
  const double bc2 = 1.0 - std::pow(c.beta2, (double)step);
  const AdamConst ac{(float)c.beta1, (float)c.beta2, (float)c.eps, (float)(1.0 - c.beta1), (float)(1.0 - c.beta2),
                     (float)bc1, (float)std::sqrt(bc2)};
  auto gemm = [&](OpKind ak, OpKind bk, EpiKind e, const Launch& ln, int layer, hipStream_t s) {
    GemmArgs al = for_launch(a, ln);
    al.layer = layer;
    if (ak == OP_EMB || bk == OP_EMB) set_emb(h, al, X, N, idx, 0);
    const bool adamw = e == EPI_DW && !h->muon;  // Muon: the gradient is stored, muon_step updates W_l
    if (adamw) {
      al.theta = h->b.theta;
      al.am = h->b.m;
      al.av = h->b.v;
      al.shadow = h->b.shadow;
      al.adam = ac;
      al.keep_grad = c.keep_grads ? 1 : 0;
    }
    // AdamW fused: the weight update traffic dominates, so the HBM roofline applies
    return timed(h, gemm_name(h->prec, ak, bk, e), adamw ? 1 : 0, ln.flops, ln.bytes, s,
                 [&] { return launch_gemm(h->prec, ak, bk, e, al, s); });
  };
  // The dropout keep words alternate between two buffers by step parity.
  const int par = (int)(step & 1);
  auto words = [&](int p) { return h->b.keepw + (size_t)p * c.L * (h->A / 32); };
  auto keep_words = [&](uint64_t s_step, int p, hipStream_t s) {
    return timed(h, "dropout_words", 1, 0.0, nkeep, s, [&] {
      return launch_dropout_words(a.key0, a.key1, as_u32(s_step), h->b.d_mem, nact, c.L, max_dp, h->Bp, c.B,
                                  h->A / 32, words(p), h->b.d_active, s);
    });
  };
  // The input of group hf's first layer: the embeddings' column tables from the
  // current parameters (the first-layer GEMM produces E from them), or the
  // gathered batch unless the data is bound.
  auto input = [&](int hf, hipStream_t s) -> hipError_t {
    const int32_t* gm = h->b.d_members + h->member0[hf];
    const int gk = h->member0[hf + 1] - h->member0[hf];
    if (h->emb) return emb_tables(h, gm, h->group[hf], s);
    return timed(h, "gather", 1, 0.0, (double)gk * c.B * c.d_in * (4.0 + h->elt()), s, [&] {
      return launch_gather(h->prec, X, N, c.d_in, h->Pin, idx, c.B, 0, c.B, gk, h->Bp, h->b.H0, gm, s);
    });
  };
  auto forward = [&](int hf, int l, hipStream_t s) {
    return gemm(l == 1 && h->emb ? OP_EMB : OP_KMAJ, OP_KMAJ, EPI_FWD, h->fwd[par][hf][l - 1], l, s);
  };
  // The head: loss and dY, then dZ_L and the head's partial sums.
  auto head = [&](int hf, hipStream_t s) -> hipError_t {
    const int32_t* gm = h->b.d_members + h->member0[hf];
    const int gk = h->member0[hf + 1] - h->member0[hf];
    const double nb = act_bytes / h->ngroups;
    if (h->small)
      return timed(h, "head_train", 1, 0.0, 2.0 * nb, s, [&] {
        return launch_head_train(h->prec, h->task, h->b.H, h->b.theta, h->b.d_mem, gk, h->Bp, c.d_out, y, N, idx,
                                 c.B, h->b.dY, h->b.rowloss, h->b.dz, h->b.headpart, h->b.status, gm, s);
      });
    const hipError_t e = timed(h, "head_fwd", 1, 0.0, nb, s, [&] {
      return launch_head_fwd(h->prec, h->task, kHeadTrain, h->b.H, h->b.theta, h->b.d_mem, gk, h->Bp, h->Bp, c.d_out,
                             y, idx, c.B, c.B, 0, N, h->b.dY, h->b.rowloss, nullptr, h->b.status, gm, s);
    });
    if (e != hipSuccess) return e;
    return timed(h, "head_bwd", 1, 0.0, 2.0 * nb, s, [&] {
      return launch_head_bwd(h->prec, h->b.H, h->b.theta, h->b.d_mem, h->b.d_headtiles + h->headtile0[hf],
                             h->headtile0[hf + 1] - h->headtile0[hf], h->Bp, h->head_rb, c.d_out, h->b.dY,
                             h->b.dz, h->b.headpart, s);
    });
  };
  // The gradients of the embedding parameters: dE = dZ_1 W_1 (before W_1 is
  // updated), reduced in the GEMM's epilogue into per-64-row-block gradient
  // sums; then the sums over the blocks and the parameters' update.
  auto emb_backward = [&](int hf, hipStream_t s) -> hipError_t {
    GemmArgs ae = for_launch(a, h->de[hf]);
    ae.tile_set = TILES_SMALL;
    set_emb(h, ae, X, N, idx, 0);
    const hipError_t e =
        timed(h, gemm_name(h->prec, OP_KMAJ, OP_RMAJ, EPI_DE), 0, h->de[hf].flops, h->de[hf].bytes, s,
              [&] { return launch_gemm(h->prec, OP_KMAJ, OP_RMAJ, EPI_DE, ae, s); });
    if (e != hipSuccess) return e;
    const int gk = h->member0[hf + 1] - h->member0[hf];
    double gbytes = 0.0;
    for (int k : h->group[hf]) gbytes += 4.0 * c.d_in * h->mem[k].d_emb * (4.0 * (h->Bp / 64) + 28.0);
    return timed(h, "embed_grad", 1, 0.0, gbytes, s, [&] {
      return launch_embed_grad(c.d_in, h->Bp, h->b.d_mem, h->b.d_members + h->member0[hf], gk,
                               max_pin(h, h->group[hf]), h->b.dE, h->b.grad, h->b.theta, h->b.m, h->b.v, ac, s);
    });
  };
  // The group's gradient sums (hidden biases from the dX partials, head
  // weights and last hidden bias from the head partials, loss and head bias
  // from the per-row values) and the update of those parameters, one launch;
  // `ahead`: also the next step's keep words, into the other buffer (last read
  // by the previous step's forward pass).
  auto grad_sums = [&](int hf, bool ahead, hipStream_t s) -> hipError_t {
    const int t0 = h->sumtile0[hf], t1 = h->sumtile0[hf + 1];
    SumsArgs g{};
    g.colpart = h->b.colpart;
    g.part_stride = h->A / kPartRows;
    g.headpart = h->b.headpart;
    g.RB = h->head_rb;
    g.rowloss = h->b.rowloss;
    g.dY = h->b.dY;
    g.mem = h->b.d_mem;
    g.tiles = h->b.d_coltiles + t0;
    g.ntiles = t1 - t0;
    g.Bp = h->Bp;
    g.B = c.B;
    g.d_out = c.d_out;
    g.K = c.K;
    g.bias_off = h->b.d_bias_off;
    g.grad = h->b.grad;
    g.theta = h->b.theta;
    g.m = h->b.m;
    g.v = h->b.v;
    g.loss_out = loss_out;
    g.adam = ac;
    g.decay_bias = c.decay_bias;
    if (ahead) {
      g.words = words(par ^ 1);
      g.key0 = a.key0;
      g.key1 = a.key1;
      g.step = as_u32(step + 1);
      g.L = c.L;
      g.max_dp = max_dp;
      g.nmembers = nact;
      g.A32 = h->A / 32;
      g.members = h->b.d_active;
    }
    return timed(h, "grad_sums", 1, 0.0, (4.0 * (h->Bp / kPartRows) + 28.0) * 64.0 * (t1 - t0) + (ahead ? nkeep : 0.0),
                 s, [&] { return launch_grad_sums(g, s); });
  };
  // The kernels check the batch indices where they use them and the head flags
  // one outside [0, N); those of members that are not in the launches are
  // looked at here.
  if (nact < c.K)
    HIP_TRY(timed(h, "idx_check", 1, 0.0, 4.0 * c.K * c.B, stream,
                  [&] { return launch_idx_check(idx, (int64_t)c.K * c.B, N, h->b.status, stream); }));

  if (h->one_stream) {
    // One chain of launches on the caller's stream.  The dX chain runs first
    // (dX_l reads W_l, which the weight gradient updates), then the weight
    // gradients of all layers in one launch; a large pack of which few members
    // are left has two dZ buffers and runs them layer by layer.
    if (h->keep_ready != step) HIP_TRY(keep_words(step, par, stream));
    if (h->emb || !h->stream_rows) HIP_TRY(input(0, stream));
    for (int l = 1; l <= c.L; ++l) HIP_TRY(forward(0, l, stream));
    HIP_TRY(head(0, stream));
    for (int l = c.L; l >= 2; --l) {
      HIP_TRY(gemm(OP_KMAJ, OP_RMAJ, EPI_DX, h->dx[0][l - 1], l, stream));
      // with two dZ buffers dW_l runs before dX_{l-1} overwrites dZ_l
      if (!h->small) HIP_TRY(gemm(OP_RMAJ, OP_RMAJ, EPI_DW, h->dw[0][l - 1], l, stream));
    }
    if (h->emb) {
      HIP_TRY(emb_backward(0, stream));
      HIP_TRY(gemm(OP_RMAJ, OP_EMB, EPI_DW, h->dw[0][0], 1, stream));
    }
    if (h->small)
      HIP_TRY(gemm(OP_RMAJ, OP_RMAJ, EPI_DW, h->dw_all, 0, stream));
    else if (!h->emb)
      HIP_TRY(gemm(OP_RMAJ, OP_RMAJ, EPI_DW, h->dw[0][0], 1, stream));
    if (h->muon) HIP_TRY(muon_step(h, a, 0, stream));
    HIP_TRY(grad_sums(0, true, stream));
    h->keep_ready = step + 1;
    h->t = step;
    return PACK_OK;
  }

  // member groups: group 0 on the caller's stream, group g on gstream[g]
  hipStream_t hs[kGroups] = {stream};
  for (int g = 1; g < kGroups; ++g) hs[g] = h->gstream[g];
  const int ng = h->ngroups;
  auto split = [&]() -> hipError_t {
    hipError_t e = hipEventRecord(h->ev_split, stream);
    for (int g = 1; g < ng && e == hipSuccess; ++g) e = hipStreamWaitEvent(hs[g], h->ev_split, 0);
    return e;
  };
  auto merge = [&]() -> hipError_t {
    hipError_t e = hipSuccess;
    for (int g = 1; g < ng && e == hipSuccess; ++g) {
      e = hipEventRecord(h->ev_merge[g], hs[g]);
      if (e == hipSuccess) e = hipStreamWaitEvent(stream, h->ev_merge[g], 0);
    }
    return e;
  };
  // Dropout keep words (Philox, ALU-bound) run on the side stream: normally
  // they were produced during the previous step's backward pass; otherwise
  // (first step, or after a break in the sequence) they are produced now,
  // beside the HBM-bound gather.  Either way the forward GEMMs wait for them.
  if (h->keep_ready != step) {
    HIP_TRY(hipEventRecord(h->ev_fork, stream));
    HIP_TRY(hipStreamWaitEvent(h->side, h->ev_fork, 0));
    HIP_TRY(keep_words(step, par, h->side));
    HIP_TRY(hipEventRecord(h->ev_keep[par], h->side));
  }
  // Each member group runs its whole chain -- gather, forward GEMMs, head,
  // loss, backward GEMMs with the fused optimizer -- on its own stream; the
  // groups join at the end.
  HIP_TRY(split());
  for (int hf = 0; hf < ng; ++hf) {
    const hipStream_t s = hs[hf];
    if (h->emb) {
      HIP_TRY(input(hf, s));
    } else if (!h->stream_rows) {
      // the groups' gathers (HBM-bound) run one after another, so a group's
      // forward GEMMs overlap the next group's gather instead of every group
      // waiting for all the groups' gathers at once
      if (hf > 0) HIP_TRY(hipStreamWaitEvent(s, h->ev_gather[hf - 1], 0));
      HIP_TRY(input(hf, s));
      HIP_TRY(hipEventRecord(h->ev_gather[hf], s));
    }
    HIP_TRY(hipStreamWaitEvent(s, h->ev_keep[par], 0));
  }
  // A group's gradient sums run on the side stream once its last producer (its
  // last dX launch, or the head backward for one-block packs) is done: off the
  // group's chain.  Nothing of the step reads the parameters they update after
  // that point.
  auto side_sums = [&](int hf) -> hipError_t {
    hipError_t e = hipEventRecord(h->ev_bias[hf], hs[hf]);
    if (e == hipSuccess) e = hipStreamWaitEvent(h->side, h->ev_bias[hf], 0);
    return e != hipSuccess ? e : grad_sums(hf, false, h->side);
  };
  for (int l = 1; l <= c.L; ++l)
    for (int hf = 0; hf < ng; ++hf) HIP_TRY(forward(hf, l, hs[hf]));
  for (int hf = 0; hf < ng; ++hf) {
    HIP_TRY(head(hf, hs[hf]));
    if (c.L == 1) HIP_TRY(side_sums(hf));
  }
  // the next step's keep words go to the other buffer (last read by the
  // previous step's forward pass) while this step's backward runs
  HIP_TRY(hipEventRecord(h->ev_fork, stream));
  HIP_TRY(hipStreamWaitEvent(h->side, h->ev_fork, 0));
  HIP_TRY(keep_words(step + 1, par ^ 1, h->side));
  HIP_TRY(hipEventRecord(h->ev_keep[par ^ 1], h->side));
  h->keep_ready = step + 1;
  for (int l = c.L; l >= 1; --l)
    for (int hf = 0; hf < ng; ++hf) {
      const hipStream_t s = hs[hf];
      // dX_l reads W_l, so it runs before the weight-gradient GEMM updates W_l in place
      if (l > 1) {
        HIP_TRY(gemm(OP_KMAJ, OP_RMAJ, EPI_DX, h->dx[hf][l - 1], l, s));
        if (l == 2) HIP_TRY(side_sums(hf));
      }
      if (l == 1 && h->emb) HIP_TRY(emb_backward(hf, s));
      // the embedded E is produced in the GEMM
      HIP_TRY(gemm(OP_RMAJ, l == 1 && h->emb ? OP_EMB : OP_RMAJ, EPI_DW, h->dw[hf][l - 1], l, s));
    }
  if (h->muon)
    for (int hf = 0; hf < ng; ++hf) HIP_TRY(muon_step(h, a, hf, hs[hf]));
  HIP_TRY(merge());
  // the gradient sums and the next step's keep words join the caller's stream
  // too, so that a sync of that stream (or later work on it, such as a re-plan
  // that rewrites the member table the keep-word kernel reads) orders after
  // them
  HIP_TRY(hipEventRecord(h->ev_join, h->side));
  HIP_TRY(hipStreamWaitEvent(stream, h->ev_join, 0));
  h->t = step;
  return PACK_OK;
}

}  // extern "C"

namespace {
// The smallest chunk level that holds `rows` rows, or the largest level.
int eval_level(const pack_handle* h, int64_t rows) {
  int lv = 0;
  while (lv + 1 < h->eval_levels && h->eval_rows(lv + 1) >= rows) ++lv;
  return lv;
}

// Forward pass without dropout of every active member over rows r0 ..
// r0 + a.rows_valid - 1 of X (N rows), a chunk of the given level: the first
// layer (on the rows gathered once for all members, or, with embeddings,
// producing each member's embedded rows in the GEMM from the column tables,
// which the caller has built), then the hidden layers; the last hidden
// activations are left in H for the head.
hipError_t eval_forward(pack_handle* h, GemmArgs a, const float* X, int64_t N, int64_t r0, int level,
                        hipStream_t stream) {
  const pack_config& c = h->cfg;
  const int R = h->eval_rows(level);
  h->last_rows = R;
  h->last_valid = a.rows_valid;
  hipError_t e = hipSuccess;
  if (!h->emb)
    e = launch_gather(h->prec, X, N, c.d_in, h->Pin, nullptr, c.B, r0, a.rows_valid, 1, R, h->b.H0, nullptr, stream);
  for (int l = 1; l <= c.L && e == hipSuccess; ++l) {
    GemmArgs al = for_launch(a, h->ev[level][l - 1]);
    al.layer = l;
    const OpKind ak = l == 1 && h->emb ? OP_EMB : OP_KMAJ;
    if (ak == OP_EMB) set_emb(h, al, X, N, nullptr, r0);
    e = launch_gemm(h->prec, ak, OP_KMAJ, EPI_FWD_EVAL, al, stream);
  }
  return e;
}
}  // namespace

extern "C" {

int pack_eval_members(pack_handle* h, const float* Xv, const void* yv, int64_t Nv, float* pred_out,
                      double* score_out, hipStream_t stream) {
  if (!h) return fail(PACK_EINVAL, "handle is NULL");
  if (!h->bound) return fail(PACK_ESTATE, "pack_bind() has not been called");
  if (!Xv || !yv || !pred_out || !score_out) return fail(PACK_EINVAL, "NULL device pointer");
  if (Nv < 1) return fail(PACK_EINVAL, "Nv=%lld must be positive", (long long)Nv);
  if (h->active_ids.empty()) return fail(PACK_ESTATE, "no member is active");
  const pack_config& c = h->cfg;
  const int nact = (int)h->active_ids.size();
  GemmArgs a = base_args(h);
  if (h->emb) HIP_TRY(emb_tables(h, h->b.d_active, h->active_ids, stream));
  for (int64_t r0 = 0; r0 < Nv;) {
    const int lv = eval_level(h, Nv - r0), R = h->eval_rows(lv);
    a.rows_valid = (int)std::min({(int64_t)R, Nv - r0, h->eval_cap});
    HIP_TRY(eval_forward(h, a, Xv, Nv, r0, lv, stream));
    HIP_TRY(launch_head_fwd(h->prec, h->task, kHeadEval, h->b.H, h->b.theta, h->b.d_mem, nact, h->Bp, R, c.d_out,
                            yv, nullptr, c.B, a.rows_valid, r0, Nv, nullptr, nullptr, pred_out, nullptr,
                            h->b.d_active, stream));
    r0 += a.rows_valid;
  }
  HIP_TRY(launch_eval_score(h->task, pred_out, yv, nact, Nv, score_out, h->b.d_active, stream));
  return PACK_OK;
}

int pack_predict(pack_handle* h, const float* X, int64_t N, int32_t mode, float* out, hipStream_t stream) {
  if (!h) return fail(PACK_EINVAL, "handle is NULL");
  if (!h->bound) return fail(PACK_ESTATE, "pack_bind() has not been called");
  if (!X || !out) return fail(PACK_EINVAL, "NULL device pointer");
  if (N < 1) return fail(PACK_EINVAL, "N=%lld must be positive", (long long)N);
  if (mode != PACK_PREDICT_MEMBERS && mode != PACK_PREDICT_ENSEMBLE) return fail(PACK_EINVAL, "unknown mode %d", mode);
  if (h->active_ids.empty()) return fail(PACK_ESTATE, "no member is active");
  const pack_config& c = h->cfg;
  const int nact = (int)h->active_ids.size();
  GemmArgs a = base_args(h);
  if (h->emb) HIP_TRY(emb_tables(h, h->b.d_active, h->active_ids, stream));
  for (int64_t r0 = 0; r0 < N;) {
    const int lv = eval_level(h, N - r0), R = h->eval_rows(lv);
    a.rows_valid = (int)std::min({(int64_t)R, N - r0, h->eval_cap});
    HIP_TRY(eval_forward(h, a, X, N, r0, lv, stream));
    if (mode == PACK_PREDICT_MEMBERS) {
      // member i (i-th active id) writes rows r0.. of out[i, :, :]
      HIP_TRY(launch_head_fwd(h->prec, h->task, kHeadPredict, h->b.H, h->b.theta, h->b.d_mem, nact, h->Bp, R,
                              c.d_out, nullptr, nullptr, c.B, a.rows_valid, r0, N, nullptr, nullptr, out,
                              nullptr, h->b.d_active, stream));
    } else {
      // the chunk's member predictions go to the dY buffer ([K, R, d_out]), then their mean to out
      HIP_TRY(launch_head_fwd(h->prec, h->task, kHeadPredict, h->b.H, h->b.theta, h->b.d_mem, nact, h->Bp, R,
                              c.d_out, nullptr, nullptr, c.B, a.rows_valid, 0, R, nullptr, nullptr, h->b.dY,
                              nullptr, h->b.d_active, stream));
      HIP_TRY(launch_ensemble_mean(h->b.dY, nact, R, a.rows_valid, c.d_out, r0, out, stream));
    }
    r0 += a.rows_valid;
  }
  return PACK_OK;
}

int pack_status(pack_handle* h, uint32_t* flags, hipStream_t stream) {
  if (!h || !flags) return fail(PACK_EINVAL, "NULL argument");
  if (!h->bound) return fail(PACK_ESTATE, "pack_bind() has not been called");
  uint32_t v = 0;
  HIP_TRY(hipMemcpyAsync(&v, h->b.status, sizeof(v), hipMemcpyDeviceToHost, stream));
  HIP_TRY(hipStreamSynchronize(stream));
  if (v) {
    const uint32_t zero = 0;
    HIP_TRY(hipMemcpyAsync(h->b.status, &zero, sizeof(zero), hipMemcpyHostToDevice, stream));
    HIP_TRY(hipStreamSynchronize(stream));
  }
  *flags = v;
  return PACK_OK;
}

static_assert(kMapRows == PACK_BIND_DATA_MAX_B, "the weight-gradient kernels' row table holds a whole batch");

int pack_bind_data(pack_handle* h, const float* X, int64_t N, void* xb, size_t xb_bytes, hipStream_t stream) {
  if (!h) return fail(PACK_EINVAL, "handle is NULL");
  if (!h->bound) return fail(PACK_ESTATE, "pack_bind() has not been called");
  if (!X) {  // unbind: the batch gather feeds the first layer again
    h->stream_rows = false;
    h->data_X = nullptr;
    h->data_N = 0;
    h->xb = nullptr;
    return upload_plan(h, stream);
  }
  if (h->prec != Prec::BF16 || h->emb)
    return fail(PACK_EINVAL, "pack_bind_data needs a bf16 pack without feature embeddings");
  if (N < 1 || !xb) return fail(PACK_EINVAL, "N must be positive and xb set");
  if (h->cfg.B > kMapRows) return fail(PACK_EINVAL, "streamed rows take batches of at most %d rows", kMapRows);
  const size_t need = (size_t)N * h->Pin * 2;
  if (xb_bytes < need) return fail(PACK_EINVAL, "xb has %zu bytes, %zu needed", xb_bytes, need);
  if (reinterpret_cast<uintptr_t>(xb) % 16) return fail(PACK_EINVAL, "xb must be 16-byte aligned");
  if (need + 16 >= ((size_t)1 << 31))
    return fail(PACK_EINVAL, "N x d_in too large for streamed rows (%zu bytes; at most 2 GiB)", need);
  HIP_TRY(launch_rows_to_bf16(X, N, h->cfg.d_in, h->Pin, xb, stream));
  h->stream_rows = true;
  h->data_X = X;
  h->data_N = N;
  h->xb = xb;
  return upload_plan(h, stream);  // the first layer's descriptors read xb through the batch indices
}

int pack_stream_copy(const void* src, void* dst, size_t bytes, hipStream_t stream) {
  if (!src || !dst) return fail(PACK_EINVAL, "NULL device pointer");
  if (bytes % 16 || reinterpret_cast<uintptr_t>(src) % 16 || reinterpret_cast<uintptr_t>(dst) % 16)
    return fail(PACK_EINVAL, "bytes and both addresses must be multiples of 16");
  if (bytes == 0) return PACK_OK;
  HIP_TRY(launch_stream_copy(src, dst, (int64_t)(bytes / 16), stream));
  return PACK_OK;
}

int pack_select_workspace_size(int32_t C, int64_t Nv, size_t* bytes) {
  if (!bytes || C < 1 || Nv < 1) return fail(PACK_EINVAL, "C and Nv must be positive");
  const size_t nblk = (size_t)select_blocks(Nv);
  *bytes = (size_t)round_up(Nv * 8, 256) + (size_t)round_up((int64_t)(C * nblk * 8), 256) + 256 + 256;
  return PACK_OK;
}

extern "C++" {
int tabpack::select_with_scratch(pack_handle* h, const float* cand, const void* yv, int32_t C, int64_t Nv,
                                 int32_t m_ens, void* work, size_t work_bytes, int32_t* sel_out, int32_t* n_sel_out,
                                 double* score_out, hipStream_t stream) {
  if (!h) return fail(PACK_EINVAL, "handle is NULL");
  if (!cand || !yv || !work || !n_sel_out || !score_out || (m_ens > 0 && !sel_out))
    return fail(PACK_EINVAL, "NULL device pointer");
  if (C < 1 || C > 65535 || Nv < 1 || m_ens < 0)
    return fail(PACK_EINVAL, "need 1 <= C <= 65535, Nv >= 1 and m_ens >= 0");
  size_t need = 0;
  pack_select_workspace_size(C, Nv, &need);
  if (work_bytes < need) return fail(PACK_EINVAL, "select workspace has %zu bytes, %zu needed", work_bytes, need);
  if (reinterpret_cast<uintptr_t>(work) % 256) return fail(PACK_EINVAL, "select workspace must be 256-byte aligned");
  const int nblk = select_blocks(Nv);
  char* w = static_cast<char*>(work);
  double* sum = reinterpret_cast<double*>(w);
  double* partial = reinterpret_cast<double*>(w + round_up(Nv * 8, 256));
  int32_t* state = reinterpret_cast<int32_t*>(w + round_up(Nv * 8, 256) + round_up((int64_t)C * nblk * 8, 256));
  double* best = reinterpret_cast<double*>(reinterpret_cast<char*>(state) + 256);
  HIP_TRY(launch_select_init(sum, Nv, state, best, n_sel_out, score_out, stream));
  const int iters = std::min(m_ens, C);
  for (int it = 0; it < iters; ++it)
    HIP_TRY(launch_select_iter(h->task, cand, yv, C, Nv, m_ens, sum, partial, nblk, state, best, sel_out, stream));
  HIP_TRY(launch_select_final(state, best, n_sel_out, score_out, stream));
  return PACK_OK;
}
}  // extern "C++"

int pack_select(pack_handle* h, const float* cand, const void* yv, int32_t C, int64_t Nv, int32_t m_ens,
                void* work, size_t work_bytes, int32_t* sel_out, int32_t* n_sel_out, double* score_out,
                hipStream_t stream) {
  return select_with_scratch(h, cand, yv, C, Nv, m_ens, work, work_bytes, sel_out, n_sel_out, score_out, stream);
}

extern "C++" int tabpack::set_error(int code, const char* msg) { return fail(code, "%s", msg); }

int pack_member_param_count(const pack_handle* h, int32_t member, int64_t* count) {
  int rc = check_member(h, member);
  if (rc) return rc;
  if (!count) return fail(PACK_EINVAL, "count is NULL");
  *count = dense_count(h, member);
  return PACK_OK;
}

namespace {
int copy_member(pack_handle* h, int k, const float* dev_base, float* host_out) {
  const int64_t b = member_span_begin(h, k), e = member_span_end(h, k);
  std::vector<float> tmp((size_t)(e - b));
  if (dev_base) {
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(tmp.data(), dev_base + b, tmp.size() * 4, hipMemcpyDeviceToHost));
  } else {
    std::memcpy(tmp.data(), h->theta_host.data() + b, tmp.size() * 4);
  }
  for_each_dense(h, k, [&](int64_t di, int64_t pi) { host_out[di] = tmp[(size_t)(pi - b)]; });
  return PACK_OK;
}
}  // namespace

int pack_get_params(pack_handle* h, int32_t member, float* host_out) {
  int rc = check_member(h, member);
  if (rc) return rc;
  if (!host_out) return fail(PACK_EINVAL, "host_out is NULL");
  return copy_member(h, member, h->bound ? h->b.theta : nullptr, host_out);
}

int pack_set_params(pack_handle* h, int32_t member, const float* host_in) {
  int rc = check_member(h, member);
  if (rc) return rc;
  if (!host_in) return fail(PACK_EINVAL, "host_in is NULL");
  for_each_dense(h, member, [&](int64_t di, int64_t pi) { h->theta_host[(size_t)pi] = host_in[di]; });
  if (h->bound) {
    const int64_t b = member_span_begin(h, member), e = member_span_end(h, member);
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(h->b.theta + b, h->theta_host.data() + b, (size_t)(e - b) * 4, hipMemcpyHostToDevice));
    if (h->prec == Prec::BF16) HIP_TRY(launch_to_shadow(h->b.theta + b, h->b.shadow + b, e - b, 0));
    HIP_TRY(hipDeviceSynchronize());
  }
  return PACK_OK;
}

int pack_get_grads(pack_handle* h, int32_t member, float* host_out) {
  int rc = check_member(h, member);
  if (rc) return rc;
  if (!h->bound) return fail(PACK_ESTATE, "pack_bind() has not been called");
  if (!host_out) return fail(PACK_EINVAL, "host_out is NULL");
  if (!h->cfg.keep_grads) return fail(PACK_ESTATE, "gradients are kept only with pack_config.keep_grads = 1");
  return copy_member(h, member, h->b.grad, host_out);
}

int pack_get_moments(pack_handle* h, int32_t member, float* m_out, float* v_out) {
  int rc = check_member(h, member);
  if (rc) return rc;
  if (!h->bound) return fail(PACK_ESTATE, "pack_bind() has not been called");
  if (!m_out || !v_out) return fail(PACK_EINVAL, "NULL output");
  rc = copy_member(h, member, h->b.m, m_out);
  if (rc) return rc;
  return copy_member(h, member, h->b.v, v_out);
}

int pack_debug_dropout_mask(pack_handle* h, uint64_t step, int32_t layer, int32_t member, uint8_t* dev_out,
                            hipStream_t stream) {
  int rc = check_member(h, member);
  if (rc) return rc;
  if (layer < 1 || layer > h->mem[member].depth)
    return fail(PACK_EINVAL, "layer %d out of [1, %d] for member %d", layer, h->mem[member].depth, member);
  if (!dev_out) return fail(PACK_EINVAL, "dev_out is NULL");
  const Key kd = stream_key(h->cfg.seed, kTagDropout);
  HIP_TRY(launch_dropout_mask(kd.k0, kd.k1, as_u32(step), layer, member, h->mem[member].t, h->cfg.B,
                              h->mem[member].width, dev_out, stream));
  return PACK_OK;
}

int pack_debug_activation(pack_handle* h, int32_t layer, int32_t member, float* host_out) {
  int rc = check_member(h, member);
  if (rc) return rc;
  if (!h->bound) return fail(PACK_ESTATE, "pack_bind() has not been called");
  if (layer < 1 || layer > h->mem[member].depth)
    return fail(PACK_EINVAL, "layer %d out of [1, %d] for member %d", layer, h->mem[member].depth, member);
  if (!host_out) return fail(PACK_EINVAL, "host_out is NULL");
  const Member& m = h->mem[member];
  // blocks of last_rows rows; those past the rows of the pass (never computed by
  // a short evaluation chunk) are zeros, as are those of a member outside it
  const size_t R = (size_t)h->last_rows;
  const size_t n = h->active[member] ? (size_t)std::min(h->cfg.B, h->last_valid) * m.dp : 0;
  const size_t off = ((size_t)(layer - 1) * (h->A / h->Bp) + (size_t)(m.act_off / h->Bp)) * R;
  std::vector<uint8_t> tmp((size_t)h->Bp * m.dp * h->elt());
  HIP_TRY(hipDeviceSynchronize());
  if (n) HIP_TRY(hipMemcpy(tmp.data(), h->b.H + off * h->elt(), n * h->elt(), hipMemcpyDeviceToHost));
  for (int r = 0; r < h->cfg.B; ++r)
    for (int c = 0; c < m.width; ++c) {
      const size_t i = (size_t)r * m.dp + c;
      float val;
      if (h->prec == Prec::BF16) {
        uint16_t b16;
        std::memcpy(&b16, tmp.data() + 2 * i, 2);
        const uint32_t bits = (uint32_t)b16 << 16;
        std::memcpy(&val, &bits, 4);
      } else {
        std::memcpy(&val, tmp.data() + 4 * i, 4);
      }
      host_out[(size_t)r * m.width + c] = val;
    }
  return PACK_OK;
}

int pack_profile_enable(pack_handle* h, int32_t enable) {
  if (!h) return fail(PACK_EINVAL, "handle is NULL");
  HIP_TRY(hipDeviceSynchronize());
  h->prof = enable != 0;
  h->timed.clear();
  h->pool_used = 0;
  h->groups.clear();
  return PACK_OK;
}

int pack_profile_read(pack_handle* h, pack_kernel_stat* out, int32_t max, int32_t* n) {
  if (!h || !n || (max > 0 && !out)) return fail(PACK_EINVAL, "NULL argument");
  std::vector<ProfGroup> g = h->groups;
  for (ProfGroup& x : g) x.launches = 0, x.total_ms = 0.0;
  // launch intervals on a common time base (the first recorded event), to
  // measure each kernel's busy time: the union of its launches' intervals,
  // which differs from the summed durations when launches of concurrent
  // member groups overlap
  std::vector<std::vector<std::pair<double, double>>> iv(g.size());
  for (const TimedLaunch& t : h->timed) {
    HIP_TRY(hipEventSynchronize(t.stop));
    float ms = 0.0f, t0 = 0.0f, t1 = 0.0f;
    HIP_TRY(hipEventElapsedTime(&ms, t.start, t.stop));
    HIP_TRY(hipEventElapsedTime(&t0, h->timed.front().start, t.start));
    HIP_TRY(hipEventElapsedTime(&t1, h->timed.front().start, t.stop));
    g[t.group].launches += 1;
    g[t.group].total_ms += ms;
    iv[t.group].push_back({t0, t1});
  }
  *n = (int32_t)g.size();
  for (int i = 0; i < (int)g.size() && i < max; ++i) {
    pack_kernel_stat& s = out[i];
    std::memset(&s, 0, sizeof s);
    snprintf(s.name, sizeof s.name, "%s", g[i].name.c_str());
    s.kind = g[i].kind;
    s.launches = g[i].launches;
    s.total_ms = g[i].total_ms;
    s.flops = g[i].launches ? g[i].flops / g[i].launches : 0.0;
    s.bytes = g[i].launches ? g[i].bytes / g[i].launches : 0.0;
    std::sort(iv[i].begin(), iv[i].end());
    double busy = 0.0, a = 0.0, b = -1.0;
    for (const auto& x : iv[i]) {
      if (x.first > b) {
        if (b > a) busy += b - a;
        a = x.first;
        b = x.second;
      } else {
        b = std::max(b, x.second);
      }
    }
    if (b > a) busy += b - a;
    s.busy_ms = busy;
  }
  return PACK_OK;
}

}  // extern "C"
