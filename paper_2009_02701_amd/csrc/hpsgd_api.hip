// C-ABI layer: argument validation, the flat parameter layout, the workspace layout and
// the launch plan of one local training step.  Host code only; every arithmetic step runs
// in the kernels declared in kernels.h.
#include "../../include/hpsgd.h"

#include <algorithm>
#include <string>
#include <mutex>
#include <cstring>
#include <memory>
#include <vector>

#include "kernels.h"

using namespace hpsgd;

namespace {

struct Entry {
  std::string name;
  size_t offset;
  int rows, cols;
};

inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// fp32 weight gradients (M x N outputs, contraction over T * B): how many parts the contraction is cut
// into.  A narrow layer's gradient has a few dozen 64 x 64 tiles per worker and a contraction of
// thousands: the parts run side by side, about two workgroups per CU over all K workers (a launch holds two of these products
// and more), and the kernel that applies the update adds them in order.  A part is at least 128 long (four k-tiles: below
// that a part is mostly first loads and epilogue), 256 from a contraction of 832 on, and 1 means the update stays
// in the epilogue.  us per local step, parts of 128 / of 256, over Kd:
//   H = 48, batch 20, 16 workers   520  73.7 / 75.9   720  87.5 / 91.6   800  91.6 / 93.6   840  98.8 / 96.4   900 102.5 / 100.3   1200 122.6 / 120.7
//   H = 110, batch 20, 3 workers   520 104.7 / 106.0  720 131.1 / 131.9  800 140.3 / 140.0  840 145.8 / 144.8  900 153.4 / 152.7   1200 188.4 / 187.4
//   H = 128, batch 20, 8 workers   520 121.5 / 120.0  720 150.4 / 149.0  800 160.0 / 157.7  840 167.0 / 163.1  900 175.3 / 171.4   1200 215.7 / 213.9
// The longer parts want 96 workgroups of them at least (H = 128, batch 20, 2 workers, 72 workgroups: 840 150.6 / 151.6,
// 960 165.1 / 167.0), and products that would then be few tiles, whose form is another one, keep the shorter.
// us per round or local step, three workgroups per CU and parts of 128 / this: H = 48, batch 100, 30 steps, 16 workers 154.9 / 145.8;
// H = 90, 20, 50, 16 181.5 / 175.7; H = 128, 32, 60, 2 layers, 2 workers 403 / 390; H = 110, 60, 40, 2 layers, 3 workers 337 / 329; H = 128, 40, 40, 8
// 193.8 / 191.0; H = 256, 32, 32, 3 212.3 / 210.6; H = 100, 20, 50, 2 layers, 4 298.6 / 297.6.
// Goes by the context's K, not by how many workers a call steps: the cuts of a context are always the same.  (Whether
// dW_hh is cut at all may still depend on the call: where gru_persist_pays sends it to a launch per step.)
int wgrad_splits(int M, int N, int Kd, int K) {
  const long tiles = (long)((M + 63) / 64) * ((N + 63) / 64) * K, tiles32 = (long)((M + 31) / 32) * ((N + 31) / 32) * K;
  long n = (512 + tiles - 1) / tiles;
  if (n > Kd / 128) n = Kd / 128;
  if (n > 16) n = 16;
  if (Kd >= 832 && n > Kd / 256 && tiles * (Kd / 256) >= 96 && tiles32 * (Kd / 256) > 256) n = Kd / 256;
  return n < 2 ? 1 : (int)n;
}
// An input gradient of the head (M x N outputs, contraction over the classes: thousands, where the output
// has a few dozen tiles): the parts of its contraction, so that all K workers' tiles come to about two per
// CU; at least min_part long, 1 if the tiles already cover half the chip.
int dx_splits(int M, int N, int Kd, int K, int tile, int min_part) {
  const long tiles = (long)((M + tile - 1) / tile) * ((N + tile - 1) / tile) * K;
  long n = (512 + tiles - 1) / tiles;
  if (n > Kd / min_part) n = Kd / min_part;
  if (n > 16) n = 16;
  return tiles >= 256 || n < 2 ? 1 : (int)n;
}
// length of a part: whole k-tiles
int wgrad_part(int Kd, int splits) { return ((Kd + splits - 1) / splits + 31) / 32 * 32; }

struct Region {  // one workspace buffer: K slices of `stride` floats
  size_t offset = 0, stride = 0;
};

}  // namespace

struct hpsgd_ctx {
  hpsgd_model_desc d;
  int K;
  std::vector<Entry> entries;
  size_t P = 0;
  size_t ws_floats = 0;
  // workspace regions (floats)
  Region grad, xe, gx, dgh, gh, D, dx, logits, rowloss, wt;
  Region psync;                 // abort word and flag words of the resident-weight recurrence kernels
  Region dwp, dbp;              // their partial sums of dW_hh and of the bias gradients, one per 32-row batch tile
  Region dxp;                   // partial sums of the head's input gradient (dx_splits)
  Region dwip;                  // partial sums of a layer's weight gradients whose contraction is cut (wgrad_splits)
  Region hb, dghb, dgxb;        // bf16 copies of h, dgh and dgx (bf16 precision only)
  Region hx, dghx;              // h and dgh as the resident-weight launches exchange them (fragment-major)
  // transposed bf16 copies that bring the weight-gradient and input-gradient GEMMs into the
  // contraction-contiguous form (bf16 precision only); sizes in floats = bf16 count / 2
  Region dgxT, dghT, xT, dlogT, wihT, woT;
  Region xb, wob, dlogb;  // row-major bf16 copies: layer-0 input, head.W, dlogits
  Region colpart;               // per block of logits rows: column sums of the logit gradient
  std::vector<Region> hsT;
  std::vector<Region> whhT;     // per layer: transposed bf16 W_hh, made in the forward pass
  std::vector<Region> whhb, wihbl;  // per layer: row-major bf16 W_hh and W_ih
  // Marks left by hpsgd_prepare_replicas / hpsgd_prepare_clones, one per workspace (a schedule with
  // two generations of buffers prepares one while the other steps): the bf16 copies of these
  // replicas' weights are in that workspace.  clone_src (prepare_clones): ONE set of copies, made
  // from this model, serves every worker; head_done: the head's copies are among them (else the
  // step makes them from clone_src right before the logits GEMM).
  struct Mark { const float* rin; const float* ws; size_t stride; const float* clone_src; bool head_done; };
  std::vector<Mark> marks;
  void set_mark(const Mark& m) {
    drop_mark(m.ws);
    if (marks.size() >= 4) marks.erase(marks.begin());
    marks.push_back(m);
  }
  void drop_mark(const float* ws) {
    for (size_t i = 0; i < marks.size();)
      if (marks[i].ws == ws) marks.erase(marks.begin() + i);
      else ++i;
  }
  // the mark of this workspace if it was made for exactly these replicas; the workspace's mark is
  // gone afterwards either way (the step rewrites the copies, and changes the weights)
  bool take_mark(const float* rin, const float* ws, size_t stride, Mark& out) {
    bool found = false;
    for (const Mark& m : marks)
      if (m.ws == ws && m.rin == rin && m.stride == stride) { out = m; found = true; }
    drop_mark(ws);
    return found;
  }
  std::vector<Region> hs, sv;   // per GRU layer
  std::vector<Region> act;      // per MLP layer output
  std::vector<Region> dact;     // per MLP hidden layer: gradient w.r.t. its output
  // optional per-role kernel timing (benchmarks): event pairs recorded around launches
  // optional second stream for work that can run beside the recurrence, and the two events
  // that order it against the caller's stream
  hipStream_t aux = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  // bf16 language model: the widths of every internal buffer of a resident step - batch and embedding
  // width rounded up to 8, hidden width to 32, logit rows to 8 - so that every product takes its bf16
  // operands in whole 16-byte pieces and every recurrence whole blocks of units, whatever the model's
  // sizes.  What lies beyond the model's own sizes is zero; the model's arrays (parameters, tokens,
  // labels) keep their layout and are met where they are read (copies, biases, embedding rows) and where
  // they are updated.  padded == false: the sizes are the model's own.
  bool padded = false;
  int Bp = 0, Hp = 0, Ep = 0, Vp = 0;
  bool use_padded() const { return padded && resident; }
  bool solo_b = false;          // the same for the bf16 padded layout
  int prow = 0, prow_b = 32;    // batch rows per workgroup of the resident-weight launches, fp32 (0: not taken) and bf16
  bool solo = false;            // fp32 and narrow: a layer's recurrence needs no exchange (gru_solo.hip)
  bool stack = false;           // ... and both layers run in one launch: the buffers of the upper one are its own
  bool stack_b = false;         // the same for the bf16 padded layout
  Region gx_up, dgh_up, dx_up, dbp_up, hb_lo, dg4_up;
  // 0: the layout that the fastest forms need.  1: layers one after the other.  2: no padding, no split contractions, none of the forms whose
  // saved state is larger than the model's own sizes.  3: no resident-weight recurrence in fp32 either.
  // `small`: the same model in the first such layout that fits the static array, where layout 0 does not.
  int lean = 0;
  std::unique_ptr<hpsgd_ctx> small;
  // Row pitch of a bf16 copy of a weight matrix of `w` columns: whole lines of 128 bytes.  At 1344 bytes (H = 672) every second row of a k-tile
  // lies in two lines, and a CU's loads from the L2 arrive at 82 KB/us instead of 125.  us per local step, rows close together / on lines of
  // their own: H = 650, 4 workers 1029 / 1018 (a round 1089 / 1080), H = 800, 4 workers 747 / 739, H = 480, 8 workers 905 / 900; H = 990, 8 workers 1209 / 1209
  // (no gain there).  Narrower than 128 a pitch would be up to twice the row.  A layout that has to be
  // small keeps the rows together.
  long copy_pitch(long w) const { return lean || w < 128 ? w : (w + 63) / 64 * 64; }
  long wih_pitch(int l) const { return stack_b && l == 1 ? Hp : copy_pitch(l == 0 ? Ep : Hp); }
  long head_pitch() const { return copy_pitch(Hp); }
  int wgrad_parts(int M, int N, int Kd) const { return lean > 1 ? 1 : wgrad_splits(M, N, Kd, K); }
  bool resident = true;         // fp32 recurrence: one launch per run of time steps when supported
  bool device_scope = false;    // resident-weight launches exchange at device scope even where an XCD's L2 would do
  static constexpr unsigned kSpinLimit = 1u << 20;
  unsigned spin_limit = kSpinLimit;  // bound of every wait inside those launches
  // ... inside the launches of two narrow layers: these wait only for workgroups that run, and a model that takes them steps with any limit
  // as it does layer by layer, without a wait.  (0 is the test's limit: every wait fails.)
  unsigned link_limit() const { return spin_limit ? std::max(spin_limit, kSpinLimit) : 0u; }
  size_t last_commit_params = 0;  // parameters per worker that the commit kernel handled last step
  int last_resident = 0, last_xproj = 0, last_dw = 0;  // GRU layers of the last step, see hpsgd_recurrence_info
  unsigned timer_mask = 0;
  bool timer_nested = false;    // an enclosing scope already brackets the current launches
  struct Stamp { int role; int launches; hipEvent_t a, b; };
  std::vector<Stamp> stamps;
  std::vector<hipEvent_t> free_events;
  double role_ms[HPSGD_ROLE_COUNT] = {0};
  long role_launches[HPSGD_ROLE_COUNT] = {0};
  // per-kernel timing: event pairs recorded by the launchers themselves (KernelTimer)
  unsigned kernel_mask = 0;
  struct KStamp { int kid; double work; hipEvent_t a, b; int launches; };
  std::vector<KStamp> kstamps;
  double kernel_ms[HPSGD_KERNEL_COUNT] = {0}, kernel_work[HPSGD_KERNEL_COUNT] = {0};
  long kernel_launches[HPSGD_KERNEL_COUNT] = {0};

  // entries of the flat layout by role, filled once by build_layout: the launch plan of a step looks
  // nothing up by name
  struct LayerIdx { int wih, whh, bih, bhh; };
  std::vector<LayerIdx> lidx;       // per GRU layer
  std::vector<int> fc_w, fc_b;      // per MLP layer
  int i_embed = -1, i_head_w = -1, i_head_b = -1;
  size_t eoff(int entry) const { return entries[entry].offset; }

  // `small` steps in its owner's place: the owner's settings and timers go with it, and come back
  void lend(hpsgd_ctx& o) {
    o.aux = aux, o.ev_fork = ev_fork, o.ev_join = ev_join;
    o.resident = resident, o.device_scope = device_scope, o.spin_limit = spin_limit;
    o.timer_mask = timer_mask, o.kernel_mask = kernel_mask;
    o.stamps.swap(stamps), o.kstamps.swap(kstamps), o.free_events.swap(free_events);
  }
  void take_back(hpsgd_ctx& o) {
    o.stamps.swap(stamps), o.kstamps.swap(kstamps), o.free_events.swap(free_events);
    last_commit_params = o.last_commit_params;
    last_resident = o.last_resident, last_xproj = o.last_xproj, last_dw = o.last_dw;
  }


  // slices back to back (partial sums: the adding kernel reads part p of worker k at (k * parts + p) * n)
  Region alloc_packed(size_t per_worker) {
    Region r;
    r.stride = per_worker;
    r.offset = ws_floats;
    ws_floats += round_up(per_worker * (size_t)K, 64);
    return r;
  }
  Region alloc(size_t per_worker) {
    Region r;
    r.stride = round_up(per_worker, 64);
    r.offset = ws_floats;
    ws_floats += r.stride * (size_t)K;
    return r;
  }
};

namespace {

void add_entry(hpsgd_ctx* c, const std::string& name, int rows, int cols) {
  c->entries.push_back({name, c->P, rows, cols});
  c->P += (size_t)rows * (size_t)cols;
}

int build_layout(hpsgd_ctx* c) {
  const hpsgd_model_desc& d = c->d;
  const long big = 1L << 30;
  if (d.kind == HPSGD_GRU_CLASSIFIER || d.kind == HPSGD_GRU_LM) {
    const bool lm = d.kind == HPSGD_GRU_LM;
    if (d.layers < 1 || d.layers > 16 || d.hidden < 1 || d.seq_len < 1 || d.batch < 1) return HPSGD_ESHAPE;
    if (lm ? (d.vocab < 2 || d.embed < 1) : (d.input < 1 || d.classes < 2)) return HPSGD_ESHAPE;
    if ((long)d.seq_len * d.batch * 4L * d.hidden >= big) return HPSGD_ESHAPE;
    if (d.seq_len > 65535) return HPSGD_ESHAPE;
    int width = lm ? d.embed : d.input;
    const int classes = lm ? d.vocab : d.classes;
    if ((long)d.seq_len * d.batch * (long)classes >= big) return HPSGD_ESHAPE;
    if (lm) {
      c->i_embed = (int)c->entries.size();
      add_entry(c, "embed.E", d.vocab, d.embed);
    }
    for (int l = 0; l < d.layers; ++l) {
      const std::string p = "l" + std::to_string(l);
      const int e0 = (int)c->entries.size();
      c->lidx.push_back({e0, e0 + 1, e0 + 2, e0 + 3});
      add_entry(c, p + ".W_ih", 3 * d.hidden, width);
      add_entry(c, p + ".W_hh", 3 * d.hidden, d.hidden);
      add_entry(c, p + ".b_ih", 3 * d.hidden, 1);
      add_entry(c, p + ".b_hh", 3 * d.hidden, 1);
      width = d.hidden;
    }
    c->i_head_w = (int)c->entries.size();
    add_entry(c, "head.W", classes, d.hidden);
    c->i_head_b = (int)c->entries.size();
    add_entry(c, "head.b", classes, 1);

    c->padded = c->lean <= 1 && lm && d.prec == HPSGD_BF16_MFMA && d.vocab >= 4 && d.vocab <= 1024 * 10 && d.hidden <= 1024 &&
                (long)d.seq_len * (long)round_up(d.batch, 8) * (long)round_up(4 * d.hidden > d.vocab ? 4 * (d.hidden + 31) : d.vocab, 8) < big;
    c->Bp = c->padded ? (int)round_up(d.batch, 8) : d.batch;
    c->Hp = c->padded ? (int)round_up(d.hidden, 32) : d.hidden;
    c->Ep = c->padded ? (int)round_up(d.embed, 8) : lm ? d.embed : d.input;
    c->Vp = c->padded ? (int)round_up(classes, 8) : classes;
    const size_t Bi = c->Bp, TB = (size_t)d.seq_len * Bi, H = c->Hp;
    c->solo_b = c->padded && gru_solo_bf16_supported(c->Bp, c->Hp);
    c->stack_b = !c->lean && c->solo_b && gru_stack_bf16_supported(c->Bp, c->Hp, d.seq_len, d.layers, c->K);
    c->solo = c->lean <= 1 && d.prec != HPSGD_BF16_MFMA && gru_solo_supported(d.batch, d.hidden);
    c->stack = !c->lean && c->solo && gru_stack_supported(d.batch, d.hidden, d.seq_len, d.layers, c->K, lm);
    c->grad = c->alloc(c->P);
    if (lm) c->xe = c->alloc(TB * c->Ep);
    for (int l = 0; l < d.layers; ++l) {
      c->hs.push_back(c->alloc((TB + Bi) * H));
      const size_t sv_solo = c->solo ? gru_solo_saved_words(d.batch, d.hidden, d.seq_len, c->K) : 0;
      c->sv.push_back(c->alloc(sv_solo > TB * 4 * H ? sv_solo : TB * 4 * H));
    }
    c->gx = c->alloc(TB * 3 * H);
    c->dgh = c->alloc(TB * 3 * H);
    const size_t dbp_solo = c->solo     ? (size_t)gru_solo_row_tiles(d.batch, d.hidden, c->K) * 6 * H
                            : c->solo_b ? (size_t)gru_solo_bf16_row_tiles((int)Bi, c->K) * 6 * H
                                        : 0;
    c->gh = c->alloc(dbp_solo > Bi * 3 * H ? dbp_solo : Bi * 3 * H);
    c->D = c->alloc(Bi * H);
    c->wt = c->alloc(3 * H * H);
    // batch rows per workgroup of the fp32 resident-weight launches (0: they do not take this layer)
    c->prow = c->solo || d.prec == HPSGD_BF16_MFMA || c->lean == 3 || (c->lean > 1 && d.hidden % 16 != 0)
                  ? 0
                  : gru_persist_rows(d.batch, d.hidden, c->K);
    c->prow_b = c->lean > 1 ? 32 : gru_persist_bf16_rows((int)Bi, (int)H, c->K);
    if (c->stack || c->stack_b) {
      c->psync = c->alloc(c->stack ? gru_stack_sync_words((int)Bi, 1) : gru_stack_bf16_sync_words((int)Bi, 1));
      c->gx_up = c->alloc(TB * 3 * H);
      if (c->stack) c->dgh_up = c->alloc(TB * 3 * H);
      c->dx_up = c->alloc(TB * H);
      c->dbp_up = c->alloc_packed(dbp_solo);
    }
    // (no other step of a narrow model waits for another workgroup)
    if (!c->solo && !c->solo_b) c->psync = c->alloc(gru_persist_sync_words((int)Bi, 1, c->prow ? c->prow : c->prow_b));
    if (dbp_solo) {  // (in the place of `gh`, which a step of such launches does not use)
      c->dbp.offset = c->gh.offset;
      c->dbp.stride = dbp_solo;
    } else if (c->prow) c->dbp = c->alloc_packed(((Bi + c->prow - 1) / c->prow) * 6 * H);
    else if (d.prec == HPSGD_BF16_MFMA && gru_fused_bf16_supported((int)H)) c->dbp = c->alloc_packed(((Bi + c->prow_b - 1) / c->prow_b) * 6 * H);
    if (c->prow && gru_persist_dw_supported((int)H)) c->dwp = c->alloc_packed(((Bi + c->prow - 1) / c->prow) * 3 * H * H);
    if (d.prec != HPSGD_BF16_MFMA) {
      size_t most = 0;  // over the layers, which follow each other (or, in one launch, do not): the parts of dW_ih, then those of dW_hh
      for (int l = 0; l < d.layers; ++l) {
        const size_t win = l > 0 ? H : (size_t)(lm ? d.embed : d.input);
        const int si = c->wgrad_parts((int)(3 * H), (int)win, (int)TB), sh = c->wgrad_parts((int)(3 * H), (int)H, (int)TB);
        const size_t n = (si > 1 ? si * 3 * H * win : 0) + (sh > 1 ? sh * 3 * H * H : 0);
        if (c->stack) most += n;
        else if (n > most) most = n;
      }
      if (most) c->dwip = c->alloc_packed(most);
    }
    if (c->prow) {
      c->hx = c->alloc((size_t)(d.seq_len + 1) * gru_persist_exchange_words(d.batch, d.hidden, 1));
      c->dghx = c->alloc((size_t)d.seq_len * gru_persist_exchange_words(d.batch, d.hidden, 3));
    }
    if (d.prec == HPSGD_BF16_MFMA) {
      c->hb = c->alloc(((TB + Bi) * H + 1) / 2);
      c->dghb = c->alloc((TB * 3 * H + 1) / 2);
      c->hx = c->alloc(((size_t)(d.seq_len + 1) * gru_persist_bf16_exchange_elems((int)Bi, (int)H) + 1) / 2);
      // (the launches without an exchange keep their gate gradients there, r | z | n | q per row)
      const size_t dg4 = TB * 4 * H, dgx_elems = (size_t)d.seq_len * gru_persist_bf16_exchange_elems((int)Bi, (int)(3 * H));
      c->dghx = c->alloc(((c->solo_b && dg4 > dgx_elems ? dg4 : dgx_elems) + 1) / 2);
      if (c->stack_b) {
        c->dg4_up = c->alloc(((dg4 > dgx_elems ? dg4 : dgx_elems) + 1) / 2);
        c->hb_lo = c->alloc(((TB + Bi) * H + 1) / 2);
      }
      c->dgxb = c->alloc((TB * 3 * H + 1) / 2);
      const size_t TBp = round_up(TB, 64), TB1p = round_up(TB + Bi, 64);
      const size_t win0 = c->Ep;
      const size_t wmax = win0 > H ? win0 : H;
      c->dgxT = c->alloc(3 * H * TBp / 2);
      c->dghT = c->alloc(3 * H * TBp / 2);
      c->xT = c->alloc(win0 * TBp / 2);
      for (int l = 0; l < d.layers; ++l) {
        c->hsT.push_back(c->alloc(H * TB1p / 2));
        c->whhT.push_back(c->alloc((3 * H * H + 1) / 2));
        c->whhb.push_back(c->alloc((3 * H * H + 1) / 2));
        c->wihbl.push_back(c->alloc((c->wih_pitch(l) * 3 * H + 1) / 2));
      }
      const size_t nr = lm ? TB : Bi, Vi = c->Vp;
      // the transposed logit gradients, or (the head of bf16 operands) the loss kernel's column sums
      const size_t n_dlogT = Vi * round_up(nr, 64) / 2, n_colpart = softmax_ce_bf16_row_blocks((int)nr) * round_up(Vi, 8);
      c->dlogT = c->alloc(n_dlogT > n_colpart ? n_dlogT : n_colpart);
      c->colpart = c->dlogT;
      c->wihT = c->alloc(wmax * 3 * H / 2);
      c->woT = c->alloc(H * round_up(classes, 64) / 2);
      c->xb = c->alloc((TB * win0 + 1) / 2);
      c->wob = c->alloc((round_up(Vi, 8) * c->head_pitch() + 1) / 2);
      c->dlogb = c->alloc((nr * round_up(classes, 64) + 1) / 2);
    }
    size_t wmax = H;
    if (lm && (size_t)c->Ep > wmax) wmax = c->Ep;
    c->dx = c->alloc(TB * wmax);
    const size_t nrows = lm ? TB : Bi;
    c->logits = c->alloc(nrows * round_up(c->Vp, 8));
    {
      const bool bfp = d.prec == HPSGD_BF16_MFMA;
      const int ns = dx_splits((int)nrows, (int)H, bfp ? (int)round_up(classes, 8) : classes, c->K, bfp ? 128 : 64, bfp ? 512 : 256);
      if (ns > 1 && c->lean <= 1) c->dxp = c->alloc_packed((size_t)ns * nrows * H);
    }
    c->rowloss = c->alloc(nrows);
  } else if (d.kind == HPSGD_MLP) {
    if (d.n_mlp_dims < 2 || d.n_mlp_dims > HPSGD_MAX_MLP_DIMS || d.batch < 1) return HPSGD_ESHAPE;
    for (int i = 0; i < d.n_mlp_dims; ++i)
      if (d.mlp_dims[i] < 1 || (long)d.mlp_dims[i] * d.batch >= big) return HPSGD_ESHAPE;
    if (d.mlp_dims[d.n_mlp_dims - 1] < 2) return HPSGD_ESHAPE;
    for (int i = 0; i + 1 < d.n_mlp_dims; ++i) {
      const std::string p = "fc" + std::to_string(i);
      c->fc_w.push_back((int)c->entries.size());
      add_entry(c, p + ".W", d.mlp_dims[i + 1], d.mlp_dims[i]);
      c->fc_b.push_back((int)c->entries.size());
      add_entry(c, p + ".b", d.mlp_dims[i + 1], 1);
    }
    c->grad = c->alloc(c->P);
    for (int i = 1; i < d.n_mlp_dims; ++i) c->act.push_back(c->alloc((size_t)d.batch * d.mlp_dims[i]));
    for (int i = 1; i + 1 < d.n_mlp_dims; ++i) c->dact.push_back(c->alloc((size_t)d.batch * d.mlp_dims[i]));
    c->rowloss = c->alloc(d.batch);
  } else {
    return HPSGD_EINVAL;
  }
  return HPSGD_OK;
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

inline bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  return a0 < b0 + nb && b0 < a0 + na;
}

// Records an event pair around the launches issued while it is alive, if its role is timed.
struct TimerScope {
  hpsgd_ctx* c;
  hipStream_t s;
  int idx = -1;
  static hipEvent_t get(hpsgd_ctx* c) {
    hipEvent_t e = nullptr;
    if (!c->free_events.empty()) {
      e = c->free_events.back();
      c->free_events.pop_back();
    } else if (hipEventCreate(&e) != hipSuccess) {
      e = nullptr;
    }
    return e;
  }
  // launches: how many kernel launches the pair brackets (a whole time loop is bracketed by
  // one pair: an event record between two dependent launches costs far more than the launch)
  TimerScope(hpsgd_ctx* c_, int role, hipStream_t s_, int launches = 1) : c(c_), s(s_) {
    if (launches <= 0 || !(c->timer_mask & (1u << role)) || c->timer_nested) return;
    hipEvent_t a = get(c), b = get(c);
    if (!a || !b) return;
    c->stamps.push_back({role, launches, a, b});
    idx = (int)c->stamps.size() - 1;
    (void)hipEventRecord(a, s);
  }
  ~TimerScope() {
    if (idx >= 0) (void)hipEventRecord(c->stamps[idx].b, s);
  }
  bool active() const { return idx >= 0; }
};

// The context whose local step the calling thread is issuing (KernelTimer looks here).
thread_local hpsgd_ctx* t_step_ctx = nullptr;
struct StepCtxScope {
  hpsgd_ctx* prev;
  explicit StepCtxScope(hpsgd_ctx* c) : prev(t_step_ctx) { t_step_ctx = c; }
  ~StepCtxScope() { t_step_ctx = prev; }
};

// inside run_step: `role` names what the next launches are for
#define HIP_TRY(expr)                              \
  do {                                             \
    TimerScope ts_(c, role, s);                    \
    if ((expr) != hipSuccess) return HPSGD_EHIP;   \
  } while (0)

// GEMM helper: C = op(A) op(B) for `groups` workers.
GemmDesc gemm_desc(int groups, int bf16, int M, int N, int Kd, const float* A, long lda,
                   long sA, int tA, const float* B, long ldb, long sB, int tB, float* C, long ldc, long sC,
                   int epi, const float* aux, long sAux, int background = 0, float alpha = 0.f, int splits = 1, int Kall = 0) {
  GemmDesc g;
  g.splits = splits;
  g.Kall = Kall;
  g.background = background;
  g.alpha = alpha;
  g.A = A; g.lda = lda; g.strideA = sA; g.transA = tA;
  g.B = B; g.ldb = ldb; g.strideB = sB; g.transB = tB;
  g.C = C; g.ldc = ldc; g.strideC = sC;
  g.aux = aux; g.strideAux = sAux;
  g.M = M; g.N = N; g.Kd = Kd; g.groups = groups;
  g.workers = t_step_ctx ? t_step_ctx->K : groups;
  g.epilogue = epi; g.bf16 = bf16;
  return g;
}
int gemm(hipStream_t s, int groups, int bf16, int M, int N, int Kd, const float* A, long lda,
         long sA, int tA, const float* B, long ldb, long sB, int tB, float* C, long ldc, long sC,
         int epi, const float* aux, long sAux, int background = 0, float alpha = 0.f, int splits = 1, int Kall = 0) {
  const GemmDesc g = gemm_desc(groups, bf16, M, N, Kd, A, lda, sA, tA, B, ldb, sB, tB, C, ldc, sC, epi, aux, sAux, background,
                               alpha, splits, Kall);
  return launch_gemm(g, s) == hipSuccess ? HPSGD_OK : HPSGD_EHIP;
}

// Products (and column sums) waiting for a shared launch.  add() launches a product by itself, at once,
// when the shared launch does not take it: whatever it reads must be there when it is added, and nothing
// that is still waiting may depend on it.
struct GemmBatch {
  GemmPack pk;
  ColsumPack cs;
  hipStream_t s;
  int groups;
  GemmBatch(hipStream_t s_, int groups_, float lr) : s(s_), groups(groups_) {
    pk.n = cs.n = 0;
    cs.blk0[0] = 0;
    cs.lr = lr;
  }
  int add(const GemmDesc& d) {
    if (gemm_pack_push(pk, d)) return HPSGD_OK;
    return launch_gemm(d, s) == hipSuccess ? HPSGD_OK : HPSGD_EHIP;
  }
  // with_sums: the column sums too (else they wait on)
  int flush(bool with_sums = true) {
    ColsumPack none;
    none.n = 0;
    none.blk0[0] = 0;
    const hipError_t e = launch_gemm_pack(pk, with_sums ? cs : none, groups, s);
    pk.n = 0;
    if (with_sums) cs.n = 0;
    return e == hipSuccess ? HPSGD_OK : HPSGD_EHIP;
  }
};

// A view of a GEMM operand for the NT kernel (p == nullptr: none available): unit-stride along the contraction, or
// (outer) with the contraction's index running over its rows.
struct NtView {
  const void* p = nullptr;
  int bf16 = 0;
  long ld = 0, stride = 0;
  int outer = 0;
};

// bf16 precision: use the NT kernel when both operands have a usable contraction-contiguous
// view (C = a b^T), otherwise the generic kernel on the original fp32 operands.
int gemm2(hipStream_t s, int groups, int bf16, int M, int N, int Kd, const float* A, long lda, long sA,
          int tA, const float* B, long ldb, long sB, int tB, float* C, long ldc, long sC, int epi,
          const float* aux, long sAux, const NtView& a, const NtView& b, float alpha = 0.f,
          bool require_nt = false, int gp = 0, int gh = 0) {
  const int kd8 = a.outer ? 8 : Kd;  // (an outer A goes with an outer B: neither is read in chunks along the contraction)
  if (bf16 && a.p && b.p && (epi == EPI_STORE || epi == EPI_BIAS || epi == EPI_COMMIT) &&
      gemm_bf16_nt_supported(a.p, a.bf16, a.ld, a.stride, kd8) &&
      gemm_bf16_nt_supported(b.p, b.bf16, b.ld, b.stride, kd8) && ((uintptr_t)C & 3) == 0) {
    return launch_gemm_bf16_nt(a.p, a.bf16, a.ld, a.stride, b.p, b.bf16, b.ld, b.stride, C, ldc, sC,
                               epi == EPI_BIAS ? aux : nullptr, sAux, epi == EPI_COMMIT ? aux : nullptr, sAux,
                               alpha, M, N, Kd, groups, s, 0, gp, gh, 1, 0, a.outer | b.outer << 1) == hipSuccess
               ? HPSGD_OK
               : HPSGD_EHIP;
  }
  if (require_nt) return HPSGD_EINVAL;  // the fp32 operands of the fallback were not produced
  return gemm(s, groups, bf16, M, N, Kd, A, lda, sA, tA, B, ldb, sB, tB, C, ldc, sC, epi, aux, sAux, 0, alpha);
}

#define TRY(expr)                    \
  do {                               \
    TimerScope ts_(c, role, s);      \
    int rc_ = (expr);                \
    if (rc_ != HPSGD_OK) return rc_; \
  } while (0)
#define TRY0(expr)                   \
  do {                               \
    int rc_ = (expr);                \
    if (rc_ != HPSGD_OK) return rc_; \
  } while (0)

// The resident-weight recurrence kernels wait for each other inside a launch, which needs all
// their workgroups on the chip at once: two such launches running side by side (from two
// streams) could each hold CUs the other is waiting for.  Launches on one stream are ordered
// anyway.  Across streams, contexts and host threads they are ordered here: the one piece of
// per-process state of the library, per device, is the event recorded behind the most recent
// resident-weight launch and the stream it went to.  A local step that issues such launches
// holds the lock from its first one to its last (so that no other thread's launches fall in
// between) and, if the previous ones went to another stream, lets its stream wait for that
// event (hipStreamWaitEvent: the host never blocks).
// how far behind the training stream's product the auxiliary stream's starts where the former must
// be dispatched first (see the layers' backward pass)
constexpr unsigned kAuxHeadStartUs = 5;

struct ResidentOrder {
  std::mutex mu;
  hipEvent_t ev = nullptr;   // behind the last resident-weight launch issued on this device
  hipStream_t last = nullptr;
  bool have = false;
};
constexpr int kMaxDevices = 64;
ResidentOrder g_resident[kMaxDevices];

struct ResidentScope {
  ResidentOrder* o = nullptr;
  std::unique_lock<std::mutex> lock;
  hipStream_t s = nullptr;
  // Called before the step's first resident-weight launch.
  int begin(hipStream_t stream) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return HPSGD_EHIP;
    o = &g_resident[dev];
    s = stream;
    lock = std::unique_lock<std::mutex>(o->mu);
    if (!o->ev && hipEventCreateWithFlags(&o->ev, hipEventDisableTiming) != hipSuccess) {
      o->ev = nullptr;
      return HPSGD_EHIP;
    }
    if (o->have && o->last != s && hipStreamWaitEvent(s, o->ev, 0) != hipSuccess) return HPSGD_EHIP;
    return HPSGD_OK;
  }
  // note(): a resident-weight launch was issued; mark(): ... and the event is recorded behind
  // it (the last record stands).  The step marks behind its backward launches; a launch that was
  // only noted is marked when the step has been issued, where the lock is released too.
  bool pending = false;
  void note() { pending = o != nullptr; }
  int mark() {
    if (!o) return HPSGD_OK;
    pending = false;
    if (hipEventRecord(o->ev, s) != hipSuccess) return HPSGD_EHIP;
    o->have = true;
    o->last = s;
    return HPSGD_OK;
  }
  ~ResidentScope() {
    if (pending) (void)mark();
  }
};

// bf16 precision: the rounded copies of the weight matrices that a local step's GEMMs and
// recurrence launches read (row-major, W_hh transposed too for the backward recurrence), all
// made from the replicas `rin`.  what[l] / head say which copies exist; launch = false only
// reports.  The head's copies are made when with_head is set.
struct WeightCopies {
  bool wih[16] = {false}, whh[16] = {false}, whhT[16] = {false};
  bool head = false;
};

int weight_copies(hpsgd_ctx* c, const float* rin, long sR, int k0, int groups, float* ws, hipStream_t st, bool launch,
                  bool with_head, WeightCopies& wc) {
  const hpsgd_model_desc& d = c->d;
  if (d.prec != HPSGD_BF16_MFMA || d.kind == HPSGD_MLP || c->whhb.empty()) return HPSGD_OK;
  auto reg = [&](const Region& r) { return ws + r.offset + (size_t)k0 * r.stride; };
  auto bfreg = [&](const Region& r) { return (__bf16*)reg(r); };
  const bool lm = d.kind == HPSGD_GRU_LM;
  const bool pad = c->use_padded();
  const int B = pad ? c->Bp : d.batch, Hc = d.hidden, H = pad ? c->Hp : Hc, L = d.layers;
  const int classes = lm ? d.vocab : d.classes;
  const bool ntc = (B % 8 == 0) && (H % 8 == 0);
  const bool fused_b = gru_fused_bf16_supported(H);
  // the matrices go through one launch (each is a few hundred tiles); what the pack does not
  // take is launched by itself
  Cvt2Pack pack;
  // a matrix with rows in blocks of gh (gp in the copies) and Cs columns (C in the copies) of the padded layout
  auto copy_padded = [&](const float* in, void* out_p, long ld_p, long s_p, void* out_t, long ld_t, long s_t, int R, int C,
                         int gp, int gh, int Cs) -> bool {
    if (!launch) return true;
    if (pack.n == Cvt2Pack::MAX) {
      if (launch_cvt2_pack(pack, groups, st) != hipSuccess) return false;
      pack = Cvt2Pack();
    }
    // (a matrix that needs no padding takes the plain copies' 16-byte loads)
    if (gp == gh && Cs == C && cvt2_pack_push(pack, in, Cs, sR, out_p, ld_p, s_p, out_t, ld_t, s_t, R, C)) return true;
    return cvt2_pack_push_padded(pack, in, Cs, sR, out_p, ld_p, s_p, out_t, ld_t, s_t, R, C, gp, gh, Cs);
  };
  auto copy2 = [&](const float* in, long ld_in, void* out_p, long ld_p, long s_p, void* out_t, long ld_t, long s_t,
                   int R, int C) -> bool {
    if (!launch || cvt2_pack_push(pack, in, ld_in, sR, out_p, ld_p, s_p, out_t, ld_t, s_t, R, C)) return true;
    return launch_cvt2(in, 0, ld_in, sR, out_p, ld_p, s_p, out_t, ld_t, s_t, R, C, groups, st) == hipSuccess;
  };
  for (int l = 0; l < L && l < 16; ++l) {
    const int width = l > 0 ? Hc : (lm ? d.embed : d.input);
    const float* Wih = rin + c->eoff(c->lidx[l].wih);
    const float* Whh = rin + c->eoff(c->lidx[l].whh);
    if (pad) {
      const int wp = l > 0 ? H : c->Ep;
      const bool up = c->stack_b && l == 1;  // (its input gradient is computed beside the recurrences, from the transposed copy)
      if (!copy_padded(Wih, bfreg(c->wihbl[l]), c->wih_pitch(l), 2 * (long)c->wihbl[l].stride, up ? bfreg(c->wihT) : nullptr, up ? 3 * H : 0,
                       up ? 2 * (long)c->wihT.stride : 0, 3 * H, wp, H, Hc, width) ||
          !copy_padded(Whh, bfreg(c->whhb[l]), H, 2 * (long)c->whhb[l].stride, bfreg(c->whhT[l]), 3 * H,
                       2 * (long)c->whhT[l].stride, 3 * H, H, H, Hc, Hc))
        return HPSGD_EHIP;
      wc.wih[l] = wc.whh[l] = wc.whhT[l] = true;
      continue;
    }
    if (fused_b && ntc && width % 8 == 0) {
      const long s_wb2 = 2 * (long)c->wihbl[l].stride;
      if (cvt2_supported(Wih, 0, width, sR, bfreg(c->wihbl[l]), c->wih_pitch(l), s_wb2, nullptr, 0, 0, 3 * H, width)) {
        if (!copy2(Wih, width, bfreg(c->wihbl[l]), c->wih_pitch(l), s_wb2, nullptr, 0, 0, 3 * H, width)) return HPSGD_EHIP;
        wc.wih[l] = true;
      }
    }
    if (fused_b) {
      void* wb = reg(c->whhb[l]);
      const long s_wb = 2 * (long)c->whhb[l].stride, s_whT = 2 * (long)c->whhT[l].stride;
      if (cvt2_supported(Whh, 0, H, sR, wb, H, s_wb, bfreg(c->whhT[l]), 3 * H, s_whT, 3 * H, H)) {
        if (!copy2(Whh, H, wb, H, s_wb, bfreg(c->whhT[l]), 3 * H, s_whT, 3 * H, H)) return HPSGD_EHIP;
        wc.whhT[l] = true;
      } else if (launch && launch_cvt_bf16(Whh, H, sR, wb, H, s_wb, 3 * H, H, false, groups, st) != hipSuccess) {
        return HPSGD_EHIP;
      }
      wc.whh[l] = true;
    }
  }
  if (with_head) {
    const size_t oW = c->eoff(c->i_head_w);
    const long s_wob = 2 * (long)c->wob.stride;
    if (pad) {
      if (!copy_padded(rin + oW, bfreg(c->wob), c->head_pitch(), s_wob, nullptr, 0, 0, c->Vp, H, c->Vp, classes, Hc)) return HPSGD_EHIP;
      wc.head = true;
    } else if (ntc && fused_b && classes % 8 == 0 &&
               cvt2_supported(rin + oW, 0, H, sR, bfreg(c->wob), c->head_pitch(), s_wob, nullptr, 0, 0, classes, H)) {
      if (!copy2(rin + oW, H, bfreg(c->wob), c->head_pitch(), s_wob, nullptr, 0, 0, classes, H)) return HPSGD_EHIP;
      wc.head = true;
    }
  }
  if (launch && launch_cvt2_pack(pack, groups, st) != hipSuccess) return HPSGD_EHIP;
  return HPSGD_OK;
}

// One local step for `groups` workers whose workspace slices start at worker k0.
// acc (nullable): per-worker gradient accumulators [groups][acc_stride]; the step's gradient
// is added to them (Alg. 2 "accumulate gradients").  Every gradient then goes through the
// gradient buffer: no weight matrix is updated in a GEMM epilogue.
// cloned: rin is ONE model that every worker's replica is a clone of (Alg. 2 "make replica" not
// yet written out): parameters are read from it with group stride 0, rout receives every
// parameter of every worker.
int run_step(hpsgd_ctx* c, int k0, int groups, const float* rin, float* rout, size_t rstride,
             const void* x, const int32_t* y, float lr, float* loss_out, float* ws, hipStream_t s,
             float* acc = nullptr, size_t acc_stride = 0, bool cloned = false) {
  const hpsgd_model_desc& d = c->d;
  const int bf = d.prec == HPSGD_BF16_MFMA ? 1 : 0;
  auto reg = [&](const Region& r) { return ws + r.offset + (size_t)k0 * r.stride; };
  float* grad = reg(c->grad);
  const long sG = (long)c->grad.stride;
  const long sR = (long)rstride;            // of rout
  const long sRi = cloned ? 0L : (long)rstride;  // of rin
  const int B = d.batch;
  int role = HPSGD_ROLE_OTHER;
  c->timer_nested = false;
  StepCtxScope step_scope(c);
  ResidentScope resident;  // orders this step's resident-weight launches against other streams
  // the bf16 copies of the weights are already in this workspace (hpsgd_prepare_replicas); the
  // step changes the weights, so the mark is used once
  hpsgd_ctx::Mark mark{nullptr, nullptr, 0, nullptr, false};
  // (a mark is kept under the replicas' address: rout when they are still clones of rin)
  const bool marked = c->take_mark(cloned ? rout : rin, ws, rstride, mark);
  const bool prepared = bf && marked && k0 == 0 && groups == c->K && (!cloned || mark.clone_src == rin);
  // clones without prepared copies: the step makes the one set itself, from rin
  const bool own_set = cloned && !prepared && bf && k0 == 0;
  const float* head_src = prepared ? mark.clone_src : own_set ? rin : nullptr;
  const bool head_done = prepared && mark.head_done;
  // the replicas are clones of one model (hpsgd_prepare_clones): one set of bf16 weight copies, in
  // worker 0's slice of the workspace, is every worker's operand (group stride 0)
  const bool shared = head_src != nullptr;
  auto wstride = [&](const Region& r) { return shared ? 0L : 2 * (long)r.stride; };
  const unsigned* abort_word = nullptr;  // set when launches were made whose workgroups wait for each other
  c->last_resident = c->last_xproj = c->last_dw = 0;
  // Weight matrices whose SGD update is applied by the epilogue of their own gradient GEMM
  // (replica_out = replica_in - lr * dW, no gradient buffer round trip); every other
  // parameter goes through the gradient buffer and the commit kernel at the end.  A matrix
  // is only updated after the last kernel that reads it (the input-gradient GEMM of its
  // layer) has been issued, so the step may run in place.
  std::vector<char> fused_commit(c->entries.size(), 0);
  // Where the weight-gradient GEMM of `name` writes: the updated matrix itself (epilogue
  // W_out = W_in - lr * dW), or, when gradients are accumulated as well, the gradient buffer.
  struct WgradTarget { float* C; long sC; int epi; const float* aux; };
  auto wgrad_target = [&](int entry) -> WgradTarget {
    const size_t o = c->eoff(entry);
    if (acc) return WgradTarget{grad + o, sG, EPI_STORE, nullptr};
    fused_commit[entry] = 1;
    return WgradTarget{rout + o, sR, EPI_COMMIT, rin + o};
  };

  if (d.kind == HPSGD_MLP) {
    const int L = d.n_mlp_dims - 1;
    const int* dims = d.mlp_dims;
    // A last layer with few classes (the softmax head): forward, loss, its three gradients and its
    // update as the two small launches of the classifier head instead of three GEMMs, the loss
    // kernel and a share of the column sums
    const bool small_head = !bf && L >= 2 && cls_head_supported(B, dims[L], dims[L - 1]) && c->dact.size() + 1 >= (size_t)L;
    // forward
    const float* a_in = (const float*)x;
    long s_in = (long)B * dims[0];
    for (int i = 0; i < (small_head ? L - 1 : L); ++i) {
      float* a_out = reg(c->act[i]);
      role = HPSGD_ROLE_MLP_FWD;
      TRY(gemm(s, groups, bf, B, dims[i + 1], dims[i], a_in, dims[i], s_in, 0, rin + c->eoff(c->fc_w[i]),
               dims[i], sRi, 1, a_out, dims[i + 1], (long)c->act[i].stride,
               i + 1 < L ? EPI_BIAS_RELU : EPI_BIAS, rin + c->eoff(c->fc_b[i]), sRi));
      a_in = a_out;
      s_in = (long)c->act[i].stride;
    }
    // loss; the logits buffer becomes the output delta
    float* delta = reg(c->act[L - 1]);
    float* rowloss = reg(c->rowloss);
    role = HPSGD_ROLE_LOSS;
    if (small_head) {
      const size_t oW = c->eoff(c->fc_w[L - 1]), ob = c->eoff(c->fc_b[L - 1]);
      float* dprev = reg(c->dact[L - 2]);
      if (acc) {
        HIP_TRY(launch_cls_head(a_in, s_in, rin + oW, rin + ob, sRi, y, B, delta, (long)c->act[L - 1].stride, rowloss,
                                (long)c->rowloss.stride, dprev, (long)c->dact[L - 2].stride, grad + oW, grad + ob, sG, lr,
                                0, loss_out, B, dims[L], dims[L - 1], groups, s, 1));
      } else {
        fused_commit[c->fc_w[L - 1]] = 1;
        fused_commit[c->fc_b[L - 1]] = 1;
        HIP_TRY(launch_cls_head(a_in, s_in, rin + oW, rin + ob, sRi, y, B, delta, (long)c->act[L - 1].stride, rowloss,
                                (long)c->rowloss.stride, dprev, (long)c->dact[L - 2].stride, rout + oW, rout + ob, sR, lr,
                                1, loss_out, B, dims[L], dims[L - 1], groups, s, 1));
      }
      delta = dprev;
    } else {
      HIP_TRY(launch_softmax_ce(delta, (long)c->act[L - 1].stride, y, B, delta, rowloss,
                                (long)c->rowloss.stride, B, dims[L], groups, s));
    }
    // backward.  The input gradients form a chain from launch to launch; a weight gradient rides in the
    // launch after its layer's input gradient (which reads the weights that it updates), the last ones
    // together with the bias gradients (column sums of every layer's delta) and the mean loss, which the
    // same launch applies unless the gradients are accumulated as well.
    GemmBatch gb(s, groups, lr);
    // (the mean of the per-row losses: a column sum of a B x 1 matrix; the small head has taken it already)
    if (loss_out && !small_head &&
        !colsum_pack_push(gb.cs, rowloss, 1, (long)c->rowloss.stride, loss_out, 1, nullptr, 0, B, 1, 1.0f / (float)B))
      return HPSGD_ESHAPE;
    for (int i = (small_head ? L - 2 : L - 1); i >= 0; --i) {
      const float* a_prev = i > 0 ? reg(c->act[i - 1]) : (const float*)x;
      const long s_prev = i > 0 ? (long)c->act[i - 1].stride : (long)B * dims[0];
      const long s_delta = i == L - 1 ? (long)c->act[i].stride : (long)c->dact[i].stride;
      role = HPSGD_ROLE_MLP_BWD;  // (with the small head the loop starts at layer L-2, whose delta is dact[L-2])
      float* dprev = nullptr;
      if (i > 0) {
        // delta_prev = (delta W) * [a_prev > 0]: before W is updated
        dprev = reg(c->dact[i - 1]);
        TRY(gb.add(gemm_desc(groups, bf, B, dims[i], dims[i + 1], delta, dims[i + 1], s_delta, 0,
                             rin + c->eoff(c->fc_w[i]), dims[i], sRi, 0, dprev, dims[i], (long)c->dact[i - 1].stride,
                             EPI_RELU_MASK, a_prev, s_prev)));
        TRY(gb.flush(false));
      }
      // W' = W - lr * delta^T a_prev
      const WgradTarget wt = wgrad_target(c->fc_w[i]);
      TRY(gb.add(gemm_desc(groups, bf, dims[i + 1], dims[i], B, delta, dims[i + 1], s_delta, 1, a_prev, dims[i],
                           s_prev, 0, wt.C, dims[i], wt.sC, wt.epi, wt.aux, sRi, 0, lr)));
      {
        const size_t ob = c->eoff(c->fc_b[i]);
        const bool pushed =
            acc ? colsum_pack_push(gb.cs, delta, dims[i + 1], s_delta, grad + ob, sG, nullptr, 0, B, dims[i + 1])
                : colsum_pack_push(gb.cs, delta, dims[i + 1], s_delta, rout + ob, sR, rin + ob, sRi, B, dims[i + 1]);
        if (pushed && !acc) fused_commit[c->fc_b[i]] = 1;
        if (!pushed)
          HIP_TRY(launch_colsum(delta, dims[i + 1], s_delta, grad + ob, sG, B, dims[i + 1], groups, s));
      }
      if (i > 0) delta = dprev;
    }
    TRY(gb.flush());
  } else {
    const bool lm = d.kind == HPSGD_GRU_LM;
    // pad: internal sizes (see hpsgd_ctx::padded); Bc, Hc, Ec: the model's own
    const bool pad = c->use_padded();
    const int Bc = d.batch, Hc = d.hidden, Ec = lm ? d.embed : d.input;
    const int B = pad ? c->Bp : Bc, H = pad ? c->Hp : Hc, width0 = pad ? c->Ep : Ec;
    const int T = d.seq_len, L = d.layers;
    const int TB = T * B, TBc = T * Bc;
    const int classes = lm ? d.vocab : d.classes;
    const int ldl = pad ? c->Vp : classes;  // row pitch of the logits
    const int32_t* tok = (const int32_t*)x;
    float* gx = reg(c->gx);
    float* dgh_lo = reg(c->dgh);
    float* gh = reg(c->gh);
    float* D = reg(c->D);
    float* dx = reg(c->dx);
    float* logits = reg(c->logits);
    float* rowloss = reg(c->rowloss);
    const long s_gx = (long)c->gx.stride, s_gh = (long)c->gh.stride, s_D = (long)c->D.stride;
    const long s_dx = (long)c->dx.stride, s_log = (long)c->logits.stride;

    // bf16 precision: the weight-gradient and input-gradient GEMMs take contraction-contiguous
    // bf16 operands ("NT" form); the fused step kernels write those copies themselves
    const bool ntc = bf && (B % 8 == 0) && (H % 8 == 0);
    const long TBp = (long)round_up(TB, 64), TB1p = (long)round_up(TB + B, 64);
    auto bfreg = [&](const Region& r) { return (__bf16*)reg(r); };
    bool xT_ready = false;  // the transposed bf16 layer-0 input was made in the forward pass
    // per layer: the transposed bf16 W_hh was made in the forward pass, in the same
    // read as the row-major copy
    bool whhT_ready[16] = {false};
    // fp32: the recurrence of a layer as one launch (or a few, gru_persist_pays) with W_hh resident on the chip.
    // Its workgroups wait for each other through flag words in the workspace, zeroed here; pbase
    // follows what the flags read.  A given-up wait shows as NaN in the results (below).
    // narrow fp32 layers: the whole recurrence without any exchange between workgroups
    const bool use_solo = c->solo && c->resident;
    const bool use_stack = use_solo && c->stack;  // both layers in one launch
    const bool use_persist = c->prow != 0 && c->resident && gru_persist_pays(B, H, T, groups, c->prow);
    const int prow = use_persist ? c->prow : c->prow_b;  // rows of a synchronisation group
    // bf16: the same with the weight slices in registers; its backward launch writes only the bf16
    // copies of the gate gradients, so every GEMM that consumes them must be able to take those
    // (contraction-contiguous bf16 views: batch, hidden size and every layer width multiples of 8)
    // (the padded layout of a language model has them by construction)
    const bool use_persist_b = bf && c->resident && gru_persist_bf16_supported(B, H) && ntc && width0 % 8 == 0;
    const bool use_solo_b = pad && c->solo_b;  // (a kind of use_persist_b without the exchange)
    const bool use_stack_b = use_solo_b && c->stack_b;
    const bool exact_gates = gru_bf16_exact_gates(B, H, c->K, B != Bc || H != Hc || width0 != Ec);
    const bool exchange = use_persist || (use_persist_b && !use_solo_b);
    unsigned* psync = exchange || use_stack || use_stack_b ? (unsigned*)reg(c->psync) : nullptr;
    // the abort words of all workers of this step, cleared whether it exchanges or not: what is reported is this
    // step, not an earlier one of another form or what the memory held
    unsigned* aborts = c->psync.stride ? (unsigned*)reg(c->psync) : nullptr;
    unsigned pbase = 0;
    unsigned ticket_launches = 0;  // launches of this step that placed their workgroups by ticket
    const size_t psync_words = use_stack ? gru_stack_sync_words(B, groups) : use_stack_b ? gru_stack_bf16_sync_words(B, groups) : exchange ? gru_persist_sync_words(B, groups, prow) : 0;
    if (exchange) TRY0(resident.begin(s));
    abort_word = psync;  // (cleared together with the first layer's h_0 below)
    // ---- the head's operands
    const int nrows = lm ? TB : B;
    const size_t oW = c->eoff(c->i_head_w), ob = c->eoff(c->i_head_b);
    const long nrp = (long)round_up(nrows, 64), clp = (long)round_up(classes, 64);
    const long s_dlb = 2 * (long)c->dlogb.stride, s_wob = wstride(c->wob);
    // bf16 precision with every head operand available as bf16: h of the top layer (written
    // by its step kernels), head.W rounded once, the logit gradient emitted in bf16 by the loss kernel
    const bool headb =
        pad || (ntc && gru_fused_bf16_supported(H) && classes % 8 == 0 &&
                cvt2_supported(rin + oW, 0, H, sRi, bfreg(c->wob), c->head_pitch(), s_wob, nullptr, 0, 0, classes, H) &&
                softmax_ce_bf16_supported(logits, ldl, s_log, bfreg(c->dlogb), clp, s_dlb, classes));
    // bf16 copies of `n` workers' head matrices (one model's when the replicas are still its clones)
    auto head_copy = [&](const float* W, long s_W, int n, hipStream_t st) -> hipError_t {
      if (!pad || (Hc == H && cvt2_supported(W, 0, H, s_W, bfreg(c->wob), c->head_pitch(), s_wob, nullptr, 0, 0, classes, H)))
        return launch_cvt2(W, 0, H, s_W, bfreg(c->wob), c->head_pitch(), s_wob, nullptr, 0, 0, classes, H, n, st);
      Cvt2Pack pk;
      if (!cvt2_pack_push_padded(pk, W, Hc, s_W, bfreg(c->wob), c->head_pitch(), s_wob, nullptr, 0, 0, c->Vp, H, c->Vp, classes, Hc))
        return hipErrorInvalidValue;
      return launch_cvt2_pack(pk, n, st);
    };
    // the layers' bf16 weight copies: all at the start (nothing but the replicas feeds them),
    // unless they were made before the step
    WeightCopies wc;
    role = HPSGD_ROLE_OTHER;
    // (clones with a small head: that copy too.  By itself it goes to the second stream, with an event in each direction,
    // which costs more than its bytes.  1.4 M elements: 10 us either way, in the pack without the events; 92 M: 31 us, in
    // the shade of the top layer's input projection.)
    const bool head_with = headb && own_set && (double)classes * Hc <= 4e6;
    TRY(weight_copies(c, rin, sRi, k0, own_set ? 1 : groups, ws, s, !prepared, head_with, wc));
    const bool head_made = head_done || (head_with && wc.head);
    // a layer's arrays in the launches of two layers (the regions of both have the same strides)
    auto stack_layer = [&](int l) {
      return GruStackLayer{rin + c->eoff(c->lidx[l].whh), rin + c->eoff(c->lidx[l].bhh), l ? reg(c->gx_up) : gx, l ? reg(c->dgh_up) : dgh_lo,
                           reg(c->hs[l]), reg(c->sv[l]), l ? reg(c->dbp_up) : reg(c->dbp)};
    };
    auto stack_layer_b = [&](int l) {
      return GruStackLayerB{bfreg(c->whhb[l]), bfreg(c->whhT[l]), rin + c->eoff(c->lidx[l].bih), rin + c->eoff(c->lidx[l].bhh),
                            l ? reg(c->gx_up) : gx, l ? bfreg(c->hb) : bfreg(c->hb_lo), reg(c->hs[l]), reg(c->sv[l]), bfreg(c->hsT[l]),
                            l ? bfreg(c->dg4_up) : bfreg(c->dghx), l ? reg(c->dbp_up) : reg(c->dbp)};
    };
    // ---- forward
    const float* lin = (const float*)x;
    long s_lin = (long)TB * d.input;
    int width = d.input;
    if (pad) {
      // lookup, rounding and transpose of the embedding rows in one launch; nothing reads them in fp32
      role = HPSGD_ROLE_EMBED;
      HIP_TRY(launch_embed_bf16(rin + c->eoff(c->i_embed), sRi, tok, TBc, bfreg(c->xb), 2 * (long)c->xb.stride, bfreg(c->xT), TBp,
                                2 * (long)c->xT.stride, T, Bc, B, Ec, width0, groups, s));
      xT_ready = true;
      width = width0;
    } else if (lm) {
      float* xe = reg(c->xe);
      role = HPSGD_ROLE_EMBED;
      HIP_TRY(launch_embed_fwd(rin + c->eoff(c->i_embed), sRi, tok, TB, xe, (long)c->xe.stride, TB,
                               d.embed, groups, s));
      lin = xe;
      s_lin = (long)c->xe.stride;
      width = d.embed;
    }
    // everything a step clears before its first layer, in one launch: the flag words of the
    // resident-weight launches, h_0 of every layer (fp32, and in bf16 precision the bf16 copy and
    // the first B columns of the transposed copy)
    bool cleared = false;
    bool head_early = false;
    {
      FillPack fp;
      fp.n = 0;
      fp.blk0[0] = 0;
      fp.max_groups = 0;
      bool ok = true;
      if (psync) ok = ok && fill_pack_push(fp, (float*)psync, 0, 1, (long)psync_words, 0, 1);
      if (aborts) ok = ok && fill_pack_push(fp, (float*)aborts, 0, 1, 1, c->psync.stride, groups);
      const bool solo_any = use_solo || use_solo_b;  // (those launches write h_0 themselves)
      for (int l = 0; l < L && ok && !solo_any; ++l) {
        ok = ok && fill_pack_push(fp, reg(c->hs[l]), 0, 1, (long)B * H, c->hs[l].stride, groups);
        if (bf && gru_fused_bf16_supported(H) && ntc)
          ok = ok && fill_pack_push(fp, reg(c->hsT[l]), TB1p / 2, H, B / 2, c->hsT[l].stride, groups);
      }
      if (bf && gru_fused_bf16_supported(H) && !solo_any)
        ok = ok && fill_pack_push(fp, reg(c->hb), 0, 1, (long)B * H / 2, c->hb.stride, groups);
      if (use_persist_b && !use_solo_b)
        ok = ok && fill_pack_push(fp, reg(c->hx), 0, 1, (long)(gru_persist_bf16_exchange_elems(B, H) / 2), c->hx.stride, groups);
      if (use_persist)
        ok = ok && fill_pack_push(fp, reg(c->hx), 0, 1, (long)gru_persist_exchange_words(B, H, 1), c->hx.stride, groups);
      if (ok) {
        role = HPSGD_ROLE_OTHER;
        HIP_TRY(launch_fill_pack(fp, s));
        cleared = true;
      }
    }
    for (int l = 0; l < L; ++l) {
      float* hs = reg(c->hs[l]);
      float* sv = reg(c->sv[l]);
      const long s_hs = (long)c->hs[l].stride, s_sv = (long)c->sv[l].stride;
      role = HPSGD_ROLE_OTHER;
      if (!cleared) {
        HIP_TRY(launch_fill_zero(hs, (size_t)B * H, (size_t)s_hs, groups, s, l == 0 ? (float*)psync : nullptr,
                                 l == 0 && psync ? psync_words : 0));
        if (aborts && l == 0) HIP_TRY(launch_fill_zero((float*)aborts, 1, c->psync.stride, groups, s));
        if (use_persist && l == 0)
          HIP_TRY(launch_fill_zero(reg(c->hx), gru_persist_exchange_words(B, H, 1), c->hx.stride, groups, s));
      }
      const float* Whh = rin + c->eoff(c->lidx[l].whh);
      const bool fused = !bf && gru_fused_supported(H) && ((uintptr_t)Whh & 15) == 0 && (sRi & 3) == 0;
      const bool fused_b = bf && gru_fused_bf16_supported(H);
      const bool persist = use_persist;
      // a narrow layer input: the resident-weight kernel does the input projection itself
      const float* Wih0 = rin + c->eoff(c->lidx[l].wih);
      const bool xproj = persist && gru_persist_xproj_supported(H, width, prow) && ((uintptr_t)lin & 15) == 0 &&
                         (s_lin & 3) == 0;
      if (!xproj && !((use_stack || use_stack_b) && l > 0)) {
        const float* Wih = rin + c->eoff(c->lidx[l].wih);
        NtView va{lin, 0, width, s_lin}, vb{Wih, 0, width, sRi};
        // bf16 precision: both operands as row-major bf16 copies (the layer below wrote its
        // h in bf16; the layer-0 input and W_ih are rounded here, the input also transposed
        // for the weight-gradient GEMM)
        if (fused_b && ntc && width % 8 == 0) {
          role = HPSGD_ROLE_OTHER;
          const long s_xb = 2 * (long)c->xb.stride;
          if (pad && l == 0) {
            va = NtView{bfreg(c->xb), 1, width, s_xb};
          } else if (l > 0) {
            va = NtView{(const __bf16*)reg(c->hb) + (size_t)B * H, 1, H, 2 * (long)c->hb.stride};
          } else if (cvt2_supported(lin, 0, width, s_lin, bfreg(c->xb), width, s_xb, bfreg(c->xT), TBp,
                                    2 * (long)c->xT.stride, TB, width)) {
            HIP_TRY(launch_cvt2(lin, 0, width, s_lin, bfreg(c->xb), width, s_xb, bfreg(c->xT), TBp,
                                2 * (long)c->xT.stride, TB, width, groups, s));
            va = NtView{bfreg(c->xb), 1, width, s_xb};
            xT_ready = true;
          }
          if (wc.wih[l]) vb = NtView{bfreg(c->wihbl[l]), 1, c->wih_pitch(l), wstride(c->wihbl[l])};  // made at the start of the step, or before it
        }
        // The one copy of the head matrix that serves cloned replicas: beside the top layer's
        // input projection (between two resident-weight launches, when the synchronising stream
        // has finished), joined before the recurrence starts.
        const bool early = l == L - 1 && l > 0 && headb && !head_made && head_src && c->aux && c->ev_fork && c->ev_join;
        if (early) {
          if (hipEventRecord(c->ev_fork, s) != hipSuccess || hipStreamWaitEvent(c->aux, c->ev_fork, 0) != hipSuccess ||
              head_copy(head_src + oW, 0, 1, c->aux) != hipSuccess ||
              hipEventRecord(c->ev_join, c->aux) != hipSuccess)
            return HPSGD_EHIP;
          head_early = true;
        }
        role = HPSGD_ROLE_GEMM_INPUT;
        // (the bf16 resident-weight launches add b_ih themselves)
        TRY(gemm2(s, groups, bf, TB, 3 * H, width, lin, width, s_lin, 0, Wih, width, sRi, 1, gx, 3 * H, s_gx,
                  use_persist_b ? EPI_STORE : EPI_BIAS, use_persist_b ? nullptr : rin + c->eoff(c->lidx[l].bih), sRi, va, vb,
                  0.f, pad));
        if (early && hipStreamWaitEvent(s, c->ev_join, 0) != hipSuccess) return HPSGD_EHIP;
      }
      // bf16 path: bf16 copy of W_hh (kept in the W_hh^T region, which the forward pass does
      // not use) and of h
      void* wb = wc.whh[l] ? reg(c->whhb[l]) : reg(c->wt);
      const long s_wb = wc.whh[l] ? wstride(c->whhb[l]) : 2 * (long)c->wt.stride;
      __bf16* hb = fused_b ? (__bf16*)reg(c->hb) : nullptr;
      const long s_hb = 2 * (long)c->hb.stride;
      __bf16* hT = (fused_b && ntc) ? bfreg(c->hsT[l]) : nullptr;  // hsT exists in bf16 precision only
      const long s_hT = hT ? 2 * (long)c->hsT[l].stride : 0;
      if (fused_b) {
        role = HPSGD_ROLE_OTHER;
        if (!wc.whh[l]) return HPSGD_ESHAPE;  // (bf16 precision allocates the per-layer copies)
        whhT_ready[l] = wc.whhT[l];
        if (!cleared) {
          HIP_TRY(launch_fill_zero((float*)hb, (size_t)B * H / 2, (size_t)c->hb.stride, groups, s));
          if (use_persist_b)
            HIP_TRY(launch_fill_zero(reg(c->hx), gru_persist_bf16_exchange_elems(B, H) / 2, c->hx.stride, groups, s));
          if (hT)  // h_0 = 0: the first B columns of the transposed copy
            HIP_TRY(launch_fill_zero_2d((float*)hT, TB1p / 2, H, B / 2, c->hsT[l].stride, groups, s));
        }
      }
      // one event pair around the whole time loop when its launches are all of one role (two layers' one launch is issued for the upper one)
      const bool persist_b = fused_b && use_persist_b && hT != nullptr;
      const bool with_upper = (use_stack || use_stack_b) && l == 0;
      TimerScope loop_fwd(c, HPSGD_ROLE_GEMM_REC_FWD, s, with_upper ? 0 : (persist || persist_b || use_solo) ? 1 : (fused || fused_b) ? T : 0);
      c->timer_nested = loop_fwd.active() && (fused || fused_b || use_solo || persist);
      if (use_stack) {
        role = HPSGD_ROLE_GEMM_REC_FWD;
        if (l > 0)
          HIP_TRY(launch_gru_stack_fwd(stack_layer(0), stack_layer(1), Wih0, rin + c->eoff(c->lidx[1].bih), sRi, s_gx, s_hs, s_sv, B, H, T,
                                       groups, psync, c->link_limit(), s));
        ++c->last_resident;
      } else if (use_solo) {
        role = HPSGD_ROLE_GEMM_REC_FWD;
        HIP_TRY(launch_gru_solo_fwd(Whh, rin + c->eoff(c->lidx[l].bhh), sRi, gx, s_gx, hs, s_hs, sv, s_sv, B, H, T, groups, c->K, s));
        ++c->last_resident;
      }
      if (persist) {
        role = HPSGD_ROLE_GEMM_REC_FWD;
        HIP_TRY(launch_gru_fwd_persist(Whh, rin + c->eoff(c->lidx[l].bhh), sRi, gx, s_gx, hs, s_hs, reg(c->hx),
                                       (long)c->hx.stride, sv, s_sv, B, H, T,
                                       groups, prow, psync, pbase, c->spin_limit, xproj ? lin : nullptr, s_lin, width,
                                       Wih0, rin + c->eoff(c->lidx[l].bih), c->device_scope, &ticket_launches, s));
        pbase += (unsigned)T * gru_persist_count_per_step(H);
        ++c->last_resident;
        c->last_xproj += xproj ? 1 : 0;
        resident.note();
      }
      if (persist_b && use_stack_b) {
        role = HPSGD_ROLE_GEMM_REC_FWD;
        if (l > 0)
          HIP_TRY(launch_gru_stack_fwd_bf16(stack_layer_b(0), stack_layer_b(1), bfreg(c->wihbl[1]), wstride(c->wihbl[1]), s_wb, sRi, Hc, s_gx,
                                            s_hb, s_hs, s_sv, TB1p, s_hT, Bc, B, H, T, groups, exact_gates, psync, c->link_limit(), s));
        ++c->last_resident;
      } else if (persist_b && use_solo_b) {
        role = HPSGD_ROLE_GEMM_REC_FWD;
        HIP_TRY(launch_gru_solo_fwd_bf16(wb, s_wb, rin + c->eoff(c->lidx[l].bih), rin + c->eoff(c->lidx[l].bhh), sRi, Hc, gx, s_gx,
                                         hb, s_hb, hs, s_hs, sv, s_sv, hT, TB1p, s_hT, Bc, B, H, T, groups, c->K, exact_gates, s));
        ++c->last_resident;
      } else if (persist_b) {
        role = HPSGD_ROLE_GEMM_REC_FWD;
        HIP_TRY(launch_gru_fwd_persist_bf16(wb, s_wb, rin + c->eoff(c->lidx[l].bih), rin + c->eoff(c->lidx[l].bhh), sRi, Hc, gx, s_gx, hs, s_hs, hb, s_hb,
                                            bfreg(c->hx), 2 * (long)c->hx.stride, sv, s_sv, hT, TB1p, s_hT, Bc, B, H, T, groups, prow, exact_gates,
                                            psync, pbase, c->spin_limit, c->device_scope, &ticket_launches, s));
        pbase += (unsigned)T * gru_persist_bf16_count_per_step(H);
        ++c->last_resident;
        resident.note();
      }
      for (int t = 0; t < T && !persist && !persist_b && !use_solo; ++t) {
        role = HPSGD_ROLE_GEMM_REC_FWD;
        if (fused_b) {
          HIP_TRY(launch_gru_fwd_step_bf16(wb, s_wb, rin + c->eoff(c->lidx[l].bhh), sRi, gx + (size_t)t * B * 3 * H,
                                           s_gx, hs + (size_t)t * B * H, hs + (size_t)(t + 1) * B * H, s_hs,
                                           hb + (size_t)t * B * H, hb + (size_t)(t + 1) * B * H, s_hb,
                                           sv + (size_t)t * B * 4 * H, s_sv,
                                           hT ? hT + (size_t)(t + 1) * B : nullptr, TB1p, s_hT, B, H, groups,
                                           s));
          continue;
        }
        if (fused) {
          HIP_TRY(launch_gru_fwd_step(Whh, rin + c->eoff(c->lidx[l].bhh), sRi, gx + (size_t)t * B * 3 * H, s_gx,
                                      hs + (size_t)t * B * H, hs + (size_t)(t + 1) * B * H, s_hs,
                                      sv + (size_t)t * B * 4 * H, s_sv, B, H, groups, s));
          continue;
        }
        TRY(gemm(s, groups, bf, B, 3 * H, H, hs + (size_t)t * B * H, H, s_hs, 0, Whh, H, sRi, 1, gh, 3 * H,
                 s_gh, EPI_BIAS, rin + c->eoff(c->lidx[l].bhh), sRi));
        role = HPSGD_ROLE_CELL_FWD;
        HIP_TRY(launch_gru_cell_fwd(gx + (size_t)t * B * 3 * H, s_gx, gh, s_gh, hs + (size_t)t * B * H,
                                    hs + (size_t)(t + 1) * B * H, s_hs, sv + (size_t)t * B * 4 * H,
                                    s_sv, B, H, groups, s));
      }
      c->timer_nested = false;
      lin = hs + (size_t)B * H;
      s_lin = s_hs;
      width = H;
    }
    // ---- head and loss
    GemmBatch gb(s, groups, lr);  // fp32 products and column sums waiting for a shared launch
    const float* top = reg(c->hs[L - 1]);
    const long s_top = (long)c->hs[L - 1].stride;
    const float* feats = lm ? top + (size_t)B * H : top + (size_t)T * B * H;
    if (headb) {
      role = HPSGD_ROLE_OTHER;
      // the bf16 copies of the head's weights: here, when the synchronising stream has finished and
      // the copy has the memory system to itself (beside a resident-weight launch it takes 2.3
      // times as long and slows that launch by more than it takes alone; at the start of the step it
      // shares the bandwidth with the merge and the clone)
      if (head_made || head_early) {
        // made with the layers' copies, before the step, or beside the top layer's input projection
      } else if (head_src) {  // the replicas are clones of one model: one copy of its head matrix serves all workers
        HIP_TRY(head_copy(head_src + oW, 0, 1, s));
      } else if (!prepared) {
        HIP_TRY(head_copy(rin + oW, sRi, groups, s));
      }
      const long s_hb = 2 * (long)c->hb.stride;
      const NtView va{(const __bf16*)reg(c->hb) + (size_t)(lm ? B : T * B) * H, 1, H, s_hb};
      const NtView vb{bfreg(c->wob), 1, c->head_pitch(), s_wob};
      role = HPSGD_ROLE_GEMM_HEAD;
      TRY(gemm2(s, groups, bf, nrows, classes, H, feats, H, s_top, 0, rin + oW, H, sRi, 1, logits, ldl,
                s_log, EPI_BIAS, rin + ob, sRi, va, vb, 0.f, pad));
      role = HPSGD_ROLE_LOSS;
      // the head's bias gradient: column sums of the unrounded logit gradient, per block of rows
      // in the loss kernel, added up below
      // (the partial sums of the groups lie back to back, as the adding kernel reads them)
      // (sized for all K workers also when fewer are stepped: these sums then do not depend on the entry point)
      const int n_colparts = softmax_ce_bf16_row_blocks(nrows, c->K, classes);
      const long colpitch = (long)round_up(classes, 8), s_colpart = (long)n_colparts * colpitch;
      HIP_TRY(launch_softmax_ce_bf16(logits, ldl, s_log, y, lm ? TBc : Bc, bfreg(c->dlogb), clp, s_dlb, rowloss,
                                     (long)c->rowloss.stride, nrows, Bc, B, classes, groups, s, reg(c->colpart), s_colpart, c->K));
      role = HPSGD_ROLE_GEMM_HEAD;
      const int Kv = (int)round_up(classes, 8);  // (zeros from `classes` on, in both operands)
      // (the contractions over the classes, of the input gradient, and over the rows, of the weight gradient, run over
      // the rows of W, of the logit gradients and of h as they lie in memory)
      const NtView vdl{bfreg(c->dlogb), 1, clp, s_dlb}, vw{bfreg(c->wob), 1, c->head_pitch(), s_wob, 1};
      const NtView vdo{vdl.p, 1, clp, s_dlb, 1}, vho{va.p, 1, H, s_hb, 1};
      const WgradTarget wt = wgrad_target(c->i_head_w);
      // The head's input gradient and weight gradient need the same logit gradient and nothing of
      // each other.  The former has fewer tiles than the chip has CUs (a long contraction over
      // the classes): with an auxiliary stream the two run side by side and the tiles of the
      // weight gradient fill the CUs the other leaves idle.  One event pair brackets both.
      const bool side_by_side = c->aux && c->ev_fork && c->ev_join;
      // in parts where the product's tiles leave the chip idle (M = 480, N = 224, 10 000 classes, K = 4:
      // 32 tiles, 124 us in one piece)
      const int ns = dx_splits(nrows, H, Kv, c->K, 128, 512), part = (Kv / 64 + ns) / ns * 64;
      const int n_parts = (Kv + part - 1) / part;
      const size_t n_dx = (size_t)nrows * H;
      const bool in_parts = ns > 1 && n_parts > 1 && c->dxp.stride >= (size_t)n_parts * n_dx;
      float* dfeat = lm ? dx : D;
      const long s_dfeat = lm ? s_dx : s_D;
      // (bf16 operands only: the fp32 head matrix may be updated in place beside the input gradient)
      const GemmBf16Args jobs[2] = {
          {vdl.p, vdl.ld, vdl.stride, vw.p, vw.ld, vw.stride, in_parts ? reg(c->dxp) : dfeat, H, in_parts ? (long)n_dx : s_dfeat,
           nullptr, 0, 0.f, nrows, H, in_parts ? part : Kv, groups, 0, 0, 2, in_parts ? n_parts : 1, in_parts ? Kv : 0},
          {vdo.p, vdo.ld, vdo.stride, vho.p, vho.ld, vho.stride, wt.C, Hc, wt.sC, wt.aux, sRi, lr, classes, Hc, nrows, groups, 0, 0, 3}};
      const bool together = gemm_bf16_multi_pays(jobs, 2);
      const bool fork = side_by_side && !together;
      if (fork &&
          (hipEventRecord(c->ev_fork, s) != hipSuccess || hipStreamWaitEvent(c->aux, c->ev_fork, 0) != hipSuccess))
        return HPSGD_EHIP;
      {
        TimerScope pair(c, role, s, together ? 1 : 2);
        const bool nested = c->timer_nested;
        c->timer_nested = c->timer_nested || pair.active();
        if (together) {
          HIP_TRY(launch_gemm_bf16_multi(jobs, 2, s));
        } else if (in_parts) {
          HIP_TRY(launch_gemm_bf16_nt(vdl.p, 1, vdl.ld, vdl.stride, vw.p, 1, vw.ld, vw.stride, reg(c->dxp), H, (long)n_dx, nullptr, 0,
                                      nullptr, 0, 0.f, nrows, H, part, groups, s, 0, 0, 0, n_parts, Kv, vw.outer << 1));
        } else {
          TRY(gemm2(s, groups, bf, nrows, H, Kv, logits, ldl, s_log, 0, rin + oW, H, sRi, 0, dfeat, H, s_dfeat, EPI_STORE,
                    nullptr, 0, vdl, vw, 0.f, true));
        }
        if (!together)
          TRY(gemm2(fork ? c->aux : s, groups, bf, classes, Hc, nrows, logits, ldl, s_log, 1, feats, H, s_top,
                    0, wt.C, Hc, wt.sC, wt.epi, wt.aux, sRi, vdo, vho, lr, true));
        // What is added up from parts, and the mean loss, in one launch: the input gradient, and the bias gradient
        // from the loss kernel's column sums, with its update unless the gradients are accumulated as well.
        // (Side by side the weight gradient outlasts the input gradient: this runs beside it.)
        {
          const int saved_role = role;
          role = HPSGD_ROLE_OTHER;
          ReducePack rp;
          rp.n = 0;
          rp.blk0[0] = 0;
          rp.lr = lr;
          if (loss_out) {
            rp.rowloss = rowloss; rp.s_rowloss = (long)c->rowloss.stride;
            rp.loss = loss_out; rp.rows = nrows; rp.count = lm ? TBc : Bc;
          }
          if (!acc) fused_commit[c->i_head_b] = 1;
          if ((in_parts && !reduce_pack_push(rp, reg(c->dxp), n_parts, n_dx, nullptr, 0, dfeat, (size_t)s_dfeat, 0)) ||
              !reduce_pack_push(rp, reg(c->colpart), n_colparts, (size_t)classes, acc ? nullptr : rin + ob, (size_t)sRi,
                                acc ? grad + ob : rout + ob, (size_t)(acc ? sG : sR), acc ? 0 : 1, (size_t)colpitch))
            return HPSGD_ESHAPE;
          HIP_TRY(launch_reduce_pack(rp, groups, s));
          role = saved_role;
        }
        if (fork &&
            (hipEventRecord(c->ev_join, c->aux) != hipSuccess || hipStreamWaitEvent(s, c->ev_join, 0) != hipSuccess))
          return HPSGD_EHIP;
        c->timer_nested = nested;
      }
    } else if (!bf && !lm && cls_head_supported(nrows, classes, H)) {
      // a classifier head with few classes: forward and loss in one small launch, the three
      // gradients and the update (or the gradients, when they are accumulated as well) in another
      role = HPSGD_ROLE_GEMM_HEAD;
      TimerScope ts_(c, role, s);
      if (acc) {
        HIP_TRY(launch_cls_head(feats, s_top, rin + oW, rin + ob, sRi, y, nrows, logits, s_log, rowloss,
                                (long)c->rowloss.stride, D, s_D, grad + oW, grad + ob, sG, lr, 0, loss_out, nrows,
                                classes, H, groups, s));
      } else {
        fused_commit[c->i_head_w] = 1;
        fused_commit[c->i_head_b] = 1;
        HIP_TRY(launch_cls_head(feats, s_top, rin + oW, rin + ob, sRi, y, nrows, logits, s_log, rowloss,
                                (long)c->rowloss.stride, D, s_D, rout + oW, rout + ob, sR, lr, 1, loss_out, nrows,
                                classes, H, groups, s));
      }
    } else {
      role = HPSGD_ROLE_GEMM_HEAD;
      {
        const NtView va{feats, 0, H, s_top}, vb{rin + oW, 0, H, sRi};
        TRY(gemm2(s, groups, bf, nrows, classes, H, feats, H, s_top, 0, rin + oW, H, sRi, 1, logits, classes,
                  s_log, EPI_BIAS, rin + ob, sRi, va, vb));
      }
      role = HPSGD_ROLE_LOSS;
      HIP_TRY(launch_softmax_ce(logits, s_log, y, nrows, logits, rowloss, (long)c->rowloss.stride, nrows,
                                classes, groups, s));
      if (bf && loss_out)
        HIP_TRY(launch_loss_mean(rowloss, (long)c->rowloss.stride, loss_out, nrows, groups, s));
      // ---- backward: head
      // bf16 precision: transposed bf16 copies (contraction-contiguous operands for the NT kernel)
      if (ntc) {
        role = HPSGD_ROLE_OTHER;
        if (!gru_fused_bf16_supported(H))  // else written by the forward step kernels
          for (int l = 0; l < L; ++l)      // hs^T of every layer: [H][(T+1)B]
            HIP_TRY(launch_cvt_bf16(reg(c->hs[l]), H, (long)c->hs[l].stride, bfreg(c->hsT[l]), TB1p,
                                    2 * (long)c->hsT[l].stride, TB + B, H, true, groups, s));
        HIP_TRY(launch_cvt_bf16(logits, classes, s_log, bfreg(c->dlogT), nrp, 2 * (long)c->dlogT.stride, nrows,
                                classes, true, groups, s));
        HIP_TRY(launch_cvt_bf16(rin + oW, H, sRi, bfreg(c->woT), clp, 2 * (long)c->woT.stride, classes, H, true,
                                groups, s));
      }
      role = HPSGD_ROLE_GEMM_HEAD;
      if (!bf) {
        // the input gradient now (it reads the head's matrix), in parts where its tiles leave the chip idle;
        // weight and bias gradients and the mean loss with the top layer's products, behind its recurrence
        float* dfeat = lm ? dx : D;
        const int ns = dx_splits(nrows, H, classes, c->K, 64, 256), part = wgrad_part(classes, ns);
        const int n_parts = (classes + part - 1) / part;
        if (n_parts > 1 && H >= 4 && classes - (n_parts - 1) * part >= 4 && c->dxp.stride >= (size_t)n_parts * nrows * H) {
          const size_t n = (size_t)nrows * H;
          float* parts = reg(c->dxp);
          TRY(gemm(s, groups, 0, nrows, H, part, logits, classes, s_log, 0, rin + oW, H, sRi, 0, parts, H, (long)n, EPI_STORE,
                   nullptr, 0, 0, 0.f, n_parts, classes));
          HIP_TRY(launch_reduce_parts(parts, n_parts, n, nullptr, 0, dfeat, (size_t)(lm ? s_dx : s_D), 0.f, 0, groups, s));
        } else {
          TRY(gemm(s, groups, 0, nrows, H, classes, logits, classes, s_log, 0, rin + oW, H, sRi, 0, dfeat, H, lm ? s_dx : s_D,
                   EPI_STORE, nullptr, 0));
        }
        const WgradTarget wt = wgrad_target(c->i_head_w);
        TRY(gb.add(gemm_desc(groups, 0, classes, H, nrows, logits, classes, s_log, 1, feats, H, s_top, 0, wt.C, H, wt.sC, wt.epi,
                             wt.aux, sRi, 0, lr)));
        if (acc) {
          (void)colsum_pack_push(gb.cs, logits, classes, s_log, grad + ob, sG, nullptr, 0, nrows, classes);
        } else {
          fused_commit[c->i_head_b] = 1;
          (void)colsum_pack_push(gb.cs, logits, classes, s_log, rout + ob, sR, rin + ob, sRi, nrows, classes);
        }
        if (loss_out)
          (void)colsum_pack_push(gb.cs, rowloss, 1, (long)c->rowloss.stride, loss_out, 1, nullptr, 0, nrows, 1, 1.0f / (float)nrows);
      } else {
        NtView va, vb, vw;
        if (ntc) {
          va = NtView{bfreg(c->dlogT), 1, nrp, 2 * (long)c->dlogT.stride};
          vb = NtView{bfreg(c->hsT[L - 1]) + (lm ? B : T * B), 1, TB1p, 2 * (long)c->hsT[L - 1].stride};
          vw = NtView{bfreg(c->woT), 1, clp, 2 * (long)c->woT.stride};
        }
        const NtView vl{logits, 0, classes, s_log};
        if (lm) {
          TRY(gemm2(s, groups, bf, TB, H, classes, logits, classes, s_log, 0, rin + oW, H, sRi, 0, dx, H, s_dx,
                    EPI_STORE, nullptr, 0, vl, vw));
        } else {
          TRY(gemm2(s, groups, bf, B, H, classes, logits, classes, s_log, 0, rin + oW, H, sRi, 0, D, H, s_D,
                    EPI_STORE, nullptr, 0, vl, vw));
        }
        const WgradTarget wt = wgrad_target(c->i_head_w);
        TRY(gemm2(s, groups, bf, classes, H, nrows, logits, classes, s_log, 1, feats, H, s_top, 0, wt.C, H, wt.sC,
                  wt.epi, wt.aux, sRi, va, vb, lr));
        HIP_TRY(launch_colsum(logits, classes, s_log, grad + ob, sG, nrows, classes, groups, s));
      }
    }
    // the embedding gradient from the first layer's input gradient dx (Alg. 2 "update replica"
    // for the table, when the update is in place)
    bool embed_done = false;
    // clones: the table is written out first (one read, a write per worker), then updated like
    // one that is already there.  (Nothing of the step reads the output table, so the copy could be
    // issued earlier; beside the layer above's weight gradients it cost more than it saved here.)
    bool table_out = false;
    auto embed_table_out = [&](hipStream_t st) -> int {
      const size_t oE = c->eoff(c->i_embed);
      if (table_out || acc || !cloned || !lm || !aligned16(rin + oE) || !aligned16(rout + oE) || (sR & 3) != 0 ||
          groups > HPSGD_KMAX)
        return HPSGD_OK;
      PtrPack pk;
      for (int g = 0; g < groups; ++g) pk.p[g] = rout + oE + (size_t)g * sR;
      if (launch_sync_all(rin + oE, pk, groups, nullptr, (size_t)d.vocab * d.embed, st) != hipSuccess) return HPSGD_EHIP;
      table_out = true;
      return HPSGD_OK;
    };
    auto embed_grad = [&](hipStream_t st) -> int {
      const size_t oE = c->eoff(c->i_embed);
      TRY0(embed_table_out(st));
      if (!acc && (rin == rout || table_out)) {
        // an update in place: only the rows of the tokens of the batch change, and their owners
        // write them; no gradient table to clear, fill and stream through the commit kernel
        fused_commit[c->i_embed] = 1;
        if (launch_embed_bwd(dx, width0, s_dx, tok, TBc, rout + oE, sR, TBc, Bc, B, Ec, groups, st, rin + oE, sRi, lr) != hipSuccess)
          return HPSGD_EHIP;
      } else {
        if (launch_fill_zero(grad + oE, (size_t)d.vocab * d.embed, (size_t)sG, groups, st) != hipSuccess ||
            launch_embed_bwd(dx, width0, s_dx, tok, TBc, grad + oE, sG, TBc, Bc, B, Ec, groups, st) != hipSuccess)
          return HPSGD_EHIP;
      }
      return HPSGD_OK;
    };
    const float* above = nullptr;  // (see above: gb holds what waits for the top layer's products)
    // the gradient carried into a layer's last step is zero unless the head wrote it (the
    // classifier on the top layer): a resident-weight launch is told so, any other path has D cleared
    bool d_zero = false;
    if (lm) {
      above = dx;
      d_zero = true;
    }
    // what a layer adds up from parts (both layers of a stack, whose products go out together)
    ReducePack rp;
    float* parts = nullptr;  // the next free place for parts of weight gradients
    // ---- backward: GRU layers, top to bottom
    for (int l = L - 1; l >= 0; --l) {
      const bool joined = use_stack && l > 0;  // the layer below comes with this one
      const bool up_b = use_stack_b && l > 0;
      const float* hs = reg(c->hs[l]);
      const float* sv = reg(c->sv[l]);
      const long s_hs = (long)c->hs[l].stride, s_sv = (long)c->sv[l].stride;
      const int win = l > 0 ? H : width0, winc = l > 0 ? Hc : Ec;  // internal, and the model's own
      const int gp = H != Hc ? H : 0, gh = H != Hc ? Hc : 0;  // rows of the weight gradients in gate blocks
      if (!use_stack || l == L - 1) {
        rp.n = 0;
        rp.blk0[0] = 0;
        rp.lr = lr;
        parts = c->dwip.stride ? reg(c->dwip) : nullptr;
      }
      // queued for the layer's one adding launch; a segment that launch cannot take runs by itself
      auto queue_reduce = [&](const float* parts, int n_parts, size_t n, const float* in, size_t s_in, float* out,
                              size_t s_out, int commit) -> int {
        if (reduce_pack_push(rp, parts, n_parts, n, in, s_in, out, s_out, commit)) return HPSGD_OK;
        return launch_reduce_parts(parts, n_parts, n, in, s_in, out, s_out, lr, commit, groups, s) == hipSuccess
                   ? HPSGD_OK
                   : HPSGD_EHIP;
      };
      const float* layer_in;
      long s_layer_in;
      if (l > 0) {
        layer_in = reg(c->hs[l - 1]) + (size_t)B * H;
        s_layer_in = (long)c->hs[l - 1].stride;
      } else if (lm) {
        layer_in = reg(c->xe);  // (not made, and not read, in the padded layout)
        s_layer_in = (long)c->xe.stride;
      } else {
        layer_in = (const float*)x;
        s_layer_in = (long)TB * d.input;
      }
      float* dgx = joined ? reg(c->gx_up) : gx;  // the gate pre-activation buffer is free once the layer's forward is done
      float* dgh = joined ? reg(c->dgh_up) : dgh_lo;
      const float* Whh = rin + c->eoff(c->lidx[l].whh);
      const bool fused = !bf && gru_fused_supported(H) && ((uintptr_t)Whh & 15) == 0 && (sRi & 3) == 0;
      const bool fused_b = bf && gru_fused_bf16_supported(H);
      float* wt = reg(c->wt);
      const long s_wt = (long)c->wt.stride;
      __bf16* dghb = fused_b ? (__bf16*)reg(c->dghb) : nullptr;
      const long s_dgb = 2 * (long)c->dghb.stride;
      const bool stepT = fused_b && ntc && win % 8 == 0;  // the step kernels write the bf16 copies
      __bf16* dgxb = stepT ? bfreg(c->dgxb) : nullptr;
      const long s_T = 2 * (long)c->dgxT.stride;
      if (fused && !use_persist && !use_solo) {
        role = HPSGD_ROLE_OTHER;
        HIP_TRY(launch_transpose(Whh, sRi, wt, s_wt, 3 * H, H, groups, s));
      }
      const void* wtb = wt;   // bf16 W_hh^T of this layer
      long s_wtb = 2 * s_wt;
      if (fused_b && whhT_ready[l]) {
        wtb = bfreg(c->whhT[l]);
        s_wtb = wstride(c->whhT[l]);
      } else if (fused_b) {
        role = HPSGD_ROLE_OTHER;
        HIP_TRY(launch_cvt_bf16(Whh, H, sRi, wt, 3 * H, 2 * s_wt, 3 * H, H, true, groups, s));
      }
      // fp32 path with an auxiliary stream: the weight-gradient GEMMs of the time steps that
      // BPTT has already finished run on that stream beside the rest of the recurrence (the
      // recurrence is latency-bound and leaves the matrix cores mostly idle).  The steps are
      // cut into chunks; chunk c's GEMMs are issued when BPTT has walked past it, the last
      // one follows on the main stream after the join.  Fixed chunking: deterministic.
      const bool persist = use_persist;
      const bool persist_b = fused_b && use_persist_b && stepT;
      if (d_zero && !persist && !persist_b && !use_solo) {
        role = HPSGD_ROLE_OTHER;
        HIP_TRY(launch_fill_zero(D, (size_t)B * H, (size_t)s_D, groups, s));
      }
      // the resident-weight kernel accumulates dW_hh itself (one partial sum per batch-row tile)
      float* dwp = persist && c->dwp.stride ? reg(c->dwp) : nullptr;
      // ... and the bias gradients
      float* dbp = joined || up_b ? reg(c->dbp_up) : persist || persist_b || use_solo ? reg(c->dbp) : nullptr;
      const int NC = (c->aux && fused && !persist && !use_solo && T >= 8) ? 4 : 1;
      auto chunk_lo = [&](int ch) { return (int)((long)T * ch / NC); };
      auto wgrad_rows = [&](hipStream_t st, int t0, int t1, int epi) -> int {
        const size_t r0 = (size_t)t0 * B;
        const int rows = (t1 - t0) * B;
        const int bg = st != s;  // on the auxiliary stream: beside the recurrence
        int rc = gemm(st, groups, bf, 3 * H, win, rows, dgx + r0 * 3 * H, 3 * H, s_gx, 1, layer_in + r0 * win,
                      win, s_layer_in, 0, grad + c->eoff(c->lidx[l].wih), win, sG, epi, nullptr, 0, bg);
        if (rc != HPSGD_OK) return rc;
        return gemm(st, groups, bf, 3 * H, H, rows, dgh + r0 * 3 * H, 3 * H, s_gx, 1, hs + r0 * H, H, s_hs, 0,
                    grad + c->eoff(c->lidx[l].whh), H, sG, epi, nullptr, 0, bg);
      };
      {
      TimerScope loop_bwd(c, HPSGD_ROLE_GEMM_REC_BWD, s, use_stack && !joined ? 0 : (persist || persist_b || use_solo) ? 1 : (fused || fused_b) ? T : 0);
      c->timer_nested = loop_bwd.active() && (fused || fused_b || use_solo || persist);
      if (use_stack) {
        role = HPSGD_ROLE_GEMM_REC_BWD;
        if (joined) {
          HIP_TRY(launch_gru_stack_bwd(stack_layer(0), stack_layer(1), rin + c->eoff(c->lidx[1].wih), sRi, d_zero ? nullptr : D, s_D, above, s_dx,
                                       reg(c->dx_up), (long)c->dx_up.stride, s_gx, s_hs, s_sv, B, H, T, groups, psync, c->link_limit(), s));
        }
      } else if (use_solo) {
        role = HPSGD_ROLE_GEMM_REC_BWD;
        HIP_TRY(launch_gru_solo_bwd(Whh, sRi, dgx, dgh, s_gx, d_zero ? nullptr : D, s_D, above, s_dx, sv, s_sv, hs, s_hs, dbp,
                                    B, H, T, groups, c->K, s));
      }
      int next_chunk = NC - 1;  // the chunk BPTT is walking through
      // resident weights: all of BPTT is one launch; its weight-gradient GEMMs follow it (work
      // that shares the CUs with this launch slows its chain of waits by more than it hides)
      if (persist) {
        role = HPSGD_ROLE_GEMM_REC_BWD;
        // (the row-major gate gradients only when a later launch reads them)
        HIP_TRY(launch_gru_bwd_persist(Whh, sRi, (dwp && dbp) ? nullptr : dgh, reg(c->dghx), (long)c->dghx.stride, dgx, s_gx,
                                       D, s_D, d_zero, above, s_dx, sv, s_sv, hs, s_hs, B, H, T,
                                       groups, prow, psync, pbase, c->spin_limit, dwp, dbp, c->device_scope, &ticket_launches, s));
        c->last_dw += dwp ? 1 : 0;
        pbase += (unsigned)T * gru_persist_count_per_step(H);
        if (l == 0) TRY0(resident.mark());
        else resident.note();
      }
      if (persist_b && use_solo_b) {
        role = HPSGD_ROLE_GEMM_REC_BWD;
        if (up_b)
          HIP_TRY(launch_gru_stack_bwd_bf16(stack_layer_b(0), stack_layer_b(1), bfreg(c->wihT), wstride(c->wihT), s_wtb, above, s_dx,
                                            reg(c->dx_up), (long)c->dx_up.stride, s_hs, s_sv, 2 * (long)c->dghx.stride, Hc, B, H, T, groups,
                                            psync, c->link_limit(), s));
        // (gate gradients r | z | n | q, in the place of the exchange buffer)
        if (!use_stack_b) HIP_TRY(launch_gru_solo_bwd_bf16(wtb, s_wtb, above, s_dx, sv, s_sv, hs, s_hs, bfreg(c->dghx), 2 * (long)c->dghx.stride, dbp, Hc,
                                         B, H, T, groups, c->K, s));
        HIP_TRY(launch_transpose_dg4(up_b ? bfreg(c->dg4_up) : bfreg(c->dghx), 2 * (long)c->dghx.stride, bfreg(c->dgxT), bfreg(c->dghT), TBp, s_T, TB, H, groups, s));
      } else if (persist_b) {
        role = HPSGD_ROLE_GEMM_REC_BWD;
        HIP_TRY(launch_gru_bwd_persist_bf16(wtb, s_wtb, bfreg(c->dghx), 2 * (long)c->dghx.stride, s_dgb, D, s_D, d_zero,
                                            above, s_dx, sv, s_sv, hs, s_hs, dgxb, bfreg(c->dgxT), bfreg(c->dghT), TBp, s_T, dbp, Hc, B,
                                            H, T, groups, prow, psync, pbase, c->spin_limit, c->device_scope, &ticket_launches, s));
        pbase += (unsigned)T * gru_persist_bf16_count_per_step(H);
        if (l == 0) TRY0(resident.mark());
        else resident.note();
      }
      for (int t = T - 1; t >= 0 && !persist && !persist_b && !use_solo; --t) {
        if (NC > 1 && next_chunk >= 1 && t < chunk_lo(next_chunk)) {
          // steps [chunk_lo, chunk_hi) are done: hand their weight gradients to the aux stream
          if (hipEventRecord(c->ev_fork, s) != hipSuccess || hipStreamWaitEvent(c->aux, c->ev_fork, 0) != hipSuccess)
            return HPSGD_EHIP;
          const int rc = wgrad_rows(c->aux, chunk_lo(next_chunk), chunk_lo(next_chunk + 1),
                                    next_chunk == NC - 1 ? EPI_STORE : EPI_ACCUM);
          if (rc != HPSGD_OK) return rc;
          --next_chunk;
        }
        const float* above_t = above ? above + (size_t)t * B * H : nullptr;
        if (fused_b) {
          role = HPSGD_ROLE_GEMM_REC_BWD;
          HIP_TRY(launch_gru_bwd_step_bf16(wtb, s_wtb, t + 1 < T ? dghb + (size_t)(t + 1) * B * 3 * H : nullptr,
                                           dghb + (size_t)t * B * 3 * H, s_dgb, D, s_D, above_t, s_dx,
                                           sv + (size_t)t * B * 4 * H, s_sv, hs + (size_t)t * B * H, s_hs,
                                           dgx + (size_t)t * B * 3 * H, dgh + (size_t)t * B * 3 * H, s_gx,
                                           dgxb ? dgxb + (size_t)t * B * 3 * H : nullptr,
                                           dgxb ? bfreg(c->dgxT) + (size_t)t * B : nullptr,
                                           dgxb ? bfreg(c->dghT) + (size_t)t * B : nullptr, TBp, s_T, B, H,
                                           groups, s));
          continue;
        }
        if (fused) {
          role = HPSGD_ROLE_GEMM_REC_BWD;
          HIP_TRY(launch_gru_bwd_step(wt, s_wt, t + 1 < T ? dgh + (size_t)(t + 1) * B * 3 * H : nullptr, s_gx,
                                      D, s_D, above_t, s_dx, sv + (size_t)t * B * 4 * H, s_sv,
                                      hs + (size_t)t * B * H, s_hs, dgx + (size_t)t * B * 3 * H,
                                      dgh + (size_t)t * B * 3 * H, B, H, groups, s));
          continue;
        }
        role = HPSGD_ROLE_CELL_BWD;
        HIP_TRY(launch_gru_cell_bwd(D, s_D, above_t, s_dx, sv + (size_t)t * B * 4 * H, s_sv,
                                    hs + (size_t)t * B * H, s_hs, dgx + (size_t)t * B * 3 * H,
                                    dgh + (size_t)t * B * 3 * H, s_gx, B, H, groups, s));
        role = HPSGD_ROLE_GEMM_REC_BWD;
        if (t > 0)
          TRY(gemm(s, groups, bf, B, H, 3 * H, dgh + (size_t)t * B * 3 * H, 3 * H, s_gx, 0, Whh, H, sRi, 0, D,
                   H, s_D, EPI_ACCUM, nullptr, 0));
      }
      c->timer_nested = false;
      }
      const float* Wih = rin + c->eoff(c->lidx[l].wih);
      const bool need_dx = (l > 0 || lm) && !joined && !up_b;
      NtView v_dgxT, v_dghT, v_xT, v_hsT, v_wih;
      if (ntc && win % 8 == 0) {
        role = HPSGD_ROLE_OTHER;
        if (!stepT) {
          HIP_TRY(launch_cvt_bf16(dgx, 3 * H, s_gx, bfreg(c->dgxT), TBp, 2 * (long)c->dgxT.stride, TB, 3 * H,
                                  true, groups, s));
          HIP_TRY(launch_cvt_bf16(dgh, 3 * H, s_gx, bfreg(c->dghT), TBp, 2 * (long)c->dghT.stride, TB, 3 * H,
                                  true, groups, s));
        }
        v_dgxT = NtView{bfreg(c->dgxT), 1, TBp, 2 * (long)c->dgxT.stride};
        v_dghT = NtView{bfreg(c->dghT), 1, TBp, 2 * (long)c->dghT.stride};
        v_hsT = NtView{bfreg(c->hsT[l]), 1, TB1p, 2 * (long)c->hsT[l].stride};
        if (l > 0) {
          v_xT = NtView{bfreg(c->hsT[l - 1]) + B, 1, TB1p, 2 * (long)c->hsT[l - 1].stride};
        } else {
          if (!xT_ready)
            HIP_TRY(launch_cvt_bf16(layer_in, win, s_layer_in, bfreg(c->xT), TBp, 2 * (long)c->xT.stride, TB,
                                    win, true, groups, s));
          v_xT = NtView{bfreg(c->xT), 1, TBp, 2 * (long)c->xT.stride};
        }
        if (need_dx && wc.wih[l] && stepT) {  // (the row-major copy: the contraction runs over its rows)
          v_wih = NtView{bfreg(c->wihbl[l]), 1, c->wih_pitch(l), wstride(c->wihbl[l]), 1};
        } else if (need_dx) {
          HIP_TRY(launch_cvt_bf16(Wih, win, sRi, bfreg(c->wihT), 3 * H, 2 * (long)c->wihT.stride, 3 * H, win, true,
                                  groups, s));
          v_wih = NtView{bfreg(c->wihT), 1, 3 * H, 2 * (long)c->wihT.stride};
        }
      }
      // bf16 operands and few tiles: the input gradient (from bf16 copies, not from the weights that the others update in
      // place) and both weight gradients in one launch
      bool together = false;
      if (persist_b && stepT && NC == 1 && v_dgxT.bf16 && v_dghT.bf16 && v_xT.bf16 && v_hsT.bf16 && (!need_dx || v_wih.outer)) {
        const WgradTarget wi = wgrad_target(c->lidx[l].wih), wh = wgrad_target(c->lidx[l].whh);
        const GemmBf16Args jobs[3] = {
            {v_dghT.p, v_dghT.ld, v_dghT.stride, v_hsT.p, v_hsT.ld, v_hsT.stride, wh.C, Hc, wh.sC, wh.aux, sRi, lr, 3 * H, Hc, TB, groups,
             gp, gh},
            {v_dgxT.p, v_dgxT.ld, v_dgxT.stride, v_xT.p, v_xT.ld, v_xT.stride, wi.C, winc, wi.sC, wi.aux, sRi, lr, 3 * H, winc, TB, groups,
             gp, gh},
            {use_solo_b ? (const void*)bfreg(c->dghx) : dgxb, use_solo_b ? 4L * H : 3L * H, use_solo_b ? 2 * (long)c->dghx.stride : s_dgb,
             v_wih.p, v_wih.ld, v_wih.stride, dx, win, s_dx, nullptr, 0, 0.f, TB, win, 3 * H, groups, 0, 0, 2}};
        const int n_jobs = need_dx ? 3 : 2;
        if (gemm_bf16_multi_pays(jobs, n_jobs)) {
          role = HPSGD_ROLE_GEMM_WGRAD;
          HIP_TRY(launch_gemm_bf16_multi(jobs, n_jobs, s));
          together = true;
          if (need_dx) above = dx;
        }
      }
      role = HPSGD_ROLE_GEMM_DX;
      // bf16 operands: the input gradient reads only bf16 copies (not the weights the gradient
      // GEMMs below update in place) and has fewer tiles than the chip has CUs: with an auxiliary
      // stream it runs beside the layer's weight-gradient GEMMs (its launch is then not timed)
      bool dx_beside = false, swap = false;
      if (need_dx && !together) {  // reads W_ih: before its update
        const NtView v_dgx = use_solo_b ? NtView{bfreg(c->dghx), 1, 4 * H, 2 * (long)c->dghx.stride}
                             : stepT    ? NtView{dgxb, 1, 3 * H, s_dgb}
                                        : NtView{dgx, 0, 3 * H, s_gx};
        dx_beside = persist_b && stepT && v_wih.bf16 && c->aux && c->ev_fork && c->ev_join && NC == 1;
        // Above the first layer the input gradient is the product with the long tiles (a contraction
        // over 3H, fewer tiles than CUs): it goes first, on this stream, and the first weight
        // gradient beside it on the auxiliary one, whose many short tiles fill in around it (issued
        // the other way round, the weight gradient's first wave of tiles held every CU and the
        // long tiles started a tile late).  The first layer's input gradient is short and has the
        // embedding gradient behind it: it stays on the auxiliary stream.
        swap = dx_beside && l > 0;
        if (swap) {
          if (hipEventRecord(c->ev_fork, s) != hipSuccess || hipStreamWaitEvent(c->aux, c->ev_fork, 0) != hipSuccess)
            return HPSGD_EHIP;
          TRY(gemm2(s, groups, bf, TB, win, 3 * H, dgx, 3 * H, s_gx, 0, Wih, win, sRi, 0, dx, win, s_dx, EPI_STORE,
                    nullptr, 0, v_dgx, v_wih, 0.f, persist_b));
        } else if (dx_beside) {
          if (hipEventRecord(c->ev_fork, s) != hipSuccess || hipStreamWaitEvent(c->aux, c->ev_fork, 0) != hipSuccess)
            return HPSGD_EHIP;
          TRY0(gemm2(c->aux, groups, bf, TB, win, 3 * H, dgx, 3 * H, s_gx, 0, Wih, win, sRi, 0, dx, win, s_dx,
                     EPI_STORE, nullptr, 0, v_dgx, v_wih, 0.f, persist_b));
          // the embedding rows need this product and nothing of the weight gradients beside it
          if (l == 0 && lm) {
            TRY0(embed_grad(c->aux));
            embed_done = true;
          }
          if (hipEventRecord(c->ev_join, c->aux) != hipSuccess) return HPSGD_EHIP;
        } else if (!bf) {
          TRY(gb.add(gemm_desc(groups, 0, TB, win, 3 * H, dgx, 3 * H, s_gx, 0, Wih, win, sRi, 0, dx, win, s_dx, EPI_STORE,
                               nullptr, 0)));
        } else {
          TRY(gemm2(s, groups, bf, TB, win, 3 * H, dgx, 3 * H, s_gx, 0, Wih, win, sRi, 0, dx, win, s_dx, EPI_STORE,
                    nullptr, 0, v_dgx, v_wih, 0.f, persist_b));
        }
        above = dx;
      }
      role = HPSGD_ROLE_GEMM_WGRAD;
      if (together) {
        // issued above
      } else if (NC > 1) {
        TRY(gb.flush());
        // join, then the first chunk's share on top of what the aux stream accumulated
        if (hipEventRecord(c->ev_join, c->aux) != hipSuccess || hipStreamWaitEvent(s, c->ev_join, 0) != hipSuccess)
          return HPSGD_EHIP;
        TRY(wgrad_rows(s, 0, chunk_lo(1), EPI_ACCUM));
      } else {
        const WgradTarget wi = wgrad_target(c->lidx[l].wih);
        bool hh_first = false;
        // fp32: a gradient with few tiles has its contraction cut into parts (wgrad_splits); their sums are
        // added in order by the kernel that also applies the update
        auto split_wgrad = [&](const float* A, const float* Bm, long sB, int N, const WgradTarget& w) -> int {
          const int ns = c->wgrad_parts(3 * H, N, TB), part = wgrad_part(TB, ns);
          const int n_parts = (TB + part - 1) / part;
          const size_t n = (size_t)3 * H * N;
          int rc = gb.add(gemm_desc(groups, 0, 3 * H, N, part, A, 3 * H, s_gx, 1, Bm, N, sB, 0, parts, N, (long)n, EPI_STORE,
                                    nullptr, 0, 0, 0.f, n_parts, TB));
          if (rc != HPSGD_OK) return rc;
          rc = queue_reduce(parts, n_parts, n, w.aux, (size_t)sRi, w.C, (size_t)w.sC, w.epi == EPI_COMMIT);
          parts += (size_t)groups * n_parts * n;  // (all K workers, or one: its own slice)
          return rc;
        };
        // (the pipelined kernel takes operands of at least one vector along their unit-stride index)
        const bool split_wih = !bf && win >= 4 && 3 * H >= 4 && c->wgrad_parts(3 * H, win, TB) > 1;
        const bool split_whh = !bf && !dwp && H >= 4 && c->wgrad_parts(3 * H, H, TB) > 1;
        if (split_wih) {
          TRY(split_wgrad(dgx, layer_in, s_layer_in, win, wi));
        } else {
          // the first layer beside its input gradient: the recurrent weight gradient (the longer
          // tiles) before the input one, whose short tiles fill in at the end
          hh_first = dx_beside && !swap && !dwp;
          bool paired = false;
          if (hh_first) {
            const WgradTarget wh = wgrad_target(c->lidx[l].whh);
            // ... and both in one launch when both are updates in place: neither needs the other,
            // and on one stream the second would wait for the first one's last, partial round
            if (wh.epi == EPI_COMMIT && wi.epi == EPI_COMMIT && v_dghT.bf16 && v_hsT.bf16 && v_dgxT.bf16 && v_xT.bf16) {
              const GemmBf16Args ph{v_dghT.p, v_dghT.ld, v_dghT.stride, v_hsT.p, v_hsT.ld, v_hsT.stride, wh.C, Hc, wh.sC,
                                    wh.aux, sRi, lr, 3 * H, Hc, TB, groups, gp, gh};
              const GemmBf16Args pi{v_dgxT.p, v_dgxT.ld, v_dgxT.stride, v_xT.p, v_xT.ld, v_xT.stride, wi.C, winc, wi.sC,
                                    wi.aux, sRi, lr, 3 * H, winc, TB, groups, gp, gh};
              if (gemm_bf16_update_pair_supported(ph, pi)) {
                HIP_TRY(launch_gemm_bf16_update_pair(ph, pi, s));
                paired = true;
              }
            }
            if (!paired)
              TRY(gemm2(s, groups, bf, 3 * H, Hc, TB, dgh, 3 * H, s_gx, 1, hs, H, s_hs, 0, wh.C, Hc, wh.sC, wh.epi,
                        wh.aux, sRi, v_dghT, v_hsT, lr, persist_b, gp, gh));
          }
          if (paired) {
            // issued above
          } else if (!bf) {
            // (updates, in place, the matrix that the input gradient waiting beside it reads)
            if (need_dx) TRY(gb.flush());
            TRY(gb.add(gemm_desc(groups, 0, 3 * H, win, TB, dgx, 3 * H, s_gx, 1, layer_in, win, s_layer_in, 0, wi.C, win, wi.sC,
                                 wi.epi, wi.aux, sRi, 0, lr)));
          } else if (swap) {
            // (both streams become runnable at the same event; a few microseconds' head start keeps the
            // long tiles in front also when this stream has marker packets - a timer's events - to
            // get through first)
            if (launch_delay(kAuxHeadStartUs, c->aux) != hipSuccess) return HPSGD_EHIP;
            TRY0(gemm2(c->aux, groups, bf, 3 * H, winc, TB, dgx, 3 * H, s_gx, 1, layer_in, win, s_layer_in, 0, wi.C, winc,
                       wi.sC, wi.epi, wi.aux, sRi, v_dgxT, v_xT, lr, persist_b, gp, gh));
            if (hipEventRecord(c->ev_join, c->aux) != hipSuccess) return HPSGD_EHIP;
          } else {
            TRY(gemm2(s, groups, bf, 3 * H, winc, TB, dgx, 3 * H, s_gx, 1, layer_in, win, s_layer_in, 0, wi.C, winc,
                      wi.sC, wi.epi, wi.aux, sRi, v_dgxT, v_xT, lr, persist_b, gp, gh));
          }
        }
        if (hh_first) {
          // issued above
        } else if (dwp) {
          const WgradTarget wh = wgrad_target(c->lidx[l].whh);
          TRY0(queue_reduce(dwp, (B + prow - 1) / prow, (size_t)3 * H * H, wh.aux, (size_t)sRi, wh.C, (size_t)wh.sC,
                           wh.epi == EPI_COMMIT));
        } else if (split_whh) {
          TRY(split_wgrad(dgh, hs, s_hs, H, wgrad_target(c->lidx[l].whh)));
        } else if (!bf) {
          const WgradTarget wh = wgrad_target(c->lidx[l].whh);
          TRY(gb.add(gemm_desc(groups, 0, 3 * H, H, TB, dgh, 3 * H, s_gx, 1, hs, H, s_hs, 0, wh.C, H, wh.sC, wh.epi, wh.aux, sRi,
                               0, lr)));
        } else {
          const WgradTarget wh = wgrad_target(c->lidx[l].whh);
          TRY(gemm2(s, groups, bf, 3 * H, Hc, TB, dgh, 3 * H, s_gx, 1, hs, H, s_hs, 0, wh.C, Hc, wh.sC, wh.epi,
                    wh.aux, sRi, v_dghT, v_hsT, lr, persist_b, gp, gh));
        }
      }
      role = HPSGD_ROLE_GEMM_WGRAD;
      // Bias gradients from the recurrence's partial sums, with their update unless the gradients are accumulated as
      // well (a width off the 16-unit blocks leaves it to the commit launch, which takes all such ranges of the step
      // together): in the layer's adding launch or, where the layer has nothing else to add up, as column sums in the
      // launch of its weight gradients.
      bool bias_rides = false;
      if (dbp) {
        const size_t ob_ih = c->eoff(c->lidx[l].bih);
        const int n_dbp = use_solo ? gru_solo_row_tiles(B, H, c->K) : use_solo_b ? gru_solo_bf16_row_tiles(B, c->K) : (B + prow - 1) / prow;
        const bool update = !acc && (bf || H % 16 == 0);
        const float* b_in = update ? rin + ob_ih : nullptr;
        float* b_out = update ? rout + ob_ih : grad + ob_ih;
        const size_t s_bout = (size_t)(update ? sR : sG);
        if (update) fused_commit[c->lidx[l].bih] = fused_commit[c->lidx[l].bhh] = 1;
        bias_rides = !bf && rp.n == 0 && gb.pk.n > 0 &&
                     colsum_pack_push(gb.cs, dbp, 6L * Hc, (long)n_dbp * 6 * Hc, b_out, (long)s_bout, b_in, sRi, n_dbp, 6 * Hc);
        if (!bias_rides) TRY0(queue_reduce(dbp, n_dbp, (size_t)6 * Hc, b_in, (size_t)sRi, b_out, s_bout, update ? 1 : 0));
      }
      // The products and sums of both layers go out together, but for what a launch has no room for: an input gradient and two weight gradients, or
      // (where the input gradient is to be out before the update of what it reads, above) that one alone.  Those of
      // no room would each be a launch of their own, us per local step so / with the layer below in a launch of its own:
      // language models of 1000 words, 8 workers  H = 32, 64 rows, 4 steps 99.4 / 93.2,  48, 96, 10  191 / 187,  16, 96, 4  107 / 100.
      if (joined) {
        const int more = !lm ? 2 : width0 >= 4 && c->wgrad_parts(3 * H, width0, TB) > 1 ? 3 : 1;
        if (gb.pk.n + more > GemmPack::MAX) TRY(gb.flush());
        continue;
      }
      TRY(gb.flush());
      if (dbp) {
        // (above)
      } else {
        HIP_TRY(launch_colsum(dgx, 3 * H, s_gx, grad + c->eoff(c->lidx[l].bih), sG, TB, 3 * H, groups, s));
        HIP_TRY(launch_colsum(dgh, 3 * H, s_gx, grad + c->eoff(c->lidx[l].bhh), sG, TB, 3 * H, groups, s));
      }
      // the layer's sums of partial results (weight gradients of the resident-weight launch and
      // of the split contraction, bias gradients), with their updates: one launch
      HIP_TRY(launch_reduce_pack(rp, groups, s));
      if (dx_beside && hipStreamWaitEvent(s, c->ev_join, 0) != hipSuccess) return HPSGD_EHIP;
      role = HPSGD_ROLE_OTHER;
      d_zero = true;  // below the top layer nothing but `above` feeds a layer's gradient
    }
    if (lm && !embed_done) {
      role = HPSGD_ROLE_EMBED;
      TRY(embed_grad(s));
    }
  }
  // ---- commit (Alg. 2 "update replica")
  // the parameters not updated by a GEMM epilogue: all contiguous runs of them in one launch
  role = HPSGD_ROLE_COMMIT;
  c->last_commit_params = 0;
  CommitPack cpk;
  cpk.n_seg = 0;
  auto commit_pack = [&]() -> int {
    HIP_TRY(launch_commit_pack(cpk, rin, (size_t)sRi, rout, rstride, grad, (size_t)sG, lr, groups, s));
    cpk.n_seg = 0;
    return HPSGD_OK;
  };
  for (size_t e = 0; e < c->entries.size();) {
    if (fused_commit[e]) {
      ++e;
      continue;
    }
    const size_t lo = c->entries[e].offset;
    while (e < c->entries.size() && !fused_commit[e]) ++e;
    const size_t hi = e < c->entries.size() ? c->entries[e].offset : c->P;
    if (acc) {
      HIP_TRY(launch_commit_acc(rin + lo, (size_t)sRi, rout + lo, rstride, grad + lo, (size_t)sG, acc + lo, acc_stride, lr,
                                groups, hi - lo, s));
    } else if (!commit_pack_push(cpk, lo, hi - lo)) {
      TRY0(commit_pack());
      (void)commit_pack_push(cpk, lo, hi - lo);
    }
    c->last_commit_params += hi - lo;
  }
  TRY0(commit_pack());
  if (abort_word) HIP_TRY(launch_poison_on_abort(abort_word, loss_out, groups, rout, sR, groups, s));
  return HPSGD_OK;
}

// ---- the workspace of hpsgd_local_step_all_static: a fixed array in device memory, one copy per
// device (every device that loads the library holds it until the process ends).  In host code the
// array's name is only a handle for hipGetSymbolAddress; the address kernels and copies use is
// the one that call returns, looked up once per device with that device current.
static __device__ __align__(256) unsigned char g_static_workspace[HPSGD_STATIC_WORKSPACE_BYTES];
std::mutex g_static_mu;
void* g_static_workspace_ptr[kMaxDevices] = {nullptr};

int static_workspace(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return HPSGD_EHIP;
  std::lock_guard<std::mutex> lock(g_static_mu);
  if (!g_static_workspace_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_workspace)) != hipSuccess || !p) return HPSGD_EHIP;
    g_static_workspace_ptr[dev] = p;
  }
  *out = g_static_workspace_ptr[dev];
  return HPSGD_OK;
}

int check_step_args(const hpsgd_ctx* c, const float* rin, float* rout, size_t rstride, int groups,
                    const void* x, const int32_t* y, const void* ws) {
  if (!c || !rin || !rout || !x || !y) return HPSGD_EINVAL;
  if (!ws) return HPSGD_EWORKSPACE;
  if (((uintptr_t)ws & 255) != 0) return HPSGD_EWORKSPACE;
  if (!aligned16(rin) || !aligned16(rout) || ((uintptr_t)x & 3) != 0 || ((uintptr_t)y & 3) != 0)
    return HPSGD_EALIGN;
  if (groups > 1 && (rstride < c->P || (rstride & 3) != 0)) return HPSGD_EALIGN;
  const size_t span = ((size_t)(groups - 1) * rstride + c->P) * sizeof(float);
  if (rin != rout && overlaps(rin, span, rout, span)) return HPSGD_EALIAS;
  const size_t ws_bytes = c->ws_floats * sizeof(float);
  if (overlaps(ws, ws_bytes, rin, span) || overlaps(ws, ws_bytes, rout, span)) return HPSGD_EALIAS;
  return HPSGD_OK;
}

}  // namespace

namespace hpsgd {
static_assert((int)KID_COUNT == (int)HPSGD_KERNEL_COUNT, "kernel ids of kernels.h and hpsgd.h differ");

KernelTimer::KernelTimer(int kid, double work, hipStream_t s, int launches) : ctx_(nullptr), idx_(-1), s_(s) {
  hpsgd_ctx* c = t_step_ctx;
  if (!c || kid <= 0 || kid >= KID_COUNT || !(c->kernel_mask & (1u << kid))) return;
  hipEvent_t a = TimerScope::get(c), b = TimerScope::get(c);
  if (!a || !b) return;
  c->kstamps.push_back({kid, work, a, b, launches});
  ctx_ = c;
  idx_ = (int)c->kstamps.size() - 1;
  (void)hipEventRecord(a, s);
}
KernelTimer::~KernelTimer() {
  if (!ctx_) return;
  hpsgd_ctx* c = static_cast<hpsgd_ctx*>(ctx_);
  (void)hipEventRecord(c->kstamps[idx_].b, s_);
}
}  // namespace hpsgd

extern "C" {

int hpsgd_create(const hpsgd_model_desc* desc, int K, hpsgd_ctx** out) {
  if (!desc || !out) return HPSGD_EINVAL;
  *out = nullptr;
  if (K < 1 || K > HPSGD_MAX_WORKERS) return HPSGD_EINVAL;
  if (desc->prec != HPSGD_FP32 && desc->prec != HPSGD_BF16_MFMA) return HPSGD_EINVAL;
  hpsgd_ctx* c = new (std::nothrow) hpsgd_ctx();
  if (!c) return HPSGD_EINVAL;
  c->d = *desc;
  c->K = K;
  const int rc = build_layout(c);
  if (rc != HPSGD_OK) {
    delete c;
    return rc;
  }
  const size_t most = HPSGD_STATIC_WORKSPACE_BYTES / sizeof(float);
  for (int lean = 1; lean <= 3 && c->ws_floats > most && !c->small; ++lean) {
    std::unique_ptr<hpsgd_ctx> m(new (std::nothrow) hpsgd_ctx());
    if (!m) break;
    m->d = *desc;
    m->K = K;
    m->lean = lean;
    if (build_layout(m.get()) == HPSGD_OK && m->ws_floats <= most) c->small = std::move(m);
  }
  *out = c;
  return HPSGD_OK;
}

int hpsgd_destroy(hpsgd_ctx* ctx) {
  if (ctx) {
    for (auto& st : ctx->stamps) {
      (void)hipEventDestroy(st.a);
      (void)hipEventDestroy(st.b);
    }
    for (auto& st : ctx->kstamps) {
      (void)hipEventDestroy(st.a);
      (void)hipEventDestroy(st.b);
    }
    for (auto e : ctx->free_events) (void)hipEventDestroy(e);
    if (ctx->ev_fork) (void)hipEventDestroy(ctx->ev_fork);
    if (ctx->ev_join) (void)hipEventDestroy(ctx->ev_join);
  }
  delete ctx;
  return HPSGD_OK;
}

size_t hpsgd_param_count(const hpsgd_ctx* ctx) { return ctx ? ctx->P : 0; }
int hpsgd_param_entries(const hpsgd_ctx* ctx) { return ctx ? (int)ctx->entries.size() : 0; }

int hpsgd_param_entry(const hpsgd_ctx* ctx, int i, const char** name, size_t* offset, int* rows,
                      int* cols) {
  if (!ctx || i < 0 || i >= (int)ctx->entries.size()) return HPSGD_EINVAL;
  const Entry& e = ctx->entries[i];
  if (name) *name = e.name.c_str();
  if (offset) *offset = e.offset;
  if (rows) *rows = e.rows;
  if (cols) *cols = e.cols;
  return HPSGD_OK;
}

size_t hpsgd_workspace_bytes(const hpsgd_ctx* ctx) { return ctx ? ctx->ws_floats * sizeof(float) : 0; }

int hpsgd_local_step_all(hpsgd_ctx* ctx, const float* replicas_in, float* replicas_out,
                         size_t replica_stride, const void* x, const int32_t* y, float lr,
                         float* loss_out, void* workspace, void* hip_stream) {
  if (!ctx) return HPSGD_EINVAL;
  TRY0(check_step_args(ctx, replicas_in, replicas_out, replica_stride, ctx->K, x, y, workspace));
  return run_step(ctx, 0, ctx->K, replicas_in, replicas_out, replica_stride, x, y, lr, loss_out,
                  (float*)workspace, (hipStream_t)hip_stream);
}

int hpsgd_local_step_all_cloned(hpsgd_ctx* ctx, const float* source, float* replicas_out, size_t replica_stride,
                                const void* x, const int32_t* y, float lr, float* loss_out, void* workspace,
                                void* hip_stream) {
  if (!ctx) return HPSGD_EINVAL;
  // the output replicas alone are checked like those of a step in place, the source like a model
  TRY0(check_step_args(ctx, replicas_out, replicas_out, replica_stride, ctx->K, x, y, workspace));
  if (!source) return HPSGD_EINVAL;
  if (!aligned16(source)) return HPSGD_EALIGN;
  const size_t span = ((size_t)(ctx->K - 1) * replica_stride + ctx->P) * sizeof(float);
  const size_t pbytes = ctx->P * sizeof(float);
  if (overlaps(source, pbytes, replicas_out, span) ||
      overlaps(source, pbytes, workspace, ctx->ws_floats * sizeof(float)))
    return HPSGD_EALIAS;
  return run_step(ctx, 0, ctx->K, source, replicas_out, replica_stride, x, y, lr, loss_out, (float*)workspace,
                  (hipStream_t)hip_stream, nullptr, 0, true);
}

int hpsgd_local_step_all_static(hpsgd_ctx* ctx, const float* replicas_in, float* replicas_out,
                                size_t replica_stride, const void* x, const int32_t* y, float lr,
                                float* loss_out, void* hip_stream) {
  if (!ctx) return HPSGD_EINVAL;
  // the size check comes first and needs no device
  hpsgd_ctx* run = ctx->ws_floats * sizeof(float) <= (size_t)HPSGD_STATIC_WORKSPACE_BYTES ? ctx : ctx->small.get();
  if (!run) return HPSGD_EWORKSPACE;
  if (!replicas_in || !replicas_out || !x || !y) return HPSGD_EINVAL;
  void* ws = nullptr;
  TRY0(static_workspace(&ws));
  TRY0(check_step_args(run, replicas_in, replicas_out, replica_stride, ctx->K, x, y, ws));
  if (run != ctx) ctx->lend(*run);
  const int rc = run_step(run, 0, ctx->K, replicas_in, replicas_out, replica_stride, x, y, lr, loss_out, (float*)ws,
                          (hipStream_t)hip_stream);
  if (run != ctx) ctx->take_back(*run);
  return rc;
}

int hpsgd_prepare_replicas(hpsgd_ctx* ctx, const float* replicas, size_t replica_stride, void* workspace,
                           void* hip_stream) {
  if (!ctx || !replicas) return HPSGD_EINVAL;
  if (!workspace || ((uintptr_t)workspace & 255) != 0) return HPSGD_EWORKSPACE;
  if (!aligned16(replicas) || (ctx->K > 1 && (replica_stride < ctx->P || (replica_stride & 3) != 0)))
    return HPSGD_EALIGN;
  const size_t span = ((size_t)(ctx->K - 1) * replica_stride + ctx->P) * sizeof(float);
  if (overlaps(workspace, ctx->ws_floats * sizeof(float), replicas, span)) return HPSGD_EALIAS;
  ctx->drop_mark((const float*)workspace);
  if (ctx->d.prec != HPSGD_BF16_MFMA || ctx->d.kind == HPSGD_MLP) return HPSGD_OK;  // nothing to prepare
  WeightCopies wc;
  const int rc = weight_copies(ctx, replicas, (long)replica_stride, 0, ctx->K, (float*)workspace,
                               (hipStream_t)hip_stream, true, true, wc);
  if (rc != HPSGD_OK) return rc;
  ctx->set_mark(hpsgd_ctx::Mark{replicas, (const float*)workspace, replica_stride, nullptr, false});
  return HPSGD_OK;
}

int hpsgd_prepare_clones(hpsgd_ctx* ctx, const float* global, const float* replicas, size_t replica_stride,
                         void* workspace, int with_head, void* hip_stream) {
  if (!ctx || !global || !replicas) return HPSGD_EINVAL;
  if (!workspace || ((uintptr_t)workspace & 255) != 0) return HPSGD_EWORKSPACE;
  if (!aligned16(global) || !aligned16(replicas) ||
      (ctx->K > 1 && (replica_stride < ctx->P || (replica_stride & 3) != 0)))
    return HPSGD_EALIGN;
  const size_t span = ((size_t)(ctx->K - 1) * replica_stride + ctx->P) * sizeof(float);
  const size_t ws_bytes = ctx->ws_floats * sizeof(float);
  if (overlaps(workspace, ws_bytes, replicas, span) || overlaps(workspace, ws_bytes, global, ctx->P * sizeof(float)))
    return HPSGD_EALIAS;
  ctx->drop_mark((const float*)workspace);
  if (ctx->d.prec != HPSGD_BF16_MFMA || ctx->d.kind == HPSGD_MLP) return HPSGD_OK;  // nothing to prepare
  WeightCopies wc;
  // one set of copies, in worker 0's slice, which the step hands to every worker (the replicas are
  // clones: their copies would be the same bits).  The GRU layers' always; the head's when asked
  // for, else they are left to the step, which makes them from `global` right before the logits
  // GEMM (a training stream that makes them here, at a round's start, would share the memory
  // system with whatever the synchronising side is doing then)
  // (the step decides from the replicas' addresses which copies it has; made from another address
  // the set must come out the same, else the step makes its own)
  const bool head = with_head != 0;
  WeightCopies want;
  int rc = weight_copies(ctx, replicas, (long)replica_stride, 0, ctx->K, (float*)workspace, nullptr, false, head, want);
  if (rc == HPSGD_OK) rc = weight_copies(ctx, global, 0, 0, 1, (float*)workspace, nullptr, false, head, wc);
  if (rc != HPSGD_OK) return rc;
  if (std::memcmp(&want, &wc, sizeof(WeightCopies)) != 0) return HPSGD_OK;
  rc = weight_copies(ctx, global, 0, 0, 1, (float*)workspace, (hipStream_t)hip_stream, true, head, wc);
  if (rc != HPSGD_OK) return rc;
  ctx->set_mark(hpsgd_ctx::Mark{replicas, (const float*)workspace, replica_stride, global, head && wc.head});
  return HPSGD_OK;
}

int hpsgd_local_step_all_acc(hpsgd_ctx* ctx, const float* replicas_in, float* replicas_out,
                             size_t replica_stride, const void* x, const int32_t* y, float lr,
                             float* loss_out, float* grad_acc, size_t acc_stride, void* workspace,
                             void* hip_stream) {
  if (!ctx) return HPSGD_EINVAL;
  TRY0(check_step_args(ctx, replicas_in, replicas_out, replica_stride, ctx->K, x, y, workspace));
  if (!grad_acc) return HPSGD_EINVAL;
  if (((uintptr_t)grad_acc & 15) != 0 || (ctx->K > 1 && (acc_stride < ctx->P || (acc_stride & 3) != 0)))
    return HPSGD_EALIGN;
  const size_t span = ((size_t)(ctx->K - 1) * acc_stride + ctx->P) * sizeof(float);
  const size_t rspan = ((size_t)(ctx->K - 1) * replica_stride + ctx->P) * sizeof(float);
  if (overlaps(grad_acc, span, replicas_in, rspan) || overlaps(grad_acc, span, replicas_out, rspan))
    return HPSGD_EALIAS;
  return run_step(ctx, 0, ctx->K, replicas_in, replicas_out, replica_stride, x, y, lr, loss_out,
                  (float*)workspace, (hipStream_t)hip_stream, grad_acc, acc_stride);
}

int hpsgd_local_step(hpsgd_ctx* ctx, int worker, const float* replica_in, float* replica_out,
                     const void* x, const int32_t* y, float lr, float* loss_out, void* workspace,
                     void* hip_stream) {
  if (!ctx || worker < 0 || worker >= ctx->K) return HPSGD_EINVAL;
  TRY0(check_step_args(ctx, replica_in, replica_out, ctx->P, 1, x, y, workspace));
  return run_step(ctx, worker, 1, replica_in, replica_out, round_up(ctx->P, 4), x, y, lr, loss_out,
                  (float*)workspace, (hipStream_t)hip_stream);
}

int hpsgd_gather_batch(const void* shard, const int32_t* idx, int n_idx, size_t row_bytes,
                       int n_chunks, size_t chunk_bytes, void* out, void* hip_stream) {
  if (n_idx < 0 || n_chunks < 0) return HPSGD_EINVAL;
  if (n_idx == 0 || n_chunks == 0 || chunk_bytes == 0) return HPSGD_OK;
  if (!shard || !idx || !out) return HPSGD_EINVAL;
  if ((row_bytes & 3) || (chunk_bytes & 3) || ((uintptr_t)shard & 3) || ((uintptr_t)out & 3) ||
      ((uintptr_t)idx & 3))
    return HPSGD_EALIGN;
  if ((size_t)n_chunks * chunk_bytes > row_bytes || n_chunks > 65535) return HPSGD_ESHAPE;
  return launch_gather(shard, idx, n_idx, row_bytes, n_chunks, chunk_bytes, out,
                       (hipStream_t)hip_stream) == hipSuccess ? HPSGD_OK : HPSGD_EHIP;
}

namespace {
int check_gather(const void* const* shards, const int32_t* const* idx, int K, size_t row_bytes, int n_chunks, size_t chunk_bytes,
                 void* const* outs) {
  if (!shards || !idx || !outs) return HPSGD_EINVAL;
  if ((row_bytes & 3) || (chunk_bytes & 3)) return HPSGD_EALIGN;
  if ((size_t)n_chunks * chunk_bytes > row_bytes || n_chunks > 65535) return HPSGD_ESHAPE;
  for (int k = 0; k < K; ++k) {
    if (!shards[k] || !idx[k] || !outs[k]) return HPSGD_EINVAL;
    if (((uintptr_t)shards[k] & 3) || ((uintptr_t)outs[k] & 3) || ((uintptr_t)idx[k] & 3)) return HPSGD_EALIGN;
  }
  return HPSGD_OK;
}
}  // namespace

int hpsgd_gather_batch_all(const void* const* shards, const int32_t* const* idx, int K, int n_idx,
                           size_t row_bytes, int n_chunks, size_t chunk_bytes, void* const* outs,
                           void* hip_stream) {
  if (K < 0 || K > HPSGD_MAX_WORKERS || n_idx < 0 || n_chunks < 0) return HPSGD_EINVAL;
  if (K == 0 || n_idx == 0 || n_chunks == 0 || chunk_bytes == 0) return HPSGD_OK;
  const int rc = check_gather(shards, idx, K, row_bytes, n_chunks, chunk_bytes, outs);
  if (rc != HPSGD_OK) return rc;
  return launch_gather_all(shards, idx, K, n_idx, row_bytes, n_chunks, chunk_bytes, outs,
                           (hipStream_t)hip_stream) == hipSuccess ? HPSGD_OK : HPSGD_EHIP;
}

int hpsgd_gather_batches(const hpsgd_gather_part* parts, int n_parts, const int32_t* const* idx, int K, int n_idx,
                         void* hip_stream) {
  if (K < 0 || K > HPSGD_MAX_WORKERS || n_idx < 0 || !parts || n_parts < 1 || n_parts > HPSGD_MAX_GATHER_PARTS) return HPSGD_EINVAL;
  GatherPart q[HPSGD_MAX_GATHER_PARTS];
  bool small = true;
  int n = 0;
  for (int p = 0; p < n_parts; ++p) {
    if (parts[p].n_chunks < 0) return HPSGD_EINVAL;
    if (K == 0 || n_idx == 0 || parts[p].n_chunks == 0 || parts[p].chunk_bytes == 0) continue;
    const int rc = check_gather(parts[p].shards, idx, K, parts[p].row_bytes, parts[p].n_chunks, parts[p].chunk_bytes, parts[p].outs);
    if (rc != HPSGD_OK) return rc;
    q[n++] = GatherPart{parts[p].shards, parts[p].outs, parts[p].row_bytes, parts[p].chunk_bytes, parts[p].n_chunks};
    small = small && (size_t)parts[p].n_chunks * n_idx * (parts[p].chunk_bytes / 4) < (size_t)1 << 31;
  }
  if (n == 0) return HPSGD_OK;
  if (small) return launch_gather_parts(q, n, idx, K, n_idx, (hipStream_t)hip_stream) == hipSuccess ? HPSGD_OK : HPSGD_EHIP;
  for (int p = 0; p < n; ++p)
    if (launch_gather_all(q[p].shards, idx, K, n_idx, q[p].row_bytes, q[p].n_chunks, q[p].chunk_bytes, q[p].outs,
                          (hipStream_t)hip_stream) != hipSuccess)
      return HPSGD_EHIP;
  return HPSGD_OK;
}

int hpsgd_merge(float* global, const float* const* replicas, const float* snapshot, int K, size_t P,
                void* hip_stream) {
  if (K < 1 || K > HPSGD_MAX_WORKERS) return HPSGD_EINVAL;
  if (P == 0) return HPSGD_OK;
  if (!global || !replicas || !snapshot) return HPSGD_EINVAL;
  if (!aligned16(global) || !aligned16(snapshot)) return HPSGD_EALIGN;
  PtrPack pk;
  for (int k = 0; k < K; ++k) {
    if (!replicas[k]) return HPSGD_EINVAL;
    if (!aligned16(replicas[k])) return HPSGD_EALIGN;
    if (overlaps(global, P * sizeof(float), replicas[k], P * sizeof(float))) return HPSGD_EALIAS;
    pk.p[k] = const_cast<float*>(replicas[k]);
  }
  if (snapshot != global && overlaps(global, P * sizeof(float), snapshot, P * sizeof(float)))
    return HPSGD_EALIAS;
  return launch_merge(global, pk, snapshot, K, P, (hipStream_t)hip_stream) == hipSuccess ? HPSGD_OK
                                                                                          : HPSGD_EHIP;
}

int hpsgd_merge_sync(float* global, float* const* replicas, float* snapshot, int K, size_t P, void* hip_stream) {
  if (K < 1 || K > HPSGD_MAX_WORKERS) return HPSGD_EINVAL;
  if (P == 0) return HPSGD_OK;
  if (!global || !replicas || !snapshot) return HPSGD_EINVAL;
  if (!aligned16(global) || !aligned16(snapshot)) return HPSGD_EALIGN;
  const size_t bytes = P * sizeof(float);
  PtrPack pk;
  for (int k = 0; k < K; ++k) {
    if (!replicas[k]) return HPSGD_EINVAL;
    if (!aligned16(replicas[k])) return HPSGD_EALIGN;
    // every buffer is written here: no two may overlap
    if (overlaps(global, bytes, replicas[k], bytes) || overlaps(snapshot, bytes, replicas[k], bytes)) return HPSGD_EALIAS;
    for (int j = 0; j < k; ++j)
      if (overlaps(replicas[j], bytes, replicas[k], bytes)) return HPSGD_EALIAS;
    pk.p[k] = replicas[k];
  }
  if (overlaps(global, bytes, snapshot, bytes)) return HPSGD_EALIAS;
  return launch_merge_sync(global, pk, snapshot, K, P, (hipStream_t)hip_stream) == hipSuccess ? HPSGD_OK : HPSGD_EHIP;
}

int hpsgd_merge_snapshot(float* global, const float* const* replicas, float* snapshot, int K, size_t P,
                         void* hip_stream) {
  if (K < 1 || K > HPSGD_MAX_WORKERS) return HPSGD_EINVAL;
  if (P == 0) return HPSGD_OK;
  if (!global || !replicas || !snapshot) return HPSGD_EINVAL;
  if (!aligned16(global) || !aligned16(snapshot)) return HPSGD_EALIGN;
  const size_t bytes = P * sizeof(float);
  PtrPack pk;
  for (int k = 0; k < K; ++k) {
    if (!replicas[k]) return HPSGD_EINVAL;
    if (!aligned16(replicas[k])) return HPSGD_EALIGN;
    // the replicas are read while the two models are written
    if (overlaps(global, bytes, replicas[k], bytes) || overlaps(snapshot, bytes, replicas[k], bytes)) return HPSGD_EALIAS;
    pk.p[k] = const_cast<float*>(replicas[k]);
  }
  if (overlaps(global, bytes, snapshot, bytes)) return HPSGD_EALIAS;
  return launch_merge_sync(global, pk, snapshot, K, P, (hipStream_t)hip_stream, false) == hipSuccess ? HPSGD_OK
                                                                                                      : HPSGD_EHIP;
}

int hpsgd_merge_grad(float* global, const float* const* grad_accs, float lr, int K, size_t P,
                     void* hip_stream) {
  if (K < 1 || K > HPSGD_MAX_WORKERS) return HPSGD_EINVAL;
  if (P == 0) return HPSGD_OK;
  if (!global || !grad_accs) return HPSGD_EINVAL;
  if (!aligned16(global)) return HPSGD_EALIGN;
  PtrPack pk;
  for (int k = 0; k < K; ++k) {
    if (!grad_accs[k]) return HPSGD_EINVAL;
    if (!aligned16(grad_accs[k])) return HPSGD_EALIGN;
    if (overlaps(global, P * sizeof(float), grad_accs[k], P * sizeof(float))) return HPSGD_EALIAS;
    pk.p[k] = const_cast<float*>(grad_accs[k]);
  }
  return launch_merge_grad(global, pk, lr, K, P, (hipStream_t)hip_stream) == hipSuccess ? HPSGD_OK
                                                                                        : HPSGD_EHIP;
}

int hpsgd_sync_all(const float* global, float* const* replicas, int K, float* snapshot, size_t P,
                   void* hip_stream) {
  if (K < 0 || K > HPSGD_MAX_WORKERS) return HPSGD_EINVAL;
  if (P == 0) return HPSGD_OK;
  if (!global || (K > 0 && !replicas)) return HPSGD_EINVAL;
  if (!aligned16(global) || (snapshot && !aligned16(snapshot))) return HPSGD_EALIGN;
  PtrPack pk;
  for (int k = 0; k < K; ++k) {
    if (!replicas[k]) return HPSGD_EINVAL;
    if (!aligned16(replicas[k])) return HPSGD_EALIGN;
    if (overlaps(global, P * sizeof(float), replicas[k], P * sizeof(float))) return HPSGD_EALIAS;
    pk.p[k] = replicas[k];
  }
  if (snapshot && overlaps(global, P * sizeof(float), snapshot, P * sizeof(float))) return HPSGD_EALIAS;
  if (K == 0 && !snapshot) return HPSGD_OK;
  return launch_sync_all(global, pk, K, snapshot, P, (hipStream_t)hip_stream) == hipSuccess
             ? HPSGD_OK
             : HPSGD_EHIP;
}

int hpsgd_sync_replica(const float* global, float* replica, size_t P, void* hip_stream) {
  float* one[1] = {replica};
  if (!replica) return P == 0 ? HPSGD_OK : HPSGD_EINVAL;
  return hpsgd_sync_all(global, one, 1, nullptr, P, hip_stream);
}

int hpsgd_set_aux_stream(hpsgd_ctx* ctx, void* hip_stream) {
  if (!ctx) return HPSGD_EINVAL;
  if (hip_stream && !ctx->ev_fork) {
    if (hipEventCreateWithFlags(&ctx->ev_fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ctx->ev_join, hipEventDisableTiming) != hipSuccess)
      return HPSGD_EHIP;
  }
  ctx->aux = (hipStream_t)hip_stream;
  return HPSGD_OK;
}

int hpsgd_set_recurrence(hpsgd_ctx* ctx, int resident, unsigned spin_limit) {
  if (!ctx) return HPSGD_EINVAL;
  if (ctx->resident != (resident != 0)) ctx->marks.clear();  // (the operand copies of the two forms differ in layout)
  ctx->resident = resident != 0;
  ctx->device_scope = resident == 2;
  ctx->spin_limit = spin_limit;
  return HPSGD_OK;
}

int hpsgd_recurrence_gave_up(const hpsgd_ctx* ctx, const void* workspace, void* hip_stream, int* gave_up) {
  if (!ctx || !gave_up) return HPSGD_EINVAL;
  if (!workspace) return HPSGD_EWORKSPACE;
  *gave_up = 0;
  if (ctx->psync.stride == 0) return HPSGD_OK;  // no such kernels for this model
  // the abort word is the first word of a worker's slice (of the first worker's for a grouped step)
  std::vector<unsigned> host(ctx->psync.stride * (size_t)ctx->K);
  hipStream_t s = (hipStream_t)hip_stream;
  if (hipMemcpyAsync(host.data(), (const float*)workspace + ctx->psync.offset, host.size() * sizeof(unsigned),
                     hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return HPSGD_EHIP;
  for (int k = 0; k < ctx->K; ++k)
    if (host[(size_t)k * ctx->psync.stride] == 1u) *gave_up = 1;
  return HPSGD_OK;
}

int hpsgd_timer_enable(hpsgd_ctx* ctx, unsigned role_mask) {
  if (!ctx) return HPSGD_EINVAL;
  ctx->timer_mask = role_mask & ((1u << HPSGD_ROLE_COUNT) - 1u);
  return HPSGD_OK;
}

int hpsgd_timer_read(hpsgd_ctx* ctx, int role, long* launches, double* total_ms) {
  if (!ctx || role < 0 || role >= HPSGD_ROLE_COUNT) return HPSGD_EINVAL;
  // fold every recorded pair into the per-role totals, then hand back and clear this role's
  for (auto& st : ctx->stamps) {
    if (hipEventSynchronize(st.b) != hipSuccess) return HPSGD_EHIP;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, st.a, st.b) != hipSuccess) return HPSGD_EHIP;
    ctx->role_ms[st.role] += ms;
    ctx->role_launches[st.role] += st.launches;
    ctx->free_events.push_back(st.a);
    ctx->free_events.push_back(st.b);
  }
  ctx->stamps.clear();
  if (launches) *launches = ctx->role_launches[role];
  if (total_ms) *total_ms = ctx->role_ms[role];
  ctx->role_launches[role] = 0;
  ctx->role_ms[role] = 0.0;
  return HPSGD_OK;
}

int hpsgd_kernel_timer_enable(hpsgd_ctx* ctx, unsigned kernel_mask) {
  if (!ctx) return HPSGD_EINVAL;
  ctx->kernel_mask = kernel_mask & ((1u << HPSGD_KERNEL_COUNT) - 1u) & ~1u;
  return HPSGD_OK;
}

int hpsgd_kernel_timer_read(hpsgd_ctx* ctx, int kernel, long* launches, double* total_ms, double* work) {
  if (!ctx || kernel <= 0 || kernel >= HPSGD_KERNEL_COUNT) return HPSGD_EINVAL;
  for (auto& st : ctx->kstamps) {
    if (hipEventSynchronize(st.b) != hipSuccess) return HPSGD_EHIP;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, st.a, st.b) != hipSuccess) return HPSGD_EHIP;
    ctx->kernel_ms[st.kid] += ms;
    ctx->kernel_work[st.kid] += st.work;
    ctx->kernel_launches[st.kid] += st.launches;
    ctx->free_events.push_back(st.a);
    ctx->free_events.push_back(st.b);
  }
  ctx->kstamps.clear();
  if (launches) *launches = ctx->kernel_launches[kernel];
  if (total_ms) *total_ms = ctx->kernel_ms[kernel];
  if (work) *work = ctx->kernel_work[kernel];
  ctx->kernel_launches[kernel] = 0;
  ctx->kernel_ms[kernel] = 0.0;
  ctx->kernel_work[kernel] = 0.0;
  return HPSGD_OK;
}

const char* hpsgd_kernel_name(int kernel) {
  switch (kernel) {
    case HPSGD_KERNEL_GRU_FWD_PERSIST: return "gru_fwd_persist_kernel";
    case HPSGD_KERNEL_GRU_BWD_PERSIST: return "gru_bwd_persist_kernel";
    case HPSGD_KERNEL_GRU_FWD_PERSIST_BF16: return "gru_fwd_persist_bf16_kernel";
    case HPSGD_KERNEL_GRU_BWD_PERSIST_BF16: return "gru_bwd_persist_bf16_kernel";
    case HPSGD_KERNEL_GEMM_BF16_DL: return "gemm_bf16_dl_kernel<false>";
    case HPSGD_KERNEL_GEMM_BF16_DL_COMMIT: return "gemm_bf16_dl_kernel<true>";
    case HPSGD_KERNEL_GEMM_BF16_DLX128: return "gemm_bf16_dlx_kernel<false, 2, 4, 2, 2, 3>";
    case HPSGD_KERNEL_GEMM_BF16_DLX128_COMMIT: return "gemm_bf16_dlx_kernel<true, 2, 4, 2, 2, 3>";
    case HPSGD_KERNEL_GEMM_BF16_DLX192: return "gemm_bf16_dlx_kernel<false, 2, 4, 3, 2, 2>";
    case HPSGD_KERNEL_GEMM_BF16_DLX192_COMMIT: return "gemm_bf16_dlx_kernel<true, 2, 4, 3, 2, 2>";
    case HPSGD_KERNEL_GEMM_BF16_DLX256: return "gemm_bf16_dlx_kernel<false, 2, 4, 4, 2, 2>";
    case HPSGD_KERNEL_GEMM_BF16_DLX256_COMMIT: return "gemm_bf16_dlx_kernel<true, 2, 4, 4, 2, 2>";
    case HPSGD_KERNEL_GEMM_BF16_NT: return "gemm_bf16_nt_kernel";
    case HPSGD_KERNEL_GEMM_F32_FAST: return "gemm_f32_fast_kernel";
    case HPSGD_KERNEL_GEMM_F32: return "gemm_f32_kernel";
    case HPSGD_KERNEL_CVT2: return "cvt2_kernel";
    case HPSGD_KERNEL_SOFTMAX_CE_BF16: return "softmax_ce_bf16_rows_kernel";
    case HPSGD_KERNEL_GRU_STEP: return "gru_step_kernel";
    case HPSGD_KERNEL_COMMIT_ACC: return "commit_acc4_kernel";
    case HPSGD_KERNEL_COMMIT: return "commit_kernel";
    case HPSGD_KERNEL_CVT2_PACK: return "cvt2_pack_kernel";
    default: return nullptr;
  }
}

int hpsgd_delay_us(unsigned microseconds, void* hip_stream) {
  if (microseconds > 1000000u) return HPSGD_EINVAL;
  return launch_delay(microseconds, (hipStream_t)hip_stream) == hipSuccess ? HPSGD_OK : HPSGD_EHIP;
}

size_t hpsgd_commit_kernel_params(const hpsgd_ctx* ctx) { return ctx ? ctx->last_commit_params : 0; }

int hpsgd_recurrence_info(const hpsgd_ctx* ctx, int* resident_layers, int* xproj_layers, int* dw_layers) {
  if (!ctx) return HPSGD_EINVAL;
  if (resident_layers) *resident_layers = ctx->last_resident;
  if (xproj_layers) *xproj_layers = ctx->last_xproj;
  if (dw_layers) *dw_layers = ctx->last_dw;
  return HPSGD_OK;
}

int hpsgd_gemm_bf16_nt(const void* A, long lda, long strideA, const void* B, long ldb, long strideB, float* C,
                       long ldc, long strideC, const float* win, long strideWin, float lr, int M, int N, int Kd,
                       int groups, int form, void* hip_stream) {
  if (!A || !B || !C || M < 1 || N < 1 || Kd < 8 || Kd % 8 != 0 || groups < 1 || form < 0 || form > 4)
    return HPSGD_EINVAL;
  if (lda < Kd || ldb < Kd || ldc < N) return HPSGD_EINVAL;
  if (!gemm_bf16_nt_supported(A, 1, lda, strideA, Kd) || !gemm_bf16_nt_supported(B, 1, ldb, strideB, Kd))
    return HPSGD_EALIGN;
  return launch_gemm_bf16_nt(A, 1, lda, strideA, B, 1, ldb, strideB, C, ldc, strideC, nullptr, 0, win, strideWin, lr,
                             M, N, Kd, groups, (hipStream_t)hip_stream, form) == hipSuccess
             ? HPSGD_OK
             : HPSGD_EHIP;
}

int hpsgd_probe_mfma_rate(int precision, const void* operands, int iterations, double* result, float* sink,
                          void* hip_stream) {
  if (!operands || !result || !sink || iterations < 1) return HPSGD_EINVAL;
  if (precision != HPSGD_FP32 && precision != HPSGD_BF16_MFMA) return HPSGD_EINVAL;
  if (((uintptr_t)operands & 15) != 0) return HPSGD_EALIGN;
  return launch_mfma_probe(precision == HPSGD_BF16_MFMA, operands, iterations, result, sink,
                           (hipStream_t)hip_stream) == hipSuccess
             ? HPSGD_OK
             : HPSGD_EHIP;
}

const char* hpsgd_role_name(int role) {
  switch (role) {
    case HPSGD_ROLE_OTHER: return "other";
    case HPSGD_ROLE_GEMM_INPUT: return "gemm_input_projection";
    case HPSGD_ROLE_GEMM_REC_FWD: return "gemm_recurrent_fwd";
    case HPSGD_ROLE_GEMM_REC_BWD: return "gemm_recurrent_bwd";
    case HPSGD_ROLE_GEMM_WGRAD: return "gemm_weight_grad";
    case HPSGD_ROLE_GEMM_DX: return "gemm_input_grad";
    case HPSGD_ROLE_GEMM_HEAD: return "gemm_head";
    case HPSGD_ROLE_CELL_FWD: return "gru_cell_fwd";
    case HPSGD_ROLE_CELL_BWD: return "gru_cell_bwd";
    case HPSGD_ROLE_LOSS: return "softmax_ce";
    case HPSGD_ROLE_EMBED: return "embedding";
    case HPSGD_ROLE_COMMIT: return "commit";
    case HPSGD_ROLE_MLP_FWD: return "mlp_fwd";
    case HPSGD_ROLE_MLP_BWD: return "mlp_bwd";
    default: return nullptr;
  }
}

const char* hpsgd_strerror(int status) {
  switch (status) {
    case HPSGD_OK: return "ok";
    case HPSGD_EINVAL: return "invalid argument";
    case HPSGD_ESHAPE: return "unsupported or inconsistent shape";
    case HPSGD_EALIGN: return "pointer or stride not aligned";
    case HPSGD_EALIAS: return "buffers overlap";
    case HPSGD_EWORKSPACE: return "workspace null or misaligned";
    case HPSGD_EUNSUPPORTED: return "not supported";
    case HPSGD_EHIP: return "HIP call failed";
    default: return "unknown status";
  }
}

}  // extern "C"
