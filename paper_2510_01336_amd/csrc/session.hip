// Session state machine and C ABI of the draft / verify / rollback calls (Algorithm 2 of the paper
// with the KV-cache and hidden-state reuse of its Sec. 3.2).  Host code only decides shapes and
// keeps the integer bookkeeping; every arithmetic step runs in the kernels of kernels_*.hip.
#include "kernels.h"
#include <algorithm>
#include <cstring>
#include <mutex>

// With further verifier exits (n levels > 2) C also holds the tokens that wait for the levels above L_i,
// deepest verdict first: C = committed || V[n-1] || ... || V[2], where V[j] are the tokens accepted at exit j that
// exit j+1 has not seen; cut[j] = |committed || V[n-1] || ... || V[j]|, so cut[n] tokens are committed and
// cut[2] == |C| always.  V stays the buffer of L_i (level 1).  With the paper's three exits cut[2] = |C| is all there is.
struct SeqState {
  std::vector<int> C, V, S;   // (see above), tentative at L_i, pending draft block
  int cut[EE_MAX_GROUPS] = {0, 0, 0, 0, 0, 0, 0};
  int len[EE_MAX_GROUPS] = {0, 0, 0, 0, 0, 0, 0};     // KV length per layer group
  int n_hd = 0;               // buffered L_d hidden rows (pending draft block incl. bonus row)
  int n_pi = 0;               // rejection sampling: tokens of V whose L_i distribution is stored
  int n_pu[4] = {0, 0, 0, 0}; // ... and tokens of the buffers at the further verifier exits (levels 2..n-1) whose distribution is stored
  bool sampled = false;       // the pending draft block was drawn from p_{L_d} (its distributions are stored)
  std::vector<int> pages;     // block table
  bool started = false;
};

struct MetaSlot {             // one upload region: host (pinned) + device copy, same layout
  int* h = nullptr;
  int* d = nullptr;
  hipEvent_t copied = nullptr;
  bool in_flight = false;
};

struct KTimer { int fam; hipEvent_t a, b; };

struct ee_session {
  ee_model* m = nullptr;
  hipStream_t st = nullptr;
  int B = 0, max_ctx = 0, max_rows = 0, pps = 0, n_pages = 0, chunk = 0;
  int maxM = 0, Mp = 0, maxQT = 0;            // most rows of a pass (a context-build pass or a batch-wide call), padded to whole GEMM passes, most q-tiles
  int headM = 0, headMp = 0;                  // the same for an exit head (a context build sends it the rows that end a prompt)
  int ssq_stride = 0, inv_cap = 0;            // row stride of ssq, floats in inv_rms
  int ssq_parts = 0;                          // partial sums of squares per row that the last down projection left
  char* base = nullptr;
  size_t bytes = 0;
  // device buffers (inside the caller's arena)
  void* kv = nullptr;
  float *X = nullptr, *LOGITS = nullptr, *Hd = nullptr, *Hi = nullptr;
  float* Hup[4] = {nullptr, nullptr, nullptr, nullptr};   // hidden rows buffered at the further verifier exits (levels 2..n-1)
  int n_levels = 2;             // verifier levels: exits after L_d (2 = Alg. 2: L_i and L_f)
  void *XN = nullptr, *Qb = nullptr, *AO = nullptr, *H = nullptr;
  float2* cs = nullptr;
  int4* rowinfo = nullptr;    // [maxM] per-row lookups of the QKV epilogue, resolved once per call
  int *vtok = nullptr, *tok_next = nullptr, *out_dev = nullptr, *page_scratch = nullptr;
  // rejection-sampling acceptance (attached separately): the distributions the draft tokens were drawn from,
  // the L_i distributions of the tokens in V (rows [batch][max_rows][vocab])
  float *Pd = nullptr, *Pi = nullptr;
  float* Pup[4] = {nullptr, nullptr, nullptr, nullptr};   // the same for the buffers of levels 2..n-1
  bool need_logits = false;
  float *part_o = nullptr, *part_ml = nullptr, *pmax = nullptr, *ssq = nullptr, *gemm_part = nullptr, *inv_rms = nullptr;
  // auxiliary exit heads: adapter output rows z [maxM][d], its rank-r intermediate (T: fp32 models, the rows; TF: bf16
  // models, the operand of the up projection), that operand's unused sum-of-squares partials, unit gains
  float *Z = nullptr, *T = nullptr, *ssq_t = nullptr, *ones = nullptr;
  void* TF = nullptr;
  size_t part_units = 0;        // capacity of the attention split scratch in (q-tile, split) units per KV head
  int* pidx = nullptr;
  int max_splits = 64;
  // host side
  MetaSlot slot[2];
  size_t meta_ints = 0, meta_cap = 0;   // metadata of the call being built, and of the largest one
  int* out_host = nullptr;    // pinned, written by the kernels that decide them: n_accept[B], next[B], draft [B*max_rows]
  std::vector<SeqState> seq;
  std::vector<int> free_pages;
  bool debug_logits = false, time_kernels = false;
  int last_rows = 0, last_row0 = 0;   // rows of X behind the last exit head
  int last_attn = -1;                 // attention kernel of the last pass (ATTN_*; fp32: -1)
  std::vector<KTimer> timers;
  int launches[KF_COUNT] = {0};
  // meta layout (offsets in ints)
  size_t o_row_seq, o_row_pos, o_row_tok, o_row_src, o_row_dst, o_seq_row0, o_seq_m, o_seq_p0, o_seq_qt0, o_qt_seq,
      o_qt_local, o_cand, o_n_cand, o_bt, o_u;
  int cand_stride = 0;
};

static const char* kFamName[KF_COUNT] = {"embed", "rmsnorm", "gemm_qkv", "rope_append", "attention", "attn_combine", "gemm_o",
                                         "gemm_gate_up", "gemm_down", "gemm_head", "argmax", "accept", "copy_rows", "misc"};

// ---------------------------------------------------------------------------------------------
// arena carving
// ---------------------------------------------------------------------------------------------
struct Carver {
  char* base; size_t cur = 0;
  template <class T> T* take(size_t n) {
    cur = align_up(cur, 256);
    T* p = base ? (T*)(base + cur) : nullptr;
    cur += n * sizeof(T);
    return p;
  }
};

// offsets of the metadata block of a call with so many rows and q-tiles (a call uploads no more than it uses)
static void layout_meta(ee_session* s, int rows, int qts, int uniforms) {
  size_t o = 0;
  auto take = [&](size_t n) { size_t r = o; o += (n + 3) / 4 * 4; return r; };
  s->cand_stride = s->max_rows + 1;
  s->o_row_seq = take(rows); s->o_row_pos = take(rows); s->o_row_tok = take(rows);
  s->o_row_src = take(rows); s->o_row_dst = take(rows);
  s->o_seq_row0 = take(s->B); s->o_seq_m = take(s->B); s->o_seq_p0 = take(s->B); s->o_seq_qt0 = take(s->B);
  s->o_qt_seq = take(qts); s->o_qt_local = take(qts);
  s->o_cand = take((size_t)s->B * s->cand_stride); s->o_n_cand = take(s->B);
  s->o_bt = take((size_t)s->B * s->pps);
  s->o_u = take(uniforms);                              // (floats)
  s->meta_ints = o;
}

static size_t carve(ee_session* s, char* base) {
  const ee_model* m = s->m;
  const ee_config& c = m->cfg;
  const bool bf = m->bf16;
  const int d = c.d_model, D = c.head_dim, Hq = c.n_q_heads, Hkv = c.n_kv_heads;
  const int rep = Hq / Hkv;
  Carver cv{base};
  const size_t es = bf ? 2 : 4;
  const int Mp = s->Mp;
  s->kv = cv.take<char>((size_t)c.n_layers * s->n_pages * Hkv * 2 * EE_PAGE * kv_page_dim(D) * es);
  s->X = cv.take<float>((size_t)s->maxM * d);
  s->XN = bf ? (void*)cv.take<bf16_t>((size_t)Mp * ceil_div(d, 32) * 32) : nullptr;
  s->Qb = bf ? (void*)cv.take<bf16_t>((size_t)Hkv * s->maxQT * 16 * D) : (void*)cv.take<float>((size_t)s->maxM * Hq * D);
  s->AO = bf ? (void*)cv.take<bf16_t>((size_t)Mp * ceil_div(Hq * D, 32) * 32) : (void*)cv.take<float>((size_t)s->maxM * Hq * D);
  s->H = bf ? (void*)cv.take<bf16_t>((size_t)Mp * ceil_div(c.d_ffn, 32) * 32) : (void*)cv.take<float>((size_t)s->maxM * c.d_ffn);
  s->LOGITS = cv.take<float>((size_t)s->headM * c.vocab);
  if (c.head_rank > 0) {
    s->Z = cv.take<float>((size_t)s->headM * d);
    s->T = bf ? nullptr : cv.take<float>((size_t)s->headM * c.head_rank);
    if (bf) {
      s->TF = cv.take<bf16_t>((size_t)s->headMp * c.head_rank);
      s->ssq_t = cv.take<float>((size_t)ceil_div(c.head_rank, 16) * s->headMp);
      s->ones = cv.take<float>(c.head_rank);
    }
  }
  s->Hd = cv.take<float>((size_t)s->B * s->max_rows * d);
  s->Hi = cv.take<float>((size_t)s->B * s->max_rows * d);
  for (int j = 2; j < s->n_levels; ++j) s->Hup[j - 2] = cv.take<float>((size_t)s->B * s->max_rows * d);
  s->cs = cv.take<float2>((size_t)s->maxM * (D / 2));
  s->rowinfo = cv.take<int4>((size_t)s->maxM);
  s->vtok = cv.take<int>(s->maxM);
  s->tok_next = cv.take<int>(s->maxM);
  s->out_dev = s->tok_next;                                           // (sampling: accept counts on their way to the draw; no drafting in that call)
  s->page_scratch = cv.take<int>(s->pps);
  if (bf) {
    // attention split scratch: all 64 splits for verify-sized calls (<= 64 rows), 8 at 512 rows and fewer for larger context-build passes
    const size_t qt_small = (size_t)ceil_div(std::min(s->headM, 64) * rep, 16) + s->B;
    s->part_units = std::max(qt_small * s->max_splits, (size_t)(ceil_div(s->headM * rep, 16) + s->B) * 8);
    s->part_o = cv.take<float>(s->part_units * Hkv * 16 * D);
    s->part_ml = cv.take<float>(s->part_units * Hkv * 32);
    s->pmax = cv.take<float>((size_t)m->head.ntiles() * s->headMp);
    s->pidx = cv.take<int>((size_t)m->head.ntiles() * s->headMp);
    s->ssq = cv.take<float>((size_t)ceil_div(d, 16) * Mp);            // deferred-RMSNorm partials [d/16][Mp]
    size_t gp = 0;                                                    // K-share scratch of the row-tiled GEMM
    for (const MatLoc* ml : {&m->L[0].qkv, &m->L[0].o, &m->L[0].gu, &m->L[0].down, &m->head, &m->auxA[0], &m->auxB[0]})
      if (ml->Np > 0) gp = std::max(gp, bf16_gemm_rows_scratch_floats(ml->ntiles(), ml->ktiles()));
    s->gemm_part = s->maxM > 64 ? cv.take<float>(gp) : nullptr;
    s->inv_rms = cv.take<float>(s->inv_cap);
  }
  s->slot[0].d = cv.take<int>(s->meta_cap);
  s->slot[1].d = cv.take<int>(s->meta_cap - s->B * (s->max_rows + 1));     // (no uniform numbers there)
  (void)rep;
  return align_up(cv.cur, 256);
}

// most_rows: upper bound of the rows of a context-build pass (a multiple of 512; bf16).  At the least one no buffer is larger
// than a session with passes of 512 rows ever needed: batch-wide calls of more rows then run their GEMMs in parts.
static const int kMostPassRows = 4096, kLeastPassRows = 512;
static int shape_session(ee_session* s, const ee_model* m, int batch, int max_ctx, int max_rows, int total_pages, int most_rows = kMostPassRows) {
  if (!m || batch < 1 || max_ctx < 2 || max_rows < 2) { ee_set_error("bad session shape"); return EE_ERR_ARG; }
  if (!m->bf16 && max_ctx > 8192) { ee_set_error("EE_F32 sessions support max_ctx <= 8192"); return EE_ERR_ARG; }
  const int rep = m->cfg.n_q_heads / m->cfg.n_kv_heads;
  s->m = const_cast<ee_model*>(m);
  s->n_levels = (int)m->exits.size() - 1;
  s->B = batch; s->max_ctx = max_ctx; s->max_rows = max_rows;
  s->pps = ceil_div(max_ctx, EE_PAGE);
  s->n_pages = total_pages > 0 ? total_pages : batch * s->pps;
  // context-build rows per pass: 4096 give the blocked GEMM whole rounds of blocks (gate/up at the 8B width: a tenth more products a second
  // than at 2048 rows, see gemm_block_kernel); no more than the sequences and the page pool can hold
  const long held = std::min((long)batch * max_ctx, (long)s->n_pages * EE_PAGE);
  s->chunk = m->bf16 ? (int)std::max<long>(kLeastPassRows, std::min<long>(most_rows, (held + 511) / 512 * 512)) : 64;
  s->headM = std::max(batch * max_rows, m->bf16 ? 512 : 64);
  s->headMp = s->headM <= 64 ? 64 : ceil_div(s->headM, 512) * 512;
  s->maxM = std::max(batch * max_rows, s->chunk);
  // activation rows padded to whole GEMM passes: 64 rows (skinny kernel), blocks of 512 (the row-tiled kernel requests up to 32 row tiles)
  s->Mp = s->maxM <= 64 ? 64 : ceil_div(s->maxM, 512) * 512;
  s->maxQT = ceil_div(s->maxM * rep, 16) + batch;
  s->ssq_stride = s->Mp;
  s->inv_cap = most_rows > kLeastPassRows ? std::max(512, s->maxM) : 512;
  layout_meta(s, s->maxM, s->maxQT, s->B * s->max_rows + s->B);   // (the largest block; every call lays out its own)
  s->meta_cap = s->meta_ints;
  return EE_OK;
}

extern "C" size_t ee_session_bytes(const ee_model* m, int batch, int max_ctx, int max_rows, int total_pages) {
  ee_session tmp;
  if (shape_session(&tmp, m, batch, max_ctx, max_rows, total_pages) != EE_OK) return 0;
  return carve(&tmp, nullptr);
}

extern "C" int ee_session_create(ee_model* m, int batch, int max_ctx, int max_rows, int total_pages, void* dev_arena,
                                 size_t arena_bytes, void* stream, ee_session** out) {
  if (!out || !dev_arena || ((uintptr_t)dev_arena & 255)) { ee_set_error("arena must be non-null and 256-byte aligned"); return EE_ERR_ARG; }
  ee_session* s = new ee_session();
  int rc = shape_session(s, m, batch, max_ctx, max_rows, total_pages);
  if (rc != EE_OK) { delete s; return rc; }
  s->st = (hipStream_t)stream;
  s->base = (char*)dev_arena;
  // an arena short of ee_session_bytes() gets shorter passes, as long as one of them fits
  for (int most = kMostPassRows; (s->bytes = carve(s, s->base)) > arena_bytes && most > kLeastPassRows;) {
    most = std::max(kLeastPassRows, s->chunk - 512);
    shape_session(s, m, batch, max_ctx, max_rows, total_pages, most);
  }
  if (arena_bytes < s->bytes) {
    ee_set_error("session arena too small: %zu < %zu", arena_bytes, s->bytes);
    delete s; return EE_ERR_CAPACITY;
  }
  hipError_t e = hipMemsetAsync(s->base, 0, s->bytes, s->st);
  const std::vector<float> unit(s->ones ? m->cfg.head_rank : 0, 1.0f);
  if (e == hipSuccess && s->ones) e = hipMemcpyAsync(s->ones, unit.data(), unit.size() * sizeof(float), hipMemcpyHostToDevice, s->st);
  for (int i = 0; i < 2 && e == hipSuccess; ++i) {
    e = hipHostMalloc((void**)&s->slot[i].h, s->meta_cap * sizeof(int), hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s->slot[i].copied, hipEventDisableTiming);
  }
  if (e == hipSuccess) e = hipHostMalloc((void**)&s->out_host, (2 * (size_t)batch + (size_t)batch * max_rows) * sizeof(int), hipHostMallocDefault);
  if (e == hipSuccess) e = hipStreamSynchronize(s->st);
  if (e != hipSuccess) { ee_set_error("session create: %s", hipGetErrorString(e)); ee_session_free(s); return EE_ERR_HIP; }
  s->seq.resize(batch);
  s->free_pages.resize(s->n_pages);
  for (int i = 0; i < s->n_pages; ++i) s->free_pages[i] = s->n_pages - 1 - i;   // pop_back hands out 0, 1, 2, ...
  *out = s;
  return EE_OK;
}

extern "C" void ee_session_free(ee_session* s) {
  if (!s) return;
  if (s->st) (void)hipStreamSynchronize(s->st);
  for (auto& t : s->timers) { (void)hipEventDestroy(t.a); (void)hipEventDestroy(t.b); }
  for (int i = 0; i < 2; ++i) {
    if (s->slot[i].h) (void)hipHostFree(s->slot[i].h);
    if (s->slot[i].copied) (void)hipEventDestroy(s->slot[i].copied);
  }
  if (s->out_host) (void)hipHostFree(s->out_host);
  delete s;
}

// ---------------------------------------------------------------------------------------------
// pages
// ---------------------------------------------------------------------------------------------
static int pages_needed_total(const ee_session* s, const std::vector<int>& want_positions) {
  int need = 0;
  for (int b = 0; b < s->B; ++b) {
    int have = (int)s->seq[b].pages.size(), want = ceil_div(want_positions[b], EE_PAGE);
    if (want > have) need += want - have;
  }
  return need;
}
// make sure sequence b owns pages for positions [0, n)
static int grow_pages(ee_session* s, int b, int n) {
  SeqState& q = s->seq[b];
  while ((int)q.pages.size() * EE_PAGE < n) {
    if (s->free_pages.empty() || (int)q.pages.size() >= s->pps) { ee_set_error("KV page pool exhausted"); return EE_ERR_CAPACITY; }
    q.pages.push_back(s->free_pages.back());
    s->free_pages.pop_back();
  }
  return EE_OK;
}
static int max_len(const ee_session* s, const SeqState& q) {
  int m = 0;
  for (int g = 0; g <= s->n_levels; ++g) m = std::max(m, q.len[g]);
  return m;
}
// every group at the same length, nothing waiting above L_i: the state after a prompt, a vanilla step or the last level
static void settle(const ee_session* s, SeqState& q) {
  for (int g = 0; g <= s->n_levels; ++g) { q.len[g] = (int)q.C.size() - 1; q.cut[g] = (int)q.C.size(); }
}
// give back pages no group needs any more (Sec. 3.2 pruning: only the table tail changes)
static void trim_pages(ee_session* s, int b) {
  SeqState& q = s->seq[b];
  int keep = ceil_div(max_len(s, q) + 1, EE_PAGE);
  while ((int)q.pages.size() > keep) { s->free_pages.push_back(q.pages.back()); q.pages.pop_back(); }
}
static int check_capacity(ee_session* s, const std::vector<int>& want_positions) {
  for (int b = 0; b < s->B; ++b)
    if (want_positions[b] > s->max_ctx) { ee_set_error("sequence %d would need %d positions (max_ctx %d)", b, want_positions[b], s->max_ctx); return EE_ERR_CAPACITY; }
  if (pages_needed_total(s, want_positions) > (int)s->free_pages.size()) { ee_set_error("KV page pool exhausted"); return EE_ERR_CAPACITY; }
  return EE_OK;
}

// ---------------------------------------------------------------------------------------------
// per-call metadata
// ---------------------------------------------------------------------------------------------
struct CallPlan {
  int M = 0, max_m = 0, total_qt = 0;
  std::vector<int> m, p0;        // per sequence rows and first position (m = 0: not taking part)
};

static CallMeta meta_ptrs(const ee_session* s, const int* d) {
  CallMeta c;
  c.row_seq = d + s->o_row_seq; c.row_pos = d + s->o_row_pos; c.row_tok = d + s->o_row_tok;
  c.row_src = d + s->o_row_src; c.row_dst = d + s->o_row_dst;
  c.seq_row0 = d + s->o_seq_row0; c.seq_m = d + s->o_seq_m; c.seq_p0 = d + s->o_seq_p0; c.seq_qt0 = d + s->o_seq_qt0;
  c.qt_seq = d + s->o_qt_seq; c.qt_local = d + s->o_qt_local; c.cand = d + s->o_cand; c.n_cand = d + s->o_n_cand;
  c.block_table = d + s->o_bt;
  return c;
}

// Fill slot `si` from the plan: rows are packed sequence by sequence.  The callbacks give the
// per-row token / gather source / scatter destination; candidates are filled by the caller.
template <class RowFn>
static int build_meta(ee_session* s, int si, CallPlan& p, RowFn row_fn, int uniforms = 0) {
  MetaSlot& sl = s->slot[si];
  if (sl.in_flight) { HIP_TRY(hipEventSynchronize(sl.copied)); sl.in_flight = false; }
  int* h = sl.h;
  const int rep = s->m->cfg.n_q_heads / s->m->cfg.n_kv_heads;
  int row = 0, qt = 0;
  for (int b = 0; b < s->B; ++b) { row += p.m[b]; qt += ceil_div(p.m[b] * rep, 16); }
  if (row > s->maxM || qt > s->maxQT) { ee_set_error("internal: call exceeds work buffers (%d rows)", row); return EE_ERR_CAPACITY; }
  layout_meta(s, row, qt, uniforms);
  row = qt = 0;
  p.max_m = 0;
  for (int b = 0; b < s->B; ++b) {
    int m = p.m[b];
    h[s->o_seq_row0 + b] = row; h[s->o_seq_m + b] = m; h[s->o_seq_p0 + b] = p.p0[b]; h[s->o_seq_qt0 + b] = qt;
    h[s->o_n_cand + b] = 0;
    if (m == 0) continue;
    p.max_m = std::max(p.max_m, m);
    for (int r = 0; r < m; ++r, ++row) {
      h[s->o_row_seq + row] = b; h[s->o_row_pos + row] = p.p0[b] + r;
      int tok = 0, src = 0, dst = 0;
      row_fn(b, r, tok, src, dst);
      h[s->o_row_tok + row] = tok; h[s->o_row_src + row] = src; h[s->o_row_dst + row] = dst;
    }
    int nqt = ceil_div(m * rep, 16);
    for (int t = 0; t < nqt; ++t, ++qt) { h[s->o_qt_seq + qt] = b; h[s->o_qt_local + qt] = t; }
  }
  p.M = row; p.total_qt = qt;
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    for (size_t i = 0; i < q.pages.size(); ++i) h[s->o_bt + (size_t)b * s->pps + i] = q.pages[i];
  }
  return EE_OK;
}
static int upload_meta(ee_session* s, int si) {
  MetaSlot& sl = s->slot[si];
  if (k_store_meta(s->st, sl.h, sl.d, (int)s->meta_ints)) return EE_OK;
  HIP_TRY(hipMemcpyAsync(sl.d, sl.h, s->meta_ints * sizeof(int), hipMemcpyHostToDevice, s->st));
  HIP_TRY(hipEventRecord(sl.copied, s->st));
  sl.in_flight = true;
  return EE_OK;
}

// Behind the last layer of a context-build pass only some rows have a reader: those that end a prompt, and the last 512-row piece that the
// introspection calls report.  Of the other rows the layer has to leave K and V in the cache, nothing else.  The wanted rows are trailing
// rows of their sequences, so the rest of the layer is a call of its own over fewer rows, packed anew.  Sequences keep whole q-tiles (rows
// from a multiple of 16 on), and the reported piece starts at a row that is a multiple of 16 (rows in the gap in front of it hold copies).
struct TailPlan {
  bool on = false;
  CallPlan p;                    // the wanted rows: M (0: none), total_qt, per-sequence rows and first positions
  CallMeta mt;
  const int* row_idx = nullptr;  // [M] row of the pass
  const int* qt_src = nullptr;   // [total_qt] q-tile of the pass
  int piece = 0;                 // first row of the reported piece
  std::vector<int> row0;         // first row of every sequence
};
// keep[b]: wanted trailing rows of sequence b; piece0 >= 0: all rows from that row of the pass on are among them.  The tables lie behind the
// n_src entries that row_src holds, where a context build has no rows to gather or scatter, and the rows are moved by way of LOGITS, which the
// head fills later; off where either does not fit, or where a quarter of the rows is not saved.  Called between build_meta and upload_meta.
static void plan_tail(ee_session* s, int si, const CallPlan& p, const std::vector<int>& keep, int piece0, int n_src, TailPlan& t) {
  const ee_config& c = s->m->cfg;
  const int B = s->B, rep = c.n_q_heads / c.n_kv_heads;
  t = TailPlan();
  t.p.m.assign(B, 0); t.p.p0.assign(B, 0); t.row0.assign(B, 0);
  int row = 0, qt = 0;
  for (int b = 0, first = 0; b < B; first += p.m[b], ++b) {
    if (!keep[b]) continue;
    const int skip = (p.m[b] - keep[b]) & ~15, m = p.m[b] - skip;
    if (piece0 >= 0 && first <= piece0 && piece0 < first + p.m[b]) {       // the piece starts in this sequence
      const int before = piece0 - first - skip;
      t.piece = ceil_div(row + before, 16) * 16;
      row = t.piece - before;
    }
    t.p.m[b] = m; t.p.p0[b] = p.p0[b] + skip; t.row0[b] = row;
    t.p.max_m = std::max(t.p.max_m, m);
    row += m; qt += ceil_div(m * rep, 16);
  }
  t.p.M = row; t.p.total_qt = qt;
  auto pad = [](int n) { return (n + 3) / 4 * 4; };
  const size_t moved = (size_t)row * c.d_model * sizeof(float) + (size_t)c.n_kv_heads * qt * 16 * c.head_dim * sizeof(bf16_t);
  if (4 * row > 3 * p.M || pad(n_src) + pad(row) + 4 * pad(B) + 3 * pad(qt) > 2 * pad(p.M) ||
      moved > (size_t)s->headM * c.vocab * sizeof(float)) return;
  t.on = true;
  int* h = s->slot[si].h;
  size_t o = s->o_row_src + pad(n_src);
  auto take = [&](int n) { const size_t r = o; o += pad(n); return r; };
  const size_t o_idx = take(row), o_row0 = take(B), o_m = take(B), o_p0 = take(B), o_qt0 = take(B), o_qseq = take(qt), o_qloc = take(qt), o_qsrc = take(qt);
  std::fill(h + o_idx, h + o_idx + row, 0);
  qt = 0;
  for (int b = 0, first = 0; b < B; first += p.m[b], ++b) {
    const int m = t.p.m[b], skip = p.m[b] - m;
    h[o_row0 + b] = t.row0[b]; h[o_m + b] = m; h[o_p0 + b] = t.p.p0[b]; h[o_qt0 + b] = qt;
    for (int r = 0; r < m; ++r) h[o_idx + t.row0[b] + r] = first + skip + r;
    for (int i = 0; i < ceil_div(m * rep, 16); ++i, ++qt) {
      h[o_qseq + qt] = b; h[o_qloc + qt] = i; h[o_qsrc + qt] = h[s->o_seq_qt0 + b] + skip * rep / 16 + i;
    }
  }
  const int* d = s->slot[si].d;
  t.mt = meta_ptrs(s, d);
  t.mt.seq_row0 = d + o_row0; t.mt.seq_m = d + o_m; t.mt.seq_p0 = d + o_p0; t.mt.seq_qt0 = d + o_qt0;
  t.mt.qt_seq = d + o_qseq; t.mt.qt_local = d + o_qloc;
  t.row_idx = d + o_idx; t.qt_src = d + o_qsrc;
}

// ---------------------------------------------------------------------------------------------
// launch accounting
// ---------------------------------------------------------------------------------------------
// With timing on, a family call is bracketed by two recorded events; a call that is one skinny-GEMM launch takes
// the second pair instead, attached to its dispatch (the kernel's own start and end: what a kernel trace reports,
// 2-5 us less than the bracket, which also spans the launch gap).
struct Scope {
  ee_session* s; int fam; hipEvent_t a = nullptr, b = nullptr;
  LaunchEvents own{nullptr, nullptr, false};
  Scope(ee_session* s_, int f) : s(s_), fam(f) {
    s->launches[fam]++;
    if (s->time_kernels) {
      (void)hipEventCreate(&a); (void)hipEventCreate(&b); (void)hipEventRecord(a, s->st);
      (void)hipEventCreate(&own.start); (void)hipEventCreate(&own.stop);
      g_launch_events = &own;
    }
  }
  ~Scope() {
    if (!a) return;
    g_launch_events = nullptr;
    if (own.used) {
      s->timers.push_back({fam, own.start, own.stop});
      (void)hipEventDestroy(a); (void)hipEventDestroy(b);
    } else {
      (void)hipEventRecord(b, s->st);
      s->timers.push_back({fam, a, b});
      (void)hipEventDestroy(own.start); (void)hipEventDestroy(own.stop);
    }
  }
};
#define KF(fam, call) do { Scope sc_(s, fam); call; } while (0)

static void reset_accounting(ee_session* s) {
  for (auto& t : s->timers) { (void)hipEventDestroy(t.a); (void)hipEventDestroy(t.b); }
  s->timers.clear();
  memset(s->launches, 0, sizeof(s->launches));
}

// ---------------------------------------------------------------------------------------------
// forward pass pieces
// ---------------------------------------------------------------------------------------------
// the skinny kernel for few rows (see strips_serve), the row-tiled one up to 512 (wide matrices: 256), beyond the blocked one or the row-tiled one
// in parts (see runs_blocked)
// returns the number of partial sums of squares per row that an EPI_ADD call with a next operand leaves
static int gemm(ee_session* s, int epi, const MatLoc& ml, const bf16_t* A, int M, const GemmOut& o) {
  const bf16_t* W = (const bf16_t*)(s->m->base + ml.off);
  if (!bf16_takes_strips(ml.ntiles(), ml.ktiles(), M)) return bf16_gemm_rows(s->st, epi, W, ml.ntiles(), ml.ktiles(), A, M, ml.N, o, s->gemm_part, s->inv_rms, s->inv_cap);
  bf16_gemm(s->st, epi, W, ml.ntiles(), ml.ktiles(), A, M, ml.N, o);
  return ml.ntiles();
}

// offset of the gain that normalises the hidden state behind layer l1: the adapter's own gain at an early exit
// with an auxiliary head, else the shared final gain
static size_t closing_gain(const ee_model* m, int l1) {
  if (m->cfg.head_rank > 0)
    for (size_t e = 0; e + 1 < m->exits.size(); ++e)
      if (l1 == m->exits[e]) return m->auxg[e];
  return m->gfinal;
}

// attention plan of a call (the same for all its layers) and the scratch handed to the kernels
static AttnPlan attention_plan(const ee_session* s, const CallPlan& p, int pos_add, AttnScratch& scr) {
  const ee_config& c = s->m->cfg;
  scr = AttnScratch{s->part_o, s->part_ml, (int)std::min<size_t>(s->max_splits, s->part_units / std::max(1, p.total_qt))};
  if (!s->m->bf16) return AttnPlan{ATTN_RING, 1, 1};
  std::vector<int> kv_end(s->B);
  for (int b = 0; b < s->B; ++b) kv_end[b] = p.m[b] > 0 ? p.p0[b] + p.m[b] + pos_add : 0;
  return bf16_attention_plan(kv_end.data(), p.m.data(), s->B, c.n_q_heads, c.n_kv_heads, scr.max_splits);
}

// where the rows of a pass come from: the embedding of tokens (a1 of a pass that starts at layer 0), kept hidden rows
// gathered by index (hidden-state reuse of Alg. 2), or the residual stream as it stands
struct PassSource {
  const int* tok = nullptr;
  const float* rows = nullptr; const int* row_idx = nullptr;
};
// where the hidden rows behind the last layer of a pass are kept besides the stream (H_d, H_i, a level's rows): row r
// goes to rows[row_idx[r] + add]; the last down projection's epilogue writes them
struct PassSink {
  float* rows = nullptr; const int* row_idx = nullptr; int add = 0;
};

// tail: the rows of the last layer that have a reader, where those are few (context builds of bf16 models)
static void run_layers(ee_session* s, int l0, int l1, const CallPlan& p, const CallMeta& mt, int pos_add, const PassSource& src = PassSource(),
                       const PassSink& sink = PassSink(), const TailPlan* tail = nullptr) {
  const ee_model* m = s->m;
  const ee_config& c = m->cfg;
  const int d = c.d_model, D = c.head_dim, Hq = c.n_q_heads, Hkv = c.n_kv_heads;
  int M = p.M;
  hipStream_t st = s->st;
  if (m->bf16) {
    // one launch: rows into the stream, the first layer's operand, the rotary table and the epilogue lookups
    KF(KF_NORM, bf16_begin_pass(st, src.tok ? (const bf16_t*)(m->base + m->emb) : nullptr, src.tok, src.rows, src.row_idx, s->X,
                                (const float*)(m->base + m->L[l0].g1), c.rms_eps, (bf16_t*)s->XN, m->L[l0].qkv.ktiles(), M, d, mt,
                                pos_add, m->inv_freq, s->cs, D / 2, s->pps, s->rowinfo));
  } else {
    KF(KF_EMBED, f32_begin_pass(st, src.tok ? (const float*)(m->base + m->emb) : nullptr, src.tok, src.rows, src.row_idx, s->X, M, d, mt,
                                pos_add, m->inv_freq, s->cs, D / 2, s->pps, s->rowinfo));
  }
  AttnScratch scr;
  const AttnPlan attn = attention_plan(s, p, pos_add, scr);
  s->last_attn = m->bf16 ? attn.kind : -1;
  for (int l = l0; l < l1; ++l) {
    const LayerLoc& L = m->L[l];
    const float* g1 = (const float*)(m->base + L.g1);
    const float* g2 = (const float*)(m->base + L.g2);
    if (m->bf16) {
      // five launches per layer (six with the merge of a split attention); RMSNorm is deferred into the projections (see NormIn / NormOut)
      const int Mp = s->ssq_stride;
      NormIn nin;         // operand left by the previous EPI_ADD launch
      nin.ssq = s->ssq; nin.n_part = s->ssq_parts; nin.stride = Mp; nin.inv_d = 1.0f / (float)d; nin.eps = c.rms_eps;
      NormOut nout;
      nout.xn = (bf16_t*)s->XN; nout.ktiles = ceil_div(d, 32); nout.ssq = s->ssq; nout.stride = Mp;
      GemmOut o;
      if (l != l0) o.nin = nin;            // (the first layer's operand was normalised when the pass was opened)
      RopeOut& ro = o.rope;
      ro.cs = s->cs; ro.rowinfo = s->rowinfo; ro.Hq = Hq; ro.Hkv = Hkv; ro.D = D; ro.layer = l;
      ro.n_pages = s->n_pages; ro.total_qt = p.total_qt; ro.Q = (bf16_t*)s->Qb; ro.kv = (bf16_t*)s->kv;
      KF(KF_GEMM_QKV, gemm(s, EPI_ROPE, L.qkv, (const bf16_t*)s->XN, M, o));
      const float* R = s->X;
      if (l + 1 == l1 && tail) {
        // K and V of all rows are in the cache; the rest of the layer runs over the wanted rows, moved to the front (their stream rows and Q
        // tiles by way of LOGITS; H must keep the zeros behind d_ffn)
        M = tail->p.M;
        if (M == 0) break;
        float* rows = s->LOGITS;
        bf16_t* q = (bf16_t*)(rows + (size_t)M * d);
        AttnScratch few;
        const AttnPlan plan = attention_plan(s, tail->p, pos_add, few);
        KF(KF_ATTN, bf16_gather_tail(st, s->X, tail->row_idx, M, d, rows, (const bf16_t*)s->Qb, tail->qt_src, tail->p.total_qt, p.total_qt, Hkv, D, q);
                    bf16_attention(st, plan, q, (const bf16_t*)s->kv, tail->mt, pos_add, s->B, tail->p.max_m, tail->p.total_qt,
                                   Hq, Hkv, D, l, s->n_pages, s->pps, few, (bf16_t*)s->AO, L.o.ktiles()));
        R = rows;
      } else {
        KF(KF_ATTN, bf16_attention(st, attn, (const bf16_t*)s->Qb, (const bf16_t*)s->kv, mt, pos_add, s->B, p.max_m, p.total_qt,
                                   Hq, Hkv, D, l, s->n_pages, s->pps, scr, (bf16_t*)s->AO, L.o.ktiles()));
      }
      o = GemmOut(); o.Y = s->X; o.R = R; o.ldy = d; o.nout = nout; o.nout.g = g2;
      KF(KF_GEMM_O, nin.n_part = gemm(s, EPI_ADD, L.o, (const bf16_t*)s->AO, M, o));
      o = GemmOut(); o.H = (bf16_t*)s->H; o.h_ktiles = L.down.ktiles(); o.nin = nin;
      KF(KF_GEMM_GU, gemm(s, EPI_SWIGLU, L.gu, (const bf16_t*)s->XN, M, o));
      // the down projection leaves the operand of whatever reads the stream next: the next layer's QKV
      // projection, or the shared exit head behind the last layer of the pass
      o = GemmOut(); o.Y = s->X; o.R = s->X; o.ldy = d; o.nout = nout;
      o.nout.g = l + 1 < l1 ? (const float*)(m->base + m->L[l + 1].g1) : (const float*)(m->base + closing_gain(m, l1));
      if (l + 1 == l1) { o.Y2 = sink.rows; o.y2_idx = sink.row_idx; o.y2_add = sink.add; }
      KF(KF_GEMM_DOWN, s->ssq_parts = gemm(s, EPI_ADD, L.down, (const bf16_t*)s->H, M, o));
    } else {
      const float* Wqkv = (const float*)(m->base + L.qkv.off);
      const float* Wo = (const float*)(m->base + L.o.off);
      const float* Wgu = (const float*)(m->base + L.gu.off);
      const float* Wd = (const float*)(m->base + L.down.off);
      // five launches per layer: norms, rotary embedding, KV append and activation sit in the projections
      const bool end = l + 1 == l1;
      F32Out o;
      o.Y = (float*)s->Qb; o.cs = s->cs; o.rowinfo = s->rowinfo; o.Hq = Hq; o.Hkv = Hkv; o.D = D; o.layer = l; o.n_pages = s->n_pages;
      o.kv = (float*)s->kv;
      KF(KF_GEMM_QKV, f32_qkv(st, s->X, g1, c.rms_eps, Wqkv, M, d, o));
      KF(KF_ATTN, f32_attention(st, (const float*)s->Qb, (const float*)s->kv, mt, pos_add, M, Hq, Hkv, D, l, s->n_pages, s->pps,
                                s->max_ctx, (float*)s->AO));
      KF(KF_GEMM_O, f32_gemm(st, (const float*)s->AO, Hq * D, nullptr, 0.f, Wo, s->X, d, M, d, Hq * D, true));
      KF(KF_GEMM_GU, f32_gate_up(st, s->X, g2, c.rms_eps, Wgu, (float*)s->H, M, c.d_ffn, d));
      KF(KF_GEMM_DOWN, f32_gemm(st, (const float*)s->H, c.d_ffn, nullptr, 0.f, Wd, s->X, d, M, d, c.d_ffn, true, end ? sink.rows : nullptr,
                                sink.row_idx, sink.add));
    }
  }
}

// Prediction head of exit `which` (0 = L_d, 1 = L_i, ..., n_levels = L_f) + arg max for rows 0..M-1 of X -> vtok.
// The shared final RMSNorm and LM head (Sec. 3.1); at an early exit of a model with auxiliary heads
// (App. I) behind that exit's rank-r adapter  z = x + B (A RMSNorm(x; g)),  which leaves X itself alone.
// row0 (a multiple of 16): the rows are row0 .. row0+M-1 of the pass instead (final exit only).  ended: the rows are those
// listed on the device (the ends of prompts in a context build), normalised here; X's other rows need no head.
// take: hand every row's token on (drafting, decoding).
static void exit_head(ee_session* s, int M, int which, int row0 = 0, const int* ended = nullptr, const TakeToken& take = TakeToken()) {
  const ee_model* m = s->m;
  const ee_config& c = m->cfg;
  hipStream_t st = s->st;
  const int d = c.d_model, r = c.head_rank;
  const float* gf = (const float*)(m->base + m->gfinal);
  const bool aux = r > 0 && which < s->n_levels;
  if (m->bf16) {
    // the last down projection of the pass left XN = bf16(x * gain) and the partial sums of squares
    const int Mp = s->ssq_stride;
    const bf16_t* operand = (const bf16_t*)s->XN + (size_t)row0 * ceil_div(d, 32) * 32;
    NormIn nin;
    nin.ssq = s->ssq + row0; nin.n_part = s->ssq_parts; nin.stride = Mp; nin.inv_d = 1.0f / (float)d; nin.eps = c.rms_eps;
    if (aux) {
      // t = A n(x): only as the next operand TF; z = x + B t: into rows of its own (the stream itself stays as it is),
      // leaving the shared head's operand XN = bf16(z * gfinal)
      GemmOut o;
      o.nin = nin;
      o.nout.xn = (bf16_t*)s->TF; o.nout.ktiles = r / 32; o.nout.ssq = s->ssq_t; o.nout.stride = s->headMp; o.nout.g = s->ones;
      KF(KF_GEMM_HEAD, gemm(s, EPI_ADD, m->auxA[which], (const bf16_t*)s->XN, M, o));
      o = GemmOut(); o.Y = s->Z; o.R = s->X; o.ldy = d;
      o.nout.xn = (bf16_t*)s->XN; o.nout.ktiles = ceil_div(d, 32); o.nout.ssq = s->ssq; o.nout.stride = Mp; o.nout.g = gf;
      KF(KF_GEMM_HEAD, nin.n_part = gemm(s, EPI_ADD, m->auxB[which], (const bf16_t*)s->TF, M, o));
    }
    GemmOut o;
    if (ended) {
      // (XN's first rows: the pass is over, and a piece that gets a head of its own lies behind the rows that end in front of it)
      KF(KF_NORM, bf16_rmsnorm(st, s->X, ended, gf, c.rms_eps, (bf16_t*)s->XN, ceil_div(d, 32), M, d));
    } else {
      o.nin = nin;
    }
    // (max, arg max) partials [row][tile]: the reduction of a row then reads one contiguous strip
    const int pstride = m->head.ntiles();
    o.pmax = s->pmax; o.pidx = s->pidx; o.pstride = pstride;
    if (s->debug_logits || s->need_logits) { o.Y = s->LOGITS; o.ldy = c.vocab; }
    KF(KF_GEMM_HEAD, gemm(s, EPI_ARGMAX, m->head, operand, M, o));
    KF(KF_ARGMAX, bf16_argmax_reduce(st, s->pmax, s->pidx, m->head.ntiles(), pstride, M, s->vtok, take));
  } else {
    const float* hidden = s->X;
    if (aux) {
      KF(KF_GEMM_HEAD, f32_gemm(st, s->X, d, (const float*)(m->base + m->auxg[which]), c.rms_eps, (const float*)(m->base + m->auxA[which].off),
                                s->T, r, M, r, d, false));
      (void)hipMemcpyAsync(s->Z, s->X, (size_t)M * d * sizeof(float), hipMemcpyDeviceToDevice, st);
      KF(KF_GEMM_HEAD, f32_gemm(st, s->T, r, nullptr, 0.f, (const float*)(m->base + m->auxB[which].off), s->Z, d, M, d, r, true));
      hidden = s->Z;
    }
    KF(KF_GEMM_HEAD, f32_gemm(st, hidden, d, gf, c.rms_eps, (const float*)(m->base + m->head.off), s->LOGITS, c.vocab, M, c.vocab, d, false));
    KF(KF_ARGMAX, f32_argmax(st, s->LOGITS, M, c.vocab, s->vtok, take));
  }
  s->last_rows = M; s->last_row0 = row0;
}

static int finish(ee_session* s) {
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipStreamSynchronize(s->st));
  for (int i = 0; i < 2; ++i) s->slot[i].in_flight = false;
  return EE_OK;
}

// ---------------------------------------------------------------------------------------------
// C ABI: prefill
// ---------------------------------------------------------------------------------------------
// (Re)start the sequences with lens[b] > 0 from their prompts (tokens: those prompts packed in sequence order);
// sequences with lens[b] == 0 keep their state.  Pages of a restarted sequence go back to the pool first.
static int prefill_impl(ee_session* s, const int32_t* tokens, const int32_t* lens, int32_t* first_token) {
  const ee_config& c = s->m->cfg;
  std::vector<int> want(s->B);
  size_t total = 0;
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    want[b] = lens[b] > 0 ? lens[b] + 1 : (q.started ? max_len(s, q) : 0);
    total += lens[b];
  }
  for (size_t i = 0; i < total; ++i)
    if (tokens[i] < 0 || tokens[i] >= c.vocab) { ee_set_error("token id out of range"); return EE_ERR_ARG; }
  // capacity is checked against the pool as it will be once the restarted sequences have given their pages back
  {
    size_t freed = 0, need = 0;
    for (int b = 0; b < s->B; ++b) {
      if (lens[b] <= 0) continue;
      if (want[b] > s->max_ctx) { ee_set_error("sequence %d would need %d positions (max_ctx %d)", b, want[b], s->max_ctx); return EE_ERR_CAPACITY; }
      freed += s->seq[b].pages.size();
      need += (size_t)ceil_div(want[b], EE_PAGE);
    }
    if (need > s->free_pages.size() + freed) { ee_set_error("KV page pool exhausted"); return EE_ERR_CAPACITY; }
  }
  for (int b = 0; b < s->B; ++b) {
    if (lens[b] <= 0) continue;
    SeqState& q = s->seq[b];
    for (int pg : q.pages) s->free_pages.push_back(pg);
    q = SeqState();
  }
  reset_accounting(s);
  std::vector<size_t> off0(s->B, 0);
  std::vector<int> done(s->B, 0);
  {
    size_t o = 0;
    for (int b = 0; b < s->B; ++b) {
      off0[b] = o;
      if (lens[b] <= 0) continue;
      o += lens[b];
      EE_TRY(grow_pages(s, b, want[b]));
    }
  }
  // Passes of up to `chunk` rows.  A pass takes one contiguous piece of every prompt that still has rows, in
  // sequence order, until it is full: a long prompt fills passes by itself, short prompts share one (the weights
  // cross HBM once per pass).  A sequence's next piece comes in a later pass, after its earlier rows are cached.
  const bool bf = s->m->bf16;
  int n_first = 0;                                       // first tokens on their way to out_host so far
  std::vector<int> end_seq(s->B), end_row(s->B), first_slot(s->B, 0);
  for (int ci = 0;; ++ci) {
    const int si = ci & 1;        // alternate upload slots so the host runs one pass ahead
    CallPlan p;
    p.m.assign(s->B, 0); p.p0.assign(s->B, 0);
    int room = s->chunk;
    for (int b = 0; b < s->B && room > 0; ++b) {
      if (lens[b] <= 0 || done[b] >= lens[b]) continue;
      p.m[b] = std::min(lens[b] - done[b], room); p.p0[b] = done[b];
      room -= p.m[b];
    }
    if (room == s->chunk) break;
    EE_TRY(build_meta(s, si, p, [&](int b, int r, int& tok, int&, int&) { tok = tokens[off0[b] + done[b] + r]; }));
    int n_end = 0;
    bool last_pass = true;
    for (int b = 0, row = 0; b < s->B; row += p.m[b], ++b) {
      if (done[b] + p.m[b] < lens[b]) last_pass = false;
      else if (p.m[b]) { end_seq[n_end] = b; end_row[n_end++] = row + p.m[b] - 1; }
    }
    // The rows that end a prompt decide its first committed token: the head runs over them alone.  What the introspection
    // calls report of a context build are the rows of its last 512-row piece; with logits kept these get a head as well.
    int r0 = (p.M - 1) / 512 * 512;
    const int piece_rows = p.M - r0, piece0 = r0;
    TailPlan tail;
    if (bf) {
      std::vector<int> keep(s->B, 0);
      for (int e = 0; e < n_end; ++e) keep[end_seq[e]] = 1;
      if (last_pass)
        for (int b = 0, first = 0; b < s->B; first += p.m[b], ++b)
          if (first + p.m[b] > piece0) keep[b] = std::max(keep[b], std::min(p.m[b], first + p.m[b] - piece0));
      plan_tail(s, si, p, keep, last_pass ? piece0 : -1, n_end, tail);
      if (tail.on) {
        r0 = last_pass ? tail.piece : 0;
        for (int e = 0; e < n_end; ++e) end_row[e] = tail.row0[end_seq[e]] + tail.p.m[end_seq[e]] - 1;
      }
    }
    std::copy(end_row.begin(), end_row.begin() + n_end, s->slot[si].h + s->o_row_src);     // (no rows are gathered here: the list of ends)
    EE_TRY(upload_meta(s, si));
    CallMeta mt = meta_ptrs(s, s->slot[si].d);
    PassSource from_tokens; from_tokens.tok = mt.row_tok;
    run_layers(s, 0, c.n_layers, p, mt, 0, from_tokens, PassSink(), tail.on ? &tail : nullptr);
    if (bf && n_end) {
      const bool kept_piece = s->debug_logits && last_pass;
      int early = 0;                                     // ends in front of that piece (all of them where it gets no head)
      while (early < n_end && !(kept_piece && end_row[early] >= r0)) ++early;
      if (early) {
        exit_head(s, early, s->n_levels, 0, mt.row_src);
        HIP_TRY(hipMemcpyAsync(s->out_host + n_first, s->vtok, early * sizeof(int), hipMemcpyDeviceToHost, s->st));
      }
      if (kept_piece) {
        exit_head(s, piece_rows, s->n_levels, r0);
        for (int e = early; e < n_end; ++e)
          HIP_TRY(hipMemcpyAsync(s->out_host + n_first + e, s->vtok + (end_row[e] - r0), sizeof(int), hipMemcpyDeviceToHost, s->st));
      }
      s->last_rows = piece_rows; s->last_row0 = r0;
    } else if (n_end) {
      exit_head(s, p.M, s->n_levels);
      for (int e = 0; e < n_end; ++e)
        HIP_TRY(hipMemcpyAsync(s->out_host + n_first + e, s->vtok + end_row[e], sizeof(int), hipMemcpyDeviceToHost, s->st));
    }
    for (int e = 0; e < n_end; ++e) first_slot[end_seq[e]] = n_first + e;
    n_first += n_end;
    for (int b = 0; b < s->B; ++b) done[b] += p.m[b];
  }
  size_t off = 0;
  EE_TRY(finish(s));
  off = 0;
  for (int b = 0; b < s->B; ++b) {
    if (lens[b] <= 0) continue;
    SeqState& q = s->seq[b];
    q.C.assign(tokens + off, tokens + off + lens[b]);
    q.C.push_back(s->out_host[first_slot[b]]);
    settle(s, q);
    q.started = true;
    first_token[b] = s->out_host[first_slot[b]];
    off += lens[b];
  }
  return EE_OK;
}

extern "C" int ee_prefill(ee_session* s, const int32_t* tokens, const int32_t* lens, int32_t* first_token) {
  if (!s || !tokens || !lens || !first_token) { ee_set_error("null argument"); return EE_ERR_ARG; }
  for (int b = 0; b < s->B; ++b)
    if (lens[b] < 1) { ee_set_error("prompt %d is empty", b); return EE_ERR_ARG; }
  return prefill_impl(s, tokens, lens, first_token);
}

extern "C" int ee_prefill_seq(ee_session* s, int seq, const int32_t* tokens, int len, int32_t* first_token) {
  if (!s || !tokens || !first_token || seq < 0 || seq >= s->B) { ee_set_error("bad argument"); return EE_ERR_ARG; }
  if (len < 1) { ee_set_error("prompt is empty"); return EE_ERR_ARG; }
  std::vector<int32_t> lens(s->B, 0), first(s->B, -1);
  lens[seq] = len;
  EE_TRY(prefill_impl(s, tokens, lens.data(), first.data()));
  *first_token = first[seq];
  return EE_OK;
}

// ---------------------------------------------------------------------------------------------
// C ABI: vanilla greedy generation at full depth (Sec. 3.1)
// ---------------------------------------------------------------------------------------------
extern "C" int ee_seq_release(ee_session* s, int seq) {
  if (!s || seq < 0 || seq >= s->B) { ee_set_error("bad sequence index"); return EE_ERR_ARG; }
  SeqState& q = s->seq[seq];
  while (!q.pages.empty()) { s->free_pages.push_back(q.pages.back()); q.pages.pop_back(); }
  q = SeqState();
  return EE_OK;
}

extern "C" int ee_free_pages(const ee_session* s) { return s ? (int)s->free_pages.size() : -1; }

extern "C" int ee_decode_ar(ee_session* s, int n, int32_t* out) {
  if (!s || !out) { ee_set_error("null argument"); return EE_ERR_ARG; }
  const ee_config& c = s->m->cfg;
  if (n < 1 || n > s->max_rows) { ee_set_error("%d tokens per call do not fit max_rows %d", n, s->max_rows); return EE_ERR_ARG; }
  std::vector<int> want(s->B, 0);
  int live = 0;
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    if (!q.started) continue;                         // an idle slot takes no part
    if (q.n_hd || !q.V.empty() || q.cut[s->n_levels] != (int)q.C.size()) { ee_set_error("sequence %d has unverified tokens", b); return EE_ERR_STATE; }
    want[b] = (int)q.C.size() + n;
    live++;
  }
  if (!live) { ee_set_error("no sequence has a context (call ee_prefill)"); return EE_ERR_STATE; }
  EE_TRY(check_capacity(s, want));
  reset_accounting(s);
  CallPlan p;
  p.m.assign(s->B, 0); p.p0.assign(s->B, 0);
  for (int b = 0; b < s->B; ++b) {
    if (!s->seq[b].started) continue;
    p.m[b] = 1;
    p.p0[b] = (int)s->seq[b].C.size() - 1;          // the pending token's position
    EE_TRY(grow_pages(s, b, want[b]));
  }
  EE_TRY(build_meta(s, 0, p, [&](int b, int, int& tok, int&, int&) { tok = s->seq[b].C.back(); }));
  EE_TRY(upload_meta(s, 0));
  CallMeta mt = meta_ptrs(s, s->slot[0].d);
  int* dh = s->out_host + 2 * s->B;   // (pinned: the kernels store the tokens there)
  for (int j = 0; j < n; ++j) {       // the next token stays on the device; positions advance through pos_add
    PassSource from_tokens; from_tokens.tok = j == 0 ? mt.row_tok : s->tok_next;
    run_layers(s, 0, c.n_layers, p, mt, j, from_tokens);
    exit_head(s, p.M, s->n_levels, 0, nullptr, TakeToken{s->tok_next, dh, mt.row_seq, s->max_rows, j});
  }
  EE_TRY(finish(s));
  for (int b = 0; b < s->B; ++b) {
    SeqState& q = s->seq[b];
    if (!p.m[b]) { for (int j = 0; j < n; ++j) out[b * n + j] = -1; continue; }
    for (int j = 0; j < n; ++j) { out[b * n + j] = dh[b * s->max_rows + j]; q.C.push_back(dh[b * s->max_rows + j]); }
    settle(s, q);
  }
  return EE_OK;
}

// ---------------------------------------------------------------------------------------------
// C ABI: drafting at exit L_d
// ---------------------------------------------------------------------------------------------
static int draft_precheck(ee_session* s, int k, int rows) {
  if (k < 1 || rows > s->max_rows) { ee_set_error("draft length %d does not fit max_rows %d", k, s->max_rows); return EE_ERR_ARG; }
  std::vector<int> want(s->B, 0);
  int live = 0;
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    if (!q.started) continue;                         // an idle slot takes no part
    live++;
    if (q.n_hd) { ee_set_error("sequence %d already has an unverified draft block", b); return EE_ERR_STATE; }
    int nT = (int)(q.C.size() + q.V.size());
    if ((int)q.V.size() + rows + 1 > s->max_rows) { ee_set_error("tentative buffer of sequence %d would overflow max_rows", b); return EE_ERR_CAPACITY; }
    want[b] = nT - 1 + rows + 1;   // one spare position for the pending token's later catch-up
  }
  if (!live) { ee_set_error("no sequence has a context (call ee_prefill)"); return EE_ERR_STATE; }
  return check_capacity(s, want);
}

static int check_uniforms(const float* u, size_t n) {
  for (size_t i = 0; i < n; ++i)
    if (!(u[i] >= 0.0f && u[i] < 1.0f)) { ee_set_error("uniform numbers must lie in [0, 1)"); return EE_ERR_ARG; }
  return EE_OK;
}
// The uniform numbers of a call travel in its metadata block: acc [B][max_rows] (stride numbers of each participating
// sequence), then one more per sequence (res; null: none).
static void put_uniforms(ee_session* s, const CallPlan& p, const float* acc, int stride, const float* res) {
  float* u = (float*)(s->slot[0].h + s->o_u);
  for (int b = 0; b < s->B; ++b) {
    if (!p.m[b]) continue;
    std::copy(acc + (size_t)b * stride, acc + (size_t)b * stride + std::min(stride, s->max_rows), u + (size_t)b * s->max_rows);
    if (res) u[(size_t)s->B * s->max_rows + b] = res[b];
  }
}
static const float* uniforms(const ee_session* s) { return (const float*)(s->slot[0].d + s->o_u); }

// u == null: arg max of p_{L_d} (Alg. 2); otherwise token j of sequence b is drawn from p_{L_d} with u[b*k + j] (App. G)
static int draft_impl(ee_session* s, int k, int32_t* draft, const float* u) {
  if (!s || !draft) { ee_set_error("null argument"); return EE_ERR_ARG; }
  const ee_config& c = s->m->cfg;
  const int rows = k + (c.bonus_inter ? 1 : 0);
  if (u && !s->Pd) { ee_set_error("sampling buffers are not attached (ee_sampling_attach)"); return EE_ERR_STATE; }
  EE_TRY(draft_precheck(s, k, rows));
  if (u)
    for (int b = 0; b < s->B; ++b)      // an idle slot's numbers are neither read nor checked
      if (s->seq[b].started) EE_TRY(check_uniforms(u + (size_t)b * k, k));
  reset_accounting(s);
  s->need_logits = u != nullptr;
  CallPlan p;
  p.m.assign(s->B, 0); p.p0.assign(s->B, 0);
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    if (!q.started) continue;
    p.m[b] = 1;
    p.p0[b] = (int)(q.C.size() + q.V.size()) - 1;
    EE_TRY(grow_pages(s, b, p.p0[b] + rows + 1));
  }
  EE_TRY(build_meta(s, 0, p, [&](int b, int, int& tok, int&, int& dst) {
    const SeqState& q = s->seq[b];
    tok = q.V.empty() ? q.C.back() : q.V.back();
    dst = b * s->max_rows;
  }, u ? s->B * s->max_rows : 0));
  if (u) put_uniforms(s, p, u, k, nullptr);
  EE_TRY(upload_meta(s, 0));
  CallMeta mt = meta_ptrs(s, s->slot[0].d);
  int* dh = s->out_host + 2 * s->B;   // (pinned: the kernels store the tokens there)
  for (int j = 0; j < rows; ++j) {
    PassSource from_tokens; from_tokens.tok = j == 0 ? mt.row_tok : s->tok_next;
    PassSink keep; keep.rows = s->Hd; keep.row_idx = mt.row_dst; keep.add = j;
    run_layers(s, 0, c.exit_draft, p, mt, j, from_tokens, keep);
    if (j < k) {
      exit_head(s, p.M, 0, 0, nullptr, u ? TakeToken() : TakeToken{s->tok_next, dh, mt.row_seq, s->max_rows, j});
      if (u)      // p_{L_d} of this position into the draft-distribution store, then the draw
        KF(KF_MISC, k_softmax_draw(s->st, s->LOGITS, s->Pd, mt.row_dst, j, p.M, c.vocab, uniforms(s), s->max_rows, j, mt.row_seq, s->tok_next,
                                   dh, s->max_rows));
    }
  }
  s->need_logits = false;
  EE_TRY(finish(s));
  for (int b = 0; b < s->B; ++b) {
    SeqState& q = s->seq[b];
    if (!p.m[b]) { for (int j = 0; j < k; ++j) draft[b * k + j] = -1; continue; }
    q.S.assign(dh + b * s->max_rows, dh + b * s->max_rows + k);
    q.n_hd = rows;
    q.sampled = u != nullptr;
    q.len[0] = p.p0[b] + rows;
    for (int j = 0; j < k; ++j) draft[b * k + j] = q.S[j];
  }
  return EE_OK;
}

extern "C" int ee_draft(ee_session* s, int k, int32_t* draft) { return draft_impl(s, k, draft, nullptr); }

extern "C" int ee_draft_sample(ee_session* s, int k, const float* u, int32_t* draft) {
  if (!u) { ee_set_error("null argument"); return EE_ERR_ARG; }
  return draft_impl(s, k, draft, u);
}

extern "C" int ee_draft_inject(ee_session* s, int k, const int32_t* draft) {
  if (!s || !draft) { ee_set_error("null argument"); return EE_ERR_ARG; }
  const ee_config& c = s->m->cfg;
  const int rows = k + (c.bonus_inter ? 1 : 0);
  EE_TRY(draft_precheck(s, k, rows));
  for (int i = 0; i < s->B * k; ++i)
    if (s->seq[i / k].started && (draft[i] < 0 || draft[i] >= c.vocab)) { ee_set_error("draft token out of range"); return EE_ERR_ARG; }
  reset_accounting(s);
  CallPlan p;
  p.m.assign(s->B, 0); p.p0.assign(s->B, 0);
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    if (!q.started) continue;                         // an idle slot's entries of `draft` are ignored
    p.m[b] = rows;
    p.p0[b] = (int)(q.C.size() + q.V.size()) - 1;
    EE_TRY(grow_pages(s, b, p.p0[b] + rows + 1));
  }
  EE_TRY(build_meta(s, 0, p, [&](int b, int r, int& tok, int&, int& dst) {
    const SeqState& q = s->seq[b];
    tok = r == 0 ? (q.V.empty() ? q.C.back() : q.V.back()) : draft[b * k + r - 1];
    dst = b * s->max_rows + r;
  }));
  EE_TRY(upload_meta(s, 0));
  CallMeta mt = meta_ptrs(s, s->slot[0].d);
  PassSource from_tokens; from_tokens.tok = mt.row_tok;
  PassSink keep; keep.rows = s->Hd; keep.row_idx = mt.row_dst;
  run_layers(s, 0, c.exit_draft, p, mt, 0, from_tokens, keep);
  HIP_TRY(hipGetLastError());
  for (int b = 0; b < s->B; ++b) {
    SeqState& q = s->seq[b];
    if (!p.m[b]) continue;
    q.S.assign(draft + b * k, draft + b * k + k);
    q.n_hd = rows;
    q.sampled = false;
    q.len[0] = p.p0[b] + rows;
  }
  return EE_OK;
}

// ---------------------------------------------------------------------------------------------
// Scratch of one call in the library's own static device array, for callers that cannot allocate
// ---------------------------------------------------------------------------------------------
// What a verify call needs beyond its inputs, outputs and the session's state -- the attention's split partials, the
// exit head's (max, arg max) tile partials, the deferred-RMSNorm partial sums and factors, the K-share partials of
// the row-tiled GEMM -- normally sits in the caller's session arena.  ee_verify_intermediate_static places it in
// this array instead.  Every GPU holds its own copy of the array at its own address, found once per device with
// hipGetSymbolAddress; the array's name itself is only a host-side stand-in and never goes to a kernel.
#define EE_STATIC_SCRATCH_BYTES ((size_t)32 << 20)
#define EE_STATIC_MAX_DEVICES 64
static __device__ __align__(256) unsigned char scratch[EE_STATIC_SCRATCH_BYTES];
static void* g_scratch_ptr[EE_STATIC_MAX_DEVICES] = {nullptr};
static std::mutex g_scratch_mutex;

static int static_scratch_base(char** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= EE_STATIC_MAX_DEVICES) { ee_set_error("device %d outside the static scratch table", dev); return EE_ERR_HIP; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) { ee_set_error("static scratch has no device address"); return EE_ERR_HIP; }
    g_scratch_ptr[dev] = ptr;
  }
  *out = (char*)g_scratch_ptr[dev];
  return EE_OK;
}

// the session's scratch pointers, swapped for the length of one call and put back whatever happens
struct ScratchSwap {
  ee_session* s;
  float *part_o, *part_ml, *pmax, *ssq, *gemm_part, *inv_rms;
  int* pidx;
  int ssq_stride, inv_cap;
  explicit ScratchSwap(ee_session* s_) : s(s_), part_o(s_->part_o), part_ml(s_->part_ml), pmax(s_->pmax), ssq(s_->ssq),
                                         gemm_part(s_->gemm_part), inv_rms(s_->inv_rms), pidx(s_->pidx),
                                         ssq_stride(s_->ssq_stride), inv_cap(s_->inv_cap) {}
  ~ScratchSwap() {
    s->part_o = part_o; s->part_ml = part_ml; s->pmax = pmax; s->ssq = ssq; s->gemm_part = gemm_part; s->inv_rms = inv_rms;
    s->pidx = pidx; s->ssq_stride = ssq_stride; s->inv_cap = inv_cap;
  }
};

// Lay the scratch of the call with plan p (pass over layers [l0, l1), then the shared exit head) out in the static
// array and point the session at it.  The split plan is the one the session arena would have given (its capacity
// only enters as a number), so the call computes exactly what ee_verify_intermediate computes.
static int place_scratch_static(ee_session* s, const CallPlan& p) {
  const ee_model* m = s->m;
  const ee_config& c = m->cfg;
  if (!m->bf16) return EE_OK;                       // the fp32 kernels use no scratch
  char* base = nullptr;
  EE_TRY(static_scratch_base(&base));
  AttnScratch scr;
  const int nsplit = attention_plan(s, p, 0, scr).nsplit;
  Carver cv{base};
  const size_t slots = (size_t)p.total_qt * c.n_kv_heads * nsplit;
  float* part_o = cv.take<float>(slots * 16 * c.head_dim);
  float* part_ml = cv.take<float>(slots * 32);
  const size_t pstride = (size_t)ceil_div(p.M, 16) * 16;
  float* pmax = cv.take<float>((size_t)m->head.ntiles() * pstride);
  int* pidx = cv.take<int>((size_t)m->head.ntiles() * pstride);
  const int stride = p.M <= 64 ? 64 : ceil_div(p.M, 512) * 512;      // whole GEMM passes of this call's rows
  float* ssq = cv.take<float>((size_t)ceil_div(c.d_model, 16) * stride);
  float* inv_rms = cv.take<float>(512);
  size_t gp = 0;                                    // room for the K shares of the projections that the row-tiled GEMM serves
  for (const MatLoc* ml : {&m->L[0].qkv, &m->L[0].o, &m->L[0].gu, &m->L[0].down, &m->head, &m->auxA[0], &m->auxB[0]})
    if (ml->Np > 0 && !bf16_takes_strips(ml->ntiles(), ml->ktiles(), p.M)) gp = std::max(gp, bf16_gemm_rows_scratch_floats(ml->ntiles(), ml->ktiles()));
  float* gemm_part = cv.take<float>(gp);
  if (cv.cur > EE_STATIC_SCRATCH_BYTES) {
    ee_set_error("this call needs %zu bytes of scratch, the static array holds %zu: use ee_verify_intermediate", cv.cur,
                 (size_t)EE_STATIC_SCRATCH_BYTES);
    return EE_ERR_CAPACITY;
  }
  s->part_o = part_o; s->part_ml = part_ml; s->pmax = pmax; s->pidx = pidx; s->ssq = ssq; s->inv_rms = inv_rms;
  s->gemm_part = gemm_part; s->ssq_stride = stride; s->inv_cap = 512;
  return EE_OK;
}

// ---------------------------------------------------------------------------------------------
// C ABI: intermediate verification at exit L_i
// ---------------------------------------------------------------------------------------------
// u_acc == null: LeadingSubstringVerify on arg max tokens (Alg. 2); otherwise the acceptance rule of App. G with the
// uniform numbers u_acc [batch, u_stride] (one per draft token) and u_res [batch] (the replacement / next-token draw)
static int verify_intermediate_impl(ee_session* s, int32_t* n_accept, int32_t* next_token, const float* u_acc, int u_stride,
                                    const float* u_res, bool static_scratch = false) {
  if (!s || !n_accept || !next_token) { ee_set_error("null argument"); return EE_ERR_ARG; }
  const ee_config& c = s->m->cfg;
  const bool rs = u_acc != nullptr;
  ScratchSwap restore(s);
  CallPlan p;
  p.m.assign(s->B, 0); p.p0.assign(s->B, 0);
  int any = 0;
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    if (!q.n_hd) continue;
    if (rs && (!q.sampled || q.n_pi != (int)q.V.size())) {
      ee_set_error("sequence %d: the pending block or the tentative tokens were not produced by the sampling calls", b);
      return EE_ERR_STATE;
    }
    p.m[b] = q.n_hd; p.p0[b] = (int)(q.C.size() + q.V.size()) - 1;
    any++;
  }
  if (!any) { ee_set_error("no draft block is pending"); return EE_ERR_STATE; }
  if (rs) {
    if (!s->Pd) { ee_set_error("sampling buffers are not attached (ee_sampling_attach)"); return EE_ERR_STATE; }
    if (u_stride < 1 || u_stride > s->max_rows) { ee_set_error("bad stride of the uniform numbers"); return EE_ERR_ARG; }
    for (int b = 0; b < s->B; ++b) {                         // idle sequences' numbers are neither read nor checked
      if (!p.m[b]) continue;
      if ((int)s->seq[b].S.size() > u_stride) { ee_set_error("sequence %d: %d draft tokens need as many uniform numbers (u_stride %d)", b, (int)s->seq[b].S.size(), u_stride); return EE_ERR_ARG; }
      EE_TRY(check_uniforms(u_acc + (size_t)b * u_stride, u_stride));
      EE_TRY(check_uniforms(u_res + b, 1));
    }
  }
  reset_accounting(s);
  EE_TRY(build_meta(s, 0, p, [&](int b, int r, int&, int& src, int& dst) {
    src = b * s->max_rows + r;                               // H_d row
    dst = b * s->max_rows + (int)s->seq[b].V.size() + r;     // H_i row
  }, rs ? s->B * s->max_rows + s->B : 0));
  if (rs) put_uniforms(s, p, u_acc, u_stride, u_res);
  if (static_scratch) EE_TRY(place_scratch_static(s, p));
  int* h = s->slot[0].h;
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    if (!p.m[b]) continue;
    h[s->o_n_cand + b] = (int)q.S.size();
    for (size_t j = 0; j < q.S.size(); ++j) h[s->o_cand + (size_t)b * s->cand_stride + j] = q.S[j];
  }
  EE_TRY(upload_meta(s, 0));
  CallMeta mt = meta_ptrs(s, s->slot[0].d);
  PassSource kept; kept.rows = s->Hd; kept.row_idx = mt.row_src;       // a1: consume buffered H_d
  PassSink keep; keep.rows = s->Hi; keep.row_idx = mt.row_dst;          // keep L_i hidden rows
  run_layers(s, c.exit_draft, c.exit_inter, p, mt, 0, kept, keep);
  s->need_logits = rs;
  exit_head(s, p.M, 1);
  s->need_logits = false;
  if (rs) {
    // p_{L_i} in place, and kept for the rows that may stay
    KF(KF_MISC, k_softmax_rows(s->st, s->LOGITS, s->LOGITS, nullptr, 0, s->Pi, mt.row_dst, p.M, c.vocab));
    KF(KF_ACCEPT, k_rs_accept(s->st, s->LOGITS, s->Pd, s->max_rows, c.vocab, mt, s->cand_stride, s->B, uniforms(s), s->max_rows, s->out_dev));
    KF(KF_ACCEPT, k_rs_draw(s->st, s->LOGITS, s->Pd, s->max_rows, c.vocab, mt, s->B, s->out_dev, uniforms(s) + (size_t)s->B * s->max_rows,
                            s->out_host));
  } else {
    KF(KF_ACCEPT, k_accept(s->st, s->vtok, mt, s->cand_stride, s->B, s->out_host, s->out_host + s->B));
  }
  EE_TRY(finish(s));
  for (int b = 0; b < s->B; ++b) {
    SeqState& q = s->seq[b];
    n_accept[b] = s->out_host[b]; next_token[b] = s->out_host[s->B + b];
    if (!p.m[b]) continue;
    const int a = n_accept[b];
    q.V.insert(q.V.end(), q.S.begin(), q.S.begin() + a);
    int keep = a;
    if (a < p.m[b]) { q.V.push_back(next_token[b]); keep = a + 1; }
    q.len[0] = q.len[1] = p.p0[b] + keep;                    // prune rejected rows (lengths only)
    q.n_hd = 0; q.S.clear(); q.sampled = false;
    if (rs) q.n_pi = (int)q.V.size();
    trim_pages(s, b);
  }
  return EE_OK;
}

extern "C" int ee_verify_intermediate(ee_session* s, int32_t* n_accept, int32_t* next_token) {
  return verify_intermediate_impl(s, n_accept, next_token, nullptr, 0, nullptr);
}

extern "C" int ee_verify_intermediate_static(ee_session* s, int32_t* n_accept, int32_t* next_token) {
  if (s && s->time_kernels) { ee_set_error("kernel timing creates events: switch it off for the call that allocates nothing"); return EE_ERR_STATE; }
  return verify_intermediate_impl(s, n_accept, next_token, nullptr, 0, nullptr, true);
}

extern "C" int ee_verify_intermediate_rs(ee_session* s, const float* u_acc, int u_stride, const float* u_res, int32_t* n_accept,
                                         int32_t* next_token) {
  if (!u_acc || !u_res) { ee_set_error("null argument"); return EE_ERR_ARG; }
  return verify_intermediate_impl(s, n_accept, next_token, u_acc, u_stride, u_res);
}

// ---------------------------------------------------------------------------------------------
// C ABI: verification at the levels above L_i -- full verification at L_f (Alg. 2) and, with further
// verifier exits, the levels in between (the hierarchy of the paper's Future Work section)
// ---------------------------------------------------------------------------------------------
static float* level_rows(const ee_session* s, int j) { return j == 0 ? s->Hd : (j == 1 ? s->Hi : s->Hup[j - 2]); }
// stored distributions of the tokens in level j's buffer (0: the draft block's)
static float* level_dist(const ee_session* s, int j) { return j == 0 ? s->Pd : (j == 1 ? s->Pi : s->Pup[j - 2]); }

// Level j (2 <= j <= n) takes the buffer of level j-1 as its draft: V for j = 2, else the tail C[cut[j]..) (every
// buffer below it must be empty).  The buffered rows of exit j-1 plus, in bonus mode, one row for the buffer's
// last token (through the groups below first) run through layer group j; LeadingSubstringVerify keeps the
// matching prefix and exit j's own next token.  What is kept joins level j's buffer (the committed tokens at
// the last level); the KV lengths of the groups up to j are pruned to it.
static int verify_upper_impl(ee_session* s, int level, const uint8_t* active, int32_t* n_accept, int32_t* next_token,
                             int32_t* committed, int32_t* n_committed, const float* u_acc, int u_stride, const float* u_res) {
  if (!s || !n_accept || !next_token || !committed || !n_committed) { ee_set_error("null argument"); return EE_ERR_ARG; }
  const ee_config& c = s->m->cfg;
  const int n = s->n_levels, j = level;
  if (j < 2 || j > n) { ee_set_error("level must be 2..%d", n); return EE_ERR_ARG; }
  const std::vector<int>& ex = s->m->exits;
  const int bonus = c.bonus_full ? 1 : 0;
  const bool rs = u_acc != nullptr;
  std::vector<int> act(s->B, 0), m_src(s->B, 0), base(s->B, 0);
  int any = 0;
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    if (active && !active[b]) continue;
    // base: tokens already past level j; m_src: tokens of the buffer below it
    base[b] = j == 2 ? (int)q.C.size() : q.cut[j];
    m_src[b] = j == 2 ? (int)q.V.size() : (int)q.C.size() - q.cut[j];
    if (!q.started || m_src[b] == 0) continue;
    if (q.n_hd) { ee_set_error("sequence %d still has an unverified draft block", b); return EE_ERR_STATE; }
    if (j > 2 && (!q.V.empty() || q.cut[j - 1] != (int)q.C.size())) {
      ee_set_error("sequence %d: the buffers below level %d must be verified first", b, j - 1); return EE_ERR_STATE;
    }
    if (rs && (j == 2 ? q.n_pi : q.n_pu[j - 3]) != m_src[b]) {
      ee_set_error("sequence %d: the tokens waiting below level %d were not produced by the sampling calls", b, j);
      return EE_ERR_STATE;
    }
    // level j's buffer is level j+1's draft: its rows sit in a [max_rows] slab per sequence together with the
    // catch-up row that level j+1 appends behind them, so it may hold max_rows - bonus tokens at most
    if (j < n && (q.cut[j] - q.cut[j + 1]) + m_src[b] + bonus > s->max_rows - bonus) {
      ee_set_error("level %d buffer of sequence %d would exceed %d tokens", j, b, s->max_rows - bonus); return EE_ERR_CAPACITY;
    }
    if (m_src[b] + bonus > s->max_rows) {      // (cannot happen given the bound above and the one on V in the draft calls)
      ee_set_error("sequence %d: %d rows do not fit max_rows", b, m_src[b] + bonus); return EE_ERR_CAPACITY;
    }
    act[b] = 1; any++;
  }
  if (!any) { ee_set_error("no sequence has tentative tokens to verify"); return EE_ERR_STATE; }
  if (rs) {
    if (!s->Pi) { ee_set_error("sampling buffers are not attached (ee_sampling_attach)"); return EE_ERR_STATE; }
    if (u_stride < 1 || u_stride > s->max_rows) { ee_set_error("bad stride of the uniform numbers"); return EE_ERR_ARG; }
    for (int b = 0; b < s->B; ++b) {                         // idle sequences' numbers are neither read nor checked
      if (!act[b]) continue;
      if (m_src[b] > u_stride) { ee_set_error("sequence %d: %d tentative tokens need as many uniform numbers (u_stride %d)", b, m_src[b], u_stride); return EE_ERR_ARG; }
      EE_TRY(check_uniforms(u_acc + (size_t)b * u_stride, u_stride));
      EE_TRY(check_uniforms(u_res + b, 1));
    }
  }
  auto src_tok = [&](int b, int i) { const SeqState& q = s->seq[b]; return j == 2 ? q.V[i] : q.C[q.cut[j] + i]; };
  float* rows_below = level_rows(s, j - 1);
  reset_accounting(s);
  if (bonus) {
    // the buffer's last token owns no hidden state yet: one row per sequence through the groups below level j
    CallPlan p;
    p.m.assign(s->B, 0); p.p0.assign(s->B, 0);
    for (int b = 0; b < s->B; ++b) {
      if (!act[b]) continue;
      p.m[b] = 1; p.p0[b] = base[b] + m_src[b] - 1;
      EE_TRY(grow_pages(s, b, p.p0[b] + 1));
    }
    EE_TRY(build_meta(s, 1, p, [&](int b, int, int& tok, int&, int& dst) {
      tok = src_tok(b, m_src[b] - 1);
      dst = b * s->max_rows + m_src[b];
    }));
    EE_TRY(upload_meta(s, 1));
    CallMeta mt = meta_ptrs(s, s->slot[1].d);
    PassSource from_tokens; from_tokens.tok = mt.row_tok;
    PassSink keep; keep.rows = rows_below; keep.row_idx = mt.row_dst;
    run_layers(s, 0, ex[j - 1], p, mt, 0, from_tokens, keep);
  }
  CallPlan p;
  p.m.assign(s->B, 0); p.p0.assign(s->B, 0);
  for (int b = 0; b < s->B; ++b) {
    if (!act[b]) continue;
    p.m[b] = m_src[b] + bonus; p.p0[b] = base[b] - 1;
  }
  EE_TRY(build_meta(s, 0, p, [&](int b, int r, int&, int& src, int& dst) {
    src = b * s->max_rows + r;
    dst = b * s->max_rows + (j < n ? s->seq[b].cut[j] - s->seq[b].cut[j + 1] : 0) + r;     // row of level j's own buffer
  }, rs ? s->B * s->max_rows + s->B : 0));
  if (rs) put_uniforms(s, p, u_acc, u_stride, u_res);
  int* h = s->slot[0].h;
  for (int b = 0; b < s->B; ++b) {
    if (!act[b]) continue;
    h[s->o_n_cand + b] = m_src[b];
    for (int i = 0; i < m_src[b]; ++i) h[s->o_cand + (size_t)b * s->cand_stride + i] = src_tok(b, i);
  }
  EE_TRY(upload_meta(s, 0));
  CallMeta mt = meta_ptrs(s, s->slot[0].d);
  PassSource kept; kept.rows = rows_below; kept.row_idx = mt.row_src;  // consume the buffered rows
  PassSink keep;
  if (j < n) { keep.rows = level_rows(s, j); keep.row_idx = mt.row_dst; }   // keep exit j's rows
  run_layers(s, ex[j - 1], ex[j], p, mt, 0, kept, keep);
  s->need_logits = rs;
  exit_head(s, p.M, j);
  s->need_logits = false;
  if (rs) {      // a further stage of App. G: the buffer below, distributed as exit j-1's p, is the draft; exit j's p the target
    const float* q_below = level_dist(s, j - 1);
    // exit j's distributions in place and, below L_f, kept for the rows that may stay: the law of the tokens that wait for exit j+1
    KF(KF_MISC, k_softmax_rows(s->st, s->LOGITS, s->LOGITS, nullptr, 0, j < n ? level_dist(s, j) : nullptr, mt.row_dst, p.M, c.vocab));
    KF(KF_ACCEPT, k_rs_accept(s->st, s->LOGITS, q_below, s->max_rows, c.vocab, mt, s->cand_stride, s->B, uniforms(s), s->max_rows, s->out_dev));
    KF(KF_ACCEPT, k_rs_draw(s->st, s->LOGITS, q_below, s->max_rows, c.vocab, mt, s->B, s->out_dev, uniforms(s) + (size_t)s->B * s->max_rows,
                            s->out_host));
  } else {
    KF(KF_ACCEPT, k_accept(s->st, s->vtok, mt, s->cand_stride, s->B, s->out_host, s->out_host + s->B));
  }
  EE_TRY(finish(s));
  for (int b = 0; b < s->B; ++b) {
    SeqState& q = s->seq[b];
    n_accept[b] = s->out_host[b]; next_token[b] = s->out_host[s->B + b];
    n_committed[b] = 0;
    if (!act[b]) continue;
    const int f = n_accept[b];
    int32_t* out = committed + (size_t)b * (s->max_rows + 1);
    int cnt = 0;
    for (int i = 0; i < f; ++i) out[cnt++] = src_tok(b, i);
    if (f < p.m[b]) out[cnt++] = next_token[b];
    n_committed[b] = cnt;
    if (j > 2) q.C.resize(q.cut[j]);
    const int held = j < n ? q.cut[j] - q.cut[j + 1] : 0;      // tokens level j's buffer held before this call
    q.C.insert(q.C.end(), out, out + cnt);
    q.V.clear(); q.n_pi = 0;
    for (int i = 2; i < j; ++i) q.n_pu[i - 2] = 0;
    if (j < n) q.n_pu[j - 2] = (rs && q.n_pu[j - 2] == held) ? held + cnt : -1;   // -1: holds tokens without a stored law
    for (int g = 2; g <= j; ++g) q.cut[g] = (int)q.C.size();
    for (int g = 0; g <= j; ++g) q.len[g] = (int)q.C.size() - 1;
    trim_pages(s, b);
  }
  return EE_OK;
}

extern "C" int ee_verify_full(ee_session* s, const uint8_t* active, int32_t* n_accept, int32_t* next_token,
                              int32_t* committed, int32_t* n_committed) {
  if (!s) { ee_set_error("null argument"); return EE_ERR_ARG; }
  return verify_upper_impl(s, s->n_levels, active, n_accept, next_token, committed, n_committed, nullptr, 0, nullptr);
}

extern "C" int ee_verify_level(ee_session* s, int level, const uint8_t* active, int32_t* n_accept, int32_t* next_token,
                               int32_t* moved, int32_t* n_moved) {
  return verify_upper_impl(s, level, active, n_accept, next_token, moved, n_moved, nullptr, 0, nullptr);
}

extern "C" int ee_verify_level_rs(ee_session* s, int level, const uint8_t* active, const float* u_acc, int u_stride, const float* u_res,
                                  int32_t* n_accept, int32_t* next_token, int32_t* moved, int32_t* n_moved) {
  if (!s || !u_acc || !u_res) { ee_set_error("null argument"); return EE_ERR_ARG; }
  return verify_upper_impl(s, level, active, n_accept, next_token, moved, n_moved, u_acc, u_stride, u_res);
}

extern "C" int ee_n_levels(const ee_session* s) { return s ? s->n_levels : -1; }

extern "C" int ee_verify_full_rs(ee_session* s, const uint8_t* active, const float* u_acc, int u_stride, const float* u_res,
                                 int32_t* n_accept, int32_t* next_token, int32_t* committed, int32_t* n_committed) {
  if (!s || !u_acc || !u_res) { ee_set_error("null argument"); return EE_ERR_ARG; }
  return verify_upper_impl(s, s->n_levels, active, n_accept, next_token, committed, n_committed, u_acc, u_stride, u_res);
}

// ---------------------------------------------------------------------------------------------
// C ABI: buffers of the rejection-sampling acceptance (caller-owned, like the session arena)
// ---------------------------------------------------------------------------------------------
static size_t sampling_floats(const ee_session* s) {
  const size_t rows = (size_t)s->B * s->max_rows;
  return (size_t)s->n_levels * rows * s->m->cfg.vocab + 64;     // one store per level below L_f
}
extern "C" size_t ee_sampling_bytes(const ee_session* s) { return s ? sampling_floats(s) * sizeof(float) : 0; }

extern "C" int ee_sampling_attach(ee_session* s, void* dev_arena, size_t arena_bytes) {
  if (!s || !dev_arena || ((uintptr_t)dev_arena & 255)) { ee_set_error("arena must be non-null and 256-byte aligned"); return EE_ERR_ARG; }
  if (arena_bytes < sampling_floats(s) * sizeof(float)) { ee_set_error("sampling arena too small"); return EE_ERR_ARG; }
  const size_t rows = (size_t)s->B * s->max_rows;
  float* f = (float*)dev_arena;
  const size_t store = rows * s->m->cfg.vocab;
  s->Pd = f; s->Pi = f + store;
  for (int j = 2; j < s->n_levels; ++j) s->Pup[j - 2] = f + (size_t)j * store;
  return EE_OK;
}

// ---------------------------------------------------------------------------------------------
// C ABI: rollback
// ---------------------------------------------------------------------------------------------
extern "C" int kv_rollback(ee_session* s, int seq, int group_mask, int new_len) {
  if (!s || seq < 0 || seq >= s->B) { ee_set_error("bad sequence index"); return EE_ERR_ARG; }
  SeqState& q = s->seq[seq];
  if (!q.started) { ee_set_error("sequence %d has no context", seq); return EE_ERR_STATE; }
  const int n = s->n_levels;
  const int m12 = group_mask & 3;
  if (m12 != 0 && m12 != 3) { ee_set_error("G1 and G2 roll back together"); return EE_ERR_ARG; }
  if (group_mask & ~((1 << (n + 1)) - 1)) { ee_set_error("bad group mask"); return EE_ERR_ARG; }
  if (m12 == 0) {
    for (int g = 2; g <= n; ++g)
      if ((group_mask & (1 << g)) && new_len != q.len[g]) { ee_set_error("the groups above G2 cannot roll back alone"); return EE_ERR_ARG; }
    q.n_hd = 0; q.S.clear(); q.sampled = false; q.len[0] = q.len[1];
    trim_pages(s, seq);
    return EE_OK;
  }
  if (new_len < 0 || new_len > q.len[1]) { ee_set_error("rollback can only shrink (len %d -> %d)", q.len[1], new_len); return EE_ERR_ARG; }
  const int nT = new_len + 1;
  if (nT <= (int)q.C.size()) {
    for (int g = 2; g <= n; ++g)
      if (new_len < q.len[g] && !(group_mask & (1 << g))) {
        ee_set_error("cut reaches tokens that group %d has seen: it must roll back too", g + 1); return EE_ERR_ARG;
      }
    q.C.resize(nT); q.V.clear();
    for (int g = 2; g <= n; ++g) { q.len[g] = std::min(q.len[g], new_len); q.cut[g] = std::min(q.cut[g], nT); }
  } else {
    q.V.resize(nT - q.C.size());
  }
  q.n_pi = std::min(q.n_pi, (int)q.V.size());
  for (int g = 2; g < n; ++g) q.n_pu[g - 2] = std::min(q.n_pu[g - 2], q.cut[g] - q.cut[g + 1]);
  q.n_hd = 0; q.S.clear(); q.sampled = false;
  q.len[0] = q.len[1] = new_len;
  trim_pages(s, seq);
  return EE_OK;
}

// ---------------------------------------------------------------------------------------------
// C ABI: introspection
// ---------------------------------------------------------------------------------------------
extern "C" int ee_get_lengths(const ee_session* s, int32_t* out) {
  if (!s || !out) { ee_set_error("null argument"); return EE_ERR_ARG; }
  const int G = s->n_levels + 1;
  for (int b = 0; b < s->B; ++b) for (int g = 0; g < G; ++g) out[b * G + g] = s->seq[b].len[g];
  return EE_OK;
}
extern "C" int ee_get_counts(const ee_session* s, int32_t* nc, int32_t* nv) {
  if (!s || !nc || !nv) { ee_set_error("null argument"); return EE_ERR_ARG; }
  for (int b = 0; b < s->B; ++b) {
    const SeqState& q = s->seq[b];
    nc[b] = q.cut[s->n_levels]; nv[b] = (int)(q.C.size() + q.V.size()) - nc[b];
  }
  return EE_OK;
}
extern "C" int ee_get_tokens(const ee_session* s, int seq, int32_t* out, int cap, int32_t* n_out) {
  if (!s || !out || !n_out || seq < 0 || seq >= s->B) { ee_set_error("bad argument"); return EE_ERR_ARG; }
  const SeqState& q = s->seq[seq];
  int n = (int)(q.C.size() + q.V.size());
  if (n > cap) { ee_set_error("buffer too small: %d tokens", n); return EE_ERR_CAPACITY; }
  std::copy(q.C.begin(), q.C.end(), out);
  std::copy(q.V.begin(), q.V.end(), out + q.C.size());
  *n_out = n;
  return EE_OK;
}
extern "C" int ee_debug_enable_logits(ee_session* s, int on) {
  if (!s) { ee_set_error("null session"); return EE_ERR_ARG; }
  s->debug_logits = on != 0;
  return EE_OK;
}
extern "C" int ee_debug_last_logits(ee_session* s, float* host_out, int max_rows, int32_t* n_rows) {
  if (!s || !host_out || !n_rows) { ee_set_error("null argument"); return EE_ERR_ARG; }
  if (s->m->bf16 && !s->debug_logits) { ee_set_error("logits were not kept: call ee_debug_enable_logits first"); return EE_ERR_STATE; }
  int n = std::min(max_rows, s->last_rows);
  HIP_TRY(hipMemcpy(host_out, s->LOGITS, (size_t)n * s->m->cfg.vocab * sizeof(float), hipMemcpyDeviceToHost));
  *n_rows = n;
  return EE_OK;
}
extern "C" int ee_debug_last_hidden(ee_session* s, float* host_out, int max_rows, int32_t* n_rows) {
  if (!s || !host_out || !n_rows) { ee_set_error("null argument"); return EE_ERR_ARG; }
  int n = std::min(max_rows, s->last_rows);
  HIP_TRY(hipMemcpy(host_out, s->X + (size_t)s->last_row0 * s->m->cfg.d_model, (size_t)n * s->m->cfg.d_model * sizeof(float), hipMemcpyDeviceToHost));
  *n_rows = n;
  return EE_OK;
}
extern "C" int ee_debug_read_dist(ee_session* s, int which, int seq, int row0, int n, float* host_out) {
  if (!s || !host_out || seq < 0 || seq >= s->B || (which != 0 && which != 1)) { ee_set_error("bad argument"); return EE_ERR_ARG; }
  if (!s->Pd) { ee_set_error("sampling buffers are not attached"); return EE_ERR_STATE; }
  if (row0 < 0 || n < 0 || row0 + n > s->max_rows) { ee_set_error("rows outside the store"); return EE_ERR_ARG; }
  const size_t V = s->m->cfg.vocab;
  const float* src = (which == 0 ? s->Pd : s->Pi) + ((size_t)seq * s->max_rows + row0) * V;
  HIP_TRY(hipStreamSynchronize(s->st));
  HIP_TRY(hipMemcpy(host_out, src, (size_t)n * V * sizeof(float), hipMemcpyDeviceToHost));
  return EE_OK;
}

static int upload_pages(ee_session* s, int seq) {
  const SeqState& q = s->seq[seq];
  if (q.pages.empty()) return EE_OK;
  HIP_TRY(hipMemcpy(s->page_scratch, q.pages.data(), q.pages.size() * sizeof(int), hipMemcpyHostToDevice));
  return EE_OK;
}
extern "C" int ee_debug_read_kv(ee_session* s, int seq, int layer, int pos0, int n, float* k_out, float* v_out) {
  if (!s || !k_out || !v_out || seq < 0 || seq >= s->B) { ee_set_error("bad argument"); return EE_ERR_ARG; }
  const ee_config& c = s->m->cfg;
  const SeqState& q = s->seq[seq];
  if (layer < 0 || layer >= c.n_layers || pos0 < 0 || n < 0 || pos0 + n > (int)q.pages.size() * EE_PAGE) { ee_set_error("KV range not owned by the sequence"); return EE_ERR_ARG; }
  if (!n) return EE_OK;
  size_t cnt = (size_t)n * c.n_kv_heads * c.head_dim;
  float* stage = nullptr;
  HIP_TRY(hipMalloc(&stage, 2 * cnt * sizeof(float)));
  int rc = upload_pages(s, seq);
  if (rc == EE_OK) {
    k_read_kv(s->st, s->m->bf16, s->kv, s->page_scratch, layer, pos0, n, s->n_pages, c.n_kv_heads, c.head_dim, stage, stage + cnt);
    hipError_t e = hipStreamSynchronize(s->st);
    if (e == hipSuccess) e = hipMemcpy(k_out, stage, cnt * sizeof(float), hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(v_out, stage + cnt, cnt * sizeof(float), hipMemcpyDeviceToHost);
    if (e != hipSuccess) { ee_set_error("read_kv: %s", hipGetErrorString(e)); rc = EE_ERR_HIP; }
  }
  (void)hipFree(stage);
  return rc;
}
extern "C" int ee_debug_write_kv(ee_session* s, int seq, int layer, int pos0, int n, const float* k_in, const float* v_in) {
  if (!s || !k_in || !v_in || seq < 0 || seq >= s->B) { ee_set_error("bad argument"); return EE_ERR_ARG; }
  const ee_config& c = s->m->cfg;
  const SeqState& q = s->seq[seq];
  if (layer < 0 || layer >= c.n_layers || pos0 < 0 || n < 0 || pos0 + n > (int)q.pages.size() * EE_PAGE) { ee_set_error("KV range not owned by the sequence"); return EE_ERR_ARG; }
  if (!n) return EE_OK;
  size_t cnt = (size_t)n * c.n_kv_heads * c.head_dim;
  float* stage = nullptr;
  HIP_TRY(hipMalloc(&stage, 2 * cnt * sizeof(float)));
  int rc = upload_pages(s, seq);
  if (rc == EE_OK) {
    hipError_t e = hipMemcpy(stage, k_in, cnt * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(stage + cnt, v_in, cnt * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
      k_write_kv(s->st, s->m->bf16, s->kv, s->page_scratch, layer, pos0, n, s->n_pages, c.n_kv_heads, c.head_dim, stage, stage + cnt);
      e = hipStreamSynchronize(s->st);
    }
    if (e != hipSuccess) { ee_set_error("write_kv: %s", hipGetErrorString(e)); rc = EE_ERR_HIP; }
  }
  (void)hipFree(stage);
  return rc;
}

extern "C" int ee_debug_poison_dead_kv(ee_session* s, int seq) {
  if (!s || seq < 0 || seq >= s->B) { ee_set_error("bad argument"); return EE_ERR_ARG; }
  const ee_config& c = s->m->cfg;
  const SeqState& q = s->seq[seq];
  EE_TRY(upload_pages(s, seq));
  std::vector<int> bounds = {0};
  bounds.insert(bounds.end(), s->m->exits.begin(), s->m->exits.end());
  for (int g = 0; g <= s->n_levels; ++g)
    k_fill_nan_dead_kv(s->st, s->m->bf16, s->kv, s->page_scratch, (int)q.pages.size(), q.len[g], bounds[g], bounds[g + 1],
                       s->n_pages, c.n_kv_heads, c.head_dim);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipStreamSynchronize(s->st));
  return EE_OK;
}
extern "C" int ee_debug_gemm_row_blocks(int row_tiles) {
  if (row_tiles == 1000 || row_tiles == 1016) {      // wide matrices beyond 256 rows: parts of up to 512 rows / blocks of 256
    g_rows_wide = row_tiles == 1016;
    return EE_OK;
  }
  if (row_tiles != -1 && row_tiles != 0 && row_tiles != 4 && row_tiles != 8 && row_tiles != 16 && row_tiles != 104 && row_tiles != 108) {
    ee_set_error("row_tiles must be -1, 0, 4, 8, 16, 104, 108, 1000 or 1016");
    return EE_ERR_ARG;
  }
  if (row_tiles == -1) g_rows_wide = 1;
  g_rows_blocks_override = row_tiles;
  return EE_OK;
}

extern "C" int ee_debug_gemm_block_tiles(int weight_tiles) {
  if (weight_tiles != 0 && weight_tiles != 8 && weight_tiles != 12 && weight_tiles != 16 && weight_tiles != 808 && weight_tiles != 1208 && weight_tiles != 1212) {
    ee_set_error("weight_tiles must be 0, 8, 12 or 16, or 808, 1208 or 1212 (with row tiles)");
    return EE_ERR_ARG;
  }
  g_block_tiles = weight_tiles;
  return EE_OK;
}

extern "C" int ee_debug_attention_split_pages(int pages) {
  if (pages < 0 || pages > 65536) { ee_set_error("pages per split must be 0 (built-in choice) or positive"); return EE_ERR_ARG; }
  g_attn_pages_override = pages;
  return EE_OK;
}

extern "C" int ee_debug_attention_form(int form) {
  if (form < -1 || form > ATTN_TILE) { ee_set_error("form must be -1 (built-in choice), 0, 1 or 2"); return EE_ERR_ARG; }
  g_attn_form = form;
  return EE_OK;
}
extern "C" int ee_debug_last_attention(const ee_session* s) { return s ? s->last_attn : -1; }

extern "C" int ee_debug_time_kernels(ee_session* s, int on) {
  if (!s) { ee_set_error("null session"); return EE_ERR_ARG; }
  s->time_kernels = on != 0;
  return EE_OK;
}
extern "C" int ee_debug_kernel_times(ee_session* s, int32_t* n_families, const char** names, float* ms, int32_t* launches) {
  if (!s || !n_families || !names || !ms || !launches) { ee_set_error("null argument"); return EE_ERR_ARG; }
  HIP_TRY(hipStreamSynchronize(s->st));
  for (int f = 0; f < KF_COUNT; ++f) { names[f] = kFamName[f]; ms[f] = 0.f; launches[f] = s->launches[f]; }
  for (auto& t : s->timers) {
    float x = 0.f;
    if (hipEventElapsedTime(&x, t.a, t.b) == hipSuccess) ms[t.fam] += x;
  }
  *n_families = KF_COUNT;
  return EE_OK;
}
