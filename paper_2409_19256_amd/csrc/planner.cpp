// Host planner: rank coordinates, tensor tables, copy descriptors and tiles for the
// train <-> generation weight reshard of the HybridFlow 3D-HybridEngine.
//
// Paper passages implemented here (arXiv 2409.19256):
//   Section 5.1  sizes: N = p*t*d = p_g*t_g*d_g*d, d_g = p*t/(p_g*t_g)
//   Section 5.3  grouping: training TP/PP groups are consecutive ranks and DP groups sit
//                at stride p*t; HybridFlow generation TP/PP groups take ranks at stride
//                t/t_g and p/p_g and micro-DP groups are consecutive ranks; the vanilla
//                variant reuses the training rule with the smaller sizes
//   Section 5.2  step 1 = gather of the updated parameters inside each micro-DP group,
//                step 4 = re-partition for training
//   Section 5.4  only the remote parameters of the micro-DP group are collected; the own
//                training shard is reused in place (zero redundancy)
// Pure host code: no HIP calls in this file.
#include "plan.hpp"

#include <algorithm>
#include <cstring>
#include <map>
#include <numeric>
#include <set>
#include <tuple>

namespace hf {

namespace {

constexpr uint64_t kTensorAlign = 256;
constexpr uint64_t kRankAlign = 4096;

uint64_t round_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

const int kTrainLayerIds[] = {HF_T_LN1, HF_T_QKV, HF_T_O, HF_T_LN2, HF_T_GATE_UP, HF_T_DOWN};
const int kGenLayerIds[] = {HF_G_LN1, HF_G_Q, HF_G_K, HF_G_V, HF_G_O, HF_G_LN2, HF_G_GATE, HF_G_UP, HF_G_DOWN};

// [rows, cols] of a training-shard tensor (Megatron layout, TP size t)
void train_shape(const hf_model_desc &m, int t, int id, uint32_t &rows, uint32_t &cols) {
  const uint32_t h = m.hidden, hd = m.head_dim;
  switch (id) {
  case HF_T_EMBED: case HF_T_HEAD: rows = m.vocab / t; cols = h; break;
  case HF_T_LN1: case HF_T_LN2: case HF_T_LNF: rows = 1; cols = h; break;
  case HF_T_QKV: rows = (uint32_t)(m.n_q_heads + 2 * m.n_kv_heads) / t * hd; cols = h; break;
  case HF_T_O: rows = h; cols = (uint32_t)m.n_q_heads * hd / t; break;
  case HF_T_GATE_UP: rows = 2u * m.ffn / t; cols = h; break;
  case HF_T_DOWN: rows = h; cols = (uint32_t)m.ffn / t; break;
  default: rows = cols = 0;
  }
}

// [rows, cols] of a generation-buffer tensor (separate q/k/v/gate/up, TP size tg)
void gen_shape(const hf_model_desc &m, int tg, int id, uint32_t &rows, uint32_t &cols) {
  const uint32_t h = m.hidden, hd = m.head_dim;
  switch (id) {
  case HF_G_EMBED: case HF_G_HEAD: rows = m.vocab / tg; cols = h; break;
  case HF_G_LN1: case HF_G_LN2: case HF_G_LNF: rows = 1; cols = h; break;
  case HF_G_Q: rows = (uint32_t)m.n_q_heads * hd / tg; cols = h; break;
  case HF_G_K: case HF_G_V: rows = (uint32_t)m.n_kv_heads * hd / tg; cols = h; break;
  case HF_G_O: rows = h; cols = (uint32_t)m.n_q_heads * hd / tg; break;
  case HF_G_GATE: case HF_G_UP: rows = (uint32_t)m.ffn / tg; cols = h; break;
  case HF_G_DOWN: rows = h; cols = (uint32_t)m.ffn / tg; break;
  default: rows = cols = 0;
  }
}

template <typename ShapeFn>
void lay_out(RankTable &tab, bool first, bool last, int layer0, int n_layers, const int *layer_ids, int n_ids,
             int id_embed, int id_lnf, int id_head, ShapeFn shape) {
  uint64_t off = 0;
  auto put = [&](int id, int layer) {
    TensorRec r;
    r.id = id;
    r.layer = layer;
    shape(id, r.rows, r.cols);
    off = round_up(off, kTensorAlign);
    r.off = off;
    off += (uint64_t)r.rows * r.cols * 2;
    tab.index[{id, layer}] = (int)tab.tensors.size();
    tab.tensors.push_back(r);
  };
  if (first) put(id_embed, -1);
  for (int l = layer0; l < layer0 + n_layers; ++l)
    for (int k = 0; k < n_ids; ++k) put(layer_ids[k], l);
  if (last) {
    put(id_lnf, -1);
    put(id_head, -1);
  }
  tab.size = round_up(off, kRankAlign);
}

uint32_t align_flag(uint64_t x) {
  if (x % 16 == 0) return HF_DESC_ALIGN16;
  if (x % 8 == 0) return HF_DESC_ALIGN8;
  if (x % 4 == 0) return HF_DESC_ALIGN4;
  return HF_DESC_ALIGN2;
}

// widest vector that divides every offset, size and (used) stride of the descriptor
uint32_t desc_align(const hf_desc &d) {
  uint64_t g = d.src_off | d.dst_off | d.row_bytes;
  if (d.rows > 1) g |= d.src_row_stride | d.dst_row_stride;
  if (d.n_blocks > 1) g |= d.src_block_stride | d.dst_block_stride;
  return align_flag(g); // low set bit of the OR = gcd with a power of two
}

struct Emitter {
  Plan &pl;
  int dst_rank;
  // offsets are relative to the START OF THE TENSOR on either side
  void add(int src_rank, const TensorRec &src_t, const TensorRec &dst_t, uint32_t kind, uint64_t src_delta,
           uint64_t dst_delta, uint32_t n_blocks, uint32_t rows, uint32_t row_bytes, uint64_t sbs, uint64_t dbs,
           uint64_t srs, uint64_t drs) {
    hf_desc d;
    std::memset(&d, 0, sizeof d);
    d.src_rank = src_rank;
    d.dst_rank = dst_rank;
    d.tensor_id = dst_t.id;
    d.layer = dst_t.layer;
    d.kind = kind;
    d.src_off = pl.train_tab[src_rank].base + src_t.off + src_delta;
    d.dst_off = pl.gen_tab[dst_rank].base + dst_t.off + dst_delta;
    d.n_blocks = n_blocks;
    d.rows = rows;
    d.row_bytes = row_bytes;
    d.src_block_stride = sbs;
    d.dst_block_stride = dbs;
    d.src_row_stride = srs;
    d.dst_row_stride = drs;
    if ((pl.flags & HF_GATHER_FROM_GEN) && src_rank != dst_rank) {
      // The peer is a member of the destination's micro-DP group: same generation stage and
      // TP index, hence the same generation tensors at the same offsets inside its region, and
      // the piece it trains sits there exactly where it is wanted here.
      d.src_off = pl.gen_tab[src_rank].base + dst_t.off + dst_delta;
      d.src_block_stride = dbs;
      d.src_row_stride = drs;
    }
    d.flags = desc_align(d) | (src_rank == dst_rank ? HF_DESC_OWN : 0u);
    (src_rank == dst_rank ? pl.fwd_own : pl.fwd_peer).push_back(d);
  }
};

} // namespace

uint64_t desc_bytes(const hf_desc &d) { return (uint64_t)d.n_blocks * d.rows * d.row_bytes; }

uint64_t unique_src_bytes(const std::vector<const hf_desc *> &descs) {
  // pieces read by several destinations are byte-identical descriptors on the source
  // side; different pieces never overlap (checked by validate_plan through coverage)
  std::set<std::tuple<uint64_t, uint64_t, uint32_t, uint32_t, uint32_t>> seen;
  uint64_t total = 0;
  for (const hf_desc *d : descs)
    if (seen.insert({d->src_off, d->src_block_stride, d->n_blocks, d->rows, d->row_bytes}).second)
      total += desc_bytes(*d);
  return total;
}

int build_plan(const hf_model_desc &m, const hf_train_layout &tl, const hf_gen_layout &gl, Plan &pl, std::string &err) {
  // ---- validation -------------------------------------------------------------
  const int32_t sizes[] = {m.n_layers, m.hidden, m.n_q_heads, m.n_kv_heads, m.head_dim, m.ffn, m.vocab,
                           tl.pp, tl.tp, tl.dp, gl.pp, gl.tp};
  for (int32_t v : sizes)
    if (v <= 0) { err = "all model and layout sizes must be positive"; return HF_EINVAL; }
  if (m.elem_bytes != 2) { err = "elem_bytes must be 2 (bf16)"; return HF_EINVAL; }
  if (m.tied_embed != 0) { err = "tied embedding / LM head is not supported"; return HF_EINVAL; }
  if (gl.flags & ~(HF_COPY_OWN | HF_GROUPING_VANILLA | HF_PLAN_HOST_ONLY | HF_PLAN_OFFLOAD | HF_GATHER_FROM_GEN)) { err = "unknown flag bits"; return HF_EINVAL; }
  if ((gl.flags & HF_GATHER_FROM_GEN) && (gl.flags & (HF_COPY_OWN | HF_GROUPING_VANILLA))) {
    err = "HF_GATHER_FROM_GEN needs the HybridFlow grouping and HF_SKIP_OWN: the own pieces are the source";
    return HF_EINVAL;
  }
  if (gl.mat_ranks && gl.n_mat <= 0) { err = "mat_ranks given but n_mat <= 0"; return HF_EINVAL; }
  struct { bool bad; const char *what; } div[] = {
      {tl.tp % gl.tp != 0, "t % t_g"}, {tl.pp % gl.pp != 0, "p % p_g"}, {m.n_layers % tl.pp != 0, "L % p"},
      {m.n_layers % gl.pp != 0, "L % p_g"}, {m.vocab % tl.tp != 0, "V % t"}, {m.ffn % tl.tp != 0, "F % t"},
      {m.n_q_heads % m.n_kv_heads != 0, "n_q % n_kv"}, {m.n_kv_heads % tl.tp != 0, "n_kv % t"},
      {m.n_kv_heads % gl.tp != 0, "n_kv % t_g"}};
  for (auto &c : div)
    if (c.bad) { err = std::string("not divisible: ") + c.what; return HF_EDIVIS; }
  const int64_t n64 = (int64_t)tl.pp * tl.tp * tl.dp;
  if (n64 > (1 << 20)) { err = "too many ranks"; return HF_ERANGE; }
  // row lengths and block strides must fit 32-bit fields of descriptors and tiles
  const uint64_t widest_row = 2ull * std::max<uint64_t>(m.hidden, std::max<uint64_t>(m.ffn, (uint64_t)m.n_q_heads * m.head_dim));
  const uint64_t qkv_group = 2ull * ((uint64_t)m.n_q_heads / m.n_kv_heads + 2) * m.head_dim * m.hidden;
  if (widest_row >= (1ull << 31) || qkv_group >= (1ull << 32)) { err = "tensor rows too long for 32-bit strides"; return HF_ERANGE; }

  pl.m = m;
  pl.p = tl.pp; pl.t = tl.tp; pl.d = tl.dp; pl.pg = gl.pp; pl.tg = gl.tp;
  pl.flags = gl.flags;
  pl.multicast_auto = true; // build_tiles picks the mode from the fan-out of the list
  pl.a = pl.t / pl.tg;
  pl.b = pl.p / pl.pg;
  pl.dg = pl.a * pl.b;
  pl.N = (int)n64;
  pl.lps = m.n_layers / pl.p;
  pl.lpgs = m.n_layers / pl.pg;
  const int N = pl.N, p = pl.p, t = pl.t, pg = pl.pg, tg = pl.tg, a = pl.a, b = pl.b;
  const bool vanilla = (gl.flags & HF_GROUPING_VANILLA) != 0;

  // ---- materialised ranks ------------------------------------------------------
  pl.mat_pos.assign(N, -1);
  if (gl.mat_ranks) {
    for (int i = 0; i < gl.n_mat; ++i) {
      const int r = gl.mat_ranks[i];
      if (r < 0 || r >= N) { err = "materialised rank out of range"; return HF_ERANGE; }
      if (pl.mat_pos[r] >= 0) { err = "materialised rank listed twice"; return HF_ERANGE; }
      pl.mat_pos[r] = i;
      pl.mat.push_back(r);
    }
  } else {
    for (int r = 0; r < N; ++r) { pl.mat_pos[r] = r; pl.mat.push_back(r); }
  }

  // ---- rank coordinates ----------------------------------------------------------
  pl.coords.resize(N);
  for (int r = 0; r < N; ++r) {
    Coords &c = pl.coords[r];
    c.dp = r / (p * t);
    c.pp = (r % (p * t)) / t;
    c.tp = r % t;
    if (!vanilla) {
      // generation TP peers are t/t_g training ranks apart and generation PP peers p/p_g
      // stages apart: quotient = generation index, remainder = place in the micro-DP group
      c.gtp = c.tp / a;
      c.gpp = c.pp / b;
      c.micro = (c.pp % b) * a + (c.tp % a);
    } else {
      const int i = c.pp * t + c.tp; // place inside the replica; consecutive ranks per group
      c.gtp = i % tg;
      c.gpp = (i / tg) % pg;
      c.micro = i / (tg * pg);
    }
  }

  // micro-DP groups: the d_g ranks of a replica that share (gpp, gtp), by micro-DP index
  pl.micro_peers.assign((size_t)N * pl.dg, -1);
  for (int r = 0; r < N; ++r)
    for (int q = 0; q < N; ++q) {
      const Coords &x = pl.coords[r], &y = pl.coords[q];
      if (x.dp == y.dp && x.gpp == y.gpp && x.gtp == y.gtp) pl.micro_peers[(size_t)r * pl.dg + y.micro] = q;
    }
  for (int32_t q : pl.micro_peers)
    if (q < 0) { err = "internal: incomplete micro-DP group"; return HF_EINVAL; }
  pl.gather_out.resize(pl.micro_peers.size());
  for (int r = 0; r < N; ++r)
    for (int j = 0; j < pl.dg; ++j)
      pl.gather_out[(size_t)r * pl.dg + j] = (uint32_t)pl.micro_peers[(size_t)r * pl.dg + j] * pl.dg + pl.coords[r].micro;

  // ---- tensor tables -----------------------------------------------------------
  pl.train_tab.assign(N, RankTable());
  pl.gen_tab.assign(N, RankTable());
  uint64_t base = 0;
  for (int r = 0; r < N; ++r) {
    const Coords &c = pl.coords[r];
    lay_out(pl.train_tab[r], c.pp == 0, c.pp == p - 1, c.pp * pl.lps, pl.lps, kTrainLayerIds, 6, HF_T_EMBED, HF_T_LNF,
            HF_T_HEAD, [&](int id, uint32_t &rows, uint32_t &cols) { train_shape(m, t, id, rows, cols); });
    pl.train_tab[r].base = base;
    base += pl.train_tab[r].size;
    lay_out(pl.gen_tab[r], c.gpp == 0, c.gpp == pg - 1, c.gpp * pl.lpgs, pl.lpgs, kGenLayerIds, 9, HF_G_EMBED, HF_G_LNF,
            HF_G_HEAD, [&](int id, uint32_t &rows, uint32_t &cols) { gen_shape(m, tg, id, rows, cols); });
  }
  pl.train_bytes = base;
  base = 0;
  for (int r : pl.mat) {
    pl.gen_tab[r].base = base;
    base += pl.gen_tab[r].size;
  }
  pl.gen_bytes = base;

  // ---- step 1 descriptors: for every materialised rank, every generation tensor, every
  // training shard that contributes to it ------------------------------------------
  const uint64_t h2 = 2ull * m.hidden;                 // bytes of one [*, h] row
  const uint32_t hd = m.head_dim, qpg = m.n_q_heads / m.n_kv_heads;
  const uint32_t ng = m.n_kv_heads / t;                // KV groups per training shard
  const uint64_t grp = (uint64_t)(qpg + 2) * hd * h2;  // bytes of one fused [q..q k v] group
  for (int r : pl.mat) {
    const Coords &c = pl.coords[r];
    Emitter em{pl, r};
    auto rank_of = [&](int pp, int tp) { return c.dp * p * t + pp * t + tp; };
    for (const TensorRec &g : pl.gen_tab[r].tensors) {
      // training stage that owns the tensor
      const int spp = g.id == HF_G_EMBED ? 0 : (g.id == HF_G_LNF || g.id == HF_G_HEAD) ? p - 1 : g.layer / pl.lps;
      if (g.id == HF_G_LN1 || g.id == HF_G_LN2 || g.id == HF_G_LNF) {
        // replicated: take the copy of the rank with the same TP index in the owning stage
        const int q = rank_of(spp, c.tp);
        if ((gl.flags & HF_GATHER_FROM_GEN) && pl.mat_pos[q] < 0) { err = "HF_GATHER_FROM_GEN: a micro-DP peer of a materialised rank is not materialised"; return HF_EINVAL; }
        const int tid = g.id == HF_G_LN1 ? HF_T_LN1 : g.id == HF_G_LN2 ? HF_T_LN2 : HF_T_LNF;
        em.add(q, pl.train_tab[q].at(tid, g.layer), g, HF_REPL, 0, 0, 1, 1, (uint32_t)h2, h2, h2, h2, h2);
        continue;
      }
      for (int k = 0; k < a; ++k) {                    // the a training TP shards inside generation shard gtp
        const int q = rank_of(spp, c.gtp * a + k);
        if ((gl.flags & HF_GATHER_FROM_GEN) && pl.mat_pos[q] < 0) { err = "HF_GATHER_FROM_GEN: a micro-DP peer of a materialised rank is not materialised"; return HF_EINVAL; }
        const RankTable &st = pl.train_tab[q];
        switch (g.id) {
        case HF_G_EMBED: case HF_G_HEAD: {
          const TensorRec &s = st.at(g.id == HF_G_EMBED ? HF_T_EMBED : HF_T_HEAD, -1);
          em.add(q, s, g, HF_COL, 0, (uint64_t)k * s.rows * h2, 1, s.rows, (uint32_t)h2, 0, 0, h2, h2);
          break;
        }
        case HF_G_Q: case HF_G_K: case HF_G_V: {
          const TensorRec &s = st.at(HF_T_QKV, g.layer);
          const uint32_t rows = g.id == HF_G_Q ? qpg * hd : hd;             // rows of one group's piece
          const uint64_t in_group = g.id == HF_G_Q ? 0 : g.id == HF_G_K ? (uint64_t)qpg * hd * h2 : (uint64_t)(qpg + 1) * hd * h2;
          em.add(q, s, g, HF_QKV_DEINT, in_group, (uint64_t)k * ng * rows * h2, ng, rows, (uint32_t)h2, grp,
                 (uint64_t)rows * h2, h2, h2);
          break;
        }
        case HF_G_GATE: case HF_G_UP: {
          const TensorRec &s = st.at(HF_T_GATE_UP, g.layer);
          const uint32_t rows = s.rows / 2;                                  // F/t
          em.add(q, s, g, HF_GATEUP_DEINT, g.id == HF_G_GATE ? 0 : (uint64_t)rows * h2, (uint64_t)k * rows * h2, 1, rows,
                 (uint32_t)h2, 0, 0, h2, h2);
          break;
        }
        case HF_G_O: case HF_G_DOWN: {
          const TensorRec &s = st.at(g.id == HF_G_O ? HF_T_O : HF_T_DOWN, g.layer);
          em.add(q, s, g, HF_ROW, 0, (uint64_t)k * s.cols * 2, 1, s.rows, s.cols * 2, 0, 0, (uint64_t)s.cols * 2,
                 (uint64_t)g.cols * 2);
          break;
        }
        default: err = "internal: unknown generation tensor"; return HF_EINVAL;
        }
      }
    }
  }

  // ---- step 4 descriptors: the own pieces, run backwards ----------------------------
  if (!vanilla) {
    pl.back.reserve(pl.fwd_own.size());
    for (const hf_desc &o : pl.fwd_own) {
      hf_desc d = o;
      std::swap(d.src_off, d.dst_off);
      std::swap(d.src_block_stride, d.dst_block_stride);
      std::swap(d.src_row_stride, d.dst_row_stride);
      pl.back.push_back(d);
    }
  }

  // ---- offload image of the remote pieces (Section 7: the generation copy of the weights
  // leaves the GPU while the model trains).  The peer descriptors of one (rank, generation
  // tensor) are consecutive and ordered by the position of their piece in the tensor, so
  // the remote elements of the tensor in row-major order are: for column-parallel kinds the
  // pieces one after another, for row-parallel kinds a matrix [rows, n_remote * piece cols].
  // Tensor parts start at 256-byte boundaries, rank parts at 4096-byte boundaries.
  {
    uint64_t hoff = 0;
    int cur_rank = -1;
    for (size_t i = 0; i < pl.fwd_peer.size();) {
      const hf_desc &d0 = pl.fwd_peer[i];
      size_t j = i + 1;
      while (j < pl.fwd_peer.size() && pl.fwd_peer[j].dst_rank == d0.dst_rank && pl.fwd_peer[j].tensor_id == d0.tensor_id &&
             pl.fwd_peer[j].layer == d0.layer)
        ++j;
      if (d0.dst_rank != cur_rank) {
        // ranks appear in buffer order; a rank without remote pieces gets an empty part
        while (pl.remote_rank_off.size() <= (size_t)pl.mat_pos[d0.dst_rank]) {
          hoff = round_up(hoff, kRankAlign);
          pl.remote_rank_off.push_back(hoff);
        }
        cur_rank = d0.dst_rank;
      }
      hoff = round_up(hoff, kTensorAlign);
      const uint64_t n_remote = j - i;
      for (size_t k = i; k < j; ++k) {
        const hf_desc &f = pl.fwd_peer[k];
        hf_desc d;
        std::memset(&d, 0, sizeof d);
        d.src_rank = d.dst_rank = f.dst_rank;
        d.tensor_id = f.tensor_id;
        d.layer = f.layer;
        d.kind = f.kind;
        d.src_off = f.dst_off;
        d.n_blocks = 1;
        d.row_bytes = f.row_bytes;
        if (f.kind == HF_ROW) {
          d.rows = f.rows;
          d.src_row_stride = f.dst_row_stride;
          d.dst_row_stride = n_remote * f.row_bytes;
          d.dst_off = hoff + (k - i) * f.row_bytes;
        } else { // contiguous in the generation tensor
          d.rows = f.n_blocks * f.rows;
          d.src_row_stride = d.dst_row_stride = f.row_bytes;
          d.dst_off = hoff + (k - i) * desc_bytes(f);
        }
        d.src_block_stride = (uint64_t)d.rows * d.src_row_stride;
        d.dst_block_stride = (uint64_t)d.rows * d.dst_row_stride;
        d.flags = desc_align(d);
        pl.remote.push_back(d);
      }
      hoff += n_remote * desc_bytes(d0);
      i = j;
    }
    while (pl.remote_rank_off.size() < pl.mat.size()) {
      hoff = round_up(hoff, kRankAlign);
      pl.remote_rank_off.push_back(hoff);
    }
    pl.remote_bytes = round_up(hoff, kRankAlign);
  }
  return build_tiles(pl, err);
}

// ---- tiler --------------------------------------------------------------------------
namespace {

uint32_t vec_of(uint64_t g) { return g % 16 == 0 ? 16 : g % 8 == 0 ? 8 : g % 4 == 0 ? 4 : 2; }

void push_tile(std::vector<hf_tile> &out, uint64_t src, uint64_t dst, uint32_t rows, uint32_t row_bytes, uint32_t sstr,
               uint32_t dstr) {
  hf_tile tl;
  std::memset(&tl, 0, sizeof tl);
  tl.src_off = src;
  tl.dst_off = dst;
  tl.rows = rows;
  tl.row_bytes = row_bytes;
  tl.src_row_stride = rows > 1 ? sstr : row_bytes;
  tl.dst_row_stride = rows > 1 ? dstr : row_bytes;
  uint64_t g = src | dst | row_bytes;
  if (rows > 1) g |= (uint64_t)sstr | dstr;
  tl.vec_bytes = vec_of(g);
  tl.n_dst = 1;
  out.push_back(tl);
}

// how much of a run of `len` bytes that starts at `dst` goes into the next piece of at most `most`
// bytes: up to a 128-byte line of the destination, and never so much that less than a slot is left
uint32_t run_piece(uint64_t dst, uint64_t len, uint32_t most) {
  const uint32_t n = most - (uint32_t)(dst % 128);
  if (len <= n) return (uint32_t)len;
  return len - n < kSlot ? n - 128 : n;
}

// What a tile is measured by: the slots the kernels move (slots.hpp), or its payload, equal chunks
// of a run, whatever the rows are cut into on the device.  The second measure is the one that
// hf_reshard_execute_static's limit counts in (see build_static_list).
enum class Measure { kSlots, kPayload };

uint64_t payload_chunk(uint64_t len, uint64_t tile_bytes) {
  const uint64_t n = (len + tile_bytes - 1) / tile_bytes;
  return round_up((len + n - 1) / n, 256);
}

// one contiguous run of `len` bytes -> tiles of tile_bytes, and what is left
void tile_run(std::vector<hf_tile> &out, uint64_t src, uint64_t dst, uint64_t len, uint64_t tile_bytes, Measure by) {
  const uint64_t chunk = by == Measure::kPayload ? payload_chunk(len, tile_bytes) : 0;
  for (uint64_t o = 0, n; o < len; o += n) {
    n = by == Measure::kPayload ? std::min(chunk, len - o) : run_piece(dst + o, len - o, (uint32_t)tile_bytes);
    push_tile(out, src + o, dst + o, 1, (uint32_t)n, 0, 0);
  }
}

uint32_t desc_vec(const hf_desc &d) {
  return d.flags & HF_DESC_ALIGN16 ? 16 : d.flags & HF_DESC_ALIGN8 ? 8 : d.flags & HF_DESC_ALIGN4 ? 4 : 2;
}

// How a descriptor falls apart: one run, one run per block, one run per row, or tiles of several rows.
enum class Form { kRun, kBlockRuns, kRowRuns, kRows };

Form form_of(const hf_desc &d, uint64_t tile_bytes) {
  const bool rows_contig = d.rows == 1 || (d.src_row_stride == d.row_bytes && d.dst_row_stride == d.row_bytes);
  const uint64_t block_len = (uint64_t)d.rows * d.row_bytes;
  const bool blocks_contig = d.n_blocks == 1 || (d.src_block_stride == block_len && d.dst_block_stride == block_len);
  if (rows_contig) return blocks_contig ? Form::kRun : Form::kBlockRuns;
  return d.row_bytes >= tile_bytes ? Form::kRowRuns : Form::kRows;
}

// rows per tile of a Form::kRows descriptor: tile_bytes of slots or of payload, and offsets inside a
// tile below 4 GiB (the kernel computes row*stride in 32 bits)
uint32_t rows_per_tile(const hf_desc &d, uint64_t tile_bytes, Measure by) {
  uint64_t row = d.row_bytes;
  if (by == Measure::kSlots) {
    uint32_t unused;
    row = slot_geometry(d.dst_off, 2, d.row_bytes, (uint32_t)d.dst_row_stride, desc_vec(d), unused) / 2 * kSlot;
  }
  const uint64_t widest = std::max(d.src_row_stride, d.dst_row_stride);
  const uint64_t fit = ((1ull << 32) - 1 - d.row_bytes) / std::max<uint64_t>(widest, 1) + 1;
  return (uint32_t)std::max<uint64_t>(1, std::min(tile_bytes / row, fit));
}

void tile_desc(std::vector<hf_tile> &out, const hf_desc &d, uint64_t tile_bytes, Measure by) {
  const Form form = form_of(d, tile_bytes);
  const uint64_t block_len = (uint64_t)d.rows * d.row_bytes;
  if (form == Form::kRun) {
    tile_run(out, d.src_off, d.dst_off, block_len * d.n_blocks, tile_bytes, by);
    return;
  }
  const uint32_t per = form == Form::kRows ? rows_per_tile(d, tile_bytes, by) : 0;
  for (uint32_t bidx = 0; bidx < d.n_blocks; ++bidx) {
    const uint64_t s = d.src_off + bidx * d.src_block_stride, t = d.dst_off + bidx * d.dst_block_stride;
    if (form == Form::kBlockRuns) {
      tile_run(out, s, t, block_len, tile_bytes, by);
    } else if (form == Form::kRowRuns) {
      for (uint32_t r = 0; r < d.rows; ++r) tile_run(out, s + r * d.src_row_stride, t + r * d.dst_row_stride, d.row_bytes, tile_bytes, by);
    } else {
      for (uint32_t r = 0; r < d.rows; r += per)
        push_tile(out, s + r * d.src_row_stride, t + r * d.dst_row_stride, std::min(per, d.rows - r), d.row_bytes,
                  (uint32_t)d.src_row_stride, (uint32_t)d.dst_row_stride);
    }
  }
}

// the number of tiles that tile_desc makes by payload
uint64_t payload_tiles(const hf_desc &d, uint64_t tile_bytes) {
  const uint64_t block_len = (uint64_t)d.rows * d.row_bytes;
  const auto run = [&](uint64_t len) { const uint64_t c = payload_chunk(len, tile_bytes); return (len + c - 1) / c; };
  switch (form_of(d, tile_bytes)) {
  case Form::kRun: return run(block_len * d.n_blocks);
  case Form::kBlockRuns: return d.n_blocks * run(block_len);
  case Form::kRowRuns: return (uint64_t)d.n_blocks * d.rows * run(d.row_bytes);
  case Form::kRows: break;
  }
  const uint64_t per = rows_per_tile(d, tile_bytes, Measure::kPayload);
  return d.n_blocks * ((d.rows + per - 1) / per);
}

} // namespace

// Multicast mode when the caller leaves the choice to the library, from the list's fan-out
// (bytes written per distinct byte read).  Measured on the Llama-7B, 13B and 34B shapes under
// training TP 8 (and TP 4 x PP 2) with generation TP 1, 2, 4, own pieces in the list or not, in
// several processes on several machines:
//   2 destinations per piece: registers and prefetched level, cache-blocked 3-5 % behind;
//   3: prefetched 1-3 % ahead of cache-blocked on average and never behind it; registers
//      between 3 % ahead and 10 % behind from process to process;
//   4: prefetched 3-8 % ahead of the others;
//   7 and 8: prefetched and registers level, cache-blocked 10-13 % behind.
int64_t default_multicast(const Plan &pl) {
  if (!pl.unique_bytes[0]) return HF_MULTICAST_PREFETCHED;
  return pl.fan_out() < 2.5 ? HF_MULTICAST_REGISTERS : HF_MULTICAST_PREFETCHED;
}

// Copy tiles per chunked load-only tile of the prefetched list when the caller leaves it to
// the library.  Measured on the same workloads: two chunks against one gain 7 % at 3
// destinations per piece (Llama-7B TP8->TP2: 8.29 against 8.88 ms), 3 % at 4, nothing at 7
// and 8; four and eight chunks lose the gain again at 3 and 4 and are level at 7 and 8.
int64_t default_prefetch_merge(const Plan &) { return 2; }

namespace {

bool wanted(const Plan &pl, const hf_desc &d) { return (pl.kind_mask >> d.kind) & 1; }

// one-destination lists in descriptor order, except that a run of row-parallel
// descriptors into the same destination tensor (its column stripes) is tiled round-robin,
// for the DRAM-row reason given at the multicast list below
void tile_list(const Plan &pl, const std::vector<hf_desc> &descs, std::vector<hf_tile> &out, Measure by = Measure::kSlots) {
  std::vector<std::vector<hf_tile>> run;
  for (size_t i = 0; i < descs.size();) {
    if (!wanted(pl, descs[i])) { ++i; continue; }
    size_t j = i + 1;
    if (descs[i].kind == HF_ROW && pl.row_interleave)
      while (j < descs.size() && descs[j].kind == HF_ROW && descs[j].dst_rank == descs[i].dst_rank &&
             descs[j].tensor_id == descs[i].tensor_id && descs[j].layer == descs[i].layer)
        ++j;
    if (j == i + 1) {
      tile_desc(out, descs[i], (uint64_t)pl.tile_bytes, by);
    } else {
      run.assign(j - i, {});
      size_t longest = 0;
      for (size_t k = i; k < j; ++k) {
        tile_desc(run[k - i], descs[k], (uint64_t)pl.tile_bytes, by);
        longest = std::max(longest, run[k - i].size());
      }
      for (size_t t = 0; t < longest; ++t)
        for (auto &r : run)
          if (t < r.size()) out.push_back(r[t]);
    }
    i = j;
  }
}

// one-destination lists of all four directions
void build_plain_lists(Plan &pl) {
  pl.tiles_fwd.clear();
  pl.tiles_back.clear();
  tile_list(pl, pl.fwd_peer, pl.tiles_fwd);
  pl.n_tiles_fwd_peer = pl.tiles_fwd.size();
  tile_list(pl, pl.fwd_own, pl.tiles_fwd);
  tile_list(pl, pl.back, pl.tiles_back);
  pl.tiles_offload.clear();
  pl.tiles_reload.clear();
  if (pl.flags & HF_PLAN_OFFLOAD) {
    for (const hf_desc &d : pl.remote) tile_desc(pl.tiles_offload, d, (uint64_t)pl.tile_bytes, Measure::kSlots);
    pl.tiles_reload = pl.tiles_offload;
    for (hf_tile &t : pl.tiles_reload) {
      std::swap(t.src_off, t.dst_off);
      std::swap(t.src_row_stride, t.dst_row_stride);
    }
  }
}

// totals of the descriptors that take part (queried on the hot path of harnesses)
void cache_totals(Plan &pl) {
  std::vector<const hf_desc *> fwd, back;
  for (const hf_desc &d : pl.fwd_peer) if (wanted(pl, d)) fwd.push_back(&d);
  if (pl.flags & HF_COPY_OWN)
    for (const hf_desc &d : pl.fwd_own) if (wanted(pl, d)) fwd.push_back(&d);
  for (const hf_desc &d : pl.back) if (wanted(pl, d)) back.push_back(&d);
  pl.moved_bytes[0] = pl.moved_bytes[1] = 0;
  for (const hf_desc *d : fwd) pl.moved_bytes[0] += desc_bytes(*d);
  for (const hf_desc *d : back) pl.moved_bytes[1] += desc_bytes(*d);
  pl.unique_bytes[0] = unique_src_bytes(fwd);
  pl.unique_bytes[1] = unique_src_bytes(back);
}

// The descriptors execute performs, grouped by what they read: same source bytes and same geometry, in order
// of first appearance.
typedef std::vector<std::vector<const hf_desc *>> Groups;
Groups sharing_groups(const Plan &pl) {
  std::vector<const hf_desc *> active;
  for (const hf_desc &d : pl.fwd_peer) if (wanted(pl, d)) active.push_back(&d);
  if (pl.flags & HF_COPY_OWN)
    for (const hf_desc &d : pl.fwd_own) if (wanted(pl, d)) active.push_back(&d);
  typedef std::tuple<uint64_t, uint32_t, uint32_t, uint32_t, uint64_t, uint64_t, uint64_t, uint64_t> Key;
  std::map<Key, size_t> group_of;
  Groups groups;
  for (const hf_desc *d : active) {
    const Key k{d->src_off, d->n_blocks, d->rows, d->row_bytes, d->src_block_stride, d->src_row_stride,
                d->dst_block_stride, d->dst_row_stride};
    auto it = group_of.find(k);
    if (it == group_of.end()) {
      group_of[k] = groups.size();
      groups.push_back({d});
    } else {
      groups[it->second].push_back(d);
    }
  }
  return groups;
}

// The groups of the column stripes of one row-parallel generation tensor, by tensor.
typedef std::tuple<int, int, int, int, int> SibKey; // tensor, layer, dp, gpp, gtp of the destination
typedef std::map<SibKey, std::vector<size_t>> Siblings;
Siblings stripe_siblings(const Plan &pl, const Groups &groups) {
  Siblings siblings;
  for (size_t gi = 0; gi < groups.size(); ++gi) {
    const hf_desc &d0 = *groups[gi][0];
    if (d0.kind != HF_ROW) continue;
    const Coords &c = pl.coords[d0.dst_rank];
    siblings[SibKey{d0.tensor_id, d0.layer, c.dp, c.gpp, c.gtp}].push_back(gi);
  }
  return siblings;
}

// multicast list: one tile with several destinations per group
int build_multicast_list(Plan &pl, const Groups &groups, const Siblings &siblings, std::string &err, Measure by = Measure::kSlots) {
  pl.tiles_fwd_mc.clear();
  pl.mc_dst.clear();
  pl.payload_mc = PayloadCount();
  pl.has_sharing = false;
  for (const auto &g : groups) pl.has_sharing = pl.has_sharing || g.size() > 1;
  // tiles of every group (destinations 2..n already appended to mc_dst)
  std::vector<std::vector<hf_tile>> group_tiles(groups.size());
  for (size_t gi = 0; gi < groups.size(); ++gi) {
    const auto &grp_descs = groups[gi];
    const hf_desc &d0 = *grp_descs[0];
    tile_desc(group_tiles[gi], d0, (uint64_t)pl.tile_bytes, by);
    pl.payload_mc.add(payload_tiles(d0, (uint64_t)pl.tile_bytes), grp_descs.size());
    for (hf_tile &tl : group_tiles[gi]) {
      tl.n_dst = (uint32_t)grp_descs.size();
      tl.dst_list = (uint32_t)pl.mc_dst.size();
      uint64_t g = tl.vec_bytes; // already covers source, first destination, sizes, strides
      for (size_t j = 1; j < grp_descs.size(); ++j) {
        const uint64_t off = tl.dst_off - d0.dst_off + grp_descs[j]->dst_off;
        pl.mc_dst.push_back(off);
        g |= off;
      }
      tl.vec_bytes = vec_of(g);
    }
  }
  // Row-parallel tensors: the a training pieces of one generation tensor are column
  // stripes of the same destination rows.  Their tiles are emitted round-robin (rows
  // 0..R of every piece, then the next rows of every piece, ...) so that each
  // destination row is completed while it is still open in DRAM, instead of being
  // visited once per stripe with a fraction of a row each time.
  std::vector<char> emitted(groups.size(), 0);
  for (size_t gi = 0; gi < groups.size(); ++gi) {
    if (emitted[gi]) continue;
    const hf_desc &d0 = *groups[gi][0];
    std::vector<size_t> set{gi};
    if (d0.kind == HF_ROW && pl.row_interleave) {
      const Coords &c = pl.coords[d0.dst_rank];
      set = siblings.at(SibKey{d0.tensor_id, d0.layer, c.dp, c.gpp, c.gtp});
    }
    size_t longest = 0;
    for (size_t g2 : set) { emitted[g2] = 1; longest = std::max(longest, group_tiles[g2].size()); }
    for (size_t i = 0; i < longest; ++i)
      for (size_t g2 : set)
        if (i < group_tiles[g2].size()) pl.tiles_fwd_mc.push_back(group_tiles[g2][i]);
  }
  if (pl.mc_dst.size() >= (1ull << 32)) { err = "too many multicast destinations; raise the tile size"; return HF_ERANGE; }
  return HF_OK;
}

// cache-blocked multicast order: the same work as one-destination tiles, arranged so that
// a block of at most mc_block_bytes of source is copied to its first destination, then
// the same block to the second, ...: only the first pass reads HBM, the later passes
// find the block in the caches (workgroups are handed out in list order).  In the L2 of the XCD that
// read it first where every record has a multiple of eight workgroups, as at the tile size of 128 KiB and
// 8 KiB per workgroup; where short pieces have brought the records below 64 KiB (choose_unit) often in the
// L2 of another XCD only, and then in the memory-side cache.
void build_cache_blocked_list(const Plan &pl, std::vector<hf_tile> &out) {
  out.clear();
  std::vector<const hf_tile *> batch;
  uint64_t batch_bytes = 0;
  auto flush = [&]() {
    if (batch.empty()) return;
    for (uint32_t j = 0; j < batch[0]->n_dst; ++j)
      for (const hf_tile *t : batch) {
        hf_tile one = *t;
        one.dst_off = j == 0 ? t->dst_off : pl.mc_dst[t->dst_list + j - 1];
        one.n_dst = 1;
        one.dst_list = 0;
        out.push_back(one);
      }
    batch.clear();
    batch_bytes = 0;
  };
  for (const hf_tile &t : pl.tiles_fwd_mc) {
    const uint64_t payload = (uint64_t)t.rows * t.row_bytes;
    if (!batch.empty() && (t.n_dst != batch[0]->n_dst || batch_bytes + payload > (uint64_t)pl.mc_block_bytes)) flush();
    batch.push_back(&t);
    batch_bytes += payload;
  }
  flush();
}

// prefetched multicast order: the multicast tiles in blocks of at most prefetch_block_bytes of
// source; in front of every block the load-only tiles (n_dst == 0) that stand for its shared
// source bytes.  This is the list that hf_plan_get_tile shows and that the static limit counts; the
// device takes the blocks from it and makes load-only records of its own, after the copy records
// (compile_prefetched_list).  A shared tile whose source is one contiguous run takes part in a
// chunked load-only tile (dst_list = number of chunks): up to prefetch_merge tiles of the
// block that follow one another in the source and have the same size share one.  A shared tile
// with a strided source gets a load-only copy of itself.
void build_prefetched_list(const Plan &pl, std::vector<hf_tile> &out) {
  out.clear();
  std::vector<const hf_tile *> batch;
  uint64_t batch_bytes = 0;
  const uint32_t merge = (uint32_t)std::max<int64_t>(1, std::min<int64_t>(pl.effective_prefetch_merge(), HF_MAX_PREFETCH_CHUNKS));
  std::map<uint64_t, size_t> open; // source offset a chain would continue at -> its load-only tile
  auto flush = [&]() {
    open.clear();
    for (const hf_tile *t : batch) {
      if (t->n_dst <= 1) continue; // a piece with one destination is read once anyway
      const uint64_t payload = (uint64_t)t->rows * t->row_bytes;
      const bool flat = t->rows == 1 || t->src_row_stride == t->row_bytes;
      if (!flat || t->src_off % 16 || payload % 16) {
        hf_tile pre = *t;
        pre.n_dst = 0;
        pre.dst_list = 0;
        out.push_back(pre);
        continue;
      }
      auto it = open.find(t->src_off);
      if (it != open.end() && out[it->second].row_bytes == payload) {
        const size_t at = it->second;
        hf_tile &pre = out[at];
        pre.rows = ++pre.dst_list;
        open.erase(it);
        if (pre.dst_list < merge) open[t->src_off + payload] = at;
        continue;
      }
      hf_tile pre;
      std::memset(&pre, 0, sizeof pre);
      pre.src_off = t->src_off;
      pre.rows = 1;
      pre.row_bytes = (uint32_t)payload;
      pre.src_row_stride = pre.dst_row_stride = (uint32_t)payload;
      pre.vec_bytes = 16;
      pre.dst_list = 1;
      if (merge > 1) open[t->src_off + payload] = out.size();
      out.push_back(pre);
    }
    for (const hf_tile *t : batch) out.push_back(*t);
    batch.clear();
    batch_bytes = 0;
  };
  for (const hf_tile &t : pl.tiles_fwd_mc) {
    const uint64_t payload = (uint64_t)t.rows * t.row_bytes;
    if (!batch.empty() && batch_bytes + payload > (uint64_t)pl.prefetch_block_bytes) flush();
    batch.push_back(&t);
    batch_bytes += payload;
  }
  flush();
}

// ---- device lists ---------------------------------------------------------------------

// the records of a tile, at most `unit` slots each (offsets stay those of the tile: its further
// destinations are listed for the tile as a whole).  on_kib: for kernels whose wavefronts begin at
// KiB of the destination
template <typename F> void cut_tile(const hf_tile &t, uint32_t unit, F take, bool lines = true, bool on_kib = false) {
  DevTile r;
  r.src_off = t.src_off;
  r.dst_off = t.dst_off;
  r.row_bytes = t.row_bytes;
  r.src_row_stride = t.src_row_stride;
  r.dst_row_stride = t.dst_row_stride;
  r.n_dst = t.n_dst;
  r.dst_list = t.dst_list;
  const uint32_t total = slot_geometry(t.dst_off, t.rows, t.row_bytes, t.dst_row_stride, t.vec_bytes, r.slots, lines);
  r.slots |= source_lines(t.src_off, t.dst_off, t.rows, t.row_bytes, t.src_row_stride, r.slots);
  for (r.first = 0; r.first < total; r.first = r.end) {
    r.end = std::min(r.first + unit - (on_kib ? slots_into_kib(r) : 0), total);
    take(r);
  }
}

// Bytes of slots per record.  Every record of a list takes the same number of workgroups, so what a piece does not fill
// of its last record are workgroups with nothing to do; smaller records leave fewer of them, but there are more records to fetch.
// Looked for are units that leave at most one workgroup in nine empty, among lists of at most 64 Ki records (beyond that the list is long
// enough for the tile size to fit); where none is small enough, the smallest is taken.  Always a multiple
// of 8 KiB below the tile size: at 1 KiB per workgroup (the prefetched list's own) part k of any record runs on
// XCD k mod 8, so that a copy finds in L2 what the load-only record's part k has loaded, and an XCD fetches a record
// once for all its parts (units of any KiB: hidden 160, 272 MB 43.4 -> 44.3 us).  Larger
// workgroups on records below eight of them lose that, and still gain more from fewer empty ones: hidden 256, TP
// 8 -> 2, pieces of 22 to 64 KiB, us, records of 16 KiB against 64 KiB (cache-blocked, 8 KiB per workgroup)
// or against grids filled up to eight parts per record (prefetched, 256 lanes, 4 KiB): 257 MB 60 / 79 and
// 62 / 73, 1016 MB 246 / 320 and 252 / 285; hidden 512 and up level.
// Measured: a plan of 64-lane workgroups with 79 % of them empty (pieces of 24 to 64 KiB) 40.5 us for
// 79 MB, 14.5 us with 8 KiB records.
// `copies` receives the number of copy records.
enum class Units {
  // One-to-one lists: of the multiples of 8 KiB the one that costs least, a record as much as an empty KiB.  The largest half of the tile size
  // that fits (5-11 % empty) / this choice (1-3 %), us: hidden 384, back, 20 MB 4.63 / 4.41, hidden 640, back, 39 MB 7.06 / 6.86, hidden 1280, 78
  // MB 12.44 / 12.28, hidden 640, 1.9 GB 300.7 / 295.4, hidden 1280, 2.5 GB 397.5 / 391.1; 22 ways back of 0.09 to 3.7 GB together 0.3 % ahead, none
  // more than 0.4 % behind.  A record as much as 8 empty KiB or as a third of one: level.  Once one fits, finer ones only up to 24 Ki
  // records: with up to 64 Ki the same 22 are level (0.994 to 1.005) and a plan can take longer (3.2 GB, 50 Ki records for 19 Ki: 10.2 ms for 5.8).
  kMultiples,
  // The largest half of the tile size that fits.  The automatic list: the half that costs least is level (40 lists with two to seven destinations 0.992 to
  // 1.006, together 1.000; source cold 1.002) and has up to four times the records, of the units in between those of 96 to 120 KiB are 1-4 % behind (us, hidden 512
  // joined, 2.8 GB, 64 / 96 / 112 / 128 KiB: 457.2 469.3 472.7 458.9).  Lists whose later passes want the XCD of the first, at whatever workgroup they are run:
  // cache-blocked, 137 MB 20.9 us with records of 128 KiB, 23.9 with 72.
  kLargestHalf
};
struct PieceSizes {
  std::vector<std::pair<uint32_t, uint32_t>> kinds; // slots of a piece, how many pieces: a model has few
  uint64_t total = 0;
  size_t pieces = 0, last = 0;
  // `empty`: what the piece's first record leaves empty in front of it (on_kib, see cut_tile)
  void add(uint32_t slots, uint32_t empty = 0) {
    ++pieces;
    total += slots;
    slots += empty;
    if (last == kinds.size() || kinds[last].first != slots) {
      for (last = 0; last < kinds.size() && kinds[last].first != slots;) ++last;
      if (last == kinds.size()) kinds.push_back({slots, 0});
    }
    ++kinds[last].second;
  }
};
uint32_t choose_unit(const Plan &pl, const PieceSizes &sizes, size_t &copies, Units units) {
  copies = sizes.pieces;
  if (sizes.pieces > 65536) return (uint32_t)pl.tile_bytes;
  uint32_t best = (uint32_t)pl.tile_bytes;
  uint64_t least = ~0ull;
  for (uint64_t unit = best;; unit = units == Units::kMultiples ? (unit - 1) / 8192 * 8192 : unit / 2) {
    const uint32_t slots = (uint32_t)unit / kSlot;
    uint64_t records = 0;
    for (const auto &k : sizes.kinds) records += (uint64_t)k.second * ((k.first + slots - 1) / slots);
    if (records > (least == ~0ull ? 65536u : 24576u)) break;
    const bool fits = records * slots <= sizes.total + sizes.total / 8;
    const uint64_t cost = fits ? records * (unit / 1024 + 1) : ~0ull;
    if (cost < least || least == ~0ull) {
      best = (uint32_t)unit;
      least = cost;
      copies = records;
    }
    if (units == Units::kMultiples ? unit <= 8192 : unit % 16384 || fits) break;
  }
  return best;
}

// Whether tile `b` goes on where `a` ends, on both sides and in the same rows; if so, `a` becomes the two.  Records are cut
// from the whole, so that a piece has one remainder and not one of the tile size beside one of its own.  Up to
// 128 MiB on either side: a row has fewer than 2^24 slots, and offsets stay below 4 GiB.  Lists of more than 64 Ki tiles,
// whose unit is the tile size anyway, keep their tiles: rows that begin with a record are 0.4 % ahead there (Llama-7B
// back 4162 us, joined 4178).
bool join(hf_tile &a, const hf_tile &b) {
  constexpr uint64_t kLongest = 1u << 27;
  if (a.n_dst != 1 || b.n_dst != 1) return false;
  if (a.rows == 1 && b.rows == 1) {
    if (a.src_off + a.row_bytes != b.src_off || a.dst_off + a.row_bytes != b.dst_off || (uint64_t)a.row_bytes + b.row_bytes > kLongest) return false;
    a.row_bytes += b.row_bytes;
  } else {
    const uint64_t rows = (uint64_t)a.rows + b.rows;
    if (a.rows == 1 || a.row_bytes != b.row_bytes || a.src_row_stride != b.src_row_stride || a.dst_row_stride != b.dst_row_stride ||
        a.src_off + (uint64_t)a.rows * a.src_row_stride != b.src_off || a.dst_off + (uint64_t)a.rows * a.dst_row_stride != b.dst_off ||
        rows * std::max(a.src_row_stride, a.dst_row_stride) > kLongest)
      return false;
    a.rows = (uint32_t)rows;
  }
  a.vec_bytes = std::min(a.vec_bytes, b.vec_bytes);
  return true;
}
std::vector<hf_tile> join_tiles(const hf_tile *t, size_t n) {
  std::vector<hf_tile> pieces;
  for (size_t i = 0; i < n; ++i)
    if (pieces.empty() || !join(pieces.back(), t[i])) pieces.push_back(t[i]);
  return pieces;
}

uint32_t choose_unit(const Plan &pl, const hf_tile *t, size_t n, size_t &copies, Units units) {
  copies = n;
  if (n > 65536) return (uint32_t)pl.tile_bytes;
  PieceSizes sizes; // of the copy tiles
  for (size_t i = 0; i < n; ++i) {
    uint32_t unused;
    if (t[i].n_dst) sizes.add(slot_geometry(t[i].dst_off, t[i].rows, t[i].row_bytes, t[i].dst_row_stride, t[i].vec_bytes, unused));
  }
  return choose_unit(pl, sizes, copies, units);
}

// unit: bytes of slots per record, 0 = see choose_unit; `one_to_one`: see DevList, the tiles are joined to pieces first
void compile_list(const Plan &pl, const hf_tile *t, size_t n, uint32_t unit_bytes, bool one_to_one, DevList &out, bool lines = true) {
  out.tiles.clear();
  out.one_to_one = one_to_one;
  std::vector<hf_tile> pieces;
  if (one_to_one && n <= 65536) {
    pieces = join_tiles(t, n);
    t = pieces.data();
    n = pieces.size();
  }
  size_t records = n;
  if (unit_bytes)
    for (size_t i = 0; i < n; ++i) records += (uint64_t)t[i].rows * t[i].row_bytes / unit_bytes;
  out.unit_bytes = unit_bytes ? unit_bytes : choose_unit(pl, t, n, records, one_to_one ? Units::kMultiples : Units::kLargestHalf);
  out.tiles.reserve(records);
  out.bytes = 0;
  out.short_rows = false;
  uint64_t written = 0, in_part = 0; // lines
  const uint32_t unit = out.unit_bytes / kSlot;
  for (size_t i = 0; i < n; ++i) {
    const uint64_t payload = (uint64_t)t[i].rows * t[i].row_bytes;
    out.short_rows = out.short_rows || t[i].row_bytes < kSlot;
    out.bytes += payload * (1 + t[i].n_dst);
    written += payload / 128;
    if (t[i].rows > 1 && t[i].dst_row_stride != t[i].row_bytes) // both ends of a row, or its end
      in_part += (uint64_t)t[i].rows * ((t[i].dst_off | t[i].dst_row_stride) % 128 ? 2 : t[i].row_bytes % 128 ? 1 : 0);
    cut_tile(t[i], unit, [&](const DevTile &r) { out.tiles.push_back(r); }, lines);
  }
  out.parts_of_lines = in_part * 16 > written;
}

// the prefetched list: in front of the copy records of every block, load-only records with the
// slots of its shared copy records, so that the workgroup with part number k loads just what the
// copying workgroup with part number k will want.  Up to prefetch_merge copy records of the same
// geometry whose sources follow one another share one.
void compile_prefetched_list(const Plan &pl, const std::vector<hf_tile> &t, DevList &out) {
  out.tiles.clear();
  size_t records;
  out.unit_bytes = choose_unit(pl, t.data(), t.size(), records, Units::kLargestHalf);
  out.tiles.reserve(records + records / 2);
  out.bytes = 0;
  const uint32_t merge = (uint32_t)std::max<int64_t>(1, std::min<int64_t>(pl.effective_prefetch_merge(), HF_MAX_PREFETCH_CHUNKS));
  struct Copy { DevTile t; uint64_t step; }; // step: distance to the source of a tile that follows it
  std::vector<Copy> copies;
  // (source, first slot) of a copy record that would join a load-only record of its block: a hash
  // table that forgets with the block
  struct Open { uint64_t src; uint32_t first; uint32_t block; size_t at; };
  std::vector<Open> table(256, Open{0, 0, 0, 0});
  uint32_t block = 0;
  const auto slot_of = [&](uint64_t src, uint32_t first) -> Open & { // the entry of the key, or a free one
    size_t h = (size_t)(((src >> 1) + first * 0x9E3779B9ull) * 0x9E3779B97F4A7C15ull >> 32);
    for (;; ++h) {
      Open &o = table[h & (table.size() - 1)];
      if (o.block != block || (o.src == src && o.first == first)) return o;
    }
  };
  const size_t none = ~(size_t)0;
  for (size_t i = 0; i < t.size();) {
    copies.clear();
    ++block;
    while (i < t.size() && t[i].n_dst == 0) ++i;
    for (; i < t.size() && t[i].n_dst != 0; ++i) {
      const uint64_t step = t[i].rows > 1 ? (uint64_t)t[i].rows * t[i].src_row_stride : t[i].row_bytes;
      out.bytes += (uint64_t)t[i].rows * t[i].row_bytes * (1 + t[i].n_dst);
      cut_tile(t[i], out.unit_bytes / kSlot, [&](const DevTile &r) { copies.push_back({r, step}); });
    }
    if (table.size() < 4 * copies.size()) {
      size_t n = table.size();
      while (n < 4 * copies.size()) n *= 2;
      table.assign(n, Open{0, 0, 0, 0});
    }
    for (const Copy &copy : copies) {
      const DevTile &c = copy.t;
      // a piece with one destination is read once anyway; rows below a slot are not loaded ahead: the
      // loads are of whole slots, which such a row does not hold (the next bytes may be another's, or nobody's)
      if (c.n_dst == 1 || c.row_bytes < kSlot) continue;
      const uint64_t step = copy.step, next = c.src_off + step;
      Open &mine = slot_of(c.src_off, c.first);
      if (mine.block == block && mine.at != none) {
        DevTile &pre = out.tiles[mine.at];
        if (pre.end == c.end && pre.row_bytes == c.row_bytes && pre.slots == (c.slots & ~kSharesLines) && pre.src_row_stride == c.src_row_stride &&
            pre.dst_list == step) {
          if (((++pre.n_dst) & ~kLoadOnly) < merge) slot_of(next, c.first) = Open{next, c.first, block, mine.at};
          mine.at = none;
          continue;
        }
      }
      DevTile pre = c;
      pre.slots &= ~kSharesLines; // loaded plainly anyway
      pre.n_dst = kLoadOnly | 1u;
      pre.dst_list = (uint32_t)step;
      if (merge > 1 && step < (1ull << 32)) slot_of(next, c.first) = Open{next, c.first, block, out.tiles.size()};
      out.tiles.push_back(pre);
    }
    for (const Copy &copy : copies) out.tiles.push_back(copy.t);
  }
}

// Whether the stripes `set` of a row-parallel tensor can go as a band, and the band: stripe k of the rows of every
// destination from pages that lie evenly apart, at most one stripe per destination left out.
struct Band {
  DevTile t;
  uint32_t total = 0;             // slots in all
  std::vector<uint64_t> members;  // entries of the destination list
  // while it is made: the stripes' sources, and which stripes a destination takes (how many, and the sum of their numbers)
  struct Member { int rank; uint64_t at; uint32_t stripes, sum; };
  std::vector<uint64_t> src;
  std::vector<Member> takers;
};
bool make_band(const Plan &pl, const Groups &groups, const std::vector<size_t> &set, Band &band) {
  const hf_desc &d0 = *groups[set[0]][0];
  const uint32_t row = (uint32_t)d0.dst_row_stride, piece = d0.row_bytes, a = row / piece;
  const uint64_t bytes = (uint64_t)d0.rows * row;
  if (set.size() < 2 || a < 2 || row % piece || a != (uint32_t)pl.a || a > 254 || piece < kSlot || row > kBandLargest || (uint64_t)pl.tile_bytes > kBandLargest ||
      d0.n_blocks != 1 || bytes % kSlot || bytes >= 1ull << 32)
    return false;
  const bool apart = d0.src_row_stride != piece;
  if (apart && d0.src_row_stride != row) return false;
  const uint64_t unknown = ~0ull;
  std::vector<uint64_t> &src = band.src;
  std::vector<Band::Member> &members = band.takers;
  src.assign(a, unknown);
  members.clear();
  for (size_t gi : set) {
    size_t m = 0; // the destinations of all stripes come in the same order
    for (const hf_desc *d : groups[gi]) {
      const uint32_t k = (uint32_t)(pl.coords[d->src_rank].tp - pl.coords[d->dst_rank].gtp * pl.a);
      const uint64_t at = d->dst_off - (uint64_t)k * piece, from = d->src_off - (apart ? (uint64_t)k * piece : 0);
      if (k >= a || d->rows != d0.rows || d->row_bytes != piece || d->dst_row_stride != row || d->src_row_stride != d0.src_row_stride ||
          d->n_blocks != 1 || at % 128 || (src[k] != unknown && src[k] != from))
        return false;
      src[k] = from;
      size_t looked = 0;
      while (looked < members.size() && members[m % members.size()].rank != d->dst_rank) { ++m; ++looked; }
      if (looked == members.size()) {
        m = members.size();
        members.push_back({d->dst_rank, at, 0, 0});
      }
      Band::Member &mem = members[m % members.size()];
      if (mem.at != at) return false;
      ++mem.stripes;
      mem.sum += k;
      ++m;
    }
  }
  const uint64_t step = src[0] != unknown && src[1] != unknown && src[1] > src[0] ? src[1] - src[0] : 0;
  if (!step || step % 4096 || step >> 44 || members.size() >= 65536) return false;
  for (uint32_t k = 0; k < a; ++k)
    if (src[k] != src[0] + k * step) return false; // all stripes are wanted by somebody, so all are looked at
  uint64_t first = unknown;
  for (const Band::Member &m : members) first = std::min(first, m.at);
  band.members.clear();
  for (const Band::Member &m : members) {
    if (m.stripes + 1 < a) return false;
    const uint64_t skip = m.stripes < a ? a * (a - 1) / 2 - m.sum + 1 : 0;
    // one destination alone would leave lanes idle, and has no neighbours to join where it skips one of two
    if (skip && members.size() == 1) return false;
    band.members.push_back(skip << 56 | (m.at - first));
  }
  std::memset(&band.t, 0, sizeof band.t);
  band.t.src_off = src[0];
  band.t.dst_off = first;
  band.t.row_bytes = piece;
  band.t.src_row_stride = (uint32_t)(step >> 12);
  band.t.dst_row_stride = row;
  const bool edges = piece % 128 && std::any_of(band.members.begin(), band.members.end(), [](uint64_t e) { return e >> 56; });
  band.t.n_dst = kBand | (apart ? kBandApart : 0u) | (edges ? kBandParts : 0u) | (uint32_t)band.members.size();
  band.total = (uint32_t)(bytes / kSlot);
  return true;
}

// one record per tile, whatever its slots come to
void compile_whole_tiles(const hf_tile *t, size_t n, DevList &out) {
  uint32_t most = 0, unused;
  for (size_t i = 0; i < n; ++i)
    most = std::max(most, slot_geometry(t[i].dst_off, t[i].rows, t[i].row_bytes, t[i].dst_row_stride, t[i].vec_bytes, unused));
  out.unit_bytes = (uint32_t)round_up((uint64_t)most * kSlot, 8192);
  out.tiles.reserve(n);
  for (size_t i = 0; i < n; ++i) {
    out.bytes += (uint64_t)t[i].rows * t[i].row_bytes * (1 + t[i].n_dst);
    cut_tile(t[i], most, [&](const DevTile &r) { out.tiles.push_back(r); });
  }
}

} // namespace

// The limit of hf_reshard_execute_static counts tiles of tile_bytes of payload (48 bytes each, a
// load-only one like any other) and extra destinations (8 bytes).  The records that are staged are cut by
// slots: for odd rows there are more of them than of those tiles, up to one in eight for rows of some
// length, more for rows of a few slots.  So the count is taken from the descriptors, and where a list
// that the limit admits has more records than the array holds (`room`), it is staged in a form of one
// record per counted copy tile, without load-only records; that form is never larger than the count.
void build_static_list(Plan &pl, uint64_t limit, uint64_t room) {
  pl.dev_static = DevList();
  pl.static_dst.clear();
  const int64_t mode = pl.effective_multicast();
  const bool listed_dst = pl.active_fwd_uses_mc_dst();
  const auto bytes = [&](uint64_t tiles) { return round_up(tiles * sizeof(hf_tile), 256) + (listed_dst ? pl.payload_mc.extra * sizeof(uint64_t) : 0); };
  // between `least` and `most` tiles, the same wherever it can be told without making them
  uint64_t least = pl.payload_mc.tiles, most = least;
  if (mode == HF_MULTICAST_OFF) {
    least = 0;
    for (const hf_desc &d : pl.fwd_peer) if (wanted(pl, d)) least += payload_tiles(d, (uint64_t)pl.tile_bytes);
    if (pl.flags & HF_COPY_OWN)
      for (const hf_desc &d : pl.fwd_own) if (wanted(pl, d)) least += payload_tiles(d, (uint64_t)pl.tile_bytes);
    most = least;
  } else if (mode == HF_MULTICAST_CACHE_BLOCKED) {
    least = most = pl.payload_mc.tiles + pl.payload_mc.extra;
  } else if (mode == HF_MULTICAST_PREFETCHED) {
    least += pl.payload_mc.shared / std::max<uint64_t>(1, std::min<uint64_t>(pl.effective_prefetch_merge(), HF_MAX_PREFETCH_CHUNKS));
    most += pl.payload_mc.shared;
  }
  pl.static_bytes = bytes(least);
  const uint64_t staged = round_up(pl.dev_fwd.tiles.size() * sizeof(DevTile), 256) + (listed_dst ? pl.mc_dst.size() * sizeof(uint64_t) : 0);
  if (bytes(least) > limit || (bytes(most) <= limit && staged <= room)) return;
  // the payload tiles themselves, in the place of the plan's lists
  DevList list;
  std::vector<uint64_t> dst;
  {
    struct Aside {
      Plan &pl;
      WorkLists lists;
      explicit Aside(Plan &p) : pl(p), lists(std::move(static_cast<WorkLists &>(p))) {
        static_cast<WorkLists &>(pl) = WorkLists();
        pl.multicast = lists.multicast;
      }
      ~Aside() { static_cast<WorkLists &>(pl) = std::move(lists); }
    } aside(pl);
    std::string err;
    const Groups groups = sharing_groups(pl);
    (void)build_multicast_list(pl, groups, stripe_siblings(pl, groups), err, Measure::kPayload); // fewer destinations than the list that was built before
    const std::vector<hf_tile> *tiles = &pl.tiles_fwd_mc;
    if (mode == HF_MULTICAST_OFF) {
      tile_list(pl, pl.fwd_peer, pl.tiles_fwd, Measure::kPayload);
      if (pl.flags & HF_COPY_OWN) tile_list(pl, pl.fwd_own, pl.tiles_fwd, Measure::kPayload);
      tiles = &pl.tiles_fwd;
    } else if (mode == HF_MULTICAST_CACHE_BLOCKED) {
      build_cache_blocked_list(pl, pl.tiles_fwd_cb);
      tiles = &pl.tiles_fwd_cb;
    } else if (mode == HF_MULTICAST_PREFETCHED) {
      build_prefetched_list(pl, pl.tiles_fwd_pf);
      aside.lists.static_bytes = bytes(pl.tiles_fwd_pf.size());
    }
    if (aside.lists.static_bytes <= limit && staged > room) {
      compile_whole_tiles(tiles->data(), tiles->size(), list);
      if (listed_dst) dst = std::move(pl.mc_dst);
    }
  }
  pl.dev_static = std::move(list);
  pl.static_dst = std::move(dst);
}

void build_forward_lists(Plan &pl) {
  pl.tiles_fwd_cb.clear();
  pl.tiles_fwd_pf.clear();
  if (pl.effective_multicast() == HF_MULTICAST_CACHE_BLOCKED) build_cache_blocked_list(pl, pl.tiles_fwd_cb);
  if (pl.effective_multicast() == HF_MULTICAST_PREFETCHED) {
    build_prefetched_list(pl, pl.tiles_fwd_pf);
    compile_prefetched_list(pl, pl.tiles_fwd_pf, pl.dev_fwd);
  } else {
    compile_list(pl, pl.active_fwd().data(), pl.active_fwd_count(), 0, !pl.has_sharing, pl.dev_fwd);
  }
  build_static_list(pl, HF_STATIC_SCRATCH_BYTES, kStaticRoom);
}

// What hf_reshard_execute runs while every choice is the library's, where pieces are shared: every piece loaded once
// and stored to each destination, without load-only records, row-parallel tensors as bands; destinations as
// distances from the first, which are the same for all tensors that one set of ranks wants, so that the
// list of them is short and stays in the scalar caches.
void build_auto_list(Plan &pl, const Groups &groups, const Siblings &siblings) {
  pl.dev_auto = DevList();
  pl.auto_dst.clear();
  pl.auto_joins = false;
  if (!pl.has_sharing) return;
  std::map<std::vector<uint64_t>, uint32_t> known;
  const auto listed = [&](const std::vector<uint64_t> &d) {
    const auto it = known.emplace(d, (uint32_t)pl.auto_dst.size());
    if (it.second) pl.auto_dst.insert(pl.auto_dst.end(), d.begin(), d.end());
    return it.first->second;
  };
  // pieces stay whole up to here, records are cut from them; a row of this length has fewer than 2^24 slots
  constexpr uint64_t kLongest = 1u << 27;
  std::vector<hf_tile> tiles;
  std::vector<DevTile> bands;  // the place of a band in `tiles` is an entry without rows
  std::vector<uint32_t> band_slots;
  std::vector<char> emitted(groups.size(), 0);
  std::vector<std::vector<hf_tile>> parts;
  std::vector<uint64_t> dst;
  Band band;
  tiles.reserve(groups.size());
  for (size_t gi = 0; gi < groups.size(); ++gi) {
    if (emitted[gi]) continue;
    const hf_desc &d0 = *groups[gi][0];
    std::vector<size_t> set{gi};
    if (d0.kind == HF_ROW) {
      const Coords &c = pl.coords[d0.dst_rank];
      set = siblings.at(SibKey{d0.tensor_id, d0.layer, c.dp, c.gpp, c.gtp});
      if (pl.row_interleave && make_band(pl, groups, set, band)) {
        for (size_t g2 : set) emitted[g2] = 1;
        band.t.dst_list = listed(band.members);
        hf_tile place;
        std::memset(&place, 0, sizeof place);
        tiles.push_back(place);
        bands.push_back(band.t);
        band_slots.push_back(band.total);
        pl.auto_joins = pl.auto_joins || band.t.row_bytes % kSlot;
        continue;
      }
      if (!pl.row_interleave) set.assign(1, gi);
    }
    parts.assign(set.size(), {});
    size_t longest = 0;
    for (size_t k = 0; k < set.size(); ++k) {
      const auto &g = groups[set[k]];
      emitted[set[k]] = 1;
      tile_desc(parts[k], *g[0], set.size() > 1 ? (uint64_t)pl.tile_bytes : kLongest, Measure::kSlots);
      dst.clear();
      for (size_t j = 1; j < g.size(); ++j) dst.push_back(g[j]->dst_off - g[0]->dst_off);
      const uint32_t list = listed(dst);
      uint64_t align = 0;
      for (uint64_t d : dst) align |= d;
      for (hf_tile &t : parts[k]) {
        t.n_dst = (uint32_t)g.size();
        t.dst_list = list;
        t.vec_bytes = vec_of(t.vec_bytes | align);
      }
      longest = std::max(longest, parts[k].size());
    }
    for (size_t i = 0; i < longest; ++i)
      for (const auto &p : parts)
        if (i < p.size()) tiles.push_back(p[i]);
  }
  pl.dev_auto.bytes = pl.moved_bytes[0] + pl.unique_bytes[0];
  // About two destinations: the registers list, whose second destinations arrive late and so spread the stores by
  // themselves, is ahead where bands join nothing and the list is long.  GB, us, this list / registers: 0.18 26.1 /
  // 27.2; 3.1 482 / 473, 7.4 1164 / 1134; joined 0.53 83.9 / 86.4, 1.7 266 / 275, 4.1 636 / 654.
  if (pl.fan_out() < 2.5 && !pl.auto_joins && pl.dev_auto.bytes > 256ull << 20) {
    pl.auto_dst.clear();
    return;
  }
  PieceSizes sizes;
  size_t records = 0, band_at = 0;
  for (const hf_tile &t : tiles) {
    DevTile r = t.rows ? DevTile() : bands[band_at];
    uint32_t n;
    if (t.rows) {
      n = slot_geometry(t.dst_off, t.rows, t.row_bytes, t.dst_row_stride, t.vec_bytes, r.slots);
      r.dst_off = t.dst_off;
    } else {
      n = band_slots[band_at++];
    }
    sizes.add(n, slots_into_kib(r));
  }
  pl.dev_auto.unit_bytes = choose_unit(pl, sizes, records, Units::kLargestHalf);
  const uint32_t unit = pl.dev_auto.unit_bytes / kSlot;
  pl.dev_auto.tiles.reserve(records);
  size_t next = 0;
  for (const hf_tile &t : tiles) {
    if (t.rows) {
      cut_tile(t, unit, [&](const DevTile &r) { pl.dev_auto.tiles.push_back(r); }, true, true);
      continue;
    }
    DevTile r = bands[next];
    const uint32_t total = band_slots[next++];
    for (r.first = 0; r.first < total; r.first = r.end) {
      r.end = std::min(r.first + unit - slots_into_kib(r), total);
      r.slots = (uint32_t)((uint64_t)r.first * kSlot / r.dst_row_stride);
      pl.dev_auto.tiles.push_back(r);
    }
  }
  pl.auto_dst.push_back(0); // the kernel looks at the entry behind a record's own, and at one where it has none
}

// How the automatic list is launched.  us for whole calls, hidden 1024 and
// (joined slots: stripes of 1026 bytes) hidden 768, plain loads with system-scope stores and all wavefronts that fit / 25
// a CU / 21 a CU | non-temporal stores, the same three | the prefetched list:
//   3 destinations, 4.1 GB 653 675 730 | 680 637 676 | 689; joined, 2.3 GB 385 412 434 | 373 388 413 | 419
//   4, 5.2 GB              857 807 854 | 881 826 798 | 853; joined, 2.9 GB 471 482 520 | 475 452 480 | 518
//   7, 8.3 GB             1447 1351 1392 | 1495 1462 1417 | 1477; joined, 7.6 GB 1349 1275 1319 | 1412 1384 1340 | 1541
// Five and six destinations (TP 6 -> 1, without and with own pieces), system-scope stores, 25 a CU | non-temporal, 25 a CU: hidden 768, 1.4 GB 220 | 221, 1.6 GB 249 | 270, hidden
// 1536, 2.8 GB 445 | 472, 3.3 GB 514 | 563, joined 460 | 474, 527 | 559.
// Four destinations and records of 8 KiB, where pieces are short: eight wavefronts share the fetch of one and each waits for it longer, so that stores are
// wanted that are acknowledged sooner, once the memory-side cache no longer takes a good part of them.  System-scope / non-temporal, 25 a CU: hidden
// 256, 504 MB 83.8 / 80.2, 745 MB 125.2 / 120.6, TP 8 -> 2, 840 MB 145.9 / 138.5, hidden 192, 441 MB 71.4 / 69.7; below, hidden 256, 323 MB 46.9 / 47.8, hidden 288, 422 MB 63.3
// / 64.2 (8 lists of 270 to 431 MB 1.5 % behind, 19 from 441 MB to 1.9 GB 2.5 % ahead).  Three destinations and short records: all wavefronts that fit are ahead by up to
// 3 % at some (hidden 384, 931 MB 154.7 with 25 a CU / 152.2) and behind by up to 10 % at others (TP 8 -> 2, hidden 320, 1.0 GB 191.3 / 210.9; hidden 192 out of the generation
// buffers, 366 MB 68.0 / 74.4), 35 lists together 2.2 % behind.
// What these lines miss: joined slots at three destinations and hidden 1536 and up, 1.9 GB 305 with all that fit, 296 with 25 a CU; four and five destinations of
// pieces of 16 KiB, hidden 384, 1.7 GB 283 with system-scope stores, 274 with non-temporal ones, 679 MB 123 / 113.
// Lists of 32 to 300 MB are level or 1-4 % ahead with the same choices.  System-scope stores take longer to be
// acknowledged, and lanes that join two stripes to get there: either wants more wavefronts.  About two destinations (build_auto_list
// says when): not paced, 1.7 GB joined 266 | 271, paced 278 | 279.  What one line by destinations misses: four of them at hidden 8192 with
// own pieces, 84 GB (34B shape, one micro-DP group), ms: 12.70, the registers list 12.12, the prefetched one 12.76-13.45.
// Up to 32 MiB the stores of a call do not pile up, and single wavefronts are handed out no faster than they finish: eight wavefronts to a
// workgroup, not paced, non-temporal stores (two destinations: system-scope).  Against paced wavefronts, rows of calls (a replayed graph of 60, three sets of buffers in turn) | one call
// that is waited for, 15 to 20 us with the host's part, on the same buffers | after an optimizer step over the source | source cold after 1 GiB of reads | after 1 GiB of other writes: 49 lists with three
// destinations 0.99 (0.89-1.06) | 0.99 | 0.99 | 0.98 | 1.00, 29 with four 0.94 | 0.99 | 0.98 | 0.96 | 0.98, 6 with seven and eight 0.88 | 0.96 | 0.95 | 0.94 | 0.96 (30 MB 7.11 / 6.15 us); 20
// with two (not paced before either), kernels alone, 0.97 | 0.97 | 0.94 | 1.00 | 1.02.  System-scope stores instead: at three destinations 1.03 of these (0.88-1.37).  Above 32 MiB it is ahead only where the
// source is in the caches: three, joined 74 MB 12.84 / 12.54 | 17.84 / 17.92 | 20.76 / 21.52 (us; source cold, after writes).  From five destinations on twice that: seven 60 MB
// 11.00 / 10.57 | 16.64 / 15.92 | 17.80 / 17.12, 111 MB 18.59 / 18.21 | 25.16 / 25.96 | 27.60 / 29.60.
constexpr uint64_t kShortAutoList = 32ull << 20;
AutoLaunch auto_launch(const Plan &pl) {
  const double fan = pl.fan_out();
  const uint64_t bytes = pl.dev_auto.bytes;
  AutoLaunch a;
  a.short_list = bytes <= (fan < 5 ? kShortAutoList : 2 * kShortAutoList);
  a.paced = fan >= 2.5 && !a.short_list;
  const bool short_records = pl.dev_auto.unit_bytes <= 8192 && bytes > 416ull << 20;
  a.policy = fan >= 2.5 && (a.short_list || fan < 3.5 || (fan < 5 && (pl.auto_joins || short_records))) ? 5 : 1;
  a.wgs_per_cu = !a.paced || (fan < 3.5 && pl.auto_joins) ? 0 : 25;
  return a;
}

// Short one-to-one lists that write many lines in part: non-temporal stores from 12 MiB on, system-scope ones below.  Non-temporal against
// system-scope, 62 lists, up to 10 MB / 12 / 14 / 17 / 19 / 25: three sets of buffers in turn, calls in a replayed graph 0.99 0.97 0.94 0.92 0.90 0.93; a
// call alone that is waited for, in all of 14 to 16 us, the same buffers 1.045 1.055 1.03 1.02 0.99 0.97, after an optimizer step over the source 1.00 0.99 0.99 0.98 0.97
// 0.97.  So below the line a call alone would take longer than with single wavefronts (1.02; 0.97 with system-scope stores), for little in a row of calls.  Lists of whole lines
// stay with system-scope stores: 21 MB 3.71 / 3.74 and 3.44 / 3.69.
bool non_temporal_when_short(const DevList &list) { return list.parts_of_lines && list.bytes >= 12ull << 20; }

int build_tiles(Plan &pl, std::string &err) {
  if (pl.tile_bytes < 4096 || pl.tile_bytes > (4 << 20) || pl.tile_bytes % 4096) {
    err = "tile bytes must be a multiple of 4096 in [4096, 4 MiB]";
    return HF_EINVAL;
  }
  build_plain_lists(pl);
  cache_totals(pl);
  const Groups groups = sharing_groups(pl);
  const Siblings siblings = stripe_siblings(pl, groups);
  if (int rc = build_multicast_list(pl, groups, siblings, err)) return rc;
  if (pl.multicast_auto) pl.multicast = default_multicast(pl);
  if (pl.tiles_fwd.size() >= (1ull << 31) || pl.tiles_back.size() >= (1ull << 31)) {
    err = "too many tiles; raise the tile size";
    return HF_ERANGE;
  }
  build_forward_lists(pl);
  build_auto_list(pl, groups, siblings);
  compile_list(pl, pl.tiles_fwd.data() + pl.n_tiles_fwd_peer, pl.tiles_fwd.size() - pl.n_tiles_fwd_peer, 0, true, pl.dev_own);
  compile_list(pl, pl.tiles_back.data(), pl.tiles_back.size(), 0, true, pl.dev_back);
  // The eight workgroups of a reload take the records in turn, and each has to wait for the link: 32 KiB (one batch) keep
  // them busy to the end where pieces of two sizes alternate.  GB/s in, records of 128 / 32 KiB: Llama-7B 56.8 /
  // 57.0, hidden 640 (pieces of 50 to 200 KiB) 52.1 / 56.9, hidden 1040 53.9 / 55.8, hidden 256 50.9 / 54.2.  Out, where stores are
  // not waited for, 128 KiB are ahead (55.4 / 52.9).
  compile_list(pl, pl.tiles_offload.data(), pl.tiles_offload.size(), (uint32_t)pl.tile_bytes, false, pl.dev_offload);
  compile_list(pl, pl.tiles_reload.data(), pl.tiles_reload.size(), (uint32_t)std::min<int64_t>(pl.tile_bytes, 32768), false, pl.dev_reload, false);
  return HF_OK;
}

// ---- validation -------------------------------------------------------------------------
namespace {

struct Seg { uint64_t dst, src, len; };

void desc_segments(const hf_desc &d, std::vector<Seg> &out) {
  for (uint32_t b = 0; b < d.n_blocks; ++b)
    for (uint32_t r = 0; r < d.rows; ++r)
      out.push_back({d.dst_off + b * d.dst_block_stride + r * d.dst_row_stride,
                     d.src_off + b * d.src_block_stride + r * d.src_row_stride, d.row_bytes});
}

void tile_segments(const hf_tile &t, std::vector<Seg> &out) {
  for (uint32_t r = 0; r < t.rows; ++r)
    out.push_back({t.dst_off + (uint64_t)r * t.dst_row_stride, t.src_off + (uint64_t)r * t.src_row_stride, t.row_bytes});
}

// sort by destination and merge neighbours that are contiguous on both sides
bool normalise(std::vector<Seg> &v, std::string &err, const char *what) {
  std::sort(v.begin(), v.end(), [](const Seg &x, const Seg &y) { return x.dst < y.dst; });
  std::vector<Seg> m;
  for (const Seg &s : v) {
    if (!m.empty()) {
      Seg &l = m.back();
      if (l.dst + l.len > s.dst) { err = std::string(what) + ": overlapping destinations"; return false; }
      if (l.dst + l.len == s.dst && l.src + l.len == s.src) { l.len += s.len; continue; }
    }
    m.push_back(s);
  }
  v.swap(m);
  return true;
}

bool same(const std::vector<Seg> &x, const std::vector<Seg> &y) {
  if (x.size() != y.size()) return false;
  for (size_t i = 0; i < x.size(); ++i)
    if (x[i].dst != y[i].dst || x[i].src != y[i].src || x[i].len != y[i].len) return false;
  return true;
}

// what a band moves, one segment per stripe's row and destination, with every slot where its rows and stripes say
bool band_segments(const DevTile &t, const std::vector<uint64_t> &dst_list, std::vector<Seg> &out) {
  const uint32_t n = band_members(t), row = t.dst_row_stride, piece = t.row_bytes;
  if (!n || (uint64_t)t.dst_list + n >= dst_list.size() || piece < kSlot || row < piece || row % piece || row > kBandLargest || t.dst_off % 128) return false;
  if ((uint64_t)t.slots * row > (uint64_t)t.first * kSlot || (uint64_t)t.end * kSlot - (uint64_t)t.slots * row >= 1u << 24) return false;
  for (uint64_t at = (uint64_t)t.first * kSlot, to = (uint64_t)t.end * kSlot, len; at < to; at += len) {
    const BandSlot b = band_slot(t, (uint32_t)(at / kSlot));
    // from the slot's stripe on to the byte
    uint32_t r = b.row, k = b.stripe, in = b.at + (uint32_t)(at % kSlot);
    for (; in >= piece; in -= piece)
      if (++k == row / piece) { k = 0; ++r; }
    if ((uint64_t)r * row + k * piece + in != at) return false;
    len = std::min<uint64_t>(piece - in, to - at);
    for (uint32_t j = 0; j < n; ++j) {
      const uint64_t entry = dst_list[t.dst_list + j];
      if (entry >> 56 != k + 1) out.push_back({t.dst_off + (entry & kBandDistance) + at, band_source(t, r, k) + in, len});
    }
  }
  return true;
}

// what the copy records of a device list move, one segment per record and row, with every slot inside its
// row; and, block by block, whether the load-only records are those of the block's shared copy records
// (prefetched), or there are none
bool record_segments(const DevList &l, const std::vector<uint64_t> &dst_list, bool prefetched, bool distances, std::vector<Seg> &out) {
  typedef std::tuple<uint64_t, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t> Key;
  std::vector<Key> loads, shared;
  const auto same_keys = [&]() {
    std::sort(loads.begin(), loads.end());
    std::sort(shared.begin(), shared.end());
    const bool ok = loads == shared;
    loads.clear();
    shared.clear();
    return ok;
  };
  bool copying = false;
  for (const DevTile &t : l.tiles) {
    if (distances && (t.dst_list >= dst_list.size() || (uint64_t)(t.end - t.first + slots_into_kib(t)) * kSlot > l.unit_bytes)) return false;
    if (distances && (t.n_dst & kBand) == kBand) {
      if (t.first >= t.end || (uint64_t)(t.end - t.first) * kSlot > l.unit_bytes || !band_segments(t, dst_list, out)) return false;
      continue;
    }
    const bool load_only = t.n_dst & kLoadOnly;
    const uint32_t per_row = slots_per_row(t), chunks = load_only ? t.n_dst & ~kLoadOnly : 1;
    if (t.first >= t.end || (uint64_t)(t.end - t.first) * kSlot > l.unit_bytes || t.n_dst == 0 || t.row_bytes == 0) return false;
    if (load_only && (!prefetched || chunks == 0 || chunks > HF_MAX_PREFETCH_CHUNKS || t.row_bytes < kSlot)) return false;
    if (!load_only && t.n_dst > 1 && (uint64_t)t.dst_list + t.n_dst - 1 > dst_list.size()) return false;
    if (load_only && copying && !same_keys()) return false;
    copying = !load_only;
    for (uint32_t c = 0; c < chunks; ++c) {
      const Key key{t.src_off + (uint64_t)c * (load_only ? t.dst_list : 0), t.first, t.end, t.row_bytes, t.src_row_stride, t.slots & ~kSharesLines};
      if (load_only) loads.push_back(key);
      else if (t.n_dst > 1 && t.row_bytes >= kSlot) shared.push_back(key);
    }
    for (uint32_t first = t.first, end; first < t.end; first = end) {
      const uint32_t row = per_row ? first / per_row : 0;
      end = per_row ? std::min((row + 1) * per_row, t.end) : t.end;
      const uint64_t src_row = (uint64_t)row * t.src_row_stride, dst_row = (uint64_t)row * t.dst_row_stride;
      int64_t lo = 0, hi = t.row_bytes;
      if (t.row_bytes >= kSlot) {
        // the bytes of the row that slots [first, end) stand for, and the accesses at either end of them
        const int64_t lead = boundary_mask(t) ? (t.dst_off + dst_row) & boundary_mask(t) : 0;
        const int64_t from = (int64_t)(first - row * per_row) * kSlot - lead, to = (int64_t)(end - row * per_row) * kSlot - lead;
        lo = std::max<int64_t>(from, 0);
        hi = std::min<int64_t>(to, t.row_bytes);
        for (uint32_t i : {first, end - 1}) {
          uint32_t s, d;
          const bool live = slot_offsets(t, i, s, d);
          const int64_t at = (int64_t)s - (int64_t)src_row, want = (int64_t)(i - row * per_row) * kSlot - lead;
          if ((int64_t)d - (int64_t)dst_row != at || at < 0 || at + kSlot > t.row_bytes) return false;
          if (live != (want > -(int64_t)kSlot && want < (int64_t)t.row_bytes)) return false;
          if (live && at != std::max<int64_t>(0, std::min<int64_t>(want, t.row_bytes - kSlot))) return false;
        }
      } else if (per_row != 1 || boundary_mask(t)) {
        return false;
      }
      if (lo >= hi || load_only) continue;
      for (uint32_t j = 0; j < t.n_dst; ++j)
        out.push_back({(j ? dst_list[t.dst_list + j - 1] + (distances ? t.dst_off : 0) : t.dst_off) + dst_row + lo, t.src_off + src_row + lo, (uint64_t)(hi - lo)});
    }
  }
  return !prefetched || same_keys();
}

int train_id_of(int gen_id) {
  switch (gen_id) {
  case HF_G_EMBED: return HF_T_EMBED;
  case HF_G_HEAD: return HF_T_HEAD;
  case HF_G_LN1: return HF_T_LN1;
  case HF_G_LN2: return HF_T_LN2;
  case HF_G_LNF: return HF_T_LNF;
  case HF_G_Q: case HF_G_K: case HF_G_V: return HF_T_QKV;
  case HF_G_O: return HF_T_O;
  case HF_G_GATE: case HF_G_UP: return HF_T_GATE_UP;
  case HF_G_DOWN: return HF_T_DOWN;
  }
  return -1;
}

} // namespace

int validate_plan(const Plan &pl, std::string &err) {
  if (pl.kind_mask != 0x1F) { err = "plan is restricted to some descriptor kinds (hf_debug_restrict_kinds)"; return HF_EINVAL; }
  // (1) every descriptor stays inside the payload of the tensors it names
  auto inside = [&](const hf_desc &d, bool forward) -> bool {
    const int train_rank = forward ? d.src_rank : d.dst_rank, gen_rank = forward ? d.dst_rank : d.src_rank;
    const RankTable &tt = pl.train_tab[train_rank], &gt = pl.gen_tab[gen_rank];
    const TensorRec &tr = tt.at(train_id_of(d.tensor_id), d.layer), &gr = gt.at(d.tensor_id, d.layer);
    const uint64_t t0 = tt.base + tr.off, t1 = t0 + 2ull * tr.rows * tr.cols;
    const uint64_t g0 = gt.base + gr.off, g1 = g0 + 2ull * gr.rows * gr.cols;
    const uint64_t s_lo = d.src_off, s_hi = d.src_off + (d.n_blocks - 1) * d.src_block_stride + (d.rows - 1) * d.src_row_stride + d.row_bytes;
    const uint64_t d_lo = d.dst_off, d_hi = d.dst_off + (d.n_blocks - 1) * d.dst_block_stride + (d.rows - 1) * d.dst_row_stride + d.row_bytes;
    if (forward && (pl.flags & HF_GATHER_FROM_GEN) && d.src_rank != d.dst_rank) {
      const RankTable &sg = pl.gen_tab[d.src_rank];
      if (pl.mat_pos[d.src_rank] < 0) return false;
      const TensorRec &sr = sg.at(d.tensor_id, d.layer);
      const uint64_t q0 = sg.base + sr.off, q1 = q0 + 2ull * sr.rows * sr.cols;
      return s_lo >= q0 && s_hi <= q1 && d_lo >= g0 && d_hi <= g1;
    }
    if (forward) return s_lo >= t0 && s_hi <= t1 && d_lo >= g0 && d_hi <= g1;
    return s_lo >= g0 && s_hi <= g1 && d_lo >= t0 && d_hi <= t1;
  };
  for (const hf_desc &d : pl.fwd_peer) if (!inside(d, true)) { err = "peer descriptor leaves its tensor"; return HF_ERANGE; }
  for (const hf_desc &d : pl.fwd_own) if (!inside(d, true)) { err = "own descriptor leaves its tensor"; return HF_ERANGE; }
  for (const hf_desc &d : pl.back) if (!inside(d, false)) { err = "reverse descriptor leaves its tensor"; return HF_ERANGE; }

  // (2) destinations pairwise disjoint, and together exactly the payload
  std::vector<Seg> fwd, fwd_peer_only, back;
  for (const hf_desc &d : pl.fwd_peer) desc_segments(d, fwd);
  fwd_peer_only = fwd;
  for (const hf_desc &d : pl.fwd_own) desc_segments(d, fwd);
  for (const hf_desc &d : pl.back) desc_segments(d, back);
  uint64_t gen_payload = 0, train_payload = 0, fwd_total = 0, back_total = 0;
  for (int r : pl.mat) {
    for (const TensorRec &g : pl.gen_tab[r].tensors) gen_payload += 2ull * g.rows * g.cols;
    for (const TensorRec &s : pl.train_tab[r].tensors) train_payload += 2ull * s.rows * s.cols;
  }
  for (const Seg &s : fwd) fwd_total += s.len;
  for (const Seg &s : back) back_total += s.len;
  if (!normalise(fwd, err, "train->gen") || !normalise(back, err, "gen->train")) return HF_ERANGE;
  if (fwd_total != gen_payload) { err = "train->gen descriptors do not cover the generation payload"; return HF_ERANGE; }
  if (!(pl.flags & HF_GROUPING_VANILLA) && back_total != train_payload) {
    err = "gen->train descriptors do not cover the training payload";
    return HF_ERANGE;
  }

  // (3) the tiles are exactly the descriptors
  std::vector<Seg> tf, tf_peer, tb;
  for (size_t i = 0; i < pl.tiles_fwd.size(); ++i) {
    tile_segments(pl.tiles_fwd[i], tf);
    if (i + 1 == pl.n_tiles_fwd_peer) tf_peer = tf;
  }
  for (const hf_tile &t : pl.tiles_back) tile_segments(t, tb);
  if (!normalise(tf, err, "train->gen tiles") || !normalise(tb, err, "gen->train tiles") ||
      !normalise(tf_peer, err, "peer tiles") || !normalise(fwd_peer_only, err, "peer descriptors"))
    return HF_ERANGE;
  if (!same(tf, fwd) || !same(tb, back) || !same(tf_peer, fwd_peer_only)) { err = "tiles differ from descriptors"; return HF_ERANGE; }
  // the multicast list, expanded per destination, is the list execute would run one by one
  std::vector<Seg> mc;
  for (const hf_tile &t : pl.tiles_fwd_mc) {
    if (t.n_dst == 0 || (t.n_dst > 1 && (uint64_t)t.dst_list + t.n_dst - 1 > pl.mc_dst.size())) { err = "multicast tile: bad destination list"; return HF_ERANGE; }
    for (uint32_t k = 0; k < t.n_dst; ++k) {
      hf_tile one = t;
      one.dst_off = k == 0 ? t.dst_off : pl.mc_dst[t.dst_list + k - 1];
      uint64_t g = one.src_off | one.dst_off | one.row_bytes;
      if (one.rows > 1) g |= (uint64_t)one.src_row_stride | one.dst_row_stride;
      if (g % t.vec_bytes) { err = "multicast tile alignment wrong"; return HF_ERANGE; }
      tile_segments(one, mc);
    }
  }
  if (!normalise(mc, err, "multicast tiles")) return HF_ERANGE;
  if (!same(mc, (pl.flags & HF_COPY_OWN) ? fwd : fwd_peer_only)) { err = "multicast tiles differ from descriptors"; return HF_ERANGE; }
  std::vector<Seg> cb;
  std::vector<hf_tile> tiles_cb, tiles_pf; // whichever mode is in force
  build_cache_blocked_list(pl, tiles_cb);
  build_prefetched_list(pl, tiles_pf);
  for (const hf_tile &t : tiles_cb) {
    if (t.n_dst != 1) { err = "cache-blocked tile with several destinations"; return HF_ERANGE; }
    tile_segments(t, cb);
  }
  if (!normalise(cb, err, "cache-blocked tiles")) return HF_ERANGE;
  if (!same(cb, mc)) { err = "cache-blocked tiles differ from descriptors"; return HF_ERANGE; }
  // the prefetched list without its load-only tiles is the multicast list, and in every block
  // the load-only tiles read exactly the source bytes of the block's shared tiles
  {
    size_t k = 0;
    typedef std::pair<uint64_t, uint64_t> Run; // source offset, length
    std::vector<Run> pre, shared;
    auto tidy = [](std::vector<Run> &v) {
      std::sort(v.begin(), v.end());
      std::vector<Run> m;
      for (const Run &r : v) {
        if (!m.empty() && m.back().first + m.back().second == r.first) m.back().second += r.second;
        else m.push_back(r);
      }
      v.swap(m);
    };
    auto close_block = [&]() {
      tidy(pre);
      tidy(shared);
      const bool ok = pre == shared;
      pre.clear();
      shared.clear();
      return ok;
    };
    bool copying = false;
    for (const hf_tile &t : tiles_pf) {
      if (t.n_dst == 0) {
        if (copying && !close_block()) { err = "prefetched list: load-only tiles do not cover the shared tiles of their block"; return HF_ERANGE; }
        copying = false;
        if (t.dst_list > HF_MAX_PREFETCH_CHUNKS || (t.dst_list && (t.rows != t.dst_list || t.src_off % 16 || t.row_bytes % 16 || t.vec_bytes != 16))) {
          err = "prefetched list: malformed chunked load-only tile";
          return HF_ERANGE;
        }
        for (uint32_t r = 0; r < t.rows; ++r) pre.push_back({t.src_off + (uint64_t)r * t.src_row_stride, t.row_bytes});
        continue;
      }
      copying = true;
      if (k >= pl.tiles_fwd_mc.size() || std::memcmp(&t, &pl.tiles_fwd_mc[k], sizeof t) != 0) { err = "prefetched list differs from the multicast list"; return HF_ERANGE; }
      ++k;
      if (t.n_dst > 1)
        for (uint32_t r = 0; r < t.rows; ++r) shared.push_back({t.src_off + (uint64_t)r * t.src_row_stride, t.row_bytes});
    }
    if (k != pl.tiles_fwd_mc.size() || !close_block()) { err = "prefetched list: load-only tiles do not cover the shared tiles of their block"; return HF_ERANGE; }
  }
  // (3b) gathering out of the generation buffers: every source lies inside an own piece of
  // its rank (resident, and never a destination of the same launch)
  if (pl.flags & HF_GATHER_FROM_GEN) {
    std::vector<Seg> own;
    for (const hf_desc &d : pl.fwd_own) desc_segments(d, own);
    for (Seg &s : own) s.src = s.dst;
    if (!normalise(own, err, "own pieces")) return HF_ERANGE;
    std::vector<Seg> srcs;
    for (const hf_desc &d : pl.fwd_peer) desc_segments(d, srcs);
    for (const Seg &s : srcs) {
      // last own interval that starts at or before the source segment
      auto it = std::upper_bound(own.begin(), own.end(), s.src, [](uint64_t v, const Seg &o) { return v < o.dst; });
      if (it == own.begin() || (--it, s.src + s.len > it->dst + it->len)) { err = "a gather source is not inside an own piece"; return HF_ERANGE; }
    }
  }

  // (4) offload image: its generation side is exactly the peer destinations, its host side
  // is pairwise disjoint and inside the image; the offload tiles are its descriptors
  {
    std::vector<Seg> gen_side, host_side, peers = fwd_peer_only, tiles;
    for (const hf_desc &d : pl.remote) {
      std::vector<Seg> one;
      desc_segments(d, one); // Seg.dst = host image offset, Seg.src = generation offset
      for (const Seg &s : one) {
        if (s.dst + s.len > pl.remote_bytes) { err = "offload descriptor leaves the image"; return HF_ERANGE; }
        host_side.push_back(s);
        gen_side.push_back({s.src, s.src, s.len});
      }
    }
    for (Seg &s : peers) s.src = s.dst; // compare coverage of gen_buf only
    std::vector<Seg> host_sorted = host_side;
    if (!normalise(host_sorted, err, "offload image") || !normalise(gen_side, err, "offload sources") ||
        !normalise(peers, err, "peer destinations"))
      return HF_ERANGE;
    if (!same(gen_side, peers)) { err = "offload image does not cover the remote pieces"; return HF_ERANGE; }
    if (pl.flags & HF_PLAN_OFFLOAD) {
      for (const hf_tile &t : pl.tiles_offload) tile_segments(t, tiles);
      if (!normalise(tiles, err, "offload tiles")) return HF_ERANGE;
      if (!same(tiles, host_sorted)) { err = "offload tiles differ from descriptors"; return HF_ERANGE; }
      if (pl.tiles_reload.size() != pl.tiles_offload.size()) { err = "reload tiles differ from offload tiles"; return HF_ERANGE; }
      for (size_t i = 0; i < pl.tiles_reload.size(); ++i) {
        const hf_tile &x = pl.tiles_offload[i], &y = pl.tiles_reload[i];
        if (x.src_off != y.dst_off || x.dst_off != y.src_off || x.src_row_stride != y.dst_row_stride ||
            x.dst_row_stride != y.src_row_stride || x.rows != y.rows || x.row_bytes != y.row_bytes || x.vec_bytes != y.vec_bytes) {
          err = "reload tiles differ from offload tiles";
          return HF_ERANGE;
        }
      }
    }
  }
  // (5) the records that the kernels walk are exactly the descriptors too
  {
    std::vector<Seg> own, image, image_back;
    for (const hf_desc &d : pl.fwd_own) desc_segments(d, own);
    if (pl.flags & HF_PLAN_OFFLOAD)
      for (const hf_desc &d : pl.remote) desc_segments(d, image);
    for (const Seg &s : image) image_back.push_back({s.src, s.dst, s.len});
    if (!normalise(own, err, "own pieces") || !normalise(image, err, "offload image") || !normalise(image_back, err, "reload")) return HF_ERANGE;
    const std::vector<Seg> &forward = (pl.flags & HF_COPY_OWN) ? fwd : fwd_peer_only;
    const bool staged = !pl.dev_static.tiles.empty(), ahead = pl.effective_multicast() == HF_MULTICAST_PREFETCHED;
    const struct { const DevList &list; const std::vector<uint64_t> &dst; const std::vector<Seg> &want; const char *name; bool prefetched = false, distances = false; } lists[] = {
        {pl.dev_fwd, pl.mc_dst, forward, "train->gen records", ahead},     {pl.dev_own, pl.mc_dst, own, "own records"},
        {pl.dev_back, pl.mc_dst, back, "gen->train records"},       {pl.dev_offload, pl.mc_dst, image, "offload records"},
        {pl.dev_reload, pl.mc_dst, image_back, "reload records"},   {staged ? pl.dev_static : pl.dev_fwd, staged ? pl.static_dst : pl.mc_dst, forward, "staged records", ahead && !staged},
        {pl.dev_auto, pl.auto_dst, forward, "records of the automatic choice", false, true}};
    for (const auto &l : lists) {
      if (l.distances && l.list.tiles.empty()) continue;
      std::vector<Seg> moved;
      if (!record_segments(l.list, l.dst, l.prefetched, l.distances, moved)) { err = std::string(l.name) + ": a record leaves its rows, or is not loaded as it is copied"; return HF_ERANGE; }
      if (!normalise(moved, err, l.name)) return HF_ERANGE;
      if (!same(moved, l.want)) { err = std::string(l.name) + " differ from descriptors"; return HF_ERANGE; }
    }
  }
  for (const std::vector<hf_tile> *lst : {&pl.tiles_fwd, &pl.tiles_back, &pl.tiles_offload, &pl.tiles_reload})
    for (const hf_tile &t : *lst) {
      uint64_t g = t.src_off | t.dst_off | t.row_bytes;
      if (t.rows > 1) g |= (uint64_t)t.src_row_stride | t.dst_row_stride;
      if (g % t.vec_bytes || t.row_bytes == 0 || t.rows == 0) { err = "tile alignment wrong"; return HF_ERANGE; }
    }
  return HF_OK;
}

} // namespace hf
