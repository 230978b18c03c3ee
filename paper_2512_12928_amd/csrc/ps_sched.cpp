// Host-only batch former behind ps_sched_* / ps_form_batch: SlideBatching (Alg. 1) with the
// eviction, offload and copy-budget rules of Sec. 4.3.  Integer picoseconds, exact arithmetic.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <unordered_map>
#include <unordered_set>
#include <vector>

#include "../../include/ps.h"

// defined next to ps_last_error(): stores the thread-local error text
extern "C" void ps_internal_set_error(const char* text);

namespace {

typedef __int128 i128;

int sched_fail(int code, const char* fmt, ...);

// A round walks all requests several times, and a queue of a hundred is 20 KB: what the walks read of every request is
// its first cache line.
struct alignas(64) Req {
  int64_t arrival, last_sched;
  int64_t computed = 0;   // tokens whose KV exists (on the device, or on the host if evicted)
  int64_t exec = 0;       // of this round
  int32_t prompt_len, out_len;
  int32_t generated = 0;  // output tokens delivered
  int32_t n_dev = 0, n_host = 0;  // sizes of dev_blocks and host_slots
  int32_t tag = -1;       // the caller's index of the request (ps_sched_simulate), not used by the rounds
  uint8_t prio;
  bool decoding = false, urgent = false, in_batch = false, evicted_now = false;  // of this round
  // the second line
  alignas(64) int64_t rid;
  int64_t weight = 0;     // of this round
  std::vector<int32_t> dev_blocks;  // logical order
  std::vector<int32_t> host_slots;  // host copies of logical blocks 0..n-1 (issued, maybe still in flight)
  std::vector<std::pair<int64_t, int32_t>> host_rounds;  // the scheduling rounds that issued them, oldest first: (round, copies up to and with it)

  int64_t need() const { return (int64_t)prompt_len + generated; }
  int64_t b_miss() const { return std::max(0, n_host - n_dev); }
  void count() {
    n_dev = (int32_t)dev_blocks.size();
    n_host = (int32_t)host_slots.size();
  }
};

}  // namespace

// One entry of the queue while it is being ordered: the sort key of its request next to it, so that a comparison reads
// nothing but the two entries (except where two densities are too close for doubles).
struct OrderKey {
  Req* r;
  union {
    double density;  // group 1: weight / exec, rounded
    int64_t k;       // group 0: time last scheduled; group 2: remaining time
  };
  int32_t group;     // 0 starving, 1 URGENT, 2 NORMAL, 3 arrival order only
};

struct ps_sched {
  ps_sched_cfg cfg;
  std::vector<int32_t> dev_free, host_free;  // LIFO: back() is handed out next
  std::unordered_map<int64_t, Req*> by_id;
  std::vector<Req*> reqs;  // active requests, in the order of the last round, new ones behind
  std::vector<OrderKey> keys, moved;                 // scratch of a round
  std::vector<Req*> later, offload;                  // not arrived; with enough blocks to offload
  std::vector<size_t> ended;                         // places in the queue of the requests that are through with their output
  std::vector<std::pair<Req*, int64_t>> members;
  int64_t round = 0;        // ps_form_batch calls so far
  int64_t done_upto = 0;    // offloads issued in rounds <= this have completed (ps_sched_offloads_done)
  // result storage
  std::vector<int32_t> q_start, kv_len, bt_start, block_ids, si_host, si_dev, so_dev, so_host, emitted_index;
  std::vector<uint8_t> prio;
  std::vector<int64_t> req_ids, order, urgent, evicted, emitted_req, finished;
};

namespace {

inline int64_t t_prefill(const ps_sched_cfg& c, int64_t lq, int64_t lkv) {
  return c.a_p * lq * lq + c.b_p * lq * lkv + c.c_p * lq;
}
inline int64_t t_decode(const ps_sched_cfg& c, int64_t lkv) { return c.a_d * lkv + c.b_d; }

// GetMaxChunk: largest c in [0, lq] with T~_p(c, lkv) <= T (the cost is non-decreasing in c).
int64_t max_chunk(const ps_sched_cfg& c, int64_t lq, int64_t lkv, int64_t T) {
  if (lq <= 0 || T < 0 || t_prefill(c, 1, lkv) > T) return 0;
  if (t_prefill(c, lq, lkv) <= T) return lq;
  int64_t lo = 1, hi = lq - 1;  // cost(lo) <= T holds for lo = 1
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo + 1) / 2;
    if (t_prefill(c, mid, lkv) <= T)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Adaptive copy-budget control (Sec. 4.3).  Case 2(ii): transfer time B * t_block rises with B,
// the batch latency T_fwd^min + (B_missing - B) * s_blk * c_p falls (blocks not copied are
// recomputed); the answer is the largest B with transfer <= latency, found by bisection.
int64_t copy_budget(const ps_sched_cfg& c, int64_t t_budget, int64_t t_fwd_min, int64_t b_missing) {
  if (t_fwd_min >= t_budget) return t_budget / c.t_block_ps;
  if ((i128)t_fwd_min >= (i128)b_missing * c.t_block_ps) return b_missing;
  auto ok = [&](int64_t B) {
    return (i128)B * c.t_block_ps <= (i128)t_fwd_min + (i128)(b_missing - B) * c.block_tokens * c.c_p;
  };
  int64_t lo = 0, hi = b_missing;  // ok(0) holds: 0 <= t_fwd_min + ...
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo + 1) / 2;
    if (ok(mid))
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Hands out n blocks of a free list, last freed first, behind those `to` has.
void take(std::vector<int32_t>& from, size_t n, std::vector<int32_t>& to) {
  const size_t had = to.size();
  to.resize(had + n);
  const int32_t* src = from.data() + from.size();
  int32_t* dst = to.data() + had;
  for (size_t i = 0; i < n; ++i) dst[i] = src[-1 - (ptrdiff_t)i];
  from.resize(from.size() - n);
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Alg. 1 line 13 and the starvation rule: starving (longest wait first), URGENT by density descending, NORMAL by
// remaining time ascending; ties by arrival, then id.  A total order, so every sorting algorithm gives the same queue.
bool before(const OrderKey& a, const OrderKey& b) {
  if (a.group != b.group) return a.group < b.group;
  if (a.group == 1) {
    const double diff = a.density - b.density;
    if (std::fabs(diff) > 1e-14 * (std::fabs(a.density) + std::fabs(b.density))) return diff > 0;
    const i128 da = (i128)a.r->weight * std::max<int64_t>(b.r->exec, 1);  // a.w/a.exec vs b.w/b.exec
    const i128 db = (i128)b.r->weight * std::max<int64_t>(a.r->exec, 1);
    if (da != db) return da > db;
  } else if (a.k != b.k) {
    return a.k < b.k;
  }
  if (a.r->arrival != b.r->arrival) return a.r->arrival < b.r->arrival;
  return a.r->rid < b.r->rid;
}

// Sorts the queue, which comes in the order of the round before with new requests behind: from one round to the next few
// requests change places.  Those that stand out of order are taken out (the larger one of a pair if it alone disturbs the
// order, the smaller one otherwise), the rest closes up, and the sorted few go back from the largest down, each to the
// place that bisection finds: every key moves twice at most, however far they go.  When more than a third of the requests
// have moved, a full sort takes over.
void order_queue(std::vector<OrderKey>& keys, std::vector<OrderKey>& moved) {
  const size_t n = keys.size();
  const size_t most = n / 3 + 16;
  moved.clear();
  OrderKey* const kept = keys.data();
  size_t w = n > 0 ? 1 : 0;
  for (size_t i = 1; i < n; ++i) {
    const OrderKey x = keys[i];
    if (!before(x, kept[w - 1])) {
      kept[w++] = x;
      continue;
    }
    if (moved.size() == most) {  // the keys in [w, i) have been copied: to the front, or to the list
      std::copy(moved.begin(), moved.end(), kept + w);
      std::sort(keys.begin(), keys.end(), before);
      return;
    }
    if (i + 1 < n && before(keys[i + 1], kept[w - 1]) && (w == 1 || !before(x, kept[w - 2]))) {
      moved.push_back(kept[w - 1]);
      kept[w - 1] = x;
    } else {
      moved.push_back(x);
    }
  }
  std::sort(moved.begin(), moved.end(), before);
  size_t to = n;
  for (size_t m = moved.size(); m-- > 0;) {
    OrderKey* const at = std::upper_bound(kept, kept + w, moved[m], before);
    std::move_backward(at, kept + w, kept + to);
    to -= (size_t)(kept + w - at) + 1;
    w = (size_t)(at - kept);
    kept[to] = moved[m];
  }
}

// Whether a list of block ids names one twice: a table of marks where the ids span a range not much longer than the
// list (a pool is usually a permutation of 0..n-1), a sort otherwise.
bool has_duplicate(const int32_t* ids, int32_t n) {
  if (n < 2) return false;
  int32_t lo = ids[0], hi = ids[0];
  for (int32_t i = 1; i < n; ++i) {
    lo = std::min(lo, ids[i]);
    hi = std::max(hi, ids[i]);
  }
  const int64_t span = (int64_t)hi - lo + 1;
  if (span < n) return true;
  if (span <= 16 * (int64_t)n + 1024) {
    std::vector<uint8_t> seen((size_t)span, 0);
    for (int32_t i = 0; i < n; ++i)
      if (seen[(size_t)((int64_t)ids[i] - lo)]++) return true;
    return false;
  }
  std::vector<int32_t> v(ids, ids + n);
  std::sort(v.begin(), v.end());
  return std::adjacent_find(v.begin(), v.end()) != v.end();
}

}  // namespace

namespace {
int sched_fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  ps_internal_set_error(buf);
  return code;
}
}  // namespace

extern "C" {

int ps_sched_create(const ps_sched_cfg* cfg, const int32_t* dev_free_order, int32_t n_dev,
                    const int32_t* host_free_order, int32_t n_host, ps_sched** out) {
  if (!cfg || !out) return sched_fail(PS_EINVAL, "ps_sched_create: NULL argument");
  *out = nullptr;
  if (cfg->n_classes < 1 || cfg->n_classes > 8) return sched_fail(PS_EINVAL, "n_classes must be in 1..8");
  if (cfg->block_tokens < 1) return sched_fail(PS_EINVAL, "block_tokens must be positive");
  if (cfg->eta_ps <= cfg->t_c) return sched_fail(PS_EINVAL, "eta must exceed t_c (denominator of Eq. 8)");
  if (cfg->gamma_den <= 0 || cfg->beta_den <= 0 || cfg->rho_den <= 0 || cfg->gamma_num < 0 || cfg->beta_num < 0 ||
      cfg->rho_num < 0)
    return sched_fail(PS_EINVAL, "gamma / beta / rho must be non-negative fractions with positive denominators");
  if (cfg->t_block_ps <= 0) return sched_fail(PS_EINVAL, "t_block must be positive");
  if (cfg->order_policy != PS_ORDER_SLIDEBATCHING && cfg->order_policy != PS_ORDER_FCFS)
    return sched_fail(PS_EINVAL, "order_policy must be PS_ORDER_SLIDEBATCHING or PS_ORDER_FCFS");
  if (cfg->a_p < 0 || cfg->b_p < 0 || cfg->c_p < 0 || cfg->a_d < 0 || cfg->b_d < 0 || cfg->t_c < 0)
    return sched_fail(PS_EINVAL, "estimator coefficients must be non-negative");
  if (n_dev < 0 || n_host < 0 || (n_dev > 0 && !dev_free_order) || (n_host > 0 && !host_free_order))
    return sched_fail(PS_EINVAL, "bad pool description");
  for (int p = 0; p < cfg->n_classes; ++p)
    if (cfg->class_weight[p] <= 0) return sched_fail(PS_EINVAL, "class weights must be positive");
  if (has_duplicate(dev_free_order, n_dev) || has_duplicate(host_free_order, n_host))
    return sched_fail(PS_EINVAL, "duplicate block id in a pool");
  ps_sched* s = new (std::nothrow) ps_sched();
  if (!s) return sched_fail(PS_ENOMEM, "out of host memory");
  s->cfg = *cfg;
  s->dev_free.resize((size_t)n_dev);
  std::reverse_copy(dev_free_order, dev_free_order + n_dev, s->dev_free.begin());
  s->host_free.resize((size_t)n_host);
  std::reverse_copy(host_free_order, host_free_order + n_host, s->host_free.begin());
  *out = s;
  return PS_OK;
}

void ps_sched_destroy(ps_sched* s) {
  if (!s) return;
  for (Req* r : s->reqs) delete r;
  delete s;
}

int ps_sched_add_request(ps_sched* s, int64_t rid, int64_t arrival_ps, int32_t prio, int32_t prompt_len,
                         int32_t out_len) {
  if (!s) return sched_fail(PS_EINVAL, "NULL scheduler");
  if (prio < 1 || prio > s->cfg.n_classes) return sched_fail(PS_EINVAL, "priority class %d outside 1..%d", prio, s->cfg.n_classes);
  if (prompt_len < 1 || out_len < 1) return sched_fail(PS_EINVAL, "prompt_len and out_len must be >= 1");
  if (s->by_id.count(rid)) return sched_fail(PS_EINVAL, "request %lld already queued", (long long)rid);
  Req* r = new (std::nothrow) Req();
  if (!r) return sched_fail(PS_ENOMEM, "out of host memory");
  r->rid = rid;
  r->arrival = arrival_ps;
  r->prio = (uint8_t)prio;
  r->prompt_len = prompt_len;
  r->out_len = out_len;
  r->last_sched = arrival_ps;  // "waiting time" counts from arrival until first scheduled
  const size_t blocks = (size_t)std::min<int64_t>(ceil_div((int64_t)prompt_len + out_len, s->cfg.block_tokens), 4096);
  r->dev_blocks.reserve(blocks);
  r->host_slots.reserve(blocks);
  s->reqs.push_back(r);
  s->by_id[rid] = r;
  return PS_OK;
}

int ps_sched_counts(const ps_sched* s, int32_t* n_queued, int32_t* n_dev_free, int32_t* n_host_free) {
  if (!s) return sched_fail(PS_EINVAL, "NULL scheduler");
  if (n_queued) *n_queued = (int32_t)s->reqs.size();
  if (n_dev_free) *n_dev_free = (int32_t)s->dev_free.size();
  if (n_host_free) *n_host_free = (int32_t)s->host_free.size();
  return PS_OK;
}

int ps_sched_offloads_done(ps_sched* s, int64_t upto_round) {
  if (!s) return sched_fail(PS_EINVAL, "NULL scheduler");
  if (upto_round > s->round) return sched_fail(PS_EINVAL, "round %lld has not been formed yet", (long long)upto_round);
  if (upto_round > s->done_upto) s->done_upto = upto_round;
  return PS_OK;
}

// One round.  want_batch false: the batch's token offsets and block tables, the queue's order and the lists of blocks
// to copy, which only a caller that runs the batch needs, are not written out (the simulation delivers tokens and takes
// the number of offloaded blocks, nothing else).
static int form_round(ps_sched* s, int64_t now, bool want_batch, ps_batch_out* out) {
  s->round += 1;
  const ps_sched_cfg& c = s->cfg;
  const int64_t blk = c.block_tokens;
  for (auto* v : {&s->q_start, &s->kv_len, &s->bt_start, &s->block_ids, &s->si_host, &s->si_dev, &s->so_dev,
                  &s->so_host, &s->emitted_index})
    v->clear();
  for (auto* v : {&s->req_ids, &s->order, &s->urgent, &s->evicted, &s->emitted_req, &s->finished}) v->clear();
  s->prio.clear();
  std::memset(out, 0, sizeof *out);

  // the queue: requests that have arrived, in the order of the round before; Alg. 1 lines 1-6: exec, remain, t_min
  std::vector<OrderKey>& keys = s->keys;
  keys.clear();
  s->later.clear();
  int64_t t_budget = 0, phi = 0, b_copy = 0, t_batch = 0;
  int64_t t_min = INT64_MAX, sum_exec = 0, b_missing = 0;
  const size_t n_active = s->reqs.size();
  for (size_t i = 0; i < n_active; ++i) {
    Req* const r = s->reqs[i];
    __builtin_prefetch(s->reqs[std::min(i + 12, n_active - 1)]);
    if (r->arrival > now) {
      s->later.push_back(r);
      continue;
    }
    const int64_t lq = r->need() - r->computed, generated = r->generated;
    const bool dec = generated >= 1 && lq == 1;
    r->decoding = dec && r->n_host <= r->n_dev;  // and nothing of it is on the host only
    r->exec = dec ? t_decode(c, r->need()) : t_prefill(c, lq, r->computed);
    r->in_batch = r->evicted_now = false;
    OrderKey k;
    k.k = c.ttft_slo_ps + generated * c.tpot_slo_ps - (now - r->arrival);  // remain: time left to the next token's deadline
    k.r = r;
    keys.push_back(k);
    t_min = std::min(t_min, k.k);
    sum_exec += r->exec;
    b_missing += r->b_miss();
  }
  std::vector<std::pair<Req*, int64_t>>& members = s->members;
  members.clear();
  s->offload.clear();
  s->ended.clear();
  size_t n_emitted = 0, n_members = 0;
  if (!keys.empty()) {
    // line 7
    t_budget = std::max(t_min, c.eta_ps);
    // Eq. 8 and lines 8-12
    phi = (int64_t)(((i128)t_budget * sum_exec) / (t_budget - c.t_c));
    // lines 8-13 and the starvation rule (see before())
    const bool fcfs = c.order_policy == PS_ORDER_FCFS;  // comparison arm: arrival order, nothing else
    const i128 urgent_below = (i128)c.gamma_num * phi;
    for (OrderKey& k : keys) {
      Req* r = k.r;
      r->urgent = (i128)k.k * c.gamma_den < urgent_below;
      const bool starving = now - r->last_sched > c.tau_ps;
      if (fcfs) {
        k.group = 3;
        k.k = 0;
      } else if (starving) {
        k.group = 0;
        k.k = r->last_sched;
      } else if (r->urgent) {  // density: weight / exec
        k.group = 1;
        r->weight = (r->generated == 0 ? c.w_first : c.w_decode) * c.class_weight[r->prio - 1];
        k.density = (double)r->weight / (double)std::max<int64_t>(r->exec, 1);
      } else {
        k.group = 2;
      }
    }
    order_queue(keys, s->moved);
    // the active requests take over this order; those that have not arrived yet follow
    for (size_t i = 0; i < keys.size(); ++i) s->reqs[i] = keys[i].r;
    std::copy(s->later.begin(), s->later.end(), s->reqs.begin() + (ptrdiff_t)keys.size());
    Req* const* Q = s->reqs.data();
    const size_t n_queue = keys.size();
    if (want_batch)
      for (size_t i = 0; i < n_queue; ++i) {
        s->order.push_back(Q[i]->rid);
        if (Q[i]->urgent) s->urgent.push_back(Q[i]->rid);
      }
    size_t idx = 0;
    // what a member's turn ends with: its token, if it has computed everything before it, is delivered when the batch ends;
    // blocks are given back and copied once the batch stands
    members.resize(n_queue);
    s->emitted_req.resize(n_queue);
    s->emitted_index.resize(n_queue);
    auto* const to_members = members.data();
    int64_t* const to_req = s->emitted_req.data();
    int32_t* const to_index = s->emitted_index.data();
    int64_t n_off[8];  // full blocks without a host copy that start an offload, by class
    for (int p = 0; p < 8; ++p) n_off[p] = std::max<int64_t>(1, (int64_t)c.n_off_base >> p);
    const auto admitted = [&](Req* r, int64_t chunk) {
      r->computed += chunk;
      r->last_sched = now;
      r->in_batch = true;
      to_members[n_members].first = r;
      to_members[n_members++].second = chunk;
      if (r->computed == r->need()) {
        r->generated += 1;
        to_req[n_emitted] = want_batch ? r->rid : r->tag;
        to_index[n_emitted++] = r->generated;
        if (r->generated == r->out_len) {
          s->ended.push_back(idx - 1);
          return;
        }
      }
      if (r->computed >= (r->n_host + n_off[r->prio - 1]) * blk) s->offload.push_back(r);
    };
    // line 14
    b_copy = copy_budget(c, t_budget, c.t_c + sum_exec, b_missing);
    int64_t b_rem = b_copy;
    // lines 15-23
    t_batch = c.t_c;
    size_t tail = n_queue;  // requests from here on have been looked at as victims: none becomes one later in the round
    while (idx < n_queue && t_batch < t_budget) {
      Req* r = Q[idx++];
      if (r->evicted_now) continue;
      if (r->decoding && r->need() <= r->n_dev * blk) {  // a decode token that needs no block: most of a round
        t_batch += r->exec;
        admitted(r, 1);
        continue;
      }
      const int64_t T = t_budget - t_batch;
      const int64_t miss = r->b_miss();
      int64_t k = 0, comp = r->computed;
      if (miss > 0) {
        k = b_rem >= miss ? miss : b_rem;
        comp = k * blk;  // what is not reloaded is recomputed
      }
      const bool partial = miss > 0 && k < miss;
      const int64_t lq = r->need() - comp;
      const bool dec = r->generated >= 1 && lq == 1;
      int64_t chunk, t;
      if (dec) {
        chunk = 1;  // a decode token is atomic
        t = miss > 0 ? t_decode(c, r->need()) : r->exec;
      } else {
        chunk = max_chunk(c, lq, comp, T);
        if (chunk == 0) continue;
        t = t_prefill(c, chunk, comp);
      }
      if (partial) {
        const bool ok = chunk == lq || (i128)chunk * c.beta_den > (i128)c.beta_num * (miss - k) * blk;
        if (!ok) continue;
      }
      const int64_t held = r->n_dev;
      int64_t want = ceil_div(comp + chunk, blk) - held;
      if (want > (int64_t)s->dev_free.size()) {
        // victims from the tail of the sorted queue, behind r, never a near-starved request
        while (tail > idx && want > (int64_t)s->dev_free.size()) {
          Req* v = Q[--tail];
          if (v->in_batch || v->evicted_now || v->dev_blocks.empty()) continue;
          if ((i128)(now - v->last_sched) * c.rho_den >= (i128)c.rho_num * c.tau_ps) continue;
          s->dev_free.insert(s->dev_free.end(), v->dev_blocks.begin(), v->dev_blocks.end());
          v->dev_blocks.clear();
          // host copies still in flight are discarded with the eviction (Sec. 4.3, Asynchronous
          // Offloading): only completed ones keep their tokens from being recomputed
          while (!v->host_rounds.empty() && v->host_rounds.back().first > s->done_upto) v->host_rounds.pop_back();
          const size_t conf = v->host_rounds.empty() ? 0 : (size_t)v->host_rounds.back().second;
          s->host_free.insert(s->host_free.end(), v->host_slots.begin() + (ptrdiff_t)conf, v->host_slots.end());
          v->host_slots.resize(conf);
          v->count();
          v->computed = std::min<int64_t>(v->computed, (int64_t)conf * blk);
          v->evicted_now = true;
          s->evicted.push_back(v->rid);
        }
      }
      if (want > (int64_t)s->dev_free.size()) {
        const int64_t fit = (held + (int64_t)s->dev_free.size()) * blk - comp;
        if (dec || fit <= 0) break;  // memory is not enough
        chunk = std::min(chunk, fit);
        t = t_prefill(c, chunk, comp);
        want = ceil_div(comp + chunk, blk) - held;
      }
      // admit
      if (miss > 0) {
        r->dev_blocks.clear();
        take(s->dev_free, (size_t)k, r->dev_blocks);
        if (want_batch) {
          s->si_host.insert(s->si_host.end(), r->host_slots.begin(), r->host_slots.begin() + (ptrdiff_t)k);
          s->si_dev.insert(s->si_dev.end(), r->dev_blocks.begin(), r->dev_blocks.end());
        }
        s->host_free.insert(s->host_free.end(), r->host_slots.begin() + (ptrdiff_t)k, r->host_slots.end());
        r->host_slots.resize((size_t)k);
        while (r->host_rounds.size() > 1 && r->host_rounds[r->host_rounds.size() - 2].second >= k) r->host_rounds.pop_back();
        if (!r->host_rounds.empty()) r->host_rounds.back().second = (int32_t)k;  // k is less than all copies, or all of them
        r->computed = comp;
        b_rem -= k;
        want -= k;
      }
      if (want > 0) take(s->dev_free, (size_t)want, r->dev_blocks);
      r->count();
      t_batch += t;
      admitted(r, chunk);
    }
    members.resize(n_members);
    s->emitted_req.resize(n_emitted);
    s->emitted_index.resize(n_emitted);
    if (members.empty()) t_batch = 0;
  }

  // the batch as the attention layer takes it, in admission order
  s->q_start.push_back(0);
  s->bt_start.push_back(0);
  if (want_batch)
    for (auto& mc : members) {
      Req* r = mc.first;
      s->req_ids.push_back(r->rid);
      s->q_start.push_back(s->q_start.back() + (int32_t)mc.second);
      s->kv_len.push_back((int32_t)r->computed);
      const int64_t nb = ceil_div(r->computed, blk);
      s->block_ids.insert(s->block_ids.end(), r->dev_blocks.begin(), r->dev_blocks.begin() + (ptrdiff_t)nb);
      s->bt_start.push_back((int32_t)s->block_ids.size());
      s->prio.push_back((uint8_t)r->prio);
    }
  // completion
  for (size_t at : s->ended) {
    Req* r = s->reqs[at];
    s->dev_free.insert(s->dev_free.end(), r->dev_blocks.begin(), r->dev_blocks.end());
    s->host_free.insert(s->host_free.end(), r->host_slots.begin(), r->host_slots.end());
    s->finished.push_back(want_batch ? r->rid : r->tag);
  }
  // asynchronous offload: every n_off^r newly completed full blocks of r get a host copy
  int32_t n_offloaded = 0;
  for (Req* r : s->offload) {
    const int64_t copied = r->n_host;
    const int64_t pending = r->computed / blk - copied;
    if ((int64_t)s->host_free.size() < pending) continue;
    take(s->host_free, (size_t)pending, r->host_slots);
    r->count();
    r->host_rounds.emplace_back(s->round, r->n_host);
    n_offloaded += (int32_t)pending;
    if (want_batch) {
      s->so_dev.insert(s->so_dev.end(), r->dev_blocks.begin() + (ptrdiff_t)copied, r->dev_blocks.begin() + (ptrdiff_t)(copied + pending));
      s->so_host.insert(s->so_host.end(), r->host_slots.end() - (ptrdiff_t)pending, r->host_slots.end());
    }
  }
  if (!s->ended.empty()) {  // the others close up
    auto w = s->reqs.begin() + (ptrdiff_t)s->ended[0];
    for (size_t i = 0; i < s->ended.size(); ++i) {
      Req* r = s->reqs[s->ended[i]];
      const auto next = i + 1 < s->ended.size() ? s->reqs.begin() + (ptrdiff_t)s->ended[i + 1] : s->reqs.end();
      w = std::copy(s->reqs.begin() + (ptrdiff_t)s->ended[i] + 1, next, w);
      s->by_id.erase(r->rid);
      delete r;
    }
    s->reqs.resize(s->reqs.size() - s->ended.size());
  }

  out->batch.n_req = (int32_t)members.size();
  out->batch.n_tokens = s->q_start.back();
  out->batch.q_start = s->q_start.data();
  out->batch.kv_len = s->kv_len.data();
  out->batch.bt_start = s->bt_start.data();
  out->batch.block_ids = s->block_ids.data();
  out->batch.prio = s->prio.data();
  out->req_ids = s->req_ids.data();
  out->t_budget_ps = t_budget;
  out->phi_ps = phi;
  out->t_batch_ps = t_batch;
  out->copy_budget = b_copy;
  out->n_order = (int32_t)s->order.size();
  out->order = s->order.data();
  out->n_urgent = (int32_t)s->urgent.size();
  out->urgent = s->urgent.data();
  out->n_swap_in = (int32_t)s->si_host.size();
  out->swap_in_host_slots = s->si_host.data();
  out->swap_in_dev_blocks = s->si_dev.data();
  out->n_swap_out = n_offloaded;
  out->swap_out_dev_blocks = s->so_dev.data();
  out->swap_out_host_slots = s->so_host.data();
  out->n_evicted = (int32_t)s->evicted.size();
  out->evicted = s->evicted.data();
  out->n_emitted = (int32_t)s->emitted_req.size();
  out->emitted_req = s->emitted_req.data();
  out->emitted_index = s->emitted_index.data();
  out->n_finished = (int32_t)s->finished.size();
  out->finished = s->finished.data();
  out->round = s->round;
  return PS_OK;
}

int ps_form_batch(ps_sched* s, int64_t now, ps_batch_out* out) {
  if (!s || !out) return sched_fail(PS_EINVAL, "ps_form_batch: NULL argument");
  return form_round(s, now, true, out);
}

// Eq. 3 and the two metrics of Sec. 5.1 for one request.
int ps_tdg_score(const ps_sched_cfg* cfg, int32_t prio, int32_t out_len, const int64_t* token_times, int32_t n_times,
                 int64_t* gain, int64_t* ideal_gain, int32_t* slo_attained) {
  if (!cfg || (n_times > 0 && !token_times)) return sched_fail(PS_EINVAL, "ps_tdg_score: NULL argument");
  if (prio < 1 || prio > cfg->n_classes || cfg->n_classes > 8 || out_len < 0 || n_times < 0)
    return sched_fail(PS_EINVAL, "ps_tdg_score: bad class, out_len or n_times");
  const int64_t wc = cfg->class_weight[prio - 1];
  int64_t g = 0;
  for (int32_t i = 1; i <= n_times; ++i) {
    const int64_t deadline = cfg->ttft_slo_ps + (int64_t)(i - 1) * cfg->tpot_slo_ps;
    if (token_times[i - 1] < deadline) g += (i == 1 ? cfg->w_first : cfg->w_decode) * wc;
  }
  if (gain) *gain = g;
  if (ideal_gain) *ideal_gain = out_len > 0 ? (cfg->w_first + (int64_t)(out_len - 1) * cfg->w_decode) * wc : 0;
  if (slo_attained) {
    bool ok = n_times > 0 && token_times[0] < cfg->ttft_slo_ps;
    if (ok && n_times > 1)
      ok = (i128)(token_times[n_times - 1] - token_times[0]) < (i128)cfg->tpot_slo_ps * (n_times - 1);
    *slo_attained = ok ? 1 : 0;
  }
  return PS_OK;
}

// Virtual-clock run of the batch former over an arrival trace.
int ps_sched_simulate(const ps_sched_cfg* cfg, const int32_t* dev_free_order, int32_t n_dev, const int32_t* host_free_order,
                      int32_t n_host, const ps_trace_req* trace, int32_t n_trace, int32_t max_steps, int64_t* token_times,
                      int32_t* n_delivered, ps_sim_result* out) {
  if (!cfg || !out || (n_trace > 0 && !trace) || n_trace < 0 || max_steps < 0)
    return sched_fail(PS_EINVAL, "ps_sched_simulate: bad argument");
  std::memset(out, 0, sizeof *out);
  ps_sched* s = nullptr;
  int rc = ps_sched_create(cfg, dev_free_order, n_dev, host_free_order, n_host, &s);
  if (rc != PS_OK) return rc;
  // arrival order (ties by id); where each request's token times go, and its arrival beside that
  struct Deliver {
    int64_t* to;
    int64_t arrival;
  };
  std::vector<int32_t> by_arrival((size_t)n_trace);
  std::vector<int64_t> t_off((size_t)n_trace + 1, 0);
  std::unordered_set<int64_t> ids;
  ids.reserve((size_t)n_trace);
  for (int32_t i = 0; i < n_trace; ++i) {
    by_arrival[(size_t)i] = i;
    t_off[(size_t)i + 1] = t_off[(size_t)i] + std::max(trace[i].out_len, 0);
    if (!ids.insert(trace[i].rid).second) {
      ps_sched_destroy(s);
      return sched_fail(PS_EINVAL, "ps_sched_simulate: duplicate request id %lld", (long long)trace[i].rid);
    }
  }
  std::sort(by_arrival.begin(), by_arrival.end(), [&](int32_t a, int32_t b) {
    if (trace[a].arrival_ps != trace[b].arrival_ps) return trace[a].arrival_ps < trace[b].arrival_ps;
    return trace[a].rid < trace[b].rid;
  });
  std::vector<int64_t> own_times;
  std::vector<int32_t> own_counts;
  if (!token_times) {
    own_times.assign((size_t)t_off[(size_t)n_trace], 0);
    token_times = own_times.data();
  }
  if (!n_delivered) {
    own_counts.assign((size_t)n_trace, 0);
    n_delivered = own_counts.data();
  }
  std::vector<Deliver> deliver((size_t)n_trace);
  for (int32_t i = 0; i < n_trace; ++i) deliver[(size_t)i] = Deliver{token_times + t_off[(size_t)i], trace[i].arrival_ps};
  std::fill(n_delivered, n_delivered + n_trace, 0);
  const auto count = [&](int32_t i) { return n_delivered[i] = (int32_t)(deliver[(size_t)i].to - (token_times + t_off[(size_t)i])); };
  // the offload thread on the same clock: a round's copies start when its batch has been computed and
  // the earlier copies are through, and take t_block per block
  std::vector<std::pair<int64_t, int64_t>> inflight;  // (round, completion time), oldest first
  size_t inflight_head = 0;
  int64_t copy_free_at = 0, now = 0;
  int32_t nxt = 0, steps = 0;
  ps_batch_out fb;
  while (steps < max_steps) {
    while (nxt < n_trace && trace[by_arrival[(size_t)nxt]].arrival_ps <= now) {
      const ps_trace_req& p = trace[by_arrival[(size_t)nxt]];
      rc = ps_sched_add_request(s, p.rid, p.arrival_ps, p.prio, p.prompt_len, p.out_len);
      if (rc != PS_OK) {
        ps_sched_destroy(s);
        return rc;
      }
      s->reqs.back()->tag = by_arrival[(size_t)nxt];  // what form_round reports in place of the id
      ++nxt;
    }
    if (s->reqs.empty()) {
      if (nxt >= n_trace) break;
      now = trace[by_arrival[(size_t)nxt]].arrival_ps;
      continue;
    }
    while (inflight_head < inflight.size() && inflight[inflight_head].second <= now)
      (void)ps_sched_offloads_done(s, inflight[inflight_head++].first);
    (void)form_round(s, now, false, &fb);
    ++steps;
    if (fb.n_swap_out > 0) {
      copy_free_at = std::max(copy_free_at, now + fb.t_batch_ps) + (int64_t)fb.n_swap_out * cfg->t_block_ps;
      inflight.emplace_back(fb.round, copy_free_at);
    }
    for (int32_t e = 0; e < fb.n_emitted; ++e) {  // tokens are delivered when the batch ends
      if (e + 12 < fb.n_emitted) __builtin_prefetch(deliver[(size_t)fb.emitted_req[e + 12]].to, 1);
      Deliver& d = deliver[(size_t)fb.emitted_req[e]];
      *d.to++ = now + fb.t_batch_ps - d.arrival;
    }
    for (int32_t f = 0; f < fb.n_finished; ++f) {
      const int32_t i = (int32_t)fb.finished[f];
      int64_t g = 0, ideal = 0;
      int32_t ok = 0;
      (void)ps_tdg_score(cfg, trace[i].prio, trace[i].out_len, token_times + t_off[(size_t)i], count(i), &g, &ideal, &ok);
      out->gain += g;
      out->ideal_gain += ideal;
      out->slo_attained += ok;
      out->finished += 1;
    }
    now += fb.t_batch_ps > 0 ? fb.t_batch_ps : cfg->eta_ps;
  }
  for (int32_t i = 0; i < n_trace; ++i) (void)count(i);
  out->steps = steps;
  out->end_ps = now;
  ps_sched_destroy(s);
  return PS_OK;
}

}  // extern "C"
