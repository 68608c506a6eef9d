// Host-side plans: mode validation, grouping of modes into one recurrence
// chain per alpha = |m| (Algorithm 1 of the paper: a chain serves every n of
// its alpha), per-step coefficients, and a small device-side cache.
#include <algorithm>
#include <cstdlib>
#include <iterator>
#include <list>
#include <mutex>

#include "zp_internal.hpp"

namespace zp {

zp_status validate_modes(const int32_t *n, const int32_t *m, int64_t M, int64_t *bad)
{
    for (int64_t i = 0; i < M; ++i) {
        const int64_t a = m[i] < 0 ? -(int64_t)m[i] : (int64_t)m[i];
        // Sec. 2: n >= 0, |m| <= n, n - |m| even.
        if (n[i] < 0 || a > n[i] || ((n[i] - a) & 1) || n[i] > ZP_N_MAX) {
            *bad = i;
            return ZP_ERR_MODE;
        }
    }
    return ZP_OK;
}

// Ratio of two exactly representable integers: correctly rounded.
static double ratio(int64_t num, int64_t den) { return (double)num / (double)den; }

// (-1)^K C(K + alpha, K), rounded to double from 64-bit-significand
// arithmetic (at most ~2K roundings of 2^-64 each before the final one).
static double signed_binom(int K, int alpha)
{
    long double v = 1.0L;
    for (int i = 1; i <= K; ++i) v = v * (long double)(alpha + i) / (long double)i;
    return (double)((K & 1) ? -v : v);
}

// Recurrence step k >= 1 of the chain of alpha (the formulas of zp_internal.hpp).
static Coef step_coef(int64_t K, int64_t A)
{
    Coef cf{};
    if (K > 1) {
        cf.cc_lo = ratio((K - 1) * (K - 1) * (2 * K + A), (K + A) * (K + A) * (2 * K + A - 2));
        cf.cc_hi = ratio((K + A - 1) * (K - 1) * (2 * K + A), K * (K + A) * (2 * K + A - 2));
    }
    cf.bs_lo = ratio((2 * K + A - 1) * (2 * K + A), 2 * (K + A) * (K + A));
    cf.bs_hi = ratio((2 * K + A - 1) * (2 * K + A), 2 * K * (K + A));
    return cf;
}

// The fused series kernels' tables, from the whole chains in emission order.
static void build_quads(Plan &plan)
{
    const std::vector<Chain> &ch = plan.achains;
    for (size_t c = 0; c < ch.size(); ++c)
        while (plan.row_chain.size() * 16 < (size_t)(ch[c].emit_off + ch[c].emit_cnt)) plan.row_chain.push_back((int32_t)c);
    std::vector<int32_t> order(ch.size());
    for (size_t c = 0; c < ch.size(); ++c) order[c] = (int32_t)c;
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return ch[(size_t)x].kmax > ch[(size_t)y].kmax; });
    // four chains at a time, longest first; each quad to the slice with the
    // least work so far (contraction steps, recurrence steps, and the set-up
    // of a chain's angle and power, about six contraction steps' worth)
    const size_t nq = (ch.size() + 3) / 4;
    std::vector<std::vector<size_t>> slice(kSlices);
    std::vector<double> load(kSlices, 0.0);
    auto chain_of = [&](size_t q, size_t y) { return order[std::min(4 * q + y, ch.size() - 1)]; };
    for (size_t q = 0; q < nq; ++q) {
        int most = 0;
        for (size_t y = 0; y < 4 && 4 * q + y < ch.size(); ++y) most = std::max(most, ch[(size_t)chain_of(q, y)].emit_cnt);
        const size_t w = (size_t)(std::min_element(load.begin(), load.end()) - load.begin());
        slice[w].push_back(q);
        load[w] += (double)most + 0.5 * ch[(size_t)chain_of(q, 0)].kmax + 6.0;
    }
    plan.slice_off.push_back(0);
    for (int w = 0; w < kSlices; ++w) {
        for (size_t q : slice[(size_t)w]) {
            Quad Q{};
            Q.kmax = ch[(size_t)chain_of(q, 0)].kmax;
            Q.step_off = (int32_t)(plan.qsteps.size() / 8);
            Q.entry_off = (int32_t)plan.entry_hdr.size();
            long double a_lo[4] = {1.0L, 1.0L, 1.0L, 1.0L};
            int next[4], end[4];
            for (size_t y = 0; y < 4; ++y) {
                const Chain &c = ch[(size_t)chain_of(q, y)];
                Q.alpha[y] = c.alpha;
                next[y] = c.emit_off;
                end[y] = 4 * q + y < ch.size() ? c.emit_off + c.emit_cnt : c.emit_off; // a repeated chain has no columns
            }
            Q.alpha_min = *std::min_element(Q.alpha, Q.alpha + 4);
            Q.spread = *std::max_element(Q.alpha, Q.alpha + 4) - Q.alpha_min;
            for (int k = 0; k <= Q.kmax; ++k) {
                for (size_t y = 0; y < 4; ++y) {
                    // past its own last degree a chain stands still: beyond the
                    // disc it would go on growing, to infinity before the others
                    const bool own = k <= ch[(size_t)chain_of(q, y)].kmax;
                    const Coef cf = k && own ? step_coef(k, Q.alpha[y]) : Coef{};
                    if (k && own) a_lo[y] = -a_lo[y] * (long double)(Q.alpha[y] + k) / (long double)k;
                    plan.qsteps.push_back({cf.cc_lo, cf.bs_lo, (double)a_lo[y], 0.0});
                    plan.qsteps.push_back({cf.cc_hi, cf.bs_hi, 1.0, 0.0});
                }
                // columns of degree k: cos and sin lists per chain, one entry per position
                std::vector<int32_t> cols[2][4];
                size_t depth = 0;
                for (size_t y = 0; y < 4; ++y)
                    for (; next[y] < end[y] && plan.emits[(size_t)next[y]].K == k; ++next[y]) {
                        const Emit &e = plan.emits[(size_t)next[y]];
                        cols[e.flags & 1][y].push_back(e.col);
                        depth = std::max(depth, cols[e.flags & 1][y].size());
                    }
                for (size_t d = 0; d < depth; ++d) {
                    int hdr = k;
                    for (int f = 0; f < 2; ++f)
                        for (size_t y = 0; y < 4; ++y) {
                            const bool has = d < cols[f][y].size();
                            hdr |= has ? 1 << (16 + 4 * f + (int)y) : 0;
                            plan.entry_cols.push_back(has ? cols[f][y][d] : 0);
                        }
                    plan.entry_hdr.push_back(hdr);
                }
            }
            Q.entry_end = (int32_t)plan.entry_hdr.size();
            if (plan.entry_hdr.size() % 2) {
                plan.entry_hdr.push_back(Q.kmax);
                plan.entry_cols.insert(plan.entry_cols.end(), 8, 0);
            }
            plan.quads.push_back(Q);
        }
        plan.slice_off.push_back((int32_t)plan.quads.size());
    }
    plan.entry_hdr.insert(plan.entry_hdr.end(), kEntryTail, 0);
    plan.entry_cols.insert(plan.entry_cols.end(), 8 * kEntryTail, 0);
    plan.qsteps.insert(plan.qsteps.end(), 8 * kStepTail, QuadStep{});
}

std::shared_ptr<Plan> build_plan_host(const int32_t *n, const int32_t *m, int64_t M)
{
    auto plan = std::make_shared<Plan>();
    plan->n.assign(n, n + M);
    plan->m.assign(m, m + M);
    int amax = -1;
    for (int64_t i = 0; i < M; ++i) {
        amax = std::max(amax, std::abs(m[i]));
        plan->nmax = std::max(plan->nmax, n[i]);
    }
    // Emits grouped by alpha; within a chain sorted by K (stable, so
    // duplicates keep the caller's column order).
    std::vector<std::vector<Emit>> by_alpha(amax + 1);
    for (int64_t i = 0; i < M; ++i) {
        const int a = std::abs(m[i]);
        Emit e{};
        e.K = (n[i] - a) / 2;
        e.col = (int32_t)i;
        e.flags = m[i] < 0 ? 1 : 0;
        e.a_lo = signed_binom(e.K, a);
        by_alpha[a].push_back(e);
    }
    struct Tmp {
        Chain c;
        double cost;
    };
    std::vector<Tmp> tmp;
    for (int a = 0; a <= amax; ++a) {
        auto &v = by_alpha[a];
        if (v.empty()) continue;
        std::stable_sort(v.begin(), v.end(), [](const Emit &x, const Emit &y) { return x.K < y.K; });
        Chain c{};
        c.alpha = a;
        c.kmax = v.back().K;
        c.coef_off = (int32_t)plan->coefs.size();
        c.emit_off = (int32_t)plan->emits.size();
        c.emit_cnt = (int32_t)v.size();
        for (int k = 1; k <= c.kmax; ++k) plan->coefs.push_back(step_coef(k, a));
        plan->emits.insert(plan->emits.end(), v.begin(), v.end());
        // Work estimate: stores dominate; the recurrence costs about one
        // store-equivalent per few steps.
        tmp.push_back({c, 4.0 * c.emit_cnt + 0.5 * c.kmax});
    }
    for (auto &t : tmp) plan->achains.push_back(t.c); // still in emission order
    build_quads(*plan);
    std::stable_sort(tmp.begin(), tmp.end(), [](const Tmp &x, const Tmp &y) { return x.cost > y.cost; });
    for (auto &t : tmp) plan->chains.push_back(t.c);

    // Pieces of at most kSegEmits emissions, cut on multiples of 8.
    std::vector<Tmp> pieces;
    for (const Chain &c : plan->chains) {
        int e0 = c.emit_off;
        const int end = c.emit_off + c.emit_cnt;
        while (e0 < end) {
            int e1 = std::min(end, (e0 / 8) * 8 + kSegEmits);
            if (e1 <= e0) e1 = std::min(end, e0 + kSegEmits);
            Chain p = c;
            p.emit_off = e0;
            p.emit_cnt = e1 - e0;
            p.kmax = plan->emits[e1 - 1].K;
            pieces.push_back({p, 4.0 * p.emit_cnt + 0.5 * p.kmax});
            e0 = e1;
        }
    }
    std::stable_sort(pieces.begin(), pieces.end(), [](const Tmp &x, const Tmp &y) { return x.cost > y.cost; });
    for (auto &t : pieces) plan->pieces.push_back(t.c);
    return plan;
}

// c_s = (-1)^s C(n-s, s) C(n-2s, (n-m)/2 - s) (Eq. radial-part-eq-binom), in
// 64-bit-significand arithmetic, times (n-2s)!/(n-2s-j)!.
static double direct_coef(int n, int m, int s, int j)
{
    const int e = n - 2 * s;
    if (e < j) return 0.0;
    auto binom = [](int top, int k) {
        long double v = 1.0L;
        for (int i = 1; i <= k; ++i) v = v * (long double)(top - k + i) / (long double)i;
        return v;
    };
    long double c = binom(n - s, s) * binom(n - 2 * s, (n - m) / 2 - s);
    for (int t = 0; t < j; ++t) c *= (long double)(e - t);
    return (double)((s & 1) ? -c : c);
}

zp_status get_direct_table(Plan &plan)
{
    std::call_once(plan.direct_once, [&plan] {
        const size_t M = plan.n.size();
        std::vector<int64_t> off(M + 1, 0);
        for (size_t i = 0; i < M; ++i) {
            const int K = (plan.n[i] - std::abs(plan.m[i])) / 2;
            off[i + 1] = off[i] + 4 * (K + 1);
        }
        std::vector<double> coef((size_t)off[M]);
        for (size_t i = 0; i < M; ++i) {
            const int n = plan.n[i], m = std::abs(plan.m[i]), K = (n - m) / 2;
            for (int j = 0; j < 4; ++j)
                for (int s = 0; s <= K; ++s) coef[(size_t)off[i] + (size_t)j * (K + 1) + s] = direct_coef(n, m, s, j);
        }
        // layout: offsets int64[M+1] | n int32[M] | m int32[M] | coefficients
        const size_t a = (M + 1) * sizeof(int64_t), a_al = (a + 255) / 256 * 256;
        const size_t b = M * sizeof(int32_t), b_al = (b + 255) / 256 * 256;
        const size_t total = a_al + 2 * b_al + coef.size() * sizeof(double);
        std::vector<unsigned char> host(total, 0);
        std::copy_n((const unsigned char *)off.data(), a, host.data());
        std::copy_n((const unsigned char *)plan.n.data(), b, host.data() + a_al);
        std::copy_n((const unsigned char *)plan.m.data(), b, host.data() + a_al + b_al);
        std::copy_n((const unsigned char *)coef.data(), coef.size() * sizeof(double), host.data() + a_al + 2 * b_al);
        void *d = nullptr;
        zp_status st = hip_check(hipMalloc(&d, total), "hipMalloc(direct table)");
        if (st == ZP_OK) st = hip_check(hipMemcpy(d, host.data(), total, hipMemcpyHostToDevice), "hipMemcpy(direct table)");
        plan.direct_status = st;
        if (st == ZP_OK) {
            plan.d_direct = d;
            plan.d_direct_off = (const int64_t *)d;
            plan.d_direct_n = (const int32_t *)((unsigned char *)d + a_al);
            plan.d_direct_m = (const int32_t *)((unsigned char *)d + a_al + b_al);
            plan.d_direct_coef = (const double *)((unsigned char *)d + a_al + 2 * b_al);
        }
    });
    return plan.direct_status == ZP_OK ? ZP_OK : set_error(plan.direct_status, "direct table upload failed");
}

zp_status get_zrec_table(Plan &plan)
{
    std::call_once(plan.zrec_once, [&plan] {
        const int nmax = plan.nmax;
        // triangle entry of (n, alpha): rows k < n hold k/2 + 1 entries each
        auto entry = [](int n, int a) {
            int t = 0;
            for (int k = 0; k < n; ++k) t += k / 2 + 1;
            return t + (a - (n & 1)) / 2;
        };
        const int T = entry(nmax + 1, (nmax + 1) & 1);
        std::vector<int32_t> cnt((size_t)T + 1, 0), cols(plan.n.size());
        for (size_t i = 0; i < plan.n.size(); ++i) ++cnt[(size_t)entry(plan.n[i], std::abs(plan.m[i])) + 1];
        for (int t = 0; t < T; ++t) cnt[(size_t)t + 1] += cnt[(size_t)t];
        std::vector<int32_t> fill(cnt.begin(), cnt.end() - 1);
        for (size_t i = 0; i < plan.n.size(); ++i) // caller's order within an entry
            cols[(size_t)fill[(size_t)entry(plan.n[i], std::abs(plan.m[i]))]++] = (int32_t)i;
        const size_t a = cnt.size() * sizeof(int32_t), a_al = (a + 255) / 256 * 256;
        const size_t total = a_al + cols.size() * sizeof(int32_t);
        std::vector<unsigned char> host(total, 0);
        std::copy_n((const unsigned char *)cnt.data(), a, host.data());
        std::copy_n((const unsigned char *)cols.data(), cols.size() * sizeof(int32_t), host.data() + a_al);
        void *d = nullptr;
        zp_status st = hip_check(hipMalloc(&d, total), "hipMalloc(recursion table)");
        if (st == ZP_OK) st = hip_check(hipMemcpy(d, host.data(), total, hipMemcpyHostToDevice), "hipMemcpy(recursion table)");
        plan.zrec_status = st;
        if (st == ZP_OK) {
            plan.d_zrec = d;
            plan.d_zrec_off = (const int32_t *)d;
            plan.d_zrec_cols = (const int32_t *)((unsigned char *)d + a_al);
        }
    });
    return plan.zrec_status == ZP_OK ? ZP_OK : set_error(plan.zrec_status, "recursion table upload failed");
}

Plan::~Plan()
{
    if (!dmem && !d_direct && !d_zrec) return;
    int cur = -1;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(device);
    (void)hipDeviceSynchronize(); // kernels may still read the tables
    if (d_zrec) (void)hipFree(d_zrec);
    if (d_direct) (void)hipFree(d_direct);
    if (dmem) (void)hipFree(dmem);
    if (cur >= 0) (void)hipSetDevice(cur);
}

// Device image of a plan's tables: chains and pieces side by side, then the
// coefficients, the emissions, the permutation and the fused series kernels'
// tables, each 256-byte aligned.
size_t plan_image(const Plan &p, std::vector<unsigned char> *host, PlanOffsets *o)
{
    const size_t a = (p.chains.size() + p.pieces.size()) * sizeof(Chain);
    const size_t b = std::max<size_t>(p.coefs.size(), 1) * sizeof(Coef);
    const size_t c = p.emits.size() * sizeof(Emit);
    const size_t d = p.emits.size() * sizeof(int32_t);
    o->coefs = (a + 255) / 256 * 256;
    o->emits = o->coefs + (b + 255) / 256 * 256;
    o->perm = o->emits + (c + 255) / 256 * 256;
    size_t end = o->base = o->perm + d;
    auto place = [&end](size_t bytes) {
        const size_t at = (end + 255) / 256 * 256;
        end = at + bytes;
        return at;
    };
    o->achains = place(p.achains.size() * sizeof(Chain));
    o->row_chain = place(p.row_chain.size() * sizeof(int32_t));
    o->quads = place(p.quads.size() * sizeof(Quad));
    o->slice_off = place(p.slice_off.size() * sizeof(int32_t));
    o->qsteps = place(p.qsteps.size() * sizeof(QuadStep));
    o->entry_hdr = place(p.entry_hdr.size() * sizeof(int32_t));
    o->entry_cols = place(p.entry_cols.size() * sizeof(int32_t));
    o->total = end;
    if (!host) return o->total;
    host->assign(o->total, 0);
    unsigned char *h = host->data();
    auto put = [h](size_t at, const auto &v) {
        std::copy_n((const unsigned char *)v.data(), v.size() * sizeof(v[0]), h + at);
    };
    put(o->achains, p.achains);
    put(o->row_chain, p.row_chain);
    put(o->quads, p.quads);
    put(o->slice_off, p.slice_off);
    put(o->qsteps, p.qsteps);
    put(o->entry_hdr, p.entry_hdr);
    put(o->entry_cols, p.entry_cols);
    std::copy_n((const unsigned char *)p.chains.data(), p.chains.size() * sizeof(Chain), h);
    std::copy_n((const unsigned char *)p.pieces.data(), p.pieces.size() * sizeof(Chain),
                h + p.chains.size() * sizeof(Chain));
    if (!p.coefs.empty()) std::copy_n((const unsigned char *)p.coefs.data(), p.coefs.size() * sizeof(Coef), h + o->coefs);
    std::copy_n((const unsigned char *)p.emits.data(), c, h + o->emits);
    for (size_t e = 0; e < p.emits.size(); ++e) {
        const int32_t col = p.emits[e].col;
        std::copy_n((const unsigned char *)&col, sizeof col, h + o->perm + e * sizeof(int32_t));
    }
    return o->total;
}

void plan_bind(Plan &p, const void *base, const PlanOffsets &o, const void *fused)
{
    const unsigned char *b = (const unsigned char *)base;
    p.d_chains = (const Chain *)b;
    p.d_pieces = p.d_chains + p.chains.size();
    p.d_coefs = (const Coef *)(b + o.coefs);
    p.d_emits = (const Emit *)(b + o.emits);
    p.d_perm = (const int32_t *)(b + o.perm);
    p.d_quads = nullptr;
    if (!fused) return;
    const unsigned char *f = (const unsigned char *)fused;
    auto at = [&](size_t off) { return f + (off - o.achains); };
    p.d_achains = (const Chain *)at(o.achains);
    p.d_row_chain = (const int32_t *)at(o.row_chain);
    p.d_quads = (const Quad *)at(o.quads);
    p.d_slice_off = (const int32_t *)at(o.slice_off);
    p.d_qsteps = (const QuadStep *)at(o.qsteps);
    p.d_entry_hdr = (const int32_t *)at(o.entry_hdr);
    p.d_entry_cols = (const int32_t *)at(o.entry_cols);
}

static zp_status upload(Plan &p)
{
    std::vector<unsigned char> host;
    PlanOffsets o;
    plan_image(p, &host, &o);
    zp_status st = hip_check(hipMalloc(&p.dmem, o.total), "hipMalloc(plan)");
    if (st != ZP_OK) return st;
    st = hip_check(hipMemcpy(p.dmem, host.data(), o.total, hipMemcpyHostToDevice), "hipMemcpy(plan)");
    if (st != ZP_OK) return st;
    plan_bind(p, p.dmem, o, (const unsigned char *)p.dmem + o.achains);
    return ZP_OK;
}

namespace {
std::mutex g_mu;
// Most recently used first.  Heap-allocated and never destroyed, so no HIP
// call runs during static destruction at process exit.
std::list<std::shared_ptr<Plan>> &g_cache = *new std::list<std::shared_ptr<Plan>>();

size_t cache_capacity()
{
    static size_t cap = [] {
        const char *e = std::getenv("ZP_PLAN_CACHE");
        long v = e ? std::strtol(e, nullptr, 10) : 16;
        return (size_t)std::max(1L, v);
    }();
    return cap;
}
} // namespace

// Looks the mode list up under the cache lock.  A missing plan is built and
// uploaded without the lock (a plan of the same list built meanwhile by another
// thread wins), and plans pushed out of the cache are released after the lock
// is dropped: releasing one synchronizes its device, since kernels may still
// read its tables.
zp_status get_plan(const int32_t *n, const int32_t *m, int64_t M, std::shared_ptr<Plan> *out)
{
    int dev = 0;
    zp_status st = hip_check(hipGetDevice(&dev), "hipGetDevice");
    if (st != ZP_OK) return st;
    auto same = [&](const Plan &p) {
        return p.device == dev && (int64_t)p.n.size() == M && std::equal(p.n.begin(), p.n.end(), n) &&
               std::equal(p.m.begin(), p.m.end(), m);
    };
    auto lookup = [&]() -> bool { // under the lock
        for (auto it = g_cache.begin(); it != g_cache.end(); ++it) {
            if (same(**it)) {
                g_cache.splice(g_cache.begin(), g_cache, it);
                *out = g_cache.front();
                return true;
            }
        }
        return false;
    };
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (lookup()) return ZP_OK;
    }
    std::shared_ptr<Plan> plan = build_plan_host(n, m, M);
    plan->device = dev;
    st = upload(*plan);
    if (st != ZP_OK) return st;
    std::list<std::shared_ptr<Plan>> released; // destroyed after the lock below
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (lookup()) {
            released.push_back(std::move(plan));
        } else {
            g_cache.push_front(plan);
            *out = plan;
            while (g_cache.size() > cache_capacity()) released.splice(released.end(), g_cache, std::prev(g_cache.end()));
        }
    }
    return ZP_OK;
}

void clear_plans()
{
    std::list<std::shared_ptr<Plan>> drop;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        drop.swap(g_cache);
    }
    drop.clear();
}

} // namespace zp
