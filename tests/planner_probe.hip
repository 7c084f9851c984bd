// Host-side probe of the dispatch planners (test infrastructure): reads one
// call per line from stdin and prints the plan the library would use, so
// that the CPU tests can check the plans' invariants and the documented
// choices without a GPU.  It includes the dispatch source itself, so the
// functions it calls are the library's own.
//
//   wide <fmt> <epi> <M> <N1> <K1> [<N2> <K2> ...]  -> plan_splits (large M)
//   stream <fmt> <M> <N1> <K1> [...]                 -> stream_plan (few rows)
//   kg <fmt> <fp32 X> <epi> <M> <N1> <K1> [...]      -> kg_choose
//   route <fmt> <fp32 X> <epi> <forced> <M1> <N1> <K1> [...] -> choose_path
//   w8a8 <address of the scales> <M> <N> <K>         -> w8a8_plan
//
// Output, one line per input: "wide ext S1 ps1 S2 ps2 ..." (layers in the
// order the library launches them: longest reduction first) or
// "stream rw kw mx S1 pb1 S2 pb2 ...", "w8a8 kernel workgroups threads"
// or "kg kept planned use K1 shape1 rows1 columns1 ..." (kept: the choice was
// in its cache; planned: afterwards the large-M plan is in its own; use 1: the
// K-group kernel runs; the tile of each layer's shape).
// "route <kernel> K1 v1 ...": the kernel family of a group and, per layer in
// launch order, its shape (kg), few-row kernel (rows: 0 GEMV, 1 streaming, 2
// few-row MFMA; in call order) or number of K parts (mid, tiled, wide in the
// kernel, wideext by the sum launch).
#include "../paper_2607_08526_amd/csrc/qlinear.hip"

#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>

static void route(std::istringstream &in)
{
    using namespace qlk;
    int fmt = 0, xf32 = 0, epi = 0, forced = 0, n = 0;
    in >> fmt >> xf32 >> epi >> forced;
    ql_linear_ep l[QL_MAX_GROUP];
    const ql_linear_ep *p[QL_MAX_GROUP], *o[QL_MAX_GROUP];
    int64_t M, N, K, maxM = 0;
    while (n < QL_MAX_GROUP && in >> M >> N >> K) {
        l[n] = ql_linear_ep{};
        l[n].ep = NO_EPILOGUE;
        if (epi)
            l[n].ep.bias = reinterpret_cast<const float *>(16);
        l[n].lin.fmt = fmt;
        l[n].lin.xdt = xf32 ? QL_DT_F32 : QL_DT_BF16;
        l[n].lin.M = M;
        l[n].lin.N = N;
        l[n].lin.K = K;
        maxM = std::max(maxM, M);
        p[n] = &l[n];
        ++n;
    }
    KgPlan kg{};
    const GroupPath path = choose_path(p, n, forced, kg);
    launch_order(p, n, o);
    LinDesc d[QL_MAX_GROUP]{};
    auto tiles = [&](const ql_linear_ep *const *q, int bm, int bn) {
        for (int i = 0; i < n; ++i) {
            d[i].M = (int)q[i]->lin.M;
            d[i].N = (int)q[i]->lin.N;
            d[i].K = (int)q[i]->lin.K;
            d[i].ep = to_epilogue(q[i]->ep);
            d[i].tiles_m = (d[i].M + bm - 1) / bm;
            d[i].tiles_n = (d[i].N + bn - 1) / bn;
        }
    };
    int v[QL_MAX_GROUP] = {};
    const char *name = "refused";
    switch (path) {
    case GroupPath::KG:
        name = "kg";
        tiles(o, 1, 1);
        std::copy(kg.shape, kg.shape + n, v);
        break;
    case GroupPath::ROWS:
        name = "rows";
        tiles(p, 1, 1);
        for (int i = 0; i < n; ++i)
            v[i] = forced ? forced - QL_PATH_GEMV : (int)auto_row_path(fmt, d[i]);
        break;
    case GroupPath::MID: {
        name = "mid";
        tiles(o, mid_tile_bm(), mid_tile_bn());
        GroupArgs a{};
        a.n = n;
        std::copy(d, d + n, a.d);
        plan_mid(a);
        for (int i = 0; i < n; ++i)
            v[i] = a.d[i].ksplit;
        break;
    }
    case GroupPath::WIDE: {
        tiles(o, wide_tile_bm(), wide_tile_bn());
        const SplitPlan sp = plan_splits(fmt, d, n);
        name = sp.ext ? "wideext" : "wide";
        std::copy(sp.S, sp.S + n, v);
        break;
    }
    case GroupPath::TILED: {
        name = "tiled";
        const TileCfg t = choose_tile(maxM, xf32 != 0);
        tiles(o, tile_bm(t), tile_bn(t));
        plan_tiled(d, n);
        for (int i = 0; i < n; ++i)
            v[i] = d[i].ksplit;
        break;
    }
    default: break;
    }
    std::printf("route %s", name);
    for (int i = 0; i < n; ++i)
        std::printf(" %d %d", d[i].K, v[i]);
    std::printf("\n");
}

int main()
{
    using namespace qlk;
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::string kind;
        int fmt = 0, epi = 0, M = 0;
        in >> kind;
        if (kind == "w8a8") {
            W8Args a{};
            uintptr_t scales = 0;
            in >> scales >> a.M >> a.N >> a.K;
            a.scales = reinterpret_cast<const uint16_t *>(scales);
            const W8Plan p = w8a8_plan(a, device_cus());
            std::printf("w8a8 %d %lld %d\n", (int)p.kernel, (long long)p.wgs, p.threads);
            continue;
        }
        if (kind == "route") {
            route(in);
            continue;
        }
        in >> fmt;
        int xf32 = 0;
        if (kind == "kg")
            in >> xf32;
        if (kind == "wide" || kind == "kg")
            in >> epi;
        in >> M;
        LinDesc d[QL_MAX_GROUP]{};
        int n = 0, N, K;
        if (kind == "kg") {
            ql_linear_ep l[QL_MAX_GROUP];
            const ql_linear_ep *o[QL_MAX_GROUP];
            while (n < QL_MAX_GROUP && in >> N >> K) {
                l[n] = ql_linear_ep{};
                l[n].ep = NO_EPILOGUE;
                if (epi)
                    l[n].ep.bias = reinterpret_cast<const float *>(16);
                l[n].lin.fmt = fmt;
                l[n].lin.xdt = xf32 ? QL_DT_F32 : QL_DT_BF16;
                l[n].lin.M = M;
                l[n].lin.N = N;
                l[n].lin.K = K;
                o[n] = &l[n];
                ++n;
            }
            std::stable_sort(o, o + n, [](const ql_linear_ep *a, const ql_linear_ep *b) {
                return a->lin.K > b->lin.K;
            });
            // whether the choice was kept, then, after it, the large-M plan
            KgChoice c{};
            const bool kept = kg_choices().find(kg_key(fmt, o, n), c);
            c = cached_kg_choice(fmt, o, n);
            for (int i = 0; i < n; ++i) {
                d[i].M = M;
                d[i].N = (int)o[i]->lin.N;
                d[i].K = (int)o[i]->lin.K;
                if (epi)
                    d[i].ep.bias = reinterpret_cast<const float *>(16);
            }
            SplitPlan sp{};
            const bool planned = wide_plans().find(wide_key(fmt, d, n), sp);
            std::printf("kg %d %d %d", kept, planned, c.use ? 1 : 0);
            for (int i = 0; i < n; ++i) {
                const KgTile t = kg_tile_shape(fmt, xf32 != 0, M, c.plan.shape[i]);
                std::printf(" %d %d %d %d", (int)o[i]->lin.K, c.plan.shape[i], t.m, t.n);
            }
            std::printf("\n");
            continue;
        }
        while (n < QL_MAX_GROUP && in >> N >> K) {
            LinDesc &x = d[n++];
            x.M = M;
            x.N = N;
            x.K = K;
            x.tiles_m = (M + wide_tile_bm() - 1) / wide_tile_bm();
            x.tiles_n = (N + wide_tile_bn() - 1) / wide_tile_bn();
            x.ksplit = 1;
            x.psteps = K / 64;
            if (epi)
                x.ep.bias = reinterpret_cast<const float *>(16);
        }
        if (kind == "wide") {
            std::stable_sort(d, d + n, [](const LinDesc &a, const LinDesc &b) { return a.K > b.K; });
            const SplitPlan pl = plan_splits(fmt, d, n);
            std::printf("wide %d", pl.ext ? 1 : 0);
            for (int i = 0; i < n; ++i)
                std::printf(" %d %d %d %d", d[i].K, d[i].tiles_m * d[i].tiles_n, pl.S[i], pl.psteps[i]);
        } else {
            int S[QL_MAX_GROUP], P[QL_MAX_GROUP];
            const StreamPlan sp = stream_plan(fmt, d, n, device_cus(), S, P);
            std::printf("stream %d %d %d", sp.rw, sp.kw, sp.mx);
            for (int i = 0; i < n; ++i)
                std::printf(" %d %d %d", d[i].K, S[i], P[i]);
        }
        std::printf("\n");
    }
    return 0;
}
