// TEST INFRASTRUCTURE ONLY: drives the library's C ABI on the CPU emulation (host memory stands in
// for device memory) and writes everything it produced to files, for comparison with the oracle.
//   emu_driver route <n> <dtype 0|1> <t_steps> <stride> [<bits>]: only names the search that such a tensor takes (of 16 bits; the
//   caller's rounds of 13); with bits also whether a workspace of such a call has room for value buckets
//   emu_driver <in.bin> <n> <dtype 0|1> <bits> <t_steps> <dist> <flags> <stride> <nbins> <cus> <outdir> [cands_per_round]
#include <hip/hip_runtime.h>

#include <sys/mman.h>

#include <algorithm>
#include <string>
#include <vector>

#include "qp_bucket.hpp"

namespace emu { extern int g_occupancy, g_cus; void *shared_alloc(size_t); }

static void dump(const std::string &dir, const char *name, const void *p, size_t bytes)
{
    FILE *f = fopen((dir + "/" + name).c_str(), "wb");
    if (!f || fwrite(p, 1, bytes, f) != bytes) { perror(name); exit(3); }
    fclose(f);
}

static bool g_shared = false;             // blocks run as processes: "device memory" must be shared between them
static void *alloc_exact(size_t bytes)   // 16-byte aligned; the sanitizer sees any overrun past `bytes` (rounded to 16)
{
    void *p = g_shared ? emu::shared_alloc(bytes)   // ends at an inaccessible page instead
                       : aligned_alloc(16, (bytes + 15) / 16 * 16);
    if (!p) exit(3);
    emu::know(p, bytes, hipMemoryTypeDevice, 0, false);
    return p;
}
// Memory that no kernel of this device reaches: the host's, or another device's without peer access.
static void *alloc_unreachable(size_t bytes, hipMemoryType type, int device)
{
    void *p = mmap(nullptr, (bytes + 4095) / 4096 * 4096, PROT_READ | PROT_WRITE, MAP_SHARED | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED) exit(3);
    emu::know(p, bytes, type, device, true);
    return p;
}
static void release(void *p)
{
    if (!g_shared) free(p);
}

int main(int argc, char **argv)
{
    if ((argc == 6 || argc == 7) && std::string(argv[1]) == "route") {
        const uint64_t n = strtoull(argv[2], nullptr, 10);
        qp::SearchPlan plan{};
        plan.t_steps = (uint32_t)atoi(argv[4]);
        plan.stride = (uint32_t)atoi(argv[5]);
        plan.bits = argc == 7 ? (uint32_t)atoi(argv[6]) : 16u;
        plan.bucket_room = 1u;
        const bool streams = !qp::searches_value_table(n, atoi(argv[3]), plan) && !qp::tile_search_eligible(n, plan);
        const bool tile = plan.stride > 1u || (argc == 7 && plan.t_steps + 1u <= 13u);
        if (streams && !tile && qp::bucket_search_eligible(n, atoi(argv[3]), plan)) {
            plan.bucket_at = 0u;
            puts(qp::bucket_setup_args(nullptr, n, plan, reinterpret_cast<void *>(uintptr_t{1} << 20)).dense_width ? "buckets" : "buckets, or streaming if dense");
        } else {
            puts(qp::searches_value_table(n, atoi(argv[3]), plan) ? "table" : !streams || (argc == 7 && tile) ? "tile" : "streaming");
        }
        if (argc == 7) {
            qp_search_cfg_t cfg;
            qp_default_search_cfg(&cfg);
            cfg.t_steps = plan.t_steps;
            if (plan.stride > 1u) {
                cfg.flags = QP_SEARCH_COARSE_TO_FINE;
                cfg.coarse_stride = plan.stride;
            }
            puts(qp_workspace_bytes(n, &cfg) > (4u << 20) ? "room" : "no room");
        }
        return 0;
    }
    if (argc != 12 && argc != 13) { fprintf(stderr, "usage: see source\n"); return 2; }
    const char *in = argv[1];
    const uint64_t n = strtoull(argv[2], nullptr, 10);
    const qp_dtype dtype = (qp_dtype)atoi(argv[3]);
    const uint32_t bits = (uint32_t)atoi(argv[4]);
    qp_search_cfg_t cfg;
    qp_default_search_cfg(&cfg);
    cfg.t_steps = (uint32_t)atoi(argv[5]);
    cfg.dist = (uint32_t)atoi(argv[6]);
    cfg.flags = (uint32_t)atoi(argv[7]);
    cfg.coarse_stride = (uint32_t)atoi(argv[8]);
    cfg.nbins = (uint32_t)atoi(argv[9]);
    emu::g_cus = atoi(argv[10]);
    const std::string out = argv[11];
    if (argc == 13) cfg.cands_per_round = (uint32_t)atoi(argv[12]);

    g_shared = getenv("EMU_CONCURRENT_BLOCKS") && atoi(getenv("EMU_CONCURRENT_BLOCKS")) > 0;
    const size_t esz = dtype == QP_BF16 ? 2 : 4;
    void *x = alloc_exact(n * esz);
    FILE *f = fopen(in, "rb");
    if (!f || fread(x, esz, n, f) != n) { perror("input"); return 3; }
    fclose(f);

    const size_t wsb = qp_workspace_bytes(n, &cfg), pkb = qp_packed_bytes(n, bits);
    void *ws = alloc_exact(wsb), *ws2 = alloc_exact(wsb);
    memset(ws, 0xC3, wsb);
    memset(ws2, 0x5A, wsb);
    void *packed = alloc_exact(pkb), *packed2 = alloc_exact(pkb);
    memset(packed, 0x77, pkb);
    memset(packed2, 0x11, pkb);
    float *y = (float *)alloc_exact(n * 4);

    qp_stats_t st;
    qp_search_result_t res;
    qp_qparams_t q;
    memset(&res, 0, sizeof res);
    memset(&q, 0, sizeof q);
    int rc_stats = qp_stats(x, n, dtype, cfg.nbins, ws, wsb, nullptr, &st);
    int rc_search = qp_dsaciq_search(x, n, dtype, &st, bits, &cfg, ws, wsb, nullptr, &res, &q);
    int rc_pack = -100, rc_unpack = -100, rc_compress = -100, same = -1;
    if (rc_search == QP_OK) {
        rc_pack = qp_quant_pack(x, n, dtype, &q, packed, pkb, nullptr);
        rc_unpack = qp_unpack_dequant(packed, pkb, &q, y, n, nullptr);
        // where the fused path's record goes: memory of its own, the last bytes of the input or of the payload, where the
        // search leaves it anyway, memory that kernels do not reach, or an allocation too short for it
        const char *env = getenv("EMU_RECORD");
        const std::string where = env ? env : "own";
        qp_qparams_t qread;
        char *qout;   // (any alignment)
        if (where == "in_x") qout = (char *)x + (n * esz - sizeof q);
        else if (where == "in_packed") qout = (char *)packed2 + (pkb - sizeof q);
        else if (where == "on_itself") qout = (char *)ws2 + qp_ws_offset(QP_WS_QPARAMS);
        else if (where == "host") qout = (char *)alloc_unreachable(sizeof q, hipMemoryTypeHost, 0);
        else if (where == "peer") qout = (char *)alloc_unreachable(sizeof q, hipMemoryTypeDevice, 1);
        else if (where == "short") qout = (char *)alloc_exact(sizeof q - 8);
        else qout = (char *)alloc_exact(sizeof q);
        rc_compress = qp_compress_async(x, n, dtype, bits, &cfg, ws2, wsb, packed2, pkb, (qp_qparams_t *)qout, nullptr);
        if (rc_compress == QP_OK) {
            const emu::Allocation *m = emu::find(qout);
            if (m->unreachable) mprotect(m->base, 4096, PROT_READ);
            memcpy(&qread, qout, sizeof q);
            if (where == "in_packed") memcpy(qout, (char *)packed + (pkb - sizeof q), sizeof q);   // the codes it replaced
            const char *a = (const char *)ws, *b = (const char *)ws2;
            same = memcmp(a + qp_ws_offset(QP_WS_STATS), b + qp_ws_offset(QP_WS_STATS), sizeof(qp_stats_t)) == 0 &&
                   memcmp(a + qp_ws_offset(QP_WS_QPARAMS), b + qp_ws_offset(QP_WS_QPARAMS), sizeof(qp_qparams_t)) == 0 &&
                   memcmp(&qread, &q, sizeof q) == 0 && memcmp(packed, packed2, pkb) == 0;
        }
    }
    dump(out, "stats.bin", &st, sizeof st);
    dump(out, "hist.bin", (const char *)ws + qp_ws_offset(QP_WS_HIST), (size_t)cfg.nbins * 4);
    dump(out, "result.bin", &res, sizeof res);
    dump(out, "qparams.bin", &q, sizeof q);
    dump(out, "scores.bin", (const char *)ws + qp_ws_offset(QP_WS_SCORES), ((size_t)cfg.t_steps + 1) * 8);
    // what the fused sender path left in its own workspace (its search may run a different kernel sequence)
    dump(out, "scores2.bin", (const char *)ws2 + qp_ws_offset(QP_WS_SCORES), ((size_t)cfg.t_steps + 1) * 8);
    dump(out, "result2.bin", (const char *)ws2 + qp_ws_offset(QP_WS_RESULT), sizeof res);
    // what the search by value buckets made of the tensor, where the workspace holds such: its plan
    {
        const size_t cols = std::max(qp::search_blocks(n), qp::tile_search_blocks(n)), rows = std::max(cfg.t_steps + 1u, 128u);
        const size_t least = qp::kOffSearchPart + cols * rows * sizeof(double);
        qp::BucketPlan plan;
        memset(&plan, 0xff, sizeof plan);
        const qp::BucketLayout l = qp::bucket_layout(n, least);
        if (wsb > least) memcpy(&plan, (const char *)ws + l.plan, sizeof plan);
        dump(out, "plan.bin", &plan, offsetof(qp::BucketPlan, uneven));
        // ... and how many elements it counted in each bucket, segment by segment
        const uint32_t parts[2] = {l.segments, l.tile * l.tiles};
        dump(out, "segments.bin", parts, sizeof parts);
        if (wsb > least) dump(out, "totals.bin", (const char *)ws + l.totals, (size_t)l.segments * qp::kBkKeys * 4);
        // ... and the classes of each bucket, in their order
        if (wsb > least && plan.fallback == 0) {
            std::vector<float> list;
            const char *p = (const char *)ws;
            for (uint32_t b = 0; b < 2 * plan.width; ++b) {
                if (b == plan.centre) continue;
                const qp::BucketRec &r = reinterpret_cast<const qp::BucketRec *>(p + l.recs)[b];
                const qp::BucketClass *c = reinterpret_cast<const qp::BucketClass *>(p + l.classes) + r.cls;
                list.push_back((float)r.ncls);
                for (uint32_t i = 0; i < r.ncls; ++i) list.insert(list.end(), {c[i].add, c[i].m, c[i].unit});
            }
            dump(out, "classes.bin", list.data(), list.size() * 4);
        }
    }
    dump(out, "packed.bin", packed, pkb);
    dump(out, "y.bin", y, n * 4);
    char line[256];
    snprintf(line, sizeof line, "%d %d %d %d %d %d\n", rc_stats, rc_search, rc_pack, rc_unpack, rc_compress, same);
    dump(out, "status.txt", line, strlen(line));
    release(x); release(ws); release(ws2); release(packed); release(packed2); release(y);
    return 0;
}
