// Drives the C ABI's host half (argument validation, layout, pointer-table bookkeeping, launch sequencing) with
// stand-in launchers, under AddressSanitizer and UndefinedBehaviorSanitizer.  "Device" pointers are host buffers
// nobody dereferences (the stand-in kernels do nothing); the workspace is a host buffer the tables are written to.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "cf_internal.h"
#include "compactfusion.h"

extern std::vector<std::string> g_launch_log;
extern bool g_single_pass_short, g_single_pass_wide, g_single_pass_blocks;
extern int g_short_workgroups;
extern bool g_capturing;
extern int g_compute_units;
extern bool g_overlapping;
extern std::vector<uint8_t> g_states;
extern bool g_single_pass_slim, g_occupancy_slim;
extern bool g_project_many;
extern int g_split;
extern std::vector<cf::TensorPtrs> g_direct;

static int g_failed = 0;
#define EXPECT(cond)                                                                    \
    do {                                                                                \
        if (!(cond)) { std::printf("line %d: %s\n", __LINE__, #cond); ++g_failed; }     \
    } while (0)

static std::string joined()
{
    std::string s;
    for (auto &k : g_launch_log) s += k + " ";
    g_launch_log.clear();
    return s;
}

// the call brought pointers to the table
static bool uploaded(const std::string &seq) { return seq.find("k_upload_ptrs") != std::string::npos; }

static cf_tensor_desc desc(int64_t n, int64_t c, int dt, int bits, int scale, int group = 128)
{
    cf_tensor_desc d;
    d.n_tokens = n; d.n_channels = c; d.dtype = dt; d.bits = bits; d.scale = scale; d.group = group;
    return d;
}

struct Buffers {       // one tensor's buffers, sized by cf_sizes, 256-byte aligned
    void *x = nullptr, *recon = nullptr, *err = nullptr, *codes = nullptr, *scales = nullptr;
    size_t cb = 0, sb = 0, rb = 0, eb = 0;
    Buffers(const cf_tensor_desc &d, const cf_options *o)
    {
        EXPECT(cf_sizes(&d, o, &cb, &sb, &rb, &eb) == CF_OK);
        auto get = [](size_t n) { void *p = nullptr; if (posix_memalign(&p, 256, n ? n : 256) != 0) std::abort(); return p; };
        x = get(rb); recon = get(rb); err = get(eb); codes = get(cb); scales = get(sb);
    }
    ~Buffers() { std::free(x); std::free(recon); std::free(err); std::free(codes); std::free(scales); }
};

int main()
{
    // ---- descriptors and options
    size_t a = 0, b = 0, c = 0, e = 0;
    cf_tensor_desc good = desc(4096, 3072, CF_BF16, 1, CF_SCALE_CHANNEL);
    EXPECT(cf_sizes(&good, nullptr, &a, &b, &c, &e) == CF_OK && a == 4096u * 384 && b == 3072u * 4 && c == 4096u * 3072 * 2 && e == 4096u * 3072 * 4);
    EXPECT(cf_sizes(nullptr, nullptr, &a, &b, &c, &e) == CF_ERR_INVALID_ARG);
    cf_tensor_desc bad = desc(0, 3072, CF_BF16, 1, CF_SCALE_CHANNEL);
    EXPECT(cf_sizes(&bad, nullptr, &a, nullptr, nullptr, nullptr) == CF_ERR_SHAPE);
    bad = desc(16, 100, CF_BF16, 1, CF_SCALE_CHANNEL);
    EXPECT(cf_sizes(&bad, nullptr, &a, nullptr, nullptr, nullptr) == CF_ERR_SHAPE);
    bad = desc(16, 128, CF_BF16, 3, CF_SCALE_CHANNEL);
    EXPECT(cf_sizes(&bad, nullptr, &a, nullptr, nullptr, nullptr) == CF_ERR_UNSUPPORTED);
    bad = desc(16, 128, CF_BF16, 2, CF_SCALE_GROUP);
    EXPECT(cf_sizes(&bad, nullptr, &a, nullptr, nullptr, nullptr) == CF_ERR_UNSUPPORTED);
    bad = desc(16, 192, CF_BF16, 4, CF_SCALE_GROUP);
    EXPECT(cf_sizes(&bad, nullptr, &a, nullptr, nullptr, nullptr) == CF_ERR_SHAPE);
    bad = desc(16, 128, 7, 2, CF_SCALE_CHANNEL);
    EXPECT(cf_sizes(&bad, nullptr, &a, nullptr, nullptr, nullptr) == CF_ERR_UNSUPPORTED);
    cf_options o;
    std::memset(&o, 0, sizeof o);
    o.flags = 0x40;
    EXPECT(cf_sizes(&good, &o, &a, nullptr, nullptr, nullptr) == CF_ERR_UNSUPPORTED);
    o.flags = 0; o.ef = 9;
    EXPECT(cf_workspace_bytes(&good, 1, &o) == 0);
    o.ef = CF_EF_RECON;
    EXPECT(cf_workspace_bytes(&good, 0, &o) == 0 && cf_workspace_bytes(nullptr, 1, &o) == 0);
    EXPECT(std::strlen(cf_status_string(CF_ERR_WORKSPACE)) > 0 && std::strlen(cf_status_string((cf_status)99)) > 0);

    // ---- a mixed context: every compressor kind, ragged shapes
    std::vector<cf_tensor_desc> descs = {desc(1500, 1096, CF_BF16, 1, CF_SCALE_CHANNEL), desc(700, 520, CF_F32, 2, CF_SCALE_CHANNEL),
                                         desc(300, 384, CF_BF16, 4, CF_SCALE_GROUP, 128), desc(130, 1096, CF_BF16, 2, CF_SPARSE_NM, 8),
                                         desc(67, 3072, CF_BF16, 2, CF_SPARSE_NM, 16), desc(203, 1024, CF_BF16, 1, CF_LOWRANK, 32),
                                         desc(1, 8, CF_F32, 4, CF_SCALE_CHANNEL)};
    const int n = (int)descs.size();
    for (uint32_t flags : {0u, (uint32_t)CF_FLAG_SINGLE_PASS, (uint32_t)CF_FLAG_TWO_KERNEL, (uint32_t)(CF_FLAG_SINGLE_PASS | CF_FLAG_FIXED_GRID),
                           (uint32_t)CF_FLAG_LOWRANK_INT4}) {
        std::memset(&o, 0, sizeof o);
        o.flags = flags;
        const size_t ws_bytes = cf_workspace_bytes(descs.data(), n, &o);
        EXPECT(ws_bytes > 0);
        void *ws = nullptr;
        if (posix_memalign(&ws, 256, ws_bytes) != 0) return 2;
        cf_ctx *ctx = nullptr;
        EXPECT(cf_init(&ctx, descs.data(), n, &o, nullptr, ws_bytes, nullptr) == CF_ERR_WORKSPACE && ctx == nullptr);
        EXPECT(cf_init(&ctx, descs.data(), n, &o, (char *)ws + 16, ws_bytes, nullptr) == CF_ERR_WORKSPACE);
        EXPECT(cf_init(&ctx, descs.data(), n, &o, ws, ws_bytes - 1, nullptr) == CF_ERR_WORKSPACE);
        EXPECT(cf_init(nullptr, descs.data(), n, &o, ws, ws_bytes, nullptr) == CF_ERR_INVALID_ARG);
        EXPECT(cf_init(&ctx, descs.data(), n, &o, ws, ws_bytes, nullptr) == CF_OK && ctx != nullptr);
        g_launch_log.clear();

        std::vector<Buffers *> buf;
        std::vector<const void *> x;
        std::vector<void *> recon, err, codes, scales;
        for (auto &d : descs) {
            buf.push_back(new Buffers(d, &o));
            x.push_back(buf.back()->x); recon.push_back(buf.back()->recon); err.push_back(buf.back()->err);
            codes.push_back(buf.back()->codes); scales.push_back(buf.back()->scales);
        }
        // state errors, range errors, pointer errors: nothing may be launched
        EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_ERR_STATE);
        EXPECT(cf_step_fused(ctx, 0, n + 1, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_ERR_INVALID_ARG);
        EXPECT(cf_step_fused(ctx, -1, 1, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_ERR_INVALID_ARG);
        EXPECT(cf_step_fused(nullptr, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_ERR_INVALID_ARG);
        EXPECT(cf_warmup(ctx, 0, n, nullptr, recon.data(), err.data(), nullptr) == CF_ERR_INVALID_ARG);
        EXPECT(joined().empty());
        EXPECT(cf_warmup(ctx, 0, n, x.data(), recon.data(), err.data(), nullptr) == CF_OK);
        EXPECT(joined().find("k_warmup") != std::string::npos);
        {   // overlapping and misaligned buffers
            std::vector<void *> r2 = recon;
            r2[0] = (char *)buf[0]->x + 256;                                    // inside x
            EXPECT(cf_step_fused(ctx, 0, n, x.data(), r2.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_ERR_INVALID_ARG);
            r2 = recon; r2[1] = (char *)recon[1] + 4;                           // not 16-byte aligned
            EXPECT(cf_step_fused(ctx, 0, n, x.data(), r2.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_ERR_INVALID_ARG);
            std::vector<void *> c2 = codes;
            c2[2] = (char *)buf[2]->err + buf[2]->eb - 16;                      // tail of err
            EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), c2.data(), scales.data(), nullptr) == CF_ERR_INVALID_ARG);
            c2 = codes; c2[3] = nullptr;
            EXPECT(cf_compress(ctx, 0, n, x.data(), recon.data(), err.data(), c2.data(), scales.data(), nullptr) == CF_ERR_INVALID_ARG);
            std::vector<void *> s2 = scales;
            s2[3] = nullptr;                                                    // the sparsifier has no scales: allowed
            EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), s2.data(), nullptr) == CF_OK);
            joined();
            EXPECT(cf_decompress(ctx, 0, n, (const void *const *)codes.data(), (const void *const *)recon.data(), recon.data(), nullptr) == CF_ERR_INVALID_ARG);
            EXPECT(joined().empty());
        }
        // launch sequences
        EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_OK);
        EXPECT(uploaded(joined()));              // a pointer changed since the last call
        EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_OK);
        std::string seq = joined();
        if (flags & CF_FLAG_TWO_KERNEL) EXPECT(seq.find("k_colreduce k_finalize k_encode k_encode_nm k_encode_nm k_lr_orth") != std::string::npos);
        if (flags & CF_FLAG_SINGLE_PASS) EXPECT(seq.find("k_single_pass k_encode k_encode_nm k_encode_nm k_lr_orth") != std::string::npos);
        if (flags & CF_FLAG_LOWRANK_INT4) EXPECT(seq.find("k_lr_quant_u") != std::string::npos);
        EXPECT(!uploaded(seq));                   // same pointers, same stream: no upload
        EXPECT(cf_step_fused(ctx, 2, 3, x.data() + 2, recon.data() + 2, err.data() + 2, codes.data() + 2, scales.data() + 2, nullptr) == CF_OK);
        seq = joined();
        EXPECT(seq.find("k_single_pass") == std::string::npos && seq.find("k_colreduce") == std::string::npos && seq.find("k_encode ") != std::string::npos);
        EXPECT(cf_step_fused(ctx, 0, 0, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_OK && joined().empty());
        // another stream, then a captured call: the table is uploaded again each time, and once more afterwards
        EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), (void *)0x1000) == CF_OK);
        EXPECT(uploaded(joined()));
        g_capturing = true;
        EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), (void *)0x1000) == CF_OK);
        EXPECT(uploaded(joined()));
        g_capturing = false;
        EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), (void *)0x1000) == CF_OK);
        EXPECT(uploaded(joined()));
        EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), (void *)0x1000) == CF_OK);
        EXPECT(!uploaded(joined()));
        // receiver, profile hooks, bookkeeping calls
        EXPECT(cf_decompress(ctx, 0, n, (const void *const *)codes.data(), (const void *const *)scales.data(), recon.data(), (void *)0x1000) == CF_OK);
        seq = joined();
        EXPECT(seq.find("k_decode") != std::string::npos && seq.find("k_lr_apply") != std::string::npos);
        void *events[8] = {(void *)1, (void *)2, (void *)3, (void *)4, (void *)5, (void *)6, (void *)7, (void *)8};
        EXPECT(cf_profile_next_call(ctx, events, 4) == CF_OK);
        EXPECT(cf_compress(ctx, 0, 2, x.data(), (const void *const *)recon.data(), err.data(), codes.data(), scales.data(), (void *)0x1000) == CF_OK);
        EXPECT(cf_profile_launch_count(ctx) >= 1 && cf_profile_kernel_name(ctx, 0) != nullptr && cf_profile_kernel_name(ctx, 99) == nullptr);
        joined();
        uint32_t gave_up = 7;
        EXPECT(cf_given_up_items(ctx, nullptr, &gave_up) == CF_OK && gave_up == 0);
        EXPECT(cf_check_device(ctx, nullptr) == CF_OK && cf_last_hip_error(ctx) == 0);
        EXPECT(cf_set_warm(ctx, 0, n, 0) == CF_OK);
        EXPECT(cf_decompress(ctx, 0, n, (const void *const *)codes.data(), (const void *const *)scales.data(), recon.data(), nullptr) == CF_ERR_STATE);
        EXPECT(cf_set_warm(ctx, 0, n + 1, 1) == CF_ERR_INVALID_ARG);
        cf_destroy(ctx);
        for (auto *p : buf) delete p;
        std::free(ws);
    }
    cf_destroy(nullptr);

    // ---- calls of one kernel over at most kDirectTensors tensors: their pointers go into its arguments, on any stream and while one is
    // captured, the table stays as it is and counts as before
    {
        std::vector<cf_tensor_desc> d;
        for (int t = 0; t < 12; ++t)
            d.push_back(t % 3 == 0 ? desc(40 + t, 384, CF_BF16, 4, CF_SCALE_GROUP) : desc(40 + t, 384, CF_F32, 2, CF_SPARSE_NM, t % 3 == 1 ? 8 : 16));
        d.push_back(desc(60, 64, CF_BF16, 1, CF_LOWRANK, 32));
        d.push_back(desc(60, 64, CF_BF16, 1, CF_SCALE_RANK1));
        const int n = (int)d.size(), most = cf::kDirectTensors;
        std::memset(&o, 0, sizeof o);
        const size_t wsb = cf_workspace_bytes(d.data(), n, &o);
        void *ws = nullptr;
        if (posix_memalign(&ws, 256, wsb) != 0) std::abort();
        std::memset(ws, 0, wsb);
        cf_ctx *ctx = nullptr;
        EXPECT(cf_init(&ctx, d.data(), n, &o, ws, wsb, nullptr) == CF_OK);
        EXPECT(cf_set_warm(ctx, 0, n, 1) == CF_OK);
        uintptr_t at = (uintptr_t)1 << 40;                          // addresses nobody looks behind
        auto take = [&](int count) { std::vector<void *> p; for (int t = 0; t < count; ++t, at += (uintptr_t)1 << 24) p.push_back((void *)at); return p; };
        std::vector<void *> recon = take(n), err = take(n), codes = take(n), scales = take(n), xs = take(n);
        const void *const *x = (const void *const *)xs.data();
        joined();
        enum What { WARMUP, STEP, COMPRESS, DECOMPRESS };
        auto call = [&](What what, int first, int count, void *stream) {
            switch (what) {
            case WARMUP: return cf_warmup(ctx, first, count, x + first, recon.data() + first, err.data() + first, stream);
            case STEP: return cf_step_fused(ctx, first, count, x + first, recon.data() + first, err.data() + first, codes.data() + first, scales.data() + first, stream);
            case COMPRESS: return cf_compress(ctx, first, count, x + first, recon.data() + first, err.data() + first, codes.data() + first, scales.data() + first, stream);
            default: return cf_decompress(ctx, first, count, (const void *const *)codes.data() + first, (const void *const *)scales.data() + first, recon.data() + first, stream);
            }
        };
        EXPECT(call(STEP, 0, n, nullptr) == CF_OK && uploaded(joined()));
        EXPECT(call(STEP, 0, n, nullptr) == CF_OK && !uploaded(joined()));
        const auto table_pointers = recon;
        recon = take(n);                                            // other buffers than the table's
        const std::vector<uint8_t> before((uint8_t *)ws, (uint8_t *)ws + wsb);
        for (What what : {WARMUP, STEP, COMPRESS, DECOMPRESS})
            for (int first : {0, 2, n - 3})
                for (int count : {1, 3, most}) {
                    if (first + count > n || ((what == STEP || what == COMPRESS) && first + count > 12)) continue;    // those senders read the table
                    for (int how = 0; how < 3; ++how) {             // the table's stream, another, a capture
                        g_capturing = how == 2;
                        EXPECT(call(what, first, count, how == 1 ? (void *)0x1000 : nullptr) == CF_OK);
                        g_capturing = false;
                        const std::string seq = joined();
                        EXPECT(!seq.empty() && !uploaded(seq));
                        EXPECT((int)g_direct.size() == count);
                        for (int k = 0; k < (int)g_direct.size(); ++k) {
                            const cf::TensorPtrs &p = g_direct[(size_t)k];
                            const int t = first + k;
                            EXPECT(p.recon == recon[t]);
                            EXPECT(p.x == (what == DECOMPRESS ? nullptr : xs[t]) && p.err == (what == DECOMPRESS ? nullptr : err[t]));
                            EXPECT((void *)p.codes == (what == WARMUP ? nullptr : codes[t]) && (void *)p.scales == (what == WARMUP ? nullptr : scales[t]));
                        }
                        EXPECT(std::memcmp(ws, before.data(), wsb) == 0);
                    }
                }
        recon = table_pointers;
        EXPECT(call(STEP, 0, n, nullptr) == CF_OK && !uploaded(joined()));         // the table still holds what it did, and is known to
        // one tensor more, and senders of kinds that several kernels work on: by the table
        recon = take(n);
        for (What what : {WARMUP, STEP, COMPRESS, DECOMPRESS}) {
            EXPECT(call(what, 1, most + 1, nullptr) == CF_OK);
            EXPECT((uploaded(joined()) == (what == WARMUP)) && g_direct.empty());
        }
        for (int t : {12, 13}) {
            EXPECT(call(STEP, t, 1, nullptr) == CF_OK && uploaded(joined()));
            EXPECT(call(DECOMPRESS, t, 1, (void *)0x1000) == CF_OK && !uploaded(joined()) && g_direct.size() == 1);
        }
        cf_destroy(ctx);
        std::free(ws);
    }

    // ---- which path a call takes by default: the single pass in calls of a round of workgroups (512 items here) and for tensors that
    // fill enough of their items, two kernels for larger calls over shorter ones
    {
        struct Case { int64_t n, c; const char *must, *must_not; uint32_t flags; };
        const Case cases[] = {
            {4096, 512, "k_single_pass", "k_colreduce", 0},             // 16 items per group, 64 in all
            {16384, 64, "k_single_pass", "k_colreduce", 0},             // 32 items of 512 rows in all
            {16384, 64, "k_single_pass", "k_colreduce", CF_FLAG_SINGLE_PASS},
            {4096, 256, "k_single_pass", "k_colreduce", 0},             // 32 items in all
            {128, 8192, "k_single_pass", "k_colreduce", 0},             // a short tensor
            {42, 131072, "k_single_pass", "k_colreduce", 0},            // 512 items a third full
            {42, 131080, "k_colreduce k_finalize k_encode", "k_single_pass", 0},       // 513
            {43, 131080, "k_single_pass", "k_colreduce", 0},            // a third of an item's 128 rows
            {42, 131080, "k_single_pass", "k_colreduce", CF_FLAG_SINGLE_PASS},
            {4096, 512, "k_colreduce k_finalize k_encode", "k_single_pass", CF_FLAG_TWO_KERNEL},
        };
        for (const Case &cs : cases) {
            std::memset(&o, 0, sizeof o);
            o.flags = cs.flags;
            cf_tensor_desc d = desc(cs.n, cs.c, CF_BF16, 2, CF_SCALE_CHANNEL);
            Buffers b(d, &o), other(d, &o);
            const size_t wsb = cf_workspace_bytes(&d, 1, &o);
            void *ws = nullptr;
            if (posix_memalign(&ws, 256, wsb) != 0) std::abort();
            cf_ctx *ctx = nullptr;
            EXPECT(cf_init(&ctx, &d, 1, &o, ws, wsb, nullptr) == CF_OK);
            const void *x = b.x;
            EXPECT(cf_warmup(ctx, 0, 1, &x, &b.recon, &b.err, nullptr) == CF_OK);
            joined();
            EXPECT(cf_step_fused(ctx, 0, 1, &x, &b.recon, &b.err, &b.codes, &b.scales, nullptr) == CF_OK);
            std::string seq = joined();
            EXPECT(seq.find(cs.must) != std::string::npos);
            EXPECT(seq.find(cs.must_not) == std::string::npos);
            const bool direct = std::string(cs.must) == "k_single_pass";      // takes its pointers along
            EXPECT(uploaded(seq) == !direct);       // the first call that reads the table
            EXPECT(cf_step_fused(ctx, 0, 1, &x, &b.recon, &b.err, &b.codes, &b.scales, nullptr) == CF_OK);
            EXPECT(!uploaded(joined()));
            // a new pointer
            EXPECT(cf_step_fused(ctx, 0, 1, &x, &b.recon, &b.err, &other.codes, &b.scales, nullptr) == CF_OK);
            EXPECT(uploaded(joined()) == !direct);
            EXPECT(!direct || (g_direct.size() == 1 && (void *)g_direct[0].codes == other.codes));
            cf_destroy(ctx);
            std::free(ws);
        }
    }

    // ---- both sides of every line of that rule for tall tensors: items of 256 rows x 128 channels (half the rows for fp32
    // and for a third operand), of 512 x 64 in contexts of mostly tall tensors
    {
        enum Path { TWO, NARROW, SLIM };
        struct Call { int32_t ef, dtype; std::vector<std::vector<int64_t>> shapes; Path path; };     // shapes: count, tokens, channels
        const int R = CF_EF_RECON, L = CF_EF_LITERAL, O = CF_EF_OFF, N = CF_EF_NAIVE, B = CF_BF16, F = CF_F32;
        const std::vector<Call> calls = {
            {R, B, {{1, 9728, 2048}}, NARROW}, {R, B, {{1, 9729, 2048}}, NARROW}, {R, B, {{4, 10000, 512}}, NARROW},     // 38, 39, 40 items
            {R, B, {{1, 10240, 2048}}, NARROW}, {R, B, {{1, 10241, 2048}}, SLIM},                                         // 40, 41
            {R, F, {{1, 4865, 2048}}, NARROW}, {R, F, {{1, 5120, 2048}}, NARROW}, {R, F, {{1, 5121, 2048}}, SLIM},
            {L, B, {{1, 4865, 2048}}, NARROW}, {L, B, {{1, 5120, 2048}}, NARROW}, {L, B, {{1, 5121, 2048}}, SLIM},
            {O, F, {{1, 2433, 2048}}, NARROW}, {O, F, {{1, 2560, 2048}}, NARROW}, {O, F, {{1, 2561, 2048}}, SLIM},
            {R, B, {{1, 32768, 1920}}, SLIM}, {R, B, {{1, 32769, 1920}}, TWO}, {R, F, {{1, 16384, 2048}}, SLIM}, {R, F, {{1, 16385, 2048}}, TWO},      // 64 items of 512 rows, 65
            {N, B, {{1, 10240, 2048}}, NARROW}, {N, B, {{1, 32768, 1920}}, SLIM}, {N, B, {{1, 32769, 1920}}, TWO},
            // rows of no whole lines of 128 bytes, and of multiples of 1024 channels: 38 items, 24
            {R, B, {{1, 19456, 2056}}, SLIM}, {R, B, {{1, 19457, 2056}}, TWO}, {R, B, {{1, 19457, 2112}}, SLIM}, {R, B, {{1, 19457, 2096}}, TWO},
            {R, B, {{1, 19456, 2048}}, SLIM}, {R, B, {{1, 19457, 2048}}, TWO}, {R, F, {{1, 9728, 2056}}, SLIM}, {R, F, {{1, 9729, 2056}}, TWO}, {R, F, {{1, 9729, 2080}}, SLIM},
            {N, B, {{1, 12288, 2056}}, SLIM}, {N, B, {{1, 12289, 2056}}, TWO}, {N, B, {{1, 12288, 2048}}, SLIM}, {N, B, {{1, 12289, 2048}}, TWO}, {N, B, {{1, 12289, 1984}}, SLIM},
            {N, F, {{1, 6144, 2056}}, SLIM}, {N, F, {{1, 6145, 2056}}, TWO}, {N, F, {{1, 12288, 2048}}, SLIM}, {N, F, {{1, 12289, 2048}}, TWO}, {N, F, {{1, 16384, 2080}}, SLIM},
            {L, B, {{1, 9728, 2056}}, SLIM}, {L, B, {{1, 9729, 2056}}, TWO}, {L, B, {{1, 16384, 2048}}, SLIM}, {L, B, {{1, 16385, 2048}}, TWO},
            {O, F, {{1, 4864, 2056}}, SLIM}, {O, F, {{1, 4865, 2056}}, TWO}, {O, F, {{1, 8192, 2048}}, SLIM}, {O, F, {{1, 8193, 2048}}, TWO},
            {R, B, {{8, 20000, 1920}, {1, 20000, 2056}}, TWO}, {R, B, {{8, 20000, 1920}, {1, 12300, 2056}}, SLIM},           // each by its own
            {R, B, {{1, 65536, 256}}, SLIM}, {R, B, {{1, 65536, 264}}, TWO},                                              // 512 items in all, 640
            {N, B, {{1, 65536, 256}}, SLIM}, {N, B, {{1, 65536, 264}}, TWO},
            {R, B, {{20, 10240, 80}}, NARROW}, {R, B, {{20, 10500, 80}}, TWO}, {R, B, {{20, 10500, 96}}, SLIM},            // slivers: 72 to 88 channels
            {R, B, {{16, 4096, 3072}, {1, 10500, 80}}, NARROW}, {R, B, {{4, 12288, 3072}, {1, 10500, 80}}, SLIM},          // one of them among others
            {R, B, {{16, 4096, 3072}, {1, 12288, 3072}}, NARROW}, {R, B, {{16, 4096, 3072}, {1, 12289, 3072}}, SLIM},      // few tall ones: 48, 49 items
            {R, B, {{2, 4096, 3072}, {1, 12288, 3072}}, SLIM}, {R, B, {{16, 1024, 3072}, {1, 32769, 3072}}, TWO},
            // short tensors: how much of its items a group of one fills, 128 rows of bf16, 64 of fp32 or with a third operand, 32 of both, in up to two
            // rounds and more; a group of two, in up to three and more
            {R, B, {{57, 42, 3072}}, TWO}, {R, B, {{57, 43, 3072}}, NARROW}, {R, B, {{114, 51, 3072}}, TWO}, {R, B, {{114, 52, 3072}}, NARROW},
            {R, B, {{114, 49, 1096}}, TWO}, {R, B, {{114, 50, 1096}}, NARROW},             // its last stripe is 72 channels of 256
            {N, B, {{114, 51, 3072}}, TWO}, {N, B, {{114, 52, 3072}}, NARROW}, {O, B, {{57, 15, 3072}}, TWO}, {O, B, {{57, 16, 3072}}, NARROW},
            {R, F, {{57, 15, 3072}}, TWO}, {R, F, {{57, 16, 3072}}, NARROW}, {O, F, {{57, 3, 3072}}, TWO}, {L, F, {{57, 4, 3072}}, NARROW},
            {R, B, {{42, 13, 3072}}, NARROW},                                              // 504 items
            {R, B, {{57, 128, 3072}}, NARROW}, {R, B, {{57, 129, 3072}}, TWO}, {R, B, {{57, 153, 3072}}, TWO}, {R, B, {{57, 154, 3072}}, NARROW},
            {R, B, {{114, 179, 3072}}, TWO}, {R, B, {{114, 180, 3072}}, NARROW}, {R, F, {{57, 76, 3072}}, TWO}, {R, F, {{57, 77, 3072}}, NARROW},
            {R, F, {{114, 89, 3072}}, TWO}, {R, F, {{114, 90, 3072}}, NARROW}, {R, F, {{114, 129, 3072}}, NARROW},
            {O, F, {{57, 38, 3072}}, TWO}, {O, F, {{57, 39, 3072}}, NARROW}, {O, F, {{57, 65, 3072}}, NARROW},
            {R, B, {{57, 256, 3072}, {1, 4000, 3072}}, NARROW}, {R, B, {{57, 257, 3072}, {1, 4000, 3072}}, NARROW},           // items of 256 rows
            // several widths, by their items; up to three rounds with a tall tensor
            {R, B, {{114, 16, 3072}, {20, 3072, 64}}, TWO}, {R, B, {{114, 30, 3072}, {30, 3072, 64}}, TWO}, {R, B, {{30, 1024, 64}, {90, 16, 3072}}, TWO},
            {R, B, {{20, 1024, 3072}, {200, 16, 256}}, NARROW}, {R, B, {{60, 128, 3072}, {100, 16, 256}}, NARROW}, {R, B, {{57, 77, 3072}, {57, 1024, 3072}}, NARROW},
            {R, B, {{20, 256, 3072}, {80, 20, 3072}}, TWO}, {R, B, {{57, 256, 3072}, {57, 20, 3072}}, NARROW},
            {R, B, {{60, 16, 3072}, {1, 2047, 64}}, TWO}, {R, B, {{60, 16, 3072}, {1, 2048, 64}}, NARROW},
            {R, B, {{126, 16, 3072}, {1, 3072, 64}}, NARROW}, {R, B, {{127, 16, 3072}, {1, 3072, 64}}, TWO},
            // rows of no whole blocks of 64 bytes: 18 items of 128 channels, 32 where the channels are a multiple of 16, more than 1280 items in all, none of 64 channels up to 64 items
            {R, B, {{30, 4608, 1096}}, NARROW}, {R, B, {{30, 4609, 1096}}, TWO}, {R, B, {{30, 4609, 1120}}, NARROW}, {R, B, {{30, 4609, 1104}}, NARROW}, {N, B, {{30, 4609, 1096}}, NARROW},
            {R, F, {{30, 4609, 1096}}, NARROW}, {R, B, {{30, 8192, 1104}}, NARROW}, {R, B, {{30, 8193, 1104}}, TWO}, {R, B, {{1, 7936, 5064}}, NARROW}, {R, B, {{1, 7936, 5256}}, TWO},
            {R, B, {{1, 12288, 1096}}, NARROW}, {R, B, {{1, 12288, 1120}}, SLIM}, {R, B, {{30, 4609, 1096}, {30, 4609, 1120}}, NARROW}, {R, B, {{31, 4609, 1096}, {30, 4609, 1088}}, TWO},
        };
        for (const Call &c : calls) {
            std::vector<cf_tensor_desc> d;
            for (auto &s : c.shapes) d.insert(d.end(), (size_t)s[0], desc(s[1], s[2], c.dtype, c.ef == L ? 4 : 2, CF_SCALE_CHANNEL));
            const int n = (int)d.size();
            std::memset(&o, 0, sizeof o);
            o.ef = c.ef;
            std::vector<const void *> x;
            std::vector<void *> recon, err, codes, scales;
            uintptr_t at = (uintptr_t)1 << 40;                      // addresses nobody looks behind
            auto take = [&] { void *p = (void *)at; at += (uintptr_t)1 << 32; return p; };
            for (int t = 0; t < n; ++t) { x.push_back(take()); recon.push_back(take()); err.push_back(take()); codes.push_back(take()); scales.push_back(take()); }
            const size_t wsb = cf_workspace_bytes(d.data(), n, &o);
            void *ws = nullptr;
            if (posix_memalign(&ws, 256, wsb) != 0) std::abort();
            cf_ctx *ctx = nullptr;
            EXPECT(cf_init(&ctx, d.data(), n, &o, ws, wsb, nullptr) == CF_OK);
            EXPECT(cf_set_warm(ctx, 0, n, 1) == CF_OK);
            joined();
            g_single_pass_slim = false;
            EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_OK);
            const bool single = joined().find("k_single_pass ") != std::string::npos;
            EXPECT(!single || g_occupancy_slim == g_single_pass_slim);      // the device's capacity for the kernel that runs
            const Path took = !single ? TWO : g_single_pass_slim ? SLIM : NARROW;
            if (took != c.path) {
                const auto &s = c.shapes.back();
                std::printf("ef %d dtype %d ... %d x [%d, %d]: path %d instead of %d\n", c.ef, c.dtype, (int)s[0], (int)s[1], (int)s[2], (int)took, (int)c.path);
                ++g_failed;
            }
            cf_destroy(ctx);
            std::free(ws);
        }
    }

    // ---- bf16 rows that are no whole blocks of 64 bytes: stripes by the context, kernels and stores by the call
    {
        enum Path { TWO, WIDE, NARROW, SLIM, SHORT };
        enum Stores { WHOLE, BLOCKS, STEPS };           // whether parts of blocks are left to the L2: in neither, both, or in steps alone
        struct Call { std::vector<std::vector<int64_t>> shapes; Path step, send; Stores stores; int first = 0, count = 0; uint32_t flags = 0; int err = CF_F32; };       // count 0: the whole context
        const int E = CF_BF16;
        const uint32_t FORCED = CF_FLAG_SINGLE_PASS;
        const std::vector<Call> calls = {
            // 48 and 49 items of 256 rows, 64 and 65: 128-channel stripes up to there; two kernels for steps of more than 1280 items alone
            {{{2, 12288, 1096}}, NARROW, NARROW, BLOCKS}, {{{2, 12289, 1096}}, NARROW, NARROW, BLOCKS}, {{{10, 12289, 1096}}, TWO, NARROW, BLOCKS},
            {{{2, 16384, 1096}}, NARROW, NARROW, BLOCKS}, {{{10, 16384, 1096}}, TWO, NARROW, BLOCKS}, {{{2, 16385, 1096}}, SLIM, SLIM, BLOCKS}, {{{10, 16385, 1096}}, TWO, SLIM, BLOCKS},
            {{{2, 12289, 1104}}, NARROW, NARROW, WHOLE}, {{{10, 12289, 1104}}, TWO, NARROW, WHOLE}, {{{10, 16384, 1104}}, TWO, NARROW, WHOLE}, {{{10, 16385, 1104}}, TWO, SLIM, WHOLE},
            // 256 channels where three quarters of a context are uneven rows, or most are such of up to 12 items, and nothing is of more than 18; or four fifths are of 4 to 12 and nothing is of more than 24
            {{{30, 4608, 1096}}, WIDE, WIDE, BLOCKS}, {{{30, 4609, 1096}}, TWO, NARROW, BLOCKS}, {{{30, 4608, 1104}}, WIDE, WIDE, WHOLE}, {{{30, 1024, 1104}}, WIDE, WIDE, BLOCKS},
            {{{30, 1025, 1104}}, WIDE, WIDE, WHOLE}, {{{110, 1024, 1096}, {1, 5000, 3072}}, WIDE, WIDE, BLOCKS}, {{{110, 1024, 1096}, {1, 5000, 1096}}, WIDE, WIDE, BLOCKS},
            {{{110, 1024, 1096}, {1, 6144, 3072}}, WIDE, WIDE, BLOCKS}, {{{110, 1024, 1096}, {1, 6145, 3072}}, TWO, NARROW, BLOCKS}, {{{110, 1024, 1096}, {40, 5000, 3072}}, NARROW, NARROW, WHOLE},
            {{{15, 4096, 1096}, {16, 4609, 1096}}, TWO, NARROW, BLOCKS}, {{{34, 4609, 1096}, {40, 4608, 1096}}, NARROW, NARROW, BLOCKS},
            {{{60, 4096, 1096}, {20, 4096, 1088}}, WIDE, WIDE, BLOCKS}, {{{60, 4096, 1096}, {21, 4096, 1088}}, NARROW, NARROW, BLOCKS},
            {{{30, 1027, 1976}, {15, 4608, 768}}, WIDE, WIDE, BLOCKS}, {{{30, 1027, 1976}, {18, 4608, 768}}, NARROW, NARROW, WHOLE}, {{{30, 1027, 1976}, {2, 4700, 1536}}, WIDE, WIDE, BLOCKS},
            {{{30, 1027, 1976}, {3, 4700, 1536}}, TWO, NARROW, BLOCKS}, {{{30, 700, 1976}, {1, 4700, 64}}, TWO, NARROW, BLOCKS},
            // next to tall tensors, ones of few row blocks or of more than 12 take two kernels, in 64 channels all do
            {{{20, 3072, 2696}, {1, 6457, 192}}, NARROW, NARROW, BLOCKS}, {{{20, 3073, 2696}, {1, 6457, 192}}, TWO, NARROW, BLOCKS}, {{{20, 3073, 2704}, {1, 6457, 192}}, NARROW, NARROW, WHOLE},
            {{{30, 1700, 1976}, {3, 7000, 1536}}, TWO, NARROW, BLOCKS}, {{{30, 2000, 1976}, {3, 7000, 1536}}, NARROW, NARROW, BLOCKS}, {{{30, 3000, 1976}, {3, 17000, 1536}}, TWO, SLIM, BLOCKS},
            // calls over a part of a context: two kernels, and parts of blocks left, by what most of the call is
            {{{110, 1024, 1096}, {1, 5000, 3072}}, WIDE, WIDE, BLOCKS, 0, 110}, {{{110, 1024, 1096}, {1, 5000, 3072}}, WIDE, WIDE, WHOLE, 110, 1},
            {{{30, 4800, 1096}, {25, 4800, 1088}}, TWO, NARROW, BLOCKS}, {{{30, 4800, 1096}, {25, 4800, 1088}}, TWO, NARROW, BLOCKS, 0, 30},
            {{{30, 4800, 1096}, {25, 4800, 1088}}, NARROW, NARROW, WHOLE, 30, 25}, {{{30, 4800, 1096}, {25, 4800, 1088}}, NARROW, NARROW, WHOLE, 25, 12},
            {{{30, 4800, 1096}, {25, 4800, 1088}}, TWO, NARROW, BLOCKS, 20, 19}, {{{20, 9000, 1104}, {10, 4096, 1104}}, TWO, NARROW, WHOLE},
            {{{20, 9000, 1104}, {10, 4096, 1104}}, NARROW, NARROW, WHOLE, 20, 10}, {{{20, 9000, 1104}, {15, 9000, 1088}}, NARROW, NARROW, WHOLE, 20, 15},
            {{{60, 4096, 1096}, {20, 4096, 1088}}, WIDE, WIDE, WHOLE, 60, 20}, {{{60, 4096, 1096}, {30, 4096, 1088}}, NARROW, NARROW, WHOLE, 60, 30}, {{{10, 13000, 1096}, {8, 13000, 1088}}, NARROW, NARROW, WHOLE, 10, 8},
            // parts of blocks from 54 MB on (45 in 128 channels, 36 in 64): 9 x 10^6 elements of a step with fp32 errors, 13.5 of one sent or of a step with bf16 errors, 27 sent with bf16 errors
            {{{9, 1000, 1000}}, WIDE, WIDE, STEPS}, {{{9, 1000, 984}}, WIDE, WIDE, WHOLE}, {{{9, 1500, 1000}}, WIDE, WIDE, BLOCKS}, {{{9, 1500, 984}}, WIDE, WIDE, STEPS},
            {{{9, 1500, 1000}}, WIDE, WIDE, STEPS, 0, 0, 0, E}, {{{9, 1500, 984}}, WIDE, WIDE, WHOLE, 0, 0, 0, E}, {{{9, 3000, 1000}}, WIDE, WIDE, BLOCKS, 0, 0, 0, E},
            {{{9, 3000, 984}}, WIDE, WIDE, STEPS, 0, 0, 0, E}, {{{40, 1000, 1000}}, WIDE, WIDE, STEPS, 3, 9},
            {{{1, 9000, 840}}, NARROW, NARROW, STEPS}, {{{1, 9000, 824}}, NARROW, NARROW, WHOLE}, {{{1, 9000, 1256}}, NARROW, NARROW, BLOCKS}, {{{1, 9000, 1240}}, NARROW, NARROW, STEPS},
            {{{1, 16400, 376}}, SLIM, SLIM, STEPS}, {{{1, 16400, 360}}, SLIM, SLIM, WHOLE}, {{{1, 16400, 552}}, SLIM, SLIM, BLOCKS}, {{{1, 16400, 536}}, SLIM, SLIM, STEPS},
            // short items: from 449 items and 17 MB on
            {{{30, 1024, 1096}, {9, 1024, 1088}}, SHORT, SHORT, BLOCKS, 0, 6}, {{{30, 1024, 1096}, {9, 1024, 1088}}, SHORT, SHORT, WHOLE, 0, 3},
            {{{30, 1024, 1096}, {9, 1024, 1088}}, SHORT, SHORT, WHOLE, 30, 6}, {{{30, 1024, 1104}}, SHORT, SHORT, BLOCKS, 0, 6}, {{{30, 1024, 1096}}, SHORT, SHORT, STEPS, 0, 6, 0, E},
            {{{8, 449, 984}}, SHORT, SHORT, STEPS}, {{{8, 449, 984}}, SHORT, SHORT, WHOLE, 0, 0, 0, E}, {{{8, 1024, 440}}, SHORT, SHORT, WHOLE}, {{{8, 1024, 456}}, SHORT, SHORT, STEPS}, {{{8, 1024, 520}}, SHORT, SHORT, BLOCKS},
            // the kernels that the GPU tests of the single pass are for: a rule that changes must not take a test to another one unnoticed (tokens x channels; a fourth number: fp32)
            {{{1, 10241, 64}, {1, 10241, 160}, {1, 512, 120}, {1, 513, 136}, {1, 1, 64}, {1, 255, 56}}, SLIM, SLIM, WHOLE, 0, 0, FORCED},
            {{{5, 3072, 288}, {5, 1000, 1120}}, WIDE, WIDE, WHOLE, 0, 0, FORCED}, {{{5, 3073, 288}, {5, 1000, 1120}}, NARROW, NARROW, WHOLE, 0, 0, FORCED},
            {{{5, 4096, 288}, {5, 4000, 160}}, NARROW, NARROW, WHOLE, 0, 0, FORCED}, {{{5, 4608, 264}, {5, 1000, 1096}}, WIDE, WIDE, STEPS, 0, 0, FORCED},
            {{{5, 4609, 264}, {5, 1000, 1096}}, NARROW, NARROW, BLOCKS, 0, 0, FORCED},
            {{{6, 1500, 1096}, {3, 700, 520, CF_F32}}, WIDE, WIDE, STEPS, 0, 0, FORCED}, {{{6, 1500, 1120}, {3, 700, 544, CF_F32}}, WIDE, WIDE, WHOLE, 0, 0, FORCED},
            {{{3, 1500, 1096}, {3, 700, 520, CF_F32}, {1, 130, 72}, {1, 1, 8, CF_F32}}, SHORT, SHORT, BLOCKS, 0, 0, FORCED},
            {{{3, 1500, 1120}, {3, 700, 544, CF_F32}, {1, 130, 96}, {1, 1, 8, CF_F32}, {2, 300, 96}}, WIDE, WIDE, WHOLE, 0, 0, FORCED},
            {{{6, 40000, 72}}, NARROW, NARROW, BLOCKS, 0, 0, FORCED}, {{{6, 40000, 80}}, NARROW, NARROW, WHOLE, 0, 0, FORCED}, {{{6, 40000, 96}}, SLIM, SLIM, WHOLE, 0, 0, FORCED},
            {{{7, 1153, 328}, {7, 1152, 264}, {7, 1151, 1096}}, WIDE, WIDE, BLOCKS, 0, 0, FORCED}, {{{10, 1024, 1104}, {10, 1023, 336}, {10, 1022, 16}}, WIDE, WIDE, BLOCKS, 0, 0, FORCED},
            {{{10, 4700, 104}, {10, 4699, 136}, {10, 4698, 72}}, NARROW, NARROW, BLOCKS, 0, 0, FORCED}, {{{1, 12291, 552}, {1, 12290, 568}}, NARROW, NARROW, BLOCKS, 0, 0, FORCED},
            {{{1, 16387, 424}, {1, 16386, 408}}, SLIM, SLIM, BLOCKS, 0, 0, FORCED}, {{{1, 4097, 760}, {1, 4096, 776}}, SHORT, SHORT, BLOCKS, 0, 0, FORCED},
            {{{1, 4097, 752}, {1, 4096, 784}}, SHORT, SHORT, BLOCKS, 0, 0, FORCED},
            {{{7, 1153, 328}, {7, 1152, 264}, {7, 1151, 1096}}, WIDE, WIDE, STEPS, 0, 0, FORCED, E}, {{{10, 1024, 1104}, {10, 1023, 336}, {10, 1022, 16}}, WIDE, WIDE, STEPS, 0, 0, FORCED, E},
            {{{10, 4700, 104}, {10, 4699, 136}, {10, 4698, 72}}, NARROW, NARROW, STEPS, 0, 0, FORCED, E}, {{{1, 12291, 552}, {1, 12290, 568}}, NARROW, NARROW, STEPS, 0, 0, FORCED, E},
            {{{1, 16387, 424}, {1, 16386, 408}}, SLIM, SLIM, STEPS, 0, 0, FORCED, E}, {{{1, 4097, 760}, {1, 4096, 776}}, SHORT, SHORT, STEPS, 0, 0, FORCED, E},
            {{{14, 1153, 328}, {14, 1152, 264}, {14, 1151, 1096}}, WIDE, WIDE, BLOCKS, 0, 0, FORCED, E}, {{{20, 4700, 104}, {20, 4699, 136}, {20, 4698, 72}}, NARROW, NARROW, BLOCKS, 0, 0, FORCED, E},
            {{{2, 16387, 424}, {2, 16386, 408}}, SLIM, SLIM, BLOCKS, 0, 0, FORCED, E}, {{{1, 8192, 64}, {1, 4096, 512}, {1, 1000, 136}}, SHORT, SHORT, WHOLE, 0, 0, FORCED},
            {{{1, 4097, 760}, {1, 4097, 776}}, SHORT, SHORT, BLOCKS, 0, 0, FORCED}, {{{1, 9000, 136}, {1, 4096, 512}}, NARROW, NARROW, WHOLE, 0, 0, FORCED},
            {{{1, 9000, 520}, {1, 9000, 536}}, NARROW, NARROW, STEPS, 0, 0, FORCED}, {{{1, 12500, 224}, {1, 20000, 96}}, SLIM, SLIM, WHOLE, 0, 0, FORCED},
            {{{1, 12500, 224}, {1, 20000, 96}}, SLIM, SLIM, WHOLE, 0, 0, FORCED, E}, {{{1, 16400, 424}, {1, 20000, 136}}, SLIM, SLIM, BLOCKS, 0, 0, FORCED},
            {{{9, 2000, 1056}}, WIDE, WIDE, WHOLE, 0, 0, FORCED}, {{{9, 2000, 1032}}, WIDE, WIDE, BLOCKS, 0, 0, FORCED},
        };
        for (size_t k = 0; k < calls.size(); ++k) {
            const Call &c = calls[k];
            std::vector<cf_tensor_desc> d;
            for (auto &s : c.shapes) d.insert(d.end(), (size_t)s[0], desc(s[1], s[2], s.size() > 3 ? (int)s[3] : CF_BF16, 2, CF_SCALE_CHANNEL));
            const int n = (int)d.size(), first = c.first, count = c.count ? c.count : n - first;
            std::memset(&o, 0, sizeof o);
            o.flags = c.flags;
            o.err_dtype = c.err;
            std::vector<void *> bufs[5];
            uintptr_t at = (uintptr_t)1 << 40;
            for (auto &b : bufs)
                for (int t = 0; t < n; ++t, at += (uintptr_t)1 << 32) b.push_back((void *)at);
            const size_t wsb = cf_workspace_bytes(d.data(), n, &o);
            void *ws = nullptr;
            if (posix_memalign(&ws, 256, wsb) != 0) std::abort();
            cf_ctx *ctx = nullptr;
            EXPECT(cf_init(&ctx, d.data(), n, &o, ws, wsb, nullptr) == CF_OK);
            EXPECT(cf_set_warm(ctx, 0, n, 1) == CF_OK);
            for (bool send : {false, true}) {
                joined();
                g_single_pass_slim = g_single_pass_wide = g_single_pass_short = g_single_pass_blocks = false;
                EXPECT((send ? cf_compress(ctx, first, count, (const void *const *)bufs[0].data() + first, (const void *const *)bufs[1].data() + first, bufs[2].data() + first,
                                           bufs[3].data() + first, bufs[4].data() + first, nullptr)
                             : cf_step_fused(ctx, first, count, (const void *const *)bufs[0].data() + first, bufs[1].data() + first, bufs[2].data() + first,
                                             bufs[3].data() + first, bufs[4].data() + first, nullptr)) == CF_OK);
                const Path took = joined().find("k_single_pass ") == std::string::npos ? TWO : g_single_pass_short ? SHORT : g_single_pass_slim ? SLIM : g_single_pass_wide ? WIDE : NARROW;
                if (took != (send ? c.send : c.step) || (took != TWO && g_single_pass_blocks != (c.stores == BLOCKS || (c.stores == STEPS && !send)))) {
                    std::printf("uneven call %zu %s: path %d, parts of blocks %d\n", k, send ? "sent" : "step", (int)took, (int)g_single_pass_blocks);
                    ++g_failed;
                }
            }
            cf_destroy(ctx);
            std::free(ws);
        }
    }

    // ---- short items: calls of at most 8 channel-scale tensors, 1024 items and 64 items of 128 rows (64 of fp32) x 64 channels a group
    {
        struct Call { int32_t ef, dtype; uint32_t flags; std::vector<std::vector<int64_t>> shapes; bool is_short; int compute_units = 256; };
        const int R = CF_EF_RECON, B = CF_BF16, F = CF_F32;
        const std::vector<Call> calls = {
            {R, F, 0, {{1, 256, 64}}, true}, {R, B, 0, {{1, 1, 8}}, true}, {R, B, 0, {{2, 1024, 3072}}, true},
            {R, B, 0, {{1, 8192, 1024}}, true}, {R, B, 0, {{1, 8193, 64}}, false}, {R, F, 0, {{1, 4096, 1024}}, true}, {R, F, 0, {{1, 4097, 64}}, false},
            {R, B, 0, {{1, 8192, 1032}}, false}, {R, B, 0, {{1, 128, 65536}}, true}, {R, B, 0, {{1, 129, 65536}}, false},
            {R, B, 0, {{8, 128, 8192}}, true}, {R, B, 0, {{8, 129, 8192}}, false}, {R, B, 0, {{9, 64, 256}}, false},
            {R, B, CF_FLAG_FIXED_GRID, {{1, 256, 64}}, false}, {R, B, CF_FLAG_TEST_NO_WAIT, {{1, 256, 64}}, true},
            {CF_EF_OFF, B, 0, {{1, 256, 64}}, false}, {CF_EF_NAIVE, B, 0, {{1, 256, 64}}, false},
            {R, B, 0, {{1, 256, 64}, {1, 9000, 64}, {1, 300, 64}}, false},
            {R, B, 0, {{64, 64, 256}}, false}, {R, B, 0, {{65, 64, 256}}, false},      // 64 take their pointers along
            // tensors of several shapes: no more than 64 workgroups without an item, whatever the largest numbers of row blocks and stripes are
            {R, B, 0, {{7, 8192, 64}, {1, 64, 4096}}, true}, {R, B, 0, {{1, 8192, 64}, {1, 8, 61440}}, true}, {R, B, 0, {{1, 8192, 64}, {1, 128, 3072}}, true},
            {R, B, 0, {{1, 2048, 512}, {1, 1024, 512}}, true}, {R, B, 0, {{1, 2048, 512}, {1, 896, 512}}, true}, {R, B, 0, {{1, 1024, 3072}, {2, 256, 2048}}, true}, {R, F, 0, {{3, 1, 8}, {1, 4096, 64}, {1, 70, 2048}, {1, 65, 64}}, true},
            {R, B, 0, {{1, 8192, 128}}, true, 32}, {R, B, 0, {{1, 8192, 136}}, false, 32}, {R, B, 0, {{1, 8192, 136}}, true, 64},     // a smaller device: 128 items
        };
        for (const Call &c : calls) {
            std::vector<cf_tensor_desc> d;
            for (auto &s : c.shapes) d.insert(d.end(), (size_t)s[0], desc(s[1], s[2], c.dtype, 2, CF_SCALE_CHANNEL));
            const int n = (int)d.size();
            std::memset(&o, 0, sizeof o);
            o.ef = c.ef;
            o.flags = c.flags;
            g_compute_units = c.compute_units;
            std::vector<void *> bufs[5];
            uintptr_t at = (uintptr_t)1 << 40;
            for (auto &b : bufs)
                for (int t = 0; t < n; ++t, at += (uintptr_t)1 << 32) b.push_back((void *)at);
            const size_t wsb = cf_workspace_bytes(d.data(), n, &o);
            void *ws = nullptr;
            if (posix_memalign(&ws, 256, wsb) != 0) std::abort();
            cf_ctx *ctx = nullptr;
            EXPECT(cf_init(&ctx, d.data(), n, &o, ws, wsb, nullptr) == CF_OK);
            EXPECT(cf_set_warm(ctx, 0, n, 1) == CF_OK);
            joined();
            for (int first = 0; first < n; first += n > 1 ? n - 1 : 1) {        // the whole context, and its last tensor alone
                g_single_pass_short = false;
                EXPECT(cf_step_fused(ctx, first, n - first, (const void *const *)bufs[0].data() + first, bufs[1].data() + first, bufs[2].data() + first,
                                     bufs[3].data() + first, bufs[4].data() + first, nullptr) == CF_OK);
                const std::string seq = joined();
                {
                    void *events[2] = {(void *)0x10, (void *)0x20};
                    EXPECT(cf_profile_next_call(ctx, events, 1) == CF_OK);
                    EXPECT(cf_step_fused(ctx, first, n - first, (const void *const *)bufs[0].data() + first, bufs[1].data() + first, bufs[2].data() + first,
                                         bufs[3].data() + first, bufs[4].data() + first, nullptr) == CF_OK);
                    joined();
                    const char *name = cf_profile_kernel_name(ctx, cf_profile_launch_count(ctx) - 1);
                    EXPECT(name && std::strcmp(name, g_single_pass_short ? "k_short_items" : "k_single_pass") == 0);
                }
                EXPECT(seq.find("wrong items") == std::string::npos && seq.find("wrong grid") == std::string::npos);
                if (g_single_pass_short) {
                    int items = 0;
                    for (int t = first; t < n; ++t) {
                        const int rows = d[(size_t)t].dtype == F ? 64 : 128;
                        items += (int)((d[(size_t)t].n_tokens + rows - 1) / rows * ((d[(size_t)t].n_channels + 63) / 64));
                    }
                    if (g_short_workgroups < items || g_short_workgroups > items + 64) {
                        std::printf("%d tensors from [%d, %d] on: %d workgroups for %d short items\n", n - first, (int)d[(size_t)first].n_tokens, (int)d[(size_t)first].n_channels, g_short_workgroups, items);
                        ++g_failed;
                    }
                }
                EXPECT(seq.find("k_single_pass") != std::string::npos && uploaded(seq) == (n - first > 64));
                if (first > 0 && !c.is_short) continue;
                if (g_single_pass_short != c.is_short) {
                    const auto &s = c.shapes.back();
                    std::printf("ef %d dtype %d ... %d x [%d, %d]: short items %d\n", c.ef, c.dtype, (int)s[0], (int)s[1], (int)s[2], (int)g_single_pass_short);
                    ++g_failed;
                }
            }
            cf_destroy(ctx);
            std::free(ws);
        }
        g_compute_units = 256;
    }

    // ---- single passes carry their item states on from call to call; once they came on several streams, on hipStreamPerThread or under
    // capture, a warm-up makes them agree again, whatever calls that overlapped have left, and leaves its neighbours' alone
    for (int64_t tokens : {1000, 60000}) {      // short items, and tall ones
        const std::vector<cf_tensor_desc> d = {desc(tokens, 72, CF_BF16, 1, CF_SCALE_CHANNEL), desc(tokens, 200, CF_BF16, 1, CF_SCALE_CHANNEL),
                                               desc(64, 128, CF_BF16, 4, CF_SCALE_GROUP), desc(tokens, 72, CF_BF16, 1, CF_SCALE_CHANNEL)};
        const int n = (int)d.size();
        std::memset(&o, 0, sizeof o);
        o.flags = CF_FLAG_SINGLE_PASS;
        std::vector<void *> bufs[5];
        uintptr_t at = (uintptr_t)1 << 40;
        for (auto &b : bufs)
            for (int t = 0; t < n; ++t, at += (uintptr_t)1 << 32) b.push_back((void *)at);
        const size_t wsb = cf_workspace_bytes(d.data(), n, &o);
        void *ws = nullptr;
        if (posix_memalign(&ws, 256, wsb) != 0) std::abort();
        std::memset(ws, 0, wsb);
        cf_ctx *ctx = nullptr;
        void *const a = (void *)0x1000, *const b = (void *)0x2000;
        const auto step = [&](int first, int count, void *stream) {
            EXPECT(cf_step_fused(ctx, first, count, (const void *const *)bufs[0].data() + first, bufs[1].data() + first, bufs[2].data() + first,
                                 bufs[3].data() + first, bufs[4].data() + first, stream) == CF_OK);
            const std::string seq = joined();
            EXPECT(seq.find("k_single_pass") != std::string::npos && seq.find("k_fresh_partials") == std::string::npos);
        };
        const auto warm_up = [&](int first, int count, void *stream) {     // how many launches set states anew
            EXPECT(cf_warmup(ctx, first, count, (const void *const *)bufs[0].data() + first, bufs[1].data() + first, bufs[2].data() + first, stream) == CF_OK);
            const std::string seq = joined();
            EXPECT(seq.find("k_warmup") != std::string::npos && seq.find("misplaced") == std::string::npos);
            int times = 0;
            for (size_t p = seq.find("k_fresh_partials"); p != std::string::npos; p = seq.find("k_fresh_partials", p + 1)) ++times;
            return times;
        };
        const int geometries = tokens == 1000 ? 2 : 1;
        const auto set_up = [&] {
            cf_destroy(ctx);
            EXPECT(cf_init(&ctx, d.data(), n, &o, ws, wsb, b) == CF_OK);
            joined();
            EXPECT(warm_up(0, n, b) == 0);
        };
        const auto agree = [&](uint8_t state) {
            for (uint8_t found : g_states)
                if (found != state) return false;
            return !g_states.empty();
        };
        for (int how = 0; how < 4; ++how) {
            set_up();
            for (int k = 0; k < 3; ++k) {       // cf_init's own stream, or the warm-up's, may be another one
                step(0, 2, a);
                EXPECT(agree(k % 2 ? 0u : 0x80u) && g_single_pass_short == (tokens == 1000));
                EXPECT(warm_up(1, 1, a) == 0);
            }
            step(0, n, a);                      // by the table: items as elsewhere
            EXPECT(!g_single_pass_short);
            if (how == 0) step(0, 1, b);
            if (how == 1) step(0, 1, (void *)hipStreamPerThread);
            g_capturing = how == 2;
            step(0, 1, a);
            g_capturing = false;
            if (how == 3) {                     // one stream, no capture
                EXPECT(warm_up(0, n, a) == 0);
                continue;
            }
            g_overlapping = true;
            step(0, 2, a);
            if (geometries == 2) step(0, n, a);
            g_overlapping = false;
            step(0, 2, a);
            EXPECT(!agree(0u) && !agree(0x80u));
            EXPECT(warm_up(2, 1, b) == 0);      // no channel scales
            EXPECT(warm_up(1, 1, a) == geometries);
            step(1, 1, a);
            EXPECT(agree(0x80u));
            EXPECT(warm_up(0, n, a) == geometries);
            step(0, 2, a);
            EXPECT(agree(0x80u));
            EXPECT(warm_up(0, n, a) == geometries);
            step(0, n, a);
            EXPECT(agree(0x80u) && !g_single_pass_short);
        }
        // a warm-up leaves what lies next to it as it was
        set_up();
        step(0, 2, a);
        step(0, 4, b);
        EXPECT(warm_up(1, 1, a) == geometries);
        const std::vector<uint8_t> before((const uint8_t *)ws, (const uint8_t *)ws + wsb);
        step(1, 1, a);
        EXPECT(std::memcmp(before.data(), ws, wsb) != 0);
        EXPECT(warm_up(1, 1, a) == geometries);
        EXPECT(std::memcmp(before.data(), ws, wsb) == 0);
        cf_destroy(ctx);
        std::free(ws);
    }

    // ---- the low-rank kernels' rules count the low-rank tensors of a call as they are, and nothing else
    {
        struct Group { int count; int64_t n, c; int dtype, scale; };
        struct Call { std::vector<Group> groups; bool many; int split; };
        const int B = CF_BF16, F = CF_F32, L = CF_LOWRANK, Q = CF_SCALE_CHANNEL;
        const std::vector<Call> calls = {
            {{{4, 4096, 3072, B, L}}, false, 4}, {{{13, 4096, 1536, B, L}}, false, 2}, {{{14, 4096, 1536, B, L}}, true, 2},       // 512, 1664, 1792 blocks of 128 tokens
            {{{14, 4096, 1536, F, L}}, false, 2},
            {{{1, 4096, 3072, B, L}, {7, 4096, 3072, B, Q}}, false, 4}, {{{100, 64, 64, B, Q}, {1, 4096, 3072, B, L}}, false, 4},
            {{{1, 8192, 3072, B, L}, {9, 64, 96, B, L}}, false, 4}, {{{8, 64, 96, F, L}, {1, 65536, 1536, B, L}}, true, 4},     // 256 + 9, 2048 blocks
            {{{64, 4096, 3072, B, L}}, true, 2}, {{{65, 4096, 3072, B, L}}, true, 1},                                           // 768, 780 stripes
            {{{65, 4096, 256, F, L}, {1, 4096, 2048, B, L}}, false, 2},                                                         // 73 stripes: what the workspace holds
        };
        for (size_t k = 0; k < calls.size(); ++k) {
            std::vector<cf_tensor_desc> d;
            for (auto &g : calls[k].groups) d.insert(d.end(), (size_t)g.count, desc(g.n, g.c, g.dtype, g.scale == L ? 1 : 2, g.scale, g.scale == L ? 32 : 128));
            const int n = (int)d.size();
            std::memset(&o, 0, sizeof o);
            std::vector<const void *> x;
            std::vector<void *> recon, err, codes, scales;
            uintptr_t at = (uintptr_t)1 << 40;
            auto take = [&] { void *p = (void *)at; at += (uintptr_t)1 << 32; return p; };
            for (int t = 0; t < n; ++t) { x.push_back(take()); recon.push_back(take()); err.push_back(take()); codes.push_back(take()); scales.push_back(take()); }
            const size_t wsb = cf_workspace_bytes(d.data(), n, &o);
            void *ws = nullptr;
            if (posix_memalign(&ws, 256, wsb) != 0) std::abort();
            cf_ctx *ctx = nullptr;
            EXPECT(cf_init(&ctx, d.data(), n, &o, ws, wsb, nullptr) == CF_OK);
            EXPECT(cf_set_warm(ctx, 0, n, 1) == CF_OK);
            EXPECT(cf_step_fused(ctx, 0, n, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_OK);
            joined();
            if (g_project_many != calls[k].many || g_split != calls[k].split) {
                std::printf("low-rank call %zu: several blocks a wave %d, shares %d\n", k, (int)g_project_many, g_split);
                ++g_failed;
            }
            cf_destroy(ctx);
            std::free(ws);
        }
    }

    // ---- the low-rank apply kernel's tiles: each of a row to one wave, and at most one wave short of a tile
    for (int channels = 32; channels <= cf::kLowRankMaxChannels; channels += 32)
        for (int per_wave = 1; per_wave <= 2; ++per_wave) {
            const int n_tiles = (channels + 63) / 64, waves = cf::lowrank_apply_waves(channels, per_wave);
            std::vector<int> owners((size_t)n_tiles, 0);
            for (int w = 0; w < waves; ++w) {
                const cf::ApplyTiles a = cf::lowrank_apply_tiles(channels, per_wave, w);
                int mine = 0;
                EXPECT(a.first >= 0 && a.step >= 1 && a.end <= n_tiles);
                for (int t = a.first; t < a.end; t += a.step, ++mine) ++owners[(size_t)t];
                EXPECT(mine >= 1 && mine <= per_wave);
            }
            for (int o : owners) EXPECT(o == 1);
            EXPECT(waves * per_wave <= n_tiles + 1);
        }

    // ---- the entry point that brings no workspace
    {
        std::memset(&o, 0, sizeof o);
        std::vector<cf_tensor_desc> many(40, desc(4096, 3072, CF_BF16, 2, CF_SCALE_CHANNEL));
        const void *nothing[40] = {};
        EXPECT(cf_step_fused_static(many.data(), 40, &o, nothing, (void *const *)nothing, (void *const *)nothing, (void *const *)nothing,
                                    (void *const *)nothing, nullptr) == CF_ERR_WORKSPACE);
        EXPECT(cf_workspace_bytes(many.data(), 40, &o) > CF_STATIC_SCRATCH_BYTES);
        // what fits with the stripes of other rows is taken, though a context of the caller's would have the larger partials of rows that are no whole blocks of 64 bytes
        struct Batch { int64_t n, c; std::vector<int> counts; };
        for (const Batch &b : {Batch{4096, 1096, {14, 24, 26, 40, 47}}, Batch{4096, 3080, {5, 9, 16}}, Batch{3300, 3080, {6, 11, 20}}, Batch{4000, 520, {29, 30, 52, 57, 85, 101}},
                               Batch{12500, 1096, {9, 16, 17}}, Batch{16000, 1096, {7, 13}}})
            for (int count : b.counts) {
                const std::vector<cf_tensor_desc> d((size_t)count, desc(b.n, b.c, CF_BF16, 2, CF_SCALE_CHANNEL));
                std::vector<void *> bufs[5];
                uintptr_t at = (uintptr_t)1 << 40;
                for (auto &v : bufs)
                    for (int t = 0; t < count; ++t, at += (uintptr_t)1 << 32) v.push_back((void *)at);
                joined();
                EXPECT(cf_workspace_bytes(d.data(), count, &o) > CF_STATIC_SCRATCH_BYTES);
                for (int round = 0; round < 2; ++round) {
                    const cf_status st = cf_step_fused_static(d.data(), count, &o, (const void *const *)bufs[0].data(), bufs[1].data(), bufs[2].data(), bufs[3].data(), bufs[4].data(), nullptr);
                    if (st != CF_OK) { std::printf("static step over %d x [%d, %d]: status %d\n", count, (int)b.n, (int)b.c, (int)st); ++g_failed; }
                    EXPECT(st != CF_OK || !joined().empty());
                }
            }
        for (int round = 0; round < 3; ++round) {
            std::vector<cf_tensor_desc> some = round == 1 ? std::vector<cf_tensor_desc>{desc(256, 64, CF_F32, 2, CF_SCALE_CHANNEL)}
                                                          : std::vector<cf_tensor_desc>{desc(2048, 1024, CF_BF16, 1, CF_SCALE_CHANNEL), desc(300, 384, CF_BF16, 4, CF_SCALE_GROUP)};
            std::vector<Buffers *> buf;
            std::vector<const void *> x;
            std::vector<void *> recon, err, codes, scales;
            for (auto &d : some) {
                buf.push_back(new Buffers(d, &o));
                x.push_back(buf.back()->x); recon.push_back(buf.back()->recon); err.push_back(buf.back()->err);
                codes.push_back(buf.back()->codes); scales.push_back(buf.back()->scales);
            }
            EXPECT(cf_step_fused_static(some.data(), (int)some.size(), &o, x.data(), recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_OK);
            EXPECT(!joined().empty());
            EXPECT(cf_step_fused_static(some.data(), (int)some.size(), &o, nullptr, recon.data(), err.data(), codes.data(), scales.data(), nullptr) == CF_ERR_INVALID_ARG);
            for (auto *p : buf) delete p;
        }
    }
    if (g_failed) { std::printf("%d expectations failed\n", g_failed); return 1; }
    std::printf("host half of the C ABI: all expectations hold\n");
    return 0;
}
