// Which launch a net's update takes and how much scratch it asks for, without a GPU: the library's host code on handles that
// only have a configuration.  Prints "ok" or what is wrong.
#include <stdio.h>
#include <unistd.h>
#include "../../paper_2104_06272_amd/csrc/anakin.hip"

static anakin handle(int rows, int cols, std::initializer_list<int> hidden, int B, int T)
{
    anakin h{};
    anakin_env_cfg env{ANAKIN_ENV_CATCH, rows, cols, rows - 1, 0.0f};
    anakin_net_cfg net{};
    for (int w : hidden) net.hidden[net.n_hidden++] = w;
    net.policy = ANAKIN_POLICY_CATEGORICAL; net.dtype = ANAKIN_DTYPE_FP32;
    net.gamma = 0.99f; net.lambda_ = 1.0f; net.lr = 1e-3f; net.beta1 = 0.9f; net.beta2 = 0.999f; net.eps = 1e-8f;
    std::string err;
    if (build_shapes(&env, &net, B, T, h.env, h.net, err) != ANAKIN_OK) { printf("not taken: %d x %d, %d x %d: %s\n", rows, cols, B, T, err.c_str()); fflush(stdout); _exit(1); }
    h.env_cfg = env; h.net_cfg = net; h.B = B; h.T = T; h.n_updates = 1;
    plan(h.env, h.net, B, T, h.splits, h.quanta, &h.splits_w, &h.head_fan, &h.loss_blocks);
    return h;
}

int main()
{
    auto bad = [](const char* what, int rows, int cols, int B, int T, long long v) {
        printf("%s: %d x %d cells, %d environments, T = %d: %lld\n", what, rows, cols, B, T, v);
        fflush(stdout); _exit(1);
    };
    // Catch, 32 units: one launch for the whole update where it was measured to be the faster one, and not where it was not
    struct { int B, T; bool one; } route[] = {
        {24576, 1, true}, {49152, 1, true}, {16384, 1, false}, {24576, 2, true}, {16384, 2, false}, {40960, 4, true}, {49152, 4, true}, {32768, 4, false},
        {4096, 4, false}, {40960, 8, false}, {45056, 8, false}, {34816, 4, true}, {53248, 8, true}, {49152, 16, false}, {65536, 16, true}, {49152, 64, false}, {262144, 16, true}};
    for (const auto& r : route) {
        const anakin h = handle(10, 5, {32}, r.B, r.T);
        if (catch_fused_shape(h.net, h.env, r.B, r.T) != r.one) bad(r.one ? "should be one launch" : "should not be one launch", 10, 5, r.B, r.T, h.splits[0]);
        // the launch's workgroups have whole blocks of 256 environments and room for their sums; the same net's other updates keep
        // chunks of 64 samples, as many as they would have without it
        const int groups = catch_fused_groups(h.net, h.env, r.B, r.T);
        if (r.one != (groups > 0) || (r.one && ((r.B / 256) % groups || groups > h.splits[0] || h.splits[0] != h.splits[1]))) bad("workgroups", 10, 5, r.B, r.T, groups);
        const int fine = pick_splits(r.B * r.T, 1, 512, 64);
        if (h.splits[0] != fine) bad("chunks of the other updates", 10, 5, r.B, r.T, h.splits[0]);
    }
    // Catch, 256 units: boards in two tiles of 32 cells
    for (int rows = 2; rows <= 40; ++rows)
        for (int cols = 1; cols <= 40; ++cols) {
            const anakin h = handle(rows, cols, {256}, 64, 3);
            if (one_layer_learn_shape(h.net, h.env) != (rows * cols <= 64)) bad("256 units", rows, cols, 64, 3, rows * cols);
        }
    // Catch, 32 units, boards beyond the one-layer kernels: whatever the static scratch held with a chunk per 256 environments
    // (halved down to 512), and a first stage of the head gradient of 16 workgroups for each, it still holds
    auto scratch = [](const anakin& h) { Layout L; return carve_update_scratch(h.env, h.net, h.B, h.T, h.splits, h.splits_w, h.head_fan, L, 0); };
    auto holds = [&](int rows, int cols, int B, int T) {
        const anakin h = handle(rows, cols, {32}, B, T);
        if (one_layer_shape(h.net, h.env) || (h.env.kind == ANAKIN_ENV_CATCH && h.net.dims[0] <= 102)) bad("a board of the one-layer kernels", rows, cols, B, T, h.net.dims[0]);
        long long had = B / 256;
        while (had > 512 && had % 2 == 0) had /= 2;
        const long long was = (long long)B * T * (32 + 4) * 4 + had * ((rows * cols + 1) * 32 + 17 * 33 * 4) * 4 + 16 * 256;
        const long long now = (long long)scratch(h), fits = ANAKIN_STATIC_SCRATCH_BYTES;
        if (was <= fits && now > fits) bad("fitted before", rows, cols, B, T, now);
        if ((long long)h.splits[0] * chunk_rows(B * T, h.splits[0], h.quanta[0]) < (long long)B * T) bad("samples without a chunk", rows, cols, B, T, h.splits[0]);
        if ((long long)(h.splits[0] - 1) * chunk_rows(B * T, h.splits[0], h.quanta[0]) >= (long long)B * T) bad("empty chunk", rows, cols, B, T, h.splits[0]);
        return was <= fits;
    };
    int near = 0;
    near += holds(16, 14, 8192, 48) + holds(11, 12, 8704, 50) + holds(13, 9, 8704, 49) + holds(11, 11, 53504, 8) + holds(16, 11, 10752, 42);
    if (near != 5) bad("a fixed shape did not fit before", 0, 0, 0, 0, near);
    unsigned state = 11;
    auto rnd = [&](int n) { state = state * 1664525u + 1013904223u; return (int)((state >> 8) % (unsigned)n); };
    for (int k = 0; k < 20000; ++k) {
        const int rows = 2 + rnd(30), cols = (103 + rows - 1) / rows + rnd(16), B = 256 * (1 + rnd(1 << rnd(10)));
        if (cols <= 255) holds(rows, cols, B, 1 + rnd(64));
    }
    printf("ok\n");
    fflush(stdout);
    _exit(0);                                                    // no GPU: nothing of the runtime to take down
}
