// Which forms of the split-operand products (gemm_split.hip) a shape runs, without a GPU.  Standard input: one shape a line,
// "env bf16 rows cols B T width width ...".  Output, a line for each: "samples<few|many> tile_i x tile_j / dX columns, heads,
// first layer" of every layer that takes them, joined by spaces; "off" where the bf16 matrix path takes the net.
#include <stdio.h>
#include <unistd.h>
#include <sstream>
#include <iostream>
#include "../../paper_2104_06272_amd/csrc/anakin.hip"

int main()
{
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        anakin_env_cfg env;
        anakin_net_cfg net;
        memset(&env, 0, sizeof env); memset(&net, 0, sizeof net);
        int B = 0, T = 0;
        in >> env.kind >> net.dtype >> env.rows >> env.cols >> B >> T;
        for (int w; in >> w;) net.hidden[net.n_hidden++] = w;
        env.max_steps = 9;
        net.policy = env.kind == ANAKIN_ENV_PENDULUM ? ANAKIN_POLICY_TANH_GAUSSIAN : ANAKIN_POLICY_CATEGORICAL;
        net.gamma = 0.99f; net.lambda_ = 1.0f; net.lr = 1e-3f; net.beta1 = 0.9f; net.beta2 = 0.999f; net.eps = 1e-8f;
        EnvDims ed; NetShape ns; std::string err, out;
        if (build_shapes(&env, &net, B, T, ed, ns, err) != ANAKIN_OK) { printf("refused: %s\n", err.c_str()); continue; }
        if (!ns.split) { printf("off\n"); continue; }
        for (int l = 1; l < ns.L; ++l) {
            if (!split_gemm_shape(ns, l)) continue;
            const bool heads = heads_fused_shape(ns) && l == ns.L - 1, first = first_fused_splits(ns, ed, B * T) > 0 && l == 1;
            out += std::string(ns.split == 2 ? "few" : "many") + ":" + std::to_string(split_tile_i(ns, l)) + "x" + std::to_string(split_tile_j(ns, l)) + "/" +
                   std::to_string(split_nt_cols(ns, l)) + (heads ? ns.NH > 4 ? ":heads5" : ":heads" : "") +
                   (!first ? "" : ed.kind == ENV_CATCH ? ":board" : ":first") + " ";
        }
        printf("%s\n", out.c_str());
    }
    fflush(stdout);
    _exit(0);                                                    // no GPU: nothing of the runtime to take down
}
