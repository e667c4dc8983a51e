"""MI355X-native GAS layer step: hand-written HIP kernels behind a C ABI
(include/gas.h), with a binding of the same names."""
from .binding import (  # noqa: F401
    F32, BF16, GasError, Plan, HostTable, DiskTable, lib, gas_version,
    gas_pull, gas_push, gas_gcn_norm, gas_plan_create, gas_plan_destroy, gas_validate_indices,
    gas_spmm, gas_spmm_hist, gas_spmm_table, gas_fuse_sources, gas_spmm_t, gas_spmm_t_relu,
    gas_linear, gas_linear_in_order, gas_mlp2, gas_linear_push, gas_mlp2_push, gas_mlp2_keep, gas_spmm_linear, gas_spmm_t_relu_linear, spmm_linear_supported,
    gas_spmm_linear_layers, gas_spmm_t_relu_linear_layers,
    gas_relu_bwd, gas_linear_bwd_input, gas_linear_bwd_input_add, gas_linear_bwd_weight, gas_linear_bwd_weight_workspace, gas_linear_bwd_weight_static, gas_linear_bwd_weights,
    gas_softmax_xent, gas_sgd_step, gas_sgd_steps, gas_sq_norm, gas_sgd_step_clipped, gas_axpy, gas_row_distance, gas_row_distance_bwd, gas_row_dot,
    gas_pna_aggregate, gas_gat_aggregate, gas_pna_aggregate_bwd, gas_gat_aggregate_bwd)
