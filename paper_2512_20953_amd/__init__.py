"""MI355X-native pipeline-stage compute (forward + backward of a run of decoder
layers on one tensor-parallel shard).  Thin ctypes binding over libahstage.so;
every step runs in the HIP kernels of that library."""
import importlib

_LAZY = ("AH_ARCH_GPT", "AH_ARCH_LLAMA", "AH_ARCH_BERT", "PARAM_INDEX", "AhError", "Stage", "StageConfig", "attention_bwd",
         "attention_fwd", "attention_bwd_static", "ATTENTION_STATIC_MAX_ROWS", "gemm_nn", "gemm_nn_swiglu", "gemm_nt", "gemm_plan", "gemm_tn", "gemm_tn_segmented", "lib", "library_path", "query_sizes", "cost_layers_time",
         "cost_pipeline_time", "cost_iteration_time", "cost_idle_fractions", "cost_partition_layers")


def __getattr__(name):
    # the binding loads libahstage.so on first use, so that importing the package
    # (to reach paper_2512_20953_amd.build) works before the library is built.  A name found is kept: the search costs
    # 3.5 us, as much as a small call spends in the library and the runtime (three products of 256 x 256 x 1024: 23.6 -> 15.6 us)
    if name in _LAZY:
        value = globals()[name] = getattr(importlib.import_module(__name__ + ".binding"), name)
        return value
    raise AttributeError(name)
